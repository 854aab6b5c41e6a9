// mlp.hip -- learned warm start: features, a 3-layer FP32 MLP (8 -> 256 ->
// 256 -> 4) with hand-written forward / backward / Adam kernels on the fp32
// matrix cores (v_mfma_f32_16x16x4_f32), and the amplitude head.
//
// Per packed T2 element: u = MP2 amplitude, r = residual at u, D = its
// denominator, v = r / D (the next Jacobi correction), s = |u| + |v| + 1e-30;
// features x = (Re u/s, Im u/s, Re v/s, Im v/s, clip(ln((|v|+1e-30)/(|u|+1e-30)),
// -10, 10)/10, D/10, ln(s)/10, |v|/s); the network output y gives
// a = y0 + i y1, b = y2 + i y3 and the prediction t = u + v + a v + b u; the
// training loss is mean |t - t_converged|^2 / s^2 (relative) or
// sum |t - t_converged|^2 / sum s^2 (absolute).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "../../include/fscc.h"
#include "kernels.hpp"

namespace fscc {
namespace {

typedef float f4v __attribute__((ext_vector_type(4)));
constexpr int kT = 256;
constexpr int F_IN = 8, HID = 256, F_OUT = 4;
// flat parameter layout: W1 [8][256], b1, W2 [256][256], b2, W3 [256][4], b3
constexpr size_t OFF_W1 = 0, OFF_B1 = OFF_W1 + F_IN * HID, OFF_W2 = OFF_B1 + HID, OFF_B2 = OFF_W2 + HID * HID,
                 OFF_W3 = OFF_B2 + HID, OFF_B3 = OFF_W3 + HID * F_OUT, N_PARAMS = OFF_B3 + F_OUT;

// ---------------------------------------------------------------------------
// Network kernels.  One workgroup carries 16 * FM rows through whole layers:
// the activations (64 KB for 64 rows, two workgroups per CU) stay in LDS
// between the layers, and the weights (256 KB, resident in every L2) are read
// as MFMA fragments straight from memory one 16-deep k block ahead.  Four
// waves, each all rows x 64 columns: for 64 rows 16 accumulators, 64 MFMAs
// (2048 cycles) per k block against 4 LDS reads and 16 loads.
//
// LDS rows hold 64 chunks of four floats; chunk c of row r sits at c ^ (r & 15),
// so the 16 rows of a fragment read 16 different 16-byte bank groups.

// Row fragments per workgroup: 64-row tiles read the weights least often;
// fewer rows per workgroup where 64 (from 16384 rows down) or 32 (from 8192
// down) would leave CUs without a workgroup (a training step on 8192 rows:
// forward and backward 97 -> 52 us).  At the lines the forward launch takes
// 18.7 us for 8192 rows and 27.9 for 8193, 29.5 for 16384 and 43.2 for 16385.
int mlp_fm(long long rows) { return rows > 32 * 512 ? 4 : rows > 16 * 512 ? 2 : 1; }

__device__ __forceinline__ int lds_chunk(int row, int chunk) { return row * HID + ((chunk ^ (row & 15)) << 2); }

// Forward: Y = relu(relu(X W1 + b1) W2 + b2) W3 + b3 in one launch (STORE: the
// hidden activations go to h1, h2 for the backward pass).  Every output is one
// MFMA chain in ascending k, 4 at a time.  An activation column k is stored in
// chunk 4 (k / 16) + k % 4, element (k % 16) / 4: a lane's 16-byte read then
// holds its k of four consecutive MFMA steps.  Bound by the fp32 matrix cores
// (138 kflop a row, no activation leaves the CU): features, network and
// prediction of 600001 rows 1.88 -> 0.73 ms against one launch per layer with
// the activations in device memory.
template <int FM, bool STORE>
__global__ __launch_bounds__(256, 2) void k_mlp_fwd(const float* __restrict__ P, const float* __restrict__ X,
                                                 long long rows, float* __restrict__ h1, float* __restrict__ h2,
                                                 float* __restrict__ Y) {
    constexpr int kRows = 16 * FM;
    __shared__ float act[kRows * HID];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 15, lq = lane >> 4;
    const long long r0 = (long long)blockIdx.x * kRows;
    const int n0 = wave * 64;
    auto put = [&](int row, int col, float v) {
        act[lds_chunk(row, (col >> 4) * 4 + (col & 3)) + ((col & 15) >> 2)] = v;
    };
    {
        float a[FM][2], b[4][2];
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            const long long r = min(r0 + 16 * i + lr, rows - 1);
#pragma unroll
            for (int k = 0; k < 2; ++k) a[i][k] = X[r * F_IN + 4 * k + lq];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int k = 0; k < 2; ++k) b[j][k] = P[OFF_W1 + (4 * k + lq) * HID + n0 + 16 * j + lr];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int col = n0 + 16 * j + lr;
            const float bias = P[OFF_B1 + col];
#pragma unroll
            for (int i = 0; i < FM; ++i) {
                f4v c = f4v{0.f, 0.f, 0.f, 0.f};
                c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][0], b[j][0], c, 0, 0, 0);
                c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][1], b[j][1], c, 0, 0, 0);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int row = 16 * i + 4 * lq + q;
                    const float v = fmaxf(c[q] + bias, 0.f);
                    put(row, col, v);
                    if (STORE && r0 + row < rows) h1[(r0 + row) * HID + col] = v;
                }
            }
        }
    }
    f4v acc[FM][4];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f4v{0.f, 0.f, 0.f, 0.f};
    const float* W2 = P + OFF_W2 + lq * HID + n0 + lr;
    float b[4][4], bn[4][4];
    auto load_b = [&](float (&d)[4][4], int kb) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) d[j][k] = W2[(16 * kb + 4 * k) * HID + 16 * j];
    };
    auto block = [&](int kb, const float (&w)[4][4]) {
        f4v a[FM];
#pragma unroll
        for (int i = 0; i < FM; ++i) a[i] = *(const f4v*)&act[lds_chunk(16 * i + lr, 4 * kb + lq)];
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][k], w[j][k], acc[i][j], 0, 0, 0);
    };
    load_b(b, 0);
    __syncthreads();
    for (int kb = 0; kb < HID / 16; kb += 2) {
        load_b(bn, kb + 1);
        block(kb, b);
        load_b(b, min(kb + 2, HID / 16 - 1));
        block(kb + 1, bn);
    }
    __syncthreads();   // every wave has read the first layer's activations
    // the last layer's weights, under way during the epilogue (lanes past the
    // four outputs read in range and take zero)
    const uint32_t keep = lr < F_OUT ? 0xFFFFFFFFu : 0u;
    uint32_t w3[HID / 16][4];
    if (wave < FM)
#pragma unroll
        for (int kb = 0; kb < HID / 16; ++kb)
#pragma unroll
            for (int k = 0; k < 4; ++k)
                w3[kb][k] = ((const uint32_t*)P)[OFF_W3 + (16 * kb + 4 * k + lq) * F_OUT + (lr & 3)];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int col = n0 + 16 * j + lr;
        const float bias = P[OFF_B2 + col];
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int row = 16 * i + 4 * lq + q;
                const float v = fmaxf(acc[i][j][q] + bias, 0.f);
                put(row, col, v);
                if (STORE && r0 + row < rows) h2[(r0 + row) * HID + col] = v;
            }
    }
    __syncthreads();
    if (wave >= FM) return;
    // last layer: 16 rows per wave, the four outputs padded to one fragment
    f4v c = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < HID / 16; ++kb) {
        const f4v a = *(const f4v*)&act[lds_chunk(16 * wave + lr, 4 * kb + lq)];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[k], __uint_as_float(w3[kb][k] & keep), c, 0, 0, 0);
    }
    if (lr < F_OUT) {
        const float bias = P[OFF_B3 + lr];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const long long row = r0 + 16 * wave + 4 * lq + q;
            if (row < rows) Y[row * F_OUT + lr] = c[q] + bias;
        }
    }
}

// Backward through the hidden layers in one launch:
// dh2 = (dY W3^T) o (h2 > 0) into LDS and memory, dh1 = (dh2 W2^T) o (h1 > 0).
template <int FM>
__global__ __launch_bounds__(256, 2) void k_mlp_bwd(const float* __restrict__ P, const float* __restrict__ dY, int rows,
                                                 const float* __restrict__ h1, const float* __restrict__ h2,
                                                 float* __restrict__ dh1, float* __restrict__ dh2) {
    constexpr int kRows = 16 * FM;
    __shared__ float act[kRows * HID];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 15, lq = lane >> 4;
    const long long r0 = (long long)blockIdx.x * kRows;
    {
        const f4v w = *(const f4v*)&P[OFF_W3 + tid * F_OUT];
#pragma unroll 8
        for (int r = 0; r < kRows; ++r) {
            const long long row = min(r0 + r, (long long)rows - 1);
            const f4v d = *(const f4v*)&dY[row * F_OUT];
            float v = d[0] * w[0] + d[1] * w[1] + d[2] * w[2] + d[3] * w[3];
            v = h2[row * HID + tid] > 0.f ? v : 0.f;
            act[lds_chunk(r, tid >> 2) + (tid & 3)] = v;
            if (r0 + r < rows) dh2[row * HID + tid] = v;
        }
    }
    f4v acc[FM][4];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f4v{0.f, 0.f, 0.f, 0.f};
    const int n0 = wave * 64;
    const float* W2 = P + OFF_W2 + (n0 + lr) * HID + 4 * lq;   // row n of W2: k contiguous
    f4v b[4], bn[4];
    auto load_b = [&](f4v (&d)[4], int kb) {
#pragma unroll
        for (int j = 0; j < 4; ++j) d[j] = *(const f4v*)&W2[16 * j * HID + 16 * kb];
    };
    auto block = [&](int kb, const f4v (&w)[4]) {
        f4v a[FM];
#pragma unroll
        for (int i = 0; i < FM; ++i) a[i] = *(const f4v*)&act[lds_chunk(16 * i + lr, 4 * kb + lq)];
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][k], w[j][k], acc[i][j], 0, 0, 0);
    };
    load_b(b, 0);
    __syncthreads();
    for (int kb = 0; kb < HID / 16; kb += 2) {
        load_b(bn, kb + 1);
        block(kb, b);
        load_b(b, min(kb + 2, HID / 16 - 1));
        block(kb + 1, bn);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int col = n0 + 16 * j + lr;
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const long long row = r0 + 16 * i + 4 * lq + q;
                if (row < rows) dh1[row * HID + col] = h1[row * HID + col] > 0.f ? acc[i][j][q] : 0.f;
            }
    }
}

// Parameter gradients, split along the rows: gW2 = h1^T dh2, gW1 = X^T dh1,
// gW3 = h2^T dY and the column sums gb2, gb1, gb3 of one row chunk, written to
// part[chunk] in the layout of the parameter vector.  blockIdx.x: 16 64 x 64
// tiles of gW2, 4 column tiles of gW1, 4 row tiles of gW3; blockIdx.y: chunk.
// Bound by launch and load latency at these sizes: 128 rows per chunk give 1536
// workgroups for a minibatch of 8192.  (With the rows unsplit, 16 and 4
// workgroups walked all of them: 3.4 ms of a 3.75 ms training step on 8192
// rows; the whole step now takes 0.14 ms.)  A column sum adds the sums of its
// 32-row slices, so its longest chain of roundings is 32 + n / 2048 + 64 for n
// rows (in one running sum it would be n / 64 + 64, which costs two digits at
// half a million rows).
constexpr int kGradTiles = 24, kGradBK = 32, kMaxChunks = 64;
__global__ __launch_bounds__(256) void k_mlp_wgrad(const float* __restrict__ X, const float* __restrict__ h1,
                                                   const float* __restrict__ h2, const float* __restrict__ dh1,
                                                   const float* __restrict__ dh2, const float* __restrict__ dY,
                                                   int rows, int rows_per, float* __restrict__ part) {
    constexpr int LD = 80;   // four k rows of a fragment start 16 banks apart
    __shared__ float As[kGradBK * LD];
    __shared__ float Bs[kGradBK * LD];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 15, lq = lane >> 4;
    const int t = blockIdx.x;
    const float *A, *B;
    int MA, NB, m0, n0;
    size_t off, boff;
    if (t < 16) {
        A = h1, B = dh2, MA = HID, NB = HID, m0 = (t >> 2) * 64, n0 = (t & 3) * 64, off = OFF_W2, boff = OFF_B2;
    } else if (t < 20) {
        A = X, B = dh1, MA = F_IN, NB = HID, m0 = 0, n0 = (t - 16) * 64, off = OFF_W1, boff = OFF_B1;
    } else {
        A = h2, B = dY, MA = HID, NB = F_OUT, m0 = (t - 20) * 64, n0 = 0, off = OFF_W3, boff = OFF_B3;
    }
    const int k_lo = blockIdx.y * rows_per, k_hi = min(rows, k_lo + rows_per);
    f4v ra[2], rb[2];
    // 32 rows x 16 chunks of four floats per operand, two per thread
    auto fetch = [&](int k0) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int k = k0 + (tid >> 4) + 16 * u, c = (tid & 15) * 4;
            const bool in = k < k_hi;
            ra[u] = rb[u] = f4v{0.f, 0.f, 0.f, 0.f};
            if (in && m0 + c < MA) ra[u] = *(const f4v*)&A[(long long)k * MA + m0 + c];
            if (in && n0 + c < NB) rb[u] = *(const f4v*)&B[(long long)k * NB + n0 + c];
        }
    };
    f4v acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f4v{0.f, 0.f, 0.f, 0.f};
    const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
    float bsum = 0.f;
    if (k_lo < k_hi) fetch(k_lo);
    for (int k0 = k_lo; k0 < k_hi; k0 += kGradBK) {
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int at = ((tid >> 4) + 16 * u) * LD + (tid & 15) * 4;
            *(f4v*)&As[at] = ra[u];
            *(f4v*)&Bs[at] = rb[u];
        }
        __syncthreads();
        if (k0 + kGradBK < k_hi) fetch(k0 + kGradBK);
        if (m0 == 0 && tid < 64) {
            float s = 0.f;
#pragma unroll 8
            for (int k = 0; k < kGradBK; ++k) s += Bs[k * LD + tid];
            bsum += s;
        }
#pragma unroll
        for (int k = 0; k < kGradBK; k += 4) {
            float a[2], b[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                a[i] = As[(k + lq) * LD + wm + 16 * i + lr];
                b[i] = Bs[(k + lq) * LD + wn + 16 * i + lr];
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[j], acc[i][j], 0, 0, 0);
        }
    }
    float* G = part + (size_t)blockIdx.y * N_PARAMS;
    if (m0 == 0 && tid < 64 && n0 + tid < NB) G[boff + n0 + tid] = bsum;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int col = n0 + wn + 16 * j + lr;
            if (col >= NB) continue;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int row = m0 + wm + 16 * i + 4 * lq + q;
                if (row < MA) G[off + (size_t)row * NB + col] = acc[i][j][q];
            }
        }
}

// gradient = sum of the chunks' parts in chunk order; block 0 also finishes
// the loss (its block partials are already weighted) into host memory
__global__ __launch_bounds__(256) void k_mlp_gsum(const float* __restrict__ part, int nchunk, float* __restrict__ g,
                                                  const double* __restrict__ lpart, int nl, double* __restrict__ loss) {
    const int k = blockIdx.x * kT + threadIdx.x;
    if (k < (int)N_PARAMS) {
        float s = 0.f;
#pragma unroll 8
        for (int c = 0; c < nchunk; ++c) s += part[(size_t)c * N_PARAMS + k];
        g[k] = s;
    }
    if (blockIdx.x == 0) {
        __shared__ double sh[kT];
        double v = 0.0;
        for (int b = threadIdx.x; b < nl; b += kT) v += lpart[b];
        sh[threadIdx.x] = v;
        __syncthreads();
        for (int s2 = kT / 2; s2 > 0; s2 >>= 1) {
            if ((int)threadIdx.x < s2) sh[threadIdx.x] += sh[threadIdx.x + s2];
            __syncthreads();
        }
        if (threadIdx.x == 0) *loss = sh[0];
    }
}

__device__ inline void ws_v_s(double2 u, double2 r, double d, double2* v, double* s) {
    *v = make_double2(r.x / d, r.y / d);
    *s = hypot(u.x, u.y) + hypot(v->x, v->y) + 1e-30;
}

// the eight features of one row; returns s
__device__ inline double ws_row(double2 uu, double2 rr, double d, float* __restrict__ x) {
    double2 v;
    double s;
    ws_v_s(uu, rr, d, &v, &s);
    const double au = hypot(uu.x, uu.y), av = hypot(v.x, v.y);
    const double lr = fmin(fmax(log((av + 1e-30) / (au + 1e-30)), -10.0), 10.0);
    x[0] = (float)(uu.x / s);
    x[1] = (float)(uu.y / s);
    x[2] = (float)(v.x / s);
    x[3] = (float)(v.y / s);
    x[4] = (float)(lr / 10.0);
    x[5] = (float)(d / 10.0);
    x[6] = (float)(log(s) / 10.0);
    x[7] = (float)(av / s);
    return s;
}

__global__ __launch_bounds__(256) void k_ws_features(const double2* __restrict__ u, const double2* __restrict__ r,
                                                     const double* __restrict__ D, long long n, float* __restrict__ X) {
    const long long k = (long long)blockIdx.x * kT + threadIdx.x;
    if (k >= n) return;
    ws_row(u[k], r[k], D[k], X + k * F_IN);
}

// Training rows idx[0..n) (idx null: 0..n-1) copied to the staging arrays with
// their features, and per-block partial sums of s^2 (the absolute loss
// normaliser).
__global__ __launch_bounds__(256) void k_ws_stage(const double2* __restrict__ u, const double2* __restrict__ r,
                                                  const double* __restrict__ D, const double2* __restrict__ t,
                                                  const long long* __restrict__ idx, long long n,
                                                  double2* __restrict__ bu, double2* __restrict__ br,
                                                  double* __restrict__ bD, double2* __restrict__ bt,
                                                  float* __restrict__ X, double* __restrict__ part) {
    __shared__ double sh[kT];
    double q = 0.0;
    for (long long k = (long long)blockIdx.x * kT + threadIdx.x; k < n; k += (long long)gridDim.x * kT) {
        const long long i = idx ? idx[k] : k;
        const double2 uu = u[i], rr = r[i], tt = t[i];
        const double d = D[i];
        bu[k] = uu;
        br[k] = rr;
        bD[k] = d;
        bt[k] = tt;
        const double s = ws_row(uu, rr, d, X + k * F_IN);
        q += s * s;
    }
    sh[threadIdx.x] = q;
    __syncthreads();
    for (int s2 = kT / 2; s2 > 0; s2 >>= 1) {
        if ((int)threadIdx.x < s2) sh[threadIdx.x] += sh[threadIdx.x + s2];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

// prediction u + v + a v + b u  (Y may be null: a = b = 0)
__global__ __launch_bounds__(256) void k_ws_apply(const float* __restrict__ Y, const double2* __restrict__ u,
                                                  const double2* __restrict__ r, const double* __restrict__ D,
                                                  long long n, double2* __restrict__ out) {
    const long long k = (long long)blockIdx.x * kT + threadIdx.x;
    if (k >= n) return;
    const double2 uu = u[k];
    double2 v;
    double s;
    ws_v_s(uu, r[k], D[k], &v, &s);
    double ar = 0, ai = 0, br = 0, bi = 0;
    if (Y) {
        ar = Y[k * F_OUT];
        ai = Y[k * F_OUT + 1];
        br = Y[k * F_OUT + 2];
        bi = Y[k * F_OUT + 3];
    }
    out[k] = make_double2(uu.x + v.x + (ar * v.x - ai * v.y) + (br * uu.x - bi * uu.y),
                          uu.y + v.y + (ar * v.y + ai * v.x) + (br * uu.y + bi * uu.x));
}

// loss rows and dL/dy; weight w_k = 1/(n s_k^2) (mode 0) or 1/sum s^2 (mode 1,
// every block adds the np partial sums); per-block loss partials (already
// weighted)
__global__ __launch_bounds__(256) void k_ws_head(const float* __restrict__ Y, const double2* __restrict__ u,
                                                 const double2* __restrict__ r, const double* __restrict__ D,
                                                 const double2* __restrict__ t, long long n, int mode,
                                                 const double* __restrict__ spart, int np, float* __restrict__ dY,
                                                 double* __restrict__ part) {
    __shared__ double sh[kT];
    auto block_sum = [&](double v) {
        sh[threadIdx.x] = v;
        __syncthreads();
        for (int s2 = kT / 2; s2 > 0; s2 >>= 1) {
            if ((int)threadIdx.x < s2) sh[threadIdx.x] += sh[threadIdx.x + s2];
            __syncthreads();
        }
        const double x = sh[0];
        __syncthreads();
        return x;
    };
    double norm = 1.0;
    if (mode == 1) {
        double q = 0.0;
        for (int b = threadIdx.x; b < np; b += kT) q += spart[b];
        norm = block_sum(q);
    }
    double l = 0.0;
    for (long long k = (long long)blockIdx.x * kT + threadIdx.x; k < n; k += (long long)gridDim.x * kT) {
        const double2 uu = u[k];
        double2 v;
        double s;
        ws_v_s(uu, r[k], D[k], &v, &s);
        const double ar = Y[k * F_OUT], ai = Y[k * F_OUT + 1], br = Y[k * F_OUT + 2], bi = Y[k * F_OUT + 3];
        const double2 tt = t[k];
        const double er = uu.x + v.x + (ar * v.x - ai * v.y) + (br * uu.x - bi * uu.y) - tt.x;
        const double ei = uu.y + v.y + (ar * v.y + ai * v.x) + (br * uu.y + bi * uu.x) - tt.y;
        const double w = mode == 0 ? 1.0 / (s * s) / (double)n : 1.0 / norm;
        l += (er * er + ei * ei) * w;
        const double f = 2.0 * w;
        // conj(e) * v = (er v.x + ei v.y) + i (er v.y - ei v.x)
        dY[k * F_OUT] = (float)(f * (er * v.x + ei * v.y));
        dY[k * F_OUT + 1] = (float)(-f * (er * v.y - ei * v.x));
        dY[k * F_OUT + 2] = (float)(f * (er * uu.x + ei * uu.y));
        dY[k * F_OUT + 3] = (float)(-f * (er * uu.y - ei * uu.x));
    }
    l = block_sum(l);
    if (threadIdx.x == 0) part[blockIdx.x] = l;
}

__global__ __launch_bounds__(256) void k_adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                                              float* __restrict__ w, long long n, float lr, float b1, float b2,
                                              float eps, float bc1, float bc2) {
    const long long k = (long long)blockIdx.x * kT + threadIdx.x;
    if (k >= n) return;
    const float gg = g[k];
    const float mm = b1 * m[k] + (1.f - b1) * gg;
    const float ww = b2 * w[k] + (1.f - b2) * gg * gg;
    m[k] = mm;
    w[k] = ww;
    p[k] -= lr * (mm / bc1) / (sqrtf(ww / bc2) + eps);
}

__global__ __launch_bounds__(256) void k_gather_rows(const unsigned char* __restrict__ src, int eb,
                                                     const long long* __restrict__ idx, long long n,
                                                     unsigned char* __restrict__ dst) {
    const long long k = (long long)blockIdx.x * kT + threadIdx.x;
    if (k >= n) return;
    const long long i = idx[k];
    if (eb == 16) ((double2*)dst)[k] = ((const double2*)src)[i];
    else ((double*)dst)[k] = ((const double*)src)[i];
}

__global__ __launch_bounds__(256) void k_ws_step(const double2* __restrict__ t, const double2* __restrict__ r,
                                                 const double* __restrict__ D, long long n, double2* __restrict__ out) {
    const long long k = (long long)blockIdx.x * kT + threadIdx.x;
    if (k >= n) return;
    const double d = D[k];
    const double2 tt = t ? t[k] : make_double2(0.0, 0.0), rr = r[k];
    out[k] = make_double2(tt.x + rr.x / d, tt.y + rr.y / d);
}

template <bool STORE>
void launch_fwd(const float* P, const float* X, long long rows, float* h1, float* h2, float* Y, hipStream_t st) {
    const int fm = mlp_fm(rows);
    const unsigned nt = (unsigned)((rows + 16 * fm - 1) / (16 * fm));
    if (fm == 4) k_mlp_fwd<4, STORE><<<nt, kT, 0, st>>>(P, X, rows, h1, h2, Y);
    else if (fm == 2) k_mlp_fwd<2, STORE><<<nt, kT, 0, st>>>(P, X, rows, h1, h2, Y);
    else k_mlp_fwd<1, STORE><<<nt, kT, 0, st>>>(P, X, rows, h1, h2, Y);
}

unsigned grid1(long long n) { return (unsigned)((n + kT - 1) / kT); }

}  // namespace
}  // namespace fscc

using namespace fscc;

struct fscc_mlp {
    hipStream_t st = nullptr;
    float *p = nullptr, *g = nullptr, *m = nullptr, *w = nullptr;
    long long step = 0;
    // training scratch (rows <= maxb)
    size_t maxb = 0;
    float *X = nullptr, *h1 = nullptr, *h2 = nullptr, *dh1 = nullptr, *dh2 = nullptr, *Y = nullptr, *dY = nullptr,
          *gpart = nullptr;
    double *spart = nullptr, *lpart = nullptr, *bD = nullptr;
    double2 *bu = nullptr, *br = nullptr, *bt = nullptr;
    float* yhold = nullptr;   // outputs of a chunk of rows that replace its inputs
    double* hloss = nullptr;
    std::string err;

    void free_train() {
        void* ps[] = {X, h1, h2, dh1, dh2, Y, dY, gpart, spart, lpart, bD, bu, br, bt};
        for (void* q : ps)
            if (q) (void)hipFree(q);
        X = h1 = h2 = dh1 = dh2 = Y = dY = gpart = nullptr;
        spart = lpart = bD = nullptr;
        bu = br = bt = nullptr;
        maxb = 0;
    }
    ~fscc_mlp() {
        if (st) (void)hipStreamSynchronize(st);
        else (void)hipDeviceSynchronize();
        free_train();
        void* ps[] = {p, g, m, w, yhold};
        for (void* q : ps)
            if (q) (void)hipFree(q);
        if (hloss) (void)hipHostFree(hloss);
    }
};

namespace {

bool ok(hipError_t e) { return e == hipSuccess; }

fscc_status herr(fscc_mlp* n, hipError_t e, const char* what) {
    if (n) n->err = std::string(what) + ": " + hipGetErrorString(e);
    return FSCC_EHIP;
}

template <class T>
hipError_t dalloc(T** q, size_t count) {
    return hipMalloc((void**)q, sizeof(T) * (count ? count : 1));
}

// blocks of the staging and loss launches (each loss block adds the partial
// sums of every staging block)
constexpr unsigned kStageBlocks = 512;

hipError_t ensure_train(fscc_mlp* n, size_t rows) {
    if (rows <= n->maxb) return hipSuccess;
    n->free_train();
    size_t b = 1024;
    while (b < rows) b *= 2;
    hipError_t e = hipSuccess;
    if (ok(e)) e = dalloc(&n->X, b * F_IN);
    if (ok(e)) e = dalloc(&n->h1, b * HID);
    if (ok(e)) e = dalloc(&n->h2, b * HID);
    if (ok(e)) e = dalloc(&n->dh1, b * HID);
    if (ok(e)) e = dalloc(&n->dh2, b * HID);
    if (ok(e)) e = dalloc(&n->Y, b * F_OUT);
    if (ok(e)) e = dalloc(&n->dY, b * F_OUT);
    if (ok(e)) e = dalloc(&n->gpart, (size_t)kMaxChunks * N_PARAMS);
    if (ok(e)) e = dalloc(&n->spart, kStageBlocks);
    if (ok(e)) e = dalloc(&n->lpart, kStageBlocks);
    if (ok(e)) e = dalloc(&n->bD, b);
    if (ok(e)) e = dalloc(&n->bu, b);
    if (ok(e)) e = dalloc(&n->br, b);
    if (ok(e)) e = dalloc(&n->bt, b);
    if (ok(e)) n->maxb = b;
    return e;
}

// forward + loss + backward on the rows idx[0..rows) -> n->g, *n->hloss
hipError_t loss_grad_rows(fscc_mlp* n, const double2* u, const double2* r, const double* D, const double2* t,
                          const long long* idx, size_t rows, int mode) {
    const int M = (int)rows;
    const float* P = n->p;
    hipStream_t st = n->st;
    const unsigned nb = std::min(grid1(M), kStageBlocks);
    k_ws_stage<<<nb, kT, 0, st>>>(u, r, D, t, idx, M, n->bu, n->br, n->bD, n->bt, n->X, n->spart);
    launch_fwd<true>(P, n->X, M, n->h1, n->h2, n->Y, st);
    k_ws_head<<<nb, kT, 0, st>>>(n->Y, n->bu, n->br, n->bD, n->bt, M, mode, n->spart, (int)nb, n->dY, n->lpart);
    const int fm = mlp_fm(M);
    const unsigned nt = (unsigned)((M + 16 * fm - 1) / (16 * fm));
    if (fm == 4) k_mlp_bwd<4><<<nt, kT, 0, st>>>(P, n->dY, M, n->h1, n->h2, n->dh1, n->dh2);
    else if (fm == 2) k_mlp_bwd<2><<<nt, kT, 0, st>>>(P, n->dY, M, n->h1, n->h2, n->dh1, n->dh2);
    else k_mlp_bwd<1><<<nt, kT, 0, st>>>(P, n->dY, M, n->h1, n->h2, n->dh1, n->dh2);
    // row chunks of at least 128 rows (four k blocks), at most kMaxChunks
    int per = std::max(128, (M + kMaxChunks - 1) / kMaxChunks);
    per = (per + kGradBK - 1) / kGradBK * kGradBK;
    const int nc = (M + per - 1) / per;
    k_mlp_wgrad<<<dim3(kGradTiles, nc), kT, 0, st>>>(n->X, n->h1, n->h2, n->dh1, n->dh2, n->dY, M, per, n->gpart);
    k_mlp_gsum<<<grid1(N_PARAMS), kT, 0, st>>>(n->gpart, nc, n->g, n->lpart, (int)nb, n->hloss);
    return hipGetLastError();
}

hipError_t adam(fscc_mlp* n, float lr) {
    n->step += 1;
    const float b1 = 0.9f, b2 = 0.999f;
    const float bc1 = (float)(1.0 - std::pow(0.9, (double)n->step));
    const float bc2 = (float)(1.0 - std::pow(0.999, (double)n->step));
    k_adam<<<grid1(N_PARAMS), kT, 0, n->st>>>(n->p, n->g, n->m, n->w, (long long)N_PARAMS, lr, b1, b2, 1e-8f, bc1,
                                             bc2);
    return hipGetLastError();
}

// SplitMix64 (Steele, Lea, Flood 2014) + Box-Muller for the initial weights
struct InitRng {
    uint64_t s;
    uint64_t next() {
        uint64_t z = (s += 0x9E3779B97F4A7C15ULL);
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
        return z ^ (z >> 31);
    }
    double normal() {
        const double u1 = ((double)(next() >> 11) + 1.0) * 0x1.0p-53, u2 = (double)(next() >> 11) * 0x1.0p-53;
        return std::sqrt(-2.0 * std::log(u1)) * std::cos(6.283185307179586 * u2);
    }
};

}  // namespace

extern "C" {

fscc_status fscc_mlp_num_params(size_t* n) {
    if (!n) return FSCC_EINVAL;
    *n = N_PARAMS;
    return FSCC_OK;
}

fscc_status fscc_mlp_create(uint64_t seed, void* hip_stream, fscc_mlp** out) {
    if (!out) return FSCC_EINVAL;
    *out = nullptr;
    fscc_mlp* n = new (std::nothrow) fscc_mlp();
    if (!n) return FSCC_ENOMEM;
    n->st = (hipStream_t)hip_stream;
    hipError_t e = dalloc(&n->p, N_PARAMS);
    if (ok(e)) e = dalloc(&n->g, N_PARAMS);
    if (ok(e)) e = dalloc(&n->m, N_PARAMS);
    if (ok(e)) e = dalloc(&n->w, N_PARAMS);
    if (ok(e)) e = hipHostMalloc((void**)&n->hloss, sizeof(double), hipHostMallocDefault);
    if (ok(e)) {
        std::vector<float> h(N_PARAMS, 0.f);
        InitRng r{seed};
        const double s1 = std::sqrt(2.0 / F_IN), s2 = std::sqrt(2.0 / HID);
        for (size_t k = 0; k < (size_t)F_IN * HID; ++k) h[OFF_W1 + k] = (float)(s1 * r.normal());
        for (size_t k = 0; k < (size_t)HID * HID; ++k) h[OFF_W2 + k] = (float)(s2 * r.normal());
        std::vector<float> z(N_PARAMS, 0.f);
        e = hipMemcpy(n->p, h.data(), sizeof(float) * N_PARAMS, hipMemcpyHostToDevice);
        if (ok(e)) e = hipMemcpy(n->m, z.data(), sizeof(float) * N_PARAMS, hipMemcpyHostToDevice);
        if (ok(e)) e = hipMemcpy(n->w, z.data(), sizeof(float) * N_PARAMS, hipMemcpyHostToDevice);
        if (ok(e)) e = hipMemcpy(n->g, z.data(), sizeof(float) * N_PARAMS, hipMemcpyHostToDevice);
    }
    if (!ok(e)) {
        delete n;
        return e == hipErrorOutOfMemory ? FSCC_ENOMEM : FSCC_EHIP;
    }
    *out = n;
    return FSCC_OK;
}

void fscc_mlp_destroy(fscc_mlp* n) { delete n; }

const char* fscc_mlp_last_error(const fscc_mlp* n) { return n ? n->err.c_str() : "null network"; }

fscc_status fscc_mlp_set_params(fscc_mlp* n, const float* host, size_t count) {
    if (!n || !host || count != N_PARAMS) return FSCC_EINVAL;
    std::vector<float> z(N_PARAMS, 0.f);
    hipError_t e = hipMemcpy(n->p, host, sizeof(float) * N_PARAMS, hipMemcpyHostToDevice);
    if (ok(e)) e = hipMemcpy(n->m, z.data(), sizeof(float) * N_PARAMS, hipMemcpyHostToDevice);
    if (ok(e)) e = hipMemcpy(n->w, z.data(), sizeof(float) * N_PARAMS, hipMemcpyHostToDevice);
    n->step = 0;
    return ok(e) ? FSCC_OK : herr(n, e, "set params");
}

fscc_status fscc_mlp_get_params(fscc_mlp* n, float* host, size_t count) {
    if (!n || !host || count != N_PARAMS) return FSCC_EINVAL;
    hipError_t e = hipStreamSynchronize(n->st);
    if (ok(e)) e = hipMemcpy(host, n->p, sizeof(float) * N_PARAMS, hipMemcpyDeviceToHost);
    return ok(e) ? FSCC_OK : herr(n, e, "get params");
}

fscc_status fscc_mlp_get_grad(fscc_mlp* n, float* host, size_t count) {
    if (!n || !host || count != N_PARAMS) return FSCC_EINVAL;
    hipError_t e = hipStreamSynchronize(n->st);
    if (ok(e)) e = hipMemcpy(host, n->g, sizeof(float) * N_PARAMS, hipMemcpyDeviceToHost);
    return ok(e) ? FSCC_OK : herr(n, e, "get grad");
}

fscc_status fscc_ws_features(const fscc_c128* u, const fscc_c128* r, const double* D, size_t n, float* X,
                             void* hip_stream) {
    if (n && (!u || !r || !D || !X)) return FSCC_EINVAL;
    if (!n) return FSCC_OK;
    k_ws_features<<<grid1((long long)n), kT, 0, (hipStream_t)hip_stream>>>((const double2*)u, (const double2*)r, D,
                                                                           (long long)n, X);
    return ok(hipGetLastError()) ? FSCC_OK : FSCC_EHIP;
}

fscc_status fscc_ws_apply(const float* Y, const fscc_c128* u, const fscc_c128* r, const double* D, size_t n,
                          fscc_c128* out, void* hip_stream) {
    if (n && (!u || !r || !D || !out)) return FSCC_EINVAL;
    if (!n) return FSCC_OK;
    k_ws_apply<<<grid1((long long)n), kT, 0, (hipStream_t)hip_stream>>>(Y, (const double2*)u, (const double2*)r, D,
                                                                        (long long)n, (double2*)out);
    return ok(hipGetLastError()) ? FSCC_OK : FSCC_EHIP;
}

fscc_status fscc_ws_step(const fscc_c128* t, const fscc_c128* r, const double* D, size_t n, fscc_c128* out,
                         void* hip_stream) {
    if (n && (!r || !D || !out)) return FSCC_EINVAL;
    if (!n) return FSCC_OK;
    k_ws_step<<<grid1((long long)n), kT, 0, (hipStream_t)hip_stream>>>((const double2*)t, (const double2*)r, D,
                                                                       (long long)n, (double2*)out);
    return ok(hipGetLastError()) ? FSCC_OK : FSCC_EHIP;
}

fscc_status fscc_ws_gather(const void* src, size_t elem_bytes, const int64_t* idx, size_t n, void* dst,
                           void* hip_stream) {
    if ((elem_bytes != 8 && elem_bytes != 16) || (n && (!src || !idx || !dst))) return FSCC_EINVAL;
    if (!n) return FSCC_OK;
    k_gather_rows<<<grid1((long long)n), kT, 0, (hipStream_t)hip_stream>>>(
        (const unsigned char*)src, (int)elem_bytes, (const long long*)idx, (long long)n, (unsigned char*)dst);
    return ok(hipGetLastError()) ? FSCC_OK : FSCC_EHIP;
}

fscc_status fscc_mlp_forward(fscc_mlp* n, const float* X, size_t rows, float* Y) {
    if (!n || (rows && (!X || !Y))) return FSCC_EINVAL;
    if (!rows) return FSCC_OK;
    hipError_t e = hipSuccess;
    if (X < Y + rows * F_OUT && Y < X + rows * F_IN) {
        // Y over X: the workgroups of a launch read and write rows of each
        // other's, so the outputs of 2^20 rows at a time wait in a buffer
        // until the chunk's inputs have been read
        const size_t ch = (size_t)1 << 20;
        if (!n->yhold) e = dalloc(&n->yhold, ch * F_OUT);
        for (size_t r0 = 0; r0 < rows && ok(e); r0 += ch) {
            const size_t m = std::min(rows - r0, ch);
            launch_fwd<false>(n->p, X + r0 * F_IN, (long long)m, nullptr, nullptr, n->yhold, n->st);
            e = hipGetLastError();
            if (ok(e))
                e = hipMemcpyAsync(Y + r0 * F_OUT, n->yhold, m * F_OUT * sizeof(float), hipMemcpyDeviceToDevice, n->st);
        }
        return ok(e) ? FSCC_OK : herr(n, e, "forward");
    }
    // grids of at most 2^30 rows
    for (size_t r0 = 0; r0 < rows && ok(e); r0 += (size_t)1 << 30) {
        const size_t m = std::min(rows - r0, (size_t)1 << 30);
        launch_fwd<false>(n->p, X + r0 * F_IN, (long long)m, nullptr, nullptr, Y + r0 * F_OUT, n->st);
        e = hipGetLastError();
    }
    return ok(e) ? FSCC_OK : herr(n, e, "forward");
}

fscc_status fscc_mlp_loss_grad(fscc_mlp* n, const fscc_c128* u, const fscc_c128* r, const double* D,
                               const fscc_c128* t, const int64_t* idx, size_t rows, int mode, double* loss) {
    if (!n || !loss || rows == 0 || !u || !r || !D || !t || rows > (size_t)1 << 24 || mode < 0 || mode > 1)
        return FSCC_EINVAL;
    hipError_t e = ensure_train(n, rows);
    if (!ok(e)) return herr(n, e, "training scratch");
    e = loss_grad_rows(n, (const double2*)u, (const double2*)r, D, (const double2*)t, (const long long*)idx, rows, mode);
    if (ok(e)) e = hipStreamSynchronize(n->st);
    if (!ok(e)) return herr(n, e, "loss/grad");
    *loss = *n->hloss;
    return FSCC_OK;
}

fscc_status fscc_mlp_adam(fscc_mlp* n, float lr) {
    if (!n || !(lr > 0.f)) return FSCC_EINVAL;
    hipError_t e = adam(n, lr);
    return ok(e) ? FSCC_OK : herr(n, e, "adam");
}

}  // extern "C"
