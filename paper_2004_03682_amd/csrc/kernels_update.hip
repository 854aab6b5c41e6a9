// kernels_update.hip -- the amplitude update of Eq. (3) and the correlation
// energy: Jacobi step, DIIS subspace, extrapolation, for one system (complex
// or real arithmetic) and for a batch of systems.
//
// One system takes four launches: k_step (Jacobi step of T1 and T2, its
// largest element and its dot products with the stored steps in one pass over
// the vectors), k_finish (bordered solve), k_extrapolate and k_energy.  The
// results the host needs go straight to pinned host memory.  Up to a few
// hundred thousand amplitudes the sequence is bound by its launches: against
// thirteen launches with a one-thread solve and two copies an iteration of 8
// occupied and 24 virtual spinors went from 656 to 601 us (k_finish 47 -> 12 us
// at eight vectors).  Reductions are
// deterministic: fixed grid, per-block partials added in a fixed order.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "kernels.hpp"

namespace fscc {

int reduce_blocks(long long n) {
    long long b = (n + 255) / 256;
    if (b < 1) b = 1;
    if (b > kReduceBlocks) b = kReduceBlocks;
    return (int)b;
}

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;

__device__ __forceinline__ double block_sum(double v, double* sh) {
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int s = kThreads / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    double r = sh[0];
    __syncthreads();
    return r;
}

__device__ __forceinline__ double nan_max(double a, double b) { return (a > b || a != a) ? a : b; }   // NaN propagates

__device__ __forceinline__ double block_max(double v, double* sh) {
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int s = kThreads / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) sh[threadIdx.x] = nan_max(sh[threadIdx.x], sh[threadIdx.x + s]);
        __syncthreads();
    }
    double r = sh[0];
    __syncthreads();
    return r;
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d);
    return v;
}

__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v = nan_max(v, __shfl_xor(v, d));
    return v;
}

// value of lane p (uniform) in every lane
__device__ __forceinline__ double lane_value(double v, int p) {
    union {
        double d;
        int i[2];
    } u;
    u.d = v;
    u.i[0] = __builtin_amdgcn_readlane(u.i[0], p);
    u.i[1] = __builtin_amdgcn_readlane(u.i[1], p);
    return u.d;
}

// ---- the element types: complex (double2) and real (double)
__device__ __forceinline__ double re_dot(double2 x, double2 y) { return x.x * y.x + x.y * y.y; }
__device__ __forceinline__ double re_dot(double x, double y) { return x * y; }
__device__ __forceinline__ double2 over(double2 x, double d) { return make_double2(x.x / d, x.y / d); }
__device__ __forceinline__ double over(double x, double d) { return x / d; }
__device__ __forceinline__ double2 axpy(double a, double2 x, double2 y) { return make_double2(y.x + a * x.x, y.y + a * x.y); }
__device__ __forceinline__ double axpy(double a, double x, double y) { return y + a * x; }
__device__ __forceinline__ double size(double2 x) { return sqrt(x.x * x.x + x.y * x.y); }
__device__ __forceinline__ double size(double x) { return fabs(x); }
__device__ __forceinline__ double2 times(double2 a, double2 b) { return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); }
__device__ __forceinline__ double times(double a, double b) { return a * b; }
__device__ __forceinline__ double re(double2 x) { return x.x; }
__device__ __forceinline__ double re(double x) { return x; }
__device__ __forceinline__ double im(double2 x) { return x.y; }
__device__ __forceinline__ double im(double) { return 0.0; }

// Dynamic denominator shift of one amplitude (sector shift S < 0, exponent
// n >= 1): Delta = S (S / (min(D, 0) + S))^n; the shifted equations are
// R = Delta t, solved by the step (R - Delta t) / (D + Delta).
__device__ __forceinline__ double dyn_delta(double d, double S, int n) {
    const double q = S / (fmin(d, 0.0) + S);
    double p = q;
    for (int i = 1; i < n; ++i) p *= q;
    return S * p;
}

// Jacobi step of every amplitude (T1 then T2) into history slot `slot`, with
// the block's largest |step| and the dot products Re <e_j, e> with the m - 1
// stored steps ord[0..m-1) and with itself: part[j * gridDim.x + block], the
// maximum in row m.  Bound by memory: 72 + 16 (m - 1) bytes per complex
// amplitude, each read or written once (a step pass and a dot pass read the
// new step twice and took three launches).
template <typename T>
__global__ __launch_bounds__(256) void k_step(const T* __restrict__ t1, const T* __restrict__ r1,
                                              const double* __restrict__ D1, const T* __restrict__ t2,
                                              const T* __restrict__ r2, const double* __restrict__ D2,
                                              T* __restrict__ ht, T* __restrict__ he, long long n1, long long n,
                                              int slot, int m, DiisOrder ord, double* __restrict__ part,
                                              double shift, double dS, int dn) {
    __shared__ double sh[kDiisMax + 1][kWaves];
    double acc[kDiisMax], mx = 0.0;
#pragma unroll
    for (int j = 0; j < kDiisMax; ++j) acc[j] = 0.0;
    T* hts = ht + slot * n;
    T* hes = he + slot * n;
    for (long long k = (long long)blockIdx.x * kThreads + threadIdx.x; k < n; k += (long long)gridDim.x * kThreads) {
        const bool one = k < n1;
        const long long q = one ? k : k - n1;
        T rr = one ? r1[q] : r2[q];
        const T tt = one ? t1[q] : t2[q];
        double d = one ? D1[q] : D2[q];
        // the stored steps, all loads under way together (here and in
        // k_extrapolate; each load waiting for the one before it made an
        // iteration of 8 / 24 spinors 121 instead of 119 us, the (0,2) sector
        // step of 20 / 200 in eight irreps 250 instead of 245)
        T x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (j < m - 1) x[j] = he[ord.v[j] * n + k];
        if (dS != 0.0) {
            const double dl = dyn_delta(d, dS, dn);
            rr = axpy(-dl, tt, rr);
            d += dl;
        }
        d -= shift;
        const T e = over(rr, d);
        hes[k] = e;
        hts[k] = axpy(1.0, e, tt);
        mx = nan_max(size(e), mx);
#pragma unroll
        for (int j = 0; j < kDiisMax; ++j) {
            if (j < m - 1) acc[j] += re_dot(j < 8 ? x[j & 7] : he[ord.v[j] * n + k], e);
            else if (j == m - 1) acc[j] += re_dot(e, e);
        }
    }
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
    for (int j = 0; j < kDiisMax; ++j)
        if (j < m) {
            const double v = wave_sum(acc[j]);
            if (lane == 0) sh[j][wave] = v;
        }
    mx = wave_max(mx);
    if (lane == 0) sh[m][wave] = mx;
    __syncthreads();
    if ((int)threadIdx.x <= m) {
        double v = sh[threadIdx.x][0];
        for (int w = 1; w < kWaves; ++w)
            v = (int)threadIdx.x < m ? v + sh[threadIdx.x][w] : nan_max(v, sh[threadIdx.x][w]);
        part[(long long)threadIdx.x * gridDim.x + blockIdx.x] = v;
    }
}

// Bordered Pulay system over the slots order[0..m) (oldest first) of the
// symmetric matrix B (leading dimension ldb): Gaussian elimination with
// partial pivoting in FP64; a pivot below 1e-14 * max|A| drops the oldest
// slot and the solve is repeated.  One wave: lane i holds row i in registers,
// the pivot row is broadcast lane by lane, so a step costs a pivot search, one
// division and one update per column (a single thread walking the matrix in
// LDS took 45 us at nine vectors).  B and order are in LDS and only read.
// Every lane of the wave calls it, gets the number of dropped slots and, in
// *coef, the coefficient of slot `lane` (0 for a slot not used): the unknowns
// go from lane to lane through registers, so no lane reads memory that another
// has just written.
template <int MAXM>
__device__ int diis_solve(const double* B, int ldb, const int* order, int m, double* coef) {
    constexpr int SPAN = MAXM < 16 ? 8 : 16;   // lanes 0..MAXM hold rows: butterflies over 2 * SPAN lanes
    static_assert(MAXM < 2 * SPAN, "rows in one butterfly");
    const int lane = threadIdx.x & 63;
    for (int first = 0;; ++first) {
        const int k = m - first;
        if (k <= 1) {
            *coef = lane == order[m - 1] ? 1.0 : 0.0;
            return first;
        }
        const int mine = order[first + min(lane, k - 1)];
        double scale = lane < k ? fabs(B[mine * ldb + mine]) : 0.0;
        for (int d = SPAN; d > 0; d >>= 1) scale = fmax(scale, __shfl_xor(scale, d));
        scale = lane_value(scale, 0);
        if (!(scale > 0.0)) scale = 1.0;
        // columns 0..k-1, the border column and the right-hand side of row `lane`
        double a[MAXM + 1], rhs = lane == k ? -1.0 : 0.0, amax = 1.0;
#pragma unroll
        for (int c = 0; c < MAXM; ++c) {
            a[c] = 0.0;
            if (c < k && lane < k) a[c] = B[mine * ldb + order[first + c]] / scale;
            if (c < k && lane == k) a[c] = -1.0;
            amax = fmax(amax, fabs(a[c]));
        }
        a[MAXM] = lane < k ? -1.0 : 0.0;
        for (int d = SPAN; d > 0; d >>= 1) amax = fmax(amax, __shfl_xor(amax, d));
        amax = lane_value(amax, 0);
        bool free_row = lane <= k, singular = false;
        int piv[MAXM + 1];
#pragma unroll
        for (int c = 0; c <= MAXM; ++c) {
            piv[c] = 0;
            if (singular || (c >= k && c < MAXM)) continue;
            // the largest entry of the column among the free rows (the lowest row of equal ones)
            double v = free_row && a[c] == a[c] ? fabs(a[c]) : -1.0;
            int p = lane;
#pragma unroll
            for (int d = SPAN; d > 0; d >>= 1) {
                const double w = __shfl_xor(v, d);
                const int q = __shfl_xor(p, d);
                if (w > v || (w == v && q < p)) {
                    v = w;
                    p = q;
                }
            }
            p = __builtin_amdgcn_readlane(p, 0);
            if (!(lane_value(v, 0) >= 1e-14 * amax)) {
                singular = true;
                continue;
            }
            piv[c] = p;
            if (lane == p) free_row = false;
            const double f = free_row ? a[c] / lane_value(a[c], p) : 0.0;
#pragma unroll
            for (int j = c + 1; j <= MAXM; ++j) a[j] -= f * lane_value(a[j], p);
            rhs -= f * lane_value(rhs, p);
        }
        if (singular) continue;
        double mycoef = 0.0;
#pragma unroll
        for (int c = MAXM; c >= 0; --c) {
            if (c >= k && c < MAXM) continue;
            const double xc = lane_value(rhs, piv[c]) / lane_value(a[c], piv[c]);
            if (c < k && lane == order[first + c]) mycoef = xc;   // column c is slot order[first + c]
            rhs -= a[c] * xc;
        }
        *coef = mycoef;
        return first;
    }
}

// One workgroup: sum the block partials of k_step into row/column `newslot` of
// B, then solve the bordered system over the slots `ord` (oldest first).
// coef[slot] receives the coefficient (0 for unused slots); out[0] = max |step|,
// out[1] = number of dropped slots (pinned host memory).  A step that is not
// finite sets coef[kDiisMax] = 1 (the extrapolation then leaves the amplitudes
// at their input values) and leaves B untouched; otherwise coef[kDiisMax] = 0.
constexpr int kFinish = 1024;   // a wave per dot product
__global__ __launch_bounds__(1024) void k_finish(const double* __restrict__ part, int nblk, int m,
                                                double* __restrict__ B, int newslot, DiisOrder ord,
                                                double* __restrict__ coef, double* __restrict__ out) {
    constexpr int N = kDiisMax;
    __shared__ double row[N + 1], Bs[N * N];
    __shared__ int order[N];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    if (tid < N) order[tid] = tid < m ? ord.v[tid] : 0;
    if (tid < N * N) Bs[tid] = B[tid];
    for (int j = wave; j <= m; j += kFinish / 64) {
        const double* p = part + (long long)j * nblk;
        double v = 0.0;
        if (j < m) {
#pragma unroll 8
            for (int b = lane; b < nblk; b += 64) v += p[b];
            v = wave_sum(v);
        } else {
#pragma unroll 8
            for (int b = lane; b < nblk; b += 64) v = nan_max(p[b], v);
            v = wave_max(v);
        }
        if (lane == 0) row[j] = v;
    }
    __syncthreads();
    const double mx = row[m];
    const bool finite = isfinite(mx);
    // row[j] pairs the new vector with the slot order[j]
    if (finite && tid < m) {
        const int o = order[tid];
        B[newslot * N + o] = Bs[newslot * N + o] = row[tid];
        B[o * N + newslot] = Bs[o * N + newslot] = row[tid];
    }
    __syncthreads();
    if (wave != 0) return;
    double c = 0.0;   // of slot `lane`
    const int dropped = !finite ? 0 : m <= 8 ? diis_solve<8>(Bs, N, order, m, &c) : diis_solve<N>(Bs, N, order, m, &c);
    if (lane < N) coef[lane] = c;
    if (lane == 0) {
        coef[N] = finite ? 0.0 : 1.0;
        out[0] = mx;
        out[1] = (double)dropped;
    }
}

// t1, t2 = sum_j coef[j] (history slot j), unless coef[kDiisMax] marks a
// non-finite step
template <typename T>
__global__ __launch_bounds__(256) void k_extrapolate(T* __restrict__ t1, T* __restrict__ t2,
                                                     const T* __restrict__ ht, const double* __restrict__ coef,
                                                     long long n1, long long n) {
    const long long k = (long long)blockIdx.x * kThreads + threadIdx.x;
    if (k >= n || coef[kDiisMax] != 0.0) return;
    T s{};
#pragma unroll
    for (int g = 0; g < kDiisMax; g += 8) {
        T x[8];
        double c[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            c[j] = coef[g + j];
            if (c[j] != 0.0) x[j] = ht[(g + j) * n + k];
        }
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (c[j] != 0.0) s = axpy(c[j], x[j], s);
    }
    if (k < n1) t1[k] = s;
    else t2[k - n1] = s;
}

template <typename T>
__device__ __forceinline__ T signed_elem(const T* __restrict__ s, uint32_t m) {
    const T x = s[m & 0x7FFFFFFFu];
    return (m & 0x80000000u) ? axpy(-1.0, x, T{}) : x;
}

// sum <ij||ab> tau_ij^ab with tau = t2 + t1 t1 - t1 t1 formed on the fly from
// the maps of the plan's t1 x t1 reorder; block partials (re, im) go to pinned
// host memory, where they are added in block order.
template <typename T>
__global__ __launch_bounds__(256) void k_energy(const T* __restrict__ oovv, const T* __restrict__ t1,
                                                const T* __restrict__ t2, GatherMaps maps, long long n,
                                                double* __restrict__ part) {
    __shared__ double sh[2][kWaves];
    double sr = 0.0, si = 0.0;
    for (long long k = (long long)blockIdx.x * kThreads + threadIdx.x; k < n; k += (long long)gridDim.x * kThreads) {
        T tau = t2[k];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const uint32_t ma = maps.a[t][k], mb = maps.b[t][k];
            if (ma != 0xFFFFFFFFu && mb != 0xFFFFFFFFu)
                tau = axpy(1.0, times(signed_elem(t1, ma), signed_elem(t1, mb)), tau);
        }
        const T e = times(oovv[k], tau);
        sr += re(e);
        si += im(e);
    }
    sr = wave_sum(sr);
    si = wave_sum(si);
    if ((threadIdx.x & 63) == 0) {
        sh[0][threadIdx.x >> 6] = sr;
        sh[1][threadIdx.x >> 6] = si;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        double v = 0.0;
        for (int w = 0; w < kWaves; ++w) v += sh[threadIdx.x][w];
        part[2 * blockIdx.x + threadIdx.x] = v;
    }
}

template <typename T>
hipError_t update(const UpdateArgs& u, hipStream_t st) {
    const long long n = u.n1 + u.n2;
    const int nblk = reduce_blocks(n);
    k_step<T><<<nblk, kThreads, 0, st>>>((const T*)u.t1, (const T*)u.r1, u.D1, (const T*)u.t2, (const T*)u.r2, u.D2,
                                         (T*)u.ht, (T*)u.he, u.n1, n, u.slot, u.m, u.order, u.part, u.shift, u.dyn_S,
                                         u.dyn_n);
    k_finish<<<1, kFinish, 0, st>>>(u.part, nblk, u.m, u.B, u.slot, u.order, u.coef, u.out);
    if (n > 0)
        k_extrapolate<T><<<(unsigned)((n + kThreads - 1) / kThreads), kThreads, 0, st>>>(
            (T*)u.t1, (T*)u.t2, (const T*)u.ht, u.coef, u.n1, n);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_update(const UpdateArgs& u, bool real, hipStream_t st) {
    if (u.dyn_S != 0.0 && !(u.dyn_S < 0.0 && u.dyn_n >= 1)) return hipErrorInvalidValue;
    if (u.m < 1 || u.m > kDiisMax) return hipErrorInvalidValue;
    return real ? update<double>(u, st) : update<double2>(u, st);
}

hipError_t launch_energy(const void* oovv, const void* t1, const void* t2, const GatherMaps& maps, long long n,
                         double* part, int nblk, bool real, hipStream_t st) {
    if (real)
        k_energy<double><<<nblk, kThreads, 0, st>>>((const double*)oovv, (const double*)t1, (const double*)t2, maps, n,
                                                    part);
    else
        k_energy<double2><<<nblk, kThreads, 0, st>>>((const double2*)oovv, (const double2*)t1, (const double2*)t2, maps,
                                                     n, part);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// batched Jacobi + DIIS update and energy: blockIdx.y (or x) = system; each
// system keeps its own circular DIIS history on the device, so an iteration
// needs no host decision and can be replayed as a graph.

__global__ __launch_bounds__(256) void k_bjacobi(const double2* __restrict__ t1, const double2* __restrict__ t2,
                                                 const double2* __restrict__ r1, const double2* __restrict__ r2,
                                                 const double* __restrict__ D1, const double* __restrict__ D2,
                                                 const BSeg* __restrict__ segs, const BState* __restrict__ state,
                                                 double2* __restrict__ ht, double2* __restrict__ he,
                                                 double* __restrict__ part_max, double shift) {
    __shared__ double sh[kThreads];
    const int s = blockIdx.y;
    const BState stt = state[s];
    if (!stt.active) {
        if (threadIdx.x == 0) part_max[(long long)s * gridDim.x + blockIdx.x] = 0.0;
        return;
    }
    const BSeg g = segs[s];
    const long long n = g.n1 + g.n2;
    const int slot = (stt.newest + 1) % stt.nd;
    double2* hts = ht + g.hoff + (long long)slot * n;
    double2* hes = he + g.hoff + (long long)slot * n;
    double mx = 0.0;
    for (long long k = (long long)blockIdx.x * kThreads + threadIdx.x; k < n; k += (long long)gridDim.x * kThreads) {
        double2 rr, tt;
        double d;
        if (k < g.n1) {
            rr = r1[g.off1 + k];
            tt = t1[g.off1 + k];
            d = D1[g.off1 + k];
        } else {
            rr = r2[g.off2 + k - g.n1];
            tt = t2[g.off2 + k - g.n1];
            d = D2[g.off2 + k - g.n1];
        }
        d -= shift;   // level shift: D < 0 for every amplitude, so |D| grows and the step is damped
        const double2 st = make_double2(rr.x / d, rr.y / d);
        hes[k] = st;
        hts[k] = make_double2(tt.x + st.x, tt.y + st.y);
        const double a = sqrt(st.x * st.x + st.y * st.y);
        mx = (a > mx || a != a) ? a : mx;
    }
    const double b = block_max(mx, sh);
    if (threadIdx.x == 0) part_max[(long long)s * gridDim.x + blockIdx.x] = b;
}

// live slots of system state `st` after adding the new vector: oldest first
__device__ inline int bslots(const BState& st, int* order) {
    const int nw = (st.newest + 1) % st.nd;
    const int m = min(st.count + 1, st.nd);
    for (int j = 0; j < m; ++j) order[j] = ((nw - (m - 1) + j) % st.nd + st.nd) % st.nd;
    return m;
}

__global__ __launch_bounds__(256) void k_bdots(const BSeg* __restrict__ segs, const BState* __restrict__ state,
                                               const double2* __restrict__ he, double* __restrict__ part) {
    __shared__ double sh[kThreads];
    const int s = blockIdx.y;
    const BState stt = state[s];
    if (!stt.active) return;
    const BSeg g = segs[s];
    const long long n = g.n1 + g.n2;
    int order[8];
    const int m = bslots(stt, order);
    const double2* enew = he + g.hoff + (long long)order[m - 1] * n;
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (long long k = (long long)blockIdx.x * kThreads + threadIdx.x; k < n; k += (long long)gridDim.x * kThreads) {
        const double2 y = enew[k];
        for (int j = 0; j < m; ++j) {
            const double2 x = he[g.hoff + (long long)order[j] * n + k];
            acc[j] += x.x * y.x + x.y * y.y;
        }
    }
    for (int j = 0; j < m; ++j) {
        const double b = block_sum(acc[j], sh);
        if (threadIdx.x == 0) part[((long long)s * gridDim.x + blockIdx.x) * 8 + j] = b;
    }
}

// one workgroup per system: finish the dots, update B, solve, advance the
// circular history, apply the convergence test (max|step| < tol freezes the
// system after this update; a non-finite step freezes it as failed)
__global__ __launch_bounds__(256) void k_bfinish(BState* __restrict__ state, const double* __restrict__ part, int nblk,
                                                 const double* __restrict__ part_max, double* __restrict__ Bm,
                                                 double* __restrict__ coef, double* __restrict__ maxstep, double tol,
                                                 int* __restrict__ active, int* __restrict__ upd) {
    __shared__ double sh[kThreads];
    __shared__ double row[8], Bs[64];
    __shared__ int ord[8];
    const int s = blockIdx.x;
    BState stt = state[s];
    if (!stt.active) {
        if (threadIdx.x == 0) {
            state[s].upd = 0;
            active[s] = 0;
            upd[s] = 0;
        }
        return;
    }
    int order[8];
    const int m = bslots(stt, order);
    for (int j = 0; j < m; ++j) {
        double v = 0.0;
        for (int b = threadIdx.x; b < nblk; b += kThreads) v += part[((long long)s * nblk + b) * 8 + j];
        const double r = block_sum(v, sh);
        if (threadIdx.x == 0) row[j] = r;
    }
    double mx = 0.0;
    for (int b = threadIdx.x; b < nblk; b += kThreads) {
        const double a = part_max[(long long)s * nblk + b];
        mx = (a > mx || a != a) ? a : mx;
    }
    mx = block_max(mx, sh);
    double* B = Bm + (long long)s * 64;
    const int nw = order[m - 1];
    if (threadIdx.x < 64) Bs[threadIdx.x] = B[threadIdx.x];
    if (threadIdx.x == 0)
        for (int j = 0; j < m; ++j) ord[j] = order[j];
    __syncthreads();
    if ((int)threadIdx.x < m) {
        const int o = ord[threadIdx.x];
        B[nw * 8 + o] = Bs[nw * 8 + o] = row[threadIdx.x];
        B[o * 8 + nw] = Bs[o * 8 + nw] = row[threadIdx.x];
    }
    __syncthreads();
    if (threadIdx.x >= 64) return;
    double c;   // of slot threadIdx.x
    const int dropped = diis_solve<8>(Bs, 8, ord, m, &c);
    if (threadIdx.x < 8) coef[(long long)s * 8 + threadIdx.x] = c;
    if (threadIdx.x != 0) return;
    stt.newest = nw;
    stt.count = max(1, m - dropped);
    stt.iters += 1;
    stt.upd = 1;
    if (!(mx == mx) || mx > 1.7976931348623157e308) {
        stt.failed = 1;
        stt.active = 0;
        stt.upd = 0;
    } else if (mx < tol) {
        stt.active = 0;
    }
    state[s] = stt;
    active[s] = stt.active;
    upd[s] = stt.upd;
    maxstep[s] = mx;
}

__global__ __launch_bounds__(256) void k_blincomb(double2* __restrict__ t1, double2* __restrict__ t2,
                                                  const BSeg* __restrict__ segs, const BState* __restrict__ state,
                                                  const double2* __restrict__ ht, const double* __restrict__ coef) {
    const int s = blockIdx.y;
    const BState stt = state[s];
    if (!stt.upd) return;
    const BSeg g = segs[s];
    const long long n = g.n1 + g.n2;
    double c[8];
    for (int j = 0; j < 8; ++j) c[j] = j < stt.nd ? coef[s * 8 + j] : 0.0;
    for (long long k = (long long)blockIdx.x * kThreads + threadIdx.x; k < n; k += (long long)gridDim.x * kThreads) {
        double sr = 0.0, si = 0.0;
        for (int j = 0; j < stt.nd; ++j)
            if (c[j] != 0.0) {
                const double2 x = ht[g.hoff + (long long)j * n + k];
                sr += c[j] * x.x;
                si += c[j] * x.y;
            }
        if (k < g.n1) t1[g.off1 + k] = make_double2(sr, si);
        else t2[g.off2 + k - g.n1] = make_double2(sr, si);
    }
}

__global__ __launch_bounds__(256) void k_benergy(const double2* __restrict__ x, const double2* __restrict__ y,
                                                 const BSeg* __restrict__ segs, double* __restrict__ part) {
    __shared__ double sh[kThreads];
    const int s = blockIdx.y;
    const BSeg g = segs[s];
    double sr = 0.0, si = 0.0;
    for (long long k = (long long)blockIdx.x * kThreads + threadIdx.x; k < g.n2; k += (long long)gridDim.x * kThreads) {
        const double2 a = x[g.off2 + k], b = y[g.off2 + k];
        sr += a.x * b.x - a.y * b.y;
        si += a.x * b.y + a.y * b.x;
    }
    const double r = block_sum(sr, sh);
    const double i = block_sum(si, sh);
    if (threadIdx.x == 0) {
        part[((long long)s * gridDim.x + blockIdx.x) * 2] = r;
        part[((long long)s * gridDim.x + blockIdx.x) * 2 + 1] = i;
    }
}

// per-system report row: E_re, E_im, max|step|, active, iterations, failed
__global__ __launch_bounds__(256) void k_breport(const double* __restrict__ part, int nblk,
                                                 const BState* __restrict__ state, const double* __restrict__ maxstep,
                                                 double* __restrict__ out) {
    __shared__ double sh[kThreads];
    const int s = blockIdx.x;
    double r = 0.0, i = 0.0;
    for (int b = threadIdx.x; b < nblk; b += kThreads) {
        r += part[((long long)s * nblk + b) * 2];
        i += part[((long long)s * nblk + b) * 2 + 1];
    }
    r = block_sum(r, sh);
    i = block_sum(i, sh);
    if (threadIdx.x == 0) {
        const BState st = state[s];
        double* o = out + (long long)s * 6;
        o[0] = r;
        o[1] = i;
        o[2] = maxstep[s];
        o[3] = st.active;
        o[4] = st.iters;
        o[5] = st.failed;
    }
}

hipError_t launch_batch_update(const double2* t1, const double2* t2, const double2* r1, const double2* r2,
                               double2* t1o, double2* t2o, const double* D1, const double* D2, const BSeg* segs,
                               BState* state, double2* ht, double2* he, double* part_max, double* part, double* Bm,
                               double* coef, double* maxstep, double tol, double shift, int* active, int* upd,
                               int nsys, int nblk, hipStream_t st) {
    if (nsys <= 0) return hipSuccess;
    dim3 grid(nblk, nsys);
    k_bjacobi<<<grid, kThreads, 0, st>>>(t1, t2, r1, r2, D1, D2, segs, state, ht, he, part_max, shift);
    k_bdots<<<grid, kThreads, 0, st>>>(segs, state, he, part);
    k_bfinish<<<nsys, kThreads, 0, st>>>(state, part, nblk, part_max, Bm, coef, maxstep, tol, active, upd);
    k_blincomb<<<grid, kThreads, 0, st>>>(t1o, t2o, segs, state, ht, coef);
    return hipGetLastError();
}

hipError_t launch_batch_energy(const double2* oovv, const double2* tau, const BSeg* segs, const BState* state,
                               const double* maxstep, double* part, double* out, int nsys, int nblk, hipStream_t st) {
    if (nsys <= 0) return hipSuccess;
    k_benergy<<<dim3(nblk, nsys), kThreads, 0, st>>>(oovv, tau, segs, part);
    k_breport<<<nsys, kThreads, 0, st>>>(part, nblk, state, maxstep, out);
    return hipGetLastError();
}


// per-system max |r / D| over the T1 and T2 segments
__global__ __launch_bounds__(256) void k_bmaxnorm(const double2* __restrict__ r1, const double2* __restrict__ r2,
                                                  const double* __restrict__ D1, const double* __restrict__ D2,
                                                  const BSeg* __restrict__ segs, double* __restrict__ part) {
    __shared__ double sh[kThreads];
    const int s = blockIdx.y;
    const BSeg g = segs[s];
    const long long n = g.n1 + g.n2;
    double mx = 0.0;
    for (long long k = (long long)blockIdx.x * kThreads + threadIdx.x; k < n; k += (long long)gridDim.x * kThreads) {
        double2 rr;
        double d;
        if (k < g.n1) {
            rr = r1[g.off1 + k];
            d = D1[g.off1 + k];
        } else {
            rr = r2[g.off2 + k - g.n1];
            d = D2[g.off2 + k - g.n1];
        }
        const double a = sqrt(rr.x * rr.x + rr.y * rr.y) / fabs(d);
        mx = (a > mx || a != a) ? a : mx;
    }
    const double b = block_max(mx, sh);
    if (threadIdx.x == 0) part[(long long)s * gridDim.x + blockIdx.x] = b;
}

__global__ __launch_bounds__(256) void k_bmaxnorm_final(const double* __restrict__ part, int nblk,
                                                        double* __restrict__ out) {
    __shared__ double sh[kThreads];
    const int s = blockIdx.x;
    double mx = 0.0;
    for (int b = threadIdx.x; b < nblk; b += kThreads) {
        const double a = part[(long long)s * nblk + b];
        mx = (a > mx || a != a) ? a : mx;
    }
    mx = block_max(mx, sh);
    if (threadIdx.x == 0) out[s] = mx;
}

hipError_t launch_batch_maxnorm(const double2* r1, const double2* r2, const double* D1, const double* D2,
                                const BSeg* segs, double* part, double* out, int nsys, int nblk, hipStream_t st) {
    if (nsys <= 0) return hipSuccess;
    k_bmaxnorm<<<dim3(nblk, nsys), kThreads, 0, st>>>(r1, r2, D1, D2, segs, part);
    k_bmaxnorm_final<<<nsys, kThreads, 0, st>>>(part, nblk, out);
    return hipGetLastError();
}

}  // namespace fscc
