// kernels_fused.hip -- many small independent operations of a residual in one
// launch.
//
// A launch that depends on the previous one takes 4.5 us however little it
// does, and a tile of the grouped GEMM walks its K slices one memory latency
// at a time: the 56 operations of a small system's residual are bound by
// that, not by work (8 occupied and 24 virtual spinors: 0.55 ms for 146 Mflop).
// The host (schedule.hpp) puts all operations whose inputs are ready into one
// list of work items; every workgroup takes one item:
//   * 1024 or 2048 destination elements of a chain of elementwise operations and
//     reorders with one destination (tau = t2, then += t1 t1; the
//     contributions to a residual), the values kept in registers from one
//     operation to the next,
//   * output tiles of 16 x 16 of a small GEMM, 16 waves over 16/kw tiles.  The kw
//     waves of a tile share its K range, every wave loads its fragments
//     straight from memory (the operands sit in the L2) eight at a time with
//     the next eight under way, and the partial tiles are summed through LDS
//     in wave order.  A longer K range is split over workgroups as well, or
//   * the sum of such parts, as an operation of its own in a later launch.
// Complex and real (T = double2, double).  Results are deterministic.
//
// Measured (whole iteration, before -> after): 8 occupied / 24 virtual spinors
// 601 -> 168 us (10 launches of 5-15 us instead of 56), real 13 / 67 in three
// irreps 706 -> 249 us, 20 / 120 in eight irreps 1004 -> 638 us; what is left
// of a launch is its start (4.5 us) and five dependent memory latencies.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "elem_math.hpp"
#include "kernels.hpp"

namespace fscc {
namespace {

typedef double dbl4 __attribute__((ext_vector_type(4)));
constexpr int kWaves = kFusedThreads / 64;

template <typename T>
__device__ __forceinline__ T* ptr(const FRef& r, const FIo& io) {
    return (T*)(r.io >= 0 ? io.p[r.io] : r.p);
}

__device__ __forceinline__ double2 mapped(const double2* __restrict__ s, uint32_t m) {
    if (m == 0xFFFFFFFFu) return make_double2(0.0, 0.0);
    double2 x = s[m & 0x7FFFFFFFu];
    if (m & 0x80000000u) {
        x.x = -x.x;
        x.y = -x.y;
    }
    return x;
}

__device__ __forceinline__ double mapped(const double* __restrict__ s, uint32_t m) {
    if (m == 0xFFFFFFFFu) return 0.0;
    const double x = s[m & 0x7FFFFFFFu];
    return (m & 0x80000000u) ? -x : x;
}

__device__ __forceinline__ void conjugate(double2& x) { x.y = -x.y; }
__device__ __forceinline__ void conjugate(double&) {}
__device__ __forceinline__ void add(double2& a, double2 b) {
    a.x += b.x;
    a.y += b.y;
}
__device__ __forceinline__ void add(double& a, double b) { a += b; }
__device__ __forceinline__ void scale(double2& o, double d) {
    o.x *= d;
    o.y *= d;
}
__device__ __forceinline__ void scale(double& o, double d) { o *= d; }

// E destination elements per thread (kFusedThreads apart) through a chain of
// operations: the loads of all elements are under way together, so a workgroup
// pays the memory latencies of the chain once for all of them (two elements,
// where one per thread would take more than the workgroups resident at once;
// four need more registers than a 1024-thread workgroup has).
template <int E, typename T>
__device__ void fused_elements(const FOp* __restrict__ op, const FIo& io, long long k0) {
    constexpr int TG = E == 1 ? 4 : 2;   // terms whose sources are under way together
    T v[E];
    bool held[E], in[E];   // v holds the element's value; the element exists
    long long at[E];
    const long long n = op->n;
    T* dst = ptr<T>(op->dst, io);
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const long long k = k0 + (long long)e * kFusedThreads;
        in[e] = k < n;
        at[e] = in[e] ? k : n - 1;   // past the end: the last element's loads, nothing stored
        held[e] = false;
        v[e] = T{};
    }
    auto old = [&](int e) {
        if (!held[e]) v[e] = dst[at[e]];
        held[e] = true;
    };
    for (;; ++op) {
        const FOp o = *op;
        const T* src = ptr<const T>(o.src, io);
        if (o.kind == FK_GATHER) {
            // the maps of all terms, then the sources of TG terms at a time
            const T* src2 = ptr<const T>(o.src2, io);
            const bool bil = o.b[0] != nullptr;
            uint32_t ma[4][E], mb[4][E];
            T s[E];
            bool any[E];
#pragma unroll
            for (int e = 0; e < E; ++e) {
                s[e] = T{};
                any[e] = false;
            }
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    ma[t][e] = t < o.nt ? o.a[t][at[e]] : 0xFFFFFFFFu;
                    mb[t][e] = bil && t < o.nt ? o.b[t][at[e]] : 0u;
                }
#pragma unroll
            for (int t = 0; t < 4; t += TG) {
                if (t >= o.nt) break;
                T x[TG][E], y[TG][E];
#pragma unroll
                for (int u = 0; u < TG; ++u)
#pragma unroll
                    for (int e = 0; e < E; ++e) {
                        x[u][e] = mapped(ptr<const T>(o.srct[t + u], io), ma[t + u][e]);
                        if (bil) y[u][e] = mapped(src2, mb[t + u][e]);
                    }
#pragma unroll
                for (int u = 0; u < TG; ++u)
                    if (t + u < o.nt)
#pragma unroll
                        for (int e = 0; e < E; ++e) {
                            any[e] = any[e] || (ma[t + u][e] != 0xFFFFFFFFu && mb[t + u][e] != 0xFFFFFFFFu);
                            T z = x[u][e];
                            if (o.conj) conjugate(z);
                            if (bil) z = elem_mul(z, y[u][e]);
                            add(s[e], z);
                        }
            }
#pragma unroll
            for (int e = 0; e < E; ++e) {
                // an accumulating gather leaves an element whose terms are
                // all structural zeros as it is
                if (o.beta && !any[e]) continue;
                T out = elem_scale(o.ar, o.ai, s[e]);
                if (o.beta) {
                    old(e);
                    add(out, v[e]);
                }
                v[e] = out;
                held[e] = true;
            }
        } else if (o.kind == FK_AXPBY) {
            T x[E];
#pragma unroll
            for (int e = 0; e < E; ++e) x[e] = src[at[e]];
#pragma unroll
            for (int e = 0; e < E; ++e) {
                if (o.conj) conjugate(x[e]);
                T out = elem_scale(o.ar, o.ai, x[e]);
                if (o.beta) {
                    old(e);
                    add(out, v[e]);
                }
                v[e] = out;
                held[e] = true;
            }
        } else {
            const double* d = ptr<const double>(o.src2, io);
            const bool diag = o.kind == FK_DIAG;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                old(e);
                if (diag) v[e] = elem_sub(v[e], d[at[e]], src[at[e]]);
                else scale(v[e], d[at[e]]);
            }
        }
        if (!o.more) break;
    }
#pragma unroll
    for (int e = 0; e < E; ++e)
        if (held[e] && in[e]) dst[at[e]] = v[e];
}

// Accumulators of one 16 x 16 tile.  Complex: three real products (p = Ar Br,
// q = Ai Bi, s = (Ar + Ai)(Br + Bi); re = p - q, im = s - p - q).
struct AccZ {
    dbl4 p, q, s;
};
struct AccD {
    dbl4 p;
};
__device__ __forceinline__ void clear(AccZ& c) { c.p = c.q = c.s = dbl4{0.0, 0.0, 0.0, 0.0}; }
__device__ __forceinline__ void clear(AccD& c) { c.p = dbl4{0.0, 0.0, 0.0, 0.0}; }
__device__ __forceinline__ void mma(AccZ& c, double2 a, double2 b) {
    c.p = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.x, c.p, 0, 0, 0);
    c.q = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.y, c.q, 0, 0, 0);
    c.s = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x + a.y, b.x + b.y, c.s, 0, 0, 0);
}
__device__ __forceinline__ void mma(AccD& c, double a, double b) {
    c.p = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c.p, 0, 0, 0);
}
__device__ __forceinline__ void put(double2* x, const AccZ& c, int e) {
    *x = make_double2(c.p[e] - c.q[e], c.s[e] - c.p[e] - c.q[e]);
}
__device__ __forceinline__ void put(double* x, const AccD& c, int e) { *x = c.p[e]; }
template <typename T>
struct AccOf {
    typedef AccZ type;
};
template <>
struct AccOf<double> {
    typedef AccD type;
};

// output element e (0..255) of a tile, in the order in which the accumulators
// hold it: element q of a lane is row 4 q + lane / 16, column lane % 16
template <typename T>
__device__ __forceinline__ void tile_store(const FOp& o, T* C, const ZTile& tl, const ZProb& pr, int e, T s) {
    const int row = tl.m0 + (e >> 6) * 4 + ((e & 63) >> 4), col = tl.n0 + (e & 15);
    if (row >= pr.M || col >= pr.N) return;
    T* p = C + pr.c_off + (long long)row * pr.ldc + col;
    T out = elem_scale(o.ar, o.ai, s);
    if (o.beta) add(out, *p);
    *p = out;
}

// Units [first, first + 16/kw) of a GEMM: unit = (tile, K part of `split`).
template <typename T>
__device__ void fused_gemm(const FOp* __restrict__ op, const FIo& io, int first, T* __restrict__ red) {
    const FOp o = *op;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kw = o.kw, g = wave / kw, unit = first + g;
    const bool live = unit < o.ntiles * o.split;   // uniform per wave
    const int tile = unit / o.split, part = unit % o.split;
    ZTile tl{};
    ZProb pr{};
    if (live) {
        tl = o.tiles[tile];
        pr = o.probs[tl.prob];
        const int lr = lane & 15, lq = lane >> 4;
        const int waves = kw * o.split, chunk = ((pr.K + waves - 1) / waves + 3) & ~3;
        const int kb = min(pr.K, (part * kw + wave % kw) * chunk), ke = min(pr.K, kb + chunk);
        const long long ska = o.tA ? pr.lda : 1, skb = o.tB ? 1 : pr.ldb;
        const long long sma = o.tA ? 1 : pr.lda, snb = o.tB ? pr.ldb : 1;
        // rows and columns past the edge read the last one; they reach no stored output
        const T* pa = ptr<const T>(o.src, io) + pr.a_off + min(tl.m0 + lr, pr.M - 1) * sma;
        const T* pb = ptr<const T>(o.src2, io) + pr.b_off + min(tl.n0 + lr, pr.N - 1) * snb;
        const bool cA = o.cA, cB = o.cB;
        typename AccOf<T>::type c;
        clear(c);
        // 16 k per round: step s of lane group q takes k0 + 4 s + q; k past the
        // end reads the last one and counts as zero in both operands
        auto load = [&](T (&a)[4], T (&b)[4], int k0) {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int k = min(k0 + 4 * s + lq, ke - 1);
                a[s] = pa[k * ska];
                b[s] = pb[k * skb];
            }
        };
        auto work = [&](T (&a)[4], T (&b)[4], int k0) {
            const bool edge = k0 + 16 > ke;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                if (edge && k0 + 4 * s + lq >= ke) a[s] = b[s] = T{};
                if (cA) conjugate(a[s]);
                if (cB) conjugate(b[s]);
                mma(c, a[s], b[s]);
            }
        };
        if (kb < ke) {
            T a0[4], b0[4], a1[4], b1[4];
            load(a0, b0, kb);
            for (int k0 = kb; k0 < ke; k0 += 32) {
                if (k0 + 16 < ke) load(a1, b1, k0 + 16);
                work(a0, b0, k0);
                if (k0 + 16 < ke) {
                    if (k0 + 32 < ke) load(a0, b0, k0 + 32);
                    work(a1, b1, k0 + 16);
                }
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) put(&red[(wave * 4 + q) * 64 + lane], c, q);
    }
    __syncthreads();
    if (!live) return;
    T* C = ptr<T>(o.dst, io);
    T* W = (T*)o.work + (long long)unit * 256;
    for (int e = tid - g * kw * 64; e < 256; e += kw * 64) {
        T s{};
        for (int w = 0; w < kw; ++w) add(s, red[(g * kw + w) * 256 + e]);
        if (o.split > 1) W[e] = s;
        else tile_store(o, C, tl, pr, e, s);
    }
}

// Second pass of a GEMM whose K range is split over workgroups: four tiles per
// workgroup, the parts added in order.
template <typename T>
__device__ void fused_reduce(const FOp* __restrict__ op, const FIo& io, int first) {
    const FOp o = *op;
    const int tile = first + (threadIdx.x >> 8), e = threadIdx.x & 255;
    if (tile >= o.ntiles) return;
    const ZTile tl = o.tiles[tile];
    const ZProb pr = o.probs[tl.prob];
    const T* W = (const T*)o.work + (long long)tile * o.split * 256 + e;
    T s{};
    for (int p = 0; p < o.split; ++p) add(s, W[p * 256]);
    tile_store(o, ptr<T>(o.dst, io), tl, pr, e, s);
}

template <typename T>
__global__ __launch_bounds__(1024) void k_fused(const FItem* __restrict__ items, const FOp* __restrict__ ops, FIo io) {
    __shared__ T red[kWaves * 256];
    const FItem it = items[blockIdx.x];
    const FOp* o = ops + it.op;
    if (o->kind == FK_GEMM) fused_gemm<T>(o, io, it.first, red);
    else if (o->kind == FK_REDUCE) fused_reduce<T>(o, io, it.first);
    else if (o->elems == 1) fused_elements<1, T>(o, io, (long long)it.first * kFusedThreads + threadIdx.x);
    else fused_elements<2, T>(o, io, (long long)it.first * (2 * kFusedThreads) + threadIdx.x);
}

}  // namespace

hipError_t launch_fused(const FItem* items, int nitems, const FOp* ops, const FIo& io, bool real, hipStream_t st) {
    if (nitems <= 0) return hipSuccess;
    if (real) k_fused<double><<<nitems, kFusedThreads, 0, st>>>(items, ops, io);
    else k_fused<double2><<<nitems, kFusedThreads, 0, st>>>(items, ops, io);
    return hipGetLastError();
}

}  // namespace fscc
