// kernels_fused.hip -- many small independent operations of a residual in one
// launch.
//
// A launch that depends on the previous one takes 4.5 us however little it
// does, and a tile of the grouped GEMM walks its K slices one memory latency
// at a time: the 56 operations of a small system's residual are bound by
// that, not by work (8 occupied and 24 virtual spinors: 0.55 ms for 146 Mflop).
// The host (schedule.hpp) puts all operations whose inputs are ready into one
// list of work items; every workgroup (four waves, one per SIMD) takes one item:
//   * 256 destination elements of a chain of elementwise operations and
//     reorders with one destination (tau = t2, then += t1 t1; the
//     contributions to a residual), the values kept in registers from one
//     operation to the next, or
//   * output tiles of 16 x 16 of a small GEMM, 4 waves over 4/kw tiles.  The kw
//     waves of a tile share its K range, every wave loads its fragments
//     straight from memory (the operands sit in the L2) with two rounds of
//     loads under way, and the partial tiles are summed through LDS in wave
//     order.  A longer K range is split over workgroups as well; the workgroup
//     that finishes a tile's last part adds the parts in order.
// Complex and real (T = double2, double).  Results are deterministic.
//
// A launch of 16-wave workgroups took 11-13 us at 8 occupied / 24 virtual
// spinors, of which 9 were the matrix pipes of the few CUs that had the tiles:
// 16 waves of 64 k share four pipes.  With one wave per SIMD, so that a tile's
// K range reaches over four CUs, and with descriptors and maps loaded ahead of
// the chains the launches take 6-9 us; what is left are the start and five
// dependent memory latencies.  Measured (whole iteration; every operation its
// own launch, 16-wave workgroups, this): 8/24 in one irrep 601, 168, 123 us;
// real 13/67 in three 706, 217, 186 us; 20/120 in eight 1004, 560, 536 us; the
// (0,2) sector step of 20/200 in eight 304, 273, 249 us.
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "elem_math.hpp"
#include "kernels.hpp"

namespace fscc {
namespace {

typedef double dbl4 __attribute__((ext_vector_type(4)));
constexpr int kWaves = kFusedThreads / 64;
static_assert(kWaves == 4, "one wave per SIMD, 4 / kw tiles");

// Descriptors in LDS: the workgroup copies all operations of its item at once
// (one memory latency however long the chain), with the callers' buffers put
// in, and reads each into scalar registers when its turn comes.
constexpr int kOpWords = sizeof(FOp) / 8;
constexpr int kRefWord = offsetof(FOp, dst) / 8;   // dst, src2, src[4]
static_assert(sizeof(FOp) % 8 == 0 && offsetof(FOp, src2) == (kRefWord + 1) * 8 && offsetof(FOp, src) == (kRefWord + 2) * 8,
              "buffer references in a row");

__device__ __forceinline__ void stage_ops(const FOp* __restrict__ ops, int n, const FIo& io, unsigned long long* lds) {
    const unsigned long long* w = (const unsigned long long*)ops;
    for (int k = threadIdx.x; k < n * kOpWords; k += kFusedThreads) {
        unsigned long long x = w[k];
        const int f = k % kOpWords - kRefWord;
        if (f >= 0 && f < 6 && x != 0 && x <= (unsigned long long)kFusedIo) x = (unsigned long long)io.p[x - 1];
        lds[k] = x;
    }
}
__device__ __forceinline__ FOp staged_op(const unsigned long long* lds) {
    struct Words {
        int w[2 * kOpWords];
    } u;
    const int* p = (const int*)lds;
#pragma unroll
    for (int k = 0; k < 2 * kOpWords; ++k) u.w[k] = __builtin_amdgcn_readfirstlane(p[k]);
    return __builtin_bit_cast(FOp, u);
}
template <typename T>
__device__ __forceinline__ T* ptr(FRef r) {
    return (T*)r;
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

// maps of a reorder's terms at a thread's element
struct Maps {
    uint32_t a[4], b[4];
};
__device__ __forceinline__ void load_maps(Maps& m, const FOp& o, int at) {
    if (o.kind != FK_GATHER) return;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        m.a[t] = t < o.nt ? o.g.a[t][at] : 0xFFFFFFFFu;
        m.b[t] = o.bil && t < o.nt ? o.g.b[t][at] : 0u;
    }
}

// One destination element per thread through a chain of operations.  The
// memory latencies are what a chain costs, so the sources of all terms are
// under way together, and with them the next operation's maps.  (Several
// chunks per workgroup, the next one's maps loaded ahead: no faster.)
template <typename T>
__device__ void fused_elements(const unsigned long long* __restrict__ lds, FOp o, int k) {
    const int at = min(k, o.n - 1);   // past the end: the last element's loads, nothing stored
    T* dst = ptr<T>(o.dst);
    const bool in = k < o.n;
    T v{};
    bool have = false, held = false;   // v holds the element's value; it has changed
    Maps m;
    load_maps(m, o, at);
    for (;;) {
        if (!have && (o.beta || o.kind == FK_DIAG || o.kind == FK_MUL)) v = dst[at];
        have = true;
        Maps mn;
        auto next = [&] {
            if (o.more) load_maps(mn, staged_op(lds + kOpWords), at);
        };
        if (o.kind == FK_GATHER) {
            T x[4], y[4];
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (t < o.nt) {
                    x[t] = mapped(ptr<const T>(o.src[t]), m.a[t]);
                    if (o.bil) y[t] = mapped(ptr<const T>(o.src2), m.b[t]);
                }
            next();
            T s{};
            bool any = false;
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (t < o.nt) {
                    any = any || (m.a[t] != 0xFFFFFFFFu && m.b[t] != 0xFFFFFFFFu);
                    T z = x[t];
                    if (o.conj) conjugate(z);
                    if (o.bil) s = elem_add_mul(s, z, y[t]);
                    else add(s, z);
                }
            // an accumulating gather leaves an element whose terms are all
            // structural zeros as it is
            if (!o.beta || any) {
                v = o.beta ? elem_scale_add(o.ar, o.ai, s, v) : elem_scale(o.ar, o.ai, s);
                held = true;
            }
        } else if (o.kind == FK_AXPBY) {
            T x = ptr<const T>(o.src[0])[at];
            next();
            if (o.conj) conjugate(x);
            v = o.beta ? elem_scale_add(o.ar, o.ai, x, v) : elem_scale(o.ar, o.ai, x);
            held = true;
        } else {
            const double f = ptr<const double>(o.src2)[at];
            T x{};
            if (o.kind == FK_DIAG) x = ptr<const T>(o.src[0])[at];
            next();
            if (o.kind == FK_DIAG) v = elem_sub(v, f, x);
            else scale(v, f);
            held = true;
        }
        if (!o.more) break;
        lds += kOpWords;
        o = staged_op(lds);
        m = mn;
    }
    if (held && in) dst[at] = v;
}

// Accumulators of one 16 x 16 tile.  Complex: four real products, so that each
// part of an output carries the rounding of its own terms only (three products
// take the imaginary part from a difference as large as the real one).
struct AccZ {
    dbl4 re, im;
};
struct AccD {
    dbl4 p;
};
__device__ __forceinline__ void clear(AccZ& c) { c.re = c.im = dbl4{0.0, 0.0, 0.0, 0.0}; }
__device__ __forceinline__ void clear(AccD& c) { c.p = dbl4{0.0, 0.0, 0.0, 0.0}; }
__device__ __forceinline__ void mma(AccZ& c, double2 a, double2 b) {
    c.re = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.x, c.re, 0, 0, 0);
    c.im = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.y, c.im, 0, 0, 0);
    c.re = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, -b.y, c.re, 0, 0, 0);
    c.im = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.x, c.im, 0, 0, 0);
}
__device__ __forceinline__ void mma(AccD& c, double a, double b) {
    c.p = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c.p, 0, 0, 0);
}
__device__ __forceinline__ void put(double2* x, const AccZ& c, int e) {
    *x = make_double2(c.re[e], c.im[e]);
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
// hold it: element q of a lane is row 4 q + lane / 16, column lane % 16;
// nullptr past the edge
template <typename T>
__device__ __forceinline__ T* tile_at(T* C, const ZTile& tl, const ZProb& pr, int e) {
    const int row = tl.m0 + (e >> 6) * 4 + ((e & 63) >> 4), col = tl.n0 + (e & 15);
    return row < pr.M && col < pr.N ? C + pr.c_off + (long long)row * pr.ldc + col : nullptr;
}

__device__ __forceinline__ void part_store(double* p, double x) {
    __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double part_load(const double* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void part_store(double2* p, double2 x) {
    part_store(&p->x, x.x);
    part_store(&p->y, x.y);
}
__device__ __forceinline__ double2 part_load(const double2* p) {
    return make_double2(part_load(&p->x), part_load(&p->y));
}

// Units [first, first + 4/kw) of a GEMM: unit = (tile, K part of `split`).
template <typename T>
__device__ void fused_gemm(const FOp o, int first, T* __restrict__ red) {
    // steps per round of loads; three rounds of registers.  Four steps for
    // complex as well would take the kernel over 128 registers, which spills
    // (unspilled at three waves per SIMD: 3 % slower at 8/24 and 20/120).
    constexpr int R = sizeof(T) == 16 ? 2 : 4;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kw = o.kw, g = wave / kw, unit = first + g;
    const bool live = unit < o.ntiles * o.split;   // uniform per wave
    const int tile = unit / o.split, part = unit % o.split;
    const int e0 = tid - g * kw * 64, es = kw * 64;   // the thread's elements of its tile: e0, e0 + es, ..
    T* C = ptr<T>(o.dst);
    T* at = nullptr;   // of the first of them, and what it held
    T old{};
    ZTile tl{};
    ZProb pr{};
    if (live) {
        tl = o.m.tiles[tile];
        pr = o.m.probs[tl.prob];
        const int lr = lane & 15, lq = lane >> 4;
        const int waves = kw * o.split, chunk = ((pr.K + waves - 1) / waves + 3) & ~3;
        const int kb = min(pr.K, (part * kw + wave % kw) * chunk), ke = min(pr.K, kb + chunk);
        const long long ska = o.tA ? pr.lda : 1, skb = o.tB ? 1 : pr.ldb;
        const long long sma = o.tA ? 1 : pr.lda, snb = o.tB ? pr.ldb : 1;
        // rows and columns past the edge read the last one; they reach no stored output
        const T* pa = ptr<const T>(o.src[0]) + pr.a_off + min(tl.m0 + lr, pr.M - 1) * sma;
        const T* pb = ptr<const T>(o.src2) + pr.b_off + min(tl.n0 + lr, pr.N - 1) * snb;
        const bool cA = o.cA, cB = o.cB;
        typename AccOf<T>::type c;
        clear(c);
        // R steps of 4 k per round: step s of lane group q takes k0 + 4 s + q;
        // k past the end reads the last one and counts as zero in both operands
        auto load = [&](T (&a)[R], T (&b)[R], int k0) {
            if (k0 >= ke) return;
#pragma unroll
            for (int s = 0; s < R; ++s) {
                const int k = min(k0 + 4 * s + lq, ke - 1);
                a[s] = pa[k * ska];
                b[s] = pb[k * skb];
            }
        };
        auto work = [&](T (&a)[R], T (&b)[R], int k0) {
            if (k0 >= ke) return;
            const bool edge = k0 + 4 * R > ke;
#pragma unroll
            for (int s = 0; s < R; ++s) {
                if (edge && k0 + 4 * s + lq >= ke) a[s] = b[s] = T{};
                if (cA) conjugate(a[s]);
                if (cB) conjugate(b[s]);
                mma(c, a[s], b[s]);
            }
        };
        T a0[R], b0[R], a1[R], b1[R], a2[R], b2[R];
        load(a0, b0, kb);
        load(a1, b1, kb + 4 * R);
        // the destination, long before its value is needed
        at = tile_at(C, tl, pr, e0);
        if (o.beta && o.split == 1 && at) old = *at;
        for (int k0 = kb; k0 < ke; k0 += 12 * R) {
            load(a2, b2, k0 + 8 * R);
            work(a0, b0, k0);
            load(a0, b0, k0 + 12 * R);
            work(a1, b1, k0 + 4 * R);
            load(a1, b1, k0 + 16 * R);
            work(a2, b2, k0 + 8 * R);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) put(&red[(wave * 4 + q) * 64 + lane], c, q);
    }
    __syncthreads();
    if (o.split == 1) {
        if (!live) return;
        for (int e = e0; e < 256; e += es) {
            if (e > e0) {
                at = tile_at(C, tl, pr, e);
                if (o.beta && at) old = *at;
            }
            if (!at) continue;
            T s{};
            for (int w = 0; w < kw; ++w) add(s, red[(g * kw + w) * 256 + e]);
            T out = elem_scale(o.ar, o.ai, s);
            if (o.beta) add(out, old);
            *at = out;
        }
        return;
    }
    // Split over workgroups (kw = 4: one part of one tile, one element per
    // thread; the grid has no dead part): the parts meet in memory.  Parts and
    // counter are accessed by device-scope atomics only, which no cache holds
    // back, so no fence has to write back or drop the L2 (fences here: 10-15
    // us for the whole launch).  A part is complete before its workgroup is
    // counted, and only the workgroup counted last reads.
    T* W = (T*)o.m.work + (long long)tile * o.split * 256 + tid;
    T s{};
#pragma unroll
    for (int w = 0; w < 4; ++w) add(s, red[w * 256 + tid]);
    part_store(W + part * 256, s);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    int* last = (int*)red;
    if (tid == 0)
        *last = __hip_atomic_fetch_add(&o.m.arrived[tile], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == o.split - 1;
    __syncthreads();
    if (!*last) return;
    if (tid == 0) __hip_atomic_store(&o.m.arrived[tile], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // for the next launch
    if (o.beta && at) old = *at;
    s = T{};
#pragma unroll 8
    for (int p = 0; p < o.split; ++p) add(s, part_load(W + p * 256));
    if (!at) return;
    T out = elem_scale(o.ar, o.ai, s);
    if (o.beta) add(out, old);
    *at = out;
}

template <typename T>
__global__ __launch_bounds__(kFusedThreads, 4) void k_fused(const FItem* __restrict__ items, const FOp* __restrict__ ops,
                                                         FIo io) {
    __shared__ T red[kWaves * 256];
    unsigned long long* lds = (unsigned long long*)red;
    static_assert(kMaxChain * sizeof(FOp) <= sizeof red, "descriptors fit");
    const FItem it = items[blockIdx.x];
    stage_ops(ops + it.op, it.nops, io, lds);
    __syncthreads();
    const FOp o = staged_op(lds);
    if (o.kind == FK_GEMM) {
        __syncthreads();   // the partial tiles take the descriptor's place
        fused_gemm<T>(o, it.first, red);
    } else {
        fused_elements<T>(lds, o, it.first * kFusedThreads + (int)threadIdx.x);
    }
}

}  // namespace

// Loads the kernel's code onto the current device, which its first launch would
// do otherwise (some milliseconds, once per process).
hipError_t load_fused(bool real) {
    hipFuncAttributes a;
    return hipFuncGetAttributes(&a, real ? (const void*)k_fused<double> : (const void*)k_fused<double2>);
}

hipError_t launch_fused(const FItem* items, int nitems, const FOp* ops, const FIo& io, bool real, hipStream_t st) {
    if (nitems <= 0) return hipSuccess;
    if (real) k_fused<double><<<nitems, kFusedThreads, 0, st>>>(items, ops, io);
    else k_fused<double2><<<nitems, kFusedThreads, 0, st>>>(items, ops, io);
    return hipGetLastError();
}

}  // namespace fscc
