// schedule.hpp -- the order in which an operation list is launched (plain host
// code, no HIP).
//
// A schedule is a sequence of steps; a step is one operation on its own
// kernel, or a set of small operations that run in one fused launch
// (kernels_fused.hip).  An operation may join a fused step once everything it
// depends on ran in earlier steps, so the steps in order, one after the other
// on a stream, respect every dependency.
#pragma once

#include <algorithm>
#include <cstdint>
#include <stdexcept>
#include <vector>

#include "plan.hpp"

namespace fscc {

// Dependencies of an operation list through its buffers: operation k reads
// src, src2, every term source and, when it accumulates (beta = 1, diagonal
// and multiply forms), dst; it writes dst.  k depends on the last writer of
// every buffer it reads or writes (read after write, write after write) and
// on every reader of dst since that writer (write after read).  Buffers are
// separate allocations, so distinct ids never overlap.
inline std::vector<std::vector<int>> op_dependencies(const std::vector<Op>& ops) {
    std::vector<std::vector<int>> deps(ops.size());
    std::vector<int> last_w;
    std::vector<std::vector<int>> readers;
    auto grow = [&](int b) {
        if (b >= (int)last_w.size()) {
            last_w.resize(b + 1, -1);
            readers.resize(b + 1);
        }
    };
    for (size_t k = 0; k < ops.size(); ++k) {
        const Op& o = ops[k];
        std::vector<int> rd;
        for (int b : {o.src, o.src2})
            if (b >= 0) rd.push_back(b);
        for (int b : o.srcT)
            if (b >= 0) rd.push_back(b);
        if (o.beta || o.kind == OP_DIAG || o.kind == OP_MUL) rd.push_back(o.dst);
        std::vector<int>& d = deps[k];
        for (int b : rd) {
            grow(b);
            if (last_w[b] >= 0) d.push_back(last_w[b]);
        }
        if (o.dst >= 0) {
            grow(o.dst);
            if (last_w[o.dst] >= 0) d.push_back(last_w[o.dst]);
            for (int r : readers[o.dst]) d.push_back(r);
        }
        std::sort(d.begin(), d.end());
        d.erase(std::unique(d.begin(), d.end()), d.end());
        d.erase(std::remove(d.begin(), d.end(), (int)k), d.end());
        for (int b : rd) readers[b].push_back((int)k);
        if (o.dst >= 0) {
            last_w[o.dst] = (int)k;
            readers[o.dst].clear();
        }
    }
    return deps;
}

// One step: ops.size() == 1 and !fused: the operation on its own kernel;
// fused: chains of operations (each chain works on one destination, element by
// element, in order; a GEMM is a chain of its own).
struct ScheduleStep {
    bool fused = false;
    std::vector<std::vector<int>> chains;
};

// May operation k run in a fused launch?  It has to be small: the fused GEMM
// reads its operands once per 16 x 16 output tile.
//   * traffic of all tiles <= 48 MB (5 us at the rate the L2s deliver) and
//     padded work <= 0.4 Gflop (8 us at half the matrix peak): above, the
//     grouped tiles with operands shared through LDS are faster (twice both:
//     20/120 in eight irreps 0.7 % slower).  A real operation has less work
//     to share a launch's cost, and twice the traffic pays: 13/67 in three
//     irreps 207 us at 48 MB and 0.2 Gflop, 186 us at 96 MB and 0.4 Gflop (one
//     system measured);
//   * elementwise operations and reorders of up to 2^19 elements: above,
//     their own launch costs less than 5 % of their time (chains: small_ops).
inline bool fusable(const Op& o, bool real) {
    if (o.kind != OP_GEMM) return o.n <= (1 << 19);
    double bytes = 0.0, flops = 0.0;
    for (const GemmProblem& p : o.probs) {
        const double tiles = (double)((p.M + 15) / 16) * ((p.N + 15) / 16);
        bytes += tiles * p.K * 32 * (real ? 8 : 16);
        flops += tiles * p.K * 256 * (real ? 2 : 8);
    }
    return bytes <= (real ? 96e6 : 48e6) && flops <= 0.4e9;
}

// Waves of a 16 x 16 tile of a fused GEMM: kw waves in a workgroup, one per
// SIMD, times split workgroups.  The matrix pipe of a SIMD takes 1.7 us for 64
// k of a complex tile and 0.9 us for 128 k of a real one, so K is split down to
// that while the tiles alone do not give the chip its 4096 waves.  Parts of a tile on
// other workgroups have to meet through memory (2 us), so that split is for
// tiles that would keep a CU for longer than that (real 13/67, split above
// 1024 or 512 k: 208, 203 us; complex 8/24, above 512 or 256: no difference).
struct FusedSplit {
    int kw = 1, split = 1, tiles = 0;
};
inline FusedSplit fused_split(const Op& o, bool real) {
    FusedSplit f;
    int K = 0;
    for (const GemmProblem& p : o.probs) {
        f.tiles += ((p.M + 15) / 16) * ((p.N + 15) / 16);
        K = std::max(K, p.K);
    }
    const int kwave = real ? 128 : 64;
    while (f.kw < 4 && K > kwave * f.kw && (long long)f.tiles * f.kw < 4096) f.kw *= 2;
    if (f.kw == 4 && K > 512)
        f.split = std::min((K + 4 * kwave - 1) / (4 * kwave), std::max(1, 1024 / std::max(1, f.tiles)));
    return f;
}

// What may share a launch: 0: an operation on its own kernel, 1: any small
// one, 2: a larger elementwise operation or reorder (up to 2^30 elements, the
// kernel counts in 32 bits), in a chain only: a chain
// reads and writes its destination once (r2 of 40 occupied / 300 virtual
// spinors in 16 irreps collects five terms in 179 us instead of 218; the
// iteration 5040 -> 4999 us, 29/174 in seven irreps 4321 -> 4255, the (0,1)
// sector step 1860 -> 1780).
inline std::vector<char> small_ops(const std::vector<Op>& ops, const std::vector<char>& alone, bool real) {
    std::vector<char> small(ops.size(), 0);
    for (size_t k = 0; k < ops.size(); ++k)
        if (!alone[k]) small[k] = fusable(ops[k], real) ? 1 : ops[k].kind != OP_GEMM && ops[k].n <= (1 << 30) ? 2 : 0;
    return small;
}

// Most operations of a chain: their descriptors share a workgroup's LDS in the
// fused kernel (runtime.hpp checks that it has room for as many).
constexpr size_t kScheduleChain = 8;

// The schedule of an operation list.
// Elementwise operations on the same destination are chained when nothing
// reads the destination between them and the chains can still be ordered.
// Then, repeatedly: all small operations and all chains that are ready form one
// fused step; if there are none, every other ready operation follows as a step of its own, in
// list order.
inline std::vector<ScheduleStep> build_schedule(const std::vector<Op>& ops, const std::vector<char>& small) {
    const int n = (int)ops.size();
    const std::vector<std::vector<int>> deps = op_dependencies(ops);
    auto elementwise = [&](int k) { return small[k] && ops[k].kind != OP_GEMM; };
    auto reads = [&](int k, int b) {
        const Op& o = ops[k];
        return o.src == b || o.src2 == b || std::find(o.srcT.begin(), o.srcT.end(), b) != o.srcT.end();
    };
    std::vector<int> node(n, -1);   // chain of each operation
    std::vector<std::vector<int>> chain;
    // can the chains of operations 0..k be put in an order that respects every dependency?
    auto orderable = [&](int k) {
        const int m = (int)chain.size();
        std::vector<std::vector<int>> need(m);
        for (int j = 0; j <= k; ++j)
            for (int d : deps[j])
                if (node[d] != node[j]) need[node[j]].push_back(node[d]);
        std::vector<char> done(m, 0);
        for (int left = m, before = m + 1; left < before && left > 0;) {
            before = left;
            for (int c = 0; c < m; ++c)
                if (!done[c] && std::all_of(need[c].begin(), need[c].end(), [&](int d) { return done[d] != 0; })) {
                    done[c] = 1;
                    --left;
                }
            if (left == 0) return true;
        }
        return m == 0;
    };
    for (int k = 0; k < n; ++k) {
        // the last writer of the destination, if it can be continued
        int w = -1;
        bool read_since = false;
        for (int j = 0; j < k; ++j) {
            if (ops[j].dst == ops[k].dst) {
                w = j;
                read_since = reads(j, ops[k].dst);
            } else if (reads(j, ops[k].dst)) {
                read_since = true;
            }
        }
        if (elementwise(k) && w >= 0 && !read_since && elementwise(w) && ops[w].n == ops[k].n && !reads(k, ops[k].dst) && chain[node[w]].size() < kScheduleChain &&
            chain[node[w]].back() == w) {
            node[k] = node[w];
            if (!orderable(k)) node[k] = -1;
        }
        if (node[k] < 0) {
            node[k] = (int)chain.size();
            chain.emplace_back();
        }
        chain[node[k]].push_back(k);
    }
    const int m = (int)chain.size();
    std::vector<std::vector<int>> need(m);
    for (int c = 0; c < m; ++c)
        for (int k : chain[c])
            for (int d : deps[k])
                if (node[d] != c) need[c].push_back(node[d]);
    std::vector<char> done(m, 0);
    auto ready = [&](int c) {
        if (done[c]) return false;
        for (int d : need[c])
            if (!done[d]) return false;
        return true;
    };
    std::vector<ScheduleStep> steps;
    for (int left = m; left > 0;) {
        std::vector<int> fuse, single;
        for (int c = 0; c < m; ++c)
            if (ready(c)) (small[chain[c][0]] == 1 || chain[c].size() > 1 ? fuse : single).push_back(c);
        if (!fuse.empty()) {
            ScheduleStep s;
            s.fused = true;
            for (int c : fuse) s.chains.push_back(chain[c]);
            steps.push_back(std::move(s));
            for (int c : fuse) done[c] = 1;
            left -= (int)fuse.size();
        } else if (!single.empty()) {
            for (int c : single) {
                ScheduleStep s;
                s.chains.push_back(chain[c]);
                steps.push_back(std::move(s));
                done[c] = 1;
            }
            left -= (int)single.size();
        } else {
            throw std::logic_error("operation list cannot be ordered");
        }
    }
    return steps;
}

// Every operation on its own kernel, in list order.
inline std::vector<ScheduleStep> plain_schedule(size_t n) {
    std::vector<ScheduleStep> steps;
    for (size_t k = 0; k < n; ++k) steps.push_back(ScheduleStep{false, {{(int)k}}});
    return steps;
}

}  // namespace fscc
