// Checks the launch schedules of every operation list of one system (plain
// host code): every operation appears once, everything it depends on ran in an
// earlier step or earlier in its own chain, chains share one destination and
// hold no GEMM beside others, and operations kept alone are.  Dependencies are
// derived here from the buffers, independently of the planner's.  Returns the
// number of violations; steps[i], fused[i]: steps and fused steps of list i.
#include <cstdint>
#include <vector>

#include "plan.hpp"
#include "schedule.hpp"

using namespace fscc;

static bool touches(const Op& o, int b) {
    if (o.src == b || o.src2 == b || o.dst == b) return true;
    for (int s : o.srcT)
        if (s == b) return true;
    return false;
}

static int check(const std::vector<Op>& list, const std::vector<char>& alone, bool real, int* nsteps,
                 int* nfused) {
    const std::vector<Op>& ops = list;
    const std::vector<ScheduleStep> st = build_schedule(ops, small_ops(ops, alone, real));
    const int n = (int)ops.size();
    std::vector<int> step(n, -1), pos(n, -1), chain(n, -1);
    int bad = 0, id = 0;
    *nsteps = (int)st.size();
    *nfused = 0;
    for (size_t k = 0; k < st.size(); ++k) {
        *nfused += st[k].fused;
        if (!st[k].fused && (st[k].chains.size() != 1 || st[k].chains[0].size() != 1)) ++bad;
        for (const auto& c : st[k].chains) {
            for (size_t q = 0; q < c.size(); ++q) {
                const Op& o = ops[c[q]];
                if (step[c[q]] >= 0) ++bad;
                step[c[q]] = (int)k;
                pos[c[q]] = (int)q;
                chain[c[q]] = id;
                const int j = c[q];
                if (st[k].fused && (alone[j] || !(fusable(list[j], real) || (c.size() > 1 && o.kind != OP_GEMM)))) ++bad;
                if (c.size() > 1 && (o.kind == OP_GEMM || o.dst != ops[c[0]].dst || o.n != ops[c[0]].n)) ++bad;
            }
            ++id;
        }
    }
    for (const Op& o : list) {
        const FusedSplit f = fused_split(o, real);
        if (f.kw < 1 || f.kw > 4 || (f.kw & (f.kw - 1)) || f.split < 1 || (f.split > 1 && f.kw != 4)) ++bad;
    }
    for (int k = 0; k < n; ++k) {
        if (step[k] < 0) ++bad;
        // two operations of which one writes a buffer the other touches keep their order
        for (int j = 0; j < k; ++j) {
            if (!touches(ops[k], ops[j].dst) && !touches(ops[j], ops[k].dst)) continue;
            const bool before = step[j] < step[k] || (chain[j] == chain[k] && pos[j] < pos[k]);
            if (!before) ++bad;
        }
    }
    return bad;
}

extern "C" int schedule_check(int nocc, int nvirt, int G, const int32_t* irrep, const double* eps, int nact,
                              const int32_t* active, int keep_every, int real, int* steps, int* fused, int* count) {
    System S;
    S.nocc = nocc;
    S.nvirt = nvirt;
    S.G = G;
    S.irrep.assign(irrep, irrep + nocc + nvirt);
    S.eps.assign(eps, eps + nocc + nvirt);
    S.active.assign(active, active + nact);
    Plan P;
    build_plan_ccsd(S, P);
    int bad = 0, i = 0;
    for (std::vector<Op>* L : {&P.ops, &P.ops01_prep, &P.ops01, &P.ops02_prep, &P.ops02}) {
        std::vector<char> alone(L->size(), 0);
        if (keep_every > 0)
            for (size_t k = 0; k < alone.size(); k += keep_every) alone[k] = 1;
        bad += check(*L, alone, real != 0, &steps[i], &fused[i]);
        count[i] = (int)L->size();
        ++i;
    }
    return bad;
}
