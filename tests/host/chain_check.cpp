// Chains of a synthetic operation list (plain host code): n accumulating
// elementwise operations on one destination from n sources.  Returns the
// number of chains, -1 if one is longer than the fused kernel's limit or the
// operations are out of order.
#include <vector>

#include "plan.hpp"
#include "schedule.hpp"

using namespace fscc;

extern "C" int chain_check(int n, int* limit) {
    std::vector<Op> ops;
    for (int k = 0; k < n; ++k) {
        Op o;
        o.kind = OP_AXPBY;
        o.dst = 0;
        o.src = 1 + k;
        o.n = 1000;
        o.beta = k > 0;
        ops.push_back(o);
    }
    *limit = (int)kScheduleChain;
    int chains = 0, next = 0;
    for (const ScheduleStep& s : build_schedule(ops, std::vector<char>(n, 1)))
        for (const auto& c : s.chains) {
            ++chains;
            if (c.size() > kScheduleChain) return -1;
            for (int k : c)
                if (k != next++) return -1;
        }
    return next == n ? chains : -1;
}
