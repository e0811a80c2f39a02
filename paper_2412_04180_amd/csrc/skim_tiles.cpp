// The plan that shares the 256 x 256 output tiles of a product out to the compute units (host code).
#include "skim_tiles.h"

namespace {

// Estimated length of the plan for `rem` tiles in stages, and the plan itself: whole rounds of one workgroup per tile
// while there are as many tiles as workgroups; what is left either in one phase (every tile in floor(G / rem) parts)
// or first as many tiles as ceil(G / rem) parts each fill the chip with, then the rest likewise.
long long plan_rest(int rem, int G, int nstage, int maxsplit, int phase_cost, int depth, int *nts, int *sps, int &n) {
    n = 0;
    if (rem == 0) return 0;
    if (rem >= G || depth <= 1) {
        const bool all = depth <= 1;       // (the last phase takes what is left: a partly filled round)
        const int whole = all ? rem : rem - rem % G;
        nts[0] = whole;
        sps[0] = all && rem < G ? (G / rem < maxsplit ? G / rem : maxsplit) : 1;
        int k = 0;
        const long long c = (long long)((whole + G - 1) / G) * ((nstage + sps[0] - 1) / sps[0]) + phase_cost +
                            plan_rest(rem - whole, G, nstage, maxsplit, phase_cost, depth - 1, nts + 1, sps + 1, k);
        n = 1 + k;
        return c;
    }
    const int one = G / rem < maxsplit ? G / rem : maxsplit;
    const long long cost_one = (nstage + one - 1) / one + phase_cost;
    const int more = (G + rem - 1) / rem;
    if (more <= maxsplit && more > one) {
        int nts2[PLAN_MAX_PHASES], sps2[PLAN_MAX_PHASES], k = 0;
        const int take = G / more;
        const long long c = (nstage + more - 1) / more + phase_cost +
                            plan_rest(rem - take, G, nstage, maxsplit, phase_cost, depth - 1, nts2, sps2, k);
        if (c < cost_one) {
            nts[0] = take;
            sps[0] = more;
            for (int i = 0; i < k; ++i) {
                nts[1 + i] = nts2[i];
                sps[1 + i] = sps2[i];
            }
            n = 1 + k;
            return c;
        }
    }
    nts[0] = rem;
    sps[0] = one;
    n = 1;
    return cost_one;
}

}  // namespace

long long skim_make_plan(TilePlan &plan, int G, long long tiles, int nstage, int min_stages, int phase_cost, bool whole) {
    const int maxsplit = !whole && nstage / min_stages > 1 ? nstage / min_stages : 1;
    plan = TilePlan{};
    plan_rest((int)tiles, G, nstage, maxsplit, phase_cost, whole ? 1 : PLAN_SPLIT_PHASES, plan.ntile, plan.split, plan.nph);
    long long t = 0, slots = 0;
    for (int p = 0; p < plan.nph; ++p) {
        plan.tile0[p] = (int)t;
        t += plan.ntile[p];
        plan.slot0[p] = (int)slots;
        slots += (long long)plan.ntile[p] * plan.split[p];
    }
    return slots;
}
