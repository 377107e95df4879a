// The host side of the schedule (csrc/la_plan.h) on its own: reads calls from stdin, prints their plans.
//   in   target_waves min_chunks fold_max bwd_group block  BH N C M dtype tok_heads
//   out  nchunks nseg cps fold fwd_block bwd_block bwd_group  states_bytes(plan) causal_states_bytes causal_bwd_bytes
//        step_streams (of a decode step of BH sequences) steps_one_by_one (N decode steps of BH sequences) nt_outputs (causal, non-causal) fwd_direct
#include <cstdio>

#include "../paper_2006_16236_amd/csrc/la_plan.h"

int main() {
    la_plan::Tuning tn{};
    long BH;
    int N, C, M, t, heads;
    tn.stream = -1;
    while (std::scanf("%d %d %d %d %d %ld %d %d %d %d %d", &tn.target_waves, &tn.min_chunks, &tn.fold_max, &tn.bwd_group, &tn.block, &BH,
                      &N, &C, &M, &t, &heads) == 11) {
        const la_dtype dt = static_cast<la_dtype>(t);
        const la_plan::Plan p = la_plan::causal_plan(tn, BH, N, C, M, dt, heads);
        std::printf("%d %d %d %d %d %d %d %zu %zu %zu %d %d %d %d %d\n", p.nchunks, p.nseg, p.cps, p.fold, p.fwd_block, p.bwd_block, p.bwd_group,
                    p.nseg > 1 ? la_plan::states_bytes(BH, p, C, M) : 0, la_plan::causal_states_bytes(tn, BH, N, C, M),
                    la_plan::causal_bwd_bytes(tn, BH, N, C, M), la_plan::step_streams(BH, C, M, dt),
                    la_plan::steps_one_by_one(N, BH, C, M, dt), la_plan::nt_outputs(BH, N, C, M, dt, true), la_plan::nt_outputs(BH, N, C, M, dt, false),
                    p.fwd_direct);
    }
    return 0;
}
