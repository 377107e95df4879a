// Forward passes: causal (eq. 9-12), global read-out (eq. 5-6) and the K,V segment totals.
#include "la_block.h"
#include "la_launch.h"

namespace la {

hipError_t launch_pass_fwd(bool global, bool block, int D, int M, int dtype, const PassArgs &a, int nblocks,
                           hipStream_t s) {
    LA_DISPATCH(D, M, dtype, {
        if (block && !global) {
            if (a.tok_heads > 1) fwd_block_kernel<kD, kM, TT, true><<<nblocks, kWave * kFwdWaves, 0, s>>>(a);
            else fwd_block_kernel<kD, kM, TT><<<nblocks, kWave * kFwdWaves, 0, s>>>(a);
            return hipGetLastError();
        }
        if (a.tok_heads > 1) {
            if (global) causal_pass_kernel<kGlobal, kD, kM, TT, true><<<nblocks, kWave, 0, s>>>(a);
            else causal_pass_kernel<kFwd, kD, kM, TT, true><<<nblocks, kWave, 0, s>>>(a);
        } else {
            if (global) causal_pass_kernel<kGlobal, kD, kM, TT><<<nblocks, kWave, 0, s>>>(a);
            else causal_pass_kernel<kFwd, kD, kM, TT><<<nblocks, kWave, 0, s>>>(a);
        }
    });
    return hipGetLastError();
}

hipError_t launch_fwd_direct(int D, int M, int dtype, const PassArgs &a, const SegArgs &sa, int ndirect, int nsegs,
                             hipStream_t s) {
    LA_DISPATCH(D, M, dtype, {
        if (a.tok_heads > 1) fwd_direct_kernel<kD, kM, TT, true><<<ndirect + nsegs, kWave * kDirectWaves, 0, s>>>(a, sa, ndirect);
        else fwd_direct_kernel<kD, kM, TT><<<ndirect + nsegs, kWave * kDirectWaves, 0, s>>>(a, sa, ndirect);
    });
    return hipGetLastError();
}

hipError_t launch_segment_state(bool block, int D, int M, int dtype, const SegArgs &a, int nblocks,
                                hipStream_t s) {
    LA_DISPATCH(D, M, dtype, {
        if (block) {
            if (a.tok_heads > 1) segment_state_kernel<kD, kM, TT, true, 4><<<nblocks, 4 * kWave, 0, s>>>(a);
            else segment_state_kernel<kD, kM, TT, false, 4><<<nblocks, 4 * kWave, 0, s>>>(a);
            return hipGetLastError();
        }
        if (a.tok_heads > 1) segment_state_kernel<kD, kM, TT, true><<<nblocks, kWave, 0, s>>>(a);
        else segment_state_kernel<kD, kM, TT><<<nblocks, kWave, 0, s>>>(a);
    });
    return hipGetLastError();
}

}  // namespace la
