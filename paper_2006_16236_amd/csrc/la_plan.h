// Host side of the segment schedule: how a call cuts its sequences, which kernels take the pieces, and the
// workspace that follows from it.  Plain C++ without a GPU header; every function takes the tuning values as an
// argument, so that a call works from one snapshot of them.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include "../../include/la.h"

namespace la_plan {

constexpr int kChunk = 16;                                        // tokens per chunk (la_device.h)
constexpr int kBlk = 32;                                          // tokens per block (la_block.h)
constexpr int kDirectTokens = 256;                                // most tokens of fwd_direct_kernel (la_block.h)
constexpr int kDirectGroups = 256;                                // most workgroups of it: one per CU
constexpr int state_stride(int D, int M) { return D * M + D; }    // floats per state (la_passes.h)

// ---- schedule ---------------------------------------------------------------------------------
// One wavefront (forward) or one two-wave workgroup (backward) walks one segment of one
// sequence.  MI355X holds 256 CUs x 4 SIMDs x 2 such waves; a sequence is cut into segments
// only as far as needed to reach that many waves, never into segments shorter than a couple of
// chunks, and not at all once the sequences alone fill half the machine.
struct Plan {
    int nchunks, nseg, cps;
    bool fold;      // few segments per sequence: no scan launch, every pass adds up the
                    // segment totals before (after) its own segment itself
    bool fwd_block; // the forward (and its segment sums) by the workgroup kernels of la_block.h
    bool bwd_block; // the causal backward
    bool fwd_direct; // the forward from no state by fwd_direct_kernel, the segment totals in the same launch
    int bwd_group;  // how many of the forward's segments a workgroup of the backward takes
    // Whether the call fetches its tiles with non-temporal loads.  A step sweeps Q, K, V (and dO) several
    // times, one kernel after the other.  Where those tensors fit the last-level cache (256 MB) the
    // later sweeps find them there if the loads are plain (measured: MNIST / CIFAR shapes 2 % and 9 %
    // faster than with non-temporal loads); where they do not, the two kinds are equally fast for fp32
    // tensors and plain loads 1.5 % faster for bf16 ones (N = 65536).  So plain loads are the default
    // and LA_STREAM_LOADS=1 is there for measuring.  (How the outputs are stored: nt_outputs; the segment states are always
    // loaded plain.)
    int nt_loads;
};

// The schedule's knobs.  The environment is read once, at the first call that needs a value (and
// again only on la_tuning_reload): a workspace query and the calls that use the workspace then see
// the same values, and no entry point calls getenv while another thread changes the environment.
struct Tuning {
    int target_waves;   // LA_TARGET_WAVES
    int min_chunks;     // LA_MIN_SEG_CHUNKS
    int fold_max;       // LA_FOLD_MAX_SEGS
    int bwd_group;      // LA_BWD_SEG_GROUP, 0 = by head size
    int stream;         // LA_STREAM_LOADS: 0, 1, or -1 = by tensor size
    int block;          // LA_BLOCK_KERNELS: 0 never, 1 wherever they exist, or -1 = by size
};

inline Plan make_plan(const Tuning &tn, long BH, int N) {
    const int target_waves = tn.target_waves;
    const int min_chunks = tn.min_chunks;
    Plan p;
    p.nchunks = (N + kChunk - 1) / kChunk;
    long want = (target_waves + BH - 1) / BH;
    long maxseg = p.nchunks / min_chunks;
    if (maxseg < 1) maxseg = 1;
    long nseg = want < 1 ? 1 : (want > maxseg ? maxseg : want);
    // Cutting costs a second sweep over K, V (and Q, dO) plus the scan: measured on MI355X it
    // pays from four segments per sequence on; with half the target already there, don't cut.
    if (2 * BH >= target_waves) nseg = 1;
    p.cps = (int)((p.nchunks + nseg - 1) / nseg);
    p.nseg = (p.nchunks + p.cps - 1) / p.cps;
    p.fold = p.nseg > 1 && p.nseg <= tn.fold_max;
    p.nt_loads = tn.stream == 1 ? 1 : 0;
    p.fwd_block = p.bwd_block = p.fwd_direct = false;
    p.bwd_group = 0;      // see backward_group
    return p;
}

// How many of the forward's segments one workgroup of the backward takes.  The backward's kernels
// run two waves per workgroup; with a 64-wide head dimension they need so many registers that
// two waves fill a SIMD, half as many workgroups fill the machine, and taking the segments in
// pairs is 10 % faster.  At D = M = 32 four waves fit a SIMD and the finer cut wins.
inline int backward_group(const Tuning &tn, int C, int M) {
    const int g = tn.bwd_group;
    if (g == 0) return (C == 32 && M == 32) ? 1 : 2;
    return g == 1 ? 1 : 2;
}

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

inline size_t esize(la_dtype t) { return (t == LA_BF16 || t == LA_BF16_FEATURES) ? 2 : 4; }

inline size_t states_bytes(long BH, const Plan &p, int D, int M) {
    return align256((size_t)BH * p.nseg * state_stride(D, M) * sizeof(float));
}

// The plan of a causal call: which kernels, and the cut that suits them.  The workgroup kernels
// (la_block.h) put four or eight waves on a segment, so a quarter as many segments fill the machine
// (512 workgroups, two per CU), in whole 32-token blocks: fewer, longer segments, hence less state to
// write, scan and read.  The wave kernels (la_passes.h) have the shorter chain per token and win
// where segments are long.  Measured on MI355X, step times wave / workgroup kernels in us (B*H x N):
//   fp32, D = M = 64   16 x 65536  1048/1019   16 x 16384  286/251   16 x 8192  162/137   16 x 2048  81/55
//   bf16, D = M = 64   16 x 65536   709/568    16 x 16384  193/150   16 x 8192  121/88    16 x 2048  66/44
//   fp32, D = M = 32   16 x 65536   462/464    16 x 16384  123/115   16 x 8192   76/66    16 x 2048  36/32
//   bf16, D = M = 32   16 x 65536   302/305    16 x 16384   91/84    16 x 8192   60/52    16 x 2048  34/28
//   fp32, 64 x 32      16 x 65536   750/712    16 x 16384  185/176   16 x 8192  111/98    16 x 2048  57/40
//   bf16, 64 x 32      16 x 65536   529/457    16 x 16384  147/122   16 x 8192   92/72    16 x 2048  51/37
//   fp32, 32 x 64      16 x 65536   721/671    16 x 16384  175/161   16 x 8192  105/90    16 x 2048  52/38
//   bf16, 32 x 64      16 x 65536   475/389    16 x 16384  133/101   16 x 8192   84/63    16 x 2048  45/35
// (wave / workgroup as LA_BLOCK_KERNELS=0 / 1 forces them.)
// so the line lies at 512 tokens per segment (fp32 with D = M = 64, bf16 with a 64-wide head dimension) or
// 256 (fp32 with a 32-wide D or M, where the two were within 2 to 4 % at 512, and bf16 32 x 32).  The fp32 lines were
// drawn while the workgroup backward had four waves and the wave kernels were ahead at 16 x 65536 (1028/1047, 736/767, 702/710);
// with eight they could lie higher for a 64-wide D or M.  The line of bf16
// 32 x 32 heads could lie higher: at 512 tokens per segment they take 0.92 of the wave kernels' step, 100 x 2000
// 83/71 us, and only the forward is slower (31/34 us at 16 x 16384); it was drawn when the backward took 0.97.
// Above it bf16 tensors with a 64-wide head dimension keep the wave kernel in the forward only (16 x 65536,
// D = M = 64: forward 198/218 us, backward 470/372; 64 x 32 132/178, 349/298; 32 x 64 128/145, 303/251).
// As many segments as fill the machine, not one more: 52 sequences of 3524 tokens in 10 pieces are 520 workgroups
// for 512 places, and the step took 289 us (wave kernels 222, 9 pieces 218).  One piece more only where the
// shorter segments are within the lines above and the second round is not nearly empty, or three pieces in all
// (two / three pieces: 200 x 1340 fp32 430/333, 175 x 1248 324/287; six of 96 x 2944, 576 workgroups, bf16
// forward 46 -> 64); bf16 32 x 32 heads, of which a CU holds three or four workgroups, may always have it
// (211 x 480 step 46/41).  257 to 383 sequences, which alone leave a third of the places empty, in
// three or two pieces (fp32 D = M = 64, 257 .. 320: whole 0.92 of the wave kernels' time, two 0.87, three 0.76).
// Short segments: where one workgroup per CU does with at most eight chunks each (ten for one segment per
// sequence, four where a sequence has more than four segments), two per CU gain nothing and double the
// states.  Two / one per CU in us (B*H x N, D = M = 64):
//   fp32 forward  40 x 256  20.7/13.1   64 x 512  27.5/19.3   step  160 x 128  52.0/38.2   64 x 480  64.6/52.4
//   bf16 forward  40 x 256  18.7/11.5   110 x 128  15.0/10.5  step  160 x 128  31.2/24.0   64 x 480  53.9/36.6
// (96 x 300 in ten chunks, 32-wide heads: step 27.1/30.1; 80 x 384, D = 64, M = 32: step 37.6/40.3.)  Up to 64
// tokens one segment does (forward of one sequence, D = M = 32 6.3/3.9 us, bf16 7.6/4.9; the step of fp32 tensors
// with D = 64, M = 32 17.2/17.8: those only when the batch fills a quarter of the CUs).
// Sequences are left whole from 384 on (from 256 if they are short: 256 x 512 136 us, 128 x 1024 in
// four pieces 135), narrow heads of more than 1024 tokens from 512 (bf16 406 x 1711 whole took 1.08 of the
// wave kernels' step when that line was drawn, 0.92 with the present backward, forward 1.25).  Whole sequences, each kernel by what fills the machine
// (fp32 D = M = 64, forward / dQ / dV+dK in us):
//   1024 x 1024  wave 337 / 292 / 330   workgroup 248 / 296 / 359
//   2048 x 512   wave 213 / 341 / 414   workgroup 229 / 271 / 324
//   2048 x 512, D = M = 32   wave 113 / 133 / 144   workgroup 105 / 132 / 154
//   64 x 32   1024 x 1024  wave 227 / 229 / 227   workgroup 167 / 203 / 240     2048 x 512  152 / 279 / 252   167 / 210 / 234
//   32 x 64   1024 x 1024  wave 201 / 208 / 228   workgroup 154 / 189 / 238     2048 x 512  152 / 216 / 255   158 / 184 / 235
// (Forced.  The lines were drawn with the four-wave backward; wave kernels that they keep and that are behind now: backward 2048 x 512
// 64 x 32 531/444, 32 x 64 471/419, 1024 x 1024 456/443 and 436/427, forward 2048 x 512, D = M = 32 113/105.)
// Workgroup / wave kernels of whole sequences, geometric mean over drawn lengths:
//   bf16 forward from 1024 on     D = M = 64  1.09 .. 1.31   64 x 32  1.15 .. 1.52   32 x 32  1.03 .. 1.22   32 x 64  0.88
//   backward with M = 32, fp32, from 1434 on  1.04 .. 1.24 (64 x 32 with four waves; with eight 0.82 .. 0.98, 300 to 1000 tokens)
//   bf16 64 x 32, 513 .. 640 of more than 512 tokens (wave kernels in several pieces)  step 1.06, forward 1.08; with
//   the present backward 550 x 700 has 0.87 and 0.94: the rule that keeps the wave kernels there could go
// A block is 32 tokens: of one chunk, or three, half a block is padding, and from 256 or 512 sequences on that
// is not hidden (fp32 979 x 16 forward 5.5/9.7, bf16 1260 x 40 9.7/13.8; three chunks of bf16 D = M = 64 keep
// the backward, 0.73 .. 0.77 of the wave kernels' time at 1100 .. 1400 x 40).  One block in all has no next one to
// fetch meanwhile: from 769 sequences on (a fourth per CU) workgroup / wave kernels, 24 tokens
//   bf16 D = M = 64  forward 1.13 .. 1.19, step with only the backward by workgroups 0.90, beyond 1024 0.75 .. 0.86;  other
//   heads forward 1.01 .. 1.17, step 0.91 .. 1.03, from 1536 on with only the backward 0.93 .. 1.02 (the line was drawn when
//   they took 1.12 .. 1.27, 0.98 .. 1.06, 0.91 .. 1.05)
//   fp32 D = M = 64  forward 1.07, step with the wave backward 0.92, beyond 1024 with either 0.83;  other heads 1.06 .. 1.20,
//   0.95 .. 1.06, beyond 1024 forward 0.91 .. 1.00
// (768 sequences: all 0.83 .. 0.97 but the bf16 forward, 0.99 .. 1.08).
// Left as they are: 257 .. 383 sequences of 257 .. 512 narrow tokens (step 0.81 .. 1.16 of the wave kernels' time,
// forward 0.67 .. 0.95) and fp32 32-wide D, 513 .. 700 sequences of more than 512 tokens (step 1.01 .. 1.10,
// forward 0.70 .. 0.88): every plan that helps the one harms the other.
// It never has more segments than make_plan's, which size the workspaces.
// (The polynomial map is cut like fp32 tensors of 64 features.)
// tok_heads: H of token-major tensors, else 0.  The workgroup kernels address the 32 tokens of a block with
// 32-bit byte offsets, which token-major tensors of a few hundred thousand heads exceed; the wave kernels do not.
inline Plan causal_cut(const Tuning &tn, long BH, int N, int C, int M, la_dtype t, int tok_heads) {
    Plan wave = make_plan(tn, BH, N);
    wave.bwd_group = backward_group(tn, C, M);
    const int64_t block_bytes = (int64_t)kBlk * (tok_heads > 1 ? tok_heads : 1) * (C > M ? C : M) * (int64_t)esize(t);
    if (tn.block == 0 || block_bytes > INT32_MAX) return wave;
    const long target = tn.target_waves >= 4 ? tn.target_waves / 4 : 1;
    const long min_chunks = tn.min_chunks > 2 ? tn.min_chunks : 2;
    const long waves = tn.target_waves;
    const bool bf16 = esize(t) == 2, narrow = C == 32 && M == 32, widest = C == 64 && M == 64;
    const int longest = (bf16 ? !narrow : widest) ? 512 : 256;     // tokens per segment
    Plan p = wave;
    // p.cps: at least make_plan's, so that there are never more segments than its
    auto at_least = [&](long chunks) { if (p.cps < chunks) p.cps = (int)chunks; };
    // tokens per segment if a sequence is cut into `pieces`
    auto tokens = [&](long pieces) {
        long chunks = (p.nchunks + pieces - 1) / pieces;
        if (chunks < wave.cps) chunks = wave.cps;
        return kChunk * (chunks + (chunks & 1));
    };
    const long up = (target + BH - 1) / BH;
    long pieces = bf16 && narrow ? up : BH < target ? target / BH : 1;
    if (N > 512) {
        if (2 * BH > target && 4 * BH < 3 * target) pieces = 2 * target / BH;
        else if ((up <= 3 || 7 * up * BH >= 8 * target) && tokens(pieces) > longest && tokens(up) <= longest) pieces = up;
    }
    at_least((p.nchunks + pieces - 1) / pieces);
    at_least(min_chunks);
    const long per_cu = target / (2 * BH);                  // segments a sequence may have at one per CU
    if (per_cu > 0) {
        const long chunks = (p.nchunks + per_cu - 1) / per_cu;
        const bool fills = 8 * BH * per_cu > 3 * target;    // more than three quarters of the CUs
        const int limit = per_cu > 4 ? 4 : per_cu == 1 && 8 * BH >= 3 * target ? 10 : bf16 || fills || per_cu == 1 ? 8 : 4;
        if (chunks <= limit) at_least(chunks);
    }
    const bool shortest = N <= 64 && (bf16 || C == 32 || 8 * BH >= target);
    if (shortest || (2 * BH >= target && N <= 512) || p.cps > p.nchunks) p.cps = p.nchunks;
    p.cps += p.cps & 1;
    p.nseg = (p.nchunks + p.cps - 1) / p.cps;
    p.fold = p.nseg > 1 && p.nseg <= tn.fold_max;
    p.fwd_block = p.bwd_block = true;
    p.bwd_group = tn.bwd_group == 2 ? 2 : 1;
    if (tn.block == 1) return p;
    if (p.nseg > 1) {
        if (p.cps * kChunk <= longest) return p;
        if (bf16 && !narrow) {
            wave.bwd_block = true;
            // four of the forward's segments each where that is within the places, else two (bf16 64 x 32,
            // 150 x 4096: four make 600 workgroups and took 1.06 of the wave kernels' step where two took 0.90; two now
            // take 0.80, 300/373 us)
            wave.bwd_group = tn.bwd_group != 0 ? (tn.bwd_group == 1 ? 1 : 2) : BH * ((wave.nseg + 3) / 4) > target ? 2 : 4;
            if (wave.bwd_group == 1) {       // its workgroups take whole blocks
                wave.cps += wave.cps & 1;
                wave.nseg = (wave.nchunks + wave.cps - 1) / wave.cps;
                wave.fold = wave.nseg > 1 && wave.nseg <= tn.fold_max;
            }
        }
        return wave;
    }
    // whole sequences
    if (narrow && BH < target && N > 1024) return wave;
    if (bf16 && C == 64 && M == 32 && N > 512 && BH > target && 4 * BH <= 5 * target) return wave;
    const bool one = p.nchunks == 1, three = p.nchunks == 3;
    if ((one && 2 * BH >= target) || (three && BH >= target)) {
        p.fwd_block = false;
        p.bwd_block = bf16 && widest && three && 2 * BH >= waves;
        return p;
    }
    if (p.nchunks == 2 && 2 * BH > 3 * target && (bf16 ? 4 * BH < 3 * waves : 2 * BH <= waves)) {
        p.fwd_block = !bf16 && widest;
        p.bwd_block = bf16 && widest;
        return p;
    }
    // one wave per sequence (forward) fills three quarters of the machine from 1536 on, two waves per sequence
    // (backward) nearly all of it at 1024
    p.fwd_block = bf16 && (C == 64 || narrow) ? 2 * BH < waves : 4 * BH < 3 * waves;
    const bool one_round = 16 * BH >= 7 * waves && 2 * BH <= waves;
    p.bwd_block = bf16 || !(one || one_round || (C == 32 && 2 * BH > waves) || (M == 32 && 10 * BH > 7 * waves));
    return p;
}

// ... and whether the forward of short sequences goes by definition (fwd_direct_kernel: one launch, 32 queries per
// workgroup, up to eight blocks of 32 keys).  Its work grows with the square of the length, so it is for launches that
// leave compute units idle: up to one workgroup on each, beyond that it loses (fp32 D = M = 64, segments / direct in us:
// 64 x 96, 192 workgroups, 10.6/8.4; 32 x 256, 256 workgroups, 17.0/11.6; 128 x 96, 384, 11.7/12.1; 64 x 256, 512,
// 13.9/19.0; bf16 32 x 256 15.7/10.3, 64 x 256 12.5/16.1).  One sequence of 256: fp32 D = M = 32 7.5/5.5, D = M = 64
// 10.7/8.2, bf16 9.8/6.6; of 65: 6.3/3.9, 9.6/4.9, 8.2/4.5.  Up to 64 tokens of bf16 or of a 32-wide D, one segment in
// one launch is as fast (3.8/3.9, bf16 4.4/4.5) and stays.  Calls that carry a state in or out go by segments.
// (The workgroups counted are the queries'; those of the segment totals come behind them.  Both layouts and all element
// types, 33 to 256 tokens, 1 to 256 workgroups, 2772 calls: direct takes 0.44 to 1.01 of the segments' time, medians
// 0.55 (bf16 features, 32-wide D) to 0.75 (fp32, token-major, D = 64); the polynomial map 0.65 and, token-major, 0.70.)
inline Plan causal_plan(const Tuning &tn, long BH, int N, int C, int M, la_dtype t, int tok_heads) {
    Plan p = causal_cut(tn, BH, N, C, M, t, tok_heads);
    const long groups = BH * ((N + kBlk - 1) / kBlk);
    const bool short_one = N <= kBlk || (N <= 2 * kBlk && (esize(t) == 2 || C == 32));
    p.fwd_direct = tn.block == -1 && p.fwd_block && !short_one && N <= kDirectTokens && groups <= kDirectGroups;
    return p;
}

// What a causal call asks its caller for: the states of make_plan's segments
inline size_t causal_states_bytes(const Tuning &tn, long BH, int N, int C, int M) {
    const Plan p = make_plan(tn, BH, N);
    return p.nseg > 1 ? states_bytes(BH, p, C, M) : 0;
}

// ... and a backward: 1/den, delta, and den if it is recomputed; the S and R states
inline size_t causal_bwd_bytes(const Tuning &tn, long BH, int N, int C, int M) {
    return 3 * align256((size_t)BH * N * sizeof(float)) + 2 * causal_states_bytes(tn, BH, N, C, M);
}
// non-causal: the two grand totals; den if it is recomputed
inline size_t global_bwd_bytes(const Tuning &tn, long BH, int N, int C, int M) {
    return 2 * states_bytes(BH, make_plan(tn, BH, N), C, M) + align256((size_t)BH * N * sizeof(float));
}

// Whether a call's outputs leave with non-temporal stores, where that goes by size: bf16 rows (16 bytes per lane), and
// the element-wise stores of fp32 calls with the caller's features (all other fp32 stores always do, two-byte ones never).
// The call's own next kernel reads faster, but what reads the outputs behind the call no longer finds them in the
// last-level cache.  The time with plain stores over that with non-temporal ones, token-major, H = 8, means over 1001, 3072 and 12000
// tokens, by MB of the wider outputs: the step by itself / the forward and a projection of O / the step with sums of O, dQ, dK, dV
// with other tensors / the step with the projection and the weight and input gradients of dQ, dK, dV:
//   bf16 causal 64 x 64   13 1.04 .97 .98 .87   32 1.01 .97 1.01 .99   48 1.04 .98 1.01 .99   64 1.04 1.00 1.00 1.00 (8192
//               tokens 1.03 .97 .97 1.00)   80 1.04 1.02 1.00 1.00   96 1.02 1.01 .99 1.00   128 1.02 1.01 1.00 1.00
//               64 x 32   32 1.01 .99 1.00 .98   48 1.02 .99 1.01 1.00   64 1.02 .99 1.01 1.00   96 1.02 .99 1.00 1.00   128 1.01 1.00 1.00 1.00
//               32 x 64   32 1.00 .95 1.00 1.00   64 1.04 .99 1.01 1.00   96 1.05 1.01 1.00 1.00   128 1.01 1.00 1.00 1.00
//   bf16 non-causal 64 x 64   13 1.03 .97 1.00 .91   64 1.02 1.00 .98 1.00   96 1.00 1.00 .98 1.00   128 1.02 1.01 1.00 1.00
//               64 x 32   64 1.00 1.00 .98 1.00   96 1.00 .96 .98 1.00     32 x 32   64 1.00 .97 .97 .99   128 1.00 1.00 .99 .99
//   given features (one call each)   non-causal 8 x 1024 17 1.00 1.00 .99 .97   8 x 3072 50 1.10 1.00 1.01 1.00
//               causal 33 x 1000 68 1.04 1.00 1.02 1.01   3 x 16384 101 1.04 1.03 1.02 1.00
// (bf16, 4 x 3072 tokens, 64 x 64, us: step 73.4/70.7, with projection and gradients 352/404.)
inline bool nt_outputs(long BH, int N, int C, int M, la_dtype t, bool causal) {
    const size_t mb = (size_t)BH * N * (C > M ? C : M) * esize(t) >> 20;
    if (esize(t) == 2) return C == 64 && (causal ? mb >= 80 : M == 64 && mb >= 128);
    return t != LA_F32_FEATURES || mb >= 64;
}

// Whether a decode step's states pass the caches by (non-temporal loads and stores; one without the other is not
// faster).  What is left of them in the last-level cache (256 MB) when a step has gone through them serves the next
// step; where they are so much larger that little of it does, they had better pass.  fp32 calls had better from the
// size of the L2s (32 MB) on already: with plain ones they are slower there than with the loads and stores of the
// sweep in turn, bf16 calls are not.  Plain / non-temporal in us, D = M = 64, one state again and again, by MB of S:
//   fp32  23 6.7/6.6  31 10.1/9.6  34 11.7/10.8  67 24.4/21.6  134 45.3/42.6  201 67.3/63.8  229 76/73  268 81/86
//         295 93/94  341 120/108  537 201/173    in turn  31 9.4  34 10.7  67 23.6  134 43.6  201 63.6  229 72  268 86
//   bf16  34 9.4/10.8  67 21.5/21.3  134 41.0/42.0  201 60/63  268 81/84  295 91/93
// Four states in turn, as of the layers of a model: fp32 33 13.4/12.2, 100 37/33, 200 74/64; bf16 11.6/12.1, 37/33, 73/64.
// Other head sizes: fp32 64 x 32 34 12.9/11.6, 67 25.2/22.5; 32 x 32 34 15.4/14.6.
inline bool step_streams(long BH, int D, int M, la_dtype t) {
    const size_t mb = (size_t)BH * D * M * sizeof(float) >> 20;
    return mb >= 288 || (esize(t) == 4 && mb >= 24 && mb < 240);
}

// Which kernel takes the steps of a launch: one at a time, or a batch of up to eight (and more batches after it).
// One at a time / in batches, us on the device (B*H sequences, fp32 unless noted):
//   T = 1   64 x 64  512 4.1/4.2  1024 5.8/6.9  2048 11.0/11.5  4096 23.9/22.9  8192 43.5/42.2  16384 81/85 (polynomial 82/96)
//                    bf16 4096 21.6/22.7  8192 41.0/41.7  16384 79/85
//           32 x 32  1024 3.4/3.4  8192 14.7/17.7   64 x 32  8192 24.7/24.9  bf16 21.9/25.0   32 x 64  8192 24.4/22.9  bf16 21.5/22.7
//   T = 2   64 x 64  512 4.7/4.4  1024 6.8/7.2  2048 11.9/13.0  3000 19.8/18.5  4096 25.1/23.7  bf16 2048 10.8/12.1  8192 41.9/42.5
//           32 x 32  512 3.3/3.0  8192 19.9/18.6   32 x 64  8192 27.9/24.0  bf16 23.7/23.6
//           64 x 32  2048 8.3/7.2  4096 15.8/15.7  8192 26.9/26.2  bf16 2048 8.4/7.4  4096 14.4/15.3  8192 24.8/25.9  polynomial 28.6/30.3
//   T = 3   64 x 64  1024 8.0/7.5  4096 27.5/24.4  bf16 4096 24.4/23.7   32 x 32  4096 14.0/9.7   64 x 32  4096 18.7/16.2
inline bool steps_one_by_one(int steps, long BH, int D, int M, la_dtype t) {
    const bool widest = D == 64 && M == 64, fp32 = esize(t) == 4;
    if (steps == 1) return !(widest && fp32 && BH >= 4096 && BH < 15360);     // (64 to 240 MB of S)
    if (steps == 2 && widest) return BH >= 1024 && !(fp32 && BH >= 2560);
    return steps == 2 && D == 64 && BH >= 4096;
}

}  // namespace la_plan
