// Small bandwidth-bound kernels: the scan over segment states and the recurrent
// decode step (eq. 16-20).
#include "la_launch.h"

namespace la {

// ---- scan over the segment states of each sequence ------------------------------------------
// state: [BH, nseg, stride], stride a multiple of 4.  A thread owns four consecutive elements
// (16-byte loads and stores); a workgroup takes 4 * 256 / PARTS consecutive elements of one
// sequence, and its PARTS groups of threads split the nseg slots into PARTS consecutive runs.
// Each group first sums its run (all loads independent), the run totals are exchanged through
// LDS, then the group walks its run again and writes the exclusive prefix.
// Slots are visited in scan order: ascending for the prefix, descending for the suffix.
// Fixed order: deterministic.  PARTS grows with nseg (1 for a handful of slots: every thread
// then has elements of its own and no thread idles).
template <int PARTS>
__global__ __launch_bounds__(256) void scan_states_kernel(float *state, int nseg, int stride,
                                                          int mode, const float *init_S,
                                                          const float *init_z, int DM) {
    constexpr int EPW = 256 / PARTS;          // threads (quads of elements) per run
    __shared__ f32x4 part_total[PARTS][EPW];
    const int el = threadIdx.x % EPW, part = threadIdx.x / EPW;
    const int e = 4 * (blockIdx.x * EPW + el);
    const bool live = e < stride;
    float *p = state + (size_t)blockIdx.y * nseg * stride + (live ? e : 0);
    const bool reverse = mode == kScanReverse;
    const int per = (nseg + PARTS - 1) / PARTS;
    const int k0 = min(part * per, nseg), k1 = min(k0 + per, nseg);
    // the last slot in scan order holds no total (nobody reads past it): never read it
    const int klast = mode == kScanTotal ? nseg : nseg - 1;
    const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
    auto slot = [&](const int k) { return reinterpret_cast<f32x4 *>(p + (size_t)(reverse ? nseg - 1 - k : k) * stride); };

    // eight independent loads in flight per thread (a plain loop waits for each in turn)
    constexpr int kBlock = 8;
    // a run of one block (up to 64 slots) is kept and read once (16 slots x 32 sequences 7.5 -> 7.1 us,
    // 20 slots x 24 sequences 7.8 -> 7.3)
    const int kread = min(k1, klast);
    const bool kept = per <= kBlock;
    f32x4 total = zero4, t[kBlock] = {};
    for (int kb = k0; kb < kread; kb += kBlock) {
#pragma unroll
        for (int j = 0; j < kBlock; ++j) t[j] = *slot(min(kb + j, kread - 1));
#pragma unroll
        for (int j = 0; j < kBlock; ++j) total += kb + j < kread ? t[j] : zero4;
    }
    // the scan starts from the caller's initial state when there is one (forward prefix only)
    f32x4 acc = zero4;
    if (init_S != nullptr && live)
        acc = e < DM ? *reinterpret_cast<const f32x4 *>(init_S + (size_t)blockIdx.y * DM + e)
                     : *reinterpret_cast<const f32x4 *>(init_z + (size_t)blockIdx.y * (stride - DM) + (e - DM));
    if constexpr (PARTS > 1) {
        part_total[part][el] = total;
        __syncthreads();
        for (int q = 0; q < part; ++q) acc += part_total[q][el];
    }
    if (mode == kScanTotal) {
        if (part == PARTS - 1 && live) *reinterpret_cast<f32x4 *>(p) = acc + total;
        return;
    }
    for (int kb = k0; kb < k1; kb += kBlock) {
        if (!kept) {
#pragma unroll
            for (int j = 0; j < kBlock; ++j) {
                const int k = min(kb + j, k1 - 1);
                t[j] = k < klast ? *slot(k) : zero4;
            }
        }
#pragma unroll
        for (int j = 0; j < kBlock; ++j) {
            const int k = kb + j;
            if (k < k1) {
                if (live) *slot(k) = acc;
                acc += t[j];
            }
        }
    }
}

hipError_t launch_scan(float *state, int BH, int nseg, int stride, int mode, hipStream_t s,
                       const float *init_S, const float *init_z, int DM) {
    const int quads = (stride + 3) / 4;
    if (nseg <= 4) {
        dim3 grid((quads + 255) / 256, BH);
        scan_states_kernel<1><<<grid, 256, 0, s>>>(state, nseg, stride, mode, init_S, init_z, DM);
    } else if (nseg <= 16) {
        dim3 grid((quads + 127) / 128, BH);
        scan_states_kernel<2><<<grid, 256, 0, s>>>(state, nseg, stride, mode, init_S, init_z, DM);
    } else if (nseg <= 32) {
        dim3 grid((quads + 63) / 64, BH);
        scan_states_kernel<4><<<grid, 256, 0, s>>>(state, nseg, stride, mode, init_S, init_z, DM);
    } else {
        dim3 grid((quads + 31) / 32, BH);
        scan_states_kernel<8><<<grid, 256, 0, s>>>(state, nseg, stride, mode, init_S, init_z, DM);
    }
    return hipGetLastError();
}

// feature d of one token's q or k: eq. 7 of element d, the element itself when the caller has
// applied the map, or x_i x_j with 8i + j = d for the degree-2 polynomial map (section 3.2)
// (rounded by itself: not to be folded into the addition to z, which the kernels of several steps add it to from LDS)
template <typename T> __device__ __forceinline__ float feature_of(const T *row, int d) {
#pragma clang fp contract(off)
    if constexpr (is_poly<T>) return to_f32(row[d >> 3]) * to_f32(row[d & 7]);
    else return feature<T>(to_f32(row[d]));
}

// ---- recurrent decode step (eq. 16-20) -------------------------------------------------------
// One workgroup of four waves per head.  Every lane owns four adjacent columns of
// S; M/4 lanes cover a row, a wave covers 256/M rows per iteration.  The rank-1
// update, the z update and the read-out run in one sweep over S (read once,
// written once); the column sums are combined by wave shuffles, then across the
// four waves through LDS.  Fixed order everywhere: bit-identical run to run.
//
// A step of a serving batch is one trip to memory and back, so everything it reads is on its way before anything
// is computed or stored: with loads and stores in turn the compiler cannot move a load ahead of a store that might
// alias it, and a workgroup makes up to eight trips one after the other (B*H = 512, D = M = 64, back to back 4.4 -> 3.9 us;
// 32768: 208.6 -> 200.7).  kStream: S passes the caches by, see launch_recurrent_step.
template <int D, int M, typename T, bool kStream>
__global__ __launch_bounds__(256) void recurrent_step_kernel(const T *q, const T *k, const T *v,
                                                             float *S, float *z, T *out,
                                                             float eps) {
    constexpr int LPR = M / 4;            // lanes per row of S
    constexpr int RPW = kWave / LPR;      // rows per wave per iteration
    constexpr int RPI = 4 * RPW;          // rows per workgroup per iteration
    constexpr int NIT = D / RPI;
    static_assert(D % RPI == 0, "D must be a multiple of the rows swept per iteration");
    __shared__ __attribute__((aligned(16))) float red[4][M];
    __shared__ float dred[4];

    const int bh = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int col4 = (lane % LPR) * 4, rsub = lane / LPR, r0 = wave * RPW + rsub;
    constexpr int W = qk_width<T>(D);          // elements per token of q and k
    const T *qh = q + (size_t)bh * W, *kh = k + (size_t)bh * W;
    float *Sh = S + (size_t)bh * D * M + r0 * M + col4, *zh = z + (size_t)bh * D + r0;

    f32x4 s4[NIT];
    float zr[NIT], kd[NIT], qd[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        const f32x4 *p = reinterpret_cast<const f32x4 *>(Sh + it * RPI * M);
        if constexpr (kStream) s4[it] = __builtin_nontemporal_load(p);
        else s4[it] = *p;
    }
    const f32x4 v4 = load4(v + (size_t)bh * M + col4);
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        zr[it] = zh[it * RPI];                 // (the same in all lanes of a row)
        kd[it] = feature_of<T>(kh, it * RPI + r0);
        qd[it] = feature_of<T>(qh, it * RPI + r0);
    }
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    float dpart = 0.f;
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            s4[it][e] = fmaf(kd[it], v4[e], s4[it][e]);          // eq. 18
            acc[e] = fmaf(qd[it], s4[it][e], acc[e]);
        }
        zr[it] += kd[it];                                        // eq. 19
        dpart = fmaf(qd[it], zr[it], dpart);
        f32x4 *p = reinterpret_cast<f32x4 *>(Sh + it * RPI * M);
        if constexpr (kStream) __builtin_nontemporal_store(s4[it], p);
        else *p = s4[it];
    }
    if (col4 == 0) {
#pragma unroll
        for (int it = 0; it < NIT; ++it) zh[it * RPI] = zr[it];
    }
#pragma unroll
    for (int off = LPR; off < kWave; off <<= 1) {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += __shfl_xor(acc[e], off);
        dpart += __shfl_xor(dpart, off);
    }
    if (rsub == 0) *reinterpret_cast<f32x4 *>(&red[wave][col4]) = acc;
    if (lane == 0) dred[wave] = dpart;
    __syncthreads();
    if (tid < M) {
        const float num = (red[0][tid] + red[1][tid]) + (red[2][tid] + red[3][tid]);
        const float den = ((dred[0] + dred[1]) + (dred[2] + dred[3])) + eps;
        store_elem(out + (size_t)bh * M + tid, num / den);     // eq. 20 (the fraction)
    }
}

// T consecutive decode steps in one launch, for callers that already hold the q, k, v of
// all T tokens (scoring, teacher forcing): the state stays in registers between steps.  The
// additions of a step are those of recurrent_step_kernel in the same order: T steps here and T
// launches of the single step give bit-identical outputs and states.
//
// Steps are taken kStepBatch at a time: every wave runs the rank-1 updates and its lanes' partial
// read-outs of all steps without a barrier, leaving the partial sums in LDS; after one barrier all threads
// add them up and store the batch's outputs.  The threads stage the next batch's k, q (each feature
// mapped once) and v in LDS on the way, the one after that is in flight.  Bounded by instruction issue and LDS:
// 16 state elements per lane (D = M = 64) take 40 vector instructions and four 16-byte LDS accesses
// per step.  B*H = 512, T = 784: 742 us with the sums formed step by step (shuffles, one barrier
// each), 208 us so; 253 us with the features passed between the lanes of a row by DPP (moves of their
// own) instead of read from LDS.
constexpr int kStepBatch = 8;
// (x0 + x1) + (x2 + x3) ...: the order in which the single step's shuffles add
template <int N> __device__ __forceinline__ float tree_sum(const float (&x)[N]) {
    if constexpr (N == 1) return x[0];
    else {
        float y[N / 2];
#pragma unroll
        for (int i = 0; i < N / 2; ++i) y[i] = x[2 * i] + x[2 * i + 1];
        return tree_sum<N / 2>(y);
    }
}
template <int D, int M, typename T>
__global__ __launch_bounds__(256) void recurrent_steps_kernel(const T *q, const T *k, const T *v,
                                                              float *S, float *z, T *out,
                                                              float eps, int steps, size_t BH) {
    constexpr int LPR = M / 4, RPW = kWave / LPR, RPI = 4 * RPW, NIT = D / RPI;
    constexpr int W = qk_width<T>(D);          // elements per token of q and k
    constexpr int NF = kStepBatch * 2 * D / 256, NV = kStepBatch * M / 256;      // values a thread stages per batch
    typedef float fN __attribute__((ext_vector_type(NIT)));
    __shared__ __attribute__((aligned(16))) float feat[2][kStepBatch][2][D];          // k, q; row (wave, rsub, it) order
    __shared__ __attribute__((aligned(16))) float vals[2][kStepBatch][M];
    __shared__ __attribute__((aligned(16))) float part[2][kStepBatch][4][kWave][4];   // read-out partial sums
    __shared__ __attribute__((aligned(16))) float dpart[2][4][RPW][kStepBatch];

    const int bh = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int col4 = (lane % LPR) * 4, rsub = lane / LPR, r0 = wave * RPW + rsub;
    float *Sh = S + (size_t)bh * D * M, *zh = z + (size_t)bh * D;

    f32x4 s4[NIT];
    float zr[NIT];                            // (the same in all lanes of a row)
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        s4[it] = *reinterpret_cast<const f32x4 *>(Sh + (size_t)(it * RPI + r0) * M + col4);
        zr[it] = zh[it * RPI + r0];
    }
    // value j of a thread: step tf + j * TF of the batch, of k or q, feature df; step tv + j * TV, column tid % M of v
    constexpr int TF = 256 / (2 * D), TV = 256 / M;
    const size_t hop_f = BH * W, hop_v = BH * M;             // from one step to the next
    const int tf = tid / (2 * D), df = tid % D, tv = tid / M, fq = (tid / D) & 1;
    const T *pf = (fq ? q : k) + (size_t)bh * W, *pv = v + (size_t)bh * M + tid % M;
    float xf[NF], xv[NV];
    const size_t of = (size_t)tf * hop_f, ov = (size_t)tv * hop_v;
    auto one_f = [&](const T *row) {
        if constexpr (is_poly<T>) return feature_of<T>(row, df);      // the feature itself (x_i x_j)
        else return to_f32(row[df]);
    };
    auto fetch = [&](const int t0) {
        if (t0 + kStepBatch <= steps) {
#pragma unroll
            for (int j = 0; j < NF; ++j) xf[j] = one_f(pf + (size_t)(t0 + j * TF) * hop_f + of);
#pragma unroll
            for (int j = 0; j < NV; ++j) xv[j] = to_f32(pv[(size_t)(t0 + j * TV) * hop_v + ov]);
        } else {                              // steps past the end repeat the last one, unused
#pragma unroll
            for (int j = 0; j < NF; ++j) xf[j] = one_f(pf + min(t0 + tf + j * TF, steps - 1) * hop_f);
#pragma unroll
            for (int j = 0; j < NV; ++j) xv[j] = to_f32(pv[min(t0 + tv + j * TV, steps - 1) * hop_v]);
        }
    };
    float *const fput = &feat[0][tf][fq][(df % RPI) * NIT + df / RPI];       // df = it * RPI + r
    auto stage = [&](const int buf) {
#pragma unroll
        for (int j = 0; j < NF; ++j) fput[buf * kStepBatch * 2 * D + j * TF * 2 * D] = feature<T>(xf[j]);
#pragma unroll
        for (int j = 0; j < NV; ++j) (&vals[buf][0][0])[tid + 256 * j] = xv[j];
    };
    fetch(0);
    stage(0);
    if (kStepBatch < steps) fetch(kStepBatch);
    __syncthreads();
    int buf = 0;
    for (int t0 = 0; t0 < steps; t0 += kStepBatch, buf ^= 1) {
        const int n = min(kStepBatch, steps - t0);
        float dp8[kStepBatch];
        auto step = [&](const int t) {
            const fN kd = *reinterpret_cast<const fN *>(&feat[buf][t][0][r0 * NIT]);
            const fN qd = *reinterpret_cast<const fN *>(&feat[buf][t][1][r0 * NIT]);
            const f32x4 v4 = *reinterpret_cast<const f32x4 *>(&vals[buf][t][col4]);
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
            float dp = 0.f;
#pragma unroll
            for (int it = 0; it < NIT; ++it) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    s4[it][e] = fmaf(kd[it], v4[e], s4[it][e]);          // eq. 18
                    acc[e] = fmaf(qd[it], s4[it][e], acc[e]);
                }
                zr[it] += kd[it];                                        // eq. 19
                dp = fmaf(qd[it], zr[it], dp);
            }
            *reinterpret_cast<f32x4 *>(&part[buf][t][wave][lane][0]) = acc;
            return dp;
        };
        if (n == kStepBatch) {
#pragma unroll
            for (int t = 0; t < kStepBatch; ++t) dp8[t] = step(t);
        } else {
#pragma unroll
            for (int t = 0; t < kStepBatch; ++t) dp8[t] = t < n ? step(t) : 0.f;
        }
        if (col4 == 0) {
#pragma unroll
            for (int t = 0; t < kStepBatch; t += 4)
                *reinterpret_cast<f32x4 *>(&dpart[buf][wave][rsub][t]) = f32x4{dp8[t], dp8[t + 1], dp8[t + 2], dp8[t + 3]};
        }
        if (t0 + kStepBatch < steps) {
            stage(buf ^ 1);
            if (t0 + 2 * kStepBatch < steps) fetch(t0 + 2 * kStepBatch);
        }
        // one barrier per batch: what is read behind it is written again two batches on, behind the next one
        __syncthreads();
        // NV adjacent columns of one step per thread
        const int t = tid / (M / NV), m = NV * (tid % (M / NV));
        if (t < n) {
            float num[NV][4], den[4];
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                float x[NV][RPW], y[RPW];
#pragma unroll
                for (int r = 0; r < RPW; ++r) {
#pragma unroll
                    for (int i = 0; i < NV; ++i) x[i][r] = part[buf][t][w][r * LPR + m / 4][m % 4 + i];
                    y[r] = dpart[buf][w][r][t];
                }
#pragma unroll
                for (int i = 0; i < NV; ++i) num[i][w] = tree_sum<RPW>(x[i]);
                den[w] = tree_sum<RPW>(y);
            }
            const float dn = tree_sum<4>(den) + eps;
#pragma unroll
            for (int i = 0; i < NV; ++i) store_elem(out + ((size_t)(t0 + t) * BH + bh) * M + m + i, tree_sum<4>(num[i]) / dn);   // eq. 20
        }
    }
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        *reinterpret_cast<f32x4 *>(Sh + (size_t)(it * RPI + r0) * M + col4) = s4[it];
        if (col4 == 0) zh[it * RPI + r0] = zr[it];
    }
}

// The same a step at a time, for launches of a few steps: the next token's q, k, v are fetched while the
// current one is processed, one barrier per step.  What bounds such a launch is the state's way in and out, and
// that wants many workgroups in flight: 2 KB of LDS instead of 77, and no fetch of eight steps for one.
template <int D, int M, typename T>
__global__ __launch_bounds__(256) void recurrent_steps_few_kernel(const T *q, const T *k, const T *v,
                                                              float *S, float *z, T *out,
                                                              float eps, int steps, size_t BH) {
    constexpr int LPR = M / 4, RPW = kWave / LPR, RPI = 4 * RPW, NIT = D / RPI;
    __shared__ float red[2][4][M];
    __shared__ float dred[2][4];

    const int bh = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int col4 = (lane % LPR) * 4, rsub = lane / LPR;
    float *Sh = S + (size_t)bh * D * M, *zh = z + (size_t)bh * D;

    f32x4 s4[NIT];
    float zr[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        const int d = it * RPI + wave * RPW + rsub;
        s4[it] = *reinterpret_cast<const f32x4 *>(Sh + (size_t)d * M + col4);
        zr[it] = zh[d];
    }
    constexpr int W = qk_width<T>(D);          // elements per token of q and k
    // The wave sweeps NR rows of S per step, and every lane of a row needs that row's feature of
    // k and of q.  The feature map is evaluated once per row and wave, not once per lane: lane
    // j < NR fetches and maps k's element of row j of the sweep, lane NR + j the same of q (the
    // lanes above 2 NR repeat them, unused), and the lanes of a row pick the values up with a
    // shuffle.
    constexpr int NR = NIT * RPW;
    static_assert(2 * NR <= kWave, "one lane per row and operand");
    const int j = lane % NR;
    const bool mine_is_q = ((lane / NR) & 1) != 0;
    const int dj = (j / RPW) * RPI + wave * RPW + (j % RPW);
    auto fetch = [&](int t, float &x, f32x4 &v4) {
        const T *row = (mine_is_q ? q : k) + ((size_t)t * BH + bh) * W;
        if constexpr (is_poly<T>) x = feature_of<T>(row, dj);   // the feature itself (x_i x_j): nothing is left to map
        else x = to_f32(row[dj]);
        v4 = load4(v + ((size_t)t * BH + bh) * M + col4);
    };
    float x_next;
    f32x4 v_next;
    fetch(0, x_next, v_next);
    for (int t = 0; t < steps; ++t) {
        const float f = feature<T>(x_next);
        const f32x4 v4 = v_next;
        if (t + 1 < steps) fetch(t + 1, x_next, v_next);

        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        float dpart = 0.f;
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            const float kd = __shfl(f, it * RPW + rsub);
            const float qd = __shfl(f, NR + it * RPW + rsub);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                s4[it][e] = fmaf(kd, v4[e], s4[it][e]);
                acc[e] = fmaf(qd, s4[it][e], acc[e]);
            }
            if (col4 == 0) {
                zr[it] += kd;
                dpart = fmaf(qd, zr[it], dpart);
            }
        }
#pragma unroll
        for (int off = LPR; off < kWave; off <<= 1) {
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] += __shfl_xor(acc[e], off);
        }
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) dpart += __shfl_xor(dpart, off);
        const int buf = t & 1;            // two LDS buffers: one barrier per step suffices
        if (rsub == 0) {
#pragma unroll
            for (int e = 0; e < 4; ++e) red[buf][wave][col4 + e] = acc[e];
        }
        if (lane == 0) dred[buf][wave] = dpart;
        __syncthreads();
        if (tid < M) {
            const float num = (red[buf][0][tid] + red[buf][1][tid]) + (red[buf][2][tid] + red[buf][3][tid]);
            const float den = ((dred[buf][0] + dred[buf][1]) + (dred[buf][2] + dred[buf][3])) + eps;
            store_elem(out + ((size_t)t * BH + bh) * M + tid, num / den);
        }
    }
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        const int d = it * RPI + wave * RPW + rsub;
        *reinterpret_cast<f32x4 *>(Sh + (size_t)d * M + col4) = s4[it];
        if (col4 == 0) zh[d] = zr[it];
    }
}

// Which of the two.  Few / batched steps in us on the device (B*H sequences, fp32 unless noted):
//   T = 1   64 x 64  64: 2.9/3.3  1024: 6.3/7.5  2048: 11.8/14.2  bf16 4096: 22.0/27.5   32 x 32  8192: 15.6/29.0
//   T = 2   64 x 64  1024: 7.4/7.7  4096: 26.6/27.6  8192: 49.4/46.2   32 x 32  1024: 4.9/5.1  8192: 21.9/31.0
//   T = 3   64 x 64  1024: 8.6/8.0  2048: 15.9/17.2  8192: 53.6/46.7   32 x 32  1024: 6.1/5.4  8192: 29.4/32.4
//   T = 4   64 x 64  2048: 17.9/17.6  bf16 2048: 16.9/17.6  8192: 46.7/50.3   32 x 32  8192: 36.8/33.6
inline bool few_steps(int steps, int BH, int D, int M, bool bf16) {
    if (steps == 1) return true;
    const bool widest = D == 64 && M == 64;
    if (widest && !bf16 && BH > 4096) return false;
    return BH >= (steps == 2 ? 1024 : 2048) && steps <= (widest && bf16 ? 4 : 3);
}

hipError_t launch_recurrent_steps(const void *q, const void *k, const void *v, float *S, float *z,
                                  void *out, int steps, int BH, int D, int M, float eps, int dtype,
                                  hipStream_t s) {
    LA_DISPATCH(D, M, dtype, {
        if (few_steps(steps, BH, D, M, is_bf16<TT>)) {
            recurrent_steps_few_kernel<kD, kM, TT><<<BH, 256, 0, s>>>((const TT *)q, (const TT *)k, (const TT *)v, S, z, (TT *)out,
                                                                      eps, steps, (size_t)BH);
            return hipGetLastError();
        }
        recurrent_steps_kernel<kD, kM, TT><<<BH, 256, 0, s>>>((const TT *)q, (const TT *)k,
                                                             (const TT *)v, S, z, (TT *)out, eps,
                                                             steps, (size_t)BH);
    });
    return hipGetLastError();
}

hipError_t launch_recurrent_step(const void *q, const void *k, const void *v, float *S, float *z,
                                 void *out, int BH, int D, int M, float eps, int dtype,
                                 hipStream_t s) {
    // What is left of the states in the last-level cache (256 MB) when a step has gone through them serves the next
    // step; where they are so much larger that little of it does, non-temporal loads and stores are faster (one
    // without the other is not).  Plain / non-temporal in us, D = M = 64, by MB of S: 134 42.9/42.5, 268 75.7/84.7,
    // 282 84.0/89.3, 295 92.9/93.5, 308 101/98, 341 120/108, 537 201/173, 786 296/255.
    const bool stream = (size_t)BH * D * M * sizeof(float) > ((size_t)288 << 20);
    LA_DISPATCH(D, M, dtype, {
        if (stream) recurrent_step_kernel<kD, kM, TT, true><<<BH, 256, 0, s>>>((const TT *)q, (const TT *)k, (const TT *)v, S, z, (TT *)out, eps);
        else recurrent_step_kernel<kD, kM, TT, false><<<BH, 256, 0, s>>>((const TT *)q, (const TT *)k, (const TT *)v, S, z, (TT *)out, eps);
    });
    return hipGetLastError();
}

}  // namespace la
