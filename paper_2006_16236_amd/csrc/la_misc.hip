// Small bandwidth-bound kernels: the scan over segment states and the recurrent
// decode step (eq. 16-20).
#include "la_launch.h"
#include "la_plan.h"

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

// The denominators of the three decode kernels: the products q z of the NIT rows that a lane sweeps, row after row, each
// added unrounded; over the lanes and waves in the order of the columns' sums.  (Rounded products, added pairwise, lose where
// they cancel: outputs of the polynomial map, 300 steps, 3.5e-6 -> 6.8e-6 against 64 bits.)
template <int NIT, typename Q> __device__ __forceinline__ float rows_dot(const Q &q, const float (&z)[NIT]) {
    float d = 0.f;
#pragma unroll
    for (int it = 0; it < NIT; ++it) d = fmaf(q[it], z[it], d);
    return d;
}
// the same from z as the lanes of a row keep it: lane `it` of each four (of each two: NIT = 2) has row it's
template <int NIT> __device__ __forceinline__ float rows_dot_of_lanes(const float (&q)[NIT], const float zr) {
    float z[4] = {dpp_move<0x00>(zr), NIT > 1 ? dpp_move<0x55>(zr) : 0.f, NIT > 2 ? dpp_move<0xaa>(zr) : 0.f, NIT > 2 ? dpp_move<0xff>(zr) : 0.f};
    float zn[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it) zn[it] = z[it];
    return rows_dot<NIT>(q, zn);
}
// (x0 + x1) + (x2 + x3) ... over each 2^LEVELS neighbouring lanes (up to 16), result in all of them
template <int LEVELS> __device__ __forceinline__ float tree_sum_lanes(float v) {
    if constexpr (LEVELS > 0) v += dpp_move<0xb1>(v);       // quad_perm: lane ^ 1
    if constexpr (LEVELS > 1) v += dpp_move<0x4e>(v);       // lane ^ 2
    if constexpr (LEVELS > 2) v += dpp_move<0x141>(v);      // row_half_mirror: the other four of eight
    if constexpr (LEVELS > 3) v += dpp_move<0x140>(v);      // row_mirror: the other eight of sixteen
    return v;
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
// 32768: 208.6 -> 200.7).  kStream: S passes the caches by, see la_plan::step_streams.
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
    // lane `own` of a row's lanes keeps z of row `own` of its rows
    const int own = (lane % LPR) % NIT;
    const bool keeps = lane % LPR < NIT;
    float *Sh = S + (size_t)bh * D * M + r0 * M + col4, *zh = z + (size_t)bh * D + own * RPI + r0;

    f32x4 s4[NIT];
    float kd[NIT], qd[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        const f32x4 *p = reinterpret_cast<const f32x4 *>(Sh + it * RPI * M);
        if constexpr (kStream) s4[it] = __builtin_nontemporal_load(p);
        else s4[it] = *p;
    }
    const f32x4 v4 = load4(v + (size_t)bh * M + col4);
    float zr = *zh;
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        kd[it] = feature_of<T>(kh, it * RPI + r0);
        qd[it] = feature_of<T>(qh, it * RPI + r0);
    }
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    float kz = kd[0];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            s4[it][e] = fmaf(kd[it], v4[e], s4[it][e]);          // eq. 18
            acc[e] = fmaf(qd[it], s4[it][e], acc[e]);
        }
        if (own == it) kz = kd[it];
        f32x4 *p = reinterpret_cast<f32x4 *>(Sh + it * RPI * M);
        if constexpr (kStream) __builtin_nontemporal_store(s4[it], p);
        else *p = s4[it];
    }
    zr += kz;                                                    // eq. 19
    if (keeps) *zh = zr;
    float dpart = rows_dot_of_lanes<NIT>(qd, zr);
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
// Steps are taken kStepBatch at a time by two groups of four waves.  The first runs the rank-1 updates and its lanes'
// partial read-outs of a batch and leaves the partial sums in LDS, neighbouring rows added where a row takes 16 lanes
// (D = M = 64: 41 vector instructions and four LDS accesses per step, no barrier inside a batch).  The second meanwhile
// adds up and stores the batch before, with its denominators (q and z of each row), stages k, q (each feature mapped once) and v of the one to come, and has the one
// after that in flight: chains of LDS reads, additions and divisions that leave a SIMD idle half of the time where
// the first group has to walk them itself.  One barrier per batch.
// B*H = 512, T = 784, D = M = 64: 742 us with the sums formed step by step, 184 with four waves that do everything, 160
// so.  Bounded by vector instructions: the counters have the SIMDs' vector pipes busy throughout, the LDS half of the time.  (The features
// taken from a neighbouring lane by the instruction itself, `v_fmac_f32_dpp`, instead of from LDS: 187 -> 199 with four waves.)
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
// x0 and x1, columns of four rows in 16 lanes each: the sums of rows 0, 1 and of rows 2, 3; even rows get x0's, odd ones x1's
__device__ __forceinline__ float add_row_pairs(float x0, float x1) {
    const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(x0), __float_as_uint(x1), false, false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}
typedef float f32x2_t __attribute__((ext_vector_type(2)));
// kOne: one batch in all, and one buffer for it, half of the LDS: such a launch wants many workgroups in flight (eight steps
// of 4096 sequences, 64 x 32 heads 23.7 -> 18.7 us, 64 x 64 29.4 -> 28.0; with four waves 22.9 and 30.3).
template <int D, int M, typename T, bool kOne>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(4))) void recurrent_steps_kernel(const T *q, const T *k, const T *v,
                                                              float *S, float *z, T *out,
                                                              float eps, int steps, size_t BH) {
    constexpr int LPR = M / 4, RPW = kWave / LPR, RPI = 4 * RPW, NIT = D / RPI;
    constexpr int W = qk_width<T>(D);          // elements per token of q and k
    constexpr int NF = kStepBatch * 2 * D / 256, NV = kStepBatch * M / 256;      // values a thread stages per batch
    typedef float fN __attribute__((ext_vector_type(NIT)));
    constexpr int kBufs = kOne ? 1 : 2;
    __shared__ __attribute__((aligned(16))) float feat[kBufs][kStepBatch][2][D];          // k, q; row (wave, rsub, it) order
    __shared__ __attribute__((aligned(16))) float vals[kBufs][kStepBatch][M];
    constexpr bool kPairs = LPR == 16;         // the sums of neighbouring rows are added before they go to LDS
    constexpr int kSums = kPairs ? RPW / 2 : RPW;
    __shared__ __attribute__((aligned(16))) float part[kBufs][kStepBatch][4][kWave][kPairs ? 2 : 4];   // read-out partial sums
    __shared__ __attribute__((aligned(16))) float zrow[kBufs][kStepBatch][D];             // z after a step; row order as in feat

    const int bh = blockIdx.x, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int batches = kOne ? 1 : (steps + kStepBatch - 1) / kStepBatch;
    if (wave < 4) {
        __builtin_amdgcn_s_setprio(2);            // every batch waits for these
        const int lane = threadIdx.x & 63, col4 = (lane % LPR) * 4, rsub = lane / LPR, r0 = wave * RPW + rsub;
        const int own = (lane % LPR) % NIT;       // z: as in recurrent_step_kernel
        const bool keeps = lane % LPR < NIT;
        float *Sh = S + (size_t)bh * D * M, *zh = z + (size_t)bh * D + own * RPI + r0;

        f32x4 s4[NIT];
        float zr = *zh;
#pragma unroll
        for (int it = 0; it < NIT; ++it) s4[it] = *reinterpret_cast<const f32x4 *>(Sh + (size_t)(it * RPI + r0) * M + col4);
        __syncthreads();
        for (int b = 0; b < batches; ++b) {
            const int n = min(kStepBatch, steps - b * kStepBatch), buf = b & (kBufs - 1);
            float z8[kStepBatch];
            auto step = [&](const int t) {
                const fN kd = *reinterpret_cast<const fN *>(&feat[buf][t][0][r0 * NIT]);
                const fN qd = *reinterpret_cast<const fN *>(&feat[buf][t][1][r0 * NIT]);
                const f32x4 v4 = *reinterpret_cast<const f32x4 *>(&vals[buf][t][col4]);
                f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int it = 0; it < NIT; ++it) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        s4[it][e] = fmaf(kd[it], v4[e], s4[it][e]);          // eq. 18
                        acc[e] = fmaf(qd[it], s4[it][e], acc[e]);
                    }
                }
                if constexpr (kPairs) {
                    const float p0 = add_row_pairs(acc[0], acc[1]), p1 = add_row_pairs(acc[2], acc[3]);
                    *reinterpret_cast<f32x2_t *>(&part[buf][t][wave][lane][0]) = f32x2_t{p0, p1};
                } else {
                    *reinterpret_cast<f32x4 *>(&part[buf][t][wave][lane][0]) = acc;
                }
                zr += feat[buf][t][0][r0 * NIT + own];                       // eq. 19
                return zr;
            };
            if (n == kStepBatch) {
#pragma unroll
                for (int t = 0; t < kStepBatch; ++t) z8[t] = step(t);
            } else {
#pragma unroll
                for (int t = 0; t < kStepBatch; ++t) z8[t] = t < n ? step(t) : 0.f;
            }
            if (keeps) {
#pragma unroll
                for (int t = 0; t < kStepBatch; ++t) zrow[buf][t][r0 * NIT + own] = z8[t];
            }
            __syncthreads();
        }
#pragma unroll
        for (int it = 0; it < NIT; ++it) *reinterpret_cast<f32x4 *>(Sh + (size_t)(it * RPI + r0) * M + col4) = s4[it];
        if (keeps) *zh = zr;
        return;
    }
    // value j of a thread: step tf + j * TF of the batch, of k or q, feature df; step tv + j * TV, column tid % M of v
    const int tid = threadIdx.x - 256;
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
    // NV adjacent columns of one step per thread, 32 threads per step, which add up the step's denominator between them
    static_assert(M / NV == 32 && (RPI == 16 || RPI == 32), "32 threads per step");
    const int t = tid / 32, m = NV * (tid % 32), own_rows = NIT * (tid % RPI);
    auto outputs = [&](const int b, const fN qn) {       // qn: q of the thread's rows in that batch
        const int buf = b & (kBufs - 1);
        const fN zv = *reinterpret_cast<const fN *>(&zrow[buf][t][own_rows]);
        float zn[NIT];
#pragma unroll
        for (int it = 0; it < NIT; ++it) zn[it] = zv[it];
        float dn = tree_sum_lanes<4>(rows_dot<NIT>(qn, zn));
        if constexpr (RPI == 32) dn += __shfl_xor(dn, 16);
        dn += eps;
        if (b * kStepBatch + t < steps) {
            float num[NV][4];
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                float x[NV][kSums];
#pragma unroll
                for (int r = 0; r < kSums; ++r) {
#pragma unroll
                    for (int i = 0; i < NV; ++i)
                        x[i][r] = kPairs ? part[buf][t][w][(2 * r + i) * LPR + m / 4][m % 4 / 2] : part[buf][t][w][r * LPR + m / 4][m % 4 + i];
                }
#pragma unroll
                for (int i = 0; i < NV; ++i) num[i][w] = tree_sum<kSums>(x[i]);
            }
#pragma unroll
            for (int i = 0; i < NV; ++i)
                store_elem(out + ((size_t)(b * kStepBatch + t) * BH + bh) * M + m + i, tree_sum<4>(num[i]) / dn);   // eq. 20
        }
    };
    fetch(0);
    stage(0);
    if (kStepBatch < steps) fetch(kStepBatch);
    __syncthreads();
    fN qn;
    for (int b = 0; b < batches; ++b) {
        if (b > 0) outputs(b - 1, qn);
        qn = *reinterpret_cast<const fN *>(&feat[b & (kBufs - 1)][t][1][own_rows]);     // (the next batch but one takes their place)
        if (b + 1 < batches) {
            stage((b + 1) & 1);
            if (b + 2 < batches) fetch((b + 2) * kStepBatch);
        }
        __syncthreads();
    }
    outputs(batches - 1, qn);
}

// The same a step at a time, for launches of a few steps: the next token's q, k, v are fetched while the
// current one is processed, one barrier per step.  What bounds such a launch is the state's way in and out, and
// that wants many workgroups in flight: 2 KB of LDS instead of 20 to 40, and no fetch of eight steps for one.
template <int D, int M, typename T>
__global__ __launch_bounds__(256) void recurrent_steps_few_kernel(const T *q, const T *k, const T *v,
                                                              float *S, float *z, T *out,
                                                              float eps, int steps, size_t BH) {
    constexpr int LPR = M / 4, RPW = kWave / LPR, RPI = 4 * RPW, NIT = D / RPI;
    __shared__ float red[2][4][M];
    __shared__ float dred[2][4];

    const int bh = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int col4 = (lane % LPR) * 4, rsub = lane / LPR;
    const int own = (lane % LPR) % NIT;       // z: as in recurrent_step_kernel
    const bool keeps = lane % LPR < NIT;
    float *Sh = S + (size_t)bh * D * M, *zh = z + (size_t)bh * D + own * RPI + wave * RPW + rsub;

    f32x4 s4[NIT];
    float zr = *zh;
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        const int d = it * RPI + wave * RPW + rsub;
        s4[it] = *reinterpret_cast<const f32x4 *>(Sh + (size_t)d * M + col4);
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
        float qd[NIT];
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            const float kd = __shfl(f, it * RPW + rsub);
            qd[it] = __shfl(f, NR + it * RPW + rsub);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                s4[it][e] = fmaf(kd, v4[e], s4[it][e]);
                acc[e] = fmaf(qd[it], s4[it][e], acc[e]);
            }
        }
        zr += __shfl(f, own * RPW + rsub);
        float dpart = rows_dot_of_lanes<NIT>(qd, zr);
#pragma unroll
        for (int off = LPR; off < kWave; off <<= 1) {
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] += __shfl_xor(acc[e], off);
            dpart += __shfl_xor(dpart, off);
        }
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
    }
    if (keeps) *zh = zr;
}

hipError_t launch_recurrent_steps(const void *q, const void *k, const void *v, float *S, float *z,
                                  void *out, int steps, int BH, int D, int M, float eps, int dtype,
                                  hipStream_t s) {
    LA_DISPATCH(D, M, dtype, {
        if (la_plan::steps_one_by_one(steps, BH, D, M, (la_dtype)dtype)) {
            recurrent_steps_few_kernel<kD, kM, TT><<<BH, 256, 0, s>>>((const TT *)q, (const TT *)k, (const TT *)v, S, z, (TT *)out,
                                                                      eps, steps, (size_t)BH);
            return hipGetLastError();
        }
        if (steps <= kStepBatch) recurrent_steps_kernel<kD, kM, TT, true><<<BH, 512, 0, s>>>((const TT *)q, (const TT *)k, (const TT *)v, S, z, (TT *)out,
                                                                                            eps, steps, (size_t)BH);
        else recurrent_steps_kernel<kD, kM, TT, false><<<BH, 512, 0, s>>>((const TT *)q, (const TT *)k, (const TT *)v, S, z, (TT *)out, eps, steps,
                                                                          (size_t)BH);
    });
    return hipGetLastError();
}

hipError_t launch_recurrent_step(const void *q, const void *k, const void *v, float *S, float *z,
                                 void *out, int BH, int D, int M, float eps, int dtype,
                                 hipStream_t s) {
    const bool stream = la_plan::step_streams(BH, D, M, (la_dtype)dtype);
    LA_DISPATCH(D, M, dtype, {
        if (stream) recurrent_step_kernel<kD, kM, TT, true><<<BH, 256, 0, s>>>((const TT *)q, (const TT *)k, (const TT *)v, S, z, (TT *)out, eps);
        else recurrent_step_kernel<kD, kM, TT, false><<<BH, 256, 0, s>>>((const TT *)q, (const TT *)k, (const TT *)v, S, z, (TT *)out, eps);
    });
    return hipGetLastError();
}

}  // namespace la
