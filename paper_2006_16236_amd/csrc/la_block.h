// Causal passes by workgroups of eight (or four) waves on 32-token blocks.
//
// The products of la_passes.h (out_a = sum_{b <= a} (X_a . Y_b) Z_b with a carried state U, see
// the table there) on the bf16 matrix pipe only: every operand is cut into its bf16 parts ONCE,
// when its tile is parked in LDS, and the waves of the workgroup read it from there in whichever
// of the two orders a product needs.  fp32 tensors take three parts (exact, see split3), bf16
// tensors two (V and dO, exact in bf16, one).
//
// What bounds these kernels: a SIMD's bf16 MFMAs and vector instructions hardly overlap (24 MFMAs
// 165 ns, 144 fp32 instructions 158 ns, both 295 ns, four waves), so their times add, and both
// compete with the fetches.  Against one or two waves per segment on 16-token chunks an operand is
// split once instead of once per product that reads it, the state once per 32 tokens instead of
// 16, and a quarter as many segments fill the machine (512 workgroups): a state of 16.6 KB per
// segment less to write, scan and read, and fewer starts of the chain state - first tile - products.
// Measured (dQ / dV + dK in us, kernel trace, wave -> workgroup kernels): bf16 B*H = 16, N = 65536: 256 / 260 -> 174 / 186;
// fp32 B*H = 32, N = 1024: 24.4 / 21.3 -> 16.4 / 15.0; fp32 B*H = 32, N = 3072: 43.3 / 40.8 -> 40.9 / 40.9, and the
// scans 19 -> 12.
//
// Four "out" roles form the outputs (one per half of the tokens and half of the columns, or dV and
// dK), four "state" roles keep the carried state in fp32 accumulators, its tiles spread over them.
// One block:
//   barrier    tiles of the block and the carried state are in LDS, as bf16 parts
//   products   out roles: scores, read-out against the state, in-chunk term; state roles: update
//   barrier    nobody reads the tiles any more
//   park       outputs leave, the next block (fetched a block ago into registers) is mapped, cut
//              and parked, the state is cut and published, the block after that is fetched
// Two such workgroups share a compute unit (LDS: 74 KB each at D = M = 64, fp32; one alone takes 1.3
// to 1.4 times as long), so that one parks while the other multiplies.  Eight waves with one role each in 128
// registers; four waves with two roles each only for the polynomial map.  The fp32 backward with a 64-wide D or M had
// four while its state roles took all of their products at once and its two out roles shared their code, and with it
// the registers of both: at 128 they went to scratch memory, whose loads wait for the fetch that is under way.
// dQ + dV + dK of whole calls as the plan cuts them, four -> eight waves (B*H x N, us): D = M = 64 32 x 3072 77.1 -> 71.3,
// 64 x 512 33.3 -> 30.0, 200 x 512 80.2 -> 73.4, 256 x 1024 175 -> 163, 512 x 512 164 -> 152, 700 x 1024 514 -> 486; 64 x 32
// 32 x 3072 51.8 -> 48.2, 128 x 1024 67.3 -> 60.5, 512 x 1024 256 -> 230; 32 x 64 48.5 -> 45.0, 61.0 -> 57.4, 233 -> 214.
// At D = M = 64 dQ is one register short (8 bytes of scratch per lane), dV + dK none; while they were four and two short,
// workgroups of one to three blocks were slower than with four waves (32 x 1024 in pieces of two 34.9 us, 33.3 so, four waves
// 33.7; 512 x 32 14.3, 13.9, 14.0; 768 x 64 36.1, 33.0, 34.3), and 256 x 1024 is 2 to 3 % slower so than it was then.
// A second block in flight per thread changes nothing (bf16 0.606 -> 0.610 ms per step).
#pragma once

#include "la_passes.h"
#include "la_plan.h"

namespace la {

using la_plan::kBlk;              // tokens per block
// waves per workgroup of the forward and of the two backward kernels
constexpr int kFwdWaves = 8;
template <int D, int M, typename T> constexpr int kBwdWaves = is_poly<T> ? 4 : 8;     // (blk_chain is written for 4)

// ---- tiles of bf16 parts in LDS ----------------------------------------------------------------
// A plane holds one part of a tile, row-major, F bf16 per row, in 16-byte pieces that are permuted
// within a row by swz(row).  Both ways an operand is read then spread over the banks: 16 rows of
// one piece each (read_tok) and 4 or 8 rows of two neighbouring pieces (read_feat).
template <int F>
__device__ __forceinline__ constexpr int swz(int row) {
    if constexpr (F == 64) return (row & 6) ^ (5 * ((row >> 3) & 1));
    else return ((row >> 1) & 2) ^ (3 * ((row >> 3) & 1));
}
template <int F>
__device__ __forceinline__ int part_at(int row, int piece) {     // in elements
    return row * F + ((piece ^ swz<F>(row)) << 3);
}

// The operand of a 16x16x32 product: P parts of eight values per lane.
template <int P> struct Op {
    bf16x8_t p[P];
};
// acc[n] += a[n] b[n] over the 32 contraction slots, to the parts the operands have: the smallest part
// products first, those below the last part of the finer operand left out (P = 3: 2^-26 of the
// product).  The N products take turns, so that none waits for its own last result.
template <int N, int PA, int PB>
__device__ __forceinline__ void mma_n(const Op<PA> (&a)[N], const Op<PB> (&b)[N], f32x4 (&acc)[N]) {
    constexpr int top = (PA > PB ? PA : PB) - 1;
#pragma unroll
    for (int s = top; s >= 0; --s)
#pragma unroll
        for (int x = 0; x <= s; ++x)
            if (x < PA && s - x < PB) {
#pragma unroll
                for (int n = 0; n < N; ++n) acc[n] = mfma32_bf16(a[n].p[x], b[n].p[s - x], acc[n]);
            }
}

// Token-lane operand: lane (c, g) holds features 8 * piece .. + 7 of row `row`; a contraction over
// features takes pieces 4s + g for its step s.
template <int F, int P>
__device__ __forceinline__ Op<P> read_tok(const uint16_t *tile, int plane, int row, int piece) {
    Op<P> o;
    const uint16_t *p = tile + part_at<F>(row, piece);
#pragma unroll
    for (int k = 0; k < P; ++k) o.p[k] = *reinterpret_cast<const bf16x8_t *>(p + k * plane);
    return o;
}

// Transposed reads (ds_read_b64_tr_b16): of each group of 16 lanes, lane q supplies the address of
// four consecutive elements of row q / 4; lane i gets element i % 4 of the pieces of lanes i / 4,
// 4 + i / 4, ...: four rows of one column.
typedef short s16x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ u32x2_t read_tr(const uint16_t *p) {
    const auto v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t *)p);
    return __builtin_bit_cast(u32x2_t, v);
}
// Which of the F columns a lane's operand row rho = 4g + r of tile t stands for.  Natural: 16t + rho.
// Paired (bf16 outputs): two tiles of a pair give a lane eight consecutive columns, one 16-byte store.
template <bool kPair>
__device__ __forceinline__ int col_of(int t, int rho) {
    if constexpr (kPair) return 32 * (t >> 1) + 8 * (rho >> 2) + 4 * (t & 1) + (rho & 3);
    else return 16 * t + rho;
}
// Feature-lane operand: lane (c, g) holds column col_of(t, c) of eight rows.  kNatural = false: rows
// 4g .. + 3 and 16 + 4g .. + 3 (the order in which a pair of score tiles comes out of the accumulators),
// true: rows 8g .. + 7 (the order of read_tok).  `row0` = first of the 32 rows.
template <int F, bool kPair, bool kNatural = false>
__device__ __forceinline__ bf16x8_t read_feat_part(const uint16_t *tile, int row0, int t, int lane) {      // of the plane at `tile`
    const int q = lane & 15, g = lane >> 4;
    const int ra = row0 + (kNatural ? 8 * g : 4 * g) + (q >> 2), rb = ra + (kNatural ? 4 : 16);
    const int piece = kPair ? 4 * (t >> 1) + (q & 3) : 2 * t + ((q >> 1) & 1);
    const int half = kPair ? 4 * (t & 1) : 4 * (q & 1);
    return cat_parts(read_tr(tile + part_at<F>(ra, piece) + half), read_tr(tile + part_at<F>(rb, piece) + half));
}
template <int F, int P, bool kPair, bool kNatural = false>
__device__ __forceinline__ Op<P> read_feat(const uint16_t *tile, int plane, int row0, int t, int lane) {
    Op<P> o;
#pragma unroll
    for (int k = 0; k < P; ++k) o.p[k] = read_feat_part<F, kPair, kNatural>(tile + k * plane, row0, t, lane);
    return o;
}
// three parts of such an operand of which P are there already
template <int F, int P>
__device__ __forceinline__ Op<3> full_feat(const Op<P> &have, const uint16_t *tile, int plane, int t, int lane) {
    Op<3> o;
#pragma unroll
    for (int k = 0; k < P; ++k) o.p[k] = have.p[k];
    if constexpr (P == 2) o.p[2] = read_feat_part<F, false>(tile + 2 * plane, 0, t, lane);
    return o;
}

// The first parts of N quads and what is left of them, leaving the quads as they are: the two-address form that
// the compiler picks for minus_low and minus_high has them copied first (16 copies beside 48 vector instructions of a
// state role's publishing).  The compiler sees no vector instruction in an asm block and inserts no wait states for
// it.  Behind it: the three cycles a dot product needs before another kind of instruction may read its result are
// part of the block.  Ahead of it: a quad may come straight from a matrix product, so the block takes roundings that
// are made here, of the same quad; the compiler has the rounding wait for the product, and the block needs the
// rounding.  (The registers it writes: in the code built here no product within 15 instructions ahead of a block has
// one of them as its result or its addend.)
template <int N>
__device__ __forceinline__ void first_parts(const f32x4 (&q)[N], u32x2_t (&pair)[N], f32x4 (&r)[N]) {
#pragma unroll
    for (int n = 0; n < N; ++n)
#pragma unroll
        for (int j = 0; j < 2; ++j) pair[n][j] = round_pair(q[n][2 * j], q[n][2 * j + 1]);
#pragma unroll
    for (int n = 0; n < N; ++n) {
        float a, b, c, d;
        asm("v_dot2_f32_bf16 %0, %4, %10, %6\n\t"
            "v_dot2_f32_bf16 %1, %4, %11, %7\n\t"
            "v_dot2_f32_bf16 %2, %5, %10, %8\n\t"
            "v_dot2_f32_bf16 %3, %5, %11, %9\n\t"
            "s_nop 2"
            : "=&v"(a), "=&v"(b), "=&v"(c), "=&v"(d)
            : "v"(pair[n][0]), "v"(pair[n][1]), "v"(q[n][0]), "v"(q[n][1]), "v"(q[n][2]), "v"(q[n][3]), "s"(0x8000bf80u),
              "s"(0xbf808000u));
        r[n] = f32x4{a, b, c, d};
    }
}

// N quads cut into P parts stage by stage (an instruction and the one that needs its result are
// then several instructions apart; quad by quad the compiler fills the gaps with idle cycles)
template <int P, int N, bool kLive = false>      // kLive: the quads are needed afterwards
__device__ __forceinline__ void split_batch(const f32x4 (&q)[N], u32x2_t (&s)[N][P]) {
    f32x4 r[N];
#pragma unroll
    for (int n = 0; n < N; ++n) r[n] = q[n];
#pragma unroll
    for (int k = 0; k < P; ++k) {
        if (kLive && k == 0 && P > 1) {
            u32x2_t pair[N];
            first_parts(q, pair, r);
#pragma unroll
            for (int n = 0; n < N; ++n) s[n][0] = pair[n];
            continue;
        }
#pragma unroll
        for (int n = 0; n < N; ++n)
#pragma unroll
            for (int j = 0; j < 2; ++j) s[n][k][j] = round_pair(r[n][2 * j], r[n][2 * j + 1]);
        if (k + 1 < P) {
#pragma unroll
            for (int n = 0; n < N; ++n)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    r[n][2 * j] = minus_low(s[n][k][j], r[n][2 * j]);
                    r[n][2 * j + 1] = minus_high(s[n][k][j], r[n][2 * j + 1]);
                }
        }
    }
}
// the parts of four values, at four consecutive columns of a row (`p`: the first of them)
template <int P>
__device__ __forceinline__ void put_parts(uint16_t *p, int plane, const u32x2_t (&s)[P]) {
#pragma unroll
    for (int k = 0; k < P; ++k) *reinterpret_cast<u32x2_t *>(p + k * plane) = s[k];
}
template <int F> __device__ __forceinline__ int quad_at(int row, int col) {
    return part_at<F>(row, col >> 3) + (col & 4);
}
// ... and back (three parts: exactly the value that was put)
template <int F>
__device__ __forceinline__ f32x4 get_parts3(const uint16_t *tile, int plane, int row, int col) {
    const uint16_t *p = tile + quad_at<F>(row, col);
    const f32x4 h = widen(*reinterpret_cast<const u32x2_t *>(p));
    const f32x4 m = widen(*reinterpret_cast<const u32x2_t *>(p + plane));
    const f32x4 l = widen(*reinterpret_cast<const u32x2_t *>(p + 2 * plane));
    return (h + m) + l;
}

// a pair of accumulator tiles (rows 16 * blk + 4g + r of a contraction) as the operand of the next product
template <int P>
__device__ __forceinline__ Op<P> op_of(f32x4 a, f32x4 b) {
    const f32x4 q[2] = {a, b};
    u32x2_t s[2][P];
    split_batch<P>(q, s);
    Op<P> o;
#pragma unroll
    for (int k = 0; k < P; ++k) o.p[k] = cat_parts(s[0][k], s[1][k]);
    return o;
}

// ---- fetch and park ------------------------------------------------------------------------------
// The 32 tokens of a block are read and written through a buffer descriptor of exactly the tokens that
// exist: the addresses are a scalar base and one 32-bit offset per lane, rows past the end read as
// zero and are not written.  The whole offset goes into the lane's own, which is what the descriptor's
// size is compared with; of the instruction's scalar offset the compiler's documentation says that it is not.
typedef __amdgpu_buffer_rsrc_t Rows;
template <typename T>
__device__ __forceinline__ Rows rows_of(const T *first, int ts, int nv) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<T *>(first), 0, nv * ts * (int)sizeof(T), 0x00020000);
}
constexpr int kAuxNt = 2;         // the non-temporal bit of a buffer instruction
template <int kAux> __device__ __forceinline__ f32x4 rows_load(Rows r, int at, f32x4) {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, at, 0, kAux));
}
template <int kAux> __device__ __forceinline__ u32x2_t rows_load(Rows r, int at, u32x2_t) {
    return __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(r, at, 0, kAux));
}
__device__ __forceinline__ float rows_load1(Rows r, int at) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, at, 0, 0));
}

// Parts of the operands by element type: tile values and states; V, exact in bf16
template <typename T> constexpr int kOpParts = is_bf16<T> ? 2 : 3;
template <typename T> constexpr int kVParts = is_bf16<T> ? 1 : 3;

// The tiles of a block in LDS and their way there.  Besides the products of P parts the feature values of Q and K
// are needed in full, for phi' and for the sums that stay fp32, den in the forward, z and delta in the dQ pass, rho in
// the reverse pass: three parts for every element type, but for one tensor of the bf16 backward (kRaw, below).
// kLead: the pass, by the tensor whose gradient it ends in (kLeadQK: the forward, no dO there).
// bf16 backward (kRaw): dO takes the power of two of 1/den only, which leaves it one exact part, and the rest, 1 to 2
// in size, goes with phi(Q) where a product needs it (every sum over tokens a takes dO_a and phi(Q_a) together) or to
// the finished row.  (dO as it is and all of 1/den with phi(Q) saves 1 % of the step, 576 -> 570 us at B*H = 16,
// N = 65536, but its sums are den times as large: they overflow for gradients for which dO/den is nowhere near it.)
// And the pass that needs a tensor's feature values in full per token, phi(Q) in the dQ pass, phi(K) in the other,
// reads them from an fp32 plane and has two parts of that tensor; of the other tensor sums over tokens (z, rho) take
// three.  Against dO/den in two parts and three parts of Q and K throughout: 40 instead of 51 products per SIMD and
// block in the dQ pass, 50 instead of 58 in the other, 13 to 14 % fewer vector instructions, of which either kind costs
// its own issue time (bf16 step, B*H = 16, N = 65536, with the parking in one version: 617 -> 570 us; dQ / dV + dK at
// B*H = 32, N = 3072 21.6 / 21.9 -> 19.3 / 19.9, kernel traces on two boxes).
// A 32 x F block is fetched in quads of four elements, one or two per thread: quad k of thread t is
// row row(t) + k * kStep, columns col(t) .. + 3 (a wave reads whole rows).  Where a block has fewer quads
// than there are threads, the two blocks of a pair (Q and K, or dO and V) take half of them each.
// r = pow2_of(r) rest_of(r): a power of two not above |r|, and 1 <= |rest| < 2 (r = 0: 0 and 1; infinite: itself and 1)
__device__ __forceinline__ float pow2_of(float r) {
    return r == r ? __builtin_bit_cast(float, __builtin_bit_cast(unsigned, r) & 0x7f800000u) : r;
}
__device__ __forceinline__ float rest_of(float r) {
    return __builtin_bit_cast(float, (__builtin_bit_cast(unsigned, r) & 0x807fffffu) | 0x3f800000u);
}
enum Lead { kLeadQ = 0, kLeadK = 1, kLeadQK = 2 };
template <int kLead, int D, int M, typename T, bool kStrided>
struct BlkTiles {
    static constexpr int kWaves = kLead == kLeadQK ? kFwdWaves : kBwdWaves<D, M, T>, kThreads = kWave * kWaves;
    static constexpr bool kG = kLead != kLeadQK, kRaw = kG && is_bf16<T>;
    static constexpr int P = kOpParts<T>, PV = kVParts<T>, PG = kRaw ? 1 : P;
    static constexpr int PQ = kRaw && kLead == kLeadQ ? 2 : 3, PK = kRaw && kLead == kLeadK ? 2 : 3;
    static constexpr int kPlaneElems = kRaw ? 2 * kBlk * D : 0;
    static constexpr int kElems = (PQ + PK) * kBlk * D + (PV + (kG ? PG : 0)) * kBlk * M + kPlaneElems;
    template <int F> static constexpr int kQuads = 8 * F > kThreads ? 8 * F / kThreads : 1;
    template <int F> static constexpr int kStep = 4 * kThreads / F;
    template <int F> static constexpr bool kShared = 8 * F < kThreads;
    template <int F> static __device__ __forceinline__ int row(int tid) { return (tid % (8 * F)) / (F / 4); }
    template <int F> static __device__ __forceinline__ int col(int tid) { return 4 * (tid % (F / 4)); }

    uint16_t *sq, *sk, *sv, *sg;            // phi(Q), phi(K), V, dO/den; kRaw: the rest of 1/den with phi(Q)
    float *sf;                              // kRaw: phi(Q) (kLeadQ) or phi(K), fp32
    const T *Qs, *Ks, *Vs, *Gs;
    const float *scale;                     // of the rows of dO: den (kLeadQ, its reciprocal is taken) or 1/den
    int N, tid, half, tsd, tsm;
    bool nt, nt_out;
    int offd, offm;                         // bytes
    int qd, qm;
    staged_t<T> fq[kQuads<D>], fk[kQuads<D>], fv[kQuads<M>], fg[kQuads<M>];
    float sc[kQuads<M>], rest[kQuads<D>];   // of the rows of dO; kRaw: of Q
    // polynomial map: feature 8i + j = x_i x_j; fq, fk hold x_j .. x_j+3 of a quad, xq, xk its x_i
    static constexpr int W = qk_width<T>(D);
    float xq[kQuads<D>], xk[kQuads<D>];
    int offx;

    __device__ __forceinline__ BlkTiles(const PassArgs &a, uint16_t *lds, int bh, int tid_, int wave)
        : N(a.N), tid(tid_), half(wave >= kWaves / 2), tsd(tok_stride<kStrided>(a.tok_heads, qk_width<T>(D))),
          tsm(tok_stride<kStrided>(a.tok_heads, M)), nt(a.stream != 0), nt_out(a.nt_out != 0) {
        sq = lds, sk = sq + PQ * kBlk * D, sv = sk + PK * kBlk * D, sg = sv + PV * kBlk * M;
        if constexpr (kRaw) sf = reinterpret_cast<float *>(sg + PG * kBlk * M);
        Qs = static_cast<const T *>(a.Q) + seq_base<kStrided>(a.N, a.heads, bh, W);
        Ks = static_cast<const T *>(a.K) + seq_base<kStrided>(a.N, a.heads, bh, W);
        Vs = static_cast<const T *>(a.V) + seq_base<kStrided>(a.N, a.heads, bh, M);
        if constexpr (kG) {
            Gs = static_cast<const T *>(a.G) + seq_base<kStrided>(a.N, a.heads, bh, M);
            scale = (kLead == kLeadQ ? a.den_in : a.rden) + (size_t)bh * a.N;
        }
        offd = (row<D>(tid) * tsd + (is_poly<T> ? col<D>(tid) & 4 : col<D>(tid))) * (int)sizeof(T), offm = (row<M>(tid) * tsm + col<M>(tid)) * (int)sizeof(T);
        offx = (row<D>(tid) * tsd + (col<D>(tid) >> 3)) * (int)sizeof(T);
        qd = quad_at<D>(row<D>(tid), col<D>(tid)), qm = quad_at<M>(row<M>(tid), col<M>(tid));
    }
    template <int F> __device__ __forceinline__ bool mine(int which) const { return !kShared<F> || half == which; }

    template <int F, int kAux>
    __device__ __forceinline__ void load(const T *first, int off, int ts, int nv, staged_t<T> (&st)[kQuads<F>]) const {
        const Rows r = rows_of(first, ts, nv);
#pragma unroll
        for (int k = 0; k < kQuads<F>; ++k) st[k] = rows_load<kAux>(r, off + k * kStep<F> * ts * (int)sizeof(T), staged_t<T>{});
    }
    template <int kAux>
    __device__ __forceinline__ void load_all(const int t0, const int nv) {
        if constexpr (kG) {
            const Rows r = rows_of(scale + t0, 1, nv);
            if (mine<M>(0)) {
#pragma unroll
                for (int k = 0; k < kQuads<M>; ++k) sc[k] = rows_load1(r, 4 * (row<M>(tid) + k * kStep<M>));
            }
            if (kRaw && D != M && mine<D>(0)) {
#pragma unroll
                for (int k = 0; k < kQuads<D>; ++k) rest[k] = rows_load1(r, 4 * (row<D>(tid) + k * kStep<D>));
            }
        }
        if (kG && mine<M>(0)) load<M, kAux>(Gs + (size_t)t0 * tsm, offm, tsm, nv, fg);
        if (mine<M>(1)) load<M, kAux>(Vs + (size_t)t0 * tsm, offm, tsm, nv, fv);
        if (mine<D>(0)) load<D, kAux>(Qs + (size_t)t0 * tsd, offd, tsd, nv, fq);
        if (mine<D>(1)) load<D, kAux>(Ks + (size_t)t0 * tsd, offd, tsd, nv, fk);
        if constexpr (is_poly<T>) {
            const Rows q = rows_of(Qs + (size_t)t0 * tsd, tsd, nv), k_ = rows_of(Ks + (size_t)t0 * tsd, tsd, nv);
#pragma unroll
            for (int k = 0; k < kQuads<D>; ++k) {
                xq[k] = rows_load1(q, offx + k * kStep<D> * tsd * (int)sizeof(T));
                xk[k] = rows_load1(k_, offx + k * kStep<D> * tsd * (int)sizeof(T));
            }
        }
    }
    __device__ __forceinline__ void fetch(const int blk) {
        const int t0 = blk * kBlk, nv = min(kBlk, N - t0);
        if (nt) load_all<kAuxNt>(t0, nv);     // uniform
        else load_all<0>(t0, nv);
    }

    // where the fp32 plane holds columns 4 * piece .. + 3 of a row: the pieces of sixteen rows spread over all banks
    static __device__ __forceinline__ int plane_at(int row, int piece) {
        return row * D + ((piece ^ (D == 64 ? row & 15 : (row >> 1) & 7)) << 2);
    }
    // kKeep: the mapped values go to the fp32 plane too; kBy: their rows are scaled by `by` before they are cut;
    // kZero: rows past the end are zero
    template <int F, int PT, int MAP_, bool kKeep = false, bool kBy = false, bool kZero = false>
    __device__ __forceinline__ void put(uint16_t *tile, int at, const staged_t<T> (&st)[kQuads<F>], const float *by, int nv = kBlk) const {
        constexpr int MAP = is_poly<T> && MAP_ == kMapPhi ? kMapScale : is_feat<T> && MAP_ == kMapPhi ? kMapId : MAP_;
        if constexpr (PT == 1 && MAP == kMapId && is_bf16<T>) {         // as it is
#pragma unroll
            for (int k = 0; k < kQuads<F>; ++k) *reinterpret_cast<u32x2_t *>(tile + at + k * kStep<F> * F) = st[k];
        } else {
            f32x4 v[kQuads<F>];
#pragma unroll
            for (int k = 0; k < kQuads<F>; ++k) {
                const f32x4 w = widen(st[k]);
                const int at_row = row<F>(tid) + k * kStep<F>;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float m = map_value<MAP>(w[r], MAP == kMapScale ? by[k] : 1.0f);
                    v[k][r] = !kZero || at_row < nv ? m : 0.0f;
                }
                if constexpr (kKeep) *reinterpret_cast<f32x4 *>(sf + plane_at(at_row, col<F>(tid) >> 2)) = v[k];
                if constexpr (kBy) v[k] *= by[k];
            }
            u32x2_t s[kQuads<F>][PT];
            split_batch<PT>(v, s);
#pragma unroll
            for (int k = 0; k < kQuads<F>; ++k) put_parts<PT>(tile + at + k * kStep<F> * F, kBlk * F, s[k]);
        }
    }
    // 1/den of a row from what was fetched for it (rows past the end: 0)
    static __device__ __forceinline__ float rden_of(float fetched, int at_row, int nv) {
        return kLead != kLeadQ ? fetched : at_row < nv ? __builtin_amdgcn_rcpf(fetched) : 0.0f;
    }
    // Rows past the end were fetched as zeros, so V and dO are zero there and phi(0) = 1 of Q and K meets only those
    // zeros, a delta that is set to zero, or rows of an output that are not stored.  It must be finite, hence
    // no reciprocal of a denominator that is not there; and the forward's z counts keys: those are zeroed,
    // in code of their own for the one block that has such rows.  With all tiles in two versions the
    // compiler copied what both share (that and the state's copies, see first_parts: bf16 step, B*H = 16, N = 65536,
    // 570 -> 560 us; fp32 B*H = 32, N = 3072, forward 28.0 -> 27.1, dQ 37.9 -> 36.5, dV + dK 37.5 -> 36.8).
    __device__ __forceinline__ void park(const int blk) {
        const int nv = min(kBlk, N - blk * kBlk);
        if (kG && mine<M>(0)) {
#pragma unroll
            for (int k = 0; k < kQuads<M>; ++k) {
                const float r = rden_of(sc[k], row<M>(tid) + k * kStep<M>, nv);
                if constexpr (kRaw && D == M) rest[k] = rest_of(r);
                sc[k] = kRaw ? pow2_of(r) : r;
            }
            put<M, PG, kMapScale>(sg, qm, fg, sc);
        }
        if (kRaw && D != M && mine<D>(0)) {
#pragma unroll
            for (int k = 0; k < kQuads<D>; ++k) rest[k] = rest_of(rden_of(rest[k], row<D>(tid) + k * kStep<D>, nv));
        }
        if (mine<M>(1)) put<M, PV, kG ? kMapId : kMapFinite>(sv, qm, fv, nullptr);
        if (mine<D>(0)) put<D, PQ, kMapPhi, kRaw && kLead == kLeadQ, kRaw>(sq, qd, fq, kRaw ? rest : xq);
        if (mine<D>(1)) {
            if (kG || nv == kBlk) put<D, PK, kMapPhi, kRaw && kLead == kLeadK>(sk, qd, fk, xk);
            else put<D, PK, kMapPhi, false, false, true>(sk, qd, fk, xk, nv);
        }
    }
    // feature values of the pass's tensor in full, columns 4 * piece .. + 3 of a row
    __device__ __forceinline__ f32x4 full_values(int row, int piece) const {
        if constexpr (kRaw) return *reinterpret_cast<const f32x4 *>(sf + plane_at(row, piece));
        else return get_parts3<D>(kLead == kLeadQ ? sq : sk, kBlk * D, row, 4 * piece);
    }
};
// accumulator tiles of a carried state, cut and published (rows = columns of the tiles)
template <int F, int P, int NX, int NY>
__device__ __forceinline__ void publish(uint16_t *tile, int plane, const f32x4 (&U)[NX][NY], int x0, int y0, int c, int g) {
#pragma unroll
    for (int y = 0; y < NY; ++y) {
        f32x4 q[NX];
        u32x2_t s[NX][P];
#pragma unroll
        for (int x = 0; x < NX; ++x) q[x] = U[x][y];
        split_batch<P, NX, true>(q, s);
#pragma unroll
        for (int x = 0; x < NX; ++x) put_parts<P>(tile + quad_at<F>(16 * (y0 + y) + c, 16 * (x0 + x) + 4 * g), plane, s[x]);
    }
}

// ---- outputs -------------------------------------------------------------------------------------
// A wave's output, 16 tokens x 16 NT columns (lane (c, g): token c, four columns per tile), goes to
// memory through LDS scratch of the wave's own, 16 bytes per lane and whole rows of the wave's columns
// per instruction: straight from the accumulators a store instruction would touch 64 bytes of 16 rows
// each (measured at N = 65536, fp32: dV + dK 0.58 against 0.43 ms without its stores).
// The scratch is cut into pieces of 512 bytes, `stride` bytes apart.  At D = M = 64 it is the memory of the
// rows that the wave itself will park next (four rows of each plane), so it costs no LDS.
template <int D, int M> constexpr bool kScratchInTiles = D == 64 && M == 64;
template <typename T, int NT>
struct OutRows {
    static constexpr int kBytes = 16 * NT * (int)sizeof(T);       // of one row
    static constexpr int kPieces = kBytes / 16;                   // 16-byte pieces per row
    static constexpr bool kDirect = is_bf16<T> && NT == 1;        // half pieces: stored as they are
    static constexpr int kScratch = kDirect ? 0 : 16 * kBytes;    // bytes per wave
    template <int stride> static __device__ __forceinline__ int at(int row, int piece) {
        return (row / (512 / kBytes)) * stride + (row % (512 / kBytes)) * kBytes +
               ((piece ^ (row * kBytes / 256)) << 4);
    }
    // `r`: the tokens of the block, `at0`: byte offset of the wave's first token and column, `ts`: token stride in elements,
    // `nt`: PassArgs::nt_out
    template <int kStride>
    static __device__ __forceinline__ void store(char *scratch, Rows r, int at0, int ts, const f32x4 (&out)[NT], int lane, bool nt) {
        const int c = lane & 15, g = lane >> 4;
        if constexpr (kDirect) {
            __builtin_amdgcn_raw_buffer_store_b64(u32x2_t{round_pair(out[0][0], out[0][1]), round_pair(out[0][2], out[0][3])}, r,
                                                  (c * ts + 4 * g) * (int)sizeof(T) + at0, 0, 0);
        } else {
            if constexpr (is_bf16<T>) {
#pragma unroll
                for (int t = 0; t < NT; t += 2)
                    *reinterpret_cast<u32x4_t *>(scratch + at<kStride>(c, 2 * t + g)) =
                        u32x4_t{round_pair(out[t][0], out[t][1]), round_pair(out[t][2], out[t][3]),
                                round_pair(out[t + 1][0], out[t + 1][1]), round_pair(out[t + 1][2], out[t + 1][3])};
            } else {
#pragma unroll
                for (int t = 0; t < NT; ++t) *reinterpret_cast<f32x4 *>(scratch + at<kStride>(c, 4 * t + g)) = out[t];
            }
            __builtin_amdgcn_wave_barrier();
            constexpr int kRows = kWave / kPieces;
            const int row0 = lane / kPieces, piece = lane % kPieces;
#pragma unroll
            for (int k = 0; k < 16 / kRows; ++k) {
                const u32x4_t v = *reinterpret_cast<const u32x4_t *>(scratch + at<kStride>(row0 + kRows * k, piece));
                const int to = (row0 + kRows * k) * ts * (int)sizeof(T) + 16 * piece + at0;
                if (LA_NT_STORES != 0 && (!is_bf16<T> || nt)) __builtin_amdgcn_raw_buffer_store_b128(v, r, to, 0, kAuxNt);      // (uniform)
                else __builtin_amdgcn_raw_buffer_store_b128(v, r, to, 0, 0);
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
};

// the blocks [begin, begin + count) of a segment
__device__ __forceinline__ void blk_range(const PassArgs &a, int seg, int &begin, int &count) {
    const int nblk = (a.N + kBlk - 1) / kBlk, per = (a.chunks_per_seg + 1) / 2;
    begin = seg * per;
    count = min(begin + per, nblk) - begin;
}

// Chain rule of x -> vec(x x^T) (see poly2_chain) for a block: `rows` holds the gradients for the 64
// features of its 32 tokens (stride 68 floats), 256 threads take one of the 32 x 8 raw gradients each.
constexpr int kChainStride = 68;
template <typename T>
__device__ __forceinline__ void blk_chain(const float *rows, const T *raw, T *out, int ts, int nv, int tid) {
    const int token = tid >> 3, k = tid & 7;
    const Rows r = rows_of(raw, ts, nv);
    const f32x4 x0 = rows_load<0>(r, token * ts * 4, f32x4{}), x1 = rows_load<0>(r, token * ts * 4 + 16, f32x4{});
    const float *p = rows + token * kChainStride;
    const f32x4 a = *reinterpret_cast<const f32x4 *>(p + 8 * k), b = *reinterpret_cast<const f32x4 *>(p + 8 * k + 4);
    float acc = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        acc = fmaf(a[j] + p[8 * j + k], x0[j], acc);
        acc = fmaf(b[j] + p[8 * (j + 4) + k], x1[j], acc);
    }
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, acc), rows_of(out, ts, nv), (token * ts + k) * 4, 0, 0);
}

// ---- the loop over the blocks --------------------------------------------------------------------
// first, first + dir, ..: `count` of them.  A role: init (its part of the starting state, after the first
// fetch is under way), publish (its state to LDS), fetch / parked (what it needs per token), products
// (between the barriers), finish (after the second: outputs leave).
template <typename Tiles, typename... Role>
__device__ __forceinline__ void blk_loop(Tiles &tiles, const int first, const int dir, const int count, Role &...role) {
    // Nothing is in flight here, but the compiler's count of it does not know which role's code a wave has come
    // through: without this the out roles' products of the bf16 forward and dV + dK pass wait, block after block, for
    // registers of the state roles' fetch, that is for their own.
    __builtin_amdgcn_s_waitcnt(0x0f70);           // vmcnt(0)
    tiles.fetch(first);
    (role.fetch(first), ...);
    (role.init(), ...);
    (role.publish(), ...);
    tiles.park(first);
    (role.parked(first), ...);
    if (count > 1) {
        tiles.fetch(first + dir);
        (role.fetch(first + dir), ...);
    }
    for (int n = 0; n < count; ++n) {
        const int blk = first + dir * n;
        __syncthreads();
        (role.products(), ...);
        __syncthreads();
        (role.finish(blk), ...);
        if (n + 1 < count) {
            (role.publish(), ...);
            tiles.park(blk + dir);
            (role.parked(blk + dir), ...);
            if (n + 2 < count) {
                tiles.fetch(blk + 2 * dir);
                (role.fetch(blk + 2 * dir), ...);
            }
        }
    }
}
struct BlkLane {
    int lane, c, g, i, h;                // i, h: the wave's quarter
    __device__ __forceinline__ BlkLane(int tid, int wave) : lane(tid & (kWave - 1)), c(lane & 15), g(lane >> 4), i(wave & 1), h((wave >> 1) & 1) {}
};
// acc + a b summed over the S contraction steps, a chain of products per step
template <int S, int PA, int PB>
__device__ __forceinline__ f32x4 dot(const Op<PA> (&a)[S], const Op<PB> (&b)[S], f32x4 acc) {
    f32x4 w[S];
#pragma unroll
    for (int s = 0; s < S; ++s) w[s] = f32x4{0.f, 0.f, 0.f, 0.f};
    w[0] = acc;
    mma_n(a, b, w);
    return S == 2 ? w[0] + w[S - 1] : w[0];
}
// the same in one chain, the smallest part products of all steps first: one rounding at the size of the
// result per step (for den, whose own rounding counts; one chain throughout costs the forward 6 %)
template <int S, int PA, int PB>
__device__ __forceinline__ f32x4 dot_chain(const Op<PA> (&a)[S], const Op<PB> (&b)[S], f32x4 acc) {
    constexpr int top = (PA > PB ? PA : PB) - 1;
#pragma unroll
    for (int k = top; k >= 0; --k)
#pragma unroll
        for (int x = 0; x <= k; ++x)
            if (x < PA && k - x < PB) {
#pragma unroll
                for (int s = 0; s < S; ++s) acc = mfma32_bf16(a[s].p[x], b[s].p[k - x], acc);
            }
    return acc;
}
template <int F, int P, int S>
__device__ __forceinline__ void read_toks(const uint16_t *tile, int plane, int row, int g, Op<P> (&o)[S]) {
#pragma unroll
    for (int s = 0; s < S; ++s) o[s] = read_tok<F, P>(tile, plane, row, 4 * s + g);
}

// ---- causal forward (eq. 9-12) ---------------------------------------------------------------------
// Out role (i, h): the 16 tokens of sub-block i, columns of half h of V; the scores and with them the
// denominators of a sub-block are formed by both of its roles.  bf16 tensors: den comes from three-part
// operands (it is an fp32 result), the numerator from bf16 products, the scores in two parts.
template <int D, int M, typename T, bool kStrided>
struct FwdOut : BlkLane {
    using Tiles = BlkTiles<kLeadQK, D, M, T, kStrided>;
    static constexpr int PV = Tiles::PV, PS = is_bf16<T> ? 1 : 3, NT = M / 32, SD = D / 32;
    static constexpr int PW = is_bf16<T> ? 2 : 3;      // scores: a block's own part of the output is twice as long as
                                                       // a 16-token chunk's
    static constexpr bool kPair = is_bf16<T> && NT == 2;
    using OutTile = OutRows<T, NT>;
    const Tiles &tl;
    const uint16_t *ss, *sz;
    char *scratch;
    T *outs;
    float *den_out, eps, den;
    int N, row;
    f32x4 out[NT];                       // columns col_of(h NT + y, 4g + r) of the token

    __device__ __forceinline__ FwdOut(const PassArgs &a, const Tiles &t, int bh, int tid, int wave, const uint16_t *ss_,
                                      const uint16_t *sz_, char *scratch_)
        : BlkLane(tid, wave), tl(t), ss(ss_), sz(sz_), scratch(scratch_ + 512 * (wave & 3)) {
        outs = a.out != nullptr ? static_cast<T *>(a.out) + seq_base<kStrided>(a.N, a.heads, bh, M) : nullptr;
        den_out = a.den != nullptr ? a.den + (size_t)bh * a.N : nullptr;
        eps = a.eps, N = a.N, row = 16 * i + c;
    }
    __device__ __forceinline__ void init() {}
    __device__ __forceinline__ void publish() {}
    __device__ __forceinline__ void fetch(int) {}
    __device__ __forceinline__ void parked(int) {}
    __device__ __forceinline__ void products() {
        const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
        // scores phi(Q_a) . phi(K_b): rows b, lane (c = a)
        Op<3> qt[SD];
        read_toks<D, 3>(tl.sq, kBlk * D, row, g, qt);
        f32x4 w0, w1 = zero4;
        {
            Op<3> kt[SD];
            read_toks<D, 3>(tl.sk, kBlk * D, c, g, kt);
            w0 = dot(kt, qt, zero4);
        }
        if (i != 0) {
            Op<3> kt[SD];
            read_toks<D, 3>(tl.sk, kBlk * D, 16 + c, g, kt);
            w1 = dot(kt, qt, zero4);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {        // select, never multiply
            w0[r] = (i != 0 || 4 * g + r <= c) ? w0[r] : 0.f;
            w1[r] = 4 * g + r <= c ? w1[r] : 0.f;
        }
        // den: phi(Q) . z (the same operand row in every lane c) and the row sums of the scores
        {
            Op<3> zt[SD];
#pragma unroll
            for (int s = 0; s < SD; ++s)
#pragma unroll
                for (int k = 0; k < 3; ++k) zt[s].p[k] = *reinterpret_cast<const bf16x8_t *>(sz + k * D + 32 * s + 8 * g);
            const float p = ((w0[0] + w0[1]) + (w0[2] + w0[3])) + ((w1[0] + w1[1]) + (w1[2] + w1[3]));
            den = dot_chain(zt, qt, mfma16(1.0f, p, f32x4{eps, eps, eps, eps}))[0];
        }
        Op<PS> qs[SD];
#pragma unroll
        for (int s = 0; s < SD; ++s)
#pragma unroll
            for (int k = 0; k < PS; ++k) qs[s].p[k] = qt[s].p[k];
#pragma unroll
        for (int y = 0; y < NT; ++y) {
            Op<PS> st[SD];
            read_toks<D, PS>(ss, M * D, col_of<kPair>(h * NT + y, c), g, st);
            out[y] = dot(st, qs, zero4);
        }
        const Op<PW> wop[1] = {op_of<PW>(w0, w1)};
#pragma unroll
        for (int y = 0; y < NT; ++y) {
            const Op<PV> vf[1] = {read_feat<M, PV, kPair>(tl.sv, kBlk * M, 0, h * NT + y, lane)};
            f32x4 o[1] = {out[y]};
            mma_n(vf, wop, o);
            out[y] = o[0];
        }
    }
    __device__ __forceinline__ void finish(int blk) {
        const int t0 = blk * kBlk, nv = min(kBlk, N - t0);
        const float ri = __builtin_amdgcn_rcpf(den);
#pragma unroll
        for (int y = 0; y < NT; ++y)
#pragma unroll
            for (int r = 0; r < 4; ++r) out[y][r] *= ri;
        if (outs != nullptr)             // (a forward that is run for its denominators only)
            OutTile::template store<kScratchInTiles<D, M> ? 2 * kBlk * D : 4 * 512>(
                scratch, rows_of(outs + (size_t)t0 * tl.tsm, tl.tsm, nv), (16 * i * tl.tsm + h * (M / 2)) * (int)sizeof(T), tl.tsm, out, lane, tl.nt_out);
        if (den_out != nullptr && h == 0 && g == 0 && row < nv) den_out[t0 + row] = den;
    }
};

// State role (i, h): S (D x M), D / 32 x M / 32 tiles, published as [m][d]; (i, 0) also z.
template <int D, int M, typename T, bool kStrided>
struct FwdState : BlkLane {
    using Tiles = BlkTiles<kLeadQK, D, M, T, kStrided>;
    static constexpr int PV = Tiles::PV, PS = is_bf16<T> ? 1 : 3, DT = D / 32, MT = M / 32;
    static constexpr int PU = is_bf16<T> ? 2 : 3;      // phi(K) in the update: the state also leaves the call
    const PassArgs &a;
    const Tiles &tl;
    uint16_t *ss, *sz;
    int bh, seg;
    f32x4 U[DT][MT];       // element (d = 16 (i DT + x) + 4g + r, m = 16 (h MT + y) + c)
    f32x4 z[DT];           // z[16 (i DT + x) + 4g + r]

    __device__ __forceinline__ FwdState(const PassArgs &a_, const Tiles &t, int bh_, int seg_, int tid, int wave, uint16_t *ss_, uint16_t *sz_)
        : BlkLane(tid, wave), a(a_), tl(t), ss(ss_), sz(sz_), bh(bh_), seg(seg_) {}
    __device__ __forceinline__ void add(const float *sm, const float *v) {
#pragma unroll
        for (int x = 0; x < DT; ++x) {
#pragma unroll
            for (int y = 0; y < MT; ++y)
#pragma unroll
                for (int r = 0; r < 4; ++r) U[x][y][r] += sm[(16 * (i * DT + x) + 4 * g + r) * M + 16 * (h * MT + y) + c];
            z[x] += load4_state(v + 16 * (i * DT + x) + 4 * g);
        }
    }
    __device__ __forceinline__ void init() {
#pragma unroll
        for (int x = 0; x < DT; ++x) {
            z[x] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int y = 0; y < MT; ++y) U[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        if (a.init_S != nullptr) add(a.init_S + (size_t)bh * D * M, a.init_z + (size_t)bh * D);
        if (a.state != nullptr) {
            int nslots, lo, hi;
            state_slots(a, seg, kStatePrefix, nslots, lo, hi);
            for (int j = lo; j < hi; ++j) {
                const float *st = a.state + ((size_t)bh * nslots + j) * state_stride(D, M);
                add(st, st + D * M);
            }
        }
    }
    __device__ __forceinline__ void publish() {
        la::publish<D, PS>(ss, M * D, U, i * DT, h * MT, c, g);
        if (h == 0) {
            // every lane c has all of z: lane x cuts and stores quad x
            f32x4 q[1];
            u32x2_t s[1][3];
#pragma unroll
            for (int r = 0; r < 4; ++r) q[0][r] = DT == 2 && c != 0 ? z[DT - 1][r] : z[0][r];
            split_batch<3>(q, s);
            if (c < DT) put_parts<3>(sz + 16 * (i * DT + c) + 4 * g, D, s[0]);
        }
    }
    __device__ __forceinline__ void fetch(int) {}
    __device__ __forceinline__ void parked(int) {}
    __device__ __forceinline__ void products() {
        const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
        Op<3> kn[DT];
        Op<PU> kk[DT * MT];
        Op<PV> vn[MT], vv[DT * MT];
        f32x4 u[DT * MT];
#pragma unroll
        for (int y = 0; y < MT; ++y) vn[y] = read_feat<M, PV, false>(tl.sv, kBlk * M, 0, h * MT + y, lane);
#pragma unroll
        for (int x = 0; x < DT; ++x) {
            kn[x] = read_feat<D, 3, false>(tl.sk, kBlk * D, 0, i * DT + x, lane);
#pragma unroll
            for (int y = 0; y < MT; ++y) {
#pragma unroll
                for (int k = 0; k < PU; ++k) kk[x * MT + y].p[k] = kn[x].p[k];
                vv[x * MT + y] = vn[y], u[x * MT + y] = zero4;
            }
        }
        mma_n(kk, vv, u);
#pragma unroll
        for (int x = 0; x < DT; ++x)
#pragma unroll
            for (int y = 0; y < MT; ++y) U[x][y] += u[x * MT + y];
        if (h == 0) {
            const unsigned one2 = 0x3f803f80u;
            Op<1> ones[DT];
            f32x4 zz[DT];
#pragma unroll
            for (int x = 0; x < DT; ++x) ones[x].p[0] = cat_parts(u32x2_t{one2, one2}, u32x2_t{one2, one2}), zz[x] = zero4;
            mma_n(kn, ones, zz);
#pragma unroll
            for (int x = 0; x < DT; ++x) z[x] += zz[x];
        }
    }
    __device__ __forceinline__ void finish(int) {}
    __device__ __forceinline__ void end() {       // the last segment ends with the final state
        if (a.final_S == nullptr || seg != a.nseg - 1) return;
        float *s1 = a.final_S + (size_t)bh * D * M;
#pragma unroll
        for (int x = 0; x < DT; ++x) {
#pragma unroll
            for (int y = 0; y < MT; ++y)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    s1[(16 * (i * DT + x) + 4 * g + r) * M + 16 * (h * MT + y) + c] = U[x][y][r];
            if (h == 0 && c == 0) *reinterpret_cast<f32x4 *>(a.final_z + (size_t)bh * D + 16 * (i * DT + x) + 4 * g) = z[x];
        }
    }
};

template <int D, int M, typename T, bool kStrided = false>
__global__ __launch_bounds__((kWave * kFwdWaves)) __attribute__((amdgpu_waves_per_eu((kFwdWaves / 2)))) void fwd_block_kernel(
    const PassArgs a) {
    using Tiles = BlkTiles<kLeadQK, D, M, T, kStrided>;
    using OutRole = FwdOut<D, M, T, kStrided>;
    using StateRole = FwdState<D, M, T, kStrided>;
    constexpr bool kOwn = kScratchInTiles<D, M>;
    __shared__ __attribute__((aligned(16))) uint16_t tiles[Tiles::kElems + (kOwn ? 0 : 4 * OutRole::OutTile::kScratch / 2)];
    __shared__ __attribute__((aligned(16))) uint16_t ss[OutRole::PS * M * D];     // S before the block, [m][d]
    __shared__ __attribute__((aligned(16))) uint16_t sz[3 * D];                   // z before the block, in parts
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int seg = blockIdx.x % a.nseg, bh = blockIdx.x / a.nseg;
    int blk0, count;
    blk_range(a, seg, blk0, count);
    char *const scratch = reinterpret_cast<char *>(kOwn ? tiles : tiles + Tiles::kElems);
    Tiles tl(a, tiles, bh, tid, wave);
    if (wave < 4) {
        OutRole out(a, tl, bh, tid, wave, ss, sz, scratch);
        blk_loop(tl, blk0, 1, count, out);
    } else {
        StateRole st(a, tl, bh, seg, tid, wave, ss, sz);
        blk_loop(tl, blk0, 1, count, st);
        st.end();
    }
}

// ---- causal forward of a few short sequences -------------------------------------------------------
// Up to kDirectTokens tokens, few enough of them that every 32 queries have a compute unit to themselves: nothing is
// carried, a workgroup takes 32 queries and its waves one block of 32 keys each, up to the queries' own, by
// definition (eq. 8-9): scores, their sums and their product with V; the partial results are added up in LDS.  Such a
// call is bound by latency: launches, and in each the way to memory and back.  Cut into segments it takes two
// launches that depend on each other, here one: the segment totals, which a backward may ask the workspace for, come
// from workgroups of their own in the same launch (block ndirect on).  (One workgroup of either kind fills a compute unit:
// D = M = 64, fp32, 185 registers and 70 KB of LDS; where the queries' own fill the machine, the totals come in a second round.)
// All operands come straight from memory in the order the products need, split by the wave that reads them; the
// arithmetic is that of FwdOut (three-part scores, den in fp32, scores of bf16 tensors in two parts against V).
constexpr int kDirectTokens = la_plan::kDirectTokens, kDirectWaves = kDirectTokens / kBlk;
// features 8 piece .. + 7 of a row, in three parts
template <int D, typename T>
__device__ __forceinline__ Op<3> direct_tok(const Rows r, const int row, const int ts, const int piece) {
    f32x4 lo, hi;
    if constexpr (is_bf16<T>) {
        const u32x4_t u = __builtin_bit_cast(u32x4_t, rows_load<0>(r, (row * ts + 8 * piece) * 2, f32x4{}));
        lo = widen(u32x2_t{u[0], u[1]}), hi = widen(u32x2_t{u[2], u[3]});
    } else {
        const int at = (row * ts + (is_poly<T> ? 0 : 8 * piece)) * 4;
        lo = rows_load<0>(r, at, f32x4{}), hi = rows_load<0>(r, at + 16, f32x4{});
    }
    const float by = is_poly<T> ? rows_load1(r, (row * ts + piece) * 4) : 1.0f;        // feature 8i + j = x_i x_j
    constexpr int kMap = is_poly<T> ? kMapScale : is_feat<T> ? kMapId : kMapPhi;
#pragma unroll
    for (int k = 0; k < 4; ++k) lo[k] = map_value<kMap>(lo[k], by), hi[k] = map_value<kMap>(hi[k], by);
    return op_of<3>(lo, hi);
}
template <typename T> __device__ __forceinline__ float direct_v(const Rows r, const int at) {      // at: in elements
    float v;
    if constexpr (is_bf16<T>)
        v = __builtin_bit_cast(float, (unsigned)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r, 2 * at, 0, 0) << 16);
    else v = rows_load1(r, 4 * at);
    return map_value<kMapFinite>(v, 1.0f);
}

template <int D, int M, typename T, bool kStrided = false>
__global__ __launch_bounds__((kWave * kDirectWaves)) void fwd_direct_kernel(const PassArgs a, const SegArgs sa, const int ndirect) {
    constexpr int SD = D / 32, YT = M / 16, PV = kVParts<T>, PW = is_bf16<T> ? 2 : 3, kSegWaves = 4;
    constexpr int kRow = M + 4, kPart = kBlk * kRow, kRed = kDirectWaves * (kPart + kBlk);
    __shared__ __attribute__((aligned(16))) float lds[kRed > seg_lds(D, M, kSegWaves) ? kRed : seg_lds(D, M, kSegWaves)];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), c = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if ((int)blockIdx.x >= ndirect) {
        // (the other waves are done: a workgroup's barrier does not wait for waves that have ended)
        if (wave < kSegWaves) segment_totals<D, M, T, kStrided, kSegWaves>(sa, blockIdx.x - ndirect, lds);
        return;
    }
    const int nblk = (a.N + kBlk - 1) / kBlk, qb = blockIdx.x % nblk, bh = blockIdx.x / nblk;
    const int tsd = tok_stride<kStrided>(a.tok_heads, qk_width<T>(D)), tsm = tok_stride<kStrided>(a.tok_heads, M);
    const int q0 = qb * kBlk, nq = min(kBlk, a.N - q0);
    float *const sden = lds + kDirectWaves * kPart;
    const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
    if (wave <= qb) {
        const int k0 = wave * kBlk, nk = min(kBlk, a.N - k0);
        const size_t based = seq_base<kStrided>(a.N, a.heads, bh, qk_width<T>(D)), basem = seq_base<kStrided>(a.N, a.heads, bh, M);
        const Rows rq = rows_of(static_cast<const T *>(a.Q) + based + (size_t)q0 * tsd, tsd, nq);
        const Rows rk = rows_of(static_cast<const T *>(a.K) + based + (size_t)k0 * tsd, tsd, nk);
        const Rows rv = rows_of(static_cast<const T *>(a.V) + basem + (size_t)k0 * tsm, tsm, nk);
        Op<3> kt[2][SD], qt[2][SD];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int s = 0; s < SD; ++s) {
                kt[i][s] = direct_tok<D, T>(rk, 16 * i + c, tsd, 4 * s + g);
                qt[i][s] = direct_tok<D, T>(rq, 16 * i + c, tsd, 4 * s + g);
            }
        // V as the operand that a pair of score tiles meets: column 16 y + c of rows 4g .. + 3 and 16 + 4g .. + 3
        Op<PV> vt[YT];
#pragma unroll
        for (int y = 0; y < YT; ++y) {
            f32x4 lo, hi;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                lo[r] = direct_v<T>(rv, (4 * g + r) * tsm + 16 * y + c);
                hi[r] = direct_v<T>(rv, (16 + 4 * g + r) * tsm + 16 * y + c);
            }
            vt[y] = op_of<PV>(lo, hi);
        }
        const bool own = wave == qb;         // the queries' own block: keys up to each query
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            f32x4 w0 = dot(kt[0], qt[i], zero4), w1 = dot(kt[1], qt[i], zero4);     // rows: keys, lane c: query 16 i + c
#pragma unroll
            for (int r = 0; r < 4; ++r) {    // select, never multiply
                w0[r] = !own || i != 0 || 4 * g + r <= c ? w0[r] : 0.f;
                w1[r] = !own || (i != 0 && 4 * g + r <= c) ? w1[r] : 0.f;
            }
            const float p = sum_over_groups(((w0[0] + w0[1]) + (w0[2] + w0[3])) + ((w1[0] + w1[1]) + (w1[2] + w1[3])));
            if (g == 0) sden[wave * kBlk + 16 * i + c] = p;
            const Op<PW> wop = op_of<PW>(w0, w1);
            Op<PW> wo[YT];
            f32x4 o[YT];
#pragma unroll
            for (int y = 0; y < YT; ++y) wo[y] = wop, o[y] = zero4;
            mma_n(vt, wo, o);
#pragma unroll
            for (int y = 0; y < YT; ++y)
                *reinterpret_cast<f32x4 *>(lds + wave * kPart + (16 * i + c) * kRow + 16 * y + 4 * g) = o[y];
        }
    }
    __syncthreads();
    constexpr int kQuads = M / 4;            // of a row
    if (tid >= kBlk * kQuads) return;
    const int row = tid / kQuads, col = 4 * (tid % kQuads);
    f32x4 o = zero4;
    float den = 0.f;
    for (int w = 0; w <= qb; ++w) {          // (all eight read at once, the others not taken: 0.2 to 0.4 us more)
        o += *reinterpret_cast<const f32x4 *>(lds + w * kPart + row * kRow + col);
        den += sden[w * kBlk + row];
    }
    if (row >= nq) return;
    den += a.eps;
    const float ri = __builtin_amdgcn_rcpf(den);
    if (a.out != nullptr) {
        T *p = static_cast<T *>(a.out) + seq_base<kStrided>(a.N, a.heads, bh, M) + (size_t)(q0 + row) * tsm + col;
        if constexpr (is_bf16<T>) *reinterpret_cast<u32x2_t *>(p) = u32x2_t{round_pair(o[0] * ri, o[1] * ri), round_pair(o[2] * ri, o[3] * ri)};
        else *reinterpret_cast<f32x4 *>(p) = o * ri;
    }
    if (a.den != nullptr && col == 0) a.den[(size_t)bh * a.N + q0 + row] = den;
}

// ---- causal dQ (eq. 13) ----------------------------------------------------------------------------
// Out role (i, h): dQ of the 16 tokens of sub-block i, columns of half h.  The scores of a sub-block
// are formed by both of its roles (12 or 24 of 54 to 66 products per block, against a barrier and an
// exchange).  As in dq_causal_kernel delta comes from the role's own results,
// delta_a = -(phi(Q_a) . A_a) / den_a; each of the two has half of that sum.
template <int D, int M, typename T, bool kStrided>
struct DqOut : BlkLane {
    using Tiles = BlkTiles<kLeadQ, D, M, T, kStrided>;
    static constexpr int P = Tiles::P, PV = Tiles::PV, PG = Tiles::PG, NT = D / 32, SM = M / 32;
    static constexpr bool kPair = is_bf16<T> && NT == 2;
    static constexpr bool kFresh = Tiles::kWaves == 8 && !is_bf16<T> && D == 64 && M == 64;
    using OutTile = OutRows<T, NT>;
    const Tiles &tl;
    const uint16_t *ss;
    const float *sz, *den;
    float (*sdel)[2][16], (*srho)[D];
    char *scratch;
    T *outs;
    float *delta_out, *rden_out;
    int N, row;
    float nden, rd;
    Op<1> mask;                          // token b <= token 16i + c over the 32 tokens of the block
    f32x4 out[NT], cz[NT], fq[NT];       // columns col_of(h NT + y, 4g + r) of the token
    f32x4 rho[NT];                       // this segment's delta phi(Q), per token lane

    __device__ __forceinline__ DqOut(const PassArgs &a, const Tiles &t, int bh, int tid, int wave, const uint16_t *ss_,
                                     const float *sz_, float (*sdel_)[2][16], float (*srho_)[D], char *scratch_)
        : BlkLane(tid, wave), tl(t), ss(ss_), sz(sz_), sdel(sdel_), srho(srho_), scratch(scratch_ + 512 * (wave & 3)) {
        const size_t rowbase = (size_t)bh * a.N;
        den = a.den_in + rowbase;
        outs = static_cast<T *>(a.out) + seq_base<kStrided>(a.N, a.heads, bh, qk_width<T>(D));
        delta_out = a.delta_out + rowbase, rden_out = a.rden_out + rowbase;
        N = a.N, row = 16 * i + c, nden = 1.f, rd = 0.f;
        auto bit = [&](int b) { return b <= row ? 0x3f80u : 0u; };
        const int b0 = 4 * g, b1 = 16 + 4 * g;
        mask.p[0] = cat_parts(u32x2_t{bit(b0) | (bit(b0 + 1) << 16), bit(b0 + 2) | (bit(b0 + 3) << 16)},
                              u32x2_t{bit(b1) | (bit(b1 + 1) << 16), bit(b1 + 2) | (bit(b1 + 3) << 16)});
#pragma unroll
        for (int y = 0; y < NT; ++y) rho[y] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    __device__ __forceinline__ void init() {}
    __device__ __forceinline__ void publish() {}
    __device__ __forceinline__ void fetch(int blk) { nden = den[min(blk * kBlk + row, N - 1)]; }
    // Kept ahead of the next fetch: sunk behind it, the old and the new denominator take two registers, and the copy
    // from one to the other waits for the fetch that has just been sent, a trip to memory per block (dQ pass,
    // B*H = 16, N = 65536: bf16 206 -> 190 us, fp32, for which the plan takes the wave kernel there, forced 381 -> 334;
    // step, fp32 B*H = 32, N = 3072, with the wait ahead of the loop: 117.4 -> 113.9)
    __device__ __forceinline__ void parked(int blk) {
        rd = __builtin_amdgcn_rcpf(nden);
        asm volatile("" : "+v"(rd));
    }
    __device__ __forceinline__ void products() {
        const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
        // scores (dO_a/den_a) . V_b (kRaw: the whole row waits for the rest of its 1/den): rows b, lane (c = a)
        Op<PG> gt[SM];
        read_toks<M, PG>(tl.sg, kBlk * M, row, g, gt);
        f32x4 w0, w1 = zero4;
        {
            Op<PV> vt[SM];
            read_toks<M, PV>(tl.sv, kBlk * M, c, g, vt);
            w0 = dot(vt, gt, zero4);
        }
        if (i != 0) {
            Op<PV> vt[SM];
            read_toks<M, PV>(tl.sv, kBlk * M, 16 + c, g, vt);
            w1 = dot(vt, gt, zero4);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {        // select, never multiply
            w0[r] = (i != 0 || 4 * g + r <= c) ? w0[r] : 0.f;
            w1[r] = 4 * g + r <= c ? w1[r] : 0.f;
        }
        // read-out against the state, in-chunk term, z up to each token
#pragma unroll
        for (int y = 0; y < NT; ++y) {
            Op<P> st[SM];
            read_toks<M, P>(ss, D * M, col_of<kPair>(h * NT + y, c), g, st);
            out[y] = dot(st, gt, zero4);
        }
        const Op<P> wop = op_of<P>(w0, w1);
        float p = 0.f;
        int lk = lane;
        if constexpr (kFresh) asm volatile("" : "+v"(lk));      // addresses formed per block, not kept: 128 registers
#pragma unroll
        for (int y = 0; y < NT; ++y) {
            const Op<P> kf[1] = {read_feat<D, P, kPair>(tl.sk, kBlk * D, 0, h * NT + y, lk)};
            const Op<P> wo[1] = {wop};
            const Op<1> mo[1] = {mask};
            f32x4 o[1] = {out[y]};
            f32x4 cc[1] = {*reinterpret_cast<const f32x4 *>(sz + col_of<kPair>(h * NT + y, 4 * g))};
            mma_n(kf, mo, cc);
            mma_n(kf, wo, o);
            out[y] = o[0];
            cz[y] = cc[0];
            fq[y] = tl.full_values(row, col_of<kPair>(h * NT + y, 4 * g) >> 2);
#pragma unroll
            for (int r = 0; r < 4; ++r) p = fmaf(out[y][r], fq[y][r], p);
        }
        p = sum_over_groups(p);
        if (g == 0) sdel[i][h][c] = p;
    }
    __device__ __forceinline__ void finish(int blk) {
        const int t0 = blk * kBlk, nv = min(kBlk, N - t0);
        const float rest = Tiles::kRaw ? rest_of(rd) : 1.f;
        const float dr = row < nv ? -(sdel[i][0][c] + sdel[i][1][c]) * rd : 0.f;     // delta / rest, as the row is
        const float d = Tiles::kRaw ? (row < nv ? dr * rest : 0.f) : dr;
#pragma unroll
        for (int y = 0; y < NT; ++y)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                rho[y][r] = fmaf(d, fq[y][r], rho[y][r]);
                out[y][r] = fmaf(dr, cz[y][r], out[y][r]) * feature_slope<T>(fq[y][r]);
                if constexpr (Tiles::kRaw) out[y][r] *= rest;
            }
        if constexpr (is_poly<T>) {      // (four waves, each with an out role: all of them are here)
            float *rows = reinterpret_cast<float *>(tl.sq);
#pragma unroll
            for (int y = 0; y < NT; ++y)
                *reinterpret_cast<f32x4 *>(rows + row * kChainStride + 16 * (h * NT + y) + 4 * g) = out[y];
            __syncthreads();
            blk_chain(rows, tl.Qs + (size_t)t0 * tl.tsd, outs + (size_t)t0 * tl.tsd, tl.tsd, nv, tl.tid);
            __syncthreads();
        } else {
            OutTile::template store<kScratchInTiles<D, M> ? 2 * kBlk * D : 4 * 512>(
                scratch, rows_of(outs + (size_t)t0 * tl.tsd, tl.tsd, nv), (16 * i * tl.tsd + h * (D / 2)) * (int)sizeof(T), tl.tsd, out, lane, tl.nt_out);
        }
        if (h == 0 && g == 0 && row < nv) {
            delta_out[t0 + row] = d;
            rden_out[t0 + row] = rd;
        }
    }
    __device__ __forceinline__ void end() {
#pragma unroll
        for (int y = 0; y < NT; ++y)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float e = row_sum16(rho[y][r]);
                if (c == 0) srho[i][col_of<kPair>(h * NT + y, 4 * g + r)] = e;
            }
    }
};

// State role (i, h): S^T (M x D) and, when the sequences are cut, this segment's phi(Q)^T dO/den, D / 32 x
// M / 32 tiles of each; (0, h) also z.  The products of a block are summed on their own and added to
// the running sums in one fp32 addition per element and block.
template <int D, int M, typename T, bool kStrided>
struct DqState : BlkLane {
    using Tiles = BlkTiles<kLeadQ, D, M, T, kStrided>;
    static constexpr int P = Tiles::P, PV = Tiles::PV, PG = Tiles::PG, NT = D / 32, MT = M / 32;
    const PassArgs &a;
    const Tiles &tl;
    uint16_t *ss;
    float *sz;
    int bh, seg;
    f32x4 U[MT][NT];       // S^T: element (m = 16 (i MT + x) + 4g + r, d = 16 (h NT + y) + c)
    f32x4 R[NT][MT];       // element (d = 16 (h NT + y) + 4g + r, m = 16 (i MT + x) + c)
    f32x4 z[NT];           // z[16 (h NT + y) + 4g + r]

    __device__ __forceinline__ DqState(const PassArgs &a_, const Tiles &t, int bh_, int seg_, int tid, int wave, uint16_t *ss_, float *sz_)
        : BlkLane(tid, wave), a(a_), tl(t), ss(ss_), sz(sz_), bh(bh_), seg(seg_) {}
    __device__ __forceinline__ void add(const float *sm, const float *v) {     // sm: S as [D][M], v: z
#pragma unroll
        for (int y = 0; y < NT; ++y) {
#pragma unroll
            for (int x = 0; x < MT; ++x)
                U[x][y] += load4_state(sm + (16 * (h * NT + y) + c) * M + 16 * (i * MT + x) + 4 * g);
            z[y] += load4_state(v + 16 * (h * NT + y) + 4 * g);
        }
    }
    __device__ __forceinline__ void init() {
#pragma unroll
        for (int y = 0; y < NT; ++y) {
            z[y] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int x = 0; x < MT; ++x) U[x][y] = R[y][x] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        if (a.init_S != nullptr) add(a.init_S + (size_t)bh * D * M, a.init_z + (size_t)bh * D);
        if (a.state != nullptr) {
            int nslots, lo, hi;
            state_slots(a, seg, kStatePrefix, nslots, lo, hi);
            for (int j = lo; j < hi; ++j) {
                const float *st = a.state + ((size_t)bh * nslots + j) * state_stride(D, M);
                add(st, st + D * M);
            }
        }
    }
    __device__ __forceinline__ void publish() {
        la::publish<M, P>(ss, D * M, U, i * MT, h * NT, c, g);
        if (i == 0 && c == 0) {
#pragma unroll
            for (int y = 0; y < NT; ++y) *reinterpret_cast<f32x4 *>(sz + 16 * (h * NT + y) + 4 * g) = z[y];
        }
    }
    __device__ __forceinline__ void fetch(int) {}
    __device__ __forceinline__ void parked(int) {}
    __device__ __forceinline__ void products() {
        const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
        {
            Op<P> kn[NT];
#pragma unroll
            for (int y = 0; y < NT; ++y) kn[y] = read_feat<D, P, false>(tl.sk, kBlk * D, 0, h * NT + y, lane);
#pragma unroll
            for (int x = 0; x < MT; ++x) {
                const Op<PV> vf = read_feat<M, PV, false>(tl.sv, kBlk * M, 0, i * MT + x, lane);
                Op<PV> vv[NT];
                f32x4 u[NT];
#pragma unroll
                for (int y = 0; y < NT; ++y) vv[y] = vf, u[y] = zero4;
                mma_n(vv, kn, u);
#pragma unroll
                for (int y = 0; y < NT; ++y) U[x][y] += u[y];
            }
            if (i == 0) {
                const unsigned one2 = 0x3f803f80u;
                Op<1> ones[NT];
                Op<3> kf[NT];             // z is an fp32 sum: three parts whatever P is
                f32x4 zz[NT];
#pragma unroll
                for (int y = 0; y < NT; ++y) {
                    kf[y] = full_feat<D>(kn[y], tl.sk, kBlk * D, h * NT + y, lane);
                    ones[y].p[0] = cat_parts(u32x2_t{one2, one2}, u32x2_t{one2, one2}), zz[y] = zero4;
                }
                mma_n(kf, ones, zz);
#pragma unroll
                for (int y = 0; y < NT; ++y) z[y] += zz[y];
            }
        }
        if (a.totals != nullptr) {
            Op<PG> gn[MT];
#pragma unroll
            for (int x = 0; x < MT; ++x) gn[x] = read_feat<M, PG, false>(tl.sg, kBlk * M, 0, i * MT + x, lane);
#pragma unroll
            for (int y = 0; y < NT; ++y) {
                const Op<P> qf = read_feat<D, P, false>(tl.sq, kBlk * D, 0, h * NT + y, lane);
                Op<P> qq[MT];
                f32x4 u[MT];
#pragma unroll
                for (int x = 0; x < MT; ++x) qq[x] = qf, u[x] = zero4;
                mma_n(qq, gn, u);
#pragma unroll
                for (int x = 0; x < MT; ++x) R[y][x] += u[x];
            }
        }
    }
    __device__ __forceinline__ void finish(int) {}
    __device__ __forceinline__ void end(float *tot) {
#pragma unroll
        for (int y = 0; y < NT; ++y)
#pragma unroll
            for (int x = 0; x < MT; ++x)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    tot[(16 * (h * NT + y) + 4 * g + r) * M + 16 * (i * MT + x) + c] = R[y][x][r];
    }
};

template <int D, int M, typename T, bool kStrided = false>
__global__ __launch_bounds__((kWave * kBwdWaves<D, M, T>)) __attribute__((amdgpu_waves_per_eu((kBwdWaves<D, M, T> / 2)))) void dq_block_kernel(
    const PassArgs a) {
    using Tiles = BlkTiles<kLeadQ, D, M, T, kStrided>;
    using OutRole = DqOut<D, M, T, kStrided>;
    using StateRole = DqState<D, M, T, kStrided>;
    constexpr bool kOwn = kScratchInTiles<D, M>;
    __shared__ __attribute__((aligned(16))) uint16_t tiles[Tiles::kElems + (kOwn ? 0 : 4 * OutRole::OutTile::kScratch / 2)];
    __shared__ __attribute__((aligned(16))) uint16_t ss[Tiles::P * D * M];        // S before the block, [d][m]
    __shared__ __attribute__((aligned(16))) float sz[D];                          // z before the block
    __shared__ float sdel[2][2][16];
    __shared__ float srho[2][D];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int seg = blockIdx.x % a.nseg, bh = blockIdx.x / a.nseg;
    int blk0, count;
    blk_range(a, seg, blk0, count);
    char *const scratch = reinterpret_cast<char *>(kOwn ? tiles : tiles + Tiles::kElems);
    float *const tot = a.totals != nullptr ? a.totals + ((size_t)bh * a.nseg + seg) * state_stride(D, M) : nullptr;
    Tiles tl(a, tiles, bh, tid, wave);
    if constexpr (Tiles::kWaves == 8) {
        if (wave < 4) {
            OutRole out(a, tl, bh, tid, wave, ss, sz, sdel, srho, scratch);
            blk_loop(tl, blk0, 1, count, out);
            if (tot != nullptr) out.end();
        } else {
            StateRole st(a, tl, bh, seg, tid, wave, ss, sz);
            blk_loop(tl, blk0, 1, count, st);
            if (tot != nullptr) st.end(tot);
        }
    } else {
        OutRole out(a, tl, bh, tid, wave, ss, sz, sdel, srho, scratch);
        StateRole st(a, tl, bh, seg, tid, wave, ss, sz);
        blk_loop(tl, blk0, 1, count, out, st);
        if (tot != nullptr) {
            out.end();
            st.end(tot);
        }
    }
    if (tot != nullptr) {
        __syncthreads();
        if (tid < D) tot[D * M + tid] = srho[0][tid] + srho[1][tid];
    }
}

// ---- dV and dK (eq. 14-15) -------------------------------------------------------------------------
// Out role (i, j): the 16 tokens of sub-block i, dV (j = 0) or dK (j = 1).  kJ: j where the waves of either have code
// of their own, and registers for what that code keeps over the blocks; -1 where a wave may have both.
template <int D, int M, typename T, bool kStrided, int kJ>
struct RevOut : BlkLane {
    using Tiles = BlkTiles<kLeadK, D, M, T, kStrided>;
    static constexpr int P = Tiles::P, PV = Tiles::PV, PG = Tiles::PG, TD = D / 16, TM = M / 16, SD = D / 32, SM = M / 32;
    static constexpr int TX = TD > TM ? TD : TM;
    static constexpr bool kPair = is_bf16<T>;
    using RowsV = OutRows<T, TM>;
    using RowsK = OutRows<T, TD>;
    static constexpr int kScratch = RowsV::kScratch > RowsK::kScratch ? RowsV::kScratch : RowsK::kScratch;
    const Tiles &tl;
    const uint16_t *sr;
    const float *srho, *sdel;
    char *scratch;
    T *outv, *outk;
    int N, row;
    f32x4 out[TX];           // dV: columns m, dK: columns d, col_of(t, 4g + r) of the token

    __device__ __forceinline__ RevOut(const PassArgs &a, const Tiles &t, int bh, int tid, int wave, const uint16_t *sr_,
                                      const float *srho_, const float *sdel_, char *scratch_)
        : BlkLane(tid, wave), tl(t), sr(sr_), srho(srho_), sdel(sdel_), scratch(scratch_ + 512 * (wave & 3)) {
        outv = static_cast<T *>(a.out) + seq_base<kStrided>(a.N, a.heads, bh, M);
        outk = static_cast<T *>(a.out2) + seq_base<kStrided>(a.N, a.heads, bh, qk_width<T>(D));
        N = a.N, row = 16 * i + c;
    }
    __device__ __forceinline__ int j() const { return kJ < 0 ? h : kJ; }
    __device__ __forceinline__ void init() {}
    __device__ __forceinline__ void publish() {}
    __device__ __forceinline__ void fetch(int) {}
    __device__ __forceinline__ void parked(int) {}
    // rows a of the block against the role's tokens b (lane c), kept where a >= b
    __device__ __forceinline__ void keep(f32x4 &w0, f32x4 &w1) const {
#pragma unroll
        for (int r = 0; r < 4; ++r) {        // select, never multiply
            w0[r] = (i == 0 && 4 * g + r >= c) ? w0[r] : 0.f;
            w1[r] = (i == 0 || 4 * g + r >= c) ? w1[r] : 0.f;
        }
    }
    __device__ __forceinline__ void products() {
        const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
        f32x4 w0 = zero4, w1;
        if (j() == 0) {
            // scores phi(Q_a) . phi(K_b) (kRaw: times the rest of 1/den_a)
            Op<P> kt[SD];
            read_toks<D, P>(tl.sk, kBlk * D, row, g, kt);
            if (i == 0) {
                Op<P> qt[SD];
                read_toks<D, P>(tl.sq, kBlk * D, c, g, qt);
                w0 = dot(qt, kt, zero4);
            }
            {
                Op<P> qt[SD];
                read_toks<D, P>(tl.sq, kBlk * D, 16 + c, g, qt);
                w1 = dot(qt, kt, zero4);
            }
            keep(w0, w1);
#pragma unroll
            for (int t = 0; t < TM; ++t) {
                Op<P> rr[SD];
                read_toks<D, P>(sr, M * D, col_of<kPair>(t, c), g, rr);
                out[t] = dot(rr, kt, zero4);
            }
            const Op<P> wop = op_of<P>(w0, w1);
#pragma unroll
            for (int t = 0; t < TM; t += 2) {
                const Op<PG> gf[2] = {read_feat<M, PG, kPair>(tl.sg, kBlk * M, 0, t, lane),
                                      read_feat<M, PG, kPair>(tl.sg, kBlk * M, 0, t + 1, lane)};
                const Op<P> wo[2] = {wop, wop};
                f32x4 o[2] = {out[t], out[t + 1]};
                mma_n(gf, wo, o);
                out[t] = o[0], out[t + 1] = o[1];
            }
        } else {
            // scores V_b . dO_a/den_a + delta_a (kRaw: over the rest of 1/den_a, which phi(Q_a) brings)
            Op<PV> vt[SM];
            read_toks<M, PV>(tl.sv, kBlk * M, row, g, vt);
            if (i == 0) {
                Op<PG> gt[SM];
                read_toks<M, PG>(tl.sg, kBlk * M, c, g, gt);
                w0 = dot(gt, vt, *reinterpret_cast<const f32x4 *>(sdel + 4 * g));
            }
            {
                Op<PG> gt[SM];
                read_toks<M, PG>(tl.sg, kBlk * M, 16 + c, g, gt);
                w1 = dot(gt, vt, *reinterpret_cast<const f32x4 *>(sdel + 16 + 4 * g));
            }
            keep(w0, w1);
#pragma unroll
            for (int t = 0; t < TD; ++t) {
                Op<P> rr[SM];
#pragma unroll
                for (int s = 0; s < SM; ++s) rr[s] = read_feat<D, P, kPair, true>(sr, M * D, 32 * s, t, lane);
                out[t] = dot(rr, vt, *reinterpret_cast<const f32x4 *>(srho + col_of<kPair>(t, 4 * g)));
            }
            const Op<P> wop = op_of<P>(w0, w1);
            int rowk = row, lk = lane;
            if constexpr (kJ >= 0) asm volatile("" : "+v"(rowk), "+v"(lk));      // addresses formed per block, not kept: 128 registers
#pragma unroll
            for (int t = 0; t < TD; t += 2) {
                const Op<P> qf[2] = {read_feat<D, P, kPair>(tl.sq, kBlk * D, 0, t, lk),
                                     read_feat<D, P, kPair>(tl.sq, kBlk * D, 0, t + 1, lk)};
                const Op<P> wo[2] = {wop, wop};
                f32x4 o[2] = {out[t], out[t + 1]};
                mma_n(qf, wo, o);
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const f32x4 f = tl.full_values(rowk, col_of<kPair>(t + u, 4 * (lk >> 4)) >> 2);
#pragma unroll
                    for (int r = 0; r < 4; ++r) out[t + u][r] = o[u][r] * feature_slope<T>(f[r]);
                }
            }
        }
    }
    __device__ __forceinline__ void finish(int blk) {
        const int t0 = blk * kBlk, nv = min(kBlk, N - t0);
        constexpr int kStride = kScratchInTiles<D, M> ? 2 * kBlk * D : 4 * 512;
        if constexpr (is_poly<T>) {      // (four waves, as in the dQ pass)
            if (j() == 0)
                RowsV::template store<kStride>(scratch, rows_of(outv + (size_t)t0 * tl.tsm, tl.tsm, nv), 16 * i * tl.tsm * (int)sizeof(T),
                                               tl.tsm, reinterpret_cast<const f32x4 (&)[TM]>(out), lane, tl.nt_out);
            __syncthreads();
            float *rows = reinterpret_cast<float *>(tl.sk);
            if (j() != 0) {
#pragma unroll
                for (int t = 0; t < TD; ++t) *reinterpret_cast<f32x4 *>(rows + row * kChainStride + 16 * t + 4 * g) = out[t];
            }
            __syncthreads();
            blk_chain(rows, tl.Ks + (size_t)t0 * tl.tsd, outk + (size_t)t0 * tl.tsd, tl.tsd, nv, tl.tid);
            __syncthreads();
        } else if (TD == TM || j() == 0) {
            T *o = TD == TM && j() != 0 ? outk : outv;
            RowsV::template store<kStride>(scratch, rows_of(o + (size_t)t0 * tl.tsm, tl.tsm, nv), 16 * i * tl.tsm * (int)sizeof(T), tl.tsm,
                                           reinterpret_cast<const f32x4 (&)[TM]>(out), lane, tl.nt_out);
        } else {
            RowsK::template store<kStride>(scratch, rows_of(outk + (size_t)t0 * tl.tsd, tl.tsd, nv), 16 * i * tl.tsd * (int)sizeof(T), tl.tsd,
                                           reinterpret_cast<const f32x4 (&)[TD]>(out), lane, tl.nt_out);
        }
    }
};

// State role (i, j): R (D x M), D / 32 x M / 32 tiles, published as [m][d]: dV reads its rows, dK reads them
// transposed; and one tile of rho = sum delta phi(Q), the ones column.
template <int D, int M, typename T, bool kStrided>
struct RevState : BlkLane {
    using Tiles = BlkTiles<kLeadK, D, M, T, kStrided>;
    static constexpr int P = Tiles::P, PG = Tiles::PG, DT = D / 32, MT = M / 32;
    const PassArgs &a;
    const Tiles &tl;
    uint16_t *sr;
    float *srho, *sdel;
    const float *delta, *rden;
    int bh, seg, rt, tid;
    float ndel, nrden;
    f32x4 U[DT][MT];       // element (d = 16 (i DT + x) + 4g + r, m = 16 (h MT + y) + c)
    f32x4 rho;             // element d = 16 rt + 4g + r

    __device__ __forceinline__ RevState(const PassArgs &a_, const Tiles &t, int bh_, int seg_, int tid_, int wave, uint16_t *sr_, float *srho_, float *sdel_)
        : BlkLane(tid_, wave), a(a_), tl(t), sr(sr_), srho(srho_), sdel(sdel_), bh(bh_), seg(seg_), tid(tid_) {
        delta = a.delta + (size_t)bh * a.N, rden = a.rden + (size_t)bh * a.N;
        rt = DT == 2 ? 2 * i + h : i;
        ndel = 0.f, nrden = 1.f;
    }
    __device__ __forceinline__ void add(const float *sm, const float *v) {
#pragma unroll
        for (int x = 0; x < DT; ++x)
#pragma unroll
            for (int y = 0; y < MT; ++y)
#pragma unroll
                for (int r = 0; r < 4; ++r) U[x][y][r] += sm[(16 * (i * DT + x) + 4 * g + r) * M + 16 * (h * MT + y) + c];
        rho += load4_state(v + 16 * rt + 4 * g);
    }
    __device__ __forceinline__ void init() {
        rho = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int x = 0; x < DT; ++x)
#pragma unroll
            for (int y = 0; y < MT; ++y) U[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (a.init_S != nullptr) add(a.init_S + (size_t)bh * D * M, a.init_z + (size_t)bh * D);
        if (a.state != nullptr) {
            int nslots, lo, hi;
            state_slots(a, seg, kStateSuffix, nslots, lo, hi);
            for (int j = lo; j < hi; ++j) {
                const float *st = a.state + ((size_t)bh * nslots + j) * state_stride(D, M);
                add(st, st + D * M);
            }
        }
    }
    __device__ __forceinline__ void publish() {
        la::publish<D, P>(sr, M * D, U, i * DT, h * MT, c, g);
        if (c == 0) *reinterpret_cast<f32x4 *>(srho + 16 * rt + 4 * g) = rho;
    }
    // one wave brings delta (kRaw: over the rest of 1/den, as the scores of dK are)
    __device__ __forceinline__ void fetch(int blk) {
        if (i == 0 && h == 0) {
            const int token = min(blk * kBlk + (lane & 31), a.N - 1);
            ndel = delta[token];
            if constexpr (Tiles::kRaw) nrden = rden[token];
        }
    }
    __device__ __forceinline__ void parked(int blk) {
        if (i == 0 && h == 0 && lane < kBlk) {
            const float d = Tiles::kRaw ? ndel * __builtin_amdgcn_rcpf(rest_of(nrden)) : ndel;
            sdel[lane] = blk * kBlk + lane < a.N ? d : 0.f;
        }
    }
    __device__ __forceinline__ void products() {
        const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
        Op<P> qn[DT];
#pragma unroll
        for (int x = 0; x < DT; ++x) qn[x] = read_feat<D, P, false>(tl.sq, kBlk * D, 0, i * DT + x, lane);
#pragma unroll
        for (int y = 0; y < MT; ++y) {
            const Op<PG> gf = read_feat<M, PG, false>(tl.sg, kBlk * M, 0, h * MT + y, lane);
            Op<PG> gg[DT];
            f32x4 u[DT];
#pragma unroll
            for (int x = 0; x < DT; ++x) gg[x] = gf, u[x] = zero4;
            mma_n(qn, gg, u);
#pragma unroll
            for (int x = 0; x < DT; ++x) U[x][y] += u[x];
        }
        // rho, an fp32 sum: three parts on both sides whatever P is
        const Op<3> dop[1] = {op_of<3>(*reinterpret_cast<const f32x4 *>(sdel + 4 * g),
                                       *reinterpret_cast<const f32x4 *>(sdel + 16 + 4 * g))};
        f32x4 rr[1] = {zero4};
        if (DT == 1 || h == 0) {
            const Op<3> q1[1] = {full_feat<D>(qn[0], tl.sq, kBlk * D, rt, lane)};
            mma_n(q1, dop, rr);
        } else {
            const Op<3> q1[1] = {full_feat<D>(qn[DT - 1], tl.sq, kBlk * D, rt, lane)};
            mma_n(q1, dop, rr);
        }
        rho += rr[0];
    }
    __device__ __forceinline__ void finish(int) {}
    // what has piled up when the first segment is through is the gradient for the initial state
    __device__ __forceinline__ void end() {
        if (seg == 0 && a.final_S != nullptr) {
            float *s1 = a.final_S + (size_t)bh * D * M;
#pragma unroll
            for (int x = 0; x < DT; ++x)
#pragma unroll
                for (int y = 0; y < MT; ++y)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        s1[(16 * (i * DT + x) + 4 * g + r) * M + 16 * (h * MT + y) + c] = U[x][y][r];
        }
        if (seg == 0 && a.final_z != nullptr && c == 0 && (DT == 2 || h == 0))
            *reinterpret_cast<f32x4 *>(a.final_z + (size_t)bh * D + 16 * rt + 4 * g) = rho;
    }
};

template <int D, int M, typename T, bool kStrided = false>
__global__ __launch_bounds__((kWave * kBwdWaves<D, M, T>)) __attribute__((amdgpu_waves_per_eu((kBwdWaves<D, M, T> / 2)))) void reverse_block_kernel(
    const PassArgs a) {
    using Tiles = BlkTiles<kLeadK, D, M, T, kStrided>;
    using OutRole = RevOut<D, M, T, kStrided, -1>;
    using StateRole = RevState<D, M, T, kStrided>;
    constexpr bool kOwn = kScratchInTiles<D, M>;
    __shared__ __attribute__((aligned(16))) uint16_t tiles[Tiles::kElems + (kOwn ? 0 : 4 * OutRole::kScratch / 2)];
    __shared__ __attribute__((aligned(16))) uint16_t sr[Tiles::P * M * D];        // R after the block, [m][d]
    __shared__ __attribute__((aligned(16))) float srho[D];
    __shared__ __attribute__((aligned(16))) float sdel[kBlk];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int seg = blockIdx.x % a.nseg, bh = blockIdx.x / a.nseg;
    int blk0, count;
    blk_range(a, seg, blk0, count);
    char *const scratch = reinterpret_cast<char *>(kOwn ? tiles : tiles + Tiles::kElems);
    Tiles tl(a, tiles, bh, tid, wave);
    if constexpr (Tiles::kWaves == 8) {
        constexpr bool kOwnCode = !is_bf16<T> && (D == 64 || M == 64);        // (fp32 32 x 32 step 64 x 784 36.5 -> 36.8 us with it)
        if (kOwnCode && wave < 2) {
            RevOut<D, M, T, kStrided, 0> out(a, tl, bh, tid, wave, sr, srho, sdel, scratch);
            blk_loop(tl, blk0 + count - 1, -1, count, out);
        } else if (wave < 4) {
            RevOut<D, M, T, kStrided, kOwnCode ? 1 : -1> out(a, tl, bh, tid, wave, sr, srho, sdel, scratch);
            blk_loop(tl, blk0 + count - 1, -1, count, out);
        } else {
            StateRole st(a, tl, bh, seg, tid, wave, sr, srho, sdel);
            blk_loop(tl, blk0 + count - 1, -1, count, st);
            st.end();
        }
    } else {
        OutRole out(a, tl, bh, tid, wave, sr, srho, sdel, scratch);
        StateRole st(a, tl, bh, seg, tid, wave, sr, srho, sdel);
        blk_loop(tl, blk0 + count - 1, -1, count, out, st);
        st.end();
    }
}

}  // namespace la
