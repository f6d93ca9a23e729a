// RNTN cell (Section 6.1 names the model; the form used is h_k = tanh(a^T V_k a + (a W)_k + b_k)
// with a = [h_left ; h_right], V of shape d x 2d x 2d).
//
// a^T V_k a does not change when V_k[p][q] and V_k[q][p] are put together on one side of the diagonal:
//     a^T V_k a = sum_q a_q T_q[k],    T_q[k] = sum_{p <= q} a_p S_k[p][q],    S_k[p][q] = V_k[p][q] + V_k[q][p] (p < q), V_k[q][q] (p = q)
// so for every q (a "slice") the tile's rows are multiplied with the first q + 1 rows of a [2d x 16] matrix of one column group
// (16 outputs k), and the 16x16 result is scaled per row by a_q and added up in registers: ceil((q + 1) / 32) k-steps of 32 instead
// of all of them, 5/8 of the products at d = 64.  The linear term is one more slice (B = W, no factor).
//
// The products run on the 16-bit matrix unit with fp32 operands as two fp16 terms, three products each (cell_split.hpp says what
// that does to a value): a row of the tile is scaled by the power of two that brings its largest magnitude into [2^14, 2^15) - leaves hold
// embedding rows of any magnitude - and every column of a slice to [2^13, 2^14).  The factor a_q is the fp32 value itself.  A sum
// that does not come out finite (an infinite operand has no two terms, and scaled sums overflow 2^15 earlier) is taken again in fp32 from the parameters
// as given.
// Measured (level kernel, whole forward; before: fp32 instructions, all products): 256 parse trees at d = 64 342 -> 205 us, 150 at d = 96 808 -> 288,
// 8 at d = 64 201 -> 132, 4 at d = 8 101 -> 80; error against 64 bits unchanged (1.4e-6 to 1.7e-6).  What is left is the chain of a frontier (records, rows,
// parts, barrier), about 12 us each.
#pragma once

#include <utility>

#include "cell_tile.hpp"
#include "cell_split.hpp"

namespace tl {

// Packed S (+ W) of one column group: units of one k-step, [unit][hi, lo][lane][8] with p = 32 s + 8 (lane / 16) + i on the padded axis
// (segments of Lp rows, zeros up to 32 n_steps) and k = 16 cg + lane % 16; slice q has q / 32 + 1 units from rntn_unit(q) on, the
// linear one n_steps units from rntn_unit(32 n_steps) on.  Scales: [column group][slice 0 .. 32 n_steps][16].
__host__ __device__ constexpr int rntn_unit(int q) { return 16 * (q >> 5) * ((q >> 5) + 1) + (q & 31) * ((q >> 5) + 1); }
__host__ __device__ constexpr int rntn_units_of(int n_steps) { return rntn_unit(32 * n_steps) + n_steps; }

// One column of a slice (q < Q, unit k; q = Q: the linear term) from the matrix of k_rntn_build_s (backward.hpp): s[(k, q)][p] = V[k][p][q] +
// V[k][q][p], s[d * 2d + k][p] = W[p][k].  A lane holds, of the column of lane % 16, eight neighbours of every k-step.
constexpr int RNTN_MAX_STEPS = 8;
struct RntnColumn {
    halfx8 hi[RNTN_MAX_STEPS], lo[RNTN_MAX_STEPS];
    float scale;            // what a sum of products is multiplied by
};
// (full: all rows p, as they stand in s - the operand gradient's matrix)
__device__ inline RntnColumn rntn_column(const float *__restrict__ s, int d, int Lp, int Q, int q, int k, int lane, bool full = false)
{
    const int D2 = 2 * d;
    const bool linear = q == Q;
    const int qseg = q / Lp, ql = qseg * d + (q - qseg * Lp);       // logical index of a_q
    const bool live = k < d && (linear || (qseg < 2 && q - qseg * Lp < d));
    const float *row = s + (linear ? (size_t)d * D2 + k : (size_t)k * D2 + ql) * D2;
    float x[RNTN_MAX_STEPS][8];
    unsigned m = 0u;
#pragma unroll
    for (int t = 0; t < RNTN_MAX_STEPS; ++t)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int p = 32 * t + 8 * (lane >> 4) + i, pseg = p / Lp, off = p - pseg * Lp;
            float v = 0.f;
            if (live && pseg < 2 && off < d && (linear || full || p <= q)) v = row[pseg * d + off] * (!linear && !full && p == q ? 0.5f : 1.f);
            x[t][i] = v;
            const unsigned u = __float_as_uint(v) & 0x7FFFFFFFu;
            if (u < 0x7F800000u) m = max(m, u);                     // (an infinity or a NaN is packed as NaN terms: lo = inf - inf)
        }
    m = max(m, (unsigned)__shfl_xor((int)m, 16));
    m = max(m, (unsigned)__shfl_xor((int)m, 32));
    const int e = min(13 - ((int)(m >> 23) - 127), 100);            // the column is scaled by 2^e
    RntnColumn c;
    c.scale = k < d ? ldexpf(1.f, -e) : 0.f;
#pragma unroll
    for (int t = 0; t < RNTN_MAX_STEPS; ++t)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float v = ldexpf(x[t][i], e);
            c.hi[t][i] = (_Float16)v;
            c.lo[t][i] = (_Float16)(v - (float)c.hi[t][i]);
        }
    return c;
}
// One wave per column group and slice.
__device__ inline void pack_rntn_tile(const float *__restrict__ s, _Float16 *__restrict__ vp, float *__restrict__ scale, int d, int Lp, int n_steps,
                                      int item, int lane)
{
    const int Q = 32 * n_steps, cg = item / (Q + 1), q = item - cg * (Q + 1);
    const int steps = q == Q ? n_steps : (q >> 5) + 1;
    const RntnColumn c = rntn_column(s, d, Lp, Q, q, cg * HU + (lane & 15), lane);
    if (lane < 16) scale[((size_t)cg * (Q + 1) + q) * HU + lane] = c.scale;
    halfx8 *dst = reinterpret_cast<halfx8 *>(vp) + ((size_t)cg * rntn_units_of(n_steps) + rntn_unit(q)) * 2 * 64 + lane;
#pragma unroll
    for (int t = 0; t < RNTN_MAX_STEPS; ++t) {
        if (t >= steps) break;
        dst[(size_t)t * 128] = c.hi[t];
        dst[(size_t)t * 128 + 64] = c.lo[t];
    }
}

// Order of summation over q, the same however the work is spread: the slices fall into 16 classes by
// q mod 16; a class is added up in ascending q on one accumulator, class s < n_steps then takes k-step s of the linear slice; part p
// (p = 0..3) is the sum of the classes p, p + 4, p + 8, p + 12 in that order; the result is ((part 0 + part 1) + part 2) + part 3,
// then the row's scale and the bias.
// A workgroup evaluates one part of a tile and column group (sm.cmd[5] = p; its four waves take one class each),
// or all four parts one after the other (sm.cmd[5] = -1).  With one part per workgroup, four workgroups share a
// tile and column group: each leaves its part in a scratch area (unit sm.cmd[6] of it), counts itself done, and
// the one that completes the count adds the parts up and writes h.  A height of a few rows thus spreads over
// four times as many workgroups, each with a quarter of the slices: with d = 64 there are only four column
// groups, and a block of 16 rows costs the same products whatever the number of rows.
constexpr int RNTN_PARTS = 4;
constexpr int RNTN_PART_FLOATS = TILE_ROWS * HU;            // one part of one tile and column group in the scratch area
// Tiles that the grid works on at once when a tile and column group is shared by RNTN_PARTS workgroups: a frontier is cut
// (plan_level) so that its tiles fill one round of the grid where they can - a second round of small tiles costs a whole
// item's latency more (records, child rows, first slice, exchange, scratch area), taller tiles only their matrix instructions.
__host__ __device__ inline int rntn_cap_tiles(int cap_tiles, int rntn_units)
{
    return rntn_units > 0 && cap_tiles >= RNTN_PARTS ? cap_tiles / RNTN_PARTS : cap_tiles;
}

template <typename F, int... I> __device__ __forceinline__ void static_for_each(F &&f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F> __device__ __forceinline__ void static_for(F &&f)
{
    static_for_each(f, std::make_integer_sequence<int, N>{});
}

// LDS of a tile, in the streaming cell's staging area.  Up to 64 hidden units the rows are split once, by the wave that has the row
// block, and read back as matrix operands by all; above (NS = 8) there is no room beside the fp32 rows, and every wave splits
// them for itself, two row blocks at a time.
template <int NS> struct RntnSmem {
    static constexpr int LD = 32 * NS + 4;
    static constexpr bool SPLIT_ONCE = NS <= 4;
    float a[TILE_ROWS * LD];                                // the tile's gathered rows
    float red[4 * 2 * 4 * 64];                              // [wave][2 row blocks x 4 values][lane]
    float back[TILE_ROWS];                                  // what a row's sums are multiplied by
    halfx8 split[SPLIT_ONCE ? 4 * NS * 2 * 64 : 1];         // [row block][k-step][hi, lo][lane]
};

// The k-steps of a class as one stream of units: slice j of the class is q = class + 16 j with j / 2 + 1 k-steps.
__host__ __device__ constexpr int rntn_first(int j) { return (j >> 1) * ((j >> 1) + 1) + (j & 1) * ((j >> 1) + 1); }
constexpr int rntn_slice_of(int u) { int j = 0; while (rntn_first(j + 1) <= u) ++j; return j; }

// Row blocks rb0 .. rb0 + RB - 1 of a tile: sums of this wave's class of part pp, accumulated into out.  RING units of the packed matrix
// are kept in flight (an L2 round trip is longer than a slice's products when there are few rows); the first of them are
// requested by rntn_start, before the rows are waited for.
template <int NS, int RB, int RING> struct RntnStream {
    static constexpr int UNITS = NS * (NS + 1);
    halfx8 b[RING][2];
    __amdgpu_buffer_rsrc_t vp;                              // the column group's matrix (scalar base and offsets: vector registers are short)
    int cls, nq, lane_off;
    static __device__ __forceinline__ halfx8 fetch(__amdgpu_buffer_rsrc_t r, int lane_off, int unit, int e)
    {
        return __builtin_bit_cast(halfx8, __builtin_amdgcn_raw_buffer_load_b128(r, lane_off, (unit * 2 + e) * 1024, 0));
    }
    template <int U> __device__ __forceinline__ void load()
    {
        if constexpr (U < UNITS) {
            constexpr int J = rntn_slice_of(U), G = J >> 1, S = U - rntn_first(J);
            if (cls + 16 * J < nq) {
                const int unit = rntn_unit(16 * J) + cls * (G + 1) + S;
                b[U % RING][0] = fetch(vp, lane_off, unit, 0);
                b[U % RING][1] = fetch(vp, lane_off, unit, 1);
            }
        }
    }
    __device__ __forceinline__ void start(__amdgpu_buffer_rsrc_t vp_, int cls_, int nq_, int lane)
    {
        vp = vp_; cls = cls_; nq = nq_; lane_off = lane * 16;
        static_for<RING>([&](auto u) __attribute__((always_inline)) { load<decltype(u)::value>(); });
    }
    static __device__ __forceinline__ float scale_of(__amdgpu_buffer_rsrc_t scale, int lane, int slice)
    {
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(scale, (lane & 15) * 4, slice * (HU * 4), 0));
    }
    // scale: of this column group, [slice][16]; rows: the fp32 rows of block rb0
    __device__ __forceinline__ void run(const halfx8 (&a)[RB][NS][2], __amdgpu_buffer_rsrc_t scale, const float *rows, int ld, int lane, floatx4 (&out)[RB])
    {
        floatx4 t[RB];
        float sc = scale_of(scale, lane, cls);
        static_for<UNITS>([&](auto uc) __attribute__((always_inline)) {
            constexpr int U = decltype(uc)::value, J = rntn_slice_of(U), S = U - rntn_first(J);
            constexpr bool FIRST = S == 0, LAST = S == (J >> 1);
            if (cls + 16 * J < nq) {
                if constexpr (FIRST) {
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) t[rb] = floatx4{0.f, 0.f, 0.f, 0.f};
                }
                const halfx8 hi = b[U % RING][0], lo = b[U % RING][1];
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) t[rb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[rb][S][0], hi, t[rb], 0, 0, 0);
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) t[rb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[rb][S][0], lo, t[rb], 0, 0, 0);
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) t[rb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[rb][S][1], hi, t[rb], 0, 0, 0);
                load<U + RING>();
                if constexpr (LAST) {
                    // scale accumulator row (4 (lane/16) + v) by that row's a_q
                    const float *m = rows + (size_t)(lane >> 4) * 4 * ld + cls + 16 * J;
                    const float sc_now = sc;
                    sc = scale_of(scale, lane, min(cls + 16 * (J + 1), 32 * NS));
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                        for (int v = 0; v < 4; ++v) out[rb][v] = __builtin_fmaf(m[(rb * 16 + v) * ld] * sc_now, t[rb][v], out[rb][v]);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        });
    }
};

template <int NS, bool VEC4, bool COH>
__device__ __forceinline__ void rntn_gather(RntnSmem<NS> &s, const TileSmem &sm, const Fwd &f, const Gemm &gm, int nrb)
{
    for (int g = threadIdx.x; g < nrb * 16 * NS * 8; g += WG_THREADS) {
        const int row = g / (NS * 8), k4 = g - row * (NS * 8);
        const floatx4 v = load_a_granule<2, VEC4, COH>(f.h, f.zeros, gm.L, gm.Lp, sm.src0[row], sm.src1[row], k4 * 4);
        *reinterpret_cast<floatx4 *>(&s.a[row * RntnSmem<NS>::LD + k4 * 4]) = v;
    }
}

// Row block rb as matrix operands: lane l holds row l & 15, k = 32 step + 8 (l >> 4) ... + 7.
template <int NS> __device__ __forceinline__ void rntn_split_rows(RntnSmem<NS> &s, int rb, int lane, halfx8 (&a)[NS][2])
{
    const float *row = &s.a[(rb * 16 + (lane & 15)) * RntnSmem<NS>::LD + 8 * (lane >> 4)];
    float m = 0.f;
#pragma unroll
    for (int t = 0; t < NS; ++t)
#pragma unroll
        for (int i = 0; i < 8; ++i) m = fmaxf(m, fabsf(row[32 * t + i]));
    m = max_across_quarters(m);
    const unsigned eb = max(__float_as_uint(m) >> 23, 15u);
    const float scale = __uint_as_float((268u - eb) << 23);
    if (lane < 16) s.back[rb * 16 + lane] = __uint_as_float((eb - 14u) << 23);
#pragma unroll
    for (int t = 0; t < NS; ++t)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float v = row[32 * t + i] * scale;
            a[t][0][i] = (_Float16)v;
            a[t][1][i] = (_Float16)(v - (float)a[t][0][i]);
        }
}

// A node's sum in fp32 from the parameters as given; `row`: its gathered row (rare, and slow).
__device__ __forceinline__ float rntn_sum_plain(const Fwd &f, const Gemm &gm, const float *row, int k)
{
    const int d = f.H, D2 = 2 * d;
    float sum = 0.f;
#pragma unroll 1
    for (int q = 0; q < D2; ++q) {
        float t = 0.f;
#pragma unroll 1
        for (int p = 0; p < D2; ++p) t = __builtin_fmaf(row[p < d ? p : gm.Lp + p - d], f.rntn_v[((size_t)k * D2 + p) * D2 + q], t);
        const float aq = row[q < d ? q : gm.Lp + q - d];
        sum = __builtin_fmaf(aq, t, sum);
        sum = __builtin_fmaf(aq, f.xi.w[(size_t)q * d + k], sum);
    }
    return sum;
}

// The parts of this workgroup for row blocks rb0 .. rb0 + RB - 1; mine: what wave w has of row block w when they meet.
template <int NS, int RB, bool VEC4, bool COH>
__device__ __forceinline__ void rntn_blocks(RntnSmem<NS> &s, const TileSmem &sm, const Fwd &f, const Gemm &gm, int nrb, int rb0, int cg, float (&mine)[4])
{
    constexpr int LD = RntnSmem<NS>::LD, UNITS = NS * (NS + 1);
    // Beside the operands of few rows there are registers for many units.  Four row blocks at NS = 4 (two at 8) take 128 of the 256 for
    // operands, and with more than two units the kernels that walk all heights spill (4 / 3 / 2 units: 21 / 10 / 4 registers; 256 parse trees at
    // d = 64, level by level 219 / 210 / 205 us, 6 chains of 250 leaves 2 842 / 2 752 / 2 670).
    constexpr int RING = RB * NS <= 8 ? (UNITS < 12 ? UNITS : 12) : 2;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int part = __builtin_amdgcn_readfirstlane(sm.cmd[5]);             // written by the caller before its barrier
    constexpr unsigned CG_BYTES = rntn_units_of(NS) * 2048u, CG_SLICES = 32 * NS + 1;
    const __amdgpu_buffer_rsrc_t vp = buf_of(static_cast<const char *>(gm.wp) + (size_t)cg * CG_BYTES, CG_BYTES),
                                 scale = buf_of(f.xi.scale + (size_t)cg * CG_SLICES * HU, CG_SLICES * HU * 4u);
    const int nq = 2 * gm.Lp;
    const int p_lo = part < 0 ? 0 : part, p_hi = part < 0 ? RNTN_PARTS - 1 : part;
    using Stream = RntnStream<NS, RB, RING>;
    Stream stream;
    stream.start(vp, p_lo + RNTN_PARTS * wave, nq, lane);
    halfx8 a[RB][NS][2];
    if (rb0 == 0) {
        rntn_gather<NS, VEC4, COH>(s, sm, f, gm, nrb);
        __syncthreads();
    }
    if constexpr (RntnSmem<NS>::SPLIT_ONCE) {
        if (wave < nrb) {
            halfx8 own[NS][2];
            rntn_split_rows<NS>(s, wave, lane, own);
#pragma unroll
            for (int t = 0; t < NS; ++t)
#pragma unroll
                for (int e = 0; e < 2; ++e) s.split[((wave * NS + t) * 2 + e) * 64 + lane] = own[t][e];
        }
        __syncthreads();
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int t = 0; t < NS; ++t)
#pragma unroll
                for (int e = 0; e < 2; ++e) a[rb][t][e] = s.split[((rb * NS + t) * 2 + e) * 64 + lane];
    } else {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) rntn_split_rows<NS>(s, rb0 + rb, lane, a[rb]);
    }
#pragma unroll 1
    for (int pp = p_lo; pp <= p_hi; ++pp) {
        const int cls = pp + RNTN_PARTS * wave;             // this wave's class of the part
        if (pp != p_lo) stream.start(vp, cls, nq, lane);
        floatx4 out[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) out[rb] = floatx4{0.f, 0.f, 0.f, 0.f};
        halfx8 lin[2];
        float lin_scale = 0.f;
        if (cls < NS) {                                     // k-step cls of the linear slice
            lin[0] = Stream::fetch(vp, lane * 16, rntn_unit(32 * NS) + cls, 0);
            lin[1] = Stream::fetch(vp, lane * 16, rntn_unit(32 * NS) + cls, 1);
            lin_scale = Stream::scale_of(scale, lane, 32 * NS);
        }
        stream.run(a, scale, &s.a[rb0 * 16 * LD], LD, lane, out);
        if (cls < NS) {
            // (not a loop with `t == cls` in it: that becomes an index known at run time, and the operands go to memory)
            static_for<NS>([&](auto tc) __attribute__((always_inline)) {
                constexpr int t = decltype(tc)::value;
                if (t == cls) {
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) {
                        floatx4 x = {0.f, 0.f, 0.f, 0.f};
                        x = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[rb][t][0], lin[0], x, 0, 0, 0);
                        x = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[rb][t][0], lin[1], x, 0, 0, 0);
                        x = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[rb][t][1], lin[0], x, 0, 0, 0);
#pragma unroll
                        for (int v = 0; v < 4; ++v) out[rb][v] = __builtin_fmaf(lin_scale, x[v], out[rb][v]);
                    }
                }
            });
        }
        // the part: the four waves' class sums in wave order; wave w takes row block w, two row blocks per round
#pragma unroll
        for (int r0 = 0; r0 < RB; r0 += 2) {
            if (rb0 + r0 >= nrb) break;
            __syncthreads();                                // the exchange area is free again
#pragma unroll
            for (int rbi = 0; rbi < 2 && r0 + rbi < RB; ++rbi)
#pragma unroll
                for (int v = 0; v < 4; ++v) s.red[(wave * 8 + rbi * 4 + v) * 64 + lane] = out[r0 + rbi][v];
            __syncthreads();
            const int rbi = wave - rb0 - r0;
            if (rbi >= 0 && rbi < 2 && r0 + rbi < RB) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float sum = ((s.red[(0 * 8 + rbi * 4 + v) * 64 + lane] + s.red[(1 * 8 + rbi * 4 + v) * 64 + lane]) +
                                       s.red[(2 * 8 + rbi * 4 + v) * 64 + lane]) + s.red[(3 * 8 + rbi * 4 + v) * 64 + lane];
                    mine[v] = pp == p_lo ? sum : mine[v] + sum;
                }
            }
        }
    }
}

template <int NS, bool COH>
__device__ __forceinline__ void rntn_finish(const RntnSmem<NS> &s, const TileSmem &sm, const Fwd &f, const Gemm &gm, int count, int hu, int row, float sum,
                                            float bias)
{
    const int node = row < count ? sm.node[row] : -1;
    if (node < 0) return;
    sum *= s.back[row];
    if (__builtin_expect(!__builtin_isfinite(sum), 0)) sum = rntn_sum_plain(f, gm, &s.a[row * RntnSmem<NS>::LD], hu);
    st_f<COH>(f.h + (size_t)node * f.H + hu, tanh_f(sum + bias));
}

template <int NS, bool VEC4, bool COH>
__device__ __forceinline__ void rntn_tile(TileSmem &sm, const Fwd &f, const Gemm &gm, int count, int cg)
{
    static_assert(sizeof(RntnSmem<NS>) <= sizeof(TileSmem::a) + sizeof(TileSmem::b), "the tile must fit the staging area");
    RntnSmem<NS> &s = reinterpret_cast<RntnSmem<NS> &>(sm);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nrb = (count + 15) >> 4;
    float mine[4] = {0.f, 0.f, 0.f, 0.f};                   // wave w: row block w, parts added up so far
    if (nrb <= 1) rntn_blocks<NS, 1, VEC4, COH>(s, sm, f, gm, nrb, 0, cg, mine);
    else if (nrb <= 2 || NS > 4) {
        rntn_blocks<NS, 2, VEC4, COH>(s, sm, f, gm, nrb, 0, cg, mine);
        if (nrb > 2) rntn_blocks<NS, 2, VEC4, COH>(s, sm, f, gm, nrb, 2, cg, mine);
    } else if constexpr (NS <= 4) rntn_blocks<NS, 4, VEC4, COH>(s, sm, f, gm, nrb, 0, cg, mine);
    const int part = sm.cmd[5], unit = sm.cmd[6];
    const int rb = wave;
    const int hu = cg * HU + (lane & 15);
    const float bias = gm.bp[cg * HU + (lane & 15)];
    if (part < 0) {
        if (rb < nrb && hu < f.H) {
#pragma unroll
            for (int v = 0; v < 4; ++v) rntn_finish<NS, COH>(s, sm, f, gm, count, hu, rb * 16 + (lane >> 4) * 4 + v, mine[v], bias);
        }
        return;
    }
    // ---- one part per workgroup: parts meet in the scratch area, the last one to arrive finishes ----
    float *sc = f.rntn_part + (size_t)(unit * f.n_cg + cg) * RNTN_PARTS * RNTN_PART_FLOATS;
    unsigned int *done = f.rntn_done + (size_t)unit * f.n_cg + cg;
    if (rb < nrb) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = rb * 16 + (lane >> 4) * 4 + v;
            st_dev(sc + part * RNTN_PART_FLOATS + row * HU + (lane & 15), mine[v]);
        }
    }
    wait_mem();
    __syncthreads();
    if (tid == 0) sm.cmd[7] = (int)add_dev(done, 1u);
    __syncthreads();
    if (sm.cmd[7] != RNTN_PARTS - 1) return;                // uniform: not the last part of this tile and column group
    if (tid == 0) st_dev(done, 0u);                         // the counter is ready for its next use
    if (rb < nrb && hu < f.H) {
        float e[4][RNTN_PARTS];
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int p = 0; p < RNTN_PARTS; ++p) e[v][p] = ld_dev(sc + p * RNTN_PART_FLOATS + (rb * 16 + (lane >> 4) * 4 + v) * HU + (lane & 15));
#pragma unroll
        for (int v = 0; v < 4; ++v) rntn_finish<NS, COH>(s, sm, f, gm, count, hu, rb * 16 + (lane >> 4) * 4 + v, ((e[v][0] + e[v][1]) + e[v][2]) + e[v][3], bias);
    }
}

}  // namespace tl
