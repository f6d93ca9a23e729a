// fp32 RNTN cell of the data-flow scheduler: every wave by itself, with the whole matrix of one hidden unit in registers.
//
// The blocks of a slot are those that flow_schedule (structure.hpp) has prepared: 16 internal nodes each, every node's children
// in earlier blocks.  For a block the workgroup gathers the children's fp32 rows (a row by 16 threads, eight neighbouring values at a
// time, requested a block ahead), scales every row [h_left ; h_right] by the power of two that brings its largest magnitude into
// [2^14, 2^15), splits it into two fp16 terms (cell_split.hpp: what that does to a value) and leaves it in LDS as matrix operands; one
// barrier later its four waves read them, each for ONE hidden unit k: the columns of its matrix are the q of the bilinear form
// (cell_rntn.hpp), 16 side by side, with rows p <= q only; the products are scaled by a_q where they are and added up across the lanes
// at the end.  So no sums are exchanged between waves or workgroups.  Lane q mod 16 holds what the other schedulers
// call a class, and classes are added in their order: the same bits.
// Rows that are not written yet show the pattern of cell_ws.hpp (validity carried by the data); no NaN of the parameters or embeddings is
// taken for it.
// d <= 96: 21 units of 8 registers at d = 64, 43 at d = 96 (above, the matrix does not fit and the level kernel stands in).
// Measured (whole forward; level kernel with fp32 instructions / with this cell's products -> this): 256 parse trees at d = 64 342 / 205 -> 105 us, 150 at
// d = 96 808 / 288 -> 157, 8 at d = 64 201 / 132 -> 52, 4 at d = 8 101 / 80 -> 29.  Of the kernel's 84 us at d = 64 the products are 22, the rest
// is the chain of its 33 blocks a slot: rows, split, barrier, store.  (Two workgroups per CU at d = 64, for 32 slots: 144 us, spills.)
#pragma once

#include "cell_rntn.hpp"
#include "structure.hpp"

namespace tl {

constexpr int ROWS_UNITS = 4;     // hidden units of a workgroup, one per wave
constexpr int ROWS_SETTLE_SPINS = 16;   // unsuccessful requests after which a wave asks whether the pattern stands in a leaf's row

template <int NS> struct RowsSmem {
    static constexpr int LD = 32 * NS + 4;
    halfx8 split[2][NS * 2 * 64];                           // alternating per block: [k-step][hi, lo][slot of (k / 8 mod 4, row)]
    float a[2][16 * LD];                         // the rows themselves
    float back[2][16];                                      // what a row's sums are multiplied by
    int node[2][16], tree[2][16];                           // the block's nodes; the tree of which a node is the root, or -1
    int gave_up, leave;
};
// Where the operand of k-step s, eight values `quarter`, row r lies inside its 64 slots: rows are written by threads that differ in the k-step
// and quarter, and read by threads that differ in the row; turned like this both meet all banks.
__device__ inline int rows_slot(int s, int quarter, int r) { return quarter * 16 + (r ^ ((4 * s + quarter) & 15)); }

// Units of a wave's matrix: those of cell_rntn.hpp for one k - slice column q = 16 j + lane % 16, j / 2 + 1 k-steps - and one for the linear term,
// whose column s holds k-step s.
template <int NS> struct RowsGeom {
    static constexpr int QUAD = NS * (NS + 1), UNITS = QUAD + 1;
    static constexpr int SCALES = 2 * NS + 1;               // [scale][lane % 16]
    static constexpr int CPT = (NS + 3) / 4;                // groups of eight values a thread looks after
    static constexpr int SETS_PER_CU = NS <= 3 ? 2 : 1;
};

// The matrices of the RNTN form, from s (see k_pack_rntn): [k][unit][hi, lo][lane][8], scales [k][2 NS + 1][16].  One wave per k and j.
__device__ inline void pack_rntn_rows(const float *__restrict__ s, _Float16 *__restrict__ wp, float *__restrict__ scale, int d, int Lp, int n_steps,
                                      int item, int lane)
{
    const int k = item / (2 * n_steps + 1), j = item - k * (2 * n_steps + 1);
    const bool linear = j == 2 * n_steps;
    const int q = 16 * j + (lane & 15);
    const RntnColumn c = linear ? rntn_column(s, d, Lp, 32 * n_steps, 32 * n_steps, k, lane) : rntn_column(s, d, Lp, 32 * n_steps, q, k, lane);
    if (lane < 16) scale[((size_t)k * (2 * n_steps + 1) + j) * HU + lane] = c.scale;
    halfx8 *dst = reinterpret_cast<halfx8 *>(wp) + ((size_t)k * (n_steps * (n_steps + 1) + 1) + (linear ? n_steps * (n_steps + 1) : rntn_first(j))) * 128 + lane;
#pragma unroll
    for (int t = 0; t < RNTN_MAX_STEPS; ++t) {
        if (linear) {
            if (t == (lane & 15) && t < n_steps) { dst[0] = c.hi[t]; dst[64] = c.lo[t]; }
        } else if (t <= (j >> 1)) {
            dst[(size_t)t * 128] = c.hi[t];
            dst[(size_t)t * 128 + 64] = c.lo[t];
        }
    }
    if (linear && (lane & 15) >= n_steps) dst[0] = dst[64] = halfx8{};
}

// The matrices of the operand gradient (backward.hpp): [p][k / 16][k-step over q][hi, lo][lane][8], scales and linear terms [p][2 n_steps][16].
// One wave per p and 16 of the k.
__device__ inline void pack_rntn_operand(const float *__restrict__ s, _Float16 *__restrict__ wp, float *__restrict__ scale, int d, int Lp, int n_steps,
                                         int item, int lane)
{
    const int p = item / n_steps, j = item - p * n_steps, k = 16 * j + (lane & 15);
    const RntnColumn c = rntn_column(s, d, Lp, 32 * RNTN_MAX_STEPS, (p >= d ? Lp - d : 0) + p, k, lane, true);
    if (lane < 16) {
        scale[((size_t)p * 2 * n_steps + j) * HU + lane] = c.scale;
        scale[((size_t)p * 2 * n_steps + n_steps + j) * HU + lane] = k < d ? s[((size_t)d * 2 * d + k) * 2 * d + p] : 0.f;
    }
    halfx8 *dst = reinterpret_cast<halfx8 *>(wp) + (((size_t)p * n_steps + j) * n_steps) * 128 + lane;
#pragma unroll
    for (int t = 0; t < RNTN_MAX_STEPS; ++t) {
        if (t >= n_steps) break;
        dst[(size_t)t * 128] = c.hi[t];
        dst[(size_t)t * 128 + 64] = c.lo[t];
    }
}

// The packed forms of the RNTN parameters (and the bias) in one launch, a wave per item: those of the tiles, of the rows (rows.steps > 0) and of the operand
// gradient (operand.steps > 0).
struct RntnPack {
    _Float16 *wp;
    float *scale;
    int steps;
};
__global__ __launch_bounds__(256) void k_pack_rntn(const float *__restrict__ s, int d, int Lp, int n_cg, RntnPack tile, RntnPack rows, RntnPack operand,
                                                   const float *__restrict__ b, float *__restrict__ bp)
{
    const int lane = threadIdx.x & 63;
    int item = blockIdx.x * 4 + (threadIdx.x >> 6);
    for (int u = blockIdx.x * blockDim.x + threadIdx.x; u < n_cg * HU; u += gridDim.x * blockDim.x) bp[u] = u < d ? b[u] : 0.f;
    const int n_tiles = n_cg * (32 * tile.steps + 1), n_rows = rows.steps > 0 ? d * (2 * rows.steps + 1) : 0, n_operand = 2 * d * operand.steps;
    if (item < n_tiles) return pack_rntn_tile(s, tile.wp, tile.scale, d, Lp, tile.steps, item, lane);
    item -= n_tiles;
    if (item < n_rows) return pack_rntn_rows(s, rows.wp, rows.scale, d, Lp, rows.steps, item, lane);
    item -= n_rows;
    if (item < n_operand) pack_rntn_operand(s, operand.wp, operand.scale, d, Lp, operand.steps, item, lane);
}

template <int N> __device__ inline float from_lane_above(float x) { return dpp<0x100 + N>(x); }      // row_shl: lane i of 16 reads lane i + N

template <int NS>
__device__ __forceinline__ void rows_run(RowsSmem<NS> &sm, const Fwd &f, const int4 *__restrict__ entries, int n_blocks, int member)
{
    using G = RowsGeom<NS>;
    constexpr int CPT = G::CPT, LD = RowsSmem<NS>::LD;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int H = f.H, seg = f.seg_chunks;                  // groups of eight values per segment of the K axis
    const unsigned row_b = (unsigned)H * 4u;
    const __amdgpu_buffer_rsrc_t rs_h = buf_of(f.h, (unsigned long long)f.n_nodes * row_b);
    // ---- the wave's weights ---------------------------------------------------------------
    const int hu = member * ROWS_UNITS + wave;
    halfx8 w[G::UNITS][2];
    float sc[G::SCALES], bias = 0.f;
    {
        const int g = hu < H ? hu : 0;                      // (a wave beyond the last unit computes the first one's sums and stores nothing)
        const halfx8 *wp = reinterpret_cast<const halfx8 *>(f.xi.wp) + (size_t)g * G::UNITS * 128 + lane;
#pragma unroll
        for (int u = 0; u < G::UNITS; ++u)
#pragma unroll
            for (int e = 0; e < 2; ++e) w[u][e] = wp[(u * 2 + e) * 64];
#pragma unroll
        for (int j = 0; j < G::SCALES; ++j) sc[j] = f.xi.scale[((size_t)g * G::SCALES + j) * HU + (lane & 15)];
        bias = f.inner.bp[g];
    }
    // ---- this thread's part of the gather: row my_row of the block, values 8 (t16 + 16 i) ... + 7 -----------------------------
    const int my_row = tid >> 4, t16 = tid & 15;
    uintx4_t rows[CPT][2];
    unsigned base0 = 0, base1 = 0;
    auto request = [&](auto past_caches) __attribute__((always_inline)) {
        constexpr int POLICY = decltype(past_caches)::value ? 16 : 0;
#pragma unroll
        for (int i = 0; i < CPT; ++i) {
            const int c = t16 + 16 * i;
            const bool right = c >= seg;
            const unsigned off = c < 2 * seg ? (right ? base1 + (unsigned)(c - seg) * 32u : base0 + (unsigned)c * 32u) : ~0u - 63u;
            rows[i][0] = __builtin_amdgcn_raw_buffer_load_b128(rs_h, (int)off, 0, POLICY);
            rows[i][1] = __builtin_amdgcn_raw_buffer_load_b128(rs_h, (int)off + 16, 0, POLICY);
        }
    };
    // values beyond the end of a row (the next row's, or nothing's) count as zero
    const bool ragged = H != seg * 8;
    auto cut = [&]() __attribute__((always_inline)) {
        if (!ragged) return;
#pragma unroll
        for (int i = 0; i < CPT; ++i) {
            const int c = t16 + 16 * i, in = (c >= seg ? c - seg : c) * 8;
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (in + e >= H) rows[i][e >> 2][e & 3] = 0u;
        }
    };
    auto shows_pattern = [&]() __attribute__((always_inline)) {
        unsigned m = 0u;
#pragma unroll
        for (int i = 0; i < CPT; ++i)
#pragma unroll
            for (int t = 0; t < 2; ++t) m = max(max(m, max(rows[i][t].x, rows[i][t].y)), max(rows[i][t].z, rows[i][t].w));
        return __ballot(m == FLOW_SENTINEL) != 0ull;
    };
    // A leaf's row was there before the kernel: a word of it that shows the pattern is a NaN of the embedding's own, and any other NaN
    // stands for it.  Asked only when a wait lasts (legitimate ones are mostly shorter).
    auto settle_leaves = [&](bool leaf0, bool leaf1) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < CPT; ++i) {
            const bool leaf = t16 + 16 * i >= seg ? leaf1 : leaf0;
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (leaf && rows[i][e >> 2][e & 3] == FLOW_SENTINEL) rows[i][e >> 2][e & 3] = 0x7FC00000u;
        }
    };
    auto prepare = [&](const int4 &q) __attribute__((always_inline)) {
        base0 = __umul24((unsigned)q.y, row_b);
        base1 = __umul24((unsigned)q.z, row_b);
    };
    int4 q = entries[my_row];
    int4 q_next = n_blocks > 1 ? entries[16 + my_row] : q;
    prepare(q);
    request(std::false_type{});
#pragma unroll 1
    for (int b = 0; b < n_blocks; ++b) {
        const int buf = b & 1;
        const bool last = b + 1 >= n_blocks;
        const bool late = last || __builtin_amdgcn_readfirstlane(q_next.w) < 0;     // the next block waits for this one
        const int4 q_ahead = entries[(size_t)min(b + 2, n_blocks - 1) * 16 + my_row];
        cut();
        if (shows_pattern()) {
            // requests repeated until no word shows the pattern; bounded by the spin budget and the abort flag
            int spins = 0;
            unsigned aborted = 0u;
            do {
                if (++spins > f.spin_limit || aborted != 0u) {
                    flow_give_up(f);
                    sm.gave_up = 1;
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
                request(std::true_type{});
                aborted = ld_dev(&f.ctl->abort.v);              // arrives with the rows
                cut();
                if (spins >= min(ROWS_SETTLE_SPINS, f.spin_limit)) settle_leaves(f.left[q.y] < 0, f.left[q.z] < 0);
            } while (shows_pattern());
        }
        // ---- split ---------------------------------------------------------------------
        {
            float m = 0.f;
#pragma unroll
            for (int i = 0; i < CPT; ++i)
#pragma unroll
                for (int e = 0; e < 8; ++e) m = fmaxf(m, fabsf(__uint_as_float(rows[i][e >> 2][e & 3])));
            m = fmaxf(m, dpp<DPP_XOR1>(m));
            m = fmaxf(m, dpp<DPP_XOR2>(m));
            m = fmaxf(m, dpp<DPP_HALF_MIRROR>(m));
            m = fmaxf(m, dpp<DPP_MIRROR>(m));
            const unsigned eb = max(__float_as_uint(m) >> 23, 15u);
            const float scale = __uint_as_float((268u - eb) << 23);
            if (t16 == 0) {
                sm.back[buf][my_row] = __uint_as_float((eb - 14u) << 23);
                sm.node[buf][my_row] = q.x;
                sm.tree[buf][my_row] = q.x >= 0 ? (q.w & 0x7FFFFFFF) - 1 : -1;
            }
#pragma unroll
            for (int i = 0; i < CPT; ++i) {
                const int c = t16 + 16 * i, s = c >> 2, quarter = c & 3;
                if (NS % 4 != 0 && c >= 4 * NS) continue;
                halfx8 hi, lo;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float v = __uint_as_float(rows[i][e >> 2][e & 3]) * scale;
                    hi[e] = (_Float16)v;
                    lo[e] = (_Float16)(v - (float)hi[e]);
                }
                halfx8 *dst = &sm.split[buf][s * 128 + rows_slot(s, quarter, my_row)];
                dst[0] = hi;
                dst[64] = lo;
                *reinterpret_cast<uintx4_t *>(&sm.a[buf][my_row * LD + c * 8]) = rows[i][0];
                *reinterpret_cast<uintx4_t *>(&sm.a[buf][my_row * LD + c * 8 + 4]) = rows[i][1];
            }
        }
        prepare(q_next);
        if (!late) request(std::false_type{});
        __syncthreads();
        if (sm.gave_up != 0) return;
        // ---- products -------------------------------------------------------------------
        const halfx8 *op = sm.split[buf];
        auto operand = [&](int s, int e) __attribute__((always_inline)) { return op[s * 128 + e * 64 + rows_slot(s, lane >> 4, lane & 15)]; };
        const floatx4 back = *reinterpret_cast<const floatx4 *>(&sm.back[buf][4 * (lane >> 4)]);
        {
            halfx8 a[NS][2];
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
                for (int e = 0; e < 2; ++e) a[s][e] = operand(s, e);
            const float *m = &sm.a[buf][4 * (lane >> 4) * LD + (lane & 15)];
            floatx4 out = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < 2 * NS; ++j) {
                floatx4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s <= j / 2; ++s) {
                    const int u = rntn_first(j) + s;
                    t = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[s][0], w[u][0], t, 0, 0, 0);
                    t = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[s][0], w[u][1], t, 0, 0, 0);
                    t = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[s][1], w[u][0], t, 0, 0, 0);
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) out[v] = __builtin_fmaf(m[v * LD + 16 * j] * sc[j], t[v], out[v]);
            }
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                floatx4 x = {0.f, 0.f, 0.f, 0.f};
                x = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[s][0], w[G::QUAD][0], x, 0, 0, 0);
                x = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[s][0], w[G::QUAD][1], x, 0, 0, 0);
                x = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[s][1], w[G::QUAD][0], x, 0, 0, 0);
                if ((lane & 15) == s) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) out[v] = __builtin_fmaf(sc[2 * NS], x[v], out[v]);
                }
            }
            // lanes p, p + 4, p + 8, p + 12 of 16 are part p, the parts in order: lanes 0 .. 3 of every 16 then all hold the sums of
            // the four rows, and lane v takes row v
            float sum = 0.f;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float x = out[v];
                const float part = ((x + from_lane_above<4>(x)) + from_lane_above<8>(x)) + from_lane_above<12>(x);
                const float all = ((dpp<0x00>(part) + dpp<0x55>(part)) + dpp<0xAA>(part)) + dpp<0xFF>(part);    // quad_perm: one lane to all four
                if ((lane & 15) == v) sum = all * back[v];
            }
            const int row = 4 * (lane >> 4) + (lane & 3), node = sm.node[buf][row];
            if ((lane & 15) < 4 && node >= 0 && hu < H) {
                if (__builtin_expect(!__builtin_isfinite(sum), 0)) sum = rntn_sum_plain(f, f.inner, &sm.a[buf][row * LD], hu);
                const float h = tanh_f(sum + bias);
                buf_st_f<true>(rs_h, __umul24((unsigned)node, row_b) + (unsigned)hu * 4u, h);
                const int t = sm.tree[buf][row];
                if (t >= 0 && f.h_root) f.h_root[(size_t)t * H + hu] = h;
            }
        }
        if (late && !last) request(std::true_type{});     // (past the caches: what they hold of these rows is too old)
        q = q_next;
        q_next = q_ahead;
    }
}

template <int NS>
__global__ __launch_bounds__(WG_THREADS, (RowsGeom<NS>::SETS_PER_CU)) void k_flow_rows(Fwd f)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    using G = RowsGeom<NS>;
    RowsSmem<NS> &sm = *reinterpret_cast<RowsSmem<NS> *>(smem_raw);
    const int tid = threadIdx.x;
    const bool leave = tid == 0 && (batch_rejected(f) || internal_kernel_skipped(f));      // (a workgroup that gives up latches that)
    int member, slot;
    split_place(f, &slot, &member);
    if (tid == 0) sm.gave_up = 0;
    const int4 head = f.sched_head[slot];         // (of an earlier batch where this one is rejected: not used then)
    if (decided_to_leave(&sm.leave, leave)) return;
    if (f.flow_roots && f.h_root) {               // trees of one node: the leaf is the root
        for (int i = tid; i < (head.w - head.z) * ROWS_UNITS; i += WG_THREADS) {
            const int t = head.z + i / ROWS_UNITS, hu = member * ROWS_UNITS + i % ROWS_UNITS, n = f.tree_off[t];
            if (hu < f.H && f.tree_off[t + 1] - n == 1) f.h_root[(size_t)t * f.H + hu] = f.h[(size_t)n * f.H + hu];
        }
    }
    if (head.y > 0) rows_run<NS>(sm, f, f.sched + (size_t)head.x * 16, head.y, member);
}

}  // namespace tl
