// Backward pass of TreeLSTM (from kept gate activations) and TreeRNN, H <= 512: the mirror image of the data-flow forward.
//
// A workgroup owns 16 hidden units u for the whole call: the 32 output columns of the operand gradient [dh_l | dh_r] = dG U^T that
// belong to them, with their slice of U^T in registers.  What it computes for a block of 16 nodes - dh of both children at its
// units - is all that the children's gate gradients at those units need beside values of the forward and the dc chain, which is
// its own.  So it finishes the children at once: their rows of gate gradients (what the next blocks gather) are written from
// registers, dh and dc of a node never exist in memory, and nothing is left of the phases and grid barriers per height that a
// gate-gradient pass and a contraction pass need.  Blocks, their order and what waits for what are those of the forward's
// schedule (structure.hpp, flow_schedule) read from the last block to the first: a block is `late` after the one
// whose entries say that that one depended on it.  A row that is not there yet shows the pattern of the forward's rows.
//
// Contraction: operands as two fp16 terms, as in cell_split.hpp (three 16-bit products, fp32 accumulation).  A row of dG (NG H
// values, any magnitude) is written by n_cg workgroups, each of which knows its own 16 units only; so every piece (a
// node's NG x 16 values of one workgroup) has a power of two of its own, which brings its largest magnitude into [2^14, 2^15).  The
// reader of a quarter of a row multiplies the pieces by powers of two that bring them to the largest of its quarter, down to 2^-14 (which keeps a piece to 2^-25 of its
// own largest value), and its partial sums by that one's; pieces further below are summed apart (far_bands).
// Sums that are not finite (an infinity has no two terms, and a scaled sum may overflow) are taken again in fp32.
//
// Layout of the copy that the blocks read (`gx`): a node's row is read once, in a block and a row of it that the schedule knows beforehand, so
// it is written where that block's operands lie: block by block in list order, a block of m nodes as m n_pairs NG 128 bytes, unit
// (pair, gate, term) of 64 m bytes = [quarter of 8 hidden units][row][16 bytes], the operand of a matrix instruction in lane order.  A block's loads
// are whole lines, 1 KB an instruction.  (Rows by node cost the address unit a line per lane, 64 clocks for 1 KB instead of 16: 40 loads of a wave
// are 4.4 us of a CU at H = 512; read by lines and turned through LDS they keep LDS busy for 1.6 us.)  Units 32 pair ... 32 pair + 31 belong to two
// workgroups; `gs` holds the pieces' exponents, block by block [n_cg][row].  K axis: pairs w P ... w P + P - 1 for wave w, a k-step of 32 per pair and
// gate; what lies beyond the last pair (or, for an odd number of workgroups, in its second half) is read beyond the end of the table, as zeros.
//
// Measured (profiler, all heights; before: gate gradients and operand gradients with fp32 instructions, two grid barriers per height): 256 parse trees at
// H = 512 658 + 23 (leaves' gate gradients) -> 305 us, 25 at H = 150 99 + 5 -> 47 us.  A block at H = 512 is 11 900 clocks of a wave: 4 800 products (20
// k-steps of six instructions of 16 clocks, eight multiplications by the pieces' powers of two, two loads), 3 500 the children's gate gradients,
// 2 400 the start of the next block and its rows, 650 the exchange.  Bound by one wave per SIMD doing these one after the other: the weights leave
// registers for no second one.
#pragma once

#include "cell_split.hpp"
#include "cell_rows.hpp"

namespace tl {

struct BackFlow {
    const float *g_h;           // upstream gradient [N x H]
    float *dc;                  // [N x H][2]: what of an internal node's dc arrives at its left and its right child (TreeLSTM)
    unsigned *gx, *gs;
    float *dg;                  // gate gradients in fp32, row n = node n, NG H values (leaves: the first 3 H), for the weight gradients
    const void *wp;             // U^T packed, see pack_rows_block
    const float *scale;         // [n_cg][2][16] what a column's sums are multiplied by
    const float *u;             // the matrix as given, [2 H x NG H]
    int32_t *int_list;          // internal nodes, in no particular order
    int n_pairs;
    SchedPlaces at;
};

template <int NG, int P> struct BackGeom {
    static constexpr int S = NG * P;                    // k-steps of a wave
    // Weights of the largest size: 13 of 20 k-steps in registers, the others in LDS (112 KB), read a step ahead.  The registers that frees hold
    // the rows of a whole block in flight: a load waits for the stores in front of it, so no row may be asked for behind a block's stores
    // that the block before could have asked for.
    static constexpr int IN_LDS = S > 16 ? 7 : 0;
    static_assert(S <= 16 || S == 20, "places of the weights");
    static constexpr bool in_lds(int s) { return S > 16 && s < S && (s % 3 == 2 || s == 19); }
    static constexpr int lds(int s) { return s == 19 ? 6 : s / 3; }         // place there
    static constexpr int reg(int s) { return S > 16 ? s - s / 3 : s; }      // ... in registers
    // (a k-step's weights are read while the step before is computed, into registers that this one must not need)
    static constexpr bool apart() { for (int s = 0; s < S; ++s) if (in_lds(s) && in_lds(s + 1)) return false; return true; }
};
static_assert(BackGeom<5, 4>::apart(), "weights in LDS");
template <int L> struct BackSmemT {
    unsigned char stage[4][16 * 320 + 128];             // see BackUnit::finish
    int4 ring[4][32];                                   // entries of four blocks: {node, left, right, flags} of 16 rows, their children's places
    float red[2][4 * 2 * 64 * 4];                       // quarter sums, alternating per block: [wave][side][lane][v]
    float row_scale[4][16];
    float scale[2 * HU];
    int gave_up, leave;
    int cmd[8];                                         // (grid_barrier's)
    halfx8 w[L > 0 ? 4 * L * 4 * 64 : 1];               // [wave][k-step][side][term][lane]
};
template <int NG, int P> using BackSmem = BackSmemT<BackGeom<NG, P>::IN_LDS>;

template <int NG, int P> struct BackWeights {
    halfx8 t[BackGeom<NG, P>::S - BackGeom<NG, P>::IN_LDS][2][2];     // [k-step][side][term]
};
template <int NG, int P>
__device__ __forceinline__ void back_load(BackWeights<NG, P> &w, BackSmem<NG, P> &sm, const BackFlow &b, int cg, int wave, int lane)
{
    using G = BackGeom<NG, P>;
    constexpr int S = G::S;
    const halfx8 *wp = reinterpret_cast<const halfx8 *>(b.wp) + ((size_t)cg * 4 * S + (size_t)wave * S) * 4 * 64 + lane;
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
        for (int d = 0; d < 2; ++d)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const halfx8 v = wp[(size_t)((s * 2 + d) * 2 + t) * 64];
                if (G::in_lds(s)) sm.w[(((wave * G::IN_LDS + G::lds(s)) * 2 + d) * 2 + t) * 64 + lane] = v;
                else w.t[G::reg(s)][d][t] = v;
            }
    if (wave == 0 && lane < 2 * HU) sm.scale[lane] = b.scale[cg * 2 * HU + lane];
    // (in the accumulation registers: see split_load)
    if constexpr (S > 8) {
#pragma unroll
        for (int s = 0; s < S - G::IN_LDS; ++s)
#pragma unroll
            for (int d = 0; d < 2; ++d)
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    floatx4 v = __builtin_bit_cast(floatx4, w.t[s][d][t]);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        float e = v[i];
                        asm volatile("" : "+a"(e));     // no instruction: a register-class constraint only
                        v[i] = e;
                    }
                    w.t[s][d][t] = __builtin_bit_cast(halfx8, v);
                }
    }
}

typedef unsigned int uintx2_t __attribute__((ext_vector_type(2)));

// One hidden unit of nodes: from dh and what arrives of dc to their gate gradients.  The 16 lanes of a row hold the 16 units of one
// node's piece.
template <int NG> struct BackUnit {
    static constexpr bool LSTM = NG == 5;
    static constexpr unsigned ALL_ZERO = 15u;           // in the place of an exponent
    static constexpr int PIECE = NG * 64, CHUNKS = 8 * NG * 4, STORES = (CHUNKS + 63) / 64;      // bytes of a piece; of 8 pieces, in 16 bytes and in wave-wide stores
    const Fwd &f;
    const BackFlow &b;
    int cg, hu, lane;
    bool hu_ok, whole;
    unsigned char *stage;       // this wave's own LDS
    unsigned hu_b, row_b, gx_row_b;
    __amdgpu_buffer_rsrc_t rs_gh, rs_k0, rs_k1, rs_dc, rs_gx, rs_gs, rs_dg;     // TreeRNN: rs_k0 is h, rs_dc d_x
    __device__ inline BackUnit(const Fwd &f_, const BackFlow &b_, unsigned char *stage_, int cg_, int lane_) : f(f_), b(b_), cg(cg_), lane(lane_), stage(stage_)
    {
        const int H = f.H;
        hu = cg * HU + (lane & 15);
        hu_ok = hu < H;
        whole = cg * HU + HU <= H;
        hu_b = (unsigned)(hu_ok ? hu : 0) * 4u;
        row_b = (unsigned)H * 4u;
        gx_row_b = (unsigned)(b.n_pairs * NG) * 128u;
        const unsigned long long n = (unsigned long long)f.n_nodes;
        rs_gh = buf_of(b.g_h, n * row_b);
        rs_k0 = LSTM ? buf_of(f.keep0, n * row_b * 4) : buf_of(f.h, n * row_b);
        rs_k1 = buf_of(f.keep1, n * row_b * 4);
        rs_dc = LSTM ? buf_of(b.dc, n * row_b * 2) : buf_of(f.d_x, n * row_b);
        rs_gx = buf_of(b.gx, (unsigned long long)f.n_int * gx_row_b);
        rs_gs = buf_of(b.gs, (unsigned long long)f.n_int * (unsigned)f.n_cg * 4u);
        rs_dg = buf_of(b.dg, n * row_b * NG);
    }
    struct In {
        float gh;
        floatx4 k0, k1;         // (TreeRNN: k0[0] is h)
    };
    __device__ inline unsigned at(int node) const { return (unsigned)node * row_b + hu_b; }
    __device__ inline In load(int node) const
    {
        In in{};
        in.gh = buf_ld_f<false>(rs_gh, at(node));
        if constexpr (LSTM) {
            in.k0 = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(rs_k0, (int)(at(node) * 4u), 0, 0));
            in.k1 = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(rs_k1, (int)(at(node) * 4u), 0, 0));      // (a leaf's is not used)
        } else {
            in.k0[0] = buf_ld_f<false>(rs_k0, at(node));
        }
        return in;
    }
    // Two nodes per row of 16 lanes.  here: there is a node; place: its SchedPlaces::of.  Called by whole waves.  The pieces of the eight nodes
    // meet in LDS and leave it in wave-wide stores of 16 bytes a lane.  Stored without branches, so that the compiler knows how many stores lie behind
    // the rows in flight and waits for none of them (what is not to be stored goes beyond the end of its table and is dropped); few of them, so that a
    // wave has no more accesses in flight than it can count (63).
    __device__ __forceinline__ void finish(const bool (&here)[2], const int (&node)[2], const int2 (&place)[2], const In (&in)[2], const float (&dh)[2], const float (&dc)[2]) const
    {
        unsigned eb[2];
        float out[2][NG], dcx[2][2] = {};
        const int row = lane >> 4, u = lane & 15;
        int *const ids = reinterpret_cast<int *>(stage + 16 * PIECE);           // [8 pieces]{place of an internal node, or -1; node or -1; -}
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            const bool leaf = place[d].x < 0, inner = here[d] && !leaf;
            if constexpr (LSTM) {
                const floatx4 k0 = in[d].k0, k1 = in[d].k1;
                const float dct = __builtin_fmaf(dh[d], k0[0], dc[d]), d_i = dct * k0[1], d_o = dh[d] * k0[2], d_u = dct * k0[3];
                out[d][0] = d_i;
                out[d][1] = leaf ? d_o : dct * k1[0];
                out[d][2] = leaf ? d_u : dct * k1[1];
                out[d][3] = d_o;
                out[d][4] = d_u;
                dcx[d][0] = dct * k1[2];
                dcx[d][1] = dct * k1[3];
            } else {
                out[d][0] = dh[d] * __builtin_fmaf(-in[d].k0[0], in[d].k0[0], 1.f);
            }
            unsigned m = 0u;                            // largest magnitude, as bits (those of a NaN are above all others)
#pragma unroll
            for (int q = 0; q < NG; ++q) {
                if (!whole && !hu_ok) out[d][q] = 0.f;
                m = max(m, __float_as_uint(out[d][q]) & 0x7FFFFFFFu);
            }
            m = max(m, __float_as_uint(dpp<DPP_XOR1>(__uint_as_float(m))));
            m = max(m, __float_as_uint(dpp<DPP_XOR2>(__uint_as_float(m))));
            m = max(m, __float_as_uint(dpp<DPP_HALF_MIRROR>(__uint_as_float(m))));
            m = max(m, __float_as_uint(dpp<DPP_MIRROR>(__uint_as_float(m))));
            eb[d] = max(m >> 23, ALL_ZERO + min(m, 1u));
            const float scale = __uint_as_float((268u - eb[d]) << 23);
            if (__builtin_expect(__ballot(eb[d] == 255u) != 0ull, 0)) {         // no NaN may look like "not written"
#pragma unroll
                for (int q = 0; q < NG; ++q) out[d][q] = __builtin_isnan(out[d][q]) ? __uint_as_float(0x7FC00000u) : out[d][q];
#pragma unroll
                for (int i = 0; i < 2; ++i) dcx[d][i] = __builtin_isnan(dcx[d][i]) ? __uint_as_float(0x7FC00000u) : dcx[d][i];
            }
            unsigned char *const p = stage + (d * 4 + row) * PIECE;
#pragma unroll
            for (int q = 0; q < NG; ++q) {
                // (the product is exact: no rounding in between)
                const _Float16 hi = (_Float16)(out[d][q] * scale), lo = (_Float16)__builtin_fmaf(out[d][q], scale, -(float)hi);
                *reinterpret_cast<_Float16 *>(p + q * 64 + u * 2) = hi;
                *reinterpret_cast<_Float16 *>(p + q * 64 + 32 + u * 2) = lo;
                *reinterpret_cast<float *>(p + 8 * PIECE + q * 64 + u * 4) = out[d][q];
            }
            if (u == 0) *reinterpret_cast<uintx4_t *>(ids + (d * 4 + row) * 4) = uintx4_t{(unsigned)(inner ? place[d].x : -1), (unsigned)place[d].y, (unsigned)(here[d] ? node[d] : -1), 0u};
        }
        {
            const bool right = (u & 1) != 0, inner = right ? here[1] && place[1].x >= 0 : here[0] && place[0].x >= 0;
            const int start = right ? place[1].x : place[0].x, at_row = right ? place[1].y : place[0].y;
            __builtin_amdgcn_raw_buffer_store_b32(right ? eb[1] : eb[0], rs_gs, (int)(inner && u < 2 ? ((unsigned)start * (unsigned)f.n_cg + (unsigned)(cg * (at_row & 0xFF) + (at_row >> 8))) * 4u : ~0u), 0, 16);
        }
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            const bool leaf = place[d].x < 0, inner = here[d] && !leaf;
            if constexpr (LSTM) {
                const uintx2_t v = {__float_as_uint(dcx[d][0]), __float_as_uint(dcx[d][1])};
                __builtin_amdgcn_raw_buffer_store_b64(v, rs_dc, (int)(inner && hu_ok ? at(node[d]) * 2u : ~0u), 0, 16);
            } else {
                buf_st_f<false>(rs_dc, here[d] && leaf && hu_ok ? at(node[d]) : ~0u, dh[d]);      // d_x: the embedding row is the state itself
            }
        }
        int first = lane;
        asm volatile("" : "+v"(first));                 // no instruction: what follows from the lane number is worked out here, not kept through the products
#pragma unroll
        for (int kind = 0; kind < 2; ++kind) {          // the split copy first: other workgroups wait for it
            if (kind == 1 && !whole) {                  // (the last column group of a number of units that is no multiple of 16)
#pragma unroll
                for (int d = 0; d < 2; ++d)
#pragma unroll
                    for (int q = 0; q < NG; ++q)
                        buf_st_f<false>(rs_dg, (LSTM && q < 3 ? here[d] : here[d] && place[d].x >= 0) && hu_ok ? (unsigned)node[d] * (NG * row_b) + (unsigned)q * row_b + hu_b : ~0u, out[d][q]);
                break;
            }
#pragma unroll
            for (int j = 0; j < STORES; ++j) {
                const int c = j * 64 + first, p = c / (NG * 4), k = c % (NG * 4), q = k >> 2, part = k & 3;
                const bool there = CHUNKS % 64 == 0 || c < CHUNKS;
                const uintx4_t id = *reinterpret_cast<const uintx4_t *>(ids + (there ? p : 0) * 4);
                const uintx4_t v = *reinterpret_cast<const uintx4_t *>(stage + (there ? p : 0) * PIECE + kind * 8 * PIECE + k * 16);
                if (kind == 0) {
                    const unsigned unit = (unsigned)((((cg >> 1) * NG + q) * 2 + (part >> 1)) * 4 + (cg & 1) * 2 + (part & 1));      // of 16 m bytes
                    const unsigned o = id.x * gx_row_b + (unit * (id.y & 0xFFu) + (id.y >> 8)) * 16u;
                    __builtin_amdgcn_raw_buffer_store_b128(v, rs_gx, (int)(there && (int)id.x >= 0 ? o : ~0u), 0, 16);
                } else {
                    const unsigned o = id.z * (NG * row_b) + (unsigned)q * row_b + (unsigned)(cg * HU + part * 4) * 4u;
                    const bool gate = (int)id.z >= 0 && ((LSTM && q < 3) || (int)id.x >= 0);
                    __builtin_amdgcn_raw_buffer_store_b128(v, rs_dg, (int)(there && gate ? o : ~0u), 0, 0);
                }
            }
        }
    }
    // A sum of the operand gradient in fp32 from the parameters as given (rare, and slow): row `row` of the block of m nodes at position start,
    // whose copy is complete.  A sum that is a NaN stays one: a step that has diverged, all of whose rows hold nothing else, does not get here value by value.
    __device__ __forceinline__ float plain(int start, int m, int row, int side) const
    {
        const int H = f.H;
        const float *w = b.u + (size_t)(side * H + hu) * (NG * H);
        const unsigned short *gx = reinterpret_cast<const unsigned short *>(b.gx) + (size_t)start * (gx_row_b / 2);
        const unsigned *gs = b.gs + (size_t)start * f.n_cg;
        float sum = 0.f;
#pragma unroll 1
        for (int q = 0; q < NG; ++q)
#pragma unroll 1
            for (int u = 0; u < H && !__builtin_isnan(sum); ++u) {
                const unsigned short *p = gx + ((((u >> 5) * NG + q) * 8 + (u >> 3 & 3)) * m + row) * 8 + (u & 7);
                const float hi = (float)__builtin_bit_cast(_Float16, ld_dev(p)), lo = (float)__builtin_bit_cast(_Float16, ld_dev(p + 4 * m * 8));
                const int e = (int)ld_dev(gs + (u >> 4) * m + row) - 141;
                sum = __builtin_fmaf(ldexpf(__builtin_isfinite(hi) ? hi + lo : hi, e), w[(size_t)q * H + u], sum);
            }
        return sum;
    }
};

// The roots of trees [t_lo, t_hi): wave number `wave` of `waves` takes four at a time.  Nothing arrives but the upstream gradient.
template <int NG>
__device__ __forceinline__ void back_roots(const Fwd &f, const BackFlow &b, const BackUnit<NG> &unit, int t_lo, int t_hi, int wave, int waves)
{
    for (int t0 = t_lo + 4 * wave; t0 < t_hi; t0 += 4 * waves) {
        const int t = t0 + (unit.lane >> 4), root = f.root_ws[min(t, t_hi - 1)];
        const bool here[2] = {t < t_hi && root >= 0, false};
        const int node[2] = {max(root, 0), 0};
        const int2 place[2] = {b.at.of[max(root, 0)], int2{-1, 0}};
        const typename BackUnit<NG>::In in[2] = {unit.load(node[0]), typename BackUnit<NG>::In{}};
        const float dh[2] = {in[0].gh, 0.f}, dc[2] = {0.f, 0.f};
        unit.finish(here, node, place, in, dh, dc);
    }
}

// Blocks 0 ... n_blocks - 1 of up to 16 nodes each, `fetch(block, i)` = {node or -1, left, right, flags} of row i < 16 (row 0 is always a node) or the places of the
// children of row i - 16, `start(block, m)` the position of a block of m nodes, asked for in order.  FLOW: the rows of a block may not be written yet, and block b + 1 waits for block b where the flags of b say so.
// Else all rows are there.
template <int NG, int P, bool FLOW, typename Fetch, typename Start>
__device__ __forceinline__ void back_run(BackSmem<NG, P> &sm, const Fwd &f, const BackFlow &b, const BackUnit<NG> &unit, int n_blocks, const BackWeights<NG, P> &w, Fetch fetch, Start start_of)
{
    using G = BackGeom<NG, P>;
    constexpr int S = G::S;
    constexpr bool LSTM = NG == 5;
    constexpr int COH = FLOW ? 0 : 16;                  // (of the first requests)
    constexpr int FAR = 14;                             // 2^-14 is the smallest number that fp16 holds with all its bits
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr unsigned NOWHERE = ~0u - 0xFFFFu;         // beyond the end of every table
    uintx4_t rows[S][2];
    unsigned ex[P];                                     // exponents of the pieces this lane holds, one per pair
    int start = 0, m = 0;                               // the block that is asked for
    unsigned lane_off = 0;
    // Every wave fetches the entries of a block three blocks ahead and writes them to LDS a block later (all the same: a wave reads what it
    // has written itself, and is never more than a block's barrier ahead of another one).
    auto keep = [&](int blk, const int4 &v) __attribute__((always_inline)) { sm.ring[blk & 3][lane & 31] = v; };
    auto fetch_block = [&](int blk) __attribute__((always_inline)) { return fetch(min(blk, n_blocks - 1), lane & 31); };
    auto prepare = [&](int blk) __attribute__((always_inline)) {
        m = __popcll(__ballot(sm.ring[blk & 3][lane & 15].x >= 0) & 0xFFFFull);
        start = start_of(blk, m);
        lane_off = (unsigned)((lane >> 4) * m + min(lane & 15, m - 1)) * 16u;
    };
    auto request = [&](bool wanted, int s, auto policy) __attribute__((always_inline)) {
        constexpr int POLICY = decltype(policy)::value;
        const int pair = wave * P + s / NG, line = min(pair, b.n_pairs - 1) * NG + s % NG;
        // (beyond the last pair, and in the second half of the last one of an odd number of column groups: zeros)
        const bool none = pair >= b.n_pairs, half = 2 * pair + 1 >= f.n_cg;
        const unsigned o = !wanted || none || (half && lane >= 32) ? NOWHERE : lane_off;
        const unsigned base = (unsigned)start * unit.gx_row_b + (unsigned)(line * 128 * m);       // (beyond 2^31 in tables of less than 4 GiB)
        rows[s][0] = __builtin_amdgcn_raw_buffer_load_b128(unit.rs_gx, (int)o, (int)base, POLICY);
        rows[s][1] = __builtin_amdgcn_raw_buffer_load_b128(unit.rs_gx, (int)o, (int)(base + 64u * (unsigned)m), POLICY);
    };
    auto request_ex = [&](bool wanted, auto policy) __attribute__((always_inline)) {
        constexpr int POLICY = decltype(policy)::value;
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const int c = min(2 * min(wave * P + p, b.n_pairs - 1) + (lane >> 5), f.n_cg - 1);
            ex[p] = __builtin_amdgcn_raw_buffer_load_b32(unit.rs_gs, wanted ? (c * m + min(lane & 15, m - 1)) * 4 : (int)NOWHERE, start * f.n_cg * 4, POLICY);
        }
    };
    auto shows_pattern = [&]() __attribute__((always_inline)) {
        unsigned v = 0u;
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int t = 0; t < 2; ++t) v = max(max(v, max(rows[s][t].x, rows[s][t].y)), max(rows[s][t].z, rows[s][t].w));
#pragma unroll
        for (int p = 0; p < P; ++p) v = max(v, ex[p]);
        return __ballot(v == FLOW_SENTINEL) != 0ull;
    };
    auto request_first = [&](auto policy) __attribute__((always_inline)) {
        request_ex(true, policy);
#pragma unroll
        for (int s = 0; s < S; ++s) request(true, s, policy);
    };
    typedef std::integral_constant<int, COH> first_policy;
    typedef std::integral_constant<int, 16> past_caches;
    // Pieces further below their quarter's largest than FAR bits: brought there they would lose bits of their own, or all of them.  Rare: their rows and the weights are asked
    // for again and summed band by band, in a loop that is not unrolled (with the weights where the products have them it needs registers that the block's own code then lacks: H = 48,
    // 166 trees 48.2 -> 51.2 us).  (Block of m nodes at position start; top: the largest of this lane's row's quarter.)
    auto far_bands = [&](int start, int m, unsigned top, floatx4 *own) __attribute__((always_inline)) {
        const unsigned off = (unsigned)((lane >> 4) * m + min(lane & 15, m - 1)) * 16u;
        unsigned limit = top < 255u ? top : 0u;         // a band begins below limit - FAR (none in a row with an infinity, a NaN, or whose wait was given up)
        for (;;) {
            unsigned next = 0u;
            auto piece = [&](int p) __attribute__((always_inline)) {
                const int c = min(2 * min(wave * P + p, b.n_pairs - 1) + (lane >> 5), f.n_cg - 1);
                return (unsigned)__builtin_amdgcn_raw_buffer_load_b32(unit.rs_gs, (c * m + min(lane & 15, m - 1)) * 4, start * f.n_cg * 4, 16);
            };
#pragma unroll 1
            for (int p = 0; p < P; ++p) {
                const unsigned e = piece(p);
                if (e != BackUnit<NG>::ALL_ZERO && e + FAR < limit) next = max(next, e);
            }
            next = max(next, (unsigned)__shfl_xor((int)next, 32));
            if (__ballot(next != 0u) == 0ull) break;
            floatx4 acc[2] = {};
#pragma unroll 1
            for (int s = 0; s < S; ++s) {
                const int pair = wave * P + s / NG, line = min(pair, b.n_pairs - 1) * NG + s % NG;
                const unsigned e = piece(s / NG), base = (unsigned)start * unit.gx_row_b + (unsigned)(line * 128 * m);
                const bool none = pair >= b.n_pairs || (2 * pair + 1 >= f.n_cg && lane >= 32), band = e + FAR < limit && next - e <= (unsigned)FAR;
                const _Float16 by = __builtin_bit_cast(_Float16, (unsigned short)(band ? (FAR + 1 + e - next) << 10 : 0u));
                const halfx8 hi = __builtin_bit_cast(halfx8, __builtin_amdgcn_raw_buffer_load_b128(unit.rs_gx, (int)(none ? NOWHERE : off), (int)base, 16)) * by,
                             lo = __builtin_bit_cast(halfx8, __builtin_amdgcn_raw_buffer_load_b128(unit.rs_gx, (int)(none ? NOWHERE : off), (int)(base + 64u * (unsigned)m), 16)) * by;
                const halfx8 *wt = reinterpret_cast<const halfx8 *>(b.wp) + ((size_t)unit.cg * 4 * S + (size_t)wave * S + s) * 4 * 64 + lane;
#pragma unroll
                for (int d = 0; d < 2; ++d) {
                    acc[d] = __builtin_amdgcn_mfma_f32_16x16x32_f16(hi, wt[2 * d * 64], acc[d], 0, 0, 0);
                    acc[d] = __builtin_amdgcn_mfma_f32_16x16x32_f16(hi, wt[(2 * d + 1) * 64], acc[d], 0, 0, 0);
                    acc[d] = __builtin_amdgcn_mfma_f32_16x16x32_f16(lo, wt[2 * d * 64], acc[d], 0, 0, 0);
                    if constexpr (S > 16) __builtin_amdgcn_sched_barrier(0);        // (no registers for more than one side's weights)
                }
            }
            if (lane < 16) sm.row_scale[wave][lane] = __uint_as_float((max(next, 15u) - 14u) << 23);
            const floatx4 r4 = *reinterpret_cast<const floatx4 *>(&sm.row_scale[wave][4 * (lane >> 4)]);
#pragma unroll
            for (int d = 0; d < 2; ++d) own[64 * d] += acc[d] * r4;
            limit = next;
        }
    };
    const int fin_row = 4 * wave + (lane >> 4), last_b = n_blocks - 1;
    typename BackUnit<NG>::In in[2] = {};
    auto load_children = [&](int blk, typename BackUnit<NG>::In (&in)[2]) __attribute__((always_inline)) {
        const int4 e = sm.ring[blk & 3][fin_row];
        in[0] = unit.load(e.y);
        in[1] = unit.load(e.z);
    };
    {
        const int4 v0 = fetch_block(0), v1 = fetch_block(1);
        keep(0, v0);
        keep(1, v1);
    }
    int4 ahead = fetch_block(2);
    prepare(0);
    load_children(0, in);
    request_first(first_policy{});
#pragma unroll 1
    for (int blk = 0; blk < n_blocks; ++blk) {
        const bool last = blk == last_b;
        const bool late = last || (FLOW && __builtin_amdgcn_readfirstlane(sm.ring[blk & 3][0].w) < 0);      // the next block waits for this one
        keep(blk + 2, ahead);
        ahead = fetch_block(blk + 3);
        // what the children of the next block's nodes need (it is asked for a block ahead)
        typename BackUnit<NG>::In in_next[2];
        load_children(min(blk + 1, last_b), in_next);
        const int4 e = sm.ring[blk & 3][fin_row];
        const int parent = e.x < 0 ? __builtin_amdgcn_readfirstlane(sm.ring[blk & 3][0].x) : e.x;
        int spins = 0;
        auto give_up = [&](unsigned aborted) __attribute__((always_inline)) {           // waits are bounded by the spin budget and the abort flag
            if (++spins <= f.spin_limit && aborted == 0u) return false;
            flow_give_up(f);
            sm.gave_up = 1;
            return true;
        };
        if (FLOW && shows_pattern()) {
            unsigned aborted = 0u;
            do {
                if (give_up(aborted)) break;
                __builtin_amdgcn_s_sleep(1);
                request_first(past_caches{});
                aborted = ld_dev(&f.ctl->abort.v);      // arrives with the rows
            } while (shows_pattern());
        }
        uintx2_t dc2{};                                 // (this workgroup's own stores, in flight at most)
        if constexpr (LSTM) dc2 = __builtin_amdgcn_raw_buffer_load_b64(unit.rs_dc, (int)(unit.at(parent) * 2u), 0, COH);
        // this lane's pieces are brought to the largest of its row's quarter
        unsigned top = ex[0];
#pragma unroll
        for (int p = 1; p < P; ++p) top = max(top, ex[p]);
        top = max(top, (unsigned)__shfl_xor((int)top, 32));
        _Float16 factor[P];                             // (beyond FAR bits: zero)
        unsigned ex_now[P];
#pragma unroll
        for (int p = 0; p < P; ++p) {
            factor[p] = __builtin_bit_cast(_Float16, (unsigned short)((unsigned)max(FAR + 1 + (int)ex[p] - (int)top, 0) << 10));
            ex_now[p] = ex[p];
        }
        const float back = __uint_as_float((top - 14u) << 23);
        const int here_start = start, here_m = m;
        if (!last) prepare(blk + 1);
        // (requests that are not to be made yet go beyond the end of the table: they return at once and read nothing)
        request_ex(!late, first_policy{});
        __builtin_amdgcn_sched_barrier(0);
        // The matrix instruction drops what does not fit downwards, and a column sum over all nodes adds that up (d_b of 256 parse trees at H = 512: off by
        // 3.2e-7 of its norm): every other k-step is taken with its rows negated, into a sum of its own that is subtracted.
        floatx4 acc[2][2] = {};
        bool far = false;
        halfx8 wl[2][2] = {};                           // the next k-step's weights, where they are in LDS
#pragma unroll
        for (int s = 0; s < S; ++s) {
            if (G::in_lds(s + 1)) {
#pragma unroll
                for (int d = 0; d < 2; ++d)
#pragma unroll
                    for (int t = 0; t < 2; ++t) wl[d][t] = sm.w[(((wave * G::IN_LDS + G::lds(s + 1)) * 2 + d) * 2 + t) * 64 + lane];
            }
            const _Float16 by = (s & 1) != 0 ? -factor[s / NG] : factor[s / NG];
            const halfx8 hi = __builtin_bit_cast(halfx8, rows[s][0]) * by, lo = __builtin_bit_cast(halfx8, rows[s][1]) * by;
            request(!late, s, first_policy{});
            if (s == 0) {                                   // is there a piece, not of zeros, that the factors leave out?  (Here, beside the matrix instructions.)
                unsigned least = 0x7FFFu;
#pragma unroll
                for (int p = 0; p < P; ++p) least = min(least, ex_now[p] - (BackUnit<NG>::ALL_ZERO + 1));       // (a piece of zeros: the largest number)
                far = __ballot(least + (BackUnit<NG>::ALL_ZERO + 1 + FAR) < top && top < 255u) != 0ull;
            }
#pragma unroll
            for (int d = 0; d < 2; ++d) acc[s & 1][d] = __builtin_amdgcn_mfma_f32_16x16x32_f16(hi, G::in_lds(s) ? wl[d][0] : w.t[G::reg(s)][d][0], acc[s & 1][d], 0, 0, 0);
#pragma unroll
            for (int d = 0; d < 2; ++d) acc[s & 1][d] = __builtin_amdgcn_mfma_f32_16x16x32_f16(hi, G::in_lds(s) ? wl[d][1] : w.t[G::reg(s)][d][1], acc[s & 1][d], 0, 0, 0);
#pragma unroll
            for (int d = 0; d < 2; ++d) acc[s & 1][d] = __builtin_amdgcn_mfma_f32_16x16x32_f16(lo, G::in_lds(s) ? wl[d][0] : w.t[G::reg(s)][d][0], acc[s & 1][d], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (lane < 16) sm.row_scale[wave][lane] = back;
        const floatx4 r4 = *reinterpret_cast<const floatx4 *>(&sm.row_scale[wave][4 * (lane >> 4)]);    // this wave's own writes
        float *red = sm.red[blk & 1];
        floatx4 *const own = reinterpret_cast<floatx4 *>(&red[(wave * 2 * 64 + lane) * 4]);             // [side] 64 apart
#pragma unroll
        for (int d = 0; d < 2; ++d) own[64 * d] = (acc[0][d] - acc[1][d]) * r4;
        if (__builtin_expect(far, 0)) far_bands(here_start, here_m, top, own);
        __syncthreads();
        if (FLOW && sm.gave_up != 0) return;
        float da[2];
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            float p[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) p[k] = red[((k * 2 + d) * 64 + 16 * wave + (lane & 15)) * 4 + (lane >> 4)];
            da[d] = (((p[0] + p[1]) + p[2]) + p[3]) * sm.scale[d * HU + (lane & 15)];
        }
        const bool again = e.x >= 0 && unit.hu_ok && !(__builtin_isfinite(da[0]) && __builtin_isfinite(da[1]));
        if (__builtin_expect(__ballot(again) != 0ull, 0)) {
            if (again) {
                da[0] = unit.plain(here_start, here_m, fin_row, 0);
                da[1] = unit.plain(here_start, here_m, fin_row, 1);
            }
            __builtin_amdgcn_s_waitcnt(0);
        }
        float dc[2] = {__uint_as_float(dc2.x), __uint_as_float(dc2.y)};
        if constexpr (LSTM && FLOW) {
            dc[0] = flow_wait_c<true>(f, unit.rs_dc, unit.at(parent) * 2u, dc[0]);
            dc[1] = flow_wait_c<true>(f, unit.rs_dc, unit.at(parent) * 2u + 4u, dc[1]);
        }
        const bool there[2] = {e.x >= 0, e.x >= 0};
        const int4 pl = sm.ring[blk & 3][16 + fin_row];
        const int node[2] = {e.y, e.z};
        const int2 place[2] = {int2{pl.x, pl.y}, int2{pl.z, pl.w}};
        const float dh[2] = {in[0].gh + da[0], in[1].gh + da[1]};
        unit.finish(there, node, place, in, dh, dc);
        if (late && !last) request_first(first_policy{});
        in[0] = in_next[0];
        in[1] = in_next[1];
    }
}

template <int NG, int P>
__global__ __launch_bounds__(WG_THREADS, 1) void k_back_flow(Fwd f, BackFlow b)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    using Smem = BackSmem<NG, P>;
    Smem &sm = *reinterpret_cast<Smem *>(smem_raw);
    const int tid = threadIdx.x;
    const bool leave = tid == 0 && (batch_rejected(f) || back_by_heights(f));      // (a workgroup that gives up latches that)
    int member, slot;
    split_place(f, &slot, &member);
    member = gang_cg(member, f.n_cg, f.n_cg);     // (neighbouring units from one L2 domain)
    if (tid == 0) sm.gave_up = 0;
    BackWeights<NG, P> w;
    back_load<NG, P>(w, sm, b, member, tid >> 6, tid & 63);
    const int4 head = f.sched_head[slot];         // (of an earlier batch where this one is rejected: not used then)
    const int4 trees = b.at.trees[slot];
    if (decided_to_leave(&sm.leave, leave)) return;
    const BackUnit<NG> unit(f, b, sm.stage[tid >> 6], member, tid & 63);
    back_roots<NG>(f, b, unit, trees.x, trees.y, tid >> 6, WG_THREADS / 64);
    const int4 *entries = f.sched + (size_t)head.x * 16;
    const size_t apart = (size_t)(b.at.children - f.sched);
    const int n_blocks = head.y;
    if (n_blocks > 0)
        back_run<NG, P, true>(sm, f, b, unit, n_blocks, w, [=](int blk, int i) { return entries[(size_t)(n_blocks - 1 - blk) * 16 + (i & 15) + (i < 16 ? 0 : apart)]; },
                             [end = trees.z + trees.w](int, int m) mutable { return end -= m; });
}

// A batch with trees that are large beside the others (back_by_heights): the host does not know whether it is one, and the five launches that list the heights
// elsewhere would leave at once for almost all batches, at 2 us each.  So the work is done beside other work.  Here, in k_back_prepare: the roots, the heights, how many nodes have each.
// (Counters in LDS first, HIST_BINS of them: some thousand additions to one address from all over the chip are 50 us.)
__device__ __forceinline__ void back_heights_of(const Fwd &f, int *hist, size_t first, size_t stride)
{
    Ctl *ctl = f.ctl;
    for (int i = threadIdx.x; i < HIST_BINS; i += WG_THREADS) hist[i] = 0;
    if (decided_to_leave(hist + HIST_BINS, threadIdx.x == 0 && batch_rejected(f))) return;
    for (size_t n = first; n < (size_t)f.n_nodes; n += stride)
        if (f.parent[n] < 0) {
            if (atomicCAS(&f.root_ws[tree_of(f.tree_off, f.n_trees, (int)n)], -1, (int)n) != -1) latch_error(ctl, TL_ESTRUCT);      // a second root of the same tree
            atomicAdd(&ctl->n_roots, 1);
        }
    for (size_t i = first; i < (size_t)f.n_leaf; i += stride) {
        int top = 0, count = 0;
        climb_from(f, f.leaf_list[i], [&](int height) {
            atomicAdd(height < HIST_BINS ? &hist[height] : &f.level_cnt[height], 1);
            top = height;
            count += 1;
        });
        if (count > 0) {
            atomicMax(&ctl->max_height, top);
            atomicAdd(&ctl->reached, count);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < HIST_BINS; i += WG_THREADS)
        if (hist[i] != 0) atomicAdd(&f.level_cnt[i], hist[i]);
}
// ... before any row is computed: a tree without a root, or nodes that no leaf leads to (a cycle)?  (Counts that are final; the host's copy of them says the same.)
__device__ inline bool back_rejected(const Fwd &f)
{
    if (f.ctl->n_roots == f.n_trees && f.ctl->reached == f.n_int) return false;
    latch_error(f.ctl, TL_ESTRUCT);
    return true;
}
// ... and from these counts the lists of all heights and the places of all nodes.  False where a wait was given up.
template <typename Smem> __device__ __forceinline__ bool back_lists(Smem &sm, const Fwd &f, const BackFlow &b, unsigned &epoch)
{
    static_assert(sizeof(sm.red) >= 2 * HIST_BINS * sizeof(int), "counters");
    const int tid = threadIdx.x, n_levels = f.ctl->max_height + 1;
    unsigned unused = 0;
    if (blockIdx.x == 0) {                                  // exclusive sums of the counts, a share of the heights per thread
        int *sums = reinterpret_cast<int *>(sm.red);
        const int share = (n_levels + WG_THREADS - 1) / WG_THREADS, lo = min(tid * share, n_levels), hi = min(lo + share, n_levels);
        int sum = 0;
        for (int l = lo; l < hi; ++l) sum += f.level_cnt[l];
        sums[tid] = sum;
        __syncthreads();
        for (int d = 1; d < WG_THREADS; d <<= 1) {
            const int add = tid >= d ? sums[tid - d] : 0;
            __syncthreads();
            sums[tid] += add;
            __syncthreads();
        }
        int at = sums[tid] - sum;
        for (int l = lo; l < hi; ++l) {
            st_dev(f.level_off + l, at);
            at += f.level_cnt[l];
        }
        if (tid == WG_THREADS - 1) {
            st_dev(f.level_off + n_levels, at);
            st_dev(&f.ctl->n_levels, n_levels);
        }
    }
    if (!grid_barrier(sm, f, epoch, 0u, 0u, &unused)) return false;
    int *hist = reinterpret_cast<int *>(sm.red), *place = hist + HIST_BINS;
    for (long long n0 = (long long)blockIdx.x * WG_THREADS; n0 < f.n_nodes; n0 += (long long)gridDim.x * WG_THREADS) {
        const int n = (int)n0 + tid;
        for (int i = tid; i < HIST_BINS; i += WG_THREADS) hist[i] = 0;
        __syncthreads();
        const bool inner = n < f.n_nodes && f.left[n] >= 0;
        const int height = inner ? f.height[n] : 0;
        int i = !inner ? 0 : height < HIST_BINS ? atomicAdd(&hist[height], 1) : add_dev(f.level_fill + height, 1);
        __syncthreads();
        for (int k = tid; k < HIST_BINS; k += WG_THREADS)
            if (hist[k] != 0) place[k] = add_dev(f.level_fill + k, hist[k]);
        __syncthreads();
        if (inner) {
            if (height < HIST_BINS) i += place[height];
            const int lo = ld_dev(f.level_off + height), block = i & ~15;
            st_dev(f.level_nodes + lo + i, n);
            st_dev(reinterpret_cast<unsigned long long *>(b.at.of + n),
                   pack2((unsigned)(lo + block), (unsigned)(min(16, ld_dev(f.level_off + height + 1) - lo - block) | (i - block) << 8)));
        }
    }
    if (!grid_barrier(sm, f, epoch, 0u, 0u, &unused)) return false;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");      // the lists and places are read with ordinary loads from here on
    return true;
}

// The same cell height by height: all workgroups share the blocks of a height.  The whole walk in one launch, a grid barrier per height (back_by_heights), or a
// launch for the roots and for each height.
constexpr int BACK_ALL = 0, BACK_ROOTS = 1, BACK_HEIGHT = 2;
template <int NG, int P>
__global__ __launch_bounds__(WG_THREADS, 1) void k_back_heights(Fwd f, BackFlow b, int what, int lo0, int rows0)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    using Smem = BackSmem<NG, P>;
    Smem &sm = *reinterpret_cast<Smem *>(smem_raw);
    const int tid = threadIdx.x;
    const bool leave = tid == 0 && (batch_rejected(f) || (what == BACK_ALL && (!back_by_heights(f) || back_rejected(f))));
    const int member = (int)blockIdx.x % f.n_cg, slot = (int)blockIdx.x / f.n_cg, n_slots = (int)gridDim.x / f.n_cg;
    if (decided_to_leave(&sm.leave, leave)) return;
    const BackUnit<NG> unit(f, b, sm.stage[tid >> 6], member, tid & 63);
    unsigned epoch = 0, unused = 0;
    if (what == BACK_ALL && !back_lists(sm, f, b, epoch)) return;
    if (what != BACK_HEIGHT) back_roots<NG>(f, b, unit, 0, f.n_trees, slot * (WG_THREADS / 64) + (tid >> 6), n_slots * (WG_THREADS / 64));
    if (what == BACK_ROOTS) return;
    const bool all = what == BACK_ALL;
    BackWeights<NG, P> w;
    back_load<NG, P>(w, sm, b, member, tid >> 6, tid & 63);
    if (all && !grid_barrier(sm, f, epoch, 0u, 0u, &unused)) return;
    __syncthreads();
    const int n_levels = all ? f.ctl->max_height + 1 : 2;
#pragma unroll 1
    for (int lvl = n_levels - 1; lvl >= 1; --lvl) {         // roots first: a parent is always higher than its children
        const int lo = all ? ld_dev(f.level_off + lvl) : lo0, n_rows = all ? ld_dev(f.level_off + lvl + 1) - lo : rows0;
        const int32_t *list = f.level_nodes + lo;
        const int n_blocks = (n_rows + 15) >> 4, mine = slot < n_blocks ? (n_blocks - slot + n_slots - 1) / n_slots : 0;
        if (mine > 0)
            back_run<NG, P, false>(sm, f, b, unit, mine, w, [&](int blk, int at) {
                const int first = (slot + blk * n_slots) * 16, i = first + (at & 15);
                const int n = list[i < n_rows ? i : first], l = f.left[n], r = f.right[n];
                if (at < 16) return int4{i < n_rows ? n : -1, l, r, 0};
                const int2 pl = b.at.of[l], pr = b.at.of[r];
                return int4{pl.x, pl.y, pr.x, pr.y};
            }, [&](int blk, int) { return lo + (slot + blk * n_slots) * 16; });
        if (all && !grid_barrier(sm, f, epoch, 0u, 0u, &unused)) return;
    }
}

// In front of them: marks the rows that internal nodes will produce ("not written"), clears their rows of d_x and what the weight gradients add to,
// and prepares the schedule in the first n_sched workgroups beside it.
struct ClearList {
    float *p[4];
    size_t n[4];
};
__global__ __launch_bounds__(WG_THREADS) void k_back_prepare(Fwd f, BackFlow b, ClearList z, int ng, int marks, int n_sched, int lds_bytes)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    if ((int)blockIdx.x < n_sched) {
        flow_schedule<true>(f, blockIdx.x, smem_raw, (size_t)lds_bytes, b.at);
        return;
    }
    const int lane = threadIdx.x & 63, H = f.H, n_cg = f.n_cg;
    const bool by_heights = back_by_heights(f);
    marks = marks && !by_heights;                           // (where the heights are walked nobody reads them)
    const size_t first = (size_t)(blockIdx.x - n_sched) * WG_THREADS + threadIdx.x, stride = (size_t)(gridDim.x - n_sched) * WG_THREADS;
    if (by_heights) back_heights_of(f, reinterpret_cast<int *>(smem_raw), first, stride);
    const float ones = __uint_as_float(0xFFFFFFFFu);
    const floatx4 ones4 = floatx4{ones, ones, ones, ones};
    if (marks) {
        const size_t n_gx = (size_t)f.n_int * (b.n_pairs * ng * 8);
        floatx4 *gx = reinterpret_cast<floatx4 *>(b.gx);
        for (size_t e = first; e < n_gx; e += stride) gx[e] = ones4;
        for (size_t e = first; e < (size_t)f.n_int * n_cg; e += stride) b.gs[e] = 0xFFFFFFFFu;
    }
    auto node_row = [&](size_t n) {
        if (marks && b.dc)
            for (int e = lane; e < 2 * H; e += 64) b.dc[n * 2 * H + e] = ones;
        for (int e = lane; e < f.E; e += 64) f.d_x[n * f.E + e] = 0.f;
    };
    // (the kinds of up to 64 nodes in one load, as in flow_fill)
    const size_t N = (size_t)f.n_nodes, wave = first >> 6, n_waves = stride >> 6;
    const size_t share = (N + n_waves - 1) / n_waves, chunk = share < 64 ? share : 64;
    for (size_t n0 = wave * chunk; n0 < N; n0 += n_waves * chunk) {
        const size_t n = n0 + lane;
        const bool here = (size_t)lane < chunk && n < N, inner = f.left[n < N ? n : N - 1] >= 0;
        if (here && !inner) b.at.of[n] = int2{-1, 0};
        unsigned long long todo = __ballot(here && inner);
        for (; todo != 0ull; todo &= todo - 1ull) node_row(n0 + __builtin_ctzll(todo));
    }
#pragma unroll
    for (int a = 0; a < 4; ++a)
        for (size_t e = first; e < z.n[a]; e += stride) z.p[a][e] = 0.f;
}

// ---- leaves of the TreeLSTM ------------------------------------------------------------------------
// d_x[leaf] = dG_leaf W_leaf^T: the contraction of k_leaf_split with the roles of its columns exchanged.  A workgroup keeps NC column groups (16 values of the
// embedding each) of W_leaf^T and walks a contiguous share of the leaf list; a row of 3 H gate gradients is split in registers, a quarter (a wave's part of the
// K axis) by the power of two of its largest magnitude.
// Lane l asks for the values 32 step + 4 (l & 3) ... + 3 of row l / 4 and those 16 further on: as an operand it would hold row l & 15, and a load in that
// order costs the address unit a line per lane, 64 clocks for 1 KB, where four lanes on 64 consecutive bytes cost 16 (16 rows of 2 KB by a
// workgroup, rows in the L2: 866 -> 304 ns).  The terms are turned through LDS that is the wave's own; the 16-byte pieces of a row are permuted so that eight
// neighbouring lanes of a read meet 32 different banks.  (6 914 leaves, H = 512, E = 300, profiler: 86 us with fp32 instructions, 77 in operand order, 68.
// The forward's rows gain nothing by it: there a block waits for rows that are few, or for the conversion.)
constexpr int TURN_BYTES = 2048;            // of a k-step: 16 rows of 64 bytes, hi and lo
__device__ inline unsigned turn_read(int lane) { return (unsigned)((lane & 15) * 64 + (((lane >> 4) ^ (lane >> 2 & 3)) << 4)); }       // row l & 15, piece l >> 4
typedef _Float16 halfx4 __attribute__((ext_vector_type(4)));
template <int S, int NC> struct BackLeafSmem {
    unsigned char turn[4][S * TURN_BYTES];
    float red[2][4 * NC * 64 * 4];
    float scale[NC * HU];
    float row_scale[4][16];
    int leave;
};
template <int S, int NC>
__global__ __launch_bounds__(WG_THREADS, S * NC * 8 <= 96 ? 2 : 1) void k_back_leaf(Fwd f, const float *__restrict__ dg, int stride, const void *packed,
                                                                                    const float *__restrict__ scales, const float *__restrict__ w_leaf)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    using Smem = BackLeafSmem<S, NC>;
    Smem &sm = *reinterpret_cast<Smem *>(smem_raw);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (decided_to_leave(&sm.leave, tid == 0 && batch_rejected(f))) return;
    const int E = f.E, K = 3 * f.H, n_cge = (E + HU - 1) / HU, groups = (n_cge + NC - 1) / NC;
    // the workgroups that read the same rows lie on one L2 domain (the grid is a whole number of slots on each)
    const int group = (int)blockIdx.x / N_XCD % groups, slot = (int)blockIdx.x / N_XCD / groups * N_XCD + (int)blockIdx.x % N_XCD, n_slots = (int)gridDim.x / groups;
    halfx8 w[S][NC][2];
#pragma unroll
    for (int g = 0; g < NC; ++g) {
        // (column groups beyond the last repeat it; their results are not stored)
        const halfx8 *wp = reinterpret_cast<const halfx8 *>(packed) + ((size_t)min(group * NC + g, n_cge - 1) * 4 * S + (size_t)wave * S) * 2 * 64 + lane;
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int t = 0; t < 2; ++t) w[s][g][t] = wp[(size_t)(s * 2 + t) * 64];
    }
    if (tid < NC * HU) sm.scale[tid] = group * NC * HU + tid < E ? scales[group * NC * HU + tid] : 0.f;
    if constexpr (S * NC * 8 > 128) {
        constexpr int KEEP = S * NC * 8 > 256 ? (S * NC * 8 - 256 + NC * 8 - 1) / (NC * 8) : 0;
#pragma unroll
        for (int s = KEEP; s < S; ++s)
#pragma unroll
            for (int g = 0; g < NC; ++g)
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    floatx4 v = __builtin_bit_cast(floatx4, w[s][g][t]);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        float e = v[i];
                        asm volatile("" : "+a"(e));             // no instruction: a register-class constraint only
                        v[i] = e;
                    }
                    w[s][g][t] = __builtin_bit_cast(halfx8, v);
                }
    }
    __syncthreads();
    const int share = ((f.n_leaf + n_slots - 1) / n_slots + 15) & ~15;
    const int lo = slot * share, hi = min(f.n_leaf, lo + share), n_blocks = (hi - lo + 15) >> 4;
    if (n_blocks <= 0) return;
    const unsigned row_b = (unsigned)stride * 4u;
    const __amdgpu_buffer_rsrc_t rs = buf_of(dg, (unsigned long long)f.n_nodes * row_b), rs_x = buf_of(f.d_x, (unsigned long long)f.n_nodes * E * 4);
    const int k0 = wave * S * 32 + 4 * (lane & 3), w_row = lane >> 2;      // as in split_leaves
    const bool whole = (wave + 1) * S * 32 <= K;                // no step of this wave reaches beyond the row
    unsigned char *const a_w = sm.turn[wave];
    unsigned to[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) to[t] = (unsigned)(w_row * 64 + ((((lane & 3) / 2 + 2 * t) ^ (w_row >> 2 & 3)) << 4) + (lane & 1) * 8);
    const unsigned from = turn_read(lane);
    uintx4_t rows[S][2];
    auto request = [&](int node) __attribute__((always_inline)) {
        const unsigned base = (unsigned)node * row_b;
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int t = 0; t < 2; ++t) rows[s][t] = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(base + 4u * (unsigned)min(k0 + 32 * s + 16 * t, K)), 0, 0);
    };
    auto node_of = [&](int blk) { return f.leaf_list[min(lo + blk * 16 + w_row, hi - 1)]; };
    int node0 = node_of(0), node1 = node_of(1);
    request(node0);
#pragma unroll 1
    for (int blk = 0; blk < n_blocks; ++blk) {
        const int node2 = node_of(blk + 2);
        float m = 0.f;
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                if (!whole && k0 + 32 * s + 16 * (i >> 2) + (i & 3) >= K) rows[s][i >> 2][i & 3] = 0u;
                m = fmaxf(m, fabsf(__uint_as_float(rows[s][i >> 2][i & 3])));
            }
        m = fmaxf(m, dpp<DPP_XOR1>(m));
        m = fmaxf(m, dpp<DPP_XOR2>(m));
        const unsigned eb = max(__float_as_uint(m) >> 23, 15u);
        const float scale = __uint_as_float((268u - eb) << 23), back = __uint_as_float((eb - 14u) << 23);
        if ((lane & 3) == 0) sm.row_scale[wave][w_row] = back;
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                halfx4 vh, vl;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float v = __uint_as_float(rows[s][t][i]) * ((s & 1) != 0 ? -scale : scale);
                    vh[i] = (_Float16)v;
                    vl[i] = (_Float16)(v - (float)vh[i]);
                }
                *reinterpret_cast<halfx4 *>(a_w + s * TURN_BYTES + to[t]) = vh;
                *reinterpret_cast<halfx4 *>(a_w + s * TURN_BYTES + TURN_BYTES / 2 + to[t]) = vl;
            }
        request(node1);                                         // (behind the last block: the last leaf's row again)
        floatx4 acc[2][NC] = {};                                // (every other k-step is negated and subtracted, as in back_run)
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const halfx8 vh = *reinterpret_cast<const halfx8 *>(a_w + s * TURN_BYTES + from), vl = *reinterpret_cast<const halfx8 *>(a_w + s * TURN_BYTES + TURN_BYTES / 2 + from);
#pragma unroll
            for (int g = 0; g < NC; ++g) acc[s & 1][g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vh, w[s][g][0], acc[s & 1][g], 0, 0, 0);
#pragma unroll
            for (int g = 0; g < NC; ++g) acc[s & 1][g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vh, w[s][g][1], acc[s & 1][g], 0, 0, 0);
#pragma unroll
            for (int g = 0; g < NC; ++g) acc[s & 1][g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vl, w[s][g][0], acc[s & 1][g], 0, 0, 0);
        }
        float *red = sm.red[blk & 1];
        const floatx4 r4 = *reinterpret_cast<const floatx4 *>(&sm.row_scale[wave][4 * (lane >> 4)]);    // this wave's own writes
#pragma unroll
        for (int g = 0; g < NC; ++g) *reinterpret_cast<floatx4 *>(&red[((wave * NC + g) * 64 + lane) * 4]) = (acc[0][g] - acc[1][g]) * r4;
        const int fin_row = 4 * wave + (lane >> 4), node = __shfl(node0, 4 * fin_row);
        __syncthreads();
#pragma unroll
        for (int g = 0; g < NC; ++g) {
            float p[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) p[k] = red[((k * NC + g) * 64 + 16 * wave + (lane & 15)) * 4 + (lane >> 4)];
            float sum = (((p[0] + p[1]) + p[2]) + p[3]) * sm.scale[g * HU + (lane & 15)];
            const int col = (group * NC + g) * HU + (lane & 15);
            const bool here = col < E && lo + blk * 16 + fin_row < hi, again = here && !__builtin_isfinite(sum);
            if (__builtin_expect(__ballot(again) != 0ull, 0)) {
                if (again) {                                                // in fp32 from the parameters as given (a NaN stays one, as in BackUnit::plain)
                    const float *a = dg + (size_t)node * stride, *wr = w_leaf + (size_t)col * K;
                    sum = 0.f;
#pragma unroll 1
                    for (int k = 0; k < K && !__builtin_isnan(sum); ++k) sum = __builtin_fmaf(a[k], wr[k], sum);
                }
                __builtin_amdgcn_s_waitcnt(0);
            }
            // (without a branch: see split_leaves)
            buf_st_f<false>(rs_x, here ? ((unsigned)node * (unsigned)E + (unsigned)col) * 4u : ~0u, sum);
        }
        node0 = node1;
        node1 = node2;
    }
}

}  // namespace tl
