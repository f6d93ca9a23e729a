// fp32 cell of the data-flow scheduler on the 16-bit matrix unit: every fp32 operand as the sum of two fp16 terms.
//
// v_mfma_f32_16x16x4_f32 does 32 multiply-adds per clock and SIMD and occupies the vector pipe while it runs; the 16-bit
// instruction v_mfma_f32_16x16x32_f16 does 512 and runs beside vector instructions.  A value x is split into
// hi = fp16(x) and lo = fp16(x - hi), 11 bits each and a sign between them: hi + lo misses x by at most 2^-24 |x|, as much as
// rounding to fp32 does.  x w = hi hi' + hi lo' + lo hi' (+ lo lo', below 2^-24 of the product, left out): three instructions,
// exact products, fp32 accumulation, 3/16 of the fp32 instruction's time.  (Error of a forward against 64 bits, relative
// 2-norm, H=512 batch: see split_tile.)
// fp16 has five exponent bits, so both sides are scaled by powers of two: h (|h| <= 1) by 2^14, every column of the weights to
// a largest magnitude in [2^13, 2^14); a gate's sum is scaled back when its partial sums meet.  What lies more than
// 2^28 below the largest value of its kind keeps an absolute error of 2^-39 of that value.
//
// Layout of the split copy of h (`hx`, workspace): row n holds hx_steps groups of 32 hidden units, a group is one 128-byte line
// [32 hi][32 lo], pads zero.  It is written next to h by whoever computes a node, and lane l of a wave reads the A operand
// of a k-step straight from memory into registers: row l & 15, 16 bytes at 16 (l >> 4) of the hi and of the lo half.  No LDS
// stands between the row and the matrix instruction.
// The two halves of a 32-bit word belong to two hidden units and are stored together, so a word that shows all ones has not
// been written yet (see cell_ws.hpp, validity carried by the data).
//
// A column that holds an infinity has no such split; the pack kernel then raises `special`, and every gate is summed
// in fp32 from the parameters as given (slow, and only there).
#pragma once

#include "cell_ws.hpp"

namespace tl {

typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef unsigned int uintx4_t __attribute__((ext_vector_type(4)));

constexpr int SPLIT_MAX_S = 8;

struct SplitSmem {
    float red[2][4 * MAX_GATES * 64 * 4];   // K-split partial sums, alternating per block: [wave][gate][lane][v]
    int node[WS_TABLE_ROWS];                // tables as in WsSmemT
    int src0[WS_TABLE_ROWS];
    int src1[WS_TABLE_ROWS];
    int par[WS_TABLE_ROWS];
    int nxt[4][FLOW_NXT_ROWS];
    int roots[FLOW_ROOTS_KEPT];
    int cmd[8];
};

template <int NG, int S> struct SplitWeights {
    halfx8 hi[S][NG], lo[S][NG];
    float bias[NG], scale[NG];
    int special;
};

// k-steps [wave * S, (wave + 1) * S) of column group cg; the packed matrix has exactly 4 * S of them.
template <int NG, int S>
__device__ inline void split_load(SplitWeights<NG, S> &w, const SplitGemm &x, const Gemm &gm, int cg, int wave, int lane)
{
    const halfx8 *wp = reinterpret_cast<const halfx8 *>(x.wp) + ((size_t)cg * 4 * S + (size_t)wave * S) * NG * 2 * 64 + lane;
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            w.hi[s][g] = wp[(size_t)((s * NG + g) * 2) * 64];
            w.lo[s][g] = wp[(size_t)((s * NG + g) * 2 + 1) * 64];
        }
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        w.bias[g] = gm.bp[(cg * NG + g) * HU + (lane & 15)];
        w.scale[g] = x.scale[(cg * NG + g) * HU + (lane & 15)];
    }
    int special = 0;
#pragma unroll
    for (int g = 0; g < NG; ++g) special |= x.special[cg * NG + g];
    w.special = __builtin_amdgcn_readfirstlane(special);
    // With more weights than fit into the vector registers beside the rows in flight, say which of them live in the
    // accumulation registers (a matrix instruction reads either; see ws_load).
    if constexpr (S * NG * 8 > 128) {
#pragma unroll
        for (int s = 2; s < S; ++s)
#pragma unroll
            for (int g = 0; g < NG; ++g)
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    floatx4 v = __builtin_bit_cast(floatx4, t ? w.lo[s][g] : w.hi[s][g]);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        float e = v[i];
                        asm volatile("" : "+a"(e));             // no instruction: a register-class constraint only
                        v[i] = e;
                    }
                    (t ? w.lo[s][g] : w.hi[s][g]) = __builtin_bit_cast(halfx8, v);
                }
    }
}

// Gates of one node and hidden unit summed in fp32 from the parameters as given (weights that hold infinities); the
// children's h from their split copies, which all waves have seen complete.
template <int NG>
__device__ inline void split_gates_plain(const Fwd &f, const SplitGemm &x, int s0, int s1, int hu, float (&gate)[NG])
{
    const int H = f.H;
#pragma unroll
    for (int g = 0; g < NG; ++g) gate[g] = 0.f;
#pragma unroll 1
    for (int k = 0; k < 2 * H; ++k) {
        const int u = k < H ? k : k - H;
        const unsigned short *p = reinterpret_cast<const unsigned short *>(f.hx) + (size_t)(k < H ? s0 : s1) * f.hx_steps * 64 + (u >> 5) * 64 + (u & 31);
        const float a = ((float)__builtin_bit_cast(_Float16, ld_dev(p)) + (float)__builtin_bit_cast(_Float16, ld_dev(p + 32))) * (1.f / SPLIT_H_SCALE);
#pragma unroll
        for (int g = 0; g < NG; ++g) gate[g] = __builtin_fmaf(a, x.w[(size_t)k * ((size_t)NG * H) + (size_t)g * H + hu], gate[g]);
    }
}

// Evaluates the `count` <= WS_TABLE_ROWS internal nodes of the row tables for column group cg, 16 at a time, the rows of a
// block requested while the block before is computed.  Called and synchronised like ws_tile (cell_ws.hpp), same hooks.
// K axis: hx_steps k-steps of 32 units of the left child, then as many of the right one; wave w walks quarter w of
// 4 * S steps (those beyond the axis re-read the right child's last step against zero weights), each step's three
// products in the order hi hi, hi lo, lo hi; the four quarter sums are added in wave order.  A node's result so depends neither
// on its place in a block nor on the batch.
template <int S, typename Hook>
__device__ inline void split_tile(SplitSmem &sm, const Fwd &f, int count, int cg, const SplitWeights<5, S> &w, Hook hook)
{
    constexpr int NG = 5;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nrb = (count + 15) >> 4;
    const int H = f.H, steps = f.hx_steps;
    const int hu = cg * HU + (lane & 15);
    const bool hu_ok = hu < H;
    const unsigned row_b = (unsigned)H * 4u, hu_b = (unsigned)(hu_ok ? hu : 0) * 4u;
    const unsigned hx_row_b = (unsigned)steps * 128u;
    const unsigned long long hx_bytes = (unsigned long long)f.n_nodes * hx_row_b;
    const __amdgpu_buffer_rsrc_t rs_h = buf_of(f.h, (unsigned long long)f.n_nodes * H * 4), rs_c = buf_of(f.c, (unsigned long long)f.n_nodes * H * 4),
                                 rs_x = buf_of(f.hx, hx_bytes);
    const unsigned lane_off = (unsigned)(lane >> 4) * 16u;
    unsigned base0 = 0, base1 = 0;                              // this lane's row in the left and the right child's segment

    auto prepare = [&](int row0) {
        const int row = (row0 + (lane & 15)) & (WS_TABLE_ROWS - 1);
        base0 = __umul24((unsigned)sm.src0[row], hx_row_b) + lane_off;
        base1 = __umul24((unsigned)sm.src1[row], hx_row_b) + lane_off;
    };
    uintx4_t rows[S][2];
    auto request = [&](__amdgpu_buffer_rsrc_t rs, int s) {
        const int k = wave * S + s;
        const bool right = k >= steps;
        const int kk = min(right ? k - steps : k, steps - 1);
        const unsigned b = right ? base1 : base0;
        rows[s][0] = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)b, kk * 128, 16);
        rows[s][1] = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)b + 64, kk * 128, 16);
    };
    // The block's rows: requests repeated until no word shows the pattern.  Bounded by the spin budget and the abort flag.
    auto wait_rows = [&]() {
        int spins = 0;
        unsigned aborted = 0u;
        for (;;) {
            unsigned m = 0u;
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int t = 0; t < 2; ++t) m = max(max(m, max(rows[s][t].x, rows[s][t].y)), max(rows[s][t].z, rows[s][t].w));
            if (__ballot(m == FLOW_SENTINEL) == 0ull) return;
            if (++spins > f.spin_limit || aborted != 0u) {
                flow_give_up(f);
                sm.cmd[7] = 1;
                return;
            }
            backoff();
#pragma unroll
            for (int s = 0; s < S; ++s) request(rs_x, s);
            aborted = ld_dev(&f.ctl->abort.v);                  // arrives with the rows
        }
    };
    // Second half of a block: wave w finishes its rows 4 w .. 4 w + 3, lane l row 4 w + (l >> 4), hidden unit l & 15.
    auto finish = [&](const float *red, int enode, float cl, float cr, int erow) {
        float gate[NG];
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            float p[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) p[q] = red[((q * NG + g) * 64 + 16 * wave + (lane & 15)) * 4 + (lane >> 4)];
            gate[g] = __builtin_fmaf(((p[0] + p[1]) + p[2]) + p[3], w.scale[g], w.bias[g]);
        }
        if (enode >= 0) {
            const int s0 = sm.src0[erow & (WS_TABLE_ROWS - 1)], s1 = sm.src1[erow & (WS_TABLE_ROWS - 1)];
            float cc = 0.f, hh = 0.f;
            if (hu_ok) {
                cl = flow_wait_c<true>(f, rs_c, (unsigned)s0 * row_b + hu_b, cl);     // a child's c element may arrive after its h row
                cr = flow_wait_c<true>(f, rs_c, (unsigned)s1 * row_b + hu_b, cr);
                if (w.special) {
                    split_gates_plain<NG>(f, f.xi, s0, s1, hu, gate);
#pragma unroll
                    for (int g = 0; g < NG; ++g) gate[g] += w.bias[g];
                }
                lstm_inner_out(gate[0], gate[1], gate[2], gate[3], gate[4], cl, cr, &cc, &hh, kept_gates(f, enode, hu), H);
            }
            const unsigned word = split_word(hh * SPLIT_H_SCALE, hu);
            const unsigned o = (unsigned)enode * row_b + hu_b;
            if (hu_ok) {
                buf_st_f<true>(rs_h, o, hh);
                buf_st_f<true>(rs_c, o, cc);
            }
            if ((hu & ~1) < H) buf_st_f<true>(rs_x, (unsigned)enode * hx_row_b + split_word_off(hu), __uint_as_float(word));
        }
    };

    prepare(0);
#pragma unroll
    for (int s = 0; s < S; ++s) request(rs_x, s);
    hook(-1);
    int p_enode = -1, p_erow = 0;
    float p_cl = 0.f, p_cr = 0.f;
    constexpr int FINISH_AFTER = S > 1 ? 1 : 0;                 // k-step after which the block before is finished
    for (int rb = 0; rb < nrb; ++rb) {
        wait_rows();
        prepare((rb + 1) * 16);
        // (behind the last block the requests go to a table of no bytes: they return at once and read nothing)
        const __amdgpu_buffer_rsrc_t rs_next = buf_of(f.hx, rb + 1 < nrb ? hx_bytes : 0ull);
        hook(rb);
        const int erow = rb * 16 + 4 * wave + (lane >> 4);
        const int enode = erow < count ? sm.node[erow] : -1;
        const float cl = buf_ld_f<true>(rs_c, (unsigned)sm.src0[erow & (WS_TABLE_ROWS - 1)] * row_b + hu_b);
        const float cr = buf_ld_f<true>(rs_c, (unsigned)sm.src1[erow & (WS_TABLE_ROWS - 1)] * row_b + hu_b);
        __builtin_amdgcn_sched_barrier(0);
        floatx4 acc[NG];
#pragma unroll
        for (int g = 0; g < NG; ++g) acc[g] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const halfx8 hi = __builtin_bit_cast(halfx8, rows[s][0]), lo = __builtin_bit_cast(halfx8, rows[s][1]);
#pragma unroll
            for (int g = 0; g < NG; ++g) acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(hi, w.hi[s][g], acc[g], 0, 0, 0);
#pragma unroll
            for (int g = 0; g < NG; ++g) acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(hi, w.lo[s][g], acc[g], 0, 0, 0);
#pragma unroll
            for (int g = 0; g < NG; ++g) acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(lo, w.hi[s][g], acc[g], 0, 0, 0);
            request(rs_next, s);
            __builtin_amdgcn_sched_barrier(0);
            if (s == FINISH_AFTER && rb > 0) {
                __syncthreads();                                // every wave has written its partial sums of block rb - 1
                finish(sm.red[(rb - 1) & 1], p_enode, p_cl, p_cr, p_erow);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        float *red = sm.red[rb & 1];
#pragma unroll
        for (int g = 0; g < NG; ++g) *reinterpret_cast<floatx4 *>(&red[((wave * NG + g) * 64 + lane) * 4]) = acc[g];
        p_enode = enode;
        p_cl = cl;
        p_cr = cr;
        p_erow = erow;
    }
    hook(-2);
    __syncthreads();
    if (nrb > 0) finish(sm.red[(nrb - 1) & 1], p_enode, p_cl, p_cr, p_erow);
    __syncthreads();                                            // row tables and LDS may be rewritten after this call
}

}  // namespace tl
