// fp32 cell of the data-flow scheduler on the 16-bit matrix unit: every fp32 operand as the sum of two fp16 terms.
//
// v_mfma_f32_16x16x4_f32 does 32 multiply-adds per clock and SIMD and occupies the vector pipe while it runs; the 16-bit
// instruction v_mfma_f32_16x16x32_f16 does 512 and runs beside vector instructions.  A value x is split into
// hi = fp16(x) and lo = fp16(x - hi), 11 bits each and a sign between them: hi + lo misses x by at most 2^-23 |x| (three quarters of
// all fp32 values are met exactly).  x w = hi hi' + hi lo' + lo hi' (+ lo lo', up to 2^-22 of the product, left out): three
// instructions, exact products, fp32 accumulation, 3/16 of the fp32 instruction's time; a product is off by 2^-21 at most,
// where the fp32 instruction rounds it to 2^-24.  (Relative 2-norm error of h and c
// against 64 bits, with fp32 instructions / with the split: 256 parse trees at H = 512 1.1e-6 / 1.1e-6, 25 at H = 150 8.9e-7 /
// 8.9e-7, chains of 1 024 leaves at H = 256 8.1e-7 / 8.1e-7: the gate functions decide it, whose absolute error of about
// 1e-7 is that of all paths.)
// fp16 has five exponent bits, so both sides are scaled by powers of two: h (|h| <= 1) by 2^14, every column of the weights to
// a largest magnitude in [2^13, 2^14); a gate's sum is scaled back when its partial sums meet.  The lower term of what lies
// more than 2^15 below the largest value of its kind runs out of exponents: from there on the error is absolute, 2^-38 of that
// largest value (2^-39 for h), so 2^-22 of a value 2^-16 of the largest, 2^-18 of one 2^-20, 2^-10 of one 2^-28.  Embedding
// values of 1e-1 ... 1e-8 (h down to 1e-9; 25 trees, H = 150, no biases) give the errors of the fp32 instructions to two digits.
//
// Layout of the split copy of h (`hx`, workspace): row n holds hx_steps groups of 32 hidden units, a group is one 128-byte line
// [32 hi][32 lo], pads zero.  It is written next to h by whoever computes a node, and lane l of a wave reads the A operand
// of a k-step straight from memory into registers: row l & 15, 16 bytes at 16 (l >> 4) of the hi and of the lo half.  No LDS
// stands between the row and the matrix instruction.
// The two halves of a 32-bit word belong to two hidden units and are stored together, so a word that shows all ones has not
// been written yet (see cell_ws.hpp, validity carried by the data).
//
// An infinite weight has no such split; the scale of a column that holds one is a NaN, and its sums are taken in fp32
// from the parameters as given (slow, and only there).
#pragma once

#include "cell_ws.hpp"

namespace tl {

typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef unsigned int uintx4_t __attribute__((ext_vector_type(4)));

constexpr int SPLIT_MAX_S = 8;

struct SplitSmem {
    float red[2][4 * MAX_GATES * 64 * 4];   // K-split partial sums, alternating per block: [wave][gate][lane][v]
    float sum_of[MAX_GATES * HU * 2];       // scale and bias of every column (registers are short)
    int gave_up, leave;
};

template <int NG, int S> struct SplitWeights {
    halfx8 hi[S][NG], lo[S][NG];
    bool plain;                                                 // some unit of the column group has a weight that is infinite
};

// k-steps [wave * S, (wave + 1) * S) of column group cg; the packed matrix has exactly 4 * S of them.  sum_of: [gate][unit] {scale,
// bias} in LDS.  Called by all threads; a barrier must be passed before the first use.
template <int NG, int S>
__device__ inline void split_load(SplitWeights<NG, S> &w, float *sum_of, const SplitGemm &x, const Gemm &gm, int cg, int wave, int lane)
{
    const int t = wave * 64 + lane;
    float scale = 0.f, bias = 0.f;                              // requested first: nothing is waited for but themselves
    if (t < NG * HU) {
        scale = x.scale[cg * NG * HU + t];
        bias = gm.bp[cg * NG * HU + t];
    }
    __builtin_amdgcn_sched_barrier(0);
    const halfx8 *wp = reinterpret_cast<const halfx8 *>(x.wp) + ((size_t)cg * 4 * S + (size_t)wave * S) * NG * 2 * 64 + lane;
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            w.hi[s][g] = wp[(size_t)((s * NG + g) * 2) * 64];
            w.lo[s][g] = wp[(size_t)((s * NG + g) * 2 + 1) * 64];
        }
    if (t < NG * HU) {
        sum_of[2 * t] = scale;
        sum_of[2 * t + 1] = bias;
    }
    float scales = 0.f;
#pragma unroll
    for (int g = 0; g < NG; ++g) scales += x.scale[(cg * NG + g) * HU + (lane & 15)];
    w.plain = __ballot(__builtin_isnan(scales)) != 0ull;
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

// Gates of one node and hidden unit summed in fp32 from the parameters as given; the children's h from their split copies,
// which all waves have seen complete.
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

// Slot and column group of a workgroup.  Workgroups are dealt to the L2 domains round-robin; with f.place the slots are taken from
// one domain each as far as whole slots fit (a multiple of N_XCD of them; what is left over lies on all domains), so that a
// slot's rows cross the fabric once and its dependent rows not at all - and its requests queue at one L2.
__device__ inline void split_place(const Fwd &f, int *slot, int *member)
{
    const int b = blockIdx.x, inside = f.place ? f.n_slots / N_XCD * N_XCD : 0, first = inside * f.n_cg;
    if (b < first) {
        const int i = b / N_XCD;
        *member = i % f.n_cg;
        *slot = i / f.n_cg * N_XCD + b % N_XCD;
    } else {
        *member = (b - first) % f.n_cg;
        *slot = inside + (b - first) / f.n_cg;
    }
}

// Evaluates the blocks of one slot's schedule (structure.hpp, flow_schedule) for column group cg: 16 internal nodes a block,
// every node's children in earlier blocks, the rows of a block requested while the block before is computed - or,
// where a row of it comes out of that very block, once its results are stored.
// K axis: hx_steps k-steps of 32 units of the left child, then as many of the right one; wave w walks quarter w of
// 4 * S steps (those beyond the axis re-read the right child's last step against zero weights), each step's three
// products in the order hi hi, hi lo, lo hi; the four quarter sums are added in wave order.  A node's result so depends neither
// on its place in a block nor on the batch.
// Measured (H = 512, 256 parse trees, kernel): 388 us with fp32 instructions and lists taken in pieces, 236 with these instructions
// and the same lists, 173 on finished blocks, 151 with the slots spread over all L2 domains.  A wave's block is 120 matrix
// instructions of 16 clocks and 171 other vector instructions in 6 700 clocks (matrix unit 29 % busy): products, exchange of
// the quarters, gates and stores follow each other, and the dependent blocks at the top of the trees wait for their children's
// rows (a dependent block of few rows takes 2.3 us at H = 256, most of it the way of those rows through the L2).
template <int S>
__device__ inline void split_run(SplitSmem &sm, const Fwd &f, const int4 *__restrict__ entries, int n_blocks, int cg, const SplitWeights<5, S> &w)
{
    constexpr int NG = 5;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
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

    auto prepare = [&](const int4 &q) {
        base0 = __umul24((unsigned)q.y, hx_row_b) + lane_off;
        base1 = __umul24((unsigned)q.z, hx_row_b) + lane_off;
    };
    uintx4_t rows[S][2];
    // Rows are first asked for with ordinary loads: a line that this CU's or this L2's copy shows too early shows the pattern,
    // and only the repeated requests go past the caches.
    auto request = [&](__amdgpu_buffer_rsrc_t rs, int s, auto past_caches) {
        constexpr int POLICY = decltype(past_caches)::value ? 16 : 0;
        const int k = wave * S + s;
        const bool right = k >= steps;
        const int kk = min(right ? k - steps : k, steps - 1);
        const unsigned b = right ? base1 : base0;
        rows[s][0] = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)b, kk * 128, POLICY);
        rows[s][1] = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)b + 64, kk * 128, POLICY);
    };
    auto shows_pattern = [&]() {
        unsigned m = 0u;
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int t = 0; t < 2; ++t) m = max(max(m, max(rows[s][t].x, rows[s][t].y)), max(rows[s][t].z, rows[s][t].w));
        return __ballot(m == FLOW_SENTINEL) != 0ull;
    };
    // The block's rows: requests repeated until no word shows the pattern.  Bounded by the spin budget and the abort flag.
    auto repeat_rows = [&]() {
        int spins = 0;
        unsigned aborted = 0u;
        do {
            if (++spins > f.spin_limit || aborted != 0u) {
                flow_give_up(f);
                sm.gave_up = 1;
                return;
            }
            __builtin_amdgcn_s_sleep(1);
#pragma unroll
            for (int s = 0; s < S; ++s) request(rs_x, s, std::true_type{});
            aborted = ld_dev(&f.ctl->abort.v);                  // arrives with the rows
        } while (shows_pattern());
    };

    const int my_row = lane & 15, fin_row = 4 * wave + (lane >> 4);
    int4 q = entries[my_row], e = entries[fin_row];
    int4 q_next = n_blocks > 1 ? entries[16 + my_row] : q;
    prepare(q);
#pragma unroll
    for (int s = 0; s < S; ++s) request(rs_x, s, std::false_type{});
    for (int b = 0; b < n_blocks; ++b) {
        const bool last = b + 1 >= n_blocks;
        const bool late = last || __builtin_amdgcn_readfirstlane(q_next.w) < 0;     // the next block waits for this one
        const float cl0 = buf_ld_f<false>(rs_c, (unsigned)e.y * row_b + hu_b);
        const float cr0 = buf_ld_f<false>(rs_c, (unsigned)e.z * row_b + hu_b);
        const int4 *ahead = entries + (size_t)min(b + 2, n_blocks - 1) * 16;
        const int4 q_ahead = ahead[my_row];
        const int4 e_next = entries[(size_t)min(b + 1, n_blocks - 1) * 16 + fin_row];
        if (shows_pattern()) repeat_rows();
        prepare(q_next);
        // (requests that are not to be made yet go to a table of no bytes: they return at once and read nothing)
        const __amdgpu_buffer_rsrc_t rs_next = buf_of(f.hx, late ? 0ull : hx_bytes);
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
            request(rs_next, s, std::false_type{});
            __builtin_amdgcn_sched_barrier(0);
        }
        // The four quarter sums meet in LDS; wave w finishes the block's rows 4 w .. 4 w + 3, lane l row 4 w + (l >> 4), hidden
        // unit l & 15.  (The two buffers alternate: one is written again two blocks later, behind the next block's barrier.)
        float *red = sm.red[b & 1];
#pragma unroll
        for (int g = 0; g < NG; ++g) *reinterpret_cast<floatx4 *>(&red[((wave * NG + g) * 64 + lane) * 4]) = acc[g];
        __syncthreads();
        if (sm.gave_up != 0) return;
        float gate[NG];
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const float *sb = &sm.sum_of[(g * HU + (lane & 15)) * 2];
            float p[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) p[k] = red[((k * NG + g) * 64 + 16 * wave + (lane & 15)) * 4 + (lane >> 4)];
            gate[g] = __builtin_fmaf(((p[0] + p[1]) + p[2]) + p[3], sb[0], sb[1]);
        }
        if (e.x >= 0) {
            float cc = 0.f, hh = 0.f;
            if (hu_ok) {
                const float cl = flow_wait_c<true>(f, rs_c, (unsigned)e.y * row_b + hu_b, cl0);     // a child's c element may arrive after its h row
                const float cr = flow_wait_c<true>(f, rs_c, (unsigned)e.z * row_b + hu_b, cr0);
                if (__builtin_expect(w.plain, 0)) {
                    split_gates_plain<NG>(f, f.xi, e.y, e.z, hu, gate);
#pragma unroll
                    for (int g = 0; g < NG; ++g) gate[g] += sm.sum_of[(g * HU + (lane & 15)) * 2 + 1];
                }
                lstm_inner_out(gate[0], gate[1], gate[2], gate[3], gate[4], cl, cr, &cc, &hh, kept_planes(f, e.x, hu));
            }
            const unsigned word = split_word(hh * SPLIT_H_SCALE, hu);
            if ((hu & ~1) < H) buf_st_f<true>(rs_x, (unsigned)e.x * hx_row_b + split_word_off(hu), __uint_as_float(word));
            if (hu_ok) {
                const unsigned o = (unsigned)e.x * row_b + hu_b;
                buf_st_f<true>(rs_c, o, cc);
                buf_st_f<true>(rs_h, o, hh);
                const int t = (e.w & 0x7FFFFFFF) - 1;           // a root's tree
                if (t >= 0) {
                    if (f.h_root) f.h_root[(size_t)t * H + hu] = hh;
                    if (f.c_root) f.c_root[(size_t)t * H + hu] = cc;
                }
            }
        }
        if (late && !last) {
#pragma unroll
            for (int s = 0; s < S; ++s) request(rs_x, s, std::false_type{});
        }
        q_next = q_ahead;
        e = e_next;
    }
}

// ---- TreeRNN ---------------------------------------------------------------------------------------
// The same blocks for h = tanh(a W + b): NG column groups side by side in a workgroup take the place of the gates, and waves 0, 1 hold the
// left child's K axis, waves 2, 3 the right one's (S k-steps of 32 each).  Leaves are embedding rows of any magnitude, so every row of the
// split copy has a scale of its own, and f.hx_back[node] says what its sums are multiplied by (2^-14 for internal nodes).
// Few weights (32 registers per column group at H = 256), so that two workgroups fit on a CU; where one a CU is the faster way, and where a
// workgroup takes one column group or two that share the rows they gather, is decided in forward_impl, with the figures.  (NG = 1 / 2 / 4, two a
// CU, forward: 25 trees at H = 50 30.8 / 35.7 / 40.3 us, at H = 256 43.6 / 44.1 / 47.8, 256 trees there 80.4 / 71.9 / 74.6.  Before, with fp32
// instructions and lists taken in pieces: 41.7, 49.7, 86.0; with rows of h scaled, split and left in LDS for four waves of 16 units each: 34.6,
// 56.1, 79.6.  One a CU: 29.2, 41.5, 67.2.)
template <int NG> struct SplitRnnSmem {
    float red[2][4 * NG * 64 * 4];
    float sum_of[NG * HU * 2];
    float row_scale[4][16];
    int gave_up, leave;
};

// A node's sum in fp32 from the parameters as given (rare, and slow).  Leaves' rows are those of h; the rest of h may not be there yet
// when the split copy is, whose values are finite (or NaN).
__device__ __forceinline__ float split_rnn_plain(const Fwd &f, int l, int r, int hu)
{
    const int H = f.H;
    float sum = 0.f;
#pragma unroll 1
    for (int k = 0; k < 2 * H; ++k) {
        const int u = k < H ? k : k - H, n = k < H ? l : r;
        float a;
        if (f.left[n] < 0) {
            a = f.h[(size_t)n * H + u];
        } else {
            const unsigned short *p = reinterpret_cast<const unsigned short *>(f.hx) + (size_t)n * f.hx_steps * 64 + (u >> 5) * 64 + (u & 31);
            a = ((float)__builtin_bit_cast(_Float16, ld_dev(p)) + (float)__builtin_bit_cast(_Float16, ld_dev(p + 32))) * (1.f / SPLIT_H_SCALE);
        }
        sum = __builtin_fmaf(a, f.xi.w[(size_t)k * H + hu], sum);
    }
    return sum;
}

// The packed matrix is [column group][4 S k-steps][hi, lo][lane][8] whatever NG; groups beyond the last are zeros up to an even number.
template <int NG, int S>
__device__ __forceinline__ void split_rnn_load(SplitWeights<NG, S> &w, float *sum_of, const Fwd &f, int cg, int wave, int lane)
{
    const int t = wave * 64 + lane, u = cg * NG * HU + t;
    if (t < NG * HU) {
        sum_of[2 * t] = u < f.H ? f.xi.scale[u] : 0.f;
        sum_of[2 * t + 1] = u < f.H ? f.inner.bp[u] : 0.f;
    }
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        const halfx8 *wp = reinterpret_cast<const halfx8 *>(f.xi.wp) + ((size_t)(cg * NG + g) * 4 * S + (size_t)wave * S) * 2 * 64 + lane;
#pragma unroll
        for (int s = 0; s < S; ++s) {
            w.hi[s][g] = wp[(size_t)(s * 2) * 64];
            w.lo[s][g] = wp[(size_t)(s * 2 + 1) * 64];
        }
    }
}

template <int NG, int S>
__device__ __forceinline__ void split_rnn_run(SplitRnnSmem<NG> &sm, const Fwd &f, const int4 *__restrict__ entries, int n_blocks, int cg, const SplitWeights<NG, S> &w)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int H = f.H, steps = f.hx_steps, hu0 = cg * NG * HU + (lane & 15);
    const unsigned row_b = (unsigned)H * 4u, hx_row_b = (unsigned)steps * 128u;
    const unsigned long long hx_bytes = (unsigned long long)f.n_nodes * hx_row_b;
    const __amdgpu_buffer_rsrc_t rs_h = buf_of(f.h, (unsigned long long)f.n_nodes * row_b), rs_x = buf_of(f.hx, hx_bytes);
    const unsigned lane_off = (unsigned)(lane >> 4) * 16u;
    unsigned base = 0;                                          // this lane's row in the split copy: of its wave's child
    float back = 0.f;
    uintx4_t rows[S][2];
    auto prepare = [&](const int4 &q) __attribute__((always_inline)) {
        const int child = wave < 2 ? q.y : q.z;
        base = __umul24((unsigned)child, hx_row_b) + lane_off;
        return f.hx_back[child];
    };
    auto request = [&](auto past_caches) __attribute__((always_inline)) {
        constexpr int POLICY = decltype(past_caches)::value ? 16 : 0;
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int kk = min((wave & 1) * S + s, steps - 1);  // (beyond the row: its last step again, against zero weights)
            rows[s][0] = __builtin_amdgcn_raw_buffer_load_b128(rs_x, (int)base, kk * 128, POLICY);
            rows[s][1] = __builtin_amdgcn_raw_buffer_load_b128(rs_x, (int)base + 64, kk * 128, POLICY);
        }
    };
    auto shows_pattern = [&]() __attribute__((always_inline)) {
        unsigned m = 0u;
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int t = 0; t < 2; ++t) m = max(max(m, max(rows[s][t].x, rows[s][t].y)), max(rows[s][t].z, rows[s][t].w));
        return __ballot(m == FLOW_SENTINEL) != 0ull;
    };
    const int my_row = lane & 15, fin_row = 4 * wave + (lane >> 4);
    int4 q = entries[my_row], e = entries[fin_row];
    int4 q_next = n_blocks > 1 ? entries[16 + my_row] : q;
    back = prepare(q);
    request(std::false_type{});
#pragma unroll 1
    for (int b = 0; b < n_blocks; ++b) {
        const bool last = b + 1 >= n_blocks;
        const bool late = last || __builtin_amdgcn_readfirstlane(q_next.w) < 0;     // the next block waits for this one
        const int4 q_ahead = entries[(size_t)min(b + 2, n_blocks - 1) * 16 + my_row];
        const int4 e_next = entries[(size_t)min(b + 1, n_blocks - 1) * 16 + fin_row];
        if (shows_pattern()) {
            int spins = 0;
            unsigned aborted = 0u;
            do {                                                // bounded by the spin budget and the abort flag
                if (++spins > f.spin_limit || aborted != 0u) {
                    flow_give_up(f);
                    sm.gave_up = 1;
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
                request(std::true_type{});
                aborted = ld_dev(&f.ctl->abort.v);              // arrives with the rows
            } while (shows_pattern());
        }
        if (lane < 16) sm.row_scale[wave][lane] = back;
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
        }
        const float back_next = prepare(q_next);
        if (!late) request(std::false_type{});
        // the four quarter sums meet in LDS, as in split_run
        float *red = sm.red[b & 1];
        const floatx4 r4 = *reinterpret_cast<const floatx4 *>(&sm.row_scale[wave][4 * (lane >> 4)]);    // this wave's own writes
#pragma unroll
        for (int g = 0; g < NG; ++g) *reinterpret_cast<floatx4 *>(&red[((wave * NG + g) * 64 + lane) * 4]) = acc[g] * r4;
        __syncthreads();
        if (sm.gave_up != 0) return;
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const float *sb = &sm.sum_of[(g * HU + (lane & 15)) * 2];
            float p[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) p[k] = red[((k * NG + g) * 64 + 16 * wave + (lane & 15)) * 4 + (lane >> 4)];
            const int hu = hu0 + g * HU;
            float sum = (((p[0] + p[1]) + p[2]) + p[3]) * sb[0];
            if (e.x >= 0) {
                if (__builtin_expect(!__builtin_isfinite(sum) && hu < H, 0)) sum = split_rnn_plain(f, e.y, e.z, hu);
                const float hh = hu < H ? tanh_f(sum + sb[1]) : 0.f;
                const unsigned word = split_word(hh * SPLIT_H_SCALE, hu);
                if ((hu & ~1) < H) buf_st_f<true>(rs_x, (unsigned)e.x * hx_row_b + split_word_off(hu), __uint_as_float(word));
                if (hu < H) {
                    buf_st_f<true>(rs_h, (unsigned)e.x * row_b + (unsigned)hu * 4u, hh);
                    const int t = (e.w & 0x7FFFFFFF) - 1;       // a root's tree
                    if (t >= 0 && f.h_root) f.h_root[(size_t)t * H + hu] = hh;
                }
            }
        }
        if (late && !last) request(std::true_type{});           // (past the caches: what they hold of these rows is too old)
        back = back_next;
        q_next = q_ahead;
        e = e_next;
    }
}

// ---- leaves ----------------------------------------------------------------------------------------
// Lane l of a wave holds, for row l & 15, the eight embedding values k = 32 step + 8 (l >> 4) ... + 7 of each of its wave's S
// steps: 16-byte loads (rows need 4-byte alignment only), straight into the registers that become the A operands.  An
// embedding may have any magnitude, so every row is scaled for itself, and for each quarter of the K axis: by the power of two
// that brings the quarter's largest magnitude into [2^14, 2^15); the wave scales its partial sums back before they meet.
// What lies beyond the row's end counts as zero.  A row that holds an infinity or a NaN (and a column of weights that holds an
// infinity) comes out as NaN here, and a partial sum may overflow because it is scaled; such sums are then taken in fp32.
// Measured (6 914 leaves, E = 300, H = 512): 81 us with fp32 instructions, 64 with these and the schedule prepared on the side; tiny
// and ragged batches gain most.  What bounds it now is not the matrix unit (27 instructions a block) but the chain of a
// block: row maximum across lanes, conversion, exchange, gates, three rows of stores.
struct SplitLeafSmem {
    static constexpr int NG = 3;
    float red[2][4 * NG * 64 * 4];
    float sum_of[NG * HU * 2];
    float row_scale[4][16];
    int leave;
};

__device__ inline float max_across_quarters(float m)
{
    // lanes l, l ^ 16, l ^ 32, l ^ 48
    m = fmaxf(m, __shfl_xor(m, 16));
    return fmaxf(m, __shfl_xor(m, 32));
}

// Leaves [lo, hi) of the leaf list for column group cg; every workgroup keeps its slice of W_leaf.
// Stores count like loads in a wave's in-order memory counter, and a load is as late as the stores in front of it.  The results of
// a block are therefore stored without branches (what is not to be stored goes beyond the end of its table and is dropped):
// the compiler then knows how many stores lie behind the rows it waits for, and waits for none of them.
template <int S, bool KEEP>
__device__ inline void split_leaves(SplitLeafSmem &sm, const Fwd &f, int lo, int hi, int cg, const SplitWeights<3, S> &w)
{
    constexpr int NG = 3;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int H = f.H, E = f.E;
    const int hu = cg * HU + (lane & 15);
    const bool hu_ok = hu < H;
    const unsigned row_b = (unsigned)H * 4u, hu_b = (unsigned)(hu_ok ? hu : 0) * 4u, hx_row_b = (unsigned)f.hx_steps * 128u, emb_row_b = (unsigned)E * 4u;
    const __amdgpu_buffer_rsrc_t rs_h = buf_of(f.h, (unsigned long long)f.n_nodes * H * 4), rs_c = buf_of(f.c, (unsigned long long)f.n_nodes * H * 4),
                                 rs_x = buf_of(f.hx, (unsigned long long)f.n_nodes * hx_row_b),
                                 rs_e = buf_of(f.emb, (unsigned long long)f.vocab * emb_row_b);
    const int k0 = wave * S * 32 + 8 * (lane >> 4);             // this lane's first k of step 0
    const bool whole = (wave + 1) * S * 32 <= E;                // no step of this wave reaches beyond the row
    uintx4_t rows[S][2];
    auto request = [&](int word) {
        const unsigned base = __umul24((unsigned)word, emb_row_b);
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int k = k0 + 32 * s + 4 * t;
                rows[s][t] = __builtin_amdgcn_raw_buffer_load_b128(rs_e, (int)(base + 4u * (unsigned)min(k, E)), 0, 0);
            }
    };
    const int n_blocks = (hi - lo + 15) >> 4;
    if (n_blocks <= 0) return;
    // node of row l & 15 three blocks ahead, its word two, its values one
    auto node_of = [&](int b) { return f.leaf_list[min(lo + b * 16 + (lane & 15), hi - 1)]; };
    int node0 = node_of(0), node1 = node_of(1), node2 = node_of(2);
    int word1 = f.word[node1];
    request(f.word[node0]);
    for (int b = 0; b < n_blocks; ++b) {
        const int node3 = node_of(b + 3), word2 = f.word[node2];
        float x[S][8], m = 0.f;
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                float v = __uint_as_float(rows[s][i >> 2][i & 3]);
                if (!whole && k0 + 32 * s + i >= E) v = 0.f;
                x[s][i] = v;
                m = fmaxf(m, fabsf(v));
            }
        request(word1);                                         // (behind the last block: the last leaf's row again)
        m = max_across_quarters(m);
        const unsigned eb = max(__float_as_uint(m) >> 23, 15u);
        const float scale = __uint_as_float((268u - eb) << 23), back = __uint_as_float((eb - 14u) << 23);
        if (lane < 16) sm.row_scale[wave][lane] = back;
        floatx4 acc[NG];
#pragma unroll
        for (int g = 0; g < NG; ++g) acc[g] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < S; ++s) {
            halfx8 vh, vl;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float v = x[s][i] * scale;
                vh[i] = (_Float16)v;
                vl[i] = (_Float16)(v - (float)vh[i]);
            }
#pragma unroll
            for (int g = 0; g < NG; ++g) acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vh, w.hi[s][g], acc[g], 0, 0, 0);
#pragma unroll
            for (int g = 0; g < NG; ++g) acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vh, w.lo[s][g], acc[g], 0, 0, 0);
#pragma unroll
            for (int g = 0; g < NG; ++g) acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vl, w.hi[s][g], acc[g], 0, 0, 0);
        }
        float *red = sm.red[b & 1];
        const floatx4 r4 = *reinterpret_cast<const floatx4 *>(&sm.row_scale[wave][4 * (lane >> 4)]);    // this wave's own writes
#pragma unroll
        for (int g = 0; g < NG; ++g) *reinterpret_cast<floatx4 *>(&red[((wave * NG + g) * 64 + lane) * 4]) = acc[g] * r4;
        const int fin_row = 4 * wave + (lane >> 4);
        const int node = __shfl(node0, fin_row);
        __syncthreads();
        float gate[NG];
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const float *sb = &sm.sum_of[(g * HU + (lane & 15)) * 2];
            float p[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) p[k] = red[((k * NG + g) * 64 + 16 * wave + (lane & 15)) * 4 + (lane >> 4)];
            gate[g] = __builtin_fmaf(((p[0] + p[1]) + p[2]) + p[3], sb[0], sb[1]);
        }
        const bool again = !__builtin_isfinite(gate[0] + gate[1] + gate[2]);
        if (__builtin_expect(__ballot(again) != 0ull, 0)) {
            if (again) {
                const float *xr = f.emb + (size_t)f.word[node] * E, *wr = f.xl.w + (hu_ok ? hu : 0);
#pragma unroll
                for (int g = 0; g < NG; ++g) gate[g] = 0.f;
                for (int k = 0; k < E; ++k)
#pragma unroll
                    for (int g = 0; g < NG; ++g) gate[g] = __builtin_fmaf(xr[k], wr[(size_t)k * (NG * H) + (size_t)g * H], gate[g]);
#pragma unroll
                for (int g = 0; g < NG; ++g) gate[g] += sm.sum_of[(g * HU + (lane & 15)) * 2 + 1];
            }
            __builtin_amdgcn_s_waitcnt(0);
        }
        const bool here = lo + b * 16 + fin_row < hi, ok = here && hu_ok;
        float cc, hh;
        lstm_leaf_out(gate[0], gate[1], gate[2], &cc, &hh, KEEP ? Keep{ok ? f.keep0 + ((size_t)node * H + hu) : f.keep0 - HU + (lane & 15), nullptr, 0} : Keep());
        const unsigned o = ok ? __umul24((unsigned)node, row_b) + hu_b : ~0u;
        const unsigned word = split_word(hu_ok ? hh * SPLIT_H_SCALE : 0.f, hu);
        buf_st_f<false>(rs_c, o, cc);
        buf_st_f<false>(rs_h, o, hh);
        // (without a split copy its table has no bytes and the store is dropped)
        buf_st_f<false>(rs_x, here && (hu & ~1) < H ? __umul24((unsigned)node, hx_row_b) + split_word_off(hu) : ~0u, __uint_as_float(word));
        node0 = node1;
        node1 = node2;
        node2 = node3;
        word1 = word2;
    }
}

}  // namespace tl
