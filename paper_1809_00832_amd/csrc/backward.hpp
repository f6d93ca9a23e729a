// Backward pass of the TreeLSTM forward (Section 4.2.2, recursive backpropagation): the gradient
// of a node's cell is applied to the node, then to its children, with the forward values of each
// node found by node index in the h / c rows.  TreeLSTM from kept activations and TreeRNN at H <= 512 have a form of their own (back_flow.hpp), RNTN at d <= 96 another
// (k_backward_rntn below); here are the weight gradients of all, and what the rest takes: heights walked from the roots down (a parent
// is always higher than its children), one pair of launches per height, or all of them in one kernel (k_backward_heights):
//   1. gate gradients: the forward contraction G = [h_l ; h_r] U + b is recomputed with the
//      streaming cell, and its epilogue turns (dh, dc, c, c_l, c_r, gates) into the gradient of
//      the five gate pre-activations (a row of 5H values per node, kept by list position) and
//      sends dc to the children; if the forward kept its gate activations, an elementwise
//      kernel does the same from those, without the contraction;
//   2. operand gradient: [dh_l ; dh_r] += dG U^T, the same streaming cell with the rows of dG as
//      the gathered operand and U^T as the packed weights; its epilogue adds the result to the
//      children's dh rows (every node has one parent, so plain read-modify-write).
// Leaves likewise (dG W_x^T gives the gradient of each leaf's embedding row).  The weight
// gradients dU = sum_n a_n^T dG_n, dW_x = sum_n x_n^T dG_n are two contractions over all nodes at
// the end (k_weight_grad), which also sums the columns of the dG rows it passes over (bias
// gradients).
#pragma once

#include "cell_tile.hpp"
#include "schedulers.hpp"

namespace tl {

// COH: the rows of dh that the operand gradient adds to are read by other workgroups of the same kernel (the
// persistent form below): device-scope accesses, as in the forward's persistent kernels.
template <int EPI, int NG, bool COH>
__device__ inline void bwd_epilogue(const TileSmem &sm, const Fwd &f, const Gemm &gm, const floatx4 (&acc)[NG], int rb,
                                    int count, int cg, int lane)
{
    const int col = cg * HU + (lane & 15);
    const int H = f.H;
    if constexpr (EPI == EPI_BWD_INNER_GATES || EPI == EPI_BWD_LEAF_GATES) {
        if (col >= H) return;
        float bias[NG];
#pragma unroll
        for (int g = 0; g < NG; ++g) bias[g] = gm.bp[(cg * NG + g) * HU + (lane & 15)];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = rb * 16 + (lane >> 4) * 4 + v;
            if (row >= count) continue;
            const int node = sm.node[row];
            if (node < 0) continue;
            const size_t o = (size_t)node * H + col;
            const float t = tanh_f(f.c[o]);
            const float dh = f.dh[o], dc = f.dc[o];
            float *dg = f.dg + (size_t)(sm.cmd[3] + row) * (NG * H) + col;
            if constexpr (EPI == EPI_BWD_INNER_GATES) {
                const int l = sm.src0[row], r = sm.src1[row];
                const float cl = f.c[(size_t)l * H + col], cr = f.c[(size_t)r * H + col];
                const float i = sigmoid_f(acc[0][v] + bias[0]), fl = sigmoid_f(acc[1][v] + bias[1]);
                const float fr = sigmoid_f(acc[2][v] + bias[2]), og = sigmoid_f(acc[3][v] + bias[3]);
                const float u = tanh_f(acc[4][v] + bias[4]);
                const float dct = dc + dh * og * (1.f - t * t);
                dg[0] = dct * u * i * (1.f - i);
                dg[H] = dct * cl * fl * (1.f - fl);
                dg[2 * H] = dct * cr * fr * (1.f - fr);
                dg[3 * H] = dh * t * og * (1.f - og);
                dg[4 * H] = dct * i * (1.f - u * u);
                f.dc[(size_t)l * H + col] = dct * fl;
                f.dc[(size_t)r * H + col] = dct * fr;
            } else {
                const float i = sigmoid_f(acc[0][v] + bias[0]), og = sigmoid_f(acc[1][v] + bias[1]);
                const float u = tanh_f(acc[2][v] + bias[2]);
                const float dct = dc + dh * og * (1.f - t * t);
                dg[0] = dct * u * i * (1.f - i);
                dg[H] = dh * t * og * (1.f - og);
                dg[2 * H] = dct * i * (1.f - u * u);
            }
        }
    } else {
        // operand gradient: the NG blocks of output columns of this column group start at g * (out_cols / NG)
        constexpr bool INNER = EPI == EPI_BWD_INNER_OPERAND || EPI == EPI_BWD_INNER_OPERAND4;
        const int block = f.out_cols / NG;
        if (col >= block) return;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = rb * 16 + (lane >> 4) * 4 + v;
            if (row >= count) continue;
            const int node = sm.node[row];
            if (node < 0) continue;
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                const int oc = g * block + col;
                if constexpr (INNER) {
                    const int child = oc < H ? f.left[node] : f.right[node];
                    float *p = f.dh + (size_t)child * H + (oc < H ? oc : oc - H);
                    // one contribution per element (a node has one parent): inside a persistent kernel it is added at the memory side
                    if constexpr (COH) (void)add_dev(p, acc[g][v]);
                    else *p += acc[g][v];
                } else {
                    f.d_x[(size_t)node * f.E + oc] = acc[g][v];
                }
            }
        }
    }
}

// Gate gradients from what the forward kept (Fwd::keep0, keep1): the elementwise part of bwd_epilogue without the
// contraction in front of it.  One thread per (row of `list`, group of V hidden units); same outputs as the EPI_BWD_*_GATES
// epilogues (dg rows by list position from pos0 on, dc of the children).
// (COH: dh, dc and dg are exchanged between workgroups of one kernel, see the persistent form below.)
template <bool INNER, int V, bool COH>
__device__ inline void gate_grad_kept_rows(const Fwd &f, const int32_t *__restrict__ list, int n_rows, int pos0, long long first,
                                           long long stride)
{
    const int H = f.H, per_row = H / V;
    const int NG = INNER ? 5 : 3;
    const long long total = (long long)n_rows * per_row;
    for (long long e = first; e < total; e += stride) {
        const int row = (int)(e / per_row), col = (int)(e - (long long)row * per_row) * V;
        const int node = list[row];
        const size_t o = (size_t)node * H + col;
        float *dg = f.dg + (size_t)(pos0 + row) * (NG * H) + col;
        int l = 0, r = 0;
        if (INNER) { l = f.left[node]; r = f.right[node]; }
        float dh[V], dc[V], out[5][V], dcl[V], dcr[V];
        floatx4 k0[V], k1[V];
        auto load_x = [&](float (&dst)[V], const float *src) {      // what another workgroup may have written
            if constexpr (V == 4) { const floatx4 t = ld_f4<COH>(src); dst[0] = t.x; dst[1] = t.y; dst[2] = t.z; dst[3] = t.w; }
            else dst[0] = ld_f<COH>(src);
        };
        auto store = [&](float *dst, const float (&src)[V]) {       // ... and what another one will read
            if constexpr (V == 4 && COH) {
                st_dev(reinterpret_cast<unsigned long long *>(dst), pack2(__float_as_uint(src[0]), __float_as_uint(src[1])));
                st_dev(reinterpret_cast<unsigned long long *>(dst) + 1, pack2(__float_as_uint(src[2]), __float_as_uint(src[3])));
            } else if constexpr (V == 4) {
                *reinterpret_cast<floatx4 *>(dst) = floatx4{src[0], src[1], src[2], src[3]};
            } else {
                st_f<COH>(dst, src[0]);
            }
        };
        load_x(dh, f.dh + o); load_x(dc, f.dc + o);
#pragma unroll
        for (int v = 0; v < V; ++v) {
            k0[v] = f.keep0[o + v];
            if (INNER) k1[v] = f.keep1[o + v];
        }
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const float dct = __builtin_fmaf(dh[v], k0[v][0], dc[v]), d_i = dct * k0[v][1], d_o = dh[v] * k0[v][2], d_u = dct * k0[v][3];
            out[0][v] = d_i;
            out[1][v] = INNER ? dct * k1[v][0] : d_o;
            out[2][v] = INNER ? dct * k1[v][1] : d_u;
            out[3][v] = d_o;
            out[4][v] = d_u;
            dcl[v] = INNER ? dct * k1[v][2] : 0.f;
            dcr[v] = INNER ? dct * k1[v][3] : 0.f;
        }
#pragma unroll
        for (int q = 0; q < NG; ++q) store(dg + (size_t)q * H, out[q]);
        if (INNER) { store(f.dc + (size_t)l * H + col, dcl); store(f.dc + (size_t)r * H + col, dcr); }
    }
}
template <bool INNER, int V>
__global__ __launch_bounds__(256) void k_gate_grad_kept(Fwd f, const int32_t *__restrict__ list, int n_rows, int pos0)
{
    if (batch_rejected(f)) return;                            // (the lists of a malformed batch are not complete)
    gate_grad_kept_rows<INNER, V, false>(f, list, n_rows, pos0, (long long)blockIdx.x * blockDim.x + threadIdx.x,
                                         (long long)gridDim.x * blockDim.x);
}

// TreeRNN (h = tanh(a W + b), leaves h = x): the gradient of the pre-activation needs only the stored h,
// dpre = dh (1 - h^2), one row of H values per listed node (by list position from pos0 on).
template <int V, bool COH>
__device__ inline void rnn_gate_grad_rows(const Fwd &f, const int32_t *__restrict__ list, int n_rows, int pos0, long long first,
                                          long long stride)
{
    const int H = f.H, per_row = H / V;
    const long long total = (long long)n_rows * per_row;
    for (long long e = first; e < total; e += stride) {
        const int row = (int)(e / per_row), col = (int)(e - (long long)row * per_row) * V;
        const size_t o = (size_t)list[row] * H + col;
        float *dg = f.dg + (size_t)(pos0 + row) * H + col;
        if constexpr (V == 4) {
            const floatx4 hv = *reinterpret_cast<const floatx4 *>(f.h + o), dh = ld_f4<COH>(f.dh + o);
            const floatx4 out = {dh.x * (1.f - hv.x * hv.x), dh.y * (1.f - hv.y * hv.y), dh.z * (1.f - hv.z * hv.z),
                                 dh.w * (1.f - hv.w * hv.w)};
            if constexpr (COH) {
                st_dev(reinterpret_cast<unsigned long long *>(dg), pack2(__float_as_uint(out.x), __float_as_uint(out.y)));
                st_dev(reinterpret_cast<unsigned long long *>(dg) + 1, pack2(__float_as_uint(out.z), __float_as_uint(out.w)));
            } else {
                *reinterpret_cast<floatx4 *>(dg) = out;
            }
        } else {
            const float hv = f.h[o];
            st_f<COH>(dg, ld_f<COH>(f.dh + o) * (1.f - hv * hv));
        }
    }
}
template <int V>
__global__ __launch_bounds__(256) void k_rnn_gate_grad(Fwd f, const int32_t *__restrict__ list, int n_rows, int pos0)
{
    rnn_gate_grad_rows<V, false>(f, list, n_rows, pos0, (long long)blockIdx.x * blockDim.x + threadIdx.x,
                                 (long long)gridDim.x * blockDim.x);
}

// TreeRNN leaves: the embedding row is the state itself, so its gradient is the row of dh.
__global__ void k_rnn_leaf_grad(Fwd f)
{
    if (batch_rejected(f)) return;                            // (its leaf list is not complete)
    const size_t total = (size_t)f.n_leaf * f.H;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x) {
        const int i = (int)(e / f.H), j = (int)(e - (size_t)i * f.H);
        const size_t o = (size_t)f.leaf_list[i] * f.H + j;
        f.d_x[o] = f.dh[o];
    }
}

// ---- RNTN (h_k = tanh(a^T V_k a + (a W)_k + b_k)) -----------------------------------------------
// With dz = dh (1 - h^2) and the row y = [ dz_k a_q for all (k, q) | dz ] of length d * 2d + d per node, both
// gradients are ordinary contractions that the kernels above already do:
//   da = y S          S[(k, q)][p] = V[k][p][q] + V[k][q][p],  S[d * 2d + k][p] = W[p][k]       (operand gradient)
//   sum_n a_n^T y_n   gives dV (as [p][(k, q)]) and dW (the last d columns), its column sums db   (weight gradient)
// k_rntn_build_s makes S from the parameters, k_rntn_rows the rows y of the listed nodes, k_rntn_unpack puts the
// weight-gradient contraction back into the layouts of V, W and b.
__global__ void k_rntn_build_s(const float *__restrict__ v, const float *__restrict__ w, float *__restrict__ s, int d)
{
    const int D2 = 2 * d;
    const size_t total = ((size_t)d * D2 + d) * D2;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x) {
        const int p = (int)(e % D2);
        const size_t r = e / D2;
        if (r < (size_t)d * D2) {
            const int k = (int)(r / D2), q = (int)(r - (size_t)k * D2);
            s[e] = v[((size_t)k * D2 + p) * D2 + q] + v[((size_t)k * D2 + q) * D2 + p];
        } else {
            const int k = (int)(r - (size_t)d * D2);
            s[e] = w[(size_t)p * d + k];
        }
    }
}

__global__ __launch_bounds__(256) void k_rntn_rows(Fwd f, const int32_t *__restrict__ list, int n_rows, int pos0)
{
    const int d = f.H, D2 = 2 * d;
    const int L = d * D2 + d;
    const long long total = (long long)n_rows * L;
    for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (long long)gridDim.x * blockDim.x) {
        const int row = (int)(e / L), j = (int)(e - (long long)row * L);
        const int node = list[row];
        const int k = j < d * D2 ? j / D2 : j - d * D2;
        const float hv = f.h[(size_t)node * d + k];
        const float dz = f.dh[(size_t)node * d + k] * (1.f - hv * hv);
        float y = dz;
        if (j < d * D2) {
            const int q = j - k * D2;
            const int child = q < d ? f.left[node] : f.right[node];
            y = dz * f.h[(size_t)child * d + (q < d ? q : q - d)];
        }
        f.dg[(size_t)(pos0 + row) * L + j] = y;
    }
}

// acc [2d x (d * 2d + d)] = sum_n a_n^T y_n, colsum [d * 2d + d] = sum_n y_n  ->  d_v [d][2d][2d], d_w [2d][d], d_b [d].  upper: of the symmetric part
// only p <= q has been computed (else it is not read that way: half of the reads go down columns, d = 128 27 -> 50 us).
__global__ void k_rntn_unpack(const float *__restrict__ acc, const float *__restrict__ colsum, float *__restrict__ d_v,
                              float *__restrict__ d_w, float *__restrict__ d_b, int d, int upper)
{
    const int D2 = 2 * d, L = d * D2 + d;
    const size_t n_v = (size_t)d * D2 * D2, total = n_v + (size_t)D2 * d + d;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x) {
        if (e < n_v) {
            const int q = (int)(e % D2), p = (int)((e / D2) % D2), k = (int)(e / ((size_t)D2 * D2));
            const bool turn = upper && p > q;
            d_v[e] = acc[(size_t)(turn ? q : p) * L + (size_t)k * D2 + (turn ? p : q)];
        } else if (e < n_v + (size_t)D2 * d) {
            const size_t r = e - n_v;
            const int k = (int)(r % d), p = (int)(r / d);
            d_w[r] = acc[(size_t)p * L + (size_t)d * D2 + k];
        } else {
            const int k = (int)(e - n_v - (size_t)D2 * d);
            d_b[k] = colsum[(size_t)d * D2 + k];
        }
    }
}

// out[r][c] = in[c][r] for a row-major [rows x cols] input
__global__ void k_transpose(const float *__restrict__ in, float *__restrict__ out, int rows, int cols)
{
    const size_t total = (size_t)rows * cols;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x) {
        const size_t c = e / rows, r = e - c * rows;          // e indexes the output [cols x rows]
        out[e] = in[r * cols + c];
    }
}

// Weight gradient: out[k][j] += sum_q a_q[k] * dg[q][j] over the n_rows nodes of `list` (dg rows by
// list position; ld > 0: by node, ld values apart), a_q = [h[left]; h[right]] (SEG 2, L = H) or the embedding row of the leaf's
// word (SEG 1, L = E).  K_out = SEG * L rows, n_cols columns, row-major; `out` is zero beforehand.
// Two kernels; wg_plan() says which, and why the line lies where it does.  Both cut the node axis into slices (blockIdx.z; the
// slices' partial tiles are added with atomics: the node axis is long and the output small, so without
// slices there are too few workgroups to hide the latency of the gathers).
//
// The one for small outputs and few nodes: one workgroup per 64 x 64 tile of the output and slice, wave w on the
// 32 x 32 quarter (w / 2, w % 2).  The contraction runs over the nodes, 16 at a time through LDS,
// on v_mfma_f32_16x16x4_f32 with the node index as the k of the instruction; the next 16 nodes'
// operands are requested into registers before the current ones are multiplied.
constexpr int WN_TILE = 64, WN_Q = 16, WN_LD = WN_TILE + 4;

// RNTN: the rows contracted with are y = [dz_k a_q for all (k, q) | dz] (see k_rntn_rows), made from dz (d values a node) and the children's rows
// where they are needed: column j is (k, q), its value dz[k] times element q of [h_left ; h_right].
struct RntnY {
    int k, seg, in;         // seg < 0: a column of dz itself
};
__device__ inline RntnY rntn_y(int j, int d)
{
    const int k = j / (2 * d), q = j - k * 2 * d;
    if (k >= d) return RntnY{j - 2 * d * d, -1, 0};
    return RntnY{k, q >= d ? 1 : 0, q >= d ? q - d : q};
}

struct WnSmem {
    float as[2][WN_Q][WN_LD], bs[2][WN_Q][WN_LD];               // two buffers each: a step's operands are parked while the
};                                                              // step before is still being multiplied (one barrier per step)
template <int SEG, bool VEC4, bool RNTN>
__device__ __forceinline__ void weight_grad_tile(WnSmem &sm, int bx, int by, int bz, int nz, const Fwd &f, const int32_t *__restrict__ list, int n_rows,
                                                 const float *__restrict__ table, int L, const float *__restrict__ dg, int ld, int n_cols,
                                                 float *__restrict__ out, float *__restrict__ bias_out)
{
    auto &as = sm.as, &bs = sm.bs;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int k0 = bx * WN_TILE, j0 = by * WN_TILE;
    const int K_out = SEG * L;
    const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;
    const int per = ((n_rows + nz - 1) / nz + WN_Q - 1) / WN_Q * WN_Q;
    const int q_lo = bz * per, q_hi = min(n_rows, q_lo + per);
    if (q_lo >= q_hi) return;
    floatx4 acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
    const int lq = tid >> 4, lk = (tid & 15) * 4;             // this thread stages 4 consecutive columns of row lq
    float ra[4], rb[4];
    // the workgroups of the first row of output tiles also sum the columns of dg they pass over (bias gradient)
    const bool with_bias = bias_out != nullptr && bx == 0;
    float bsum[4] = {0.f, 0.f, 0.f, 0.f};
    // The operands of a step (16 nodes) hang on a chain of three loads: the node from the list, its source rows from
    // the child (or word) arrays, the data from those rows.  A step has only 16 MFMAs per wave to hide it, so the chain
    // is spread over three steps: step i requests the data of step i + 1, the source rows of step i + 2 and the node
    // of step i + 3, each from what the step before has requested.
    auto node_of = [&](int q0) {                              // stage 1
        const int q = q0 + lq;
        return q < q_hi ? list[q] : -1;
    };
    auto sources_of = [&](int node, int *s0, int *s1) {       // stage 2
        *s0 = *s1 = 0;
        if (node >= 0) {
            if (SEG == 2) { *s0 = f.left[node]; *s1 = f.right[node]; } else { *s0 = f.word[node]; }
        }
    };
    auto request = [&](int q0, int node, int s0, int s1) {    // stage 3: operands of nodes q0 .. q0 + 15 into registers
        const bool live = node >= 0;
        const float *dg_row = ld > 0 ? dg + (size_t)max(node, 0) * ld : dg + (size_t)(q0 + lq) * (RNTN ? L : n_cols);
        if constexpr (VEC4) {      // L and n_cols multiples of 4, rows 16-byte aligned: 4 consecutive columns never leave a segment
            const int k = k0 + lk, j = j0 + lk;
            const int seg = (SEG == 2 && k >= L) ? 1 : 0;
            floatx4 a = floatx4{0.f, 0.f, 0.f, 0.f}, b = a;
            if (live && k < K_out) a = *reinterpret_cast<const floatx4 *>(table + (size_t)(seg ? s1 : s0) * L + (k - seg * L));
            if constexpr (RNTN) {                               // (four neighbouring columns of one k, or of dz)
                if (live && j < n_cols) {
                    const RntnY y = rntn_y(j, L);
                    const float *z = dg_row + y.k;
                    if (y.seg < 0) b = *reinterpret_cast<const floatx4 *>(z);
                    else b = *reinterpret_cast<const floatx4 *>(table + (size_t)(y.seg ? s1 : s0) * L + y.in) * *z;
                }
            } else if (live && j < n_cols) {
                b = *reinterpret_cast<const floatx4 *>(dg_row + j);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) { ra[e] = a[e]; rb[e] = b[e]; }
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int k = k0 + lk + e, j = j0 + lk + e;
                const int seg = (SEG == 2 && k >= L) ? 1 : 0;
                ra[e] = (live && k < K_out) ? table[(size_t)(seg ? s1 : s0) * L + (k - seg * L)] : 0.f;
                if constexpr (RNTN) {
                    rb[e] = 0.f;
                    if (live && j < n_cols) {
                        const RntnY y = rntn_y(j, L);
                        rb[e] = dg_row[y.k];
                        if (y.seg >= 0) rb[e] *= table[(size_t)(y.seg ? s1 : s0) * L + y.in];
                    }
                } else {
                    rb[e] = (live && j < n_cols) ? dg_row[j] : 0.f;
                }
            }
        }
    };
    int node1 = node_of(q_lo), s0_1, s1_1;                    // step q_lo: all three stages at once
    sources_of(node1, &s0_1, &s1_1);
    request(q_lo, node1, s0_1, s1_1);
    node1 = node_of(q_lo + WN_Q);                             // step q_lo + 16: node and source rows
    sources_of(node1, &s0_1, &s1_1);
    int node2 = node_of(q_lo + 2 * WN_Q);                     // step q_lo + 32: node
    auto park = [&](int buf) {
        *reinterpret_cast<floatx4 *>(&as[buf][lq][lk]) = floatx4{ra[0], ra[1], ra[2], ra[3]};
        *reinterpret_cast<floatx4 *>(&bs[buf][lq][lk]) = floatx4{rb[0], rb[1], rb[2], rb[3]};
        if (with_bias) {
#pragma unroll
            for (int e = 0; e < 4; ++e) bsum[e] += rb[e];
        }
    };
    park(0);
    __syncthreads();
    int buf = 0;
    for (int q0 = q_lo; q0 < q_hi; q0 += WN_Q) {
        request(q0 + WN_Q, node1, s0_1, s1_1);                // (beyond the end: node -1, nothing is loaded)
        node1 = node2;
        sources_of(node1, &s0_1, &s1_1);
        node2 = node_of(q0 + 3 * WN_Q);
#pragma unroll
        for (int kk = 0; kk < WN_Q / 4; ++kk) {
            const int qq = kk * 4 + (lane >> 4);
            float a[2], b[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                a[t] = as[buf][qq][wr + t * 16 + (lane & 15)];
                b[t] = bs[buf][qq][wc + t * 16 + (lane & 15)];
            }
#pragma unroll
            for (int ta = 0; ta < 2; ++ta)
#pragma unroll
                for (int tb = 0; tb < 2; ++tb)
                    acc[ta][tb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[ta], b[tb], acc[ta][tb], 0, 0, 0);
        }
        // the other buffer was read in the step before this one, and every wave has passed the barrier since
        if (q0 + WN_Q < q_hi) park(buf ^ 1);
        __syncthreads();
        buf ^= 1;
    }
#pragma unroll
    for (int ta = 0; ta < 2; ++ta)
#pragma unroll
        for (int tb = 0; tb < 2; ++tb)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int k = k0 + wr + ta * 16 + (lane >> 4) * 4 + v, j = j0 + wc + tb * 16 + (lane & 15);
                if (k < K_out && j < n_cols) atomicAdd(&out[(size_t)k * n_cols + j], acc[ta][tb][v]);
            }
    if (with_bias) {                                          // uniform per workgroup; the loop ended with a barrier
        *reinterpret_cast<floatx4 *>(&bs[0][lq][lk]) = floatx4{bsum[0], bsum[1], bsum[2], bsum[3]};
        __syncthreads();
        if (tid < WN_TILE && j0 + tid < n_cols) {
            float t = 0.f;
#pragma unroll
            for (int q = 0; q < WN_Q; ++q) t += bs[0][q][tid];
            atomicAdd(&bias_out[j0 + tid], t);
        }
    }
}

template <int SEG, bool VEC4, bool RNTN = false>
__global__ __launch_bounds__(256) void k_weight_grad(Fwd f, const int32_t *__restrict__ list, int n_rows, const float *__restrict__ table, int L,
                                                     const float *__restrict__ dg, int ld, int n_cols, float *__restrict__ out, float *__restrict__ bias_out)
{
    if (batch_rejected(f)) return;                            // (the lists of a malformed batch are not complete)
    __shared__ __align__(16) WnSmem sm;
    weight_grad_tile<SEG, VEC4, RNTN>(sm, blockIdx.x, blockIdx.y, blockIdx.z, gridDim.z, f, list, n_rows, table, L, dg, ld, n_cols, out, bias_out);
}

// The one for large outputs and many nodes: one workgroup per 128 x 128 tile of the output and slice, wave w on the
// 64 x 64 quarter (w / 2, w % 2).
// The contraction runs over the nodes on the 16-bit matrix unit with fp32 operands: a value is the sum of three bf16 terms
// (8 bits each and the range of fp32, so gradients of any magnitude need no scaling), and of the nine products the six
// that reach 2^-24 of the whole are taken, accumulated in fp32: 6/16 of the fp32 instruction's time, beside which vector
// instructions run.
// An infinity has no such terms (x - hi is a NaN), a finite value above the largest bf16 number rounds to one, and below 2^-109
// the last term runs out of exponents.  A wave that ends with a sum that is not finite, or is below 2^-100 and not zero, therefore takes
// its sums again with fp32 instructions (wg_sums_again): what comes out is what those give.  (In a larger sum a
// value below 2^-109 is off by 2^-134 at most.)
// A thread loads one column of 16 of a step's 32 nodes (a wave: 256 consecutive bytes a row), splits them and parks each term's
// eight neighbours as the 16 bytes that are an operand of v_mfma_f32_16x16x32_bf16; the next 32 nodes' values are
// requested before the current ones are multiplied.  Bound by the reads of the rows, each of which goes to every
// tile: hence the tile of 128.
constexpr int WG_TILE = 128, WG_Q = 32, WG_LD = WG_Q + 8, WG_SRC = 512;

// Which of the two kernels, and its grid.  A workgroup of the wide form starts with a longer chain (source rows, 64 KB of LDS,
// no second buffer), ends with four times the atomics, and does the products of a whole tile wherever the output ends; per
// product it needs half the reads and 6/16 of the matrix time.
// Slices of the wide form: two workgroups are resident per CU, so the grid is a number of whole rounds of 2 n_cu or of half a round (one per CU:
// 0.72 of a full round's time), whichever is shortest when a workgroup costs its nodes and 256 more for its start and its atomics.
// Measured (profiler, 1 / 2 / 3 / 4 / 6 / 7 slices, U of TreeLSTM at H = 512 and 6 772 nodes, 160 tiles): 454, 313, 236, 287, 261, 271 us;
// four workgroups per CU in all, rounded up, were 7 slices, a third round for the last 96 of 1 120 workgroups.
// RNTN takes two rounds at least: a tile's sums are one chain there, whose error grows with the nodes of a slice (d = 64, 6 772 nodes, error of d_u
// against 64 bits: 1.00e-6 with 7 slices, 0.96e-6 with 15; 106 and 108 us).
// The 64 x 64 form where slices of 64 nodes don't give every CU a workgroup of the wide one.  Measured on 73 outputs and node counts (TreeLSTM H = 32 ...
// 700, TreeRNN d = 64 ... 512, RNTN d = 16 ... 96; 25 to 1 000 trees of 5 to 50 leaves), time of the 64 x 64 form over that of the wide one:
//   fewer workgroups of the wide form than CUs (24)        0.59 ... 0.99
//   more (49)                                              1.00 ... 2.69
struct WgPlan {
    bool wide;
    unsigned tiles_k, tiles_j, slices;
};
inline long long wg_slices(int n_rows, int nodes) { return std::max(1ll, ((long long)n_rows + nodes - 1) / nodes); }       // of no fewer nodes
inline long long wg_tiles(WgPlan &p, int K_out, int n_cols, int tile)
{
    p.tiles_k = (unsigned)((K_out + tile - 1) / tile);
    p.tiles_j = (unsigned)((n_cols + tile - 1) / tile);
    return (long long)p.tiles_k * p.tiles_j;
}
// slices of the wide form for that many tiles, and what they cost (in nodes)
inline double wg_rounds(long long tiles, int n_rows, long long max_z, int n_cu, bool rntn, unsigned *slices)
{
    double best = 0.0;
    *slices = 0;
    for (int half = rntn ? 4 : 0; half <= 8; ++half) {                            // (0: one slice, however many tiles there are)
        const long long z = std::min(std::max((long long)half * n_cu / tiles, 1ll), max_z), halves = (tiles * z + n_cu - 1) / n_cu;
        const double rounds = (double)(halves / 2) + (halves % 2 != 0 ? 0.72 : 0.0), cost = rounds * ((double)n_rows / (double)z + 256.0);
        if (*slices == 0 || cost < best) {
            best = cost;
            *slices = (unsigned)z;
        }
    }
    return best;
}
inline void wg_small(WgPlan &p, int K_out, int n_cols, int n_rows, int n_cu)
{
    const long long small = wg_tiles(p, K_out, n_cols, WN_TILE);
    p.wide = false;
    p.slices = (unsigned)std::min((8ll * n_cu + small - 1) / small, wg_slices(n_rows, 4 * WN_Q));
}
inline WgPlan wg_plan(int K_out, int n_cols, int n_rows, int n_cu, bool rntn)
{
    WgPlan p{};
    const long long tiles = wg_tiles(p, K_out, n_cols, WG_TILE), max_z = wg_slices(n_rows, 2 * WG_Q);
    p.wide = tiles * max_z >= n_cu;
    if (p.wide) wg_rounds(tiles, n_rows, max_z, n_cu, rntn, &p.slices);
    else wg_small(p, K_out, n_cols, n_rows, n_cu);
    return p;
}
// The two gradients of TreeLSTM (U's: 2 H x 5 H over n_int nodes, W_leaf's: E x 3 H over n_leaf) in one launch: in the wide form, with the same number
// of slices, where the tiles of both fill the chip and one launch's rounds are no longer than those of two; in the 64 x 64 form where not
// even both together fill it.  Measured (profiler): 25 parse trees at H = 150 22 + 15 us apart (64 x 64), 34 in one launch of that form, 26.7 of
// the wide one; 256 at H = 512 226 + 65 us apart, which one launch's rounds would exceed.
struct WgPair {
    bool one;
    WgPlan u, w;
};
inline WgPair wg_pair(int H, int E, int n_int, int n_leaf, int n_cu)
{
    WgPair p{};
    const long long tiles_u = wg_tiles(p.u, 2 * H, 5 * H, WG_TILE), tiles_w = wg_tiles(p.w, E, 3 * H, WG_TILE);
    const long long z_u = wg_slices(n_int, 2 * WG_Q), z_w = wg_slices(n_leaf, 2 * WG_Q), max_z = std::min(z_u, z_w);
    const long long tiles = tiles_u + tiles_w;
    if (tiles * max_z >= n_cu) {
        unsigned z = 0, zu = 0, zw = 0;
        const double apart = wg_rounds(tiles_u, n_int, z_u, n_cu, false, &zu) + wg_rounds(tiles_w, n_leaf, z_w, n_cu, false, &zw);
        p.one = wg_rounds(tiles, std::max(n_int, n_leaf), max_z, n_cu, false, &z) <= apart;
        p.u.wide = p.w.wide = true;
        p.u.slices = p.w.slices = z;
    } else {
        wg_small(p.u, 2 * H, 5 * H, n_int, n_cu);
        wg_small(p.w, E, 3 * H, n_leaf, n_cu);
        p.one = tiles_u * z_u < n_cu && tiles_w * z_w < n_cu;
    }
    return p;
}

struct WgSmem {
    unsigned short a[3][WG_TILE][WG_LD], b[3][WG_TILE][WG_LD];      // [term][column][node]
    unsigned src[2][WG_SRC];                                        // source rows of the slice's next nodes, as byte offsets (BIG: row numbers)
    unsigned row[WG_SRC];                                           // ... and their rows of dg
};
constexpr unsigned WG_NOWHERE = 0xFFFF0000u;

// Eight values as three vectors of bf16 terms, parked as [term][.. 8 neighbours ..].
__device__ inline void wg_park(unsigned short (*dst)[WG_TILE][WG_LD], int col, int q, const float *x)
{
    bf16x8 hi, mid, lo;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        hi[i] = (__bf16)x[i];
        const float r = x[i] - (float)hi[i];
        mid[i] = (__bf16)r;
        lo[i] = (__bf16)(r - (float)mid[i]);
    }
    *reinterpret_cast<bf16x8 *>(&dst[0][col][q]) = hi;
    *reinterpret_cast<bf16x8 *>(&dst[1][col][q]) = mid;
    *reinterpret_cast<bf16x8 *>(&dst[2][col][q]) = lo;
}

// The sums of a wave's 64 x 64 quarter at (k0, j0) over nodes [q_lo, q_hi) with fp32 instructions, straight from memory (rare, and
// slow: every four nodes are a chain of three loads).
template <int SEG, bool RNTN>
__device__ __forceinline__ void wg_sums_again(const Fwd &f, const int32_t *list, const float *table, int L, const float *dg, int n_cols, int k0,
                                                        int j0, int q_lo, int q_hi, int ld, floatx4 (&acc)[4][4])
{
    const int lane = threadIdx.x & 63, K_out = SEG * L;
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int q0 = q_lo; q0 < q_hi; q0 += 4) {
        const bool live = q0 + (lane >> 4) < q_hi;
        const int q = live ? q0 + (lane >> 4) : q_hi - 1, node = list[q];
        const int s0 = SEG == 2 ? f.left[node] : f.word[node], s1 = SEG == 2 ? f.right[node] : 0;
        const float *dg_row = ld > 0 ? dg + (size_t)node * ld : dg + (size_t)q * (RNTN ? L : n_cols);
        float a[4], b[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int k = min(k0 + t * (RNTN ? 32 : 16) + (lane & 15), K_out - 1), j = min(j0 + t * (RNTN ? 32 : 16) + (lane & 15), n_cols - 1);
            const bool second = SEG == 2 && k >= L;
            a[t] = live ? table[(size_t)(second ? s1 : s0) * L + (second ? k - L : k)] : 0.f;
            if constexpr (RNTN) {
                const RntnY y = rntn_y(j, L);
                b[t] = live ? dg_row[y.k] : 0.f;
                if (live && y.seg >= 0) b[t] *= table[(size_t)(y.seg ? s1 : s0) * L + y.in];
            } else {
                b[t] = live ? dg_row[j] : 0.f;
            }
        }
#pragma unroll
        for (int ta = 0; ta < 4; ++ta)
#pragma unroll
            for (int tb = 0; tb < 4; ++tb) acc[ta][tb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[ta], b[tb], acc[ta][tb], 0, 0, 0);
    }
}

// BIG: tables of 4 GiB and more, or rows of 60 000 bytes (addresses in 64 bits: some 250 of a step's vector instructions, which the conversion leaves
// no room for; else the byte offsets of a slice's rows lie in LDS, and rows beyond its end are beyond the end of the table and read as zeros).
template <int SEG, bool RNTN, bool BIG>
__device__ __forceinline__ void weight_grad_wide_tile(WgSmem &sm, int bx, int by, int bz, int nz, const Fwd &f, const int32_t *__restrict__ list, int n_rows,
                                                      const float *__restrict__ table, int L, const float *__restrict__ dg, int ld,
                                                      int n_cols, float *__restrict__ out, float *__restrict__ bias_out, unsigned long long table_bytes,
                                                      unsigned long long dg_bytes)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int k0 = bx * WG_TILE, j0 = by * WG_TILE;
    const int K_out = SEG * L;
    // RNTN: dV is symmetric, so only tiles of 16 x 16 that hold a p <= q are computed; the tiles of the four waves are interleaved, so that
    // each has at most ten of its sixteen (36 of 64 in all).
    constexpr int TS = RNTN ? 32 : 16;                        // distance of a wave's tiles
    const int wr = (wave >> 1) * (RNTN ? 16 : 64), wc = (wave & 1) * (RNTN ? 16 : 64);
    bool live_tile[4][4];
    if constexpr (RNTN) {
#pragma unroll
        for (int tb = 0; tb < 4; ++tb) {
            const int c = j0 + wc + tb * TS, q0 = c % (2 * L);
            const int top = c + 15 >= 2 * L * L || q0 + 15 >= 2 * L ? K_out : q0 + 15;      // largest q among the columns (the linear ones: all rows)
#pragma unroll
            for (int ta = 0; ta < 4; ++ta) live_tile[ta][tb] = k0 + wr + ta * TS <= top;
        }
    }
    const int per = ((n_rows + nz - 1) / nz + WG_Q - 1) / WG_Q * WG_Q;
    const int q_lo = bz * per, q_hi = min(n_rows, q_lo + per);
    if (q_lo >= q_hi) return;
    // The five lower products have sums of their own: a step rounds a large sum once, not six times (error of dU against 64 bits, H = 512, 6 772
    // nodes: 5.7e-7 -> 5.6e-7, and 6.5e-7 without it for the nodes in the order that the lists now have).
    floatx4 acc[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
    // this thread stages column `col` of nodes half, half + 1, ... half + 15 of a step; columns beyond the matrix repeat its last one
    // (their results are not stored)
    const int col = tid & (WG_TILE - 1), half = (tid >> 7) * 16;
    const int k = min(k0 + col, K_out - 1), j = min(j0 + col, n_cols - 1);
    const int seg = (SEG == 2 && k >= L) ? 1 : 0, k_in = k - seg * L;
    const RntnY y = RNTN ? rntn_y(j, L) : RntnY{0, 0, 0};
    float ra[16], rb[16], ry[RNTN ? 16 : 1];                 // (ry: the other factor of an RNTN column)
    // the workgroups of the first row of output tiles also sum the columns of dg they pass over (bias gradient)
    const bool with_bias = bias_out != nullptr && bx == 0;
    float bsum = 0.f;
    const int n_row = ld > 0 ? ld : RNTN ? L : n_cols;
    const __amdgpu_buffer_rsrc_t rs_t = buf_of(table, BIG ? 0ull : table_bytes), rs_dg = buf_of(dg, BIG ? 0ull : dg_bytes);
    const unsigned a_off = (unsigned)k_in * 4u, b_off = (unsigned)(RNTN ? y.k : j) * 4u, y_off = (unsigned)y.in * 4u;
    auto request = [&](int q0, int chunk) {                   // operands of nodes q0 ... q0 + 31 into registers
        if constexpr (!BIG) {
            const unsigned *src = &sm.src[seg][q0 - chunk + half], *row = &sm.row[q0 - chunk + half], *src_y = &sm.src[y.seg > 0 ? 1 : 0][q0 - chunk + half];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                ra[i] = buf_ld_f<false>(rs_t, src[i] + a_off);
                rb[i] = buf_ld_f<false>(rs_dg, row[i] + b_off);
                if constexpr (RNTN) ry[i] = buf_ld_f<false>(rs_t, src_y[i] + y_off);
            }
        } else {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int q = q0 + half + i, at = min(q, q_hi - 1) - chunk;
                const bool live = q < q_hi;
                ra[i] = live ? table[(size_t)sm.src[seg][at] * L + k_in] : 0.f;
                rb[i] = live ? dg[(size_t)sm.row[at] * n_row + (RNTN ? y.k : j)] : 0.f;
                if constexpr (RNTN) ry[i] = live ? table[(size_t)sm.src[y.seg > 0 ? 1 : 0][at] * L + y.in] : 0.f;
            }
        }
    };
    for (int chunk = q_lo; chunk < q_hi; chunk += WG_SRC) {
        const int end = min(q_hi, chunk + WG_SRC);
        for (int i = tid; i < (end - chunk + WG_Q - 1) / WG_Q * WG_Q; i += 256) {
            const bool live = chunk + i < end;
            const int node = list[live ? chunk + i : end - 1];
            const unsigned unit = BIG ? 1u : (unsigned)L * 4u, row = (unsigned)(ld > 0 ? node : chunk + i) * (BIG ? 1u : (unsigned)n_row * 4u);
            sm.src[0][i] = live ? (unsigned)(SEG == 2 ? f.left[node] : f.word[node]) * unit : WG_NOWHERE;
            if (SEG == 2) sm.src[1][i] = live ? (unsigned)f.right[node] * unit : WG_NOWHERE;
            sm.row[i] = live ? row : WG_NOWHERE;
        }
        __syncthreads();
        request(chunk, chunk);
        for (int q0 = chunk; q0 < end; q0 += WG_Q) {
            if constexpr (RNTN) {                             // (here, where they are waited for anyway)
#pragma unroll
                for (int i = 0; i < 16; ++i) rb[i] *= y.seg >= 0 ? ry[i] : 1.f;
            }
            wg_park(sm.a, col, half, ra);
            wg_park(sm.a, col, half + 8, ra + 8);
            wg_park(sm.b, col, half, rb);
            wg_park(sm.b, col, half + 8, rb + 8);
            if (with_bias) {
                float pair[8];                                // (in pairs: an eighth of the roundings of a sum of one by one)
#pragma unroll
                for (int i = 0; i < 8; ++i) pair[i] = rb[i] + rb[i + 8];
                bsum += ((pair[0] + pair[4]) + (pair[2] + pair[6])) + ((pair[1] + pair[5]) + (pair[3] + pair[7]));
            }
            __syncthreads();
            if (q0 + WG_Q < end) request(q0 + WG_Q, chunk);
            bf16x8 vb[4][3];
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int m = 0; m < 3; ++m) vb[t][m] = *reinterpret_cast<const bf16x8 *>(&sm.b[m][wc + t * TS + (lane & 15)][8 * (lane >> 4)]);
#pragma unroll
            for (int ta = 0; ta < 4; ++ta) {
                bf16x8 va[3];
#pragma unroll
                for (int m = 0; m < 3; ++m) va[m] = *reinterpret_cast<const bf16x8 *>(&sm.a[m][wr + ta * TS + (lane & 15)][8 * (lane >> 4)]);
                constexpr int TERM[6][2] = {{1, 1}, {0, 2}, {2, 0}, {0, 1}, {1, 0}, {0, 0}};
                if constexpr (RNTN) {
#pragma unroll
                    for (int tb = 0; tb < 4; ++tb)
                        if (live_tile[ta][tb]) {
#pragma unroll
                            for (int p = 0; p < 6; ++p) acc[ta][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[TERM[p][0]], vb[tb][TERM[p][1]], acc[ta][tb], 0, 0, 0);
                        }
                } else {
                    // a step's products are summed from zero, smallest first, and added to the whole with one rounding to nearest (four chains of RNTN's
                    // tiles spill registers, and one by one they wait for each other: 101 -> 111 us)
                    floatx4 sum[4] = {};
#pragma unroll
                    for (int p = 0; p < 6; ++p)
#pragma unroll
                        for (int tb = 0; tb < 4; ++tb) sum[tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[TERM[p][0]], vb[tb][TERM[p][1]], sum[tb], 0, 0, 0);
#pragma unroll
                    for (int tb = 0; tb < 4; ++tb) acc[ta][tb] += sum[tb];
                }
            }
            __syncthreads();
        }
    }
    bool again = false;
#pragma unroll
    for (int ta = 0; ta < 4; ++ta)
#pragma unroll
        for (int tb = 0; tb < 4; ++tb)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float m = fabsf(acc[ta][tb][v]);
                again |= !(m == 0.f || (m >= 0x1p-100f && m < __builtin_inff()));
            }
    if (__builtin_expect(__ballot(again) != 0ull, 0)) wg_sums_again<SEG, RNTN>(f, list, table, L, dg, n_cols, k0 + wr, j0 + wc, q_lo, q_hi, ld, acc);
#pragma unroll
    for (int ta = 0; ta < 4; ++ta)
#pragma unroll
        for (int tb = 0; tb < 4; ++tb)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int ko = k0 + wr + ta * TS + (lane >> 4) * 4 + v, jo = j0 + wc + tb * TS + (lane & 15);
                if (ko < K_out && jo < n_cols && (!RNTN || live_tile[ta][tb])) atomicAdd(&out[(size_t)ko * n_cols + jo], acc[ta][tb][v]);
            }
    if (with_bias) {                                          // uniform per workgroup; the loop ended with a barrier
        float *part = reinterpret_cast<float *>(sm.src[0]);
        if (tid >= WG_TILE) part[col] = bsum;
        __syncthreads();
        if (tid < WG_TILE && j0 + col < n_cols) atomicAdd(&bias_out[j0 + col], bsum + part[col]);
    }
}

template <int SEG, bool RNTN, bool BIG>
__global__ __launch_bounds__(256, 2) void k_weight_grad_wide(Fwd f, const int32_t *__restrict__ list, int n_rows,
                                                             const float *__restrict__ table, int L, const float *__restrict__ dg, int ld,
                                                             int n_cols, float *__restrict__ out, float *__restrict__ bias_out, unsigned long long table_bytes,
                                                             unsigned long long dg_bytes)
{
    if (batch_rejected(f)) return;
    __shared__ __align__(16) WgSmem sm;
    weight_grad_wide_tile<SEG, RNTN, BIG>(sm, blockIdx.x, blockIdx.y, blockIdx.z, gridDim.z, f, list, n_rows, table, L, dg, ld, n_cols, out, bias_out, table_bytes, dg_bytes);
}

// Both gradients of TreeLSTM, U's and W_leaf's, in one launch: they need nothing of each other (WgPair says when).
struct WgradArgs {
    const int32_t *list;
    const float *table, *dg;
    float *out, *bias_out;
    int n_rows, L, n_cols, tiles_k, tiles_j, slices;
    unsigned long long table_bytes, dg_bytes;
};
template <bool VEC4>
__global__ __launch_bounds__(256) void k_weight_grad_both(Fwd f, WgradArgs u, WgradArgs w, int ld)
{
    if (batch_rejected(f)) return;
    __shared__ __align__(16) WnSmem sm;
    const int n_u = u.tiles_k * u.tiles_j * u.slices, b = (int)blockIdx.x < n_u ? (int)blockIdx.x : (int)blockIdx.x - n_u;
    if ((int)blockIdx.x < n_u) {
        const int t = b / u.tiles_k;
        weight_grad_tile<2, VEC4, false>(sm, b - t * u.tiles_k, t % u.tiles_j, t / u.tiles_j, u.slices, f, u.list, u.n_rows, u.table, u.L, u.dg, ld, u.n_cols, u.out, u.bias_out);
    } else {
        const int t = b / w.tiles_k;
        weight_grad_tile<1, VEC4, false>(sm, b - t * w.tiles_k, t % w.tiles_j, t / w.tiles_j, w.slices, f, w.list, w.n_rows, w.table, w.L, w.dg, ld, w.n_cols, w.out, w.bias_out);
    }
}
__global__ __launch_bounds__(256, 2) void k_weight_grad_wide_both(Fwd f, WgradArgs u, WgradArgs w, int ld)
{
    if (batch_rejected(f)) return;
    __shared__ __align__(16) WgSmem sm;
    const int n_u = u.tiles_k * u.tiles_j * u.slices, b = (int)blockIdx.x < n_u ? (int)blockIdx.x : (int)blockIdx.x - n_u;
    if ((int)blockIdx.x < n_u) {
        const int t = b / u.tiles_k;
        weight_grad_wide_tile<2, false, false>(sm, b - t * u.tiles_k, t % u.tiles_j, t / u.tiles_j, u.slices, f, u.list, u.n_rows, u.table, u.L, u.dg, ld, u.n_cols, u.out,
                                               u.bias_out, u.table_bytes, u.dg_bytes);
    } else {
        const int t = b / w.tiles_k;
        weight_grad_wide_tile<1, false, false>(sm, b - t * w.tiles_k, t % w.tiles_j, t / w.tiles_j, w.slices, f, w.list, w.n_rows, w.table, w.L, w.dg, ld, w.n_cols, w.out,
                                               w.bias_out, w.table_bytes, w.dg_bytes);
    }
}

// Plain stochastic gradient descent, theta <- theta - lr * g (the product rounded, then the difference: the two
// roundings of the definition written as two operations), for up to four dense arrays in one launch.
struct SgdList {
    float *theta[4];
    const float *grad[4];
    size_t n[4];
};
__global__ void k_sgd_dense(SgdList z, float lr)
{
#pragma clang fp contract(off)          // two roundings, as the definition says: no fused multiply-add here
    const size_t stride = (size_t)gridDim.x * blockDim.x;
#pragma unroll
    for (int a = 0; a < 4; ++a)
        for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < z.n[a]; e += stride) {
            const float step = lr * z.grad[a][e];
            z.theta[a][e] = z.theta[a][e] - step;
        }
}

// The embedding table: row word[n] -= lr * d_x[n] for every leaf n.  Several leaves may share a word, so the
// rows are updated with atomics (the order of those additions is not fixed).
__global__ void k_sgd_embedding(float *__restrict__ emb, const float *__restrict__ d_x, const int32_t *__restrict__ left,
                                const int32_t *__restrict__ word, int n_nodes, int E, int vocab, float lr)
{
    const size_t total = (size_t)n_nodes * E;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x) {
        const int n = (int)(e / E), j = (int)(e - (size_t)n * E);
        if (left[n] >= 0) continue;
        const int w = word[n];
        if (w < 0 || w >= vocab) continue;
        atomicAdd(&emb[(size_t)w * E + j], -(lr * d_x[e]));
    }
}

// ---- all heights in one launch ------------------------------------------------------------------
// The walk over the heights above as one persistent kernel: the per-height lists are on the device already (the
// counting sort of the structure pass), so the host needs neither the number of heights nor their sizes and
// tl_backward returns without waiting for the device.  Per height, from the roots down:
//   gate gradients   from the gate activations that the forward kept (TreeLSTM) or from h (TreeRNN), elementwise, the
//                    rows shared out over all threads of the grid
//   (grid barrier)
//   operand gradient tiles of the height's rows x column groups on the streaming cell, as in the per-height launches
//                    (four column blocks per group for heights of more than 64 rows, one otherwise)
//   (grid barrier)
// What one phase writes and the next reads on another workgroup (dg, dh, dc) goes through device-scope stores and
// loads; the barrier is the bounded one of the level scheduler.  (Gate gradients that recompute the forward
// contraction, and the RNTN cell, keep the per-height launches.)
struct BwdHeights {
    Gemm bwd4, bwd1;              // packed U^T with four column blocks per group / with one
    int ng_inner;                 // 4: both forms exist, 1: only bwd4 holds weights (one block per group)
    float *dg_int;
    int kept_v4;                  // rows of h, c, gates and dg are 16-byte aligned and H % 4 == 0
};

template <bool LSTM, bool VEC4>
__global__ __launch_bounds__(WG_THREADS, 2) void k_backward_heights(Fwd f, BwdHeights b)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    TileSmem &sm = *reinterpret_cast<TileSmem *>(smem_raw);
    const int tid = threadIdx.x;
    if (decided_to_leave(&sm.cmd[7], tid == 0 && batch_rejected(f))) return;
    const int H = f.H;
    const int n_levels = f.ctl->n_levels;
    const long long first = (long long)blockIdx.x * blockDim.x + tid, stride = (long long)gridDim.x * blockDim.x;
    unsigned epoch = 0, unused = 0;
    Fwd g = f;
    g.dg = b.dg_int;
    g.out_cols = 2 * H;
    for (int lvl = n_levels - 1; lvl >= 1; --lvl) {         // roots first: a parent is always higher than its children
        const int lo = f.level_off[lvl], rows = f.level_off[lvl + 1] - lo;
        const int32_t *list = f.level_nodes + lo;
        g.pos0 = lo;
        if constexpr (LSTM) {
            if (b.kept_v4) gate_grad_kept_rows<true, 4, true>(g, list, rows, lo, first, stride);
            else gate_grad_kept_rows<true, 1, true>(g, list, rows, lo, first, stride);
        } else {
            if (b.kept_v4) rnn_gate_grad_rows<4, true>(g, list, rows, lo, first, stride);
            else rnn_gate_grad_rows<1, true>(g, list, rows, lo, first, stride);
        }
        if (!grid_barrier(sm, f, epoch, 0u, 0u, &unused)) return;
        const int ng = (b.ng_inner == 4 && rows > 64) ? 4 : 1;
        g.bwd = (b.ng_inner == 4 && ng == 1) ? b.bwd1 : b.bwd4;
        g.n_cg = (2 * H / ng + HU - 1) / HU;
        const LevelPlan plan = plan_level(rows, f.cap_tiles);
        for (int item = blockIdx.x; item < plan.n_tiles * g.n_cg; item += gridDim.x) {
            const int tile = item / g.n_cg, cg = item - tile * g.n_cg;
            int start, count;
            plan_tile(plan, rows, tile, &start, &count);
            __syncthreads();                                // the row tables are free
            tile_set_rows<EPI_BWD_INNER_OPERAND>(sm, g, tid, tid < count ? list[start + tid] : -1, lo + start + tid);
            if (tid == 0) sm.cmd[3] = lo + start;
            __syncthreads();
            if (ng == 4) cell_tile<EPI_BWD_INNER_OPERAND4, VEC4, true>(sm, g, g.bwd, g.dg, count, cg);
            else cell_tile<EPI_BWD_INNER_OPERAND, VEC4, true>(sm, g, g.bwd, g.dg, count, cg);
        }
        if (!grid_barrier(sm, f, epoch, 0u, 0u, &unused)) return;
    }
}

// RNTN (d <= 96): the same walk, one phase and one grid barrier per height.  The gradient of the operand,
//     da_p = sum_k dz_k (sum_q S[(k, q)][p] a_q + W[p][k]),    dz = dh (1 - h^2),
// has the shape of the forward's bilinear form (cell_rows.hpp): a wave keeps the whole matrix of ONE p - 16 k side by side in d / 16 blocks, the
// contraction over q - as two fp16 terms in registers (128 at d = 64), multiplies the gathered rows [h_left ; h_right] of 16 nodes
// with it, scales the products by dz_k where they are and adds them up across the lanes.  Nothing of the d (2d + 1) values per node
// that the gradient is a contraction of is ever written (33 KB a node at d = 64); dz is (f.dg, by list position), for the weight gradient.
// A child's dh has one contribution, added at the memory side.
// Measured (training step; before: rows written, then contracted by the streaming cell with fp32 instructions, two launches per height): 256 parse
// trees at d = 64 1 311 -> 580 us (operand gradient, rows and launches 880 -> 150), 200 at d = 48 1 037 -> 397, 150 at d = 96 2 877 -> 984, 8 at d = 64
// 591 -> 243, 4 at d = 8 306 -> 161 (the last three with the forward's own change).  Error against 64 bits unchanged.
template <int NS> struct RntnBwdSmem {
    static constexpr int LDZ = 16 * NS + 4;
    halfx8 split[2][NS * 2 * 64];                           // as in RowsSmem
    float dz[2][16 * LDZ];
    int back[2][16];                                        // a row's sums are multiplied by two to this
    int child[2][2][16];
    int cmd[8];
};
constexpr int rntn_bwd_sets_per_cu(int ns) { return ns <= 4 ? 2 : 1; }

template <int NS>
__global__ __launch_bounds__(WG_THREADS, (rntn_bwd_sets_per_cu(NS))) void k_backward_rntn(Fwd f, int n_sets)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    using Smem = RntnBwdSmem<NS>;
    Smem &sm = *reinterpret_cast<Smem *>(smem_raw);
    constexpr int CPT = (NS + 3) / 4, LDZ = Smem::LDZ;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int d = f.H, seg = f.seg_chunks;
    const int set_size = (int)gridDim.x / n_sets, member = (int)blockIdx.x % set_size, slot = (int)blockIdx.x / set_size;
    if (decided_to_leave(&sm.cmd[7], tid == 0 && batch_rejected(f))) return;
    const int p = member * ROWS_UNITS + wave, pp = p < 2 * d ? p : 0;      // (a wave beyond the last p computes the first one's sums and adds nothing)
    halfx8 w[NS][NS][2];                                    // [k / 16][k-step over q]
    int sc[NS];                                             // ... and a column's by two to this
    float lin[NS];
    {
        const halfx8 *wp = reinterpret_cast<const halfx8 *>(f.xi.wp) + (size_t)pp * NS * NS * 128 + lane;
#pragma unroll
        for (int j = 0; j < NS; ++j)
#pragma unroll
            for (int t = 0; t < NS; ++t)
#pragma unroll
                for (int e = 0; e < 2; ++e) w[j][t][e] = wp[(size_t)((j * NS + t) * 2 + e) * 64];
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            sc[j] = (int)(__float_as_uint(f.xi.scale[((size_t)pp * 2 * NS + j) * HU + (lane & 15)]) >> 23) - 127;      // (columns beyond the last: products are zero)
            lin[j] = f.xi.scale[((size_t)pp * 2 * NS + NS + j) * HU + (lane & 15)];
        }
    }
    const unsigned row_b = (unsigned)d * 4u;
    const __amdgpu_buffer_rsrc_t rs_h = buf_of(f.h, (unsigned long long)f.n_nodes * row_b);
    const int my_row = tid >> 4, t16 = tid & 15;
    const bool ragged = d != seg * 8;
    uintx4_t rows[CPT][2];
    float dh[NS], hn[NS];
    int left = 0, right = 0;
    auto request = [&](int node) __attribute__((always_inline)) {
        left = f.left[node];
        right = f.right[node];
        const unsigned base0 = __umul24((unsigned)left, row_b), base1 = __umul24((unsigned)right, row_b);
#pragma unroll
        for (int i = 0; i < CPT; ++i) {
            const int c = t16 + 16 * i;
            const unsigned off = c < 2 * seg ? (c >= seg ? base1 + (unsigned)(c - seg) * 32u : base0 + (unsigned)c * 32u) : ~0u - 63u;
            rows[i][0] = __builtin_amdgcn_raw_buffer_load_b128(rs_h, (int)off, 0, 0);
            rows[i][1] = __builtin_amdgcn_raw_buffer_load_b128(rs_h, (int)off + 16, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            const int k = min(t16 + 16 * i, d - 1);
            hn[i] = f.h[(size_t)node * d + k];
            dh[i] = ld_dev(f.dh + (size_t)node * d + k);
        }
    };
    unsigned epoch = 0, unused = 0;
    int buf = 0;
    const int n_levels = f.ctl->n_levels;
#pragma unroll 1
    for (int lvl = n_levels - 1; lvl >= 1; --lvl) {         // roots first: a parent is always higher than its children
        const int lo = f.level_off[lvl], n_rows = f.level_off[lvl + 1] - lo, n_blocks = (n_rows + 15) >> 4;
        const int32_t *list = f.level_nodes + lo;
        // (rows beyond the height's last one stand in with that one: they are computed and not stored)
        auto node_of = [&](int blk) __attribute__((always_inline)) { return list[min(blk * 16 + my_row, n_rows - 1)]; };
        int node_next = 0;
        if (slot < n_blocks) {
            request(node_of(slot));
            node_next = node_of(slot + n_sets);
        }
#pragma unroll 1
        for (int blk = slot; blk < n_blocks; blk += n_sets, buf ^= 1) {
            const bool here = blk * 16 + my_row < n_rows;
            float m = 0.f;
#pragma unroll
            for (int i = 0; i < CPT; ++i) {
                const int c = t16 + 16 * i, in = (c >= seg ? c - seg : c) * 8;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    if (ragged && in + e >= d) rows[i][e >> 2][e & 3] = 0u;      // the next row's, or nothing's
                    m = fmaxf(m, fabsf(__uint_as_float(rows[i][e >> 2][e & 3])));
                }
            }
            m = fmaxf(m, dpp<DPP_XOR1>(m));
            m = fmaxf(m, dpp<DPP_XOR2>(m));
            m = fmaxf(m, dpp<DPP_HALF_MIRROR>(m));
            m = fmaxf(m, dpp<DPP_MIRROR>(m));
            const unsigned eb = max(__float_as_uint(m) >> 23, 15u);
            const float scale = __uint_as_float((268u - eb) << 23);
            if (t16 == 0) {
                sm.back[buf][my_row] = (int)eb - 14 - 127;
                sm.child[buf][0][my_row] = here ? left : -1;
                sm.child[buf][1][my_row] = here ? right : -1;
            }
#pragma unroll
            for (int i = 0; i < CPT; ++i) {
                const int c = t16 + 16 * i, s = c >> 2, quarter = c & 3;
                if (NS % 4 != 0 && c >= 4 * NS) continue;
                halfx8 hi, lo8;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float v = __uint_as_float(rows[i][e >> 2][e & 3]) * scale;
                    hi[e] = (_Float16)v;
                    lo8[e] = (_Float16)(v - (float)hi[e]);
                }
                halfx8 *dst = &sm.split[buf][s * 128 + rows_slot(s, quarter, my_row)];
                dst[0] = hi;
                dst[64] = lo8;
            }
#pragma unroll
            for (int i = 0; i < NS; ++i) {
                const int k = t16 + 16 * i;
                const float dz = k < d ? dh[i] * (1.f - hn[i] * hn[i]) : 0.f;
                sm.dz[buf][my_row * LDZ + k] = dz;
                if (member == 0 && here && k < d) f.dg[(size_t)(lo + blk * 16 + my_row) * d + k] = dz;
            }
            if (blk + n_sets < n_blocks) {
                request(node_next);
                node_next = node_of(blk + 2 * n_sets);
            }
            __syncthreads();
            const halfx8 *op = sm.split[buf];
            floatx4 t[NS];
#pragma unroll
            for (int j = 0; j < NS; ++j) t[j] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const halfx8 *o = &op[s * 128 + rows_slot(s, lane >> 4, lane & 15)];
                const halfx8 hi = o[0], lo8 = o[64];
#pragma unroll
                for (int j = 0; j < NS; ++j) t[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(hi, w[j][s][0], t[j], 0, 0, 0);
#pragma unroll
                for (int j = 0; j < NS; ++j) t[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(hi, w[j][s][1], t[j], 0, 0, 0);
#pragma unroll
                for (int j = 0; j < NS; ++j) t[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(lo8, w[j][s][0], t[j], 0, 0, 0);
            }
            const int *back = &sm.back[buf][4 * (lane >> 4)];
            const float *z = &sm.dz[buf][4 * (lane >> 4) * LDZ + (lane & 15)];
            float sum = 0.f;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                float x = 0.f;
                const int back_v = back[v];
                // (both scales at once: t times the column's alone may be infinite where the product with both is not)
#pragma unroll
                for (int j = 0; j < NS; ++j) x = __builtin_fmaf(z[v * LDZ + 16 * j], __builtin_amdgcn_ldexpf(t[j][v], sc[j] + back_v) + lin[j], x);
                x += dpp<DPP_XOR1>(x);
                x += dpp<DPP_XOR2>(x);
                x += dpp<DPP_HALF_MIRROR>(x);
                x += dpp<DPP_MIRROR>(x);
                if ((lane & 3) == v) sum = x;
            }
            const int row = 4 * (lane >> 4) + (lane & 3), child = sm.child[buf][p < d ? 0 : 1][row];
            if ((lane & 15) < 4 && child >= 0 && p < 2 * d) {
                bool again = __builtin_isnan(sum);
                if (__builtin_expect(again, 0))
                    for (int k = 0; k < d; ++k) again = again && !__builtin_isnan(sm.dz[buf][row * LDZ + k]);      // (nothing to gain there)
                if (__builtin_expect(again, 0)) {
                    // (an infinity has no two terms: in fp32 from the parameters as given)
                    const float *hl = f.h + (size_t)sm.child[buf][0][row] * d, *hr = f.h + (size_t)sm.child[buf][1][row] * d;
                    sum = 0.f;
#pragma unroll 1
                    for (int k = 0; k < d; ++k) {
                        const float *v = f.rntn_v + (size_t)k * 4 * d * d;
                        float x = f.xi.w[(size_t)p * d + k];
#pragma unroll 1
                        for (int q = 0; q < 2 * d; ++q) x = __builtin_fmaf(v[(size_t)p * 2 * d + q] + v[(size_t)q * 2 * d + p], q < d ? hl[q] : hr[q - d], x);
                        sum = __builtin_fmaf(sm.dz[buf][row * LDZ + k], x, sum);
                    }
                }
                (void)add_dev(f.dh + (size_t)child * d + (p < d ? p : p - d), sum);
            }
        }
        if (!grid_barrier(sm, f, epoch, 0u, 0u, &unused)) return;
    }
}

// Zeroes up to six arrays in one launch (outputs and workspace of the backward pass).
struct ZeroList {
    float *p[6];
    size_t n[6];
    const float *src;       // and one copy in the same launch: dst[0 .. n_copy) = src (n_copy = 0: none); a multiple of
    float *dst;             // four floats with both ends 16-byte aligned is moved 16 bytes at a time
    size_t n_copy;
};
__global__ void k_zero_many(ZeroList z)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x, first = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (z.n_copy % 4 == 0 && (((uintptr_t)z.src | (uintptr_t)z.dst) & 15) == 0) {
        const floatx4 *s4 = reinterpret_cast<const floatx4 *>(z.src);
        floatx4 *d4 = reinterpret_cast<floatx4 *>(z.dst);
        for (size_t e = first; e < z.n_copy / 4; e += stride) d4[e] = s4[e];
    } else {
        for (size_t e = first; e < z.n_copy; e += stride) z.dst[e] = z.src[e];
    }
#pragma unroll
    for (int a = 0; a < 6; ++a)
        for (size_t e = first; e < z.n[a]; e += stride) z.p[a][e] = 0.f;
}

}  // namespace tl
