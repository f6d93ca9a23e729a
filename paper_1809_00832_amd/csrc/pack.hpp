// Re-packing of the caller's row-major parameters into the operand order of the MFMA tiles.
//
// The caller's matrix W is [SEG*L x NG*H] (NG gate blocks of H columns).  The packed copy is
// indexed [column group cg][k-step s][gate g][lane][i]:
//   fp32 (16x16x4 MFMA, i < 4):  k = 16 s + 4 (lane / 16) + i
//   bf16 (16x16x32 MFMA, i < 8): k = 32 s + 8 (lane / 16) + i
// holds W[row(k)][g*H + 16 cg + lane % 16], so that one 16-byte read per lane yields the B
// operands of consecutive MFMAs and the five gates of a hidden unit meet in one lane.
// k runs over the padded K axis: SEG segments of Lp = roundup(L, 4) rows each, then zeros up
// to a multiple of KC; padded rows and hidden units >= H hold zeros.
#pragma once

#include <hip/hip_bf16.h>

#include "common.hpp"

namespace tl {

__device__ inline unsigned short f32_to_bf16_rne(float x)
{
    unsigned int bits = __float_as_uint(x);
    bits += 0x7FFFu + ((bits >> 16) & 1u);
    return (unsigned short)(bits >> 16);
}

__device__ inline float pack_source(const float *w, int k, int g, int hu, int NG, int H, int SEG, int L, int Lp)
{
    int seg = k / Lp, off = k - seg * Lp;
    if (seg >= SEG || off >= L || hu >= H) return 0.f;
    return w[(size_t)(seg * L + off) * ((size_t)NG * H) + (size_t)g * H + hu];
}

__global__ void k_pack_f32(const float *__restrict__ w, float *__restrict__ wp, int NG, int H, int SEG, int L, int Lp,
                           int n_steps, int n_cg)
{
    size_t total = (size_t)n_cg * n_steps * NG * 64 * 4;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x) {
        int i = (int)(e & 3);
        int lane = (int)((e >> 2) & 63);
        size_t r = e >> 8;
        int g = (int)(r % NG);
        r /= NG;
        int s = (int)(r % n_steps);
        int cg = (int)(r / n_steps);
        int k = 16 * s + 4 * (lane >> 4) + i;
        wp[e] = pack_source(w, k, g, cg * HU + (lane & 15), NG, H, SEG, L, Lp);
    }
}

__global__ void k_pack_bf16(const float *__restrict__ w, unsigned short *__restrict__ wp, int NG, int H, int SEG, int L,
                            int Lp, int n_steps32, int n_cg)
{
    size_t total = (size_t)n_cg * n_steps32 * NG * 64 * 8;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x) {
        int i = (int)(e & 7);
        int lane = (int)((e >> 3) & 63);
        size_t r = e >> 9;
        int g = (int)(r % NG);
        r /= NG;
        int s = (int)(r % n_steps32);
        int cg = (int)(r / n_steps32);
        int k = 32 * s + 8 * (lane >> 4) + i;
        wp[e] = f32_to_bf16_rne(pack_source(w, k, g, cg * HU + (lane & 15), NG, H, SEG, L, Lp));
    }
}

__global__ void k_pack_bias(const float *__restrict__ b, float *__restrict__ bp, int NG, int H, int n_cg)
{
    int total = n_cg * NG * HU;
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < total; e += gridDim.x * blockDim.x) {
        int j = e % HU, g = (e / HU) % NG, cg = e / (HU * NG);
        int hu = cg * HU + j;
        bp[e] = hu < H ? b[g * H + hu] : 0.f;
    }
}

// Several fp32 matrices packed over in one launch (the re-packing after a parameter update: the buffers exist, only their
// contents change).  A job is what k_pack_f32 and k_pack_bias do for one matrix; element (row, col) of the matrix to pack
// is src[row * rs + col * cs], so the transposed matrices of the backward pass are read straight from the parameters
// (rs = 1, cs = number of rows) with no transposed copy in between.
struct PackJob {
    const float *w;
    float *wp;
    const float *b;         // null: the bias is not touched (the backward pass's contractions have none)
    float *bp;
    int NG, H, SEG, L, Lp, n_steps, n_cg;
    long long rs, cs;
};
constexpr int PACK_JOBS = 6;
struct PackList {
    PackJob job[PACK_JOBS];
    int n;
};
// A thread takes four consecutive k of a column (one 16-byte store).  Element by element, with three divisions in 64 bits each, an update's
// packing is bound by that arithmetic: 33 us at H = 512 and 17 at H = 150; by quads and in 32 bits, wherever a job's quads can be counted in them, 30 and 13.7.
template <class I> __device__ inline void pack_quads(const PackJob &j, I first, I stride)
{
    const I total = (I)j.n_cg * (I)j.n_steps * (I)j.NG * 64;
    for (I e = first; e < total; e += stride) {
        const int lane = (int)(e & 63);
        const I r = e >> 6, r2 = r / (unsigned)j.NG;
        const int g = (int)(r - r2 * (unsigned)j.NG), cg = (int)(r2 / (unsigned)j.n_steps), s = (int)(r2 - (I)cg * (unsigned)j.n_steps);
        const int k = 16 * s + 4 * (lane >> 4), hu = cg * HU + (lane & 15);
        const float *src = j.w + (long long)(g * j.H + hu) * j.cs;
        int seg = k / j.Lp, off = k - seg * j.Lp;
        floatx4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (seg < j.SEG && off < j.L && hu < j.H) v[i] = src[(long long)(seg * j.L + off) * j.rs];
            if (++off == j.Lp) {
                off = 0;
                ++seg;
            }
        }
        *reinterpret_cast<floatx4 *>(j.wp + 4 * (size_t)e) = v;
    }
}
__device__ inline void pack_many(const PackList &pl, size_t first, size_t stride)
{
    for (int a = 0; a < pl.n; ++a) {
        const PackJob &j = pl.job[a];
        const size_t quads = (size_t)j.n_cg * j.n_steps * j.NG * 64;
        if (quads + stride < 0x80000000ull) pack_quads<unsigned>(j, (unsigned)first, (unsigned)stride);
        else pack_quads<size_t>(j, first, stride);
        if (j.b) {
            const size_t nb = (size_t)j.n_cg * j.NG * HU;
            for (size_t at = first; at < nb; at += stride) {
                const int e = (int)at, q = e % HU, g = (e / HU) % j.NG, cg = e / (HU * j.NG);
                const int hu = cg * HU + q;
                j.bp[e] = hu < j.H ? j.b[g * j.H + hu] : 0.f;
            }
        }
    }
}

// The two fp16 terms of a matrix for the split cell (cell_split.hpp): [column group][k-step of 32][gate][hi, lo][lane][8].
// The K axis is SEG segments of `steps` k-steps (L rows, zero padded), then zeros up to n_steps k-steps.  Every column is
// scaled by the power of two that brings its largest magnitude into [2^13, 2^14) (exponents beyond what fp32 can undo are cut
// off); `scale` receives what a sum of products is to be multiplied by (NaN: the column holds an infinity, which has no two terms).  One workgroup per column group and gate holds
// its 16 columns in registers, looks for their largest magnitudes and packs them.
struct SplitPackJob {
    const float *w;
    _Float16 *wp;
    float *scale;
    int NG, H, SEG, L, steps, n_steps, n_cg;
    float operand_scale;    // of the other side
};
constexpr int SPLIT_PACK_JOBS = 2, SPLIT_PACK_T = 8;      // n_steps <= 4 * SPLIT_PACK_T
struct SplitPackList {
    SplitPackJob job[SPLIT_PACK_JOBS];
    int n;
};
__device__ inline void pack_split_block(const SplitPackList &pl, int b)
{
    __shared__ unsigned s_max[16], s_inf[16];
    int a = 0;
    while (a + 1 < pl.n && b >= pl.job[a].n_cg * pl.job[a].NG) {
        b -= pl.job[a].n_cg * pl.job[a].NG;
        a += 1;
    }
    const SplitPackJob &j = pl.job[a];
    if (b >= j.n_cg * j.NG) return;
    const int g = b % j.NG, cg = b / j.NG, tid = threadIdx.x;
    const int col = tid & 15, unit = cg * HU + col, kg = tid >> 4 & 3;
    const size_t ld = (size_t)j.NG * j.H;
    const float *w = j.w + (size_t)g * j.H + unit;
    if (tid < 16) s_max[tid] = s_inf[tid] = 0u;
    __syncthreads();
    // thread: eight consecutive k of its column in every fourth k-step, all requested together
    float x[SPLIT_PACK_T][8];
    unsigned m = 0u;                                            // largest finite magnitude, as bits
    bool inf = false;
#pragma unroll
    for (int t = 0; t < SPLIT_PACK_T; ++t) {
#pragma unroll
        for (int i = 0; i < 8; ++i) x[t][i] = 0.f;
        if (4 * t >= j.n_steps) continue;
        const int s = 4 * t + (tid >> 6), seg = s / j.steps, off = (s - seg * j.steps) * 32 + 8 * kg;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (seg < j.SEG && off + i < j.L && unit < j.H) x[t][i] = w[(size_t)(seg * j.L + off + i) * ld];
        }
    }
#pragma unroll
    for (int t = 0; t < SPLIT_PACK_T; ++t)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const unsigned v = __float_as_uint(x[t][i]) & 0x7FFFFFFFu;
            if (v < 0x7F800000u) m = max(m, v);
            else if (v == 0x7F800000u) inf = true;
        }
    atomicMax(&s_max[col], m);
    if (inf) s_inf[col] = 1u;
    __syncthreads();
    const int top = (int)(s_max[col] >> 23);                    // biased exponent of the column's largest magnitude
    const int e = min(13 - (top - 127), 100);                   // the column is scaled by 2^e
    if (tid < 16) j.scale[(cg * j.NG + g) * HU + col] = s_inf[col] ? __uint_as_float(0x7FC00000u) : unit < j.H ? ldexpf(1.f / j.operand_scale, -e) : 0.f;
#pragma unroll
    for (int t = 0; t < SPLIT_PACK_T; ++t) {
        const int s = 4 * t + (tid >> 6);
        if (s >= j.n_steps) continue;
        typedef _Float16 half8 __attribute__((ext_vector_type(8)));
        half8 hi, lo;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float v = ldexpf(x[t][i], e);
            hi[i] = (_Float16)v;
            lo[i] = (_Float16)(v - (float)hi[i]);
        }
        half8 *dst = reinterpret_cast<half8 *>(j.wp) + (((size_t)cg * j.n_steps + s) * j.NG + g) * 2 * 64 + kg * 16 + col;
        dst[0] = hi;
        dst[64] = lo;
    }
}

// The two fp16 terms of a matrix whose rows are the columns of a contraction (the transposed matrices of the backward pass, read along their
// rows): [column group][k-step of 32][side][hi, lo][lane][8].  Column (side, c) is row side * n + c of w, NG * K values; k-step s holds values
// 32 (s / NG) ... + 31 of the (s % NG)th K of them.  Scales as above, for an operand whose own scale is not known here.  One workgroup
// per column group and side, 16 threads a column.
constexpr int ROWS_PACK_T = 20;     // n_steps <= 4 * ROWS_PACK_T
struct RowsPackJob {
    const float *w;
    _Float16 *wp;
    float *scale;
    int NG, K, n, sides, n_steps, n_cg;
};
struct RowsPackList {
    RowsPackJob job[2];
    int n, blocks;
};
__device__ inline void pack_rows_block(const RowsPackList &pl, int b)
{
    int a = 0;
    while (a + 1 < pl.n && b >= pl.job[a].n_cg * pl.job[a].sides) {
        b -= pl.job[a].n_cg * pl.job[a].sides;
        a += 1;
    }
    const RowsPackJob &j = pl.job[a];
    if (b >= j.n_cg * j.sides) return;
    const int side = b % j.sides, cg = b / j.sides, col = threadIdx.x >> 4, t16 = threadIdx.x & 15, c = cg * HU + col, len = j.NG * j.K;
    const bool here = c < j.n;
    const float *w = j.w + (size_t)(side * j.n + (here ? c : 0)) * len;
    // thread: every sixteenth piece of eight consecutive values of its column, all requested together
    float x[ROWS_PACK_T][8];
    const bool quad = (j.K & 3) == 0 && ((uintptr_t)j.w & 15) == 0;
#pragma unroll
    for (int t = 0; t < ROWS_PACK_T; ++t) {
#pragma unroll
        for (int q = 0; q < 8; ++q) x[t][q] = 0.f;
        if (4 * t >= j.n_steps) continue;
        const int i = t16 + 16 * t, s = i >> 2, k0 = s / j.NG * 32 + 8 * (i & 3);
        const float *src = w + (size_t)(s % j.NG) * j.K + k0;
        const bool piece = here && i < j.n_steps * 4;
        if (quad) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const floatx4 v = piece && k0 + 4 * h < j.K ? *reinterpret_cast<const floatx4 *>(src + 4 * h) : floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int q = 0; q < 4; ++q) x[t][4 * h + q] = v[q];
            }
        } else {
#pragma unroll
            for (int q = 0; q < 8; ++q) x[t][q] = piece && k0 + q < j.K ? src[q] : 0.f;
        }
    }
    unsigned m = 0u;                                            // largest finite magnitude, as bits
    int inf = 0;
#pragma unroll
    for (int t = 0; t < ROWS_PACK_T; ++t)
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const unsigned v = __float_as_uint(x[t][q]) & 0x7FFFFFFFu;
            if (v < 0x7F800000u) m = max(m, v);
            else if (v == 0x7F800000u) inf = 1;
        }
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
        m = max(m, (unsigned)__shfl_xor((int)m, o));
        inf |= __shfl_xor(inf, o);
    }
    const int e = min(13 - ((int)(m >> 23) - 127), 100);
    if (t16 == 0) j.scale[(cg * j.sides + side) * HU + col] = inf ? __uint_as_float(0x7FC00000u) : here ? ldexpf(1.f, -e) : 0.f;
    typedef _Float16 half8 __attribute__((ext_vector_type(8)));
#pragma unroll
    for (int t = 0; t < ROWS_PACK_T; ++t) {
        const int i = t16 + 16 * t, s = i >> 2;
        if (i >= j.n_steps * 4) continue;
        half8 hi, lo;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const float v = ldexpf(x[t][q], e);
            hi[q] = (_Float16)v;
            lo[q] = (_Float16)(v - (float)hi[q]);
        }
        half8 *dst = reinterpret_cast<half8 *>(j.wp) + (((size_t)cg * j.n_steps + s) * j.sides + side) * 2 * 64 + (i & 3) * 16 + col;
        dst[0] = hi;
        dst[64] = lo;
    }
}

// All of them, side by side: the first n_split workgroups pack the split weights, the next ones those of the backward pass, the others the rest (one launch
// after an update; the split weights' workgroups are a chain of loads, maximum and stores, 7 to 12 us, and few).
__global__ __launch_bounds__(256) void k_repack(PackList pl, SplitPackList sl, RowsPackList rl, int n_split)
{
    const int b = (int)blockIdx.x - n_split, rest = b - rl.blocks;
    if (b < 0) pack_split_block(sl, blockIdx.x);
    else if (rest < 0) pack_rows_block(rl, b);
    else pack_many(pl, (size_t)rest * blockDim.x + threadIdx.x, (size_t)(gridDim.x - n_split - rl.blocks) * blockDim.x);
}

// bf16 copy of a row-major table with rows padded to Ls elements (pads zero)
__global__ void k_pad_bf16(const float *__restrict__ src, unsigned short *__restrict__ dst, size_t rows, int L, int Ls)
{
    const size_t total = rows * (size_t)Ls;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (size_t)gridDim.x * blockDim.x) {
        const size_t r = e / Ls;
        const int j = (int)(e - r * Ls);
        dst[e] = j < L ? f32_to_bf16_rne(src[r * L + j]) : (unsigned short)0;
    }
}

}  // namespace tl
