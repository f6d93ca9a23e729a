// Structure pass: integer-only kernels that turn the child arrays of a batch into what the
// schedulers need.  This is the device counterpart of the master that sorts operations into a
// ready queue or a waiting list by their number of unresolved inputs (Section 4.1, Figure 4
// step 2) and of the parent pointers that stand in for a call stack ("Graph execution stack").
//
// Counters that many threads bump at once are bumped once per workgroup (ballot + popcount per
// wave, combined in LDS; LDS histograms): atomics on one address are served one after the other.
#pragma once

#include "common.hpp"

namespace tl {

// Largest t with tree_off[t] <= n, by bisection over [0, n_trees).  Always returns an index in
// range, whatever the array holds.
__device__ inline int tree_of(const int32_t *tree_off, int n_trees, int n)
{
    int lo = 0, hi = n_trees - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (tree_off[mid] <= n) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Slot in an append-only list for every thread with pred set (-1 for the others): one atomic per
// workgroup of up to 1024 threads.  Must be called by
// all threads of the workgroup; s_cnt is shared scratch of APPEND_SCRATCH ints.
constexpr int APPEND_SCRATCH = 17;
template <typename T> __device__ inline int block_append(T *counter, bool pred, int *s_cnt)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n_waves = (blockDim.x + 63) >> 6;
    const unsigned long long mask = __ballot(pred);
    if (lane == 0) s_cnt[wave] = __popcll(mask);
    __syncthreads();
    if (threadIdx.x == 0) {
        int total = 0;
        for (int w = 0; w < n_waves; ++w) {
            const int c = s_cnt[w];
            s_cnt[w] = total;
            total += c;
        }
        s_cnt[16] = total ? (int)atomicAdd(counter, (T)total) : 0;
    }
    __syncthreads();
    const int slot = pred ? s_cnt[16] + s_cnt[wave] + __popcll(mask & ((1ull << lane) - 1ull)) : -1;
    __syncthreads();
    return slot;
}

// Threads per workgroup of the per-node kernels that append to lists.
constexpr int NODE_BLOCK = 1024;

// Data-flow scheduler: the rows that internal nodes will produce - c, and the h row their parents gather (the bf16
// or the split copy when there is one) - show "not written" (all ones) in every element until they are.  One wave per row; called
// by all lanes of wave number `wave` of `n_waves`.
__device__ inline void flow_fill(const Fwd &f, size_t wave, size_t n_waves)
{
    const int H = f.H, lane = threadIdx.x & 63;
    const bool quad = (H & 3) == 0 && (((uintptr_t)f.h | (uintptr_t)f.c) & 15) == 0;
    const float ones = __uint_as_float(0xFFFFFFFFu);
    const floatx4 ones4 = floatx4{ones, ones, ones, ones};
    auto fill_row = [&](size_t n) {
        float *c = f.c ? f.c + n * H : nullptr, *h = f.hb || f.hx ? nullptr : f.h + n * H;
        if (quad) {
            for (int e = lane * 4; e < H; e += 256) {
                if (c) *reinterpret_cast<floatx4 *>(c + e) = ones4;
                if (h) *reinterpret_cast<floatx4 *>(h + e) = ones4;
            }
        } else {
            for (int e = lane; e < H; e += 64) {
                if (c) c[e] = ones;
                if (h) h[e] = ones;
            }
        }
        if (f.hb) {
            unsigned short *hb = f.hb + n * f.hs;             // rows 16-byte aligned; what lies beyond H stays zero
            for (int e = lane * 8; e < H; e += 512) {
                if (e + 8 <= H) *reinterpret_cast<floatx4 *>(hb + e) = ones4;
                else for (int k = e; k < H; ++k) hb[k] = (unsigned short)0xFFFFu;
            }
        }
        if (f.hx) {
            unsigned *hx = f.hx + n * (size_t)(f.hx_steps * 32);        // rows of whole 128-byte lines; words of pad units alone stay zero
            for (int q = lane; q < f.hx_steps * 8; q += 64) {
                const int unit = (q >> 3) * 32 + (q & 3) * 8;           // first of the 8 units of these 16 bytes
                if (unit + 8 <= H) *reinterpret_cast<floatx4 *>(hx + 4 * q) = ones4;
                else for (int k = 0; k < 4; ++k) if (unit + 2 * k < H) hx[4 * q + k] = 0xFFFFFFFFu;
            }
        }
    };
    const size_t N = (size_t)f.n_nodes;
    if (n_waves >= N) {
        if (wave < N && f.left[wave] >= 0) fill_row(wave);
        return;
    }
    // fewer waves than nodes: the kinds of up to 64 nodes in one load, then their rows one after the other (a load per row
    // would make every row a round trip)
    const size_t share = (N + n_waves - 1) / n_waves, chunk = share < 64 ? share : 64;
    for (size_t n0 = wave * chunk; n0 < N; n0 += n_waves * chunk) {
        const size_t n = n0 + lane;
        unsigned long long todo = __ballot((size_t)lane < chunk && n < N && f.left[n < N ? n : N - 1] >= 0);
        for (; todo != 0ull; todo &= todo - 1ull) fill_row(n0 + __builtin_ctzll(todo));
    }
}

// Resets the per-forward scheduler state.  A fill kernel rather than memsets so that a caller
// may capture the forward in a HIP graph.
__global__ void k_reset(Fwd f, int with_levels)
{
    const int N = f.n_nodes;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    const size_t ctl_words = sizeof(Ctl) / 4, gang_words = (size_t)MAX_GANGS * sizeof(GangBox) / 4;
    size_t total = (size_t)N + 1;
    if (total < ctl_words) total = ctl_words;
    if (total < gang_words) total = gang_words;
    if (f.rntn_done && total < (size_t)f.rntn_units * f.n_cg) total = (size_t)f.rntn_units * f.n_cg;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += stride) {
        if (i < (size_t)N) {
            f.parent[i] = -1;
            f.pending[i] = 0;
            if (with_levels) { f.height[i] = 0; f.arrive[i] = 0; f.level_fill[i] = 0; }
        }
        if (with_levels && i <= (size_t)N) f.level_cnt[i] = 0;
        if (i < (size_t)f.n_int) { f.q_rec[i].lo = 0; f.q_rec[i].hi = 0; }
        if (i < (size_t)f.n_trees) f.root_ws[i] = -1;
        if (f.rntn_done && i < (size_t)f.rntn_units * f.n_cg) f.rntn_done[i] = 0u;   // (a forward that gave up may have left counts)
        if (i < ctl_words) ((unsigned int *)f.ctl)[i] = 0;
        if (i < gang_words) ((unsigned int *)f.gangs)[i] = 0;
    }
    if (f.flow == 1) flow_fill(f, ((size_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6, stride >> 6);
}

// One thread per node: checks, parent scatter, leaf list, counters of unfinished children.
// Leaves are evaluated by a kernel of their own before any internal node, so pending[] counts
// internal children only, and an internal node whose children are both leaves starts ready.
// int_list: null, or (backward pass) receives the internal nodes, in no particular order.  large: 0, or the nodes that make a tree large (back_by_heights).
__device__ __forceinline__ void scatter_nodes(const Fwd &f, int32_t *int_list, int large)
{
    __shared__ int s_cnt[APPEND_SCRATCH];
    const int n = blockIdx.x * blockDim.x + threadIdx.x;
    Ctl *ctl = f.ctl;
    if (n <= f.n_trees) {   // offsets: 0 = off[0] < off[1] < ... < off[B] = N
        int v = f.tree_off[n];
        bool ok = (n == 0) ? (v == 0) : (v > f.tree_off[n - 1]);
        if (n == f.n_trees) ok = ok && (v == f.n_nodes);
        if (!ok) latch_error(ctl, TL_ESTRUCT);
    }
    bool is_leaf = false, is_seed = false;
    int l = -1, r = -1;
    if (n < f.n_nodes) {
        const int t = tree_of(f.tree_off, f.n_trees, n);
        const int lo = f.tree_off[t], hi = f.tree_off[t + 1];
        l = f.left[n];
        r = f.right[n];
        if (large > 0 && n == lo && hi - lo >= large) atomicAdd(&ctl->n_large, 1);
        if (n < lo || n >= hi) {
            latch_error(ctl, TL_ESTRUCT);
        } else if (l < 0 && r < 0) {
            const int w = f.word[n];
            if (w < 0 || w >= f.vocab) latch_error(ctl, TL_ESTRUCT); else is_leaf = true;
        } else if (l >= lo && l < hi && r >= lo && r < hi && l < f.n_nodes && r < f.n_nodes && l != r && l != n &&
                   r != n) {
            if (atomicCAS(&f.parent[l], -1, n) != -1) latch_error(ctl, TL_ESTRUCT);
            if (atomicCAS(&f.parent[r], -1, n) != -1) latch_error(ctl, TL_ESTRUCT);
            const int pend = (f.left[l] >= 0) + (f.left[r] >= 0);
            f.pending[n] = pend;
            is_seed = pend == 0;
            if (large > 0 && is_seed && hi - lo >= large) atomicAdd(&ctl->n_large_seeds, 1);
        } else {
            latch_error(ctl, TL_ESTRUCT);
        }
    }
    const int leaf_slot = block_append(&ctl->n_leaf_seen, is_leaf, s_cnt);
    if (is_leaf && leaf_slot < f.n_leaf) f.leaf_list[leaf_slot] = n;
    const int seed_slot = block_append(&ctl->q_tail.v, is_seed, s_cnt);
    if (is_seed && seed_slot < f.n_int) qrec_store<false>(&f.q_rec[seed_slot], n, l, r);
    if (int_list) {
        const bool inner = n < f.n_nodes && l >= 0;
        const int slot = block_append(&ctl->n_int_seen, inner, s_cnt);
        if (inner && slot < f.n_int) int_list[slot] = n;
    }
}
__global__ __launch_bounds__(NODE_BLOCK) void k_scatter(Fwd f) { scatter_nodes(f, nullptr, 0); }
__global__ __launch_bounds__(NODE_BLOCK) void k_scatter_list(Fwd f, int32_t *int_list, int large) { scatter_nodes(f, int_list, large); }

// One thread per node: the node nobody points to is its tree's root; there must be exactly one.
__global__ __launch_bounds__(NODE_BLOCK) void k_roots(Fwd f)
{
    __shared__ int s_cnt[APPEND_SCRATCH];
    const int n = blockIdx.x * blockDim.x + threadIdx.x;
    Ctl *ctl = f.ctl;
    if (n == 0) {
        if (ctl->n_leaf_seen != f.n_leaf) latch_error(ctl, TL_ESTRUCT);
        ctl->n_seed = (int)ctl->q_tail.v;                // the first frontier: internal nodes over two leaves
    }
    const bool is_root = n < f.n_nodes && f.parent[n] == -1;
    if (is_root) {
        const int t = tree_of(f.tree_off, f.n_trees, n);
        if (atomicCAS(&f.root_ws[t], -1, n) != -1) latch_error(ctl, TL_ESTRUCT);     // a second root of the same tree
    }
    // no tree has two roots, so "as many roots as trees" means one each; later kernels compare the two
    // numbers (batch_rejected) and the root gather reports a mismatch
    block_append(&ctl->n_roots, is_root, s_cnt);
}

// ---- distance from the root (priority scheduling) -----------------------------------------
// One thread per node walks up the parent links and counts, giving up after DEPTH_CAP steps: the
// priority rule only asks whether a node is far from its root compared with the rest of the
// batch, so a distance of "DEPTH_CAP or more" is as good as the exact one, and the longest walk
// (which sets the duration of the kernel) stays short however deep a tree is.  The parent array
// of a batch fits the L2, so a step costs a cache hit.
constexpr int DEPTH_CAP = 128;

__global__ __launch_bounds__(NODE_BLOCK) void k_depth_walk(Fwd f)
{
    __shared__ unsigned s_sum[16];
    if (batch_rejected(f)) return;
    const int n = blockIdx.x * blockDim.x + threadIdx.x;
    unsigned d = 0;
    if (n < f.n_nodes) {
        int p = f.parent[n];
        while (p >= 0 && d < (unsigned)DEPTH_CAP) {
            d += 1;
            p = f.parent[p];
        }
        f.depth_root[n] = (int)d;
    }
    unsigned sum = d;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) sum += __shfl_xor(sum, o);
    if ((threadIdx.x & 63) == 0) s_sum[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long total = 0;
        for (int w = 0; w < (int)((blockDim.x + 63) >> 6); ++w) total += s_sum[w];
        if (total) atomicAdd(&f.ctl->depth_sum.v, total);
    }
}

// A node is critical when at least this many dependent steps are still above it: 32, or four times the
// batch's mean if that is more (then nothing is critical in a batch whose mean exceeds DEPTH_CAP / 4).
__device__ inline int critical_threshold(const Fwd &f)
{
    const unsigned long long mean4 = 4ull * f.ctl->depth_sum.v / (unsigned long long)f.n_nodes;
    return mean4 > 32ull ? (mean4 > 0x7fffffffull ? 0x7fffffff : (int)mean4) : 32;
}

// Rewrites the first n_seed records of the ready queue (the internal nodes over two leaves) with the
// critical ones at the front, the others filled in from the back.
__global__ __launch_bounds__(NODE_BLOCK) void k_seed_place(Fwd f)
{
    __shared__ int s_cnt[APPEND_SCRATCH];
    if (batch_rejected(f)) return;
    const int n = blockIdx.x * blockDim.x + threadIdx.x;
    Ctl *ctl = f.ctl;
    const int thr = critical_threshold(f);
    bool seed = false, crit = false;
    int l = -1, r = -1;
    if (n < f.n_nodes) {
        l = f.left[n];
        r = f.right[n];
        seed = l >= 0 && f.pending[n] == 0;
        crit = seed && f.depth_root[n] >= thr;
    }
    const int front = block_append(&ctl->seed_front.v, crit, s_cnt);
    const int back = block_append(&ctl->seed_back.v, seed && !crit, s_cnt);
    const int slot = crit ? front : ctl->n_seed - 1 - back;
    if (seed && slot >= 0 && slot < f.n_int) qrec_store<false>(&f.q_rec[slot], n, l, r);
}

// Heights by climbing: one thread per leaf walks towards the root; at every internal node the
// first child to arrive stops, the second continues with height 1 + max.  The walk passes each
// node once, so a thread's loop is bounded by the tree height.  The two children meet through one
// exchange on height[p] (zero before the pass): the first leaves 1 + its own height there and
// finds zero, the second finds the first one's value - the data travels in the word that is
// exchanged, so a step costs two memory round trips (the parent, the exchange) and no fence.
// arrive[p] = 2 marks the nodes whose height is final.  Called by one thread per leaf n; final(height) for every node whose height it settles.
template <typename Final> __device__ __forceinline__ void climb_from(const Fwd &f, int n, Final final)
{
    int hcur = 0;
    for (int guard = 0; guard < f.n_nodes; ++guard) {
        const int p = f.parent[n];
        if (p < 0) break;
        const int other = atomicExch(&f.height[p], hcur + 1);
        if (other == 0) break;                   // the sibling's subtree is not done yet: its thread will carry on
        hcur = other > hcur + 1 ? other : hcur + 1;
        f.height[p] = hcur;
        f.arrive[p] = 2;
        final(hcur);
        n = p;
    }
}
__global__ void k_climb(Fwd f)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (batch_rejected(f) || internal_kernel_skipped(f) || i >= f.n_leaf) return;
    climb_from(f, f.leaf_list[i], [](int) {});
}

constexpr int HIST_BINS = 1024;

// One thread per node: histogram of the heights of the internal nodes that the climb reached
// (both children arrived), and the largest height.
__global__ void k_level_hist(Fwd f)
{
    __shared__ int s_hist[HIST_BINS];
    __shared__ int s_max;
    const int n = blockIdx.x * blockDim.x + threadIdx.x;
    if (batch_rejected(f) || internal_kernel_skipped(f)) return;
    for (int b = threadIdx.x; b < HIST_BINS; b += blockDim.x) s_hist[b] = 0;
    if (threadIdx.x == 0) s_max = 0;
    __syncthreads();
    if (n < f.n_nodes && f.left[n] >= 0 && f.arrive[n] == 2) {
        const int hgt = f.height[n];
        if (hgt < HIST_BINS) atomicAdd(&s_hist[hgt], 1); else atomicAdd(&f.level_cnt[hgt], 1);
        atomicMax(&s_max, hgt);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < HIST_BINS; b += blockDim.x)
        if (s_hist[b]) atomicAdd(&f.level_cnt[b], s_hist[b]);
    if (threadIdx.x == 0 && s_max > 0) atomicMax(&f.ctl->max_height, s_max);
}

// Single workgroup: exclusive scan of the height histogram into level offsets.  Height 0 (the
// leaves) has no list: leaves are taken from leaf_list.
__global__ void k_scan_levels(Fwd f)
{
    __shared__ int s_part[1024];
    __shared__ int s_carry;
    Ctl *ctl = f.ctl;
    const int tid = threadIdx.x;
    if (batch_rejected(f)) {
        if (tid == 0) {
            ctl->n_levels = 0;
            latch_error(ctl, TL_ESTRUCT);
        }
        return;
    }
    if (internal_kernel_skipped(f)) return;
    const int n_levels = ctl->max_height + 1;
    if (tid == 0) s_carry = 0;
    __syncthreads();
    for (int base = 0; base < n_levels; base += 1024) {
        const int idx = base + tid;
        const int v = idx < n_levels ? f.level_cnt[idx] : 0;
        s_part[tid] = v;
        __syncthreads();
        for (int d = 1; d < 1024; d <<= 1) {
            int add = tid >= d ? s_part[tid - d] : 0;
            __syncthreads();
            s_part[tid] += add;
            __syncthreads();
        }
        const int carry = s_carry;
        if (idx < n_levels) f.level_off[idx] = carry + s_part[tid] - v;
        __syncthreads();
        if (tid == 1023) s_carry = carry + s_part[1023];
        __syncthreads();
    }
    if (tid == 0) {
        f.level_off[n_levels] = s_carry;
        ctl->n_levels = n_levels;
        ctl->reached = s_carry + f.n_leaf;
        if (s_carry != f.n_int) latch_error(ctl, TL_ESTRUCT);   // nodes no leaf leads to (cycle)
    }
}

// One thread per node: append every reached internal node to the list of its height.
// place_of: null, or (backward pass) see SchedPlaces.
__device__ __forceinline__ void fill_levels(const Fwd &f, int2 *place_of)
{
    __shared__ int s_hist[HIST_BINS];
    __shared__ int s_base[HIST_BINS];
    const int n = blockIdx.x * blockDim.x + threadIdx.x;
    if (batch_rejected(f) || internal_kernel_skipped(f)) return;
    for (int b = threadIdx.x; b < HIST_BINS; b += blockDim.x) s_hist[b] = 0;
    __syncthreads();
    const bool mine = n < f.n_nodes && f.left[n] >= 0 && f.arrive[n] == 2;
    int hgt = 0, rank = 0;
    if (mine) {
        hgt = f.height[n];
        rank = hgt < HIST_BINS ? atomicAdd(&s_hist[hgt], 1) : atomicAdd(&f.level_fill[hgt], 1);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < HIST_BINS; b += blockDim.x)
        if (s_hist[b]) s_base[b] = atomicAdd(&f.level_fill[b], s_hist[b]);
    __syncthreads();
    if (mine) {
        const int slot = f.level_off[hgt] + rank + (hgt < HIST_BINS ? s_base[hgt] : 0);
        if (slot < f.n_int) f.level_nodes[slot] = n;
        if (place_of) {
            const int lo = f.level_off[hgt], block = (slot - lo) & ~15;
            place_of[n] = int2{lo + block, min(16, f.level_off[hgt + 1] - lo - block) | (slot - lo - block) << 8};
        }
    }
}
__global__ void k_fill_levels(Fwd f) { fill_levels(f, nullptr); }
__global__ void k_fill_places(Fwd f, int2 *place_of) { fill_levels(f, place_of); }

// h_root / c_root / root outputs.
__global__ void k_root_gather(Fwd f)
{
    if (batch_rejected(f)) {
        if (blockIdx.x == 0 && threadIdx.x == 0) latch_error(f.ctl, TL_ESTRUCT);    // a tree without a root
        return;
    }
    const int t = blockIdx.x;
    const int r = f.root_ws[t];
    if (r < 0) return;
    if (threadIdx.x == 0 && f.root_out) f.root_out[t] = r;
    for (int j = threadIdx.x; j < f.H; j += blockDim.x) {
        if (f.h_root) f.h_root[(size_t)t * f.H + j] = f.h[(size_t)r * f.H + j];
        if (f.c_root && f.c) f.c_root[(size_t)t * f.H + j] = f.c[(size_t)r * f.H + j];
    }
}

// ---- schedule of the data-flow kernel ------------------------------------------------------------
// The trees of the batch are dealt to the slots (sets of workgroups that cover all column groups) in contiguous ranges of
// about equal node count.  For every slot one workgroup orders the internal nodes of its trees with the ready
// counters of Section 4.1: it starts with the nodes over two leaves; handing a node out counts it at its parent, and a
// parent whose internal children have all been handed out goes to the end of the list.  The list is cut into blocks of up to
// 16 nodes whose children all lie in earlier blocks: rounds of whole blocks as long as enough nodes wait, what is left of the
// list (at most 16) otherwise.  A block is `late` if a node of it became ready with the block right before it.
// The order depends on the trees alone, so one workgroup prepares it for all, beside the leaf cells; the cell kernel then
// walks finished blocks and knows two blocks ahead what it will need.  The rounds are a chain of LDS accesses of one wave
// (0.2 us each), the lists of a slot in LDS (5 bytes per node) or, for slots of more nodes than fit, in the workspace.
constexpr unsigned SCHED_LATE = 0x80000000u;
constexpr size_t SCHED_LDS_BYTES = 52 * 1024;     // three workgroups of the kernel that does it beside its own work fit on a CU
__host__ __device__ constexpr size_t sched_lds_bytes(size_t n) { return 16 + 64 + ((2 * n + 3) & ~(size_t)3) + ((n + 3) & ~(size_t)3) + 2 * (2 * (n / 2 + 1) + 2); }

template <bool IN_LDS> struct SchedLists;
template <> struct SchedLists<true> {
    typedef unsigned short T;
    static constexpr unsigned NONE = 0xFFFFu, LATE = 0x8000u;
    T *par, *pool, *start;              // parent and (list position ->) node, relative to the slot's first node; first list position of a block
    unsigned *cnt;                      // internal children not handed out yet, one byte per node
    __device__ inline void carve(const Fwd &, unsigned char *lds, int n, int, int)
    {
        cnt = reinterpret_cast<unsigned *>(lds);
        par = reinterpret_cast<T *>(lds + ((n + 3) & ~3));
        pool = reinterpret_cast<T *>(lds + ((n + 3) & ~3) + ((2 * n + 3) & ~3));
        start = pool + (n / 2 + 1);
    }
    __device__ inline void set_node(int i, int p, int pend)
    {
        par[i] = p < 0 ? (T)NONE : (T)p;
        reinterpret_cast<unsigned char *>(cnt)[i] = (unsigned char)pend;
    }
    __device__ inline int parent(int i) const { return par[i] == (T)NONE ? -1 : (int)par[i]; }
    __device__ inline int count_down(int i) { return (int)(atomicSub(&cnt[i >> 2], 1u << (8 * (i & 3))) >> (8 * (i & 3)) & 0xFFu); }
    __device__ inline int node(int pos) const { return pool[pos]; }
    __device__ inline void list(int pos, int i) { pool[pos] = (T)i; }
    __device__ inline void block(int b, int pos, bool late) { start[b] = (T)((unsigned)pos | (late ? LATE : 0u)); }
    __device__ inline int block_start(int b) const { return start[b] & 0x7FFF; }
    __device__ inline bool block_late(int b) const { return (start[b] & LATE) != 0u; }
    __device__ inline void settle() const { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }
};
template <> struct SchedLists<false> {
    int32_t *par, *pool, *cnt;
    unsigned *start;
    int nb;
    __device__ inline void carve(const Fwd &f, unsigned char *, int, int nb_, int first)
    {
        nb = nb_;
        par = f.parent + nb;
        cnt = f.arrive + nb;
        pool = f.level_nodes + first;
        start = reinterpret_cast<unsigned *>(f.level_fill) + first;
    }
    __device__ inline void set_node(int i, int, int pend) { st_dev(&cnt[i], pend); }
    __device__ inline int parent(int i) const { const int p = par[i]; return p < 0 ? -1 : p - nb; }
    __device__ inline int count_down(int i) { return add_dev(&cnt[i], -1); }
    __device__ inline int node(int pos) const { return ld_dev(&pool[pos]); }
    __device__ inline void list(int pos, int i) { st_dev(&pool[pos], (int32_t)i); }
    __device__ inline void block(int b, int pos, bool late) { st_dev(&start[b], (unsigned)pos | (late ? SCHED_LATE : 0u)); }
    __device__ inline int block_start(int b) const { return (int)(ld_dev(&start[b]) & ~SCHED_LATE); }
    __device__ inline bool block_late(int b) const { return (ld_dev(&start[b]) & SCHED_LATE) != 0u; }
    __device__ inline void settle() const { wait_mem(); }
};

// The part of the batch that belongs to a slot: trees [t_lo, t_hi), cut where the node count passes slot / n_slots of the batch.
// Both cuts are looked for at once, lanes 0-31 of every wave for this slot's and lanes 32-63 for the next one's, 32
// candidates per round trip (a bisection is one dependent load per halving).  The offsets at the cuts are among what has been read.
__device__ inline void flow_cut(const Fwd &f, int slot, int n_slots, int *t_lo, int *t_hi, int *n_lo, int *n_hi)
{
    const int lane = threadIdx.x & 63, half = lane >> 5, i = lane & 31;
    const long long bound = ((long long)(slot + half) * f.n_nodes + n_slots - 1) / n_slots;
    int lo = 0, hi = f.n_trees;                   // smallest t with tree_off[t] >= bound is in [lo, hi]; tree_off[n_trees] = n_nodes >= bound
    int at_hi = f.n_nodes;                        // tree_off[hi]
    while (__ballot(lo < hi) != 0ull) {
        const int step = (hi - lo + 30) / 31;     // candidates lo, lo + step, ..., the last one clamped to hi
        const int cand = min(lo + i * step, hi);
        const int off = cand >= hi ? at_hi : f.tree_off[cand];
        const bool ge = cand >= hi || off >= bound;                                 // (at hi it holds by the invariant)
        const unsigned long long m = __ballot(ge) >> (32 * half) & 0xFFFFFFFFull;   // never empty: the last candidate is hi
        const int k = __builtin_ctzll(m);         // first candidate at or above the cut
        const int off_k = __shfl(off, 32 * half + k);
        if (lo < hi) {
            const int new_hi = min(lo + k * step, hi);
            lo = k == 0 ? lo : min(lo + (k - 1) * step, hi) + 1;                    // (k == 0: the cut is lo itself)
            hi = new_hi;
            at_hi = off_k;
        }
    }
    *t_lo = __builtin_amdgcn_readlane(lo, 0);     // (scalar values, like everything derived from them)
    *t_hi = __builtin_amdgcn_readlane(lo, 32);
    *n_lo = __builtin_amdgcn_readlane(at_hi, 0);
    *n_hi = __builtin_amdgcn_readlane(at_hi, 32);
}

template <bool IN_LDS, bool PLACES>
__device__ inline void flow_schedule_slot(const Fwd &f, const SchedPlaces &sp, int slot, int t_lo, int t_hi, int nb, int ne, unsigned char *lds)
{
    const int tid = threadIdx.x, lane = tid & 63, n = ne - nb, first = (nb - t_lo) / 2;
    const int cap = (n - (t_hi - t_lo)) / 2;      // internal nodes (full binary trees)
    int *s_ctl = reinterpret_cast<int *>(lds);    // leave (read) | roots, later nodes handed out | blocks | a tree of one node exists
    SchedLists<IN_LDS> q;
    constexpr int Q = 4;
    int *s_cnt = s_ctl + 4;                       // seeds of a pass, [Q][waves]
    q.carve(f, lds + 16 + 4 * Q * 4, n, nb, first);
    int n_seeds = 0;
    for (int base = 0; base < n; base += WG_THREADS * Q) {
        int l[Q], up[Q], pend[Q];
        unsigned seeds = 0u;
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            const int i = min(base + j * WG_THREADS + tid, n - 1);
            l[j] = f.left[nb + i];
            up[j] = f.parent[nb + i];
            pend[j] = f.pending[nb + i];
        }
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            const int i = base + j * WG_THREADS + tid;
            const bool here = i < n;
            if (here) q.set_node(i, up[j] < 0 ? -1 : up[j] - nb, pend[j]);
            const bool seed = here && l[j] >= 0 && pend[j] == 0;
            seeds |= (seed ? 1u : 0u) << j;
            const unsigned long long m = __ballot(seed);
            if (lane == 0) s_cnt[j * 4 + (tid >> 6)] = __popcll(m);
            if (f.flow_roots && here && up[j] < 0) {
                // a root: one per tree (a second one of a tree is found here, a missing one by the count)
                atomicAdd(&s_ctl[1], 1);
                const int t = t_lo + tree_of(f.tree_off + t_lo, t_hi - t_lo, nb + i);
                f.depth_root[nb + i] = t;
                if (f.root_out) f.root_out[t] = nb + i;
                if (l[j] < 0) atomicOr(&s_ctl[3], 1);
                if (atomicCAS(&f.root_ws[t], -1, nb + i) != -1) latch_error(f.ctl, TL_ESTRUCT);
            }
        }
        __syncthreads();
        // in node order, so that the schedule is the same every time
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            const unsigned long long m = __ballot(seeds >> j & 1u);
            int pos = n_seeds + __popcll(m & ((1ull << lane) - 1ull));
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int c = s_cnt[j * 4 + k];
                if (k < (tid >> 6)) pos += c;
                n_seeds += c;
            }
            if ((seeds >> j & 1u) && pos < cap) q.list(pos, base + j * WG_THREADS + tid);
        }
        __syncthreads();
    }
    wait_mem();
    __syncthreads();
    if (tid < 64) {
        int head = 0, tail = min(n_seeds, cap), blocks = 0, rounds = 0;
        int fresh = cap;                          // list positions from here on became ready in the round before
        // hands out this lane's node: does its parent p become ready with it (said by one of two siblings)?
        auto hand_out = [&](int p) {
            bool ready = false;
            int old = 0;
            if (p >= 0) {
                old = q.count_down(p);
                ready = old == 1;
            }
            if constexpr (!IN_LDS) {
                // Siblings handed out together: which of them memory counts second is not fixed, the higher lane lists the parent.
                // (In LDS the lanes of one instruction are served in order.)
                unsigned long long first_of_two = __ballot(old == 2);
                while (first_of_two != 0ull) {
                    const int k = __builtin_ctzll(first_of_two);
                    first_of_two &= first_of_two - 1ull;
                    const unsigned long long pair = __ballot(p >= 0 && p == __shfl(p, k));
                    if (__popcll(pair) == 2 && (pair >> lane & 1ull)) ready = lane == 63 - __builtin_clzll(pair);
                }
            }
            return ready;
        };
        while (head < tail) {
            int take = min(tail - head, 64);
            if (take > 16) take &= ~15;
            const bool mine = lane < take;
            int p = -1;
            if (mine) p = q.parent(q.node(head + lane));
            bool ready = hand_out(p);
            unsigned long long m = __ballot(ready);
            const int pos = tail + __popcll(m & ((1ull << lane) - 1ull));
            if (ready && pos < cap) q.list(pos, p);
            if (lane * 16 < take) q.block(blocks + lane, head + lane * 16, lane == 0 && head + min(take, 16) > fresh);
            fresh = tail;
            blocks += (take + 15) >> 4;
            head += take;
            tail = min(tail + __popcll(m), cap);
            rounds += 1;
            if (head == fresh && __popcll(m) <= 16) {
                // Nothing waits but the few nodes that this round made ready: the rounds of a deep tree.  They stay in the lanes
                // that found them, and a node's parent is looked up beside the count that makes the node ready: a round is one
                // LDS access deep.
                int up = ready ? q.parent(p) : -1;
                while (m != 0ull && __popcll(m) <= 16 && head < tail) {
                    if (lane == 0) q.block(blocks, head, true);
                    const int above = up >= 0 ? q.parent(up) : -1;
                    ready = hand_out(up);
                    m = __ballot(ready);
                    const int at = tail + __popcll(m & ((1ull << lane) - 1ull));
                    if (ready && at < cap) q.list(at, up);
                    fresh = tail;
                    blocks += 1;
                    head = tail;
                    tail = min(tail + __popcll(m), cap);
                    rounds += 1;
                    up = ready ? above : -1;
                }
            }
            q.settle();
        }
        if (lane == 0) {
            s_ctl[2] = blocks;
            f.sched_head[slot] = int4{first, blocks, t_lo, s_ctl[3] != 0 ? t_hi : t_lo};
            atomicMax(&f.ctl->n_levels, rounds + 1);
            // nodes that never became ready (a cycle), or a tree without a root
            if (head < cap || (f.flow_roots && s_ctl[1] != t_hi - t_lo)) latch_error(f.ctl, TL_ESTRUCT);
            s_ctl[1] = head;
        }
    }
    __syncthreads();
    // the blocks' entries; rows beyond a block's nodes stand in with the sources of its first row: they are requested like
    // the others (a request needs no test), so they must be rows that do become valid
    const int blocks = s_ctl[2], handed = s_ctl[1];
    int4 *out = f.sched + (size_t)first * 16;
#pragma unroll 4
    for (int i = tid; i < blocks * 16; i += WG_THREADS) {
        const int b = i >> 4, r = i & 15;
        const int st = q.block_start(b), end = b + 1 < blocks ? q.block_start(b + 1) : handed;
        const bool here = st + r < end;
        const int node = nb + q.node(here ? st + r : st);
        int w = q.block_late(b) ? (int)SCHED_LATE : 0;
        // (asked for together: only a root's tree is there)
        const int up = f.parent[node], tree = f.flow_roots ? ld_dev(&f.depth_root[node]) : 0;
        if (f.flow_roots && here && up < 0) w |= tree + 1;
        out[i] = int4{here ? node : -1, f.left[node], f.right[node], w};
        if (PLACES && here) sp.of[node] = int2{first + st, (end - st) | r << 8};
    }
    if constexpr (!PLACES) return;
    // (leaves' places are written by other workgroups)
    wait_mem();
    __syncthreads();
    auto place = [&](int n) {
        if (f.left[n] < 0) return pack2(0xFFFFFFFFu, 0u);
        return ld_dev(reinterpret_cast<const unsigned long long *>(sp.of + n));
    };
    int4 *places = sp.children + (size_t)first * 16;
#pragma unroll 4
    for (int i = tid; i < blocks * 16; i += WG_THREADS) {
        const unsigned long long l = place(out[i].y), r = place(out[i].z);      // (this thread's own entry)
        places[i] = int4{(int)(unsigned)l, (int)(unsigned)(l >> 32), (int)(unsigned)r, (int)(unsigned)(r >> 32)};
    }
}
template <bool PLACES = false>
__device__ inline void flow_schedule(const Fwd &f, int slot, unsigned char *lds, size_t lds_bytes, const SchedPlaces &sp = SchedPlaces{})
{
    // (workgroups of other slots may latch an error meanwhile)
    int *s_ctl = reinterpret_cast<int *>(lds);
    if (threadIdx.x >= 1 && threadIdx.x < 4) s_ctl[threadIdx.x] = 0;
    // the cuts first: what they read of a batch that is rejected is not used, and the status arrives beside it
    const bool leave = threadIdx.x == 0 && (batch_rejected(f) || (PLACES ? back_by_heights(f) : internal_kernel_skipped(f)));
    int t_lo, t_hi, nb, ne;
    flow_cut(f, slot, f.n_slots, &t_lo, &t_hi, &nb, &ne);
    if (decided_to_leave(&s_ctl[0], leave)) return;
    if (ne <= nb) {
        if (threadIdx.x == 0) {
            f.sched_head[slot] = int4{0, 0, 0, 0};
            if (PLACES) sp.trees[slot] = int4{0, 0, 0, 0};
        }
        return;
    }
    if (PLACES && threadIdx.x == 0) sp.trees[slot] = int4{t_lo, t_hi, (ne - nb - (t_hi - t_lo)) / 2, (nb - t_lo) / 2};
    if (ne - nb < 0xFFFF && sched_lds_bytes((size_t)(ne - nb)) <= lds_bytes) flow_schedule_slot<true, PLACES>(f, sp, slot, t_lo, t_hi, nb, ne, lds);
    else flow_schedule_slot<false, PLACES>(f, sp, slot, t_lo, t_hi, nb, ne, lds);
}
// As a launch of its own, where the leaves are evaluated by a kernel that does not do it on the side.

__global__ __launch_bounds__(WG_THREADS) void k_flow_schedule(Fwd f)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    flow_schedule(f, blockIdx.x, smem_raw, SCHED_LDS_BYTES);
}

}  // namespace tl
