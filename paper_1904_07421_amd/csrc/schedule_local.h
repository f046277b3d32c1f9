// The schedule of a forest whose trees are filed one after another, analysed in LDS (part of schedule.hip).
//
// Batches are made by laying trees out one after another, so a node's parent, children and level-mates of the
// same tree have ids close to its own.  Where that holds, everything but the place of a run of trees in the whole
// table can be worked out by one block in LDS: heights, child lists, the rank of a node among those of its level.
// A CUT is an id i that no edge crosses (no v with min(v, parent) < i <= max(v, parent)): the trees before and
// after it are independent.  Block b takes the ids from the first cut at or after b W to the first cut at or
// after (b + 1) W; neighbours find the same cuts because both look at every edge that could cross them.
//
//   window_kernel   per block: cuts, child counts, heights (pointer jumping), child lists, rank of every node
//                   among the block's nodes of equal key, and the block's key histogram
//   prefix_kernel   per key: exclusive scan of the histogram over the blocks (and the sums the host is told)
//   place_kernel    per block: key starts + prefix + rank = position; perm, inv_perm, child_ptr, child_idx
//
// Four launches (report_done_kernel, one store, is the last) and one wait of the host instead of about sixty launches
// and two; a forest of up to kWholeNodes nodes is ONE launch of one block (window_kernel with WHOLE: no cuts needed, so
// any order of ids will do).  What does not fit (an edge longer than M ids, no cut within M ids, more than kMaxArity
// children, more keys than the tables hold) takes the general path; nothing here reads or writes out of bounds for any
// parent array.
//
// The try must cost such a forest little.  A window that sees a misfit stops there and sets a word in pinned memory, and the
// host, which watches that word too, enqueues the general path behind the kernels that are still draining.  A table of so
// many signatures that two levels of it have more keys than the tables hold is not tried.  Call to return, us, general path
// alone / behind a try that runs to its end / as it is (the general path's own waits take 15 us each off): scrambled ids,
// 10.8 k nodes 210 / 230 / 165, 108 k 305 / 329 / 255, 2.36 M 746 / 818 / 727; 200 k nodes in trees of 1000 389 / 418 / 344;
// stars of 350 and chains of 350, 105 k nodes, 290 / 315 / 244 and 416 / 445 / 376; chains of 2000, 8 k nodes, 251 / 284 / 243;
// 108 k nodes under 24 and 64 signatures 375 / 403 / 304 and 383 / 404 / 353.
//
// Every step is bound by LDS latency and barriers, not by memory: the parent array is read (W + 3 M) / W times
// (W = 2048 for large forests: 1.75), each output is written once.  Measured, call to return, general path ->
// here: 74 nodes 131 -> 21 us, 4.7 k 162 -> 40, 106 k 313 -> 33, 192 k (128 levels) 374 -> 55, 2.36 M 560 -> 123.
#pragma once

#include <atomic>
#include <mutex>
#include <string.h>
#include <vector>

namespace jitdb {
namespace {

constexpr int kLocThreads = 1024;
constexpr int kLocWaves = kLocThreads / 64;
constexpr int kLocSpan = 512;            // M: the longest edge, and the farthest cut from its window's start
constexpr int kMaxArity = 256;           // siblings are ranked by counting: quadratic in the list's length
constexpr int kKeysPlain = 256;          // levels a forest over several windows may have
constexpr int kKeysTyped = 1024;         // (height, signature, parent's signature) keys; also the levels of a one-block forest
constexpr int kWholeNodes = 8192;
constexpr int kReportKeys = kWholeNodes; // what a report has room for: every level of a forest of one block, chains too
constexpr uint16_t kNoParent = 0xFFFF;

enum : int { LF_RANGE = 1, LF_SIG = 2, LF_CYCLE = 4, LF_GENERAL = 8 };

// Words the host reads, in pinned memory: written by the last kernel, valid once the stream is done.
struct LocalReport {
    int32_t done;                            // set last (report_done_kernel, or the one block of a small forest)
    int32_t misfit;                          // set by any window whose ids do not fit, long before `done`
    int32_t step;                            // general path: how many of its two reports are there (report_words_kernel)
    int32_t meta[META_WORDS];                // ... the first
    int32_t flags, n_levels, n_edges, tree_window;
    int32_t level_ptr[kKeysTyped + 1];
    int32_t kids[kReportKeys];
    int32_t slot_ptr[kReportKeys + 1];
};

struct LocalArgs {
    const int32_t *parent, *sig;
    int32_t n, n_sig;
    int32_t *height, *level_ptr, *perm, *inv_perm, *child_ptr, *child_idx, *key, *slot_ptr;
    int64_t slot_capacity;
    // between the kernels (several windows)
    int32_t nb, n_keys_max;                  // windows; rows of hist
    int32_t *hist;                           // [n_keys_max][nb] nodes per key, then their exclusive prefix over the blocks
    int32_t *kid_hist;                       // [kKeysPlain][nb] children by the height of the parent
    int32_t *first, *count, *edges, *maxh, *flags, *gap;   // [nb] per window
    int32_t *edge_base;                      // [nb] exclusive prefix of edges
    int32_t *key_total, *kid_total;          // [n_keys_max], [kKeysPlain]
    int32_t *meta;                           // flags, max height, edges, largest distance between cuts; `call` once a window misfits
    int32_t call;                            // differs from call to call: what meta[4] holds from before is another number
    uint16_t *rank;                          // [n] rank among the window's nodes of equal key
    int32_t *child_tmp;                      // [n] child lists, window after window
    LocalReport *report;                     // pinned host memory
};

__device__ __forceinline__ int loc_wave_incl_scan(int v) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int t = __shfl_up(v, d, 64);
        if (lane >= d) v += t;
    }
    return v;
}

// Exclusive prefix of one value per thread over the block's 1024 threads (s: kLocWaves words).
__device__ __forceinline__ int loc_block_excl_scan(int v, int *s, int &total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int inc = loc_wave_incl_scan(v);
    __syncthreads();
    if (lane == 63) s[wave] = inc;
    __syncthreads();
    int before = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < kLocWaves; ++w) {
        const int x = s[w];
        if (w < wave) before += x;
        total += x;
    }
    return before + inc - v;
}

// Exclusive prefix maximum over the block (-1 before the first thread).
__device__ __forceinline__ int loc_block_excl_max(int v, int *s) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int t = __shfl_up(inc, d, 64);
        if (lane >= d) inc = max(inc, t);
    }
    int ex = __shfl_up(inc, 1, 64);
    if (lane == 0) ex = -1;
    __syncthreads();
    if (lane == 63) s[wave] = inc;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kLocWaves; ++w)
        if (w < wave) ex = max(ex, s[w]);
    return ex;
}

// W: ids per window; CAP: nodes a block may own; KEYS: keys it can count; WHOLE: the only block, all n <= CAP nodes.
template <int W, int CAP, int KEYS, bool WHOLE>
__global__ void __launch_bounds__(kLocThreads)
window_kernel(const LocalArgs a) {
    constexpr int M = kLocSpan;
    constexpr int RANGE = WHOLE ? CAP : W + 3 * M;                           // ids the block looks at
    constexpr int RIT = (RANGE + 1 + kLocThreads - 1) / kLocThreads;        // scan positions per thread
    constexpr int IT = CAP / kLocThreads;                                   // own nodes per thread
    static_assert(CAP % kLocThreads == 0 && (WHOLE || CAP >= W + M), "whole rounds; room for the largest own range");
    static_assert(CAP < kNoParent, "local ids are 16 bits");
    // The cover scan's words are dead before the key counters are filled; the pointers of the jumping before
    // the child lists are.
    constexpr int kCoverBytes = RIT * kLocThreads * 4, kCountBytes = kLocWaves * KEYS * 2;
    __shared__ __attribute__((aligned(16))) char s_u[kCoverBytes > kCountBytes ? kCoverBytes : kCountBytes];
    __shared__ uint16_t s_par[CAP];
    __shared__ uint16_t s_anc[2][CAP];
    __shared__ int s_hgt[CAP];
    __shared__ int s_cnt[CAP];
    __shared__ int s_kid[KEYS];
    __shared__ int s_scan[kLocWaves];
    __shared__ int s_lo, s_hi, s_gap, s_flags, s_maxh;
    int *cover = reinterpret_cast<int *>(s_u);
    uint16_t *wave_cnt = reinterpret_cast<uint16_t *>(s_u);                  // [wave][key]

    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, b = blockIdx.x;
    const int n = a.n;
    const int64_t i0 = WHOLE ? 0 : (int64_t)b * W;                          // this window's start and the next one's
    const int64_t i1 = WHOLE ? n : (i0 + W < n ? i0 + W : n);
    const int64_t base = WHOLE ? 0 : i0 - M;                                // id of scan position 0
    const int ns2 = a.n_sig * a.n_sig;
    // The first window to come here tells the host (a thousand stores to one word of its memory hold up the kernel's end)
    auto tell_misfit = [&]() __attribute__((always_inline)) {
        if (atomicExch(&a.meta[4], a.call) != a.call) __hip_atomic_store(&a.report->misfit, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    };
    // The whole block leaves: its ids do not fit (the general path looks for faults anew).
    auto leave = [&]() __attribute__((always_inline)) {
        if (t != 0) return;
        if constexpr (WHOLE) {
            a.report->flags = LF_GENERAL;
            __hip_atomic_store(&a.report->done, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        } else {
            a.first[b] = a.count[b] = a.edges[b] = a.gap[b] = 0;
            a.flags[b] = LF_GENERAL;
            a.maxh[b] = -1;
            tell_misfit();
        }
    };
    if (t == 0) { s_lo = INT32_MAX; s_hi = INT32_MAX; s_gap = 0; s_flags = 0; s_maxh = 0; }
#pragma unroll
    for (int r = 0; r < RIT; ++r) cover[r * kLocThreads + t] = 0;
    __syncthreads();

    // ---- validity, and how many edges cross every position: +1 behind the lower end, -1 behind the upper one
    int flags = 0;
    auto add_edge = [&](int64_t v, int p) __attribute__((always_inline)) {
        const bool bad = p < -1 || p >= n || p == (int)v;
        const bool mine = v >= i0 && v < i1;
        if (bad) {
            if (mine) flags |= LF_RANGE;
            return;
        }
        if (p < 0) return;
        int64_t lo = (v < p ? v : p) + 1 - base, hi = (v < p ? p : v) + 1 - base;
        if (!WHOLE) {
            if (hi - lo > M && mine) flags |= LF_GENERAL;
            lo = lo < 0 ? 0 : lo;
            hi = hi < 0 ? 0 : hi;
        }
        if (lo <= RANGE) atomicAdd(&cover[lo], 1);
        if (hi <= RANGE) atomicAdd(&cover[hi], -1);
    };
    {
        constexpr int LIT = (RANGE + kLocThreads - 1) / kLocThreads;
        int pv[LIT];
#pragma unroll
        for (int r = 0; r < LIT; ++r) {          // all loads in flight together
            const int64_t v = base + r * kLocThreads + t;
            pv[r] = (r * kLocThreads + t < RANGE && v >= 0 && v < n) ? a.parent[v] : -1;
        }
#pragma unroll
        for (int r = 0; r < LIT; ++r) add_edge(base + r * kLocThreads + t, pv[r]);
    }
    __syncthreads();
    {
        int d[RIT], sum = 0;
#pragma unroll
        for (int r = 0; r < RIT; ++r) { d[r] = cover[t * RIT + r]; sum += d[r]; }
        int total;
        int run = loc_block_excl_scan(sum, s_scan, total);
        int lo = INT32_MAX, hi = INT32_MAX, last = -1;
        bool cut[RIT];
#pragma unroll
        for (int r = 0; r < RIT; ++r) {
            run += d[r];
            const int64_t i = base + t * RIT + r;
            cut[r] = run == 0 && i >= i0 && i <= n && t * RIT + r <= (WHOLE ? RANGE : W + 2 * M);
            if (cut[r]) {
                if (lo == INT32_MAX) lo = (int)i;
                if (hi == INT32_MAX && i >= i1) hi = (int)i;
                last = (int)i;
            }
        }
        if (flags & LF_GENERAL) s_lo = INT32_MIN;          // an edge too long (a store: no atomicMin beside it undoes it)
        else if (lo != INT32_MAX) atomicMin(&s_lo, lo);
        if (hi != INT32_MAX) atomicMin(&s_hi, hi);
        int prev = loc_block_excl_max(last, s_scan);      // (its barriers also publish s_lo, s_hi)
        int gap = 0;
#pragma unroll
        for (int r = 0; r < RIT; ++r) {
            if (!cut[r]) continue;
            const int i = (int)(base + t * RIT + r);
            if (i > s_hi) break;
            if (prev >= 0) gap = max(gap, i - prev);
            prev = i;
        }
        if (gap) atomicMax(&s_gap, gap);
    }
    __syncthreads();
    int lo = __builtin_amdgcn_readfirstlane(s_lo), hi = __builtin_amdgcn_readfirstlane(s_hi);
    if constexpr (WHOLE) {
        lo = 0; hi = n;
    } else if (lo == INT32_MIN || lo == INT32_MAX || hi == INT32_MAX || lo >= i0 + M || hi > i1 + M || hi - lo > CAP) {
        leave();
        return;
    }
    const int own = hi - lo;

    // ---- the block's own nodes by local id
    {
        int pv[IT];
#pragma unroll
        for (int r = 0; r < IT; ++r) pv[r] = r * kLocThreads + t < own ? a.parent[lo + r * kLocThreads + t] : -1;
#pragma unroll
        for (int r = 0; r < IT; ++r) {
            const int i = r * kLocThreads + t, p = pv[r];
            uint16_t lp = kNoParent;
            if (p >= lo && p < hi && p != lo + i) lp = (uint16_t)(p - lo);
            else if (p >= 0) flags |= LF_GENERAL;         // (an invalid one has set LF_RANGE where it is checked)
            s_par[i] = lp;
            s_anc[0][i] = lp;
            s_hgt[i] = 0;
            s_cnt[i] = 0;
        }
    }
    // signatures here and not with the keys, which a block with a cycle does not reach: a bad one is reported first
    if (a.sig) {
#pragma unroll
        for (int r = 0; r < IT; ++r) {
            const int i = r * kLocThreads + t;
            if (i < own && (a.sig[lo + i] < 0 || a.sig[lo + i] >= a.n_sig)) flags |= LF_SIG;
        }
    }
    if (t < KEYS) s_kid[t] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < IT; ++r) {
        const uint16_t lp = s_par[r * kLocThreads + t];
        if (lp != kNoParent) atomicAdd(&s_cnt[lp], 1);
    }

    // ---- heights by pointer jumping (see jump_kernel): a pointer still alive after the last round means a cycle
    int rounds = 0;
    while ((1 << rounds) < own) ++rounds;
    int live = 0;
    for (int k = 0; k < rounds; ++k) {
        const uint16_t *in = s_anc[k & 1];
        uint16_t *out = s_anc[(k + 1) & 1];
        live = 0;
        uint16_t p[IT], next[IT];
        int h[IT];
#pragma unroll
        for (int r = 0; r < IT; ++r) {                    // (nodes past the block's own have no parent)
            p[r] = in[r * kLocThreads + t];
            h[r] = __atomic_load_n(&s_hgt[r * kLocThreads + t], __ATOMIC_RELAXED);
        }
#pragma unroll
        for (int r = 0; r < IT; ++r) next[r] = p[r] != kNoParent ? in[p[r]] : kNoParent;
#pragma unroll
        for (int r = 0; r < IT; ++r) {
            if (p[r] != kNoParent) atomicMax(&s_hgt[p[r]], h[r] + (1 << k));
            live |= next[r] != kNoParent;
            out[r * kLocThreads + t] = next[r];
        }
        live = __builtin_amdgcn_readfirstlane(__syncthreads_or(live));
        if (!live) break;
    }
    if (live) flags |= LF_CYCLE;

    // ---- child lists: start of every list by a scan of the counts, lists filled in any order, every node's place
    //      in its parent's list = the number of siblings with a smaller id
    int n_edges;
    {
        int c[IT], sum = 0;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < IT; ++r) {
            c[r] = s_cnt[t * IT + r];
            if (c[r] > kMaxArity) flags |= LF_GENERAL;
            sum += c[r];
        }
        int run = loc_block_excl_scan(sum, s_scan, n_edges);
        int m = 0;
#pragma unroll
        for (int r = 0; r < IT; ++r) {
            const int i = t * IT + r;
            s_cnt[i] = run;                                // becomes the list's end while it is filled
            run += c[r];
            if (i < own) {
                const int hgt = s_hgt[i];
                m = max(m, hgt);
                if (c[r] && hgt < KEYS) atomicAdd(&s_kid[hgt], c[r]);
            }
        }
        if (m) atomicMax(&s_maxh, m);
    }
    if (flags) atomicOr(&s_flags, flags);
    __syncthreads();
    flags = s_flags;
    const int maxh = s_maxh;
    if (own > 0 && ((int64_t)(maxh + 1) * ns2 > KEYS || (!WHOLE && maxh >= kKeysPlain))) flags |= LF_GENERAL;
    const int n_keys = own > 0 && flags == 0 ? (maxh + 1) * ns2 : 0;
    uint16_t *list = s_anc[0];
    if (flags == 0) {
#pragma unroll
        for (int r = 0; r < IT; ++r) {
            const int i = r * kLocThreads + t;
            const uint16_t lp = s_par[i];
            if (lp != kNoParent) list[atomicAdd(&s_cnt[lp], 1)] = (uint16_t)i;
        }
    }
    __syncthreads();
    int32_t *child_dst = WHOLE ? a.child_idx : a.child_tmp + lo;
    // keys and the rank of every node among the block's nodes of the same key, in id order: a wave owns 64 IT
    // consecutive nodes and visits them 64 at a time (as in radix_scatter_kernel)
    for (int k = t; k < kLocWaves * n_keys; k += kLocThreads) wave_cnt[(k / n_keys) * KEYS + k % n_keys] = 0;
    int bits = 1;
    while ((1 << bits) < n_keys) ++bits;
    if (flags == 0) {
#pragma unroll
        for (int r = 0; r < IT; ++r) {
            const int i = r * kLocThreads + t;
            if (i >= own) break;
            const uint16_t lp = s_par[i];
            if (lp != kNoParent) {
                const int l0 = lp ? s_cnt[lp - 1] : 0, l1 = s_cnt[lp];
                int slot = l0;
                for (int e = l0; e < l1; ++e) slot += list[e] < i;
                child_dst[slot] = lo + i;
            }
            a.child_ptr[lo + i] = i ? s_cnt[i - 1] : 0;    // (relative to the window until place_kernel)
            a.height[lo + i] = s_hgt[i];
        }
    }
    __syncthreads();
    uint16_t *keys = s_anc[1];
    if (flags == 0) {
#pragma unroll
        for (int r = 0; r < IT; ++r) {
            const int i = r * kLocThreads + t;
            if (i >= own) break;
            int key = s_hgt[i];
            if (a.sig) {
                const uint16_t lp = s_par[i];
                const int sg = a.sig[lo + i], ps = lp != kNoParent ? a.sig[lo + lp] : sg;
                key = (key * a.n_sig + sg) * a.n_sig + ps;
                a.key[lo + i] = key;
            }
            keys[i] = (uint16_t)key;
        }
    }
    __syncthreads();
    int rank[IT], dk[IT];
#pragma unroll
    for (int r = 0; r < IT; ++r) {
        const int i = wave * (64 * IT) + r * 64 + lane;
        dk[r] = i < own && flags == 0 ? keys[i] : 0;
    }
    const unsigned long long below = (1ull << lane) - 1ull;
    volatile uint16_t *my_cnt = wave_cnt + wave * KEYS;
    if (flags == 0) {
#pragma unroll
        for (int r = 0; r < IT; ++r) {
            const bool valid = wave * (64 * IT) + r * 64 + lane < own;
            const int d = dk[r];
            unsigned long long same = __ballot(valid);
            for (int q = 0; q < bits; ++q) {
                const bool bit = (d >> q) & 1;
                const unsigned long long bal = __ballot(bit);
                same &= bit ? bal : ~bal;
            }
            rank[r] = 0;
            if (valid) {
                const int prev = my_cnt[d];
                rank[r] = prev + (int)__popcll(same & below);
                __builtin_amdgcn_wave_barrier();
                if ((same & below) == 0) my_cnt[d] = (uint16_t)(prev + (int)__popcll(same));
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
    __syncthreads();
    int total = 0;
    if (t < n_keys) {
#pragma unroll
        for (int w = 0; w < kLocWaves; ++w) {
            const int c = wave_cnt[w * KEYS + t];
            wave_cnt[w * KEYS + t] = (uint16_t)total;
            total += c;
        }
    }
    if constexpr (!WHOLE) {
        __syncthreads();
        if (t < n_keys) a.hist[(int64_t)t * a.nb + b] = total;
        if (flags == 0 && own > 0 && t <= maxh) a.kid_hist[(int64_t)t * a.nb + b] = s_kid[t];
        if (t == 0) {
            a.first[b] = lo; a.count[b] = own; a.edges[b] = n_edges; a.flags[b] = flags; a.gap[b] = s_gap;
            a.maxh[b] = own > 0 && flags == 0 ? maxh : -1;
            if (flags & LF_GENERAL) tell_misfit();
        }
        if (flags == 0) {
#pragma unroll
            for (int r = 0; r < IT; ++r) {
                const int i = wave * (64 * IT) + r * 64 + lane;
                if (i < own) a.rank[lo + i] = (uint16_t)(wave_cnt[wave * KEYS + dk[r]] + rank[r]);
            }
        }
    } else {
        int sum;
        const int start = loc_block_excl_scan(total, s_scan, sum);
        int *key_start = s_cnt;                            // the child lists' ends have been written out
        if (t < n_keys) key_start[t] = start;
        if (t == 0) key_start[n_keys] = n;
        __syncthreads();
        const int L = maxh + 1;
        LocalReport *rep = a.report;
        if (a.sig && (int64_t)n_keys + 1 > a.slot_capacity) flags |= LF_GENERAL;   // the general path reports it
        if (flags == 0) {
#pragma unroll
            for (int r = 0; r < IT; ++r) {
                const int i = wave * (64 * IT) + r * 64 + lane;
                if (i >= own) continue;
                const int pos = key_start[dk[r]] + wave_cnt[wave * KEYS + dk[r]] + rank[r];
                a.perm[pos] = i;
                a.inv_perm[i] = pos;
            }
            if (t == 0) a.child_ptr[n] = n_edges;
            for (int l = t; l <= L; l += kLocThreads) {
                const int v = key_start[l * ns2];
                a.level_ptr[l] = v;
                rep->level_ptr[l] = v;
                if (l < L) rep->kids[l] = s_kid[l];
            }
            if (a.sig)
                for (int k = t; k <= n_keys; k += kLocThreads) {
                    a.slot_ptr[k] = key_start[k];
                    rep->slot_ptr[k] = key_start[k];
                }
        }
        if (t == 0) {
            rep->flags = flags; rep->n_levels = L; rep->n_edges = n_edges; rep->tree_window = s_gap;
        }
        __threadfence_system();      // every thread's stores are out before the host is told
        __syncthreads();
        if (t == 0) __hip_atomic_store(&rep->done, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// Behind the last kernel of an analysis: the kernels before it are complete when it runs.
__global__ void report_done_kernel(LocalReport *rep) {
    if (threadIdx.x == 0) __hip_atomic_store(&rep->done, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// One block: up to two arrays of the general path's into a report, then its step.
__global__ void __launch_bounds__(kLocThreads)
report_words_kernel(const int32_t *from0, int n0, int32_t *to0, const int32_t *from1, int n1, int32_t *to1, int32_t *step, int value) {
    for (int i = threadIdx.x; i < n0; i += kLocThreads) to0[i] = from0[i];
    for (int i = threadIdx.x; i < n1; i += kLocThreads) to1[i] = from1[i];
    __threadfence_system();
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(step, value, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Blocks [0, n_keys_max): exclusive scan of one key's row over the windows.  Blocks [n_keys_max, + kKeysPlain): sum of one
// level's children.  Last block: edges before every window, flags, largest height, largest distance between cuts.
__global__ void __launch_bounds__(kThreads)
prefix_kernel(const LocalArgs a) {
    const int row = blockIdx.x, t = threadIdx.x, nb = a.nb;
    const int ns2 = a.n_sig * a.n_sig;
    if (row < a.n_keys_max + kKeysPlain) {
        const bool keys = row < a.n_keys_max;
        const int k = keys ? row : row - a.n_keys_max;
        const int level = keys ? k / ns2 : k;
        int32_t *src = keys ? a.hist + (int64_t)k * nb : a.kid_hist + (int64_t)k * nb;
        int carry = 0;
        for (int base = 0; base < nb; base += kThreads) {
            const int i = base + t;
            const bool ok = i < nb && a.maxh[i] >= level;       // windows without this level have not written the entry
            const int v = ok ? src[i] : 0;
            int total;
            const int ex = block_exclusive_scan(v, &total);
            if (keys && i < nb) src[i] = carry + ex;
            carry += total;
        }
        if (t == 0) (keys ? a.key_total : a.kid_total)[k] = carry;
        return;
    }
    int carry = 0, fl = 0, mh = -1, gap = 0;
    for (int base = 0; base < nb; base += kThreads) {
        const int i = base + t;
        int v = 0;
        if (i < nb) {
            v = a.edges[i];
            fl |= a.flags[i];
            mh = max(mh, a.maxh[i]);
            gap = max(gap, a.gap[i]);
        }
        int total;
        const int ex = block_exclusive_scan(v, &total);
        if (i < nb) a.edge_base[i] = carry + ex;
        carry += total;
    }
    __shared__ int s_fl, s_mh, s_gap;
    if (t == 0) { s_fl = 0; s_mh = -1; s_gap = 0; }
    __syncthreads();
    if (fl) atomicOr(&s_fl, fl);
    atomicMax(&s_mh, mh);
    atomicMax(&s_gap, gap);
    __syncthreads();
    if (t == 0) { a.meta[0] = s_fl; a.meta[1] = s_mh; a.meta[2] = carry; a.meta[3] = s_gap; }
}

__global__ void __launch_bounds__(kLocThreads)
place_kernel(const LocalArgs a) {
    __shared__ int s_base[kKeysTyped + 1];
    __shared__ int s_scan[kLocWaves];
    const int t = threadIdx.x, b = blockIdx.x;
    const int ns2 = a.n_sig * a.n_sig;
    int flags = a.meta[0];
    const int L = a.meta[1] + 1, E = a.meta[2];
    if ((int64_t)L * ns2 > a.n_keys_max || (a.sig && (int64_t)L * ns2 + 1 > a.slot_capacity)) flags |= LF_GENERAL;
    if (b == 0 && t == 0) {
        a.report->flags = flags; a.report->n_levels = L; a.report->n_edges = E; a.report->tree_window = a.meta[3];
    }
    if (flags) return;
    const int S = L * ns2;
    int sum;
    const int start = loc_block_excl_scan(t < S ? a.key_total[t] : 0, s_scan, sum);
    if (b == 0) {                   // the table's boundaries, for the device and for the host
        if (t < S) s_base[t] = start;
        if (t == 0) s_base[S] = a.n;
        __syncthreads();
        for (int l = t; l <= L; l += kLocThreads) {
            const int v = s_base[l * ns2];
            a.level_ptr[l] = v;
            a.report->level_ptr[l] = v;
            if (l < L) a.report->kids[l] = a.kid_total[l];
        }
        if (a.sig)
            for (int k = t; k <= S; k += kLocThreads) {
                a.slot_ptr[k] = s_base[k];
                a.report->slot_ptr[k] = s_base[k];
            }
        if (t == 0) a.child_ptr[a.n] = E;
        __syncthreads();
    }
    if (t < S) s_base[t] = start + a.hist[(int64_t)t * a.nb + b];
    __syncthreads();
    const int lo = a.first[b], own = a.count[b], e0 = a.edge_base[b], ne = a.edges[b];
    const int32_t *key = a.sig ? a.key : a.height;
    for (int i = t; i < own; i += kLocThreads) {
        const int v = lo + i;
        const int pos = s_base[key[v]] + a.rank[v];
        a.perm[pos] = v;
        a.inv_perm[v] = pos;
        a.child_ptr[v] += e0;
        if (i < ne) a.child_idx[e0 + i] = a.child_tmp[lo + i];
    }
}

// ---- host side ---------------------------------------------------------------------------
// Reports in pinned memory.  A call takes one, its kernels write it, the call reads it after its synchronisation and
// gives it back.
using ReportPool = PinnedPool<LocalReport>;
inline ReportPool &report_pool() {
    static ReportPool *pool = new ReportPool();      // never destroyed: the runtime may be gone before static destructors run
    return *pool;
}

// ids per window: small windows keep all CUs busy with mid-sized forests, large ones read the overlap less often
// (100 k nodes: 512 -> 205 blocks; from 512 k nodes on a window of 2048 already gives a block per CU)
inline int local_window(int64_t n) { return n < 524288 ? 512 : 2048; }

struct LocalWs {
    LocalArgs a;
    size_t bytes;
};
inline LocalWs carve_local_ws(int64_t n, void *base, int64_t n_keys) {
    Carver c(base);
    LocalWs w = {};
    if (n <= kWholeNodes) return w;
    const int64_t nb = ceil_div(n, local_window(n));
    w.a.nb = (int32_t)nb;
    w.a.n_keys_max = n_keys > 1 ? kKeysTyped : kKeysPlain;
    w.a.hist = c.take<int32_t>((size_t)w.a.n_keys_max * nb);
    w.a.kid_hist = c.take<int32_t>((size_t)kKeysPlain * nb);
    int32_t **per_window[] = {&w.a.first, &w.a.count, &w.a.edges, &w.a.maxh, &w.a.flags, &w.a.gap, &w.a.edge_base};
    for (int32_t **p : per_window) *p = c.take<int32_t>(nb);
    w.a.key_total = c.take<int32_t>(w.a.n_keys_max);
    w.a.kid_total = c.take<int32_t>(kKeysPlain);
    w.a.meta = c.take<int32_t>(8);
    w.a.rank = c.take<uint16_t>(n);
    w.a.child_tmp = c.take<int32_t>(n);
    w.bytes = c.off;
    return w;
}

inline int launch_local_schedule(const LocalArgs &a, hipStream_t st) {
    if (a.n <= 1024 && a.n_sig == 1) {
        window_kernel<0, 1024, 256, true><<<1, kLocThreads, 0, st>>>(a);
        JITDB_LAUNCH_CHECK();
        return JITDB_OK;
    }
    if (a.n <= kWholeNodes) {        // (a block's time goes with the rounds it is compiled for)
        if (a.n <= 2048) window_kernel<0, 2048, kKeysTyped, true><<<1, kLocThreads, 0, st>>>(a);
        else if (a.n <= 5120) window_kernel<0, 5120, kKeysTyped, true><<<1, kLocThreads, 0, st>>>(a);
        else window_kernel<0, kWholeNodes, kKeysTyped, true><<<1, kLocThreads, 0, st>>>(a);
        JITDB_LAUNCH_CHECK();
        return JITDB_OK;
    }
    const bool typed = a.n_keys_max > kKeysPlain;
    if (local_window(a.n) == 512) {
        if (typed) window_kernel<512, 1024, kKeysTyped, false><<<a.nb, kLocThreads, 0, st>>>(a);
        else window_kernel<512, 1024, kKeysPlain, false><<<a.nb, kLocThreads, 0, st>>>(a);
    } else {
        if (typed) window_kernel<2048, 3072, kKeysTyped, false><<<a.nb, kLocThreads, 0, st>>>(a);
        else window_kernel<2048, 3072, kKeysPlain, false><<<a.nb, kLocThreads, 0, st>>>(a);
    }
    JITDB_LAUNCH_CHECK();
    prefix_kernel<<<a.n_keys_max + kKeysPlain + 1, kThreads, 0, st>>>(a);
    JITDB_LAUNCH_CHECK();
    place_kernel<<<a.nb, kLocThreads, 0, st>>>(a);
    JITDB_LAUNCH_CHECK();
    report_done_kernel<<<1, 64, 0, st>>>(a.report);
    JITDB_LAUNCH_CHECK();
    return JITDB_OK;
}

}  // namespace
}  // namespace jitdb
