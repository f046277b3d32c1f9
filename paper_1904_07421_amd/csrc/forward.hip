// jitdb_treelstm_forward: the execution half of the method for gfx950.
//
// The paper runs the look-up table slot by slot in depth order; per slot it
// stacks the samples, runs the shared subgraph once and slices the results
// (section 4.3).  Here a slot is one height level of the forest and the
// subgraph is the Child-Sum Tree-LSTM cell (section 3).  Per level:
//
//   stack_kernel       row r of the level's input matrix = [x_j | sum_k h_k] over the
//                      child CSR (the arity-dependent operator; HBM-bound, 16-byte
//                      coalesced row pieces)
//   level_kernel<LEAF|INTERNAL>   [x_j ; hs_j] x [W ; U]^T on MFMA with the whole cell
//                      fused into the epilogue: per-child forget gates from the
//                      precomputed P_k = U_f h_k, c_j and h_j written once
//   level_kernel<PROJ> P_k = U_f h_k for the nodes just produced, so that their
//                      parent reads one row per child (every non-root node is a
//                      child exactly once)
//   thin_kernel        the same three jobs for levels too small to fill the chip with
//                      128 x 256 tiles: one 32 x 32-unit tile per wave, operands straight
//                      from L2; a thin level's projection and the next level's stack
//                      step share one launch (thin_proj_stack_kernel)
//   chain_kernel       the thin levels whose nodes all have exactly one child (sequences, the long
//                      tail of a deep forest), many of them in one launch: x and the child's h read in place,
//                      all four gates over the full K, no stack step and no projection
//   tree_x_kernel, trees_kernel   (trees.hip) a forest of small trees filed one after another: all of the above in two launches
//
// With cells of different type in the table (jitdb_treelstm_forward_cells) a slot of N-ary cells
// runs nary_level_kernel below: the same GEMM core with the N-ary cell update as its epilogue.
// With a typed table (jitdb_treelstm_forward_typed) a slot is (level, signature): each
// signature has its own packed weights, the projection of a sub-slot uses the parent
// cell's, and the slots of a level run in one grouped launch (enter_range).
// gemm_kb_kernel is the same GEMM core as a plain C = A B^T.
//
// "Stack" is the row gather through perm (level-major order) done by
// stack_kernel, "slice" is the scatter of rows back to node-id order in the
// epilogue.
//
// Weights are re-packed once per call: gate rows of 32 hidden units are
// interleaved (i|o|u|f blocks of 32 rows), so that one wave holds all four
// gates of a hidden unit in its own accumulators and the cell update needs no
// exchange between lanes; rows and K are zero padded to tile multiples.

#include "tile_gemm.h"
#include "bounded_wait.h"

#include <mutex>
#include <vector>

namespace jitdb {
namespace {

// ---- weight packing ----------------------------------------------------------------
// Packed row r = tile*128 + gate*32 + uu holds gate `gate` of hidden unit tile*32 + uu as
// [ W row (D values, zero padded to Dp) | U row (H values, zero padded to Hp) ].  There are
// NPU >= NP rows; rows of units >= H are zero.
// Several cells that lie one behind the other (a typed table's) are packed in one launch.
struct PackArgs {
    const void *W, *U; const float *b;
    int D, H, Dp, Hp, NP, NPU, n_cells;
    void *Bp; float *bp;
};
__host__ __device__ __forceinline__ int64_t pack_pieces(int NPU, int Dp, int Hp, size_t esz) { return (int64_t)NPU * (Dp + Hp) * (int64_t)esz / 16; }

// block `block` of `n_blocks` (NT threads each, stride loop).  A thread writes sixteen bytes, in the order of the packed memory;
// their source is sixteen bytes of one row of W or U, on any element boundary.
template <typename T, int NT = kThreads>
__device__ __forceinline__ void pack_weights_body(const PackArgs &p, int64_t block, int64_t n_blocks) {
    constexpr int VEC = Traits<T>::VEC;
    const int64_t per_cell = pack_pieces(p.NPU, p.Dp, p.Hp, sizeof(T)), total = per_cell * p.n_cells;
    for (int64_t idx = block * NT + threadIdx.x; idx < total; idx += n_blocks * NT) {
        int cell = 0;
        uint32_t i = (uint32_t)idx;                          // (a cell has at most 2^31 pieces)
        if (p.n_cells > 1) { cell = (int)(idx / per_cell); i = (uint32_t)(idx - cell * per_cell); }
        const uint32_t row_slab = i >> 2;
        const int s = (int)(row_slab / (uint32_t)p.NPU), r = (int)(row_slab - (uint32_t)s * p.NPU), q = (int)(i & 3);
        const int tile = r / kGateTile, gate = (r % kGateTile) / kUnit, unit = tile * kUnit + r % kUnit;
        const int64_t src = (int64_t)cell * 4 * p.H + (int64_t)gate * p.H + unit;
        const int k = (s * 4 + q) * VEC, of = k < p.Dp ? p.D : p.H, at = k < p.Dp ? k : k - p.Dp;
        u32x4 v = {0u, 0u, 0u, 0u};
        if (unit < p.H && at < of) {
            const T *row = static_cast<const T *>(k < p.Dp ? p.W : p.U) + src * of + at;
            if (at + VEC <= of) {
                __builtin_memcpy(&v, row, 16);
            } else {
                T e[VEC];
#pragma unroll
                for (int j = 0; j < VEC; ++j) e[j] = at + j < of ? row[j] : T(0);
                __builtin_memcpy(&v, e, 16);
            }
        }
        *reinterpret_cast<u32x4 *>(static_cast<char *>(p.Bp) + (cell * per_cell + i) * 16) = v;
        if (k == 0 && r < p.NP) p.bp[(int64_t)cell * p.NP + r] = unit < p.H ? p.b[src] : 0.0f;
    }
}

template <typename T>
__global__ void __launch_bounds__(kThreads)
pack_weights_kernel(const PackArgs p) {
    pack_weights_body<T>(p, blockIdx.x, gridDim.x);
}

// ---- row records -------------------------------------------------------------------
// What the stack step and the cell update need to know about the node in row r of a
// level, in one 32-byte record: { node, arity, CSR start, - } { first four child ids (-1
// where there is none) }.  Written once per forward for all levels, so that the per-level
// kernels start from one load instead of the chain perm -> child_ptr -> child_idx.
//
// The rows of a level are independent, so their order inside the level is free.  The
// cell update walks the child lists of 32 rows in lock step and takes as many rounds as
// the longest of them; with rows in node-id order that is about twice the average need.
// The records are therefore ordered by falling arity inside windows of kRecWindow level
// positions (a counting sort in LDS; positions are already ordered by level, and the
// level is the major key so every row stays inside its level).  A window that spans 16 or
// more levels is left in position order: its levels are too small for the order to matter.
// The longer the runs of equal arity, the fewer passes of the cell update mix child lists of different length: a
// large forest takes windows of 16384 positions (blocks of 1024 threads, a launch of their own); measured on
// 2.36 M nodes, windows of 4096 -> 8192 -> 16384 rows take the internal levels from 5.26 to 5.17 to 5.10 ms (32768: 5.13).
// What bounds the step is what one compute unit can ask for: every record touches scattered lines, so the loads of a record
// are as few and as wide as they can be (child_ptr's two entries in one, the first four child ids in one: 2.36 M nodes
// 117 -> 86 us), and a forest whose large windows are fewer than 32 blocks leaves the chip idle and takes the small ones.  Schedule
// and forward with large / small windows, us: 296 k nodes H 512 bf16 1720 / 1696, H 256 1037 / 1001, four cells 1851 / 1792, N-ary
// 1506 / 1479; 432 k nodes H 300 fp32 6298 / 6269; 595 k H 512 2993 / 2997; 1.18 M 5561 / 5631; 2.36 M 10 651 / 10 767.
// The training forward's cell update writes the gates as well and loses more to lists of different length in one pass; it takes the large ones from
// half as many nodes on.  Training step, us, large / small: 286 k nodes of skewed arity H 512 bf16 5725 / 5780, 468 k 8800 / 8860, 338 k H 200 fp32
// 12 350 / 12 440, 468 k of even arity H 512 bf16 9100 / 9210, H 256 3640 / 3640, of skewed arity 3615 / 3595.
constexpr int kRecPerThread = 16;
constexpr int kRecWindow = kRecPerThread * kThreads;          // 4096
constexpr int kRecThreadsLarge = 1024;
constexpr int kRecWindowLarge = kRecPerThread * kRecThreadsLarge;   // 16384
constexpr int64_t kRecLargeMinNodes = 524288;      // forests of at least this many nodes take the large windows
constexpr int64_t kRecLargeMinNodesSave = 262144;  // ... in the training forward

// window `window` of the records (NT threads, kRecPerThread records each) of the positions below `end`, in a forest of n nodes
template <int NT>
__device__ __forceinline__ void row_record_body(const int32_t *__restrict__ perm, const int32_t *__restrict__ height,
                                                const int32_t *__restrict__ child_ptr,
                                                const int32_t *__restrict__ child_idx,
                                                int4 *__restrict__ row_rec, int n, int end, int window) {
    constexpr int kWin = kRecPerThread * NT;
    typedef u32x2 __attribute__((aligned(4))) u32x2a;
    typedef u32x4 __attribute__((aligned(4))) u32x4a;
    __shared__ int s_count[256];   // per key: count, then the next free slot
    __shared__ int s_scan[256];
    const int t = threadIdx.x;
    const int w0 = window * kWin;
    const int wn = (end - w0) < kWin ? (end - w0) : kWin;
    const int lvl0 = height[perm[w0]];
    const int lvl1 = height[perm[w0 + wn - 1]];
    const bool sorted = (lvl1 - lvl0) < 16;
    if (t < 256) s_count[t] = 0;
    __syncthreads();
    // A thread's sixteen records are fetched side by side, not one after the other: every load of a step is
    // unconditional (a position past the window reads the window's last one and is dropped afterwards), so the
    // chain perm -> child_ptr / height costs its two trips to memory once per thread, not once per record.
    int node[kRecPerThread], ar[kRecPerThread], cb[kRecPerThread], key[kRecPerThread];
    bool live[kRecPerThread];
#pragma unroll
    for (int i = 0; i < kRecPerThread; ++i) {
        const int p = w0 + i * NT + t;
        live[i] = p < w0 + wn;
        node[i] = perm[live[i] ? p : w0 + wn - 1];
    }
    int hgt[kRecPerThread];
#pragma unroll
    for (int i = 0; i < kRecPerThread; ++i) {
        const u32x2a q = *reinterpret_cast<const u32x2a *>(child_ptr + node[i]);
        cb[i] = (int)q[0];
        ar[i] = (int)(q[1] - q[0]);
        hgt[i] = sorted ? height[node[i]] : 0;
    }
#pragma unroll
    for (int i = 0; i < kRecPerThread; ++i) {
        key[i] = 0;
        if (!live[i]) {
            node[i] = -1; ar[i] = 0; cb[i] = 0;
        } else if (sorted) {
            key[i] = (hgt[i] - lvl0) * 16 + (15 - (ar[i] < 15 ? ar[i] : 15));
            atomicAdd(&s_count[key[i]], 1);
        }
    }
    __syncthreads();
    // exclusive scan of the 256 counts (by the first 256 threads; every thread meets the barriers)
    const int v = t < 256 ? s_count[t] : 0;
    if (t < 256) s_scan[t] = v;
    __syncthreads();
    for (int d = 1; d < 256; d <<= 1) {
        const int add = (t < 256 && t >= d) ? s_scan[t - d] : 0;
        __syncthreads();
        if (t < 256) s_scan[t] += add;
        __syncthreads();
    }
    if (t < 256) s_count[t] = s_scan[t] - v;
    __syncthreads();
    // The first four child ids of every record, again all loads of the thread side by side: sixteen bytes from its CSR start on,
    // from the array's last four entries where it starts behind those (child_ptr <= E < N, and the array has N entries).  Ids that
    // are not the node's are replaced by -1.
    // (in two halves: eight records' ids are in flight at a time, which keeps the large-window form in its registers)
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        constexpr int HB = kRecPerThread / 2;
        u32x4 kid[HB];
#pragma unroll
        for (int i = 0; i < HB; ++i) {
            const int c = cb[half * HB + i];
            if (n >= 4) {
                kid[i] = *reinterpret_cast<const u32x4a *>(child_idx + (c < n - 4 ? c : n - 4));
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) kid[i][j] = (uint32_t)child_idx[j < ar[half * HB + i] ? c + j : 0];
            }
        }
#pragma unroll
        for (int k = 0; k < HB; ++k) {
            const int i = half * HB + k;
            if (node[i] < 0) continue;
            const int64_t q = sorted ? (int64_t)w0 + atomicAdd(&s_count[key[i]], 1) : (int64_t)w0 + i * NT + t;
            u32x4 v = kid[k];
            for (int up = n >= 4 ? cb[i] - (n - 4) : 0; up > 0; --up) v = u32x4{v[1], v[2], v[3], 0u};
            row_rec[2 * q] = make_int4(node[i], ar[i], cb[i], 0);
            row_rec[2 * q + 1] = make_int4(0 < ar[i] ? (int)v[0] : -1, 1 < ar[i] ? (int)v[1] : -1,
                                           2 < ar[i] ? (int)v[2] : -1, 3 < ar[i] ? (int)v[3] : -1);
        }
    }
}

// Once per forward, in one launch: the row records of the level positions below `end` (blocks [0, n_windows)), the packed
// weights (the remaining blocks), and zeros in the n_clear words from `clear` on (all of them); none needs the others.
template <typename T>
__global__ void __launch_bounds__(kThreads)
prepare_kernel(const int32_t *__restrict__ perm, const int32_t *__restrict__ key,
               const int32_t *__restrict__ child_ptr, const int32_t *__restrict__ child_idx,
               int4 *__restrict__ row_rec, int n, int end, int n_windows, const PackArgs p, int *__restrict__ clear, int64_t n_clear) {
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n_clear; i += (int64_t)gridDim.x * kThreads) clear[i] = 0;
    if ((int)blockIdx.x < n_windows)
        row_record_body<kThreads>(perm, key, child_ptr, child_idx, row_rec, n, end, (int)blockIdx.x);
    else
        pack_weights_body<T>(p, (int64_t)blockIdx.x - n_windows, (int64_t)gridDim.x - n_windows);
}

// The same launch for large forests: row records in windows of kRecWindowLarge positions, blocks of 1024 threads.
template <typename T>
__global__ void __launch_bounds__(kRecThreadsLarge)
prepare_large_kernel(const int32_t *__restrict__ perm, const int32_t *__restrict__ key,
                     const int32_t *__restrict__ child_ptr, const int32_t *__restrict__ child_idx,
                     int4 *__restrict__ row_rec, int n, int end, int n_windows, const PackArgs p, int *__restrict__ clear, int64_t n_clear) {
    for (int64_t i = (int64_t)blockIdx.x * kRecThreadsLarge + threadIdx.x; i < n_clear; i += (int64_t)gridDim.x * kRecThreadsLarge) clear[i] = 0;
    if ((int)blockIdx.x < n_windows)
        row_record_body<kRecThreadsLarge>(perm, key, child_ptr, child_idx, row_rec, n, end, blockIdx.x);
    else
        pack_weights_body<T, kRecThreadsLarge>(p, (int64_t)blockIdx.x - n_windows, (int64_t)gridDim.x - n_windows);
}

// ---- stack -------------------------------------------------------------------------
// The paper's "stack" step (section 4.3): the samples of one slot are laid side by
// side on the batch axis.  Row r of the level's dense input matrix A is
//     [ x_j (D values, zero padded to Dp) | hsum_j = sum over children of h_k (Hp values) ]
// for the r-th node j of the level; leaves have the x part only.  Child rows come from hs (stride Hp, pad columns zero,
// rows by node id) in 16-byte pieces, up to four children of each of a thread's rows in flight.
template <typename T>
__device__ __forceinline__ void add_piece(float (&acc)[Traits<T>::VEC], const u32x4 &v) {
    if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] += __uint_as_float(v[j]);
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            acc[2 * j] += __uint_as_float(v[j] << 16);
            acc[2 * j + 1] += __uint_as_float(v[j] & 0xFFFF0000u);
        }
    }
}

struct StackArgs {
    const void *x; int D, Dp; const void *hs; int Hp;
    const int4 *row_rec; const int32_t *child_idx;
    void *A; int n_rows, n_rows_alloc;
};

// block `block` of the stack step (kThreads threads): the pair of slabs is x's or hs's, all of it
template <typename T>
__device__ __forceinline__ void stack_body(const T *__restrict__ x, int D, int Dp, const T *__restrict__ hs, int Hp,
                                           const int4 *__restrict__ row_rec, const int32_t *__restrict__ child_idx,
                                           T *__restrict__ A, int n_rows, int n_rows_alloc, unsigned block) {
    constexpr int VEC = Traits<T>::VEC;
    int64_t row;
    int pair;
    stack_place(block, (Dp + Hp) / (8 * VEC), n_rows, row, pair);
    if (row >= n_rows) return;
    const int k0 = (pair * 8 + (int)(threadIdx.x & 7)) * VEC;
    const int4 r0 = row_rec[2 * row];
    u32x4 o;
    if (k0 < Dp) {
        o = load_x_piece<T>(x + (int64_t)r0.x * D, k0, D);
    } else {
        const T *h = hs + (k0 - Dp);
        const int4 kids = row_rec[2 * row + 1];
        const int kid[4] = {kids.x, kids.y, kids.z, kids.w};
        u32x4 v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            v[j] = u32x4{0u, 0u, 0u, 0u};
            if (j < r0.y) v[j] = *reinterpret_cast<const u32x4 *>(h + (int64_t)kid[j] * Hp);
        }
        float acc[VEC];
#pragma unroll
        for (int j = 0; j < VEC; ++j) acc[j] = 0.0f;
#pragma unroll
        for (int j = 0; j < 4; ++j) add_piece<T>(acc, v[j]);   // ascending child id; zeros add nothing
        for (int c = 4; c < r0.y; ++c)
            add_piece<T>(acc, *reinterpret_cast<const u32x4 *>(h + (int64_t)child_idx[r0.z + c] * Hp));
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if constexpr (sizeof(T) == 4) o[j] = __float_as_uint(acc[j]);
            else o[j] = (uint32_t)f32_to_bf16(acc[2 * j]) | ((uint32_t)f32_to_bf16(acc[2 * j + 1]) << 16);
        }
    }
    *reinterpret_cast<u32x4 *>(reinterpret_cast<char *>(A) + operand_offset(row, (int64_t)k0 * sizeof(T), n_rows_alloc)) = o;
}

template <typename T>
__global__ void __launch_bounds__(kThreads)
stack_kernel(const StackArgs s) {
    stack_body<T>(static_cast<const T *>(s.x), s.D, s.Dp, static_cast<const T *>(s.hs), s.Hp, s.row_rec, s.child_idx,
                  static_cast<T *>(s.A), s.n_rows, s.n_rows_alloc, stack_block());
}

// Leaves: x alone.  One thread per 16 bytes in row order: a row's x is at most a few lines, and reading each of them once is worth more than
// the wider writes (1.33 M leaves, D 300, bf16 276 us against 293 as above; 162 k of four cells 35.5 against 38.9).
template <typename T>
__global__ void __launch_bounds__(kThreads)
stack_x_kernel(const StackArgs s) {
    constexpr int VEC = Traits<T>::VEC;
    const unsigned per_row = (unsigned)(s.Dp / VEC);
    const uint64_t first = (uint64_t)stack_block() * kThreads, row0 = first / per_row;      // of the block
    const unsigned at = (unsigned)(first - row0 * per_row) + threadIdx.x;
    const int64_t row = (int64_t)row0 + at / per_row;
    if (row >= s.n_rows) return;
    const int k0 = (int)(at % per_row) * VEC;
    const u32x4 o = load_x_piece<T>(static_cast<const T *>(s.x) + (int64_t)s.row_rec[2 * row].x * s.D, k0, s.D);
    *reinterpret_cast<u32x4 *>(static_cast<char *>(s.A) + operand_offset(row, (int64_t)k0 * sizeof(T), s.n_rows_alloc)) = o;
}

// The bf16 leaf level's blocks spend more time getting started and in the cell update than in their short K loop
// (K = D only): there a block keeps two stage buffers instead of three and three blocks share a CU instead of
// two (its three gate tiles leave the registers for that).  (fp32 leaves, whose K loop is bound by the fp32
// matrix rate, lose 3 % that way and keep three buffers.)
template <typename T, int MODE> constexpr bool kLeafDense = MODE == MODE_LEAF && sizeof(T) == 2;
template <typename T, int MODE> constexpr int kLevelBufs = kLeafDense<T, MODE> ? 2 : kDmaBufs;
template <typename T, int MODE> constexpr int kLevelBlocksPerCu = kLeafDense<T, MODE> ? 3 : 2;
template <int MODE> constexpr int kEpiArrays = MODE == MODE_LEAF ? 2 : 3;      // i u and o; with children also W_f x + b_f

template <typename T, int MODE, bool SAVE = false, bool GROUPED = false>
__global__ void __launch_bounds__(kDmaThreads, (kLevelBlocksPerCu<T, MODE>))
level_kernel(const LevelArgs a_in) {
    LevelArgs a = a_in;
    constexpr int NBUF = kLevelBufs<T, MODE>;
    __shared__ __attribute__((aligned(1024))) char lds[NBUF * kDmaBuf];
    static_assert(4 * kEpiArrays<MODE> * 32 * kEpiStride * 4 <= NBUF * kDmaBuf, "epilogue regions must fit the stage buffers");
    static_assert(MODE != MODE_PROJ || 4 * 32 * kDmaProjStride * 4 <= NBUF * kDmaBuf, "projection regions must fit the stage buffers");
    __shared__ int row_node[kDmaBM];
    __shared__ int row_ar[kDmaBM];
    __shared__ int row_cb[kDmaBM];
    __shared__ int4 row_kid[kDmaBM];
    __shared__ __attribute__((aligned(256))) char sink[4 * 256];   // where the L2 warm-up loads end up

    const int t = threadIdx.x;
    const int lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave >> 1, wn = wave & 1;

    int row_tile, col_tile;
    if (!block_to_tile(blockIdx.x, a.n_row_tiles, a.n_col_tiles, row_tile, col_tile)) return;
    int tile_row0 = row_tile * kDmaBM;
    if constexpr (GROUPED) {     // the tile's slot: where its rows start and end, whose weights apply
        if (!enter_range<kDmaBM>(a, row_tile, tile_row0)) return;
    }

    int node_reg = -1;
    int4 rec0 = make_int4(-1, 0, 0, 0), rec1 = make_int4(-1, -1, -1, -1);
    if (t < kDmaBM && tile_row0 + t < a.n_rows) {
        if constexpr (MODE == MODE_INTERNAL) {
            rec0 = a.row_rec[2 * (int64_t)(tile_row0 + t)];
            rec1 = a.row_rec[2 * (int64_t)(tile_row0 + t) + 1];
        } else {
            node_reg = (MODE == MODE_PROJ && !GROUPED && a.proj_nodes) ? a.proj_nodes[tile_row0 + t]
                                                                     : a.row_rec[2 * (int64_t)(tile_row0 + t)].x;
        }
    }
    auto publish_rows = [&]() __attribute__((always_inline)) {
        if (t < kDmaBM) {
            if constexpr (MODE == MODE_INTERNAL) {
                row_node[t] = rec0.x;
                row_ar[t] = rec0.y;
                row_cb[t] = rec0.z;
                row_kid[t] = rec1;
            } else {
                row_node[t] = node_reg;
            }
        }
    };

    floatx16 acc[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][g][v] = 0.0f;

    CellBias bias = {};
    if constexpr (MODE == MODE_PROJ) {
        publish_rows();
        __syncthreads();
        dma_gemm<T, MODE, NBUF>(a, lds, row_node, tile_row0, col_tile, acc, sink, []() {});
    } else {
        bias = load_cell_bias<MODE>(a, col_tile * 2 + wn, lane);     // on its way while the GEMM runs
        dma_gemm<T, MODE, NBUF>(a, lds, row_node, tile_row0, col_tile, acc, sink, publish_rows);
    }

    if constexpr (MODE == MODE_PROJ) {
        // Each wave turns its 64 rows x 128 units around in a private LDS region, 32 rows at
        // a time, so that 16 lanes store one row's 128 units in 8-unit pieces.
        float *region = reinterpret_cast<float *>(lds) + wave * (32 * kDmaProjStride);
#pragma unroll
        for (int p = 0; p < 2; ++p)
            proj_pass<T>(a, acc[p], region, row_node + wm * 64 + p * 32, col_tile * 256 + wn * 128, lane);
    } else {
        float *region = reinterpret_cast<float *>(lds) + wave * (kEpiArrays<MODE> * 32 * kEpiStride);
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int r0 = wm * 64 + p * 32;
            cell_pass<T, MODE, SAVE>(a, acc[p], region, row_node + r0, row_ar + r0, row_cb + r0, row_kid + r0,
                               col_tile * 2 + wn, lane, bias);
        }
    }
}

// ---- the same GEMM core as a plain C = A B^T ------------------------------------------
// For the further forget gates of N-ary cells (cells.hip): both operands K-blocked, all four column groups multiplied in
// every stage, no cell update; C in fp32, row-major.
struct KbEpiArgs { float *out; int ldc, M, N; };

template <typename T>
__global__ void __launch_bounds__(kDmaThreads, 2)
gemm_kb_kernel(const LevelArgs a, const KbEpiArgs e) {
    __shared__ __attribute__((aligned(1024))) char lds[kDmaBufs * kDmaBuf];
    __shared__ __attribute__((aligned(256))) char sink[4 * 256];
    const int t = threadIdx.x;
    const int lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int hf = lane >> 5, l32 = lane & 31;
    int row_tile, col_tile;
    if (!block_to_tile(blockIdx.x, a.n_row_tiles, a.n_col_tiles, row_tile, col_tile)) return;
    const int tile_row0 = row_tile * kDmaBM;

    floatx16 acc[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][g][v] = 0.0f;
    dma_gemm<T, MODE_GENERIC>(a, lds, nullptr, tile_row0, col_tile, acc, sink, []() {});
    __syncthreads();

    // A wave turns its 64 x 128 sub-tile, 32 rows at a time, through a region of the (now free) stage buffers, so
    // that a lane ends up with four consecutive columns of one row and the wave stores whole 512-byte row segments.
    constexpr int kStride = 128 + 4;
    static_assert(4 * 32 * kStride * 4 <= kDmaBufs * kDmaBuf, "epilogue regions must fit the stage buffers");
    float *region = reinterpret_cast<float *>(lds) + wave * (32 * kStride);
    const int c4 = (lane & 31) * 4;
    const int col = col_tile * kBN + wn * 128 + c4;
    const bool vec_ok = (e.ldc & 3) == 0;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                region[((v >> 2) * 8 + hf * 4 + (v & 3)) * kStride + g * 32 + l32] = acc[i][g][v];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll 4
        for (int sweep = 0; sweep < 16; ++sweep) {
            const int rl = (lane >> 5) + 2 * sweep;
            const int row = tile_row0 + wm * 64 + i * 32 + rl;
            if (row >= e.M || col >= e.N) continue;
            const float4 q = *reinterpret_cast<const float4 *>(region + rl * kStride + c4);
            const float f[4] = {q.x, q.y, q.z, q.w};
            float *dst = e.out + (int64_t)row * e.ldc + col;
            if (vec_ok && col + 4 <= e.N) {
                *reinterpret_cast<float4 *>(dst) = q;
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (col + j < e.N) dst[j] = f[j];
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

// ---- a slot of N-ary Tree-LSTM nodes: contraction and cell update in one kernel -----------
// The same GEMM core on the slot's stacked rows [x | h_1 | ... | h_N] and the cell's weights packed like
// the child-sum cell's (nary_pack in cells.hip): row = unit tile * 128 + slot * 32 + u with the slots
// i, o, u, f_1, so a block's 256 columns are two unit tiles and every wave holds the four gates of its
// 64 rows x 32 units in its own accumulators.  The forget gates of the further child positions,
// f_2 .. f_N, are a plain GEMM of their own that runs before this kernel (no padding to whole slots that
// way) and leaves its pre-activations in F; the cell update reads them from there.  A slot of leaves
// runs the same kernel over the x part of K (the first slabs of the same packed weights) and uses i, o, u.
// Rows, child ids and arities come with the row records; outputs go out by node id, 32 lanes on 32
// consecutive units of a row, the c values of eight rows' children requested together.
struct NaryEpi {
    const int4 *row_rec; const float *bias; const float *cs; const float *F;
    float *c_out; void *h_out; void *hs_out; float *cs_out;
    int M, H, Hp, Hq, N;
};

template <typename T, bool LEAF>
__global__ void __launch_bounds__(kDmaThreads, 2)
nary_level_kernel(LevelArgs a, const NaryEpi e) {
    __shared__ __attribute__((aligned(1024))) char lds[kDmaBufs * kDmaBuf];
    __shared__ __attribute__((aligned(256))) char sink[4 * 256];
    __shared__ int s_node[kDmaBM];
    __shared__ int s_ar[kDmaBM];
    __shared__ int4 s_kid[kDmaBM];
    const int t = threadIdx.x;
    const int lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int hf = lane >> 5, l32 = lane & 31;
    int row_tile, col_tile;
    if (!block_to_tile(blockIdx.x, a.n_row_tiles, a.n_col_tiles, row_tile, col_tile)) return;
    const int tile_row0 = row_tile * kDmaBM;

    floatx16 acc[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][g][v] = 0.0f;
    if (t < kDmaBM) {       // the tile's rows, fetched while the GEMM runs
        const int row = tile_row0 + t;
        const bool ok = row < e.M;
        const int4 r0 = e.row_rec[2 * (int64_t)(ok ? row : e.M - 1)];
        s_node[t] = ok ? r0.x : -1;
        if constexpr (!LEAF) {
            s_ar[t] = r0.y < e.N ? r0.y : e.N;
            s_kid[t] = e.row_rec[2 * (int64_t)(ok ? row : e.M - 1) + 1];
        }
    }
    dma_gemm<T, MODE_GENERIC>(a, lds, nullptr, tile_row0, col_tile, acc, sink, []() {});
    __syncthreads();

    const int unit = (col_tile * 2 + wn) * kUnit + l32;
    T *h_out = static_cast<T *>(e.h_out);
    T *hs_out = static_cast<T *>(e.hs_out);
    const bool separate_hs = hs_out != h_out;
    const bool separate_cs = e.cs_out != e.c_out;
    const int H = e.H;
    const bool live = unit < H;
    const int unit_ld = live ? unit : 0;
    const float bi = e.bias[unit_ld], bo = e.bias[H + unit_ld], bu = e.bias[2 * H + unit_ld];
    float bf[4] = {0.f, 0.f, 0.f, 0.f};
    if constexpr (!LEAF) {
#pragma unroll
        for (int l = 0; l < 4; ++l)
            if (l < e.N) bf[l] = e.bias[(3 + l) * H + unit_ld];
    }
    const int ldf = (e.N - 1) * H;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
        for (int vh = 0; vh < 2; ++vh) {
            int64_t node[8];
            float ck[8][4], fx[8][3];
            int m[8];
#pragma unroll
            for (int vv = 0; vv < 8; ++vv) {       // what eight rows need from memory first: loads in flight together
                const int v = vh * 8 + vv;
                const int lr = wm * 64 + i * 32 + (v >> 2) * 8 + hf * 4 + (v & 3);
                node[vv] = s_node[lr];
                m[vv] = 0;
#pragma unroll
                for (int l = 0; l < 4; ++l) ck[vv][l] = 0.0f;
#pragma unroll
                for (int l = 0; l < 3; ++l) fx[vv][l] = 0.0f;
                if constexpr (!LEAF) {
                    if (node[vv] >= 0) m[vv] = s_ar[lr];
                    const int4 k4 = s_kid[lr];
                    const int kid[4] = {k4.x, k4.y, k4.z, k4.w};
#pragma unroll
                    for (int l = 0; l < 4; ++l)
                        if (l < m[vv]) {
                            ck[vv][l] = e.cs[(int64_t)kid[l] * e.Hq + unit_ld];
                            if (l > 0) fx[vv][l - 1] = e.F[(int64_t)(tile_row0 + lr) * ldf + (l - 1) * H + unit_ld];
                        }
                }
            }
#pragma unroll
            for (int vv = 0; vv < 8; ++vv) {
                const int v = vh * 8 + vv;
                if (node[vv] < 0) continue;
                const int64_t nd = node[vv];
                if (!live) {                        // pad columns of the padded h copy
                    if (separate_hs && unit < e.Hp) hs_out[nd * e.Hp + unit] = T(0);
                    continue;
                }
                const float gi = sigmoid_t<T>(acc[i][0][v] + bi);
                const float go = sigmoid_t<T>(acc[i][1][v] + bo);
                const float gu = tanh_t<T>(acc[i][2][v] + bu);
                float c = gi * gu;
                if constexpr (!LEAF) {
#pragma unroll
                    for (int l = 0; l < 4; ++l)
                        if (l < m[vv]) c += sigmoid_t<T>((l == 0 ? acc[i][3][v] : fx[vv][l > 0 ? l - 1 : 0]) + bf[l]) * ck[vv][l];
                }
                const T hv = from_f32<T>(go * tanh_t<T>(c));
                e.c_out[nd * H + unit] = c;
                if (separate_cs) e.cs_out[nd * e.Hq + unit] = c;
                h_out[nd * H + unit] = hv;
                if (separate_hs) hs_out[nd * e.Hp + unit] = hv;
            }
        }
    }
}

// ---- thin levels ---------------------------------------------------------------------
// A level with a few thousand rows gives the 128 x 256 tiles too few blocks to fill 256
// CUs, and each block then runs a whole K loop back to back: the level costs that
// latency, not its work.  thin_kernel spreads such a level over many more waves.  A block
// of four waves owns one tile of 32 rows x 32 hidden units; wave g multiplies gate g (the
// projection: wave g one of four unit tiles of forget rows), taking its MFMA operands
// straight from global memory / L2 in fragment layout (16 bytes per lane, no LDS staging,
// kThinAhead K groups requested ahead), so the K loop of a tile is a quarter as long as
// with one wave per tile.  The gates meet in LDS and every wave finishes eight of the tile's
// rows (cell_rows).  One block barrier, none in the K loop.
constexpr int kThinWaves = 4;
constexpr int kThinMaxRows = 8192; // levels up to this many rows use the thin kernel
// ... in bf16 only where the 128 x 256 tiles are at most this many, one per compute unit: more of them hide behind each
// other what one costs, and a thin tile reads its weights from L2 for 32 rows.  (fp32's long K loops gain from the thin
// kernel's spread up to kThinMaxRows.)  Schedule + forward at 2048 / 4096 / 8192 rows, us: H 512 bf16, 256 tiles = 4096
// rows, 72 k nodes 710 / 698 / 725, four cells over 295 k nodes 1895 / 1894 / 1972; H 320 bf16, 286 k nodes 1270 / 1242 / 1234;
// H 512 fp32, 72 k nodes 2412 / 2346 / 2282.
constexpr int kThinMaxTiles = 256;
// ... and larger ones too, up to this size, if their nodes average kThinLongLists children or more: the thin
// kernel's cell update walks every row's own child list, the tiled kernel's makes 32 rows wait for the longest
constexpr int kThinMaxRowsLongLists = 16384;
constexpr int kThinLongLists = 5;
constexpr int kThinAhead = 8;      // K groups in flight per wave

template <typename T, int MODE, bool SAVE = false, bool GROUPED = false>
__device__ __forceinline__ void thin_body(const LevelArgs &a_in, int tile) {
    LevelArgs a = a_in;
    constexpr int ESZ = (int)sizeof(T);
    __shared__ __attribute__((aligned(16))) float smem[4 * 32 * kEpiStride];    // the four gates' pre-activations
    __shared__ int s_node[32];
    __shared__ int s_ar[32];
    __shared__ int s_cb[32];
    __shared__ int4 s_kid[32];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int hf = lane >> 5, l32 = lane & 31;
    int row0 = (tile / a.n_col_tiles) * 32;
    if constexpr (GROUPED) {
        if (!enter_range<32>(a, tile / a.n_col_tiles, row0)) return;      // (the same for all waves of the block)
    }
    const int col = tile % a.n_col_tiles;     // unit tile (gates) or group of four unit tiles (projection)
    // (leaves have no forget gate: its wave multiplies nothing, but takes its share of the cell update)
    if (MODE == MODE_PROJ && (col * 4 + wave) * kUnit >= a.Hu) return;            // past the last unit tile

    // ---- the tile's rows
    int my_row = row0 + l32;
    const bool row_ok = my_row < a.n_rows;
    if (!row_ok) my_row = a.n_rows - 1;       // computed twice, stored never
    int my_node;
    if constexpr (MODE == MODE_INTERNAL) {
        const int4 r0 = a.row_rec[2 * (int64_t)my_row];
        my_node = r0.x;
        if (wave == 0 && hf == 0) {
            const int4 r1 = a.row_rec[2 * (int64_t)my_row + 1];
            s_node[l32] = row_ok ? r0.x : -1;
            s_ar[l32] = row_ok ? r0.y : 0;
            s_cb[l32] = r0.z;
            s_kid[l32] = r1;
        }
    } else {
        my_node = a.row_rec[2 * (int64_t)my_row].x;
        if (wave == 0 && hf == 0) s_node[l32] = row_ok ? my_node : -1;
    }

    // ---- operand addresses: lane (l32, hf) supplies row l32, bytes [hf*16, +16) of each
    //      32-byte K group, for A and B alike.  K group g is bytes [32 g, 32 g + 32) of a
    //      row's K: half of slab g/2 in the K-blocked operands.
    const char *ap, *bp;
    int64_t a_pair, b_pair;                   // from K group g to g + 2
    int n_groups;                             // K groups this wave multiplies
    if constexpr (MODE == MODE_PROJ) {
        ap = static_cast<const char *>(a.hs) + (int64_t)my_node * a.Hp * ESZ + hf * 16;
        a_pair = 64;
        const int64_t row = (int64_t)(col * 4 + wave) * kGateTile + 3 * kUnit + l32;
        bp = static_cast<const char *>(a.Bp) + operand_offset(row, (int64_t)a.Dp * ESZ, a.NPU) + hf * 16;
        n_groups = a.Hp * ESZ / 32;
    } else {
        ap = static_cast<const char *>(a.stack) + operand_offset(my_row, 0, a.n_rows_alloc) + hf * 16;
        a_pair = (int64_t)a.n_rows_alloc * 64;
        const int64_t row = (int64_t)col * kGateTile + wave * kUnit + l32;
        bp = static_cast<const char *>(a.Bp) + operand_offset(row, 0, a.NPU) + hf * 16;
        // the forget rows take part in the x part only (U_f applies to each child's own h)
        n_groups = (a.Dp + (MODE == MODE_INTERNAL && wave != 3 ? a.Hp : 0)) * ESZ / 32;
        if (MODE == MODE_LEAF && wave == 3) n_groups = 0;
    }
    b_pair = (int64_t)a.NPU * 64;

    floatx16 acc[1];
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[0][v] = 0.0f;

    u32x4 fa[kThinAhead], fb[kThinAhead];
    auto request = [&](int g, int slot) __attribute__((always_inline)) {
        const int64_t ka = (int64_t)(g >> 1) * a_pair + (g & 1) * 32;
        const int64_t kb = (int64_t)(g >> 1) * b_pair + (g & 1) * 32;
        fa[slot] = *reinterpret_cast<const u32x4 *>(ap + ka);
        fb[slot] = *reinterpret_cast<const u32x4 *>(bp + kb);
    };
#pragma unroll
    for (int s = 0; s < kThinAhead; ++s)
        if (s < n_groups) request(s, s);
    for (int g0 = 0; g0 < n_groups; g0 += kThinAhead) {
#pragma unroll
        for (int s = 0; s < kThinAhead; ++s) {
            const int g = g0 + s;
            if (g < n_groups) {
                mfma_step<T>(fa[s], fb[s], acc[0]);
                if (g + kThinAhead < n_groups) request(g + kThinAhead, s);
            }
        }
    }

    if constexpr (MODE == MODE_PROJ) {
        T *P = static_cast<T *>(a.P);
        const int unit = (col * 4 + wave) * kUnit + l32;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int rl = (v >> 2) * 8 + hf * 4 + (v & 3);
            const int node = __shfl(my_node, rl, 64);      // lane rl holds the node of tile row rl (all lanes take part)
            if (unit < a.H && row0 + rl < a.n_rows) P[(int64_t)node * a.Hq + unit] = from_f32<T>(acc[0][v]);
        }
    } else {
        // the gates meet in LDS; every wave finishes eight of the tile's rows
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int rl = (v >> 2) * 8 + hf * 4 + (v & 3);
            smem[wave * (32 * kEpiStride) + rl * kEpiStride + l32] = acc[0][v];
        }
        __syncthreads();
        cell_rows<T, MODE, SAVE>(a, smem, s_node, s_ar, s_cb, s_kid, col, wave, lane);
    }
}

template <typename T, int MODE, bool SAVE = false, bool GROUPED = false>
__global__ void __launch_bounds__(kThinWaves * 64, 2)
thin_kernel(const LevelArgs a) {
    thin_body<T, MODE, SAVE, GROUPED>(a, blockIdx.x);
}

// The projection of a thin slot and the stack step of the slot after it in one launch: both
// only need what the level kernel before them wrote, and a thin level costs its chain of
// launches, not its work.  Blocks [0, a.n_blocks) are projection tiles, the rest stack blocks.
template <typename T, bool GROUPED = false>
__global__ void __launch_bounds__(kThinWaves * 64, 2)
thin_proj_stack_kernel(const LevelArgs a, const StackArgs s) {
    static_assert(kThinWaves * 64 == kThreads, "both bodies use the same block size");
    if ((int)blockIdx.x < a.n_blocks)
        thin_body<T, MODE_PROJ, false, GROUPED>(a, blockIdx.x);
    else
        stack_body<T>(static_cast<const T *>(s.x), s.D, s.Dp, static_cast<const T *>(s.hs), s.Hp, s.row_rec,
                            s.child_idx, static_cast<T *>(s.A), s.n_rows, s.n_rows_alloc,
                            blockIdx.x - (unsigned)a.n_blocks);
}

// ---- thin slots of N-ary nodes ----------------------------------------------------------
// A slot with few 128 x 256 tiles costs the tiled kernels' latency whatever it holds (16 us for the GEMM of f_2 .. f_N
// and 30 us for the level kernel behind it, D 300 H 256 N 2).  Here a block owns 32 rows x 32 units as in thin_kernel and
// has one wave per gate, 3 + N of them (leaves: i, o, u), on the same stacked rows and packed weights: all gates meet in
// LDS, so F is neither written nor read and the slot is one launch after its stack step.  The children's c are requested
// before the K loop.  Bound by one wave's chain of K groups.  Schedule + forward, before -> now: 571 nodes D 300 H 256 N 2
// bf16 438 -> 214 us, 4.5 k nodes fp32 2949 -> 573, 270 k nodes bf16 1732 -> 1551.
constexpr int kNaryThinWaves = 7;      // 3 + N, N <= 4
template <typename T, bool LEAF>
__global__ void __launch_bounds__(kNaryThinWaves * 64, 4)
nary_thin_kernel(const LevelArgs a, const NaryEpi e, const void *__restrict__ Bx, int rows_x) {
    constexpr int ESZ = (int)sizeof(T);
    __shared__ __attribute__((aligned(16))) float smem[(LEAF ? 3 : kNaryThinWaves) * 32 * kEpiStride];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);      // the gate: i, o, u, f_1 .. f_N
    const int hf = lane >> 5, l32 = lane & 31;
    const int row0 = ((int)blockIdx.x / a.n_col_tiles) * 32;
    const int col = (int)blockIdx.x % a.n_col_tiles;

    // ---- the weights' and the rows' K groups (thin_body)
    const int my_row = min(row0 + l32, e.M - 1);           // past the end: computed twice, stored never
    const char *ap = static_cast<const char *>(a.stack) + operand_offset(my_row, 0, a.n_rows_alloc) + hf * 16;
    const int64_t a_pair = (int64_t)a.n_rows_alloc * 64;
    const char *bp;
    int64_t b_pair;
    if (wave < 4) {
        bp = static_cast<const char *>(a.Bp) + operand_offset((int64_t)col * kGateTile + wave * kUnit + l32, 0, a.NPU) + hf * 16;
        b_pair = (int64_t)a.NPU * 64;
    } else {                                               // row of f_2 .. f_N; a unit past H reads the gate's first row
        const int unit = col * kUnit + l32;
        bp = static_cast<const char *>(Bx) + operand_offset((int64_t)(wave - 4) * e.H + (unit < e.H ? unit : 0), 0, rows_x) + hf * 16;
        b_pair = (int64_t)rows_x * 64;
    }
    const int n_groups = a.Dp * ESZ / 32;
    floatx16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
    u32x4 fa[kThinAhead], fb[kThinAhead];
    auto request = [&](int g, int slot) __attribute__((always_inline)) {
        fa[slot] = *reinterpret_cast<const u32x4 *>(ap + (int64_t)(g >> 1) * a_pair + (g & 1) * 32);
        fb[slot] = *reinterpret_cast<const u32x4 *>(bp + (int64_t)(g >> 1) * b_pair + (g & 1) * 32);
    };
#pragma unroll
    for (int s = 0; s < kThinAhead; ++s)
        if (s < n_groups) request(s, s);

    // ---- eight lanes per row, four units each, by the first four waves (leaves have three: they go round again)
    const int u4 = (lane & 7) * 4, unit0 = col * kUnit + u4;
    int node = -1, m = 0;
    float4 ck[4];
    if constexpr (!LEAF) {
        if (wave < 4) {
            const int row = row0 + (int)(threadIdx.x >> 3);
            const int4 r0 = e.row_rec[2 * (int64_t)min(row, e.M - 1)];
            const int4 kids = e.row_rec[2 * (int64_t)min(row, e.M - 1) + 1];
            if (row < e.M) { node = r0.x; m = r0.y < e.N ? r0.y : e.N; }
            const int kid[4] = {kids.x, kids.y, kids.z, kids.w};
            const int unit_ld = unit0 < e.Hq ? unit0 : 0;
#pragma unroll
            for (int l = 0; l < 4; ++l) {
                ck[l] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (l < m) ck[l] = *reinterpret_cast<const float4 *>(e.cs + (int64_t)kid[l] * e.Hq + unit_ld);
            }
        }
    }
    for (int g0 = 0; g0 < n_groups; g0 += kThinAhead) {
#pragma unroll
        for (int s = 0; s < kThinAhead; ++s) {
            const int g = g0 + s;
            if (g < n_groups) {
                mfma_step<T>(fa[s], fb[s], acc);
                if (g + kThinAhead < n_groups) request(g + kThinAhead, s);
            }
        }
    }
#pragma unroll
    for (int v = 0; v < 16; ++v)
        smem[wave * (32 * kEpiStride) + ((v >> 2) * 8 + hf * 4 + (v & 3)) * kEpiStride + l32] = acc[v];
    __syncthreads();

    auto finish = [&](int tr) __attribute__((always_inline)) {
        auto gate = [&](int g) __attribute__((always_inline)) {
            float4 q = *reinterpret_cast<const float4 *>(smem + g * (32 * kEpiStride) + tr * kEpiStride + u4);
            const float *b = e.bias + (int64_t)g * e.H + unit0;      // (the caller's array: any alignment)
            if (unit0 < e.H) q.x += b[0];
            if (unit0 + 1 < e.H) q.y += b[1];
            if (unit0 + 2 < e.H) q.z += b[2];
            if (unit0 + 3 < e.H) q.w += b[3];
            return q;
        };
        const float4 zi = gate(0), zo = gate(1), zu = gate(2);
        float4 cc = make_float4(sigmoid_t<T>(zi.x) * tanh_t<T>(zu.x), sigmoid_t<T>(zi.y) * tanh_t<T>(zu.y),
                                sigmoid_t<T>(zi.z) * tanh_t<T>(zu.z), sigmoid_t<T>(zi.w) * tanh_t<T>(zu.w));
        if constexpr (!LEAF) {
#pragma unroll
            for (int l = 0; l < 4; ++l)
                if (l < m) {
                    const float4 f = gate(3 + l);
                    cc.x += sigmoid_t<T>(f.x) * ck[l].x;
                    cc.y += sigmoid_t<T>(f.y) * ck[l].y;
                    cc.z += sigmoid_t<T>(f.z) * ck[l].z;
                    cc.w += sigmoid_t<T>(f.w) * ck[l].w;
                }
        }
        store_state<T>(a, node, unit0, cc, make_float4(sigmoid_t<T>(zo.x), sigmoid_t<T>(zo.y), sigmoid_t<T>(zo.z), sigmoid_t<T>(zo.w)));
    };
    if constexpr (LEAF) {
        for (int tr = (int)(threadIdx.x >> 3); tr < 32 && row0 + tr < e.M; tr += 24) {
            node = e.row_rec[2 * (int64_t)(row0 + tr)].x;
            finish(tr);
        }
    } else if (wave < 4 && node >= 0) {
        finish((int)(threadIdx.x >> 3));
    }
}

// ---- chain levels ---------------------------------------------------------------------
// A level in which every node has exactly one child (sequences filed as chains, the long thin tail of a forest) needs
// neither the stack step nor the projection: the child sum is the child's h, read in place, and U_f h_k belongs to the
// same row, so the forget gate is a fourth full-K product like i, o and u.  What such levels cost is not their work but
// the string of dependent trips to memory inside each of them and the gap between launches, so up to kChainLevels of them run in
// one launch that follows each row through the levels (one that fills the chip goes alone, kChainAloneTiles):
//
//   * a tile is 16 RT rows x 32 units, wave w multiplies gate w % 4; a block takes ONE tile and is done;
//   * blocks draw their tiles from a counter, in the order of the levels, and a tile waits for the row tiles of
//     the level below that hold its rows' children: each has a word that counts its finished unit tiles.  Whatever a block
//     waits for was drawn before, by a block that runs already, so every wait ends, whichever blocks share the chip.  (Should something
//     else write into the workspace meanwhile, it ends too: after kChainLooks looks the block marks the counter, no block waits any
//     more, and c and h of the tiles that did not see their children are NaN);
//   * everything that does not depend on the child is there before the wait: the wave's weights (the first kChainAhead K
//     groups), the row's ids, x rows in LDS or Z.  Two or more blocks of later levels sit beside the one that multiplies;
//   * behind the wait the block fetches the children's h once, all loads in flight together, into LDS; the K loop has no
//     barrier (A fragments from LDS, weights kChainAhead groups ahead); the gates meet in LDS and each of
//     the first 2 RT waves finishes eight of the tile's rows;
//   * h and c of a child may come from another XCD's block, whose L2 is not this one's.  They, the words and the counter are only
//     touched by atomic accesses of agent scope, which are carried out where all XCDs see them (loads and stores go past the L2s, sc1):
//     one that vmcnt counts as done has been done for every block.  So no cache need be written back or dropped; what is left is
//     order, and each half of it is made by hand: a block's waves wait for vmcnt 0 and meet at the barrier before the word is raised,
//     and no wave asks for h or c before wave 0 has seen the words and met it at the barrier (a load is not started before the branch
//     that it stands behind is decided);
//   * US = 2 (fp32, whose MFMAs are a long chain for one wave): eight waves, wave w has units 16 (w / 4) .. of its gate;
//   * RT = 1 spreads a level over more blocks and shortens each one's part of the chain; where bf16 levels have
//     kChainWideTiles such tiles on average the chip is full and RT = 2 asks half as much of the weights and the words.  A launch that
//     holds one level has no counter, no words and no wait.
//
// Schedule + forward, chains / stars / trees in turn, us, one launch a level (13 - 20 us each) -> RT = 2 -> RT = 1:
// 4096 trees of up to 128 nodes, D 300, H 256 fp32 3567 -> 3231 -> 3033, bf16 2052 -> 1644 -> 1691; 500 trees H 150 fp32
// 1443 -> 1090 -> 891, bf16 981 -> 608 -> 539; 12 k trees, D 128, H 128, bf16 1978 -> 1612 -> 1786; x part not in Z: 2 k trees of
// up to 64, H 400 fp32 2643 -> 2478 -> 2301, H 512 bf16 1506 -> 1437 -> 1484.  What is left of a level (about 5 us where it is
// small) is the way of h from one block to the next: stores, word, look, loads.  (Words side by side in one line, all blocks
// looking at it: 4084 instead of 3255 in the first case.)
//
// Needs D % 4 == 0 (an 8- / 16-byte piece of an x row is inside D or outside) and rows of A that leave room for two blocks on a CU.
constexpr int kChainAhead = 16;                         // weight loads in flight per wave
constexpr int kChainLevels = 256;                       // levels one launch may hold (its table travels with the arguments)
constexpr int kChainLooks = 1 << 21;                    // a microsecond or more each; the longest launches take some ten thousand
constexpr int kChainGaveUp = 1 << 30;                   // in the counter: a block has given up waiting
constexpr int kChainLost = -2;                          // a child that was not seen
constexpr int kChainMaxKBytes = 4304;                   // of a row, RT = 1: two blocks share a CU's LDS
constexpr int kChainMaxKBytes2 = 1840;                  // ... RT = 2
// A level of many tiles goes alone, its tiles by block index: thousands of draws from one counter take longer than a launch (8000
// chains of 4 - 5 nodes, bf16, all levels in one launch / each alone: H 256 192 / 172 us, H 512 453 / 436).  Such a level fills the
// chip, and what counts is no longer one block's chain but how often the weights are read and how soon a block is at work: tiles of
// 32 rows (fp32: up to kChainAloneMaxKBytes2 of a row; above that the second block on a CU, which 32 rows leave no room for, is worth
// more), and in fp32 half as many loads ahead.  The same forests, us, (a) a launch a level of 32-row tiles whose waves had a part of K
// each, (b) 16-row tiles, 16 loads ahead, (c) 32 rows, 16, (d) 32 rows, 8, (e) 16 rows, 8:
//                          bytes     a      b      c      d      e
//   fp32  D  64  H  384     1792    653    658    553    535    556
//         D 300  H  256     2304    482    541    481    468    527
//         D 300  H  320     2560    737    752    782    755    645
//         D 512  H  128     2560    355    366    366    356    332
//         D 512  H  256     3072    714    704    728    710    683
//         D 300  H  512     3328   1325   1322   1380   1330   1240
//   bf16  D 300  H  256     1152    185           171
//         D 512  H  512     2048    662    609    595
//         D 1024 H  512     3072    858    936    768
//         D 512  H 1024     3072   1595   1725   1435
constexpr int kChainAloneTiles = 1536;
constexpr int kChainAloneMaxKBytes2 = 2304;
constexpr int kChainAloneAhead = 8;
constexpr int kChainWideTiles = 192;                    // (330 tiles a level: 3 % for RT = 2, 500: 10 %, 31: 13 % for RT = 1)
// LDS pitch of an A row: K bytes + 16, so that 16 lanes' 16-byte reads of one K group fall in 64 different banks
__host__ __device__ inline constexpr int chain_row_pitch(int k_bytes) { return k_bytes + 16; }
inline constexpr int chain_lds_bytes(int k_bytes, int rt) { return 16 * rt * chain_row_pitch(k_bytes); }
constexpr int kChainLdsMax = chain_lds_bytes(kChainMaxKBytes, 2);
static_assert(kChainLdsMax + 4 * 32 * kEpiStride * 4 + 1024 <= 160 * 1024, "a level alone: 32 rows of any width");
static_assert(2 * (chain_lds_bytes(kChainMaxKBytes, 1) + 4 * 16 * kEpiStride * 4 + 1024) <= 160 * 1024, "two blocks share a CU");
static_assert(2 * (chain_lds_bytes(kChainMaxKBytes2, 2) + 4 * 32 * kEpiStride * 4 + 1024) <= 160 * 1024, "two blocks share a CU");

struct ChainArgs {
    const int32_t *perm, *inv_perm, *child_ptr, *child_idx;     // inv_perm is not read, and may be nullptr, where n_levels is 1
    int *ticket;                         // tiles drawn so far
    int *done;                           // per row tile of the launch, `stride` words apart: unit tiles finished
    int stride;
    int n_levels;
    int tiles[kChainLevels + 1];         // row tiles before the launch's level
    int pos[kChainLevels + 1];           // positions of the launch's levels
};

__device__ __forceinline__ void store_shared(void *p, const u32x2 &v) {
    __hip_atomic_store(static_cast<uint64_t *>(p), __builtin_bit_cast(uint64_t, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u32x2 load_shared(const void *p) {
    return __builtin_bit_cast(u32x2, __hip_atomic_load(static_cast<const uint64_t *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// store_state for rows that a later tile of the same launch reads: the copies it reads (hs_out and cs) leave past the L2.
template <typename T>
__device__ __forceinline__ void store_state_shared(const LevelArgs &a, int64_t nd, int unit0, const float4 &cc, const float4 &go) {
    const float c4[4] = {cc.x, cc.y, cc.z, cc.w};
    const float o4[4] = {go.x, go.y, go.z, go.w};
    T hv[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) hv[j] = unit0 + j < a.H ? from_f32<T>(o4[j] * tanh_t<T>(c4[j])) : T(0);
    if (unit0 < a.Hp) {                  // (H != Hp: pad columns of the padded copy are zeroed)
        T *dst = static_cast<T *>(a.hs_out) + nd * a.Hp + unit0;
        if constexpr (sizeof(T) == 4) {
            store_shared(dst, u32x2{__float_as_uint(hv[0]), __float_as_uint(hv[1])});
            store_shared(dst + 2, u32x2{__float_as_uint(hv[2]), __float_as_uint(hv[3])});
        } else {
            store_shared(dst, u32x2{(uint32_t)hv[0] | ((uint32_t)hv[1] << 16), (uint32_t)hv[2] | ((uint32_t)hv[3] << 16)});
        }
    }
    if (unit0 < a.Hq) {
        float *dst = a.cs + nd * a.Hq + unit0;
        store_shared(dst, u32x2{__float_as_uint(c4[0]), __float_as_uint(c4[1])});
        store_shared(dst + 2, u32x2{__float_as_uint(c4[2]), __float_as_uint(c4[3])});
    }
    if (a.hs_out != a.h_out) {
        T *dst = static_cast<T *>(a.h_out) + nd * a.H + unit0;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (unit0 + j < a.H) dst[j] = hv[j];
    }
    if (a.cs != a.c_out) {
        float *dst = a.c_out + nd * a.H + unit0;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (unit0 + j < a.H) dst[j] = c4[j];
    }
}

//
// HAS_Z: the x part of the pre-activations (and the bias) is in Z already (tree_x_kernel has been over all nodes): A is the
// child's h alone and K is H.
template <typename T, int US, int RT, bool HAS_Z, int AHEAD = kChainAhead>
__global__ void __launch_bounds__(kThinWaves * 64 * US, 4)
chain_kernel(const LevelArgs a, const ChainArgs lv) {
    constexpr int ESZ = (int)sizeof(T);
    constexpr int ROWS = 16 * RT;
    constexpr int NB = 2 / US;                                            // tiles of 16 units per wave
    constexpr int RING = AHEAD / NB;                                      // slabs of weights in flight
    extern __shared__ __attribute__((aligned(16))) char a_lds[];          // [16 RT][chain_row_pitch]
    __shared__ __attribute__((aligned(16))) float zt[4][ROWS * kEpiStride];   // pre-activations, [gate][row][unit]
    __shared__ int s_node[ROWS];
    __shared__ int s_kid[ROWS];
    __shared__ int s_tile, s_level;
    __shared__ __attribute__((aligned(16))) float s_bias[HAS_Z ? 4 : kGateTile];
    static_assert(kChainLevels <= kThinWaves * 64, "a thread per level");

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int gate = wave & 3, half = wave >> 2;
    const int q4 = lane >> 4, l16 = lane & 15;
    if (tid == 0) s_tile = lv.n_levels == 1 ? (int)blockIdx.x : __hip_atomic_fetch_add(lv.ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int t_lo = lv.tiles[tid < lv.n_levels ? tid : lv.n_levels], t_hi = lv.tiles[tid < lv.n_levels ? tid + 1 : lv.n_levels];
    __syncthreads();
    const int drawn = __builtin_amdgcn_readfirstlane(s_tile), place = drawn & (kChainGaveUp - 1);
    const int tile = place < a.n_blocks ? place : a.n_blocks - 1;     // (always below: the grid has as many blocks as there are tiles)
    const int row_tile = tile / a.n_col_tiles;
    const int col = tile - row_tile * a.n_col_tiles;             // unit tile
    if (t_lo <= row_tile && row_tile < t_hi) s_level = tid;

    // ---- weights: lane (l16, q4) supplies row l16 of a tile of the wave's gate, bytes [q4*16, +16) of each slab (64 bytes of K).
    //      Every load of the ring is unconditional (a slab past the end is clamped to the last one, whose data is
    //      then not used): the number of loads between a request and its use is the same on every path, so the waits
    //      the compiler places are counted, not "all".
    const int x_bytes = HAS_Z ? 0 : a.Dp * ESZ;          // K bytes of the x part
    const int h_bytes = a.Hp * ESZ;
    const int k_bytes = x_bytes + h_bytes;
    const int pitch = chain_row_pitch(k_bytes);
    const int n_slabs = k_bytes / 64;
    const int64_t brow = (int64_t)col * kGateTile + gate * kUnit + half * 16 + l16;
    const char *bp = static_cast<const char *>(a.Bp) + operand_offset(brow, HAS_Z ? (int64_t)a.Dp * ESZ : 0, a.NPU) + q4 * 16;
    const int64_t b_slab = (int64_t)a.NPU * 64;
    u32x4 fb[RING][NB];
    auto request = [&](int s, int slot) __attribute__((always_inline)) {
        const char *p = bp + (int64_t)(s < n_slabs ? s : n_slabs - 1) * b_slab;
#pragma unroll
        for (int q = 0; q < NB; ++q) fb[slot][q] = *reinterpret_cast<const u32x4 *>(p + q * 16 * 64);
    };
#pragma unroll
    for (int s = 0; s < RING; ++s) request(s, s);
    __syncthreads();

    // ---- the rows: node, child, and, in wave 0, the row tiles below that hold the children
    const int l = __builtin_amdgcn_readfirstlane(s_level);
    const int rt_level = row_tile - lv.tiles[l];                 // row tile within the level
    const int row0 = lv.pos[l] + rt_level * ROWS;
    const int n_rows = lv.pos[l + 1] - row0 < ROWS ? lv.pos[l + 1] - row0 : ROWS;
    int wait_lo = 0, wait_hi = -1;                               // row tiles of the launch
    int astray = 0;                                              // not 0: the row's child is not where inv_perm says
    if (wave == 0) {
        const int mine = lane & (ROWS - 1), r = mine < n_rows ? mine : n_rows - 1;   // past the end: computed twice, stored never
        const int node = lv.perm[row0 + r];
        typedef u32x2 __attribute__((aligned(4))) u32x2a;
        const u32x2a cp = *reinterpret_cast<const u32x2a *>(lv.child_ptr + node);
        const int kid = (int)cp[1] > (int)cp[0] ? lv.child_idx[(int)cp[0]] : -1;   // (always one, in a level this kernel is launched for)
        if (lane < ROWS) {
            s_node[mine] = mine < n_rows ? node : -1;
            s_kid[mine] = kid;
        }
        if (l > 0) {
            // (a position outside the level below, or another node's, is dealt with at the first look)
            int q = lv.inv_perm[kid < 0 ? 0 : kid];
            q = q < lv.pos[l - 1] ? lv.pos[l - 1] : q < lv.pos[l] ? q : lv.pos[l] - 1;
            astray = lv.perm[q] - kid;
            int lo = lv.tiles[l - 1] + (q - lv.pos[l - 1]) / ROWS, hi = lo;
#pragma unroll
            for (int d = 1; d < ROWS; d <<= 1) {
                const int lo2 = __shfl_xor(lo, d, 64), hi2 = __shfl_xor(hi, d, 64);
                lo = lo2 < lo ? lo2 : lo;
                hi = hi2 > hi ? hi2 : hi;
            }
            wait_lo = __builtin_amdgcn_readfirstlane(lo);
            wait_hi = __builtin_amdgcn_readfirstlane(hi);
        }
    }
    __syncthreads();

    // ---- what does not depend on the child.  A: thread t moves pieces (t & 31) + 32 i of rows (t >> 5) + RPP j
    constexpr int RPP = 8 * US;           // rows per pass of the block's threads
    constexpr int NJ = ROWS / RPP;
    constexpr int kUpdateWaves = ROWS / 8;
    const int tr = (wave & (kUpdateWaves - 1)) * 8 + (lane >> 3);   // the cell update's row and units
    const int u4 = (lane & 7) * 4;
    const int unit0 = col * kUnit + u4;
    const int node = s_node[tr];
    float4 bq[4];
    if constexpr (HAS_Z) {
        if (wave < kUpdateWaves) {      // Z with the bias in it (unit groups past its width read the first)
            const float *z = a.Z + (int64_t)(node < 0 ? 0 : node) * 4 * a.Hz + (unit0 < a.Hz ? unit0 : 0);
#pragma unroll
            for (int g = 0; g < 4; ++g) bq[g] = *reinterpret_cast<const float4 *>(z + g * a.Hz);
        }
    } else {
        if (tid < kGateTile) s_bias[tid] = a.bp[col * kGateTile + tid];
        const int n_rounds = (x_bytes / 16 + 31) / 32;
        const char *src[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int nd = s_node[(tid >> 5) + RPP * j];
            src[j] = static_cast<const char *>(a.x) + (int64_t)(nd < 0 ? 0 : nd) * a.D * ESZ;
        }
#pragma unroll 2
        for (int i = 0; i < n_rounds; ++i) {
            const int kb = ((tid & 31) + 32 * i) * 16;
            if (kb >= x_bytes) break;
            // a piece past D comes from the start of the row (always valid: D >= 4) and is replaced by zero
            const bool ok0 = kb / ESZ < a.D, ok1 = ESZ == 4 ? ok0 : kb / ESZ + 4 < a.D;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                u32x4 v;
                if constexpr (ESZ == 4) {
                    v = *reinterpret_cast<const u32x4 *>(ok0 ? src[j] + kb : src[j]);
                } else {
                    const u32x2 q0 = *reinterpret_cast<const u32x2 *>(ok0 ? src[j] + kb : src[j]);
                    const u32x2 q1 = *reinterpret_cast<const u32x2 *>(ok1 ? src[j] + kb + 8 : src[j]);
                    v[0] = q0[0]; v[1] = q0[1]; v[2] = q1[0]; v[3] = q1[1];
                }
                v[0] = ok0 ? v[0] : 0u; v[1] = ok0 ? v[1] : 0u; v[2] = ok1 ? v[2] : 0u; v[3] = ok1 ? v[3] : 0u;
                *reinterpret_cast<u32x4 *>(a_lds + ((tid >> 5) + RPP * j) * pitch + kb) = v;
            }
        }
    }

    // ---- wait for the children (wave 0; the others stand at the barrier)
    if (wait_lo <= wait_hi) {
        auto look = [&](int w, int least) {
            const int *word = lv.done + (int64_t)(w + lane <= wait_hi ? w + lane : wait_hi) * lv.stride;
            return (bool)__all(__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= least);
        };
        // A position that is not the child's, or not in the level below (a schedule made by hand), says nothing: the tile then
        // waits for every tile of the launch's levels below.  Whether there is one is known with the first look; what stands behind the
        // later ones is on the way of h from one block to the next.
        int w = wait_lo;
        const bool first = look(w, a.n_col_tiles) && w + 64 > wait_hi, stray = __any(astray != 0);
        if (!first || stray) {
            if (stray) {
                w = 0;
                wait_hi = lv.tiles[l] - 1;
            }
            int looks = drawn == place ? kChainLooks : 0;
            bool there;
            do {
                there = wait_bounded(a.n_col_tiles, looks, [&](int least) { return look(w, least); }, [] { __builtin_amdgcn_s_sleep(1); });
                w += 64;
            } while (w <= wait_hi);
            if (!there) {
                if (lane < ROWS) s_kid[lane] = kChainLost;
                if (lane == 0) __hip_atomic_fetch_or(lv.ticket, kChainGaveUp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
    asm volatile("" ::: "memory");
    __syncthreads();

    // ---- the children's h into LDS, c into registers
    float4 ck = make_float4(0.f, 0.f, 0.f, 0.f);
    {
        const int n_rounds = (h_bytes / 16 + 31) / 32;
        const char *src[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int kid = s_kid[(tid >> 5) + RPP * j];
            src[j] = static_cast<const char *>(a.hs) + (int64_t)(kid < 0 ? 0 : kid) * h_bytes;
        }
        constexpr int NR = 2 * US / RT;          // rounds whose loads are in flight together
        for (int i = 0; i < n_rounds; i += NR) {
            u32x2 v[NR][NJ][2];
#pragma unroll
            for (int q = 0; q < NR; ++q) {
                int kb = ((tid & 31) + 32 * (i + q)) * 16;
                kb = kb < h_bytes ? kb : 0;
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    v[q][j][0] = load_shared(src[j] + kb);
                    v[q][j][1] = load_shared(src[j] + kb + 8);
                }
            }
            if (i == 0 && wave < kUpdateWaves) {            // unit groups past the padded width read the first group (and store nothing)
                const int kid = s_kid[tr];
                const float *c = a.cs + (int64_t)(kid < 0 ? 0 : kid) * a.Hq + (unit0 < a.Hq ? unit0 : 0);
                const u32x2 c0 = load_shared(c), c1 = load_shared(c + 2);
                if (kid >= 0) ck = make_float4(__uint_as_float(c0[0]), __uint_as_float(c0[1]), __uint_as_float(c1[0]), __uint_as_float(c1[1]));
            }
#pragma unroll
            for (int q = 0; q < NR; ++q) {
                const int kb = ((tid & 31) + 32 * (i + q)) * 16;
                if (kb < h_bytes) {
#pragma unroll
                    for (int j = 0; j < NJ; ++j)
                        *reinterpret_cast<u32x4 *>(a_lds + ((tid >> 5) + RPP * j) * pitch + x_bytes + kb) =
                            u32x4{v[q][j][0][0], v[q][j][0][1], v[q][j][1][0], v[q][j][1][1]};
                }
            }
        }
#pragma unroll 1
        for (int j = 0; j < NJ; ++j) {
            const int kid = s_kid[(tid >> 5) + RPP * j];
            const uint32_t fill = kid == kChainLost ? 0xFFFFFFFFu : 0u;           // NaN; or no child after all: zeros
            if (kid < 0)
                for (int kb = (tid & 31) * 16; kb < h_bytes; kb += 512)
                    *reinterpret_cast<u32x4 *>(a_lds + ((tid >> 5) + RPP * j) * pitch + x_bytes + kb) = u32x4{fill, fill, fill, fill};
        }
    }
    floatx4 acc[RT][NB];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int q = 0; q < NB; ++q) acc[i][q] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    __syncthreads();

    // ---- K loop: whole turns of the ring, then the last one, which requests nothing any more
    const char *abuf = a_lds + l16 * pitch + q4 * 16;    // this lane's A fragment, slab 0
    const int n_full = (n_slabs - 1) / RING;
    u32x4 fa[RT];
    auto step = [&](int s, int next) __attribute__((always_inline)) {      // the next A fragment leaves LDS while this one is multiplied
        u32x4 fa_next[RT];
#pragma unroll
        for (int i = 0; i < RT; ++i) fa_next[i] = *reinterpret_cast<const u32x4 *>(abuf + i * 16 * pitch + next * 64);
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int q = 0; q < NB; ++q) mfma16<T>(fa[i], fb[s][q], acc[i][q]);
#pragma unroll
        for (int i = 0; i < RT; ++i) fa[i] = fa_next[i];
    };
#pragma unroll
    for (int i = 0; i < RT; ++i) fa[i] = *reinterpret_cast<const u32x4 *>(abuf + i * 16 * pitch);
    for (int c = 0; c < n_full; ++c) {
#pragma unroll
        for (int s = 0; s < RING; ++s) {            // (behind these turns at least one slab is left)
            step(s, c * RING + s + 1);
            request(c * RING + s + RING, s);
            __builtin_amdgcn_sched_barrier(0);      // the ring is refilled slot by slot, not in a burst at the end
        }
    }
#pragma unroll
    for (int s = 0; s < RING; ++s)
        if (n_full * RING + s < n_slabs) step(s, n_full * RING + s + 1 < n_slabs ? n_full * RING + s + 1 : n_slabs - 1);

    // ---- the gates meet in LDS; the first waves finish eight rows each: eight lanes per row, four units per lane
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int q = 0; q < NB; ++q)
#pragma unroll
            for (int v = 0; v < 4; ++v) zt[gate][(i * 16 + q4 * 4 + v) * kEpiStride + (half + q) * 16 + l16] = acc[i][q][v];
    __syncthreads();
    if (wave < kUpdateWaves && node >= 0) {
        float z[4][4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const float4 q = *reinterpret_cast<const float4 *>(&zt[g][tr * kEpiStride + u4]);
            if constexpr (!HAS_Z) bq[g] = *reinterpret_cast<const float4 *>(s_bias + g * kUnit + u4);
            z[g][0] = q.x + bq[g].x; z[g][1] = q.y + bq[g].y; z[g][2] = q.z + bq[g].z; z[g][3] = q.w + bq[g].w;
        }
        const float ckv[4] = {ck.x, ck.y, ck.z, ck.w};
        float cc[4], go[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float gi = sigmoid_t<T>(z[0][e]);
            go[e] = sigmoid_t<T>(z[1][e]);
            const float gu = tanh_t<T>(z[2][e]);
            const float gf = sigmoid_t<T>(z[3][e]);
            cc[e] = gi * gu + gf * ckv[e];
        }
        store_state_shared<T>(a, node, unit0, make_float4(cc[0], cc[1], cc[2], cc[3]), make_float4(go[0], go[1], go[2], go[3]));
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // this wave's rows have arrived
    __syncthreads();
    if (tid == 0 && lv.n_levels > 1) __hip_atomic_fetch_add(lv.done + (int64_t)row_tile * lv.stride, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---- host side ---------------------------------------------------------------------
// Optional per-launch event pairs (see jitdb_profile_start in the header).
struct Profiler {
    bool on = false;
    int capacity = 0, used = 0;
    int64_t dropped = 0;
    hipEvent_t *begin = nullptr, *end = nullptr;
    int *cls = nullptr;
    int64_t *rows = nullptr;
    int64_t *edges = nullptr;
};
Profiler g_prof;

struct ScopedLaunchTimer {
    int slot = -1;
    hipStream_t st;
    // edges: children whose forget gates the launch computes in full (chain levels); else 0
    ScopedLaunchTimer(int kernel_class, int64_t rows, hipStream_t s, int64_t edges = 0) : st(s) {
        if (!g_prof.on) return;
        if (g_prof.used >= g_prof.capacity) { ++g_prof.dropped; return; }
        slot = g_prof.used++;
        g_prof.cls[slot] = kernel_class;
        g_prof.rows[slot] = rows;
        g_prof.edges[slot] = edges;
        (void)hipEventRecord(g_prof.begin[slot], st);
    }
    ~ScopedLaunchTimer() {
        if (slot >= 0) (void)hipEventRecord(g_prof.end[slot], st);
    }
};

// Forests filed tree after tree run as whole trees (trees.hip) up to kTreesMaxLevels levels below the chain levels.
constexpr int kTreesMaxLevels = 32;
constexpr int kTreesMaxSpan = 256;         // ... of trees of up to this many ids: one block runs a tree alone

struct ForwardWs {
    void *Bp;
    float *bp;
    void *stack;  // the current level's stacked input, (N + 256) rows of Dp + Hp
    float *Z;     // trees.hip: x parts of the gates [N][4][H rounded up to 16], in the memory of stack and P; nullptr: no room
    float *FC;    // trees.hip: every node's f c, [N, H rounded up to 16], behind Z
    int4 *row_rec; // row records of all level positions, two int4 each
    void *hs;     // nullptr when h_out can serve (H == Hp)
    void *P;
    float *cs;    // nullptr when c_out can serve (H == Hq)
    // tables that hold N-ary cells (jitdb_treelstm_forward_cells): one slot's stacked input and
    // pre-activations, each such cell's packed weights, the flag for nodes with too many children
    void *nary_A;
    float *nary_F;   // pre-activations of the forget gates of child positions 2 .. N of one slot
    void *nary_B[JITDB_MAX_SIGNATURES];
    int *nary_err;
    size_t bytes;
};

struct Dims {
    int D, H, Dp, Hp, Hu, NP;
    int Hq;       // H rounded up to 8: row stride of the side buffers (P, padded c)
    int NPU;      // rows of the packed U: padded so the projection's 8-unit-tile blocks stay inside
    size_t esz;
};

Dims make_dims(int D, int H, jitdb_dtype dtype) {
    Dims d;
    d.D = D; d.H = H;
    // K is padded to whole pipeline stages, so that only the last x stage can straddle D
    const int kpad = dtype == JITDB_F32 ? Traits<float>::BK : Traits<bf16_t>::BK;
    d.Dp = (int)round_up(D, kpad);
    d.Hp = (int)round_up(H, kpad);
    d.Hu = (int)round_up(H, 2 * kUnit);
    d.NP = 4 * d.Hu;
    d.Hq = (int)round_up(H, 8);
    d.NPU = (int)round_up(d.Hu / kUnit, 8) * kGateTile;
    d.esz = dtype == JITDB_F32 ? 4 : 2;
    return d;
}

// packed weights of one cell: bytes of Bp, floats of bp (one set per signature, back to back)
size_t packed_w_bytes(const Dims &d) { return (size_t)d.NPU * (d.Dp + d.Hp) * d.esz; }
ForwardWs carve_forward_ws(int64_t n, int64_t e, const Dims &d, void *base, int n_sig = 1,
                           const jitdb_cell_t *cells = nullptr, bool with_z = true) {
    Carver c(base);
    ForwardWs w = {};
    (void)e;
    w.Bp = c.take<char>(packed_w_bytes(d) * n_sig);
    w.bp = c.take<float>((size_t)d.NP * n_sig);
    w.row_rec = c.take<int4>((size_t)2 * (n + kRowPad));   // every level position
    w.hs = (d.H == d.Hp) ? nullptr : c.take<char>((size_t)n * d.Hp * d.esz);
    // The stacked input of one level at a time (whole row tiles are read, hence the 256 spare rows) and P, or, where whole trees
    // can run (one cell, at most n_trees nodes), Z and f c.  (Larger forests ask for no less than those, so that their
    // workspace holds any smaller one.)
    const int64_t n_trees = with_z && n_sig == 1 && !cells ? trees_max_nodes(d.D, d.H, d.esz) : 0;
    const int64_t n_z = n < n_trees ? n : n_trees;
    const size_t stack_bytes = (size_t)round_up((n + kRowPad) * (d.Dp + d.Hp) * (int64_t)d.esz, 256);
    const size_t level_bytes = stack_bytes + (size_t)n * d.Hq * d.esz;
    const size_t z_bytes = (size_t)n_z * 4 * round_up(d.H, 16) * 4, tree_bytes = z_bytes + z_bytes / 4;
    char *shared = c.take<char>(level_bytes > tree_bytes ? level_bytes : tree_bytes);
    w.stack = shared;
    if (shared) w.P = shared + stack_bytes;
    if (shared && n <= n_trees) {
        w.Z = reinterpret_cast<float *>(shared);
        w.FC = reinterpret_cast<float *>(shared + z_bytes);
    }
    w.cs = (d.H == d.Hq) ? nullptr : c.take<float>((size_t)n * d.Hq);
    int n_max = 0;
    for (int t = 0; cells && t < n_sig; ++t)
        if (cells[t].kind == JITDB_CELL_NARY) {
            n_max = cells[t].arity > n_max ? cells[t].arity : n_max;
            w.nary_B[t] = c.take<char>(nary_packed_bytes(d.D, d.H, d.Dp, d.Hp, cells[t].arity, d.esz));
        }
    if (n_max > 0) {
        w.nary_A = c.take<char>((size_t)(n + kRowPad) * (d.Dp + (size_t)n_max * d.Hp) * d.esz);
        w.nary_F = n_max > 1 ? c.take<float>((size_t)n * (n_max - 1) * d.H) : nullptr;
        w.nary_err = c.take<int>(1);
    }
    w.bytes = c.off;
    return w;
}

bool dims_ok(int64_t n, int64_t e, int32_t D, int32_t H, int dtype) {
    if (n < 0 || n > JITDB_MAX_NODES || e < 0 || e > n) return false;
    if (D < 1 || D > (1 << 16)) return false;
    if (H < 1 || H > (1 << 14)) return false;
    if (dtype != JITDB_F32 && dtype != JITDB_BF16) return false;
    return true;
}

// One batched evaluation per slot of the table, levels in ascending order.  Without `slots` a
// level is one slot and there is one cell; with it, slot (l, t) is evaluated by cell t (its
// own packed weights), and the records keep every row inside its slot.
// With `cells` (one per signature) every signature names a cell of its own TYPE: child-sum cells
// take the path of this file, N-ary cells the three steps of cells.hip; W, U, b then come from the
// cells.
template <typename T, bool SAVE>
int run_forward(const void *x, const void *W, const void *U, const float *b, const Dims &d,
                const jitdb_schedule_t *s, const jitdb_slots_t *slots, const jitdb_cell_t *cells,
                void *h_out, float *c_out, void *gates, void *fgate,
                const ForwardWs &w_in, const void *packed, bool chains, hipStream_t st) {
    // weights packed by an earlier jitdb_treelstm_pack are used where they lie
    ForwardWs w = w_in;
    const int n_sig_w = slots ? slots->n_sig : 1;
    if (packed) {
        w.Bp = const_cast<void *>(packed);
        w.bp = reinterpret_cast<float *>(static_cast<char *>(w.Bp) + round_up(packed_w_bytes(d) * n_sig_w, 256));
    }
    const int L = s->n_levels;
    const int n_sig = slots ? slots->n_sig : 1;
    const int32_t *sp = slots ? slots->host_slot_ptr : s->host_level_ptr;
    const jitdb_dtype dtype = std::is_same<T, float>::value ? JITDB_F32 : JITDB_BF16;
    auto is_nary = [&](int t) { return cells != nullptr && t >= 0 && cells[t].kind == JITDB_CELL_NARY; };
    bool any_nary = false;
    for (int t = 0; t < n_sig; ++t) any_nary = any_nary || is_nary(t);

    int thin_max = kThinMaxRows;
    if (sizeof(T) == 2 && thin_max > kThinMaxTiles * kDmaBM / (d.NP / kBN)) thin_max = kThinMaxTiles * kDmaBM / (d.NP / kBN);

    // Levels from chain_from on are thin and hold only nodes with exactly one child (the schedule says
    // how many children each level has): launches they share, no stack step, no projection.  A child
    // below chain_from whose parent is such a node needs no projection either, so the level right
    // below skips it too.
    int chain_from = L;
    const int chain_k_bytes = (d.Dp + d.Hp) * d.esz;
    constexpr int chain_us = sizeof(T) == 4 ? 2 : 1, chain_ahead = sizeof(T) == 4 ? kChainAloneAhead : kChainAhead;
    if (!SAVE && !slots && chains && s->host_level_kids && (d.D & 3) == 0 && chain_k_bytes <= kChainMaxKBytes) {
        for (int l = L - 1; l >= 1; --l) {
            const int rows = sp[l + 1] - sp[l];
            if (rows > kThinMaxRows || s->host_level_kids[l] != rows) break;
            chain_from = l;
        }
    }
    // The chain levels' words (a word per row tile, a counter per launch) stand where those levels' row records would.
    // With the library's event pairs on, a launch holds one level, so that every level has a time of its own; so it does without
    // inv_perm, which says where the rows are that a tile waits for.
    const int chain_per_launch = g_prof.on || !s->inv_perm ? 1 : kChainLevels;
    int *chain_words = nullptr;
    int64_t n_chain_words = 0, n_chain_tiles = 0;
    int chain_stride = 1, chain_rt = 1;
    if (chain_from < L) {
        chain_words = reinterpret_cast<int *>(w.row_rec + 2 * (int64_t)sp[chain_from]);
        for (int l = chain_from; l < L; ++l) n_chain_tiles += ceil_div(sp[l + 1] - sp[l], 16);
        if (sizeof(T) == 2 && chain_k_bytes <= kChainMaxKBytes2 && n_chain_tiles * (d.Hu / kUnit) >= (int64_t)kChainWideTiles * (L - chain_from)) {
            chain_rt = 2;
            n_chain_tiles = 0;
            for (int l = chain_from; l < L; ++l) n_chain_tiles += ceil_div(sp[l + 1] - sp[l], 32);
        }
        // (blocks that look at one line wait for each other: a line per word where the records' memory has room, else a fourth)
        const int64_t room = 8 * (s->n_nodes - sp[chain_from] + kRowPad) - (L - chain_from);
        chain_stride = 32 * n_chain_tiles <= room ? 32 : 4;
        n_chain_words = n_chain_tiles * chain_stride + (L - chain_from);
    }
    // A forest of small trees filed one after another: its levels below the chain levels in one launch
    TreesArgs ta = {};
    bool trees = false;
    const int32_t tree_window = known_tree_window(s);
    if (!slots && !any_nary && w.Z && tree_window > 0 && tree_window <= kTreesMaxSpan && s->inv_perm && chain_from <= kTreesMaxLevels) {
        ta.x = x; ta.Bp = w.Bp; ta.bp = w.bp;
        ta.height = s->height; ta.perm = s->perm; ta.inv_perm = s->inv_perm; ta.child_ptr = s->child_ptr; ta.child_idx = s->child_idx;
        ta.h_out = h_out; ta.hs = w.hs ? w.hs : h_out; ta.FC = w.FC; ta.gates = gates; ta.fgate = fgate;
        ta.c_out = c_out; ta.cs = chain_from < L ? w.cs : nullptr; ta.Z = w.Z;
        ta.n = (int)s->n_nodes; ta.n_leaves = sp[1]; ta.tree_window = tree_window; ta.l_end = chain_from;
        ta.D = d.D; ta.H = d.H; ta.Hp = d.Hp; ta.Hq = d.Hq; ta.NPU = d.NPU; ta.sx_packed = (int)(d.Dp * d.esz / 64);
        TreesShape shape = {L, sp[chain_from], 0.0, 0.0};
        for (int l = 1; l < chain_from; ++l) {
            const double per_node = (double)(sp[l] - sp[l - 1]) / (sp[l + 1] - sp[l]);
            shape.fan += per_node > 1.0 ? per_node : 1.0;
            shape.wide += per_node < 2.5 ? 0.0 : per_node < 18.5 ? per_node - 2.5 : 16.0;
        }
        trees = plan_trees(ta, d.esz, shape);
    }

    {   // row records and packed weights (one launch; cells named one by one: the further ones' weights one launch each)
        const bool one_behind_other = !cells;                       // the cells' weights: packed with the first one's
        const int64_t pieces = pack_pieces(d.NPU, d.Dp, d.Hp, d.esz) * (one_behind_other ? n_sig : 1);
        const unsigned pack_grid = (unsigned)(ceil_div(pieces, kThreads) < 4096 ? ceil_div(pieces, kThreads) : 4096);
        auto pack_args = [&](int t) {
            PackArgs p;
            if (cells) {
                p.W = cells[t].W; p.U = cells[t].U; p.b = cells[t].b;
            } else {
                p.W = static_cast<const T *>(W) + (size_t)t * 4 * d.H * d.D;
                p.U = static_cast<const T *>(U) + (size_t)t * 4 * d.H * d.H;
                p.b = b + (size_t)t * 4 * d.H;
            }
            p.D = d.D; p.H = d.H; p.Dp = d.Dp; p.Hp = d.Hp; p.NP = d.NP; p.NPU = d.NPU; p.n_cells = one_behind_other ? n_sig : 1;
            p.Bp = static_cast<char *>(w.Bp) + packed_w_bytes(d) * t;
            p.bp = w.bp + (size_t)d.NP * t;
            return p;
        };
        const bool pack_here = !(packed || is_nary(0));
        // records of the levels that run one by one; the chain levels' words are cleared in the same launch
        const int rec_end = trees ? 0 : sp[chain_from * (slots ? n_sig * n_sig : 1)];
        const bool large = rec_end > 0 && s->n_nodes >= (SAVE ? kRecLargeMinNodesSave : kRecLargeMinNodes);      // (whole trees have no records: perhaps nothing to launch)
        {
            const int per_window = large ? kRecWindowLarge : kRecWindow;
            const int n_windows = (int)ceil_div((int64_t)rec_end, per_window);
            if (large) {
                const unsigned pg = pack_here ? (unsigned)(ceil_div(pieces, kRecThreadsLarge) < 1024 ? ceil_div(pieces, kRecThreadsLarge) : 1024) : 0u;
                ScopedLaunchTimer tm(JITDB_K_PACK, 0, st);
                prepare_large_kernel<T><<<(unsigned)n_windows + pg, kRecThreadsLarge, 0, st>>>(
                    s->perm, slots ? slots->key : s->height, s->child_ptr, s->child_idx, w.row_rec, (int)s->n_nodes, rec_end,
                    n_windows, pack_args(0), chain_words, n_chain_words);
                JITDB_LAUNCH_CHECK();
            } else {
                PackArgs p = pack_args(0);
                unsigned grid = (unsigned)n_windows + (pack_here ? pack_grid : 0u);
                if (grid == 0 && n_chain_words > 0) {      // nothing but words to clear
                    grid = (unsigned)(ceil_div(n_chain_words, kThreads) < 256 ? ceil_div(n_chain_words, kThreads) : 256);
                    p.n_cells = 0;
                }
                if (grid > 0) {
                    ScopedLaunchTimer tm(JITDB_K_PACK, 0, st);
                    prepare_kernel<T><<<grid, kThreads, 0, st>>>(
                        s->perm, slots ? slots->key : s->height, s->child_ptr, s->child_idx, w.row_rec, (int)s->n_nodes, rec_end,
                        n_windows, p, chain_words, n_chain_words);
                    JITDB_LAUNCH_CHECK();
                }
            }
        }
        for (int t = 1; t < n_sig && !packed && !one_behind_other; ++t) {
            if (is_nary(t)) continue;
            ScopedLaunchTimer tm(JITDB_K_PACK, 0, st);
            pack_weights_kernel<T><<<pack_grid, kThreads, 0, st>>>(pack_args(t));
            JITDB_LAUNCH_CHECK();
        }
        for (int t = 0; t < n_sig; ++t) {
            if (!is_nary(t)) continue;
            ScopedLaunchTimer tm(JITDB_K_PACK, 0, st);
            // (every such launch also clears the flag for nodes with too many children)
            const int rc = nary_pack(dtype, cells[t].W, cells[t].U, d.D, d.H, d.Dp, d.Hp, cells[t].arity, w.nary_B[t],
                                     w.nary_err, st);
            if (rc != JITDB_OK) return rc;
        }
    }

    LevelArgs a;
    a.proj_nodes = nullptr;
    a.ranges = nullptr;
    a.n_ranges = 0; a.range_stride = 0; a.range_cells = 0;
    a.stack = w.stack;
    a.hs = w.hs ? w.hs : h_out;
    a.x = x;
    a.child_idx = s->child_idx;

    a.P = w.P; a.c_out = c_out; a.h_out = h_out;
    a.cs = w.cs ? w.cs : c_out;
    a.Hq = d.Hq;
    a.hs_out = w.hs ? w.hs : h_out;
    a.gates = gates;
    a.fgate = fgate;
    a.Z = w.Z;
    a.Hz = (int)round_up(d.H, 16);
    a.D = d.D; a.Dp = d.Dp; a.H = d.H; a.Hp = d.Hp; a.Hu = d.Hu;
    a.NPU = d.NPU;

    // The table's ranges: slot (l, t) = the cell's batch = sub-slots (l, t, 0 .. n_sig-1); the
    // projection of sub-slot (l, t, p) uses the forget weights of cell p, the parent's.
    const int T2 = n_sig * n_sig;
    auto slot_begin = [&](int l, int t) { return sp[(l * n_sig + t) * (slots ? n_sig : 1)]; };
    auto sub_begin = [&](int l, int t, int p) { return sp[(l * n_sig + t) * n_sig + p]; };
    // The launches in order: one per non-empty slot, except that a level of a typed table with more than one
    // slot or sub-slot runs them all in one grouped launch (sig = -1; n_tiles / n_proj_tiles = row tiles of
    // tile_rows rows when every slot / sub-slot is cut into tiles of its own).  One thin launch costs 12 to 20 us
    // whatever it holds: four cells in 8192 trees (295 k nodes, H 512, bf16)
    // took 2.39 ms with a launch per cell on thin levels and takes 2.00 like this, six in 2.6 k nodes (H 118, fp32) 0.89 -> 0.21.
    struct Seg { int l, sig, begin, rows, tile_rows, n_tiles, n_proj_tiles; };
    std::vector<Seg> segs;
    segs.reserve((size_t)L * n_sig);
    for (int l = 0; l < L; ++l) {
        const int lvl_rows = slot_begin(l + 1, 0) - slot_begin(l, 0);
        const int tile_rows = lvl_rows <= thin_max ? 32 : kDmaBM;
        int n_tiles = 0, n_proj_tiles = 0, used = 0, subs = 0;
        for (int t = 0; t < n_sig; ++t) {
            const int r = slot_begin(l, t + 1) - slot_begin(l, t);
            if (r < 0 || (r == 0 && !slots)) return JITDB_E_SCHEDULE;
            n_tiles += (int)ceil_div(r, tile_rows);
            used += r > 0;
            for (int p = 0; slots && p < n_sig; ++p) {
                const int rp = sub_begin(l, t, p + 1) - sub_begin(l, t, p);
                n_proj_tiles += (int)ceil_div(rp, tile_rows);
                subs += rp > 0;
            }
        }
        if ((used > 1 || subs > 1) && !any_nary) {
            segs.push_back({l, -1, slot_begin(l, 0), lvl_rows, tile_rows, n_tiles, n_proj_tiles});
        } else {
            for (int t = 0; t < n_sig; ++t) {
                const int r = slot_begin(l, t + 1) - slot_begin(l, t);
                if (r > 0) segs.push_back({l, t, slot_begin(l, t), r, 0, 0, 0});
            }
        }
    }
    // stack: gather a slot's x rows and child sums into one dense matrix
    auto stack_args = [&](const Seg &g) {
        StackArgs sa;
        sa.x = x; sa.D = d.D; sa.Dp = d.Dp; sa.hs = a.hs; sa.Hp = d.Hp;
        sa.row_rec = w.row_rec + 2 * (int64_t)g.begin; sa.child_idx = s->child_idx;
        sa.A = w.stack; sa.n_rows = g.rows; sa.n_rows_alloc = (int)round_up(g.rows, kRowPad);
        return sa;
    };
    auto stack_blocks = [&](const Seg &g) { return stack_grid(g.rows, (int64_t)(d.Dp + d.Hp) * (int64_t)sizeof(T)); };
    bool stacked_ahead = false;     // the slot's stack step already ran with the projection before it
    const int n_unit_tiles = d.Hu / kUnit;
    a.w_bytes = (int64_t)packed_w_bytes(d);
    a.NP = d.NP;

    if (trees) {
        ScopedLaunchTimer tm(JITDB_K_TREES, chain_from < L ? sp[chain_from] : s->n_nodes, st);
        const int rc = launch_trees(dtype, SAVE, ta, st);
        if (rc != JITDB_OK) return rc;
    }
    for (size_t i = 0; i < segs.size(); ++i) {
        if (trees || segs[i].l >= chain_from) break;      // (of trees, the chain levels are all that is left)
        const int l = segs[i].l, sig = segs[i].sig, n_rows = segs[i].rows;
        const bool grouped = sig < 0;
        a.Bp = static_cast<char *>(w.Bp) + packed_w_bytes(d) * (grouped ? 0 : sig);
        a.bp = w.bp + (size_t)d.NP * (grouped ? 0 : sig);
        a.row_rec = w.row_rec + 2 * (int64_t)segs[i].begin;
        a.n_rows = n_rows;
        a.n_rows_alloc = (int)round_up(n_rows, kRowPad);
        const int row_tiles = grouped ? segs[i].n_tiles : (int)ceil_div(n_rows, kDmaBM);
        if (grouped) {      // the level's ranges: its slots for the cell, its sub-slots for the projection
            a.ranges = slots->slot_ptr + (int64_t)l * T2;
            a.n_ranges = n_sig; a.range_stride = n_sig; a.range_cells = n_sig;
        }
        if (is_nary(sig)) {
            // a slot of N-ary nodes: stack, one contraction for all 3 + N gates, cell update (cells.hip)
            NarySlot ns;
            ns.x = x; ns.row_rec = a.row_rec; ns.A = w.nary_A; ns.Bn = w.nary_B[sig]; ns.b = cells[sig].b;
            ns.F = w.nary_F; ns.err = w.nary_err; ns.n_rows = n_rows; ns.N = cells[sig].arity; ns.leaves = l == 0;
            ScopedLaunchTimer tm(l == 0 ? JITDB_K_THIN_LEAF : JITDB_K_THIN_INTERNAL, n_rows, st);
            const int rc = run_nary_slot(dtype, a, ns, st);
            if (rc != JITDB_OK) return rc;
        } else {
            if (!stacked_ahead) {
                const StackArgs sa = stack_args(segs[i]);
                ScopedLaunchTimer tm(JITDB_K_STACK, n_rows, st);
                if (l == 0)
                    stack_x_kernel<T><<<stack_dims(ceil_div((int64_t)n_rows * (d.Dp / Traits<T>::VEC), kThreads)), kThreads, 0, st>>>(sa);
                else
                    stack_kernel<T><<<stack_dims(stack_blocks(segs[i])), kThreads, 0, st>>>(sa);
                JITDB_LAUNCH_CHECK();
            }
            stacked_ahead = false;
            // levels too small to fill the chip with tiles go to the thin kernel
            bool thin = n_rows <= thin_max;      // (of a grouped launch: the whole level's)
            if (!thin && !SAVE && !slots && l > 0 && s->host_level_kids && n_rows <= kThinMaxRowsLongLists &&
                s->host_level_kids[l] >= (int64_t)kThinLongLists * n_rows)
                thin = true;
            if (thin) {
                a.n_col_tiles = n_unit_tiles;
                a.n_tiles = (grouped ? row_tiles : (int)ceil_div(n_rows, 32)) * a.n_col_tiles;
                a.n_blocks = a.n_tiles;
            } else {
                a.n_col_tiles = d.NP / kBN;
                a.n_tiles = 0;
                a.n_row_tiles = row_tiles;
                a.n_blocks = 8 * (int)ceil_div(row_tiles, 8) * a.n_col_tiles;
            }
            {
                ScopedLaunchTimer tm(thin ? (l == 0 ? JITDB_K_THIN_LEAF : JITDB_K_THIN_INTERNAL)
                                          : (l == 0 ? JITDB_K_LEAF : JITDB_K_INTERNAL), n_rows, st);
                if (thin && grouped) {
                    if (l == 0)
                        thin_kernel<T, MODE_LEAF, false, true><<<a.n_blocks, kThinWaves * 64, 0, st>>>(a);
                    else
                        thin_kernel<T, MODE_INTERNAL, false, true><<<a.n_blocks, kThinWaves * 64, 0, st>>>(a);
                } else if (thin) {
                    if (l == 0)
                        thin_kernel<T, MODE_LEAF, SAVE><<<a.n_blocks, kThinWaves * 64, 0, st>>>(a);
                    else
                        thin_kernel<T, MODE_INTERNAL, SAVE><<<a.n_blocks, kThinWaves * 64, 0, st>>>(a);
                } else if (grouped) {
                    if (l == 0)
                        level_kernel<T, MODE_LEAF, false, true><<<a.n_blocks, kDmaThreads, 0, st>>>(a);
                    else
                        level_kernel<T, MODE_INTERNAL, false, true><<<a.n_blocks, kDmaThreads, 0, st>>>(a);
                } else {
                    if (l == 0)
                        level_kernel<T, MODE_LEAF, SAVE><<<a.n_blocks, kDmaThreads, 0, st>>>(a);
                    else
                        level_kernel<T, MODE_INTERNAL, SAVE><<<a.n_blocks, kDmaThreads, 0, st>>>(a);
                }
            }
            JITDB_LAUNCH_CHECK();
        }
        if (l + 1 >= L) continue;     // the top level has no parents to project for
        if (l + 1 >= chain_from) continue;   // every parent is a chain node: U_f h_k is part of its own launch

        // Forget projections of these nodes (roots' rows go unused), with the PARENT's weights.
        if (grouped) {
            const bool thin_p = n_rows <= thin_max;
            ScopedLaunchTimer tm(thin_p ? JITDB_K_THIN_PROJ : JITDB_K_PROJ, n_rows, st);
            a.Bp = w.Bp; a.bp = w.bp;
            a.n_ranges = T2; a.range_stride = 1;
            if (!thin_p) {
                a.n_col_tiles = (int)ceil_div(n_unit_tiles, 8);
                a.n_row_tiles = segs[i].n_proj_tiles;
                a.n_blocks = 8 * (int)ceil_div(a.n_row_tiles, 8) * a.n_col_tiles;
                level_kernel<T, MODE_PROJ, false, true><<<a.n_blocks, kDmaThreads, 0, st>>>(a);
            } else {
                a.n_col_tiles = (int)ceil_div(n_unit_tiles, 4);
                a.n_tiles = segs[i].n_proj_tiles * a.n_col_tiles;
                a.n_blocks = a.n_tiles;
                if (i + 1 < segs.size() && segs[i + 1].rows <= thin_max) {     // as below: the next stack step rides along
                    thin_proj_stack_kernel<T, true><<<a.n_blocks + stack_blocks(segs[i + 1]), kThinWaves * 64, 0, st>>>(
                        a, stack_args(segs[i + 1]));
                    stacked_ahead = true;
                } else {
                    thin_kernel<T, MODE_PROJ, false, true><<<a.n_blocks, kThinWaves * 64, 0, st>>>(a);
                }
            }
            JITDB_LAUNCH_CHECK();
            continue;
        }
        // one launch per non-empty sub-slot (a single one without a typed table)
        const int n_sub = slots ? n_sig : 1;
        int last_sub = -1;
        // (an N-ary parent needs no projection of its children: its forget gates are part of its own contraction)
        for (int p = 0; p < n_sub; ++p)
            if ((!slots || sub_begin(l, sig, p + 1) > sub_begin(l, sig, p)) && !is_nary(slots ? p : -1)) last_sub = p;
        for (int p = 0; p < n_sub; ++p) {
            const int begin = slots ? sub_begin(l, sig, p) : segs[i].begin;
            const int rows = slots ? sub_begin(l, sig, p + 1) - begin : n_rows;
            if (rows <= 0 || is_nary(slots ? p : -1)) continue;
            a.Bp = static_cast<char *>(w.Bp) + packed_w_bytes(d) * p;
            a.bp = w.bp + (size_t)d.NP * p;
            a.row_rec = w.row_rec + 2 * (int64_t)begin;
            a.proj_nodes = slots ? nullptr : s->perm + begin;
            a.n_rows = rows;
            const bool thin_p = rows <= thin_max;
            ScopedLaunchTimer tm(thin_p ? JITDB_K_THIN_PROJ : JITDB_K_PROJ, rows, st);
            if (thin_p) {
                a.n_col_tiles = (int)ceil_div(n_unit_tiles, 4);
                a.n_tiles = (int)ceil_div(rows, 32) * a.n_col_tiles;
                a.n_blocks = a.n_tiles;
                // the stack step of the next slot, if that is thin too, rides along with the slot's
                // last projection (the level kernel above was the stack buffer's only reader); its
                // rows are counted with this launch's class
                if (p == last_sub && i + 1 < segs.size() && segs[i + 1].l > 0 && segs[i + 1].rows <= thin_max &&
                    !is_nary(segs[i + 1].sig)) {
                    thin_proj_stack_kernel<T><<<a.n_blocks + stack_blocks(segs[i + 1]), kThinWaves * 64, 0, st>>>(
                        a, stack_args(segs[i + 1]));
                    stacked_ahead = true;
                } else {
                    thin_kernel<T, MODE_PROJ><<<a.n_blocks, kThinWaves * 64, 0, st>>>(a);
                }
            } else {
                a.n_col_tiles = (int)ceil_div(n_unit_tiles, 8);
                a.n_row_tiles = (int)ceil_div(rows, kDmaBM);
                a.n_blocks = 8 * (int)ceil_div(a.n_row_tiles, 8) * a.n_col_tiles;
                level_kernel<T, MODE_PROJ><<<a.n_blocks, kDmaThreads, 0, st>>>(a);
            }
            JITDB_LAUNCH_CHECK();
        }
    }
    const void *lds_set = nullptr;      // the kernel that may ask for its LDS
    int *done = chain_words, *ticket = chain_words ? chain_words + n_chain_tiles * chain_stride : nullptr;
    for (int l0 = chain_from; l0 < L;) {
        ChainArgs lv;
        lv.perm = s->perm; lv.inv_perm = s->inv_perm; lv.child_ptr = s->child_ptr; lv.child_idx = s->child_idx;
        lv.n_levels = 0;
        lv.done = done;
        lv.ticket = ticket++;
        lv.tiles[0] = 0;
        lv.pos[0] = sp[l0];
        int rt = chain_rt;
        bool alone = false;
        while (l0 < L && lv.n_levels < chain_per_launch) {
            const int tiles = (int)ceil_div(sp[l0 + 1] - sp[l0], 16 * chain_rt), i = lv.n_levels;
            alone = (int64_t)tiles * n_unit_tiles >= kChainAloneTiles;
            if (alone && i > 0) { alone = false; break; }
            if (alone) rt = chain_k_bytes <= (sizeof(T) == 4 ? kChainAloneMaxKBytes2 : kChainMaxKBytes) ? 2 : 1;
            lv.tiles[i + 1] = lv.tiles[i] + (rt == chain_rt ? tiles : (int)ceil_div(sp[l0 + 1] - sp[l0], 16 * rt));
            lv.pos[i + 1] = sp[++l0];
            lv.n_levels = i + 1;
            if (alone) break;
        }
        const int n_tiles = lv.tiles[lv.n_levels];
        lv.stride = chain_stride;
        done += (int64_t)n_tiles * chain_stride;
        a.Bp = w.Bp; a.bp = w.bp;
        a.n_col_tiles = n_unit_tiles;
        a.n_blocks = n_tiles * n_unit_tiles;
        const unsigned grid = (unsigned)a.n_blocks;
        const int rows = lv.pos[lv.n_levels] - lv.pos[0];
        ScopedLaunchTimer tm(JITDB_K_CHAIN, rows, st, rows);         // (one child a row)
        // (of whole trees the x part is in Z: the h part alone)
        const size_t lds = (size_t)chain_lds_bytes(trees ? d.Hp * (int)d.esz : chain_k_bytes, rt);
        constexpr int nt = kThinWaves * 64 * chain_us;
        const auto fn = alone ? (rt == 2 ? (trees ? &chain_kernel<T, chain_us, 2, true, chain_ahead> : &chain_kernel<T, chain_us, 2, false, chain_ahead>)
                                         : (trees ? &chain_kernel<T, chain_us, 1, true, chain_ahead> : &chain_kernel<T, chain_us, 1, false, chain_ahead>))
                              : (rt == 2 ? (trees ? &chain_kernel<T, chain_us, 2, true> : &chain_kernel<T, chain_us, 2, false>)
                                         : (trees ? &chain_kernel<T, chain_us, 1, true> : &chain_kernel<T, chain_us, 1, false>));
        // more dynamic LDS than a launch may ask for by default (always the same, whatever this call needs: other threads' calls set it too)
        if (reinterpret_cast<const void *>(fn) != lds_set) {
            lds_set = reinterpret_cast<const void *>(fn);
            JITDB_HIP_CHECK(hipFuncSetAttribute(lds_set, hipFuncAttributeMaxDynamicSharedMemorySize, kChainLdsMax));
        }
        fn<<<grid, nt, lds, st>>>(a, lv);
        JITDB_LAUNCH_CHECK();
    }
    return JITDB_OK;
}

}  // namespace

// Slots of up to this many 128 x 256 tiles (4096 rows at H 256) take the thin kernel.  Schedule + forward, us, at 0 / 64 /
// 128 / 256 / 512 tiles: 270 k nodes H 256 N 2 bf16 1732 / 1572 / 1551 / 1584 / 1656; 733 k nodes H 150 N 3 bf16 2431 /
// 2315 / 2293 / 2311 / 2370; 8.9 k nodes H 150 N 2 fp32 1019 / 308 / 293 / 292 / 295.
constexpr int kNaryThinTiles = 128;
bool nary_slot_is_thin(int64_t rows, int n_col_tiles) {
    return ceil_div(rows, kDmaBM) * n_col_tiles <= kNaryThinTiles;
}

int launch_nary_level(jitdb_dtype dtype, const NaryLevel &g, hipStream_t st) {
    if (g.M <= 0) return JITDB_OK;
    if (g.k_bytes <= 0 || g.k_bytes % 128 != 0) return JITDB_E_BADARG;
    LevelArgs a = {};
    a.stack = g.A;
    a.n_rows_alloc = (int)g.a_rows_alloc;
    a.Bp = g.B;
    a.NPU = (int)g.b_rows_alloc;
    a.n_rows = g.M;
    a.Dp = (int)(g.k_bytes / (dtype == JITDB_F32 ? 4 : 2));
    a.Hp = 0;
    a.n_row_tiles = (int)ceil_div(g.M, kDmaBM);
    a.n_col_tiles = g.n_col_tiles;
    a.n_blocks = 8 * (int)ceil_div(a.n_row_tiles, 8) * a.n_col_tiles;
    NaryEpi e;
    e.row_rec = g.row_rec; e.bias = g.bias; e.cs = g.cs; e.F = g.F; e.c_out = g.c_out; e.h_out = g.h_out; e.hs_out = g.hs_out;
    e.cs_out = g.cs_out; e.M = g.M; e.H = g.H; e.Hp = g.Hp; e.Hq = g.Hq; e.N = g.N;
    if (nary_slot_is_thin(g.M, g.n_col_tiles)) {
        a.c_out = g.c_out; a.h_out = g.h_out; a.hs_out = g.hs_out; a.cs = g.cs_out;
        a.H = g.H; a.Hq = g.Hq; a.Hp = g.Hp;               // (K is a.Dp here; Hp is the padded h copy's stride)
        a.n_col_tiles = 2 * g.n_col_tiles;
        const unsigned blocks = (unsigned)(ceil_div(g.M, 32) * a.n_col_tiles);
        const int threads = 64 * (g.leaves ? 3 : 3 + g.N);
        if (dtype == JITDB_F32) {
            if (g.leaves) nary_thin_kernel<float, true><<<blocks, threads, 0, st>>>(a, e, g.Bx, g.bx_rows_alloc);
            else nary_thin_kernel<float, false><<<blocks, threads, 0, st>>>(a, e, g.Bx, g.bx_rows_alloc);
        } else {
            if (g.leaves) nary_thin_kernel<bf16_t, true><<<blocks, threads, 0, st>>>(a, e, g.Bx, g.bx_rows_alloc);
            else nary_thin_kernel<bf16_t, false><<<blocks, threads, 0, st>>>(a, e, g.Bx, g.bx_rows_alloc);
        }
        JITDB_LAUNCH_CHECK();
        return JITDB_OK;
    }
    dim3 grid((unsigned)a.n_blocks);
    if (dtype == JITDB_F32) {
        if (g.leaves) nary_level_kernel<float, true><<<grid, kDmaThreads, 0, st>>>(a, e);
        else nary_level_kernel<float, false><<<grid, kDmaThreads, 0, st>>>(a, e);
    } else {
        if (g.leaves) nary_level_kernel<bf16_t, true><<<grid, kDmaThreads, 0, st>>>(a, e);
        else nary_level_kernel<bf16_t, false><<<grid, kDmaThreads, 0, st>>>(a, e);
    }
    JITDB_LAUNCH_CHECK();
    return JITDB_OK;
}

int launch_kb_gemm(jitdb_dtype dtype, const KbGemm &g, hipStream_t st) {
    if (g.M <= 0 || g.N <= 0 || g.k_bytes <= 0) return JITDB_OK;
    if (g.k_bytes % 128 != 0) return JITDB_E_BADARG;
    LevelArgs a = {};
    a.stack = g.A;
    a.n_rows_alloc = (int)g.a_rows_alloc;
    a.Bp = g.B;
    a.NPU = (int)g.b_rows_alloc;
    a.n_rows = g.M;
    a.n_row_tiles = (int)ceil_div(g.M, kDmaBM);
    a.n_col_tiles = (int)ceil_div(g.N, kBN);
    a.n_blocks = 8 * (int)ceil_div(a.n_row_tiles, 8) * a.n_col_tiles;
    a.Dp = (int)(g.k_bytes / (dtype == JITDB_F32 ? 4 : 2));
    const KbEpiArgs e = {g.out, g.ldc, g.M, g.N};
    dim3 grid((unsigned)a.n_blocks);
    if (dtype == JITDB_F32) gemm_kb_kernel<float><<<grid, kDmaThreads, 0, st>>>(a, e);
    else gemm_kb_kernel<bf16_t><<<grid, kDmaThreads, 0, st>>>(a, e);
    JITDB_LAUNCH_CHECK();
    return JITDB_OK;
}

}  // namespace jitdb

using namespace jitdb;


namespace {
void profiler_release() {
    for (int i = 0; i < g_prof.capacity; ++i) {
        if (g_prof.begin && g_prof.begin[i]) (void)hipEventDestroy(g_prof.begin[i]);
        if (g_prof.end && g_prof.end[i]) (void)hipEventDestroy(g_prof.end[i]);
    }
    delete[] g_prof.begin; delete[] g_prof.end; delete[] g_prof.cls; delete[] g_prof.rows; delete[] g_prof.edges;
    g_prof = Profiler();
}
}  // namespace

extern "C" int jitdb_profile_start(int32_t capacity) {
    if (capacity < 1 || capacity > (1 << 20)) return JITDB_E_BADARG;
    if (g_prof.on) return JITDB_E_BADARG;
    // value-initialised arrays: an event handle that was never created stays null and is not destroyed
    g_prof.begin = new (std::nothrow) hipEvent_t[capacity]();
    g_prof.end = new (std::nothrow) hipEvent_t[capacity]();
    g_prof.cls = new (std::nothrow) int[capacity]();
    g_prof.rows = new (std::nothrow) int64_t[capacity]();
    g_prof.edges = new (std::nothrow) int64_t[capacity]();
    g_prof.capacity = capacity;
    if (!g_prof.begin || !g_prof.end || !g_prof.cls || !g_prof.rows || !g_prof.edges) {
        profiler_release();
        return JITDB_E_NOMEM;
    }
    for (int i = 0; i < capacity; ++i) {
        if (hipEventCreate(&g_prof.begin[i]) != hipSuccess || hipEventCreate(&g_prof.end[i]) != hipSuccess) {
            profiler_release();      // the events created so far go back
            return JITDB_E_HIP;
        }
    }
    g_prof.used = 0;
    g_prof.dropped = 0;
    g_prof.on = true;
    return JITDB_OK;
}

extern "C" int jitdb_profile_stop(jitdb_profile_t *out) {
    if (!out) return JITDB_E_NULL;
    if (!g_prof.on) return JITDB_E_BADARG;
    g_prof.on = false;
    int rc = JITDB_OK;
    for (int c = 0; c < JITDB_K_CLASSES; ++c) { out->ms[c] = 0.0; out->launches[c] = 0; out->rows[c] = 0; out->edges[c] = 0; }
    out->dropped = g_prof.dropped;
    for (int i = 0; i < g_prof.used; ++i) {
        float ms = 0.0f;
        if (hipEventSynchronize(g_prof.end[i]) != hipSuccess ||
            hipEventElapsedTime(&ms, g_prof.begin[i], g_prof.end[i]) != hipSuccess) {
            rc = JITDB_E_HIP;
            continue;
        }
        out->ms[g_prof.cls[i]] += ms;
        out->launches[g_prof.cls[i]] += 1;
        out->rows[g_prof.cls[i]] += g_prof.rows[i];
        out->edges[g_prof.cls[i]] += g_prof.edges[i];
    }
    profiler_release();
    return rc;
}

extern "C" size_t jitdb_treelstm_workspace_bytes(int64_t n_nodes, int64_t n_edges,
                                                 int32_t D, int32_t H, jitdb_dtype dtype) {
    if (!dims_ok(n_nodes, n_edges, D, H, (int)dtype)) return 0;
    const Dims d = make_dims(D, H, dtype);
    return carve_forward_ws(n_nodes, n_edges, d, nullptr).bytes;
}

namespace {
int forward_entry(const void *x, const void *W, const void *U, const float *b, int32_t D, int32_t H,
                  jitdb_dtype dtype, const jitdb_schedule_t *s, const jitdb_slots_t *slots,
                  void *h_out, float *c_out, void *gates, void *fgate, bool save,
                  void *workspace, size_t workspace_bytes, void *hip_stream, const void *packed = nullptr,
                  const jitdb_cell_t *cells = nullptr) {
    if (!s) return JITDB_E_NULL;
    const int n_sig = slots ? slots->n_sig : 1;
    if (n_sig < 1 || n_sig > JITDB_MAX_SIGNATURES) return JITDB_E_BADARG;
    for (int t = 0; cells && t < n_sig; ++t) {
        if (cells[t].kind != JITDB_CELL_CHILDSUM && cells[t].kind != JITDB_CELL_NARY) return JITDB_E_BADARG;
        if (cells[t].kind == JITDB_CELL_NARY && (cells[t].arity < 1 || cells[t].arity > JITDB_MAX_NARY)) return JITDB_E_BADARG;
        if (!cells[t].W || !cells[t].U || !cells[t].b) return JITDB_E_NULL;
    }
    drop_stale_hip_error();
    const int64_t n = s->n_nodes;
    if (!dims_ok(n, s->n_edges, D, H, (int)dtype)) return JITDB_E_BADARG;
    if (n == 0) return JITDB_OK;
    if (!x || !h_out || !c_out || !workspace) return JITDB_E_NULL;
    if (!packed && !cells && (!W || !U || !b)) return JITDB_E_NULL;
    if (packed && (reinterpret_cast<uintptr_t>(packed) & 255) != 0) return JITDB_E_BADARG;
    if (save && (!gates || !fgate)) return JITDB_E_NULL;
    if (!s->perm || !s->height || !s->child_ptr || !s->child_idx || !s->host_level_ptr) return JITDB_E_NULL;
    if ((reinterpret_cast<uintptr_t>(workspace) & 255) != 0) return JITDB_E_BADARG;
    // rows are fetched in 16-byte pieces where their stride allows
    if ((reinterpret_cast<uintptr_t>(x) & 15) != 0) return JITDB_E_BADARG;
    if ((reinterpret_cast<uintptr_t>(h_out) & 15) != 0) return JITDB_E_BADARG;
    if ((reinterpret_cast<uintptr_t>(c_out) & 15) != 0) return JITDB_E_BADARG;
    const int L = s->n_levels;
    if (L < 1 || L > n) return JITDB_E_SCHEDULE;
    if (s->host_level_ptr[0] != 0 || s->host_level_ptr[L] != n) return JITDB_E_SCHEDULE;
    for (int l = 0; l < L; ++l)
        if (s->host_level_ptr[l + 1] <= s->host_level_ptr[l]) return JITDB_E_SCHEDULE;
    if (slots) {
        if (!slots->key || !slots->slot_ptr || !slots->host_slot_ptr) return JITDB_E_NULL;
        const int64_t T2 = (int64_t)n_sig * n_sig;
        if (slots->slot_capacity < L * T2 + 1) return JITDB_E_SCHEDULE;
        for (int64_t q = 0; q < L * T2; ++q)
            if (slots->host_slot_ptr[q + 1] < slots->host_slot_ptr[q]) return JITDB_E_SCHEDULE;
        for (int l = 0; l <= L; ++l)
            if (slots->host_slot_ptr[l * T2] != s->host_level_ptr[l]) return JITDB_E_SCHEDULE;
    }

    const Dims d = make_dims(D, H, dtype);
    ForwardWs w = carve_forward_ws(n, s->n_edges, d, workspace, n_sig, cells);
    if (workspace_bytes < w.bytes)     // without the room for whole trees: the fixed array, a workspace of a table's size
        w = carve_forward_ws(n, s->n_edges, d, workspace, n_sig, cells, false);
    if (workspace_bytes < w.bytes) return JITDB_E_WORKSPACE;
    // a table with one child-sum cell is the plain forward (but keeps the general launches for chain levels)
    const bool chains = slots == nullptr;
    if (n_sig == 1 && !cells) slots = nullptr;
    hipStream_t st = (hipStream_t)hip_stream;
    // run_forward keeps its list of launches in a std::vector: an allocation failure becomes a status
    JITDB_ABI_TRY
    if (dtype == JITDB_F32) {
        if (save) return run_forward<float, true>(x, W, U, b, d, s, slots, cells, h_out, c_out, gates, fgate, w, packed, chains, st);
        return run_forward<float, false>(x, W, U, b, d, s, slots, cells, h_out, c_out, nullptr, nullptr, w, packed, chains, st);
    }
    if (save) return run_forward<bf16_t, true>(x, W, U, b, d, s, slots, cells, h_out, c_out, gates, fgate, w, packed, chains, st);
    return run_forward<bf16_t, false>(x, W, U, b, d, s, slots, cells, h_out, c_out, nullptr, nullptr, w, packed, chains, st);
    JITDB_ABI_CATCH
}

size_t packed_total_bytes(const Dims &d, int n_sig) {
    return (size_t)round_up(packed_w_bytes(d) * n_sig, 256) + (size_t)round_up((int64_t)d.NP * n_sig * 4, 256);
}
}  // namespace

extern "C" size_t jitdb_treelstm_packed_bytes(int32_t D, int32_t H, jitdb_dtype dtype, int32_t n_sig) {
    if (!dims_ok(0, 0, D, H, (int)dtype) || n_sig < 1 || n_sig > JITDB_MAX_SIGNATURES) return 0;
    return packed_total_bytes(make_dims(D, H, dtype), n_sig);
}

extern "C" int jitdb_treelstm_pack(const void *W, const void *U, const float *b, int32_t D, int32_t H,
                                   jitdb_dtype dtype, int32_t n_sig, void *packed, size_t packed_bytes,
                                   void *hip_stream) {
    if (!W || !U || !b || !packed) return JITDB_E_NULL;
    if (!dims_ok(0, 0, D, H, (int)dtype) || n_sig < 1 || n_sig > JITDB_MAX_SIGNATURES) return JITDB_E_BADARG;
    if ((reinterpret_cast<uintptr_t>(packed) & 255) != 0) return JITDB_E_BADARG;
    drop_stale_hip_error();
    const Dims d = make_dims(D, H, dtype);
    if (packed_bytes < packed_total_bytes(d, n_sig)) return JITDB_E_WORKSPACE;
    hipStream_t st = (hipStream_t)hip_stream;
    const int64_t pieces = pack_pieces(d.NPU, d.Dp, d.Hp, d.esz) * n_sig;
    const unsigned grid = (unsigned)(ceil_div(pieces, kThreads) < 4096 ? ceil_div(pieces, kThreads) : 4096);
    PackArgs p;
    p.W = W; p.U = U; p.b = b;
    p.D = d.D; p.H = d.H; p.Dp = d.Dp; p.Hp = d.Hp; p.NP = d.NP; p.NPU = d.NPU; p.n_cells = n_sig;
    p.Bp = packed;
    p.bp = reinterpret_cast<float *>(static_cast<char *>(packed) + round_up(packed_w_bytes(d) * n_sig, 256));
    if (dtype == JITDB_F32) pack_weights_kernel<float><<<grid, kThreads, 0, st>>>(p);
    else pack_weights_kernel<bf16_t><<<grid, kThreads, 0, st>>>(p);
    JITDB_LAUNCH_CHECK();
    return JITDB_OK;
}

extern "C" int jitdb_treelstm_forward_packed(const void *x, const void *packed, int32_t D, int32_t H,
                                             jitdb_dtype dtype, const jitdb_schedule_t *s,
                                             const jitdb_slots_t *slots, void *h_out, float *c_out,
                                             void *workspace, size_t workspace_bytes, void *hip_stream) {
    if (!packed) return JITDB_E_NULL;
    return forward_entry(x, nullptr, nullptr, nullptr, D, H, dtype, s, slots, h_out, c_out, nullptr, nullptr, false,
                         workspace, workspace_bytes, hip_stream, packed);
}

extern "C" int jitdb_treelstm_forward(const void *x, const void *W, const void *U, const float *b,
                                      int32_t D, int32_t H, jitdb_dtype dtype,
                                      const jitdb_schedule_t *s, void *h_out, float *c_out,
                                      void *workspace, size_t workspace_bytes, void *hip_stream) {
    return forward_entry(x, W, U, b, D, H, dtype, s, nullptr, h_out, c_out, nullptr, nullptr, false,
                         workspace, workspace_bytes, hip_stream);
}

extern "C" size_t jitdb_treelstm_typed_workspace_bytes(int64_t n_nodes, int64_t n_edges, int32_t D, int32_t H,
                                                       jitdb_dtype dtype, int32_t n_sig) {
    if (!dims_ok(n_nodes, n_edges, D, H, (int)dtype) || n_sig < 1 || n_sig > JITDB_MAX_SIGNATURES) return 0;
    const Dims d = make_dims(D, H, dtype);
    return carve_forward_ws(n_nodes, n_edges, d, nullptr, n_sig).bytes;
}

extern "C" int jitdb_treelstm_forward_typed(const void *x, const void *W, const void *U, const float *b,
                                            int32_t D, int32_t H, jitdb_dtype dtype,
                                            const jitdb_schedule_t *s, const jitdb_slots_t *slots,
                                            void *h_out, float *c_out,
                                            void *workspace, size_t workspace_bytes, void *hip_stream) {
    if (!slots) return JITDB_E_NULL;
    return forward_entry(x, W, U, b, D, H, dtype, s, slots, h_out, c_out, nullptr, nullptr, false,
                         workspace, workspace_bytes, hip_stream);
}

extern "C" size_t jitdb_treelstm_cells_workspace_bytes(int64_t n_nodes, int64_t n_edges, int32_t D, int32_t H,
                                                       jitdb_dtype dtype, const jitdb_cell_t *cells, int32_t n_sig) {
    if (!cells || !dims_ok(n_nodes, n_edges, D, H, (int)dtype) || n_sig < 1 || n_sig > JITDB_MAX_SIGNATURES) return 0;
    for (int t = 0; t < n_sig; ++t)
        if (cells[t].kind == JITDB_CELL_NARY && (cells[t].arity < 1 || cells[t].arity > JITDB_MAX_NARY)) return 0;
    const Dims d = make_dims(D, H, dtype);
    return carve_forward_ws(n_nodes, n_edges, d, nullptr, n_sig, cells).bytes;
}

extern "C" int jitdb_treelstm_forward_cells(const void *x, const jitdb_cell_t *cells, int32_t n_sig,
                                            int32_t D, int32_t H, jitdb_dtype dtype,
                                            const jitdb_schedule_t *s, const jitdb_slots_t *slots,
                                            void *h_out, float *c_out,
                                            void *workspace, size_t workspace_bytes, void *hip_stream) {
    if (!slots || !cells) return JITDB_E_NULL;
    if (n_sig != slots->n_sig) return JITDB_E_BADARG;
    const int rc = forward_entry(x, nullptr, nullptr, nullptr, D, H, dtype, s, slots, h_out, c_out, nullptr, nullptr,
                                 false, workspace, workspace_bytes, hip_stream, nullptr, cells);
    if (rc != JITDB_OK || !s || s->n_nodes == 0) return rc;
    bool any_nary = false;
    for (int t = 0; t < n_sig; ++t) any_nary = any_nary || cells[t].kind == JITDB_CELL_NARY;
    if (!any_nary) return JITDB_OK;
    // a node with more children than its cell has positions: reported after the work has run
    const Dims d = make_dims(D, H, dtype);
    const ForwardWs w = carve_forward_ws(s->n_nodes, s->n_edges, d, workspace, n_sig, cells);
    int flag = 0;
    hipStream_t st = (hipStream_t)hip_stream;
    JITDB_HIP_CHECK(hipMemcpyAsync(&flag, w.nary_err, sizeof(int), hipMemcpyDeviceToHost, st));
    JITDB_HIP_CHECK(hipStreamSynchronize(st));
    return flag ? JITDB_E_ARITY : JITDB_OK;
}

extern "C" int jitdb_treelstm_forward_train(const void *x, const void *W, const void *U, const float *b,
                                            int32_t D, int32_t H, jitdb_dtype dtype,
                                            const jitdb_schedule_t *s, void *h_out, float *c_out,
                                            void *gates_out, void *fgate_out,
                                            void *workspace, size_t workspace_bytes, void *hip_stream) {
    return forward_entry(x, W, U, b, D, H, dtype, s, nullptr, h_out, c_out, gates_out, fgate_out, true,
                         workspace, workspace_bytes, hip_stream);
}

// ---- the forward for callers that cannot allocate ----------------------------------------
// Code under HIP graph capture, tight serving loops and harnesses that forbid hipMalloc have no
// workspace to hand over.  For them the workspace is this array, which every GPU the library
// runs on holds from the moment the code object is loaded until the process ends.  In host code
// the array's name is only a handle: the device address comes from hipGetSymbolAddress, once per
// device, and that pointer is what the kernels get.
static __device__ __align__(256) unsigned char scratch[JITDB_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
void *g_scratch_ptr[kMaxDevices] = {};
std::mutex g_scratch_lock;

int static_scratch_of_current_device(void **out) {
    int dev = -1;
    JITDB_HIP_CHECK(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return JITDB_E_BADARG;
    std::lock_guard<std::mutex> g(g_scratch_lock);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        JITDB_HIP_CHECK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));    // this device's copy of the array
        if (!p) return JITDB_E_HIP;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return JITDB_OK;
}
}  // namespace

extern "C" int jitdb_treelstm_forward_static(const void *x, const void *W, const void *U, const float *b,
                                             int32_t D, int32_t H, jitdb_dtype dtype,
                                             const jitdb_schedule_t *s, void *h_out, float *c_out,
                                             void *hip_stream) {
    if (!s) return JITDB_E_NULL;
    if (!dims_ok(s->n_nodes, s->n_edges, D, H, (int)dtype)) return JITDB_E_BADARG;
    if (s->n_nodes == 0) return JITDB_OK;
    const size_t need = carve_forward_ws(s->n_nodes, s->n_edges, make_dims(D, H, dtype), nullptr, 1, nullptr, false).bytes;
    if (need > (size_t)JITDB_STATIC_SCRATCH_BYTES) return JITDB_E_WORKSPACE;
    drop_stale_hip_error();
    void *ws = nullptr;
    JITDB_ABI_TRY
    const int rc = static_scratch_of_current_device(&ws);
    if (rc != JITDB_OK) return rc;
    JITDB_ABI_CATCH
    // Nothing in the workspace has to start at zero: every region is written in full by this call
    // before anything reads it (packed weights, row records, the stacked level, P, padded copies).
    return forward_entry(x, W, U, b, D, H, dtype, s, nullptr, h_out, c_out, nullptr, nullptr, false,
                         ws, (size_t)JITDB_STATIC_SCRATCH_BYTES, hip_stream);
}
