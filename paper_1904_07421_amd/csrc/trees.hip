// The forward of a forest of small trees in TWO launches: every node's x part, then whole trees, all levels, in a block.
//
// Level by level, a forest of a few thousand nodes costs two launches per level and the latencies inside them
// (gather, K loop, cell update, projection): 25 - 30 us a level whatever the level holds.  Two things do not depend on
// the levels: W x + b is the same for every node whenever it is evaluated, and a block that owns whole trees needs
// nothing from other blocks, so its levels may follow one another behind block barriers.
//
//   tree_x_kernel    Z = W x + b for all nodes, spread evenly over the chip; leaves finish their cells right there, the
//                    other nodes leave Z [node][i | o | u | f] in fp32 (narrow bf16 rows: tree_x_lds_kernel)
//   trees_resident_kernel, trees_kernel
//                    block b takes the trees from the first cut at or after id b G to the first at or after (b + 1) G (a
//                    cut is a place between ids that no edge crosses; jitdb_schedule_t::tree_window says that they are
//                    close together).  Rows are the block's nodes in (height, id) order, in groups of 16 to 64:
//                      gather    for a row of level l: sum of the children's h (operand, LDS) and of their f c (fp32, LDS)
//                      (barrier) i, o, u = Z + U hs;  c = i u + sum f c,  h = o tanh c; h goes out and into LDS
//                      (barrier) P = U_f h from LDS; f = sigmoid(Z_f of the PARENT + P), f c goes out for the parent
//                    A child's forget gate needs nothing of its parent but Z_f, which is there already: no P row and no
//                    c row is fetched by a parent, child sums are the only gather, in 16-byte pieces with several
//                    children in flight.
//                      (barrier, at the end of a level)
//
// A wave multiplies the gates of 16 hidden units (v_mfma_f32_16x16x32_bf16 / 16x16x4_f32), so the cell update finds a unit's
// gates in one lane.  A comes from LDS.  Where the weights of a wave's units fit its registers (bf16, and fp32 up to 128 units, or
// 160 with the block's h and f c in LDS) trees_resident_kernel loads them once: what bounds it are the barriers and memory
// latencies of each level.  Otherwise (fp32) trees_kernel reads them from L2 every level, in 1 KB pieces (64-byte slabs of 16
// packed rows), kTreeAhead slabs ahead, and is bound by that and by the fp32 matrix rate on 16-row tiles; its wide cells
// take up to 16 waves and run one block a compute unit.
#include "level_common.h"

namespace jitdb {
namespace {

constexpr int kTreeMaxWaves = 16;          // at most 128 registers each: four waves per SIMD
constexpr int kTreeRows = 32;              // most rows of a group (16 where LDS holds no more)
// weight slabs in flight per wave: the fewer MFMAs a slab feeds, the more
template <int NRT, int NG> constexpr int kTreeAhead = NRT * NG <= 1 ? 6 : NRT <= 1 ? 4 : NG == 1 ? 4 : 2;
constexpr uint16_t kNoLocal = 0xFFFF;

// The same weights times at most FOUR rows: 4 x 4 blocks, sixteen of them in one MFMA, block lane / 4 taking the columns and
// the quarter of the slab's K that this lane's 16 bytes hold.  A quarter of the 16-row form's time for fp32, and each lane
// ends up with one row of its column (quarter_sum).  a: row lane & 3, piece lane >> 4.
typedef short short4v __attribute__((ext_vector_type(4)));
template <typename T>
__device__ __forceinline__ void mfma4(const u32x4 &a, const u32x4 &b, floatx4 &acc) {
    if constexpr (sizeof(T) == 2) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const u32x2 aj = {a[2 * j], a[2 * j + 1]}, bj = {b[2 * j], b[2 * j + 1]};
            acc = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(__builtin_bit_cast(short4v, aj), __builtin_bit_cast(short4v, bj), acc, 0, 0, 0);
        }
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            acc = __builtin_amdgcn_mfma_f32_4x4x1f32(__uint_as_float(a[j]), __uint_as_float(b[j]), acc, 0, 0, 0);
    }
}

// acc[v] of the four lanes of a column (n, n + 16, n + 32, n + 48) hold row v's sums over their quarters of K; lane n + 16 q
// gets the total of row q.
__device__ __forceinline__ float quarter_sum(const floatx4 &acc, int lane) {
    const bool b1 = lane & 32, b0 = lane & 16;
    float k0 = (b1 ? acc[2] : acc[0]) + __shfl_xor(b1 ? acc[0] : acc[2], 32, 64);
    float k1 = (b1 ? acc[3] : acc[1]) + __shfl_xor(b1 ? acc[1] : acc[3], 32, 64);
    return (b0 ? k1 : k0) + __shfl_xor(b0 ? k0 : k1, 16, 64);
}

// acc[rt][g] += A rows (16 rt ..; NRT == 0: at most four rows) x packed rows of gate g, over n_slabs slabs of 64 bytes of K.
// a_lane: this lane's bytes of slab 0 (row lane & 15 or lane & 3, piece lane >> 4) in LDS or memory; b_lane likewise in the
// packed weights, the gates 2048 bytes apart.  A_AHEAD: A comes from memory and is requested with the weights.
template <typename T, int NRT, int NG, bool A_AHEAD = false, int AHEAD = kTreeAhead<NRT, NG>, typename ALoad>
__device__ __forceinline__ void tree_gemm(floatx4 (&acc)[NRT ? NRT : 1][NG], ALoad &&load_a, const char *b_lane, int64_t b_slab, int n_slabs) {
    constexpr int NA = NRT ? NRT : 1;
    u32x4 fb[AHEAD][NG], fr[A_AHEAD ? AHEAD : 1][NA];
    auto request = [&](int s, int slot) __attribute__((always_inline)) {
        if constexpr (A_AHEAD) {
#pragma unroll
            for (int rt = 0; rt < NA; ++rt) fr[slot][rt] = load_a(rt, s < n_slabs ? s : n_slabs - 1);
        }
        const char *p = b_lane + (int64_t)(s < n_slabs ? s : n_slabs - 1) * b_slab;
#pragma unroll
        for (int g = 0; g < NG; ++g) fb[slot][g] = *reinterpret_cast<const u32x4 *>(p + g * 2048);
    };
    auto multiply = [&](int s, int slot) __attribute__((always_inline)) {
        u32x4 fa[NA];
#pragma unroll
        for (int rt = 0; rt < NA; ++rt) fa[rt] = A_AHEAD ? fr[A_AHEAD ? slot : 0][rt] : load_a(rt, s);
#pragma unroll
        for (int rt = 0; rt < NA; ++rt)
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                if constexpr (NRT == 0) mfma4<T>(fa[rt], fb[slot][g], acc[rt][g]);
                else mfma16<T>(fa[rt], fb[slot][g], acc[rt][g]);
            }
    };
#pragma unroll
    for (int p = 0; p < AHEAD; ++p) request(p, p);
    const int full = n_slabs / AHEAD;
    for (int c = 0; c < full; ++c) {
#pragma unroll
        for (int p = 0; p < AHEAD; ++p) {
            multiply(c * AHEAD + p, p);
            request((c + 1) * AHEAD + p, p);
        }
    }
#pragma unroll
    for (int p = 0; p < AHEAD - 1; ++p)
        if (full * AHEAD + p < n_slabs) multiply(full * AHEAD + p, p);
}

template <typename T>
__device__ __forceinline__ void add_h_piece(float (&s)[Traits<T>::VEC], const u32x4 &v) {
    if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int j = 0; j < 4; ++j) s[j] += __uint_as_float(v[j]);
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            s[2 * j] += __uint_as_float(v[j] << 16);
            s[2 * j + 1] += __uint_as_float(v[j] & 0xFFFF0000u);
        }
    }
}

// The lane number, worked out anew: what is derived from it then belongs to one group of rows.  (Left to itself the
// compiler computes every variant's offsets ahead of the level loop and keeps them in registers it does not have.)
__device__ __forceinline__ int fresh_lane(int lane) {
    asm volatile("" : "+v"(lane));
    return lane;
}

__device__ __forceinline__ const char *tree_weights(const TreesArgs &a, int lane, int ut, int slab, int gate) {
    const int row = (ut >> 1) * kGateTile + gate * kUnit + (ut & 1) * 16 + (lane & 15);
    return static_cast<const char *>(a.Bp) + ((int64_t)slab * a.NPU + row) * 64 + (lane >> 4) * 16;
}

// h and c of one unit of one node, to every place that wants them.
template <typename T>
__device__ __forceinline__ void store_unit(const TreesArgs &a, int64_t node, int unit, float c, T hv) {
    if (unit < a.H) {
        a.c_out[node * a.H + unit] = c;
        static_cast<T *>(a.h_out)[node * a.H + unit] = hv;
        if (a.cs) a.cs[node * a.Hq + unit] = c;         // (only where chain levels follow)
    }
    if (a.hs != a.h_out) {
        T *hs = static_cast<T *>(a.hs) + node * a.Hp;
        hs[unit] = hv;
        if (unit >= a.Hz - 16)                                // the pad columns past the last unit tile
            for (int p = unit + 16; p < a.Hp; p += 16) hs[p] = T(0);
    }
}

template <typename T>
__device__ __forceinline__ void save_gates(const TreesArgs &a, int64_t node, int unit, float gi, float go, float gu) {
    T *g = static_cast<T *>(a.gates) + node * 3 * a.H + unit;
    g[0] = from_f32<T>(gi);
    g[a.H] = from_f32<T>(go);
    g[2 * a.H] = from_f32<T>(gu);
}

// All of the block's LDS writes are visible after it; stores to memory are not waited for (__syncthreads would).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// ---- the x part ----------------------------------------------------------------------------
// A wave keeps the weights of its 16 units' four gates in registers (NS slabs: 16 NS registers, which is what decides how
// many waves share a SIMD: two up to ten slabs, one beyond) and multiplies one tile of 16 nodes after another.  Tiles run in
// the schedule's order: first the leaves', then the others', so that a tile's nodes all go the same way.  Blocks of neighbouring
// units run on one XCD: they read the same rows and fill the same lines.
constexpr int kXWavesPerSimd(int ns) { return ns <= 10 ? 2 : 1; }
// Its instances: D up to 128, 224, 320, 512 and 640 in bf16, half of that in fp32.  Ten slabs are the most with which two waves
// share a SIMD, twenty the most that 512 registers hold; the others bound the slabs multiplied as zeros to five.
constexpr int kXSlabs[] = {4, 7, 10, 16, 20};
constexpr int slabs_below(int ns) {                // the instance before: slabs up to there lie inside D whenever ns is chosen
    int below = 0;
    for (int k : kXSlabs)
        if (k < ns) below = k;
    return below;
}

struct XTiles {
    const int32_t *perm;
    int n_leaves, n, leaf_tiles, n_tiles;
    __device__ __forceinline__ explicit XTiles(const TreesArgs &a)
        : perm(a.perm), n_leaves(a.n_leaves), n(a.n), leaf_tiles((a.n_leaves + 15) >> 4), n_tiles(leaf_tiles + ((a.n - a.n_leaves + 15) >> 4)) {}
    __device__ __forceinline__ int node(int tile, int i) const {      // (past the end: the last one again)
        const bool leaf = tile < leaf_tiles;
        const int p = (leaf ? 0 : n_leaves - leaf_tiles * 16) + tile * 16 + i, last = (leaf ? n_leaves : n) - 1;
        return perm[p < last ? p : last];
    }
};

template <int NS>
__device__ __forceinline__ void load_x_weights(const TreesArgs &a, int lane, int ut, u32x4 (&fb)[NS][4]) {
    const char *w = tree_weights(a, lane, ut, 0, 0);
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            fb[s][g] = *reinterpret_cast<const u32x4 *>(w + (int64_t)(s < a.sx_packed ? s : 0) * a.NPU * 64 + g * 2048);
    // slabs past the packed x part meet zeros, but 0 times an infinite weight would be NaN
#pragma unroll
    for (int s = slabs_below(NS); s < NS; ++s)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            if (s >= a.sx_packed) fb[s][g] = u32x4{0, 0, 0, 0};
}

// The biases of a wave's units, [gate][unit], in LDS: a load from memory behind the next rows' requests and the last tile's
// stores would wait for all of them.
__device__ __forceinline__ void keep_x_bias(const TreesArgs &a, int lane, int ut, float *bias) {
    bias[lane] = a.bp[(ut >> 1) * kGateTile + (lane >> 4) * kUnit + (ut & 1) * 16 + (lane & 15)];
}

// Leaves finish, the others leave Z.  node_of(i): node of row i of the tile.
template <typename T, bool SAVE, typename NodeOf>
__device__ __forceinline__ void finish_x_tile(const TreesArgs &a, int lane, int ut, bool leaf, const floatx4 (&acc)[4], const float *bias, NodeOf &&node_of) {
    lane = fresh_lane(lane);                     // (nothing derived from it stays in registers meanwhile)
    const int unit = ut * 16 + (lane & 15);
    const float *b = bias + (lane & 15), bi = b[0], bo = b[16], bu = b[32], bf = b[48];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        __builtin_amdgcn_sched_barrier(0);
        const float zi = acc[0][v] + bi, zo = acc[1][v] + bo, zu = acc[2][v] + bu;
        const int64_t node = node_of((lane >> 4) * 4 + v);
        if (leaf) {
            const float gi = sigmoid_t<T>(zi), go = sigmoid_t<T>(zo), gu = tanh_t<T>(zu);
            const float c = gi * gu;
            store_unit<T>(a, node, unit, c, unit < a.H ? from_f32<T>(go * tanh_t<T>(c)) : T(0));
            if constexpr (SAVE) {
                if (unit < a.H) save_gates<T>(a, node, unit, gi, go, gu);
            }
        } else {
            float *z = a.Z + node * 4 * a.Hz + unit;
            z[0] = zi; z[a.Hz] = zo; z[2 * a.Hz] = zu; z[3 * a.Hz] = acc[3][v] + bf;
        }
    }
}

// fp32, which the matrix rate bounds, bf16 from ten slabs on, and below as x_through_lds says: x rows come straight from memory in
// operand layout, the next tile's slab requested as soon as this one's is used, its node ids a tile earlier.  No LDS, no barrier:
// waves of a block take different units of the same nodes, which meet in L1.  (No load may be waited for behind a tile's stores,
// which it would drain first: 278 k nodes, D 300, H 256, fp32 1110 us with the biases loaded there, 1040 now.)
// Leaves have no forget gate.  Its products are left out of their tiles by a branch between the other MFMAs, except in the wide
// bf16 instances: with the accumulators in accumulation registers the compiler once read an MFMA's result there two instructions
// behind it where the branch is taken, eight too few, and every tile of leaves came out wrong.  (The build looks for such reads.)
template <typename T, int NS> constexpr bool kLeavesSkip = sizeof(T) == 4 || NS <= 10;
template <typename T, bool SAVE, int NS>
__global__ void __launch_bounds__(256, kXWavesPerSimd(NS))
tree_x_kernel(const TreesArgs a) {
    constexpr int VEC = Traits<T>::VEC;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int gw = ((blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3)) * 4 + wave;
    const int ut = gw % a.n_ut, chunk = gw / a.n_ut;
    if (chunk >= a.x_chunks) return;
    const int hf = lane >> 4, n = lane & 15;
    __shared__ float bias[4][64];
    keep_x_bias(a, lane, ut, bias[wave]);
    u32x4 fb[NS][4];
    load_x_weights<NS>(a, lane, ut, fb);
    const T *x = static_cast<const T *>(a.x);
    const XTiles tiles(a);
    auto row_of = [&](int node) __attribute__((always_inline)) { return x + (int64_t)node * a.D + hf * VEC; };
    // slab s of a row: whole 16 bytes where all four pieces lie inside D; the slab that straddles D, and those past it,
    // piece by piece
    auto load_slab = [&](const T *row, int s) __attribute__((always_inline)) {
        u32x4 v;
        if (s < slabs_below(NS) || (s + 1) * 4 * VEC <= a.D) __builtin_memcpy(&v, row + s * 4 * VEC, 16);
        else v = load_x_piece<T>(row - hf * VEC, (s * 4 + hf) * VEC, a.D);
        return v;
    };
    // (where gates are saved, ten bf16 slabs leave no registers for the last two across the cell update: those come at the tile's start)
    constexpr int PF = NS == 10 && SAVE && sizeof(T) == 2 ? 8 : NS;
    u32x4 fa[NS];
    auto nodes_of = [&](int tile) __attribute__((always_inline)) { return tiles.node(tile < tiles.n_tiles ? tile : chunk, n); };
    int id = nodes_of(chunk), id_next = nodes_of(chunk + a.x_chunks);
    const T *row = row_of(id);
#pragma unroll
    for (int s = 0; s < PF; ++s) fa[s] = load_slab(row, s);
    for (int tile = chunk; tile < tiles.n_tiles; tile += a.x_chunks) {
        const bool leaf = tile < tiles.leaf_tiles;
        const int id_after = nodes_of(tile + 2 * a.x_chunks);
        floatx4 acc[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) acc[g] = floatx4{0, 0, 0, 0};
#pragma unroll
        for (int s = PF; s < NS; ++s) fa[s] = load_slab(row, s);
        row = row_of(id_next);
#pragma unroll
        for (int s = 0; s < NS; ++s) {
#pragma unroll
            for (int g = 0; g < 3; ++g) mfma16<T>(fa[s], fb[s][g], acc[g]);
            if (!kLeavesSkip<T, NS> || !leaf) mfma16<T>(fa[s], fb[s][3], acc[3]);
            if (s < PF) fa[s] = load_slab(row, s);
        }
        finish_x_tile<T, SAVE>(a, lane, ut, leaf, acc, bias[wave], [&](int i) { return __shfl(id, i, 64); });
        id = id_next;
        id_next = id_after;
    }
}

// Elements [k0, k0 + 8) of a row of D >= 8 from one 16-byte load inside it, zero past D.
__device__ __forceinline__ u32x4 load_x_piece_inside(const bf16_t *row, int k0, int D) {
    u32x4 v = {0, 0, 0, 0};
    if (k0 >= D) return v;
    __builtin_memcpy(&v, row + (k0 + 8 <= D ? k0 : D - 8), 16);
    const int bits = ((8 - D) & 7) * 16;                      // what the piece that straddles D has to come down by
    if (k0 + 8 > D) {
        const uint64_t lo = v[0] | (uint64_t)v[1] << 32, hi = v[2] | (uint64_t)v[3] << 32;
        const uint64_t l = bits >= 64 ? hi >> (bits - 64) : lo >> bits | hi << (64 - bits), h = bits >= 64 ? 0 : hi >> bits;
        v = u32x4{(uint32_t)l, (uint32_t)(l >> 32), (uint32_t)h, (uint32_t)(h >> 32)};
    }
    return v;
}

// bf16 up to seven slabs, as x_through_lds says: a wave's own loads in operand layout touch 64 lines for 1 KB, more where rows
// start on odd elements, and every unit tile's wave repeats them.  A block of four unit tiles fetches its rows once, 16 consecutive
// bytes a lane, and multiplies from LDS (two buffers, one barrier a group of 16 x_rt rows, the next group's rows in flight
// meanwhile).  21 k nodes, D 203, H 99: 31.7 -> 25.2 us.  It hides one round trip of a group's rows, so with ten slabs, whose
// registers hold 16 rows of products and no more, it is slower: 106 k nodes, D 300, H 150 111 -> 162.
constexpr int kXLdsWaves = 4, kXLdsSlabs = 7, kXLdsRows = 32;
constexpr int kXLdsAlways = 4, kXLdsManyNodes = 160000;        // slabs, nodes: x_through_lds
template <bool SAVE, int NS>
__global__ void __launch_bounds__(kXLdsWaves * 64, kXWavesPerSimd(NS))
tree_x_lds_kernel(const TreesArgs a) {
    using T = bf16_t;
    constexpr int NT = kXLdsWaves * 64, ROWS = kXLdsRows, PX = NS * 4, PITCH = NS * 64 + 16, E = (ROWS * PX + NT - 1) / NT;
    __shared__ __attribute__((aligned(16))) char xs[2][ROWS * PITCH];
    __shared__ int ids[4][ROWS];
    __shared__ float bias[kXLdsWaves][64];
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int block = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    const int n_ug = (a.n_ut + kXLdsWaves - 1) / kXLdsWaves;
    const int chunk = block / n_ug, first_ut = block % n_ug * kXLdsWaves;
    if (chunk >= a.x_chunks) return;
    const bool mine = first_ut + wave < a.n_ut;               // (the others only fetch)
    const int ut = mine ? first_ut + wave : first_ut;
    const XTiles tiles(a);
    const int rows = 16 * a.x_rt, n_groups = (tiles.n_tiles + a.x_rt - 1) / a.x_rt;
    auto id_of = [&](int group) __attribute__((always_inline)) {          // of row t (past the end: some row again)
        const int tile = (group < n_groups ? group : chunk) * a.x_rt + (t >> 4);
        return tiles.node(tile < tiles.n_tiles ? tile : tiles.n_tiles - 1, t & 15);
    };
    if (t < rows) {
        ids[0][t] = id_of(chunk);
        ids[1][t] = id_of(chunk + a.x_chunks);
        ids[2][t] = id_of(chunk + 2 * a.x_chunks);
    }
    keep_x_bias(a, lane, ut, bias[wave]);
    u32x4 fb[NS][4];
    load_x_weights<NS>(a, lane, ut, fb);
    lds_barrier();
    u32x4 xr[E];
    auto request = [&](const int *id) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int q = t + e * NT;
            xr[e] = u32x4{0, 0, 0, 0};
            if (q >= rows * PX) continue;
            const T *row = static_cast<const T *>(a.x) + (int64_t)id[q / PX] * a.D;
            xr[e] = a.D >= 8 ? load_x_piece_inside(row, q % PX * 8, a.D) : load_x_piece<T>(row, q % PX * 8, a.D);
        }
    };
    auto write = [&](char *buf) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int q = t + e * NT;
            if (q < rows * PX) *reinterpret_cast<u32x4 *>(buf + q / PX * PITCH + q % PX * 16) = xr[e];
        }
    };
    request(ids[0]);
    write(xs[0]);
    request(ids[1]);
    lds_barrier();
    int cur = 0, k = 0;
    for (int group = chunk; group < n_groups; group += a.x_chunks, cur ^= 1, k = (k + 1) & 3) {
        int id_after = 0;
        if (t < rows) id_after = id_of(group + 3 * a.x_chunks);
        floatx4 acc[ROWS / 16][4];
#pragma unroll
        for (int j = 0; j < ROWS / 16; ++j) {
#pragma unroll
            for (int g = 0; g < 4; ++g) acc[j][g] = floatx4{0, 0, 0, 0};
            const int tile = group * a.x_rt + j;
            if (!mine || j >= a.x_rt) continue;
            const bool leaf = tile < tiles.leaf_tiles;
            const char *a_lane = xs[cur] + (j * 16 + (lane & 15)) * PITCH + (lane >> 4) * 16;
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const u32x4 fa = *reinterpret_cast<const u32x4 *>(a_lane + s * 64);
#pragma unroll
                for (int g = 0; g < 3; ++g) mfma16<T>(fa, fb[s][g], acc[j][g]);
                if (!leaf) mfma16<T>(fa, fb[s][3], acc[j][3]);
            }
        }
        // The next group's rows are here and the ones after them asked for before this group's stores: the wait for loads waits
        // for every older store, and those then have a group's time too.
        write(xs[cur ^ 1]);
        if (t < rows) ids[(k + 3) & 3][t] = id_after;
        __builtin_amdgcn_sched_barrier(0);
        request(ids[(k + 2) & 3]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < ROWS / 16; ++j) {
            const int tile = group * a.x_rt + j;
            if (!mine || j >= a.x_rt || tile >= tiles.n_tiles) continue;
            finish_x_tile<T, SAVE>(a, lane, ut, tile < tiles.leaf_tiles, acc[j], bias[wave], [&](int i) { return ids[k][j * 16 + i]; });
        }
        lds_barrier();
    }
}

// ---- the levels ------------------------------------------------------------------------------
// The block's view of its trees.
struct TreeBlock {
    char *A, *Ht;                          // LDS: child sums and h of the group's rows, [group_rows][pitch_h]
    float *Fs;                             // LDS: sums of the children's f c, [group_rows][Hz]
    uint16_t *order, *cstart, *kids, *par;         // local ids by row; child list starts, children, parents by local id
    int lo, own;
    int lane, wave, n_waves;
};

// The arrays of a block's view behind `at`: 4 cap + 8 entries.
__device__ __forceinline__ void place_view(const TreesArgs &a, TreeBlock &b, char *at) {
    b.order = reinterpret_cast<uint16_t *>(at);
    b.cstart = b.order + a.cap;
    b.kids = b.cstart + a.cap + 2;
    b.par = b.kids + a.cap;
    b.lane = threadIdx.x & 63;
    b.wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    b.n_waves = blockDim.x >> 6;
}

// Child sums of rows [r0, r_end) into A and Fs.  A wave takes 64 of a row's 16-byte pieces at a time, of ROWS rows side by side,
// KIDS children of each in flight.
template <typename T, int ROWS, int KIDS>
__device__ __forceinline__ void gather_sums(const TreesArgs &a, const TreeBlock &b, int r0, int r_end, int ph) {
    constexpr int VEC = Traits<T>::VEC;
    const int pf = a.Hz / 4;                     // 16-byte pieces of an f c row (ph: of an h row)
    const int per_row = (ph + pf + 63) >> 6, n_tasks = (r_end - r0) * per_row;
    for (int q0 = b.wave; q0 < n_tasks; q0 += ROWS * b.n_waves) {
        const char *col[ROWS];
        u32x4 w[ROWS][KIDS];
        int c0[ROWS], c1[ROWS];
        auto piece = [&](int q, int &rr, int &k) __attribute__((always_inline)) {
            rr = q / per_row;
            k = (q - rr * per_row) * 64 + fresh_lane(b.lane);
            return k < ph + pf;
        };
        const int pitch_f = a.Hz * 4, pitch_h = a.Hp * (int)sizeof(T);
#pragma unroll
        for (int j = 0; j < ROWS; ++j) {
            const int q = q0 + j * b.n_waves;
            c0[j] = c1[j] = 0;
            if (q >= n_tasks) continue;
            int rr, k;
            if (!piece(q, rr, k)) continue;
            const int i = __builtin_amdgcn_readfirstlane((int)b.order[r0 + rr]);
            c0[j] = b.cstart[i];
            c1[j] = b.cstart[i + 1];
            const bool is_h = k < ph;
            if (is_h && k * VEC >= a.Hz) c1[j] = c0[j];      // the slab's pieces past the last unit tile are zero
            // an h row or an f c row: the same loads, summed as what they are
            col[j] = is_h ? static_cast<const char *>(a.hs) + (int64_t)b.lo * pitch_h + k * 16
                          : reinterpret_cast<const char *>(a.FC) + (int64_t)b.lo * pitch_f + (k - ph) * 16;
#pragma unroll
            for (int e = 0; e < KIDS; ++e) {
                w[j][e] = u32x4{0, 0, 0, 0};
                if (c0[j] + e < c1[j]) w[j][e] = *reinterpret_cast<const u32x4 *>(col[j] + (int64_t)b.kids[c0[j] + e] * (is_h ? pitch_h : pitch_f));
            }
        }
#pragma unroll
        for (int j = 0; j < ROWS; ++j) {
            const int q = q0 + j * b.n_waves;
            if (q >= n_tasks) continue;
            int rr, k;
            if (!piece(q, rr, k)) continue;
            const bool is_h = k < ph;
            float s[VEC];
#pragma unroll
            for (int e = 0; e < VEC; ++e) s[e] = 0.0f;
            for (int c = c0[j]; c < c1[j]; c += KIDS) {      // ascending ids
                if (c > c0[j]) {
#pragma unroll
                    for (int e = 0; e < KIDS; ++e) {
                        w[j][e] = u32x4{0, 0, 0, 0};
                        if (c + e < c1[j]) w[j][e] = *reinterpret_cast<const u32x4 *>(col[j] + (int64_t)b.kids[c + e] * (is_h ? pitch_h : pitch_f));
                    }
                }
#pragma unroll
                for (int e = 0; e < KIDS; ++e) {
                    if (c + e >= c1[j]) break;
                    if (sizeof(T) == 4 || is_h) {
                        add_h_piece<T>(s, w[j][e]);
                    } else {
#pragma unroll
                        for (int u = 0; u < 4; ++u) s[u] += __uint_as_float(w[j][e][u]);
                    }
                }
            }
            if (is_h) {
                T e[VEC];
#pragma unroll
                for (int u = 0; u < VEC; ++u) e[u] = from_f32<T>(s[u]);
                u32x4 v;
                __builtin_memcpy(&v, e, 16);
                *reinterpret_cast<u32x4 *>(b.A + rr * a.pitch_h + k * 16) = v;
            } else {
                *reinterpret_cast<float4 *>(b.Fs + rr * a.Hz + (k - ph) * 4) = make_float4(s[0], s[1], s[2], s[3]);
            }
        }
    }
}

// The cells of rows [r0, r_end): at most 16 NRT, NRT == 0: at most four, one per lane quarter.
template <bool SAVE, int NRT>
__device__ __forceinline__ void level_group(const TreesArgs &a, const TreeBlock &b, int r0, int r_end) {
    constexpr int NA = NRT ? NRT : 1, NV = NRT ? 4 : 1;
    for (int ut = b.wave; ut < a.n_ut; ut += b.n_waves) {
        const int lane = fresh_lane(b.lane), hf = lane >> 4, n = lane & 15;
        const int unit = ut * 16 + n;
        floatx4 acc[NA][3];
        float z4[3];
#pragma unroll
        for (int rt = 0; rt < NA; ++rt)
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const int r = r0 + (NRT ? rt * 16 + hf * 4 + v : hf);
                const float *zp = a.Z + (int64_t)(b.lo + b.order[r < r_end ? r : r_end - 1]) * 4 * a.Hz + unit;
#pragma unroll
                for (int g = 0; g < 3; ++g) {
                    if constexpr (NRT) acc[rt][g][v] = zp[g * a.Hz];
                    else { z4[g] = zp[g * a.Hz]; acc[0][g] = floatx4{0, 0, 0, 0}; }
                }
            }
        const char *a_lane = b.A + (NRT ? n : lane & 3) * a.pitch_h + hf * 16;
        tree_gemm<float, NRT, 3>(acc, [&](int rt, int s) { return *reinterpret_cast<const u32x4 *>(a_lane + rt * 16 * a.pitch_h + s * 64); },
                             tree_weights(a, lane, ut, a.sx_packed, 0), (int64_t)a.NPU * 64, a.sh);
#pragma unroll
        for (int rt = 0; rt < NA; ++rt) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const int rr = NRT ? rt * 16 + hf * 4 + v : hf, r = r0 + rr;
                float z[3];
#pragma unroll
                for (int g = 0; g < 3; ++g) z[g] = NRT ? acc[rt][g][v] : z4[g] + quarter_sum(acc[0][g], lane);
                const float gi = sigmoid_t<float>(z[0]), go = sigmoid_t<float>(z[1]), gu = tanh_t<float>(z[2]);
                const float c = gi * gu + b.Fs[rr * a.Hz + unit];
                b.Fs[rr * a.Hz + unit] = c;          // for the forget gates' step
                const float hv = unit < a.H ? go * tanh_t<float>(c) : 0.0f;
                *reinterpret_cast<float *>(b.Ht + rr * a.pitch_h + unit * 4) = hv;
                if (r >= r_end) continue;
                const int64_t node = b.lo + b.order[r];
                store_unit<float>(a, node, unit, c, hv);
                if constexpr (SAVE) {
                    if (unit < a.H) save_gates<float>(a, node, unit, gi, go, gu);
                }
            }
        }
    }
}

// f c of rows [r0, r_end) from P = U_f h, f with the parent's Z_f.  LEAF: h and c come from memory (tree_x_kernel has
// finished the leaves' cells), else from LDS.
template <bool SAVE, int NRT, bool LEAF>
__device__ __forceinline__ void forget_tile(const TreesArgs &a, const TreeBlock &b, int ut, int r0, int r_end) {
    constexpr int NA = NRT ? NRT : 1, NV = NRT ? 4 : 1;
    const int lane = fresh_lane(b.lane), hf = lane >> 4, n = lane & 15;
    const int unit = ut * 16 + n, unit_ld = unit < a.H ? unit : 0;
    floatx4 acc[NA][1];
    float zf[NA][NV], c[NA][NV];             // on their way during the product
#pragma unroll
    for (int rt = 0; rt < NA; ++rt) {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int rr = NRT ? rt * 16 + hf * 4 + v : hf, r = r0 + rr < r_end ? r0 + rr : r_end - 1;
            const int i = b.order[r], p = b.par[i];
            zf[rt][v] = a.Z[((int64_t)(b.lo + (p != kNoLocal ? p : i)) * 4 + 3) * a.Hz + unit];
            c[rt][v] = LEAF ? a.c_out[(int64_t)(b.lo + i) * a.H + unit_ld] : b.Fs[rr * a.Hz + unit];
        }
        acc[rt][0] = floatx4{0, 0, 0, 0};
    }
    const char *w = tree_weights(a, lane, ut, a.sx_packed, 3);
    if constexpr (LEAF) {
        const char *row[NA];
#pragma unroll
        for (int rt = 0; rt < NA; ++rt) {
            const int r = r0 + (NRT ? rt * 16 + n : lane & 3);
            row[rt] = static_cast<const char *>(a.hs) + (int64_t)(b.lo + b.order[r < r_end ? r : r_end - 1]) * a.Hp * 4 + hf * 16;
        }
        tree_gemm<float, NRT, 1, true>(acc, [&](int rt, int s) { return *reinterpret_cast<const u32x4 *>(row[rt] + s * 64); }, w, (int64_t)a.NPU * 64, a.sh);
    } else {
        const char *a_lane = b.Ht + (NRT ? n : lane & 3) * a.pitch_h + hf * 16;
        tree_gemm<float, NRT, 1>(acc, [&](int rt, int s) { return *reinterpret_cast<const u32x4 *>(a_lane + rt * 16 * a.pitch_h + s * 64); }, w,
                             (int64_t)a.NPU * 64, a.sh);
    }
#pragma unroll
    for (int rt = 0; rt < NA; ++rt)
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int r = r0 + (NRT ? rt * 16 + hf * 4 + v : hf);
            const float pf = NRT ? acc[rt][0][v] : quarter_sum(acc[0][0], lane);
            if (r >= r_end) continue;
            const int i = b.order[r];
            if (b.par[i] == kNoLocal) continue;
            const float f = sigmoid_t<float>(pf + zf[rt][v]);
            a.FC[(int64_t)(b.lo + i) * a.Hz + unit] = unit < a.H ? f * c[rt][v] : 0.0f;
            if constexpr (SAVE) {
                if (unit < a.H) static_cast<float *>(a.fgate)[(int64_t)(b.lo + i) * a.H + unit] = f;
            }
        }
}

struct TreeMeta {                          // LDS of a block for the view of its trees
    int cut[2];
    int min[kTreeMaxLevels], cnt[kTreeMaxLevels], start[kTreeMaxLevels + 1];
};

// Which trees are this block's, and its rows: fills `b` and `m`; false if there are none.  A barrier still has to follow.
// `lds` is scratch in front of the arrays of `b` (its barriers wait for LDS alone: weights on their way to registers stay so).
__device__ __forceinline__ bool view_trees(const TreesArgs &a, char *lds, TreeBlock &b, TreeMeta &m) {
    const int t = threadIdx.x, nt = blockDim.x;
    // ---- where the block's trees begin and end: for both places, how many parent-child intervals cross every position
    //      from i0 - tw on (the first and the last child bound a node's interval: child lists ascend)
    const int tw = a.tree_window, span = 2 * tw + 1;
    int *cover = reinterpret_cast<int *>(lds);                 // [2][span + 1]
    for (int i = t; i < 2 * (span + 1); i += nt) cover[i] = 0;
    if (t < kTreeMaxLevels) { m.min[t] = INT32_MAX; m.cnt[t] = 0; }
    lds_barrier();
    for (int side = 0; side < 2; ++side) {
        const int64_t i0 = ((int64_t)blockIdx.x + side) * a.G;
        if (i0 == 0 || i0 >= a.n) continue;
        const int base = (int)i0 - tw;
        const int j1 = i0 + 2 * tw < a.n ? (int)i0 + 2 * tw : a.n;
        for (int j = (base > 0 ? base : 0) + t; j < j1; j += nt) {
            const int c0 = a.child_ptr[j], c1 = a.child_ptr[j + 1];
            if (c1 <= c0) continue;
            const int first = a.child_idx[c0], last = a.child_idx[c1 - 1];
            int p0 = min(j, first) + 1 - base, p1 = max(j, last) + 1 - base;
            p0 = p0 < 0 ? 0 : p0;
            p1 = p1 < 0 ? 0 : p1;
            if (p0 <= span) atomicAdd(&cover[side * (span + 1) + p0], 1);
            if (p1 <= span) atomicAdd(&cover[side * (span + 1) + p1], -1);
        }
    }
    lds_barrier();
    if (b.wave < 2) {
        const int64_t i0 = ((int64_t)blockIdx.x + b.wave) * a.G;
        int cut;
        if (i0 == 0 || i0 >= a.n) {
            cut = i0 == 0 ? 0 : a.n;
        } else {
            const int *cv = cover + b.wave * (span + 1);
            const int per = (span + 63) / 64;
            int sum = 0;
            for (int q = b.lane * per; q < (b.lane + 1) * per && q < span; ++q) sum += cv[q];
            int run = sum;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int v = __shfl_up(run, d, 64);
                if (b.lane >= d) run += v;
            }
            run -= sum;
            cut = INT32_MAX;
            for (int q = b.lane * per; q < (b.lane + 1) * per && q < span; ++q) {
                run += cv[q];
                if (run == 0 && q >= tw && cut == INT32_MAX) cut = (int)i0 - tw + q;
            }
#pragma unroll
            for (int d = 32; d > 0; d >>= 1) cut = min(cut, __shfl_xor(cut, d, 64));
            if (cut > a.n) cut = a.n;                          // (past the last node, or no cut: not a schedule of jitdb_schedule)
        }
        if (b.lane == 0) m.cut[b.wave] = cut;
    }
    lds_barrier();
    b.lo = m.cut[0];
    b.own = m.cut[1] - b.lo;
    if (b.own > a.cap) b.own = a.cap;
    if (b.own <= 0) return false;

    // ---- rows: a level's nodes of this block are consecutive positions of the schedule
    const int e0 = a.child_ptr[b.lo], n_edges = min(a.child_ptr[b.lo + b.own] - e0, b.own);
    for (int i = t; i < b.own; i += nt) {
        const int h = a.height[b.lo + i];
        if (h < kTreeMaxLevels) {
            atomicMin(&m.min[h], a.inv_perm[b.lo + i]);
            atomicAdd(&m.cnt[h], 1);
        }
        b.order[i] = 0;
        b.par[i] = kNoLocal;
    }
    for (int i = t; i <= b.own; i += nt) b.cstart[i] = (uint16_t)min(max(a.child_ptr[b.lo + i] - e0, 0), n_edges);
    for (int e = t; e < n_edges; e += nt) {
        const int k = a.child_idx[e0 + e] - b.lo;
        b.kids[e] = (uint16_t)(k >= 0 && k < b.own ? k : 0);
    }
    lds_barrier();
    if (b.wave == 0) {
        const int c = b.lane < kTreeMaxLevels ? m.cnt[b.lane] : 0;
        int inc = c;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int v = __shfl_up(inc, d, 64);
            if (b.lane >= d) inc += v;
        }
        if (b.lane < kTreeMaxLevels) m.start[b.lane] = inc - c;
        if (b.lane == kTreeMaxLevels - 1) m.start[kTreeMaxLevels] = inc;
    }
    lds_barrier();
    for (int i = t; i < b.own; i += nt) {
        const int h = a.height[b.lo + i];
        if (h < kTreeMaxLevels) {
            const int r = m.start[h] + a.inv_perm[b.lo + i] - m.min[h];
            if (r >= 0 && r < b.own) b.order[r] = (uint16_t)i;
        }
        for (int e = b.cstart[i]; e < b.cstart[i + 1]; ++e) b.par[b.kids[e]] = (uint16_t)i;
    }
    return true;
}

template <bool SAVE>
__global__ void __launch_bounds__(kTreeMaxWaves * 64, 4)
trees_kernel(const TreesArgs a) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    __shared__ TreeMeta m;
    const int t = threadIdx.x, nt = blockDim.x;
    TreeBlock b;
    b.A = lds;
    b.Ht = b.A + a.group_rows * a.pitch_h;
    b.Fs = reinterpret_cast<float *>(b.Ht + a.group_rows * a.pitch_h);
    place_view(a, b, reinterpret_cast<char *>(b.Fs + a.group_rows * a.Hz));
    if (!view_trees(a, lds, b, m)) return;
    for (int i = t * 16; i < a.group_rows * a.pitch_h; i += nt * 16)      // pad columns of the h rows stay zero
        *reinterpret_cast<u32x4 *>(b.Ht + i) = u32x4{0, 0, 0, 0};
    // levels of this block that run here: [0, n_lvl)
    int n_lvl = 0;
    while (n_lvl < a.l_end && m.cnt[n_lvl] > 0) ++n_lvl;
    __syncthreads();

    if (n_lvl < 2) return;
    {   // the leaves: every wave for itself, 16 or 32 rows of 16 units at a time (waves side by side share the rows' lines in L1)
        const int n_leaf = m.cnt[0], n32 = n_leaf >> 5, rest = n_leaf & 31, n_tasks = (n32 + (rest > 0)) * a.n_ut;
        for (int q = b.wave; q < n_tasks; q += b.n_waves) {
            const int tile = q / a.n_ut, ut = q - tile * a.n_ut;
            if (tile < n32) forget_tile<SAVE, 2, true>(a, b, ut, tile * 32, tile * 32 + 32);
            else if (rest > 16) forget_tile<SAVE, 2, true>(a, b, ut, tile * 32, n_leaf);
            else if (rest > 4) forget_tile<SAVE, 1, true>(a, b, ut, tile * 32, n_leaf);
            else forget_tile<SAVE, 0, true>(a, b, ut, tile * 32, n_leaf);
        }
        __syncthreads();
    }
    for (int l = 1; l < n_lvl; ++l) {
        const int l0 = m.start[l], l1 = m.start[l + 1];
        for (int r0 = l0; r0 < l1; r0 += a.group_rows) {
            const int r_end = r0 + a.group_rows < l1 ? r0 + a.group_rows : l1, rows = r_end - r0;
            if (r0 > l0) lds_barrier();               // the group before is done with Fs
            gather_sums<float, 1, 8>(a, b, r0, r_end, a.sh * 4);
            lds_barrier();
            if (rows > 16) level_group<SAVE, 2>(a, b, r0, r_end);
            else if (rows > 4) level_group<SAVE, 1>(a, b, r0, r_end);
            else level_group<SAVE, 0>(a, b, r0, r_end);
            if (l + 1 >= n_lvl) continue;
            lds_barrier();
            for (int ut = b.wave; ut < a.n_ut; ut += b.n_waves) {
                if (rows > 16) forget_tile<SAVE, 2, false>(a, b, ut, r0, r_end);
                else if (rows > 4) forget_tile<SAVE, 1, false>(a, b, ut, r0, r_end);
                else forget_tile<SAVE, 0, false>(a, b, ut, r0, r_end);
            }
        }
        __syncthreads();                              // the next level's sums read what this one left in memory
    }
}

// ---- the levels with the recurrent weights in registers ----------------------------------------
// trees_kernel reads U from L2 once per level, and at 50 KB a microsecond and compute unit (measured: clock stamps) that is most of
// a level.  Where the four gates' weights of 16 units fit the registers of one wave, a wave loads them once, while the block works
// out its trees, and keeps them over all levels; bf16 wider than 160 and fp32 wider than 128 have room for i, o and u, and
// for f's first slabs in what LDS has left.  bf16 wider than 192 takes eight waves of two unit tiles each: 16 waves would
// have 32 registers beside the weights, eight have 64 (inner levels in groups of 16 rows, leaves 32 at a time, so that LDS holds
// all or all but a slab of f's weights).
// Schedule + forward, from L2 -> so: 71 nodes H 150 fp32 99 -> 89 us, 4.7 k nodes H 150 fp32 156 -> 141, 21 k nodes H 99 bf16
// 150 -> 125, 54 k nodes H 180 bf16 314 -> 258, 106 k nodes H 150 bf16 368 -> 316, 216 k nodes H 64 fp32 372 -> 367.  What bounds it:
// the 4x4 MFMAs of three waves on a SIMD and the barriers (few rows), memory traffic of Z, h and f c (many rows).
// NEAR: h and f c of all of the block's nodes stay in LDS (rows by local id), so that a level's sums wait for no memory;
// otherwise they go through memory as in trees_kernel, and Ht and C hold the rows of one group.
// Waves: unit tile wave % n_ut, rows in tiles of 16 (bf16) or 4 (fp32, whose 4x4 MFMAs have the rate of the 16x16 ones),
// dealt to the n_waves / n_ut sets of waves.
template <typename T, int NS> constexpr int kResTiles = NS * 4 / (int)sizeof(T);       // most unit tiles
template <typename T, int NS> constexpr int kResPerWave = kResTiles<T, NS> <= 12 ? 1 : 2;      // unit tiles of a wave
template <typename T, int NS> constexpr int kResWaves = kResTiles<T, NS> / kResPerWave<T, NS> <= 8 ? 8 : 12;
template <typename T, int NS> constexpr bool kResForget = NS * 16 <= (kResTiles<T, NS> <= 8 ? 128 : 80);   // f's weights in registers, too
template <typename T, int NS> constexpr int kResWeights = kResPerWave<T, NS> * NS * (kResForget<T, NS> ? 16 : 12);   // registers
template <typename T, int NS> constexpr int kResPerSimd = kResWaves<T, NS> == 12 ? 3 : kResWeights<T, NS> <= (sizeof(T) == 4 ? 64 : 32) ? 4 : 2;
template <typename T> constexpr int kResRows = sizeof(T) == 4 ? 4 : 16;                 // rows of a tile
template <typename T, int NS> constexpr int kResGroup = kResPerWave<T, NS> == 1 ? 64 : 16;      // most rows of a group (not NEAR)
constexpr int kResAhead = 2;                       // slabs of f's weights on their way from L2, of those that LDS does not hold
template <typename T, int NS> constexpr bool kResNearOnly = kResForget<T, NS> == false && sizeof(T) == 4;
template <typename T, int NS> constexpr bool kResFarOnly = kResPerWave<T, NS> > 1;

template <typename T, int NS>
struct ResWeights {
    u32x4 iou[kResPerWave<T, NS>][NS][3];
    u32x4 f[kResForget<T, NS> ? NS : 1][1];
};
// What one lane adds to a tile's products: four rows (16-row tiles: row hf * 4 + v) or one (4-row tiles: row hf).
template <int NG> struct ResPre { float z[NG][4]; };

struct ResBlock : TreeBlock {
    float *C;                 // LDS [slot][Hz]: sum of the children's f c, then c, then (NEAR) f c
    int ut, set, n_sets;      // the wave's unit tiles: ut, ut + n_waves, ... (n_tiles of them)
    int n_tiles;
    int piece, piece_row, piece_rows;      // res_gather: this thread's 16-byte piece, first row and rows a step
    char *F; int f_lds;       // LDS: the first f_lds slabs of f's weights, a wave's tile after the other, in lane order
};
// Row r's place in Ht and C.
template <bool NEAR>
__device__ __forceinline__ int res_slot(const ResBlock &b, int r, int r0) { return NEAR ? (int)b.order[r] : r - r0; }
template <typename T>
__device__ __forceinline__ bool res_quad(int row, int r_end) { return sizeof(T) == 4 || r_end - row <= 4; }
__device__ __forceinline__ int res_row(bool quad, int row, int r_end, int hf, int v) {
    const int r = row + (quad ? hf : hf * 4 + v);
    return r < r_end ? r : r_end - 1;
}
template <typename T>
__device__ __forceinline__ void res_load_z(const TreesArgs &a, const ResBlock &b, int ut, int row, int r_end, ResPre<3> &p) {
    if (row >= r_end) return;
    const int lane = fresh_lane(b.lane), unit = ut * 16 + (lane & 15);
    const bool quad = res_quad<T>(row, r_end);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        if (v > 0 && quad) break;
        const float *zp = a.Z + (int64_t)(b.lo + b.order[res_row(quad, row, r_end, lane >> 4, v)]) * 4 * a.Hz + unit;
#pragma unroll
        for (int g = 0; g < 3; ++g) p.z[g][v] = zp[g * a.Hz];
    }
}
template <typename T>
__device__ __forceinline__ void res_load_zf(const TreesArgs &a, const ResBlock &b, int ut, int row, int r_end, ResPre<1> &p) {
    if (row >= r_end) return;
    const int lane = fresh_lane(b.lane), unit = ut * 16 + (lane & 15);
    const bool quad = res_quad<T>(row, r_end);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        if (v > 0 && quad) break;
        const int i = b.order[res_row(quad, row, r_end, lane >> 4, v)], q = b.par[i];
        p.z[0][v] = a.Z[((int64_t)(b.lo + (q != kNoLocal ? q : i)) * 4 + 3) * a.Hz + unit];
    }
}

// acc[g] += A rows x the weights w[s][g]; a_lane: this lane's bytes of slab 0 (row lane & 15 or lane & 3, piece lane >> 4) in LDS.
template <typename T, int NS, int NG, bool QUAD>
__device__ __forceinline__ void res_gemm(floatx4 (&acc)[NG], const char *a_lane, const u32x4 (&w)[NS][NG]) {
    u32x4 fa[2];
    fa[0] = *reinterpret_cast<const u32x4 *>(a_lane);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        if (s + 1 < NS) fa[(s + 1) & 1] = *reinterpret_cast<const u32x4 *>(a_lane + (s + 1) * 64);
        const u32x4 &f = fa[s & 1];
        if constexpr (!QUAD) {
#pragma unroll
            for (int g = 0; g < NG; ++g) mfma16<T>(f, w[s][g], acc[g]);
        } else if constexpr (sizeof(T) == 2) {
#pragma unroll
            for (int g = 0; g < NG; ++g) mfma4<T>(f, w[s][g], acc[g]);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int g = 0; g < NG; ++g)
                    acc[g] = __builtin_amdgcn_mfma_f32_4x4x1f32(__uint_as_float(f[j]), __uint_as_float(w[s][g][j]), acc[g], 0, 0, 0);
        }
    }
}

// The cells of the tile of rows from `row` on.
template <typename T, bool SAVE, int NS, bool NEAR, bool QUAD>
__device__ __forceinline__ void res_cells(const TreesArgs &a, const ResBlock &b, int ut, const u32x4 (&w)[NS][3], const ResPre<3> &p,
                                          int row, int r0, int r_end) {
    constexpr int PITCH = NS * 64 + 16;
    const int lane = fresh_lane(b.lane), hf = lane >> 4, n = lane & 15, unit = ut * 16 + n;
    constexpr bool FROM_Z = kResPerWave<T, NS> > 1 && !QUAD;       // (fewer registers)
    floatx4 acc[3];
#pragma unroll
    for (int g = 0; g < 3; ++g)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[g][v] = FROM_Z ? p.z[g][v] : 0.0f;
    res_gemm<T, NS, 3, QUAD>(acc, b.A + (row - r0 + (QUAD ? lane & 3 : n)) * PITCH + hf * 16, w);
#pragma unroll
    for (int v = 0; v < (QUAD ? 1 : 4); ++v) {
        if constexpr (FROM_Z) __builtin_amdgcn_sched_barrier(0);
        float z[3];
#pragma unroll
        for (int g = 0; g < 3; ++g) z[g] = FROM_Z ? acc[g][v] : p.z[g][v] + (QUAD ? quarter_sum(acc[g], lane) : acc[g][v]);
        const int r = row + (QUAD ? hf : hf * 4 + v);
        if (r >= r_end) continue;
        const int i = b.order[r], slot = NEAR ? i : r - r0;
        const float gi = sigmoid_t<T>(z[0]), go = sigmoid_t<T>(z[1]), gu = tanh_t<T>(z[2]);
        float *cp = b.C + slot * a.Hz + unit;
        const float c = gi * gu + *cp;
        *cp = c;                                 // for the forget gates' step
        const T hv = unit < a.H ? from_f32<T>(go * tanh_t<T>(c)) : T(0);
        *reinterpret_cast<T *>(b.Ht + slot * PITCH + unit * (int)sizeof(T)) = hv;
        store_unit<T>(a, b.lo + i, unit, c, hv);
        if constexpr (SAVE) {
            if (unit < a.H) save_gates<T>(a, b.lo + i, unit, gi, go, gu);
        }
    }
}

// f c of the tile's rows from P = U_f h, f with the parent's Z_f (in p).  FAR_LEAF: c comes from memory, in cm.
template <typename T, bool SAVE, int NS, bool NEAR, bool QUAD, bool FAR_LEAF>
__device__ __forceinline__ void res_forget(const TreesArgs &a, const ResBlock &b, int ut, const ResWeights<T, NS> &w, const ResPre<1> &p,
                                           const ResPre<1> &cm, const char *rows, int row, int r0, int r_end) {
    constexpr int PITCH = NS * 64 + 16;
    const int lane = fresh_lane(b.lane), hf = lane >> 4, n = lane & 15, unit = ut * 16 + n;
    const int ra = row + (QUAD ? lane & 3 : n);
    const char *a_lane = rows + (NEAR ? (int)b.order[ra < r_end ? ra : r_end - 1] : ra - r0) * PITCH + hf * 16;
    floatx4 acc[1] = {floatx4{0, 0, 0, 0}};
    if constexpr (kResForget<T, NS>) {
        res_gemm<T, NS, 1, QUAD>(acc, a_lane, w.f);
    } else {
        // the slabs in LDS while the others are on their way
        const char *wp = tree_weights(a, lane, ut, a.sx_packed, 3), *fl = b.F + (ut * b.f_lds * 64 + lane) * 16;
        const int64_t slab = (int64_t)a.NPU * 64;
        const int rest = a.sh - b.f_lds;
        u32x4 ahead[kResAhead];
#pragma unroll
        for (int e = 0; e < kResAhead; ++e)
            if (e < rest) ahead[e] = *reinterpret_cast<const u32x4 *>(wp + (b.f_lds + e) * slab);
        floatx4 part[1][1] = {{floatx4{0, 0, 0, 0}}};
        auto multiply = [&](const u32x4 &fb, int s) __attribute__((always_inline)) {
            const u32x4 fa = *reinterpret_cast<const u32x4 *>(a_lane + s * 64);
            if constexpr (QUAD) mfma4<T>(fa, fb, part[0][0]);
            else mfma16<T>(fa, fb, part[0][0]);
        };
        for (int s = 0; s < b.f_lds; ++s) multiply(*reinterpret_cast<const u32x4 *>(fl + s * 1024), s);
#pragma unroll
        for (int e = 0; e < kResAhead; ++e)
            if (e < rest) multiply(ahead[e], b.f_lds + e);
        const int done = b.f_lds + kResAhead;
        if (done < a.sh)
            tree_gemm<T, QUAD ? 0 : 1, 1, false, kResAhead>(part, [&](int, int s) { return *reinterpret_cast<const u32x4 *>(a_lane + (done + s) * 64); },
                                                            wp + done * slab, slab, a.sh - done);
        acc[0] = part[0][0];
    }
#pragma unroll
    for (int v = 0; v < (QUAD ? 1 : 4); ++v) {
        const float pf = QUAD ? quarter_sum(acc[0], lane) : acc[0][v];
        const int r = row + (QUAD ? hf : hf * 4 + v);
        if (r >= r_end) continue;
        const int i = b.order[r];
        if (b.par[i] == kNoLocal) continue;
        const float f = sigmoid_t<T>(pf + p.z[0][v]);
        float *cp = b.C + (NEAR ? i : r - r0) * a.Hz + unit;
        const float fc = unit < a.H ? f * (FAR_LEAF ? cm.z[0][v] : *cp) : 0.0f;
        if constexpr (NEAR) *cp = fc;
        else a.FC[(int64_t)(b.lo + i) * a.Hz + unit] = fc;
        if constexpr (SAVE) {
            if (unit < a.H) static_cast<T *>(a.fgate)[(int64_t)(b.lo + i) * a.H + unit] = from_f32<T>(f);
        }
    }
}

// NEAR: child sums of rows [r0, r_end) from LDS into A and, of f c, into the rows' own places in C.  A thread sums one 16-byte
// piece of one row.
template <typename T, int NS>
__device__ __forceinline__ void res_gather(const TreesArgs &a, const ResBlock &b, int r0, int r_end) {
    constexpr int PITCH = NS * 64 + 16, VEC = Traits<T>::VEC, PH = NS * 4;
    const int k = b.piece;
    for (int r = r0 + b.piece_row; r < r_end; r += b.piece_rows) {
        const int i = b.order[r], rr = r - r0;
        const int c0 = b.cstart[i], c1 = b.cstart[i + 1];
        float s[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) s[e] = 0.0f;
        if (k < PH) {
            for (int c = c0; c < c1; ++c)        // ascending ids; pieces past the last unit tile are zero in every row
                add_h_piece<T>(s, *reinterpret_cast<const u32x4 *>(b.Ht + (int)b.kids[c] * PITCH + k * 16));
            T e[VEC];
#pragma unroll
            for (int j = 0; j < VEC; ++j) e[j] = from_f32<T>(s[j]);
            u32x4 v;
            __builtin_memcpy(&v, e, 16);
            *reinterpret_cast<u32x4 *>(b.A + rr * PITCH + k * 16) = v;
        } else {
            const int u = (k - PH) * 4;
            float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
            for (int c = c0; c < c1; ++c) {
                const float4 w = *reinterpret_cast<const float4 *>(b.C + (int)b.kids[c] * a.Hz + u);
                o.x += w.x; o.y += w.y; o.z += w.z; o.w += w.w;
            }
            *reinterpret_cast<float4 *>(b.C + i * a.Hz + u) = o;
        }
    }
}

// 16 bytes, piece k, of the h row of local node i; zero past the last unit tile.
template <typename T>
__device__ __forceinline__ u32x4 res_h_piece(const TreesArgs &a, const ResBlock &b, int i, int k) {
    u32x4 v = {0, 0, 0, 0};
    if (k * Traits<T>::VEC < a.Hz)
        v = *reinterpret_cast<const u32x4 *>(static_cast<const char *>(a.hs) + (int64_t)(b.lo + i) * a.Hp * (int)sizeof(T) + k * 16);
    return v;
}

template <typename T, bool SAVE, int NS, bool NEAR>
__global__ void __launch_bounds__((kResWaves<T, NS> * 64), (kResPerSimd<T, NS>))
trees_resident_kernel(const TreesArgs a) {
    constexpr int PITCH = NS * 64 + 16, STEP = kResRows<T>, NW = kResWaves<T, NS>, NT = NW * 64, PH = NS * 4, TW = kResPerWave<T, NS>;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    __shared__ TreeMeta m;
    const int t = threadIdx.x;
    ResBlock b;
    b.A = lds;
    b.Ht = b.A + a.group_rows * PITCH;
    b.C = reinterpret_cast<float *>(b.Ht + (NEAR ? a.cap : a.group_rows) * PITCH);
    b.Fs = b.C;
    {
        char *end = reinterpret_cast<char *>(b.C + (NEAR ? a.cap : a.group_rows) * a.Hz);
        if (TW > 1 && end < lds + 2 * TW * a.group_rows * PITCH) end = lds + 2 * TW * a.group_rows * PITCH;      // the leaves' buffers
        place_view(a, b, end);
    }
    b.F = lds + a.lds_bytes - (size_t)a.f_lds * a.n_ut * 1024;
    b.f_lds = a.f_lds;
    b.n_sets = TW > 1 ? 1 : NW / a.n_ut;
    b.set = TW > 1 ? 0 : b.wave / a.n_ut;
    b.ut = b.wave - b.set * a.n_ut;
    b.n_tiles = TW > 1 && b.ut + NW < a.n_ut ? 2 : 1;
    {
        const int per = PH + a.Hz / 4;
        b.piece_rows = NT / per;
        b.piece_row = t / per;
        b.piece = t - b.piece_row * per;
        if (b.piece_row >= b.piece_rows) b.piece_row = 1 << 20;
    }
    if (b.set >= b.n_sets) b.set = 1 << 20;               // a wave without a tile: no row is ever its own

    ResWeights<T, NS> w;
    auto load_cells_weights = [&](int j) __attribute__((always_inline)) {
        // slabs past the packed h part meet zeros, but 0 times an infinite weight would be NaN
        const char *wp = tree_weights(a, b.lane, b.ut + j * NW, a.sx_packed, 0);
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int g = 0; g < (kResForget<T, NS> ? 4 : 3); ++g) {
                u32x4 v = {0, 0, 0, 0};
                if (s < a.sh) v = *reinterpret_cast<const u32x4 *>(wp + (int64_t)s * a.NPU * 64 + g * 2048);
                if (g < 3) w.iou[j][s][g] = v;
                else w.f[kResForget<T, NS> ? s : 0][0] = v;
            }
    };
    {
        u32x4 wf[TW][kResForget<T, NS> ? 1 : NS];
        if constexpr (!kResForget<T, NS>) {
#pragma unroll
            for (int j = 0; j < TW; ++j)
#pragma unroll
                for (int s = 0; s < NS; ++s)
                    if (j < b.n_tiles && s < a.f_lds)
                        wf[j][s] = *reinterpret_cast<const u32x4 *>(tree_weights(a, b.lane, b.ut + j * NW, a.sx_packed, 3) + (int64_t)s * a.NPU * 64);
        }
        load_cells_weights(0);
        if constexpr (!kResForget<T, NS>) {
#pragma unroll
            for (int j = 0; j < TW; ++j)
#pragma unroll
                for (int s = 0; s < NS; ++s)
                    if (j < b.n_tiles && s < a.f_lds)
                        *reinterpret_cast<u32x4 *>(b.F + (((b.ut + j * NW) * a.f_lds + s) * 64 + b.lane) * 16) = wf[j][s];
        }
    }
    if (!view_trees(a, lds, b, m)) return;
    int n_lvl = 0;                                        // levels of this block that run here: [0, n_lvl)
    lds_barrier();
    while (n_lvl < a.l_end && m.cnt[n_lvl] > 0) ++n_lvl;
    if (n_lvl < 2) return;

    const ResPre<1> none = {};
    const int n_leaf = m.cnt[0];
    ResPre<1> zf;
    // a wave's tiles of rows and units: at % TW counts the units', at / TW is the first row
    auto ut_of = [&](int at) __attribute__((always_inline)) { return TW > 1 ? b.ut + (at % TW) * NW : b.ut; };
    auto after = [&](int at) __attribute__((always_inline)) {
        return TW > 1 && at % TW + 1 < b.n_tiles ? at + 1 : (at / TW + b.n_sets * STEP) * TW;
    };
    auto forget_rows = [&](int r0, int r_end) __attribute__((always_inline)) {      // (zf: the first tile's)
        for (int at = (r0 + b.set * STEP) * TW; at / TW < r_end;) {
            const int row = at / TW, ut = ut_of(at);
            const ResPre<1> cur = zf;
            at = after(at);
            res_load_zf<T>(a, b, ut_of(at), at / TW, r_end, zf);
            if (res_quad<T>(row, r_end)) res_forget<T, SAVE, NS, NEAR, true, false>(a, b, ut, w, cur, none, b.Ht, row, r0, r_end);
            else res_forget<T, SAVE, NS, NEAR, sizeof(T) == 4, false>(a, b, ut, w, cur, none, b.Ht, row, r0, r_end);
        }
    };
    // ---- the leaves, whose cells are done: their f c
    if constexpr (NEAR) {
        res_load_zf<T>(a, b, b.ut, b.set * STEP, n_leaf, zf);
        const int per = PH + a.Hz / 4;
        for (int q = t; q < b.own * per; q += NT) {       // rows of h and c (other nodes: zero pads) side by side
            const int r = q / per, k = q - r * per, i = b.order[r];
            if (k < PH) {
                if (r < n_leaf) *reinterpret_cast<u32x4 *>(b.Ht + i * PITCH + k * 16) = res_h_piece<T>(a, b, i, k);
                else if (k * Traits<T>::VEC >= a.Hz) *reinterpret_cast<u32x4 *>(b.Ht + i * PITCH + k * 16) = u32x4{0, 0, 0, 0};
            } else if (r < n_leaf) {
                const int u = (k - PH) * 4;
                const float *c = a.c_out + (int64_t)(b.lo + i) * a.H;
                float4 o;
                o.x = u < a.H ? c[u] : 0.0f; o.y = u + 1 < a.H ? c[u + 1] : 0.0f;
                o.z = u + 2 < a.H ? c[u + 2] : 0.0f; o.w = u + 3 < a.H ? c[u + 3] : 0.0f;
                *reinterpret_cast<float4 *>(b.C + i * a.Hz + u) = o;
            }
        }
        lds_barrier();
        forget_rows(0, n_leaf);
    } else {
        // leaf_rows of them at a time through LDS (two buffers in turn), the next ones' rows on their way meanwhile
        const int leaf_rows = a.group_rows * TW;
        constexpr int MOST = (kResGroup<T, NS> * TW * PH + NT - 1) / NT;
        u32x4 ahead[MOST];
        auto request = [&](int r0) __attribute__((always_inline)) {
#pragma unroll
            for (int e = 0; e < MOST; ++e) {
                const int q = t + e * NT, r = r0 + q / PH;
                if (q < leaf_rows * PH && r < n_leaf) ahead[e] = res_h_piece<T>(a, b, b.order[r], q % PH);
            }
        };
        auto load_c = [&](int ut, int row, int r_end, ResPre<1> &p) __attribute__((always_inline)) {
            if (row >= r_end) return;
            const int lane = fresh_lane(b.lane), unit = ut * 16 + (lane & 15);
            const bool quad = res_quad<T>(row, r_end);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                if (v > 0 && quad) break;
                p.z[0][v] = a.c_out[(int64_t)(b.lo + b.order[res_row(quad, row, r_end, lane >> 4, v)]) * a.H + (unit < a.H ? unit : 0)];
            }
        };
        // this wave's tiles, one group after the other; what a tile adds is requested two tiles ahead
        auto group_end = [&](int row) __attribute__((always_inline)) {
            const int e = row / leaf_rows * leaf_rows + leaf_rows;
            return e < n_leaf ? e : n_leaf;
        };
        auto leaves_after = [&](int at) __attribute__((always_inline)) {
            if (TW > 1 && at % TW + 1 < b.n_tiles) return at + 1;
            const int row = at / TW, e = group_end(row), next = row + b.n_sets * STEP;
            return TW * (row >= n_leaf ? n_leaf : next < e ? next : e + b.set * STEP);
        };
        auto load_tile = [&](int at, ResPre<1> &zp, ResPre<1> &cp) __attribute__((always_inline)) {
            const int row = at / TW;
            if (row >= n_leaf) return;
            res_load_zf<T>(a, b, ut_of(at), row, group_end(row), zp);
            load_c(ut_of(at), row, group_end(row), cp);
        };
        request(0);
        char *const buf1 = lds + leaf_rows * PITCH, *buf = buf1;
        ResPre<1> zf1, cm, cm1;
        int at0 = TW * (b.set * STEP < leaf_rows ? b.set * STEP : n_leaf), at1 = leaves_after(at0);
        load_tile(at0, zf, cm);
        load_tile(at1, zf1, cm1);
        for (int r0 = 0; r0 < n_leaf; r0 += leaf_rows) {
            const int r_end = r0 + leaf_rows < n_leaf ? r0 + leaf_rows : n_leaf;
#pragma unroll
            for (int e = 0; e < MOST; ++e) {
                const int q = t + e * NT;
                if (q < leaf_rows * PH) *reinterpret_cast<u32x4 *>(buf + (q / PH) * PITCH + (q % PH) * 16) = ahead[e];
            }
            request(r0 + leaf_rows);
            lds_barrier();
            while (at0 / TW < r_end) {
                const int row = at0 / TW, ut = ut_of(at0);
                const ResPre<1> cur = zf, cc = cm;
                at0 = at1;
                at1 = leaves_after(at0);
                zf = zf1; cm = cm1;
                load_tile(at1, zf1, cm1);
                if (res_quad<T>(row, r_end)) res_forget<T, SAVE, NS, false, true, true>(a, b, ut, w, cur, cc, buf, row, r0, r_end);
                else res_forget<T, SAVE, NS, false, sizeof(T) == 4, true>(a, b, ut, w, cur, cc, buf, row, r0, r_end);
            }
            buf = buf == buf1 ? lds : buf1;
        }
        lds_barrier();
        for (int i = t * 16; i < a.group_rows * PITCH; i += NT * 16)      // pad columns of the h rows stay zero
            *reinterpret_cast<u32x4 *>(b.Ht + i) = u32x4{0, 0, 0, 0};
        // (the leaves' steps need the registers)
        if constexpr (TW > 1)
            if (b.n_tiles > 1) load_cells_weights(1);
    }
    ResPre<3> z;
    res_load_z<T>(a, b, b.ut, m.start[1] + b.set * STEP, m.start[1] + a.group_rows < m.start[2] ? m.start[1] + a.group_rows : m.start[2], z);
    if constexpr (NEAR) lds_barrier();
    else __syncthreads();

    for (int l = 1; l < n_lvl; ++l) {
        const int l1 = m.start[l + 1];
        for (int r0 = m.start[l]; r0 < l1; r0 += a.group_rows) {
            const int r_end = r0 + a.group_rows < l1 ? r0 + a.group_rows : l1;
            if (r0 > m.start[l]) lds_barrier();           // the group before is done with A and C
            if constexpr (NEAR) res_gather<T, NS>(a, b, r0, r_end);
            else if constexpr (kResPerSimd<T, NS> == 4) gather_sums<T, 1, 8>(a, b, r0, r_end, PH);
            else if constexpr (TW > 1) gather_sums<T, 2, 2>(a, b, r0, r_end, PH);
            else gather_sums<T, 2, 4>(a, b, r0, r_end, PH);
            lds_barrier();
            if (TW == 1 && l + 1 < n_lvl) res_load_zf<T>(a, b, b.ut, r0 + b.set * STEP, r_end, zf);
            for (int row = r0 + b.set * STEP; row < r_end; row += b.n_sets * STEP) {
#pragma unroll
                for (int j = 0; j < TW; ++j) {
                    if (j >= b.n_tiles) break;
                    const ResPre<3> cur = z;
                    if (j + 1 < b.n_tiles) res_load_z<T>(a, b, b.ut + (j + 1) * NW, row, r_end, z);
                    else res_load_z<T>(a, b, b.ut, row + b.n_sets * STEP, r_end, z);
                    if (res_quad<T>(row, r_end)) res_cells<T, SAVE, NS, NEAR, true>(a, b, b.ut + j * NW, w.iou[j], cur, row, r0, r_end);
                    else res_cells<T, SAVE, NS, NEAR, sizeof(T) == 4>(a, b, b.ut + j * NW, w.iou[j], cur, row, r0, r_end);
                }
            }
            if (TW > 1 && l + 1 < n_lvl) res_load_zf<T>(a, b, b.ut, r0, r_end, zf);      // (no registers for it before)
            {   // the next group's
                const int e1 = r_end < l1 ? l1 : l + 1 < n_lvl ? m.start[l + 2] : r_end;
                res_load_z<T>(a, b, b.ut, r_end + b.set * STEP, r_end + a.group_rows < e1 ? r_end + a.group_rows : e1, z);
            }
            if (l + 1 >= n_lvl) continue;
            lds_barrier();
            forget_rows(r0, r_end);
        }
        if constexpr (NEAR) lds_barrier();                // the next level's sums read what this one left
        else __syncthreads();
    }
}

constexpr int kTreeLdsMax = 156 * 1024;
constexpr int kTreeNodesPerBlock = 128;
constexpr int kTreeLdsStatic = 1024;               // trees_kernel's static LDS, rounded up

}  // namespace

// The largest forest that runs as whole trees; workspaces have room for no larger one.
int64_t trees_max_nodes(int D, int H, size_t esz) {
    // The gain shrinks with the number of nodes, where the level kernels fill the chip, and with what they spend on x.  Schedule +
    // forward in bf16, level by level -> here: H = 168 and 192, D = 300 384, 377 -> 258, 250 us (73 k nodes), 868, 845 -> 675, 653
    // (214 k), D = 64 337, 332 -> 261, 256 (73 k), 358, 346 -> 352, 344 (106 k), 612, 577 -> 639, 614 (214 k).  H = 200 to 256, which
    // hold fewer weights: D = 300 414 - 429 -> 361 - 389 (73 k), 558 - 586 -> 494 - 528 (106 k), 969 - 1015 -> 950 - 994 (214 k),
    // D = 64 364 - 374 -> 360 - 387 (73 k), 406 - 447 -> 494 - 520 (106 k).  fp32, D = 300: H = 64 234 -> 96 (4.7 k), 1198 -> 539 (214 k),
    // H = 150 2028 -> 1406, H = 256 296 -> 228 (4.7 k), 2530 -> 2321 (214 k).  H = 384 slower throughout.
    // fp32 and up to 160 units: the largest forest measured, rounded up.  (Its room, 20 bytes a node and unit, is more than the levels
    // take up to 0.3 - 1 M nodes.)  Wider bf16 cells stop where whole trees gain little or where a forest of kTreesRoomNodes, and
    // with it every larger one, would be asked for more than its levels take: at D = 300 that is 110 k nodes for H = 192 (262 144
    // nodes would make its 0.41 GB 0.97).
    if (H > kTreesMaxWidth || ceil_div((int64_t)D * (int64_t)esz, 64) > kXSlabs[sizeof(kXSlabs) / sizeof(int) - 1]) return 0;
    if (esz == 4 || H <= 160) return 262144;
    if (H > 192) return D >= 256 ? 81920 : 65536;       // (within that room, too)
    constexpr int64_t kTreesRoomNodes = 300000;
    const int kpad = Traits<bf16_t>::BK;
    const int64_t level_bytes = 2 * (round_up(D, kpad) + round_up(H, kpad) + round_up(H, 8));     // a row of the stacked input, one of P
    const int64_t room = kTreesRoomNodes * level_bytes / (20 * round_up(H, 16)), gains = D >= 128 ? 262144 : 106496;
    return room < gains ? room : gains;
}

// Microseconds by which whole trees take longer than the level kernels (less than zero: they are faster).  What speaks against
// them: the longest run of trees keeps one block busy while the others are done (a.tree_window nodes past its share, more the
// wider the cells), and every level costs each block the latency of its weights.  For them: a level costs no launches, and
// less the wider x is; the level kernels walk a node's children one by one (the widest node of a level that averages more than
// two or three has several times that); the chain levels above multiply no x.
// Fitted to 1400 measured forwards: D 16 - 300, H 40 - 256, one tree of 16 - 250 nodes, interleaved trees of 1 - 10 nodes, stars,
// trees of 1 - 250 nodes filed one after another up to 225 k nodes, chains.  The time over that of the faster form, mean and
// worst: always whole trees 1.18 and 4.3 in fp32, 1.13 and 3.1 in bf16; by this rule 1.005 and 1.3, 1.006 and 1.4.  Those forwards
// ran on trees_kernel, which read the weights once a level, in bf16 too.  Timed both ways since most run on
// trees_resident_kernel, the chosen form takes in 120 forwards of filed trees 1.01 of the faster one's time in the mean and 1.13 at
// worst, in 45 of interleaved trees of 1 - 10 nodes and single trees 1.03 and 1.45; the worst are 154 k nodes in trees of 1 - 3, D 32,
// H 100, which run whole: bf16, ids over each other in runs of 120, 238 us against 164, fp32, runs of 250, 501 against 386.
double trees_excess_us(const TreesArgs &a, size_t esz, const TreesShape &s) {
    const bool f32 = esz == 4;
    const double h = a.H / 100.0, d = a.D / 100.0, below = s.n_below / 1000.0, chain = (a.n - s.n_below) / 1000.0;
    const int levels = a.l_end, chain_levels = s.n_levels - a.l_end;
    const int longest = a.n - a.G < a.tree_window ? a.n - a.G : a.tree_window;
    double us = levels * (f32 ? -11.0 + 3.0 * h - 1.2 * d : -8.9 + 2.6 * h - 0.35 * d) +
                below * (f32 ? -0.80 - 0.37 * d : -0.067 - 0.097 * d) + (below + chain) * h * (f32 ? 0.16 : 0.025) +
                chain_levels * (f32 ? 0.06 - 1.26 * d : 0.15 - 0.37 * d) + chain * (f32 ? 0.47 - 0.085 * d : 0.41 - 0.053 * d);
    if (levels > 1)
        us += 20.0 - (f32 ? 3.8 : 5.5) * h + longest * h * (f32 ? 0.29 : 0.137) - s.fan * (f32 ? 0.75 : 0.49) - s.wide * (f32 ? 2.5 : 1.2);
    return us;
}

// Weight slabs of the resident form's instances (0 waves: not for this type).
constexpr int kResSlabs[] = {2, 4, 5, 6, 8, 10};
static constexpr int resident_waves(int ns, size_t esz) {
    if (esz == 2) return ns == 2 || ns == 4 || ns == 8 ? 8 : ns == 5 || ns == 6 ? 12 : 0;
    return ns == 4 || ns == 8 ? 8 : ns == 10 ? 12 : 0;
}
static constexpr bool resident_forget(int ns, size_t esz) { return esz == 4 ? ns <= 8 : ns <= 5; }
static constexpr bool resident_shares_cu(int ns, size_t esz) { return ns * (int)esz * 4 <= (esz == 4 ? 64 : 16); }

// Which of the two x kernels runs in bf16.  Whole forward, loads in operand layout -> through LDS, H 150 unless stated: up to four
// slabs D 127 93 -> 84 us (20 k nodes), D 64 80 -> 82 (20 k), 238 -> 228 (106 k), 452 -> 423 (214 k); seven slabs with odd D, D 203
// 64 -> 59 (5 k), 98 -> 89 (20 k), 297 -> 272 (106 k); rows of whole 128-byte lines, D 192, 1.00 - 1.06 times the time up to 52 k nodes,
// 0.97 - 1.02 from 106 k on; with other even D, 224 66 -> 69 (10 k), 80 -> 87 (20 k), 127 -> 140 (52 k), 250 -> 258 (106 k), D 200
// 344 -> 353 (150 k), of all of them 1.03 times the time up to there (H 64 - 160), 1.01 - 1.02 from 180 k on, where D 224 gains up to 5 %.
static bool x_through_lds(const TreesArgs &a, size_t esz) {
    if (esz != 2 || a.x_slabs > kXLdsSlabs) return false;
    return a.x_slabs <= kXLdsAlways || (a.D & 1) != 0 || a.D % 64 == 0 || a.n >= kXLdsManyNodes;
}

// Fills the launch geometry of `a`; false if the forest is better run level by level.
bool plan_trees(TreesArgs &a, size_t esz, const TreesShape &s) {
    if (a.n > trees_max_nodes(a.D, a.H, esz)) return false;
    a.sx = (int)ceil_div((int64_t)a.D * (int64_t)esz, 64);
    a.sh = (int)ceil_div((int64_t)a.H * (int64_t)esz, 64);
    a.Hz = (int)round_up(a.H, 16);
    a.n_ut = a.Hz / 16;
    const size_t cuts = (size_t)2 * (2 * a.tree_window + 2) * 4;
    a.res_slabs = 0;
    for (int ns : kResSlabs)
        if (a.res_slabs == 0 && ns >= a.sh && resident_waves(ns, esz) > 0) a.res_slabs = ns;
    if (a.res_slabs > 0) {
        a.n_waves = resident_waves(a.res_slabs, esz);
        a.pitch_h = a.res_slabs * 64 + 16;
        const int most = resident_shares_cu(a.res_slabs, esz) ? 2 : 1;      // blocks of a compute unit
        const size_t row = (size_t)a.pitch_h + 4 * a.Hz;
        a.group_rows = kTreeRows;
        a.near_rows = 0;
        const bool two_tiles = esz == 2 && a.res_slabs == 8;              // (through memory only)
        for (int per_cu = 1; per_cu <= most && !a.near_rows && !two_tiles; ++per_cu) {
            a.G = (int)ceil_div(a.n, kTreeCus * per_cu);
            a.cap = a.G + a.tree_window < a.n ? a.G + a.tree_window : a.n;
            const size_t tiles = (size_t)a.group_rows * a.pitch_h + a.cap * row;
            a.lds_bytes = (tiles > cuts ? tiles : cuts) + (size_t)(4 * a.cap + 8) * 2;
            a.near_rows = (a.lds_bytes + kTreeLdsStatic) * per_cu <= (size_t)kTreeLdsMax;
        }
        if (!a.near_rows && a.res_slabs == 10) a.res_slabs = 0;       // (fp32 wider than 128 has no other form)
        for (int rows = two_tiles ? kResGroup<bf16_t, 8> : kResGroup<bf16_t, 4>; !a.near_rows && a.res_slabs > 0; rows /= 2) {
            a.group_rows = rows;
            int per_cu = (int)ceil_div(a.n, (int64_t)kTreeCus * kTreeNodesPerBlock);
            if (per_cu > most) per_cu = most;
            for (;; --per_cu) {
                a.G = (int)ceil_div(a.n, kTreeCus * per_cu);
                a.cap = a.G + a.tree_window < a.n ? a.G + a.tree_window : a.n;
                const size_t leaves = (size_t)rows * a.pitch_h * (two_tiles ? 4 : 2);      // two buffers
                const size_t tiles = leaves > rows * (a.pitch_h + row) ? leaves : rows * (a.pitch_h + row);
                a.lds_bytes = (tiles > cuts ? tiles : cuts) + (size_t)(4 * a.cap + 8) * 2;
                if (per_cu == 1 || (a.lds_bytes + kTreeLdsStatic) * per_cu <= (size_t)kTreeLdsMax) break;
            }
            if (a.lds_bytes + kTreeLdsStatic <= (size_t)kTreeLdsMax || rows <= 16) break;
        }
    }
    a.f_lds = 0;
    if (a.res_slabs > 0 && !resident_forget(a.res_slabs, esz)) {      // what LDS has left holds f's weights
        const int64_t left = (int64_t)kTreeLdsMax - kTreeLdsStatic - 16 - (int64_t)a.lds_bytes;
        a.f_lds = left > 0 ? (int)(left / (a.n_ut * 1024)) : 0;
        if (a.f_lds > a.sh) a.f_lds = a.sh;
        a.lds_bytes = (size_t)round_up((int64_t)a.lds_bytes, 16) + (size_t)a.f_lds * a.n_ut * 1024;
    }
    if (a.res_slabs == 0) {
        a.pitch_h = a.sh * 64 + 16;
        const int passes = (int)ceil_div(a.n_ut, kTreeMaxWaves);
        a.n_waves = (int)round_up(ceil_div(a.n_ut, passes), 4);  // whole rounds of the four SIMDs, so that blocks share them evenly
        if (a.n_waves < 8) a.n_waves = 8;                       // for the gathers
        const size_t row_bytes = (size_t)2 * a.pitch_h + 4 * a.Hz;
        a.group_rows = kTreeRows * row_bytes <= (size_t)kTreeLdsMax * 9 / 10 ? kTreeRows : kTreeRows / 2;
        const size_t tiles = a.group_rows * row_bytes;
        // one block per compute unit up to kTreeNodesPerBlock nodes each, then as many as registers and LDS let it hold (two blocks
        // hide each other's latencies, but a small forest's blocks should not share a compute unit while others idle)
        int per_cu = (int)ceil_div(a.n, (int64_t)kTreeCus * kTreeNodesPerBlock);
        if (per_cu > kTreeMaxWaves / a.n_waves) per_cu = kTreeMaxWaves / a.n_waves;
        for (;; --per_cu) {
            a.G = (int)ceil_div(a.n, kTreeCus * per_cu);
            a.cap = a.G + a.tree_window;
            if (a.cap > a.n) a.cap = a.n;
            a.lds_bytes = (tiles > cuts ? tiles : cuts) + (size_t)(4 * a.cap + 8) * 2;
            if (per_cu == 1 || (a.lds_bytes + kTreeLdsStatic) * per_cu <= (size_t)kTreeLdsMax) break;
        }
    }
    if (a.lds_bytes > (size_t)kTreeLdsMax || a.cap >= kNoLocal) return false;
    a.n_blocks = (int)ceil_div(a.n, a.G);
    if (trees_excess_us(a, esz, s) > 0.0) return false;
    // x part: one wave per unit tile and run of node tiles; as many waves as the chip holds at a time
    a.x_slabs = 0;
    for (int ns : kXSlabs)
        if (a.x_slabs == 0 && ns >= a.sx) a.x_slabs = ns;
    const int64_t waves = (int64_t)kTreeCus * 4 * kXWavesPerSimd(a.x_slabs), tiles16 = ceil_div(a.n_leaves, 16) + ceil_div(a.n - a.n_leaves, 16);
    a.x_rt = 1;
    if (!x_through_lds(a, esz)) {
        a.x_chunks = (int)(waves / a.n_ut);
    } else {      // a block fetches for four unit tiles, 32 rows a time where that leaves no block without work
        a.x_chunks = (int)(waves / (kXLdsWaves * ceil_div(a.n_ut, kXLdsWaves)));
        if (tiles16 >= 2 * (int64_t)a.x_chunks) a.x_rt = kXLdsRows / 16;
    }
    if (a.x_chunks > ceil_div(tiles16, a.x_rt)) a.x_chunks = (int)ceil_div(tiles16, a.x_rt);
    if (a.x_chunks < 1) a.x_chunks = 1;
    return true;
}

namespace {
template <typename T, bool SAVE, int NS>
int launch_tree_x(const TreesArgs &a, hipStream_t st) {
    if constexpr (sizeof(T) == 2 && NS <= kXLdsSlabs) {
        if (NS <= kXLdsAlways || x_through_lds(a, sizeof(T))) {
            tree_x_lds_kernel<SAVE, NS><<<(unsigned)(8 * ceil_div(a.x_chunks * ceil_div(a.n_ut, kXLdsWaves), 8)), kXLdsWaves * 64, 0, st>>>(a);
            JITDB_LAUNCH_CHECK();
            return JITDB_OK;
        }
    }
    if constexpr (sizeof(T) == 4 || NS > kXLdsAlways) tree_x_kernel<T, SAVE, NS><<<(unsigned)(8 * ceil_div((int64_t)a.x_chunks * a.n_ut, 32)), 256, 0, st>>>(a);
    JITDB_LAUNCH_CHECK();
    return JITDB_OK;
}
template <typename T, bool SAVE, int NS>
int launch_resident(const TreesArgs &a, hipStream_t st) {
    static_assert(resident_waves(NS, sizeof(T)) == kResWaves<T, NS> && resident_forget(NS, sizeof(T)) == kResForget<T, NS> &&
                  resident_shares_cu(NS, sizeof(T)) == (kResPerSimd<T, NS> * 4 >= 2 * kResWaves<T, NS>), "plan_trees sizes LDS and blocks by these");
    auto fn = &trees_resident_kernel<T, SAVE, NS, !kResFarOnly<T, NS>>;
    if constexpr (!kResNearOnly<T, NS>)
        if (!a.near_rows) fn = &trees_resident_kernel<T, SAVE, NS, false>;
    if (a.lds_bytes > 64 * 1024)
        JITDB_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void *>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, kTreeLdsMax));
    fn<<<a.n_blocks, kResWaves<T, NS> * 64, a.lds_bytes, st>>>(a);
    JITDB_LAUNCH_CHECK();
    return JITDB_OK;
}
template <typename T, bool SAVE>
int launch_trees_t(const TreesArgs &a, hipStream_t st) {
    int rc = JITDB_E_BADARG;
    switch (a.x_slabs) {
        case 4: rc = launch_tree_x<T, SAVE, 4>(a, st); break;
        case 7: rc = launch_tree_x<T, SAVE, 7>(a, st); break;
        case 10: rc = launch_tree_x<T, SAVE, 10>(a, st); break;
        case 16: rc = launch_tree_x<T, SAVE, 16>(a, st); break;
        case 20: rc = launch_tree_x<T, SAVE, 20>(a, st); break;
    }
    if (rc != JITDB_OK || a.l_end < 2) return rc;
    switch (a.res_slabs) {
        case 2: if constexpr (sizeof(T) == 2) return launch_resident<T, SAVE, 2>(a, st); break;
        case 4: return launch_resident<T, SAVE, 4>(a, st);
        case 5: if constexpr (sizeof(T) == 2) return launch_resident<T, SAVE, 5>(a, st); break;
        case 6: if constexpr (sizeof(T) == 2) return launch_resident<T, SAVE, 6>(a, st); break;
        case 8: return launch_resident<T, SAVE, 8>(a, st);
        case 10: if constexpr (sizeof(T) == 4) return launch_resident<T, SAVE, 10>(a, st); break;
    }
    if constexpr (sizeof(T) == 4) {
        if (a.lds_bytes > 64 * 1024)
            JITDB_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void *>(&trees_kernel<SAVE>), hipFuncAttributeMaxDynamicSharedMemorySize, kTreeLdsMax));
        trees_kernel<SAVE><<<a.n_blocks, a.n_waves * 64, a.lds_bytes, st>>>(a);
        JITDB_LAUNCH_CHECK();
        return JITDB_OK;
    }
    return JITDB_E_BADARG;                      // (every bf16 width has its instance)
}
}  // namespace

int launch_trees(jitdb_dtype dtype, bool save, const TreesArgs &a, hipStream_t st) {
    if (dtype == JITDB_F32) return save ? launch_trees_t<float, true>(a, st) : launch_trees_t<float, false>(a, st);
    return save ? launch_trees_t<bf16_t, true>(a, st) : launch_trees_t<bf16_t, false>(a, st);
}

}  // namespace jitdb
