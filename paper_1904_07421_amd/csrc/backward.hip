// jitdb_treelstm_backward: reverse-mode gradients of the level-batched Tree-LSTM forward.
//
// The paper trains through the same batched graph it infers with (section 5).  Only what a node hands to its children
// has to follow the levels: the levels are visited from the roots down with two steps each,
//
//   bwd_cell_kernel      dh_j = gh_j + dhs_p + ufg_j, dc_j = gc_j + dc_p f_j + ..., then row r of
//                        dZ = [dz_i | dz_o | dz_u | sum_k dz_f,k] and each child's row of G: dz_f,k = dc_j c_k f_k (1 - f_k)
//   one product          dhs = dZ_iou U_iou for this level's rows and ufg = G U_f for the next level's
//
// and everything that sums over nodes or is nobody's input waits for the end, where it runs once over all nodes:
//
//   dx = dZ W                                        (leaves have no forget block)
//   [dW | db] = [x | 1]^T dZ,  dU_iou = hs^T dZ_iou,  dU_f = h^T G      one launch, reduction over the nodes
//
// dZ, G and the operands x, h, hs are K-blocked, rows in the schedule's position order.  The sums over nodes read the same
// rows as the other products (the transposition happens on the way out of LDS, MODE_TN of tile_gemm.h): nothing is written
// twice.  Kernel time of the backward pass, with a weight-gradient product, its transposes and a dx product in every level
// -> like this: 4683 nodes in 7 levels, D = 300, H = 150, fp32: 1.95 ms -> 0.22; 1.18 M nodes in 15 levels, D = 300,
// H = 512, bf16: 19.0 ms -> 15.1.
//
// Gradients are fp32; with JITDB_BF16 the operands of the products (dz, x, h, hs, weights) and the values handed from level
// to level through dhs and ufg are bfloat16, every sum and dc fp32.

#include <algorithm>

#include "tile_gemm.h"

namespace jitdb {
namespace {

constexpr int kT = 256;

__global__ void __launch_bounds__(kT)
fill_f32_kernel(float *p, int64_t n, float v) {
    for (int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x; i < n; i += (int64_t)gridDim.x * kT) p[i] = v;
}

// N units from p[0 ..]; those past `left` are zero.  VEC: rows start on 4-byte boundaries.
template <typename E, int N, bool VEC>
__device__ __forceinline__ void load_units(const E *__restrict__ p, int left, float (&v)[N]) {
    typedef u32x4 __attribute__((aligned(4))) u32x4a;
    constexpr int PER = 16 / (int)sizeof(E);
    if (VEC && left >= N) {
#pragma unroll
        for (int q = 0; q < N / PER; ++q) {
            const u32x4 w = reinterpret_cast<const u32x4a *>(p)[q];
#pragma unroll
            for (int e = 0; e < PER; ++e) {
                if constexpr (sizeof(E) == 4) v[q * PER + e] = __uint_as_float(w[e]);
                else v[q * PER + e] = __uint_as_float(e & 1 ? w[e / 2] & 0xFFFF0000u : w[e / 2] << 16);
            }
        }
    } else if (VEC && sizeof(E) == 2) {        // an even number of units: pairs (106 k nodes, H 150: 1.07 -> 0.86 ms of the pass)
#pragma unroll
        for (int q = 0; q < N / 2; ++q) {
            uint32_t w = 0;
            if (2 * q < left) w = reinterpret_cast<const uint32_t *>(p)[q];
            v[2 * q] = __uint_as_float(w << 16);
            v[2 * q + 1] = __uint_as_float(w & 0xFFFF0000u);
        }
    } else {
#pragma unroll
        for (int e = 0; e < N; ++e) v[e] = e < left ? to_f32<E>(p[e]) : 0.0f;
    }
}
template <typename T> constexpr int kPer = 16 / (int)sizeof(T);       // units in 16 bytes
template <typename T>
__device__ __forceinline__ u32x4 pack_units(const float (&v)[kPer<T>]) {
    u32x4 o;
    if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = __float_as_uint(v[e]);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (uint32_t)f32_to_bf16(v[2 * e]) | ((uint32_t)f32_to_bf16(v[2 * e + 1]) << 16);
    }
    return o;
}
__device__ __forceinline__ void store16(void *base, int64_t row, int64_t kbyte, int64_t rows_alloc, const u32x4 &v) {
    *reinterpret_cast<u32x4 *>(static_cast<char *>(base) + operand_offset(row, kbyte, rows_alloc)) = v;
}

// The elementwise kernels work on 64 units of a few rows: a thread has 16 bytes of T of one row, the threads of a row 64
// units side by side (whole 128- or 256-byte pieces of the row-major arrays, two or four slabs of the K-blocked ones).
template <typename T> constexpr int kPieces = 64 / kPer<T>;
template <typename T> constexpr int kRows = kT / kPieces<T>;

// ---- operands that do not depend on the gradient ------------------------------------------
struct PrepArgs {
    const void *x, *h, *W, *U;
    const int32_t *perm, *child_ptr, *child_idx;
    int32_t *parent_of;
    void *AX, *AH, *AS, *dZ, *G, *Wt, *Ut, *Uft;
    int D, H, Hk;
    int n, n_rows, first;          // nodes; rows that the sums over the nodes may read; first row of AS that anything reads
    int64_t rows_alloc, w_alloc, u_alloc;
    int x_groups, row_blocks, h_groups;
};
// Rows [0, n_rows) of AX = [x | 1], AH = h and, from row `first` on, AS = sum of the children's h (fp32 sums, rounded once as the
// forward does), zero past n; parent_of = -1; rows n .. n_rows of dZ and G zero (they meet zero rows in the sums over the
// nodes, so they only have to be finite).  Blocks past those: the weights as operands of the data gradients, Wt [D rows,
// 4 Hk], Ut [H, 3 Hk], Uft [H, Hk]: row n = column n of W / U_iou / U_f, the gates at stride Hk, pad units zero.
template <typename T, bool VX, bool VH>
__global__ void __launch_bounds__(kT)
bwd_prepare_kernel(const PrepArgs a) {
    constexpr int PER = kPer<T>;
    const int groups = a.x_groups + a.h_groups;
    const int64_t pack_blocks = (int64_t)a.row_blocks * groups;
    const int t = threadIdx.x;
    if (blockIdx.x >= pack_blocks) {
        const int64_t step = (int64_t)(gridDim.x - pack_blocks) * kT;
        const T *W = static_cast<const T *>(a.W), *U = static_cast<const T *>(a.U);
        const int p4 = a.Hk / PER;
        const int64_t total = (int64_t)(a.D + a.H) * 4 * p4;
        for (int64_t id = (int64_t)(blockIdx.x - pack_blocks) * kT + t; id < total; id += step) {
            // consecutive threads take consecutive columns of W / U (rows n of the operand): coalesced reads
            const int n = (int)(id % (a.D + a.H)), q = (int)(id / (a.D + a.H));
            const int g = q / p4, m0 = (q % p4) * PER;
            float v[PER];
#pragma unroll
            for (int e = 0; e < PER; ++e) {
                const int64_t row = (int64_t)g * a.H + m0 + e;
                v[e] = m0 + e >= a.H ? 0.0f : to_f32<T>(n < a.D ? W[row * a.D + n] : U[row * a.H + n - a.D]);
            }
            const u32x4 o = pack_units<T>(v);
            if (n < a.D) store16(a.Wt, n, (int64_t)(g * a.Hk + m0) * sizeof(T), a.w_alloc, o);
            else if (g < 3) store16(a.Ut, n - a.D, (int64_t)(g * a.Hk + m0) * sizeof(T), a.u_alloc, o);
            else store16(a.Uft, n - a.D, (int64_t)m0 * sizeof(T), a.u_alloc, o);
        }
        return;
    }
    const int group = (int)(blockIdx.x % groups), r = (int)(blockIdx.x / groups) * kRows<T> + t / kPieces<T>;
    if (r >= a.n_rows) return;
    const int piece = t % kPieces<T>;
    const int64_t j = r < a.n ? a.perm[r] : 0;
    float v[PER];
    if (group < a.x_groups) {
        const int m0 = group * 64 + piece * PER;
#pragma unroll
        for (int e = 0; e < PER; ++e) v[e] = 0.0f;
        if (r < a.n) {
            if (m0 < a.D) load_units<T, PER, VX>(static_cast<const T *>(a.x) + j * a.D + m0, a.D - m0, v);
#pragma unroll
            for (int e = 0; e < PER; ++e)
                if (m0 + e == a.D) v[e] = 1.0f;
            if (m0 == 0) a.parent_of[j] = -1;
        }
        store16(a.AX, r, (int64_t)m0 * sizeof(T), a.rows_alloc, pack_units<T>(v));
        return;
    }
    const int m0 = (group - a.x_groups) * 64 + piece * PER;
    const T *h = static_cast<const T *>(a.h) + m0;
    const int left = a.H - m0;
    const u32x4 zero = {0, 0, 0, 0};
    u32x4 own = zero;
    if (r < a.n && left > 0) {
        load_units<T, PER, VH>(h + j * a.H, left, v);
        own = pack_units<T>(v);
    }
    store16(a.AH, r, (int64_t)m0 * sizeof(T), a.rows_alloc, own);
    if (r >= a.first) {
        float sum[PER];
#pragma unroll
        for (int e = 0; e < PER; ++e) sum[e] = 0.0f;
        if (r < a.n && left > 0)
            for (int ce = a.child_ptr[j]; ce < a.child_ptr[j + 1]; ++ce) {
                load_units<T, PER, VH>(h + (int64_t)a.child_idx[ce] * a.H, left, v);
#pragma unroll
                for (int e = 0; e < PER; ++e) sum[e] += v[e];
            }
        store16(a.AS, r, (int64_t)m0 * sizeof(T), a.rows_alloc, pack_units<T>(sum));
    }
    if (r >= a.n) {
        for (int g = 0; g < 4; ++g) store16(a.dZ, r, (int64_t)(g * a.Hk + m0) * sizeof(T), a.rows_alloc, zero);
        store16(a.G, r, (int64_t)m0 * sizeof(T), a.rows_alloc, zero);
    }
}

// ---- the cell's elementwise derivative ------------------------------------------------------
// What node j receives is fetched here, by node id, from what its parent p left in a higher level (total dc_p, dhs_p =
// U_iou^T dz_iou,p):
//     dh_j = gh_j + dhs_p + ufg_r      ufg (level order) = U_f^T dz_f,j, from the product before this kernel
//     dc_j = gc_j + dc_p f_j + dh_j o_j (1 - tanh^2 c_j)
// Every child k of j gets its dz_f,k = dc_j c_k f_k (1 - f_k) written to row inv_perm[k] of G; a root writes its own row of
// zeros.  Row r of dZ = [dz_i | dz_o | dz_u | sum_k dz_f,k]; a leaf's forget block is written only where something reads
// it (zero_forget).  dc_j stays in dc[j] for the children's level.
// Bound by memory: 36 bytes a unit of the node (bf16, with gh) and 8 per child, read and written in 16-byte pieces: 591 k
// leaves, H = 512: 1.96 ms (4.6 TB/s), all 15 levels of 1.18 M nodes 5.9 ms (8.0 one unit a lane and dZ written twice).
// Few rows: bound by the chain node -> children -> their rows, so four children's rows are in flight and the next four's ids.
// Whole backward pass, two children at a time and ids on demand (four in fp32) -> so: one node with 40 k children, H 512, bf16
// 59.6 -> 45.0 ms, 60 nodes with 400, H 256, bf16 1.24 -> 0.88; 4.7 k nodes of trees, H 150, fp32 0.239 -> 0.229.
struct CellArgs {
    const int32_t *perm, *inv_perm, *child_ptr, *child_idx;
    int32_t *parent_of;
    const float *c, *gh, *gc;
    const void *gates, *fgate, *dhs, *ufg;
    float *dc;
    void *dZ, *G;
    int64_t rows_alloc;
    int row0, n_rows, H, Hk, zero_forget;      // the level's rows are positions row0 .. row0 + n_rows
};
constexpr int kKidsAhead = 4;
template <typename T, bool VEC, bool LEAVES>
__global__ void __launch_bounds__(kT)
bwd_cell_kernel(const CellArgs a) {
    constexpr int PER = kPer<T>;
    const int t = threadIdx.x;
    const int i = blockIdx.x * kRows<T> + t / kPieces<T>;          // row of the level
    if (i >= a.n_rows) return;
    const int m0 = blockIdx.y * 64 + (t % kPieces<T>) * PER, left = a.H - m0;
    const int64_t r = a.row0 + i, j = a.perm[r];
    const int64_t p = a.parent_of[j];
    const int kid0 = LEAVES ? 0 : a.child_ptr[j], kid1 = LEAVES ? 0 : a.child_ptr[j + 1];
    const int64_t kb = (int64_t)m0 * sizeof(T), gate_kb = (int64_t)a.Hk * sizeof(T);
    const u32x4 zero = {0, 0, 0, 0};
    const int64_t at = j * a.H + m0;
    float dh[PER], dcj[PER], dzf[PER];
#pragma unroll
    for (int e = 0; e < PER; ++e) dh[e] = dcj[e] = dzf[e] = 0.0f;
    if (left > 0) {
        float v[PER], w[PER], o[PER], cj[PER];
        load_units<T, PER, VEC>(static_cast<const T *>(a.gates) + j * 3 * a.H + a.H + m0, left, o);
        load_units<float, PER, true>(a.c + at, left, cj);
        if (a.gh) load_units<float, PER, true>(a.gh + at, left, dh);
        if (a.gc) load_units<float, PER, true>(a.gc + at, left, dcj);
        if (p >= 0) {
            load_units<T, PER, VEC>(static_cast<const T *>(a.ufg) + (int64_t)i * a.H + m0, left, v);
            load_units<T, PER, VEC>(static_cast<const T *>(a.dhs) + p * a.H + m0, left, w);
#pragma unroll
            for (int e = 0; e < PER; ++e) dh[e] = dh[e] + v[e] + w[e];
            load_units<T, PER, VEC>(static_cast<const T *>(a.fgate) + at, left, v);
            load_units<float, PER, true>(a.dc + p * a.H + m0, left, w);
#pragma unroll
            for (int e = 0; e < PER; ++e) dcj[e] += w[e] * v[e];
        }
        float dzo[PER];
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            const float th = tanhf(cj[e]);
            dcj[e] += dh[e] * o[e] * (1.0f - th * th);
            dzo[e] = dh[e] * th * o[e] * (1.0f - o[e]);
        }
        store16(a.dZ, r, gate_kb + kb, a.rows_alloc, pack_units<T>(dzo));
        load_units<T, PER, VEC>(static_cast<const T *>(a.gates) + j * 3 * a.H + m0, left, v);
        load_units<T, PER, VEC>(static_cast<const T *>(a.gates) + j * 3 * a.H + 2 * a.H + m0, left, w);
        float dzi[PER], dzu[PER];
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            dzi[e] = dcj[e] * w[e] * v[e] * (1.0f - v[e]);
            dzu[e] = dcj[e] * v[e] * (1.0f - w[e] * w[e]);
        }
        store16(a.dZ, r, kb, a.rows_alloc, pack_units<T>(dzi));
        store16(a.dZ, r, 2 * gate_kb + kb, a.rows_alloc, pack_units<T>(dzu));
        if (!LEAVES) {      // the children's level reads it
            if (left >= PER) {
                typedef u32x4 __attribute__((aligned(4))) u32x4a;
#pragma unroll
                for (int q = 0; q < PER / 4; ++q) {
                    const u32x4 b = {__float_as_uint(dcj[4 * q]), __float_as_uint(dcj[4 * q + 1]), __float_as_uint(dcj[4 * q + 2]), __float_as_uint(dcj[4 * q + 3])};
                    reinterpret_cast<u32x4a *>(a.dc + at)[q] = b;
                }
            } else {
#pragma unroll
                for (int e = 0; e < PER; ++e)
                    if (e < left) a.dc[at + e] = dcj[e];
            }
        }
    } else {
#pragma unroll
        for (int g = 0; g < 3; ++g) store16(a.dZ, r, g * gate_kb + kb, a.rows_alloc, zero);
    }
    if (!LEAVES) {
        // kKidsAhead children at a time: their rows and the next ones' ids, then their arithmetic (the last one's again past the end)
        constexpr int K = kKidsAhead;
        int kid[K];
#pragma unroll
        for (int q = 0; q < K; ++q) kid[q] = a.child_idx[kid0 + q < kid1 ? kid0 + q : kid1 - 1];
        for (int ce = kid0; ce < kid1; ce += K) {
            int next[K];
            float fk[K][PER], ck[K][PER];
            int pos[K];
#pragma unroll
            for (int q = 0; q < K; ++q) next[q] = a.child_idx[ce + K + q < kid1 ? ce + K + q : kid1 - 1];
#pragma unroll
            for (int q = 0; q < K; ++q) {
                pos[q] = a.inv_perm[kid[q]];
#pragma unroll
                for (int e = 0; e < PER; ++e) fk[q][e] = ck[q][e] = 0.0f;
                if (left > 0) {
                    load_units<T, PER, VEC>(static_cast<const T *>(a.fgate) + (int64_t)kid[q] * a.H + m0, left, fk[q]);
                    load_units<float, PER, true>(a.c + (int64_t)kid[q] * a.H + m0, left, ck[q]);
                }
            }
#pragma unroll
            for (int q = 0; q < K; ++q) {
                if (ce + q >= kid1) break;
#pragma unroll
                for (int e = 0; e < PER; ++e) {
                    ck[q][e] = dcj[e] * ck[q][e] * fk[q][e] * (1.0f - fk[q][e]);
                    dzf[e] += ck[q][e];
                }
                store16(a.G, pos[q], kb, a.rows_alloc, pack_units<T>(ck[q]));
                if (m0 == 0) a.parent_of[kid[q]] = (int32_t)j;
            }
#pragma unroll
            for (int q = 0; q < K; ++q) kid[q] = next[q];
        }
    }
    if (!LEAVES || a.zero_forget) store16(a.dZ, r, 3 * gate_kb + kb, a.rows_alloc, pack_units<T>(dzf));
    if (p < 0) store16(a.G, r, kb, a.rows_alloc, zero);
}

// ---- data gradients: rows of nodes times a weight operand -----------------------------------
// C [node row, feature] = A [node rows, K] B [features, K]^T, both K-blocked.  out row = map ? map[row] : row.
struct RowProduct {
    const char *A; int n_rows;
    const char *B; int64_t b_alloc; int n_feat;
    int n_slabs;                   // 64-byte slabs of K
    void *out; const int32_t *map; int ld; int f32_out;
};
template <typename T>
__device__ __forceinline__ void store4(const RowProduct &g, int64_t row, int feat, const float (&v)[4], bool vec) {
    const int64_t at = row * g.ld + feat;
    if (g.f32_out || sizeof(T) == 4) {
        float *o = static_cast<float *>(g.out) + at;
        if (vec && feat + 4 <= g.n_feat) *reinterpret_cast<float4 *>(o) = make_float4(v[0], v[1], v[2], v[3]);
        else
            for (int e = 0; e < 4; ++e)
                if (feat + e < g.n_feat) o[e] = v[e];
    } else {
        T *o = static_cast<T *>(g.out) + at;
        if (vec && feat + 4 <= g.n_feat) {
            const u32x2 b = {(uint32_t)f32_to_bf16(v[0]) | ((uint32_t)f32_to_bf16(v[1]) << 16),
                             (uint32_t)f32_to_bf16(v[2]) | ((uint32_t)f32_to_bf16(v[3]) << 16)};
            *reinterpret_cast<u32x2 *>(o) = b;
        } else
            for (int e = 0; e < 4; ++e)
                if (feat + e < g.n_feat) o[e] = from_f32<T>(v[e]);
    }
}

// Many rows (kTileMinBlocks tiles; 188 of them took 35 us, the thin kernel 56): the 128 x 256 tiles of the level kernel, features as the tile's rows and nodes as its columns (300 features
// pad to 384 that way, not to 512), so that a lane ends up with four consecutive features of one node.
template <typename T>
__global__ void __launch_bounds__(kDmaThreads, 2)
rows_tile_kernel(LevelArgs a, const RowProduct g) {
    __shared__ __attribute__((aligned(1024))) char lds[kDmaBufs * kDmaBuf];
    __shared__ __attribute__((aligned(256))) char sink[4 * 256];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1, hf = lane >> 5, l32 = lane & 31;
    int row_tile, col_tile;
    if (!block_to_tile(blockIdx.x, a.n_col_tiles, a.n_row_tiles, col_tile, row_tile)) return;
    floatx16 acc[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][q][v] = 0.0f;
    __shared__ int s_row[kBN];
    {
        const int row = col_tile * kBN + (int)threadIdx.x;
        s_row[threadIdx.x] = row >= g.n_rows ? -1 : g.map ? g.map[row] : row;
    }
    dma_gemm<T, MODE_SWAP>(a, lds, nullptr, row_tile * kDmaBM, col_tile, acc, sink, []() {});
    const int step = g.f32_out || sizeof(T) == 4 ? 16 : 8;
    const bool vec = (g.ld & 3) == 0 && (reinterpret_cast<uintptr_t>(g.out) & (step - 1)) == 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int row = s_row[wn * 128 + q * 32 + l32];
        if (row < 0) continue;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int feat = row_tile * kDmaBM + wm * 64 + i * 32 + v * 8 + hf * 4;
                if (feat >= g.n_feat) continue;
                const float four[4] = {acc[i][q][4 * v], acc[i][q][4 * v + 1], acc[i][q][4 * v + 2], acc[i][q][4 * v + 3]};
                store4<T>(g, row, feat, four, vec);
            }
    }
}

// Few rows: 16 RT rows x 16 CT features in a block, K dealt to its four waves in slabs, fragments straight from L2 (16 rows x
// 64 bytes are 1 KB of consecutive memory), partial sums added through LDS.  Two products share a launch (a level's dhs and
// the next level's ufg).  Bound by the latency of a wave's slabs, so small tiles (16 x 32) until they fill the chip.
struct ThinArgs {
    RowProduct g[2];
    int64_t rows_alloc;
    int blocks0;                   // blocks of the first product
};
template <typename T, int RT, int CT>
__global__ void __launch_bounds__(kT)
rows_thin_kernel(const ThinArgs a) {
    constexpr int kStride = 16 * CT + 4;
    __shared__ __attribute__((aligned(16))) float part[4][16 * RT * kStride];
    const bool second = (int)blockIdx.x >= a.blocks0;
    const RowProduct &g = a.g[second ? 1 : 0];
    const int b = (int)blockIdx.x - (second ? a.blocks0 : 0);
    const int col_tiles = (g.n_feat + 16 * CT - 1) / (16 * CT);
    const int row0 = b / col_tiles * 16 * RT, col0 = b % col_tiles * 16 * CT;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    floatx4 acc[RT][CT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[i][c] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    const int64_t lane_off = (lane & 15) * 64 + (lane >> 4) * 16;
    const char *pa = g.A + (int64_t)row0 * 64 + lane_off, *pb = g.B + (int64_t)col0 * 64 + lane_off;
    const int64_t a_slab = a.rows_alloc * 64, b_slab = g.b_alloc * 64;
    struct Frags { u32x4 a[RT], b[CT]; };
    auto load = [&](int s, Frags &f) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < CT; ++c) f.b[c] = *reinterpret_cast<const u32x4 *>(pb + s * b_slab + c * 1024);
#pragma unroll
        for (int i = 0; i < RT; ++i) f.a[i] = *reinterpret_cast<const u32x4 *>(pa + s * a_slab + i * 1024);
    };
    auto multiply = [&](const Frags &f) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int c = 0; c < CT; ++c) mfma16<T>(f.a[i], f.b[c], acc[i][c]);
    };
    Frags F[3];                                     // three slabs in flight
    const int n = g.n_slabs;
#pragma unroll
    for (int q = 0; q < 3; ++q)
        if (wave + 4 * q < n) load(wave + 4 * q, F[q]);
    for (int s = wave; s < n; s += 12) {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            if (s + 4 * q < n) multiply(F[q]);
            if (s + 4 * q + 12 < n) load(s + 4 * q + 12, F[q]);
        }
    }
    const int u = lane & 15;
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int v = 0; v < 4; ++v) part[wave][(i * 16 + (lane >> 4) * 4 + v) * kStride + c * 16 + u] = acc[i][c][v];
    __syncthreads();
    const int step = g.f32_out || sizeof(T) == 4 ? 16 : 8;
    const bool vec = (g.ld & 3) == 0 && (reinterpret_cast<uintptr_t>(g.out) & (step - 1)) == 0;
    for (int q = threadIdx.x; q < 16 * RT * 4 * CT; q += kT) {
        const int i = q / (4 * CT), c = q % (4 * CT) * 4;
        if (row0 + i >= g.n_rows || col0 + c >= g.n_feat) continue;
        float four[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int w = 0; w < 4; ++w)
#pragma unroll
            for (int e = 0; e < 4; ++e) four[e] += part[w][i * kStride + c + e];
        store4<T>(g, g.map ? g.map[row0 + i] : row0 + i, col0 + c, four, vec);
    }
}

// ---- weight gradients: sums over the nodes --------------------------------------------------
// Up to three products A^T B over rows [begin, n_rows) of K-blocked operands, cut into 128 x 256 tiles and `splits` ranges of
// rows_per_split rows.  Bound by the matrix cores and LDS reads (fragments are read transposed at the rate of the plain ones):
// 1.18 M nodes, D = 300, H = 512, bf16: 3.6 ms, 890 TFLOP/s of padded tiles.  A block leaves its tile of partial sums in register order (whole 1 KB stores); grad_reduce_kernel adds
// the ranges in order, so the result does not depend on timing.  Blocks of one range run on one XCD (b % 8), whose L2 then
// reads that range of every operand once.
struct TnProblem {
    const char *A, *B;
    int m_tiles, n_tiles;
    int tile0;                 // index of its first tile
    int begin, begin_f;        // first row of the reduction, a multiple of 64; of the tiles from column tile f_tile on
    int shift, shift_f;        // 0 .. 63, added to all rows: sums over the inner nodes start exactly at the first of them
    int f_tile;
};
struct TnArgs {
    TnProblem p[3];
    int64_t rows_alloc;
    int n_rows, rows_per_split, splits, tiles;
    float *partial;
    float *dW, *dU, *db;
    int D, H, Hk;
};
__device__ __forceinline__ int tn_decode(const TnArgs &a, int tile, int &m, int &n, int &begin, int &shift) {
    const int q = tile >= a.p[2].tile0 ? 2 : tile >= a.p[1].tile0 ? 1 : 0;
    const TnProblem &p = a.p[q];
    m = (tile - p.tile0) / p.n_tiles;
    n = (tile - p.tile0) % p.n_tiles;
    begin = n >= p.f_tile ? p.begin_f : p.begin;
    shift = n >= p.f_tile ? p.shift_f : p.shift;
    return q;
}
template <typename T>
__global__ void __launch_bounds__(kDmaThreads, 2)
tn_kernel(const TnArgs e) {
    __shared__ __attribute__((aligned(1024))) char lds[kDmaBufs * kDmaBuf];
    const int q = blockIdx.x >> 3, split = (blockIdx.x & 7) + 8 * (q / e.tiles), tile = q % e.tiles;
    if (split >= e.splits) return;
    int mt, nt, begin, shift;
    const int which = tn_decode(e, tile, mt, nt, begin, shift);
    int k0 = split * e.rows_per_split, k1 = k0 + e.rows_per_split;
    if (k0 < begin) k0 = begin;
    if (k1 > e.n_rows) k1 = e.n_rows;
    if (k0 >= k1) return;
    k0 += shift;
    k1 += shift;
    constexpr int ESZ = (int)sizeof(T);
    LevelArgs a = {};
    a.n_rows_alloc = (int)e.rows_alloc;
    a.NPU = (int)e.rows_alloc;
    a.stack = e.p[which].A + (int64_t)(mt * 128 * ESZ / 64) * e.rows_alloc * 64 + (int64_t)k0 * 64;
    a.Bp = e.p[which].B + (int64_t)(nt * 256 * ESZ / 64) * e.rows_alloc * 64 + (int64_t)k0 * 64;
    a.Dp = (k1 - k0) / (64 / ESZ) * kDmaStage / ESZ;         // stages of 64 / ESZ rows
    floatx16 acc[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][g][v] = 0.0f;
    dma_gemm<T, MODE_TN>(a, lds, nullptr, 0, 0, acc, nullptr, []() {});
    float4 *out = reinterpret_cast<float4 *>(e.partial + ((int64_t)split * e.tiles + tile) * (128 * 256)) + threadIdx.x;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                out[((i * 4 + g) * 4 + v) * kDmaThreads] = make_float4(acc[i][g][4 * v], acc[i][g][4 * v + 1], acc[i][g][4 * v + 2], acc[i][g][4 * v + 3]);
}

__global__ void __launch_bounds__(kT)
grad_reduce_kernel(const TnArgs e) {
    const int tile = blockIdx.x >> 5, rest = blockIdx.x & 31, t = threadIdx.x;      // (widest cells: more tiles than a grid has rows)
    int mt, nt, begin, shift;
    const int which = tn_decode(e, tile, mt, nt, begin, shift);
    const int lane = t & 63, wave = t >> 6, i = rest >> 4, g = (rest >> 2) & 3, v = rest & 3;
    const int m = mt * 128 + (wave >> 1) * 64 + i * 32 + v * 8 + (lane >> 5) * 4;
    const int n = nt * 256 + (wave & 1) * 128 + g * 32 + (lane & 31);
    const int gate = which == 2 ? 3 : n / e.Hk, u = which == 2 ? n : n % e.Hk;
    const int width = which == 0 ? e.D + 1 : e.H;
    if (m >= width || u >= e.H || gate > 3 || (which == 1 && gate == 3)) return;
    const float4 *in = reinterpret_cast<const float4 *>(e.partial + (int64_t)tile * (128 * 256)) + rest * kT + t;
    float4 s = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (begin < e.n_rows)
#pragma unroll 4
        for (int k = begin / e.rows_per_split; k < e.splits; ++k) {
            const float4 p = in[(int64_t)k * e.tiles * (128 * 256 / 4)];
            s.x += p.x; s.y += p.y; s.z += p.z; s.w += p.w;
        }
    const int64_t row = (int64_t)gate * e.H + u;
    const int ld = which == 0 ? e.D : e.H;
    float *o = (which == 0 ? e.dW : e.dU) + row * ld + m;
    if ((ld & 3) == 0 && m + 4 <= ld && (reinterpret_cast<uintptr_t>(o) & 15) == 0) {
        *reinterpret_cast<float4 *>(o) = s;
    } else {
        const float four[4] = {s.x, s.y, s.z, s.w};
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            if (m + x < ld) o[x] = four[x];
            else if (m + x == ld && which == 0) e.db[row] = four[x];
        }
        return;
    }
    // (a vector store never covers column D: m + 4 <= D)
}

// ---- workspace ---------------------------------------------------------------------
struct BwdDims {
    int D, H, Hk;         // Hk: H rounded up to 64 elements (whole stages of the tiled GEMM)
    int n_max;            // largest level
    size_t esz;
};
struct BwdWs {
    float *dc, *partial;
    void *dhs, *ufg;      // in the operands' element type
    int32_t *parent_of;
    void *Wt, *Ut, *Uft, *dZ, *G, *AX, *AH, *AS;
    int64_t rows_alloc, w_alloc, u_alloc;
    size_t bytes;
};

// How the sums over nodes are cut: as many ranges as give every compute unit two blocks, but no range under kMinSplitRows rows
// (each costs 128 KB of partial sums a tile).  Long sums are cut eight times finer: the ranges, dealt whole to the XCDs, then
// come out even (13 ranges of 90 k rows: 5.4 ms, two on five of the XCDs and one on the others).  Long from 4 x 4096 rows on;
// backward pass, ms, with 2048 / 4096 / 8192 there: 577 k nodes H 300 fp32 20.2 / 20.2 / 25.5, bf16 5.84 / 5.83 / 6.11; 286 k
// nodes H 512 fp32 16.8 / 16.7 / 21.0.
constexpr int kMinSplitRows = 128, kLongSplitRows = 4096;
// Sums over the inner nodes alone (dU_iou, dW_f) start at the first of them, not at the 64 rows it lies in: a leaf has no part
// in them, but its zero child sum times an infinite dz would be NaN.  Their ranges are those of all nodes, moved up by less
// than 64 rows, into zero rows at the end.
struct TnPlan { int tiles[3], begin[3], shift, f_tile, rows, rows_per_split, splits, total_tiles, leaf_tiles; };
TnPlan plan_tn(int64_t n, int64_t first_internal, const BwdDims &d) {
    TnPlan p = {};
    p.rows = n > 0 ? (int)round_up(n, 64) : 64;
    const int fi = (int)(first_internal / 64 * 64), n4 = 4 * d.Hk / 256;
    p.begin[1] = fi;
    p.shift = (int)(first_internal - fi);
    // the column tiles that hold nothing but the forget gate
    p.f_tile = 3 * d.Hk % 256 == 0 ? 3 * d.Hk / 256 : n4;
    const int mx = (int)ceil_div(d.D + 1, 128), mh = (int)ceil_div(d.H, 128);
    p.tiles[0] = mx * n4;
    p.tiles[1] = mh * (int)ceil_div(3 * d.Hk, 256);
    p.tiles[2] = mh * (int)ceil_div(d.Hk, 256);
    p.total_tiles = p.tiles[0] + p.tiles[1] + p.tiles[2];
    const int f_tiles = mx * (n4 - p.f_tile);
    p.leaf_tiles = p.tiles[0] - f_tiles + p.tiles[2];          // tiles that sum over the leaves too
    const int64_t work = (int64_t)p.leaf_tiles * p.rows + (int64_t)(p.tiles[1] + f_tiles) * (p.rows - fi);
    int64_t rps = round_up(ceil_div(work, 512), 64);
    if (rps >= 4 * kLongSplitRows) rps = round_up(rps / 8, 64);
    if (rps < kMinSplitRows) rps = kMinSplitRows;
    if (rps > p.rows) rps = p.rows;
    p.rows_per_split = (int)rps;
    p.splits = (int)ceil_div(p.rows, rps);
    return p;
}

// Room for the partial sums: no fewer ranges than plan_tn can make of n nodes, whichever of them are leaves, and no fewer than
// it makes of a smaller forest.  Leaves alone are the least work, so a range holds at least that work / 512 (long sums: / 4096)
// and kMinSplitRows (kLongSplitRows / 2) rows.
int64_t max_splits(int64_t n, const BwdDims &d) {
    const TnPlan p = plan_tn(n, n, d);
    const int64_t t = p.leaf_tiles, rows = p.rows;
    const int64_t lng = std::min(ceil_div(8 * 512, t), ceil_div(rows, kLongSplitRows / 2));
    return std::min(ceil_div(rows, kMinSplitRows), std::max(ceil_div(512, t), lng));
}

BwdWs carve_bwd_ws(int64_t n, const BwdDims &d, void *base) {
    Carver c(base);
    BwdWs w;
    w.rows_alloc = round_up(n, 64) + 256;             // whole tiles of 256 rows are read from any row on
    w.w_alloc = round_up(d.D, 256); w.u_alloc = round_up(d.H, 256);
    const size_t row = (size_t)w.rows_alloc * d.esz;
    w.dc = c.take<float>((size_t)n * d.H);
    w.dhs = c.take<char>((size_t)n * d.H * d.esz);
    w.ufg = c.take<char>((size_t)d.n_max * d.H * d.esz);
    w.parent_of = c.take<int32_t>((size_t)n);
    w.Wt = c.take<char>((size_t)w.w_alloc * 4 * d.Hk * d.esz);
    w.Ut = c.take<char>((size_t)w.u_alloc * 3 * d.Hk * d.esz);
    w.Uft = c.take<char>((size_t)w.u_alloc * d.Hk * d.esz);
    // whole tiles of columns are read: 128 of the left operands, 256 of the right ones
    w.dZ = c.take<char>(row * round_up(4 * d.Hk, 256));
    w.G = c.take<char>(row * round_up(d.Hk, 256));
    w.AX = c.take<char>(row * round_up(d.D + 1, 128));
    w.AH = c.take<char>(row * round_up(d.H, 128));
    w.AS = c.take<char>(row * round_up(d.H, 128));
    w.partial = c.take<float>((size_t)max_splits(n, d) * plan_tn(n, n, d).total_tiles * 128 * 256);
    w.bytes = c.off;
    return w;
}

// Half the compute units.  Backward pass, us, from 64 / 128 / 256 tiles on: 26 k nodes H 150 fp32 810 / 767 / 737, bf16 408 / 409 /
// 392; 72 k nodes H 512 fp32 5933 / 5686 / 5717, bf16 1267 / 1257 / 1297; 143 k nodes H 256 fp32 4428 / 4308 / 4312.
constexpr int kTileMinBlocks = 128;
template <typename T>
int launch_rows(const RowProduct *g, int n_products, int64_t rows_alloc, hipStream_t st) {
    RowProduct todo[2];
    int m = 0;
    for (int q = 0; q < n_products; ++q)
        if (g[q].n_rows > 0 && g[q].n_feat > 0) todo[m++] = g[q];
    // enough 128 x 256 tiles for the chip: the tile kernel
    int thin = 0;
    for (int q = 0; q < m; ++q) {
        const int64_t ft = ceil_div(todo[q].n_feat, 128), rt = ceil_div(todo[q].n_rows, kBN);
        if (ft * rt < kTileMinBlocks) { todo[thin++] = todo[q]; continue; }
        LevelArgs a = {};
        a.stack = todo[q].B; a.n_rows_alloc = (int)todo[q].b_alloc;
        a.Bp = todo[q].A; a.NPU = (int)rows_alloc;
        a.Dp = todo[q].n_slabs * kDmaStage / (int)sizeof(T);
        a.n_row_tiles = (int)ft; a.n_col_tiles = (int)rt;
        rows_tile_kernel<T><<<(unsigned)(8 * ceil_div(rt, 8) * ft), kDmaThreads, 0, st>>>(a, todo[q]);
        JITDB_LAUNCH_CHECK();
    }
    if (thin == 0) return JITDB_OK;
    ThinArgs t = {};
    t.rows_alloc = rows_alloc;
    auto blocks = [&](const RowProduct &p, int rows, int cols) { return (int)(ceil_div(p.n_rows, rows) * ceil_div(p.n_feat, cols)); };
    int big = 0;
    for (int q = 0; q < thin; ++q) { t.g[q] = todo[q]; big += blocks(todo[q], 32, 64); }
    const bool small = big < 2 * 256;
    t.blocks0 = small ? blocks(t.g[0], 16, 32) : blocks(t.g[0], 32, 64);
    int all = t.blocks0;
    if (thin == 2) all += small ? blocks(t.g[1], 16, 32) : blocks(t.g[1], 32, 64);
    if (small) rows_thin_kernel<T, 1, 2><<<(unsigned)all, kT, 0, st>>>(t);
    else rows_thin_kernel<T, 2, 4><<<(unsigned)all, kT, 0, st>>>(t);
    JITDB_LAUNCH_CHECK();
    return JITDB_OK;
}

template <typename T>
int run_backward(const T *x, const T *W, const T *U, const BwdDims &d, const jitdb_schedule_t *s,
                 const T *h, const float *c, const T *gates, const T *fgate,
                 const float *gh, const float *gc, float *dx, float *dW, float *dU, float *db,
                 const BwdWs &w, hipStream_t st) {
    const int n = (int)s->n_nodes;
    const int L = s->n_levels;
    const int32_t *lp = s->host_level_ptr;
    const int D = d.D, H = d.H, Hk = d.Hk;
    for (int l = 0; l < L; ++l)
        if (lp[l + 1] <= lp[l]) return JITDB_E_SCHEDULE;
    int rc;
    const TnPlan plan = plan_tn(n, lp[1], d);
    {
        PrepArgs a = {};
        a.x = x; a.h = h; a.W = W; a.U = U; a.perm = s->perm; a.child_ptr = s->child_ptr; a.child_idx = s->child_idx;
        a.parent_of = w.parent_of; a.AX = w.AX; a.AH = w.AH; a.AS = w.AS; a.dZ = w.dZ; a.G = w.G; a.Wt = w.Wt; a.Ut = w.Ut; a.Uft = w.Uft;
        a.D = D; a.H = H; a.Hk = Hk; a.n = n; a.n_rows = plan.rows + plan.shift; a.first = lp[1];
        a.rows_alloc = w.rows_alloc; a.w_alloc = w.w_alloc; a.u_alloc = w.u_alloc;
        a.x_groups = (int)ceil_div(D + 1, 64); a.h_groups = Hk / 64; a.row_blocks = (int)ceil_div(a.n_rows, kRows<T>);
        const int64_t w_blocks = ceil_div((int64_t)(D + H) * 4 * (Hk / kPer<T>), kT);
        const dim3 grid((unsigned)((int64_t)a.row_blocks * (a.x_groups + a.h_groups) + (w_blocks < 1024 ? w_blocks : 1024)));
        const bool vx = D * sizeof(T) % 4 == 0, vh = H * sizeof(T) % 4 == 0;
        if (vx && vh) bwd_prepare_kernel<T, true, true><<<grid, kT, 0, st>>>(a);
        else if (vx) bwd_prepare_kernel<T, true, false><<<grid, kT, 0, st>>>(a);
        else if (vh) bwd_prepare_kernel<T, false, true><<<grid, kT, 0, st>>>(a);
        else bwd_prepare_kernel<T, false, false><<<grid, kT, 0, st>>>(a);
        JITDB_LAUNCH_CHECK();
    }
    const int slabs = Hk * (int)sizeof(T) / 64;             // of one gate
    auto rows_at = [](void *base, int row) { return static_cast<const char *>(base) + (int64_t)row * 64; };
    CellArgs a = {};
    a.perm = s->perm; a.inv_perm = s->inv_perm; a.child_ptr = s->child_ptr; a.child_idx = s->child_idx; a.parent_of = w.parent_of;
    a.c = c; a.gh = gh; a.gc = gc; a.gates = gates; a.fgate = fgate; a.dhs = w.dhs; a.ufg = w.ufg; a.dc = w.dc; a.dZ = w.dZ; a.G = w.G;
    a.rows_alloc = w.rows_alloc; a.H = H; a.Hk = Hk;
    // a leaf's forget block is read where a column tile of the sums holds other gates too
    a.zero_forget = plan.f_tile * 256 != 3 * Hk;
    const bool vec = H * sizeof(T) % 4 == 0 && ((reinterpret_cast<uintptr_t>(gates) | reinterpret_cast<uintptr_t>(fgate)) & 3) == 0;
    for (int l = L - 1; l >= 0; --l) {
        a.row0 = lp[l]; a.n_rows = lp[l + 1] - lp[l];
        const dim3 grid((unsigned)ceil_div(a.n_rows, kRows<T>), (unsigned)(Hk / 64));
        if (l == 0) {
            if (vec) bwd_cell_kernel<T, true, true><<<grid, kT, 0, st>>>(a);
            else bwd_cell_kernel<T, false, true><<<grid, kT, 0, st>>>(a);
        } else {
            if (vec) bwd_cell_kernel<T, true, false><<<grid, kT, 0, st>>>(a);
            else bwd_cell_kernel<T, false, false><<<grid, kT, 0, st>>>(a);
        }
        JITDB_LAUNCH_CHECK();
        if (l == 0) break;
        RowProduct g[2] = {};
        g[0].A = rows_at(w.dZ, lp[l]); g[0].n_rows = a.n_rows; g[0].n_slabs = 3 * slabs;
        g[0].B = static_cast<const char *>(w.Ut); g[0].out = w.dhs; g[0].map = s->perm + lp[l];
        g[1].A = rows_at(w.G, lp[l - 1]); g[1].n_rows = lp[l] - lp[l - 1]; g[1].n_slabs = slabs;
        g[1].B = static_cast<const char *>(w.Uft); g[1].out = w.ufg;
        for (RowProduct &p : g) { p.b_alloc = w.u_alloc; p.n_feat = H; p.ld = H; }
        if ((rc = launch_rows<T>(g, 2, w.rows_alloc, st)) != JITDB_OK) return rc;
    }
    {
        RowProduct g[2] = {};
        for (int q = 0; q < 2; ++q) {
            const int r0 = q ? lp[1] : 0, r1 = q ? n : lp[1];
            g[q].A = rows_at(w.dZ, r0); g[q].n_rows = r1 - r0; g[q].n_slabs = (q ? 4 : 3) * slabs;
            g[q].B = static_cast<const char *>(w.Wt); g[q].b_alloc = w.w_alloc; g[q].n_feat = D;
            g[q].out = dx; g[q].map = s->perm + r0; g[q].ld = D; g[q].f32_out = 1;
        }
        if ((rc = launch_rows<T>(g, 2, w.rows_alloc, st)) != JITDB_OK) return rc;
    }
    TnArgs e = {};
    const void *A[3] = {w.AX, w.AS, w.AH}, *B[3] = {w.dZ, w.dZ, w.G};
    for (int q = 0, at = 0; q < 3; ++q) {
        TnProblem &p = e.p[q];
        p.A = static_cast<const char *>(A[q]); p.B = static_cast<const char *>(B[q]);
        p.m_tiles = (int)ceil_div(q == 0 ? D + 1 : H, 128); p.n_tiles = plan.tiles[q] / p.m_tiles;
        p.tile0 = at; p.begin = plan.begin[q]; p.begin_f = q == 0 ? plan.begin[1] : plan.begin[q];
        p.shift = q == 1 ? plan.shift : 0; p.shift_f = plan.shift;
        p.f_tile = q == 0 ? plan.f_tile : p.n_tiles;
        at += plan.tiles[q];
    }
    e.rows_alloc = w.rows_alloc; e.n_rows = plan.rows; e.rows_per_split = plan.rows_per_split; e.splits = plan.splits;
    e.tiles = plan.total_tiles; e.partial = w.partial; e.dW = dW; e.dU = dU; e.db = db; e.D = D; e.H = H; e.Hk = Hk;
    tn_kernel<T><<<(unsigned)(8 * ceil_div(e.splits, 8) * e.tiles), kDmaThreads, 0, st>>>(e);
    JITDB_LAUNCH_CHECK();
    grad_reduce_kernel<<<32u * (unsigned)e.tiles, kT, 0, st>>>(e);
    JITDB_LAUNCH_CHECK();
    return JITDB_OK;
}

bool bwd_dims(const jitdb_schedule_t *s, int32_t D, int32_t H, jitdb_dtype dtype, BwdDims &d) {
    if (!s || s->n_nodes < 0 || s->n_nodes > JITDB_MAX_NODES) return false;
    if (D < 1 || D > (1 << 16) || H < 1 || H > (1 << 14)) return false;
    if (dtype != JITDB_F32 && dtype != JITDB_BF16) return false;
    d.D = D; d.H = H; d.Hk = (int)round_up(H, 64);
    d.esz = dtype == JITDB_F32 ? 4 : 2;
    int n_max = 1;
    if (s->host_level_ptr)
        for (int l = 0; l < s->n_levels; ++l) {
            const int r = s->host_level_ptr[l + 1] - s->host_level_ptr[l];
            if (r > n_max) n_max = r;
        }
    d.n_max = n_max;
    return true;
}

}  // namespace
}  // namespace jitdb

using namespace jitdb;

extern "C" size_t jitdb_treelstm_backward_workspace_bytes(const jitdb_schedule_t *s, int32_t D, int32_t H,
                                                          jitdb_dtype dtype) {
    BwdDims d;
    if (!bwd_dims(s, D, H, dtype, d)) return 0;
    return carve_bwd_ws(s->n_nodes, d, nullptr).bytes;
}

extern "C" int jitdb_treelstm_backward(const void *x, const void *W, const void *U,
                                       int32_t D, int32_t H, jitdb_dtype dtype, const jitdb_schedule_t *s,
                                       const void *h, const float *c, const void *gates, const void *fgate,
                                       const float *gh, const float *gc,
                                       float *dx, float *dW, float *dU, float *db,
                                       void *workspace, size_t workspace_bytes, void *hip_stream) {
    if (!s) return JITDB_E_NULL;
    drop_stale_hip_error();
    BwdDims d;
    if (!bwd_dims(s, D, H, dtype, d)) return JITDB_E_BADARG;
    if (!W || !U || !dW || !dU || !db) return JITDB_E_NULL;
    const int64_t n = s->n_nodes;
    hipStream_t st = (hipStream_t)hip_stream;
    if (n == 0) {
        fill_f32_kernel<<<256, kT, 0, st>>>(dW, (int64_t)4 * H * D, 0.0f);
        JITDB_LAUNCH_CHECK();
        fill_f32_kernel<<<256, kT, 0, st>>>(dU, (int64_t)4 * H * H, 0.0f);
        JITDB_LAUNCH_CHECK();
        fill_f32_kernel<<<1, kT, 0, st>>>(db, (int64_t)4 * H, 0.0f);
        JITDB_LAUNCH_CHECK();
        return JITDB_OK;
    }
    if (!x || !h || !c || !gates || !fgate || !dx || !workspace) return JITDB_E_NULL;
    if (!s->perm || !s->inv_perm || !s->child_ptr || !s->child_idx || !s->host_level_ptr) return JITDB_E_NULL;
    if ((reinterpret_cast<uintptr_t>(workspace) & 255) != 0) return JITDB_E_BADARG;
    // operand rows are read in 16-byte pieces
    if ((reinterpret_cast<uintptr_t>(x) & 15) || (reinterpret_cast<uintptr_t>(h) & 15) ||
        (reinterpret_cast<uintptr_t>(dx) & 15))
        return JITDB_E_BADARG;
    const int L = s->n_levels;
    if (L < 1 || L > n || s->host_level_ptr[0] != 0 || s->host_level_ptr[L] != n) return JITDB_E_SCHEDULE;
    const BwdWs w = carve_bwd_ws(n, d, workspace);
    if (workspace_bytes < w.bytes) return JITDB_E_WORKSPACE;
    if (dtype == JITDB_F32)
        return run_backward<float>(static_cast<const float *>(x), static_cast<const float *>(W),
                                   static_cast<const float *>(U), d, s, static_cast<const float *>(h), c,
                                   static_cast<const float *>(gates), static_cast<const float *>(fgate), gh, gc, dx, dW, dU, db, w, st);
    return run_backward<bf16_t>(static_cast<const bf16_t *>(x), static_cast<const bf16_t *>(W),
                                static_cast<const bf16_t *>(U), d, s, static_cast<const bf16_t *>(h), c,
                                static_cast<const bf16_t *>(gates), static_cast<const bf16_t *>(fgate), gh, gc, dx, dW, dU, db, w, st);
}
