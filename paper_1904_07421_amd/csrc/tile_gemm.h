// The K loop of the tiled kernels (forward.hip: levels, projections; backward.hip: data and weight gradients): 128 x 256
// tiles of C on the matrix cores, operands moved from global memory straight into LDS.
#pragma once

#include "level_common.h"

namespace jitdb {
namespace {

// Block id -> tile of the level kernel.  The hardware deals consecutive block ids
// round-robin to the 8 XCDs, each with its own L2.  Row tile r belongs to XCD r % 8, so
// that the blocks of all its column tiles read the same A rows through one L2.  Inside an
// XCD the column tiles are taken in groups of kColGroup: the XCD sweeps all its row tiles
// with one group of columns, then with the next, which bounds the B rows in use at a
// time; A is fetched once per group.  (With 8 column tiles, H = 512, one group measured
// faster than two: re-reading A costs more than the B rows that fall out of L2.)  The
// grid holds 8 * ceil(R / 8) * C blocks; blocks past an XCD's share return at once.
constexpr int kColGroup = 8;
__device__ __forceinline__ bool block_to_tile(int b, int n_row_tiles, int n_col_tiles, int &row_tile, int &col_tile) {
    const int xcd = b & 7, idx = b >> 3;
    const int rows_x = (n_row_tiles - xcd + 7) >> 3;        // row tiles of this XCD
    if (idx >= rows_x * n_col_tiles) return false;
    const int g = idx / (rows_x * kColGroup);
    const int rem = idx - g * rows_x * kColGroup;
    const int left = n_col_tiles - g * kColGroup;
    const int cg = left < kColGroup ? left : kColGroup;    // columns in this group
    row_tile = xcd + 8 * (rem / cg);
    col_tile = g * kColGroup + rem % cg;
    return true;
}

// ---- the level GEMM ------------------------------------------------------------------
// One block of four waves computes 128 rows x 256 packed columns (2 unit tiles x 4 gates x
// 32 units); each wave a 64 x 128 sub-tile, i.e. 2 x 4 MFMA tiles of 32 x 32, so that all
// four gates of a hidden unit end up in one wave's accumulators.  Two blocks share a CU
// (half the LDS and at most 256 registers each): the start-up and the memory-bound cell
// update of one leave the matrix cores to the other.
//
// A is the level's stacked input [x | hsum], B the packed [W | U]; K runs over stages of
// 64 bytes per row, n_x stages of the x part, then n_h of the h part, in which the forget
// gate is skipped (U_f applies to each child's own h, not to the sum).  The projection
// instead reads A rows from h by node id and uses only the U part of the forget rows.
// Stages travel from global memory straight into LDS (global_load_lds, 16 bytes per lane)
// without passing through registers.  Three stage buffers: while stage g is multiplied,
// g+1 and g+2 (and for half the time g+3) are in flight; one barrier per stage.
//
// In each 16-wide (bf16) or 8-wide (fp32) K group, lanes 0-31 take the first 16 bytes and
// lanes 32-63 the next 16 for A and B alike; since the same assignment is used on both
// operands any such split of K is a valid MFMA schedule.
//
// A direct load writes the 64 lanes' pieces to 1024 consecutive LDS bytes, i.e. 16 rows of
// 64 bytes with no room for padding, so bank conflicts are avoided by permuting the four
// 16-byte pieces of a row instead: piece p of row r is kept in slot p ^ ((r >> 2) & 3).
// The lane that fills slot s of row r therefore fetches piece s ^ ((r >> 2) & 3), and a
// fragment read of 16 consecutive rows touches 16 distinct 16-byte columns.
constexpr int kDmaThreads = 256;
constexpr int kDmaBM = 128;        // rows per block
constexpr int kDmaStage = 64;      // bytes of K per row and stage
constexpr int kDmaBuf = (kDmaBM + kBN) * kDmaStage;
constexpr int kDmaBufs = 3;
constexpr int kWarmMaxStages = 256; // longest K loop whose A tile is requested up front (2 MB)


// Waits until at most N of this wave's loads are outstanding and all its LDS operations
// are done, then meets the block at a barrier.  Written as one asm statement with a memory
// clobber so that nothing moves across it, and without the fence of __syncthreads(), which
// would wait for every direct-to-LDS load in flight.
template <int N>
__device__ __forceinline__ void dma_wait_barrier() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// MODE_TN multiplies A^T B instead: K runs over the operands' ROWS (slabs of 64 bytes hold the columns), for the weight
// gradients, whose reduction is over the nodes.  A stage is 64 / sizeof(T) rows of the tile's 128 + 256 columns, the same
// 24 KB in the same 24 direct loads of 1 KB (16 rows of one slab).  A fragment wants consecutive K in one lane, so the rows are
// transposed on their way out of LDS: ds_read_b64_tr_b16 for bf16 (a half-wave's two 16-lane groups read 4 rows of 32
// columns, the wave 512 consecutive bytes, no conflicts), single words for fp32, where a lane of the 32x32x2 MFMA holds one
// k anyway (odd slabs keep their rows in pairs exchanged, so that the two slabs of a tile fall on different banks).
// MODE_SWAP is MODE_GENERIC with the long operand (the level's rows) as B: the L2 warm-up then takes B's tile.
template <typename T, int MODE, int NBUF = kDmaBufs, typename Hook>
__device__ __forceinline__ void dma_gemm(const LevelArgs &a, char *lds, const int *row_node,
                                         int tile_row0, int col_tile, floatx16 (&acc)[2][4],
                                         char *sink, Hook &&after_first_requests) {
    constexpr int ESZ = (int)sizeof(T);
    constexpr int NG_X = (MODE == MODE_LEAF) ? 3 : 4;      // gate tiles multiplied in the x part
    constexpr int NG_H = (MODE == MODE_INTERNAL) ? 3 : 4;  // ... in the h part
    constexpr int NB = (MODE == MODE_LEAF) ? 3 : 4;        // 16-row B units a wave moves per stage
    constexpr int NLOAD = 2 + NB;                          // loads per wave and stage

    const int t = threadIdx.x;
    const int lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int hf = lane >> 5, l32 = lane & 31;

    const int n_x = (MODE == MODE_PROJ) ? 0 : a.Dp * ESZ / kDmaStage;
    const int n_h = (MODE == MODE_LEAF) ? 0 : a.Hp * ESZ / kDmaStage;
    const int n_stages = n_x + n_h;   // even and >= 2: K is padded to 128 bytes

    // ---- mover: lane l fills slot l&3 of row l>>2 of each 16-row unit it is given
    const int lrow = lane >> 2;
    const int piece16 = ((lane & 3) ^ ((lane >> 4) & 3)) * 16;
    // MODE_TN: unit u of an operand's tile = 16 rows of one of its slabs
    auto tn_unit = [&](int u, int64_t rows_alloc) __attribute__((always_inline)) -> int64_t {
        const int slab = ESZ == 2 ? u >> 1 : u, rows16 = ESZ == 2 ? u & 1 : 0;
        const int row = ESZ == 2 ? lrow : lrow ^ (2 * (slab & 1));
        return ((int64_t)slab * rows_alloc + rows16 * 16 + row) * 64 + (lane & 3) * 16;
    };
    const char *pa[2];
    int a_lds[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int r = (wave + 4 * i) * 16 + lrow;      // row of the tile
        a_lds[i] = (wave + 4 * i) * 16 * kDmaStage;
        if constexpr (MODE == MODE_TN) {
            pa[i] = static_cast<const char *>(a.stack) + tn_unit(wave + 4 * i, a.n_rows_alloc);
        } else if constexpr (MODE == MODE_PROJ) {
            int g = tile_row0 + r;
            if (g >= a.n_rows) g = a.n_rows - 1;
            pa[i] = static_cast<const char *>(a.hs) + (int64_t)row_node[g - tile_row0] * a.Hp * ESZ + piece16;
        } else {
            pa[i] = static_cast<const char *>(a.stack) + (int64_t)(tile_row0 + r) * kDmaStage + piece16;
        }
    }
    // bytes from one stage to the next: a slab of A / of B; the projection's A rows are
    // rows of h in node order, K contiguous
    const int64_t a_stage = (MODE == MODE_TN) ? 64 / ESZ * 64 : (MODE == MODE_PROJ) ? kDmaStage : (int64_t)a.n_rows_alloc * kDmaStage;
    const int64_t b_stage = (MODE == MODE_TN) ? 64 / ESZ * 64 : (int64_t)a.NPU * kDmaStage;
    const char *pb[NB];
    int b_lds[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int idx = wave * NB + i;
        if constexpr (MODE == MODE_TN) {
            b_lds[i] = (8 + idx) * 1024;
            pb[i] = static_cast<const char *>(a.Bp) + tn_unit(idx, a.NPU);
            continue;
        }
        int lds_row;
        int64_t src_row;
        if constexpr (MODE == MODE_PROJ) {
            // LDS row q*32 + u holds the forget row of unit u of unit tile col_tile*8 + q
            const int q = idx >> 1;
            lds_row = q * kUnit + (idx & 1) * 16;
            src_row = (int64_t)(col_tile * 8 + q) * kGateTile + 3 * kUnit + (idx & 1) * 16 + lrow;
        } else {
            // LDS row = packed row within the block's 256; the leaf level skips the forget rows
            const int ut = idx / (2 * NB), gate = (idx % (2 * NB)) >> 1;
            lds_row = ut * kGateTile + gate * kUnit + (idx & 1) * 16;
            src_row = (int64_t)col_tile * kBN + lds_row + lrow;
        }
        b_lds[i] = (kDmaBM + lds_row) * kDmaStage;
        pb[i] = static_cast<const char *>(a.Bp) +
                operand_offset(src_row, MODE == MODE_PROJ ? (int64_t)a.Dp * ESZ : 0, a.NPU) + piece16;
    }
    // load i (0 .. NLOAD-1) of stage s
    auto issue_one = [&](int s, int buf, int i) __attribute__((always_inline)) {
        char *dst = lds + buf * kDmaBuf;
        if (i < 2)
            __builtin_amdgcn_global_load_lds(JITDB_GLOBAL_PTR(pa[i] + s * a_stage), JITDB_LDS_PTR(dst + a_lds[i]), 16, 0, 0);
        else
            __builtin_amdgcn_global_load_lds(JITDB_GLOBAL_PTR(pb[i - 2] + s * b_stage), JITDB_LDS_PTR(dst + b_lds[i - 2]), 16, 0, 0);
    };
    auto issue = [&](int s, int buf) __attribute__((always_inline)) {
        char *dst = lds + buf * kDmaBuf;
#pragma unroll
        for (int i = 0; i < 2; ++i)
            __builtin_amdgcn_global_load_lds(JITDB_GLOBAL_PTR(pa[i] + s * a_stage), JITDB_LDS_PTR(dst + a_lds[i]), 16, 0, 0);
#pragma unroll
        for (int i = 0; i < NB; ++i)
            __builtin_amdgcn_global_load_lds(JITDB_GLOBAL_PTR(pb[i] + s * b_stage), JITDB_LDS_PTR(dst + b_lds[i]), 16, 0, 0);
    };

    // ---- fragments: K group h (0, 1) of a stage is pieces 2h (lanes 0-31) and 2h+1 (lanes 32-63)
    const int sw = (l32 >> 2) & 3;
    int a_rd[2], b_rd[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int slot16 = ((2 * h + hf) ^ sw) * 16;
        a_rd[h] = (wm * 64 + l32) * kDmaStage + slot16;
        b_rd[h] = (kDmaBM + wn * 128 + l32) * kDmaStage + slot16;
    }
    if constexpr (MODE == MODE_TN) {
        // bf16: [h] is the K group (a unit of 1 KB); fp32: [h] is the parity of the k step, the K group an offset
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int sel = (lane >> 4) & 1;
            const int lane_off = ESZ == 2 ? h * 1024 + (hf * 4 + ((lane & 15) >> 2)) * 64 + sel * 32 + (lane & 3) * 8
                                          : sel * 1024 + (2 * (h ^ sel) + hf) * 64 + (lane & 15) * 4;
            a_rd[h] = wm * 4096 + lane_off;
            b_rd[h] = 8192 + wn * 8192 + lane_off;
        }
    }
    // Fragment reads are written as asm: the compiler would otherwise make every LDS read
    // wait for all direct-to-LDS loads in flight, which it cannot tell apart from the
    // buffer being read.  The waits for the reads are therefore placed by hand as well
    // (LDS operations of a wave complete in order).  A K group's fragments: two of A, NG of B.
    const uint32_t lds_base = (uint32_t)(uintptr_t)JITDB_LDS_PTR(lds);
    struct Frags {
        u32x4 a[2], b[4];
    };
    auto tn_read = [&](auto h_tag, auto tile_tag, uint32_t even, uint32_t odd, u32x4 &f) __attribute__((always_inline)) {
        constexpr int H = decltype(h_tag)::value, I = decltype(tile_tag)::value;
        u32x2 lo, hi;
        if constexpr (ESZ == 2) {
            const uint32_t p = H == 0 ? even : odd;
            asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(lo) : "v"(p), "n"(I * 2048) : "memory");
            asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(hi) : "v"(p), "n"(I * 2048 + 512) : "memory");
        } else {
            asm volatile("ds_read2st64_b32 %0, %1 offset0:%2 offset1:%3" : "=v"(lo) : "v"(even), "n"(I * 8 + H * 2), "n"(I * 8 + H * 2 + 1) : "memory");
            asm volatile("ds_read2st64_b32 %0, %1 offset0:%2 offset1:%3" : "=v"(hi) : "v"(odd), "n"(I * 8 + H * 2), "n"(I * 8 + H * 2 + 1) : "memory");
        }
        f = __builtin_shufflevector(lo, hi, 0, 1, 2, 3);
    };
    auto tn_read_group = [&](int buf, auto h_tag, Frags &f) __attribute__((always_inline)) {
        const uint32_t at = lds_base + buf * kDmaBuf;
        const uint32_t a0 = at + a_rd[0], a1 = at + a_rd[1], b0 = at + b_rd[0], b1 = at + b_rd[1];
        tn_read(h_tag, std::integral_constant<int, 0>(), a0, a1, f.a[0]);
        tn_read(h_tag, std::integral_constant<int, 0>(), b0, b1, f.b[0]);
        tn_read(h_tag, std::integral_constant<int, 1>(), a0, a1, f.a[1]);
        tn_read(h_tag, std::integral_constant<int, 1>(), b0, b1, f.b[1]);
        tn_read(h_tag, std::integral_constant<int, 2>(), b0, b1, f.b[2]);
        tn_read(h_tag, std::integral_constant<int, 3>(), b0, b1, f.b[3]);
    };
    auto read_group = [&](int buf, int h, auto ng_tag, Frags &f) __attribute__((always_inline)) {
        constexpr int NG = decltype(ng_tag)::value;
        if constexpr (MODE == MODE_TN) {
            if (h == 0) tn_read_group(buf, std::integral_constant<int, 0>(), f);
            else tn_read_group(buf, std::integral_constant<int, 1>(), f);
            return;
        }
        const uint32_t aa = lds_base + buf * kDmaBuf + a_rd[h];
        const uint32_t bb = lds_base + buf * kDmaBuf + b_rd[h];
        asm volatile("ds_read_b128 %0, %1" : "=v"(f.a[0]) : "v"(aa) : "memory");
        asm volatile("ds_read_b128 %0, %1" : "=v"(f.b[0]) : "v"(bb) : "memory");
        asm volatile("ds_read_b128 %0, %1 offset:2048" : "=v"(f.a[1]) : "v"(aa) : "memory");
        asm volatile("ds_read_b128 %0, %1 offset:2048" : "=v"(f.b[1]) : "v"(bb) : "memory");
        asm volatile("ds_read_b128 %0, %1 offset:4096" : "=v"(f.b[2]) : "v"(bb) : "memory");
        if constexpr (NG == 4)
            asm volatile("ds_read_b128 %0, %1 offset:6144" : "=v"(f.b[3]) : "v"(bb) : "memory");
    };
    // all LDS reads issued so far have arrived; ties the fragments to the wait
    auto reads_done = [&](auto ng_tag, Frags &f) __attribute__((always_inline)) {
        constexpr int NG = decltype(ng_tag)::value;
        if constexpr (NG == 4)
            asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(f.a[0]), "+v"(f.a[1]), "+v"(f.b[0]), "+v"(f.b[1]), "+v"(f.b[2]), "+v"(f.b[3]));
        else
            asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(f.a[0]), "+v"(f.a[1]), "+v"(f.b[0]), "+v"(f.b[1]), "+v"(f.b[2]));
    };
    auto multiply = [&](auto ng_tag, const Frags &f) __attribute__((always_inline)) {
        constexpr int NG = decltype(ng_tag)::value;
#pragma unroll
        for (int m = 0; m < 2 * NG; ++m)
            mfma_step<T>(f.a[m / NG], f.b[m % NG], acc[m / NG][m % NG]);
    };
    // The same with the loads of stage s dealt out between the MFMAs, one after each: a
    // wave issues in order, and a burst of loads in front of the MFMAs would hold them back
    // until the memory pipeline has taken the loads of all waves of the CU.
    // (The condition wraps each load, not the MFMAs: accumulators that meet again after
    // a branch get copied.)
    auto multiply_and_issue = [&](auto ng_tag, const Frags &f, int s, int buf, bool wanted) __attribute__((always_inline)) {
        constexpr int NG = decltype(ng_tag)::value;
#pragma unroll
        for (int m = 0; m < 2 * NG; ++m) {
            mfma_step<T>(f.a[m / NG], f.b[m % NG], acc[m / NG][m % NG]);
            __builtin_amdgcn_sched_barrier(0);
            if (m < NLOAD && wanted) issue_one(s, buf, m);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    const std::integral_constant<int, NG_X> ngx;
    const std::integral_constant<int, NG_H> ngh;

    // One stage.  On entry P holds K group 0 of stage g (buffer cur).  The reads of K group 1
    // go out, K group 0 is multiplied; once those reads are back nobody needs buffer cur any
    // more, and after the barrier (which also publishes stage g+1) it takes the request for
    // stage g+3.  K group 0 of stage g+1 is then read while K group 1 of stage g is multiplied.
    // With two buffers (NBUF == 2) a stage's request follows the barrier that frees its buffer by one stage
    // instead of two: nothing younger is in flight at a barrier, and every wait is for all loads.
    static_assert(NBUF == 2 || NBUF == 3, "two or three stage buffers");
    Frags P, Q;
    int cur = 0;
    auto next_buf = [&]() __attribute__((always_inline)) { return cur == NBUF - 1 ? 0 : cur + 1; };
    auto step = [&](int g, auto ng_cur, auto ng_next, auto wait_tag) __attribute__((always_inline)) {
        constexpr int WAIT = NBUF == 2 ? 0 : decltype(wait_tag)::value;
        read_group(cur, 1, ng_cur, Q);
        __builtin_amdgcn_sched_barrier(0);
        multiply(ng_cur, P);
        __builtin_amdgcn_sched_barrier(0);
        reads_done(ng_cur, Q);
        dma_wait_barrier<WAIT>();
        read_group(next_buf(), 0, ng_next, P);
        __builtin_amdgcn_sched_barrier(0);
        multiply_and_issue(ng_cur, Q, g + NBUF, cur, g + NBUF < n_stages);
        __builtin_amdgcn_sched_barrier(0);
        reads_done(ng_next, P);
        cur = next_buf();
    };
    const std::integral_constant<int, NLOAD> w_more;   // a younger stage stays in flight
    const std::integral_constant<int, 0> w_none;

    // Warm L2 with the block's share of its A tile, one 4-byte load per 128-byte line (the
    // data goes to a sink): the stage loads further down the K loop then find their lines
    // in L2 instead of each waiting for HBM with only two stages of lookahead.  The blocks
    // of one column group of a row tile run side by side on one XCD and split the lines.
    // (A long reduction axis, as in the weight-gradient GEMMs, would ask for far more than L2
    // holds; there the stage loads take their chances.)
    if (MODE == MODE_SWAP && n_stages <= kWarmMaxStages) {
        char *sink_w = sink + wave * 256;
        const int n_lines = n_stages * (kBN * kDmaStage / 128);
        const char *tile = static_cast<const char *>(a.Bp) + (int64_t)col_tile * kBN * kDmaStage;
        const int row_tile = tile_row0 / kDmaBM, left = a.n_row_tiles - (row_tile / kColGroup) * kColGroup;
        const int sharers = left < kColGroup ? left : kColGroup;
        for (int li = row_tile % kColGroup + sharers * t; li < n_lines; li += sharers * kDmaThreads) {
            const int slab = li >> 7, line = li & 127;
            __builtin_amdgcn_global_load_lds(JITDB_GLOBAL_PTR(tile + slab * b_stage + line * 128),
                                             JITDB_LDS_PTR(sink_w), 4, 0, 0);
        }
    } else if (MODE != MODE_PROJ && MODE != MODE_TN && n_stages <= kWarmMaxStages) {
        char *sink_w = sink + wave * 256;
        const int n_lines = n_stages * (kDmaBM * kDmaStage / 128);
        const char *tile = static_cast<const char *>(a.stack) + (int64_t)tile_row0 * kDmaStage;
        const int left = a.n_col_tiles - (col_tile / kColGroup) * kColGroup;
        const int sharers = left < kColGroup ? left : kColGroup;
        for (int li = col_tile % kColGroup + sharers * t; li < n_lines; li += sharers * kDmaThreads) {
            const int slab = li >> 6, line = li & 63;
            __builtin_amdgcn_global_load_lds(JITDB_GLOBAL_PTR(tile + slab * a_stage + line * 128),
                                             JITDB_LDS_PTR(sink_w), 4, 0, 0);
        }
    }
    issue(0, 0);
    issue(1, 1);
    if (NBUF > 2 && n_stages > 2) issue(2, 2);
    after_first_requests();
    if (NBUF > 2 && n_stages > 2) dma_wait_barrier<2 * NLOAD>(); else dma_wait_barrier<NLOAD>();   // stage 0 is there
    int g = 0;
    if constexpr (MODE == MODE_PROJ) {
        read_group(0, 0, ngh, P);
        reads_done(ngh, P);
    } else {
        read_group(0, 0, ngx, P);
        reads_done(ngx, P);
        const int x_end = n_x - 1 < n_stages - 2 ? n_x - 1 : n_stages - 2;
        for (; g < x_end; ++g) step(g, ngx, ngx, w_more);
        if constexpr (MODE == MODE_INTERNAL) {   // n_h >= 2, so this stage is not among the last two
            step(g, ngx, ngh, w_more);
            ++g;
        }
    }
    if constexpr (MODE == MODE_LEAF) {
        step(g, ngx, ngx, w_none);
        read_group(cur, 1, ngx, Q);
        multiply(ngx, P);
        reads_done(ngx, Q);
        multiply(ngx, Q);
    } else {
        for (; g < n_stages - 2; ++g) step(g, ngh, ngh, w_more);
        step(g, ngh, ngh, w_none);
        read_group(cur, 1, ngh, Q);
        multiply(ngh, P);
        reads_done(ngh, Q);
        multiply(ngh, Q);
    }
    __builtin_amdgcn_sched_barrier(0);
    dma_wait_barrier<0>();       // every wave is done reading the stage buffers
}

}  // namespace
}  // namespace jitdb
