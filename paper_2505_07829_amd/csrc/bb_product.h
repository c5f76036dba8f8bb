// Matrix products of many rows without a norm prologue: the main loop of the prefill programs.
//
//   MODE_PLAIN       C = A B [+ residual], or fp32 partial results of a share of the contraction (PARTS_APART)
//   MODE_GATEUP_PRE  H = SiLU(r A W1) (r A W3), A already carries the gain, r from its row kernel
//   MODE_LN_PRE      C = r (A W - mu c) + b, A already carries gamma
//
// for contractions of three 64-index steps and more (the last one may be incomplete) with operands below 4 GiB
// (gemm_kernel takes the rest, and the modes with the statistics inside the loop).  Any number of rows and columns: a
// ragged last tile reads its last valid row or chunk of columns in place of the missing ones and stores only the valid
// elements.
//
// What bounds it: the power the chip may draw, and weights that arrive late.  On zeros in the caches the loop runs 1.00 us
// per step of a 256 x 256 tile (85 % of the matrix cores at 2.4 GHz); on normal operands the clock falls until a full
// round takes 1.3 to 1.4 times that.  So the choices below save energy or time spent waiting (normal operands, us, both
// sides on one box; "cold": weights from memory, as a model's layers find them):
//  - 16x16x32 matrix instructions: half the accumulator traffic per operation of the 32x32x16 form.  A loop of nothing
//    else 1914 against 1760 TFLOP/s; 8192 x 4096 x 16384 869 -> 804.  Eight wavefronts, 2 x 4, 128 x 64 (64 x 64) each.
//  - The contraction runs from its first index to its last on every XCD, so that an element of C is the same sum whatever
//    tile it lies in: equal rows give equal bits.  A 16x16x32 instruction adds to the bits of two 32x32x16 instructions over the
//    same 32 indices, so the sums are gemm_kernel's too.  (Starting an eighth of the contraction apart per XCD spares the
//    memory-side cache, on zeros 720 -> 593 at 8192 x 4096 x 16384, but made the order of a sum depend on the tile, and in the FFN
//    of 4096 x 8192 x 28672 it is the slower one: 3796 against 3745 us.)
//  - Where the weights that all XCDs read during one round of 256-row tiles fit the memory-side cache well (K <= 4096),
//    groups of row tiles also start at different column tiles (p.rot): LN of 8192 x 4096 x 16384 823 -> 812.  With longer
//    contractions the other groups come too late: FFN of 4096 x 8192 x 28672 3797 -> 3915.
//  - Three stages of the weights, which come from memory (64 contraction indices each), and with 128-row tiles of A;
//    with 256-row tiles two stages of A fill the 160 KiB.  256-row tiles, two -> three stages of the weights, cold:
//    2048 x 4096 x 2*11008 284 -> 275, 4096 x 28672 x 8192 1370 -> 1278 (weights transposed 1562 -> 1367); 128-row tiles,
//    two -> three stages of both: 1000 x 2944 x 2*7680 85 -> 72.  Stages of 32 indices (four, 64 bytes of a row each):
//    2048 x 4096 x 2*11008 255 -> 265.
//  - One load-to-LDS instruction per group of four matrix instructions: the loads of a compute unit's eight wavefronts
//    then just fill its load path.  Two per group: 130 -> 143 (2048 x 8192 x 4096).  Touching the lines of a later tile first
//    gains nothing: they come back in order with the loads behind them.
//  - A in panels of 64 columns ([K / 64][M][64], written so by the kernel before): a tile is 32 KiB in one piece instead
//    of 256 pieces a row apart.  4096 x 28672 x 8192 (rows 57 KB apart) 1466 -> 1365; rows of 8 KB: equal.
// Together against the 32x32x16 loop of gemm_kernel, cold: 2048 x 4096 x 2*11008 294 -> 280, 8192 x 4096 x 16384 (LN) 833 ->
// 796, 4096 x 8192 x 2*28672 2809 -> 2588, 4096 x 28672 x 8192 1505 -> 1268.
//
// LDS: rows of 128 bytes (A, transposed weights) with the chunk index XOR row / 2 % 8 (lds_pos); row-major weights as
// they lie in memory, chunk index XOR 2 (row % 4 + 4 (row / 8 % 2)): the 32 lanes of one pass of a transposing read
// (ds_read_b64_tr_b16) take 32 bytes of each of eight rows, which then lie on eight different quarters of the banks.
// The products are computed transposed (the weight fragment is the first operand), so that a lane's four
// accumulators are four consecutive columns of one row: the epilogue needs one exchange between neighbouring groups
// of sixteen lanes to store 16 bytes per lane.
#pragma once
#include <type_traits>

#include "bb_gemm.h"

namespace bb {

constexpr int PRODUCT_THREADS = 512;

// PARTS: how a contraction of several shares of p.nk_split steps each is summed (every share from zero, then the shares in
// order): PARTS_ONE, there is one share; PARTS_APART, p.nsplit workgroups per tile, a share each (steps past the end of the
// contraction, and those that a share is shorter than the loop's stages, load zeros), which store fp32 partial results for splitk_reduce_kernel; PARTS_FOLD, one workgroup, which adds
// a finished share to a second set of accumulators: the same bits without partial results in memory.
// BN: columns of a tile (of both weight matrices together): 256, or 128 with 128 rows: five stages of 32 KiB, half
// the work per tile.  For products of so few tiles that a compute unit's loads are all that is in flight for it: cold, 128 x
// 256 -> 128 x 128 tiles, 1000 x 7680 x 2880 92.9 -> 66.0 (96 and 184 tiles; transposed 100 -> 67), 300 x 4096 x 4096 48.6 -> 33.0,
// 2048 x 8192 x 2048 90 -> 71; on a full chip they lose, 2048 x 11008 x 4096 148 -> 186.
// RAGGED: the contraction's last step is incomplete (a multiple of 8): its loads take their whole offset per lane, and what lies
// past the contraction gets one past the buffer, which loads zeros (A then row-major).
template <int MODE, int BM, int BN, int PARTS, bool BT, bool RAGGED>
__global__ __launch_bounds__(PRODUCT_THREADS) void product_kernel(const GemmArgs p) {
    static_assert(MODE == MODE_PLAIN || MODE == MODE_GATEUP_PRE || MODE == MODE_LN_PRE, "no norm prologue here");
    static_assert(PARTS == PARTS_ONE || MODE == MODE_PLAIN, "contraction in shares: plain products");
    static_assert(PARTS != PARTS_FOLD || BN == 128, "shares added in registers: 128 x 128 tiles");
    constexpr bool SPLIT = PARTS == PARTS_APART, FOLD = PARTS == PARTS_FOLD;
    static_assert((BN == 256 && (BM == 128 || BM == 256)) || (BN == 128 && BM == 128 && MODE == MODE_PLAIN), "tiles");
    constexpr bool DUAL = MODE == MODE_GATEUP_PRE;
    constexpr int WR = BM / 2;                        // rows of a wavefront (2 x 4 wavefronts, BN / 4 columns each)
    constexpr int MT = WR / 16, NT = BN / 64;         // 16x16 subtiles of a wavefront
    constexpr int NG = 2 * MT;                        // groups of NT matrix instructions per step
    constexpr int AHEAD = 4;                          // groups that A fragments are read ahead; the barrier stands there
    constexpr int ADMA = BM / 64, BDMA = BN / 64;     // load-to-LDS instructions per wavefront and step
    constexpr int NCOL = DUAL ? 128 : BN;             // output columns of a tile
    constexpr int STAGES = BN == 128 ? 5 : 3;         // stages of the weights
    constexpr int STAGES_A = BM == 256 ? 2 : STAGES;
    constexpr u32 ABYTES = BM * 128, BBYTES = BN * 128;
    __shared__ u32x4 lds[(STAGES * BBYTES + STAGES_A * ABYTES) / 16];  // weights' stages, then A's
    constexpr bool HALF = DUAL || BN == 128;          // LDS rows of 128 columns

    // tile coordinates (the order of gemm_kernel, column tiles of group number grp rotated by p.rot grp)
    const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
    const int lin = xcd * p.tiles_per_xcd + local;
    const int ntiles = p.tiles_m * p.tiles_n;
    if (local >= p.tiles_per_xcd || lin >= (SPLIT ? ntiles * p.nsplit : ntiles)) return;
    const int tile = SPLIT ? lin % ntiles : lin, split = SPLIT ? lin / ntiles : 0;
    const int per_group = p.group_m * p.tiles_n;
    const int grp = tile / per_group, in_grp = tile - grp * per_group;
    const int rows_grp = min(p.group_m, p.tiles_m - grp * p.group_m);
    const int tm = grp * p.group_m + in_grp % rows_grp, tn = (in_grp / rows_grp + p.rot * grp) % p.tiles_n;
    const int nk_all = (p.K + GEMM_BK - 1) / GEMM_BK;
    const int nk = SPLIT ? max(p.nk_split, STAGES) : nk_all;
    const int kt0 = SPLIT ? split * p.nk_split : 0;
    const int kend = SPLIT ? min(kt0 + p.nk_split, nk_all) : nk_all;
    const int m0 = tm * BM, n0 = tn * NCOL;

    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = w >> 2, wn = w & 3;
    const int l16 = lane & 15, g = lane >> 4;

    // ---- load-to-LDS roles
    const size_t bytesA = (size_t)p.M * p.K * 2, bytesB = (size_t)p.K * p.N * 2;       // (densely packed)
    u32 uA[ADMA], lA[ADMA];                           // byte offsets: wavefront-uniform, per lane
    bool inA[ADMA], inB[BDMA];                        // RAGGED: this lane's chunk of the last step is in the contraction
    const int left = p.K - (nk_all - 1) * GEMM_BK;    // its indices
#pragma unroll
    for (int j = 0; j < ADMA; ++j) {
        const int rb = 8 * (ADMA * w + j);            // first tile row of the instruction
        const int ub = min(m0 + rb, p.M - 1);
        const int kc = (lane & 7) ^ (((rb + (lane >> 3)) >> 1) & 7);
        uA[j] = (u32)ub * (u32)p.lda * 2u;
        lA[j] = (u32)((min(m0 + rb + (lane >> 3), p.M - 1) - ub) * p.lda + 8 * kc) * 2u;
        inA[j] = 8 * kc < left;
    }
    u32 uB[BDMA], lB[BDMA];
#pragma unroll
    for (int q = 0; q < BDMA; ++q) {
        if (BT) {
            const int rb = 8 * (BDMA * w + q);
            const int nb = DUAL ? n0 + (rb & 127) : n0 + rb;
            const int ub = min(nb, p.N - 1);
            const int kc = (lane & 7) ^ (((rb + (lane >> 3)) >> 1) & 7);
            uB[q] = (u32)ub * (u32)p.ldb * 2u;
            lB[q] = (u32)((min(nb + (lane >> 3), p.N - 1) - ub) * p.ldb + 8 * kc) * 2u;
            inB[q] = 8 * kc < left;
        } else {
            // rows of the weight tile as in memory; 16-byte chunk index XOR 2 ((row % 4) + 4 (row / 8 % 2))
            const int rb = HALF ? 4 * (w + 8 * (q & 1)) : 2 * (w + 8 * q);
            const int rl = HALF ? lane >> 4 : lane >> 5;
            const int row = rb + rl;
            const int chunk = (HALF ? lane & 15 : lane & 31) ^ (((row & 3) | (((row >> 3) & 1) << 2)) << 1);
            uB[q] = (u32)rb * (u32)p.ldb * 2u + (u32)n0 * 2u;
            lB[q] = (u32)(rl * p.ldb + min(8 * chunk, p.N - 8 - n0)) * 2u;
            inB[q] = row < left;
        }
    }
    // The load-to-LDS instructions of step kt into the stage at LDS address dst.  Written in asm, because the compiler
    // makes every LDS read wait for every such transfer that it sees unless stages are arrays of their own and the loop is
    // unrolled over them.  They write no register; what orders them against the reads is the wait and the barrier of
    // every step.  (One wait state between the scalar write of M0 and its use.)
    // SPLIT: past the end of the share, or of the contraction, the buffer is empty and the load writes zeros (whose products
    // change no sum).
    auto to_lds = [&](const u16* base, size_t bytes, u32 k, u32 voff, u32 soff, bool in, u32 dst) {
        const bool there = !SPLIT || (int)k < kend;
        if (RAGGED) {
            const bool last = (int)k == nk_all - 1;
            voff = !last ? voff : in ? voff + soff : 0xfffffff0u;
            soff = last ? 0u : soff;
        }
        const u32x4 rs = {(u32)(size_t)base, (u32)((size_t)base >> 32) & 0xffffu, there ? (u32)bytes : 0u, 0x00020000u};
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                     ::"s"(__builtin_amdgcn_readfirstlane(dst)), "v"(voff), "s"(rs), "s"(there ? soff : 0u) : "m0");
    };
    auto dma_a = [&](int kt, u32 dst, int j) {
        const u32 k = (u32)(kt0 + kt);
        to_lds(p.A, bytesA, k, lA[j], uA[j] + k * p.a_step, inA[j], dst + 1024u * (u32)(ADMA * w + j));
    };
    auto dma_b = [&](int kt, u32 dst, int x) {
        const u32 k = (u32)(kt0 + kt);
        if (BT) {
            const bool second = DUAL && 8 * (BDMA * w + x) >= 128;
            to_lds(second ? p.B1 : p.B0, bytesB, k, lB[x], uB[x] + k * (2u * GEMM_BK), inB[x], dst + 1024u * (u32)(BDMA * w + x));
        } else {
            const bool second = DUAL && x >= 2;
            to_lds(second ? p.B1 : p.B0, bytesB, k, lB[x], uB[x] + k * (u32)p.ldb * (2u * GEMM_BK), inB[x],
                   dst + 1024u * (u32)(HALF ? (x >> 1) * 16 + w + 8 * (x & 1) : w + 8 * x));
        }
    };

    // ---- fragment-read roles (byte offsets inside a stage)
    u32 offA[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) offA[s] = (u32)lds_pos(WR * wm + l16, 4 * s + g) * 16u;
    constexpr int BROW = HALF ? 256 : 512;
    u32 offB[NT];
#pragma unroll
    for (int tt = 0; tt < NT; ++tt) {
        if (BT) {
            const int row = (DUAL ? 128 * (tt >> 1) + 32 * wn + 16 * (tt & 1) : BN / 4 * wn + 16 * tt) + l16;
            offB[tt] = (u32)lds_pos(row, g) * 16u;                // slice 1: XOR 64
        } else {
            const int r = 8 * g + (l16 >> 2);
            const int chunk = (DUAL ? 4 * wn + 2 * (tt & 1) : BN / 32 * wn + 2 * tt) + ((l16 & 3) >> 1);
            const int key = ((r & 3) | (((r >> 3) & 1) << 2)) << 1;
            offB[tt] = (u32)((DUAL ? 64 * 256 * (tt >> 1) : 0) + r * BROW + ((chunk ^ key) << 4) + 8 * (l16 & 1));
        }
    }

    f32x4 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int tt = 0; tt < NT; ++tt) acc[i][tt] = f32x4{0.f, 0.f, 0.f, 0.f};
    f32x4 sum[FOLD ? MT : 1][FOLD ? NT : 1];          // FOLD: the finished shares
    int until = p.nk_split;                           // and the steps until the next one is finished
    if constexpr (FOLD) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int tt = 0; tt < NT; ++tt) sum[i][tt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    auto fold = [&]() {
        if constexpr (FOLD) {
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int tt = 0; tt < NT; ++tt) {
                    sum[i][tt] += acc[i][tt];
                    acc[i][tt] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
        }
    };

    Chunk fa[8], fb[2][NT];
    typedef __attribute__((address_space(3))) const char* lds_t;
    u32 vA[2], vB[NT];                                // this lane's read addresses in the stage that is read
    auto point_a = [&](u32 stage) { vA[0] = offA[0] + stage; vA[1] = offA[1] + stage; };
    auto point_b = [&](u32 stage) {
#pragma unroll
        for (int tt = 0; tt < NT; ++tt) vB[tt] = offB[tt] + stage;
    };
    auto read_a = [&](int j) {                        // A fragment of group j (slice j / MT, row subtile j % MT)
        fa[j % 8].u = *(__attribute__((address_space(3))) const u32x4*)((lds_t)(size_t)vA[j / MT] + (j % MT) * 2048);
    };
    auto read_b = [&](int s, int tt, int h) {         // half h (0, 1) of the B fragment of slice s
        if (BT) {
            if (h == 0) fb[s][tt].u = *(__attribute__((address_space(3))) const u32x4*)(lds_t)(size_t)(vB[tt] ^ (s ? 64u : 0u));
        } else {
            const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (s16x4 __attribute__((address_space(3)))*)((lds_t)(size_t)vB[tt] + s * 32 * BROW + h * 4 * BROW));
            const u32x2 d = *reinterpret_cast<const u32x2*>(&v);
            fb[s][tt].u[2 * h] = d[0];
            fb[s][tt].u[2 * h + 1] = d[1];
        }
    };

    // One contraction step; LEFT steps follow (at most STAGES are counted).  On entry the B fragments of slice 0 and the
    // first AHEAD A fragments have been requested.  The barrier stands AHEAD groups before the end: every fragment of the
    // tile is in registers by then and tile kt + 1 has landed; behind it that tile's first fragments are read.  Loads, at
    // most one per group, into stages that a barrier has freed: with as many stages of both operands (128-row tiles) the
    // weights of tile kt + STAGES behind the barrier and A of tile kt + STAGES - 1 in the first groups; with two stages of A
    // the weights of tile kt + 2 in the first groups, 1.75 steps ahead of their use, and A of that tile behind the barrier.
    constexpr bool EVEN = STAGES_A == STAGES;
    constexpr int NRB = 2 * NT;                       // halves of B fragments per slice
    const u32 B0 = lds_addr(lds), A0 = B0 + STAGES * BBYTES;
    u32 curA = A0, curB = B0;                         // stages of tile kt
    auto next_a = [&](u32 st) { return st + ABYTES == A0 + STAGES_A * ABYTES ? A0 : st + ABYTES; };
    auto next_b = [&](u32 st) { return st + BBYTES == A0 ? B0 : st + BBYTES; };
    auto step = [&](int kt, auto LEFTC) {
        constexpr int LEFT = decltype(LEFTC)::value;
        const u32 nxtA = next_a(curA), nxtB = next_b(curB);
        const u32 prvA = curA == A0 ? A0 + (STAGES_A - 1) * ABYTES : curA - ABYTES;  // (EVEN: of tile kt + STAGES - 1)
        const u32 aftB = next_b(nxtB);                                               // (of tile kt + 2)
#pragma unroll
        for (int j = 0; j < NG; ++j) {
            if (j == NG - AHEAD && LEFT >= 1) {
                constexpr int TILES = LEFT < 2 ? 0 : LEFT - 1 < STAGES - 2 ? LEFT - 1 : STAGES - 2;    // may be out
                __builtin_amdgcn_s_waitcnt(vmcnt_imm(EVEN ? TILES * (ADMA + BDMA) : LEFT < 2 ? 0 : BDMA));
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
                point_a(nxtA);
                point_b(nxtB);
            }
            if (j + AHEAD < NG) read_a(j + AHEAD);
            else if (LEFT >= 1) read_a(j + AHEAD - NG);
            if (j < MT) {
#pragma unroll
                for (int x = j * NRB / MT; x < (j + 1) * NRB / MT; ++x) read_b(1, x >> 1, x & 1);
            }
            if (j >= NG - AHEAD && LEFT >= 1) {
#pragma unroll
                for (int x = NRB / 4 * (j - NG + AHEAD); x < NRB / 4 * (j - NG + AHEAD + 1); ++x) read_b(0, x >> 1, x & 1);
            }
            const int s = j / MT, i = j % MT;
#pragma unroll
            for (int tt = 0; tt < NT; ++tt)
                acc[i][tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[s][tt].v, fa[j % 8].v, acc[i][tt], 0, 0, 0);
#pragma unroll
            for (int tt = 0; tt < NT; ++tt) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (EVEN) {
                if (j < ADMA && LEFT >= STAGES - 1) dma_a(kt + STAGES - 1, prvA, j);
                if (j >= NG - AHEAD && j - (NG - AHEAD) < BDMA && LEFT >= STAGES) dma_b(kt + STAGES, curB, j - (NG - AHEAD));
            } else {
                if (j < BDMA && LEFT >= 2) dma_b(kt + 2, aftB, j);
                if (j >= NG - AHEAD && LEFT >= 2) dma_a(kt + 2, curA, j - (NG - AHEAD));
            }
        }
        curA = nxtA;
        curB = nxtB;
        if (FOLD && --until == 0) {
            fold();
            until = p.nk_split;
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // the loads that stand before step 0: two tiles, or all but A of the last stage
    constexpr int BEFORE = EVEN ? STAGES - 1 : 2;
#pragma unroll
    for (int kt = 0; kt < BEFORE; ++kt) {
#pragma unroll
        for (int x = 0; x < BDMA; ++x) dma_b(kt, B0 + kt * BBYTES, x);
#pragma unroll
        for (int j = 0; j < ADMA; ++j) dma_a(kt, A0 + kt * ABYTES, j);
    }
    if (EVEN)
#pragma unroll
        for (int x = 0; x < BDMA; ++x) dma_b(BEFORE, B0 + BEFORE * BBYTES, x);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(vmcnt_imm((BEFORE - 1) * (ADMA + BDMA) + (EVEN ? BDMA : 0)));
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    point_a(A0);
    point_b(B0);
#pragma unroll
    for (int x = 0; x < NRB; ++x) read_b(0, x >> 1, x & 1);
#pragma unroll
    for (int j = 0; j < AHEAD; ++j) read_a(j);
    __builtin_amdgcn_sched_barrier(0);
    {
        auto tail = [&](int kt, auto IC) {
            constexpr int I = decltype(IC)::value;
            if constexpr (I < STAGES) step(kt + I, std::integral_constant<int, STAGES - 1 - I>());
        };
        int kt = 0;
        for (; kt + STAGES < nk; ++kt) step(kt, std::integral_constant<int, STAGES>());
        tail(kt, std::integral_constant<int, 0>());
        tail(kt, std::integral_constant<int, 1>());
        tail(kt, std::integral_constant<int, 2>());
        tail(kt, std::integral_constant<int, 3>());
        tail(kt, std::integral_constant<int, 4>());
    }

    // (a last share that is shorter, or nothing: the zeros change no sum, which begins at +0 and so is never -0)
    if constexpr (FOLD) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int tt = 0; tt < NT; ++tt) acc[i][tt] = sum[i][tt] + acc[i][tt];
    }

    // ---- epilogue: acc[i][tt][v] is row 16 i + l16 of the wavefront's rows, column 16 tt + 4 g + v of its columns
    if (SPLIT) {
        float* const part = p.part + (size_t)split * p.M * p.ldp;
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            const int m = m0 + WR * wm + 16 * i + l16;
#pragma unroll
            for (int tt = 0; tt < NT; ++tt) {
                const int col = n0 + BN / 4 * wn + 16 * tt + 4 * g;
                if (m < p.M && col < p.N) *reinterpret_cast<f32x4*>(part + (size_t)m * p.ldp + col) = acc[i][tt];
            }
        }
        return;
    }
    // (row-major C: ldc = its row length, c_panel = 64; panels of 64 columns: ldc = 64, c_panel = 64 M)
    auto c_at = [&](int m, int col) { return p.C + (size_t)(col >> 6) * p.c_panel + (size_t)m * p.ldc + (col & 63); };
    // two neighbouring subtiles are exchanged between odd and even groups of 16 lanes: the lane then holds eight
    // consecutive columns of one row
    auto swap16 = [&](u32& x, u32& y) {
        const auto r = __builtin_amdgcn_permlane16_swap(x, y, false, false);
        x = r[0];
        y = r[1];
    };
    const int c8 = 16 * (g & 1) + 8 * (g >> 1);         // first of the lane's eight columns in a pair of subtiles
    if constexpr (DUAL) {
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            const int m = m0 + WR * wm + 16 * i + l16;
            const float r = m < p.M ? p.colc[m] : 0.f;
            u32 d[2][2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                float h[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) h[v] = swiglu(r * acc[i][u][v], r * acc[i][u + 2][v]);
                d[u][0] = pack_bf16(h[0], h[1]);
                d[u][1] = pack_bf16(h[2], h[3]);
            }
            swap16(d[0][0], d[1][0]);
            swap16(d[0][1], d[1][1]);
            const int col = n0 + 32 * wn + c8;
            if (m < p.M && col < p.N)
                *reinterpret_cast<u32x4*>(c_at(m, col)) = u32x4{d[0][0], d[0][1], d[1][0], d[1][1]};
        }
    } else {
        f32x4 cc[NT], cb[NT];
        if (MODE == MODE_LN_PRE) {
#pragma unroll
            for (int tt = 0; tt < NT; ++tt) {
                const int col = n0 + BN / 4 * wn + 16 * tt + 4 * g;
                const bool ok = col < p.N;
                cc[tt] = ok ? *reinterpret_cast<const f32x4*>(p.colc + col) : f32x4{0.f, 0.f, 0.f, 0.f};
                cb[tt] = ok ? *reinterpret_cast<const f32x4*>(p.colb + col) : f32x4{0.f, 0.f, 0.f, 0.f};
            }
        }
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            const int m = m0 + WR * wm + 16 * i + l16;
            float r = 0.f, mu = 0.f;
            if (MODE == MODE_LN_PRE && m < p.M) {
                r = p.rowstat[2 * (size_t)m];
                mu = p.rowstat[2 * (size_t)m + 1];
            }
#pragma unroll
            for (int t2 = 0; t2 < NT; t2 += 2) {
                const int col = n0 + BN / 4 * wn + 16 * t2 + c8;
                const bool inside = m < p.M && col < p.N;
                f32x4 y[2] = {acc[i][t2], acc[i][t2 + 1]};
                if (MODE == MODE_LN_PRE) {
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int v = 0; v < 4; ++v) y[u][v] = fmaf(r, y[u][v] - mu * cc[t2 + u][v], cb[t2 + u][v]);
                }
                if (MODE == MODE_PLAIN && p.res != nullptr) {
                    // residual added in fp32 before the one rounding
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        u32 x0 = __float_as_uint(y[0][v]), x1 = __float_as_uint(y[1][v]);
                        swap16(x0, x1);
                        y[0][v] = __uint_as_float(x0);
                        y[1][v] = __uint_as_float(x1);
                    }
                    if (inside) {
                        const u32x4 rr = ldg16(p.res + (size_t)m * p.ldr + col);
                        *reinterpret_cast<u32x4*>(c_at(m, col)) =
                            u32x4{pack_bf16(y[0][0] + bf_lo(rr[0]), y[0][1] + bf_hi(rr[0])),
                                  pack_bf16(y[0][2] + bf_lo(rr[1]), y[0][3] + bf_hi(rr[1])),
                                  pack_bf16(y[1][0] + bf_lo(rr[2]), y[1][1] + bf_hi(rr[2])),
                                  pack_bf16(y[1][2] + bf_lo(rr[3]), y[1][3] + bf_hi(rr[3]))};
                    }
                    continue;
                }
                u32 d0 = pack_bf16(y[0][0], y[0][1]), d1 = pack_bf16(y[0][2], y[0][3]);
                u32 e0 = pack_bf16(y[1][0], y[1][1]), e1 = pack_bf16(y[1][2], y[1][3]);
                swap16(d0, e0);
                swap16(d1, e1);
                if (inside) *reinterpret_cast<u32x4*>(c_at(m, col)) = u32x4{d0, d1, e0, e1};
            }
        }
    }
}

}  // namespace bb
