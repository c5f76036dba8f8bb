// Products of a few dozen to 256 rows with a large weight matrix: bound by the weight stream, not by the matrix cores.
//
//   part[tile][slot][row][128] = partial sums of A[Mr, K] * B[K, N]   (few_rows_kernel)
//   epilogue over the sum of a tile's slots                          (few_reduce_kernel)
//
// Row counts in this range leave the tiled kernels with fewer tiles than compute units, and splitting a tile's
// contraction evenly still fits the 256 compute units badly (86 tiles: two splits use 172 of them) with one step of
// weights in flight.  Here the (tile of 128 columns, 64 contraction indices) items of the whole product lie in one
// line that is cut into equal ranges, one per workgroup and compute unit; a range may end in the middle of a tile and
// go on in the next.  All rows belong to every workgroup, so each weight is read from memory once.
//
// What bounds it is the number of weight bytes in flight: a ring of NS stages (A: 64 MT rows, B: 128 columns, 64
// contraction indices each) in LDS is filled with load-to-LDS instructions NS - 1 stages ahead, 48 to 80 KiB of
// weights per compute unit.  128 columns per tile keep the partial sums small (rows x 512 bytes per workgroup and
// tile touched): they are written to and read back from the caches.
//
// The load-to-LDS instructions are written in assembly: they write no register, and the compiler would otherwise
// wait for the whole ring before the first LDS read of a stage (it tells the stages apart only as separate arrays
// of a loop unrolled NS times).  The waits are explicit: loads return in order, so at most (NS - 2) stages' worth
// outstanding means that the stage about to be read has landed; the partial sums' stores only make that stricter.
#pragma once
#include "bb_gemm.h"

namespace bb {

constexpr int FEW_MAXMT = 4;             // groups of 64 rows
constexpr int FEW_THREADS = 512;         // eight wavefronts, 2 (rows) x 4 (columns)
constexpr int FEW_COLS = 128;            // columns per tile
constexpr int FEW_RROWS = 8;             // rows per workgroup of the reduction

struct FewArgs {
    const u16* A;        // [Mr, K]
    const u16* B0;       // [K, N] or, transposed, [N, K]
    const u16* B1;       // second weight matrix of the same shape, or null
    float* part;         // [tiles][slots][Mr][FEW_COLS]
    int Mr, N, K;
    int tiles_n;         // tiles of 128 columns per weight matrix
    int nk;              // items (64 contraction indices) per tile
    int items, per;      // items in all and per workgroup
    int slots;           // slots per tile
};

// ring stages that fit the LDS next to nothing else
constexpr int few_stages(int mt) { return mt == 1 ? 6 : mt == 4 ? 3 : 4; }

// One load-to-LDS instruction: lane i copies the 16 bytes at base + voff (per lane) + soff to LDS byte address
// lds + 16 i.  The scalar move to m0 needs one wait state before the instruction that reads it.
__device__ __forceinline__ void few_dma(u32x4 rs, u32 voff, u32 soff, u32 lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :: "s"(lds), "v"(voff), "s"(rs), "s"(soff) : "memory", "m0");
}
// the same with the non-temporal cache policy: the weights are read once and should not push the rows and the partial
// sums out of the L2 (100 rows x 4096 x 11008: 87.8 -> 83.1 us, 48 rows 75.9 -> 71.3)
__device__ __forceinline__ void few_dma_nt(u32x4 rs, u32 voff, u32 soff, u32 lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds"
                 :: "s"(lds), "v"(voff), "s"(rs), "s"(soff) : "memory", "m0");
}
__device__ __forceinline__ u32x4 few_rsrc(const void* base, size_t bytes) {
    const u32 lo = __builtin_amdgcn_readfirstlane((u32)(uintptr_t)base);
    const u32 hi = __builtin_amdgcn_readfirstlane((u32)((uintptr_t)base >> 32) & 0xffffu);
    const u32 nb = __builtin_amdgcn_readfirstlane((u32)bytes);
    return u32x4{lo, hi, nb, 0x00020000u};
}

#ifndef BB_HOST_ONLY
template <int MT, bool BT>
__global__ __launch_bounds__(FEW_THREADS) void few_rows_kernel(const FewArgs p) {
    constexpr int NS = few_stages(MT);
    constexpr int ACH = 64 * MT * 8, BCH = 64 * 16;             // 16-byte chunks per stage
    constexpr int NLD = MT + 2;                                 // load-to-LDS instructions per wavefront and stage
    __shared__ u32x4 ring[NS * (ACH + BCH)];
    const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int l32 = lane & 31, lhi = lane >> 5;
    const int wm = w >> 2, wn = w & 3;
    const int g = blockIdx.x;
    const int i0 = g * p.per, n = min(p.per, p.items - i0);
    if (n <= 0) return;
    const u32 lds0 = __builtin_amdgcn_readfirstlane(lds_addr(ring));
    const u32x4 rsA = few_rsrc(p.A, (size_t)p.Mr * p.K * 2);
    const size_t bbytes = (size_t)p.K * p.N * 2;
    const int ldb = BT ? p.K : p.N;

    // ---- load role (same LDS layouts as the tiled kernels).  A: instruction j fills tile rows 8 (w + 8 j) + 0..7.
    // Groups of eight rows past the last row are not loaded: whatever lies there only enters rows of the result that
    // are not stored (the last group of 64 rows is the only one that can have such rows, so a wavefront issues MT or
    // MT - 1 of these instructions).  Rows past the last one in a loaded group read the last row; chunks past the
    // contraction read its last chunk (and are zeroed as fragments).
    const bool allA = 8 * (w + 8 * (MT - 1)) < p.Mr;
    u32 voA[MT];
    int kcA[MT];
#pragma unroll
    for (int j = 0; j < MT; ++j) {
        const int row = 8 * (w + 8 * j) + (lane >> 3);
        kcA[j] = 8 * ((lane & 7) ^ ((row >> 1) & 7));
        voA[j] = (u32)min(row, p.Mr - 1) * (u32)p.K * 2u;
    }
    // B: instruction q fills four contraction rows 4 (2 w + q) + 0..3 of 256 bytes (BT: eight rows of 128 bytes)
    u32 voB[2];
    int kB[2];
    u32x4 rsB;
    // Transposed weights: a stage reads 128 bytes of 128 rows that lie 2 K bytes apart.  With K a power of two and a tile
    // per workgroup, all workgroups would walk the same few memory channels together, so the items of a tile start
    // at another place of the contraction in every tile (ROT x 128 bytes further).
    constexpr int ROT = 5;
    auto item_k = [&](int tile, int k) {                        // first contraction index of item k of a tile
        if (!BT) return k * GEMM_BK;
        const int r = k + (tile * ROT) % p.nk;
        return (r >= p.nk ? r - p.nk : r) * GEMM_BK;
    };
    int lt = i0 / p.nk, lk = i0 - lt * p.nk, ls = 0;            // the item and stage loaded next
    int ln0 = 0;
    auto load_tile = [&]() {                                    // lane offsets within the tile `lt`
        const bool second = lt >= p.tiles_n;
        rsB = few_rsrc(second ? p.B1 : p.B0, bbytes);
        ln0 = (second ? lt - p.tiles_n : lt) * FEW_COLS;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if (BT) {
                const int row = 8 * (2 * w + q) + (lane >> 3);
                kB[q] = 8 * ((lane & 7) ^ ((row >> 1) & 7));
                voB[q] = (u32)min(ln0 + row, p.N - 1) * (u32)ldb * 2u;
            } else {
                const int chunk = (lane & 15) ^ ((lane >> 4) << 2);
                kB[q] = 4 * (2 * w + q) + (lane >> 4);
                voB[q] = (u32)min(ln0 + 8 * chunk, p.N - 8) * 2u;
            }
        }
    };
    load_tile();
    auto issue = [&]() {
        const int k0 = item_k(lt, lk);
        const u32 sa = lds0 + (u32)ls * (ACH + BCH) * 16u, sb = sa + ACH * 16u;
        if (k0 + GEMM_BK <= p.K) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                if (BT) few_dma_nt(rsB, voB[q] + 2u * kB[q], (u32)k0 * 2u, sb + (2 * w + q) * 1024u);
                else few_dma_nt(rsB, voB[q] + (u32)(lane >> 4) * (u32)ldb * 2u, (u32)(k0 + 4 * (2 * w + q)) * (u32)ldb * 2u,
                             sb + (2 * w + q) * 1024u);
            }
#pragma unroll
            for (int j = 0; j < MT; ++j)
                if (j < MT - 1 || allA) few_dma(rsA, voA[j] + 2u * kcA[j], (u32)k0 * 2u, sa + (w + 8 * j) * 1024u);
        } else {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const u32 vo = BT ? voB[q] + 2u * (u32)min(k0 + kB[q], p.K - 8)
                                  : voB[q] + (u32)min(k0 + kB[q], p.K - 1) * (u32)ldb * 2u;
                few_dma_nt(rsB, vo, 0u, sb + (2 * w + q) * 1024u);
            }
#pragma unroll
            for (int j = 0; j < MT; ++j)
                if (j < MT - 1 || allA)
                    few_dma(rsA, voA[j] + 2u * (u32)min(k0 + kcA[j], p.K - 8), 0u, sa + (w + 8 * j) * 1024u);
        }
        ls = ls + 1 == NS ? 0 : ls + 1;
        if (++lk == p.nk) {
            lk = 0;
            ++lt;
            load_tile();
        }
    };

    // ---- fragment role: wavefront (wm, wn) owns rows 32 MT wm + ... and columns 32 wn + ... of the tile
    int offB;
    {
        const int b = lane >> 4, ip = lane & 15;
        const int r = 8 * (b >> 1) + (ip >> 2), piece = ip & 3;
        const int chunk = 4 * wn + 2 * (b & 1) + (piece >> 1);
        offB = r * 256 + ((chunk ^ ((r & 3) << 2)) << 4) + 8 * (piece & 1);
    }
    f32x16 acc[MT];
    auto clear = [&]() {
#pragma unroll
        for (int s = 0; s < MT; ++s)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[s][v] = 0.f;
    };
    auto compute = [&](int stage, int k0) {
        const u32x4* const sA = ring + stage * (ACH + BCH);
        const u32x4* const sB = sA + ACH;
        Chunk fa[4][MT], fb[4];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const int kc = 2 * ks + lhi;
            if (BT) {
                fb[ks].u = sB[lds_pos(32 * wn + l32, kc)];
            } else {
                const char* q = reinterpret_cast<const char*>(sB) + offB + ks * (16 * 256);
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(q));
                const s16x4 hi =
                    __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(q + 4 * 256));
                const u32x2 l2 = *reinterpret_cast<const u32x2*>(&lo), h2 = *reinterpret_cast<const u32x2*>(&hi);
                fb[ks].u = u32x4{l2[0], l2[1], h2[0], h2[1]};
            }
#pragma unroll
            for (int s = 0; s < MT; ++s) fa[ks][s].u = sA[lds_pos(32 * MT * wm + 32 * s + l32, kc)];
        }
        if (k0 + GEMM_BK > p.K) {                                // ragged contraction: what lies past it counts zero
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const bool in = k0 + 16 * ks + 8 * lhi < p.K;
                if (!in) {
                    fb[ks].u = zero4();
#pragma unroll
                    for (int s = 0; s < MT; ++s) fa[ks][s].u = zero4();
                }
            }
        }
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
            for (int s = 0; s < MT; ++s)
                acc[s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[ks][s].v, fb[ks].v, acc[s], 0, 0, 0);
    };
    auto store = [&](int tile) {
        const int slot = g - tile * p.nk / p.per;
        float* const dst = p.part + ((size_t)tile * p.slots + slot) * p.Mr * FEW_COLS + 32 * wn + 4 * (l32 >> 2);
        const int e = l32 & 3;
#pragma unroll
        for (int s = 0; s < MT; ++s)
#pragma unroll
            for (int vg = 0; vg < 4; ++vg) {
                float y[4] = {acc[s][4 * vg], acc[s][4 * vg + 1], acc[s][4 * vg + 2], acc[s][4 * vg + 3]};
                quad_transpose_f32(y, (e & 2) != 0, (e & 1) != 0);
                const int m = 32 * MT * wm + 32 * s + 8 * vg + 4 * lhi + e;
                if (m < p.Mr) *reinterpret_cast<f32x4*>(dst + (size_t)m * FEW_COLS) = f32x4{y[0], y[1], y[2], y[3]};
            }
    };

    const bool rows_w = 32 * MT * wm < p.Mr;                     // (up to 32 rows: four wavefronts only load)
    int ct = lt, ck = lk, cs = 0;                                // the item and stage multiplied next
    for (int s = 0; s < min(n, NS - 1); ++s) issue();
    clear();
    for (int i = 0; i < n; ++i) {
        // item i has landed (all but the NS - 2 stages requested after it), and every wavefront is done with the
        // stage that the next request overwrites
        if (i + NS - 2 < n && allA)
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"((NS - 2) * NLD) : "memory");
        else if (i + NS - 2 < n)
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"((NS - 2) * (NLD - 1)) : "memory");
        else
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (i + NS - 1 < n) issue();
        if (rows_w) compute(cs, item_k(ct, ck));
        cs = cs + 1 == NS ? 0 : cs + 1;
        if (++ck == p.nk || i == n - 1) {
            if (rows_w) store(ct);
            clear();
            ck = 0;
            ++ct;
        }
    }
}

// Adds a tile's slots in order and applies the epilogue:
//   MODE_PLAIN       C = bf16(sum [+ residual])
//   MODE_GATEUP_PRE  C = bf16(SiLU(r P) (r Q)), r = rowstat[m]; the W3 product lies tiles_n tiles behind the W1 product
//   MODE_LN_PRE      C = bf16(r (P - mu c) + b), (r, mu) = rowstat[2 m ...]; c and b are the rows M and M + 1 of the
//                    product, whose operand rows are gamma and beta themselves (Rule 5's column vectors out of the
//                    same pass over the weights)
// One workgroup per tile of 128 columns and FEW_RROWS rows, a thread per row and four columns: where a tile's shares lie
// is the same for the whole workgroup (scalar arithmetic), and the loads of all shares are in flight together - the
// kernel is bound by its launch and one round trip to memory (4 to 5 us).
template <int MODE>
__global__ __launch_bounds__(32 * FEW_RROWS) void few_reduce_kernel(const FewArgs p, const float* rowstat, u16* C, int M,
                                                                   const u16* res) {
    constexpr int BATCH = MODE == MODE_PLAIN ? 8 : 4;            // shares loaded together
    const int tile = blockIdx.x, q4 = 4 * (threadIdx.x & 31), c0 = tile * FEW_COLS + q4;
    const int m = min((int)(blockIdx.y * FEW_RROWS + (threadIdx.x >> 5)), M - 1);   // (the last row's threads may repeat)
    if (c0 >= p.N) return;
    const size_t stride = (size_t)p.Mr * FEW_COLS;
    auto shares = [&](int tl) {
        const u32 first = (u32)tl * p.nk, per = p.per;
        return (int)((first + p.nk - 1) / per - first / per) + 1;
    };
    auto sum = [&](int tl, int ns, int row) {                    // in order, BATCH loads at a time
        const float* const src = p.part + ((size_t)tl * p.slots * p.Mr + row) * FEW_COLS + q4;
        f32x4 s = {0, 0, 0, 0};
        for (int i = 0; i < ns; i += BATCH) {
            f32x4 v[BATCH];
#pragma unroll
            for (int j = 0; j < BATCH; ++j) v[j] = *reinterpret_cast<const f32x4*>(src + min(i + j, ns - 1) * stride);
#pragma unroll
            for (int j = 0; j < BATCH; ++j)
                if (i + j < ns) s += v[j];
        }
        return s;
    };
    const int ns = shares(tile);
    f32x4 y = sum(tile, ns, m);
    if (MODE == MODE_GATEUP_PRE) {
        const f32x4 q = sum(tile + p.tiles_n, shares(tile + p.tiles_n), m);
        const float r = rowstat[m];
#pragma unroll
        for (int j = 0; j < 4; ++j) y[j] = swiglu(r * y[j], r * q[j]);
    } else if (MODE == MODE_LN_PRE) {
        const f32x4 cc = sum(tile, ns, M), cb = sum(tile, ns, M + 1);
        const float r = rowstat[2 * m], mu = rowstat[2 * m + 1];
#pragma unroll
        for (int j = 0; j < 4; ++j) y[j] = fmaf(r, y[j] - mu * cc[j], cb[j]);
    } else if (res != nullptr) {
        const u32x2 rr = *reinterpret_cast<const u32x2*>(res + (size_t)m * p.N + c0);
        y += f32x4{bf_lo(rr[0]), bf_hi(rr[0]), bf_lo(rr[1]), bf_hi(rr[1])};
    }
    if (blockIdx.y * FEW_RROWS + (threadIdx.x >> 5) < (u32)M)    // (a repeated row is not stored twice: C may be the residual)
        *reinterpret_cast<u32x2*>(C + (size_t)m * p.N + c0) = u32x2{pack_bf16(y[0], y[1]), pack_bf16(y[2], y[3])};
}
#endif  // BB_HOST_ONLY

}  // namespace bb
