// Kernel launches across translation units.  The library is built from several
// sources compiled side by side (one per family of kernel instantiations);
// bb_api.hip owns validation, workspace and variant selection and reaches the
// kernels through the functions declared here.  A launch function only enqueues:
// the caller checks hipGetLastError().
#pragma once
#include <hip/hip_runtime.h>

namespace bb {

struct GemmArgs;
struct StreamArgs;
struct StreamTArgs;
struct AttnArgs;
struct NestArgs;
struct FewArgs;
struct SliceArgs;

// gemm_kernel<MODE, bm, full, odd, split, bt> on `grid` workgroups (defined per MODE and per weight
// layout in bb_gemm_inst_*.hip); split launches exist for MODE_PLAIN and MODE_GATEUP only, with bm = 128
template <int MODE, bool BT>
void gemm_dispatch(int bm, bool full, bool odd, bool split, dim3 grid, hipStream_t st, const GemmArgs& a);

// product_kernel<MODE, bm, bn, parts, bt>: products without a norm prologue (bn = 128 and shares: MODE_PLAIN)
template <int MODE, bool BT>
void product_dispatch(int bm, int bn, int parts, dim3 grid, hipStream_t st, const GemmArgs& a);

// splitk_reduce_kernel<mode> (mode = MODE_PLAIN or MODE_GATEUP)
void splitk_reduce_dispatch(int mode, const float* part, const float* ssqpart, unsigned short* C, int M, int N, int K,
                            int ldp, int ldc, int nsplit, float eps, const unsigned short* res, int ldr,
                            hipStream_t st);

// products of up to 64 mt rows cut into equal shares of the weight stream (bt: weights transposed; nt: loaded past the caches), and the kernel that
// adds the shares and applies the epilogue (mode = MODE_PLAIN, MODE_GATEUP_PRE or MODE_LN_PRE)
void few_rows_launch(int mt, bool bt, bool nt, int grid, hipStream_t st, const FewArgs& a);
void few_reduce_launch(int mode, hipStream_t st, const FewArgs& a, const float* rowstat, unsigned short* C, int M,
                       const unsigned short* res);

// streaming kernels: workgroups of the kernel one compute unit can hold (hipError_t in *err), launch
// (row-major weights: ffn_stream_kernel<mt>, mt = 1 or 2 groups of 16 rows)
int stream_resident(int mt, hipError_t* err);
void stream_launch(int mt, int G, hipStream_t st, const StreamArgs& a);
int stream_t_resident(int lds_bytes, hipError_t* err);
void stream_t_launch(int G, int lds_bytes, hipStream_t st, const StreamTArgs& a);

// fully fused nest for small model dimensions: ffn_nest_kernel<nd>, nd = blocks of 128 model channels (2 or 4)
void nest_launch(int nd, int grid, hipStream_t st, const NestArgs& a);

// the nest with its hidden blocks in parallel: ffn_slice_kernel, then the sum of its partial outputs (+ R) into Y
void slice_launch(bool bt, hipStream_t st, const SliceArgs& a, unsigned short* Y, const unsigned short* R);

// attention: tiled kernel (ksplit > 1: split keys + combine kernel), one-query and few-query streaming kernels
// (defined per pair of head dimensions in bb_attn_inst_*.hip)
template <int DK, int DV>
void attn_tiled_launch(int tail, int nw, int ksplit, bool flat, dim3 grid, dim3 block, hipStream_t st, const AttnArgs& a);
template <int DK, int DV>
void attn_decode_launch(dim3 grid, hipStream_t st, const AttnArgs& a);
template <int DK, int DV>       // mt = 1 or 2 groups of 16 queries
void attn_group_launch(int mt, dim3 grid, hipStream_t st, const AttnArgs& a);

}  // namespace bb
