// Host-side launch functions, one per kernel family.  Each returns 0 when every launch was
// accepted and -1 otherwise.  Arguments have been validated by the C-ABI layer (pdelta_api.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pdelta.h"

namespace pdelta {

// Whether pack reads the weights of a call, this many in each matrix, as non-temporal: from 40 MiB on, where two matrices and
// what was there before no longer share the memory-side cache.  us with ordinary loads and with non-temporal ones, three sets of
// inputs in turn: four layers of 1600 x 2176 (27 MiB) 18.7 and 21.4, seven of 768 x 3968 (41 MiB) 23.4 and 24.0, 2752 x 5632 with one
// scale (30 MiB) 17.2 and 18.0; six of 446 x 9216 (47 MiB) 27.0 and 24.8, 7552 x 4096 (59 MiB) 29.1 and 27.0, 10560 x 3968 (80 MiB)
// 38.5 and 37.0.  Out of memory non-temporal loads gain at every size (the first three: 24.4 and 22.0, 28.6 and 24.6, 20.4 and 18.0).
inline bool streams_weights(int64_t weights) { return weights * 2 >= (int64_t)40 << 20; }

// Bytes of fp64 partial sums pdelta_pack writes for these dimensions.
size_t pack_workspace_bytes(int64_t d_out, int64_t d_in);

int launch_pack_dispatch(int w_dtype, const void* W_f, const void* W_b, int64_t d_out,
                         int64_t d_in, uint32_t* B_packed, uint16_t* v_row, uint16_t* v_col,
                         void* workspace, hipStream_t stream);

// Device address of the library's own scratch array (kPackScratchBytes, one copy per GPU) on the
// current device; looked up once per device.  Returns 0, or -1 when the runtime refuses.
constexpr size_t kPackScratchBytes = (size_t)16 << 20;
int pack_static_scratch(void** ptr);

// Batched pack: geometry helpers shared by the plan (host) and the launcher.
int pack_batch_tile_blocks(int64_t d_out, int tallest);
int pack_batch_tallest(const ::pdelta_pack_job* jobs, int n_jobs);
int64_t pack_batch_tiles(int64_t d_out, int64_t d_in, int tile_blocks);
int64_t pack_batch_fin_blocks(int64_t d_out, int64_t d_in);
int launch_pack_batch(int w_dtype, const ::pdelta_pack_job* jobs_host, const ::pdelta_pack_job* jobs_device,
                      int n_jobs, hipStream_t stream);

int launch_patch_batch(int w_dtype, const ::pdelta_layer* layers_host, const ::pdelta_layer* layers_device,
                       int n_layers, hipStream_t stream);

int launch_patch_dispatch(int w_dtype, int axis, const void* W_b, const uint32_t* B_packed,
                          const uint16_t* v, void* W_out, int64_t d_out, int64_t d_in,
                          hipStream_t stream);

// Decode-shaped layer (few tokens): HBM-bound streaming kernel.  M <= kSkinnyMaxM.
constexpr int kSkinnyMaxM = 64;
int launch_linear_skinny(int x_dtype, int y_dtype, int axis, const void* X, const void* W_b,
                         const uint32_t* B_packed, const uint16_t* v, void* Y, int64_t M,
                         int64_t d_out, int64_t d_in, hipStream_t stream);

// The same with blockwise scales v[row * v_stride + (input >> g_shift)] (v_stride = 0: the rows
// share the scales; g_shift = 31: one group spans all of d_in).
int launch_linear_skinny_group(int x_dtype, int y_dtype, const void* X, const void* W_b,
                               const uint32_t* B_packed, const uint16_t* v, void* Y, int64_t M,
                               int64_t d_out, int64_t d_in, int v_stride, int g_shift, hipStream_t stream);
// Which kernel takes a decode call (axis 2: blockwise scales), and of the one with direct loads how many tiles of 16 output
// rows a workgroup takes.
enum DecodeKernel { kDecodeRegisters, kDecodeStaged, kDecodeDirect };
struct DecodeRoute { DecodeKernel kernel; int rows; };
DecodeRoute linear_skinny_route(int x_dtype, int axis, int64_t M, int64_t d_out, int64_t d_in, int g_shift);
// The kernel with direct loads into LDS: d_in a multiple of 128, rows of 1 to 3 tiles.
int launch_linear_skinny_dma(int x_dtype, int y_dtype, int axis, const void* X, const void* W_b, const uint32_t* B_packed,
                             const uint16_t* v, void* Y, int64_t M, int64_t d_out, int64_t d_in, int v_stride, int g_shift,
                             int rows, hipStream_t stream);
// Prefill: may tiles be computed in parts of d_in, and the memory for their sums (linear_gemm_workspace_bytes).
// Without the memory the same sums are formed by one workgroup per tile.
struct PrefillSplit { bool allowed; void* workspace; };
int launch_linear_gemm_group(int x_dtype, int y_dtype, const void* X, const void* W_b,
                             const uint32_t* B_packed, const uint16_t* v, void* Y, int64_t M,
                             int64_t d_out, int64_t d_in, int v_stride, int g_shift, PrefillSplit ps,
                             hipStream_t stream);
int launch_patch_group(int w_dtype, const void* W_b, const uint32_t* B_packed, const uint16_t* v,
                       void* W_out, int64_t d_out, int64_t d_in, int v_stride, int g_shift,
                       hipStream_t stream);
// pack with blockwise scales: signs + fp64 block sums (per row), then the scales; `workspace` is
// needed only when the rows share the scales (one partial sum per row and group).
size_t pack_group_workspace_bytes(int64_t d_out, int64_t d_in, int64_t group, int shared_rows);
int launch_pack_group(int w_dtype, const void* W_f, const void* W_b, int64_t d_out, int64_t d_in,
                      int64_t group, int shared_rows, uint32_t* B_packed, uint16_t* v, void* workspace,
                      hipStream_t stream);

// Several decode-shaped layers in one launch.  Returns 1 when the batched kernel does not apply
// (the caller then launches layer by layer), else 0 / -1.
int launch_linear_skinny_batch(int x_dtype, int y_dtype, const ::pdelta_layer* layers_host,
                               const ::pdelta_layer* layers_device, int n_layers, int64_t M,
                               hipStream_t stream);

// R requests (one token each) that share W_b and each have their own delta (more than 16 requests
// run in chunks of 16).  axis 0 / 1: one mode for all requests; 2: variants[r].axis per request.
// Returns 1 when the fused kernel does not apply (d_in % 128 != 0), else 0 / -1.
int launch_linear_variants(int x_dtype, int y_dtype, int axis, const void* X, const void* W_b,
                           const ::pdelta_variant* variants_device, int R, void* Y, int64_t d_out,
                           int64_t d_in, hipStream_t stream);

// dL/dv from dY (training of the scale vectors).  Workspace: partial sums per token tile, plus
// the transposed sign bits in column mode.
size_t grad_v_workspace_bytes(int64_t M, int64_t d_out, int64_t d_in, int axis);
// The same with partial sums for every part of a split contraction (at least the size above).
size_t grad_v_split_workspace_bytes(int64_t M, int64_t d_out, int64_t d_in, int axis);
int launch_grad_v(int dtype, int axis, const void* X, const void* dY, const uint32_t* B_packed, float* grad,
                  int64_t M, int64_t d_out, int64_t d_in, void* workspace, size_t workspace_bytes, hipStream_t stream);

// Prefill-shaped layer (many tokens): MFMA tile kernel.
size_t linear_gemm_workspace_bytes(int64_t M, int64_t d_out, int64_t d_in, int x_dtype);
int launch_linear_gemm(int x_dtype, int y_dtype, int axis, const void* X, const void* W_b,
                       const uint32_t* B_packed, const uint16_t* v, void* Y, int64_t M,
                       int64_t d_out, int64_t d_in, PrefillSplit ps, hipStream_t stream);

// The same on 64 x 64 tiles with the work of a workgroup split by role; d_in a multiple of 128.  axis 2: blockwise scales.
int launch_linear_gemm_roles(int x_dtype, int y_dtype, int axis, const void* X, const void* W_b, const uint32_t* B_packed,
                             const uint16_t* v, void* Y, int64_t M, int64_t d_out, int64_t d_in, int v_stride, int g_shift,
                             hipStream_t stream);

// The same on 256 x 256 tiles with direct loads into LDS; axis 2: blockwise scales.  The first `whole`
// tiles are computed in one go, the other `split` ones in `parts` pieces of d_in each, whose fp32
// sums go through the workspace.  parts = 0: another kernel is the better one, or the only one.
struct BigSplit { int whole, split, parts; };
BigSplit linear_gemm_big_split(int64_t M, int64_t d_out, int64_t d_in, int x_dtype, int axis, bool split_allowed);
// Which kernel takes a prefill call (axis 2: blockwise scales): 256 x 256 tiles as `split` says, 64 x 64 tiles with roles
// or a ring of steps in flight, 128 x 128, or 256 x 128 pipelined or with two workgroups per CU.
enum PrefillKernel { kPrefillTiles256, kPrefillRoles, kPrefillSmall, kPrefillShort, kPrefillPipelined, kPrefillTwoPerCu };
struct PrefillRoute { PrefillKernel kernel; BigSplit split; };
PrefillRoute linear_gemm_route(int x_dtype, int axis, int64_t M, int64_t d_out, int64_t d_in, bool may_split);
int launch_linear_gemm_big(int x_dtype, int y_dtype, int axis, const void* X, const void* W_b,
                           const uint32_t* B_packed, const uint16_t* v, void* Y, int64_t M, int64_t d_out,
                           int64_t d_in, int v_stride, int g_shift, void* workspace, BigSplit sp, hipStream_t stream);

// Measurement builds of the pipelined prefill kernel (bf16 operands, row scales): bit 0 of `parts`
// keeps the steady loop's global loads, bit 1 conversion and LDS writes, bit 2 fragment reads,
// bit 3 the MFMAs; 15 is that kernel whole (a library call of the same shape may run another, see
// linear_gemm_big_split).  Returns -2 for a combination that is not built.
int launch_linear_gemm_parts(int parts, int y_dtype, const void* X, const void* W_b, const uint32_t* B_packed,
                             const uint16_t* v, void* Y, int64_t M, int64_t d_out, int64_t d_in,
                             hipStream_t stream);

// Integer tuning knobs from the environment variable PDELTA_TUNE ("key=value,key=value");
// returns `fallback` when the key is absent.  Every C-ABI entry point that launches opens a
// TuneScope, which reads the variable once for the whole call.
struct TuneScope {
    TuneScope();
    ~TuneScope();
    TuneScope(const TuneScope&) = delete;
    TuneScope& operator=(const TuneScope&) = delete;
};
int tune_value(const char* key, int fallback);

// Kernels that use more dynamic LDS than the default limit have to opt in once per device.
// `done_mask` is a static word of the call site (one bit per device): the attribute is set on
// the first launch on a device and never again.  Returns 0, or -1 when the runtime refuses.
int opt_in_dynamic_lds(const void* kernel, int bytes, unsigned* done_mask);

}  // namespace pdelta
