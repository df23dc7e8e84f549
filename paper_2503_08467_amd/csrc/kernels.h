// Internal launchers of the MoE layer kernels (called by the C ABI after validation).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace moe {

int device_cus();  // CUs of the current device

// Tile constants shared by the packer and the grouped GEMM.
constexpr int kInnerAlign = 128;  // packed inner width is a multiple of this
constexpr int kDispatchChunk = 1024;  // assignments per dispatch workgroup

hipError_t launch_route(const void* x, bool bf16, int64_t T, int h, const void* wg, int E, int k,
                        const float* bias, int64_t bias_stride, int renorm, int32_t* idx, float* w,
                        hipStream_t s);

// Step 2's outputs written by the routing launch itself (moe_dispatch's counts, offsets,
// row_src, pos_of; no x_perm).
struct RouteDispatchOut {
    int32_t* counts;
    int32_t* offsets;
    int32_t* row_src;
    int32_t* pos_of;
};

// Steps 1 and 2 in one launch (only when route_groups, see shapes.h).
hipError_t launch_route_dispatch(const void* x, bool bf16, int64_t T, int h, const void* wg, int E, int k, const float* bias,
                                 int64_t bias_stride, int renorm, int32_t* idx, float* w, RouteDispatchOut out,
                                 hipStream_t s);

hipError_t launch_dispatch(const int32_t* idx, int64_t T, int k, int E, const void* x, int elem_bytes,
                           int h, int32_t* counts, int32_t* offsets, int32_t* row_src,
                           int32_t* pos_of, void* x_perm, int32_t* ws, hipStream_t s);

hipError_t launch_pack(const void* w1, const void* w3, const void* w2, int E, int64_t h, int64_t F,
                       int64_t col0, int64_t f, int64_t fp, int elem_bytes, void* w1t, void* w3t,
                       void* w2t, hipStream_t s);

hipError_t launch_ffn(const void* x_perm, const int32_t* offsets, int64_t A_max, int E, int h,
                      int64_t fp, int act, bool bf16, const void* w1t, const void* w3t,
                      const void* w2t, void* y_perm, bool y_bf16, void* hbuf, hipStream_t s);

hipError_t launch_ffn_gather(const void* x, int64_t T, const int32_t* row_src, const int32_t* offsets, int64_t A_max,
                             int E, int h, int64_t fp, int act, bool bf16, const void* w1t, const void* w3t,
                             const void* w2t, void* y_perm, bool y_bf16, void* hbuf, hipStream_t s);

// launch_ffn_gather followed by launch_combine; where hands_over_sums the second product's fp32
// sums go straight to the combine and y_perm is not written (*y_perm_written).
hipError_t launch_ffn_gather_combine(const void* x, int64_t T, const int32_t* row_src, const int32_t* offsets, int k,
                                     int E, int h, int64_t fp, int act, bool bf16, const void* w1t, const void* w3t,
                                     const void* w2t, void* y_perm, bool y_bf16, const int32_t* pos_of,
                                     const float* topk_w, void* y, bool out_bf16, void* hbuf, hipStream_t s,
                                     bool* y_perm_written);

hipError_t launch_ffn_top1(const void* x, int64_t T, const int32_t* row_src, const float* topk_w,
                           const int32_t* offsets, int64_t A_max, int E, int h, int64_t fp, int act, bool bf16,
                           const void* w1t, const void* w3t, const void* w2t, void* y, bool y_bf16, void* hbuf,
                           hipStream_t s);

hipError_t launch_ffn_per_expert(const void* x_perm, const int32_t* offsets, const int32_t* offsets_host,
                                 int64_t A_max, int E, int h, int64_t fp, int act, bool bf16, const void* w1t,
                                 const void* w3t, const void* w2t, void* y_perm, bool y_bf16, void* hbuf,
                                 hipStream_t s);

// moe_expert_ffn_shard with its workspace in the library's static per-device array.
hipError_t launch_ffn_noalloc(const void* x_perm, const int32_t* offsets, int64_t A_max, int E, int h, int64_t fp,
                              int act, bool bf16, const void* w1t, const void* w3t, const void* w2t, void* y_perm,
                              bool y_bf16, hipStream_t s);

hipError_t launch_combine(const void* y_perm, bool y_bf16, const int32_t* pos_of, const float* w,
                          int64_t T, int k, int h, void* y, bool out_bf16, hipStream_t s);

}  // namespace moe
