// loadShard: cut this device's inner slice out of every expert's weights (W_i by columns,
// W_o by the matching rows) and store it K-contiguous for the grouped GEMM:
//   W1^T[e][n][j] = W1[e][j][col0 + n]        n < f, zero for f <= n < fp
//   W2^T[e][c][n] = W2[e][col0 + n][c]        n < f, zero for f <= n < fp
// Both are batched 2-D transposes of a sub-matrix with zero padding, done through an LDS
// tile so that reads and writes are both row-contiguous.
//
// bf16 weights are stored K-blocked: the K (reduction) index is split into blocks of 32, and
// block kb holds every row's 32 elements side by side -- element (row, k) of a [rows][K]
// matrix sits at ((k / 32) * rows + row) * 32 + k % 32.  A GEMM stage that takes 32 K values
// of consecutive rows then reads one contiguous run of memory.  W1^T / W3^T (K = h) use it
// when h is a multiple of 32; W2^T (K = fp, a multiple of 128) always does.  fp32 weights
// stay row-major.
#include "common.h"
#include "kernels.h"

namespace moe {
namespace {

// dst[e](c, r) = (r < nr && c < nc) ? src[e][(r0 + r) * src_ld + c0 + c] : 0
// for c < dst_rows, r < dst_cols, where dst(c, r) is dst[c * dst_cols + r] (row-major) or,
// with blocked, dst[((r / 32) * dst_rows + c) * 32 + r % 32] (dst_cols a multiple of 32).
// dst_cols is a multiple of 8.
//
// Bound by memory (each element read and written once).  A workgroup takes kR source rows x kC
// columns: every thread issues all of its 16-byte loads before it uses one, and stores 16
// bytes of one dst row; the transposition happens between, in LDS, whose row pitch puts the
// rows that a store's lanes gather from on different banks.  VEC: source runs start on 16
// bytes (src, src_ld and c0 allow it); else the loads are single elements.
// Measured, 32 experts of 1024 x 1024 bf16 out of 4096 columns (67 MB read and written): 55 us
// with 2-byte loads and stores of a 64 x 64 tile, 27.5 us so (4.9 TB/s).
template <typename Te, bool VEC>
__global__ __launch_bounds__(256) void transpose_pad(const Te* __restrict__ src, int64_t src_estride,
                                                     int64_t src_ld, int64_t r0, int64_t c0, int64_t nr,
                                                     int64_t nc, Te* __restrict__ dst, int64_t dst_estride,
                                                     int64_t dst_rows, int64_t dst_cols, int blocked) {
    constexpr int kV = 16 / sizeof(Te);                  // elements per 16 bytes
    constexpr int kR = 64, kC = 64 * kV / 4;             // source rows x columns: 16 KiB
    constexpr int kPitch = sizeof(Te) == 2 ? kC + 2 : kC + 1;
    constexpr int kN = kR * kC / kV / 256;               // vectors per thread
    __shared__ Te tile[kR * kPitch];
    const int64_t rt = static_cast<int64_t>(blockIdx.x) * kR;  // source rows = dst cols
    const int64_t ct = static_cast<int64_t>(blockIdx.y) * kC;  // source cols = dst rows
    const Te* s = src + blockIdx.z * src_estride;
    Te* d = dst + blockIdx.z * dst_estride;
    if constexpr (VEC) {
        uint4 v[kN];
#pragma unroll
        for (int i = 0; i < kN; ++i) {
            const int u = threadIdx.x + 256 * i, r = u / (kC / kV), c = u % (kC / kV) * kV;
            // a run that starts inside the columns may end past them (nc is any number): its
            // row has c0 + nc <= src_ld elements and src_ld is a multiple of kV, so it is in bounds
            v[i] = rt + r < nr && ct + c < nc ? *reinterpret_cast<const uint4*>(s + (r0 + rt + r) * src_ld + c0 + ct + c)
                                              : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < kN; ++i) {
            const int u = threadIdx.x + 256 * i, r = u / (kC / kV), c = u % (kC / kV) * kV;
            Te e[kV];
            __builtin_memcpy(e, &v[i], 16);
#pragma unroll
            for (int j = 0; j < kV; ++j) tile[r * kPitch + c + j] = ct + c + j < nc ? e[j] : Te(0);
        }
    } else {
#pragma unroll 16
        for (int i = threadIdx.x; i < kR * kC; i += 256) {
            const int r = i / kC, c = i % kC;
            tile[r * kPitch + c] = rt + r < nr && ct + c < nc ? s[(r0 + rt + r) * src_ld + c0 + ct + c] : Te(0);
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kN; ++i) {
        // blocked: a dst row's 32 elements of a block are 64 bytes, the next row's follow;
        // row-major: the tile's kR elements of a dst row are contiguous
        const int u = threadIdx.x + 256 * i;
        const int per = blocked ? 32 / kV : kR / kV;
        const int q = u / per % kC, r = u / per / kC * 32 + u % per * kV;
        const int64_t c = ct + q;
        if (c >= dst_rows || rt + r >= dst_cols) continue;
        Te e[kV];
#pragma unroll
        for (int j = 0; j < kV; ++j) e[j] = tile[(r + j) * kPitch + q];
        uint4 v;
        __builtin_memcpy(&v, e, 16);
        *reinterpret_cast<uint4*>(d + (blocked ? (((rt + r) >> 5) * dst_rows + c) * 32 + ((rt + r) & 31)
                                               : c * dst_cols + rt + r)) = v;
    }
}

template <typename Te>
hipError_t transpose(const Te* src, int64_t src_estride, int64_t src_ld, int64_t r0, int64_t c0, int64_t nr, int64_t nc,
                     Te* dst, int64_t dst_estride, int64_t dst_rows, int64_t dst_cols, int blocked, int E, hipStream_t s) {
    constexpr int kV = 16 / sizeof(Te), kR = 64, kC = 64 * kV / 4;
    const dim3 grid(static_cast<unsigned>(ceil_div(dst_cols, kR)), static_cast<unsigned>(ceil_div(dst_rows, kC)), E);
    // expert strides are multiples of src_ld, and src is 16-byte aligned (checked by the caller)
    if (src_ld % kV == 0 && c0 % kV == 0)
        hipLaunchKernelGGL((transpose_pad<Te, true>), grid, dim3(256), 0, s, src, src_estride, src_ld, r0, c0, nr, nc, dst,
                           dst_estride, dst_rows, dst_cols, blocked);
    else
        hipLaunchKernelGGL((transpose_pad<Te, false>), grid, dim3(256), 0, s, src, src_estride, src_ld, r0, c0, nr, nc, dst,
                           dst_estride, dst_rows, dst_cols, blocked);
    return hipGetLastError();
}

template <typename Te>
hipError_t pack_t(const void* w1, const void* w3, const void* w2, int E, int64_t h, int64_t F,
                  int64_t col0, int64_t f, int64_t fp, void* w1t, void* w3t, void* w2t, hipStream_t s) {
    const int blk1 = (sizeof(Te) == 2 && h % 32 == 0) ? 1 : 0;
    const int blk2 = sizeof(Te) == 2 ? 1 : 0;
    // W1 (and W3): source [h rows][F cols] -> dst [fp rows][h cols]
    hipError_t err = transpose(static_cast<const Te*>(w1), h * F, F, int64_t(0), col0, h, f, static_cast<Te*>(w1t),
                               fp * h, fp, h, blk1, E, s);
    if (err == hipSuccess && w3)
        err = transpose(static_cast<const Te*>(w3), h * F, F, int64_t(0), col0, h, f, static_cast<Te*>(w3t), fp * h, fp, h,
                        blk1, E, s);
    // W2: source [F rows][h cols], rows col0.. -> dst [h rows][fp cols]
    if (err == hipSuccess)
        err = transpose(static_cast<const Te*>(w2), F * h, h, col0, int64_t(0), f, h, static_cast<Te*>(w2t), h * fp, h, fp,
                        blk2, E, s);
    return err;
}

}  // namespace

hipError_t launch_pack(const void* w1, const void* w3, const void* w2, int E, int64_t h, int64_t F,
                       int64_t col0, int64_t f, int64_t fp, int elem_bytes, void* w1t, void* w3t,
                       void* w2t, hipStream_t s) {
    if (elem_bytes == 2) return pack_t<uint16_t>(w1, w3, w2, E, h, F, col0, f, fp, w1t, w3t, w2t, s);
    return pack_t<uint32_t>(w1, w3, w2, E, h, F, col0, f, fp, w1t, w3t, w2t, s);
}

}  // namespace moe
