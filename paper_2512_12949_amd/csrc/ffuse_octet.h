// 16 x 16 x 32 products on weights loaded straight from global memory (ffuse_direct.hip, ffuse_stream.hip).
//
// v_mfma_f32_16x16x32: lane l holds A[l % 16][8 (l / 16) .. + 7], B[8 (l / 16) .. + 7][l % 16] and
// D[4 (l / 16) + r][l % 16].  A weight row is read as 16 lanes x 8 bytes (whole cache lines); a lane's 8 rows x 4
// columns are transposed in registers into the operands of four column tiles, tile i holding columns 4 (l % 16) + i.
#pragma once
#include "ffuse_dev.h"

namespace ffuse {

typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

template <typename T> struct Mma16;
template <> struct Mma16<__bf16> {
    static __device__ __forceinline__ f32x4 mma(u32x4 a, u32x4 b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    }
};
template <> struct Mma16<_Float16> {
    static __device__ __forceinline__ f32x4 mma(u32x4 a, u32x4 b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    }
};

// 8 rows x 4 columns: the 8 bytes of each row, the first at byte offset `lane` (kOob reads zeros) + `base`, the same in
// every lane: one address register for the block, the rows' distances are scalars
__device__ __forceinline__ void load_octet(__amdgpu_buffer_rsrc_t r, uint32_t lane, uint32_t base, uint32_t row_bytes, u32x2 (&w)[8]) {
#pragma unroll
    for (int j = 0; j < 8; ++j) w[j] = __builtin_amdgcn_raw_buffer_load_b64(r, lane, base + (uint32_t)j * row_bytes, 0);
}
// column i of such a block: 8 consecutive k
__device__ __forceinline__ u32x4 octet_column(const u32x2 (&w)[8], int i) {
    u32x4 o;
#pragma unroll
    for (int d = 0; d < 4; ++d)
        o[d] = __builtin_amdgcn_perm(w[2 * d + 1][i >> 1], w[2 * d][i >> 1], (i & 1) ? 0x07060302u : 0x05040100u);
    return o;
}

}  // namespace ffuse
