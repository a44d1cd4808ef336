// Fused chain, "reduce" family on small row blocks (16 or 32 rows): operands go from global memory STRAIGHT to the
// registers of the wave that multiplies them.
//
// A workgroup owns a row block and a range of the hidden dimension, which it walks in slices of 64 columns:
//   first product : the four waves split K (steps of 32 k, dealt in turn); every wave computes a partial
//                   [rows][64] tile with the loads of DEPTH steps in flight and no barrier between them;
//   exchange      : the four partial tiles are summed in LDS, activated on complete sums (paper Sec. 4.3, Rule 3),
//                   gated, rounded to the operand type and left in LDS as the slice's block of H;
//   second product: every wave multiplies that block with its own quarter of W2's columns into accumulators that
//                   stay in registers for the whole range.
// With one range the output goes straight to Y: one launch, no workspace traffic.  With several, each range stores
// its fp32 plane and the planes are summed in a fixed order (launch_finalize_planes).
//
// What bounds it: the problems it is for hold fewer bytes and flops than a launch lasts; what counts is how many
// memory round trips and barriers follow one another.  The two-phase kernel needs a device-wide rendezvous and,
// where a layer has few 64-column slices, leaves the first product to a handful of workgroups, each walking all of
// K alone; the 128-row reduce tiles walk K in LDS stages with a barrier each.  Here a slice costs two barriers and
// about K / (128 DEPTH) round trips.  Against that, operands are re-read from L2 by every row block.
//
// Measured (us, the best of the other plans -> this): 3x3 chains 196 pixels x 2304 x 256 x 1024 41 -> 16, 49 x 4608 x
// 512 x 2048 47 -> 25, 6272 x 576 x 64 x 256 21 -> 8; 128 x 384 x 1536 x 384 17.4 -> 10.8; 3136 x 64 x 256 x 64
// 8.9 -> 7.0.  It loses from about 1.5 Gflop on (200 x 1024 x 4096 x 1024: 28 against 34).  Issuing a slice's first W2
// loads a slice earlier was 3-5 % slower: the walk is bound by issue, not by the wait for those loads.
//
// v_mfma_f32_16x16x32: lane l holds A[l % 16][8 (l / 16) .. + 7], B[8 (l / 16) .. + 7][l % 16] and
// D[4 (l / 16) + r][l % 16].  A weight row is read as 16 lanes x 8 bytes (whole cache lines); a lane's 8 rows x 4
// columns are transposed in registers into the operands of four column tiles, tile i holding columns 4 (l % 16) + i.
#include "ffuse_dev.h"
#include "ffuse_launch.h"

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

// 8 rows x 4 columns: the 8 bytes of each row at column byte `col_bytes`; !ok reads zeros, rows past the end too
__device__ __forceinline__ void load_octet(__amdgpu_buffer_rsrc_t r, uint32_t row, uint32_t row_bytes, uint32_t col_bytes, bool ok, u32x2 (&w)[8]) {
#pragma unroll
    for (int j = 0; j < 8; ++j)
        w[j] = __builtin_amdgcn_raw_buffer_load_b64(r, ok ? (row + j) * row_bytes + col_bytes : kOob, 0, 0);
}
// column i of such a block: 8 consecutive k
__device__ __forceinline__ u32x4 octet_column(const u32x2 (&w)[8], int i) {
    u32x4 o;
#pragma unroll
    for (int d = 0; d < 4; ++d)
        o[d] = __builtin_amdgcn_perm(w[2 * d + 1][i >> 1], w[2 * d][i >> 1], (i & 1) ? 0x07060302u : 0x05040100u);
    return o;
}

// R: tiles of 16 rows; NG: blocks of 256 output columns (64 per wave each)
// SHORT (K <= 256): two steps a wave hold all of K, and steps and column blocks that do not exist are branched over
// instead of loaded out of range (a range-checked load of zeros costs its issue slots all the same: 64 x 128 x 512 x
// 128 8.6 -> 6.3 us).  Longer K keeps straight-line turns: there the branches cost the overlap of the turns
// (128 x 512 x 2048 x 512 in one range: 97 us without, 141 with).
template <typename T, bool GATED, bool CONV, int R, int NG, bool SHORT>
__global__ __launch_bounds__(256) void fused_direct_kernel(DirectArgs a) {
    constexpr int G = GATED ? 2 : 1, DEPTH = GATED || SHORT ? 2 : 4, BM = 16 * R;
    constexpr int HROW = 72;                             // elements of an H row in LDS (64 and a pad against bank conflicts)
    __shared__ __attribute__((aligned(16))) float part[G * 4][BM][64];
    __shared__ __attribute__((aligned(16))) uint16_t hs[BM][HROW];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, q = lane >> 4;
    const int range = blockIdx.x % a.ranges;             // (ranges a multiple of 8: an XCD reads its own part of the weights)
    const int64_t m0 = (int64_t)(blockIdx.x / a.ranges) * BM;
    const int K = a.K, N1 = a.N1, N2 = a.N2;
    const int ch_end = min(a.slices * (range + 1), (N1 + 63) / 64);
    const __amdgpu_buffer_rsrc_t rx = make_rsrc(a.X, (uint32_t)((uint64_t)a.M * (CONV ? a.conv_ic : K) * 2));
    const __amdgpu_buffer_rsrc_t rw[2] = {make_rsrc(a.W1, (uint32_t)((uint64_t)K * N1 * 2)),
                                          make_rsrc(GATED ? a.W3 : a.W1, (uint32_t)((uint64_t)K * N1 * 2))};
    const __amdgpu_buffer_rsrc_t r2 = make_rsrc(a.W2, (uint32_t)((uint64_t)N1 * N2 * 2));
    const uint32_t w1row = 2u * (uint32_t)N1, w2row = 2u * (uint32_t)N2;
    int py[R], px[R];                                    // CONV: the pixel of this lane's row of each row tile
    if constexpr (CONV) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t pix = (uint32_t)(m0 + 16 * r + c) % (uint32_t)(a.conv_h * a.conv_w);
            py[r] = (int)(pix / (uint32_t)a.conv_w);
            px[r] = (int)(pix % (uint32_t)a.conv_w);
        }
    }

    struct Slot {
        u32x4 x[R];
        u32x2 w[G][8];
    } slot[DEPTH];
    const int ksteps = ((K + 31) / 32 + 4 * DEPTH - 1) / (4 * DEPTH) * DEPTH;   // a wave's steps per slice, whole turns of the ring
    int lch = range * a.slices, ls = 0;                  // slice and step of the next load
    const auto load_next = [&](Slot& s) {
        const int k0 = 32 * (4 * ls + wave), k = k0 + 8 * q;
        if (!SHORT || k0 < K) {
            const bool ok = lch < ch_end && k < K;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if constexpr (CONV) {
                    // 32 k lie in one tap (conv_ic is a multiple of 32)
                    const int tap = k0 / a.conv_ic, ky = tap / 3 - 1, kx = tap % 3 - 1;
                    const int64_t row = m0 + 16 * r + c;
                    const bool in = ok && row < a.M && (uint32_t)(py[r] + ky) < (uint32_t)a.conv_h && (uint32_t)(px[r] + kx) < (uint32_t)a.conv_w;
                    const uint32_t pix = (uint32_t)((int)row + ky * a.conv_w + kx);
                    s.x[r] = buf_load16(rx, in ? (pix * (uint32_t)a.conv_ic + (uint32_t)(k - tap * a.conv_ic)) * 2u : kOob);
                } else {
                    s.x[r] = buf_load16(rx, ok ? ((uint32_t)(m0 + 16 * r + c) * (uint32_t)K + (uint32_t)k) * 2u : kOob);
                }
            }
            const int col = 64 * lch + 4 * c;
#pragma unroll
            for (int g = 0; g < G; ++g) load_octet(rw[g], (uint32_t)k, w1row, 2u * (uint32_t)col, ok && col < N1, s.w[g]);
        }
        if (++ls == ksteps) { ls = 0; ++lch; }
    };
#pragma unroll
    for (int u = 0; u < DEPTH; ++u) load_next(slot[u]);

    f32x4 acc2[NG][R][4];
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc2[g][r][i] = f32x4{0.f, 0.f, 0.f, 0.f};

    for (int ch = range * a.slices; ch < ch_end; ++ch) {
        u32x2 w2[NG > 1 ? 2 : 1][2][8];                  // column blocks in flight, two steps of 32 hidden columns each
        const auto load2 = [&](int g) {
            const int col = 64 * (4 * g + wave) + 4 * c;
            if (!SHORT || 64 * (4 * g + wave) < N2)
#pragma unroll
                for (int t = 0; t < 2; ++t) load_octet(r2, (uint32_t)(64 * ch + 32 * t + 8 * q), w2row, 2u * (uint32_t)col, col < N2, w2[g & 1][t]);
        };
        load2(0);
        f32x4 acc[G][R][4];
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[g][r][i] = f32x4{0.f, 0.f, 0.f, 0.f};
        const auto multiply = [&](const Slot& w, int step) {
            if (SHORT && 32 * (4 * step + wave) >= K) return;
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const u32x4 b = octet_column(w.w[g], i);
#pragma unroll
                    for (int r = 0; r < R; ++r) acc[g][r][i] = Mma16<T>::mma(w.x[r], b, acc[g][r][i]);
                }
        };
        for (int s = 0; s < ksteps; s += DEPTH) {
            if (s + DEPTH < ksteps || ch + 1 < ch_end) {
#pragma unroll
                for (int u = 0; u < DEPTH; ++u) {
                    multiply(slot[u], s + u);
                    load_next(slot[u]);
                }
            } else {                                     // the range's last turn: nothing left to load
#pragma unroll
                for (int u = 0; u < DEPTH; ++u) multiply(slot[u], s + u);
            }
        }
        // acc[g][r][i][e]: row 16 r + 4 q + e, column 4 c + i of the slice
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    *reinterpret_cast<f32x4*>(&part[4 * g + wave][16 * r + 4 * q + e][4 * c]) =
                        f32x4{acc[g][r][0][e], acc[g][r][1][e], acc[g][r][2][e], acc[g][r][3][e]};
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int row = 16 * r + (tid >> 4), col = 4 * (tid & 15);
            f32x4 v[G];
#pragma unroll
            for (int g = 0; g < G; ++g) {
                v[g] = *reinterpret_cast<const f32x4*>(&part[4 * g][row][col]);
#pragma unroll
                for (int p = 1; p < 4; ++p) v[g] += *reinterpret_cast<const f32x4*>(&part[4 * g + p][row][col]);
            }
            f32x4 h;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                switch (a.act) {
                    case ACT_RELU: h[i] = activate<ACT_RELU>(v[0][i]); break;
                    case ACT_GELU_TANH: h[i] = activate<ACT_GELU_TANH>(v[0][i]); break;
                    case ACT_SILU: h[i] = activate<ACT_SILU>(v[0][i]); break;
                    default: h[i] = v[0][i]; break;
                }
                if constexpr (GATED) h[i] *= v[G - 1][i];
                if (64 * ch + col >= N1) h[i] = 0.0f;    // (an infinity of X times the zero weights past N1 is not a number)
            }
            u32x2 o = {pack2<T>(h[0], h[1]), pack2<T>(h[2], h[3])};
            *reinterpret_cast<u32x2*>(&hs[row][col]) = o;
        }
        __syncthreads();
        u32x4 hf[R][2];
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int t = 0; t < 2; ++t) hf[r][t] = *reinterpret_cast<const u32x4*>(&hs[16 * r + c][32 * t + 8 * q]);
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            if (g + 1 < NG) load2(g + 1);
            if (64 * (4 * g + wave) < N2) {
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const u32x4 b = octet_column(w2[g & 1][t], i);
#pragma unroll
                        for (int r = 0; r < R; ++r) acc2[g][r][i] = Mma16<T>::mma(hf[r][t], b, acc2[g][r][i]);
                    }
            }
        }
        // (the next slice's partial tiles are written after every wave has read this one's -- the second barrier --
        //  and its H after every wave has read this one's: the next first barrier)
    }

    float* plane = a.part + (size_t)range * (size_t)a.M * N2;
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int64_t row = m0 + 16 * r + 4 * q + e;
                const int col = 64 * (4 * g + wave) + 4 * c;
                if (row < a.M && col < N2) {
                    const f32x4 v = {acc2[g][r][0][e], acc2[g][r][1][e], acc2[g][r][2][e], acc2[g][r][3][e]};
                    if (a.ranges > 1) {
                        *reinterpret_cast<f32x4*>(plane + row * N2 + col) = v;
                    } else {
                        const u32x2 o = {pack2<T>(v[0], v[1]), pack2<T>(v[2], v[3])};
                        *reinterpret_cast<u32x2*>(reinterpret_cast<char*>(a.Y) + (row * N2 + col) * 2) = o;
                    }
                }
            }
}

template <typename T, bool GATED, bool CONV> static const void* direct_fn(int bm, int ng, int K) {
    if constexpr (!CONV) {
        if (K <= 256 && ng <= 2) {
            if (bm == 16) return ng == 1 ? (const void*)fused_direct_kernel<T, GATED, false, 1, 1, true> : (const void*)fused_direct_kernel<T, GATED, false, 1, 2, true>;
            if (bm == 32) return ng == 1 ? (const void*)fused_direct_kernel<T, GATED, false, 2, 1, true> : (const void*)fused_direct_kernel<T, GATED, false, 2, 2, true>;
            return nullptr;
        }
    }
    if (bm == 16) {
        if (ng == 1) return (const void*)fused_direct_kernel<T, GATED, CONV, 1, 1, false>;
        if (ng == 2) return (const void*)fused_direct_kernel<T, GATED, CONV, 1, 2, false>;
        if (ng == 4) return (const void*)fused_direct_kernel<T, GATED, CONV, 1, 4, false>;
        if (ng == 8) return (const void*)fused_direct_kernel<T, GATED, CONV, 1, 8, false>;
    }
    if (bm == 32) {
        if (ng == 1) return (const void*)fused_direct_kernel<T, GATED, CONV, 2, 1, false>;
        if (ng == 2) return (const void*)fused_direct_kernel<T, GATED, CONV, 2, 2, false>;
    }
    return nullptr;
}

hipError_t launch_fused_direct(int dtype, const DirectArgs& a, int bm, int ng, hipStream_t st) {
    const bool g = a.W3 != nullptr, conv = a.conv_ic > 0;
    if (conv && (g || a.conv_ic % 32 || a.K != 9 * a.conv_ic || a.conv_h < 1 || a.conv_w < 1)) return hipErrorInvalidValue;
    if (a.ranges < 1 || a.slices < 1 || (int64_t)a.ranges * a.slices * 64 < a.N1 || (int64_t)(a.ranges - 1) * a.slices * 64 >= a.N1 ||
        a.N2 > 256 * ng || (a.ranges > 1 && !a.part)) return hipErrorInvalidValue;
    const void* fn;
    if (dtype == 0) fn = conv ? direct_fn<__bf16, false, true>(bm, ng, a.K) : g ? direct_fn<__bf16, true, false>(bm, ng, a.K) : direct_fn<__bf16, false, false>(bm, ng, a.K);
    else fn = conv ? direct_fn<_Float16, false, true>(bm, ng, a.K) : g ? direct_fn<_Float16, true, false>(bm, ng, a.K) : direct_fn<_Float16, false, false>(bm, ng, a.K);
    const int64_t grid = (a.M + bm - 1) / bm * a.ranges;
    if (!fn || grid > 0x7fffffff) return hipErrorInvalidValue;
    DirectArgs copy = a;
    void* params[] = {&copy};
    hipError_t e = hipLaunchKernel(fn, dim3((unsigned)grid), dim3(256), params, 0, st);
    if (e == hipSuccess && a.ranges > 1) e = launch_finalize_planes(dtype, a.part, a.Y, a.M * a.N2, a.ranges, st);
    return e;
}

}  // namespace ffuse
