// fp32 path: the same chain on the fp32 matrix instructions (full fp32 products and sums), for checking the
// schedule and the boundary at full precision.  Same "reduce" structure as the 16-bit fused kernel:
// one workgroup per (16-row block, 64-wide hidden slice), complete K sums before the
// activation (paper Sec. 4.3, Rule 3), partial second products added atomically into Y.
//
// What bounds it: on the shapes it is for (up to a few hundred rows and widths) the latency of one workgroup.
// So every operand goes straight from global memory to the registers of the wave that multiplies it, with many
// loads in flight together and no barrier between them: the four waves split K (partial tiles summed in LDS), a
// W1 row is read as 16 lanes x 16 bytes that feed four column tiles, and the second product's first weights are on
// their way while the first product is summed.  128 x 256 x 1024 x 256: 51 -> 10.5 us (with the launch that clears
// Y); before, 32 k at a time went through LDS with two barriers each, multiplied on scalar FMAs.  Many rows: 2048 x 512 x
// 2048 x 512 761 -> 152 us, 2048 x 1024 x 4096 x 1024 2825 -> 485 (71 TFLOP/s), gated 3756 -> 606 (85), 8192 x 256 x 1024 x
// 256 774 -> 153; there every row block reads the weights again and an output takes N1 / 64 atomic adds.
#include "ffuse_dev.h"
#include "ffuse_launch.h"
#include <mutex>
#include <unordered_map>

#include <cstdlib>

namespace ffuse {

static __device__ __forceinline__ float act_f32(int act, float x) {
    switch (act) {
        case ACT_RELU: return fmaxf(x, 0.0f);
        case ACT_GELU_TANH: {
            const float z = 0.7978845608028654f * (x + 0.044715f * x * x * x);
            return 0.5f * x * (1.0f + tanhf(z));
        }
        case ACT_SILU: return x / (1.0f + expf(-x));
        default: return x;
    }
}

constexpr int F_BM = 16, F_BH = 64;
constexpr int F_HLD = F_BH + 4;   // row stride of the H block in LDS (floats)

// v_mfma_f32_16x16x4_f32: lane l holds A[l % 16][l / 16], B[l / 16][l % 16] and D[4 * (l / 16) + r][l % 16].
// A group of 16 k is multiplied by four of them: instruction j takes k = 4 * (l / 16) + j, so that a lane's four
// k of A are 16 consecutive bytes.  Column tile i of the four that a wave computes side by side holds the columns
// 4 * (l % 16) + i, so that a lane's four columns of B are 16 consecutive bytes too.
__device__ __forceinline__ void mma_group_f32(const f32x4& x, const f32x4 (&w)[4], f32x4 (&acc)[4]) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[j], w[j][i], acc[i], 0, 0, 0);
}
// the 16-byte units of rows k0 + 4 * (lane / 16) + 0..3 of a [K][N] matrix at this lane's columns
__device__ __forceinline__ void load_rows_f32(__amdgpu_buffer_rsrc_t r, int k, uint32_t row_bytes, uint32_t col_bytes, bool ok, f32x4 (&w)[4]) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
        w[j] = __builtin_bit_cast(f32x4, buf_load16(r, ok ? (uint32_t)(k + j) * row_bytes + col_bytes : kOob));
}

// H block [16][64] of act(X W1) [.* X W3] for rows m0.., hidden n0.. into hs (LDS).  part: a partial tile a wave
// (and branch).  Ends with a barrier.  The groups of 16 k are dealt to the waves in turn, BATCH at a time each:
// 80 registers of operands in flight, gated 72 (up to K = 256, gated 128, all of a wave's loads are issued at once).
// Rows past M, k past K and columns past N1 read as zeros (K, N1 and N2 are multiples of 8).
template <bool GATED>
static __device__ __forceinline__ void first_product_f32(const float* X, const float* W1, const float* W3,
                                                         int64_t M, int K, int N1, int act, int64_t m0, int n0,
                                                         float (*part)[F_BM][F_BH], float (*hs)[F_HLD]) {
    constexpr int G = GATED ? 2 : 1, BATCH = GATED ? 2 : 4;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, q = lane >> 4;
    const __amdgpu_buffer_rsrc_t rx = make_rsrc(X, (uint32_t)((uint64_t)M * K * 4));
    const __amdgpu_buffer_rsrc_t rw[2] = {make_rsrc(W1, (uint32_t)((uint64_t)K * N1 * 4)),
                                          make_rsrc(GATED ? W3 : W1, (uint32_t)((uint64_t)K * N1 * 4))};
    const uint32_t xrow = (uint32_t)(m0 + c) * (uint32_t)K * 4u, wrow = (uint32_t)N1 * 4u;
    const int col = n0 + 4 * c;
    f32x4 acc[G][4];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[g][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int g0 = 0; g0 * 16 < K; g0 += 4 * BATCH) {
        f32x4 x[BATCH], w[BATCH][G][4];
#pragma unroll
        for (int b = 0; b < BATCH; ++b) {
            const int k = 16 * (g0 + 4 * b + wave) + 4 * q;
            x[b] = __builtin_bit_cast(f32x4, buf_load16(rx, k < K ? xrow + 4u * (uint32_t)k : kOob));
#pragma unroll
            for (int g = 0; g < G; ++g) load_rows_f32(rw[g], k, wrow, 4u * (uint32_t)col, k < K && col < N1, w[b][g]);
        }
#pragma unroll
        for (int b = 0; b < BATCH; ++b)
#pragma unroll
            for (int g = 0; g < G; ++g) mma_group_f32(x[b], w[b][g], acc[g]);
    }
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            *reinterpret_cast<f32x4*>(&part[4 * g + wave][4 * q + r][4 * c]) = f32x4{acc[g][0][r], acc[g][1][r], acc[g][2][r], acc[g][3][r]};
    __syncthreads();
    {
        const int row = tid >> 4, cc = 4 * (tid & 15);
        f32x4 v[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            v[g] = *reinterpret_cast<const f32x4*>(&part[4 * g][row][cc]);
#pragma unroll
            for (int p = 1; p < 4; ++p) v[g] += *reinterpret_cast<const f32x4*>(&part[4 * g + p][row][cc]);
        }
        f32x4 h;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            h[i] = act_f32(act, v[0][i]);
            if constexpr (GATED) h[i] *= v[G - 1][i];
            if (n0 + cc >= N1) h[i] = 0.0f;   // (an infinity of X times the zero weights past N1 is not a number)
        }
        *reinterpret_cast<f32x4*>(&hs[row][cc]) = h;
    }
    __syncthreads();
}

template <bool GATED> __global__ __launch_bounds__(256) void fused_f32_kernel(FusedArgs a, float* Y) {
    __shared__ __attribute__((aligned(16))) float part[GATED ? 8 : 4][F_BM][F_BH];
    __shared__ __attribute__((aligned(16))) float hs[F_BM][F_HLD];
    const int64_t m0 = (int64_t)blockIdx.x * F_BM;
    const int n0 = blockIdx.y * F_BH;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 15, q = lane >> 4;
    // the wave's blocks of 64 output columns: wave, wave + 4, ...; rows of W2 past N1 lie past the buffer (zeros)
    const __amdgpu_buffer_rsrc_t r2 = make_rsrc(a.W2, (uint32_t)((uint64_t)a.N1 * a.N2 * 4));
    const uint32_t w2row = (uint32_t)a.N2 * 4u;
    f32x4 w[4][4];
    const auto load2 = [&](int cb) {
        const int col = 64 * cb + 4 * c;
#pragma unroll
        for (int t = 0; t < 4; ++t) load_rows_f32(r2, n0 + 16 * t + 4 * q, w2row, 4u * (uint32_t)col, col < a.N2, w[t]);
    };
    load2(wave);
    first_product_f32<GATED>((const float*)a.X, (const float*)a.W1, (const float*)a.W3, a.M, a.K, a.N1, a.act, m0, n0, part, hs);
    f32x4 h[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) h[t] = *reinterpret_cast<const f32x4*>(&hs[c][16 * t + 4 * q]);
    for (int cb = wave; 64 * cb < a.N2; cb += 4) {
        f32x4 acc[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 4; ++t) mma_group_f32(h[t], w[t], acc);
        if (64 * (cb + 4) < a.N2) load2(cb + 4);
        // through the wave's own partial tile, so that the 64 lanes of an atomic add cover 256 consecutive bytes
#pragma unroll
        for (int r = 0; r < 4; ++r)
            *reinterpret_cast<f32x4*>(&part[wave][4 * q + r][4 * c]) = f32x4{acc[0][r], acc[1][r], acc[2][r], acc[3][r]};
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const int col = 64 * cb + lane;
#pragma unroll
        for (int r = 0; r < F_BM; ++r)
            if (m0 + r < a.M && col < a.N2)
                __hip_atomic_fetch_add(Y + (m0 + r) * a.N2 + col, part[wave][r][lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();   // the tile is read before the next block's is written
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

// C = act(A B) [.* A B3], fp32, 16 x 64 tile per workgroup
template <bool GATED> __global__ __launch_bounds__(256) void gemm_act_f32_kernel(GemmArgs a) {
    __shared__ __attribute__((aligned(16))) float part[GATED ? 8 : 4][F_BM][F_BH];
    __shared__ __attribute__((aligned(16))) float hs[F_BM][F_HLD];
    const int64_t m0 = (int64_t)blockIdx.x * F_BM;
    const int n0 = blockIdx.y * F_BH;
    first_product_f32<GATED>((const float*)a.A, (const float*)a.B, (const float*)a.B3, a.M, a.K, a.N, a.act, m0, n0, part, hs);
    float* C = (float*)a.C;
    for (int i = threadIdx.x; i < F_BM * F_BH; i += 256) {
        const int r = i / F_BH, c = i % F_BH;
        if (m0 + r < a.M && n0 + c < a.N) C[(m0 + r) * a.N + n0 + c] = hs[r][c];
    }
}

__global__ __launch_bounds__(256) void zero_kernel(u32x4* p, size_t n16) {
    const u32x4 z = {0u, 0u, 0u, 0u};
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n16; i += (size_t)gridDim.x * 256) p[i] = z;
}

hipError_t launch_zero(void* p, size_t bytes, hipStream_t st) {
    const size_t n16 = bytes / 16;
    if (n16 == 0) return hipSuccess;
    const size_t want = (n16 + 255) / 256;
    const int blocks = (int)(want < 4096 ? want : 4096);
    hipLaunchKernelGGL(zero_kernel, dim3(blocks), dim3(256), 0, st, reinterpret_cast<u32x4*>(p), n16);
    return hipGetLastError();
}

hipError_t launch_resident(const void* fn, int grid, void** params, hipStream_t st, int threads) {
    static const bool cooperative = getenv("FFUSE_COOPERATIVE_LAUNCH") != nullptr;
    if (cooperative) return hipLaunchCooperativeKernel(fn, dim3(grid), dim3(threads), params, 0, st);
    // how many workgroups of this kernel the device holds at once: asked once per kernel
    static std::mutex mu;
    static std::unordered_map<const void*, int> capacity;
    int cap = 0;
    {
        std::lock_guard<std::mutex> lock(mu);
        auto it = capacity.find(fn);
        if (it != capacity.end()) cap = it->second;
    }
    if (cap == 0) {
        int per_cu = 0, dev = 0, cus = 0;
        hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, threads, 0);
        if (e != hipSuccess) return e;
        if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
        if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
        cap = per_cu * cus;
        if (cap <= 0) return hipErrorCooperativeLaunchTooLarge;
        std::lock_guard<std::mutex> lock(mu);
        capacity[fn] = cap;
    }
    if (grid > cap) return hipErrorCooperativeLaunchTooLarge;
    return hipLaunchKernel(fn, dim3(grid), dim3(threads), params, 0, st);
}

hipError_t launch_fused_f32(const FusedArgs& a, float* Y, hipStream_t st) {
    // N2 is a multiple of 8, so the output is a whole number of 16-byte units
    hipError_t e = launch_zero(Y, sizeof(float) * (size_t)a.M * a.N2, st);
    if (e != hipSuccess) return e;
    dim3 grid((unsigned)((a.M + F_BM - 1) / F_BM), (unsigned)((a.N1 + F_BH - 1) / F_BH));
    if (a.W3) hipLaunchKernelGGL(fused_f32_kernel<true>, grid, dim3(256), 0, st, a, Y);
    else hipLaunchKernelGGL(fused_f32_kernel<false>, grid, dim3(256), 0, st, a, Y);
    return hipGetLastError();
}

hipError_t launch_gemm_act_f32(const GemmArgs& a, hipStream_t st) {
    dim3 grid((unsigned)((a.M + F_BM - 1) / F_BM), (unsigned)((a.N + F_BH - 1) / F_BH));
    if (a.B3) hipLaunchKernelGGL(gemm_act_f32_kernel<true>, grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL(gemm_act_f32_kernel<false>, grid, dim3(256), 0, st, a);
    return hipGetLastError();
}

}  // namespace ffuse
