// Fused chain, "two-phase" family, streaming kernel (plan.bk = 128): up to 32 rows, weights straight from memory to the
// registers of the wave that multiplies them.  ffuse_two_phase.hip describes the family.
//
//   phase 1 : an item is a slice of 64 hidden columns (of both matrices when gated), K complete: the eight waves split K,
//             64 k each and step, and sum their partial tiles in LDS; activation, gate, rounding, written through;
//   barrier : ffuse_rendezvous.h.  A workgroup's first weights of phase 2 are loaded before it waits;
//   phase 2 : an item is 64 output columns x one of `splits` ranges of the hidden dimension, the same loop over H and W2.
//
// What bounds it: the weights' way from HBM.  Column slices are read at 6.5-7 TB/s when 170 and more workgroups
// have 64 KB each in flight in whole cache lines, 16 bytes a lane, eight waves a workgroup (probe: 4096 rows of 22016 bytes,
// 168 slices of 128 bytes: 8 bytes a lane and four waves 15.9 us, eight waves 14.2, 16 bytes a lane 12.4; a second step
// in flight gives nothing).  So a slice is one cache line wide: a 7B-class layer has 172 of them, where the LDS-direct
// kernel's 128 columns gave 86 workgroups work.  Splitting K over workgroups as well, so that all 256 have an equal share,
// was no faster (61.5 us and 61.1): the parts have to meet.  Lines whose address has bits 7-9 = 3 come 20-30 % slower
// when all are read at once, whoever reads them; rows that are a multiple of 1 KB apart put them all into every eighth
// slice, and the phase ends with those.
//
// Measured (us, LDS-direct kernel -> this): gated 1 x 4096 x 11008 x 4096 72 -> 58, 16 rows 77 -> 62, 32 rows 80 -> 68;
// 16 x 2048 x 8192 x 2048 25 -> 21; 13 x 5000 x 13000 x 5000 75 -> 63; 6 x 1688 x 5760 x 1688 24 -> 19; gated 28 x 7296 x 6488 x
// 7296 130 -> 104.  Its rule and where it loses: rank_plans (ffuse_plan.cpp).
#include "ffuse_octet.h"
#include "ffuse_rendezvous.h"

namespace ffuse {

static constexpr int kWaves = 8, kStep = 64 * kWaves;   // waves of a workgroup, k of a step

// 64 columns x 64 k a wave and step.  A lane loads 16 bytes of a weight row, eight lanes a row: lane l has the columns
// 8 (l % 8) .. + 7 of the rows 32 (l / 8 % 2) + 8 (l / 16) + j, j = 0 .. 7.  Lanes l and l ^ 8 then exchange halves, so that
// each has four columns, 8 (l % 8) + 4 (l / 8 % 2) + i, of 8 rows of both 32-k halves: the operands of v_mfma_f32_16x16x32.
template <typename T, int G, int R, bool NT> struct StreamGemm {
    static constexpr int BM = 16 * R;
    struct Slot {
        u32x4 x[R][2];
        u32x4 w[G][8];
    };
    // an item: 64 columns, k0 .. k1 of K
    struct Item {
        uint32_t w;      // this lane's place in the weight rows of a step (kOob: no such columns)
        uint32_t base;   // byte offset of the item's first weight row and column
        int k0, k1;
        int steps;       // of kStep k
    };
    __amdgpu_buffer_rsrc_t rx, rw[G];
    uint32_t wrow;       // bytes of a weight row
    uint32_t x[R];       // this lane's place in its rows of X
    int wave, col, wk, xk, ncols;   // this lane's first column of the four; its first weight row and its first k of X in a step

    __device__ __forceinline__ void init(const void* X, int64_t M, int lda, const void* W, const void* W3, uint32_t w_bytes, int n, int tid) {
        rx = make_rsrc(X, (uint32_t)((uint64_t)M * lda * 2));
        rw[0] = make_rsrc(W, w_bytes);
        if (G == 2) rw[G - 1] = make_rsrc(W3, w_bytes);
        ncols = n;
        wrow = 2u * (uint32_t)n;
        wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int c = tid & 15, q = (tid >> 4) & 3;
        col = 8 * (c & 7) + 4 * (c >> 3);
        xk = 8 * q;
        wk = xk + 32 * (c >> 3);
#pragma unroll
        for (int r = 0; r < R; ++r) x[r] = 16 * r + c < M ? ((uint32_t)(16 * r + c) * (uint32_t)lda + (uint32_t)xk) * 2u : kOob;
    }
    __device__ __forceinline__ Item item(int col0, int k0, int k1, int tid) const {
        Item a;
        a.k0 = k0; a.k1 = k1;
        const uint32_t chunk = 8u * (uint32_t)(tid & 7);
        a.w = col0 + (int)chunk < ncols ? (uint32_t)wk * wrow + 2u * chunk : kOob;
        a.base = (uint32_t)k0 * wrow + 2u * (uint32_t)col0;
        a.steps = (k1 - k0 + kStep - 1) / kStep;
        return a;
    }
    // step s of an item: this wave's 64 k of it, zeros past the item's end
    __device__ __forceinline__ void load_w(Slot& t, const Item& a, int s) const {
        const int k = kStep * s + 64 * wave;
        const uint32_t v = a.k0 + k + wk < a.k1 ? a.w : kOob, so = a.base + (uint32_t)k * wrow;
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int j = 0; j < 8; ++j) t.w[g][j] = __builtin_amdgcn_raw_buffer_load_b128(rw[g], v, so + (uint32_t)j * wrow, NT ? 2 : 0);
    }
    __device__ __forceinline__ void load_x(Slot& t, const Item& a, int s) const {
        const int k = a.k0 + kStep * s + 64 * wave;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const bool ok = k + 32 * h + xk < a.k1;
#pragma unroll
            for (int r = 0; r < R; ++r) t.x[r][h] = __builtin_amdgcn_raw_buffer_load_b128(rx, ok ? x[r] : kOob, 2u * (uint32_t)(k + 32 * h), 0);
        }
    }
    static __device__ __forceinline__ void multiply(const Slot& t, f32x4 (&acc)[G][R][4]) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            u32x2 o[2][8];   // the lane's four columns in 8 rows of each half
#pragma unroll
            for (int j = 0; j < 8; ++j)
#pragma unroll
                for (int d = 0; d < 2; ++d) {
                    // row_ror:8 is lane l ^ 8; bank mask 12: lanes with l / 8 odd, 3: even
                    o[0][j][d] = (uint32_t)__builtin_amdgcn_update_dpp((int)t.w[g][j][d], (int)t.w[g][j][2 + d], 0x128, 0xf, 0xc, false);
                    o[1][j][d] = (uint32_t)__builtin_amdgcn_update_dpp((int)t.w[g][j][2 + d], (int)t.w[g][j][d], 0x128, 0xf, 0x3, false);
                }
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const u32x4 b = octet_column(o[h], i);
#pragma unroll
                    for (int r = 0; r < R; ++r) acc[g][r][i] = Mma16<T>::mma(t.x[r][h], b, acc[g][r][i]);
                }
        }
    }
    // one item whose first step is loaded; leaves that of `next` loaded
    __device__ __forceinline__ void run(Slot& slot, const Item& a, const Item& next, f32x4 (&acc)[G][R][4]) const {
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[g][r][i] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int s = 1; s < a.steps; ++s) {
            multiply(slot, acc);
            __builtin_amdgcn_sched_barrier(0);
            load_x(slot, a, s);
            load_w(slot, a, s);
            __builtin_amdgcn_sched_barrier(0);
        }
        multiply(slot, acc);
        __builtin_amdgcn_sched_barrier(0);
        load_x(slot, next, 0);
        load_w(slot, next, 0);
        __builtin_amdgcn_sched_barrier(0);
    }
    // The waves' partial tiles of one branch, summed through LDS: a thread ends up with VW columns of one row.
    static constexpr int VW = 2 * R;
    typedef __attribute__((ext_vector_type(VW))) float fvec;
    typedef __attribute__((ext_vector_type(VW / 2))) uint32_t hvec;
    static_assert(BM * 64 == VW * 64 * kWaves, "one place a thread");
    static __device__ __forceinline__ int sum_row(int tid) { return tid / (64 / VW); }
    static __device__ __forceinline__ int sum_col(int tid) { return VW * (tid % (64 / VW)); }
    __device__ __forceinline__ fvec sum(float (*part)[BM][64], const f32x4 (&acc)[R][4], int tid) const {
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                *reinterpret_cast<f32x4*>(&part[wave][16 * r + xk / 2 + e][col]) = f32x4{acc[r][0][e], acc[r][1][e], acc[r][2][e], acc[r][3][e]};
        __syncthreads();
        fvec v = *reinterpret_cast<const fvec*>(&part[0][sum_row(tid)][sum_col(tid)]);
#pragma unroll
        for (int w = 1; w < kWaves; ++w) v += *reinterpret_cast<const fvec*>(&part[w][sum_row(tid)][sum_col(tid)]);
        return v;
    }
};

template <typename T, bool GATED, int R, bool NT>
__device__ __forceinline__ void stream_first(const TwoPhaseArgs& a, float (*part)[16 * R][64], int tid, int xcd, int loc, int GX) {
    constexpr int G = GATED ? 2 : 1;
    typedef StreamGemm<T, G, R, NT> Gemm;
    const int NS = (a.N1 + 63) / 64;
    int rb, s, idx = loc;
    if (!map_item(1, NS, 1, xcd, idx, rb, s)) return;
    Gemm g;
    g.init(a.X, a.M, a.K, a.W1, a.W3, (uint32_t)((uint64_t)a.K * a.N1 * 2), a.N1, tid);
    const __amdgpu_buffer_rsrc_t rh = make_rsrc(a.H, (uint32_t)((uint64_t)a.M * a.N1 * 2));
    typename Gemm::Slot slot;
    typename Gemm::Item at = g.item(64 * s, 0, a.K, tid);
    g.load_x(slot, at, 0);
    g.load_w(slot, at, 0);
    for (;;) {
        int sn = 0;
        idx += GX;
        const bool more = map_item(1, NS, 1, xcd, idx, rb, sn);
        const typename Gemm::Item nx = more ? g.item(64 * sn, 0, a.K, tid) : g.item(a.N1, 0, 0, tid);
        f32x4 acc[G][R][4];
        g.run(slot, at, nx, acc);
        constexpr int VW = Gemm::VW;
        typename Gemm::fvec v[G];
#pragma unroll
        for (int b = 0; b < G; ++b) v[b] = g.sum(part + b * kWaves, acc[b], tid);
        float h[VW];
#pragma unroll
        for (int i = 0; i < VW; ++i) {
            switch (a.act) {
                case ACT_RELU: h[i] = activate<ACT_RELU>(v[0][i]); break;
                case ACT_GELU_TANH: h[i] = activate<ACT_GELU_TANH>(v[0][i]); break;
                case ACT_SILU: h[i] = activate<ACT_SILU>(v[0][i]); break;
                default: h[i] = v[0][i]; break;
            }
            if constexpr (GATED) h[i] *= v[G - 1][i];
        }
        const int row = Gemm::sum_row(tid), n = 64 * s + Gemm::sum_col(tid);
        if (row < a.M && n < a.N1) {
            typename Gemm::hvec o;
#pragma unroll
            for (int i = 0; i < VW / 2; ++i) o[i] = pack2<T>(h[2 * i], h[2 * i + 1]);
            const uint32_t off = (uint32_t)((row * (int64_t)a.N1 + n) * 2);   // written through
            if constexpr (VW == 2) __builtin_amdgcn_raw_buffer_store_b32(o[0], rh, off, 0, 16);
            else __builtin_amdgcn_raw_buffer_store_b64(o, rh, off, 0, 16);
        }
        __syncthreads();
        if (!more) break;
        s = sn; at = nx;
    }
}

template <typename T, bool GATED, int R, bool NT>
__device__ __forceinline__ void stream_body(const TwoPhaseArgs& a, char* smem, int tid, int xcd, int loc, int GX) {
    constexpr int BM = 16 * R;
    typedef StreamGemm<T, 1, R, NT> Gemm;
    float(*part)[BM][64] = reinterpret_cast<float(*)[BM][64]>(smem);
    volatile uint32_t& verdict = *reinterpret_cast<volatile uint32_t*>(smem);
    uint64_t t0 = 0, t1 = 0, t2 = 0;
    if (a.stats) t0 = wall_clock64();
    if (a.phases & 1) stream_first<T, GATED, R, NT>(a, part, tid, xcd, loc, GX);
    if (a.stats) t1 = wall_clock64();

    Gemm g;
    g.init(a.H, a.M, a.N1, a.W2, nullptr, (uint32_t)((uint64_t)a.N1 * a.N2 * 2), a.N2, tid);
    typename Gemm::Slot slot;
    const int NCB = (a.N2 + 63) / 64;
    int rb, u = 0, idx = loc;
    bool have = (a.phases & 2) && map_item(1, NCB * a.splits, 1, xcd, idx, rb, u);
    const auto next_item = [&](bool on, int u_) {
        if (!on) return g.item(a.N2, 0, 0, tid);
        const int cb = u_ % NCB, sp = u_ / NCB;
        const int k0 = sp * a.ksplit;
        return g.item(64 * cb, k0, min(a.N1, k0 + a.ksplit), tid);
    };
    typename Gemm::Item at = next_item(have, u);
    const auto fill_w = [&] { g.load_w(slot, at, 0); };
    bool ok = true;
    if (a.phases == 3) {
        // the first weights of the second phase travel while the workgroup waits
        ok = two_phase_rendezvous(a, verdict, tid, xcd, GX, (uint32_t)(a.wait_masks >> (8 * xcd)) & 0xffu, 1u, fill_w);
    } else {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        fill_w();
    }
    if (a.stats) t2 = wall_clock64();
    if (ok && have) {
        g.load_x(slot, at, 0);
        while (have) {
            int un = 0;
            idx += GX;
            const bool more = map_item(1, NCB * a.splits, 1, xcd, idx, rb, un);
            const typename Gemm::Item nx = next_item(more, un);
            f32x4 acc[1][R][4];
            g.run(slot, at, nx, acc);
            constexpr int VW = Gemm::VW;
            const typename Gemm::fvec v = g.sum(part, acc[0], tid);
            const int cb = u % NCB, sp = u / NCB, row = Gemm::sum_row(tid), n = 64 * cb + Gemm::sum_col(tid);
            if (row < a.M && n < a.N2) {
                if (a.splits > 1) {
                    float* plane = a.part + (size_t)sp * (size_t)a.M * a.N2;
                    *reinterpret_cast<typename Gemm::fvec*>(plane + (int64_t)row * a.N2 + n) = v;
                } else {
                    typename Gemm::hvec o;
#pragma unroll
                    for (int i = 0; i < VW / 2; ++i) o[i] = pack2<T>(v[2 * i], v[2 * i + 1]);
                    *reinterpret_cast<typename Gemm::hvec*>(reinterpret_cast<char*>(a.Y) + ((int64_t)row * a.N2 + n) * 2) = o;
                }
            }
            __syncthreads();
            have = more; u = un; at = nx;
        }
    }
    if (a.stats && tid == 0) {
        uint64_t* p = a.stats + 4 * blockIdx.x;
        p[0] = t1 - t0; p[1] = t2 - t1; p[2] = wall_clock64() - t2; p[3] = 0;
    }
}

template <typename T, bool GATED, int R> __global__ __launch_bounds__(64 * kWaves) void fused_stream_kernel(TwoPhaseArgs a) {
    __shared__ __attribute__((aligned(16))) char smem[(GATED ? 2 : 1) * kWaves * 16 * R * 64 * 4];
    const int tid = threadIdx.x, GX = gridDim.x >> 3;
    const int xcd = blockIdx.x & 7, loc = blockIdx.x >> 3;
    if (a.nt) stream_body<T, GATED, R, true>(a, smem, tid, xcd, loc, GX);
    else stream_body<T, GATED, R, false>(a, smem, tid, xcd, loc, GX);
    if (a.phases == 3) two_phase_leave(a, tid, gridDim.x);
}

template <typename T, bool GATED> static const void* stream_fn(int bm) {
    if (bm == 16) return (const void*)fused_stream_kernel<T, GATED, 1>;
    if (bm == 32) return (const void*)fused_stream_kernel<T, GATED, 2>;
    return nullptr;
}

hipError_t launch_fused_stream(int dtype, const TwoPhaseArgs& a, int bm, int grid, hipStream_t st) {
    const bool g = a.W3 != nullptr;
    if (a.U || a.conv_ic > 0 || a.M > bm) return hipErrorInvalidValue;
    const void* fn = dtype == 0 ? (g ? stream_fn<__bf16, true>(bm) : stream_fn<__bf16, false>(bm))
                                : (g ? stream_fn<_Float16, true>(bm) : stream_fn<_Float16, false>(bm));
    if (!fn || grid < 8 || (grid & 7) || a.splits < 1 || a.phases < 1 || a.phases > 3) return hipErrorInvalidValue;
    TwoPhaseArgs copy = a;
    void* params[] = {&copy};
    return launch_resident(fn, grid, params, st, 64 * kWaves);
}

}  // namespace ffuse
