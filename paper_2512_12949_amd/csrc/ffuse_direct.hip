// Fused chain, "reduce" family on small row blocks (16 or 32 rows): operands go from global memory STRAIGHT to the
// registers of the wave that multiplies them.
//
// A workgroup owns a row block and a range of the hidden dimension, which it walks in slices of 64 columns:
//   first product : the waves split K (steps of 32 k, dealt in turn); every wave computes a partial
//                   [rows][64] tile with the loads of DEPTH steps in flight and no barrier between them;
//   exchange      : the partial tiles are summed in LDS, activated on complete sums (paper Sec. 4.3, Rule 3),
//                   gated, rounded to the operand type and left in LDS as the slice's block of H;
//   second product: every wave multiplies that block with its own columns of W2 (where there are fewer column blocks
//                   than waves, half the hidden columns each) into accumulators that stay in registers for the whole range.
// With one range the output goes straight to Y: one launch, no workspace traffic.  With several, each range stores
// its fp32 plane and the planes are summed in a fixed order (launch_finalize_planes).
//
// What bounds it: the problems it is for hold fewer bytes and flops than a launch lasts; what counts is how many
// memory round trips and barriers follow one another.  The two-phase kernel needs a device-wide rendezvous and,
// where a layer has few 64-column slices, leaves the first product to a handful of workgroups, each walking all of
// K alone; the 128-row reduce tiles walk K in LDS stages with a barrier each.  Here a slice costs two barriers and
// about K / 512 round trips.  Against that, operands are re-read from L2 by every row block.  Eight waves rather than
// four issue the loads and multiplies of a slice: most of these problems have one workgroup a CU or less, and the walk
// is bound by how fast its waves issue.  (Which forms keep four: direct_waves.)  Four -> eight: 3136 x 64 x 256 x 64 7.0 -> 5.7 us, 128 x 384 x 1536 x 384 10.8 ->
// 10.2, 3x3 chains 196 x 2304 x 256 x 1024 15.7 -> 14.8, 49 x 4608 x 512 x 2048 25.5 -> 23.3; 140 drawn shapes of up to 4 Gflop
// 3 % on average, those of this kernel 6.  (A ring of three or four steps a wave, with more of K padded: 0-20 % slower.)
// Outputs above 1024 columns with ranges of several slices spill 1-4 registers (78-80 with four waves, and 5-9 % slower).
//
// Measured (us, the best of the other plans -> this): 3x3 chains 196 pixels x 2304 x 256 x 1024 41 -> 15, 49 x 4608 x
// 512 x 2048 47 -> 23, 6272 x 576 x 64 x 256 21 -> 8; 128 x 384 x 1536 x 384 17.4 -> 10.2; 3136 x 64 x 256 x 64
// 8.9 -> 5.7.  It loses from about 1.5 Gflop on (200 x 1024 x 4096 x 1024: 28 against 34).  Issuing a slice's first W2
// loads a slice earlier was 3-5 % slower: the walk is bound by issue, not by the wait for those loads.
//
// Operand layouts: ffuse_octet.h.
#include "ffuse_octet.h"
#include "ffuse_launch.h"

namespace ffuse {

// R: tiles of 16 rows.  NW: waves (4 or 8).  Each wave multiplies NG blocks of 64 output columns; HS: the waves that share
// a column block split the slice's 64 hidden columns among them (2: halves) and sum their parts at the end.
// MORE: a range has several slices (with one there is nothing to load once its first product is under way).
// SHORT: the ring's DEPTH steps a wave hold all of K, and steps and column blocks that do not exist are branched over
// instead of loaded out of range (a range-checked load of zeros costs its issue slots all the same: 64 x 128 x 512 x
// 128 8.6 -> 6.3 us).  Longer K keeps straight-line turns: there the branches cost the overlap of the turns
// (128 x 512 x 2048 x 512 in one range: 97 us without, 141 with).
template <typename T, bool GATED, bool CONV, int R, int NG, int HS, bool SHORT, bool MORE, int DEPTH, int NW>
__global__ __launch_bounds__(64 * NW) void fused_direct_kernel(DirectArgs a) {
    constexpr int G = GATED ? 2 : 1, BM = 16 * R, CG = NW / HS;
    constexpr int HROW = 72;                             // elements of an H row in LDS (64 and a pad against bank conflicts)
    __shared__ __attribute__((aligned(16))) float part[G * NW][BM][64];
    __shared__ __attribute__((aligned(16))) uint16_t hs[BM][HROW];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 15, q = lane >> 4;
    const int cg = wave % CG, th = wave / CG;            // second product: column group, share of the hidden columns
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
    const int ksteps = ((K + 31) / 32 + NW * DEPTH - 1) / (NW * DEPTH) * DEPTH;   // a wave's steps per slice, whole turns of the ring
    uint32_t xoff[R];                                    // this lane's place in its rows of X and in 8 weight rows
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t row = m0 + 16 * r + c;
        xoff[r] = row < a.M ? ((uint32_t)row * (uint32_t)(CONV ? a.conv_ic : K) + 8u * (uint32_t)q) * 2u : kOob;
    }
    const uint32_t w1off = 8u * (uint32_t)q * w1row + 8u * (uint32_t)c, w2off = 8u * (uint32_t)q * w2row + 8u * (uint32_t)c;
    const auto load = [&](Slot& s, int ch, int step) {   // a wave's step of slice ch
        const int k0 = 32 * (NW * step + wave);
        if (!SHORT || k0 < K) {
            const bool ok = ch < ch_end && k0 + 8 * q < K;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if constexpr (CONV) {
                    // 32 k lie in one tap (conv_ic is a multiple of 32)
                    const int tap = k0 / a.conv_ic, ky = tap / 3 - 1, kx = tap % 3 - 1;
                    const bool in = ok && xoff[r] != kOob && (uint32_t)(py[r] + ky) < (uint32_t)a.conv_h && (uint32_t)(px[r] + kx) < (uint32_t)a.conv_w;
                    const int shift = ((ky * a.conv_w + kx) * a.conv_ic + k0 - tap * a.conv_ic) * 2;
                    s.x[r] = buf_load16(rx, in ? xoff[r] + (uint32_t)shift : kOob);
                } else {
                    s.x[r] = __builtin_amdgcn_raw_buffer_load_b128(rx, ok ? xoff[r] : kOob, 2u * (uint32_t)k0, 0);
                }
            }
            const uint32_t off = ok && 64 * ch + 4 * c < N1 ? w1off : kOob;
#pragma unroll
            for (int g = 0; g < G; ++g) load_octet(rw[g], off, (uint32_t)k0 * w1row + 128u * (uint32_t)ch, w1row, s.w[g]);
        }
    };
    const int ch_begin = range * a.slices;
#pragma unroll
    for (int u = 0; u < DEPTH; ++u) load(slot[u], ch_begin, u);

    f32x4 acc2[NG][R][4];
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc2[g][r][i] = f32x4{0.f, 0.f, 0.f, 0.f};

    for (int ch = ch_begin; ch < ch_end; ++ch) {
        u32x2 w2[NG > 1 ? 2 : 1][2 / HS][8];             // column blocks in flight, steps of 32 hidden columns
        const auto load2 = [&](int g) {
            const int col0 = 64 * (CG * g + cg);
            if (!SHORT || col0 < N2)
#pragma unroll
                for (int t = 0; t < 2 / HS; ++t) {
                    const int n = 64 * ch + 32 * ((2 / HS) * th + t);
                    load_octet(r2, col0 + 4 * c < N2 && n + 8 * q < N1 ? w2off : kOob, (uint32_t)n * w2row + 2u * (uint32_t)col0, w2row, w2[g & 1][t]);
                }
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
            if (SHORT && 32 * (NW * step + wave) >= K) return;
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const u32x4 b = octet_column(w.w[g], i);
#pragma unroll
                    for (int r = 0; r < R; ++r) acc[g][r][i] = Mma16<T>::mma(w.x[r], b, acc[g][r][i]);
                }
        };
        for (int s = 0; s + DEPTH < ksteps; s += DEPTH) {
#pragma unroll
            for (int u = 0; u < DEPTH; ++u) {
                multiply(slot[u], s + u);
                __builtin_amdgcn_sched_barrier(0);       // (loads moved above the transposes would take registers of their own)
                load(slot[u], ch, s + DEPTH + u);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (!MORE || (!GATED && !SHORT && R == 1 && ch + 1 == ch_end)) {   // the range's last turn: nothing left to load
#pragma unroll
            for (int u = 0; u < DEPTH; ++u) multiply(slot[u], ksteps - DEPTH + u);
        } else {
#pragma unroll
            for (int u = 0; u < DEPTH; ++u) {
                multiply(slot[u], ksteps - DEPTH + u);
                __builtin_amdgcn_sched_barrier(0);
                // Loads of a slice that is not there are branched over: range-checked zeros cost their issue slots (ranges of two
                // slices, averages of 8 shapes each: gated, 16 rows, K of 129-256 9.8 -> 9.2 us; 32 rows, K above 256 14.1 -> 13.5;
                // ungated, 16 rows, K of 65-256 on more than 256 workgroups 4 %).  Not on 16 rows with ungated long K: the last
                // turn has a form of its own above.  (readfirstlane: a condition that the compiler can fold into the loop's own
                // takes 130 registers in the 32-row short form, which has 128 for two workgroups a CU.)
                if ((!GATED && !SHORT && R == 1) || __builtin_amdgcn_readfirstlane(ch_end - ch) > 1) load(slot[u], ch + 1, u);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // acc[g][r][i][e]: row 16 r + 4 q + e, column 4 c + i of the slice
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    *reinterpret_cast<f32x4*>(&part[NW * g + wave][16 * r + 4 * q + e][4 * c]) =
                        f32x4{acc[g][r][0][e], acc[g][r][1][e], acc[g][r][2][e], acc[g][r][3][e]};
        __syncthreads();
        // VW columns of a row to a thread
        constexpr int VW = 16 * R * 64 / (64 * NW) < 4 ? 2 : 4, TPR = 64 / VW, RPP = 64 * NW / TPR;
        typedef __attribute__((ext_vector_type(VW))) float fvec;
        typedef __attribute__((ext_vector_type(VW / 2))) uint32_t hvec;
#pragma unroll
        for (int r = 0; r < BM / RPP; ++r) {
            const int row = RPP * r + tid / TPR, col = VW * (tid % TPR);
            fvec v[G];
#pragma unroll
            for (int g = 0; g < G; ++g) {
                v[g] = *reinterpret_cast<const fvec*>(&part[NW * g][row][col]);
#pragma unroll
                for (int p = 1; p < NW; ++p) v[g] += *reinterpret_cast<const fvec*>(&part[NW * g + p][row][col]);
            }
            hvec o;
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
                if (64 * ch + col >= N1) h[i] = 0.0f;    // (an infinity of X times the zero weights past N1 is not a number)
            }
#pragma unroll
            for (int i = 0; i < VW / 2; ++i) o[i] = pack2<T>(h[2 * i], h[2 * i + 1]);
            *reinterpret_cast<hvec*>(&hs[row][col]) = o;
        }
        __syncthreads();
        u32x4 hf[R][2 / HS];
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int t = 0; t < 2 / HS; ++t) hf[r][t] = *reinterpret_cast<const u32x4*>(&hs[16 * r + c][32 * ((2 / HS) * th + t) + 8 * q]);
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            if (g + 1 < NG) load2(g + 1);
            if (64 * (CG * g + cg) < N2) {
#pragma unroll
                for (int t = 0; t < 2 / HS; ++t)
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

    if constexpr (HS == 2) {                             // the second half's waves hand their part to the first half's
        __syncthreads();                                 // (the last slice's partial tiles have been read)
        f32x4* mine = reinterpret_cast<f32x4*>(&part[0][0][0]) + (cg * NG * R * 4) * 64 + lane;
        if (th) {
#pragma unroll
            for (int g = 0; g < NG; ++g)
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int i = 0; i < 4; ++i) mine[((g * R + r) * 4 + i) * 64] = acc2[g][r][i];
        }
        __syncthreads();
        if (th) return;
#pragma unroll
        for (int g = 0; g < NG; ++g)
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc2[g][r][i] += mine[((g * R + r) * 4 + i) * 64];
    }
    float* plane = a.part + (size_t)range * (size_t)a.M * N2;
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int64_t row = m0 + 16 * r + 4 * q + e;
                const int col = 64 * (CG * g + cg) + 4 * c;
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

// NC: 256-column blocks of the output
template <typename T, bool GATED, bool CONV, int R, int NC, bool SHORT, bool MORE, int NW> static const void* direct_variant() {
    constexpr int DEPTH = SHORT ? 8 / NW : 2;
    if constexpr (NW == 4) return (const void*)fused_direct_kernel<T, GATED, CONV, R, NC, 1, SHORT, MORE, DEPTH, 4>;
    else if constexpr (NC == 1) return (const void*)fused_direct_kernel<T, GATED, CONV, R, 1, 2, SHORT, MORE, DEPTH, 8>;
    else return (const void*)fused_direct_kernel<T, GATED, CONV, R, NC / 2, 1, SHORT, MORE, DEPTH, 8>;
}

template <typename T, bool GATED, bool CONV, bool MORE> static const void* direct_fn(int bm, int ng, bool short_k, int waves) {
    if constexpr (!CONV) {
        if (short_k) {
            if constexpr (!GATED && !MORE)
                if (waves == 4) return bm == 16 && ng == 1 ? direct_variant<T, false, false, 1, 1, true, false, 4>() : nullptr;
            if (waves != 8) return nullptr;
            if (bm == 16) return ng == 1 ? direct_variant<T, GATED, false, 1, 1, true, MORE, 8>() : direct_variant<T, GATED, false, 1, 2, true, MORE, 8>();
            if (bm == 32) return ng == 1 ? direct_variant<T, GATED, false, 2, 1, true, MORE, 8>() : direct_variant<T, GATED, false, 2, 2, true, MORE, 8>();
            return nullptr;
        }
    }
    constexpr int NW = GATED ? 4 : 8;
    if (waves != NW) return nullptr;
    if (bm == 16) {
        if (ng == 1) return direct_variant<T, GATED, CONV, 1, 1, false, MORE, NW>();
        if (ng == 2) return direct_variant<T, GATED, CONV, 1, 2, false, MORE, NW>();
        if (ng == 4) return direct_variant<T, GATED, CONV, 1, 4, false, MORE, NW>();
        if (ng == 8) return direct_variant<T, GATED, CONV, 1, 8, false, MORE, NW>();
    }
    if (bm == 32) {
        if (ng == 1) return direct_variant<T, GATED, CONV, 2, 1, false, MORE, NW>();
        if (ng == 2) return direct_variant<T, GATED, CONV, 2, 2, false, MORE, NW>();
    }
    return nullptr;
}

template <typename T> static const void* direct_fn(bool gated, bool conv, bool more, int bm, int ng, bool short_k, int waves) {
    if (conv) return more ? direct_fn<T, false, true, true>(bm, ng, false, waves) : direct_fn<T, false, true, false>(bm, ng, false, waves);
    if (gated) return more ? direct_fn<T, true, false, true>(bm, ng, short_k, waves) : direct_fn<T, true, false, false>(bm, ng, short_k, waves);
    return more ? direct_fn<T, false, false, true>(bm, ng, short_k, waves) : direct_fn<T, false, false, false>(bm, ng, short_k, waves);
}

hipError_t launch_fused_direct(int dtype, const DirectArgs& a, int bm, int ng, int cus, hipStream_t st) {
    const bool g = a.W3 != nullptr, conv = a.conv_ic > 0;
    if (conv && (g || a.conv_ic % 32 || a.K != 9 * a.conv_ic || a.conv_h < 1 || a.conv_w < 1)) return hipErrorInvalidValue;
    if (a.ranges < 1 || a.slices < 1 || (int64_t)a.ranges * a.slices * 64 < a.N1 || (int64_t)(a.ranges - 1) * a.slices * 64 >= a.N1 ||
        a.N2 > 256 * ng || (a.ranges > 1 && !a.part)) return hipErrorInvalidValue;
    const bool short_k = !conv && a.K <= 256 && ng <= 2;
    const int64_t grid = (a.M + bm - 1) / bm * a.ranges;
    const bool shared = grid > cus;
    const int waves = direct_waves(g, short_k, bm, ng, a.slices, shared);
    // Where workgroups share a CU, the form for several slices with one slice too: it keeps less across the exchange, 128
    // registers instead of 132 (32 rows) and 124 instead of 138 (gated, 16 rows), and two workgroups of eight waves on a CU may
    // have 128 each.  us, averages of 8 shapes on 257-512 workgroups: 32 rows, K of 65-128 12.0 -> 10.6, above 16.4 -> 15.0; gated 13.8 ->
    // 12.7.
    const bool more = a.slices > 1 || (shared && short_k && ng == 1 && bm == (g ? 16 : 32));
    const void* fn = dtype == 0 ? direct_fn<__bf16>(g, conv, more, bm, ng, short_k, waves) : direct_fn<_Float16>(g, conv, more, bm, ng, short_k, waves);
    if (!fn || grid > 0x7fffffff) return hipErrorInvalidValue;
    DirectArgs copy = a;
    void* params[] = {&copy};
    hipError_t e = hipLaunchKernel(fn, dim3((unsigned)grid), dim3(64 * waves), params, 0, st);
    if (e == hipSuccess && a.ranges > 1) e = launch_finalize_planes(dtype, a.part, a.Y, a.M * a.N2, a.ranges, st);
    return e;
}

}  // namespace ffuse
