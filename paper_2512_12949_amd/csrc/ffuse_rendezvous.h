// What the two-phase family's kernels share: the item map, the device-wide rendezvous between their phases and the
// way they leave its counters (ffuse_two_phase.hip, ffuse_stream.hip).
#pragma once
#include "ffuse_dev.h"
#include "ffuse_launch.h"

namespace ffuse {

// item `idx` of XCD `xcd` -> (row block i, slice s); false past the XCD's share
__device__ __forceinline__ bool map_item(int MB, int S, int raster, int xcd, int idx, int& i, int& s) {
    const int total = MB * S;
    const int per = (total + 7) / 8;
    const int v = xcd * per + idx;
    if (idx >= per || v >= total) return false;
    const int panel = v / (raster * S);
    const int rem = v - panel * raster * S;
    const int rows = min(raster, MB - panel * raster);
    i = panel * raster + rem % rows;
    s = rem / rows;
    return true;
}

// One device-wide rendezvous of a launch's workgroups; `round` counts them from 1 (the group counters keep
// counting up: round r is complete for a group when its counter has reached r times the group's size).
// The tiles stored before it were stored write-through, so once this workgroup's stores have completed
// they are visible device-wide and arriving takes no L2 write-back (which costs 5+ us when
// the L2 holds a few MB of dirty lines).  A workgroup arrives with ONE atomic add whose
// result it does not wait for, on the counter of its group of G/8 workgroups (eight counters
// a cache line apart: 256 adds on one word take three times as long as 32 on each of 8), and
// then polls, together, the counters of the groups in `wait`: those whose tiles its own group reads next
// (a.wait_masks, enumerated on the host from the two item maps: often its own group alone, and
// then a group that is done starts phase 2 while others still stream their weights).  Measured in
// isolation, waiting for all eight: 1.8-3.9 us, against 3.8-6.5
// with a returning add plus a second, group-to-global add, and 7-12.5 with a releasing add.
// Bounded: on expiry the error word is set and every workgroup leaves (returns false).
// `between` runs after the arrival and before the wait, in every wave (loads that may be issued early: the poll returns behind
// those of its own wave, so the LDS-direct kernels leave them to the other waves; the streaming kernel's go out in all).
template <class Between>
__device__ __forceinline__ bool two_phase_rendezvous(const TwoPhaseArgs& a, volatile uint32_t& verdict, int tid, int xcd, int GX,
                                                     uint32_t wait, uint32_t round, Between&& between) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0)
        __hip_atomic_fetch_add(a.flags + kTwoPhaseGroupWord * (1 + xcd), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    between();
    if (tid == 0) {
        uint32_t ok = 1;
        uint32_t spins = 0;
        const uint32_t target = round * (uint32_t)GX + (uint32_t)a.extra_arrivals;
        for (;;) {
            uint32_t fewest = ~0u;
#pragma unroll
            for (int g = 0; g < 8; ++g)
                if ((wait >> g) & 1u) {
                    const uint32_t n = __hip_atomic_load(a.flags + kTwoPhaseGroupWord * (1 + g), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    fewest = n < fewest ? n : fewest;
                }
            if (fewest >= target) break;
            __builtin_amdgcn_s_sleep(1);
            // gives up after spin_limit polls, or (looked at every 1024 polls) when another workgroup has
            if (++spins >= a.spin_limit ||
                ((spins & 1023u) == 0 && __hip_atomic_load(a.flags + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)) {
                __hip_atomic_fetch_or(a.flags + 2, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                ok = 0;
                break;
            }
        }
        verdict = ok;
    }
    __syncthreads();
    // No cache invalidate here.  An agent-scope acquire would drop this XCD's whole L2 (measured: 4-5 us
    // with the L2 full of weight lines), and there is nothing stale to drop: the caches were emptied of
    // other agents' data when the kernel started, nobody has read a byte of H since (phase 1 only writes
    // it), and the lines this XCD wrote itself hold what it wrote.  (Probed on the device: two XCDs
    // writing halves of the same lines, then reading each other's halves after this barrier, launch
    // after launch, see fresh data without an invalidate; they see stale data only if they had READ the
    // lines earlier in the same kernel.)
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    const bool ok = verdict != 0;
    __syncthreads();   // everybody has read the word before the next loads reuse its place
    return ok;
}

// The last workgroup to get here resets the counters for the next launch, and moves this launch's
// error word to where the host reads it: a wait that expired once must not make the next launch give up.
__device__ __forceinline__ void two_phase_leave(const TwoPhaseArgs& a, int tid, int G) {
    __syncthreads();
    if (tid == 0) {
        const uint32_t prev = __hip_atomic_fetch_add(a.flags + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (prev == (uint32_t)G - 1u) {
            __hip_atomic_store(a.flags + 1, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            for (int i = 0; i < 8; ++i)
                __hip_atomic_store(a.flags + kTwoPhaseGroupWord * (1 + i), 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const uint32_t verdict_word = __hip_atomic_load(a.flags + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(a.flags + 3, verdict_word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(a.flags + 2, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

}  // namespace ffuse
