// Every layer of a small matrix in one launch, on the workgroups of one XCD.
//
// A layer of n <= ~450 takes a few microseconds of work; a launch of its own costs it 2.2 us plus the
// trip of its operands through memory (the launch boundary writes back and invalidates the L2s).
// Here the workgroups of one XCD work through the items (layer, tile) and hand them over inside that
// XCD's L2: the barrier between two layers with its data takes 0.8 us for 10 workgroups and 1.1 us
// for 36 (a cache invalidate per workgroup instead of device-coherent loads: 1.3 and 3.2 us).
//
// Protocol. The first workgroup to arrive makes its XCD the owner; workgroups on other XCDs leave.
// Those on the owner take tickets, one per item in layer-major order. An item of layer l starts when
// l x tiles items are done. Every wait is on smaller tickets, each held by a running workgroup that
// itself only waits on smaller ones, so the smallest unfinished ticket always proceeds: no deadlock
// whatever the number of resident workgroups, and no assumption on which XCD a workgroup runs on
// (the launch offers an eighth of its workgroups, those of one value of blockIdx % 8, which the
// hardware deals to one XCD; if it did not, fewer would stay). Producers' stores complete in the
// L2 (vmcnt(0) in every wave, then a barrier) before the item is counted; readers load with sc1,
// which does not take the CU's L1's word for it. Waits are bounded (~5 s): one that gives up sets
// the error flag, and its item comes out as NaN and is not counted. The layers after it then never have
// their count, so every wait of theirs gives up too (the flag ends it) and all of them come out as NaN:
// none starts on what a late workgroup has yet to store.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fe {

constexpr int kResOwner = 0, kResTicket = 32, kResDone = 64, kResErr = 96;   // ints, one line each
constexpr int kResInts = 128;
constexpr int kResMaxL = 96;   // layers whose coefficients travel with the launch
constexpr int kCoherentLoad = 16;   // cache policy sc1

struct ResidentArgs {
    int32_t* ctl;      // kResInts ints, zero before the launch
    int ntiles, L;
    int spin_limit;    // polls before a wait gives up
    int stuck;         // to test the give-up path: the item whose wait cannot end (kNoItem, kEveryItem)
};
constexpr int kNoItem = -1, kEveryItem = -2;

// Calls item(layer, tile, gave_up) for every item this workgroup gets; item may use all threads and
// barriers. Items end with all their stores complete.
template <class F>
__device__ __attribute__((always_inline)) inline void resident_items(const ResidentArgs& R, F&& item) {
    __shared__ int s_ticket, s_bad;
    if (blockIdx.x % 8 != 0) return;
    const int total = R.ntiles * R.L;
    int next = total;   // thread 0's
    if (threadIdx.x == 0) {
        int x;
        asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID, 0, 4)" : "=s"(x));
        int seen = 0;
        const bool mine = __hip_atomic_compare_exchange_strong(R.ctl + kResOwner, &seen, x + 1,
                                                               __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                               __HIP_MEMORY_SCOPE_AGENT) ||
                          seen == x + 1;
        if (mine)
            next = __hip_atomic_fetch_add(R.ctl + kResTicket, 1, __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT);
        s_ticket = next;
    }
    __syncthreads();
    int t = __builtin_amdgcn_readfirstlane(s_ticket);
    while (t < total) {
        const int layer = t / R.ntiles, tile = t - layer * R.ntiles;
        if (threadIdx.x == 0) {
            const int need = t == R.stuck || R.stuck == kEveryItem ? INT32_MAX : layer * R.ntiles;
            int spins = 0, bad = 0;
            // The next ticket now: its trip runs beside the wait (the holder of a ticket may be busy
            // with a smaller one), and it is back before the item's loads, whose waits count on
            // nothing else being in flight (an atomic's return is not ordered with loads).
            next = __hip_atomic_fetch_add(R.ctl + kResTicket, 1, __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT);
            while (__hip_atomic_load(R.ctl + kResDone, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) <
                   need) {
                ++spins;
                if (spins > R.spin_limit ||
                    (spins % 64 == 0 &&
                     __hip_atomic_load(R.ctl + kResErr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
                    __hip_atomic_store(R.ctl + kResErr, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    bad = 1;
                    break;
                }
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            s_bad = bad;
        }
        __syncthreads();
        const bool gave_up = __builtin_amdgcn_readfirstlane(s_bad) != 0;
        item(layer, tile, gave_up);
        if (threadIdx.x == 0) s_ticket = next;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (threadIdx.x == 0 && !gave_up)
            __hip_atomic_fetch_add(R.ctl + kResDone, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        t = __builtin_amdgcn_readfirstlane(s_ticket);
    }
}

}  // namespace fe
