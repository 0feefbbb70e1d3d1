// What the slice GEMM's kernels share on the device.
#pragma once

#include "oz_gemm_plan.h"

namespace oz {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int kMaxSyncSpins = 384;    // upper bound of the wait for the other workgroups of a round
constexpr int kMidSyncMinK = 24576;   // from this k on, workgroups also wait after every group of anti-diagonals

// Records this workgroup's arrival at *counter and, if `wait`, waits (bounded, about half a
// millisecond) until `target` workgroups have arrived.  The wait only improves cache locality:
// correctness does not depend on it, and every wave gets past it whatever the other workgroups do.
// A workgroup that did not meet the others in time (the chip is shared with another kernel, or workgroups are not
// placed as assumed) keeps counting its arrivals, which the others rely on, but stops waiting (`wait` of thread 0
// becomes false), so the cost of a wrong assumption is paid once.
__device__ __forceinline__ void round_sync(int32_t* counter, int target, bool& wait) {
    if (threadIdx.x == 0) {
        atomicAdd(counter, 1);
        if (wait) {
            bool met = false;
            for (int spin = 0; spin < kMaxSyncSpins && !met; ++spin) {
                met = __hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= target;
                if (!met) __builtin_amdgcn_s_sleep(8);
            }
            wait = met;
        }
    }
    asm volatile("s_barrier" ::: "memory");
}

// 64 lanes x 16 B from global memory into LDS: lane l's 16 bytes land at lds_addr + LDS_IMM + 16*l.
// The LDS byte address travels in M0 (set by the scalar add).  The compiler does not see this as a
// memory access, so completion is awaited with explicit s_waitcnt vmcnt(...) below.
// The global address is a wave-uniform base (scalar registers) plus a per-lane byte offset.
template <int LDS_IMM>
__device__ __forceinline__ void dma16(const uint8_t* gbase, uint32_t lane_off, uint32_t lds_addr) {
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(lds_addr), "v"(lane_off), "s"(gbase), "n"(LDS_IMM) : "memory", "scc");
}

// Waits until at most n of this wave's transfers are in flight, n rounded down to one of a few values.  The decision is a
// tree of three to four scalar branches: eighteen in a row cost the kernels on small tiles a tenth of a 64 of k.
__device__ __forceinline__ void wait_transfers(int n) {
#define OZ_WAIT(N) asm volatile("s_waitcnt vmcnt(" #N ")" ::: "memory")
    if (n < 4) {
        if (n <= 0) OZ_WAIT(0);
        else if (n < 2) OZ_WAIT(1);
        else OZ_WAIT(2);
    } else if (n < 12) {
        if (n < 6) OZ_WAIT(4);
        else if (n < 8) OZ_WAIT(6);
        else if (n < 10) OZ_WAIT(8);
        else OZ_WAIT(10);
    } else if (n < 24) {
        if (n < 16) OZ_WAIT(12);
        else OZ_WAIT(16);
    } else {
        if (n < 32) OZ_WAIT(24);
        else if (n < 48) OZ_WAIT(32);
        else OZ_WAIT(48);
    }
#undef OZ_WAIT
}

}  // namespace oz
