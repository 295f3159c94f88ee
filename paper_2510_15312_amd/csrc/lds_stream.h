// Direct loads from memory to LDS, the waits that go with them, and the order of workgroups over the
// compute dies: shared by the many-row GEMM and attention kernels.
#pragma once

#include <type_traits>

#include "vf_internal.h"

namespace {

template <int LO, int HI, typename F> __device__ __forceinline__ void static_for(F &&f) {
    if constexpr (LO < HI) {
        f(std::integral_constant<int, LO>{});
        static_for<LO + 1, HI>(f);
    }
}

// One fragment from memory straight to LDS (lds: its address there, the same for the whole wavefront;
// lane_off: 16 * lane).  Inline because the compiler makes every LDS read wait for all such loads in
// flight; the kernels count them themselves (vm_wait).  The destination goes through m0, which needs one
// idle cycle before the load.
// ONCE: nobody else reads it (non-temporal).
template <int LDS_OFF, bool ONCE = false> __device__ __forceinline__ void fragment_to_lds(const void *src, unsigned lane_off, unsigned lds) {
    if constexpr (ONCE)
        asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                     : : "s"(lds), "v"(lane_off), "s"(src), "n"(LDS_OFF) : "memory", "scc");
    else
        asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                     : : "s"(lds), "v"(lane_off), "s"(src), "n"(LDS_OFF) : "memory", "scc");
}
// until at most N of this wavefront's vector memory operations are outstanding
template <int N> __device__ __forceinline__ void vm_wait() { asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory"); }
// until at most min(r, R) stages of L loads each are outstanding
template <int R, int L> __device__ __forceinline__ void stage_wait(int r) {
    if constexpr (R > 0) {
        if (r >= R) vm_wait<R * L>();
        else stage_wait<R - 1, L>(r);
    } else {
        vm_wait<0>();
    }
}
__device__ __forceinline__ unsigned lds_address(const void *p) {
    return (unsigned)(uintptr_t)(__attribute__((address_space(3))) const unsigned char *)p;
}

// Position of workgroup w of `total` in an order whose neighbours share a compute die (workgroup w runs
// on die w % 8, each with an L2 of its own).
__device__ __forceinline__ int die_order(int w, int total) {
    const int die = w & 7, idx = w >> 3;
    const int per = (total + 7) >> 3, full = total & 7;   // dies below `full` hold `per`, the others one less
    return full == 0 || die < full ? die * per + idx : full * per + (die - full) * (per - 1) + idx;
}

}  // namespace
