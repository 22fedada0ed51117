// Small device helpers shared by the kernel files of libfmtc (wavefront = 64 lanes).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fmtc {

__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// x + (x of the lane the control word names), 0 where that lane does not exist or the row is masked out
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_add(uint32_t x) {
    return x + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROW_MASK, 0xf, false);
}
// Inclusive prefix sum over the 64 lanes.  row: the sum within the lane's row of 16 lanes (lane 15 of a row
// holds the row total); half: the sum within the lane's half of the wavefront (lanes 31 and 63 hold the totals).
__device__ __forceinline__ uint32_t wave_inclusive_scan_rows(uint32_t v, uint32_t& row, uint32_t& half) {
    v = dpp_add<0x111, 0xf>(v);  // row_shr:1
    v = dpp_add<0x112, 0xf>(v);  // row_shr:2
    v = dpp_add<0x114, 0xf>(v);  // row_shr:4
    v = dpp_add<0x118, 0xf>(v);  // row_shr:8
    row = v;
    v = dpp_add<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
    half = v;
    v = dpp_add<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
    return v;
}

// exclusive prefix sum over the 64 lanes
__device__ __forceinline__ uint32_t wave_exclusive_scan(uint32_t v) {
    uint32_t row, half;
    return wave_inclusive_scan_rows(v, row, half) - v;
}

// The same for 64-bit values (modulo 2^64): pieces of 20, 20 and 24 bits, whose sums over 64 lanes fit 32 bits, by the scan
// above (shuffles through the LDS crossbar instead: six dependent round trips, 0.35 us of every table build).
__device__ __forceinline__ unsigned long long wave_inclusive_scan64(unsigned long long v) {
    uint32_t row, half;
    const uint32_t a = wave_inclusive_scan_rows((uint32_t)v & 0xfffffu, row, half);
    const uint32_t b = wave_inclusive_scan_rows((uint32_t)(v >> 20) & 0xfffffu, row, half);
    const uint32_t c = wave_inclusive_scan_rows((uint32_t)(v >> 40), row, half);
    return (unsigned long long)a + ((unsigned long long)b << 20) + ((unsigned long long)c << 40);
}

// Words that other workgroups of the same kernel read while it runs go through these: device-scope relaxed
// atomics bypass the caches that are private to a part of the chip, so no fence (a cache write-back here)
// is needed as long as every such word carries its own "valid" mark.
__device__ __forceinline__ void publish64(unsigned long long* p, unsigned long long v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void publish32(uint32_t* p, uint32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long peek64(const unsigned long long* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One wavefront's 64 x 16 (or 64 x 4) bytes from global memory straight into LDS, lane l to lds_base + 16 l
// (4 l).  Written as assembly because the compiler, which cannot tell the LDS stages apart, would hold every
// later LDS read until all transfers it knows of have landed -- the full latency, in every step; the kernel
// counts its loads in flight itself (s_waitcnt vmcnt, then a barrier) before it reads a stage.
typedef __attribute__((address_space(3))) void lds_void_t;
template <int BYTES>
__device__ __forceinline__ void load_to_lds(const void* src, void* lds_base) {
    const uint32_t base = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(uintptr_t)(lds_void_t*)lds_base);
    uint32_t keep;
    if constexpr (BYTES == 16)
        asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off\n\ts_mov_b32 m0, %0"
                     : "=&s"(keep) : "v"(src), "s"(base) : "memory");
    else
        asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %1, off\n\ts_mov_b32 m0, %0"
                     : "=&s"(keep) : "v"(src), "s"(base) : "memory");
}

// Wait until at most N of this wavefront's loads are in flight (they complete in order); no memory access
// moves across it.  A memory operation the caller's count does not know of (the compiler may add some) can only
// make the wait stricter: issued after the awaited load, it takes one of the N places.
template <int N>
__device__ __forceinline__ void wait_loads() {
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

}  // namespace fmtc
