// Pieces that every kernel with asynchronous global -> LDS copies shares.
#pragma once
#include <hip/hip_runtime.h>

#include "device_once.h"

#define DDS_LDS_AS __attribute__((address_space(3)))

namespace dds {
namespace {

// Lane L of a wave copies 16 bytes from its own address to bytes [16L, 16L+16) behind an LDS address that all lanes share.
__device__ __forceinline__ void dma16(const void* gsrc, uint32_t lds_base_uniform) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(gsrc), "s"(lds_base_uniform) : "memory", "m0");
}
// Same copy with the address split into a wave-uniform 64-bit base (SGPR pair) and a per-lane
// unsigned 32-bit byte offset: the per-copy address arithmetic stays on the scalar unit.
__device__ __forceinline__ void dma16s(const void* gbase_uniform, uint32_t goff, uint32_t lds_base_uniform) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(goff), "s"(gbase_uniform), "s"(lds_base_uniform) : "memory", "m0");
}
template <int N> __device__ __forceinline__ void wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
__device__ __forceinline__ void wg_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// floor(n / d) == __umulhi(n, mul) >> shift for 0 <= n < 2^31: mul = floor(2^(31+l) / d) + 1 with 2^(l-1) < d <= 2^l
// exceeds 2^(31+l) / d by at most 2^l / d, which the division of a 31-bit n never sees
struct Divisor {
  uint32_t mul;
  int shift;
};
inline Divisor make_divisor(int d) {  // d >= 2
  int l = 1;
  while ((1ll << l) < d) ++l;
  return Divisor{(uint32_t)(((1ull << (31 + l)) / (unsigned)d) + 1), l - 1};
}
// The same with 1 among the divisors: floor(n / d) == divide(n, make_divisor1(d))
inline Divisor make_divisor1(int d) {
  int l = 0;
  while ((1ll << l) < d) ++l;
  return Divisor{(uint32_t)(((1ull << (31 + l)) / (unsigned)d) + 1), l};
}
__device__ __forceinline__ uint32_t divide(uint32_t n, Divisor d) { return __umulhi(2 * n, d.mul) >> d.shift; }

}  // namespace

// Lets a kernel have all 160 KB of LDS on the current device (gemm.hip). A failure is the launch's to report.
void allow_whole_lds(DeviceOnce& once, const void* kernel);

}  // namespace dds
