// Device-side helpers shared by the hand-scheduled kernels: compile-time loops, LDS
// operand reads issued from inline asm (so that their waits can be placed by hand) and
// the waits that go with them.
#ifndef HAT_DEVICE_UTIL_H
#define HAT_DEVICE_UTIL_H
#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

typedef _Float16 hat_f16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t hat_u32x4 __attribute__((ext_vector_type(4)));

// compile-time loop: f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>)
template <class F, int... I>
__device__ __forceinline__ void hat_static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void hat_static_for(F&& f) {
  hat_static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// 16 bytes per lane from LDS at addr + OFF (an immediate, 16 bits)
template <int OFF>
__device__ __forceinline__ hat_f16x8 hat_lds_read(uint32_t addr) {
  static_assert(OFF >= 0 && OFF < 65536, "ds_read offset field is 16 bits");
  hat_f16x8 v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
  return v;
}
// "operands have arrived": the wait is tied to the first register, the others are
// threaded through empty asm statements (volatile asm keeps its order) so that no
// MFMA using them can be scheduled above the wait.
// BEHIND: reads issued after those of v, which may still be on their way.
template <int BEHIND = 0, int N>
__device__ __forceinline__ void hat_wait_operands(hat_f16x8 (&v)[N]) {
  asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(v[0]) : "n"(BEHIND));
#pragma unroll
  for (int i = 1; i < N; ++i) asm volatile("" : "+v"(v[i]));
}
// A buffer whose loads need no vector instruction for their address (hat_load_lds).  The base is the same in all lanes; that it is, is not left to the
// compiler: what it takes for divergent it loads in a loop over the lanes' values.
__device__ __forceinline__ const void* hat_uniform(const void* p) {
  const uint64_t a = (uint64_t)(uintptr_t)p;
  return (const void*)(uintptr_t)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(a >> 32)) << 32 | (uint32_t)__builtin_amdgcn_readfirstlane((int)a));
}
// 16 bytes per lane from base + bytes + lane_bytes to LDS at dst + 16 * lane.  AUX 2: non-temporal.
template <int AUX>
__device__ __forceinline__ void hat_load_lds(const void* base, void* dst, int lane_bytes, int bytes) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc((void*)base, 0, -1, 0x00020000),
                                           (__attribute__((address_space(3))) void*)dst, 16, lane_bytes, bytes, 0, AUX);
}
template <int N>
__device__ __forceinline__ void hat_wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
#endif
