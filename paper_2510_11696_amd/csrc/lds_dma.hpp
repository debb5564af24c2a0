// Memory -> LDS requests without registers, and the waits that go with them (gfx950: 16 bytes per lane).
#pragma once
#include "common.hpp"

namespace qerl {

typedef __attribute__((address_space(3))) u32x4 lds_chunk;
__device__ __forceinline__ uint32_t lds_address(u32x4* p) { return (uint32_t)(uintptr_t)(lds_chunk*)p; }

// A pointer that is the same in every lane, in scalar registers (the compiler does not always see that it is)
__device__ __forceinline__ const uint8_t* uniform_pointer(const void* p) {
  const uint64_t v = (uint64_t)(uintptr_t)p;
  const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v), hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
  return reinterpret_cast<const uint8_t*>((uintptr_t)(hi << 32 | lo));
}

// 16 bytes per lane from base + offset to LDS, the wave's 1 KiB at lds_bytes (uniform).  In assembly because the compiler,
// which would see the builtin as a store to LDS, waits for ALL requests before every LDS read that follows; nothing it
// tracks is written here, and its own counts only become stricter.  Waiting for the data is lds_wait_barrier's.
// m0 is among the clobbers, so that the compiler sets it again should it ever use it around a request; as the register is reserved
// to it, it warns of that.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void lds_request(uint32_t lds_bytes, const void* base, uint32_t offset) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_bytes), "v"(offset), "s"(base) : "memory", "m0");
}
// the same from a 64-bit address per lane
__device__ __forceinline__ void lds_request64(uint32_t lds_bytes, const void* src) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_bytes), "v"(src) : "memory", "m0");
}
#pragma clang diagnostic pop
// Wait until at most N vector-memory requests of this wave are outstanding and its own LDS reads are over (what they read
// may be refilled next), then meet the workgroup.  Requests return in order, so N is the number issued after the ones
// needed; only requests that cannot be dropped may be counted (the compiler removes loads whose data nothing uses).
template <int N>
__device__ __forceinline__ void lds_wait_barrier() {
  static_assert(N < 64, "vmcnt has six bits");
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}
// LDS traffic only: requests to LDS stay in flight
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

}  // namespace qerl
