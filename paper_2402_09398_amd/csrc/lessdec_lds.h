// Data from memory straight into the LDS, and the waits that go with it.
#pragma once

#include "lessdec_common.h"

namespace lessdec {

typedef __attribute__((address_space(3))) unsigned char lds_bytes;
__device__ inline unsigned lds_offset(const unsigned char *p) { return (unsigned)(unsigned long long)(lds_bytes *)p; }

// BYTES (4 or 16) a lane from memory into the LDS: lane l's from base + offset (of the lane), to `to` + BYTES l.  base, bytes
// (readable from base on) and to are the same for the whole wave.  Written as asm because the compiler, which
// cannot tell the buffers of a pipeline apart, would wait for every transfer before the next LDS read; nothing is
// returned in registers.  The readers stand behind lds_arrived<..>() of the wave that loaded and a barrier.
// (The wait states between a vector instruction that writes a scalar register and a load that reads it are the compiler's affair for
// its own loads only: base, bytes and to come from scalar arithmetic, which needs none; a test reads the assembly.  m0 is a
// reserved register, about which the compiler warns in a clobber list; it is named so that no value of its own is
// expected to live there across the block.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int BYTES>
__device__ inline void lds_load(const void *base, unsigned bytes, int offset, unsigned char *to)
{
  typedef unsigned v4u __attribute__((ext_vector_type(4)));
  const unsigned long long b = reinterpret_cast<unsigned long long>(base);
  const v4u rsrc = {(unsigned)b, (unsigned)(b >> 32) & 0xffffu, bytes, 0x00020000u};
  if constexpr (BYTES == 16)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 : : "s"(lds_offset(to)), "v"(offset), "s"(rsrc) : "m0", "memory");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds"
                 : : "s"(lds_offset(to)), "v"(offset), "s"(rsrc) : "m0", "memory");
}
#pragma clang diagnostic pop
// all but the wave's latest N memory operations have arrived
template <int N>
__device__ inline void lds_arrived()
{
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}
// workgroup barrier for the LDS alone: loads from memory stay in flight
__device__ inline void lds_barrier()
{
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

}  // namespace lessdec
