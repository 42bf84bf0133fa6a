// Loads from memory straight to LDS (gfx950: 16 bytes a lane, 1 KB a wave).
// Written as asm because the compiler waits for every such load in flight before
// any LDS read (it cannot tell stages apart): whoever issues one waits for it with
// s_waitcnt vmcnt before a barrier.  There is no output register; m0 is set for
// each load, one wait state before it is used.  The compiler keeps m0 reserved (it
// cannot be named as clobbered) and does not look into asm for hazards, so nothing
// else in the kernels that include this may use m0, and no vector instruction may
// write a load's scalar operands just before it: test_lds_load_asm.py reads their
// assembly for both.
#pragma once

#include <type_traits>

#include "kernels.h"

typedef int i32x4 __attribute__((ext_vector_type(4)));

// LDS byte address of a __shared__ object
WAR_DEV uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

// Lane l's 16 bytes at rsrc + voff go to LDS byte lds + 16 l; past the
// descriptor's size they are zero.  NT: non-temporal.
template <bool NT>
WAR_DEV void load_lds16(uint32_t lds, int voff, i32x4 rsrc) {
  if constexpr (NT)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen nt lds" ::"s"(lds), "v"(voff),
                 "s"(rsrc)
                 : "memory");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds), "v"(voff),
                 "s"(rsrc)
                 : "memory");
}
WAR_DEV i32x4 make_rsrc(const void* p, int64_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(p);
  const uint32_t n = bytes < 0xffffffffLL ? (uint32_t)bytes : 0xffffffffu;
  return i32x4{__builtin_amdgcn_readfirstlane((int)(uint32_t)a), __builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32)),
               (int)n, 0x00020000};
}

// The same from base + voff, base the same for all lanes (five wait states between
// a VALU write of a scalar register and its use by a load).
WAR_DEV void load_lds16(uint32_t lds, const bf16_t* base, uint32_t voff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(voff), "s"(base)
               : "memory");
}
