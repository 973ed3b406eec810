// Copies straight from global memory to LDS, without registers, and the waits that go with them.
//
// They are issued and waited for by hand: told about them, the compiler would wait for all of them in front of every
// LDS read.  It does not see them, and loads return in order, so that its own waits (for its own loads) are for no less
// than they need.  A wavefront waits for its copies before it ends: its LDS belongs to another block then.
#pragma once
#include "any4_device.h"

namespace any4 {

// waits for LDS, leaves global loads in flight
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
// at most LEFT of this wavefront's vector memory operations are outstanding
template <int LEFT> __device__ __forceinline__ void loads_left() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LEFT) : "memory"); }

// (m0 is a reserved register: the compiler sets it in front of each use of its own and keeps no value of the
// program in it, but merges equal settings where it sees no other.  The clobber shows it this one; that nothing is
// saved and restored around the statement, which is what the warning says, is not needed.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
// 64 lanes x 16 bytes, lane l's from base + voff to lds + 16 l
__device__ __forceinline__ void copy_to_lds(uint32_t lds, const void* base, uint32_t voff) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(voff), "s"(base) : "m0", "memory");
}
// the same from an address of the lane's own
__device__ __forceinline__ void copy_to_lds_from(uint32_t lds, const void* from) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(from) : "m0", "memory");
}
// 64 lanes x 4 bytes (WORDS) or x 2 bytes, each widened with zeros to a word: lane l's goes to lds + 4 l
template <bool WORDS> __device__ __forceinline__ void copy_values_to_lds(uint32_t lds, const void* base, uint32_t voff) {
    if constexpr (WORDS) asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(lds), "v"(voff), "s"(base) : "m0", "memory");
    else asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_ushort %1, %2" ::"s"(lds), "v"(voff), "s"(base) : "m0", "memory");
}
// the same from an address of the lane's own
template <bool WORDS> __device__ __forceinline__ void copy_values_to_lds_from(uint32_t lds, const void* from) {
    if constexpr (WORDS) asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(lds), "v"(from) : "m0", "memory");
    else asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_ushort %1, off" ::"s"(lds), "v"(from) : "m0", "memory");
}
#pragma clang diagnostic pop

}  // namespace any4
