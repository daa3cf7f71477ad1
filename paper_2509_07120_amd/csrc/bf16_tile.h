// What the bf16 matrix kernels share: operand types, the swizzle of row-major tiles of 128-byte rows in LDS, and
// direct-to-LDS loads.
#pragma once

#include <hip/hip_runtime.h>

namespace bsga {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

#define LDS_PTR(T, p) ((const T __attribute__((address_space(3)))*)(p))

// chunk swizzles: 16-byte chunk c of tile row r is stored at chunk position c ^ swz(r), swz_k in tiles whose rows are read whole (K, and both
// operands of a linear layer), swz_v in those that are read transposed (V)
__device__ __forceinline__ int swz_k(int row) { return (row ^ (row >> 3)) & 7; }
__device__ __forceinline__ int swz_v(int row) { return (row & 3) << 1; }

__device__ __forceinline__ unsigned pack_bf16(float a, float b) {
  const f32x2 two = {a, b};
  return __builtin_bit_cast(unsigned, __builtin_convertvector(two, bf16x2));
}

// the lane's number, through an instruction that the compiler does not see through: nothing that is computed from it can be
// made ahead of it and kept in registers
__device__ __forceinline__ int fresh_lane() {
  int l;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
  return l;
}

// 16 bytes per lane from a raw buffer straight into LDS (buffer_load_dwordx4 ... lds): lane i's
// data lands at LDS byte address lds_base + lds_imm + 16 i.  voff is the per-lane byte offset, soff a
// wave-uniform one; lanes whose offset is past the buffer's size get zeros.  Written as inline
// assembly on purpose: the compiler then does not count these loads as LDS writes and so does not
// make later LDS reads of the *other* buffer wait for them; the kernel orders them itself
// (s_waitcnt vmcnt + barrier).  M0 (the LDS base of the load) is declared clobbered; nothing else in
// these kernels uses it.
template <unsigned LDS_IMM>
__device__ __forceinline__ void dma16(i32x4 rsrc, unsigned voff, unsigned soff, unsigned lds_base) {
  asm volatile(
      "s_add_u32 m0, %0, %4\n\t"
      "s_nop 0\n\t"  // one wait state between a scalar write of M0 and an LDS-DMA instruction that reads it
      "buffer_load_dwordx4 %1, %2, %3 offen lds"
      :
      : "s"(lds_base), "v"(voff), "s"(rsrc), "s"(soff), "n"(LDS_IMM)
      : "memory", "m0", "scc");
}

// raw buffer descriptor over [base, base + bytes): stride 0, 32-bit element data format
__device__ __forceinline__ i32x4 make_rsrc(const void* base, unsigned bytes) {
  const unsigned long long a = reinterpret_cast<unsigned long long>(base);
  const i32x4 r = {__builtin_amdgcn_readfirstlane(static_cast<int>(static_cast<unsigned>(a))),
                   __builtin_amdgcn_readfirstlane(static_cast<int>(static_cast<unsigned>(a >> 32) & 0xffffu)),
                   __builtin_amdgcn_readfirstlane(static_cast<int>(bytes)), 0x00020000};
  return r;
}

}  // namespace
}  // namespace bsga
