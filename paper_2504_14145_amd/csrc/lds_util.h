// lds_util.h -- what the simulation kernel and the direct kernel share: accesses
// to the block's dynamic LDS by byte offset, wave masks, and the order blocks
// that they stage through their rings.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "internal.h"

namespace dipsim {
namespace {

extern __shared__ __align__(16) unsigned char s_lds[];

__device__ __forceinline__ uint32_t lds32(uint32_t a) {
  return *reinterpret_cast<const uint32_t *>(s_lds + a);
}
__device__ __forceinline__ uint2 lds64(uint32_t a) {
  return *reinterpret_cast<const uint2 *>(s_lds + a);
}
__device__ __forceinline__ void st32(uint32_t a, uint32_t v) {
  *reinterpret_cast<uint32_t *>(s_lds + a) = v;
}
__device__ __forceinline__ void st16(uint32_t a, uint32_t v) {
  *reinterpret_cast<uint16_t *>(s_lds + a) = uint16_t(v);
}
__device__ __forceinline__ void st64(uint32_t a, uint32_t x, uint32_t y) {
  *reinterpret_cast<uint2 *>(s_lds + a) = make_uint2(x, y);
}
// LDS addresses as the hardware takes them (the dynamic array's own address
// added), for values computed outside the helpers above
typedef __attribute__((address_space(3))) unsigned char lds_byte_t;
__device__ __forceinline__ uint32_t lds_abs(uint32_t a) {
  return a + uint32_t(reinterpret_cast<uintptr_t>((lds_byte_t *)s_lds));
}
__device__ __forceinline__ uint32_t lds16_at(uint32_t abs_addr) {
  return *reinterpret_cast<const __attribute__((address_space(3))) uint16_t *>(uintptr_t(abs_addr));
}
// (x << s) + base in one instruction: written out, because the compiler
// turns (i & m) << s into (i << s) & (m << s) and then needs a separate add
template <int SH>
__device__ __forceinline__ uint32_t shl_add(uint32_t x, uint32_t base) {
  uint32_t d;
  asm("v_lshl_add_u32 %0, %1, %2, %3" : "=v"(d) : "v"(x), "i"(SH), "v"(base));
  return d;
}
__device__ __forceinline__ bool lane_in(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }
__device__ __forceinline__ uint64_t ballot(bool b) { return __builtin_amdgcn_ballot_w64(b); }

// A 16-byte order block of 8 ids (rows are padded to 8 ids, so a block of
// a row never reaches past it).
__device__ __forceinline__ uint4 load_block(const int16_t *row, uint32_t b) {
  return *reinterpret_cast<const uint4 *>(row + int64_t(b) * kSimBlockIds);
}
__device__ __forceinline__ void store_block(uint32_t at, const uint4 &v) {
  st64(at, v.x, v.y);
  st64(at + 8, v.z, v.w);
}

}  // namespace
}  // namespace dipsim
