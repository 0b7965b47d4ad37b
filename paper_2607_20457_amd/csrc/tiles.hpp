// K/V tiles in LDS, shared by the attention, decode and packed kernels: how they
// get there and how the matrix operands are read from them.
#pragma once

#include "common.hpp"

namespace {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) uint8_t lds_u8;
typedef __attribute__((address_space(3))) bf16x8 lds_bf16x8;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

constexpr int kBufferFlags = 0x00020000;  // raw 32-bit buffer access (word 3 of the resource)
__device__ constexpr bf16x2 kOnes2 = {(__bf16)1.0f, (__bf16)1.0f};

// One 16-byte-per-lane buffer load that writes LDS directly: lane l's 16
// bytes land at LDS byte lds_base + 16*l.  Issued from asm so that the
// compiler does not order a key loop's LDS reads after it (it cannot tell
// that they read another stage); the loop waits for it explicitly (vmcnt)
// before the stage is read.
__device__ __forceinline__ void lds_dma16(__amdgpu_buffer_rsrc_t rsrc, uint32_t voffset,
                                          uint32_t lds_base) {
  asm volatile("buffer_load_dwordx4 %0, %1, 0 offen lds"
               :
               : "v"(voffset), "s"(rsrc), "{m0}"(lds_base)
               : "memory");
}

// Bits 2 and 3 exchanged: with K row r of a 32-key step holding key
// swap_bits23(r), the scores come out of the matrix unit in the layout that PV
// takes them in.
__device__ __forceinline__ int swap_bits23(int r) {
  return (r & ~12) | ((r >> 1) & 4) | ((r << 1) & 8);
}

// Chunk c of V row r sits at 16-byte chunk position c ^ v_swizzle<D>(r), so that
// a transposing read's rows fall in different banks.
template <int D>
__device__ __forceinline__ int v_swizzle(int r) {
  constexpr int CPR = D / 8;  // chunks per row
  return (4 * ((r * CPR) / 16)) % CPR;
}

// V^T rows e*32 .. of 16 keys as the A operand of PV, from a raw V tile with
// two transposing reads.  Within each 16-lane group such a read hands lane i,
// for slot j, element i%4 of the four that lane 4j + i/4 addressed; so lane
// 16a + 4j + q addresses key row 8(a/2) + j (+4 for the second read) at
// head_dim 16(a%2) + 4q, and lane 16a + i receives head_dim 16(a%2) + i of
// keys 8(a/2) .. +7.  v_tr_base: the lane's byte offset within the tile for
// every e; v_tr_read: from that offset of the first of the 16 keys.
template <int D>
__device__ __forceinline__ void v_tr_base(int lane, uint32_t (&base)[D / 32]) {
  const int a16 = lane >> 4, j = (lane >> 2) & 3, q = lane & 3;
  const int trow = 8 * (a16 >> 1) + j;  // v_swizzle of every row read is that of trow
  const int cb = 2 * (a16 & 1) + (q >> 1);
#pragma unroll
  for (int e = 0; e < D / 32; ++e)
    base[e] = trow * (2 * D) + 16 * ((4 * e + cb) ^ v_swizzle<D>(trow)) + 8 * (q & 1);
}
template <int D>
__device__ __forceinline__ bf16x8 v_tr_read(const lds_u8* b) {
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)b);
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(b + 4 * (2 * D)));
  return __builtin_bit_cast(bf16x8,
                            (s16x8){lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
}

}  // namespace
