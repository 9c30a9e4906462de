// kata_quad.hpp -- device helpers of the quadratic-form bf16 kernels: staged
// row tiles, their fragment reads and copies.
#pragma once

#include "kata_common.hpp"

namespace kata {

typedef __attribute__((address_space(3))) void qd_lds_void_t;

// One 16-byte global -> LDS copy per lane, lane l landing at lds_wave_base +
// 16 l (wave-uniform base), counted by vmcnt.  In inline assembly because the
// compiler's wait-count pass would otherwise drain every copy in flight before
// each LDS read; the kernel waits with wait_vmcnt and issues no other vector
// memory operation inside its stage loop.
__device__ __forceinline__ void qd_copy16(const void* gsrc, void* lds_wave_base) {
  const uint32_t lds =
      static_cast<uint32_t>(reinterpret_cast<uintptr_t>((qd_lds_void_t*)lds_wave_base));
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
               :
               : "v"(gsrc), "s"(lds)
               : "memory", "m0");
}

__device__ __forceinline__ f32x16 qd_mfma(const bf16x8& a, const bf16x8& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// Transposing LDS read (ds_read_b64_tr_b16): lane j of a 16-lane group receives
// in slot s element j % 4 of the 8-byte piece that lane 4 s + j / 4 addresses.
typedef short qd_i16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint2 qd_tr16(const char* p) {
  const qd_i16x4 r = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) qd_i16x4*)(const_cast<char*>(p)));
  return __builtin_bit_cast(uint2, r);
}

// A staged row is 128 bytes; its 16-byte chunk c lies at chunk c ^ qd_swz(row).
// Bits 1..3 of the row, reversed: the eight even (odd) rows of a 16-row
// fragment read fall on distinct chunks, and so do rows r and r + 2 of the four
// rows that a transposing read takes from 64 bytes each (bit 2 differs).
__device__ __forceinline__ int qd_swz(int r) {
  return ((r >> 1) & 1) * 4 + ((r >> 2) & 1) * 2 + ((r >> 3) & 1);
}

// Per-lane LDS offsets, formed once.  row[kz]: 16 bytes of row lane % 32 at
// K-step kz.  col[m][x]: the transposing read whose 16-lane group G addresses
// rows 4 h + j / 4 (+ 8 when x) and the piece of columns
// 32 m + 16 (G % 2) + 4 (j % 4), so that the lane receives column
// 32 m + lane % 32 of rows 4 h + 0..3 (+ 8): an A operand in the row order
// 0-3, 8-11 | 4-7, 12-15 of the score accumulators.
struct QdOffsets {
  unsigned row[4], col[2][2];
  __device__ __forceinline__ explicit QdOffsets(int lane) {
    const int c = lane & 31, h = lane >> 5, jl = lane & 15;
#pragma unroll
    for (int kz = 0; kz < 4; ++kz)
      row[kz] = static_cast<unsigned>(c * 128 + 16 * ((2 * kz + h) ^ qd_swz(c)));
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        const int r = 4 * h + (jl >> 2) + 8 * x;
        const int ch = 4 * m + 2 * ((lane >> 4) & 1) + ((jl & 3) >> 1);
        col[m][x] = static_cast<unsigned>(r * 128 + 16 * (ch ^ qd_swz(r)) + 8 * (jl & 1));
      }
  }
  __device__ __forceinline__ bf16x8 rows(const char* tile, int kz) const {
    return *reinterpret_cast<const bf16x8*>(tile + row[kz]);
  }
  __device__ __forceinline__ bf16x8 cols(const char* tile, int m) const {
    const uint2 lo = qd_tr16(tile + col[m][0]), hi = qd_tr16(tile + col[m][1]);
    return __builtin_bit_cast(bf16x8, make_uint4(lo.x, lo.y, hi.x, hi.y));
  }
};

// Copies 32 rows of 128 bytes, rows past T - 1 re-reading row T - 1 (their
// pairs are masked), eight rows per wave of four.
__device__ __forceinline__ void qd_stage(const uint16_t* rows, int r0, int T, char* tile, int wave,
                                         int lane) {
  const int r = 8 * wave + (lane >> 3);
  const int t = min(r0 + r, T - 1);
  qd_copy16(rows + static_cast<long long>(t) * 64 + 8 * ((lane & 7) ^ qd_swz(r)),
            tile + 8 * wave * 128);
}

__device__ __forceinline__ f32x16 qd_zero() {
  f32x16 z;
#pragma unroll
  for (int r = 0; r < 16; ++r) z[r] = 0.f;
  return z;
}

__device__ __forceinline__ bf16x8 qd_frag(const uint32_t* w) {
  return __builtin_bit_cast(bf16x8, make_uint4(w[0], w[1], w[2], w[3]));
}

// fp32 rows of 64 from the transposed accumulators: lane c's row, columns
// 32 m + 8 r4 + 4 h + 0..3.
__device__ __forceinline__ void qd_store(float* row, const f32x16 (&acc)[2], int h, float scale) {
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4)
      *reinterpret_cast<float4*>(row + 32 * m + 8 * r4 + 4 * h) =
          make_float4(scale * acc[m][4 * r4], scale * acc[m][4 * r4 + 1],
                      scale * acc[m][4 * r4 + 2], scale * acc[m][4 * r4 + 3]);
}

// The same for 32 rows of 64 bytes (d = 32): chunk c of a row at c ^ ((r / 4) % 4),
// so that the four rows of a 16-row fragment read that share a 64-byte bank
// group fall on distinct chunks.  Waves 0 and 1 copy 16 rows each.
__device__ __forceinline__ int qd_swz32(int r) { return (r >> 2) & 3; }
__device__ __forceinline__ void qd_stage32(const uint16_t* rows, int r0, int T, char* tile,
                                           int part, int lane) {
  const int r = 16 * part + (lane >> 2);
  const int t = min(r0 + r, T - 1);
  qd_copy16(rows + static_cast<long long>(t) * 32 + 8 * ((lane & 3) ^ qd_swz32(r)),
            tile + 16 * part * 64);
}

}  // namespace kata
