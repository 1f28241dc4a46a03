// Row pieces: the operands of the chunk contractions.
//
// A float32 row x is kept as two float16 planes h and l of the row times a
// power of two, x 2^r = h + l: h = fp16(x 2^r) rounds to nearest, l = fp16 of
// the exact remainder.  Above x's power of two 2^E the remainder is a multiple
// of 2^(E-23) up to 2^(E-11), l a multiple of 2^(E-22) (2^(E-23) in the lower
// half) or of fp16's smallest step 2^-24 if that is more: h + l holds x to
// within max(2^(E-23), 2^-25), and exactly for three of four elements.  r puts
// the row's largest element in [2^14, 2^15), so elements down to 2^-16 of it
// are within 2^-23 of their own power of two, smaller ones within 2^-39 of the
// largest element's.  Rows of unit length take the fixed r = 15.
//
// A row is ceil(dim / 32) blocks of 128 bytes, 32 elements of h and the same
// 32 of l: a 32-deep slice of both planes is one cache line.  (With a plane
// after the other a slice of a row took half of two lines, and the score
// kernel's loads, not its products, set its time.)
//
// A product of two rows takes three plane products, hh + hl + lh, exact in
// float32 up to the order of the sums; the one left out is below 2^-22 of
// |a b| per term (root mean square 2^-24.8).
#pragma once

#include "device_common.h"
#include "row_ops.h"

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 h2_t __attribute__((ext_vector_type(2)));
typedef short v4s __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __amdgpu_buffer_rsrc_t rsrc_t;

// lane `lane` of the result is src, the others old (clang names no builtin for it)
extern "C" __device__ int pbg_writelane(int src, int lane, int old) __asm("llvm.amdgcn.writelane.i32");

namespace pieces {

__device__ __forceinline__ uint32_t writelane(uint32_t src, int lane, uint32_t old) {
  return (uint32_t)pbg_writelane((int)src, lane, (int)old);
}

constexpr uint32_t kOob = 0x80000000u;   // a buffer offset that reads zero

// x = h + l in the low and high half of the result
__device__ __forceinline__ uint32_t split2(float x) {
  __asm__("" : "+v"(x));
  _Float16 h = (_Float16)x;
  const _Float16 l = (_Float16)(x - (float)h);
  return (uint32_t)__builtin_bit_cast(uint16_t, h) | ((uint32_t)__builtin_bit_cast(uint16_t, l) << 16);
}

// two values: packed h pair and packed l pair
// The empty asm statement keeps a and b the rounded float32 values they are:
// a product that ends in them would otherwise be rounded to fp16 in one step
// for h and in two for the remainder, which now and then differ by a unit.
__device__ __forceinline__ void split2_pair(float a, float b, uint32_t& h, uint32_t& l) {
  __asm__("" : "+v"(a), "+v"(b));
  const h2_t hh = {(_Float16)a, (_Float16)b};
  h = __builtin_bit_cast(uint32_t, hh);
  // the exact remainders, h's halves read where they are (the compiler converts
  // each back to float32: eight instructions a pair for four)
  float ra, rb;
  __asm__("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(ra) : "v"(h), "v"(a));
  __asm__("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(rb) : "v"(h), "v"(b));
  const h2_t ll = {(_Float16)ra, (_Float16)rb};
  l = __builtin_bit_cast(uint32_t, ll);
}

// exponent field of a row's largest magnitude, clamped so that the scale
// 2^(141 - e) and its inverse are normal floats (0: a row of zeros)
__device__ __forceinline__ int scale_exponent(float rowmax) {
  const int e = (int)((__float_as_uint(rowmax) >> 23) & 0xFFu);
  return e < 15 ? 15 : e;
}
__device__ __forceinline__ float scale_of(int e) { return __uint_as_float((uint32_t)(268 - e) << 23); }
__device__ __forceinline__ float inverse_scale_of(int e) { return __uint_as_float((uint32_t)(e - 14) << 23); }

// position (16-bit words) of element f of plane 0 in a row; plane 1: + 32
__device__ __forceinline__ int element_at(int f) { return ((f >> 5) << 6) + (f & 31); }

// Writes a row's pieces at p: elements [0, dh), dh = dim rounded up to 8,
// zeros past dim (the rest of the last block is never read).  The row's lanes
// hold elements 64 apart, so neighbouring lanes swap one of every two slots
// and each lane writes a pair of consecutive elements (4 bytes a plane).
template <int RQ>
__device__ __forceinline__ void store_row(const RowT<RQ>& r, float scale, uint16_t* p, int d, int dh, bool cplx,
                                          int lane) {
  uint32_t w[RQ];
#pragma unroll
  for (int q = 0; q < RQ; ++q) w[q] = split2(r.v[q] * scale);
  const int h = d >> 1;
  if (cplx && d + lane < dh) {
    p[element_at(d + lane)] = 0;
    p[element_at(d + lane) + 32] = 0;
  }
  if (cplx && (h & 1)) {   // pairs of the two halves would straddle words
#pragma unroll
    for (int q = 0; q < RQ; ++q) {
      if (!row_valid<RQ>(q, lane, d, true)) continue;
      const int f = element_at(row_index<RQ>(q, lane, d, true));
      p[f] = (uint16_t)w[q];
      p[f + 32] = (uint16_t)(w[q] >> 16);
    }
    return;
  }
  const bool odd = lane & 1;
#pragma unroll
  for (int q = 0; q < RQ; q += 2) {
    // even lanes write the pair of slot q, odd lanes that of slot q + 1
    const uint32_t give = odd ? w[q] : w[q + 1];
    const uint32_t got = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)give, PBG_DPP_QUAD_XOR1, 0xF, 0xF, false);
    const uint32_t lo = odd ? got : w[q], hi = odd ? w[q + 1] : got;
    const int qq = odd ? q + 1 : q, ll = lane & ~1;
    int f;
    bool in;
    if (!cplx) {
      f = ll + 64 * qq;
      in = f < dh;
    } else {
      f = qq < RQ / 2 ? ll + 64 * qq : h + ll + 64 * (qq - RQ / 2);
      in = ll + 64 * (qq % (RQ / 2)) < h;
    }
    if (in) {
      uint16_t* e = p + element_at(f);
      *(uint32_t*)e = (lo & 0xFFFFu) | (hi << 16);
      *(uint32_t*)(e + 32) = (lo >> 16) | (hi & 0xFFFF0000u);
    }
  }
}

template <int RQ>
__device__ __forceinline__ float row_absmax(const RowT<RQ>& r) {
  float m = 0.0f;
#pragma unroll
  for (int q = 0; q < RQ; ++q) m = fmaxf(m, fabsf(r.v[q]));
  m = group16_max(m);
  m = fmaxf(m, __shfl_xor(m, 16, PBG_WAVE));
  return fmaxf(m, __shfl_xor(m, 32, PBG_WAVE));
}

// ---- tiles -------------------------------------------------------------------
// A buffer descriptor must be wave-uniform: the base address is read back
// from the first lane so that it stays scalar.
__device__ __forceinline__ rsrc_t make_rsrc(const void* p) {
  const uint64_t v = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return __builtin_amdgcn_make_buffer_rsrc((void*)(((uint64_t)hi << 32) | lo), (short)0, 0x7FFFFFF0, 0x00020000);
}

typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) v4s lds_v4s;

__device__ __forceinline__ uint32_t lds_offset(const void* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
}

// 16 bytes a lane from global memory to LDS at dst (wave-uniform) + 16 lane
__device__ __forceinline__ void dma16(rsrc_t rs, void* dst, uint32_t off, int soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void*)dst, 16, off, soff, 0, 0);
}

// Tiles with k contiguous: a 32-deep slice of rows, 128 bytes a row (h then
// l), the 16-byte group q of plane p of row x at slot (4 p + q) ^ (x & 7), so
// that fragment reads (16 rows, one group each) spread over all banks.
__device__ __forceinline__ int kc_slot(int x, int plane, int q) { return x * 64 + (((4 * plane + q) ^ (x & 7)) << 3); }

// what lane moves of rows [8 inst, 8 inst + 8): the group (4 p + q) of the
// row, and its byte offset at the first slice (kOob past xdim); ld: 16-bit
// words a row
__device__ __forceinline__ int kc_lane_group(int lane) { return (lane & 7) ^ (lane >> 3); }
__device__ __forceinline__ uint32_t kc_offset(int inst, int ld, int x0, int xdim, int lane) {
  const int x = x0 + 8 * inst + (lane >> 3);
  return x < xdim ? (uint32_t)(((int64_t)x * ld + 8 * kc_lane_group(lane)) * 2) : kOob;
}

// Tiles with k as rows: [32 k][BL blocks of 128 bytes] (32 columns of both
// planes each), in 32-byte pairs of 16-byte groups: pair 4 b + 2 p + h holds
// columns 32 b + 16 h .. + 15 of plane p.  Pair p of row x sits at p ^ f(x),
// f chosen so that the four rows a 16-lane group of a transposing read touches
// fall in distinct banks for both row orders in use.
template <int BL>
__device__ __forceinline__ int kr_f(int x) {
  if (BL == 1) return x & 3;
  return (x & 7) ^ ((x >> 3) & 1 ? 6 : 0);
}

// such a tile is moved 1 KB at a time, 4 BL moves: the row and the 16-bit word
// of the row (from the tile's first block) that lane fetches in move `inst`,
// and its first column
template <int BL>
__device__ __forceinline__ void kr_lane(int inst, int lane, int& row, int& word, int& col) {
  const int slot = inst * 64 + lane;
  row = slot / (8 * BL);
  const int s = slot % (8 * BL);
  const int pair = (s >> 1) ^ kr_f<BL>(row);
  word = 16 * pair + 8 * (s & 1);
  col = 32 * (pair >> 2) + 16 * (pair & 1) + 8 * (s & 1);
}

// Byte address (in the tile) of this lane's part of a transposing read of
// pair 0: the lane addresses row `row`, quad l16 % 4; pair p is at
// address ^ (32 p).
template <int BL>
__device__ __forceinline__ uint32_t kr_address(int row, int l16) {
  return (uint32_t)(row * 128 * BL + kr_f<BL>(row) * 32 + (l16 & 3) * 8);
}
// pair of 16-column block j, plane p
__device__ __forceinline__ constexpr uint32_t kr_pair(int j, int p) { return (uint32_t)(4 * (j >> 1) + 2 * p + (j & 1)); }

// eight k of one column: two transposing reads of four rows each
__device__ __forceinline__ v8h kr_fragment(uint32_t a0, uint32_t a1) {
  const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)(uintptr_t)a0);
  const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s*)(uintptr_t)a1);
  typedef short v8s __attribute__((ext_vector_type(8)));
  return __builtin_bit_cast(v8h, (v8s)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// vmcnt(0): this wave's loads (to LDS included) have landed
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// A workgroup barrier for LDS contents only: global loads, also those to LDS,
// and stores stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

}  // namespace pieces
