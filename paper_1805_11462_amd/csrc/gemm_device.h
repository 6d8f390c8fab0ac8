// Device-side pieces shared by the GEMM kernels (thin.hip, wide.hip, gen.hip): tile numbering, buffer-descriptor and
// LDS-destination loads, operand stores.
#pragma once

#include "common.h"
#include "kernels.h"
#include "split16.h"

namespace onmt {

// XCD-aware tile order: blocks are dealt round-robin to the 8 XCDs, so renumber them so that each
// XCD receives a contiguous range of logical tiles; M varies fastest, so the M tiles that share a
// weight tile run on the same XCD and share its L2.
__device__ inline int xcd_remap(int bid, int nblocks) {
  const int xcd = bid & 7, local = bid >> 3;
  const int full = nblocks >> 3, rem = nblocks & 7;
  return xcd * full + (xcd < rem ? xcd : rem) + local;
}

// Buffer resource descriptor (gfx9 family word 3). Loads through it return zeros past num_records, so a block past
// the last is given an offset beyond every buffer instead of a branch.
constexpr int kBufWord3 = 0x00020000;

__device__ inline __amdgpu_buffer_rsrc_t make_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, kBufWord3);
}

// 16 bytes at a lane's byte offset plus a wave-uniform one, and an offset past the end of a buffer of up to 4 GiB.
constexpr uint32_t kPastEnd = 0xfffffff0u;
__device__ inline uint4 buf_load16s(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, (int)soff, 0));
}

template <class A, class B>
__device__ inline f32x4 mfma_f16(const A& a, const B& b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// LDS address of a byte in a __shared__ array, as the LDS-destination buffer loads take it. (Declared at
// file scope: a local typedef of this pointer type inside a kernel template stops the host stub from
// being emitted.)
typedef __attribute__((address_space(3))) void* lds_ptr_t;
__device__ inline lds_ptr_t lds_at(char* p) { return (lds_ptr_t)p; }

// One 16-byte-per-lane buffer load into LDS (lane l writes 16 bytes at lds + 16 l). (A function of its
// own: called directly under control flow inside a kernel template, the builtin stops the host-side
// launch stub from being emitted.)
__device__ inline void dma16(__amdgpu_buffer_rsrc_t r, char* lds, uint32_t voff, uint32_t soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, lds_at(lds), 16, voff, soff, 0, 0);
}

// Wait before the barrier of a stage: at most n of this wave's vector loads outstanding (its share of the stage has
// landed) and none of its LDS reads. The second half is what allows another wave to refill the buffer this wave read
// last: the compiler may move the products that consume those reads, and with them its own wait, past the barrier.
constexpr int waitcnt_stage(int n) { return (n & 15) | (7 << 4) | (0 << 8) | (((n >> 4) & 3) << 14); }

// Four consecutive columns (k0 a multiple of 4) of row r of a two-term fp16 operand.
__device__ inline void store_act4(uint16_t* dst, int r, int k0, int kblocks, const float (&v)[4]) {
  uint16_t h[4], l[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) split_act(v[j], h[j], l[j]);
  uint16_t* d = dst + split16_at(r, k0, kblocks, 2);
  *(uint2*)d = make_uint2(h[0] | (uint32_t)h[1] << 16, h[2] | (uint32_t)h[3] << 16);
  *(uint2*)(d + kFragElems) = make_uint2(l[0] | (uint32_t)l[1] << 16, l[2] | (uint32_t)l[3] << 16);
}

}  // namespace onmt
