// Device helpers shared by the register-weight MFMA kernels (laud_head.hip, laud_tail.hip): LDS-direct loads,
// explicit counter waits, the transposed 32x32x16 bf16 MFMA tile and its lane-swap epilogue.
#pragma once

#include "laud_common.h"

namespace laud {

typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// LDS-direct load of 16 bytes per lane: lane l's chunk lands at LDS byte address lds_base + 16*l.
__device__ __forceinline__ void dma16(__amdgpu_buffer_rsrc_t rsrc, unsigned voff, unsigned soff, unsigned lds_base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               :
               : "s"(lds_base), "v"(voff), "s"(rsrc), "s"(soff)
               : "memory");
}
// ... of 4 bytes per lane
__device__ __forceinline__ void dma4(__amdgpu_buffer_rsrc_t rsrc, unsigned voff, unsigned soff, unsigned lds_base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, %3 offen lds"
               :
               : "s"(lds_base), "v"(voff), "s"(rsrc), "s"(soff)
               : "memory");
}
template <int N>
__device__ __forceinline__ void vm_wait() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void wg_barrier() { asm volatile("s_barrier" ::: "memory"); }
__device__ __forceinline__ void lds_wait() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// Requests one 128-byte line per thread of the weights a launch streams, so that they are on their way into this XCD's
// L2 before the tiles ask for them slice by slice: workgroups go round-robin over the eight XCDs, so
// workgroup b takes piece b/8 (kThreads lines) of the range.  In a model every block brings weights of its own, which no
// earlier launch has left in the L2.  Returns the value loaded, for l2_touched() to consume behind the first wait that drains
// the loads anyway (so that the request is not dropped and nobody waits for it alone).
__device__ __forceinline__ unsigned l2_touch(const void* base, int bytes, int threads) {
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
  const unsigned line = (blockIdx.x >> 3) * (unsigned)threads + threadIdx.x;
  return __builtin_amdgcn_raw_buffer_load_b32(rs, min(line, 0x1000000u) * 128u, 0, 0);  // (past the end: no request, zero)
}
__device__ __forceinline__ void l2_touched(unsigned r) { asm volatile("" ::"v"(r)); }

__device__ __forceinline__ f32x16 mma_bf16(const u32x4& first, const uint4& second, f32x16 acc) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, first), __builtin_bit_cast(bf16x8, second),
                                                 acc, 0, 0, 0);
}
__device__ __forceinline__ unsigned pack_bf16(float lo, float hi) {
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
}

// The activation after the residual add as one maximum, fmaxf(v, act_floor(relu)): of a number and a quiet NaN the maximum is
// the number, so without a ReLU every sum, NaN included, stays what it is.  (With one a NaN becomes 0, as in every kernel.)
__device__ __forceinline__ float act_floor(bool relu) { return relu ? 0.f : __builtin_nanf(""); }

// Accumulator e of a lane belongs to channel 8*(e/4) + 4*(lane/32) + e%4 of the wave's 32.  After these eight
// swaps v[] holds, in the order 0-3, 8-11, 4-7, 12-15, the sixteen consecutive channels 16*(lane/32) .. +15.
__device__ __forceinline__ void to_consecutive_channels(float (&v)[16]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[i]), __float_as_uint(v[8 + i]), false, false);
    v[i] = __uint_as_float(r[0]);
    v[8 + i] = __uint_as_float(r[1]);
    auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[4 + i]), __float_as_uint(v[12 + i]), false, false);
    v[4 + i] = __uint_as_float(q[0]);
    v[12 + i] = __uint_as_float(q[1]);
  }
}

// A wave's 32 x 32 block of results on its way to memory: the accumulators of a lane are 4 x 4 consecutive channels of one row, and
// stored from there an instruction touches 32 rows with 16 bytes a lane, 32 bytes apart.  Through 4 KB of LDS of the wave's own (LDS
// operations of a wave stay in order: no barrier, no wait) a lane gets eight consecutive channels, four lanes 64 bytes of a row, and
// residuals are read the same way: k_tail on 12544 / 18816 / 25088 pixels (128 images of 14 x 14 at 0.5, 0.75, 1) 35.6 / 47.8 / 65.0 ->
// 33.2 / 45.0 / 61.8 us.  16-byte unit u of row r lies at position u ^ ((r >> 1) & 7) of the row's eight: four cycles of bank
// conflicts an instruction on average (SQ_LDS_BANK_CONFLICT), 11 % of k_tail's LDS cycles.
constexpr int kTurnBytes = 4096;
// where a lane's channels 8 g + 4 * (lane / 32) .. +3 of row lane % 32 go
__device__ __forceinline__ unsigned turn_put(int lane, int g) {
  const unsigned r = lane & 31;
  return r * 128u + (((2u * g + (unsigned)(lane >> 5)) ^ (r >> 1 & 7u)) << 4);
}
// ... and where its channels 8 * (lane % 4) + 4 * e .. +3 of row 16 * q + lane / 4 come from
__device__ __forceinline__ unsigned turn_get(int lane, int q, int e) {
  const unsigned r = 16u * q + (unsigned)(lane >> 2);
  return r * 128u + (((2u * (lane & 3u) + e) ^ (r >> 1 & 7u)) << 4);
}

// The same for a 32 x 32 block of bf16 results in 64-byte rows (2 KB): where a lane's channels 8 * g + 4 * (lane / 32) .. +3 of row
// lane % 32 go, and where channels 8 * (lane % 4) .. +7 of row 16 * q + lane / 4 come from.  16-byte unit u of row r lies at
// position u ^ ((r >> 1) & 3): lanes that are served together cover 128 bytes.
// (Written as u32x2 and read as u32x4: the compiler takes vector types of its own to overlap with anything, and two different structs
// not to.)
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned row_put(int lane, int g) {
  const unsigned r = lane & 31;
  return r * 64u + (((unsigned)g ^ (r >> 1 & 3u)) << 4) + (unsigned)(lane >> 5) * 8u;
}
__device__ __forceinline__ unsigned row_get(int lane, int q) {
  const unsigned r = 16u * q + (unsigned)(lane >> 2);
  return r * 64u + ((((unsigned)lane & 3u) ^ (r >> 1 & 3u)) << 4);
}

}  // namespace laud
