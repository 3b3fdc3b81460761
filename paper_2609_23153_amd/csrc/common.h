// Device-side vocabulary shared by the gfx950 kernels of the library.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sa {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(8 * sizeof(int)))) int i32x8;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
typedef __attribute__((__vector_size__(2 * sizeof(uint32_t)))) uint32_t u32x2;

constexpr int kHeadDim = 128;   // d handled by every kernel
constexpr int kWave = 64;       // CDNA wavefront width
constexpr int kTile = 64;       // query rows / keys per fwd tile

// Buffer resource over `bytes` bytes from `base`: loads at offsets past the
// end return zero (the hardware range check), without branches.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes,
                                           0x00020000);
}
__device__ __forceinline__ u32x4 buf_ld16(__amdgpu_buffer_rsrc_t r, uint32_t off,
                                          uint32_t soff = 0) {
  return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, soff, 0));
}

// max of x over the lane pair (l, l ^ 32), through v_permlane32_swap.
__device__ __forceinline__ float pair_max32(float x) {
  const uint32_t u = __float_as_uint(x);
  const auto sw = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
}

// Global -> LDS copy of 16 bytes per lane (buffer_load_dwordx4 ... lds): lane
// l's bytes land at LDS byte address lds_addr + 16*l; rows past the resource
// range land as zeros.  Issued from inline asm so that the compiler does not
// track it: callers wait (vmcnt) and synchronise explicitly.  The compiler's
// own waits stay correct (they can only become more conservative), and the
// memory clobber keeps program order for every memory access around it.
__device__ __forceinline__ void dma16(uint32_t lds_addr, __amdgpu_buffer_rsrc_t r, uint32_t voff,
                                      uint32_t soff) {
  asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               :: "s"(lds_addr), "v"(voff), "s"(r), "s"(soff)
               : "memory", "m0");
}

// LDS byte address of a __shared__ pointer.
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

// Workgroup barrier for pipelined LDS staging: unlike __syncthreads() it has
// no release fence, which would wait for every load in flight (vmcnt(0)),
// including global->LDS copies meant to stay in flight across the barrier.
// The caller waits explicitly for the copies the next step reads; the memory
// clobber keeps the compiler from moving memory accesses across.
__device__ __forceinline__ void barrier_keep_loads() { asm volatile("s_barrier" ::: "memory"); }

// 16-byte global load / store (dwordx4) of raw bits.
__device__ __forceinline__ u32x4 ld16(const void* p) {
  return *reinterpret_cast<const u32x4*>(p);
}
__device__ __forceinline__ void st16(void* p, u32x4 v) { *reinterpret_cast<u32x4*>(p) = v; }

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// fp32 -> bf16 round to nearest even (finite inputs).
__device__ __forceinline__ uint32_t f32_to_bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return u >> 16;
}
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return f32_to_bf16_rne(lo) | (f32_to_bf16_rne(hi) << 16);
}

// OCP e4m3fn codes of the four bf16 values packed in (w0, w1), each times
// inv in fp32 (callers scale so that every product is within 448, up to one
// fp32 rounding): nearest value, ties to even, sign bit kept (-0 and tiny
// negatives give 0x80).  v_cvt_pk_fp8_f32 gives these codes for every fp32
// below 464 in magnitude (all of them compared with the integer rounding of
// the fp32 fields), in 2 instructions where that rounding takes about 60.
__device__ __forceinline__ uint32_t e4m3x4(uint32_t w0, uint32_t w1, float inv) {
  const int o = __builtin_amdgcn_cvt_pk_fp8_f32(bf16_lo(w0) * inv, bf16_hi(w0) * inv, 0, false);
  return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(bf16_lo(w1) * inv, bf16_hi(w1) * inv, o, true);
}

// x summed over the wave, in every lane (DPP rotations within the rows of 16
// lanes, then lane swaps).
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t x) {
#define SA_ROR(n) x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x120 + n, 0xF, 0xF, false)
  SA_ROR(8);
  SA_ROR(4);
  SA_ROR(2);
  SA_ROR(1);
#undef SA_ROR
  const auto p = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  x = p[0] + p[1];
  const auto q = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  return q[0] + q[1];
}

// Whole-wave reductions through DPP-free cross-lane shuffles.
__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) x = fmaxf(x, __shfl_xor(x, o, kWave));
  return x;
}
__device__ __forceinline__ int wave_sum(int x) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o, kWave);
  return x;
}

__device__ __forceinline__ uint64_t lanes_below_mask() {
  const int lane = threadIdx.x & (kWave - 1);
  return lane == 0 ? 0ull : (~0ull >> (kWave - lane));
}

// The softmax states of the even and the odd 32-key half tiles of a query,
// (m, l) and (m_o, l_o), put together: weights of the two accumulators, and the
// log-sum-exp.  Both bf16 forward kernels keep these two states and merge them
// here, each operation written out, so that they give the same bytes.
struct KeyHalves {
  float m, l, c0, c1;
  __device__ __forceinline__ float merge(float a, float a_o) const { return fmaf(a, c0, a_o * c1); }
  __device__ __forceinline__ float lse() const {
    return l > 0.f ? (m + __builtin_amdgcn_logf(l)) * 0.69314718055994531f : -INFINITY;
  }
};
__device__ __forceinline__ KeyHalves merge_key_halves(float m, float l, float m_o, float l_o) {
  KeyHalves k;
  k.m = fmaxf(m, m_o);
  const float ms = k.m == -INFINITY ? 0.f : k.m;
  const float a0 = __builtin_amdgcn_exp2f(m - ms);
  const float a1 = __builtin_amdgcn_exp2f(m_o - ms);
  k.l = fmaf(l, a0, l_o * a1);
  const float inv = k.l > 0.f ? 1.f / k.l : 0.f;
  k.c0 = a0 * inv;
  k.c1 = a1 * inv;
  return k;
}

// Launch slot of workgroup `w` of G.  The launch order gives each XCD
// (workgroup mod 8) runs of 256 consecutive positions of the sorted tiles in
// groups of 2048 slots and leaves the slots of a last partial group in
// position order, which would deal neighbouring tiles to different XCDs, every
// L2 then reading every key tile.  There each XCD takes runs of 32 slots, in
// groups of 256 (bf16 forward, 36 key blocks a tile: 512 tiles 84 -> 49 us,
// 1024 158 -> 102, 6000 619 -> 519).
__device__ __forceinline__ int launch_slot(int w, int G) {
  const int full = G & ~2047, r = w - full;
  if (r < 0 || r >= ((G - full) & ~255)) return w;
  return full + (r & ~255) + 32 * (r & 7) + ((r & 255) >> 3);
}

}  // namespace sa
