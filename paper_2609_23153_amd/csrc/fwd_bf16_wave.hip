// Fused block-sparse attention forward, bf16 operands, one wavefront per
// 64-row query tile (the launches with enough tiles to give every SIMD one;
// fwd_bf16.hip serves the others).  The same function as there (paper §2
// Eq. comp-sparse, §4.1): exact softmax attention of the tile over the union
// of the key blocks its query block selected.  And the same bytes: a tile's
// result must not depend on the launch that it is part of, so this kernel does
// the four waves' arithmetic, each softmax state and accumulator over the same
// keys in the same order, with the states merged by the same function.
//
// Each wave runs alone on its SIMD with the whole register file and a ring in
// LDS of its own, so there is no barrier anywhere, and every K and V fragment
// read from LDS feeds 64 query rows: per 64 x 64 keys and queries 32 KB of
// fragment reads, where the four-wave kernel reads 64.
//  * Key tiles are walked in halves of 32 keys.  The even and the odd halves
//    have a softmax state and an accumulator each, per half of the queries: 4
//    x 64 AGPRs, all 256 there are; the rest lives in 256 VGPRs.  K and V half
//    tiles (8 KB each) move L2 -> LDS with buffer_load ... lds into two slots
//    each; a half tile has about three half steps to arrive.
//  * A unit is a half tile for one half of the queries.  The step of unit u
//    runs 16 v_mfma_f32_32x32x16_bf16, 8 of the scores S^T(u + 1) = K Q^T and
//    8 of O^T(u - 1) += V^T P^T, and the softmax of unit u between them, one
//    score after each: none of the three depends on another, so the vector
//    work runs under the matrix work of the same wave.  A fragment is read
//    anew right behind the last product that used it.
//  * No instruction without need: addresses are kept in registers, the
//    reference max is raised lazily, and the row sum is one v_dot2 per pair of
//    probabilities as they are packed (in the slot of the pack; a slot later
//    it costs 2.5% of the kernel).
// Measured at 40 heads x 75,600 tokens, 36 of 1182 blocks of 64 (3.57 TFLOP):
// 4.00 ms, where the four-wave kernel takes 4.20 to 4.33 on the same box.  Sums
// of the unrounded probabilities instead of the v_dot2 take 3.88, but their
// rounding then no longer cancels against that of the products' operands.
// Bound by what one wave can issue, then by the copies: of its 7.3 M cycles (1.8
// GHz under this load) an instruction is being issued in 66%, the wave waits
// for copies in 17% and for the issue of a ready instruction in 17%; the matrix
// cores work in 47%.
#include "common.h"
#include "launch.h"

namespace sa {
namespace {

constexpr int kRowBytes = kHeadDim * 2;        // 256 B per bf16 row
constexpr int kHalf = 32;                      // keys per half tile
constexpr int kHalfBytes = kHalf * kRowBytes;  // 8 KB per K or V half tile
constexpr uint32_t kVBase = 2 * kHalfBytes;    // ring: K slots 0, 1, V slots 0, 1

// Bound on a lane's sum of 16 probabilities before the reference max is raised.
constexpr float kSumCap = 4096.f;

typedef __attribute__((__vector_size__(4 * sizeof(short)))) short i16x4;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef const __attribute__((address_space(4))) int32_t* list_ptr;

struct Params {
  const uint16_t* q;
  const uint16_t* k;
  const uint16_t* v;
  uint16_t* o;
  float* lse;
  Strides qs, ks, vs, os;
  const int32_t* idx;
  const int32_t* cnt;
  const int32_t* order;
  int kmax, H, N, block, nb, ntiles;  // ntiles = ceil(N / 64) query tiles per head
  float scale_log2;                   // tau * log2(e)
  Shape cs;                           // causal window (causal_chunk 0: none)
};

__device__ __forceinline__ void wait_vm0() {
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(0x0F70);
}
__device__ __forceinline__ void wait_vm16() {
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(0x4F70);
}
__device__ __forceinline__ void wait_lgkm0() {
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(0xC07F);
}

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }
__device__ __forceinline__ uint32_t cvt_pk(float a, float b) {
  const bf16x2 t = {(__bf16)a, (__bf16)b};
  return __builtin_bit_cast(uint32_t, t);
}

// 16-byte-chunk swizzles of the LDS rows, applied on the global side of the
// copies: conflict-free for the K reads (32 rows, one chunk) and for the
// transposed V reads (4 rows x 4 chunks per half-wave).
__device__ __forceinline__ int swz_k(int row, int chunk) { return chunk ^ (row & 15); }
__device__ __forceinline__ int swz_v(int row, int chunk) { return chunk ^ ((row & 3) << 2); }

// This lane's number, where keeping it in a register would not pay.
__device__ __forceinline__ int lane_id() {
  return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}

template <int I>
struct Int {
  static constexpr int value = I;
};

__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(1, 1))) void
fwd_bf16_wave_kernel(Params p) {
  __shared__ __attribute__((aligned(1024))) uint8_t ring[4 * kHalfBytes];
  __shared__ int2 range[2][kWave];  // allowed keys of a lane's query of each half

  const int slot = launch_slot((int)blockIdx.x, (int)gridDim.x);
  const int item = p.order ? p.order[slot] : slot;
  const int bh = item / p.ntiles;
  const int qt = item - bh * p.ntiles;
  const int b = bh / p.H, h = bh - b * p.H;
  const int q0 = qt * kTile;
  const int iblk = q0 / p.block;
  const int sh = p.block == 64 ? 0 : 1;  // log2(64-key tiles per block)
  const int lane = threadIdx.x & (kWave - 1);
  const int g = lane >> 5, l32 = lane & 31;
  // (the loads that the first step waits for are issued together: Q, the list
  // length and the first entries)
  // Q fragments (B operand of K Q^T): row 32 qh + l32, channels 16 ks + 8 g ..
  // +7 (rows past the end repeat the last one; they are not stored)
  bf16x8 qf[2][8];
#pragma unroll
  for (int qh = 0; qh < 2; ++qh) {
    const uint16_t* qp = p.q + b * p.qs.b + h * p.qs.h +
                         (int64_t)min(q0 + 32 * qh + l32, p.N - 1) * p.qs.n + 8 * g;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) qf[qh][ks] = as_bf16x8(ld16(qp + 16 * ks));
  }
  const list_ptr list = (list_ptr)(p.idx + ((int64_t)bh * p.nb + iblk) * p.kmax);
  int ahead[3];  // the entries of tiles 0..2
#pragma unroll
  for (int n = 0; n < 3; ++n) ahead[n] = list[min(n >> sh, p.kmax - 1)];
  const int total = min(max(p.cnt[(int64_t)bh * p.nb + iblk], 0), p.kmax) << sh;

  // Allowed keys [x, y) of this lane's query of each half, in LDS as the few
  // tiles on the edge of a window read them; a half tile needs the per-score
  // mask unless it lies inside every row's range: [lo of the tile's last row,
  // hi of its first).
#pragma unroll
  for (int qh = 0; qh < 2; ++qh) {
    const int t = min(q0 + 32 * qh + l32, p.N - 1);
    range[qh][lane] = make_int2(causal_lo(p.cs, t), causal_hi(p.cs, t));
  }
  const int tile_lo = causal_lo(p.cs, min(q0 + kTile - 1, p.N - 1));
  const int tile_hi = causal_hi(p.cs, q0);

  const uint32_t kst = (uint32_t)p.ks.n * 2, vst = (uint32_t)p.vs.n * 2;
  const auto kr = make_rsrc(p.k + b * p.ks.b + h * p.ks.h, (uint32_t)(p.N - 1) * kst + 256u);
  const auto vr = make_rsrc(p.v + b * p.vs.b + h * p.vs.h, (uint32_t)(p.N - 1) * vst + 256u);

  // Start of the next valid 64-key tile of the list, N when there is none.
  int pos = -1;
  auto take = [&]() __attribute__((always_inline)) {
    for (++pos; pos < total; ++pos) {
      const int j = list[pos >> sh];
      if (j < 0 || j >= p.nb) continue;
      const int st = j * p.block + (pos & ((1 << sh) - 1)) * kTile;
      if (st < p.N) return st;
    }
    return p.N;
  };
  // starts of the current tile and the two after it: from the entries read
  // together if they are all valid, else one by one
  int s0, s1, s2;
  {
    int st[3];
    bool valid = total >= 3;
#pragma unroll
    for (int n = 0; n < 3; ++n) {
      st[n] = ahead[n] * p.block + (n & ((1 << sh) - 1)) * kTile;
      valid = valid && ahead[n] >= 0 && ahead[n] < p.nb && st[n] < p.N;
    }
    if (valid) {
      s0 = st[0];
      s1 = st[1];
      s2 = st[2];
      pos = 2;
    } else {
      s0 = take();
      s1 = take();
      s2 = take();
    }
  }

  // Copies: instruction i moves rows 4 i .. 4 i + 3 of a half tile, lane l the
  // 16 bytes that the swizzle places in slot l % 16 of row 4 i + l / 16 (the
  // swizzles repeat after 16 rows, so instructions i and i + 4 share offsets).
  uint32_t kofs[4], vofs[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = 4 * i + (lane >> 4);
    kofs[i] = (uint32_t)row * kst + (uint32_t)swz_k(row, lane & 15) * 16u;
    vofs[i] = (uint32_t)row * vst + (uint32_t)swz_v(row, lane & 15) * 16u;
  }
  const uint32_t ring0 = lds_addr(ring);
  auto copy_k = [&](int slot, int i, int st) __attribute__((always_inline)) {
    dma16(ring0 + (uint32_t)(slot * kHalfBytes + i * 1024), kr, kofs[i & 3],
          (uint32_t)__builtin_amdgcn_readfirstlane(st + 4 * (i & 4)) * kst);
  };
  auto copy_v = [&](int slot, int i, int st) __attribute__((always_inline)) {
    dma16(ring0 + (uint32_t)(kVBase + slot * kHalfBytes + i * 1024), vr, vofs[i & 3],
          (uint32_t)__builtin_amdgcn_readfirstlane(st + 4 * (i & 4)) * vst);
  };
  // Fragment reads: K row l32, channels 16 ks + 8 g .. +7 (A operand of
  // K Q^T); V^T channel 32 dt + l32 of keys 16 cs + 4 g + {0..3} and + 8 (A
  // operand of V^T P^T, transposed read: lane 16 G + 4 e + q supplies the 8
  // bytes of key 4 (G >> 1) + e, channels 32 dt + 16 (G & 1) + 4 q .. +3).
  uint32_t ka[8], va[4];
  {
    const int G = lane >> 4, e4 = (lane >> 2) & 3, q4 = lane & 3;
    const int vrow = 4 * (G >> 1) + e4;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
      ka[ks] = (uint32_t)(l32 * kRowBytes + swz_k(l32, 2 * ks + g) * 16);
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
      va[dt] = kVBase + (uint32_t)(vrow * kRowBytes +
                                   swz_v(vrow, 4 * dt + 2 * (G & 1) + (q4 >> 1)) * 16 +
                                   (q4 & 1) * 8);
  }
  auto read_k = [&](int slot, int ks) __attribute__((always_inline)) {
    return as_bf16x8(*reinterpret_cast<const u32x4*>(ring + ka[ks] + slot * kHalfBytes));
  };
  auto read_v = [&](int slot, int dt, int cs) __attribute__((always_inline)) {
    u32x4 f;
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      const i16x4 t = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (__attribute__((address_space(3))) i16x4*)(ring + va[dt] + slot * kHalfBytes +
                                                     (16 * cs + 8 * hf) * kRowBytes));
      const u32x2 w = __builtin_bit_cast(u32x2, t);
      f[2 * hf] = w[0];
      f[2 * hf + 1] = w[1];
    }
    return as_bf16x8(f);
  };

  // Prologue: the first copies in the order of the steady state, K(0) before.
#pragma unroll
  for (int i = 0; i < 8; ++i) copy_k(0, i, s0);
#pragma unroll
  for (int i = 0; i < 8; ++i) copy_k(1, i, s0 + kHalf);
#pragma unroll
  for (int i = 0; i < 8; ++i) copy_v(0, i, s0);

  f32x16 acc[2][2][4], s[2];  // acc[kh][qh]: the even / odd half tiles
  bf16x8 kf[8], vf[8];  // vf[2 dt + cs]
  u32x4 pw[2][2];       // P^T of a query half, k-step cs
  float m2[2][2], lsum[2][2];  // [kh][qh]
  const bf16x8 z8 = as_bf16x8((u32x4){0u, 0u, 0u, 0u});
#pragma unroll
  for (int kh = 0; kh < 2; ++kh)
#pragma unroll
    for (int qh = 0; qh < 2; ++qh) {
      m2[kh][qh] = -INFINITY;
      lsum[kh][qh] = 0.f;
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[kh][qh][dt][r] = 0.f;
    }
#pragma unroll
  for (int f = 0; f < 8; ++f) vf[f] = z8;
  pw[1][0] = pw[1][1] = (u32x4){0u, 0u, 0u, 0u};

  const float c = p.scale_log2;
  // Keys outside the window of a lane's query (or past N): score -inf.
  auto mask = [&](int st, int qh) __attribute__((always_inline)) {
    if (__builtin_expect(st + kHalf > tile_hi || st < tile_lo, 0)) {  // wave-uniform
      const int ln = lane_id();
      const int2 allowed = range[qh][ln];
      const int hi = allowed.y - st - 4 * (ln >> 5), lo = allowed.x - st - 4 * (ln >> 5);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int off = 8 * (r >> 2) + (r & 3);
        if (off >= hi || off < lo) s[qh][r] = -INFINITY;
      }
    }
  };
  // Softmax of a unit, one score per slot: 2^(s c - m2), packed to bf16 in
  // pairs as the B operand of the PV product; the sum is taken over those bf16
  // values (v_dot2 against (1, 1)), so numerator and normaliser see the same
  // numbers.  The sum starts in a register that no product reads or writes: a
  // v_dot2c whose accumulator a product in flight reads gives wrong sums.
  const bf16x2 one = {(__bf16)1.f, (__bf16)1.f};
  float e[16], ts;
  auto clear_ts = [&]() __attribute__((always_inline)) {
    asm volatile("v_mov_b32 %0, 0" : "={v255}"(ts));
  };
  auto pack = [&](int qh, int i, float lo, float hi) __attribute__((always_inline)) {
    uint32_t x = cvt_pk(lo, hi);
    asm volatile("" : "+v"(x));  // here, not where it is used
    pw[qh][i >> 3][(i >> 1) & 3] = x;
    ts = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, x), one, ts, false);
  };
  auto soft = [&](int kh, int qh, int i) __attribute__((always_inline)) {
    e[i] = __builtin_amdgcn_exp2f(fmaf(s[qh][i], c, -m2[kh][qh]));
    if (i == 0) clear_ts();
    if (i > 1 && !(i & 1)) pack(qh, i - 2, e[i - 2], e[i - 1]);
  };
  // The operands of a run of products are written, and the two wait states
  // after vector instructions that wrote them have passed.
  auto ready = [&](int qh) __attribute__((always_inline)) {
    asm volatile("s_nop 1" : "+v"(pw[qh][0]), "+v"(pw[qh][1]));
  };
  // Wait states before other instructions read the accumulators of a product.
  auto settle = [&](int kh, int qh) __attribute__((always_inline)) {
    asm volatile("s_nop 15\n\ts_nop 7"
                 : "+a"(acc[kh][qh][0]), "+a"(acc[kh][qh][1]), "+a"(acc[kh][qh][2]),
                   "+a"(acc[kh][qh][3]));
  };
  auto soft_end = [&](int kh, int qh) __attribute__((always_inline)) {
    pack(qh, 14, e[14], e[15]);
    // with m2 = -inf every probability is +inf or NaN, so the first half tile
    // always takes the branch
    if (__builtin_expect(__any(!(ts <= kSumCap)), 0)) {  // wave-uniform: raise the reference max
      float mx = s[qh][0];
#pragma unroll
      for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[qh][r]);
      mx *= c;
      const float mnew = fmaxf(m2[kh][qh], pair_max32(mx));
      const float msafe = mnew == -INFINITY ? 0.f : mnew;
      const float alpha = __builtin_amdgcn_exp2f(m2[kh][qh] - msafe);
      lsum[kh][qh] *= alpha;
      settle(kh, qh);
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) {
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[kh][qh][dt][r] *= alpha;
        asm volatile("s_nop 1" : "+a"(acc[kh][qh][dt]));  // one at a time: registers
      }
      m2[kh][qh] = mnew;
      clear_ts();
#pragma unroll
      for (int x = 0; x < 8; ++x) {
        const float a = __builtin_amdgcn_exp2f(fmaf(s[qh][2 * x], c, -msafe));
        const float d = __builtin_amdgcn_exp2f(fmaf(s[qh][2 * x + 1], c, -msafe));
        pack(qh, 2 * x, a, d);
      }
    }
    lsum[kh][qh] += ts;
  };
  const f32x16 zero = {};
  auto score = [&](int qh, int ks) __attribute__((always_inline)) {
    s[qh] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[qh][ks], ks ? s[qh] : zero, 0, 0, 0);
  };
  auto pv = [&](int kh, int qh, int i, bool last = false) __attribute__((always_inline)) {
    // The accumulators take the AGPRs, which no other instruction of the loop
    // uses (the scores, which the vector instructions read, take VGPRs): from
    // inline asm, as the compiler gives all products of a kernel one form.
    // Its hazards: ready() covers the operands; an accumulator is used again 4
    // products later, and read otherwise after settle() or the last product.
    const int dt = i & 3, cs = i >> 2;
    if (last)  // the compiler may move the accumulators right behind
      asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0\n\ts_nop 15\n\ts_nop 7"
                   : "+a"(acc[kh][qh][dt])
                   : "v"(vf[2 * dt + cs]), "v"(pw[qh][cs]));
    else
      asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0"
                   : "+a"(acc[kh][qh][dt])
                   : "v"(vf[2 * dt + cs]), "v"(pw[qh][cs]));
  };

  // the list entry after the furthest start, read a tile ahead
  int raw = list[min((pos + 1) >> sh, p.kmax - 1)];

  // Half tile P of the tile at s0 (half tile m = 2 n + P of the walk), from
  // slots P: softmax of both its units; the scores of (m, second half) and
  // (m + 1, first half); the PV products of (m - 1, second half) and (m, first
  // half).
  auto half = [&](auto parity) __attribute__((always_inline)) {
    constexpr int P = decltype(parity)::value;
    const int st = s0 + P * kHalf;
    const int k3 = P ? s2 : s1 + kHalf, v2 = P ? s1 + kHalf : s1;  // half tiles m + 3, m + 2
    mask(st, 0);
    wait_vm16();  // K(m + 1), V(m)
    ready(1);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      score(1, i);
      kf[i] = read_k(1 - P, i);
      soft(P, 0, 2 * i);
      __builtin_amdgcn_sched_barrier(0);
      pv(1 - P, 1, i);
      vf[2 * (i & 3) + (i >> 2)] = read_v(P, i & 3, i >> 2);
      soft(P, 0, 2 * i + 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    soft_end(P, 0);
    mask(st, 1);
    ready(0);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (i == 2) wait_lgkm0();  // K(m + 1) and V(m) are in registers: their slots are free
      score(0, i);
      if (i >= 2 && i < 6) copy_k(1 - P, 2 * i - 4, k3);  // K(m + 3)
      if (i >= 6) copy_v(P, 2 * i - 8, v2);               // V(m + 2)
      soft(P, 1, 2 * i);
      __builtin_amdgcn_sched_barrier(0);
      pv(P, 0, i);
      if (i >= 2 && i < 6) copy_k(1 - P, 2 * i - 3, k3);
      if (i >= 4) copy_v(P, i < 6 ? i - 4 : 2 * i - 7, v2);
      soft(P, 1, 2 * i + 1);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 2; i < 4; ++i) copy_v(P, i, v2);
    soft_end(P, 1);
  };
  // On to the next tile; the entry read ahead decodes the furthest start
  // unless it is invalid (then the list is scanned).
  auto advance = [&]() __attribute__((always_inline)) {
    s0 = s1;
    s1 = s2;
    s2 = p.N;
    if (pos + 1 < total) {
      const int j = __builtin_amdgcn_readfirstlane(raw);
      const int st = j * p.block + ((pos + 1) & ((1 << sh) - 1)) * kTile;
      ++pos;
      if (__builtin_expect(j >= 0 && j < p.nb && st < p.N, 1))
        s2 = st;
      else
        s2 = take();
    }
    raw = list[min((pos + 1) >> sh, p.kmax - 1)];
  };

  // Q has arrived before the loop (a wait inside it would drain the copies);
  // so have the first 24 copies, which are older
#pragma unroll
  for (int qh = 0; qh < 2; ++qh)
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) asm volatile("" : "+v"(qf[qh][ks]));
  if (s0 < p.N) {
    wait_vm16();
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) kf[ks] = read_k(0, ks);
    wait_lgkm0();
#pragma unroll
    for (int i = 0; i < 8; ++i) copy_k(0, i, s1);
#pragma unroll
    for (int i = 0; i < 8; ++i) copy_v(1, i, s0 + kHalf);
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) score(0, ks);
    do {
      half(Int<0>{});
      half(Int<1>{});
      advance();
    } while (s0 < p.N);
    asm volatile("" : "+v"(vf[0]), "+v"(vf[1]), "+v"(vf[2]), "+v"(vf[3]));
    asm volatile("" : "+v"(vf[4]), "+v"(vf[5]), "+v"(vf[6]), "+v"(vf[7]));
    ready(1);
#pragma unroll
    for (int i = 0; i < 8; ++i) pv(1, 1, i, i == 7);
  }
  wait_vm0();  // the copies in flight land before the LDS is given up

  // merge the two key halves, normalise, store
#pragma unroll
  for (int qh = 0; qh < 2; ++qh) {
    const float l0 = lsum[0][qh] + __shfl_xor(lsum[0][qh], 32, kWave);
    const float l1 = lsum[1][qh] + __shfl_xor(lsum[1][qh], 32, kWave);
    const KeyHalves w = merge_key_halves(m2[0][qh], l0, m2[1][qh], l1);
    const int ln = lane_id();
    const int row = q0 + 32 * qh + (ln & 31);
    if (row < p.N) {
      uint16_t* op = p.o + b * p.os.b + h * p.os.h + (int64_t)row * p.os.n + 4 * (ln >> 5);
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) {
        asm volatile("" : "+a"(acc[0][qh][dt]), "+a"(acc[1][qh][dt]));  // one at a time
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float x[4];
#pragma unroll
          for (int r = 0; r < 4; ++r)
            x[r] = w.merge(acc[0][qh][dt][4 * j + r], acc[1][qh][dt][4 * j + r]);
          u32x2 o;
          o[0] = pack_bf16x2(x[0], x[1]);
          o[1] = pack_bf16x2(x[2], x[3]);
          *reinterpret_cast<u32x2*>(op + dt * 32 + 8 * j) = o;
        }
      }
      if (p.lse && ln < 32) p.lse[(int64_t)bh * p.N + row] = w.lse();
    }
  }
}

}  // namespace

hipError_t launch_fwd_bf16_wave(const Shape& s, const FwdArgs& a, hipStream_t stream) {
  Params p;
  p.q = static_cast<const uint16_t*>(a.q);
  p.k = static_cast<const uint16_t*>(a.k);
  p.v = static_cast<const uint16_t*>(a.v);
  p.o = static_cast<uint16_t*>(a.o);
  p.lse = a.lse;
  p.qs = a.qs;
  p.ks = a.ks;
  p.vs = a.vs;
  p.os = a.os;
  p.idx = a.idx;
  p.cnt = a.cnt;
  p.order = a.order;
  p.kmax = a.kmax;
  p.H = s.H;
  p.N = s.N;
  p.block = s.block;
  p.nb = s.nb;
  p.ntiles = (s.N + kTile - 1) / kTile;
  p.scale_log2 = a.softmax_scale * 1.4426950408889634f;
  p.cs = s;
  fwd_bf16_wave_kernel<<<s.B * s.H * p.ntiles, kWave, 0, stream>>>(p);
  return hipGetLastError();
}

}  // namespace sa
