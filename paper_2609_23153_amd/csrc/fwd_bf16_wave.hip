// Fused block-sparse attention forward, bf16 operands, one wavefront per
// 64-row query tile (the launches with enough tiles to give every SIMD one;
// fwd_bf16.hip serves the others).  The same function as there (paper §2
// Eq. comp-sparse, §4.1): exact softmax attention of the tile over the union
// of the key blocks its query block selected.
//
// Each wave runs alone on its SIMD with the whole register file and a ring in
// LDS of its own, so there is no barrier anywhere, and every K and V fragment
// read from LDS feeds 64 query rows: per 64 x 64 keys and queries 32 KB of
// fragment reads, where the four-wave kernel reads 64.
//  * Keys are walked in half tiles of 32.  K and V half tiles (8 KB each) move
//    L2 -> LDS with buffer_load ... lds into two slots each; a half tile has
//    about three half steps to arrive.
//  * A unit is a half tile for one half of the queries.  The step of unit u
//    runs 16 v_mfma_f32_32x32x16_bf16, 8 of the scores S^T(u + 1) = K Q^T and
//    8 of O^T(u - 1) += V^T P^T, and the softmax of unit u between them, one
//    score after each: none of the three depends on another, so the vector
//    work runs under the matrix work of the same wave.  A fragment is read
//    anew right behind the last product that used it.
//  * A lone wave starts one instruction every 4 cycles, 16 for an MFMA and 8
//    for an exp2 (measured), about 630 cycles a unit, against 512 of the matrix
//    cores.  Hence no instruction without need: addresses are kept in
//    registers, the row sum is 16 plain adds (v_dot2 takes 13 cycles when it
//    follows an MFMA), the reference max is raised lazily.
// Measured at 40 heads x 75,600 tokens, 36 of 1182 blocks of 64 (3.57 TFLOP):
// 3.84 ms, where the four-wave kernel takes 4.15 to 4.4 on the same box; its
// products alone take 2.63 ms (the rate of a large bf16 GEMM on this card, 1.3
// PFLOP/s), its copies alone 2.63 and all but the copies 3.02.
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

template <int I>
struct Int {
  static constexpr int value = I;
};

__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(1, 1))) void
fwd_bf16_wave_kernel(Params p) {
  __shared__ __attribute__((aligned(1024))) uint8_t ring[4 * kHalfBytes];

  const int slot = launch_slot((int)blockIdx.x, (int)gridDim.x);
  const int item = p.order ? p.order[slot] : slot;
  const int bh = item / p.ntiles;
  const int qt = item - bh * p.ntiles;
  const int b = bh / p.H, h = bh - b * p.H;
  const int q0 = qt * kTile;
  const int iblk = q0 / p.block;
  const int hsh = p.block == 64 ? 1 : 2;  // log2(half tiles per block)
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
  int ahead[4];  // the entries of half tiles 0..3
#pragma unroll
  for (int n = 0; n < 4; ++n) ahead[n] = list[min(n >> hsh, p.kmax - 1)];
  const int total = min(max(p.cnt[(int64_t)bh * p.nb + iblk], 0), p.kmax) << hsh;

  // Allowed keys [key_lo, key_hi) of this lane's query of each half; a half
  // tile needs the per-score mask unless it lies inside every row's range:
  // [lo of the tile's last row, hi of its first).
  int key_lo[2], key_hi[2];
#pragma unroll
  for (int qh = 0; qh < 2; ++qh) {
    const int t = min(q0 + 32 * qh + l32, p.N - 1);
    key_lo[qh] = causal_lo(p.cs, t);
    key_hi[qh] = causal_hi(p.cs, t);
  }
  const int tile_lo = causal_lo(p.cs, min(q0 + kTile - 1, p.N - 1));
  const int tile_hi = causal_hi(p.cs, q0);

  const uint32_t kst = (uint32_t)p.ks.n * 2, vst = (uint32_t)p.vs.n * 2;
  const auto kr = make_rsrc(p.k + b * p.ks.b + h * p.ks.h, (uint32_t)(p.N - 1) * kst + 256u);
  const auto vr = make_rsrc(p.v + b * p.vs.b + h * p.vs.h, (uint32_t)(p.N - 1) * vst + 256u);

  // Start of the next valid half tile of the list, N when there is none.
  int pos = -1;
  auto take = [&]() __attribute__((always_inline)) {
    for (++pos; pos < total; ++pos) {
      const int j = list[pos >> hsh];
      if (j < 0 || j >= p.nb) continue;
      const int st = j * p.block + (pos & ((1 << hsh) - 1)) * kHalf;
      if (st < p.N) return st;
    }
    return p.N;
  };
  // starts of the current half tile and the three after it: from the entries
  // read together if they are all valid, else one by one
  int s0, s1, s2, s3;
  {
    int st[4];
    bool valid = total >= 4;
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      st[n] = ahead[n] * p.block + (n & ((1 << hsh) - 1)) * kHalf;
      valid = valid && ahead[n] >= 0 && ahead[n] < p.nb && st[n] < p.N;
    }
    if (valid) {
      s0 = st[0];
      s1 = st[1];
      s2 = st[2];
      s3 = st[3];
      pos = 3;
    } else {
      s0 = take();
      s1 = take();
      s2 = take();
      s3 = take();
    }
  }

  // Copies: instruction i moves rows 4 i .. 4 i + 3 of a half tile, lane l the
  // 16 bytes that the swizzle places in slot l % 16 of row 4 i + l / 16.
  uint32_t kofs[8], vofs[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int row = 4 * i + (lane >> 4);
    kofs[i] = (uint32_t)row * kst + (uint32_t)swz_k(row, lane & 15) * 16u;
    vofs[i] = (uint32_t)row * vst + (uint32_t)swz_v(row, lane & 15) * 16u;
  }
  const uint32_t ring0 = lds_addr(ring);
  auto copy_k = [&](int slot, int i, int st) __attribute__((always_inline)) {
    dma16(ring0 + (uint32_t)(slot * kHalfBytes + i * 1024), kr, kofs[i],
          (uint32_t)__builtin_amdgcn_readfirstlane(st) * kst);
  };
  auto copy_v = [&](int slot, int i, int st) __attribute__((always_inline)) {
    dma16(ring0 + (uint32_t)(kVBase + slot * kHalfBytes + i * 1024), vr, vofs[i],
          (uint32_t)__builtin_amdgcn_readfirstlane(st) * vst);
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
  for (int i = 0; i < 8; ++i) copy_k(1, i, s1);
#pragma unroll
  for (int i = 0; i < 8; ++i) copy_v(0, i, s0);

  f32x16 acc[2][4], s[2];
  bf16x8 kf[8], vf[8];  // vf[2 dt + cs]
  u32x4 pw[2][2];       // P^T of a query half, k-step cs
  float m2[2] = {-INFINITY, -INFINITY}, lsum[2] = {0.f, 0.f};
  const bf16x8 z8 = as_bf16x8((u32x4){0u, 0u, 0u, 0u});
#pragma unroll
  for (int qh = 0; qh < 2; ++qh)
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[qh][dt][r] = 0.f;
#pragma unroll
  for (int f = 0; f < 8; ++f) vf[f] = z8;
  pw[1][0] = pw[1][1] = (u32x4){0u, 0u, 0u, 0u};

  const float c = p.scale_log2;
  // Keys outside the window of a lane's query (or past N): score -inf.
  auto mask = [&](int st, int qh) __attribute__((always_inline)) {
    if (__builtin_expect(st + kHalf > tile_hi || st < tile_lo, 0)) {  // wave-uniform
      const int hi = key_hi[qh] - st - 4 * g, lo = key_lo[qh] - st - 4 * g;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int off = 8 * (r >> 2) + (r & 3);
        if (off >= hi || off < lo) s[qh][r] = -INFINITY;
      }
    }
  };
  // Softmax of a unit, one score per slot: 2^(s c - m2), packed to bf16 in
  // pairs as the B operand of the PV product, summed in fp32.
  float e[16], ts;
  auto soft = [&](int qh, int i) __attribute__((always_inline)) {
    e[i] = __builtin_amdgcn_exp2f(fmaf(s[qh][i], c, -m2[qh]));
    if (i == 1) ts = e[0];
    if (i > 1) ts += e[i - 1];
    if (i > 1 && !(i & 1)) {
      uint32_t x = cvt_pk(e[i - 2], e[i - 1]);
      asm volatile("" : "+v"(x));  // here, not where it is used
      pw[qh][(i - 2) >> 3][((i - 2) >> 1) & 3] = x;
    }
  };
  // The operands of a run of products are written, and the two wait states
  // after vector instructions that wrote them have passed.
  auto ready = [&](int qh) __attribute__((always_inline)) {
    asm volatile("s_nop 1" : "+v"(pw[qh][0]), "+v"(pw[qh][1]));
  };
  // Wait states before other instructions read the accumulators of a product.
  auto settle = [&](int qh) __attribute__((always_inline)) {
    asm volatile("s_nop 15\n\ts_nop 7"
                 : "+a"(acc[qh][0]), "+a"(acc[qh][1]), "+a"(acc[qh][2]), "+a"(acc[qh][3]));
  };
  auto soft_end = [&](int qh) __attribute__((always_inline)) {
    ts += e[15];
    pw[qh][1][3] = cvt_pk(e[14], e[15]);
    // with m2 = -inf every probability is +inf or NaN, so the first half tile
    // always takes the branch
    if (__builtin_expect(__any(!(ts <= kSumCap)), 0)) {  // wave-uniform: raise the reference max
      float mx = s[qh][0];
#pragma unroll
      for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[qh][r]);
      mx *= c;
      const float mnew = fmaxf(m2[qh], pair_max32(mx));
      const float msafe = mnew == -INFINITY ? 0.f : mnew;
      const float alpha = __builtin_amdgcn_exp2f(m2[qh] - msafe);
      lsum[qh] *= alpha;
      settle(qh);
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[qh][dt][r] *= alpha;
      settle(qh);
      m2[qh] = mnew;
      ts = 0.f;
#pragma unroll
      for (int w2 = 0; w2 < 2; ++w2) {
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const float a = __builtin_amdgcn_exp2f(fmaf(s[qh][8 * w2 + 2 * x], c, -msafe));
          const float d = __builtin_amdgcn_exp2f(fmaf(s[qh][8 * w2 + 2 * x + 1], c, -msafe));
          pw[qh][w2][x] = cvt_pk(a, d);
          ts += a + d;
        }
      }
    }
    lsum[qh] += ts;
  };
  const f32x16 zero = {};
  auto score = [&](int qh, int ks) __attribute__((always_inline)) {
    s[qh] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[qh][ks], ks ? s[qh] : zero, 0, 0, 0);
  };
  auto pv = [&](int qh, int i, bool last = false) __attribute__((always_inline)) {
    // The accumulators take the AGPRs, which no other instruction of the loop
    // uses (the scores, which the vector instructions read, take VGPRs): from
    // inline asm, as the compiler gives all products of a kernel one form.
    // Its hazards: ready() covers the operands; an accumulator is used again 4
    // products later, and read otherwise after settle() or the last product.
    const int dt = i & 3, cs = i >> 2;
    if (last)  // the compiler may move the accumulators right behind
      asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0\n\ts_nop 15\n\ts_nop 7"
                   : "+a"(acc[qh][dt])
                   : "v"(vf[2 * dt + cs]), "v"(pw[qh][cs]));
    else
      asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0"
                   : "+a"(acc[qh][dt])
                   : "v"(vf[2 * dt + cs]), "v"(pw[qh][cs]));
  };

  // the list entry after the furthest start, read a half tile ahead
  int raw = list[min(max(pos + 1, 0) >> hsh, p.kmax - 1)];

  // One half tile m from slots P = m % 2: softmax of both its units; the
  // scores of (m, second half) and (m + 1, first half); the PV products of
  // (m - 1, second half) and (m, first half).
  auto pair = [&](auto parity) __attribute__((always_inline)) {
    constexpr int P = decltype(parity)::value;
    mask(s0, 0);
    wait_vm16();  // K(m + 1), V(m)
    ready(1);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      score(1, i);
      kf[i] = read_k(1 - P, i);
      soft(0, 2 * i);
      __builtin_amdgcn_sched_barrier(0);
      pv(1, i);
      vf[2 * (i & 3) + (i >> 2)] = read_v(P, i & 3, i >> 2);
      soft(0, 2 * i + 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    soft_end(0);
    mask(s0, 1);
    ready(0);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (i == 2) wait_lgkm0();  // K(m + 1) and V(m) are in registers: their slots are free
      score(0, i);
      if (i >= 2 && i < 6) copy_k(1 - P, 2 * i - 4, s3);  // K(m + 3)
      if (i >= 6) copy_v(P, 2 * i - 8, s2);               // V(m + 2)
      soft(1, 2 * i);
      __builtin_amdgcn_sched_barrier(0);
      pv(0, i);
      if (i >= 2 && i < 6) copy_k(1 - P, 2 * i - 3, s3);
      if (i >= 4) copy_v(P, i < 6 ? i - 4 : 2 * i - 7, s2);
      soft(1, 2 * i + 1);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 2; i < 4; ++i) copy_v(P, i, s2);
    soft_end(1);
    // advance; the entry read ahead decodes the next start unless it is
    // invalid (then the list is scanned)
    s0 = s1;
    s1 = s2;
    s2 = s3;
    s3 = p.N;
    if (pos + 1 < total) {
      const int j = __builtin_amdgcn_readfirstlane(raw);
      const int st = j * p.block + ((pos + 1) & ((1 << hsh) - 1)) * kHalf;
      if (__builtin_expect(j >= 0 && j < p.nb && st < p.N, 1)) {
        ++pos;
        s3 = st;
      } else {
        ++pos;
        s3 = take();
      }
    }
    raw = list[min((pos + 1) >> hsh, p.kmax - 1)];
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
    for (int i = 0; i < 8; ++i) copy_k(0, i, s2);
#pragma unroll
    for (int i = 0; i < 8; ++i) copy_v(1, i, s1);
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) score(0, ks);
    for (;;) {
      pair(Int<0>{});
      if (s0 >= p.N) break;
      pair(Int<1>{});
      if (s0 >= p.N) break;
    }
    asm volatile("" : "+v"(vf[0]), "+v"(vf[1]), "+v"(vf[2]), "+v"(vf[3]));
    asm volatile("" : "+v"(vf[4]), "+v"(vf[5]), "+v"(vf[6]), "+v"(vf[7]));
    ready(1);
#pragma unroll
    for (int i = 0; i < 8; ++i) pv(1, i, i == 7);
  }
  wait_vm0();  // the copies in flight land before the LDS is given up

  // normalise, store
#pragma unroll
  for (int qh = 0; qh < 2; ++qh) {
    const float l = lsum[qh] + __shfl_xor(lsum[qh], 32, kWave);
    const float inv = l > 0.f ? 1.f / l : 0.f;
    const int row = q0 + 32 * qh + l32;
    if (row < p.N) {
      uint16_t* op = p.o + b * p.os.b + h * p.os.h + (int64_t)row * p.os.n + 4 * g;
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          u32x2 w;
          w[0] = cvt_pk(acc[qh][dt][4 * j] * inv, acc[qh][dt][4 * j + 1] * inv);
          w[1] = cvt_pk(acc[qh][dt][4 * j + 2] * inv, acc[qh][dt][4 * j + 3] * inv);
          *reinterpret_cast<u32x2*>(op + dt * 32 + 8 * j) = w;
        }
      if (p.lse && g == 0)
        p.lse[(int64_t)bh * p.N + row] =
            l > 0.f ? (m2[qh] + __builtin_amdgcn_logf(l)) * 0.69314718055994531f : -INFINITY;
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
