// Work scheduling for the fused forward: orders the 64-row query tiles of all
// (batch, head) slices for the hardware dispatcher.
//
// The dispatcher hands workgroups out in blockIdx order as CU slots free up,
// i.e. it is a greedy list scheduler.  Two properties of the order matter:
//  * ragged cost (query blocks keep different numbers of key blocks): tiles
//    are sorted by a cost class, most expensive first (longest-processing-
//    time-first), so short tiles fill the tail of the launch;
//  * locality: within a class, tiles stay in raster order, and blockIdx is
//    remapped so that each XCD (blockIdx % 8 on MI355X) receives runs of
//    consecutive tiles, whose key-block lists overlap and share that XCD's L2.
// The cost classes are floor(log2(key tiles)), so the sort is a 16-bucket
// stable partition (a counting sort) over chunks of 1024 tiles.  Up to
// kOneChunks chunks it is one launch: every workgroup counts the classes of
// all tiles itself, work that grows with the square of the tiles.  Up to
// kTwoChunks, two: class counts per chunk, and a scatter that writes every
// tile straight into its launch slot, whose workgroups sum the counts
// themselves.  Beyond, a scan of the counts (classes descending, chunks
// ascending) between the two.  One / two / three launches, us, lists of equal
// length (which one launch need not count) and of uneven ones: 128 tiles 2.2 and
// 5.2 / 6.4 / 12.4; 8192 3.2 and 8.5 / 9.8 / 16.0; 12,288 3.5 and 10.2 / 9.8 /
// 16.0; 47,280 4.9 and 20.8 / 10.5 / 16.4 (blocks of 128: 31.8 / 11.7 / 17.4);
// 188,416 10.6 and 62.9 / 11.4 / 18.0; 500,736 - / 15 / 23.
#include <mutex>

#include "common.h"
#include "launch.h"

namespace sa {
namespace {

constexpr int kClasses = 16;
constexpr int kXcds = 8;
constexpr int kRun = 256;          // consecutive list positions handed to one XCD
constexpr int kChunk = 1024;       // tiles per counting / scatter workgroup
constexpr int kSortThreads = 256;  // 4 waves x 4 rounds of 64 tiles
constexpr int kScanThreads = 1024;

__device__ __forceinline__ int cost_class(int tiles) {
  // 0 for empty tiles; otherwise 1 + floor(log2(tiles)), capped.  Larger = costlier.
  if (tiles <= 0) return 0;
  const int c = 32 - __clz(tiles);
  return c < kClasses ? c : kClasses - 1;
}

struct SchedArgs {
  const int32_t* cnt;
  int kmax, nb, ntiles, block, G, chunks;
};

__device__ __forceinline__ int class_of(const SchedArgs& a, int item) {
  int64_t row = item;  // block 64: tiles and query blocks are the same
  if (a.block != kTile) {
    const int bh = item / a.ntiles, qt = item - bh * a.ntiles;
    row = (int64_t)bh * a.nb + (qt * kTile) / a.block;
  }
  const int c = a.cnt[row];
  return cost_class(min(max(c, 0), a.kmax) * (a.block / kTile));
}

// Launch slot that takes sorted position `pos` (of G): the inverse of the
// interleave that gives XCD x (slot % 8) runs of kRun consecutive positions;
// the positions of the last partial group keep their own slot.
__device__ __forceinline__ int pos_to_slot(int pos, int G) {
  const int group = kXcds * kRun;
  const int full = (G / group) * group;
  if (pos >= full) return pos;
  const int g = pos / group, rem = pos - g * group;
  const int x = rem / kRun, rr = rem - x * kRun;
  return (g * kRun + rr) * kXcds + x;
}

// counts[chunk][c] = tiles of class c in the chunk.
__global__ __launch_bounds__(kSortThreads) void sched_count_kernel(SchedArgs a,
                                                                   int32_t* __restrict__ counts) {
  __shared__ int wave_cnt[kSortThreads / kWave][kClasses];
  const int t = threadIdx.x, lane = t & (kWave - 1), wave = t / kWave;
  int mine = 0;  // lane c of each wave keeps the wave's count of class c
#pragma unroll
  for (int m = 0; m < kChunk / kSortThreads; ++m) {
    const int it = blockIdx.x * kChunk + m * kSortThreads + t;
    const int cls = it < a.G ? class_of(a, it) : -1;
#pragma unroll
    for (int c = 0; c < kClasses; ++c) {
      const int n = __popcll(__ballot(cls == c));
      if (lane == c) mine += n;
    }
  }
  if (lane < kClasses) wave_cnt[wave][lane] = mine;
  __syncthreads();
  if (t < kClasses) {
    int tot = 0;
#pragma unroll
    for (int w = 0; w < kSortThreads / kWave; ++w) tot += wave_cnt[w][t];
    counts[(int64_t)blockIdx.x * kClasses + t] = tot;
  }
}

// In place: counts[chunk][c] becomes the number of class-c tiles in earlier
// chunks; counts[chunks][c] receives the first sorted position of class c
// (classes in descending order).  One workgroup.
__global__ __launch_bounds__(kScanThreads) void sched_scan_kernel(int chunks,
                                                                  int32_t* __restrict__ counts) {
  __shared__ int wsum[kScanThreads / kWave][kClasses];
  __shared__ int carry[kClasses];
  const int t = threadIdx.x, lane = t & (kWave - 1), wave = t / kWave;
  if (t < kClasses) carry[t] = 0;
  __syncthreads();
  for (int ch0 = 0; ch0 < chunks; ch0 += kScanThreads) {
    const int ch = ch0 + t;
    int v[kClasses], incl[kClasses];
#pragma unroll
    for (int c = 0; c < kClasses; ++c) {
      v[c] = ch < chunks ? counts[(int64_t)ch * kClasses + c] : 0;
      incl[c] = v[c];
    }
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1)
#pragma unroll
      for (int c = 0; c < kClasses; ++c) {
        const int y = __shfl_up(incl[c], o, kWave);
        if (lane >= o) incl[c] += y;
      }
    if (lane == kWave - 1)
#pragma unroll
      for (int c = 0; c < kClasses; ++c) wsum[wave][c] = incl[c];
    __syncthreads();
    if (ch < chunks) {
#pragma unroll
      for (int c = 0; c < kClasses; ++c) {
        int before = carry[c];
        for (int w = 0; w < wave; ++w) before += wsum[w][c];
        counts[(int64_t)ch * kClasses + c] = before + incl[c] - v[c];
      }
    }
    __syncthreads();
    if (t < kClasses) {
      int tot = 0;
      for (int w = 0; w < kScanThreads / kWave; ++w) tot += wsum[w][t];
      carry[t] += tot;
    }
    __syncthreads();
  }
  if (t == 0) {
    int acc = 0;
    for (int c = kClasses - 1; c >= 0; --c) {  // costliest class first
      counts[(int64_t)chunks * kClasses + c] = acc;
      acc += carry[c];
    }
  }
}

// In lane c of a row of 16: the sum of x over the classes above c.
__device__ __forceinline__ int above_sum(int x) {
  int above = x;
#define SA_SHL(n) above += __builtin_amdgcn_update_dpp(0, above, 0x100 + n, 0xF, 0xF, true)
  SA_SHL(1);
  SA_SHL(2);
  SA_SHL(4);
  SA_SHL(8);
#undef SA_SHL
  return above - x;
}

// Each tile's sorted position = class start + class-c tiles in earlier chunks
// + class-c tiles before it in this chunk; written to order[slot(position)].
// SCANNED: counts as sched_scan_kernel leaves them; otherwise as
// sched_count_kernel does, and every workgroup sums them itself.
template <bool SCANNED>
__global__ __launch_bounds__(kSortThreads) void sched_scatter_kernel(
    SchedArgs a, const int32_t* __restrict__ counts, int32_t* __restrict__ order) {
  __shared__ int run[kClasses];
  __shared__ int wave_cnt[kSortThreads / kWave][kClasses];
  const int t = threadIdx.x, lane = t & (kWave - 1), wave = t / kWave;
  if (SCANNED) {
    if (t < kClasses)
      run[t] = counts[(int64_t)a.chunks * kClasses + t] +
               counts[(int64_t)blockIdx.x * kClasses + t];
  } else {
    constexpr int kParts = kSortThreads / kClasses;
    __shared__ int part[2][kParts][kClasses];
    const int c = t & (kClasses - 1), p = t / kClasses;
    int early = 0, all = 0;
#pragma unroll 4
    for (int ch = p; ch < a.chunks; ch += kParts) {
      const int n = counts[ch * kClasses + c];
      all += n;
      early += ch < (int)blockIdx.x ? n : 0;
    }
    part[0][p][c] = early;
    part[1][p][c] = all;
    __syncthreads();
    if (t < kClasses) {
      early = all = 0;
#pragma unroll
      for (int q = 0; q < kParts; ++q) {
        early += part[0][q][t];
        all += part[1][q][t];
      }
      run[t] = above_sum(all) + early;
    }
  }
  const uint64_t below = lanes_below_mask();
  for (int m = 0; m < kChunk / kSortThreads; ++m) {
    // tiles of round m in index order: wave w holds the w-th 64 of them
    const int it = blockIdx.x * kChunk + m * kSortThreads + t;
    const int cls = it < a.G ? class_of(a, it) : -1;
    int rank = 0;
#pragma unroll
    for (int c = 0; c < kClasses; ++c) {
      const uint64_t msk = __ballot(cls == c);
      if (cls == c) rank = __popcll(msk & below);
      if (lane == c) wave_cnt[wave][c] = __popcll(msk);
    }
    __syncthreads();
    if (cls >= 0) {
      int pos = run[cls] + rank;
      for (int w = 0; w < wave; ++w) pos += wave_cnt[w][cls];
      order[pos_to_slot(pos, a.G)] = it;
    }
    __syncthreads();
    if (t < kClasses) {
      int tot = 0;
#pragma unroll
      for (int w = 0; w < kSortThreads / kWave; ++w) tot += wave_cnt[w][t];
      run[t] += tot;
    }
    __syncthreads();
  }
}

// The whole sort in one launch, one workgroup per chunk.  When every list has
// the same length (row selection without a window) the sorted order is the
// raster order, which a pass over the lengths shows.  Otherwise a thread
// counts the classes of tiles t, t + 1024, ... in 8-bit counters (four per
// word; at most kOneChunks tiles each, so they do not overflow), those of the
// earlier chunks apart; the workgroup's sums of these give the first position
// of every class for this chunk, ballots the rank within it.  Bound by the
// latency of the loads and of the launch.
constexpr int kOneThreads = kChunk;
constexpr int kOneWaves = kOneThreads / kWave;
constexpr int kOneChunks = 8;
constexpr int kTwoChunks = 512;

__global__ __launch_bounds__(kOneThreads) void sched_one_kernel(SchedArgs a,
                                                                int32_t* __restrict__ order) {
  __shared__ uint32_t wsum[kOneWaves][2][8];  // per wave: earlier / later, two classes per word
  __shared__ int base[kOneWaves][kClasses];   // counts, then first positions, per wave and class
  const int t = threadIdx.x, lane = t & (kWave - 1), wave = t / kWave;
  const int mine = blockIdx.x, own = mine * kChunk + t;

  const int rows = a.G / a.ntiles * a.nb;  // query blocks of all heads
  const int len0 = a.cnt[0];
  int differ = 0;
#pragma unroll 8
  for (int r = t; r < rows; r += kOneThreads) differ |= a.cnt[r] ^ len0;
  if (!__syncthreads_or(differ)) {
    if (own < a.G) order[pos_to_slot(own, a.G)] = own;
    return;
  }

  uint32_t sum[2][4] = {};
  auto count = [&](int m, uint32_t (&w)[4]) {
    const int it = m * kChunk + t;
    const int c = it < a.G ? class_of(a, it) : -1;
    const uint32_t one = c >= 0 ? 1u << (8 * (c & 3)) : 0u;
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] += (c >> 2) == i ? one : 0u;
  };
#pragma unroll 8
  for (int m = 0; m < mine; ++m) count(m, sum[0]);
#pragma unroll 8
  for (int m = mine; m < a.chunks; ++m) count(m, sum[1]);
  // wave sums in 16-bit counters: word 2 i + p holds classes 4 i + p, 4 i + p + 2
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const uint32_t x = wave_sum_u32((sum[s][i] >> (8 * p)) & 0x00ff00ffu);
        if (lane == 0) wsum[wave][s][2 * i + p] = x;
      }
  const uint64_t below = lanes_below_mask();
  const int cls = own < a.G ? class_of(a, own) : -1;
  int rank = 0;
#pragma unroll
  for (int c = 0; c < kClasses; ++c) {
    const uint64_t msk = __ballot(cls == c);
    if (cls == c) rank = __popcll(msk & below);
    if (lane == c) base[wave][c] = __popcll(msk);
  }
  __syncthreads();
  if (t < kClasses) {  // lane c: class c
    const int word = 2 * (t >> 2) + (t & 1), sh = t & 2 ? 16 : 0;
    int early = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kOneWaves; ++w) {
      early += (int)(wsum[w][0][word] >> sh & 0xffffu);
      all += (int)(wsum[w][1][word] >> sh & 0xffffu);
    }
    all += early;
    int pos = above_sum(all) + early;
#pragma unroll
    for (int w = 0; w < kOneWaves; ++w) {
      const int n = base[w][t];
      base[w][t] = pos;
      pos += n;
    }
  }
  __syncthreads();
  if (cls >= 0) order[pos_to_slot(base[wave][cls] + rank, a.G)] = own;
}

}  // namespace

int64_t num_query_tiles(const Shape& s) {
  return (int64_t)s.B * s.H * ((s.N + kTile - 1) / kTile);
}

size_t schedule_workspace_bytes(const Shape& s) {
  const int64_t chunks = (num_query_tiles(s) + kChunk - 1) / kChunk;
  return (size_t)(chunks + 1) * kClasses * sizeof(int32_t);
}

// ---- allocation-free variant ----------------------------------------------
// The class counters live in one file-scope device array per GPU instead of a
// caller workspace.  In host code `scratch` names a host-side stand-in, not
// device memory: the device address of each GPU's copy is looked up once per
// device (hipGetSymbolAddress with that device current) and only that address
// is handed to the kernels.
namespace {
constexpr int kScratchInts = kStaticScheduleScratchBytes / (int)sizeof(int32_t);
static __device__ __align__(256) int32_t scratch[kScratchInts];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
int32_t* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t static_schedule_scratch(int32_t** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = static_cast<int32_t*>(p);
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

hipError_t launch_schedule(const Shape& s, const int32_t* cnt, int kmax, int32_t* order,
                           void* ws, hipStream_t stream) {
  SchedArgs a;
  a.cnt = cnt;
  a.kmax = kmax;
  a.nb = s.nb;
  a.ntiles = (s.N + kTile - 1) / kTile;
  a.block = s.block;
  a.G = (int)num_query_tiles(s);
  a.chunks = (a.G + kChunk - 1) / kChunk;
  if (a.chunks <= kOneChunks) {
    sched_one_kernel<<<a.chunks, kOneThreads, 0, stream>>>(a, order);
    return hipGetLastError();
  }
  int32_t* counts = static_cast<int32_t*>(ws);
  sched_count_kernel<<<a.chunks, kSortThreads, 0, stream>>>(a, counts);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (a.chunks <= kTwoChunks) {
    sched_scatter_kernel<false><<<a.chunks, kSortThreads, 0, stream>>>(a, counts, order);
    return hipGetLastError();
  }
  sched_scan_kernel<<<1, kScanThreads, 0, stream>>>(a.chunks, counts);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  sched_scatter_kernel<true><<<a.chunks, kSortThreads, 0, stream>>>(a, counts, order);
  return hipGetLastError();
}

}  // namespace sa
