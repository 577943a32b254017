// Device kernels of the gsmat library (CDNA4 / gfx950, wave64).
//
// All per-row work uses the same tiling: a workgroup of kBlock threads owns a
// tile of kTile consecutive items and thread t touches items t, t+kBlock, ...,
// so every global access of a tile is coalesced.  Kernels that feed a prefix
// sum also write one partial sum per tile; the offsets are then produced by a
// small single-workgroup scan over the tile sums and an add pass.  Ordered
// (stable) compaction ranks the kept items of a tile with wave ballots and
// mbcnt, so output order equals input order.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "common.hpp"
#include "device.hpp"

namespace gsmat {

namespace {

using namespace dev;

// ---------------------------------------------------------------- prefix sums
__global__ __launch_bounds__(kBlock) void k_scan_tile_sums(int64_t* ts, int64_t nt,
                                                           int64_t* total, int64_t* host_total,
                                                           uint32_t* word, uint32_t report) {
  int64_t carry = 0;
  for (int64_t c0 = 0; c0 < nt; c0 += kTile) {
    int64_t v[kItems];
    int64_t loc = 0;
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
      const int64_t i = c0 + (int64_t)threadIdx.x * kItems + j;
      v[j] = i < nt ? ts[i] : 0;
      loc += v[j];
    }
    int64_t tot;
    int64_t ex = block_excl_scan(loc, &tot) + carry;
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
      const int64_t i = c0 + (int64_t)threadIdx.x * kItems + j;
      if (i < nt) ts[i] = ex;
      ex += v[j];
    }
    carry += tot;
  }
  if (threadIdx.x == 0) {
    total[0] = carry;
    if (host_total) host_total[0] = carry;  // host memory, read after the report
  }
  report_one(word, report);
}

// Two tile-sum arrays (neither null) scanned in one pass (device.hpp).
__global__ __launch_bounds__(kScanBlock) void k_scan_tile_sums2(int64_t* ts, int64_t* ts2,
                                                                int64_t nt) {
  scan_tile_sums2_block(ts, ts2, nt);
}

template <class Tin, class Tout>
__global__ __launch_bounds__(kBlock) void k_scan_add(const Tin* __restrict__ x, int64_t n,
                                                     const int64_t* __restrict__ tile_off,
                                                     Tout* __restrict__ out, int write_total) {
  const int64_t tot = scan_add_tile<Tin, Tout>(blockIdx.x, x, n, tile_off[blockIdx.x], out);
  if (write_total && threadIdx.x == 0 && blockIdx.x == gridDim.x - 1)
    out[n] = (Tout)(tile_off[blockIdx.x] + tot);
}

// The same with the tile sums not yet scanned, for at most kBlock * kItems
// tiles: every workgroup adds up the sums before its own (a read of the sums
// each, from the cache), and the last one reports the total.  A launch less
// before the host knows the total, and one less in all.
__global__ __launch_bounds__(kBlock) void k_scan_rows(const int32_t* __restrict__ x, int64_t n,
                                                      const int64_t* __restrict__ ts,
                                                      int64_t* __restrict__ out, int64_t* total,
                                                      uint32_t* word, uint32_t report) {
  const int b = (int)blockIdx.x;
  int64_t before = 0;
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const int i = j * kBlock + threadIdx.x;
    if (i < b) before += ts[i];
  }
  const int64_t base = block_sum(before);
  const bool last = blockIdx.x == gridDim.x - 1;
  if (last) {
    if (threadIdx.x == 0) total[0] = base + ts[b];
    report_one(word, report);  // the host goes on while the offsets are written
  }
  const int64_t tot = scan_add_tile<int32_t, int64_t>(b, x, n, base, out);
  if (threadIdx.x == 0 && last) out[n] = base + tot;
}

__global__ __launch_bounds__(kBlock) void k_tile_reduce_u32(const uint32_t* __restrict__ x,
                                                            int64_t n, int64_t* ts) {
  const int64_t tile0 = (int64_t)blockIdx.x * kTile;
  int64_t loc = 0;
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const int64_t i = tile0 + (int64_t)j * kBlock + threadIdx.x;
    if (i < n) loc += x[i];
  }
  const int64_t t = block_sum(loc);
  if (threadIdx.x == 0) ts[blockIdx.x] = t;
}

// ---------------------------------------------------------------- radix sort
// LSD radix sort of 64-bit keys, RB-bit digits.  A pass reads every key twice
// (digit counts, then ranks) and writes it once.  What bounded it was the
// write: ranks were exchanged through three barriers for every 256 keys and
// each key went to its place on its own (1.6 TB/s).  A tile is now 4096 keys,
// ranked by each wave on its own for 1024 keys in a row (no barrier), turned
// into digit order in LDS and written as one run per digit: of 20 million
// keys 203 -> 80 us a pass (4.0 TB/s), the counts 56 -> 38 us.
constexpr int kRsItems = 16;
constexpr int kRsTile = kBlock * kRsItems;  // keys
constexpr int kRsWave = 64 * kRsItems;      // keys of a wave, consecutive

// A key (p, a, b) as (p, b, a): vb bits each for a and b.
__device__ inline uint64_t swap_ends(uint64_t k, int vb) {
  const uint64_t m = (1ull << vb) - 1;
  return (k >> (2 * vb) << (2 * vb)) | ((k & m) << vb) | ((k >> vb) & m);
}

// Digit counts of every tile: hist[digit * nb + tile].  kSwap: of the keys
// with their ends swapped (as k_rs_scatter).
template <int RB, bool kSwap>
__global__ __launch_bounds__(kBlock) void k_rs_hist(const uint64_t* __restrict__ keys, int64_t n,
                                                    int shift, int vb,
                                                    uint32_t* __restrict__ hist, int64_t nb) {
  constexpr int D = 1 << RB;
  __shared__ uint32_t h[kWaves][D];
  for (int i = threadIdx.x; i < kWaves * D; i += kBlock) (&h[0][0])[i] = 0;
  __syncthreads();
  const int64_t i0 = (int64_t)blockIdx.x * kRsTile + wave_id() * kRsWave + lane_id();
  uint64_t k[kRsItems];
#pragma unroll
  for (int j = 0; j < kRsItems; ++j) k[j] = i0 + j * 64 < n ? keys[i0 + j * 64] : 0;
#pragma unroll
  for (int j = 0; j < kRsItems; ++j) {
    const bool valid = i0 + j * 64 < n;
    if (kSwap) k[j] = swap_ends(k[j], vb);
    const uint32_t d = (uint32_t)(k[j] >> shift) & (D - 1);
    // the high digits of sorted keys are alike in a wave: one add for all
    const uint64_t live = __ballot(valid);
    const uint32_t d0 = __builtin_amdgcn_readfirstlane(d);
    if (__ballot(valid && d == d0) == live) {
      if (lane_id() == 0 && live) atomicAdd(&h[wave_id()][d0], (uint32_t)__popcll(live));
    } else if (valid) {
      atomicAdd(&h[wave_id()][d], 1u);
    }
  }
  __syncthreads();
  for (int d = threadIdx.x; d < D; d += kBlock) {
    uint32_t c = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) c += h[w][d];
    hist[(int64_t)d * nb + blockIdx.x] = c;
  }
}

template <int RB, bool kSwap>
__global__ __launch_bounds__(kBlock) void k_rs_scatter(const uint64_t* __restrict__ in,
                                                       uint64_t* __restrict__ out, int64_t n,
                                                       int shift, int vb,
                                                       const uint32_t* __restrict__ offs,
                                                       int64_t nb) {
  constexpr int D = 1 << RB;
  constexpr int DT = D / kBlock;  // digits per thread
  static_assert(D % kBlock == 0, "every thread takes the same number of digits");
  __shared__ uint64_t s[kRsTile];
  __shared__ uint32_t cnt[kWaves][D];  // keys of the wave so far; then its first place in s
  __shared__ uint32_t gb[D];           // first place of the digit's run, less its place in s
  for (int i = threadIdx.x; i < kWaves * D; i += kBlock) (&cnt[0][0])[i] = 0;
  __syncthreads();
  const int64_t tile0 = (int64_t)blockIdx.x * kRsTile;
  const int w = wave_id();
  const int64_t i0 = tile0 + w * kRsWave + lane_id();
  const uint64_t lt = __lanemask_lt();
  uint64_t k[kRsItems];
  uint32_t rank[kRsItems];
#pragma unroll
  for (int j = 0; j < kRsItems; ++j) k[j] = i0 + j * 64 < n ? in[i0 + j * 64] : 0;
#pragma unroll
  for (int j = 0; j < kRsItems; ++j) {
    const bool valid = i0 + j * 64 < n;
    if (kSwap) k[j] = swap_ends(k[j], vb);
    const uint32_t d = (uint32_t)(k[j] >> shift) & (D - 1);
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < RB; ++b) {
      const bool bit = (d >> b) & 1u;
      const uint64_t m = __ballot(bit);
      peers &= bit ? m : ~m;
    }
    const uint32_t before = (uint32_t)__popcll(peers & lt);
    // the wave's keys of the digit before this round; one lane per digit adds
    // this round's (the counts are the wave's own: its order is enough)
    const uint32_t base = cnt[w][d];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (valid && before == 0) cnt[w][d] = base + (uint32_t)__popcll(peers);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    rank[j] = base + before;
  }
  __syncthreads();
  // thread t's digits t * DT ...: their places in the tile, wave by wave
  {
    uint32_t c[kWaves][DT];
    int64_t sum = 0;
#pragma unroll
    for (int q = 0; q < DT; ++q)
#pragma unroll
      for (int x = 0; x < kWaves; ++x) {
        c[x][q] = cnt[x][threadIdx.x * DT + q];
        sum += c[x][q];
      }
    int64_t tot;
    uint32_t at = (uint32_t)block_excl_scan(sum, &tot);
#pragma unroll
    for (int q = 0; q < DT; ++q) {
      const int d = threadIdx.x * DT + q;
      gb[d] = offs[(int64_t)d * nb + blockIdx.x] - at;
#pragma unroll
      for (int x = 0; x < kWaves; ++x) {
        cnt[x][d] = at;
        at += c[x][q];
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kRsItems; ++j)
    if (i0 + j * 64 < n) s[cnt[w][(uint32_t)(k[j] >> shift) & (D - 1)] + rank[j]] = k[j];
  __syncthreads();
  const int m = (int)min((int64_t)kRsTile, n - tile0);
#pragma unroll
  for (int j = 0; j < kRsItems; ++j) {
    const int i = j * kBlock + threadIdx.x;
    if (i < m) {
      const uint64_t x = s[i];
      out[(uint32_t)(gb[(uint32_t)(x >> shift) & (D - 1)] + (uint32_t)i)] = x;
    }
  }
}

// ---------------------------------------------------------------- index build
// The first triple of the workgroup's with an id out of range.  Bound by the 12
// bytes a triple it reads: 20 million triples 80 us, where the host's threads
// need 1.6 ms to read them again.
__global__ __launch_bounds__(kBlock) void k_check_ids(const int32_t* __restrict__ s,
                                                      const int32_t* __restrict__ p,
                                                      const int32_t* __restrict__ o, int64_t n,
                                                      uint32_t V, uint32_t P,
                                                      int64_t* __restrict__ out) {
  constexpr int U = 4;
  __shared__ int64_t wmin[kBlock / 64];
  int64_t first = n;
  const int64_t stride = (int64_t)gridDim.x * kBlock * U;
  for (int64_t i0 = (int64_t)blockIdx.x * kBlock * U + threadIdx.x; i0 < n; i0 += stride) {
    uint32_t a[U], b[U], c[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = min(i0 + (int64_t)u * kBlock, n - 1);
      a[u] = (uint32_t)s[i];
      b[u] = (uint32_t)p[i];
      c[u] = (uint32_t)o[i];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (a[u] >= V || b[u] >= P || c[u] >= V)
        first = min(first, min(i0 + (int64_t)u * kBlock, n - 1));
  }
  for (int d = 32; d > 0; d >>= 1) first = min(first, (int64_t)__shfl_xor((long long)first, d));
  if (lane_id() == 0) wmin[wave_id()] = first;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kBlock / 64; ++w) first = min(first, wmin[w]);
    out[blockIdx.x] = first;
  }
}

__global__ void k_pack_keys(const int32_t* __restrict__ s, const int32_t* __restrict__ p,
                            const int32_t* __restrict__ o, int64_t n, int vb,
                            uint64_t* __restrict__ k) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    k[i] = (uint64_t)(uint32_t)p[i] << (2 * vb) | (uint64_t)(uint32_t)s[i] << vb | (uint32_t)o[i];
}

__global__ __launch_bounds__(kBlock) void k_flag_adjacent(const uint64_t* __restrict__ k,
                                                          int64_t n,
                                                          uint8_t* __restrict__ flags,
                                                          int64_t* __restrict__ ts) {
  const int64_t tile0 = (int64_t)blockIdx.x * kTile;
  int64_t loc = 0;
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const int64_t i = tile0 + (int64_t)j * kBlock + threadIdx.x;
    if (i < n) {
      const uint8_t f = (i == 0 || k[i] != k[i - 1]) ? 1 : 0;
      flags[i] = f;
      loc += f;
    }
  }
  const int64_t t = block_sum(loc);
  if (threadIdx.x == 0) ts[blockIdx.x] = t;
}

__global__ __launch_bounds__(kBlock) void k_compact_u64(const uint64_t* __restrict__ in,
                                                        const uint8_t* __restrict__ flags,
                                                        int64_t n,
                                                        const int64_t* __restrict__ tile_off,
                                                        uint64_t* __restrict__ out) {
  compact_tile(
      blockIdx.x, n, tile_off[blockIdx.x], [&](int64_t i) { return flags[i] != 0; },
      [&](int64_t i, int64_t pos) { out[pos] = in[i]; });
}

// Rows of one orientation from its sorted distinct keys (p, row, member), in
// two passes over them.  The first counts every tile's row heads and notes
// each predicate's first entry; the second writes the member lists and, with
// the heads' places, the row ids and offsets and each predicate's first row.
// Each key is read twice and nothing else is kept per key or per row (before:
// a flag per key, a position per row, five passes).  20 million keys: 216 ->
// 126 us an orientation.
__global__ __launch_bounds__(kBlock) void k_row_count(const uint64_t* __restrict__ k, int64_t n,
                                                      int vb, int64_t* __restrict__ pfe,
                                                      int64_t* __restrict__ ts) {
  const int64_t tile0 = (int64_t)blockIdx.x * kTile;
  uint64_t x[kItems], y[kItems];
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const int64_t i = tile0 + (int64_t)j * kBlock + threadIdx.x;
    x[j] = i < n ? k[i] : 0;
    y[j] = i > 0 && i < n ? k[i - 1] : ~0ull;
  }
  int64_t loc = 0;
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const int64_t i = tile0 + (int64_t)j * kBlock + threadIdx.x;
    if (i >= n) continue;
    if (i == 0 || x[j] >> vb != y[j] >> vb) ++loc;
    if (i == 0 || x[j] >> (2 * vb) != y[j] >> (2 * vb)) pfe[x[j] >> (2 * vb)] = i;
  }
  const int64_t t = block_sum(loc);
  if (threadIdx.x == 0) ts[blockIdx.x] = t;
}

// Thread t takes the tile's keys 8t .. 8t + 7, so one scan of the heads'
// counts places them and the members leave in 16-byte stores.
__global__ __launch_bounds__(kBlock) void k_row_fill(const uint64_t* __restrict__ k, int64_t n,
                                                     int vb, const int64_t* __restrict__ pfe,
                                                     const int64_t* __restrict__ ts,
                                                     int32_t* __restrict__ nbr,
                                                     int32_t* __restrict__ src,
                                                     int32_t* __restrict__ keys,
                                                     int32_t* __restrict__ ptr,
                                                     int64_t* __restrict__ pfr) {
  static_assert(kItems == 8, "two 16-byte stores per thread");
  const uint64_t vmask = (1ull << vb) - 1;
  const int64_t i0 = (int64_t)blockIdx.x * kTile + (int64_t)threadIdx.x * kItems;
  uint64_t x[kItems];
  uint64_t prev = ~0ull;
  const bool full = i0 + kItems <= n;
  if (full) {
#pragma unroll
    for (int j = 0; j < kItems; j += 2) {
      const ulonglong2 v = *reinterpret_cast<const ulonglong2*>(k + i0 + j);
      x[j] = v.x;
      x[j + 1] = v.y;
    }
  } else {
#pragma unroll
    for (int j = 0; j < kItems; ++j) x[j] = i0 + j < n ? k[i0 + j] : 0;
  }
  if (i0 > 0 && i0 < n) prev = k[i0 - 1];
  uint32_t head = 0, phead = 0;
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const uint64_t b = j ? x[j ? j - 1 : 0] : prev;
    const bool first = i0 + j == 0;
    if (i0 + j < n && (first || x[j] >> vb != b >> vb)) head |= 1u << j;
    if (i0 + j < n && (first || x[j] >> (2 * vb) != b >> (2 * vb))) phead |= 1u << j;
  }
  int64_t tot;
  int64_t r = ts[blockIdx.x] + block_excl_scan(__popc(head), &tot);
  if (full) {
    const int4 a = make_int4((int)(x[0] & vmask), (int)(x[1] & vmask), (int)(x[2] & vmask),
                             (int)(x[3] & vmask));
    const int4 b = make_int4((int)(x[4] & vmask), (int)(x[5] & vmask), (int)(x[6] & vmask),
                             (int)(x[7] & vmask));
    *reinterpret_cast<int4*>(nbr + i0) = a;
    *reinterpret_cast<int4*>(nbr + i0 + 4) = b;
    if (src) {
      const int4 c = make_int4((int)(x[0] >> vb & vmask), (int)(x[1] >> vb & vmask),
                               (int)(x[2] >> vb & vmask), (int)(x[3] >> vb & vmask));
      const int4 d = make_int4((int)(x[4] >> vb & vmask), (int)(x[5] >> vb & vmask),
                               (int)(x[6] >> vb & vmask), (int)(x[7] >> vb & vmask));
      *reinterpret_cast<int4*>(src + i0) = c;
      *reinterpret_cast<int4*>(src + i0 + 4) = d;
    }
  } else {
#pragma unroll
    for (int j = 0; j < kItems; ++j)
      if (i0 + j < n) {
        nbr[i0 + j] = (int32_t)(x[j] & vmask);
        if (src) src[i0 + j] = (int32_t)(x[j] >> vb & vmask);
      }
  }
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    if (!(head >> j & 1)) continue;
    const int64_t p = (int64_t)(x[j] >> (2 * vb));
    keys[r] = (int32_t)(x[j] >> vb & vmask);
    ptr[r + p] = (int32_t)(i0 + j - pfe[p]);
    if (phead >> j & 1) pfr[p] = r;
    ++r;
  }
}

__global__ void k_fill_i64(int64_t* p, int64_t n, int64_t v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

// Dense row pointers of every predicate that has them, one launch: tile b of
// the launch is kDenseTile vertices of the predicate that owns it (first[p] its
// first tile).  dense[v] is the offset of the first row >= v.  The tile's rows
// are found by one search and marked in a bit mask in LDS; a vertex's row is the
// number of marks before it, so a pointer costs no search of its own.  The
// offsets come from LDS too, where the lanes of a wave read few different
// words: from memory a gather takes a clock per lane (8192 vertices a tile: 0.33
// ms).  89 predicates of 2 million vertices: a mark per vertex and a scan over
// them 0.32 ms, this 0.26 ms (2.7 TB/s written).
__global__ __launch_bounds__(kBlock) void k_dense_ptrs(const PredDesc* __restrict__ desc,
                                                       const int64_t* __restrict__ first, int32_t P,
                                                       const int32_t* __restrict__ keys,
                                                       const int32_t* __restrict__ ptr, int64_t V,
                                                       int32_t* __restrict__ dense) {
  constexpr int kWords = kDenseTile / 64, kPerWave = kWords / (kBlock / 64);
  static_assert(kWords == 64, "a word a lane");
  __shared__ unsigned long long mark[kWords];
  __shared__ int32_t off[kDenseTile + 1];  // offsets of the tile's rows
  __shared__ int32_t lim[2];
  const int64_t b = blockIdx.x;
  const int lo = find_tile_wave(first, P, b);
  const PredDesc d = desc[lo];
  const int64_t v0 = (b - first[lo]) * kDenseTile;
  const int nv = (int)min((int64_t)kDenseTile, V + 1 - v0);
  const int32_t* const pk = keys + d.row_base;
  const int32_t* const pp = ptr + d.ptr_base;
  if (wave_id() < 2) {
    const int64_t v = v0 + wave_id() * (int64_t)nv;
    const int32_t r = wave_lower_bound(pk, (int32_t)d.nr, (int32_t)min(v, (int64_t)INT32_MAX));
    if (lane_id() == 0) lim[wave_id()] = r;
  }
  if (threadIdx.x < kWords) mark[threadIdx.x] = 0;
  __syncthreads();
  const int r0 = lim[0], nr = lim[1] - r0;  // ids in [v0, v0 + nv): at most nv rows
  for (int i = threadIdx.x; i <= nr; i += kBlock) {
    off[i] = pp[r0 + i];
    if (i == nr) break;
    const int x = (int)(pk[r0 + i] - v0);
    atomicOr(&mark[x >> 6], 1ull << (x & 63));
  }
  __syncthreads();
  // rows before each word (every wave for itself)
  const int c = (int)__popcll(mark[lane_id()]);
  const int before = (int)wave_incl_scan(c) - c;
  const int wave = __builtin_amdgcn_readfirstlane(wave_id());
  int32_t* const o = dense + d.dense_base + v0;
#pragma unroll 8
  for (int j = 0; j < kPerWave; ++j) {
    const int w = wave * kPerWave + j;
    const unsigned long long m = mark[w];
    const int at = __builtin_amdgcn_readlane(before, w);
    const int r = (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                                 __builtin_amdgcn_mbcnt_lo((unsigned)m, at));
    const int i = w * 64 + lane_id();
    if (i < nv) o[i] = off[r];
  }
}

// Bucket directories of the other predicates, one launch (tiles as above, of
// kTile buckets): dir[b] is the first row with id >= b << shift, searched among
// the rows of the tile.
__global__ __launch_bounds__(kBlock) void k_row_dirs(const PredDesc* __restrict__ desc,
                                                     const int64_t* __restrict__ first, int32_t P,
                                                     const int32_t* __restrict__ keys, int64_t V,
                                                     int32_t* __restrict__ dir) {
  __shared__ int32_t lim[2];
  const int64_t b = blockIdx.x;
  const int lo = find_tile_wave(first, P, b);
  const PredDesc d = desc[lo];
  const int64_t b0 = (b - first[lo]) * kTile;
  const int64_t nb = ((V - 1) >> d.dir_shift) + 2;  // entries
  const int n = (int)min((int64_t)kTile, nb - b0);
  const int32_t* const pk = keys + d.row_base;
  if (wave_id() < 2) {
    const int64_t v = (b0 + wave_id() * (int64_t)n) << d.dir_shift;
    const int32_t r = v >= (int64_t)INT32_MAX ? (int32_t)d.nr
                                              : wave_lower_bound(pk, (int32_t)d.nr, (int32_t)v);
    if (lane_id() == 0) lim[wave_id()] = r;
  }
  __syncthreads();
  int32_t v[kItems], at[kItems], len[kItems];
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const int i = j * kBlock + threadIdx.x;
    const int64_t x = (b0 + i) << d.dir_shift;
    const bool ok = i < n;
    at[j] = lim[0];
    len[j] = ok ? lim[1] - lim[0] : 0;
    if (ok && x >= (int64_t)INT32_MAX) {
      at[j] = (int32_t)d.nr;
      len[j] = 0;
    }
    v[j] = (int32_t)min(x, (int64_t)INT32_MAX);
  }
  lower_bound_n<kItems>(pk, v, at, len);
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const int i = j * kBlock + threadIdx.x;
    if (i < n) dir[d.dir_base + b0 + i] = at[j];
  }
}

__global__ void k_long_rows(PredView pv, int32_t min_len, int32_t* __restrict__ out,
                            int32_t* __restrict__ count, int32_t cap) {
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < pv.nr;
       r += (int64_t)gridDim.x * blockDim.x) {
    const int32_t len = pv.ptr[r + 1] - pv.ptr[r];
    if (len >= min_len) {
      const int32_t i = atomicAdd(count, 1);
      if (i < cap) {
        out[2 * i] = pv.keys[r];
        out[2 * i + 1] = len;
      }
    }
  }
}

__global__ void k_row_bitmap(PredView pv, int32_t v, uint32_t* __restrict__ bm) {
  int32_t st, len;
  row_lookup(pv, v, st, len);
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < len;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int32_t u = pv.nbr[st + i];
    atomicOr(&bm[u >> 5], 1u << (u & 31));
  }
}

__global__ void k_ptr_sentinels(const PredDesc* __restrict__ d, int32_t P, int32_t* __restrict__ ptr) {
  const int32_t p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p < P) ptr[d[p].ptr_base + d[p].nr] = (int32_t)d[p].nnz;
}

__global__ void k_lookup(LookupBatch b, const PredDesc* dout, const PredDesc* din, OriPtrs out,
                         OriPtrs in, LookupRes* res, uint32_t* word, uint32_t report) {
  const int i = (int)threadIdx.x;  // one wave
  if (i < b.n) res[i] = lookup_one(b.req[i], dout, din, out, in);
  report_wave(word, report);
}

// ---------------------------------------------------------------- join steps
__global__ __launch_bounds__(kBlock) void k_count_expand(const int32_t* __restrict__ col,
                                                         int64_t n, PredView pv,
                                                         int32_t* __restrict__ N,
                                                         int32_t* __restrict__ start,
                                                         int64_t* __restrict__ ts) {
  const int64_t t = count_expand_tile(blockIdx.x, col, n, pv, N, start);
  if (threadIdx.x == 0) ts[blockIdx.x] = t;
}

__global__ __launch_bounds__(kBlock) void k_flag_filter(ProbeArgs pa, int64_t n, PredView pv,
                                                        uint8_t* __restrict__ flags,
                                                        int64_t* __restrict__ ts) {
  const int64_t t = flag_filter_tile(blockIdx.x, pa, n, pv, flags);
  if (threadIdx.x == 0) ts[blockIdx.x] = t;
}

__global__ __launch_bounds__(kBlock) void k_flag_diag(const int32_t* __restrict__ a,
                                                      const int32_t* __restrict__ b, int64_t n,
                                                      uint8_t* __restrict__ flags,
                                                      int64_t* __restrict__ ts) {
  const int64_t tile0 = (int64_t)blockIdx.x * kTile;
  int64_t loc = 0;
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const int64_t i = tile0 + (int64_t)j * kBlock + threadIdx.x;
    if (i < n) {
      const uint8_t f = a[i] == b[i] ? 1 : 0;
      flags[i] = f;
      loc += f;
    }
  }
  const int64_t t = block_sum(loc);
  if (threadIdx.x == 0) ts[blockIdx.x] = t;
}

__global__ __launch_bounds__(kBlock) void k_flag_intersect(const int32_t* __restrict__ driver,
                                                           int64_t n, ListSet ls,
                                                           uint8_t* __restrict__ flags,
                                                           int64_t* __restrict__ ts) {
  const int64_t t = flag_intersect_tile(blockIdx.x, driver, n, ls.l, ls.n, flags);
  if (threadIdx.x == 0) ts[blockIdx.x] = t;
}

template <int K>
__global__ __launch_bounds__(kBlock) void k_compact_cols(ColSet in, int kdyn,
                                                         const uint8_t* __restrict__ flags,
                                                         int64_t n,
                                                         const int64_t* __restrict__ tile_off,
                                                         OutSet out) {
  compact_cols_tile<K>(blockIdx.x, in, kdyn, flags, n, tile_off[blockIdx.x], OutCols{&out});
}

// Merge path over A = row ends E[i] = P[i+1] (i < n) and B = output indices
// J0..J1-1, rows before outputs on ties.  split[t] = rows consumed before path
// position t*kTile.
__global__ void k_mp_partition(const int64_t* __restrict__ P, int64_t n, int64_t J0, int64_t J1,
                               int64_t* __restrict__ split, int64_t ntiles) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t > ntiles) return;
  split[t] = mp_split(P, n, J0, J1, t);
}
// A wave per split: for few splits, whose searches are one chain of loads
// however many there are (7.3 -> 4.7 us for 500; of 137 000 splits a thread
// each takes 9 us, a wave each 25 us).
constexpr int64_t kWaveSplits = 8192;
__global__ __launch_bounds__(kBlock) void k_mp_partition_wave(const int64_t* __restrict__ P,
                                                              int64_t n, int64_t J0, int64_t J1,
                                                              int64_t* __restrict__ split,
                                                              int64_t ntiles) {
  const int64_t t = (int64_t)blockIdx.x * kWaves + wave_id();
  if (t > ntiles) return;
  const int64_t a = mp_split_wave(P, n, J0, J1, t);
  if (lane_id() == 0) split[t] = a;
}

template <int K>
__global__ __launch_bounds__(kBlock) void k_write_expand(ColSet in, int kdyn,
                                                         const int64_t* __restrict__ P,
                                                         const int32_t* __restrict__ start,
                                                         int64_t n,
                                                         const int32_t* __restrict__ nbr,
                                                         int64_t J0, int64_t J1,
                                                         const int64_t* __restrict__ split,
                                                         OutSet out) {
  // 274 million rows of 3 columns: 662 us at U = 4, 618 to 648 at 8, 693 at 9
  constexpr int U = K < 0 ? 2 : K <= 2 ? 8 : K <= 8 ? 4 : 3;
  write_expand_tile<K, U>(blockIdx.x, in, kdyn, P, start, n, nbr, J0, J1, split, OutCols{&out});
}

__global__ void k_cartesian(ColSet a, int ka, ColSet b, int kb, int64_t nb, int64_t J0,
                            int64_t J1, OutSet out) {
  for (int64_t j = J0 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < J1;
       j += (int64_t)gridDim.x * blockDim.x) {
    const int64_t ia = j / nb, ib = j - ia * nb;
    const int64_t oj = j - J0;
    for (int c = 0; c < ka; ++c) out.c[c][oj] = a.c[c][ia];
    for (int c = 0; c < kb; ++c) out.c[ka + c][oj] = b.c[c][ib];
  }
}

// Sum of row lengths over a strided sample of the bound column; blockIdx.y
// selects the candidate, blockIdx.x one of kSampleBlocks slices of the sample.
__global__ __launch_bounds__(kBlock) void k_sample_fanout(SampleSet ss, int64_t* __restrict__ part,
                                                          uint32_t* words, uint32_t report) {
  const int cand = blockIdx.y;
  const int64_t t = sample_fanout_slice(blockIdx.x, ss.col[cand], ss.n, ss.pv[cand]);
  if (threadIdx.x == 0) part[cand * kSampleBlocks + blockIdx.x] = t;
  report_one(words ? words + cand * kSampleBlocks + blockIdx.x : nullptr, report);
}

// Rows to host memory, row-major.  The link (57 GB/s) is the bound, so a
// tile of kBlock rows is turned in LDS and leaves in 16-byte stores that a
// wave makes to consecutive addresses.  Writing where the host reads takes
// the device copy, the copy command and the wait for the stream out of a
// fetch: of up to 100 rows 35 -> 11.5 us, of 3 million rows of 4 columns 5.2 -> 4.3 ms.
// One wave makes a workgroup's stores, so that its report needs one write-back
// of the L2 and not one from every wave: 40 000 rows of 3 columns 21 -> 12.5 us
// (8.4 at the link's rate), 350 000 rows 99 -> 84 us.
// blockIdx.y is the task, the workgroups of a row stride over its tiles.
__global__ __launch_bounds__(kBlock) void k_pack_rows(PackTask one,
                                                      const PackTask* __restrict__ many,
                                                      uint32_t* words, uint32_t report) {
  __shared__ __align__(16) int32_t s[kBlock * kMaxCols];
  __shared__ PackTask task;
  static_assert(sizeof(PackTask) % 4 == 0 && sizeof(PackTask) / 4 <= kBlock, "one word a thread");
  if (many) {
    if (threadIdx.x < sizeof(PackTask) / 4)
      ((uint32_t*)&task)[threadIdx.x] = ((const uint32_t*)(many + blockIdx.y))[threadIdx.x];
    __syncthreads();
  }
  const int k = many ? task.k : one.k;
  const int64_t row0 = many ? task.row0 : one.row0, rows = many ? task.rows : one.rows;
  int32_t* const out = many ? task.out : one.out;
  const int64_t tiles = (rows + kBlock - 1) / kBlock;
  for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
    const int64_t r0 = t * kBlock;
    const int nr = (int)min((int64_t)kBlock, rows - r0);
    if ((int)threadIdx.x < nr)
      for (int c = 0; c < k; ++c) {
        const int32_t* col = many ? task.cols.c[c] : one.cols.c[c];  // none: unbound
        s[threadIdx.x * k + c] = col ? col[row0 + r0 + threadIdx.x] : -1;
      }
    __syncthreads();
    const int n = nr * k;
    int32_t* o = out + r0 * k;
    if (wave_id() == 0) {
      for (int i = lane_id() * 4; i + 4 <= n; i += 64 * 4)
        *reinterpret_cast<int4*>(o + i) = *reinterpret_cast<const int4*>(s + i);
      if (lane_id() < (n & 3)) o[(n & ~3) + lane_id()] = s[(n & ~3) + lane_id()];
    }
    __syncthreads();  // the next tile reuses the LDS
  }
  if (wave_id() == 0) report_wave(words + (int64_t)blockIdx.y * gridDim.x + blockIdx.x, report);
}

inline unsigned grid_for(int64_t n, int block = kBlock, int64_t cap = 65536) {
  int64_t g = ceil_div(n > 0 ? n : 1, block);
  if (g > cap) g = cap;
  return (unsigned)g;
}
inline unsigned tiles_for(int64_t n) { return (unsigned)ceil_div(n > 0 ? n : 1, kTile); }

}  // namespace

// ---------------------------------------------------------------- launchers
#define GS_LAUNCH(cls, bytes, ...)              \
  do {                                          \
    const bool _prof = prof_on(cls);            \
    if (_prof) prof_begin(s, cls);              \
    __VA_ARGS__;                                \
    GS_HIP(hipGetLastError());                  \
    if (_prof) prof_end(s, cls, bytes);         \
  } while (0)

void launch_scan_tile_sums(int64_t* tile_sum, int64_t nt, int64_t* total, hipStream_t s,
                           int64_t* host_total, uint32_t* word, uint32_t report) {
  GS_LAUNCH(GSMAT_K_SCAN, 16.0 * nt,
            hipLaunchKernelGGL(k_scan_tile_sums, dim3(1), dim3(kBlock), 0, s, tile_sum, nt, total,
                               host_total, word, report));
}

void launch_scan_tile_sums2(int64_t* ts, int64_t* ts2, int64_t nt, hipStream_t s) {
  GS_LAUNCH(GSMAT_K_SCAN, 32.0 * nt,
            hipLaunchKernelGGL(k_scan_tile_sums2, dim3(1), dim3(kScanBlock), 0, s, ts, ts2, nt));
}

void launch_scan_add_i32(const int32_t* N, int64_t n, const int64_t* tile_off, int64_t* P,
                         hipStream_t s) {
  GS_LAUNCH(GSMAT_K_SCAN, 12.0 * n,
            hipLaunchKernelGGL((k_scan_add<int32_t, int64_t>), dim3(tiles_for(n)), dim3(kBlock),
                               0, s, N, n, tile_off, P, 1));
}

bool launch_scan_rows(const int32_t* N, int64_t n, const int64_t* tile_sum, int64_t* P,
                      int64_t* host_total, uint32_t* word, uint32_t report, hipStream_t s) {
  if (ceil_div(n, kTile) > kTile) return false;
  GS_LAUNCH(GSMAT_K_SCAN, 12.0 * n,
            hipLaunchKernelGGL(k_scan_rows, dim3(tiles_for(n)), dim3(kBlock), 0, s, N, n, tile_sum,
                               P, host_total, word, report));
  return true;
}

void launch_tile_reduce_u32(const uint32_t* x, int64_t n, int64_t* tile_sum, hipStream_t s) {
  GS_LAUNCH(GSMAT_K_OTHER, 4.0 * n,
            hipLaunchKernelGGL(k_tile_reduce_u32, dim3(tiles_for(n)), dim3(kBlock), 0, s, x, n,
                               tile_sum));
}

void launch_scan_add_u32(const uint32_t* x, int64_t n, const int64_t* tile_off, uint32_t* out,
                         hipStream_t s) {
  GS_LAUNCH(GSMAT_K_OTHER, 8.0 * n,
            hipLaunchKernelGGL((k_scan_add<uint32_t, uint32_t>), dim3(tiles_for(n)),
                               dim3(kBlock), 0, s, x, n, tile_off, out, 0));
}

namespace {
template <int RB, bool kSwap>
void radix_pass(const uint64_t* src, uint64_t* dst, int64_t n, int shift, int vb, uint32_t* hist,
                uint32_t* offs, int64_t* ts, int64_t nb, hipStream_t s) {
  const int64_t hn = nb << RB;
  const int64_t ht = ceil_div(hn, kTile);
  GS_LAUNCH(GSMAT_K_OTHER, 8.0 * n,
            hipLaunchKernelGGL((k_rs_hist<RB, kSwap>), dim3((unsigned)nb), dim3(kBlock), 0, s, src,
                               n, shift, vb, hist, nb));
  launch_tile_reduce_u32(hist, hn, ts, s);
  launch_scan_tile_sums(ts, ht, ts + ht, s, nullptr);
  launch_scan_add_u32(hist, hn, ts, offs, s);
  GS_LAUNCH(GSMAT_K_OTHER, 16.0 * n,
            hipLaunchKernelGGL((k_rs_scatter<RB, kSwap>), dim3((unsigned)nb), dim3(kBlock), 0, s,
                               src, dst, n, shift, vb, offs, nb));
}
}  // namespace

uint64_t* radix_sort_u64(uint64_t* keys, uint64_t* tmp, int64_t n, int lo_bit, int hi_bit,
                         int swap_vb, DeviceMem& mem, hipStream_t s) {
  if (n <= 0) return keys;
  // 9-bit digits where they save a pass (27 bits: 3 against 4), else 8-bit
  // ones, whose runs are twice as long
  const int bits = hi_bit - lo_bit;
  const int rb = (bits + 8) / 9 < (bits + 7) / 8 ? 9 : 8;
  const int passes = std::max(1, (bits + rb - 1) / rb);
  const int64_t nb = ceil_div(n, kRsTile);
  const int64_t hn = nb << rb;
  const int64_t ht = ceil_div(hn, kTile);
  uint32_t* hist = (uint32_t*)mem.alloc(sizeof(uint32_t) * hn, s);
  uint32_t* offs = (uint32_t*)mem.alloc(sizeof(uint32_t) * hn, s);
  int64_t* ts = (int64_t*)mem.alloc(sizeof(int64_t) * (ht + 1), s);
  auto done = [&] {
    if (hist) mem.free(hist, sizeof(uint32_t) * hn, s);
    if (offs) mem.free(offs, sizeof(uint32_t) * hn, s);
    if (ts) mem.free(ts, sizeof(int64_t) * (ht + 1), s);
  };
  if (!hist || !offs || !ts) {
    done();
    throw OomFail{sizeof(uint32_t) * (size_t)hn};
  }
  uint64_t* src = keys;
  uint64_t* dst = tmp;
  try {
    for (int pass = 0; pass < passes; ++pass) {
      const int shift = lo_bit + rb * pass;
      const bool swap = swap_vb > 0 && pass == 0;
      if (rb == 8 && swap) radix_pass<8, true>(src, dst, n, shift, swap_vb, hist, offs, ts, nb, s);
      else if (rb == 8) radix_pass<8, false>(src, dst, n, shift, 0, hist, offs, ts, nb, s);
      else if (swap) radix_pass<9, true>(src, dst, n, shift, swap_vb, hist, offs, ts, nb, s);
      else radix_pass<9, false>(src, dst, n, shift, 0, hist, offs, ts, nb, s);
      std::swap(src, dst);
    }
  } catch (...) {
    done();
    throw;
  }
  done();
  return src;
}

void launch_pack_keys(const int32_t* sv, const int32_t* p, const int32_t* o, int64_t n, int vb,
                      uint64_t* k, hipStream_t s) {
  GS_LAUNCH(GSMAT_K_OTHER, 20.0 * n,
            hipLaunchKernelGGL(k_pack_keys, dim3(grid_for(n)), dim3(kBlock), 0, s, sv, p, o, n,
                               vb, k));
}

int launch_check_ids(const int32_t* sv, const int32_t* p, const int32_t* o, int64_t n, int32_t V,
                     int32_t P, int64_t* out, int max_out, hipStream_t s) {
  if (n <= 0) return 0;
  const unsigned g = (unsigned)std::min<int64_t>(max_out, ceil_div(n, 4 * kBlock));
  GS_LAUNCH(GSMAT_K_OTHER, 12.0 * n,
            hipLaunchKernelGGL(k_check_ids, dim3(g), dim3(kBlock), 0, s, sv, p, o, n, (uint32_t)V,
                               (uint32_t)P, out));
  return (int)g;
}

void launch_flag_unique(const uint64_t* k, int64_t n, uint8_t* flags, int64_t* tile_sum,
                        hipStream_t s) {
  GS_LAUNCH(GSMAT_K_OTHER, 9.0 * n,
            hipLaunchKernelGGL(k_flag_adjacent, dim3(tiles_for(n)), dim3(kBlock), 0, s, k, n,
                               flags, tile_sum));
}

void launch_row_count(const uint64_t* k, int64_t n, int vb, int64_t* pfe, int64_t* tile_sum,
                      hipStream_t s) {
  GS_LAUNCH(GSMAT_K_OTHER, 8.0 * n,
            hipLaunchKernelGGL(k_row_count, dim3(tiles_for(n)), dim3(kBlock), 0, s, k, n, vb, pfe,
                               tile_sum));
}

void launch_row_fill(const uint64_t* k, int64_t n, int vb, const int64_t* pfe,
                     const int64_t* tile_off, int32_t* nbr, int32_t* src, int32_t* keys,
                     int32_t* ptr, int64_t* pfr, hipStream_t s) {
  GS_LAUNCH(GSMAT_K_OTHER, (src ? 16.0 : 12.0) * n,
            hipLaunchKernelGGL(k_row_fill, dim3(tiles_for(n)), dim3(kBlock), 0, s, k, n, vb, pfe,
                               tile_off, nbr, src, keys, ptr, pfr));
}

void launch_compact_u64(const uint64_t* in, const uint8_t* flags, int64_t n,
                        const int64_t* tile_off, uint64_t* out, hipStream_t s) {
  GS_LAUNCH(GSMAT_K_COMPACT, 17.0 * n,
            hipLaunchKernelGGL(k_compact_u64, dim3(tiles_for(n)), dim3(kBlock), 0, s, in, flags,
                               n, tile_off, out));
}

void launch_fill_i64(int64_t* p, int64_t n, int64_t v, hipStream_t s) {
  if (n <= 0) return;
  GS_LAUNCH(GSMAT_K_OTHER, 8.0 * n,
            hipLaunchKernelGGL(k_fill_i64, dim3(grid_for(n)), dim3(kBlock), 0, s, p, n, v));
}

void launch_dense_ptrs(const PredDesc* desc, const int64_t* first, int32_t P, int64_t tiles,
                       const int32_t* keys, const int32_t* ptr, int64_t V, int32_t* dense,
                       hipStream_t s) {
  if (tiles <= 0) return;
  GS_LAUNCH(GSMAT_K_OTHER, 4.0 * kDenseTile * tiles,
            hipLaunchKernelGGL(k_dense_ptrs, dim3((unsigned)tiles), dim3(kBlock), 0, s, desc, first,
                               P, keys, ptr, V, dense));
}

void launch_row_dirs(const PredDesc* desc, const int64_t* first, int32_t P, int64_t tiles,
                     const int32_t* keys, int64_t V, int32_t* dir, hipStream_t s) {
  if (tiles <= 0) return;
  GS_LAUNCH(GSMAT_K_OTHER, 4.0 * kTile * tiles,
            hipLaunchKernelGGL(k_row_dirs, dim3((unsigned)tiles), dim3(kBlock), 0, s, desc, first, P,
                               keys, V, dir));
}

void launch_long_rows(PredView pv, int32_t min_len, int32_t* out, int32_t* count, int32_t cap,
                      hipStream_t s) {
  GS_LAUNCH(GSMAT_K_OTHER, 8.0 * pv.nr,
            hipLaunchKernelGGL(k_long_rows, dim3(grid_for(pv.nr)), dim3(kBlock), 0, s, pv, min_len,
                               out, count, cap));
}

void launch_row_bitmap(PredView pv, int32_t v, int64_t len, uint32_t* bm, hipStream_t s) {
  GS_LAUNCH(GSMAT_K_OTHER, 8.0 * len,
            hipLaunchKernelGGL(k_row_bitmap, dim3(grid_for(len)), dim3(kBlock), 0, s, pv, v, bm));
}

void launch_ptr_sentinels(const PredDesc* d, int32_t P, int32_t* ptr, hipStream_t s) {
  if (P <= 0) return;
  GS_LAUNCH(GSMAT_K_OTHER, 0.0,
            hipLaunchKernelGGL(k_ptr_sentinels, dim3((unsigned)ceil_div(P, kBlock)), dim3(kBlock), 0,
                               s, d, P, ptr));
}

void launch_lookup(const LookupBatch& b, const PredDesc* desc_out, const PredDesc* desc_in,
                   OriPtrs out, OriPtrs in, LookupRes* res, hipStream_t s, uint32_t* word,
                   uint32_t report) {
  if (b.n <= 0) return;
  GS_LAUNCH(GSMAT_K_OTHER, 32.0 * b.n,
            hipLaunchKernelGGL(k_lookup, dim3(1), dim3(64), 0, s, b, desc_out, desc_in, out, in,
                               res, word, report));
}

void launch_count_expand(const int32_t* col, int64_t n, PredView pv, int32_t* N, int32_t* start,
                         int64_t* tile_sum, hipStream_t s) {
  GS_LAUNCH(GSMAT_K_COUNT, 20.0 * n,
            hipLaunchKernelGGL(k_count_expand, dim3(tiles_for(n)), dim3(kBlock), 0, s, col, n, pv,
                               N, start, tile_sum));
}

void launch_flag_filter(ProbeArgs pa, int64_t n, PredView pv, uint8_t* flags, int64_t* tile_sum,
                        hipStream_t s) {
  GS_LAUNCH(GSMAT_K_COUNT, 21.0 * n,
            hipLaunchKernelGGL(k_flag_filter, dim3(tiles_for(n)), dim3(kBlock), 0, s, pa, n, pv,
                               flags, tile_sum));
}

void launch_flag_diag(const int32_t* a, const int32_t* b, int64_t n, uint8_t* flags,
                      int64_t* tile_sum, hipStream_t s) {
  GS_LAUNCH(GSMAT_K_COUNT, 9.0 * n,
            hipLaunchKernelGGL(k_flag_diag, dim3(tiles_for(n)), dim3(kBlock), 0, s, a, b, n, flags,
                               tile_sum));
}

void launch_flag_intersect(const int32_t* driver, int64_t n, ListSet ls, uint8_t* flags,
                           int64_t* tile_sum, hipStream_t s) {
  GS_LAUNCH(GSMAT_K_COUNT, (4.0 + 4.0 * ls.n + 1.0) * n,
            hipLaunchKernelGGL(k_flag_intersect, dim3(tiles_for(n)), dim3(kBlock), 0, s, driver, n,
                               ls, flags, tile_sum));
}

void launch_compact_cols(ColSet in, int k, const uint8_t* flags, int64_t n,
                         const int64_t* tile_off, OutSet out, hipStream_t s) {
#define GS_COMPACT_CASE(KK)                                                                    \
  case KK:                                                                                   \
    hipLaunchKernelGGL(k_compact_cols<KK>, dim3(tiles_for(n)), dim3(kBlock), 0, s, in, k, flags, \
                       n, tile_off, out);                                                    \
    break;
  GS_LAUNCH(GSMAT_K_COMPACT, (1.0 + 4.0 * k) * n, switch (k) {
    GS_COMPACT_CASE(1)
    GS_COMPACT_CASE(2)
    GS_COMPACT_CASE(3)
    GS_COMPACT_CASE(4)
    GS_COMPACT_CASE(5)
    GS_COMPACT_CASE(6)
    GS_COMPACT_CASE(7)
    GS_COMPACT_CASE(8)
    default:
      hipLaunchKernelGGL(k_compact_cols<-1>, dim3(tiles_for(n)), dim3(kBlock), 0, s, in, k, flags, n,
                         tile_off, out);
  });
#undef GS_COMPACT_CASE
}

void launch_mp_partition(const int64_t* P, int64_t n, int64_t J0, int64_t J1, int64_t* split,
                         int64_t ntiles, hipStream_t s) {
  if (ntiles < kWaveSplits) {
    GS_LAUNCH(GSMAT_K_OTHER, 8.0 * (ntiles + 1),
              hipLaunchKernelGGL(k_mp_partition_wave, dim3((unsigned)ceil_div(ntiles + 1, kWaves)),
                                 dim3(kBlock), 0, s, P, n, J0, J1, split, ntiles));
    return;
  }
  GS_LAUNCH(GSMAT_K_OTHER, 8.0 * (ntiles + 1),
            hipLaunchKernelGGL(k_mp_partition, dim3((unsigned)ceil_div(ntiles + 1, kBlock)),
                               dim3(kBlock), 0, s, P, n, J0, J1, split, ntiles));
}

void launch_write_expand(ColSet in, int k, const int64_t* P, const int32_t* start, int64_t n,
                         const int32_t* nbr, int64_t J0, int64_t J1, const int64_t* split,
                         int64_t ntiles, OutSet out, double alg_bytes, hipStream_t s) {
#define GS_WRITE_CASE(KK)                                                                        \
  case KK:                                                                                     \
    hipLaunchKernelGGL(k_write_expand<KK>, dim3((unsigned)ntiles), dim3(kBlock), 0, s, in, k, P, \
                       start, n, nbr, J0, J1, split, out);                                      \
    break;
  GS_LAUNCH(GSMAT_K_WRITE, alg_bytes, switch (k) {
    GS_WRITE_CASE(0)
    GS_WRITE_CASE(1)
    GS_WRITE_CASE(2)
    GS_WRITE_CASE(3)
    GS_WRITE_CASE(4)
    GS_WRITE_CASE(5)
    GS_WRITE_CASE(6)
    GS_WRITE_CASE(7)
    GS_WRITE_CASE(8)
    GS_WRITE_CASE(9)
    GS_WRITE_CASE(10)
    GS_WRITE_CASE(11)
    default:
      hipLaunchKernelGGL(k_write_expand<-1>, dim3((unsigned)ntiles), dim3(kBlock), 0, s, in, k, P,
                         start, n, nbr, J0, J1, split, out);
  });
#undef GS_WRITE_CASE
}

void launch_cartesian(ColSet a, int ka, int64_t na, ColSet b, int kb, int64_t nb, int64_t J0,
                      int64_t J1, OutSet out, hipStream_t s) {
  (void)na;
  GS_LAUNCH(GSMAT_K_OTHER, 4.0 * (ka + kb) * 2.0 * (J1 - J0),
            hipLaunchKernelGGL(k_cartesian, dim3(grid_for(J1 - J0)), dim3(kBlock), 0, s, a, ka, b,
                               kb, nb, J0, J1, out));
}

void launch_sample_fanout(const SampleSet& ss, int64_t* part, hipStream_t s, uint32_t* words,
                          uint32_t report) {
  GS_LAUNCH(GSMAT_K_OTHER, 0.0,
            hipLaunchKernelGGL(k_sample_fanout, dim3(kSampleBlocks, (unsigned)ss.ncand),
                               dim3(kBlock), 0, s, ss, part, words, report));
}

int launch_pack_rows(const PackTask* tasks, int n, uint32_t* words, uint32_t report,
                     hipStream_t s) {
  int64_t most = 1;
  double bytes = 0;
  for (int i = 0; i < n; ++i) {
    most = std::max(most, tasks[i].rows);
    bytes += 8.0 * tasks[i].k * (double)tasks[i].rows;
  }
  const int gx = std::min((int)grid_for(most, kBlock, kPackGroups), kPackWords / n);
  GS_LAUNCH(GSMAT_K_OTHER, bytes,
            hipLaunchKernelGGL(k_pack_rows, dim3((unsigned)gx, (unsigned)n), dim3(kBlock), 0, s,
                               tasks[0], n > 1 ? tasks : nullptr, words, report));
  return gx * n;
}

}  // namespace gsmat
