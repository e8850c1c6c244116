// Key-sorted export of a store: the live strings in ascending order of their
// integer (Appendix E.2: qubit q is the base-4 digit of weight 4^q, with
// I, X, Y, Z = 0, 1, 2, 3; the same integer that picks a representative in
// Algorithms 2 and 3), so a merged set comes out one record per
// representative, sorted by key.
//
// Least-significant-digit radix sort of slot indices, 8 bits per pass, the
// digit read from the store through the index (no key arrays): per pass a
// histogram per tile of 4096 positions, one exclusive scan over the
// digit-major histogram, and a stable scatter.  The first pass reads the
// store's slots directly and drops the dead ones, so it also compacts.
// Ordering only: no arithmetic on coefficients.
//
// That takes five launches per 8 bits, 40 for a 32-qubit set, and most sets
// are too small for any of them to run longer than it takes to launch.  Sets
// of up to samp_max<NK>() strings are sorted by sampling instead, in five
// launches whatever the width (two up to samp_cap<NK>() / 2 strings, which
// one block sorts in less time than three launches take):
//   k_samp_keys     the live strings' integers (NK words) and slots;
//   k_samp_split    one block sorts a sample and picks P - 1 splitters;
//   k_samp_rank     every string's bucket (binary search) and rank in it; the
//                   last block turns the counts into bucket bases;
//   k_samp_place    strings to bucket order;
//   k_samp_sort     one block per bucket sorts it in LDS (bitonic) and writes
//                   the rows; a bucket that outgrows the LDS is sorted a chunk
//                   at a time and each string ranked in the other chunks.
// The strings are distinct, so eight samples per bucket keep the buckets near
// their average: 1024 buckets that average a quarter of the LDS (2^19 strings of
// one or two key words) hardly ever hold one that outgrows it, at the half that
// samp_max admits about ten do.  Above, the radix passes move each string a
// fixed number of times while a block could not sort the sample.
// Whole export, before -> after: 10^5 strings of 32 qubits 640 -> 360 us (the
// rest is copies), 4349 strings 440 -> 186 us, 5 strings of 64 qubits 400 ->
// 115 us, 5.8x10^5 strings of 48 qubits 1.92 -> 1.6 ms.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "pp_kernels.hpp"
#include "pp_types.h"

constexpr int kSortBlock = 256;                       // = radix: thread t owns digit t
constexpr int kSortItems = 16;
constexpr int kSortTile = kSortBlock * kSortItems;    // positions per tile
constexpr int kSortWaves = kSortBlock / 64;
constexpr int kScanTile = 4096;                       // histogram entries per scan block

// Bit i of v moves to bit 2i (interleave by binary magic numbers).
__device__ __forceinline__ uint64_t sort_spread32(uint32_t v) {
  uint64_t r = v;
  r = (r | (r << 16)) & 0x0000FFFF0000FFFFull;
  r = (r | (r << 8)) & 0x00FF00FF00FF00FFull;
  r = (r | (r << 4)) & 0x0F0F0F0F0F0F0F0Full;
  r = (r | (r << 2)) & 0x3333333333333333ull;
  r = (r | (r << 1)) & 0x5555555555555555ull;
  return r;
}

// 64-bit word j of slot i's integer (qubits 32j .. 32j+31).  A letter's
// digit is 2z + (x xor z): I 00, X 01, Y 10, Z 11.
__device__ __forceinline__ uint64_t sort_int_word(const uint64_t* xs, const uint64_t* zs,
                                                  uint32_t cap, uint32_t i, int j) {
  const int w = j >> 1, sh = (j & 1) * 32;
  const uint64_t xw = xs[(size_t)w * cap + i], zw = zs[(size_t)w * cap + i];
  return (sort_spread32((uint32_t)(zw >> sh)) << 1) | sort_spread32((uint32_t)((xw ^ zw) >> sh));
}

struct SortPass {
  const uint64_t* x;       // store half: [W][cap]
  const uint64_t* z;
  const uint8_t* alive;    // first pass: liveness of slot i
  const uint32_t* src;     // later passes: slot at each position
  uint32_t* dst;           // slot at each output position
  uint32_t dst_cap;        // positions dst holds (a larger count is reported, not written)
  uint32_t* hist;          // [256][tiles], then exclusive offsets
  uint32_t cap;
  uint32_t n_in;           // positions read (store slots on the first pass)
  uint32_t tiles;
  int word;                // integer word j and bit shift inside it
  int shift;
  int first;
};

__device__ __forceinline__ bool sort_item(const SortPass& p, uint32_t i, uint32_t& slot,
                                          uint32_t& digit) {
  if (i >= p.n_in) return false;
  if (p.first) {
    if (!p.alive[i]) return false;
    slot = i;
  } else {
    slot = p.src[i];
  }
  digit = (uint32_t)(sort_int_word(p.x, p.z, p.cap, slot, p.word) >> p.shift) & 255u;
  return true;
}

__global__ __launch_bounds__(kSortBlock) void k_sort_hist(SortPass p) {
  __shared__ uint32_t cnt[kSortBlock];
  const int t = threadIdx.x;
  cnt[t] = 0;
  __syncthreads();
  const uint32_t base = blockIdx.x * (uint32_t)kSortTile;
  for (int k = 0; k < kSortItems; ++k) {
    uint32_t slot, digit;
    if (sort_item(p, base + k * kSortBlock + t, slot, digit)) atomicAdd(&cnt[digit], 1u);
  }
  __syncthreads();
  p.hist[(size_t)t * p.tiles + blockIdx.x] = cnt[t];
}

// Exclusive scan of n entries in three launches: per-block totals, one
// block over the totals (which also writes the grand total), per-block
// rescan with the block's offset.
__device__ __forceinline__ uint32_t sort_block_scan(uint32_t v, uint32_t* sh, uint32_t& total) {
  // inclusive scan over kSortBlock threads, returns the exclusive prefix
  const int t = threadIdx.x;
  sh[t] = v;
  __syncthreads();
  for (int o = 1; o < kSortBlock; o <<= 1) {
    const uint32_t a = t >= o ? sh[t - o] : 0u;
    __syncthreads();
    sh[t] += a;
    __syncthreads();
  }
  const uint32_t incl = sh[t];
  total = sh[kSortBlock - 1];
  __syncthreads();
  return incl - v;
}

__global__ __launch_bounds__(kSortBlock) void k_sort_scan_reduce(const uint32_t* a, uint32_t n,
                                                                 uint32_t* part) {
  __shared__ uint32_t sh[kSortBlock];
  const uint32_t base = blockIdx.x * (uint32_t)kScanTile;
  uint32_t s = 0;
  for (int k = threadIdx.x; k < kScanTile; k += kSortBlock)
    if (base + k < n) s += a[base + k];
  uint32_t total;
  (void)sort_block_scan(s, sh, total);
  if (threadIdx.x == 0) part[blockIdx.x] = total;
}

__global__ __launch_bounds__(kSortBlock) void k_sort_scan_top(uint32_t* part, uint32_t n,
                                                              uint32_t* grand) {
  __shared__ uint32_t sh[kSortBlock];
  uint32_t carry = 0;
  for (uint32_t b = 0; b < n; b += kSortBlock) {
    const uint32_t i = b + threadIdx.x;
    const uint32_t v = i < n ? part[i] : 0u;
    uint32_t total;
    const uint32_t ex = sort_block_scan(v, sh, total);
    if (i < n) part[i] = carry + ex;
    carry += total;
  }
  if (threadIdx.x == 0) *grand = carry;
}

__global__ __launch_bounds__(kSortBlock) void k_sort_scan_down(uint32_t* a, uint32_t n,
                                                               const uint32_t* part) {
  __shared__ uint32_t sh[kSortBlock];
  // thread t rescans the contiguous run [t*16, t*16 + 16) of the block's tile
  constexpr int kRun = kScanTile / kSortBlock;
  const uint32_t base = blockIdx.x * (uint32_t)kScanTile + threadIdx.x * kRun;
  uint32_t v[kRun], s = 0;
#pragma unroll
  for (int k = 0; k < kRun; ++k) {
    v[k] = base + k < n ? a[base + k] : 0u;
    s += v[k];
  }
  uint32_t total;
  uint32_t run = part[blockIdx.x] + sort_block_scan(s, sh, total);
#pragma unroll
  for (int k = 0; k < kRun; ++k) {
    if (base + k < n) a[base + k] = run;
    run += v[k];
  }
}

// Stable scatter of one tile: positions are taken 256 at a time in order;
// inside a wave, lanes with the same digit find each other with eight
// ballots, and earlier waves' counts come from LDS.
__global__ __launch_bounds__(kSortBlock) void k_sort_scatter(SortPass p) {
  __shared__ uint32_t base[kSortBlock];
  __shared__ uint32_t wcnt[kSortWaves][kSortBlock];
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
  base[t] = p.hist[(size_t)t * p.tiles + blockIdx.x];
#pragma unroll
  for (int w = 0; w < kSortWaves; ++w) wcnt[w][t] = 0;
  __syncthreads();
  const uint32_t tile = blockIdx.x * (uint32_t)kSortTile;
  const uint64_t below = (1ull << lane) - 1ull;
  for (int k = 0; k < kSortItems; ++k) {
    uint32_t slot = 0, digit = 0;
    const bool valid = sort_item(p, tile + k * kSortBlock + t, slot, digit);
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const bool bit = (digit >> b) & 1u;
      const uint64_t m = __ballot(bit);
      peers &= bit ? m : ~m;
    }
    const uint32_t rank = __popcll(peers & below);
    if (valid && lane == 63 - __clzll(peers)) wcnt[wave][digit] = __popcll(peers);
    __syncthreads();
    if (valid) {
      uint32_t pos = base[digit] + rank;
      for (int w = 0; w < wave; ++w) pos += wcnt[w][digit];
      if (pos < p.dst_cap) p.dst[pos] = slot;
    }
    __syncthreads();
    uint32_t tot = 0;
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) {
      tot += wcnt[w][t];
      wcnt[w][t] = 0;
    }
    base[t] += tot;
    __syncthreads();
  }
}

// Rows in output order: x/z as W words per row, coefficients as FP64.
__global__ __launch_bounds__(kSortBlock) void k_sort_emit(const uint32_t* order, uint32_t n,
                                                          const uint64_t* xs, const uint64_t* zs,
                                                          const void* c, int f32, uint32_t cap,
                                                          int W, uint64_t* ox, uint64_t* oz,
                                                          double* oc) {
  const uint32_t r = blockIdx.x * kSortBlock + threadIdx.x;
  if (r >= n) return;
  const uint32_t i = order[r];
  for (int w = 0; w < W; ++w) {
    ox[(size_t)r * W + w] = xs[(size_t)w * cap + i];
    oz[(size_t)r * W + w] = zs[(size_t)w * cap + i];
  }
  oc[r] = f32 ? (double)static_cast<const float*>(c)[i] : static_cast<const double*>(c)[i];
}

// ---------------------------------------------------------------------------
// sampling sort
// ---------------------------------------------------------------------------
// Key words of an n-qubit string's integer: 32 qubits a word (3 round to 4).
constexpr int samp_words(int n) { return n <= 32 ? 1 : n <= 64 ? 2 : 4; }
template <int NK> constexpr uint32_t samp_size() { return NK == 4 ? 4096 : 8192; }   // sample
template <int NK> constexpr uint32_t samp_cap() { return NK == 4 ? 1024 : 2048; }    // LDS bucket
template <int NK> constexpr uint32_t samp_buckets() { return samp_size<NK>() / 8; }
template <int NK> constexpr uint32_t samp_max() { return samp_buckets<NK>() * samp_cap<NK>() / 2; }

struct SampSort {
  const uint64_t* x;       // store half: [W][cap]
  const uint64_t* z;
  const uint8_t* alive;
  const void* c;
  uint32_t cap, M, N;      // entries, live strings
  int W, n, f32;
  uint32_t P;              // buckets (1: no splitters)
  uint64_t* key;           // [NK][N] integers, then in bucket order (key2)
  uint64_t* key2;
  uint32_t* slot;          // [N]
  uint32_t* slot2;
  uint32_t* bk;            // [N] bucket, rank
  uint32_t* rank;
  uint64_t* split;         // [NK][P]
  uint32_t* cnt;           // [1 + P] strings found, strings per bucket (cleared)
  uint32_t* base;          // [P]
  uint32_t* found;         // pinned host memory: cnt[0] for the host
  uint32_t* sync;          // done counters (pp::last_block)
  uint64_t* ox;
  uint64_t* oz;
  double* oc;
};

template <int NK>
__device__ __forceinline__ bool samp_less(const uint64_t* a, const uint64_t* b) {
#pragma unroll
  for (int w = NK - 1; w > 0; --w)
    if (a[w] != b[w]) return a[w] < b[w];
  return a[0] < b[0];
}

// Strings the kernels may read (the host checks cnt[0] == N afterwards).
__device__ __forceinline__ uint32_t samp_n(const SampSort& p) {
  return p.cnt[0] < p.N ? p.cnt[0] : p.N;
}

template <int NK>
__global__ __launch_bounds__(kSortBlock) void k_samp_keys(SampSort p) {
  __shared__ uint32_t s_n, s_base;
  constexpr int U = 4;
  if (threadIdx.x == 0) s_n = 0;
  __syncthreads();
  uint32_t at[U];
  bool live[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t i = (blockIdx.x * U + u) * kSortBlock + threadIdx.x;
    live[u] = i < p.M && p.alive[i];
    at[u] = live[u] ? atomicAdd(&s_n, 1u) : 0u;
  }
  __syncthreads();
  if (threadIdx.x == 0) s_base = s_n ? atomicAdd(&p.cnt[0], s_n) : 0u;
  __syncthreads();
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t i = (blockIdx.x * U + u) * kSortBlock + threadIdx.x, pos = s_base + at[u];
    if (!live[u] || pos >= p.N) continue;
    p.slot[pos] = i;
#pragma unroll
    for (int w = 0; w < NK; ++w)
      p.key[(size_t)w * p.N + pos] = 32 * w < p.n ? sort_int_word(p.x, p.z, p.cap, i, w) : 0ull;
  }
}

// Bitonic sort of the first sz (a power of two) of a block's LDS entries by
// (key, id); entries past the data hold all-ones keys with larger ids.
template <int NK, int CAP>
__device__ __forceinline__ void samp_bitonic(uint64_t (*key)[CAP], uint16_t* id, uint32_t sz) {
  for (uint32_t k = 2; k <= sz; k <<= 1)
    for (uint32_t j = k >> 1; j; j >>= 1) {
      for (uint32_t t = threadIdx.x; t < sz / 2; t += blockDim.x) {
        const uint32_t a = ((t & ~(j - 1)) << 1) | (t & (j - 1)), b = a | j;
        uint64_t ka[NK], kb[NK];
#pragma unroll
        for (int w = 0; w < NK; ++w) { ka[w] = key[w][a]; kb[w] = key[w][b]; }
        const uint16_t ia = id[a], ib = id[b];
        const bool bl = samp_less<NK>(kb, ka) || (!samp_less<NK>(ka, kb) && ib < ia);
        if (bl == ((a & k) == 0)) {
#pragma unroll
          for (int w = 0; w < NK; ++w) { key[w][a] = kb[w]; key[w][b] = ka[w]; }
          id[a] = ib;
          id[b] = ia;
        }
      }
      __syncthreads();
    }
}

// Eight samples per bucket (with four, one of 1024 buckets of a quarter of
// the LDS overflows it every third time), one at a hashed position in each of as
// many even stretches of the store.  At evenly spaced positions they would meet
// the store's own periods: 2^19 strings made by one rotation after another hold
// the letters of the first rotations' qubits in the low bits of their index,
// every 64th has the same, and all but 2^13 of them fell into one of 1024 buckets.
template <int NK>
__global__ __launch_bounds__(1024) void k_samp_split(SampSort p) {
  constexpr uint32_t S = samp_size<NK>();
  __shared__ uint64_t key[NK][S];
  __shared__ uint16_t id[S];
  const uint32_t n = samp_n(p), sz = 8 * p.P;    // P <= S / 8
  for (uint32_t t = threadIdx.x; t < sz; t += blockDim.x) {
    const uint32_t lo = (uint32_t)((uint64_t)t * n / sz);
    const uint32_t len = (uint32_t)((uint64_t)(t + 1) * n / sz) - lo;
    const uint32_t i = len ? lo + (uint32_t)(pp::mix64(t) % len) : lo;   // < n (n = 0: unused)
#pragma unroll
    for (int w = 0; w < NK; ++w) key[w][t] = n ? p.key[(size_t)w * p.N + i] : 0ull;
    id[t] = (uint16_t)t;
  }
  __syncthreads();
  samp_bitonic<NK, (int)S>(key, id, sz);
  for (uint32_t t = threadIdx.x; t + 1 < p.P; t += blockDim.x)
#pragma unroll
    for (int w = 0; w < NK; ++w) p.split[(size_t)w * p.P + t] = key[w][8 * (t + 1)];
}

template <int NK>
__global__ __launch_bounds__(kSortBlock) void k_samp_rank(SampSort p) {
  constexpr uint32_t PM = samp_buckets<NK>();
  constexpr int U = 4;
  __shared__ uint64_t split[NK][PM];
  __shared__ uint32_t cnt[PM], s_tmp[pp::kWaves + 1], s_flag;
  const uint32_t n = samp_n(p), P = p.P;
  const uint32_t rounds = (n + U * kSortBlock - 1) / (U * kSortBlock);
  const uint32_t workers = pp::worker_count(rounds);
  if (blockIdx.x >= workers) return;
  for (uint32_t t = threadIdx.x; t + 1 < P; t += kSortBlock)
#pragma unroll
    for (int w = 0; w < NK; ++w) split[w][t] = p.split[(size_t)w * P + t];
  for (uint32_t r = blockIdx.x; r < rounds; r += gridDim.x) {
    __syncthreads();
    for (uint32_t t = threadIdx.x; t < P; t += kSortBlock) cnt[t] = 0;
    __syncthreads();
    uint32_t bk[U], rk[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t i = (r * U + u) * kSortBlock + threadIdx.x;
      bk[u] = 0;
      if (i >= n) continue;
      uint64_t k[NK];
#pragma unroll
      for (int w = 0; w < NK; ++w) k[w] = p.key[(size_t)w * p.N + i];
      // splitters <= k: one bit of the answer per step (P - 1 of them)
      uint32_t lo = 0;
      for (uint32_t step = P >> 1; step; step >>= 1) {
        uint64_t m[NK];
#pragma unroll
        for (int w = 0; w < NK; ++w) m[w] = split[w][lo + step - 1];
        if (!samp_less<NK>(k, m)) lo += step;
      }
      bk[u] = lo;
      rk[u] = atomicAdd(&cnt[lo], 1u);
    }
    __syncthreads();
    for (uint32_t t = threadIdx.x; t < P; t += kSortBlock) {
      const uint32_t c = cnt[t];
      cnt[t] = c ? atomicAdd(&p.cnt[1 + t], c) : 0u;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t i = (r * U + u) * kSortBlock + threadIdx.x;
      if (i >= n) continue;
      p.bk[i] = bk[u];
      p.rank[i] = cnt[bk[u]] + rk[u];
    }
  }
  if (!pp::last_block(p.sync, &s_flag, workers)) return;
  __syncthreads();
  uint32_t carry = 0;
  for (uint32_t t0 = 0; t0 < P; t0 += kSortBlock) {
    const uint32_t t = t0 + threadIdx.x, c = t < P ? pp::ld_agent(&p.cnt[1 + t]) : 0u;
    uint32_t total;
    const uint32_t off = pp::block_scan(c, s_tmp, &total);
    if (t < P) p.base[t] = carry + off;
    carry += total;
  }
}

template <int NK>
__global__ __launch_bounds__(kSortBlock) void k_samp_place(SampSort p) {
  const uint32_t n = samp_n(p), i = blockIdx.x * kSortBlock + threadIdx.x;
  if (i >= n) return;
  const uint32_t pos = p.base[p.bk[i]] + p.rank[i];   // < n
  p.slot2[pos] = p.slot[i];
#pragma unroll
  for (int w = 0; w < NK; ++w) p.key2[(size_t)w * p.N + pos] = p.key[(size_t)w * p.N + i];
}

template <int NK>
__global__ __launch_bounds__(kSortBlock) void k_samp_sort(SampSort p) {
  constexpr uint32_t CAP = samp_cap<NK>();
  __shared__ uint64_t key[NK][CAP];
  __shared__ uint16_t id[CAP];
  const uint32_t n = samp_n(p);
  if (blockIdx.x == 0 && threadIdx.x == 0) *p.found = p.cnt[0];
  const uint32_t b = p.P == 1 ? n : p.cnt[1 + blockIdx.x];
  const uint32_t base = p.P == 1 ? 0u : p.base[blockIdx.x];
  auto row = [&](uint32_t r, uint32_t i) {
    for (int w = 0; w < p.W; ++w) {
      p.ox[(size_t)r * p.W + w] = p.x[(size_t)w * p.cap + i];
      p.oz[(size_t)r * p.W + w] = p.z[(size_t)w * p.cap + i];
    }
    p.oc[r] = p.f32 ? (double)static_cast<const float*>(p.c)[i] : static_cast<const double*>(p.c)[i];
  };
  // strings [at, at + m) of the bucket into LDS, sorted
  auto sort = [&](uint32_t at, uint32_t m) {
    uint32_t sz = 2;
    while (sz < m) sz <<= 1;
    for (uint32_t t = threadIdx.x; t < sz; t += kSortBlock) {
#pragma unroll
      for (int w = 0; w < NK; ++w)
        key[w][t] = t < m ? p.key2[(size_t)w * p.N + base + at + t] : ~0ull;
      id[t] = (uint16_t)t;
    }
    __syncthreads();
    samp_bitonic<NK, (int)CAP>(key, id, sz);
  };
  if (b <= CAP) {
    sort(0, b);
    for (uint32_t t = threadIdx.x; t < b; t += kSortBlock) row(base + t, p.slot2[base + id[t]]);
    return;
  }
  // past the LDS (uniform; P > 1): sorted chunks go to the bucket's part of the
  // unplaced keys and slots, which are free by now.  Export of 2^20 strings of
  // 32 qubits, about ten such buckets: 3.4 ms with every string compared to its
  // whole bucket, 1.9 ms so (radix passes 2.2).
  for (uint32_t at = 0; at < b; at += CAP) {
    const uint32_t m = b - at < CAP ? b - at : CAP;
    sort(at, m);
    for (uint32_t t = threadIdx.x; t < m; t += kSortBlock) {
#pragma unroll
      for (int w = 0; w < NK; ++w) p.key[(size_t)w * p.N + base + at + t] = key[w][t];
      p.slot[base + at + t] = p.slot2[base + at + id[t]];
    }
    __syncthreads();
  }
  for (uint32_t e = threadIdx.x; e < b; e += kSortBlock) {
    uint64_t k[NK];
#pragma unroll
    for (int w = 0; w < NK; ++w) k[w] = p.key[(size_t)w * p.N + base + e];
    const uint32_t own = e / CAP * CAP;
    uint32_t r = e - own;
    for (uint32_t at = 0; at < b; at += CAP) {   // plus the smaller strings of the others
      if (at == own) continue;
      uint32_t lo = 0, hi = b - at < CAP ? b - at : CAP;
      while (lo < hi) {
        const uint32_t q = (lo + hi) / 2;
        uint64_t m[NK];
#pragma unroll
        for (int w = 0; w < NK; ++w) m[w] = p.key[(size_t)w * p.N + base + at + q];
        if (samp_less<NK>(m, k)) lo = q + 1;
        else hi = q;
      }
      r += lo;
    }
    row(base + r, p.slot[base + e]);
  }
}
