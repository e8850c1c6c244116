// Layer op: a commuting run of rotations applied bucket by bucket.
//
// Prop. 1 with the exact merge of identical strings and the truncation
// after every rotation (Algorithm 1 step 2a), for r <= kLayerMaxRot
// pairwise commuting rotations P_1..P_r of one sub-layer, in circuit order.
//
// Why buckets are closed.  Let a(Q) be the set of g with {P_g, Q} = 0.  For
// g in a(Q), P_g Q anticommutes with P_h exactly when Q does (the P's
// commute), so a is the same on the whole set Q <P_g : g in a(Q)>, which is
// everything the r rotations can make from Q.  Multiplying by such a P_g
// flips only bits inside the union of the x- and z-supports of {P_g : g in
// a}, so the key (a, x outside that x-union, z outside that z-union) is the
// same for every member.  A bucket of a hash of the key therefore holds, for
// each string in it, its partner under every rotation and every child the
// rotations can make: a block rotates its bucket in LDS with no other block.
//
// A string runs its own rotations a(Q) in circuit order, each with its
// partner P_g Q found in the block's LDS hash table: both live -> the pair
// rotation (the lower index writes both), partner absent or dropped -> cos
// on Q and a child sin on P_g Q (a dropped partner's slot is reused), then
// the truncation of what changed, exactly as the one-rotation gate kernel
// does it, so the results are bitwise those of r gate launches.  Children
// of a step get indices past those it reads.
//
// Measured (MI355X, kernel average per launch, before -> after the apply step
// took its present form: a string's q-th own rotation per step, one
// select-based path, table probes as DS instead of FLAT loads, finer buckets
// for small sets, sums without LDS round trips): Z_8 ring untruncated 42 ->
// 19 us, the Z_32 ring (10^5 strings) 40 -> 25 us, the same circuit unmerged
// (5x10^5 strings) 124 -> 43 us.
#pragma once
#include "pp_kernels.hpp"

namespace pp {

constexpr uint32_t kAlive = 0xFFu;   // died field of a live string (see live_before)

// Key words of a string in the apply step's LDS: one (x | z << 32) for n <= 32,
// else its W x words, then its W z words.
__host__ __device__ __forceinline__ int layer_key_words(int n, int W) {
  return n <= 32 ? 1 : 2 * W;
}

// Strings per bucket in LDS: half a CU's 160 KB, or all of it (`big`: for closed
// sets that do not fit the smaller form).  One block of 512 threads runs per CU
// in either form: the kernel takes 197 registers a thread, which leave two waves
// a SIMD.  The rotations are not what takes them (66 to 89 by key width): it is
// the unrolled fold of layer_end, whose one thread holds 112 sums at once.  For
// the same reason the larger form keeps 512 threads: with 1024 that fold spills
// to scratch memory, which the runtime cannot get once a caller's allocator
// holds the device's.
template <int KW, bool Big>
constexpr int layer_cap() {
  constexpr int n = KW == 1 ? 2048 : KW == 2 ? 1792 : 1024;
  // (one word: room beside a full set of 2^12 strings)
  return Big ? (KW == 1 ? 4608 : 2 * n) : n;
}

// Bucket bits for a layer op over M entries: about 2^shift strings per
// bucket, more after failures (boost), at most maxbits.
__device__ __host__ __forceinline__ uint32_t layer_bits(uint32_t M, int32_t boost,
                                                        uint32_t maxbits, uint32_t shift) {
  uint32_t lg = 0;
  while (lg < 32 && (1ull << lg) < (uint64_t)M) ++lg;
  int bits = (int)lg - (int)shift;
  const int fine = (int)lg - kLayerFine < kLayerFillBits ? (int)lg - kLayerFine : kLayerFillBits;
  if (bits < fine) bits = fine;
  bits += boost;                             // boost: from earlier failures
  if (bits < 0) bits = 0;
  if (bits > (int)maxbits) bits = (int)maxbits;
  return (uint32_t)bits;
}

__device__ __forceinline__ uint64_t rot_word(const double* t, int k) {
  return (uint64_t)__double_as_longlong(t[k]);
}

// The bucket key's hash (anticommutation pattern and the bits no
// anticommuting rotation touches); *pat = the pattern.
template <int WW>
__device__ __forceinline__ uint64_t layer_key(const uint64_t* x, const uint64_t* z, uint32_t r,
                                              const uint64_t (*px)[WW], const uint64_t (*pz)[WW],
                                              uint64_t* pat) {
  uint64_t a = 0, ux[WW], uz[WW];
#pragma unroll
  for (int w = 0; w < WW; ++w) ux[w] = uz[w] = 0;
  for (uint32_t g = 0; g < r; ++g) {
    uint32_t par = 0;
#pragma unroll
    for (int w = 0; w < WW; ++w) par += __popcll((x[w] & pz[g][w]) ^ (z[w] & px[g][w]));
    if (par & 1u) {
      a |= 1ull << g;
#pragma unroll
      for (int w = 0; w < WW; ++w) {
        ux[w] |= px[g][w];
        uz[w] |= pz[g][w];
      }
    }
  }
  uint64_t h = mix64(a ^ 0x2545f4914f6cdd1dull);
#pragma unroll
  for (int w = 0; w < WW; ++w) {
    h = mix64(h ^ (x[w] & ~ux[w]));
    h = mix64(h ^ (z[w] & ~uz[w]) ^ 0x9e3779b97f4a7c15ull);
  }
  *pat = a;
  return h;
}

// strings per thread per scatter round: one gives the most rounds (blocks)
// and the shortest chain per block (measured faster than 2, 4 or 8)
constexpr int kLTile = 1;
constexpr int kLAggMax = 2048;             // buckets counted in LDS before the global add

// 1. Every live string of the current half to its bucket's staging slots,
// with its pattern and key hash.  A round of kBlock * kLTile strings counts
// its strings per bucket in LDS and reserves each bucket's slots with one
// global add (buckets up to kLAggMax; beyond, one global add per string).
template <int WW>
struct ScatterSh {
  uint64_t px[kLayerMaxRot][WW], pz[kLayerMaxRot][WW];
  uint32_t cnt[kLAggMax];
};

// The op's rotation strings into LDS (the caller synchronises before use).
template <int WW, int NT>
__device__ __forceinline__ void load_rot_strings(const Op& op, uint64_t (*px)[WW],
                                                 uint64_t (*pz)[WW]) {
  for (uint32_t g = threadIdx.x; g < op.nrot; g += NT) {
#pragma unroll
    for (int w = 0; w < WW; ++w) {
      px[g][w] = rot_word(op.table, g * kLayerRec + w);
      pz[g][w] = rot_word(op.table, g * kLayerRec + kMaxW + w);
    }
  }
}

// Round t (kBlock * kLTile entries from t * kBlock * kLTile) of one
// instance's scatter; M = the entries scattered (0 for a forced failure),
// bits = the op's bucket bits.  Returns true if a bucket's staging slots
// overflowed.  Every thread of the block calls it (barriers inside).
template <int WW>
__device__ __forceinline__ bool scatter_round(const InstBuf& b, const InstDyn& d, const Op& op,
                                              uint32_t M, uint32_t bits, uint32_t t,
                                              ScatterSh<WW>& sh) {
  const uint32_t r = op.nrot;
  const uint32_t P = 1u << bits, slots = b.lslots >> bits, L = b.lslots;
  const bool agg = P <= (uint32_t)kLAggMax;
  const View v = view_of(b, d);
  const uint32_t round = kBlock * kLTile;
  bool over = false;
  if (agg) {
    __syncthreads();
    for (uint32_t k = threadIdx.x; k < P; k += kBlock) sh.cnt[k] = 0;
  }
  __syncthreads();                         // rotations loaded, counts zero
  uint64_t x[kLTile][WW], z[kLTile][WW], a[kLTile];
  double c[kLTile];
  uint32_t bk[kLTile], rank[kLTile];
  bool has[kLTile];
#pragma unroll
  for (int k = 0; k < kLTile; ++k) {
    const uint32_t i = t * round + k * kBlock + threadIdx.x;
    has[k] = i < M && v.al[i];
    if (!has[k]) continue;
#pragma unroll
    for (int w = 0; w < WW; ++w) {
      x[k][w] = v.X[(size_t)w * v.cap + i];
      z[k][w] = v.Z[(size_t)w * v.cap + i];
    }
    c[k] = v.getc(i);
    const uint64_t h = layer_key<WW>(x[k], z[k], r, sh.px, sh.pz, &a[k]);
    bk[k] = bits ? (uint32_t)(h >> (64 - bits)) : 0u;
    rank[k] = agg ? atomicAdd(&sh.cnt[bk[k]], 1u) : atomicAdd(&b.lcount[bk[k]], 1u);
  }
  if (agg) {
    __syncthreads();
    for (uint32_t k = threadIdx.x; k < P; k += kBlock) {
      const uint32_t n = sh.cnt[k];
      sh.cnt[k] = n ? atomicAdd(&b.lcount[k], n) : 0u;   // this round's first slot
    }
    __syncthreads();
  }
#pragma unroll
  for (int k = 0; k < kLTile; ++k) {
    if (!has[k]) continue;
    const uint32_t rk = agg ? sh.cnt[bk[k]] + rank[k] : rank[k];
    if (rk >= slots) { over = true; continue; }
    const size_t pos = (size_t)bk[k] * slots + rk;
#pragma unroll
    for (int w = 0; w < WW; ++w) {
      b.lstx[(size_t)w * L + pos] = x[k][w];
      b.lstz[(size_t)w * L + pos] = z[k][w];
    }
    b.lstc[pos] = c[k];
    b.lsta[pos] = a[k];
  }
  return over;
}

template <int WW>
__global__ __launch_bounds__(kBlock) void k_layer_scatter(Solo S) {
  __shared__ ScatterSh<WW> sh;
  const InstBuf& b = S.b;
  InstDyn& d = *S.d;
  if (d.pc != S.k) return;                 // an earlier op did not complete
  const Op& op = b.prog[S.k];
  load_rot_strings<WW, kBlock>(op, sh.px, sh.pz);
  const uint32_t M = op.fail_test ? 0u : d.M;
  const uint32_t bits = layer_bits(d.M, d.lboost, b.lmaxbits, b.lshift);
  bool over = op.fail_test != 0 && blockIdx.x == 0 && threadIdx.x == 0;
  const uint32_t rounds = (M + kBlock * kLTile - 1) / (kBlock * kLTile);
  for (uint32_t t = blockIdx.x; t < rounds; t += gridDim.x)
    over = scatter_round<WW>(b, d, op, M, bits, t, sh) || over;
  if (over) atomicOr(&d.lfail, 1u);        // a bucket's staging slots overflowed
}

// Exact placement (one-instance path, once a bucket's staging slots have
// overflowed on the handle): closed sets of thousands of strings do not fit
// equal shares of the staging, so the strings are counted first.
// k_layer_rank computes every string's pattern, bucket and rank in it (the
// count kernel's LDS counts and one global add per block and bucket, as the
// scatter does) and its last block turns the counts into bucket bases;
// k_layer_place moves the strings to base + rank.  One launch more than the
// scatter, ~15 us at 10^6 strings, where a failed op's gate launches cost ms.
template <int WW>
__global__ __launch_bounds__(kBlock) void k_layer_rank(Solo S) {
  __shared__ ScatterSh<WW> sh;
  __shared__ uint32_t s_tmp[kWaves + 1], s_flag;
  const InstBuf& b = S.b;
  InstDyn& d = *S.d;
  if (d.pc != S.k) return;                 // an earlier op did not complete
  const Op& op = b.prog[S.k];
  load_rot_strings<WW, kBlock>(op, sh.px, sh.pz);
  const uint32_t M = op.fail_test ? 0u : d.M;
  const uint32_t bits = layer_bits(d.M, d.lboost, b.lmaxbits, b.lshift), P = 1u << bits;
  const bool agg = P <= (uint32_t)kLAggMax;
  const uint32_t rounds = (M + kBlock - 1) / kBlock, workers = worker_count(rounds);
  if (blockIdx.x >= workers) return;
  const View v = view_of(b, d);
  for (uint32_t t = blockIdx.x; t < rounds; t += gridDim.x) {
    __syncthreads();
    if (agg)
      for (uint32_t k = threadIdx.x; k < P; k += kBlock) sh.cnt[k] = 0;
    __syncthreads();                       // rotations loaded, counts zero
    const uint32_t i = t * kBlock + threadIdx.x;
    const bool has = i < M && v.al[i];
    uint32_t bk = kNone32, rank = 0;
    if (has) {
      uint64_t x[WW], z[WW], a;
#pragma unroll
      for (int w = 0; w < WW; ++w) {
        x[w] = v.X[(size_t)w * v.cap + i];
        z[w] = v.Z[(size_t)w * v.cap + i];
      }
      const uint64_t h = layer_key<WW>(x, z, op.nrot, sh.px, sh.pz, &a);
      bk = bits ? (uint32_t)(h >> (64 - bits)) : 0u;
      rank = agg ? atomicAdd(&sh.cnt[bk], 1u) : atomicAdd(&b.lcount[bk], 1u);
      b.lpat[i] = a;
    }
    if (agg) {
      __syncthreads();
      for (uint32_t k = threadIdx.x; k < P; k += kBlock) {
        const uint32_t n = sh.cnt[k];
        sh.cnt[k] = n ? atomicAdd(&b.lcount[k], n) : 0u;
      }
      __syncthreads();
      if (has) rank += sh.cnt[bk];
    }
    if (i < M) b.lbk[i] = bk;
    if (has) b.lrank[i] = rank;
  }
  if (!last_block(S.sync, &s_flag, workers)) return;
  __syncthreads();
  uint32_t carry = 0;                      // the last block: bucket bases
  for (uint32_t k0 = 0; k0 < P; k0 += kBlock) {
    const uint32_t k = k0 + threadIdx.x, n = k < P ? ld_agent(&b.lcount[k]) : 0u;
    uint32_t total;
    const uint32_t off = block_scan(n, s_tmp, &total);
    if (k < P) b.lbase[k] = carry + off;
    carry += total;
  }
  if (threadIdx.x == 0 && op.fail_test) atomicOr(&d.lfail, 1u);
}

template <int WW>
__global__ __launch_bounds__(kBlock) void k_layer_place(Solo S) {
  const InstBuf& b = S.b;
  InstDyn& d = *S.d;
  if (d.pc != S.k) return;
  const uint32_t M = b.prog[S.k].fail_test ? 0u : d.M, L = b.lslots;
  const View v = view_of(b, d);
  for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < M; i += gridDim.x * kBlock) {
    const uint32_t bk = b.lbk[i];
    if (bk == kNone32) continue;
    const uint32_t pos = b.lbase[bk] + b.lrank[i];   // < the live strings <= lslots
#pragma unroll
    for (int w = 0; w < WW; ++w) {
      b.lstx[(size_t)w * L + pos] = v.X[(size_t)w * v.cap + i];
      b.lstz[(size_t)w * L + pos] = v.Z[(size_t)w * v.cap + i];
    }
    b.lstc[pos] = v.getc(i);
    b.lsta[pos] = b.lpat[i];
  }
}

// An instance of a batch takes the layer op when it stands at one with
// staging, its key width matches the kernel's and nothing stopped it.
template <int WW>
__device__ __forceinline__ bool layer_served(const InstBuf& b, const InstDyn& d) {
  const Op* op = cur_op(b, d);
  return op && op->type == OP_LAYER && b.W == WW && b.lcount && !b.nolayer &&
         !(d.status & ST_OVERFLOW);
}

// Batched form, step 1: every instance that stands at a layer op scatters;
// rounds of all instances are dealt out to the blocks.  Block 0 records in
// each instance whether this step serves it (d.lserved, read by step 2).
template <int WW>
__global__ __launch_bounds__(kBlock) void k_layer_scatter_multi(Ctx C) {
  __shared__ uint32_t s_pref[kMaxInst];
  __shared__ uint32_t s_tmp[kWaves + 1];
  __shared__ ScatterSh<WW> sh;
  const int ninst = *C.ninst;
  const uint32_t round = kBlock * kLTile;
  const uint32_t total = plan_tiles(ninst, [&](int i) -> uint32_t {
    const InstBuf& b = *C.bufs[i];
    const InstDyn& d = *C.dyns[i];
    if (!layer_served<WW>(b, d)) return 0u;
    const uint32_t M = b.prog[d.pc].fail_test ? 0u : d.M;
    return M ? (M + round - 1) / round : 1u;   // a forced failure takes one empty round
  }, s_pref, s_tmp);
  if (blockIdx.x == 0)
    for (int i = threadIdx.x; i < ninst; i += kBlock)
      if (C.bufs[i]->W == WW) C.dyns[i]->lserved = layer_served<WW>(*C.bufs[i], *C.dyns[i]) ? 1u : 0u;
  int cur = -1;
  for (uint32_t t = blockIdx.x; t < total; t += gridDim.x) {
    const int i = find_inst(s_pref, ninst, t);
    const InstBuf& b = *C.bufs[i];
    InstDyn& d = *C.dyns[i];
    const Op& op = b.prog[d.pc];
    if (i != cur) {
      __syncthreads();                     // the last round's rotations are read
      load_rot_strings<WW, kBlock>(op, sh.px, sh.pz);
      cur = i;
    }
    const uint32_t M = op.fail_test ? 0u : d.M;
    const uint32_t bits = layer_bits(d.M, d.lboost, b.lmaxbits, b.lshift);
    const bool over = scatter_round<WW>(b, d, op, M, bits, t - s_pref[i], sh) ||
                      (op.fail_test != 0 && t == s_pref[i] && threadIdx.x == 0);
    if (over) atomicOr(&d.lfail, 1u);      // a bucket's staging slots overflowed
  }
}

// String arithmetic on KW key words (layer_key_words).
template <int KW>
__device__ __forceinline__ void lk_pack(const uint64_t* x, const uint64_t* z, uint64_t* k) {
  if constexpr (KW == 1) {
    k[0] = x[0] | (z[0] << 32);
  } else {
#pragma unroll
    for (int w = 0; w < KW / 2; ++w) { k[w] = x[w]; k[KW / 2 + w] = z[w]; }
  }
}

template <int KW>
__device__ __forceinline__ void lk_unpack(const uint64_t* k, uint64_t* x, uint64_t* z) {
  if constexpr (KW == 1) {
    x[0] = (uint32_t)k[0];
    z[0] = k[0] >> 32;
  } else {
#pragma unroll
    for (int w = 0; w < KW / 2; ++w) { x[w] = k[w]; z[w] = k[KW / 2 + w]; }
  }
}

// (x, z) swapped: Q anticommutes with P iff popc(Q & swapped(P)) is odd
template <int KW>
__device__ __forceinline__ bool lk_anti(const uint64_t* q, const uint64_t* p) {
  uint32_t par = 0;
  if constexpr (KW == 1) {
    par = __popcll(q[0] & ((p[0] << 32) | (p[0] >> 32)));
  } else {
#pragma unroll
    for (int w = 0; w < KW; ++w) par += __popcll(q[w] & p[(w + KW / 2) % KW]);
  }
  return par & 1u;
}

template <int KW>
__device__ __forceinline__ int lk_sign(const uint64_t* p, const uint64_t* q, const uint64_t* r) {
  if constexpr (KW == 1) {
    const uint32_t px = (uint32_t)p[0], pz = (uint32_t)(p[0] >> 32);
    const uint32_t qx = (uint32_t)q[0], qz = (uint32_t)(q[0] >> 32);
    const uint32_t rx = (uint32_t)r[0], rz = (uint32_t)(r[0] >> 32);
    const int phi = __popc(px & pz) + __popc(qx & qz) + 2 * __popc(pz & qx) - __popc(rx & rz);
    return ((phi & 3) == 3) ? 1 : -1;
  } else {
    constexpr int W = KW / 2;
    return product_sign(p, p + W, q, q + W, r, r + W, W);
  }
}

template <int KW>
__device__ __forceinline__ bool lk_heavy(const uint64_t* k, int wmax) {
  if (wmax < 0) return false;
  int n = 0;
  if constexpr (KW == 1) {
    n = __popc((uint32_t)k[0] | (uint32_t)(k[0] >> 32));
  } else {
#pragma unroll
    for (int w = 0; w < KW / 2; ++w) n += __popcll(k[w] | k[KW / 2 + w]);
  }
  return n > wmax;
}

// 32-bit hash of a key: one 32-bit product per half word (a 64-bit product
// takes four).  A hash linear over GF(2), which would give a partner's slot
// by one xor, maps some closed sets onto few slots: measured up to 20 times
// slower steps.
template <int KW>
__device__ __forceinline__ uint32_t lk_hash(const uint64_t* k) {
  uint32_t h = 0;
#pragma unroll
  for (int w = 0; w < KW; ++w) {
    h = (h ^ (uint32_t)k[w]) * 0x9e3779b1u;
    h ^= h >> 16;
    h = (h ^ (uint32_t)(k[w] >> 32)) * 0x85ebca77u;
    h ^= h >> 15;
  }
  return h;
}

// The bucket's hash table: open addressing, linear probing, 32-bit entries: a
// string's index + 1 in the low IB bits (0: empty) and the hash's low bits
// as a tag above, so that a probe of another string's slot hardly ever costs
// a key compare.  At most 4/7 full.
template <int CAP>
struct LdsTab {
  static constexpr int HB = 32 - __builtin_clz(CAP + CAP / 2 + CAP / 4 - 1), HS = 1 << HB;
  static constexpr int IB = HB;            // CAP < 2^IB
  static_assert(4 * HS >= 7 * CAP && CAP < (1 << IB), "at most 4/7 full");
  __device__ __forceinline__ static uint32_t slot(uint32_t h) { return h >> (32 - HB); }
  __device__ __forceinline__ static uint32_t tagged(uint32_t h) { return h << IB; }
  __device__ __forceinline__ static bool tag_is(uint32_t e, uint32_t tg) {
    return ((e ^ tg) >> IB) == 0;
  }
  __device__ __forceinline__ static uint32_t index(uint32_t e) {
    return (e & ((1u << IB) - 1)) - 1;
  }
  // an atomic load, which stays a DS instruction (a volatile one goes
  // through a generic pointer as a FLAT load, several times the latency)
  __device__ __forceinline__ static uint32_t entry(const uint32_t* tab, uint32_t sl) {
    return __hip_atomic_load(&tab[sl], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  // publishes index j under hash h from slot sl on
  __device__ __forceinline__ static void insert(uint32_t* tab, uint32_t h, uint32_t j,
                                                uint32_t sl) {
    const uint32_t e = tagged(h) | (j + 1);
#pragma unroll 1
    for (int probe = 0; probe < HS; ++probe) {
      if (atomicCAS(&tab[sl], 0u, e) == 0u) return;
      sl = (sl + 1) & (HS - 1);
    }
  }
};

// Sum over the wave, valid in lane 63 (data-parallel primitives: shifts
// within rows of 16 lanes, then row broadcasts; no LDS round trips).
__device__ __forceinline__ uint32_t wave_sum63(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, true);   // row_shr:1
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, true);   // row_shr:2
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, true);   // row_shr:4
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, true);   // row_shr:8
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);  // row_bcast:15
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);  // row_bcast:31
  return v;
}

// Maximum over the wave, valid in lane 63 (as wave_sum63).
__device__ __forceinline__ uint32_t wave_max63(uint32_t v) {
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, true));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, true));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, true));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, true));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false));
  return v;
}

// Exclusive scan of one value per thread over a block of NW waves; *total
// = block sum.  s_tmp needs NW + 1 entries.  Contains __syncthreads.
template <int NW>
__device__ __forceinline__ uint32_t block_scan_n(uint32_t v, uint32_t* s_tmp, uint32_t* total) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  uint32_t x = v;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) s_tmp[wid] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t acc = 0;
    for (int w = 0; w < NW; ++w) { const uint32_t t = s_tmp[w]; s_tmp[w] = acc; acc += t; }
    s_tmp[NW] = acc;
  }
  __syncthreads();
  const uint32_t r = x - v + s_tmp[wid];
  *total = s_tmp[NW];
  __syncthreads();
  return r;
}

// What the apply step reads of its op.
struct LayerArgs {
  const double* table;
  double eps;
  uint64_t nx[kMaxW], nz[kMaxW];
  uint32_t nrot;
  int wmax;
  bool full, has_next;
};

__device__ __forceinline__ LayerArgs layer_args(const Op& op) {
  LayerArgs a;
  a.table = op.table;
  a.eps = op.eps;
#pragma unroll
  for (int w = 0; w < kMaxW; ++w) { a.nx[w] = op.nx[w]; a.nz[w] = op.nz[w]; }
  a.nrot = op.nrot;
  a.wmax = op.wmax;
  a.full = op.full_check != 0;
  a.has_next = op.next_gate != kNone32;
  return a;
}

// rotate_pair (pair) or rotate_single with the child as *nr, by selects: the
// same products, sums and roundings.
__device__ __forceinline__ void rotate_any(bool f32, double cs, double sn, int sig, bool pair,
                                           double cq, double cr, double* nq, double* nr) {
  if (f32) {
    const float c = (float)cs, s = (float)sn, q = (float)cq, r = (float)cr;
    const float aq = c * q, bq = s * r, ar = c * r, br = s * q;
    const float sbq = sig > 0 ? -bq : bq, sbr = sig > 0 ? br : -br;
    *nq = (double)(pair ? aq + sbq : aq);
    *nr = (double)(pair ? ar + sbr : sbr);
  } else {
    const double aq = cs * cq, bq = sn * cr, ar = cs * cr, br = sn * cq;
    const double sbq = sig > 0 ? -bq : bq, sbr = sig > 0 ? br : -br;
    *nq = pair ? aq + sbq : aq;
    *nr = pair ? ar + sbr : sbr;
  }
}

// The bucket's survivors (of its ng strings) to the other half of the store
// (one atomic per block and bucket).  No gate-table entries: inserting the
// next generation's entries takes over slots of the current one, which the
// op's gate copies still need if a bucket elsewhere does not fit.
// layer_finish marks the table stale and the OP_COUNT in front of the next
// gates enters the set.
template <int KW, int NB, int CAP>
__device__ __forceinline__ void emit_survivors(const InstBuf& b, InstDyn& d, const LayerArgs& op,
                                               const uint64_t (*sk)[CAP], const double* sc,
                                               const uint16_t* life, uint32_t ng, uint32_t* s_tmp,
                                               uint32_t* s_base, uint32_t* out, uint32_t* next) {
  constexpr int NW = NB / 64, WW = KW == 1 ? 1 : KW / 2;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  uint32_t wsum = 0;                       // the wave's survivors
#pragma unroll 1
  for (uint32_t j0 = 0; j0 < ng; j0 += NB) {
    const uint32_t j = j0 + threadIdx.x;
    wsum += (uint32_t)__popcll(__ballot(j < ng && (life[j] & 0xFFu) == kAlive));
  }
  if (lane == 0) s_tmp[wid] = wsum;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t total = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) total += s_tmp[w];
    *s_base = total ? atomicAdd(&d.nuniq, total) : 0u;
    *out += total;
  }
  uint32_t off = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) off += w < wid ? s_tmp[w] : 0u;
  __syncthreads();
  uint32_t next_pos = *s_base + off;
  const uint32_t cap = b.cap, ho = d.half ^ 1u;
  const bool has_next = op.has_next;
#pragma unroll 1
  for (uint32_t j0 = 0; j0 < ng; j0 += NB) {
    const uint32_t j = j0 + threadIdx.x;
    const bool al = j < ng && (life[j] & 0xFFu) == kAlive;
    const uint64_t m = __ballot(al);
    const uint32_t pos = next_pos + (uint32_t)__popcll(m & ((1ull << lane) - 1));
    next_pos += (uint32_t)__popcll(m);
    if (!al) continue;
    uint64_t k[KW], x[kMaxW] = {}, z[kMaxW] = {};
#pragma unroll
    for (int w = 0; w < KW; ++w) k[w] = sk[w][j];
    lk_unpack<KW>(k, x, z);
    uint64_t nx[kMaxW] = {}, nz[kMaxW] = {};
#pragma unroll
    for (int w = 0; w < WW; ++w) { nx[w] = op.nx[w]; nz[w] = op.nz[w]; }
    if (has_next && anticommutes(x, z, nx, nz, WW)) ++*next;
    if (pos >= cap) { consume(atomicOr(&d.status, ST_OVERFLOW)); continue; }
#pragma unroll
    for (int w = 0; w < WW; ++w) {
      b.x[ho][(size_t)w * cap + pos] = x[w];
      b.z[ho][(size_t)w * cap + pos] = z[w];
    }
    if (b.f32)
      static_cast<float*>(b.c[ho])[pos] = (float)sc[j];
    else
      static_cast<double*>(b.c[ho])[pos] = sc[j];
    b.alive[ho][0][pos] = 1;
  }
}

// Last block, one thread, with the folded sums t (LayerSums order): on
// success the op's counts, the other half becomes current and pc passes the
// op's fallback copies.
__device__ __forceinline__ void layer_finish(const InstBuf& b, InstDyn& d, const Op& op,
                                             const uint64_t* t, bool batched) {
  const uint32_t out = ld_agent(&d.nuniq), status = ld_agent(&d.status), why = ld_agent(&d.lfail);
  consume((uint64_t)out ^ status ^ why);
  d.nuniq = 0;
  if (status & ST_OVERFLOW) {               // the survivors did not fit: grow, run again
    d.lneed = out;
    d.lfail = 0;
    d.failed_pc = d.pc;
    return;
  }
  if (why) {                                // a bucket did not fit
    d.lfail = 0;
    d.lwhy = why;                           // 1 staging slots, 2 LDS
    d.lfails += 1;
    if (batched) {                          // the batched form runs the gate copies
      d.lfb += 1;
      d.pc += 1;
      return;
    }
    d.status = status | ST_LAYER;           // the one-instance path: the host decides
    d.failed_pc = d.pc;
    return;
  }
  d.lops += 1;
  d.propagated += t[0];
  d.merged += t[0] + t[1];
  d.anti_total += t[1];
  d.key_reads += t[6];                      // each key read once
  d.coef_rw += t[6];                        // each coefficient read and written once
  d.appended += t[4];
  d.M = out;
  d.Mnext = out;
  d.live = out;
  d.count = (uint32_t)t[3];
  const uint64_t held = t[5] > out ? t[5] : out;
  if (held > d.peak) d.peak = held < 0xFFFFFFFFull ? (uint32_t)held : 0xFFFFFFFFu;
  d.half ^= 1u;
  d.parity = 0;
  d.gstale = 1;
  d.count_for = op.next_gate;
  d.pc += 1 + op.skip;
}

// Liveness of a bucket's string: born (the rotation before which it first
// exists: 0, or g + 1 for a child of rotation g) and died (the rotation
// after which it was dropped, kAlive while it lives), packed in 16 bits so
// that one store changes both.  A string is live before rotation g iff
// born <= g <= died.  Rotation g writes `died = g` for strings it drops and
// (g + 1, kAlive) for a dropped string it makes again; a string's own thread
// never reads these mid-rotation values as "live before" wrongly: died = g
// still reads live before g, and born = g + 1 reads not live.
__device__ __forceinline__ bool live_before(uint32_t life, uint32_t g) {
  return (life >> 8) <= g && (life & 0xFFu) >= g;
}
__device__ __forceinline__ uint16_t life_of(uint32_t born, uint32_t died) {
  return (uint16_t)((born << 8) | died);
}

// 2. One block per bucket: the bucket's strings into LDS (one hash table),
// then the rotations some of them anticommute with (and the first one if
// the op re-checks every string there), each over all the bucket's strings
// with a block barrier after it; then the survivors go to the other half.
// Live counts before each rotation follow from the strings entering and the
// births and drops of the rotations before it.
// A bucket's strings: in LDS, or (k_layer_huge) in HBM.
template <int KW, int CAP_>
struct alignas(16) BucketMem {
  static constexpr int CAP = CAP_, HS = LdsTab<CAP>::HS;
  uint64_t k[KW][CAP];
  double c[CAP];
  uint64_t a[CAP];                         // rotations still to run on the string
  uint32_t hash[HS];                       // LdsTab entries
  uint16_t life[CAP];
};

// Buckets that outgrow a block's LDS (at most kHugeList of an op): a list of
// (bucket, strings), then a slab per block of k_layer_huge.
constexpr uint32_t kHugeList = 1024;
constexpr int kHugeBlocks = 64, kHugeBlock = 512, kHugeCap = 32768;
constexpr size_t kHugeListBytes = 2 * sizeof(uint32_t) * kHugeList;
template <int KW> constexpr size_t huge_slab() {
  return (sizeof(BucketMem<KW, kHugeCap>) + 255) / 256 * 256;
}

// What a block keeps in LDS beside its bucket's strings.
template <int KW, int NB>
struct ApplyCtl {
  static constexpr int NW = NB / 64, NS = 7;
  static constexpr int WW = KW == 1 ? 1 : KW / 2;
  static_assert(NB >= kAccShards * 8, "one thread per shard entry (layer_end)");
  struct Rot {
    uint64_t p[KW];
    double cs, sn;
  } rot[kLayerMaxRot];
  uint32_t steps;                          // most rotations any string of the bucket takes
  uint32_t inc[3], fail, flag, tmp[NW + 1], base;
  uint32_t red[NW][NS];
  uint64_t fold[kAccShards][NS + 1];
};

template <int KW, int NB, bool Big = false>
struct ApplySh : ApplyCtl<KW, NB> {
  BucketMem<KW, layer_cap<KW, Big>()> mem;
};


// Per-thread sums of one instance: live before each rotation (as r *
// entering + weighted births - drops), anticommuting, survivors, survivors
// anticommuting with the next gate, children, strings held at the end,
// strings entering; bad: a bucket did not fit the LDS.
constexpr uint32_t kLayerFlush = 128;      // buckets between two flushes of a block's sums
struct LayerSums {
  int32_t lw = 0;
  uint32_t an = 0, out = 0, nx = 0, ch = 0, held = 0, in = 0;
  bool bad = false;
};

template <int KW, int NB>
__device__ __forceinline__ void load_rotations(const double* table, uint32_t nrot,
                                               ApplyCtl<KW, NB>& sh) {
  constexpr int WW = ApplyCtl<KW, NB>::WW;
  for (uint32_t g = threadIdx.x; g < nrot; g += NB) {
    uint64_t x[WW], z[WW], k[KW];
#pragma unroll
    for (int w = 0; w < WW; ++w) {
      x[w] = rot_word(table, g * kLayerRec + w);
      z[w] = rot_word(table, g * kLayerRec + kMaxW + w);
    }
    const double cs = table[g * kLayerRec + 2 * kMaxW], sn = table[g * kLayerRec + 2 * kMaxW + 1];
    lk_pack<KW>(x, z, k);
#pragma unroll
    for (int w = 0; w < KW; ++w) sh.rot[g].p[w] = k[w];
    sh.rot[g].cs = cs;
    sh.rot[g].sn = sn;
  }
}

// Bucket bk of one instance (bits: the op's bucket bits; cnt: its strings),
// with its strings in mm.  Every thread of the block calls it; it starts with
// a barrier (the memory of the previous bucket, and the rotations, are then
// free and loaded).  False if the bucket does not fit mm (uniform).
//
// Step q runs every string's q-th own rotation: the strings of one closed set
// anticommute with the same rotations, so they are at the same one, and sets
// that differ need no common order.  A bucket takes as many steps as the
// string with the most rotations, not as many as the union of all.  Pair and
// single rotation share one path (selects instead of branches): a wave of
// mixed lanes pays each instruction once, and the path's length is what
// bounds the kernel (a step of one wave measured about 5 cycles per
// instruction, LDS round trips included).  The loops over a thread's strings
// stay rolled: a launch starts with a cold instruction cache.
template <int KW, int NB, class Mem>
__device__ __forceinline__ bool apply_bucket(const InstBuf& b, InstDyn& d, const LayerArgs& op,
                                             uint32_t bits, uint32_t bk, uint32_t cnt,
                                             ApplyCtl<KW, NB>& sh, Mem& mm, LayerSums& sum) {
  using Sh = ApplyCtl<KW, NB>;
  constexpr int CAP = Mem::CAP, HS = Mem::HS, WW = Sh::WW;
  using T = LdsTab<CAP>;
  const uint32_t r = op.nrot;
  // (exact placement: the bucket's own base, and no limit but the staging)
  const uint32_t slots = b.lexact ? b.lslots : b.lslots >> bits;
  const size_t base = b.lexact ? (size_t)b.lbase[bk] : (size_t)bk * slots;
  __syncthreads();
  if (threadIdx.x == 0) {
    sh.fail = 0;
    sh.inc[0] = sh.inc[1] = sh.inc[2] = 0;
    sh.steps = 0;
  }
  for (int t = threadIdx.x; t < HS / 4; t += NB)
    reinterpret_cast<uint4*>(mm.hash)[t] = make_uint4(0, 0, 0, 0);
  __syncthreads();
  const uint32_t n0 = __builtin_amdgcn_readfirstlane(cnt < slots ? cnt : slots);
  if (n0 > (uint32_t)CAP) return false;                // uniform
  const double eps = op.eps;
  const int wmax = op.wmax;
  const bool full = op.full, f32 = b.f32 != 0;
  if (threadIdx.x == 0) {
    sum.in += n0;
    sum.lw += (int32_t)(r * n0);
  }
  {
    const size_t L = b.lslots;
    uint32_t most = 0;
#pragma unroll 1
    for (uint32_t j = threadIdx.x; j < n0; j += NB) {
      uint64_t x[WW], z[WW], k[KW];
#pragma unroll
      for (int q = 0; q < WW; ++q) {
        x[q] = b.lstx[(size_t)q * L + base + j];
        z[q] = b.lstz[(size_t)q * L + base + j];
      }
      const double c = b.lstc[base + j];
      const uint64_t a = b.lsta[base + j];
      lk_pack<KW>(x, z, k);
#pragma unroll
      for (int w = 0; w < KW; ++w) mm.k[w][j] = k[w];
      mm.c[j] = c;
      mm.a[j] = a;
      // the op's first rotation re-checks every string: one that commutes
      // with it is checked here and leaves after that rotation
      const bool drop = full && !(a & 1ull) && !(fabs(c) >= eps && !lk_heavy<KW>(k, wmax));
      mm.life[j] = life_of(0, drop ? 0u : kAlive);
      if (drop) sum.lw -= (int32_t)(r - 1);
      const uint32_t h = lk_hash<KW>(k);
      T::insert(mm.hash, h, j, T::slot(h));
      most = max(most, (uint32_t)__popcll(a));
    }
    most = wave_max63(most);
    if ((threadIdx.x & 63) == 63 && most) atomicMax(&sh.steps, most);
  }
  __syncthreads();
  const uint32_t steps = __builtin_amdgcn_readfirstlane(sh.steps);
  uint32_t ng = n0;                        // strings before the step
#pragma unroll 1
  for (uint32_t q = 0; q < steps; ++q) {
    if (threadIdx.x == 0) sh.inc[(q + 1) % 3] = 0;
#pragma unroll 1
    for (uint32_t j = threadIdx.x; j < ng; j += NB) {
      // (a coefficient read here is used only by a string that leads its
      // pair or has none, and no other thread writes those)
      const uint64_t rem = mm.a[j];
      const uint32_t life = mm.life[j];
      const double cq = mm.c[j];
      uint64_t qk[KW], rk[KW];
#pragma unroll
      for (int w = 0; w < KW; ++w) qk[w] = mm.k[w][j];
      if (rem == 0) continue;
      const uint32_t g = (uint32_t)__builtin_ctzll(rem);
      const uint64_t left = rem & (rem - 1);
      mm.a[j] = left;
      if (!live_before(life, g)) continue;
      const typename Sh::Rot rot = sh.rot[g];
#pragma unroll
      for (int w = 0; w < KW; ++w) rk[w] = qk[w] ^ rot.p[w];
      const uint32_t rh = lk_hash<KW>(rk);
      // the partner, its stamp and coefficient (read with the key compare);
      // strings made by this step (index >= ng) are nobody's partner in it
      const uint32_t tg = T::tagged(rh);
      uint32_t sl = T::slot(rh), p = kNone32, plife = 0;
      double cp = 0.0;
#pragma unroll 1
      for (int probe = 0; probe < HS; ++probe) {
        const uint32_t e = T::entry(mm.hash, sl);
        if (e == 0) break;
        if (T::tag_is(e, tg)) {
          const uint32_t m = T::index(e);
          bool eq = m < ng;
#pragma unroll
          for (int w = 0; w < KW; ++w) eq = eq & (mm.k[w][m] == rk[w]);
          plife = mm.life[m];
          cp = mm.c[m];
          if (eq) { p = m; break; }
        }
        sl = (sl + 1) & (HS - 1);
      }
      ++sum.an;
      const bool found = p != kNone32;
      const bool plive = found && live_before(plife, g);
      if (plive && p < j) continue;        // the partner's thread leads
      const bool chk = g == 0 && full;
      const int sig = lk_sign<KW>(rot.p, qk, rk);   // i P Q = sig R
      double nq, nr;                       // Q, and R = PQ: the pair's or the child's
      rotate_any(f32, rot.cs, rot.sn, sig, plive, cq, cp, &nq, &nr);
      const bool keep_q = fabs(nq) >= eps && !(chk && lk_heavy<KW>(qk, wmax));
      const bool keep_r = fabs(nr) >= eps && !((chk || !plive) && lk_heavy<KW>(rk, wmax));
      const bool born = keep_r && !plive;  // a new string, or a dropped one again
      // live counts before the later rotations of the op (wt of them)
      sum.lw += (int32_t)(r - 1 - g) *
                ((born ? 1 : 0) - (keep_q ? 0 : 1) - (plive && !keep_r ? 1 : 0));
      sum.ch += born ? 1u : 0u;
      mm.c[j] = nq;
      if (!keep_q) mm.life[j] = life_of(life >> 8, g);
      if (!found && born) {
        p = ng + atomicAdd(&sh.inc[q % 3], 1u);
        if (p < (uint32_t)CAP) {
#pragma unroll
          for (int w = 0; w < KW; ++w) mm.k[w][p] = rk[w];
          mm.a[p] = left;
          T::insert(mm.hash, rh, p, sl);
        } else {
          sh.fail = 1;
          p = kNone32;
        }
      }
      if (p != kNone32 && (plive || born)) {
        mm.c[p] = nr;
        if (born)
          mm.life[p] = life_of(g + 1, kAlive);
        else if (!keep_r)
          mm.life[p] = life_of(plife >> 8, g);
      }
    }
    __syncthreads();
    const uint32_t add = __builtin_amdgcn_readfirstlane(sh.inc[q % 3]);
    ng = ng + add < (uint32_t)CAP ? ng + add : (uint32_t)CAP;
  }
  if (threadIdx.x == 0) sum.held += ng;
  if (sh.fail) return false;               // uniform: read after the last barrier
  emit_survivors<KW, NB, CAP>(b, d, op, mm.k, mm.c, mm.life, ng, sh.tmp, &sh.base, &sum.out,
                              &sum.nx);
  return true;
}

// apply_bucket from the block's LDS; a bucket that outgrows it goes on the list
// of k_layer_huge (its sums undone; its strings are still staged) or, without
// one, fails the op.
template <int KW, int NB, bool Big>
__device__ __forceinline__ void apply_or_list(const InstBuf& b, InstDyn& d, const LayerArgs& op,
                                              uint32_t bits, uint32_t bk, ApplySh<KW, NB, Big>& sh,
                                              LayerSums& sum, char* huge) {
  const uint32_t cnt = b.lcount[bk];
  const LayerSums before = sum;
  const bool ok = apply_bucket<KW, NB>(b, d, op, bits, bk, cnt, sh, sh.mem, sum);
  // (every thread has read the count: apply_bucket has barriers)
  if (threadIdx.x == 0) b.lcount[bk] = 0;  // zero for the next layer op
  if (ok) return;
  sum = before;
  if (!huge) {
    sum.bad = true;
    return;
  }
  if (threadIdx.x == 0) {
    const uint32_t e = atomicAdd(&d.lnhuge, 1u);
    uint32_t* list = reinterpret_cast<uint32_t*>(huge);
    if (e < kHugeList) {
      list[2 * e] = bk;
      list[2 * e + 1] = cnt;
    } else {
      consume(atomicOr(&d.lfail, 2u));     // too many of them
    }
  }
}

// The block's sums of one instance to its shard line (entries 1..NS) and
// its LDS overflow flag; resets the sums.  Every thread calls it.  Per block
// and instance every sum is below 2^31 (a block sees at most kLayerMaxRot
// rotations of its buckets' strings).  The atomics have returned when the
// threads leave, so the last block needs no fence to read their totals.
template <int KW, int NB>
__device__ __forceinline__ void flush_sums(const InstBuf& b, InstDyn& d, ApplyCtl<KW, NB>& sh,
                                           LayerSums& sum) {
  constexpr int NS = ApplyCtl<KW, NB>::NS, NW = ApplyCtl<KW, NB>::NW;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const uint32_t v[NS] = {(uint32_t)sum.lw, sum.an, sum.out, sum.nx, sum.ch, sum.held, sum.in};
  __syncthreads();
#pragma unroll
  for (int k = 0; k < NS; ++k) {
    const uint32_t t = wave_sum63(v[k]);
    if (lane == 63) sh.red[wid][k] = t;
  }
  __syncthreads();
  if (threadIdx.x < NS) {
    uint32_t t = 0;
    for (int w = 0; w < NW; ++w) t += sh.red[w][threadIdx.x];
    if (t)
      consume(atomicAdd((unsigned long long*)&b.accs[(blockIdx.x % kAccShards) * kLineU64 + 1 + threadIdx.x],
                        (unsigned long long)(int64_t)(int32_t)t));
  }
  if (threadIdx.x == 0 && sum.bad) consume(atomicOr(&d.lfail, 2u));   // the LDS overflowed
  sum = LayerSums();
}

// Last block of a layer op, every thread: folds the shard lines, one thread per
// entry, and finishes.
template <class Sh>
__device__ __forceinline__ void layer_end(const InstBuf& b, InstDyn& d, const Op& op, Sh& sh) {
  __syncthreads();
  if (threadIdx.x < kAccShards * 8) {
    const uint32_t s = threadIdx.x >> 3, k = threadIdx.x & 7;
    sh.fold[s][k] = k < (uint32_t)Sh::NS
        ? atomicExch((unsigned long long*)&b.accs[s * kLineU64 + 1 + k], 0ull) : 0ull;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t t[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < kAccShards; ++s)
#pragma unroll
      for (int k = 0; k < Sh::NS; ++k) t[k] += sh.fold[s][k];
    layer_finish(b, d, op, t, false);
  }
}

template <int KW, int NB, bool Big>
__global__ __launch_bounds__(NB) void k_layer_apply(Solo S) {
  __shared__ ApplySh<KW, NB, Big> sh;
  const InstBuf& b = S.b;
  InstDyn& d = *S.d;
  const Op& op = b.prog[S.k];              // S.k < prog_len
  // the scatter's failure (bit 0, set before this launch); bit 1 comes from
  // blocks of this launch and must not steer a block's control flow.  The
  // state's and the op's loads are issued together.
  const uint32_t pc = d.pc, M = d.M, lfail = ld_agent(&d.lfail);
  const int32_t lboost = d.lboost;
  const LayerArgs la = layer_args(op);
  consume((uint64_t)pc ^ M ^ lfail ^ (uint32_t)lboost ^ (uint64_t)(uintptr_t)la.table ^ la.nrot);
  if (pc != S.k) return;                   // uniform: pc changes only in the last block
  load_rotations<KW, NB>(la.table, la.nrot, sh);
  const uint32_t bits = layer_bits(M, lboost, b.lmaxbits, b.lshift);
  const bool failed = (lfail & 1u) != 0;
  LayerSums sum;
  uint32_t done = 0;
  for (uint32_t bk = blockIdx.x; bk < (1u << bits); bk += gridDim.x) {
    if (failed) {                          // only zero the counts (uniform)
      if (threadIdx.x == 0) b.lcount[bk] = 0;
      continue;
    }
    apply_or_list<KW, NB, Big>(b, d, la, bits, bk, sh, sum, b.lhuge);
    if (++done % kLayerFlush == 0) flush_sums<KW, NB>(b, d, sh, sum);
  }
  flush_sums<KW, NB>(b, d, sh, sum);
  if (!last_block(S.sync, &sh.flag, gridDim.x, false)) return;
  if (threadIdx.x == 0) {                  // (sh.flag may still be being read)
    const uint32_t n = ld_agent(&d.lnhuge), why = ld_agent(&d.lfail);
    if (why) d.lnhuge = 0;
    sh.base = n && !why ? 1u : 0u;
  }
  __syncthreads();
  if (sh.base) return;                     // k_layer_huge, launched behind this, ends the op
  layer_end(b, d, op, sh);
}

// The buckets that outgrew a block's LDS, a block each, over slabs of HBM (L2,
// mostly: a slab is ~1 MB): an LDS round trip becomes an L2 one, so a bucket
// of 10^4 strings takes some hundred us, where running the sub-layer as gate
// launches for their sake takes milliseconds.  With exact placement, whole
// propagations: Z_32 ring grown to 8x10^6 strings 60 -> 39 ms, untruncated
// 12-qubit Ising ring 27 -> 18 ms (their later sub-layers were gate launches).
template <int KW>
__global__ __launch_bounds__(kHugeBlock) void k_layer_huge(Solo S) {
  __shared__ ApplyCtl<KW, kHugeBlock> sh;
  const InstBuf& b = S.b;
  InstDyn& d = *S.d;
  // nothing listed: the apply step ended the op (well, or with a failure that
  // leaves pc); lnhuge changes only in the last block, when all have read it
  const uint32_t listed = d.lnhuge;
  if (d.pc != S.k || !b.lhuge || !listed) return;
  const Op& op = b.prog[S.k];
  const uint32_t n = listed < kHugeList ? listed : kHugeList;
  const LayerArgs la = layer_args(op);
  load_rotations(la.table, la.nrot, sh);
  const uint32_t bits = layer_bits(d.M, d.lboost, b.lmaxbits, b.lshift);
  const uint32_t* list = reinterpret_cast<const uint32_t*>(b.lhuge);
  auto& mm = *reinterpret_cast<BucketMem<KW, kHugeCap>*>(b.lhuge + kHugeListBytes +
                                                         blockIdx.x * huge_slab<KW>());
  LayerSums sum;
  uint32_t done = 0;
  for (uint32_t e = blockIdx.x; e < n; e += gridDim.x) {
    if (!apply_bucket<KW, kHugeBlock>(b, d, la, bits, list[2 * e], list[2 * e + 1], sh, mm, sum))
      sum.bad = true;
    if (++done % kLayerFlush == 0) flush_sums(b, d, sh, sum);
  }
  flush_sums(b, d, sh, sum);
  if (!last_block(S.sync, &sh.flag, gridDim.x, false)) return;
  if (threadIdx.x == 0) d.lnhuge = 0;
  layer_end(b, d, op, sh);
}
// Block scan for NB-thread blocks over instances (as plan_tiles).
template <int NB, class F>
__device__ __forceinline__ uint32_t plan_tiles_n(int ninst, F tiles, uint32_t* s_pref,
                                                 uint32_t* s_tmp) {
  constexpr int kPer = (kMaxInst + NB - 1) / NB;
  uint32_t loc[kPer];
  uint32_t sum = 0;
  const int base = threadIdx.x * kPer;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int i = base + k;
    loc[k] = (i < ninst) ? tiles(i) : 0u;
    sum += loc[k];
  }
  uint32_t total;
  uint32_t off = block_scan_n<NB / 64>(sum, s_tmp, &total);
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int i = base + k;
    if (i < ninst) s_pref[i] = off;
    off += loc[k];
  }
  __syncthreads();
  return total;
}

// Batched form, step 2: the buckets of every instance whose layer op step 1
// took, dealt out to the blocks; the last block finishes those instances
// (a bucket that did not fit sends the instance to the op's gate copies).
template <int KW, int NB>
__global__ __launch_bounds__(NB) void k_layer_apply_multi(Ctx C) {
  __shared__ uint32_t s_pref[kMaxInst];
  extern __shared__ __align__(16) uint64_t s_layer_dyn[];   // sizeof(ApplySh<KW, NB>) bytes
  ApplySh<KW, NB>& sh = *reinterpret_cast<ApplySh<KW, NB>*>(s_layer_dyn);
  const int ninst = *C.ninst;
  auto served = [&](int i) {
    return C.bufs[i]->W == ApplySh<KW, NB>::WW && ld_agent(&C.dyns[i]->lserved) != 0;
  };
  const uint32_t total = plan_tiles_n<NB>(ninst, [&](int i) -> uint32_t {
    if (!served(i)) return 0u;
    const InstBuf& b = *C.bufs[i];
    const InstDyn& d = *C.dyns[i];
    return 1u << layer_bits(d.M, d.lboost, b.lmaxbits, b.lshift);
  }, s_pref, sh.tmp);
  LayerSums sum;
  LayerArgs la{};
  uint32_t done = 0;
  int cur = -1;
  for (uint32_t t = blockIdx.x; t < total; t += gridDim.x) {
    const int i = find_inst(s_pref, ninst, t);
    const InstBuf& b = *C.bufs[i];
    InstDyn& d = *C.dyns[i];
    const Op& op = b.prog[d.pc];
    if (i != cur) {
      if (cur >= 0) flush_sums<KW, NB>(*C.bufs[cur], *C.dyns[cur], sh, sum);
      __syncthreads();                     // the last bucket's rotations are read
      la = layer_args(op);
      load_rotations<KW, NB>(la.table, la.nrot, sh);
      cur = i;
    }
    const uint32_t bits = layer_bits(d.M, d.lboost, b.lmaxbits, b.lshift);
    const uint32_t bk = t - s_pref[i];
    if (ld_agent(&d.lfail) & 1u) {         // the scatter failed: only zero the counts
      if (threadIdx.x == 0) b.lcount[bk] = 0;
      continue;
    }
    apply_or_list<KW, NB, false>(b, d, la, bits, bk, sh, sum, nullptr);
    if (++done % kLayerFlush == 0) flush_sums<KW, NB>(b, d, sh, sum);
  }
  if (cur >= 0) flush_sums<KW, NB>(*C.bufs[cur], *C.dyns[cur], sh, sum);
  if (!last_block(C.sync, &sh.flag, gridDim.x, true)) return;
  for (int i = threadIdx.x; i < ninst; i += NB) {
    if (!served(i)) continue;
    const InstBuf& b = *C.bufs[i];
    InstDyn& d = *C.dyns[i];
    d.lserved = 0;
    uint64_t t[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int q = 0; q < kAccShards; ++q)
      for (int k = 0; k < ApplySh<KW, NB>::NS; ++k)
        t[k] += atomicExch((unsigned long long*)&b.accs[q * kLineU64 + 1 + k], 0ull);
    layer_finish(b, d, b.prog[d.pc], t, true);
  }
}

}  // namespace pp
