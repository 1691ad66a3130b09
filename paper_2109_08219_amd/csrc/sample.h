// Kernels of the sampled path: top-k and k-selection by a sample's order
// statistics, for the calls where one filter pass and independent bucket
// sorts beat the delegate vector or a digit-by-digit select.
//
//   k_sgather  samples, one per stratum of equal length at a hashed offset;
//              when few of them can matter, each 256 leave only their top 16
//   k_srank    every kept sample's rank among them (all pairs), so the
//              samples come out sorted
//   k_sfilter  one streaming pass: the elements ranked at or above a sample
//              chosen so that at least k elements are, appended to a buffer
//   k_spart    one pass that also groups them into buckets between samples:
//              a workgroup stages candidates in LDS and writes each stage as
//              one row grouped by bucket, with the row's bucket offsets
//   k_sbucket  one workgroup per bucket: gathers its segments of all rows,
//              sorts them in LDS and writes its slots of the output
//
// Elements are compared as composites (encoded key << L) | (2^L - 1 - position)
// with L the bit length of n - 1: larger ranks higher, ties by lower position,
// all distinct, so ties are split between buckets like any other elements
// (ranking by key alone would put a tied key into one bucket whatever its
// count), and a run of ties is dense in composite space, which the linear bins
// of the bucket sort need.
//
// The sample only decides how the work is split.  A sample that misjudges the
// input (fewer than k elements at or above its cut, or more candidates than
// the buffer holds) is noticed from exact counts, and k_sbucket then answers
// from the input itself (rescue).  The window's margin and the buffers' room
// make either rarer than exp(-24) for inputs laid out without regard to the
// sampled positions.
#pragma once

#include "internal.h"
#include "sample_win.h"

namespace drtopk {

typedef unsigned __int128 su128;
typedef uint32_t su32x4 __attribute__((ext_vector_type(4)));

constexpr int kSBins = 2048;
constexpr int kSMaxRows = 1024;      // most rows of the offset table
constexpr int kSPartThreads = 1024;
constexpr int kSBucketThreads = 512;
constexpr int kSRankThreads = 512;
constexpr int kSRankPer = 16;        // samples ranked by one workgroup
constexpr int kSFilterThreads = 1024;
constexpr uint32_t kSCells = 1024;   // cells of k_spart's bucket lookup
constexpr uint32_t kSCrowd = 128;    // elements of a bin that are still ranked one against the other
constexpr uint32_t kSSplit = 256;    // samples of a workgroup's own sort or threshold

template <typename K>
struct STraits;
template <>
struct STraits<uint32_t> {
  typedef uint64_t Comp;
  static constexpr int kStage = 12288;  // candidates staged by a workgroup of k_spart
  static constexpr int kTile = 8192;    // elements it reads at a time
  static constexpr int kCap = 7680;     // elements sorted by a workgroup of k_sbucket (two fit a CU)
  static constexpr int kMaxB = 3072;    // most buckets
  static constexpr int kList = 65536;   // candidates that every bucket's workgroup may read
  static constexpr int kTarget = 2048;  // elements a bucket is planned for
};
template <>
struct STraits<uint64_t> {
  typedef su128 Comp;
  static constexpr int kStage = 6144;
  static constexpr int kTile = 4096;
  static constexpr int kCap = 3584;
  static constexpr int kMaxB = 1536;
  static constexpr int kList = 32768;
  static constexpr int kTarget = 1024;
};

// Runtime key codec: enc(b) = b ^ (sign(b) & a) ^ c (see Codec64).
template <typename K>
struct SCodec {
  K a, c;
};
__device__ __forceinline__ uint32_t ssign(uint32_t b) { return (uint32_t)((int32_t)b >> 31); }
__device__ __forceinline__ uint64_t ssign(uint64_t b) { return (uint64_t)((int64_t)b >> 63); }
template <typename K>
__device__ __forceinline__ K senc(K b, SCodec<K> cd) { return b ^ (ssign(b) & cd.a) ^ cd.c; }
template <typename K>
__device__ __forceinline__ K sdec(K u, SCodec<K> cd) {
  const K x = u ^ cd.c;
  return x ^ (ssign(x) & cd.a);
}

// A value that every lane holds, in scalar registers.
template <typename T>
__device__ __forceinline__ T suniform(T v) {
  uint32_t w[sizeof(T) / 4];
  __builtin_memcpy(w, &v, sizeof(T));
#pragma unroll
  for (uint32_t i = 0; i < sizeof(T) / 4; ++i) w[i] = (uint32_t)__builtin_amdgcn_readfirstlane((int)w[i]);
  __builtin_memcpy(&v, w, sizeof(T));
  return v;
}

__device__ __forceinline__ uint32_t sbits(uint64_t x) { return x ? 64u - (uint32_t)__clzll((long long)x) : 0u; }
__device__ __forceinline__ uint32_t sbits(su128 x) {
  const uint64_t h = (uint64_t)(x >> 64);
  return h ? 64u + sbits(h) : sbits((uint64_t)x);
}

// Composite of (encoded key, position); posmask = 2^L - 1.
template <typename K>
__device__ __forceinline__ typename STraits<K>::Comp scomp(K key, uint32_t pos, int L, uint32_t posmask) {
  return ((typename STraits<K>::Comp)key << L) | (posmask - pos);
}
template <typename C>
__device__ __forceinline__ uint32_t scomp_pos(C c, uint32_t posmask) { return posmask - ((uint32_t)c & posmask); }

struct SCtl {
  uint64_t alloc1;  // level 1 of two: candidates (low word)
  uint64_t pad0[15];
  uint64_t alloc;   // partitioned level: rows << 32 | candidates
  uint64_t pad1[15];
  SWin win;         // window of the partitioned level
  uint32_t rare;    // a bucket kernel without the rare ways met one
  uint32_t pad2[23];
};

struct SRow {
  uint32_t base;   // first candidate of the row
  uint32_t above;  // elements above the window met by the row's workgroup since its previous row
};

__device__ __forceinline__ uint32_t shash(uint32_t x) {
  x = (x ^ (x >> 16)) * 0x7FEB352Du;
  x = (x ^ (x >> 15)) * 0x846CA68Bu;
  return x ^ (x >> 16);
}

// ---------------------------------------------------------------------------
// The stratum of sample i of M = mask + 1 (a power of two): a permutation that
// scatters strata over the workgroups, another one for another salt.
__device__ __forceinline__ uint32_t sscatter(uint32_t i, uint32_t mask, uint32_t salt) {
  i = (i + salt) * 0x9E3779B1u & mask;
  i ^= i >> 7;
  i = i * (salt | 1u) & mask;
  i ^= i >> 9;
  return i * 0x85EBCA6Bu & mask;
}

// Sampling, M samples (a multiple of 256) from a source of at least M elements.
// The sampled places depend on a salt of the process, so no input can be laid
// out to be misjudged (its rescue reads the input many times by few workgroups;
// see sbucket_rare).
// ARR: the source is level 1's candidates (their number is on the device);
// otherwise the input.  TOP: of each 256 samples the 16 largest are kept.  When
// the window's r is a few per workgroup, its top r samples are all kept but
// for odds far below the window's own, and if one is lost the r-th kept sample
// only lies lower: more candidates, never fewer.  So 65536 samples cost one
// gather and the ranks of 4096, and the r-th of 65536 leaves a tenth to a half
// of the candidates that the corresponding sample of 4096 does (n = 2^20, k =
// 1024: 28.6 us a call with 8192 plain samples, 23.9 with these).  Bound by the
// latency of one load from memory and of the count: 4.6 us.
// The launch also clears the state of the kernels after it.
constexpr uint32_t kSKeep = 16;

// With TOP the workgroup has four threads per sample, each counting the larger
// ones in a quarter of the 256.
template <typename K, bool ARR, bool TOP>
__global__ __launch_bounds__(TOP ? 1024 : 256) void k_sgather(const K* __restrict__ keys,
                                                 const typename STraits<K>::Comp* __restrict__ arr, uint64_t n,
                                                 uint32_t cap1, uint32_t k, uint32_t M, uint32_t salt,
                                                 SCodec<K> cd, int L, SWin win, int kth, uint32_t bmax, SCtl* ctl,
                                                 typename STraits<K>::Comp* __restrict__ smp,
                                                 typename STraits<K>::Comp* __restrict__ sorted) {
  typedef typename STraits<K>::Comp C;
  uint32_t i = blockIdx.x * 256 + (threadIdx.x & 255u);
  // neighbouring strata in different workgroups, so that a sorted input's top
  // samples do not meet in one
  if constexpr (TOP) i = sscatter(i, M - 1, salt);
  uint64_t count = n;
  if constexpr (ARR) {
    count = (uint32_t)ctl->alloc1;
    if (count > cap1 || count < k) return;  // level 1 misjudged: the bucket kernel answers from the input
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if constexpr (ARR) {
      SWin w = {};
      sample_window((double)count, (double)k, (double)M, kth != 0, &w);
      sample_buckets((double)count / (double)M, STraits<K>::kTarget, bmax, &w);
      ctl->win = w;
    } else {
      ctl->alloc1 = 0;
      ctl->alloc = 0;
      ctl->rare = 0;
      ctl->win = win;
    }
  }
  const uint32_t posmask = (uint32_t)((1ull << L) - 1);
  C x = 0;
  if (!TOP || threadIdx.x < 256) {
    const uint64_t lo = (uint64_t)i * count / M, hi = (uint64_t)(i + 1) * count / M;
    if (hi > lo) {
      const uint64_t p = lo + (uint64_t)(((uint64_t)shash(i + salt) * (hi - lo)) >> 32);
      if constexpr (ARR) x = arr[p];
      else x = scomp<K>(senc<K>(keys[p], cd), (uint32_t)p, L, posmask);
    }
  }
  if constexpr (ARR) {
    // with fewer elements than samples the empty strata are composites 0,
    // which share one rank: the slots after it hold 0 as well
    sorted[i] = 0;
  }
  if constexpr (!TOP) {
    smp[i] = x;
  } else {
    __shared__ C s[256];
    __shared__ uint32_t part[4][256];
    const uint32_t me = threadIdx.x & 255u, quarter = threadIdx.x >> 8;
    if (threadIdx.x < 256) s[me] = x;
    __syncthreads();
    x = s[me];
    uint32_t rk = 0;
#pragma unroll 16
    for (uint32_t j = 0; j < 64; ++j) rk += s[quarter * 64 + j] > x ? 1u : 0u;
    part[quarter][me] = rk;
    __syncthreads();
    if (threadIdx.x < 256) {
      rk = part[0][me] + part[1][me] + part[2][me] + part[3][me];
      if (rk < kSKeep) smp[blockIdx.x * kSKeep + rk] = x;
    }
  }
}

// All-pairs ranks: a wave holds J * 64 samples in registers and compares them
// with one sample at a time, a scalar operand, so 64 comparisons are one
// vector compare and a scalar bit count.  J * 512 = m samples.  The workgroup's
// own 16 samples reach the scalar side by lane reads: scalar loads in the loop
// had it wait for memory once per four (m = 4096: 6.7 us with 32 samples a
// workgroup, the launch 2 of them; now 4.4, m = 8192 8.5).
template <typename C>
__device__ __forceinline__ C sread_lane(C v, int lane) {
  uint32_t w[sizeof(C) / 4];
  __builtin_memcpy(w, &v, sizeof(C));
#pragma unroll
  for (uint32_t i = 0; i < sizeof(C) / 4; ++i) w[i] = (uint32_t)__builtin_amdgcn_readlane((int)w[i], lane);
  __builtin_memcpy(&v, w, sizeof(C));
  return v;
}

template <typename C, int J>
__global__ __launch_bounds__(kSRankThreads) void k_srank(const C* __restrict__ smp, C* __restrict__ sorted) {
  __shared__ uint32_t cnt[kSRankPer][kSRankThreads / 64];
  const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const uint32_t i0 = blockIdx.x * kSRankPer;
  const C own = smp[i0 + lane % kSRankPer];
  C v[J];
#pragma unroll
  for (int j = 0; j < J; ++j) v[j] = smp[(j * (kSRankThreads / 64) + wave) * 64 + lane];
#pragma unroll
  for (int ii = 0; ii < kSRankPer; ++ii) {
    const C x = sread_lane<C>(own, ii);
    uint32_t c = 0;
#pragma unroll
    for (int j = 0; j < J; ++j) c += (uint32_t)__popcll(__ballot(v[j] > x));
    if (lane == 0) cnt[ii][wave] = c;
  }
  __syncthreads();
  if (threadIdx.x < kSRankPer) {
    uint32_t r = 0;
#pragma unroll
    for (int w = 0; w < kSRankThreads / 64; ++w) r += cnt[threadIdx.x][w];
    sorted[r] = own;
  }
}

// ---------------------------------------------------------------------------
// Streaming filter for one bucket or a first level.  Tiles of U loads per wave
// are dealt to the workgroups in turn, so a dense stretch of candidates
// (sorted input) is shared by many; a wave's next tile is in flight while it
// works on the current one.  A wave keeps its candidates in its own LDS slots
// and its fill level in a register; no barrier before the end, and one device
// atomic a workgroup for what is left then (they are served one at a time,
// 11.5 ns each, hence few large workgroups: two of 1024 threads a CU).  Bound
// by memory from 2^25 keys on (24.5 us, 5.5 TB/s; 2^30: 630 us, 6.8 TB/s, where
// the delegate pass takes 665) and by launch, first load and atomics below
// (2^20: 6.7 us).
// head: keys before the first 16-byte boundary.
template <typename K, int U>
__global__ __launch_bounds__(kSFilterThreads) __attribute__((amdgpu_waves_per_eu(8))) void k_sfilter(
    const K* __restrict__ keys, uint64_t n, uint32_t head, SCodec<K> cd, int L, uint32_t r, uint32_t m,
    const typename STraits<K>::Comp* __restrict__ sorted, uint64_t* alloc,
    typename STraits<K>::Comp* __restrict__ out, uint32_t cap) {
  typedef typename STraits<K>::Comp C;
  constexpr int V = 16 / (int)sizeof(K);  // keys of a 128-bit load
  constexpr uint32_t step = 64 * V;       // keys of a wave's load
  constexpr uint32_t NW = kSFilterThreads / 64, SLOTS = 4096 / sizeof(C);
  __shared__ C stage[NW][SLOTS];
  __shared__ uint32_t s_n[NW];
  __shared__ uint32_t s_base;
  const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  constexpr uint64_t tile = (uint64_t)step * U * NW;
  const uint64_t full = (n - head) / tile;
  su32x4 nx[U];
  auto load = [&](uint64_t tl) {
    if (tl >= full) return;
#pragma unroll
    for (int u = 0; u < U; ++u)
      nx[u] = __builtin_nontemporal_load(
          reinterpret_cast<const su32x4*>(keys + head + tl * tile + (u * NW + wave) * step + lane * V));
  };
  load(blockIdx.x);
  const uint32_t posmask = (uint32_t)((1ull << L) - 1);
  const C t = suniform(r <= m ? sorted[r - 1] : (C)0);
  const K tkey = (K)(t >> L);
  const uint32_t tpos = scomp_pos<C>(t, posmask);
  const K tnext = tkey + 1 ? tkey + 1 : tkey;
  C* st = stage[wave];
  uint32_t fill = 0;
  auto flush = [&]() {
    uint32_t base = 0;
    if (lane == 0) base = (uint32_t)atomicAdd((unsigned long long*)alloc, (unsigned long long)fill);
    base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
    for (uint32_t i = lane; i < fill; i += 64)
      if (base + i < cap && base + i >= base) out[base + i] = st[i];
    fill = 0;
  };
  auto push = [&](bool keep, K key, uint32_t pos) {
    const uint64_t b = __ballot(keep);
    if (b) {
      if (keep) st[fill + mbcnt(b)] = scomp<K>(key, pos, L, posmask);
      fill += (uint32_t)__popcll(b);
    }
  };
  for (uint64_t tl = blockIdx.x; tl < full; tl += gridDim.x) {
    K v[U][V];
#pragma unroll
    for (int u = 0; u < U; ++u) __builtin_memcpy(v[u], &nx[u], 16);
    load(tl + gridDim.x);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      K mx = 0;
#pragma unroll
      for (int c = 0; c < V; ++c) {
        v[u][c] = senc<K>(v[u][c], cd);
        mx = v[u][c] > mx ? v[u][c] : mx;
      }
      // keys equal to the cut's matter up to its position only
      const uint32_t p1 = head + (uint32_t)(tl * tile) + (u * NW + wave) * step, p = p1 + lane * V;
      if (__ballot(mx >= (p1 > tpos ? tnext : tkey))) {
        if (fill + step > SLOTS) flush();
#pragma unroll
        for (int c = 0; c < V; ++c)
          push(v[u][c] > tkey || (v[u][c] == tkey && p + c <= tpos), v[u][c], p + c);
      }
    }
  }
  // the keys the full tiles leave: the ones behind them, 64 a wave, then the head
  const uint64_t rest = full * tile;  // offset from the head
  for (uint64_t q0 = rest + ((uint64_t)blockIdx.x * NW + wave) * 64; q0 < n; q0 += (uint64_t)gridDim.x * NW * 64) {
    if (fill + 64 > SLOTS) flush();
    const uint64_t q = q0 + lane;
    const uint64_t p = q < n - head ? q + head : q - (n - head);
    const K e = q < n ? senc<K>(keys[p], cd) : 0;
    push(q < n && (e > tkey || (e == tkey && (uint32_t)p <= tpos)), e, (uint32_t)p);
  }
  // the waves' remainders leave together
  if (lane == 0) s_n[wave] = fill;
  __syncthreads();
  uint32_t off = 0, tot = 0;
#pragma unroll
  for (uint32_t w = 0; w < NW; ++w) {
    if (w < wave) off += s_n[w];
    tot += s_n[w];
  }
  if (tot == 0) return;
  if (threadIdx.x == 0) s_base = (uint32_t)atomicAdd((unsigned long long*)alloc, (unsigned long long)tot);
  __syncthreads();
  const uint32_t base = s_base + off;
  for (uint32_t i = lane; i < fill; i += 64)
    if (base + i < cap && base + i >= off) out[base + i] = st[i];
}

// ---------------------------------------------------------------------------
// Inclusive prefix sum over the wave by DPP: shifts inside the rows of 16
// lanes, then each row's last lane added to the rows after it.
__device__ __forceinline__ uint32_t swave_scan(uint32_t x) {
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, false);  // row_shr 1, 2, 4, 8
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);  // row_bcast 15: rows 1 and 3
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false);  // row_bcast 31: rows 2 and 3
  return x;
}

// Block-wide exclusive prefix sums of one value per thread (T threads, whole
// waves); *total is the sum.  s_w: T / 64 words.
template <int T>
__device__ __forceinline__ uint32_t sblock_scan(uint32_t x, uint32_t* s_w, uint32_t* total) {
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t y = swave_scan(x);
  __syncthreads();
  if (lane == 63) s_w[wave] = y;
  __syncthreads();
  uint32_t off = 0, tot = 0;
#pragma unroll
  for (uint32_t w = 0; w < T / 64; ++w) {
    const uint32_t q = s_w[w];
    if (w < wave) off += q;
    tot += q;
  }
  *total = tot;
  return off + y - x;
}

// The same with two more values, of which only the sums are wanted.
template <int T>
__device__ __forceinline__ void sblock_scan3(uint32_t x, uint32_t a, uint32_t b, uint32_t (*s_w)[3], uint32_t* ex,
                                             uint32_t* tx, uint32_t* ta, uint32_t* tb) {
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t y = swave_scan(x);
  a = swave_scan(a);
  b = swave_scan(b);
  if (lane == 63) {
    s_w[wave][0] = y;
    s_w[wave][1] = a;
    s_w[wave][2] = b;
  }
  __syncthreads();
  uint32_t off = 0, sx = 0, sa = 0, sb = 0;
#pragma unroll
  for (uint32_t w = 0; w < T / 64; ++w) {
    if (w < wave) off += s_w[w][0];
    sx += s_w[w][0];
    sa += s_w[w][1];
    sb += s_w[w][2];
  }
  *ex = off + y - x;
  *tx = sx;
  *ta = sa;
  *tb = sb;
}

// Lower bounds of the window's buckets, highest first, from the sorted samples
// (thread t of T).
template <typename C>
__device__ __forceinline__ void sfill_splitters(C* split, const SWin& w, uint32_t m, const C* __restrict__ sorted,
                                                uint32_t t, uint32_t T) {
  if (!w.P) {
    for (uint32_t b = t; b < w.B; b += T) {
      uint32_t q = w.a + (b + 1) * w.s;
      if (q > w.r) q = w.r;
      split[b] = q <= m ? sorted[q - 1] : (C)0;
    }
    return;
  }
  const uint32_t q0 = w.a ? w.a : 1u, top = w.a ? 0u : kSTop;
  const uint32_t lgP = 31u - (uint32_t)__clz((int)w.P), thin = w.a ? 0u : kSThin, cuts = w.P2 - 1;
  const uint32_t lgP2 = 31u - (uint32_t)__clz((int)w.P2);
  auto sample = [&](uint32_t q) { return q <= m ? sorted[q - 1] : (C)0; };
  const uint32_t nthin = thin < w.s ? thin : w.s, per = thin_splits(w.P2);
  // thin groups, a thread a splitter: its slot is the number of samples and
  // cuts above it
  for (uint32_t i = t; i < nthin * per; i += T) {
    const uint32_t g = i / per, j = i % per;
    const uint32_t qa = q0 + g * kSGroup, qb = qa + kSGroup < w.r ? qa + kSGroup : w.r;
    const C x0 = sample(qa), step = (x0 - sample(qb)) >> lgP2;
    C v;
    uint32_t slot;
    if (j < cuts) {
      v = x0 - step * (j + 1);
      slot = j;
      for (uint32_t q = qa + 1; q <= qa + kSGroup; ++q) slot += sample(q < qb ? q : qb) >= v ? 1u : 0u;
    } else {
      const uint32_t q = qa + 1 + (j - cuts);
      v = sample(q < qb ? q : qb);
      slot = j - cuts;
      for (uint32_t f = 1; f <= cuts; ++f) slot += x0 - step * f > v ? 1u : 0u;
    }
    split[top + g * per + slot] = v;
  }
  for (uint32_t g = nthin + t; g < w.s; g += T) {
    const uint32_t qa = q0 + g * kSGroup, qb = qa + kSGroup < w.r ? qa + kSGroup : w.r;
    C x[kSGroup + 1];
#pragma unroll
    for (uint32_t i = 0; i <= kSGroup; ++i) x[i] = sample(qa + i < qb ? qa + i : qb);
    const C step = (x[0] - x[kSGroup]) >> lgP;
    C* const out = split + top + nthin * per + (g - nthin) * w.P;
    // Seven samples in a quarter of a part's width: the keys are clustered here,
    // and the samples divide them better.  In one part's width: they may be, or
    // the keys are even and the samples met by chance (7 to 37% of calls on normal
    // keys had a group that did; between its samples a bucket then often held
    // more than a workgroup sorts).  Where that would leave buckets of single
    // gaps, twice as wide parts and every second sample divide the keys together,
    // at most two parts and two gaps whichever it is; else the parts do.
    C least = ~(C)0;  // width of seven samples
#pragma unroll
    for (uint32_t i = 0; i + 6 <= kSGroup; ++i)
      if (qa + i + 6 <= qb && x[i] - x[i + 6] < least) least = x[i] - x[i + 6];
    const bool tight = least < (step >> 2);
    for (uint32_t f = 1; f < w.P; ++f) out[f - 1] = x[0] - step * f;
    if (least < step && !tight && w.P >= kSGroup) {
      const uint32_t half = w.P >> 1;
      for (uint32_t f = 1; f < half; ++f) {
        const C v = x[0] - step * (2 * f);
        uint32_t slot = f - 1;
#pragma unroll
        for (uint32_t i = 2; i <= kSGroup; i += 2) slot += x[i] >= v ? 1u : 0u;
        out[slot] = v;
      }
#pragma unroll
      for (uint32_t i = 2; i <= kSGroup; i += 2) {
        uint32_t slot = i / 2 - 1;
        for (uint32_t f = 1; f < half; ++f) slot += x[0] - step * (2 * f) > x[i] ? 1u : 0u;
        out[slot] = x[i];
      }
      for (uint32_t f = half - 1 + kSGroup / 2; f < w.P; ++f) out[f] = x[kSGroup];
    } else if (tight) {
      if (w.P >= kSGroup) {  // as many equal pieces of each gap as there are bounds
        const uint32_t lgq = lgP - 4, q = 1u << lgq;
#pragma unroll
        for (uint32_t i = 1; i <= kSGroup; ++i) {
          const C piece = (x[i - 1] - x[i]) >> lgq;
          for (uint32_t f = 1; f < q; ++f) out[(i - 1) * q + f - 1] = x[i - 1] - piece * f;
          out[i * q - 1] = x[i];
        }
      } else {
#pragma unroll
        for (uint32_t i = 1; i <= kSGroup; ++i)
          if (((i << lgP) & (kSGroup - 1)) == 0) out[(i << lgP) / kSGroup - 1] = x[i];
      }
    }
    out[w.P - 1] = x[kSGroup];
  }
  if (top && t < kSTop) {
    // above the first sample, by the spacing of the samples after it
    const uint32_t q = q0 + 7 < w.r ? q0 + 7 : w.r;
    const C s0 = sorted[q0 - 1], u = (s0 - (q <= m ? sorted[q - 1] : (C)0)) >> 2;
    const uint32_t f = t == 0 ? 16u : t == 1 ? 8u : t == 2 ? 6u : t == 3 ? 4u : 7u - t;
    const C d = u > (~(C)0 >> 4) ? ~(C)0 : u * f;
    split[t] = s0 + d < s0 ? ~(C)0 : s0 + d;
  }
}

// Staged candidates: key and position (composites are made when the stage is
// written), or composites when the source holds them; then the row, composites
// in bucket order.  64 slots more take what the lanes do not keep, so a put
// needs no branch.
template <typename K, bool ARR, int ST>
struct SStage {
  typedef typename STraits<K>::Comp C;
  union {
    struct {
      K key[ST + 64];
      uint32_t pos[ST + 64];
    };
    C row[ST];
  };
  __device__ __forceinline__ void put(uint32_t i, K v, uint32_t p) {
    key[i] = v;
    pos[i] = p;
  }
  __device__ __forceinline__ C get(uint32_t i, int L, uint32_t posmask) const {
    return scomp<K>(key[i], pos[i], L, posmask);
  }
};
template <typename K, int ST>
struct SStage<K, true, ST> {
  typedef typename STraits<K>::Comp C;
  C row[ST + 64];
  __device__ __forceinline__ void put(uint32_t i, C v, uint32_t) { row[i] = v; }
  __device__ __forceinline__ C get(uint32_t i, int, uint32_t) const { return row[i]; }
};

// One pass over the source: counts the elements above the window, stages
// those inside it, and writes every full stage as one row of the candidate
// buffer, grouped by bucket.  A row's place costs one device atomic; the
// bucket's size and first output slot are sums over the rows' offsets, so no
// counting pass and no global scatter are needed.  One workgroup a CU.  Bound by
// instructions (2.2 us a tile of 32 KB and CU, 1.3 of them memory) and by a
// row's chain of LDS steps: n = 2^24 float32, k = 2^21: 42 us, its median 37,
// where six passes of a digit select took 260 and the sort of the select's
// output 380.
template <typename K, bool ARR>
__global__ __launch_bounds__(kSPartThreads) void k_spart(const K* __restrict__ keys,
                                                         const typename STraits<K>::Comp* __restrict__ arr,
                                                         uint64_t n, uint32_t head, uint32_t cap1, uint32_t k,
                                                         uint32_t m, SWin win, SCodec<K> cd, int L,
                                                         const typename STraits<K>::Comp* __restrict__ sorted,
                                                         SCtl* ctl, typename STraits<K>::Comp* __restrict__ out,
                                                         uint32_t cap, uint32_t maxrows, SRow* __restrict__ rows,
                                                         uint16_t* __restrict__ offs, uint32_t pitch,
                                                         typename STraits<K>::Comp* __restrict__ bounds) {
  typedef typename STraits<K>::Comp C;
  typedef typename std::conditional<ARR, C, K>::type R;
  constexpr int ST = STraits<K>::kStage, TILE = STraits<K>::kTile, MB = STraits<K>::kMaxB, T = kSPartThreads;
  constexpr int NE = TILE / T;  // elements a thread reads at a time
  constexpr int NF = ST / T;    // elements it writes at most
  constexpr int V = ARR ? 16 / (int)sizeof(C) : 16 / (int)sizeof(K);  // elements of a 128-bit load
  constexpr int U = NE / V;
  static_assert(U >= 1 && NE % V == 0 && ST % T == 0, "a tile is whole 128-bit loads");
  constexpr int BP = (MB + T - 1) / T;  // bucket counters a thread scans
  __shared__ SStage<K, ARR, ST> stage;
  __shared__ C split[MB];
  __shared__ uint32_t hist[MB + 1];
  __shared__ uint32_t s_w[T / 64], s_above, s_maxlen;
  __shared__ uint16_t tab[kSCells + 1];  // tab[i + 1]: splitters above cell i; tab[0]: all
  __shared__ uint32_t s_n, s_row, s_base;
  uint32_t* const stage_cells = reinterpret_cast<uint32_t*>(&stage);  // before anything is staged
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t posmask = (uint32_t)((1ull << L) - 1);
  uint64_t count = n;
  if constexpr (ARR) {
    count = (uint32_t)ctl->alloc1;
    if (count > cap1 || count < k) return;
  }
  // Tiles of TILE elements from the first 16-byte boundary on (head: the
  // elements before it, a last tile of their own).  A thread's loads of the
  // next tile are in flight while it works on the current one.
  const R* src;
  if constexpr (ARR) src = arr;
  else src = keys;
  constexpr uint32_t tile = TILE;
  const uint64_t body = (count - head + tile - 1) / tile;
  const uint64_t ntile = body + (head ? 1 : 0);
  R cur[NE], nxt[NE];
  uint32_t nvalid = 0;
  // element e of thread t in a tile: load e / V, 16-byte piece t, part e % V
  auto first = [&](uint64_t tl, int u) { return tl * tile + (uint64_t)u * T * V + threadIdx.x * V; };
  auto load = [&](uint64_t tl) {
    nvalid = 0;
    if (tl >= ntile) return;
    if (tl == body) {
      if (threadIdx.x < head) {
        nxt[0] = src[threadIdx.x];
        nvalid = 1u;
      }
      return;
    }
    const uint64_t end = count - head;
    if ((tl + 1) * tile <= end) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const su32x4 q = __builtin_nontemporal_load(reinterpret_cast<const su32x4*>(src + head + first(tl, u)));
        __builtin_memcpy(&nxt[u * V], &q, 16);
      }
      nvalid = (1u << NE) - 1;
      return;
    }
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const uint64_t p = first(tl, e / V) + e % V;
      if (p < end) {
        nxt[e] = src[head + p];
        nvalid |= 1u << e;
      }
    }
  };
  load(blockIdx.x);  // in flight while the window is prepared
  SWin w = win;  // level 2's was made on the device
  if constexpr (ARR) w = suniform(ctl->win);
  const uint32_t B = w.B;
  sfill_splitters<C>(split, w, m, sorted, threadIdx.x, T);
  for (uint32_t b = threadIdx.x; b <= B; b += T) hist[b] = 0;
  if (threadIdx.x == 0) { s_n = 0; s_above = 0; }
  const C hi = suniform(w.a ? sorted[w.a - 1] : ~(C)0);
  const C lo = suniform(w.r <= m ? sorted[w.r - 1] : (C)0);
  const R hikey = ARR ? (R)hi : (R)(hi >> L), lokey = ARR ? (R)lo : (R)(lo >> L);
  const uint32_t hipos = scomp_pos<C>(hi, posmask), lopos = scomp_pos<C>(lo, posmask);
  uint32_t above = 0;
  uint32_t staged = 0;  // block-uniform fill level
  // Where to look for a composite's bucket: kSCells equal cells of [lo, top),
  // each with the number of splitters above it, so the search is over the few
  // splitters of one cell (a search over all of them was half of a row's time).
  if (threadIdx.x == 0) s_maxlen = kSTop - 1;
  stage_cells[threadIdx.x] = 0;
  __syncthreads();
  if (blockIdx.x == 0)  // for the bucket kernel
    for (uint32_t b = threadIdx.x; b < B; b += T) bounds[b] = split[b];
  // at or above `top`: one of the first ntop + 1 buckets
  const uint32_t ntop = w.P && !w.a ? kSTop - 1 : 0u;
  const C top = suniform(split[ntop]);
  const uint32_t cbits = sbits((C)(top - lo));
  const int csh = cbits > 10 ? (int)cbits - 10 : 0;
  static_assert(kSCells == T, "a cell a thread");
  for (uint32_t b = threadIdx.x; b < B; b += T)
    if (split[b] < top) atomicAdd(&stage_cells[(uint32_t)((split[b] - lo) >> csh)], 1u);
  __syncthreads();
  {
    uint32_t m = stage_cells[kSCells - 1 - threadIdx.x], tot;  // cells from the top down
    const uint32_t ex = sblock_scan<T>(m, s_w, &tot);
    tab[kSCells - threadIdx.x] = (uint16_t)(B - tot + ex);  // B - tot splitters are not below top
    if (threadIdx.x == 0) tab[0] = (uint16_t)B;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      const uint32_t q = (uint32_t)__shfl_xor((int)m, o);
      m = q > m ? q : m;
    }
    if (lane == 0) atomicMax(&s_maxlen, m);
  }
  __syncthreads();
  const uint32_t maxlen = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_maxlen);

  // Writes the `cnt` staged candidates as one row (every thread calls).
  auto flush = [&](uint32_t cnt) {
    // opaque, so that the many indices made from it are made here and not
    // carried through the tile loop in registers
    uint32_t tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    uint64_t al = 0;  // in flight while the buckets are found
    if (tid == 0) al = atomicAdd((unsigned long long*)&ctl->alloc, (1ull << 32) | cnt);
    if (w.a) {
      const uint32_t x = swave_scan(above);
      if (lane == 63 && x) atomicAdd(&s_above, x);
      above = 0;
    }
    C c[NF];
    uint32_t at[NF];  // first splitter to look at << 16 | how many; then bucket << 16 | rank in it
#pragma unroll
    for (int e = 0; e < NF; ++e) {
      const uint32_t i = e * T + tid;
      at[e] = 0;
      c[e] = 0;
      if (i < cnt) {
        c[e] = stage.get(i, L, posmask);
        at[e] = ntop;
        if (c[e] < top) {
          const uint32_t cell = (uint32_t)((c[e] - lo) >> csh), f = tab[cell + 1];
          at[e] = (f << 16) | (tab[cell] - f);
        }
      }
    }
    for (uint32_t w = maxlen; w; w >>= 1) {
#pragma unroll
      for (int e = 0; e < NF; ++e) {
        const uint32_t len = at[e] & 0xFFFFu, h = len >> 1;
        if (len) at[e] = split[(at[e] >> 16) + h] > c[e] ? at[e] + ((h + 1) << 16) - h - 1 : at[e] - len + h;
      }
    }
#pragma unroll
    for (int e = 0; e < NF; ++e)
      if (e * T + tid < cnt) at[e] = (at[e] & 0xFFFF0000u) | atomicAdd(&hist[at[e] >> 16], 1u);
    __syncthreads();
    uint32_t h[BP], sum = 0;
#pragma unroll
    for (int j = 0; j < BP; ++j) {
      const uint32_t b = tid * BP + j;
      h[j] = b < B ? hist[b] : 0;
      sum += h[j];
    }
    uint32_t tot;
    uint32_t ex = sblock_scan<T>(sum, s_w, &tot);
#pragma unroll
    for (int j = 0; j < BP; ++j) {
      const uint32_t b = tid * BP + j;
      if (b < B) hist[b] = ex;
      ex += h[j];
    }
    if (tid == 0) {
      hist[B] = cnt;
      s_row = (uint32_t)(al >> 32);
      s_base = (uint32_t)al;
    }
    __syncthreads();
    const uint32_t row = s_row, base = s_base;
    if (row < maxrows) {
      if (tid == 0) rows[row] = SRow{base, s_above};
      for (uint32_t b = tid; b <= B; b += T) offs[(size_t)row * pitch + b] = (uint16_t)hist[b];
    }
    // through LDS into bucket order, so that the row leaves in whole lines
    // (scattered stores took 10 us a row of 10^4)
#pragma unroll
    for (int e = 0; e < NF; ++e)
      if (e * T + tid < cnt) stage.row[hist[at[e] >> 16] + (at[e] & 0xFFFFu)] = c[e];
    __syncthreads();
    for (uint32_t i = tid; i < cnt; i += T)
      if ((uint64_t)base + i < cap) out[base + i] = stage.row[i];
    __syncthreads();
    for (uint32_t b = tid; b <= B; b += T) hist[b] = 0;
    if (threadIdx.x == 0) s_above = 0;
  };

  for (uint64_t tl = blockIdx.x; tl < ntile; tl += gridDim.x) {
    const uint32_t valid = nvalid;
    const bool whole = tl < body && (tl + 1) * tile <= count - head;  // every element valid
    const uint32_t p0 = tl == body ? threadIdx.x : head + (uint32_t)first(tl, 0);
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      if constexpr (ARR) cur[e] = nxt[e];
      else cur[e] = senc<K>(nxt[e], cd);
    }
    load(tl + gridDim.x);
    // Each lane marks what it keeps, a prefix sum over the lanes' counts places
    // it, and every element is written, the ones not kept to a spare slot: the
    // loop is bound by its instructions, and this takes the fewest (a branch
    // per element: 2.0 us a tile of 32 KB).  Whether keys equal to a
    // bound's are inside is settled by position for a wave's load as a whole,
    // but for the one load that the bound's own position lies in.
    bool in[NE];
    uint32_t mine = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      R low = lokey, span = hikey - lokey;  // inside: key - low <= span
      bool exact = !whole;
      if constexpr (!ARR) {
        const uint32_t p1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(p0 + (uint32_t)u * T * V));
        const uint32_t p2 = p1 + 64 * V - 1;
        const bool past = p1 > lopos, before = w.a && p2 < hipos;
        low = past ? lokey + 1 : lokey;
        const R high = before ? hikey - 1 : hikey;
        span = high - low;
        exact = exact || (!past && p2 > lopos) || (w.a && !before && p1 < hipos) || low < lokey || high > hikey ||
                high < low;
      }
#pragma unroll
      for (int j = 0; j < V; ++j) {
        const int e = u * V + j;
        if (exact) {
          const uint32_t pos = p0 + (uint32_t)u * T * V + j;
          bool ok = (valid >> e) & 1u, up;
          if constexpr (ARR) {
            ok = ok && cur[e] >= lo;
            up = ok && cur[e] > hi;
          } else {
            ok = ok && (cur[e] > lokey || (cur[e] == lokey && pos <= lopos));
            up = w.a && ok && (cur[e] > hikey || (cur[e] == hikey && pos < hipos));
          }
          above += up ? 1u : 0u;
          in[e] = ok && !up;
        } else if (w.a) {
          in[e] = (R)(cur[e] - low) <= span;
          above += !in[e] && cur[e] > low ? 1u : 0u;
        } else {
          in[e] = cur[e] >= low;
        }
        mine += in[e] ? 1u : 0u;
      }
    }
    const uint32_t upto = swave_scan(mine);
    const uint32_t wcnt = (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
    uint32_t wbase = 0;
    if (lane == 0 && wcnt) wbase = atomicAdd(&s_n, wcnt);
    wbase = (uint32_t)__builtin_amdgcn_readfirstlane((int)wbase);
    __syncthreads();
    uint32_t now = suniform(s_n);
    if (now > (uint32_t)ST) {  // block-uniform: the tile does not fit beside what is staged
      flush(staged);
      if (threadIdx.x == 0) s_n = now - staged;
      wbase -= staged;
      now -= staged;
    }
    if (wcnt) {
      uint32_t at = wbase + upto - mine;
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        stage.put(in[e] ? at : (uint32_t)ST + lane, cur[e], p0 + (uint32_t)(e / V) * T * V + e % V);
        at += in[e] ? 1u : 0u;
      }
    }
    staged = now;
    __syncthreads();
  }
  uint32_t any = staged;
  if (w.a) any |= (uint32_t)__syncthreads_or((int)(above != 0));
  if (any) flush(staged);
}

// ---------------------------------------------------------------------------
// Bucket sort.

// LDS of a workgroup of T threads that sorts up to CAP composites.
template <typename C, uint32_t CAP, int T>
struct SSortShared {
  C buf[CAP];
  uint32_t hist[kSBins + 16];  // linear bins, or 8 pieces of each of kSSplit + 1 gaps
  C red[T / 64][2];
  C split[kSSplit];
  uint32_t rank[kSSplit];
  uint32_t s_w[T / 64];
  uint32_t misc[8];
};

// Sorts kSSplit LDS composites descending in place, by all-pairs ranks (T a
// multiple of kSSplit; `rank`: kSSplit words).  TIES: equal ones keep their
// order; otherwise all are distinct.
template <typename C, int T, bool TIES>
__device__ __forceinline__ void ssplit_sort(C* split, uint32_t* rank) {
  constexpr uint32_t S = kSSplit, parts = T / S, per = S / parts;
  const uint32_t i = threadIdx.x % S, j0 = threadIdx.x / S * per;
  if (threadIdx.x < S) rank[threadIdx.x] = 0;
  __syncthreads();
  const C x = split[i];
  uint32_t r = 0;
#pragma unroll 16
  for (uint32_t j = j0; j < j0 + per; ++j) {
    const C y = split[j];
    r += y > x || (TIES && y == x && j < i) ? 1u : 0u;
  }
  if constexpr (parts == 1) rank[i] = r;
  else atomicAdd(&rank[i], r);
  __syncthreads();
  if (threadIdx.x < S) {
    const uint32_t q = rank[threadIdx.x];
    split[q] = x;
  }
  __syncthreads();
}

// The larger (UP) or smaller of v and the value of a lane in the other M-half
// of this lane's 2M-block.
template <int M, bool UP, typename C>
__device__ __forceinline__ C sbest_cross(C v) {
  uint32_t w[sizeof(C) / 4];
  __builtin_memcpy(w, &v, sizeof(C));
#pragma unroll
  for (uint32_t i = 0; i < sizeof(C) / 4; ++i) w[i] = lane_cross32<M>(w[i]);
  C o;
  __builtin_memcpy(&o, w, sizeof(C));
  return (o > v) == UP ? o : v;
}

// Largest and smallest over the workgroup, held by every thread.  red: T / 64
// pairs, free before and after.
template <typename C, int T>
__device__ __forceinline__ void sblock_minmax(C& mx, C& mn, C (*red)[2]) {
  mx = sbest_cross<32, true>(sbest_cross<16, true>(sbest_cross<8, true>(
      sbest_cross<4, true>(sbest_cross<2, true>(sbest_cross<1, true>(mx))))));
  mn = sbest_cross<32, false>(sbest_cross<16, false>(sbest_cross<8, false>(
      sbest_cross<4, false>(sbest_cross<2, false>(sbest_cross<1, false>(mn))))));
  __syncthreads();
  if ((threadIdx.x & 63) == 0) {
    red[threadIdx.x >> 6][0] = mx;
    red[threadIdx.x >> 6][1] = mn;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < T / 64; ++w) {
    const C a = red[w][0], b = red[w][1];
    mx = a > mx ? a : mx;
    mn = b < mn ? b : mn;
  }
}

// Bin of a distance from the largest composite, finest at the top: 2^MB pieces
// of every octave.
template <typename C>
__device__ __forceinline__ uint32_t slog_bin(C d) {
  constexpr uint32_t MB = sizeof(C) == 8 ? 5 : 4;  // 1920 or 1488 bins
  const uint32_t w = sbits(d);
  if (w <= MB) return (uint32_t)d;
  return ((w - MB) << MB) + ((uint32_t)(d >> (w - MB - 1)) & ((1u << MB) - 1));
}

// lo plus the number of buf[lo .. hi) above c; four LDS reads in flight (one at
// a time, a bin of 300 cost 12 us).
template <typename C>
__device__ __forceinline__ uint32_t srank_in(const C* buf, uint32_t lo, uint32_t hi, C c) {
  uint32_t rk = lo;
  for (uint32_t j = lo; j < hi; j += 4) {
    C x[4];
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) x[q] = buf[j + q < hi ? j + q : j];
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) rk += j + q < hi && x[q] > c ? 1u : 0u;
  }
  return rk;
}

// Adds the lane to bin b of an LDS histogram and returns its rank there.  Lanes
// that all hold one bin (tied keys) add themselves once for the wave: the LDS
// serves adds to one address one lane at a time.
__device__ __forceinline__ uint32_t scount(uint32_t* hist, uint32_t b) {
  const uint32_t b0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)b);
  const uint64_t on = __ballot(1);
  if (__ballot(b == b0) == on) {
    uint32_t r = 0;
    const uint32_t rk = mbcnt(on);
    if (rk == 0) r = atomicAdd(&hist[b0], (uint32_t)__popcll(on));
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)r) + rk;
  }
  return atomicAdd(&hist[b], 1u);
}

// Sorts the N (<= CAP) composites held N = e * T + thread in c[] descending
// and calls emit(slot, composite) for each of the first `need` slots (and perhaps
// a few more).  Linear bins over [min, max] (logarithmic from the
// top when at most a quarter is needed: the top of both float and integer keys
// is then spread over many bins whatever lies below), a scatter into LDS bin by
// bin, then each element's rank inside its bin; bins that start past `need`
// are left alone.  When a bin that counts is crowded (keys in far-apart
// clusters, floats of both signs) bins between samples instead.
template <typename C, uint32_t CAP, int T, int E, typename F>
__device__ __forceinline__ void ssort(SSortShared<C, CAP, T>& sm, C (&c)[E], uint32_t N, uint64_t need, F&& emit,
                                      C mn = 0, C mx = ~(C)0) {
  for (int b = threadIdx.x; b <= kSBins; b += T) sm.hist[b] = 0;
  if (threadIdx.x == 0) sm.misc[0] = 0;
  if (mx == ~(C)0) {  // uniform
    mx = 0;
    mn = ~(C)0;
#pragma unroll
    for (int e = 0; e < E; ++e)
      if (e * T + threadIdx.x < N) {
        mx = c[e] > mx ? c[e] : mx;
        mn = c[e] < mn ? c[e] : mn;
      }
    sblock_minmax<C, T>(mx, mn, sm.red);
  } else {
    __syncthreads();
  }
  const uint32_t bl = sbits((C)(mx - mn));
  const int sh = bl > 11 ? (int)bl - 11 : 0;
  const bool logb = need <= N / 4;
  uint32_t at[E];
#pragma unroll
  for (int e = 0; e < E; ++e)
    if (e * T + threadIdx.x < N) {
      const uint32_t b = logb ? slog_bin<C>(mx - c[e]) : (uint32_t)((mx - c[e]) >> sh);
      at[e] = (b << 16) | scount(sm.hist, b);
    }
  __syncthreads();
  constexpr int BP = kSBins / T;
  uint32_t h[BP], sum = 0;
#pragma unroll
  for (int j = 0; j < BP; ++j) {
    h[j] = sm.hist[threadIdx.x * BP + j];
    sum += h[j];
  }
  uint32_t tot;
  uint32_t ex = sblock_scan<T>(sum, sm.s_w, &tot);
#pragma unroll
  for (int j = 0; j < BP; ++j) {
    sm.hist[threadIdx.x * BP + j] = ex;
    if (h[j] > kSCrowd && ex < need) sm.misc[0] = 1;
    ex += h[j];
  }
  if (threadIdx.x == 0) sm.hist[kSBins] = N;
  __syncthreads();
  if (!sm.misc[0]) {
#pragma unroll
    for (int e = 0; e < E; ++e)
      if (e * T + threadIdx.x < N) {
        const uint32_t lo = sm.hist[at[e] >> 16];
        if (lo < need) sm.buf[lo + (at[e] & 0xFFFFu)] = c[e];
      }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e)
      if (e * T + threadIdx.x < N) {
        const uint32_t b = at[e] >> 16;
        const uint32_t lo = sm.hist[b], hi = sm.hist[b + 1];
        if (lo < need) {
          emit(srank_in(sm.buf, lo, hi, c[e]), c[e]);
        }
      }
    __syncthreads();
    return;
  }
  // 256 of the elements, evenly spread over the threads' order, sorted by
  // their ranks, bound the bins instead (all elements are distinct, so the bins
  // are even whatever the keys)
  constexpr uint32_t S = kSSplit;
  __syncthreads();
  if (threadIdx.x == 0) sm.misc[0] = 0;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const uint32_t i = e * T + threadIdx.x;
    if (i < N) {
      // sample q is element (q * N) / S: element i is one of them, perhaps of
      // several q when N < S (any of those will do)
      const uint32_t q = (uint32_t)(((uint64_t)i * S + N - 1) / N);
      if (q < S && (uint32_t)((uint64_t)q * N / S) == i)
        for (uint32_t j = q; j < S && (uint32_t)((uint64_t)j * N / S) == i; ++j) sm.split[j] = c[e];
    }
  }
  constexpr uint32_t SUB = 8, NB = (S + 1) * SUB;
  for (uint32_t b = threadIdx.x; b < NB; b += T) sm.hist[b] = 0;
  ssplit_sort<C, T, true>(sm.split, sm.rank);
#pragma unroll
  for (int e = 0; e < E; ++e)
    if (e * T + threadIdx.x < N) {
      uint32_t b = 0;  // splitters above c
#pragma unroll
      for (uint32_t w = S / 2; w >= 1; w >>= 1)
        if (sm.split[b + w - 1] > c[e]) b += w;
      if (b == S - 1 && sm.split[S - 1] > c[e]) b = S;
      // up to eight equal pieces of the gap [lo, hi] that holds c
      const C hi = b ? sm.split[b - 1] : mx, lo = b < S ? sm.split[b] : mn;
      const uint32_t w = sbits((C)(hi - lo));
      b = b * SUB + SUB - 1 - (uint32_t)((c[e] - lo) >> (w > 3 ? w - 3 : 0));
      at[e] = (b << 16) | atomicAdd(&sm.hist[b], 1u);
    }
  __syncthreads();
  constexpr uint32_t PB = (NB + T - 1) / T;
  uint32_t g[PB], gs = 0, all;
#pragma unroll
  for (uint32_t j = 0; j < PB; ++j) {
    const uint32_t b = threadIdx.x * PB + j;
    g[j] = b < NB ? sm.hist[b] : 0u;
    gs += g[j];
  }
  uint32_t gx = sblock_scan<T>(gs, sm.s_w, &all);
#pragma unroll
  for (uint32_t j = 0; j < PB; ++j) {
    const uint32_t b = threadIdx.x * PB + j;
    if (b <= NB) sm.hist[b] = gx;
    gx += g[j];
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < E; ++e)
    if (e * T + threadIdx.x < N) {
      const uint32_t lo = sm.hist[at[e] >> 16];
      if (lo < need) sm.buf[lo + (at[e] & 0xFFFFu)] = c[e];
    }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < E; ++e)
    if (e * T + threadIdx.x < N) {
      const uint32_t b = at[e] >> 16;
      const uint32_t lo = sm.hist[b], hi = sm.hist[b + 1];
      if (lo < need) {
        emit(srank_in(sm.buf, lo, hi, c[e]), c[e]);
      }
    }
  __syncthreads();
}

// The element of rank `rank` (from 0, descending) among the N (<= CAP) composites held as
// in ssort; emit(rank, composite) if there is one.  Bins as there, but only the
// one that holds the rank goes on: into LDS, and divided again between its own
// extremes while it is crowded (they lie in different bins, so each round leaves
// fewer, and a range of no more than a bin's width).  Bound by the chain of LDS passes,
// two barriers each: normal float64, the median of 500000 44.5 us a call, where
// sorting all of a crowded bucket by samples took 53; the 1000th of 4000 16 / 42.
template <typename C, uint32_t CAP, int T, int E, typename F>
__device__ __forceinline__ void skth(SSortShared<C, CAP, T>& sm, C (&c)[E], uint32_t N, uint64_t rank, F&& emit,
                                     C mn = 0, C mx = ~(C)0) {
  for (uint32_t off = 0;;) {  // elements above those that are left
    for (int b = threadIdx.x; b < kSBins; b += T) sm.hist[b] = 0;
    if (threadIdx.x == 0) sm.misc[7] = 0;
    if (mx == ~(C)0) {  // uniform
      mx = 0;
      mn = ~(C)0;
#pragma unroll
      for (int e = 0; e < E; ++e)
        if (e * T + threadIdx.x < N) {
          mx = c[e] > mx ? c[e] : mx;
          mn = c[e] < mn ? c[e] : mn;
        }
      sblock_minmax<C, T>(mx, mn, sm.red);
    } else {
      __syncthreads();
    }
    const uint32_t bl = sbits((C)(mx - mn));
    const int sh = bl > 11 ? (int)bl - 11 : 0;
    const bool logb = off == 0 && rank < N / 4;
    uint32_t at[E];
#pragma unroll
    for (int e = 0; e < E; ++e)
      if (e * T + threadIdx.x < N) {
        const uint32_t b = logb ? slog_bin<C>(mx - c[e]) : (uint32_t)((mx - c[e]) >> sh);
        at[e] = (b << 16) | scount(sm.hist, b);
      }
    __syncthreads();
    constexpr int BP = kSBins / T;
    uint32_t h[BP], sum = 0;
#pragma unroll
    for (int j = 0; j < BP; ++j) {
      h[j] = sm.hist[threadIdx.x * BP + j];
      sum += h[j];
    }
    uint32_t tot;
    uint32_t ex = sblock_scan<T>(sum, sm.s_w, &tot);
#pragma unroll
    for (int j = 0; j < BP; ++j) {
      if (ex <= rank && rank < ex + h[j]) {
        sm.misc[5] = threadIdx.x * BP + j;
        sm.misc[6] = ex;
        sm.misc[7] = h[j];
      }
      ex += h[j];
    }
    __syncthreads();
    const uint32_t bin = sm.misc[5], lo = sm.misc[6], cnt = sm.misc[7];
    if (cnt) {
#pragma unroll
      for (int e = 0; e < E; ++e)
        if (e * T + threadIdx.x < N && at[e] >> 16 == bin) sm.buf[at[e] & 0xFFFFu] = c[e];
    }
    __syncthreads();
    off += lo;
    rank -= lo;
    if (cnt <= kSCrowd) {
      if (threadIdx.x < cnt) {
        const C x = sm.buf[threadIdx.x];
        const uint32_t rk = srank_in(sm.buf, 0, cnt, x);
        if (rk == rank) emit(off + rk, x);
      }
      __syncthreads();
      return;
    }
    N = cnt;
#pragma unroll
    for (int e = 0; e < E; ++e)
      if (e * T + threadIdx.x < N) c[e] = sm.buf[e * T + threadIdx.x];
    mx = ~(C)0;
  }
}

template <typename K>
struct SBucketShared : SSortShared<typename STraits<K>::Comp, STraits<K>::kCap, kSBucketThreads> {
  uint32_t pre[kSMaxRows + 1];  // bucket elements in the segments before this one
  uint32_t src[kSMaxRows];      // candidate index of the segment
  uint32_t w3[kSBucketThreads / 64][3];
};

// f(get(i)) for the workgroup's i < count, four elements a thread at a time so
// that their loads overlap.
template <typename C, int TT, typename G, typename F>
__device__ __forceinline__ void sbucket_each(uint64_t count, G&& get, F&& f) {
  constexpr uint64_t T = TT;
  uint64_t i = threadIdx.x;
  for (; i + 3 * T < count; i += 4 * T) {
    C x[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) x[j] = get(i + j * T);
#pragma unroll
    for (int j = 0; j < 4; ++j) f(x[j]);
  }
  for (; i < count; i += T) f(get(i));
}

// Internal checks of the sampled path: `rec` is the stream's check record
// (nullptr: none), `hold` the most elements that a run or a fallback collects
// (the LDS's capacity; less only through the testing hook drtopk_set_run_cap).
struct SCheck {
  uint32_t* rec;
  uint32_t hold;
};

// Collects the elements get(i), i < count, lying in [lo, hi] (`want` of them, at
// most CAP, known to the caller) into registers in sort order's layout.
template <typename C, uint32_t CAP, int T, int E, typename G>
__device__ __forceinline__ uint32_t sbucket_collect(SSortShared<C, CAP, T>& sm, C (&c)[E], uint64_t count, C lo,
                                                    C hi, uint32_t want, const SCheck& ck, G&& get) {
  const uint32_t hold = ck.hold < CAP ? ck.hold : CAP;
  if (threadIdx.x == 0) sm.misc[1] = 0;
  __syncthreads();
  sbucket_each<C, T>(count, get, [&](C x) {
    if (x >= lo && x <= hi) {
      const uint32_t s = atomicAdd(&sm.misc[1], 1u);
      if (s < hold) sm.buf[s] = x;
    }
  });
  __syncthreads();
  const uint32_t got = sm.misc[1], N = got < hold ? got : hold;
  if (threadIdx.x == 0) {
    if (got > hold) record_err(ck.rec, ERR_CAP);
    if (N < want) record_err(ck.rec, ERR_FEW);
  }
#pragma unroll
  for (int e = 0; e < E; ++e)
    if (e * T + threadIdx.x < N) c[e] = sm.buf[e * T + threadIdx.x];
  __syncthreads();
  return N;
}

// Histogram of the elements get(i) in [mn, mx] over kSBins linear bins
// (descending: bin 0 holds mx), prefix-summed.  Returns the shift.
template <typename C, uint32_t CAP, int T, typename G>
__device__ __forceinline__ int sbucket_hist(SSortShared<C, CAP, T>& sm, uint64_t count, C mn,
                                            C mx, G&& get) {
  const uint32_t bl = sbits((C)(mx - mn));
  const int sh = bl > 11 ? (int)bl - 11 : 0;
  for (int b = threadIdx.x; b <= kSBins; b += T) sm.hist[b] = 0;
  __syncthreads();
  sbucket_each<C, T>(count, get, [&](C x) {
    if (x >= mn && x <= mx) atomicAdd(&sm.hist[(uint32_t)((mx - x) >> sh)], 1u);
  });
  __syncthreads();
  constexpr int BP = kSBins / T;
  uint32_t h[BP], sum = 0;
#pragma unroll
  for (int j = 0; j < BP; ++j) {
    h[j] = sm.hist[threadIdx.x * BP + j];
    sum += h[j];
  }
  uint32_t tot;
  uint32_t ex = sblock_scan<T>(sum, sm.s_w, &tot);
#pragma unroll
  for (int j = 0; j < BP; ++j) {
    sm.hist[threadIdx.x * BP + j] = ex;
    ex += h[j];
  }
  if (threadIdx.x == 0) sm.hist[kSBins] = tot;
  __syncthreads();
  return sh;
}

// The element of 1-based rank `rank` among get(i), i < count (all distinct, at most `top`).
template <typename C, uint32_t CAP, int T, typename G>
__device__ __forceinline__ C sbucket_select(SSortShared<C, CAP, T>& sm, uint64_t count, uint64_t rank, C top,
                                            const SCheck& ck, G&& get) {
  C mn = 0, mx = top;
  for (;;) {
    const int sh = sbucket_hist<C, CAP, T>(sm, count, mn, mx, get);
    if (threadIdx.x == 0) {
      sm.misc[2] = 0;
      if (rank - 1 >= sm.hist[kSBins]) record_err(ck.rec, ERR_SELECT);  // no bin holds the rank
    }
    __syncthreads();
    for (uint32_t b = threadIdx.x; b < (uint32_t)kSBins; b += T)
      if (sm.hist[b] < rank && rank <= sm.hist[b + 1]) sm.misc[2] = b;
    __syncthreads();
    const uint32_t b = sm.misc[2];
    rank -= sm.hist[b];
    __syncthreads();
    mx = mx - ((C)b << sh);
    if (sh == 0) return mx;  // the bin is one composite
    const C width = ((C)1 << sh) - 1;
    mn = mx - mn > width ? mx - width : mn;
  }
}

// Where a slot of the output goes.
template <typename K>
struct SOut {
  K* vals;
  uint32_t* idx;
  K* kth;
  uint32_t k;
  int kth_only;
  SCodec<K> cd;
  int L;
  uint32_t posmask;
  SPayload pay;
  __device__ __forceinline__ void operator()(uint64_t slot, typename STraits<K>::Comp c) const {
    if (slot >= k) return;
    const K v = sdec<K>((K)(c >> L), cd);
    if (!kth_only) {
      const uint32_t p = scomp_pos<typename STraits<K>::Comp>(c, posmask);
      if (vals) vals[slot] = v;
      if (idx) idx[slot] = p;
      if (pay.bytes == 8)
        static_cast<uint64_t*>(pay.out)[slot] = static_cast<const uint64_t*>(pay.in)[p];
      else if (pay.bytes == 4)
        static_cast<uint32_t*>(pay.out)[slot] = static_cast<const uint32_t*>(pay.in)[p];
    }
    if (kth && slot == k - 1) *kth = v;
  }
};

// Where the candidates are: one list that is one bucket; one list of a few
// buckets, which each workgroup reads whole; or rows grouped by bucket.
enum SMode { kSPlain, kSList, kSRows };

// Element i of a bucket's source: candidate i, or by the segments' prefix sums.
template <typename K, SMode MODE>
__device__ __forceinline__ typename STraits<K>::Comp sbucket_get(const SBucketShared<K>& sm,
                                                                 const typename STraits<K>::Comp* cand, uint64_t i) {
  if constexpr (MODE != kSRows) {
    return cand[i];
  } else {
    uint32_t r0 = 0;  // last segment with pre <= i
#pragma unroll
    for (uint32_t h = kSMaxRows / 2; h >= 1; h >>= 1)
      if (sm.pre[r0 + h] <= (uint32_t)i) r0 += h;
    return cand[sm.src[r0] + ((uint32_t)i - sm.pre[r0])];
  }
}

// The rare ways to the output: runs of at most CAP elements, sorted one after
// the other.  Either the leading bins of what is left of a bucket larger than
// the LDS (its `size` elements of the source's `count` lie in [low, upto], its
// first slot is `start`), or (count 0) a rescue: each workgroup answers ranks of
// its own from the input, independently of the others.
template <typename K, SMode MODE>
__device__ __forceinline__ void sbucket_rare(SBucketShared<K>& sm, const K* keys, uint64_t n,
                                             const typename STraits<K>::Comp* cand, uint64_t start, uint32_t size,
                                             uint32_t count, typename STraits<K>::Comp low,
                                             typename STraits<K>::Comp upto, const SOut<K>& out, const SCheck& ck) {
  typedef typename STraits<K>::Comp C;
  constexpr int T = kSBucketThreads;
  constexpr uint32_t CAP = STraits<K>::kCap;
  constexpr int E = (int)(CAP + T - 1) / T;
  const bool rescue = count == 0;
  const uint32_t k = out.k;
  auto input = [&](uint64_t i) { return scomp<K>(senc<K>(keys[i], out.cd), (uint32_t)i, out.L, out.posmask); };
  auto get = [&](uint64_t i) { return sbucket_get<K, MODE>(sm, cand, i); };
  if (rescue && out.kth_only && blockIdx.x > 0) return;
  uint64_t base = rescue ? (out.kth_only ? (uint64_t)k - 1 : (uint64_t)blockIdx.x * CAP) : start;
  C c[E];
  bool more = true;
  while (more && base < k) {
    uint32_t N;
    uint64_t next;
    if (rescue) {
      const uint64_t r1 = base + CAP < k ? base + CAP : k;
      C bound[2];
#pragma unroll 1
      for (int s = 0; s < 2; ++s)
        bound[s] =
            sbucket_select<C, CAP, T>(sm, n, s ? r1 : base + 1, ((C)(K)~(K)0 << out.L) | out.posmask, ck, input);
      N = sbucket_collect<C, CAP, T, E>(sm, c, n, bound[1], bound[0], (uint32_t)(r1 - base), ck, input);
      next = base + (uint64_t)gridDim.x * CAP;
    } else {
      C mn = ~(C)0, mx = 0;
      sbucket_each<C, T>(count, get, [&](C x) {
        if (x >= low && x <= upto) {
          mx = x > mx ? x : mx;
          mn = x < mn ? x : mn;
        }
      });
      sblock_minmax<C, T>(mx, mn, sm.red);
      if (mx < mn) break;  // nothing is left
      C cut = mn;
      uint32_t fit;
      for (;;) {
        const int sh = sbucket_hist<C, CAP, T>(sm, count, mn, mx, get);
        // the most leading bins whose elements fit
        if (threadIdx.x == 0) sm.misc[3] = 0;
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < (uint32_t)kSBins; i += T)
          if (sm.hist[i + 1] <= CAP && (i + 1 == (uint32_t)kSBins || sm.hist[i + 2] > CAP)) sm.misc[3] = i + 1;
        __syncthreads();
        fit = sm.misc[3];
        __syncthreads();
        cut = leading_bins_cut<C>(mx, mn, fit ? fit : 1u, sh);
        if (fit || sh == 0) break;
        mn = cut;  // the first bin alone is too large: look inside it
      }
      N = sbucket_collect<C, CAP, T, E>(sm, c, count, cut, mx, sm.hist[fit ? fit : 1u], ck, get);
      if (N == 0) break;
      next = base + N;
      more = cut > low;
      upto = cut - 1;
    }
    const auto emit = [&](uint32_t rk, C x) { out(base + rk, x); };
    if (out.kth_only) skth<C, CAP, T, E>(sm, c, N, k - 1 - base, emit);
    else ssort<C, CAP, T, E>(sm, c, N, k - base, emit);
    base = next;
  }
  // the runs are the whole bucket, or reach the last slot
  if (!rescue && base < k && base != start + size && threadIdx.x == 0) record_err(ck.rec, ERR_FEW);
}

// One workgroup per bucket.  RARE: the rare ways are part of the kernel, which
// then takes so many registers that one workgroup fills a CU: for few buckets.
// With many, a kernel without them runs first (two workgroups a CU) and only
// notes in ctl->rare that they are needed; `second` then runs this kernel for
// those buckets, or for nothing.  Bound by the chain of LDS passes of one
// bucket: one bucket of up to 7680, 8 us; 2^21 elements in 1300 buckets, 37 us,
// where LDS tiles and merges took 320; a list of 10^4 with payloads 18 us.
template <typename K, SMode MODE, bool RARE>
__global__ __launch_bounds__(kSBucketThreads) __attribute__((amdgpu_waves_per_eu(RARE ? 2 : 4))) void k_sbucket(
    const K* __restrict__ keys, uint64_t n, uint32_t k, int kth_only, int levels, int second, SCodec<K> cd, int L,
    SCtl* __restrict__ ctl, const typename STraits<K>::Comp* __restrict__ cand, uint32_t cap1, uint32_t cap,
    uint32_t maxrows, const SRow* __restrict__ rows, const uint16_t* __restrict__ offs, uint32_t pitch, uint32_t m,
    SWin win, const typename STraits<K>::Comp* __restrict__ sorted,
    const typename STraits<K>::Comp* __restrict__ bounds, K* __restrict__ out_vals, uint32_t* __restrict__ out_idx,
    K* __restrict__ out_kth, SPayload pay, SCheck ck) {
  typedef typename STraits<K>::Comp C;
  constexpr int T = kSBucketThreads;
  constexpr uint32_t CAP = STraits<K>::kCap;
  constexpr int E = (int)(CAP + T - 1) / T;
  __shared__ SBucketShared<K> sm;
  if (second && !ctl->rare) return;
  const SOut<K> out{out_vals, out_idx, out_kth, k, kth_only, cd, L, (uint32_t)((1ull << L) - 1), pay};
  const uint64_t al = ctl->alloc;
  const uint32_t nc = (uint32_t)al, nrows = (uint32_t)(al >> 32);
  const uint32_t b = blockIdx.x;
  bool bad = nc > cap;
  if (levels == 2) {
    const uint32_t c1 = (uint32_t)ctl->alloc1;
    bad = bad || c1 > cap1 || c1 < k;
  }
  uint64_t start = 0;  // elements ranked above the bucket
  uint32_t count = nc, source = nc;
  C low = 0, upto = ~(C)0;  // the bucket's bounds in its source
  C c[E];
  if constexpr (MODE == kSPlain) {
    bad = bad || nc < k;
    if (!bad && count <= CAP) {
#pragma unroll
      for (int e = 0; e < E; ++e)
        if (e * T + threadIdx.x < count) c[e] = cand[e * T + threadIdx.x];
    }
  } else if constexpr (MODE == kSList) {
    bad = bad || nc < k;
    if (!bad) {
      const SWin w = win;
      C* const split = sm.buf;  // before anything is collected
      sfill_splitters<C>(split, w, m, sorted, threadIdx.x, T);
      if (threadIdx.x == 0) sm.misc[4] = 0;
      __syncthreads();
      if (b >= w.B) return;
      low = suniform(split[b]);
      if (b) upto = suniform(split[b - 1]) - 1;
      __syncthreads();
      uint32_t above = 0, seen = 0;
      if (low <= upto) {
        // eight 16-byte loads a thread in flight; what a wave keeps of them is
        // placed by a prefix sum over its lanes and one LDS atomic
        constexpr uint32_t V = 16 / sizeof(C), U = 8;
        const uint32_t pieces = (nc + V - 1) / V;  // the buffer is whole pieces
        for (uint32_t g0 = 0; g0 < pieces; g0 += U * T) {
          C x[U * V];
#pragma unroll
          for (uint32_t u = 0; u < U; ++u) {
            const uint32_t g = g0 + u * T + threadIdx.x;
            su32x4 q = {};
            if (g < pieces) q = *reinterpret_cast<const su32x4*>(cand + (size_t)g * V);
            __builtin_memcpy(&x[u * V], &q, 16);
          }
          uint32_t mine = 0;
#pragma unroll
          for (uint32_t j = 0; j < U * V; ++j) {
            if ((g0 + j / V * T + threadIdx.x) * V + j % V >= nc) x[j] = 0;  // below every bucket that is looked at
            above += x[j] > upto ? 1u : 0u;
            mine += x[j] >= low ? 1u : 0u;
          }
          mine -= above - seen;
          seen = above;
          const uint32_t inc = swave_scan(mine);
          uint32_t at = 0;
          if ((threadIdx.x & 63) == 63 && inc) at = atomicAdd(&sm.misc[4], inc);
          at = (uint32_t)__builtin_amdgcn_readlane((int)at, 63) + inc - mine;
#pragma unroll
          for (uint32_t j = 0; j < U * V; ++j)
            if (x[j] >= low && x[j] <= upto) {
              if (at < CAP) sm.buf[at] = x[j];
              ++at;
            }
        }
        __syncthreads();
      }
      uint32_t tot, zero;
      sblock_scan3<T>(0, above, 0, sm.w3, &zero, &zero, &tot, &zero);
      start = tot;
      count = sm.misc[4];
      if (start >= k || count == 0 || (kth_only && start + count < k)) return;
#pragma unroll
      for (int e = 0; e < E; ++e)
        if (e * T + threadIdx.x < count && count <= CAP) c[e] = sm.buf[e * T + threadIdx.x];
      __syncthreads();
    }
  } else {
    bad = bad || nrows > maxrows;
    const uint32_t B = ctl->win.B;
    low = bounds[b];
    if (b) upto = bounds[b - 1];
    low = suniform(low);
    upto = suniform(upto);
    // this bucket's segments: thread t takes rows t and t + T, whose loads do
    // not wait for the number of rows
    static_assert(kSMaxRows == 2 * T, "two rows a thread");
    uint32_t len[2], from[2], sum = 0, before = 0, ab = 0;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const uint32_t r = threadIdx.x + j * T;
      SRow rw = {};
      uint32_t o0 = 0, o1 = 0;
      if (r < maxrows) {
        rw = rows[r];
        o0 = offs[(size_t)r * pitch + b];
        o1 = offs[(size_t)r * pitch + b + 1];
      }
      const bool on = r < nrows && !bad;
      ab += on ? rw.above : 0u;
      len[j] = on && b < B ? o1 - o0 : 0u;
      before += on && b < B ? o0 : 0u;
      from[j] = rw.base + o0;
      sum += len[j];
    }
    uint32_t ex, tb, ta;
    sblock_scan3<T>(sum, before, ab, sm.w3, &ex, &count, &tb, &ta);
    start = (uint64_t)ta + tb;
    source = count;
    bad = bad || (uint64_t)ta + nc < k || ta >= k;  // too few at or above the cut, or too many above the window
    if (!bad && (b >= B || start >= k || count == 0 || (kth_only && start + count < k))) return;
    if (!bad) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        sm.pre[2 * threadIdx.x + j] = ex;
        sm.src[2 * threadIdx.x + j] = from[j];
        ex += len[j];
      }
      if (threadIdx.x == T - 1) sm.pre[kSMaxRows] = ex;
      __syncthreads();
      if (count <= CAP && !second) {
#pragma unroll
        for (int e = 0; e < E; ++e)
          if (e * T + threadIdx.x < count) c[e] = sbucket_get<K, MODE>(sm, cand, e * T + threadIdx.x);
      }
    }
  }
  if (bad || count > CAP) {
    if constexpr (RARE) {
      sbucket_rare<K, MODE>(sm, keys, n, cand, start, count, bad ? 0u : source, low, upto, out, ck);
    } else {
      if (threadIdx.x == 0) ctl->rare = 1;
    }
    return;
  }
  if (second) return;
  // (the lowest bucket may reach down to composite 0, far below its elements)
  const auto emit = [&](uint32_t rk, C x) { out(start + rk, x); };
  if (kth_only) skth<C, CAP, T, E>(sm, c, count, k - 1 - start, emit, low, low ? upto : ~(C)0);
  else ssort<C, CAP, T, E>(sm, c, count, k - start, emit, low, low ? upto : ~(C)0);
}

// The whole problem in one workgroup.  n <= CAP: every element goes into the
// sort.  Otherwise the r-th of 256 samples cuts the input to between k and
// CAP elements in one streaming pass, the survivors collected in LDS and
// sorted; when the sample misjudges that, the k-th element is found by
// histograms of the input instead.  k <= CAP.  Bound by the issue of one CU's
// vector units, about 15 instructions a key: 50000 float32, k = 64, 19.9 us a
// call against 21.9 for the delegate method in one workgroup; a few thousand 8-byte keys
// 7 against 43 for the passes over the device.
template <typename K>
struct SOne {
  typedef typename STraits<K>::Comp C;
  static constexpr uint32_t kCap = 65536 / sizeof(C);
};

template <typename K, int T, bool KTH>
__global__ __launch_bounds__(T) void k_sone(const K* __restrict__ keys, uint32_t n, uint32_t k, uint32_t r,
                                            int kth_only, SCodec<K> cd, int L, K* __restrict__ out_vals,
                                            uint32_t* __restrict__ out_idx, K* __restrict__ out_kth, SPayload pay,
                                            SCheck ck) {
  typedef typename STraits<K>::Comp C;
  constexpr uint32_t CAP = T == 1024 ? SOne<K>::kCap : 1024;
  constexpr int E = (int)(CAP / T);
  constexpr int V = 16 / (int)sizeof(K), U = 4;
  __shared__ SSortShared<C, CAP, T> sm;
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t posmask = (uint32_t)((1ull << L) - 1);
  auto get = [&](uint64_t i) { return scomp<K>(senc<K>(keys[i], cd), (uint32_t)i, L, posmask); };
  C c[E];
  uint32_t N = n;
  if (r == 0) {
#pragma unroll
    for (int e = 0; e < E; ++e)
      if (e * T + threadIdx.x < n) c[e] = get(e * T + threadIdx.x);
  } else {
    const uint32_t head0 = (uint32_t)(((16 - (reinterpret_cast<uintptr_t>(keys) & 15u)) & 15u) / sizeof(K));
    const uint32_t head = head0 < n ? head0 : n;
    const uint32_t loads = (n - head) / V;  // whole 16-byte pieces
    su32x4 nx[U];
    auto load = [&](uint32_t g0) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t g = g0 + u * T + threadIdx.x;
        if (g < loads) nx[u] = *reinterpret_cast<const su32x4*>(keys + head + (size_t)g * V);
      }
    };
    load(0);  // in flight while the samples are ranked
    if (threadIdx.x < kSSplit) {
      const uint32_t i = threadIdx.x;
      const uint32_t lo = (uint32_t)((uint64_t)i * n / kSSplit), hi = (uint32_t)((uint64_t)(i + 1) * n / kSSplit);
      sm.split[i] = get(lo + (uint32_t)(((uint64_t)shash(i) * (hi - lo)) >> 32));
    }
    if (threadIdx.x == 0) sm.misc[4] = 0;
    ssplit_sort<C, T, false>(sm.split, sm.rank);
    const C t = r <= kSSplit ? sm.split[r - 1] : (C)0;
    const K tkey = (K)(t >> L);
    const uint32_t tpos = scomp_pos<C>(t, posmask);
    for (uint32_t g0 = 0; g0 < loads; g0 += U * T) {
      K v[U][V];
#pragma unroll
      for (int u = 0; u < U; ++u) __builtin_memcpy(v[u], &nx[u], 16);
      load(g0 + U * T);
      uint64_t bal[U][V];
      uint32_t cnt = 0;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t g = g0 + u * T + threadIdx.x, p = head + g * V;
#pragma unroll
        for (int e = 0; e < V; ++e) {
          v[u][e] = senc<K>(v[u][e], cd);
          bal[u][e] = __ballot(g < loads && (v[u][e] > tkey || (v[u][e] == tkey && p + e <= tpos)));
          cnt += (uint32_t)__popcll(bal[u][e]);
        }
      }
      if (cnt == 0) continue;
      uint32_t base = 0;
      if (lane == 0) base = atomicAdd(&sm.misc[4], cnt);
      base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t p = head + (g0 + u * T + threadIdx.x) * V;
#pragma unroll
        for (int e = 0; e < V; ++e) {
          const uint32_t at = base + mbcnt(bal[u][e]);
          if (__builtin_amdgcn_inverse_ballot_w64(bal[u][e]) && at < CAP)
            sm.buf[at] = scomp<K>(v[u][e], p + e, L, posmask);
          base += (uint32_t)__popcll(bal[u][e]);
        }
      }
    }
    if (threadIdx.x < 64) {  // fewer than V keys before the pieces and after them
      const uint32_t rest = n - head - loads * V;
      const uint32_t p = lane < head ? lane : head + loads * V + (lane - head);
      const K e = lane < head + rest ? senc<K>(keys[p], cd) : (K)0;
      if (lane < head + rest && (e > tkey || (e == tkey && p <= tpos))) {
        const uint32_t at = atomicAdd(&sm.misc[4], 1u);
        if (at < CAP) sm.buf[at] = scomp<K>(e, p, L, posmask);
      }
    }
    __syncthreads();
    N = sm.misc[4];
    if (N < k || N > CAP) {
      const C kth = sbucket_select<C, CAP, T>(sm, n, k, ((C)(K)~(K)0 << L) | posmask, ck, get);
      N = sbucket_collect<C, CAP, T, E>(sm, c, n, kth, ~(C)0, k, ck, get);
    } else {
#pragma unroll
      for (int e = 0; e < E; ++e)
        if (e * T + threadIdx.x < N) c[e] = sm.buf[e * T + threadIdx.x];
    }
    __syncthreads();
  }
  const SOut<K> out{out_vals, out_idx, out_kth, k, kth_only, cd, L, posmask, pay};
  const auto emit = [&](uint32_t slot, C x) { out(slot, x); };
  // (a k-th value near the top of what a cut left of 4-byte keys: bins are not
  // crowded there, and the sort is the shorter chain; 24 of 12000 11.5 us a call
  // against 12.5; of lists sorted whole, 250 of 4000, 10.8 against 8.9)
  if (KTH && (sizeof(K) == 8 || r == 0 || k > N / 8)) skth<C, CAP, T, E>(sm, c, N, k - 1, emit);
  else ssort<C, CAP, T, E>(sm, c, N, k, emit);
}

}  // namespace drtopk
