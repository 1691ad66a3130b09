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
// from the input itself (rescue); the window's margin makes that rarer than
// 10^-10 for inputs laid out without regard to the sampled positions.
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
constexpr int kSRankPer = 32;        // samples ranked by one workgroup
constexpr int kSFilterThreads = 256;
constexpr uint32_t kSSplit = 256;    // samples of a workgroup's own sort or threshold

template <typename K>
struct STraits;
template <>
struct STraits<uint32_t> {
  typedef uint64_t Comp;
  static constexpr int kStage = 8192;   // candidates staged by a workgroup of k_spart
  static constexpr int kCap = 7680;     // elements sorted by a workgroup of k_sbucket (two fit a CU)
  static constexpr int kMaxB = 3072;    // most buckets
  static constexpr int kTarget = 2048;  // elements a bucket is planned for
};
template <>
struct STraits<uint64_t> {
  typedef su128 Comp;
  static constexpr int kStage = 4096;
  static constexpr int kCap = 3584;
  static constexpr int kMaxB = 1536;
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
  uint32_t pad2[24];
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
// Sampling, M samples (a multiple of 256) from a source of at least M elements.
// ARR: the source is level 1's candidates (their number is on the device);
// otherwise the input.  TOP: of each 256 samples the 16 largest are kept.  When
// the window's r is a few per workgroup, its top r samples are all kept but
// for odds far below the window's own, and if one is lost the r-th kept sample
// only lies lower: more candidates, never fewer.  So 65536 samples cost one
// gather and the ranks of 4096, and the r-th of 65536 leaves a tenth to a half
// of the candidates that the corresponding sample of 4096 does.
// The launch also clears the state of the kernels after it.
constexpr uint32_t kSKeep = 16;

template <typename K, bool ARR, bool TOP>
__global__ __launch_bounds__(256) void k_sgather(const K* __restrict__ keys,
                                                 const typename STraits<K>::Comp* __restrict__ arr, uint64_t n,
                                                 uint32_t cap1, uint32_t k, uint32_t M, SCodec<K> cd, int L,
                                                 SWin win, int kth, uint32_t bmax, SCtl* ctl,
                                                 typename STraits<K>::Comp* __restrict__ smp,
                                                 typename STraits<K>::Comp* __restrict__ sorted) {
  typedef typename STraits<K>::Comp C;
  const uint32_t i = blockIdx.x * 256 + threadIdx.x;
  uint64_t count = n;
  if constexpr (ARR) {
    count = (uint32_t)ctl->alloc1;
    if (count > cap1 || count < k) return;  // level 1 misjudged: the bucket kernel answers from the input
  }
  if (i == 0) {
    if constexpr (ARR) {
      SWin w = {};
      sample_window((double)count, (double)k, (double)M, kth != 0, &w);
      sample_buckets((double)count / (double)M, STraits<K>::kTarget, bmax, &w);
      ctl->win = w;
    } else {
      ctl->alloc1 = 0;
      ctl->alloc = 0;
      ctl->win = win;
    }
  }
  const uint32_t posmask = (uint32_t)((1ull << L) - 1);
  const uint64_t lo = (uint64_t)i * count / M, hi = (uint64_t)(i + 1) * count / M;
  C x = 0;
  if (hi > lo) {
    const uint64_t p = lo + (uint64_t)(((uint64_t)shash(i) * (hi - lo)) >> 32);
    if constexpr (ARR) x = arr[p];
    else x = scomp<K>(senc<K>(keys[p], cd), (uint32_t)p, L, posmask);
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
    s[threadIdx.x] = x;
    __syncthreads();
    uint32_t rk = 0;
#pragma unroll 16
    for (uint32_t j = 0; j < 256; ++j) rk += s[j] > x ? 1u : 0u;
    if (rk < kSKeep) smp[blockIdx.x * kSKeep + rk] = x;
  }
}

// All-pairs ranks: a wave holds J * 64 samples in registers and compares them
// with one sample at a time, a scalar operand, so 64 comparisons are one
// vector compare and a scalar bit count.  J * 512 = m samples.
template <typename C, int J>
__global__ __launch_bounds__(kSRankThreads) void k_srank(const C* __restrict__ smp, C* __restrict__ sorted) {
  __shared__ uint32_t cnt[kSRankPer][kSRankThreads / 64];
  const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  C v[J];
#pragma unroll
  for (int j = 0; j < J; ++j) v[j] = smp[(j * (kSRankThreads / 64) + wave) * 64 + lane];
  const uint32_t i0 = blockIdx.x * kSRankPer;
#pragma unroll 4
  for (int ii = 0; ii < kSRankPer; ++ii) {
    const C x = smp[i0 + ii];
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
    sorted[r] = smp[i0 + threadIdx.x];
  }
}

// ---------------------------------------------------------------------------
// Streaming filter for one bucket or a first level.  Tiles of U loads per wave
// are dealt to the workgroups in turn, so a dense stretch of candidates
// (sorted input) is shared by many.  A wave keeps its candidates in its own
// LDS slots and its fill level in a register; no barrier before the end.
// head: keys before the first 16-byte boundary.
constexpr uint32_t kSWaveSlots = 512;

template <typename K, int U>
__global__ __launch_bounds__(kSFilterThreads) void k_sfilter(const K* __restrict__ keys, uint64_t n, uint32_t head,
                                                             SCodec<K> cd, int L, uint32_t r, uint32_t m,
                                                             const typename STraits<K>::Comp* __restrict__ sorted,
                                                             uint64_t* alloc,
                                                             typename STraits<K>::Comp* __restrict__ out,
                                                             uint32_t cap) {
  typedef typename STraits<K>::Comp C;
  constexpr int V = 16 / (int)sizeof(K);  // keys of a 128-bit load
  constexpr uint32_t step = 64 * V;       // keys of a wave's load
  __shared__ C stage[kSFilterThreads / 64][kSWaveSlots];
  __shared__ uint32_t s_n[kSFilterThreads / 64];
  __shared__ uint32_t s_base;
  const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const uint32_t posmask = (uint32_t)((1ull << L) - 1);
  const C t = r <= m ? sorted[r - 1] : (C)0;
  const K tkey = (K)(t >> L);
  const uint32_t tpos = scomp_pos<C>(t, posmask);
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
  constexpr uint64_t tile = (uint64_t)step * U * (kSFilterThreads / 64);
  const uint64_t full = (n - head) / tile;
  for (uint64_t tl = blockIdx.x; tl < full; tl += gridDim.x) {
    const uint64_t lo = head + tl * tile + wave * step;
    K v[U][V];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const su32x4 x = __builtin_nontemporal_load(
          reinterpret_cast<const su32x4*>(keys + lo + (uint64_t)u * step * (kSFilterThreads / 64) + lane * V));
      __builtin_memcpy(v[u], &x, 16);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      K mx = 0;
#pragma unroll
      for (int c = 0; c < V; ++c) {
        v[u][c] = senc<K>(v[u][c], cd);
        mx = v[u][c] > mx ? v[u][c] : mx;
      }
      if (__ballot(mx >= tkey)) {
        const uint32_t p = (uint32_t)(lo + (uint64_t)u * step * (kSFilterThreads / 64)) + lane * V;
        if (fill + step > kSWaveSlots) flush();
#pragma unroll
        for (int c = 0; c < V; ++c)
          push(v[u][c] > tkey || (v[u][c] == tkey && p + c <= tpos), v[u][c], p + c);
      }
    }
  }
  // the keys the full tiles leave: the ones behind them, 64 a wave, then the head
  const uint64_t rest = full * tile;  // offset from the head
  for (uint64_t q0 = rest + ((uint64_t)blockIdx.x * (kSFilterThreads / 64) + wave) * 64; q0 < n;
       q0 += (uint64_t)gridDim.x * (kSFilterThreads / 64) * 64) {
    if (fill + 64 > kSWaveSlots) flush();
    const uint64_t q = q0 + lane;
    const uint64_t p = q < n - head ? q + head : q - (n - head);
    const K e = q < n ? senc<K>(keys[p], cd) : 0;
    push(q < n && (e > tkey || (e == tkey && (uint32_t)p <= tpos)), e, (uint32_t)p);
  }
  // the waves' remainders leave together: one device atomic per workgroup
  if (lane == 0) s_n[wave] = fill;
  __syncthreads();
  uint32_t off = 0, tot = 0;
#pragma unroll
  for (uint32_t w = 0; w < kSFilterThreads / 64; ++w) {
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
// Block-wide exclusive prefix sums of one value per thread (T threads, whole
// waves); *total is the sum.  s_w: T / 64 words.
template <int T>
__device__ __forceinline__ uint32_t sblock_scan(uint32_t x, uint32_t* s_w, uint32_t* total) {
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t y = x;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t z = (uint32_t)__shfl_up((int)y, o);
    if ((int)lane >= o) y += z;
  }
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
  const uint32_t lgP = 31u - (uint32_t)__clz((int)w.P), groups = (w.B - top) >> lgP;
  for (uint32_t g = t; g < groups; g += T) {
    const uint32_t qa = q0 + g * kSGroup, qb = qa + kSGroup < w.r ? qa + kSGroup : w.r;
    C x[kSGroup + 1];
#pragma unroll
    for (uint32_t i = 0; i <= kSGroup; ++i) {
      const uint32_t q = qa + i < qb ? qa + i : qb;
      x[i] = q <= m ? sorted[q - 1] : (C)0;
    }
    const C step = (x[0] - x[kSGroup]) >> lgP;
    // six (of four pieces: seven) of the nine samples inside one piece's
    // width: the keys are clustered here, the samples divide them better
    bool crowded = false;
    const bool four = w.P == 4;
#pragma unroll
    for (uint32_t i = 0; i + 5 <= kSGroup; ++i) crowded = crowded || (!four && x[i] - x[i + 5] < step);
#pragma unroll
    for (uint32_t i = 0; i + 6 <= kSGroup; ++i) crowded = crowded || (four && x[i] - x[i + 6] < step);
    for (uint32_t f = 1; f <= w.P; ++f) {
      C v = x[0] - step * f;
      if (crowded || f == w.P) {
        const uint32_t i = (f * kSGroup) >> lgP;
        const uint32_t q = qa + i < qb ? qa + i : qb;
        v = q <= m ? sorted[q - 1] : (C)0;
      }
      split[top + g * w.P + f - 1] = v;
    }
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
// written), or composites when the source holds them.
template <typename K, bool ARR, int ST>
struct SStage {
  K key[ST];
  uint32_t pos[ST];
  __device__ __forceinline__ void put(uint32_t i, K v, uint32_t p) {
    key[i] = v;
    pos[i] = p;
  }
  __device__ __forceinline__ typename STraits<K>::Comp get(uint32_t i, int L, uint32_t posmask) const {
    return scomp<K>(key[i], pos[i], L, posmask);
  }
};
template <typename K, int ST>
struct SStage<K, true, ST> {
  typename STraits<K>::Comp c[ST];
  __device__ __forceinline__ void put(uint32_t i, typename STraits<K>::Comp v, uint32_t) { c[i] = v; }
  __device__ __forceinline__ typename STraits<K>::Comp get(uint32_t i, int, uint32_t) const { return c[i]; }
};

// One pass over the source: counts the elements above the window, stages
// those inside it, and writes every full stage as one row of the candidate
// buffer, grouped by bucket.  A row's place costs one device atomic; the
// bucket's size and first output slot are sums over the rows' offsets, so no
// counting pass and no global scatter are needed.  One workgroup a CU.
template <typename K, bool ARR>
__global__ __launch_bounds__(kSPartThreads) void k_spart(const K* __restrict__ keys,
                                                         const typename STraits<K>::Comp* __restrict__ arr,
                                                         uint64_t n, uint32_t head, uint32_t cap1, uint32_t k,
                                                         uint32_t m, SCodec<K> cd, int L,
                                                         const typename STraits<K>::Comp* __restrict__ sorted,
                                                         SCtl* ctl, typename STraits<K>::Comp* __restrict__ out,
                                                         uint32_t cap, uint32_t maxrows, SRow* __restrict__ rows,
                                                         uint16_t* __restrict__ offs, uint32_t pitch) {
  typedef typename STraits<K>::Comp C;
  typedef typename std::conditional<ARR, C, K>::type R;
  constexpr int ST = STraits<K>::kStage, MB = STraits<K>::kMaxB, T = kSPartThreads;
  constexpr int NE = ST / T;                                       // elements a thread stages at most
  constexpr int V = ARR ? 16 / (int)sizeof(C) : 16 / (int)sizeof(K);  // elements of a 128-bit load
  constexpr int U = NE / V;
  static_assert(U >= 1 && NE % V == 0, "a tile is whole 128-bit loads");
  constexpr int BP = (MB + T - 1) / T;  // bucket counters a thread scans
  __shared__ SStage<K, ARR, ST> stage;
  __shared__ C split[MB];
  __shared__ uint32_t hist[MB + 1];
  __shared__ uint32_t s_w[T / 64], s_above;
  __shared__ uint32_t s_n, s_row, s_base;
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t posmask = (uint32_t)((1ull << L) - 1);
  uint64_t count = n;
  if constexpr (ARR) {
    count = (uint32_t)ctl->alloc1;
    if (count > cap1 || count < k) return;
  }
  const SWin w = ctl->win;
  const uint32_t B = w.B;
  sfill_splitters<C>(split, w, m, sorted, threadIdx.x, T);
  for (uint32_t b = threadIdx.x; b <= B; b += T) hist[b] = 0;
  if (threadIdx.x == 0) { s_n = 0; s_above = 0; }
  const C hi = w.a ? sorted[w.a - 1] : ~(C)0;
  const C lo = w.r <= m ? sorted[w.r - 1] : (C)0;
  const R hikey = ARR ? (R)hi : (R)(hi >> L), lokey = ARR ? (R)lo : (R)(lo >> L);
  const uint32_t hipos = scomp_pos<C>(hi, posmask), lopos = scomp_pos<C>(lo, posmask);
  uint32_t above = 0;  // wave-uniform
  __syncthreads();

  // Writes the `cnt` staged candidates as one row (every thread calls).
  auto flush = [&](uint32_t cnt) {
    if (above && lane == 0) atomicAdd(&s_above, above);
    above = 0;
    C c[NE];
    uint32_t at[NE];  // bucket << 16 | rank in it
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const uint32_t i = e * T + threadIdx.x;
      if (i < cnt) {
        c[e] = stage.get(i, L, posmask);
        uint32_t b0 = 0, len = B;  // splitters above c: the first len candidates of [b0, b0 + len)
        while (len) {
          const uint32_t h = len >> 1;
          const bool g = split[b0 + h] > c[e];
          b0 = g ? b0 + h + 1 : b0;
          len = g ? len - h - 1 : h;
        }
        at[e] = (b0 << 16) | atomicAdd(&hist[b0], 1u);
      }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      const uint64_t al = atomicAdd((unsigned long long*)&ctl->alloc, (1ull << 32) | cnt);
      s_row = (uint32_t)(al >> 32);
      s_base = (uint32_t)al;
    }
    uint32_t h[BP], sum = 0;
#pragma unroll
    for (int j = 0; j < BP; ++j) {
      const uint32_t b = threadIdx.x * BP + j;
      h[j] = b < B ? hist[b] : 0;
      sum += h[j];
    }
    uint32_t tot;
    uint32_t ex = sblock_scan<T>(sum, s_w, &tot);
#pragma unroll
    for (int j = 0; j < BP; ++j) {
      const uint32_t b = threadIdx.x * BP + j;
      if (b < B) hist[b] = ex;
      ex += h[j];
    }
    if (threadIdx.x == 0) hist[B] = cnt;
    __syncthreads();
    const uint32_t row = s_row, base = s_base;
    if (row < maxrows) {
      if (threadIdx.x == 0) rows[row] = SRow{base, s_above};
      for (uint32_t b = threadIdx.x; b <= B; b += T) offs[(size_t)row * pitch + b] = (uint16_t)hist[b];
    }
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const uint32_t i = e * T + threadIdx.x;
      if (i < cnt) {
        const uint64_t o = (uint64_t)base + hist[at[e] >> 16] + (at[e] & 0xFFFFu);
        if (o < cap) out[o] = c[e];
      }
    }
    __syncthreads();
    for (uint32_t b = threadIdx.x; b <= B; b += T) hist[b] = 0;
    if (threadIdx.x == 0) s_above = 0;
  };

  // Tiles of ST elements from the first 16-byte boundary on (head: the
  // elements before it, a last tile of their own).  A thread's loads of the
  // next tile are in flight while it works on the current one.
  const R* src;
  if constexpr (ARR) src = arr;
  else src = keys;
  constexpr uint32_t tile = ST;
  const uint64_t body = (count - head + tile - 1) / tile;
  const uint64_t ntile = body + (head ? 1 : 0);
  uint32_t staged = 0;  // block-uniform fill level
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
  load(blockIdx.x);
  for (uint64_t tl = blockIdx.x; tl < ntile; tl += gridDim.x) {
    const uint32_t valid = nvalid;
    const uint32_t p0 = tl == body ? threadIdx.x : head + (uint32_t)first(tl, 0);
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      if constexpr (ARR) cur[e] = nxt[e];
      else cur[e] = senc<K>(nxt[e], cd);
    }
    load(tl + gridDim.x);
    uint32_t wcnt = 0;
    uint64_t bal[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const uint32_t pos = p0 + (uint32_t)(e / V) * T * V + e % V;
      bal[e] = __ballot(cur[e] >= lokey);
      if constexpr (!ARR) {
        if (__ballot(cur[e] == lokey)) bal[e] &= ~__ballot(cur[e] == lokey && pos > lopos);
      }
      if (!__all(valid == (1u << NE) - 1)) bal[e] &= __ballot((valid >> e) & 1u);
      if (w.a) {
        uint64_t up = __ballot(cur[e] > hikey);
        if constexpr (!ARR) {
          if (__ballot(cur[e] == hikey)) up |= __ballot(cur[e] == hikey && pos < hipos);
        }
        up &= bal[e];
        above += (uint32_t)__popcll(up);
        bal[e] &= ~up;
      }
      wcnt += (uint32_t)__popcll(bal[e]);
    }
    uint32_t wbase = 0;
    if (lane == 0 && wcnt) wbase = atomicAdd(&s_n, wcnt);
    wbase = (uint32_t)__builtin_amdgcn_readfirstlane((int)wbase);
    __syncthreads();
    uint32_t now = s_n;
    if (now > (uint32_t)ST) {  // block-uniform: the tile does not fit beside what is staged
      flush(staged);
      if (threadIdx.x == 0) s_n = now - staged;
      wbase -= staged;
      now -= staged;
    }
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const uint32_t pos = p0 + (uint32_t)(e / V) * T * V + e % V;
      if (__builtin_amdgcn_inverse_ballot_w64(bal[e])) stage.put(wbase + mbcnt(bal[e]), cur[e], pos);
      wbase += (uint32_t)__popcll(bal[e]);
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

template <typename C>
__device__ __forceinline__ C sshfl_xor(C v, int o) {
  uint32_t w[sizeof(C) / 4];
  __builtin_memcpy(w, &v, sizeof(C));
#pragma unroll
  for (uint32_t i = 0; i < sizeof(C) / 4; ++i) w[i] = (uint32_t)__shfl_xor((int)w[i], o);
  __builtin_memcpy(&v, w, sizeof(C));
  return v;
}

// Largest and smallest over the workgroup, held by every thread.  red: T / 64
// pairs, free before and after.
template <typename C, int T>
__device__ __forceinline__ void sblock_minmax(C& mx, C& mn, C (*red)[2]) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const C a = sshfl_xor(mx, o), b = sshfl_xor(mn, o);
    mx = a > mx ? a : mx;
    mn = b < mn ? b : mn;
  }
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

// Sorts the N (<= CAP) composites held N = e * T + thread in c[] descending
// and calls emit(slot, composite) for each of the first `need` slots (and
// perhaps a few after them).  Linear bins over [min, max] (logarithmic from the
// top when at most a quarter is needed: the top of both float and integer keys
// is then spread over many bins whatever lies below), a scatter into LDS bin by
// bin, then each element's rank inside its bin; bins that start past `need`
// are left alone.  When a bin that counts is crowded (keys in far-apart
// clusters, floats of both signs) bins between samples instead.
template <typename C, uint32_t CAP, int T, int E, typename F>
__device__ __forceinline__ void ssort(SSortShared<C, CAP, T>& sm, C (&c)[E], uint32_t N, uint64_t need, F&& emit) {
  C mx = 0, mn = ~(C)0;
#pragma unroll
  for (int e = 0; e < E; ++e)
    if (e * T + threadIdx.x < N) {
      mx = c[e] > mx ? c[e] : mx;
      mn = c[e] < mn ? c[e] : mn;
    }
  for (int b = threadIdx.x; b <= kSBins; b += T) sm.hist[b] = 0;
  if (threadIdx.x == 0) sm.misc[0] = 0;
  sblock_minmax<C, T>(mx, mn, sm.red);
  const uint32_t bl = sbits((C)(mx - mn));
  const int sh = bl > 11 ? (int)bl - 11 : 0;
  const bool logb = need <= N / 4;
  uint32_t at[E];
#pragma unroll
  for (int e = 0; e < E; ++e)
    if (e * T + threadIdx.x < N) {
      const uint32_t b = logb ? slog_bin<C>(mx - c[e]) : (uint32_t)((mx - c[e]) >> sh);
      at[e] = (b << 16) | atomicAdd(&sm.hist[b], 1u);
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
    if (h[j] > 96u && ex < need) sm.misc[0] = 1;
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
          uint32_t rk = lo;
          for (uint32_t j = lo; j < hi; ++j) rk += sm.buf[j] > c[e] ? 1u : 0u;
          emit(rk, c[e]);
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
        uint32_t rk = lo;
        for (uint32_t j = lo; j < hi; ++j) rk += sm.buf[j] > c[e] ? 1u : 0u;
        emit(rk, c[e]);
      }
    }
  __syncthreads();
}

template <typename K>
struct SBucketShared : SSortShared<typename STraits<K>::Comp, STraits<K>::kCap, kSBucketThreads> {
  uint32_t pre[kSMaxRows + 1];  // bucket elements in the rows before this one
  uint32_t src[kSMaxRows];      // candidate index of the row's segment
};

template <typename K, int E, typename F>
__device__ __forceinline__ void sbucket_sort(SBucketShared<K>& sm, typename STraits<K>::Comp (&c)[E], uint32_t N,
                                             uint64_t need, F&& emit) {
  ssort<typename STraits<K>::Comp, STraits<K>::kCap, kSBucketThreads, E>(sm, c, N, need, emit);
}

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

// Collects the elements get(i), i < count, lying in [lo, hi] (N of them, at
// most CAP, known to the caller) into registers in sort order's layout.
template <typename C, uint32_t CAP, int T, int E, typename G>
__device__ __forceinline__ uint32_t sbucket_collect(SSortShared<C, CAP, T>& sm, C (&c)[E],
                                                    uint64_t count, C lo,
                                                    C hi, G&& get) {
  if (threadIdx.x == 0) sm.misc[1] = 0;
  __syncthreads();
  sbucket_each<C, T>(count, get, [&](C x) {
    if (x >= lo && x <= hi) {
      const uint32_t s = atomicAdd(&sm.misc[1], 1u);
      if (s < CAP) sm.buf[s] = x;
    }
  });
  __syncthreads();
  const uint32_t N = sm.misc[1] < CAP ? sm.misc[1] : CAP;
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

// The element of 1-based rank `rank` among get(i), i < count (all distinct).
template <typename C, uint32_t CAP, int T, typename G>
__device__ __forceinline__ C sbucket_select(SSortShared<C, CAP, T>& sm, uint64_t count,
                                                                    uint64_t rank, G&& get) {
  C mn = 0, mx = ~(C)0;
  for (;;) {
    const int sh = sbucket_hist<C, CAP, T>(sm, count, mn, mx, get);
    if (threadIdx.x == 0) sm.misc[2] = 0;
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

// One workgroup per bucket.  B buckets from the rows (PLAIN false), or the
// candidate buffer as the only bucket (PLAIN true).
template <typename K, bool PLAIN>
__global__ __launch_bounds__(kSBucketThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_sbucket(
    const K* __restrict__ keys, uint64_t n, uint32_t k, int kth_only, int levels, SCodec<K> cd, int L,
    const SCtl* __restrict__ ctl, const typename STraits<K>::Comp* __restrict__ cand, uint32_t cap1, uint32_t cap,
    uint32_t maxrows, const SRow* __restrict__ rows, const uint16_t* __restrict__ offs, uint32_t pitch, K* __restrict__ out_vals,
    uint32_t* __restrict__ out_idx, K* __restrict__ out_kth) {
  typedef typename STraits<K>::Comp C;
  constexpr int T = kSBucketThreads;
  constexpr uint32_t CAP = STraits<K>::kCap;
  constexpr int E = (int)(CAP + T - 1) / T;
  __shared__ SBucketShared<K> sm;
  const uint32_t posmask = (uint32_t)((1ull << L) - 1);
  const uint64_t al = ctl->alloc;
  const uint32_t nc = (uint32_t)al, nrows = (uint32_t)(al >> 32);
  uint64_t start = 0;  // elements ranked above the bucket
  uint32_t count = 0;
  auto emit = [&](uint64_t slot, C c) {  // slot: 0-based rank in the whole input
    if (slot >= k) return;
    const K v = sdec<K>((K)(c >> L), cd);
    if (!kth_only) {
      if (out_vals) out_vals[slot] = v;
      if (out_idx) out_idx[slot] = scomp_pos<C>(c, posmask);
    }
    if (out_kth && slot == k - 1) *out_kth = v;
  };
  bool bad = nc > cap;
  if (levels == 2) {
    const uint32_t c1 = (uint32_t)ctl->alloc1;
    bad = bad || c1 > cap1 || c1 < k;
  }
  C c[E];
  uint64_t total = 0, over = 0;  // elements at or above the cut; above the window
  if constexpr (PLAIN) {
    count = nc;
    total = nc;
  } else {
    bad = bad || nrows > maxrows;
    const uint32_t b = blockIdx.x;
    const uint32_t B = ctl->win.B;
    if (!bad) {
      // this bucket's segments: thread t takes rows 2t and 2t + 1
      static_assert(kSMaxRows == 2 * T, "two rows a thread");
      uint32_t len[2], sum = 0, before = 0, ab = 0;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const uint32_t r = 2 * threadIdx.x + j;
        len[j] = 0;
        if (r < nrows) {
          const SRow rw = rows[r];
          ab += rw.above;
          if (b < B) {
            const uint32_t o0 = offs[(size_t)r * pitch + b], o1 = offs[(size_t)r * pitch + b + 1];
            len[j] = o1 - o0;
            before += o0;
            sm.src[r] = rw.base + o0;
          }
        }
        sum += len[j];
      }
      uint32_t tb, ta;
      (void)sblock_scan<T>(before, sm.s_w, &tb);
      (void)sblock_scan<T>(ab, sm.s_w, &ta);
      uint32_t ex = sblock_scan<T>(sum, sm.s_w, &count);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        sm.pre[2 * threadIdx.x + j] = ex;
        ex += len[j];
      }
      if (threadIdx.x == T - 1) sm.pre[kSMaxRows] = ex;
      start = (uint64_t)ta + tb;
      over = ta;
      total = (uint64_t)ta + nc;
      __syncthreads();
    }
    if (!bad && total >= k && over < k) {
      if (b >= B || start >= k || count == 0) return;
      if (kth_only && start + count < k) return;
    }
  }
  if (bad || total < k || over >= k) {
    // rescue: the sample misjudged this input.  Each workgroup answers its
    // own ranks from the input, independently of the others.
    auto get = [&](uint64_t i) { return scomp<K>(senc<K>(keys[i], cd), (uint32_t)i, L, posmask); };
    if (kth_only) {
      if (blockIdx.x == 0) {
        const C x = sbucket_select<C, CAP, T>(sm, n, k, get);
        if (threadIdx.x == 0) emit((uint64_t)k - 1, x);
      }
      return;
    }
    for (uint64_t j = blockIdx.x; j * CAP < k; j += gridDim.x) {
      const uint64_t r0 = j * CAP, r1 = r0 + CAP < k ? r0 + CAP : k;
      const C hi = sbucket_select<C, CAP, T>(sm, n, r0 + 1, get);
      const C lo = sbucket_select<C, CAP, T>(sm, n, r1, get);
      const uint32_t N = sbucket_collect<C, CAP, T, E>(sm, c, n, lo, hi, get);
      sbucket_sort<K, E>(sm, c, N, N, [&](uint32_t rk, C x) { emit(r0 + rk, x); });
    }
    return;
  }
  auto get = [&](uint64_t i) {
    if constexpr (PLAIN) {
      return cand[i];
    } else {
      uint32_t r0 = 0;  // last row with pre <= i
#pragma unroll
      for (uint32_t h = kSMaxRows / 2; h >= 1; h >>= 1)
        if (sm.pre[r0 + h] <= (uint32_t)i) r0 += h;
      return cand[sm.src[r0] + ((uint32_t)i - sm.pre[r0])];
    }
  };
  if (count <= CAP) {
#pragma unroll
    for (int e = 0; e < E; ++e)
      if (e * T + threadIdx.x < count) c[e] = get(e * T + threadIdx.x);
    sbucket_sort<K, E>(sm, c, count, k - start, [&](uint32_t rk, C x) { emit(start + rk, x); });
    return;
  }
  // a bucket larger than the LDS: descending runs of at most CAP elements,
  // each the leading bins of a histogram of what is left
  uint64_t done = 0;
  C top = ~(C)0;  // elements above it are written
  while (done < count && start + done < k) {
    C mn = ~(C)0, mx = 0;
    sbucket_each<C, T>(count, get, [&](C x) {
      if (x <= top) {
        mx = x > mx ? x : mx;
        mn = x < mn ? x : mn;
      }
    });
    sblock_minmax<C, T>(mx, mn, sm.red);
    C cut = mn;
    for (;;) {
      const int sh = sbucket_hist<C, CAP, T>(sm, count, mn, mx, get);
      // the most leading bins whose elements fit
      if (threadIdx.x == 0) sm.misc[3] = 0;
      __syncthreads();
      for (uint32_t b = threadIdx.x; b < (uint32_t)kSBins; b += T)
        if (sm.hist[b + 1] <= CAP && (b + 1 == (uint32_t)kSBins || sm.hist[b + 2] > CAP)) sm.misc[3] = b + 1;
      __syncthreads();
      const uint32_t nb = sm.misc[3];
      __syncthreads();
      const C width = (C)(nb ? nb : 1u) << sh;  // composites of the kept bins
      const bool all = mx - mn < width;
      cut = all ? mn : mx - (width - 1);
      if (nb || sh == 0) break;
      mn = cut;  // the first bin alone is too large: look inside it
    }
    const uint32_t N = sbucket_collect<C, CAP, T, E>(sm, c, count, cut, mx, get);
    sbucket_sort<K, E>(sm, c, N, k - start - done, [&](uint32_t rk, C x) { emit(start + done + rk, x); });
    done += N;
    if (N == 0 || cut == 0) break;
    top = cut - 1;
  }
}

// ---------------------------------------------------------------------------
// The whole problem in one workgroup.  n <= CAP: every element goes into the
// sort.  Otherwise the r-th of 256 samples cuts the input to between k and
// CAP elements in one streaming pass, the survivors collected in LDS and
// sorted; when the sample misjudges that, the k-th element is found by
// histograms of the input instead.  k <= CAP.
template <typename K>
struct SOne {
  typedef typename STraits<K>::Comp C;
  static constexpr uint32_t kCap = 65536 / sizeof(C);
};

template <typename K, int T>
__global__ __launch_bounds__(T) void k_sone(const K* __restrict__ keys, uint32_t n, uint32_t k, uint32_t r,
                                            int kth_only, SCodec<K> cd, int L, K* __restrict__ out_vals,
                                            uint32_t* __restrict__ out_idx, K* __restrict__ out_kth) {
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
      const C kth = sbucket_select<C, CAP, T>(sm, n, k, get);
      N = sbucket_collect<C, CAP, T, E>(sm, c, n, kth, ~(C)0, get);
    } else {
#pragma unroll
      for (int e = 0; e < E; ++e)
        if (e * T + threadIdx.x < N) c[e] = sm.buf[e * T + threadIdx.x];
    }
    __syncthreads();
  }
  ssort<C, CAP, T, E>(sm, c, N, k, [&](uint32_t slot, C x) {
    if (slot >= k) return;
    const K v = sdec<K>((K)(x >> L), cd);
    if (!kth_only) {
      if (out_vals) out_vals[slot] = v;
      if (out_idx) out_idx[slot] = scomp_pos<C>(x, posmask);
    }
    if (out_kth && slot == k - 1) *out_kth = v;
  });
}

}  // namespace drtopk
