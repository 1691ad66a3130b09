// Many independent top-k problems in one launch.
//
// A workgroup (kBT threads, two share a CU, so one streams keys while the other
// sorts) takes one problem, by the rule in routes.h one of two ways:
//   b_stream: up to kBSmallN keys are sorted in LDS, more in one pass over them;
//   b_problem: up to kBSmallN keys are selected first (the k-th by radix select,
//     then the k at or above it sorted), more by the delegate method in one
//     workgroup's LDS.
// Problems of more than a slot's share of the batch's keys are split, and run
// the delegate method over several workgroups:
//   delegate vector (Rules 1 and 3): the top beta (1 or 2) of each subrange
//     of 2^alpha keys, built in LDS by waves streaming the keys, a tile a
//     workgroup, and published; the workgroup that arrives last goes on:
//   t = the k-th largest delegate: an LDS radix select over the delegates;
//   survivors (Rules 2 and 3): t itself, every element ranked >= t in the
//     subranges whose last delegate ranks above t (read as one virtual
//     concatenated vector), and with beta = 2 the first delegates above t of
//     the other subranges;
//   output: survivors sorted in registers, the first k written.
// When there are many tiles of split problems (k_batched_split), and for one
// problem alone (k_one), whole problems take b_problem too.  One whose delegate
// vector would not exceed k takes a block-level MSD radix select over its keys; one
// whose survivors overflow the LDS (adversarial inputs) is streamed after all, or
// radix-selected if split or claimed.  No workgroup ever waits for another.
#pragma once

#include "sample.h"
#include "tail.h"

namespace drtopk {

constexpr int kBT = 512;                  // threads per workgroup (two workgroups per CU)
constexpr int kBWaves = kBT / 64;
constexpr uint32_t kBSmallN = 4096;       // problems this small are selected in LDS directly
constexpr uint32_t kBMaxS = 4096;         // delegate vector capacity (LDS)
constexpr uint32_t kBMaxSG = 32768;       // delegate vector of a split problem (global memory)
constexpr uint32_t kBSurv = 4096;         // survivor capacity (LDS)
constexpr uint32_t kBMaxK = 2048;         // largest k handled in a workgroup
constexpr uint64_t kBMaxN = 1ull << 22;   // largest n handled in a workgroup
constexpr int kBU = 8;                    // 1 KiB wave loads in flight per wave step
constexpr uint32_t kBStep = 256 * kBU;    // keys per wave step
constexpr int kBufWord3 = 0x00020000;     // buffer resource word 3 for gfx9-family raw buffers
constexpr uint64_t kBSplitMinN = 1u << 16;  // problems above this may keep their delegate vector in global memory
constexpr uint32_t kBTileLog = 18;        // a split problem's delegate vector is built in tiles of
                                          // 2^max(kBTileLog, alpha) keys, one workgroup each (fewer where a
                                          // tile's delegates would not fit its LDS: at most 4096 entries)
__host__ __device__ constexpr uint32_t tile_log(uint32_t alpha, uint32_t beta) {
  return alpha + 12 - (beta > 1 ? 1 : 0) < kBTileLog ? alpha + 12 - (beta > 1 ? 1 : 0)
                                                     : (alpha > kBTileLog ? alpha : kBTileLog);
}

// One problem as the kernel sees it (64 bytes).
struct BatchDesc {
  const uint32_t* keys;
  uint64_t n;
  uint32_t k;
  uint32_t dtype;
  uint16_t alpha;  // subrange exponent, >= 2; 0 = radix select without delegates
  uint16_t beta;   // delegates per subrange (Rule 3): 1 or 2
  uint32_t tiles;  // > 1: the delegate vector is built by this many workgroups; 0: whole, by b_problem
  uint32_t* out_vals;
  uint32_t* out_idx;
  uint32_t* out_kth;
  uint64_t doff;   // tiles > 1: offset of the problem's delegate vector in the global buffer
};
static_assert(sizeof(BatchDesc) == 64, "BatchDesc layout");

struct BatchSmem {
  uint64_t D[kBMaxS];     // delegate composites; also the exchange buffer of small sorts
  uint64_t surv[kBSurv];  // survivors, also the exchange buffer of their sort
  uint32_t hist[kBins];   // digit histograms; then the list of qualifying subranges
  uint32_t wsum[kBWaves];
  uint32_t wbig[kBWaves];
  uint64_t red[2 * kBWaves];
  uint64_t sel;
  uint64_t tail_del;      // delegate of the subrange holding the last n mod 4 keys
  uint32_t nsurv;
  uint32_t nq;
  uint32_t item;
  uint32_t out[4];
};

template <int M>
__device__ __forceinline__ uint64_t max_cross(uint64_t m) {
  const uint64_t y = lane_cross64<M>(m);
  return y > m ? y : m;
}
// Maximum over each block of G consecutive lanes (G a wave-uniform power of
// two, at most 64), held by all of its lanes; VALU lane operations only.
__device__ __forceinline__ uint64_t group_max64(uint64_t m, uint32_t G) {
  if (G > 1) m = max_cross<1>(m);
  if (G > 2) m = max_cross<2>(m);
  if (G > 4) m = max_cross<4>(m);
  if (G > 8) m = max_cross<8>(m);
  if (G > 16) m = max_cross<16>(m);
  if (G > 32) m = max_cross<32>(m);
  return m;
}
__device__ __forceinline__ uint64_t wave_max64(uint64_t m) {
  return max_cross<32>(max_cross<16>(max_cross<8>(max_cross<4>(max_cross<2>(max_cross<1>(m))))));
}

// The top BETA (1 or 2) of a stream of distinct composites, m1 > m2 (0 =
// none yet; 0 is below every composite of a real element, so pushing it
// changes nothing).
template <int BETA>
__device__ __forceinline__ void top_push(uint64_t& m1, uint64_t& m2, uint64_t x) {
  if constexpr (BETA == 2) {
    const uint64_t lo = x < m1 ? x : m1;
    m2 = lo > m2 ? lo : m2;
  }
  m1 = x > m1 ? x : m1;
}
template <int BETA>
__device__ __forceinline__ void top_merge(uint64_t& m1, uint64_t& m2, uint64_t b1, uint64_t b2) {
  if constexpr (BETA == 2) {
    const uint64_t lo = b1 < m1 ? b1 : m1;
    const uint64_t hi2 = b2 > m2 ? b2 : m2;
    m2 = lo > hi2 ? lo : hi2;
  }
  m1 = b1 > m1 ? b1 : m1;
}
template <int BETA, int M>
__device__ __forceinline__ void top_cross(uint64_t& m1, uint64_t& m2) {
  const uint64_t b1 = lane_cross64<M>(m1);
  const uint64_t b2 = BETA == 2 ? lane_cross64<M>(m2) : 0ull;
  top_merge<BETA>(m1, m2, b1, b2);
}
// Top BETA over each block of G consecutive lanes (G a wave-uniform power of
// two, at most 64), held by all of its lanes.
template <int BETA>
__device__ __forceinline__ void group_top(uint64_t& m1, uint64_t& m2, uint32_t G) {
  if (G > 1) top_cross<BETA, 1>(m1, m2);
  if (G > 2) top_cross<BETA, 2>(m1, m2);
  if (G > 4) top_cross<BETA, 4>(m1, m2);
  if (G > 8) top_cross<BETA, 8>(m1, m2);
  if (G > 16) top_cross<BETA, 16>(m1, m2);
  if (G > 32) top_cross<BETA, 32>(m1, m2);
}

// Folds a block's top BETA (m1 > m2) into subrange j of an LDS delegate
// vector of BETA entries per subrange (zeroed first).  BETA 1: an atomic
// maximum.  BETA 2: m1 goes into the first entry by an atomic maximum, and
// the larger of m2 and whichever of m1 and the displaced value is smaller
// into the second.  Each update of the first entry hands the smaller of its
// two values to the second, so every value except the overall maximum
// reaches the second entry once: it ends as the runner-up in any order of
// updates.
template <int BETA>
__device__ __forceinline__ void d_fold(uint64_t* D, uint32_t j, uint64_t m1, uint64_t m2) {
  if constexpr (BETA == 1) {
    atomicMax((unsigned long long*)&D[j], (unsigned long long)m1);
  } else {
    const uint64_t old = atomicMax((unsigned long long*)&D[2 * j], (unsigned long long)m1);
    const uint64_t lo = old < m1 ? old : m1;
    const uint64_t v = lo > m2 ? lo : m2;
    if (v) atomicMax((unsigned long long*)&D[2 * j + 1], (unsigned long long)v);
  }
}

// The keys of one problem behind a raw buffer resource: loads are plain
// buffer loads (base address in scalar registers, 32-bit offsets), and whole
// dwords at or beyond `nrec` keys read 0.  VEC: 16-byte loads of 4 keys at a
// multiple of 4 (the base is 16-byte aligned and nrec a multiple of 4, so a
// load is either wholly inside or wholly outside); otherwise 4-byte loads.
template <bool VEC>
struct Keys {
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ Keys(const uint32_t* p, uint32_t nrec)
      : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(p), (short)0, (int)(nrec * 4u), kBufWord3)) {}
  // NT: read once, not to be kept in the caches
  template <int NT = 0>
  __device__ __forceinline__ void load4(uint32_t p, uint32_t (&v)[4]) const {
    if constexpr (VEC) {
      const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(r, (int)(p * 4u), 0, NT ? 2 : 0);
      v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c) v[c] = __builtin_amdgcn_raw_buffer_load_b32(r, (int)((p + c) * 4u), 0, 0);
    }
  }
};

// Keys [0, n4) go through the streaming loops; with 16-byte loads n4 = n
// rounded down to a multiple of 4 and the last n - n4 keys are read one by one.
template <bool VEC>
__device__ __forceinline__ uint32_t vec_end(uint32_t n) {
  return VEC ? (n & ~3u) : n;
}

// Bin holding the rank-th largest entry of an LDS histogram (each thread owns
// kBins / kBT consecutive bins, highest first; wave prefix sums, one barrier):
// sm.out = {bin, rank within the bin, found, count of the bin}.
__device__ inline void bb_bucket(const uint32_t* h, uint32_t rank, BatchSmem& sm) {
  constexpr int PER = kBins / kBT;
  const int t = threadIdx.x;
  const uint32_t lane = lane_id(), wave = t >> 6;
  uint32_t c[PER], sum = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    c[j] = h[kBins - 1 - PER * t - j];
    sum += c[j];
  }
  uint32_t x = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = (uint32_t)__shfl_up((int)x, o);
    if ((int)lane >= o) x += y;
  }
  if (lane == 63) sm.wsum[wave] = x;
  if (t == 0) { sm.out[0] = 0; sm.out[1] = 0; sm.out[2] = 0; sm.out[3] = 0; }
  __syncthreads();
  uint32_t excl = x - sum;
  for (uint32_t w = 0; w < wave; ++w) excl += sm.wsum[w];
  if (excl < rank && rank <= excl + sum) {
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      if (excl < rank && rank <= excl + c[j]) {
        sm.out[0] = kBins - 1 - PER * t - j;
        sm.out[1] = rank - excl;
        sm.out[3] = c[j];
        sm.out[2] = 1;
      }
      excl += c[j];
    }
  }
  __syncthreads();
}

// Key codec of a batched problem, applied at run time so one kernel serves
// batches that mix key types and orders: enc(b) = b ^ (sign(b) & a) ^ c
// equals enc<DT> of the problem's codec (float32: a = 0x7FFFFFFF, c = the
// sign bit; int32: a = 0, c = the sign bit; uint32: both 0; the k smallest:
// c complemented).  a leaves bit 31 alone, so b ^ (sign(b) & a) keeps b's
// sign and dec recovers b from it.
struct Codec {
  uint32_t a, c;
  __device__ __forceinline__ uint32_t enc(uint32_t b) const {
    return b ^ ((uint32_t)((int32_t)b >> 31) & a) ^ c;
  }
  __device__ __forceinline__ uint32_t dec(uint32_t e) const {
    const uint32_t v = e ^ c;
    return v ^ ((uint32_t)((int32_t)v >> 31) & a);
  }
};
__device__ __forceinline__ Codec codec_of(uint32_t code) {
  Codec x;
  x.a = (code & 3u) == (uint32_t)DT_F32 ? 0x7FFFFFFFu : 0u;
  x.c = ((code & 3u) == (uint32_t)DT_U32 ? 0u : 0x80000000u) ^ ((code & (uint32_t)DT_MIN) ? 0xFFFFFFFFu : 0u);
  return x;
}
__device__ __forceinline__ void b_write_out(uint64_t c, uint32_t r, uint32_t k, uint32_t* out_vals, uint32_t* out_idx,
                                            uint32_t* out_kth, Codec cx) {
  const uint32_t v = cx.dec(comp_key(c));
  if (out_vals) out_vals[r] = v;
  if (out_idx) out_idx[r] = comp_pos(c);
  if (out_kth && r == k - 1) *out_kth = v;
}

// Wave-wide append to an LDS list: the lanes with `pred` take consecutive
// slots from *count with one LDS atomic per wave (whole wave active); slots at
// or past cap are counted but not stored.
__device__ __forceinline__ void lds_append(bool pred, uint64_t x, uint32_t* count, uint64_t* list, uint32_t cap) {
  const uint64_t b = __ballot(pred);
  if (!b) return;
  const int leader = __ffsll((unsigned long long)b) - 1;
  uint32_t base = 0;
  if ((int)lane_id() == leader) base = atomicAdd(count, (uint32_t)__popcll(b));
  base = (uint32_t)__shfl((int)base, leader) + mbcnt(b);
  if (pred && base < cap) list[base] = x;
}

// Sorts `cnt` composites from LDS array `src` and writes the first `k` as
// outputs 0..k-1.  `src` holds at least E * kBT entries and serves as the
// exchange buffer of the sort once every thread has loaded its elements.
template <int E>
__device__ __noinline__ void b_sort_write_e(uint64_t* src, uint32_t cnt, uint32_t k, uint32_t* out_vals,
                                            uint32_t* out_idx, uint32_t* out_kth, Codec cx) {
  uint64_t v[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const uint32_t g = threadIdx.x * E + e;
    v[e] = g < cnt ? src[g] : 0ull;
  }
  block_bitonic<E, kBT>(v, src);
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const uint32_t g = threadIdx.x * E + e;
    if (g < k) b_write_out(v[e], g, k, out_vals, out_idx, out_kth, cx);
  }
}

// Bucket-rank sort of the cnt (<= E * kBT) distinct composites src[0..cnt),
// writing the first k as outputs: the composites are binned by the top 11
// bits of their distance from the smallest (bin 0 holds the largest),
// counted in `bins` (kBins words), scattered bin by bin into `buf`, and each
// takes the slot (start of its bin) + (number of larger composites in its
// bin).  Gives up (false, nothing written) when a bin holds more than
// kRankMaxBin: keys crowded into a narrow range go to the network instead.
template <int E>
__device__ __noinline__ bool b_rank_write_e(const uint64_t* src, uint32_t cnt, uint32_t k, uint32_t* out_vals,
                                            uint32_t* out_idx, uint32_t* out_kth, Codec cx, uint64_t* buf,
                                            uint32_t* bins, BatchSmem& sm) {
  constexpr int NW = kBWaves, PER = kBins / kBT;
  const uint32_t t = threadIdx.x, lane = lane_id(), w = t >> 6;
  uint64_t v[E];
  uint64_t mx = 0, nmn = 0;  // largest composite, and the complement of the smallest
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const uint32_t g = e * kBT + t;
    v[e] = g < cnt ? src[g] : 0ull;
    if (g < cnt) {
      mx = v[e] > mx ? v[e] : mx;
      nmn = ~v[e] > nmn ? ~v[e] : nmn;
    }
  }
  mx = wave_max64(mx);
  nmn = wave_max64(nmn);
  __syncthreads();  // src may alias the reduction slots' neighbours: every load done
  if (lane == 0) {
    sm.red[w] = mx;
    sm.red[NW + w] = nmn;
  }
  for (int i = t; i < kBins; i += kBT) bins[i] = 0;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    mx = sm.red[i] > mx ? sm.red[i] : mx;
    nmn = sm.red[NW + i] > nmn ? sm.red[NW + i] : nmn;
  }
  const uint64_t lo = ~nmn;
  const uint32_t bits = bitlen64(mx - lo);
  const uint32_t sh = bits > 11u ? bits - 11u : 0u;
  uint32_t b[E], r[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const uint32_t g = e * kBT + t;
    b[e] = (uint32_t)(kBins - 1) - (uint32_t)((v[e] - lo) >> sh);
    r[e] = g < cnt ? atomicAdd(&bins[b[e]], 1u) : 0u;
  }
  __syncthreads();
  uint32_t c[PER], sum = 0, big = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    c[j] = bins[t * PER + j];
    sum += c[j];
    big = c[j] > big ? c[j] : big;
  }
  uint32_t inc = sum;
#pragma unroll
  for (uint32_t d = 1; d < 64; d <<= 1) {
    const uint32_t y = (uint32_t)__shfl_up((int)inc, d);
    if (lane >= d) inc += y;
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const uint32_t y = (uint32_t)__shfl_xor((int)big, o);
    big = y > big ? y : big;
  }
  if (lane == 63) sm.wsum[w] = inc;
  if (lane == 0) sm.wbig[w] = big;
  __syncthreads();
  uint32_t off = inc - sum;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    if ((uint32_t)i < w) off += sm.wsum[i];
    big = sm.wbig[i] > big ? sm.wbig[i] : big;
  }
  if (big > kRankMaxBin) {  // block-uniform
    __syncthreads();
    return false;
  }
  __syncthreads();  // every count read before it becomes a bin start
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    bins[t * PER + j] = off;
    off += c[j];
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < E; ++e)
    if (e * kBT + t < cnt) buf[bins[b[e]] + r[e]] = v[e];
  __syncthreads();
#pragma unroll
  for (int e = 0; e < E; ++e) {
    if (e * kBT + t >= cnt) continue;
    const uint32_t st = bins[b[e]], en = b[e] + 1 < (uint32_t)kBins ? bins[b[e] + 1] : cnt;
    uint32_t slot = st;
    for (uint32_t j = st; j < en; ++j) slot += buf[j] > v[e] ? 1u : 0u;
    if (slot < k) b_write_out(v[e], slot, k, out_vals, out_idx, out_kth, cx);
  }
  __syncthreads();  // the caller reuses the LDS
  return true;
}

// cnt <= kBT * 8, k <= cnt.  `buf` (cnt entries) and `bins` (kBins words) are
// free LDS that the bucket-rank sort may use; src must not alias them.
__device__ inline void b_sort_write(uint64_t* src, uint32_t cnt, uint32_t k, uint32_t* out_vals, uint32_t* out_idx,
                                    uint32_t* out_kth, Codec cx, uint64_t* buf, uint32_t* bins, BatchSmem& sm) {
  if (cnt > 1u * kBT) {
    bool done;
    if (cnt <= 2u * kBT) done = b_rank_write_e<2>(src, cnt, k, out_vals, out_idx, out_kth, cx, buf, bins, sm);
    else if (cnt <= 4u * kBT) done = b_rank_write_e<4>(src, cnt, k, out_vals, out_idx, out_kth, cx, buf, bins, sm);
    else done = b_rank_write_e<8>(src, cnt, k, out_vals, out_idx, out_kth, cx, buf, bins, sm);
    if (done) return;
  }
  if (cnt <= 1u * kBT) b_sort_write_e<1>(src, cnt, k, out_vals, out_idx, out_kth, cx);
  else if (cnt <= 2u * kBT) b_sort_write_e<2>(src, cnt, k, out_vals, out_idx, out_kth, cx);
  else if (cnt <= 4u * kBT) b_sort_write_e<4>(src, cnt, k, out_vals, out_idx, out_kth, cx);
  else b_sort_write_e<8>(src, cnt, k, out_vals, out_idx, out_kth, cx);
}

// The rank-th largest (1-based) of the distinct composites a[0..cnt) in LDS:
// MSD radix select, one 11/11/10-bit digit per pass, stopping once the class
// holding rank r has a single member.  Identical in every thread.
__device__ inline uint64_t lds_select(const uint64_t* a, uint32_t cnt, uint32_t rank, BatchSmem& sm) {
  uint64_t prefix = 0, mask = 0;
  uint32_t r = rank;
  for (int p = 0; p < kPasses; ++p) {
    for (int i = threadIdx.x; i < kBins; i += kBT) sm.hist[i] = 0;
    __syncthreads();
    const int sh = pass_shift(p);
    const uint32_t dm = (1u << pass_bits(p)) - 1;
    for (uint32_t i = threadIdx.x; i < cnt; i += kBT) {
      const uint64_t x = a[i];
      if ((x & mask) == prefix) atomicAdd(&sm.hist[(uint32_t)(x >> sh) & dm], 1u);
    }
    __syncthreads();
    bb_bucket(sm.hist, r, sm);
    prefix |= (uint64_t)sm.out[0] << sh;
    mask |= (uint64_t)dm << sh;
    r = sm.out[1];
    if (sm.out[3] == 1u) break;  // always so after the last digit
  }
  for (uint32_t i = threadIdx.x; i < cnt; i += kBT) {
    const uint64_t x = a[i];
    if ((x & mask) == prefix) sm.sel = x;  // the class's single member
  }
  __syncthreads();
  const uint64_t t = sm.sel;
  __syncthreads();
  return t;
}

// Problems of at most kBSmallN keys: composites into LDS, the k-th by radix
// select, the k at or above it compacted and sorted.
template <bool VEC>
__device__ inline void b_small(const BatchDesc& d, BatchSmem& sm) {
  const Codec cx = codec_of(d.dtype);
  const uint32_t n = (uint32_t)d.n, k = d.k, n4 = vec_end<VEC>(n);
  const Keys<VEC> ks(d.keys, n4);
  for (uint32_t i = threadIdx.x * 4; i < n4; i += kBT * 4) {
    uint32_t v[4];
    ks.load4(i, v);
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (i + c < n4) sm.surv[i + c] = comp(cx.enc(v[c]), i + c);
  }
  if (threadIdx.x == 0)
    for (uint32_t i = n4; i < n; ++i) sm.surv[i] = comp(codec_of(d.dtype).enc(d.keys[i]), i);
  __syncthreads();
  uint32_t cnt = n;
  uint64_t* src = sm.surv;
  if (k < n) {
    const uint64_t T = lds_select(sm.surv, n, k, sm);
    if (threadIdx.x == 0) sm.nsurv = 0;
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < n; i += kBT) {
      const uint64_t x = sm.surv[i];
      if (x >= T) sm.D[atomicAdd(&sm.nsurv, 1u)] = x;  // exactly k
    }
    __syncthreads();
    cnt = k;
    src = sm.D;
  }
  b_sort_write(src, cnt, k, d.out_vals, d.out_idx, d.out_kth, codec_of(d.dtype), src == sm.D ? sm.surv : sm.D,
               sm.hist, sm);
}

// Block-level MSD radix select over the problem's 64-bit composites: each
// pass histograms one digit of the elements in the current class (those
// matching the digits chosen so far) and picks the bin holding rank r.  As
// soon as the elements ranked above the class plus the class itself fit the
// LDS, they are compacted, sorted and the first k written: two passes over
// the keys for typical inputs, at most seven for massive ties.
template <bool VEC>
__device__ inline void b_radix(const BatchDesc& d, BatchSmem& sm, uint32_t* rec) {
  const Codec cx = codec_of(d.dtype);
  const uint32_t n = (uint32_t)d.n, k = d.k, n4 = vec_end<VEC>(n);
  const Keys<VEC> ks(d.keys, n4);
  const uint32_t lane = lane_id(), wave = threadIdx.x >> 6;
  uint64_t prefix = 0, mask = 0;
  uint32_t r = k, above = 0;
  for (int p = 0; p < kPasses; ++p) {
    for (int i = threadIdx.x; i < kBins; i += kBT) sm.hist[i] = 0;
    __syncthreads();
    const int sh = pass_shift(p);
    const uint32_t dm = (1u << pass_bits(p)) - 1;
    for (uint32_t base = wave * kBStep; base < n4; base += kBWaves * kBStep) {
      uint32_t v[kBU][4];
#pragma unroll
      for (int j = 0; j < kBU; ++j) ks.load4(base + j * 256 + lane * 4, v[j]);
#pragma unroll
      for (int j = 0; j < kBU; ++j)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const uint32_t i = base + j * 256 + lane * 4 + c;
          const uint64_t x = comp(cx.enc(v[j][c]), i);
          if (i < n4 && (x & mask) == prefix) atomicAdd(&sm.hist[(uint32_t)(x >> sh) & dm], 1u);
        }
    }
    if (threadIdx.x == 0)
      for (uint32_t i = n4; i < n; ++i) {
        const uint64_t x = comp(codec_of(d.dtype).enc(d.keys[i]), i);
        if ((x & mask) == prefix) atomicAdd(&sm.hist[(uint32_t)(x >> sh) & dm], 1u);
      }
    __syncthreads();
    bb_bucket(sm.hist, r, sm);
    prefix |= (uint64_t)sm.out[0] << sh;
    mask |= (uint64_t)dm << sh;
    above += r - sm.out[1];
    r = sm.out[1];
    if (above + sm.out[3] <= kBSurv) break;  // always true after the last pass (class of one)
  }
  // every element ranked above the class, and the class: (x & mask) >= prefix
  if (threadIdx.x == 0) sm.nsurv = 0;
  __syncthreads();
  for (uint32_t base = wave * kBStep; base < n4; base += kBWaves * kBStep) {
    uint32_t v[kBU][4];
#pragma unroll
    for (int j = 0; j < kBU; ++j) ks.load4(base + j * 256 + lane * 4, v[j]);
#pragma unroll
    for (int j = 0; j < kBU; ++j)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const uint32_t i = base + j * 256 + lane * 4 + c;
        const uint64_t x = comp(cx.enc(v[j][c]), i);
        lds_append(i < n4 && (x & mask) >= prefix, x, &sm.nsurv, sm.surv, kBSurv);
      }
  }
  if (threadIdx.x == 0)
    for (uint32_t i = n4; i < n; ++i) {
      const uint64_t x = comp(codec_of(d.dtype).enc(d.keys[i]), i);
      if ((x & mask) >= prefix) {
        const uint32_t slot = atomicAdd(&sm.nsurv, 1u);
        if (slot < kBSurv) sm.surv[slot] = x;
      }
    }
  __syncthreads();
  const uint32_t ns = sm.nsurv < kBSurv ? sm.nsurv : kBSurv;
  // the class chosen last fits by construction (a single member after the last digit)
  if (threadIdx.x == 0 && sm.nsurv > kBSurv) record_err(rec, ERR_CAP);
  b_sort_write(sm.surv, ns, k, d.out_vals, d.out_idx, d.out_kth, codec_of(d.dtype), sm.D, sm.hist, sm);
}

// Delegate vector for subranges of at least 256 keys, over the keys
// [lo, min(hi, n4)) (lo a multiple of kBStep and of 2^alpha): waves stream
// them in steps of kBStep with kBU 1 KiB loads in flight; each 256-key block
// lies inside one subrange s, whose BETA entries (from sm.D[(s - lo /
// 2^alpha) * BETA]) take the block's top BETA by LDS atomics (D starts at 0,
// below every composite of a real element).
template <bool VEC, int BETA>
__device__ inline void b_delegates_wide(const Keys<VEC>& ks, uint32_t lo, uint32_t hi, uint32_t n4, uint32_t alpha,
                                        Codec cx, BatchSmem& sm) {
  const uint32_t L = 1u << alpha;
  const uint32_t end = hi < n4 ? hi : n4;
  const uint32_t s0 = lo >> alpha;
  const uint32_t lane = lane_id(), wave = threadIdx.x >> 6;
  for (uint32_t base = lo + wave * kBStep; base < end; base += kBWaves * kBStep) {
    uint32_t v[kBU][4];
#pragma unroll
    for (int j = 0; j < kBU; ++j) ks.load4(base + j * 256 + lane * 4, v[j]);
    if (L >= kBStep) {
      uint64_t m1 = 0, m2 = 0;
#pragma unroll
      for (int j = 0; j < kBU; ++j)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const uint32_t p = base + j * 256 + lane * 4 + c;
          const uint64_t x = comp(cx.enc(v[j][c]), p);
          top_push<BETA>(m1, m2, p < end ? x : 0ull);
        }
      group_top<BETA>(m1, m2, 64);
      if (lane == 0) d_fold<BETA>(sm.D, (base >> alpha) - s0, m1, m2);
    } else {
#pragma unroll
      for (int j = 0; j < kBU; ++j) {
        uint64_t m1 = 0, m2 = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const uint32_t p = base + j * 256 + lane * 4 + c;
          const uint64_t x = comp(cx.enc(v[j][c]), p);
          top_push<BETA>(m1, m2, p < end ? x : 0ull);
        }
        group_top<BETA>(m1, m2, 64);
        if (lane == 0 && base + j * 256 < end) d_fold<BETA>(sm.D, ((base + j * 256) >> alpha) - s0, m1, m2);
      }
    }
  }
}

// The last n mod 4 keys (16-byte loads stop at n4), all in one subrange:
// one thread folds them into that subrange's delegates (index n4 / 2^alpha - s0).
template <int BETA>
__device__ __forceinline__ void b_delegates_tail(const BatchDesc& d, uint32_t n4, uint32_t s0, BatchSmem& sm) {
  const uint32_t n = (uint32_t)d.n;
  if (threadIdx.x == 0 && n4 < n) {
    uint64_t m1 = 0, m2 = 0;
    for (uint32_t i = n4; i < n; ++i) top_push<BETA>(m1, m2, comp(codec_of(d.dtype).enc(d.keys[i]), i));
    d_fold<BETA>(sm.D, (n4 >> d.alpha) - s0, m1, m2);
  }
}

// Delegate vector for subranges of 4..128 keys, over the keys
// [lo, min(hi, n4)) (lo a multiple of kBStep): each 256-key wave-load holds
// whole subranges, 2^(alpha-2) lanes each; a segmented butterfly gives each
// subrange's top BETA to its first lane, which folds them into entries
// (s - lo / 2^alpha) * BETA.. of sm.D.
template <bool VEC, int BETA>
__device__ inline void b_delegates_narrow(const Keys<VEC>& ks, uint32_t lo, uint32_t hi, uint32_t n4,
                                          uint32_t alpha, Codec cx, BatchSmem& sm) {
  const uint32_t G = 1u << (alpha - 2);  // lanes per subrange
  const uint32_t end = hi < n4 ? hi : n4;
  const uint32_t s0 = lo >> alpha;
  const uint32_t lane = lane_id(), wave = threadIdx.x >> 6;
  for (uint32_t base = lo + wave * kBStep; base < end; base += kBWaves * kBStep) {
    uint32_t v[kBU][4];
#pragma unroll
    for (int j = 0; j < kBU; ++j) ks.load4(base + j * 256 + lane * 4, v[j]);
#pragma unroll
    for (int j = 0; j < kBU; ++j) {
      const uint32_t p = base + j * 256 + lane * 4;
      uint64_t m1 = 0, m2 = 0;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const uint64_t x = comp(cx.enc(v[j][c]), p + c);
        top_push<BETA>(m1, m2, p + c < end ? x : 0ull);
      }
      group_top<BETA>(m1, m2, G);
      if ((lane & (G - 1)) == 0 && p < end) d_fold<BETA>(sm.D, (p >> alpha) - s0, m1, m2);
    }
  }
}

// Survivors: every element ranked >= t in the nq subranges listed in Q,
// read as one virtual vector of nq * 2^alpha keys in 4-key pieces (a piece
// never crosses a subrange).
template <bool VEC>
__device__ inline void b_survivors(const Keys<VEC>& ks, uint32_t n4, uint32_t nq, uint32_t alpha, const uint32_t* Q,
                                   uint64_t t, Codec cx, BatchSmem& sm) {
  const uint32_t L = 1u << alpha;
  const uint32_t total = nq << alpha;
  const uint32_t lane = lane_id(), wave = threadIdx.x >> 6;
  for (uint32_t base = wave * kBStep; base < total; base += kBWaves * kBStep) {
    uint32_t v[kBU][4], pb[kBU];
#pragma unroll
    for (int j = 0; j < kBU; ++j) {
      const uint32_t e = base + j * 256 + lane * 4;
      // past the virtual vector: a position at n4 or beyond reads zeros and is ignored
      pb[j] = e < total ? (Q[e >> alpha] << alpha) + (e & (L - 1)) : n4;
      ks.load4(pb[j], v[j]);
    }
#pragma unroll
    for (int j = 0; j < kBU; ++j)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const uint32_t p = pb[j] + c;
        const uint64_t x = comp(cx.enc(v[j][c]), p);
        lds_append(p < n4 && x >= t, x, &sm.nsurv, sm.surv, kBSurv);
      }
  }
}

// Everything after the delegate vector: t, the qualifying subranges, the
// survivors and the output.  sm.D[0..cnt) holds every delegate ranked at or
// above the k-th (the whole vector, or its top part when a split problem's
// vector lives in global memory), BETA = 2 as (first, second) pairs of one
// subrange each; sm.tail_del is the last delegate of the subrange holding
// the last n mod 4 keys.
//   BETA 1: the k-1 subranges whose delegate ranks above t are re-read.
//   BETA 2 (Rule 3): a subrange is re-read only if its second delegate ranks
//     above t (at most (k-1)/2 of them); of any other subrange only its
//     first delegate can rank above t (every other element is at most its
//     second delegate, so at most t), and that delegate survives as is.
// t itself survives once: its subrange is never re-read.  False if the
// survivors overflow LDS (nothing has been written then).
template <bool VEC, int BETA>
__device__ inline bool b_finish(const BatchDesc& d, uint32_t cnt, BatchSmem& sm) {
  const uint32_t n = (uint32_t)d.n, k = d.k, alpha = d.alpha, n4 = vec_end<VEC>(n);
  const Keys<VEC> ks(d.keys, n4);
  const uint64_t t = lds_select(sm.D, cnt, k, sm);  // Rule 2: the k-th delegate
  uint32_t* Q = sm.hist;  // the subranges to re-read (order irrelevant)
  if (threadIdx.x == 0) { sm.nq = 0; sm.nsurv = 1; sm.surv[0] = t; }
  __syncthreads();
  if constexpr (BETA == 1) {
    for (uint32_t i = threadIdx.x; i < cnt; i += kBT) {
      const uint64_t x = sm.D[i];
      if (x > t) Q[atomicAdd(&sm.nq, 1u)] = comp_pos(x) >> alpha;
    }
  } else {
    for (uint32_t i = threadIdx.x; i < cnt / 2; i += kBT) {
      const uint64_t a = sm.D[2 * i], b = sm.D[2 * i + 1];
      if (b > t) Q[atomicAdd(&sm.nq, 1u)] = comp_pos(b) >> alpha;
      else if (a > t) sm.surv[atomicAdd(&sm.nsurv, 1u)] = a;  // fewer than k of them
    }
  }
  __syncthreads();
  b_survivors<VEC>(ks, n4, sm.nq, alpha, Q, t, codec_of(d.dtype), sm);
  if (threadIdx.x == 0 && n4 < n && sm.tail_del > t) {  // the last keys, when their subrange is re-read
    for (uint32_t i = n4; i < n; ++i) {
      const uint64_t x = comp(codec_of(d.dtype).enc(d.keys[i]), i);
      if (x >= t) {
        const uint32_t slot = atomicAdd(&sm.nsurv, 1u);
        if (slot < kBSurv) sm.surv[slot] = x;
      }
    }
  }
  __syncthreads();
  const uint32_t ns = sm.nsurv;
  if (ns > kBSurv) return false;
  b_sort_write(sm.surv, ns, k, d.out_vals, d.out_idx, d.out_kth, codec_of(d.dtype), sm.D, sm.hist, sm);
  return true;
}

template <bool VEC, int BETA>
__device__ inline void b_delegates(const Keys<VEC>& ks, uint32_t lo, uint32_t hi, uint32_t n4, uint32_t alpha,
                                   Codec cx, BatchSmem& sm) {
  if (alpha >= 8) b_delegates_wide<VEC, BETA>(ks, lo, hi, n4, alpha, cx, sm);
  else b_delegates_narrow<VEC, BETA>(ks, lo, hi, n4, alpha, cx, sm);
}

// The delegate method for one problem in one workgroup; false if the
// survivors overflow LDS (nothing has been written then).
template <bool VEC, int BETA>
__device__ inline bool b_delegate(const BatchDesc& d, BatchSmem& sm) {
  const uint32_t n = (uint32_t)d.n, alpha = d.alpha, n4 = vec_end<VEC>(n);
  const uint32_t E = ((n + (1u << alpha) - 1) >> alpha) * BETA;
  const Keys<VEC> ks(d.keys, n4);
  for (uint32_t i = threadIdx.x; i < E; i += kBT) sm.D[i] = 0;
  __syncthreads();
  b_delegates<VEC, BETA>(ks, 0, n, n4, alpha, codec_of(d.dtype), sm);
  b_delegates_tail<BETA>(d, n4, 0, sm);
  __syncthreads();
  if (threadIdx.x == 0) sm.tail_del = n4 < n ? sm.D[(n4 >> alpha) * BETA + BETA - 1] : 0;
  return b_finish<VEC, BETA>(d, E, sm);
}

// A split problem's delegate vector (S subranges of BETA entries, global
// memory, written by the tiles' workgroups with coherent stores) cut down to
// LDS: MSD digits of the composites are histogrammed over it until the
// class holding the k-th delegate plus everything ranked above the class
// fit sm.D (kBMaxS entries, counting BETA per such entry), then the
// subranges whose first delegate lies in that class or above are copied
// there whole (the k-th delegate and all delegates above it among them).
// Returns the number of entries copied, or 0 if no cut fits (massive ties).
template <int BETA>
__device__ inline uint32_t b_cut_global(const uint64_t* Dg, uint32_t S, uint32_t k, BatchSmem& sm) {
  const uint32_t E = S * BETA;
  uint64_t prefix = 0, mask = 0;
  uint32_t r = k, above = 0, cls = 0;
  bool fits = false;
  for (int p = 0; p < kPasses; ++p) {
    for (int i = threadIdx.x; i < kBins; i += kBT) sm.hist[i] = 0;
    __syncthreads();
    const int sh = pass_shift(p);
    const uint32_t dm = (1u << pass_bits(p)) - 1;
    // eight coherent loads in flight per thread before any is counted
    for (uint32_t i0 = threadIdx.x; i0 < E; i0 += 8 * kBT) {
      uint64_t x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] = i0 + u * kBT < E ? ld_coh64(&Dg[i0 + u * kBT]) : 0ull;
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (i0 + u * kBT < E && (x[u] & mask) == prefix) atomicAdd(&sm.hist[(uint32_t)(x[u] >> sh) & dm], 1u);
    }
    __syncthreads();
    bb_bucket(sm.hist, r, sm);
    prefix |= (uint64_t)sm.out[0] << sh;
    mask |= (uint64_t)dm << sh;
    above += r - sm.out[1];
    r = sm.out[1];
    cls = sm.out[3];
    __syncthreads();
    if ((above + cls) * BETA <= kBMaxS) {
      fits = true;
      break;
    }
  }
  if (!fits) return 0;
  if (threadIdx.x == 0) sm.nq = 0;
  __syncthreads();
  // a subrange's first delegate is its largest: any of its entries in the
  // class or above puts the first there, so at most above + cls subranges
  for (uint32_t s0 = threadIdx.x; s0 < S; s0 += 8 * kBT) {
    uint64_t x[8], y[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const uint32_t s = s0 + u * kBT;
      x[u] = s < S ? ld_coh64(&Dg[s * BETA]) : 0ull;
      y[u] = BETA == 2 && s < S ? ld_coh64(&Dg[s * BETA + 1]) : 0ull;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (s0 + u * kBT < S && (x[u] & mask) >= prefix) {
        const uint32_t j = atomicAdd(&sm.nq, 1u);
        sm.D[j * BETA] = x[u];
        if constexpr (BETA == 2) sm.D[j * BETA + 1] = y[u];
      }
  }
  __syncthreads();
  const uint32_t cnt = sm.nq * BETA;
  __syncthreads();
  return cnt;
}

// Tile `tile` of a split problem (alpha >= 4): this workgroup builds the
// delegates of its tile and publishes them to Dg with coherent stores, then
// counts itself in; the workgroup that arrives last loads the whole delegate
// vector and finishes the problem (radix select over the keys if its
// survivors overflow).  Nobody waits for anybody.
template <bool VEC, int BETA>
__device__ inline void b_tile(const BatchDesc& d, uint32_t tile, uint32_t* arrive, uint64_t* Dg, BatchSmem& sm,
                              uint32_t* rec);

// ---------------------------------------------------------------------------
// Top-k of one problem by one workgroup in one pass over its keys.
//
// A sample of the keys gives a first cut.  Elements that reach the cut are
// appended to LDS, each wave to a region of its own.  When a region is full,
// everything below the k-th of what is held (roughly: below the bin of a
// 2048-bin histogram that the k-th lies in) is dropped and the cut raised to
// it.  What is left at the end is sorted.  Exact for every input: an element is
// dropped only if k others rank above it or by the first cut, and if fewer
// than k reach that, the keys are read once more without it.
//
// Bound by memory (4096 problems of 2^10 to 2^20 keys, k <= 2048: 499 us, 5.0
// TB/s; by delegates and a re-read of 25 to 50% of the large problems' keys, or
// several passes where k is large: 649) as long as what an element costs stays
// small: about five instructions a key, and a load with hits four compares more.
// Placing hits by a scan and an LDS atomic a chunk took 600 instructions a chunk
// and 560 -> 690 us; raising the cut from the first keys instead of a sample,
// four more sorts of the buffer a problem.  Loads marked for one use: 616 -> 582.
constexpr uint32_t kBStreamCap = 7680;               // elements held (two workgroups fit a CU)
constexpr uint32_t kBRegion = kBStreamCap / kBWaves; // of them by one wave
constexpr uint32_t kBStreamSlack = kBStreamCap / 4;  // elements kept beyond k when the cut is raised
// Keys a wave takes at a time, the next as many in flight: 1536 spill registers
// (582 us where 1280 and 1024 take 534).
constexpr uint32_t kBChunk = 1024;
static_assert((kBMaxK + kBStreamSlack) / kBWaves + 1 + 256 <= kBRegion, "room for a load after every raise");
static_assert(kBRegion % 64 == 0, "a region is whole rows of a wave");

struct BStreamSmem : SSortShared<uint64_t, kBStreamCap, kBT> {
  uint32_t fill[kBWaves];  // elements in each region
  uint32_t full;           // a region is full
};

// A composite that at least k and at most k + slack of the N in sm.buf reach
// (those above `hi` or below `lo` are not looked at; every thread calls).
__device__ __forceinline__ uint64_t b_stream_cut(BStreamSmem& sm, uint32_t N, uint32_t k, uint32_t slack, uint64_t lo,
                                                 uint64_t hi, uint32_t* rec) {
  uint32_t above = 0;  // elements above hi
  for (;;) {
    const int sh = sbucket_hist<uint64_t, kBStreamCap, kBT>(sm, N, lo, hi, [&](uint64_t i) { return sm.buf[i]; });
    const uint32_t need = k - above;
    if (sm.hist[kSBins] < need) {  // no bin holds the rank (uniform)
      if (threadIdx.x == 0) record_err(rec, ERR_SELECT);
      return suniform(lo);
    }
    for (uint32_t b = threadIdx.x; b < (uint32_t)kSBins; b += kBT)
      if (sm.hist[b] < need && need <= sm.hist[b + 1]) sm.misc[2] = b;
    __syncthreads();
    const uint32_t b = sm.misc[2], before = sm.hist[b], upto = sm.hist[b + 1];
    __syncthreads();
    const uint64_t first = hi - ((uint64_t)b << sh), width = ((uint64_t)1 << sh) - 1;
    lo = first - lo > width ? first - width : lo;
    if (sh == 0 || above + upto <= k + slack) return suniform(lo);
    hi = first;
    above += before;
  }
}

// Moves the regions' elements to the front of sm.buf and returns their number.
__device__ __forceinline__ uint32_t b_stream_gather(BStreamSmem& sm) {
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t at = 0, N = 0;
  for (uint32_t w = 0; w < (uint32_t)kBWaves; ++w) {
    if (w == wave) at = N;
    N += sm.fill[w];
  }
  const uint32_t mine = sm.fill[wave];
  uint64_t c[kBRegion / 64];
#pragma unroll
  for (int e = 0; e < (int)(kBRegion / 64); ++e)
    if (e * 64 + lane < mine) c[e] = sm.buf[wave * kBRegion + e * 64 + lane];
  __syncthreads();
#pragma unroll
  for (int e = 0; e < (int)(kBRegion / 64); ++e)
    if (e * 64 + lane < mine) sm.buf[at + e * 64 + lane] = c[e];
  __syncthreads();
  return N;
}

// Raises the cut to one that the elements held leave k of, and at most
// kBStreamSlack more, drops those under it and deals the rest to the regions.
// Returns the new cut.
__device__ __forceinline__ uint64_t b_stream_raise(BStreamSmem& sm, uint32_t k, uint64_t cut, uint64_t top,
                                                   uint32_t* rec) {
  constexpr int E = kBStreamCap / kBT;
  const uint32_t N = b_stream_gather(sm);
  // few held in all, but unevenly: dealing them out makes the room
  const uint64_t lo = N > k + kBStreamSlack ? b_stream_cut(sm, N, k, kBStreamSlack, cut, top, rec) : cut;
  uint64_t c[E];
  uint32_t mine = 0;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const uint32_t i = e * kBT + threadIdx.x;
    c[e] = i < N ? sm.buf[i] : 0;
    mine += i < N && c[e] >= lo ? 1u : 0u;
  }
  uint32_t tot;
  uint32_t at = sblock_scan<kBT>(mine, sm.s_w, &tot);
#pragma unroll
  for (int e = 0; e < E; ++e)
    if (e * kBT + threadIdx.x < N && c[e] >= lo) {
      sm.buf[at % kBWaves * kBRegion + at / kBWaves] = c[e];
      ++at;
    }
  if (threadIdx.x < kBWaves) sm.fill[threadIdx.x] = (tot + kBWaves - 1 - threadIdx.x) / kBWaves;
  if (threadIdx.x == 0) sm.full = 0;
  __syncthreads();
  return lo;
}

// The pass over the keys.  Waves stream independently, the next chunk in
// flight; one whose region is full sets sm.full, and every wave comes to the
// barrier below when it sees that or has no chunk left, so they meet there the
// same number of times.
template <bool VEC>
__device__ __forceinline__ void b_stream_keys(const uint32_t* keys, uint32_t n, uint32_t k, Codec cx, int L,
                                              uint32_t posmask, uint64_t cut, BStreamSmem& sm, uint32_t* rec) {
  constexpr int U = kBChunk / 256;
  const uint32_t n4 = vec_end<VEC>(n);
  const Keys<VEC> ks(keys, n4);
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t nch = (n4 + kBChunk - 1) / kBChunk;
  uint64_t* st = sm.buf + wave * kBRegion;
  uint32_t nx[U][4], v[U][4];
  uint32_t i = wave, done = 0, fill = 0;  // the chunk in nx; its loads worked off; elements in the region
  uint32_t tkey = 0, tpos = 0;
  auto fetch = [&]() {  // past the last chunk: beyond the buffer resource, nothing is read
#pragma unroll
    for (int u = 0; u < U; ++u) ks.template load4<1>(i * kBChunk + u * 256 + lane * 4, nx[u]);
  };
  auto push = [&](bool in, uint32_t key, uint32_t p) {
    const uint64_t b = __ballot(in);
    if (b) {
      if (in) st[fill + mbcnt(b)] = scomp<uint32_t>(key, p, L, posmask);
      fill += (uint32_t)__popcll(b);
    }
  };
  auto begin = [&]() {
    tkey = (uint32_t)(cut >> L);
    tpos = posmask - ((uint32_t)cut & posmask);
    fill = done = 0;
    i = wave;
    fetch();
    if (threadIdx.x == 0) sm.full = 0;
    if (wave == 0 && n4 < n) {  // the keys after the last whole 16 bytes
      const uint32_t p = n4 + lane;
      const uint32_t x = p < n ? cx.enc(keys[p]) : 0u;
      push(p < n && (x > tkey || (x == tkey && p <= tpos)), x, p);
    }
    if (tpos >= n4) tpos = n4 - 1;  // zeros read past n4 are keys of no position
    __syncthreads();
  };
  // one chunk; false: a load (the one after `done` loads) may not fit
  auto work = [&](uint32_t base) -> bool {
    const uint32_t tnext = tkey + 1 ? tkey + 1 : tkey;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if ((uint32_t)u < done) continue;
      const uint32_t a = v[u][0] > v[u][1] ? v[u][0] : v[u][1], b = v[u][2] > v[u][3] ? v[u][2] : v[u][3];
      const uint32_t p1 = base + u * 256, p = p1 + lane * 4;
      // keys equal to the cut's matter up to its position only
      if (__ballot((a > b ? a : b) >= (p1 > tpos ? tnext : tkey))) {
        if (fill + 256 > kBRegion) {
          done = u;
          return false;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) push(v[u][c] > tkey || (v[u][c] == tkey && p + c <= tpos), v[u][c], p + c);
      }
    }
    done = 0;
    return true;
  };
  begin();
  for (;;) {
    while (i < nch) {
      const uint32_t base = i * kBChunk;
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int c = 0; c < 4; ++c) v[u][c] = cx.enc(nx[u][c]);
      i += kBWaves;
      fetch();
      if (base + kBChunk > n4) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int c = 0; c < 4; ++c)
            if (base + u * 256 + lane * 4 + c >= n4) v[u][c] = 0;
      }
      if (!work(base)) {
        i -= kBWaves;  // read again once there is room: rare, and no registers held meanwhile
        if (lane == 0) __hip_atomic_store(&sm.full, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        break;
      }
      if (__builtin_amdgcn_readfirstlane(
              (int)__hip_atomic_load(&sm.full, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)))
        break;
    }
    if (lane == 0) sm.fill[wave] = fill;
    __syncthreads();
    if (!sm.full) {  // every wave came here without a chunk left
      uint32_t N = 0;
      for (uint32_t w = 0; w < (uint32_t)kBWaves; ++w) N += sm.fill[w];
      if (N >= k) return;
      if (cut == 0) {  // uniform
        if (threadIdx.x == 0) record_err(rec, ERR_FEW);
        return;
      }
      cut = 0;  // the sample misjudged the keys: once more without it
      __syncthreads();
      begin();
      continue;
    }
    cut = b_stream_raise(sm, k, cut, ((uint64_t)0xFFFFFFFFu << L) | posmask, rec);
    fill = (uint32_t)__builtin_amdgcn_readfirstlane((int)sm.fill[wave]);
    tkey = (uint32_t)(cut >> L);
    tpos = posmask - ((uint32_t)cut & posmask);
    if (tpos >= n4) tpos = n4 - 1;
    fetch();
  }
}

// The first cut: of 2048 or 6144 keys (of more than kBSmallN), in runs of 16 (a line of memory) at
// hashed places of equal strata, about the one that as many are expected above
// as of the k largest, and four and a half standard deviations more.  Fewer
// than k above it means a second pass, so no more margin is needed.
__device__ __forceinline__ uint64_t b_stream_sample(const uint32_t* keys, uint32_t n, uint32_t k, Codec cx, int L,
                                                    uint32_t posmask, BStreamSmem& sm, uint32_t* rec) {
  const int loads = n < (1u << 17) ? 1 : 3;
  const Keys<false> ks(keys, n);
  uint32_t x[3][4], p[3];
#pragma unroll
  for (int u = 0; u < 3; ++u)
    if (u < loads) {
      const uint32_t g = (threadIdx.x >> 2) + u * (kBT / 4), G = loads * (kBT / 4);
      const uint32_t lo = (uint32_t)((uint64_t)g * n / G), len = (uint32_t)((uint64_t)(g + 1) * n / G) - lo;
      p[u] = ((lo + (uint32_t)(((uint64_t)shash(g) * len) >> 32)) & ~15u) + (threadIdx.x & 3u) * 4;
      ks.load4(p[u], x[u]);
    }
#pragma unroll
  for (int u = 0; u < 3; ++u)
    if (u < loads)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        sm.buf[(u * 4 + c) * kBT + threadIdx.x] = p[u] + c < n ? scomp<uint32_t>(cx.enc(x[u][c]), p[u] + c, L, posmask) : 0;
  __syncthreads();
  const uint32_t S = loads * 4 * kBT;
  const float lam = (float)k * (float)S / (float)n;
  const uint32_t r = (uint32_t)(lam + 4.5f * sqrtf(lam) + 6.0f);
  return b_stream_cut(sm, S, r < S ? r : S, r / 8, 0, ((uint64_t)0xFFFFFFFFu << L) | posmask, rec);
}

// Sorts the N composites in c and writes the first k.
template <int E>
__device__ __forceinline__ void b_stream_write(const BatchDesc& d, uint64_t (&c)[E], uint32_t N, Codec cx, int L,
                                               uint32_t posmask, BStreamSmem& sm) {
  const uint32_t k = d.k;
  ssort<uint64_t, kBStreamCap, kBT, E>(sm, c, N, k, [&](uint32_t r, uint64_t x) {
    if (r >= k) return;
    const uint32_t val = cx.dec((uint32_t)(x >> L));
    if (d.out_vals) d.out_vals[r] = val;
    if (d.out_idx) d.out_idx[r] = posmask - ((uint32_t)x & posmask);
    if (d.out_kth && r == k - 1) *d.out_kth = val;
  });
}

// Lists above kBSmallN of which more than this by n * k is wanted are cut before
// they are sorted: most of a list that is wanted crowds the sort's bins.
constexpr uint32_t kBSortWork = 3u << 17;

// Sorts all of at most N keys.  (Up to the LDS's capacity: streamed with a cut
// that keeps every key, a wave's region of 960 overflowed in its first chunk, and
// every problem of 4097 to 7680 keys dealt its elements out anew: 8 of 5000, k = 24,
// 14.8 us, so 10.1; by the delegate method 11.5.)
template <uint32_t N>
__device__ __forceinline__ void b_sort_all(const BatchDesc& d, Codec cx, int L, uint32_t posmask, BStreamSmem& sm) {
  constexpr int E = N / kBT;
  static_assert(N % kBT == 0 && N <= kBStreamCap, "whole rows of the workgroup, in its LDS");
  const uint32_t n = (uint32_t)d.n;
  uint64_t c[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const uint32_t p = e * kBT + threadIdx.x;
    if (p < n) c[e] = scomp<uint32_t>(cx.enc(d.keys[p]), p, L, posmask);
  }
  b_stream_write<E>(d, c, n, cx, L, posmask, sm);
}

__device__ __forceinline__ void b_stream(const BatchDesc& d, BStreamSmem& sm, uint32_t* rec) {
  const uint32_t n = (uint32_t)d.n, k = d.k;
  const Codec cx = codec_of(d.dtype);
  const int L = n > 1 ? 32 - __clz((int)(n - 1)) : 1;
  const uint32_t posmask = (1u << L) - 1;
  if (n <= kBSmallN) return b_sort_all<kBSmallN>(d, cx, L, posmask, sm);
  if (n <= kBStreamCap && n * k <= kBSortWork) return b_sort_all<kBStreamCap>(d, cx, L, posmask, sm);
  const bool vec = (reinterpret_cast<uintptr_t>(d.keys) & 15u) == 0;
  const uint64_t cut = b_stream_sample(d.keys, n, k, cx, L, posmask, sm, rec);
  if (vec) b_stream_keys<true>(d.keys, n, k, cx, L, posmask, cut, sm, rec);
  else b_stream_keys<false>(d.keys, n, k, cx, L, posmask, cut, sm, rec);
  const uint32_t N = b_stream_gather(sm);
  constexpr int E = kBStreamCap / kBT;
  uint64_t c[E];
#pragma unroll
  for (int e = 0; e < E; ++e)
    if (e * kBT + threadIdx.x < N) c[e] = sm.buf[e * kBT + threadIdx.x];
  __syncthreads();
  b_stream_write<E>(d, c, N, cx, L, posmask, sm);
}

// LDS of a workgroup.
union BatchLds {
  BatchSmem b;
  BStreamSmem s;
};

// By the descriptor's alpha and beta.  OVER: survivors that overflow the LDS
// (ordered or tied keys) are left to the caller, who gets false.
template <bool VEC, bool OVER>
__device__ inline bool b_problem_v(const BatchDesc& d, BatchSmem& sm, uint32_t* rec) {
  if (d.n <= kBSmallN) {
    b_small<VEC>(d, sm);
    return true;
  }
  if (d.alpha >= 2) {
    const uint64_t E = ((d.n + (1ull << d.alpha) - 1) >> d.alpha) * d.beta;
    if (E <= kBMaxS && E > d.k && (d.beta == 2 ? b_delegate<VEC, 2>(d, sm) : b_delegate<VEC, 1>(d, sm))) return true;
    __syncthreads();
    if constexpr (OVER) return false;
  }
  b_radix<VEC>(d, sm, rec);
  return true;
}

template <bool VEC, int BETA>
__device__ inline void b_tile(const BatchDesc& d, uint32_t tile, uint32_t* arrive, uint64_t* Dg, BatchSmem& sm,
                              uint32_t* rec) {
  const uint32_t n = (uint32_t)d.n, alpha = d.alpha, n4 = vec_end<VEC>(n);
  const uint32_t tlog = tile_log(alpha, BETA);
  const uint32_t lo = tile << tlog;
  const uint32_t hi = n - lo > (1u << tlog) ? lo + (1u << tlog) : n;
  const uint32_t s0 = lo >> alpha;
  const uint32_t ne = (((hi - lo) + (1u << alpha) - 1) >> alpha) * BETA;  // entries of this tile
  const Keys<VEC> ks(d.keys, n4);
  for (uint32_t i = threadIdx.x; i < ne; i += kBT) sm.D[i] = 0;
  __syncthreads();
  b_delegates<VEC, BETA>(ks, lo, hi, n4, alpha, codec_of(d.dtype), sm);
  if (hi == n) b_delegates_tail<BETA>(d, n4, s0, sm);
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < ne; i += kBT) st_coh64(&Dg[d.doff + s0 * BETA + i], sm.D[i]);
  __builtin_amdgcn_s_waitcnt(0);  // this thread's stores have completed
  __syncthreads();
  if (threadIdx.x == 0) sm.item = atomicAdd(arrive, 1u) == d.tiles - 1 ? 1u : 0u;
  __syncthreads();
  if (!sm.item) return;
  const uint32_t S = (n + (1u << alpha) - 1) >> alpha;
  if (threadIdx.x == 0) sm.tail_del = n4 < n ? ld_coh64(&Dg[d.doff + (n4 >> alpha) * BETA + BETA - 1]) : 0;
  uint32_t cnt = S * BETA;
  if (cnt <= kBMaxS) {
    for (uint32_t i0 = threadIdx.x; i0 < cnt; i0 += 8 * kBT) {  // eight loads in flight per thread
      uint64_t x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] = i0 + u * kBT < cnt ? ld_coh64(&Dg[d.doff + i0 + u * kBT]) : 0ull;
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (i0 + u * kBT < cnt) sm.D[i0 + u * kBT] = x[u];
    }
    __syncthreads();
  } else {
    cnt = b_cut_global<BETA>(Dg + d.doff, S, d.k, sm);
  }
  if (cnt && b_finish<VEC, BETA>(d, cnt, sm)) return;
  __syncthreads();
  b_radix<VEC>(d, sm, rec);
}

template <bool OVER = false>
__device__ inline bool b_problem(const BatchDesc& d, BatchSmem& sm, uint32_t* rec) {
  const bool vec = (reinterpret_cast<uintptr_t>(d.keys) & 15u) == 0;
  return vec ? b_problem_v<true, OVER>(d, sm, rec) : b_problem_v<false, OVER>(d, sm, rec);
}

// One whole problem of a batch.  WAYS: which of the two ways some item takes: 1
// b_problem, for items with tiles = 0; 2 b_stream; 3 both.  What overflows the
// delegate method is streamed (two lists of 65536 ordered float32, k = 4: 34 us
// where a radix select of the keys took 108).
template <int WAYS>
__device__ __forceinline__ void b_whole(const BatchDesc& d, BatchLds& lds, uint32_t* rec) {
  if ((WAYS == 1 || (WAYS == 3 && d.tiles == 0)) && b_problem<true>(d, lds.b, rec)) return;
  b_stream(d, lds.s, rec);
}

__device__ inline void b_tile_any(const BatchDesc& d, uint32_t tile, uint32_t* arrive, uint64_t* Dg, BatchSmem& sm,
                                  uint32_t* rec) {
  const bool vec = (reinterpret_cast<uintptr_t>(d.keys) & 15u) == 0;
  if (d.beta == 2) {
    if (vec) b_tile<true, 2>(d, tile, arrive, Dg, sm, rec);
    else b_tile<false, 2>(d, tile, arrive, Dg, sm, rec);
  } else {
    if (vec) b_tile<true, 1>(d, tile, arrive, Dg, sm, rec);
    else b_tile<false, 1>(d, tile, arrive, Dg, sm, rec);
  }
}

// Work items are problem << 8 | tile, longest problems first: a problem with
// tiles <= 1 is one item and runs whole in its workgroup; a split problem is
// `tiles` items whose workgroups share its delegate vector through Dg, with
// arrive[problem] (starts at 0) counting finished tiles.  No workgroup waits for
// another.
//
// Tiles come first.  CLAIM: `claimers` workgroups take one each and claim the others
// from *counter (starts at 0); otherwise claimers = tiles.  With a workgroup each, those beyond what runs at
// once were not started before workgroups that finish problems had ended
// (150 problems of 400000 float32, k = 2048, 600 tiles: 160 us; claimed 110).
// Up to one round the loop only costs registers (400 tiles: 94 us, 90 without).
// Whole problems have a workgroup each.  (In a loop over them their many indices
// made from the thread's number are carried through it in registers: 4000 of
// them spilled; and the code of a call costs 20 us a launch.)
template <int WAYS, bool CLAIM>
__global__ __launch_bounds__(kBT) __attribute__((amdgpu_waves_per_eu(4))) void k_batched(
    const BatchDesc* __restrict__ descs, const uint32_t* __restrict__ items, uint32_t claimers, uint32_t tiles,
    uint32_t* counter, uint32_t* arrive, uint64_t* Dg, uint32_t* rec) {
  __shared__ BatchLds lds;
  if (blockIdx.x >= claimers) {
    const BatchDesc d = descs[items[tiles + (blockIdx.x - claimers)] >> 8];
    b_whole<WAYS>(d, lds, rec);
    return;
  }
  for (uint32_t w = blockIdx.x; w < tiles;) {
    const uint32_t it = items[w], i = it >> 8;
    const BatchDesc d = descs[i];
    b_tile_any(d, it & 0xFFu, &arrive[i], Dg, lds.b, rec);
    if constexpr (!CLAIM) return;
    __syncthreads();
    if (threadIdx.x == 0) lds.b.item = atomicAdd(counter, 1u);
    __syncthreads();
    w = claimers + lds.b.item;
    __syncthreads();
  }
}

// Items claimed from *counter (starts at 0), any grid size: for more tiles of
// split problems than run at once, whose uneven ends a claim evens out better
// than the order of launch does (512 problems of 2^20, k <= 2048: 558 us; 677 with
// a workgroup per tile).
__global__ __launch_bounds__(kBT) __attribute__((amdgpu_waves_per_eu(4))) void k_batched_split(
    const BatchDesc* __restrict__ descs, const uint32_t* __restrict__ items, uint32_t nitems, uint32_t* counter,
    uint32_t* arrive, uint64_t* Dg, uint32_t* rec) {
  __shared__ BatchSmem sm;
  for (;;) {
    __syncthreads();
    if (threadIdx.x == 0) sm.item = atomicAdd(counter, 1u);
    __syncthreads();
    const uint32_t w = sm.item;
    __syncthreads();
    if (w >= nitems) break;
    const uint32_t it = items[w];
    const uint32_t i = it >> 8;
    const BatchDesc d = descs[i];
    if (d.tiles > 1) b_tile_any(d, it & 0xFFu, &arrive[i], Dg, sm, rec);
    else b_problem(d, sm, rec);
  }
}

// Up to kBInline problems with the descriptors passed by value: no copy of
// descriptors and no claim counter.  Grid = count: workgroup i owns problem i.
constexpr uint32_t kBInline = 32;
struct BatchInline {
  BatchDesc d[kBInline];
};
template <int WAYS>
__global__ __launch_bounds__(kBT) __attribute__((amdgpu_waves_per_eu(4))) void k_batched_inline(BatchInline b, uint32_t* rec) {
  __shared__ BatchLds lds;
  const BatchDesc d = b.d[blockIdx.x];
  b_whole<WAYS>(d, lds, rec);
}

// One problem, descriptor by value: the single-problem path for small inputs.
__global__ __launch_bounds__(kBT) __attribute__((amdgpu_waves_per_eu(4))) void k_one(BatchDesc d, uint32_t* rec) {
  __shared__ BatchSmem sm;
  b_problem(d, sm, rec);
}

}  // namespace drtopk
