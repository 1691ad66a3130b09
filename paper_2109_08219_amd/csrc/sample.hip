// The sampled path: planner and kernel sequence.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>

#include "host.h"
#include "routes.h"
#include "sample.h"
#include "sample_host.h"
#include "wide_host.h"

namespace drtopk {

namespace {

constexpr uint32_t kSLevel2 = 4096;  // samples of the second level

size_t salign(size_t x) { return (x + 255) & ~(size_t)255; }

// Fewest samples r such that at least r of them fall among the k largest with
// probability below exp(-24), for lam = k * m / n expected (Chernoff's bound of
// the Poisson tail): tighter than Bernstein's inequality when few are expected.
uint32_t small_rank(double lam) {
  uint32_t r = (uint32_t)lam + 1;
  while (r * std::log(r / (2.718281828459045 * lam)) + lam < 24.0) ++r;
  return r + 1;
}

// Candidates from the first sample down to the `span`-th, planned for: but for
// six standard deviations.
double span_cap(double span, double gap) { return (span + 6.0 * std::sqrt(span) + 10.0) * gap; }

// Room for them: more with probability below exp(-24) (Chernoff's bound of
// fewer than `span` samples among as many elements).
double span_room(double span, double gap) {
  double lam = span + 6.0 * std::sqrt(span) + 10.0;
  while (lam - span - span * std::log(lam / span) < 24.0) lam += 0.125 * std::sqrt(span) + 0.5;
  return lam * gap;
}

template <typename K>
void plan_for(SPlan& p) {
  typedef STraits<K> T;
  typedef typename T::Comp C;
  const double n = (double)p.n, k = (double)p.k;
  SWin w = {};
  uint64_t cap1 = 0, cap = 0;             // room for the candidates
  uint64_t planned1 = 0, planned = 0;     // as many as are planned for
  double cap_top = 0, gap = 0;
  // the r-th of 16 m samples, of which the top 16 of each 256 are kept, when
  // r is at most a fifth of what is kept
  for (uint32_t m = 4096; m >= 1024 && !p.top; m /= 4) {
    if (p.n < 32 * (uint64_t)m) continue;
    gap = n / (16.0 * m);
    const double lam = k / gap;
    sample_window(n, k, 16.0 * m, false, &w);
    if (lam < 64) {
      const uint32_t r = small_rank(lam);
      if (r < w.r) w.r = r;
    }
    if (w.r > m / 5) break;
    p.top = true;
    p.m = m;
    cap_top = span_cap(w.r, gap);
  }
  if (!p.top) {
    p.m = p.n < 16384 ? 1024 : 8192;
    if (p.n < 2 * (uint64_t)p.m) return;
    gap = n / p.m;
    sample_window(n, k, p.m, p.kth_only, &w);
    cap_top = span_cap(w.r, gap);
  }
  if (cap_top <= T::kCap) {  // one workgroup sorts all candidates
    p.plain = 1;
    w.a = 0;
    w.B = p.bmax = 1;
    planned = T::kCap;
    cap = std::max<uint64_t>((uint64_t)span_room(w.r, gap), T::kCap);
  } else if (p.top && gap <= 2.0 * T::kTarget && cap_top <= T::kList) {
    // few enough that each bucket's workgroup can read all of them
    p.plain = 1;
    sample_buckets(gap, T::kTarget, T::kMaxB, &w);
    planned = (uint64_t)cap_top;
    cap = (uint64_t)span_room(w.r, gap);
    p.bmax = w.B;
  } else if (p.top) {
    // few of many: the streaming filter, and its candidates partitioned; the
    // partition's own pass over the input (2.2 us per 32 KB and CU) is for
    // windows that keep a share of it
    p.levels = 2;
    planned1 = std::min<uint64_t>((uint64_t)cap_top, p.n);
    if (planned1 > (1u << 24)) return;
    SWin w2 = {};
    sample_window((double)planned1, k, kSLevel2, false, &w2);
    planned = std::min<uint64_t>((uint64_t)span_cap(w2.r, (double)planned1 / kSLevel2), planned1);
    const uint64_t b = 4 * planned / T::kTarget + 64;
    cap1 = std::min<uint64_t>((uint64_t)span_room(w.r, gap), p.n);
    sample_window((double)cap1, k, kSLevel2, false, &w2);
    cap = std::min<uint64_t>((uint64_t)span_room(w2.r, (double)cap1 / kSLevel2), cap1);
    p.bmax = b < (uint64_t)T::kMaxB ? (uint32_t)b : (uint32_t)T::kMaxB;
  } else if (gap <= 2.0 * T::kTarget) {
    sample_buckets(gap, T::kTarget, T::kMaxB, &w);
    planned = (uint64_t)span_cap(w.r - w.a, gap);
    cap = (uint64_t)span_room(w.r - w.a, gap);
    p.bmax = w.B;
  } else {
    return;
  }
  p.win = w;
  if (cap > p.n) cap = p.n;
  // rows: a workgroup's last, and those written because a tile did not fit (two of
  // these in a row hold more than a stage, so the limit leaves enough for `cap`)
  if (planned > p.n) planned = p.n;
  auto rows = [&](uint64_t c1, uint64_t c) {
    return grid_for(p.levels == 2 ? c1 : p.n, T::kTile, 256) + c / (T::kStage - T::kTile) + 1;
  };
  if (!p.plain && rows(planned1, planned) > (uint64_t)kSMaxRows) return;
  p.pitch = (p.bmax + 1 + 31) & ~31u;
  auto layout = [&](uint64_t c1, uint64_t c) {
    p.cap1 = (uint32_t)c1;
    p.cap = (uint32_t)c;
    p.rows = (uint32_t)std::min<uint64_t>(rows(c1, c), kSMaxRows);
    size_t off = 0;
    auto seg = [&](size_t bytes) {
      const size_t o = off;
      off = salign(off + bytes);
      return o;
    };
    p.off_ctl = seg(sizeof(SCtl));
    const size_t ms = p.levels == 2 && p.m < kSLevel2 ? kSLevel2 : p.m;
    p.off_smp = seg(ms * sizeof(C));
    p.off_sorted = seg(ms * sizeof(C));
    if (p.levels == 2) p.off_c1 = seg((size_t)p.cap1 * sizeof(C));
    p.off_cand = seg(((size_t)p.cap + 1) * sizeof(C));  // whole 16-byte pieces
    if (!p.plain) {
      p.off_rows = seg(p.rows * sizeof(SRow));
      p.off_bounds = seg((size_t)p.bmax * sizeof(C));
      p.off_offs = seg((size_t)p.rows * p.pitch * sizeof(uint16_t));
    }
    return off;
  };
  p.planned = layout(planned1, planned);
  p.total = layout(cap1, cap);
  p.on = true;
}

// Whether one workgroup takes the call whole, and its cut: r = 0 sends every
// element to the sort, else the r-th of 256 samples.  A miss only costs a few passes over
// at most 65536 keys, so four and a half standard deviations will do.
template <typename K>
bool one_fits(uint64_t n, uint32_t k, uint32_t* r) {
  const uint32_t cap = n <= 1024 ? 1024u : SOne<K>::kCap;
  *r = 0;
  if (n <= cap && !one_cuts(n, k)) return true;
  if (n > 65536) return false;
  const double lam = (double)k * kSSplit / n, q = lam + 4.5 * std::sqrt(lam) + 6.0;
  *r = (uint32_t)q;
  return (q + 4.0 * std::sqrt(q) + 4.0) * n / kSSplit <= cap;
}

template <typename K>
void enqueue_one(const SPlan& p, const void* keys_v, K* out_vals, uint32_t* out_idx, K* out_kth, SCheck ck,
                 hipStream_t s) {
  const K* keys = static_cast<const K*>(keys_v);
  const SCodec<K> cd{(K)p.codec_a, (K)p.codec_c};
  const uint32_t n = (uint32_t)p.n;
  const int kth = p.kth_only ? 1 : 0;
#define DRTOPK_ONE(T, KTH)                                                                                       \
  hipLaunchKernelGGL((k_sone<K, T, KTH>), dim3(1), dim3(T), 0, s, keys, n, p.k, p.win.r, kth, cd, p.L, out_vals, \
                     out_idx, out_kth, p.pay, ck)
  if (n <= 1024) {
    if (kth) DRTOPK_ONE(256, true);
    else DRTOPK_ONE(256, false);
  } else if (kth) {
    DRTOPK_ONE(1024, true);
  } else {
    DRTOPK_ONE(1024, false);
  }
#undef DRTOPK_ONE
}

template <typename K>
void enqueue_for(const SPlan& p, const void* keys_v, void* ws, K* out_vals, uint32_t* out_idx, K* out_kth,
                 SCheck ck, hipStream_t s, PhaseMarks& pm) {
  typedef STraits<K> T;
  typedef typename T::Comp C;
  const K* keys = static_cast<const K*>(keys_v);
  const SCodec<K> cd{(K)p.codec_a, (K)p.codec_c};
  SCtl* ctl = at<SCtl>(ws, p.off_ctl);
  C* smp = at<C>(ws, p.off_smp);
  C* sorted = at<C>(ws, p.off_sorted);
  C* c1 = at<C>(ws, p.off_c1);
  C* cand = at<C>(ws, p.off_cand);
  SRow* rows = at<SRow>(ws, p.off_rows);
  uint16_t* offs = at<uint16_t>(ws, p.off_offs);
  C* bounds = at<C>(ws, p.off_bounds);
  const int kth = p.kth_only ? 1 : 0;
  auto rank = [&](uint32_t m) {
    const dim3 g(m / kSRankPer), t(kSRankThreads);
    if (m == 1024) hipLaunchKernelGGL((k_srank<C, 2>), g, t, 0, s, smp, sorted);
    else if (m == 4096) hipLaunchKernelGGL((k_srank<C, 8>), g, t, 0, s, smp, sorted);
    else hipLaunchKernelGGL((k_srank<C, 16>), g, t, 0, s, smp, sorted);
  };
  pm.start(s);  // the timed pass: the sample and the one pass over the input
  if (p.top)
    hipLaunchKernelGGL((k_sgather<K, false, true>), dim3(p.m / kSKeep), dim3(1024), 0, s, keys, (const C*)nullptr, p.n,
                       0u, p.k, p.m * 16, p.salt, cd, p.L, p.win, kth, p.bmax, ctl, smp, sorted);
  else
    hipLaunchKernelGGL((k_sgather<K, false, false>), dim3(p.m / 256), dim3(256), 0, s, keys, (const C*)nullptr, p.n,
                       0u, p.k, p.m, p.salt, cd, p.L, p.win, kth, p.bmax, ctl, smp, sorted);
  rank(p.m);
  if (p.plain || p.levels == 2) {
    constexpr uint64_t load = (uint64_t)64 * (16 / sizeof(K)) * (kSFilterThreads / 64);
    uint64_t* al = p.plain ? &ctl->alloc : &ctl->alloc1;
    C* o = p.plain ? cand : c1;
    const uint32_t c = p.plain ? p.cap : p.cap1;
#define DRTOPK_FILTER(U)                                                                                            \
  hipLaunchKernelGGL((k_sfilter<K, U>), dim3(grid_for(p.n, U * load, 512)), dim3(kSFilterThreads), 0, s, keys, p.n, \
                     p.head, cd, p.L, p.win.r, p.m, sorted, al, o, c)
    // as many loads a tile as leave every workgroup two tiles
    if (p.n < 2 * 2 * load * 512) DRTOPK_FILTER(1);
    else if (p.n < 4 * 2 * load * 512) DRTOPK_FILTER(2);
    else DRTOPK_FILTER(4);
#undef DRTOPK_FILTER
  } else {
    const unsigned g = grid_for(p.n, T::kTile, 256);
    hipLaunchKernelGGL((k_spart<K, false>), dim3(g), dim3(kSPartThreads), 0, s, keys, (const C*)nullptr, p.n, p.head,
                       0u, p.k, p.m, p.win, cd, p.L, sorted, ctl, cand, p.cap, p.rows, rows, offs, p.pitch, bounds);
  }
  pm.mid(s);
  if (p.levels == 2) {
    hipLaunchKernelGGL((k_sgather<K, true, false>), dim3(kSLevel2 / 256), dim3(256), 0, s, keys, c1, p.n, p.cap1, p.k,
                       kSLevel2, p.salt, cd, p.L, p.win, kth, p.bmax, ctl, smp, sorted);
    rank(kSLevel2);
    const unsigned g = grid_for(p.cap1, T::kTile, 256);
    hipLaunchKernelGGL((k_spart<K, true>), dim3(g), dim3(kSPartThreads), 0, s, keys, c1, p.n, 0u, p.cap1, p.k,
                       kSLevel2, p.win, cd, p.L, sorted, ctl, cand, p.cap, p.rows, rows, offs, p.pitch, bounds);
  }
#define DRTOPK_BUCKET(MODE, RARE, GRID, SECOND)                                                                    \
  hipLaunchKernelGGL((k_sbucket<K, MODE, RARE>), dim3(GRID), dim3(kSBucketThreads), 0, s, keys, p.n, p.k, kth,     \
                     p.levels, SECOND, cd, p.L, ctl, cand, p.cap1, p.cap, p.rows, rows, offs, p.pitch, p.m, p.win,   \
                     sorted, bounds, out_vals, out_idx, out_kth, p.pay, ck)
  if (p.plain && p.bmax == 1) {
    DRTOPK_BUCKET(kSPlain, true, 1, 0);
  } else if (p.plain) {
    DRTOPK_BUCKET(kSList, true, p.bmax, 0);
  } else if (p.bmax <= 512 || kth) {  // one workgroup a CU, two rounds at most; of one bucket
    DRTOPK_BUCKET(kSRows, true, p.bmax, 0);
  } else {
    DRTOPK_BUCKET(kSRows, false, p.bmax, 0);
    DRTOPK_BUCKET(kSRows, true, p.bmax, 1);
  }
#undef DRTOPK_BUCKET
}

}  // namespace

namespace {

std::atomic<uint64_t> g_fixed_salt{0};  // testing hook: 2^32 + salt, or 0

// The sampled places' salt: another one in each process, so that no input can be
// laid out to be misjudged.  (Another one for each call would do as well, but
// the sampled lines that one call leaves in the caches then serve no later call
// on the same keys: 2 to 4% of a call of 2^20 to 2^24 keys.)
uint32_t sample_salt() {
  if (const uint64_t f = g_fixed_salt.load(std::memory_order_relaxed)) return (uint32_t)f;
  static const uint32_t salt = [] {
    uint64_t z = (uint64_t)std::chrono::steady_clock::now().time_since_epoch().count();
    z ^= (uint64_t)std::chrono::system_clock::now().time_since_epoch().count() * 0x9E3779B97F4A7C15ull;
    z ^= (uint64_t)reinterpret_cast<uintptr_t>(&g_fixed_salt);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;  // SplitMix64's output function
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return (uint32_t)(z >> 32);
  }();
  return salt;
}

}  // namespace

void sample_fix_salt(bool on, uint32_t salt) {
  g_fixed_salt.store(on ? (uint64_t(1) << 32) | salt : 0, std::memory_order_relaxed);
}

void sample_plan(const void* keys, uint64_t n, uint32_t k, int dtype, bool kth_only, SPlan* out) {
  SPlan p;
  p.n = n;
  p.k = k;
  p.kth_only = kth_only;
  p.wide = wide_dtype(dtype);
  const int base = dtype & ~DRTOPK_SMALLEST;
  const bool fl = base == DRTOPK_F32 || base == DRTOPK_F64;
  const bool raw = base == DRTOPK_U32 || base == DRTOPK_U64;
  const uint64_t top = p.wide ? 0x8000000000000000ull : 0x80000000ull;
  p.codec_a = fl ? top - 1 : 0;
  p.codec_c = raw ? 0 : top;
  if (dtype & DRTOPK_SMALLEST) p.codec_c = ~p.codec_c;
  p.L = 1;
  while (p.L < 32 && ((n - 1) >> p.L)) ++p.L;
  const uint32_t word = p.wide ? 8 : 4;
  p.head = (uint32_t)(((16 - (reinterpret_cast<uintptr_t>(keys) & 15u)) & 15u) / word);
  // (k = 1 of 4-byte keys: the delegate pass alone answers it)
  if ((k > 1 || p.wide) && (reinterpret_cast<uintptr_t>(keys) & (word - 1)) == 0) {
    const bool old = !p.wide && one_delegates(n, k);
    // a k-th value past the middle is found from the other end: the first
    // samples bound what a few of the topmost keys are, and nothing below the last
    // sample is so bounded (the last of 2^24 int64 116 to 313 us, from there 49)
    if (kth_only && k > n / 2) {
      p.k = k = (uint32_t)(n - k + 1);
      p.codec_c = ~p.codec_c;
    }
    p.one = !old &&
            (p.wide ? one_fits<uint64_t>(n, k, &p.win.r) : one_fits<uint32_t>(n, k, &p.win.r));
    if (p.one) p.on = true;
    else if (old) ;
    else if (p.wide) plan_for<uint64_t>(p);
    else plan_for<uint32_t>(p);
  }
  if (p.on && !p.one) p.salt = sample_salt();
  *out = p;
}

int sample_enqueue(const SPlan& p, const void* keys, void* ws, uint32_t* rec, void* out_vals, uint32_t* out_idx,
                   void* out_kth, hipStream_t s, bool marks) {
  const SCheck ck{rec, p.hold};
  if (p.one) {
    if (p.wide)
      enqueue_one<uint64_t>(p, keys, static_cast<uint64_t*>(out_vals), out_idx, static_cast<uint64_t*>(out_kth), ck, s);
    else
      enqueue_one<uint32_t>(p, keys, static_cast<uint32_t*>(out_vals), out_idx, static_cast<uint32_t*>(out_kth), ck, s);
    return hipGetLastError() == hipSuccess ? (int)DRTOPK_OK : (int)DRTOPK_EDEVICE;
  }
  PhaseMarks pm;
  if (marks) pm.begin(s);
  if (p.wide)
    enqueue_for<uint64_t>(p, keys, ws, static_cast<uint64_t*>(out_vals), out_idx, static_cast<uint64_t*>(out_kth), ck,
                          s, pm);
  else
    enqueue_for<uint32_t>(p, keys, ws, static_cast<uint32_t*>(out_vals), out_idx, static_cast<uint32_t*>(out_kth), ck,
                          s, pm);
  pm.end(s);
  return hipGetLastError() == hipSuccess ? (int)DRTOPK_OK : (int)DRTOPK_EDEVICE;
}

}  // namespace drtopk
