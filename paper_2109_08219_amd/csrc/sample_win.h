// The window of the sampled path: which sample ranks bound the elements that
// can be in the answer, and how they are divided into buckets.  Shared by the
// planner and the kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace drtopk {

// Payload of each selected key, gathered where its slot is written (bytes 0:
// none; 4 or 8).
struct SPayload {
  const void* in;
  void* out;
  uint32_t bytes, pad;
};

// The window of sample ranks of one level: elements above the a-th sample are
// counted only, those from it down to the r-th sample are the candidates.
// Buckets: with P = 0, every s samples from rank a on.  Otherwise, with P a
// power of two, from rank max(a, 1) on: P equal intervals of composite space
// between every kSGroup-th sample; and when the window is open (a = 0), where
// the keys thin out, before that kSTop intervals above the first sample and over
// the first kSThin groups the samples themselves besides P2 intervals (twice as
// many, unless they would make too many buckets: the keys of the first group
// thin out so fast that its lowest interval of P held more than a workgroup sorts
// in 1 of 80 calls, normal float32, n = 2^24, k = 2^21).  s: groups in all.
struct SWin {
  uint32_t r, a, s, P, B, P2, pad[2];
};
constexpr uint32_t kSTop = 8;
constexpr uint32_t kSGroup = 16;
constexpr uint32_t kSThin = 4;

// Window for rank k of `count` elements under m samples: the number of
// samples among the k largest is bounded both ways but for a probability below
// 2 * exp(-24) (Bernstein's inequality).
__host__ __device__ inline void sample_window(double count, double k, double m, bool kth, SWin* w) {
  const double lam = k * m / count, v = lam * (1.0 - k / count);
#ifdef __HIP_DEVICE_COMPILE__
  const double x = 8.0 + (double)sqrtf((float)(64.0 + 48.0 * v));
#else
  const double x = 8.0 + __builtin_sqrt(64.0 + 48.0 * v);
#endif
  const double hi = lam + x + 2.0, lo = lam - x - 2.0;
  w->r = hi < m ? (uint32_t)hi : (uint32_t)m + 1;  // m + 1: no cut, every element is a candidate
  w->a = kth && lo >= 1.0 ? (uint32_t)lo : 0u;
}
// Splitters of one of the first kSThin groups (see SWin).
__host__ __device__ inline uint32_t thin_splits(uint32_t P2) { return P2 + kSGroup - 1; }

// Buckets are planned for `target` elements.  Gaps between neighbouring samples
// are as uneven as exponential variables (one in 43 holds 3.75 times the mean,
// a workgroup's capacity), so where a bucket would be less than six gaps it is
// an equal part of the space between every sixteenth sample instead: as even as
// that space, a quarter of the mean in one standard deviation, where the density
// changes little over it.
__host__ __device__ inline void sample_buckets(double gap, uint32_t target, uint32_t bmax, SWin* w) {
  const uint32_t q0 = w->a ? w->a : 1u, top = w->a ? 0u : kSTop;
  const uint32_t groups = (w->r - q0 + kSGroup - 1) / kSGroup;
  uint32_t P = 0, P2 = 0;
  if (6.0 * gap > (double)target) {
    P = 4;
    while (P < 64 && (double)kSGroup * gap > (double)target * P) P <<= 1;
    const uint32_t thin = w->a ? 0u : groups < kSThin ? groups : kSThin;
    uint64_t B = 0;
    for (P2 = 2 * P; P2 >= P; P2 >>= 1) {
      B = top + (uint64_t)thin * thin_splits(P2) + (uint64_t)(groups - thin) * P;
      if (B <= bmax || P2 == P) break;
    }
    w->B = (uint32_t)B;
    if (B > bmax) P = 0;
  }
  w->P = P;
  w->P2 = P2;
  if (P) {
    w->s = groups;
    return;
  }
  const double per = 0.75 * (double)target / gap;
  uint32_t s = per > 1.0 ? (per < 1e6 ? (uint32_t)per : 1000000u) : 1u;
  const uint32_t span = w->r - w->a;
  if ((uint64_t)s * bmax < span) s = (span + bmax - 1) / bmax;
  w->s = s;
  w->B = (span + s - 1) / s;
}

// The lowest composite of the first `bins` of at most 2048 bins of 2^sh
// composites each, from mx down to mn.  All of them can span the whole of C
// (64-bit composites of more than 2^31 keys), whose number of composites C does
// not hold.
template <typename C>
__host__ __device__ inline C leading_bins_cut(C mx, C mn, uint32_t bins, int sh) {
  return (mx - mn) >> sh < (C)bins ? mn : mx - (((C)bins << sh) - 1);
}

}  // namespace drtopk
