// Which of two ways takes a call whose size allows both, by measurement on
// MI355X (float32 normal, uint32 uniform, 16-bit values in 32 bits; the lower of the
// three; times against the other way).  Plain C++: the planner's, not the kernels'.
#pragma once

#include <cstddef>
#include <cstdint>

namespace drtopk {

// A single call of 4-byte keys that the batched form's kernel takes (k_one: sorted
// by a network up to 4096 keys, then by the delegate method or a radix select),
// where one workgroup's sort or cut (k_sone) is slower: most of a few keys, which
// crowd the bins of a sort where they lie in clusters or, floats, on both sides
// of zero (2048 of 4096 normal float32: 12.7 against 19.9 us), and a handful of
// many (4 of 50000 uint32: 14.8 / 19.3; 64 of them: 21.5 / 19.1; 24 of 8193: 10.6 /
// 11.2, but 31 / 11.1 where they are tied).
inline bool one_delegates(uint64_t n, uint32_t k) {
  if (n <= 8192) return k <= 2048 && (uint64_t)k * 8 > n;
  return n <= 65536 && k <= 16;
}

// Whether one workgroup cuts even a list that fits its LDS by a sample before it
// sorts: where so much is wanted that the sort's bins are crowded.  us a call of
// normal float32 / uint32 / 16-bit values, sorted whole, cut, by k_one:
//   4096 keys, k = 256  11.2 9.4 11.8,  10.6 10.8 10.7,  11.0 10.7 16.0
//   4096 keys, k = 512  14.1 9.9 13.8,  11.2 10.9 11.4,  11.0  9.0 15.9
//   6000 keys, k = 256  13.2 11.1 13.2, 10.8 10.9 11.0,  13.5 13.4 13.6
//   8192 keys, k = 96   11.8 10.6 12.0, 11.4 11.2 11.2,  13.3 12.2 13.3
//   8192 keys, k = 512  21.2 14.9 21.3, 11.5 11.6 12.3,  14.8 14.2 15.0
inline bool one_cuts(uint64_t n, uint32_t k) { return n * n * k > 1ull << 32 && (uint64_t)k * 8 <= n; }

// A problem of a batch of `items`, whole in one workgroup: sorted whole or
// streamed once (b_stream), or else selected first (n <= 4096) or by the delegate
// method (b_problem).  Sorting all of a short list loses where so many are wanted
// that the sort's bins are crowded (float keys of both signs), streaming where so
// few are that a delegate per subrange tells them apart.  Few items leave CUs
// idle, and a problem's own chain of steps counts; many share the CUs, and the
// work counts, which streaming has less of.  us a call, this way / the other:
//   8 lists of 1000: k = 128 6.7 / 8.6, k = 512 11.0 / 8.9
//   8 of 4096: k = 64 9.8 / 11.0, k = 128 13.3 / 12.5, k = 512 21 / 12
//   4 of 6000: k = 32 10.7 / 11.7, k = 512 14.5 / 15; of 7680: k = 8 12.1 / 11.2
//   30 of 4500: k = 2048 32 / 19
//   8 of 8192: k = 8 12.8 / 10.4, k = 64 13.5 / 13.8
//   8 of 16000: k = 64 15.4 / 12.8, k = 512 17.7 / 17.7; 500 of them: 12 and 18% faster
//   8 of 50000: k = 2 18.6 / 15.7, k = 16 20 / 21
//   30 of 100000: k = 8 27 / 22, k = 16 27 / 30
// k = 1 has nothing to sort: 8 of 31000, 16.6 / 11.4.
inline bool batch_streams(uint64_t n, uint32_t k, size_t items) {
  const int many = items < 48 ? 0 : items < 128 ? 1 : 2;
  if (n <= 512) return many == 2 || (uint64_t)k * 8 <= n * 7;
  if (n <= 1024) return many == 2 || (uint64_t)k * 5 <= n || (k > 512 && k < n);
  if (k == 1 && n > 4096) return false;
  if (n <= 4096) return (uint64_t)k * 5 <= n && n * k <= (many == 0 ? 3u << 17 : many == 1 ? 9u << 16 : 6u << 17);
  if (n <= 7680) return (uint64_t)k * 5 <= n * 2 && (many || n <= 6144 || k >= 64);
  if (n < 9000) return k >= (many ? 32u : 64u);
  if (n < 18000) return k >= (many == 0 ? 512u : many == 1 ? 96u : 32u);
  if (n <= 65536) return k >= (many == 2 ? 4u : 16u);
  return k >= (items >= 384 ? 2u : 16u);
}

}  // namespace drtopk
