// Host side of the sampled path: plan and enqueue (implemented in sample.hip,
// its own translation unit).
#pragma once

#include <cstddef>
#include <cstdint>

#include <hip/hip_runtime.h>

#include "drtopk.h"
#include "host.h"
#include "sample_win.h"

namespace drtopk {

struct SPlan {
  bool on = false;
  bool wide = false;      // 8-byte keys
  uint32_t head = 0;      // keys before the first 16-byte boundary
  bool kth_only = false;
  SPayload pay = {};      // set by the caller
  uint32_t hold = ~0u;    // most elements that a run or a fallback collects (below the LDS's capacity: testing hook)
  bool one = false;       // one workgroup takes the whole problem
  int levels = 1;         // 2: the first filter's candidates are sampled and partitioned again
  int plain = 0;          // the candidates are one list, not grouped by bucket
  uint64_t n = 0;
  uint32_t k = 0;
  int L = 1;              // position bits of a composite
  bool top = false;       // 16 m samples, the top 16 of each 256 kept
  uint32_t m = 0;         // samples kept
  uint32_t salt = 0;      // of the sampled places
  SWin win = {};          // level 1's window
  uint32_t bmax = 1;      // most buckets of the partitioned level
  uint32_t cap1 = 0, cap = 0;    // candidates kept by level 1, by the partitioned level
  uint32_t rows = 0;      // rows of the offset table
  uint32_t pitch = 0;            // entries of a row of the offset table
  uint64_t codec_a = 0, codec_c = 0;
  size_t off_ctl = 0, off_smp = 0, off_sorted = 0, off_c1 = 0, off_cand = 0, off_rows = 0, off_offs = 0, off_bounds = 0;
  size_t total = 0;
  size_t planned = 0;     // of that, without the room for more candidates than are planned for
};

// Fills *out (out->on false: the path does not take this call).
void sample_plan(const void* keys, uint64_t n, uint32_t k, int dtype, bool kth_only, SPlan* out);

// Testing hook: the salt of every call planned after it (off: the process's own).
void sample_fix_salt(bool on, uint32_t salt);

// Enqueues the whole path on `s` over the workspace `ws` (p.total bytes); failed
// internal checks are recorded in `rec` (nullptr: nowhere).
int sample_enqueue(const SPlan& p, const void* keys, void* ws, uint32_t* rec, void* out_vals, uint32_t* out_idx,
                   void* out_kth, hipStream_t s, bool marks);

}  // namespace drtopk
