// kp_cut.h -- how an interval of output codes that holds too many products is
// cut into pieces, which wait on a stack of the workgroup's (in LDS) until
// they are done.  Plain C++ beside its two kernels, so that what it promises
// (the cuts end, the stack is never left) can be checked on the host.
#pragma once

#include <cstdint>

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define KP_CUT_FN __host__ __device__ __forceinline__
#define KP_CUT_ROLLED _Pragma("nounroll")   // the kernels are short of registers, cuts are rare
#else
#define KP_CUT_FN inline
#define KP_CUT_ROLLED
#endif

namespace kp {

constexpr int CUT_SAMPLES = 64;   // offsets that a cut looks at, at most
constexpr int CUT_PIECES = 9;     // pieces of a cut, at most (one more than its parts)
constexpr int CUT_FEW = 16;       // fewer samples than this: equally wide pieces

// Stack entries and log2 of the width that is not cut any more, for the
// products found from the sorted factors and for packs.  An interval that only
// equal cuts are left for takes 7 * cut_levels + 1 entries: 134 and 120 for
// 2^62 codes; the rest is room for sampled cuts, one that takes as many as it
// has points.
constexpr int DIRECT_STACK = 144, DIRECT_DONE_LOG = 6;
constexpr int PACK_STACK = 176, PACK_DONE_LOG = 11;
// Parts of a sampled cut.  A pack's samples are keys of a full table, the
// products of the rows walked so far: quartiles, since octiles make pieces of
// 250 products (a batch of 24 products, some crowded, 695 us instead of 617).
constexpr int DIRECT_PARTS = 8, PACK_PARTS = 4;

// Equal cuts in eight that lead from width codes to at most 2^done.
KP_CUT_FN int cut_levels(uint64_t width, int done) {
  const int bits = width <= 1 ? 0 : 64 - __builtin_clzll(width - 1);   // ceil(log2(width))
  return bits <= done ? 0 : (bits - done + 2) / 3;
}

// The pieces of the interval [0, width) of more than 2^done codes, which lies
// at stack index sp: put(p, x, y) takes piece p, the offsets [x, y).  Returns
// how many.  get(i): offset i of n products in the interval, ascending (they
// may repeat).
//
// The cut is at the quantiles of the samples (into `parts`, at most eight),
// since products that crowd on several scales would take a cut per scale, with
// two additions:
//  * When a piece would keep more than seven eighths of the codes, it is also
//    cut in the middle of the interval: whatever the samples are, cuts end.
//  * Quantiles that coincide at a code that many products share cut that code
//    off as a piece of its own.
// A sampled cut is made only if equal cuts of a piece that follows would still
// fit the stack; otherwise the cut is equal, in eight.  So every entry, at index
// i with w codes, keeps i + 7 * cut_levels(w) + 1 <= stack: an equal cut adds
// seven entries and takes a level off.  (Widths are at most 2^62.)
template <typename K, int PARTS, typename Get, typename Put>
KP_CUT_FN int cut_points(Get&& get, int n, K width, int sp, int stack, int done, Put&& put) {
  static_assert(PARTS <= 8, "at most nine pieces");
  const K half = width / 2, most = width - width / 8;
  K from = 0;   // where the last piece begins
  int m = 0;
  const auto next = [&](K x) {
    if (x > from && x < width) {
      put(m++, from, x);
      from = x;
    }
  };
  if (n >= CUT_FEW && sp + PARTS + 7 * cut_levels((uint64_t)most + 1, done) + 1 <= stack) {
    K q[PARTS + 1];
    q[0] = 0;
    q[PARTS] = width;
    for (int i = 1; i < PARTS; ++i) q[i] = get(i * n / PARTS);
    bool mid = false;
    for (int i = 0; i < PARTS; ++i) mid = mid || q[i + 1] - q[i] > most;
    for (int i = 1; i < PARTS; ++i) {
      const K point = q[i] + (q[i] == q[i - 1] ? 1 : 0);
      if (mid && point > half) next(half);   // (not again once a piece begins there or later)
      next(point);
    }
    if (mid) next(half);
  } else {
    const K step = width / 8 + (width % 8 != 0 ? 1 : 0);
    KP_CUT_ROLLED
    for (int i = 1; i < 8; ++i)
      if (step < width - from) next(from + step);
  }
  put(m++, from, width);
  return m;
}

}  // namespace kp
