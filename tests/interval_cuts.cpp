// Host model of the cuts of crowded intervals: `cut_points` over samples that
// an adversary picks.  Prints the largest stack index and the most cuts of a
// path; exits with 1 and a line that names the case when a promise is broken.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "kp_cut.h"

using namespace kp;

static std::mt19937_64 rng(12345);

static uint64_t below(uint64_t n) { return n ? rng() % n : 0; }

// n offsets of [0, width), ascending, of one of the kinds of crowding.
template <typename K>
static int sample(int kind, K width, K* s) {
  int n = kind == 0 ? 0 : CUT_SAMPLES - (int)below(CUT_SAMPLES / 2);
  const uint64_t w = (uint64_t)width, heavy = below(w);
  for (int i = 0; i < n; ++i) {
    uint64_t x = 0;
    switch (kind) {
      case 1: x = 0; break;                                      // the first code only
      case 2: x = w - 1; break;                                  // the last code only
      case 3: x = std::min<uint64_t>(below(3), w - 1); break;    // crowded at the start
      case 4: x = w - 1 - std::min<uint64_t>(below(3), w - 1); break;
      case 5: x = below(2) ? heavy : below(w); break;            // one heavy code
      case 6: x = below(w); break;
      case 7: x = w >> below(62); x = x < w ? x : w - 1; break;  // on every scale
      case 8: x = heavy; break;
      default: x = i < n / 8 ? 0 : w - 1; break;                 // both ends
    }
    s[i] = (K)x;
  }
  std::sort(s, s + n);
  return n;
}

static int most_sp = 0, most_cuts = 0;

template <typename K, int PARTS>
static void check_cut(int kind, K width, int sp, int stack, int done, K* at, int* m) {
  K s[CUT_SAMPLES];
  const int n = sample(kind, width, s);
  *m = cut_points<K, PARTS>([&](int i) { return s[i]; }, n, width, sp, stack, done,
                     [&](int p, K x, K y) {
                       at[p] = x;
                       at[p + 1] = y;
                     });
  bool ok = *m >= 2 && *m <= CUT_PIECES && at[0] == 0 && sp + *m <= stack && at[*m] == width;
  for (int p = 0; ok && p < *m; ++p) {
    ok = at[p] < at[p + 1] && at[p + 1] - at[p] <= width - width / 8 + 1;
  }
  most_sp = std::max(most_sp, sp + *m);
  if (!ok) {
    std::printf("kind %d width %llu sp %d: %d pieces\n", kind, (unsigned long long)width, sp, *m);
    std::exit(1);
  }
}

// A path of cuts: the piece that goes on is the widest, the last or any one.
template <typename K, int PARTS>
static void path(uint64_t width0, int stack, int done) {
  K width = (K)width0;
  int sp = 0, cuts = 0;
  const int way = (int)below(4), one = (int)below(10);
  const bool mixed = below(2) != 0;
  while ((uint64_t)width > ((uint64_t)1 << done)) {
    K at[CUT_PIECES + 1];
    int m = 0;
    check_cut<K, PARTS>(mixed ? (int)below(10) : one, width, sp, stack, done, at, &m);
    const auto wide = [&](int p) { return at[p + 1] - at[p]; };
    int p = m - 1;
    if (way == 1) p = (int)below(m);
    if (way >= 2)
      for (int q = 0; q < m; ++q) p = wide(q) > wide(p) || (way == 3 && wide(q) == wide(p)) ? q : p;
    width = wide(p);
    sp += p;
    if (++cuts > 320) {   // 57 halvings, at most log(2) / log(8 / 7) = 5.2 cuts each
      std::printf("more than 320 cuts from %llu codes\n", (unsigned long long)width0);
      std::exit(1);
    }
  }
  most_cuts = std::max(most_cuts, cuts);
}

// A whole product: offsets (with repeats) of one interval, cut until a piece
// has at most `most` of them or 2^done codes; every offset is met once.
template <int PARTS>
static void whole(std::vector<uint64_t> x, uint64_t width0, size_t most, int stack, int done,
                  bool first_lanes) {
  std::sort(x.begin(), x.end());
  std::vector<uint64_t> lo(stack + CUT_PIECES), width(stack + CUT_PIECES);
  lo[0] = 0;
  width[0] = width0;
  size_t met = 0, cuts = 0;
  for (int sp = 1; sp > 0;) {
    --sp;
    const uint64_t a = lo[sp], w = width[sp];
    const auto b = std::lower_bound(x.begin(), x.end(), a), e = std::lower_bound(b, x.end(), a + w);
    const size_t k = (size_t)(e - b);
    if (k <= most || w <= ((uint64_t)1 << done)) {
      met += k;
      continue;
    }
    if (++cuts > 100000) {
      std::printf("a product of %zu offsets is cut without end\n", x.size());
      std::exit(1);
    }
    uint64_t s[CUT_SAMPLES];
    for (int i = 0; i < CUT_SAMPLES; ++i) s[i] = first_lanes ? *b - a : *(b + (long)below(k)) - a;
    std::sort(s, s + CUT_SAMPLES);
    const int m = cut_points<uint64_t, PARTS>([&](int i) { return s[i]; }, CUT_SAMPLES, w, sp, stack, done,
                                       [&](int p, uint64_t v, uint64_t y) {
                                         lo[sp + p] = a + v;
                                         width[sp + p] = y - v;
                                       });
    if (sp + m > stack) {
      std::printf("stack left: %d of %d\n", sp + m, stack);
      std::exit(1);
    }
    sp += m;
    most_sp = std::max(most_sp, sp);
  }
  if (met != x.size()) {
    std::printf("%zu of %zu offsets met\n", met, x.size());
    std::exit(1);
  }
}

template <int PARTS>
static void check(int stack, int done) {
  most_sp = most_cuts = 0;
  for (int k = 0; k < 100000; ++k) {
    const int log = done + 1 + (int)below(62 - done);
    uint64_t w = ((uint64_t)1 << (log - 1)) + 1 + below((uint64_t)1 << (log - 1));
    if (below(8) == 0) w = (uint64_t)1 << log;
    path<uint64_t, PARTS>(w, stack, done);
    if (w <= ((uint64_t)1 << 31)) path<uint32_t, PARTS>(w, stack, done);
  }
  for (int rep = 0; rep < 20; ++rep) {
    const uint64_t w = (uint64_t)1 << (20 + 2 * rep);
    std::vector<uint64_t> heavy(40000, 0), two(40000), many;
    heavy.push_back(below(w));
    for (size_t i = 0; i < two.size(); ++i) two[i] = i % 2 ? 100 : 0;
    for (int i = 0; i < 60000; ++i) many.push_back((w - 1) >> below(60));
    for (bool first : {false, true}) {
      whole<PARTS>(heavy, w, 7281, stack, done, first);
      whole<PARTS>(two, w, 29127, stack, done, first);
      whole<PARTS>(many, w, 1024, stack, done, first);
    }
  }
  std::printf("done 2^%d: stack %d of %d, %d cuts\n", done, most_sp, stack, most_cuts);
}

int main() {
  check<DIRECT_PARTS>(DIRECT_STACK, DIRECT_DONE_LOG);
  check<PACK_PARTS>(PACK_STACK, PACK_DONE_LOG);
  return 0;
}
