// kp_pack.hip -- many whole Laurent products in one fixed sequence of
// persistent launches.
//
// A pack keeps the products of a batch in a device task table.  Each stage is
// one launch of a fixed grid whose workgroups walk the work of every task, and
// the kernels read nothing but the table, so the sequence (the table's upload
// included) can be captured once into a HIP graph and replayed for every
// batch, whatever its products.
//
// Each product is the schoolbook sum of Section 3 over Kronecker codes
// (Section 2), restricted to intervals of output codes as Section 4 restricts
// threads: a workgroup finds the products of an interval from the factors
// sorted by code and adds them in LDS, indexed by code when the interval is no
// wider than the table (the dense array of Section 3.1), else in an
// open-addressing hash table keyed by code (Section 3.2).  Nonzero sums are
// decoded to exponents on the way out, and each task's count is posted to
// pinned host memory.
//
// The products used to be added in tables in device memory, one atomic or two
// per product: 1.07e7 products of 24 tasks of 50 to 2,000 terms took 1.31 ms,
// bound by atomics on the same few lines (8e9 a second), and 0.29 ms more to
// read the tables back (2.00 ms the whole batch).  In LDS they take 0.32 ms and
// nothing is read back; with sorting, counting and planning 0.38 ms (0.61 the
// batch).

#include <algorithm>
#include <climits>

#include "kp_cut.h"
#include "kp_internal.h"

namespace kp {

namespace {

constexpr int PACK_BOX_BLOCK = 1024;
constexpr int PACK_SORT_BLOCK = 1024;
constexpr int PACK_SLOTS = 2048;        // of an interval's table in LDS
constexpr int PACK_STEPS = 2;           // candidates per lane with their loads in flight
constexpr int PACK_COUNT_GROUPS = 16, PACK_COUNT_QUARTERS = 4;   // of cells and rows, for counting
constexpr int PACK_MAX_PROBE = 32;      // longer chains: the table counts as full
constexpr int PACK_PER_CU = 3;          // multiplying workgroups that fit a compute unit (LDS)
static_assert(PACK_SLOTS == 1 << PACK_DONE_LOG, "an interval the table indexes is not cut");

struct PackView {
  PackHeader* h;
  PackTask* tasks;
};

__device__ __forceinline__ PackView view(void* table) {
  return PackView{static_cast<PackHeader*>(table),
                  reinterpret_cast<PackTask*>(static_cast<char*>(table) + sizeof(PackHeader))};
}

// ------------------------------------------------------------ boxes
// One workgroup per array: per-variable minimum and maximum, posted as tagged
// words (side 0 the minima, side 1 the maxima) to host-mapped memory.

__global__ void __launch_bounds__(PACK_BOX_BLOCK)
k_pack_boxes(const int32_t* const* vals, const int64_t* ns, const int32_t* nvs, uint64_t* post,
             uint64_t seq) {
  __shared__ int32_t smin[KP_MAX_VARS][PACK_BOX_BLOCK / 64];
  __shared__ int32_t smax[KP_MAX_VARS][PACK_BOX_BLOCK / 64];
  const int g = blockIdx.x;
  const int64_t n = ns[g];
  const int32_t nv = nvs[g];
  const int32_t* __restrict__ x = vals[g];
  int32_t lo[KP_MAX_VARS], hi[KP_MAX_VARS];
#pragma unroll
  for (int v = 0; v < KP_MAX_VARS; ++v) {
    lo[v] = INT_MAX;
    hi[v] = INT_MIN;
  }
  // rows, one per thread at a time (each row's nv words)
  for (int64_t r = threadIdx.x; r < n; r += PACK_BOX_BLOCK) {
#pragma unroll
    for (int v = 0; v < KP_MAX_VARS; ++v)
      if (v < nv) {
        const int32_t e = x[r * nv + v];
        lo[v] = min(lo[v], e);
        hi[v] = max(hi[v], e);
      }
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int v = 0; v < KP_MAX_VARS; ++v) {
    if (v >= nv) break;
    int32_t a = lo[v], b = hi[v];
    for (int off = 32; off > 0; off >>= 1) {
      a = min(a, __shfl_xor(a, off));
      b = max(b, __shfl_xor(b, off));
    }
    if (lane == 0) {
      smin[v][wave] = a;
      smax[v][wave] = b;
    }
  }
  __syncthreads();
  if (threadIdx.x < 2 * KP_MAX_VARS) {
    const int v = threadIdx.x % KP_MAX_VARS;
    const bool is_max = threadIdx.x >= KP_MAX_VARS;
    if (v < nv) {
      int32_t r = is_max ? INT_MIN : INT_MAX;
      for (int w = 0; w < PACK_BOX_BLOCK / 64; ++w)
        r = is_max ? max(r, smax[v][w]) : min(r, smin[v][w]);
      const uint64_t word = ((uint64_t)(uint32_t)seq << 32) | (uint32_t)r;
      __hip_atomic_store(&post[(size_t)g * 2 * KP_MAX_VARS + threadIdx.x], word, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_SYSTEM);
    }
  }
}

// ------------------------------------------------------------ sort
// One workgroup per (task, factor): codes of the terms, bucket histogram in
// LDS, bucket starts, and the terms by bucket (encoded twice rather than kept:
// a factor of a pack has some hundreds of terms).  Crowded columns are sorted
// within their buckets too, so that an interval finds exactly its own, and the
// task's cells are then bounded by a sorted sample of its products instead of
// being equally wide: a product of two factors of 600 terms crowded in one of
// 16,384 buckets would otherwise be one workgroup's work, with every product
// looked at for every interval.
__global__ void __launch_bounds__(PACK_SORT_BLOCK) k_pack_sort(void* table) {
  extern __shared__ __align__(8) int32_t hist[];
  __shared__ uint32_t s_ws[PACK_SORT_BLOCK / 64];
  __shared__ unsigned long long s_sq;
  __shared__ uint32_t s_most;   // columns of the fullest bucket
  const PackView P = view(table);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int u = blockIdx.x; u < 2 * P.h->ntasks; u += gridDim.x) {
    const PackTask& T = P.tasks[u >> 1];
    const int role = u & 1;                       // 0: rows, 1: columns
    const bool isb = (role == 1) != (T.swap != 0);
    const PackSet& S = T.set[role];
    const uint64_t* __restrict__ c = static_cast<const uint64_t*>(isb ? T.bc : T.ac);
    if (role == 0) {
      if (tid == 0) *T.count = 0;
      for (int k = tid; k < T.ncrowd && S.n > 0; k += PACK_SORT_BLOCK) T.cells[k] = 0;
    }
    if (tid == 0) {
      s_sq = 0;
      s_most = 0;
    }
    for (int k = tid; k < S.nbk; k += PACK_SORT_BLOCK) hist[k] = 0;
    __syncthreads();
    uint32_t bad = 0;
    // (codes outside the planned box are reported; the clamp keeps them inside
    // the buckets)
    const auto code_in = [&](const DevLayout& L, const int32_t* __restrict__ x, int64_t maxc,
                             int64_t r) -> int64_t {
      int64_t k = 0;
      for (int v = 0; v < L.nx; ++v) {
        const int32_t e = x[r * L.nx + v];
        if (e < L.fmin[v] || e > L.fmax[v]) bad |= ERR_RANGE;
        k += L.xc[v] * (int64_t)(e - L.fmin[v]);
      }
      return k < 0 ? 0 : k > maxc ? maxc : k;
    };
    const auto code_of = [&](int64_t r) {
      return code_in(isb ? T.lb : T.la, isb ? T.bx : T.ax, S.maxc, r);
    };
    for (int64_t r = tid; r < S.n; r += PACK_SORT_BLOCK)
      S.rank[r] = atomicAdd(&hist[code_of(r) >> S.shift], 1);
    __syncthreads();
    // exclusive scan: each wavefront a contiguous stretch of buckets, 64 at a time
    const int per = (S.nbk + PACK_SORT_BLOCK - 1) / PACK_SORT_BLOCK * 64;
    const int b0 = min(S.nbk, wave * per), b1 = min(S.nbk, b0 + per);
    uint32_t sum = 0, most = 0;
    uint64_t sq = 0;
    for (int b = b0; b < b1; b += 64) {
      const uint32_t v = b + lane < b1 ? (uint32_t)hist[b + lane] : 0u;
      sum += lane_value(wave_scan_add(v), 63);
      most = max(most, v);
      sq += (uint64_t)v * v;
    }
    if (lane == 0) s_ws[wave] = sum;
    if (role == 1 && sq) atomicAdd(&s_sq, (unsigned long long)sq);
    if (role == 1) {
      most = lane_value(wave_scan_max(most), 63);
      if (lane == 0) atomicMax(&s_most, most);
    }
    __syncthreads();
    uint32_t run = 0;
    for (int w = 0; w < wave; ++w) run += s_ws[w];
    for (int b = b0; b < b1; b += 64) {
      const uint32_t v = b + lane < b1 ? (uint32_t)hist[b + lane] : 0u;
      const uint32_t incl = wave_scan_add(v);
      if (b + lane < b1) hist[b + lane] = S.start[b + lane] = (int32_t)(run + incl - v);
      run += lane_value(incl, 63);
    }
    if (tid == 0) S.start[S.nbk] = (int32_t)S.n;
    __syncthreads();
    // (a product of fewer than 64 codes a pair has directly indexed
    // intervals, or not many times more: simplices share a bucket with 30, and
    // exact intervals cost them 130 us of a batch's 710 for nothing)
    const int64_t pairs = S.n * T.set[0].n;
    const bool thin = role == 1 && pairs > 0 && T.nkeys / 64 >= pairs;
    bool crowd = thin && s_sq > (uint64_t)CROWDED * (uint64_t)max(S.n, S.n * S.n / S.nbk);
    // Rows that crowd make crowds of products of columns that do not: when one
    // bucket of columns could give an interval many times its products, a
    // sample of the products tells whether any has them (random terms, ten to
    // the fullest bucket, do without up to 2,000 rows).
    const bool look = crowd || (thin && (int64_t)s_most * T.set[0].n >
                                            max((int64_t)PACK_PEAK, pairs / 256));
    if (look) {   // the same for every thread
      __syncthreads();   // hist has been read (start[] has the buckets)
      const PackSet& A = T.set[0];
      int64_t* key = reinterpret_cast<int64_t*>(hist);
      for (int o = tid; o < T.ncrowd; o += PACK_SORT_BLOCK)
        key[o] = code_in(isb ? T.la : T.lb, isb ? T.ax : T.bx, A.maxc, sample_of(o, 0, A.n)) +
                 code_of(sample_of(o, PACK_CROWD_CELLS, S.n));
      __syncthreads();
      block_sort<PACK_SORT_BLOCK>(key, T.ncrowd);
      crowd = samples_crowd<PACK_SORT_BLOCK>(key, T.ncrowd, T.cw, (double)PACK_HASHED,
                                             (double)pairs) || crowd;
      if (crowd)
        for (int o = tid; o <= T.ncrowd; o += PACK_SORT_BLOCK)
          T.bounds[o] = sample_bound(key, T.ncrowd, o, T.nkeys);
    }
    if (role == 1 && tid == 0) *T.crowd = crowd ? 1u : 0u;
    const int32_t* start = look ? S.start : hist;
    for (int64_t r = tid; r < S.n; r += PACK_SORT_BLOCK) {
      const int64_t k = code_of(r);
      const int64_t at = start[k >> S.shift] + S.rank[r];
      if (crowd) {
        T.tmp_k[at] = k;
        T.tmp_i[at] = (int32_t)r;
      } else {
        S.k[at] = k;
        S.c[at] = c[r];
      }
    }
    if (crowd) {   // the same for every thread
      __syncthreads();
      // merge sort: a term's place in two merged runs is its own index plus the
      // terms of the other run before it (the ranks are no longer needed)
      int64_t *src = T.tmp_k, *dst = S.k;
      int32_t *si = T.tmp_i, *di = S.rank;
      for (int64_t run = 1; run < S.n; run *= 2) {
        for (int64_t t = tid; t < S.n; t += PACK_SORT_BLOCK) {
          const int64_t k = src[t], first = t / (2 * run) * (2 * run);
          const bool left = t < first + run;
          const int64_t o0 = left ? min(S.n, first + run) : first;
          const int64_t o1 = left ? min(S.n, first + 2 * run) : first + run;
          // (equal codes: the left run's terms first)
          const int64_t o = first_from(src, (uint32_t)o0, (uint32_t)o1, left ? k : k + 1);
          const int64_t at = first + (t - (left ? first : first + run)) + (o - o0);
          dst[at] = k;
          di[at] = si[t];
        }
        __syncthreads();
        int64_t* const k0 = src;
        src = dst;
        dst = k0;
        int32_t* const i0 = si;
        si = di;
        di = i0;
      }
      for (int64_t t = tid; t < S.n; t += PACK_SORT_BLOCK) {
        S.c[t] = c[si[t]];
        if (src != S.k) S.k[t] = src[t];
      }
    }
    if (bad) atomicOr(&P.h->err, bad);
    __syncthreads();   // the next factor clears hist
  }
}

// ------------------------------------------------------------ intervals
// Cell c of a task: its first code and the one after its last (no cell: both 0).
__device__ __forceinline__ void cell_of(const PackTask& T, bool crowd, int c, int64_t* lo,
                                        int64_t* end) {
  *lo = *end = 0;
  if (crowd) {
    *lo = T.bounds[c];
    *end = T.bounds[c + 1];
  } else if (c < T.ncell) {
    *lo = (int64_t)c << T.cw;
    *end = min(T.nkeys, *lo + ((int64_t)1 << T.cw));
  }
}
// The columns of codes xlo .. xhi (in a crowded task exactly, else their
// whole buckets).
__device__ __forceinline__ void columns_of(const PackSet& B, bool crowd, int64_t xlo, int64_t xhi,
                                           uint32_t* j0, uint32_t* j1) {
  const int64_t lo = max((int64_t)0, min(xlo, B.maxc)), hi = max((int64_t)0, min(xhi, B.maxc));
  const int64_t q0 = lo >> B.shift, q1 = hi >> B.shift;
  *j0 = (uint32_t)B.start[q0];
  *j1 = (uint32_t)B.start[q1 + 1];
  if (crowd) {   // (each end by itself: they may lie in one bucket or in two)
    *j0 = first_from(B.k, *j0, (uint32_t)B.start[q0 + 1], lo);
    *j1 = first_from(B.k, (uint32_t)B.start[q1], *j1, hi + 1);
  }
}

// The products of each cell of 2^cw codes (whole buckets of the columns: a
// bound): one workgroup per task, 64 cells and a quarter of the rows, a cell
// per lane and a slice of the rows per wavefront, four rows' loads in flight.
// (Sixteen groups of cells for the sake of crowded tasks, which have up to
// 4,096 cells: with the four of the others one such task of 6,000 x 6,000 terms
// took 4 ms to count.)
__global__ void __launch_bounds__(PACK_BLOCK) k_pack_count(void* table) {
  constexpr int GROUPS = PACK_COUNT_GROUPS, QUARTERS = PACK_COUNT_QUARTERS;
  __shared__ unsigned long long s_count[64];
  const PackView P = view(table);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int FIRST = PACK_CELLS / 64;   // groups of a task that is not crowded
  const int units = P.h->ntasks * GROUPS * QUARTERS, first = P.h->ntasks * FIRST * QUARTERS;
  for (int u = blockIdx.x; u < units; u += gridDim.x) {
    // (the groups that every task has come first)
    const int v = u < first ? u : u - first, per_task = u < first ? FIRST : GROUPS - FIRST;
    const PackTask& T = P.tasks[v / (per_task * QUARTERS)];
    const int group = (v / QUARTERS) % per_task + (u < first ? 0 : FIRST), quarter = v % QUARTERS;
    const int64_t* __restrict__ ak = T.set[0].k;
    const PackSet B = T.set[1];
    const int64_t an = T.set[0].n, per = (an + QUARTERS - 1) / QUARTERS;
    const bool crowd = B.n > 0 && *T.crowd != 0;
    const int64_t i1 = min(an, per * (quarter + 1));
    for (int c0 = group * 64; c0 < (crowd ? T.ncrowd : T.ncell); c0 += GROUPS * 64) {
      const int c = c0 + lane;
      if (tid < 64) s_count[tid] = 0;
      __syncthreads();
      int64_t lo, hi;
      cell_of(T, crowd, c, &lo, &hi);
      if (hi > lo) {
        hi -= 1;
        unsigned long long n = 0;
#pragma unroll 4
        for (int64_t i = per * quarter + wave; i < i1; i += PACK_BLOCK / 64) {
          const int64_t a = ak[i], xlo = lo - a, xhi = hi - a;
          uint32_t j0, j1;
          columns_of(B, crowd, xlo, xhi, &j0, &j1);
          n += xhi >= 0 && xlo <= B.maxc ? (unsigned long long)(j1 - j0) : 0ull;
        }
        if (n) atomicAdd(&s_count[lane], n);
      }
      __syncthreads();
      if (tid < 64 && s_count[lane]) atomicAdd(&T.cells[c], s_count[lane]);
      __syncthreads();   // the next cells clear s_count
    }
  }
}

// One workgroup per task: the intervals of its cells.  A cell is cut into
// intervals that the table indexes directly (at most PACK_SLOTS codes, about
// PACK_DENSE products) or into hashed ones of about PACK_HASHED products,
// whichever are fewer.
__global__ void __launch_bounds__(PACK_BLOCK) k_pack_plan(void* table) {
  __shared__ int64_t s_ws[PACK_BLOCK / 64];
  __shared__ int64_t s_first;
  const PackView P = view(table);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int t = blockIdx.x; t < P.h->ntasks; t += gridDim.x) {
    const PackTask& T = P.tasks[t];
    const bool live = T.set[1].n > 0, crowd = live && *T.crowd != 0;
    const int cells = live ? (crowd ? T.ncrowd : T.ncell) : 0;
    const int per = (cells + PACK_BLOCK - 1) / PACK_BLOCK;
    const int c0 = min(cells, tid * per), c1 = min(cells, c0 + per);
    const auto block_sum = [&](int64_t v, int64_t* before) -> int64_t {
      int64_t incl = v;
      for (int off = 1; off < 64; off <<= 1) {
        const int64_t y = __shfl_up(incl, off);
        if (lane >= off) incl += y;
      }
      __syncthreads();
      if (lane == 63) s_ws[wave] = incl;
      __syncthreads();
      int64_t tot = 0, b = 0;
      for (int w = 0; w < PACK_BLOCK / 64; ++w) {
        if (w < wave) b += s_ws[w];
        tot += s_ws[w];
      }
      *before = b + incl - v;
      return tot;
    };
    int64_t before, n = 0;
    for (int c = c0; c < c1; ++c) n += (int64_t)T.cells[c];
    const int64_t all = block_sum(n, &before);
    // hashed intervals are made larger when they would outgrow the task's array
    const int64_t room = max((int64_t)1, T.max_units - cells);
    const int64_t target = max((int64_t)PACK_HASHED, (all + room - 1) / room);
    // (sampled cells, which are uneven, are taken together while they fill one interval)
    const auto each_run = [&](auto&& each) {
      each_interval(c0, c1, crowd, target, INT64_MAX,
                    [&](int64_t c, int64_t* lo, int64_t* end) { cell_of(T, crowd, (int)c, lo, end); },
                    [&](int64_t c) { return (int64_t)T.cells[c]; },
                    [&](int64_t m, int64_t width) {
                      const int64_t dense = max((m + PACK_DENSE - 1) / PACK_DENSE,
                                                (width + PACK_SLOTS - 1) / PACK_SLOTS);
                      return min((m + target - 1) / target, dense);
                    },
                    each);
    };
    int64_t mine = 0;
    each_run([&](int64_t, int64_t, int64_t k) { mine += k; });
    const int64_t total = block_sum(mine, &before);
    if (tid == 0) s_first = (int64_t)atomicAdd(&P.h->nunits, (unsigned long long)total);
    __syncthreads();
    PackUnit* out = P.h->units + s_first + before;
    each_run([&](int64_t lo, int64_t end, int64_t k) {
      const int64_t width = end - lo, step = (width + k - 1) / k;
      for (int64_t u = 0; u < k; ++u) {
        const int64_t a = min(width, u * step), z = min(width, a + step);
        *out++ = PackUnit{lo + a, z - a, t};
      }
    });
    __syncthreads();   // the next task uses s_ws
  }
}

// ------------------------------------------------------------ multiply
__device__ __forceinline__ void add_value(uint64_t* p, bool f64, uint64_t a, uint64_t b) {
  if (f64) {
    atomicAdd(reinterpret_cast<double*>(p), __longlong_as_double((long long)a) *
                                                __longlong_as_double((long long)b));
  } else {
    atomicAdd(reinterpret_cast<unsigned long long*>(p), (unsigned long long)(a * b));   // wraps modulo 2^64
  }
}

__device__ __forceinline__ uint32_t pack_hash(uint64_t k) {   // top bits depend on all of k
  uint32_t h = ((uint32_t)(k >> 32) * 0x9E3779B1u) ^ (uint32_t)k;
  h *= 0x9E3779B1u;
  h ^= h >> 15;
  return h * 0x85EBCA6Bu;
}

// What the decode of one variable takes, and its exponent of the code whose
// quotient by the widths before it is q.
struct PackDigit {
  FastDiv d;
  FastDiv32 d32;
  int32_t least;
};
__device__ __forceinline__ int32_t pack_digit(const PackDigit& D, uint64_t& q) {
  uint32_t e;
  if ((q >> 32) == 0 && D.d32.d != 0) {
    const uint32_t n = (uint32_t)q, qq = fdiv32(n, D.d32);
    e = n - qq * D.d32.d;
    q = qq;
  } else {
    const uint64_t qq = fdiv(q, D.d);
    e = (uint32_t)(q - qq * D.d.d);
    q = qq;
  }
  return (int32_t)e + D.least;
}

// A set of the table in scalar registers.
template <typename P>
__device__ __forceinline__ P* uniform_ptr(P* p) {
  return reinterpret_cast<P*>(uniform(reinterpret_cast<uint64_t>(p)));
}
__device__ __forceinline__ PackSet uniform_set(const PackSet& s) {
  PackSet r;
  r.n = uniform(s.n);
  r.maxc = uniform(s.maxc);
  r.shift = (int32_t)uniform((uint32_t)s.shift);
  r.nbk = 0;
  r.rank = nullptr;
  r.start = uniform_ptr(s.start);
  r.k = uniform_ptr(s.k);
  r.c = uniform_ptr(s.c);
  return r;
}

// What bounds it: the latency of row -> columns -> slot (wavefronts wait 65 % of
// their cycles; the vector units are busy 26 %, the LDS 22 %) at three workgroups
// of 52 KB of LDS per compute unit, not bytes.  Intervals are taken
// at a fixed stride: handing them out from one counter cost 1.03 ms instead of
// 0.41 on the batch named above, 64 coarser cells a task 1.2 ms, probe chains
// of up to 256 slots 1.9 ms.  A wavefront waits for its longest chain, so a
// table that fills is given up early (the walk ends, chains of 32 in growing
// steps): 0.32 ms instead of 0.41.
// The grid takes the intervals of every task; see the head of the file.  A
// full table (only codes crowded in part of a cell make one, intervals being
// sized from their cell's products) has its interval cut at keys that it holds;
// one of at most PACK_SLOTS codes is indexed directly and always fits.  Those
// keys are of the rows walked so far, the least ones: a piece may hold nearly
// all that is left, which is why the cut's own bounds (kp_cut.h) keep the stack.
__global__ void __launch_bounds__(PACK_BLOCK, PACK_PER_CU) k_pack_mul(void* table) {
  constexpr int NW = PACK_BLOCK / 64, PER = PACK_SLOTS / PACK_BLOCK;
  __shared__ uint64_t keys[PACK_SLOTS], vals[PACK_SLOTS];
  __shared__ uint64_t row_off[NW][64], row_coef[NW][64];
  __shared__ uint32_t row_col[NW][64];
  __shared__ uint16_t seg[NW][PACK_STEPS * 64];
  __shared__ uint32_t s_cnt[NW], s_next, s_over;
  __shared__ int64_t s_base, s_lo[PACK_STACK];
  __shared__ PackDigit s_dig[KP_MAX_VARS];   // the task's decode
  __shared__ uint64_t s_width[PACK_STACK];
  __shared__ int s_pieces;                   // of a cut
  const PackView P = view(table);
  const unsigned long long units = P.h->nunits;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (unsigned long long u = blockIdx.x; u < units; u += gridDim.x) {
    const PackUnit unit = P.h->units[u];
    const PackTask& T = P.tasks[uniform((uint32_t)unit.task)];
    const PackSet A = uniform_set(T.set[0]), B = uniform_set(T.set[1]);
    const bool f64 = T.f64 != 0, crowd = *T.crowd != 0;
    // (counts of a batch are 32-bit)
    const uint32_t batch = B.n < ((int64_t)1 << 26) ? 64u : 1u;
    const int nx = (int)uniform((uint32_t)T.la.nx);
    if (tid < nx) s_dig[tid] = PackDigit{T.la.dx[tid], T.la.dx32[tid], (int32_t)T.la.xmin[tid]};
    if (tid == 0) {
      s_lo[0] = unit.lo;
      s_width[0] = (uint64_t)unit.width;
    }
    __syncthreads();
    for (int sp = 1; sp > 0;) {
      --sp;
      const int64_t lo = uniform(s_lo[sp]);
      const uint64_t width = uniform(s_width[sp]);
      const bool direct = width <= PACK_SLOTS;
#pragma unroll
      for (int r = 0; r < PER; ++r) {
        keys[r * PACK_BLOCK + tid] = ~0ull;
        vals[r * PACK_BLOCK + tid] = 0;
      }
      if (tid == 0) s_next = s_over = 0;
      __syncthreads();
      const int64_t hi = lo + (int64_t)width - 1, amin = lo - B.maxc;
      uint32_t i0 = 0, i1 = 0;
      if (width > 0 && amin <= A.maxc) {   // rows that meet the interval
        i0 = (uint32_t)A.start[max((int64_t)0, amin) >> A.shift];
        i1 = (uint32_t)A.start[(min(hi, A.maxc) >> A.shift) + 1];
      }
      for (;;) {
        uint32_t bt = 0;
        if (lane == 0) bt = atomicAdd(&s_next, batch);
        const uint32_t ib = i0 + lane_value(bt, 0);
        if (ib >= i1 || *(volatile uint32_t*)&s_over) break;
        const uint32_t i = min(ib + lane, i1 - 1);
        const int64_t a = A.k[i], xlo = lo - a, xhi = hi - a;
        const bool in = lane < (int)batch && ib + lane < i1 && xhi >= 0 && xlo <= B.maxc;
        uint32_t j0, j1;
        columns_of(B, crowd, xlo, xhi, &j0, &j1);
        const uint32_t cnt = in ? j1 - j0 : 0u;
        const uint32_t incl = wave_scan_add(cnt), excl = incl - cnt;
        const uint32_t total = lane_value(incl, 63);
        wave_sync();
        row_col[wave][lane] = j0 - excl;
        row_off[wave][lane] = (uint64_t)(a - lo);
        row_coef[wave][lane] = A.c[i];
        uint32_t carry = 0;
        // candidates 64 at a time: candidate q belongs to the last row whose
        // first candidate is at or before it
        for (uint32_t q0 = 0; q0 < total; q0 += PACK_STEPS * 64) {
          if (uniform(*(volatile uint32_t*)&s_over)) break;
#pragma unroll
          for (int v = 0; v < PACK_STEPS; ++v) seg[wave][v * 64 + lane] = 0;
          wave_sync();
          if (cnt && excl - q0 < PACK_STEPS * 64u) seg[wave][excl - q0] = (uint16_t)lane;
          wave_sync();
          uint64_t off[PACK_STEPS], ca[PACK_STEPS], cb[PACK_STEPS];
#pragma unroll
          for (int v = 0; v < PACK_STEPS; ++v) {
            const uint32_t m = max(carry, wave_scan_max(seg[wave][v * 64 + lane]));
            carry = lane_value(m, 63);
            const uint32_t j = row_col[wave][m] + min(q0 + v * 64 + lane, total - 1);
            off[v] = row_off[wave][m] + (uint64_t)B.k[j];
            ca[v] = row_coef[wave][m];
            cb[v] = B.c[j];
          }
          wave_sync();
#pragma unroll
          for (int v = 0; v < PACK_STEPS; ++v) {
            if (q0 + v * 64 + lane >= total || off[v] >= width) continue;
            uint32_t s = (uint32_t)off[v];
            if (!direct) {
              const unsigned long long key = off[v];
              s = pack_hash(key) >> 21;
              unsigned long long c =
                  atomicCAS(reinterpret_cast<unsigned long long*>(&keys[s]), ~0ull, key);
              int q = 0;
#pragma nounroll
              while (c != ~0ull && c != key && q < PACK_MAX_PROBE) {
                ++q;
                s = (s + q) & (PACK_SLOTS - 1);   // every slot once, in growing steps
                c = atomicCAS(reinterpret_cast<unsigned long long*>(&keys[s]), ~0ull, key);
              }
              if (c != ~0ull && c != key) {
                s_over = 1;
                continue;
              }
            }
            add_value(&vals[s], f64, ca[v], cb[v]);
          }
        }
      }
      __syncthreads();
      if (s_over) {   // the same for every thread
        __syncthreads();
        if (wave == 0) {
          const uint64_t key = keys[lane * (PACK_SLOTS / CUT_SAMPLES)];
          int rank = 0;
#pragma unroll 8
          for (int o = 0; o < CUT_SAMPLES; ++o) {
            const uint64_t y = keys[o * (PACK_SLOTS / CUT_SAMPLES)];
            rank += y < key || (y == key && o < lane) ? 1 : 0;
          }
          const int n = (int)__popcll(__ballot(key != ~0ull));   // (empty slots are the greatest)
          uint64_t* sorted = row_off[0];   // (no row is being walked)
          sorted[rank] = key;
          wave_sync();
          // (the same in every lane)
          const int m = cut_points<uint64_t, PACK_PARTS>([&](int i) { return uniform(sorted[i]); }, n, width,
                                             sp, PACK_STACK, PACK_DONE_LOG,
                                             [&](int p, uint64_t x, uint64_t y) {
                                               s_lo[sp + p] = lo + (int64_t)x;
                                               s_width[sp + p] = y - x;
                                             });
          if (lane == 0) s_pieces = m;
        }
        __syncthreads();
        sp += (int)uniform((uint32_t)s_pieces);
        continue;
      }
      // nonzero sums (for fp64 both signed zeros are dropped) to the front of
      // each wavefront's stretch, then out at slots taken from the task's counter
      const int r0 = wave * PER * 64;
      uint64_t kk[PER], vv[PER], ball[PER];
      uint32_t cnt = 0;
#pragma unroll
      for (int r = 0; r < PER; ++r) {
        const int s = r0 + r * 64 + lane;
        kk[r] = direct ? (uint64_t)s : keys[s];
        vv[r] = vals[s];
        ball[r] = __ballot(f64 ? (vv[r] << 1) != 0 : vv[r] != 0);
        cnt += (uint32_t)__popcll(ball[r]);
      }
      if (lane == 0) s_cnt[wave] = cnt;
      __syncthreads();
      uint32_t tot = 0, before = 0;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        if (w < wave) before += s_cnt[w];
        tot += s_cnt[w];
      }
      if (tid == 0)
        s_base = tot ? (int64_t)atomicAdd(T.count, (unsigned long long)tot) : 0;
      uint32_t pos = 0;
#pragma unroll
      for (int r = 0; r < PER; ++r) {
        if (ball[r] & (1ull << lane)) {
          const uint32_t at = r0 + pos + (uint32_t)__popcll(ball[r] & ((1ull << lane) - 1));
          keys[at] = kk[r];
          vals[at] = vv[r];
        }
        pos += (uint32_t)__popcll(ball[r]);
      }
      __syncthreads();
      const int64_t out0 = s_base + before;
      int32_t* ox = uniform_ptr(T.out_x);
      int64_t* oc = uniform_ptr(static_cast<int64_t*>(T.out_c));
      const int64_t cap = uniform(T.out_cap);
      for (uint32_t t = lane; t < cnt; t += 64) {
        const int64_t at = out0 + t;
        if (at >= cap) break;
        uint64_t c = (uint64_t)lo + keys[r0 + t];
        for (int v = 0; v < nx; ++v) ox[at * nx + v] = pack_digit(s_dig[v], c);
        oc[at] = (int64_t)vals[r0 + t];
      }
      __syncthreads();   // the next interval clears the table
    }
  }
}

// ------------------------------------------------------------ counts
// One workgroup: every task's count (or -(status) after a device error) as
// two tagged words in host-mapped memory.
__global__ void __launch_bounds__(PACK_BLOCK) k_pack_post(void* table) {
  const PackView P = view(table);
  const int nt = P.h->ntasks;
  const uint32_t err = P.h->err;
  const uint64_t tag = (uint64_t)(uint32_t)P.h->seq << 32;
  for (int k = threadIdx.x; k < nt; k += PACK_BLOCK) {
    int64_t n = (int64_t)*P.tasks[k].count;
    if (n > P.tasks[k].out_cap) n = -(int64_t)KP_E_CAPACITY;
    if (err) n = -(int64_t)first_error(err);
    const uint64_t w = (uint64_t)n;
    __hip_atomic_store(&P.h->post[2 * k], tag | (w & 0xffffffffu), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&P.h->post[2 * k + 1], tag | (w >> 32), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

}  // namespace

size_t pack_table_bytes(int max_tasks) {
  return sizeof(PackHeader) + sizeof(PackTask) * (size_t)max_tasks;
}

hipError_t launch_pack_boxes(const int32_t* const* vals, const int64_t* n, const int32_t* nv,
                             int nseg, uint64_t* post_dev, uint64_t seq, hipStream_t s) {
  if (nseg <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_pack_boxes, dim3((unsigned)nseg), dim3(PACK_BOX_BLOCK), 0, s, vals, n, nv,
                     post_dev, seq);
  return hipGetLastError();
}

hipError_t pack_setup() {   // once per context's device
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&k_pack_sort),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)(PACK_BUCKETS * 4));
}

hipError_t launch_pack_run(void* table_dev, int max_tasks, int num_cu, hipStream_t s) {
  const int tasks = std::min(2 * max_tasks, num_cu);
  hipLaunchKernelGGL(k_pack_sort, dim3((unsigned)tasks), dim3(PACK_SORT_BLOCK),
                     (size_t)PACK_BUCKETS * 4, s, table_dev);
  const int counts = std::min(PACK_COUNT_GROUPS * PACK_COUNT_QUARTERS * max_tasks, 8 * num_cu);
  hipLaunchKernelGGL(k_pack_count, dim3((unsigned)counts), dim3(PACK_BLOCK), 0, s, table_dev);
  hipLaunchKernelGGL(k_pack_plan, dim3((unsigned)std::min(max_tasks, num_cu)), dim3(PACK_BLOCK),
                     0, s, table_dev);
  hipLaunchKernelGGL(k_pack_mul, dim3((unsigned)(PACK_PER_CU * num_cu)), dim3(PACK_BLOCK), 0, s,
                     table_dev);
  hipLaunchKernelGGL(k_pack_post, dim3(1), dim3(PACK_BLOCK), 0, s, table_dev);
  return hipGetLastError();
}

}  // namespace kp
