// kp_direct.hip -- hash accumulation of sparse products straight from the
// sorted factors: nothing is written before the result.
//
// Section 3.2 accumulates the products of a highly sparse multiplication in a
// hash table keyed by the product's code, and Section 4 lets every thread work
// on an interval of output codes of its own.  Here one workgroup takes an
// interval of output codes, finds the products that fall into it from the
// sorted factors (for each row, the terms of an interval of the columns), and
// tells in LDS which of them meet in one code.  No product and no grouping
// goes through HBM: the traffic is the factors (which stay in the L2) and the
// result.
//
// Intervals: the code space is cut into cells of 2^cw codes; a counting pass
// bounds the products of every cell, and a cell is cut into equal intervals of
// about `target` products.  Crowded columns (a box that an outlier makes huge),
// and columns whose products crowd because the rows do, are sorted within their
// buckets too, so that a row finds exactly the columns of an interval, and the
// cells are then bounded by a sorted sample of the products: 600 x 900 terms of
// three variables in [0, 24) and one outlier each would otherwise be one
// workgroup's, 95 ms instead of 0.31 (0.50 through the groups); 5,000 x 6,000
// terms of five variables take 1.9 ms (141 through the groups); 5,000 rows in a
// box and 5,000 columns, 400 of them in a clump, 0.73 instead of 4.2 (1.06).
//
// Five launches in all (sort, count, plan, multiply, finish), and three more for
// a factor of more than 4,096 terms (place, and chunk and order, which end at
// once unless the columns crowd), against eighteen of the range-grouped layout,
// which writes every product to HBM once before it is accumulated.  Measured,
// whole call: 7,919 x 12,347 terms in five variables, fp64, 3.15 -> 1.66 ms; 500
// x 500 terms, int64, 0.150 -> 0.105 ms.
#include <algorithm>
#include <climits>
#include <type_traits>

#include "kp_cut.h"
#include "kp_internal.h"

namespace kp {

namespace {

constexpr int SORT_BLOCK = 1024;
constexpr int SMALL_BLOCK = 256;
constexpr int COUNT_CELLS = 8;          // cells per counting workgroup
constexpr int PLAN_BLOCK = 1024;
constexpr uint32_t HASH_MUL = 0x9E3779B1u;  // odd, 2^32 / golden ratio
constexpr uint32_t PART_MUL = 0x85EBCA6Bu;  // odd: the table's hash
constexpr int MAX_PROBE = 64;   // a longer chain means a full table
constexpr int PARTS = 72;   // stretches still to do, one more per halving
constexpr int ROWS = 1;     // rows per lane and batch
constexpr int STEPS = 2;    // candidates per lane with their loads in flight

// A bijection of 32 bits whose top bits depend on all of the key's: products'
// codes are sums of digits times strides, which a multiplication alone leaves
// clustered.
__device__ __forceinline__ uint32_t mix(uint32_t k) {
  k *= HASH_MUL;
  k ^= k >> 15;
  return k * PART_MUL;
}
__device__ __forceinline__ uint32_t mix(uint64_t k) {
  return mix((uint32_t)k ^ mix((uint32_t)(k >> 32)));
}

// ------------------------------------------------------------ sorted sets
// Code of term i of a set, checked against the set's box.
__device__ __forceinline__ int64_t set_code(const DirectSet& S, int64_t i, uint32_t* err) {
  const int64_t c = S.k_in[i];
  if (c >= 0 && c <= S.maxc) return c;
  *err |= ERR_RANGE;
  return c < 0 ? 0 : S.maxc;
}
__device__ __forceinline__ void place_term(const DirectArgs& R, const DirectSet& S, int64_t i,
                                           int64_t code, int64_t at) {
  if (S.k64) S.k64[at] = code;
  if (S.k32) S.k32[at] = (uint32_t)code;
  S.c[at] = S.c_in[i];
  if (R.field) {
    // the term's digits over the product's widths, in fields that add up to
    // the product's digits
    uint64_t q = (uint64_t)code, w[2] = {0, 0};
    for (int k = 0; k < R.dec.nx; ++k) {
      const uint64_t qq = fdiv(q, R.dec.dx[k]), e = q - qq * R.dec.dx[k].d;
      q = qq;
      const int bit = k * 8 * R.field;
      if (bit < 64) w[0] |= e << bit;
      else w[1] |= e << (bit - 64);
    }
    S.px[at] = make_uint4((uint32_t)w[0], (uint32_t)(w[0] >> 32), (uint32_t)w[1],
                          (uint32_t)(w[1] >> 32));
  }
}

// Term t of the crowded columns by bucket, to its place among the terms
// [b0, b1) of its bucket.
__device__ __forceinline__ void place_sorted(const DirectArgs& R, const DirectSet& S, int64_t t,
                                             int32_t b0, int32_t b1) {
  const int64_t k = R.tmp_k[t];
  int32_t at = b0;
#pragma unroll 4
  for (int32_t o = b0; o < b1; ++o) {
    const int64_t y = R.tmp_k[o];
    at += y < k || (y == k && o < t) ? 1 : 0;
  }
  place_term(R, S, R.tmp_i[t], k, at);
}

// Sorts the terms [first, first + n) of the crowded columns by bucket in LDS
// (DIRECT_PLACE at most; `mem` holds twelve bytes for each of their next power
// of two): the codes at mem, their terms where it returns.  The workgroup calls
// it together, after a barrier of its own.
__device__ __forceinline__ const int32_t* sort_chunk(const DirectArgs& R, int64_t first, int n,
                                                     void* mem) {
  int size = 1;
  while (size < n) size <<= 1;
  int64_t* key = static_cast<int64_t*>(mem);
  int32_t* term = reinterpret_cast<int32_t*>(key + size);
  for (int t = threadIdx.x; t < size; t += SORT_BLOCK) {
    key[t] = t < n ? R.tmp_k[first + t] : INT64_MAX;
    term[t] = t < n ? R.tmp_i[first + t] : t;
  }
  __syncthreads();
  block_sort_terms<SORT_BLOCK>(key, term, size);
  return term;
}

// One workgroup per set: bucket histogram of its codes in LDS, each term's
// rank in its bucket, bucket starts.  Sets of at most DIRECT_PLACE terms are
// also placed here (one launch less; more terms than that are placed by many
// workgroups, one compute unit being slow at scattered stores).  The first
// workgroup clears the cells' counters.
__global__ void __launch_bounds__(SORT_BLOCK) k_rd_sort(DirectArgs R) {
  extern __shared__ __align__(8) int32_t hist[];
  __shared__ uint32_t s_ws[SORT_BLOCK / 64 + 1];
  __shared__ unsigned long long s_sq;
  __shared__ uint32_t s_most;   // terms of the fullest bucket
  if (threadIdx.x == 0) {
    s_sq = 0;
    s_most = 0;
  }
  const DirectSet& S = R.set[blockIdx.x];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int64_t k = tid; k < S.nbk; k += SORT_BLOCK) hist[k] = 0;
  if (blockIdx.x == 0)
    for (int64_t k = tid; k < max(R.ncell, (int64_t)R.ncrowd); k += SORT_BLOCK) R.ccount[k] = 0;
  __syncthreads();
  uint32_t err = 0;
  uint64_t cmin = ~0ull, cmax = 0;   // sizes of the coefficients (fp64: of their bits)
  for (int64_t i = tid; i < S.n; i += SORT_BLOCK) {
    S.rank[i] = atomicAdd(&hist[set_code(S, i, &err) >> S.shift], 1);
    const uint64_t coef = S.c_in[i];
    const uint64_t size = R.f64 ? coef & 0x7FFFFFFFFFFFFFFFull
                                : (int64_t)coef < 0 ? 0ull - coef : coef;
    cmin = size < cmin ? size : cmin;
    cmax = size > cmax ? size : cmax;
  }
  __syncthreads();
  // exclusive scan: each wavefront a contiguous stretch of buckets, 64 at a time
  const int64_t per = ((S.nbk + SORT_BLOCK - 1) / SORT_BLOCK) * 64;
  const int64_t b0 = min(S.nbk, wave * per), b1 = min(S.nbk, b0 + per);
  uint32_t sum = 0, most = 0;
  uint64_t sq = 0;
  for (int64_t b = b0; b < b1; b += 64) {
    const uint32_t v = b + lane < b1 ? (uint32_t)hist[b + lane] : 0u;
    sum += lane_value(wave_scan_add(v), 63);
    most = max(most, v);
    sq += (uint64_t)v * v;
  }
  if (lane == 0) s_ws[wave] = sum;
  if (blockIdx.x == 1 && sq) atomicAdd(&s_sq, (unsigned long long)sq);
  if (blockIdx.x == 1) {
    most = lane_value(wave_scan_max(most), 63);
    if (lane == 0) atomicMax(&s_most, most);
  }
  __syncthreads();
  uint32_t run = 0;
  for (int w = 0; w < wave; ++w) run += s_ws[w];
  for (int64_t b = b0; b < b1; b += 64) {
    const uint32_t v = b + lane < b1 ? (uint32_t)hist[b + lane] : 0u;
    const uint32_t incl = wave_scan_add(v);
    if (b + lane < b1) {
      hist[b + lane] = (int32_t)(run + incl - v);
      S.start[b + lane] = (int32_t)(run + incl - v);
    }
    run += lane_value(incl, 63);
  }
  if (tid == 0) S.start[S.nbk] = (int32_t)S.n;
  err = block_or<SORT_BLOCK>(err);
  __shared__ unsigned long long s_min, s_max;
  if (tid == 0) {
    s_min = ~0ull;
    s_max = 0;
  }
  __syncthreads();
  atomicMin(&s_min, (unsigned long long)cmin);
  atomicMax(&s_max, (unsigned long long)cmax);
  __syncthreads();
  bool crowd = blockIdx.x == 1 && s_sq > (uint64_t)CROWDED * (uint64_t)max(S.n, S.n * S.n / S.nbk);
  // Rows that crowd make crowds of products of columns that do not: when one
  // bucket of columns could give an interval several times its products, a
  // sorted sample of the products tells whether any interval has them.
  const bool look = blockIdx.x == 1 && (crowd || (uint64_t)s_most * (uint64_t)R.set[0].n > R.peak);
  if (look) {   // the same for every thread
    int64_t* key = reinterpret_cast<int64_t*>(hist);   // (start[] has the buckets)
    const DirectSet& A = R.set[0];
    __syncthreads();
    for (int o = tid; o < R.ncrowd; o += SORT_BLOCK)
      key[o] = set_code(A, sample_of(o, 0, A.n), &err) +
               set_code(S, sample_of(o, DIRECT_CROWD_CELLS, S.n), &err);
    __syncthreads();
    block_sort<SORT_BLOCK>(key, R.ncrowd);
    const double pairs = (double)R.set[0].n * (double)S.n;
    const bool near = samples_crowd<SORT_BLOCK>(key, R.ncrowd, R.cw, (double)R.target, pairs);
    crowd = crowd || near;
    if (crowd)
      for (int o = tid; o <= R.ncrowd; o += SORT_BLOCK)
        R.bounds[o] = sample_bound(key, R.ncrowd, o, R.ncodes);
  }
  if (tid == 0) {
    R.meta->set_err[blockIdx.x] = err;
    R.meta->set_min[blockIdx.x] = s_min;
    R.meta->set_max[blockIdx.x] = s_max;
    if (blockIdx.x == 1) R.meta->crowd = !crowd ? 0u : s_most > DIRECT_COUNTED ? 2u : 1u;
  }
  if (S.n > DIRECT_PLACE) return;
  const int32_t* start = look ? S.start : hist;
  for (int64_t i = tid; i < S.n; i += SORT_BLOCK) {
    const int64_t code = set_code(S, i, &err);
    const int64_t at = start[code >> S.shift] + S.rank[i];
    if (crowd) {
      R.tmp_k[at] = code;
      R.tmp_i[at] = (int32_t)i;
    } else {
      place_term(R, S, i, code, at);
    }
  }
  if (!crowd) return;
  __syncthreads();
  if (s_most <= DIRECT_COUNTED) {
    for (int64_t t = tid; t < S.n; t += SORT_BLOCK) {
      const int64_t b = R.tmp_k[t] >> S.shift;
      place_sorted(R, S, t, S.start[b], S.start[b + 1]);
    }
    return;
  }
  const int32_t* term = sort_chunk(R, 0, (int)S.n, hist);
  const int64_t* key = reinterpret_cast<const int64_t*>(hist);
  for (int t = tid; t < S.n; t += SORT_BLOCK) place_term(R, S, term[t], key[t], t);
}

__global__ void __launch_bounds__(SMALL_BLOCK) k_rd_place(DirectArgs R) {
  const DirectSet& S = R.set[blockIdx.y];
  const int64_t i = (int64_t)blockIdx.x * SMALL_BLOCK + threadIdx.x;
  if (i >= S.n || S.n <= DIRECT_PLACE) return;
  uint32_t err = 0;   // (reported by the sort)
  const int64_t code = set_code(S, i, &err);
  const int64_t at = S.start[code >> S.shift] + S.rank[i];
  if (blockIdx.y == 1 && R.meta->crowd) {
    R.tmp_k[at] = code;
    R.tmp_i[at] = (int32_t)i;
  } else {
    place_term(R, S, i, code, at);
  }
}

// Crowded columns of more than DIRECT_PLACE terms (else nothing to do), when a
// bucket is too full to count each term's place: chunks sorted in LDS, then
// each term's place among the terms of its bucket, found in the sorted chunks
// that hold some of them.  2 x 2^18 terms, the columns of eight codes, take 1.1
// ms; counting them took 19 (8.4 through the groups).
__global__ void __launch_bounds__(SORT_BLOCK) k_rd_chunk(DirectArgs R) {
  extern __shared__ __align__(8) int32_t hist[];
  const DirectSet& S = R.set[1];
  const int64_t first = (int64_t)blockIdx.x * DIRECT_PLACE;
  if (R.meta->crowd != 2 || S.n <= DIRECT_PLACE || first >= S.n) return;
  const int n = (int)min(DIRECT_PLACE, S.n - first);
  const int32_t* term = sort_chunk(R, first, n, hist);
  const int64_t* key = reinterpret_cast<const int64_t*>(hist);
  for (int t = threadIdx.x; t < n; t += SORT_BLOCK) {
    R.tmp_k[first + t] = key[t];
    R.tmp_i[first + t] = term[t];
  }
}
__global__ void __launch_bounds__(SMALL_BLOCK) k_rd_order(DirectArgs R) {
  const DirectSet& S = R.set[1];
  const int64_t t = (int64_t)blockIdx.x * SMALL_BLOCK + threadIdx.x;
  if (!R.meta->crowd || t >= S.n || S.n <= DIRECT_PLACE) return;
  const int64_t k = R.tmp_k[t], b = k >> S.shift, own = t / DIRECT_PLACE;
  const int64_t b0 = S.start[b], b1 = S.start[b + 1];
  if (R.meta->crowd == 1) {
    place_sorted(R, S, t, (int32_t)b0, (int32_t)b1);
    return;
  }
  int64_t at = b0;
  for (int64_t c = b0 / DIRECT_PLACE; c * DIRECT_PLACE < b1; ++c) {
    const int64_t lo = max(b0, c * DIRECT_PLACE), hi = min(b1, (c + 1) * DIRECT_PLACE);
    // (equal codes: those of earlier chunks first)
    at += c == own ? t - lo
                   : (int64_t)first_from(R.tmp_k, (uint32_t)lo, (uint32_t)hi, c < own ? k + 1 : k) - lo;
  }
  place_term(R, S, R.tmp_i[t], k, at);
}

// The columns of codes xlo .. xhi: exactly when they are crowded, else their
// whole buckets (start[0] = 0 and start[nbk] = n close the ends).
__device__ __forceinline__ uint32_t column_from(const DirectSet& B, uint32_t j0, uint32_t j1,
                                                int64_t base, int64_t x) {
  if (B.k64) return first_from(B.k64, j0, j1, x);
  const uint32_t off = (uint32_t)(x - base);   // at most a bucket's 2^30 codes past base
  while (j0 < j1) {
    const uint32_t m = (j0 + j1) >> 1;
    if (B.k32[m] - (uint32_t)base < off) j0 = m + 1;
    else j1 = m;
  }
  return j0;
}
__device__ __forceinline__ void columns_of(const DirectSet& B, bool crowd, int64_t xlo,
                                           int64_t xhi, uint32_t* j0, uint32_t* j1) {
  const int64_t lo = max((int64_t)0, min(xlo, B.maxc)), hi = max((int64_t)0, min(xhi, B.maxc));
  const int64_t q0 = lo >> B.shift, q1 = hi >> B.shift;
  *j0 = (uint32_t)B.start[q0];
  *j1 = (uint32_t)B.start[q1 + 1];
  if (crowd) {
    *j0 = column_from(B, *j0, (uint32_t)B.start[q0 + 1], q0 << B.shift, lo);
    *j1 = column_from(B, (uint32_t)B.start[q1], *j1, q1 << B.shift, hi + 1);
  }
}

// ------------------------------------------------------------ counting
// Bound on the products of each cell (whole buckets of the columns), for
// COUNT_CELLS cells and a slice of the rows per workgroup: a row's buckets
// are looked up once per cell boundary.
__global__ void __launch_bounds__(SMALL_BLOCK) k_rd_count(DirectArgs R) {
  __shared__ unsigned long long s_sum[COUNT_CELLS];
  const int tid = threadIdx.x;
  const DirectSet& A = R.set[0];
  const DirectSet& B = R.set[1];
  const int64_t per = (A.n + gridDim.y - 1) / gridDim.y;
  const int64_t i0 = per * blockIdx.y, i1 = min(A.n, i0 + per);
  const bool crowd = R.meta->crowd != 0;
  const int64_t cells = crowd ? R.ncrowd : R.ncell;
  for (int64_t c0 = (int64_t)blockIdx.x * COUNT_CELLS; c0 < cells;
       c0 += (int64_t)gridDim.x * COUNT_CELLS) {
    if (tid < COUNT_CELLS) s_sum[tid] = 0;
    __syncthreads();
    uint32_t cnt[COUNT_CELLS];
#pragma unroll
    for (int q = 0; q < COUNT_CELLS; ++q) cnt[q] = 0;
    if (crowd) {
      for (int64_t i = i0 + tid; i < i1; i += SMALL_BLOCK) {
        const int64_t a = A.k64[i];
#pragma unroll
        for (int q = 0; q < COUNT_CELLS; ++q) {
          const int64_t lo = R.bounds[c0 + q] - a, hi = R.bounds[c0 + q + 1] - 1 - a;
          if (hi < lo || hi < 0 || lo > B.maxc) continue;
          uint32_t j0, j1;
          columns_of(B, true, lo, hi, &j0, &j1);
          cnt[q] += j1 - j0;
        }
      }
    } else {
      for (int64_t i = i0 + tid; i < i1; i += SMALL_BLOCK) {
        const int64_t x0 = (c0 << R.cw) - A.k64[i];   // lowest column code of the first cell
#pragma unroll
        for (int q = 0; q < COUNT_CELLS; ++q) {
          const int64_t lo = x0 + ((int64_t)q << R.cw), hi = lo + ((int64_t)1 << R.cw) - 1;
          if (hi < 0 || lo > B.maxc) continue;
          const int64_t j0 = lo <= 0 ? 0 : B.start[lo >> B.shift];
          const int64_t j1 = hi >= B.maxc ? B.n : B.start[(hi >> B.shift) + 1];
          cnt[q] += (uint32_t)(j1 - j0);
        }
      }
    }
#pragma unroll
    for (int q = 0; q < COUNT_CELLS; ++q) {
      const uint32_t w = lane_value(wave_scan_add(cnt[q]), 63);
      if ((tid & 63) == 0 && w) atomicAdd(&s_sum[q], (unsigned long long)w);
    }
    __syncthreads();
    if (tid < COUNT_CELLS && c0 + tid < cells && s_sum[tid])
      atomicAdd(reinterpret_cast<unsigned long long*>(&R.ccount[c0 + tid]), s_sum[tid]);
    __syncthreads();   // the next cells clear s_sum
  }
}

// Every workgroup scans the cells' interval counts and writes the intervals
// of its share of the cells: {first code, codes}.
__global__ void __launch_bounds__(PLAN_BLOCK) k_rd_plan(DirectArgs R) {
  __shared__ int64_t s_ws[PLAN_BLOCK / 64 + 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bool crowd = R.meta->crowd != 0;
  const int64_t cells = crowd ? R.ncrowd : R.ncell;
  const int64_t per = (cells + PLAN_BLOCK - 1) / PLAN_BLOCK;
  const int64_t c0 = min(cells, tid * per), c1 = min(cells, c0 + per);
  const auto block_total = [&](int64_t v) -> int64_t {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    __syncthreads();
    if (lane == 0) s_ws[wave] = v;
    __syncthreads();
    int64_t t = 0;
    for (int w = 0; w < PLAN_BLOCK / 64; ++w) t += s_ws[w];
    return t;
  };
  int64_t local = 0;
  for (int64_t c = c0; c < c1; ++c) local += R.ccount[c];
  const int64_t all = block_total(local);
  // sum of ceil(count / t) <= cells + all / t, kept within the array; sampled
  // cells are also cut at 2^31 codes when offsets are 32-bit, at most once per
  // cell of equal width
  const int64_t room = max((int64_t)1, crowd ? R.max_units - cells - R.ncell : R.grid - cells);
  const int64_t t = max(R.target, (all + room - 1) / room);
  const auto cell_of = [&](int64_t c, int64_t* lo, int64_t* hi) {
    if (crowd) {
      *lo = R.bounds[c];
      *hi = R.bounds[c + 1];
    } else {
      *lo = c << R.cw;
      *hi = min(R.ncodes, *lo + ((int64_t)1 << R.cw));
    }
  };
  // Intervals of this thread's cells: each(lo, end, k) takes the codes [lo, end),
  // cut into k.  A cell is cut by its own products; sampled cells, which are
  // uneven, are taken together while they fill one interval.
  const int64_t most = R.wide_codes ? INT64_MAX : (int64_t)1 << 31;
  const auto each_run = [&](auto&& each) {
    each_interval(c0, c1, crowd, t, most, cell_of, [&](int64_t c) { return R.ccount[c]; },
                  [&](int64_t n, int64_t width) {
                    const int64_t k = (n + t - 1) / t;
                    return crowd && !R.wide_codes ? max(k, (width - 1) / most + 1) : k;
                  },
                  each);
  };
  int64_t mine = 0;
  each_run([&](int64_t, int64_t, int64_t k) { mine += k; });
  int64_t incl = mine;
  for (int off = 1; off < 64; off <<= 1) {
    const int64_t y = __shfl_up(incl, off);
    if (lane >= off) incl += y;
  }
  __syncthreads();
  if (lane == 63) s_ws[wave] = incl;
  __syncthreads();
  int64_t run = incl - mine, total = 0;
  for (int w = 0; w < PLAN_BLOCK / 64; ++w) {
    if (w < wave) run += s_ws[w];
    total += s_ws[w];
  }
  // this workgroup writes the intervals of every gridDim.x-th thread
  if (tid % gridDim.x == blockIdx.x)
    each_run([&](int64_t lo, int64_t end, int64_t k) {
      const int64_t step = (end - lo + k - 1) / k;
      for (int64_t u = 0; u < k; ++u) {
        const int64_t a = min(end, lo + u * step), z = min(end, a + step);
        R.units[run + u] = make_longlong2(a, z - a);
      }
      run += k;
    });
  if (blockIdx.x == 0 && tid == 0) {
    R.meta->err = R.meta->set_err[0] | R.meta->set_err[1];
    R.meta->out_count = 0;
    // can a product of two terms be zero (a zero term, a product that wraps
    // to zero or falls below the least normal number)
    const uint64_t n0 = R.meta->set_min[0], n1 = R.meta->set_min[1];
    const uint64_t x0 = R.meta->set_max[0], x1 = R.meta->set_max[1];
    bool z = n0 == 0 || n1 == 0;
    if (R.f64)
      z = z || !(__longlong_as_double((long long)n0) * __longlong_as_double((long long)n1) > 2.3e-308);
    else if (!R.wide)
      z = z || __umul64hi(x0, x1) != 0 || x0 * x1 >= 0x8000000000000000ull;
    R.meta->zeros = z ? 1u : 0u;
    R.meta->nbins = total;
  }
}

// ------------------------------------------------------------ multiply
template <typename T>
struct Prod;
template <>
struct Prod<int64_t> {
  static __device__ __forceinline__ int64_t mul(uint64_t a, uint64_t b) {
    return (int64_t)(a * b);   // wraps modulo 2^64
  }
};
template <>
struct Prod<double> {
  static __device__ __forceinline__ double mul(uint64_t a, uint64_t b) {
    return __longlong_as_double((long long)a) * __longlong_as_double((long long)b);
  }
};
template <>
struct Prod<I128> {
  static __device__ __forceinline__ I128 mul(uint64_t a, uint64_t b) {
    return I128(a * b, __mul64hi((long long)a, (long long)b));
  }
};

// Claims an empty slot for the key, or returns the key that is there.
__device__ __forceinline__ uint32_t claim(uint32_t* slot, uint32_t key) {
  return atomicCAS(slot, ~0u, key);
}
__device__ __forceinline__ uint64_t claim(uint64_t* slot, uint64_t key) {
  return atomicCAS(reinterpret_cast<unsigned long long*>(slot), ~0ull, (unsigned long long)key);
}

template <int SLOTS>
__device__ __forceinline__ void table_add(uint64_t* vals, uint32_t s, int64_t v) {
  atomicAdd(reinterpret_cast<unsigned long long*>(&vals[s]), (unsigned long long)v);
}
template <int SLOTS>
__device__ __forceinline__ void table_add(uint64_t* vals, uint32_t s, double v) {
  atomicAdd(reinterpret_cast<double*>(&vals[s]), v);
}
// 128-bit: the low word's returning add gives its carry, which the high word
// receives with the product's high word
template <int SLOTS>
__device__ __forceinline__ void table_add(uint64_t* vals, uint32_t s, I128 v) {
  const uint64_t old =
      atomicAdd(reinterpret_cast<unsigned long long*>(&vals[s]), (unsigned long long)v.lo);
  const uint64_t carry = old + v.lo < old ? 1u : 0u;
  atomicAdd(reinterpret_cast<unsigned long long*>(&vals[SLOTS + s]),
            (unsigned long long)((uint64_t)v.hi + carry));
}

// What a workgroup's terms share when their codes become digits: the code of
// the interval's start as hi * D + lo, D the product of the low digits.
struct UnitDigits {
  uint64_t start;
  uint32_t lo;
  uint64_t hi;
};

// Digits of the code `start of the interval + off`: put(k, e) for digit k.
template <typename F>
__device__ __forceinline__ void each_digit(const DirectArgs& R, const UnitDigits& U, uint64_t off,
                                           F&& put) {
  uint64_t c = U.start + off;
  for (int k = 0; k < R.ndig; ++k) {
    const uint64_t q = fdiv(c, R.dec.dx[k]);
    put(k, (int32_t)(c - q * R.dec.dx[k].d));
    c = q;
  }
}
template <typename F>
__device__ __forceinline__ void each_digit(const DirectArgs& R, const UnitDigits& U, uint32_t off,
                                           F&& put) {
  uint32_t t = U.lo + off;             // below 2^32
  uint64_t h = U.hi;
  if (R.nlow < R.ndig) {               // t = c * D + low part
    const uint32_t c = fdiv32(t, R.div_low);
    t -= c * R.div_low.d;
    h += c;
  }
  for (int k = 0; k < R.nlow; ++k) {
    const uint32_t q = fdiv32(t, R.dec.dx32[k]);
    put(k, (int32_t)(t - q * R.dec.dx32[k].d));
    t = q;
  }
  for (int k = R.nlow; k < R.ndig; ++k) {
    int32_t e;
    if ((h >> 32) == 0 && R.dec.dx32[k].d != 0) {
      const uint32_t q = fdiv32((uint32_t)h, R.dec.dx32[k]);
      e = (int32_t)((uint32_t)h - q * R.dec.dx32[k].d);
      h = q;
    } else {
      const uint64_t q = fdiv(h, R.dec.dx[k]);
      e = (int32_t)(h - q * R.dec.dx[k].d);
      h = q;
    }
    put(k, e);
  }
}

// One workgroup per interval of output codes.  Nearly every product of a
// thinly spread multiplication is a term of its own, so a table that holds
// every product would spend its LDS on telling apart codes that never meet.
// Two passes over the interval's products need two bits per hash cell instead:
//   0. every product marks its cell, and a cell marked twice is marked shared;
//   1. a product alone in its cell is a term and is written out at once; the
//      others (about one in eleven at the planned load) are added in an
//      open-addressing table, whose nonzero sums are written last.
// An interval then holds five times the products that a table in the same LDS
// would, and a row's stretch of the columns is that much longer.
//   2. When the codes of products that share cells are more than the table
//      takes, they are added one stretch of codes at a time, halving a stretch
//      that still overflows.
// An interval of far more products than planned (codes that crowd in a small
// part of a cell) is cut into pieces before anything is written.
//
// What bounds it: VALU issue and the latency of the chain row -> columns ->
// cell -> result slot, not bytes (the vector units are busy 60 % of the time,
// the LDS 24 %, wavefronts wait 56 % of theirs).  Of 1.66 ms on 7,919 x 12,347
// terms (9.8e7 products, 2.7 GB of result) the two walks alone take 0.94 ms,
// adding the shared products 0.20, writing the others 0.54.  One workgroup of 1024
// threads per compute unit with 2^18 cells beats two of 512 with 2^17 (1.77
// ms) and three of 512 with 2^16 (2.78 ms): a row is looked at once per
// interval whatever it finds there.  A table that holds every product, with
// 5,000 products to an interval, took 2.25 ms.
// K: offsets in an interval, 32 bits, or 64 for products so few that an
// interval of 2^31 codes would hold next to none.
// FEW: few of the rows meet an interval, where the columns span little of the
// code space.  Batches of 64 rows then leave most wavefronts idle: 12,000 x 12,000
// terms whose columns span a 1,000th of the rows' 14.1 ms instead of 2.1.  (In
// every kernel the smaller batches cost 4 %: scalar registers are short.)
template <typename T, typename K, int NT, int MLOG, int SLOTS, bool FEW>
__global__ void __launch_bounds__(NT, NT == 256 ? 3 : 4) k_rd_mul(DirectArgs R) {
  constexpr int NW = NT / 64, PER = SLOTS / NT, W = sizeof(T) / 8, WORDS = 1 << (MLOG - 5);
  constexpr bool WIDE = sizeof(K) == 8;
  constexpr K NONE = ~K(0);
  // products of an interval that is cut; fewer when its codes crowd, since
  // those that share cells must then fit the table
  constexpr uint32_t CROWD = (1u << MLOG) / 4, CROWD_FEW = (1u << MLOG) / 9;
  constexpr K UNCUT = (K)1 << DIRECT_DONE_LOG;   // codes of an interval that is never cut
  static_assert(SLOTS % NT == 0, "each wavefront owns a stretch of the table");
  static_assert(WORDS % NT == 0, "each thread owns words of the marks");
  __shared__ uint32_t marked[WORDS], shared[WORDS];
  __shared__ K keys[SLOTS];
  __shared__ uint64_t vals[SLOTS * W];
  __shared__ uint16_t seg[NW][STEPS * 64];
  __shared__ uint4 rowd[NW][ROWS * 64];   // first column - first candidate, code, coefficient
  __shared__ uint32_t rowh[WIDE ? NW : 1][WIDE ? ROWS * 64 : 1];   // high words of the codes
  __shared__ uint4 stage[NW][64];         // the digits of a wavefront's terms on their way out
  __shared__ int32_t s_min[2 * KP_MAX_VARS];
  __shared__ uint32_t s_cnt[NW];
  __shared__ int64_t s_base;
  __shared__ uint32_t s_cursor, s_products, s_over;
  __shared__ uint32_t s_next;             // rows handed out
  __shared__ int64_t s_lo[DIRECT_STACK];  // intervals still to do
  __shared__ K s_width[DIRECT_STACK];
  __shared__ K s_sample[CUT_SAMPLES];     // offsets of products, when the columns are crowded
  __shared__ int s_pieces;                // of a cut
  __shared__ K p_lo[PARTS], p_hi[PARTS];   // stretches of the shared products
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t units = uniform(R.meta->nbins);
  if ((int64_t)blockIdx.x >= units) return;
  const bool crowd = uniform(R.meta->crowd) != 0;
  const uint32_t most = crowd ? CROWD_FEW : CROWD;
  int64_t lo = 0;
  K width = 0;   // codes of the interval
  const bool stats = R.stats != nullptr;
  const bool zeros = uniform(R.meta->zeros) != 0;   // a product of two terms may be zero
  T* out_c = static_cast<T*>(R.out_c);
  const int nx = R.dec.nx;
  int64_t ins = 0, extra = 0;
  UnitDigits U{0, 0, 0};
  // Word 64 r + lane of a wavefront's staged exponents: where it lies in the
  // stage, and its least value
  constexpr int NX = 6;
  uint32_t word_at[NX];
  int32_t word_min[NX];
  if (R.field != 0 && nx > 0)
#pragma unroll
    for (int r = 0; r < NX; ++r) {
      const uint32_t t = (64 * r + lane) / nx, d = (64 * r + lane) - t * nx;
      word_at[r] = min(t, 63u) * 16 + d * R.field;
      word_min[r] = (int32_t)R.dec.xmin[d];
    }
  if (tid < R.ndig) s_min[tid] = (int32_t)R.dec.xmin[tid];

  // Writes one term per lane with `on`: the wavefront's terms go to the
  // result slots q, q + 1, ... in lane order.  Their digits (px, or from the
  // key when `decode`) are staged in LDS, so that consecutive lanes write
  // consecutive words: rows of words written by their own lanes take four
  // times the requests.
  const auto write = [&](int64_t q, bool on, K key, T v, const uint4& px, bool decode) {
    const uint64_t mask = __ballot(on);
    const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                  __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
    const uint32_t n = (uint32_t)max((int64_t)0, min((int64_t)__popcll(mask), R.out_cap - q));
    on = on && at < n;
    if (on) (out_c + q)[at] = v;
    if (R.field == 0) {
      if (R.ndig == 0) {   // codes
        if (on) (R.out_k + q)[at] = lo + (int64_t)key;
      } else if (on) {
        int32_t* x = R.out_x + (q + at) * nx;
        each_digit(R, U, key, [&](int k, int32_t e) { x[k] = e + (int32_t)R.dec.xmin[k]; });
      }
      return;
    }
    uint8_t* st = reinterpret_cast<uint8_t*>(stage[wave]);
    wave_sync();
    if (on) {
      if (!decode)
        stage[wave][at] = px;
      else
        each_digit(R, U, key, [&](int k, int32_t e) {
          if (R.field == 1) st[at * 16 + k] = (uint8_t)e;
          else *reinterpret_cast<uint16_t*>(st + at * 16 + 2 * k) = (uint16_t)e;
        });
    }
    wave_sync();
    int32_t* x = R.out_x + q * nx;
    const uint32_t words = n * nx;
    if (nx > NX) {
      for (uint32_t i = lane; i < words; i += 64) {
        const uint32_t t = i / nx, d = i - t * nx;
        const uint32_t e = R.field == 1 ? (uint32_t)st[t * 16 + d]
                                        : (uint32_t)*reinterpret_cast<uint16_t*>(st + t * 16 + 2 * d);
        x[i] = (int32_t)e + s_min[d];
      }
    } else {
      uint32_t e[NX];
#pragma unroll
      for (int r = 0; r < NX; ++r)
        e[r] = R.field == 1 ? (uint32_t)st[word_at[r]]
                            : (uint32_t)*reinterpret_cast<uint16_t*>(st + word_at[r]);
#pragma unroll
      for (int r = 0; r < NX; ++r)
        if (64 * r + lane < words) x[64 * r + lane] = (int32_t)e[r] + word_min[r];
    }
  };
  // adds v at key; a full table (or a probe sequence too long) sets s_over
  const auto insert = [&](K key, uint32_t h, T v) {
    uint32_t s = __umulhi(h << MLOG, (uint32_t)SLOTS);   // the hash's bits below the cell's
    K c = claim(&keys[s], key);
    int q = 0;
    const uint32_t step = 1 + 6 * (h & 63);   // odd and no multiple of 3: every slot once
#pragma nounroll
    while (c != NONE && c != key && q < MAX_PROBE) {
      ++q;
      s += step;
      s = s >= (uint32_t)SLOTS ? s - SLOTS : s;
      c = claim(&keys[s], key);
    }
    if (c != NONE && c != key) {
      s_over = 1;
      return;
    }
    table_add<SLOTS>(vals, s, v);
    if (stats) extra += q;
  };
  // The products whose offsets in the interval lie in [w0, w1), 64 per
  // wavefront and step.  PASS 0 marks, PASS 1 writes the terms alone in their
  // cells and (when `add`) adds the others, PASS 2 adds the others.
  const auto walk_as = [&](auto pass, auto crowded, K w0, K w1, bool add) {
    constexpr int PASS = decltype(pass)::value;
    constexpr bool CROWDS = decltype(crowded)::value;
    constexpr uint32_t MOST = CROWDS ? CROWD_FEW : CROWD;
    const int64_t out0 = uniform(s_base);
    const DirectSet& A = R.set[0];
    const DirectSet& B = R.set[1];
    const K span = w1 - w0;
    const int64_t blo = lo + w0, bhi = lo + (w1 - 1);
    {
      // rows that meet the interval
      const int64_t amin = blo - B.maxc;
      if (span == 0 || amin > A.maxc) return;
      const uint32_t i0 = amin <= 0 ? 0u : uniform((uint32_t)A.start[amin >> A.shift]);
      const uint32_t i1 = bhi >= A.maxc ? (uint32_t)A.n
                                        : uniform((uint32_t)A.start[(bhi >> A.shift) + 1]);
      // ROWS * 64 rows at a time (lane l holds rows l, 64 + l, ...), all their
      // loads in flight together; a wavefront takes the next batch when it is
      // done with its last, rows being unequal.  FEW: a batch is fewer rows when
      // few meet the interval, and one of up to 32 parts of their columns, so
      // that every wavefront has some.
      uint32_t batch = ROWS * 64, plog = 0;
      if constexpr (FEW) {
        batch = min(batch, (i1 - i0 + 2 * NW - 1) / (2 * NW));
        while (plog < 5 && (i1 - i0) << plog < 2 * NW * batch) ++plog;
      }
      for (;;) {
        uint32_t bt = 0;
        if (lane == 0) bt = atomicAdd(&s_next, FEW ? 1u : batch);
        bt = lane_value(bt, 0);
        const uint32_t ib = i0 + (FEW ? (bt >> plog) * batch : bt);
        if (ib >= i1) break;
        const uint32_t ie = FEW ? min(i1, ib + batch) : i1;
        if (PASS == 0 && *(volatile uint32_t*)&s_products > MOST && width > UNCUT) return;
        if (PASS == 2 && *(volatile uint32_t*)&s_over) return;
        int64_t a[ROWS];
        uint32_t cnt[ROWS], excl[ROWS];
#pragma unroll
        for (int u = 0; u < ROWS; ++u) a[u] = A.k64[min(ib + u * 64 + lane, ie - 1)];
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
          const int64_t xlo = blo - a[u], xhi = bhi - a[u];
          const bool in = ib + u * 64 + lane < ie && xhi >= 0 && xlo <= B.maxc;
          columns_of(B, CROWDS, xlo, xhi, &excl[u], &cnt[u]);
          cnt[u] = in ? cnt[u] - excl[u] : 0;
          if (FEW && plog) {   // (at most 2^18 columns)
            const uint32_t p = bt & ((1u << plog) - 1), n = cnt[u];
            excl[u] += (n * p) >> plog;
            cnt[u] = ((n * (p + 1)) >> plog) - ((n * p) >> plog);
          }
        }
        uint32_t total = 0;
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
          const uint32_t incl = wave_scan_add(cnt[u]);
          const uint32_t first_cand = total + incl - cnt[u];
          const uint32_t i = min(ib + u * 64 + lane, ie - 1);
          const uint64_t ca = PASS != 0 || zeros ? A.c[i] : 0;
          rowd[wave][u * 64 + lane] = make_uint4(excl[u] - first_cand, (uint32_t)(a[u] - lo),
                                                 (uint32_t)ca, (uint32_t)(ca >> 32));
          if (WIDE) rowh[wave][u * 64 + lane] = (uint32_t)((uint64_t)(a[u] - lo) >> 32);
          excl[u] = first_cand;
          total += lane_value(incl, 63);
        }
        uint32_t carry = 0, products = 0;
        // candidates STEPS * 64 at a time: candidate k belongs to the last
        // row whose first candidate is at or before it
        for (uint32_t k0 = 0; k0 < total; k0 += STEPS * 64) {
          // (a full table's chains are long: what is left is not looked at)
          if (PASS == 2 && uniform(*(volatile uint32_t*)&s_over)) return;
#pragma unroll
          for (int v = 0; v < STEPS; ++v) seg[wave][v * 64 + lane] = 0;
          wave_sync();
#pragma unroll
          for (int u = 0; u < ROWS; ++u) {
            const uint32_t at = excl[u] - k0;
            if (cnt[u] && at < STEPS * 64u) seg[wave][at] = (uint16_t)(u * 64 + lane);
          }
          wave_sync();
          K off[STEPS];
          uint4 px[STEPS];
          uint64_t ca[STEPS], cb[STEPS];
#pragma unroll
          for (int v = 0; v < STEPS; ++v) {
            const uint32_t m = max(carry, wave_scan_max(seg[wave][v * 64 + lane]));
            carry = lane_value(m, 63);
            const uint32_t k = min(k0 + v * 64 + lane, total - 1);
            const uint4 rd = rowd[wave][m];
            const uint32_t j = rd.x + k;
            // (the offset's low 32 bits identify it: bucket widths and
            // intervals are small enough that no other multiple of 2^32 occurs)
            if constexpr (WIDE)
              off[v] = (((uint64_t)rowh[wave][m] << 32) | rd.y) + (uint64_t)B.k64[j];
            else
              off[v] = rd.y + B.k32[j];
            if (PASS != 0 || zeros) {
              ca[v] = ((uint64_t)rd.w << 32) | rd.z;
              cb[v] = B.c[j];
            }
            if (PASS == 1 && R.field != 0) {   // digits add without carries
              const uint4 pa = A.px[ib + m], pb = B.px[j];
              px[v] = make_uint4(pa.x + pb.x, pa.y + pb.y, pa.z + pb.z, pa.w + pb.w);
            }
          }
          wave_sync();
#pragma unroll
          for (int v = 0; v < STEPS; ++v) {
            if (k0 + v * 64 >= total) break;
            bool ok = k0 + v * 64 + lane < total && off[v] - w0 < span;
            const K key = off[v];
            T x{};
            if (PASS != 0 || zeros) {
              x = Prod<T>::mul(ca[v], cb[v]);
              if (zeros) ok = ok && x != T(0);
            }
            const uint32_t h = mix(key), cell = h >> (32 - MLOG);
            const uint32_t bit = 1u << (cell & 31);
            if (PASS == 0) {
              const uint64_t oks = __ballot(ok);
              products += (uint32_t)__popcll(oks);
              if (CROWDS && oks) {
                // a sample per step, from a lane that changes: a step that
                // begins with a row begins with the row's least code
                const uint32_t z = ((products + wave) * HASH_MUL) >> 26;
                const uint64_t turned = (oks >> z) | (oks << ((64 - z) & 63));
                if (lane == (((int)__builtin_ctzll(turned) + (int)z) & 63))
                  s_sample[(wave + NW * (products >> 6)) & (CUT_SAMPLES - 1)] = key;
              }
              // (crowds may share one cell: what is shared is not marked again)
              if (CROWDS && ok && (shared[cell >> 5] & bit) != 0) continue;
              if (ok && (atomicOr(&marked[cell >> 5], bit) & bit)) atomicOr(&shared[cell >> 5], bit);
              continue;
            }
            const bool both = (shared[cell >> 5] & bit) != 0;
            if (PASS == 1) {
              const bool alone = ok && !both;
              const uint32_t n = (uint32_t)__popcll(__ballot(alone));
              if (n) {
                uint32_t at = 0;
                if (lane == 0) at = atomicAdd(&s_cursor, n);
                write(out0 + lane_value(at, 0), alone, key, x, px[v], false);
              }
              if (stats) ins += ok ? 1 : 0;
            }
            if (ok && both && (PASS == 2 || add)) insert(key, h, x);
          }
        }
        if (PASS == 0 && lane == 0) atomicAdd(&s_products, products);
      }
    }
  };
  const auto walk = [&](auto pass, K w0, K w1, bool add) {
    if (crowd) walk_as(pass, std::true_type{}, w0, w1, add);
    else walk_as(pass, std::false_type{}, w0, w1, add);
  };
  const auto clear_table = [&]() {
#pragma unroll
    for (int r = 0; r < PER; ++r) keys[r * NT + tid] = NONE;
#pragma unroll
    for (int r = 0; r < PER * W; ++r) vals[r * NT + tid] = 0;
    if (tid == 0) s_over = 0;
  };
  // sum over the workgroup of one value per thread, and the sum before this wavefront
  const auto total_of = [&](uint32_t v, uint32_t* before) -> uint32_t {
    const uint32_t w = lane_value(wave_scan_add(v), 63);
    if (lane == 0) s_cnt[wave] = w;
    __syncthreads();
    uint32_t tot = 0, b = 0;
#pragma unroll
    for (int k = 0; k < NW; ++k) {
      const uint32_t x = s_cnt[k];
      if (k < wave) b += x;
      tot += x;
    }
    *before = b;
    return tot;
  };
  const auto reserve = [&](uint32_t n) {   // n result slots from s_base on
    if (tid == 0)
      s_base = n ? (int64_t)atomicAdd(reinterpret_cast<unsigned long long*>(&R.meta->out_count),
                                      (unsigned long long)n)
                 : 0;
    __syncthreads();
  };
  // writes the table's nonzero sums
  const auto emit = [&]() {
    const int r0 = wave * PER * 64;   // this wavefront's stretch
    K kk[PER];
    uint64_t vv[PER * W];
    uint64_t ball[PER];
    uint32_t cnt = 0;
#pragma unroll
    for (int r = 0; r < PER; ++r) {
      const int i = r0 + r * 64 + lane;
      kk[r] = keys[i];
      vv[r] = vals[i];
      bool keep;
      if constexpr (W == 2) {
        vv[PER + r] = vals[SLOTS + i];
        keep = (vv[r] | vv[PER + r]) != 0;
      } else if constexpr (std::is_same<T, double>::value) {
        keep = (vv[r] << 1) != 0;   // both signed zeros are dropped
      } else {
        keep = vv[r] != 0;
      }
      ball[r] = __ballot(keep);
      cnt += (uint32_t)__popcll(ball[r]);
    }
    uint32_t before;
    const uint32_t tot = total_of(lane == 0 ? cnt : 0u, &before);
    // this wavefront's terms to the front of its stretch
    const uint64_t lt = (1ull << lane) - 1;
    uint32_t pos = 0;
#pragma unroll
    for (int r = 0; r < PER; ++r) {
      if (ball[r] & (1ull << lane)) {
        const int q = r0 + (int)pos + (int)__popcll(ball[r] & lt);
        keys[q] = kk[r];
        vals[q] = vv[r];
        if constexpr (W == 2) vals[SLOTS + q] = vv[PER + r];
      }
      pos += (uint32_t)__popcll(ball[r]);
    }
    reserve(tot);
    const int64_t q0 = uniform(s_base) + before;
    for (uint32_t t0 = 0; t0 < cnt; t0 += 64) {
      const uint32_t t = min(t0 + lane, cnt - 1);
      T v;
      if constexpr (W == 2) v = T(vals[r0 + t], (int64_t)vals[SLOTS + r0 + t]);
      else __builtin_memcpy(&v, &vals[r0 + t], 8);
      write(q0 + t0, t0 + lane < cnt, keys[r0 + t], v, uint4{}, true);
    }
  };

  // (the grid has an interval per workgroup unless the columns are crowded)
  for (int64_t unit = blockIdx.x; unit < units; unit += gridDim.x) {
  if (tid == 0) {
    s_lo[0] = R.units[unit].x;
    s_width[0] = (K)R.units[unit].y;
  }
  __syncthreads();
  for (int sp = 1; sp > 0;) {
    --sp;
    lo = uniform(s_lo[sp]);
    width = uniform(s_width[sp]);
    if (width == 0) {
      __syncthreads();   // the next interval's start is written
      continue;
    }
    if (R.ndig > 0) {
      const uint64_t c = (uint64_t)lo;
      U.start = c;
      U.hi = R.nlow < R.ndig ? fdiv(c, R.div_low64) : 0;
      U.lo = (uint32_t)(c - U.hi * (uint64_t)R.div_low.d);
    }
#pragma unroll
    for (int r = 0; r < WORDS / NT; ++r) {
      marked[r * NT + tid] = 0;
      shared[r * NT + tid] = 0;
    }
    clear_table();
    if (tid == 0) s_next = 0;
    if (tid == 0) s_cursor = s_products = 0;
    if (tid < CUT_SAMPLES) s_sample[tid] = NONE;
    __syncthreads();
    walk(std::integral_constant<int, 0>{}, 0, width, false);
    __syncthreads();
    const uint32_t products = uniform(s_products);
    if (products > most && width > UNCUT) {   // the same for every thread
      if (wave == 0) {
        const K key = s_sample[lane];
        int rank = 0;
#pragma unroll 8
        for (int o = 0; o < CUT_SAMPLES; ++o) {
          const K y = s_sample[o];
          rank += y < key || (y == key && o < lane) ? 1 : 0;
        }
        const int n = (int)__popcll(__ballot(key != NONE));   // (NONE is the greatest)
        wave_sync();
        s_sample[rank] = key;
        wave_sync();
        // (the same in every lane)
        const int m = cut_points<K, DIRECT_PARTS>([&](int i) { return uniform(s_sample[i]); }, n, width, sp,
                                    DIRECT_STACK, DIRECT_DONE_LOG, [&](int p, K x, K y) {
                                      s_lo[sp + p] = lo + (int64_t)x;
                                      s_width[sp + p] = y - x;
                                    });
        if (lane == 0) s_pieces = m;
      }
      __syncthreads();
      sp += (int)uniform((uint32_t)s_pieces);
      continue;
    }
    // products alone in their cells: cells marked but not shared
    uint32_t alone = 0;
#pragma unroll
    for (int r = 0; r < WORDS / NT; ++r)
      alone += __popc(marked[r * NT + tid] & ~shared[r * NT + tid]);
    uint32_t before;
    alone = uniform(total_of(alone, &before));
    reserve(alone);
    if (tid == 0) s_next = 0;
    __syncthreads();
    // The table takes the others if their codes fit.  Terms that repeat and
    // dense rows have several products a code (stretches sized by the products
    // would look at every row that many times more): c codes mark m of M cells
    // when c = -M log(1 - m / M), here to the second power of m / M < 1 / 4.
    const uint32_t others = products - alone;
    uint32_t codes = others;
    bool add = others <= (uint32_t)SLOTS * 7 / 8;
    if (!add) {
      uint32_t cells = 0;
      for (int r = 0; r < WORDS / NT; ++r) cells += __popc(marked[r * NT + tid]);
      cells = total_of(cells, &before);
      __syncthreads();
      cells = uniform(cells);
      const uint32_t twice = (uint32_t)(((uint64_t)cells * cells) >> (MLOG + 1));   // m^2 / 2 M
      const uint32_t more = (uint32_t)(((uint64_t)twice * cells) >> MLOG) * 2 / 3;   // m^3 / 3 M^2
      codes = min(others, cells - alone + twice + more + 1);
      add = codes <= (uint32_t)SLOTS * 3 / 4;
    }
    if (add || alone) walk(std::integral_constant<int, 1>{}, 0, width, add);
    else if (stats && tid == 0) ins += products;
    __syncthreads();
    if (add && !s_over) {
      if (others) emit();
      __syncthreads();
      continue;
    }
    const uint32_t parts = codes / (SLOTS * 5 / 8) + 1;
    const K step = (width + parts - 1) / parts;
    for (K w0 = 0; w0 < width; w0 += step) {
      __syncthreads();
      if (tid == 0) {
        p_lo[0] = w0;
        p_hi[0] = min(width, w0 + step);
      }
      __syncthreads();
      for (int pp = 1; pp > 0;) {
        --pp;
        const K a = uniform(p_lo[pp]), z = uniform(p_hi[pp]);
        clear_table();
        if (tid == 0) s_next = 0;
        __syncthreads();
        walk(std::integral_constant<int, 2>{}, a, z, true);
        __syncthreads();
        if (s_over) {
          if (tid == 0) {
            const K mid = a + (z - a) / 2;
            p_lo[pp] = mid;
            p_hi[pp] = z;
            p_lo[pp + 1] = a;
            p_hi[pp + 1] = mid;
          }
          pp += 2;
        } else {
          emit();
        }
        __syncthreads();
      }
    }
  }
  }
  if (stats) {
    for (int off = 32; off > 0; off >>= 1) {
      ins += __shfl_xor(ins, off);
      extra += __shfl_xor(extra, off);
    }
    if (lane == 0) {
      atomicAdd(&R.stats[0], (unsigned long long)ins);
      atomicAdd(&R.stats[1], (unsigned long long)extra);
    }
  }
}

template <typename T, typename K, int NT, int MLOG, int SLOTS>
void launch_mul(const DirectArgs& R, hipStream_t s) {
  // less than a batch a wavefront, and a few of the rows (60 to 250 rows that all
  // meet an interval take 5 to 9 us longer in parts: 93 against 101, 122 against 132)
  if (R.meet < NT && 4 * R.meet < R.set[0].n)
    hipLaunchKernelGGL((k_rd_mul<T, K, NT, MLOG, SLOTS, true>), dim3((unsigned)R.grid), dim3(NT), 0,
                       s, R);
  else
    hipLaunchKernelGGL((k_rd_mul<T, K, NT, MLOG, SLOTS, false>), dim3((unsigned)R.grid), dim3(NT),
                       0, s, R);
}

// Table slots of large and small intervals, and of large ones of 64-bit offsets.
template <typename T, int SLOTS, int SMALL, int WIDE>
void launch_mul_typed(const DirectArgs& R, hipStream_t s) {
  if (R.small) {
    if (R.wide_codes) launch_mul<T, uint64_t, 256, DIRECT_SMALL_CELLS_LOG, SMALL>(R, s);
    else launch_mul<T, uint32_t, 256, DIRECT_SMALL_CELLS_LOG, SMALL>(R, s);
  } else {
    if (R.wide_codes) launch_mul<T, uint64_t, 1024, DIRECT_CELLS_LOG, WIDE>(R, s);
    else launch_mul<T, uint32_t, 1024, DIRECT_CELLS_LOG, SLOTS>(R, s);
  }
}

}  // namespace

hipError_t direct_setup() {
  static bool done = false;
  if (done) return hipSuccess;
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_rd_sort),
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)(DENSE_MAX_BUCKETS * 4));
  if (e == hipSuccess) done = true;
  return e;
}

hipError_t launch_direct(const DirectArgs& R, kp_dtype dt, int64_t* out_n, uint32_t* ctx_err,
                         Mailbox* mb, uint64_t seq, hipStream_t s) {
  hipError_t e = direct_setup();
  if (e != hipSuccess) return e;
  if (R.ev0) (void)hipEventRecord(R.ev0, s);
  int64_t chunk = 1;   // terms of a sorted chunk's array
  while (chunk < std::min(R.set[1].n, DIRECT_PLACE)) chunk *= 2;
  const int64_t lds = std::max({R.set[0].nbk * 4, R.set[1].nbk * 4, (int64_t)R.ncrowd * 8, chunk * 12});
  const int64_t rows = R.set[0].n, n = std::max(rows, R.set[1].n);
  hipLaunchKernelGGL(k_rd_sort, dim3(2), dim3(SORT_BLOCK), (size_t)lds, s, R);
  if (n > DIRECT_PLACE) {
    const unsigned blocks = (unsigned)((n + SMALL_BLOCK - 1) / SMALL_BLOCK);
    hipLaunchKernelGGL(k_rd_place, dim3(blocks, 2), dim3(SMALL_BLOCK), 0, s, R);
    const unsigned chunks = (unsigned)((R.set[1].n + DIRECT_PLACE - 1) / DIRECT_PLACE);
    hipLaunchKernelGGL(k_rd_chunk, dim3(chunks), dim3(SORT_BLOCK), (size_t)(chunk * 12), s, R);
    hipLaunchKernelGGL(k_rd_order, dim3(blocks), dim3(SMALL_BLOCK), 0, s, R);
  }
  const int64_t groups = (R.ncell + COUNT_CELLS - 1) / COUNT_CELLS;
  // enough row slices for about 2048 counting workgroups, of at least 256 rows
  int64_t ys = (2048 + groups - 1) / groups;
  const int64_t most = (rows + SMALL_BLOCK - 1) / SMALL_BLOCK;
  ys = ys > most ? most : ys;
  ys = ys > 0 ? ys : 1;
  // crowded columns have more cells; the workgroups for them end at once otherwise
  const int64_t xs = std::max(groups, std::min<int64_t>(R.ncrowd / COUNT_CELLS, 2048 / ys));
  hipLaunchKernelGGL(k_rd_count, dim3((unsigned)xs, (unsigned)ys), dim3(SMALL_BLOCK), 0, s, R);
  const int64_t pg = R.grid / 2048 + 1;
  hipLaunchKernelGGL(k_rd_plan, dim3((unsigned)(pg > 64 ? 64 : pg)), dim3(PLAN_BLOCK), 0, s, R);
  if (dt == KP_F64) launch_mul_typed<double, 4096, 1024, 3072>(R, s);
  else if (dt == KP_I128) launch_mul_typed<I128, 2048, 512, 2048>(R, s);
  else launch_mul_typed<int64_t, 4096, 1024, 3072>(R, s);
  if (R.ev1) (void)hipEventRecord(R.ev1, s);
  return launch_finalize(R.meta, R.out_cap, out_n, ctx_err, s, mb, seq);
}

}  // namespace kp
