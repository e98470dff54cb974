// Index builder kernels (partial indexing, Section 3.2.2).
//
//  k_check_rowptr                     row offsets (Section 2.1), longest row
//  k_validate_count                   the other input checks; non-zero count and
//                                     maxweight_d(V) per dimension
//  k_dim_keys / k_rank_from_sorted    density order: decreasing count, ties by id
//  k_sort_rows / k_sort_long_rows     every row's components re-ordered densest first
//  k_row_keys / k_unpack_rows         the same by radix passes, for rows past kLongRow
//  k_cutoff                           running bound b = sum x[d] maxweight_d(V) in double;
//                                     the leading components with b < t are x' (or, for
//                                     the head-cut index of the screened join, the
//                                     components of rank < head)
//  k_emit_indexed / k_list_offsets    inverted lists of the indexed parts, by vector id
//  k_query_rows                       external query rows: checked, ranked, sorted
//  k_block_offsets                    where each dense list enters each corpus block
#include "apss_internal.h"
#include "index_build.h"

namespace apss {

namespace {

// Orders the LDS accesses of one wave around an exchange between its lanes.
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// v of lane l (l the same on every lane), in scalar registers.
__device__ __forceinline__ double lane_value(double v, int l) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), l);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

__global__ void k_check_rowptr(const int64_t* __restrict__ rp, int64_t n, int64_t nnz, uint32_t* __restrict__ err,
                               unsigned long long* __restrict__ bad_row, unsigned long long* __restrict__ longest) {
  unsigned long long len = 0;
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r <= n; r += (int64_t)gridDim.x * blockDim.x) {
    bool bad = false;
    if (r == 0 && rp[0] != 0) bad = true;
    if (r == n && rp[n] != nnz) bad = true;
    if (r < n && rp[r + 1] < rp[r]) bad = true;
    else if (r < n && (unsigned long long)(rp[r + 1] - rp[r]) > len) len = (unsigned long long)(rp[r + 1] - rp[r]);
    if (bad) {
      atomicOr(err, ERR_ROWPTR);
      atomicMin(bad_row, (unsigned long long)r);
    }
  }
  if (longest) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      const unsigned long long u = __shfl_xor(len, o, 64);
      len = u > len ? u : len;
    }
    if ((threadIdx.x & 63u) == 0 && len) atomicMax(longest, len);
  }
}

// Dimension range, positive finite weights, unit norm; non-zero count and
// maxweight_d(V) of every dimension.  One wave per row, lanes over its
// components (coalesced).  The bound is the two atomics per component: on
// the dense dimensions they meet at one address.  Each workgroup therefore
// keeps the dimensions it meets first in a direct-mapped LDS table (dense
// ones appear within its first rows) and adds a table entry to the global
// counters once, at its end; only dimensions without an entry go to global
// memory at every component.  500,000 rows of mean 120: 8.8 ms for a
// thread per row and plain atomics.
constexpr int kCountBits = 12;
constexpr int kCountSlots = 1 << kCountBits;

__global__ __launch_bounds__(1024) void k_validate_count(const int64_t* __restrict__ rp, const int32_t* __restrict__ col,
                                                         const float* __restrict__ val, int64_t n, int64_t m,
                                                         double norm_tol, uint32_t* cnt, uint32_t* mwbits,
                                                         uint32_t* __restrict__ err,
                                                         unsigned long long* __restrict__ bad_row) {
  __shared__ uint32_t tag[kCountSlots], tcnt[kCountSlots], tmax[kCountSlots];
  for (int i = (int)threadIdx.x; i < kCountSlots; i += (int)blockDim.x) {
    tag[i] = 0xFFFFFFFFu;  // free: dimension ids are below 2^31
    tcnt[i] = 0u;
    tmax[i] = 0u;
  }
  __syncthreads();
  const int lane = (int)(threadIdx.x & 63u);
  const int64_t wpb = (int64_t)(blockDim.x >> 6);
  for (int64_t r = (int64_t)blockIdx.x * wpb + (int64_t)(threadIdx.x >> 6); r < n; r += (int64_t)gridDim.x * wpb) {
    const int64_t a = rp[r], b = rp[r + 1];
    uint32_t e = 0;
    double ss = 0.0;
    for (int64_t k = a + lane; k < b; k += 64) {
      const int32_t d = col[k];
      const float w = val[k];
      if (!(w > 0.0f) || !isfinite(w)) e |= ERR_WEIGHT;
      ss += (double)w * (double)w;
      if (d < 0 || (int64_t)d >= m) {
        e |= ERR_DIM;
        continue;
      }
      // weights are positive floats, whose bit patterns order like the values
      const uint32_t wb = __float_as_uint(w);
      const uint32_t h = ((uint32_t)d * 0x9E3779B1u) >> (32 - kCountBits);
      uint32_t own = tag[h];
      if (own == 0xFFFFFFFFu) {
        own = atomicCAS(&tag[h], 0xFFFFFFFFu, (uint32_t)d);
        if (own == 0xFFFFFFFFu) own = (uint32_t)d;
      }
      if (own == (uint32_t)d) {
        atomicAdd(&tcnt[h], 1u);
        atomicMax(&tmax[h], wb);
      } else {
        atomicAdd(&cnt[d], 1u);
        // (a stale value read here is at most the current one)
        if (wb > mwbits[d]) atomicMax(&mwbits[d], wb);
      }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      ss += __shfl_xor(ss, o, 64);
      e |= __shfl_xor(e, o, 64);
    }
    if (lane == 0) {
      if (b > a && !(fabs(sqrt(ss) - 1.0) <= norm_tol)) e |= ERR_NORM;
      if (e) {
        atomicOr(err, e);
        atomicMin(bad_row, (unsigned long long)r);
      }
    }
  }
  __syncthreads();
  for (int i = (int)threadIdx.x; i < kCountSlots; i += (int)blockDim.x) {
    const uint32_t d = tag[i];
    if (d != 0xFFFFFFFFu) {
      atomicAdd(&cnt[d], tcnt[i]);
      if (tmax[i] > mwbits[d]) atomicMax(&mwbits[d], tmax[i]);
    }
  }
}

__global__ void k_dim_keys(const uint32_t* __restrict__ cnt, int64_t m, int64_t n, int dbits, uint64_t* __restrict__ keys,
                           uint64_t* __restrict__ vals) {
  for (int64_t d = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; d < m; d += (int64_t)gridDim.x * blockDim.x) {
    keys[d] = ((uint64_t)(n - (int64_t)cnt[d]) << dbits) | (uint64_t)d;
    vals[d] = (uint64_t)d;
  }
}

__global__ void k_rank_from_sorted(const uint64_t* __restrict__ vals, int64_t m, const uint32_t* __restrict__ cnt,
                                   const uint32_t* __restrict__ mwbits, int32_t* __restrict__ rank,
                                   float* __restrict__ mw_by_rank, uint32_t* __restrict__ cnt_by_rank) {
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < m; r += (int64_t)gridDim.x * blockDim.x) {
    const int32_t d = (int32_t)vals[r];
    rank[d] = (int32_t)r;
    mw_by_rank[r] = __uint_as_float(mwbits[d]);
    cnt_by_rank[r] = cnt[d];
  }
}

// One thread per row: keys (row, rank) for every component, values = weight bits.
__global__ void k_row_keys(const int64_t* __restrict__ rp, const int32_t* __restrict__ col, const float* __restrict__ val,
                           const int32_t* __restrict__ rank, int64_t n, int rbits, uint64_t* __restrict__ keys,
                           uint32_t* __restrict__ vals) {
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n; r += (int64_t)gridDim.x * blockDim.x) {
    for (int64_t k = rp[r]; k < rp[r + 1]; ++k) {
      keys[k] = ((uint64_t)r << rbits) | (uint64_t)rank[col[k]];
      vals[k] = __float_as_uint(val[k]);
    }
  }
}

__global__ void k_unpack_rows(const uint64_t* __restrict__ keys, const uint32_t* __restrict__ vals, int64_t nnz,
                              int rbits, RComp* __restrict__ rc, uint32_t* __restrict__ err) {
  const uint64_t rmask = (1ull << rbits) - 1;
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < nnz; k += (int64_t)gridDim.x * blockDim.x) {
    const uint64_t key = keys[k];
    RComp c;
    c.r = (int32_t)(key & rmask);
    c.w = __uint_as_float(vals[k]);
    rc[k] = c;
    if (k > 0 && keys[k - 1] == key) atomicOr(err, ERR_DUP);
  }
}

// Rows of at most kWaveRow components, one wave each: ranks gathered, (rank,
// weight) sorted by a bitonic network in the wave's own LDS, equal
// neighbours (a repeated dimension) reported.  Longer rows (up to kLongRow)
// go to a list for k_sort_long_rows.  The row is read and written once;
// 64-bit radix passes over (row, rank) keys moved it 12 times (500,000 rows
// of mean 120: 5.5 ms for the keys and 5.4 ms for the passes).
__device__ __forceinline__ void compare_exchange(uint64_t* __restrict__ ck, int i, int stride, int size) {
  const int lo = 2 * i - (i & (stride - 1));  // lower index of pair i
  const uint64_t x = ck[lo], y = ck[lo + stride];
  if ((x > y) == ((lo & size) == 0)) {
    ck[lo] = y;
    ck[lo + stride] = x;
  }
}

__global__ __launch_bounds__(256) void k_sort_rows(const int64_t* __restrict__ rp, const int32_t* __restrict__ col,
                                                   const float* __restrict__ val, const int32_t* __restrict__ rank,
                                                   int64_t n, RComp* __restrict__ rc, uint32_t* __restrict__ err,
                                                   unsigned int* __restrict__ nlong, uint32_t* __restrict__ longs) {
  __shared__ uint64_t buf[4][kWaveRow];
  const int lane = (int)(threadIdx.x & 63u);
  const int wave = (int)(threadIdx.x >> 6);
  uint64_t* ck = buf[wave];
  for (int64_t r = (int64_t)blockIdx.x * 4 + wave; r < n; r += (int64_t)gridDim.x * 4) {
    const int64_t a = rp[r];
    const int64_t len64 = rp[r + 1] - a;
    if (len64 > kWaveRow) {
      if (lane == 0) longs[atomicAdd(nlong, 1u)] = (uint32_t)r;
      continue;
    }
    const int len = (int)len64;
    int n2 = 1;
    while (n2 < len) n2 <<= 1;
    for (int i = lane; i < n2; i += 64) {
      uint64_t c = ~0ull;  // above every component
      if (i < len) c = ((uint64_t)(uint32_t)rank[col[a + i]] << 32) | (uint64_t)__float_as_uint(val[a + i]);
      ck[i] = c;
    }
    wave_lds_order();
    for (int size = 2; size <= n2; size <<= 1)
      for (int stride = size >> 1; stride > 0; stride >>= 1) {
        for (int i = lane; i < n2 / 2; i += 64) compare_exchange(ck, i, stride, size);
        wave_lds_order();
      }
    bool dup = false;
    for (int i = lane; i < len; i += 64) {
      const uint64_t c = ck[i];
      dup = dup || (i > 0 && (uint32_t)(ck[i - 1] >> 32) == (uint32_t)(c >> 32));
      rc[a + i] = RComp{(int32_t)(c >> 32), __uint_as_float((uint32_t)c)};
    }
    if (dup) atomicOr(err, ERR_DUP);
    wave_lds_order();
  }
}

// The listed longer rows, one workgroup each (64 KB of LDS).
__global__ __launch_bounds__(1024) void k_sort_long_rows(const int64_t* __restrict__ rp, const int32_t* __restrict__ col,
                                                         const float* __restrict__ val, const int32_t* __restrict__ rank,
                                                         RComp* __restrict__ rc, uint32_t* __restrict__ err,
                                                         const unsigned int* __restrict__ nlong,
                                                         const uint32_t* __restrict__ longs) {
  __shared__ uint64_t ck[kLongRow];
  const unsigned int nl = *nlong;
  const int tid = (int)threadIdx.x;
  for (unsigned int e = blockIdx.x; e < nl; e += gridDim.x) {
    const int64_t r = longs[e];
    const int64_t a = rp[r];
    const int len = (int)(rp[r + 1] - a);
    int n2 = 1;
    while (n2 < len) n2 <<= 1;
    for (int i = tid; i < n2; i += (int)blockDim.x) {
      uint64_t c = ~0ull;
      if (i < len) c = ((uint64_t)(uint32_t)rank[col[a + i]] << 32) | (uint64_t)__float_as_uint(val[a + i]);
      ck[i] = c;
    }
    __syncthreads();
    for (int size = 2; size <= n2; size <<= 1)
      for (int stride = size >> 1; stride > 0; stride >>= 1) {
        for (int i = tid; i < n2 / 2; i += (int)blockDim.x) compare_exchange(ck, i, stride, size);
        __syncthreads();
      }
    bool dup = false;
    for (int i = tid; i < len; i += (int)blockDim.x) {
      const uint64_t c = ck[i];
      dup = dup || (i > 0 && (uint32_t)(ck[i - 1] >> 32) == (uint32_t)(c >> 32));
      rc[a + i] = RComp{(int32_t)(c >> 32), __uint_as_float((uint32_t)c)};
    }
    if (dup) atomicOr(err, ERR_DUP);
    __syncthreads();
  }
}

// Partial indexing cutoff, one wave per row.  The running bound and norm are
// summed in double in the order of the components (densest dimension first;
// the products of two floats are exact in double), so the cut does not
// depend on the lanes: each lane prepares one component's terms and the wave
// adds them up one after another from its lanes.  A component is indexed as
// soon as the running bound including it reaches t; with l2 the unindexed
// part also ends once its own squared norm reaches t^2 (exact for float t).
// Rows are read coalesced (500,000 rows of mean 120: 1.3 ms for a thread per
// row).  Also: the largest unindexed-part norm over the rows (*pmax, as float
// bits: norms are >= 0, so their bit patterns order like the values), and
// each row's norm as a one-byte upper bound: the smallest k with
// pnrm <= k / 254 (in double), or kPn8None.
__global__ __launch_bounds__(256) void k_cutoff(const int64_t* __restrict__ rp, const RComp* __restrict__ rc,
                                                const float* __restrict__ mw_r, int64_t n, float t, int l2,
                                                int32_t head, RowStat* __restrict__ rs, float* __restrict__ xmw,
                                                int64_t* __restrict__ nidx, uint32_t* __restrict__ pmax,
                                                uint8_t* __restrict__ pn8) {
  __shared__ uint32_t smax;
  if (threadIdx.x == 0) smax = 0u;
  __syncthreads();
  const double td = (double)t;
  const double t2 = td * td;
  const int lane = (int)(threadIdx.x & 63u);
  uint32_t wmax = 0u;
  for (int64_t r = (int64_t)blockIdx.x * 4 + (int64_t)(threadIdx.x >> 6); r < n; r += (int64_t)gridDim.x * 4) {
    const int64_t a = rp[r];
    const int32_t len = (int32_t)(rp[r + 1] - a);
    double b = 0.0, sq = 0.0, sqp = 0.0;
    int32_t cut = len;
    float pm = 0.0f, xm = 0.0f;
    bool done = false;
    for (int32_t k0 = 0; k0 < len; k0 += 64) {
      const int32_t k = k0 + lane;
      RComp c{0, 0.0f};
      if (k < len) c = rc[a + k];
      xm = fmaxf(xm, c.w);
      if (!done) {
        const double w = (double)c.w;
        const double tb = (head >= 0 || k >= len) ? 0.0 : w * (double)mw_r[c.r];
        const double tq = w * w;
        const int cnt = len - k0 < 64 ? (int)(len - k0) : 64;
        for (int l = 0; l < cnt; ++l) {
          bool stop;
          sq += lane_value(tq, l);
          if (head >= 0) {
            // head cut: the unindexed part is the head (with head = 0 it is
            // empty and every component is indexed)
            stop = __builtin_amdgcn_readlane(c.r, l) >= head;
          } else {
            b += lane_value(tb, l);
            stop = b >= td || (l2 && sq >= t2);
          }
          if (stop) {
            cut = k0 + l;
            done = true;
            break;
          }
          sqp = sq;
        }
        if (k < cut) pm = fmaxf(pm, c.w);
      }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      pm = fmaxf(pm, __shfl_xor(pm, o, 64));
      xm = fmaxf(xm, __shfl_xor(xm, o, 64));
    }
    RowStat s;
    s.cut = cut;
    s.len = len;
    s.pmw = pm;
    // ||x'||_2 rounded up, with a relative nudge covering the double sqrt's rounding
    s.pnrm = sqp > 0.0 ? __double2float_ru(sqrt(sqp) * (1.0 + 0x1p-50)) : 0.0f;
    wmax = max(wmax, __float_as_uint(s.pnrm));
    if (lane == 0) {
      rs[r] = s;
      xmw[r] = xm;
      nidx[r] = (int64_t)(len - cut);
      const double kk = ceil((double)s.pnrm * 254.0);
      pn8[r] = kk <= 254.0 ? (uint8_t)kk : kPn8None;
    }
  }
  if (lane == 0) atomicMax(&smax, wmax);
  __syncthreads();
  if (threadIdx.x == 0 && smax) atomicMax(pmax, smax);
}

// Indexed components in row-major order -> (key = rank, value = y << 32 | weight bits),
// one wave per row.  DEEP: the weight's sign bit marks the components whose
// row's norm over the ranks up to them reaches the build threshold (squared
// norm at least lim; lim is a little low, so that rounding here and norms a
// little over 1 lose none).
template <bool DEEP>
__global__ __launch_bounds__(256) void k_emit_indexed(const int64_t* __restrict__ rp, const RComp* __restrict__ rc,
                                                      const RowStat* __restrict__ rs, const int64_t* __restrict__ ibase,
                                                      int64_t n, double lim, uint64_t* __restrict__ keys,
                                                      uint64_t* __restrict__ vals) {
  const int lane = (int)(threadIdx.x & 63u);
  for (int64_t r = (int64_t)blockIdx.x * 4 + (int64_t)(threadIdx.x >> 6); r < n; r += (int64_t)gridDim.x * 4) {
    const int64_t first = rp[r] + rs[r].cut, b = rp[r + 1];
    const int64_t o = ibase[r] - first;
    double before = 0.0;  // squared norm of the components before this chunk
    for (int64_t k0 = DEEP ? rp[r] : first; k0 < b; k0 += 64) {
      const int64_t k = k0 + lane;
      RComp c{0, 0.0f};
      if (k < b) c = rc[k];
      uint32_t deep = 0u;
      if constexpr (DEEP) {
        double sq = (double)c.w * (double)c.w;
#pragma unroll
        for (int s = 1; s < 64; s <<= 1) {
          const double u = __shfl_up(sq, s, 64);
          if (lane >= s) sq += u;
        }
        sq += before;
        deep = sq >= lim ? 0x80000000u : 0u;
        before = lane_value(sq, 63);
      }
      if (k >= first && k < b) {
        keys[o + k] = (uint64_t)(uint32_t)c.r;
        vals[o + k] = ((uint64_t)(uint32_t)r << 32) | (uint64_t)(__float_as_uint(c.w) | deep);
      }
    }
  }
}

// off[r] = first position whose (sorted) rank is >= r, r = 0..m, so list r is
// [off[r], off[r + 1]).  One thread per rank bisects the sorted keys: m log P
// reads that mostly hit L2, where counting the postings with one atomic per
// posting serialised on the dense ranks (500,000 rows of mean 120: 33.1 ms of
// atomics, and a scan after them).
__global__ void k_list_offsets(const uint64_t* __restrict__ keys, int64_t P, int64_t m, int64_t* __restrict__ off) {
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r <= m; r += (int64_t)gridDim.x * blockDim.x) {
    int64_t lo = 0, hi = P;
    while (lo < hi) {
      const int64_t mid = (lo + hi) >> 1;
      if (keys[mid] < (uint64_t)r) lo = mid + 1;
      else hi = mid;
    }
    off[r] = lo;
  }
}

// The sorted list entries, in tiles of kListTile: marked (deep) entries per
// tile, and after a scan of those counts the lists themselves.
constexpr int kListTile = 2048;

__global__ __launch_bounds__(256) void k_count_deep(const uint64_t* __restrict__ vals, int64_t P,
                                                    int64_t* __restrict__ tiles) {
  __shared__ uint32_t total;
  if (threadIdx.x == 0) total = 0u;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * kListTile;
  uint32_t c = 0;
#pragma unroll
  for (int it = 0; it < kListTile / 256; ++it) {
    const int64_t k = base + it * 256 + (int64_t)threadIdx.x;
    c += (uint32_t)__popcll(__ballot(k < P && ((uint32_t)vals[k < P ? k : 0] >> 31)));
  }
  if ((threadIdx.x & 63u) == 0) atomicAdd(&total, c);
  __syncthreads();
  if (threadIdx.x == 0) tiles[blockIdx.x] = (int64_t)total;
}

// List entries {id, weight} and their packed copy for streaming: low 16 bits
// = vector id mod 2^16 (its offset inside any power-of-two block), high 16
// bits = the weight in units of 2^-15 rounded up (w * 2^15 is exact in float,
// so the ceiling is the smallest such unit count not below w).  DEEP: the
// marked entries' ids close up into dl and their ranks (the keys) into dlr,
// and pos[k] counts those before k.
template <bool DEEP>
__global__ __launch_bounds__(256) void k_lists(const uint64_t* __restrict__ keys, const uint64_t* __restrict__ vals,
                                               int64_t P, Post* __restrict__ post, uint32_t* __restrict__ post4,
                                               const int64_t* __restrict__ tiles, uint32_t* __restrict__ pos,
                                               uint32_t* __restrict__ dl, uint32_t* __restrict__ dlr) {
  __shared__ uint32_t wtot[4];
  const int lane = (int)(threadIdx.x & 63u), wave = (int)(threadIdx.x >> 6);
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  // each wave takes consecutive entries, so that its marked ones close up in order
  constexpr int kPer = kListTile / 256;
  const int64_t base = (int64_t)blockIdx.x * kListTile + wave * (64 * kPer) + lane;
  uint64_t m[kPer];
  uint32_t y[kPer], mine = 0u;
#pragma unroll
  for (int it = 0; it < kPer; ++it) {
    const int64_t k = base + it * 64;
    bool deep = false;
    y[it] = 0u;
    if (k < P) {
      const uint64_t v = vals[k];
      Post p;
      p.y = (uint32_t)(v >> 32);
      p.w = __uint_as_float((uint32_t)v & 0x7FFFFFFFu);
      post[k] = p;
      uint32_t w15 = (uint32_t)ceilf(p.w * 32768.0f);
      if (w15 > 0xFFFFu) w15 = 0xFFFFu;
      post4[k] = (p.y & 0xFFFFu) | (w15 << 16);
      deep = ((uint32_t)v >> 31) != 0u;
      y[it] = p.y;
    }
    m[it] = __ballot(deep);
    mine += (uint32_t)__popcll(m[it]);
  }
  if constexpr (DEEP) {
    if (lane == 0) wtot[wave] = mine;
    __syncthreads();
    uint32_t at = (uint32_t)tiles[blockIdx.x];
    for (int w = 0; w < wave; ++w) at += wtot[w];
#pragma unroll
    for (int it = 0; it < kPer; ++it) {
      const int64_t k = base + it * 64;
      const uint32_t here = at + (uint32_t)__popcll(m[it] & lt);
      if (k < P) pos[k] = here;
      if ((m[it] >> lane) & 1ull) {
        dl[here] = y[it];
        dlr[here] = (uint32_t)keys[k];
      }
      at += (uint32_t)__popcll(m[it]);
    }
  }
}

// doff[r] = marked entries before list r
__global__ void k_deep_offsets(const int64_t* __restrict__ off, const uint32_t* __restrict__ pos, int64_t P, int64_t m,
                               int64_t deep, int64_t* __restrict__ doff) {
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r <= m; r += (int64_t)gridDim.x * blockDim.x)
    doff[r] = off[r] < P ? (int64_t)pos[off[r]] : deep;
}

// hoff[b * H + r] = first position in list r whose vector id is >= b * CB.
// (Several offsets of a list by one thread in turn, as in k_range_offsets, are
// slower here: 1.20 ms against 0.93 for 500,000 rows, the lists are long and
// there are fewer threads.)
__global__ void k_block_offsets(const int64_t* __restrict__ off, const Post* __restrict__ post, int32_t H, int64_t nb,
                                int32_t CB, uint32_t* __restrict__ hoff) {
  const int64_t total = (nb + 1) * (int64_t)H;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t b = e / H;
    const int32_t r = (int32_t)(e - b * H);
    int64_t lo = off[r], hi = off[r + 1];
    const uint64_t y0 = (uint64_t)b * (uint64_t)CB;
    while (lo < hi) {
      const int64_t mid = (lo + hi) >> 1;
      if ((uint64_t)post[mid].y < y0) lo = mid + 1;
      else hi = mid;
    }
    hoff[e] = (uint32_t)lo;
  }
}

// Query rows: dimension ids -> ranks (keys (row, rank)), with input checks.
// One wave per row: lanes over its components (coalesced), then the row's
// squared norm, maxweight and error flags reduced across the wave in a
// fixed order.
__global__ void k_query_keys(const int64_t* __restrict__ rp, const int32_t* __restrict__ col, const float* __restrict__ val,
                             const int32_t* __restrict__ rank, int64_t nq, int64_t m, int rbits, double norm_tol,
                             uint64_t* __restrict__ keys, uint32_t* __restrict__ vals, float* __restrict__ qmw,
                             uint32_t* __restrict__ err, unsigned long long* __restrict__ bad_row) {
  const int lane = (int)(threadIdx.x & 63u);
  const int64_t wpb = (int64_t)(blockDim.x >> 6);
  for (int64_t r = (int64_t)blockIdx.x * wpb + (int64_t)(threadIdx.x >> 6); r < nq; r += (int64_t)gridDim.x * wpb) {
    const int64_t a = rp[r], b = rp[r + 1];
    uint32_t e = 0;
    double ss = 0.0;
    float mx = 0.0f;
    for (int64_t k = a + lane; k < b; k += 64) {
      const int32_t d = col[k];
      const float w = val[k];
      if (d < 0 || (int64_t)d >= m) {
        e |= ERR_DIM;
        keys[k] = ((uint64_t)r << rbits);
      } else {
        keys[k] = ((uint64_t)r << rbits) | (uint64_t)rank[d];
      }
      if (!(w > 0.0f) || !isfinite(w)) e |= ERR_WEIGHT;
      ss += (double)w * (double)w;
      mx = fmaxf(mx, w);
      vals[k] = __float_as_uint(w);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      ss += __shfl_xor(ss, o, 64);
      mx = fmaxf(mx, __shfl_xor(mx, o, 64));
      e |= __shfl_xor(e, o, 64);
    }
    if (lane == 0) {
      if (b > a && !(fabs(sqrt(ss) - 1.0) <= norm_tol)) e |= ERR_NORM;
      qmw[r] = mx;
      if (e) {
        atomicOr(err, e);
        atomicMin(bad_row, (unsigned long long)r);
      }
    }
  }
}

// Query rows of at most kQueryRow components in rank space, one workgroup per
// row: checked, ranks gathered and sorted in LDS (n2: the longest row's length
// as a power of two) and written once, with the row's largest weight.  A row
// that fails a check is written with zero weights, which meet nothing, so the
// kernels that follow need not wait for the host to read the flags.  Also
// makes the call's copies of row_ptr and the thresholds and clears its
// counters: a small batch is bound by launches and copies (keys, sort,
// unpacking, fills and copies of the parts were 100 us of a query's 167).
__global__ __launch_bounds__(256) void k_query_rows(QueryRowsArgs a, int n2max) {
  extern __shared__ uint64_t row[];
  __shared__ double ssq[4];
  __shared__ float smx[4];
  __shared__ uint32_t flags;
  const int tid = (int)threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  if (blockIdx.x == 0)
    for (int k = tid; k < a.zeros; k += 256) a.zero[k] = 0ull;
  for (int64_t r = blockIdx.x; r < a.nq; r += gridDim.x) {
    const int64_t beg = a.rp[r];
    const int len = (int)(a.rp[r + 1] - beg);
    if (tid == 0) {
      flags = 0u;
      if (a.rp_out) {
        a.rp_out[r] = beg;
        if (r + 1 == a.nq) a.rp_out[a.nq] = beg + len;
      }
      if (a.t_out) a.t_out[r] = a.t[r];
    }
    int n2 = 1;
    while (n2 < len) n2 <<= 1;
    if (n2 > n2max) n2 = n2max;  // (never: the host has the longest row)
    uint32_t e = 0u;
    double ss = 0.0;
    float mx = 0.0f;
    for (int i = tid; i < n2; i += 256) {
      uint64_t c = ~0ull;  // above every component
      if (i < len) {
        const int32_t d = a.col[beg + i];
        const float w = a.val[beg + i];
        uint32_t rk = 0u;
        if (d < 0 || (int64_t)d >= a.m) e |= ERR_DIM;
        else rk = (uint32_t)a.rank[d];
        if (!(w > 0.0f) || !isfinite(w)) e |= ERR_WEIGHT;
        ss += (double)w * (double)w;
        mx = fmaxf(mx, w);
        c = ((uint64_t)rk << 32) | (uint64_t)__float_as_uint(w);
      }
      row[i] = c;
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      ss += __shfl_xor(ss, o, 64);
      mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    }
    if (lane == 0) {
      ssq[wave] = ss;
      smx[wave] = mx;
    }
    __syncthreads();
    if (e) atomicOr(&flags, e);
    for (int size = 2; size <= n2; size <<= 1)
      for (int stride = size >> 1; stride > 0; stride >>= 1) {
        for (int i = tid; i < n2 / 2; i += 256) compare_exchange(row, i, stride, size);
        __syncthreads();
      }
    ss = ssq[0] + ssq[1] + ssq[2] + ssq[3];
    bool dup = false;
    for (int i = tid + 1; i < len; i += 256) dup = dup || (uint32_t)(row[i - 1] >> 32) == (uint32_t)(row[i] >> 32);
    if (dup) atomicOr(&flags, ERR_DUP);
    if (tid == 0 && len > 0 && !(fabs(sqrt(ss) - 1.0) <= a.tol)) atomicOr(&flags, ERR_NORM);
    __syncthreads();
    const uint32_t f = flags;
    for (int i = tid; i < len; i += 256)
      a.rc[beg + i] = RComp{(int32_t)(row[i] >> 32), f ? 0.0f : __uint_as_float((uint32_t)row[i])};
    if (tid == 0) {
      a.qmw[r] = f ? 0.0f : fmaxf(fmaxf(smx[0], smx[1]), fmaxf(smx[2], smx[3]));
      if (f) {
        atomicOr(a.err, f);
        atomicMin(a.bad, (unsigned long long)r);
      }
    }
    __syncthreads();
  }
}

// maxweight by dimension id, and the rows' cuts
__global__ void k_export(const int32_t* __restrict__ rank, const float* __restrict__ mw_r, int64_t m,
                         const RowStat* __restrict__ rs, int64_t n, float* __restrict__ mw, int32_t* __restrict__ cut) {
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < m || k < n; k += (int64_t)gridDim.x * blockDim.x) {
    if (mw && k < m) mw[k] = mw_r[rank[k]];
    if (cut && k < n) cut[k] = rs[k].cut;
  }
}

unsigned grid(int64_t n, int threads = 256) {
  int64_t g = (n + threads - 1) / threads;
  if (g > 32768) g = 32768;
  if (g < 1) g = 1;
  return (unsigned)g;
}

// Workgroups of four waves for kernels that take one row per wave: enough to
// fill the device several times over, the rest by striding.
unsigned row_grid(int64_t n) {
  const int64_t g = (n + 3) / 4;
  return (unsigned)(g < 8192 ? g : 8192);
}

}  // namespace

#define LAUNCH(k, n, ...)                                                 \
  do {                                                                    \
    hipLaunchKernelGGL(k, dim3(grid(n)), dim3(256), 0, s, __VA_ARGS__);   \
    hipError_t e_ = hipGetLastError();                                    \
    if (e_ != hipSuccess) return e_;                                      \
  } while (0)

hipError_t launch_check_rowptr(const int64_t* rp, int64_t n, int64_t nnz, uint32_t* err, unsigned long long* bad,
                               unsigned long long* longest, hipStream_t s) {
  // (few waves: each ends with one atomic on the longest length)
  const unsigned g = grid(n + 1);
  hipLaunchKernelGGL(k_check_rowptr, dim3(g < 256 ? g : 256), dim3(256), 0, s, rp, n, nnz, err, bad, longest);
  return hipGetLastError();
}

hipError_t launch_validate_count(const int64_t* rp, const int32_t* col, const float* val, int64_t n, int64_t m,
                                 double tol, uint32_t* cnt, uint32_t* mwbits, uint32_t* err, unsigned long long* bad,
                                 hipStream_t s) {
  // few enough workgroups that their tables pay (each ends with up to
  // kCountSlots pairs of atomics), enough to fill the device
  const int64_t g = (n + 15) / 16;
  hipLaunchKernelGGL(k_validate_count, dim3((unsigned)(g < 1 ? 1 : g < 512 ? g : 512)), dim3(1024), 0, s, rp, col, val, n,
                     m, tol, cnt, mwbits, err, bad);
  return hipGetLastError();
}

hipError_t launch_sort_rows(const int64_t* rp, const int32_t* col, const float* val, const int32_t* rank, int64_t n,
                            int64_t longest, RComp* rc, uint32_t* err, unsigned int* nlong, uint32_t* longs,
                            hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (longest > kLongRow) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_sort_rows, dim3(row_grid(n)), dim3(256), 0, s, rp, col, val, rank, n, rc, err, nlong, longs);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || longest <= kWaveRow) return e;
  hipLaunchKernelGGL(k_sort_long_rows, dim3((unsigned)(n < 1024 ? n : 1024)), dim3(1024), 0, s, rp, col, val, rank, rc,
                     err, nlong, longs);
  return hipGetLastError();
}

hipError_t launch_dim_keys(const uint32_t* cnt, int64_t m, int64_t n, int dbits, uint64_t* keys, uint64_t* vals,
                           hipStream_t s) {
  LAUNCH(k_dim_keys, m, cnt, m, n, dbits, keys, vals);
  return hipSuccess;
}

hipError_t launch_rank_from_sorted(const uint64_t* vals, int64_t m, const uint32_t* cnt, const uint32_t* mwbits,
                                   int32_t* rank, float* mw_r, uint32_t* cnt_r, hipStream_t s) {
  LAUNCH(k_rank_from_sorted, m, vals, m, cnt, mwbits, rank, mw_r, cnt_r);
  return hipSuccess;
}

hipError_t launch_row_keys(const int64_t* rp, const int32_t* col, const float* val, const int32_t* rank, int64_t n,
                           int rbits, uint64_t* keys, uint32_t* vals, hipStream_t s) {
  LAUNCH(k_row_keys, n, rp, col, val, rank, n, rbits, keys, vals);
  return hipSuccess;
}

hipError_t launch_unpack_rows(const uint64_t* keys, const uint32_t* vals, int64_t nnz, int rbits, RComp* rc,
                              uint32_t* err, hipStream_t s) {
  LAUNCH(k_unpack_rows, nnz, keys, vals, nnz, rbits, rc, err);
  return hipSuccess;
}

hipError_t launch_cutoff(const int64_t* rp, const RComp* rc, const float* mw_r, int64_t n, float t, int l2,
                         int32_t head, RowStat* rs, float* xmw, int64_t* nidx, uint32_t* pmax, uint8_t* pn8,
                         hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_cutoff, dim3(row_grid(n)), dim3(256), 0, s, rp, rc, mw_r, n, t, l2, head, rs, xmw, nidx, pmax,
                     pn8);
  return hipGetLastError();
}

hipError_t launch_emit_indexed(const int64_t* rp, const RComp* rc, const RowStat* rs, const int64_t* ibase, int64_t n,
                               double lim, uint64_t* keys, uint64_t* vals, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (lim >= 0.0)
    hipLaunchKernelGGL(k_emit_indexed<true>, dim3(row_grid(n)), dim3(256), 0, s, rp, rc, rs, ibase, n, lim, keys, vals);
  else
    hipLaunchKernelGGL(k_emit_indexed<false>, dim3(row_grid(n)), dim3(256), 0, s, rp, rc, rs, ibase, n, lim, keys, vals);
  return hipGetLastError();
}

hipError_t launch_list_offsets(const uint64_t* keys, int64_t P, int64_t m, int64_t* off, hipStream_t s) {
  LAUNCH(k_list_offsets, m + 1, keys, P, m, off);
  return hipSuccess;
}

int64_t list_tiles(int64_t P) { return (P + kListTile - 1) / kListTile; }

hipError_t launch_count_deep(const uint64_t* vals, int64_t P, int64_t* tiles, hipStream_t s) {
  if (P <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_count_deep, dim3((unsigned)list_tiles(P)), dim3(256), 0, s, vals, P, tiles);
  return hipGetLastError();
}

hipError_t launch_lists(const uint64_t* keys, const uint64_t* vals, int64_t P, Post* post, uint32_t* post4,
                        const int64_t* tiles, uint32_t* pos, uint32_t* dl, uint32_t* dlr, hipStream_t s) {
  if (P <= 0) return hipSuccess;
  const unsigned g = (unsigned)list_tiles(P);
  if (dl)
    hipLaunchKernelGGL(k_lists<true>, dim3(g), dim3(256), 0, s, keys, vals, P, post, post4, tiles, pos, dl, dlr);
  else
    hipLaunchKernelGGL(k_lists<false>, dim3(g), dim3(256), 0, s, keys, vals, P, post, post4, tiles, pos, dl, dlr);
  return hipGetLastError();
}

hipError_t launch_deep_offsets(const int64_t* off, const uint32_t* pos, int64_t P, int64_t m, int64_t deep,
                               int64_t* doff, hipStream_t s) {
  LAUNCH(k_deep_offsets, m + 1, off, pos, P, m, deep, doff);
  return hipSuccess;
}

hipError_t launch_block_offsets(const int64_t* off, const Post* post, int32_t H, int64_t nb, int32_t CB,
                                uint32_t* hoff, hipStream_t s) {
  LAUNCH(k_block_offsets, (nb + 1) * (int64_t)H, off, post, H, nb, CB, hoff);
  return hipSuccess;
}

hipError_t launch_export(const int32_t* rank, const float* mw_r, int64_t m, const RowStat* rs, int64_t n, float* mw,
                         int32_t* cut, hipStream_t s) {
  hipLaunchKernelGGL(k_export, dim3(grid(m > n ? m : n)), dim3(256), 0, s, rank, mw_r, m, rs, n, mw, cut);
  return hipGetLastError();
}

hipError_t launch_query_rows(const QueryRowsArgs& a, int64_t longest, hipStream_t s) {
  if (a.nq <= 0) return hipSuccess;
  if (!a.rp || !a.rank || !a.rc || !a.qmw || !a.err || !a.bad || longest < 0 || longest > kQueryRow ||
      (longest > 0 && (!a.col || !a.val)) || (a.zeros > 0 && !a.zero) || (a.t_out && !a.t))
    return hipErrorInvalidValue;
  int n2 = 1;
  while (n2 < longest) n2 <<= 1;
  hipLaunchKernelGGL(k_query_rows, dim3((unsigned)(a.nq < 16384 ? a.nq : 16384)), dim3(256),
                     sizeof(uint64_t) * (size_t)n2, s, a, n2);
  return hipGetLastError();
}

hipError_t launch_query_keys(const int64_t* rp, const int32_t* col, const float* val, const int32_t* rank, int64_t nq,
                             int64_t m, int rbits, double tol, uint64_t* keys, uint32_t* vals, float* qmw,
                             uint32_t* err, unsigned long long* bad, hipStream_t s) {
  if (nq <= 0) return hipSuccess;
  const int64_t blocks = (nq + 3) / 4;  // 4 waves of 64 lanes per block, one row per wave
  hipLaunchKernelGGL(k_query_keys, dim3((unsigned)(blocks < 32768 ? blocks : 32768)), dim3(256), 0, s, rp, col, val, rank,
                     nq, m, rbits, tol, keys, vals, qmw, err, bad);
  return hipGetLastError();
}

}  // namespace apss
