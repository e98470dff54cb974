// The self-join by pairs of list entries under a row-sketch bound.
//
// Let d be the rarest dimension (largest rank) that two rows share.  Then
//   sim(x, y) = sum over ranks <= d  <=  ||x_{<=d}|| ||y_{<=d}||,
// so both rows' norms over the ranks up to d reach t: both are in the deep
// list of d, which holds the rows y with y[d] > 0 and ||y_{<=d}|| >= t (a
// part of the inverted list of the indexed components, Section 3.2.2, since
// the unindexed part's norm stays below t).  It is enough to test, in every
// deep list, the pairs of its entries, and to keep a pair in the list of its
// rarest shared dimension.
//
// The test is a bound too: with the ranks cut into kSkGroups groups of about
// equal postings and n_g(x) the norm of x over group g, Cauchy-Schwarz group
// by group gives
//   sim(x, y) <= sum over groups g <= group(d) of n_g(x) n_g(y).
// The norms are kept as bytes rounded up (a row's sketch), so the sum of
// their products is an exact upper bound in integers, and it is a small
// matrix product: the sketches of 64 entries against those of 32 others, on
// the int8 matrix cores.  No list entry is added into an accumulator and no
// score is kept: a pair below the bound is done, and a pair that reaches it
// is decided on its two rows by the rescore every kernel shares, so the pairs
// reported and their similarities are those of the accumulating join.
#include "apss_internal.h"
#include "join.h"
#include <algorithm>

#include "pairs.h"
#include "rescore.h"

namespace apss {

namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ float lane_float(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }

__global__ void k_groups(const int64_t* __restrict__ cum, const uint32_t* __restrict__ cnt_r, int64_t m, int64_t nnz,
                         uint16_t* __restrict__ gid) {
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < m; r += (int64_t)gridDim.x * blockDim.x) {
    // the group of the rank's last component when all are laid out by rank
    const int64_t last = cum[r] + (int64_t)cnt_r[r] - 1;
    const int64_t g = nnz > 0 && last >= 0 ? last * kFineGroups / nnz : 0;
    gid[r] = (uint16_t)(g < kFineGroups ? g : kFineGroups - 1);
  }
}

// out[0] += sum over ranks of components times postings, halved: the list
// entries an accumulating self-join visits; out[1] those of ranks >= hb.
__global__ void k_visits(const uint32_t* __restrict__ cnt_r, const int64_t* __restrict__ off, int64_t m, int64_t hb,
                         unsigned long long* __restrict__ out) {
  __shared__ unsigned long long sum[2];
  if (threadIdx.x < 2) sum[threadIdx.x] = 0ull;
  __syncthreads();
  unsigned long long v = 0ull, tail = 0ull;
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < m; r += (int64_t)gridDim.x * blockDim.x) {
    const unsigned long long x = (unsigned long long)cnt_r[r] * (unsigned long long)(off[r + 1] - off[r]) / 2;
    v += x;
    if (r >= hb) tail += x;
  }
  if (v) atomicAdd(&sum[0], v);
  if (tail) atomicAdd(&sum[1], tail);
  __syncthreads();
  if (threadIdx.x < 2 && sum[threadIdx.x]) atomicAdd(&out[threadIdx.x], sum[threadIdx.x]);
}

__global__ __launch_bounds__(256) void k_norm_codes(const uint8_t* __restrict__ pn8, int64_t n,
                                                    unsigned long long* __restrict__ hist) {
  __shared__ unsigned int h[256];
  h[threadIdx.x] = 0u;
  __syncthreads();
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n; r += (int64_t)gridDim.x * blockDim.x)
    atomicAdd(&h[pn8[r]], 1u);
  __syncthreads();
  if (h[threadIdx.x]) atomicAdd(&hist[threadIdx.x], (unsigned long long)h[threadIdx.x]);
}

__global__ void k_widen(const uint32_t* __restrict__ in, int64_t n, int64_t* __restrict__ out) {
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x)
    out[k] = (int64_t)in[k];
}

// Least code of a squared norm in units of 2^-31 (rounded up).
__device__ __forceinline__ uint32_t norm_code(uint32_t v) {
  const uint32_t c = (uint32_t)ceil(sqrt((double)v * 0x1p-31) * (kSkScale * (1.0 + 1e-12)));
  return c > 127u ? 127u : c;  // past any validated norm
}

// Sketches, one wave per row.  Squared weights are summed per group as
// integers in units of 2^-31, each rounded up, so the sums bound the squared
// norms from above and do not depend on the order of the LDS atomics.  A row
// has one of kMidGroups groups, one of kSkGroups (pairs of those; sk may be
// NULL), and if it has more than kFineRow components one of kFineGroups
// (quarters of those), in the order the waves reach them.
__global__ __launch_bounds__(256) void k_sketch(const int64_t* __restrict__ rp, const RComp* __restrict__ rc,
                                                const uint16_t* __restrict__ gid, int64_t n, uint8_t* __restrict__ sk,
                                                uint8_t* __restrict__ mid, unsigned int* __restrict__ nfine,
                                                uint32_t* __restrict__ fidx, uint8_t* __restrict__ fsk) {
  __shared__ uint32_t acc[4][kFineGroups];
  static_assert(kFineGroups == 4 * kMidGroups && kMidGroups == 2 * kSkGroups && kMidGroups == 256, "group levels");
  const int lane = (int)(threadIdx.x & 63u);
  uint32_t* const mine = acc[threadIdx.x >> 6];
  for (int g = lane; g < kFineGroups; g += 64) mine[g] = 0u;
  wave_lds_order();
  for (int64_t r = (int64_t)blockIdx.x * 4 + (int64_t)(threadIdx.x >> 6); r < n; r += (int64_t)gridDim.x * 4) {
    const int64_t a = rp[r], b = rp[r + 1];
    const bool fine = b - a > kFineRow;
    const int shift = fine ? 0 : 2;
    for (int64_t k = a + lane; k < b; k += 64) {
      const RComp c = rc[k];
      atomicAdd(&mine[gid[c.r] >> shift], (uint32_t)ceil((double)c.w * (double)c.w * 2147483648.0));
    }
    wave_lds_order();
    // lane l holds the mid groups 4 l .. 4 l + 3
    uint32_t v[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) v[g] = mine[4 * lane + g];
    uint32_t at = 0xFFFFFFFFu;
    if (fine) {
      if (lane == 0) at = atomicAdd(nfine, 1u);
      at = (uint32_t)uni((int)at);
      uint32_t word[4] = {0u, 0u, 0u, 0u};
#pragma unroll
      for (int g = 0; g < 4; ++g) v[g] = 0u;
#pragma unroll
      for (int g = 0; g < 16; ++g) {
        const uint32_t x = mine[16 * lane + g];
        v[g >> 2] += x;
        word[g >> 2] |= norm_code(x) << (8 * (g & 3));
      }
      *reinterpret_cast<uint4*>(fsk + (int64_t)at * kFineGroups + 16 * lane) = make_uint4(word[0], word[1], word[2], word[3]);
    }
    if (lane == 0) fidx[r] = at;
    *reinterpret_cast<uint32_t*>(mid + r * kMidGroups + 4 * lane) =
        norm_code(v[0]) | (norm_code(v[1]) << 8) | (norm_code(v[2]) << 16) | (norm_code(v[3]) << 24);
    if (sk)
      *reinterpret_cast<uint16_t*>(sk + r * kSkGroups + 2 * lane) =
          (uint16_t)(norm_code(v[0] + v[1]) | (norm_code(v[2] + v[3]) << 8));
    wave_lds_order();
    for (int g = lane; g < (fine ? kFineGroups : kMidGroups); g += 64) mine[g] = 0u;
    wave_lds_order();
  }
}

// A list of at least kWideList entries is cut into blocks of kWideRows (the
// last may be short); a unit is a block a against one chunk of kWideSpan of
// the blocks up to it, so that no unit is long: block a has a / kWideSpan + 1
// chunks.  units_before(a) = units of the blocks before a.
__host__ __device__ __forceinline__ int64_t units_before(int64_t a) {
  const int64_t k = a / kWideSpan;
  return kWideSpan * k * (k + 1) / 2 + (a - kWideSpan * k) * (k + 1);
}

// Block and chunk of a long list's u-th unit.
__device__ __forceinline__ void unit_at(uint32_t u, int* a, int* chunk) {
  // kWideSpan k (k + 1) / 2 <= u: k from the square root, mended by one
  int k = (int)((sqrtf(1.0f + (8.0f / kWideSpan) * (float)u) - 1.0f) * 0.5f);
  while (units_before((int64_t)kWideSpan * (k + 1)) <= (int64_t)u) ++k;
  while (k > 0 && units_before((int64_t)kWideSpan * k) > (int64_t)u) --k;
  const int rem = (int)((int64_t)u - units_before((int64_t)kWideSpan * k));
  *a = kWideSpan * k + rem / (k + 1);
  *chunk = rem % (k + 1);
}

// Units of a list: wide ones of a long list, blocks of kUnitRows of a short one.
__device__ __forceinline__ int64_t wide_count(int64_t len) {
  return len < kWideList ? 0 : units_before((len + kWideRows - 1) / kWideRows);
}
__device__ __forceinline__ int64_t short_count(int64_t len) {
  return len <= kTinyList || len >= kWideList ? 0 : (len + kUnitRows - 1) / kUnitRows;
}

template <bool WIDE>
__global__ void k_unit_counts(const int64_t* __restrict__ doff, int64_t m, int64_t* __restrict__ ucnt) {
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < m; r += (int64_t)gridDim.x * blockDim.x) {
    const int64_t len = doff[r + 1] - doff[r];
    ucnt[r] = WIDE ? wide_count(len) : short_count(len);
  }
}

template <bool WIDE>
__global__ void k_unit_fill(const int64_t* __restrict__ doff, const int64_t* __restrict__ uoff, int64_t m,
                            uint2* __restrict__ units) {
  const int lane = (int)(threadIdx.x & 63u);
  const int64_t nw = ((int64_t)gridDim.x * blockDim.x) >> 6;
  for (int64_t r0 = (((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6) * 64; r0 < m; r0 += nw * 64) {
    // 64 ranks per wave: few units by lane, the many of a long list by all lanes
    const int64_t r = r0 + lane;
    const int64_t len = r < m ? doff[r + 1] - doff[r] : 0;
    const int64_t nu = WIDE ? wide_count(len) : short_count(len);
    if (nu > 0 && nu <= 4)
      for (int64_t u = 0; u < nu; ++u) units[uoff[r] + u] = make_uint2((uint32_t)r, (uint32_t)u);
    uint64_t big = __ballot(nu > 4);
    while (big) {
      const int l = __ffsll((unsigned long long)big) - 1;
      big &= big - 1;
      const int64_t rr = r0 + l;
      const int64_t nn = __shfl(nu, l, 64);
      for (int64_t u = lane; u < nn; u += 64) units[uoff[rr] + u] = make_uint2((uint32_t)rr, (uint32_t)u);
    }
  }
}

// q's weight in rank r by binary search of its rank-ordered row (0 if absent)
__device__ __forceinline__ float row_lookup(const RComp* __restrict__ q, int qlen, int32_t r) {
  int lo = 0, hi = qlen;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (q[mid].r < r) lo = mid + 1;
    else hi = mid;
  }
  return (lo < qlen && q[lo].r == r) ? q[lo].w : 0.0f;
}

// A row held by a wave in LDS for lookups: ranks, padded to a power of two
// with a rank no row has, and for rows of at most kStageRow components the
// weights too; of longer rows (up to kStageRanks) the weights found are read
// from memory.
constexpr int kStageRow = 1024;
static_assert(kStageRanks == 2 * kStageRow, "ranks, or ranks and weights");
struct StagedRow {
  int32_t v[kStageRanks];  // ranks, then (from kStageRow on) weights' bits or more ranks
};

// Weights of a staged row in the ranks of N components per lane (0 if
// absent); the N searches advance together, so their LDS reads overlap.
template <int N>
__device__ __forceinline__ void staged_lookup(const StagedRow& st, const RComp* __restrict__ row, int len, int p2,
                                              const int32_t (&r)[N], float (&v)[N]) {
  const int32_t* const ranks = st.v;
  int at[N];
#pragma unroll
  for (int u = 0; u < N; ++u) at[u] = 0;  // entries before at have smaller ranks
  for (int step = p2 >> 1; step > 0; step >>= 1) {
#pragma unroll
    for (int u = 0; u < N; ++u) at[u] += ranks[at[u] + step - 1] < r[u] ? step : 0;
  }
  int32_t got[N];
#pragma unroll
  for (int u = 0; u < N; ++u) got[u] = ranks[at[u]];
#pragma unroll
  for (int u = 0; u < N; ++u) {
    // at < p2; entry at may still be smaller when it is the last
    const bool hit = got[u] == r[u];
    if (len <= kStageRow) v[u] = hit ? __int_as_float(ranks[kStageRow + at[u]]) : 0.0f;
    else v[u] = hit ? row[at[u]].w : 0.0f;
  }
}

// Keeps the bytes of the word of groups g0 .. g0 + 3 whose group is at most g.
__device__ __forceinline__ uint32_t group_mask(int g0, int g) {
  return g0 + 3 <= g ? 0xFFFFFFFFu : (g0 > g ? 0u : 0xFFFFFFFFu >> (8 * (g0 + 3 - g)));
}

struct Decided {
  unsigned long long surv = 0, ver = 0, band = 0;  // wave-uniform
};

// A pair's two rows: y, whose components the lanes take, and q, whose weights
// are looked up -- the smaller and the larger id of a self-join's pair, or
// the corpus row and the query, the orientations of the join kernel.
__device__ __forceinline__ uint32_t pair_y(const PairArgs& a, uint32_t x, uint32_t z) { return a.query || x < z ? x : z; }
__device__ __forceinline__ uint32_t pair_q(const PairArgs& a, uint32_t x, uint32_t z) { return a.query || x < z ? z : x; }
__device__ __forceinline__ float pair_t(const PairArgs& a, uint32_t q) { return a.qt ? a.qt[q] : a.t; }
__device__ __forceinline__ uint64_t pair_key(const PairArgs& a, uint32_t y, uint32_t q) {
  return a.query ? ((uint64_t)q << a.bj) | (uint64_t)y : ((uint64_t)y << a.bj) | (uint64_t)q;
}

// Longest row whose plain sum drops a pair: 64 chains of its components and a
// butterfly of six levels add, each step within 2^-24 of a sum of at most
// 1 + 1e-5, so the error stays below (ceil(k / 64) + 6) 2^-24, for this many a
// third of the slack.  (At a million components it can be three times the
// slack.)
constexpr int kPlainRow = 32768;
static_assert((kPlainRow / 64 + 6) * 0x1p-24 < 0.5f * kSlack, "plain sums decide inside the slack");

// Decide `here` (at most 64) pairs, lane l's being (x, z) from the deep list
// of rank d (a query's pairs: past every rank), one at a time by the whole
// wave: row q goes to LDS, the lanes take y's components and look them up.
// Row bounds are read for all pairs at once, and the next pair's rows (their
// first 128 components) are loaded while a pair is decided, so that a pair of
// ordinary rows costs LDS latencies only; a binary search in global memory
// cost 15-30 us per pair and wave.  Long rows are first gone through from
// their rare end, 256 components at a time: a pair that belongs to a rarer
// list (long rows share many) leaves at once, and one whose plain sum stays
// below t is not summed again.
__device__ __forceinline__ void decide_pairs(const PairArgs& a, StagedRow& st, int lane, int here, uint32_t x,
                                             uint32_t z, int d, WaveEmit& em, Decided& dc) {
  uint32_t y = pair_y(a, x, z), q = pair_q(a, x, z);
  uint32_t ys = 0u, qs = 0u;
  int yl = 0, ql = 0;
  float tq = 0.0f;
  if (lane < here) {
    ys = (uint32_t)a.rp[y];  // row offsets fit 32 bits (nnz < 2^32)
    yl = (int)((uint32_t)a.rp[y + 1] - ys);
    qs = (uint32_t)a.qrp[q];
    ql = (int)((uint32_t)a.qrp[q + 1] - qs);
    tq = pair_t(a, q);
  }
  // two long rows: first the finer sketch bound, two kilobytes in place of
  // rows several times that (flat long rows pass the coarse one with each other)
  {
    const bool longs = lane < here && yl > kFineRow && ql > kFineRow;
    uint32_t fy = 0u, fq = 0u;
    int gd = 0;
    if (longs) {
      fy = a.fidx[y];
      fq = a.qfidx[q];
      gd = a.query ? kFineGroups - 1 : a.gid[d];
    }
    uint64_t lm = __ballot(longs);
    uint64_t out = 0ull;
    while (lm) {
      const int l = __ffsll((unsigned long long)lm) - 1;
      lm &= lm - 1;
      const i32x4 u = *reinterpret_cast<const i32x4*>(
          a.fsk + (int64_t)(uint32_t)__builtin_amdgcn_readlane((int)fy, l) * kFineGroups + 16 * lane);
      const i32x4 w = *reinterpret_cast<const i32x4*>(
          a.qfsk + (int64_t)(uint32_t)__builtin_amdgcn_readlane((int)fq, l) * kFineGroups + 16 * lane);
      const int g = __builtin_amdgcn_readlane(gd, l);
      int dot = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) dot = __builtin_amdgcn_sdot4(u[i] & (int)group_mask(16 * lane + 4 * i, g), w[i], dot, false);
      dot = wave_sum(dot);
      if (dot < pair_threshold(lane_float(tq, l))) out |= 1ull << l;
    }
    if (out) {
      // close up the pairs that are left, in order
      const bool stays = lane < here && !((out >> lane) & 1ull);
      const uint64_t sm = __ballot(stays);
      const int to = (int)__popcll(sm & ((lane == 0) ? 0ull : (~0ull >> (64 - lane))));
      here = (int)__popcll(sm);
      wave_lds_order();
      if (stays) {
        st.v[to] = lane;
      }
      wave_lds_order();
      const int from = lane < here ? st.v[lane] : 0;
      wave_lds_order();
      x = (uint32_t)__shfl((int)x, from, 64);
      z = (uint32_t)__shfl((int)z, from, 64);
      d = __shfl(d, from, 64);
      ys = (uint32_t)__shfl((int)ys, from, 64);
      qs = (uint32_t)__shfl((int)qs, from, 64);
      yl = __shfl(yl, from, 64);
      ql = __shfl(ql, from, 64);
      tq = __shfl(tq, from, 64);
      y = pair_y(a, x, z);
      q = pair_q(a, x, z);
      if (here == 0) return;
    }
  }
  RComp ny[2], nq[2];
  auto fetch = [&](int l) {
    const RComp* yrow = a.rc + (uint32_t)__builtin_amdgcn_readlane((int)ys, l);
    const RComp* qrow = a.qrc + (uint32_t)__builtin_amdgcn_readlane((int)qs, l);
    const int yn = __builtin_amdgcn_readlane(yl, l), qm = __builtin_amdgcn_readlane(ql, l);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k = 64 * h + lane;
      ny[h] = yrow[k < yn ? k : 0];
      nq[h] = qrow[k < qm ? k : 0];
    }
  };
  fetch(0);
  for (int l = 0; l < here; ++l) {
    const RComp cy[2] = {ny[0], ny[1]}, cq[2] = {nq[0], nq[1]};
    const RComp* yrow = a.rc + (uint32_t)__builtin_amdgcn_readlane((int)ys, l);
    const RComp* qrow = a.qrc + (uint32_t)__builtin_amdgcn_readlane((int)qs, l);
    const int ylen = __builtin_amdgcn_readlane(yl, l), qlen = __builtin_amdgcn_readlane(ql, l);
    const int32_t dl = __builtin_amdgcn_readlane(d, l);
    const float t = lane_float(tq, l);
    if (l + 1 < here) fetch(l + 1);
    const bool staged = qlen <= kStageRanks;
    int p2 = 64;
    if (staged) {
      while (p2 < qlen) p2 <<= 1;
      int32_t* const ranks = st.v;
      ranks[lane] = lane < qlen ? cq[0].r : 0x7FFFFFFF;
      ranks[kStageRow + lane] = __float_as_int(cq[0].w);
      if (qlen > 64) {
        ranks[64 + lane] = 64 + lane < qlen ? cq[1].r : 0x7FFFFFFF;
        ranks[kStageRow + 64 + lane] = __float_as_int(cq[1].w);
      }
      const bool both = qlen <= kStageRow;
      for (int k0 = 128; k0 < p2; k0 += 256) {
        RComp c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int k = k0 + 64 * u + lane;
          c[u] = qrow[k < qlen ? k : qlen - 1];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int k = k0 + 64 * u + lane;
          if (k < p2) {
            ranks[k] = k < qlen ? c[u].r : 0x7FFFFFFF;
            if (both) ranks[kStageRow + k] = __float_as_int(c[u].w);
          }
        }
      }
      wave_lds_order();
    }
    bool rarer = false;  // a shared dimension rarer than d: another list's pair
    auto look = [&](int32_t r) {
      float v;
      if (staged) {
        const int32_t rr[1] = {r};
        float vv[1];
        staged_lookup<1>(st, qrow, qlen, p2, rr, vv);
        v = vv[0];
      } else {
        v = row_lookup(qrow, qlen, r);
      }
      return v;
    };
    float s32;
    if (staged && ylen <= 128) {
      // (most rows of ordinary corpora have one chunk: the vector units bind)
      const int32_t rr[2] = {lane < ylen ? cy[0].r : -1, 64 + lane < ylen ? cy[1].r : -1};
      float vv[2] = {0.0f, 0.0f};
      if (ylen <= 64) {
        const int32_t r1[1] = {rr[0]};
        float v1[1];
        staged_lookup<1>(st, qrow, qlen, p2, r1, v1);
        vv[0] = v1[0];
      } else {
        staged_lookup<2>(st, qrow, qlen, p2, rr, vv);
      }
      rarer = (rr[0] > dl && vv[0] != 0.0f) || (rr[1] > dl && vv[1] != 0.0f);
      if (__ballot(rarer)) {
        wave_lds_order();
        continue;
      }
      s32 = wave_dot2_of([&](int k) { return k < 64 ? cy[0] : cy[1]; }, ylen, lane,
                         [&](int k, int32_t) { return k < 64 ? vv[0] : vv[1]; });
    } else {
      float part = 0.0f;
      for (int k1 = (ylen - 1) & ~255; k1 >= 0; k1 -= 256) {
        int32_t rr[4];
        float ww[4], vv[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int k = k1 + 64 * u + lane;
          const RComp c = yrow[k < ylen ? k : ylen - 1];
          rr[u] = k < ylen ? c.r : -1;
          ww[u] = c.w;
        }
        if (staged) {
          staged_lookup<4>(st, qrow, qlen, p2, rr, vv);
        } else {
#pragma unroll
          for (int u = 0; u < 4; ++u) vv[u] = row_lookup(qrow, qlen, rr[u]);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          part += vv[u] * ww[u];
          rarer = rarer || (rr[u] > dl && vv[u] != 0.0f);
        }
        if (__ballot(rarer)) break;
      }
      if (__ballot(rarer)) {
        wave_lds_order();
        continue;
      }
      part = wave_sum(part);
      if (ylen <= kPlainRow && part < t - kSlack) {
        ++dc.surv;
        wave_lds_order();
        continue;
      }
      s32 = wave_dot2_of([&](int k) { return k < 64 ? cy[0] : (k < 128 ? cy[1] : yrow[k]); }, ylen, lane,
                         [&](int, int32_t r) { return look(r); });
    }
    ++dc.surv;
    if (s32 >= t - kSlack) ++dc.ver;
    float sim;
    bool banded;
    const bool keep = wave_decide(yrow, ylen, lane, look, s32, t, &sim, &banded);
    if (banded) ++dc.band;
    if (keep) {
      em.add(lane, pair_key(a, (uint32_t)__builtin_amdgcn_readlane((int)y, l),
                            (uint32_t)__builtin_amdgcn_readlane((int)q, l)),
             sim);
      if (em.n == 64) em.flush(lane, a.counters, a.out_key, a.out_sim, a.cap);
    }
    wave_lds_order();
  }
}

// The same for one pair, without the staging: what a full queue leaves to the
// wave that found it (kept small: it shares that kernel's registers).
__device__ __forceinline__ void decide_one(const PairArgs& a, int lane, uint32_t x, uint32_t z, int32_t d, Decided& dc) {
  const uint32_t y = pair_y(a, x, z), q = pair_q(a, x, z);
  const float t = pair_t(a, q);
  const int64_t ys = a.rp[y], qs = a.qrp[q];
  const int ylen = (int)(a.rp[y + 1] - ys), qlen = (int)(a.qrp[q + 1] - qs);
  const RComp* yrow = a.rc + ys;
  const RComp* qrow = a.qrc + qs;
  bool rarer = false;
  auto look = [&](int32_t r) {
    const float v = row_lookup(qrow, qlen, r);
    rarer = rarer || (r > d && v != 0.0f);
    return v;
  };
  const float s32 = wave_dot2(yrow, ylen, lane, look);
  if (__ballot(rarer)) return;
  ++dc.surv;
  if (s32 >= t - kSlack) ++dc.ver;
  float sim;
  bool banded;
  const bool keep = wave_decide(yrow, ylen, lane, look, s32, t, &sim, &banded);
  if (banded) ++dc.band;
  if (keep) {
    WaveEmit em;
    em.add(lane, pair_key(a, y, q), sim);
    em.flush(lane, a.counters, a.out_key, a.out_sim, a.cap);
  }
}

// Add a workgroup's counts to the global counters, one atomic each: atomics
// of the whole device on one address take about 20 ns apiece, so one per wave
// would cost small joins more than their tests.  Called by all threads.
__device__ __forceinline__ void add_counts(const PairArgs& a, unsigned long long visits, const Decided& dc) {
  __shared__ unsigned long long sum[4];
  const int tid = (int)threadIdx.x;
  if (tid < 4) sum[tid] = 0ull;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) visits += __shfl_xor(visits, o, 64);
  __syncthreads();
  if ((tid & 63) == 0) {
    atomicAdd(&sum[0], visits);
    atomicAdd(&sum[1], dc.surv);
    atomicAdd(&sum[2], dc.ver);
    atomicAdd(&sum[3], dc.band);
  }
  __syncthreads();
  if (tid < 4 && sum[tid]) {
    const int c = tid == 0 ? C_VISITS : (tid == 1 ? C_SURVIVORS : (tid == 2 ? C_VERIFIED : C_BAND));
    atomicAdd(&a.counters[c], sum[tid]);
  }
}

// The pairs that a workgroup's waves still hold, with one reservation (see
// add_counts for what one per wave costs).  Called by all threads.
__device__ __forceinline__ void flush_all(const PairArgs& a, int lane, int wave, WaveEmit& em) {
  __shared__ unsigned int held[4];
  __shared__ unsigned long long base;
  if (lane == 0) held[wave] = (unsigned int)em.n;
  __syncthreads();
  const unsigned int total = held[0] + held[1] + held[2] + held[3];
  if (total == 0u) return;
  if (threadIdx.x == 0) base = atomicAdd(&a.counters[C_MATCHES], (unsigned long long)total);
  __syncthreads();
  int64_t k = (int64_t)base + lane;
  for (int w = 0; w < wave; ++w) k += held[w];
  if (lane < em.n && k < a.cap) {
    a.out_key[k] = em.key;
    a.out_sim[k] = em.sim;
  }
  em.n = 0;
}

// The queued survivors: consecutive ones (which share rows) to each wave, 64
// at a time, or fewer (at least 4) when there are not enough for every wave.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_decide(PairArgs a) {
  __shared__ StagedRow rows[4];
  const int lane = (int)(threadIdx.x & 63u);
  const int wave = uni((int)(threadIdx.x >> 6));
  const unsigned int queued = a.uctr[1];
  if (a.query && a.counters[C_OVERFLOW]) return;  // (the call is made by the accumulating kernel)
  const int64_t held = (int64_t)queued < a.qcap ? (int64_t)queued : a.qcap;
  const int64_t waves = (int64_t)gridDim.x * 4;
  const int64_t even = (held + waves - 1) / waves;
  // (each wave ends with atomics on the same few counters)
  const int per = even < 4 ? 4 : (even < 64 ? (int)even : 64);
  WaveEmit em;
  Decided dc;
  for (int64_t e0 = ((int64_t)blockIdx.x * 4 + wave) * per; e0 < held; e0 += waves * per) {
    const int here = held - e0 < per ? (int)(held - e0) : per;
    uint32_t x = 0u, z = 0u, d = 0u;
    if (lane < here) {
      const uint32_t* const o = a.queue + 3 * (e0 + lane);
      x = o[0];
      z = o[1];
      d = o[2];
    }
    decide_pairs(a, rows[wave], lane, here, x, z, (int)d, em, dc);
  }
  flush_all(a, lane, wave, em);
  add_counts(a, 0ull, dc);
}

// ---------------------------------------------------------------- pair tests

constexpr int kPairQueue = 512;  // survivors a wave holds before it passes them on
constexpr int kSteps = kSkGroups / 32;

// Survivors of one wave.  They go to the global queue, where all waves of
// k_decide share them evenly (they come in clusters: most tiles have none and
// a few have thousands); what does not fit there is decided at once, or for
// queries flagged (the call is then made by the accumulating kernel).
struct Survivors {
  uint32_t* a;  // LDS, kPairQueue entries each
  uint32_t* b;
  uint32_t* d;
  int n = 0;

  __device__ __forceinline__ void pass_on(const PairArgs& pa, int lane, Decided& dc) {
    if (n == 0) return;
    if (pa.sample) {  // counted only
      dc.surv += (unsigned long long)n;
      n = 0;
      return;
    }
    wave_lds_order();
    // a full queue's counter is left alone, so it stays within a few hundred
    // entries per wave of the capacity
    unsigned int at = 0;
    if (lane == 0) {
      at = __hip_atomic_load(&pa.uctr[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if ((int64_t)at < pa.qcap) at = atomicAdd(&pa.uctr[1], (unsigned int)n);
    }
    at = (unsigned int)uni((int)at);
    const int64_t room = pa.qcap - (int64_t)at;
    const int fit = room <= 0 ? 0 : (room < n ? (int)room : n);
    put(pa, lane, at, fit);
    if (pa.query) {
      if (fit < n && lane == 0) pa.counters[C_OVERFLOW] = 1ull;
      n = 0;
      wave_lds_order();
      return;
    }
    for (int e = fit; e < n; ++e)
      decide_one(pa, lane, (uint32_t)uni((int)a[e]), (uint32_t)uni((int)b[e]), uni((int)d[e]), dc);
    n = 0;
    wave_lds_order();
  }

  __device__ __forceinline__ void put(const PairArgs& pa, int lane, unsigned int at, int fit) const {
    for (int e = lane; e < fit; e += 64) {
      uint32_t* const o = pa.queue + 3 * ((int64_t)at + e);
      o[0] = a[e];
      o[1] = b[e];
      o[2] = d[e];
    }
  }

  // What the waves of a workgroup still hold, with one reservation; if that
  // does not fit, wave by wave.  Called by all threads.
  __device__ __forceinline__ void pass_on_all(const PairArgs& pa, int lane, int wave, Decided& dc) {
    __shared__ unsigned int held[4];
    __shared__ unsigned int base;
    if (lane == 0) held[wave] = (unsigned int)n;
    __syncthreads();
    const unsigned int total = held[0] + held[1] + held[2] + held[3];
    if (total == 0u) return;
    if (threadIdx.x == 0) {
      unsigned int at = 0xFFFFFFFFu;
      if (!pa.sample) {
        at = __hip_atomic_load(&pa.uctr[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        at = (int64_t)at + (int64_t)total <= pa.qcap ? atomicAdd(&pa.uctr[1], total) : 0xFFFFFFFFu;
      }
      base = at;
    }
    __syncthreads();
    unsigned int at = base;
    if (at == 0xFFFFFFFFu) {
      pass_on(pa, lane, dc);
      return;
    }
    // (others may have taken the room between the load and the reservation)
    for (int w = 0; w < wave; ++w) at += held[w];
    const int64_t room = pa.qcap - (int64_t)at;
    const int fit = room <= 0 ? 0 : (room < n ? (int)room : n);
    put(pa, lane, at, fit);
    if (fit < n) {
      if (pa.query) {
        if (lane == 0) pa.counters[C_OVERFLOW] = 1ull;
      } else {
        for (int e = fit; e < n; ++e)
          decide_one(pa, lane, (uint32_t)uni((int)a[e]), (uint32_t)uni((int)b[e]), uni((int)d[e]), dc);
      }
    }
    n = 0;
  }

  // Products of 64 rows (lane l holds the id of row l) with 32 columns (lane
  // l % 32 holds the id of its column, the rows that pair with it, `first` to
  // na - 1, and the product of a survivor).
  __device__ __forceinline__ void take(const PairArgs& pa, int lane, const i32x16 (&acc)[2], uint32_t ida, uint32_t idb,
                                       int first, int na, uint32_t rank, int thr, Decided& dc) {
    // the largest product first: most tiles have no survivor
    int mx = acc[0][0];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = mx > acc[i][r] ? mx : acc[i][r];
    if (!__ballot(mx >= thr)) return;
    uint32_t hits = 0u;  // bit 16 i + r: this lane's survivors
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) hits |= acc[i][r] >= thr ? 1u << (16 * i + r) : 0u;
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    // one survivor per lane at a time
    do {
      const int bit = hits ? __ffs((int)hits) - 1 : 0;
      const int row = 32 * (bit >> 4) + 8 * ((bit & 15) >> 2) + 4 * (lane >> 5) + (bit & 3);
      const bool hit = hits != 0u && row >= first && row < na;
      const uint64_t hm = __ballot(hit);
      if (hm) {
        const int cnt = (int)__popcll(hm);
        if (n + cnt > kPairQueue) pass_on(pa, lane, dc);
        const uint32_t idr = (uint32_t)__shfl((int)ida, row, 64);
        if (hit) {
          const int s = n + (int)__popcll(hm & lt);
          a[s] = idr;
          b[s] = idb;
          d[s] = rank;
        }
        n += cnt;
      }
      hits &= hits - 1u;
    } while (__ballot(hits != 0u));
  }
};

// The 32-group steps of lane l's part (16 of 32 groups) of a row's sketch.
__device__ __forceinline__ void load_sketch(const PairArgs& a, int lane, uint32_t row, int ksteps, i32x4 (&f)[kSteps]) {
  const uint8_t* p = a.sk + (int64_t)row * kSkGroups + 16 * (lane >> 5);
#pragma unroll
  for (int ks = 0; ks < kSteps; ++ks) f[ks] = ks < ksteps ? *reinterpret_cast<const i32x4*>(p + 32 * ks) : i32x4{0, 0, 0, 0};
}

// Groups past g hold no dimension up to the list's: their bytes count nothing.
__device__ __forceinline__ void mask_sketch(int lane, int g, i32x4 (&f)[kSteps]) {
#pragma unroll
  for (int ks = 0; ks < kSteps; ++ks)
#pragma unroll
    for (int w = 0; w < 4; ++w) f[ks][w] &= (int)group_mask(32 * ks + 16 * (lane >> 5) + 4 * w, g);
}

// Lane l of a 32 x 32 x 32 int8 MFMA holds operand row l % 32, k = 16 (l / 32)
// .. + 15; result element r of lane l is row 8 (r / 4) + 4 (l / 32) + r % 4,
// column l % 32.  A row's sketch is one 128-byte line, read whole by four
// steps of 32 groups.

// Long lists: a workgroup holds 256 entries' sketches in registers (64 per
// wave) and meets the earlier entries 64 at a time through LDS, so a gathered
// sketch is read once per 256 rows and by whole lines; a wave that gathers
// its own operands reads 32 bytes of each line at a time, and the address
// units bind (100,000 rows of mean 80 at t = 0.5: 7.3 ms).  The loads run a
// step ahead, their ids two steps.  Chunk c of column r sits at position
// c ^ (r / 2 % 8) of its LDS row, so that the 16 lanes of a 128-bit read
// phase hit 16 different bank groups.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_pairs_wide(PairArgs a) {
  __shared__ i32x4 cols[2][64 * 8];
  __shared__ uint32_t cid[2][64];
  __shared__ uint32_t qa[4][kPairQueue], qb[4][kPairQueue], qd[4][kPairQueue];
  __shared__ unsigned int next;
  const int tid = (int)threadIdx.x;
  const int lane = tid & 63;
  const int wave = uni(tid >> 6);
  Survivors sv{qa[wave], qb[wave], qd[wave]};
  Decided dc;
  unsigned long long c_visit = 0;
  for (;;) {
    __syncthreads();
    if (tid == 0) next = atomicAdd(&a.uctr[0], 1u);
    __syncthreads();
    const int64_t un = (int64_t)(unsigned int)uni((int)next) * a.every + a.first;
    if (un >= a.nwide) break;
    const uint2 u = a.wide[un];
    const int64_t base = a.doff[u.x];
    const int len = (int)(a.doff[u.x + 1] - base);
    const uint32_t* const ids = a.dl + base;
    const int g = a.gid[u.x] >> 3;  // kFineGroups / kSkGroups = 8
    const int ksteps = g / 32 + 1;
    int ablk, chunk;
    unit_at(u.y, &ablk, &chunk);
    const int blk0 = ablk * kWideRows;
    const int from = chunk * (kWideSpan * kWideRows);
    // columns [from, to): the entries before the block's last one, or the chunk's
    const int bend = blk0 + kWideRows < len ? blk0 + kWideRows : len;
    const int to = bend < from + kWideSpan * kWideRows ? bend : from + kWideSpan * kWideRows;
    const int a0 = blk0 + 64 * wave;  // this wave's rows
    const int na = len - a0 < 64 ? len - a0 : 64;  // may be <= 0
    // lanes past the list's end take its last entry (their results are not used)
    const uint32_t ida = ids[a0 + lane < len ? a0 + lane : len - 1];
    if (lane < na) c_visit += (unsigned long long)((a0 + lane < to ? a0 + lane : to) - from);
    // this thread's part of a step's columns: 32 groups of column tid / 4
    const int col = tid >> 2, part = tid & 3;
    auto id_at = [&](int b0) { return ids[b0 + col < len ? b0 + col : len - 1]; };
    i32x4 x0 = {0, 0, 0, 0}, x1 = {0, 0, 0, 0};
    auto fetch = [&](uint32_t id) {
      if (part < ksteps) {
        const i32x4* p = reinterpret_cast<const i32x4*>(a.sk + (int64_t)id * kSkGroups + 32 * part);
        x0 = p[0];
        x1 = p[1];
      }
    };
    uint32_t id0 = id_at(from), id1 = id_at(from + 64);
    fetch(id0);
    i32x4 fa[2][kSteps];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      load_sketch(a, lane, (uint32_t)__shfl((int)ida, 32 * i + (lane & 31), 64), ksteps, fa[i]);
      mask_sketch(lane, g, fa[i]);
    }
    const int s0 = col * 8 + ((2 * part) ^ ((col >> 1) & 7)), s1 = col * 8 + ((2 * part + 1) ^ ((col >> 1) & 7));
    int buf = 0;
    for (int b0 = from; b0 < to; b0 += 64, buf ^= 1) {
      cols[buf][s0] = x0;
      cols[buf][s1] = x1;
      if (part == 0) cid[buf][col] = id0;
      id0 = id1;
      if (b0 + 64 < to) {
        fetch(id0);
        id1 = id_at(b0 + 128);
      }
      // one barrier a step: a wave here has finished the step before, whose
      // buffer is written next
      __syncthreads();
      if (na > 0 && b0 < a0 + na - 1) {  // some row of the wave comes after the first column
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          i32x16 acc[2];
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][r] = 0;
          const int r0 = 32 * j + (lane & 31);
#pragma unroll
          for (int ks = 0; ks < kSteps; ++ks) {
            if (ks < ksteps) {
              const i32x4 fb = cols[buf][r0 * 8 + ((2 * ks + (lane >> 5)) ^ ((r0 >> 1) & 7))];
              acc[0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[0][ks], fb, acc[0], 0, 0, 0);
              acc[1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[1][ks], fb, acc[1], 0, 0, 0);
            }
          }
          // each pair once: the row's entry comes after the column's
          sv.take(a, lane, acc, ida, cid[buf][r0], b0 + r0 - a0 + 1, b0 + r0 < to ? na : 0, u.x, a.thr, dc);
        }
      }
    }
  }
  sv.pass_on_all(a, lane, wave, dc);
  add_counts(a, c_visit, dc);
}

// Short lists, most of them a handful of entries: one wave per block of 64
// entries, a.sstep units at a time with their bounds read together and a
// unit's ids while the unit before is tested, so that a unit costs one round
// of sketch loads.  A list of one block meets itself only, from the same
// registers.
//
// Lists of at most kTinyList entries, most of them two or three, share tiles:
// a wave takes the 64 consecutive entries from a multiple of 32 on and tests
// the lists that begin in the first half of them, each row masked to its own
// list's groups, each column meeting the later rows of its own list: 41 us for
// 3,001 rows and 97 for 20,011, where a wave per list took 61 and 217.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_pairs_short(PairArgs a) {
  __shared__ uint32_t qa[4][kPairQueue], qb[4][kPairQueue], qd[4][kPairQueue];
  const int lane = (int)(threadIdx.x & 63u);
  const int wave = uni((int)(threadIdx.x >> 6));
  Survivors sv{qa[wave], qb[wave], qd[wave]};
  Decided dc;
  unsigned long long c_visit = 0;
  static_assert(kShortUnits <= 64, "a unit per lane");
  // (units are alike, and a shared counter costs more than it evens out)
  const int64_t step = (int64_t)a.sstep * a.every;
  for (int64_t u0 = ((int64_t)blockIdx.x * 4 + wave) * step + a.first * a.sstep; u0 < a.nshort;
       u0 += (int64_t)gridDim.x * 4 * step) {
    const int cnt = a.nshort - u0 < a.sstep ? (int)(a.nshort - u0) : a.sstep;
    uint2 un = make_uint2(0u, 0u);
    uint32_t ubase = 0u;
    int ulen = 0, ug = 0;
    if (lane < cnt) {
      un = a.shorts[u0 + lane];
      ubase = (uint32_t)a.doff[un.x];  // list positions fit 32 bits
      ulen = (int)((uint32_t)a.doff[un.x + 1] - ubase);
      ug = a.gid[un.x] >> 3;
    }
    auto block_ids = [&](int l) {
      const uint32_t* ids = a.dl + (uint32_t)__builtin_amdgcn_readlane((int)ubase, l);
      const int len = __builtin_amdgcn_readlane(ulen, l);
      const int k = __builtin_amdgcn_readlane((int)un.y, l) * kUnitRows + lane;
      return ids[k < len ? k : len - 1];
    };
    uint32_t idn = block_ids(0);
    for (int l = 0; l < cnt; ++l) {
      const uint32_t ida = idn;
      if (l + 1 < cnt) idn = block_ids(l + 1);
      const uint32_t rank = (uint32_t)__builtin_amdgcn_readlane((int)un.x, l);
      const uint32_t* const ids = a.dl + (uint32_t)__builtin_amdgcn_readlane((int)ubase, l);
      const int len = __builtin_amdgcn_readlane(ulen, l);
      const int a0 = __builtin_amdgcn_readlane((int)un.y, l) * kUnitRows;
      const int g = __builtin_amdgcn_readlane(ug, l);
      const int ksteps = g / 32 + 1;
      const int na = len - a0 < kUnitRows ? len - a0 : kUnitRows;
      if (lane < na) c_visit += (unsigned long long)(a0 + lane);
      i32x4 fa[2][kSteps];
      load_sketch(a, lane, (uint32_t)__shfl((int)ida, lane & 31, 64), ksteps, fa[0]);
      if (na > 32) load_sketch(a, lane, (uint32_t)__shfl((int)ida, 32 + (lane & 31), 64), ksteps, fa[1]);
      mask_sketch(lane, g, fa[0]);
      if (na > 32) mask_sketch(lane, g, fa[1]);
      // columns before the block, then the block's own
      for (int b0 = 0; b0 < a0 + na; b0 += 32) {
        i32x4 fb[kSteps];
        uint32_t idb;
        if (b0 < a0) {
          idb = ids[b0 + (lane & 31)];
          load_sketch(a, lane, idb, ksteps, fb);
        } else {
          const int j = b0 - a0;  // 0 or 32
          idb = (uint32_t)__shfl((int)ida, j + (lane & 31), 64);
#pragma unroll
          for (int ks = 0; ks < kSteps; ++ks) fb[ks] = j ? fa[1][ks] : fa[0][ks];
        }
        i32x16 acc[2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[i][r] = 0;
#pragma unroll
        for (int ks = 0; ks < kSteps; ++ks)
          if (ks < ksteps) {
            acc[0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[0][ks], fb[ks], acc[0], 0, 0, 0);
            if (na > 32) acc[1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[1][ks], fb[ks], acc[1], 0, 0, 0);
          }
        const int bl = b0 + (lane & 31);
        sv.take(a, lane, acc, ida, idb, bl - a0 + 1, na, rank, a.thr, dc);
      }
    }
  }
  const int64_t windows = (a.ndeep + kTinyList - 1) / kTinyList;
  for (int64_t w = ((int64_t)blockIdx.x * 4 + wave) * a.every + a.first; w < windows;
       w += (int64_t)gridDim.x * 4 * a.every) {
    const int64_t e0 = w * kTinyList;
    const int64_t e = e0 + lane;
    uint32_t r = 0u, id = 0u;
    int beg = -1, end = 0, g = 0;  // of this lane's entry's list, from e0
    if (e < a.ndeep) {
      r = a.dlr[e];
      id = a.dl[e];
      const int64_t st = a.doff[r], len = a.doff[r + 1] - st;
      if (len >= 2 && len <= kTinyList && st >= e0 && st < e0 + kTinyList) {
        beg = (int)(st - e0);
        end = beg + (int)len;
        g = a.gid[r] >> 3;
        c_visit += (unsigned long long)(lane - beg);
      }
    }
    const uint64_t own = __ballot(beg >= 0);
    if (!own) continue;
    int gmax = beg >= 0 ? g : 0;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      const int v = __shfl_xor(gmax, o, 64);
      gmax = v > gmax ? v : gmax;
    }
    const int ksteps = uni(gmax) / 32 + 1;
    const bool upper = (own >> 32) != 0ull;
    i32x4 fa[2][kSteps];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int row = 32 * i + (lane & 31);
      const uint32_t rid = (uint32_t)__shfl((int)id, row, 64);
      if ((own >> row) & 1ull) {
        load_sketch(a, lane, rid, ksteps, fa[i]);
      } else {
#pragma unroll
        for (int ks = 0; ks < kSteps; ++ks) fa[i][ks] = i32x4{0, 0, 0, 0};
      }
      mask_sketch(lane, __shfl(g, row, 64), fa[i]);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if (j == 1 && !upper) break;
      i32x16 acc[2];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int k = 0; k < 16; ++k) acc[i][k] = 0;
#pragma unroll
      for (int ks = 0; ks < kSteps; ++ks)
        if (ks < ksteps) {
          if (j == 0) acc[0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[0][ks], fa[0][ks], acc[0], 0, 0, 0);
          if (upper) acc[1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[1][ks], fa[j][ks], acc[1], 0, 0, 0);
        }
      const int col = 32 * j + (lane & 31);
      sv.take(a, lane, acc, id, (uint32_t)__shfl((int)id, col, 64), col + 1, __shfl(end, col, 64),
              (uint32_t)__shfl((int)r, col, 64), a.thr, dc);
    }
  }
  sv.pass_on_all(a, lane, wave, dc);
  add_counts(a, c_visit, dc);
}

// ---------------------------------------------------------------- queries

// Query rows against the whole corpus by the sketch bound over all groups: a
// product of n x 256 with 256 x nq bytes, every pair tested.  A workgroup
// holds 256 corpus rows' sketches in registers (64 per wave) and meets the
// queries 64 at a time through LDS (laid out as in k_pairs_wide, a step
// ahead), so the corpus sketches are read once, in order, by the workgroups
// that fit the device, each for several blocks of rows (their last survivors
// cost an atomic each: one per wave of 1,954 workgroups was 150 of 184 us for
// 64 queries over 500,000 rows); a few queries are
// bound by that (128 MB for 500,000 rows), thousands by the matrix cores:
// 4,096 queries over 1,000,000 rows take 1.29 ms (1.6e15 operations a
// second), with the exact count 3.1 ms and the decisions 0.8 ms where the
// accumulating kernel took 15 ms.  256 groups where a self-join's lists have
// 128: no list narrows the pairs here.
// Once the survivors have outgrown their queue the rest of the rows is left
// out: thread 0 reads the flag with each block's sketches and passes it on at
// the block's end, when it has long arrived; all threads follow it at the end
// of the next block, whose barriers lie between (two words in turn, so that
// nobody still reads the one that is written).  Batches of a few steps are over
// too soon for it (64 queries: 41 us, and 43 with the reads).
// SAMPLE: every a.every-th workgroup only, counting the pairs that reach
// each of kRateBins thresholds, evenly between s.t and 1.
constexpr int kMidSteps = kMidGroups / 32;

template <bool SAMPLE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_query_screen(PairArgs a, QueryArgs s) {
  __shared__ i32x4 cols[2][64 * 16];
  constexpr int kHeld = SAMPLE ? 1 : kPairQueue;
  __shared__ uint32_t qa[4][kHeld], qb[4][kHeld], qd[4][kHeld];
  __shared__ unsigned int bins[kRateBins];
  __shared__ unsigned int full[2];
  const int tid = (int)threadIdx.x;
  const int lane = tid & 63;
  const int wave = uni(tid >> 6);
  Survivors sv{qa[wave], qb[wave], qd[wave]};
  Decided dc;
  if (SAMPLE && tid < kRateBins) bins[tid] = 0u;
  if (tid == 0) full[1] = 0u;
  // this thread's part of a step's columns: 64 groups of column tid / 4
  const int col = tid >> 2, part = tid & 3;
  i32x4 x[4];
  auto fetch = [&](int64_t b0) {
    int64_t q = b0 + col;
    if (q >= s.nq) q = s.nq - 1;
    const i32x4* p = reinterpret_cast<const i32x4*>(s.qsk + q * s.qstride * kMidGroups + 64 * part);
#pragma unroll
    for (int c = 0; c < 4; ++c) x[c] = p[c];
  };
  // chunk c of column r at position c ^ (r % 16) of its row
  auto at = [](int r, int c) { return r * 16 + (c ^ (r & 15)); };
  const int64_t step = (int64_t)gridDim.x * kWideRows * (SAMPLE ? a.every : 1);
  const bool watch = !SAMPLE && s.nq - s.q0 > 512;
  int buf = 0, turn = 0;
  for (int64_t block0 = (int64_t)blockIdx.x * kWideRows * (SAMPLE ? a.every : 1); block0 < s.n;
       block0 += step, turn ^= 1) {
    unsigned long long flag = 0ull;
    if (watch && tid == 0)
      flag = __hip_atomic_load(&a.counters[C_OVERFLOW], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int64_t row0 = block0 + 64 * wave;
    const int na = s.n - row0 < 64 ? (int)(s.n - row0) : 64;  // may be <= 0
    i32x4 fa[2][kMidSteps];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      int64_t r = row0 + 32 * i + (lane & 31);
      if (r >= s.n) r = s.n - 1;  // (results of rows past the end are not used)
      const uint8_t* p = s.sk + r * kMidGroups + 16 * (lane >> 5);
#pragma unroll
      for (int ks = 0; ks < kMidSteps; ++ks) fa[i][ks] = *reinterpret_cast<const i32x4*>(p + 32 * ks);
    }
    fetch(s.q0);
    for (int64_t b0 = s.q0; b0 < s.nq; b0 += 64, buf ^= 1) {
#pragma unroll
      for (int c = 0; c < 4; ++c) cols[buf][at(col, 4 * part + c)] = x[c];
      if (b0 + 64 < s.nq) fetch(b0 + 64);
      __syncthreads();
      if (na > 0) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          if (b0 + 32 * j >= s.nq) break;
          const int r0 = 32 * j + (lane & 31);
          const int64_t q = b0 + r0;
          const int thr = q < s.nq ? pair_threshold(s.qt ? s.qt[q] : s.t) : 0x7FFFFFFF;
          i32x16 acc[2];
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][r] = 0;
#pragma unroll
          for (int ks = 0; ks < kMidSteps; ++ks) {
            const i32x4 fb = cols[buf][at(r0, 2 * ks + (lane >> 5))];
            acc[0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[0][ks], fb, acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[1][ks], fb, acc[1], 0, 0, 0);
          }
          if (SAMPLE) {
            const float per_bin = (float)kRateBins / (float)(pair_threshold(1.0f) - pair_threshold(s.t) + 1);
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
              for (int r = 0; r < 16; ++r)
                if (acc[i][r] >= thr && 32 * i + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3) < na) {
                  const int bin = (int)((float)(acc[i][r] - thr) * per_bin);
                  atomicAdd(&bins[bin < kRateBins ? bin : kRateBins - 1], 1u);
                }
          } else {
            sv.take(a, lane, acc, (uint32_t)(row0 + lane), (uint32_t)q, 0, na, 0x7FFFFFFFu, thr, dc);
          }
        }
      }
    }
    if (watch) {
      if (full[turn ^ 1]) break;
      if (tid == 0) full[turn] = flag != 0ull ? 1u : 0u;
    }
  }
  if (SAMPLE) {
    __syncthreads();
    if (tid < kRateBins && bins[tid]) atomicAdd(&a.counters[tid], (unsigned long long)bins[tid]);
  } else {
    sv.pass_on_all(a, lane, wave, dc);
  }
}

// ---------------------------------------------------------------- candidates

// Bitmaps of the dense ranks, one wave per (block, rank): the rows of the
// block in the rank's list.
__global__ __launch_bounds__(256) void k_bitmaps(const Post* __restrict__ post, const uint32_t* __restrict__ hoff,
                                                 int32_t H, int32_t cb, int64_t nb, int32_t HB, int64_t nblk,
                                                 uint32_t* __restrict__ bm) {
  __shared__ uint32_t words[4][kCountWords];
  const int lane = (int)(threadIdx.x & 63u);
  uint32_t* const w = words[threadIdx.x >> 6];
  const int64_t step = kCountRows / cb;
  const int64_t total = nblk * (int64_t)HB;
  for (int64_t e = (int64_t)blockIdx.x * 4 + (int64_t)(threadIdx.x >> 6); e < total; e += (int64_t)gridDim.x * 4) {
    const int64_t b = e / HB;
    const int64_t r = e - b * HB;
    const int64_t b1 = (b + 1) * step < nb ? (b + 1) * step : nb;
    const uint32_t p0 = hoff[b * step * (int64_t)H + r], p1 = hoff[b1 * (int64_t)H + r];
#pragma unroll
    for (int j = 0; j < kCountWords / 64; ++j) w[lane + 64 * j] = 0u;
    wave_lds_order();
    for (uint32_t p = p0 + lane; p < p1; p += 64) {
      const uint32_t yl = post[p].y - (uint32_t)(b * kCountRows);
      atomicOr(&w[yl >> 5], 1u << (yl & 31u));
    }
    wave_lds_order();
#pragma unroll
    for (int j = 0; j < kCountWords / 64; ++j) bm[e * kCountWords + lane + 64 * j] = w[lane + 64 * j];
    wave_lds_order();
  }
}

// Which of the ranks >= H have an entry in each block: one bit per (block,
// rank), lists by lane.
__global__ void k_present(const int64_t* __restrict__ off, const Post* __restrict__ post, int32_t H, int64_t m,
                          int64_t words, uint32_t* __restrict__ present) {
  for (int64_t r = H + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < m; r += (int64_t)gridDim.x * blockDim.x) {
    const int64_t e = off[r + 1];
    int64_t last = -1;
    for (int64_t k = off[r]; k < e; ++k) {
      const int64_t b = (int64_t)post[k].y / kCountRows;
      if (b != last) atomicOr(&present[b * words + ((r - H) >> 5)], 1u << ((r - H) & 31));
      last = b;
    }
  }
}

// Segment {first entry, end} of every rank < H in each block, side by side.
__global__ void k_segments(const uint32_t* __restrict__ hoff, int32_t H, int32_t cb, int64_t nb, int64_t nblk,
                           uint2* __restrict__ seg) {
  const int64_t step = kCountRows / cb;
  const int64_t total = nblk * (int64_t)H;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t b = e / H;
    const int64_t r = e - b * H;
    const int64_t b1 = (b + 1) * step < nb ? (b + 1) * step : nb;
    const uint32_t p = hoff[b * step * (int64_t)H + r];
    seg[e] = make_uint2(p, hoff[b1 * (int64_t)H + r]);
  }
}

// Candidates of one (block of 4,096 corpus rows, chunk of queries): a wave
// takes a query at a time and forms the union of its dimensions' lists over
// the block, 64 rows in each lane: bitmaps of the densest ranks from LDS, of
// the next ones from L2, and the entries of the sparse lists by lane.  What
// binds is reading bitmaps and lines through the L1, whose address units are
// busy 80% of the time (500,000 rows of mean 120: 64 ms, of which the bitmaps
// alone, with the rest taken out, were 54).  A block's
// bitmaps, list entries and offsets fit an XCD's L2, except the offsets of
// the ranks >= H (8 bytes of every one of them): one bit per (block, rank)
// says which have an entry there at all, about a fifth of a query's.  A
// query's components are loaded while the query before it is processed, its
// list offsets while the LDS bitmaps are read, and its first list entries
// while the L2 bitmaps are, with two workgroups of 16 waves per CU.  Longer
// spans of rows for the sparse ranks read fewer lines but miss the L2 (16,384
// rows: 138 ms, 65,536 rows: 209 ms), and the sparse ranks by whole lists,
// through a buffer of bits, take longer by themselves (100 ms).
constexpr int kCountWaves = 16;
constexpr int kChunks = 3;   // 64-component chunks of a row in registers
constexpr int kEntries = 4;  // list entries loaded ahead per component
constexpr int kNoRank = 0x7FFFFFFF;
constexpr int64_t kSpreadBlocks = 16;

// List entries as row offsets in the block: from the packed copy (ids modulo
// 2^16) where a segment spans fewer rows than that, else from the ids.
template <bool PACKED>
__device__ __forceinline__ uint32_t entry_row(const CountArgs& a, uint32_t p, uint32_t row0) {
  if constexpr (PACKED) return (a.post4[p] - row0) & 0xFFFFu;
  else return a.post[p].y - row0;
}

// The kEntries entries from p on that lie before pe (packed: four in one
// load, whose reads past the last list its padding covers).
template <bool PACKED>
__device__ __forceinline__ void entry_rows(const CountArgs& a, uint32_t p, uint32_t pe, uint32_t row0,
                                           uint32_t (&y)[kEntries]) {
  static_assert(kEntries == 4, "one 16-byte load");
#pragma unroll
  for (int u = 0; u < kEntries; ++u) y[u] = 0xFFFFFFFFu;
  if (p >= pe) return;
  if constexpr (PACKED) {
    uint32_t w[kEntries];
    __builtin_memcpy(w, a.post4 + p, sizeof(w));
#pragma unroll
    for (int u = 0; u < kEntries; ++u)
      if (p + u < pe) y[u] = (w[u] - row0) & 0xFFFFu;
  } else {
#pragma unroll
    for (int u = 0; u < kEntries; ++u)
      if (p + u < pe) y[u] = entry_row<PACKED>(a, p + u, row0);
  }
}

// Block and chunk of a workgroup: those of an XCD (round-robin over blockIdx)
// take whole blocks; few blocks are spread over all of them.
__device__ __forceinline__ void count_item(const CountArgs& a, int64_t nchunk, int64_t* b, int64_t* j) {
  *j = (int64_t)(blockIdx.x >> 3);
  if (a.nblk < kSpreadBlocks) {
    *b = (int64_t)blockIdx.x % a.nblk;
    *j = (int64_t)blockIdx.x / a.nblk;
  } else {
    *b = (int64_t)(blockIdx.x & 7u) + 8 * (*j / nchunk);
    *j %= nchunk;
  }
}

template <bool PACKED>
__global__ __launch_bounds__(64 * kCountWaves) __attribute__((amdgpu_waves_per_eu(8))) void k_count(CountArgs a,
                                                                                                   int64_t nchunk) {
  __shared__ uint2 tile[kLdsRanks * kCountWords / 2];
  __shared__ uint32_t spare[kCountWaves][kCountWords];
  const int tid = (int)threadIdx.x;
  const int lane = tid & 63;
  const int wave = uni(tid >> 6);
  int64_t b, j;
  count_item(a, nchunk, &b, &j);
  if (b >= a.nblk) return;
  // (a batch of queries that outgrew its queue is not counted; read with the first loads)
  const unsigned long long flag = a.triangle ? 0ull : a.counters[C_OVERFLOW];
  const int64_t row0 = b * kCountRows;
  const int64_t qbeg = j * a.chunk;
  const int64_t qend = qbeg + a.chunk < a.nq ? qbeg + a.chunk : a.nq;
  int64_t q0 = qbeg;
  if (a.triangle && q0 <= row0) q0 = row0 + 1;
  if (q0 >= qend) return;
  const int hl = a.HB < a.lds_ranks ? a.HB : a.lds_ranks;
  const uint32_t* const bmb = a.bm + b * (int64_t)a.HB * kCountWords;
  {
    const uint4* src = reinterpret_cast<const uint4*>(bmb);
    uint4* dst = reinterpret_cast<uint4*>(tile);
    for (int e = tid; e < hl * kCountWords / 4; e += 64 * kCountWaves) dst[e] = src[e];
  }
  uint32_t* const sp = spare[wave];
  sp[2 * lane] = 0u;
  sp[2 * lane + 1] = 0u;
  if (flag) return;
  __syncthreads();

  const uint2* const seg = a.seg + b * (int64_t)a.H;
  const int64_t rg0 = row0 / a.rr;
  int64_t rg1 = (row0 + kCountRows + a.rr - 1) / a.rr;
  if (rg1 > a.nR) rg1 = a.nR;
  const uint32_t* const t0 = a.toff + rg0 * (int64_t)a.m_tail;
  const uint32_t* const t1 = a.toff + rg1 * (int64_t)a.m_tail;
  const uint32_t* const present = a.present + b * a.present_words;
  const uint2* const bm2 = reinterpret_cast<const uint2*>(bmb) + lane;
  const uint2* const tl = tile + lane;
  const int H = a.H, HB = a.HB;

  uint32_t cand = 0;
  int64_t q = q0 + wave;
  const bool busy = q < qend;
  if (!busy) q = q0;  // (a query to load: nothing of it is counted)
  // row bounds two queries ahead, components one query ahead
  auto start = [&](int64_t k) { return a.rp[k] + (a.skip ? (int64_t)a.skip[k].cut : 0); };
  int64_t s = start(q);
  int len = (int)(a.rp[q + 1] - s);
  int64_t qn = q + kCountWaves < qend ? q + kCountWaves : q;
  int64_t sn = start(qn);
  int lenn = (int)(a.rp[qn + 1] - sn);
  int lenq = len;
  int rn[kChunks];
#pragma unroll
  for (int c = 0; c < kChunks; ++c) rn[c] = 64 * c + lane < len ? a.rc[s + 64 * c + lane].r : kNoRank;
  while (busy) {
    uint2 v = make_uint2(0u, 0u);
    bool any = false;
    int r[kChunks];
#pragma unroll
    for (int c = 0; c < kChunks; ++c) r[c] = rn[c];
    for (int k0 = 0;;) {
      // offsets of the sparse lists, one component per lane
      uint32_t p[kChunks], pe[kChunks], pw[kChunks];
#pragma unroll
      for (int c = 0; c < kChunks; ++c) {
        p[c] = pe[c] = pw[c] = 0u;
        if (r[c] >= H && r[c] != kNoRank) {
          pw[c] = present[(r[c] - H) >> 5];
        } else if (r[c] >= HB && r[c] != kNoRank) {
          const uint2 g = seg[r[c]];
          p[c] = g.x;
          pe[c] = g.y;
        }
      }
      const bool last = k0 + 64 * kChunks >= len;
      if (last) {
        // the next query's components, and the bounds of the one after it
#pragma unroll
        for (int c = 0; c < kChunks; ++c) rn[c] = 64 * c + lane < lenn ? a.rc[sn + 64 * c + lane].r : kNoRank;
        s = sn;
        lenq = lenn;
        qn = qn + kCountWaves < qend ? qn + kCountWaves : qn;
        sn = start(qn);
        lenn = (int)(a.rp[qn + 1] - sn);
      }
      // ranks ascend, so each kind is a run of lanes
#pragma unroll
      for (int c = 0; c < kChunks; ++c) {
        const int n1 = (int)__popcll(__ballot(r[c] < hl));
        int k = 0;
        for (; k + 4 <= n1; k += 4) {
          uint2 x[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) x[u] = tl[__builtin_amdgcn_readlane(r[c], k + u) * (kCountWords / 2)];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            v.x |= x[u].x;
            v.y |= x[u].y;
          }
        }
        for (; k < n1; ++k) {
          const uint2 x = tl[__builtin_amdgcn_readlane(r[c], k) * (kCountWords / 2)];
          v.x |= x.x;
          v.y |= x.y;
        }
      }
#pragma unroll
      for (int c = 0; c < kChunks; ++c)
        if (r[c] >= H && r[c] != kNoRank && ((pw[c] >> ((r[c] - H) & 31)) & 1u)) {
          p[c] = t0[r[c] - H];
          pe[c] = t1[r[c] - H];
        }
      // this lane's first entries of each sparse list
      uint32_t yl[kChunks][kEntries];
#pragma unroll
      for (int c = 0; c < kChunks; ++c)
        entry_rows<PACKED>(a, p[c], pe[c], (uint32_t)row0, yl[c]);
#pragma unroll
      for (int c = 0; c < kChunks; ++c) {
        const int n1 = (int)__popcll(__ballot(r[c] < hl));
        const int n2 = (int)__popcll(__ballot(r[c] < HB));
        int k = n1;
        for (; k + 4 <= n2; k += 4) {
          uint2 x[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) x[u] = bm2[__builtin_amdgcn_readlane(r[c], k + u) * (kCountWords / 2)];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            v.x |= x[u].x;
            v.y |= x[u].y;
          }
        }
        for (; k < n2; ++k) {
          const uint2 x = bm2[__builtin_amdgcn_readlane(r[c], k) * (kCountWords / 2)];
          v.x |= x.x;
          v.y |= x.y;
        }
      }
#pragma unroll
      for (int c = 0; c < kChunks; ++c) {
        any = any || __ballot(p[c] < pe[c]) != 0ull;
#pragma unroll
        for (int u = 0; u < kEntries; ++u)
          if (yl[c][u] < (uint32_t)kCountRows) atomicOr(&sp[yl[c][u] >> 5], 1u << (yl[c][u] & 31u));
        for (uint32_t e = p[c] + kEntries; e < pe[c]; e += kEntries) {
          uint32_t y[kEntries];
          entry_rows<PACKED>(a, e, pe[c], (uint32_t)row0, y);
#pragma unroll
          for (int u = 0; u < kEntries; ++u)
            if (y[u] < (uint32_t)kCountRows) atomicOr(&sp[y[u] >> 5], 1u << (y[u] & 31u));
        }
      }
      if (last) break;
      k0 += 64 * kChunks;
#pragma unroll
      for (int c = 0; c < kChunks; ++c) r[c] = k0 + 64 * c + lane < len ? a.rc[s + k0 + 64 * c + lane].r : kNoRank;
    }
    if (any) {
      wave_lds_order();
      v.x |= sp[2 * lane];
      v.y |= sp[2 * lane + 1];
      wave_lds_order();
      sp[2 * lane] = 0u;
      sp[2 * lane + 1] = 0u;
      wave_lds_order();
    }
    if (a.triangle && q < row0 + kCountRows) {
      // rows before q only: q - row0 of the block's rows
      const int lim = (int)(q - row0) - 64 * lane;  // rows of this lane's 64
      const uint64_t mask = lim <= 0 ? 0ull : (lim >= 64 ? ~0ull : (1ull << lim) - 1ull);
      v.x &= (uint32_t)mask;
      v.y &= (uint32_t)(mask >> 32);
    }
    cand += (uint32_t)__popc(v.x) + (uint32_t)__popc(v.y);
    q += kCountWaves;
    if (q >= qend) break;
    len = lenq;  // s and rn hold this query's row already
  }
  // one atomic per workgroup
  unsigned long long c = cand;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) c += __shfl_xor(c, o, 64);
  __syncthreads();
  unsigned long long* const total = reinterpret_cast<unsigned long long*>(tile);
  if (tid == 0) *total = 0ull;
  __syncthreads();
  if (lane == 0 && c) atomicAdd(total, c);
  __syncthreads();
  if (tid == 0 && *total) atomicAdd(&a.counters[C_CANDIDATES], *total);
}

// The same count for few rows (a chunk has one query per wave, and no bitmaps
// go to LDS): what binds there is the longest row of a workgroup, whose
// bitmaps a wave reads at some 20 ns a component.  So the rows' components
// are cut into pieces of 64, the waves take them in turn, and the unions meet
// in LDS; eight bitmaps are loaded at once, since few waves run.
// Device time of a captured self-join's replay with it, and with a wave for
// each row: 3,001 rows of mean 80 (up to 2,000) 86 us and 116, 4,000 of mean
// 120 106 and 170, 8,960 of 10 to 60 components even; the call takes some 17 us
// more.  64 queries of 500,000 rows, the call: 187 us and 199.
template <bool PACKED>
__global__ __launch_bounds__(64 * kCountWaves) void k_count_pieces(CountArgs a, int64_t nchunk) {
  __shared__ uint32_t bits[kCountWaves][kCountWords];
  __shared__ unsigned long long total;
  const int tid = (int)threadIdx.x;
  const int lane = tid & 63;
  const int wave = uni(tid >> 6);
  int64_t b, j;
  count_item(a, nchunk, &b, &j);
  if (b >= a.nblk) return;
  // (a batch of queries that outgrew its queue is not counted; read with the first loads)
  const unsigned long long flag = a.triangle ? 0ull : a.counters[C_OVERFLOW];
  const int64_t row0 = b * kCountRows;
  int64_t q0 = j * a.chunk;
  const int64_t qend = q0 + a.chunk < a.nq ? q0 + a.chunk : a.nq;
  if (a.triangle && q0 <= row0) q0 = row0 + 1;
  if (q0 >= qend) return;
  uint32_t* const own = bits[wave];
  own[2 * lane] = 0u;
  own[2 * lane + 1] = 0u;
  if (tid == 0) total = 0ull;
  // lane i: the i-th query's components, and the pieces up to and with it
  int64_t s = 0;
  int len = 0;
  if (lane < kCountWaves && q0 + lane < qend) {
    s = a.rp[q0 + lane] + (a.skip ? (int64_t)a.skip[q0 + lane].cut : 0);
    len = (int)(a.rp[q0 + lane + 1] - s);
  }
  if (flag) return;
  const int own_pieces = (len + 63) >> 6;
  int upto = own_pieces;
#pragma unroll
  for (int o = 1; o < kCountWaves; o <<= 1) {
    const int x = __shfl_up(upto, o, 64);
    if (lane >= o) upto += x;
  }
  const int pieces = __builtin_amdgcn_readlane(upto, kCountWaves - 1);
  const uint32_t* const bmb = a.bm + b * (int64_t)a.HB * kCountWords;
  const uint2* const bm2 = reinterpret_cast<const uint2*>(bmb) + lane;
  const uint2* const seg = a.seg + b * (int64_t)a.H;
  const int64_t rg0 = row0 / a.rr;
  int64_t rg1 = (row0 + kCountRows + a.rr - 1) / a.rr;
  if (rg1 > a.nR) rg1 = a.nR;
  const uint32_t* const t0 = a.toff + rg0 * (int64_t)a.m_tail;
  const uint32_t* const t1 = a.toff + rg1 * (int64_t)a.m_tail;
  const uint32_t* const present = a.present + b * a.present_words;
  __syncthreads();

  for (int t = wave; t < pieces; t += kCountWaves) {
    const int i = (int)__popcll(__ballot(lane < kCountWaves && upto <= t));
    const int k = 64 * (t - __builtin_amdgcn_readlane(upto - own_pieces, i)) + lane;
    const int64_t si = __shfl(s, i, 64);  // (from a lane that has to be active)
    const int r = k < __builtin_amdgcn_readlane(len, i) ? a.rc[si + k].r : kNoRank;
    uint32_t p = 0u, pe = 0u;
    if (r >= a.H && r != kNoRank) {
      if ((present[(r - a.H) >> 5] >> ((r - a.H) & 31)) & 1u) {
        p = t0[r - a.H];
        pe = t1[r - a.H];
      }
    } else if (r >= a.HB && r != kNoRank) {
      const uint2 g = seg[r];
      p = g.x;
      pe = g.y;
    }
    uint32_t y[kEntries];
    entry_rows<PACKED>(a, p, pe, (uint32_t)row0, y);
    // ranks ascend: the bitmaps' are the first lanes (one read twice changes nothing)
    uint2 v = make_uint2(0u, 0u);
    const int n = (int)__popcll(__ballot(r < a.HB));
    for (int c = 0; c < n; c += 8) {
      uint2 x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        x[u] = bm2[__builtin_amdgcn_readlane(r, c + u < n ? c + u : n - 1) * (kCountWords / 2)];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        v.x |= x[u].x;
        v.y |= x[u].y;
      }
    }
    uint32_t* const to = bits[i];
    if (v.x) atomicOr(&to[2 * lane], v.x);
    if (v.y) atomicOr(&to[2 * lane + 1], v.y);
    while (true) {
#pragma unroll
      for (int u = 0; u < kEntries; ++u)
        if (y[u] < (uint32_t)kCountRows) atomicOr(&to[y[u] >> 5], 1u << (y[u] & 31u));
      if (p >= pe || pe - p <= (uint32_t)kEntries) break;
      p += kEntries;
      entry_rows<PACKED>(a, p, pe, (uint32_t)row0, y);
    }
  }
  __syncthreads();
  const int64_t q = q0 + wave;
  unsigned long long c = 0ull;
  if (q < qend) {
    uint64_t v = (uint64_t)own[2 * lane] | ((uint64_t)own[2 * lane + 1] << 32);
    if (a.triangle && q < row0 + kCountRows) {
      const int lim = (int)(q - row0) - 64 * lane;  // rows of this lane's 64 before q
      v &= lim <= 0 ? 0ull : (lim >= 64 ? ~0ull : (1ull << lim) - 1ull);
    }
    c = (unsigned long long)__popcll(v);
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) c += __shfl_xor(c, o, 64);
  if (lane == 0 && c) atomicAdd(&total, c);
  __syncthreads();
  if (tid == 0 && total) atomicAdd(&a.counters[C_CANDIDATES], total);
}

// The same count where every list is sparse (the head-cut index of the
// screened join): a workgroup takes a query at a time and sets one bit per
// corpus row of its lists, in LDS over kCountSpan rows at once, so a list is
// one run of memory with nothing to look up per block (200,000 rows of mean
// 150 less the 4,096 densest dimensions: 10.5 ms by blocks, 3.35 ms so).  A wave takes every
// eighth list, four at a time.
constexpr int kSpanWaves = 8;

__global__ __launch_bounds__(64 * kSpanWaves) void k_count_sparse(CountArgs a, int32_t words) {
  extern __shared__ uint4 span4[];
  uint32_t* const bits = reinterpret_cast<uint32_t*>(span4);
  __shared__ unsigned long long total;
  const int tid = (int)threadIdx.x;
  const int lane = tid & 63;
  const int wave = uni(tid >> 6);
  if (tid == 0) total = 0ull;
  for (int w = tid; w < words / 4; w += 64 * kSpanWaves) span4[w] = make_uint4(0u, 0u, 0u, 0u);
  uint32_t cand = 0;
  for (int64_t q = blockIdx.x; q < a.nq; q += gridDim.x) {
    const int64_t s = a.rp[q] + (a.skip ? (int64_t)a.skip[q].cut : 0);
    const int len = (int)(a.rp[q + 1] - s);
    const int64_t rows = a.triangle ? q : a.n;  // the query meets the rows before this one
    for (int64_t row0 = 0; row0 < rows; row0 += kCountSpan) {
      const uint32_t lim = (uint32_t)(rows - row0 < kCountSpan ? rows - row0 : kCountSpan);
      __syncthreads();
      for (int k0 = 0; k0 < len; k0 += 64 * kSpanWaves) {
        // lane l's list of this wave
        const int k = k0 + wave + kSpanWaves * lane;
        uint32_t p = 0u, pe = 0u;
        if (k < len) {
          const int32_t r = a.rc[s + k].r;
          p = (uint32_t)a.off[r];  // list positions fit 32 bits
          pe = (uint32_t)a.off[r + 1];
          if (row0 > 0) {
            uint32_t lo = p, hi = pe;
            while (lo < hi) {
              const uint32_t mid = (lo + hi) >> 1;
              if ((int64_t)a.post[mid].y < row0) lo = mid + 1;
              else hi = mid;
            }
            p = lo;
          }
        }
        uint64_t m = __ballot(p < pe);
        while (m) {
          uint32_t e[4], f[4];
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const int l = m ? __ffsll((unsigned long long)m) - 1 : 0;
            e[g] = (uint32_t)__builtin_amdgcn_readlane((int)p, l) + lane;
            f[g] = m ? (uint32_t)__builtin_amdgcn_readlane((int)pe, l) : 0u;
            m &= m - 1;
          }
          bool more = true;
          while (more) {
            uint32_t y[4][2];
#pragma unroll
            for (int g = 0; g < 4; ++g)
#pragma unroll
              for (int u = 0; u < 2; ++u)
                y[g][u] = e[g] + 64 * u < f[g] ? a.post[e[g] + 64 * u].y - (uint32_t)row0 : 0xFFFFFFFFu;
            more = false;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
#pragma unroll
              for (int u = 0; u < 2; ++u)
                if (y[g][u] < lim) atomicOr(&bits[y[g][u] >> 5], 1u << (y[g][u] & 31u));
              // ids ascend: a list is done once they leave the rows met
              e[g] += 128;
              if (y[g][1] >= lim) e[g] = f[g];
              more = more || e[g] < f[g];
            }
            more = __ballot(more) != 0ull;
          }
        }
      }
      __syncthreads();
      const int nw = (int)((lim + 127u) / 128u);
      for (int w = tid; w < nw; w += 64 * kSpanWaves) {
        const uint4 v = span4[w];
        span4[w] = make_uint4(0u, 0u, 0u, 0u);
        cand += (uint32_t)(__popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w));
      }
    }
  }
  unsigned long long c = cand;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) c += __shfl_xor(c, o, 64);
  __syncthreads();
  if (lane == 0 && c) atomicAdd(&total, c);
  __syncthreads();
  if (tid == 0 && total) atomicAdd(&a.counters[C_CANDIDATES], total);
}

unsigned grid1d(int64_t n) {
  int64_t g = (n + 255) / 256;
  return (unsigned)(g < 1 ? 1 : g < 32768 ? g : 32768);
}

unsigned row_grid(int64_t n) {
  const int64_t g = (n + 3) / 4;
  return (unsigned)(g < 1 ? 1 : g < 8192 ? g : 8192);
}

}  // namespace

hipError_t launch_groups(const int64_t* cum, const uint32_t* cnt_r, int64_t m, int64_t nnz, uint16_t* gid, hipStream_t s) {
  if (m <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_groups, dim3(grid1d(m)), dim3(256), 0, s, cum, cnt_r, m, nnz, gid);
  return hipGetLastError();
}

hipError_t launch_visits(const uint32_t* cnt_r, const int64_t* off, int64_t m, int64_t hb, unsigned long long* out,
                         hipStream_t s) {
  if (m <= 0) return hipSuccess;
  const unsigned g = grid1d(m);
  hipLaunchKernelGGL(k_visits, dim3(g < 256 ? g : 256), dim3(256), 0, s, cnt_r, off, m, hb, out);
  return hipGetLastError();
}

hipError_t launch_norm_codes(const uint8_t* pn8, int64_t n, unsigned long long* hist, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const unsigned g = grid1d(n);
  hipLaunchKernelGGL(k_norm_codes, dim3(g < 256 ? g : 256), dim3(256), 0, s, pn8, n, hist);
  return hipGetLastError();
}

hipError_t launch_widen(const uint32_t* in, int64_t n, int64_t* out, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_widen, dim3(grid1d(n)), dim3(256), 0, s, in, n, out);
  return hipGetLastError();
}

hipError_t launch_sketch(const int64_t* rp, const RComp* rc, const uint16_t* gid, int64_t n, uint8_t* sk,
                         uint8_t* mid, unsigned int* nfine, uint32_t* fidx, uint8_t* fsk, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_sketch, dim3(row_grid(n)), dim3(256), 0, s, rp, rc, gid, n, sk, mid, nfine, fidx, fsk);
  return hipGetLastError();
}

hipError_t launch_unit_counts(const int64_t* doff, int64_t m, bool wide, int64_t* ucnt, hipStream_t s) {
  if (m <= 0) return hipSuccess;
  if (wide) hipLaunchKernelGGL(k_unit_counts<true>, dim3(grid1d(m)), dim3(256), 0, s, doff, m, ucnt);
  else hipLaunchKernelGGL(k_unit_counts<false>, dim3(grid1d(m)), dim3(256), 0, s, doff, m, ucnt);
  return hipGetLastError();
}

hipError_t launch_unit_fill(const int64_t* doff, const int64_t* uoff, int64_t m, bool wide, uint2* units, hipStream_t s) {
  if (m <= 0) return hipSuccess;
  if (wide) hipLaunchKernelGGL(k_unit_fill<true>, dim3(grid1d(m)), dim3(256), 0, s, doff, uoff, m, units);
  else hipLaunchKernelGGL(k_unit_fill<false>, dim3(grid1d(m)), dim3(256), 0, s, doff, uoff, m, units);
  return hipGetLastError();
}

hipError_t launch_bitmaps(const Post* post, const uint32_t* hoff, int32_t H, int32_t cb, int64_t nb, int32_t HB,
                          int64_t nblk, uint32_t* bm, hipStream_t s) {
  if (nblk <= 0 || HB <= 0) return hipSuccess;
  if (HB > H || cb <= 0 || kCountRows % cb) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_bitmaps, dim3(row_grid(nblk * HB)), dim3(256), 0, s, post, hoff, H, cb, nb, HB, nblk, bm);
  return hipGetLastError();
}

PairGroups pairs_resident_groups() {
  int dev = 0, cus = 0;
  (void)hipGetDevice(&dev);
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) cus = 1;
  auto resident = [&](const void* f) {
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, f, 256, 0) != hipSuccess || per_cu < 1) per_cu = 1;
    return per_cu * cus;
  };
  PairGroups g;
  g.wide = resident(reinterpret_cast<const void*>(&k_pairs_wide));
  g.shorts = resident(reinterpret_cast<const void*>(&k_pairs_short));
  g.screen = resident(reinterpret_cast<const void*>(&k_query_screen<false>));
  g.decide = resident(reinterpret_cast<const void*>(&k_decide));
  return g;
}

hipError_t launch_pairs(PairArgs a, const PairGroups& g, hipStream_t s) {
  if (a.ndeep <= 0) return hipSuccess;
  if (!a.dlr || !a.rp || !a.rc || !a.sk || !a.gid || !a.fidx || !a.fsk || !a.qrp || !a.qrc || !a.qfidx || !a.qfsk ||
      !a.dl || !a.doff || !a.wide || !a.shorts || !a.uctr || !a.counters || (a.qcap > 0 && !a.queue) ||
      a.nwide > kMaxUnits || a.nshort > kMaxUnits)
    return hipErrorInvalidValue;
  if (a.sample ? a.every < 1 || a.first != 0 : !a.out_key || !a.out_sim || a.turns < 1) return hipErrorInvalidValue;
  hipError_t e = hipSuccess;
  if (!a.sample) a.every = a.turns;
  const int64_t every = a.every, turns = a.sample ? 1 : a.turns;
  const int64_t wide = (a.nwide + every - 1) / every;
  // every resident wave gets some units, where there are enough
  const int64_t windows = (a.ndeep + kTinyList - 1) / kTinyList;
  const int64_t even = a.nshort / every / ((int64_t)g.shorts * 4);
  a.sstep = (int32_t)(even < 1 ? 1 : (even < kShortUnits ? even : kShortUnits));
  const int64_t steps = std::max((a.nshort + a.sstep * every - 1) / (a.sstep * every), (windows + every - 1) / every);
  // (a workgroup ends with atomics on the same counters, 20 ns each: one
  // step per wave only as far as 256 of them, then four)
  const int64_t need = std::max((steps + 15) / 16, std::min<int64_t>((steps + 3) / 4, 256));
  for (int64_t turn = 0; turn < turns; ++turn) {
    if (!a.sample) a.first = turn;
    if (turn > 0 && (e = fill_u32(a.uctr, 0u, 2, s)) != hipSuccess) return e;
    if (wide > 0) {
      hipLaunchKernelGGL(k_pairs_wide, dim3((unsigned)(wide < g.wide ? wide : g.wide)), dim3(256), 0, s, a);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_pairs_short, dim3((unsigned)(need < g.shorts ? need : g.shorts)), dim3(256), 0, s, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (a.qcap > 0 && !a.sample) {
      hipLaunchKernelGGL(k_decide, dim3((unsigned)g.decide), dim3(256), 0, s, a);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    }
  }
  return e;
}

hipError_t launch_query_screen(const PairArgs& a, const QueryArgs& q, const PairGroups& g, hipStream_t s) {
  if (q.n <= 0 || q.nq <= q.q0) return hipSuccess;
  if (!q.sk || !q.qsk || q.q0 < 0 || q.qstride <= 0 || !a.uctr || !a.counters || a.qcap <= 0 || !a.queue || !a.rp ||
      !a.rc || !a.qrp || !a.qrc || !a.fidx || !a.fsk || !a.qfidx || !a.qfsk || !a.out_key || !a.out_sim || !a.query)
    return hipErrorInvalidValue;
  const int64_t blocks = (q.n + kWideRows - 1) / kWideRows;
  hipLaunchKernelGGL(k_query_screen<false>, dim3((unsigned)(blocks < g.screen ? blocks : g.screen)), dim3(256), 0, s, a, q);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_decide, dim3((unsigned)g.decide), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_query_sample(const PairArgs& a, const QueryArgs& q, hipStream_t s) {
  if (q.n <= 0 || q.nq <= 0) return hipSuccess;
  if (!q.sk || !q.qsk || q.q0 != 0 || q.qstride <= 0 || q.qt || a.every < 1 || !a.counters) return hipErrorInvalidValue;
  const int64_t every = kWideRows * a.every;
  const int64_t grid = (q.n + every - 1) / every;
  if (grid > 0x7FFFFFFF) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_query_screen<true>, dim3((unsigned)grid), dim3(256), 0, s, a, q);
  return hipGetLastError();
}

hipError_t launch_segments(const uint32_t* hoff, int32_t H, int32_t cb, int64_t nb, int64_t nblk, uint2* seg,
                           hipStream_t s) {
  if (nblk <= 0 || H <= 0) return hipSuccess;
  if (cb <= 0 || kCountRows % cb) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_segments, dim3(grid1d(nblk * H)), dim3(256), 0, s, hoff, H, cb, nb, nblk, seg);
  return hipGetLastError();
}

hipError_t launch_present(const int64_t* off, const Post* post, int32_t H, int64_t m, int64_t words, uint32_t* present,
                          hipStream_t s) {
  if (m <= H) return hipSuccess;
  hipLaunchKernelGGL(k_present, dim3(grid1d(m - H)), dim3(256), 0, s, off, post, H, m, words, present);
  return hipGetLastError();
}

hipError_t launch_count(const CountArgs& a, hipStream_t s) {
  if (a.nq <= 0 || a.n <= 0) return hipSuccess;
  if (!a.rp || !a.rc || !a.bm || !a.present || !a.post || !a.post4 || !a.seg || !a.toff || !a.counters || a.chunk <= 0 ||
      a.rr <= 0 || a.HB > a.H || a.lds_ranks < 0 || a.lds_ranks > kLdsRanks)
    return hipErrorInvalidValue;
  if (a.HB == 0) {
    if (!a.off) return hipErrorInvalidValue;
    const int64_t rows = a.n < kCountSpan ? a.n : kCountSpan;
    const int32_t words = (int32_t)((rows + 127) / 128 * 4);
    int dev = 0, cus = 0, per_cu = 0;
    (void)hipGetDevice(&dev);
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) cus = 1;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(&k_count_sparse),
                                                     64 * kSpanWaves, (size_t)words * 4) != hipSuccess ||
        per_cu < 1)
      per_cu = 1;
    const int64_t g = (int64_t)per_cu * cus < a.nq ? (int64_t)per_cu * cus : a.nq;
    hipLaunchKernelGGL(k_count_sparse, dim3((unsigned)g), dim3(64 * kSpanWaves), (size_t)words * 4, s, a, words);
    return hipGetLastError();
  }
  const int64_t nchunk = (a.nq + a.chunk - 1) / a.chunk;
  const int64_t grid = (a.nblk < kSpreadBlocks ? a.nblk : 8 * ((a.nblk + 7) / 8)) * nchunk;
  if (grid > 0x7FFFFFFF) return hipErrorInvalidValue;
  // a segment spans at most the ranges that meet a block
  const bool packed = kCountRows + 2 * a.rr <= 65536;
  static_assert(kPieceRows == kCountWaves, "a query per wave");
  const bool pieces = a.chunk <= kPieceRows && a.lds_ranks == 0;
  if (pieces && packed)
    hipLaunchKernelGGL(k_count_pieces<true>, dim3((unsigned)grid), dim3(64 * kCountWaves), 0, s, a, nchunk);
  else if (pieces)
    hipLaunchKernelGGL(k_count_pieces<false>, dim3((unsigned)grid), dim3(64 * kCountWaves), 0, s, a, nchunk);
  else if (packed)
    hipLaunchKernelGGL(k_count<true>, dim3((unsigned)grid), dim3(64 * kCountWaves), 0, s, a, nchunk);
  else
    hipLaunchKernelGGL(k_count<false>, dim3((unsigned)grid), dim3(64 * kCountWaves), 0, s, a, nchunk);
  return hipGetLastError();
}

}  // namespace apss
