// Queries that come a few at a time: one workgroup per query and 2,048 rows.
//
// The join kernel gives a tile of queries a range of 16,384 rows, which it
// meets block by block: one query over 500,000 rows is 31 workgroups that
// each wait for 16 blocks' lists in turn (115 us).  Here a query's lists are
// cut into 245 parts that are all in flight at once (30 us); nothing is
// shared between queries, which is why larger batches go elsewhere.
#include "few.h"
#include "rescore.h"

namespace apss {

namespace {

constexpr int kThreads = 512;
constexpr int kFewQuery = 1024;  // components of a query looked up in LDS
// accumulator units of a score: sums stay below 2^30 (1 + 1e-5) plus one unit
// per component
constexpr float kUnits = 1073741824.0f;

__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }

// q's weight in rank r by binary search of its rank-ordered row (0 if absent)
__device__ __forceinline__ float weight_of(const RComp* q, int qlen, int32_t r) {
  int lo = 0, hi = qlen;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (q[mid].r < r) lo = mid + 1;
    else hi = mid;
  }
  return (lo < qlen && q[lo].r == r) ? q[lo].w : 0.0f;
}

// A thread looks up one component's list segment; then the threads share the
// entries of all segments evenly (an entry's component by bisection in the
// running lengths, in LDS).  Sparse lists are entered at their range of
// 16,384 rows and filtered: dense ranks are the 32,768 most frequent ones,
// so a sparse list has a few entries there.  Every term is rounded up by at
// least one unit, so a row is a candidate if and only if its accumulator is
// not zero, and the sums are upper bounds in whichever order they are made.
// Bounds and decisions are those of the join kernel.
__global__ __launch_bounds__(kThreads) void k_few(FewArgs a) {
  __shared__ uint32_t acc[kFewRows];
  __shared__ uint32_t from[kThreads], before[kThreads + 1], wsum[kThreads / 64];
  __shared__ float weight[kThreads];
  __shared__ RComp qrow[kFewQuery];
  __shared__ uint16_t survivors[kFewRows];
  __shared__ unsigned int nsurv;
  __shared__ unsigned int sums[4];
  const int tid = (int)threadIdx.x;
  const int lane = tid & 63;
  const int wave = uni(tid >> 6);
  const int64_t nblk = (a.n + kFewRows - 1) / kFewRows;
  const int64_t q = (int64_t)blockIdx.x / nblk;
  const int64_t row0 = ((int64_t)blockIdx.x - q * nblk) * kFewRows;
  const int rows = a.n - row0 < kFewRows ? (int)(a.n - row0) : kFewRows;
  const int64_t qs = a.qrp[q];
  const int qlen = (int)(a.qrp[q + 1] - qs);
  const RComp* const qg = a.qrc + qs;
  for (int e = tid; e < kFewRows; e += kThreads) acc[e] = 0u;
  if (tid == 0) nsurv = 0u;
  if (tid < 4) sums[tid] = 0u;
  const int64_t b0 = row0 / a.cb;
  int64_t b1 = (row0 + kFewRows) / a.cb;
  if (b1 > a.nb) b1 = a.nb;
  const int64_t R = row0 / a.rr;
  unsigned int visits = 0u;
  for (int k0 = 0; k0 < qlen; k0 += kThreads) {
    const int k = k0 + tid;
    uint32_t p0 = 0u, p1 = 0u;
    float w = 0.0f;
    if (k < qlen) {
      const RComp c = qg[k];
      w = c.w;
      if (k < kFewQuery) qrow[k] = c;
      if (c.r < a.H) {
        p0 = a.hoff[b0 * (int64_t)a.H + c.r];
        p1 = a.hoff[b1 * (int64_t)a.H + c.r];
      } else {
        p0 = a.toff[R * a.m_tail + (c.r - a.H)];
        p1 = a.toff[(R + 1) * a.m_tail + (c.r - a.H)];
      }
    }
    // running lengths
    uint32_t sum = p1 - p0;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t v = (uint32_t)__shfl_up((int)sum, o, 64);
      if (lane >= o) sum += v;
    }
    if (lane == 63) wsum[wave] = sum;
    __syncthreads();
    uint32_t base = 0u;
    for (int v = 0; v < wave; ++v) base += wsum[v];
    from[tid] = p0;
    weight[tid] = w * kUnits;
    before[tid + 1] = base + sum;
    if (tid == 0) before[0] = 0u;
    __syncthreads();
    const uint32_t total = before[kThreads];
    for (uint32_t e = (uint32_t)tid; e < total; e += kThreads) {
      int lo = 0, hi = kThreads;  // last component with before[lo] <= e
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (before[mid] <= e) lo = mid;
        else hi = mid;
      }
      const Post p = a.post[from[lo] + (e - before[lo])];
      const int64_t y = (int64_t)p.y - row0;
      if (y >= 0 && y < rows) {
        ++visits;
        atomicAdd(&acc[y], (uint32_t)(p.w * weight[lo]) + 1u);
      }
    }
    __syncthreads();
  }
  if (qlen == 0) return;
  // candidates and their bounds
  const float t = a.qt ? a.qt[q] : a.t;
  const float thr = (t - kSlack) * kUnits, qm = a.qmw[q] * kUnits, qn = 1.0001f * kUnits;
  const float qsum = (float)qlen * qm;
  unsigned int cand = 0u;
  for (int y = tid; y < rows; y += kThreads) {
    const uint32_t v = acc[y];
    if (v == 0u) continue;
    ++cand;
    const float A = (float)v + 256.0f;
    const uint8_t code = a.pn8[row0 + y];
    if (code != kPn8None && A + qn * ((float)code * (1.0f / 254.0f)) < thr) continue;
    const RowStat st = a.rs[row0 + y];
    const float u = (float)st.cut * qm;
    if ((float)st.len * qm >= thr && A + (u < qsum ? u : qsum) * st.pmw >= thr && A + qn * st.pnrm >= thr)
      survivors[atomicAdd(&nsurv, 1u)] = (uint16_t)y;
  }
  __syncthreads();
  const int ns = (int)nsurv;
  const bool staged = qlen <= kFewQuery;
  unsigned int ver = 0u, band = 0u;
  WaveEmit em;
  for (int s = wave; s < ns; s += kThreads / 64) {
    const int64_t y = row0 + uni((int)survivors[s]);
    const int64_t ys = a.rp[y];
    const int ylen = (int)(a.rp[y + 1] - ys);
    const RComp* const yrow = a.rc + ys;
    auto look = [&](int32_t r) { return staged ? weight_of(qrow, qlen, r) : weight_of(qg, qlen, r); };
    const float s32 = wave_dot2(yrow, ylen, lane, look);
    if (s32 >= t - kSlack) ++ver;
    float sim;
    bool banded;
    const bool keep = wave_decide(yrow, ylen, lane, look, s32, t, &sim, &banded);
    if (banded) ++band;
    if (keep) {
      em.add(lane, ((uint64_t)q << a.bj) | (uint64_t)y, sim);
      if (em.n == 64) em.flush(lane, a.counters, a.out_key, a.out_sim, a.cap);
    }
  }
  em.flush(lane, a.counters, a.out_key, a.out_sim, a.cap);
  // the workgroup's counts, one atomic each
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    visits += __shfl_xor(visits, o, 64);
    cand += __shfl_xor(cand, o, 64);
  }
  if (lane == 0) {
    atomicAdd(&sums[0], visits);
    atomicAdd(&sums[1], cand);
    atomicAdd(&sums[2], ver);
    atomicAdd(&sums[3], band);
  }
  __syncthreads();
  if (tid < 4 && sums[tid]) {
    const int c = tid == 0 ? C_VISITS : (tid == 1 ? C_CANDIDATES : (tid == 2 ? C_VERIFIED : C_BAND));
    atomicAdd(&a.counters[c], (unsigned long long)sums[tid]);
  }
  if (tid == 4 && ns) atomicAdd(&a.counters[C_SURVIVORS], (unsigned long long)ns);
}

}  // namespace

hipError_t launch_few(const FewArgs& a, hipStream_t s) {
  if (a.n <= 0 || a.nq <= 0) return hipSuccess;
  if (!a.rp || !a.rc || !a.rs || !a.pn8 || !a.post || !a.hoff || !a.toff || !a.qrp || !a.qrc || !a.qmw || !a.out_key ||
      !a.out_sim || !a.counters || a.cb <= 0 || kFewRows % a.cb != 0 || a.rr <= 0 || a.rr % kFewRows != 0)
    return hipErrorInvalidValue;
  const int64_t grid = (a.n + kFewRows - 1) / kFewRows * a.nq;
  if (grid > 0x7FFFFFFF) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_few, dim3((unsigned)grid), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

}  // namespace apss
