// End of a call with few pairs: sort, unpack and hand over in one launch.
//
// A small call is bound by its launches and waits: counters to the host,
// a wait, a sort, an unpacking kernel, another wait (and a copy for host
// results) were 60 us of the 190 of a self-join of 2,000 rows.  Here the
// kernel that follows the join reads the number of pairs on the device and
// writes the result where it goes -- device arrays, or pinned host memory
// directly -- along with the counters, so that one wait ends the call.
#include "finish.h"

namespace apss {

namespace {

constexpr int kOwn = 64;     // pairs a workgroup places
constexpr int kWaves = 16;

// Each of a workgroup's 64 pairs is placed by the number of smaller keys,
// which its 16 waves count over shares of all keys, 64 at a time out of a
// register that readlane broadcasts from: no barriers and no passes over
// memory, n^2 compares of the whole device.  With NARROW keys (below 2^32)
// 1,500 pairs take 5 us, 7,000 12 and 21,000 64, where a one-workgroup bitonic
// sort of 8,192 took 75 for its 91 barriers and four radix passes take 150;
// both are even at some 32,000.
template <bool NARROW>
__global__ __launch_bounds__(64 * kWaves) void k_finish(FinishArgs a) {
  __shared__ uint32_t place[kOwn];
  const int tid = (int)threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  if (blockIdx.x == 0 && tid < C_NUM) a.host[tid] = a.counters[tid];
  if (blockIdx.x == 0 && tid >= C_NUM && tid < C_NUM + 2) a.host[tid] = a.checks ? a.checks[tid - C_NUM] : 0ull;
  // (three words in one wait)
  const unsigned long long matches = a.counters[C_MATCHES], full = a.counters[C_OVERFLOW];
  const uint32_t failed = (uint32_t)*(a.checks ? a.checks : a.counters + C_OVERFLOW);
  if (matches > (unsigned long long)kFinishPairs || matches > (unsigned long long)a.cap ||
      matches > (unsigned long long)a.room || ((uint32_t)full | failed) != 0u)
    return;
  const int n = (int)matches;
  const int own = (int)blockIdx.x * kOwn + lane;
  if ((int)blockIdx.x * kOwn >= n) return;
  if (tid < kOwn) place[tid] = 0u;
  __syncthreads();
  const uint64_t key = own < n ? a.key[own] : 0ull;
  uint32_t less = 0u;
  for (int c = wave * 64; c < n; c += kWaves * 64) {
    const uint64_t other = c + lane < n ? a.key[c + lane] : ~0ull;  // (above every key)
    const int lo = (int)(uint32_t)other, hi = (int)(uint32_t)(other >> 32);
#pragma unroll
    for (int l = 0; l < 64; ++l) {
      const uint32_t kl = (uint32_t)__builtin_amdgcn_readlane(lo, l);
      if constexpr (NARROW) {
        less += kl < (uint32_t)key ? 1u : 0u;
      } else {
        const uint64_t k = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane(hi, l) << 32) | (uint64_t)kl;
        less += k < key ? 1u : 0u;
      }
    }
  }
  if (less) atomicAdd(&place[lane], less);
  __syncthreads();
  if (wave == 0 && own < n) {
    const uint32_t p = place[lane];
    a.out_i[p] = (uint32_t)(key >> a.bj);
    a.out_j[p] = (uint32_t)(key & ((1ull << a.bj) - 1));
    a.out_sim[p] = a.sim[own];
  }
}

}  // namespace

hipError_t launch_finish(const FinishArgs& a, hipStream_t s) {
  if (!a.key || !a.sim || a.cap < 0 || a.room < 0 || !a.counters || !a.host || a.bj < 0 || a.bj > 63 || a.bits < 0 ||
      (a.room > 0 && (!a.out_i || !a.out_j || !a.out_sim)))
    return hipErrorInvalidValue;
  const int64_t most = a.room < a.cap ? a.room : a.cap;
  const int64_t grid = ((most < kFinishPairs ? most : kFinishPairs) + kOwn - 1) / kOwn;
  if (a.bits <= 32)
    hipLaunchKernelGGL(k_finish<true>, dim3((unsigned)(grid < 1 ? 1 : grid)), dim3(64 * kWaves), 0, s, a);
  else
    hipLaunchKernelGGL(k_finish<false>, dim3((unsigned)(grid < 1 ? 1 : grid)), dim3(64 * kWaves), 0, s, a);
  return hipGetLastError();
}

}  // namespace apss
