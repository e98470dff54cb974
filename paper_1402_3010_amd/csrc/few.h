// Launcher of the kernel for queries that come few at a time (few.hip).
#pragma once

#include "apss_internal.h"

namespace apss {

struct FewArgs {
  const int64_t* rp;  // corpus rows
  const RComp* rc;
  const RowStat* rs;
  const uint8_t* pn8;
  int64_t n;
  const Post* post;
  const uint32_t* hoff;   // [(nb+1) * H] first entry of a dense list in each block of cb rows
  int32_t H;
  int32_t cb;             // divides kFewRows, or is that
  int64_t nb;
  const uint32_t* toff;   // [(nR+1) * m_tail] first entry of a sparse list in each range of rr rows
  int64_t m_tail, rr, nR; // rr is a multiple of kFewRows
  const int64_t* qrp;     // query rows
  const RComp* qrc;
  const float* qmw;       // largest weight
  const float* qt;        // [nq] thresholds, or NULL: t
  float t;
  int64_t nq;
  int bj;
  uint64_t* out_key;      // query << bj | row
  float* out_sim;
  int64_t cap;
  unsigned long long* counters;
};

// Rows of one workgroup.
constexpr int kFewRows = 2048;

hipError_t launch_few(const FewArgs& a, hipStream_t s);

}  // namespace apss
