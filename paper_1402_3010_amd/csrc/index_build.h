// Launchers of the index builder kernels (index_build.hip).
#pragma once

#include "apss_internal.h"

namespace apss {

enum ErrBits : uint32_t {
  ERR_ROWPTR = 1u,   // row_ptr not monotone or not spanning [0, nnz]
  ERR_DIM = 2u,      // dimension id outside [0, m)
  ERR_WEIGHT = 4u,   // weight not finite or not > 0
  ERR_NORM = 8u,     // |norm - 1| above tolerance
  ERR_DUP = 16u,     // repeated dimension inside a row
};

// longest (may be NULL): *longest = max(*longest, longest row)
hipError_t launch_check_rowptr(const int64_t* rp, int64_t n, int64_t nnz, uint32_t* err, unsigned long long* bad,
                               unsigned long long* longest, hipStream_t s);
// also counts every dimension's components and takes its largest weight (cnt and mwbits zeroed before)
hipError_t launch_validate_count(const int64_t* rp, const int32_t* col, const float* val, int64_t n, int64_t m,
                                 double tol, uint32_t* cnt, uint32_t* mwbits, uint32_t* err, unsigned long long* bad,
                                 hipStream_t s);
// Rows in rank space for rows of at most kLongRow components (longest: the
// longest one).  nlong: one zeroed counter; longs: room for the rows longer
// than kWaveRow, at most nnz / kWaveRow.
constexpr int kWaveRow = 512;
constexpr int kLongRow = 8192;
hipError_t launch_sort_rows(const int64_t* rp, const int32_t* col, const float* val, const int32_t* rank, int64_t n,
                            int64_t longest, RComp* rc, uint32_t* err, unsigned int* nlong, uint32_t* longs,
                            hipStream_t s);
hipError_t launch_dim_keys(const uint32_t* cnt, int64_t m, int64_t n, int dbits, uint64_t* keys, uint64_t* vals,
                           hipStream_t s);
hipError_t launch_rank_from_sorted(const uint64_t* vals, int64_t m, const uint32_t* cnt, const uint32_t* mwbits,
                                   int32_t* rank, float* mw_r, uint32_t* cnt_r, hipStream_t s);
hipError_t launch_row_keys(const int64_t* rp, const int32_t* col, const float* val, const int32_t* rank, int64_t n,
                           int rbits, uint64_t* keys, uint32_t* vals, hipStream_t s);
hipError_t launch_unpack_rows(const uint64_t* keys, const uint32_t* vals, int64_t nnz, int rbits, RComp* rc,
                              uint32_t* err, hipStream_t s);
// head >= 0: the unindexed part of every row is its components of rank < head (t and l2 unused;
// head = 0 indexes every component); head < 0: the running-bound cutoff at t.
// *pmax = max over rows of rs[r].pnrm as float bits (atomicMax; zeroed before); pn8[r]: its byte code
hipError_t launch_cutoff(const int64_t* rp, const RComp* rc, const float* mw_r, int64_t n, float t, int l2,
                         int32_t head, RowStat* rs, float* xmw, int64_t* nidx, uint32_t* pmax, uint8_t* pn8,
                         hipStream_t s);
// lim >= 0: mark (sign bit of the weight) the components up to which the row's squared norm is at least lim
hipError_t launch_emit_indexed(const int64_t* rp, const RComp* rc, const RowStat* rs, const int64_t* ibase, int64_t n,
                               double lim, uint64_t* keys, uint64_t* vals, hipStream_t s);
// off[r] = first position of the sorted keys[0, P) that is >= r, r = 0..m
hipError_t launch_list_offsets(const uint64_t* keys, int64_t P, int64_t m, int64_t* off, hipStream_t s);
// Lists from the sorted values: entries and their packed copy; with dl, the
// marked entries' ids and ranks (tiles: exclusive scan of launch_count_deep's
// list_tiles(P) counts) and the marked entries before each position
int64_t list_tiles(int64_t P);
hipError_t launch_count_deep(const uint64_t* vals, int64_t P, int64_t* tiles, hipStream_t s);
hipError_t launch_lists(const uint64_t* keys, const uint64_t* vals, int64_t P, Post* post, uint32_t* post4,
                        const int64_t* tiles, uint32_t* pos, uint32_t* dl, uint32_t* dlr, hipStream_t s);
hipError_t launch_deep_offsets(const int64_t* off, const uint32_t* pos, int64_t P, int64_t m, int64_t deep,
                               int64_t* doff, hipStream_t s);
hipError_t launch_block_offsets(const int64_t* off, const Post* post, int32_t H, int64_t nb, int32_t CB,
                                uint32_t* hoff, hipStream_t s);
// mw[d] = maxweight of dimension d, cut[i] = unindexed components of row i (either may be NULL)
hipError_t launch_export(const int32_t* rank, const float* mw_r, int64_t m, const RowStat* rs, int64_t n, float* mw,
                         int32_t* cut, hipStream_t s);
// Query rows of at most kQueryRow components (longest: the longest one) in rank
// space.  err and bad are set up before; the rest is optional (NULL, 0).
constexpr int kQueryRow = 4096;
struct QueryRowsArgs {
  const int64_t* rp;
  const int32_t* col;
  const float* val;
  const float* t;
  const int32_t* rank;
  int64_t nq, m;
  double tol;
  RComp* rc;
  float* qmw;
  int64_t* rp_out;  // copy of rp
  float* t_out;     // copy of t
  unsigned long long* zero;  // cleared
  int32_t zeros;
  uint32_t* err;
  unsigned long long* bad;
};
hipError_t launch_query_rows(const QueryRowsArgs& a, int64_t longest, hipStream_t s);
// The same for any rows, as keys (row, rank) to be sorted
hipError_t launch_query_keys(const int64_t* rp, const int32_t* col, const float* val, const int32_t* rank, int64_t nq,
                             int64_t m, int rbits, double tol, uint64_t* keys, uint32_t* vals, float* qmw,
                             uint32_t* err, unsigned long long* bad, hipStream_t s);

}  // namespace apss
