// Launchers of the list-pair join (pairs.hip): the self-join by pairs of
// list entries under a row-sketch bound, and the exact candidate count.
#pragma once

#include "apss_internal.h"

namespace apss {

// A row's sketch: its norm in each of kSkGroups groups of consecutive ranks,
// in units of 1 / kSkScale rounded up (at most 127 for rows of norm up to
// 1.0079; validated norms are within 1e-5 of 1).
constexpr int kSkGroups = 128;
constexpr double kSkScale = 126.0;
// the sketch that queries are tested with (halves of those groups)
constexpr int kMidGroups = 256;
// rows longer than kFineRow also have a sketch of kFineGroups groups
constexpr int kFineGroups = 1024;
constexpr int kFineRow = 256;
// Work units of the pair tests: lists of at least kWideList entries by
// workgroups, in blocks of kWideRows entries against at most kWideSpan blocks
// at a time; shorter lists by waves, in blocks of kUnitRows entries, which a
// wave takes up to kShortUnits at a time; lists of at most kTinyList entries
// several to a tile.
constexpr int kWideList = 256;
constexpr int kWideRows = 256;
constexpr int kWideSpan = 16;
constexpr int kUnitRows = 64;
constexpr int kTinyList = 32;
constexpr int kShortUnits = 16;
// Longest row that the decision of a pair looks up in LDS.
constexpr int kStageRanks = 2048;
constexpr int64_t kMaxUnits = 0x7FFFFFFF;  // of either kind
// The candidate count: corpus rows per block, and the densest ranks with a
// bitmap per block (one bit per row whose indexed part holds the rank).
constexpr int kCountRows = 4096;
// rows whose bits a workgroup holds in LDS when there are no dense lists
// (just under 64 KB)
constexpr int kCountSpan = 516096;
// (as many as leave room for two workgroups of k_count on a compute unit: 128
// are 76.6 and 5.05 ms for a join of 500,000 rows and 4,096 queries, 144 are
// 75.4 and 4.95)
constexpr int kLdsRanks = 144;
constexpr int kCountWords = kCountRows / 32;
constexpr int kCountRanks = 2048;
// queries of a work item that counts them by pieces (one per wave)
constexpr int64_t kPieceRows = 16;

struct PairArgs {
  const int64_t* rp;      // [n+1] row offsets of the rank-space rows
  const RComp* rc;        // components, densest dimension first
  const uint8_t* sk;      // [n * kSkGroups] sketches
  const uint16_t* gid;    // [m] fine group of each rank (its group: an eighth of that)
  const uint32_t* fidx;   // [n] index of the row's fine sketch (long rows only)
  const uint8_t* fsk;     // fine sketches
  // the rows of the pairs' second ids: the same rows in a self-join, or the
  // query rows (query = 1: pairs are a corpus row and a query)
  int32_t query;
  const int64_t* qrp;
  const RComp* qrc;
  const uint32_t* qfidx;
  const uint8_t* qfsk;
  const float* qt;        // [nq] per-query threshold, or NULL: t
  const uint32_t* dl;     // deep lists: vector ids, by rank, ascending within a rank
  const int64_t* doff;    // [m+1] first entry of each rank's deep list
  const uint32_t* dlr;    // [ndeep] the entries' ranks
  int64_t ndeep;
  const uint2* wide;      // [nwide] (rank, unit of its list)
  const uint2* shorts;    // [nshort]
  int64_t nwide, nshort;
  int32_t sample;         // 1: just count the visits and survivors of units 0, every, 2 every, ...
  int64_t turns;          // times that the queue is filled and decided, each with the units of one turn
  int64_t every, first;   // wide units, groups of short units and windows first, first + every, ...
                          // (of a join set from turns by its launcher)
  int32_t sstep;          // short units a wave takes at a time (at most kShortUnits)
  unsigned int* uctr;     // [2] next wide unit, queued survivors (zero at launch)
  uint32_t* queue;        // [3 * qcap] survivors to decide: two row ids and the list's rank
  int64_t qcap;
  float t;
  int32_t thr;            // least sketch product of a pair that can reach t
  int32_t bj;
  uint64_t* out_key;      // [cap] (i << bj) | j
  float* out_sim;         // [cap]
  int64_t cap;
  unsigned long long* counters;  // [C_NUM]
};

// Query rows tested against every corpus row.
struct QueryArgs {
  const uint8_t* sk;   // [n * kMidGroups] corpus sketches
  int64_t n;
  const uint8_t* qsk;  // query q's sketch at row q * qstride
  int64_t q0, nq, qstride;  // queries q0 .. nq - 1
  const float* qt;     // [nq] thresholds, or NULL: t
  float t;
};

// Exact number of (query, earlier corpus row) pairs that share a dimension of
// the row's indexed part.
struct CountArgs {
  const int64_t* rp;      // [n+1] query rows in rank space
  const RComp* rc;
  const RowStat* skip;    // [nq] or NULL: the first skip[q].cut components of query q have no lists
  int64_t nq;
  int32_t triangle;       // 1: query q meets corpus rows y < q only
  const uint32_t* bm;     // [nblk * HB * kCountWords] bitmaps of ranks below HB
  int32_t HB;             // 0: every list is sparse
  const int64_t* off;     // [m+1] list offsets by rank
  int64_t n;              // corpus rows
  int64_t nblk;           // blocks of kCountRows corpus rows
  const Post* post;       // list entries
  const uint32_t* post4;  // their packed copy
  const uint2* seg;       // [nblk * H] {first entry, end} of list r < H in block b
  int32_t H;
  const uint32_t* toff;   // [(nR+1) * m_tail] first entry of list H + rt at or after range R of rr rows
  int32_t m_tail;
  int64_t rr, nR;
  const uint32_t* present;  // [nblk * present_words] bit r - H of a block: rank r >= H has an entry there
  int64_t present_words;
  int64_t chunk;          // queries per work item
  int32_t lds_ranks;      // densest ranks whose bitmaps go through LDS (at most kLdsRanks)
  unsigned long long* counters;
};

// Least sketch product of a pair that can reach t: a pair with sim >= t has a
// product of at least t * kSkScale^2; the 1e-3 covers the rounding of that
// many times over.  At least 1, the product of rows that share a group: rows
// without components (whose first one is not to be read) survive at no t.
__host__ __device__ inline int32_t pair_threshold(float t) {
  const double v = (double)t * kSkScale * kSkScale - 1e-3;
  const int32_t k = (int32_t)v;
  const int32_t up = (double)k < v ? k + 1 : k;
  return up < 1 ? 1 : up;
}

// gid[r] from the cumulative component counts by rank (exclusive scan cum[m], total nnz)
hipError_t launch_groups(const int64_t* cum, const uint32_t* cnt_r, int64_t m, int64_t nnz, uint16_t* gid, hipStream_t s);
// out[0] (zeroed before) = list entries an accumulating self-join visits, out[1] = those of ranks >= hb
hipError_t launch_visits(const uint32_t* cnt_r, const int64_t* off, int64_t m, int64_t hb, unsigned long long* out,
                         hipStream_t s);
// hist[c] (zeroed before, 256 words) = rows whose unindexed part's norm has byte code c
hipError_t launch_norm_codes(const uint8_t* pn8, int64_t n, unsigned long long* hist, hipStream_t s);
hipError_t launch_widen(const uint32_t* in, int64_t n, int64_t* out, hipStream_t s);
// sk (may be NULL), mid and fine sketches of n rows; nfine: a zeroed counter;
// fsk: room for every row longer than kFineRow
hipError_t launch_sketch(const int64_t* rp, const RComp* rc, const uint16_t* gid, int64_t n, uint8_t* sk,
                         uint8_t* mid, unsigned int* nfine, uint32_t* fidx, uint8_t* fsk, hipStream_t s);
// units per rank of its deep list, as int64 for the scan, and the units
hipError_t launch_unit_counts(const int64_t* doff, int64_t m, bool wide, int64_t* ucnt, hipStream_t s);
hipError_t launch_unit_fill(const int64_t* doff, const int64_t* uoff, int64_t m, bool wide, uint2* units, hipStream_t s);
hipError_t launch_bitmaps(const Post* post, const uint32_t* hoff, int32_t H, int32_t cb, int64_t nb, int32_t HB,
                          int64_t nblk, uint32_t* bm, hipStream_t s);
// Workgroups of the kernels that fit on the device at once.
struct PairGroups {
  int wide = 0, shorts = 0, screen = 0, decide = 0;
};
PairGroups pairs_resident_groups();
// The pair tests, then the queued survivors' decisions, a.turns times (uctr is
// cleared between them).  Survivors past a.qcap are decided by the wave that finds them, so any
// capacity (0 too) gives the whole result; but one at a time and from memory,
// some fifty times slower: hence the turns.  (a.sstep is set here.)
hipError_t launch_pairs(PairArgs a, const PairGroups& g, hipStream_t s);
// Thresholds that a sample of the sketch products is counted at.
constexpr int kRateBins = 32;
// a.counters[k] += pairs with a product in the k-th of kRateBins equal parts
// of the range from q.t to 1, over every a.every-th 256 rows
hipError_t launch_query_sample(const PairArgs& a, const QueryArgs& q, hipStream_t s);
// Queries against the corpus (a.query = 1), then the survivors' decisions.
hipError_t launch_query_screen(const PairArgs& a, const QueryArgs& q, const PairGroups& g, hipStream_t s);
hipError_t launch_segments(const uint32_t* hoff, int32_t H, int32_t cb, int64_t nb, int64_t nblk, uint2* seg,
                           hipStream_t s);
// present must be zero before
hipError_t launch_present(const int64_t* off, const Post* post, int32_t H, int64_t m, int64_t words, uint32_t* present,
                          hipStream_t s);
hipError_t launch_count(const CountArgs& a, hipStream_t s);

}  // namespace apss
