// C ABI of the apss library: index construction, self-join, external
// queries.  Host code only orchestrates device work; every step of the
// join runs in the kernels of index_build.hip (index, query rows), pairs.hip
// (list pairs, sketches, candidate count), few.hip (few queries), join.hip
// (accumulating join), screen.hip (head screen), finish.hip and primitives.hip
// (pairs sorted and handed over).
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <array>
#include <cmath>
#include <cstddef>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "../../include/apss.h"
#include "apss_internal.h"
#include "finish.h"
#include "index_build.h"
#include "join.h"
#include "lib.h"
#include "screen.h"

namespace apss {

std::string& last_error() {
  static thread_local std::string s;
  return s;
}

void set_error(const char* fmt, ...) {
  char buf[1024];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  last_error() = buf;
}

int dev_err(hipError_t e, const char* what) {
  if (e == hipErrorOutOfMemory || e == hipErrorMemoryAllocation) {
    set_error("%s: out of device memory", what);
    (void)hipGetLastError();
    return APSS_ENOMEM;
  }
  set_error("%s: %s", what, hipGetErrorString(e));
  return APSS_EDEVICE;
}

namespace {

struct Spare {
  void* p;
  size_t size;
  int device;
  uint64_t stamp;  // requests made before it was put here
};
// (never destroyed: indexes may end after the library's statics)
std::mutex& g_spare_mu = *new std::mutex;
std::vector<Spare>& g_spare = *new std::vector<Spare>;  // oldest first
uint64_t g_spare_requests = 0;
constexpr uint64_t kSpareAge = 32;

// Most bytes kept on a device.  Locked.
size_t spare_limit(int device) {
  static std::vector<size_t>& limit = *new std::vector<size_t>;
  if ((size_t)device >= limit.size()) limit.resize((size_t)device + 1, 0);
  if (!limit[(size_t)device]) {
    hipDeviceProp_t prop;
    limit[(size_t)device] =
        hipGetDeviceProperties(&prop, device) == hipSuccess ? std::max<size_t>(prop.totalGlobalMem / 32, 1) : 1;
  }
  return limit[(size_t)device];
}

// Take out (into gone) what is old and what exceeds the device's limit.  Locked.
void spare_trim(int device, std::vector<void*>& gone) {
  const size_t limit = spare_limit(device);
  size_t held = 0;
  for (const Spare& c : g_spare) held += c.device == device ? c.size : 0;
  for (size_t k = 0; k < g_spare.size();) {
    const Spare& c = g_spare[k];
    if (g_spare_requests - c.stamp > kSpareAge || (c.device == device && held > limit)) {
      held -= c.device == device ? c.size : 0;
      gone.push_back(c.p);
      g_spare.erase(g_spare.begin() + (std::ptrdiff_t)k);
    } else {
      ++k;
    }
  }
}

}  // namespace

hipError_t spare_take(size_t bytes, void** p, size_t* size, int* device_out) {
  // (sizes in steps of up to a sixteenth, so that builds of like inputs match)
  size_t step = 1 << 20;
  while (step * 32 <= bytes) step *= 2;
  bytes = (bytes + step - 1) / step * step;
  int device = 0;
  hipError_t e = hipGetDevice(&device);
  if (e != hipSuccess) return e;
  *device_out = device;
  std::vector<void*> gone;
  *p = nullptr;
  {
    std::lock_guard<std::mutex> lock(g_spare_mu);
    ++g_spare_requests;
    size_t best = g_spare.size();
    for (size_t k = 0; k < g_spare.size(); ++k)
      if (g_spare[k].device == device && g_spare[k].size >= bytes && g_spare[k].size <= bytes + bytes / 4 &&
          (best == g_spare.size() || g_spare[k].size < g_spare[best].size))
        best = k;
    if (best < g_spare.size()) {
      *p = g_spare[best].p;
      *size = g_spare[best].size;
      g_spare.erase(g_spare.begin() + (std::ptrdiff_t)best);
    }
    try {
      spare_trim(device, gone);
    } catch (const std::bad_alloc&) {  // (the next request's turn)
    }
  }
  for (void* q : gone) (void)hipFree(q);
  if (*p) return hipSuccess;
  e = hipMalloc(p, bytes);
  if (e != hipSuccess) {
    (void)hipGetLastError();  // (kept until asked for: the next launch's check would find it)
    spare_release();
    e = hipMalloc(p, bytes);
  }
  if (e != hipSuccess) {
    *p = nullptr;
    return e;
  }
  *size = bytes;
  return hipSuccess;
}

void spare_put(void* p, size_t size, int device) {
  if (!p) return;
  std::vector<void*> gone;
  {
    std::lock_guard<std::mutex> lock(g_spare_mu);
    try {  // (called by destructors)
      g_spare.push_back(Spare{p, size, device, g_spare_requests});
      p = nullptr;
      spare_trim(device, gone);
    } catch (const std::bad_alloc&) {
    }
  }
  if (p) (void)hipFree(p);
  for (void* q : gone) (void)hipFree(q);
}

size_t spare_release() {
  std::vector<Spare> all;
  {
    std::lock_guard<std::mutex> lock(g_spare_mu);
    all.swap(g_spare);
  }
  size_t bytes = 0;
  for (const Spare& c : all) {
    (void)hipFree(c.p);
    bytes += c.size;
  }
  return bytes;
}

namespace {

const char* err_bits_text(uint32_t e) {
  if (e & ERR_ROWPTR) return "row_ptr must start at 0, be non-decreasing and end at nnz";
  if (e & ERR_DIM) return "dimension id outside [0, m)";
  if (e & ERR_WEIGHT) return "weights must be finite and > 0";
  if (e & ERR_NORM) return "non-empty rows must have unit L2 norm (|norm - 1| <= 1e-5)";
  if (e & ERR_DUP) return "repeated dimension id inside a row";
  return "invalid input";
}

}  // namespace
}  // namespace apss


using namespace apss;

#define CHK APSS_CHK

namespace {

// True when rows of at most longest entries are sorted by segments.
bool sorts_segments(int64_t nnz, int64_t longest, int key_bits) {
  return nnz > kSortSegment && longest <= kSortSegment && key_bits <= 51;
}

// Sort (row, rank) keys with float payload into rank-space rows; checks for duplicates.
// Rows are contiguous in row-major order, so with the row index in the key's
// high bits sorting groups of whole rows independently sorts the whole
// array: given the host row offsets, rows are grouped into segments of at
// most kSortSegment entries, one workgroup each (one launch); otherwise, or
// when a row is longer, radix passes over the whole array.
int sort_rows(Workspace& ws, uint64_t* keys, uint32_t* vals, int64_t nnz, int key_bits, int rbits, RComp* rc_out,
              uint32_t* err_dev, const int64_t* rp_host = nullptr, int64_t nrows = 0) {
  hipStream_t s = ws.stream;
  SortScratch& ss = ws.ss;
  if (rp_host && nnz > kSortSegment && key_bits <= 51) {
    std::vector<int64_t>& seg = ss.seg_host;
    seg.clear();
    seg.push_back(0);
    bool fits = true;
    for (int64_t r = 0; r < nrows && fits; ++r) {
      const int64_t e = rp_host[r + 1];
      if (e - rp_host[r] > kSortSegment) fits = false;
      else if (e - seg.back() > kSortSegment) seg.push_back(rp_host[r]);
    }
    if (fits) {
      if (seg.back() != nnz) seg.push_back(nnz);
      const int64_t nseg = (int64_t)seg.size() - 1;
      CHK(ss.seg.reserve(nseg + 1), "sort scratch");
      CHK(hipMemcpyAsync(ss.seg.p, seg.data(), sizeof(int64_t) * (nseg + 1), hipMemcpyHostToDevice, s), "row sort");
      CHK(segment_sort_u64_u32(keys, vals, ss.seg.p, nseg, s), "row sort");
      CHK(launch_unpack_rows(keys, vals, nnz, rbits, rc_out, err_dev, s), "row unpack");
      return APSS_OK;
    }
  }
  CHK(ss.k2.reserve(nnz), "sort scratch");
  CHK(ss.v32b.reserve(nnz), "sort scratch");
  CHK(ss.hist.reserve(radix_hist_elems(nnz)), "sort scratch");
  CHK(ss.scan.reserve(radix_scan_tmp_elems(nnz)), "sort scratch");
  CHK(radix_sort_u64_u32(keys, vals, ss.k2.p, ss.v32b.p, nnz, key_bits, ss.hist.p, ss.scan.p, s), "row sort");
  CHK(launch_unpack_rows(keys, vals, nnz, rbits, rc_out, err_dev, s), "row unpack");
  return APSS_OK;
}

int check_bits(uint32_t err, unsigned long long bad, const char* what) {
  if (!err) return APSS_OK;
  if (bad != ~0ull) set_error("%s: %s (row %llu)", what, err_bits_text(err), bad);
  else set_error("%s: %s", what, err_bits_text(err));
  return APSS_EINVAL;
}

// The checks' words on the device: error bits, first bad row, longest row.
int check_err(hipStream_t s, const unsigned long long* checks, const char* what, bool row = true,
              unsigned long long* longest = nullptr) {
  unsigned long long w[3] = {0ull, ~0ull, 0ull};
  CHK(hipMemcpyAsync(w, checks, sizeof(unsigned long long) * (longest ? 3 : 2), hipMemcpyDeviceToHost, s), what);
  CHK(hipStreamSynchronize(s), what);
  if (longest) *longest = w[2];
  return check_bits((uint32_t)w[0], row ? w[1] : ~0ull, what);
}

int reset_err(Workspace& ws) {
  static const unsigned long long clear[3] = {0ull, ~0ull, 0ull};
  CHK(ws.checks.reserve(3), "alloc");
  CHK(hipMemcpyAsync(ws.checks.p, clear, sizeof(clear), hipMemcpyHostToDevice, ws.stream), "clear checks");
  return APSS_OK;
}

// Device copies of a CSR given on host or device.
struct CsrDev {
  DBuf<int64_t> rp;
  DBuf<int32_t> col;
  DBuf<float> val;
  const int64_t* prp = nullptr;
  const int32_t* pcol = nullptr;
  const float* pval = nullptr;
};

int read_nnz(hipStream_t s, int64_t n, const int64_t* row_ptr, int on_device, int64_t* nnz) {
  if (!on_device) {
    *nnz = row_ptr[n];
    return APSS_OK;
  }
  CHK(hipMemcpyAsync(nnz, row_ptr + n, sizeof(int64_t), hipMemcpyDeviceToHost, s), "read nnz");
  CHK(hipStreamSynchronize(s), "read nnz");
  return APSS_OK;
}

int stage_csr(hipStream_t s, int64_t n, int64_t nnz, const int64_t* row_ptr, const int32_t* col, const float* val,
              int on_device, Arena& tmp, CsrDev& d) {
  if (on_device) {
    d.prp = row_ptr;
    d.pcol = col;
    d.pval = val;
  } else {
    CHK(d.rp.take(tmp, n + 1), "alloc csr");
    CHK(d.col.take(tmp, nnz), "alloc csr");
    CHK(d.val.take(tmp, nnz), "alloc csr");
    CHK(hipMemcpyAsync(d.rp.p, row_ptr, sizeof(int64_t) * (n + 1), hipMemcpyHostToDevice, s), "copy csr");
    if (nnz) {
      CHK(hipMemcpyAsync(d.col.p, col, sizeof(int32_t) * nnz, hipMemcpyHostToDevice, s), "copy csr");
      CHK(hipMemcpyAsync(d.val.p, val, sizeof(float) * nnz, hipMemcpyHostToDevice, s), "copy csr");
    }
    d.prp = d.rp.p;
    d.pcol = d.col.p;
    d.pval = d.val.p;
  }
  return APSS_OK;
}

int hoff_slot(int cb) { return cb == 1024 ? 0 : 1; }

// cnt_r: components of each dimension, by rank (device)
int build_lists(apss_index* ix, const uint32_t* cnt_r, Arena& tmp);
int build_screen(apss_index* ix, int32_t head, const uint32_t* cnt_r, Arena& tmp);

int build_impl(apss_index* ix, const int64_t* row_ptr, const int32_t* col, const float* val, int on_device) {
  Workspace& ws = ix->ws;
  hipStream_t s = ws.stream;
  const int64_t n = ix->n, m = ix->m;
  int64_t nnz = 0;
  int rc = read_nnz(s, n, row_ptr, on_device, &nnz);
  if (rc) return rc;
  if (!on_device && (row_ptr[0] != 0 || nnz < 0)) {
    set_error("row_ptr must start at 0 and end at nnz >= 0");
    return APSS_EINVAL;
  }
  if (nnz < 0 || nnz >= (1ll << 32)) {
    set_error("nnz must be in [0, 2^32)");
    return APSS_EINVAL;
  }
  if ((rc = reset_err(ws))) return rc;
  uint32_t* err = ws.err();
  unsigned long long* bad = ws.bad();
  unsigned long long longest = 0;
  if (on_device) {
    CHK(launch_check_rowptr(row_ptr, n, nnz, err, bad, ws.checks.p + 2, s), "check row_ptr");
    if ((rc = check_err(s, ws.checks.p, "build_index", true, &longest))) return rc;
  } else {
    for (int64_t r = 0; r < n; ++r) {
      if (row_ptr[r + 1] < row_ptr[r]) {
        set_error("row_ptr must be non-decreasing (row %lld)", (long long)r);
        return APSS_EINVAL;
      }
      longest = std::max(longest, (unsigned long long)(row_ptr[r + 1] - row_ptr[r]));
    }
  }
  // the build's scratch, sized for the list sort too (at most nnz postings)
  const int64_t big = std::max<int64_t>(nnz, m + 1);
  Arena tmp;
  struct Scratch {  // (the sort buffers are pieces of tmp, and end before it)
    SortScratch& ss;
    hipStream_t s;
    ~Scratch() {
      (void)hipStreamSynchronize(s);
      for (DBuf<uint64_t>* b : {&ss.k1, &ss.k2, &ss.v64a, &ss.v64b}) b->release();
      for (DBuf<uint32_t>* b : {&ss.v32a, &ss.v32b}) b->release();
      for (DBuf<int64_t>* b : {&ss.hist, &ss.scan}) b->release();
    }
  } scratch{ws.ss, s};
  const int lists = ix->opts.screen_dims > 0 ? 2 : 1;  // (with the head-cut index's)
  CHK(tmp.reserve(4 * Arena::bytes<uint64_t>(big) + Arena::bytes<int64_t>(radix_hist_elems(big)) +
                  Arena::bytes<int64_t>(radix_scan_tmp_elems(big)) + 3 * Arena::bytes<uint32_t>(m) +
                  Arena::bytes<uint32_t>(nnz / kWaveRow + 1) +
                  lists * (Arena::bytes<int64_t>(n + 1) + Arena::bytes<int64_t>(scan_tmp_elems(n + 1)) +
                           Arena::bytes<int64_t>(scan_tmp_elems(big))) +
                  (on_device ? 0 : Arena::bytes<int64_t>(n + 1) + 2 * Arena::bytes<float>(nnz)) + 64 * 256),
      "alloc scratch");
  CHK(ix->mem.reserve(Arena::bytes<int64_t>(n + 1) + Arena::bytes<RComp>(nnz) + 2 * Arena::bytes<uint32_t>(m) +
                      Arena::bytes<RowStat>(n) + Arena::bytes<float>(n) + Arena::bytes<uint8_t>(n) +
                      Arena::bytes<uint32_t>(m + n)),
      "alloc index");
  CsrDev in;
  if ((rc = stage_csr(s, n, nnz, row_ptr, col, val, on_device, tmp, in))) return rc;
  ix->nnz = nnz;

  // the remaining checks, density order and maxweight_d(V)
  DBuf<uint32_t> cnt, mwbits, cnt_r;
  CHK(cnt.take(tmp, m), "alloc");
  CHK(mwbits.take(tmp, m), "alloc");
  CHK(cnt_r.take(tmp, m), "alloc");
  CHK(fill_u32(cnt.p, 0u, m, s), "fill");
  CHK(fill_u32(mwbits.p, 0u, m, s), "fill");
  CHK(launch_validate_count(in.prp, in.pcol, in.pval, n, m, 1e-5, cnt.p, mwbits.p, err, bad, s), "validate");
  if ((rc = check_err(s, ws.checks.p, "build_index"))) return rc;
  const int dbits = ceil_log2((uint64_t)m);
  const int cbits = ceil_log2((uint64_t)n + 1);
  SortScratch& ss = ws.ss;
  CHK(ss.k1.take(tmp, big), "alloc sort");
  CHK(ss.v64a.take(tmp, big), "alloc sort");
  CHK(ss.k2.take(tmp, big), "alloc sort");
  CHK(ss.v64b.take(tmp, big), "alloc sort");
  CHK(ss.hist.take(tmp, radix_hist_elems(big)), "alloc sort");
  CHK(ss.scan.take(tmp, radix_scan_tmp_elems(big)), "alloc sort");
  CHK(launch_dim_keys(cnt.p, m, n, dbits, ss.k1.p, ss.v64a.p, s), "dim keys");
  CHK(radix_sort_u64(ss.k1.p, ss.v64a.p, ss.k2.p, ss.v64b.p, m, dbits + cbits, ss.hist.p, ss.scan.p, s), "dim sort");
  CHK(ix->rank.take(ix->mem, m), "alloc");
  CHK(ix->mw_r.take(ix->mem, m), "alloc");
  CHK(launch_rank_from_sorted(ss.v64a.p, m, cnt.p, mwbits.p, ix->rank.p, ix->mw_r.p, cnt_r.p, s), "ranks");

  CHK(ix->out.take(ix->mem, m + n), "alloc");

  // rows in rank space, densest dimension first
  const int rbits = dbits;
  const int nbits = ceil_log2((uint64_t)std::max<int64_t>(n, 1));
  ix->rows.n = n;
  ix->rows.nnz = nnz;
  CHK(ix->rows.rp.take(ix->mem, n + 1), "alloc");
  CHK(hipMemcpyAsync(ix->rows.rp.p, in.prp, sizeof(int64_t) * (n + 1), hipMemcpyDeviceToDevice, s), "copy");
  ix->rows.rp_host.resize((size_t)n + 1);
  if (on_device)
    CHK(hipMemcpyAsync(ix->rows.rp_host.data(), in.prp, sizeof(int64_t) * (n + 1), hipMemcpyDeviceToHost, s), "copy");
  else memcpy(ix->rows.rp_host.data(), row_ptr, sizeof(int64_t) * (size_t)(n + 1));
  CHK(ix->rows.rc.take(ix->mem, nnz), "alloc");
  if (longest <= (unsigned long long)kLongRow) {
    DBuf<unsigned int> nlong;
    DBuf<uint32_t> longs;
    CHK(nlong.take(tmp, 1), "alloc");
    CHK(longs.take(tmp, nnz / kWaveRow + 1), "alloc");
    CHK(fill_u32(nlong.p, 0u, 1, s), "fill");
    CHK(launch_sort_rows(in.prp, in.pcol, in.pval, ix->rank.p, n, (int64_t)longest, ix->rows.rc.p, err, nlong.p,
                         longs.p, s),
        "row sort");
    if ((rc = check_err(s, ws.checks.p, "build_index", false))) return rc;
  } else {
    // a row past one workgroup's LDS: radix passes over (row, rank) keys
    CHK(ss.k1.reserve(nnz), "alloc sort");
    CHK(ss.v32a.reserve(nnz), "alloc");
    CHK(launch_row_keys(in.prp, in.pcol, in.pval, ix->rank.p, n, rbits, ss.k1.p, ss.v32a.p, s), "row keys");
    if ((rc = sort_rows(ws, ss.k1.p, ss.v32a.p, nnz, nbits + rbits, rbits, ix->rows.rc.p, err))) return rc;
    if ((rc = check_err(s, ws.checks.p, "build_index", false))) return rc;
  }
  if ((rc = build_lists(ix, cnt_r.p, tmp))) return rc;
  if (ix->opts.screen_dims <= 0) return APSS_OK;
  return build_screen(ix, (int32_t)std::min<int64_t>(ix->opts.screen_dims, m), cnt_r.p, tmp);
}

// No geometry asked for: a tile variant, range width or group given by the
// caller, or by the environment when the index is built, names the
// accumulating kernel.
bool default_geometry(const apss_opts& o) {
  return o.variant < 0 && o.range_rows == 0 && o.range_group == 0 && !getenv("APSS_VARIANT") &&
         !getenv("APSS_RANGE_ROWS") && !getenv("APSS_RANGE_GROUP");
}

// An index whose self-joins may take the list-pair kernels: the default
// algorithm and geometry, and the sparse pass of the screened join (whose
// geometry is that of the accumulating kernel wherever the cost rule leaves it
// there).
bool pairs_eligible(const apss_index* ix) {
  const apss_opts& o = ix->opts;
  if (o.index_all || o.local_parts > 1 || o.remscore || o.screen_dims) return false;
  if (ix->n <= 1 || ix->n > (1 << 25)) return false;  // (a list's units are counted in 32 bits)
  return ix->head_cut > 0 || ix->default_geometry;
}

int32_t dense_ranks(const apss_index* ix) {
  return (int32_t)std::min<int64_t>(ix->opts.head_dims > 0 ? ix->opts.head_dims : 32768, ix->m);
}

// Bytes of the candidate count's tables.
int64_t count_bytes(const apss_index* ix) {
  const int64_t H = dense_ranks(ix), blocks = (ix->n + kCountRows - 1) / kCountRows;
  return Arena::bytes<uint32_t>(blocks * std::min<int64_t>(kCountRanks, H) * kCountWords) +
         Arena::bytes<uint2>(blocks * H) +
         Arena::bytes<uint32_t>(blocks * std::max<int64_t>(1, (ix->m - H + 31) / 32));
}

// Queries per work item of a self-join's candidate count: about eight items per
// compute unit, of at least a few queries per wave; where that leaves the
// device idle kPieceRows, counted by pieces of rows (a replay of 12,000 rows of
// mean 80: 350 us by the larger items, 269 so; 30,000 of mean 150: 1,069 us
// and 1,241; about even at 20,000).
int64_t count_chunk(int64_t n, int64_t blocks) {
  const int64_t want = n * blocks / 2 / 2048;
  const int64_t chunk = std::max<int64_t>(64, std::min<int64_t>(4096, (want + 63) / 64 * 64));
  return n * blocks / 2 / chunk < 512 ? kPieceRows : chunk;
}

// An index without the list-pair and sketch tables: its joins and queries take
// the accumulating kernel.
int drop_pair_tables(apss_index* ix) {
  CHK(hipStreamSynchronize(ix->ws.stream), "build_index");
  ix->pairs_ready = ix->screen_queries = false;
  for (DBuf<uint8_t>* b : {&ix->sk, &ix->mid, &ix->fsk}) b->release();
  for (DBuf<uint32_t>* b : {&ix->dl, &ix->dlr, &ix->fidx}) b->release();
  for (DBuf<uint2>* b : {&ix->wide, &ix->shorts}) b->release();
  ix->gid.release();
  ix->doff.release();
  ix->ndeep = ix->nwide = ix->nshort = 0;
  ix->pair_mem.release();
  return APSS_OK;
}

// About the norm that a byte code stands for (an upper bound in 1/254 steps).
double norm_of_code(int c) { return c >= kPn8None ? 1.0 : c > 0 ? ((double)c - 0.5) / 254.0 : 0.0; }

// Memory for those tables.  *have is false, and the index does without them,
// if the device has too little.
int reserve_pair_tables(apss_index* ix, int64_t bytes, bool* have) {
  const hipError_t e = ix->pair_mem.reserve(bytes);
  *have = e == hipSuccess;
  if (*have) return APSS_OK;
  const int rc = dev_err(e, "alloc tables");
  return rc == APSS_ENOMEM ? drop_pair_tables(ix) : rc;
}

// Sketches, deep lists and work units, from the sorted list values in the
// sort scratch (with the lists of every index).  The sort's other buffers, of
// at least m + 1 entries, hold what is passing.
int build_pair_lists(apss_index* ix, const uint32_t* cnt_r, Arena& tmp) {
  Workspace& ws = ix->ws;
  hipStream_t s = ws.stream;
  SortScratch& ss = ws.ss;
  const int64_t n = ix->n, m = ix->m, P = ix->P;
  const int64_t nt = list_tiles(P);
  int64_t* const tiles = (int64_t*)ss.v64b.p;
  DBuf<int64_t> scan, total;
  CHK(scan.take(tmp, scan_tmp_elems(std::max(nt, m + 1))), "alloc");
  CHK(total.take(tmp, 1), "alloc");
  int64_t deep = 0;
  CHK(launch_count_deep(ss.v64a.p, P, tiles, s), "deep lists");
  CHK(exclusive_scan_i64(tiles, nt, scan.p, total.p, s), "scan");
  CHK(hipMemcpyAsync(&deep, total.p, sizeof(int64_t), hipMemcpyDeviceToHost, s), "deep lists");
  CHK(hipStreamSynchronize(s), "deep lists");
  int64_t longs = 0;
  double unstaged = 0.0;  // share of the components that lie in rows whose lookups go to memory
  for (int64_t r = 0; r < n; ++r) {
    const int64_t len = ix->rows.rp_host[(size_t)r + 1] - ix->rows.rp_host[(size_t)r];
    longs += len > kFineRow;
    if (len > kStageRanks) unstaged += (double)len / (double)ix->nnz;
  }
  bool have = false;
  int rc = reserve_pair_tables(ix, 2 * Arena::bytes<uint32_t>(deep) + Arena::bytes<int64_t>(m + 1) +
                                       Arena::bytes<uint16_t>(m) + Arena::bytes<uint8_t>(n * kSkGroups) +
                                       Arena::bytes<uint8_t>(n * kMidGroups) + Arena::bytes<uint32_t>(n) +
                                       Arena::bytes<uint8_t>(longs * kFineGroups),
                               &have);
  if (rc) return rc;
  if (!have) {
    CHK(launch_lists(nullptr, ss.v64a.p, P, ix->post.p, ix->post4.p, nullptr, nullptr, nullptr, nullptr, s), "lists");
    return APSS_OK;
  }
  ix->ndeep = deep;
  CHK(ix->dl.take(ix->pair_mem, deep), "alloc");
  CHK(ix->dlr.take(ix->pair_mem, deep), "alloc");
  CHK(ix->doff.take(ix->pair_mem, m + 1), "alloc");
  uint32_t* pos = (uint32_t*)ss.k2.p;
  CHK(launch_lists(ss.k1.p, ss.v64a.p, P, ix->post.p, ix->post4.p, tiles, pos, ix->dl.p, ix->dlr.p, s), "lists");
  CHK(launch_deep_offsets(ix->off.p, pos, P, m, deep, ix->doff.p, s), "deep lists");
  // groups of ranks of about equal component counts, and the sketches
  CHK(ix->gid.take(ix->pair_mem, m), "alloc");
  CHK(ix->sk.take(ix->pair_mem, n * kSkGroups), "alloc");
  CHK(launch_widen(cnt_r, m, tiles, s), "groups");
  CHK(exclusive_scan_i64(tiles, m, scan.p, nullptr, s), "scan");
  CHK(launch_groups(tiles, cnt_r, m, ix->nnz, ix->gid.p, s), "groups");
  CHK(ix->mid.take(ix->pair_mem, n * kMidGroups), "alloc");
  CHK(ix->fidx.take(ix->pair_mem, n), "alloc");
  CHK(ix->fsk.take(ix->pair_mem, longs * kFineGroups), "alloc");
  DBuf<unsigned int> nfine;
  CHK(nfine.take(tmp, 1), "alloc");
  CHK(fill_u32(nfine.p, 0u, 1, s), "fill");
  CHK(launch_sketch(ix->rows.rp.p, ix->rows.rc.p, ix->gid.p, n, ix->sk.p, ix->mid.p, nfine.p, ix->fidx.p,
                    ix->fsk.p, s), "sketches");
  // work units by rank
  int64_t* const stiles = (int64_t*)ss.k1.p;
  CHK(launch_unit_counts(ix->doff.p, m, true, tiles, s), "units");
  CHK(launch_unit_counts(ix->doff.p, m, false, stiles, s), "units");
  CHK(exclusive_scan_i64(tiles, m, scan.p, total.p, s), "scan");
  CHK(hipMemcpyAsync(&ix->nwide, total.p, sizeof(int64_t), hipMemcpyDeviceToHost, s), "units");
  CHK(exclusive_scan_i64(stiles, m, scan.p, total.p, s), "scan");
  CHK(hipMemcpyAsync(&ix->nshort, total.p, sizeof(int64_t), hipMemcpyDeviceToHost, s), "units");
  CHK(hipStreamSynchronize(s), "units");
  // (with the candidate count's tables: see build_bitmaps.  The kernels count
  // units in 31 bits; whole-corpus lists of some 20 million rows have more)
  if (ix->nwide > kMaxUnits || ix->nshort > kMaxUnits) return drop_pair_tables(ix);
  rc = reserve_pair_tables(ix, Arena::bytes<uint2>(ix->nwide) + Arena::bytes<uint2>(ix->nshort) + count_bytes(ix), &have);
  if (rc || !have) return rc;
  CHK(ix->wide.take(ix->pair_mem, ix->nwide), "alloc");
  CHK(ix->shorts.take(ix->pair_mem, ix->nshort), "alloc");
  CHK(launch_unit_fill(ix->doff.p, tiles, m, true, ix->wide.p, s), "units");
  CHK(launch_unit_fill(ix->doff.p, stiles, m, false, ix->shorts.p, s), "units");
  ix->pair_groups = pairs_resident_groups();
  // The list-pair kernels or the accumulating one, whichever should take
  // less, by their measured rates (MI355X): the accumulating kernel visits
  // 1.2e12 list entries and filters 1.1e12 pairs of rows a second, beside
  // which it takes 25 ps to enter a query's component in 1,024 rows; the
  // list-pair kernels test 1.5e12 pairs a second, take 1.6 ns per short unit
  // (a wave's), decide a survivor in 0.45 ns, and count the candidates of a
  // query in a block of 4,096 rows in 2 ns (at 120 components with lists, in
  // proportion to them).  Measured, accumulating and list pairs: 30 and 13 ms
  // (100,000 rows of mean 80, t = 0.5), 490 and 77 ms (500,000 of mean 120,
  // 0.7).  The survivors are estimated from every k-th unit, and doubled: on
  // rows that the sketches do not tell apart (flat weights over few dimensions)
  // they are most pairs, and the accumulating kernel is ahead.  A join at a
  // higher threshold than the index's has fewer.
  DBuf<unsigned long long> cnt;
  constexpr int kCodes = 256;
  constexpr int kWords = C_NUM + kRateBins + 2 + kCodes;  // the pairs' counters, the queries' bins, visits, norms
  CHK(cnt.take(tmp, kWords), "alloc");
  if (int rc = reserve_control(ws)) return rc;
  CHK(fill_u64((uint64_t*)cnt.p, 0ull, kWords, s), "fill");
  CHK(fill_u32(ws.qctr, 0u, kQueueCounters, s), "fill");
  JoinPlan plan;
  bind_pairs(ix, ix->t_build, ws.qctr, nullptr, 0, plan);
  plan.pa.counters = cnt.p;
  const int64_t windows = (ix->ndeep + kTinyList - 1) / kTinyList;
  const int64_t units = ix->nwide + ix->nshort / kShortUnits + windows / 64;
  plan.pa.sample = 1;
  plan.pa.every = std::max<int64_t>(1, units / 4096);
  CHK(launch_pairs(plan.pa, plan.pg, s), "sample");
  CHK(launch_visits(cnt_r, ix->off.p, m, kCountRanks, cnt.p + C_NUM + kRateBins, s), "sample");
  if (ix->head_cut > 0) CHK(launch_norm_codes(ix->pn8.p, n, cnt.p + C_NUM + kRateBins + 2, s), "sample");
  // ... and for queries the survivors among about 2^24 pairs of rows
  plan.qa.sk = ix->mid.p;
  plan.qa.n = n;
  plan.qa.qsk = ix->mid.p;
  plan.qa.nq = std::min<int64_t>(n, 1024);
  plan.qa.qstride = n / plan.qa.nq;
  plan.qa.t = ix->t_build;
  PairArgs qsample = plan.pa;
  qsample.counters = cnt.p + C_NUM;
  qsample.every = std::max<int64_t>(1, n / kWideRows / 64);
  CHK(launch_query_sample(qsample, plan.qa, s), "sample");
  unsigned long long c[kWords];
  const unsigned long long* const qc = c + C_NUM;
  CHK(hipMemcpyAsync(c, cnt.p, sizeof(c), hipMemcpyDeviceToHost, s), "sample");
  CHK(hipStreamSynchronize(s), "sample");
  const double k = (double)plan.pa.every;
  const double blocks = (double)((n + kCountRows - 1) / kCountRows);
  const double survivors = k * (double)c[C_SURVIVORS];
  const double visits = (double)c[C_NUM + kRateBins], entries = (double)c[C_NUM + kRateBins + 1];
  // What long rows cost beyond that: in the count the entries of lists past the
  // bitmaps, by lane (4 ps, 6 by pieces), and a wave's share of the rows, one
  // piece after another; in the decisions lookups of rows too long for LDS.
  // Rows of mean 1,500 over a million dimensions, accumulating and list pairs:
  // 2,000 rows 0.44 and 0.93 ms, 10,000 4.2 and 8.0, 30,000 35.5 and 59.6; of
  // mean 500: 2,000 rows 0.19 and 0.17, 5,000 0.45 and 0.57, 12,000 1.55 and
  // 0.86, 60,000 34.1 and 14.4.
  const double stream_s = visits / 1.2e12 + 0.5 * (double)n * (double)n / 1.1e12;
  const double test_s = k * (double)c[C_VISITS] / 1.5e12 + (double)ix->nshort * 1.6e-9 + (double)windows * 0.4e-9;
  if (ix->head_cut > 0) {
    // The sparse pass.  Its accumulating kernel adds a product of the head's
    // norms to what it has accumulated, and what passes is rescored one pair at
    // a time, some 4 ns each: half of the pairs that share a tail dimension and
    // whose heads' norms alone could reach t.  Without such heads it is ahead
    // of the list pairs where those have many survivors.  Accumulating and list
    // pairs, measured: heads of 4,096 dimensions, 30,000 rows of mean 300 at t =
    // 0.6 415 and 6.2 ms, 50,000 flat rows at 0.6 15.3 and 1.1; 40,000 text rows,
    // 0.6, head 512 20 and 0.7; but heads of 64, 30,000 rows of mean 300 6.0 and
    // 16.2, of mean 500 at 0.5 8.4 and 24; and rows of mean 1,500 and 6,000 with
    // any head, 8,000 at 0.8 1.8 and 4.6, 4,500 at 0.8 5.1 and 532.  Over 109
    // such pairs of corpus and head the rule is within 0.06 ms or an eighth of
    // the better one.
    double reach = 0.0, above = 0.0;
    for (int lo = 0, hi = kCodes; lo < kCodes; ++lo) {  // codes lo whose products with hi and up reach t
      while (hi > 0 && norm_of_code(lo) * norm_of_code(hi - 1) >= (double)ix->t_build)
        above += (double)c[C_NUM + kRateBins + 2 + --hi];
      reach += 0.5 * (double)c[C_NUM + kRateBins + 2 + lo] * above;
    }
    const double rows2 = 0.5 * (double)n * (double)n;
    const double chain_s = n <= 4 * kCountRows ? 10e-6 * (double)ix->P / (64.0 * (double)n) : 0.0;
    const double pairs_s = test_s + survivors * (0.6e-9 + 3e-9 * unstaged) + visits * 1.6e-12 + chain_s;
    const double stage_s = 25e-12 * (double)ix->P * 0.5 * (double)n / 1024.0;
    const double rescored = 0.5 * reach * std::min(1.0, visits / rows2);
    ix->pairs_ready = pairs_s < std::sqrt(stream_s * stream_s + stage_s * stage_s) + rescored * 4e-9;
  } else {
    const bool pieces = count_chunk(n, (int64_t)blocks) <= kPieceRows;
    const double chain_s = pieces ? 10e-6 * (double)ix->nnz / (64.0 * (double)n) : 0.0;
    const double long_s = entries * (pieces ? 6e-12 : 4e-12) + chain_s + survivors * 3e-9 * unstaged;
    const double count_s = 0.5 * blocks * (double)ix->P * (2e-9 / 110.0);
    const double pairs_s = test_s + 2.0 * survivors * 0.45e-9 + count_s + long_s;
    const double stage_s = 25e-12 * (double)ix->nnz * 0.5 * (double)n / 1024.0;
    const double lists_s = std::sqrt(stream_s * stream_s + stage_s * stage_s);
    // (up to one block of rows launches and waits are most of either: 0.24 ms
    // against 0.27 ms for 2,000 rows, so there only many survivors and long rows
    // decide)
    const bool few = survivors <= 64.0 * (double)n;
    ix->pairs_ready = n <= kCountRows ? few && long_s <= lists_s + 0.15e-3 : pairs_s < lists_s;
  }
  ix->pair_survivors = survivors;
  if (ix->opts.reserved[0] == kProbePairs) ix->pairs_ready = true;
  // Queries, per pair of a query and a row: 0.32 ps for the test and 0.49 for
  // the count at 110 indexed components a row, against 0.9 and 0.83 per list
  // entry; 1.2 ns per survivor (4,096 queries of mean 100 over 1,000,000
  // rows: 6.0 ms against 16.1 ms by the accumulating kernel).  The survivors
  // are known when the thresholds are; the tables are kept if the kernels
  // would win halfway between t_build and 1.
  const double rows2 = (double)n * (double)n;
  const int64_t span = kWideRows * qsample.every;
  const int64_t qrows = std::min<int64_t>(n, (n + span - 1) / span * kWideRows);
  double reach = 0.0;
  for (int b = kRateBins - 1; b >= 0; --b) {
    reach += (double)qc[b];
    ix->rate[b] = reach / ((double)plan.qa.nq * (double)qrows);
  }
  ix->screen_ps = 0.32 + 0.49 * (double)ix->P / (110.0 * (double)n);
  ix->accumulate_ps = 0.9 + 0.83 * 2.0 * visits / rows2;
  ix->screen_queries = ix->head_cut == 0 && ix->opts.query_safe &&
                       (ix->screen_ps + kSurvivorPs * ix->rate[kRateBins / 2] < ix->accumulate_ps ||
                        ix->opts.reserved[0] == kProbePairs);
  if (!ix->pairs_ready && !ix->screen_queries) return drop_pair_tables(ix);
  return APSS_OK;
}

// Bitmaps of the densest ranks for the candidate count (after prepare()).
int build_bitmaps(apss_index* ix) {
  const int slot = ix->hoff[0].p ? 0 : 1;
  const int cb = slot == 0 ? 1024 : 2048;
  // (the head-cut index of the screened join has no dense lists)
  ix->count_ranks = ix->head_cut > 0 ? 0 : std::min<int32_t>(kCountRanks, ix->H);
  ix->count_blocks = (ix->n + kCountRows - 1) / kCountRows;
  CHK(ix->bm.take(ix->pair_mem, ix->count_blocks * ix->count_ranks * kCountWords), "alloc");
  CHK(ix->seg.take(ix->pair_mem, ix->count_blocks * ix->H), "alloc");
  CHK(launch_segments(ix->hoff[slot].p, ix->H, cb, ix->hoff_nb[slot], ix->count_blocks, ix->seg.p, ix->ws.stream),
      "bitmaps");
  ix->present_words = std::max<int64_t>(1, (ix->m - ix->H + 31) / 32);
  const int64_t nw = ix->count_blocks * ix->present_words;
  CHK(ix->present.take(ix->pair_mem, nw), "alloc");
  CHK(fill_u32(ix->present.p, 0u, nw, ix->ws.stream), "fill");
  CHK(launch_present(ix->off.p, ix->post.p, ix->H, ix->m, ix->present_words, ix->present.p, ix->ws.stream), "bitmaps");
  CHK(launch_bitmaps(ix->post.p, ix->hoff[slot].p, ix->H, cb, ix->hoff_nb[slot], ix->count_ranks, ix->count_blocks,
                     ix->bm.p, ix->ws.stream),
      "bitmaps");
  return APSS_OK;
}

// From the rank-space rows on: cutoff of every row, the inverted lists of
// the indexed parts and the lookup tables of the join.
int build_lists(apss_index* ix, const uint32_t* cnt_r, Arena& tmp) {
  Workspace& ws = ix->ws;
  hipStream_t s = ws.stream;
  SortScratch& ss = ws.ss;
  const int64_t n = ix->n, m = ix->m;
  const int rbits = ceil_log2((uint64_t)m);
  int rc = APSS_OK;

  // cutoff of the unindexed part
  CHK(ix->rs.take(ix->mem, n), "alloc");
  CHK(ix->rows.mw.take(ix->mem, n), "alloc");
  DBuf<int64_t> nidx, scan_tmp, total;
  CHK(nidx.take(tmp, n + 1), "alloc");
  CHK(scan_tmp.take(tmp, scan_tmp_elems(n + 1)), "alloc");
  CHK(total.take(tmp, 1), "alloc");
  // head >= 0: the unindexed part of every row is its components of rank
  // below head (the screened join's head cut, or nothing at all for the
  // all-pairs-0-array index); -1: the paper's cutoff
  const int32_t head = ix->opts.index_all ? 0 : (ix->head_cut > 0 ? ix->head_cut : -1);
  // (with the largest unindexed-part norm and each row's as a byte: the
  // hashed filter's tests before it reads a row's statistics)
  DBuf<uint32_t> pmax;
  CHK(pmax.take(tmp, 1), "alloc");
  CHK(ix->pn8.take(ix->mem, std::max<int64_t>(n, 1)), "alloc");
  CHK(fill_u32(pmax.p, 0u, 1, s), "fill");
  CHK(launch_cutoff(ix->rows.rp.p, ix->rows.rc.p, ix->mw_r.p, n, ix->t_build, ix->opts.query_safe ? 1 : 0, head,
                    ix->rs.p, ix->rows.mw.p, nidx.p, pmax.p, ix->pn8.p, s),
      "cutoff");
  CHK(exclusive_scan_i64(nidx.p, n, scan_tmp.p, total.p, s), "scan");
  int64_t P = 0;
  uint32_t pmax_bits = 0u;
  CHK(hipMemcpyAsync(&P, total.p, sizeof(int64_t), hipMemcpyDeviceToHost, s), "read P");
  CHK(hipMemcpyAsync(&pmax_bits, pmax.p, sizeof(uint32_t), hipMemcpyDeviceToHost, s), "read max norm");
  CHK(hipStreamSynchronize(s), "read P");
  ix->P = P;
  memcpy(&ix->pnrm_max, &pmax_bits, sizeof(float));
  if (4 * (P + kPost4Pad) >= (1ll << 32)) {
    set_error("index too large: %lld postings (the packed lists must stay below 4 GiB)", (long long)P);
    return APSS_EINVAL;
  }

  {
    int qt = 0, cb = 1024;
    (void)join_variant_geometry(ix->variant, &qt, &cb);
    const int64_t H = dense_ranks(ix), nb = (n + cb - 1) / cb;
    const int64_t K = std::max<int64_t>(1, ix->range_rows / cb), nR = (nb + K - 1) / K;
    CHK(ix->mem.reserve(Arena::bytes<int64_t>(m + 1) + Arena::bytes<Post>(P + 2) + Arena::bytes<uint32_t>(P + kPost4Pad) +
                        Arena::bytes<uint32_t>((nb + 1) * H) + Arena::bytes<uint32_t>((nR + 1) * std::max<int64_t>(m - H, 1))),
        "alloc index");
  }
  // inverted lists of the indexed parts: stable sort by rank keeps vector ids ascending
  const bool pairs = pairs_eligible(ix) && P > 0;
  const int64_t room = pairs ? std::max<int64_t>(P, m + 1) : P;
  CHK(ss.k1.reserve(room), "alloc");
  CHK(ss.k2.reserve(P), "alloc");
  CHK(ss.v64a.reserve(P), "alloc");
  CHK(ss.v64b.reserve(room), "alloc");
  CHK(ss.hist.reserve(radix_hist_elems(P)), "alloc");
  CHK(ss.scan.reserve(radix_scan_tmp_elems(P)), "alloc");
  // rows may exceed norm 1 by 1e-5, and the scan rounds: 1e-4 covers both
  const double lim = pairs ? (double)ix->t_build * (double)ix->t_build * (1.0 - 1e-4) : -1.0;
  CHK(launch_emit_indexed(ix->rows.rp.p, ix->rows.rc.p, ix->rs.p, nidx.p, n, lim, ss.k1.p, ss.v64a.p, s), "emit");
  CHK(radix_sort_u64(ss.k1.p, ss.v64a.p, ss.k2.p, ss.v64b.p, P, rbits, ss.hist.p, ss.scan.p, s), "list sort");
  CHK(ix->off.take(ix->mem, m + 1), "alloc");
  CHK(launch_list_offsets(ss.k1.p, P, m, ix->off.p, s), "list offsets");
  // two padding entries after the last list let the join read positions p
  // and p + 1 for any p <= P (p = 0 too when there are no lists)
  CHK(ix->post.take(ix->mem, P + 2), "alloc");
  CHK(fill_u64((uint64_t*)ix->post.p + P, ~0ull, 2, s), "fill");
  // the join's list loads put a chunk's base in the scalar offset, which the
  // hardware range check does not cover: 64 zero entries after the last list
  // keep a chunk's lanes past its end inside the allocation
  CHK(ix->post4.take(ix->mem, P + kPost4Pad), "alloc");
  CHK(fill_u32(ix->post4.p + P, 0u, kPost4Pad, s), "fill");
  if (pairs) {
    if ((rc = build_pair_lists(ix, cnt_r, tmp))) return rc;
  } else {
    CHK(launch_lists(nullptr, ss.v64a.p, P, ix->post.p, ix->post4.p, nullptr, nullptr, nullptr, nullptr, s), "lists");
  }

  // local pruning: split the indexed ranks into parts of about equal
  // postings; ranks are in decreasing density, so the first parts hold the
  // few heaviest lists and the last ones the long tail
  ix->parts = ix->opts.local_parts > 1 ? ix->opts.local_parts : 1;
  if (ix->parts > 1) {
    std::vector<int64_t> off_h((size_t)m + 1);
    CHK(hipMemcpyAsync(off_h.data(), ix->off.p, sizeof(int64_t) * (m + 1), hipMemcpyDeviceToHost, s), "read lists");
    CHK(hipStreamSynchronize(s), "read lists");
    ix->part_lo_host.assign((size_t)ix->parts + 1, 0);
    for (int r = 1; r < ix->parts; ++r) {
      const int64_t target = (P * r + ix->parts - 1) / ix->parts;
      const int64_t k = std::lower_bound(off_h.begin(), off_h.end(), target) - off_h.begin();
      ix->part_lo_host[(size_t)r] = (int32_t)std::max<int64_t>(ix->part_lo_host[(size_t)r - 1], std::min<int64_t>(k, m));
    }
    ix->part_lo_host[(size_t)ix->parts] = (int32_t)m;
    CHK(ix->part_lo.take(ix->mem, ix->parts + 1), "alloc");
    CHK(hipMemcpyAsync(ix->part_lo.p, ix->part_lo_host.data(), sizeof(int32_t) * (ix->parts + 1),
                       hipMemcpyHostToDevice, s),
        "parts");
  }

  // per-block offsets of the dense lists, for the default tile variant
  ix->H = dense_ranks(ix);
  ix->building = true;
  rc = prepare(ix, s, ix->variant, ix->range_rows);
  ix->building = false;
  if (rc) return rc;
  if ((ix->pairs_ready || ix->screen_queries) && (rc = build_bitmaps(ix))) return rc;
  CHK(hipStreamSynchronize(s), "build_index");
  // sort scratch is re-grown on demand by the joins
  ss.k1.release();
  ss.k2.release();
  ss.v64a.release();
  ss.v64b.release();
  ss.v32a.release();
  ss.v32b.release();
  return APSS_OK;
}

template <typename T>
int copy_buf(Arena& a, DBuf<T>& dst, const DBuf<T>& src, int64_t count, hipStream_t s) {
  CHK(dst.take(a, count), "alloc");
  if (count > 0) CHK(hipMemcpyAsync(dst.p, src.p, sizeof(T) * count, hipMemcpyDeviceToDevice, s), "copy");
  return APSS_OK;
}

// The head-cut index of the screened join: the same rank-space rows, with
// every row's unindexed part set to its components of rank < head.
int build_screen(apss_index* ix, int32_t head, const uint32_t* cnt_r, Arena& tmp) {
  apss_index* sx = new (std::nothrow) apss_index();
  if (!sx) {
    set_error("host allocation failed");
    return APSS_ENOMEM;
  }
  ix->screen = sx;
  hipStream_t s = ix->ws.stream;
  sx->device = ix->device;
  sx->opts = ix->opts;
  sx->opts.screen_dims = 0;
  sx->ws.stream = s;
  sx->n = ix->n;
  sx->m = ix->m;
  sx->nnz = ix->nnz;
  sx->t_build = ix->t_build;
  sx->variant = ix->variant;
  sx->range_rows = ix->range_rows;
  sx->range_group = ix->range_group;
  sx->default_geometry = ix->default_geometry;
  sx->head_cut = head;
  sx->rows.n = ix->rows.n;
  sx->rows.nnz = ix->rows.nnz;
  sx->rows.rp_host = ix->rows.rp_host;
  int rc;
  if ((rc = copy_buf(sx->mem, sx->rows.rp, ix->rows.rp, ix->n + 1, s))) return rc;
  if ((rc = copy_buf(sx->mem, sx->rows.rc, ix->rows.rc, ix->nnz, s))) return rc;
  if ((rc = copy_buf(sx->mem, sx->mw_r, ix->mw_r, ix->m, s))) return rc;
  return build_lists(sx, cnt_r, tmp);
}

// Query tiles: consecutive queries, at most QT of them and, unless a single
// query is larger, at most QB components, so that a tile fits the LDS staging.
Tiles make_tiles(const int64_t* rp, int64_t n, int QT, int QB) {
  Tiles T;
  T.start.push_back(0);
  int64_t nnz = 0;
  for (int64_t q = 0; q < n; ++q) {
    const int64_t len = rp[q + 1] - rp[q];
    const int64_t cur = T.start.back();
    if (q > cur && (q - cur == QT || nnz + len > QB)) {
      T.max_nnz = std::max(T.max_nnz, nnz);
      T.start.push_back(q);
      nnz = 0;
    }
    nnz += len;
  }
  T.max_nnz = std::max(T.max_nnz, nnz);
  T.start.push_back(n);
  return T;
}

}  // namespace

namespace apss {

int64_t default_range_rows(int variant) {
  int qt = 0, cb = 1024;
  (void)join_variant_geometry(variant, &qt, &cb);
  // 16,384 rows: the measured best for the self-join and for query batches
  // on corpora of 0.5-2M vectors (the autotuner refines it per workload)
  return (int64_t)std::max(1, 16384 / cb) * cb;
}

int prepare(apss_index* ix, hipStream_t s, int variant, int64_t range_rows) {
  int qt = 0, cb = 0;
  if (join_variant_geometry(variant, &qt, &cb)) {
    set_error("unknown join variant %d", variant);
    return APSS_EINVAL;
  }
  const int64_t K = std::max<int64_t>(1, range_rows / cb);
  range_rows = K * cb;
  std::lock_guard<std::mutex> lock(ix->prep_mu);
  bool built = false;
  const int slot = hoff_slot(cb);
  if (!ix->hoff[slot].p) {
    const int64_t nb = (ix->n + cb - 1) / cb;
    const int64_t words = (nb + 1) * (int64_t)ix->H;
    CHK(ix->building ? ix->hoff[slot].take(ix->mem, words) : ix->hoff[slot].alloc(words), "alloc block offsets");
    CHK(launch_block_offsets(ix->off.p, ix->post.p, ix->H, nb, cb, ix->hoff[slot].p, s), "block offsets");
    ix->hoff_nb[slot] = nb;
    built = true;
  }
  if (!ix->toff.p || ix->toff_rows != range_rows) {
    const int64_t nb = (ix->n + cb - 1) / cb;
    const int64_t nR = (nb + K - 1) / K;
    const int64_t words = (nR + 1) * std::max<int64_t>(ix->m - ix->H, 1);
    CHK(ix->building ? ix->toff.take(ix->mem, words) : ix->toff.alloc(words), "alloc range offsets");
    CHK(launch_range_offsets(ix->off.p, ix->post.p, ix->H, ix->m, nR, range_rows, ix->toff.p, s), "range offsets");
    ix->toff_rows = range_rows;
    ix->toff_nR = nR;
    built = true;
  }
  if (!ix->grid[variant]) ix->grid[variant] = join_resident_groups(variant, ix->opts.remscore != 0);
  // other streams read the tables as soon as the lock is released
  if (built) CHK(hipStreamSynchronize(s), "prepare");
  return APSS_OK;
}

int plan_layout(apss_index* ix, const QuerySet& Q, int triangle, JoinLayout& L) {
  const int variant = ix->variant;
  if (join_variant_geometry(variant, &L.QT, &L.CB)) {
    set_error("unknown join variant %d", variant);
    return APSS_EINVAL;
  }
  L.variant = variant;
  L.slot = hoff_slot(L.CB);
  L.nb = ix->hoff_nb[L.slot];
  // work items: ranges of K blocks x query tiles
  const int64_t range_rows = ix->toff_rows;
  L.K = (int)(range_rows / L.CB);
  L.nR = ix->toff_nR;
  L.rg = std::max(1, std::min<int>(ix->range_group, kMaxRangeGroup));
  L.tiles = make_tiles(Q.rp_host, Q.n, L.QT, join_variant_staging(variant));
  L.ntiles = (int64_t)L.tiles.start.size() - 1;
  const int64_t ngroups = (L.nR + L.rg - 1) / L.rg;
  L.nrx = (ngroups + 7) / 8;
  L.parts = ix->parts;
  L.cum.assign((size_t)(8 * (L.nrx + 1)), 0);
  for (int x = 0; x < 8; ++x) {
    int64_t c = 0;
    for (int64_t j = 0; j <= L.nrx; ++j) {
      L.cum[(size_t)(x * (L.nrx + 1) + j)] = c;
      const int64_t g = x + 8 * j;
      const int64_t R = g * L.rg;  // the group's first range
      if (j < L.nrx && g < ngroups) {
        // first tile whose last query reaches the group's first range (self-join triangle)
        const int64_t tmin =
            triangle ? (int64_t)(std::upper_bound(L.tiles.start.begin() + 1, L.tiles.start.end(), R * range_rows) -
                                 (L.tiles.start.begin() + 1))
                     : 0;
        c += (L.ntiles - tmin) * L.parts;
      }
    }
  }
  // no more workgroups than work items: a small batch leaves the rest of
  // the device to work running beside it (another serving slot)
  int64_t items = 0;
  for (int x = 0; x < 8; ++x) items += L.cum[(size_t)(x * (L.nrx + 1) + L.nrx)];
  L.G = (int)std::max<int64_t>(1, std::min<int64_t>(ix->grid[variant], items));
  // per-workgroup cursor space for tiles too large to stage in LDS
  L.wg_stride = 2 * std::max<int64_t>(L.tiles.max_nnz, 1);
  return APSS_OK;
}

void bind_plan(apss_index* ix, const QuerySet& Q, int triangle, float t, const float* qt_dev, const RowStat* qrs,
               const JoinLayout& L, const int64_t* tstart_dev, const int64_t* qcum_dev, unsigned int* qctr_dev,
               uint32_t* wg_cur_dev, JoinPlan& P) {
  JoinArgs& a = P.a;
  a = JoinArgs{};
  a.rp = ix->rows.rp.p;
  a.rc = ix->rows.rc.p;
  a.rs = ix->rs.p;
  a.pnrm_max = ix->pnrm_max;
  a.pn8 = ix->pn8.p;
  a.off = ix->off.p;
  a.post = ix->post.p;
  a.post4 = ix->post4.p;
  a.post4_bytes = (uint32_t)(4 * (ix->P + kPost4Pad));
  a.hoff = ix->hoff[L.slot].p;
  a.H = ix->H;
  a.nb = L.nb;
  a.n = ix->n;
  a.qrp = Q.rp;
  a.qrc = Q.rc;
  a.qmw = Q.mw;
  a.qrs = qrs;
  a.qt = qt_dev;
  a.t = t;
  a.nq = Q.n;
  a.triangle = triangle;
  a.ntiles = L.ntiles;
  a.tstart = tstart_dev;
  a.toff = ix->toff.p;
  a.m_tail = (int32_t)(ix->m - ix->H);
  a.K = L.K;
  a.rg = L.rg;
  a.nR = (int32_t)L.nR;
  a.nrx = L.nrx;
  a.qcum = qcum_dev;
  a.qctr = qctr_dev;
  a.wg_cur = wg_cur_dev;
  a.wg_cur_stride = L.wg_stride;
  a.parts = L.parts;
  a.part_lo = L.parts > 1 ? ix->part_lo.p : nullptr;
  a.qadm = nullptr;
  P.variant = L.variant;
  P.G = L.G;
  P.bj = ceil_log2((uint64_t)ix->n);
  P.bi = ceil_log2((uint64_t)(triangle ? ix->n : Q.n));
  a.bj = P.bj;
}

int plan_join(apss_index* ix, Workspace& ws, const QuerySet& Q, int triangle, float t, const float* qt_dev,
              const RowStat* qrs, JoinPlan& P) {
  hipStream_t s = ws.stream;
  int rc0 = prepare(ix, s, ix->variant, ix->range_rows);
  if (rc0) return rc0;
  if (triangle && use_pairs(ix)) {
    if (int rc = reserve_control(ws)) return rc;
    // (a smaller queue where memory is short: it is filled more often)
    int64_t entries = pair_queue_entries(ix);
    hipError_t e = ws.pq.reserve(3 * entries);
    while (e != hipSuccess && (entries /= 4) >= (1 << 16)) {
      (void)hipGetLastError();
      e = ws.pq.reserve(3 * entries);
    }
    CHK(e, "alloc queues");
    bind_pairs(ix, t, ws.qctr, ws.pq.p, ws.pq.n / 3, P);
    return APSS_OK;
  }
  JoinLayout L;
  if ((rc0 = plan_layout(ix, Q, triangle, L))) return rc0;
  CHK(ws.tstart.reserve(L.ntiles + 1), "alloc tiles");
  CHK(hipMemcpyAsync(ws.tstart.p, L.tiles.start.data(), sizeof(int64_t) * (L.ntiles + 1), hipMemcpyHostToDevice, s),
      "tiles");
  CHK(ws.qcum.reserve((int64_t)L.cum.size()), "alloc queues");
  CHK(hipMemcpyAsync(ws.qcum.p, L.cum.data(), sizeof(int64_t) * L.cum.size(), hipMemcpyHostToDevice, s), "queues");
  if (int rc = reserve_control(ws)) return rc;
  CHK(ws.wg_cur.reserve((int64_t)L.G * L.wg_stride), "alloc cursors");
  bind_plan(ix, Q, triangle, t, qt_dev, qrs, L, ws.tstart.p, ws.qcum.p, ws.qctr, ws.wg_cur.p, P);
  return APSS_OK;
}

bool use_pairs(const apss_index* ix) { return ix->pairs_ready && !ix->pairs_off; }

// Twice the survivors that the sample foretells for the lowest threshold, up
// to kPairQueueMost entries of 12 bytes.
int64_t pair_queue_entries(const apss_index* ix) {
  return (int64_t)std::min(2.0 * ix->pair_survivors + 65536.0, (double)kPairQueueMost);
}

// Turns that a queue of qcap entries is filled in, where it does not hold one
// and a half times those survivors.  What is past a full queue is decided from
// memory, some 4 us a pair and wave: 60,000 rows of mean 80 at t = 0.5, 5
// million pairs' room in the fixed scratch beside 0.4 of 6 million survivors,
// took 54 ms where the accumulating kernel takes 11.3, in turns 5.2; 300,000
// such rows, 64M entries for 150 million, 645 ms, 266 and 102.  Turns cost
// little (150,000 rows in two 27.1 ms, in one 26.3, by 16M entries 29.5;
// 1,000,000 of mean 120 at 0.7 in two 293.3, in one 291.4).
int64_t pair_turns(const apss_index* ix, int64_t qcap) {
  return qcap > 0 ? 1 + (int64_t)((1.5 * ix->pair_survivors) / (double)qcap) : 1;
}

// The index's part of a candidate count.
void bind_count(apss_index* ix, CountArgs& c) {
  c = CountArgs{};
  c.bm = ix->bm.p;
  c.HB = ix->count_ranks;
  c.off = ix->off.p;
  c.n = ix->n;
  c.nblk = ix->count_blocks;
  c.post = ix->post.p;
  c.post4 = ix->post4.p;
  c.seg = ix->seg.p;
  c.H = ix->H;
  c.toff = ix->toff.p;
  c.m_tail = (int32_t)(ix->m - ix->H);
  c.rr = ix->toff_rows;
  c.nR = ix->toff_nR;
  c.present = ix->present.p;
  c.present_words = ix->present_words;
  c.lds_ranks = kLdsRanks;
}

void bind_pairs(apss_index* ix, float t, unsigned int* uctr_dev, uint32_t* queue_dev, int64_t qcap, JoinPlan& P) {
  P = JoinPlan{};
  P.pairs = true;
  P.bj = ceil_log2((uint64_t)ix->n);
  P.bi = P.bj;
  P.pg = ix->pair_groups;
  PairArgs& a = P.pa;
  a.rp = ix->rows.rp.p;
  a.rc = ix->rows.rc.p;
  a.sk = ix->sk.p;
  a.gid = ix->gid.p;
  a.fidx = ix->fidx.p;
  a.fsk = ix->fsk.p;
  a.qrp = a.rp;
  a.qrc = a.rc;
  a.qfidx = a.fidx;
  a.qfsk = a.fsk;
  a.dl = ix->dl.p;
  a.doff = ix->doff.p;
  a.dlr = ix->dlr.p;
  a.ndeep = ix->ndeep;
  a.wide = ix->wide.p;
  a.shorts = ix->shorts.p;
  a.nwide = ix->nwide;
  a.nshort = ix->nshort;
  a.uctr = uctr_dev;
  a.queue = queue_dev;
  a.qcap = qcap;
  a.turns = pair_turns(ix, qcap);
  a.t = t;
  a.thr = pair_threshold(t);
  a.bj = P.bj;
  bind_count(ix, P.ca);
  CountArgs& c = P.ca;
  c.rp = a.rp;
  c.rc = a.rc;
  c.skip = ix->head_cut > 0 ? ix->rs.p : nullptr;
  c.nq = ix->n;
  c.triangle = 1;
  c.chunk = count_chunk(ix->n, ix->count_blocks);
  if (c.chunk <= kPieceRows) c.lds_ranks = 0;
}

// True when a batch of nq queries takes the few-query kernel: default
// algorithm and geometry, and list offsets at its row bounds.
bool takes_few(const apss_index* ix, int64_t nq) {
  return nq <= kFewQueries && ix->opts.reserved[0] != kProbePairs && ix->parts == 1 && !ix->opts.remscore &&
         ix->head_cut == 0 && ix->default_geometry &&
         ix->toff_rows > 0 && ix->toff_rows % kFewRows == 0;
}

int plan_few(apss_index* ix, Workspace& ws, const QuerySet& Q, float t, const float* qt_dev, JoinPlan& P) {
  if (int rc = reserve_control(ws)) return rc;
  P = JoinPlan{};
  P.few = true;
  P.bj = ceil_log2((uint64_t)ix->n);
  P.bi = ceil_log2((uint64_t)Q.n);
  const int slot = ix->hoff[0].p ? 0 : 1;
  FewArgs& a = P.fa;
  a.rp = ix->rows.rp.p;
  a.rc = ix->rows.rc.p;
  a.rs = ix->rs.p;
  a.pn8 = ix->pn8.p;
  a.n = ix->n;
  a.post = ix->post.p;
  a.hoff = ix->hoff[slot].p;
  a.H = ix->H;
  a.cb = slot == 0 ? 1024 : 2048;
  a.nb = ix->hoff_nb[slot];
  a.toff = ix->toff.p;
  a.m_tail = ix->m - ix->H;
  a.rr = ix->toff_rows;
  a.nR = ix->toff_nR;
  a.qrp = Q.rp;
  a.qrc = Q.rc;
  a.qmw = Q.mw;
  a.qt = qt_dev;
  a.t = t;
  a.nq = Q.n;
  a.bj = P.bj;
  return APSS_OK;
}

// Share of a query's pairs expected to survive the sketch test at t.
double survivor_rate(const apss_index* ix, float t) {
  const int32_t lo = pair_threshold(ix->t_build), hi = pair_threshold(1.0f);
  const int b = (int)((double)(pair_threshold(t) - lo) * kRateBins / (double)(hi - lo + 1));
  return ix->rate[std::max(0, std::min(kRateBins - 1, b))];
}

// Bytes of the sketches of a batch: every row's, long rows' fine ones, and
// which of those a row has.
int64_t sketch_bytes(const QuerySet& Q) {
  int64_t longs = 0;
  for (int64_t q = 0; q < Q.n; ++q) longs += Q.rp_host[q + 1] - Q.rp_host[q] > kFineRow;
  return Q.n * kMidGroups + longs * kFineGroups + Q.n * (int64_t)sizeof(uint32_t);
}

// Sketches of the query rows, and the plan of testing them against the corpus.
// The sketches lie where the pair sort has its second values, after the tests.
int plan_queries(apss_index* ix, Workspace& ws, const QuerySet& Q, float t, const float* qt_dev, JoinPlan& P) {
  hipStream_t s = ws.stream;
  const int64_t bytes = sketch_bytes(Q);
  CHK(ws.ss.v32b.reserve((bytes + 3) / 4), "alloc sketches");
  uint8_t* const mid = (uint8_t*)ws.ss.v32b.p;
  uint8_t* const fsk = mid + Q.n * kMidGroups;
  uint32_t* const fidx = (uint32_t*)(mid + bytes) - Q.n;
  if (int rc = reserve_control(ws)) return rc;
  CHK(launch_sketch(Q.rp, Q.rc, ix->gid.p, Q.n, nullptr, mid, ws.nfine, fidx, fsk, s), "sketches");
  P = JoinPlan{};
  P.query = true;
  P.bj = ceil_log2((uint64_t)ix->n);
  P.bi = ceil_log2((uint64_t)Q.n);
  P.pg = ix->pair_groups;
  PairArgs& a = P.pa;
  a.rp = ix->rows.rp.p;
  a.rc = ix->rows.rc.p;
  a.gid = ix->gid.p;
  a.fidx = ix->fidx.p;
  a.fsk = ix->fsk.p;
  a.query = 1;
  a.qrp = Q.rp;
  a.qrc = Q.rc;
  a.qfidx = fidx;
  a.qfsk = fsk;
  a.qt = qt_dev;
  a.uctr = ws.qctr;
  a.t = t;
  a.bj = P.bj;
  QueryArgs& q = P.qa;
  q.sk = ix->mid.p;
  q.n = ix->n;
  q.qsk = mid;
  q.nq = Q.n;
  q.qstride = 1;
  q.qt = qt_dev;
  q.t = t;
  bind_count(ix, P.ca);
  CountArgs& c = P.ca;
  c.rp = Q.rp;
  c.rc = Q.rc;
  c.nq = Q.n;
  // a few work items per compute unit; where those are of few queries, of one
  // per wave, counted by pieces of rows (500,000 rows: 250 queries 424 -> 378
  // us, 600 592 -> 600; 1,000,000 rows: 150 queries 544 -> 460, 400 740 ->
  // 754; 200,000 rows: 400 queries 301 -> 263).  From 1,024 queries on, 64 of
  // a block's items (as many as run on an XCD at once) take the batch, so that
  // they share one block's bitmaps in its L2
  const int64_t want = Q.n >= 1024 ? std::max<int64_t>(64, Q.n / 64) : Q.n * ix->count_blocks / 1024;
  c.chunk = std::max<int64_t>(kPieceRows, std::min<int64_t>(4096, (want + 15) / 16 * 16));
  if (c.chunk < 64) {
    c.chunk = kPieceRows;
    c.lds_ranks = 0;
  }
  return APSS_OK;
}

// The caller has cleared the counters and queue counters.
int launch_plan(JoinPlan& P, uint64_t* out_key, float* out_sim, int64_t cap, unsigned long long* counters,
                unsigned int* qctr, hipStream_t s) {
  if (P.pairs) {
    P.pa.out_key = out_key;
    P.pa.out_sim = out_sim;
    P.pa.cap = cap;
    P.pa.counters = counters;
    P.ca.counters = counters;
    CHK(launch_count(P.ca, s), "count kernel");
    CHK(launch_pairs(P.pa, P.pg, s), "pair kernel");
    return APSS_OK;
  }
  if (P.query) {
    P.pa.out_key = out_key;
    P.pa.out_sim = out_sim;
    P.pa.cap = cap;
    P.pa.counters = counters;
    P.ca.counters = counters;
    for (size_t r = 0; r < P.qend.size(); ++r) {
      if (r > 0) CHK(fill_u32(qctr, 0u, kQueueCounters, s), "fill");
      QueryArgs q = P.qa;
      q.q0 = r > 0 ? P.qend[r - 1] : 0;
      q.nq = P.qend[r];
      CHK(launch_query_screen(P.pa, q, P.pg, s), "query kernel");
    }
    // (last: a batch whose survivors outgrew their queue is not counted here)
    CHK(launch_count(P.ca, s), "count kernel");
    return APSS_OK;
  }
  if (P.few) {
    P.fa.out_key = out_key;
    P.fa.out_sim = out_sim;
    P.fa.cap = cap;
    P.fa.counters = counters;
    CHK(launch_few(P.fa, s), "query kernel");
    return APSS_OK;
  }
  JoinArgs& a = P.a;
  a.out_key = out_key;
  a.out_sim = out_sim;
  a.cap = cap;
  a.counters = counters;
  a.qctr = qctr;
  if (!join_args_complete(a)) {
    set_error("internal: join launched with a missing device buffer");
    return APSS_EDEVICE;
  }
  CHK(launch_join(a, P.variant, P.G, s), "join kernel");
  return APSS_OK;
}

// Launch a planned join writing pairs into ws.raw_key / raw_sim through ws.counters.
int launch_planned(Workspace& ws, JoinPlan& P) {
  return launch_plan(P, ws.raw_key.p, ws.raw_sim.p, ws.raw_key.n, ws.counters.p, ws.qctr, ws.stream);
}

int reserve_control(Workspace& ws) {
  static_assert(kQueueCounters % 2 == 0, "control words");
  CHK(ws.counters.reserve(kControlWords), "alloc counters");
  ws.qctr = (unsigned int*)(ws.counters.p + C_NUM);
  ws.nfine = ws.qctr + kQueueCounters;
  return APSS_OK;
}

int ensure_pair_capacity(Workspace& ws, int64_t cap) {
  if (ws.raw_key.p && ws.raw_key.n >= cap) return APSS_OK;
  cap = std::max<int64_t>(cap, 1 << 16);
  CHK(ws.raw_key.alloc(cap), "alloc pairs");
  CHK(ws.raw_sim.alloc(cap), "alloc pairs");
  return APSS_OK;
}

int sort_pairs(Workspace& ws, int64_t matches, int key_bits) {
  SortScratch& ss = ws.ss;
  // 1.5x: after the sort this scratch holds the unpacked (i, j, sim) arrays
  // of finish_host, so that call never reallocates it under queued work
  CHK(ss.k2.reserve(matches + matches / 2 + 1), "alloc sort");
  CHK(ss.v32b.reserve(matches), "alloc sort");
  CHK(ss.hist.reserve(radix_hist_elems(matches)), "alloc sort");
  CHK(ss.scan.reserve(radix_scan_tmp_elems(matches)), "alloc sort");
  CHK(radix_sort_u64_u32(ws.raw_key.p, (uint32_t*)ws.raw_sim.p, ss.k2.p, ss.v32b.p, matches, key_bits, ss.hist.p,
                         ss.scan.p, ws.stream),
      "pair sort");
  return APSS_OK;
}

void take_counters(Workspace& ws, const unsigned long long* c) {
  ws.last.posting_visits = (int64_t)(c[C_VISITS] + c[C_TAILVISITS]);
  ws.last.candidates = (int64_t)c[C_CANDIDATES];
  ws.last.bound_survivors = (int64_t)c[C_SURVIVORS];
  ws.last.verified = (int64_t)c[C_VERIFIED];
  ws.last.band = (int64_t)c[C_BAND];
  ws.last.matches = (int64_t)c[C_MATCHES];
}

// Every call on a workspace starts here.  Any call other than a graph
// replay may rewrite buffers a captured graph reads, so it drops the graph.
int start_call(Workspace& ws, bool keep_graph = false) {
  if (!keep_graph) ws.graph.reset();
  memset(&ws.last, 0, sizeof(ws.last));
  for (int e = 0; e < 6; ++e)
    if (!ws.ev[e]) CHK(hipEventCreateWithFlags(&ws.ev[e], hipEventDefault), "event");
  CHK(hipEventRecord(ws.ev[0], ws.stream), "event");
  return APSS_OK;
}

int reserve_host(Workspace& ws) {
  if (ws.host_counters.reserve(kHostWords)) return APSS_OK;
  set_error("pinned host allocation failed");
  return APSS_ENOMEM;
}

int host_sink(Workspace& ws, Sink* sink) {
  if (int rc = reserve_host(ws)) return rc;
  sink->i = (uint32_t*)(ws.host_counters.p + C_NUM + 2);
  sink->j = sink->i + kFinishPairs;
  sink->sim = (float*)(sink->j + kFinishPairs);
  sink->room = kFinishPairs;
  return APSS_OK;
}

// After a join's kernels: its counters in ws.host_counters once the stream
// has drained, and the pairs at the sink if they are few.
int hand_over(Workspace& ws, int bj, int bits, const Sink* sink, const unsigned long long* checks = nullptr) {
  hipStream_t s = ws.stream;
  if (int rc = reserve_host(ws)) return rc;
  FinishArgs f{};
  f.key = ws.raw_key.p;
  f.sim = ws.raw_sim.p;
  f.cap = ws.raw_key.n;
  f.bj = bj;
  f.bits = bits;
  if (sink) {
    f.out_i = sink->i;
    f.out_j = sink->j;
    f.out_sim = sink->sim;
    f.room = std::max<int64_t>(sink->room, 0);  // (a negative capacity is refused by finish_device)
  }
  f.counters = ws.counters.p;
  f.checks = checks;
  f.host = ws.host_counters.p;
  CHK(launch_finish(f, s), "finish kernel");
  CHK(hipEventRecord(ws.ev[3], s), "event");
  return APSS_OK;
}

int run_join(apss_index* ix, Workspace& ws, const QuerySet& Q, int triangle, float t, const float* qt_dev,
             int64_t cap_hint, int64_t* count, const float* t_host, Sink* sink) {
  hipStream_t s = ws.stream;
  *count = 0;
  // what the staging of a batch of queries leaves to this call, and to no other
  const unsigned long long* const checks = ws.pending;
  const bool cleared = ws.cleared;
  ws.pending = nullptr;
  ws.cleared = false;
  int rc = start_call(ws);
  if (rc) return rc;
  if (Q.n == 0) return APSS_OK;
  if (ix->n == 0) return checks ? check_err(s, checks, "query") : APSS_OK;
  if (!cleared) {
    if ((rc = reserve_control(ws))) return rc;
    CHK(fill_u64((uint64_t*)ws.counters.p, 0ull, kControlWords, s), "fill");
  }
  JoinPlan P;
  // A batch of queries takes the sketch kernels when they are expected to be
  // ahead at its thresholds, and again the accumulating kernel if more pairs
  // survive than the queue was sized for (twice those of the corpus's own
  // rows): the sketch kernels then end early (4,096 copies of one query, 2,000
  // of it among 1,000,000 rows: 21.1 ms, by the accumulating kernel alone 21.4,
  // where the whole tests and the count came first 23.2).  (More than 2^24
  // queries would need 4 GB of sketches.)
  const bool few = !triangle && takes_few(ix, Q.n);
  bool screen = !triangle && !few && ix->screen_queries && !ix->pairs_off && Q.n <= (1 << 24);
  if (screen) {
    double survivors = 0.0;
    for (int64_t q = 0; q < Q.n; ++q) survivors += survivor_rate(ix, t_host ? t_host[q] : t) * (double)ix->n;
    screen = ix->opts.reserved[0] == kProbePairs ||
             (double)Q.n * (double)ix->n * ix->screen_ps + kSurvivorPs * survivors <
                 (double)Q.n * (double)ix->n * ix->accumulate_ps;
    if (screen) {
      if ((rc = ensure_pair_capacity(ws, cap_hint))) return rc;
      // a server's slot holds no more than its batch's reservation: the sketches
      // fit the sort's second values (of pairs or components) or, where the rows
      // were sorted in LDS, those and the row sort's 24 bytes a component; else,
      // few pairs and rows of a few components, the accumulating kernel
      if (ws.slot)
        screen = sketch_bytes(Q) <=
                 (cleared ? 4 * ws.raw_key.n + 24 * Q.nnz : 4 * std::max<int64_t>(ws.raw_key.n, Q.nnz));
    }
    if (screen) {
      if ((rc = plan_queries(ix, ws, Q, t, qt_dev, P))) return rc;
      // survivor queue: in a server's slot the pair sort's second keys (part
      // of the batch's reservation, free until the sort), else its own buffer
      if (ws.slot) {
        CHK(ws.ss.k2.reserve(ws.raw_key.n + ws.raw_key.n / 2 + 1), "alloc sort");
        P.pa.queue = (uint32_t*)ws.ss.k2.p;
        P.pa.qcap = ws.raw_key.n;
      } else {
        const double want = std::min(2.0 * survivors + 65536.0, 16.0 * (1 << 20));
        CHK(ws.pq.reserve(3 * (int64_t)want), "alloc queues");
        P.pa.queue = ws.pq.p;
        P.pa.qcap = ws.pq.n / 3;
      }
      // runs of queries whose survivors fit the queue (whole tiles)
      double held = 0.0;
      for (int64_t q = 0; q < Q.n; q += kQueryTile) {
        double tile = 0.0;
        for (int64_t k = q; k < std::min<int64_t>(q + kQueryTile, Q.n); ++k)
          tile += 2.0 * survivor_rate(ix, t_host ? t_host[k] : t) * (double)ix->n;
        if (q > 0 && held + tile > (double)P.pa.qcap) {
          P.qend.push_back(q);
          held = 0.0;
        }
        held += tile;
      }
      P.qend.push_back(Q.n);
    }
  }
  if (!screen) {
    rc = few ? plan_few(ix, ws, Q, t, qt_dev, P) : plan_join(ix, ws, Q, triangle, t, qt_dev, nullptr, P);
    if (rc) return rc;
    if ((rc = ensure_pair_capacity(ws, cap_hint))) return rc;
  }
  if (ix->opts.remscore) {
    // each query's first component that admits new candidates (remscore)
    CHK(ws.qadm.reserve(Q.n), "alloc");
    CHK(launch_admit_pos(Q.rp, Q.rc, ix->mw_r.p, qt_dev, t, Q.n, ws.qadm.p, s), "admission");
    P.a.qadm = ws.qadm.p;
  }
  for (int attempt = 0; attempt < 3; ++attempt) {  // (once more with the other kernel, once with more room)
    if (attempt > 0) CHK(fill_u64((uint64_t*)ws.counters.p, 0ull, kControlWords, s), "fill");
    CHK(hipEventRecord(ws.ev[1], s), "event");
    if ((rc = launch_planned(ws, P))) return rc;
    CHK(hipEventRecord(ws.ev[2], s), "event");
    // (a pair that several parts keep is still there several times)
    const Sink* to = P.a.parts > 1 ? nullptr : sink;
    if ((rc = hand_over(ws, P.bj, P.bi + P.bj, to, checks))) return rc;
    CHK(hipStreamSynchronize(s), "join");
    const unsigned long long* const c = ws.host_counters.p;
    if (checks && (rc = check_bits((uint32_t)c[C_NUM], c[C_NUM + 1], "query"))) return rc;
    if (screen && c[C_OVERFLOW]) {
      screen = false;
      P = JoinPlan{};
      if ((rc = plan_join(ix, ws, Q, triangle, t, qt_dev, nullptr, P))) return rc;
      continue;
    }
    const int64_t matches = (int64_t)c[C_MATCHES];
    if (matches > ws.raw_key.n) {
      if ((rc = ensure_pair_capacity(ws, matches + matches / 8 + 1024))) return rc;
      ++ws.regrows;
      continue;  // rerun with room for every pair
    }
    take_counters(ws, c);
    float ms = 0.0f;
    CHK(hipEventElapsedTime(&ms, ws.ev[1], ws.ev[2]), "event");
    ws.last.ms_candidates = ms;
    if (to && finish_delivers(matches, ws.raw_key.n, to->room)) {
      sink->done = true;
      *count = matches;
      return APSS_OK;
    }
    if ((rc = sort_pairs(ws, matches, P.bi + P.bj))) return rc;
    int64_t distinct = matches;
    if (P.a.parts > 1 && matches > 1) {
      // a pair kept by several parts was emitted once by each, with the same
      // rescored similarity: keep one copy
      SortScratch& ss = ws.ss;
      CHK(ss.v64a.reserve(matches), "alloc");
      CHK(ss.v64b.reserve(scan_tmp_elems(matches)), "alloc");
      CHK(ws.uniq_total.reserve(1), "alloc");
      CHK(unique_sorted_u64_u32(ws.raw_key.p, (uint32_t*)ws.raw_sim.p, matches, (int64_t*)ss.v64a.p,
                                (int64_t*)ss.v64b.p, ws.uniq_total.p, ss.k2.p, ss.v32b.p, s),
          "unique pairs");
      CHK(hipMemcpyAsync(&distinct, ws.uniq_total.p, sizeof(int64_t), hipMemcpyDeviceToHost, s), "unique pairs");
      CHK(hipStreamSynchronize(s), "unique pairs");
      ws.last.matches = distinct;
    }
    *count = distinct;
    return APSS_OK;
  }
  set_error("pair buffer kept overflowing");
  return APSS_ENOMEM;
}

// Screened self-join: the bf16 MFMA head screen (pairs that share no tail
// dimension) and the sparse pass over the head-cut index (pairs that share
// one), written into one pair buffer and sorted together.
int run_screen_join(apss_index* ix, Workspace& ws, float t, int64_t cap_hint, int64_t* count, Sink* sink) {
  apss_index* sx = ix->screen;
  hipStream_t s = ws.stream;
  *count = 0;
  if (!screen_variant_ok(sx->variant)) {
    set_error("tile variant %d is not available for the screened join", sx->variant);
    return APSS_EINVAL;
  }
  int rc = start_call(ws);
  if (rc) return rc;
  const int64_t n = sx->n;
  if (n == 0) return APSS_OK;
  const int32_t head = sx->head_cut;
  const int32_t ld = (int32_t)((head + kScreenK - 1) / kScreenK * kScreenK);
  const int bj = ceil_log2((uint64_t)n);

  // rows whose head norm reaches t, by decreasing head norm
  CHK(ws.s_keys.reserve(n), "alloc screen");
  CHK(ws.s_cnt.reserve(1), "alloc screen");
  CHK(fill_u64((uint64_t*)ws.s_cnt.p, 0ull, 1, s), "fill");
  CHK(launch_screen_select(sx->rs.p, n, t, ws.s_keys.p, ws.s_cnt.p, s), "screen select");
  unsigned long long S64 = 0;
  CHK(hipMemcpyAsync(&S64, ws.s_cnt.p, sizeof(S64), hipMemcpyDeviceToHost, s), "screen select");
  CHK(hipStreamSynchronize(s), "screen select");
  const int64_t S = (int64_t)S64;
  const int64_t Sp = (S + kScreenTileB - 1) / kScreenTileB * kScreenTileB;
  int64_t nc = 0, ntiles = 0, useful = 0;
  if (S > 1) {
    SortScratch& ss = ws.ss;
    CHK(ss.k2.reserve(S), "alloc sort");
    CHK(ss.v32a.reserve(S), "alloc sort");
    CHK(ss.v32b.reserve(S), "alloc sort");
    CHK(ss.hist.reserve(radix_hist_elems(S)), "alloc sort");
    CHK(ss.scan.reserve(radix_scan_tmp_elems(S)), "alloc sort");
    CHK(radix_sort_u64_u32(ws.s_keys.p, ss.v32a.p, ss.k2.p, ss.v32b.p, S, 64, ss.hist.p, ss.scan.p, s), "screen sort");
    CHK(ws.s_sid.reserve(Sp), "alloc screen");
    CHK(ws.s_nh.reserve(Sp), "alloc screen");
    CHK(launch_screen_unpack(ws.s_keys.p, S, Sp, ws.s_sid.p, ws.s_nh.p, s), "screen unpack");
    CHK(ws.s_X.reserve(Sp * ld), "alloc screen block");
    CHK(fill_u32((uint32_t*)ws.s_X.p, 0u, Sp * ld / 2, s), "fill");
    CHK(launch_screen_pack(sx->rows.rp.p, sx->rows.rc.p, ws.s_sid.p, S, head, ld, ws.s_X.p, s), "screen pack");
    // tiles (I, J) of kScreenTile x kScreenTileB rows that reach the upper
    // triangle (2 J + 1 >= I) and whose largest norm product reaches t (rows
    // are in decreasing head norm, so a tile's first rows have the largest);
    // `useful` counts the kScreenTile x kScreenTile pairs I <= J among them
    std::vector<float> nh((size_t)Sp);
    CHK(hipMemcpyAsync(nh.data(), ws.s_nh.p, sizeof(float) * Sp, hipMemcpyDeviceToHost, s), "screen norms");
    CHK(hipStreamSynchronize(s), "screen norms");
    const int64_t T = Sp / kScreenTile, TB = Sp / kScreenTileB;
    std::vector<int32_t> tl;
    for (int64_t I = 0; I < T; ++I) {
      const float nI = nh[(size_t)(I * kScreenTile)];
      for (int64_t J = I; J < T; ++J) {
        if (nI * nh[(size_t)(J * kScreenTile)] * (1.0f + 0x1p-20f) < t) break;
        ++useful;
      }
      for (int64_t J = I / 2; J < TB; ++J) {
        if (nI * nh[(size_t)(J * kScreenTileB)] * (1.0f + 0x1p-20f) < t) break;
        tl.push_back((int32_t)I);
        tl.push_back((int32_t)J);
      }
    }
    ntiles = (int64_t)tl.size() / 2;
    // blocks of kScreenBlock x kScreenBlock row tiles in turn: the
    // workgroups that run at once on an XCD then share a few panels of each
    // operand (from L2 and the last-level cache) instead of streaming a new
    // second operand panel per tile from HBM (C4 with 128 x 128 tiles:
    // 8.0 -> 6.6 ms; blocks of 4 and 16 within 0.1 ms of 8, of 32 7.5 ms)
    {
      const int B = kScreenBlock;
      if (B > 1) {
        std::vector<std::array<int32_t, 4>> key((size_t)ntiles);
        for (int64_t k = 0; k < ntiles; ++k) {
          const int32_t I = tl[(size_t)(2 * k)], J = tl[(size_t)(2 * k + 1)];
          key[(size_t)k] = {I / B, J / (B * kScreenTile / kScreenTileB), I, J};
        }
        std::sort(key.begin(), key.end());
        for (int64_t k = 0; k < ntiles; ++k) {
          tl[(size_t)(2 * k)] = key[(size_t)k][2];
          tl[(size_t)(2 * k + 1)] = key[(size_t)k][3];
        }
      }
    }
    if (ntiles > 0) {
      CHK(ws.s_tiles.reserve((int64_t)tl.size()), "alloc screen");
      CHK(hipMemcpyAsync(ws.s_tiles.p, tl.data(), sizeof(int32_t) * tl.size(), hipMemcpyHostToDevice, s),
          "screen tiles");
      CHK(ws.s_cand.reserve(std::max<int64_t>(1 << 16, 4 * S)), "alloc screen");
      for (int attempt = 0; attempt < 2; ++attempt) {
        CHK(fill_u64((uint64_t*)ws.s_cnt.p, 0ull, 1, s), "fill");
        ScreenArgs A{};
        A.X = ws.s_X.p;
        A.ld = ld;
        A.nh = ws.s_nh.p;
        A.sid = ws.s_sid.p;
        A.tiles = ws.s_tiles.p;
        A.ntiles = ntiles;
        A.t = t;
        A.bj = bj;
        A.out = ws.s_cand.p;
        A.cap = ws.s_cand.n;
        A.count = ws.s_cnt.p;
        CHK(hipEventRecord(ws.ev[4], s), "event");
        CHK(launch_screen_mfma(A, s), "screen kernel");
        CHK(hipEventRecord(ws.ev[5], s), "event");
        unsigned long long c = 0;
        CHK(hipMemcpyAsync(&c, ws.s_cnt.p, sizeof(c), hipMemcpyDeviceToHost, s), "screen count");
        CHK(hipStreamSynchronize(s), "screen kernel");
        nc = (int64_t)c;
        if (nc > ws.s_cand.n) {
          CHK(ws.s_cand.alloc(nc + nc / 8 + 1024), "alloc screen");
          continue;
        }
        float ms = 0.0f;
        CHK(hipEventElapsedTime(&ms, ws.ev[4], ws.ev[5]), "event");
        ws.last.ms_screen = ms;
        break;
      }
      if (nc > ws.s_cand.n) {
        set_error("screen candidate buffer kept overflowing");
        return APSS_ENOMEM;
      }
    }
  }

  // sparse pass over the head-cut index, then the exact check of the screen's candidates
  JoinPlan P;
  if ((rc = plan_join(sx, ws, QuerySet{sx->rows.rp.p, sx->rows.rc.p, sx->rows.mw.p, n, sx->nnz,
                                       sx->rows.rp_host.data()},
                      1, t, nullptr, sx->rs.p, P)))
    return rc;
  if ((rc = ensure_pair_capacity(ws, cap_hint))) return rc;
  for (int attempt = 0; attempt < 2; ++attempt) {
    CHK(fill_u64((uint64_t*)ws.counters.p, 0ull, kControlWords, s), "fill");
    CHK(hipEventRecord(ws.ev[1], s), "event");
    if ((rc = launch_planned(ws, P))) return rc;
    CHK(hipEventRecord(ws.ev[2], s), "event");
    CHK(launch_screen_verify(ws.s_cand.p, nc, bj, sx->rows.rp.p, sx->rows.rc.p, head, t, ws.raw_key.p, ws.raw_sim.p,
                             ws.raw_key.n, ws.counters.p, s),
        "screen verify");
    if ((rc = hand_over(ws, bj, 2 * bj, sink))) return rc;
    CHK(hipStreamSynchronize(s), "join");
    const unsigned long long* const c = ws.host_counters.p;
    const int64_t matches = (int64_t)c[C_MATCHES];
    if (matches > ws.raw_key.n) {
      if ((rc = ensure_pair_capacity(ws, matches + matches / 8 + 1024))) return rc;
      ++ws.regrows;
      continue;
    }
    const double ms_screen = ws.last.ms_screen;
    take_counters(ws, c);
    ws.last.ms_screen = ms_screen;
    ws.last.screen_rows = S;
    ws.last.screen_tiles = useful;
    ws.last.screen_candidates = nc;
    ws.last.screen_ld = ld;
    float ms = 0.0f;
    CHK(hipEventElapsedTime(&ms, ws.ev[1], ws.ev[2]), "event");
    ws.last.ms_candidates = ms;
    *count = matches;
    if (sink && finish_delivers(matches, ws.raw_key.n, sink->room)) sink->done = true;
    else if ((rc = sort_pairs(ws, matches, 2 * bj))) return rc;
    return APSS_OK;
  }
  set_error("pair buffer kept overflowing");
  return APSS_ENOMEM;
}

}  // namespace apss

namespace {

// Pair capacity a self-join starts with (grows on overflow, which reruns
// the join kernel): 32 pairs per vector, 384 MB of pair buffers per million
// vectors, which holds the matches of the million-vector workloads at their
// thresholds (about 22 per vector at t = 0.7) on the first call.
int64_t join_cap_hint(const apss_index* ix) { return std::max<int64_t>(1 << 20, 32 * ix->n); }

std::vector<const void*> graph_buffers(const apss_index* ix, const Workspace& ws) {
  return {ws.tstart.p, ws.qcum.p, ws.qctr, ws.counters.p, ws.wg_cur.p, ws.pq.p, ws.raw_key.p, ws.raw_sim.p, ws.ss.k2.p,
          ws.ss.v32b.p, ws.ss.hist.p, ws.ss.scan.p, ix->toff.p, ix->hoff[0].p, ix->hoff[1].p,
          (const void*)(intptr_t)ix->variant, (const void*)(intptr_t)ix->range_rows,
          (const void*)(intptr_t)ix->range_group};
}

// Capture the launch sequence of the self-join that just ran (count pairs).
int capture_join_graph(apss_index* ix, float t, uint32_t* out_i, uint32_t* out_j, float* out_sim, int64_t capacity,
                       int64_t cnt) {
  Workspace& ws = ix->ws;
  JoinGraph& g = ws.graph;
  hipStream_t s = ws.stream;
  g.reset();
  if (!s) return APSS_OK;  // the legacy default stream cannot be captured
  if (!g.hctr) CHK(hipHostMalloc((void**)&g.hctr, sizeof(unsigned long long) * (C_NUM + 2), hipHostMallocDefault),
                   "pinned counters");
  JoinPlan P;
  int rc = plan_join(ix, ws, QuerySet{ix->rows.rp.p, ix->rows.rc.p, ix->rows.mw.p, ix->n, ix->nnz,
                                      ix->rows.rp_host.data()},
                     1, t, nullptr, nullptr, P);
  if (rc) return rc;
  CHK(hipStreamSynchronize(s), "graph capture");
  CHK(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal), "graph capture");
  auto body = [&]() -> int {
    CHK(fill_u64((uint64_t*)ws.counters.p, 0ull, kControlWords, s), "fill");
    int r = launch_planned(ws, P);
    if (r) return r;
    if (finish_delivers(cnt, ws.raw_key.n, capacity)) {
      const FinishArgs f{ws.raw_key.p, ws.raw_sim.p, ws.raw_key.n, P.bj,          P.bi + P.bj, out_i,
                         out_j,        out_sim,      capacity,     ws.counters.p, nullptr,     g.hctr};
      CHK(launch_finish(f, s), "finish kernel");
      return APSS_OK;
    }
    CHK(hipMemcpyAsync(g.hctr, ws.counters.p, sizeof(unsigned long long) * C_NUM, hipMemcpyDeviceToHost, s),
        "read counters");
    if ((r = sort_pairs(ws, cnt, P.bi + P.bj))) return r;
    CHK(launch_unpack_pairs(ws.raw_key.p, ws.raw_sim.p, cnt, P.bj, out_i, out_j, out_sim, s), "unpack");
    return APSS_OK;
  };
  rc = body();
  hipGraph_t graph = nullptr;
  const hipError_t ee = hipStreamEndCapture(s, &graph);
  if (!rc && ee != hipSuccess) rc = dev_err(ee, "graph capture");
  if (!rc) {
    const hipError_t ei = hipGraphInstantiate(&g.exec, graph, nullptr, nullptr, 0);
    if (ei != hipSuccess) {
      g.exec = nullptr;
      rc = dev_err(ei, "graph instantiate");
    }
  }
  if (graph) (void)hipGraphDestroy(graph);
  if (rc) return rc;
  g.t = t;
  g.out[0] = out_i;
  g.out[1] = out_j;
  g.out[2] = out_sim;
  g.capacity = capacity;
  g.count = cnt;
  g.baked = graph_buffers(ix, ws);
  return APSS_OK;
}

// apss_join_device with graph replay (plain self-join).
int graph_join(apss_index* ix, float t, uint32_t* out_i, uint32_t* out_j, float* out_sim, int64_t capacity,
               int64_t* count) {
  Workspace& ws = ix->ws;
  JoinGraph& g = ws.graph;
  hipStream_t s = ws.stream;
  int rc;
  if (g.exec && g.t == t && g.out[0] == out_i && g.out[1] == out_j && g.out[2] == out_sim &&
      g.capacity == capacity && g.baked == graph_buffers(ix, ws)) {
    if ((rc = start_call(ws, true))) return rc;
    CHK(hipEventRecord(ws.ev[1], s), "event");
    CHK(hipGraphLaunch(g.exec, s), "graph launch");
    CHK(hipEventRecord(ws.ev[2], s), "event");
    CHK(hipStreamSynchronize(s), "graph launch");
    if ((int64_t)g.hctr[C_MATCHES] == g.count) {
      take_counters(ws, g.hctr);
      float ms = 0.0f;
      CHK(hipEventElapsedTime(&ms, ws.ev[1], ws.ev[2]), "event");
      ws.last.ms_candidates = ms;
      CHK(hipEventElapsedTime(&ms, ws.ev[0], ws.ev[2]), "event");
      ws.last.ms_total = ms;
      *count = g.count;
      return APSS_OK;
    }
    g.reset();  // cannot happen for a deterministic join; recompute eagerly
  }
  int64_t cnt = 0;
  Sink sink{out_i, out_j, out_sim, capacity};
  if ((rc = run_join(ix, ws, QuerySet{ix->rows.rp.p, ix->rows.rc.p, ix->rows.mw.p, ix->n, ix->nnz,
                                      ix->rows.rp_host.data()},
                     1, t, nullptr, join_cap_hint(ix), &cnt, nullptr, &sink)))
    return rc;
  if ((rc = finish_device(ws, cnt, ceil_log2((uint64_t)ix->n), sink, count))) return rc;
  const apss_stats keep = ws.last;
  rc = capture_join_graph(ix, t, out_i, out_j, out_sim, capacity, cnt);
  ws.last = keep;
  return rc;
}

}  // namespace

namespace apss {

int check_t(const apss_index* ix, float t) {
  if (!(t > 0.0f && t <= 1.0f)) {
    set_error("threshold %g outside (0, 1]", (double)t);
    return APSS_ETHRESH;
  }
  if (t < ix->t_build) {
    set_error("threshold %g below the index build threshold %g", (double)t, (double)ix->t_build);
    return APSS_ETHRESH;
  }
  return APSS_OK;
}

// wait = false leaves the stream running; the caller synchronises and then
// calls record_total.
int record_total(Workspace& ws) {
  float ms = 0.0f;
  CHK(hipEventElapsedTime(&ms, ws.ev[0], ws.ev[3]), "event");
  ws.last.ms_total = ms;
  return APSS_OK;
}

int finish_device(Workspace& ws, int64_t cnt, int bj, const Sink& sink, int64_t* count, bool wait) {
  *count = cnt;
  if (cnt > sink.room) {
    set_error("output capacity %lld too small for %lld pairs", (long long)sink.room, (long long)cnt);
    return APSS_ERANGE;
  }
  if (sink.done) return record_total(ws);
  CHK(launch_unpack_pairs(ws.raw_key.p, ws.raw_sim.p, cnt, bj, sink.i, sink.j, sink.sim, ws.stream), "unpack");
  CHK(hipEventRecord(ws.ev[3], ws.stream), "event");
  if (!wait) return APSS_OK;
  CHK(hipStreamSynchronize(ws.stream), "unpack");
  return record_total(ws);
}

int finish_host(Workspace& ws, int64_t cnt, int bj, const Sink& sink, apss_pairs* out) {
  out->count = 0;
  out->i = out->j = nullptr;
  out->sim = nullptr;
  const size_t nb = (size_t)(cnt > 0 ? cnt : 1);
  out->i = (uint32_t*)malloc(nb * sizeof(uint32_t));
  out->j = (uint32_t*)malloc(nb * sizeof(uint32_t));
  out->sim = (float*)malloc(nb * sizeof(float));
  if (!out->i || !out->j || !out->sim) {
    free(out->i);
    free(out->j);
    free(out->sim);
    out->i = out->j = nullptr;
    out->sim = nullptr;
    (void)hipStreamSynchronize(ws.stream);
    set_error("host allocation failed");
    return APSS_ENOMEM;
  }
  if (sink.done) {  // already in pinned memory
    memcpy(out->i, sink.i, sizeof(uint32_t) * cnt);
    memcpy(out->j, sink.j, sizeof(uint32_t) * cnt);
    memcpy(out->sim, sink.sim, sizeof(float) * cnt);
    out->count = cnt;
    return record_total(ws);
  }
  // the sort's second key buffer is free once the pairs are sorted: unpack
  // there, i, j and sim one after another, so that one copy brings them over
  SortScratch& ss = ws.ss;
  CHK(ss.k2.reserve(cnt + cnt / 2 + 1), "alloc");
  uint32_t* di = (uint32_t*)ss.k2.p;
  uint32_t* dj = di + cnt;
  float* ds = (float*)(dj + cnt);
  int64_t c2 = 0;
  int rc = finish_device(ws, cnt, bj, Sink{di, dj, ds, cnt}, &c2, false);
  if (rc) {
    (void)hipStreamSynchronize(ws.stream);
    return rc;
  }
  // up to 4M pairs through the workspace's pinned staging in one copy;
  // larger results straight into the output arrays
  if (cnt && cnt <= (4ll << 20) && ws.host_out.reserve((size_t)(3 * cnt))) {
    CHK(hipMemcpyAsync(ws.host_out.p, di, sizeof(uint32_t) * 3 * cnt, hipMemcpyDeviceToHost, ws.stream), "copy out");
    CHK(hipStreamSynchronize(ws.stream), "copy out");
    memcpy(out->i, ws.host_out.p, sizeof(uint32_t) * cnt);
    memcpy(out->j, ws.host_out.p + cnt, sizeof(uint32_t) * cnt);
    memcpy(out->sim, ws.host_out.p + 2 * cnt, sizeof(float) * cnt);
  } else {
    if (cnt) {
      CHK(hipMemcpyAsync(out->i, di, sizeof(uint32_t) * cnt, hipMemcpyDeviceToHost, ws.stream), "copy out");
      CHK(hipMemcpyAsync(out->j, dj, sizeof(uint32_t) * cnt, hipMemcpyDeviceToHost, ws.stream), "copy out");
      CHK(hipMemcpyAsync(out->sim, ds, sizeof(float) * cnt, hipMemcpyDeviceToHost, ws.stream), "copy out");
    }
    CHK(hipStreamSynchronize(ws.stream), "copy out");
  }
  if ((rc = record_total(ws))) return rc;
  out->count = cnt;
  return APSS_OK;
}

int stage_queries(apss_index* ix, Workspace& ws, int64_t nq, const int64_t* q_row_ptr, const int32_t* q_col,
                  const float* q_val, int on_device, const float* t_per_row, float t, RankRows& rows) {
  hipStream_t s = ws.stream;
  ws.graph.reset();  // the staging reuses buffers a captured join graph reads
  if (!ix->opts.query_safe) {
    set_error("index was built with query_safe = 0; external queries need the L2 cutoff clause");
    return APSS_EINVAL;
  }
  if (t_per_row) {
    for (int64_t q = 0; q < nq; ++q) {
      int rc = check_t(ix, t_per_row[q]);
      if (rc) return rc;
    }
  } else {
    int rc = check_t(ix, t);
    if (rc) return rc;
  }
  int rc;
  rows.n = nq;
  const int64_t* rp_host = q_row_ptr;
  int64_t nnz = 0;
  if (on_device) {
    if (!ws.host_in.reserve(sizeof(int64_t) * (size_t)(nq + 1))) {
      set_error("pinned host allocation failed");
      return APSS_ENOMEM;
    }
    CHK(hipMemcpyAsync(ws.host_in.p, q_row_ptr, sizeof(int64_t) * (nq + 1), hipMemcpyDeviceToHost, s), "read row_ptr");
    CHK(hipStreamSynchronize(s), "read row_ptr");
    rp_host = (const int64_t*)ws.host_in.p;
    nnz = rp_host[nq];
    if (nnz < 0 || nnz >= (1ll << 32)) {
      set_error("nnz must be in [0, 2^32)");
      return APSS_EINVAL;
    }
    for (int64_t r = 0; r <= nq; ++r)
      if ((r == 0 && rp_host[0] != 0) || (r < nq && rp_host[r + 1] < rp_host[r]))
        return check_bits(ERR_ROWPTR, (unsigned long long)r, "query");
  } else {
    nnz = q_row_ptr[nq];
    if (q_row_ptr[0] != 0 || nnz < 0 || nnz >= (1ll << 32)) {
      set_error("row_ptr must start at 0 and end at nnz in [0, 2^32)");
      return APSS_EINVAL;
    }
    for (int64_t r = 0; r < nq; ++r)
      if (q_row_ptr[r + 1] < q_row_ptr[r]) {
        set_error("row_ptr must be non-decreasing (row %lld)", (long long)r);
        return APSS_EINVAL;
      }
  }
  if (nnz > 0 && (!q_col || !q_val)) {
    set_error("NULL argument");
    return APSS_EINVAL;
  }
  rows.nnz = nnz;
  rows.rp_host.assign(rp_host, rp_host + nq + 1);
  int64_t longest = 0;
  for (int64_t r = 0; r < nq; ++r) longest = std::max(longest, rows.rp_host[(size_t)r + 1] - rows.rp_host[(size_t)r]);
  // One copy brings what is small: the cleared check words, the thresholds
  // and row_ptr, and the components of a batch of up to 128 KB (larger ones
  // straight from the caller's memory).
  constexpr size_t kPacked = 128 << 10;
  const size_t t_at = 2 * sizeof(unsigned long long);
  const size_t rp_at = t_at + ((t_per_row ? sizeof(float) * (size_t)nq : 0) + 7) / 8 * 8;
  const size_t col_at = rp_at + sizeof(int64_t) * (size_t)(nq + 1);
  const bool packed = !on_device && 2 * sizeof(float) * (size_t)nnz <= kPacked;
  const size_t val_at = col_at + (packed ? sizeof(int32_t) * (size_t)nnz : 0);
  const size_t total = val_at + (packed ? sizeof(float) * (size_t)nnz : 0);
  // every buffer is reserved before the first copy of the caller's memory is
  // queued, so no early return leaves such a copy in flight
  CHK(rows.rp.reserve(nq + 1), "alloc");
  CHK(rows.rc.reserve(nnz), "alloc");
  CHK(rows.mw.reserve(nq), "alloc");
  CHK(ws.q_in.reserve((int64_t)total), "alloc");
  if (t_per_row) CHK(ws.qt.reserve(nq), "alloc");
  if (!on_device && !packed) {
    CHK(ws.q_col.reserve(nnz), "alloc");
    CHK(ws.q_val.reserve(nnz), "alloc");
  }
  if ((rc = reserve_control(ws))) return rc;
  const bool lds = longest <= kQueryRow;
  SortScratch& ss = ws.ss;
  const int rbits = ceil_log2((uint64_t)ix->m);
  const int nbits = ceil_log2((uint64_t)std::max<int64_t>(nq, 1));
  if (!lds) {
    CHK(ss.k1.reserve(nnz), "alloc");
    CHK(ss.v32a.reserve(nnz), "alloc");
    if (!sorts_segments(nnz, longest, nbits + rbits)) {
      CHK(ss.k2.reserve(nnz), "sort scratch");
      CHK(ss.v32b.reserve(nnz), "sort scratch");
      CHK(ss.hist.reserve(radix_hist_elems(nnz)), "sort scratch");
      CHK(ss.scan.reserve(radix_scan_tmp_elems(nnz)), "sort scratch");
    }
    CHK(ss.seg.reserve(nq + 2), "sort scratch");
  }
  if (!ws.host_in.reserve(total)) {
    set_error("pinned host allocation failed");
    return APSS_ENOMEM;
  }
  unsigned char* const h = ws.host_in.p;
  const unsigned long long clear[2] = {0ull, ~0ull};
  memcpy(h, clear, sizeof(clear));
  if (t_per_row) memcpy(h + t_at, t_per_row, sizeof(float) * (size_t)nq);
  memcpy(h + rp_at, rows.rp_host.data(), sizeof(int64_t) * (size_t)(nq + 1));
  if (packed && nnz) {
    memcpy(h + col_at, q_col, sizeof(int32_t) * (size_t)nnz);
    memcpy(h + val_at, q_val, sizeof(float) * (size_t)nnz);
  }
  unsigned char* const in = ws.q_in.p;
  CHK(hipMemcpyAsync(in, h, total, hipMemcpyHostToDevice, s), "copy csr");
  if (!on_device && !packed) {
    CHK(hipMemcpyAsync(ws.q_col.p, q_col, sizeof(int32_t) * nnz, hipMemcpyHostToDevice, s), "copy csr");
    CHK(hipMemcpyAsync(ws.q_val.p, q_val, sizeof(float) * nnz, hipMemcpyHostToDevice, s), "copy csr");
  }
  const int64_t* const prp = (const int64_t*)(in + rp_at);
  const int32_t* const pcol = on_device ? q_col : packed ? (const int32_t*)(in + col_at) : ws.q_col.p;
  const float* const pval = on_device ? q_val : packed ? (const float*)(in + val_at) : ws.q_val.p;
  uint32_t* const err = (uint32_t*)in;
  unsigned long long* const bad = (unsigned long long*)in + 1;
  if (lds) {
    // the flags come over with the call's counters: rows that fail a check
    // meet nothing
    QueryRowsArgs a{};
    a.rp = prp;
    a.col = pcol;
    a.val = pval;
    a.t = t_per_row ? (const float*)(in + t_at) : nullptr;
    a.rank = ix->rank.p;
    a.nq = nq;
    a.m = ix->m;
    a.tol = 1e-5;
    a.rc = rows.rc.p;
    a.qmw = rows.mw.p;
    a.rp_out = rows.rp.p;
    a.t_out = t_per_row ? ws.qt.p : nullptr;
    a.zero = ws.counters.p;
    a.zeros = (int32_t)kControlWords;
    a.err = err;
    a.bad = bad;
    CHK(launch_query_rows(a, longest, s), "query rows");
    ws.pending = (const unsigned long long*)in;
    ws.cleared = nq > 0;
    return APSS_OK;
  }
  CHK(hipMemcpyAsync(rows.rp.p, prp, sizeof(int64_t) * (nq + 1), hipMemcpyDeviceToDevice, s), "copy");
  if (t_per_row) CHK(hipMemcpyAsync(ws.qt.p, in + t_at, sizeof(float) * nq, hipMemcpyDeviceToDevice, s), "copy");
  // invalid dimensions get a valid key, so the sort runs before the check
  CHK(launch_query_keys(prp, pcol, pval, ix->rank.p, nq, ix->m, rbits, 1e-5, ss.k1.p, ss.v32a.p, rows.mw.p, err, bad, s),
      "query keys");
  if ((rc = sort_rows(ws, ss.k1.p, ss.v32a.p, nnz, nbits + rbits, rbits, rows.rc.p, err, rows.rp_host.data(), nq)))
    return rc;
  return check_err(s, (const unsigned long long*)in, "query");
}

}  // namespace apss

namespace {

QuerySet corpus_queries(const apss_index* ix) {
  return QuerySet{ix->rows.rp.p, ix->rows.rc.p, ix->rows.mw.p, ix->n, ix->nnz, ix->rows.rp_host.data()};
}

QuerySet staged_queries(const RankRows& r) {
  return QuerySet{r.rp.p, r.rc.p, r.mw.p, r.n, r.nnz, r.rp_host.data()};
}

int self_join(apss_index* ix, float t, int64_t* cnt, Sink* sink) {
  if (ix->screen) return run_screen_join(ix, ix->ws, t, join_cap_hint(ix), cnt, sink);
  return run_join(ix, ix->ws, corpus_queries(ix), 1, t, nullptr, join_cap_hint(ix), cnt, nullptr, sink);
}

}  // namespace

extern "C" {

void apss_default_opts(apss_opts* o) {
  if (!o) return;
  memset(o, 0, sizeof(*o));
  o->struct_size = (int32_t)sizeof(apss_opts);
  o->stream = nullptr;
  o->query_safe = 1;
  o->variant = -1;
  o->head_dims = 0;
  o->range_rows = 0;
  o->screen_dims = 0;
  o->graph = 0;
}

int apss_build_index(int64_t n, int64_t m, const int64_t* row_ptr, const int32_t* col, const float* val, int on_device,
                     float t_build, const apss_opts* opts, apss_index** out) {
  if (!out || !row_ptr || (!col && n > 0) || (!val && n > 0)) {
    set_error("NULL argument");
    return APSS_EINVAL;
  }
  *out = nullptr;
  if (n < 0 || n >= (1ll << 31) || m <= 0 || m >= (1ll << 31)) {
    set_error("need 0 <= n < 2^31 and 0 < m < 2^31");
    return APSS_EINVAL;
  }
  if (!(t_build > 0.0f && t_build <= 1.0f)) {
    set_error("t_build %g outside (0, 1]", (double)t_build);
    return APSS_ETHRESH;
  }
  apss_opts o;
  apss_default_opts(&o);
  if (opts) {
    if (opts->struct_size != (int32_t)sizeof(apss_opts)) {
      set_error("apss_opts.struct_size mismatch (use apss_default_opts)");
      return APSS_EINVAL;
    }
    o = *opts;
  }
  if (o.variant < -1 || o.variant >= join_num_variants() || (o.variant >= 0 && !variant_available(o.variant))) {
    set_error("variant %d is not available (outside [-1, %d) or withdrawn)", o.variant, join_num_variants());
    return APSS_EINVAL;
  }
  if (o.range_rows < 0) {
    set_error("range_rows must be >= 0");
    return APSS_EINVAL;
  }
  if (o.range_group < 0 || o.range_group > kMaxRangeGroup) {
    set_error("range_group must be in [0, %d]", kMaxRangeGroup);
    return APSS_EINVAL;
  }
  if (o.screen_dims < 0 || o.screen_dims > kScreenMaxHead) {
    set_error("screen_dims must be in [0, %d]", kScreenMaxHead);
    return APSS_EINVAL;
  }
  if (o.index_all < 0 || o.index_all > 1 || o.remscore < 0 || o.remscore > 1) {
    set_error("index_all and remscore must be 0 or 1");
    return APSS_EINVAL;
  }
  if (!(o.local_parts == 0 || o.local_parts == 1 || o.local_parts == 2 || o.local_parts == 4 || o.local_parts == 8)) {
    set_error("local_parts must be 0, 1, 2, 4 or 8");
    return APSS_EINVAL;
  }
  if (o.screen_dims > 0 && (o.index_all || o.local_parts > 1 || o.remscore)) {
    set_error("screen_dims does not combine with index_all, local_parts or remscore");
    return APSS_EINVAL;
  }
  apss_index* ix = new (std::nothrow) apss_index();
  if (!ix) {
    set_error("host allocation failed");
    return APSS_ENOMEM;
  }
  ix->opts = o;
  ix->ws.stream = (hipStream_t)o.stream;
  ix->n = n;
  ix->m = m;
  ix->t_build = t_build;
  ix->variant = o.variant >= 0 ? o.variant : 1;
  if (const char* ev = getenv("APSS_VARIANT")) {
    const int v = atoi(ev);
    if (v >= 0 && v < join_num_variants() && variant_available(v)) ix->variant = v;
  }
  ix->range_rows = o.range_rows > 0 ? o.range_rows : default_range_rows(ix->variant);
  if (const char* ev = getenv("APSS_RANGE_ROWS")) {
    const long long rr = atoll(ev);
    if (rr > 0) ix->range_rows = rr;
  }
  ix->range_group = o.range_group > 0 ? o.range_group : 1;
  if (const char* ev = getenv("APSS_RANGE_GROUP")) {
    const int g = atoi(ev);
    if (g >= 1 && g <= kMaxRangeGroup) ix->range_group = g;
  }
  ix->default_geometry = default_geometry(o);
  (void)hipGetDevice(&ix->device);
  if (o.screen_dims > 0 && !screen_variant_ok(ix->variant)) {
    set_error("tile variant %d is not available for the screened join", ix->variant);
    delete ix;
    return APSS_EINVAL;
  }
  int rc = build_impl(ix, row_ptr, col, val, on_device);
  // the join's lookup tables for the index's geometry, the call timers and
  // the pinned counters exist from here on, so apss_join_device_noalloc needs
  // no allocation
  if (!rc && o.screen_dims == 0 && n > 0) rc = prepare(ix, ix->ws.stream, ix->variant, ix->range_rows);
  if (!rc) rc = reserve_host(ix->ws);
  for (int e = 0; !rc && e < 6; ++e)
    if (hipEventCreateWithFlags(&ix->ws.ev[e], hipEventDefault) != hipSuccess) {
      set_error("hipEventCreateWithFlags failed");
      rc = APSS_EDEVICE;
    }
  if (rc) {
    (void)hipStreamSynchronize(ix->ws.stream);
    apss_index_free(ix);
    return rc;
  }
  *out = ix;
  return APSS_OK;
}

void apss_index_free(apss_index* idx) {
  if (!idx) return;
  (void)hipStreamSynchronize(idx->ws.stream);
  apss_index_free(idx->screen);
  delete idx;
}

int64_t apss_release_memory(void) { return (int64_t)spare_release(); }

int apss_join_device(apss_index* ix, float t, uint32_t* out_i, uint32_t* out_j, float* out_sim, int64_t capacity,
                     int64_t* count) {
  if (!ix || !count || (capacity > 0 && (!out_i || !out_j || !out_sim))) {
    set_error("NULL argument");
    return APSS_EINVAL;
  }
  int rc = check_t(ix, t);
  if (rc) return rc;
  if (ix->opts.graph && !ix->screen && ix->parts == 1 && !ix->opts.remscore && ix->n > 0)
    return graph_join(ix, t, out_i, out_j, out_sim, capacity, count);
  int64_t cnt = 0;
  Sink sink{out_i, out_j, out_sim, capacity};
  if ((rc = self_join(ix, t, &cnt, &sink))) return rc;
  return finish_device(ix->ws, cnt, ceil_log2((uint64_t)ix->n), sink, count);
}

int apss_join(apss_index* ix, float t, apss_pairs* out) {
  if (!ix || !out) {
    set_error("NULL argument");
    return APSS_EINVAL;
  }
  out->count = 0;
  out->i = out->j = nullptr;
  out->sim = nullptr;
  int rc = check_t(ix, t);
  if (rc) return rc;
  int64_t cnt = 0;
  Sink sink;
  if ((rc = host_sink(ix->ws, &sink))) return rc;
  if ((rc = self_join(ix, t, &cnt, &sink))) return rc;
  return finish_host(ix->ws, cnt, ceil_log2((uint64_t)ix->n), sink, out);
}

int apss_query_device(apss_index* ix, int64_t nq, const int64_t* q_row_ptr, const int32_t* q_col, const float* q_val,
                      int on_device, const float* t_per_row, float t, uint32_t* out_i, uint32_t* out_j,
                      float* out_sim, int64_t capacity, int64_t* count) {
  if (!ix || !count || !q_row_ptr || nq < 0 || nq >= (1ll << 31) ||
      (capacity > 0 && (!out_i || !out_j || !out_sim))) {
    set_error("NULL or invalid argument");
    return APSS_EINVAL;
  }
  RankRows& rows = ix->ws.q_rows;
  int rc = stage_queries(ix, ix->ws, nq, q_row_ptr, q_col, q_val, on_device, t_per_row, t, rows);
  if (rc) return rc;
  int64_t cnt = 0;
  Sink sink{out_i, out_j, out_sim, capacity};
  if ((rc = run_join(ix, ix->ws, staged_queries(rows), 0, t, t_per_row ? ix->ws.qt.p : nullptr, 16 * nq, &cnt, t_per_row,
                     &sink))) {
    (void)hipStreamSynchronize(ix->ws.stream);  // (the caller's rows may still be read)
    return rc;
  }
  return finish_device(ix->ws, cnt, ceil_log2((uint64_t)ix->n), sink, count);
}

int apss_query(apss_index* ix, int64_t nq, const int64_t* q_row_ptr, const int32_t* q_col, const float* q_val,
               int on_device, const float* t_per_row, float t, apss_pairs* out) {
  if (!ix || !out || !q_row_ptr || nq < 0 || nq >= (1ll << 31)) {
    set_error("NULL or invalid argument");
    return APSS_EINVAL;
  }
  out->count = 0;
  out->i = out->j = nullptr;
  out->sim = nullptr;
  Sink sink;
  int rc = host_sink(ix->ws, &sink);
  if (rc) return rc;
  RankRows& rows = ix->ws.q_rows;
  if ((rc = stage_queries(ix, ix->ws, nq, q_row_ptr, q_col, q_val, on_device, t_per_row, t, rows))) return rc;
  int64_t cnt = 0;
  if ((rc = run_join(ix, ix->ws, staged_queries(rows), 0, t, t_per_row ? ix->ws.qt.p : nullptr, 16 * nq, &cnt, t_per_row,
                     &sink))) {
    (void)hipStreamSynchronize(ix->ws.stream);  // (the caller's rows may still be read)
    return rc;
  }
  return finish_host(ix->ws, cnt, ceil_log2((uint64_t)ix->n), sink, out);
}

void apss_pairs_free(apss_pairs* p) {
  if (!p) return;
  free(p->i);
  free(p->j);
  free(p->sim);
  p->i = p->j = nullptr;
  p->sim = nullptr;
  p->count = 0;
}

int apss_last_stats(const apss_index* ix, apss_stats* out) {
  if (!ix || !out) {
    set_error("NULL argument");
    return APSS_EINVAL;
  }
  *out = ix->ws.last;
  return APSS_OK;
}

int apss_index_export(const apss_index* ix, int32_t* rank, float* maxweight, int32_t* cut) {
  if (!ix) {
    set_error("NULL argument");
    return APSS_EINVAL;
  }
  hipStream_t s = ix->ws.stream;
  if (rank) CHK(hipMemcpyAsync(rank, ix->rank.p, sizeof(int32_t) * ix->m, hipMemcpyDeviceToHost, s), "export");
  if (maxweight || (cut && ix->n)) {
    float* const mw = (float*)ix->out.p;
    int32_t* const cuts = (int32_t*)ix->out.p + ix->m;
    CHK(launch_export(ix->rank.p, ix->mw_r.p, ix->m, ix->rs.p, ix->n, maxweight ? mw : nullptr, cut ? cuts : nullptr, s),
        "export");
    if (maxweight) CHK(hipMemcpyAsync(maxweight, mw, sizeof(float) * ix->m, hipMemcpyDeviceToHost, s), "export");
    if (cut && ix->n) CHK(hipMemcpyAsync(cut, cuts, sizeof(int32_t) * ix->n, hipMemcpyDeviceToHost, s), "export");
  }
  CHK(hipStreamSynchronize(s), "export");
  return APSS_OK;
}

int apss_index_sizes(const apss_index* ix, int64_t* n, int64_t* m, int64_t* nnz, int64_t* postings) {
  if (!ix) {
    set_error("NULL argument");
    return APSS_EINVAL;
  }
  if (n) *n = ix->n;
  if (m) *m = ix->m;
  if (nnz) *nnz = ix->nnz;
  if (postings) *postings = ix->P;
  return APSS_OK;
}

const char* apss_strerror(int code) {
  switch (code) {
    case APSS_OK: return "ok";
    case APSS_EINVAL: return "invalid argument";
    case APSS_ETHRESH: return "threshold out of range";
    case APSS_ENOMEM: return "out of memory";
    case APSS_EDEVICE: return "device error";
    case APSS_ERANGE: return "output buffer too small";
    case APSS_EBUSY: return "busy";
    case APSS_PENDING: return "pending";
    default: return "unknown error";
  }
}

const char* apss_last_error(void) { return last_error().c_str(); }

}  // extern "C"
