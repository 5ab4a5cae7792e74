// Host-side state shared by the single-problem and batched entry points.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/arrow.h"
#include "bodies.hpp"

constexpr int LANE_TABLE_MAX = 16;

struct arrow_handle_s {
  int device;
  hipStream_t stream;
  double* ws;
  size_t ws_cap;      // doubles
  ahd::Options opt;
  int lanes;          // single problems: 0 = automatic, else lanes per eigenvalue
  int timing;         // record stage events
  // stage events of the two most recent timed calls, used in turn, so that a
  // caller may read one call's stages after queuing the next
  hipEvent_t ev[2][6];
  int ev_made;
  int ev_set;         // set of the most recent timed call
  int timed_calls;    // timed calls launched so far, up to 2
  int64_t last_n;
  double* last_ws;    // workspace of the most recent single-problem call (the handle's, or the scratch)
  size_t lds_max;     // bytes of dynamic LDS one block may use
  int cus;            // compute units of the device
  // lanes per eigenvalue by order n: [ARROW_SCHEDULE_SINGLE] for single
  // problems (empty: the built-in rule), [ARROW_SCHEDULE_BATCH] inside batches
  int ntab[2];
  int32_t tab_n[2][LANE_TABLE_MAX];
  int32_t tab_g[2][LANE_TABLE_MAX];
  int tab_default;    // the single-problem table came by arrow_set_default_lanes
  void* blas;         // rocBLAS handle of tridiag_eig's GEMMs, made on first use
  void* td_ws;        // tridiag_eig's device buffers (grown on demand, kept)
  size_t td_cap;      // bytes
  void* td_plan;      // its merge plans' device block (grown on demand, kept)
  size_t td_plan_cap; // bytes
  void* td_host;      // its pinned staging (grown on demand, kept)
  size_t td_host_cap; // bytes
  uint32_t magic;
};

static constexpr uint32_t HANDLE_MAGIC = 0xA770E16u;

static inline bool valid(arrow_handle_t h) { return h && h->magic == HANDLE_MAGIC; }

struct DeviceGuard {
  int prev = -1;
  explicit DeviceGuard(int dev) {
    if (hipGetDevice(&prev) != hipSuccess) prev = -1;
    if (prev != dev) (void)hipSetDevice(dev);
  }
  ~DeviceGuard() {
    if (prev >= 0) (void)hipSetDevice(prev);
  }
};

// Zeros in the header of a new workspace, where the sort's completion count starts at 0
// (each call leaves it there).  On a stream of its own while the caller's is captured: a
// first call may be (relaxed capture mode allows the allocation), and neither a wait nor
// a memset belongs in its graph.
static inline bool clear_header(double* ws, hipStream_t stream) {
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  hipStream_t own = nullptr;
  if (hipStreamIsCapturing(stream, &status) == hipSuccess && status != hipStreamCaptureStatusNone) {
    if (hipStreamCreateWithFlags(&own, hipStreamNonBlocking) != hipSuccess) return false;
    stream = own;
  }
  const bool ok = hipMemsetAsync(ws, 0, 16 * sizeof(double), stream) == hipSuccess &&
                  hipStreamSynchronize(stream) == hipSuccess;
  if (own) (void)hipStreamDestroy(own);
  return ok;
}

static inline int ensure_ws(arrow_handle_t h, size_t doubles) {
  if (doubles <= h->ws_cap) return ARROW_OK;
  if (h->ws) {
    (void)hipStreamSynchronize(h->stream);
    (void)hipFree(h->ws);
    h->ws = nullptr;
    h->ws_cap = 0;
  }
  if (hipMalloc((void**)&h->ws, doubles * sizeof(double)) != hipSuccess) {
    h->ws = nullptr;
    return ARROW_ERR_NOMEM;
  }
  if (!clear_header(h->ws, h->stream)) {
    (void)hipFree(h->ws);
    h->ws = nullptr;
    return ARROW_ERR_HIP;
  }
  h->ws_cap = doubles;
  return ARROW_OK;
}

static inline int table_lookup(const arrow_handle_s* h, int scope, int64_t n, int fallback) {
  for (int e = 0; e < h->ntab[scope]; ++e)
    if (n <= h->tab_n[scope][e]) return h->tab_g[scope][e];
  return fallback;
}

// lanes per eigenvalue for a single problem: a fixed option, else the tuned
// table, else about 8 pole terms per lane
static inline int single_lanes(const arrow_handle_s* h, int64_t n) {
  if (h->lanes) return h->lanes;
  int g = 1;
  while (g < 64 && g < n / 8) g <<= 1;
  return table_lookup(h, ARROW_SCHEDULE_SINGLE, n, g);
}

// whether the large problems' kernel, 64 lanes per eigenvalue, may take a call of order
// n: a caller's own lane count comes first (64 is its own), a default table does not
static inline bool large_kernel_lanes(const arrow_handle_s* h, int64_t n) {
  return h->lanes == 0 && (h->tab_default || single_lanes(h, n) == 64);
}

// Blocks of the launch that finishes a small problem that re-solve its listed
// eigenvalues: three a compute unit, which run two at a time.  An eigenvalue each up to
// three times the compute units; two listed ones in one block run in turn, and with one
// block a compute unit one such pair in the whole problem held up the launch (graded,
// values alone, n = 1000: 57.5 us, now 52.3; as launches of their own 53.4).  A block
// each up to n = 1280 costs the others their dispatch (uniform, n = 1280: 51.0 -> 53.6 us,
// three a unit 52.4).  And no fewer blocks than let one of `block` threads ask each of its
// eigenvalues with a thread of its own.
static inline int finish_redo_blocks(int64_t n, int cus, int block) {
  const int64_t want = 3 * (int64_t)cus, least = (n + block - 1) / block;
  const int64_t b = want > least ? want : least;
  return (int)(n < b ? n : b);
}

// Root items of a batched plan that a wavefront takes from the queue at a time, of
// `items` beside the shared ones, for `waves` resident wavefronts: two, unless that
// leaves wavefronts without any, below one and a half a wavefront.  By ones, 10,000
// problems of n = 16..64 (6.4 items a wavefront) take 433 us, by twos 320; 5000 (3.2)
// 253 and 198; 1200 of n = 64..128 (1.8) 180 and 152; but 300 of n = 128..512 (1.3) 174
// and 207, 150 of n = 256..600 (0.9) 163 and 211.
static inline int root_chunk(int64_t items, int64_t waves) { return 2 * items < 3 * waves ? 1 : 2; }

// all launches of one single-problem solve (defined with the single-problem kernels)
int launch_single(arrow_handle_t h, const ahd::ProbDesc& D);

// frees what tridiag_eig keeps in the handle
void tridiag_release(arrow_handle_t h);

// lanes per eigenvalue for a problem of order n inside a batch
static inline int batch_lanes(const arrow_handle_s* h, int64_t n) {
  return table_lookup(h, ARROW_SCHEDULE_BATCH, n, 64);
}

// the built-in batched table
static inline void default_batch_table(arrow_handle_s* h) {
  static const int32_t tn[5] = {24, 48, 96, 192, 2147483647};
  static const int32_t tg[5] = {4, 8, 16, 32, 64};
  h->ntab[ARROW_SCHEDULE_BATCH] = 5;
  for (int e = 0; e < 5; ++e) {
    h->tab_n[ARROW_SCHEDULE_BATCH][e] = tn[e];
    h->tab_g[ARROW_SCHEDULE_BATCH][e] = tg[e];
  }
}
