// libarrow: gfx950 kernels and the C ABI declared in include/arrow.h.
//
// One call runs these launches on the handle's stream:
//   k_prep      rank of every pole (symmetric permutation to decreasing order,
//               Sec. 1), the permuted copy and the prologue: shaft weights and
//               corner of the (reduced) arrowhead in double-double, and the
//               deflation of a reducible arrowhead (Sec. 1).  Above PREP_MAX poles
//               k_front (order check; for ordered input all of that) and k_sort
//               (the rank count of unordered input) take its place
//   k_root      per eigenvalue: shift selection, b, root of the inverse (Algorithms 1-3, Theorem 6)
//   k_finish    per eigenvalue: K_nu test (Algorithm 5), repairs (Remarks 1-2, DPR1
//               re-measure), norm, then its eigenvector, streamed to HBM
//               (eq. eigenvecAi, Algorithm 4; complex for a Hermitian arrowhead, Sec. 6.1).
//               Above FIN_MAX (by bisection three times the compute units) k_check,
//               k_repair and k_vec take its place, with the eigenpairs a reducible
//               arrowhead deflated (Sec. 1) in k_vec's launch, without vectors in
//               k_repair's
// k_root gives G lanes of a wavefront to each eigenvalue (G = 64: one
// wavefront per eigenvalue); the vectors are bound by the n^2 FP64 stores.

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <math.h>
#include <mutex>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
#include <type_traits>

#include "../../include/arrow.h"
#include "blocks.hpp"
#include "host.hpp"

using namespace ahd;

// orders the single-problem calls accept: the root and check launches index
// n * G <= 2^31 lanes (G <= 64) in 64-bit arithmetic
static bool order_ok(int64_t n) { return n >= 1 && n <= ARROW_N_MAX; }

static_assert(ARROW_INFO_DD_B == INFO_DD_B && ARROW_INFO_REMEDY_A == INFO_REMEDY_A &&
                  ARROW_INFO_REMEDY_B == INFO_REMEDY_B && ARROW_INFO_NEAR_ZERO == INFO_NEAR_ZERO &&
                  ARROW_INFO_REDUCIBLE == INFO_REDUCIBLE && ARROW_INFO_NONFINITE == INFO_NONFINITE &&
                  ARROW_INFO_KB_LARGE == INFO_KB_LARGE && ARROW_INFO_BAD_INPUT == INFO_BAD_INPUT &&
                  ARROW_INFO_POLE_SHIFT == INFO_POLE_SHIFT && ARROW_INFO_DEFLATED == INFO_DEFLATED &&
                  ARROW_INFO_F0_UNRESOLVED == INFO_F0_UNRESOLVED,
              "info bits");


// ---------------------------------------------------------------------------
// kernels

// Sorting (symmetric permutation to decreasing poles, Sec. 1) and the prologue,
// up to PREP_MAX poles, in one launch.  Every block asks whether the input already
// is in that order, or in the reverse one (the usual cases); only if not, a pole's
// rank is counted: a wavefront holds 64 keys, one a lane, and reads the keys it
// compares them with through the scalar cache (the same for all lanes), the next
// 16 under way while it compares, two instructions a comparison; the block's
// wavefronts share the keys out.  The thread that has the rank writes the sorted
// entry and its weight, and the last block to finish (the only one up to PREP_ONE
// poles) reduces the statuses and the corner.  Bound by latency (a chain of
// dependent loads and one pass through the device-scope release and acquire).
// An order check in one block and a rank count whose last block scattered
// everything took 33 us at n = 199 shuffled, 44 us at 1025, 56 us at 2047 (ordered:
// 6.5 us at 512, 13.6 us at 4096); this 11, 12 and 24 us (7.6 and 9.3 us).
constexpr int PREP_BLOCK = 1024;
constexpr int PREP_WAVES = PREP_BLOCK / 64;
constexpr int PREP_ONE = 256;     // poles one block ranks alone: 64 comparisons a lane
constexpr int PREP_MAX = 16384;   // the blocks' order checks read n^2 / 64 keys from the L2
constexpr uint32_t ST_NAN = 1u << 30;   // input status: a pole that is not a number (it has no rank)

// blocks of the sort that are done: 0 between calls
__host__ __device__ inline uint32_t* sort_done(const Ws& w) { return (uint32_t*)(w.hdr + 7); }
// 1 when the caller's poles already are in the sorted order
__host__ __device__ inline uint32_t* in_order(const Ws& w) { return (uint32_t*)(w.hdr + 11); }

template <int KIND, bool ONE>
__global__ __launch_bounds__(PREP_BLOCK) void k_prep(ProbDesc D, const double* __restrict__ poles, int groups) {
  __shared__ int part[PREP_WAVES][64];
  __shared__ double least[PREP_WAVES];
  __shared__ int last;
  const Ws w = ws_view(D.ws, D.n);
  const int ms = sorted_count(D), m = D.n - 1;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // `groups` groups of 64 keys a block, PREP_WAVES / groups wavefronts each
  const int grp = wave % groups, share = wave / groups, shares = PREP_WAVES / groups;
  const int j0 = (blockIdx.x * groups + grp) * 64, j = j0 + lane;
  auto key = [&](double d) { return sort_key<KIND>((KIND == KIND_DPR1 && D.neg) ? -d : d); };
  // this lane's entry
  constexpr int S = (KIND == KIND_HERM) ? 2 : 1;
  const bool has = share == 0 && j < ms;
  const double dj = (j < ms) ? poles[j] : NAN, kj = key(dj);
  const double re = has ? D.z[S * j] : 0.0, im = (KIND == KIND_HERM && has) ? D.z[S * j + 1] : 0.0;
  double dn = INFINITY;   // DPR1: the last sorted pole
  int down = 0, up = 0;   // some pair not strictly decreasing / not strictly increasing
  for (int q = threadIdx.x; q < ms; q += PREP_BLOCK) {
    const double a = key(poles[q]), b = (q + 1 < ms) ? key(poles[q + 1]) : 0.0;
    if (q + 1 < ms) {
      if (!(a > b)) down = 1;
      if (!(a < b)) up = 1;
    }
    if (KIND == KIND_DPR1) dn = fmin(dn, a);
  }
  if constexpr (KIND == KIND_DPR1) {
    dn = gmin<64>(dn);
    if (lane == 0) least[wave] = dn;
  }
  down = __syncthreads_or(down);
  up = __syncthreads_or(up);
  if constexpr (KIND == KIND_DPR1) {
    dn = least[0];
    for (int q = 1; q < PREP_WAVES; ++q) dn = fmin(dn, least[q]);
  }
  int r = down ? ms - 1 - j : j;
  if (down && up) {
    const int chunk = (ms + shares - 1) / shares;
    const int l0 = min(ms, share * chunk), l1 = min(ms, l0 + chunk);
    int cnt = 0;   // keys in front of j's: greater ones, and equal ones of smaller index
    auto scan = [&](int a, int b, auto&& before) {
      constexpr int N = 16;
      int l = a;
      if (l + N <= b) {
        double now[N];
#pragma unroll
        for (int u = 0; u < N; ++u) now[u] = poles[l + u];
        for (; l + 2 * N <= b; l += N) {
          double next[N];
#pragma unroll
          for (int u = 0; u < N; ++u) next[u] = poles[l + N + u];
#pragma unroll
          for (int u = 0; u < N; ++u) cnt += before(key(now[u]), l + u) ? 1 : 0;
#pragma unroll
          for (int u = 0; u < N; ++u) now[u] = next[u];
        }
#pragma unroll
        for (int u = 0; u < N; ++u) cnt += before(key(now[u]), l + u) ? 1 : 0;
        l += N;
      }
      for (; l < b; ++l) cnt += before(key(poles[l]), l) ? 1 : 0;
    };
    scan(l0, min(l1, j0), [&](double kl, int) { return kl >= kj; });
    scan(max(l0, j0), min(l1, j0 + 64), [&](double kl, int l) { return kl > kj || (kl == kj && l < j); });
    scan(max(l0, j0 + 64), l1, [&](double kl, int) { return kl > kj; });
    part[wave][lane] = cnt;
    __syncthreads();
    r = 0;
    for (int q = 0; q < shares; ++q) r += part[q * groups + grp][lane];
  }
  if (kj != kj) r = ms - 1;   // behind every number: those fill the first entries
  if (has) {   // r < ms: the other keys in front of j's
    const SortedEntry e = put_sorted_vals<KIND>(w, r, j, (KIND == KIND_DPR1 && D.neg) ? -dj : dj, re, im);
    w.st[j] = input_status_vals<KIND>(dj, re, im, false) | (kj == kj ? 0u : ST_NAN);
    if (r < m) prologue_vals<KIND>(D, w, r, e.d, e.z, e.c, dn);
  }
  if constexpr (!ONE) {
    // behind the barrier one thread releases the block's entries at device scope
    // (a write-back of the L2 a wavefront, so one is enough) and counts the block
    // in; the last block acquires.  The count wraps to 0, and a later launch of every
    // call (k_finish, k_check, k_check_edges) stores 0 as well: calls that overlapped
    // in one workspace may leave another value, and the first one ordered behind them
    // must find 0
    __syncthreads();
    if (threadIdx.x == 0) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      last = atomicInc(sort_done(w), gridDim.x - 1) == gridDim.x - 1;
      if (last) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
    if (!last) return;
  } else {
    __syncthreads();
  }
  // the corner's partial sums run over the sorted entries r = t, t + PREP_BLOCK,
  // ...: the same bits whatever the order of the input; equal poles are neighbours
  uint32_t st = 0, zp = 0;
  int dup = 0;
  dd acc = {0.0, 0.0};
  for (int r = threadIdx.x; r < ms; r += PREP_BLOCK) {
    const double d = w.ds[r];
    st |= w.st[r];
    if (r + 1 < ms && sort_key<KIND>(d) == sort_key<KIND>(w.ds[r + 1])) dup = 1;
    if (r < m && d == 0.0) zp = 1;
    acc = dd_add(acc, corner_term<KIND>(D, w, r));
  }
  if (__syncthreads_or(st & ST_NAN)) {
    // the poles that are numbers, ranked among themselves, fill the first entries; most
    // of the others hold what was there (nothing is solved, so nothing else reads them)
    int written = 0;
    for (int r0 = 0; r0 < ms; r0 += PREP_BLOCK) {
      const int r = r0 + threadIdx.x;
      written += __syncthreads_count(r < ms && !(w.st[r] & ST_NAN));
    }
    dup = 0;
    for (int r = threadIdx.x; r + 1 < written; r += PREP_BLOCK)
      dup |= sort_key<KIND>(w.ds[r]) == sort_key<KIND>(w.ds[r + 1]);
  }
  if (threadIdx.x == 0) *in_order(w) = down ? 0u : 1u;
  prologue_reduce<KIND, PREP_BLOCK>(D, w, acc, (st & ~ST_NAN) | (dup ? INFO_REDUCIBLE : 0u), zp);
}

// Above PREP_MAX poles: a one-block check whether the input already is in that
// order, or in the reverse one (the usual cases), then, only if not, a rank
// count over a 2-D grid of (pole tile, comparison chunk) blocks, then the
// scatter.  rank[] holds the count in its low 30 bits and a duplicate marker in bit 30.
constexpr int SORT_CHUNK = 256;   // keys of one comparison chunk
constexpr int SORT_BLOCK = 1024;  // the last block also scatters and runs the prologue: a wide one

__host__ __device__ inline uint32_t* rank_array(const Ws& w, int64_t n) { return w.st + n; }

// One block of FRONT_BLOCK threads: whether the input already is in that
// order (the usual case); if it is, the copy to the workspace and the whole
// prologue are done here and k_sort returns at once, else the rank array and
// k_sort's completion counter are cleared for it.
constexpr int FRONT_BLOCK = 1024;

template <int KIND>
__global__ __launch_bounds__(FRONT_BLOCK) void k_front(ProbDesc D) {
  const Ws w = ws_view(D.ws, D.n);
  const int ms = sorted_count(D);
  int down = 0, up = 0;   // some pair not strictly decreasing / not strictly increasing
  for (int j = threadIdx.x; j + 1 < ms; j += FRONT_BLOCK) {
    const double a = sort_key<KIND>(in_pole<KIND>(D, j)), b = sort_key<KIND>(in_pole<KIND>(D, j + 1));
    if (!(a > b)) down = 1;
    if (!(a < b)) up = 1;
  }
  down = __syncthreads_or(down);
  up = __syncthreads_or(up);
  const bool rev = down && !up;   // strictly increasing: sorted index ms-1-j
  const int bad = down && up;
  if (threadIdx.x == 0) *in_order(w) = down ? 0u : 1u;
  if (bad) {
    uint32_t* rank = rank_array(w, D.n);
    for (int j = threadIdx.x; j < ms; j += FRONT_BLOCK) rank[j] = 0;
    if (threadIdx.x == 0) {
      w.hdr[5] = 1.0;
      *sort_done(w) = 0u;
    }
    return;
  }
  // the copy and the prologue of each sorted entry r by the thread that reads
  // its source q, from registers; the corner partial sums run over r = t,
  // t + FRONT_BLOCK, ... as in prologue_block, so the corner is the same bits
  // either way the input arrives
  const int m = D.n - 1;
  const double dn = (KIND == KIND_DPR1) ? in_pole<KIND>(D, rev ? 0 : ms - 1) : 0.0;   // the last sorted pole
  uint32_t st = 0, zp = 0;
  dd acc = {0.0, 0.0};
  for (int r = threadIdx.x; r < ms; r += FRONT_BLOCK) {
    const int q = rev ? ms - 1 - r : r;
    const SortedEntry e = put_sorted_v<KIND>(D, w, r, q);
    st |= input_status<KIND>(D, q, false);
    acc = dd_add(acc, corner_term_v<KIND>(D, e.z));
    if (r < m) {
      prologue_vals<KIND>(D, w, r, e.d, e.z, e.c, dn);
      zp |= (e.d == 0.0) ? 1u : 0u;
    }
  }
  prologue_reduce<KIND, FRONT_BLOCK>(D, w, acc, st, zp);
  if (threadIdx.x == 0) w.hdr[5] = 0.0;
}

// Unsorted input: the rank of every key over a 2-D grid of (key tile,
// comparison chunk) blocks, accumulated with atomics; the last block to finish
// (a completion count) then holds every rank, scatters the poles into
// decreasing order and runs the prologue.
template <int KIND>
__global__ __launch_bounds__(SORT_BLOCK) void k_sort(ProbDesc D, int chunk, int nchunks) {
  __shared__ double tile[SORT_BLOCK];
  __shared__ int last;
  const Ws w = ws_view(D.ws, D.n);
  if (w.hdr[5] == 0.0) return;  // already sorted: k_front did everything
  const int ms = sorted_count(D);
  uint32_t* rank = rank_array(w, D.n);
  const int j = blockIdx.x * SORT_BLOCK + threadIdx.x;
  const double kj = (j < ms) ? sort_key<KIND>(in_pole<KIND>(D, j)) : NAN;
  uint32_t cnt = 0;
  bool dup = false;
  for (int cy = blockIdx.y; cy < nchunks; cy += gridDim.y) {   // this block's comparison chunks
    const int l0 = cy * chunk;
    const int l1 = min(ms, l0 + chunk);
    for (int base = l0; base < l1; base += SORT_BLOCK) {
      const int l = base + threadIdx.x;
      tile[threadIdx.x] = (l < l1) ? sort_key<KIND>(in_pole<KIND>(D, l)) : NAN;
      __syncthreads();
      const int lim = min(SORT_BLOCK, l1 - base);
      for (int t = 0; t < lim; ++t) {
        const double kl = tile[t];
        const int idx = base + t;
        cnt += (kl > kj) || (kl == kj && idx < j);
        dup |= (kl == kj) && (idx != j);
      }
      __syncthreads();
    }
  }
  if (j < ms) {
    if (cnt) atomicAdd(&rank[j], cnt);
    if (dup) atomicOr(&rank[j], 1u << 30);
  }
  // Every thread releases its counts at device scope (a write-back, no
  // invalidation of the L2), then one thread counts the block in; only the
  // last block acquires before it reads the ranks.
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
  __syncthreads();
  if (threadIdx.x == 0) last = atomicAdd(sort_done(w), 1u) == gridDim.x * gridDim.y - 1;
  __syncthreads();
  if (!last) return;
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  for (int q = threadIdx.x; q < ms; q += SORT_BLOCK) {
    const uint32_t raw = __hip_atomic_load(&rank[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int r = (int)(raw & 0x3fffffffu);
    if (r < ms) put_sorted<KIND>(D, w, r, q);   // a rank is < ms by construction
    w.st[q] = input_status<KIND>(D, q, (raw >> 30) & 1u);
  }
  __syncthreads();
  prologue_block<KIND, SORT_BLOCK>(D);
}

// Root stage: ROOT_BLOCK threads per block, G lanes per
// eigenvalue.  When the sorted poles and shaft weights fit, the block first
// copies them to LDS and every O(n) pass reads them from there.
constexpr int ROOT_BLOCK = 512;

__device__ inline void stage_hot(const ProbDesc& D, double* lds) {
  const Ws w = ws_view(D.ws, D.n);
  const int ns = sorted_count(D), m = D.n - 1;
  const int top = ns > m ? ns : m;
  // four rows of both arrays in flight per thread before the LDS stores
  for (int j0 = threadIdx.x; j0 < top; j0 += 4 * blockDim.x) {
    double a[4], c[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int j = j0 + q * blockDim.x;
      a[q] = (j < ns) ? w.ds[j] : 0.0;
      c[q] = (j < m) ? w.ch[j] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int j = j0 + q * blockDim.x;
      if (j < ns) lds[j] = a[q];
      if (j < m) lds[ns + j] = c[q];
    }
  }
  __syncthreads();
}

// STAGE is a template argument so that, once the bodies are inlined, the
// compiler sees the hot arrays as LDS and reads them with ds_read.
template <int KIND, int G, bool STAGE>
__global__ __launch_bounds__(ROOT_BLOCK) void k_root(ProbDesc D, Options opt) {
  extern __shared__ double lds[];
  if constexpr (STAGE) stage_hot(D, lds);
  const int64_t gid = (int64_t)blockIdx.x * ROOT_BLOCK + threadIdx.x;
  const int k = (int)(gid / G);
  if (k >= D.n) return;
  if constexpr (STAGE) root_body<KIND, G, true>(D, opt, k, (int)(gid % G), lds, lds + sorted_count(D));
  else root_body<KIND, G>(D, opt, k, (int)(gid % G));
}

// After the root stage: the K_nu test and the outputs of every eigenvalue, the
// repairs of the few that need O(n) passes (check_body, DEFER_BLOCK), the vectors.
//
// Up to FIN_MAX, one launch (k_finish).  Column blocks take `cols` consecutive
// eigenvalues: test and outputs, one lane each, then the columns that are final,
// BLOCK * RPT rows at a time with the rows' data in registers.  The repairs are
// left to the redo blocks, first in the grid: block b asks of k = b, b +
// redo_blocks, ... (one each up to three times the compute units, finish_redo_blocks),
// re-solves those on all its lanes from arrays staged in LDS and writes their columns,
// so a repair's chain of passes (10 us) runs beside the other blocks instead of between
// two launches (n = 512: 11.6 us against 20 us for check, repair and vectors; n = 1025
// complex 16 us against 23 us).
//
// Above, a launch each (k_check, k_repair, k_vec): the redo blocks would reserve
// 16 n bytes of LDS in every block of the launch, and clusters of listed
// eigenvalues need the even spread of a list that a launch boundary completes
// (graded n = 4096: 49 us against 66 us in one launch; handing the list out
// inside the launch by device-scope atomics 430 us).
constexpr int FIN_MAX = 1280;
constexpr int FIN_COLS = 32;       // most columns a block takes
constexpr int FIN_VALUES = 64;     // eigenvalues a column block takes, without vectors

struct FinStage {
  double pv[FIN_COLS], sf[FIN_COLS], mu[FIN_COLS], inrm[FIN_COLS], sig[FIN_COLS];
  int col[FIN_COLS];     // output column, -1: none (past a deflated problem's order, or a redo block's)
  int redo[BLOCK];       // eigenvalues this block re-solves
  int redo_count;
};

template <int KIND, int W, int RPT>
__device__ inline void finish_rows(const ProbDesc& D, int rt, int nc, const FinStage& L) {
  static_assert(W == 1 || W == 2, "one or two rows per store");
  static_assert(RPT % W == 0, "rows per thread");
  constexpr int PER = RPT / W;   // stores per column per thread
  const int n = D.n;
  const int r0 = rt * BLOCK * RPT + threadIdx.x * W;
  double dr[RPT], num[RPT], im[KIND == KIND_HERM ? RPT : 1];
#pragma unroll
  for (int q = 0; q < PER; ++q) {
#pragma unroll
    for (int e = 0; e < W; ++e) {
      const int r = r0 + q * BLOCK * W + e;
      const bool body = (KIND == KIND_DPR1) ? (r < n) : (r < n - 1);
      dr[q * W + e] = body ? in_pole<KIND>(D, r) : 0.0;
      if constexpr (KIND == KIND_HERM) {
        num[q] = body ? D.z[2 * r] : 0.0;
        im[q] = body ? D.z[2 * r + 1] : 0.0;
      } else {
        num[q * W + e] = body ? ((KIND == KIND_SVD) ? dr[q * W + e] * D.z[r] : D.z[r]) : 0.0;
      }
    }
  }
  for (int c = 0; c < nc; ++c) {
    const int col = L.col[c];
    if (col < 0) continue;
    const double pv = L.pv[c], s = L.sf[c], mu = L.mu[c], inrm = L.inrm[c];
    const double sigma = (KIND == KIND_SVD) ? L.sig[c] : 0.0;
    double* vc = D.V + (size_t)col * (size_t)D.ldv * (KIND == KIND_HERM ? 2 : 1);
    double* uc = (KIND == KIND_SVD && D.U) ? D.U + (size_t)col * (size_t)D.ldu : nullptr;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int r = r0 + q * BLOCK * W;
      if (r >= n) continue;   // W = 2: n is even, so r + 1 < n as well
      if constexpr (KIND == KIND_HERM) {
        double ur, ui;
        vec_entry_c(dr[q], num[q], im[q], r == n - 1, pv, s, mu, inrm, &ur, &ui);
        const v2d u = {ur, ui};
        __builtin_nontemporal_store(u, (v2d*)vc + r);
      } else if constexpr (W == 1) {
        const double v = vec_entry<KIND>(dr[q], num[q], r == n - 1, pv, s, mu, inrm);
        __builtin_nontemporal_store(v, vc + r);
        if (KIND == KIND_SVD && uc) __builtin_nontemporal_store(svd_left_d(D, sigma, v, r == n - 1, dr[q]), uc + r);
      } else {
        const double v0 = vec_entry<KIND>(dr[2 * q], num[2 * q], false, pv, s, mu, inrm);
        const double v1 = vec_entry<KIND>(dr[2 * q + 1], num[2 * q + 1], r + 1 == n - 1, pv, s, mu, inrm);
        const v2d vv = {v0, v1};
        __builtin_nontemporal_store(vv, (v2d*)(vc + r));
        if (KIND == KIND_SVD && uc) {
          const v2d uu = {svd_left_d(D, sigma, v0, false, dr[2 * q]),
                          svd_left_d(D, sigma, v1, r + 1 == n - 1, dr[2 * q + 1])};
          __builtin_nontemporal_store(uu, (v2d*)(uc + r));
        }
      }
    }
  }
}

// output column of the finished eigenvalue k, -1 past a deflated problem's order
template <int KIND>
__device__ inline int finish_col(const ProbDesc& D, const Ws& w, int k) {
  if constexpr (KIND == KIND_ARROW) {
    const int nd = deflated_count(w);
    if (nd > 0) return (k <= reduced_m(w)) ? k + count_above(w.dv, nd, w.lr[k], false) : -1;
  }
  if constexpr (KIND == KIND_DPR1) {
    if (D.neg) return D.n - 1 - k;
  }
  return k;
}

// column data of the finished eigenvalue k into slot c (its final shift pair is
// in the workspace)
template <int KIND>
__device__ inline void finish_stage(const ProbDesc& D, const Ws& w, int k, int c, FinStage& L) {
  const int col = finish_col<KIND>(D, w, k);
  L.col[c] = col;
  if (col < 0) return;
  L.pv[c] = w.pv[col];
  L.sf[c] = w.sf[col];
  L.mu[c] = w.mu[col];
  L.inrm[c] = w.inrm[col];
  if constexpr (KIND == KIND_SVD) L.sig[c] = D.lam[col];
}

template <int KIND, int W, int RPT>
__global__ __launch_bounds__(BLOCK) void k_finish(ProbDesc D, Options opt, int redo_blocks, int cols) {
  extern __shared__ double lds[];
  constexpr int SK = (KIND == KIND_HERM) ? KIND_ARROW : KIND;   // solved as the real arrowhead on |z|
  __shared__ FinStage L;
  const Ws w = ws_view(D.ws, D.n);
  const int t = threadIdx.x;
  const bool redo = (int)blockIdx.x < redo_blocks;
  const int step = redo ? redo_blocks : 1;
  const int k0 = redo ? (int)blockIdx.x : ((int)blockIdx.x - redo_blocks) * cols;
  // at most BLOCK (finish_redo_blocks), at most cols
  const int mine = redo ? (D.n - k0 + step - 1) / step : min(D.n - k0, cols);
  if (t == 0) L.redo_count = 0;
  if (blockIdx.x == 0 && t == 0) *sort_done(w) = 0u;   // for the next call
  __syncthreads();
  if (t < mine) {
    const int k = k0 + t * step;
    const bool ask = check_body<SK, 1, false, DEFER_BLOCK>(D, opt, k, 0, nullptr, nullptr, !redo);
    if (redo && ask) L.redo[atomicAdd(&L.redo_count, 1)] = k;
    if (!redo && D.V) {
      if (ask) L.col[t] = -1;
      else finish_stage<KIND>(D, w, k, t, L);
    }
  }
  __syncthreads();
  const int count = redo ? L.redo_count : (D.V ? mine : 0);
  bool staged = redo && count > 0;
  if (staged) stage_hot(D, lds);
  for (int q0 = 0; q0 < count; q0 += FIN_COLS) {
    const int nc = min(FIN_COLS, count - q0);
    if (redo) {
      for (int q = 0; q < nc; ++q) {
        check_body<SK, BLOCK, true>(D, opt, L.redo[q0 + q], t, lds, lds + sorted_count(D));
        if (t == 0 && D.V) finish_stage<KIND>(D, w, L.redo[q0 + q], q, L);   // thread 0 wrote what it reads
      }
      if (!D.V) continue;
      __syncthreads();
    }
    for (int rt = 0; rt * BLOCK * RPT < D.n; ++rt) finish_rows<KIND, W, RPT>(D, rt, nc, L);
    if (redo) __syncthreads();
  }
  if constexpr (KIND == KIND_ARROW) {
    // The deflated eigenpairs, in turn.  The one eigenvalue that decides a pair's
    // column is re-solved here as well where it is to be repaired (the same values as
    // its own block's).  The poles above the pair's are counted by the whole block, as
    // a search would be a chain of loads (62 us a call at n = 300, counted 57).
    const int nd = redo ? deflated_count(w) : 0;
    const int mr = reduced_m(w);
    for (int s = (int)blockIdx.x; s < nd; s += redo_blocks) {
      const double v = w.dv[s];
      double d[FIN_MAX / BLOCK];
#pragma unroll
      for (int q = 0; q < FIN_MAX / BLOCK; ++q) d[q] = t + q * BLOCK < mr ? w.ds[t + q * BLOCK] : NAN;
      int above = 0;
#pragma unroll
      for (int q = 0; q < FIN_MAX / BLOCK; ++q) above += __syncthreads_count(d[q] >= v);
      const bool solve = check_body<SK, 1, false, DEFER_BLOCK>(D, opt, above, 0, nullptr, nullptr, false);
      if (solve) {
        if (!staged) stage_hot(D, lds);
        staged = true;
        check_body<SK, BLOCK, true>(D, opt, above, t, lds, lds + sorted_count(D));
        __syncthreads();
      }
      const int col = s + above + (rival_key<SK>(w, above, solve) >= v ? 1 : 0);
      if (t == 0) place_deflated_at(D, w, s, col);
      if (D.V) {
        double* vc = D.V + (size_t)col * (size_t)D.ldv;
        for (int r = t; r < D.n; r += BLOCK)
          __builtin_nontemporal_store(r < D.n - 1 ? deflated_entry(w, s, w.iperm[r], D.z[r]) : 0.0, vc + r);
      }
    }
  }
}

// One lane per eigenvalue, in small blocks that spread over the compute units:
// scalar work bound by latency.  Eigenvalues that need a repair are listed.
constexpr int CHECK_BLOCK = 64;

template <int KIND>
__global__ __launch_bounds__(CHECK_BLOCK) void k_check(ProbDesc D, Options opt) {
  const int k = (int)(blockIdx.x * CHECK_BLOCK + threadIdx.x);
  if (k >= D.n) return;
  if (k == 0) *sort_done(ws_view(D.ws, D.n)) = 0u;   // for the next call
  if (check_body<KIND, 1, false, DEFER_BLOCK>(D, opt, k, 0)) defer_repair(ws_view(D.ws, D.n), D.n, k, 0);
}

// The listed eigenvalues, a block each; blocks beyond the list's length return.  Without
// vectors also the deflated pairs of a reducible arrowhead, each of which needs one final
// eigenvalue (deflated_rival): a thread places those whose rival the check finished, and
// the block that re-solves a listed one places its pairs.  A launch behind this one for
// them costs every call (n = 1281, values alone: 53.7 -> 52.3 us,
// graded n = 4096 with a quarter of the shaft zero 111.8 -> 106.0).
constexpr int REPAIR_BLOCK = 256;

template <int KIND, bool STAGE>
__global__ __launch_bounds__(REPAIR_BLOCK) void k_repair(ProbDesc D, Options opt) {
  extern __shared__ double lds[];
  __shared__ int first[REPAIR_BLOCK], past[REPAIR_BLOCK];   // the pairs of the block's listed eigenvalues
  const Ws w = ws_view(D.ws, D.n);
  const uint32_t count = min(*repair_count(w), (uint32_t)D.n);
  const uint32_t pairs = (KIND == KIND_ARROW && !D.V) ? (uint32_t)deflated_count(w) : 0u;
  const uint32_t step = gridDim.x, total = max(count, pairs);
  if (blockIdx.x >= total) return;
  if constexpr (STAGE) stage_hot(D, lds);
  const uint32_t* list = repair_list(w, D.n);
  for (uint64_t e0 = blockIdx.x; e0 < total; e0 += (uint64_t)REPAIR_BLOCK * step) {   // e0 + t step: thread t's
    if (KIND == KIND_ARROW && pairs > 0u) {
      const uint64_t e = e0 + (uint64_t)threadIdx.x * step;
      if (e < count) {
        rival_pairs(w, (int)list[e], &first[threadIdx.x], &past[threadIdx.x]);
      }
      if (e < pairs) {
        const int s = (int)e, k = deflated_rival(w, w.dv[s]);
        if (!check_body<KIND, 1, false, DEFER_BLOCK>(D, opt, k, 0, nullptr, nullptr, false))
          place_deflated_at(D, w, s, s + k + (rival_key<KIND>(w, k, false) >= w.dv[s] ? 1 : 0));
      }
      __syncthreads();
    }
    for (uint32_t q = 0; q < (uint32_t)REPAIR_BLOCK && e0 + (uint64_t)q * step < count; ++q) {
      const int k = (int)list[e0 + (uint64_t)q * step];
      if (k < 0 || k >= D.n) continue;
      check_body<KIND, REPAIR_BLOCK, STAGE>(D, opt, k, threadIdx.x, lds, lds + sorted_count(D));
      if (KIND == KIND_ARROW && pairs > 0u) {
        __syncthreads();
        const double key = rival_key<KIND>(w, k, true);
        for (int s = first[q] + (int)threadIdx.x; s < past[q]; s += REPAIR_BLOCK)
          place_deflated_at(D, w, s, s + k + (key >= w.dv[s] ? 1 : 0));
      }
    }
    if (KIND == KIND_ARROW && pairs > 0u) __syncthreads();
  }
}

// The deflated eigenpairs of a reducible arrowhead (n > FIN_MAX), by `blocks` blocks in
// turn: placed among the solved ones, whose values are final, and their vectors.  The
// columns are nobody else's, so these blocks ride behind the others of the vector
// launch; a launch of their own takes 4.6 us also for the usual irreducible input,
// where every block returns at once.
__device__ inline void defl_pairs(const ProbDesc& D, int b, int blocks) {
  __shared__ int col;
  const Ws w = ws_view(D.ws, D.n);
  const int nd = deflated_count(w);
  for (int s = b; s < nd; s += blocks) {
    if (threadIdx.x == 0) col = place_deflated(D, w, s);
    __syncthreads();
    double* vc = D.V + (size_t)col * (size_t)D.ldv;
    for (int r = threadIdx.x; r < D.n; r += BLOCK)
      __builtin_nontemporal_store(r < D.n - 1 ? deflated_entry(w, s, w.iperm[r], D.z[r]) : 0.0, vc + r);
    __syncthreads();
  }
}

// BLOCK * RPT rows of `cols` columns a block; blocks from `tiles` on: the deflated pairs
template <int KIND, int W, int RPT>
__global__ __launch_bounds__(BLOCK) void k_vec(ProbDesc D, int row_tiles, int cols, int tiles) {
  __shared__ FinStage L;
  if constexpr (KIND == KIND_ARROW) {
    if ((int)blockIdx.x >= tiles) {
      defl_pairs(D, (int)blockIdx.x - tiles, (int)gridDim.x - tiles);
      return;
    }
  }
  const Ws w = ws_view(D.ws, D.n);
  const int ct = blockIdx.x / row_tiles, k0 = ct * cols;
  const int nc = min(D.n - k0, cols);
  if ((int)threadIdx.x < nc) finish_stage<KIND>(D, w, k0 + threadIdx.x, threadIdx.x, L);
  __syncthreads();
  finish_rows<KIND, W, RPT>(D, blockIdx.x - ct * row_tiles, nc, L);
}

__device__ inline double from_lane(double v, int src) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), src),
                          __builtin_amdgcn_readlane(__double2loint(v), src));
}

// The columns that the lanes of `mask` hold (output column, shift pair, 1/||x||,
// sigma), by one wavefront: COL_ROWS rows a lane at a time, loaded together, then
// every column's entries from them.  W rows a store (2: 16-byte stores, n and the
// leading dimensions even).  ds: the poles in the caller's row order in LDS, or null
// (read from the caller's array).  The values are vec_entry's; its tests are taken
// out of the entries, which share the wavefronts' issue slots with the root stage:
// the corner row is written on its own, a zero shaft entry occurs only in a deflated
// problem (zeros), and an offset of 0 (all but Remark 2(b)) is not subtracted.
constexpr int COL_ROWS = 8;

template <int KIND, int W>
__device__ __forceinline__ void wave_columns(const ProbDesc& D, uint64_t mask, int col, double pv, double s, double mu,
                                             double inrm, double sig, int lane, const double* ds, bool zeros) {
  constexpr int R = COL_ROWS, PER = R / W;
  constexpr bool CPLX = KIND == KIND_HERM;
  const int n = D.n;
  const int body = (KIND == KIND_DPR1) ? n : n - 1;   // rows of the formula; the corner row is the last one else
  for (int base = 0; base < n; base += 64 * R) {
    double dr[R], num[R], im[CPLX ? R : 1];
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int r = base + (q / W) * 64 * W + lane * W + q % W;
      const bool in = r < body;
      dr[q] = in ? (ds ? ds[r] : in_pole<KIND>(D, r)) : 0.0;
      num[q] = in ? D.z[CPLX ? 2 * r : r] : 0.0;
      if constexpr (CPLX) im[q] = in ? D.z[2 * r + 1] : 0.0;
      if constexpr (KIND == KIND_SVD) num[q] *= dr[q];
    }
    for (uint64_t left = mask; left; left &= left - 1) {
      const int src = __builtin_ctzll(left);
      const size_t c = (size_t)__builtin_amdgcn_readlane(col, src);
      const double cpv = from_lane(pv, src), cs = from_lane(s, src), cmu = from_lane(mu, src), ci = from_lane(inrm, src);
      const double csig = (KIND == KIND_SVD) ? from_lane(sig, src) : 0.0;
      double* vc = D.V + c * (size_t)D.ldv * (CPLX ? 2 : 1);
      double* uc = (KIND == KIND_SVD && D.U) ? D.U + c * (size_t)D.ldu : nullptr;
      double f[R];   // 1 / ((d_r - pole - s) - mu)
      if (cs == 0.0) {
#pragma unroll
        for (int q = 0; q < R; ++q) f[q] = recip(pdiff<KIND>(dr[q], cpv) - cmu);
      } else {
#pragma unroll
        for (int q = 0; q < R; ++q) f[q] = recip((pdiff<KIND>(dr[q], cpv) - cs) - cmu);
      }
#pragma unroll
      for (int q = 0; q < PER; ++q) {
        const int r = base + q * 64 * W + lane * W;
        if (r >= n) continue;   // W = 2: n is even, so r + 1 < n as well
        auto value = [&](int e, int row) {
          if (KIND != KIND_DPR1 && row >= body) return -ci;
          if (KIND == KIND_ARROW && zeros && num[e] == 0.0) return 0.0;
          return (num[e] * ci) * f[e];
        };
        if constexpr (CPLX) {
          const v2d u = {r < body ? (num[q] * ci) * f[q] : -ci, r < body ? (im[q] * ci) * f[q] : 0.0};
          __builtin_nontemporal_store(u, (v2d*)vc + r);
        } else if constexpr (W == 1) {
          const double v = value(q, r);
          __builtin_nontemporal_store(v, vc + r);
          if (KIND == KIND_SVD && uc) __builtin_nontemporal_store(svd_left(D, csig, v, r), uc + r);
        } else {
          const v2d vv = {value(2 * q, r), value(2 * q + 1, r + 1)};
          __builtin_nontemporal_store(vv, (v2d*)(vc + r));
          if (KIND == KIND_SVD && uc) {
            const v2d uu = {svd_left(D, csig, vv.x, r), svd_left(D, csig, vv.y, r + 1)};
            __builtin_nontemporal_store(uu, (v2d*)(uc + r));
          }
        }
      }
    }
  }
}

// Root stage and vectors of a large problem (n > BIG_MIN) in one launch.  A block
// of BIG_BLOCK threads (a compute unit's, with the staged arrays) takes `each`
// consecutive eigenvalues; its wavefronts take them one by one, all 64 lanes each,
// and an eigenvalue whose neighbours' first passes are done too is tested and
// output by whichever wavefront completes the three; its column waits in LDS.  At
// most BIG_WRITERS wavefronts at a time write waiting columns, BIG_TAKE a sweep,
// so that the stores run while the others compute (all 16 would write together,
// since they compute in step); when the eigenvalues are taken, all do.  Nobody
// waits: the wavefront that adds the last column finds it.
// Left for the launches behind it (BigTail): the first and last eigenvalue of each
// block, whose neighbours are another block's, and those that need a repair.
//
// HOT 1: poles and weights in LDS; HOT 2: the poles alone, where both do not fit.
// At n = 16384 the root stage was bound by the L2: 72 bytes a term, 860 us at 22
// TB/s; with the poles in LDS 40 bytes, and bound by issued instructions, 603 us
// (n = 8192 285 -> 209 us, 5000 120 -> 101 us).  With the columns 890 us, where
// root stage and vectors took 860 + 387: a writing wavefront is one fewer computing
// (two or eight writers at a time: 900 and 920 us).
constexpr int BIG_BLOCK = 1024;
constexpr int BIG_MIN = 4608;              // below, k_root's smaller blocks spread better: 4096 graded 67 us against 82
constexpr int BIG_EACH = BIG_BLOCK / 64;   // fewest eigenvalues a block takes
constexpr int BIG_WRITERS = 4;
constexpr int BIG_TAKE = 4;

struct BigCol {   // a waiting column
  double pv, sf, mu, inrm, sig;
  int col;
  int done;       // first passes done of the eigenvalue and its neighbours
};

static size_t big_lds(int each) { return (size_t)each * sizeof(BigCol) + (size_t)((each + 31) / 32) * sizeof(uint32_t); }

template <int KIND, int HOT>
__global__ __launch_bounds__(BIG_BLOCK) void k_root_big(ProbDesc D, Options opt, int each, bool pair) {
  constexpr int SK = (KIND == KIND_HERM) ? KIND_ARROW : KIND;
  extern __shared__ double lds[];
  __shared__ int next, writers;
  const Ws w = ws_view(D.ws, D.n);
  const int ns = sorted_count(D);
  BigCol* cols = (BigCol*)(lds + (HOT == 1 ? ns + D.n - 1 : ns));
  uint32_t* waiting = (uint32_t*)(cols + each);   // a bit per column
  const int words = (each + 31) / 32;
  const int k0 = (int)blockIdx.x * each, k1 = min(D.n, k0 + each);
  const int lane = threadIdx.x & 63;
  if (threadIdx.x == 0) {
    next = k0;
    writers = 0;
  }
  for (int q = threadIdx.x; q < each; q += BIG_BLOCK) cols[q].done = 0;
  for (int q = threadIdx.x; q < words; q += BIG_BLOCK) waiting[q] = 0u;
  if constexpr (HOT == 1) {
    stage_hot(D, lds);
  } else {
    for (int j = threadIdx.x; j < ns; j += BIG_BLOCK) lds[j] = w.ds[j];
    __syncthreads();
  }
  const bool zeros = KIND == KIND_ARROW && deflated_count(w) > 0;
  const double* rows = (*in_order(w) && !zeros) ? lds : nullptr;
  const bool vec = D.V != nullptr;
  // one sweep over up to BIG_TAKE waiting columns; false when there are none
  auto write_some = [&]() -> bool {
    uint32_t got = 0u;
    int at = 0;
    if (lane == 0) {
      for (; at < words; ++at) {
        uint32_t pick = 0u, have = waiting[at];
        for (int q = 0; q < BIG_TAKE && have; ++q) {
          pick |= have & (0u - have);
          have &= have - 1u;
        }
        if (pick) got = atomicAnd(&waiting[at], ~pick) & pick;
        if (got) break;
      }
    }
    got = __builtin_amdgcn_readfirstlane(got);
    if (!got) return false;
    at = __builtin_amdgcn_readfirstlane(at);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    const int count = __popc(got);
    uint32_t left = got;
    for (int q = 0; q < lane && q < count - 1; ++q) left &= left - 1u;   // lane q: the q-th column
    const BigCol c = cols[32 * at + __ffs(left) - 1];
    const uint64_t mask = (1ull << count) - 1ull;
    if (KIND != KIND_HERM && pair)
      wave_columns<KIND, KIND == KIND_HERM ? 1 : 2>(D, mask, c.col, c.pv, c.sf, c.mu, c.inrm, c.sig, lane, rows, zeros);
    else wave_columns<KIND, 1>(D, mask, c.col, c.pv, c.sf, c.mu, c.inrm, c.sig, lane, rows, zeros);
    return true;
  };
  for (;;) {
    int k = 0;
    if (lane == 0) k = atomicAdd(&next, 1);
    k = __builtin_amdgcn_readfirstlane(k);
    const bool more = k < k1;
    if (more) {
      root_body<SK, 64, HOT>(D, opt, k, lane, lds, lds + ns);
      // lanes 0..2: k - 1, k and k + 1 have one more first pass
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      const int q = k - 1 + lane;
      bool ready = false;
      if (lane < 3 && q >= k0 && q < k1) {
        const int need = 1 + (q > 0 ? 1 : 0) + (q < D.n - 1 ? 1 : 0);   // at a block's edge never reached
        ready = atomicAdd(&cols[q - k0].done, 1) + 1 == need;
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
      if (ready) {
        if (check_body<SK, 1, false, DEFER_BLOCK>(D, opt, q, 0)) {
          defer_repair(w, D.n, q, 0);
        } else if (vec) {
          const int col = finish_col<KIND>(D, w, q);
          if (col >= 0) {   // this lane wrote them
            BigCol& c = cols[q - k0];
            c.col = col;
            c.pv = w.pv[col];
            c.sf = w.sf[col];
            c.mu = w.mu[col];
            c.inrm = w.inrm[col];
            c.sig = (KIND == KIND_SVD) ? D.lam[col] : 0.0;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            atomicOr(&waiting[(q - k0) >> 5], 1u << ((q - k0) & 31));
          }
        }
      }
    }
    // all lanes together again before the next uniform test: without an operation
    // that the compiler keeps convergent here, it may send the lanes that know the
    // test's outcome from above (no vectors) straight round the loop, whose head then
    // reads lane 0 without lane 0
    __builtin_amdgcn_wave_barrier();
    if (!more) break;
    if (vec) {
      int place = 0;
      if (lane == 0) place = atomicAdd(&writers, 1);
      if (__builtin_amdgcn_readfirstlane(place) < BIG_WRITERS) write_some();
      if (lane == 0) atomicSub(&writers, 1);
    }
    __builtin_amdgcn_wave_barrier();
  }
  // every eigenvalue is taken: what waits, and what this wavefront added
  if (vec)
    while (write_some()) __builtin_amdgcn_wave_barrier();
}

// What k_root_big leaves: index e of a block's edge eigenvalue, or -1 where the
// problem's own end makes it no edge
struct BigTail {
  int each, blocks;
  __device__ int edge(int e, int n) const {
    const int b = e >> 1;
    if (e & 1) return b + 1 < blocks ? (b + 1) * each - 1 : -1;
    return b > 0 ? b * each : -1;
  }
};

// the test and outputs of the edges, one lane each
template <int KIND>
__global__ __launch_bounds__(CHECK_BLOCK) void k_check_edges(ProbDesc D, Options opt, BigTail T) {
  const int e = (int)(blockIdx.x * CHECK_BLOCK + threadIdx.x);
  if (e >= 2 * T.blocks) return;
  if (e == 0) *sort_done(ws_view(D.ws, D.n)) = 0u;   // for the next call
  const int k = T.edge(e, D.n);
  if (k < 0) return;
  if (check_body<KIND, 1, false, DEFER_BLOCK>(D, opt, k, 0)) defer_repair(ws_view(D.ws, D.n), D.n, k, 0);
}

// the columns of the edges and of the repaired eigenvalues (an edge that was
// repaired is written twice, with the same values), BLOCK * RPT rows of TAIL_COLS a
// turn; blocks from `takers` on: the deflated pairs
constexpr int TAIL_COLS = 4;

template <int KIND, int W, int RPT>
__global__ __launch_bounds__(BLOCK) void k_vec_tail(ProbDesc D, int row_tiles, BigTail T, int takers) {
  __shared__ FinStage L;
  if constexpr (KIND == KIND_ARROW) {
    if ((int)blockIdx.x >= takers) {
      defl_pairs(D, (int)blockIdx.x - takers, (int)gridDim.x - takers);
      return;
    }
  }
  const Ws w = ws_view(D.ws, D.n);
  const int listed = (int)min(*repair_count(w), (uint32_t)D.n);
  const uint32_t* list = repair_list(w, D.n);
  const int total = 2 * T.blocks + listed;
  const int turns = (total + TAIL_COLS - 1) / TAIL_COLS * row_tiles;
  for (int turn = blockIdx.x; turn < turns; turn += takers) {
    const int ct = turn / row_tiles, e0 = ct * TAIL_COLS;
    const int nc = min(total - e0, TAIL_COLS);
    if ((int)threadIdx.x < nc) {
      const int e = e0 + threadIdx.x;
      const int k = e < 2 * T.blocks ? T.edge(e, D.n) : (int)list[e - 2 * T.blocks];
      if (k >= 0 && k < D.n) finish_stage<KIND>(D, w, k, threadIdx.x, L);
      else L.col[threadIdx.x] = -1;
    }
    __syncthreads();
    finish_rows<KIND, W, RPT>(D, turn - ct * row_tiles, nc, L);
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// host side

// A launch whose timing events, when given, are stamped by the dispatch itself
// at the kernel's start and end: no marker packets between the launches, which
// would add a dispatch gap of their own at every stage boundary.
template <typename F, typename... A>
static void launch_timed(F kern, dim3 grid, dim3 block, size_t lds, hipStream_t st, hipEvent_t e0, hipEvent_t e1,
                         A... args) {
  if (e0 || e1) hipExtLaunchKernelGGL(kern, grid, block, (uint32_t)lds, st, e0, e1, 0u, args...);
  else hipLaunchKernelGGL(kern, grid, block, lds, st, args...);
}

template <int KIND, int G>
static void launch_root(const ProbDesc& D, const Options& opt, hipStream_t st, size_t lds, hipEvent_t e0,
                        hipEvent_t e1) {
  const dim3 grid((unsigned)(((int64_t)D.n * G + ROOT_BLOCK - 1) / ROOT_BLOCK));
  if (lds > 0) launch_timed(k_root<KIND, G, true>, grid, dim3(ROOT_BLOCK), lds, st, e0, e1, D, opt);
  else launch_timed(k_root<KIND, G, false>, grid, dim3(ROOT_BLOCK), 0, st, e0, e1, D, opt);
}

template <int KIND>
static void launch_root_any(int G, const ProbDesc& D, const Options& opt, hipStream_t st, size_t lds, hipEvent_t e0,
                            hipEvent_t e1) {
  switch (G) {
    case 1: launch_root<KIND, 1>(D, opt, st, lds, e0, e1); break;
    case 2: launch_root<KIND, 2>(D, opt, st, lds, e0, e1); break;
    case 4: launch_root<KIND, 4>(D, opt, st, lds, e0, e1); break;
    case 8: launch_root<KIND, 8>(D, opt, st, lds, e0, e1); break;
    case 16: launch_root<KIND, 16>(D, opt, st, lds, e0, e1); break;
    case 32: launch_root<KIND, 32>(D, opt, st, lds, e0, e1); break;
    default: launch_root<KIND, 64>(D, opt, st, lds, e0, e1); break;
  }
}

// Rows per thread and columns per block of the vectors: whole columns up to
// FIN_MAX (k_finish), few of them so that the grid keeps a few hundred blocks;
// above (k_vec) wide tiles around n = 4096 and tall ones for larger n.
struct VecShape {
  int rpt, cols;
};

static VecShape vec_shape(int64_t n) {
  if (n > 4096) return VecShape{8, 16};
  if (n > 2048) return VecShape{4, 32};
  if (n > FIN_MAX) return VecShape{4, 8};
  if (n > 512) return VecShape{4, 4};
  return VecShape{2, n > 256 ? 2 : 1};
}

template <int KIND>
static int launch_problem(arrow_handle_t h, const ProbDesc& D);

// one single-problem solve (all launches) on the handle's stream; used by the
// sequential reference path of the batched API
int launch_single(arrow_handle_t h, const ProbDesc& D) {
  switch (D.kind) {
    case KIND_ARROW: return launch_problem<KIND_ARROW>(h, D);
    case KIND_DPR1: return launch_problem<KIND_DPR1>(h, D);
    case KIND_HERM: return launch_problem<KIND_HERM>(h, D);
    default: return launch_problem<KIND_SVD>(h, D);
  }
}

// A Hermitian problem is sorted and its weights formed as KIND_HERM, then
// solved by the real arrowhead's root, check and repair kernels.
template <int KIND>
static int launch_problem(arrow_handle_t h, const ProbDesc& D) {
  constexpr int SK = (KIND == KIND_HERM) ? KIND_ARROW : KIND;
  hipStream_t st = h->stream;
  (void)hipGetLastError();
  const bool tm = h->timing && h->ev_made;
  // a timed call takes the event set the previous timed call did not use
  const int es = (tm && h->timed_calls > 0) ? 1 - h->ev_set : 0;
  hipEvent_t* ev = h->ev[es];
  auto at = [&](int e) -> hipEvent_t { return tm ? ev[e] : nullptr; };
  const int ms = sorted_count(D);
  // every stage boundary is the start (or end) of a kernel
  if (ms <= PREP_MAX) {
    if (ms <= PREP_ONE) {
      const int groups = ms <= 64 ? 1 : (ms <= 128 ? 2 : 4);
      launch_timed(k_prep<KIND, true>, dim3(1), dim3(PREP_BLOCK), 0, st, at(0), at(1), D, D.d, groups);
    } else {
      launch_timed(k_prep<KIND, false>, dim3((unsigned)((ms + 63) / 64)), dim3(PREP_BLOCK), 0, st, at(0), at(1), D,
                   D.d, 1);
    }
  } else {
    launch_timed(k_front<KIND>, dim3(1), dim3(FRONT_BLOCK), 0, st, at(0), nullptr, D);
    // about SORT_GRID blocks in all (they return at once when k_front found the
    // order), each comparing its key tile against one or more chunks
    constexpr int64_t SORT_GRID = 256;
    const int64_t jt = (ms + SORT_BLOCK - 1) / SORT_BLOCK;
    const int64_t nchunks = (ms + SORT_CHUNK - 1) / SORT_CHUNK;
    const int64_t lc = std::max<int64_t>(1, std::min<int64_t>({nchunks, SORT_GRID / jt, 65535}));
    launch_timed(k_sort<KIND>, dim3((unsigned)jt, (unsigned)lc), dim3(SORT_BLOCK), 0, st, at(1), nullptr, D,
                 SORT_CHUNK, (int)nchunks);
  }
  // the root and finish stages are timed by their kernels' own start and end;
  // the stages between take up the dispatch gaps
  const size_t hot = (size_t)(ms + D.n - 1) * sizeof(double);
  // the large problems' kernel, where at least the poles fit a compute unit's LDS
  // and the caller did not ask for another number of lanes
  const int each = (int)std::max<int64_t>(BIG_EACH, (D.n + h->cus - 1) / h->cus);
  const size_t poles = (size_t)ms * sizeof(double), extra = big_lds(each) + 1024;   // and a little static LDS
  // Not where the caller takes the shift pairs or either half of them: the shift of
  // Remark 2(b) is formed from the first pass's mu, of which an ill-conditioned eigenvalue
  // has few digits, and the pair's mu shows all of them (20 decades, n = 6000: 5e-9 between
  // two lane counts, the eigenvalues equal).  The pairs stay those of the tuned lane count.
  const bool big = D.n > BIG_MIN && large_kernel_lanes(h, D.n) && !D.shift && !D.mu && poles + extra <= h->lds_max;
  const BigTail tail{each, (D.n + each - 1) / each};
  const bool hot_both = hot + extra <= h->lds_max;
  const bool pair_rows = KIND != KIND_HERM && (D.n % 2 == 0) && (D.ldv % 2 == 0) && (((uintptr_t)D.V & 15) == 0) &&
                         (!D.U || ((D.ldu % 2 == 0) && (((uintptr_t)D.U & 15) == 0)));
  if (big) {
    const dim3 grid((unsigned)tail.blocks);
    const size_t lds = (hot_both ? hot : poles) + big_lds(each);
    if (hot_both) launch_timed(k_root_big<KIND, 1>, grid, dim3(BIG_BLOCK), lds, st, at(2), at(3), D, h->opt, each, pair_rows);
    else launch_timed(k_root_big<KIND, 2>, grid, dim3(BIG_BLOCK), lds, st, at(2), at(3), D, h->opt, each, pair_rows);
  } else {
    const size_t lds = (hot <= h->lds_max) ? hot : 0;
    launch_root_any<SK>(single_lanes(h, D.n), D, h->opt, st, lds, at(2), at(3));
  }
  // One launch finishes small problems.  By bisection (ARROW_OPT_ROOT 0) a repair takes
  // 30 us instead of 10, so there only while every redo block has one eigenvalue: two
  // listed ones in turn cost more than the launches saved (one block a compute unit,
  // arrowhead n = 257 129 -> 140 us, DPR1 n = 1000 193 -> 223)
  const int redo_blocks = finish_redo_blocks(D.n, h->cus, BLOCK);
  const bool one_finish = D.n <= FIN_MAX && (h->opt.root == ROOT_RATIONAL || redo_blocks == D.n);
  {
    VecShape sh = vec_shape(D.n);
    if (!one_finish && sh.rpt < 4) sh = VecShape{4, 4};   // k_vec's smallest
    // 16-byte stores: a complex entry each, or two rows where every column starts on 16 bytes
    const bool pair = pair_rows;
    constexpr int W2 = KIND == KIND_HERM ? 1 : 2;
    auto by_shape = [&](auto&& go) {   // go(rows per store, rows per thread)
      using one = std::integral_constant<int, 1>;
      using two = std::integral_constant<int, W2>;
      if (sh.rpt == 8) { if (pair) go(two(), std::integral_constant<int, 8>()); else go(one(), std::integral_constant<int, 8>()); }
      else if (sh.rpt == 4) { if (pair) go(two(), std::integral_constant<int, 4>()); else go(one(), std::integral_constant<int, 4>()); }
      else { if (pair) go(two(), std::integral_constant<int, 2>()); else go(one(), std::integral_constant<int, 2>()); }
    };
    if (one_finish) {
      const int cols = D.V ? sh.cols : FIN_VALUES;
      const dim3 grid((unsigned)(redo_blocks + (D.n + cols - 1) / cols));
      by_shape([&](auto wd, auto rpt) {
        if constexpr (decltype(rpt)::value <= 4)
          launch_timed(k_finish<KIND, decltype(wd)::value, decltype(rpt)::value>, grid, dim3(BLOCK), hot, st, at(4),
                       at(5), D, h->opt, redo_blocks, cols);
      });
    } else {
      if (big) {
        hipLaunchKernelGGL(k_check_edges<SK>, dim3((unsigned)((2 * tail.blocks + CHECK_BLOCK - 1) / CHECK_BLOCK)),
                           dim3(CHECK_BLOCK), 0, st, D, h->opt, tail);
      } else {
        hipLaunchKernelGGL(k_check<SK>, dim3((unsigned)((D.n + CHECK_BLOCK - 1) / CHECK_BLOCK)), dim3(CHECK_BLOCK), 0,
                           st, D, h->opt);
      }
      const size_t lds_r = (hot + 4096 <= h->lds_max) ? hot : 0;   // the block reductions add a little static LDS
      const dim3 grid((unsigned)std::min<int64_t>(D.n, h->cus));
      hipEvent_t r0 = D.V ? nullptr : at(4), r1 = D.V ? nullptr : at(5);
      if (lds_r > 0) launch_timed(k_repair<SK, true>, grid, dim3(REPAIR_BLOCK), lds_r, st, r0, r1, D, h->opt);
      else launch_timed(k_repair<SK, false>, grid, dim3(REPAIR_BLOCK), 0, st, r0, r1, D, h->opt);
      if (D.V) {
        by_shape([&](auto wd, auto rpt) {
          if constexpr (decltype(rpt)::value >= 4) {
            const int row_tiles = (int)((D.n + (int64_t)BLOCK * sh.rpt - 1) / ((int64_t)BLOCK * sh.rpt));
            const int defl = KIND == KIND_ARROW ? (int)std::min<int64_t>(D.n - 1, h->cus) : 0;
            if (big) {
              const int takers = 2 * h->cus;
              launch_timed(k_vec_tail<KIND, decltype(wd)::value, decltype(rpt)::value>,
                           dim3((unsigned)(takers + defl)), dim3(BLOCK), 0, st, at(4), at(5), D, row_tiles, tail,
                           takers);
              return;
            }
            const int tiles = (int)(row_tiles * ((D.n + sh.cols - 1) / sh.cols));
            launch_timed(k_vec<KIND, decltype(wd)::value, decltype(rpt)::value>, dim3((unsigned)(tiles + defl)),
                         dim3(BLOCK), 0, st, at(4), at(5), D, row_tiles, sh.cols, tiles);
          }
        });
      }
    }
  }
  if (tm) {
    h->ev_set = es;
    h->timed_calls = std::min(h->timed_calls + 1, 2);
  }
  h->last_n = D.n;
  h->last_ws = D.ws;
  return hipGetLastError() == hipSuccess ? ARROW_OK : ARROW_ERR_HIP;
}

static bool finite_h(double x) { return x - x == 0.0; }

// ---------------------------------------------------------------------------
// Scratch of arrow_eig_noalloc: one problem's workspace at the largest order
// that call takes, in static device memory (each device holds its own copy
// until the process ends).  Host code never uses the array's name as a device
// address: arrow_create looks up each device's address once, with that device
// current, and every later use goes through scratch_dev[].
constexpr size_t NOALLOC_WS_DOUBLES = 16 + (size_t)ARROW_NOALLOC_N_MAX * 26;
static __device__ __align__(256) double scratch[NOALLOC_WS_DOUBLES];
constexpr int SCRATCH_DEVICES = 64;
static double* scratch_dev[SCRATCH_DEVICES];
static int scratch_rc[SCRATCH_DEVICES];   // 0: not looked up yet, 1: found, -1: lookup failed
static std::mutex scratch_mu;

static void scratch_lookup(int device) {
  if (device < 0 || device >= SCRATCH_DEVICES) return;
  std::lock_guard<std::mutex> lock(scratch_mu);
  if (scratch_rc[device] != 0) return;
  DeviceGuard g(device);
  void* ptr = nullptr;
  if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) == hipSuccess && ptr) {
    scratch_dev[device] = (double*)ptr;
    scratch_rc[device] = 1;
  } else {
    (void)hipGetLastError();
    scratch_rc[device] = -1;
  }
}

static double* scratch_of(int device) {
  if (device < 0 || device >= SCRATCH_DEVICES) return nullptr;
  std::lock_guard<std::mutex> lock(scratch_mu);
  return scratch_rc[device] == 1 ? scratch_dev[device] : nullptr;
}

static_assert(NOALLOC_WS_DOUBLES == 16 + (size_t)ARROW_NOALLOC_N_MAX * 26, "workspace of ws_doubles()");

extern "C" {

int arrow_create(arrow_handle_t* h, int device) {
  if (!h) return -1;
  int count = 0;
  if (hipGetDeviceCount(&count) != hipSuccess) return ARROW_ERR_HIP;
  if (device < 0 || device >= count) return -2;
  arrow_handle_t p = (arrow_handle_t)calloc(1, sizeof(*p));
  if (!p) return ARROW_ERR_NOMEM;
  p->device = device;
  p->stream = nullptr;
  p->opt.tau_nu = 100.0;
  p->opt.tau_zero = 10.0;
  p->opt.fp64_b = 0;
  p->opt.tau_b = 0.0;
  p->opt.remedies = 1;
  p->opt.root = ROOT_RATIONAL;
  p->lanes = 0;
  {
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, device) != hipSuccess) v = 0;
    p->lds_max = v > 0 ? (size_t)v : 0;
    v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) v = 0;
    p->cus = v > 0 ? v : 1;
  }
  p->ntab[ARROW_SCHEDULE_SINGLE] = 0;
  default_batch_table(p);
  scratch_lookup(device);   // arrow_eig_noalloc's scratch address on this device
  p->magic = HANDLE_MAGIC;
  *h = p;
  return ARROW_OK;
}

int arrow_destroy(arrow_handle_t h) {
  if (!valid(h)) return ARROW_ERR_STATE;
  DeviceGuard g(h->device);
  (void)hipStreamSynchronize(h->stream);
  tridiag_release(h);
  if (h->ws) (void)hipFree(h->ws);
  if (h->ev_made)
    for (int k = 0; k < 2; ++k)
      for (int e = 0; e < 6; ++e) (void)hipEventDestroy(h->ev[k][e]);
  h->magic = 0;
  free(h);
  return ARROW_OK;
}

int arrow_set_stream(arrow_handle_t h, void* hip_stream) {
  if (!valid(h)) return ARROW_ERR_STATE;
  h->stream = (hipStream_t)hip_stream;
  return ARROW_OK;
}

int arrow_set_option(arrow_handle_t h, int option, double value) {
  if (!valid(h)) return ARROW_ERR_STATE;
  switch (option) {
    case ARROW_OPT_TAU_NU:
      if (!(value >= 1.0)) return -3;
      h->opt.tau_nu = value;
      return ARROW_OK;
    case ARROW_OPT_TAU_ZERO:
      if (!(value >= 1.0)) return -3;
      h->opt.tau_zero = value;
      return ARROW_OK;
    case ARROW_OPT_TAU_B:
      if (!(value >= 0.0 && value < INFINITY)) return -3;
      h->opt.tau_b = value;
      return ARROW_OK;
    case ARROW_OPT_FP64_B:
      h->opt.fp64_b = value != 0.0;
      return ARROW_OK;
    case ARROW_OPT_REMEDIES:
      h->opt.remedies = value != 0.0;
      return ARROW_OK;
    case ARROW_OPT_ROOT:
      if (value != 0.0 && value != 1.0) return -3;
      h->opt.root = (int)value;
      return ARROW_OK;
    case ARROW_OPT_CHECK_LANES: {   // accepted without effect
      const int g = (int)value;
      return ((double)g == value && (g == 0 || (g >= 4 && g <= 64 && (g & (g - 1)) == 0))) ? ARROW_OK : -3;
    }
    case ARROW_OPT_TIMING:
      if (value != 0.0 && !h->ev_made) {
        DeviceGuard g(h->device);
        for (int k = 0; k < 2; ++k)
          for (int e = 0; e < 6; ++e)
            if (hipEventCreate(&h->ev[k][e]) != hipSuccess) return ARROW_ERR_HIP;
        h->ev_made = 1;
      }
      h->timing = value != 0.0;
      return ARROW_OK;
    case ARROW_OPT_LANES: {
      const int g = (int)value;
      if (g != 0 && g != 1 && g != 2 && g != 4 && g != 8 && g != 16 && g != 32 && g != 64) return -3;
      h->lanes = g;
      return ARROW_OK;
    }
    default:
      return -2;
  }
}

size_t arrow_workspace_size(int64_t n) { return order_ok(n) ? ws_doubles(n) * sizeof(double) : 0; }

int arrow_timing_of(arrow_handle_t h, int age, double* ms) {
  if (!valid(h)) return -1;
  if (!ms) return -2;
  if (age != 0 && age != 1) return -3;
  if (h->timed_calls <= age) return ARROW_ERR_STATE;
  DeviceGuard g(h->device);
  hipEvent_t* ev = h->ev[age == 0 ? h->ev_set : 1 - h->ev_set];
  if (hipEventSynchronize(ev[5]) != hipSuccess) return ARROW_ERR_HIP;
  for (int e = 0; e < 5; ++e) {
    float t = 0.0f;
    if (hipEventElapsedTime(&t, ev[e], ev[e + 1]) != hipSuccess) return ARROW_ERR_HIP;
    ms[e] = t;
  }
  return ARROW_OK;
}

int arrow_last_timing(arrow_handle_t h, double* ms) { return arrow_timing_of(h, 0, ms); }

int arrow_conditions(arrow_handle_t h, double* kb, double* knu) {
  if (!valid(h)) return -1;
  if (!h->last_ws || h->last_n < 1) return ARROW_ERR_STATE;
  DeviceGuard g(h->device);
  const Ws w = ws_view(h->last_ws, h->last_n);
  const size_t bytes = (size_t)h->last_n * sizeof(double);
  if (kb && hipMemcpyAsync(kb, w.kbc, bytes, hipMemcpyDeviceToDevice, h->stream) != hipSuccess) return ARROW_ERR_HIP;
  if (knu && hipMemcpyAsync(knu, w.knu, bytes, hipMemcpyDeviceToDevice, h->stream) != hipSuccess) return ARROW_ERR_HIP;
  return ARROW_OK;
}

int arrow_last_counters(arrow_handle_t h, int64_t* out) {
  if (!valid(h)) return -1;
  if (!out) return -2;
  if (!h->ws || h->last_n < 1) return ARROW_ERR_STATE;
  DeviceGuard g(h->device);
  if (hipStreamSynchronize(h->stream) != hipSuccess) return ARROW_ERR_HIP;
  const int64_t n = h->last_n;
  const Ws w = ws_view(h->ws, n);
  int32_t* host = (int32_t*)malloc((size_t)n * 6 * sizeof(int32_t));
  if (!host) return ARROW_ERR_NOMEM;
  if (hipMemcpy(host, w.cnt, (size_t)n * 6 * sizeof(int32_t), hipMemcpyDeviceToHost) != hipSuccess) {
    free(host);
    return ARROW_ERR_HIP;
  }
  for (int c = 0; c < 6; ++c) out[c] = 0;
  for (int64_t k = 0; k < n; ++k)
    for (int c = 0; c < 6; ++c) out[c] += host[6 * k + c];
  out[6] = n;
  free(host);
  return ARROW_OK;
}

}  // extern "C"

// arrow_eig's body: ws = null grows and uses the handle's workspace, else ws
// (room for ws_doubles(n) doubles) is used and nothing is allocated
static int arrow_eig_in(arrow_handle_t h, int64_t n, const double* d, const double* z, double alpha,
                        double* lambda, double* V, int64_t ldv, double* shift, double* mu, uint32_t* info,
                        double* ws) {
  if (!valid(h)) return -1;
  if (!order_ok(n)) return -2;
  if (n > 1 && !d) return -3;
  if (n > 1 && !z) return -4;
  if (!finite_h(alpha)) return -5;
  if (!lambda) return -6;
  if (V && ldv < n) return -8;
  DeviceGuard g(h->device);
  if (!ws) {
    const int rc = ensure_ws(h, ws_doubles(n));
    if (rc) return rc;
    ws = h->ws;
  }
  ProbDesc D{};
  D.kind = KIND_ARROW;
  D.n = (int32_t)n;
  D.d = d;
  D.z = z;
  D.scalar = alpha;
  D.lam = lambda;
  D.V = V;
  D.ldv = ldv;
  D.shift = shift;
  D.mu = mu;
  D.info = info;
  D.ws = ws;
  return launch_problem<KIND_ARROW>(h, D);
}

extern "C" {

int arrow_eig(arrow_handle_t h, int64_t n, const double* d, const double* z, double alpha, double* lambda,
              double* V, int64_t ldv, double* shift, double* mu, uint32_t* info) {
  return arrow_eig_in(h, n, d, z, alpha, lambda, V, ldv, shift, mu, info, nullptr);
}

int arrow_eig_noalloc(arrow_handle_t h, int64_t n, const double* d, const double* z, double alpha,
                      double* lambda, double* V, int64_t ldv, double* shift, double* mu, uint32_t* info) {
  if (!valid(h)) return -1;
  if (n > ARROW_NOALLOC_N_MAX) return -2;   // beyond what the scratch holds
  double* ws = scratch_of(h->device);
  if (!ws) return ARROW_ERR_HIP;            // the address lookup at arrow_create failed
  return arrow_eig_in(h, n, d, z, alpha, lambda, V, ldv, shift, mu, info, ws);
}

int arrow_eig_herm(arrow_handle_t h, int64_t n, const double* d, const double* z, double alpha, double* lambda,
                   double* U, int64_t ldu, double* shift, double* mu, uint32_t* info) {
  if (!valid(h)) return -1;
  if (!order_ok(n)) return -2;
  if (n > 1 && !d) return -3;
  if (n > 1 && (!z || ((uintptr_t)z & 7))) return -4;
  if (!finite_h(alpha)) return -5;
  if (!lambda) return -6;
  if (U && ((uintptr_t)U & 15)) return -7;
  if (U && ldu < n) return -8;
  DeviceGuard g(h->device);
  const int rc = ensure_ws(h, ws_doubles(n));
  if (rc) return rc;
  ProbDesc D{};
  D.kind = KIND_HERM;
  D.n = (int32_t)n;
  D.d = d;
  D.z = z;
  D.scalar = alpha;
  D.lam = lambda;
  D.V = U;
  D.ldv = ldu;
  D.shift = shift;
  D.mu = mu;
  D.info = info;
  D.ws = h->ws;
  return launch_problem<KIND_HERM>(h, D);
}

int dpr1_eig(arrow_handle_t h, int64_t n, const double* d, const double* u, double rho, double* lambda,
             double* Q, int64_t ldq, uint32_t* info) {
  if (!valid(h)) return -1;
  if (!order_ok(n)) return -2;
  if (!d) return -3;
  if (!u) return -4;
  if (!finite_h(rho) || rho == 0.0) return -5;
  if (!lambda) return -6;
  if (Q && ldq < n) return -8;
  DeviceGuard g(h->device);
  const int rc = ensure_ws(h, ws_doubles(n));
  if (rc) return rc;
  ProbDesc D{};
  D.kind = KIND_DPR1;
  D.n = (int32_t)n;
  D.neg = rho < 0.0;
  D.d = d;
  D.z = u;
  D.scalar = fabs(rho);
  D.lam = lambda;
  D.V = Q;
  D.ldv = ldq;
  D.info = info;
  D.ws = h->ws;
  return launch_problem<KIND_DPR1>(h, D);
}

int arrow_svd(arrow_handle_t h, int64_t n, const double* d, const double* z, double alpha, double* sigma,
              double* U, int64_t ldu, double* V, int64_t ldv, uint32_t* info) {
  if (!valid(h)) return -1;
  if (!order_ok(n)) return -2;
  if (n > 1 && !d) return -3;
  if (n > 1 && !z) return -4;
  if (!finite_h(alpha)) return -5;
  if (!sigma) return -6;
  if (U && ldu < n) return -8;
  if (V && ldv < n) return -10;
  if (U && !V) return -9;  // left vectors are formed from the right ones
  DeviceGuard g(h->device);
  const int rc = ensure_ws(h, ws_doubles(n));
  if (rc) return rc;
  ProbDesc D{};
  D.kind = KIND_SVD;
  D.n = (int32_t)n;
  D.d = d;
  D.z = z;
  D.scalar = alpha;
  D.lam = sigma;
  D.V = V;
  D.ldv = ldv;
  D.U = U;
  D.ldu = ldu;
  D.info = info;
  D.ws = h->ws;
  return launch_problem<KIND_SVD>(h, D);
}

}  // extern "C"
