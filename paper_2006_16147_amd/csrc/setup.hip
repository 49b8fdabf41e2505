// Hierarchy construction on the GPU: coupled aggregation based on compatible
// weighted matching (Section 3.2) and Galerkin coarse operators (Section 3.1).
//
// Built with -ffp-contract=off: weights, prolongator values, Galerkin sums
// and restricted smooth vectors round exactly as written, so the hierarchy is
// bit-for-bit reproducible and equal to the FP64 reference computation.
//
// Per level l (until n_l <= max_coarse):
//   for each of `sweeps` pairwise sweeps on (A_k, w_k):
//     1. edge weights, eq. (weights), sorted into a preference list per vertex
//     2. matching of locally dominant edges under the strict key (weight
//        desc, lo asc, hi asc), in one asynchronous kernel -- the
//        half-approximate maximum-weight matching class of the paper; under
//        a strict key it equals the greedy matching, in whatever order
//     3. aggregate numbering by smallest member (prefix scan)
//     4. pairwise prolongator, eq. (prolongator)
//     5. A_{k+1} = P_k^T A_k P_k, w_{k+1} = P_k^T w_k
//   P_l = P_1 P_2 ... P_m (composed per fine row), A_{l+1} = A_{k=m}.
// Then the l1-Jacobi diagonal (Section 3.3) and, on the coarsest level, a
// dense Cholesky factor and its triangular inverse.

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>

#include "internal.h"

namespace amg {

namespace {

constexpr int32_t kDead = -1;
constexpr int kRapLongCap = 2048;  // per-block buffer for long rows
constexpr int kScanBlock = 1024;
constexpr int kScanPer = 4;

enum : int32_t { kErrArg = 1, kErrSpd = 2, kErrSym = 4 };

double now_ms() {
  return std::chrono::duration<double, std::milli>(
             std::chrono::steady_clock::now().time_since_epoch())
      .count();
}

// ---------------------------------------------------------------------------
// exclusive prefix sum (three passes)
// ---------------------------------------------------------------------------

__device__ int32_t block_exclusive_scan(int32_t v, int32_t *total) {
  __shared__ int32_t wsum[kScanBlock / kWave];
  const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
  int32_t x = v;
  for (int o = 1; o < kWave; o <<= 1) {
    int32_t y = __shfl_up(x, o, kWave);
    if (lane >= o) x += y;
  }
  if (lane == kWave - 1) wsum[wid] = x;
  __syncthreads();
  if (wid == 0) {
    int32_t s = lane < kScanBlock / kWave ? wsum[lane] : 0;
    for (int o = 1; o < kWave; o <<= 1) {
      int32_t y = __shfl_up(s, o, kWave);
      if (lane >= o) s += y;
    }
    if (lane < kScanBlock / kWave) wsum[lane] = s;
  }
  __syncthreads();
  int32_t off = wid > 0 ? wsum[wid - 1] : 0;
  *total = wsum[kScanBlock / kWave - 1];
  __syncthreads();
  return off + x - v;
}

// When a sweep's stages begin on the device, in ticks of its wall clock: kernels
// write it to pinned host memory as they start: no event, wait or copy, and less
// than a microsecond for each of the three per sweep (in device memory, cleared at
// the start and copied at the end, 9 to 17 us a set-up more). The count of the aggregates,
// which the host waits for, goes with the matching.
struct Stamps {
  uint64_t assign, product, end;
};
__device__ __forceinline__ void stamp(uint64_t *at) {
  if (at && blockIdx.x == 0 && threadIdx.x == 0) *at = wall_clock64();
}

// Control block of a pairwise sweep (device), and what the host reads of it:
// the kernel that knows a total writes it, with the block's words, to pinned
// host memory, which saves a copy of its own. Errors have one word for all
// sweeps of a setup (Report::err): a product's error is known only after the
// host has gone on to the next sweep, and is read there.
constexpr int kCtl = 16;
enum : int32_t {
  kCtlErr = 0,       // kErr* (in the host's copy)
  kCtlRounds = 1,    // largest matching round
  kCtlPrefLong = 2,  // rows listed for k_pref_long
  kCtlRapLong = 3,   // rows listed for k_rap_long
  kCtlEntries = 4,   // entries of the sweep's matrix
  kCtlLongest = 5,   // its longest row
  kCtlFlags = 6      // kMatchFlags per queued launch of k_match
};
constexpr int kMatchFlags = 2;  // kLeft, kMoved
constexpr int kMatchQueue = 4;  // launches of k_match between host checks, at most
static_assert(kCtlFlags + kMatchQueue * kMatchFlags <= kCtl, "control block");
struct Report {
  const int32_t *from = nullptr;  // kCtl words
  const int32_t *err = nullptr;   // the setup's kErr* so far
  int32_t *to = nullptr;          // kCtl + 1 words, the total last; null: no report
};

__device__ __forceinline__ void report(const Report &R, int32_t total) {
  if (!R.to) return;
  for (int k = 0; k < kCtl; ++k)
    R.to[k] = __hip_atomic_load(k == kCtlErr ? R.err : &R.from[k], __ATOMIC_RELAXED,
                                __HIP_MEMORY_SCOPE_AGENT);
  R.to[kCtl] = total;
}

// the end of a block's part of a scan (one thread): its sum; a scan of one
// block is complete with it (end: where the total goes, may be null)
__device__ __forceinline__ void scan_block_end(int32_t total, int32_t *bsum, int32_t *end,
                                               const Report &R) {
  if (gridDim.x > 1) {
    bsum[blockIdx.x] = total;
    return;
  }
  bsum[0] = 0;
  bsum[1] = total;
  if (end) *end = total;
  report(R, total);
}

// scan of in[i], or of the lengths e[i] - in[i] of rows [in[i], e[i])
__global__ void __launch_bounds__(kScanBlock) k_scan_local(const int32_t *in, const int32_t *e,
                                                           int32_t *out, int32_t *bsum, int32_t n,
                                                           Report R) {
  const int64_t base = ((int64_t)blockIdx.x * kScanBlock + threadIdx.x) * kScanPer;
  int32_t v[kScanPer];
  int32_t s = 0;
  for (int k = 0; k < kScanPer; ++k) {
    v[k] = base + k < n ? (e ? e[base + k] - in[base + k] : in[base + k]) : 0;
    s += v[k];
  }
  int32_t total;
  int32_t off = block_exclusive_scan(s, &total);
  for (int k = 0; k < kScanPer; ++k) {
    if (base + k < n) out[base + k] = off;
    off += v[k];
  }
  if (threadIdx.x == 0) scan_block_end(total, bsum, out + n, R);
}

// block sums of a scan of more than one block
__global__ void __launch_bounds__(kScanBlock) k_scan_sums(int32_t *bsum, int32_t nb, Report R) {
  int32_t carry = 0;
  for (int32_t c0 = 0; c0 < nb; c0 += kScanBlock * kScanPer) {
    const int32_t base = c0 + threadIdx.x * kScanPer;
    int32_t v[kScanPer];
    int32_t s = 0;
    for (int k = 0; k < kScanPer; ++k) {
      v[k] = base + k < nb ? bsum[base + k] : 0;
      s += v[k];
    }
    int32_t total;
    int32_t off = block_exclusive_scan(s, &total);
    for (int k = 0; k < kScanPer; ++k) {
      if (base + k < nb) bsum[base + k] = carry + off;
      off += v[k];
    }
    carry += total;
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    bsum[nb] = carry;
    report(R, carry);
  }
}

__global__ void k_scan_add(int32_t *out, const int32_t *bsum, int32_t n, int32_t nb) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] += bsum[i / (kScanBlock * kScanPer)];
  if (i == 0) out[n] = bsum[nb];
}

// ---------------------------------------------------------------------------
// small utilities
// ---------------------------------------------------------------------------

template <typename T>
__global__ void k_fill(T *a, T v, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) a[i] = v;
}

// ---------------------------------------------------------------------------
// input validation: structure, positive diagonal, bitwise symmetry
// ---------------------------------------------------------------------------

__device__ __forceinline__ int64_t find_col(const int32_t *ci, int64_t b, int64_t e, int32_t j) {
  int64_t lo = b, hi = e - 1;
  while (lo <= hi) {
    int64_t mid = lo + (hi - lo) / 2;
    int32_t c = ci[mid];
    if (c == j) return mid;
    if (c < j) lo = mid + 1; else hi = mid - 1;
  }
  return -1;
}

// eight lanes per row, each its own entries: an entry's search in the other
// row is a chain of loads (a thread per row: 0.50 ms at 160^3)
__global__ void k_validate(int32_t n, int64_t nnz, const int32_t *rp, const int32_t *ci,
                           const double *val, int32_t *err) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int32_t i = (int32_t)(t / 8), lane = (int32_t)(t % 8);
  if (t / 8 >= n) return;
  int32_t flags = 0;
  if (i == 0 && rp[0] != 0) flags |= kErrArg;
  if (i == n - 1 && (int64_t)rp[n] != nnz) flags |= kErrArg;
  const int64_t b = rp[i], e = rp[i + 1];
  int32_t diag = 0;
  if (b < 0 || e < b || e > nnz) {
    flags |= kErrArg;
  } else {
    for (int64_t k = b + lane; k < e; k += 8) {
      const int32_t j = ci[k];
      const double a = val[k];
      if (j < 0 || j >= n || (k > b && j <= ci[k - 1]) || !isfinite(a)) {
        flags |= kErrArg;
        break;
      }
      if (j == i) {
        diag = 1;
        if (!(a > 0.0)) flags |= kErrSpd;
        continue;
      }
      const int64_t bj = rp[j], ej = rp[j + 1];
      if (bj < 0 || ej < bj || ej > nnz) {
        flags |= kErrArg;
        break;
      }
      const int64_t at = find_col(ci, bj, ej, i);
      if (at < 0 || __double_as_longlong(val[at]) != __double_as_longlong(a)) flags |= kErrSym;
    }
  }
  for (int o = 4; o > 0; o >>= 1) {
    diag |= __shfl_xor(diag, o, 8);
    flags |= __shfl_xor(flags, o, 8);
  }
  if (!diag) flags |= kErrSpd;
  if (flags && lane == 0) atomicOr(err, flags);
}

__global__ void k_check_w(int32_t n, const double *w, int32_t *err) {
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n && !(w[i] != 0.0 && isfinite(w[i]))) atomicOr(err, kErrArg);
}

// One sweep of the smoother on A w = 0: w_out = w - (A w) / m (row sums
// left to right from the first term, as the serial definition)
__global__ void k_smooth_w(int32_t n, const int32_t *rp, const int32_t *ci, const double *val,
                           const double *m, const double *w, double *w_out) {
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int32_t b = rp[i], e = rp[i + 1];
  double t = 0.0;
  if (e > b) {
    t = val[b] * w[ci[b]];
    for (int32_t k = b + 1; k < e; ++k) t = t + val[k] * w[ci[k]];
  }
  w_out[i] = w[i] - t / m[i];
}

// ---------------------------------------------------------------------------
// 1. eq. (weights) and every row's neighbours in order of preference
// ---------------------------------------------------------------------------
//
// c = 1 - ((2 a) w_lo w_hi) / ((a_lolo w_lo) w_lo + (a_hihi w_hi) w_hi) for
// each stored off-diagonal entry, computed in (lo, hi) order so that both
// copies of an edge carry the same bits (A is bitwise symmetric).
//
// The matching's strict key (c descending, lo ascending, hi ascending) orders
// the neighbours j of one vertex v by (c descending, j ascending): those below
// v have lo = j < v, those above lo = v and hi = j. Each row's neighbours are
// sorted once in that order (pref, laid out like the row's entries, the unused
// slot of the diagonal closed by -1); the matching then walks each list once
// and reads no weight again.

// Rows of a sweep's matrix: row i holds the entries [b[i], e[i]) of ci / val.
// A level's CSR is {rp, rp + 1}; the matrices between the sweeps of a level
// keep their rows where the Galerkin product put them, with gaps.
struct RowsOf {
  const int32_t *b, *e, *ci;
  const double *val;
};

// the weight as an unsigned key that orders like it (NaN below every number)
__device__ __forceinline__ uint64_t weight_key(double c) {
  if (!(c == c)) return 0;
  const uint64_t u = (uint64_t)__double_as_longlong(c + 0.0);
  return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}

__device__ __forceinline__ uint64_t edge_key(int32_t i, int32_t j, double a, double wi, double wj,
                                             double di, double dj) {
  const double wl = i < j ? wi : wj, wh = i < j ? wj : wi;
  const double dl = i < j ? di : dj, dh = i < j ? dj : di;
  const double num = ((2.0 * a) * wl) * wh;
  const double den = (dl * wl) * wl + (dh * wh) * wh;
  return weight_key(1.0 - num / den);
}

// diagonal entry of each row
__global__ void k_diag(int32_t n, RowsOf A, double *dg) {
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int64_t k = find_col(A.ci, A.b[i], A.e[i], i);
  dg[i] = k >= 0 ? A.val[k] : 0.0;
}

// Matching state of a vertex, one 64-bit word (read and written whole):
// the low half says whether it is free and proposes to a neighbour (>= 0),
// is a singleton (kDead) or matched to u (kMatched - u); the high half is the
// round in which it came to propose or was settled, see k_match.
constexpr int32_t kMatched = -3;
__device__ __forceinline__ uint64_t pack_state(int32_t round, int32_t s) {
  return ((uint64_t)(uint32_t)round << 32) | (uint32_t)s;
}
__device__ __forceinline__ int32_t state_of(uint64_t w) { return (int32_t)(uint32_t)w; }
__device__ __forceinline__ int32_t round_of(uint64_t w) { return (int32_t)(w >> 32); }

// G lanes per row, two entries per lane: a row of at most 2 G entries is
// ranked in registers, every lane counting the entries ahead of its own while
// each in turn is broadcast. Longer rows are listed for k_pref_long. The
// entries of a wave's rows are consecutive, so its loads are coalesced, and
// every lane has one division; a thread per row measured 120 us a sweep on
// average over a 192^3 setup for the weights alone, stored as 8 bytes each.
// Also the first proposal of every vertex: its first choice.
template <int G>
__global__ void __launch_bounds__(kBlock) k_pref(int32_t n, RowsOf A, const double *__restrict__ w,
                                                 const double *__restrict__ dg,
                                                 int32_t *__restrict__ pref,
                                                 uint64_t *__restrict__ st, int32_t *ovf,
                                                 int32_t *novf, uint64_t *began) {
  stamp(began);
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int32_t i = (int32_t)(t / G);
  const int lane = (int)(t % G);
  if (t / G >= n) return;  // whole groups: no lane of a live group is missing
  const int32_t b = A.b[i], len = A.e[i] - b;
  if (len > 2 * G) {
    if (lane == 0) ovf[atomicAdd(novf, 1)] = i;
    return;
  }
  const double wi = w[i], di = dg[i];
  int32_t j[2];
  uint64_t key[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int32_t e = lane + q * G;
    j[q] = e < len ? A.ci[b + e] : i;
    key[q] = 0;
    if (j[q] != i) key[q] = edge_key(i, j[q], A.val[b + e], wi, w[j[q]], di, dg[j[q]]);
  }
  int32_t rank[2] = {0, 0}, deg = 0;
  const int32_t l0 = min(len, G);
  for (int32_t f = 0; f < l0; ++f) {
    const int32_t jf = __shfl(j[0], f, G);
    const uint64_t kf = __shfl((unsigned long long)key[0], f, G);
    if (jf == i) continue;
    ++deg;
    // entries ascend in j: of two equal weights the earlier entry comes first
    if (kf > key[0] || (kf == key[0] && f < lane)) ++rank[0];
    if (kf >= key[1]) ++rank[1];
  }
  for (int32_t f = G; f < len; ++f) {
    const int32_t jf = __shfl(j[1], f - G, G);
    const uint64_t kf = __shfl((unsigned long long)key[1], f - G, G);
    if (jf == i) continue;
    ++deg;
    if (kf > key[0]) ++rank[0];
    if (kf > key[1] || (kf == key[1] && f - G < lane)) ++rank[1];
  }
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    if (j[q] == i) continue;
    pref[b + rank[q]] = j[q];
    if (rank[q] == 0) st[i] = pack_state(0, j[q]);
  }
  if (lane == 0) {
    if (deg < len) pref[b + deg] = -1;
    if (deg == 0) st[i] = pack_state(0, kDead);
  }
}

// Rows listed by k_pref, one block each, their keys in LDS. A row of more
// than kRapLongCap entries cannot be assembled into a coarse row later: it is
// refused here already (kErrArg) and gets an empty list.
__global__ void __launch_bounds__(kBlock) k_pref_long(
    RowsOf A, const double *__restrict__ w, const double *__restrict__ dg,
    int32_t *__restrict__ pref, uint64_t *__restrict__ st, const int32_t *__restrict__ ovf,
    const int32_t *__restrict__ novf, int32_t *err) {
  __shared__ uint64_t key[kRapLongCap];
  const int32_t count = *novf;
  for (int32_t o = blockIdx.x; o < count; o += gridDim.x) {
    const int32_t i = ovf[o];
    const int32_t b = A.b[i], len = A.e[i] - b;
    if (len > kRapLongCap) {
      if (threadIdx.x == 0) {
        atomicOr(err, kErrArg);
        pref[b] = -1;
        st[i] = pack_state(0, kDead);
      }
      continue;
    }
    const double wi = w[i], di = dg[i];
    __syncthreads();  // the previous row's keys are read no more
    for (int32_t e = threadIdx.x; e < len; e += kBlock) {
      const int32_t j = A.ci[b + e];
      key[e] = j == i ? 0 : edge_key(i, j, A.val[b + e], wi, w[j], di, dg[j]);
    }
    const int64_t dk = find_col(A.ci, b, A.e[i], i);
    const int32_t de = dk >= 0 ? (int32_t)(dk - b) : -1;  // the diagonal's place, not ranked
    const int32_t deg = len - (de >= 0 ? 1 : 0);
    __syncthreads();
    for (int32_t e = threadIdx.x; e < len; e += kBlock) {
      if (e == de) continue;
      const uint64_t ke = key[e];
      int32_t rank = 0;
      for (int32_t f = 0; f < len; ++f) {
        const uint64_t kf = key[f];
        rank += (f != de && (kf > ke || (kf == ke && f < e))) ? 1 : 0;
      }
      const int32_t j = A.ci[b + e];
      pref[b + rank] = j;
      if (rank == 0) st[i] = pack_state(0, j);
    }
    if (threadIdx.x == 0) {
      if (deg < len) pref[b + deg] = -1;
      if (deg == 0) st[i] = pack_state(0, kDead);
    }
  }
}

// ---------------------------------------------------------------------------
// 2. matching: locally dominant edges
// ---------------------------------------------------------------------------
//
// A free vertex proposes to the first vertex of its list that is not taken; a
// mutual proposal is a locally dominant edge and is matched; a free vertex
// whose list is used up is a singleton. Under the strict key the result does
// not depend on the order of these steps, and each holds on stale reads too:
// a vertex is taken for good, so one seen as taken is; one seen as free that
// is taken by now only delays its proposer; and a proposal from u seen by the
// free vertex v stands, since u leaves v only for v being taken. So there are
// no rounds to wait for: every wave works on its own vertices at its own pace.
// A vertex's word is written by its own thread, to memory for the other blocks
// and to LDS for its own; the one that finds a mutual proposal also writes the
// other end's, with the same value that its thread will write. (Where that
// thread's earlier store of the proposal lands later, the end looks free until
// its thread has seen the match: a delay like any other.)
//
// What bounds it is the chain of dependent steps, not bytes: with every weight
// the same (the Poisson grid) the order of the indices decides, and vertex by
// vertex the matching runs across the grid, about 2.5 N steps on N^3. As one
// kernel per round over all vertices a step cost a launch and a pass over the
// states (29 us at 160^3, 444 rounds, 12.9 ms). Here a block owns a run of
// consecutive vertices, their words in LDS and the next entries of their lists
// in registers, so a step inside it touches no memory; between blocks it costs
// a store and a poll (2.4 ms; 3.3 in the version that the variants here were
// measured against). A wave looks outside when nothing moved inside,
// and waves that wait sleep 2048 clocks between their looks and yield the
// issue slots to those that move: with 64 clocks it was 4.4 ms, and with every
// waiting wave polling all the time the polls filled the fabric and a step
// took 8 us (16.5 ms). Blocks of 256 and 1024 vertices were 5 % and 1 % slower;
// two vertices per thread (twice as many in flight) made no difference.
//
// A wave leaves when its vertices are settled, or when it found nothing new
// kMatchSpin times (it may wait for a block that has not started); the next
// launch goes on from the words in memory. In every launch the best edge left
// is matched or gets nearer to it: a launch without any change (kMoved) means
// that the input was not symmetric.
//
// The high half of a word carries the round of the synchronous algorithm
// (everybody proposes, then all mutual proposals are matched): a vertex
// proposes to x from the round in which the last vertex ahead of x in its list
// was taken, an edge is matched in the round after both ends propose. The
// largest one is the number of rounds that amg_matching_rounds reports.
constexpr int kMatchThreads = 512;  // a vertex per thread
constexpr int kMatchAhead = 8;      // list entries held
constexpr int kMatchSpin = 1024;
enum : int32_t { kLeft = 0, kMoved = 1 };

__global__ void __launch_bounds__(kMatchThreads, 8) k_match(int32_t n,
                                                            const int32_t *__restrict__ rb,
                                                            const int32_t *__restrict__ re,
                                                            const int32_t *__restrict__ pref,
                                                            uint64_t *st, const int32_t *prev,
                                                            int32_t *flags) {
  constexpr int H = kMatchAhead;
  __shared__ uint64_t own[kMatchThreads];
  if (prev && prev[kLeft] == 0) return;
  const int tid = threadIdx.x;
  const int32_t v0 = blockIdx.x * kMatchThreads, v = v0 + tid;
  uint64_t w = v < n ? st[v] : pack_state(0, kDead);
  own[tid] = w;
  int32_t r = round_of(w);  // round of the proposal
  bool live = state_of(w) >= 0;
  int32_t c[H];             // c[0]: the proposal; then the entries after it, -1: the list's end
  int32_t k = 0, e = 0;     // place in the list of the first entry not held, its bound
  auto fetch = [&]() {
#pragma unroll
    for (int i = 0; i < H; ++i) c[i] = k + i < e ? pref[k + i] : -1;
    k += H;
  };
  auto advance = [&]() {
#pragma unroll
    for (int i = 1; i < H; ++i) c[i - 1] = c[i];
    c[H - 1] = -1;
    if (c[0] < 0) fetch();
  };
  if (live) {
    k = rb[v];
    e = re[v];
    fetch();
    // entries ahead of the proposal were found taken by an earlier launch
    while (c[0] != state_of(w)) advance();
  }
  __syncthreads();
  auto inside = [&](int32_t x) { return (uint32_t)(x - v0) < (uint32_t)kMatchThreads; };
  auto look = [&](int32_t x) -> uint64_t {
    if (inside(x))
      return __hip_atomic_load(&own[x - v0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    return __hip_atomic_load(&st[x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  bool outside = true, moved = false;
  int idle = 0, turn = 0;
  while (__any(live)) {
    bool step = false;
    if (live && (outside || inside(c[0]))) {
      w = look(c[0]);
      int32_t s = state_of(w);
      if (s < 0 || s == v) {
        // taken: on to the first of the list that is not
        while (s < 0 && s != kMatched - v) {
          r = max(r, round_of(w));
          advance();
          if (c[0] < 0) break;
          w = look(c[0]);
          s = state_of(w);
        }
        int32_t next = c[0];
        if (next < 0) {  // none left: a singleton
          next = kDead;
        } else if (s == v) {  // mutual: settle both, u waits for nothing else
          r = max(r, round_of(w)) + 1;
          const uint64_t wu = pack_state(r, kMatched - v);
          if (inside(next))
            __hip_atomic_store(&own[next - v0], wu, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_WORKGROUP);
          __hip_atomic_store(&st[next], wu, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          next = kMatched - next;
        } else if (s == kMatched - v) {  // the other end matched it already
          r = round_of(w);
          next = kMatched - next;
        }
        w = pack_state(r, next);
        __hip_atomic_store(&own[tid], w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __hip_atomic_store(&st[v], w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        live = next >= 0;
        step = true;
      }
    }
    if (__any(step)) {
      moved = true;
      idle = 0;
      __builtin_amdgcn_s_setprio(3);
      outside = ++turn % 8 == 0;
    } else if (!outside) {
      outside = true;
    } else {
      if (++idle >= kMatchSpin) break;
      outside = idle < 8 || idle % 4 == 0;
      if (idle >= 8) __builtin_amdgcn_s_setprio(0);
      __builtin_amdgcn_s_sleep(32);
    }
  }
  if (__any(live) && (tid & (kWave - 1)) == 0) flags[kLeft] = 1;
  if (moved && (tid & (kWave - 1)) == 0) flags[kMoved] = 1;
}

// ---------------------------------------------------------------------------
// 3. numbering, 4. eq. (prolongator)
// ---------------------------------------------------------------------------

// mate of every vertex (-1: singleton) from its state; block scan of the
// leaders (the smaller end of a pair, a singleton itself); the largest round,
// the matrix's entries and its longest row
__global__ void __launch_bounds__(kScanBlock) k_lead_scan(int32_t n, const uint64_t *st,
                                                          const int32_t *rb, const int32_t *re,
                                                          int32_t *mate, int32_t *id,
                                                          int32_t *bsum, int32_t *ctl, Report R) {
  __shared__ int32_t most, sum, wide;
  if (threadIdx.x == 0) most = sum = wide = 0;
  const int64_t base = ((int64_t)blockIdx.x * kScanBlock + threadIdx.x) * kScanPer;
  int32_t lead[kScanPer];
  int32_t s = 0, r = 0, c = 0, l = 0;
  for (int k = 0; k < kScanPer; ++k) {
    lead[k] = 0;
    if (base + k >= n) continue;
    const int32_t v = (int32_t)(base + k);
    const uint64_t w = st[v];
    const int32_t x = state_of(w), m = x <= kMatched ? kMatched - x : -1;
    if (x < 0) r = max(r, round_of(w));
    mate[v] = m;
    const int32_t len = re[v] - rb[v];
    c += len;
    l = max(l, len);
    lead[k] = m < 0 || v < m ? 1 : 0;
    s += lead[k];
  }
  int32_t total;
  int32_t off = block_exclusive_scan(s, &total);
  for (int k = 0; k < kScanPer; ++k) {
    if (base + k < n) id[base + k] = off;
    off += lead[k];
  }
  for (int o = kWave / 2; o > 0; o >>= 1) {
    r = max(r, __shfl_xor(r, o, kWave));
    l = max(l, __shfl_xor(l, o, kWave));
    c += __shfl_xor(c, o, kWave);
  }
  if ((threadIdx.x & (kWave - 1)) == 0) {
    atomicMax(&most, r);
    atomicMax(&wide, l);
    atomicAdd(&sum, c);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    if (most > 0) atomicMax(ctl + kCtlRounds, most);
    atomicMax(ctl + kCtlLongest, wide);
    atomicAdd(ctl + kCtlEntries, sum);
    __threadfence();
    scan_block_end(total, bsum, nullptr, R);
  }
}

// aggregates by their smallest member, and the pairwise prolongator:
// pair {i < j}: p_v = w_v / sqrt(w_i w_i + w_j w_j); singleton: w_s / |w_s|
__global__ void k_assign(int32_t n, const int32_t *mate, const int32_t *id, const int32_t *bsum,
                         const double *w, int32_t *agg, int32_t *lead, double *p,
                         uint64_t *began) {
  stamp(began);
  const int32_t v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= n) return;
  const int32_t m = mate[v];
  const int32_t l = m >= 0 && m < v ? m : v;
  const int32_t I = id[l] + bsum[l / (kScanBlock * kScanPer)];
  agg[v] = I;
  if (l == v) lead[I] = v;
  if (m < 0) {
    p[v] = w[v] / fabs(w[v]);
  } else {
    const double wi = w[min(v, m)], wj = w[max(v, m)];
    p[v] = w[v] / sqrt(wi * wi + wj * wj);
  }
}

// ---------------------------------------------------------------------------
// 5. pairwise Galerkin product A_c = P^T A P, w_c = P^T w
// ---------------------------------------------------------------------------
// Entry (I, J) sums (p_lo a_lo,hi) p_hi over the stored fine entries (i, j),
// i in I, j in J, mapped to (lo, hi) = (min, max) and taken in ascending
// (lo, hi) order, starting from the first term. Every structural entry is
// kept. Row I's terms are those of its smaller member's row, then the other's,
// each ascending in j: sorted by (J, lo) with equal keys in that order, they
// are in ascending (lo, hi) order within each J. Row I is left in the first
// slots of the room its terms need; only a level's own matrix is packed.

// block scan of the terms of the coarse rows
__global__ void __launch_bounds__(kScanBlock) k_terms_scan(int32_t nc, const int32_t *lead,
                                                           const int32_t *mate, const int32_t *rb,
                                                           const int32_t *re, int32_t *off,
                                                           int32_t *bsum, uint64_t *began) {
  stamp(began);
  const int64_t base = ((int64_t)blockIdx.x * kScanBlock + threadIdx.x) * kScanPer;
  int32_t len[kScanPer];
  int32_t s = 0;
  for (int k = 0; k < kScanPer; ++k) {
    len[k] = 0;
    if (base + k >= nc) continue;
    const int32_t i0 = lead[base + k], i1 = mate[i0];
    len[k] = re[i0] - rb[i0] + (i1 >= 0 ? re[i1] - rb[i1] : 0);
    s += len[k];
  }
  int32_t total;
  int32_t o = block_exclusive_scan(s, &total);
  for (int k = 0; k < kScanPer; ++k) {
    if (base + k < nc) off[base + k] = o;
    o += len[k];
  }
  if (threadIdx.x == 0) scan_block_end(total, bsum, nullptr, Report{});
}

// LDS written by lanes of this wave is read by its other lanes
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One sweep's coarse matrix in the making
struct Coarsened {
  const int32_t *lead, *mate, *agg;  // coarse -> smaller member, pairs, fine -> coarse
  const double *p, *w;               // prolongator and smooth vector of the fine level
  const int32_t *off, *bsum;         // where row I's room starts: off[I] + its block's bsum
  int32_t *b, *e, *ci;               // the coarse rows
  double *val, *wc, *dg;             // their values, restricted w, diagonal
  const int32_t *size;               // finest members of the fine rows (null: one each)
  int32_t *csize;                    // and of the coarse ones
};

__device__ __forceinline__ void term_of(const RowsOf &A, const Coarsened &C, int32_t f, int32_t k,
                                        uint64_t *key, double *t) {
  const int32_t j = A.ci[k];
  const int32_t lo = min(f, j), hi = max(f, j);
  *key = ((uint64_t)(uint32_t)C.agg[j] << 32) | (uint32_t)lo;
  *t = (C.p[lo] * A.val[k]) * C.p[hi];
}

// G lanes per coarse row, two terms per lane (rows of at most 2 G terms; longer
// ones are listed for k_rap_long): the terms are ranked against the row's keys
// in LDS, put in order there, and the first lane of every run of one column
// adds it up (four terms at most). What bounds it is the gathers of agg and p
// per term; loads of the fine rows and stores of the coarse ones are coalesced.
template <int G>
__global__ void __launch_bounds__(kBlock) k_rap(int32_t nc, RowsOf A, Coarsened C, int32_t *ovf,
                                                int32_t *novf) {
  constexpr int kCap = 2 * G;
  __shared__ uint64_t skey[kBlock / G][kCap];
  __shared__ double sval[kBlock / G][kCap];
  __shared__ int32_t scol[kBlock / G][kCap];
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int32_t I = (int32_t)(t / G);
  const int lane = (int)(t % G), grp = threadIdx.x / G;
  if (t / G >= nc) return;  // whole groups
  const int32_t i0 = C.lead[I], i1 = C.mate[i0];
  const int32_t b0 = A.b[i0], l0 = A.e[i0] - b0;
  const int32_t b1 = i1 >= 0 ? A.b[i1] : 0, l1 = i1 >= 0 ? A.e[i1] - b1 : 0;
  const int32_t len = l0 + l1;
  const int32_t base = C.off[I] + C.bsum[I / (kScanBlock * kScanPer)];
  if (lane == 0) {
    C.b[I] = base;
    double s = C.p[i0] * C.w[i0];
    if (i1 >= 0) s = s + C.p[i1] * C.w[i1];
    C.wc[I] = s;
    C.csize[I] = C.size ? C.size[i0] + (i1 >= 0 ? C.size[i1] : 0) : (i1 >= 0 ? 2 : 1);
  }
  if (len > kCap) {
    if (lane == 0) {
      C.e[I] = base;
      C.dg[I] = 0.0;
      ovf[atomicAdd(novf, 1)] = I;
    }
    return;
  }
  uint64_t key[2];
  double v[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int32_t e = lane + q * G;
    key[q] = 0;
    v[q] = 0.0;
    if (e < len) {
      if (e < l0) term_of(A, C, i0, b0 + e, &key[q], &v[q]);
      else term_of(A, C, i1, b1 + (e - l0), &key[q], &v[q]);
      skey[grp][e] = key[q];
    }
  }
  wave_sync();
  int32_t rank[2] = {0, 0};
  for (int32_t f = 0; f < len; ++f) {
    const uint64_t kf = skey[grp][f];
#pragma unroll
    for (int q = 0; q < 2; ++q)
      if (kf < key[q] || (kf == key[q] && f < lane + q * G)) ++rank[q];
  }
#pragma unroll
  for (int q = 0; q < 2; ++q)
    if (lane + q * G < len) {
      scol[grp][rank[q]] = (int32_t)(key[q] >> 32);
      sval[grp][rank[q]] = v[q];
    }
  wave_sync();
  const int shift = (int)(threadIdx.x & (kWave - 1)) / G * G;
  const uint64_t mask = G == kWave ? ~0ull : (1ull << (G % kWave)) - 1;
  const uint64_t below = lane == 0 ? 0ull : (~0ull >> (kWave - lane));
  int32_t before = 0;
  bool dg = false;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int32_t e = lane + q * G;
    const int32_t J = e < len ? scol[grp][e] : -1;
    const bool head = e < len && (e == 0 || scol[grp][e - 1] != J);
    const uint64_t heads = (__ballot(head) >> shift) & mask;
    if (head) {
      double s = sval[grp][e];
      for (int32_t f = e + 1; f < len && scol[grp][f] == J; ++f) s = s + sval[grp][f];
      const int32_t o = base + before + __popcll(heads & below);
      C.ci[o] = J;
      C.val[o] = s;
      if (J == I) {
        C.dg[I] = s;
        dg = true;
      }
    }
    before += __popcll(heads);
  }
  const uint64_t has = (__ballot(dg) >> shift) & mask;
  if (lane == 0) {
    C.e[I] = base + before;
    if (!has) C.dg[I] = 0.0;
  }
}

// Listed rows, one block each. More than kRapLongCap terms: kErrArg.
__global__ void __launch_bounds__(kBlock) k_rap_long(RowsOf A, Coarsened C, const int32_t *ovf,
                                                     const int32_t *novf, int32_t *err) {
  __shared__ uint64_t skey[kRapLongCap];
  __shared__ double sval[kRapLongCap];
  __shared__ int32_t scol[kRapLongCap];
  __shared__ int32_t wsum[kBlock / kWave];
  constexpr int kPer = kRapLongCap / kBlock;
  const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
  const int32_t count = *novf;
  for (int32_t o = blockIdx.x; o < count; o += gridDim.x) {
    const int32_t I = ovf[o];
    const int32_t i0 = C.lead[I], i1 = C.mate[i0];
    const int32_t b0 = A.b[i0], l0 = A.e[i0] - b0;
    const int32_t b1 = i1 >= 0 ? A.b[i1] : 0, l1 = i1 >= 0 ? A.e[i1] - b1 : 0;
    const int32_t len = l0 + l1, base = C.b[I];
    if (len > kRapLongCap || len < 0) {
      if (threadIdx.x == 0) atomicOr(err, kErrArg);
      continue;
    }
    __syncthreads();  // the previous row's terms are read no more
    double v[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int32_t e = threadIdx.x + q * kBlock;
      v[q] = 0.0;
      if (e >= len) continue;
      uint64_t key;
      if (e < l0) term_of(A, C, i0, b0 + e, &key, &v[q]);
      else term_of(A, C, i1, b1 + (e - l0), &key, &v[q]);
      skey[e] = key;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int32_t e = threadIdx.x + q * kBlock;
      if (e >= len) continue;
      const uint64_t ke = skey[e];
      int32_t rank = 0;
      for (int32_t f = 0; f < len; ++f) {
        const uint64_t kf = skey[f];
        rank += (kf < ke || (kf == ke && f < e)) ? 1 : 0;
      }
      scol[rank] = (int32_t)(ke >> 32);
      sval[rank] = v[q];
    }
    __syncthreads();
    int32_t out = base;
    for (int32_t e0 = 0; e0 < len; e0 += kBlock) {
      const int32_t e = e0 + threadIdx.x;
      const int32_t J = e < len ? scol[e] : -1;
      const bool head = e < len && (e == 0 || scol[e - 1] != J);
      const uint64_t heads = __ballot(head);
      if (lane == 0) wsum[wid] = __popcll(heads);
      __syncthreads();
      int32_t at = out, all = 0;
      for (int k = 0; k < kBlock / kWave; ++k) {
        if (k < wid) at += wsum[k];
        all += wsum[k];
      }
      if (head) {
        double s = sval[e];
        for (int32_t f = e + 1; f < len && scol[f] == J; ++f) s = s + sval[f];
        at += __popcll(heads & (lane == 0 ? 0ull : (~0ull >> (kWave - lane))));
        C.ci[at] = J;
        C.val[at] = s;
        if (J == I) C.dg[I] = s;
      }
      out += all;
      __syncthreads();
    }
    if (threadIdx.x == 0) C.e[I] = out;
  }
}

// rows packed into a CSR, eight lanes per row; and w
__global__ void k_pack(int32_t n, RowsOf A, const double *__restrict__ w,
                       const int32_t *__restrict__ rp, int32_t *__restrict__ ci,
                       double *__restrict__ val, double *__restrict__ wo) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int32_t i = (int32_t)(t / 8), lane = (int32_t)(t % 8);
  if (t / 8 >= n) return;
  if (lane == 0) wo[i] = w[i];
  const int32_t b = A.b[i], len = A.e[i] - b, d = rp[i];
  for (int32_t k = lane; k < len; k += 8) {
    ci[d + k] = A.ci[b + k];
    val[d + k] = A.val[b + k];
  }
}

// ---------------------------------------------------------------------------
// composition of sweeps and aggregate member lists
// ---------------------------------------------------------------------------

// P_l(i) = ((p_1(i) p_2(agg_1(i))) p_3(...)), agg_l = ... o agg_2 o agg_1
constexpr int kMaxSweeps = 8;  // amg_params.sweeps
struct SweepMaps {
  const int32_t *agg[kMaxSweeps];  // fine -> coarse
  const double *p[kMaxSweeps];
  const int32_t *lead[kMaxSweeps], *mate[kMaxSweeps];  // coarse -> members
};
__global__ void k_compose(int32_t n, int32_t sweeps, SweepMaps M, int32_t *agg, double *p,
                          uint64_t *began) {
  stamp(began);
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int32_t a = M.agg[0][i];
  double v = M.p[0][i];
  for (int32_t k = 1; k < sweeps; ++k) {
    v = v * M.p[k][a];
    a = M.agg[k][a];
  }
  agg[i] = a;
  p[i] = v;
}

// The finest members of aggregate I, ascending, at mem[mptr[I]]: the leaves of
// its tree of pairs (at most 2^sweeps), put in order as they come. The first
// of a pair being its smallest member, most come in order.
__global__ void k_members(int32_t nc, int32_t sweeps, SweepMaps M, const int32_t *mptr,
                          int32_t *mem) {
  const int32_t I = blockIdx.x * blockDim.x + threadIdx.x;
  if (I >= nc) return;
  const int32_t o = mptr[I];
  int32_t m = 0;
  for (int32_t t = 0; t < 1 << sweeps; ++t) {
    int32_t v = I;
    for (int32_t k = sweeps - 1; k >= 0 && v >= 0; --k) {
      v = M.lead[k][v];
      if ((t >> k) & 1) v = M.mate[k][v];
    }
    if (v < 0) continue;
    int32_t q = m++;
    for (; q > 0 && mem[o + q - 1] > v; --q) mem[o + q] = mem[o + q - 1];
    mem[o + q] = v;
  }
}

// ---------------------------------------------------------------------------
// l1-Jacobi diagonal, eq. (l1weights) with blocks of one row
// ---------------------------------------------------------------------------

// (a thread per row, the sum's order being fixed; eight loads at a time)
__global__ void k_l1_diag(int32_t n, const int32_t *__restrict__ rp,
                          const int32_t *__restrict__ ci, const double *__restrict__ val,
                          double *__restrict__ m, double *__restrict__ minv) {
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double aii = 0.0, s = 0.0;
  bool first = true;
  const int32_t b = rp[i], e = rp[i + 1];
  for (int32_t k0 = b; k0 < e; k0 += 8) {
    double a[8];
    int32_t c[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int32_t k = k0 + u < e ? k0 + u : e - 1;
      a[u] = val[k];
      c[u] = ci[k];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (k0 + u >= e) continue;
      if (c[u] == i) {
        aii = a[u];
      } else if (first) {
        s = fabs(a[u]);
        first = false;
      } else {
        s = s + fabs(a[u]);
      }
    }
  }
  const double mi = aii + s;
  m[i] = mi;
  minv[i] = 1.0 / mi;
}

// ---------------------------------------------------------------------------
// coarsest level: dense Cholesky A_L = L L^T and L^-1
// ---------------------------------------------------------------------------

__global__ void k_dense_scatter(int32_t n, const int32_t *rp, const int32_t *ci,
                                const double *val, double *D) {
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  for (int32_t k = rp[i]; k < rp[i + 1]; ++k) D[(int64_t)i * n + ci[k]] = val[k];
}

// Right-looking Cholesky of a row-major n x n matrix, above kCholLdsMax: the
// lower triangle becomes L, the strict upper triangle is zeroed. Panels of
// kPanel columns: k_chol_panel factors the panel's diagonal block (every
// block for itself, in LDS: a launch of its own would cost as much) and solves
// the rows below it, k_chol_update takes the panel's terms off the triangle
// behind it in tiles. Every entry loses its terms one at a time in the order k = 0, 1,
// ..., each product rounded before it is taken off, as column after column would.
// A chain of two kernels per panel, 31 us (the block's 32 columns one after the
// other) and 11 us: n = 1155 takes 1.57 ms, and took 192 ms in one block that went
// through the columns with the triangle in L2; n = 337: 4.5 -> 0.43 ms.
constexpr int kPanel = 32;
constexpr int kCholTile = 64;

// diag: kPanel x kPanel doubles per panel, the factored diagonal blocks
__global__ void __launch_bounds__(kBlock) k_chol_panel(int32_t n, int32_t k0, double *D,
                                                       double *diag, int32_t *err) {
  __shared__ double A[kPanel][kPanel + 1];
  const int32_t nb = min(kPanel, n - k0), tid = threadIdx.x;
  for (int32_t e = tid; e < kPanel * kPanel; e += kBlock) {
    const int32_t i = e / kPanel, j = e % kPanel;
    // (past n: the unit matrix, which its steps leave alone)
    A[i][j] = i < nb && j < nb ? (j <= i ? D[(int64_t)(k0 + i) * n + k0 + j] : 0.0)
                               : (i == j ? 1.0 : 0.0);
  }
  __syncthreads();
  for (int32_t k = 0; k < nb; ++k) {
    const double d2 = A[k][k];
    if (!(d2 > 0.0)) {  // the same for every thread
      if (tid == 0 && blockIdx.x == 0) atomicOr(err, kErrSpd);
      return;
    }
    const double d = sqrt(d2);
    __syncthreads();
    if (tid > k && tid < kPanel) A[tid][k] /= d;
    if (tid == k) A[k][k] = d;
    __syncthreads();
    for (int32_t e = tid; e < kPanel * kPanel; e += kBlock) {
      const int32_t i = e / kPanel, j = e % kPanel;
      if (j > k && j <= i) A[i][j] -= A[i][k] * A[j][k];
    }
    __syncthreads();
  }
  if (blockIdx.x == 0)
    for (int32_t e = tid; e < kPanel * kPanel; e += kBlock)
      diag[(int64_t)(k0 / kPanel) * kPanel * kPanel + e] = A[e / kPanel][e % kPanel];
  // the rows below: x_k = t_k / L_kk, later columns lose x_k L_jk
  const int32_t row = k0 + kPanel + blockIdx.x * kBlock + tid;
  if (row >= n) return;
  double *const R = D + (int64_t)row * n + k0;
  double t[kPanel];
#pragma unroll
  for (int k = 0; k < kPanel; ++k) t[k] = R[k];
#pragma unroll
  for (int k = 0; k < kPanel; ++k) {
    t[k] /= A[k][k];
#pragma unroll
    for (int j = k + 1; j < kPanel; ++j) t[j] -= t[k] * A[j][k];
  }
#pragma unroll
  for (int k = 0; k < kPanel; ++k) R[k] = t[k];
}

// rows and columns from c0 on: D_ij -= sum_k L_ik L_jk over the panel before
// c0; block (x, y): tile (y, x) of the lower triangle
__global__ void __launch_bounds__(kBlock) k_chol_update(int32_t n, int32_t c0, double *D) {
  const int32_t bi = blockIdx.y, bj = blockIdx.x;
  if (bj > bi) return;
  __shared__ double Pi[kPanel][kCholTile], Pj[kPanel][kCholTile];
  const int32_t i0 = c0 + bi * kCholTile, j0 = c0 + bj * kCholTile, tid = threadIdx.x;
  for (int32_t e = tid; e < kPanel * kCholTile; e += kBlock) {
    const int32_t r = e / kPanel, k = e % kPanel;
    Pi[k][r] = i0 + r < n ? D[(int64_t)(i0 + r) * n + c0 - kPanel + k] : 0.0;
    Pj[k][r] = j0 + r < n ? D[(int64_t)(j0 + r) * n + c0 - kPanel + k] : 0.0;
  }
  __syncthreads();
  // a thread: rows i0 + ty + 16 u, columns j0 + tx + 16 v
  const int32_t tx = tid % 16, ty = tid / 16;
  double d[4][4];
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int32_t i = i0 + ty + 16 * u, j = j0 + tx + 16 * v;
      d[u][v] = i < n && j <= i ? D[(int64_t)i * n + j] : 0.0;
    }
#pragma unroll 4
  for (int32_t k = 0; k < kPanel; ++k) {
    double a[4], b[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      a[u] = Pi[k][ty + 16 * u];
      b[u] = Pj[k][tx + 16 * u];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int v = 0; v < 4; ++v) d[u][v] -= a[u] * b[v];
  }
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int32_t i = i0 + ty + 16 * u, j = j0 + tx + 16 * v;
      if (i < n && j <= i) D[(int64_t)i * n + j] = d[u][v];
    }
}

// the diagonal blocks into D, zeros above the diagonal
__global__ void k_chol_finish(int32_t n, const double *diag, double *D) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)n * n) return;
  const int32_t i = (int32_t)(e / n), j = (int32_t)(e % n);
  if (j > i)
    D[e] = 0.0;
  else if (i / kPanel == j / kPanel)
    D[e] = diag[((int64_t)(i / kPanel) * kPanel + i % kPanel) * kPanel + j % kPanel];
}

// Cholesky column by column of the packed lower triangle held in LDS (n (n + 1) / 2 doubles
// and the factor's diagonal, up to 159.4 KB: n <= 200, the default max_coarse):
// the same steps on the same numbers, with every access of the n steps in LDS
// instead of L2. The pivot's square root is taken by every thread that divides
// by it, so a step has two barriers. What bounds it is the chain of n steps of
// a square root, a division and two LDS trips (1.1 us each): 137 us at n = 125;
// n = 141, through L2 before, 435 -> 168 us.
constexpr int kCholLdsMax = 200;
static_assert((kCholLdsMax * (kCholLdsMax + 1) / 2 + kCholLdsMax) * sizeof(double) <= 163840 - 64,
              "LDS triangle");
__global__ void __launch_bounds__(1024) k_cholesky_lds(int32_t n, double *D, int32_t *err) {
  extern __shared__ double tri[];  // row i of the lower triangle at i (i + 1) / 2
  double *const piv = tri + n * (n + 1) / 2;
  auto at = [&](int32_t i, int32_t j) -> double & { return tri[i * (i + 1) / 2 + j]; };
  for (int32_t e = threadIdx.x; e < n * (n + 1) / 2; e += blockDim.x) {
    int32_t i = (int32_t)((sqrt(8.0 * e + 1.0) - 1.0) / 2.0);
    while (i * (i + 1) / 2 > e) --i;
    while ((i + 1) * (i + 2) / 2 <= e) ++i;
    tri[e] = D[(int64_t)i * n + (e - i * (i + 1) / 2)];
  }
  __syncthreads();
  for (int32_t k = 0; k < n; ++k) {
    const double d2 = at(k, k);
    if (!(d2 > 0.0)) {  // the same for every thread
      if (threadIdx.x == 0) atomicOr(err, kErrSpd);
      return;
    }
    const double d = sqrt(d2);
    if (threadIdx.x == 0) piv[k] = d;
    for (int32_t i = k + 1 + threadIdx.x; i < n; i += blockDim.x) at(i, k) /= d;
    __syncthreads();
    for (int32_t i = k + 1 + (int32_t)threadIdx.x / 32; i < n; i += (int32_t)blockDim.x / 32)
      for (int32_t j = k + 1 + (int32_t)threadIdx.x % 32; j <= i; j += 32)
        at(i, j) -= at(i, k) * at(j, k);
    __syncthreads();
  }
  for (int32_t e = threadIdx.x; e < n * n; e += blockDim.x) {
    const int32_t i = e / n, j = e % n;
    D[e] = j > i ? 0.0 : (j == i ? piv[i] : at(i, j));
  }
}

// X = L^-1, one block per column j: forward substitution of L x = e_j in its
// right-looking form. Once x_i = t_i / L_ii is known, every later row r takes
// off its term L_ri x_i, so each partial sum t_r loses its terms in the order
// k = j, j + 1, ..., r - 1 of the row-by-row substitution (the same numbers).
// t and the diagonal of L live in LDS; each thread owns the rows tid + s *
// kTriThreads and loads their entries of the next column of L while the
// current step runs, so a step waits on no memory access.
constexpr int kTriThreads = 256;
static_assert(AMG_MAX_DENSE % kTriThreads == 0, "whole rows per thread");
static_assert(2 * sizeof(double) * AMG_MAX_DENSE <= 65536, "t and the diagonal fit in LDS");
template <int S>  // rows per thread: S * kTriThreads >= n
__global__ void __launch_bounds__(kTriThreads) k_tri_inverse(int32_t n,
                                                             const double *__restrict__ L,
                                                             double *__restrict__ X) {
  extern __shared__ double tri_sh[];  // t[n], then the diagonal of L
  double *t = tri_sh, *dg = tri_sh + n;
  const int32_t j = blockIdx.x, tid = threadIdx.x;
  for (int32_t r = tid; r < n; r += kTriThreads) {
    t[r] = r == j ? 1.0 : 0.0;
    dg[r] = L[(int64_t)r * n + r];
    if (r < j) X[(int64_t)r * n + j] = 0.0;
  }
  double ln[S];  // this thread's rows' entries of column i of L
#pragma unroll
  for (int q = 0; q < S; ++q) {
    const int32_t r = tid + q * kTriThreads;
    ln[q] = r > j && r < n ? L[(int64_t)r * n + j] : 0.0;
  }
  __syncthreads();
  for (int32_t i = j; i < n; ++i) {
    const double x = t[i] / dg[i];
    if (tid == 0) X[(int64_t)i * n + j] = x;
    double lc[S];
#pragma unroll
    for (int q = 0; q < S; ++q) {
      const int32_t r = tid + q * kTriThreads;
      lc[q] = ln[q];
      ln[q] = r > i + 1 && r < n ? L[(int64_t)r * n + i + 1] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < S; ++q) {
      const int32_t r = tid + q * kTriThreads;
      if (r > i && r < n) t[r] -= lc[q] * x;
    }
    __syncthreads();
  }
}

// A^-1 = L^-T L^-1: entry (i, j) sums X(k, i) X(k, j) over k >= max(i, j)
__global__ void k_inverse_from_factor(int32_t n, const double *X, double *Ainv) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)n * n) return;
  const int32_t i = (int32_t)(e / n), j = (int32_t)(e % n);
  double s = 0.0;
  for (int32_t k = max(i, j); k < n; ++k) s += X[(int64_t)k * n + i] * X[(int64_t)k * n + j];
  Ainv[e] = s;
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

inline int32_t grid(int64_t n) { return ceil_div(n > 0 ? n : 1, kBlock); }

// block count of the exclusive scan of n values (its block sums take nb + 1)
int32_t scan_blocks(int32_t n) { return ceil_div(n > 0 ? n : 1, kScanBlock * kScanPer); }

// exclusive scan with the caller's block-sum scratch (scan_blocks(n) + 1
// ints): of in[i], or with `e` of e[i] - in[i]; one kernel for one block
void scan_exclusive_i32_with(const int32_t *in, const int32_t *e, int32_t *out, int32_t n,
                             int32_t *bsum, hipStream_t s, const Report &R = Report{}) {
  const int32_t nb = scan_blocks(n);
  k_scan_local<<<nb, kScanBlock, 0, s>>>(in, e, out, bsum, n, R);
  if (nb == 1) return;
  k_scan_sums<<<1, kScanBlock, 0, s>>>(bsum, nb, R);
  k_scan_add<<<grid((int64_t)n + 1), kBlock, 0, s>>>(out, bsum, n, nb);
}

// Device memory for the temporaries of one setup call: a few large pool
// blocks, cut in order and given back together when the setup ends. On this
// runtime a stream-ordered allocation or free takes tens of microseconds of
// host time, a setup needs hundreds of them, and between its latency-bound
// kernels the GPU waits for the host; cut from the arena they cost nothing,
// at the price of keeping every temporary of the setup until its end.
struct Arena {
  int device;
  hipStream_t s;
  size_t chunk;  // block size: a quarter of the first sweep's temporaries, 1-256 MB
  std::vector<void *> blocks;
  char *cur = nullptr;
  size_t left = 0;
  Arena(const amg_hierarchy *h, int64_t n, int64_t nnz) : device(h->device), s(h->stream) {
    const double q = (36.0 * (double)n + 32.0 * (double)nnz) / 4;
    const double mb = double(1 << 20);
    chunk = (size_t)(q < mb ? mb : (q > 256 * mb ? 256 * mb : q));
    chunk = (chunk + (1 << 20) - 1) / (1 << 20) * (1 << 20);
  }
  Arena(const Arena &) = delete;
  Arena &operator=(const Arena &) = delete;
  ~Arena() { stream_free(device, s, blocks); }
  amg_status get(void **p, size_t bytes) {
    bytes = (bytes + 255) / 256 * 256;
    if (bytes > chunk / 4) {  // a large request gets a block of its own
      void *q = nullptr;
      AMG_TRY(stream_alloc(device, s, &q, bytes));
      blocks.push_back(q);
      *p = q;
      return AMG_OK;
    }
    if (bytes > left) {
      void *q = nullptr;
      AMG_TRY(stream_alloc(device, s, &q, chunk));
      blocks.push_back(q);
      cur = static_cast<char *>(q);
      left = chunk;
    }
    *p = cur;
    cur += bytes;
    left -= bytes;
    return AMG_OK;
  }
};

// temporaries of one setup call (not owned by the hierarchy): cut from the
// setup's arena while one runs (dropping them then does nothing), else pool
// allocations released in stream order when dropped or destroyed
struct Tmp {
  int device;
  hipStream_t s;
  Arena *arena;
  std::vector<void *> ptrs;
  explicit Tmp(const amg_hierarchy *h)
      : device(h->device), s(h->stream), arena(static_cast<Arena *>(h->setup_arena)) {}
  Tmp(const Tmp &) = delete;
  Tmp &operator=(const Tmp &) = delete;
  ~Tmp() { stream_free(device, s, ptrs); }
  template <typename T>
  amg_status get(T **p, size_t count) {
    void *q = nullptr;
    if (arena) {
      AMG_TRY(arena->get(&q, count * sizeof(T) + 16));
    } else {
      AMG_TRY(stream_alloc(device, s, &q, count * sizeof(T) + 16));
      ptrs.push_back(q);
    }
    *p = reinterpret_cast<T *>(q);
    return AMG_OK;
  }
  // exclusive scan of n values, its block sums in this object's memory
  amg_status scan(const int32_t *in, int32_t *out, int32_t n) {
    int32_t *bsum = nullptr;
    AMG_TRY(get(&bsum, (size_t)scan_blocks(n) + 1));
    scan_exclusive_i32_with(in, nullptr, out, n, bsum, s);
    return AMG_OK;
  }
};

// (by way of the pinned block)
amg_status read_i32(const amg_hierarchy *h, const int32_t *dev, int32_t *host) {
  int32_t *const pinned = reinterpret_cast<int32_t *>(h->scal_host);
  AMG_HIP(hipMemcpyAsync(pinned, dev, sizeof(int32_t), hipMemcpyDeviceToHost, h->stream));
  AMG_HIP(hipStreamSynchronize(h->stream));
  *host = *pinned;
  return AMG_OK;
}

amg_status map_err(int32_t flags) {
  if (flags & kErrArg) return AMG_ERR_ARG;
  if (flags & kErrSpd) return AMG_ERR_NOT_SPD;
  if (flags & kErrSym) return AMG_ERR_NOT_SYMMETRIC;
  return AMG_OK;
}

// A matrix of the current sweep: a level's (borrowed) or a temporary.
struct Mat {
  int32_t n = 0;
  int64_t most = 0;   // at least its number of entries
  double mean = 0.0;  // about the mean row's entries
  int32_t longest = 0;  // its longest row at most (0: not known)
  RowsOf rows{};
  const double *w = nullptr;
  const double *dg = nullptr;  // its diagonal
  const int32_t *size = nullptr;  // members of each row on the level (null: one each)
};

// One pairwise sweep on A (Section 3.2). nc == n means nothing was matched;
// else the outputs hold the coarse matrix and the maps.
struct SweepOut {
  Mat Ac;
  int32_t nc = 0;
  int32_t *agg = nullptr;   // fine -> coarse (n)
  double *p = nullptr;      // pairwise prolongator values (n)
  int32_t *lead = nullptr;  // coarse -> smallest member (nc)
  int32_t *mate = nullptr;  // n
  int32_t rounds = 0;
};

template <int G>
void launch_pref(const Mat &A, int32_t *pref, uint64_t *st, int32_t *ovf, int32_t *ctl,
                 int32_t *err, uint64_t *began, hipStream_t s) {
  k_pref<G><<<grid((int64_t)A.n * G), kBlock, 0, s>>>(A.n, A.rows, A.w, A.dg, pref, st, ovf,
                                                      ctl + kCtlPrefLong, began);
  if (A.longest == 0 || A.longest > 2 * G)
    k_pref_long<<<A.n < 2048 ? A.n : 2048, kBlock, 0, s>>>(A.rows, A.w, A.dg, pref, st, ovf,
                                                           ctl + kCtlPrefLong, err);
}

template <int G>
void launch_rap(int32_t nc, const RowsOf &A, const Coarsened &C, int32_t longest, int32_t *ovf,
                int32_t *ctl, int32_t *err, hipStream_t s) {
  k_rap<G><<<grid((int64_t)nc * G), kBlock, 0, s>>>(nc, A, C, ovf, ctl + kCtlRapLong);
  if (longest > 2 * G)
    k_rap_long<<<nc < 1024 ? nc : 1024, kBlock, 0, s>>>(A, C, ovf, ctl + kCtlRapLong, err);
}

// the host's copy of the control block and of the total scanned last
amg_status read_ctl(const int32_t *pinned, int32_t *host, hipStream_t s) {
  AMG_HIP(hipStreamSynchronize(s));
  for (int k = 0; k <= kCtl; ++k) host[k] = reinterpret_cast<const volatile int32_t *>(pinned)[k];
  return AMG_OK;
}

// (ctl: a zeroed control block; err: the setup's error word; when: the sweep's
// stamps, before: where the sweep before it takes its end from, may be null)
amg_status pairwise_sweep(amg_hierarchy *h, Tmp &tmp, const Mat &A, int32_t *ctl, int32_t *err,
                          Stamps *when, uint64_t *before, SweepOut &o) {
  hipStream_t s = h->stream;
  const int32_t n = A.n;
  const Report R{ctl, err, reinterpret_cast<int32_t *>(h->scal_host)};
  int32_t *pref, *id, *bsum, *ovf;
  uint64_t *st;
  AMG_TRY(tmp.get(&pref, A.most));
  AMG_TRY(tmp.get(&st, n));
  AMG_TRY(tmp.get(&id, n));
  AMG_TRY(tmp.get(&bsum, (size_t)scan_blocks(n) + 1));
  AMG_TRY(tmp.get(&ovf, n));
  AMG_TRY(tmp.get(&o.mate, n));
  // lanes per row: the mean row (of a sweep's matrix: of the one before it)
  // fills half of a group's places, so that most rows still fit
  if (A.mean <= 8.0) launch_pref<8>(A, pref, st, ovf, ctl, err, before, s);
  else if (A.mean <= 16.0) launch_pref<16>(A, pref, st, ovf, ctl, err, before, s);
  else if (A.mean <= 32.0) launch_pref<32>(A, pref, st, ovf, ctl, err, before, s);
  else launch_pref<64>(A, pref, st, ovf, ctl, err, before, s);
  // matching, and the numbering of what it gives; where it takes more than
  // the launches queued, both again from there on
  int32_t hc[kCtl + 1];
  for (int queue = 1;; queue = kMatchQueue) {
    for (int r = 0; r < queue; ++r) {
      int32_t *f = ctl + kCtlFlags + r * kMatchFlags;
      k_match<<<ceil_div(n, kMatchThreads), kMatchThreads, 0, s>>>(
          n, A.rows.b, A.rows.e, pref, st, r > 0 ? f - kMatchFlags : nullptr, f);
    }
    k_lead_scan<<<scan_blocks(n), kScanBlock, 0, s>>>(n, st, A.rows.b, A.rows.e, o.mate, id, bsum,
                                                      ctl, R);
    if (scan_blocks(n) > 1) k_scan_sums<<<1, kScanBlock, 0, s>>>(bsum, scan_blocks(n), R);
    AMG_HIP(hipGetLastError());
    AMG_TRY(read_ctl(R.to, hc, s));
    // a row too long for this sweep's product, or one that was for the sweep
    // before it (whose product left that row empty: nothing else here holds then)
    if (hc[kCtlErr]) return AMG_ERR_ARG;
    const int32_t *last = hc + kCtlFlags + (queue - 1) * kMatchFlags;
    if (!last[kLeft]) break;  // (the last launch does nothing once one before it left nothing)
    if (!last[kMoved]) return AMG_ERR_HIP;  // cannot happen on a symmetric matrix
    k_fill<int32_t><<<1, kCtl - kCtlEntries, 0, s>>>(ctl + kCtlEntries, 0, kCtl - kCtlEntries);
  }
  o.rounds = hc[kCtlRounds] > 0 ? hc[kCtlRounds] - 1 : 0;
  const int32_t nc = hc[kCtl], nnz = hc[kCtlEntries];
  o.nc = nc;
  if (nc == n) return AMG_OK;
  AMG_TRY(tmp.get(&o.agg, n));
  AMG_TRY(tmp.get(&o.lead, nc));
  AMG_TRY(tmp.get(&o.p, n));
  k_assign<<<grid(n), kBlock, 0, s>>>(n, o.mate, id, bsum, A.w, o.agg, o.lead, o.p,
                                      &when->assign);

  // Galerkin product and restricted w
  Coarsened C{};
  int32_t *off, *bsum2;
  AMG_TRY(tmp.get(&off, nc));
  AMG_TRY(tmp.get(&bsum2, (size_t)scan_blocks(nc) + 1));
  AMG_TRY(tmp.get(&C.b, nc));
  AMG_TRY(tmp.get(&C.e, nc));
  AMG_TRY(tmp.get(&C.ci, nnz));
  AMG_TRY(tmp.get(&C.val, nnz));
  AMG_TRY(tmp.get(&C.wc, nc));
  AMG_TRY(tmp.get(&C.dg, nc));
  AMG_TRY(tmp.get(&C.csize, nc));
  C.lead = o.lead;
  C.mate = o.mate;
  C.agg = o.agg;
  C.p = o.p;
  C.w = A.w;
  C.off = off;
  C.bsum = bsum2;
  C.size = A.size;
  k_terms_scan<<<scan_blocks(nc), kScanBlock, 0, s>>>(nc, o.lead, o.mate, A.rows.b, A.rows.e, off,
                                                      bsum2, &when->product);
  if (scan_blocks(nc) > 1)
    k_scan_sums<<<1, kScanBlock, 0, s>>>(bsum2, scan_blocks(nc), Report{});
  // lanes per coarse row: room for the mean row's terms and an eighth more (the
  // 7-point stencil's 14 terms take the 16 places of eight lanes)
  const double terms = 1.125 * nnz / nc;
  const int32_t longest = hc[kCtlLongest] > kRapLongCap ? 2 * kRapLongCap : 2 * hc[kCtlLongest];
  if (terms <= 16.0) launch_rap<8>(nc, A.rows, C, longest, ovf, ctl, err, s);
  else if (terms <= 32.0) launch_rap<16>(nc, A.rows, C, longest, ovf, ctl, err, s);
  else if (terms <= 64.0) launch_rap<32>(nc, A.rows, C, longest, ovf, ctl, err, s);
  else launch_rap<64>(nc, A.rows, C, longest, ovf, ctl, err, s);
  AMG_HIP(hipGetLastError());
  o.Ac.n = nc;
  o.Ac.most = nnz;
  o.Ac.mean = (double)nnz / n;
  o.Ac.longest = longest;
  o.Ac.rows = RowsOf{C.b, C.e, C.ci, C.val};
  o.Ac.w = C.wc;
  o.Ac.dg = C.dg;
  o.Ac.size = C.csize;
  return AMG_OK;
}

// the last sweep's matrix, packed into level storage
amg_status adopt_level(amg_hierarchy *h, Tmp &tmp, const Mat &M, const int32_t *ctl,
                       const int32_t *err, Level &L) {
  hipStream_t s = h->stream;
  const Report R{ctl, err, reinterpret_cast<int32_t *>(h->scal_host)};
  int32_t *bsum;
  AMG_TRY(tmp.get(&bsum, (size_t)scan_blocks(M.n) + 1));
  L.n = M.n;
  AMG_TRY(dalloc(h, &L.rp, (size_t)M.n + 1));
  scan_exclusive_i32_with(M.rows.b, M.rows.e, L.rp, M.n, bsum, s, R);
  int32_t hc[kCtl + 1];
  AMG_TRY(read_ctl(R.to, hc, s));
  if (hc[kCtlErr]) return AMG_ERR_ARG;  // a coarse row gathers more than kRapLongCap entries
  L.nnz = hc[kCtl];
  AMG_TRY(dalloc(h, &L.ci, (size_t)L.nnz));
  AMG_TRY(dalloc(h, &L.val, (size_t)L.nnz));
  AMG_TRY(dalloc(h, &L.w, (size_t)M.n));
  k_pack<<<grid((int64_t)M.n * 8), kBlock, 0, s>>>(M.n, M.rows, M.w, L.rp, L.ci, L.val, L.w);
  return AMG_OK;
}

}  // namespace

amg_status setup_tmp_alloc(amg_hierarchy *h, void **p, size_t bytes) {
  if (h->setup_arena) return static_cast<Arena *>(h->setup_arena)->get(p, bytes);
  return stream_alloc(h->device, h->stream, p, bytes);
}

void setup_tmp_free(amg_hierarchy *h, void *p) {
  if (!h->setup_arena) stream_free(h->device, h->stream, {p});
}

amg_status setup_scan(amg_hierarchy *h, const int32_t *in, int32_t *out, int32_t n) {
  int32_t *bsum = nullptr;
  AMG_TRY(setup_tmp_alloc(h, reinterpret_cast<void **>(&bsum),
                          sizeof(int32_t) * ((size_t)scan_blocks(n) + 1)));
  scan_exclusive_i32_with(in, nullptr, out, n, bsum, h->stream);
  setup_tmp_free(h, bsum);
  return AMG_OK;
}

size_t scan_sums(int32_t n) { return (size_t)scan_blocks(n) + 1; }

void scan_exclusive_i32(const int32_t *in, int32_t *out, int32_t n, int32_t *bsum,
                        hipStream_t s) {
  scan_exclusive_i32_with(in, nullptr, out, n, bsum, s);
}

// Cholesky by panels (k_chol_panel, k_chol_update)
amg_status cholesky_panels(const amg_hierarchy *h, Tmp &tmp, int32_t n, double *D, int32_t *err) {
  hipStream_t s = h->stream;
  double *diag;
  AMG_TRY(tmp.get(&diag, (size_t)ceil_div(n, kPanel) * kPanel * kPanel));
  for (int32_t k0 = 0; k0 < n; k0 += kPanel) {
    const int32_t c0 = k0 + kPanel, rest = n - c0;
    k_chol_panel<<<grid(rest), kBlock, 0, s>>>(n, k0, D, diag, err);
    if (rest <= 0) break;
    const unsigned t = (unsigned)ceil_div(rest, kCholTile);
    k_chol_update<<<dim3(t, t), kBlock, 0, s>>>(n, c0, D);
  }
  k_chol_finish<<<grid((int64_t)n * n), kBlock, 0, s>>>(n, diag, D);
  return AMG_OK;
}

amg_status build_hierarchy(amg_hierarchy *h, const amg_csr *A) {
  hipStream_t s = h->stream;
  const amg_params &P = h->params;
  const int32_t n0 = (int32_t)A->n;
  double T[8] = {0};
  double t_start = now_ms();
  // every temporary of this setup comes from one arena (declared before the
  // Tmp objects, so it outlives them), detached again on every way out
  Arena arena(h, A->n, A->nnz);
  struct Attach {
    amg_hierarchy *h;
    ~Attach() { h->setup_arena = nullptr; }
  } attach{h};
  h->setup_arena = &arena;
  Tmp tmp(h);
  // pinned: the scalars of a solve later, small results of the setup's kernels
  // now, and behind them the sweeps' stamps
  const size_t stamps = sizeof(Stamps) * (size_t)P.max_levels * P.sweeps;
  static_assert(2 * sizeof(PcgScal) % alignof(Stamps) == 0, "stamps behind the scalars");
  if (!h->scal_host)
    AMG_HIP(hipHostMalloc(reinterpret_cast<void **>(&h->scal_host), 2 * sizeof(PcgScal) + stamps));
  Stamps *const when = reinterpret_cast<Stamps *>(h->scal_host + 2);
  std::memset(when, 0, stamps);
  static_assert(sizeof(PcgScal) >= sizeof(int32_t) * (kCtl + 1), "control block and total");
  int32_t ran = 0;

  // validation
  int32_t *err;  // kErr*, one word for the whole setup: read, and 0, after each stage
  AMG_TRY(tmp.get(&err, 1));
  k_fill<int32_t><<<1, 1, 0, s>>>(err, 0, 1);
  if (!(P.flags & AMG_FLAG_SKIP_CHECKS))
    k_validate<<<grid((int64_t)n0 * 8), kBlock, 0, s>>>(n0, A->nnz, A->row_ptr, A->col, A->val, err);
  if (P.w) k_check_w<<<grid(n0), kBlock, 0, s>>>(n0, P.w, err);
  int32_t herr = 0;
  AMG_TRY(read_i32(h, err, &herr));
  AMG_TRY(map_err(herr));
  T[0] = now_ms() - t_start;

  // level 0: a copy of A and w
  h->lv.clear();
  h->lv.emplace_back();
  {
    Level &L0 = h->lv[0];
    L0.n = n0;
    L0.nnz = A->nnz;
    AMG_TRY(dalloc(h, &L0.rp, (size_t)n0 + 1));
    AMG_TRY(dalloc(h, &L0.ci, (size_t)A->nnz));
    AMG_TRY(dalloc(h, &L0.val, (size_t)A->nnz));
    AMG_TRY(dalloc(h, &L0.w, (size_t)n0));
    AMG_HIP(hipMemcpyAsync(L0.rp, A->row_ptr, sizeof(int32_t) * (n0 + 1),
                           hipMemcpyDeviceToDevice, s));
    AMG_HIP(hipMemcpyAsync(L0.ci, A->col, sizeof(int32_t) * A->nnz, hipMemcpyDeviceToDevice, s));
    AMG_HIP(hipMemcpyAsync(L0.val, A->val, sizeof(double) * A->nnz, hipMemcpyDeviceToDevice, s));
    if (P.w)
      AMG_HIP(hipMemcpyAsync(L0.w, P.w, sizeof(double) * n0, hipMemcpyDeviceToDevice, s));
    else
      k_fill<double><<<grid(n0), kBlock, 0, s>>>(L0.w, 1.0, n0);
    // algebraically smooth w: w_sweeps l1-Jacobi sweeps on A w = 0 from the
    // sample; the result must still have no zero entry
    if (P.w_sweeps > 0) {
      double *m, *minv, *w2;
      AMG_TRY(tmp.get(&m, n0));
      AMG_TRY(tmp.get(&minv, n0));
      AMG_TRY(tmp.get(&w2, n0));
      k_l1_diag<<<grid(n0), kBlock, 0, s>>>(n0, L0.rp, L0.ci, L0.val, m, minv);
      double *src = L0.w, *dst = w2;
      for (int32_t k = 0; k < P.w_sweeps; ++k) {
        k_smooth_w<<<grid(n0), kBlock, 0, s>>>(n0, L0.rp, L0.ci, L0.val, m, src, dst);
        std::swap(src, dst);
      }
      if (src != L0.w)
        AMG_HIP(hipMemcpyAsync(L0.w, src, sizeof(double) * n0, hipMemcpyDeviceToDevice, s));
      k_fill<int32_t><<<1, 1, 0, s>>>(err, 0, 1);
      k_check_w<<<grid(n0), kBlock, 0, s>>>(n0, L0.w, err);
      AMG_TRY(read_i32(h, err, &herr));
      AMG_TRY(map_err(herr));
    }
  }

  double t_sweeps = 0, t_smooth = 0, t_compose = 0;
  std::vector<int32_t> last_of_level;  // sweeps whose product the host waits for as composition
  // control blocks of the sweeps to come, zeroed a level's worth or more at a time
  constexpr int kCtlBlocks = 32;
  static_assert(kCtlBlocks >= kMaxSweeps, "a level's sweeps");
  int32_t *ctls = nullptr;
  int ctl_left = 0;
  const double *dg = nullptr;  // the level's diagonal, where the sweep before left it
  int32_t longest = 0;
  for (int32_t l = 0;; ++l) {
    const int32_t n = h->lv[l].n;
    if (n <= P.max_coarse || l == P.max_levels - 1) break;
    const Level &A0 = h->lv[l];
    if (ctl_left < P.sweeps) {
      AMG_TRY(tmp.get(&ctls, kCtlBlocks * kCtl));
      k_fill<int32_t><<<grid(kCtlBlocks * kCtl), kBlock, 0, s>>>(ctls, 0, kCtlBlocks * kCtl);
      ctl_left = kCtlBlocks;
    }
    const RowsOf rows{A0.rp, A0.rp + 1, A0.ci, A0.val};
    if (!dg) {
      double *d;
      AMG_TRY(tmp.get(&d, n));
      k_diag<<<grid(n), kBlock, 0, s>>>(n, rows, d);
      dg = d;
    }
    Mat cur;
    cur.n = n;
    cur.most = A0.nnz;
    cur.mean = (double)A0.nnz / n;
    cur.longest = longest;
    cur.rows = rows;
    cur.w = A0.w;
    cur.dg = dg;
    int32_t done = 0, rounds = 0;
    SweepMaps maps{};
    const int32_t *last_ctl = nullptr;
    for (int32_t k = 0; k < P.sweeps; ++k) {
      SweepOut o;
      const double t0 = now_ms();
      AMG_TRY(pairwise_sweep(h, tmp, cur, ctls, err, when + ran,
                             k > 0 ? &when[ran - 1].end : nullptr, o));
      t_sweeps += now_ms() - t0;
      ++ran;
      last_ctl = ctls;
      ctls += kCtl;
      --ctl_left;
      rounds += o.rounds;
      if (o.nc == cur.n) break;  // nothing matched: end this level's sweeps
      maps.agg[k] = o.agg;
      maps.p[k] = o.p;
      maps.lead[k] = o.lead;
      maps.mate[k] = o.mate;
      cur = o.Ac;
      ++done;
    }
    if (done == 0) break;  // level l does not coarsen: it is the coarsest
    double tc = now_ms();
    Level &F = h->lv[l];
    F.sweeps = done;
    F.rounds = rounds;
    AMG_TRY(dalloc(h, &F.agg, (size_t)n));
    AMG_TRY(dalloc(h, &F.p64, (size_t)n));
    AMG_TRY(dalloc(h, &F.mptr, (size_t)cur.n + 1));
    AMG_TRY(dalloc(h, &F.mem, (size_t)n));
    const bool all = done == P.sweeps;  // (else one more sweep began after the last product)
    if (all) last_of_level.push_back(ran - 1);
    k_compose<<<grid(n), kBlock, 0, s>>>(n, done, maps, F.agg, F.p64,
                                         all ? &when[ran - 1].end : nullptr);
    AMG_TRY(tmp.scan(cur.size, F.mptr, cur.n));
    k_members<<<grid(cur.n), kBlock, 0, s>>>(cur.n, done, maps, F.mptr, F.mem);
    Level Cn;
    if (P.smooth_p) {
      // the tentative product chose the aggregates and restricted w; the
      // next level is the Galerkin product with the smoothed prolongator
      int32_t herr = 0;
      AMG_TRY(read_i32(h, err, &herr));
      if (herr) return AMG_ERR_ARG;
      const double tr = now_ms();
      Cn.n = cur.n;
      const amg_status st =
          smooth_level(h, F, cur.n, F.agg, F.p64, &Cn.rp, &Cn.ci, &Cn.val, &Cn.nnz);
      // a row over every limit: too wide a coarsest level if it was to be the last
      if (st == AMG_ERR_ARG && l + 1 == P.max_levels - 1 && cur.n > AMG_MAX_DENSE)
        return AMG_ERR_STALL;
      AMG_TRY(st);
      AMG_TRY(dalloc(h, &Cn.w, (size_t)cur.n));
      AMG_HIP(hipMemcpyAsync(Cn.w, cur.w, sizeof(double) * cur.n, hipMemcpyDeviceToDevice, s));
      tc += now_ms() - tr;  // counted as Galerkin time, not composition
      t_smooth += now_ms() - tr;
      dg = nullptr;
      longest = 0;
    } else {
      AMG_TRY(adopt_level(h, tmp, cur, last_ctl, err, Cn));
      dg = cur.dg;
      longest = cur.longest;
    }
    h->lv.push_back(Cn);
    t_compose += now_ms() - tc;
  }

  // smoother diagonals
  double ts = now_ms();
  const int32_t nlev = (int32_t)h->lv.size();
  // (the coarsest level too when its system is solved by CG with them)
  const int32_t nsmooth = h->params.coarse_solver == AMG_COARSE_PCG ? nlev : nlev - 1;
  for (int32_t l = 0; l < nsmooth; ++l) {
    Level &L = h->lv[l];
    AMG_TRY(dalloc(h, &L.m, (size_t)L.n));
    AMG_TRY(dalloc(h, &L.minv64, (size_t)L.n));
    k_l1_diag<<<grid(L.n), kBlock, 0, s>>>(L.n, L.rp, L.ci, L.val, L.m, L.minv64);
  }
  // coarsest: dense Cholesky and the inverse factor
  {
    Level &L = h->lv[nlev - 1];
    const int32_t nL = L.n;
    if (nL > AMG_MAX_DENSE) return AMG_ERR_STALL;
    double *D;
    AMG_TRY(tmp.get(&D, (size_t)nL * nL));
    AMG_HIP(hipMemsetAsync(D, 0, sizeof(double) * (size_t)nL * nL, s));
    k_dense_scatter<<<grid(nL), kBlock, 0, s>>>(nL, L.rp, L.ci, L.val, D);
    k_fill<int32_t><<<1, 1, 0, s>>>(err, 0, 1);
    const size_t chol_lds = sizeof(double) * ((size_t)nL * (nL + 1) / 2 + nL);
    if (nL <= kCholLdsMax && chol_lds > 65536)
      AMG_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(k_cholesky_lds),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)chol_lds));
    if (nL <= kCholLdsMax)
      k_cholesky_lds<<<1, 1024, chol_lds, s>>>(nL, D, err);
    else
      AMG_TRY(cholesky_panels(h, tmp, nL, D, err));
    AMG_HIP(hipGetLastError());
    AMG_TRY(read_i32(h, err, &herr));
    if (herr) return AMG_ERR_NOT_SPD;
    h->C.n = nL;
    AMG_TRY(dalloc(h, &h->C.Linv, (size_t)nL * nL));
    AMG_TRY(dalloc(h, &h->C.Ainv, (size_t)nL * nL));
    const size_t tri_lds = 2 * sizeof(double) * (size_t)nL;  // <= 64 KB (nL <= AMG_MAX_DENSE)
    if (nL <= kTriThreads)
      k_tri_inverse<1><<<nL, kTriThreads, tri_lds, s>>>(nL, D, h->C.Linv);
    else if (nL <= 4 * kTriThreads)
      k_tri_inverse<4><<<nL, kTriThreads, tri_lds, s>>>(nL, D, h->C.Linv);
    else
      k_tri_inverse<AMG_MAX_DENSE / kTriThreads><<<nL, kTriThreads, tri_lds, s>>>(nL, D,
                                                                                  h->C.Linv);
    k_inverse_from_factor<<<grid((int64_t)nL * nL), kBlock, 0, s>>>(nL, h->C.Linv, h->C.Ainv);
    AMG_HIP(hipStreamSynchronize(s));
  }
  T[5] = now_ms() - ts;
  double tf = now_ms();
  AMG_TRY(build_solve_formats(h));
  AMG_HIP(hipStreamSynchronize(s));
  T[6] = now_ms() - tf;
  // numbering and Galerkin product as the device saw them; what is left of the
  // host's time in the sweeps is the matching's
  int khz = 0;
  AMG_HIP(hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, h->device));
  const auto ms = [&](uint64_t from, uint64_t to) {
    return khz > 0 && from && to > from ? (double)(to - from) / khz : 0.0;
  };
  for (int32_t k = 0; k < ran; ++k) {
    T[2] += ms(when[k].assign, when[k].product);
    T[3] += ms(when[k].product, when[k].end);
  }
  double waited = 0;
  for (int32_t k : last_of_level) waited += ms(when[k].product, when[k].end);
  T[1] = std::max(0.0, t_sweeps - T[2] - (T[3] - waited));
  T[4] = std::max(0.0, t_compose - waited);
  T[3] += t_smooth;
  T[7] = now_ms() - t_start;
  for (int k = 0; k < 8; ++k) h->setup_ms[k] = T[k];
  return AMG_OK;
}

}  // namespace amg
