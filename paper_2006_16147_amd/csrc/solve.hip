// Solve phase: the V-cycle of eq. (amg) with l1-Jacobi smoothing (Section 3.3)
// inside preconditioned CG (Section 5), on one gfx950 GPU.
//
// Layout. Every level is stored in an aggregate-major order (the unknowns of
// an aggregate of P_l are one contiguous segment, segments ordered like the
// coarse unknowns, recursively from the coarsest level), as sliced ELLPACK
// with 64-row slices (one slice per wavefront, column-major inside a slice),
// so lane i of a wavefront loads row i's k-th value and column index from
// consecutive addresses. The matrix arrays are loaded with a nontemporal
// hint: they stream once per SpMV while the gathered vector stays in L2.
//
// Kernels of a V-cycle (zero initial guess), per level l < L:
//   down  pre_restrict : z = M^-1 r ; r_{l+1} = P^T (r - A z)
//         (A M^-1 is stored, so one vector is gathered; a block owns whole
//          aggregates and sums their members in LDS: the residual never
//          goes to HBM)
//   up    post_prolong : y = z + M^-1 (r - A z) on level l + 1, and at once
//         z_l += P y for the segments of the block's coarse rows
//   level L: coarse_prolong: z_L = A_L^-1 r_L and z_{L-1} += P z_L
//   level 0: post with the (r, z) partial sums for CG
//
// CG scalars live on the device; reductions are two-stage and deterministic:
// every block writes its partial sums, a one-block finalize kernel adds them
// in block order and updates the scalars. Kernels test a device flag and
// return at once after convergence, so the host queues several iterations
// (captured in a hipGraph) between checks.

#include <chrono>
#include <cmath>

#include <hip/hip_ext.h>

#include "internal.h"

namespace amg {

namespace {

double now_ms() {
  return std::chrono::duration<double, std::milli>(
             std::chrono::steady_clock::now().time_since_epoch())
      .count();
}

inline int32_t grid1(int64_t n) { return ceil_div(n > 0 ? n : 1, kBlock); }

// ---------------------------------------------------------------------------
// launch geometry of the row-streaming kernels: each block a contiguous
// chunk of 1 to kMaxRowsPerThread rows per thread, about kTargetBlocks
// blocks (more rows per thread only beyond kMaxParts blocks)
// ---------------------------------------------------------------------------

struct Geom {
  int32_t grid;
  int32_t chunk;  // rows per block, a multiple of kBlock
};

Geom geom(int64_t n) {
  int64_t rows = (n + (int64_t)kBlock * kTargetBlocks - 1) / ((int64_t)kBlock * kTargetBlocks);
  rows = rows < 1 || n >= kManyRows ? 1 : (rows > kMaxRowsPerThread ? kMaxRowsPerThread : rows);
  int64_t chunk = kBlock * rows;
  int64_t blocks = (n + chunk - 1) / chunk;
  if (blocks < 1) blocks = 1;
  if (blocks > kMaxParts) {
    chunk = ((n + kMaxParts - 1) / kMaxParts + kBlock - 1) / kBlock * kBlock;
    blocks = (n + chunk - 1) / chunk;
  }
  return {(int32_t)blocks, (int32_t)chunk};
}

__device__ __forceinline__ void rows_of_block(int32_t n, int32_t chunk, int32_t *b, int32_t *e) {
  const int64_t bb = (int64_t)blockIdx.x * chunk;
  *b = (int32_t)bb;
  *e = (int32_t)(bb + chunk < n ? bb + chunk : n);
}

__device__ __forceinline__ void sell_row(const int32_t *sptr, int32_t row, int32_t *base,
                                         int32_t *w) {
  const int32_t s = row / kSlice;
  const int32_t b0 = sptr[s];
  *base = b0 + (row % kSlice);
  *w = (sptr[s + 1] - b0) / kSlice;
}

// zf[k] += pp[k] * y(aggp[k]) for k = k0 + t, k0 + t + nth, ... < k1: each
// thread issues the loads of four of its positions before their use.
template <typename TV, typename Y>
__device__ __forceinline__ void prolong_add(int32_t k0, int32_t k1, int32_t t, int32_t nth,
                                            const int32_t *__restrict__ aggp,
                                            const TV *__restrict__ pp, TV *__restrict__ zf, Y y) {
  for (int32_t kb = k0 + t; kb < k1; kb += 4 * nth) {
    int32_t a[4];
    TV pv[4], zv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int32_t k = kb + u * nth;
      a[u] = 0;
      pv[u] = zv[u] = 0;
      if (k < k1) {
        a[u] = aggp[k];
        pv[u] = pp[k];
        zv[u] = zf[k];
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int32_t k = kb + u * nth;
      if (k < k1) zf[k] = zv[u] + pv[u] * y(a[u]);
    }
  }
}

// ---------------------------------------------------------------------------
// deterministic two-stage reductions (no in-kernel cross-block handshake: on
// gfx950 a device-scope fence per block writes back the XCD's L2 and costs
// more than the extra launch)
// ---------------------------------------------------------------------------

template <int NV>
__device__ void block_partial(double (&v)[NV], double *partials) {
  __shared__ double sh[NV][kBlock / kWave];
  const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    double x = v[q];
    for (int o = kWave / 2; o > 0; o >>= 1) x += __shfl_down(x, o, kWave);
    if (lane == 0) sh[q][wid] = x;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      double t = sh[q][0];
      for (int k = 1; k < kBlock / kWave; ++k) t += sh[q][k];
      partials[(int64_t)q * kMaxParts + blockIdx.x] = t;
    }
  }
}

// planes of the partials that a folded iteration's dot products use: each is
// still read while the next is written
constexpr int kRZPlane = 0, kPQPlane = 1, kRRPlane = 2;
static_assert(kRRPlane < kPartPlanes, "planes");

enum FinOp : int32_t {
  kFinInit = 0,  // (b, b), (r, r) of the initial residual
  kFinPQ = 1,    // CG: (p, q), alpha = rho / (p, q)
  kFinRR = 2,    // (r, r), stop test
  kFinRZ = 3,    // CG: (r, z), beta
  kFinTrue = 4,  // true residual
  kFinPQR = 5,   // flexible CG: (p, q), (p, r), alpha = (p, r) / (p, q)
  kFinZQ = 6     // flexible CG: beta = -(z, q) / (p, q)
};

__device__ __forceinline__ bool converged(double rr, double bb, double rtol) {
  return sqrt(rr) <= rtol * sqrt(bb);
}

// Sums nparts partials of one or two quantities in a fixed order and applies
// the CG scalar update of `op`.
__global__ void __launch_bounds__(1024) k_finalize(int32_t op, int32_t nparts,
                                                   const double *__restrict__ partials,
                                                   PcgScal *scal, const int32_t *done) {
  // the stop flag and the scalars are loaded with the partials, not before
  const int32_t stop = done ? *done : 0;
  PcgScal sc;
  if (threadIdx.x == 0) sc = *scal;
  __shared__ double sh[2][1024 / kWave];
  const int nv = op == kFinInit || op == kFinPQR ? 2 : 1;
  const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
  for (int q = 0; q < nv; ++q) {
    // this thread's partials in index order, sixteen loads at a time
    const double *src = partials + (int64_t)q * kMaxParts;
    double a = 0.0;
    for (int32_t b0 = threadIdx.x; b0 < nparts; b0 += 16 * blockDim.x) {
      double v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int32_t b = b0 + u * (int32_t)blockDim.x;
        v[u] = b < nparts ? src[b] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < 16; ++u)
        if (b0 + u * (int32_t)blockDim.x < nparts) a += v[u];
    }
    for (int o = kWave / 2; o > 0; o >>= 1) a += __shfl_down(a, o, kWave);
    if (lane == 0) sh[q][wid] = a;
  }
  __syncthreads();
  if (threadIdx.x != 0 || stop) return;
  double tot[2] = {0.0, 0.0};
  for (int q = 0; q < nv; ++q) {
    double t = sh[q][0];
    for (int k = 1; k < (int)(blockDim.x / kWave); ++k) t += sh[q][k];
    tot[q] = t;
  }
  switch (op) {
    case kFinInit: {
      const double rtol = sc.rtol;
      scal->bb = tot[0];
      scal->rr = tot[1];
      scal->tol2 = rtol * rtol * tot[0];
      if (tot[0] == 0.0) scal->done = 4;
      else if (converged(tot[1], tot[0], rtol)) scal->done = 1;
      else if (sc.maxit <= 0) scal->done = 2;
      break;
    }
    case kFinPQ:
      scal->pq = tot[0];
      if (!(tot[0] > 0.0)) scal->done = 3;
      else scal->alpha = sc.rho / tot[0];
      break;
    case kFinRR:
      scal->rr = tot[0];
      scal->iter = sc.iter + 1;
      if (converged(tot[0], sc.bb, sc.rtol)) scal->done = 1;
      else if (sc.iter + 1 >= sc.maxit) scal->done = 2;
      break;
    case kFinRZ:
      if (!(tot[0] > 0.0)) {
        scal->done = 3;
      } else if (sc.phase == 0) {
        scal->rho = tot[0];
        scal->phase = 1;
      } else {
        scal->beta = tot[0] / sc.rho;
        scal->rho = tot[0];
      }
      break;
    case kFinPQR:
      scal->pq = tot[0];
      if (!(tot[0] > 0.0)) scal->done = 3;
      else scal->alpha = tot[1] / tot[0];
      break;
    case kFinZQ:
      scal->beta = -tot[0] / sc.pq;
      break;
    default:
      scal->rr_true = tot[0];
      break;
  }
}

// The sum of nparts partials by a block of kBlock threads, every one of which
// gets it: k_finalize's sum in its order, thread t adding up what the threads
// t, t + kBlock, ... of its 1024 would. *stopped: whether *done was set, one
// look for the whole block. Block 0 of the same launch may be setting it, and
// waves that looked for themselves could part ways in a block that starts late:
// those that go on would add up slots of the sum that nobody has written.
__device__ __forceinline__ double sum_partials(const double *__restrict__ src, int32_t nparts,
                                               const int32_t *done, bool *stopped) {
  constexpr int kRuns = 1024 / kBlock, kWaves = kBlock / kWave;
  __shared__ double wsum[kRuns * kWaves];
  __shared__ int32_t seen;
  if (threadIdx.x == 0) seen = *done;
  const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
#pragma unroll
  for (int k = 0; k < kRuns; ++k) {
    double a = 0.0;
    for (int32_t b0 = threadIdx.x + k * kBlock; b0 < nparts; b0 += 4 * 1024) {
      double v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = b0 + u * 1024 < nparts ? src[b0 + u * 1024] : 0.0;
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (b0 + u * 1024 < nparts) a += v[u];
    }
    if (k * kBlock < nparts)
      for (int o = kWave / 2; o > 0; o >>= 1) a += __shfl_down(a, o, kWave);
    if (lane == 0) wsum[k * kWaves + wid] = a;
  }
  __syncthreads();
  *stopped = seen != 0;
  double t = wsum[0];
  for (int k = 1; k < kRuns * kWaves; ++k) t += wsum[k];
  return t;
}

// (r, r) and the stop test, by the level-0 down step of a folded iteration:
// true if the solve goes on. Only block 0 writes, and nothing that a block
// still starting reads but the flag, which then says what it would find (and
// is read once per block, see sum_partials).
struct FinRR {
  PcgScal *scal;
  const double *partials;
  int32_t nparts;
};
__device__ __forceinline__ bool stop_test(const FinRR &F) {
  const int32_t iter = F.scal->iter1, maxit = F.scal->maxit;
  const double bb = F.scal->bb, rtol = F.scal->rtol;
  bool stopped;
  const double rr = sum_partials(F.partials, F.nparts, &F.scal->done, &stopped);
  if (stopped) return false;
  const int32_t done = converged(rr, bb, rtol) ? 1 : (iter >= maxit ? 2 : 0);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    F.scal->rr = rr;
    F.scal->iter = iter;
    if (done) F.scal->done = done;
  }
  return done == 0;
}

// ---------------------------------------------------------------------------
// aggregate-major order, SELL construction, precision demotion
// ---------------------------------------------------------------------------

// number of members of the aggregate at each coarse position
__global__ void k_seg_count(int32_t nc, const int32_t *perm_c, const int32_t *mptr,
                            int32_t *cnt) {
  const int32_t J = blockIdx.x * blockDim.x + threadIdx.x;
  if (J >= nc) return;
  const int32_t I = perm_c[J];
  cnt[J] = mptr[I + 1] - mptr[I];
}

// positions of the members of each aggregate (in ascending original index)
__global__ void k_order_fill(int32_t nc, const int32_t *perm_c, const int32_t *mptr,
                             const int32_t *mem, const int32_t *seg, const double *p,
                             int32_t *perm, int32_t *iperm, int32_t *aggp, double *pp) {
  const int32_t J = blockIdx.x * blockDim.x + threadIdx.x;
  if (J >= nc) return;
  const int32_t I = perm_c[J];
  const int32_t b = mptr[I], e = mptr[I + 1], k0 = seg[J];
  for (int32_t m = b; m < e; ++m) {
    const int32_t i = mem[m], k = k0 + (m - b);
    perm[k] = i;
    iperm[i] = k;
    aggp[k] = J;
    pp[k] = p[i];
  }
}

__global__ void k_iota_i32(int32_t *a, int32_t n) {
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) a[i] = i;
}

// Entries of each 64-row slice (width = longest row, times 64), a wave per
// slice; stat[0]: their 64-bit total (the int32 offsets of the format must not
// overflow), stat[1]: the widest slice.
__global__ void __launch_bounds__(1024) k_sell_width(int32_t n, int32_t ns,
                                                     const int32_t *__restrict__ rp,
                                                     const int32_t *__restrict__ perm,
                                                     int32_t *__restrict__ w64,
                                                     unsigned long long *stat) {
  __shared__ unsigned long long total, widest;
  if (threadIdx.x == 0) total = widest = 0;
  __syncthreads();
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int32_t s = (int32_t)(k / kSlice);
  int32_t w = 0;
  if (k < n) {
    const int32_t i = perm[k];
    w = rp[i + 1] - rp[i];
  }
  for (int o = kWave / 2; o > 0; o >>= 1) w = max(w, __shfl_xor(w, o, kWave));
  if (s < ns && threadIdx.x % kWave == 0) {
    const int64_t e = (int64_t)w * kSlice;
    w64[s] = e > INT32_MAX ? INT32_MAX : (int32_t)e;
    atomicAdd(&total, (unsigned long long)e);
    atomicMax(&widest, (unsigned long long)w);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    atomicAdd(&stat[0], total);
    atomicMax(&stat[1], widest);
  }
}

// What k_sell_fill writes: the SELL arrays (null: not wanted), and by position
// the diagonal scaling and the prolongator's FP32 copy.
struct SellOut {
  int32_t *col;
  double *v64;
  float *v32;
  double *s64;
  float *s32;
  double *minv64;
  float *minv32;
  const double *pp64;
  float *pp32;
};

// Row k of the permuted matrix is original row perm[k] with columns renumbered
// by iperm and sorted (rows up to kSortCap entries); padding entries point at
// the row itself with value 0. A block per slice, four lanes per row (and
// gridDim.y blocks over the entries of long rows): an entry's place is its rank
// among the row's columns, held in LDS with consecutive rows in consecutive
// banks. (A thread per row with an insertion sort of indices in scratch, every
// comparison two dependent loads, took 0.79 ms at 160^3, and 0.9 ms for 1019
// rows of 428 entries.)
constexpr int kSortCap = 64;
__global__ void __launch_bounds__(kBlock) k_sell_fill(
    int32_t n, const int32_t *__restrict__ rp, const int32_t *__restrict__ ci,
    const double *__restrict__ val, const int32_t *__restrict__ perm,
    const int32_t *__restrict__ iperm, const double *__restrict__ minv,
    const int32_t *__restrict__ sptr, SellOut O) {
  __shared__ int32_t key[kSortCap][kSlice];
  constexpr int kParts = kBlock / kSlice;
  const int32_t s = blockIdx.x, row = threadIdx.x % kSlice, part = threadIdx.x / kSlice;
  const int64_t k = (int64_t)s * kSlice + row;
  const int32_t base = sptr[s], w = (sptr[s + 1] - base) / kSlice;
  const int32_t i = k < n ? perm[k] : 0;
  const int32_t b = k < n ? rp[i] : 0, len = k < n ? rp[i + 1] - b : 0;
  const bool sorted = len <= kSortCap;
  if (sorted)
    for (int32_t e = part; e < len; e += kParts) key[e][row] = iperm[ci[b + e]];
  __syncthreads();
  for (int32_t e = part + kParts * (int32_t)blockIdx.y; e < w; e += kParts * (int32_t)gridDim.y) {
    int32_t at = e, J = k < n ? (int32_t)k : 0;
    double a = 0.0, m = 0.0;
    if (e < len) {
      const int32_t c = ci[b + e];
      a = val[b + e];
      if (O.s64 || O.s32) m = minv[c];
      if (sorted) {
        J = key[e][row];
        at = 0;
        for (int32_t f = 0; f < len; ++f)
          at += key[f][row] < J || (key[f][row] == J && f < e) ? 1 : 0;
      } else {
        J = iperm[c];
      }
    }
    const int64_t idx = base + (int64_t)at * kSlice + row;
    O.col[idx] = J;
    if (O.v64) O.v64[idx] = a;
    if (O.v32) O.v32[idx] = (float)a;
    if (O.s64) O.s64[idx] = a * m;
    if (O.s32) O.s32[idx] = (float)(a * m);
  }
  if (blockIdx.y == 0 && part == 0 && k < n && O.minv64) {
    const double m = minv[i];
    O.minv64[k] = m;
    if (O.minv32) O.minv32[k] = (float)m;
    if (O.pp32) O.pp32[k] = (float)O.pp64[k];
  }
}

// flags a value that an FP32 number cannot hold exactly (or a NaN)
__global__ void k_not_fp32_exact(int64_t n, const double *a, int32_t *flag) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n && !((double)(float)a[i] == a[i])) *flag = 1;
}

__global__ void k_permute_in(int32_t n, const int32_t *__restrict__ perm,
                             const double *__restrict__ src, double *__restrict__ dst) {
  const int32_t k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) dst[k] = src[perm[k]];
}

__global__ void k_permute_out(int32_t n, const int32_t *__restrict__ perm,
                              const double *__restrict__ src, double *__restrict__ dst) {
  const int32_t k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) dst[perm[k]] = src[k];
}

// ---------------------------------------------------------------------------
// V-cycle kernels. TV: hierarchy precision; TR: type of the level's
// right-hand side (double on level 0, TV below); TO: type of its output.
// ---------------------------------------------------------------------------

// Down step on level l for the coarse positions [J0, J0 + G) of this block:
// z = M^-1 r with the residual through the stored A M^-1 (kPreScaled) or,
// after extra pre-smoothing sweeps, the given z (kPreFromZ, plain A stored
// as TA), or z = M^-1 r formed while staging r in LDS and the residual
// through the plain A (kPreStagedZ, LDS kernel only: where A is stored in
// fewer bytes than A M^-1, i.e. level 0's exact FP32 copy in an FP64
// hierarchy); then
// r_{l+1}(J) = sum over the segment of J, in order, of p_k (r - A z)_k.
// The block's fine rows are the union of its segments (at most R kBlock
// rows; thread t takes rows t, t + kBlock, ...).
enum PreMode : int { kPreScaled = 0, kPreFromZ = 1, kPreStagedZ = 2 };

// A K-cycle level's first flexible-CG step: its vectors and block partials of
// rho1 = (c1, v1) and (c1, b).
template <typename TV>
struct KSub {
  const TV *b, *v1;
  const double *partials;
  int32_t nparts;
  double *ks;
};

// s1 = (c1, b) / rho1, summed by every block in the same order (so all blocks
// hold the same s1); block 0 keeps both for the second step and the prolongation
template <typename TV>
__device__ __forceinline__ double first_step(const KSub<TV> &S) {
  __shared__ double sh[2][kBlock / kWave];
  const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
  for (int q = 0; q < 2; ++q) {
    const double *src = S.partials + (int64_t)q * kMaxParts;
    double a = 0.0;
    for (int32_t b0 = threadIdx.x; b0 < S.nparts; b0 += 16 * kBlock) {
      double v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int32_t bb = b0 + u * kBlock;
        v[u] = bb < S.nparts ? src[bb] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < 16; ++u)
        if (b0 + u * kBlock < S.nparts) a += v[u];
    }
    for (int o = kWave / 2; o > 0; o >>= 1) a += __shfl_down(a, o, kWave);
    if (lane == 0) sh[q][wid] = a;
  }
  __syncthreads();
  double rho1 = sh[0][0], cb = sh[1][0];
  for (int k = 1; k < kBlock / kWave; ++k) {
    rho1 += sh[0][k];
    cb += sh[1][k];
  }
  const double s1 = rho1 > 0.0 ? cb / rho1 : 0.0;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    S.ks[kRho1] = rho1;
    S.ks[kS1] = s1;
  }
  return s1;
}

template <typename TV, typename TR, int MODE, typename TA = TV, int R = 1, bool FIN = false>
__global__ void __launch_bounds__(kBlock) k_pre_restrict(
    int32_t nc, int32_t G, const int32_t *__restrict__ seg, const int32_t *__restrict__ sptr,
    const int32_t *__restrict__ col, const TA *__restrict__ val, const TV *__restrict__ minv,
    const TV *__restrict__ pp, const TR *__restrict__ r, TV *__restrict__ z,
    TV *__restrict__ rc, const int32_t *__restrict__ done, FinRR fin = FinRR{}) {
  __shared__ TV sh[kBlock * R];
  if (FIN ? !stop_test(fin) : *done != 0) return;
  const int32_t J0 = blockIdx.x * G;
  const int32_t J1 = min(nc, J0 + G);
  const int32_t f0 = seg[J0], f1 = seg[J1];
  // the thread's segment bounds for the sums after the barrier, loaded now
  const int32_t Jt = J0 + (int32_t)threadIdx.x;
  const int32_t sb = Jt < J1 ? seg[Jt] : 0, se = Jt < J1 ? seg[Jt + 1] : 0;
#pragma unroll
  for (int u = 0; u < R; ++u) {
    const int32_t row = f0 + (int32_t)threadIdx.x + u * kBlock;
    if (row < f1) {
      // the row's own operands first: their loads overlap the gathers
      const TV ri = (TV)r[row];
      const TV mi = MODE == kPreScaled ? minv[row] : TV(0);
      const TV pv = pp[row];
      int32_t base, w;
      sell_row(sptr, row, &base, &w);
      const TV acc =
          MODE == kPreFromZ
              ? sell_dot_t<TV, TA>(col, val, base, w, [&](int32_t c) { return z[c]; })
              : sell_dot_t<TV, TA>(col, val, base, w, [&](int32_t c) { return (TV)r[c]; });
      if (MODE == kPreScaled) z[row] = ri * mi;
      sh[threadIdx.x + u * kBlock] = pv * (ri - acc);
    }
  }
  __syncthreads();
  for (int32_t J = Jt; J < J1; J += kBlock) {
    const int32_t b = (J == Jt ? sb : seg[J]) - f0, e = (J == Jt ? se : seg[J + 1]) - f0;
    TV s = 0;
    for (int32_t m = b; m < e; ++m) s += sh[m];
    rc[J] = s;
  }
}

// k_pre_restrict (one sweep, A M^-1, one row per thread) of r1 = b - s1 v1, which is formed at
// each entry that is gathered and stored in r1 for the kernels that follow:
// k_kresid and its launch less in the second step of a K-cycle level
template <typename TV>
__global__ void __launch_bounds__(kBlock) k_kdown(
    int32_t nc, int32_t G, const int32_t *__restrict__ seg, const int32_t *__restrict__ sptr,
    const int32_t *__restrict__ col, const TV *__restrict__ val, const TV *__restrict__ minv,
    const TV *__restrict__ pp, KSub<TV> sub, TV *__restrict__ r1, TV *__restrict__ z,
    TV *__restrict__ rc, const int32_t *__restrict__ done) {
  __shared__ TV sh[kBlock];
  if (*done) return;
  const TV *__restrict__ b = sub.b, *__restrict__ v1 = sub.v1;
  const int32_t J0 = blockIdx.x * G;
  const int32_t J1 = min(nc, J0 + G);
  const int32_t f0 = seg[J0], f1 = seg[J1];
  const int32_t Jt = J0 + (int32_t)threadIdx.x;
  const int32_t sb = Jt < J1 ? seg[Jt] : 0, se = Jt < J1 ? seg[Jt + 1] : 0;
  const TV s1 = (TV)first_step(sub);
  const int32_t row = f0 + (int32_t)threadIdx.x;
  if (row < f1) {
    const TV ri = b[row] - s1 * v1[row];
    const TV mi = minv[row], pv = pp[row];
    int32_t base, w;
    sell_row(sptr, row, &base, &w);
    const TV acc =
        sell_dot_t<TV, TV>(col, val, base, w, [&](int32_t c) { return b[c] - s1 * v1[c]; });
    r1[row] = ri;
    z[row] = ri * mi;
    sh[threadIdx.x] = pv * (ri - acc);
  }
  __syncthreads();
  for (int32_t J = Jt; J < J1; J += kBlock) {
    const int32_t m0 = (J == Jt ? sb : seg[J]) - f0, e = (J == Jt ? se : seg[J + 1]) - f0;
    TV s = 0;
    for (int32_t m = m0; m < e; ++m) s += sh[m];
    rc[J] = s;
  }
}

// y = z + M^-1 (r - A z); with DOT also the block partials of (r, y)
// (with a dot partner dv, the partials are of (dv, y) instead)
// (OUT: y in the caller's numbering, position row of it at perm[row])
template <typename TV, typename TR, typename TO, bool DOT, typename TA = TV, bool OUT = false>
__global__ void __launch_bounds__(kBlock) k_post(
    int32_t n, int32_t chunk, const int32_t *__restrict__ sptr, const int32_t *__restrict__ col,
    const TA *__restrict__ val, const TV *__restrict__ minv, const TR *__restrict__ r,
    const TV *__restrict__ z, TO *__restrict__ y, double *__restrict__ partials,
    const int32_t *__restrict__ done, const double *__restrict__ dv = nullptr,
    const int32_t *__restrict__ perm = nullptr) {
  if (*done) return;
  int32_t rb, re;
  rows_of_block(n, chunk, &rb, &re);
  double d[1] = {0.0};
  for (int32_t row = rb + threadIdx.x; row < re; row += kBlock) {
    const TR rr = r[row];
    const TV zr = z[row], mr = minv[row];
    int32_t base, w;
    sell_row(sptr, row, &base, &w);
    const TV acc = sell_dot_t<TV, TA>(col, val, base, w, [&](int32_t c) { return z[c]; });
    const TO yo = (TO)(zr + ((TV)rr - acc) * mr);
    y[OUT ? perm[row] : row] = yo;
    if (DOT) d[0] += (dv ? dv[row] : (double)rr) * (double)yo;
  }
  if (DOT) block_partial<1>(d, partials);
}

// ---- LDS-staged gathers (level 0): the same products as above, with the
// gathered vector's entries of the block's tile loaded into LDS first ----

// xs[i] = x(hidx[h0 + i]) for the block's list of u entries, eight loads in
// flight per thread, then a barrier
template <typename TV, typename X>
__device__ __forceinline__ void stage_tile(TV *xs, const int32_t *__restrict__ hidx, int32_t h0,
                                           int32_t u, X x) {
  for (int32_t i0 = threadIdx.x; i0 < u; i0 += 8 * kBlock) {
    int32_t c[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int32_t i = i0 + q * kBlock;
      c[q] = i < u ? hidx[h0 + i] : 0;
    }
    TV v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = i0 + q * kBlock < u ? x(c[q]) : TV(0);
#pragma unroll
    for (int q = 0; q < 8; ++q)
      if (i0 + q * kBlock < u) xs[i0 + q * kBlock] = v[q];
  }
  __syncthreads();
}

// sum_k val[k] * xs[lcol[k]] over one SELL row: the products and sums of
// sell_dot_t, in the same order and with the same unconditional batched
// loads, with the operands read from LDS
template <typename TV, typename TA>
__device__ __forceinline__ TV sell_dot_lds(const uint16_t *__restrict__ lcol,
                                           const TA *__restrict__ val, int32_t base, int32_t w,
                                           const TV *xs) {
  TV acc = 0;
  for (int32_t k0 = 0; k0 < w; k0 += kRowBatch) {
    int32_t c[kRowBatch];
    TA va[kRowBatch];
#pragma unroll
    for (int u = 0; u < kRowBatch; ++u) {
      const int32_t idx = base + (k0 + u < w ? k0 + u : w - 1) * kSlice;
      c[u] = ld_stream(&lcol[idx]);
      va[u] = ld_stream(&val[idx]);
    }
    TV g[kRowBatch];
#pragma unroll
    for (int u = 0; u < kRowBatch; ++u) g[u] = xs[c[u]];
#pragma unroll
    for (int u = 0; u < kRowBatch; ++u)
      if (k0 + u < w) acc += (TV)va[u] * g[u];
  }
  return acc;
}

// k_pre_restrict with the tile of block b = its segment rows (tiles hseg).
// The LDS kernels take their tiles in XCD-aware order (xcd_block): each XCD
// works down one contiguous range of tiles, so a tile's staged neighbours
// were mostly just loaded into the same L2 by the tiles before it (160^3
// FP64 down step 73.6 -> 64.4 us). The partial sums stay indexed by blockIdx.
template <typename TV, typename TR, int MODE, typename TA = TV, int R = 1, bool FIN = false>
__global__ void __launch_bounds__(kBlock) k_pre_restrict_lds(
    int32_t nc, int32_t G, const int32_t *__restrict__ seg, const int32_t *__restrict__ sptr,
    const uint16_t *__restrict__ lcol, const int32_t *__restrict__ hptr,
    const int32_t *__restrict__ hidx, const TA *__restrict__ val, const TV *__restrict__ minv,
    const TV *__restrict__ pp, const TR *__restrict__ r, TV *__restrict__ z,
    TV *__restrict__ rc, const int32_t *__restrict__ done, FinRR fin = FinRR{}) {
  extern __shared__ double lds_d[];
  TV *xs = reinterpret_cast<TV *>(lds_d);
  __shared__ TV sh[kBlock * R];
  if (FIN ? !stop_test(fin) : *done != 0) return;
  const int32_t tb = xcd_block(blockIdx.x, gridDim.x);
  const int32_t J0 = tb * G;
  const int32_t J1 = min(nc, J0 + G);
  const int32_t f0 = seg[J0], f1 = seg[J1];
  const int32_t h0 = hptr[tb];
  // the operands that do not come from the staged tile are loaded first, so
  // their latency overlaps the staging
  int32_t pb[R], pw[R];
  TV pr[R], pm[R], pq[R];
#pragma unroll
  for (int u = 0; u < R; ++u) {
    const int32_t row = f0 + (int32_t)threadIdx.x + u * kBlock;
    pb[u] = pw[u] = 0;
    pr[u] = pm[u] = pq[u] = TV(0);
    if (row < f1) {
      sell_row(sptr, row, &pb[u], &pw[u]);
      pr[u] = (TV)r[row];
      if (MODE != kPreFromZ) pm[u] = minv[row];
      pq[u] = pp[row];
    }
  }
  const int32_t Jt = J0 + (int32_t)threadIdx.x;
  const int32_t sb = Jt < J1 ? seg[Jt] : 0, se = Jt < J1 ? seg[Jt + 1] : 0;
  if (MODE == kPreFromZ)
    stage_tile(xs, hidx, h0, hptr[tb + 1] - h0, [&](int32_t c) { return z[c]; });
  else if (MODE == kPreStagedZ)
    stage_tile(xs, hidx, h0, hptr[tb + 1] - h0,
               [&](int32_t c) { return (TV)r[c] * minv[c]; });
  else
    stage_tile(xs, hidx, h0, hptr[tb + 1] - h0, [&](int32_t c) { return (TV)r[c]; });
#pragma unroll
  for (int u = 0; u < R; ++u) {
    const int32_t row = f0 + (int32_t)threadIdx.x + u * kBlock;
    if (row < f1) {
      const TV acc = sell_dot_lds<TV, TA>(lcol, val, pb[u], pw[u], xs);
      const TV ri = pr[u];
      if (MODE != kPreFromZ) z[row] = ri * pm[u];
      sh[threadIdx.x + u * kBlock] = pq[u] * (ri - acc);
    }
  }
  __syncthreads();
  for (int32_t J = Jt; J < J1; J += kBlock) {
    const int32_t b = (J == Jt ? sb : seg[J]) - f0, e = (J == Jt ? se : seg[J + 1]) - f0;
    TV s = 0;
    for (int32_t m = b; m < e; ++m) s += sh[m];
    rc[J] = s;
  }
}

// k_post with the tile of block b = its row chunk (tiles hrow), XCD-aware order
template <typename TV, typename TR, typename TO, bool DOT, typename TA = TV, bool OUT = false>
__global__ void __launch_bounds__(kBlock) k_post_lds(
    int32_t n, int32_t chunk, const int32_t *__restrict__ sptr, const uint16_t *__restrict__ lcol,
    const int32_t *__restrict__ hptr, const int32_t *__restrict__ hidx,
    const TA *__restrict__ val, const TV *__restrict__ minv, const TR *__restrict__ r,
    const TV *__restrict__ z, TO *__restrict__ y, double *__restrict__ partials,
    const int32_t *__restrict__ done, const double *__restrict__ dv = nullptr,
    const int32_t *__restrict__ perm = nullptr) {
  extern __shared__ double lds_d[];
  TV *xs = reinterpret_cast<TV *>(lds_d);
  if (*done) return;
  int32_t rb, re;
  const int32_t tb = xcd_block(blockIdx.x, gridDim.x);
  rb = (int32_t)((int64_t)tb * chunk);
  re = (int32_t)min((int64_t)n, (int64_t)rb + chunk);
  const int32_t h0 = hptr[tb];
  int32_t row = rb + (int32_t)threadIdx.x, nb = 0, nw = 0;
  if (row < re) sell_row(sptr, row, &nb, &nw);
  stage_tile(xs, hidx, h0, hptr[tb + 1] - h0, [&](int32_t c) { return z[c]; });
  double d[1] = {0.0};
  for (; row < re; row += kBlock) {
    const int32_t base = nb, w = nw;
    if (row + kBlock < re) sell_row(sptr, row + kBlock, &nb, &nw);
    const TV acc = sell_dot_lds<TV, TA>(lcol, val, base, w, xs);
    const TR rr = r[row];
    const TO yo = (TO)(z[row] + ((TV)rr - acc) * minv[row]);
    y[OUT ? perm[row] : row] = yo;
    if (DOT) d[0] += (dv ? dv[row] : (double)rr) * (double)yo;
  }
  if (DOT) block_partial<1>(d, partials);
}

// ---- smoothed aggregation: unfused down and up steps (Pbar is not a
// segment map, so restriction and prolongation are CSR products) ----

// z = M^-1 r and t = r - A z = r - (A M^-1) r (the first sweep from zero)
template <typename TV, typename TR>
__global__ void __launch_bounds__(kBlock) k_pre_resid(
    int32_t n, int32_t chunk, const int32_t *__restrict__ sptr, const int32_t *__restrict__ col,
    const TV *__restrict__ sval, const TV *__restrict__ minv, const TR *__restrict__ r,
    TV *__restrict__ z, TV *__restrict__ t, const int32_t *__restrict__ done) {
  if (*done) return;
  int32_t rb, re;
  rows_of_block(n, chunk, &rb, &re);
  for (int32_t row = rb + threadIdx.x; row < re; row += kBlock) {
    int32_t base, w;
    sell_row(sptr, row, &base, &w);
    const TV acc = sell_dot(col, sval, base, w, [&](int32_t c) { return (TV)r[c]; });
    const TV ri = (TV)r[row];
    z[row] = ri * minv[row];
    t[row] = ri - acc;
  }
}

// t = r - A z
template <typename TV, typename TR, typename TA = TV>
__global__ void __launch_bounds__(kBlock) k_resid(
    int32_t n, int32_t chunk, const int32_t *__restrict__ sptr, const int32_t *__restrict__ col,
    const TA *__restrict__ val, const TR *__restrict__ r, const TV *__restrict__ z,
    TV *__restrict__ t, const int32_t *__restrict__ done) {
  if (*done) return;
  int32_t rb, re;
  rows_of_block(n, chunk, &rb, &re);
  for (int32_t row = rb + threadIdx.x; row < re; row += kBlock) {
    int32_t base, w;
    sell_row(sptr, row, &base, &w);
    const TV acc = sell_dot_t<TV, TA>(col, val, base, w, [&](int32_t c) { return z[c]; });
    t[row] = (TV)r[row] - acc;
  }
}

// sum over row i of a CSR matrix of val * x(col), with LPR consecutive lanes
// per row: lane k takes the entries k, k + LPR, ..., then the lanes' sums
// are added across the group (every lane of the group gets the total)
template <typename TV, int LPR, typename TA, typename X>
__device__ __forceinline__ TV csr_row_dot(int32_t i, int32_t nr, const int32_t *__restrict__ rp,
                                          const int32_t *__restrict__ ci,
                                          const TA *__restrict__ val, X x) {
  const int lane = threadIdx.x % LPR;
  TV acc = 0;
  if (i < nr) {
    // a lane's entries in batches of kRowBatch: all index and value loads,
    // then all gathers, then the products in order
    const int32_t e1 = rp[i + 1];
    for (int32_t e0 = rp[i] + lane; e0 < e1; e0 += LPR * kRowBatch) {
      int32_t c[kRowBatch];
      TV v[kRowBatch], g[kRowBatch];
#pragma unroll
      for (int u = 0; u < kRowBatch; ++u) {
        const int32_t e = e0 + u * LPR;
        c[u] = 0;
        v[u] = 0;
        if (e < e1) {
          c[u] = ci[e];
          v[u] = (TV)val[e];
        }
      }
#pragma unroll
      for (int u = 0; u < kRowBatch; ++u) g[u] = e0 + u * LPR < e1 ? x(c[u]) : TV(0);
#pragma unroll
      for (int u = 0; u < kRowBatch; ++u)
        if (e0 + u * LPR < e1) acc += v[u] * g[u];
    }
  }
  for (int o = LPR / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o, LPR);
  return acc;
}

// y = M x for a CSR M, or with ADD y += M x (LPR lanes per row)
template <typename TV, bool ADD, int LPR>
__global__ void __launch_bounds__(kBlock) k_csr_apply(int32_t nr, const int32_t *__restrict__ rp,
                                                      const int32_t *__restrict__ ci,
                                                      const TV *__restrict__ val,
                                                      const TV *__restrict__ x, TV *__restrict__ y,
                                                      const int32_t *__restrict__ done) {
  if (*done) return;
  const int32_t i = (int32_t)(((int64_t)blockIdx.x * kBlock + threadIdx.x) / LPR);
  const TV acc = csr_row_dot<TV, LPR>(i, nr, rp, ci, val, [&](int32_t c) { return x[c]; });
  if (i < nr && threadIdx.x % LPR == 0) y[i] = ADD ? y[i] + acc : acc;
}

// smoothing on a long-row level (CSR in the solve order, LPR lanes per row):
// MODE 0: y = z + M^-1 (r - A z); MODE 1: y = r - A z (the residual)
template <typename TV, typename TR, int MODE, int LPR>
__global__ void __launch_bounds__(kBlock) k_smooth_rows(
    int32_t n, const int32_t *__restrict__ rp, const int32_t *__restrict__ ci,
    const TV *__restrict__ val, const TV *__restrict__ minv, const TR *__restrict__ r,
    const TV *__restrict__ z, TV *__restrict__ y, const int32_t *__restrict__ done) {
  if (*done) return;
  const int32_t i = (int32_t)(((int64_t)blockIdx.x * kBlock + threadIdx.x) / LPR);
  const TV acc = csr_row_dot<TV, LPR>(i, n, rp, ci, val, [&](int32_t c) { return z[c]; });
  if (i < n && threadIdx.x % LPR == 0) {
    const TV res = (TV)r[i] - acc;
    y[i] = MODE == 0 ? z[i] + res * minv[i] : res;
  }
}

// lanes per row for nr rows of nnz entries: two to three entries per lane
// (rows shorter than 6 entries: one lane, a single batch of loads), and more
// lanes (up to a wavefront) while fewer than 2^19 threads would be in
// flight. At 160^3 (smoothed hierarchy) one lane per entry made the big
// levels' products up to 30 % slower, about 8 entries per lane 7 % slower
// per iteration; whole wavefronts made the small levels' twice as fast.
inline int lanes_for(int64_t nr, int64_t nnz) {
  const double avg = nr > 0 ? (double)nnz / nr : 1.0;
  int l = avg >= 96 ? 32 : avg >= 40 ? 16 : avg >= 12 ? 8 : avg >= 6 ? 4 : 1;
  while (l < 64 && (double)nr * l < (double)(1 << 19) && l < avg) l *= 2;
  return l;
}

template <typename TV, bool ADD>
void csr_apply(hipStream_t s, int32_t nr, int64_t nnz, const int32_t *rp, const int32_t *ci,
               const TV *val, const TV *x, TV *y, const int32_t *done) {
  const int lpr = lanes_for(nr, nnz);
  const int32_t g = ceil_div((int64_t)nr * lpr, kBlock);
  switch (lpr) {
    case 1: k_csr_apply<TV, ADD, 1><<<g, kBlock, 0, s>>>(nr, rp, ci, val, x, y, done); break;
    case 2: k_csr_apply<TV, ADD, 2><<<g, kBlock, 0, s>>>(nr, rp, ci, val, x, y, done); break;
    case 4: k_csr_apply<TV, ADD, 4><<<g, kBlock, 0, s>>>(nr, rp, ci, val, x, y, done); break;
    case 8: k_csr_apply<TV, ADD, 8><<<g, kBlock, 0, s>>>(nr, rp, ci, val, x, y, done); break;
    case 16: k_csr_apply<TV, ADD, 16><<<g, kBlock, 0, s>>>(nr, rp, ci, val, x, y, done); break;
    case 32: k_csr_apply<TV, ADD, 32><<<g, kBlock, 0, s>>>(nr, rp, ci, val, x, y, done); break;
    default: k_csr_apply<TV, ADD, 64><<<g, kBlock, 0, s>>>(nr, rp, ci, val, x, y, done); break;
  }
}

template <typename TV, typename TR, int MODE>
void smooth_rows(hipStream_t s, int32_t n, int64_t nnz, const int32_t *rp, const int32_t *ci,
                 const TV *val, const TV *minv, const TR *r, const TV *z, TV *y,
                 const int32_t *done) {
  const int lpr = lanes_for(n, nnz);
  const int32_t g = ceil_div((int64_t)n * lpr, kBlock);
  switch (lpr) {
    case 1: k_smooth_rows<TV, TR, MODE, 1><<<g, kBlock, 0, s>>>(n, rp, ci, val, minv, r, z, y, done); break;
    case 2: k_smooth_rows<TV, TR, MODE, 2><<<g, kBlock, 0, s>>>(n, rp, ci, val, minv, r, z, y, done); break;
    case 4: k_smooth_rows<TV, TR, MODE, 4><<<g, kBlock, 0, s>>>(n, rp, ci, val, minv, r, z, y, done); break;
    case 8: k_smooth_rows<TV, TR, MODE, 8><<<g, kBlock, 0, s>>>(n, rp, ci, val, minv, r, z, y, done); break;
    case 16: k_smooth_rows<TV, TR, MODE, 16><<<g, kBlock, 0, s>>>(n, rp, ci, val, minv, r, z, y, done); break;
    case 32: k_smooth_rows<TV, TR, MODE, 32><<<g, kBlock, 0, s>>>(n, rp, ci, val, minv, r, z, y, done); break;
    default: k_smooth_rows<TV, TR, MODE, 64><<<g, kBlock, 0, s>>>(n, rp, ci, val, minv, r, z, y, done); break;
  }
}

// Up step: post-smoothing of the coarse level c for this block's kBlock
// coarse rows, y = z_c + M^-1 (r_c - A_c z_c) (kept in LDS), then the
// prolongation z_f += P y over the fine segments of those rows.
template <typename TV>
__global__ void __launch_bounds__(kBlock) k_post_prolong(
    int32_t nc, const int32_t *__restrict__ sptr, const int32_t *__restrict__ col,
    const TV *__restrict__ val, const TV *__restrict__ minv, const TV *__restrict__ rcv,
    const TV *__restrict__ zc, const int32_t *__restrict__ seg, const int32_t *__restrict__ aggp,
    const TV *__restrict__ pp, TV *__restrict__ zf, const int32_t *__restrict__ done) {
  __shared__ TV sh[kBlock];
  if (*done) return;
  const int32_t J0 = blockIdx.x * kBlock;
  const int32_t J = J0 + threadIdx.x;
  // the fine range and the row's own operands first: their loads overlap the gathers
  const int32_t J1 = min(nc, J0 + kBlock);
  const int32_t f0 = seg[J0], f1 = seg[J1];
  if (J < nc) {
    const TV zj = zc[J], rj = rcv[J], mj = minv[J];
    int32_t base, w;
    sell_row(sptr, J, &base, &w);
    const TV acc = sell_dot(col, val, base, w, [&](int32_t c) { return zc[c]; });
    sh[threadIdx.x] = zj + (rj - acc) * mj;
  }
  __syncthreads();
  prolong_add(f0, f1, (int32_t)threadIdx.x, kBlock, aggp, pp, zf,
              [&](int32_t a) { return sh[a - J0]; });
}

// ---- levels of wide rows ----
//
// The coarse levels of an irregular matrix have few rows, some of them of
// hundreds of entries: with a thread per row a kernel takes what one thread's
// chain of gathers takes. Here a block takes kWideRows rows, its 256 threads load
// kWideStep entries of each and the gathered values into LDS, a step ahead of
// their use, and a lane per row adds up the products: the same sums in the same
// order as sell_dot. A random graph of 100003 rows and degree 9 (levels of 14101
// rows of 52 entries and of 1908 of 331): 3.53 -> 2.04 ms a solve; one of 50000 and
// degree 4.5, whose last 25 levels hold a row of all 1200 columns: 43 -> 12 us a
// kernel, 45.3 -> 15.6 ms a solve, 15.9 with 64 entries a step. (32 entries in
// flight per thread instead, still a thread per row: 7.3 ms for the 3.53.)
// Where the level above the coarsest is of that kind, its kernels in this form and
// the coarsest product also beat k_tail, one block for all its rows: 2.04 -> 1.73 ms;
// 10000 rows, degree 9: 1.18 -> 0.69 ms.
// kWideMean: stored entries per row, padding included, from which a level takes it
// (16, 24 and 32 are the same on these), at up to kWideMany rows; with 64 blocks of
// 96^3 and 128^3, whose coarse levels store 32 to 64, take 7.16 and 12.25 ms for 6.61
// and 11.69. Above kWideMany rows a thread per row fills the chip, and only rows of
// twice as many entries pay for the LDS: 256^3 in blocks 95.0 -> 93.9 ms without them on
// its fourth level, the graph of 200000 and degree 13 (29000 rows) 3.14 -> 2.99 with.
constexpr int kWideMean = 32;
constexpr int32_t kWideMany = 32768;
constexpr int kWideRows = 16;
constexpr int kWideStep = 128;
constexpr int kWideLanes = kBlock / kWideRows;

// the product of row f0 + threadIdx.x % kWideRows (rows below f1) with x: the
// result is threads 0 .. kWideRows - 1's
template <typename TV, typename X>
__device__ __forceinline__ TV wide_dot(const int32_t *__restrict__ sptr,
                                       const int32_t *__restrict__ col,
                                       const TV *__restrict__ val, int32_t f0, int32_t f1, X x) {
  constexpr int kPer = kWideStep / kWideLanes;
  __shared__ TV sv[2][kWideStep][kWideRows], sg[2][kWideStep][kWideRows];
  const int32_t rl = (int32_t)threadIdx.x % kWideRows, el = (int32_t)threadIdx.x / kWideRows;
  const int32_t row = f0 + rl;
  int32_t base = 0, w = 0, b0, w0, w1;
  if (row < f1) sell_row(sptr, row, &base, &w);
  sell_row(sptr, f0, &b0, &w0);  // (the rows are in at most two slices)
  sell_row(sptr, f1 - 1, &b0, &w1);
  const int32_t steps = (max(w0, w1) + kWideStep - 1) / kWideStep;
  int32_t c[kPer];
  TV v[kPer], g[kPer];
  auto entries = [&](int32_t k0) {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int32_t e = k0 + el + u * kWideLanes;
      c[u] = -1;
      v[u] = 0;
      if (e < w) {
        c[u] = ld_stream(&col[base + e * kSlice]);
        v[u] = ld_stream(&val[base + e * kSlice]);
      }
    }
  };
  auto gather = [&](int32_t b) {
#pragma unroll
    for (int u = 0; u < kPer; ++u) g[u] = c[u] >= 0 ? x(c[u]) : TV(0);
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      sv[b][el + u * kWideLanes][rl] = v[u];
      sg[b][el + u * kWideLanes][rl] = g[u];
    }
  };
  TV acc = 0;
  entries(0);
  gather(0);
  for (int32_t st = 0; st < steps; ++st) {
    __syncthreads();  // step st is in LDS, and the one before it has been added
    const int32_t b = st & 1, k0 = st * kWideStep;
    if (st + 1 < steps) entries(k0 + kWideStep);
    if (threadIdx.x < kWideRows) {
      const int32_t m = min(w - k0, kWideStep);
#pragma unroll 8
      for (int32_t e = 0; e < m; ++e) acc += sv[b][e][rl] * sg[b][e][rl];
    }
    if (st + 1 < steps) gather(b ^ 1);
  }
  return acc;
}

// k_pre_restrict (one sweep, A M^-1) and k_post_prolong in that form; G coarse
// positions hold at most kWideRows rows
template <typename TV>
__global__ void __launch_bounds__(kBlock) k_pre_restrict_wide(
    int32_t nc, int32_t G, const int32_t *__restrict__ seg, const int32_t *__restrict__ sptr,
    const int32_t *__restrict__ col, const TV *__restrict__ val, const TV *__restrict__ minv,
    const TV *__restrict__ pp, const TV *__restrict__ r, TV *__restrict__ z, TV *__restrict__ rc,
    const int32_t *__restrict__ done) {
  __shared__ TV sh[kWideRows];
  if (*done) return;
  const int32_t J0 = blockIdx.x * G, J1 = min(nc, J0 + G);
  const int32_t f0 = seg[J0], f1 = seg[J1];
  const TV acc = wide_dot(sptr, col, val, f0, f1, [&](int32_t c) { return r[c]; });
  const int32_t row = f0 + (int32_t)threadIdx.x;
  if (threadIdx.x < kWideRows && row < f1) {
    const TV ri = r[row];
    z[row] = ri * minv[row];
    sh[threadIdx.x] = pp[row] * (ri - acc);
  }
  __syncthreads();
  const int32_t J = J0 + (int32_t)threadIdx.x;
  if (J < J1) {
    TV s = 0;
    for (int32_t m = seg[J]; m < seg[J + 1]; ++m) s += sh[m - f0];
    rc[J] = s;
  }
}

template <typename TV>
__global__ void __launch_bounds__(kBlock) k_post_prolong_wide(
    int32_t nc, const int32_t *__restrict__ sptr, const int32_t *__restrict__ col,
    const TV *__restrict__ val, const TV *__restrict__ minv, const TV *__restrict__ rcv,
    const TV *__restrict__ zc, const int32_t *__restrict__ seg, const int32_t *__restrict__ aggp,
    const TV *__restrict__ pp, TV *__restrict__ zf, const int32_t *__restrict__ done) {
  __shared__ TV sh[kWideRows];
  if (*done) return;
  const int32_t J0 = blockIdx.x * kWideRows, J1 = min(nc, J0 + kWideRows);
  const TV acc = wide_dot(sptr, col, val, J0, J1, [&](int32_t c) { return zc[c]; });
  const int32_t J = J0 + (int32_t)threadIdx.x;
  if (J < J1) sh[threadIdx.x] = zc[J] + (rcv[J] - acc) * minv[J];
  __syncthreads();
  prolong_add(seg[J0], seg[J1], (int32_t)threadIdx.x, kBlock, aggp, pp, zf,
              [&](int32_t c) { return sh[c - J0]; });
}

// Coarsest level with prolongation: z_L = A_L^-1 r_L, then z_f += P z_L over
// all fine positions; one block of 1024 threads. Eight consecutive threads
// share a row (coalesced 64-byte pieces of it), each summing every eighth
// entry against r_L staged in LDS, so 128 rows are in flight per pass.
constexpr int kCoarseSplit = 8;
template <typename TV>
__global__ void __launch_bounds__(1024) k_coarse_prolong(
    int32_t nL, const double *__restrict__ Ainv, const TV *__restrict__ rL, int32_t nf,
    const int32_t *__restrict__ aggp, const TV *__restrict__ pp, TV *__restrict__ zf,
    const int32_t *__restrict__ done) {
  extern __shared__ double sm[];
  if (*done) return;
  double *rs = sm, *zs = sm + nL;
  for (int32_t k = threadIdx.x; k < nL; k += blockDim.x) rs[k] = (double)rL[k];
  __syncthreads();
  const int32_t part = threadIdx.x % kCoarseSplit;
  const int32_t rows_per_pass = blockDim.x / kCoarseSplit;
  for (int32_t i0 = 0; i0 < nL; i0 += rows_per_pass) {
    const int32_t i = i0 + (int32_t)threadIdx.x / kCoarseSplit;
    double s = 0.0;
    if (i < nL) {
      const double *row = Ainv + (int64_t)i * nL;
#pragma unroll 8
      for (int32_t k = part; k < nL; k += kCoarseSplit) s += row[k] * rs[k];
    }
    for (int o = kCoarseSplit / 2; o > 0; o >>= 1) s += __shfl_down(s, o, kCoarseSplit);
    if (i < nL && part == 0) zs[i] = s;
  }
  __syncthreads();
  prolong_add(0, nf, (int32_t)threadIdx.x, (int32_t)blockDim.x, aggp, pp, zf,
              [&](int32_t a) { return (TV)zs[a]; });
}

// The two halves of k_coarse_prolong with many blocks, the same sums in the same
// order, for n_L above kCoarseOne: one block reads A_L^-1 at the rate of one CU
// (n_L = 1155: 123 us, these two 11.7 + 4.0; at 256 the read is 0.5 MB, 6 us).
constexpr int kCoarseOne = 256;
template <typename TV>
__global__ void __launch_bounds__(kBlock) k_coarse_rows(int32_t nL,
                                                        const double *__restrict__ Ainv,
                                                        const TV *__restrict__ rL,
                                                        TV *__restrict__ zL,
                                                        const int32_t *__restrict__ done) {
  if (*done) return;
  const int32_t part = threadIdx.x % kCoarseSplit;
  const int32_t i = (int32_t)(blockIdx.x * kBlock + threadIdx.x) / kCoarseSplit;
  double s = 0.0;
  if (i < nL) {
    const double *row = Ainv + (int64_t)i * nL;
#pragma unroll 8
    for (int32_t k = part; k < nL; k += kCoarseSplit) s += row[k] * (double)rL[k];
  }
  for (int o = kCoarseSplit / 2; o > 0; o >>= 1) s += __shfl_down(s, o, kCoarseSplit);
  if (i < nL && part == 0) zL[i] = (TV)s;
}

// z_f += P y
template <typename TV>
__global__ void __launch_bounds__(kBlock) k_prolong(int32_t nf, const int32_t *__restrict__ aggp,
                                                    const TV *__restrict__ pp,
                                                    const TV *__restrict__ y,
                                                    TV *__restrict__ zf,
                                                    const int32_t *__restrict__ done) {
  if (*done) return;
  prolong_add(0, nf, (int32_t)(blockIdx.x * kBlock + threadIdx.x), (int32_t)(gridDim.x * kBlock),
              aggp, pp, zf, [&](int32_t a) { return y[a]; });
}

// Tail of the V-cycle in one block, for a level t = L - 1 small enough for
// LDS (t >= 1, one pre- and one post-sweep): starting from r_t it does the
// down step on t, the coarsest solve, the up step on t, and the
// prolongation into level t - 1 (zf += P_{t-1} y_t), with level t's vectors
// in LDS. Replaces the three latency-bound kernels of the last two levels.
constexpr int kTailMax = 2048;  // largest level t handled in LDS
constexpr int kTailCoarseMax = 512;
constexpr int kTailPro = 8;    // prolongation positions per thread loaded up front (FP32;
                               // half as many in FP64, within the register budget)
constexpr int kTailRow = 16;   // A_L^-1 entries per thread loaded up front (n_L <= 128)
template <typename TV>
__global__ void __launch_bounds__(1024) k_tail(
    int32_t nt, const int32_t *__restrict__ sptr, const int32_t *__restrict__ col,
    const TV *__restrict__ sval, const TV *__restrict__ val, const TV *__restrict__ minv,
    const TV *__restrict__ rt, const int32_t *__restrict__ seg, const int32_t *__restrict__ aggp,
    const TV *__restrict__ pp, int32_t nL, const double *__restrict__ Ainv, int32_t nf,
    const int32_t *__restrict__ aggp_f, const TV *__restrict__ pp_f, TV *__restrict__ zf,
    const int32_t *__restrict__ done) {
  __shared__ TV rs[kTailMax], zs[kTailMax], ys[kTailMax];
  __shared__ double rl[kTailCoarseMax], zl[kTailCoarseMax];
  if (*done) return;
  const int32_t tid = threadIdx.x, nth = blockDim.x;
  // The operands of the last two phases do not depend on the first ones:
  // load them now so their latency overlaps the phases before.
  constexpr int kPro = sizeof(TV) == 8 ? kTailPro / 2 : kTailPro;
  int32_t fa[kPro];  // prolongation: this thread's first kPro positions
  TV fp[kPro], fz[kPro];
#pragma unroll
  for (int u = 0; u < kPro; ++u) {
    const int32_t k = tid + u * nth;
    fa[u] = 0;
    fp[u] = fz[u] = 0;
    if (k < nf) {
      fa[u] = aggp_f[k];
      fp[u] = pp_f[k];
      fz[u] = zf[k];
    }
  }
  const int32_t part = tid % kCoarseSplit, irow = tid / kCoarseSplit;
  const bool one_pass = nL <= nth / kCoarseSplit && nL <= kCoarseSplit * kTailRow;
  double av[kTailRow];  // this thread's entries of its A_L^-1 row (one pass)
#pragma unroll
  for (int m = 0; m < kTailRow; ++m) {
    const int32_t k = part + m * kCoarseSplit;
    av[m] = one_pass && irow < nL && k < nL ? Ainv[(int64_t)irow * nL + k] : 0.0;
  }
  // the thread's first row of level t: its slice position, p, its coarse
  // position and its segment bounds, loaded with r so that the later phases
  // start without a round trip to memory
  int32_t b0 = 0, w0 = 0, a0 = 0, sb0 = 0, se0 = 0;
  TV p0 = 0;
  if (tid < nt) {
    const int32_t s = tid / kSlice;
    const int32_t s0 = sptr[s], s1 = sptr[s + 1];
    b0 = s0 + tid % kSlice;
    w0 = (s1 - s0) / kSlice;
    p0 = pp[tid];
    a0 = aggp[tid];
  }
  if (tid < nL) {
    sb0 = seg[tid];
    se0 = seg[tid + 1];
  }
  for (int32_t k = tid; k < nt; k += nth) {
    const TV r = rt[k];
    rs[k] = r;
    zs[k] = r * minv[k];
  }
  __syncthreads();
  // t = p (r - A M^-1 r), kept in ys
  for (int32_t k = tid; k < nt; k += nth) {
    int32_t base = b0, w = w0;
    if (k != tid) {
      const int32_t s = k / kSlice;
      base = sptr[s] + k % kSlice;
      w = (sptr[s + 1] - sptr[s]) / kSlice;
    }
    const TV acc = sell_dot(col, sval, base, w, [&](int32_t c) { return rs[c]; });
    ys[k] = (k == tid ? p0 : pp[k]) * (rs[k] - acc);
  }
  __syncthreads();
  for (int32_t J = tid; J < nL; J += nth) {
    TV a = 0;
    const int32_t mb = J == tid ? sb0 : seg[J], me = J == tid ? se0 : seg[J + 1];
    for (int32_t m = mb; m < me; ++m) a += ys[m];
    rl[J] = (double)a;
  }
  __syncthreads();
  // coarsest: eight threads per row of A_L^-1
  if (one_pass) {
    double a = 0.0;
#pragma unroll
    for (int m = 0; m < kTailRow; ++m)
      if (part + m * kCoarseSplit < nL) a += av[m] * rl[part + m * kCoarseSplit];
    for (int o = kCoarseSplit / 2; o > 0; o >>= 1) a += __shfl_down(a, o, kCoarseSplit);
    if (irow < nL && part == 0) zl[irow] = a;
  } else {
    for (int32_t i0 = 0; i0 < nL; i0 += nth / kCoarseSplit) {
      const int32_t i = i0 + irow;
      double a = 0.0;
      if (i < nL) {
        const double *row = Ainv + (int64_t)i * nL;
#pragma unroll 8
        for (int32_t k = part; k < nL; k += kCoarseSplit) a += row[k] * rl[k];
      }
      for (int o = kCoarseSplit / 2; o > 0; o >>= 1) a += __shfl_down(a, o, kCoarseSplit);
      if (i < nL && part == 0) zl[i] = a;
    }
  }
  __syncthreads();
  for (int32_t k = tid; k < nt; k += nth)
    zs[k] += (k == tid ? p0 : pp[k]) * (TV)zl[k == tid ? a0 : aggp[k]];
  __syncthreads();
  // post-smoothing on level t
  for (int32_t k = tid; k < nt; k += nth) {
    int32_t base = b0, w = w0;
    if (k != tid) {
      const int32_t s = k / kSlice;
      base = sptr[s] + k % kSlice;
      w = (sptr[s + 1] - sptr[s]) / kSlice;
    }
    const TV acc = sell_dot(col, val, base, w, [&](int32_t c) { return zs[c]; });
    ys[k] = zs[k] + (rs[k] - acc) * minv[k];
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kPro; ++u) {
    const int32_t k = tid + u * nth;
    if (k < nf) zf[k] = fz[u] + fp[u] * ys[fa[u]];
  }
  prolong_add(kPro * nth, nf, tid, nth, aggp_f, pp_f, zf, [&](int32_t a) { return ys[a]; });
}

// Single-level hierarchy: z = A_0^-1 r, one wavefront per row.
constexpr int kCoarseWaves = 4;
template <typename TI, typename TO>
__global__ void __launch_bounds__(kWave *kCoarseWaves) k_coarse_solve(
    int32_t n, const double *__restrict__ Ainv, const TI *__restrict__ r, TO *__restrict__ z,
    const int32_t *__restrict__ done) {
  if (*done) return;
  const int lane = threadIdx.x & (kWave - 1);
  const int32_t i = blockIdx.x * kCoarseWaves + threadIdx.x / kWave;
  if (i >= n) return;
  const double *row = Ainv + (int64_t)i * n;
  double s = 0.0;
  for (int32_t k = lane; k < n; k += kWave) s += row[k] * (double)r[k];
  for (int o = kWave / 2; o > 0; o >>= 1) s += __shfl_down(s, o, kWave);
  if (lane == 0) z[i] = (TO)s;
}

// z = M^-1 r (first of several pre-smoothing sweeps)
template <typename TV, typename TR>
__global__ void k_jacobi0(int32_t n, const TV *minv, const TR *r, TV *z, const int32_t *done) {
  if (*done) return;
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) z[i] = (TV)r[i] * minv[i];
}

// partials of (r, z) when level 0 is itself the coarsest level
__global__ void __launch_bounds__(kBlock) k_dot_rz(int32_t n, int32_t chunk, const double *r,
                                                   const double *z, double *partials,
                                                   const int32_t *done) {
  if (*done) return;
  int32_t rb, re;
  rows_of_block(n, chunk, &rb, &re);
  double d[1] = {0.0};
  for (int32_t i = rb + threadIdx.x; i < re; i += kBlock) d[0] += r[i] * z[i];
  block_partial<1>(d, partials);
}

// ---------------------------------------------------------------------------
// outer CG kernels (FP64, aggregate-major order of level 0)
// ---------------------------------------------------------------------------

__global__ void k_scal_init(PcgScal *s, double rtol, int32_t maxit) {
  s->rho = 0.0;
  s->pq = 0.0;
  s->alpha = 0.0;
  s->beta = 0.0;
  s->rr = 0.0;
  s->bb = 0.0;
  s->rtol = rtol;
  s->tol2 = 0.0;
  s->rr_true = 0.0;
  s->iter = 0;
  s->maxit = maxit;
  s->done = 0;
  s->phase = 0;
  s->rho1 = 0.0;
  s->iter1 = 0;
}

// MODE 0: r = b - A x and partials of (b, b), (r, r)
// MODE 1: partials of ||b - A x||^2 only
template <int MODE, typename TA>
__global__ void __launch_bounds__(kBlock) k_residual_norms(
    int32_t n, int32_t chunk, const int32_t *__restrict__ sptr, const int32_t *__restrict__ col,
    const TA *__restrict__ val, const double *__restrict__ b, const double *__restrict__ x,
    double *__restrict__ r, double *__restrict__ partials) {
  constexpr int NV = MODE == 0 ? 2 : 1;
  int32_t rb, re;
  rows_of_block(n, chunk, &rb, &re);
  double d[NV];
  for (int q = 0; q < NV; ++q) d[q] = 0.0;
  for (int32_t row = rb + threadIdx.x; row < re; row += kBlock) {
    int32_t base, w;
    sell_row(sptr, row, &base, &w);
    const double acc = sell_dot_t<double, TA>(col, val, base, w, [&](int32_t c) { return x[c]; });
    const double bi = b[row];
    const double ri = bi - acc;
    if (MODE == 0) {
      r[row] = ri;
      d[0] += bi * bi;
      d[NV - 1] += ri * ri;
    } else {
      d[0] += ri * ri;
    }
  }
  block_partial<NV>(d, partials);
}

__global__ void k_zero_if_zero_rhs(int32_t n, double *x, const PcgScal *scal) {
  if (scal->done != 4) return;
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) x[i] = 0.0;
}

// q = A p ; partials of (p, q)
template <typename TA>
__global__ void __launch_bounds__(kBlock) k_spmv_dot(
    int32_t n, int32_t chunk, const int32_t *__restrict__ sptr, const int32_t *__restrict__ col,
    const TA *__restrict__ val, const double *__restrict__ p, double *__restrict__ q,
    double *__restrict__ partials, const int32_t *__restrict__ done) {
  if (*done) return;
  int32_t rb, re;
  rows_of_block(n, chunk, &rb, &re);
  double d[1] = {0.0};
  for (int32_t row = rb + threadIdx.x; row < re; row += kBlock) {
    int32_t base, w;
    sell_row(sptr, row, &base, &w);
    const double acc = sell_dot_t<double, TA>(col, val, base, w, [&](int32_t c) { return p[c]; });
    q[row] = acc;
    d[0] += p[row] * acc;
  }
  block_partial<1>(d, partials);
}

// k_spmv_dot with the tile of block b = its row chunk (tiles hrow), XCD-aware order
template <typename TA>
__global__ void __launch_bounds__(kBlock) k_spmv_dot_lds(
    int32_t n, int32_t chunk, const int32_t *__restrict__ sptr, const uint16_t *__restrict__ lcol,
    const int32_t *__restrict__ hptr, const int32_t *__restrict__ hidx,
    const TA *__restrict__ val, const double *__restrict__ p, double *__restrict__ q,
    double *__restrict__ partials, const int32_t *__restrict__ done) {
  extern __shared__ double lds_d[];
  if (*done) return;
  int32_t rb, re;
  const int32_t tb = xcd_block(blockIdx.x, gridDim.x);
  rb = (int32_t)((int64_t)tb * chunk);
  re = (int32_t)min((int64_t)n, (int64_t)rb + chunk);
  const int32_t h0 = hptr[tb];
  int32_t row = rb + (int32_t)threadIdx.x, nb = 0, nw = 0;
  if (row < re) sell_row(sptr, row, &nb, &nw);
  stage_tile(lds_d, hidx, h0, hptr[tb + 1] - h0, [&](int32_t c) { return p[c]; });
  double d[1] = {0.0};
  for (; row < re; row += kBlock) {
    const int32_t base = nb, w = nw;
    if (row + kBlock < re) sell_row(sptr, row + kBlock, &nb, &nw);
    const double acc = sell_dot_lds<double, TA>(lcol, val, base, w, lds_d);
    q[row] = acc;
    d[0] += p[row] * acc;
  }
  block_partial<1>(d, partials);
}

// x += alpha p ; r -= alpha q ; partials of (r, r)
__global__ void __launch_bounds__(kBlock) k_update_xr(int32_t n, int32_t chunk,
                                                      double *__restrict__ x,
                                                      double *__restrict__ r,
                                                      const double *__restrict__ p,
                                                      const double *__restrict__ q,
                                                      double *__restrict__ partials,
                                                      const PcgScal *__restrict__ scal,
                                                      const int32_t *__restrict__ done) {
  if (*done) return;
  const double alpha = scal->alpha;
  int32_t rb, re;
  rows_of_block(n, chunk, &rb, &re);
  double d[1] = {0.0};
  for (int32_t i = rb + threadIdx.x; i < re; i += kBlock) {
    x[i] += alpha * p[i];
    const double ri = r[i] - alpha * q[i];
    r[i] = ri;
    d[0] += ri * ri;
  }
  block_partial<1>(d, partials);
}

// p = z + beta p (copy: p = z), W consecutive entries per thread: with W = 2
// one 16-byte access each (z and p 16-byte aligned; an odd last entry alone)
template <int W>
__global__ void k_xpay(int32_t n, const double *__restrict__ z, double *__restrict__ p,
                       const PcgScal *__restrict__ scal, int32_t copy,
                       const int32_t *__restrict__ done) {
  if (*done) return;
  const double beta = scal->beta;
  const int64_t i = W * ((int64_t)blockIdx.x * blockDim.x + threadIdx.x);
  if (W == 2 && i + 1 < n) {
    const double2 zv = reinterpret_cast<const double2 *>(z)[i / 2];
    double2 pv = zv;
    if (!copy) {
      pv = reinterpret_cast<const double2 *>(p)[i / 2];
      pv.x = zv.x + beta * pv.x;
      pv.y = zv.y + beta * pv.y;
    }
    reinterpret_cast<double2 *>(p)[i / 2] = pv;
  } else if (i < n) {
    p[i] = copy ? z[i] : z[i] + beta * p[i];
  }
}

// ---- folded iterations ----
//
// On a small system a kernel costs its launch, about 4.6 us behind another one
// of the graph, whatever it does: 9 kernels of an iteration at 20^3 took 42 us,
// 15 at 96^3 110 us. The three one-block kernels that sum the partials are left
// out: each block of the kernel that needs a sum forms it by itself, as long
// as the partials are few (kFoldParts). And p = z + beta p joins the product
// with A, which forms the entries it gathers from z and the old p and writes
// the new p beside it, in the buffer of the other parity. What a kernel's
// blocks read of the scalars its block 0 does not write, except the flag,
// which each block reads once (sum_partials).
//
// Measured with every form at 8^3 to 192^3 (FP64, 1e-8; us a solve): all of it
// 20^3 922 -> 739, 32^3 1263 -> 1040, 48^3 1885 -> 1715; up to 512 partials
// (131 k rows): with 1024 (64^3) the blocks' sums cost what the kernels did, and
// with 4000 10 % more. The direction in the product alone: 64^3 2570 -> 2497,
// 75^3 5178 -> 5106, 100^3 5614 -> 5546; above 2^20 rows, where a block takes two
// rows per thread, 102^3 6111 -> 6158, 116^3 7127 -> 7075, 124^3 8394 -> 8433,
// 128^3 8908 -> 8855, 160^3 15874 -> 15919 and 192^3 31449 -> 31554 (it gathers
// two vectors, and staging them costs what the kernel saved): up to kDirRows. ((r, r) summed by the kernel that sums (r, z), one kernel less
// for a V-cycle too many at the end, gave 64^3 2480 -> 2459 and 96^3 4895 -> 4892,
// and cost a solve of one iteration at 96^3 258 -> 307.)
constexpr int32_t kFoldParts = 512;
// iterations that run while the host looks at the first ones; levels up to which
// an iteration is of at most nine kernels (see pcg)
constexpr int32_t kAhead = 4;
constexpr size_t kAheadLevels = 5;
constexpr int32_t kDirRows = 1 << 20;
// K-cycle levels of up to so many rows take the prolongation in the post-sweep
// (k_kpost) and r1 = b - s1 v1 in the down step (k_kdown): 80^3 to 1e-6 in FP64
// 3797 -> 3318 us with limit 131 k, 3304 with 1 M and 3348 with 16 k rows, 160^3
// 10655, 10738 and 10759: where launches cost more than the larger gathers. And
// where rows are as short as a 7-point level's (kUpMean stored entries a row): the
// chain of gathers per entry grows with them, and levels of long rows have kernels
// of their own. Random graphs of 10000 rows, degree 9, 1994 us on every level, 1238
// so (1392 without the two kernels); 60000, degree 11, 16.1, 7.64 and 10.1 ms;
// 100^3 anisotropic 12.37, 12.05 and 12.34; 96^3 in blocks 23.4, 21.1 and 22.3.
// (With 10 to 14 entries the same but for the anisotropic one, 12.35; with 20
// 64^3 in blocks 10.68 for 10.34.)
constexpr int32_t kUpRows = 131072;
constexpr int32_t kUpMean = 8;

// beta, the old and the new p; FOLD: beta from the partials of (r, z), summed
// here. false: done, or a breakdown.
struct Direction {
  double beta;
  bool first;
  const double *po;
  double *pn;
};
template <bool FOLD>
__device__ __forceinline__ bool next_direction(PcgScal *scal, const double *partials,
                                               int32_t nparts, double *p0, double *p1,
                                               Direction *D) {
  if (!FOLD && scal->done) return false;
  const int32_t iter = scal->iter;
  D->po = iter & 1 ? p1 : p0;
  D->pn = iter & 1 ? p0 : p1;
  D->first = iter == 0;
  if (!FOLD) {
    D->beta = scal->beta;
    return true;
  }
  const double rho = scal->rho;
  bool stopped;
  const double rz =
      sum_partials(partials + (int64_t)kRZPlane * kMaxParts, nparts, &scal->done, &stopped);
  if (stopped) return false;
  if (!(rz > 0.0)) {
    if (blockIdx.x == 0 && threadIdx.x == 0) scal->done = 3;
    return false;
  }
  D->beta = D->first ? 0.0 : rz / rho;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    scal->rho1 = rz;
    if (!D->first) scal->beta = D->beta;
  }
  return true;
}

// p = z + beta p, q = A p, partials of (p, q)
template <typename TA, bool FOLD>
__global__ void __launch_bounds__(kBlock) k_dir_spmv(
    int32_t n, int32_t chunk, const int32_t *__restrict__ sptr, const int32_t *__restrict__ col,
    const TA *__restrict__ val, const double *__restrict__ z, double *p0, double *p1,
    double *__restrict__ q, double *__restrict__ partials, PcgScal *scal) {
  Direction D;
  if (!next_direction<FOLD>(scal, partials, gridDim.x, p0, p1, &D)) return;
  auto dir = [&](int32_t c) -> double {
    return D.first ? z[c] : z[c] + D.beta * D.po[c];
  };
  int32_t rb, re;
  rows_of_block(n, chunk, &rb, &re);
  double d[1] = {0.0};
  for (int32_t row = rb + threadIdx.x; row < re; row += kBlock) {
    int32_t base, w;
    sell_row(sptr, row, &base, &w);
    const double pi = dir(row);
    const double acc = sell_dot_t<double, TA>(col, val, base, w, dir);
    D.pn[row] = pi;
    q[row] = acc;
    d[0] += pi * acc;
  }
  block_partial<1>(d, partials + (int64_t)kPQPlane * kMaxParts);
}

// the same with the tile of block b = its row chunk (tiles hrow), XCD-aware order
template <typename TA, bool FOLD>
__global__ void __launch_bounds__(kBlock) k_dir_spmv_lds(
    int32_t n, int32_t chunk, const int32_t *__restrict__ sptr, const uint16_t *__restrict__ lcol,
    const int32_t *__restrict__ hptr, const int32_t *__restrict__ hidx,
    const TA *__restrict__ val, const double *__restrict__ z, double *p0, double *p1,
    double *__restrict__ q, double *__restrict__ partials, PcgScal *scal) {
  extern __shared__ double lds_d[];
  Direction D;
  if (!next_direction<FOLD>(scal, partials, gridDim.x, p0, p1, &D)) return;
  auto dir = [&](int32_t c) -> double {
    return D.first ? z[c] : z[c] + D.beta * D.po[c];
  };
  int32_t rb, re;
  const int32_t tb = xcd_block(blockIdx.x, gridDim.x);
  rb = (int32_t)((int64_t)tb * chunk);
  re = (int32_t)min((int64_t)n, (int64_t)rb + chunk);
  const int32_t h0 = hptr[tb];
  int32_t row = rb + (int32_t)threadIdx.x, nb = 0, nw = 0;
  if (row < re) sell_row(sptr, row, &nb, &nw);
  stage_tile(lds_d, hidx, h0, hptr[tb + 1] - h0, dir);
  double d[1] = {0.0};
  for (; row < re; row += kBlock) {
    const int32_t base = nb, w = nw;
    if (row + kBlock < re) sell_row(sptr, row + kBlock, &nb, &nw);
    const double pi = dir(row);
    const double acc = sell_dot_lds<double, TA>(lcol, val, base, w, lds_d);
    D.pn[row] = pi;
    q[row] = acc;
    d[0] += pi * acc;
  }
  block_partial<1>(d, partials + (int64_t)kPQPlane * kMaxParts);
}

// alpha from the partials of (p, q); x += alpha p, r -= alpha q, partials of (r, r)
__global__ void __launch_bounds__(kBlock) k_update_fold(int32_t n, int32_t chunk,
                                                        double *__restrict__ x,
                                                        double *__restrict__ r, const double *p0,
                                                        const double *p1,
                                                        const double *__restrict__ q,
                                                        double *__restrict__ partials,
                                                        PcgScal *scal) {
  const double rho = scal->rho1;
  const int32_t iter = scal->iter;
  bool stopped;
  const double pq =
      sum_partials(partials + (int64_t)kPQPlane * kMaxParts, gridDim.x, &scal->done, &stopped);
  if (stopped) return;
  const bool lead = blockIdx.x == 0 && threadIdx.x == 0;
  if (!(pq > 0.0)) {
    if (lead) scal->done = 3;
    return;
  }
  const double alpha = rho / pq;
  if (lead) {
    scal->pq = pq;
    scal->alpha = alpha;
    scal->rho = rho;
    scal->iter1 = iter + 1;
  }
  const double *__restrict__ p = iter & 1 ? p0 : p1;
  int32_t rb, re;
  rows_of_block(n, chunk, &rb, &re);
  double d[1] = {0.0};
  for (int32_t i = rb + threadIdx.x; i < re; i += kBlock) {
    x[i] += alpha * p[i];
    const double ri = r[i] - alpha * q[i];
    r[i] = ri;
    d[0] += ri * ri;
  }
  block_partial<1>(d, partials + (int64_t)kRRPlane * kMaxParts);
}

// x += alpha p, r -= alpha q with alpha in the scalars, partials of (r, r)
__global__ void __launch_bounds__(kBlock) k_update_dir(int32_t n, int32_t chunk,
                                                       double *__restrict__ x,
                                                       double *__restrict__ r, const double *p0,
                                                       const double *p1,
                                                       const double *__restrict__ q,
                                                       double *__restrict__ partials,
                                                       const PcgScal *__restrict__ scal) {
  if (scal->done) return;
  const double alpha = scal->alpha;
  const double *__restrict__ p = scal->iter & 1 ? p0 : p1;
  int32_t rb, re;
  rows_of_block(n, chunk, &rb, &re);
  double d[1] = {0.0};
  for (int32_t i = rb + threadIdx.x; i < re; i += kBlock) {
    x[i] += alpha * p[i];
    const double ri = r[i] - alpha * q[i];
    r[i] = ri;
    d[0] += ri * ri;
  }
  block_partial<1>(d, partials + (int64_t)kRRPlane * kMaxParts);
}

// ---------------------------------------------------------------------------
// K-cycle: two flexible-CG iterations per intermediate level (Section 3.1)
// ---------------------------------------------------------------------------

// v = A c and the block partials of (c, v) and of (c, u) for each given u
// (plane 0: (c, v); plane q >= 1: (c, u_q)), sums in FP64
template <typename TV, int NV, typename TA = TV>
__global__ void __launch_bounds__(kBlock) k_spmv_dots(
    int32_t n, int32_t chunk, const int32_t *__restrict__ sptr, const int32_t *__restrict__ col,
    const TA *__restrict__ val, const TV *__restrict__ c, TV *__restrict__ v,
    const TV *__restrict__ u1, const TV *__restrict__ u2, double *__restrict__ partials,
    const int32_t *__restrict__ done) {
  if (*done) return;
  int32_t rb, re;
  rows_of_block(n, chunk, &rb, &re);
  double d[NV];
#pragma unroll
  for (int q = 0; q < NV; ++q) d[q] = 0.0;
  for (int32_t row = rb + threadIdx.x; row < re; row += kBlock) {
    int32_t base, w;
    sell_row(sptr, row, &base, &w);
    const TV acc = sell_dot_t<TV, TA>(col, val, base, w, [&](int32_t cc) { return c[cc]; });
    v[row] = acc;
    const double ci = (double)c[row];
    d[0] += ci * (double)acc;
    if (NV > 1) d[1] += ci * (double)u1[row];
    if (NV > 2) d[2] += ci * (double)u2[row];
  }
  block_partial<NV>(d, partials);
}

// The scalars of a level's second flexible-CG step from beta = (c2, v2), gamma =
// (c2, v1) and a2 = (c2, r1) (rho1 and s1 = (c1, b) / rho1 come from the first):
// rho2 = beta - gamma^2 / rho1, s2 = a2 / rho2, a1 = s1 - s2 (gamma / rho1);
// x = a1 c1 + s2 c2. rho1 <= 0 gives x = 0, rho2 <= 0 gives x = s1 c1.
__device__ __forceinline__ void second_step(const double *ks, double beta, double gamma, double a2,
                                            double *a1, double *s2) {
  const double rho1 = ks[kRho1], s1 = ks[kS1];
  *a1 = *s2 = 0.0;
  if (!(rho1 > 0.0)) return;
  const double rho2 = beta - gamma * gamma / rho1;
  *a1 = s1;
  if (!(rho2 > 0.0)) return;
  *s2 = a2 / rho2;
  *a1 = s1 - *s2 * (gamma / rho1);
}

// The sums of N planes of at most 1024 partials by a block of kBlock threads:
// those of sum_partials, with all loads before the first barrier.
template <int N>
__device__ __forceinline__ void sum_planes(const double *__restrict__ partials, int32_t nparts,
                                           double (&out)[N]) {
  constexpr int kRuns = 1024 / kBlock, kWaves = kBlock / kWave;
  __shared__ double wsum[N][kRuns * kWaves];
  const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
  double v[N][kRuns];
#pragma unroll
  for (int q = 0; q < N; ++q)
#pragma unroll
    for (int k = 0; k < kRuns; ++k) {
      const int32_t b = (int32_t)threadIdx.x + k * kBlock;
      v[q][k] = b < nparts ? partials[(int64_t)q * kMaxParts + b] : 0.0;
    }
#pragma unroll
  for (int q = 0; q < N; ++q)
#pragma unroll
    for (int k = 0; k < kRuns; ++k) {
      if (k * kBlock < nparts)
        for (int o = kWave / 2; o > 0; o >>= 1) v[q][k] += __shfl_down(v[q][k], o, kWave);
      if (lane == 0) wsum[q][k * kWaves + wid] = v[q][k];
    }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < N; ++q) {
    out[q] = wsum[q][0];
    for (int k = 1; k < kRuns * kWaves; ++k) out[q] += wsum[q][k];
  }
}

// a1 and s2 of a level: those k_kfin or k_ktail stored, or, with nparts > 0,
// from the partials of the second step, summed here by every block
__device__ __forceinline__ void step_scalars(const double *__restrict__ partials, int32_t nparts,
                                             const double *ks, double *a1, double *s2) {
  if (nparts == 0) {
    *a1 = ks[kA1];
    *s2 = ks[kS2];
    return;
  }
  double t[3];
  sum_planes(partials, nparts, t);
  second_step(ks, t[0], t[1], t[2], a1, s2);
}

// One block: the level's second step from its block partials, where there are
// more of them than kFoldParts
__global__ void __launch_bounds__(1024) k_kfin(int32_t nparts,
                                               const double *__restrict__ partials,
                                               double *__restrict__ ks,
                                               const int32_t *__restrict__ done) {
  const int32_t stop = *done;
  __shared__ double sh[3][1024 / kWave];
  constexpr int nv = 3;
  const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
  for (int q = 0; q < nv; ++q) {
    const double *src = partials + (int64_t)q * kMaxParts;
    double a = 0.0;
    for (int32_t b0 = threadIdx.x; b0 < nparts; b0 += 16 * blockDim.x) {
      double v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int32_t b = b0 + u * (int32_t)blockDim.x;
        v[u] = b < nparts ? src[b] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < 16; ++u)
        if (b0 + u * (int32_t)blockDim.x < nparts) a += v[u];
    }
    for (int o = kWave / 2; o > 0; o >>= 1) a += __shfl_down(a, o, kWave);
    if (lane == 0) sh[q][wid] = a;
  }
  __syncthreads();
  if (threadIdx.x != 0 || stop) return;
  double tot[3] = {0.0, 0.0, 0.0};
  for (int q = 0; q < nv; ++q) {
    double t = sh[q][0];
    for (int k = 1; k < (int)(blockDim.x / kWave); ++k) t += sh[q][k];
    tot[q] = t;
  }
  double a1, s2;
  second_step(ks, tot[0], tot[1], tot[2], &a1, &s2);
  ks[kA1] = a1;
  ks[kS2] = s2;
}

// ---- the deepest flexible-CG step in one block ----
// For the level t just above the coarsest (pre = post = 1), the K-cycle's two
// flexible-CG iterations, each with its cycle (down step, A_L^-1, up step),
// the products and the dot products, in one 1024-thread block with the level's
// vectors in LDS. The prolongation of x = a1 c1 + s2 c2 is left to the post-sweep
// of the level above (k_kpost), or done here where that level has its own (one
// block's 8 rows per thread took 4 us). Same arithmetic as the multi-kernel form; the dot
// products are summed in a fixed order of their own. A chain of latencies: what
// both cycles read is loaded at the start (24.2 -> 20 us at 1000 rows in FP64).
// Against the multi-kernel form a level of 1331 rows over 166 took 974 -> 916 us
// a solve of 22^3, one of 1728 over 216 the same: larger ones gain nothing. Levels
// of more than kKTailAny rows or over more than kKTailAnyCoarse unknowns take it up
// to kKTailEntries stored entries, which one block goes through six times: a random
// graph of 3000 rows, degree 4, 836 for 967 us; of 10000, degree 9, 1994 for 1238.
constexpr int kKTailMax = 2048;   // largest level t in LDS (five vectors)
constexpr int kKTailCoarse = 256; // largest coarsest size
constexpr int kKTailAny = 1536, kKTailAnyCoarse = 128;
constexpr int64_t kKTailEntries = 24576;

// N sums over the block at once; every thread gets them (fixed order)
template <int N>
__device__ __forceinline__ void block_sums(double (&v)[N], double (*red)[1024 / kWave]) {
  const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
  const int nw = blockDim.x / kWave;
#pragma unroll
  for (int q = 0; q < N; ++q)
    for (int o = kWave / 2; o > 0; o >>= 1) v[q] += __shfl_down(v[q], o, kWave);
  __syncthreads();
  if (lane == 0)
#pragma unroll
    for (int q = 0; q < N; ++q) red[q][wid] = v[q];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < N; ++q) {
    v[q] = red[q][0];
    for (int k = 1; k < nw; ++k) v[q] += red[q][k];
  }
}

// One SELL row of the level held in registers (w <= kRowBatch entries):
// loaded once per launch when every thread owns at most one row, then used
// by all six products of the step.
template <typename TV>
struct RegRow {
  int32_t w = 0;
  int32_t c[kRowBatch];
  TV v[kRowBatch], sv[kRowBatch];
  __device__ void load(const int32_t *sptr, const int32_t *col, const TV *val, const TV *sval,
                       int32_t k) {
    const int32_t s = k / kSlice, base = sptr[s] + k % kSlice;
    w = (sptr[s + 1] - sptr[s]) / kSlice;
#pragma unroll
    for (int u = 0; u < kRowBatch; ++u) {
      c[u] = 0;
      v[u] = sv[u] = 0;
      if (u < w) {
        c[u] = col[base + u * kSlice];
        v[u] = val[base + u * kSlice];
        sv[u] = sval[base + u * kSlice];
      }
    }
  }
  // sum_e a_e x[c_e] (scaled: A M^-1) in entry order
  template <bool SCALED>
  __device__ TV dot(const TV *x) const {
    TV acc = 0;
#pragma unroll
    for (int u = 0; u < kRowBatch; ++u)
      if (u < w) acc += (SCALED ? sv[u] : v[u]) * x[c[u]];
    return acc;
  }
};

// What a thread uses in both cycles, loaded once at the start of the launch:
// the segment of its coarse position, its entries of its row of A_L^-1 and,
// with REG, its row of level t.
template <typename TV>
struct KTailRegs {
  RegRow<TV> rr;
  TV mi = 0, p = 0;
  int32_t agg = 0, sb = 0, se = 0;
  double a[kTailRow];  // (n_L <= kTailRow kCoarseSplit)
};

// one K-cycle on level t (iv -> out; the coarse correction is A_L^-1)
template <typename TV, bool REG>
__device__ void ktail_cycle(int32_t nt, const int32_t *__restrict__ sptr,
                            const int32_t *__restrict__ col, const TV *__restrict__ sval,
                            const TV *__restrict__ val, const TV *__restrict__ minv,
                            const TV *__restrict__ pp, const int32_t *__restrict__ aggp, int32_t nL,
                            const double *__restrict__ Ainv, const TV *iv, TV *zs, TV *ys,
                            TV *out, double *rl, double *zl,
                            const KTailRegs<TV> &T) {
  const int32_t tid = threadIdx.x, nth = blockDim.x;
  for (int32_t k = tid; k < nt; k += nth) zs[k] = iv[k] * (REG ? T.mi : minv[k]);
  for (int32_t k = tid; k < nt; k += nth) {
    TV acc;
    if (REG) {
      acc = T.rr.template dot<true>(iv);
    } else {
      const int32_t s = k / kSlice, base = sptr[s] + k % kSlice,
                    w = (sptr[s + 1] - sptr[s]) / kSlice;
      acc = sell_dot(col, sval, base, w, [&](int32_t c) { return iv[c]; });
    }
    ys[k] = (REG ? T.p : pp[k]) * (iv[k] - acc);
  }
  __syncthreads();
  if (tid < nL) {
    TV a = 0;
#pragma unroll 8
    for (int32_t m = T.sb; m < T.se; ++m) a += ys[m];
    rl[tid] = (double)a;
  }
  __syncthreads();
  const int32_t part = tid % kCoarseSplit, irow = tid / kCoarseSplit;
  if (nL <= kTailRow * kCoarseSplit) {
    double a = 0.0;  // (entries past n_L are 0 in both factors)
#pragma unroll
    for (int m = 0; m < kTailRow; ++m) a += T.a[m] * rl[part + m * kCoarseSplit];
    for (int o = kCoarseSplit / 2; o > 0; o >>= 1) a += __shfl_down(a, o, kCoarseSplit);
    if (irow < nL && part == 0) zl[irow] = a;
  } else {
    for (int32_t i = irow; i - irow < nL; i += nth / kCoarseSplit) {
      double a = 0.0;
      if (i < nL) {
        const double *row = Ainv + (int64_t)i * nL;
#pragma unroll 8
        for (int32_t k = part; k < nL; k += kCoarseSplit) a += row[k] * rl[k];
      }
      for (int o = kCoarseSplit / 2; o > 0; o >>= 1) a += __shfl_down(a, o, kCoarseSplit);
      if (i < nL && part == 0) zl[i] = a;
    }
  }
  __syncthreads();
  for (int32_t k = tid; k < nt; k += nth) zs[k] += (REG ? T.p : pp[k]) * (TV)zl[REG ? T.agg : aggp[k]];
  __syncthreads();
  for (int32_t k = tid; k < nt; k += nth) {
    TV acc;
    if (REG) {
      acc = T.rr.template dot<false>(zs);
    } else {
      const int32_t s = k / kSlice, base = sptr[s] + k % kSlice,
                    w = (sptr[s + 1] - sptr[s]) / kSlice;
      acc = sell_dot(col, val, base, w, [&](int32_t c) { return zs[c]; });
    }
    out[k] = zs[k] + (iv[k] - acc) * (REG ? T.mi : minv[k]);
  }
  __syncthreads();
}

template <typename TV, bool REG>
__global__ void __launch_bounds__(1024) k_ktail(
    int32_t nt, const int32_t *__restrict__ sptr, const int32_t *__restrict__ col,
    const TV *__restrict__ sval, const TV *__restrict__ val, const TV *__restrict__ minv,
    const TV *__restrict__ pp, const int32_t *__restrict__ seg, const int32_t *__restrict__ aggp,
    int32_t nL, const double *__restrict__ Ainv, const TV *__restrict__ b, int32_t nf,
    const int32_t *__restrict__ aggp_f, const TV *__restrict__ pp_f, TV *__restrict__ zf,
    TV *__restrict__ c1, TV *__restrict__ c2, double *__restrict__ ks,
    const int32_t *__restrict__ done) {
  __shared__ TV IV[kKTailMax], ZS[kKTailMax], YS[kKTailMax], C1[kKTailMax], C2[kKTailMax];
  __shared__ double rl[kKTailCoarse], zl[kKTailCoarse], red[3][1024 / kWave];
  if (*done) return;
  const int32_t tid = threadIdx.x, nth = blockDim.x;
  constexpr int kRows = kKTailMax / 1024 + 1;  // rows per thread
  // REG: one row per thread (nt <= blockDim.x, rows of at most kRowBatch
  // entries), held in registers for every product of the step
  KTailRegs<TV> T;
  if (REG && tid < nt) {
    T.rr.load(sptr, col, val, sval, tid);
    T.mi = minv[tid];
    T.p = pp[tid];
    T.agg = aggp[tid];
  }
  if (tid < nL) {
    T.sb = seg[tid];
    T.se = seg[tid + 1];
  }
  if (tid < kKTailCoarse) rl[tid] = 0.0;
#pragma unroll
  for (int m = 0; m < kTailRow; ++m) {
    const int32_t i = tid / kCoarseSplit, k = tid % kCoarseSplit + m * kCoarseSplit;
    T.a[m] = nL <= kTailRow * kCoarseSplit && i < nL && k < nL ? Ainv[(int64_t)i * nL + k] : 0.0;
  }
  for (int32_t k = tid; k < nt; k += nth) IV[k] = b[k];
  __syncthreads();
  ktail_cycle<TV, REG>(nt, sptr, col, sval, val, minv, pp, aggp, nL, Ainv, IV, ZS, YS, C1, rl, zl,
                       T);
  // v1 = A c1, rho1 = (c1, v1), s1 = (c1, b) / rho1
  TV v1[kRows];
  double d[2] = {0.0, 0.0};
#pragma unroll
  for (int u = 0; u < kRows; ++u) {
    const int32_t k = tid + u * nth;
    v1[u] = 0;
    if (k < nt) {
      TV acc;
      if (REG) {
        acc = T.rr.template dot<false>(C1);
      } else {
        const int32_t s = k / kSlice, base = sptr[s] + k % kSlice,
                      w = (sptr[s + 1] - sptr[s]) / kSlice;
        acc = sell_dot(col, val, base, w, [&](int32_t c) { return C1[c]; });
      }
      v1[u] = acc;
      d[0] += (double)C1[k] * (double)acc;
      d[1] += (double)C1[k] * (double)IV[k];
    }
  }
  block_sums(d, red);
  const double rho1 = d[0], cb = d[1];
  const double s1 = rho1 > 0.0 ? cb / rho1 : 0.0;
  // r1 = b - s1 v1 (in IV)
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kRows; ++u) {
    const int32_t k = tid + u * nth;
    if (k < nt) IV[k] = IV[k] - (TV)s1 * v1[u];
  }
  __syncthreads();
  ktail_cycle<TV, REG>(nt, sptr, col, sval, val, minv, pp, aggp, nL, Ainv, IV, ZS, YS, C2, rl, zl,
                       T);
  // v2 = A c2; (c2, v2), gamma = (c2, v1), (c2, r1)
  double e[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int u = 0; u < kRows; ++u) {
    const int32_t k = tid + u * nth;
    if (k < nt) {
      TV acc;
      if (REG) {
        acc = T.rr.template dot<false>(C2);
      } else {
        const int32_t s = k / kSlice, base = sptr[s] + k % kSlice,
                      w = (sptr[s + 1] - sptr[s]) / kSlice;
        acc = sell_dot(col, val, base, w, [&](int32_t c) { return C2[c]; });
      }
      const double c2 = (double)C2[k];
      e[0] += c2 * (double)acc;
      e[1] += c2 * (double)v1[u];
      e[2] += c2 * (double)IV[k];
    }
  }
  block_sums(e, red);
  const double beta = e[0], gamma = e[1], a2 = e[2];
  double a1 = 0.0, s2 = 0.0;
  if (rho1 > 0.0) {
    const double rho2 = beta - gamma * gamma / rho1;
    if (!(rho2 > 0.0)) {
      a1 = s1;
    } else {
      s2 = a2 / rho2;
      a1 = s1 - s2 * (gamma / rho1);
    }
  }
  if (tid == 0) {
    ks[kRho1] = rho1;
    ks[kS1] = s1;
    ks[kA1] = a1;
    ks[kS2] = s2;
  }
  if (c1) {  // left to the kernel that smooths the level above
    for (int32_t k = tid; k < nt; k += nth) {
      c1[k] = C1[k];
      c2[k] = C2[k];
    }
    return;
  }
  // z_f += P x, x = a1 c1 + s2 c2
  const TV ta1 = (TV)a1, ts2 = (TV)s2;
  constexpr int kU = 4;  // positions per thread in flight
  int32_t k = tid;
  for (; k + (kU - 1) * nth < nf; k += kU * nth) {
    int32_t J[kU];
    TV p[kU], z[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      J[u] = aggp_f[k + u * nth];
      p[u] = pp_f[k + u * nth];
      z[u] = zf[k + u * nth];
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) zf[k + u * nth] = z[u] + p[u] * (ta1 * C1[J[u]] + ts2 * C2[J[u]]);
  }
  for (; k < nf; k += nth) {
    const int32_t J = aggp_f[k];
    zf[k] += pp_f[k] * (ta1 * C1[J] + ts2 * C2[J]);
  }
}

// ---------------------------------------------------------------------------
// iterative coarsest solver (Section 5): CG with the l1-Jacobi diagonal
// ---------------------------------------------------------------------------

// two sums over the block at once; every thread gets both (fixed order)
__device__ __forceinline__ void block_sum2(double &a, double &b, double (*red)[1024 / kWave]) {
  const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
  const int nw = blockDim.x / kWave;
  for (int o = kWave / 2; o > 0; o >>= 1) {
    a += __shfl_down(a, o, kWave);
    b += __shfl_down(b, o, kWave);
  }
  __syncthreads();
  if (lane == 0) {
    red[0][wid] = a;
    red[1][wid] = b;
  }
  __syncthreads();
  double ta = red[0][0], tb = red[1][0];
  for (int k = 1; k < nw; ++k) {
    ta += red[0][k];
    tb += red[1][k];
  }
  a = ta;
  b = tb;
}

// z_L from A_L z_L = r_L by CG from zero with z = r / m (minv = 1 / m),
// stopped as soon as ||r_k|| < rtol ||r_L|| or after maxit steps. zout (if
// given) receives z_L; then z_f += P z_L over the nf positions of the level
// above (nf = 0: none). One block; thread t owns rows t, t + blockDim.x, ...
// (at most kCgRows), keeps its rows' x, r, q in registers and the search
// direction in LDS for the products; FP64 throughout, A_L in CSR.
constexpr int kCgRows = AMG_MAX_DENSE / 1024;
template <typename TI, typename TO>
__global__ void __launch_bounds__(1024) k_coarse_pcg(
    int32_t nL, const int32_t *__restrict__ rp, const int32_t *__restrict__ ci,
    const double *__restrict__ val, const double *__restrict__ minv, double rtol,
    int32_t maxit, const TI *__restrict__ rL, TO *__restrict__ zout, int32_t nf,
    const int32_t *__restrict__ aggp, const TO *__restrict__ pp, TO *__restrict__ zf,
    const int32_t *__restrict__ done) {
  __shared__ double P[AMG_MAX_DENSE];
  __shared__ double red[2][1024 / kWave];
  if (*done) return;
  const int32_t tid = threadIdx.x, nth = blockDim.x;
  double x[kCgRows], r[kCgRows], q[kCgRows];
  double bb = 0.0, rz0 = 0.0;
#pragma unroll
  for (int u = 0; u < kCgRows; ++u) {
    const int32_t i = tid + u * nth;
    x[u] = r[u] = q[u] = 0.0;
    if (i < nL) {
      r[u] = (double)rL[i];
      const double z = r[u] * minv[i];
      P[i] = z;
      bb += r[u] * r[u];
      rz0 += r[u] * z;
    }
  }
  block_sum2(bb, rz0, red);  // also orders the P writes before the first product
  const double bstop = rtol * sqrt(bb);
  for (int32_t it = 0; bb > 0.0 && it < maxit; ++it) {
    // q = A p and (p, q)
    double pq = 0.0, unused = 0.0;
#pragma unroll
    for (int u = 0; u < kCgRows; ++u) {
      const int32_t i = tid + u * nth;
      if (i < nL) {
        double acc = 0.0;
        for (int32_t k = rp[i]; k < rp[i + 1]; ++k) acc += val[k] * P[ci[k]];
        q[u] = acc;
        pq += P[i] * acc;
      }
    }
    block_sum2(pq, unused, red);
    if (!(pq > 0.0)) break;
    const double step = rz0 / pq;
    // x += step p, r -= step q, then ||r||^2 and (r, z) with z = r / m
    double rr = 0.0, rz1 = 0.0;
    double z[kCgRows];
#pragma unroll
    for (int u = 0; u < kCgRows; ++u) {
      const int32_t i = tid + u * nth;
      z[u] = 0.0;
      if (i < nL) {
        x[u] += step * P[i];
        r[u] -= step * q[u];
        z[u] = r[u] * minv[i];
        rr += r[u] * r[u];
        rz1 += r[u] * z[u];
      }
    }
    block_sum2(rr, rz1, red);  // every thread has read P before any rewrites it
    if (sqrt(rr) < bstop) break;
    const double beta = rz1 / rz0;
    rz0 = rz1;
#pragma unroll
    for (int u = 0; u < kCgRows; ++u) {
      const int32_t i = tid + u * nth;
      if (i < nL) P[i] = z[u] + beta * P[i];
    }
    __syncthreads();
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kCgRows; ++u) {
    const int32_t i = tid + u * nth;
    if (i < nL) {
      P[i] = x[u];
      if (zout) zout[i] = (TO)x[u];
    }
  }
  __syncthreads();
  for (int32_t k = tid; k < nf; k += nth) zf[k] += pp[k] * (TO)P[aggp[k]];
}

// threads of the coarsest CG block: one wavefront per 64 rows, at most 1024
inline int32_t coarse_pcg_threads(int32_t nL) {
  const int32_t t = ceil_div(nL, kWave) * kWave;
  return t < kWave ? kWave : (t > 1024 ? 1024 : t);
}

// r1 = b - s1 v1, with s1 from the first step's partials
template <typename TV>
__global__ void __launch_bounds__(kBlock) k_kresid(int32_t n, KSub<TV> sub, TV *__restrict__ r1,
                                                   const int32_t *__restrict__ done) {
  if (*done) return;
  const TV s1 = (TV)first_step(sub);
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) r1[i] = sub.b[i] - s1 * sub.v1[i];
}

// z_f += P x with x = a1 c1 + s2 c2 formed per coarse position
template <typename TV>
__global__ void __launch_bounds__(kBlock) k_kprolong(
    int32_t nf, const int32_t *__restrict__ aggp, const TV *__restrict__ pp,
    const TV *__restrict__ c1, const TV *__restrict__ c2, const double *__restrict__ partials,
    int32_t nparts, const double *__restrict__ ks, TV *__restrict__ zf,
    const int32_t *__restrict__ done) {
  if (*done) return;
  const int32_t k = blockIdx.x * blockDim.x + threadIdx.x;
  int32_t J = 0;
  TV p = 0, z = 0;
  if (k < nf) {
    J = aggp[k];
    p = pp[k];
    z = zf[k];
  }
  double a1, s2;
  step_scalars(partials, nparts, ks, &a1, &s2);
  if (k < nf) zf[k] = z + p * ((TV)a1 * c1[J] + (TV)s2 * c2[J]);
}

// The up step of the K-cycle in one kernel: y = z' + M^-1 (r - A z') with z' =
// z + P (a1 c1 + s2 c2) formed at each entry of z that is gathered (k_post after
// k_kprolong, without the launch between them)
template <typename TV, typename TR, typename TO, bool DOT>
__global__ void __launch_bounds__(kBlock) k_kpost(
    int32_t n, int32_t chunk, const int32_t *__restrict__ sptr, const int32_t *__restrict__ col,
    const TV *__restrict__ val, const TV *__restrict__ minv, const TR *__restrict__ r,
    const TV *__restrict__ z, const int32_t *__restrict__ aggp, const TV *__restrict__ pp,
    const TV *__restrict__ c1, const TV *__restrict__ c2, double *__restrict__ partials,
    int32_t nparts, const double *__restrict__ ks, TO *__restrict__ y,
    const int32_t *__restrict__ done, const double *__restrict__ dv) {
  if (*done) return;
  double a1, s2;
  step_scalars(partials, DOT ? 0 : nparts, ks, &a1, &s2);  // (with DOT they are written below)
  const TV ta1 = (TV)a1, ts2 = (TV)s2;
  auto zx = [&](int32_t k) {
    const int32_t J = aggp[k];
    return z[k] + pp[k] * (ta1 * c1[J] + ts2 * c2[J]);
  };
  int32_t rb, re;
  rows_of_block(n, chunk, &rb, &re);
  double d[1] = {0.0};
  for (int32_t row = rb + threadIdx.x; row < re; row += kBlock) {
    const TR rr = r[row];
    const TV mr = minv[row], zr = zx(row);
    int32_t base, w;
    sell_row(sptr, row, &base, &w);
    const TV acc = sell_dot_t<TV, TV>(col, val, base, w, zx);
    const TO yo = (TO)(zr + ((TV)rr - acc) * mr);
    y[row] = yo;
    if (DOT) d[0] += (dv ? dv[row] : (double)rr) * (double)yo;
  }
  if (DOT) block_partial<1>(d, partials);
}

// ---------------------------------------------------------------------------
// host: the V-cycle for one hierarchy precision
// ---------------------------------------------------------------------------

template <typename TV>
const TV *vals(const Level &L);
template <>
const double *vals<double>(const Level &L) { return L.S.v64; }
template <>
const float *vals<float>(const Level &L) { return L.S.v32; }
template <typename TV>
const TV *svals(const Level &L);
template <>
const double *svals<double>(const Level &L) { return L.S.s64; }
template <>
const float *svals<float>(const Level &L) { return L.S.s32; }
template <typename TV>
const TV *minv(const Level &L);
template <>
const double *minv<double>(const Level &L) { return L.sminv64; }
template <>
const float *minv<float>(const Level &L) { return L.sminv32; }
template <typename TV>
const TV *ppv(const Level &L);
template <>
const double *ppv<double>(const Level &L) { return L.pp64; }
template <>
const float *ppv<float>(const Level &L) { return L.pp32; }

template <typename TV>
const TV *pbar_vals(const Level &L);
template <>
const double *pbar_vals<double>(const Level &L) { return L.sp_v64; }
template <>
const float *pbar_vals<float>(const Level &L) { return L.sp_v32; }
template <typename TV>
const TV *lr_vals(const Level &L);
template <>
const double *lr_vals<double>(const Level &L) { return L.lr_v64; }
template <>
const float *lr_vals<float>(const Level &L) { return L.lr_v32; }
template <typename TV>
const TV *pbart_vals(const Level &L);
template <>
const double *pbart_vals<double>(const Level &L) { return L.st_v64; }
template <>
const float *pbart_vals<float>(const Level &L) { return L.st_v32; }

// In-solve timing probe. arm_probe(h, id) marks the next launch made through
// launch_k as the timed one when kernel `id` is being timed (never during
// graph capture, whose probe_id is -1); launch_k then launches it with
// hipExtLaunchKernelGGL and the next pair of probe events, which the runtime
// stamps at that dispatch's own start and end (no marker packets around it).
inline void arm_probe(amg_hierarchy *h, int32_t id) { h->probe_armed = h->probe_id == id; }

template <typename K, typename... Args>
void launch_k(const amg_hierarchy *h, K k, dim3 grid, dim3 block, uint32_t shmem, hipStream_t s,
              Args... args) {
  if (h->probe_armed && h->probe_next + 2 <= h->probe_ev.size()) {
    h->probe_armed = false;
    hipEvent_t e0 = h->probe_ev[h->probe_next], e1 = h->probe_ev[h->probe_next + 1];
    h->probe_next += 2;
    hipExtLaunchKernelGGL(k, grid, block, shmem, s, e0, e1, 0, args...);
    return;
  }
  hipLaunchKernelGGL(k, grid, block, shmem, s, args...);
}

// rows per thread of the down step on a level of n rows: 2 on levels of 2^21
// to kManyRows rows (160^3 level 0: 79.4 -> 78.1 us; 4 rows: 83 us; on
// 16.7 M rows 2 rows were slower)
inline int down_rows(int64_t n) { return n >= (1 << 21) && n < kManyRows ? 2 : 1; }

void finalize(amg_hierarchy *h, int32_t op, int32_t nparts, const int32_t *done, int plane = 0) {
  k_finalize<<<1, 1024, 0, h->stream>>>(op, nparts, h->partials + (int64_t)plane * kMaxParts,
                                        h->scal, done);
}

int32_t coarse_per_block(const amg_hierarchy *h) {
  const int32_t g = kBlock / h->max_seg;
  return g < 1 ? 1 : g;
}

// coarse rows per block of the LDS-staged down step (one fine row per thread:
// with its operands loaded ahead of the staging barrier, two rows per thread
// held more registers than they hid latency)
int32_t staged_down_G(const amg_hierarchy *h) { return coarse_per_block(h); }

// whether a level's products take a block per kWideRows rows
bool wide_rows(const amg_hierarchy *h, const Level &L) {
  const int64_t mean = L.n <= kWideMany ? kWideMean : 2 * kWideMean;
  return h->max_seg <= kWideRows && L.S.nnz_padded >= mean * L.n;
}

// whether a K-cycle level's steps may form a vector at every entry they gather
bool short_rows(const Level &L) {
  return L.n <= kUpRows && L.S.nnz_padded <= (int64_t)kUpMean * L.n;
}

// whether the level above the coarsest goes into the one-block step
bool ktail_fits(const Level &T, int32_t nL) {
  return (T.n <= kKTailAny && nL <= kKTailAnyCoarse) ||
         (T.n <= kKTailMax && nL <= kKTailCoarse && T.S.nnz_padded <= kKTailEntries);
}

// Down step of level F into C: LDS-staged gathers where the level has tiles of
// that geometry, else down_rows(n) fine rows per thread gathering from memory.
template <typename TV, typename TR, int MODE, typename TA, bool FIN>
void pre_restrict_fin(const amg_hierarchy *h, const Level &F, const Level &C, const TA *val,
                      const TV *mv, const TV *pp, const TR *r, TV *z, TV *rc,
                      const int32_t *done, const FinRR &fin) {
  hipStream_t s = h->stream;
  const int32_t Gt = staged_down_G(h);
  if (F.hseg.ok() && F.hseg.param == Gt && F.hseg.ntiles == ceil_div(C.n, Gt)) {
    const Halo &H = F.hseg;
    launch_k(h, k_pre_restrict_lds<TV, TR, MODE, TA, 1, FIN>, dim3(ceil_div(C.n, Gt)),
             dim3(kBlock), (uint32_t)(sizeof(TV) * H.umax), s, C.n, Gt, F.seg, F.S.sptr,
             (const uint16_t *)H.lcol, (const int32_t *)H.hptr, (const int32_t *)H.hidx, val, mv,
             pp, r, z, rc, done, fin);
    return;
  }
  if constexpr (MODE == kPreScaled && std::is_same<TR, TV>::value && !FIN)
    if (wide_rows(h, F)) {
      const int32_t Gw = kWideRows / h->max_seg;
      launch_k(h, k_pre_restrict_wide<TV>, dim3(ceil_div(C.n, Gw)), dim3(kBlock), 0u, s, C.n, Gw,
               F.seg, F.S.sptr, F.S.col, val, mv, pp, r, z, rc, done);
      return;
    }
  const int R = down_rows(F.n);
  const int32_t G = coarse_per_block(h) * R;
  const int32_t grid = ceil_div(C.n, G);
  auto k = R == 2 ? k_pre_restrict<TV, TR, MODE, TA, 2, FIN>
                  : k_pre_restrict<TV, TR, MODE, TA, 1, FIN>;
  launch_k(h, k, dim3(grid), dim3(kBlock), 0u, s, C.n, G, F.seg, F.S.sptr, F.S.col, val, mv, pp,
           r, z, rc, done, fin);
}

template <typename TV, typename TR, int MODE, typename TA>
void pre_restrict(const amg_hierarchy *h, const Level &F, const Level &C, const TA *val,
                  const TV *mv, const TV *pp, const TR *r, TV *z, TV *rc, const int32_t *done) {
  // (only level 0's right-hand side is double in both precisions)
  if (MODE != kPreFromZ && h->rr_in_down && &F == &h->lv[0])
    pre_restrict_fin<TV, TR, MODE, TA, MODE != kPreFromZ>(
        h, F, C, val, mv, pp, r, z, rc, done,
        FinRR{h->scal, h->partials + kRRPlane * kMaxParts, geom(F.n).grid});
  else
    pre_restrict_fin<TV, TR, MODE, TA, false>(h, F, C, val, mv, pp, r, z, rc, done, FinRR{});
}

// y = z + M^-1 (r - A z) on a level (DOT: with the block partials of the CG
// dot), with LDS-staged gathers where the level has row tiles
template <typename TV, typename TR, typename TO, bool DOT, typename TA, bool OUT = false>
void post_sweep(const amg_hierarchy *h, const Level &F, const TA *val, const TV *minv,
                const TR *r, const TV *z, TO *y, double *partials, const int32_t *done,
                const double *dv = nullptr) {
  hipStream_t s = h->stream;
  const Geom g = geom(F.n);
  if (F.hrow.ok() && F.hrow.param == g.chunk && F.hrow.ntiles == g.grid) {
    const Halo &H = F.hrow;
    launch_k(h, k_post_lds<TV, TR, TO, DOT, TA, OUT>, dim3(g.grid), dim3(kBlock),
             (uint32_t)(sizeof(TV) * H.umax), s, F.n, g.chunk, F.S.sptr,
             (const uint16_t *)H.lcol, (const int32_t *)H.hptr, (const int32_t *)H.hidx, val,
             minv, r, z, y, partials, done, dv, (const int32_t *)F.perm);
    return;
  }
  launch_k(h, k_post<TV, TR, TO, DOT, TA, OUT>, dim3(g.grid), dim3(kBlock), 0u, s, F.n, g.chunk,
           F.S.sptr, F.S.col, val, minv, r, z, y, partials, done, dv, (const int32_t *)F.perm);
}

// q = A p with the block partials of (p, q) on level 0 (A from its exact FP32
// copy when there is one), with LDS-staged gathers where there are row tiles
inline void spmv_dot0(const amg_hierarchy *h, const double *p, double *q, const int32_t *done) {
  hipStream_t s = h->stream;
  const Level &F = h->lv[0];
  const Geom g = geom(F.n);
  if (F.hrow.ok() && F.hrow.param == g.chunk && F.hrow.ntiles == g.grid) {
    const Halo &H = F.hrow;
    const uint32_t shmem = (uint32_t)(sizeof(double) * H.umax);
    if (F.S.exact32)
      launch_k(h, k_spmv_dot_lds<float>, dim3(g.grid), dim3(kBlock), shmem, s, F.n, g.chunk,
               F.S.sptr, (const uint16_t *)H.lcol, (const int32_t *)H.hptr,
               (const int32_t *)H.hidx, (const float *)F.S.v32, p, q, h->partials, done);
    else
      launch_k(h, k_spmv_dot_lds<double>, dim3(g.grid), dim3(kBlock), shmem, s, F.n, g.chunk,
               F.S.sptr, (const uint16_t *)H.lcol, (const int32_t *)H.hptr,
               (const int32_t *)H.hidx, (const double *)F.S.v64, p, q, h->partials, done);
    return;
  }
  if (F.S.exact32)
    launch_k(h, k_spmv_dot<float>, dim3(g.grid), dim3(kBlock), 0u, s, F.n, g.chunk, F.S.sptr,
             F.S.col, (const float *)F.S.v32, p, q, h->partials, done);
  else
    launch_k(h, k_spmv_dot<double>, dim3(g.grid), dim3(kBlock), 0u, s, F.n, g.chunk, F.S.sptr,
             F.S.col, (const double *)F.S.v64, p, q, h->partials, done);
}

// whether the products of level l read A from its exact FP32 copy: level 0
// of an FP64 hierarchy whose values are all FP32 numbers (same arithmetic)
template <typename TV>
bool reads32(const Level &F, int32_t l) {
  return l == 0 && sizeof(TV) == 8 && F.S.exact32;
}

// whether level F's one-sweep down step forms z = M^-1 r in LDS and reads
// the plain A: an FP64 level with down-step tiles whose values are all FP32
// numbers. With level 0's exact FP32 copy of A that is 4 value bytes per
// entry instead of the 8 of A M^-1; with the copy switched off the same
// arithmetic (so the copy changes no result bit) at 8 bytes. Other operators
// stage r alone and read A M^-1: staging M^-1 r would gather 1 / m as well
// for no saving.
template <typename TV>
bool staged_down(const amg_hierarchy *h, const Level &F, const Level &C) {
  const int32_t G = staged_down_G(h);
  return sizeof(TV) == 8 && F.S.fp32_values && F.hseg.ok() && F.hseg.param == G &&
         F.hseg.ntiles == ceil_div(C.n, G);
}

// the one-sweep down step of level F (z = M^-1 r, residual, restriction)
template <typename TV, typename TR>
void down_one_sweep(const amg_hierarchy *h, const Level &F, const Level &C, const TR *r, TV *z,
                    const int32_t *done) {
  if (staged_down<TV>(h, F, C) && F.S.exact32)
    pre_restrict<TV, TR, kPreStagedZ, float>(h, F, C, F.S.v32, minv<TV>(F), ppv<TV>(F), r, z,
                                             (TV *)C.r, done);
  else if (staged_down<TV>(h, F, C))
    pre_restrict<TV, TR, kPreStagedZ, TV>(h, F, C, vals<TV>(F), minv<TV>(F), ppv<TV>(F), r, z,
                                          (TV *)C.r, done);
  else
    pre_restrict<TV, TR, kPreScaled, TV>(h, F, C, svals<TV>(F), minv<TV>(F), ppv<TV>(F), r, z,
                                         (TV *)C.r, done);
}

// down step on level l: smoothing from zero, residual, restriction into
// level l + 1's right-hand side; returns the buffer holding z_l
template <typename TV, typename TR>
TV *launch_down(amg_hierarchy *h, int32_t l, const TR *r, const int32_t *done) {
  hipStream_t s = h->stream;
  Level &F = h->lv[l];
  Level &C = h->lv[l + 1];
  TV *z = (TV *)F.z, *tmp = (TV *)F.y;
  if (h->params.pre == 1) {
    down_one_sweep<TV, TR>(h, F, C, r, z, done);
    return z;
  }
  const Geom g = geom(F.n);
  const bool a32 = reads32<TV>(F, l);
  k_jacobi0<TV, TR><<<grid1(F.n), kBlock, 0, s>>>(F.n, minv<TV>(F), r, z, done);
  for (int32_t k = 1; k < h->params.pre; ++k) {
    if (a32)
      k_post<TV, TR, TV, false, float><<<g.grid, kBlock, 0, s>>>(
          F.n, g.chunk, F.S.sptr, F.S.col, F.S.v32, minv<TV>(F), r, z, tmp, nullptr, done);
    else
      k_post<TV, TR, TV, false><<<g.grid, kBlock, 0, s>>>(F.n, g.chunk, F.S.sptr, F.S.col,
                                                         vals<TV>(F), minv<TV>(F), r, z, tmp,
                                                         nullptr, done);
    std::swap(z, tmp);
  }
  if (a32)
    pre_restrict<TV, TR, kPreFromZ, float>(h, F, C, F.S.v32, minv<TV>(F), ppv<TV>(F), r, z,
                                           (TV *)C.r, done);
  else
    pre_restrict<TV, TR, kPreFromZ, TV>(h, F, C, vals<TV>(F), minv<TV>(F), ppv<TV>(F), r, z,
                                        (TV *)C.r, done);
  return z;
}

// A_L^-1 r_L and its prolongation into the z of the level above, F
template <typename TV>
void launch_coarse_prolong(amg_hierarchy *h, const Level &F, TV *z, const int32_t *done) {
  hipStream_t s = h->stream;
  const Level &C = h->lv.back();
  const int32_t nL = h->C.n;
  if (nL <= kCoarseOne) {
    k_coarse_prolong<TV><<<1, 1024, 2 * sizeof(double) * nL, s>>>(
        nL, h->C.Ainv, (const TV *)C.r, F.n, F.aggp, ppv<TV>(F), z, done);
    return;
  }
  k_coarse_rows<TV><<<ceil_div((int64_t)nL * kCoarseSplit, kBlock), kBlock, 0, s>>>(
      nL, h->C.Ainv, (const TV *)C.r, (TV *)C.z, done);
  k_prolong<TV><<<ceil_div(F.n, 4 * kBlock), kBlock, 0, s>>>(F.n, F.aggp, ppv<TV>(F),
                                                           (const TV *)C.z, z, done);
}

// up step on coarse level c >= 1: extra post sweeps, then the last sweep
// fused with the prolongation into the finer level's z (zf)
template <typename TV>
void launch_up(amg_hierarchy *h, int32_t c, TV *zc, TV *zf, const int32_t *done) {
  hipStream_t s = h->stream;
  Level &C = h->lv[c];
  Level &F = h->lv[c - 1];
  TV *tmp = (TV *)C.y;
  if (tmp == zc) tmp = (TV *)C.z;
  const Geom g = geom(C.n);
  for (int32_t k = 1; k < h->params.post; ++k) {
    k_post<TV, TV, TV, false><<<g.grid, kBlock, 0, s>>>(C.n, g.chunk, C.S.sptr, C.S.col,
                                                       vals<TV>(C), minv<TV>(C), (const TV *)C.r,
                                                       zc, tmp, nullptr, done);
    std::swap(zc, tmp);
  }
  if (wide_rows(h, C))
    k_post_prolong_wide<TV><<<ceil_div(C.n, kWideRows), kBlock, 0, s>>>(
        C.n, C.S.sptr, C.S.col, vals<TV>(C), minv<TV>(C), (const TV *)C.r, zc, F.seg, F.aggp,
        ppv<TV>(F), zf, done);
  else
    k_post_prolong<TV><<<grid1(C.n), kBlock, 0, s>>>(C.n, C.S.sptr, C.S.col, vals<TV>(C),
                                                     minv<TV>(C), (const TV *)C.r, zc, F.seg,
                                                     F.aggp, ppv<TV>(F), zf, done);
}

inline bool coarse_is_pcg(const amg_hierarchy *h) {
  return h->params.coarse_solver == AMG_COARSE_PCG;
}

// The coarsest solve by CG (coarse_is_pcg): z_L into zout and/or
// prolongated into zf (nf positions of the level above).
template <typename TI, typename TO>
void launch_coarse_pcg(amg_hierarchy *h, const TI *rL, TO *zout, int32_t nf,
                       const int32_t *aggp, const TO *pp, TO *zf, const int32_t *done) {
  const Level &C = h->lv.back();
  k_coarse_pcg<TI, TO><<<1, coarse_pcg_threads(C.n), 0, h->stream>>>(
      C.n, C.rp, C.ci, C.val, C.minv64, h->params.coarse_rtol, h->params.coarse_maxit, rL, zout,
      nf, aggp, pp, zf, done);
}

// z0 = coarsest solve of r0 when level 0 is the coarsest level; with dot,
// the partials of (dv, z0) (dv = NULL: of (r0, z0), finalized into rho)
void one_level_cycle(amg_hierarchy *h, const double *r0, double *z0, bool dot, const double *dv,
                     const int32_t *done) {
  hipStream_t s = h->stream;
  const int32_t n = h->C.n;
  if (coarse_is_pcg(h))
    launch_coarse_pcg<double, double>(h, r0, z0, 0, nullptr, nullptr, nullptr, done);
  else
    k_coarse_solve<double, double><<<ceil_div(n, kCoarseWaves), kWave * kCoarseWaves, 0, s>>>(
        n, h->C.Ainv, r0, z0, done);
  if (dot) {
    const Geom g = geom(h->lv[0].n);
    k_dot_rz<<<g.grid, kBlock, 0, s>>>(h->lv[0].n, g.chunk, dv ? dv : r0, z0, h->partials, done);
    if (!dv) finalize(h, kFinRZ, g.grid, done);
  }
}

// Level 0 after the coarse correction (z holds it): post - 1 extra sweeps,
// then the last into z0, with dot the block partials of (r0, z0) finalized
// into the CG scalars, or of (dv, z0) left to the caller.
template <typename TV>
void level0_post(amg_hierarchy *h, const double *r0, TV *z, double *z0, bool dot,
                 const double *dv, const int32_t *done) {
  hipStream_t s = h->stream;
  Level &F = h->lv[0];
  TV *tmp = (TV *)F.y;
  if (tmp == z) tmp = (TV *)F.z;
  const Geom g = geom(F.n);
  // an FP64 hierarchy reads A from its exact FP32 copy when there is one
  const bool a32 = reads32<TV>(F, 0);
  for (int32_t k = 1; k < h->params.post; ++k) {
    if (a32)
      post_sweep<TV, double, TV, false, float>(h, F, F.S.v32, minv<TV>(F), r0, z, tmp, nullptr,
                                               done);
    else
      post_sweep<TV, double, TV, false, TV>(h, F, vals<TV>(F), minv<TV>(F), r0, z, tmp, nullptr,
                                            done);
    std::swap(z, tmp);
  }
  if (dot) {
    arm_probe(h, 1);
    if (a32)
      post_sweep<TV, double, double, true, float>(h, F, F.S.v32, minv<TV>(F), r0, z, z0,
                                                  h->partials, done, dv);
    else
      post_sweep<TV, double, double, true, TV>(h, F, vals<TV>(F), minv<TV>(F), r0, z, z0,
                                               h->partials, done, dv);
    h->probe_armed = false;
    if (!dv && !h->fold) finalize(h, kFinRZ, g.grid, done);
  } else if (h->z_out) {
    if (a32)
      post_sweep<TV, double, double, false, float, true>(h, F, F.S.v32, minv<TV>(F), r0, z,
                                                         h->z_out, nullptr, done);
    else
      post_sweep<TV, double, double, false, TV, true>(h, F, vals<TV>(F), minv<TV>(F), r0, z,
                                                      h->z_out, nullptr, done);
  } else {
    if (a32)
      post_sweep<TV, double, double, false, float>(h, F, F.S.v32, minv<TV>(F), r0, z, z0,
                                                   nullptr, done);
    else
      post_sweep<TV, double, double, false, TV>(h, F, vals<TV>(F), minv<TV>(F), r0, z, z0,
                                                nullptr, done);
  }
}

// Down step of the smoothed-aggregation cycle on level l: z from the
// pre-smoothing sweeps and the residual t = r - A z (both left in the level's
// buffers); returns the buffer holding z.
template <typename TV, typename TR>
TV *down_sa(amg_hierarchy *h, int32_t l, const TR *r, const int32_t *done) {
  hipStream_t s = h->stream;
  Level &F = h->lv[l];
  TV *z = (TV *)F.z, *y = (TV *)F.y, *t = (TV *)F.t;
  const Geom g = geom(F.n);
  if (F.lr_rp) {  // long rows: several lanes per row
    k_jacobi0<TV, TR><<<grid1(F.n), kBlock, 0, s>>>(F.n, minv<TV>(F), r, z, done);
    for (int32_t k = 1; k < h->params.pre; ++k) {
      smooth_rows<TV, TR, 0>(s, F.n, F.nnz, F.lr_rp, F.lr_ci, lr_vals<TV>(F), minv<TV>(F), r, z,
                             y, done);
      std::swap(z, y);
    }
    smooth_rows<TV, TR, 1>(s, F.n, F.nnz, F.lr_rp, F.lr_ci, lr_vals<TV>(F), minv<TV>(F), r, z, t,
                           done);
    return z;
  }
  if (h->params.pre == 1) {
    k_pre_resid<TV, TR><<<g.grid, kBlock, 0, s>>>(F.n, g.chunk, F.S.sptr, F.S.col, svals<TV>(F),
                                                  minv<TV>(F), r, z, t, done);
    return z;
  }
  const bool a32 = reads32<TV>(F, l);
  k_jacobi0<TV, TR><<<grid1(F.n), kBlock, 0, s>>>(F.n, minv<TV>(F), r, z, done);
  for (int32_t k = 1; k < h->params.pre; ++k) {
    if (a32)
      k_post<TV, TR, TV, false, float><<<g.grid, kBlock, 0, s>>>(
          F.n, g.chunk, F.S.sptr, F.S.col, F.S.v32, minv<TV>(F), r, z, y, nullptr, done);
    else
      k_post<TV, TR, TV, false><<<g.grid, kBlock, 0, s>>>(F.n, g.chunk, F.S.sptr, F.S.col,
                                                         vals<TV>(F), minv<TV>(F), r, z, y,
                                                         nullptr, done);
    std::swap(z, y);
  }
  if (a32)
    k_resid<TV, TR, float><<<g.grid, kBlock, 0, s>>>(F.n, g.chunk, F.S.sptr, F.S.col, F.S.v32, r,
                                                     z, t, done);
  else
    k_resid<TV, TR><<<g.grid, kBlock, 0, s>>>(F.n, g.chunk, F.S.sptr, F.S.col, vals<TV>(F), r, z,
                                              t, done);
  return z;
}

// The V-cycle with smoothed prolongators (L >= 1): per level the down step,
// r_{l+1} = Pbar^T t; the coarsest solve; then per level z_l += Pbar z_{l+1}
// and the post-smoothing sweeps.
template <typename TV>
void vcycle_sa_t(amg_hierarchy *h, const double *r0, double *z0, bool dot, const double *dv,
                 const int32_t *done) {
  hipStream_t s = h->stream;
  const int32_t L = (int32_t)h->lv.size() - 1;
  std::vector<TV *> zb(L);
  for (int32_t l = 0; l < L; ++l) {
    Level &F = h->lv[l];
    Level &C = h->lv[l + 1];
    zb[l] = l == 0 ? down_sa<TV, double>(h, 0, r0, done)
                   : down_sa<TV, TV>(h, l, (const TV *)F.r, done);
    csr_apply<TV, false>(s, C.n, F.pb_nnz, F.st_rp, F.st_ci, pbart_vals<TV>(F), (const TV *)F.t,
                         (TV *)C.r, done);
  }
  Level &Cl = h->lv[L];
  TV *zc = (TV *)Cl.z;
  const int32_t nL = h->C.n;
  if (coarse_is_pcg(h))
    launch_coarse_pcg<TV, TV>(h, (const TV *)Cl.r, zc, 0, nullptr, nullptr, nullptr, done);
  else
    k_coarse_solve<TV, TV><<<ceil_div(nL, kCoarseWaves), kWave * kCoarseWaves, 0, s>>>(
        nL, h->C.Ainv, (const TV *)Cl.r, zc, done);
  for (int32_t l = L - 1; l >= 1; --l) {
    Level &F = h->lv[l];
    csr_apply<TV, true>(s, F.n, F.pb_nnz, F.sp_rp, F.sp_ci, pbar_vals<TV>(F), zc, zb[l], done);
    TV *z = zb[l], *tmp = z == (TV *)F.z ? (TV *)F.y : (TV *)F.z;
    const Geom g = geom(F.n);
    for (int32_t k = 0; k < h->params.post; ++k) {
      if (F.lr_rp)
        smooth_rows<TV, TV, 0>(s, F.n, F.nnz, F.lr_rp, F.lr_ci, lr_vals<TV>(F), minv<TV>(F),
                               (const TV *)F.r, z, tmp, done);
      else
        k_post<TV, TV, TV, false><<<g.grid, kBlock, 0, s>>>(F.n, g.chunk, F.S.sptr, F.S.col,
                                                           vals<TV>(F), minv<TV>(F),
                                                           (const TV *)F.r, z, tmp, nullptr,
                                                           done);
      std::swap(z, tmp);
    }
    zc = z;
  }
  Level &F0 = h->lv[0];
  csr_apply<TV, true>(s, F0.n, F0.pb_nnz, F0.sp_rp, F0.sp_ci, pbar_vals<TV>(F0), zc, zb[0],
                      done);
  level0_post<TV>(h, r0, zb[0], z0, dot, dv, done);
}

// V-cycle z0 = B r0 on the aggregate-major vectors of level 0. With dot, the
// last kernel also writes the block partials of (r0, z0), finalized into the
// CG scalars, or, with a dot partner dv, of (dv, z0), left to the caller.
template <typename TV>
void vcycle_t(amg_hierarchy *h, const double *r0, double *z0, bool dot, const double *dv,
              const int32_t *done) {
  hipStream_t s = h->stream;
  const int32_t L = (int32_t)h->lv.size() - 1;
  if (L == 0) {
    one_level_cycle(h, r0, z0, dot, dv, done);
    return;
  }
  if (h->params.smooth_p) {
    vcycle_sa_t<TV>(h, r0, z0, dot, dv, done);
    return;
  }
  std::vector<TV *> zb(L);
  const bool tail = L >= 2 && h->params.pre == 1 && h->params.post == 1 &&
                    h->lv[L - 1].n <= kTailMax && h->C.n <= kTailCoarseMax && !coarse_is_pcg(h) &&
                    !wide_rows(h, h->lv[L - 1]);
  const int32_t down_end = tail ? L - 1 : L;  // levels [0, down_end) take the down step
  arm_probe(h, 0);
  zb[0] = launch_down<TV, double>(h, 0, r0, done);
  h->probe_armed = false;
  for (int32_t l = 1; l < down_end; ++l)
    zb[l] = launch_down<TV, TV>(h, l, (const TV *)h->lv[l].r, done);
  if (tail) {
    Level &T = h->lv[L - 1];
    Level &F = h->lv[L - 2];
    k_tail<TV><<<1, 1024, 0, s>>>(T.n, T.S.sptr, T.S.col, svals<TV>(T), vals<TV>(T), minv<TV>(T),
                                  (const TV *)T.r, T.seg, T.aggp, ppv<TV>(T), h->C.n, h->C.Ainv,
                                  F.n, F.aggp, ppv<TV>(F), zb[L - 2], done);
    for (int32_t c = L - 2; c >= 1; --c) launch_up<TV>(h, c, zb[c], zb[c - 1], done);
  } else {
    Level &F = h->lv[L - 1];
    if (coarse_is_pcg(h))
      launch_coarse_pcg<TV, TV>(h, (const TV *)h->lv[L].r, nullptr, F.n, F.aggp, ppv<TV>(F),
                                zb[L - 1], done);
    else
      launch_coarse_prolong<TV>(h, F, zb[L - 1], done);
    for (int32_t c = L - 1; c >= 1; --c) launch_up<TV>(h, c, zb[c], zb[c - 1], done);
  }
  level0_post<TV>(h, r0, zb[0], z0, dot, dv, done);
}

// ---- K-cycle (Section 3.1) ----

template <typename TV>
int32_t fcg2_t(amg_hierarchy *h, int32_t m, const int32_t *done);

// K-cycle on level l < L. in: the level's right-hand side (level 0: the FP64
// CG residual); out: the result (level 0: FP64). With a dot partner dv the
// last post-sweep also writes the block partials of (dv, out). zdown: the level's
// z where its down step has been done.
template <typename TV, typename TR, typename TO>
void kcycle_t(amg_hierarchy *h, int32_t l, const TR *in, TO *out, const double *dv,
              const int32_t *done, TV *zdown = nullptr) {
  hipStream_t s = h->stream;
  const int32_t L = (int32_t)h->lv.size() - 1;
  Level &F = h->lv[l];
  TV *z = zdown ? zdown : launch_down<TV, TR>(h, l, in, done);
  const Geom g = geom(F.n);
  const bool a32 = reads32<TV>(F, l);
  double *ks = h->kscal + (int64_t)(l + 1) * kKScal;
  // the prolongation in the one post-sweep
  const bool up = l > 0 && h->params.post == 1 && short_rows(F);
  auto kpost = [&](int32_t nparts) {
    const Level &C = h->lv[l + 1];
    if constexpr (std::is_same<TR, TV>::value && std::is_same<TO, TV>::value)
      if (!dv) {
        k_kpost<TV, TR, TO, false><<<g.grid, kBlock, 0, s>>>(
            F.n, g.chunk, F.S.sptr, F.S.col, vals<TV>(F), minv<TV>(F), in, z, F.aggp, ppv<TV>(F),
            (const TV *)C.c1, (const TV *)C.c2, h->partials, nparts, ks, out, done, nullptr);
      }
  };
  if (l + 1 == L) {
    if (coarse_is_pcg(h))
      launch_coarse_pcg<TV, TV>(h, (const TV *)h->lv[L].r, nullptr, F.n, F.aggp, ppv<TV>(F), z,
                                done);
    else
      launch_coarse_prolong<TV>(h, F, z, done);
  } else if (l + 2 == L && h->params.pre == 1 && h->params.post == 1 &&
             ktail_fits(h->lv[l + 1], h->C.n) && !coarse_is_pcg(h)) {
    const Level &T = h->lv[l + 1];
    auto kt = T.n <= 1024 && T.S.max_width <= kRowBatch ? k_ktail<TV, true> : k_ktail<TV, false>;
    kt<<<1, 1024, 0, s>>>(T.n, T.S.sptr, T.S.col, svals<TV>(T), vals<TV>(T), minv<TV>(T),
                          ppv<TV>(T), T.seg, T.aggp, h->C.n, h->C.Ainv, (const TV *)T.r, F.n,
                          F.aggp, ppv<TV>(F), z, up ? (TV *)T.c1 : nullptr,
                          up ? (TV *)T.c2 : nullptr, ks, done);
    if (up) {
      kpost(0);
      return;
    }
  } else {
    const Level &C = h->lv[l + 1];
    const int32_t nparts = fcg2_t<TV>(h, l + 1, done);
    if (up) {
      kpost(nparts);
      return;
    }
    k_kprolong<TV><<<grid1(F.n), kBlock, 0, s>>>(F.n, F.aggp, ppv<TV>(F), (const TV *)C.c1,
                                                 (const TV *)C.c2, h->partials, nparts, ks, z,
                                                 done);
  }
  // post-smoothing: post - 1 sweeps alternating two level buffers, the last
  // into out
  TV *tmp = (TV *)F.y;
  if (tmp == z) tmp = (TV *)F.z;
  for (int32_t k = 1; k < h->params.post; ++k) {
    if (a32)
      k_post<TV, TR, TV, false, float><<<g.grid, kBlock, 0, s>>>(
          F.n, g.chunk, F.S.sptr, F.S.col, F.S.v32, minv<TV>(F), in, z, tmp, nullptr, done);
    else
      k_post<TV, TR, TV, false><<<g.grid, kBlock, 0, s>>>(F.n, g.chunk, F.S.sptr, F.S.col,
                                                         vals<TV>(F), minv<TV>(F), in, z, tmp,
                                                         nullptr, done);
    std::swap(z, tmp);
  }
  if (dv && a32)
    k_post<TV, TR, TO, true, float><<<g.grid, kBlock, 0, s>>>(
        F.n, g.chunk, F.S.sptr, F.S.col, F.S.v32, minv<TV>(F), in, z, out, h->partials, done, dv);
  else if (dv)
    k_post<TV, TR, TO, true><<<g.grid, kBlock, 0, s>>>(F.n, g.chunk, F.S.sptr, F.S.col,
                                                      vals<TV>(F), minv<TV>(F), in, z, out,
                                                      h->partials, done, dv);
  else if (a32)
    k_post<TV, TR, TO, false, float><<<g.grid, kBlock, 0, s>>>(
        F.n, g.chunk, F.S.sptr, F.S.col, F.S.v32, minv<TV>(F), in, z, out, nullptr, done);
  else
    k_post<TV, TR, TO, false><<<g.grid, kBlock, 0, s>>>(F.n, g.chunk, F.S.sptr, F.S.col,
                                                       vals<TV>(F), minv<TV>(F), in, z, out,
                                                       nullptr, done);
}

// Two flexible-CG iterations on level m (0 < m < L) for the right-hand side
// the level above restricted into lv[m].r, from zero; the result stays as
// x = a1 c1 + s2 c2 (vectors c1, c2 of the level) for the prolongation to
// combine: scalars in the level's kscal slot, or, where a number of partials
// is returned, to be summed from them.
template <typename TV>
int32_t fcg2_t(amg_hierarchy *h, int32_t m, const int32_t *done) {
  hipStream_t s = h->stream;
  Level &M = h->lv[m];
  const int32_t n = M.n;
  const TV *b = (const TV *)M.r;
  double *ks = h->kscal + (int64_t)m * kKScal;
  const Geom g = geom(n);
  kcycle_t<TV, TV, TV>(h, m, b, (TV *)M.c1, nullptr, done);
  k_spmv_dots<TV, 2><<<g.grid, kBlock, 0, s>>>(n, g.chunk, M.S.sptr, M.S.col, vals<TV>(M),
                                               (const TV *)M.c1, (TV *)M.v1, b, nullptr,
                                               h->partials, done);
  const KSub<TV> sub{b, (const TV *)M.v1, h->partials, g.grid, ks};
  TV *z1 = nullptr;  // of the second cycle, where its down step is done here
  if (h->params.pre == 1 && short_rows(M) && !M.hseg.ok()) {
    const Level &C = h->lv[m + 1];
    const int32_t G = coarse_per_block(h);
    z1 = (TV *)M.z;
    k_kdown<TV><<<ceil_div(C.n, G), kBlock, 0, s>>>(C.n, G, M.seg, M.S.sptr, M.S.col, svals<TV>(M),
                                                    minv<TV>(M), ppv<TV>(M), sub, (TV *)M.r1, z1,
                                                    (TV *)C.r, done);
  } else {
    k_kresid<TV><<<grid1(n), kBlock, 0, s>>>(n, sub, (TV *)M.r1, done);
  }
  kcycle_t<TV, TV, TV>(h, m, (const TV *)M.r1, (TV *)M.c2, nullptr, done, z1);
  k_spmv_dots<TV, 3><<<g.grid, kBlock, 0, s>>>(n, g.chunk, M.S.sptr, M.S.col, vals<TV>(M),
                                               (const TV *)M.c2, (TV *)M.v2,
                                               (const TV *)M.v1, (const TV *)M.r1,
                                               h->partials, done);
  if (g.grid <= kFoldParts) return g.grid;
  k_kfin<<<1, 1024, 0, s>>>(g.grid, h->partials, ks, done);
  return 0;
}

// z0 = K r0 on the aggregate-major level-0 vectors (with dv: the partials of
// (dv, z0) as well)
template <typename TV>
void kcycle_top(amg_hierarchy *h, const double *r0, double *z0, const double *dv,
                const int32_t *done) {
  const int32_t L = (int32_t)h->lv.size() - 1;
  if (L == 0) {
    if (dv) one_level_cycle(h, r0, z0, true, dv, done);
    else one_level_cycle(h, r0, z0, false, nullptr, done);
    return;
  }
  kcycle_t<TV, double, double>(h, 0, r0, z0, dv, done);
}

amg_status alloc_level_vectors(amg_hierarchy *h, Level &L, size_t vbytes) {
  AMG_TRY(dev_alloc(h, &L.r, vbytes * L.n + 16));
  AMG_TRY(dev_alloc(h, &L.z, vbytes * L.n + 16));
  AMG_TRY(dev_alloc(h, &L.t, vbytes * L.n + 16));
  AMG_TRY(dev_alloc(h, &L.y, vbytes * L.n + 16));
  return AMG_OK;
}

}  // namespace

// ---- LDS-staged gathers: tile lists (setup) ----

constexpr int kHaloCap = 8192;        // padded entries of one tile sorted in LDS
constexpr int32_t kHaloMaxList = 4096;  // longest list a level may have (LDS of a block)

__global__ void k_tile_starts(int32_t ntiles, int32_t step, int32_t nmax,
                              const int32_t *__restrict__ seg, int32_t *__restrict__ tb) {
  const int32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t > ntiles) return;
  const int64_t v = (int64_t)t * step;
  const int32_t c = (int32_t)(v < nmax ? v : nmax);
  tb[t] = seg ? seg[c] : c;  // row chunks, or the first row of coarse row c
}

// Tile t = rows [tb[t], tb[t + 1]). Its list is the sorted distinct columns
// of its SELL positions (W per row, W the widest slice among its rows; at
// most CAP positions, else count[t] = -1 and no list): the columns below
// the tile's own rows, then the own rows themselves (every row holds its
// diagonal), then the columns above. Only the columns outside the own rows
// are sorted (bitonic, in LDS) and made distinct; an own row's index in the
// list follows from its offset. Pass 0 writes the list length to count[t];
// pass 1 writes the list at hidx + hptr[t] and, at every position, the index
// of its column in the list. What bounds it is the barriers of the sort, so a
// tile takes a block of no more threads than its columns need: 256 for the
// down step's tiles of 256 rows (0.52 and 0.64 ms a pass with 1024 at 160^3).
template <int NT, int CAP>
__global__ void __launch_bounds__(NT) k_halo(
    int32_t pass, const int32_t *__restrict__ tb, const int32_t *__restrict__ sptr,
    const int32_t *__restrict__ col, int32_t *__restrict__ count,
    const int32_t *__restrict__ hptr, int32_t *__restrict__ hidx, uint16_t *__restrict__ lcol) {
  __shared__ int32_t keys[CAP];
  __shared__ int32_t part[NT];
  __shared__ int32_t wmax, nout;
  const int32_t t = blockIdx.x, tid = threadIdx.x;
  constexpr int32_t nt = NT;
  const int32_t r0 = tb[t], r1 = tb[t + 1], rows = r1 - r0;
  if (tid == 0) {
    wmax = 0;
    nout = 0;
  }
  __syncthreads();
  if (rows > 0) {
    int32_t wl = 0;
    for (int32_t q = r0 / kSlice + tid; q <= (r1 - 1) / kSlice; q += nt)
      wl = max(wl, (sptr[q + 1] - sptr[q]) / kSlice);
    atomicMax(&wmax, wl);
  }
  __syncthreads();
  const int32_t W = wmax;
  const int64_t E = (int64_t)rows * W;
  if (E > CAP) {
    if (pass == 0 && tid == 0) count[t] = -1;
    return;
  }
  // the columns outside [r0, r1), in any order
  for (int32_t i = tid; i < E; i += nt) {
    int32_t base, w;
    sell_row(sptr, r0 + i / W, &base, &w);
    if (i % W < w) {
      const int32_t c = col[base + (i % W) * kSlice];
      if (c < r0 || c >= r1) keys[atomicAdd(&nout, 1)] = c;
    }
  }
  __syncthreads();
  const int32_t no = nout;
  int32_t P = 1;
  while (P < no) P <<= 1;
  for (int32_t i = no + tid; i < P; i += nt) keys[i] = INT32_MAX;
  __syncthreads();
  for (int32_t size = 2; size <= P; size <<= 1)  // bitonic sort, ascending
    for (int32_t stride = size >> 1; stride > 0; stride >>= 1) {
      for (int32_t i = tid; i < P; i += nt) {
        const int32_t j = i ^ stride;
        if (j > i) {
          const int32_t a = keys[i], b = keys[j];
          if ((a > b) == ((i & size) == 0)) {
            keys[i] = b;
            keys[j] = a;
          }
        }
      }
      __syncthreads();
    }
  // distinct keys: thread tid takes positions [tid * per, tid * per + per)
  const int32_t per = (P + nt - 1) / nt;  // at most CAP / NT
  int32_t kv[CAP / NT];
  uint32_t first = 0;
  int32_t mine = 0;
  for (int32_t q = 0; q < per; ++q) {
    const int32_t i = tid * per + q;
    kv[q] = i < P ? keys[i] : INT32_MAX;
    if (i < P && kv[q] != INT32_MAX && (i == 0 || keys[i - 1] != kv[q])) {
      first |= 1u << q;
      ++mine;
    }
  }
  part[tid] = mine;
  __syncthreads();
  for (int32_t off = 1; off < nt; off <<= 1) {  // inclusive scan of the counts
    const int32_t add = tid >= off ? part[tid - off] : 0;
    __syncthreads();
    part[tid] += add;
    __syncthreads();
  }
  const int32_t uo = part[nt - 1];
  int32_t pos = part[tid] - mine;
  for (int32_t q = 0; q < per; ++q)  // every key was read before the scan
    if (first & (1u << q)) keys[pos++] = kv[q];
  __syncthreads();
  if (pass == 0) {
    if (tid == 0) count[t] = uo + rows;
    return;
  }
  // nb = distinct outside columns below r0 (they precede the own rows)
  int32_t lo = 0, hi = uo;
  while (lo < hi) {
    const int32_t mid = (lo + hi) >> 1;
    if (keys[mid] < r0) lo = mid + 1;
    else hi = mid;
  }
  const int32_t nb = lo;
  const int32_t h0 = hptr[t];
  for (int32_t j = tid; j < uo + rows; j += nt)
    hidx[h0 + j] = j < nb ? keys[j] : (j < nb + rows ? r0 + (j - nb) : keys[j - rows]);
  for (int64_t i = tid; i < E; i += nt) {
    int32_t base, w;
    sell_row(sptr, r0 + (int32_t)(i / W), &base, &w);
    const int32_t k = (int32_t)(i % W);
    if (k >= w) continue;
    const int32_t idx = base + k * kSlice;
    const int32_t c = col[idx];
    int32_t at;
    if (c >= r0 && c < r1) {
      at = nb + (c - r0);
    } else {
      int32_t a = 0, b = uo - 1;  // c is in the list
      while (a < b) {
        const int32_t mid = (a + b) >> 1;
        if (keys[mid] < c) a = mid + 1;
        else b = mid;
      }
      at = a < nb ? a : a + rows;
    }
    lcol[idx] = (uint16_t)at;
  }
}

// A tiling in the making: `ntiles` tiles starting at tb (device, ntiles + 1
// entries) of at most `rows` rows, their list lengths in count.
struct Tiling {
  int32_t ntiles = 0, param = 0;
  int64_t rows = 0;
  int32_t *tb = nullptr, *count = nullptr;
  std::vector<int32_t> hc;
};

void launch_halo(amg_hierarchy *h, const Level &L, const Tiling &T, int32_t pass,
                 const Halo &H) {
  hipStream_t s = h->stream;
  if (T.rows * L.S.max_width <= 2048)
    k_halo<256, 2048><<<T.ntiles, 256, 0, s>>>(pass, T.tb, L.S.sptr, L.S.col, T.count, H.hptr,
                                               H.hidx, H.lcol);
  else
    k_halo<1024, kHaloCap><<<T.ntiles, 1024, 0, s>>>(pass, T.tb, L.S.sptr, L.S.col, T.count,
                                                     H.hptr, H.hidx, H.lcol);
}

amg_status alloc_tiling(amg_hierarchy *h, Tiling *T) {
  AMG_TRY(setup_tmp_alloc(h, reinterpret_cast<void **>(&T->tb),
                          sizeof(int32_t) * ((size_t)T->ntiles + 1)));
  return setup_tmp_alloc(h, reinterpret_cast<void **>(&T->count),
                         sizeof(int32_t) * ((size_t)T->ntiles + 1));
}

// the tiles' starts and list lengths (the lengths on their way to T->hc: the
// caller waits for the stream before that goes, whatever is returned)
amg_status count_halo(amg_hierarchy *h, const Level &L, int32_t step, int32_t nmax,
                      const int32_t *seg, Tiling *T) {
  hipStream_t s = h->stream;
  k_tile_starts<<<ceil_div(T->ntiles + 1, kBlock), kBlock, 0, s>>>(T->ntiles, step, nmax, seg,
                                                                   T->tb);
  launch_halo(h, L, *T, 0, Halo{});
  T->hc.resize(T->ntiles);
  AMG_HIP(hipMemcpyAsync(T->hc.data(), T->count, sizeof(int32_t) * T->ntiles,
                         hipMemcpyDeviceToHost, s));
  return AMG_OK;
}

// Tile lists of level L. Leaves H empty (the kernels then gather from memory)
// when a tile has too many entries to sort in LDS or too long a list for a
// block's LDS.
amg_status build_halo(amg_hierarchy *h, const Level &L, const Tiling &T, Halo *H) {
  int64_t total = 0;
  int32_t umax = 0;
  bool fits = true;
  for (int32_t c : T.hc) {
    fits = fits && c >= 0;
    umax = std::max(umax, c);
    total += c > 0 ? c : 0;
  }
  if (!fits || umax > kHaloMaxList || total > INT32_MAX) return AMG_OK;
  Halo G;
  G.ntiles = T.ntiles;
  G.param = T.param;
  G.umax = umax;
  AMG_TRY(dalloc(h, &G.hptr, (size_t)T.ntiles + 1));
  AMG_TRY(setup_scan(h, T.count, G.hptr, T.ntiles));
  AMG_TRY(dalloc(h, &G.hidx, (size_t)(total > 0 ? total : 1)));
  AMG_TRY(dalloc(h, &G.lcol, (size_t)L.S.nnz_padded));
  launch_halo(h, L, T, 1, G);
  AMG_HIP(hipGetLastError());
  *H = G;
  return AMG_OK;
}

// Level 0's tiles: the row chunks of the streaming kernels and the blocks of
// the down step (coarse rows by coarse_per_block, fine rows by segment).
amg_status build_level0_halos(amg_hierarchy *h) {
  Level &F = h->lv[0];
  // none on levels of kManyRows rows or more: there the kernels take one row
  // per thread (256-row tiles), and staging lost to the gathers from memory
  // (256^3 anisotropic blocks: 144.2 -> 138.6 ms per FP64 solve without tiles)
  if (F.n >= kManyRows) return AMG_OK;
  const Level &C = h->lv[1];
  const Geom g = geom(F.n);
  const int32_t G = staged_down_G(h);
  Tiling rows, segs;
  rows.ntiles = g.grid;
  rows.param = g.chunk;
  rows.rows = g.chunk;
  segs.ntiles = ceil_div(C.n, G);
  segs.param = G;
  segs.rows = (int64_t)G * h->max_seg;
  AMG_TRY(alloc_tiling(h, &rows));
  AMG_TRY(alloc_tiling(h, &segs));
  amg_status st = count_halo(h, F, g.chunk, F.n, nullptr, &rows);
  if (st == AMG_OK) st = count_halo(h, F, G, C.n, F.seg, &segs);
  AMG_HIP(hipStreamSynchronize(h->stream));
  AMG_TRY(st);
  AMG_TRY(build_halo(h, F, rows, &F.hrow));
  return build_halo(h, F, segs, &F.hseg);
}

// average row length from which a level of a smoothed hierarchy is smoothed
// with several lanes per row
constexpr double kLongRow = 48.0;

amg_status build_solve_formats(amg_hierarchy *h) {
  hipStream_t s = h->stream;
  const bool fp32 = h->params.precision == AMG_FP32;
  const size_t vbytes = fp32 ? sizeof(float) : sizeof(double);
  const int32_t nlev = (int32_t)h->lv.size();
  // aggregate-major order, from the coarsest level down
  {
    Level &C = h->lv[nlev - 1];
    AMG_TRY(dalloc(h, &C.perm, (size_t)C.n));
    AMG_TRY(dalloc(h, &C.iperm, (size_t)C.n));
    k_iota_i32<<<grid1(C.n), kBlock, 0, s>>>(C.perm, C.n);
    k_iota_i32<<<grid1(C.n), kBlock, 0, s>>>(C.iperm, C.n);
  }
  h->max_seg = 1;
  for (int32_t l = nlev - 2; l >= 0; --l) {
    Level &F = h->lv[l];
    Level &C = h->lv[l + 1];
    int32_t *cnt;
    AMG_TRY(setup_tmp_alloc(h, reinterpret_cast<void **>(&cnt), sizeof(int32_t) * C.n + 16));
    AMG_TRY(dalloc(h, &F.seg, (size_t)C.n + 1));
    k_seg_count<<<grid1(C.n), kBlock, 0, s>>>(C.n, C.perm, F.mptr, cnt);
    AMG_TRY(setup_scan(h, cnt, F.seg, C.n));
    setup_tmp_free(h, cnt);
    AMG_TRY(dalloc(h, &F.perm, (size_t)F.n));
    AMG_TRY(dalloc(h, &F.iperm, (size_t)F.n));
    AMG_TRY(dalloc(h, &F.aggp, (size_t)F.n));
    AMG_TRY(dalloc(h, &F.pp64, (size_t)F.n));
    k_order_fill<<<grid1(C.n), kBlock, 0, s>>>(C.n, C.perm, F.mptr, F.mem, F.seg, F.p64, F.perm,
                                              F.iperm, F.aggp, F.pp64);
    h->max_seg = std::max(h->max_seg, 1 << F.sweeps);
  }
  // The widths of every level's slices, and whether every value of A on level
  // 0 is an FP32 number: one wait for all of them. The coarsest level of
  // several uses A_L^-1 only.
  const auto has_sell = [&](int32_t l) { return l == 0 || l + 1 < nlev; };
  std::vector<unsigned long long> stat(2 * nlev + 1, 0);
  {
    unsigned long long *dstat;
    const size_t bytes = sizeof(unsigned long long) * stat.size();
    AMG_TRY(setup_tmp_alloc(h, reinterpret_cast<void **>(&dstat), bytes));
    AMG_HIP(hipMemsetAsync(dstat, 0, bytes, s));
    const Level &L0 = h->lv[0];
    k_not_fp32_exact<<<grid1(L0.nnz), kBlock, 0, s>>>(
        L0.nnz, L0.val, reinterpret_cast<int32_t *>(dstat + 2 * nlev));
    for (int32_t l = 0; l < nlev; ++l) {
      if (!has_sell(l)) continue;
      Level &L = h->lv[l];
      L.S.n = L.n;
      L.S.nslices = ceil_div(L.n, kSlice);
      int32_t *w64;
      AMG_TRY(setup_tmp_alloc(h, reinterpret_cast<void **>(&w64),
                              sizeof(int32_t) * L.S.nslices + 16));
      AMG_TRY(dalloc(h, &L.S.sptr, (size_t)L.S.nslices + 1));
      k_sell_width<<<ceil_div(L.S.nslices, 1024 / kSlice), 1024, 0, s>>>(
          L.n, L.S.nslices, L.rp, L.perm, w64, dstat + 2 * l);
      AMG_TRY(setup_scan(h, w64, L.S.sptr, L.S.nslices));
    }
    AMG_HIP(hipMemcpyAsync(stat.data(), dstat, bytes, hipMemcpyDeviceToHost, s));
    AMG_HIP(hipStreamSynchronize(s));
  }
  for (int32_t l = 0; l < nlev; ++l)
    if (stat[2 * l] > (unsigned long long)INT32_MAX)
      return AMG_ERR_ARG;  // padded rows exceed the format's 32-bit offsets
  for (int32_t l = 0; l < nlev; ++l) {
    Level &L = h->lv[l];
    const bool coarsest = (l == nlev - 1);
    // level 0 needs FP64 values for the outer CG; V-cycle levels need the
    // hierarchy precision (plain and scaled)
    const bool need64 = (l == 0) || (!coarsest && !fp32);
    bool need32 = !coarsest && fp32;
    if (l == 0) {
      // every value of A an FP32 number: the FP64 products of level 0 read
      // the exact FP32 copy (identical arithmetic, half the value bytes)
      // unless AMG_FLAG_NO_VALUE_COMPRESSION switches it off
      L.S.fp32_values = stat[2 * nlev] == 0;
      L.S.exact32 = L.S.fp32_values && !(h->params.flags & AMG_FLAG_NO_VALUE_COMPRESSION);
      need32 = need32 || L.S.exact32;
    }
    if (has_sell(l)) {
      Sell &S = L.S;
      const size_t padded = (size_t)stat[2 * l];
      S.nnz_padded = (int64_t)padded;
      S.max_width = (int32_t)stat[2 * l + 1];
      AMG_TRY(dalloc(h, &S.col, padded));
      if (need64) AMG_TRY(dalloc(h, &S.v64, padded));
      if (need32) AMG_TRY(dalloc(h, &S.v32, padded));
      if (!coarsest && !fp32) AMG_TRY(dalloc(h, &S.s64, padded));
      if (!coarsest && fp32) AMG_TRY(dalloc(h, &S.s32, padded));
      if (!coarsest) {
        AMG_TRY(dalloc(h, &L.sminv64, (size_t)L.n));
        if (fp32) {
          AMG_TRY(dalloc(h, &L.sminv32, (size_t)L.n));
          AMG_TRY(dalloc(h, &L.pp32, (size_t)L.n));
        }
      }
      // long rows: their entries over several blocks
      const int64_t mean = L.nnz / L.n;
      const int32_t split = mean < 32 ? 1 : (mean < 512 ? (int32_t)(mean / 32) + 1 : 16);
      k_sell_fill<<<dim3(S.nslices, split), kBlock, 0, s>>>(
          L.n, L.rp, L.ci, L.val, L.perm, L.iperm, L.minv64, S.sptr,
          SellOut{S.col, S.v64, S.v32, S.s64, S.s32, L.sminv64, L.sminv32, L.pp64, L.pp32});
    }
    AMG_TRY(alloc_level_vectors(h, L, vbytes));
    // K-cycle flexible-CG vectors on the levels strictly between the finest
    // and the coarsest
    if (h->params.cycle == AMG_CYCLE_K && l > 0 && l + 1 < nlev) {
      AMG_TRY(dev_alloc(h, &L.c1, vbytes * L.n + 16));
      AMG_TRY(dev_alloc(h, &L.v1, vbytes * L.n + 16));
      AMG_TRY(dev_alloc(h, &L.r1, vbytes * L.n + 16));
      AMG_TRY(dev_alloc(h, &L.c2, vbytes * L.n + 16));
      AMG_TRY(dev_alloc(h, &L.v2, vbytes * L.n + 16));
    }
  }
  // LDS-staged gathers of level 0's products (where every tile's list fits)
  if (nlev > 1) AMG_TRY(build_level0_halos(h));
  if (h->params.cycle == AMG_CYCLE_K) AMG_TRY(dalloc(h, &h->kscal, (size_t)kKScal * nlev));
  if (h->params.smooth_p)
    for (int32_t l = 0; l + 1 < nlev; ++l) {
      AMG_TRY(smooth_solve_format(h, l, fp32));
      // the denser coarse levels: CSR for the kernels with several lanes per row
      if (l > 0 && (double)h->lv[l].nnz > kLongRow * (double)h->lv[l].n)
        AMG_TRY(long_row_csr(h, l, fp32));
    }
  // outer CG vectors and scalars (aggregate-major order of level 0)
  const int32_t n0 = h->lv[0].n;
  AMG_TRY(dalloc(h, &h->x, (size_t)n0));
  AMG_TRY(dalloc(h, &h->b, (size_t)n0));
  AMG_TRY(dalloc(h, &h->r, (size_t)n0));
  AMG_TRY(dalloc(h, &h->z, (size_t)n0));
  AMG_TRY(dalloc(h, &h->p, (size_t)n0));
  AMG_TRY(dalloc(h, &h->q, (size_t)n0));
  AMG_TRY(dalloc(h, &h->partials, (size_t)kMaxParts * kPartPlanes));
  AMG_TRY(dalloc(h, &h->scal, 1));
  AMG_TRY(dalloc(h, &h->zero_flag, 4));
  h->fold = h->params.cycle == AMG_CYCLE_V && !coarse_is_pcg(h) && nlev > 1 &&
            geom(n0).grid <= kFoldParts;
  if (h->params.cycle == AMG_CYCLE_V && !coarse_is_pcg(h) && nlev > 1 && n0 <= kDirRows)
    AMG_TRY(dalloc(h, &h->p2, (size_t)n0));
  AMG_HIP(hipMemsetAsync(h->zero_flag, 0, sizeof(int32_t) * 4, s));
  AMG_HIP(hipMemsetAsync(h->scal, 0, sizeof(PcgScal), s));
  return AMG_OK;
}

// Applies the V-cycle to vectors in the aggregate-major order of level 0.
// The K-cycle with an optional dot partner (see kcycle_top)
amg_status kcycle_perm(amg_hierarchy *h, const double *r, double *z, const double *dv,
                       const int32_t *done) {
  if (h->params.precision == AMG_FP32) kcycle_top<float>(h, r, z, dv, done);
  else kcycle_top<double>(h, r, z, dv, done);
  AMG_HIP(hipGetLastError());
  return AMG_OK;
}

amg_status vcycle_perm(amg_hierarchy *h, const double *r, double *z, bool fuse_dot,
                       const int32_t *done) {
  if (h->params.cycle == AMG_CYCLE_K) return kcycle_perm(h, r, z, nullptr, done);
  if (h->params.precision == AMG_FP32) vcycle_t<float>(h, r, z, fuse_dot, nullptr, done);
  else vcycle_t<double>(h, r, z, fuse_dot, nullptr, done);
  AMG_HIP(hipGetLastError());
  return AMG_OK;
}

// The preconditioner of flexible CG (K-cycle, or a cycle with the iterative
// coarsest solve): z = B r with the block partials of (dv, z) when dv is
// given, left for the caller's finalize.
amg_status precond_perm(amg_hierarchy *h, const double *r, double *z, const double *dv,
                        const int32_t *done) {
  if (h->params.cycle == AMG_CYCLE_K) return kcycle_perm(h, r, z, dv, done);
  if (h->params.precision == AMG_FP32) vcycle_t<float>(h, r, z, dv != nullptr, dv, done);
  else vcycle_t<double>(h, r, z, dv != nullptr, dv, done);
  AMG_HIP(hipGetLastError());
  return AMG_OK;
}

// flexible CG is the outer solver when the preconditioner is not a fixed
// linear operator
inline bool flexible(const amg_hierarchy *h) {
  return h->params.cycle == AMG_CYCLE_K || h->params.coarse_solver == AMG_COARSE_PCG;
}

// z = B r on vectors in the caller's numbering
amg_status vcycle(amg_hierarchy *h, const double *r, double *z, bool fuse_dot,
                  const int32_t *done) {
  hipStream_t s = h->stream;
  const int32_t n = h->lv[0].n;
  k_permute_in<<<grid1(n), kBlock, 0, s>>>(n, h->lv[0].perm, r, h->r);
  // the last post-sweep of a V-cycle stores z in the caller's numbering itself, a
  // launch and a read and a write of z less (160^3 271 -> 259 us a call, 80^3
  // 93.9 -> 90.3; a one-level hierarchy and the K-cycle have no such sweep here)
  const bool out = h->params.cycle == AMG_CYCLE_V && h->lv.size() > 1 && !fuse_dot;
  h->z_out = out ? z : nullptr;
  const amg_status st = vcycle_perm(h, h->r, h->z, fuse_dot, done);
  h->z_out = nullptr;
  AMG_TRY(st);
  if (!out) k_permute_out<<<grid1(n), kBlock, 0, s>>>(n, h->lv[0].perm, h->z, z);
  AMG_HIP(hipGetLastError());
  return AMG_OK;
}

namespace {

// p = z + beta p (copy: p = z) on the CG vectors of level 0
void launch_xpay(amg_hierarchy *h, int32_t n, int32_t copy, const int32_t *done) {
  const bool pairs = reinterpret_cast<uintptr_t>(h->z) % 16 == 0 &&
                     reinterpret_cast<uintptr_t>(h->p) % 16 == 0;
  if (pairs)
    k_xpay<2><<<grid1((n + 1) / 2), kBlock, 0, h->stream>>>(n, h->z, h->p, h->scal, copy, done);
  else
    k_xpay<1><<<grid1(n), kBlock, 0, h->stream>>>(n, h->z, h->p, h->scal, copy, done);
}

// One flexible-CG iteration (K-cycle, or the iterative coarsest solve):
// q = A p with (p, q), (p, r), alpha = (p, r) / (p, q), the x and r updates
// with the stop test, z = B r with (q, z), beta = -(z, q) / (p, q),
// p = z + beta p.
void fcg_iteration(amg_hierarchy *h) {
  hipStream_t s = h->stream;
  Level &L0 = h->lv[0];
  const int32_t n = L0.n;
  const int32_t *done = &h->scal->done;
  const Geom g = geom(n);
  if (L0.S.exact32)
    k_spmv_dots<double, 2, float><<<g.grid, kBlock, 0, s>>>(n, g.chunk, L0.S.sptr, L0.S.col,
                                                            L0.S.v32, h->p, h->q, h->r, nullptr,
                                                            h->partials, done);
  else
    k_spmv_dots<double, 2><<<g.grid, kBlock, 0, s>>>(n, g.chunk, L0.S.sptr, L0.S.col, L0.S.v64,
                                                     h->p, h->q, h->r, nullptr, h->partials,
                                                     done);
  finalize(h, kFinPQR, g.grid, done);
  k_update_xr<<<g.grid, kBlock, 0, s>>>(n, g.chunk, h->x, h->r, h->p, h->q, h->partials, h->scal,
                                        done);
  finalize(h, kFinRR, g.grid, done);
  precond_perm(h, h->r, h->z, h->q, done);
  finalize(h, kFinZQ, g.grid, done);
  launch_xpay(h, n, 0, done);
}

// the direction and the outer product
template <bool FOLD, typename TA>
void dir_spmv(amg_hierarchy *h, const TA *val) {
  hipStream_t s = h->stream;
  const Level &F = h->lv[0];
  const Geom g = geom(F.n);
  if (F.hrow.ok() && F.hrow.param == g.chunk && F.hrow.ntiles == g.grid) {
    const Halo &H = F.hrow;
    launch_k(h, k_dir_spmv_lds<TA, FOLD>, dim3(g.grid), dim3(kBlock),
             (uint32_t)(sizeof(double) * H.umax), s, F.n, g.chunk, F.S.sptr,
             (const uint16_t *)H.lcol, (const int32_t *)H.hptr, (const int32_t *)H.hidx, val,
             (const double *)h->z, h->p, h->p2, h->q, h->partials, h->scal);
    return;
  }
  launch_k(h, k_dir_spmv<TA, FOLD>, dim3(g.grid), dim3(kBlock), 0u, s, F.n, g.chunk, F.S.sptr,
           F.S.col, val, (const double *)h->z, h->p, h->p2, h->q, h->partials, h->scal);
}

template <bool FOLD>
void dir_spmv(amg_hierarchy *h) {
  arm_probe(h, 4);
  if (h->lv[0].S.exact32) dir_spmv<FOLD, float>(h, h->lv[0].S.v32);
  else dir_spmv<FOLD, double>(h, h->lv[0].S.v64);
  h->probe_armed = false;
}

// One CG iteration: (p = z + beta p,) q = A p, alpha, x and r updates with the
// stop test, z = B r with (r, z) and beta(, p = z + beta p). Touches only
// hierarchy buffers, so it is captured once and replayed.
void cg_iteration(amg_hierarchy *h) {
  if (flexible(h)) {
    fcg_iteration(h);
    return;
  }
  hipStream_t s = h->stream;
  if (h->fold) {
    const int32_t *done = &h->scal->done;
    const Geom g = geom(h->lv[0].n);
    dir_spmv<true>(h);
    k_update_fold<<<g.grid, kBlock, 0, s>>>(h->lv[0].n, g.chunk, h->x, h->r, h->p, h->p2, h->q,
                                            h->partials, h->scal);
    // the stop test in the first kernel of the V-cycle, where that is the
    // one-sweep down step
    h->rr_in_down = h->params.pre == 1 && !h->params.smooth_p;
    if (!h->rr_in_down) finalize(h, kFinRR, g.grid, done, kRRPlane);
    vcycle_perm(h, h->r, h->z, true, done);
    h->rr_in_down = false;
    return;
  }
  Level &L0 = h->lv[0];
  const int32_t n = L0.n;
  const int32_t *done = &h->scal->done;
  const Geom g = geom(n);
  if (h->p2) {
    dir_spmv<false>(h);
    finalize(h, kFinPQ, g.grid, done, kPQPlane);
    k_update_dir<<<g.grid, kBlock, 0, s>>>(n, g.chunk, h->x, h->r, h->p, h->p2, h->q,
                                           h->partials, h->scal);
    finalize(h, kFinRR, g.grid, done, kRRPlane);
    vcycle_perm(h, h->r, h->z, true, done);
    return;
  }
  arm_probe(h, 4);
  spmv_dot0(h, h->p, h->q, done);
  h->probe_armed = false;
  finalize(h, kFinPQ, g.grid, done);
  k_update_xr<<<g.grid, kBlock, 0, s>>>(n, g.chunk, h->x, h->r, h->p, h->q, h->partials, h->scal,
                                        done);
  finalize(h, kFinRR, g.grid, done);
  vcycle_perm(h, h->r, h->z, true, done);
  launch_xpay(h, n, 0, done);
}

// Captures `count` CG iterations into one instantiated hipGraph.
bool capture_iterations(amg_hierarchy *h, int32_t count, hipGraph_t *graph, hipGraphExec_t *exec) {
  hipGraph_t g = nullptr;
  if (hipStreamBeginCapture(h->stream, hipStreamCaptureModeThreadLocal) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  for (int32_t k = 0; k < count; ++k) cg_iteration(h);
  hipError_t e = hipStreamEndCapture(h->stream, &g);
  if (e != hipSuccess || !g) {
    (void)hipGetLastError();
    return false;
  }
  hipGraphExec_t ex = nullptr;
  e = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    (void)hipGraphDestroy(g);
    return false;
  }
  *graph = g;
  *exec = ex;
  return true;
}

// The graph of kIterGroups[i] CG iterations, made when it is first wanted: a
// group replay saves the launch gap between consecutive graphs. Null without
// graphs. (With one of eight too, 20^3 to 1e-6 takes 601 us for 606, and the first
// solve, which makes the graphs, 80 us more.)
constexpr int32_t kIterGroups[kIterGraphs] = {1, 4};
hipGraphExec_t iteration_graph(amg_hierarchy *h, int i) {
  if (h->iter_exec[i] || h->graph_failed[i] || (h->params.flags & AMG_FLAG_NO_GRAPH))
    return h->iter_exec[i];
  if (!capture_iterations(h, kIterGroups[i], &h->iter_graph[i], &h->iter_exec[i]))
    h->graph_failed[i] = true;
  return h->iter_exec[i];
}

// `count` iterations onto the stream
amg_status launch_iterations(amg_hierarchy *h, int32_t count, bool use_graph) {
  int32_t k = 0;
  // (the graphs hold the hierarchy's own scratch buffers: launched only when the
  // solve uses them)
  for (int i = kIterGraphs - 1; i >= 0; --i)
    while (use_graph && k + kIterGroups[i] <= count) {
      hipGraphExec_t exec = iteration_graph(h, i);
      if (!exec) break;
      AMG_HIP(hipGraphLaunch(exec, h->stream));
      k += kIterGroups[i];
    }
  for (; k < count; ++k) cg_iteration(h);
  AMG_HIP(hipGetLastError());
  return AMG_OK;
}

}  // namespace

amg_status pcg(amg_hierarchy *h, const double *b_user, double *x_user, double rtol,
               int32_t maxit, amg_solve_info *info, bool use_graph) {
  const double t0 = now_ms();
  hipStream_t s = h->stream;
  Level &L0 = h->lv[0];
  const int32_t n = L0.n;
  const int32_t *done = &h->scal->done;
  const Geom g = geom(n);
  k_permute_in<<<grid1(n), kBlock, 0, s>>>(n, L0.perm, b_user, h->b);
  h->has_rhs = true;
  k_permute_in<<<grid1(n), kBlock, 0, s>>>(n, L0.perm, x_user, h->x);
  k_scal_init<<<1, 1, 0, s>>>(h->scal, rtol, maxit);
  if (L0.S.exact32)
    k_residual_norms<0, float><<<g.grid, kBlock, 0, s>>>(n, g.chunk, L0.S.sptr, L0.S.col,
                                                         L0.S.v32, h->b, h->x, h->r, h->partials);
  else
    k_residual_norms<0, double><<<g.grid, kBlock, 0, s>>>(n, g.chunk, L0.S.sptr, L0.S.col,
                                                          L0.S.v64, h->b, h->x, h->r,
                                                          h->partials);
  finalize(h, kFinInit, g.grid, nullptr);
  k_zero_if_zero_rhs<<<grid1(n), kBlock, 0, s>>>(n, h->x, h->scal);
  if (flexible(h)) AMG_TRY(precond_perm(h, h->r, h->z, nullptr, done));
  else AMG_TRY(vcycle_perm(h, h->r, h->z, true, done));
  if (!h->p2) launch_xpay(h, n, 1, done);
  // (the first solve makes it while the device is busy with the above)
  if (use_graph && maxit >= kIterGroups[1]) (void)iteration_graph(h, 1);
  // Iterations in chunks, whose length follows the observed convergence; after
  // each chunk the host looks at the scalars.
  int32_t queued = 0, chunk = 0;
  double rr_prev = -1.0;
  int32_t it_prev = 0;
  auto queue = [&](int32_t count) -> amg_status {
    const int32_t c = std::min(count, maxit - queued);
    queued += c > 0 ? c : 0;
    return c > 0 ? launch_iterations(h, c, use_graph) : AMG_OK;
  };
  // the iterations still wanted, seen from scalars that the host has looked at
  auto wanted = [&](const PcgScal &sc) -> int32_t {
    if (rr_prev < 0.0) chunk = 4;
    if (rr_prev > 0.0 && sc.iter > it_prev && sc.rr > 0.0 && sc.rr < rr_prev) {
      const double rate = std::pow(sc.rr / rr_prev, 1.0 / (sc.iter - it_prev));
      const double need = std::log(sc.tol2 / sc.rr) / std::log(rate);
      chunk = need < 1.0 ? 1 : (need > 32.0 ? 32 : (int32_t)std::ceil(need));
    }
    rr_prev = sc.rr;
    it_prev = sc.iter;
    return chunk - (queued - sc.iter);
  };
  // A look costs 50 us in which the GPU waits, more than an iteration of few
  // kernels. Where the solve has such, and the residual has to fall further
  // than four iterations bring it (a tenth each, which is fast), the first chunk
  // is of twelve; where it has to fall further than seven tenths, four of them
  // run while the host looks at the first eight. Queued in vain, an iteration
  // costs its launches, 1.7 us a kernel: with 16 in the first chunk of every
  // folded solve, 20^3 took 576 us to 1e-6 and 364 to 1e-2, 48^3 1344 and 583,
  // 50^3 with 2 + 2 sweeps 2042 and 1074; now 600 and 293, 1314 and 497, 2125 and
  // 743. (With kernels for the scalars, in chunks of four: 727 and 316, 1452 and
  // 521, 2168 and 761. Four ahead in every first chunk: 16^3 to 1e-6 548 for 524,
  // in none: 8^3 to 1e-8 454 for 432.)
  const bool few = h->fold && h->params.pre == 1 && h->params.post == 1 &&
                   !h->params.smooth_p && h->lv.size() <= kAheadLevels;
  bool ahead = false;
  for (int32_t next = 0;;) {
    AMG_TRY(queue(next));
    if (ahead) {
      ahead = false;
      AMG_HIP(hipMemcpyAsync(h->scal_host + 1, h->scal, sizeof(PcgScal), hipMemcpyDeviceToHost, s));
      AMG_HIP(hipEventRecord(h->join_event, s));
      AMG_TRY(queue(kAhead));
      AMG_HIP(hipEventSynchronize(h->join_event));
      const PcgScal sc = h->scal_host[1];
      if (sc.done) break;
      AMG_TRY(queue(wanted(sc)));
    }
    AMG_HIP(hipMemcpyAsync(h->scal_host, h->scal, sizeof(PcgScal), hipMemcpyDeviceToHost, s));
    AMG_HIP(hipStreamSynchronize(s));
    const PcgScal sc = *h->scal_host;
    if (sc.done) break;
    if (queued >= maxit) break;  // not reached: the maxit test sets done
    const double tenths = few && rr_prev < 0.0 ? std::log10(sc.rr / sc.tol2) / 2.0 : 0.0;
    next = wanted(sc);
    if (tenths > 4.0) {
      ahead = tenths > 7.0;
      next = ahead ? 12 - kAhead : 12;
    }
  }
  if (L0.S.exact32)
    k_residual_norms<1, float><<<g.grid, kBlock, 0, s>>>(n, g.chunk, L0.S.sptr, L0.S.col,
                                                         L0.S.v32, h->b, h->x, nullptr,
                                                         h->partials);
  else
    k_residual_norms<1, double><<<g.grid, kBlock, 0, s>>>(n, g.chunk, L0.S.sptr, L0.S.col,
                                                          L0.S.v64, h->b, h->x, nullptr,
                                                          h->partials);
  finalize(h, kFinTrue, g.grid, nullptr);
  k_permute_out<<<grid1(n), kBlock, 0, s>>>(n, L0.perm, h->x, x_user);
  AMG_HIP(hipMemcpyAsync(h->scal_host, h->scal, sizeof(PcgScal), hipMemcpyDeviceToHost, s));
  AMG_HIP(hipStreamSynchronize(s));
  const PcgScal sc = *h->scal_host;
  amg_status st = AMG_OK;
  if (sc.done == 2) st = AMG_NOT_CONVERGED;
  if (sc.done == 3) st = AMG_ERR_BREAKDOWN;
  if (info) {
    info->iterations = sc.iter;
    info->converged = (sc.done == 1 || sc.done == 4) ? 1 : 0;
    info->rel_res_recursive = sc.bb > 0.0 ? std::sqrt(sc.rr / sc.bb) : 0.0;
    info->rel_res_true = sc.bb > 0.0 ? std::sqrt(sc.rr_true / sc.bb) : 0.0;
    info->ms = now_ms() - t0;
  }
  return st;
}

namespace {

// One V-cycle exactly as the solve runs it (aggregate-major vectors, no
// permutation, no host work between launches), timed with HIP events; bytes
// = the cycle's algorithmic HBM bytes (0 for a K-cycle hierarchy, whose
// traffic depends on the level visits).
amg_status time_vcycle(amg_hierarchy *h, int32_t reps, double *ms, double *bytes) {
  if (reps < 1 || h->params.cycle != AMG_CYCLE_V) return AMG_ERR_ARG;
  hipStream_t s = h->stream;
  const int32_t *done = h->zero_flag;
  AMG_TRY(vcycle_perm(h, h->r, h->z, false, done));  // warm
  hipEvent_t e0, e1;
  AMG_HIP(hipEventCreate(&e0));
  AMG_HIP(hipEventCreate(&e1));
  AMG_HIP(hipEventRecord(e0, s));
  for (int32_t k = 0; k < reps; ++k) AMG_TRY(vcycle_perm(h, h->r, h->z, false, done));
  AMG_HIP(hipEventRecord(e1, s));
  AMG_HIP(hipEventSynchronize(e1));
  float t = 0.f;
  AMG_HIP(hipEventElapsedTime(&t, e0, e1));
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  *ms = (double)t / reps;
  // per level l < L: down step z(V+4) + 4(n+1) + n(Vr+3V) + n_c(V+4) and the
  // prolongation into it n(3V+4); per coarse level 0 < c < L its
  // post-smoothing z(V+4) + 4(n+1) + 3V n; the coarsest 8 n_L^2 + V n_L; the
  // level-0 post-smoothing z(V+4) + 4(n+1) + n(16+2V); the iterative
  // coarsest solve is not counted (its traffic stays in L2)
  const int32_t L = (int32_t)h->lv.size() - 1;
  const double V = h->params.precision == AMG_FP32 ? 4.0 : 8.0;
  const double nL = h->C.n;
  if (h->params.smooth_p && L > 0) {
    // smoothed prolongators, per level l < L: down step z(V+4) + 4(n+1) +
    // n(Vr+3V); restriction by Pbar^T p(V+4) + 4(n_c+1) + V(n + n_c);
    // prolongation by Pbar p(V+4) + 4(n+1) + V(n_c + 2n); post-smoothing of
    // 0 < l < L z(V+4) + 4(n+1) + 4Vn; the coarsest (Cholesky) 8 n_L^2 +
    // 2V n_L; the level-0 post-smoothing as above
    double b = coarse_is_pcg(h) ? 0.0 : 8.0 * nL * nL + 2.0 * V * nL;
    for (int32_t l = 0; l < L; ++l) {
      const Level &F = h->lv[l];
      const double n = F.n, z = (double)F.nnz, nc = h->lv[l + 1].n, p = (double)F.pb_nnz;
      const double Vr = l == 0 ? 8.0 : V;
      b += z * (V + 4) + 4 * (n + 1) + n * (Vr + 3 * V);
      b += p * (V + 4) + 4 * (nc + 1) + V * (n + nc);
      b += p * (V + 4) + 4 * (n + 1) + V * (nc + 2 * n);
      if (l > 0) b += z * (V + 4) + 4 * (n + 1) + 4 * V * n;
    }
    const double n0 = h->lv[0].n, z0 = (double)h->lv[0].nnz;
    const double Va = V == 8.0 && h->lv[0].S.exact32 ? 4.0 : V;
    b += z0 * (Va + 4) + 4 * (n0 + 1) + n0 * (16 + 2 * V);
    *bytes = b;
    return AMG_OK;
  }
  double b = coarse_is_pcg(h) ? 0.0 : 8.0 * nL * nL + (L == 0 ? 16.0 : V) * nL;
  for (int32_t l = 0; l < L; ++l) {
    const double n = h->lv[l].n, z = (double)h->lv[l].nnz, nc = h->lv[l + 1].n;
    const double Vr = l == 0 ? 8.0 : V;
    // the down step reads A M^-1, or A's exact FP32 copy where it stages M^-1 r
    const double Vs =
        l == 0 && V == 8.0 && h->lv[0].S.exact32 && staged_down<double>(h, h->lv[0], h->lv[1])
            ? 4.0 : V;
    b += z * (Vs + 4) + 4 * (n + 1) + n * (Vr + 3 * V) + nc * (V + 4) + n * (3 * V + 4);
    if (l > 0) b += z * (V + 4) + 4 * (n + 1) + 3 * V * n;
  }
  if (L > 0) {
    const double n0 = h->lv[0].n, z0 = (double)h->lv[0].nnz;
    const double Va = V == 8.0 && h->lv[0].S.exact32 ? 4.0 : V;  // level-0 A as stored
    b += z0 * (Va + 4) + 4 * (n0 + 1) + n0 * (16 + 2 * V);
  }
  *bytes = b;
  return AMG_OK;
}

// algorithmic HBM bytes of one launch of kernel 0-4 on `level`: CSR values +
// int32 columns + int32 row offsets once per SpMV, every vector entry once
double kernel_bytes(const amg_hierarchy *h, int32_t kernel, int32_t level) {
  const Level &F = h->lv[level];
  const Level &C = h->lv[level + 1];
  const bool fp32 = h->params.precision == AMG_FP32;
  const double V = fp32 ? 4.0 : 8.0;
  const double n = F.n, nnz = (double)F.nnz, nc = C.n, nnzc = (double)C.nnz;
  const double Vr = level == 0 ? 8.0 : V;  // level 0 reads/writes the FP64 CG vectors
  switch (kernel) {
    case 0:  // A M^-1 (or A from its exact FP32 copy), r, minv, p read; z, r_c
             // written; segment offsets
      return nnz * ((level == 0 && V == 8.0 && staged_down<double>(h, F, C) && F.S.exact32
                         ? 4.0 : V) + 4) +
             4 * (n + 1) + n * (Vr + 3 * V) + nc * (V + 4);
    case 1:  // A, r, z, minv read; y written (level 0: A from its exact FP32 copy if any)
      return nnz * ((level == 0 && F.S.exact32 ? 4.0 : V) + 4) + 4 * (n + 1) +
             n * (Vr + V + V + Vr);
    case 2:
    case 3:  // coarse A, r_c, z_c, minv_c; fine z read + written, p, positions
      return nnzc * (V + 4) + 4 * (nc + 1) + nc * (3 * V + 4) + n * (3 * V + 4);
    default:  // A (8 or, from the exact FP32 copy, 4 bytes per value), p read; q written
      return nnz * ((F.S.exact32 ? 4.0 : 8.0) + 4) + 4 * (n + 1) + n * 16;
  }
}


// One of the level-0 kernels 0 (down step), 1 (post-smoothing with the CG
// dot) or 4 (outer SpMV with its dot) timed where the solve runs it: `reps`
// CG iterations from x = 0 on the last right-hand side, launched directly
// (the graph cannot hold the events), rtol 0 and maxit reps + 1 so that no
// kernel takes its early exit; the kernel's own dispatch start and end,
// stamped into events by hipExtLaunchKernelGGL, give its mean duration with
// the caches as the iteration leaves them. Hierarchies with one pre- and one
// post-sweep only (otherwise these steps are several kernels).
amg_status time_in_solve(amg_hierarchy *h, int32_t kernel, int32_t reps, double *ms,
                         double *bytes) {
  if (kernel != 0 && kernel != 1 && kernel != 4) return AMG_ERR_ARG;
  if (reps < 1 || reps > 10000 || flexible(h) || h->params.smooth_p || h->lv.size() < 2 ||
      h->params.pre != 1 || h->params.post != 1 || !h->has_rhs)
    return AMG_ERR_ARG;
  hipStream_t s = h->stream;
  Level &L0 = h->lv[0];
  const int32_t n = L0.n;
  const int32_t *done = &h->scal->done;
  const Geom g = geom(n);
  AMG_HIP(hipMemsetAsync(h->x, 0, sizeof(double) * n, s));
  k_scal_init<<<1, 1, 0, s>>>(h->scal, 0.0, reps + 1);
  if (L0.S.exact32)
    k_residual_norms<0, float><<<g.grid, kBlock, 0, s>>>(n, g.chunk, L0.S.sptr, L0.S.col,
                                                         L0.S.v32, h->b, h->x, h->r, h->partials);
  else
    k_residual_norms<0, double><<<g.grid, kBlock, 0, s>>>(n, g.chunk, L0.S.sptr, L0.S.col,
                                                          L0.S.v64, h->b, h->x, h->r,
                                                          h->partials);
  finalize(h, kFinInit, g.grid, nullptr);
  AMG_TRY(vcycle_perm(h, h->r, h->z, true, done));
  if (!h->p2) launch_xpay(h, n, 1, done);
  h->probe_ev.assign(2 * (size_t)reps, nullptr);
  amg_status st = AMG_OK;
  // timing-only events: no system-scope release at the timed dispatch's end
  // (that writeback of L2 is not part of the kernel inside the solve)
  for (auto &e : h->probe_ev)
    if (hipEventCreateWithFlags(&e, hipEventDisableSystemFence) != hipSuccess) st = AMG_ERR_HIP;
  if (st == AMG_OK) {
    h->probe_next = 0;
    h->probe_id = kernel;
    for (int32_t k = 0; k < reps; ++k) cg_iteration(h);
    h->probe_id = -1;
    if (hipGetLastError() != hipSuccess || h->probe_next != h->probe_ev.size() ||
        hipStreamSynchronize(s) != hipSuccess || hipEventSynchronize(h->probe_ev.back()) != hipSuccess)
      st = AMG_ERR_HIP;
  }
  double total = 0.0;
  for (size_t k = 0; st == AMG_OK && k + 1 < h->probe_ev.size(); k += 2) {
    float t = 0.f;
    if (hipEventElapsedTime(&t, h->probe_ev[k], h->probe_ev[k + 1]) != hipSuccess)
      st = AMG_ERR_HIP;
    total += t;
  }
  for (auto e : h->probe_ev)
    if (e) (void)hipEventDestroy(e);
  h->probe_ev.clear();
  (void)hipGetLastError();
  if (st != AMG_OK) return st;
  *ms = total / reps;
  *bytes = kernel_bytes(h, kernel, 0);
  return AMG_OK;
}

}  // namespace

amg_status time_kernel(amg_hierarchy *h, int32_t kernel, int32_t level, int32_t reps,
                       double *ms, double *bytes) {
  const int32_t L = (int32_t)h->lv.size() - 1;
  if (kernel & AMG_TIME_IN_SOLVE) {
    if (level != 0) return AMG_ERR_ARG;
    return time_in_solve(h, kernel & ~AMG_TIME_IN_SOLVE, reps, ms, bytes);
  }
  if (kernel == 5) return time_vcycle(h, reps, ms, bytes);
  if (level < 0 || level >= L || reps < 1 || kernel < 0 || kernel > 4) return AMG_ERR_ARG;
  if (kernel == 4 && level != 0) return AMG_ERR_ARG;
  // the fused down and up kernels are those of the tentative prolongator
  if (h->params.smooth_p && (kernel == 0 || kernel == 2 || kernel == 3)) return AMG_ERR_ARG;
  if ((kernel == 2 || kernel == 3) && level + 1 >= L) return AMG_ERR_ARG;
  hipStream_t s = h->stream;
  Level &F = h->lv[level];
  Level &C = h->lv[level + 1];
  const bool fp32 = h->params.precision == AMG_FP32;
  const double V = fp32 ? 4.0 : 8.0;
  const double n = F.n, nnz = (double)F.nnz, nc = C.n, nnzc = (double)C.nnz;
  const double Vr = level == 0 ? 8.0 : V;  // level 0 reads/writes the FP64 CG vectors
  const int32_t *done = h->zero_flag;
  auto launch = [&]() {
    const Geom g = geom(F.n);
    switch (kernel) {
      case 0:  // pre-smoothing + residual + restriction on `level`
        if (fp32) {
          if (level == 0)
            pre_restrict<float, double, kPreScaled, float>(h, F, C, F.S.s32, F.sminv32, F.pp32,
                                                           h->r, (float *)F.z, (float *)C.r,
                                                           done);
          else
            pre_restrict<float, float, kPreScaled, float>(h, F, C, F.S.s32, F.sminv32, F.pp32,
                                                          (const float *)F.r, (float *)F.z,
                                                          (float *)C.r, done);
        } else {
          down_one_sweep<double, double>(h, F, C, level == 0 ? h->r : (const double *)F.r,
                                         (double *)F.z, done);
        }
        break;
      case 1:  // post-smoothing on `level` (level 0: with the CG dot product)
        if (fp32) {
          if (level == 0)
            post_sweep<float, double, double, true, float>(h, F, F.S.v32, F.sminv32, h->r,
                                                           (const float *)F.z, h->z,
                                                           h->partials, done);
          else
            post_sweep<float, float, float, false, float>(h, F, F.S.v32, F.sminv32,
                                                          (const float *)F.r, (const float *)F.z,
                                                          (float *)F.y, nullptr, done);
        } else {
          if (level == 0 && F.S.exact32)
            post_sweep<double, double, double, true, float>(h, F, F.S.v32, F.sminv64, h->r,
                                                            (const double *)F.z, h->z,
                                                            h->partials, done);
          else if (level == 0)
            post_sweep<double, double, double, true, double>(h, F, F.S.v64, F.sminv64, h->r,
                                                             (const double *)F.z, h->z,
                                                             h->partials, done);
          else
            post_sweep<double, double, double, false, double>(
                h, F, F.S.v64, F.sminv64, (const double *)F.r, (const double *)F.z,
                (double *)F.y, nullptr, done);
        }
        break;
      case 2:  // post-smoothing on level + 1 fused with prolongation into level
      case 3:
        if (fp32)
          k_post_prolong<float><<<grid1(C.n), kBlock, 0, s>>>(
              C.n, C.S.sptr, C.S.col, C.S.v32, C.sminv32, (const float *)C.r,
              (const float *)C.z, F.seg, F.aggp, F.pp32, (float *)F.t, done);
        else
          k_post_prolong<double><<<grid1(C.n), kBlock, 0, s>>>(
              C.n, C.S.sptr, C.S.col, C.S.v64, C.sminv64, (const double *)C.r,
              (const double *)C.z, F.seg, F.aggp, F.pp64, (double *)F.t, done);
        break;
      default:
        spmv_dot0(h, h->p, h->q, done);
        break;
    }
  };
  hipEvent_t e0, e1;
  AMG_HIP(hipEventCreate(&e0));
  AMG_HIP(hipEventCreate(&e1));
  launch();  // warm
  AMG_HIP(hipEventRecord(e0, s));
  for (int32_t k = 0; k < reps; ++k) launch();
  AMG_HIP(hipEventRecord(e1, s));
  AMG_HIP(hipEventSynchronize(e1));
  float t = 0.f;
  AMG_HIP(hipEventElapsedTime(&t, e0, e1));
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  *ms = (double)t / reps;
  *bytes = kernel_bytes(h, kernel, level);
  return AMG_OK;
}

}  // namespace amg
