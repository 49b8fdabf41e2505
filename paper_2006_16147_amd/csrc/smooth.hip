// Smoothed aggregation on the GPU (the alternative to the K-cycle in
// Section 3.2): omega = 4 / (3 ||D^-1 A||_inf) (the damping 4 / (3 rho(D^-1 A))
// with rho estimated by the infinity norm, which reproduces the supplement's
// convergence constant of the smoothed prolongator), the smoothed prolongator
// Pbar = (I - omega D^-1 A) P of the composed tentative P, and the next level
// Pbar^T A Pbar; plus Pbar and Pbar^T in the solve numbering.
//
// Every sum is the sequential sum of its definition: the terms of one position
// in a fixed order (the order of the row's entries, then of the entries of the
// rows they select), each added onto the first. So the hierarchy is the same
// bit for bit on every run (built with -ffp-contract=off).
//
// A product's row is formed by a group of lanes with a table of its columns in
// LDS: the combining entries one after the other, the lanes over the entries
// of the row each one selects, which have different columns; then the columns
// are ranked and the row is written. That reads every operand once and writes
// the row once. (As expand - sort - reduce, every term written to memory, six
// to eight passes of a radix sort over 16 bytes per term and a thread per sum,
// it took 27 of the 40 ms of an 80^3 setup.) The radix sort is left for the
// transpose of a matrix with a column too long to be sorted in LDS.

#include <cstring>
#include <map>
#include <mutex>
#include <utility>

#include "internal.h"

namespace amg {

namespace {

constexpr int kSortThreads = 256;
constexpr int kSortItems = 8;  // elements per thread in a block's tile
constexpr int kSortTile = kSortThreads * kSortItems;
constexpr int kRadixBits = 8;
constexpr int kRadix = 1 << kRadixBits;  // one digit per thread of a block
static_assert(kRadix == kSortThreads, "one thread per digit");

inline int32_t grid(int64_t n) { return ceil_div(n > 0 ? n : 1, kBlock); }

// bits needed for the values 0 .. n - 1
int bits_for(int64_t n) {
  int b = 0;
  while ((int64_t(1) << b) < n) ++b;
  return b;
}

// Temporaries of the smoothed setup: carved from one workspace per device
// that grows on demand (blocks of at least twice the previous size) and is
// kept until the process ends; a Scratch holds the device's workspace lock
// for its lifetime, so smoothed setups on one device take turns. A product
// takes a dozen buffers of up to several GiB; allocating and freeing them per
// call (through the stream-ordered pool or hipMalloc/hipFree) cost far more
// than the kernels, up to seconds per call once such blocks had been freed.
struct Workspace {
  std::mutex m;
  std::vector<std::pair<char *, size_t>> blocks;
};

Workspace &workspace(int device) {
  static std::mutex guard;
  static std::map<int, Workspace *> all;
  std::lock_guard<std::mutex> g(guard);
  Workspace *&w = all[device];
  if (!w) w = new Workspace();  // process lifetime
  return *w;
}

struct Scratch {
  int device;
  hipStream_t s;
  Workspace &ws;
  std::unique_lock<std::mutex> lock;
  size_t block = 0, used = 0;  // current block and bytes taken from it
  explicit Scratch(const amg_hierarchy *h)
      : device(h->device), s(h->stream), ws(workspace(h->device)), lock(ws.m) {}
  Scratch(const Scratch &) = delete;
  Scratch &operator=(const Scratch &) = delete;
  ~Scratch() { (void)hipStreamSynchronize(s); }  // the next user may be another stream
  template <typename T>
  amg_status get(T **p, size_t count) {
    const size_t bytes = (count * sizeof(T) + 16 + 255) & ~size_t(255);
    while (block < ws.blocks.size() && used + bytes > ws.blocks[block].second) {
      ++block;
      used = 0;
    }
    if (block == ws.blocks.size()) {
      size_t sz = size_t(256) << 20;
      for (const auto &b : ws.blocks) sz = b.second * 2 > sz ? b.second * 2 : sz;
      if (bytes > sz) sz = bytes;
      void *q = nullptr;
      hipError_t e = hipMalloc(&q, sz);
      if (e == hipErrorOutOfMemory) {  // the blocks kept for hierarchies first
        (void)hipGetLastError();
        release_kept(device, s);
        e = hipMalloc(&q, sz);
      }
      AMG_HIP(e);
      ws.blocks.emplace_back(reinterpret_cast<char *>(q), sz);
      used = 0;
    }
    *p = reinterpret_cast<T *>(ws.blocks[block].first + used);
    used += bytes;
    return AMG_OK;
  }
};

// ---------------------------------------------------------------------------
// stable LSD radix sort of (64-bit key, double) pairs, 8 bits per pass
// ---------------------------------------------------------------------------

// digit counts of each block's tile, digit-major: hist[d * nblocks + block]
__global__ void __launch_bounds__(kSortThreads) k_radix_hist(int32_t count,
                                                            const uint64_t *__restrict__ key,
                                                            int shift, int32_t nblocks,
                                                            int32_t *__restrict__ hist) {
  __shared__ int32_t c[kRadix];
  c[threadIdx.x] = 0;
  __syncthreads();
  const int64_t t0 = (int64_t)blockIdx.x * kSortTile;
  for (int u = 0; u < kSortItems; ++u) {
    const int64_t i = t0 + (int64_t)u * kSortThreads + threadIdx.x;
    if (i < count) atomicAdd(&c[(key[i] >> shift) & (kRadix - 1)], 1);
  }
  __syncthreads();
  hist[(int64_t)threadIdx.x * nblocks + blockIdx.x] = c[threadIdx.x];
}

// Writes every element of the block's tile to its place: the exclusive scan
// of the digit-major counts (offs) gives where the block's run of each digit
// starts; inside the tile, elements keep their index order (rounds of one
// element per thread, waves in order, lanes in order).
__global__ void __launch_bounds__(kSortThreads) k_radix_scatter(
    int32_t count, const uint64_t *__restrict__ key, const double *__restrict__ val, int shift,
    int32_t nblocks, const int32_t *__restrict__ offs, uint64_t *__restrict__ key_out,
    double *__restrict__ val_out) {
  constexpr int kW = kSortThreads / kWave;
  __shared__ int32_t base[kRadix];
  __shared__ int32_t wcnt[kW][kRadix];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wid = tid / kWave;
  base[tid] = offs[(int64_t)tid * nblocks + blockIdx.x];
  const uint64_t below = lane == 0 ? 0ull : (~0ull >> (kWave - lane));
  const int64_t t0 = (int64_t)blockIdx.x * kSortTile;
  for (int u = 0; u < kSortItems; ++u) {
    for (int w = 0; w < kW; ++w) wcnt[w][tid] = 0;
    __syncthreads();
    const int64_t i = t0 + (int64_t)u * kSortThreads + tid;
    const bool ok = i < count;
    uint64_t k = 0;
    double v = 0.0;
    int d = 0;
    if (ok) {
      k = key[i];
      v = val[i];
      d = (int)((k >> shift) & (kRadix - 1));
    }
    // lanes of this wave holding the same digit
    uint64_t m = __ballot(ok);
    for (int b = 0; b < kRadixBits; ++b) {
      const bool bit = (d >> b) & 1;
      const uint64_t bb = __ballot(bit);
      m &= bit ? bb : ~bb;
    }
    const int rank = __popcll(m & below);
    if (ok && rank == 0) wcnt[wid][d] = __popcll(m);
    __syncthreads();
    {  // digit tid: where each wave's group starts, and the block's new base
      int32_t sacc = base[tid];
      for (int w = 0; w < kW; ++w) {
        const int32_t c = wcnt[w][tid];
        wcnt[w][tid] = sacc;
        sacc += c;
      }
      base[tid] = sacc;
    }
    __syncthreads();
    if (ok) {
      const int32_t pos = wcnt[wid][d] + rank;
      key_out[pos] = k;
      val_out[pos] = v;
    }
    __syncthreads();
  }
}

// sorts count pairs by the low `bits` bits of the key, stably; *key and *val
// point at the sorted arrays on return (buffers of the scratch set)
amg_status radix_sort(Scratch &S, int32_t count, int bits, uint64_t **key, double **val) {
  if (count <= 1 || bits <= 0) return AMG_OK;
  hipStream_t s = S.s;
  const int32_t nblocks = ceil_div(count, kSortTile);
  if ((int64_t)nblocks * kRadix >= INT32_MAX) return AMG_ERR_ARG;
  uint64_t *k2;
  double *v2;
  int32_t *hist, *offs, *bsum;
  AMG_TRY(S.get(&k2, (size_t)count));
  AMG_TRY(S.get(&v2, (size_t)count));
  AMG_TRY(S.get(&hist, (size_t)nblocks * kRadix));
  AMG_TRY(S.get(&offs, (size_t)nblocks * kRadix + 1));
  AMG_TRY(S.get(&bsum, scan_sums(nblocks * kRadix)));
  for (int shift = 0; shift < bits; shift += kRadixBits) {
    k_radix_hist<<<nblocks, kSortThreads, 0, s>>>(count, *key, shift, nblocks, hist);
    scan_exclusive_i32(hist, offs, nblocks * kRadix, bsum, s);
    k_radix_scatter<<<nblocks, kSortThreads, 0, s>>>(count, *key, *val, shift, nblocks, offs, k2,
                                                     v2);
    std::swap(*key, k2);
    std::swap(*val, v2);
  }
  AMG_HIP(hipGetLastError());
  return AMG_OK;
}

// ---------------------------------------------------------------------------
// sorted (row << cb | column, term) pairs -> CSR with the runs summed in order
// ---------------------------------------------------------------------------

__global__ void k_heads(int32_t count, const uint64_t *__restrict__ key, int32_t *__restrict__ h) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) h[i] = (i == 0 || key[i] != key[i - 1]) ? 1 : 0;
}

__global__ void k_run_start(int32_t count, const int32_t *__restrict__ h,
                            const int32_t *__restrict__ run, int32_t *__restrict__ start) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count && h[i]) start[run[i]] = (int32_t)i;
  if (i == 0) start[run[count]] = count;  // run[count] = number of runs
}

// one thread per run: the first term, then the others added in order
__global__ void k_run_sum(int32_t nrun, const int32_t *__restrict__ start,
                          const uint64_t *__restrict__ key, const double *__restrict__ val,
                          int cb, int32_t *__restrict__ row_of, int32_t *__restrict__ col,
                          double *__restrict__ out) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= nrun) return;
  const int32_t b = start[r], e = start[r + 1];
  double v = val[b];
  for (int32_t t = b + 1; t < e; ++t) v = v + val[t];
  out[r] = v;
  const uint64_t k = key[b];
  col[r] = (int32_t)(k & ((uint64_t(1) << cb) - 1));
  row_of[r] = (int32_t)(k >> cb);
}

// rp[q] = first run of row q (runs are sorted by row); rp[nrows] = nrun
__global__ void k_row_ptr(int32_t nrun, int32_t nrows, const int32_t *__restrict__ row_of,
                          int32_t *__restrict__ rp) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s > nrun) return;
  const int32_t lo = s == 0 ? -1 : row_of[s - 1];
  const int32_t hi = s == nrun ? nrows : row_of[s];
  for (int32_t q = lo + 1; q <= hi; ++q) rp[q] = (int32_t)s;
}

// destination of a reduced CSR: owned by the hierarchy or by the scratch set
struct CsrOut {
  int32_t *rp = nullptr, *ci = nullptr;
  double *val = nullptr;
  int64_t nnz = 0;
};

// for a result whose arrays are there
amg_status kept(int32_t **, size_t, int32_t **, double **, size_t) { return AMG_OK; }

template <typename Alloc>
amg_status reduce_sorted(Scratch &S, int32_t count, const uint64_t *key, const double *val,
                         int32_t nrows, int cb, Alloc alloc, CsrOut *out) {
  hipStream_t s = S.s;
  int32_t *h, *run, *bsum;
  AMG_TRY(S.get(&h, (size_t)count + 1));
  AMG_TRY(S.get(&run, (size_t)count + 1));
  AMG_TRY(S.get(&bsum, scan_sums(count)));
  k_heads<<<grid(count), kBlock, 0, s>>>(count, key, h);
  scan_exclusive_i32(h, run, count, bsum, s);
  int32_t nrun = 0;
  AMG_HIP(hipMemcpyAsync(&nrun, run + count, sizeof(int32_t), hipMemcpyDeviceToHost, s));
  AMG_HIP(hipStreamSynchronize(s));
  int32_t *start, *row_of;
  AMG_TRY(S.get(&start, (size_t)nrun + 1));
  AMG_TRY(S.get(&row_of, (size_t)nrun + 1));
  AMG_TRY(alloc(&out->rp, (size_t)nrows + 1, &out->ci, &out->val, (size_t)nrun));
  k_run_start<<<grid((int64_t)count + 1), kBlock, 0, s>>>(count, h, run, start);
  k_run_sum<<<grid(nrun), kBlock, 0, s>>>(nrun, start, key, val, cb, row_of, out->ci, out->val);
  k_row_ptr<<<grid((int64_t)nrun + 1), kBlock, 0, s>>>(nrun, nrows, row_of, out->rp);
  AMG_HIP(hipGetLastError());
  out->nnz = nrun;
  return AMG_OK;
}

// ---------------------------------------------------------------------------
// small steps of the products and the transposes
// ---------------------------------------------------------------------------

// (sum over ascending j of |a_ij|) / a_ii per row; maximum over rows (the
// bits of non-negative doubles order like the values). A thread per row, the
// sum's order being fixed; its loads go eight at a time.
__global__ void k_absnorm(int32_t n, const int32_t *__restrict__ rp, const int32_t *__restrict__ ci,
                          const double *__restrict__ val, unsigned long long *__restrict__ mx) {
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double sum = 0.0, aii = 0.0;
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
      sum = sum + fabs(a[u]);
      if (c[u] == i) aii = a[u];
    }
  }
  const double r = sum / aii;
  atomicMax(mx, (unsigned long long)__double_as_longlong(r));
}

// entries of an nr-row CSR keyed as (column << cb | row), i.e. transposed
__global__ void k_transpose_keys(int32_t nr, const int32_t *__restrict__ rp,
                                 const int32_t *__restrict__ ci, const double *__restrict__ val,
                                 int cb, uint64_t *__restrict__ key, double *__restrict__ v) {
  const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nr) return;
  for (int32_t e = rp[i]; e < rp[i + 1]; ++e) {
    key[e] = ((uint64_t)ci[e] << cb) | (uint64_t)i;
    v[e] = val[e];
  }
}

// lower triangle := upper triangle, so the product is bitwise symmetric; G
// lanes per row, each its own entries (a thread per row: 465 us on average)
template <int G>
__global__ void k_mirror_lower(int32_t n, const int32_t *__restrict__ rp,
                               const int32_t *__restrict__ ci, double *__restrict__ val,
                               int32_t *__restrict__ err) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int32_t I = (int32_t)(t / G);
  if (t / G >= n) return;
  for (int32_t k = rp[I] + (int32_t)(t % G), e = rp[I + 1]; k < e; k += G) {
    const int32_t J = ci[k];
    if (J >= I) break;
    int32_t lo = rp[J], hi = rp[J + 1] - 1, m = -1;
    while (lo <= hi) {
      const int32_t mid = lo + (hi - lo) / 2;
      if (ci[mid] == I) {
        m = mid;
        break;
      }
      if (ci[mid] < I) lo = mid + 1;
      else hi = mid - 1;
    }
    if (m < 0) {
      atomicOr(err, 1);
      return;
    }
    val[k] = val[m];
  }
}

__global__ void k_demote_f64(int64_t n, const double *__restrict__ a, float *__restrict__ b) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) b[i] = (float)a[i];
}

// ---------------------------------------------------------------------------
// rows formed in LDS
// ---------------------------------------------------------------------------

// LDS written by lanes of a group is read by its other lanes: a group is part
// of a wave, or a whole block
template <int G>
__device__ __forceinline__ void group_sync() {
  if (G > kWave) {
    __syncthreads();
  } else {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

// a matrix whose row i holds the entries [b[i], e[i])
struct Rows {
  const int32_t *b, *e, *ci;
  const double *val;
};

// entries [b[r], e[r]) of the result, in the room that starts at off[r]
struct RowsOut {
  const int32_t *off;
  int32_t *b, *e, *ci;
  double *val;
};

// rows still to do: all of them, or those listed; and where to list the rows
// that do not fit here
struct Work {
  int32_t nr;
  const int32_t *list, *nlist;
  int32_t *ovf, *novf;
};

// Number of terms of each row: the lengths of the rows of B its entries
// select (eight lanes per row); and their 64-bit total
__global__ void __launch_bounds__(kBlock) k_comb_len(int32_t nr, const int32_t *__restrict__ xp,
                                                     const int32_t *__restrict__ src, Rows B,
                                                     int32_t *__restrict__ len,
                                                     unsigned long long *__restrict__ total) {
  __shared__ unsigned long long sum;
  if (threadIdx.x == 0) sum = 0;
  __syncthreads();
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int32_t r = (int32_t)(t / 8);
  int64_t c = 0;
  if (t / 8 < nr)
    for (int32_t k = xp[r] + (int32_t)(t % 8), e = xp[r + 1]; k < e; k += 8) {
      const int32_t j = src[k];
      c += B.e[j] - B.b[j];
    }
  for (int o = 4; o > 0; o >>= 1) c += __shfl_xor(c, o, 8);
  if (t / 8 < nr && t % 8 == 0) {
    len[r] = c > INT32_MAX ? INT32_MAX : (int32_t)c;
    atomicAdd(&sum, (unsigned long long)c);
  }
  __syncthreads();
  if (threadIdx.x == 0 && sum) atomicAdd(total, sum);
}

// Row r of sum_k coef_k B(src_k, :), k in [xp[r], xp[r + 1]): G lanes and a
// table of H slots per row. What bounds it is the latency of the entries'
// loads and of the insertions' trips through LDS, one after the other for a
// row: the row bounds come for G combining entries at a time, and the next G
// entries are loaded while the last are inserted; a group is as wide as the
// selected rows are long. The table has room for 3 H / 4 columns and one more
// step's; a row that might not fit is listed. The columns found are counted
// again only when they might have become too many.
template <int G, int H>
__global__ void __launch_bounds__(kBlock) k_comb_rows(Work W, const int32_t *__restrict__ xp,
                                                      const int32_t *__restrict__ src,
                                                      const double *__restrict__ coef, Rows B,
                                                      RowsOut O) {
  static_assert(H >= 4 * G && (H & (H - 1)) == 0 && G <= kBlock, "table size");
  constexpr int kGroups = kBlock / G, kMost = 3 * H / 4 + G;
  constexpr int kBits = __builtin_ctz(H);
  __shared__ int32_t key[kGroups][H];
  __shared__ double sum[kGroups][H];
  __shared__ int32_t col[kGroups][kMost];
  __shared__ uint16_t at[kGroups][kMost];
  __shared__ int32_t count[kGroups];
  __shared__ int32_t kb[kGroups][G], ke[kGroups][G];
  __shared__ double kc[kGroups][G];
  const int lane = threadIdx.x % G, grp = threadIdx.x / G;
  const int32_t rows = W.list ? *W.nlist : W.nr;
  for (int32_t o = blockIdx.x * kGroups + grp; o < rows; o += gridDim.x * kGroups) {
    const int32_t r = W.list ? W.list[o] : o;
    group_sync<G>();  // the previous row's table is read no more
    for (int s = lane; s < H; s += G) key[grp][s] = -1;
    if (lane == 0) count[grp] = 0;
    const int32_t x0 = xp[r], x1 = xp[r + 1];
    bool full = false;
    int32_t most = 0;  // at least the columns found
    for (int32_t k0 = x0; k0 < x1 && !full; k0 += G) {
      group_sync<G>();
      if (k0 + lane < x1) {
        const int32_t j = src[k0 + lane];
        kb[grp][lane] = B.b[j];
        ke[grp][lane] = B.e[j];
        kc[grp][lane] = coef[k0 + lane];
      }
      group_sync<G>();
      const int32_t nk = min(G, x1 - k0);
      // the steps: G entries at a time of the rows selected by q = 0 .. nk - 1
      int32_t q = 0, e0 = kb[grp][0], e1 = ke[grp][0];
      while (q < nk && e0 >= e1)
        if (++q < nk) {
          e0 = kb[grp][q];
          e1 = ke[grp][q];
        }
      int32_t J = -1;
      double v = 0.0;
      if (q < nk && e0 + lane < e1) {
        J = B.ci[e0 + lane];
        v = B.val[e0 + lane];
      }
      while (q < nk) {
        const double t = kc[grp][q] * v;
        const int32_t Jt = J, n = min(G, e1 - e0);
        // on to the next step, its loads first
        e0 += G;
        while (q < nk && e0 >= e1)
          if (++q < nk) {
            e0 = kb[grp][q];
            e1 = ke[grp][q];
          }
        J = -1;
        if (q < nk && e0 + lane < e1) {
          J = B.ci[e0 + lane];
          v = B.val[e0 + lane];
        }
        if (most + n > 3 * H / 4) {
          group_sync<G>();
          most = count[grp];
          group_sync<G>();
          if (most + n > kMost) {
            full = true;
            break;
          }
        }
        most += n;
        if (Jt >= 0) {
          uint32_t s = ((uint32_t)Jt * 2654435761u) >> (32 - kBits);
          for (;;) {
            const int32_t had = atomicCAS(&key[grp][s], -1, Jt);
            if (had == Jt) {
              sum[grp][s] = sum[grp][s] + t;
              break;
            }
            if (had < 0) {
              sum[grp][s] = t;
              atomicAdd(&count[grp], 1);
              break;
            }
            s = (s + 1) & (H - 1);
          }
        }
        group_sync<G>();
      }
    }
    group_sync<G>();
    if (full) {
      if (lane == 0) W.ovf[atomicAdd(W.novf, 1)] = r;
      continue;
    }
    const int32_t m = count[grp], base = O.off[r];
    group_sync<G>();
    if (lane == 0) count[grp] = 0;
    group_sync<G>();
    for (int s = lane; s < H; s += G)
      if (key[grp][s] >= 0) {
        const int32_t i = atomicAdd(&count[grp], 1);
        col[grp][i] = key[grp][s];
        at[grp][i] = (uint16_t)s;
      }
    group_sync<G>();
    for (int32_t i = lane; i < m; i += G) {
      const int32_t J = col[grp][i];
      int32_t rank = 0;
      for (int32_t f = 0; f < m; ++f) rank += col[grp][f] < J ? 1 : 0;
      O.ci[base + rank] = J;
      O.val[base + rank] = sum[grp][at[grp][i]];
    }
    if (lane == 0) {
      O.b[r] = base;
      O.e[r] = base + m;
    }
  }
}

// Rows of Pbar from the terms a_ij p_j, one per entry of A's row i: ranked by
// (aggregate, entry) against the row's keys in LDS, every run of an aggregate
// added up by its first lane, then Pbar(i, J) = (J = agg[i] ? p_i : 0) -
// omega (s / a_ii). G lanes per row with E terms each; longer rows are listed.
template <int G, int E>
__global__ void __launch_bounds__(kBlock) k_pbar_rows(
    Work W, const int32_t *__restrict__ rp, const int32_t *__restrict__ ci,
    const double *__restrict__ val, const int32_t *__restrict__ agg, const double *__restrict__ p,
    double omega, RowsOut O) {
  constexpr int kGroups = kBlock / G, kCap = G * E;
  __shared__ int32_t key[kGroups][kCap], col[kGroups][kCap];
  __shared__ double sum[kGroups][kCap];
  __shared__ double diag[kGroups];
  __shared__ int32_t heads[kGroups][G];
  const int lane = threadIdx.x % G, grp = threadIdx.x / G;
  const int32_t rows = W.list ? *W.nlist : W.nr;
  for (int32_t o = blockIdx.x * kGroups + grp; o < rows; o += gridDim.x * kGroups) {
    const int32_t i = W.list ? W.list[o] : o;
    const int32_t b = rp[i], len = rp[i + 1] - b;
    if (len > kCap) {
      if (lane == 0) W.ovf[atomicAdd(W.novf, 1)] = i;
      continue;
    }
    group_sync<G>();  // the previous row's terms are read no more
    if (lane == 0) diag[grp] = 0.0;
    group_sync<G>();
    double t[E];
    int32_t kq[E];
#pragma unroll
    for (int q = 0; q < E; ++q) {
      const int32_t e = lane + q * G;
      t[q] = 0.0;
      kq[q] = -1;
      if (e >= len) continue;
      const int32_t j = ci[b + e];
      const double a = val[b + e];
      key[grp][e] = kq[q] = agg[j];
      t[q] = a * p[j];
      if (j == i) diag[grp] = a;
    }
    group_sync<G>();
    int32_t rank[E];
#pragma unroll
    for (int q = 0; q < E; ++q) rank[q] = 0;
    for (int32_t f = 0; f < len; ++f) {
      const int32_t kf = key[grp][f];
#pragma unroll
      for (int q = 0; q < E; ++q)
        rank[q] += kf < kq[q] || (kf == kq[q] && f < lane + q * G) ? 1 : 0;
    }
#pragma unroll
    for (int q = 0; q < E; ++q) {
      const int32_t e = lane + q * G;
      if (e >= len) continue;
      col[grp][rank[q]] = kq[q];
      sum[grp][rank[q]] = t[q];
    }
    group_sync<G>();
    // lane's positions [lane E, lane E + E): its runs, and those before them
    int32_t mine = 0;
    for (int32_t e = lane * E; e < min(len, lane * E + E); ++e)
      mine += e == 0 || col[grp][e] != col[grp][e - 1] ? 1 : 0;
    heads[grp][lane] = mine;
    group_sync<G>();
    int32_t before = 0, all = 0;
    for (int f = 0; f < G; ++f) {
      before += f < lane ? heads[grp][f] : 0;
      all += heads[grp][f];
    }
    const double aii = diag[grp];
    const int32_t own = agg[i], base = O.off[i];
    for (int32_t e = lane * E; e < min(len, lane * E + E); ++e) {
      const int32_t J = col[grp][e];
      if (e > 0 && col[grp][e - 1] == J) continue;
      double v = sum[grp][e];
      for (int32_t f = e + 1; f < len && col[grp][f] == J; ++f) v = v + sum[grp][f];
      const double w = v / aii;
      O.ci[base + before] = J;
      O.val[base + before] = (J == own ? p[i] : 0.0) - omega * w;
      ++before;
    }
    if (lane == 0) {
      O.b[i] = base;
      O.e[i] = base + all;
    }
  }
}

// Rows sorted by column: row q of the result is row `of[q]` of A (NULL: q)
// with its columns renumbered by `map` (NULL: unchanged); equal columns keep their
// order. An entry's place is the number of keys before its own, a quadratic
// count that LDS reads and compares bound: N entries per lane at a time share the
// reads of four keys each, N four for rows longer than the group (80^3 smoothed
// setup: 548 us for 2245 with one key per read and entry).
template <int G, int N>
__device__ __forceinline__ void rank_rows(const int32_t *key, int32_t len, int lane, int32_t d,
                                          const double *__restrict__ val, int32_t *dci,
                                          double *dval) {
  for (int32_t e0 = lane; e0 < len; e0 += N * G) {
    int32_t c[N], rank[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const int32_t e = e0 + u * G;
      c[u] = key[e < len ? e : 0];
      rank[u] = 0;
    }
    // (past len the keys are INT32_MAX: never before another)
    for (int32_t f = 0; f < len; f += 4) {
      const int4 k = *reinterpret_cast<const int4 *>(&key[f]);
#pragma unroll
      for (int u = 0; u < N; ++u) {
        const int32_t t = f + 3 < e0 + u * G ? c[u] + 1 : c[u];  // equal ones before e count
        rank[u] += (k.x < t) + (k.y < t) + (k.z < t) + (k.w < t);
      }
    }
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const int32_t e = e0 + u * G;
      if (e >= len) continue;
      for (int32_t f = e & ~3; f < e; ++f) rank[u] += key[f] == c[u] ? 1 : 0;
      dci[d + rank[u]] = c[u];
      dval[d + rank[u]] = val[e];
    }
  }
}

template <int G, int E>
__global__ void __launch_bounds__(kBlock) k_sort_rows(Work W, const int32_t *__restrict__ of,
                                                      const int32_t *__restrict__ map,
                                                      const int32_t *__restrict__ rp,
                                                      const int32_t *__restrict__ ci,
                                                      const double *__restrict__ val,
                                                      const int32_t *__restrict__ drp,
                                                      int32_t *__restrict__ dci,
                                                      double *__restrict__ dval) {
  constexpr int kGroups = kBlock / G, kCap = G * E;
  __shared__ __align__(16) int32_t key[kGroups][kCap];
  const int lane = threadIdx.x % G, grp = threadIdx.x / G;
  const int32_t rows = W.list ? *W.nlist : W.nr;
  for (int32_t o = blockIdx.x * kGroups + grp; o < rows; o += gridDim.x * kGroups) {
    const int32_t q = W.list ? W.list[o] : o;
    const int32_t i = of ? of[q] : q;
    const int32_t b = rp[i], len = rp[i + 1] - b, d = drp[q];
    if (len > kCap) {
      if (lane == 0) W.ovf[atomicAdd(W.novf, 1)] = q;
      continue;
    }
    group_sync<G>();
    for (int32_t e = lane; e < len; e += G) {
      const int32_t c = ci[b + e];
      key[grp][e] = map ? map[c] : c;
    }
    // (kCap is a multiple of four)
    if (lane < 4 && (len & ~3) + lane >= len && len % 4) key[grp][(len & ~3) + lane] = INT32_MAX;
    group_sync<G>();
    if (len <= G)
      rank_rows<G, 1>(key[grp], len, lane, d, val + b, dci, dval);
    else
      rank_rows<G, 4>(key[grp], len, lane, d, val + b, dci, dval);
  }
}

// lengths of rows [b, e), or of the rows `of` of a CSR
__global__ void k_lengths(int32_t n, const int32_t *__restrict__ of, const int32_t *__restrict__ b,
                          const int32_t *__restrict__ e, int32_t *__restrict__ len) {
  const int32_t q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= n) return;
  const int32_t i = of ? of[q] : q;
  len[q] = e[i] - b[i];
}

// rows packed into a CSR, eight lanes per row
__global__ void k_pack_rows(int32_t n, Rows A, const int32_t *__restrict__ rp,
                            int32_t *__restrict__ ci, double *__restrict__ val) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int32_t i = (int32_t)(t / 8);
  if (t / 8 >= n) return;
  const int32_t b = A.b[i], len = A.e[i] - b, d = rp[i];
  for (int32_t k = (int32_t)(t % 8); k < len; k += 8) {
    ci[d + k] = A.ci[b + k];
    val[d + k] = A.val[b + k];
  }
}

// entries per column; then every entry's row and value in its column's part
// (in any order: the rows are sorted afterwards)
__global__ void k_column_count(int64_t nnz, const int32_t *__restrict__ ci,
                               int32_t *__restrict__ cnt) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < nnz) atomicAdd(&cnt[ci[k]], 1);
}

__global__ void k_column_fill(int32_t nr, const int32_t *__restrict__ rp,
                              const int32_t *__restrict__ ci, const double *__restrict__ val,
                              int32_t *__restrict__ next, int32_t *__restrict__ row,
                              double *__restrict__ v) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int32_t i = (int32_t)(t / 8);
  if (t / 8 >= nr) return;
  for (int32_t k = rp[i] + (int32_t)(t % 8), e = rp[i + 1]; k < e; k += 8) {
    const int32_t d = atomicAdd(&next[ci[k]], 1);
    row[d] = i;
    v[d] = val[k];
  }
}

__global__ void k_zero_i32(int64_t n, int32_t *a) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) a[i] = 0;
}

// The two lists a cascade of kernels hands its long rows on with; left() says
// how many the last one listed.
struct Lists {
  static constexpr int kSteps = 4;  // kernels in a cascade, at most
  int32_t nr;
  int32_t *rows[2] = {nullptr, nullptr}, *n = nullptr;
  int used = 0;
  amg_status init(Scratch &S, int32_t nrows) {
    nr = nrows;
    AMG_TRY(S.get(&rows[0], (size_t)nrows));
    AMG_TRY(S.get(&rows[1], (size_t)nrows));
    AMG_TRY(S.get(&n, kSteps));
    k_zero_i32<<<1, kSteps, 0, S.s>>>(kSteps, n);
    return AMG_OK;
  }
  Work next() {  // the first time all rows, then those the step before listed
    const int k = used++;
    return Work{nr, k ? rows[(k + 1) % 2] : nullptr, k ? n + k - 1 : nullptr, rows[k % 2], n + k};
  }
  amg_status left(hipStream_t s, int32_t *count) const {
    AMG_HIP(hipMemcpyAsync(count, n + used - 1, sizeof(int32_t), hipMemcpyDeviceToHost, s));
    AMG_HIP(hipStreamSynchronize(s));
    return AMG_OK;
  }
};

// blocks for `rows` rows of G lanes (the kernels stride over what is left)
template <int G>
int32_t row_blocks(int64_t rows) {
  const int64_t b = (rows * G + kBlock - 1) / kBlock;
  return (int32_t)(b < 1 ? 1 : (b > 65536 ? 65536 : b));
}
constexpr int kListBlocks = 1024;  // blocks of a kernel over listed rows

// Sorted rows of an nr-row CSR (see k_sort_rows) into drp (given) / dci /
// dval; *done = false if a row was too long.
amg_status sort_rows(Scratch &S, int32_t nr, int64_t nnz, const int32_t *of, const int32_t *map,
                     const int32_t *rp, const int32_t *ci, const double *val, const int32_t *drp,
                     int32_t *dci, double *dval, bool *done) {
  hipStream_t s = S.s;
  Lists L;
  AMG_TRY(L.init(S, nr));
  if (nnz <= 16 * (int64_t)nr)
    k_sort_rows<8, 4><<<row_blocks<8>(nr), kBlock, 0, s>>>(L.next(), of, map, rp, ci, val, drp,
                                                          dci, dval);
  else
    k_sort_rows<64, 8><<<row_blocks<64>(nr), kBlock, 0, s>>>(L.next(), of, map, rp, ci, val, drp,
                                                             dci, dval);
  k_sort_rows<256, 32><<<kListBlocks, kBlock, 0, s>>>(L.next(), of, map, rp, ci, val, drp, dci,
                                                      dval);
  AMG_HIP(hipGetLastError());
  int32_t left = 0;
  AMG_TRY(L.left(s, &left));
  *done = left == 0;
  return AMG_OK;
}

// Transpose of an nr x nc CSR, entries ascending in each row, into trp (nc +
// 1), tci, tval. A column of more than 8192 entries: by the sort of all.
amg_status transpose(amg_hierarchy *h, Scratch &S, int32_t nr, int32_t nc, int64_t nnz,
                     const int32_t *rp, const int32_t *ci, const double *val, int32_t *trp,
                     int32_t *tci, double *tval) {
  hipStream_t s = S.s;
  int32_t *cnt, *next, *row;
  double *v;
  AMG_TRY(S.get(&cnt, (size_t)nc));
  AMG_TRY(S.get(&next, (size_t)nc));
  AMG_TRY(S.get(&row, (size_t)nnz + 1));
  AMG_TRY(S.get(&v, (size_t)nnz + 1));
  k_zero_i32<<<grid(nc), kBlock, 0, s>>>(nc, cnt);
  k_column_count<<<grid(nnz), kBlock, 0, s>>>(nnz, ci, cnt);
  AMG_TRY(setup_scan(h, cnt, trp, nc));
  AMG_HIP(hipMemcpyAsync(next, trp, sizeof(int32_t) * nc, hipMemcpyDeviceToDevice, s));
  k_column_fill<<<grid((int64_t)nr * 8), kBlock, 0, s>>>(nr, rp, ci, val, next, row, v);
  bool done = false;
  AMG_TRY(sort_rows(S, nc, nnz, nullptr, nullptr, trp, row, v, trp, tci, tval, &done));
  if (done) return AMG_OK;
  uint64_t *key;
  AMG_TRY(S.get(&key, (size_t)nnz + 1));
  const int cb = bits_for(nr);
  k_transpose_keys<<<grid(nr), kBlock, 0, s>>>(nr, rp, ci, val, cb, key, v);
  AMG_TRY(radix_sort(S, (int32_t)nnz, cb + bits_for(nc), &key, &v));
  CsrOut T{trp, tci, tval, 0};
  return reduce_sorted(S, (int32_t)nnz, key, v, nc, cb, kept, &T);
}

// rows in a scratch room for `most` entries, row r's part starting at off[r]
amg_status rows_out(Scratch &S, int32_t nr, int64_t most, const int32_t *off, RowsOut *O) {
  O->off = off;
  AMG_TRY(S.get(&O->b, (size_t)nr));
  AMG_TRY(S.get(&O->e, (size_t)nr));
  AMG_TRY(S.get(&O->ci, (size_t)most + 1));
  AMG_TRY(S.get(&O->val, (size_t)most + 1));
  return AMG_OK;
}

// a result with gaps packed into a CSR
template <typename Alloc>
amg_status pack(amg_hierarchy *h, Scratch &S, int32_t nr, const Rows &R, Alloc alloc,
                CsrOut *out) {
  hipStream_t s = S.s;
  int32_t *len, *rp;
  AMG_TRY(S.get(&len, (size_t)nr));
  AMG_TRY(S.get(&rp, (size_t)nr + 1));
  k_lengths<<<grid(nr), kBlock, 0, s>>>(nr, nullptr, R.b, R.e, len);
  AMG_TRY(setup_scan(h, len, rp, nr));
  int32_t nnz = 0;
  AMG_HIP(hipMemcpyAsync(&nnz, rp + nr, sizeof(int32_t), hipMemcpyDeviceToHost, s));
  AMG_HIP(hipStreamSynchronize(s));
  AMG_TRY(alloc(&out->rp, (size_t)nr + 1, &out->ci, &out->val, (size_t)nnz));
  AMG_HIP(hipMemcpyAsync(out->rp, rp, sizeof(int32_t) * ((size_t)nr + 1), hipMemcpyDeviceToDevice,
                         s));
  k_pack_rows<<<grid((int64_t)nr * 8), kBlock, 0, s>>>(nr, R, out->rp, out->ci, out->val);
  AMG_HIP(hipGetLastError());
  out->nnz = nnz;
  return AMG_OK;
}

// sum_k coef_k B(src_k, :) for every row r < nr, k in [xp[r], xp[r + 1]);
// AMG_ERR_ARG for a row of more than 6144 columns, which no level can have: it
// is too long for the next level's sweeps and too wide for the coarsest. The lanes per row follow the mean row's terms: at
// 80^3 17 for A Pbar on the finest level (8 columns), about 200 for the coarse
// matrix (31) and over 1000 below.
amg_status combine_rows(amg_hierarchy *h, Scratch &S, int32_t nr, const int32_t *xp,
                        const int32_t *src, const double *coef, const Rows &B, Rows *out) {
  hipStream_t s = S.s;
  RowsOut R;
  int32_t *len, *off;
  unsigned long long *total;
  AMG_TRY(S.get(&len, (size_t)nr));
  AMG_TRY(S.get(&off, (size_t)nr + 1));
  AMG_TRY(S.get(&total, 1));
  k_zero_i32<<<1, 2, 0, s>>>(2, reinterpret_cast<int32_t *>(total));
  k_comb_len<<<grid((int64_t)nr * 8), kBlock, 0, s>>>(nr, xp, src, B, len, total);
  unsigned long long terms = 0;
  AMG_HIP(hipMemcpyAsync(&terms, total, sizeof(terms), hipMemcpyDeviceToHost, s));
  AMG_HIP(hipStreamSynchronize(s));
  if (terms >= (unsigned long long)(INT32_MAX - kSortTile)) return AMG_ERR_ARG;
  AMG_TRY(setup_scan(h, len, off, nr));
  AMG_TRY(rows_out(S, nr, (int64_t)terms, off, &R));
  Lists L;
  AMG_TRY(L.init(S, nr));
  const double mean = (double)terms / nr;
  if (mean <= 48.0)
    k_comb_rows<8, 32><<<row_blocks<8>(nr), kBlock, 0, s>>>(L.next(), xp, src, coef, B, R);
  else if (mean <= 512.0)
    k_comb_rows<16, 128><<<row_blocks<16>(nr), kBlock, 0, s>>>(L.next(), xp, src, coef, B, R);
  // over 4096 terms a row takes a block, unless the rows fill the card as waves
  // (8056 rows at 80^3: 0.34 ms as waves, 0.79 as blocks; 1019: 2.3 and 0.43)
  const bool waves = mean <= 4096.0 || nr >= 4096;
  if (waves) {
    const int32_t blocks = mean <= 512.0 ? kListBlocks : row_blocks<64>(nr);
    k_comb_rows<64, 512><<<blocks, kBlock, 0, s>>>(L.next(), xp, src, coef, B, R);
  }
  k_comb_rows<256, 2048><<<row_blocks<256>(waves ? kListBlocks : nr), kBlock, 0, s>>>(
      L.next(), xp, src, coef, B, R);
  k_comb_rows<256, 8192><<<kListBlocks, kBlock, 0, s>>>(L.next(), xp, src, coef, B, R);
  AMG_HIP(hipGetLastError());
  int32_t left = 0;
  AMG_TRY(L.left(s, &left));
  if (left) return AMG_ERR_ARG;
  *out = Rows{R.b, R.e, R.ci, R.val};
  return AMG_OK;
}

}  // namespace

amg_status smooth_level(amg_hierarchy *h, Level &F, int32_t nc, const int32_t *agg,
                        const double *p, int32_t **rp, int32_t **ci, double **val,
                        int64_t *nnz) {
  hipStream_t s = h->stream;
  const int32_t n = F.n;
  Scratch S(h);
  // hierarchy-owned and scratch destinations
  auto owned = [&](int32_t **r, size_t nr1, int32_t **c, double **v, size_t nz) -> amg_status {
    AMG_TRY(dalloc(h, r, nr1));
    AMG_TRY(dalloc(h, c, nz));
    AMG_TRY(dalloc(h, v, nz));
    return AMG_OK;
  };
  auto scratch = [&](int32_t **r, size_t nr1, int32_t **c, double **v, size_t nz) -> amg_status {
    AMG_TRY(S.get(r, nr1));
    AMG_TRY(S.get(c, nz));
    AMG_TRY(S.get(v, nz));
    return AMG_OK;
  };
  // omega
  unsigned long long *mx;
  AMG_TRY(S.get(&mx, 1));
  AMG_HIP(hipMemsetAsync(mx, 0, sizeof(unsigned long long), s));
  k_absnorm<<<grid(n), kBlock, 0, s>>>(n, F.rp, F.ci, F.val, mx);
  unsigned long long hmx = 0;
  AMG_HIP(hipMemcpyAsync(&hmx, mx, sizeof(hmx), hipMemcpyDeviceToHost, s));
  AMG_HIP(hipStreamSynchronize(s));
  double nrm;
  std::memcpy(&nrm, &hmx, sizeof(double));
  if (!(nrm > 0.0) || !std::isfinite(nrm)) return AMG_ERR_NOT_SPD;
  F.omega = 4.0 / (3.0 * nrm);
  // Pbar: one term per entry of A, summed per (i, J), then finished. No row is
  // longer than the sweeps before accepted (2048).
  CsrOut Pb;
  {
    RowsOut R;
    AMG_TRY(rows_out(S, n, F.nnz, F.rp, &R));
    Lists L;
    AMG_TRY(L.init(S, n));
    if (F.nnz <= 14 * (int64_t)n)
      k_pbar_rows<8, 2><<<row_blocks<8>(n), kBlock, 0, s>>>(L.next(), F.rp, F.ci, F.val, agg, p,
                                                           F.omega, R);
    else
      k_pbar_rows<64, 4><<<row_blocks<64>(n), kBlock, 0, s>>>(L.next(), F.rp, F.ci, F.val, agg, p,
                                                              F.omega, R);
    k_pbar_rows<256, 8><<<kListBlocks, kBlock, 0, s>>>(L.next(), F.rp, F.ci, F.val, agg, p,
                                                       F.omega, R);
    AMG_HIP(hipGetLastError());
    int32_t left = 0;
    AMG_TRY(L.left(s, &left));
    if (left) return AMG_ERR_ARG;
    AMG_TRY(pack(h, S, n, Rows{R.b, R.e, R.ci, R.val}, owned, &Pb));
  }
  F.pb_rp = Pb.rp;
  F.pb_ci = Pb.ci;
  F.pb_val = Pb.val;
  F.pb_nnz = Pb.nnz;
  // AP = A Pbar: row i combines the rows j of Pbar with the coefficients a_ij
  Rows AP{}, AcR{};
  AMG_TRY(combine_rows(h, S, n, F.rp, F.ci, F.val, Rows{Pb.rp, Pb.rp + 1, Pb.ci, Pb.val}, &AP));
  // Pbar^T (rows J, entries ascending i)
  CsrOut PT;
  AMG_TRY(scratch(&PT.rp, (size_t)nc + 1, &PT.ci, &PT.val, (size_t)Pb.nnz));
  AMG_TRY(transpose(h, S, n, nc, Pb.nnz, Pb.rp, Pb.ci, Pb.val, PT.rp, PT.ci, PT.val));
  // A_c = Pbar^T AP: row I combines the rows i of AP with Pbar(i, I)
  CsrOut Ac;
  AMG_TRY(combine_rows(h, S, nc, PT.rp, PT.ci, PT.val, AP, &AcR));
  AMG_TRY(pack(h, S, nc, AcR, owned, &Ac));
  int32_t *err;
  AMG_TRY(S.get(&err, 1));
  AMG_HIP(hipMemsetAsync(err, 0, sizeof(int32_t), s));
  if (Ac.nnz <= 24 * (int64_t)nc)
    k_mirror_lower<8><<<grid((int64_t)nc * 8), kBlock, 0, s>>>(nc, Ac.rp, Ac.ci, Ac.val, err);
  else
    k_mirror_lower<64><<<grid((int64_t)nc * 64), kBlock, 0, s>>>(nc, Ac.rp, Ac.ci, Ac.val, err);
  int32_t herr = 0;
  AMG_HIP(hipMemcpyAsync(&herr, err, sizeof(int32_t), hipMemcpyDeviceToHost, s));
  AMG_HIP(hipStreamSynchronize(s));
  if (herr) return AMG_ERR_ARG;
  *rp = Ac.rp;
  *ci = Ac.ci;
  *val = Ac.val;
  *nnz = Ac.nnz;
  return AMG_OK;
}

// row lengths of `of`'s rows of a CSR as the row pointer of the renumbered one
static amg_status permuted_row_ptr(amg_hierarchy *h, Scratch &S, int32_t n, const int32_t *of,
                                   const int32_t *rp, int32_t *out) {
  int32_t *len;
  AMG_TRY(S.get(&len, (size_t)n));
  k_lengths<<<grid(n), kBlock, 0, S.s>>>(n, of, rp, rp + 1, len);
  return setup_scan(h, len, out, n);
}

amg_status long_row_csr(amg_hierarchy *h, int32_t l, bool fp32) {
  hipStream_t s = h->stream;
  Level &F = h->lv[l];
  const int32_t n = F.n;
  const int32_t count = (int32_t)F.nnz;
  Scratch S(h);
  AMG_TRY(dalloc(h, &F.lr_rp, (size_t)n + 1));
  AMG_TRY(dalloc(h, &F.lr_ci, (size_t)count));
  AMG_TRY(dalloc(h, &F.lr_v64, (size_t)count));
  AMG_TRY(permuted_row_ptr(h, S, n, F.perm, F.rp, F.lr_rp));
  bool done = false;
  AMG_TRY(sort_rows(S, n, count, F.perm, F.iperm, F.rp, F.ci, F.val, F.lr_rp, F.lr_ci, F.lr_v64,
                    &done));
  if (!done) return AMG_ERR_ARG;  // (no row is longer than the sweeps accepted)
  if (fp32) {
    AMG_TRY(dalloc(h, &F.lr_v32, (size_t)count));
    k_demote_f64<<<grid(count), kBlock, 0, s>>>(count, F.lr_v64, F.lr_v32);
  }
  AMG_HIP(hipGetLastError());
  AMG_HIP(hipStreamSynchronize(s));
  return AMG_OK;
}

amg_status smooth_solve_format(amg_hierarchy *h, int32_t l, bool fp32) {
  hipStream_t s = h->stream;
  Level &F = h->lv[l];
  const Level &C = h->lv[l + 1];
  const int32_t n = F.n, nc = C.n;
  const int32_t count = (int32_t)F.pb_nnz;
  Scratch S(h);
  AMG_TRY(dalloc(h, &F.sp_rp, (size_t)n + 1));
  AMG_TRY(dalloc(h, &F.sp_ci, (size_t)count));
  AMG_TRY(dalloc(h, &F.sp_v64, (size_t)count));
  AMG_TRY(dalloc(h, &F.st_rp, (size_t)nc + 1));
  AMG_TRY(dalloc(h, &F.st_ci, (size_t)count));
  AMG_TRY(dalloc(h, &F.st_v64, (size_t)count));
  // Pbar by fine position, columns by coarse position; then its transpose
  bool done = false;
  AMG_TRY(permuted_row_ptr(h, S, n, F.perm, F.pb_rp, F.sp_rp));
  AMG_TRY(sort_rows(S, n, count, F.perm, C.iperm, F.pb_rp, F.pb_ci, F.pb_val, F.sp_rp, F.sp_ci,
                    F.sp_v64, &done));
  if (!done) return AMG_ERR_ARG;  // (no row is longer than the sweeps accepted)
  AMG_TRY(transpose(h, S, n, nc, count, F.sp_rp, F.sp_ci, F.sp_v64, F.st_rp, F.st_ci, F.st_v64));
  if (fp32) {
    AMG_TRY(dalloc(h, &F.sp_v32, (size_t)count));
    AMG_TRY(dalloc(h, &F.st_v32, (size_t)count));
    k_demote_f64<<<grid(count), kBlock, 0, s>>>(count, F.sp_v64, F.sp_v32);
    k_demote_f64<<<grid(count), kBlock, 0, s>>>(count, F.st_v64, F.st_v32);
  }
  AMG_HIP(hipGetLastError());
  AMG_HIP(hipStreamSynchronize(s));
  return AMG_OK;
}

}  // namespace amg
