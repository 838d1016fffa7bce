// Affinity construction on the device: CSR check and mirror index, squared
// edge distances, per-row perplexity calibration and symmetrisation
// (section 2.1, eqs. (2)-(3), over graph neighbours as in section 2.2).
#include <cmath>

#include "internal.h"

namespace tsgne {
namespace {

constexpr int kBlock = 256;

// Row checks and counts without contended atomics (atomics on one address
// serialise across the whole device): per-block counts, one block turns
// them into offsets, then each block writes its selected rows in order.
__device__ __forceinline__ bool row_ok(const int32_t* __restrict__ row_ptr, int32_t i, int32_t n, int64_t nnz,
                                       int64_t* deg) {
  const int64_t a = row_ptr[i], b = row_ptr[i + 1];
  bool bad = b < a || a < 0 || b > nnz;
  if (i == 0 && a != 0) bad = true;
  if (i == n - 1 && b != nnz) bad = true;
  *deg = b - a;
  return !bad;
}

__global__ __launch_bounds__(kBlock) void k_row_counts(const int32_t* __restrict__ row_ptr, int32_t n, int64_t nnz,
                                                       int32_t threshold, uint32_t* __restrict__ err,
                                                       int2* __restrict__ partial) {
  const int32_t i = blockIdx.x * kBlock + threadIdx.x;
  bool nonempty = false, sel = false;
  if (i < n) {
    int64_t deg;
    if (!row_ok(row_ptr, i, n, nnz, &deg)) {
      atomicOr(err, kErrRowPtr);
    } else {
      nonempty = deg > 0;
      sel = deg > threshold;
    }
  }
  if (!partial) return;
  const int c_ne = __syncthreads_count(nonempty);
  const int c_sel = __syncthreads_count(sel);
  if (threadIdx.x == 0) partial[blockIdx.x] = make_int2(c_ne, c_sel);
}

constexpr int kScanBlock = 1024;
constexpr int kRowOfRun = 8;     // entries per thread in k_row_of
constexpr int kMirrorPer = 4;    // entries per thread in k_mirror

// One block: partial[b].y becomes the number of selected rows in blocks
// before b; counters = (rows with entries, selected rows).
__global__ __launch_bounds__(kScanBlock) void k_row_offsets(int2* __restrict__ partial, int32_t blocks,
                                                            int32_t* __restrict__ counters) {
  __shared__ int32_t s_sel[kScanBlock / kWave], s_ne[kScanBlock / kWave];
  const int t = threadIdx.x, lane = t & (kWave - 1), wv = t >> 6;
  const int32_t per = (blocks + kScanBlock - 1) / kScanBlock;
  const int32_t lo = min(blocks, t * per), hi = min(blocks, lo + per);
  int32_t sel = 0, ne = 0;
  for (int32_t b = lo; b < hi; ++b) {
    sel += partial[b].y;
    ne += partial[b].x;
  }
  int32_t inc = sel;
  for (int off = 1; off < kWave; off <<= 1) {
    const int32_t y = __shfl_up(inc, off, kWave);
    if (lane >= off) inc += y;
  }
  for (int off = kWave / 2; off > 0; off >>= 1) ne += __shfl_xor(ne, off, kWave);
  if (lane == kWave - 1) s_sel[wv] = inc;
  if (lane == 0) s_ne[wv] = ne;
  __syncthreads();
  int32_t base = 0, tot_sel = 0, tot_ne = 0;
  for (int w = 0; w < kScanBlock / kWave; ++w) {
    base += (w < wv) ? s_sel[w] : 0;
    tot_sel += s_sel[w];
    tot_ne += s_ne[w];
  }
  int32_t run = base + inc - sel;
  for (int32_t b = lo; b < hi; ++b) {
    const int32_t c = partial[b].y;
    partial[b].y = run;
    run += c;
  }
  if (t == 0) {
    counters[0] = tot_ne;
    counters[1] = tot_sel;
  }
}

__global__ __launch_bounds__(kBlock) void k_row_select(const int32_t* __restrict__ row_ptr, int32_t n, int64_t nnz,
                                                       int32_t threshold, const int2* __restrict__ partial,
                                                       int32_t* __restrict__ ids, int4* __restrict__ recs,
                                                       int32_t cap) {
  __shared__ int32_t s_wave[kBlock / kWave];
  const int32_t i = blockIdx.x * kBlock + threadIdx.x;
  const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x >> 6;
  bool sel = false;
  if (i < n) {
    int64_t deg;
    sel = row_ok(row_ptr, i, n, nnz, &deg) && deg > threshold;
  }
  const unsigned long long m = __ballot(sel);
  if (lane == 0) s_wave[wv] = __popcll(m);
  __syncthreads();
  int32_t pos = partial[blockIdx.x].y + __popcll(m & ((1ull << lane) - 1));
  for (int w = 0; w < wv; ++w) pos += s_wave[w];
  if (sel && pos < cap) {
    if (ids) ids[pos] = i;
    if (recs) recs[pos] = make_int4(i, row_ptr[i], row_ptr[i + 1], 0);
  }
}

// row_of[e] = the row of entry e: one block per kBlock rows shares out the
// entries of its rows.  Does nothing when the row check has failed, so it
// may be queued behind that check without waiting for its result.
__global__ __launch_bounds__(kBlock) void k_row_of(const int32_t* __restrict__ row_ptr, int32_t n,
                                                   int32_t* __restrict__ row_of, const uint32_t* __restrict__ err) {
  __shared__ int32_t s_ptr[kBlock + 1];
  if (*err & kErrRowPtr) return;
  const int32_t r0 = blockIdx.x * kBlock;
  const int32_t rows = min(kBlock, n - r0);
  for (int t = threadIdx.x; t <= rows; t += kBlock) s_ptr[t] = row_ptr[r0 + t];
  __syncthreads();
  const int32_t first = s_ptr[0], end = s_ptr[rows];
  // kRowOfRun consecutive entries per thread: one search, then a walk
  for (int32_t e0 = first + threadIdx.x * kRowOfRun; e0 < end; e0 += kBlock * kRowOfRun) {
    int lo = 0, hi = rows;  // s_ptr[lo] <= e0 < s_ptr[hi]
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (s_ptr[mid] <= e0) lo = mid;
      else hi = mid;
    }
#pragma unroll
    for (int k = 0; k < kRowOfRun; ++k) {
      const int32_t e = e0 + k;
      if (e < end) {
        while (s_ptr[lo + 1] <= e) ++lo;  // stops below rows since e < s_ptr[rows]
        row_of[e] = r0 + lo;
      }
    }
  }
}

// kMirrorPer entries per thread (row from row_of): the checks on each
// entry's column and the position of the reverse entry, with the binary
// searches of the entries advancing together so that their loads overlap.
// Does nothing when the row check has failed.
//
// Bound by the searches' chains of dependent gathers.  Of the two entries of
// an edge only the one whose far row is the shorter (of equal ones: the lower)
// searches it, and fills in both positions.  Searched entries that are found
// have distinct reverse entries, none of them searched, so when there are as
// many searched as others the pattern is symmetric: check's counters take the
// difference.  At 300,000 nodes and 2.0 M entries a search for every entry
// (hubs' rows are the ones met most) took 67 us, this 36 where only the check
// is wanted and 66 with the positions, half of them scattered writes; a search
// for every entry with its loads together 83.
__global__ __launch_bounds__(kBlock) void k_mirror(const int32_t* __restrict__ row_ptr,
                                                   const int32_t* __restrict__ col, int32_t n, int64_t nnz,
                                                   int32_t* __restrict__ mirror, const int32_t* __restrict__ row_of,
                                                   uint32_t* __restrict__ check) {
  if (check[0] & kErrRowPtr) return;  // row_of is not filled after a failed row check
  const int64_t e0 = (int64_t)blockIdx.x * kBlock * kMirrorPer + threadIdx.x;
  // Without branches (entries past the end and columns out of range are
  // clamped), so that the entries' loads go out together.
  int32_t row[kMirrorPer], far[kMirrorPer], before[kMirrorPer];
#pragma unroll
  for (int k = 0; k < kMirrorPer; ++k) {
    const int64_t e = min(e0 + (int64_t)k * kBlock, nnz - 1);
    row[k] = row_of[e];
    far[k] = col[e];
    before[k] = col[max(e - 1, (int64_t)0)];
  }
  int32_t own[kMirrorPer], own_end[kMirrorPer], lo[kMirrorPer], hi[kMirrorPer];
#pragma unroll
  for (int k = 0; k < kMirrorPer; ++k) {
    const int32_t j = min(max(far[k], 0), n - 1);
    own[k] = row_ptr[row[k]];
    own_end[k] = row_ptr[row[k] + 1];
    lo[k] = row_ptr[j];
    hi[k] = row_ptr[j + 1];
  }
  int32_t key[kMirrorPer];  // the row to find in [lo, hi), or -1
  uint32_t bits = 0;
  int32_t balance = 0;
#pragma unroll
  for (int k = 0; k < kMirrorPer; ++k) {
    const int64_t e = e0 + (int64_t)k * kBlock;
    const int32_t i = row[k], j = far[k];
    const int32_t di = own_end[k] - own[k], dj = hi[k] - lo[k];
    const bool live = e < nnz, ok = live & (j >= 0) & (j < n), edge = ok & (j != i);
    const bool search = edge & ((dj < di) | ((dj == di) & (j < i)));
    bits |= (live & !ok ? kErrColRange : 0u) | (ok & (j == i) ? kErrSelfLoop : 0u) |
            (ok & (e > own[k]) & (before[k] >= j) ? kErrOrder : 0u);
    balance += search ? 1 : edge ? -1 : 0;
    key[k] = search ? i : -1;
    hi[k] = search ? hi[k] : lo[k];
  }
  bool any = true;
  while (any) {
    any = false;
    int32_t c[kMirrorPer], mid[kMirrorPer];
#pragma unroll
    for (int k = 0; k < kMirrorPer; ++k) {
      mid[k] = lo[k] + (hi[k] - lo[k]) / 2;
      c[k] = lo[k] < hi[k] ? col[mid[k]] : 0;
    }
#pragma unroll
    for (int k = 0; k < kMirrorPer; ++k) {
      if (lo[k] >= hi[k]) continue;
      if (c[k] == key[k]) {
        if (mirror) {
          const int64_t e = e0 + (int64_t)k * kBlock;
          mirror[e] = mid[k];
          mirror[mid[k]] = (int32_t)e;
        }
        key[k] = -1;
        hi[k] = lo[k];
      } else {
        if (c[k] < key[k]) lo[k] = mid[k] + 1;
        else hi[k] = mid[k];
        any |= lo[k] < hi[k];
      }
    }
  }
#pragma unroll
  for (int k = 0; k < kMirrorPer; ++k) {
    if (key[k] >= 0) bits |= kErrAsym;  // searched and not found
  }
  for (int off = kWave / 2; off > 0; off >>= 1) balance += __shfl_xor(balance, off, kWave);
  const int wave = (int)blockIdx.x * (kBlock / kWave) + (int)(threadIdx.x >> 6);
  if ((threadIdx.x & (kWave - 1)) == 0 && balance != 0)
    atomicAdd(&check[(1 + wave % kCheckCounters) * kCheckStride], (uint32_t)balance);
  if (bits) atomicOr(check, bits);
}

// D_e = ||x_i - x_j||^2 (the squared distance of eq. (2)) from FP32 rows,
// accumulated in FP64.  Sixteen lanes per entry stride over the d
// coordinates (consecutive lanes read consecutive floats of a row).
//
// Bound by the rows gathered (d = 128, 800,000 entries: 820 MB, mostly from
// beyond the L2).  An edge's two entries have the same distance to the last
// bit, so the first of them computes it for both, and a group of lanes takes
// two entries, their loads in groups: 92 -> 46 us.
constexpr int kDistLanes = 16;
constexpr int kDistPer = 2;  // entries per group of lanes

__global__ __launch_bounds__(kBlock) void k_sqdist(const int32_t* __restrict__ row_of, const int32_t* __restrict__ col,
                                                   const int32_t* __restrict__ mirror, int64_t nnz,
                                                   const float* __restrict__ X, int32_t d, double* __restrict__ D) {
  constexpr int64_t kGroups = kBlock / kDistLanes;
  const int64_t e0 = (int64_t)folded_block() * kGroups * kDistPer + threadIdx.x / kDistLanes;
  const int sub = threadIdx.x & (kDistLanes - 1);
  int32_t other[kDistPer], row[kDistPer], far[kDistPer];
#pragma unroll
  for (int q = 0; q < kDistPer; ++q) {
    const int64_t e = min(e0 + q * kGroups, nnz - 1);
    other[q] = mirror[e];
    row[q] = row_of[e];
    far[q] = col[e];
  }
#pragma unroll
  for (int q = 0; q < kDistPer; ++q) {
    const int64_t e = e0 + q * kGroups;
    const bool mine = e < nnz && e < other[q];  // the same for all lanes of the group
    double acc = 0.0;
    if (mine) {
      const float* xi = X + (int64_t)row[q] * d;
      const float* xj = X + (int64_t)far[q] * d;
      constexpr int U = 4;  // coordinates per lane whose loads are issued together
      int32_t k = sub;
      for (; k + (U - 1) * kDistLanes < d; k += U * kDistLanes) {
        float a[U], b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          a[u] = xi[k + u * kDistLanes];
          b[u] = xj[k + u * kDistLanes];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const double diff = (double)a[u] - (double)b[u];
          acc = fma(diff, diff, acc);
        }
      }
      for (; k < d; k += kDistLanes) {
        const double diff = (double)xi[k] - (double)xj[k];
        acc = fma(diff, diff, acc);
      }
    }
    for (int off = kDistLanes / 2; off > 0; off >>= 1) acc += __shfl_xor(acc, off, kDistLanes);
    if (mine && sub == 0) {
      D[e] = acc;
      D[other[q]] = acc;
    }
  }
}

// ---------------------------------------------------------------------------
// Per-row calibration by a group of LANES lanes: 16 for rows of at most
// kHeavyDegree entries, a wave for longer ones.  Entries are strided over the
// lanes, sums reduced with butterflies so that every lane of the group holds
// the same bits and takes the same branch.
// ---------------------------------------------------------------------------

constexpr int kCalLanes = 16;
// Steps of the search at most.  Squared distances of FP32 coordinates span up
// to 1e166, 280 steps of a factor of 4; with 200, rows that span 1e121 and more
// were left short of their beta.  Ordinary rows take 5 to 8.
constexpr int kCalSteps = 1000;

template <int LANES>
__device__ __forceinline__ double group_sum(double v) {
  for (int off = LANES / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, LANES);
  return v;
}

template <int LANES>
__device__ __forceinline__ double group_min(double v) {
  for (int off = LANES / 2; off > 0; off >>= 1) v = fmin(v, __shfl_xor(v, off, LANES));
  return v;
}

// beta_i = 1/(2 sigma_i^2) such that the row's entropy is log(perp) (section
// 2.1: sigma_i is found by a search).  With p_k = exp(-beta delta_k) / S the
// entropy in nats is H = log(S) + beta <delta>, and dH / d(log beta) =
// -beta^2 Var(delta): Newton's iteration on log(beta) from 1/mean(delta), inside
// the bracket that the signs of H - log(perp) give, and doubling, halving or
// bisecting wherever a step would leave it.  It ends when the bracket is 1e-13
// of beta wide or the steps no longer shrink, at the rounding of H: log(beta) is
// then within that rounding over beta^2 Var(delta) of the root, which is more
// than 1e-13 where H is flat, that is, where p hardly depends on beta.
//
// Bound by the FP64 exponentials.  One thread per row and bisection alone took
// 1.66 ms at 100,000 nodes (perplexity 30, 45 to 50 evaluations of up to 64
// entries one after the other in the few lanes whose rows need any); 5 to 8
// evaluations of 4 entries a lane are left.
template <int LANES>
__device__ void calibrate_row(const double* __restrict__ Dr, int64_t deg, double perp, double* __restrict__ pc,
                              double* __restrict__ beta_out, int lane) {
  if (deg == 0) {
    if (lane == 0) *beta_out = 0.0;
    return;
  }
  if ((double)deg <= perp) {  // target entropy out of reach: uniform row
    const double u = 1.0 / (double)deg;
    for (int64_t k = lane; k < deg; k += LANES) pc[k] = u;
    if (lane == 0) *beta_out = 0.0;
    return;
  }
  double dmin = INFINITY;
  for (int64_t k = lane; k < deg; k += LANES) dmin = fmin(dmin, Dr[k]);
  dmin = group_min<LANES>(dmin);
  double ties = 0.0, mean = 0.0;
  for (int64_t k = lane; k < deg; k += LANES) {
    ties += (Dr[k] == dmin) ? 1.0 : 0.0;
    mean += Dr[k] - dmin;
  }
  ties = group_sum<LANES>(ties);
  mean = group_sum<LANES>(mean) / (double)deg;
  if (ties >= perp) {  // uniform over the nearest neighbours (beta -> infinity)
    const double u = 1.0 / ties;
    for (int64_t k = lane; k < deg; k += LANES) pc[k] = (Dr[k] == dmin) ? u : 0.0;
    if (lane == 0) *beta_out = INFINITY;
    return;
  }
  const double target = log(perp);
  double lo = 0.0, hi = INFINITY, bt = 1.0 / mean, last = INFINITY;
  for (int it = 0; it < kCalSteps; ++it) {
    double S = 0.0, T = 0.0, V = 0.0;
    for (int64_t k = lane; k < deg; k += LANES) {
      const double dk = Dr[k] - dmin;
      const double ek = exp(-bt * dk);
      S += ek;
      T += dk * ek;
      V += dk * (dk * ek);
    }
    S = group_sum<LANES>(S);
    T = group_sum<LANES>(T) / S;
    V = group_sum<LANES>(V) / S - T * T;
    const double over = log(S) + bt * T - target;
    if (over > 0.0) lo = bt; else hi = bt;
    if (hi < INFINITY && hi - lo <= 1e-13 * hi) break;
    // of log(beta), at most a factor of 4: far off, H is flat
    const double step = fmax(-1.4, fmin(1.4, over / (bt * bt * V)));
    // at the rounding of H itself steps stop shrinking
    const bool settled = fabs(step) <= 1e-14 || (fabs(step) < 1e-9 && fabs(step) > 0.25 * last);
    last = fabs(step);
    const double next = bt * exp(step);
    const bool inside = next > lo && next < hi;
    if (settled) {
      if (inside) bt = next;
      break;
    }
    bt = inside && V > 0.0 ? next : hi == INFINITY ? 2.0 * bt : lo == 0.0 ? 0.5 * bt : 0.5 * (lo + hi);
  }
  double S = 0.0;
  for (int64_t k = lane; k < deg; k += LANES) S += exp(-bt * (Dr[k] - dmin));
  S = group_sum<LANES>(S);
  for (int64_t k = lane; k < deg; k += LANES) pc[k] = exp(-bt * (Dr[k] - dmin)) / S;
  if (lane == 0) *beta_out = bt;
}

// The first heavy_blocks workgroups take the heavy rows, a wave each, the
// others the light ones: hubs' rows, the longest chains, start first, and run
// beside the rest (as two launches 56 + 47 us at 100,000 nodes, as one 60).
__global__ __launch_bounds__(kBlock) void k_calibrate(const int32_t* __restrict__ row_ptr, int32_t n,
                                                      const int32_t* __restrict__ heavy, int32_t n_heavy,
                                                      int32_t heavy_blocks, const double* __restrict__ D, double perp,
                                                      double* __restrict__ pcond, double* __restrict__ beta) {
  const int32_t block = (int32_t)folded_block();  // at most 2^31 / 16 + heavy_blocks
  if (block < heavy_blocks) {
    const int32_t w = __builtin_amdgcn_readfirstlane((int32_t)(block * (kBlock / kWave) + (threadIdx.x >> 6)));
    if (w >= n_heavy) return;
    const int32_t i = heavy[w];
    const int64_t b = row_ptr[i], deg = (int64_t)row_ptr[i + 1] - b;
    calibrate_row<kWave>(D + b, deg, perp, pcond + b, beta + i, (int)(threadIdx.x & (kWave - 1)));
    return;
  }
  const int64_t i = ((int64_t)(block - heavy_blocks) * kBlock + threadIdx.x) / kCalLanes;
  if (i >= n) return;  // whole groups
  const int64_t b = row_ptr[i], deg = (int64_t)row_ptr[i + 1] - b;
  if (deg > kHeavyDegree) return;
  calibrate_row<kCalLanes>(D + b, deg, perp, pcond + b, beta + i, (int)(threadIdx.x & (kCalLanes - 1)));
}

// p_ij = (p_{j|i} + p_{i|j}) / S, eq. (3), with S = 2 * (non-isolated nodes).
__global__ __launch_bounds__(kBlock) void k_symmetrise(const int32_t* __restrict__ mirror, int64_t nnz,
                                                       const double* __restrict__ pcond, double S,
                                                       float* __restrict__ P) {
  const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (e >= nnz) return;
  P[e] = (float)((pcond[e] + pcond[mirror[e]]) / S);
}

inline unsigned blocks_for(int64_t work) { return (unsigned)((work + kBlock - 1) / kBlock); }

}  // namespace

int64_t row_check_blocks(int32_t n) { return ((int64_t)n + kBlock - 1) / kBlock; }

hipError_t launch_check_rows(const int32_t* row_ptr, int32_t n, int64_t nnz, int32_t threshold, uint32_t* check,
                             int32_t* counters, int2* partial, int32_t* ids, int4* recs, int32_t cap,
                             hipStream_t s) {
  const int32_t blocks = (int32_t)row_check_blocks(n);
  hipLaunchKernelGGL(k_row_counts, dim3(blocks), dim3(kBlock), 0, s, row_ptr, n, nnz, threshold, check,
                     counters ? partial : nullptr);
  if (!counters) return hipGetLastError();
  hipLaunchKernelGGL(k_row_offsets, dim3(1), dim3(kScanBlock), 0, s, partial, blocks, counters);
  hipLaunchKernelGGL(k_row_select, dim3(blocks), dim3(kBlock), 0, s, row_ptr, n, nnz, threshold, partial, ids, recs,
                     cap);
  return hipGetLastError();
}

hipError_t launch_mirror(const int32_t* row_ptr, const int32_t* col, int32_t n, int64_t nnz, int32_t* mirror,
                         int32_t* row_of, uint32_t* check, hipStream_t s) {
  if (nnz == 0) return hipSuccess;
  hipLaunchKernelGGL(k_row_of, dim3((unsigned)row_check_blocks(n)), dim3(kBlock), 0, s, row_ptr, n, row_of, check);
  hipLaunchKernelGGL(k_mirror, dim3(blocks_for((nnz + kMirrorPer - 1) / kMirrorPer)), dim3(kBlock), 0, s, row_ptr, col,
                     n, nnz, mirror, row_of, check);
  return hipGetLastError();
}

hipError_t launch_sqdist(const int32_t* row_of, const int32_t* col, const int32_t* mirror, int64_t nnz,
                         const float* X, int32_t d, double* D, hipStream_t s) {
  if (nnz == 0) return hipSuccess;
  hipLaunchKernelGGL(k_sqdist, folded_grid(blocks_for((nnz + kDistPer - 1) / kDistPer * kDistLanes), kBlock),
                     dim3(kBlock), 0, s, row_of, col, mirror, nnz, X, d, D);
  return hipGetLastError();
}

hipError_t launch_calibrate(const int32_t* row_ptr, int32_t n, const int32_t* heavy, int32_t n_heavy, const double* D,
                            double perplexity, double* pcond, double* beta, hipStream_t s) {
  const int32_t heavy_blocks = (n_heavy + kBlock / kWave - 1) / (kBlock / kWave);
  hipLaunchKernelGGL(k_calibrate, folded_grid(heavy_blocks + (int64_t)blocks_for((int64_t)n * kCalLanes), kBlock),
                     dim3(kBlock), 0, s, row_ptr, n, heavy, n_heavy, heavy_blocks, D, perplexity, pcond, beta);
  return hipGetLastError();
}

hipError_t launch_symmetrise(const int32_t* mirror, int64_t nnz, const double* pcond, double S, float* P,
                             hipStream_t s) {
  if (nnz == 0) return hipSuccess;
  hipLaunchKernelGGL(k_symmetrise, dim3(blocks_for(nnz)), dim3(kBlock), 0, s, mirror, nnz, pcond, S, P);
  return hipGetLastError();
}

}  // namespace tsgne
