// The t-SGNE neighbourhood graph G_knn,G (section 2.2, eq. (7)): nodes i and
// j are joined when one is among the first k nearest neighbours of the other
// on G, nearest by breadth-first search.  The first k neighbours of i are the
// k smallest nodes j != i under (hop distance from i, node id).
//
// One wave per source node.  Level 1 is the source's own row.  Every further
// level is enumerated in ascending id order by a wave-wide k-way merge of the
// frontier's adjacency rows (CSR rows are sorted): every lane owns up to U
// frontier rows with a cursor, the wave takes the minimum head, advances every
// cursor holding it (duplicates), and keeps it if it is not yet visited.  The
// visited set and the frontier are striped over the lanes' registers
// (membership is one ballot), so nothing is shared through memory inside a
// wave.  Each list leaves the kernel sorted by id.
//
// The lists are made symmetric by transposing them (a stable radix sort of
// the pairs by their target, whose sources stay ascending) and merging every
// node's list with its column of the transpose: an entry's place is its index
// plus the number of smaller entries of the other list, less the pairs chosen
// from both ends that come before it.
#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>

#include <algorithm>
#include <climits>
#include <vector>

#include "internal.h"

namespace tsgne {
namespace {

constexpr int kBlock = 256;
constexpr int kWavesPerBlock = kBlock / kWave;
constexpr int kMaxPerLane = 4;                 // frontier rows per lane
constexpr int kMaxK = kWave * kMaxPerLane;     // 256

// Minimum over the wave, to every lane: DPP row shifts and broadcasts leave it
// in the last lane (a shuffle goes through LDS; six of them were most of a
// merge step).
__device__ __forceinline__ int32_t wave_min(int32_t v) {
  v = min(v, __builtin_amdgcn_update_dpp(INT_MAX, v, 0x111, 0xF, 0xF, false));  // row_shr:1
  v = min(v, __builtin_amdgcn_update_dpp(INT_MAX, v, 0x112, 0xF, 0xF, false));
  v = min(v, __builtin_amdgcn_update_dpp(INT_MAX, v, 0x114, 0xF, 0xF, false));
  v = min(v, __builtin_amdgcn_update_dpp(INT_MAX, v, 0x118, 0xF, 0xF, false));
  v = min(v, __builtin_amdgcn_update_dpp(INT_MAX, v, 0x142, 0xA, 0xF, false));  // row_bcast:15
  v = min(v, __builtin_amdgcn_update_dpp(INT_MAX, v, 0x143, 0xC, 0xF, false));  // row_bcast:31
  return __builtin_amdgcn_readlane(v, kWave - 1);
}

// U = ceil(k / 64) rows and found nodes per lane.  Bound by instruction issue
// (some hundred merge steps per node): 0.83 ms for k = 90 on 100,000 nodes
// with shuffles and U = 4 for every k.
template <int U>
__global__ __launch_bounds__(kBlock) void k_knn_bfs(const int32_t* __restrict__ row_ptr,
                                                    const int32_t* __restrict__ col, int32_t n, int32_t k,
                                                    int32_t* __restrict__ out, int32_t* __restrict__ out_count) {
  // at most 2^30 / k nodes, so a wave's index fits
  const int32_t i = __builtin_amdgcn_readfirstlane((int32_t)(folded_block() * kWavesPerBlock + (threadIdx.x >> 6)));
  if (i >= n) return;
  const int lane = threadIdx.x & (kWave - 1);
  int32_t hit[U];                          // node found at index lane + 64 u
  int32_t fcur[U], fend[U], fhead[U];
  int32_t nfront[U];                       // the level being taken (next frontier)
  const int32_t b = row_ptr[i], deg = row_ptr[i + 1] - b;
  int32_t found = min(deg, k), taken = found;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int t = u * kWave + lane;
    hit[u] = t < found ? col[b + t] : -1;
    nfront[u] = hit[u];
  }
  while (taken > 0 && found < k) {
    // the level just taken becomes the frontier
#pragma unroll
    for (int u = 0; u < U; ++u) {
      fcur[u] = fend[u] = 0;
      fhead[u] = INT_MAX;
      if (u * kWave + lane < taken) {
        const int32_t v = nfront[u];
        fcur[u] = row_ptr[v];
        fend[u] = row_ptr[v + 1];
        fhead[u] = fcur[u] < fend[u] ? col[fcur[u]] : INT_MAX;
      }
    }
    taken = 0;
    for (;;) {
      int32_t h = fhead[0];
#pragma unroll
      for (int u = 1; u < U; ++u) h = min(h, fhead[u]);
      const int32_t m = wave_min(h);
      if (m == INT_MAX) break;  // level exhausted
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (fhead[u] == m) {
          ++fcur[u];
          fhead[u] = fcur[u] < fend[u] ? col[fcur[u]] : INT_MAX;
        }
      }
      if (m == i) continue;  // the source
      bool mine = false;
#pragma unroll
      for (int u = 0; u < U; ++u) mine |= (hit[u] == m);
      if (__ballot(mine) != 0) continue;  // visited on this or an earlier level
      // take m: found and next frontier (striped by index)
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (found == u * kWave + lane) hit[u] = m;
        if (taken == u * kWave + lane) nfront[u] = m;
      }
      ++taken;
      ++found;
      if (found == k) break;
    }
  }
  // in order of id: every node's rank among the found
  int32_t rank[U];
#pragma unroll
  for (int u = 0; u < U; ++u) rank[u] = 0;
#pragma unroll
  for (int v = 0; v < U; ++v) {
    const int32_t count = min(kWave, found - v * kWave);
    for (int32_t t = 0; t < count; ++t) {
      const int32_t other = __builtin_amdgcn_readlane(hit[v], t);
#pragma unroll
      for (int u = 0; u < U; ++u) rank[u] += other < hit[u] ? 1 : 0;
    }
  }
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (u * kWave + lane < found) out[(int64_t)i * k + rank[u]] = hit[u];
  if (lane == 0) out_count[i] = found;
}

// The chosen pairs by target and source; empty slots get the target n, which
// sorts last.
__global__ __launch_bounds__(kBlock) void k_knn_pairs(const int32_t* __restrict__ out,
                                                      const int32_t* __restrict__ count, int32_t n, int32_t k,
                                                      uint32_t* __restrict__ target, int32_t* __restrict__ source) {
  const uint32_t t = blockIdx.x * kBlock + threadIdx.x;  // n * k < 2^30
  if (t >= (uint32_t)n * (uint32_t)k) return;
  const int32_t i = (int32_t)(t / (uint32_t)k);
  target[t] = (int32_t)(t - (uint32_t)i * (uint32_t)k) < count[i] ? (uint32_t)out[t] : (uint32_t)n;
  source[t] = i;
}

// First index in sorted[lo, hi) whose value is not below x.
template <typename V>
__device__ __forceinline__ int64_t lower_bound_of(const V* __restrict__ sorted, int64_t lo, int64_t hi, V x) {
  while (lo < hi) {
    const int64_t mid = lo + (hi - lo) / 2;
    if (sorted[mid] < x) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// in_ptr[j] = first pair of target j, j <= n.
__global__ __launch_bounds__(kBlock) void k_knn_in_ptr(const uint32_t* __restrict__ target, int64_t slots, int32_t n,
                                                       int32_t* __restrict__ in_ptr) {
  const int32_t j = blockIdx.x * kBlock + threadIdx.x;
  if (j <= n) in_ptr[j] = (int32_t)lower_bound_of<uint32_t>(target, 0, slots, (uint32_t)j);
}

// One wave per node j, its list out[0, m) against the sorted sources that chose
// j: before[t] = sources below out[t] less the pairs chosen from both ends
// among out[0, t), both[t] = those pairs (both[m] all of them), size = the
// length of the union.
template <int U>
__global__ __launch_bounds__(kBlock) void k_knn_overlap(const int32_t* __restrict__ out,
                                                        const int32_t* __restrict__ count,
                                                        const int32_t* __restrict__ in_ptr,
                                                        const int32_t* __restrict__ source, int32_t n, int32_t k,
                                                        int32_t* __restrict__ before, int32_t* __restrict__ both,
                                                        int32_t* __restrict__ size) {
  const int32_t j = __builtin_amdgcn_readfirstlane((int32_t)(folded_block() * kWavesPerBlock + (threadIdx.x >> 6)));
  if (j > n) return;
  const int lane = threadIdx.x & (kWave - 1);
  if (j == n) {  // one more entry, so that a scan of the sizes ends with their sum
    if (lane == 0) size[n] = 0;
    return;
  }
  const int32_t m = count[j];
  const int64_t lo = in_ptr[j], hi = in_ptr[j + 1];
  int32_t shared = 0;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int t = u * kWave + lane;
    bool dup = false;
    int64_t at = lo;
    if (t < m) {
      const int32_t x = out[(int64_t)j * k + t];
      at = lower_bound_of<int32_t>(source, lo, hi, x);
      dup = at < hi && source[at] == x;
    }
    const unsigned long long mask = __ballot(dup);
    const int32_t ahead = shared + __popcll(mask & ((1ull << lane) - 1));
    if (t < m) {
      before[(int64_t)j * k + t] = (int32_t)(at - lo) - ahead;
      both[(int64_t)j * (k + 1) + t] = ahead;
    }
    shared += __popcll(mask);
  }
  if (lane == 0) {
    both[(int64_t)j * (k + 1) + m] = shared;
    size[j] = m + (int32_t)(hi - lo) - shared;
  }
}

// Entry t of the lists and pair t of the transpose into their places, and the
// row pointers to the caller (only now: a call that is refused because col is
// too small has written neither).
__global__ __launch_bounds__(kBlock) void k_knn_merge(const int32_t* __restrict__ out,
                                                      const int32_t* __restrict__ count,
                                                      const int32_t* __restrict__ before,
                                                      const int32_t* __restrict__ both,
                                                      const uint32_t* __restrict__ target,
                                                      const int32_t* __restrict__ source,
                                                      const int32_t* __restrict__ in_ptr, int32_t n, int32_t k,
                                                      const int32_t* __restrict__ row_ptr,
                                                      int32_t* __restrict__ row_ptr_out, int32_t* __restrict__ col) {
  const uint32_t t = blockIdx.x * kBlock + threadIdx.x;  // n * k < 2^30
  if (t >= (uint32_t)n * (uint32_t)k) return;
  if (t < (uint32_t)n) row_ptr_out[t] = row_ptr[t];
  if (t == 0) row_ptr_out[n] = row_ptr[n];
  const int32_t i = (int32_t)(t / (uint32_t)k), at = (int32_t)(t - (uint32_t)i * (uint32_t)k);
  if (at < count[i]) col[row_ptr[i] + at + before[t]] = out[t];
  const int32_t j = (int32_t)target[t];
  if (j == n) return;
  const int32_t x = source[t], m = count[j];
  const int32_t* __restrict__ list = out + (int64_t)j * k;
  const int32_t below = (int32_t)lower_bound_of<int32_t>(list, 0, m, x);
  if (below < m && list[below] == x) return;  // chosen from both ends: the list has it
  col[row_ptr[j] + ((int32_t)t - in_ptr[j]) - both[(int64_t)j * (k + 1) + below] + below] = x;
}

template <int U>
void launch_lists(const int32_t* row_ptr, const int32_t* col, int32_t n, int32_t k, int32_t* out, int32_t* count,
                  hipStream_t s) {
  hipLaunchKernelGGL(k_knn_bfs<U>, folded_grid(((int64_t)n + kWavesPerBlock - 1) / kWavesPerBlock, kBlock),
                     dim3(kBlock), 0, s, row_ptr, col, n, k, out, count);
}

template <int U>
void launch_overlap(const int32_t* out, const int32_t* count, const int32_t* in_ptr, const int32_t* source, int32_t n,
                    int32_t k, int32_t* before, int32_t* both, int32_t* size, hipStream_t s) {
  hipLaunchKernelGGL(k_knn_overlap<U>, folded_grid(((int64_t)n + 1 + kWavesPerBlock - 1) / kWavesPerBlock, kBlock),
                     dim3(kBlock), 0, s, out, count, in_ptr, source, n, k, before, both, size);
}

// Stable sort of the pairs by their target's low `bits` bits.  rocPRIM takes 8
// bits a pass over the pairs; where that leaves a third pass for one or two
// bits (n from 2^16 to 2^18), 9 bits a pass do in two: 9.0 M pairs of 100,000
// nodes 281 -> 177 us, a call with 1.05 M pairs 350 -> 308 us.  Up to 2^20 pairs
// it merges instead, which other settings only slow down (70,000 nodes, k =
// 10: 357 -> 375 us).
using NineBitPasses = rocprim::radix_sort_config<
    rocprim::default_config, rocprim::default_config,
    rocprim::radix_sort_onesweep_config<rocprim::kernel_config<1024, 12>, rocprim::kernel_config<512, 12>, 9,
                                         rocprim::block_radix_rank_algorithm::match>>;

hipError_t sort_pairs(void* temp, size_t& bytes, uint32_t* t0, uint32_t* t1, int32_t* s0, int32_t* s1, size_t count,
                      int bits, hipStream_t s) {
  if ((bits == 17 || bits == 18) && count > ((size_t)1 << 20))
    return rocprim::radix_sort_pairs<NineBitPasses>(temp, bytes, t0, t1, s0, s1, count, 0, bits, s);
  return rocprim::radix_sort_pairs(temp, bytes, t0, t1, s0, s1, count, 0, bits, s);
}

unsigned blocks_for(int64_t work) { return (unsigned)((work + kBlock - 1) / kBlock); }

}  // namespace

size_t validate_csr_bytes(int32_t, int64_t nnz) { return sizeof(int32_t) * (kCheckWords + (size_t)nnz); }

// Checks that (row_ptr, col) is a canonical symmetric CSR, in scratch of
// validate_csr_bytes(n, nnz): check words, row index.
tsgne_status validate_csr_in(int32_t n, int64_t nnz, const int32_t* row_ptr, const int32_t* col, void* scratch,
                             hipStream_t s, int32_t** row_of_out) {
  uint32_t* const check = static_cast<uint32_t*>(scratch);
  int32_t* const row_of = static_cast<int32_t*>(scratch) + kCheckWords;
  TSGNE_HIP(hipMemsetAsync(check, 0, sizeof(uint32_t) * kCheckWords, s), "clear check words");
  TSGNE_HIP(launch_check_rows(row_ptr, n, nnz, INT32_MAX, check, nullptr, nullptr, nullptr, nullptr, 0, s),
            "launch row check");
  // the column checks skip themselves when the row check failed
  TSGNE_HIP(launch_mirror(row_ptr, col, n, nnz, nullptr, row_of, check, s), "launch CSR check");
  uint32_t words[kCheckWords];
  TSGNE_HIP(hipMemcpyAsync(words, check, sizeof(words), hipMemcpyDeviceToHost, s), "read check words");
  TSGNE_HIP(hipStreamSynchronize(s), "synchronise CSR check");
  const uint32_t errors = check_errors(words);
  if (errors & kErrRowPtr) return fail(TSGNE_E_GRAPH, "row_ptr is not nondecreasing from 0 to nnz");
  if (errors) return fail(TSGNE_E_GRAPH, "CSR is not canonical and symmetric");
  if (row_of_out) *row_of_out = row_of;
  return TSGNE_OK;
}

}  // namespace tsgne

using namespace tsgne;

extern "C" {

tsgne_status tsgne_knn_graph(int32_t n, int64_t nnz, const int32_t* row_ptr_d, const int32_t* col_d, int32_t k,
                             int32_t* knn_row_ptr_d, int32_t* knn_col_d, int64_t knn_capacity, int64_t* knn_nnz,
                             void* stream) {
  if (!knn_nnz) return fail(TSGNE_E_INVAL, "knn_nnz is NULL");
  *knn_nnz = 0;
  if (n < 1) return fail(TSGNE_E_INVAL, "n must be >= 1");
  if (nnz < 0 || nnz >= ((int64_t)1 << 31)) return fail(TSGNE_E_INVAL, "nnz must lie in [0, 2^31)");
  if (k < 1 || k > kMaxK) return fail(TSGNE_E_INVAL, "k must lie in [1, 256]");
  if (!row_ptr_d || (nnz > 0 && !col_d) || !knn_row_ptr_d || (knn_capacity > 0 && !knn_col_d))
    return fail(TSGNE_E_INVAL, "null pointer");
  if ((int64_t)n * k * 2 >= ((int64_t)1 << 31)) return fail(TSGNE_E_INVAL, "n * k too large");
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  const int64_t slots = (int64_t)n * k;
  int bits = 1;  // targets 0 .. n
  while (((int64_t)1 << bits) <= n) ++bits;
  size_t sort_bytes = 0, scan_bytes = 0;
  TSGNE_HIP(sort_pairs(nullptr, sort_bytes, nullptr, nullptr, nullptr, nullptr, (size_t)slots, bits, s), "size sort");
  TSGNE_HIP(rocprim::exclusive_scan(nullptr, scan_bytes, (int32_t*)nullptr, (int32_t*)nullptr, 0, (size_t)n + 1,
                                    rocprim::plus<int32_t>(), s), "size scan");
  // scratch: lists | counts | in_ptr | sizes | row pointers | pairs before and after the sort
  // (the unsorted ones' place is taken by before and both) | rocPRIM's own;
  // the CSR check, which is done before any of them, from the same start.  One
  // allocation: with a second, small one before it the pool now and then gave
  // that one the large block and took 5 ms to make room for the other.
  size_t o = 0;
  auto place = [&](size_t bytes) {
    const size_t at = o;
    o += (bytes + 255) & ~(size_t)255;
    return at;
  };
  const size_t o_out = place(sizeof(int32_t) * (size_t)slots);
  const size_t o_count = place(sizeof(int32_t) * (size_t)n);
  const size_t o_in = place(sizeof(int32_t) * ((size_t)n + 1));
  const size_t o_size = place(sizeof(int32_t) * ((size_t)n + 1));
  const size_t o_ptr = place(sizeof(int32_t) * ((size_t)n + 1));
  const size_t o_t0 = place(sizeof(int32_t) * (size_t)slots);
  const size_t o_s0 = place(sizeof(int32_t) * ((size_t)slots + (size_t)n));
  const size_t o_t1 = place(sizeof(int32_t) * (size_t)slots);
  const size_t o_s1 = place(sizeof(int32_t) * (size_t)slots);
  const size_t o_temp = place(std::max<size_t>(std::max(sort_bytes, scan_bytes), 1));
  ScratchBlock tmp;
  tmp.s = s;
  TSGNE_HIP(scratch_alloc(&tmp.p, std::max(o, validate_csr_bytes(n, nnz)), s), "allocate neighbour lists");
  char* const base = static_cast<char*>(tmp.p);
  if (tsgne_status st = validate_csr_in(n, nnz, row_ptr_d, col_d, base, s)) return st;
  auto ints = [&](size_t at) { return reinterpret_cast<int32_t*>(base + at); };
  int32_t *out = ints(o_out), *count = ints(o_count), *in_ptr = ints(o_in), *size = ints(o_size), *ptr = ints(o_ptr);
  uint32_t *t0 = reinterpret_cast<uint32_t*>(base + o_t0), *t1 = reinterpret_cast<uint32_t*>(base + o_t1);
  int32_t *s0 = ints(o_s0), *s1 = ints(o_s1), *before = ints(o_t0), *both = ints(o_s0);
  void* const temp = base + o_temp;

  switch ((k + kWave - 1) / kWave) {
    case 1: launch_lists<1>(row_ptr_d, col_d, n, k, out, count, s); break;
    case 2: launch_lists<2>(row_ptr_d, col_d, n, k, out, count, s); break;
    case 3: launch_lists<3>(row_ptr_d, col_d, n, k, out, count, s); break;
    default: launch_lists<4>(row_ptr_d, col_d, n, k, out, count, s); break;
  }
  TSGNE_HIP(hipGetLastError(), "launch BFS");
  hipLaunchKernelGGL(k_knn_pairs, dim3(blocks_for(slots)), dim3(kBlock), 0, s, out, count, n, k, t0, s0);
  TSGNE_HIP(hipGetLastError(), "launch pairs");
  TSGNE_HIP(sort_pairs(temp, sort_bytes, t0, t1, s0, s1, (size_t)slots, bits, s), "sort pairs");
  hipLaunchKernelGGL(k_knn_in_ptr, dim3(blocks_for((int64_t)n + 1)), dim3(kBlock), 0, s, t1, slots, n, in_ptr);
  TSGNE_HIP(hipGetLastError(), "launch transpose");
  switch ((k + kWave - 1) / kWave) {
    case 1: launch_overlap<1>(out, count, in_ptr, s1, n, k, before, both, size, s); break;
    case 2: launch_overlap<2>(out, count, in_ptr, s1, n, k, before, both, size, s); break;
    case 3: launch_overlap<3>(out, count, in_ptr, s1, n, k, before, both, size, s); break;
    default: launch_overlap<4>(out, count, in_ptr, s1, n, k, before, both, size, s); break;
  }
  TSGNE_HIP(hipGetLastError(), "launch overlap");
  TSGNE_HIP(rocprim::exclusive_scan(temp, scan_bytes, size, ptr, 0, (size_t)n + 1, rocprim::plus<int32_t>(), s),
            "scan row sizes");
  int32_t total = 0;
  TSGNE_HIP(hipMemcpyAsync(&total, ptr + n, sizeof(int32_t), hipMemcpyDeviceToHost, s), "read size");
  TSGNE_HIP(hipStreamSynchronize(s), "synchronise row sizes");
  *knn_nnz = total;
  if (total > knn_capacity) return fail(TSGNE_E_INVAL, "knn_col capacity is smaller than the result (see *knn_nnz)");
  hipLaunchKernelGGL(k_knn_merge, dim3(blocks_for(slots)), dim3(kBlock), 0, s, out, count, before, both, t1, s1,
                     in_ptr, n, k, ptr, knn_row_ptr_d, knn_col_d);
  TSGNE_HIP(hipGetLastError(), "launch merge");
  TSGNE_HIP(hipStreamSynchronize(s), "synchronise kNN graph");
  return TSGNE_OK;
}

}  // extern "C"
