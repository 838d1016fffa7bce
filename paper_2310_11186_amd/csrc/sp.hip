// ShortestPath graph embedding (section 2.3, eq. (8)): X[i][j] is the hop
// distance from node i to target t_j when it is at most l0, otherwise l0 + 1
// (also when t_j cannot be reached).
//
// All d breadth-first searches advance together, level-synchronously, with
// one bit per target.  Per node v the device holds
//   vis[v]    -- targets that have reached v (W words of 32 bits),
//   F[v]      -- targets that reached v at the previous level (the frontier;
//                meaningful only if v's activity bit of that level is set),
//   plane_k[v]-- bit k of the hop distance, for each target (bit-sliced).
// Level L pulls: N = (OR of F[u] over the neighbours u of v) & ~vis[v]; the
// bits of N get distance L, written into the planes where L has a one bit.
// A node every target has reached reads nothing.  The searches stop at
// level floor(l0) or when a level finds nothing.  A final pass decodes the
// planes into X with one coalesced write of every element, so X is written
// once and never read.
//
// Level activity is kept in a ring of three flag sets (levels L-1, L, L+1),
// each spread over 64 cache lines so that the waves reporting activity do
// not all write one line.  Levels are launched in chunks; a launched level
// whose predecessor found nothing returns at once.  The host waits once per
// chunk and reads the last flag set then; the CSR check's result comes with the
// first (a bad graph's levels find no activity to start from).  The first
// chunk, in which most graphs' searches end, has the final pass behind it,
// which writes nothing if a search goes on; after later chunks the pass waits
// for the host.  Behind every chunk, its reads of the state made a path of
// 100,000 nodes with 256 targets (316 levels) take 3.87 ms and a mesh of 302,500
// (777 levels) 18.7, now 3.32 and 16.3.
#include <algorithm>
#include <cmath>
#include <vector>

#include "internal.h"

namespace tsgne {
namespace {

constexpr int kBlock = 256;
constexpr int kLightMax = 256;        // larger degrees are split into chunks
constexpr int kChunk = 1024;          // edges per chunk, a wave's work
constexpr int kChunkBlock = 1024;     // threads of the chunk-table kernel

// Edges in flight per thread: as many as the registers for their frontier
// words allow.
template <int W>
constexpr int unroll_for() {
  return W <= 2 ? 8 : 4;
}
constexpr int kWavesPerBlock = kBlock / kWave;
constexpr int kListShift = 20;        // a block's light nodes have at most kBlock * kLightMax edges
static_assert(kBlock * kLightMax < (1 << kListShift) && kBlock < (1 << (31 - kListShift)), "packed sums");
constexpr int kSlots = 64;            // flags per level
constexpr int kSlotStride = 32;       // ints: one flag per 128-byte line
constexpr int kRing = 3;
constexpr int kFlagInts = kSlots * kSlotStride;
constexpr int kMaxTargets = 256;
constexpr int kLevelsPerCheck = 12;
constexpr int kHeavyBlocks = 1024;    // at most so many workgroups share the chunks of heavy nodes
constexpr uint32_t kErrTarget = 1u << 16;  // in the check's error word

// Bits of word w that belong to one of the d targets.
__device__ __forceinline__ uint32_t word_mask(int w, int32_t d) {
  const int lo = 32 * w;
  if (d >= lo + 32) return ~0u;
  if (d <= lo) return 0u;
  return (1u << (d - lo)) - 1u;
}

template <int W>
__device__ __forceinline__ void load_words(const uint32_t* __restrict__ p, uint32_t (&m)[W]) {
  if constexpr (W >= 4) {
#pragma unroll
    for (int q = 0; q < W / 4; ++q) {
      const uint4 v = reinterpret_cast<const uint4*>(p)[q];
      m[4 * q] = v.x;
      m[4 * q + 1] = v.y;
      m[4 * q + 2] = v.z;
      m[4 * q + 3] = v.w;
    }
  } else if constexpr (W == 2) {
    const uint2 v = *reinterpret_cast<const uint2*>(p);
    m[0] = v.x;
    m[1] = v.y;
  } else {
    m[0] = p[0];
  }
}

template <int W>
__device__ __forceinline__ void store_words(uint32_t* __restrict__ p, const uint32_t (&m)[W]) {
  if constexpr (W >= 4) {
#pragma unroll
    for (int q = 0; q < W / 4; ++q)
      reinterpret_cast<uint4*>(p)[q] = make_uint4(m[4 * q], m[4 * q + 1], m[4 * q + 2], m[4 * q + 3]);
  } else if constexpr (W == 2) {
    *reinterpret_cast<uint2*>(p) = make_uint2(m[0], m[1]);
  } else {
    p[0] = m[0];
  }
}

// Search state of one level: the previous level's frontier (words and
// activity bits) is read, this level's is written over the one before; the
// bits of the level to come are cleared.
struct SpState {
  const uint32_t* fcur;     // [n][W] frontier of the previous level
  uint32_t* fnext;          // [n][W] frontier of this level
  const uint32_t* bits_cur; // bit v: fcur[v] is of the previous level and not empty
  uint32_t* bits_next;
  uint32_t* bits_clear;
  uint32_t* vis;            // [n][W]
  uint32_t* planes;         // [n_planes][n][W]
  int64_t plane_stride;
  int n_planes;
};

// True in every lane if the check has found an error.  Called by whole waves.
__device__ __forceinline__ bool csr_failed(const uint32_t* __restrict__ check) {
  const int lane = threadIdx.x & (kWave - 1);
  uint32_t sum = lane < kCheckCounters ? check[(1 + lane) * kCheckStride] : 0u;
  for (int off = kWave / 2; off > 0; off >>= 1) sum += __shfl_xor(sum, off, kWave);
  return (check[0] | sum) != 0;
}

// Level 0: every target has reached itself.  vis, F0 and the planes are zero.
__global__ __launch_bounds__(kBlock) void k_sp_init(const int32_t* __restrict__ targets, int32_t d, int32_t n,
                                                    int W, uint32_t* __restrict__ vis, uint32_t* __restrict__ f0,
                                                    uint32_t* __restrict__ bits0, int32_t* __restrict__ flags,
                                                    uint32_t* __restrict__ check) {
  const int32_t j = blockIdx.x * kBlock + threadIdx.x;
  const bool failed = csr_failed(check);
  if (j < kRing * kFlagInts) flags[j] = (j == 0 && !failed) ? 1 : 0;  // level 0 counts as active
  if (j >= d) return;
  const int32_t t = targets[j];
  if (t < 0 || t >= n) {
    atomicOr(check, kErrTarget);
    return;
  }
  const uint32_t bit = 1u << (j & 31);
  atomicOr(&vis[(int64_t)t * W + (j >> 5)], bit);  // targets may repeat
  atomicOr(&f0[(int64_t)t * W + (j >> 5)], bit);
  atomicOr(&bits0[t >> 5], 1u << (t & 31));
}

// The new bits of node v at this level, given the OR of its neighbours'
// frontier words: frontier, visited set and distance planes.  Called by one
// lane per node.  Returns whether anything was new.
template <int W>
__device__ __forceinline__ bool settle(int32_t v, const uint32_t (&acc)[W], const uint32_t (&seen)[W],
                                       const SpState& st, int32_t level) {
  uint32_t nw[W];
  uint32_t any = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    nw[w] = acc[w] & ~seen[w];
    any |= nw[w];
  }
  if (any == 0) return false;
  store_words<W>(st.fnext + (int64_t)v * W, nw);
  uint32_t nv[W];
#pragma unroll
  for (int w = 0; w < W; ++w) nv[w] = seen[w] | nw[w];
  store_words<W>(st.vis + (int64_t)v * W, nv);
  // planes[k] |= new bits where the level has a one bit; loads in groups
  // of four, ahead of their stores
  for (int k0 = 0; k0 < st.n_planes; k0 += 4) {
    uint32_t pw[4][W];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int k = k0 + q;
      if (k < st.n_planes && ((level >> k) & 1))
        load_words<W>(st.planes + k * st.plane_stride + (int64_t)v * W, pw[q]);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int k = k0 + q;
      if (k < st.n_planes && ((level >> k) & 1)) {
#pragma unroll
        for (int w = 0; w < W; ++w) pw[q][w] |= nw[w];
        store_words<W>(st.planes + k * st.plane_stride + (int64_t)v * W, pw[q]);
      }
    }
  }
  return true;
}

// Exclusive prefix sum over the block (kBlock threads); *total gets the sum.
__device__ __forceinline__ int32_t block_exclusive_scan(int32_t x, int32_t* s_wave, int32_t* total) {
  const int lane = threadIdx.x & (kWave - 1), wv = threadIdx.x >> 6;
  int32_t inc = x;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int32_t y = __shfl_up(inc, off, kWave);
    if (lane >= off) inc += y;
  }
  if (lane == kWave - 1) s_wave[wv] = inc;
  __syncthreads();
  int32_t base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < kWavesPerBlock; ++w) {
    const int32_t t = s_wave[w];
    base += (w < wv) ? t : 0;
    tot += t;
  }
  *total = tot;
  return base + inc - x;
}

// use(k, words) for the frontier words of the far end of each edge e[k], zero
// for a far end without its activity bit (whose words are not read: those of
// node 0 are, one line for all such lanes); not called if no lane has any.  No
// other branches: the loads of a group go out together, where each waited for
// the one before when they were skipped one by one.
template <int W, int N, typename Use>
__device__ __forceinline__ void gather_words(const int32_t* __restrict__ col, const int32_t (&e)[N],
                                             const SpState& st, Use use) {
  int32_t u[N];
  uint32_t mask[N], f[N][W], any = 0u;
#pragma unroll
  for (int k = 0; k < N; ++k) u[k] = col[e[k]];
#pragma unroll
  for (int k = 0; k < N; ++k) {
    mask[k] = 0u - ((st.bits_cur[u[k] >> 5] >> (u[k] & 31)) & 1u);
    any |= mask[k];
  }
  if (__ballot(any != 0u) == 0) return;
#pragma unroll
  for (int k = 0; k < N; ++k) load_words<W>(st.fcur + (int64_t)(u[k] & mask[k]) * W, f[k]);
#pragma unroll
  for (int k = 0; k < N; ++k) {
#pragma unroll
    for (int w = 0; w < W; ++w) f[k][w] &= mask[k];
    use(k, f[k]);
  }
}

// One chunk (node, first edge, end edge, slot or -1 if it is the node's only
// one) by a wave.  Returns whether the node has new bits, in the lane that
// settled it.
template <int W>
__device__ __forceinline__ bool take_chunk(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
                                           int32_t d, const int4 c, uint32_t* __restrict__ heavy_acc,
                                           int32_t* __restrict__ heavy_done, const SpState& st, int32_t level) {
  const int lane = threadIdx.x & (kWave - 1);
  const int32_t v = c.x;
  uint32_t seen[W], acc[W];
  load_words<W>(st.vis + (int64_t)v * W, seen);
  bool full = true;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    full &= (seen[w] == word_mask(w, d));
    acc[w] = 0u;
  }
  if (full) return false;  // at every chunk of the node alike
  constexpr int kUnroll = unroll_for<W>();
  for (int32_t base = c.y; base < c.z; base += kWave * kUnroll) {
    int32_t e[kUnroll];  // past the end: the last edge again
#pragma unroll
    for (int k = 0; k < kUnroll; ++k) e[k] = min(base + k * kWave + lane, c.z - 1);
    gather_words<W, kUnroll>(col, e, st, [&](int, const uint32_t(&f)[W]) {
#pragma unroll
      for (int w = 0; w < W; ++w) acc[w] |= f[w];
    });
  }
#pragma unroll
  for (int w = 0; w < W; ++w) {
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) acc[w] |= __shfl_xor(acc[w], off, kWave);
  }
  bool found = false;
  if (lane == 0) {
    if (c.w < 0) {
      found = settle<W>(v, acc, seen, st, level);
    } else {
      uint32_t* const hacc = heavy_acc + (int64_t)c.w * W;
#pragma unroll
      for (int w = 0; w < W; ++w)
        if (acc[w]) atomicOr(&hacc[w], acc[w]);
      // The bits are exchanged by device atomics alone, so it is enough that
      // they have been performed before the count: a fence would write back
      // the L2 as well, with every chunk.  This relies on gfx950, not on the
      // language's memory model: there vmcnt counts atomics without a result
      // until the memory that device scope names has performed them (targets
      // from gfx10 on count those apart).
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      const int32_t n_chunks = (row_ptr[v + 1] - row_ptr[v] + kChunk - 1) / kChunk;
      if (atomicAdd(&heavy_done[c.w], 1) == n_chunks - 1) {  // every other chunk has added its bits
#pragma unroll
        for (int w = 0; w < W; ++w) acc[w] = atomicExch(&hacc[w], 0u);
        atomicExch(&heavy_done[c.w], 0);
        found = settle<W>(v, acc, seen, st, level);
      }
    }
    if (found) atomicOr(&st.bits_next[v >> 5], 1u << (v & 31));
  }
  return found;
}

// One level of all searches.  The last light_blocks blocks take kBlock
// consecutive nodes each (one thread per node for the node's own words) and
// share out the edges of those of degree <= kLightMax over the block: the
// edges are numbered by a prefix sum of the degrees, each thread takes a few
// consecutive ones at a time, and the frontier words of the far ends are ORed
// into the node's word in LDS.  The waves of the blocks before them share the
// chunks of at most kChunk edges of the nodes of larger degree; the chunks of
// one node combine their ORs with device atomics, and the last chunk to finish
// settles the node.
//
// Bound by gathers: most edges have to be looked at on every level (a target
// without a path keeps every node open), and most far ends are not active.
// Their activity is a bit, so that a CU's L1 holds that of 256 K nodes: with a
// byte per node, one gather after the other, a chunk to a workgroup and a
// fence per chunk, the levels of 300,000 nodes, 2.0 M entries and 128 targets
// took 19 to 36 us each (300 in all), now 9 to 32 (217).  Copying the bits to LDS first
// was no faster (100,000 nodes and 32 targets: 213 us a call against 209,
// 300,000 and 128: 421 against 409 with workgroups of 1,024).
template <int W>
__global__ __launch_bounds__(kBlock, W <= 4 ? 8 : 4) void k_sp_level(const int32_t* __restrict__ row_ptr,
                                                    const int32_t* __restrict__ col, int32_t n, int32_t d,
                                                    int32_t light_blocks, const int4* __restrict__ chunks,
                                                    const int32_t* __restrict__ n_chunks,
                                                    uint32_t* __restrict__ heavy_acc, int32_t* __restrict__ heavy_done,
                                                    const SpState st, int32_t level, int32_t* __restrict__ flags) {
  __shared__ int32_t s_pref[kBlock + 1];
  __shared__ int32_t s_start[kBlock];
  __shared__ uint32_t s_acc[W * kBlock];
  __shared__ int32_t s_wave[kWavesPerBlock];

  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wv = tid >> 6;
  const int32_t heavy_blocks = (int32_t)gridDim.x - light_blocks;
  const bool light_block = (int32_t)blockIdx.x >= heavy_blocks;
  int32_t* const prev = flags + ((level - 1) % kRing) * kFlagInts;
  int32_t* const mine = flags + (level % kRing) * kFlagInts;
  int32_t* const next = flags + ((level + 1) % kRing) * kFlagInts;
  if (blockIdx.x == 0 && tid < kSlots) next[tid * kSlotStride] = 0;
  const int active = tid < kSlots ? prev[tid * kSlotStride] : 0;
  const int32_t v = ((int32_t)blockIdx.x - heavy_blocks) * kBlock + tid;
  int32_t a = 0, deg = 0;
  uint32_t seen[W];
#pragma unroll
  for (int w = 0; w < W; ++w) seen[w] = 0u;
  if (light_block && v < n) {
    a = row_ptr[v];
    deg = row_ptr[v + 1] - a;
    load_words<W>(st.vis + (int64_t)v * W, seen);
  }
  const int32_t total_chunks = light_block ? 0 : n_chunks[0];
  const int32_t first_chunk = ((int32_t)blockIdx.x * kWavesPerBlock) + wv;
  if (!__syncthreads_or(active)) return;

  bool found = false;
  if (light_block) {
    bool full = true;
#pragma unroll
    for (int w = 0; w < W; ++w) full &= (seen[w] == word_mask(w, d));
    // The nodes with edges to look at, packed: one pass over the edges of the
    // block then moves on by at most one of them per edge.
    const bool listed = v < n && deg <= kLightMax && !full && deg > 0;
    int32_t sums;  // edges below, nodes above kListShift
    const int32_t before = block_exclusive_scan(listed ? deg + (1 << kListShift) : 0, s_wave, &sums);
    const int32_t pos = before >> kListShift, listed_nodes = sums >> kListShift;
    const int32_t total = sums & ((1 << kListShift) - 1);
    if (listed) {
      s_pref[pos] = before & ((1 << kListShift) - 1);
      s_start[pos] = a;
    }
    if (tid == 0) s_pref[listed_nodes] = total;
#pragma unroll
    for (int w = 0; w < W; ++w) s_acc[w * kBlock + tid] = 0u;
    __syncthreads();
    // Each thread takes kUnroll consecutive edges of the numbering, so that
    // they mostly share one node: their words are ORed in registers and
    // reach LDS once per node rather than once per edge.
    constexpr int kUnroll = unroll_for<W>();
    for (int32_t base = tid * kUnroll; base < total; base += kBlock * kUnroll) {
      int lo = 0, hi = listed_nodes;  // s_pref[lo] <= base < s_pref[hi]
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (s_pref[mid] <= base) lo = mid;
        else hi = mid;
      }
      int32_t e[kUnroll], node[kUnroll];
#pragma unroll
      for (int k = 0; k < kUnroll; ++k) {
        const int32_t t = min(base + k, total - 1);  // past the end: the last edge again
        lo += s_pref[lo + 1] <= t ? 1 : 0;           // every listed node has an edge
        node[k] = lo;
        e[k] = s_start[lo] + (t - s_pref[lo]);
      }
      uint32_t run[W];
      int rn = node[0];
#pragma unroll
      for (int w = 0; w < W; ++w) run[w] = 0u;
      gather_words<W, kUnroll>(col, e, st, [&](int k, const uint32_t(&f)[W]) {
        if (node[k] != rn) {  // nodes only increase along the run
#pragma unroll
          for (int w = 0; w < W; ++w) {
            if (run[w]) atomicOr(&s_acc[w * kBlock + rn], run[w]);
            run[w] = 0u;
          }
          rn = node[k];
        }
#pragma unroll
        for (int w = 0; w < W; ++w) run[w] |= f[w];
      });
#pragma unroll
      for (int w = 0; w < W; ++w)
        if (run[w]) atomicOr(&s_acc[w * kBlock + rn], run[w]);
    }
    __syncthreads();
    if (listed) {
      uint32_t acc[W];
#pragma unroll
      for (int w = 0; w < W; ++w) acc[w] = s_acc[w * kBlock + pos];
      found = settle<W>(v, acc, seen, st, level);
    }
    const unsigned long long here = __ballot(found);
    if (lane == 0 && v < n) {  // these bits share words with heavy nodes'
      if (here) atomicOr(reinterpret_cast<unsigned long long*>(st.bits_next) + (v >> 6), here);
      reinterpret_cast<unsigned long long*>(st.bits_clear)[v >> 6] = 0;
    }
  } else {
    for (int32_t c = first_chunk; c < total_chunks; c += heavy_blocks * kWavesPerBlock)
      found |= take_chunk<W>(row_ptr, col, d, chunks[c], heavy_acc, heavy_done, st, level);
  }
  if (__ballot(found) != 0 && lane == 0)
    mine[((blockIdx.x * kWavesPerBlock + wv) % kSlots) * kSlotStride] = 1;
}

// X[v][j] from the planes, unless a search goes on after the last launched
// level (its flags; NULL if none was wanted) or the CSR check has failed.  A
// block takes kDecodeNodes rows: their words go to LDS, each read once, and X
// is written as one run of 16-byte pieces, consecutive over the lanes.  A piece
// of four targets lies in one word if d % 4 == 0 (QUAD).
//
// Bound by writing X (d = 128, 300,000 nodes: 154 MB, 22 us at a fill's rate).
// With 64 bytes a lane and all the planes that l0 could need this took 57 us,
// now 32.
constexpr int kDecodeNodes = 64;

template <int W, bool QUAD>
__global__ __launch_bounds__(kBlock) void k_sp_decode(int32_t n, int32_t d, uint32_t recip_d,
                                                      const uint32_t* __restrict__ vis,
                                                      const uint32_t* __restrict__ planes, int64_t plane_stride,
                                                      int n_planes, float beyond, const uint32_t* __restrict__ check,
                                                      const int32_t* __restrict__ last_flags, float* __restrict__ X) {
  extern __shared__ uint32_t s_word[];  // [1 + n_planes][kDecodeNodes * W]: vis, then the planes
  constexpr int kWords = kDecodeNodes * W;
  const int tid = threadIdx.x;
  const int64_t v0 = (int64_t)folded_block() * kDecodeNodes;
  if (v0 >= n) return;
  const int32_t rows = (int32_t)min<int64_t>(kDecodeNodes, n - v0);
  int stop = csr_failed(check) ? 1 : 0;
  if (last_flags && tid < kSlots) stop |= last_flags[tid * kSlotStride];
  for (int32_t q = tid; q < (1 + n_planes) * kWords; q += kBlock) {
    const int32_t k = q / kWords, o = q - k * kWords;
    if (o < rows * W)
      s_word[q] = k == 0 ? vis[v0 * W + o] : planes[(k - 1) * plane_stride + v0 * W + o];
  }
  if (__syncthreads_or(stop)) return;
  const int32_t count = rows * d;
  float* const out = X + v0 * d;
  for (int32_t f = 4 * tid; f < count; f += 4 * kBlock) {
    int32_t r = d == 1 ? f : (int32_t)__umulhi((uint32_t)f, recip_d);  // f / d
    int32_t j = f - r * d;
    float x[4];
    if constexpr (QUAD) {
      const int o = r * W + (j >> 5);
      const uint32_t seen = s_word[o] >> (j & 31);
      uint32_t dist[4] = {0u, 0u, 0u, 0u};
      for (int k = 0; k < n_planes; ++k) {
        const uint32_t p = s_word[(1 + k) * kWords + o] >> (j & 31);
#pragma unroll
        for (int c = 0; c < 4; ++c) dist[c] |= ((p >> c) & 1u) << k;
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) x[c] = ((seen >> c) & 1u) ? (float)dist[c] : beyond;
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int o = min(r, rows - 1) * W + (j >> 5);  // past the last row's end nothing is written
        uint32_t dist = 0u;
        for (int k = 0; k < n_planes; ++k) dist |= ((s_word[(1 + k) * kWords + o] >> (j & 31)) & 1u) << k;
        x[c] = ((s_word[o] >> (j & 31)) & 1u) ? (float)dist : beyond;
        if (++j == d) {
          j = 0;
          ++r;
        }
      }
    }
    if (f + 4 <= count && (reinterpret_cast<uintptr_t>(out) & 15) == 0) {
      *reinterpret_cast<float4*>(out + f) = make_float4(x[0], x[1], x[2], x[3]);
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (f + c < count) out[f + c] = x[c];
    }
  }
}

// The chunk table, in one block: heavy nodes (ascending) are cut into runs
// of kChunk edges; a node of several runs gets the next accumulator slot.
// counts[1] holds the number of heavy nodes, counts[4] receives the number
// of chunks (none when the row check has failed).
__global__ __launch_bounds__(kChunkBlock) void k_sp_chunks(const int4* __restrict__ heavy, int32_t* __restrict__ counts,
                                                           int32_t heavy_cap, int4* __restrict__ chunks,
                                                           int32_t chunk_cap, const uint32_t* __restrict__ check) {
  __shared__ int32_t s_c[kChunkBlock / kWave], s_s[kChunkBlock / kWave];
  const int t = threadIdx.x, lane = t & (kWave - 1), wv = t >> 6;
  const int32_t nh = (check[0] & kErrRowPtr) ? 0 : min(counts[1], heavy_cap);
  const int32_t per = (nh + kChunkBlock - 1) / kChunkBlock;
  const int32_t lo = min(nh, t * per), hi = min(nh, lo + per);
  int32_t nc = 0, ns = 0;
  for (int32_t h = lo; h < hi; ++h) {
    const int32_t deg = heavy[h].z - heavy[h].y;
    nc += (deg + kChunk - 1) / kChunk;
    ns += deg > kChunk ? 1 : 0;
  }
  int32_t ic = nc, is = ns;
  for (int off = 1; off < kWave; off <<= 1) {
    const int32_t yc = __shfl_up(ic, off, kWave), ys = __shfl_up(is, off, kWave);
    if (lane >= off) {
      ic += yc;
      is += ys;
    }
  }
  if (lane == kWave - 1) {
    s_c[wv] = ic;
    s_s[wv] = is;
  }
  __syncthreads();
  int32_t bc = 0, bs = 0, total = 0;
  for (int w = 0; w < kChunkBlock / kWave; ++w) {
    bc += (w < wv) ? s_c[w] : 0;
    bs += (w < wv) ? s_s[w] : 0;
    total += s_c[w];
  }
  int32_t c = bc + ic - nc, slot = bs + is - ns;
  for (int32_t h = lo; h < hi; ++h) {
    const int4 r = heavy[h];
    const bool split = r.z - r.y > kChunk;
    for (int32_t e = r.y; e < r.z; e += kChunk, ++c)
      if (c < chunk_cap) chunks[c] = make_int4(r.x, e, min(r.z, e + kChunk), split ? slot : -1);
    slot += split ? 1 : 0;
  }
  if (t == 0) counts[4] = min(total, chunk_cap);
}

template <int W>
hipError_t launch_level(const int32_t* row_ptr, const int32_t* col, int32_t n, int32_t d, const int4* chunks,
                        const int32_t* n_chunks, int64_t chunk_cap, uint32_t* heavy_acc, int32_t* heavy_done,
                        const SpState& st, int32_t level, int32_t* flags, hipStream_t s) {
  const int32_t light_blocks = (n + kBlock - 1) / kBlock;
  const int32_t heavy_blocks = (int32_t)std::min<int64_t>((chunk_cap + kWavesPerBlock - 1) / kWavesPerBlock, kHeavyBlocks);
  hipLaunchKernelGGL(k_sp_level<W>, dim3((unsigned)(light_blocks + heavy_blocks)), dim3(kBlock), 0, s, row_ptr, col, n,
                     d, light_blocks, chunks, n_chunks, heavy_acc, heavy_done, st, level, flags);
  return hipGetLastError();
}

template <int W>
hipError_t launch_decode(int32_t n, int32_t d, const uint32_t* vis, const uint32_t* planes, int64_t plane_stride,
                         int n_planes, float beyond, const uint32_t* check, const int32_t* last_flags, float* X,
                         hipStream_t s) {
  const dim3 grid = folded_grid(((int64_t)n + kDecodeNodes - 1) / kDecodeNodes, kBlock);
  const size_t lds = sizeof(uint32_t) * (1 + (size_t)n_planes) * kDecodeNodes * W;  // at most 64 KB
  // ceil(2^32 / d): the high word of its product with f is f / d for f up to kDecodeNodes * 256
  const uint32_t recip_d = d == 1 ? 0u : (uint32_t)((((uint64_t)1 << 32) + d - 1) / d);
  if (d % 4 == 0)
    hipLaunchKernelGGL((k_sp_decode<W, true>), grid, dim3(kBlock), lds, s, n, d, recip_d, vis, planes,
                       plane_stride, n_planes, beyond, check, last_flags, X);
  else
    hipLaunchKernelGGL((k_sp_decode<W, false>), grid, dim3(kBlock), lds, s, n, d, recip_d, vis, planes,
                       plane_stride, n_planes, beyond, check, last_flags, X);
  return hipGetLastError();
}

struct SpKernels {
  hipError_t (*level)(const int32_t*, const int32_t*, int32_t, int32_t, const int4*, const int32_t*, int64_t,
                      uint32_t*, int32_t*, const SpState&, int32_t, int32_t*, hipStream_t);
  hipError_t (*decode)(int32_t, int32_t, const uint32_t*, const uint32_t*, int64_t, int, float, const uint32_t*,
                       const int32_t*, float*, hipStream_t);
};

SpKernels kernels_for(int W) {
  switch (W) {
    case 1: return {launch_level<1>, launch_decode<1>};
    case 2: return {launch_level<2>, launch_decode<2>};
    case 4: return {launch_level<4>, launch_decode<4>};
    default: return {launch_level<8>, launch_decode<8>};
  }
}

// Offsets of the per-call buffers inside one device allocation.  The CSR
// check's row index lies where the search state comes to lie after it.
struct SpLayout {
  size_t counts, check, flags;        // the host reads from check to the end of a flag set
  size_t hacc, hdone, cleared;        // [counts, cleared) is cleared ahead of the check
  size_t partial, heavy, chunks;
  size_t vis, f0, bits, planes;       // [vis, planes + those of the first levels) is cleared
  size_t f1, row_of, total;
};

size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

// Activity bits of all nodes, in whole waves' words.
size_t bitmap_bytes(int32_t n) { return 8 * (((size_t)n + 63) / 64); }

SpLayout make_layout(int32_t n, int64_t nnz, int64_t words, int n_planes, int64_t blocks, int64_t heavy_cap,
                     int64_t chunk_cap, int W) {
  SpLayout L{};
  size_t o = 0;
  auto place = [&](size_t bytes) {
    const size_t at = o;
    o = align_up(o + bytes);
    return at;
  };
  L.counts = place(8 * sizeof(int32_t));
  L.check = place(sizeof(uint32_t) * kCheckWords);
  L.flags = place(sizeof(int32_t) * kRing * kFlagInts);
  L.hacc = place(4 * (size_t)heavy_cap * W);
  L.hdone = place(4 * (size_t)heavy_cap);
  L.cleared = o;
  L.partial = place(sizeof(int2) * (size_t)blocks);
  L.heavy = place(sizeof(int4) * (size_t)heavy_cap);
  L.chunks = place(sizeof(int4) * (size_t)chunk_cap);
  L.row_of = o;
  L.f1 = place(4 * (size_t)words);
  L.vis = place(4 * (size_t)words);
  L.f0 = place(4 * (size_t)words);
  L.bits = place(kRing * align_up(bitmap_bytes(n)));
  L.planes = place(4 * (size_t)words * n_planes);
  L.total = std::max(o, L.row_of + sizeof(int32_t) * (size_t)nnz);
  return L;
}

int bits_of(int32_t x) {
  int b = 0;
  while (b < 31 && (x >> b) != 0) ++b;
  return b;
}

}  // namespace
}  // namespace tsgne

using namespace tsgne;

extern "C" {

tsgne_status tsgne_shortest_path_embedding(int32_t n, int64_t nnz, const int32_t* row_ptr_d, const int32_t* col_d,
                                           int32_t d, const int32_t* targets_d, double l0, float* X_d,
                                           int32_t* levels_out, void* stream) {
  if (levels_out) *levels_out = 0;
  if (n < 1) return fail(TSGNE_E_INVAL, "n must be >= 1");
  if (nnz < 0 || nnz >= ((int64_t)1 << 31)) return fail(TSGNE_E_INVAL, "nnz must lie in [0, 2^31)");
  if (d < 1 || d > kMaxTargets) return fail(TSGNE_E_INVAL, "d must lie in [1, 256]");
  if (std::isnan(l0)) return fail(TSGNE_E_INVAL, "l0 is NaN");
  if (!row_ptr_d || (nnz > 0 && !col_d) || !targets_d || !X_d) return fail(TSGNE_E_INVAL, "null pointer");
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  if (l0 < 0) l0 = std::sqrt((double)(nnz / 2));  // the default threshold sqrt(|E|)
  const float beyond = (float)(l0 + 1.0);
  // Distances beyond n - 1 do not occur, so the searches stop there too.
  const int32_t max_level = (int32_t)std::min<double>(std::floor(l0), (double)(n - 1));
  const int n_planes = bits_of(max_level);
  const int W = d <= 32 ? 1 : d <= 64 ? 2 : d <= 128 ? 4 : 8;
  const int64_t words = (int64_t)n * W;
  // a valid CSR has at most nnz / (kLightMax + 1) nodes above kLightMax, and
  // they have at most that many plus nnz / kChunk chunks
  const int64_t heavy_cap = std::min<int64_t>(n, nnz / (kLightMax + 1) + 1);
  const int64_t chunk_cap = heavy_cap + nnz / kChunk + 1;
  const SpLayout lay = make_layout(n, nnz, words, n_planes, row_check_blocks(n), heavy_cap, chunk_cap, W);

  ScratchBlock tmp;
  tmp.s = s;
  TSGNE_HIP(scratch_alloc(&tmp.p, lay.total, s), "allocate search state");
  char* const base = static_cast<char*>(tmp.p);
  uint32_t* const check = reinterpret_cast<uint32_t*>(base + lay.check);
  // [0] rows with entries, [1] heavy nodes, [4] chunks
  int32_t* const counts = reinterpret_cast<int32_t*>(base + lay.counts);
  uint32_t* const vis = reinterpret_cast<uint32_t*>(base + lay.vis);
  uint32_t* const f[2] = {reinterpret_cast<uint32_t*>(base + lay.f0), reinterpret_cast<uint32_t*>(base + lay.f1)};
  uint32_t* bits[kRing];  // level L reads those of L - 1, sets those of L, clears those of L + 1
  for (int r = 0; r < kRing; ++r)
    bits[r] = reinterpret_cast<uint32_t*>(base + lay.bits + r * align_up(bitmap_bytes(n)));
  uint32_t* const planes = reinterpret_cast<uint32_t*>(base + lay.planes);
  int2* const partial = reinterpret_cast<int2*>(base + lay.partial);
  uint32_t* const heavy_acc = reinterpret_cast<uint32_t*>(base + lay.hacc);
  int32_t* const heavy_done = reinterpret_cast<int32_t*>(base + lay.hdone);
  int4* const heavy = reinterpret_cast<int4*>(base + lay.heavy);
  int4* const chunks = reinterpret_cast<int4*>(base + lay.chunks);
  int32_t* const flags = reinterpret_cast<int32_t*>(base + lay.flags);

  // the check, with the heavy nodes from its row pass
  TSGNE_HIP(hipMemsetAsync(base, 0, lay.cleared, s), "clear counters");
  TSGNE_HIP(launch_check_rows(row_ptr_d, n, nnz, kLightMax, check, counts, partial, nullptr, heavy,
                              (int32_t)heavy_cap, s),
            "launch row check");
  hipLaunchKernelGGL(k_sp_chunks, dim3(1), dim3(kChunkBlock), 0, s, heavy, counts, (int32_t)heavy_cap, chunks,
                     (int32_t)chunk_cap, check);
  TSGNE_HIP(hipGetLastError(), "launch chunk table");
  TSGNE_HIP(launch_mirror(row_ptr_d, col_d, n, nnz, nullptr, reinterpret_cast<int32_t*>(base + lay.row_of), check, s),
            "launch CSR check");

  // Planes are cleared as levels come to need them, and the last pass reads
  // no others.
  const int64_t plane_stride = words;
  int clear_planes = bits_of(std::min<int32_t>(max_level, kLevelsPerCheck));
  TSGNE_HIP(hipMemsetAsync(vis, 0, lay.planes - lay.vis + 4 * (size_t)words * clear_planes, s), "clear search state");
  hipLaunchKernelGGL(k_sp_init, dim3((unsigned)((std::max(d, kRing * kFlagInts) + kBlock - 1) / kBlock)),
                     dim3(kBlock), 0, s, targets_d, d, n, W, vis, f[0], bits[0], flags, check);
  TSGNE_HIP(hipGetLastError(), "launch target set-up");

  const SpKernels kern = kernels_for(W);
  const size_t flags_at = (lay.flags - lay.check) / sizeof(uint32_t);  // in what the host reads
  std::vector<uint32_t> host(flags_at + kRing * kFlagInts);
  int32_t level = 1, levels_run = 0, use = 0;
  bool active = true, first = true;
  auto decode = [&](const int32_t* last_flags) {
    return kern.decode(n, d, vis, planes, plane_stride, use, beyond, check, last_flags, X_d, s);
  };
  do {
    const int32_t last = std::min<int32_t>(max_level, level + kLevelsPerCheck - 1);
    use = bits_of(last);
    if (use > clear_planes) {
      TSGNE_HIP(hipMemsetAsync(planes + clear_planes * plane_stride, 0, 4 * (size_t)words * (use - clear_planes), s),
                "clear planes");
      clear_planes = use;
    }
    for (int32_t L = level; L <= last; ++L) {
      const SpState st{f[(L - 1) & 1], f[L & 1], bits[(L - 1) % kRing], bits[L % kRing], bits[(L + 1) % kRing],
                       vis, planes, plane_stride, use};
      TSGNE_HIP(kern.level(row_ptr_d, col_d, n, d, chunks, counts + 4, chunk_cap, heavy_acc, heavy_done, st, L, flags,
                           s),
                "launch search level");
    }
    const size_t set = (size_t)(last % kRing) * kFlagInts;  // the last level's flags
    const bool ended = last == max_level;  // no search goes on, whatever the flags say
    if (first) TSGNE_HIP(decode(ended ? nullptr : flags + set), "launch decode");
    const size_t from = first ? 0 : flags_at + set, count = flags_at + set + kFlagInts - from;
    TSGNE_HIP(hipMemcpyAsync(host.data() + from, check + from, sizeof(uint32_t) * count, hipMemcpyDeviceToHost, s),
              "read level flags");
    TSGNE_HIP(hipStreamSynchronize(s), "synchronise search levels");
    const uint32_t errors = first ? check_errors(host.data()) : 0;
    if (errors & kErrRowPtr) return fail(TSGNE_E_GRAPH, "row_ptr is not nondecreasing from 0 to nnz");
    if (errors & ~kErrTarget) return fail(TSGNE_E_GRAPH, "CSR is not canonical and symmetric");
    if (errors & kErrTarget) return fail(TSGNE_E_INVAL, "a target lies outside [0, n)");
    active = false;
    for (int i = 0; i < kSlots; ++i) active |= host[flags_at + set + (size_t)i * kSlotStride] != 0;
    active &= !ended;
    if (!active && !first) {
      TSGNE_HIP(decode(nullptr), "launch decode");
      TSGNE_HIP(hipStreamSynchronize(s), "synchronise embedding");
    }
    first = false;
    levels_run = last;
    level = last + 1;
  } while (active);
  if (levels_out) *levels_out = levels_run;
  return TSGNE_OK;
}

}  // extern "C"
