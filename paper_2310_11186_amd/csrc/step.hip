// Per-step kernels of the t-SGNE loop: all-pairs Student-t repulsion with its
// normaliser Z (eq. (4)), the sparse attraction over graph edges, the gradient
// of eq. (5) and the momentum/gains update, and KL(P || Q).
//
// Repulsion tiling.  Positions are cut into nb blocks of T = 64 * R.  A work
// item is one tile (a, b), processed by one wave (symmetric tiles of 2 and 4 rows
// by as many waves, a diagonal one by a workgroup); each lane keeps R "resident"
// rows of block a in registers.
//  - Symmetric tiles (a < b): the 64-position sub-blocks of b travel around the
//    wave (every lane reads the next column from LDS, and a column's force
//    moves one lane on per step), so every unordered pair (i, j) is met exactly
//    once; w_ij is computed once and its force is added to the resident row (+)
//    and to the travelling column (-).  After 64 steps each column's sum is
//    back in the column's own lane.
//  - Direct tiles (every tile of the direct variant): columns of b are read as
//    wave-uniform values and each ordered pair is computed by the row's lane;
//    the i == j term is masked by index.  Diagonal tiles of the symmetric
//    variant use the same scheme one resident row at a time, by a workgroup each.
// Each tile writes its row sums to part[a][b] and (symmetric) its column sums
// to part[b][a], so part[k][*] holds every contribution to block k exactly
// once and the update kernel adds them in a fixed order: results do not
// depend on scheduling.  Z partials are per tile.
#include <algorithm>
#include <cmath>

#include "internal.h"

namespace tsgne {
namespace {

constexpr int kBlock = 256;
constexpr int kWavesPerBlock = kBlock / kWave;

__device__ __forceinline__ float rotate_lanes(float v) {
  // wave_ror:1 -- every lane takes the value of its neighbour on a 64-lane
  // ring.  Every source lane exists, so the "old" operand is never used; passing
  // the value itself lets the move happen in place.
  const int b = __builtin_bit_cast(int, v);
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(b, b, 0x13C, 0xF, 0xF, false));
}

__device__ __forceinline__ double wave_sum(double v) {
  for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
  return v;
}

__device__ __forceinline__ float wave_sum(float v) {
  for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
  return v;
}

// The same rotation for a value read once, by the instruction that consumes
// it.  With a constant "old" operand (never used: every source lane exists)
// the compiler folds the move into that instruction as its DPP source, so the
// rotation costs no instruction of its own.
__device__ __forceinline__ float rotate_lanes_once(float v) {
  const int b = __builtin_bit_cast(int, v);
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, b, 0x13C, 0xF, 0xF, false));
}

// w = 1 / (1 + dx^2 + dy^2) with the hardware reciprocal (q >= 1, <= 1 ulp).
__device__ __forceinline__ float student_w(float dx, float dy) {
  return __builtin_amdgcn_rcpf(__builtin_fmaf(dx, dx, __builtin_fmaf(dy, dy, 1.0f)));
}

// Two values the compiler keeps in an aligned pair of registers, the first in
// an even one and the second in the odd one after it.  A three-operand FP32
// instruction whose operands all sit in registers of one parity takes 4.6
// cycles per wave, any other 2.4 (measured with 8 waves per SIMD), and left to
// itself the compiler lets a third of the loop's FMAs fall on one parity.
typedef float reg_pair __attribute__((ext_vector_type(2)));

__device__ __forceinline__ void keep_paired(reg_pair& v) { asm("" : "+v"(v)); }

// Rows whose reciprocals are issued back to back (see sym_step).
template <int R>
constexpr int recip_group() {
  return R == 15 ? 3 : R == 12 ? 6 : R == 14 ? 7 : R >= 8 ? 4 : R >= 2 ? 2 : 1;
}

// One step of a symmetric tile: the R resident rows of this lane against the
// column c now in it.  The step's Z terms go on the chain zs; OPENS starts
// that chain at the first weight rather than adding it to +0 (an add the
// compiler must keep, as -0 + 0 = +0; no weight is -0).  res holds the rows'
// sums and s the column's, both as (y, x).
// FORCES = false keeps only the Z terms (the same weights, added in the same
// order, so Z is bitwise the one the force pass gives).
//
// What a step costs is issue: an FP32 add, mul or FMA takes 2.4 cycles per
// wave as long as two waves' such instructions can be issued side by side, a
// reciprocal 8.3 and whatever else its place among them breaks up.  So the
// reciprocals of recip_group rows go out together, at a raised wave priority
// so that no other wave's instructions fall between them (10 FMAs and a
// reciprocal: 47 cycles alternating, 37 in groups of four, 31 with the
// priority), and the operands are kept in registers of both parities.
// Measured at 300,000 nodes, 15 rows: 11.27 -> 9.43 ms a launch, 39.4 -> 33.0
// cycles per pair of a wave, of a least 10 * 2.4 + 8.3 = 32.3.
template <int R, bool MASKED, bool OPENS, bool FORCES>
__device__ __forceinline__ void sym_step(const float2 (&y)[R], reg_pair (&res)[R], reg_pair (&tw)[recip_group<R>()],
                                         float2 c, float m, float& zs, reg_pair& s) {
  constexpr int G = recip_group<R>();
  s = reg_pair{0.f, 0.f};
#pragma unroll
  for (int r0 = 0; r0 < R; r0 += G) {
    reg_pair d[G];  // (dx, dy)
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if (r0 + g >= R) continue;
      d[g] = reg_pair{y[r0 + g].x - c.x, y[r0 + g].y - c.y};
      keep_paired(d[g]);
      tw[g].y = __builtin_fmaf(d[g].y, d[g].y, 1.0f);  // tw: (w^2, w)
      keep_paired(tw[g]);
      tw[g].y = __builtin_fmaf(d[g].x, d[g].x, tw[g].y);
    }
    // w = 1 / (1 + dx^2 + dy^2) with the hardware reciprocal (<= 1 ulp)
    if (G > 1) __builtin_amdgcn_s_setprio(3);
#pragma unroll
    for (int g = 0; g < G; ++g)
      if (r0 + g < R) tw[g].y = __builtin_amdgcn_rcpf(tw[g].y);
    if (G > 1) __builtin_amdgcn_s_setprio(0);
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int r = r0 + g;
      if (r >= R) continue;
      if (MASKED) tw[g].y *= m;
      zs = (OPENS && r == 0) ? tw[g].y : zs + tw[g].y;
      if (FORCES) {
        tw[g].x = tw[g].y * tw[g].y;
        res[r] = reg_pair{__builtin_fmaf(tw[g].x, d[g].y, res[r].x), __builtin_fmaf(tw[g].x, d[g].x, res[r].y)};
        keep_paired(res[r]);
        s = reg_pair{__builtin_fmaf(tw[g].x, d[g].y, s.x), __builtin_fmaf(tw[g].x, d[g].x, s.y)};
        keep_paired(s);
      }
    }
  }
}

// A 64-step pass of a symmetric tile (a < b; block a is always full,
// a < nb - 1): in step t lane l meets column (l - t) mod 64, read from cols,
// which holds the 64 columns twice so that a step is a fixed offset.  A
// column's force trails it by one lane: it is carried across and reduced in
// one instruction, by the DPP operand of the subtraction.  Accumulation is
// two-level to keep FP32 chains short: the travelling sum of one step (R
// terms) is formed apart and then added, the resident sums are folded into a
// second FP32 sum after every pass, and Z is summed in FP32 over two steps (2R
// terms) before its FP64 sum.  MASKED: columns from `valid` on count for nothing.
template <int R, bool SPLIT, bool MASKED, bool FORCES>
__device__ __forceinline__ void sym_pass(const float2 (&y)[R], reg_pair (&res)[R], reg_pair (&tw)[recip_group<R>()],
                                         const float2* cols, int lane, int valid, float& fx, float& fy, double& z64,
                                         float& z32) {
  // One row per lane is the tile of graphs too small to fill the chip, where a
  // wave's own latency counts: its columns rotate through the lanes instead.
  constexpr bool kRotate = R == 1;
  const float2* mine = cols + kWave + lane;
  float2 c = mine[0];
  for (int t = 0; t < kWave; t += 2) {
    float zs = 0.f;
    reg_pair s;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (!kRotate) c = mine[-(t + u)];
      const float m = !MASKED || ((lane - t - u) & (kWave - 1)) < valid ? 1.f : 0.f;
      if (u == 0) sym_step<R, MASKED, true, FORCES>(y, res, tw, c, m, zs, s);
      else sym_step<R, MASKED, false, FORCES>(y, res, tw, c, m, zs, s);
      if (FORCES) {
        fx = rotate_lanes_once(fx) - s.y;
        fy = rotate_lanes_once(fy) - s.x;
      }
      if (kRotate) c = make_float2(rotate_lanes(c.x), rotate_lanes(c.y));
    }
    if (SPLIT) z64 += (double)zs; else z32 += zs;
  }
  // after the last step the forces are one lane short of their columns
  if (FORCES) {
    fx = rotate_lanes(fx);
    fy = rotate_lanes(fy);
  }
}

// Orders a wave's own accesses to LDS by other lanes (the hardware keeps them
// in order; this keeps the compiler from moving them).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// cols: this wave's 2 * kWave columns of LDS.  Reading the travelling
// positions from LDS takes two DPP moves per step (4.3 cycles each, and
// nothing else is issued beside them) off the vector pipe.
template <int R, bool SPLIT, bool FORCES = true>
__device__ __forceinline__ void tile_symmetric(const float2* __restrict__ Y, int32_t n, int32_t nb, int32_t a, int32_t b,
                               float2* __restrict__ part, double* __restrict__ zpart, float* __restrict__ zpart32,
                               int64_t item, int lane, float2* cols) {
  constexpr int T = kWave * R;
  constexpr int G = recip_group<R>();
  const int32_t valid_b = min(T, n - b * T);
  float2 y[R];
  reg_pair res[R], sum[R], tw[G];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    y[r] = Y[(int64_t)a * T + r * kWave + lane];
    res[r] = sum[r] = reg_pair{0.f, 0.f};
  }
#pragma unroll
  for (int g = 0; g < G; ++g) tw[g] = reg_pair{0.f, 0.f};
  double z64 = 0.0;
  float z32 = 0.f;
#pragma unroll 1
  for (int q = 0; q < R; ++q) {
    if (q * kWave >= valid_b) break;  // wave-uniform
    const int jl = q * kWave + lane;
    const bool vj = jl < valid_b;
    const float2 v = vj ? Y[(int64_t)b * T + jl] : make_float2(0.f, 0.f);
    wave_lds_fence();
    cols[lane] = v;
    cols[lane + kWave] = v;
    wave_lds_fence();
    float fx = 0.f, fy = 0.f;
    // a partially valid sub-block (last block only) is masked
    const int valid = valid_b - q * kWave;
    if (valid >= kWave) sym_pass<R, SPLIT, false, FORCES>(y, res, tw, cols, lane, valid, fx, fy, z64, z32);
    else sym_pass<R, SPLIT, true, FORCES>(y, res, tw, cols, lane, valid, fx, fy, z64, z32);
    if (FORCES) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        sum[r] = reg_pair{sum[r].x + res[r].x, sum[r].y + res[r].y};
        res[r] = reg_pair{0.f, 0.f};
      }
      if (vj) part[((int64_t)b * nb + a) * T + jl] = make_float2(fx, fy);
    }
  }
  if (FORCES) {
#pragma unroll
    for (int r = 0; r < R; ++r)
      part[((int64_t)a * nb + b) * T + r * kWave + lane] = make_float2(sum[r].y, sum[r].x);
  }
  // every unordered pair stands for the two ordered pairs of Z
  if (SPLIT) {
    const double z = wave_sum(z64);
    if (lane == 0) zpart[item] = 2.0 * z;
  } else {
    const float z = wave_sum(z32);
    if (lane == 0) zpart32[item] = 2.0f * z;
  }
}

// Waves that share a symmetric tile, each with one of its R passes: tiles of 2
// and 4 rows are those of graphs that leave the chip short of waves, where a
// step waits for one wave's tile (9,001 nodes, 2 rows: 2.4 tiles per SIMD).
template <int R>
constexpr int tile_waves() {
  return R == 2 || R == 4 ? R : 1;
}
// The same for the host, and tiles per workgroup.
__host__ __device__ __forceinline__ int tiles_per_block(int R) {
  return kWavesPerBlock / (R == 2 || R == 4 ? R : 1);
}

// LDS of the waves that share a tile.
template <int R>
struct SharedTile {
  reg_pair rows[R][R][kWave];  // [pass][row] sums of the resident rows
  double z[R][kWave];          // [pass] Z terms
};

// A symmetric tile by R waves: wave q of them takes pass q, and the sums of
// the resident rows and of Z are added in pass order through LDS, so the
// forces are bitwise those of the passes one after the other.  Every wave of
// the workgroup calls this (live = false without a tile).
template <int R, bool SPLIT, bool FORCES = true>
__device__ __forceinline__ void tile_symmetric_shared(const float2* __restrict__ Y, int32_t n, int32_t nb, int32_t a,
                                                      int32_t b, float2* __restrict__ part,
                                                      double* __restrict__ zpart, float* __restrict__ zpart32,
                                                      int64_t item, bool live, int q, int lane, float2* cols,
                                                      SharedTile<R>& sh) {
  constexpr int T = kWave * R;
  constexpr int G = recip_group<R>();
  if (live) {
    const int32_t valid_b = min(T, n - b * T);
    const int jl = q * kWave + lane;
    const bool vj = jl < valid_b;
    const float2 v = vj ? Y[(int64_t)b * T + jl] : make_float2(0.f, 0.f);
    float2 y[R];
    reg_pair res[R], tw[G];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      y[r] = Y[(int64_t)a * T + r * kWave + lane];
      res[r] = reg_pair{0.f, 0.f};
    }
#pragma unroll
    for (int g = 0; g < G; ++g) tw[g] = reg_pair{0.f, 0.f};
    double z64 = 0.0;
    float z32 = 0.f;
    float fx = 0.f, fy = 0.f;
    cols[lane] = v;
    cols[lane + kWave] = v;
    wave_lds_fence();
    const int valid = valid_b - q * kWave;
    if (valid >= kWave) sym_pass<R, SPLIT, false, FORCES>(y, res, tw, cols, lane, valid, fx, fy, z64, z32);
    else if (valid > 0) sym_pass<R, SPLIT, true, FORCES>(y, res, tw, cols, lane, valid, fx, fy, z64, z32);
    if (FORCES) {
#pragma unroll
      for (int r = 0; r < R; ++r) sh.rows[q][r][lane] = res[r];
      if (vj) part[((int64_t)b * nb + a) * T + jl] = make_float2(fx, fy);
    }
    sh.z[q][lane] = SPLIT ? z64 : (double)z32;
  }
  __syncthreads();
  if (!live) return;
  if (FORCES) {
    reg_pair sum = reg_pair{0.f, 0.f};
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const reg_pair r = sh.rows[k][q][lane];
      sum = reg_pair{sum.x + r.x, sum.y + r.y};
    }
    part[((int64_t)a * nb + b) * T + q * kWave + lane] = make_float2(sum.y, sum.x);
  }
  if (q != 0) return;
  // every unordered pair stands for the two ordered pairs of Z
  if (SPLIT) {
    double z = sh.z[0][lane];
#pragma unroll
    for (int k = 1; k < R; ++k) z += sh.z[k][lane];
    z = wave_sum(z);
    if (lane == 0) zpart[item] = 2.0 * z;
  } else {
    float z = (float)sh.z[0][lane];
#pragma unroll
    for (int k = 1; k < R; ++k) z += (float)sh.z[k][lane];
    z = wave_sum(z);
    if (lane == 0) zpart32[item] = 2.0f * z;
  }
}

// Direct tile: rows of block a against every valid column of block b.
// SELF (a == b) masks the i == j term by index; MASK_I masks rows past n
// (only the last block is partial).  Full off-diagonal tiles run unmasked.
template <int R, bool SPLIT, bool SELF, bool MASK_I, bool FORCES>
__device__ __forceinline__ void tile_direct_body(const float2* __restrict__ Y, int32_t n, int32_t nb, int32_t a, int32_t b,
                                 float2* __restrict__ part, double* __restrict__ zpart, float* __restrict__ zpart32,
                                 int64_t item, int lane) {
  constexpr int T = kWave * R;
  const int32_t valid_a = min(T, n - a * T);
  const int32_t valid_b = min(T, n - b * T);
  float yix[R], yiy[R], rix[R], riy[R], hix[R], hiy[R];
  bool vi[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int il = r * kWave + lane;
    vi[r] = !MASK_I || il < valid_a;
    const float2 v = vi[r] ? Y[(int64_t)a * T + il] : make_float2(0.f, 0.f);
    yix[r] = v.x;
    yiy[r] = v.y;
    rix[r] = riy[r] = hix[r] = hiy[r] = 0.f;
  }
  const float2* __restrict__ Yb = Y + (int64_t)b * T;
  double z64 = 0.0;
  float z32 = 0.f;
  // columns in chunks of 64, each chunk's row sums folded into a second sum
  for (int j0 = 0; j0 < valid_b; j0 += kWave) {
    const int j1 = min(j0 + kWave, valid_b);
    for (int jl = j0; jl < j1; ++jl) {
      const float2 v = Yb[jl];
      float zs = 0.f;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const float dx = yix[r] - v.x, dy = yiy[r] - v.y;
        float w = student_w(dx, dy);
        if (SELF || MASK_I) {
          const bool keep = vi[r] && !(SELF && jl == r * kWave + lane);
          w = keep ? w : 0.f;
        }
        zs += w;
        if (FORCES) {
          const float w2 = w * w;
          rix[r] = __builtin_fmaf(w2, dx, rix[r]);
          riy[r] = __builtin_fmaf(w2, dy, riy[r]);
        }
      }
      if (SPLIT) z64 += (double)zs; else z32 += zs;
    }
    if (FORCES) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        hix[r] += rix[r];
        hiy[r] += riy[r];
        rix[r] = riy[r] = 0.f;
      }
    }
  }
  if (FORCES) {
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (vi[r]) part[((int64_t)a * nb + b) * T + r * kWave + lane] = make_float2(hix[r], hiy[r]);
  }
  if (SPLIT) {
    const double z = wave_sum(z64);
    if (lane == 0) zpart[item] = z;
  } else {
    const float z = wave_sum(z32);
    if (lane == 0) zpart32[item] = z;
  }
}

template <int R, bool SPLIT, bool FORCES = true>
__device__ __forceinline__ void tile_direct(const float2* __restrict__ Y, int32_t n, int32_t nb, int32_t a, int32_t b,
                            float2* __restrict__ part, double* __restrict__ zpart, float* __restrict__ zpart32,
                            int64_t item, int lane) {
  const bool partial_a = (int64_t)(a + 1) * (kWave * R) > n;
  if (a == b) {
    if (partial_a) tile_direct_body<R, SPLIT, true, true, FORCES>(Y, n, nb, a, b, part, zpart, zpart32, item, lane);
    else tile_direct_body<R, SPLIT, true, false, FORCES>(Y, n, nb, a, b, part, zpart, zpart32, item, lane);
  } else {
    if (partial_a) tile_direct_body<R, SPLIT, false, true, FORCES>(Y, n, nb, a, b, part, zpart, zpart32, item, lane);
    else tile_direct_body<R, SPLIT, false, false, FORCES>(Y, n, nb, a, b, part, zpart, zpart32, item, lane);
  }
}

// The columns cols[0 .. count) against this lane's row, every ordered pair, in
// four interleaved partial sums per coordinate; SELF leaves out column `lane`.
// Adds the row's force to h (y, x) and returns the sum of the weights.
template <bool SELF, bool FORCES>
__device__ __forceinline__ float diag_chunk(float2 yi, const float2* cols, int count, int lane, reg_pair& h) {
  reg_pair acc[4], tw[4];
  float az[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < 4; ++k) acc[k] = tw[k] = reg_pair{0.f, 0.f};
  int j = 0;
#pragma unroll 2
  for (; j + 4 <= count; j += 4) {
    reg_pair d[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float2 c = cols[j + k];
      d[k] = reg_pair{yi.x - c.x, yi.y - c.y};
      keep_paired(d[k]);
      tw[k].y = __builtin_fmaf(d[k].y, d[k].y, 1.0f);
      keep_paired(tw[k]);
      tw[k].y = __builtin_fmaf(d[k].x, d[k].x, tw[k].y);
    }
    __builtin_amdgcn_s_setprio(3);
#pragma unroll
    for (int k = 0; k < 4; ++k) tw[k].y = __builtin_amdgcn_rcpf(tw[k].y);
    __builtin_amdgcn_s_setprio(0);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (SELF) tw[k].y = j + k == lane ? 0.f : tw[k].y;
      az[k] += tw[k].y;
      if (FORCES) {
        tw[k].x = tw[k].y * tw[k].y;
        acc[k] = reg_pair{__builtin_fmaf(tw[k].x, d[k].y, acc[k].x), __builtin_fmaf(tw[k].x, d[k].x, acc[k].y)};
        keep_paired(acc[k]);
      }
    }
  }
  for (; j < count; ++j) {
    const float2 c = cols[j];
    const float dx = yi.x - c.x, dy = yi.y - c.y;
    float w = student_w(dx, dy);
    if (SELF) w = j == lane ? 0.f : w;
    az[0] += w;
    if (FORCES) {
      const float w2 = w * w;
      acc[0] = reg_pair{__builtin_fmaf(w2, dy, acc[0].x), __builtin_fmaf(w2, dx, acc[0].y)};
    }
  }
  if (FORCES) {
    h.x += (acc[0].x + acc[1].x) + (acc[2].x + acc[3].x);
    h.y += (acc[0].y + acc[1].y) + (acc[2].y + acc[3].y);
  }
  return (az[0] + az[1]) + (az[2] + az[3]);
}

// Diagonal tile (a, a) inside the symmetric kernel, by a whole workgroup: each
// wave takes every kWavesPerBlock-th group of 64 rows, one row per lane,
// against all columns of the block (every ordered pair i != j), read from LDS
// as one address for all lanes.  On one wave, with the columns in scalar
// registers, such a tile took 1.5 times an off-diagonal one's time and was all
// that graphs of some ten thousand nodes waited for (8 rows per lane at 31,013
// nodes: 0.176 -> 0.146 ms a launch; 12 rows: 0.39 -> 0.23).  s_z: one double
// per wave.
template <int R, bool SPLIT, bool FORCES = true>
__device__ __forceinline__ void tile_diag(const float2* __restrict__ Y, int32_t n, int32_t nb, int32_t a,
                                          float2* __restrict__ part, double* __restrict__ zpart,
                                          float* __restrict__ zpart32, int64_t item, int wave, int lane, float2* cols,
                                          double* s_z) {
  constexpr int T = kWave * R;
  const int32_t valid = min(T, n - a * T);
  const float2* __restrict__ Ya = Y + (int64_t)a * T;
  double z64 = 0.0;
  float z32 = 0.f;
  for (int r = wave; r * kWave < valid; r += kWavesPerBlock) {
    const int il = r * kWave + lane;
    const bool vi = il < valid;
    const float2 yi = vi ? Ya[il] : make_float2(0.f, 0.f);
    reg_pair h = reg_pair{0.f, 0.f};
    for (int q = 0; q * kWave < valid; ++q) {
      const int jl = q * kWave + lane;
      const float2 v = jl < valid ? Ya[jl] : make_float2(0.f, 0.f);
      wave_lds_fence();
      cols[lane] = v;
      wave_lds_fence();
      const int count = min(kWave, valid - q * kWave);
      const float zc = q == r ? diag_chunk<true, FORCES>(yi, cols, count, lane, h)
                              : diag_chunk<false, FORCES>(yi, cols, count, lane, h);
      if (SPLIT) z64 += vi ? (double)zc : 0.0; else z32 += vi ? zc : 0.f;
    }
    if (FORCES && vi) part[((int64_t)a * nb + a) * T + il] = make_float2(h.y, h.x);
  }
  const double z = SPLIT ? wave_sum(z64) : (double)wave_sum(z32);
  if (lane == 0) s_z[wave] = z;
  __syncthreads();
  if (threadIdx.x == 0) {
    if (SPLIT) zpart[item] = (s_z[0] + s_z[1]) + (s_z[2] + s_z[3]);
    else zpart32[item] = ((float)s_z[0] + (float)s_z[1]) + ((float)s_z[2] + (float)s_z[3]);
  }
  static_assert(kWavesPerBlock == 4, "the fixed-order combination above adds four sums");
}

// Waves per SIMD the repulsion kernels must allow: with fewer, two waves'
// FP32 instructions are side by side less often (an FMA issues every 3.1
// cycles with 4 waves per SIMD, every 2.4 with 8).  R <= 4 fits 8 waves
// without spills; at R = 8 and from R = 14 on a few of the sums that the inner
// loop does not touch are spilled.
template <int R>
constexpr int repulse_min_waves() {
  return R <= 4 ? 8 : R <= 8 ? 6 : R <= 16 ? 4 : 1;
}

// Workgroups of the off-diagonal tiles; those after them take one of the
// n_diag diagonal tiles (the first of the list) each.
__host__ __device__ __forceinline__ int64_t wave_tile_blocks(int64_t n_items, int64_t n_diag, int R) {
  const int per = tiles_per_block(R);
  return (n_items - n_diag + per - 1) / per;
}

// LDS of a workgroup of off-diagonal tiles (or of a diagonal one, which uses
// the columns only).
template <int R>
struct TileLds {
  float2 cols[kWavesPerBlock][2 * kWave];
  SharedTile<tile_waves<R>() == 1 ? 1 : R> tile[tile_waves<R>() == 1 ? 1 : kWavesPerBlock / tile_waves<R>()];
};

// The off-diagonal tiles of workgroup `block`: tile k of the list's n_off.
// find(k, &view) gives a tile's graph and blocks, false if it is not to run.
struct TileView {
  const float2* Y;
  float2* part;
  double* zpart;
  float* zpart32;
  int64_t slot;  // of the Z partial
  int32_t n, nb, a, b;
};

template <int R, bool SPLIT, bool FORCES, typename Find>
__device__ __forceinline__ void off_diagonal_tiles(int64_t block, int64_t n_off, int wave, int lane, TileLds<R>& lds,
                                                   Find find) {
  constexpr int W = tile_waves<R>();
  const int64_t k = block * tiles_per_block(R) + wave / W;
  TileView v;
  const bool live = k < n_off && find(k, &v);
  if (W == 1) {
    if (live)
      tile_symmetric<R, SPLIT, FORCES>(v.Y, v.n, v.nb, v.a, v.b, v.part, v.zpart, v.zpart32, v.slot, lane,
                                       lds.cols[wave]);
  } else {
    tile_symmetric_shared<W == 1 ? 1 : R, SPLIT, FORCES>(v.Y, v.n, v.nb, v.a, v.b, v.part, v.zpart, v.zpart32, v.slot,
                                                         live, wave % W, lane, lds.cols[wave],
                                                         lds.tile[W == 1 ? 0 : wave / W]);
  }
}

template <int R, bool SPLIT, bool SYM>
__global__ __launch_bounds__(kBlock, repulse_min_waves<R>()) void k_repulse(const float2* __restrict__ Y, int32_t n, int32_t nb,
                                                    const int2* __restrict__ items, int64_t n_items, int64_t n_diag,
                                                    float2* __restrict__ part, double* __restrict__ zpart,
                                                    float* __restrict__ zpart32) {
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t block = folded_block();
  if (SYM) {
    __shared__ TileLds<R> lds;
    __shared__ double s_z[kWavesPerBlock];
    const int64_t wave_blocks = wave_tile_blocks(n_items, n_diag, R);
    if (block >= wave_blocks) {
      const int64_t item = block - wave_blocks;
      if (item >= n_diag) return;
      const int32_t a = __builtin_amdgcn_readfirstlane(items[item].x);
      tile_diag<R, SPLIT>(Y, n, nb, a, part, zpart, zpart32, item, wave, lane, lds.cols[wave], s_z);
      return;
    }
    off_diagonal_tiles<R, SPLIT, true>(
        block, n_items - n_diag, wave, lane, lds, [&](int64_t k, TileView* v) {
          const int2 ab = items[n_diag + k];
          *v = TileView{Y, part, zpart, zpart32, n_diag + k, n, nb, __builtin_amdgcn_readfirstlane(ab.x),
                        __builtin_amdgcn_readfirstlane(ab.y)};
          return true;
        });
  } else {
    const int64_t item = block * kWavesPerBlock + wave;
    if (item >= n_items) return;
    const int2 ab = items[item];
    const int32_t a = __builtin_amdgcn_readfirstlane(ab.x), b = __builtin_amdgcn_readfirstlane(ab.y);
    tile_direct<R, SPLIT>(Y, n, nb, a, b, part, zpart, zpart32, item, lane);
  }
}

// Z alone (no forces, no partials written): the weights and their sums in the
// order k_repulse uses, so the Z partials are bitwise those of the force pass.
template <int R, bool SPLIT, bool SYM>
__global__ __launch_bounds__(kBlock, repulse_min_waves<R>()) void k_zonly(const float2* __restrict__ Y, int32_t n, int32_t nb,
                                                    const int2* __restrict__ items, int64_t n_items, int64_t n_diag,
                                                    double* __restrict__ zpart,
                                                    float* __restrict__ zpart32) {
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t block = folded_block();
  if (SYM) {
    __shared__ TileLds<R> lds;
    __shared__ double s_z[kWavesPerBlock];
    const int64_t wave_blocks = wave_tile_blocks(n_items, n_diag, R);
    if (block >= wave_blocks) {
      const int64_t item = block - wave_blocks;
      if (item >= n_diag) return;
      const int32_t a = __builtin_amdgcn_readfirstlane(items[item].x);
      tile_diag<R, SPLIT, false>(Y, n, nb, a, nullptr, zpart, zpart32, item, wave, lane, lds.cols[wave], s_z);
      return;
    }
    off_diagonal_tiles<R, SPLIT, false>(
        block, n_items - n_diag, wave, lane, lds, [&](int64_t k, TileView* v) {
          const int2 ab = items[n_diag + k];
          *v = TileView{Y, nullptr, zpart, zpart32, n_diag + k, n, nb, __builtin_amdgcn_readfirstlane(ab.x),
                        __builtin_amdgcn_readfirstlane(ab.y)};
          return true;
        });
  } else {
    const int64_t item = block * kWavesPerBlock + wave;
    if (item >= n_items) return;
    const int2 ab = items[item];
    const int32_t a = __builtin_amdgcn_readfirstlane(ab.x), b = __builtin_amdgcn_readfirstlane(ab.y);
    tile_direct<R, SPLIT, false>(Y, n, nb, a, b, nullptr, zpart, zpart32, item, lane);
  }
}

// Workgroups of a plan's tiles: symmetric ones as in wave_tile_blocks, direct
// ones a wave each whatever their rows.
int64_t plan_blocks(const RepulsionPlan& p) {
  if (p.variant != TSGNE_REPULSION_SYMMETRIC) return (p.items + kWavesPerBlock - 1) / kWavesPerBlock;
  return wave_tile_blocks(p.items, p.diag, p.R) + p.diag;
}

template <int R>
hipError_t launch_zonly_r(const Workspace& ws, int32_t n, const float2* Y, int precision, hipStream_t s) {
  const RepulsionPlan& p = ws.plan;
  const dim3 grid = folded_grid(plan_blocks(p), kBlock);
  const bool split = precision != TSGNE_PREC_FP32;
  const bool sym = p.variant == TSGNE_REPULSION_SYMMETRIC;
  if (split && sym)
    hipLaunchKernelGGL((k_zonly<R, true, true>), grid, dim3(kBlock), 0, s, Y, n, p.nb, ws.items, p.items, p.diag, ws.zpart,
                       ws.zpart32);
  else if (split)
    hipLaunchKernelGGL((k_zonly<R, true, false>), grid, dim3(kBlock), 0, s, Y, n, p.nb, ws.items, p.items, p.diag, ws.zpart,
                       ws.zpart32);
  else if (sym)
    hipLaunchKernelGGL((k_zonly<R, false, true>), grid, dim3(kBlock), 0, s, Y, n, p.nb, ws.items, p.items, p.diag, ws.zpart,
                       ws.zpart32);
  else
    hipLaunchKernelGGL((k_zonly<R, false, false>), grid, dim3(kBlock), 0, s, Y, n, p.nb, ws.items, p.items, p.diag,
                       ws.zpart, ws.zpart32);
  return hipGetLastError();
}

template <int R>
hipError_t launch_repulsion_r(const Workspace& ws, int32_t n, const float2* Y, int precision, hipStream_t s) {
  const RepulsionPlan& p = ws.plan;
  const dim3 grid = folded_grid(plan_blocks(p), kBlock);
  const bool split = precision != TSGNE_PREC_FP32;
  const bool sym = p.variant == TSGNE_REPULSION_SYMMETRIC;
  if (split && sym)
    hipLaunchKernelGGL((k_repulse<R, true, true>), grid, dim3(kBlock), 0, s, Y, n, p.nb, ws.items, p.items, p.diag, ws.part,
                       ws.zpart, ws.zpart32);
  else if (split)
    hipLaunchKernelGGL((k_repulse<R, true, false>), grid, dim3(kBlock), 0, s, Y, n, p.nb, ws.items, p.items, p.diag, ws.part,
                       ws.zpart, ws.zpart32);
  else if (sym)
    hipLaunchKernelGGL((k_repulse<R, false, true>), grid, dim3(kBlock), 0, s, Y, n, p.nb, ws.items, p.items, p.diag, ws.part,
                       ws.zpart, ws.zpart32);
  else
    hipLaunchKernelGGL((k_repulse<R, false, false>), grid, dim3(kBlock), 0, s, Y, n, p.nb, ws.items, p.items, p.diag,
                       ws.part, ws.zpart, ws.zpart32);
  return hipGetLastError();
}

// Z = sum of the tile partials, one workgroup, fixed order (strided partial
// sums then a tree in LDS).
constexpr int kZThreads = 1024;

template <bool SPLIT>
__device__ __forceinline__ void zsum_block(const double* __restrict__ zpart, const float* __restrict__ zpart32, int64_t n_items,
                           double* __restrict__ Z) {
  __shared__ double sh64[kZThreads];
  __shared__ float sh32[kZThreads];
  const int t = threadIdx.x;
  // Each thread keeps kZLoads independent sums, so that kZLoads loads are in
  // flight at once (a single running sum waits for every load in turn: 25 µs
  // for the 25K tiles of a 200K-node graph), then adds them in a fixed order.
  constexpr int kZLoads = 8;
  const int64_t stride = (int64_t)kZThreads * kZLoads;
  if (SPLIT) {
    double acc[kZLoads] = {};
    int64_t k = t;
    for (; k + (kZLoads - 1) * (int64_t)kZThreads < n_items; k += stride) {
      double v[kZLoads];
#pragma unroll
      for (int u = 0; u < kZLoads; ++u) v[u] = zpart[k + u * kZThreads];
#pragma unroll
      for (int u = 0; u < kZLoads; ++u) acc[u] += v[u];
    }
    for (int u = 0; k < n_items; k += kZThreads, ++u) acc[u] += zpart[k];   // fewer than kZLoads left
    sh64[t] = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
  } else {
    float acc[kZLoads] = {};
    int64_t k = t;
    for (; k + (kZLoads - 1) * (int64_t)kZThreads < n_items; k += stride) {
      float v[kZLoads];
#pragma unroll
      for (int u = 0; u < kZLoads; ++u) v[u] = zpart32[k + u * kZThreads];
#pragma unroll
      for (int u = 0; u < kZLoads; ++u) acc[u] += v[u];
    }
    for (int u = 0; k < n_items; k += kZThreads, ++u) acc[u] += zpart32[k];
    sh32[t] = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
  }
  static_assert(kZLoads == 8, "the fixed-order combination above adds eight sums");
  __syncthreads();
  for (int w = kZThreads / 2; w > 0; w >>= 1) {
    if (t < w) {
      if (SPLIT) sh64[t] += sh64[t + w]; else sh32[t] += sh32[t + w];
    }
    __syncthreads();
  }
  if (t == 0) *Z = SPLIT ? sh64[0] : (double)sh32[0];
}

// tstep (nullable) is the device step counter of a run: {next step, step being
// run}.  The Z sum, the one single-workgroup kernel of a step and the first
// after the repulsion, takes the step's index from it for the kernels after it.
template <bool SPLIT>
__global__ __launch_bounds__(kZThreads) void k_zsum(const double* __restrict__ zpart, const float* __restrict__ zpart32,
                                                    int64_t n_items, double* __restrict__ Z,
                                                    int32_t* __restrict__ tstep) {
  zsum_block<SPLIT>(zpart, zpart32, n_items, Z);
  if (tstep && threadIdx.x == 0) {
    const int32_t t = tstep[0];
    tstep[1] = t;
    tstep[0] = t + 1;
  }
}

// Attraction sum_j p_ij w_ij (y_i - y_j) over the stored entries of row i
// (the p-part of the gradient of eq. (5); alpha is applied in the update).
// Light rows: eight lanes per row.  Heavy rows: one wave per row.
constexpr int kRowLanes = kAttractRowLanes;
constexpr uint32_t kXcds = 8;  // XCDs of an MI355X (gfx950)

template <int LANES, bool SPLIT>
__device__ __forceinline__ void attract_row(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
                                            const float* __restrict__ P, const float2* __restrict__ Y, int32_t i,
                                            int sub, double2* __restrict__ out) {
  constexpr int U = 4;  // entries per lane whose loads are issued together
  const int32_t b = row_ptr[i], e_end = row_ptr[i + 1];
  const float2 yi = Y[i];
  double ax = 0.0, ay = 0.0;
  float fx = 0.f, fy = 0.f;
  for (int32_t e0 = b + sub; e0 < e_end; e0 += U * LANES) {
    int32_t j[U];
    float p[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int32_t e = e0 + u * LANES;
      j[u] = e < e_end ? col[e] : i;
      p[u] = e < e_end ? P[e] : 0.f;
    }
    float2 yj[U];
#pragma unroll
    for (int u = 0; u < U; ++u) yj[u] = Y[j[u]];
    // entries in increasing order per lane, exactly as a one-at-a-time loop.
    // An entry past the row's end (j = i, p = 0) adds exactly +0, which leaves
    // a sum started at +0 unchanged; with no branch here the gathers of Y are
    // all issued before the first is used (a branch would put each behind its
    // own check and wait).
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float dx = yi.x - yj[u].x, dy = yi.y - yj[u].y;
      const float pw = p[u] * student_w(dx, dy);
      if (SPLIT) {
        ax += (double)(pw * dx);
        ay += (double)(pw * dy);
      } else {
        fx = __builtin_fmaf(pw, dx, fx);
        fy = __builtin_fmaf(pw, dy, fy);
      }
    }
  }
  if (!SPLIT) {
    ax = fx;
    ay = fy;
  }
  for (int off = LANES / 2; off > 0; off >>= 1) {
    if (SPLIT) {
      ax += __shfl_xor(ax, off, LANES);
      ay += __shfl_xor(ay, off, LANES);
    } else {
      fx += __shfl_xor(fx, off, LANES);
      fy += __shfl_xor(fy, off, LANES);
    }
  }
  if (!SPLIT) {
    ax = fx;
    ay = fy;
  }
  if (sub == 0) out[i] = make_double2(ax, ay);
}

template <bool SPLIT>
__global__ __launch_bounds__(kBlock) void k_attract_light(const int32_t* __restrict__ row_ptr,
                                                          const int32_t* __restrict__ col, const float* __restrict__ P,
                                                          const float2* __restrict__ Y, int32_t n,
                                                          double2* __restrict__ out) {
  // Blocks are dealt to the XCDs in turn; renumber them so that each XCD
  // takes one contiguous range of rows, and its L2 sees the neighbours of
  // nearby rows (the grid is a multiple of kXcds).
  const uint32_t per_xcd = gridDim.x * gridDim.y / kXcds, i0 = folded_block();
  const uint32_t block = (i0 % kXcds) * per_xcd + i0 / kXcds;
  const int64_t t = (int64_t)block * kBlock + threadIdx.x;
  const int32_t i = (int32_t)min<int64_t>(t / kRowLanes, n - 1);
  const bool live = t / kRowLanes < n && (row_ptr[i + 1] - row_ptr[i]) <= kHeavyDegree;
  // whole 8-lane groups share `live`, so the shuffles inside stay in step
  if (live) attract_row<kRowLanes, SPLIT>(row_ptr, col, P, Y, i, (int)(threadIdx.x & (kRowLanes - 1)), out);
}

template <bool SPLIT>
__global__ __launch_bounds__(kBlock) void k_attract_heavy(const int32_t* __restrict__ row_ptr,
                                                          const int32_t* __restrict__ col, const float* __restrict__ P,
                                                          const float2* __restrict__ Y,
                                                          const int32_t* __restrict__ heavy, int32_t n_heavy,
                                                          double2* __restrict__ out) {
  const int32_t w = __builtin_amdgcn_readfirstlane((int32_t)(blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6)));
  if (w >= n_heavy) return;
  attract_row<kWave, SPLIT>(row_ptr, col, P, Y, heavy[w], (int)(threadIdx.x & (kWave - 1)), out);
}

// Workgroups of the attraction inside a launch of the repulsion, so that their
// loads' latency passes while tiles are computed beside them.  Workgroups are
// dealt to the XCDs in turn and inside each to its 32 compute units in turn,
// so the unit is one per XCD, every stride-th group of kXcds workgroups is the
// attraction's, and stride is odd: with every second one its, half of the
// compute units got no tile at all (104 us a launch at 20,000 nodes, 64 us for
// the tiles alone).  With stride 1 the attraction goes first.
struct AttractBlocks {
  uint32_t light = 0, heavy = 0;  // workgroups with work
  uint32_t groups = 0;            // groups of kXcds
  uint32_t stride = 1;
};

AttractBlocks mix_attract(int64_t tile_blocks, int64_t light, int64_t heavy) {
  AttractBlocks m;
  m.light = (uint32_t)light;
  m.heavy = (uint32_t)heavy;
  m.groups = (uint32_t)((light + heavy + kXcds - 1) / kXcds);
  if (m.groups > 0) m.stride = ((uint32_t)((tile_blocks / kXcds + m.groups) / m.groups) - 1) | 1;
  return m;
}

dim3 mixed_grid(int64_t tile_blocks, const AttractBlocks& m) {
  return folded_grid(tile_blocks + (int64_t)m.groups * kXcds, kBlock);
}

// Which workgroup of the launch this is: >= 0 its index among the
// attraction's (which may lie past its last one), otherwise -1 - its index
// among the tiles'.
__device__ __forceinline__ int64_t mixed_block(const AttractBlocks& m) {
  const uint32_t i = folded_block(), group = i / kXcds, q = group / m.stride;
  if (q < m.groups && group - q * m.stride == m.stride - 1) return (int64_t)q * kXcds + i % kXcds;
  return -1 - (int64_t)(i - min(q, m.groups) * kXcds);
}

// The forces at Y in one launch: the tiles of a symmetric plan (as k_repulse)
// and the attraction (as k_attract_light and _heavy), which needs nothing of
// them.  tstep (nullable): a run's device step counter {next step, step being
// run}, advanced here for the kernels after this one.  At 2,000 nodes a step
// was four launches of 5.5, 2.7, 2.7 and 5.5 us, mostly latency.
template <int R, bool SPLIT>
__global__ __launch_bounds__(kBlock, repulse_min_waves<R>()) void k_forces(
    const float2* __restrict__ Y, int32_t n, int32_t nb, const int2* __restrict__ items, int64_t n_items,
    int64_t n_diag, float2* __restrict__ part, double* __restrict__ zpart, float* __restrict__ zpart32,
    const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col, const float* __restrict__ P,
    const int32_t* __restrict__ heavy, int32_t n_heavy, double2* __restrict__ attract, AttractBlocks mix,
    int32_t* __restrict__ tstep) {
  __shared__ TileLds<R> lds;
  __shared__ double s_z[kWavesPerBlock];
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & (kWave - 1);
  if (tstep && folded_block() == 0 && threadIdx.x == 0) {
    const int32_t t = tstep[0];
    tstep[1] = t;
    tstep[0] = t + 1;
  }
  const int64_t mixed = mixed_block(mix);
  if (mixed >= 0) {
    if (mixed < mix.light) {
      const int32_t i0 = (int32_t)(mixed * (kBlock / kRowLanes) + threadIdx.x / kRowLanes);
      const int32_t i = min(i0, n - 1);
      // whole 8-lane groups take the branch together, so the shuffles inside stay in step
      if (i0 < n && row_ptr[i + 1] - row_ptr[i] <= kHeavyDegree)
        attract_row<kRowLanes, SPLIT>(row_ptr, col, P, Y, i, (int)(threadIdx.x & (kRowLanes - 1)), attract);
    } else {
      const int32_t w = (int32_t)(mixed - mix.light) * kWavesPerBlock + wave;
      if (w < n_heavy) attract_row<kWave, SPLIT>(row_ptr, col, P, Y, heavy[w], lane, attract);
    }
    return;
  }
  const int64_t block = -1 - mixed, wave_blocks = wave_tile_blocks(n_items, n_diag, R);
  if (block >= wave_blocks) {
    const int64_t item = block - wave_blocks;
    if (item >= n_diag) return;
    const int32_t a = __builtin_amdgcn_readfirstlane(items[item].x);
    tile_diag<R, SPLIT>(Y, n, nb, a, part, zpart, zpart32, item, wave, lane, lds.cols[wave], s_z);
    return;
  }
  off_diagonal_tiles<R, SPLIT, true>(block, n_items - n_diag, wave, lane, lds, [&](int64_t k, TileView* v) {
    const int2 ab = items[n_diag + k];
    *v = TileView{Y, part, zpart, zpart32, n_diag + k, n, nb, __builtin_amdgcn_readfirstlane(ab.x),
                  __builtin_amdgcn_readfirstlane(ab.y)};
    return true;
  });
}

// Plans of at most this many tiles have their Z summed by every workgroup of
// the update for itself (see block_Z) instead of by a kernel of its own: up to
// here the 64 KB of partials are read from L2 in the shadow of the force
// partials' loads, and a launch is saved.
constexpr int64_t kOwnZItems = 8192;
constexpr int kUpdateRows = kUpdateBlockRows;  // rows per workgroup of the update
static_assert(kUpdateRows == kWave, "one row per lane");

// Z of at most kOwnZItems tile partials by a workgroup of kBlock threads: the
// additions of zsum_block in its order, each thread standing for four of its
// 1024, so bitwise the same Z.  First each thread's part, then (block_Z) the
// sum, to every thread.
template <typename V>
__device__ __forceinline__ V thread_Z(const V* __restrict__ zpart, int32_t n_items) {
  constexpr int kPer = kZThreads / kBlock, kLoads = (int)(kOwnZItems / kZThreads);
  static_assert(kPer == 4 && kLoads == 8, "the combinations below add four threads' sums of eight loads");
  const int t = threadIdx.x;
  V a[kPer];
#pragma unroll
  for (int p = 0; p < kPer; ++p) {
    V v[kLoads];
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
      const int32_t k = t + p * kBlock + u * kZThreads;
      v[u] = u * kZThreads < n_items ? zpart[min(k, n_items - 1)] : (V)0;
      v[u] = k < n_items ? v[u] : (V)0;
    }
    a[p] = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
  }
  return (a[0] + a[2]) + (a[1] + a[3]);  // the tree's levels 512 and 256
}

template <typename V>
__device__ __forceinline__ V block_Z(V z, V* s_z) {
  const int t = threadIdx.x;
  s_z[t] = z;
  __syncthreads();
  if (t < kWave) {
    z = s_z[t] + s_z[t + 2 * kWave];
    z += s_z[t + kWave] + s_z[t + 3 * kWave];
    for (int w = kWave / 2; w > 0; w >>= 1) z += __shfl_down(z, w, kWave);
    if (t == 0) s_z[0] = z;
  }
  __syncthreads();
  return s_z[0];
}

// What the update needs of one graph.
struct UpdateView {
  const float2* part;
  const double2* attract;
  const double* zpart;
  const float* zpart32;
  double* Z;  // read, or written by the first workgroup where it sums Z itself
  float2* Y;
  float2* U;
  float2* G;
  int32_t n, nb, n_items;
};

// g_i = 4 (alpha * A_i - R_i / Z) and the momentum/gains update of rows
// i0 .. i0 + 63, one row per lane.  Each wave of the workgroup sums a
// contiguous quarter of the rows' force partials in block order (FP64 in the
// split mode), the quarters are added in order, and the first wave finishes.
// Bound by latency for small graphs (a chain of loads and sums) and by the
// partials' 8 n nb bytes for large ones; four waves per 64 rows keep four
// times the loads in flight that a wave per 64 rows did.
template <bool SPLIT, bool OWN_Z>
__device__ __forceinline__ void update_rows(const UpdateView& v, int32_t T, int32_t i0, float alpha, float momentum,
                                            float eta, float min_gain, bool do_update, float2* __restrict__ grad_out,
                                            double* __restrict__ Z_out) {
  __shared__ double2 s_r[kWavesPerBlock][kWave];
  __shared__ double s_z[kBlock];
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & (kWave - 1);
  const int32_t i = i0 + lane;
  // a row block holds whole groups of 64 rows; rows past n read the partial
  // buffer inside their own row block and store nothing
  const int32_t k = i0 / T;
  const float2* __restrict__ pp = v.part + (int64_t)k * v.nb * T + (i0 - k * T) + lane;
  const int32_t quarter = (v.nb + kWavesPerBlock - 1) / kWavesPerBlock;
  const int32_t first = wave * quarter, end = min(v.nb, first + quarter);
  double rx = 0.0, ry = 0.0;
  float sx = 0.f, sy = 0.f;
  // Partials are read in batches of kBatchLoads whose loads are all issued
  // before the first is added.  The loop body has no branch (a branch around
  // a load makes the compiler wait for it before the next one is issued), so
  // past the last block an index is clamped to it: an in-bounds re-read that
  // adds +0, which leaves a sum started at +0 unchanged.
  //
  // The first batch's loads go out before anything waits, and with them those
  // of Z's partials and of the rows' own state: one after the other these were
  // three trips to memory of a 2,000-node update's 5.5 us.
  constexpr int kBatchLoads = 16;
  float2 p[kBatchLoads];
#pragma unroll
  for (int u = 0; u < kBatchLoads; ++u) p[u] = pp[(int64_t)max(min(first + u, end - 1), 0) * T];
  const int32_t own = min(i, v.n - 1);
  double2 A = make_double2(0.0, 0.0);
  float2 y = make_float2(0.f, 0.f), uu = y, gn = y;
  if (wave == 0) {
    A = v.attract[own];
    if (do_update) {
      y = v.Y[own];
      uu = v.U[own];
      gn = v.G[own];
    }
  }
  double z64 = 0.0;
  float z32 = 0.f;
  if (OWN_Z) {
    if (SPLIT) z64 = thread_Z<double>(v.zpart, v.n_items);
    else z32 = thread_Z<float>(v.zpart32, v.n_items);
  }
  for (int32_t o0 = first; o0 < end; o0 += kBatchLoads) {
    if (o0 != first) {
#pragma unroll
      for (int u = 0; u < kBatchLoads; ++u) p[u] = pp[(int64_t)min(o0 + u, end - 1) * T];
    }
    const int32_t count = end - o0;
#pragma unroll
    for (int u = 0; u < kBatchLoads; ++u) {
      const bool in = u < count;
      if (SPLIT) {
        rx += in ? (double)p[u].x : 0.0;
        ry += in ? (double)p[u].y : 0.0;
      } else {
        sx += in ? p[u].x : 0.f;
        sy += in ? p[u].y : 0.f;
      }
    }
  }
  s_r[wave][lane] = SPLIT ? make_double2(rx, ry) : make_double2(sx, sy);
  double Z;
  if (OWN_Z) {
    Z = SPLIT ? block_Z<double>(z64, s_z) : (double)block_Z<float>(z32, reinterpret_cast<float*>(s_z));
  } else {
    Z = *v.Z;
    __syncthreads();
  }
  if (i0 == 0 && threadIdx.x == 0) {
    if (OWN_Z) *v.Z = Z;
    if (Z_out) *Z_out = Z;
  }
  if (wave != 0 || i >= v.n) return;
  rx = sx = 0.f;
  ry = sy = 0.f;
#pragma unroll
  for (int w = 0; w < kWavesPerBlock; ++w) {
    const double2 r = s_r[w][lane];
    if (SPLIT) {
      rx += r.x;
      ry += r.y;
    } else {
      sx += (float)r.x;
      sy += (float)r.y;
    }
  }
  float2 g;
  if (SPLIT) {
    const double invZ = Z > 0.0 ? 1.0 / Z : 0.0;
    g.x = (float)(4.0 * ((double)alpha * A.x - rx * invZ));
    g.y = (float)(4.0 * ((double)alpha * A.y - ry * invZ));
  } else {
    const float invZ = Z > 0.0 ? (float)(1.0 / Z) : 0.f;
    g.x = 4.0f * (alpha * (float)A.x - sx * invZ);
    g.y = 4.0f * (alpha * (float)A.y - sy * invZ);
  }
  if (grad_out) grad_out[i] = g;
  if (!do_update) return;
  gn.x = (g.x * uu.x < 0.f) ? gn.x + 0.2f : gn.x * 0.8f;
  gn.y = (g.y * uu.y < 0.f) ? gn.y + 0.2f : gn.y * 0.8f;
  gn.x = fmaxf(gn.x, min_gain);
  gn.y = fmaxf(gn.y, min_gain);
  uu.x = momentum * uu.x - eta * gn.x * g.x;
  uu.y = momentum * uu.y - eta * gn.y * g.y;
  y.x += uu.x;
  y.y += uu.y;
  v.Y[i] = y;
  v.U[i] = uu;
  v.G[i] = gn;
}

// With sched.tstep set, alpha and the momentum come from the step index on the
// device (early exaggeration while t < t_ee); otherwise the host's values are
// used.
template <bool SPLIT, bool OWN_Z>
__global__ __launch_bounds__(kBlock) void k_update(UpdateView v, int32_t T, float alpha, float momentum, float eta,
                                                   float min_gain, int do_update, float2* __restrict__ grad_out,
                                                   double* __restrict__ Z_out, StepSchedule sched) {
  if (sched.tstep) {
    const bool early = sched.tstep[1] < sched.exaggeration_iters;
    alpha = early ? sched.early_exaggeration : 1.0f;
    momentum = early ? sched.momentum_early : sched.momentum_late;
  }
  update_rows<SPLIT, OWN_Z>(v, T, (int32_t)blockIdx.x * kUpdateRows, alpha, momentum, eta, min_gain, do_update != 0,
                            grad_out, Z_out);
}

// ---------------------------------------------------------------------------
// Batched step over many graphs.  Every graph keeps its own tiling, item
// order, partial buffers and reduction order, so a graph advanced inside a
// batch computes exactly what it computes alone with the same tile size.  Each
// graph's step index lives in device memory (advanced by the last kernel of a
// step), so a step's launches are the same every time and graphs at different
// progress can share one; graphs with t >= n_iter are skipped.
// ---------------------------------------------------------------------------

// A graph's step index is kept twice, so that no launch reads what it writes:
// the forces read t and leave t + 1 in t_run (-1 where the graph has no step
// to take), the update reads t_run and leaves it in t.
__device__ __forceinline__ bool batch_live(const BatchDesc& d) {
  const int32_t t = *d.t;
  return t < d.n_iter && t < *d.limit;
}

// The forces of every live graph in one launch, as k_forces.
template <int R, bool SPLIT>
__global__ __launch_bounds__(kBlock, repulse_min_waves<R>()) void k_batch_forces(
    const BatchDesc* __restrict__ descs, const int4* __restrict__ items, int64_t n_items, int64_t n_diag,
    const int2* __restrict__ chunks, const int2* __restrict__ heavy, int32_t n_heavy, AttractBlocks mix) {
  __shared__ TileLds<R> lds;
  __shared__ double s_z[kWavesPerBlock];
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t mixed = mixed_block(mix);
  if (mixed >= 0) {
    if (mixed < mix.light) {  // kBlock / kRowLanes light rows of one graph
      const int2 ch = chunks[mixed];
      const BatchDesc& d = descs[ch.x];
      if (!batch_live(d)) return;
      const int32_t i0 = ch.y + (int32_t)(threadIdx.x / kRowLanes);
      const int32_t i = min(i0, d.n - 1);
      if (i0 < d.n && d.row_ptr[i + 1] - d.row_ptr[i] <= kHeavyDegree)
        attract_row<kRowLanes, SPLIT>(d.row_ptr, d.col, d.P, d.Y, i, (int)(threadIdx.x & (kRowLanes - 1)), d.attract);
    } else {
      const int32_t w = (int32_t)(mixed - mix.light) * kWavesPerBlock + wave;
      if (w >= n_heavy) return;
      const int2 hr = heavy[w];
      const BatchDesc& d = descs[hr.x];
      if (batch_live(d)) attract_row<kWave, SPLIT>(d.row_ptr, d.col, d.P, d.Y, hr.y, lane, d.attract);
    }
    return;
  }
  const int64_t block = -1 - mixed, wave_blocks = wave_tile_blocks(n_items, n_diag, R);
  if (block >= wave_blocks) {
    if (block - wave_blocks >= n_diag) return;
    const int4 it = items[block - wave_blocks];
    const BatchDesc& d = descs[__builtin_amdgcn_readfirstlane(it.x)];
    const int32_t a = __builtin_amdgcn_readfirstlane(it.y);
    const bool live = batch_live(d);
    if (a == 0 && threadIdx.x == 0) *d.t_run = live ? *d.t + 1 : -1;
    if (live)
      tile_diag<R, SPLIT>(d.Y, d.n, d.nb, a, d.part, d.zpart, d.zpart32, __builtin_amdgcn_readfirstlane(it.w), wave,
                          lane, lds.cols[wave], s_z);
    return;
  }
  off_diagonal_tiles<R, SPLIT, true>(block, n_items - n_diag, wave, lane, lds, [&](int64_t k, TileView* v) {
    const int4 it = items[n_diag + k];
    const BatchDesc& d = descs[__builtin_amdgcn_readfirstlane(it.x)];
    if (!batch_live(d)) return false;
    *v = TileView{d.Y, d.part, d.zpart, d.zpart32, __builtin_amdgcn_readfirstlane(it.w), d.n, d.nb,
                  __builtin_amdgcn_readfirstlane(it.y), __builtin_amdgcn_readfirstlane(it.z)};
    return true;
  });
}

template <bool SPLIT>
__global__ __launch_bounds__(kZThreads) void k_batch_zsum(const BatchDesc* __restrict__ descs) {
  const BatchDesc& d = descs[blockIdx.x];
  if (*d.t_run < 0) return;
  zsum_block<SPLIT>(d.zpart, d.zpart32, d.n_items, d.Z);
}

// One workgroup covers kUpdateRows rows of one graph.
template <bool SPLIT, bool OWN_Z>
__global__ __launch_bounds__(kBlock) void k_batch_update(const BatchDesc* __restrict__ descs,
                                                         const int2* __restrict__ blocks, int32_t T, float ee,
                                                         int32_t t_ee, float m_early, float m_late, float min_gain) {
  const int2 bl = blocks[blockIdx.x];
  const BatchDesc& d = descs[bl.x];
  const int32_t next = *d.t_run;
  if (next < 0) return;
  if (bl.y == 0 && threadIdx.x == 0) *d.t = next;
  const bool early = next - 1 < t_ee;
  const UpdateView v{d.part, d.attract, d.zpart, d.zpart32, d.Z, d.Y, d.U, d.G, d.n, d.nb, (int32_t)d.n_items};
  update_rows<SPLIT, OWN_Z>(v, T, bl.y, early ? ee : 1.0f, early ? m_early : m_late, d.eta, min_gain, true, nullptr,
                            nullptr);
}

// KL = sum_e P_e log(P_e / q_e), q_e = w_e / Z, in FP64: fixed grid, strided
// per-thread sums, tree per block, then one block over the block sums.
constexpr int kKLThreads = 256;

// KL sampling inside a run (trace != nullptr): the step being run (tstep[1])
// holds the layout after t steps; it is sampled when t is a positive multiple
// of kl_every, into trace[t / kl_every - 1], with the Z this step has just
// summed at that layout.  Other steps return at once.
__device__ __forceinline__ bool kl_skip(const int32_t* tstep, int32_t kl_every) {
  if (!tstep) return false;
  const int32_t t = tstep[1];
  return t <= 0 || t % kl_every != 0;
}

__global__ __launch_bounds__(kKLThreads) void k_kl_edges(const int32_t* __restrict__ row_of,
                                                         const int32_t* __restrict__ col, const float* __restrict__ P,
                                                         const float2* __restrict__ Y, int64_t nnz,
                                                         const double* __restrict__ Zp, double* __restrict__ klpart,
                                                         const int32_t* __restrict__ tstep, int32_t kl_every) {
  if (kl_skip(tstep, kl_every)) return;
  __shared__ double sh[kKLThreads];
  const double logZ = *Zp > 0.0 ? log(*Zp) : 0.0;
  double acc = 0.0;
  const int64_t stride = (int64_t)gridDim.x * kKLThreads;
  for (int64_t e = (int64_t)blockIdx.x * kKLThreads + threadIdx.x; e < nnz; e += stride) {
    const double p = P[e];
    if (p <= 0.0) continue;
    const float2 yi = Y[row_of[e]], yj = Y[col[e]];
    const double dx = (double)yi.x - (double)yj.x, dy = (double)yi.y - (double)yj.y;
    acc += p * (log(p) + logZ + log1p(dx * dx + dy * dy));
  }
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int w = kKLThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) klpart[blockIdx.x] = sh[0];
}

__global__ __launch_bounds__(kKLThreads) void k_kl_final(const double* __restrict__ klpart, int32_t nparts,
                                                         double* __restrict__ out, const int32_t* __restrict__ tstep,
                                                         int32_t kl_every, double* __restrict__ trace) {
  if (kl_skip(tstep, kl_every)) return;
  __shared__ double sh[kKLThreads];
  double acc = 0.0;
  for (int32_t k = threadIdx.x; k < nparts; k += kKLThreads) acc += klpart[k];
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int w = kKLThreads / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    *out = sh[0];
    if (trace) trace[tstep ? tstep[1] / kl_every - 1 : 0] = sh[0];
  }
}

__global__ __launch_bounds__(kBlock) void k_nonfinite(const float2* __restrict__ Y, int32_t n,
                                                      uint32_t* __restrict__ flag) {
  const int32_t i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  const float2 y = Y[i];
  if (!isfinite(y.x) || !isfinite(y.y)) atomicOr(flag, 1u);
}

__global__ __launch_bounds__(kUpdateRows) void k_batch_nonfinite(const BatchDesc* __restrict__ descs,
                                                                 const int2* __restrict__ blocks,
                                                                 uint32_t* __restrict__ flag) {
  const int2 bl = blocks[blockIdx.x];
  const int32_t i = bl.y + (int32_t)threadIdx.x;
  if (i >= descs[bl.x].n) return;
  const float2 y = descs[bl.x].Y[i];
  if (!isfinite(y.x) || !isfinite(y.y)) atomicOr(flag, 1u);
}

__global__ __launch_bounds__(kBlock) void k_run_init(float2* __restrict__ U, float2* __restrict__ gains, int32_t n,
                                                     int32_t* __restrict__ tstep, uint32_t* __restrict__ flag) {
  const int32_t i = blockIdx.x * kBlock + threadIdx.x;
  if (i == 0) {
    tstep[0] = tstep[1] = 0;
    *flag = 0;
  }
  if (i >= n) return;
  U[i] = make_float2(0.f, 0.f);
  gains[i] = make_float2(1.f, 1.f);
}

inline unsigned blocks_for(int64_t work, int per) { return (unsigned)((work + per - 1) / per); }

}  // namespace

// SIMDs of the chip (256 CUs x 4).
constexpr int64_t kSimds = 1024;
// Largest graphs that take 1 and 2 rows per lane automatically (see make_plan).
constexpr int32_t kOneRowMaxNodes = 3500;
constexpr int32_t kTwoRowMaxNodes = 11000;

RepulsionPlan make_plan(int32_t n, int32_t R, int32_t variant) {
  RepulsionPlan p;
  p.variant = (variant == TSGNE_REPULSION_DIRECT) ? TSGNE_REPULSION_DIRECT : TSGNE_REPULSION_SYMMETRIC;
  auto items_for = [&](int32_t r) {
    const int64_t nb = (n + kWave * r - 1) / (kWave * r);
    return p.variant == TSGNE_REPULSION_DIRECT ? nb * nb : nb * (nb + 1) / 2;
  };
  // Small graphs have too few tiles of 4 or more rows to fill the chip: a
  // layout step is then set by one tile's latency, and smaller tiles win in
  // spite of their lower per-pair efficiency.  Crossovers measured on MI355X
  // over whole layout steps: 1 row per lane up to about 3,500 nodes (a step of
  // 2,000 nodes takes 12.4 us with 1 row, 12.9 with 2, 16.3 with 4; of 3,500
  // 12.2, 13.1 and 16.4), 2 rows up to 11,000, and from there on the cost model
  // below.  2 rows are ahead of 4 at 5,000 nodes (15.3 us and 16.4; 1 row 16.8)
  // and no longer at 9,001 (23.6 and 22.8) and 11,500 (32.6 and 31.0): since waves
  // share their tiles the crossover lies between 5,000 and 9,001, and the bound,
  // measured before, costs the sizes between up to 5 %.
  if (!tile_rows_supported(R) && p.variant == TSGNE_REPULSION_SYMMETRIC) {
    if (n <= kOneRowMaxNodes) R = 1;
    else if (n <= kTwoRowMaxNodes) R = 2;
  }
  if (!tile_rows_supported(R)) {
    // Cost model: the tiles of the busiest SIMD (one wave each; those of 4 rows,
    // now four waves each, are counted alike), i.e. the
    // tile count over the chip's 1024 SIMDs rounded up, times the tile area,
    // divided by the per-pair efficiency of that tile relative to R = 16
    // (tile-pair slots per second of the repulsion at 200K-500K nodes, where
    // every SIMD holds 19 or more tiles, measured before the reciprocals were
    // grouped: 1.004 for R = 15, 0.996 for 14, 0.997 for 12, 0.969 for 8, 0.827
    // for 4; now 0.93 for 4, 0.99 for 8, 1.01 to 1.03 for 12 to 15, with which
    // the picks stay within 3 % of the best as they are: a step of 20,000 nodes
    // takes 67.6 us against 67.5, of 60,000 453 against 449, of 300,000 9.84 ms
    // against 9.88 with 16 rows and 9.98 with 14).  A SIMD
    // needs about 64 / R resident tiles (64 independent pairs per step over
    // its waves) to hide the dependent-issue latency, so fewer tiles than that
    // take as long as that many.  Small graphs get small tiles (every SIMD
    // busy), large graphs the tile whose count divides best over the SIMDs.
    const int32_t rs[6] = {16, 15, 14, 12, 8, 4};
    const double eff[6] = {1.0, 1.004, 0.996, 0.997, 0.969, 0.827};
    double best = 0.0;
    for (int k = 0; k < 6; ++k) {
      const double T = (double)(kWave * rs[k]);
      const int64_t per_simd = std::max<int64_t>((items_for(rs[k]) + kSimds - 1) / kSimds, kWave / rs[k]);
      const double cost = (double)per_simd * T * T / eff[k];
      if (best == 0.0 || cost < best) {
        best = cost;
        R = rs[k];
      }
    }
  }
  p.R = R;
  p.T = kWave * R;
  p.nb = (n + p.T - 1) / p.T;
  p.items = items_for(R);
  p.diag = p.variant == TSGNE_REPULSION_SYMMETRIC ? p.nb : 0;
  return p;
}

hipError_t launch_repulsion(const Workspace& ws, int32_t n, const float2* Y, int precision, hipStream_t s) {
  switch (ws.plan.R) {
    case 1: return launch_repulsion_r<1>(ws, n, Y, precision, s);
    case 2: return launch_repulsion_r<2>(ws, n, Y, precision, s);
    case 4: return launch_repulsion_r<4>(ws, n, Y, precision, s);
    case 8: return launch_repulsion_r<8>(ws, n, Y, precision, s);
    case 16: return launch_repulsion_r<16>(ws, n, Y, precision, s);
    case 12: return launch_repulsion_r<12>(ws, n, Y, precision, s);
    case 14: return launch_repulsion_r<14>(ws, n, Y, precision, s);
    case 15: return launch_repulsion_r<15>(ws, n, Y, precision, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_zonly(const Workspace& ws, int32_t n, const float2* Y, int precision, hipStream_t s) {
  switch (ws.plan.R) {
    case 1: return launch_zonly_r<1>(ws, n, Y, precision, s);
    case 2: return launch_zonly_r<2>(ws, n, Y, precision, s);
    case 4: return launch_zonly_r<4>(ws, n, Y, precision, s);
    case 8: return launch_zonly_r<8>(ws, n, Y, precision, s);
    case 16: return launch_zonly_r<16>(ws, n, Y, precision, s);
    case 12: return launch_zonly_r<12>(ws, n, Y, precision, s);
    case 14: return launch_zonly_r<14>(ws, n, Y, precision, s);
    case 15: return launch_zonly_r<15>(ws, n, Y, precision, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_zsum(const Workspace& ws, int precision, hipStream_t s, int32_t* tstep) {
  if (precision == TSGNE_PREC_FP32)
    hipLaunchKernelGGL(k_zsum<false>, dim3(1), dim3(kZThreads), 0, s, ws.zpart, ws.zpart32, ws.plan.items, ws.Z,
                       tstep);
  else
    hipLaunchKernelGGL(k_zsum<true>, dim3(1), dim3(kZThreads), 0, s, ws.zpart, ws.zpart32, ws.plan.items, ws.Z,
                       tstep);
  return hipGetLastError();
}

hipError_t launch_attract(const tsgne_graph* g, const float2* Y, int precision, double2* out, hipStream_t s) {
  const bool split = precision != TSGNE_PREC_FP32;
  const unsigned lb = blocks_for((int64_t)g->n * kRowLanes, kBlock);
  dim3 lb8 = folded_grid((lb + kXcds - 1) / kXcds, kBlock * kXcds);  // whole rounds over the XCDs
  lb8.x *= kXcds;
  if (split)
    hipLaunchKernelGGL(k_attract_light<true>, lb8, dim3(kBlock), 0, s, g->row_ptr, g->col, g->P, Y, g->n, out);
  else
    hipLaunchKernelGGL(k_attract_light<false>, lb8, dim3(kBlock), 0, s, g->row_ptr, g->col, g->P, Y, g->n, out);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || g->n_heavy == 0) return e;
  const unsigned hb = blocks_for(g->n_heavy, kWavesPerBlock);
  if (split)
    hipLaunchKernelGGL(k_attract_heavy<true>, dim3(hb), dim3(kBlock), 0, s, g->row_ptr, g->col, g->P, Y, g->heavy,
                       g->n_heavy, out);
  else
    hipLaunchKernelGGL(k_attract_heavy<false>, dim3(hb), dim3(kBlock), 0, s, g->row_ptr, g->col, g->P, Y, g->heavy,
                       g->n_heavy, out);
  return hipGetLastError();
}

bool plan_fuses_z(const RepulsionPlan& plan) { return plan.items <= kOwnZItems; }

template <int R>
hipError_t launch_forces_r(const tsgne_graph* g, const float2* Y, bool split, int32_t* tstep, hipStream_t s) {
  const Workspace& ws = g->ws;
  const RepulsionPlan& p = ws.plan;
  const int64_t tiles = wave_tile_blocks(p.items, p.diag, R) + p.diag;
  const AttractBlocks mix = mix_attract(tiles, blocks_for((int64_t)g->n * kRowLanes, kBlock),
                                        blocks_for(g->n_heavy, kWavesPerBlock));
  const dim3 grid = mixed_grid(tiles, mix);
  if (split)
    hipLaunchKernelGGL((k_forces<R, true>), grid, dim3(kBlock), 0, s, Y, g->n, p.nb, ws.items, p.items, p.diag,
                       ws.part, ws.zpart, ws.zpart32, g->row_ptr, g->col, g->P, g->heavy, g->n_heavy, ws.attract, mix,
                       tstep);
  else
    hipLaunchKernelGGL((k_forces<R, false>), grid, dim3(kBlock), 0, s, Y, g->n, p.nb, ws.items, p.items, p.diag,
                       ws.part, ws.zpart, ws.zpart32, g->row_ptr, g->col, g->P, g->heavy, g->n_heavy, ws.attract, mix,
                       tstep);
  return hipGetLastError();
}

hipError_t launch_forces(const tsgne_graph* g, const float2* Y, int precision, int32_t* tstep, hipStream_t s) {
  const bool split = precision != TSGNE_PREC_FP32;
  switch (g->ws.plan.R) {
    case 1: return launch_forces_r<1>(g, Y, split, tstep, s);
    case 2: return launch_forces_r<2>(g, Y, split, tstep, s);
    case 4: return launch_forces_r<4>(g, Y, split, tstep, s);
    case 8: return launch_forces_r<8>(g, Y, split, tstep, s);
    case 16: return launch_forces_r<16>(g, Y, split, tstep, s);
    case 12: return launch_forces_r<12>(g, Y, split, tstep, s);
    case 14: return launch_forces_r<14>(g, Y, split, tstep, s);
    case 15: return launch_forces_r<15>(g, Y, split, tstep, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_update(const tsgne_graph* g, float2* Y, float2* U, float2* gains, float alpha, float momentum,
                         float eta, float min_gain, int precision, bool do_update, float2* grad_out, double* Z_out,
                         bool own_z, hipStream_t s, const StepSchedule& sched) {
  const Workspace& ws = g->ws;
  const dim3 grid(blocks_for(g->n, kUpdateRows));
  const bool split = precision != TSGNE_PREC_FP32;
  const UpdateView v{ws.part, ws.attract, ws.zpart, ws.zpart32, ws.Z, Y, U, gains, g->n, ws.plan.nb,
                     own_z ? (int32_t)ws.plan.items : 0};
  if (split && own_z)
    hipLaunchKernelGGL((k_update<true, true>), grid, dim3(kBlock), 0, s, v, ws.plan.T, alpha, momentum, eta, min_gain,
                       (int)do_update, grad_out, Z_out, sched);
  else if (split)
    hipLaunchKernelGGL((k_update<true, false>), grid, dim3(kBlock), 0, s, v, ws.plan.T, alpha, momentum, eta, min_gain,
                       (int)do_update, grad_out, Z_out, sched);
  else if (own_z)
    hipLaunchKernelGGL((k_update<false, true>), grid, dim3(kBlock), 0, s, v, ws.plan.T, alpha, momentum, eta, min_gain,
                       (int)do_update, grad_out, Z_out, sched);
  else
    hipLaunchKernelGGL((k_update<false, false>), grid, dim3(kBlock), 0, s, v, ws.plan.T, alpha, momentum, eta,
                       min_gain, (int)do_update, grad_out, Z_out, sched);
  return hipGetLastError();
}

hipError_t launch_kl(const tsgne_graph* g, const float2* Y, hipStream_t s, const int32_t* tstep, int32_t kl_every,
                     double* trace) {
  const Workspace& ws = g->ws;
  hipLaunchKernelGGL(k_kl_edges, dim3(ws.kl_blocks), dim3(kKLThreads), 0, s, g->row_of, g->col, g->P, Y, g->nnz, ws.Z,
                     ws.klpart, tstep, kl_every);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_kl_final, dim3(1), dim3(kKLThreads), 0, s, ws.klpart, ws.kl_blocks, ws.klout, tstep, kl_every,
                     trace);
  return hipGetLastError();
}

hipError_t launch_kl_ws(const tsgne_graph* g, const Workspace& ws, const float2* Y, hipStream_t s) {
  hipLaunchKernelGGL(k_kl_edges, dim3(ws.kl_blocks), dim3(kKLThreads), 0, s, g->row_of, g->col, g->P, Y, g->nnz, ws.Z,
                     ws.klpart, nullptr, 0);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_kl_final, dim3(1), dim3(kKLThreads), 0, s, ws.klpart, ws.kl_blocks, ws.klout, nullptr, 0,
                     nullptr);
  return hipGetLastError();
}

template <int R>
hipError_t launch_batch_forces_r(const BatchPlan& bp, bool split, hipStream_t s) {
  const int64_t tiles = wave_tile_blocks(bp.n_items, bp.n_diag, R) + bp.n_diag;
  const AttractBlocks mix = mix_attract(tiles, bp.n_light_chunks, blocks_for(bp.n_heavy, kWavesPerBlock));
  const dim3 grid = mixed_grid(tiles, mix);
  if (split)
    hipLaunchKernelGGL((k_batch_forces<R, true>), grid, dim3(kBlock), 0, s, bp.descs, bp.items, bp.n_items, bp.n_diag,
                       bp.light_chunks, bp.heavy, bp.n_heavy, mix);
  else
    hipLaunchKernelGGL((k_batch_forces<R, false>), grid, dim3(kBlock), 0, s, bp.descs, bp.items, bp.n_items, bp.n_diag,
                       bp.light_chunks, bp.heavy, bp.n_heavy, mix);
  return hipGetLastError();
}

hipError_t launch_batch_step(const BatchPlan& bp, const tsgne_params& p, hipStream_t s) {
  const bool split = p.precision != TSGNE_PREC_FP32;
  hipError_t e = hipSuccess;
  switch (bp.R) {
    case 1: e = launch_batch_forces_r<1>(bp, split, s); break;
    case 2: e = launch_batch_forces_r<2>(bp, split, s); break;
    case 4: e = launch_batch_forces_r<4>(bp, split, s); break;
    case 8: e = launch_batch_forces_r<8>(bp, split, s); break;
    case 16: e = launch_batch_forces_r<16>(bp, split, s); break;
    case 12: e = launch_batch_forces_r<12>(bp, split, s); break;
    case 14: e = launch_batch_forces_r<14>(bp, split, s); break;
    case 15: e = launch_batch_forces_r<15>(bp, split, s); break;
    default: e = hipErrorInvalidValue;
  }
  if (e != hipSuccess) return e;
  const bool own_z = bp.max_items <= kOwnZItems;
  if (!own_z) {
    if (split) hipLaunchKernelGGL(k_batch_zsum<true>, dim3(bp.count), dim3(kZThreads), 0, s, bp.descs);
    else hipLaunchKernelGGL(k_batch_zsum<false>, dim3(bp.count), dim3(kZThreads), 0, s, bp.descs);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  const dim3 rows(bp.n_row_blocks);
  if (split && own_z)
    hipLaunchKernelGGL((k_batch_update<true, true>), rows, dim3(kBlock), 0, s, bp.descs, bp.row_blocks, bp.T,
                       p.early_exaggeration, p.exaggeration_iters, p.momentum_early, p.momentum_late, p.min_gain);
  else if (split)
    hipLaunchKernelGGL((k_batch_update<true, false>), rows, dim3(kBlock), 0, s, bp.descs, bp.row_blocks, bp.T,
                       p.early_exaggeration, p.exaggeration_iters, p.momentum_early, p.momentum_late, p.min_gain);
  else if (own_z)
    hipLaunchKernelGGL((k_batch_update<false, true>), rows, dim3(kBlock), 0, s, bp.descs, bp.row_blocks, bp.T,
                       p.early_exaggeration, p.exaggeration_iters, p.momentum_early, p.momentum_late, p.min_gain);
  else
    hipLaunchKernelGGL((k_batch_update<false, false>), rows, dim3(kBlock), 0, s, bp.descs, bp.row_blocks, bp.T,
                       p.early_exaggeration, p.exaggeration_iters, p.momentum_early, p.momentum_late, p.min_gain);
  return hipGetLastError();
}

hipError_t launch_run_init(float2* U, float2* gains, int32_t n, int32_t* tstep, uint32_t* flag, hipStream_t s) {
  hipLaunchKernelGGL(k_run_init, dim3(blocks_for(n, kBlock)), dim3(kBlock), 0, s, U, gains, n, tstep, flag);
  return hipGetLastError();
}

hipError_t launch_nonfinite_check(const float2* Y, int32_t n, uint32_t* flag, hipStream_t s) {
  hipLaunchKernelGGL(k_nonfinite, dim3(blocks_for(n, kBlock)), dim3(kBlock), 0, s, Y, n, flag);
  return hipGetLastError();
}

hipError_t launch_batch_nonfinite_check(const BatchPlan& bp, uint32_t* flag, hipStream_t s) {
  hipLaunchKernelGGL(k_batch_nonfinite, dim3(bp.n_row_blocks), dim3(kUpdateRows), 0, s, bp.descs, bp.row_blocks, flag);
  return hipGetLastError();
}

}  // namespace tsgne
