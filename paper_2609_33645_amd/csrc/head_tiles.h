// Output-tile order and epilogue pieces shared by the bf16 and fp32 vocabulary-head products
// (head_gemm_bf16.hip, head_gemm_f32.hip).  G is a tile engine: a WR x WC grid of wavefronts,
// each with FR x FC accumulator blocks of 32 x 32 (row_of / col_of give an accumulator's place).
#pragma once

#include "pctc_device.h"

namespace pctc {

__device__ __forceinline__ int xcd_swz(int bid, int nblocks) {
  const int full = (nblocks / 8) * 8;
  if (bid >= full) return bid;
  return (bid % 8) * (full / 8) + bid / 8;
}

// Tile order for an nA x nB grid of output tiles, A = frame tiles (few), B = vocabulary
// tiles or partitions (many).  Consecutive work ids walk groups of ga x gb tiles (a
// fastest) with about 64 tiles per group (what one XCD runs at a time) and ga ~ 11 frame
// tiles; the groups walk the frame groups fastest, so the few groups that cover every frame
// tile of a run of vocabulary rows are consecutive: that XCD fetches the rows once and the
// frame tiles (the small operand) stay in its L2.  Grid = ceil(nA/ga) ga * ceil(nB/gb) gb;
// ids past the edge return false.
__host__ __device__ __forceinline__ void group_shape(int nA, int& ga, int& gb) {
  const int groups = (nA + 10) / 11;
  ga = (nA + groups - 1) / groups;
  gb = 64 / ga;
  if (gb < 1) gb = 1;
}
__host__ __device__ __forceinline__ int grouped_grid(int nA, int nB) {
  int ga, gb;
  group_shape(nA, ga, gb);
  return ((nA + ga - 1) / ga) * ga * ((nB + gb - 1) / gb) * gb;
}
__device__ __forceinline__ bool grouped_tile(int work, int nA, int nB, int& a, int& b) {
  int ga, gb;
  group_shape(nA, ga, gb);
  const int gA = (nA + ga - 1) / ga;
  const int blk = work / (ga * gb), in = work % (ga * gb);
  a = (blk % gA) * ga + in % ga;
  b = (blk / gA) * gb + in / ga;
  return a < nA && b < nB;
}

// Accumulators of a tile start at the bias of their row (bt: the tile's rows, in LDS).
template <int FR, int FC, class G>
__device__ __forceinline__ void bias_init(f32x16 (&acc)[FR][FC], const float* bt, int wave, int lane) {
#pragma unroll
  for (int i = 0; i < FR; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 b4 = *reinterpret_cast<const float4*>(bt + G::row_of(wave, lane, i, 4 * q));
#pragma unroll
      for (int j = 0; j < FC; ++j) {
        acc[i][j][4 * q + 0] = b4.x;
        acc[i][j][4 * q + 1] = b4.y;
        acc[i][j][4 * q + 2] = b4.z;
        acc[i][j][4 * q + 3] = b4.w;
      }
    }
}

// Adds the bias of each row to a tile (bt: the tile's rows, in LDS).
template <int FR, int FC, class G>
__device__ __forceinline__ void bias_add(f32x16 (&acc)[FR][FC], const float* bt, int wave, int lane) {
#pragma unroll
  for (int i = 0; i < FR; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 b4 = *reinterpret_cast<const float4*>(bt + G::row_of(wave, lane, i, 4 * q));
#pragma unroll
      for (int j = 0; j < FC; ++j) {
        acc[i][j][4 * q + 0] += b4.x;
        acc[i][j][4 * q + 1] += b4.y;
        acc[i][j][4 * q + 2] += b4.z;
        acc[i][j][4 * q + 3] += b4.w;
      }
    }
}

// Logits of rows at or past vend (a partition's ragged last tile, whose rows read as zeros)
// become -inf in place, so that the update below treats every tile alike.  Each row test is
// used at once for the FC columns it covers (a lane holds 4 consecutive rows per group):
// keeping one test per accumulator live across both passes of the update would take a mask
// register pair per element.
template <int FR, int FC, class G>
__device__ __forceinline__ void mask_rows_inf(f32x16 (&acc)[FR][FC], int v0, int vend, int wave, int lane) {
#pragma unroll
  for (int i = 0; i < FR; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int lim = vend - v0 - G::row_of(wave, lane, i, 4 * q);  // rows e < lim are in range
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool out = e >= lim;
#pragma unroll
        for (int j = 0; j < FC; ++j) acc[i][j][4 * q + e] = out ? -INFINITY : acc[i][j][4 * q + e];
      }
    }
}

// Online log-sum-exp update of the running (max, sum) of this lane's frames with one
// tile of logits (bias included; out-of-range rows already -inf).
template <int FR, int FC, class G>
__device__ __forceinline__ void lse_tile_update(const f32x16 (&acc)[FR][FC], float (&run_max)[FC],
                                                float (&run_sum)[FC]) {
#pragma unroll
  for (int j = 0; j < FC; ++j) {
    float tmax = -INFINITY;
#pragma unroll
    for (int i = 0; i < FR; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) tmax = fmaxf(tmax, acc[i][j][r]);
    tmax = fmaxf(tmax, swap_halves(tmax));
    const float nmax = fmaxf(run_max[j], tmax);
    // a column with no finite logit yet (rows masked by a -inf bias) adds nothing
    const float ms = (nmax == -INFINITY) ? 0.f : nmax * kLog2e;
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < FR; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) s += fast_exp2(fmaf(acc[i][j][r], kLog2e, -ms));
    s += swap_halves(s);
    const float scale = (run_max[j] == -INFINITY) ? 0.f : fast_exp2((run_max[j] - nmax) * kLog2e);
    run_sum[j] = fmaf(run_sum[j], scale, s);
    run_max[j] = nmax;
  }
}

// The two wavefronts of each frame column (row halves) combine their running (max, sum)
// pairs through LDS (xch: any drained stage) and write the partition's pair of every frame.
template <class G>
__device__ __forceinline__ void lse_store_partials(const float (&run_max)[G::FC], const float (&run_sum)[G::FC],
                                                   char* xchb, int wave, int lane, int m0, int M,
                                                   float2* __restrict__ out) {
  constexpr int FC = G::FC;
  __syncthreads();
  constexpr int WC = G::NW / 2;  // column groups (the wave grid is 2 x WC)
  float2* xch = reinterpret_cast<float2*>(xchb);
  const int rowhalf = wave / WC, colq = wave % WC;
  if (rowhalf == 1 && lane < 32) {
#pragma unroll
    for (int j = 0; j < FC; ++j) xch[colq * (FC * 32) + j * 32 + lane] = make_float2(run_max[j], run_sum[j]);
  }
  __syncthreads();
  if (rowhalf == 0 && lane < 32) {
#pragma unroll
    for (int j = 0; j < FC; ++j) {
      const float2 o = xch[colq * (FC * 32) + j * 32 + lane];
      const float nmax = fmaxf(run_max[j], o.x);
      float s = 0.f;
      if (run_max[j] != -INFINITY) s += run_sum[j] * fast_exp2((run_max[j] - nmax) * kLog2e);
      if (o.x != -INFINITY) s += o.y * fast_exp2((o.x - nmax) * kLog2e);
      if (nmax != nmax) s = nmax;
      const int m = m0 + G::col_of(wave, lane, j);
      if (m < M) out[m] = make_float2(nmax, s);
    }
  }
}

__device__ __forceinline__ void amax_merge(float& bv, int& bi, float ov, int oi) {
  if (ov > bv || (ov == bv && oi < bi)) {
    bv = ov;
    bi = oi;
  }
}

// Framewise best (value, class) of this lane's rows with one tile of logits (out-of-range rows
// already -inf, which never replaces the best).
template <int FR, int FC, class G>
__device__ __forceinline__ void amax_tile_update(const f32x16 (&a)[FR][FC], int v0, int wave, int lane,
                                                 float (&bv)[FC], int (&bi)[FC]) {
  // the lane's rows increase with (i, r): the tile's best is its largest logit at the first
  // row holding it (found scanning backwards), and it replaces the running best only when
  // strictly larger, so ties keep the smallest id; NaN never compares equal or larger
  const int rbase = v0 + G::row_of(wave, lane, 0, 0);
#pragma unroll
  for (int j = 0; j < FC; ++j) {
    float tmax = -INFINITY;
#pragma unroll
    for (int i = 0; i < FR; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) tmax = fmaxf(tmax, a[i][j][r]);
    int off = 0;
#pragma unroll
    for (int i = FR - 1; i >= 0; --i)
#pragma unroll
      for (int r = 15; r >= 0; --r) off = (a[i][j][r] == tmax) ? 32 * i + 8 * (r >> 2) + (r & 3) : off;
    if (tmax > bv[j]) {
      bv[j] = tmax;
      bi[j] = rbase + off;
    }
  }
}

// The lane halves, then the two wavefronts of each frame column, combine their best pairs
// (xchb: any drained stage) and write the partition's pair of every frame.
template <class G>
__device__ __forceinline__ void amax_store_partials(float (&bv)[G::FC], int (&bi)[G::FC], char* xchb, int wave,
                                                    int lane, int m0, int M, float2* __restrict__ out) {
  constexpr int FC = G::FC;
  // lane halves hold the other half of each 32-row block, then the row halves of the tile
#pragma unroll
  for (int j = 0; j < FC; ++j) {
    const float ov = swap_halves(bv[j]);
    const int oi = __shfl_xor(bi[j], 32, 64);
    amax_merge(bv[j], bi[j], ov, oi);
  }
  __syncthreads();
  float2* xch = reinterpret_cast<float2*>(xchb);
  constexpr int WC = G::NW / 2;  // column groups (the wave grid is 2 x WC)
  const int rowhalf = wave / WC, colq = wave % WC;
  if (rowhalf == 1 && lane < 32) {
#pragma unroll
    for (int j = 0; j < FC; ++j)
      xch[colq * (FC * 32) + j * 32 + lane] = make_float2(bv[j], __int_as_float(bi[j]));
  }
  __syncthreads();
  if (rowhalf == 0 && lane < 32) {
#pragma unroll
    for (int j = 0; j < FC; ++j) {
      const float2 o = xch[colq * (FC * 32) + j * 32 + lane];
      amax_merge(bv[j], bi[j], o.x, __float_as_int(o.y));
      const int m = m0 + G::col_of(wave, lane, j);
      if (m < M) out[m] = make_float2(bv[j], __int_as_float(bi[j]));
    }
  }
}

}  // namespace pctc
