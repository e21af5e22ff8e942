// fp32 vocabulary-head products of Pruned CTC on the split tile engine (gemm_f32.h):
//  * lse_partial_f32:   Z^T tile = W H^T with the online log-sum-exp epilogue (Eq. lognorm;
//    Algorithm 1 online log-sum-exp over vocabulary chunks);
//  * amax_partial_f32:  the same tiles with a framewise argmax (greedy emission head);
//  * gather_s_f32:      S = Z[:, U] - lambda, subtraction in double, one rounding to float
//    (Algorithm 1; App. B.1 "Forward computation");
//  * recompute_dz_f32:  dZ = scatter_U(G) - g p for one vocabulary chunk (Eq. vjp), fp32;
//  * products_f32:      dH += dZ W_c and dW_c = dZ^T H in one launch (App. A, Step 3).
// M = 16,000 frames, D = 512, V = 180,000 (160 utterances, one call): the fp32 matrix units ran
// these products at 110 TFLOP/s; see each kernel for what it measures now.
#include <algorithm>

#include "gemm_f32.h"
#include "head_tiles.h"
#include "pctc_internal.h"

namespace pctc {

namespace {

using f3::GOp;
using bf::LL;

using GZ = f3::Gemm<LL::KC, LL::KC>;               // Z^T = W H^T
using GZGather = f3::Gemm<LL::KC, LL::KC, false>;  // the same over gathered W rows
using GH = f3::Gemm<LL::KC, LL::MC>;               // dH = dZ W
using GW = f3::Gemm<LL::MC, LL::MC>;               // dW = dZ^T H
constexpr int kTile = f3::kT;
// dZ is kept times 2^24 (exact, and taken off where its products and sums are written), so that
// probabilities down to fp32's least split into parts without loss (see gemm_f32.h); loss weights and
// gradients up to 2^103 stay finite.
constexpr float kDzScale = 16777216.f, kDzUnscale = 1.f / kDzScale;

#define PCTC_F3_STAGES                                                          \
  __shared__ __attribute__((aligned(1024))) char st0_[GZ::kStageBytes];         \
  __shared__ __attribute__((aligned(1024))) char st1_[GZ::kStageBytes];         \
  __shared__ __attribute__((aligned(1024))) char st2_[GZ::kStageBytes];         \
  __shared__ __attribute__((aligned(1024))) char st3_[GZ::kStageBytes];         \
  char* const st[4] = {st0_, st1_, st2_, st3_};

// Workgroup of a partitioned vocabulary pass: `run` vocabulary tiles of partition p for frame
// tile mt; epi(v0, lane, acc) after each tile, the bias added.  A tile's bias waits in LDS (two
// tiles' room, in turn: no wavefront is two tiles ahead of another), so a partition may be any
// number of tiles.
template <bool BIAS, class Epi>
__device__ __forceinline__ void vocab_tiles(const float* H, int M, int D, const float* W, const float* bias, int m0,
                                            int vbeg, int vend, char* const (&st)[4], Epi&& epi) {
  __shared__ __attribute__((aligned(16))) float bsh[2][BIAS ? kTile : 4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int ntiles = (vend - vbeg + kTile - 1) / kTile;
  const GOp A{W, D, vend, D, nullptr};
  const GOp B{H, D, M, D, nullptr};
  f32x16 acc[GZ::FR][GZ::FC];
  for (int i = 0; i < ntiles; ++i) {
    const int v0 = vbeg + i * kTile;
    if (BIAS && tid < kTile) bsh[i & 1][tid] = (v0 + tid < vend) ? bias[v0 + tid] : 0.f;
    GZ::run(A, B, v0, m0, 0, D, st, acc);
    // an opaque lane: what the epilogue derives from it is not kept in registers through the next
    // tile's products (it would spill there)
    int el = lane;
    asm volatile("" : "+v"(el));
    if (BIAS) bias_add<GZ::FR, GZ::FC, GZ>(acc, bsh[i & 1], wave, el);
    if (v0 + kTile > vend) mask_rows_inf<GZ::FR, GZ::FC, GZ>(acc, v0, vend, wave, el);
    epi(v0, el, acc);
  }
}

// A wave's block of 32 frames x 128 tile rows (row_of order) through its own 16 KB of the drained
// stages, so that global memory is written in runs along the rows: lane 32 h + f holds frame f
// and, in put(i, q, v), its rows 32 i + 8 q + 4 h ..+3; get(f, c) gives rows 4 c ..+3 of frame f
// (16-byte slots XORed with f mod 16: 16 lanes of a write phase fall in 16 different bank
// groups).  A wave's LDS accesses are ordered; no barrier is needed.
struct WaveBlock {
  char* base;
  int lane;
  __device__ __forceinline__ void put(int i, int q, const float4& v) {
    const int f = lane & 31, c = 8 * i + 2 * q + (lane >> 5);
    *reinterpret_cast<float4*>(base + f * 512 + ((c ^ (f & 15)) << 4)) = v;
  }
  __device__ __forceinline__ float4 get(int f, int c) const {
    return *reinterpret_cast<const float4*>(base + f * 512 + ((c ^ (f & 15)) << 4));
  }
};
__device__ __forceinline__ WaveBlock wave_block(char* const (&st)[4], int wave, int lane) {
  static_assert(GZ::kStageBytes == 32768, "two waves per stage");
  char* const s = (wave >> 1) == 0 ? st[0] : (wave >> 1) == 1 ? st[1] : (wave >> 1) == 2 ? st[2] : st[3];
  return WaveBlock{s + (wave & 1) * 16384, lane};
}

}  // namespace

template <bool BIAS>
__global__ void __launch_bounds__(512, 1)
lse_partial_f32(const float* __restrict__ H, int M, int D, const float* __restrict__ W, const float* __restrict__ bias,
                int V, int P, int vper, float2* __restrict__ partials) {
  PCTC_F3_STAGES
  int mt, p;
  if (!grouped_tile(xcd_swz(blockIdx.x, gridDim.x), (M + kTile - 1) / kTile, P, mt, p)) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int m0 = mt * kTile, vbeg = p * vper, vend = min(V, vbeg + vper);
  float run_max[GZ::FC], run_sum[GZ::FC];
#pragma unroll
  for (int j = 0; j < GZ::FC; ++j) {
    run_max[j] = -INFINITY;
    run_sum[j] = 0.f;
  }
  vocab_tiles<BIAS>(H, M, D, W, bias, m0, vbeg, vend, st, [&](int, int, f32x16 (&a)[GZ::FR][GZ::FC]) {
    lse_tile_update<GZ::FR, GZ::FC, GZ>(a, run_max, run_sum);
  });
  lse_store_partials<GZ>(run_max, run_sum, st0_, wave, lane, m0, M, partials + static_cast<int64_t>(p) * M);
}

template <bool BIAS>
__global__ void __launch_bounds__(512, 1)
amax_partial_f32(const float* __restrict__ H, int M, int D, const float* __restrict__ W,
                 const float* __restrict__ bias, int V, int P, int vper, float2* __restrict__ partials) {
  PCTC_F3_STAGES
  int mt, p;
  if (!grouped_tile(xcd_swz(blockIdx.x, gridDim.x), (M + kTile - 1) / kTile, P, mt, p)) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int m0 = mt * kTile, vbeg = p * vper, vend = min(V, vbeg + vper);
  float bv[GZ::FC];
  int bi[GZ::FC];
#pragma unroll
  for (int j = 0; j < GZ::FC; ++j) {
    bv[j] = -INFINITY;
    bi[j] = 0x7fffffff;
  }
  vocab_tiles<BIAS>(H, M, D, W, bias, m0, vbeg, vend, st, [&](int v0, int el, f32x16 (&a)[GZ::FR][GZ::FC]) {
    amax_tile_update<GZ::FR, GZ::FC, GZ>(a, v0, wave, el, bv, bi);
  });
  amax_store_partials<GZ>(bv, bi, st0_, wave, lane, m0, M, partials + static_cast<int64_t>(p) * M);
}

__global__ void __launch_bounds__(512, 1)
gather_s_f32(const float* __restrict__ H, int M, int D, const float* __restrict__ W, const float* __restrict__ bias,
             const int32_t* __restrict__ u_ids, const int32_t* __restrict__ Kdev, const double* __restrict__ lam,
             float* __restrict__ S, int ldS, float* __restrict__ Gz) {
  using G = GZGather;
  PCTC_F3_STAGES
  const int nMt = (M + kTile - 1) / kTile;
  const int m0 = (blockIdx.x % nMt) * kTile, j0 = (blockIdx.x / nMt) * kTile;
  const int K = *Kdev;
  if (j0 >= K) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const GOp A{W, D, K, D, u_ids};
  const GOp B{H, D, M, D, nullptr};
  f32x16 acc[G::FR][G::FC];
  G::run(A, B, j0, m0, 0, D, st, acc);
  WaveBlock blk = wave_block(st, wave, lane);
  const int jw = j0 + (wave / G::WC) * (kTile / G::WR);  // the wave's first selected class
#pragma unroll
  for (int j = 0; j < G::FC; ++j) {
#pragma unroll
    for (int i = 0; i < G::FR; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        blk.put(i, q, make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]));
    const int mw = m0 + (wave % G::WC) * (kTile / G::WC) + 32 * j;  // its first frame
    const int n = min(32, M - mw);
    for (int f = lane >> 5; f < n; f += 2) {
      const double l = lam[mw + f];
      const float4 z = blk.get(f, lane & 31);
      float* const srow = S + static_cast<int64_t>(mw + f) * ldS;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int jj = jw + 4 * (lane & 31) + e;
        if (jj < K) {
          double v = static_cast<double>(e == 0 ? z.x : e == 1 ? z.y : e == 2 ? z.z : z.w);
          if (bias) v += static_cast<double>(bias[u_ids[jj]]);
          srow[jj] = static_cast<float>(v - l);
          if (Gz) Gz[static_cast<int64_t>(mw + f) * ldS + jj] = 0.f;
        }
      }
    }
  }
}

// dZ chunk [M][chunk] (row pitch `chunk`): columns v_local in [0, cw) hold scatter_U(G) - g p of
// class c0 + v_local, times kDzScale, columns in [cw, tile end) zeros; rows of excluded frames (g = 0) zeros.
template <bool BIAS>
__global__ void __launch_bounds__(512, 1)
recompute_dz_f32(const float* __restrict__ H, int M, int D, const float* __restrict__ W,
                 const float* __restrict__ bias, int c0, int cw, const float2* __restrict__ lam2,
                 const float* __restrict__ G, int ldG, const float* __restrict__ g, const int32_t* __restrict__ remap,
                 float* __restrict__ dZ, int chunk) {
  PCTC_F3_STAGES
  __shared__ __attribute__((aligned(16))) float bl[BIAS ? kTile : 4];
  __shared__ int sel[kTile];
  int mt, vt;
  if (!grouped_tile(xcd_swz(blockIdx.x, gridDim.x), (M + kTile - 1) / kTile, (cw + kTile - 1) / kTile, mt, vt)) return;
  const int m0 = mt * kTile, vl0 = vt * kTile;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int jsel = -1;
  if (tid < kTile) {
    const bool in = vl0 + tid < cw;
    jsel = in ? remap[c0 + vl0 + tid] : -1;
    sel[tid] = jsel;
    if (BIAS) bl[tid] = in ? bias[c0 + vl0 + tid] : 0.f;
  }
  const int any_sel = __syncthreads_or(jsel >= 0);
  const GOp A{W + static_cast<int64_t>(c0) * D, D, cw, D, nullptr};
  const GOp B{H, D, M, D, nullptr};
  f32x16 acc[GZ::FR][GZ::FC];
  GZ::run(A, B, vl0, m0, 0, D, st, acc);
  if (BIAS) bias_add<GZ::FR, GZ::FC, GZ>(acc, bl, wave, lane);
  const bool ragged = vl0 + kTile > cw;
  WaveBlock blk = wave_block(st, wave, lane);
  const int rw = (wave / GZ::WC) * (kTile / GZ::WR);  // the wave's first tile row
#pragma unroll
  for (int j = 0; j < GZ::FC; ++j) {
    const int m = min(m0 + GZ::col_of(wave, lane, j), M - 1);  // frames past M are not stored
    const float gm = g[m] * kDzScale;
    const float2 l2 = lam2[m];
    const bool inc = gm != 0.f;
#pragma unroll
    for (int i = 0; i < GZ::FR; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int rl0 = GZ::row_of(wave, lane, i, 4 * q);  // 4 consecutive classes
        float out[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float t = fmaf(acc[i][j][4 * q + e], kLog2e, -l2.x) - l2.y;
          out[e] = inc ? -gm * fast_exp2(t) : 0.f;
        }
        if (ragged) {
#pragma unroll
          for (int e = 0; e < 4; ++e) out[e] = (vl0 + rl0 + e < cw) ? out[e] : 0.f;
        }
        blk.put(i, q, make_float4(out[0], out[1], out[2], out[3]));
      }
    const int mw = m0 + (wave % GZ::WC) * (kTile / GZ::WC) + 32 * j;
    float* const dw = dZ + static_cast<int64_t>(mw) * chunk + vl0 + rw + 4 * (lane & 31);
    // streaming stores (dZ is read back by the products only): 820 us a launch of 8192 columns at
    // M = 16,000, 870 cached, 800 without any
    if (any_sel) {
      // the union columns of the lane's 4: their indices rise with the class, so a frame's G
      // values are read in runs (other columns read column 0: no branch, so that the loads of
      // several frames are in flight)
      int sj[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) sj[e] = sel[rw + 4 * (lane & 31) + e];
#pragma unroll 8
      for (int f = lane >> 5; f < 32; f += 2) {
        const int mf = min(mw + f, M - 1);
        const float* const grow = G + static_cast<int64_t>(mf) * ldG;
        const bool inc = g[mf] != 0.f;
        float gv[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) gv[e] = grow[max(sj[e], 0)];
        const float4 zz = blk.get(f, lane & 31);
        f3::f32x4 z = {zz.x, zz.y, zz.z, zz.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) z[e] += (inc && sj[e] >= 0) ? gv[e] * kDzScale : 0.f;
        if (mw + f < M) __builtin_nontemporal_store(z, reinterpret_cast<f3::f32x4*>(dw + static_cast<int64_t>(f) * chunk));
      }
    } else {
#pragma unroll 4
      for (int f = lane >> 5; f < 32; f += 2) {
        const float4 zz = blk.get(f, lane & 31);
        const f3::f32x4 z = {zz.x, zz.y, zz.z, zz.w};
        if (mw + f < M) __builtin_nontemporal_store(z, reinterpret_cast<f3::f32x4*>(dw + static_cast<int64_t>(f) * chunk));
      }
    }
  }
}

// One launch for both products of a chunk.
//   dH: part[s] (+)= dZ[:, slice s] W[c0 + slice s, :] over ns slices of `slice` columns; the
//       first chunk writes every slice (zeros when its range is empty), later ones add.
//   dW: dW[c0 + v, :] = sum over frames of dZ[m][v] Hs[m, :], the frames cut into nz slices of
//       mslice; slice 0 writes dW itself, slice z > 0 its partial sums at wpart[z - 1].
// The two have the same work, but neither fills the chip evenly alone; the slices (plan_bwd) are
// chosen so that the union of both does, and the longer workgroups come first.
struct ProductsF32 {
  const float* dZ;
  int M, chunk;
  const float* W;   // row c0
  const float* Hs;  // excluded rows zero
  int D, cw, slice, ns, nh;  // nh: dH workgroups (0: no dH)
  float* part;
  bool first;
  int nz, mslice, nw;  // nw: dW workgroups (0: no dW)
  float *dW, *wpart;   // dW: row c0
  bool dw_first;       // dW's workgroups first
};

__global__ void __launch_bounds__(512, 1) products_f32(ProductsF32 P) {
  PCTC_F3_STAGES
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int nfirst = P.dw_first ? P.nw : P.nh;
  const bool lead = static_cast<int>(blockIdx.x) < nfirst;
  const int bid = lead ? blockIdx.x : blockIdx.x - nfirst;
  const int nDt = (P.D + kTile - 1) / kTile;
  f32x16 acc[GH::FR][GH::FC];
  if (lead != P.dw_first) {  // dH
    const int work = xcd_swz(bid, P.nh);
    const int nMt = (P.M + kTile - 1) / kTile;
    const int dt = work % nDt, mt = (work / nDt) % nMt, s = work / (nDt * nMt);
    const int m0 = mt * kTile, d0 = dt * kTile;
    const int kb = s * P.slice, ke = min(P.cw, kb + P.slice);
    if (kb >= ke && !P.first) return;
    float* const dst = P.part + static_cast<int64_t>(s) * P.M * P.D;
    // zero starting values, the earlier chunks' sums added at the end: a chain of additions onto
    // a sum that the union columns made large loses more (1.4e-5 against 1.4e-6 at V = 180,000)
    const GOp A{P.dZ, P.chunk, P.M, P.cw, nullptr};
    const GOp B{P.W, P.D, P.D, P.cw, nullptr};
    GH::run(A, B, m0, d0, kb, ke, st, acc);
#pragma unroll
    for (int i = 0; i < GH::FR; ++i)
#pragma unroll
      for (int j = 0; j < GH::FC; ++j) {
        const int d = d0 + GH::col_of(wave, lane, j);
        if (d >= P.D) continue;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int m = m0 + GH::row_of(wave, lane, i, r);
          if (m < P.M) {
            float* const o = dst + static_cast<int64_t>(m) * P.D + d;
            const float x = acc[i][j][r] * kDzUnscale;
            *o = P.first ? x : *o + x;
          }
        }
      }
  } else {  // dW
    const int work = xcd_swz(bid, P.nw);
    const int nVt = (P.cw + kTile - 1) / kTile;
    const int dt = work % nDt, vt = (work / nDt) % nVt, z = work / (nDt * nVt);
    const int v0 = vt * kTile, d0 = dt * kTile;
    const int kb = z * P.mslice, ke = min(P.M, kb + P.mslice);
    const GOp A{P.dZ, P.chunk, P.cw, P.M, nullptr};
    const GOp B{P.Hs, P.D, P.D, P.M, nullptr};
    GW::run(A, B, v0, d0, kb, ke, st, acc);
    float* const dst = z == 0 ? P.dW : P.wpart + static_cast<int64_t>(z - 1) * P.cw * P.D;
#pragma unroll
    for (int i = 0; i < GW::FR; ++i)
#pragma unroll
      for (int j = 0; j < GW::FC; ++j) {
        const int d = d0 + GW::col_of(wave, lane, j);
        if (d >= P.D) continue;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int v = v0 + GW::row_of(wave, lane, i, r);
          if (v < P.cw) dst[static_cast<int64_t>(v) * P.D + d] = acc[i][j][r] * kDzUnscale;
        }
      }
  }
}

// dW[i] += sum over the further frame slices (fixed order), n a multiple of 4.
__global__ void __launch_bounds__(256)
dw_reduce_f32(const float* __restrict__ wpart, int slices, int64_t n, float* __restrict__ dW) {
  const int64_t i = (static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x) * 4;
  if (i >= n) return;
  float4 s = *reinterpret_cast<const float4*>(dW + i);
  for (int z = 0; z < slices; ++z) {
    const float4 p = *reinterpret_cast<const float4*>(wpart + z * n + i);
    s.x += p.x;
    s.y += p.y;
    s.z += p.z;
    s.w += p.w;
  }
  *reinterpret_cast<float4*>(dW + i) = s;
}

// Hs = H with the rows of excluded frames (g[m] == 0) set to zero.
__global__ void __launch_bounds__(256)
hs_build_f32(const float* __restrict__ H, int64_t n, int D, const float* __restrict__ g, float* __restrict__ Hs) {
  const int64_t i = (static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x) * 4;
  if (i >= n) return;
  float4 v = *reinterpret_cast<const float4*>(H + i);
  if (g[i / D] == 0.f) v = make_float4(0.f, 0.f, 0.f, 0.f);
  *reinterpret_cast<float4*>(Hs + i) = v;
}

// db[v] = sum over frames of dZ[m][v], v < cw, in two launches.  The first cuts the frames into
// slices, a workgroup per slice and 256 columns (64 lanes x 4 columns, its four wavefronts taking
// every fourth frame); the second adds the slices.  Bound by reading dZ: one workgroup per 256
// columns walking all frames took 6.0 ms at M = 16,000, V = 5,000 (a 16,000-load serial chain
// on 20 workgroups).
__global__ void __launch_bounds__(256)
db_colsum_f32(const float* dZ, int M, int chunk, int mper, float* dbpart) {  // dbpart may be dZ (one slice)
  __shared__ float4 x[4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int v = blockIdx.x * 256 + lane * 4;  // the chunk's pitch is a multiple of 256
  const int mb = blockIdx.y * mper, me = min(M, mb + mper);
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
  for (int m = mb + wave; m < me; m += 4) {
    const float4 z = *reinterpret_cast<const float4*>(dZ + static_cast<int64_t>(m) * chunk + v);
    s.x += z.x;
    s.y += z.y;
    s.z += z.z;
    s.w += z.w;
  }
  x[wave][lane] = s;
  __syncthreads();
  if (wave == 0) {
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      const float4 z = x[w][lane];
      s.x += z.x;
      s.y += z.y;
      s.z += z.z;
      s.w += z.w;
    }
    *reinterpret_cast<float4*>(dbpart + static_cast<int64_t>(blockIdx.y) * chunk + v) = s;
  }
}
__global__ void __launch_bounds__(256)
db_reduce_f32(const float* __restrict__ dbpart, int slices, int chunk, int cw, float* __restrict__ db) {
  const int v = blockIdx.x * 256 + threadIdx.x;
  if (v >= cw) return;
  float s = 0.f;
  for (int z = 0; z < slices; ++z) s += dbpart[static_cast<int64_t>(z) * chunk + v];
  db[v] = s * kDzUnscale;
}

// ---------------------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------------------

// One vocabulary tile per workgroup while the partitions fit the partial buffer (every tile
// starts its own copy pipeline, so longer runs would only coarsen the last round).
static void lse_split_f32(int D, int V, int* vper, int* P) {
  const int vtiles = (V + kTile - 1) / kTile;
  const int run = (vtiles + lse_max_parts(D) - 1) / lse_max_parts(D);
  *vper = run * kTile;
  *P = (V + *vper - 1) / *vper;
}

hipError_t launch_lse_partial_f32(const float* H, int M, int D, const float* W, const float* bias, int V,
                                  float2* partials, int* P_out, hipStream_t stream) {
  int vper, P;
  lse_split_f32(D, V, &vper, &P);
  *P_out = P;
  const dim3 grid(grouped_grid((M + kTile - 1) / kTile, P));
  Prof pr("lse_partial", stream);
  if (bias)
    hipLaunchKernelGGL(lse_partial_f32<true>, grid, dim3(512), 0, stream, H, M, D, W, bias, V, P,
                       vper, partials);
  else
    hipLaunchKernelGGL(lse_partial_f32<false>, grid, dim3(512), 0, stream, H, M, D, W, bias, V, P, vper, partials);
  return hipGetLastError();
}

hipError_t launch_amax_partial_f32(const float* H, int M, int D, const float* W, const float* bias, int V,
                                   float2* partials, int* P_out, hipStream_t stream) {
  int vper, P;
  lse_split_f32(D, V, &vper, &P);
  *P_out = P;
  const dim3 grid(grouped_grid((M + kTile - 1) / kTile, P));
  Prof pr("amax_partial", stream);
  if (bias)
    hipLaunchKernelGGL(amax_partial_f32<true>, grid, dim3(512), 0, stream, H, M, D, W, bias, V, P,
                       vper, partials);
  else
    hipLaunchKernelGGL(amax_partial_f32<false>, grid, dim3(512), 0, stream, H, M, D, W, bias, V, P, vper, partials);
  return hipGetLastError();
}

hipError_t launch_gather_s_f32(const float* H, int M, int D, const float* W, const float* bias, const int32_t* u_ids,
                               const int32_t* K, int K_max, const double* lam, float* S, int ldS, hipStream_t stream,
                               float* Gz) {
  const int tiles = ((M + kTile - 1) / kTile) * ((K_max + kTile - 1) / kTile);
  Prof pr("gather_s", stream);
  hipLaunchKernelGGL(gather_s_f32, dim3(tiles), dim3(512), 0, stream, H, M, D, W, bias, u_ids, K, lam, S, ldS, Gz);
  return hipGetLastError();
}

// Time of nl workgroups of length ll (the longer) then ns of length ls on 256 compute units.
static double two_class_span(int nl, double ll, int ns, double ls) {
  const int full = nl / 256, rem = nl % 256;
  const double t0 = full * ll, t1 = (full + 1) * ll;  // 256 - rem units are free at t0, rem at t1
  const double end = rem ? t1 : t0;
  if (ns == 0) return end;
  for (int a = 1;; ++a) {  // the a-th short workgroup of the units free at t0
    const double t = t0 + a * ls;
    int64_t done = static_cast<int64_t>(256 - rem) * a;
    if (rem && t >= t1 + ls) done += static_cast<int64_t>(rem) * static_cast<int>((t - t1) / ls);
    if (done >= ns) return std::max(end, t);
    if (a > 1 << 16) return t;
  }
}

// Slices of the two products of a chunk (see products_f32): the pair whose launch is shortest by
// a model of a 16-deep k-step of 1.6 us, 4 us per workgroup, and partial sums written and read
// at 3 TB/s; partial sums stay within 64 MiB each.  At M = 16,000, D = 512, 8192 columns: 126 dH
// tiles of 512 steps whole, 64 dW tiles of 1000 steps in two slices, 254 workgroups.
void plan_products_f32(int M, int D, int cols, int* splits, int* wsplits) {
  static const int cand[] = {1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 24, 32, 48, 64};
  const int nMt = (M + kTile - 1) / kTile, nDt = (D + kTile - 1) / kTile, nVt = (cols + kTile - 1) / kTile;
  const double kCap = 64.0 * 1024 * 1024, kBw = 3.0e6;  // bytes per us
  *splits = *wsplits = 1;
  double best = -1;
  for (int sh : cand) {
    if (sh > 1 && (cols / sh < 64 || static_cast<double>(sh) * M * D * 4 > kCap)) break;
    const int slice = ((cols + sh - 1) / sh + 63) / 64 * 64;
    const double lh = slice / 16 * 1.6 + 4, ch = sh > 1 ? sh * (static_cast<double>(M) * D * 8) / kBw + 4 : 0;
    for (int sw : cand) {
      if (sw > 1 && (M / sw < 64 || static_cast<double>(sw - 1) * cols * D * 4 > kCap)) break;
      const double lw = ((M + sw - 1) / sw + 15) / 16 * 1.6 + 4;
      const double cw = sw > 1 ? (sw - 1) * (static_cast<double>(cols) * D * 8) / kBw + 6 : 0;
      const int nh = nMt * nDt * sh, nw = nVt * nDt * sw;
      const double t = ch + cw + (lh >= lw ? two_class_span(nh, lh, nw, lw) : two_class_span(nw, lw, nh, lh));
      if (best < 0 || t < best) {
        best = t;
        *splits = sh;
        *wsplits = sw;
      }
    }
  }
}

hipError_t head_bwd_f32(const float* H, int M, int D, const float* W, const float* bias, int V, const float2* lam2,
                        const float* G, int ldG, const float* g, const int32_t* remap, float* dH, float* dW, float* db,
                        char* scratch, const BwdPlan& plan, hipStream_t stream) {
  float* dZ = reinterpret_cast<float*>(scratch);
  float* Hs = reinterpret_cast<float*>(scratch + plan.dz_bytes);
  // a single dH slice accumulates in the caller's dH
  const bool in_place = plan.part_bytes == 0;
  float* part = in_place ? dH : reinterpret_cast<float*>(scratch + plan.dz_bytes + plan.ht_bytes);
  float* dbpart = reinterpret_cast<float*>(scratch + plan.dz_bytes + plan.ht_bytes + plan.part_bytes + plan.lam2_bytes);
  float* wpart = reinterpret_cast<float*>(reinterpret_cast<char*>(dbpart) + plan.dbpart_bytes + plan.hst_bytes);
  const int chunk = plan.chunk;
  const int nMt = (M + kTile - 1) / kTile, nDt = (D + kTile - 1) / kTile;
  const int64_t nH = static_cast<int64_t>(M) * D;
  if (dW) {
    Prof pr("hs_build", stream);
    hipLaunchKernelGGL(hs_build_f32, dim3(static_cast<unsigned>((nH / 4 + 255) / 256)), dim3(256), 0, stream, H, nH, D,
                       g, Hs);
  }
  const int cmax = std::min(chunk, V);
  const int slice = ((cmax + plan.splits - 1) / plan.splits + 63) / 64 * 64;
  const int nslices = (cmax + slice - 1) / slice;  // slices the first (widest) chunk starts
  const int mslice = ((M + plan.wsplits - 1) / plan.wsplits + 15) / 16 * 16;
  const int nz = (M + mslice - 1) / mslice;
  for (int c0 = 0; c0 < V; c0 += chunk) {
    const int cw = std::min(chunk, V - c0);
    const int nVt = (cw + kTile - 1) / kTile;
    {
      Prof pr("recompute_dz", stream);
      const dim3 grid(grouped_grid(nMt, nVt));
      if (bias)
        hipLaunchKernelGGL(recompute_dz_f32<true>, grid, dim3(512), 0, stream, H, M, D, W, bias, c0, cw, lam2, G, ldG,
                           g, remap, dZ, chunk);
      else
        hipLaunchKernelGGL(recompute_dz_f32<false>, grid, dim3(512), 0, stream, H, M, D, W, bias, c0, cw, lam2, G, ldG,
                           g, remap, dZ, chunk);
    }
    auto col_sums = [&](int maxs, float* sums) {
      const int mper = ((M + maxs - 1) / maxs + 3) / 4 * 4;
      const int slices = (M + mper - 1) / mper;
      Prof pr("db_colsum", stream);
      hipLaunchKernelGGL(db_colsum_f32, dim3(nVt, slices), dim3(256), 0, stream, dZ, M, chunk, mper, sums);
      hipLaunchKernelGGL(db_reduce_f32, dim3(nVt), dim3(256), 0, stream, sums, slices, chunk, cw, db + c0);
    };
    if (db && !plan.lean) col_sums(kDbSlicesF32, dbpart);
    if (dH || dW) {
      ProductsF32 p;
      p.dZ = dZ;
      p.M = M;
      p.chunk = chunk;
      p.W = W + static_cast<int64_t>(c0) * D;
      p.Hs = Hs;
      p.D = D;
      p.cw = cw;
      // a narrower later chunk spreads its columns over as many (shorter) slices
      p.slice = c0 == 0 ? slice : std::max(64, ((cw + nslices - 1) / nslices + 63) / 64 * 64);
      p.ns = (cw + p.slice - 1) / p.slice;
      p.nh = dH ? nMt * nDt * p.ns : 0;
      p.part = part;
      p.first = c0 == 0;
      p.nz = nz;
      p.mslice = mslice;
      p.nw = dW ? nVt * nDt * nz : 0;
      p.dW = dW ? dW + static_cast<int64_t>(c0) * D : nullptr;
      p.wpart = wpart;
      p.dw_first = mslice > p.slice;
      {
        Prof pr("products", stream);
        hipLaunchKernelGGL(products_f32, dim3(p.nh + p.nw), dim3(512), 0, stream, p);
      }
      if (dW && nz > 1) {
        const int64_t n = static_cast<int64_t>(cw) * D;
        Prof pr("dw_reduce", stream);
        hipLaunchKernelGGL(dw_reduce_f32, dim3(static_cast<unsigned>((n / 4 + 255) / 256)), dim3(256), 0, stream,
                           wpart, nz - 1, n, p.dW);
      }
    }
    // one slice; its sums go to the first row of dZ, dead after the products (a workgroup has read
    // its columns before it writes them)
    if (db && plan.lean) col_sums(1, dZ);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (dH && !in_place) return launch_dh_reduce(part, nslices, nH, nullptr, dH, stream);
  return hipGetLastError();
}

}  // namespace pctc
