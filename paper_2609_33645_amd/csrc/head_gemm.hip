// Vocabulary head of Pruned CTC: what the bf16 and fp32 products share (gfx950).
//
//  * lse_finalize: lambda from the normaliser's per-partition (max, sum) pairs, in double, and
//    S = Z[:, U] - lambda where the selected logits wait for it;
//  * greedy emission head: the best of the partitions and the CTC collapse;
//  * plan and chunk loop of the recomputed backward (Eq. vjp; Algorithm 1 backward loop; App. A,
//    Step 3), with the second stream's gates in the bf16 schedule.
// The products themselves are in head_gemm_bf16.hip and head_gemm_f32.hip.
#include <algorithm>

#include "head_tiles.h"
#include "pctc_internal.h"

namespace pctc {

// lambda_m from the per-partition (max, sum) pairs: 16 frames per block, 16 lanes per frame
// splitting the partitions; the maximum is exact, the rescaled sum is accumulated in double
// (each term's exponent taken in float on the exact difference to the maximum).  With Zd,
// also S[m][j] = float(Zd[m][j] - lambda_m) for j < *K (one rounding).
constexpr int kFinFrames = 16;
template <int PER>  // partitions per lane held in registers: P <= 16 PER
__global__ void __launch_bounds__(256)
lse_finalize_kernel(const float2* __restrict__ partials, int M, int P, double* __restrict__ lam,
                    float2* __restrict__ lam2, const double* __restrict__ Zd, const int32_t* __restrict__ Kdev,
                    float* __restrict__ S, int ldS, const float* __restrict__ g, float* __restrict__ rowscale,
                    int32_t* __restrict__ einv) {
  const int ph = threadIdx.x & 15;
  const int m = blockIdx.x * kFinFrames + (threadIdx.x >> 4);
  const bool live = m < M;
  // this lane's partitions ph, ph + 16, ... (at most PER), read once
  constexpr int kPer = PER;
  float2 q[kPer];
  float mx = -INFINITY;
  int nan = 0;
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int p = ph + 16 * i;
    q[i] = (live && p < P) ? partials[static_cast<int64_t>(p) * M + m] : make_float2(-INFINITY, 0.f);
    nan |= (q[i].x != q[i].x) | (q[i].y != q[i].y);
    mx = fmaxf(mx, q[i].x);
  }
#pragma unroll
  for (int o = 8; o >= 1; o >>= 1) {
    mx = fmaxf(mx, __shfl_xor(mx, o, 16));
    nan |= __shfl_xor(nan, o, 16);
  }
  double s = 0.0;
  if (mx != -INFINITY)
#pragma unroll
    for (int i = 0; i < kPer; ++i)
      if (q[i].x != -INFINITY)
        s += static_cast<double>(q[i].y) *
             static_cast<double>(fast_exp2(static_cast<float>(static_cast<double>(q[i].x) - mx) * kLog2e));
#pragma unroll
  for (int o = 8; o >= 1; o >>= 1) s += __shfl_xor(s, o, 16);
  if (!live) return;
  double l = static_cast<double>(mx) + log(s);
  if (mx == -INFINITY) l = -INFINITY;
  if (nan) l = __longlong_as_double(0x7ff8000000000000LL);
  if (ph == 0) {
    lam[m] = l;
    const double l2 = l * kLog2eD;
    const float hi = static_cast<float>(l2);
    lam2[m] = make_float2(hi, static_cast<float>(l2 - static_cast<double>(hi)));
    if (g) {
      if (!(l >= kEMin && l <= kEMax)) atomicOr(einv, 1);
      rowscale[m] = static_cast<float>(-static_cast<double>(g[m]) * exp(-l));
    }
  }
  if (Zd) {
    const int K = *Kdev;
    const double* zr = Zd + static_cast<int64_t>(m) * ldS;
    float* sr = S + static_cast<int64_t>(m) * ldS;
#pragma unroll 4
    for (int j = ph; j < K; j += 16) sr[j] = static_cast<float>(zr[j] - l);
  }
}

__global__ void lam2_kernel(const double* __restrict__ lam, int M, float2* __restrict__ lam2) {
  const int m = blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= M) return;
  const double l2 = lam[m] * kLog2eD;
  const float hi = static_cast<float>(l2);
  lam2[m] = make_float2(hi, static_cast<float>(l2 - static_cast<double>(hi)));
}

size_t lse_partial_bytes(int M, int D) {
  return align_up(static_cast<size_t>(lse_max_parts(D)) * M * sizeof(float2), 256);
}

hipError_t launch_lam2(const double* lam, int M, float2* lam2, hipStream_t stream) {
  if (M <= 0) return hipSuccess;
  Prof pr("lam2", stream);
  hipLaunchKernelGGL(lam2_kernel, dim3((M + 255) / 256), dim3(256), 0, stream, lam, M, lam2);
  return hipGetLastError();
}

hipError_t launch_lse(int dtype, const void* H, int M, int D, const void* W, const float* bias, int V,
                      float2* partials, double* lam, float2* lam2, hipStream_t stream, uint16_t* Ht, bool any_m) {
  if (M <= 0) return hipSuccess;
  int P = 0;
  hipError_t e;
  if (dtype == 1 && Ht) {
    const int Mp = (M + 63) / 64 * 64;
    e = launch_ht_build_bf16(static_cast<const uint16_t*>(H), M, D, nullptr, nullptr, Ht, Mp, stream);
    if (e == hipSuccess)
      e = launch_lse_partial_e_bf16(static_cast<const uint16_t*>(H), M, D, static_cast<const uint16_t*>(W), bias, V,
                                    partials, &P, nullptr, 0, 0, nullptr, stream, Ht, Mp, any_m);
  } else {
    e = launch_lse_partials(dtype, H, M, D, W, bias, V, partials, &P, stream, any_m);
  }
  if (e != hipSuccess) return e;
  return launch_lse_finalize(partials, M, P, lam, lam2, nullptr, nullptr, nullptr, 0, stream);
}

hipError_t launch_lse_partials(int dtype, const void* H, int M, int D, const void* W, const float* bias, int V,
                               float2* partials, int* P_out, hipStream_t stream, bool any_m) {
  *P_out = 0;
  if (M <= 0) return hipSuccess;
  if (dtype == 1)
    return launch_lse_partial_bf16(static_cast<const uint16_t*>(H), M, D, static_cast<const uint16_t*>(W), bias, V,
                                   partials, P_out, stream, any_m);
  return launch_lse_partial_f32(static_cast<const float*>(H), M, D, static_cast<const float*>(W), bias, V, partials,
                                P_out, stream);
}

hipError_t launch_lse_finalize(const float2* partials, int M, int P, double* lam, float2* lam2, const double* Zd,
                               const int32_t* K, float* S, int ldS, hipStream_t stream, const float* g,
                               float* rowscale, int32_t* einv) {
  if (M <= 0) return hipSuccess;
  if (P < 1 || P > kMaxLseParts) return hipErrorInvalidValue;
  Prof pr("lse_finalize", stream);
  const dim3 grid((M + kFinFrames - 1) / kFinFrames);
  if (P <= 256)
    hipLaunchKernelGGL(lse_finalize_kernel<16>, grid, dim3(256), 0, stream, partials, M, P, lam, lam2, Zd, K, S, ldS,
                       g, rowscale, einv);
  else
    hipLaunchKernelGGL(lse_finalize_kernel<kMaxLseParts / 16>, grid, dim3(256), 0, stream, partials, M, P, lam, lam2,
                       Zd, K, S, ldS, g, rowscale, einv);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Greedy emission head (framewise argmax over V, smallest class id on ties) and the CTC
// collapse of each utterance's argmax sequence (Sec. 3.1: merge repeats, drop blanks)
// ---------------------------------------------------------------------------------------

// ids[m]: the best of the partitions' (value, id) pairs, in partition order.
// 16 frames per block, 16 lanes per frame splitting the partitions; the merge (larger value,
// then smaller id) is order-independent, so the result does not depend on the split.
__global__ void __launch_bounds__(256)
amax_finalize_kernel(const float2* __restrict__ partials, int M, int P, int32_t* __restrict__ ids) {
  const int ph = threadIdx.x & 15;
  const int m = blockIdx.x * kFinFrames + (threadIdx.x >> 4);
  const bool live = m < M;
  float bv = -INFINITY;
  int bi = 0x7fffffff;
  if (live) {
#pragma unroll 4
    for (int p = ph; p < P; p += 16) {
      const float2 q = partials[static_cast<int64_t>(p) * M + m];
      amax_merge(bv, bi, q.x, __float_as_int(q.y));
    }
  }
#pragma unroll
  for (int o = 8; o >= 1; o >>= 1) {
    const float ov = __shfl_xor(bv, o, 16);
    const int oi = __shfl_xor(bi, o, 16);
    amax_merge(bv, bi, ov, oi);
  }
  if (live && ph == 0) ids[m] = (bi == 0x7fffffff) ? 0 : bi;
}

// One wavefront per utterance: frame m keeps its id when it is not blank and differs from
// the previous frame's (Sec. 3.1), and a ballot prefix count gives its output position.
__global__ void __launch_bounds__(256)
ctc_collapse_kernel(const int32_t* __restrict__ ids, const int32_t* __restrict__ toff, int N, int blank,
                    int32_t* __restrict__ tokens, int32_t* __restrict__ lengths) {
  const int lane = threadIdx.x & 63;
  const int n = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (n >= N) return;
  const int t0 = toff[n], t1 = toff[n + 1];
  int k = 0;
  for (int b = t0; b < t1; b += 64) {
    const int m = b + lane;
    const int c = (m < t1) ? ids[m] : blank;
    const int prev = (m > t0 && m < t1) ? ids[m - 1] : -1;
    const bool keep = c != blank && c != prev;
    const uint64_t mask = __ballot(keep);
    const int before = __popcll(mask & ((uint64_t{1} << lane) - 1));
    if (keep) tokens[t0 + k + before] = c;
    k += __popcll(mask);
  }
  if (lane == 0) lengths[n] = k;
}

hipError_t launch_greedy(int dtype, const void* H, int M, int D, const void* W, const float* bias, int V,
                         const int32_t* toff, int N, int blank, float2* partials, int32_t* ids, int32_t* tokens,
                         int32_t* lengths, hipStream_t stream, uint16_t* Ht) {
  if (M > 0) {
    int Pfin;
    hipError_t e;
    const int Mp = (M + 63) / 64 * 64;
    if (Ht) {
      e = launch_ht_build_bf16(static_cast<const uint16_t*>(H), M, D, nullptr, nullptr, Ht, Mp, stream);
      if (e != hipSuccess) return e;
    }
    e =
        dtype == 1 ? launch_amax_partial_bf16(static_cast<const uint16_t*>(H), M, D, static_cast<const uint16_t*>(W),
                                              bias, V, partials, &Pfin, stream, Ht, Mp)
                   : launch_amax_partial_f32(static_cast<const float*>(H), M, D, static_cast<const float*>(W), bias, V,
                                             partials, &Pfin, stream);
    if (e != hipSuccess) return e;
    Prof pr("amax_finalize", stream);
    hipLaunchKernelGGL(amax_finalize_kernel, dim3((M + kFinFrames - 1) / kFinFrames), dim3(256), 0, stream, partials,
                       M, Pfin, ids);
  }
  if (N > 0) {
    Prof pr("ctc_collapse", stream);
    hipLaunchKernelGGL(ctc_collapse_kernel, dim3((N + 3) / 4), dim3(256), 0, stream, ids, toff, N, blank, tokens,
                       lengths);
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Selected-class log-probabilities S
// ---------------------------------------------------------------------------------------

hipError_t launch_gather_s(int dtype, const void* H, int M, int D, const void* W, const float* bias,
                           const int32_t* u_ids, const int32_t* K, int K_max, const double* lam, float* S, int ldS,
                           hipStream_t stream, float* Gz) {
  if (M <= 0) return hipSuccess;
  if (dtype == 1)
    return launch_gather_s_bf16(static_cast<const uint16_t*>(H), M, D, static_cast<const uint16_t*>(W), bias, u_ids, K,
                                K_max, lam, S, ldS, stream, nullptr, Gz);
  return launch_gather_s_f32(static_cast<const float*>(H), M, D, static_cast<const float*>(W), bias, u_ids, K, K_max,
                             lam, S, ldS, stream, Gz);
}

// ---------------------------------------------------------------------------------------
// Backward
// ---------------------------------------------------------------------------------------

// dH = sum of the split-K partials (+ extra, which may be dH itself: each element is read
// before it is written by the same thread)
__global__ void dh_reduce_kernel(const float* __restrict__ part, int splits, int64_t n, const float* extra,
                                 float* dH) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float s = 0.f;
  for (int k = 0; k < splits; ++k) s += part[k * n + i];
  if (extra) s += extra[i];
  dH[i] = s;
}

hipError_t launch_dh_reduce(const float* part, int splits, int64_t n, const float* extra, float* dH,
                            hipStream_t stream) {
  Prof pr("dh_reduce", stream);
  hipLaunchKernelGGL(dh_reduce_kernel, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, stream, part,
                     splits, n, extra, dH);
  return hipGetLastError();
}

BwdPlan plan_bwd(int dtype, int M, int D, int V, int chunk, bool lean) {
  BwdPlan p{};
  p.lean = lean;
  int cap;  // columns the gradient buffer holds (sizes the workspace; independent of V)
  if (chunk > 0) {
    // a step never needs more columns than the vocabulary has (rounded up to whole tiles)
    const int vr = (V > 0 ? V + 255 : 256) / 256 * 256;
    p.chunk = cap = chunk < vr ? chunk : vr;
  } else {
    // default buffer: M x cap in the input dtype, about 512 MiB (at most 65536 columns);
    // V is then cut into as few equal chunks (multiples of 256 columns) as fit in it, so
    // that no launch works on a short remainder
    const size_t es0 = (dtype == 1) ? 2 : 4;
    size_t cmax = (static_cast<size_t>(512) << 20) / (es0 * static_cast<size_t>(M > 0 ? M : 1));
    if (cmax > 65536) cmax = 65536;
    cmax = cmax / 256 * 256;
    if (cmax < 256) cmax = 256;
    const size_t v = static_cast<size_t>(V > 0 ? V : 1);
    const size_t n = (v + cmax - 1) / cmax;
    size_t c = ((v + n - 1) / n + 255) / 256 * 256;
    if (c > cmax) c = cmax;
    if (dtype == 1 && D < kWideD) {
      // narrow bf16 heads: whole normaliser partitions, so that the first chunk's dZ rows can
      // come from the normaliser (lse_partial_e_bf16)
      size_t al = static_cast<size_t>(lse_part_columns_bf16(M, D, V));
      if (2048 % al == 0) al = 2048;  // whole partitions of every number of frames that has such runs
      size_t n2 = n, c2 = ((v + n2 - 1) / n2 + al - 1) / al * al;
      while (c2 > cmax && c2 > al) {
        ++n2;
        c2 = ((v + n2 - 1) / n2 + al - 1) / al * al;
      }
      if (c2 <= cmax) c = c2;
    }
    p.chunk = static_cast<int>(c);
    cap = static_cast<int>(cmax);
  }
  const size_t es = (dtype == 1) ? 2 : 4;
  p.splits = p.wsplits = 1;
  int room = 0;  // slices the partial buffer has room for, if more than p.splits
  if (dtype == 1) {
    const int tiles = ((M + 255) / 256) * ((D + 255) / 256);
    // k-slices of the dH product (one workgroup per CU): when the tiles alone make less than
    // two 256-workgroup waves, at most ~12,800 columns per slice (a launch of a few long
    // workgroups is exposed to any CU that is held up); then the fewest slices whose launch
    // fills its waves to at least 90%, else the fullest; at most 8
    const int maxs = p.chunk / 256 < 8 ? (p.chunk / 256 > 0 ? p.chunk / 256 : 1) : 8;
    int mins = (tiles < 512) ? (p.chunk + 12799) / 12800 : 1;
    if (mins > maxs) mins = maxs;
    if (mins < 1) mins = 1;
    int splits = mins;
    double best = -1.0;
    for (int sp = mins; sp <= maxs; ++sp) {
      const int wgs = tiles * sp;
      const double fill = static_cast<double>(wgs) / (256.0 * ((wgs + 255) / 256));
      if (fill > best + 1e-9) {
        best = fill;
        splits = sp;
      }
      if (fill >= 0.9) break;
    }
    if (!lean && M > 0 && tiles * maxs < 256 && p.chunk > 256 * maxs) {
      // few frames: eight slices leave most of the chip idle (331 frames, D = 512, chunks of
      // 60,000 columns: 16 or 32 workgroups, 160 us a launch).  The count whose launch is
      // shortest by 0.7 us a 32-deep k-tile and 4 us a workgroup, with every slice's partial sums
      // read and written at 3 TB/s; at most 32 slices and 32 MiB of them (there 32: 60 us).  The
      // buffer holds the most slices of any vocabulary: its size does not grow with V
      room = std::min(32, static_cast<int>(32.0 * 1024 * 1024 / (static_cast<double>(M) * D * sizeof(float))));
      room = std::min(room, cap / 256);
      double best_t = -1;
      for (int sp = maxs; sp <= 32 && sp * 256 <= p.chunk; ++sp) {
        const double bytes = static_cast<double>(sp) * M * D * sizeof(float);
        if (sp > maxs && bytes > 32.0 * 1024 * 1024) break;
        const int wgs = tiles * sp, len = ((p.chunk / sp + 63) / 64 * 64 + 31) / 32;
        const double t = ((wgs + 255) / 256) * (len * 0.7 + 4) + 2 * bytes / 3.0e6;
        if (best_t < 0 || t < best_t) {
          best_t = t;
          splits = sp;
        }
      }
    }
    p.splits = splits;
  } else if (!lean) {
    plan_products_f32(M, D, p.chunk < V ? p.chunk : V, &p.splits, &p.wsplits);
  }
  p.Mp = ((M + 63) / 64) * 64;
  p.dz_bytes = align_up(static_cast<size_t>(M) * cap * es, 256);
  p.ht_bytes = align_up(static_cast<size_t>(D) * p.Mp * es, 256);  // >= M x D (bf16 masked copy of H)
  // a single slice: the dH product accumulates in the caller's dH (no partial buffer)
  p.part_bytes =
      p.splits == 1 ? 0 : align_up(static_cast<size_t>(std::max(p.splits, room)) * M * D * sizeof(float), 256);
  p.lam2_bytes = align_up(static_cast<size_t>(M) * sizeof(float2), 256);
  // column sums of dZ for db, per 128-frame tile (bf16) or frame slice (fp32)
  p.dbpart_bytes =
      align_up((dtype == 1 ? static_cast<size_t>((M + 127) / 128) * cap
                           : (lean ? 0 : static_cast<size_t>(kDbSlicesF32) * p.chunk)) *
                   sizeof(float), 256);
  // narrow bf16 heads: the dense recompute reads its frames from Hs transposed (whole k-lines)
  p.hst_bytes = (dtype == 1 && D < kWideD && D % 128 == 0) ? align_up(static_cast<size_t>(D) * p.Mp * 2, 256) : 0;
  // fp32: dW's partial sums over the frame slices past the first
  p.wpart_bytes = align_up(static_cast<size_t>(p.wsplits - 1) * p.chunk * D * sizeof(float), 256);
  p.total = p.dz_bytes + p.ht_bytes + p.part_bytes + p.lam2_bytes + p.dbpart_bytes + p.hst_bytes + p.wpart_bytes;
  return p;
}

uint16_t* bwd_hs(void* scratch, const BwdPlan& plan) {
  return reinterpret_cast<uint16_t*>(static_cast<char*>(scratch) + plan.dz_bytes);
}

uint16_t* bwd_hst(void* scratch, const BwdPlan& plan) {
  if (plan.hst_bytes == 0) return nullptr;
  return reinterpret_cast<uint16_t*>(static_cast<char*>(scratch) + plan.dz_bytes + plan.ht_bytes + plan.part_bytes +
                                     plan.lam2_bytes + plan.dbpart_bytes);
}

static hipError_t head_bwd_bf16(const uint16_t* H, int M, int D, const uint16_t* W, const float* bias, int V,
                                const float2* lam2, const float* G, int ldG, const float* g, const int32_t* remap,
                                const float* S, int ldS, float* dH, float* dW, float* db, char* scratch,
                                const BwdPlan& plan, hipStream_t stream, const BwdSide* side) {
  uint16_t* dZ = reinterpret_cast<uint16_t*>(scratch);
  uint16_t* Hs = bwd_hs(scratch, plan);
  uint16_t* Hst = bwd_hst(scratch, plan);
  // a single split-K slice accumulates straight into dH: no partials and no reduction
  const bool in_place = plan.part_bytes == 0;
  float* part = in_place ? dH : reinterpret_cast<float*>(scratch + plan.dz_bytes + plan.ht_bytes);
  float* dbpart = reinterpret_cast<float*>(scratch + plan.dz_bytes + plan.ht_bytes + plan.part_bytes + plan.lam2_bytes);
  const int chunk = plan.chunk;
  const bool two = side && side->stream;
  hipError_t e;
  // Hs: H with the rows of excluded frames zeroed (read by the recompute and by dW), and its
  // transpose where the recompute reads that
  if (!(side && side->hs_built)) {
    e = Hst ? launch_ht_build_bf16(H, M, D, g, Hs, Hst, plan.Mp, stream) : launch_hs_build_bf16(H, M, D, g, Hs, stream);
    if (e != hipSuccess) return e;
  }
  const int slice = ((chunk / plan.splits + 63) / 64) * 64;
  // split-K slices any chunk fills: the first chunk (the widest) starts them all from zero
  const int nslices = (min(chunk, V) + slice - 1) / slice;
  const int64_t n = static_cast<int64_t>(M) * D;
  const float* dH_extra = side ? side->dH_extra : nullptr;
  int started = two ? 0 : 2;  // works of the second stream enqueued so far
  const int nwork = two ? side->nwork : 0;
  auto start_side = [&](int upto) -> hipError_t {  // enqueue works [started, upto)
    for (; started < upto && started < nwork; ++started) {
      hipError_t err;
      if (!side->eager) {
        if ((err = hipEventRecord(side->gate[started], stream)) != hipSuccess) return err;
        if ((err = hipStreamWaitEvent(side->stream, side->gate[started], 0)) != hipSuccess) return err;
      }
      if ((err = side->work[started].fn(side->work[started].ctx)) != hipSuccess) return err;
    }
    return hipSuccess;
  };
  bool front_pending = two && side->front.fn;
  auto start_front = [&]() -> hipError_t {
    if (!front_pending) return hipSuccess;
    front_pending = false;
    hipError_t err;
    if ((err = hipEventRecord(side->front_gate, stream)) != hipSuccess) return err;
    if ((err = hipStreamWaitEvent(side->stream, side->front_gate, 0)) != hipSuccess) return err;
    return side->front.fn(side->front.ctx);
  };
  if (two && side->eager && (e = start_side(1)) != hipSuccess) return e;
  auto due = [&](bool last, int done) { return last || (two && side->eager) ? nwork : done; };
  int ci = 0;  // chunk index
  for (int c0 = 0; c0 < V; c0 += chunk, ++ci) {
    const int cw = min(chunk, V - c0);
    const bool last = c0 + chunk >= V;
    const ChunkE* ce = (c0 == 0 && side) ? side->ce : nullptr;
    // the first chunk (the widest) sets the slices; a narrower later chunk spreads its columns
    // over as many slices (shorter ones), so that its dH launch keeps its workgroups
    const int sl = (c0 == 0) ? slice : std::max(64, ((cw + nslices - 1) / nslices + 63) / 64 * 64);
    if (last && two && dH) {
      // the last chunk's dW product runs beside the final dH reduction (second stream)
      e = launch_bwd_chunk_bf16(Hs, M, D, W, bias, c0, cw, lam2, G, ldG, g, remap, S, ldS, dZ, chunk, part, sl,
                                true, true, false, dW, db, dbpart, stream, nullptr, ce, Hst, plan.Mp);
      if (e != hipSuccess) return e;
      if ((e = start_front()) != hipSuccess) return e;
      if ((e = start_side(nwork)) != hipSuccess) return e;
      if ((e = hipEventRecord(side->dh_done, stream)) != hipSuccess) return e;
      if ((e = hipStreamWaitEvent(side->stream, side->dh_done, 0)) != hipSuccess) return e;
      if (in_place) {
        if (side->after_dh.fn && (e = side->after_dh.fn(side->after_dh.ctx)) != hipSuccess) return e;
      } else {
        if ((e = launch_dh_reduce(part, nslices, n, dH_extra, dH, side->stream)) != hipSuccess) return e;
      }
      if (dW) {
        // the union columns' dW_u rides in this launch's last round once their bf16 G is written
        const DwExtra* udw = side->udw.Z ? &side->udw : nullptr;
        if (udw && (e = hipStreamWaitEvent(stream, udw->ready, 0)) != hipSuccess) return e;
        e = launch_bwd_chunk_bf16(Hs, M, D, W, bias, c0, cw, lam2, G, ldG, g, remap, S, ldS, dZ, chunk, part, sl,
                                  false, false, true, dW, db, dbpart, stream, udw, ce, Hst, plan.Mp);
        if (e != hipSuccess) return e;
      }
    } else if (front_pending) {
      // the first chunk: the second stream's front starts beside its dW product, not its dH
      e = launch_bwd_chunk_bf16(Hs, M, D, W, bias, c0, cw, lam2, G, ldG, g, remap, S, ldS, dZ, chunk, part, sl,
                                true, dH != nullptr, false, dW, db, dbpart, stream, nullptr, ce, Hst, plan.Mp);
      if (e != hipSuccess) return e;
      if ((e = start_front()) != hipSuccess) return e;
      e = launch_bwd_chunk_bf16(Hs, M, D, W, bias, c0, cw, lam2, G, ldG, g, remap, S, ldS, dZ, chunk, part, sl,
                                false, false, dW != nullptr, dW, db, dbpart, stream, nullptr, ce, Hst, plan.Mp);
      if (e != hipSuccess) return e;
      if ((e = start_side(due(last, ci + 1))) != hipSuccess) return e;
    } else {
      e = launch_bwd_chunk_bf16(Hs, M, D, W, bias, c0, cw, lam2, G, ldG, g, remap, S, ldS, dZ, chunk, part, sl,
                                true, dH != nullptr, dW != nullptr, dW, db, dbpart, stream, nullptr, ce, Hst, plan.Mp);
      if (e != hipSuccess) return e;
      if ((e = start_side(due(last, ci + 1))) != hipSuccess) return e;
    }
  }
  if ((e = start_front()) != hipSuccess) return e;
  if ((e = start_side(nwork)) != hipSuccess) return e;
  if (two) {
    // the second stream's work (its union-column part and, with dH, the reduction) is done
    // before this call's work on the caller's stream is
    if ((e = hipEventRecord(side->reduced, side->stream)) != hipSuccess) return e;
    if ((e = hipStreamWaitEvent(stream, side->reduced, 0)) != hipSuccess) return e;
  } else if (dH && !in_place) {
    return launch_dh_reduce(part, nslices, n, dH_extra, dH, stream);
  }
  return hipGetLastError();
}

hipError_t launch_head_bwd(int dtype, const void* H, int M, int D, const void* W, const float* bias, int V,
                           const float2* lam2, const float* G, int ldG, const float* g, const int32_t* remap,
                           const float* S, int ldS, float* dH, float* dW, float* db, void* scratch,
                           const BwdPlan& plan, hipStream_t stream, const BwdSide* side) {
  if (M <= 0) {
    if (db) {
      hipError_t e = hipMemsetAsync(db, 0, static_cast<size_t>(V) * sizeof(float), stream);
      if (e != hipSuccess) return e;
    }
    if (dW) return hipMemsetAsync(dW, 0, static_cast<size_t>(V) * D * sizeof(float), stream);
    return hipSuccess;
  }
  char* sc = static_cast<char*>(scratch);
  if (dtype == 1)
    return head_bwd_bf16(static_cast<const uint16_t*>(H), M, D, static_cast<const uint16_t*>(W), bias, V, lam2, G, ldG,
                         g, remap, S, ldS, dH, dW, db, sc, plan, stream, side);
  return head_bwd_f32(static_cast<const float*>(H), M, D, static_cast<const float*>(W), bias, V, lam2, G, ldG, g,
                           remap, dH, dW, db, sc, plan, stream);
}

}  // namespace pctc
