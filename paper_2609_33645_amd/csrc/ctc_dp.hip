// Alignment lattice of Pruned CTC (Sec. 3.1 CTC; Sec. 3.3 and App. B.3 beam pruning;
// Algorithm 1 lattice, total scores, zeroing of nonfinite losses and dL/dS).
//
// The lattice of utterance n is the extended label sequence l' = (blank, y1, blank, ...,
// yU, blank) of S' = 2U+1 states per frame; it is implicit (states are indices).  Arcs:
// start -> (0, s) for s < 2; (t-1, s) -> (t, s); (t-1, s-1) -> (t, s); (t-1, s-2) -> (t, s)
// when l'_s is a label different from l'_{s-2}; (T-1, s) -> end for s >= S'-2.
//
// Kernels:
//   dp_prep      per utterance: alignability T >= U + r (App. B.1), duplicate-label links,
//                frame -> utterance map.
//   dp_pass      one or four wavefronts per (utterance, direction); lane l of them holds states
//                [lQ, lQ+Q).  Viterbi (max-plus, float) or total score (log-sum-exp,
//                accumulated in double), renormalised every frame by the wave maximum
//                with the running offsets kept in double.
//   dp_mask      beam rule: keep an arc iff the best complete alignment through it scores
//                at least (best alignment) - beam - slack.
//   dp_occupancy gamma_t(s) = alpha_t(s) beta_t(s) / P, summed per selected class into
//                G = dL/dS = -gamma (Algorithm 1 output), and g = row sums of G.
//   dp_tail      sum of finite per-utterance losses (Algorithm 1, zero nonfinite), outputs.
#include <type_traits>

#include "pctc_internal.h"
#include "prunedctc.h"

namespace pctc {

constexpr float kNeg = -1.0e30f;  // "impossible" score; absorbs finite additions
constexpr int kMaxQ = 8;          // most states per lane of a lattice pass
constexpr int kMaxStates = 256 * kMaxQ;
static_assert(2 * PCTC_MAX_TARGET + 1 <= kMaxStates, "the longest target fits a lattice pass");
// arc flags of a pass without a mask: every arc kept
constexpr int kAllArcs = 0x0f;
// bytes the mask region extends past its last cell: a pass reads each lane's flags as whole
// aligned words, up to (kMaxQ + 5) / 4 + 1 words from the lane's first cell
constexpr int kMaskPad = 64;
static_assert(4 * ((kMaxQ + 5) / 4 + 1) <= kMaskPad, "mask padding covers a lane's word reads");

DpPlan plan_dp(int N, const int32_t* T, const int32_t* U, float beam) {
  DpPlan p{};
  p.N = N;
  p.pruned = (beam == beam) && beam >= 0.f && beam < INFINITY;
  int64_t M = 0, Y = 0, L = 0;
  int Smax = 1;
  for (int n = 0; n < N; ++n) {
    M += T[n];
    Y += U[n];
    L += static_cast<int64_t>(T[n]) * (2 * U[n] + 1);
    Smax = U[n] * 2 + 1 > Smax ? U[n] * 2 + 1 : Smax;
  }
  p.M = static_cast<int>(M);
  p.Y = static_cast<int>(Y);
  p.Smax = Smax;
  p.lattice = L;
  size_t o = 0;
  auto take = [&](size_t bytes) {
    size_t at = o;
    o += align_up(bytes > 0 ? bytes : 1, 256);
    return at;
  };
  p.off_toff = take((N + 1) * sizeof(int32_t));
  p.off_yoff = take((N + 1) * sizeof(int32_t));
  p.off_soff = take((N + 1) * sizeof(int64_t));
  p.off_frame_utt = take(M * sizeof(int32_t));
  p.off_dup_next = take(Y * sizeof(int32_t));
  p.off_dup_first = take(Y * sizeof(int32_t));
  p.off_logp = take(N * sizeof(double));
  p.off_status = take(N * sizeof(int32_t));
  p.off_tab_fa = take(L * sizeof(float));
  p.off_tab_fb = take(L * sizeof(float));
  p.off_sc_fa = take(M * sizeof(double));
  p.off_sc_fb = take(M * sizeof(double));
  p.off_dummy = take(static_cast<size_t>(2 * N) * kMaxStates * sizeof(float));
  if (p.pruned) {
    p.off_tab_va = take(L * sizeof(float));
    p.off_tab_vb = take(L * sizeof(float));
    p.off_sc_va = take(M * sizeof(double));
    p.off_sc_vb = take(M * sizeof(double));
    p.off_vbest = take(N * sizeof(double));
    p.off_mask = take(L * sizeof(uint8_t) + kMaskPad);  // the passes read whole words past a row's end
  }
  p.total = o;
  return p;
}

// ---------------------------------------------------------------------------------------

// Per-utterance set-up, and the inclusion forecast (g_pred, pred; null: none).  For an included
// utterance every frame's occupancies sum to one (each retained alignment occupies exactly one
// state per frame), so g_m = -w_n there and 0 on excluded utterances.  Before the lattice runs an
// utterance is forecast included when its targets fit its frames (T_n >= U_n + repeats) and
// w_n != 0; the lattice's statuses are checked against it afterwards (dp_tail).
__global__ void __launch_bounds__(256)
dp_prep_kernel(const int32_t* __restrict__ toff, const int32_t* __restrict__ yoff,
                               const int32_t* __restrict__ y_rel, int ncols, int32_t* __restrict__ status,
                               int32_t* __restrict__ dup_next, int32_t* __restrict__ dup_first,
                               int32_t* __restrict__ frame_utt, double* __restrict__ loss_n, float* __restrict__ g,
                               const float* __restrict__ weight, float* __restrict__ g_pred,
                               int32_t* __restrict__ pred) {
  const int n = blockIdx.x;
  const int t0 = toff[n], T = toff[n + 1] - t0;
  const int y0 = yoff[n], U = yoff[n + 1] - y0;
  // the utterance's targets in LDS (every entry point rejects U > PCTC_MAX_TARGET before
  // any launch): the duplicate search below compares every pair
  __shared__ __attribute__((aligned(16))) int y[PCTC_MAX_TARGET + 4];
  __shared__ int reps, badlab;
  if (threadIdx.x == 0) {
    reps = 0;
    badlab = 0;
  }
  for (int i = threadIdx.x; i < U; i += blockDim.x) y[i] = y_rel[y0 + i];
  if (threadIdx.x < 4) y[U + threadIdx.x] = -2;  // up to the next multiple of four: equal to no target
  __syncthreads();
  int myreps = 0;
  for (int i = threadIdx.x; i < U; i += blockDim.x) {
    const int yi = y[i];
    if (yi < 1 || yi >= ncols) badlab = 1;  // not a label column of S
    if (i > 0 && yi == y[i - 1]) ++myreps;
    // every target four at a time, the same ones in every lane, without a branch (a scan that
    // stops at its match waits for each read: 400 targets 76 us against 30)
    int nx = 0x7fffffff, first = 1;
#pragma unroll 4
    for (int j = 0; j < U; j += 4) {
      const int4 v = *reinterpret_cast<const int4*>(y + j);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const bool eq = (k == 0 ? v.x : k == 1 ? v.y : k == 2 ? v.z : v.w) == yi;
        first = (eq && j + k < i) ? 0 : first;
        nx = min(nx, (eq && j + k > i) ? j + k : 0x7fffffff);
      }
    }
    dup_next[y0 + i] = nx == 0x7fffffff ? -1 : nx;
    dup_first[y0 + i] = first;
  }
  if (myreps) atomicAdd(&reps, myreps);
  for (int t = threadIdx.x; t < T; t += blockDim.x) {
    frame_utt[t0 + t] = n;
    if (g) g[t0 + t] = 0.f;  // excluded utterances' frames stay zero
  }
  __syncthreads();
  if (g_pred) {
    const float w = weight ? weight[n] : 1.f;
    const bool inc = T >= U + reps && w != 0.f;
    for (int t = threadIdx.x; t < T; t += blockDim.x) g_pred[t0 + t] = inc ? -w : 0.f;
    if (threadIdx.x == 0) pred[n] = inc ? 1 : 0;
  }
  if (threadIdx.x == 0) {
    // 3: a relabelled target is not a label column; the lattice is not evaluated
    status[n] = badlab ? 3 : ((T >= U + reps) ? 0 : 1);
    loss_n[n] = 0.0;
  }
}

// ---------------------------------------------------------------------------------------

// Cross-lane moves with DPP (VALU, no LDS round trip).
// wave_shr:1 -> lane l receives lane l-1 (lane 0 keeps `old`); wave_shl:1 -> lane l
// receives lane l+1 (lane 63 keeps `old`).
__device__ __forceinline__ int dpp_up_i(int x, int old) { return __builtin_amdgcn_update_dpp(old, x, 0x138, 0xf, 0xf, false); }
__device__ __forceinline__ int dpp_dn_i(int x, int old) { return __builtin_amdgcn_update_dpp(old, x, 0x130, 0xf, 0xf, false); }
__device__ __forceinline__ float lane_up(float x) { return __int_as_float(dpp_up_i(__float_as_int(x), __float_as_int(kNeg))); }
__device__ __forceinline__ float lane_down(float x) { return __int_as_float(dpp_dn_i(__float_as_int(x), __float_as_int(kNeg))); }
__device__ __forceinline__ double lane_up(double x) {
  const long long b = __double_as_longlong(x);
  const long long nb = __double_as_longlong(static_cast<double>(kNeg));
  const int lo = dpp_up_i(static_cast<int>(b), static_cast<int>(nb));
  const int hi = dpp_up_i(static_cast<int>(b >> 32), static_cast<int>(nb >> 32));
  return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<unsigned int>(lo));
}
__device__ __forceinline__ double lane_down(double x) {
  const long long b = __double_as_longlong(x);
  const long long nb = __double_as_longlong(static_cast<double>(kNeg));
  const int lo = dpp_dn_i(static_cast<int>(b), static_cast<int>(nb));
  const int hi = dpp_dn_i(static_cast<int>(b >> 32), static_cast<int>(nb >> 32));
  return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<unsigned int>(lo));
}
__device__ __forceinline__ int lane_down_i(int x) { return dpp_dn_i(x, 0); }

// Maximum over the wavefront: DPP reductions within each row of 16 lanes, then the four
// row results read as scalars.
template <int CTRL>
__device__ __forceinline__ float dpp_max_step(float v) {
  return fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), CTRL, 0xf, 0xf,
                                                               false)));
}
__device__ __forceinline__ float wave_max_dpp(float x) {
  x = dpp_max_step<0xB1>(x);   // quad_perm [1,0,3,2]
  x = dpp_max_step<0x4E>(x);   // quad_perm [2,3,0,1]
  x = dpp_max_step<0x141>(x);  // row_half_mirror
  x = dpp_max_step<0x140>(x);  // row_mirror
  const float a = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 0));
  const float b = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 16));
  const float c = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 32));
  const float d = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 48));
  return fmaxf(fmaxf(a, b), fmaxf(c, d));
}

// Max (Viterbi) or log-sum-exp (natural log) of three scores.  The log-sum-exp keeps
// the scores in Acc (double for the total-score pass) and evaluates exp/log in float on
// differences from the maximum, where float is accurate.
template <bool VIT, typename Acc>
__device__ __forceinline__ Acc comb3(Acc a, Acc b, Acc c) {
  const Acc m = fmax(fmax(a, b), c);
  if constexpr (VIT) {
    return m;
  } else {
    const float s = fast_exp2(static_cast<float>(a - m) * kLog2e) + fast_exp2(static_cast<float>(b - m) * kLog2e) +
                    fast_exp2(static_cast<float>(c - m) * kLog2e);
    return m + static_cast<Acc>(fast_log2(s) * kLn2);
  }
}

// Frames of emissions (and arc flags) loaded ahead of the recursion: the frames in flight are
// bounded by the wave's memory counter (63 instructions: per frame Q emission loads (and two of
// the next wavefront's states), Q table stores and the offset store, and with a mask up to
// (Q + 5) / 4 + 1 flag-word loads) and by registers.
template <int Q>
constexpr int prefetch_depth() {
  return Q <= 2 ? 8 : (Q <= 4 ? 6 : (Q <= 6 ? 4 : 3));
}
// The discarded-mass pass loads one flag byte per state.
template <int Q>
constexpr int prefetch_depth_bytes() {
  return Q <= 3 ? 8 : (Q <= 4 ? 6 : (Q <= 6 ? 4 : 3));
}

// What the wavefronts of one lattice pass exchange each frame (two sets, used in turn, so that one
// barrier per frame is enough): their maxima and, of every lane (a write under a lane condition
// would be a branch in the frame loop), the states next to the neighbour's.
template <int NWV, typename Acc, int NV>
struct Exchange {
  float mx[2][NWV];
  Acc v[2][64 * NWV][NV];
};
// LDS writes of every wavefront of the workgroup done and visible; loads and stores to global
// memory stay in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// NWV wavefronts per (utterance, direction), natural-log units.  VIT: Viterbi (max-plus)
// accumulated in float; otherwise the total score (log-sum-exp) accumulated in double,
// so the per-frame additions do not round at the magnitude of the path's score.
// Tables hold scores minus a per-frame offset (rounded to float once); the offsets are
// kept per frame in double.  Emissions and arc flags for the next PF frames are held in
// a register ring so that the gathers are issued well before they are needed.
// kPassWaves wavefronts per workgroup: with NWV = 1 independent ones (no barriers), so that the
// few wavefronts of this latency-bound stage occupy few compute units; with NWV = 4 the four
// of one unit, which exchange their maxima and edge states through LDS, one barrier per frame.
// A frame's time grows with the states per lane (1500 frames, 801 states, beside the products:
// 3.07 us a frame with 13 states per lane of one wavefront, 0.75 with 4 per lane of four), the
// exchange costs about 0.1 us; so targets of more than 128 states take four wavefronts.  The
// maxima are exact and every state's arithmetic is the same, so the tables do not depend on NWV.
constexpr int kPassWaves = 4;

template <int Q, bool VIT, bool MASK, int NWV>
__global__ void __launch_bounds__(64 * kPassWaves)
dp_pass_kernel(const float* __restrict__ S, int ldS, const int32_t* __restrict__ toff,
               const int32_t* __restrict__ yoff, const int64_t* __restrict__ soff, const int32_t* __restrict__ y_rel,
               int32_t* __restrict__ status, const uint8_t* __restrict__ mask, float* __restrict__ tab_f,
               float* __restrict__ tab_b, double* __restrict__ sc_f, double* __restrict__ sc_b,
               double* __restrict__ total_out, double* __restrict__ loss_n, int N, float* __restrict__ dummy) {
  using Acc = typename std::conditional<VIT, float, double>::type;
  constexpr int PF = prefetch_depth<Q>();
  constexpr bool MULTI = NWV > 1;
  static_assert(NWV == 1 || NWV == kPassWaves, "a unit is one wavefront or the workgroup");
  __shared__ Exchange<MULTI ? NWV : 1, Acc, 2> xch;
  const int unit = MULTI ? blockIdx.x : blockIdx.x * kPassWaves + (threadIdx.x >> 6);  // (utterance, direction)
  if (unit >= 2 * N) return;
  const int n = unit >> 1;
  const int dir = unit & 1;
  const int wl = threadIdx.x & 63;                        // lane of the wavefront
  const int wv = MULTI ? static_cast<int>(threadIdx.x >> 6) : 0;
  const int lane = MULTI ? static_cast<int>(threadIdx.x) : wl;  // lane of the unit
  // The forward unit of this launch sets status[n] = 2 where the total is not finite, perhaps before
  // this unit has begun: one read decides for all wavefronts of a unit, which meet at barriers below
  // (tables of such an utterance are not used, so either value will do).
  if constexpr (MULTI) {
    __shared__ int excluded;
    if (threadIdx.x == 0) excluded = status[n];
    __syncthreads();
    if (excluded != 0) return;
  } else if (status[n] != 0) {
    return;
  }
  const int t0 = toff[n], T = toff[n + 1] - t0;
  const int y0 = yoff[n], U = yoff[n + 1] - y0;
  const int Sp = 2 * U + 1;
  const int64_t base = soff[n];
  const int* y = y_rel + y0;
  const Acc neg = kNeg;

  // The blank column index is an opaque per-lane zero: with a literal 0 the compiler would
  // turn the (uniform) blank emission load into a scalar load and wait for it on the spot,
  // defeating the prefetch ring.
  int zero_v;
  asm volatile("v_mov_b32 %0, 0" : "=v"(zero_v));
  // HX: the next wavefront's first two states, which the backward pass's last lane needs too
  constexpr int HX = MULTI ? 2 : 0;
  int col[Q + HX];
  bool valid[Q + HX], skip_in[Q], skip_out[Q], fin[Q];
#pragma unroll
  for (int q = 0; q < Q + HX; ++q) {
    const int s = lane * Q + q;
    valid[q] = s < Sp && (q < Q || (wl == 63 && dir == 1));
    col[q] = (valid[q] && (s & 1)) ? y[(s - 1) >> 1] : zero_v;
  }
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int s = lane * Q + q;
    skip_in[q] = valid[q] && (s & 1) && s >= 3 && y[(s - 1) >> 1] != y[(s - 3) >> 1];
    const int s2 = s + 2;
    skip_out[q] = (s2 < Sp) && (s2 & 1) && y[(s2 - 1) >> 1] != y[(s2 - 3) >> 1];
    fin[q] = valid[q] && s >= Sp - 2;
  }
  // One frame of emissions and arc flags for this lane's states.  No load, store or prefetch
  // of the frame loop sits under a branch (addresses are clamped in bounds, lanes past the
  // last state store to this wave's dummy row): a branch around memory operations makes the
  // compiler wait for every outstanding load at the join, which would serialise the ring.
  float* const drow = dummy + static_cast<int64_t>(unit) * kMaxStates + lane * Q;
  // The flags stay as the words that hold them until the frame is used (decode): decoded where
  // they are fetched, the loop waited for its own loads before it went round.
  constexpr int NWD = MASK ? (Q + HX + 3) / 4 + 1 : 1;
  auto flag_at = [&](int t) { return base + static_cast<int64_t>(t) * Sp + min(lane * Q, Sp - 1); };
  auto fetch = [&](int t, float (&e)[Q + HX], uint32_t (&w)[NWD]) {
    const float* row = S + static_cast<int64_t>(t0 + t) * ldS;
#pragma unroll
    for (int q = 0; q < Q + HX; ++q) e[q] = row[col[q]];  // invalid states read the blank column (a valid address)
    if constexpr (MASK) {
      // this lane's Q flag bytes (from its first cell, clamped into the row) as the NWD aligned
      // words that cover them: a few loads instead of Q byte loads (the bytes past the row's end,
      // read only for cells past the last state, are not used; the region starts 256-byte aligned,
      // so the offset's low bits are the address's)
      const uint32_t* wp = reinterpret_cast<const uint32_t*>(mask + (flag_at(t) & ~static_cast<int64_t>(3)));
#pragma unroll
      for (int j = 0; j < NWD; ++j) w[j] = wp[j];
    }
  };
  auto decode = [&](int t, const uint32_t (&w)[NWD], int (&mk)[Q + HX]) {
    const uint32_t sh = MASK ? static_cast<uint32_t>(flag_at(t) & 3) : 0u;
#pragma unroll
    for (int q = 0; q < Q + HX; ++q) {
      if constexpr (MASK) {
        const uint32_t d = __builtin_amdgcn_alignbyte(w[(q >> 2) + 1], w[q >> 2], sh);
        mk[q] = valid[q] ? static_cast<int>((d >> (8 * (q & 3))) & 0xffu) : 0;
      } else {
        mk[q] = valid[q] ? kAllArcs : 0;
      }
    }
  };
  int par = 0;  // exchange set in use
  // The edge states a wavefront hands to its neighbour, and (mx) its maximum of a frame, into the
  // exchange set in use; read are, forward, lane 63's last state and the one before (Q = 1: lane
  // 62's), backward lane 0's first two (Q = 1: lane 1's second).
  auto publish = [&](const Acc (&v)[Q], float mx) {
    xch.mx[par][wv] = mx;  // the same value in every lane
    xch.v[par][MULTI ? lane : 0][0] = dir == 0 ? v[Q - 1] : v[0];
    if (Q >= 2) xch.v[par][MULTI ? lane : 0][1] = dir == 0 ? v[Q >= 2 ? Q - 2 : 0] : v[Q >= 2 ? 1 : 0];
  };
  // The other side, after a barrier: the maximum of all wavefronts' mx, and h0, h1: the previous
  // wavefront's last two states (forward: h0 the last) or the next one's first two (backward: h0
  // the first); kNeg at the ends.
  auto collect = [&](Acc& h0, Acc& h1) {
    float mx = kNeg;
#pragma unroll
    for (int w = 0; w < NWV; ++w) mx = fmaxf(mx, xch.mx[par][MULTI ? w : 0]);
    const int nb = dir == 0 ? wv - 1 : wv + 1;
    const bool have = nb >= 0 && nb < NWV;
    const int at = MULTI ? (have ? nb : 0) * 64 + (dir == 0 ? 63 : 0) : 0;
    const Acc x0 = xch.v[par][at][0];
    const Acc x1 = Q >= 2 ? xch.v[par][at][Q >= 2 ? 1 : 0] : xch.v[par][MULTI ? (dir == 0 ? at - 1 : at + 1) : 0][0];
    h0 = have ? x0 : neg;
    h1 = have ? x1 : neg;
    par ^= 1;
    return mx;
  };
  auto lane_max = [&](const Acc (&v)[Q]) {
    float mx = kNeg;
#pragma unroll
    for (int q = 0; q < Q; ++q) mx = fmaxf(mx, static_cast<float>(v[q]));
    return wave_max_dpp(mx);
  };
  // Table row of a frame: the scores below mx, mx's running total beside them.
  auto store_row = [&](const Acc (&v)[Q], double off, float* tab, double* sc, int t) {
    float* trow = tab + base + static_cast<int64_t>(t) * Sp + lane * Q;
#pragma unroll
    for (int q = 0; q < Q; ++q) *(valid[q] ? trow + q : drow + q) = static_cast<float>(v[q]);
    sc[t0 + t] = off;  // uniform: every lane stores the same value
  };
  // A frame's end.  Viterbi (float: the scores must not round at the magnitude of the whole path)
  // and one wavefront: renormalised by its maximum and stored.  Total score over four wavefronts:
  // the recursion goes on with the scores as they are (double holds any path's score to 1e-10 and
  // better) and only the stored row is taken below the frame's maximum, so the maximum
  // (conversions, DPP steps, four scalar reads) is not between a frame and the next: a frame's
  // maxima travel with the next frame's edge states and its row is stored one frame late (vp, mwp;
  // first: none is pending).  1000 frames, 401 / 801 states: 542 -> 459, 809 -> 701 us; one
  // wavefront is bound by its instructions, about 170 a frame, not by this chain.
  Acc vp[Q];
  float mwp = kNeg;
  auto settle = [&](float mx) { return (mx <= kNeg * 0.5f || mx != mx) ? 0.f : mx; };  // all impossible (or NaN): as is
  auto store_below = [&](const Acc (&v)[Q], float mx, float* tab, double* sc, int t) {
    Acc r[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) r[q] = (v[q] <= Acc(kNeg * 0.5f)) ? Acc(kNeg) : v[q] - Acc(mx);
    store_row(r, static_cast<double>(mx), tab, sc, t);
  };
  auto finish = [&](auto first, Acc (&v)[Q], Acc& h0, Acc& h1, double& off, float* tab, double* sc, int t) {
    if constexpr (VIT || !MULTI) {
      float mx = lane_max(v);
      if constexpr (MULTI) {
        publish(v, mx);
        lds_barrier();
        mx = collect(h0, h1);
      }
      mx = settle(mx);
#pragma unroll
      for (int q = 0; q < Q; ++q) v[q] = (v[q] <= Acc(kNeg * 0.5f)) ? Acc(kNeg) : v[q] - Acc(mx);
      if constexpr (MULTI) {
        h0 = (h0 <= Acc(kNeg * 0.5f)) ? Acc(kNeg) : h0 - Acc(mx);
        h1 = (h1 <= Acc(kNeg * 0.5f)) ? Acc(kNeg) : h1 - Acc(mx);
      }
      off += static_cast<double>(mx);
      store_row(v, off, tab, sc, t);
      return;
    }
    // impossible states stay at kNeg (an emission of -inf would make the next frame's differences
    // NaN; NaN scores stay NaN)
#pragma unroll
    for (int q = 0; q < Q; ++q) v[q] = (v[q] <= Acc(kNeg * 0.5f)) ? Acc(kNeg) : v[q];
    if constexpr (!VIT && MULTI) {
      publish(v, mwp);
      lds_barrier();
      const float mx = settle(collect(h0, h1));
      if constexpr (!decltype(first)::value) store_below(vp, mx, tab, sc, dir == 0 ? t - 1 : t + 1);
#pragma unroll
      for (int q = 0; q < Q; ++q) vp[q] = v[q];
      mwp = lane_max(v);
    }
  };
  // The row still pending after the last frame.
  auto flush = [&](float* tab, double* sc, int t) {
    if constexpr (!VIT && MULTI) {
      Acc x0, x1;
      publish(vp, mwp);
      lds_barrier();
      store_below(vp, settle(collect(x0, x1)), tab, sc, t);
    }
  };
  constexpr std::true_type kFirst{};
  constexpr std::false_type kLater{};

  float ring_e[PF][Q + HX];
  uint32_t ring_m[PF][NWD];
  Acc h0 = neg, h1 = neg;
  if (dir == 0) {
    // ---------------- forward ----------------
    Acc a[Q];
    {
      float e[Q + HX];
      uint32_t w[NWD];
      int mk[Q + HX];
      fetch(0, e, w);
      decode(0, w, mk);
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const int s = lane * Q + q;
        a[q] = (valid[q] && s < 2 && (mk[q] & 1)) ? static_cast<Acc>(e[q]) : neg;
      }
    }
#pragma unroll
    for (int k = 0; k < PF; ++k) fetch(min(1 + k, T - 1), ring_e[k], ring_m[k]);
    double off = 0.0;
    finish(kFirst, a, h0, h1, off, tab_f, sc_f, 0);
    // frame t from ring slot k, which then prefetches frame t + PF (clamped to the last)
    auto fstep = [&](int t, float (&re)[Q + HX], uint32_t (&rm)[NWD]) {
          float e[Q];
          int mk[Q + HX];
#pragma unroll
          for (int q = 0; q < Q; ++q) e[q] = re[q];
          decode(t, rm, mk);
          fetch(min(t + PF, T - 1), re, rm);
          // lane 0 of a wavefront takes the previous wavefront's last states
          Acc up1 = lane_up(a[Q - 1]);
          if (MULTI && wl == 0) up1 = h0;
          Acc up2 = (Q >= 2) ? lane_up(a[Q >= 2 ? Q - 2 : 0]) : lane_up(up1);
          if (MULTI && wl == 0) up2 = h1;
          Acc na[Q];
#pragma unroll
          for (int q = 0; q < Q; ++q) {
            const Acc p0 = a[q];
            const Acc p1 = (q >= 1) ? a[q >= 1 ? q - 1 : 0] : up1;
            const Acc p2 = (q >= 2) ? a[q >= 2 ? q - 2 : 0] : (q == 1 ? up1 : up2);
            // a mask has bits of arcs that exist only; without one every arc that exists is kept.
            // States past the last keep none, and e + kNeg is as impossible as kNeg: the result is
            // not selected by valid[q] (the compiler makes a branch of that, with a wait for the
            // loads in flight at its end: 331 frames, 111 states 220 us against 148)
            const Acc c0 = (MASK ? (mk[q] & 1) != 0 : valid[q]) ? p0 : neg;
            const Acc c1 = (MASK ? (mk[q] & 2) != 0 : valid[q]) ? p1 : neg;
            const Acc c2 = (MASK ? (mk[q] & 4) != 0 : skip_in[q]) ? p2 : neg;
            na[q] = static_cast<Acc>(e[q]) + comb3<VIT, Acc>(c0, c1, c2);
          }
#pragma unroll
          for (int q = 0; q < Q; ++q) a[q] = na[q];
          finish(kLater, a, h0, h1, off, tab_f, sc_f, t);
    };
    int tb = 1;
    for (; tb + PF <= T; tb += PF) {
#pragma unroll
      for (int k = 0; k < PF; ++k) fstep(tb + k, ring_e[k], ring_m[k]);
    }
#pragma unroll
    for (int k = 0; k < PF; ++k)
      if (tb + k < T) fstep(tb + k, ring_e[k], ring_m[k]);
    flush(tab_f, sc_f, T - 1);
    // total over final states (with final-arc flags)
    int fk[Q + HX];
    {
      float e[Q + HX];
      uint32_t w[NWD];
      fetch(T - 1, e, w);
      decode(T - 1, w, fk);
    }
    float fm = kNeg;
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if (fin[q] && (fk[q] & 8)) fm = fmaxf(fm, static_cast<float>(a[q]));
    fm = wave_max_dpp(fm);
    if constexpr (MULTI) {
      if (wl == 0) xch.mx[par][wv] = fm;
      lds_barrier();
#pragma unroll
      for (int w = 0; w < NWV; ++w) fm = fmaxf(fm, xch.mx[par][w]);
      par ^= 1;
    }
    double total;
    if (VIT) {
      total = off + static_cast<double>(fm);
    } else {
      float s = 0.f;
#pragma unroll
      for (int q = 0; q < Q; ++q)
        if (fin[q] && (fk[q] & 8)) s += fast_exp2(static_cast<float>(a[q] - Acc(fm)) * kLog2e);
      s = wave_sum(s);
      if constexpr (MULTI) {
        if (wl == 0) xch.mx[par][wv] = s;
        lds_barrier();
        s = 0.f;
#pragma unroll
        for (int w = 0; w < NWV; ++w) s += xch.mx[par][w];
      }
      total = off + static_cast<double>(fm) + static_cast<double>(fast_log2(s) * kLn2);
      if (fm <= kNeg * 0.5f) total = -INFINITY;
    }
    if (lane == 0) {
      total_out[n] = total;
      if (!VIT) {
        const double L = -total;
        const bool finite = (L == L) && L < INFINITY && L > -INFINITY;
        loss_n[n] = finite ? L : 0.0;
        if (!finite) status[n] = 2;
      }
    }
  } else {
    // ---------------- backward ----------------
    Acc b[Q];
    {
      float e[Q + HX];
      uint32_t w[NWD];
      int mk[Q + HX];
      fetch(T - 1, e, w);
      decode(T - 1, w, mk);
#pragma unroll
      for (int q = 0; q < Q; ++q) b[q] = (fin[q] && (mk[q] & 8)) ? Acc(0) : neg;
    }
    // ring slot k holds frame (T-1) - k - ... : frames T-1, T-2, ... are consumed as t+1
#pragma unroll
    for (int k = 0; k < PF; ++k) fetch(max(T - 1 - k, 0), ring_e[k], ring_m[k]);
    double off = 0.0;
    finish(kFirst, b, h0, h1, off, tab_b, sc_b, T - 1);
    // frame t uses the emissions and arcs of frame t + 1 from ring slot k, which then
    // prefetches frame t + 1 - PF (clamped to the first)
    auto bstep = [&](int t, float (&re)[Q + HX], uint32_t (&rm)[NWD]) {
          float e[Q + HX];
          int mk[Q + HX];
#pragma unroll
          for (int q = 0; q < Q + HX; ++q) e[q] = re[q];
          decode(t + 1, rm, mk);
          fetch(max(t + 1 - PF, 0), re, rm);
          Acc nb[Q];
#pragma unroll
          for (int q = 0; q < Q; ++q) nb[q] = valid[q] ? static_cast<Acc>(e[q]) + b[q] : neg;
          // the last lane of a wavefront takes the next wavefront's first states
          Acc dn0 = lane_down(nb[0]);
          int mdn0 = lane_down_i(mk[0]);
          if (MULTI && wl == 63) {
            dn0 = valid[Q + HX - 2] ? static_cast<Acc>(e[Q + HX - 2]) + h0 : neg;
            mdn0 = mk[Q + HX - 2];
          }
          Acc dn1 = (Q >= 2) ? lane_down(nb[Q >= 2 ? 1 : 0]) : lane_down(dn0);
          int mdn1 = (Q >= 2) ? lane_down_i(mk[Q >= 2 ? 1 : 0]) : lane_down_i(mdn0);
          if (MULTI && wl == 63) {
            dn1 = valid[Q + HX - 1] ? static_cast<Acc>(e[Q + HX - 1]) + h1 : neg;
            mdn1 = mk[Q + HX - 1];
          }
          Acc nbb[Q];
#pragma unroll
          for (int q = 0; q < Q; ++q) {
            const Acc s0 = nb[q];
            const Acc s1 = (q + 1 < Q) ? nb[q + 1 < Q ? q + 1 : 0] : dn0;
            const Acc s2 = (q + 2 < Q) ? nb[q + 2 < Q ? q + 2 : 0] : (q + 1 < Q ? dn0 : dn1);
            const int m0 = mk[q];
            const int m1 = (q + 1 < Q) ? mk[q + 1 < Q ? q + 1 : 0] : mdn0;
            const int m2 = (q + 2 < Q) ? mk[q + 2 < Q ? q + 2 : 0] : (q + 1 < Q ? mdn0 : mdn1);
            const Acc c0 = (MASK ? (m0 & 1) != 0 : valid[q]) ? s0 : neg;
            const Acc c1 = (MASK ? (m1 & 2) != 0 : valid[q]) ? s1 : neg;
            const Acc c2 = (MASK ? (m2 & 4) != 0 : skip_out[q]) ? s2 : neg;
            nbb[q] = comb3<VIT, Acc>(c0, c1, c2);
          }
#pragma unroll
          for (int q = 0; q < Q; ++q) b[q] = nbb[q];
          finish(kLater, b, h0, h1, off, tab_b, sc_b, t);
    };
    int tb = T - 2;
    for (; tb - (PF - 1) >= 0; tb -= PF) {
#pragma unroll
      for (int k = 0; k < PF; ++k) bstep(tb - k, ring_e[k], ring_m[k]);
    }
#pragma unroll
    for (int k = 0; k < PF; ++k)
      if (tb - k >= 0) bstep(tb - k, ring_e[k], ring_m[k]);
    flush(tab_b, sc_b, 0);
  }
}

// ---------------------------------------------------------------------------------------

// The beams of one mask launch and where their masks go.
constexpr int kMaskBeams = 9;
struct MaskBeams {
  float beam[kMaskBeams];
  uint8_t* mask[kMaskBeams];
};

// One workgroup per frame.  Margin of each arc into (t, s):
//   alpha^(t-1, s') + E_t(s) + beta^(t, s) - (best - beam - slack) >= 0 keeps it.
// The arcs' scores are read once for all beams of the launch.
template <int NB>
__global__ void dp_mask_kernel(const float* __restrict__ S, int ldS, const int32_t* __restrict__ toff,
                               const int32_t* __restrict__ yoff, const int64_t* __restrict__ soff,
                               const int32_t* __restrict__ y_rel, const int32_t* __restrict__ frame_utt,
                               const int32_t* __restrict__ status, const float* __restrict__ va,
                               const float* __restrict__ vb, const double* __restrict__ sva,
                               const double* __restrict__ svb, const double* __restrict__ vbest, int nb,
                               MaskBeams beams, float slack) {
  const int m = blockIdx.x;
  const int n = frame_utt[m];
  if (status[n] != 0) return;
  const int t0 = toff[n], T = toff[n + 1] - t0;
  const int t = m - t0;
  const int y0 = yoff[n], U = yoff[n + 1] - y0;
  const int Sp = 2 * U + 1;
  const int64_t base = soff[n];
  const int* y = y_rel + y0;
  const double best = vbest[n], sv_b = svb[m];
  const double sv_prev = (t > 0) ? sva[m - 1] : 0.0, sv_last = (t == T - 1) ? sva[m] : 0.0;
  const float* row = S + static_cast<int64_t>(m) * ldS;
  for (int s = threadIdx.x; s < Sp; s += blockDim.x) {
    const int c = (s & 1) ? y[(s - 1) >> 1] : 0;
    const float e = row[c];
    const float bt = vb[base + static_cast<int64_t>(t) * Sp + s];
    const bool skip = (s & 1) && s >= 3 && y[(s - 1) >> 1] != y[(s - 3) >> 1];
    const bool last = t == T - 1 && s >= Sp - 2;
    const float at = last ? va[base + static_cast<int64_t>(t) * Sp + s] : 0.f;
    const float* ap = va + base + static_cast<int64_t>(t > 0 ? t - 1 : 0) * Sp;
    const float a0 = ap[s], a1 = (s >= 1) ? ap[s - 1] : 0.f, a2 = skip ? ap[s - 2] : 0.f;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      if (NB > 1 && b >= nb) break;
      const double thr = best - static_cast<double>(beams.beam[b]) - static_cast<double>(slack);
      uint8_t bits = 0;
      if (t == 0) {
        if (s < 2 && e + bt + static_cast<float>(sv_b - thr) >= 0.f) bits |= 1;
      } else {
        // frame offsets: alpha^ at t-1 and beta^ at t
        const float through = e + bt + static_cast<float>(sv_prev + sv_b - thr);
        if (a0 + through >= 0.f) bits |= 1;
        if (s >= 1 && a1 + through >= 0.f) bits |= 2;
        if (skip && a2 + through >= 0.f) bits |= 4;
      }
      if (last && at + static_cast<float>(sv_last - thr) >= 0.f) bits |= 8;
      beams.mask[b][base + static_cast<int64_t>(t) * Sp + s] = bits;
    }
  }
}

// ---------------------------------------------------------------------------------------

constexpr int kOccFrames = 4;  // frames per block, one wavefront each

// One wavefront per frame (no block barriers: a wavefront's LDS accesses are performed in
// program order, and the fence keeps the compiler from reordering them).
__global__ void __launch_bounds__(64 * kOccFrames)
dp_occupancy_kernel(const int32_t* __restrict__ toff, const int32_t* __restrict__ yoff,
                    const int64_t* __restrict__ soff, const int32_t* __restrict__ y_rel,
                    const int32_t* __restrict__ frame_utt, const int32_t* __restrict__ status,
                    const int32_t* __restrict__ dup_next, const int32_t* __restrict__ dup_first,
                    const float* __restrict__ fa, const float* __restrict__ fb, const double* __restrict__ sfa,
                    const double* __restrict__ sfb, const double* __restrict__ logp,
                    const float* __restrict__ weight, float* __restrict__ G, int ldG, float* __restrict__ g, int M,
                    int Smax) {
  extern __shared__ float gam_all[];  // [kOccFrames][Smax]
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int m = blockIdx.x * kOccFrames + wv;
  if (m >= M) return;
  const int n = frame_utt[m];
  if (status[n] != 0) return;  // G row stays zero, g stays zero
  float* gam = gam_all + wv * Smax;
  const int t0 = toff[n];
  const int t = m - t0;
  const int y0 = yoff[n], U = yoff[n + 1] - y0;
  const int Sp = 2 * U + 1;
  const int64_t rowb = soff[n] + static_cast<int64_t>(t) * Sp;
  const float off = static_cast<float>(sfa[m] + sfb[m] - logp[n]);
  const float w = weight ? weight[n] : 1.f;  // loss weight of the utterance: G = -w gamma
  for (int s = lane; s < Sp; s += 64) {
    const float x = fa[rowb + s] + fb[rowb + s] + off;
    gam[s] = fast_exp2(x * kLog2e);
  }
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
  // blank column: sum over even states (fixed order per lane, then across lanes)
  float bsum = 0.f;
  for (int s = 2 * lane; s < Sp; s += 128) bsum += gam[s];
  // label columns: the first occurrence of each label sums its states in target order
  float lsum = 0.f;
  for (int i = lane; i < U; i += 64) {
    if (!dup_first[y0 + i]) continue;
    float acc = gam[2 * i + 1];
    int j = dup_next[y0 + i];
    while (j >= 0) {
      acc += gam[2 * j + 1];
      j = dup_next[y0 + j];
    }
    G[static_cast<int64_t>(m) * ldG + y_rel[y0 + i]] = -w * acc;
    lsum += acc;
  }
  const float blank_total = wave_sum(bsum);
  const float label_total = wave_sum(lsum);
  if (lane == 0) {
    G[static_cast<int64_t>(m) * ldG + 0] = -w * blank_total;
    g[m] = -w * (blank_total + label_total);
  }
}

// The lattice's end in one launch: loss = sum over included utterances of w_n L_n (w_n = 1 without
// weights), in order; the caller's copies of the losses and statuses; and, in the two-stream
// schedule, flag = 1 if an utterance's inclusion (status 0 and w_n != 0) differs from the forecast
// (dp_prep).  The values pass through LDS: one thread adding 160 losses from memory took 20 us.
constexpr int kTailThreads = 256;
__global__ void __launch_bounds__(kTailThreads)
dp_tail_kernel(int N, const double* __restrict__ loss_n, const int32_t* __restrict__ status,
               const float* __restrict__ weight, const int32_t* __restrict__ pred, double* __restrict__ loss,
               double* __restrict__ loss_out, int32_t* __restrict__ status_out, int32_t* __restrict__ flag) {
  __shared__ double term[kTailThreads];
  double sum = 0.0;
  int bad = 0;
  for (int b = 0; b < N; b += kTailThreads) {
    const int n = b + threadIdx.x;
    double x = 0.0;
    if (n < N) {
      const double l = loss_n[n];
      const int st = status[n];
      const float w = weight ? weight[n] : 1.f;
      if (st == 0) x = static_cast<double>(w) * l;
      if (loss_out) loss_out[n] = l;
      if (status_out) status_out[n] = st;
      if (pred) bad |= ((st == 0 && w != 0.f) ? 1 : 0) != pred[n];
    }
    term[threadIdx.x] = x;
    __syncthreads();
    if (threadIdx.x == 0)
      for (int i = 0; i < min(kTailThreads, N - b); ++i) sum += term[i];
    __syncthreads();
  }
  bad = __syncthreads_or(bad);
  if (threadIdx.x == 0) {
    *loss = sum;
    if (pred) *flag = bad;
  }
}

hipError_t launch_dp_tail(int N, const double* loss_n, const int32_t* status, const float* weight, const int32_t* pred,
                          double* loss, double* loss_out, int32_t* status_out, int32_t* flag, hipStream_t stream) {
  Prof pr("dp_tail", stream);
  hipLaunchKernelGGL(dp_tail_kernel, dim3(1), dim3(kTailThreads), 0, stream, N, loss_n, status, weight, pred, loss,
                     loss_out, status_out, flag);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------

// LDS that keeps a workgroup off a compute unit where a dW product's runs (128 of 160 KB).  Beside it
// a pass of up to 96 registers would fit, and both run slower than on units of their own, which
// dW's launches of narrow heads leave free: 30 x 200 frames, D = 256, V = 150,000 (152 workgroups),
// the Viterbi pass 167 us and dW 179, apart 61 and 141.  For the passes whose registers do not see
// to it themselves (one wavefront of one state a lane has always run beside dW).
constexpr size_t kOffDw = 32768 + 512;
constexpr bool reserve_lds(int Q, int nwv, bool vit, bool mask) {
  return nwv == 1 ? Q == 2 && vit : Q == 1 && (vit || !mask);
}

template <bool VIT>
static hipError_t launch_pass(int Q, int nwv, int N, hipStream_t stream, const float* S, int ldS, const int32_t* toff,
                              const int32_t* yoff, const int64_t* soff, const int32_t* y_rel, int32_t* status,
                              const uint8_t* mask, float* tf, float* tb, double* sf, double* sb, double* total,
                              double* loss_n, float* dummy) {
#define PCTC_PASS(QQ, NWV)                                                                                        \
  if (Q == QQ && nwv == NWV) {                                                                                    \
    const dim3 grid(NWV > 1 ? 2 * N : (2 * N + kPassWaves - 1) / kPassWaves);                                     \
    const size_t lds = reserve_lds(QQ, NWV, VIT, mask != nullptr) ? kOffDw : 0;                                   \
    if (mask)                                                                                                     \
      hipLaunchKernelGGL((dp_pass_kernel<QQ, VIT, !VIT, NWV>), grid, dim3(64 * kPassWaves), lds, stream, S, ldS,   \
                         toff, yoff, soff, y_rel, status, mask, tf, tb, sf, sb, total, loss_n, N, dummy);         \
    else                                                                                                          \
      hipLaunchKernelGGL((dp_pass_kernel<QQ, VIT, false, NWV>), grid, dim3(64 * kPassWaves), lds, stream, S, ldS,  \
                         toff, yoff, soff, y_rel, status, nullptr, tf, tb, sf, sb, total, loss_n, N, dummy);      \
    return hipGetLastError();                                                                                     \
  }
  PCTC_PASS(1, 1)
  PCTC_PASS(2, 1)
  PCTC_PASS(1, 4)
  PCTC_PASS(2, 4)
  PCTC_PASS(3, 4)
  PCTC_PASS(4, 4)
  PCTC_PASS(6, 4)
  PCTC_PASS(8, 4)
#undef PCTC_PASS
  return hipErrorInvalidValue;
}

// States per lane and wavefronts per utterance and direction (or beam) for lattices of up to
// Smax states per frame.
static void pick_lanes(int Smax, int* Q, int* nwv) {
  *nwv = Smax <= 128 ? 1 : 4;
  const int need = (Smax + 64 * *nwv - 1) / (64 * *nwv);
  *Q = need <= 4 ? need : (need <= 6 ? 6 : kMaxQ);
}

hipError_t launch_ctc_dp(const DpPlan& plan, const int32_t* T, const int32_t* U, const float* S, int ldS,
                         const int32_t* y_rel, float beam, const float* weight, double* loss_n, int32_t* status,
                         float* G, float* g, uint8_t* keep_mask_out, void* scratch, int K_max, hipStream_t stream,
                         int phase, bool g_zeroed, float* g_pred, int32_t* pred) {
  const int N = plan.N;
  const bool prep = phase == kDpAll || phase == kDpPrep;
  const bool vit = phase == kDpAll || phase == kDpVit;
  const bool back = phase == kDpAll || phase == kDpBack;
  char* sc = static_cast<char*>(scratch);
  int32_t* toff = reinterpret_cast<int32_t*>(sc + plan.off_toff);
  int32_t* yoff = reinterpret_cast<int32_t*>(sc + plan.off_yoff);
  int64_t* soff = reinterpret_cast<int64_t*>(sc + plan.off_soff);
  int32_t* frame_utt = reinterpret_cast<int32_t*>(sc + plan.off_frame_utt);
  int32_t* dnext = reinterpret_cast<int32_t*>(sc + plan.off_dup_next);
  int32_t* dfirst = reinterpret_cast<int32_t*>(sc + plan.off_dup_first);
  double* logp = reinterpret_cast<double*>(sc + plan.off_logp);
  float* tfa = reinterpret_cast<float*>(sc + plan.off_tab_fa);
  float* dummy = reinterpret_cast<float*>(sc + plan.off_dummy);
  float* tfb = reinterpret_cast<float*>(sc + plan.off_tab_fb);
  double* sfa = reinterpret_cast<double*>(sc + plan.off_sc_fa);
  double* sfb = reinterpret_cast<double*>(sc + plan.off_sc_fb);
  hipError_t e;
  int Q, nwv;
  pick_lanes(plan.Smax, &Q, &nwv);
  uint8_t* mask = plan.pruned ? reinterpret_cast<uint8_t*>(sc + plan.off_mask) : nullptr;
  if (prep) {
    // G starts at zero: excluded utterances and unused columns stay zero
    if (plan.M > 0 && !g_zeroed) {
      e = hipMemsetAsync(G, 0, static_cast<size_t>(plan.M) * ldS * sizeof(float), stream);
      if (e != hipSuccess) return e;
    }
    if (N == 0) return hipSuccess;
    Prof pr("dp_prep", stream);
    hipLaunchKernelGGL(dp_prep_kernel, dim3(N), dim3(256), 0, stream, toff, yoff, y_rel, K_max, status, dnext, dfirst,
                       frame_utt, loss_n, g, weight, g_pred, pred);
  }
  if (N == 0) return hipGetLastError();
  if (vit) {
    if (plan.pruned) {
      float* tva = reinterpret_cast<float*>(sc + plan.off_tab_va);
      float* tvb = reinterpret_cast<float*>(sc + plan.off_tab_vb);
      double* sva = reinterpret_cast<double*>(sc + plan.off_sc_va);
      double* svb = reinterpret_cast<double*>(sc + plan.off_sc_vb);
      double* vbest = reinterpret_cast<double*>(sc + plan.off_vbest);
      {
        Prof pr("dp_viterbi", stream);
        e = launch_pass<true>(Q, nwv, N, stream, S, ldS, toff, yoff, soff, y_rel, status, nullptr, tva, tvb, sva,
                              svb, vbest, loss_n, dummy);
        if (e != hipSuccess) return e;
      }
      if (plan.M > 0) {
        Prof pr("dp_mask", stream);
        MaskBeams one{};
        one.beam[0] = beam;
        one.mask[0] = mask;
        hipLaunchKernelGGL(dp_mask_kernel<1>, dim3(plan.M), dim3(256), 0, stream, S, ldS, toff, yoff, soff, y_rel,
                           frame_utt, status, tva, tvb, sva, svb, vbest, 1, one, kKeepSlack);
      }
    }
  }
  if (!back || N == 0) return hipGetLastError();
  {
    Prof pr("dp_alpha_beta", stream);
    e = launch_pass<false>(Q, nwv, N, stream, S, ldS, toff, yoff, soff, y_rel, status, mask, tfa, tfb, sfa, sfb,
                           logp, loss_n, dummy);
    if (e != hipSuccess) return e;
  }
  if (plan.M > 0) {
    Prof pr("dp_occupancy", stream);
    hipLaunchKernelGGL(dp_occupancy_kernel, dim3((plan.M + kOccFrames - 1) / kOccFrames), dim3(64 * kOccFrames),
                       static_cast<size_t>(kOccFrames) * plan.Smax * sizeof(float), stream, toff, yoff, soff, y_rel,
                       frame_utt, status, dnext, dfirst, tfa, tfb, sfa, sfb, logp, weight, G, ldS, g, plan.M,
                       plan.Smax);
  }
  if (keep_mask_out && mask && plan.lattice > 0) {
    e = hipMemcpyAsync(keep_mask_out, mask, plan.lattice, hipMemcpyDeviceToDevice, stream);
    if (e != hipSuccess) return e;
  }
  (void)T;
  (void)U;
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Discarded posterior mass (App. B.3): delta_n = 1 - (sum over retained alignments) /
// (sum over all valid alignments), both of prod_t p_{pi_t}(t) on the same scores.  One wavefront
// (four above 128 states) per utterance and beam runs the two forward recursions in lockstep in
// linear space and double precision, with one shared scale per frame (a power of two near the full
// recursion's maximum), so the per-frame scaling is exact and cancels in the ratio.  Bound by
// the latency of its T sequential frames, so all beams run at once (the full recursion again
// for each of them): nine beams, 16 utterances of up to 375 frames, 9 x 180 us one after
// another, 104 us together.  The emission factor exp(S), the same for both recursions, is a float
// significand with its own power of two in double: it loses precision for S below -708 and is zero
// below -745, so an utterance with a frame whose every reachable state scores less gets NaN, as
// those that are not alignable do.
// ---------------------------------------------------------------------------------------

// Linear-space neighbour move: lane l receives lane l-1, lane 0 receives 0 (no state).
__device__ __forceinline__ double lane_up_d(double x) {
  const long long b = __double_as_longlong(x);
  const int lo = dpp_up_i(static_cast<int>(b), 0);
  const int hi = dpp_up_i(static_cast<int>(b >> 32), 0);
  return __longlong_as_double((static_cast<long long>(hi) << 32) | static_cast<unsigned int>(lo));
}

// Maximum over the wavefront of the high words of non-negative doubles (they order as the
// doubles do, to 20 significand bits).
template <int CTRL>
__device__ __forceinline__ int dpp_max_step_i(int v) {
  return max(v, __builtin_amdgcn_update_dpp(v, v, CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ int wave_max_i(int x) {
  x = dpp_max_step_i<0xB1>(x);   // quad_perm [1,0,3,2]
  x = dpp_max_step_i<0x4E>(x);   // quad_perm [2,3,0,1]
  x = dpp_max_step_i<0x141>(x);  // row_half_mirror
  x = dpp_max_step_i<0x140>(x);  // row_mirror
  return max(max(__builtin_amdgcn_readlane(x, 0), __builtin_amdgcn_readlane(x, 16)),
             max(__builtin_amdgcn_readlane(x, 32), __builtin_amdgcn_readlane(x, 48)));
}
__device__ __forceinline__ double wave_sum_d(double x) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}

template <int Q, int NWV>
__global__ void __launch_bounds__(64 * NWV)
dp_discarded_kernel(const float* __restrict__ S, int ldS, const int32_t* __restrict__ toff,
                    const int32_t* __restrict__ yoff, const int64_t* __restrict__ soff,
                    const int32_t* __restrict__ y_rel, const int32_t* __restrict__ status,
                    MaskBeams beams, double* __restrict__ delta_all) {
  const int n = blockIdx.x;
  constexpr bool MULTI = NWV > 1;
  __shared__ struct {
    int hi[2][NWV];
    double v[2][MULTI ? 64 * NWV : 1][4];  // each lane's last two states: full, retained, full, retained
  } xch;
  const int lane = threadIdx.x;  // of the utterance's wavefronts
  const int wl = lane & 63, wv = MULTI ? lane >> 6 : 0;
  const uint8_t* const mask = beams.mask[blockIdx.y];
  double* const delta = delta_all + static_cast<int64_t>(blockIdx.y) * gridDim.x;
  if (status[n] != 0) {
    if (lane == 0) delta[n] = __longlong_as_double(0x7ff8000000000000LL);
    return;
  }
  const int t0 = toff[n], T = toff[n + 1] - t0;
  const int y0 = yoff[n], U = yoff[n + 1] - y0;
  const int Sp = 2 * U + 1;
  const int64_t base = soff[n];
  const int* y = y_rel + y0;
  int col[Q];
  bool valid[Q], skip_in[Q], fin[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int s = lane * Q + q;
    valid[q] = s < Sp;
    col[q] = (valid[q] && (s & 1)) ? y[(s - 1) >> 1] : 0;
    skip_in[q] = valid[q] && (s & 1) && s >= 3 && y[(s - 1) >> 1] != y[(s - 3) >> 1];
    fin[q] = valid[q] && s >= Sp - 2;
  }
  double af[Q], ap[Q];  // full and retained forward sums, scaled per frame
  double edge[4];       // the previous wavefront's last two states, scaled alike
  int par = 0;          // exchange set in use
  // Emissions and arc flags of the next PF frames are held in a register ring; the loop has
  // only loads and no branch around them (clamped addresses), so each frame waits only for
  // its own ring slot.
  constexpr int PF = prefetch_depth_bytes<Q>();
  float ring_e[PF][Q];
  int ring_m[PF][Q];
  auto load_frame = [&](int t, float (&e)[Q], int (&mk)[Q]) {
    const float* row = S + static_cast<int64_t>(t0 + t) * ldS;
    const uint8_t* mrow = mask + base + static_cast<int64_t>(t) * Sp;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const float v = row[col[q]];  // invalid states read the blank column (a valid address)
      e[q] = valid[q] ? v : -INFINITY;
      const int m = static_cast<int>(mrow[min(lane * Q + q, Sp - 1)]);
      mk[q] = valid[q] ? m : 0;
    }
  };
  // exp(e) in double over the whole range without a per-frame shift: 2^x = 2^i 2^(x - i),
  // i = floor(x), the fraction's power in float and the integer one exact
  auto emit = [&](const float (&e)[Q], double (&pe)[Q]) {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const float x = e[q] * kLog2e;
      const float fi = fminf(fmaxf(floorf(x), -2000.f), 2000.f);
      pe[q] = (valid[q] && x > -INFINITY) ? ldexp(static_cast<double>(fast_exp2(x - fi)), static_cast<int>(fi)) : 0.0;
    }
  };
  // any positive scale serves (both sums take the same one): the power of two that brings the
  // wave's largest value to [1, 2) (its exponent kept within a normal number's), which is exact
  // and needs only the high words, one register and four DPP steps instead of shuffled doubles
  auto rescale = [&](double (&nf)[Q], double (&np)[Q]) {
    int hi = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) hi = max(hi, static_cast<int>(__double_as_longlong(nf[q]) >> 32));
    hi = wave_max_i(hi);
    if constexpr (MULTI) {
      xch.v[par][lane][0] = nf[Q - 1];
      xch.v[par][lane][1] = np[Q - 1];
      if (Q >= 2) {
        xch.v[par][lane][2] = nf[Q >= 2 ? Q - 2 : 0];
        xch.v[par][lane][3] = np[Q >= 2 ? Q - 2 : 0];
      }
      xch.hi[par][wv] = hi;
      lds_barrier();
#pragma unroll
      for (int w = 0; w < NWV; ++w) hi = max(hi, xch.hi[par][w]);
    }
    const int ex = min(max(2046 - (hi >> 20), 1), 2046);
    const double inv = __longlong_as_double(static_cast<long long>(ex) << 52);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      af[q] = nf[q] * inv;
      ap[q] = np[q] * inv;
    }
    if constexpr (MULTI) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {  // (Q = 1: the state before the last is lane 62's last)
        const int at = (wv > 0 ? wv - 1 : 0) * 64 + 63;
        const double x = (Q == 1 && i >= 2) ? xch.v[par][at - 1][i - 2] : xch.v[par][at][i];
        edge[i] = (wv > 0) ? x * inv : 0.0;
      }
      par ^= 1;
    }
  };
  {  // frame 0: the start arcs
    float e[Q];
    int mk[Q];
    load_frame(0, e, mk);
#pragma unroll
    for (int k = 0; k < PF; ++k) load_frame(min(1 + k, T - 1), ring_e[k], ring_m[k]);
    double pe[Q], nf[Q], np[Q];
    emit(e, pe);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int s = lane * Q + q;
      nf[q] = (valid[q] && s < 2) ? pe[q] : 0.0;
      np[q] = (valid[q] && s < 2 && (mk[q] & 1)) ? pe[q] : 0.0;
    }
    rescale(nf, np);
  }
  // frame t from ring slot k, which then prefetches frame t + PF (clamped to the last)
  auto step = [&](int t, float (&re)[Q], int (&rm)[Q]) {
    float e[Q];
    int mk[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      e[q] = re[q];
      mk[q] = rm[q];
    }
    load_frame(min(t + PF, T - 1), re, rm);
    double pe[Q], nf[Q], np[Q];
    emit(e, pe);
    double uf1 = lane_up_d(af[Q - 1]), up1 = lane_up_d(ap[Q - 1]);
    if (MULTI && wl == 0) {
      uf1 = edge[0];
      up1 = edge[1];
    }
    double uf2 = (Q >= 2) ? lane_up_d(af[Q >= 2 ? Q - 2 : 0]) : lane_up_d(uf1);
    double up2 = (Q >= 2) ? lane_up_d(ap[Q >= 2 ? Q - 2 : 0]) : lane_up_d(up1);
    if (MULTI && wl == 0) {
      uf2 = edge[2];
      up2 = edge[3];
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const double f0 = af[q], p0 = ap[q];
      const double f1 = (q >= 1) ? af[q >= 1 ? q - 1 : 0] : uf1;
      const double p1 = (q >= 1) ? ap[q >= 1 ? q - 1 : 0] : up1;
      const double f2 = (q >= 2) ? af[q >= 2 ? q - 2 : 0] : (q == 1 ? uf1 : uf2);
      const double p2 = (q >= 2) ? ap[q >= 2 ? q - 2 : 0] : (q == 1 ? up1 : up2);
      nf[q] = valid[q] ? pe[q] * (f0 + f1 + (skip_in[q] ? f2 : 0.0)) : 0.0;
      np[q] = valid[q] ? pe[q] * (((mk[q] & 1) ? p0 : 0.0) + ((mk[q] & 2) ? p1 : 0.0) +
                                  ((skip_in[q] && (mk[q] & 4)) ? p2 : 0.0))
                       : 0.0;
    }
    rescale(nf, np);
  };
  int tb = 1;
  for (; tb + PF <= T; tb += PF) {
#pragma unroll
    for (int k = 0; k < PF; ++k) step(tb + k, ring_e[k], ring_m[k]);
  }
#pragma unroll
  for (int k = 0; k < PF; ++k)
    if (tb + k < T) step(tb + k, ring_e[k], ring_m[k]);
  double sf = 0.0, sp = 0.0;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    if (!fin[q]) continue;
    const int mk = static_cast<int>(mask[base + static_cast<int64_t>(T - 1) * Sp + lane * Q + q]);
    sf += af[q];
    if (mk & 8) sp += ap[q];
  }
  sf = wave_sum_d(sf);
  sp = wave_sum_d(sp);
  if constexpr (MULTI) {
    if (wl == 0) {
      xch.v[par][wv][0] = sf;  // any slot of this set
      xch.v[par][wv][1] = sp;
    }
    lds_barrier();
    sf = sp = 0.0;
#pragma unroll
    for (int w = 0; w < NWV; ++w) {
      sf += xch.v[par][w][0];
      sp += xch.v[par][w][1];
    }
  }
  if (lane == 0) delta[n] = (sf > 0.0) ? 1.0 - sp / sf : __longlong_as_double(0x7ff8000000000000LL);
}

static hipError_t launch_discarded(int Q, int nwv, int N, int nb, hipStream_t stream, const float* S, int ldS,
                                   const int32_t* toff, const int32_t* yoff, const int64_t* soff,
                                   const int32_t* y_rel, const int32_t* status, const MaskBeams& beams,
                                   double* delta) {
#define PCTC_DISC(QQ, NWV)                                                                                     \
  if (Q == QQ && nwv == NWV) {                                                                                 \
    hipLaunchKernelGGL((dp_discarded_kernel<QQ, NWV>), dim3(N, nb), dim3(64 * NWV), 0, stream, S, ldS, toff, yoff, \
                       soff, y_rel, status, beams, delta);                                                     \
    return hipGetLastError();                                                                                  \
  }
  PCTC_DISC(1, 1)
  PCTC_DISC(2, 1)
  PCTC_DISC(1, 4)
  PCTC_DISC(2, 4)
  PCTC_DISC(3, 4)
  PCTC_DISC(4, 4)
  PCTC_DISC(6, 4)
  PCTC_DISC(8, 4)
#undef PCTC_DISC
  return hipErrorInvalidValue;
}

hipError_t launch_discarded_mass(const DpPlan& plan, const float* S, int ldS, const int32_t* y_rel, const float* beams,
                                 int nbeams, double* delta, void* scratch, int K_max, hipStream_t stream) {
  const int N = plan.N;
  if (N == 0 || nbeams == 0) return hipSuccess;
  if (!plan.pruned) return hipErrorInvalidValue;
  char* sc = static_cast<char*>(scratch);
  int32_t* toff = reinterpret_cast<int32_t*>(sc + plan.off_toff);
  int32_t* yoff = reinterpret_cast<int32_t*>(sc + plan.off_yoff);
  int64_t* soff = reinterpret_cast<int64_t*>(sc + plan.off_soff);
  int32_t* frame_utt = reinterpret_cast<int32_t*>(sc + plan.off_frame_utt);
  int32_t* dnext = reinterpret_cast<int32_t*>(sc + plan.off_dup_next);
  int32_t* dfirst = reinterpret_cast<int32_t*>(sc + plan.off_dup_first);
  int32_t* status = reinterpret_cast<int32_t*>(sc + plan.off_status);
  double* loss_n = reinterpret_cast<double*>(sc + plan.off_logp);  // scratch use only
  float* tva = reinterpret_cast<float*>(sc + plan.off_tab_va);
  float* dummy = reinterpret_cast<float*>(sc + plan.off_dummy);
  float* tvb = reinterpret_cast<float*>(sc + plan.off_tab_vb);
  double* sva = reinterpret_cast<double*>(sc + plan.off_sc_va);
  double* svb = reinterpret_cast<double*>(sc + plan.off_sc_vb);
  double* vbest = reinterpret_cast<double*>(sc + plan.off_vbest);
  // arc masks of kMaskBeams beams: the plan's own, and four each in the two log-sum tables, which
  // this path does not use (a float per cell)
  uint8_t* mask_of[kMaskBeams];
  mask_of[0] = reinterpret_cast<uint8_t*>(sc + plan.off_mask);
  for (int b = 0; b < 4; ++b) {
    mask_of[1 + b] = reinterpret_cast<uint8_t*>(sc + plan.off_tab_fa) + b * plan.lattice;
    mask_of[5 + b] = reinterpret_cast<uint8_t*>(sc + plan.off_tab_fb) + b * plan.lattice;
  }
  static_assert(kMaskBeams == 9 && sizeof(float) == 4, "one mask region and two tables of four");
  {
    Prof pr("dp_prep", stream);
    hipLaunchKernelGGL(dp_prep_kernel, dim3(N), dim3(256), 0, stream, toff, yoff, y_rel, K_max, status, dnext, dfirst,
                       frame_utt, loss_n, nullptr, nullptr, nullptr, nullptr);
  }
  int Q, nwv;
  pick_lanes(plan.Smax, &Q, &nwv);
  hipError_t e;
  {  // the best alignments, the same for every beam
    Prof pr("dp_viterbi", stream);
    e = launch_pass<true>(Q, nwv, N, stream, S, ldS, toff, yoff, soff, y_rel, status, nullptr, tva, tvb, sva, svb, vbest,
                          loss_n, dummy);
    if (e != hipSuccess) return e;
  }
  for (int b0 = 0; b0 < nbeams; b0 += kMaskBeams) {
    const int nb = nbeams - b0 < kMaskBeams ? nbeams - b0 : kMaskBeams;
    MaskBeams mb{};
    for (int b = 0; b < nb; ++b) {
      mb.beam[b] = beams[b0 + b];
      mb.mask[b] = mask_of[b];
    }
    if (plan.M > 0) {
      Prof pr("dp_mask", stream);
      if (nb == 1)
        hipLaunchKernelGGL(dp_mask_kernel<1>, dim3(plan.M), dim3(256), 0, stream, S, ldS, toff, yoff, soff, y_rel,
                           frame_utt, status, tva, tvb, sva, svb, vbest, nb, mb, kKeepSlack);
      else
        hipLaunchKernelGGL(dp_mask_kernel<kMaskBeams>, dim3(plan.M), dim3(256), 0, stream, S, ldS, toff, yoff, soff,
                           y_rel, frame_utt, status, tva, tvb, sva, svb, vbest, nb, mb, kKeepSlack);
    }
    {
      Prof pr("dp_discarded", stream);
      e = launch_discarded(Q, nwv, N, nb, stream, S, ldS, toff, yoff, soff, y_rel, status, mb,
                           delta + static_cast<int64_t>(b0) * N);
      if (e != hipSuccess) return e;
    }
  }
  return hipGetLastError();
}

}  // namespace pctc
