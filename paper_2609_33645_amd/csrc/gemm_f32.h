// fp32 tile engine for gfx950: C[i][j] = sum_k A[i][k] B[j][k] over a 256 x 256 tile with fp32
// operands, on the bf16 matrix instructions.
//
// Every operand value is split into three bf16 parts, x = x0 + x1 + x2, each the rounding to nearest
// of what the earlier ones leave (exact for |x| of 2^-110 and more: below that the last part's low
// bits fall under bf16's least, 2^-133, and at 2^-126 eight significand bits are left), and the
// product is taken as the six part products of weight 2^-16 and more,
//   a b = a0 b0 + (a0 b1 + a1 b0) + (a0 b2 + a1 b1 + a2 b0) + dropped,
// each a v_mfma_f32_32x32x16_bf16 accumulated in fp32, a k-tile's smallest first.  What is dropped is
// at most 2^-24.2 |a b| and 2^-27.5 |a b| root mean square (one rounding of an fp32 product: at most
// 2^-24; with x0 cut to 8 bits instead of rounded, 2^-22.3 and 2^-25.5).  A sum is rounded six times
// per 16 products, on v_mfma_f32_32x32x2_f32 eight times.  At M = 16,000, D = 512, V = 180,000 the
// gradients are 1.5e-6 off 64 bits (on the fp32 instructions 2.4e-6, with x0 cut 1.7e-6).
// A value that is infinite, or rounds to infinity in bf16 (from 3.39e38), has no such parts: tiles
// that hold one are taken on the fp32 instructions (Gemm::run).
//
// What bounds it: six bf16 instructions of 32 cycles do the work of eight fp32 ones of 64, so the
// ceiling is 2500 / 6 = 417 TFLOP/s (fp32 units: 157).
//
// Tiles stay fp32 in global memory and LDS (buffer_load_dwordx4 ... lds, no register staging):
// a 16-deep k-tile is 16 KB per operand, four stages.  Each wavefront splits the fragments it
// reads: 11 vector instructions per pair of values, 264 per k-tile beside 48 matrix
// instructions.  The schedule is the ping-pong of gemm_bf16.h: waves 0-3 and 4-7 form two
// groups, one a phase behind the other, so that on every SIMD one wave issues its 48 products
// (1536 cycles, registers only) while the other copies, reads and splits its next k-tile.
// Measured (normaliser pass over M = 16,000, D = 512, V = 16,384; the fp32 units took 2390 us):
// 1250 us (with x0 cut 1260, and then 1135 with the splitting left out); with the splits
// interleaved with the products in each wave instead of the phases 1540; with the remainders from
// v_dot2_f32_bf16 (7 instructions per pair instead of 11) 1430: that instruction keeps the matrix
// pipe from issuing.
//
// LDS layouts: KC [row][k] (k contiguous in memory; 64-byte rows, 16-byte slots XORed with
// (row >> 2) mod 4, as KC<32> of gemm_bf16.h) and MC [k][row] (rows contiguous; 1 KB k-lines,
// those of k >= 8 with their 128-byte halves swapped, so that the two lane halves, which read
// k and k + 8, fall in different banks).
#pragma once

#include "gemm_bf16.h"

namespace pctc {
namespace f3 {

using bf::LL;

struct GOp {
  const float* base;
  int64_t pitch;  // elements between consecutive rows (KC) or k-lines (MC)
  int rows;       // valid rows
  int kmax;       // valid k
  const int* rowidx;  // KC only: row gather table (needs a Gemm with BUF false)
};

constexpr int kT = 256;  // tile rows and columns
constexpr int kBK = 16;  // k per stage

__device__ __attribute__((aligned(16))) static const float kZero4[4] = {0.f, 0.f, 0.f, 0.f};

// Copies of one operand's k-tile (256 rows x 16 k, 16 KB): wave w of 8 issues the 1 KB copies w
// and w + 8.  Through a buffer resource whose size ends at the tile's last valid row (KC) or
// k-line (MC); lanes past the last valid column (MC), or past k in the one partial k-tile (KC),
// carry bit 31 in their offset and read zeros.  A 16-byte slot that straddles the last valid
// k or row holds values of the operand's own padding: the callers' dZ rows are whole tiles.
template <LL L, bool BUF>
struct TileCopy {
  static constexpr int kPerWave = 2;
  const float* tbase;
  int row0_or_left;  // KC: valid rows of the tile; MC: row0
  int kpart;         // KC: k0 of the partial k-tile (none: -1)
  uint32_t poob;     // KC: bit 31 if this lane's slot is past the partial k-tile's limit
  uint32_t off[kPerWave];
  const float* src[BUF ? 1 : kPerWave];  // !BUF: this lane's rows
  int slotk;                             // !BUF: this lane's k within the tile

  __device__ __forceinline__ void init(const GOp& op, int row0, int w, int lane, int kbeg, int klim) {
    const int rem = (klim > kbeg) ? (klim - kbeg) % kBK : 0;
    kpart = rem ? klim - rem : -1;
    poob = 0u;
#pragma unroll
    for (int i = 0; i < kPerWave; ++i) {
      const int c = w + 8 * i;
      if constexpr (L == LL::KC) {
        const int r = c * 16 + (lane >> 2);
        const int slot = (lane & 3) ^ ((r >> 2) & 3);  // the same for every i: copies are 16 rows apart
        off[i] = static_cast<uint32_t>(r * op.pitch * 4 + slot * 16);
        poob = (slot * 4 < rem) ? 0u : bf::kOob;
        if constexpr (!BUF) {
          const bool ok = row0 + r < op.rows;
          slotk = slot * 4;
          src[i] = ok ? op.base + static_cast<int64_t>(op.rowidx[row0 + r]) * op.pitch + slot * 4 : nullptr;
        }
      } else {
        const int slot = lane ^ ((c >> 3) << 3);
        off[i] = static_cast<uint32_t>(c * op.pitch * 4 + slot * 16) | ((row0 + slot * 4 < op.rows) ? 0u : bf::kOob);
      }
    }
    if constexpr (L == LL::KC) {
      tbase = op.base + static_cast<int64_t>(row0) * op.pitch;
      row0_or_left = min(max(op.rows - row0, 0), kT);
    } else {
      tbase = op.base + row0;
      row0_or_left = row0;
    }
  }

  __device__ __forceinline__ void issue(const GOp& op, int k0, int klim, char* lds, int w) const {
#if defined(__HIP_DEVICE_COMPILE__)
    if constexpr (!BUF) {
#pragma unroll
      for (int i = 0; i < kPerWave; ++i) {
        const bool valid = src[i] && k0 + slotk < klim;
        bf::lds_copy16(valid ? static_cast<const void*>(src[i] + k0) : static_cast<const void*>(kZero4),
                       (bf::lds_void*)(lds + (w + 8 * i) * 1024));
      }
    } else {
      const int p4 = static_cast<int>(op.pitch) * 4;
      int size;
      const float* b;
      if constexpr (L == LL::KC) {
        b = tbase + k0;
        size = (k0 < klim) ? row0_or_left * p4 - k0 * 4 : 0;
      } else {
        b = tbase + static_cast<int64_t>(k0) * op.pitch;
        size = min(klim - k0, kBK) * p4 - row0_or_left * 4;
      }
      size = __builtin_amdgcn_readfirstlane(max(size, 0));
      const uint64_t ba = reinterpret_cast<uint64_t>(b);
      const uint64_t bu =
          (static_cast<uint64_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(ba >> 32))) << 32) |
          static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(ba)));
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
          reinterpret_cast<void*>(bu), static_cast<short>(0), size, bf::kBufWord3);
      uint32_t adj = 0u;
      if constexpr (L == LL::KC) {
        adj = (k0 == kpart) ? poob : 0u;
        asm volatile("" : "+v"(adj));  // one register per issue, not a hoisted second offset set
      }
#pragma unroll
      for (int i = 0; i < kPerWave; ++i)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (bf::lds_void*)(lds + (w + 8 * i) * 1024), 16, off[i] | adj, 0,
                                                 0, 0);
    }
#endif
  }
};

typedef __attribute__((ext_vector_type(4))) float f32x4;

// The three bf16 parts of a matrix-core fragment (8 values).  x0 and x1 are roundings to nearest of
// x and of x - x0, x2 what is left (at most 8 bits: exact).  A value whose x0 rounds to infinity has
// NaN remainders (see Gemm::run).
struct Tri {
  uint32_t d[3][4];
};
// Values 4 HALF .. 4 HALF + 3 of the fragment.
template <int HALF>
__device__ __forceinline__ void split4(const f32x4& x, Tri& t) {
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const uint32_t a = pack_bf16x2(x[2 * q], x[2 * q + 1]);
    t.d[0][2 * HALF + q] = a;
    const float r0 = x[2 * q] - __uint_as_float(a << 16), r1 = x[2 * q + 1] - __uint_as_float(a & 0xffff0000u);
    const uint32_t m = pack_bf16x2(r0, r1);
    t.d[1][2 * HALF + q] = m;
    t.d[2][2 * HALF + q] = pack_bf16x2(r0 - __uint_as_float(m << 16), r1 - __uint_as_float(m & 0xffff0000u));
  }
}

// 4 consecutive k of row rb + lane % 32, k = 8 (lane / 32) + 4 HALF .., from a stage.
template <LL L, int HALF>
__device__ __forceinline__ f32x4 frag4(const char* lds, int rb, int lane) {
  const int r = rb + (lane & 31), h = lane >> 5;
  if constexpr (L == LL::KC) {
    return *reinterpret_cast<const f32x4*>(lds + r * 64 + (((2 * h + HALF) ^ ((r >> 2) & 3)) << 4));
  } else {
    f32x4 x;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      x[e] = *reinterpret_cast<const float*>(lds + (8 * h + 4 * HALF + e) * 1024 + ((r * 4) ^ (h << 7)));
    return x;
  }
}

// Value k of row r from a stage.
template <LL L>
__device__ __forceinline__ float value(const char* lds, int r, int k) {
  if constexpr (L == LL::KC) {
    return *reinterpret_cast<const float*>(lds + r * 64 + (((k >> 2) ^ ((r >> 2) & 3)) << 4) + ((k & 3) << 2));
  } else {
    return *reinterpret_cast<const float*>(lds + k * 1024 + ((r * 4) ^ ((k >> 3) << 7)));
  }
}

// BUF false: A's rows through its gather table.
template <LL LA, LL LB, bool BUF = true>
struct Gemm {
  static constexpr int kNS = 4;
  static constexpr int kBR = kT, kBC = kT;
  static constexpr int NW = 8, kThreads = 512, WR = 2, WC = 4;
  static constexpr int FR = 4, FC = 2;
  static constexpr int kABytes = kT * kBK * 4, kStageBytes = 2 * kABytes;
  using CA = TileCopy<LA, BUF>;
  using CB = TileCopy<LB, true>;
  static constexpr int CPW = CA::kPerWave + CB::kPerWave;

  __device__ static __forceinline__ int row_of(int wave, int lane, int i, int r) {
    return (wave / WC) * (kT / WR) + 32 * i + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
  }
  __device__ static __forceinline__ int col_of(int wave, int lane, int j) {
    return (wave % WC) * (kT / WC) + 32 * j + (lane & 31);
  }
  __device__ static __forceinline__ void zero(f32x16 (&acc)[FR][FC]) {
#pragma unroll
    for (int i = 0; i < FR; ++i)
#pragma unroll
      for (int j = 0; j < FC; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  }
  __device__ static __forceinline__ void phase_barrier() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  }

  template <int S, class Issue>
  __device__ static __forceinline__ void pp_tile(char* const (&st)[kNS], int wave, int lane,
                                                 f32x16 (&acc)[FR][FC], Tri (&f)[FR + FC], Issue&& issue) {
    const int wr0 = (wave / WC) * (kT / WR), wc0 = (wave % WC) * (kT / WC);
    // fragment n: column block n, then row block n - FC; each is read while the one before is split
    f32x4 x[2][2];
    auto read = [&](int n, f32x4 (&v)[2]) {
      if (n < FC) {
        v[0] = frag4<LB, 0>(st[S] + kABytes, wc0 + 32 * n, lane);
        v[1] = frag4<LB, 1>(st[S] + kABytes, wc0 + 32 * n, lane);
      } else {
        v[0] = frag4<LA, 0>(st[S], wr0 + 32 * (n - FC), lane);
        v[1] = frag4<LA, 1>(st[S], wr0 + 32 * (n - FC), lane);
      }
    };
    read(0, x[0]);
    read(1, x[1]);
    issue(st[(S + kNS - 1) % kNS]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int n = 0; n < FR + FC; ++n) {
      split4<0>(x[n & 1][0], f[n]);
      split4<1>(x[n & 1][1], f[n]);
      if (n + 2 < FR + FC) read(n + 2, x[n & 1]);
      __builtin_amdgcn_sched_barrier(0);
    }
    // this group's copies up to the next k-tile have landed (kNS - 2 newer ones may still be in
    // flight); its reads of stage S are done before anyone refills it
    bf::wait_vmcnt<(kNS - 2) * CPW>();
    __builtin_amdgcn_s_waitcnt(0xC07F);
    phase_barrier();
#pragma unroll
    for (int w = 2; w >= 0; --w)  // smallest part products first: a_p b_(w - p)
#pragma unroll
      for (int p = w; p >= 0; --p)
#pragma unroll
        for (int i = 0; i < FR; ++i)
#pragma unroll
          for (int j = 0; j < FC; ++j) {
            bf16x8 u, v;
            __builtin_memcpy(&u, f[FC + i].d[p], 16);
            __builtin_memcpy(&v, f[j].d[w - p], 16);
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(u, v, acc[i][j], 0, 0, 0);
          }
    phase_barrier();
  }

  // acc = the sum over k in [kbeg, kend) (kbeg a multiple of 16).  All 512 threads must call;
  // contains barriers.  On return every copy has landed and every wave is past its last LDS read.
  __device__ static __forceinline__ void run(const GOp& A, const GOp& B, int row0, int col0, int kbeg, int kend,
                                             char* const (&st)[kNS], f32x16 (&acc)[FR][FC]) {
    zero(acc);
    if (kend <= kbeg) return;
    run_split(A, B, row0, col0, kbeg, kend, st, acc);
    // An operand that is infinite, or too large to round to bf16, has NaN remainders: its whole row
    // (or column) of the tile is NaN, so one column and one row of each block show it.  Such tiles
    // are taken again on the fp32 instructions, which give what fp32 arithmetic gives.
    bool nan = false;
#pragma unroll
    for (int i = 0; i < FR; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) nan |= acc[i][0][r] != acc[i][0][r];
#pragma unroll
    for (int j = 1; j < FC; ++j) nan |= acc[0][j][0] != acc[0][j][0];
    __shared__ __attribute__((aligned(16))) uint32_t wave_nan[NW];
    wave_nan[threadIdx.x >> 6] = __ballot(nan) != 0;  // the same value in every lane
    __syncthreads();  // also: before anyone reuses the stages
    uint32_t any = 0u;
#pragma unroll
    for (int w = 0; w < NW; ++w) any |= wave_nan[w];
    if (__builtin_expect(__builtin_amdgcn_readfirstlane(any) != 0u, 0)) {
      zero(acc);
      run_plain(A, B, row0, col0, kbeg, kend, st, acc);
    }
  }

  // The same on v_mfma_f32_32x32x2_f32 (one k-tile at a time, no overlap: for few tiles only).
  __device__ static __forceinline__ void run_plain(const GOp& A, const GOp& B, int row0, int col0, int kbeg, int kend,
                                                   char* const (&st)[kNS], f32x16 (&acc)[FR][FC]) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wr0 = (wave / WC) * (kT / WR), wc0 = (wave % WC) * (kT / WC);
    const int klimA = min(A.kmax, kend), klimB = min(B.kmax, kend);
    CA ca;
    CB cb;
    ca.init(A, row0, wave, lane, kbeg, klimA);
    cb.init(B, col0, wave, lane, kbeg, klimB);
#pragma unroll 1
    for (int k0 = kbeg; k0 < kend; k0 += kBK) {
      ca.issue(A, k0, klimA, st[0], wave);
      cb.issue(B, k0, klimB, st[0] + kABytes, wave);
      bf::wait_vmcnt<0>();
      __builtin_amdgcn_s_barrier();
#pragma unroll 1
      for (int kk = 0; kk < kBK; kk += 2) {
        const int k = kk + (lane >> 5);
        float a[FR], b[FC];
#pragma unroll
        for (int i = 0; i < FR; ++i) a[i] = value<LA>(st[0], wr0 + 32 * i + (lane & 31), k);
#pragma unroll
        for (int j = 0; j < FC; ++j) b[j] = value<LB>(st[0] + kABytes, wc0 + 32 * j + (lane & 31), k);
#pragma unroll
        for (int i = 0; i < FR; ++i)
#pragma unroll
          for (int j = 0; j < FC; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j], acc[i][j], 0, 0, 0);
      }
      __builtin_amdgcn_s_waitcnt(0xC07F);
      __builtin_amdgcn_s_barrier();  // before the stage is filled again
    }
  }

  // Accumulates the split products into acc.  On return this wave's copies have landed; a barrier is
  // left to the caller.
  __device__ static __forceinline__ void run_split(const GOp& A, const GOp& B, int row0, int col0, int kbeg, int kend,
                                                   char* const (&st)[kNS], f32x16 (&acc)[FR][FC]) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nk = (kend - kbeg + kBK - 1) / kBK;
    const int klimA = min(A.kmax, kend), klimB = min(B.kmax, kend);
    CA ca;
    CB cb;
    ca.init(A, row0, wave, lane, kbeg, klimA);
    cb.init(B, col0, wave, lane, kbeg, klimB);
    int knext = kbeg;  // k of the next tile to copy (past the end: zeros)
    auto issue = [&](char* stage) {
      ca.issue(A, knext, klimA, stage, wave);
      cb.issue(B, knext, klimB, stage + kABytes, wave);
      knext += kBK;
    };
    __builtin_amdgcn_s_barrier();  // previous users of the stages are done
#pragma unroll
    for (int s = 0; s < kNS - 1; ++s) issue(st[s]);
    bf::wait_vmcnt<(kNS - 2) * CPW>();  // tile 0
    __builtin_amdgcn_s_barrier();
    const bool lag = wave >= 4;
    if (lag) phase_barrier();  // group 1 starts one phase behind
    Tri f[FR + FC];
    int t = 0;
    for (; t + kNS <= nk; t += kNS) {
      pp_tile<0>(st, wave, lane, acc, f, issue);
      pp_tile<1>(st, wave, lane, acc, f, issue);
      pp_tile<2>(st, wave, lane, acc, f, issue);
      pp_tile<3>(st, wave, lane, acc, f, issue);
    }
    if (t < nk) pp_tile<0>(st, wave, lane, acc, f, issue);
    if (t + 1 < nk) pp_tile<1>(st, wave, lane, acc, f, issue);
    if (t + 2 < nk) pp_tile<2>(st, wave, lane, acc, f, issue);
    if (!lag) phase_barrier();  // the barrier group 1 took at the start
    bf::wait_vmcnt<0>();  // the copies past the end (zeros) have landed
  }
};

}  // namespace f3
}  // namespace pctc
