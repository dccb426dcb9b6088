// FP64 products on v_mfma_f64_16x16x4f64 with operands that go from memory
// straight to LDS: the main loop shared by the general product (linalg.hip) and
// the exchange contraction (jk_f64.hip).
#pragma once
#include <type_traits>

#include "gemm_small.h"

namespace dfx {

constexpr int GK = 16, GT = 256;  // k-width of a stage, threads of a workgroup

// For operands whose rows are 16-byte aligned.
// What bounds it: v_mfma_f64_16x16x4f64 occupies a SIMD's matrix core for 64
// cycles, and no vector ALU instruction of any wave on that SIMD runs meanwhile
// (measured: 64 cycles become 77 with one VALU instruction per MFMA, about 9 for
// the change-over and 4 for each instruction, however many waves are resident),
// while LDS reads, scalar instructions and memory requests do.  So the k-stages
// go from memory straight to LDS (buffer loads with the lds bit: addresses are
// a per-lane offset that never changes and a scalar base), and the main loop
// has next to no VALU instructions.  Two LDS buffers; the fragments of a k-step
// are read during the MFMAs of the step before, across stages too; one barrier
// per stage, where every fragment of the stage is in registers and its buffer
// can be refilled.  At 128 x 131072 x 1728 with random operands: 54 TFLOP/s
// register-staged, 66 so (72% and 88% of what the matrix cores reach alone, 77.7).
//
// The LDS image of a stage is what the loads make it, 16 bytes per lane in
// order, so the bank swizzle is in the lanes' source offsets:
//   k contiguous (A, or B transposed): rows of 16 k; the pair of k at 2 c of row
//     x is at place c ^ (x & 7), so that 16 rows read at one k spread over the banks;
//   otherwise: rows k of TX; on odd k the 16-column blocks are swapped in pairs.
template <bool KC, int TX>
struct DmaOp {
  static constexpr int N = TX / 32;  // loads per wave and stage (1 KB each)
  const double* P;                   // the operand at the tile's first row or column
  int64_t ld, kst;                   // KC: distance of rows, and of a stage's first k from k = 0 over k
  int X, K;                          // rows or columns left from there, k range
  int w, lane;
  int vo[2];                         // byte offsets of the lane

  __device__ __forceinline__ void init(const double* base, int64_t ld_, int x0, int x, int k, int wave, int ln,
                                       int64_t kst_ = 1) {
    P = KC ? base + (int64_t)x0 * ld_ : base + x0;
    ld = ld_;
    kst = kst_;
    X = x - x0;
    K = k;
    w = wave;
    lane = ln;
    if (KC) {
      vo[0] = (lane >> 3) * (int)ld * 8 + (((lane & 7) ^ (lane >> 3)) << 4);
    } else {
      // TX = 128: a row per load; TX = 64: two rows per load, lane / 32 the row
      const int row = TX == 128 ? 0 : lane >> 5, c = TX == 128 ? lane : lane & 31;
      vo[0] = row * (int)ld * 8 + (TX == 128 ? c : c ^ (row << 3)) * 16;
      vo[1] = (lane ^ 8) * 16;
    }
  }
  __device__ __forceinline__ void load(double* S, int k0) const {
    if (k0 + GK > K) {  // the last, partial stage: through registers, zero beyond the k range
#pragma unroll
      for (int e = 0; e < 2 * N; ++e) {
        const int q = (w * 64 + lane) + 256 * e;  // element of the TX x 16 stage
        const int x = KC ? q >> 4 : q % TX, k = KC ? q & 15 : q / TX;
        double v = 0.0;
        if (x < X && k0 + k < K) v = KC ? P[(int64_t)x * ld + k0 * kst + k] : P[(int64_t)(k0 + k) * ld + x];
        S[at(x, k)] = v;
      }
      return;
    }
#pragma unroll
    for (int e = 0; e < N; ++e) {
      if (KC) {
        const int r = w * (8 * N) + 8 * e;
        const int64_t left = r < X ? ((int64_t)(X - 1 - r) * ld + GK) * 8 : 0;
        dma(P + (int64_t)r * ld + k0 * kst, left, S + r * GK, vo[0]);
      } else if (TX == 128) {
        const int k = 4 * w + e;
        dma(P + (int64_t)(k0 + k) * ld, (int64_t)min(X, TX) * 8, S + k * TX, vo[e & 1]);
      } else {
        const int k = 4 * w + 2 * e;
        dma(P + (int64_t)(k0 + k) * ld, (ld + min(X, TX)) * 8, S + k * TX, vo[0]);
      }
    }
  }
  // place of element (x, k) in the stage
  __device__ __forceinline__ static int at(int x, int k) {
    return KC ? x * GK + (((k >> 1) ^ (x & 7)) << 1) + (k & 1) : k * TX + (x ^ ((k & 1) << 4));
  }
  // 64 lanes x 16 bytes from p + vo to LDS; reads past `bytes` give zero
  __device__ __forceinline__ static void dma(const double* p, int64_t bytes, double* S, int vo) {
    typedef __attribute__((address_space(3))) void lds_void;
    const int n = (int)min(bytes, (int64_t)0x7ffffff0);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(p), 0, n, 0x00027000), (lds_void*)S, 16, vo, 0, 0, 0);
  }
};

// The stage's loads have landed for every wave; nothing moves across.  (The
// compiler does not see the loads as writes of LDS: the buffers have to be
// dynamic shared memory, which anything may write, or their reads are moved
// past barriers.)
__device__ __forceinline__ void stage_sync() {
  __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0)
  asm volatile("" ::: "memory");
  __syncthreads();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// acc += op(A) op(B) for one TM x TN tile: four waves in a 2 x 2 grid of
// (TM / 2) x (TN / 2) sub-tiles at (wm, wn), each FA x FB blocks of 16 x 16;
// acc[i][j][r] is element (wm + 16 i + 4 r + lk, wn + 16 j + li).  lds: 2 (TM + TN)
// GK doubles, 1 KB aligned.  A wave with active = false only loads and waits.
template <bool KCA, bool KCB, int TM, int TN>
__device__ __forceinline__ void dma_gemm(const DmaOp<KCA, TM>& a, const DmaOp<KCB, TN>& b, int kmax, double* lds,
                                         int wm, int wn, bool active, v4d (&acc)[TM / 32][TN / 32]) {
  constexpr int FA = TM / 32, FB = TN / 32;
  double* const As[2] = {lds, lds + TM * GK};
  double* const Bs[2] = {lds + 2 * TM * GK, lds + 2 * TM * GK + TN * GK};
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
#pragma unroll
  for (int i = 0; i < FA; ++i)
#pragma unroll
    for (int j = 0; j < FB; ++j) acc[i][j] = v4d{0.0, 0.0, 0.0, 0.0};

  // fragment x of k-step kk: element (x0 + 16 f + li, kk + lk), at a lane address
  // plus constants
  double fa[2][FA], fb[2][FB];
  auto frag_op = [&](auto kc, auto txc, const double* S, int x0, int kk, auto nfc, double* f) {
    constexpr bool KC = decltype(kc)::value;
    constexpr int TX = decltype(txc)::value;
#pragma unroll
    for (int i = 0; i < decltype(nfc)::value; ++i)
      f[i] = KC ? S[(x0 + li) * GK + (((kk >> 1) ^ ((lk >> 1) ^ (li & 7))) << 1) + (lk & 1) + 16 * i * GK]
                : S[lk * TX + x0 + li + (((i & 1) ^ (lk & 1)) << 4) + 32 * (i >> 1) + kk * TX];
  };
  auto frag = [&](int buf, int kk, int f) {
    frag_op(std::bool_constant<KCA>{}, std::integral_constant<int, TM>{}, As[buf], wm, kk,
            std::integral_constant<int, FA>{}, fa[f]);
    frag_op(std::bool_constant<KCB>{}, std::integral_constant<int, TN>{}, Bs[buf], wn, kk,
            std::integral_constant<int, FB>{}, fb[f]);
  };
  auto mma = [&](int f) {
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int i = 0; i < FA; ++i)
#pragma unroll
      for (int j = 0; j < FB; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[f][i], fb[f][j], acc[i][j], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
  };
  static_assert(GK == 16, "a stage is four k-steps");
  auto stage = [&](int k0, auto bufc) {
    constexpr int BUF = decltype(bufc)::value;
    frag(BUF, 4, 1);
    __builtin_amdgcn_sched_barrier(0);
    if (active) mma(0);
    frag(BUF, 8, 0);
    __builtin_amdgcn_sched_barrier(0);
    if (active) mma(1);
    frag(BUF, 12, 1);
    __builtin_amdgcn_sched_barrier(0);
    if (active) mma(0);
    stage_sync();
    if (k0 + GK < kmax) frag(BUF ^ 1, 0, 0);
    if (k0 + 2 * GK < kmax) {
      a.load(As[BUF], k0 + 2 * GK);
      b.load(Bs[BUF], k0 + 2 * GK);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (active) mma(1);
  };
  if (kmax > 0) {
    a.load(As[0], 0);
    b.load(Bs[0], 0);
    if (GK < kmax) {
      a.load(As[1], GK);
      b.load(Bs[1], GK);
    }
    stage_sync();
    frag(0, 0, 0);
  }
  for (int k0 = 0; k0 < kmax; k0 += 2 * GK) {
    stage(k0, std::integral_constant<int, 0>{});
    if (k0 + GK < kmax) stage(k0 + GK, std::integral_constant<int, 1>{});
  }
}

}  // namespace dfx
