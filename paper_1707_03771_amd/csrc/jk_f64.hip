// Exchange build K = sum_Q (B_Q C)(B_Q C)^T (Eqs. 1a, 2a) in FP64 on gfx950
// v_mfma_f64_16x16x4f64, with B_Q = hi + lo (two FP32 words per element).
// Phase 1 (half transform) streams each packed 32x32 tile of B_Q once per
// block of 64 or 128 rows and multiplies it by all occupied columns of C at
// once: kx64s_kernel up to 160 columns, from the kept tiles only, kx64_kernel
// beyond.  Phase 2 is a split-K SYRK over the (Q, i) index, from memory straight
// to LDS (gemm_dma.h), into FP64 partial sums with an XCD-aware tile map,
// reduced in a fixed order.
#include <algorithm>

#include <string>
#include <type_traits>

#include "gemm_dma.h"
#include "kernels.h"

namespace dfx {

constexpr int S64 = 16;   // k-width of one LDS stage (half a tile column of B_Q)
constexpr int PA = 1;     // row padding (doubles) of [row][k] tiles: odd row strides keep the
                          // fragment reads of 16 consecutive rows on distinct banks
constexpr int PB = 16;    // row padding (doubles) of the [k][i] C stage

// Place of X[mu][k], k = (Q, i): rows of stride ldx, or with ldx = 0 in blocks of
// 16 k, [k / 16][mu][k % 16]: a stage of the contraction below then reads
// consecutive kilobytes.  With rows of 10 to 20 MB it took 128 bytes from each of
// 256 pages per stage: the
// contraction at nbf = 1200, nocc = 120, naux = 3600 in 12.4 ms, in blocks 11.0.
__device__ __forceinline__ int64_t x_place(int64_t ldx, int nbf, int mu, int64_t k) {
  return ldx ? (int64_t)mu * ldx + k : ((k >> 4) * nbf + mu) * 16 + (k & 15);
}

// C_occ zero-padded to Cp[nbfp][np] (np = 64 NCB, nbfp = 32 ntiles), so that a
// k-stage of C is one contiguous, aligned block
__global__ void cpad_kernel(const double* __restrict__ C, int nbf, int nocc, int nbfp, int np,
                            double* __restrict__ Cp) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)nbfp * np) return;
  const int nu = (int)(idx / np), i = (int)(idx % np);
  Cp[idx] = (nu < nbf && i < nocc) ? C[(int64_t)nu * nocc + i] : 0.0;
}

// ---- phase 1: X_Q[mu][i] = sum_nu B_Q[mu][nu] C[nu][i] for a block of MR = 64 RB
// rows of mu and all occupied columns (padded to NP = 64 NCB).  Eight waves in
// a 2 x 4 grid: wave w owns rows [(w & 1) MR / 2, +MR / 2) and columns
// [(w >> 1) NCB 16, +NCB 16), i.e. 2 RB x NCB accumulator blocks.
constexpr int KX_T = 512;
// Rows per block in units of 64.  128 rows halve the L2 reads of C per flop,
// which pays from 256 occupied columns on (measured); beyond 320 columns the
// 128-row accumulators no longer fit in 256 registers.
constexpr int kx_rb(int ncb) { return (ncb >= 4 && ncb <= 5) ? 2 : 1; }
template <int NCB, int RB>
__global__ void __launch_bounds__(KX_T) kx64_kernel(const float* __restrict__ hi, const float* __restrict__ lo,
                                                    int64_t ncols, int nbf, int q0, const double* __restrict__ Cp,
                                                    int nocc, double* __restrict__ X, int64_t ldx) {
  constexpr int NP = 64 * NCB;
  constexpr int MR = 64 * RB;
  constexpr int WA = 2 * RB;                  // 16-row fragments per wave
  constexpr int EP = 2 * RB;                  // consecutive A elements per thread per stage
  constexpr int TPR = KX_T / (MR / 32);       // threads per 32-row tile row
  constexpr int NCL = S64 * NP / (2 * KX_T);  // 16-byte pairs of C per thread per stage
  static_assert(NCL * 2 * KX_T == S64 * NP, "C stage must split evenly");
  static_assert(TPR * EP == 32 * S64, "A stage must split evenly");
  typedef float vfa __attribute__((ext_vector_type(EP)));
  __shared__ double As[2][MR][S64 + PA];
  __shared__ double Bs[2][S64][NP + PB];
  const int Q = q0 + blockIdx.y;
  const int m0 = blockIdx.x * MR;
  const int I0 = m0 >> 5;
  const int nt = ntiles_for(nbf);
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int wr = (w & 1) * (MR / 2), wc = (w >> 1) * NCB * 16;
  const float* __restrict__ rh = hi + (int64_t)Q * ncols;
  const float* __restrict__ rl = lo + (int64_t)Q * ncols;
  // A loader: thread group `half` serves tile row I0 + half, EP consecutive
  // elements per thread (along nu in a direct tile, along mu in a mirrored one)
  const int half = tid / TPR, t = tid % TPR;
  const int I = I0 + half;
  constexpr int DK = S64 / EP;  // threads per row of a direct stage
  constexpr int TM = 32 / EP;   // threads per row of a mirrored stage

  vfa ah, al;
  double2 cr[NCL];
  auto load = [&](int stage) {
    const int J = stage >> 1, h = stage & 1;
    ah = al = vfa(0.f);
    if (I < nt) {
      int64_t off;
      if (I >= J)  // direct tile (I, J): row mu = t / DK, nu = 16 h + EP (t % DK) ..
        off = tile_base(I, J) + (t / DK) * 32 + 16 * h + (t % DK) * EP;
      else         // tile (J, I): row nu = 16 h + t / TM, mu = EP (t % TM) ..
        off = tile_base(J, I) + (16 * h + t / TM) * 32 + (t % TM) * EP;
      ah = *reinterpret_cast<const vfa*>(rh + off);
      al = *reinterpret_cast<const vfa*>(rl + off);
    }
    const double2* __restrict__ cs = reinterpret_cast<const double2*>(Cp + (int64_t)stage * S64 * NP);
#pragma unroll
    for (int c = 0; c < NCL; ++c) cr[c] = cs[tid + KX_T * c];
  };
  // stage s goes to LDS buffer s & 1: one barrier per stage, since stage s's
  // buffer was last read in stage s - 2, which every wave finished before the
  // barrier of stage s - 1
  auto store = [&](int stage) {
    const int J = stage >> 1, b = stage & 1;
    if (I >= J) {
      const int r = half * 32 + t / DK, k0 = (t % DK) * EP;
#pragma unroll
      for (int e = 0; e < EP; ++e) As[b][r][k0 + e] = (double)ah[e] + (double)al[e];
    } else {
      const int k = t / TM, r0 = half * 32 + (t % TM) * EP;
#pragma unroll
      for (int e = 0; e < EP; ++e) As[b][r0 + e][k] = (double)ah[e] + (double)al[e];
    }
#pragma unroll
    for (int c = 0; c < NCL; ++c) {
      const int e = 2 * (tid + KX_T * c);  // NP is even: a pair never straddles rows
      Bs[b][e / NP][e % NP] = cr[c].x;
      Bs[b][e / NP][e % NP + 1] = cr[c].y;
    }
  };

  v4d acc[WA][NCB];
#pragma unroll
  for (int a = 0; a < WA; ++a)
#pragma unroll
    for (int b = 0; b < NCB; ++b) acc[a][b] = v4d{0.0, 0.0, 0.0, 0.0};

  auto mma = [&](auto bufc) {
    constexpr int BUF = decltype(bufc)::value;
#pragma unroll
    for (int kk = 0; kk < S64; kk += 4) {
      double fa[WA];
#pragma unroll
      for (int a = 0; a < WA; ++a) fa[a] = As[BUF][wr + a * 16 + li][kk + lk];
#pragma unroll
      for (int b = 0; b < NCB; ++b) {
        const double fb = Bs[BUF][kk + lk][wc + b * 16 + li];
#pragma unroll
        for (int a = 0; a < WA; ++a) acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[a], fb, acc[a][b], 0, 0, 0);
      }
    }
  };
  const int nstage = 2 * nt;  // even: the stages pair up over the two buffers
  load(0);
  for (int s = 0; s < nstage; s += 2) {
    store(s);
    __syncthreads();
    load(s + 1);  // in flight during the MFMAs below
    mma(std::integral_constant<int, 0>{});
    store(s + 1);
    __syncthreads();
    if (s + 2 < nstage) load(s + 2);
    mma(std::integral_constant<int, 1>{});
  }
  // f64 MFMA output: element r of lane (li, lk) is row 4 r + lk, column li
#pragma unroll
  for (int a = 0; a < WA; ++a)
#pragma unroll
    for (int b = 0; b < NCB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int mu = m0 + wr + a * 16 + 4 * r + lk;
        const int i = wc + b * 16 + li;
        if (mu < nbf && i < nocc) X[x_place(ldx, nbf, mu, (int64_t)blockIdx.y * nocc + i)] = acc[a][b][r];
      }
}

// ---- phase 1 with up to 160 occupied columns: NB blocks of 16 columns, so that
// no more than 15 columns are padding (a multiple of 64 wasted 49% at nocc = 65
// and 38% at 40).  Four waves own RW x 16 rows each and all NB column blocks.
// Only the tiles of B that hold a kept pair are visited: a workgroup walks the
// union of its tile rows' masks, and a tile row without the tile reads nothing
// (a buffer of length zero gives zeros).  In long molecules half of the tiles
// hold none (zigzag C30H62: 56% of the columns screened).
// As for the products of gemm_dma.h, vector instructions stop the matrix cores:
// C goes to LDS by DMA from a padded copy (whose rows of odd nu have their
// 16-column blocks swapped in pairs when NB is even, so that fragment reads
// spread over the banks), B's words come by buffer loads at scalar bases, and
// what is left is their conversion, in one place per stage.
// A column of C with an Inf or NaN is NaN throughout in the copy: skipping a tile's zeros
// must not lose it, as zero times either is NaN.
constexpr int KS_T = 256;
// One workgroup per 64 rows and 16 columns of the copy; every one reads its columns whole
// (some 1000 rows by 64 at a time: a few loads in flight each, from L2).
__global__ void __launch_bounds__(1024) cpad16_kernel(const double* __restrict__ C, int nbf, int nocc, int nbfp, int np,
                                                      double* __restrict__ Cp) {
  __shared__ double red[16][16];
  const int r = threadIdx.x >> 4, c = threadIdx.x & 15, i = 16 * blockIdx.y + c, nu = 64 * blockIdx.x + r;
  const double own = nu < nbf && i < nocc ? C[(int64_t)nu * nocc + i] : 0.0;
  double z = 0.0;  // 0 or NaN
  if (i < nocc) {
#pragma unroll 8
    for (int k = r; k < nbf; k += 64) z = fma(0.0, C[(int64_t)k * nocc + i], z);
  }
  z += __shfl_xor(z, 16);  // a wave has 4 of the 64 rows
  z += __shfl_xor(z, 32);
  if ((r & 3) == 0) red[r >> 2][c] = z;
  __syncthreads();
  z = 0.0;
#pragma unroll
  for (int q = 0; q < 16; ++q) z += red[q][c];
  if (nu < nbfp) Cp[(int64_t)nu * np + ((nu & 1) && np % 32 == 0 ? i ^ 16 : i)] = own + z;
}

extern __shared__ __attribute__((aligned(1024))) double kxs_lds[];
template <int NB, int RW>
__global__ void __launch_bounds__(KS_T, 2) kx64s_kernel(const float* __restrict__ hi, const float* __restrict__ lo,
                                                        int64_t ncols, int nbf, int q0,
                                                        const unsigned long long* __restrict__ mask, int mw,
                                                        const double* __restrict__ Cp, int nocc,
                                                        double* __restrict__ X, int64_t ldx) {
  constexpr int NP = 16 * NB;
  constexpr int MR = 64 * RW;                 // rows of the workgroup
  constexpr int TR = MR / 32;                 // its tile rows
  constexpr int TPR = KS_T / TR;              // threads per tile row
  constexpr int EP = 32 * S64 / TPR;          // consecutive A elements per thread per stage: 4 or 8
  constexpr int DK = S64 / EP;                // threads per row of a direct stage
  constexpr int TM = 32 / EP;                 // threads per row of a mirrored stage
  typedef unsigned v4u __attribute__((ext_vector_type(4)));
  typedef float v4fl __attribute__((ext_vector_type(4)));
  __shared__ double As[2][MR][S64 + PA];
  // dynamic: the compiler does not see the DMA loads write it, and must not take
  // it for memory that nothing writes
  double* const Bs[2] = {kxs_lds, kxs_lds + S64 * NP};
  const int Q = q0 + blockIdx.y;
  const int m0 = blockIdx.x * MR;
  const int I0 = m0 >> 5;
  const int nt = ntiles_for(nbf);
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const int wr = w * 16 * RW;
  const float* __restrict__ rh = hi + (int64_t)Q * ncols;
  const float* __restrict__ rl = lo + (int64_t)Q * ncols;
  const int grp = __builtin_amdgcn_readfirstlane(tid / TPR), t = tid % TPR;  // a wave is in one tile row
  const int I = I0 + grp;
  const unsigned long long* __restrict__ mrow = mask + (int64_t)(I < nt ? I : 0) * mw;

  // the next tile column J of the union of the workgroup's tile rows (uniform),
  // or nt
  int word = -1, J = nt;
  unsigned long long bits = 0;
  auto advance = [&]() {
    while (bits == 0) {
      if (++word >= mw) {
        J = nt;
        return;
      }
#pragma unroll
      for (int r = 0; r < TR; ++r)
        if (I0 + r < nt) bits |= mask[(int64_t)(I0 + r) * mw + word];
    }
    J = word * 64 + __builtin_ctzll(bits);
    bits &= bits - 1;
  };

  // byte offsets of the lane in a tile: direct tile (I, J): row mu = t / DK, nu =
  // EP (t % DK) ..; tile (J, I), mirrored: row nu = t / TM, mu = EP (t % TM) ..
  const int vod = ((t / DK) * 32 + (t % DK) * EP) * 4, vom = ((t / TM) * 32 + (t % TM) * EP) * 4;
  v4u ah[EP / 4], al[EP / 4];
  bool direct = false;
  auto load = [&](int Jt, int h, int buf) {
    direct = I >= Jt;
    const bool kept = I < nt && (mrow[Jt >> 6] >> (Jt & 63) & 1);
    const int64_t base = kept ? (direct ? tile_base(I, Jt) : tile_base(Jt, I)) : 0;
    const int n = kept ? TILE2 * 4 : 0;
    const __amdgpu_buffer_rsrc_t dh =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(rh + base), 0, n, 0x00027000);
    const __amdgpu_buffer_rsrc_t dl =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(rl + base), 0, n, 0x00027000);
    const int vo = direct ? vod : vom, so = direct ? 64 * h : 2048 * h;
#pragma unroll
    for (int v = 0; v < EP / 4; ++v) {
      ah[v] = __builtin_amdgcn_raw_buffer_load_b128(dh, vo, so + 16 * v, 0);
      al[v] = __builtin_amdgcn_raw_buffer_load_b128(dl, vo, so + 16 * v, 0);
    }
    // the C stage: 2 NB loads of 1 KB, dealt to the waves
    const double* cs = Cp + (int64_t)(2 * Jt + h) * S64 * NP;
#pragma unroll
    for (int c = 0; c < (2 * NB + 3) / 4; ++c)
      if (4 * c + w < 2 * NB)
        DmaOp<true, 32>::dma(cs + (4 * c + w) * 128, 1024, &Bs[buf][(4 * c + w) * 128], lane * 16);
  };
  auto store = [&](int b) {
    double v[EP];
#pragma unroll
    for (int e = 0; e < EP; ++e) {
      const v4fl h = __builtin_bit_cast(v4fl, ah[e >> 2]), l = __builtin_bit_cast(v4fl, al[e >> 2]);
      v[e] = (double)h[e & 3] + (double)l[e & 3];
    }
    if (direct) {
      const int r = grp * 32 + t / DK, k0 = (t % DK) * EP;
#pragma unroll
      for (int e = 0; e < EP; ++e) As[b][r][k0 + e] = v[e];
    } else {
      const int k = t / TM, r0 = grp * 32 + (t % TM) * EP;
#pragma unroll
      for (int e = 0; e < EP; ++e) As[b][r0 + e][k] = v[e];
    }
  };

  v4d acc[RW][NB];
#pragma unroll
  for (int a = 0; a < RW; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[a][b] = v4d{0.0, 0.0, 0.0, 0.0};
  double fa[2][RW], fb[2][NB];  // the fragments of the current and the next k-step
  const int sw = NB % 2 == 0 ? (lk & 1) << 4 : 0;
  auto frag = [&](int buf, int kk, int f) {
#pragma unroll
    for (int a = 0; a < RW; ++a) fa[f][a] = As[buf][wr + a * 16 + li][kk + lk];
#pragma unroll
    for (int b = 0; b < NB; ++b)
      fb[f][b] = NB % 2 == 0 ? Bs[buf][lk * NP + li + (((b & 1) << 4) ^ sw) + (b >> 1) * 32 + kk * NP]
                             : Bs[buf][lk * NP + li + b * 16 + kk * NP];
  };
  auto mma = [&](int f) {
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int a = 0; a < RW; ++a)
        acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[f][a], fb[f][b], acc[a][b], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
  };
  // The two halves of a tile column alternate over the two LDS buffers.  In a
  // stage, the fragments of a k-step are read during the MFMAs of the step
  // before it, across stages too.  After the barrier, where every fragment of
  // the stage is in registers, the next stage but one is requested: C straight
  // into the buffer just read, B's words into registers, from which they reach
  // that buffer in the middle of the next stage.
  auto stage = [&](auto bufc, bool next, bool next2, int Jt, int h) {
    constexpr int BUF = decltype(bufc)::value;
    frag(BUF, 4, 1);
    __builtin_amdgcn_sched_barrier(0);
    mma(0);
    frag(BUF, 8, 0);
    if (next) store(BUF ^ 1);
    __builtin_amdgcn_sched_barrier(0);
    mma(1);
    frag(BUF, 12, 1);
    __builtin_amdgcn_sched_barrier(0);
    mma(0);
    stage_sync();
    if (next) frag(BUF ^ 1, 0, 0);
    if (next2) load(Jt, h, BUF);
    __builtin_amdgcn_sched_barrier(0);
    mma(1);
  };
  advance();
  if (J < nt) {
    load(J, 0, 0);
    store(0);
    load(J, 1, 1);
    stage_sync();
    frag(0, 0, 0);
  } else {  // no tile at all: zero times C, of which one row tells whether it is finite
#pragma unroll
    for (int a = 0; a < RW; ++a)
#pragma unroll
      for (int b = 0; b < NB; ++b) acc[a][b] = v4d(0.0 * Cp[16 * b + li]);
  }
  while (J < nt) {
    advance();
    const bool more = J < nt;
    stage(std::integral_constant<int, 0>{}, true, more, J, 0);
    stage(std::integral_constant<int, 1>{}, more, more, J, 1);
  }
#pragma unroll
  for (int a = 0; a < RW; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int mu = m0 + wr + a * 16 + 4 * r + lk;
        const int i = b * 16 + li;
        if (mu < nbf && i < nocc) X[x_place(ldx, nbf, mu, (int64_t)blockIdx.y * nocc + i)] = acc[a][b][r];
      }
}

// Rows per workgroup, or 0 where the kernel above does not serve: up to 160
// columns; 128 rows halve the reads of C per flop and are taken unless the last
// workgroup of 128 would be half empty in a small matrix, or the accumulators
// and fragments of 128 rows would no longer fit in 256 registers.
static int kxs_rows(int nbf, int nocc) {
  if (nocc > 160) return 0;
  if (nocc > 128) return 64;
  const int m128 = (nbf + 127) / 128 * 128, m64 = (nbf + 63) / 64 * 64;
  return m128 <= m64 + m64 / 8 ? 128 : 64;
}

static void kx64_launch(const JKArgs& a, int nocc, int q0, int nq, const double* Cp, double* X, int64_t ldx,
                        hipStream_t st) {
  if (const int mr = kxs_rows(a.nbf, nocc)) {
    const dim3 g((a.nbf + mr - 1) / mr, nq);
    const unsigned lds = 2 * S64 * 16 * ((nocc + 15) / 16) * sizeof(double);
    switch ((nocc + 15) / 16) {
#define KXS(N)                                                                                                    \
  case N:                                                                                                         \
    if (mr == 128)                                                                                                \
      hipLaunchKernelGGL((kx64s_kernel<N, N <= 8 ? 2 : 1>), g, dim3(KS_T), lds, st, a.hi, a.lo, a.ncols, a.nbf, q0, a.mask, a.mw, \
                         Cp, nocc, X, ldx);                                                                       \
    else                                                                                                          \
      hipLaunchKernelGGL((kx64s_kernel<N, 1>), g, dim3(KS_T), lds, st, a.hi, a.lo, a.ncols, a.nbf, q0, a.mask, a.mw, \
                         Cp, nocc, X, ldx);                                                                       \
    break;
      KXS(1) KXS(2) KXS(3) KXS(4) KXS(5) KXS(6) KXS(7) KXS(8) KXS(9) KXS(10)
#undef KXS
    }
    return;
  }
  const int ncb = (nocc + 63) / 64;
  const int mr = 64 * kx_rb(ncb);
  const dim3 g((a.nbf + mr - 1) / mr, nq);
  switch (ncb) {
#define KX64(N)                                                                                                  \
  case N:                                                                                                        \
    hipLaunchKernelGGL((kx64_kernel<N, kx_rb(N)>), g, dim3(KX_T), 0, st, a.hi, a.lo, a.ncols, a.nbf, q0, Cp, nocc, \
                       X, ldx);                                                                                  \
    break;
    KX64(3) KX64(4) KX64(5) KX64(6) KX64(7) KX64(8)
#undef KX64
  }
}

// ---- phase 2: P_s = X_s X_s^T (lower TM x TM tiles) for k-slices s of X, on the
// main loop of gemm_dma.h.  Workgroups are dealt round-robin to the 8 XCDs;
// every tile of a slice goes to one XCD so that the slice of X is fetched from
// HBM once per XCD L2.  Tiles of 64 serve the sizes of which 128 leaves much of
// the border tiles empty (syrk_plan).  On a diagonal tile the wave whose
// sub-tile lies above the diagonal skips its MFMAs.  A single slice goes
// straight to both triangles of K.
extern __shared__ __attribute__((aligned(1024))) double syrk_lds[];
template <int TM>
__global__ void __launch_bounds__(GT, 2) syrk64_kernel(const double* __restrict__ X, int64_t ldx, int64_t kst,
                                                       int nbf, int64_t kslice, int64_t kdim, int nslices, int ntl,
                                                       double* __restrict__ P, int accumulate) {
  constexpr int FA = TM / 32;
  const int bid = blockIdx.x;
  const int xcd = bid & 7, local = bid >> 3;
  const int s = nslices > 1 ? xcd + 8 * (local / ntl) : 0;
  const int tl = nslices > 1 ? local % ntl : bid;
  if (s >= nslices) return;
  int ti = (int)((sqrt(8.0 * tl + 1.0) - 1.0) * 0.5);
  while ((ti + 1) * (ti + 2) / 2 <= tl) ++ti;
  while (ti * (ti + 1) / 2 > tl) --ti;
  const int tj = tl - ti * (ti + 1) / 2;
  const int m0 = ti * TM, n0 = tj * TM;
  const int64_t k0s = min((int64_t)s * kslice, kdim);
  const int klen = (int)(min(k0s + kslice, kdim) - k0s);
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = (w & 1) * (TM / 2), wn = (w >> 1) * (TM / 2);
  const bool active = ti != tj || wn <= wm;
  const int li = lane & 15, lk = lane >> 4;
  DmaOp<true, TM> a, b;
  a.init(X + k0s * kst, ldx, m0, nbf, klen, w, lane, kst);
  b.init(X + k0s * kst, ldx, n0, nbf, klen, w, lane, kst);
  v4d acc[FA][FA];
  dma_gemm<true, true, TM, TM>(a, b, klen, syrk_lds, wm, wn, active, acc);
  if (!active) return;
  double* __restrict__ Ps = P + (int64_t)s * nbf * nbf;
#pragma unroll
  for (int i = 0; i < FA; ++i)
#pragma unroll
    for (int j = 0; j < FA; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int m = m0 + wm + i * 16 + 4 * q + lk;
        const int n = n0 + wn + j * 16 + li;
        if (m >= nbf || n > m) continue;
        double v = acc[i][j][q];
        if (nslices == 1) {
          if (accumulate) v += Ps[(int64_t)m * nbf + n];
          Ps[(int64_t)n * nbf + m] = v;
        }
        Ps[(int64_t)m * nbf + n] = v;
      }
}

// K = sum_s P_s from the lower triangles, both triangles of K written: one
// workgroup per 16 x 16 tile, its four groups of 256 threads every fourth slice
// each, the groups added in order.  (One thread per element adding all slices
// in turn took 255 us at nbf = 192 with 688 slices, a chain of dependent loads.)
__global__ void __launch_bounds__(1024) k_reduce_kernel(const double* __restrict__ P, int ns, int nbf,
                                                        double* __restrict__ K, int accumulate) {
  __shared__ double red[4][16][17];
  int I = (int)((sqrt(8.0 * blockIdx.x + 1.0) - 1.0) * 0.5);
  while ((I + 1) * (I + 2) / 2 <= (int)blockIdx.x) ++I;
  while (I * (I + 1) / 2 > (int)blockIdx.x) --I;
  const int J = blockIdx.x - I * (I + 1) / 2;
  const int e = threadIdx.x & 255, g = threadIdx.x >> 8;
  const int row = e >> 4, col = e & 15;
  const int r = I * 16 + row, c = J * 16 + col;
  const bool own = r < nbf && c <= r;
  const int64_t n2 = (int64_t)nbf * nbf, idx = (int64_t)r * nbf + c;
  double s = 0.0;
  if (own) {
#pragma unroll 8
    for (int k = g; k < ns; k += 4) s += P[k * n2 + idx];
  }
  red[g][row][col] = s;
  __syncthreads();
  if (g == 0 && own) {
    s = (accumulate ? K[idx] : 0.0) + ((red[0][row][col] + red[1][row][col]) + (red[2][row][col] + red[3][row][col]));
    K[idx] = s;
    red[0][row][col] = s;
  }
  __syncthreads();
  const int mr = J * 16 + row, mc = I * 16 + col;  // the mirror image, stored as rows
  if (g == 0 && mc < nbf && mr < mc) K[(int64_t)mr * nbf + mc] = red[0][col][row];
}

void k_reduce(const double* P, int ns, int nbf, double* K, bool accumulate, hipStream_t st) {
  const int t = (nbf + 15) / 16;
  hipLaunchKernelGGL(k_reduce_kernel, dim3((unsigned)(t * (t + 1) / 2)), dim3(1024), 0, st, P, ns, nbf, K,
                     accumulate ? 1 : 0);
}

// Tile size and number of k-slices of an n x kdim SYRK.  In units of the
// cycles of one CU: a stage (16 k) of a 128-tile keeps its matrix cores 4096
// cycles and of a 64-tile 1024, at the efficiencies measured with one, two and
// more workgroups on the CU; the workgroups are dealt to 32 CUs on each of 8
// XCDs, so the CU with the most of them sets the time; every slice is written
// and read again once, and more than one slice takes another launch (5 us).
// Tiles of 64 read X through L2 twice as often.  Over a long k-range (X of several GB)
// that begins to tell between 1200 functions (11.0 ms, no slower than 128) and 1354
// and 1536 (22.9 and 22.6 ms in tiles of 64, 22.2 and 20.7 of 128), which is where the
// line lies.  Over a short one it comes later: at kdim = 51200 K takes 1.76, 2.37,
// 2.64, 2.87 and 3.42 ms in tiles of 64 and 1.89, 2.56, 3.00, 3.02 and 3.32 of 128 at
// 1280, 1472, 1600, 1664 and 1792 functions, and the plan, whose efficiencies do not
// know of kdim, takes 128 at all of these.
// Before, 128-tiles and about 2048 workgroups at any size: nbf = 192, kdim =
// 33920 (3 tiles, 688 slices): 72 us + 255 us for the sum.
struct SyrkPlan {
  int tm, ntl, ns;
};
static SyrkPlan syrk_plan(int n, int64_t kdim, int64_t most_slices) {
  SyrkPlan best{};
  double tbest = 0.0;
  for (int tm = 64; tm <= 128; tm += 64) {
    const int mt = (n + tm - 1) / tm, ntl = mt * (mt + 1) / 2;
    for (int ns = 1; ns <= 256; ns = ns == 1 ? 8 : ns + 8) {
      if (ns > 1 && (ns > most_slices || ns > (kdim + S64 - 1) / S64 + 7)) break;
      const int64_t per_xcd = ns > 1 ? (int64_t)ntl * ns / 8 : (ntl + 7) / 8;
      const int64_t per_cu = (per_xcd + 31) / 32;
      const double stages = (double)((kdim + (int64_t)ns * S64 - 1) / ((int64_t)ns * S64));
      const double eff = tm == 128 ? (per_cu == 1 ? 0.6 : 0.83) : (per_cu == 1 ? 0.45 : per_cu == 2 ? 0.62 : n > 1300 ? 0.73 : 0.78);
      double t = (double)per_cu * (stages * (tm == 128 ? 4096.0 : 1024.0) / eff + 3000.0);
      if (ns > 1) t += 12000.0 + (double)ns * n * n * 8.0 / 5.0e12 * 2.4e9;
      if (!best.tm || t < tbest) {
        best = SyrkPlan{tm, ntl, ns};
        tbest = t;
      }
    }
  }
  return best;
}

// K (+)= X X^T over k < kdim; X row-major (kst = 1), or in blocks of 16 k (ldx =
// 16, kst = n); P: ns n^2 doubles (none for one slice)
static void syrk_run(const SyrkPlan& p, const double* X, int64_t ldx, int64_t kst, int n, int64_t kdim, double* P, double* K,
                     bool accumulate, hipStream_t st) {
  const int64_t kslice = ((kdim + p.ns - 1) / p.ns + S64 - 1) / S64 * S64;
  double* out = p.ns > 1 ? P : K;
  const unsigned grid = (unsigned)(p.ns * p.ntl);
  const unsigned lds = 4 * p.tm * GK * sizeof(double);
  if (p.tm == 128)
    hipLaunchKernelGGL(syrk64_kernel<128>, dim3(grid), dim3(GT), lds, st, X, ldx, kst, n, kslice, kdim, p.ns,
                       p.ntl, out, accumulate ? 1 : 0);
  else
    hipLaunchKernelGGL(syrk64_kernel<64>, dim3(grid), dim3(GT), lds, st, X, ldx, kst, n, kslice, kdim, p.ns,
                       p.ntl, out, accumulate ? 1 : 0);
  if (p.ns > 1) k_reduce(P, p.ns, n, K, accumulate, st);
}

struct F64Plan {
  int qc, np, nbfp;
  SyrkPlan sy;
  size_t x_bytes, p_bytes, c_bytes;
};

static size_t a256(size_t b) { return (b + 255) & ~(size_t)255; }

// X chunks of at most 8 GiB, balanced over the chunks; SYRK partial sums within
// 2 GiB.  Under a work cap: at most eight slices and X in what the cap leaves.
static F64Plan f64_plan(const JKArgs& a, int nocc) {
  F64Plan p{};
  const size_t per_q = (size_t)a.nbf * nocc * sizeof(double);
  p.np = kxs_rows(a.nbf, nocc) ? 16 * ((nocc + 15) / 16) : 64 * ((nocc + 63) / 64);  // columns of the copy of C
  p.nbfp = ntiles_for(a.nbf) * TILE;
  p.c_bytes = (size_t)p.nbfp * p.np * sizeof(double);
  size_t xbytes = (size_t)8 << 30;
  int64_t by_mem = ((int64_t)2 << 30) / ((int64_t)a.nbf * a.nbf * 8);
  if (a.ws_cap) {
    // eight slices, C, the last block of X and alignment
    const size_t fixed = a256((size_t)8 * a.nbf * a.nbf * 8) + p.c_bytes + (size_t)a.nbf * 8 * S64 + 1024;
    if (a.ws_cap < fixed + per_q)
      throw Error(DFX_ENOMEM, "K work: " + std::to_string(a.ws_cap) + " bytes hold no chunk (" +
                                  std::to_string(fixed + per_q) + " needed)");
    xbytes = a.ws_cap - fixed;
    by_mem = 8;
  }
  size_t cap = xbytes / per_q;
  if (cap < 1) cap = 1;
  const int nchunks = (int)((a.naux + cap - 1) / cap);
  p.qc = (a.naux + nchunks - 1) / nchunks;
  const int64_t kdim = (int64_t)p.qc * nocc;
  // no more partial sums than 2048 tiles of 128 x 128 would have
  const int64_t mt = (a.nbf + 127) / 128, most = (2048 / (mt * (mt + 1) / 2) + 8) / 8 * 8;
  p.sy = syrk_plan(a.nbf, kdim, std::max<int64_t>(std::min(by_mem, most), 8));
  p.x_bytes = (size_t)a.nbf * ((kdim + S64 - 1) / S64 * S64) * sizeof(double);
  p.p_bytes = (size_t)p.sy.ns * a.nbf * a.nbf * sizeof(double);
  return p;
}

static void pad_cocc(const JKArgs& a, const double* C, int nocc, const F64Plan& p, double* Cp, hipStream_t st) {
  if (kxs_rows(a.nbf, nocc))
    hipLaunchKernelGGL(cpad16_kernel, dim3((p.nbfp + 63) / 64, p.np / 16), dim3(1024), 0, st, C, a.nbf, nocc, p.nbfp,
                       p.np, Cp);
  else
    hipLaunchKernelGGL(cpad_kernel, dim3((unsigned)(((int64_t)p.nbfp * p.np + 255) / 256)), dim3(256), 0, st, C, a.nbf, nocc, p.nbfp, p.np, Cp);
}

size_t half_transform_f64_work(const JKArgs& a, int nocc) {
  const F64Plan p = f64_plan(a, nocc);
  return p.c_bytes;
}

void half_transform_f64(const JKArgs& a, const double* C, int nocc, int q0, int nq, double* X, int64_t ldx,
                        void* work, hipStream_t st) {
  const F64Plan p = f64_plan(a, nocc);
  const int ncb = (nocc + 63) / 64;
  if (ncb > 8) throw Error(-6, "half transform: more than 512 columns");
  if (q0 < 0 || nq <= 0 || q0 + nq > a.naux || ldx < (int64_t)nq * nocc) throw Error(-1, "half transform: bad range");
  double* Cp = reinterpret_cast<double*>(work);
  pad_cocc(a, C, nocc, p, Cp, st);
  kx64_launch(a, nocc, q0, nq, Cp, X, ldx, st);
}

static size_t f64_work(const F64Plan& p) { return a256(p.x_bytes) + a256(p.p_bytes) + p.c_bytes + 256; }

size_t k_work_bytes_f64(const JKArgs& a, int nocc) { return f64_work(f64_plan(a, nocc)); }

void k_build_f64(const JKArgs& a, const double* C, int nocc, double* K, void* work, size_t work_bytes,
                 hipStream_t st, KTimer* timer) {
  const F64Plan p = f64_plan(a, nocc);
  const int ncb = (nocc + 63) / 64;
  if (ncb > 8) throw Error(-6, "k_build: more than 512 occupied orbitals");
  k_check_work(f64_work(p), work_bytes);
  char* w = reinterpret_cast<char*>(work);
  double* X = reinterpret_cast<double*>(w);
  double* P = reinterpret_cast<double*>(w + a256(p.x_bytes));
  double* Cp = reinterpret_cast<double*>(w + a256(p.x_bytes) + a256(p.p_bytes));
  pad_cocc(a, C, nocc, p, Cp, st);
  for (int q0 = 0; q0 < a.naux; q0 += p.qc) {
    const int nq = std::min(p.qc, a.naux - q0);
    const int64_t kdim = (int64_t)nq * nocc;
    if (timer) timer->begin_x();
    kx64_launch(a, nocc, q0, nq, Cp, X, 0, st);
    if (timer) timer->end_x();
    if (timer) timer->begin_syrk();
    syrk_run(p.sy, X, S64, a.nbf, a.nbf, kdim, P, K, q0 > 0, st);
    if (timer) timer->end_syrk();
  }
}

// C = A A^T (n x n, both triangles) for a row-major n x k matrix A with an even
// row stride lda, on the exchange build's SYRK: at most eight k-slices, summed
// in FP64 in a fixed order.  For a symmetric A this is A^2 at half the FLOPs of
// a general product.  work: syrk_f64_work_elems(n) doubles.
size_t syrk_f64_work_elems(int n) { return (size_t)8 * n * n; }

void syrk_f64(const double* A, int64_t lda, int n, int64_t k, double* C, double* work, hipStream_t st) {
  if (n <= 0) return;
  if ((lda & 1) || lda < k || (reinterpret_cast<uintptr_t>(A) & 15))
    throw Error(-1, "syrk_f64: A needs an even row stride >= k and 16-byte alignment");
  syrk_run(syrk_plan(n, k, 8), A, lda, 1, n, k, work, C, false, st);
}

}  // namespace dfx
