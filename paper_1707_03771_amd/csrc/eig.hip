// Symmetric eigen-decomposition on the GPU: the two-sided block Jacobi method
// (the cyclic Jacobi method of Golub & Van Loan, "Matrix Computations", 4th
// ed., sec. 8.5, applied to 32 x 32 blocks; parallel orderings as in their
// sec. 8.5.5).  It serves the SCF wherever a full set of eigenpairs is needed
// (section "Standard algorithms": the orthogonaliser of the overlap, the
// orbitals and orbital energies of RHF, UHF and ROHF).
//
// The matrix, zero-padded to N = 64 ceil(n / 64), is split into nb = N / 32
// blocks.  A sweep runs nb - 1 rounds; a round pairs the blocks into nb / 2
// disjoint pairs by the circle method.  Per round:
//   1. ej_pair_kernel: per pair (a, b), one workgroup loads the 64 x 64
//      principal submatrix of blocks a and b into LDS and rotates every element
//      of its off-diagonal block once (32 rounds of 32 disjoint rotations, each
//      rotation zeroing its element exactly; a round updates S by 2 x 2 blocks,
//      one thread per block, so rows and columns need no barrier in between),
//      accumulating the orthogonal U with U^T S U the reduced submatrix.  In the
//      first round of a sweep the elements inside both blocks are rotated first
//      (31 rounds), so that a sweep meets every element once.  S goes back in
//      place, U to a buffer.
//   2. ej_apply_kernel: the off-diagonal 64 x 64 blocks between pairs,
//      A_IJ <- U_I^T A_IJ U_J (one workgroup per block I > J, writing both
//      A_IJ and A_JI), and the eigenvector columns V_:I <- V_:I U_I.
// A rotation is applied only when |a_pq| > 1e-15 sqrt(|a_pp a_qq|); the
// iteration stops after a sweep without any rotation, so on return every
// off-diagonal element is below that bound.  Padded rows and columns carry
// exact zeros, which no rotation ever touches, so they never mix with the
// matrix's own.  Rotations: t = sign(th) / (|th| + sqrt(1 + th^2)),
// th = (a_qq - a_pp) / (2 a_pq), c = 1 / sqrt(1 + t^2), s = t c; the rotated
// diagonal is a_pp - t a_pq and a_qq + t a_pq (Golub & Van Loan, Alg. 8.5.1).
#include <algorithm>
#include <numeric>
#include <type_traits>
#include <vector>

#include "host.h"
#include "kernels.h"

namespace dfx {

namespace {

constexpr int EJB = 32;       // block
constexpr int EJP = 64;       // pair problem (two blocks)
constexpr int EJT = 256;      // threads per workgroup
constexpr double EJ_TOL = 1e-15;

__device__ __forceinline__ int ej_g(int i, int2 ab) { return i < EJB ? ab.x * EJB + i : ab.y * EJB + (i - EJB); }

// Round r of a visit, rotation k in [0, 32), as local indices p < q.  cross: p in
// the first block, q in the second, r in [0, 32).  Otherwise inside the blocks,
// 16 rotations each by the circle method on 32 indices, r in [0, 31).
__device__ __forceinline__ void ej_local_pair(bool cross, int r, int k, int& p, int& q) {
  if (cross) {
    p = k;
    q = EJB + ((k + r) & (EJB - 1));
    return;
  }
  const int blk = k & EJB / 2 ? EJB : 0, j = k & (EJB / 2 - 1);
  int a = r + j, b = r - j + (EJB - 1);
  if (a >= EJB - 1) a -= EJB - 1;
  if (b >= EJB - 1) b -= EJB - 1;
  if (j == 0) b = EJB - 1;
  p = blk + (a < b ? a : b);
  q = blk + (a < b ? b : a);
}

// 1 / sqrt(x) and 1 / x for x in [1e-280, 1e280]: the hardware's estimates and
// two Newton steps, half the latency of the library's
__device__ __forceinline__ double ej_rsqrt(double x) {
  double y = __builtin_amdgcn_rsq(x);
  y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
  return fma(0.5 * y, fma(-x * y, y, 1.0), y);
}
__device__ __forceinline__ double ej_rcp(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = fma(y, fma(-x, y, 1.0), y);
  return fma(y, fma(-x, y, 1.0), y);
}

// Aw = (A + A^T) / 2 zero-padded to N x N, V = I
__global__ void ej_init_kernel(const double* __restrict__ A, int n, int N, double* __restrict__ Aw,
                               double* __restrict__ V) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)N * N) return;
  const int i = (int)(e / N), j = (int)(e % N);
  Aw[e] = (i < n && j < n) ? 0.5 * (A[(int64_t)i * n + j] + A[(int64_t)j * n + i]) : 0.0;
  V[e] = i == j ? 1.0 : 0.0;
}

// What bounds it: the chain of one round after the other, so the work is arranged
// by latency.  Wave 0 forms a round's rotations (three divisions, a square root
// and an inverse square root, one rotation per lane) while the other seven apply
// the round before to U; then all eight update S.  A round moves S and U through
// LDS once, 128 KB, which is about half of its time.  Four waves doing one after
// the other, 63 rounds a visit: 150 us; the 32 rounds of a visit now 45 (105 with
// the rounds inside the blocks).  A visit that finds nothing to rotate ends at once.
constexpr int EJPT = 512;
__global__ void __launch_bounds__(EJPT) ej_pair_kernel(double* __restrict__ A, int N, const int2* __restrict__ pr,
                                                       int inside, double* __restrict__ Ub, int* __restrict__ nrot,
                                                       int* __restrict__ moved) {
  __shared__ double S[EJP][EJP + 1];
  __shared__ double Ut[EJP][EJP + 1];  // Ut[r][k] = U[k][r]: its rows rotate like those of S
  // rotations of a round, two buffers: U lags S by one round
  __shared__ double cs_c[2][EJP / 2], cs_s[2][EJP / 2], d_p[EJP / 2], d_q[EJP / 2];
  __shared__ int any, todo;
  const int2 ab = pr[blockIdx.x];
  const int t = threadIdx.x;
  if (t == 0) any = todo = 0;
#pragma unroll
  for (int e = t; e < EJP * EJP; e += EJPT) {
    const int i = e / EJP, j = e % EJP;
    S[i][j] = A[(int64_t)ej_g(i, ab) * N + ej_g(j, ab)];
    Ut[i][j] = i == j ? 1.0 : 0.0;
  }
  __syncthreads();
  bool some = false;
#pragma unroll
  for (int e = t; e < EJP * EJP; e += EJPT) {
    const int i = e / EJP, j = e % EJP;
    if (i >= j || (!inside && (i >= EJB || j < EJB))) continue;
    const double x = S[i][j];
    some |= x != 0.0 && !(fabs(x) <= EJ_TOL * sqrt(fabs(S[i][i] * S[j][j])));
  }
  if (some) todo = 1;  // every writer stores the same value
  __syncthreads();
  if (!todo) {  // U is the identity (its partner's block may still need it)
    for (int e = t; e < EJP * EJP; e += EJPT) Ub[(int64_t)blockIdx.x * EJP * EJP + e] = Ut[e / EJP][e % EJP];
    if (t == 0) moved[blockIdx.x] = 0;
    return;
  }
  // rotations of round r into buffer b
  auto rotations = [&](bool cross, int r, int b) {
    if (t >= EJP / 2) return;
    int p, q;
    ej_local_pair(cross, r, t, p, q);
    const double apq = S[p][q], app = S[p][p], aqq = S[q][q];
    double c = 1.0, s = 0.0, dp = app, dq = aqq;
    if (apq != 0.0 && fabs(apq) > EJ_TOL * sqrt(fabs(app * aqq))) {
      double tt;
      const double big = fabs(apq) > 1e-250 ? (aqq - app) * ej_rcp(2.0 * apq) : (aqq - app) / (2.0 * apq);
      const double th = fabs(big);
      if (th < 1e130) {
        const double w = fma(th, th, 1.0);
        tt = ej_rcp(th + w * ej_rsqrt(w));
      } else {  // also where it overflowed
        tt = 0.5 / th;
      }
      if (big < 0.0) tt = -tt;
      c = ej_rsqrt(fma(tt, tt, 1.0));
      s = tt * c;
      dp = app - tt * apq;
      dq = aqq + tt * apq;
      any = 1;
    }
    cs_c[b][t] = c;
    cs_s[b][t] = s;
    d_p[t] = dp;
    d_q[t] = dq;
  };
  // rows p, q of U^T for the rotations in buffer b, by the waves from w0 on: a
  // wave takes every (8 - w0)th rotation, a lane a column; all loads first
  auto rotate_u = [&](bool cross, int r, int b, auto w0c) {
    constexpr int W0 = decltype(w0c)::value, NW = EJPT / 64 - W0, NK = (EJP / 2 + NW - 1) / NW;
    const int w = (t >> 6) - W0, j = t & 63;
    double c[NK], s[NK], u[NK], v[NK];
    int pk[NK], qk[NK];
#pragma unroll
    for (int m = 0; m < NK; ++m) {
      const int k = min(w + NW * m, EJP / 2 - 1);
      ej_local_pair(cross, r, k, pk[m], qk[m]);
      c[m] = cs_c[b][k];
      s[m] = cs_s[b][k];
      u[m] = Ut[pk[m]][j];
      v[m] = Ut[qk[m]][j];
    }
#pragma unroll
    for (int m = 0; m < NK; ++m) {
      if (w + NW * m >= EJP / 2 || s[m] == 0.0) continue;
      Ut[pk[m]][j] = c[m] * u[m] - s[m] * v[m];
      Ut[qk[m]][j] = s[m] * u[m] + c[m] * v[m];
    }
  };
  // S <- J^T S J as 2 x 2 blocks (rows p_k, q_k) x (columns p_k2, q_k2): every
  // element is read and written by one thread, so rows and columns need no
  // barrier between them; the diagonal blocks take the exact rotated values.
  // Thread t takes the column pair k2 = t % 32 and the row pairs t / 32 + 16 m,
  // and issues all its loads before its stores.
  auto rotate_s = [&](bool cross, int r, int b) {
    const int k2 = t % (EJP / 2);
    const double c2 = cs_c[b][k2], s2 = cs_s[b][k2];
    int p2, q2;
    ej_local_pair(cross, r, k2, p2, q2);
    int pk[2], qk[2];
    double ck[2], sk[2], x[2][4];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      const int k = t / (EJP / 2) + 16 * m;
      ej_local_pair(cross, r, k, pk[m], qk[m]);
      ck[m] = cs_c[b][k];
      sk[m] = cs_s[b][k];
      x[m][0] = S[pk[m]][p2];
      x[m][1] = S[pk[m]][q2];
      x[m][2] = S[qk[m]][p2];
      x[m][3] = S[qk[m]][q2];
    }
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      const int k = t / (EJP / 2) + 16 * m;
      const int p = pk[m], q = qk[m];
      if (k == k2) {
        if (s2 != 0.0) {
          S[p][p] = d_p[k];
          S[q][q] = d_q[k];
          S[p][q] = 0.0;
          S[q][p] = 0.0;
        }
        continue;
      }
      const double c1 = ck[m], s1 = sk[m];
      if (s1 == 0.0 && s2 == 0.0) continue;
      // rows: J_k^T x, then columns: y J_k2
      const double ypp = c1 * x[m][0] - s1 * x[m][2], ypq = c1 * x[m][1] - s1 * x[m][3];
      const double yqp = s1 * x[m][0] + c1 * x[m][2], yqq = s1 * x[m][1] + c1 * x[m][3];
      S[p][p2] = c2 * ypp - s2 * ypq;
      S[p][q2] = s2 * ypp + c2 * ypq;
      S[q][p2] = c2 * yqp - s2 * yqq;
      S[q][q2] = s2 * yqp + c2 * yqq;
    }
  };
  const int first = inside ? EJB - 1 : 0;  // rounds inside the blocks come first
  const int rounds = first + EJB;
  for (int n = 0; n < rounds; ++n) {
    const bool cross = n >= first;
    const int r = cross ? n - first : n;
    if (t < 64)
      rotations(cross, r, n & 1);
    else if (n > 0)
      rotate_u(n - 1 >= first, n - 1 >= first ? n - 1 - first : n - 1, (n - 1) & 1,
               std::integral_constant<int, 1>{});
    __syncthreads();
    rotate_s(cross, r, n & 1);
    __syncthreads();
  }
  rotate_u(true, EJB - 1, (rounds - 1) & 1, std::integral_constant<int, 0>{});
  __syncthreads();
  for (int e = t; e < EJP * EJP; e += EJPT) {
    const int i = e / EJP, j = e % EJP;
    A[(int64_t)ej_g(i, ab) * N + ej_g(j, ab)] = S[i][j];
    Ub[(int64_t)blockIdx.x * EJP * EJP + e] = Ut[j][i];  // U[i][j]
  }
  if (t == 0) {
    moved[blockIdx.x] = any;  // 0: U is exactly the identity
    if (any) atomicAdd(nrot, 1);
  }
}

// C = A^T B of two 64 x 64 matrices in LDS, k the row index of both, on
// v_mfma_f64_16x16x4f64: wave w has the 32 x 32 quadrant (w & 1, w >> 1);
// acc[i][j][r] is C[32 (w & 1) + 16 i + 4 r + lk][32 (w >> 1) + 16 j + li]
typedef double v4d __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void ej_atb(const double (&A)[EJP][EJP + 1], const double (&B)[EJP][EJP + 1],
                                       v4d (&acc)[2][2]) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, li = lane & 15, lk = lane >> 4;
  const int m0 = (w & 1) * 32 + li, n0 = (w >> 1) * 32 + li;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
  for (int k = lk; k < EJP; k += 4) {
    const double a0 = A[k][m0], a1 = A[k][m0 + 16], b0 = B[k][n0], b1 = B[k][n0 + 16];
    acc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, acc[0][0], 0, 0, 0);
    acc[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b1, acc[0][1], 0, 0, 0);
    acc[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b0, acc[1][0], 0, 0, 0);
    acc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1, acc[1][1], 0, 0, 0);
  }
}

// blockIdx.x < ntri: off-diagonal block (I, J), I > J, of the pairs, A_IJ <- U_I^T A_IJ U_J
// (and A_JI its transpose); else the eigenvector columns of pair I over 64 rows of V.
// Pairs whose U is exactly the identity (moved[I] == 0) leave their blocks as they are.
// On the matrix cores; with four results per thread on the vector units the two
// products took 22 us a round at N = 448, this 13.
__global__ void __launch_bounds__(EJT) ej_apply_kernel(double* __restrict__ A, double* __restrict__ V, int N,
                                                       const int2* __restrict__ pr, const double* __restrict__ Ub,
                                                       const int* __restrict__ moved, int np, int ntri) {
  __shared__ double X[EJP][EJP + 1];
  __shared__ double U[EJP][EJP + 1];
  const int t = threadIdx.x;
  const int lane = t & 63, w = t >> 6, li = lane & 15, lk = lane >> 4;
  const int m0 = (w & 1) * 32 + lk, n0 = (w >> 1) * 32 + li;
  v4d acc[2][2];
  if ((int)blockIdx.x < ntri) {
    const int b = blockIdx.x;
    int I = (int)((sqrt(8.0 * b + 1.0) + 1.0) * 0.5);
    while (I * (I - 1) / 2 > b) --I;
    while ((I + 1) * I / 2 <= b) ++I;
    const int J = b - I * (I - 1) / 2;
    if (!moved[I] && !moved[J]) return;
    const int2 pI = pr[I], pJ = pr[J];
    double uj[EJP * EJP / EJT];
#pragma unroll
    for (int e = 0; e < EJP * EJP / EJT; ++e) {
      const int q = t + EJT * e, i = q / EJP, j = q % EJP;
      X[i][j] = A[(int64_t)ej_g(i, pI) * N + ej_g(j, pJ)];
      U[i][j] = Ub[(int64_t)I * EJP * EJP + q];
      uj[e] = Ub[(int64_t)J * EJP * EJP + q];
    }
    __syncthreads();
    ej_atb(X, U, acc);  // T^T = X^T U_I
    __syncthreads();
#pragma unroll
    for (int e = 0; e < EJP * EJP / EJT; ++e) U[(t + EJT * e) / EJP][(t + EJT * e) % EJP] = uj[e];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) X[m0 + 16 * i + 4 * r][n0 + 16 * j] = acc[i][j][r];
    __syncthreads();
    ej_atb(X, U, acc);  // R = T U_J
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int gr = ej_g(m0 + 16 * i + 4 * r, pI), gc = ej_g(n0 + 16 * j, pJ);
          A[(int64_t)gr * N + gc] = acc[i][j][r];
          A[(int64_t)gc * N + gr] = acc[i][j][r];
        }
    return;
  }
  // eigenvectors: rows [64 s, 64 s + 64) of V, columns of pair I: V_:I <- V_:I U_I
  const int b = blockIdx.x - ntri;
  const int I = b % np, strip = b / np;
  if (!moved[I]) return;
  const int2 pI = pr[I];
#pragma unroll
  for (int e = 0; e < EJP * EJP / EJT; ++e) {
    const int q = t + EJT * e, i = q / EJP, k = q % EJP;
    X[k][i] = V[(int64_t)(strip * EJP + i) * N + ej_g(k, pI)];  // X[k][i] = V[row i][col k]
    U[i][k] = Ub[(int64_t)I * EJP * EJP + q];
  }
  __syncthreads();
  ej_atb(X, U, acc);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        V[(int64_t)(strip * EJP + m0 + 16 * i + 4 * r) * N + ej_g(n0 + 16 * j, pI)] = acc[i][j][r];
}

__global__ void ej_diag_kernel(const double* __restrict__ Aw, int N, int n, double* __restrict__ d) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) d[i] = Aw[(int64_t)i * N + i];
}

// rows of A: eigenvectors in ascending order, w the eigenvalues
__global__ void ej_out_kernel(const double* __restrict__ Aw, const double* __restrict__ V, int N, int n,
                              const int* __restrict__ idx, double* __restrict__ A, double* __restrict__ w) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)n * n) return;
  const int k = (int)(e / n), mu = (int)(e % n);
  const int c = idx[k];
  A[e] = V[(int64_t)mu * N + c];
  if (mu == 0) w[k] = Aw[(int64_t)c * N + c];
}

struct EjDims {
  int N, nb, np;
};

EjDims ej_dims(int n) {
  EjDims d;
  d.N = (n + EJP - 1) / EJP * EJP;
  d.nb = d.N / EJB;
  d.np = d.nb / 2;
  return d;
}

}  // namespace

size_t sym_eig_work_bytes(int n) {
  const EjDims d = ej_dims(std::max(n, 1));
  auto a = [](size_t x) { return (x + 255) / 256 * 256; };
  return 2 * a(8 * (size_t)d.N * d.N) + a(8 * (size_t)d.np * EJP * EJP) +
         a(sizeof(int) * 2 * (size_t)(d.nb - 1) * d.np) + a(8 * (size_t)d.N) + a(sizeof(int) * (size_t)d.N) +
         a(sizeof(int) * (size_t)d.np) + 512;
}

int sym_eig(double* A, int n, double* w, hipStream_t st) {
  if (n <= 0) return 0;
  const EjDims d = ej_dims(n);
  const int N = d.N, nb = d.nb, np = d.np;
  DevMem Aw(8 * (size_t)N * N), V(8 * (size_t)N * N), Ub(8 * (size_t)np * EJP * EJP);
  // the rounds of a sweep: circle method over the nb blocks
  std::vector<int> prh(2 * (size_t)(nb - 1) * np);
  for (int r = 0; r < nb - 1; ++r)
    for (int k = 0; k < np; ++k) {
      int a, b;
      if (k == 0) {
        a = r;
        b = nb - 1;
      } else {
        a = (r + k) % (nb - 1);
        b = (r - k + (nb - 1)) % (nb - 1);
      }
      prh[2 * ((size_t)r * np + k)] = std::min(a, b);
      prh[2 * ((size_t)r * np + k) + 1] = std::max(a, b);
    }
  DevMem prd = upload(prh, st), cnt(sizeof(int)), dg(8 * (size_t)N), idxd(sizeof(int) * (size_t)N),
      mv(sizeof(int) * (size_t)np);
  const int64_t NN = (int64_t)N * N;
  hipLaunchKernelGGL(ej_init_kernel, dim3((unsigned)((NN + 255) / 256)), dim3(256), 0, st, A, n, N,
                     Aw.as<double>(), V.as<double>());
  const int ntri = np * (np - 1) / 2, nstrip = N / EJP;
  int sweeps = 0;
  for (;;) {
    if (sweeps == 40) throw Error(DFX_EHIP, "sym_eig: no convergence in 40 sweeps");
    DFX_HIP(hipMemsetAsync(cnt.p, 0, sizeof(int), st));
    for (int r = 0; r < nb - 1; ++r) {
      const int2* pr = reinterpret_cast<const int2*>(prd.as<int>() + 2 * (size_t)r * np);
      hipLaunchKernelGGL(ej_pair_kernel, dim3(np), dim3(EJPT), 0, st, Aw.as<double>(), N, pr, r == 0 ? 1 : 0,
                         Ub.as<double>(), cnt.as<int>(), mv.as<int>());
      hipLaunchKernelGGL(ej_apply_kernel, dim3(ntri + nstrip * np), dim3(EJT), 0, st, Aw.as<double>(),
                         V.as<double>(), N, pr, Ub.as<double>(), mv.as<int>(), np, ntri);
    }
    ++sweeps;
    int h = 0;
    DFX_HIP(hipMemcpyAsync(&h, cnt.p, sizeof(int), hipMemcpyDeviceToHost, st));
    DFX_HIP(hipStreamSynchronize(st));
    if (h == 0) break;
  }
  // ascending order (ties by index, so the result is deterministic)
  hipLaunchKernelGGL(ej_diag_kernel, dim3((n + 255) / 256), dim3(256), 0, st, Aw.as<double>(), N, n,
                     dg.as<double>());
  std::vector<double> dh(n);
  DFX_HIP(hipMemcpyAsync(dh.data(), dg.p, 8 * (size_t)n, hipMemcpyDeviceToHost, st));
  DFX_HIP(hipStreamSynchronize(st));
  std::vector<int> idx(n);
  std::iota(idx.begin(), idx.end(), 0);
  std::stable_sort(idx.begin(), idx.end(), [&](int a, int b) { return dh[a] < dh[b]; });
  DFX_HIP(hipMemcpyAsync(idxd.p, idx.data(), sizeof(int) * (size_t)n, hipMemcpyHostToDevice, st));
  const int64_t nn = (int64_t)n * n;
  hipLaunchKernelGGL(ej_out_kernel, dim3((unsigned)((nn + 255) / 256)), dim3(256), 0, st, Aw.as<double>(),
                     V.as<double>(), N, n, idxd.as<int>(), A, w);
  DFX_HIP(hipGetLastError());
  DFX_HIP(hipStreamSynchronize(st));  // the host index vector goes out of scope
  return sweeps;
}

}  // namespace dfx
