// Coulomb and exchange builds from the fitted tensor B (section "Density
// fitting utilities"):
//   J: gamma_Q = sum_{mu nu} B_Q,mu nu D_mu nu       (Eq. 3a)
//      J_mu nu = sum_Q gamma_Q B_Q,mu nu             (Eq. 3b)
//   K: X_Q = B_Q C                                   (Eq. 1a, half transform)
//      K_mu nu = sum_Q sum_i X_Q,mu i X_Q,nu i       (Eq. 2a)
// B is stored as two FP32 words (hi, lo) per element in the packed 32x32 tile
// layout (common.h).  The FP64 path reads hi + lo; the mixed path reads hi.
#include <algorithm>
#include <string>

#include "kernels.h"

namespace dfx {

typedef double v4d __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// tile index -> (I, J), I >= J
__device__ __forceinline__ void tile_ij(int t, int& I, int& J) {
  int i = (int)((sqrt(8.0 * t + 1.0) - 1.0) * 0.5);
  while ((i + 1) * (i + 2) / 2 <= t) ++i;
  while (i * (i + 1) / 2 > t) --i;
  I = i;
  J = t - i * (i + 1) / 2;
}

// A tile without a kept pair is skipped where B is streamed, but zero times Inf or NaN is
// NaN: what such a tile of D or of J owes a non-finite input is z = sum 0 x over the
// values x that meet its zeros, 0 or NaN.  The kernels below take ALL where every tile is
// kept and there is none of it.  The sum of all threads' z (256), in all threads.
__device__ __forceinline__ double wg_zsum(double z) {
  __shared__ double r[4];
  for (int o = 32; o > 0; o >>= 1) z += __shfl_xor(z, o);
  if ((threadIdx.x & 63) == 0) r[threadIdx.x >> 6] = z;
  __syncthreads();
  return r[0] + r[1] + r[2] + r[3];
}

// weighted density in the tile layout, off-diagonal tiles counted twice; of a tile that is not
// kept, z of its elements in the place of the first
template <bool ALL>
__global__ void __launch_bounds__(256) pack_density_kernel(const double* __restrict__ D, int nbf,
                                                           const int* __restrict__ tpos, double* __restrict__ d) {
  const int t = blockIdx.x;
  int I, J;
  tile_ij(t, I, J);
  const double w = (I == J) ? 1.0 : 2.0;
  if (!ALL && tpos[t] < 0) {
    double z = 0.0;
    for (int e = threadIdx.x; e < TILE2; e += 256) {
      const int r = I * TILE + (e >> 5), c = J * TILE + (e & 31);
      if (r < nbf && c < nbf) z = fma(0.0, D[(int64_t)r * nbf + c], z);
    }
    z = wg_zsum(z);
    if (threadIdx.x == 0) d[(int64_t)t * TILE2] = z;
    return;
  }
  for (int e = threadIdx.x; e < TILE2; e += blockDim.x) {
    const int r = I * TILE + (e >> 5), c = J * TILE + (e & 31);
    d[(int64_t)t * TILE2 + e] = (r < nbf && c < nbf) ? w * D[(int64_t)r * nbf + c] : 0.0;
  }
}

// The same from the occupied block, D = C C^T: one workgroup per tile, its four
// waves one 16 x 16 quadrant each on v_mfma_f64_16x16x4f64, operands straight
// from C (a few hundred KB, in L2).  Replaces a DGEMM for D (4 to 36 tiles of
// 128 x 128 at nbf = 192 to 730: 21 to 30 us on a mostly idle chip) and the
// packing pass after it; 4 us at nbf = 192, nocc = 40.
template <bool ALL>
__global__ void __launch_bounds__(256) pack_cocc_kernel(const double* __restrict__ C, int nbf, int nocc,
                                                        const int* __restrict__ tpos, double* __restrict__ d) {
  const int t = blockIdx.x;
  int I, J;
  tile_ij(t, I, J);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int r0 = (w >> 1) * 16, c0 = (w & 1) * 16;
  const int r = I * TILE + r0 + li, c = J * TILE + c0 + li;
  const double* __restrict__ pr = C + (int64_t)(r < nbf ? r : 0) * nocc;
  const double* __restrict__ pc = C + (int64_t)(c < nbf ? c : 0) * nocc;
  v4d acc = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll 8
  for (int k = 0; k < nocc; k += 4) {
    const bool in = k + lk < nocc;
    const double a = in && r < nbf ? pr[k + lk] : 0.0;
    const double b = in && c < nbf ? pc[k + lk] : 0.0;
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc, 0, 0, 0);
  }
  if (!ALL && tpos[t] < 0) {
    double z = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) z = fma(0.0, acc[q], z);
    z = wg_zsum(z);
    if (threadIdx.x == 0) d[(int64_t)t * TILE2] = z;
    return;
  }
  const double wt = (I == J) ? 1.0 : 2.0;
#pragma unroll
  for (int q = 0; q < 4; ++q) d[(int64_t)t * TILE2 + (r0 + 4 * q + lk) * TILE + c0 + li] = wt * acc[q];
}

// gamma_Q = sum_c B[Q][c] d[c], B = hi + lo, FP64 accumulation.  A workgroup
// takes JG_Q consecutive Q, so each element of d is fetched once per JG_Q rows
// of B (d is as long as a row of B: read once per Q it doubled the kernel's
// traffic), and the blockIdx.y'th part of the kept tiles: gp[y][Q] is its part of the
// sum, which the readers of gamma add in order (j_plan: enough workgroups to
// fill the chip where naux / JG_Q alone does not).
constexpr int JG_Q = 4;
template <bool ALL>
__global__ void __launch_bounds__(256) j_gamma_kernel(const float* __restrict__ hi,
                                                      const float* __restrict__ lo, int64_t ncols, int naux,
                                                      const double* __restrict__ d,
                                                      const int* __restrict__ tiles, int nt_kept, int tchunk,
                                                      const int* __restrict__ tpos, double* __restrict__ gp) {
  const int Q0 = blockIdx.x * JG_Q;
  const int nq = min(JG_Q, naux - Q0);
  const int t0 = blockIdx.y * tchunk, t1 = min(t0 + tchunk, nt_kept);
  double s[JG_Q];
#pragma unroll
  for (int k = 0; k < JG_Q; ++k) s[k] = 0.0;
  // z of the tiles that are not kept (pack_density_kernel), to one element: through it
  // every element of J takes it
  if (!ALL && blockIdx.x == 0 && blockIdx.y == 0)
    for (int t = threadIdx.x; t < (int)(ncols / TILE2); t += 256)
      if (tpos[t] < 0) s[0] += d[(int64_t)t * TILE2];
  for (int t = t0; t < t1; ++t) {
    const int64_t c = (int64_t)tiles[t] * TILE2 + 4 * threadIdx.x;
    const double4 dd = *reinterpret_cast<const double4*>(d + c);
#pragma unroll
    for (int k = 0; k < JG_Q; ++k) {
      if (k < nq) {
        const float4 h = *reinterpret_cast<const float4*>(hi + (int64_t)(Q0 + k) * ncols + c);
        const float4 l = *reinterpret_cast<const float4*>(lo + (int64_t)(Q0 + k) * ncols + c);
        s[k] += ((double)h.x + (double)l.x) * dd.x + ((double)h.y + (double)l.y) * dd.y +
                ((double)h.z + (double)l.z) * dd.z + ((double)h.w + (double)l.w) * dd.w;
      }
    }
  }
  __shared__ double red[JG_Q][256];
#pragma unroll
  for (int k = 0; k < JG_Q; ++k) red[k][threadIdx.x] = s[k];
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o)
#pragma unroll
      for (int k = 0; k < JG_Q; ++k) red[k][threadIdx.x] += red[k][threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x < nq) gp[(int64_t)blockIdx.y * naux + Q0 + threadIdx.x] = red[threadIdx.x][0];
}

// gamma = sum of the sg partial vectors, in order
__global__ void j_gamma_sum_kernel(const double* __restrict__ gp, int sg, int naux, double* __restrict__ gam) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= naux) return;
  double s = 0.0;
  for (int k = 0; k < sg; ++k) s += gp[(int64_t)k * naux + q];
  gam[q] = s;
}

// J_c = sum_Q B[Q][c] gamma_Q, B = hi + lo, over the Q of blockIdx.y, fixed Q
// order: one workgroup per kept tile, four columns per thread.  One workgroup per
// tile is 21 of them at nbf = 192 and 276 at 730, far from filling 256 CUs: the
// Q range is split until there are about 768 (j_plan), and the parts are added
// in j_unpack_kernel.
constexpr int JB_Q = 256;  // gammas staged in LDS at a time
__global__ void __launch_bounds__(256) j_back_kernel(const float* __restrict__ hi,
                                                     const float* __restrict__ lo, int64_t ncols,
                                                     int naux, const int* __restrict__ tiles,
                                                     const double* __restrict__ gp, int sg, int qchunk,
                                                     double* __restrict__ jp) {
  __shared__ double g[JB_Q];
  const int64_t c4 = (int64_t)tiles[blockIdx.x] * 256 + threadIdx.x;
  const int q0 = blockIdx.y * qchunk, q1 = min(q0 + qchunk, naux);
  double a0 = 0, a1 = 0, a2 = 0, a3 = 0;
  const float4* h4 = reinterpret_cast<const float4*>(hi) + c4;
  const float4* l4 = reinterpret_cast<const float4*>(lo) + c4;
  const int64_t stride = ncols >> 2;
  for (int qb = q0; qb < q1; qb += JB_Q) {
    const int nq = min(JB_Q, q1 - qb);
    __syncthreads();  // the previous gammas have been read
    if (threadIdx.x < nq) {
      double s = 0.0;
      for (int k = 0; k < sg; ++k) s += gp[(int64_t)k * naux + qb + threadIdx.x];
      g[threadIdx.x] = s;
    }
    __syncthreads();
#pragma unroll 4
    for (int i = 0; i < nq; ++i) {
      const float4 h = h4[(qb + i) * stride], l = l4[(qb + i) * stride];
      a0 = fma((double)h.x + (double)l.x, g[i], a0);
      a1 = fma((double)h.y + (double)l.y, g[i], a1);
      a2 = fma((double)h.z + (double)l.z, g[i], a2);
      a3 = fma((double)h.w + (double)l.w, g[i], a3);
    }
  }
  reinterpret_cast<double4*>(jp)[((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * 256 + threadIdx.x] =
      double4{a0, a1, a2, a3};
}

// the sb parts of the kept tiles of J, added in order -> dense symmetric matrix
// (where no tile was kept, zero times gamma), one workgroup per tile; the mirror image
// goes out through LDS so that both copies are stored as rows
template <bool ALL>
__global__ void __launch_bounds__(256) j_unpack_kernel(const double* __restrict__ jp, const int* __restrict__ tpos,
                                                       int nt_kept, int sb, int nbf, const double* __restrict__ gp,
                                                       int ngp, double* __restrict__ M) {
  __shared__ double tl[TILE][TILE + 1];
  int I, J;
  tile_ij(blockIdx.x, I, J);
  // four consecutive elements of a tile row per thread
  const int row = threadIdx.x >> 3, col = 4 * (threadIdx.x & 7);
  const int pos = tpos[blockIdx.x];
  const double* __restrict__ src = jp + (int64_t)(pos < 0 ? 0 : pos) * TILE2 + 4 * threadIdx.x;
  const int parts = pos < 0 ? 0 : sb;
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  if (!ALL && pos < 0) {
    double z = 0.0;
#pragma unroll 16
    for (int i = threadIdx.x; i < ngp; i += 256) z = fma(0.0, gp[i], z);
    z = wg_zsum(z);
#pragma unroll
    for (int e = 0; e < 4; ++e) s[e] = z;
  }
#pragma unroll 8
  for (int k = 0; k < parts; ++k) {
    const double4 v = *reinterpret_cast<const double4*>(src + (int64_t)k * nt_kept * TILE2);
    s[0] += v.x;
    s[1] += v.y;
    s[2] += v.z;
    s[3] += v.w;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int r = I * TILE + row, c = J * TILE + col + e;
    if (r < nbf && c < nbf) M[(int64_t)r * nbf + c] = s[e];
    tl[row][col + e] = s[e];
  }
  if (I == J) return;  // a diagonal tile holds both triangles
  __syncthreads();
#pragma unroll
  for (int e = threadIdx.x; e < TILE2; e += 256) {
    const int r = J * TILE + (e >> 5), c = I * TILE + (e & 31);
    if (r < nbf && c < nbf) M[(int64_t)r * nbf + c] = tl[e & 31][e >> 5];
  }
}

// How the two passes over B are cut.  Both stream B.  The gamma pass wants eight
// workgroups per CU (nbf = 1200, naux = 3600: 900 workgroups 4.25 ms, 2700
// 4.08 ms); the J pass is best with about three per CU, as more of them work on
// ranges of B far apart (the same system, J in 1 and 3 parts: 3.7 and 4.07 ms).
// A part of gamma has at least four tiles (four trips of its loop), a part of J
// at least 32 Q, and the parts of J stay within 32 MB, so that their traffic is
// small against B's.  Measured, gamma + J in one part each and cut: nbf = 192,
// naux = 848: 78 + 320 and 29 + 24 us; 730 / 3106: 1.42 + 1.89 and 1.40 + 1.20 ms.
// The scratch is reserved for every tile kept.  Rounding the parts to whole tiles and
// functions is not monotone (36 tiles in 7 parts become 6, 33 stay 7), so with fewer
// tiles the parts are limited by the rounded plan of all tiles: no more parts of
// gamma than it has, and no more parts of J than its scratch holds of the kept
// tiles.  Rounding only ever lowers the number of parts asked for.
static JPlan j_cut(int naux, int64_t ncols, int tiles, int64_t sg_most, int64_t sb_most) {
  auto cut = [](int64_t want, int64_t have, int64_t most) {
    return (int)std::max<int64_t>(1, std::min<int64_t>((want + have - 1) / have, most));
  };
  JPlan p{};
  p.sg = cut(2048, (naux + JG_Q - 1) / JG_Q, std::min<int64_t>(tiles / 4, sg_most));
  p.tchunk = (tiles + p.sg - 1) / p.sg;
  p.sg = (tiles + p.tchunk - 1) / p.tchunk;
  const int64_t most = std::min<int64_t>(naux / 32, ((int64_t)4 << 20) / ncols);
  p.sb = cut(768, tiles, std::min(most, sb_most));
  p.qchunk = (naux + p.sb - 1) / p.sb;
  p.sb = (naux + p.qchunk - 1) / p.qchunk;
  return p;
}
JPlan j_plan(int naux, int64_t ncols, int kept) {
  const int all = (int)(ncols / TILE2), tiles = std::max(1, kept);
  const JPlan full = j_cut(naux, ncols, all, all, naux);
  return tiles == all ? full : j_cut(naux, ncols, tiles, full.sg, (int64_t)full.sb * all / tiles);
}

static int64_t even4(int64_t n) { return (n + 3) & ~(int64_t)3; }

// packed density (ncols) and the parts of gamma (sg naux)
int64_t j_gamma_reach(const JPlan& p, int naux, int64_t ncols) { return ncols + (int64_t)p.sg * naux; }
// the same and the parts of the kept tiles of J (sb kept TILE2)
int64_t j_build_reach(const JPlan& p, int naux, int64_t ncols, int kept) {
  return ncols + even4((int64_t)p.sg * naux) + (int64_t)p.sb * kept * TILE2;
}

// with every tile kept, which no other set reaches beyond (j_plan)
size_t j_work_bytes(int nbf, int naux, int64_t ncols) {
  const int all = (int)(ncols / TILE2);
  return sizeof(double) * (size_t)j_build_reach(j_plan(naux, ncols, all), naux, ncols, all);
}

size_t j_gamma_work_bytes(int nbf, int naux, int64_t ncols) {
  return sizeof(double) * (size_t)j_gamma_reach(j_plan(naux, ncols, (int)(ncols / TILE2)), naux, ncols);
}

static bool all_kept(const JKArgs& a) { return (int64_t)a.nt_kept * TILE2 == a.ncols; }

static void pack_density(const JKArgs& a, const double* D, double* d, hipStream_t st) {
  hipLaunchKernelGGL(all_kept(a) ? pack_density_kernel<true> : pack_density_kernel<false>,
                     dim3((unsigned)(a.ncols / TILE2)), dim3(256), 0, st, D, a.nbf, a.tpos, d);
}

// both words of B in every precision: J is bandwidth-bound, and with the hi
// word alone its error (amplified by the conditioning of the metric) exceeds
// that of a reduced-precision K
static void launch_gamma(const JKArgs& a, const JPlan& p, const double* dvec, double* gp, hipStream_t st) {
  hipLaunchKernelGGL(all_kept(a) ? j_gamma_kernel<true> : j_gamma_kernel<false>,
                     dim3((a.naux + JG_Q - 1) / JG_Q, p.sg), dim3(256), 0, st, a.hi, a.lo, a.ncols, a.naux, dvec,
                     a.tiles, a.nt_kept, p.tchunk, a.tpos, gp);
}

// the launches below write up to the plan's reach and no further
static void check_reach(const char* what, int64_t reach, size_t work_bytes) {
  if (sizeof(double) * (size_t)reach > work_bytes)
    throw Error(DFX_ENOMEM, std::string(what) + ": needs " + std::to_string(sizeof(double) * (size_t)reach) +
                                " bytes of scratch, " + std::to_string(work_bytes) + " passed in");
}

void j_gamma(const JKArgs& a, const double* D, double* gam, double* work, size_t work_bytes, hipStream_t st) {
  const JPlan p = j_plan(a.naux, a.ncols, a.nt_kept);
  check_reach("j_gamma", j_gamma_reach(p, a.naux, a.ncols), work_bytes);
  double* gp = work + a.ncols;
  pack_density(a, D, work, st);
  launch_gamma(a, p, work, gp, st);
  hipLaunchKernelGGL(j_gamma_sum_kernel, dim3((a.naux + 255) / 256), dim3(256), 0, st, gp, p.sg, a.naux, gam);
}

static JPlan j_checked_plan(const JKArgs& a, size_t work_bytes) {
  const JPlan p = j_plan(a.naux, a.ncols, a.nt_kept);
  check_reach("j_build", j_build_reach(p, a.naux, a.ncols, a.nt_kept), work_bytes);
  return p;
}

static void j_build_packed(const JKArgs& a, const JPlan& p, double* J, double* work, hipStream_t st) {
  const unsigned tiles = (unsigned)(a.ncols / TILE2);
  double* gp = work + a.ncols;
  double* jp = gp + even4((int64_t)p.sg * a.naux);
  launch_gamma(a, p, work, gp, st);
  if (a.nt_kept)
    hipLaunchKernelGGL(j_back_kernel, dim3(a.nt_kept, p.sb), dim3(256), 0, st, a.hi, a.lo, a.ncols, a.naux, a.tiles,
                       gp, p.sg, p.qchunk, jp);
  hipLaunchKernelGGL(all_kept(a) ? j_unpack_kernel<true> : j_unpack_kernel<false>, dim3(tiles), dim3(256), 0, st, jp,
                     a.tpos, a.nt_kept, p.sb, a.nbf, gp, p.sg * a.naux, J);
}

void j_build(const JKArgs& a, const double* D, double* J, double* work, size_t work_bytes, hipStream_t st) {
  const JPlan p = j_checked_plan(a, work_bytes);
  pack_density(a, D, work, st);
  j_build_packed(a, p, J, work, st);
}

void j_build_cocc(const JKArgs& a, const double* C, int nocc, double* J, double* work, size_t work_bytes,
                  hipStream_t st) {
  const JPlan p = j_checked_plan(a, work_bytes);
  hipLaunchKernelGGL(all_kept(a) ? pack_cocc_kernel<true> : pack_cocc_kernel<false>, dim3((unsigned)(a.ncols / TILE2)),
                     dim3(256), 0, st, C, a.nbf, nocc, a.tpos, work);
  j_build_packed(a, p, J, work, st);
}

// ---------------------------------------------------------------------------
// K: FP64 in jk_f64.hip, FP32 / BF16 in jk_mixed.hip
size_t k_work_bytes(const JKArgs& a, int nocc) {
  return a.prec == PREC_FP64 ? k_work_bytes_f64(a, nocc) : k_work_bytes_mixed(a, nocc);
}

void k_check_work(size_t need, size_t work_bytes) {
  if (need > work_bytes)
    throw Error(DFX_ENOMEM, "k_build: needs " + std::to_string(need) + " bytes of scratch, " +
                                std::to_string(work_bytes) + " passed in");
}

size_t k_density_work_bytes(const JKArgs& a, size_t npos, size_t nneg) {
  size_t most = 0;
  for (size_t n : {npos, nneg}) {
    if (n >= (size_t)KD_CH) most = std::max(most, k_work_bytes(a, KD_CH));
    if (n % KD_CH) most = std::max(most, k_work_bytes(a, (int)(n % KD_CH)));
  }
  return most;
}

void k_build(const JKArgs& a, const double* C, int nocc, double* K, void* work, size_t work_bytes, hipStream_t st,
             KTimer* timer) {
  if (a.prec == PREC_FP64)
    k_build_f64(a, C, nocc, K, work, work_bytes, st, timer);
  else
    k_build_mixed(a, C, nocc, K, work, work_bytes, st, timer);
}

// ---------------------------------------------------------------------------
// canonical packed export: out[q - q0][c] = B[q][toff[c]] (hi + lo), or raw[q][toff[c]]
__global__ void export_kernel(const float* __restrict__ hi, const float* __restrict__ lo,
                              const double* __restrict__ raw, int64_t ld,
                              const int64_t* __restrict__ toff, int64_t ncols_p, int q0,
                              double* __restrict__ out) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= ncols_p) return;
  const int q = q0 + blockIdx.y;
  // toff[c]: the tile offset of canonical column c in B's rows, or its raw column
  out[(int64_t)blockIdx.y * ncols_p + c] =
      raw ? raw[(int64_t)q * ld + toff[c]]
          : (double)hi[(int64_t)q * ld + toff[c]] + (lo ? (double)lo[(int64_t)q * ld + toff[c]] : 0.0);
}

// out[q - q0][mu][nu] = B_q (mu, nu) = hi + lo at the packed tile position
__global__ void unpack_rows_kernel(const float* __restrict__ hi, const float* __restrict__ lo, int64_t ncols_t,
                                   int nbf, int q0, double* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t n2 = (int64_t)nbf * nbf;
  if (i >= n2) return;
  const int mu = (int)(i / nbf), nu = (int)(i % nbf);
  const int r = mu > nu ? mu : nu, c = mu > nu ? nu : mu;
  const int64_t o = (int64_t)(q0 + blockIdx.y) * ncols_t + tile_base(r >> 5, c >> 5) + ((r & 31) << 5) + (c & 31);
  out[(int64_t)blockIdx.y * n2 + i] = (double)hi[o] + (double)lo[o];
}

void unpack_rows(const float* hi, const float* lo, int64_t ncols_t, int nbf, int q0, int q1, double* out,
                 hipStream_t st) {
  if (q1 <= q0) return;
  const int64_t n2 = (int64_t)nbf * nbf;
  const dim3 g((unsigned)((n2 + 255) / 256), q1 - q0);
  hipLaunchKernelGGL(unpack_rows_kernel, g, dim3(256), 0, st, hi, lo, ncols_t, nbf, q0, out);
}

void export_rows(const float* hi, const float* lo, const double* raw, int64_t ld, int q0, int q1,
                 const int64_t* toff, int64_t ncols_p, double* out, hipStream_t st) {
  if (q1 <= q0 || ncols_p <= 0) return;
  const dim3 g((unsigned)((ncols_p + 255) / 256), q1 - q0);
  hipLaunchKernelGGL(export_kernel, g, dim3(256), 0, st, hi, lo, raw, ld, toff, ncols_p, q0, out);
}

}  // namespace dfx
