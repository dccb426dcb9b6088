// FP32 multilayer perceptron on gfx950 for the learned starting guess:
// Linear -> SiLU -> ... -> Linear, mean-squared-error loss, hand-written
// backward pass and Adam.  Parameters theta are one flat array: for each layer
// W (out x in, row-major) then b (out).
#include <cmath>

#include "host.h"
#include "mlp.h"

namespace dfx {

// ---- products on FP32 matrix cores (v_mfma_f32_16x16x4f32: FP32 products and sums) ----
// A workgroup owns a T x T tile of the result, T = 16, 32 or 64; its eight waves (one
// for long batches of narrow layers, forward_one_wave) take blocks of 16 k in turn,
// operands straight from memory to registers (two to four blocks in flight), and
// their sums are added in LDS in a fixed order.
// MFMA operands: lane (li, lk) = (lane % 16, lane / 16) gives A[row li][k lk] and
// B[k lk][col li]; the result's element r of that lane is C[row 4 lk + r][col li].
// Within a block of 16 the lane has k = 4 lk .. 4 lk + 3, one MFMA each.
// What bounds it: launches and the latency of a tile's loads, since a minibatch
// has few tiles (128 x 256: 32 of 32 x 32).  So what follows a product is in its
// epilogue: bias and SiLU, the loss and its gradient, the factor SiLU'(Z); the
// bias gradient is summed from the operands of the weight gradient, and both
// products that read a layer's gradient are one launch.  Training step of 454 x
// 256^3 x 70, batch 128: 435 us with 64 x 64 tiles through LDS and all of these
// launches apart, 100 so.
constexpr int MW = 8, MT = 64 * MW;  // waves and threads of a workgroup
// results per thread of a workgroup of NW waves on a tile of 16 F
constexpr int mlp_nout(int F, int NW) { return (256 * F * F + 64 * NW - 1) / (64 * NW); }
typedef float v4f __attribute__((ext_vector_type(4)));

typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

// x(row, k) = KC ? p[row ld + k] : p[k ld + row], n rows
struct MatOp {
  const float* p;
  int64_t ld;
  int n;
};

// the 16 F rows from x0 of an operand as a wave reads them: blocks of 16 k, NW apart
template <bool KC, int F, int NW>
struct TileOp {
  const float* p;  // x0 and the wave's first block (wave-uniform)
  int64_t ld;
  int64_t vo[F];   // the lane's k = 4 lk of its row in fragment f
  __device__ __forceinline__ void init(const MatOp& m, int x0, int w, int li, int lk) {
    ld = m.ld;
    p = KC ? m.p + x0 * ld + 16 * w : m.p + 16 * w * ld + x0;
#pragma unroll
    for (int f = 0; f < F; ++f) {
      const int r = min(16 * f + li, m.n - 1 - x0);  // rows past the end: not stored
      vo[f] = KC ? r * ld + 4 * lk : 4 * lk * ld + r;
    }
  }
  __device__ __forceinline__ void load(int64_t i, float (&v)[F][4]) const {
    const float* q = p + i * (KC ? 16 * NW : 16 * NW * ld);
#pragma unroll
    for (int f = 0; f < F; ++f) {
      if (KC) {
        const f4u x = *reinterpret_cast<const f4u*>(q + vo[f]);
#pragma unroll
        for (int t = 0; t < 4; ++t) v[f][t] = x[t];
      } else {
#pragma unroll
        for (int t = 0; t < 4; ++t) v[f][t] = q[vo[f] + t * ld];
      }
    }
  }
  // the last block, of which k < kr exist
  __device__ __forceinline__ void load_tail(int64_t i, int kr, int lk, float (&v)[F][4]) const {
    const float* q = p + i * (KC ? 16 * NW : 16 * NW * ld);
#pragma unroll
    for (int f = 0; f < F; ++f)
#pragma unroll
      for (int t = 0; t < 4; ++t) v[f][t] = 4 * lk + t < kr ? q[vo[f] + (KC ? t : t * ld)] : 0.0f;
  }
};

// element e of a tile, as its partial sums lie in LDS: fragment, register, lane
template <int F>
__device__ __forceinline__ int tile_row(int e) { return (e >> 8) / F * 16 + 4 * ((e & 63) >> 4) + ((e >> 6) & 3); }
template <int F>
__device__ __forceinline__ int tile_col(int e) { return (e >> 8) % F * 16 + (e & 15); }

// The tile's product over k < K: element e = threadIdx.x + 64 NW h < 256 F^2 in out[h].
// rsum (ROWSUM): the sums of A's 16 F rows over k, in threads 0 .. 16 F - 1.
template <bool KA, bool KB, int F, bool ROWSUM, int NW>
__device__ __forceinline__ void tile_gemm(const MatOp& A, const MatOp& B, int m0, int n0, int K, float* red,
                                          float (&out)[mlp_nout(F, NW)], float& rsum) {
  constexpr int MW = NW, MT = 64 * NW;
  constexpr int D = F == 4 ? 2 : 4;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lk = lane >> 4;
  v4f acc[F][F];
  float rs[F];
#pragma unroll
  for (int i = 0; i < F; ++i) {
    rs[i] = 0.0f;
#pragma unroll
    for (int j = 0; j < F; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
  }
  float a[D][F][4], b[D][F][4];
  TileOp<KA, F, NW> oa;
  TileOp<KB, F, NW> ob;
  oa.init(A, m0, w, li, lk);
  ob.init(B, n0, w, li, lk);
  auto step = [&](const float (&x)[F][4], const float (&y)[F][4]) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int i = 0; i < F; ++i) {
        if (ROWSUM) rs[i] += x[i][t];
#pragma unroll
        for (int j = 0; j < F; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[i][t], y[j][t], acc[i][j], 0, 0, 0);
      }
  };
  const int full = K >> 4, kr = K & 15;
  const int nb = full > w ? (full - w + MW - 1) / MW : 0;  // whole blocks of this wave
  if (nb > 0) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      oa.load(min(d, nb - 1), a[d]);
      ob.load(min(d, nb - 1), b[d]);
    }
    int i = 0;
    for (; i + D <= nb; i += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        step(a[d], b[d]);
        // past the end: the last block again, not used
        oa.load(min(i + D + d, nb - 1), a[d]);
        ob.load(min(i + D + d, nb - 1), b[d]);
      }
    }
#pragma unroll
    for (int d = 0; d < D - 1; ++d)
      if (i + d < nb) step(a[d], b[d]);
  }
  if (kr && full % MW == w) {
    oa.load_tail(nb, kr, lk, a[0]);
    ob.load_tail(nb, kr, lk, b[0]);
    step(a[0], b[0]);
  }
  // in chunks of RX fragment rows, EC elements
  constexpr int RX = F == 4 ? 1 : F, EC = 256 * F * RX, HC = (EC + MT - 1) / MT;
#pragma unroll
  for (int q = 0; q < F / RX; ++q) {
    if (q) __syncthreads();
#pragma unroll
    for (int x = 0; x < RX; ++x)
#pragma unroll
      for (int y = 0; y < F; ++y)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[w * EC + ((x * F + y) * 4 + r) * 64 + lane] = acc[q * RX + x][y][r];
    __syncthreads();
#pragma unroll
    for (int h = 0; h < HC; ++h) {
      const int e = threadIdx.x + MT * h;
      float s = 0.0f;
      if (e < EC) {
        s = red[e];
#pragma unroll
        for (int x = 1; x < MW; ++x) s += red[x * EC + e];
      }
      out[q * HC + h] = s;
    }
  }
  if (ROWSUM) {
    __syncthreads();
#pragma unroll
    for (int x = 0; x < F; ++x) {
      float s = rs[x] + __shfl_xor(rs[x], 16);
      s += __shfl_xor(s, 32);
      if (lk == 0) red[w * 16 * F + x * 16 + li] = s;
    }
    __syncthreads();
    rsum = 0.0f;
    if (threadIdx.x < 16 * F)
      for (int x = 0; x < MW; ++x) rsum += red[x * 16 * F + threadIdx.x];
  }
}

// Layer forward: z = a W^T + b.  hidden: Z = z, out = silu(z).  Otherwise out = z, or
// with T the loss: out = 2 (z - T) / n over all n = rows x cols outputs, and the
// workgroup's sum of (z - T)^2 to part.
template <int F, int NW>
__global__ void __launch_bounds__(64 * NW) layer_forward_kernel(int rows, int cols, int K, const float* __restrict__ a,
                                                                const float* __restrict__ W,
                                                                const float* __restrict__ bias, int hidden,
                                                                float* __restrict__ Z, float* __restrict__ out,
                                                                const float* __restrict__ T,
                                                                double* __restrict__ part) {
  __shared__ __attribute__((aligned(16))) float red[NW * 256 * F * (F == 4 ? 1 : F)];
  const int nt = (cols + 16 * F - 1) / (16 * F);
  const int m0 = blockIdx.x / nt * 16 * F, n0 = blockIdx.x % nt * 16 * F;
  float v[mlp_nout(F, NW)], rsum;
  tile_gemm<true, true, F, false, NW>(MatOp{a, K, rows}, MatOp{W, K, cols}, m0, n0, K, red, v, rsum);
  double s = 0.0;
#pragma unroll
  for (int h = 0; h < mlp_nout(F, NW); ++h) {
    const int e = threadIdx.x + 64 * NW * h, r = m0 + tile_row<F>(e), c = n0 + tile_col<F>(e);
    if (e >= 256 * F * F || r >= rows || c >= cols) continue;
    const int64_t i = (int64_t)r * cols + c;
    const float z = v[h] + bias[c];
    if (hidden) {
      Z[i] = z;
      out[i] = z / (1.0f + expf(-z));
    } else if (T) {
      const float d = z - T[i];
      out[i] = 2.0f * d / (float)((int64_t)rows * cols);
      s += (double)d * d;
    } else {
      out[i] = z;
    }
  }
  if (!T) return;
  double* ws = reinterpret_cast<double*>(red);
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    s = 0.0;
    for (int x = 0; x < NW; ++x) s += ws[x];
    part[blockIdx.x] = s;
  }
}

// Layer backward from G = dL/dz (rows x no): workgroups below nda the tiles of
// (G W) silu'(Zin) (rows x ni, the layer before), the others those of dW = G^T a, of
// which the first column of tiles also leaves db.
template <int F>
__global__ void __launch_bounds__(MT) layer_backward_kernel(int rows, int no, int ni, int nda,
                                                            const float* __restrict__ G, const float* __restrict__ W,
                                                            const float* __restrict__ Zin,
                                                            const float* __restrict__ a, float* __restrict__ Gin,
                                                            float* __restrict__ dW, float* __restrict__ db) {
  __shared__ __attribute__((aligned(16))) float red[MW * 256 * F * (F == 4 ? 1 : F)];
  const int nt = (ni + 16 * F - 1) / (16 * F);
  const bool da = (int)blockIdx.x < nda;
  const int t = da ? blockIdx.x : blockIdx.x - nda;
  const int m0 = t / nt * 16 * F, n0 = t % nt * 16 * F;
  float v[mlp_nout(F, MW)], rsum;
  if (da)
    tile_gemm<true, false, F, false, MW>(MatOp{G, no, rows}, MatOp{W, ni, ni}, m0, n0, no, red, v, rsum);
  else
    tile_gemm<false, false, F, true, MW>(MatOp{G, no, no}, MatOp{a, ni, ni}, m0, n0, rows, red, v, rsum);
#pragma unroll
  for (int h = 0; h < mlp_nout(F, MW); ++h) {
    const int e = threadIdx.x + MT * h, r = m0 + tile_row<F>(e), c = n0 + tile_col<F>(e);
    if (e >= 256 * F * F || r >= (da ? rows : no) || c >= ni) continue;
    const int64_t i = (int64_t)r * ni + c;
    if (da) {
      const float z = Zin[i];
      const float s = 1.0f / (1.0f + expf(-z));
      Gin[i] = v[h] * (s * (1.0f + z * (1.0f - s)));
    } else {
      dW[i] = v[h];
    }
  }
  if (!da && n0 == 0 && threadIdx.x < 16 * F && m0 + (int)threadIdx.x < no) db[m0 + threadIdx.x] = rsum;
}

static int tiles_of(int64_t m, int64_t n, int F) { return (int)(((m + 16 * F - 1) / (16 * F)) * ((n + 16 * F - 1) / (16 * F))); }

// 16 F is the tile of a launch with so many tiles of 16: small ones while the chip is
// not full, larger ones, which read their operands less often, beyond.  Loss and
// gradient with all launches in tiles of 16 / 32 / 64, us: 454 x 256^3 x 70, batch 128
// (128 tiles) 100 / 117 / 159; 454 x 512^2 x 70, batch 1024 (2048) 188 / 157 / 208;
// 1024^3 x 256, batch 1024 (4096) 454 / 320 / 290; batch 4096 1841 / 1236 / 1023.
static int tile_frags(int64_t tiles16) { return tiles16 >= 4096 ? 4 : tiles16 > 1024 ? 2 : 1; }

// A long batch through a narrow layer has tiles enough for single waves: over a short K
// (some eight blocks of 16) most of the eight waves of a workgroup have nothing to do
// but to wait for the sum, and tiles of 64 are mostly padding where there are few
// columns.  One wave a tile of 16 or 32 then.  Forward pass, batch 100000, us, eight
// waves and 64 x 64 / one wave (64 x 64 through LDS before either): 4-4-4 100 / 49
// (68), 16-16-16 96 / 55 (82), 32-32-32 387 / 335 (379), 64-16-64 370 / 328 (360).
// From K = 256 and 64 columns on neither is ahead (256^3, batch 5000: 108 / 90, 454 x
// 256 x 70, batch 100000: 940 / 949).
static bool forward_one_wave(int64_t tiles16, int K, int cols) { return tiles16 >= 4096 && (K <= 128 || cols <= 32); }

__global__ void adam_kernel(float* theta, const float* __restrict__ g, float* m, float* v, int64_t n, float lr,
                            float b1, float b2, float eps, float c1, float c2) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.0f - b1) * gi;
  const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  theta[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// out[r][:] = src[idx[r]][:]
__global__ void gather_rows_kernel(const float* __restrict__ src, const int* __restrict__ idx, int rows, int cols,
                                   float* out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)rows * cols) return;
  const int r = (int)(i / cols), c = (int)(i % cols);
  out[i] = src[(int64_t)idx[r] * cols + c];
}

static unsigned nb(int64_t n) { return (unsigned)((n + 255) / 256); }

int64_t mlp_nparams(const std::vector<int>& w) {
  int64_t n = 0;
  for (size_t i = 0; i + 1 < w.size(); ++i) n += (int64_t)w[i] * w[i + 1] + w[i + 1];
  return n;
}

size_t mlp_work_floats(const std::vector<int>& w, int batch) {
  size_t s = 0;
  for (size_t i = 1; i < w.size(); ++i) s += 2 * (size_t)batch * w[i];  // Z and A per layer
  int mx = 0;
  for (int x : w) mx = std::max(mx, x);
  return s + 2 * (size_t)batch * mx + 1024;                           // two gradient buffers + partials
}

// Network on X: Z and A of every hidden layer kept in work for the backward pass.
// out: the outputs, or with T the gradient of the loss in them, and the loss's
// partial sums (their number returned) in part
static int forward_impl(const std::vector<int>& w, const float* theta, const float* X, int batch, float* work,
                        float* out, const float* T, double* part, hipStream_t st) {
  const int nl = (int)w.size() - 1;
  const float* a = X;
  const float* p = theta;
  float* wp = work;
  int tiles = 0;
  for (int l = 0; l < nl; ++l) {
    const int ni = w[l], no = w[l + 1], hidden = l < nl - 1 ? 1 : 0;
    float* Z = wp;
    float* A = hidden ? wp + (size_t)batch * no : out;
    wp += 2 * (size_t)batch * no;
    const float* b = p + (size_t)ni * no;
    const float* Tl = hidden ? nullptr : T;
    const int64_t tiles16 = tiles_of(batch, no, 1);
    const bool one = forward_one_wave(tiles16, ni, no);
    const int F = one ? (no <= 16 ? 1 : 2) : tile_frags(tiles16);
    tiles = tiles_of(batch, no, F);
    auto* kern = F == 4   ? layer_forward_kernel<4, MW>
                 : F == 2 ? (one ? layer_forward_kernel<2, 1> : layer_forward_kernel<2, MW>)
                          : (one ? layer_forward_kernel<1, 1> : layer_forward_kernel<1, MW>);
    hipLaunchKernelGGL(kern, dim3(tiles), dim3(one ? 64 : MT), 0, st, batch, no, ni, a, p, b, hidden, Z, A, Tl, part);
    p += (size_t)ni * no + no;
    a = A;
  }
  return tiles;
}

void mlp_forward(const std::vector<int>& w, const float* theta, const float* X, int batch, float* Y, float* work,
                 hipStream_t st) {
  // a single layer reads X while it writes: Y may lie in X
  float* out = w.size() == 2 ? work : Y;
  forward_impl(w, theta, X, batch, work, out, nullptr, nullptr, st);
  if (out != Y)
    DFX_HIP(hipMemcpyAsync(Y, out, sizeof(float) * (size_t)batch * w.back(), hipMemcpyDeviceToDevice, st));
}

// acc[0] += sum of the partial sums / n  (one wave, fixed order)
__global__ void __launch_bounds__(64) loss_accumulate_kernel(const double* __restrict__ part, int np, int64_t n,
                                                             double* acc) {
  double s = 0.0;
  for (int i = threadIdx.x; i < np; i += 64) s += part[i];
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if (threadIdx.x == 0) acc[0] += s / (double)n;
}

struct LossParts {
  const double* p;
  int np;
  int64_t nout;
};

static LossParts loss_grad_impl(const std::vector<int>& w, const float* theta, const float* X, const float* T, int batch,
                                float* grad, float* work, hipStream_t st) {
  const int nl = (int)w.size() - 1;
  size_t act = 0;
  for (int l = 1; l <= nl; ++l) act += 2 * (size_t)batch * w[l];
  int mx = 0;
  for (int x : w) mx = std::max(mx, x);
  float* G = work + act;
  float* G2 = G + (size_t)batch * mx;
  // the loss's partial sums: behind the gradients up to 511 of them, else in the
  // output layer's place for Z, which has more than 8 floats for each
  size_t po = act + 2 * (size_t)batch * mx;
  if (tiles_of(batch, w[nl], 1) > 511) po = act - 2 * (size_t)batch * w[nl];
  double* part = reinterpret_cast<double*>(work + ((po + 1) & ~(size_t)1));
  const int np = forward_impl(w, theta, X, batch, work, G, T, part, st);
  // parameter offsets
  std::vector<size_t> off(nl);
  size_t o = 0;
  for (int l = 0; l < nl; ++l) {
    off[l] = o;
    o += (size_t)w[l] * w[l + 1] + w[l + 1];
  }
  // layer activations: Z_l at zofs[l], A_l at zofs[l] + batch * w[l+1]
  std::vector<size_t> zofs(nl);
  size_t zo = 0;
  for (int l = 0; l < nl; ++l) {
    zofs[l] = zo;
    zo += 2 * (size_t)batch * w[l + 1];
  }
  for (int l = nl - 1; l >= 0; --l) {
    const int ni = w[l], no = w[l + 1];
    const float* zin = l == 0 ? nullptr : work + zofs[l - 1];
    const float* a_in = l == 0 ? X : zin + (size_t)batch * ni;
    float *dW = grad + off[l], *db = dW + (size_t)ni * no;
    const float* W = theta + off[l];
    int F = tile_frags(tiles_of(no, ni, 1) + (l ? tiles_of(batch, ni, 1) : 0));
    // a long batch over few tiles of dW: smaller ones (300^3 x 30, batch 20000: 1985
    // us in tiles of 64, 1150 of 16)
    while (F > 1 && batch > no && tiles_of(no, ni, F) < 128) F /= 2;
    const int nda = l ? tiles_of(batch, ni, F) : 0, grid = nda + tiles_of(no, ni, F);
    hipLaunchKernelGGL(F == 4 ? layer_backward_kernel<4> : F == 2 ? layer_backward_kernel<2> : layer_backward_kernel<1>,
                       dim3(grid), dim3(MT), 0, st, batch, no, ni, nda, G, W, zin, a_in, G2, dW, db);
    std::swap(G, G2);
  }
  return LossParts{part, np, (int64_t)batch * w[nl]};
}

double mlp_loss_grad(const std::vector<int>& w, const float* theta, const float* X, const float* T, int batch,
                     float* grad, float* work, hipStream_t st) {
  const LossParts p = loss_grad_impl(w, theta, X, T, batch, grad, work, st);
  std::vector<double> hp(p.np);
  DFX_HIP(hipMemcpyAsync(hp.data(), p.p, sizeof(double) * p.np, hipMemcpyDeviceToHost, st));
  DFX_HIP(hipStreamSynchronize(st));
  double s = 0.0;
  for (double v : hp) s += v;
  return s / (double)p.nout;
}

void mlp_loss_grad_acc(const std::vector<int>& w, const float* theta, const float* X, const float* T, int batch,
                       float* grad, float* work, double* loss_acc, hipStream_t st) {
  const LossParts p = loss_grad_impl(w, theta, X, T, batch, grad, work, st);
  hipLaunchKernelGGL(loss_accumulate_kernel, dim3(1), dim3(64), 0, st, p.p, p.np, p.nout, loss_acc);
}

void mlp_adam(float* theta, const float* grad, float* m, float* v, int64_t n, int step, float lr, hipStream_t st) {
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  const float c1 = 1.0f - powf(b1, (float)step), c2 = 1.0f - powf(b2, (float)step);
  hipLaunchKernelGGL(adam_kernel, dim3(nb(n)), dim3(256), 0, st, theta, grad, m, v, n, lr, b1, b2, eps, c1, c2);
}

void gather_rows(const float* src, const int* idx, int rows, int cols, float* out, hipStream_t st) {
  hipLaunchKernelGGL(gather_rows_kernel, dim3(nb((int64_t)rows * cols)), dim3(256), 0, st, src, idx, rows, cols, out);
}

}  // namespace dfx

using namespace dfx;

extern "C" {

int dfx_mlp_forward(const int32_t* widths, int nlayers, const float* theta, const float* X, int batch, float* Y,
                    void* stream) {
  return guard([&] {
    if (!widths || nlayers < 1 || !theta || !X || !Y || batch <= 0) throw Error(DFX_EINVAL, "dfx_mlp_forward: bad argument");
    std::vector<int> w(widths, widths + nlayers + 1);
    DevMem work(sizeof(float) * mlp_work_floats(w, batch));
    mlp_forward(w, theta, X, batch, Y, work.as<float>(), (hipStream_t)stream);
    DFX_HIP(hipStreamSynchronize((hipStream_t)stream));
  });
}

int dfx_mlp_loss_grad(const int32_t* widths, int nlayers, const float* theta, const float* X, const float* T, int batch,
                      float* grad, double* loss, void* stream) {
  return guard([&] {
    if (!widths || nlayers < 1 || !theta || !X || !T || !grad || batch <= 0)
      throw Error(DFX_EINVAL, "dfx_mlp_loss_grad: bad argument");
    std::vector<int> w(widths, widths + nlayers + 1);
    DevMem work(sizeof(float) * mlp_work_floats(w, batch));
    const double L = mlp_loss_grad(w, theta, X, T, batch, grad, work.as<float>(), (hipStream_t)stream);
    if (loss) *loss = L;
  });
}

int dfx_mlp_adam(float* theta, const float* grad, float* m, float* v, int64_t n, int step, float lr, void* stream) {
  return guard([&] {
    if (!theta || !grad || !m || !v || n <= 0 || step < 1) throw Error(DFX_EINVAL, "dfx_mlp_adam: bad argument");
    mlp_adam(theta, grad, m, v, n, step, lr, (hipStream_t)stream);
  });
}

}  // extern "C"
