// FP64 products of a few hundred rows and columns: 32 x 32 tiles, the k-range
// split over the waves of a workgroup, operands straight to registers.
#pragma once
#include "common.h"

namespace dfx {

typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int SG_T = 32, SG_W = 8;  // tile, waves of a workgroup (512 threads)

// One operand's 32 rows (or columns) from x0: KC: k is contiguous (A, or B
// transposed), else rows of k.  A wave takes blocks of 8 k, SG_W blocks apart;
// lane (li, lk) = (lane % 16, lane / 16) holds k = 2 lk and 2 lk + 1 of rows li and
// li + 16, whatever the alignment.  Rows past the end read the last one, whose
// products are not stored.
template <bool KC>
struct RegOp {
  const char* p;      // the operand at x0 and the wave's first block (wave-uniform)
  int64_t step;       // bytes from one block of the wave to its next
  uint32_t vo[2], dk; // byte offsets of the lane, and of its second k
  __device__ __forceinline__ void init(const double* P, int64_t ld, int x0, int x, int w, int li, int lk) {
    p = reinterpret_cast<const char*>(KC ? P + (int64_t)x0 * ld + 8 * w : P + (int64_t)(8 * w) * ld + x0);
    step = KC ? 8 * SG_W * 8 : (int64_t)8 * SG_W * 8 * ld;
    dk = KC ? 8u : (uint32_t)ld * 8u;
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      const uint32_t r = (uint32_t)min(16 * f + li, x - 1 - x0);
      vo[f] = KC ? (r * (uint32_t)ld + 2u * lk) * 8u : (2u * lk * (uint32_t)ld + r) * 8u;
    }
  }
  __device__ __forceinline__ void load(int64_t blk, double (&v)[2][2]) const {
    const char* q = p + blk * step;
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int t = 0; t < 2; ++t) v[f][t] = *reinterpret_cast<const double*>(q + vo[f] + t * dk);
  }
  // the last, partial block: kr < 8 of its k exist
  __device__ __forceinline__ void load_tail(int64_t blk, int kr, int lk, double (&v)[2][2]) const {
    const char* q = p + blk * step;
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int t = 0; t < 2; ++t)
        v[f][t] = 2 * lk + t < kr ? *reinterpret_cast<const double*>(q + vo[f] + t * dk) : 0.0;
  }
};

// (row, column) in the tile of element e of the layout of the partial sums
__device__ __forceinline__ int sg_row(int e) { return (e >> 9) * 16 + ((e >> 6) & 3) * 4 + ((e & 63) >> 4); }
__device__ __forceinline__ int sg_col(int e) { return ((e >> 8) & 1) * 16 + (e & 15); }

// The tile's product over k < K.  red: SG_W * 1024 doubles of LDS.  Thread t gets
// the elements e = t and t + 512 of the tile in out, at sg_row(e), sg_col(e); the
// waves' sums are added in order.
// What bounds it: the latency of the loads for small K (four blocks of every wave
// are in flight), the matrix cores beyond.  The tiles of the general product run
// their whole k-range in one workgroup, on 9 of 256 CUs at 192 x 192.
template <bool KCA, bool KCB>
__device__ __forceinline__ void small_gemm(const RegOp<KCA>& A, const RegOp<KCB>& B, int K, int w, int lane,
                                           double* red, double (&out)[2]) {
  constexpr int D = 4;
  const int lk = lane >> 4;
  v4d acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
  auto mfma = [&](const double (&a)[2][2], const double (&b)[2][2]) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i][t], b[j][t], acc[i][j], 0, 0, 0);
  };
  const int full = K >> 3, kr = K & 7;
  const int nb = full > w ? (full - w + SG_W - 1) / SG_W : 0;  // whole blocks of this wave
  double a[D][2][2], b[D][2][2];
  if (nb > 0) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      A.load(min(d, nb - 1), a[d]);
      B.load(min(d, nb - 1), b[d]);
    }
    int i = 0;
    for (; i + D <= nb; i += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        mfma(a[d], b[d]);
        // past the end: the last block again, not used
        A.load(min(i + D + d, nb - 1), a[d]);
        B.load(min(i + D + d, nb - 1), b[d]);
      }
    }
#pragma unroll
    for (int d = 0; d < D - 1; ++d)
      if (i + d < nb) mfma(a[d], b[d]);
  }
  if (kr && (full % SG_W) == w) {
    A.load_tail(nb, kr, lk, a[0]);
    B.load_tail(nb, kr, lk, b[0]);
    mfma(a[0], b[0]);
  }
  // element (row, col) of a 16 x 16 block is in lane col + 16 (row % 4), register row / 4
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[w * 1024 + ((i * 2 + j) * 4 + r) * 64 + lane] = acc[i][j][r];
  __syncthreads();
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int e = threadIdx.x + 512 * h;
    double s = red[e];
#pragma unroll
    for (int x = 1; x < SG_W; ++x) s += red[x * 1024 + e];
    out[h] = s;
  }
}

}  // namespace dfx
