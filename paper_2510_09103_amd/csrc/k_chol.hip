// fp64 Cholesky factorisation and triangular inverse of the r x r Gram matrix R R^T.
// Used after Alg. 2 when the refresh period T exceeds 1: with R R^T = C C^T the factors are
// re-expressed as (L C, C^-1 R), which keeps the product L R and makes the rows of R
// orthonormal, so that the least-squares fit of L with R held is a plain projection.
// One workgroup per low-rank block (r <= 128: the matrix stays in LDS); fp64 keeps the orthonormality error at fp32 rounding
// level whatever the conditioning of R.
// A Gram matrix that is not positive definite in fp64 (a pivot that is zero, negative or not finite: R has lost
// rank, e.g. factors that are exactly zero) has no such factorisation; the kernel then writes C = C^-1 = I, so that
// the block's (L, R) pass through the re-expression unchanged instead of turning into NaN.
#include "k_f64_common.h"

namespace adapm {

namespace {

// r above CH_MAX: in place in global memory
__device__ void chol_inv_global(double* A, double* X, int r) {
  const int tid = threadIdx.x;
  bool bad = false;
  // right-looking Cholesky, lower triangle, in place
  for (int j = 0; j < r; ++j) {
    const double piv = A[(int64_t)j * r + j];        // the same value in every thread
    if (!(piv > 0.0) || !isfinite(piv)) { bad = true; break; }
    const double d = sqrt(piv);
    __syncthreads();
    for (int i = j + tid; i < r; i += 256) A[(int64_t)i * r + j] = (i == j) ? d : A[(int64_t)i * r + j] / d;
    __syncthreads();
    const int rem = r - j - 1;                       // trailing rows j+1 .. r-1
    for (int64_t e = tid; e < (int64_t)rem * rem; e += 256) {
      const int i = j + 1 + (int)(e / rem), k = j + 1 + (int)(e % rem);
      if (k <= i) A[(int64_t)i * r + k] -= A[(int64_t)i * r + j] * A[(int64_t)k * r + j];
    }
    __syncthreads();
  }
  __syncthreads();
  if (bad) {
    for (int64_t e = tid; e < (int64_t)r * r; e += 256) A[e] = X[e] = (e / r == e % r) ? 1.0 : 0.0;
    return;
  }
  for (int64_t e = tid; e < (int64_t)r * r; e += 256) {
    const int i = (int)(e / r), k = (int)(e % r);
    if (k > i) A[e] = 0.0;
  }
  __syncthreads();
  // X = C^-1 by forward substitution, one column per thread
  for (int j = tid; j < r; j += 256) {
    for (int a = 0; a < r; ++a) {
      double s = (a == j) ? 1.0 : 0.0;
      if (a < j) { X[(int64_t)a * r + j] = 0.0; continue; }
      for (int c = j; c < a; ++c) s -= A[(int64_t)a * r + c] * X[(int64_t)c * r + j];
      X[(int64_t)a * r + j] = s / A[(int64_t)a * r + a];
    }
  }
}

constexpr int CH_MAX = 128;   // largest r factorised in LDS (every block of the MFMA path)

// The same operations in the same order with the matrix in LDS: C in the lower triangle, the strictly
// lower part of C^-1 transposed into the (otherwise unused) upper triangle, its diagonal beside it.
__global__ __launch_bounds__(256) void chol_inv_kernel(const CholItem* __restrict__ items, Bases b) {
  __shared__ double S[CH_MAX * (CH_MAX + 1)];
  __shared__ double xd[CH_MAX];
  const CholItem it = items[blockIdx.x];
  const int r = it.r, tid = threadIdx.x;
  double* A = reinterpret_cast<double*>(b.ws + it.off_gram);
  double* X = reinterpret_cast<double*>(b.ws + it.off_inv);
  if (r > CH_MAX) { chol_inv_global(A, X, r); return; }
  const int ld = r | 1;                              // odd row stride: a column walks through all banks
  for (int e = tid; e < r * r; e += 256) S[(e / r) * ld + e % r] = A[e];
  __syncthreads();
  const int tx = tid & 15, ty = tid >> 4;
  bool bad = false;
  for (int j = 0; j < r; ++j) {
    const double piv = S[j * ld + j];                // the same value in every thread
    if (!(piv > 0.0) || !isfinite(piv)) { bad = true; break; }
    const double d = sqrt(piv);
    __syncthreads();
    for (int i = j + tid; i < r; i += 256) S[i * ld + j] = (i == j) ? d : S[i * ld + j] / d;
    __syncthreads();
    for (int i = j + 1 + ty; i < r; i += 16) {
      const double lij = S[i * ld + j];
      for (int k = j + 1 + tx; k <= i; k += 16) S[i * ld + k] -= lij * S[k * ld + j];
    }
    __syncthreads();
  }
  if (bad) {                                         // uniform: every thread saw the same pivot
    for (int e = tid; e < r * r; e += 256) A[e] = X[e] = (e / r == e % r) ? 1.0 : 0.0;
    return;
  }
  // column j of C^-1 by forward substitution, one column per thread; thread j writes row j of the upper
  // triangle and xd[j] only, and reads nothing another thread writes
  if (tid < r) {
    const int j = tid;
    for (int a = j; a < r; ++a) {
      double s = (a == j) ? 1.0 : 0.0;
      for (int c = j; c < a; ++c) s -= S[a * ld + c] * (c == j ? xd[j] : S[j * ld + c]);
      const double x = s / S[a * ld + a];
      if (a == j) xd[j] = x; else S[j * ld + a] = x;
    }
  }
  __syncthreads();
  for (int e = tid; e < r * r; e += 256) {
    const int i = e / r, k = e % r;
    A[e] = k <= i ? S[i * ld + k] : 0.0;
    X[e] = k < i ? S[k * ld + i] : (k == i ? xd[i] : 0.0);
  }
}

// R <- C^-1 R on 64 whole columns, or L <- L C on 64 whole rows, in place (fp64 products on the matrix cores, fp32 stores).
// A wave owns 16 columns of R (rows of L) with all r results of each, so it overwrites nothing that another wave reads: it
// requests its whole share of the factor first, then walks the contraction in steps of 16 and takes the triangular matrix
// straight from the caches (k_f64_common.h for the lane layouts), whose 16 x 16 (L: 16 x 32) tiles outside the triangle are skipped.
// Bound by those cache reads, 66 KB per wave at r = 128, and by the fp64 rate (25 GFLOP, 0.35 ms of the table below).  Against
// 4 x 4 pieces per thread on the vector units with the matrix staged through LDS: 288 matrices of 1600 / 6400 at r = 128
// 2.38 -> 0.87 ms (1.05 with 264 registers and the accumulators in the second half of
// the file, see mfma_f64_results).
// One body per number of 16-wide steps, RG_T = ceil(r / 16), without branches between the matrix instructions: the tiles that
// are skipped are known at compile time, and no accumulator is copied on the way (see mfma_f64_results).
template <int RG_T>
__device__ __forceinline__ void regauge_body(const RegaugeItem& it, const Bases& b) {
  const int r = it.r, len = it.len;
  const int lane = threadIdx.x & 63, l16 = lane & 15, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int u0 = it.first + 16 * wave;
  if (u0 >= len) return;
  float* X = reinterpret_cast<float*>(b.state + it.off_x);
  const double* __restrict__ Cm = reinterpret_cast<const double*>(b.ws + it.off_c);
  const int u = u0 + l16, uc = u < len ? u : len - 1;     // lanes past the end repeat the last column / row and store nothing
  // x[s][v] = element k = 16 s + 4 kq + v of this lane's column of R / row of L, zero past the rank
  float x[RG_T][4];
#pragma unroll
  for (int s = 0; s < RG_T; ++s) {
#pragma unroll
    for (int v = 0; v < 4; ++v) x[s][v] = 0.f;
    const int k = 16 * s + 4 * kq;
    if (it.is_L && s + 1 < RG_T) {
      const f32x4_a4 q = *reinterpret_cast<const f32x4_a4*>(X + (int64_t)uc * r + k);
      x[s][0] = q.x; x[s][1] = q.y; x[s][2] = q.z; x[s][3] = q.w;
    } else {
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (s + 1 < RG_T || k + v < r) x[s][v] = X[it.is_L ? (int64_t)uc * r + k + v : (int64_t)(k + v) * len + uc];
    }
  }
  f64x4 acc[RG_T + 1];
#pragma unroll
  for (int t = 0; t <= RG_T; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
  if (!it.is_L) {
    // result row a = sum over k <= a of C^-1[a][k] R[k][u]
#pragma unroll
    for (int s = 0; s < RG_T; ++s) {
      const int k = 16 * s + 4 * kq;
#pragma unroll
      for (int t = s; t < RG_T; ++t) {
        const double* row = Cm + (int64_t)(16 * t + l16 < r ? 16 * t + l16 : r - 1) * r;
        RawVec<DT_F64, 4> m;
        if (s + 1 < RG_T) m.load((const char*)(row + k));
        else {                               // x is zero past the rank: any finite element will do
#pragma unroll
          for (int v = 0; v < 4; ++v) m.r[v] = row[k + v < r ? k + v : r - 1];
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[t] = mfma_f64(m.r[v], (double)x[s][v], acc[t]);
      }
    }
    mfma_f64_results(acc);
    if (u < len) {
#pragma unroll
      for (int t = 0; t < RG_T; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int a = 16 * t + 4 * q + kq;
          if (a < r) X[(int64_t)a * len + u] = (float)acc[t][q];
        }
    }
  } else {
    // result column a = sum over k >= a of L[u][k] C[k][a]; tiles 2 p, 2 p + 1 interleave the columns 32 p .. + 31
#pragma unroll
    for (int s = 0; s < RG_T; ++s) {
      const int k = 16 * s + 4 * kq;
#pragma unroll
      for (int p = 0; p <= s / 2; ++p) {
        const int a = 32 * p + 2 * l16;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const double* row = Cm + (int64_t)(k + v < r ? k + v : r - 1) * r;
          double c0, c1;
          if (2 * p + 2 < RG_T) {
            const f64x2_a8 q = *reinterpret_cast<const f64x2_a8*>(row + a);
            c0 = q.x; c1 = q.y;
          } else {
            c0 = row[a < r ? a : r - 1];     // columns past the rank are computed and dropped
            c1 = row[a + 1 < r ? a + 1 : r - 1];
          }
          const double xv = (double)x[s][v];
          acc[2 * p] = mfma_f64(xv, c0, acc[2 * p]);
          acc[2 * p + 1] = mfma_f64(xv, c1, acc[2 * p + 1]);
        }
      }
    }
    mfma_f64_results(acc);
#pragma unroll
    for (int p = 0; p < (RG_T + 1) / 2; ++p)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int j = u0 + 4 * q + kq, a = 32 * p + 2 * l16;
        if (j >= len || a >= r) continue;
        float* o = X + (int64_t)j * r + a;
        if (a + 1 < r) *reinterpret_cast<f32x2_a4*>(o) = f32x2_a4{(float)acc[2 * p][q], (float)acc[2 * p + 1][q]};
        else *o = (float)acc[2 * p][q];
      }
  }
}

__global__ __launch_bounds__(256, 2) void regauge_apply_kernel(const RegaugeItem* __restrict__ items, Bases b) {
  const RegaugeItem it = items[blockIdx.x];
  switch ((it.r + 15) / 16) {
    case 1: regauge_body<1>(it, b); break;
    case 2: regauge_body<2>(it, b); break;
    case 3: regauge_body<3>(it, b); break;
    case 4: regauge_body<4>(it, b); break;
    case 5: regauge_body<5>(it, b); break;
    case 6: regauge_body<6>(it, b); break;
    case 7: regauge_body<7>(it, b); break;
    default: regauge_body<8>(it, b); break;     // r <= 128
  }
}

}  // namespace

void launch_regauge_apply(const RegaugeItem* items, int64_t nitems, Bases b, hipStream_t s) {
  if (nitems <= 0) return;
  hipLaunchKernelGGL(regauge_apply_kernel, dim3((unsigned)nitems), dim3(256), 0, s, items, b);
}

void launch_chol(const CholItem* items, int64_t nitems, Bases b, hipStream_t s) {
  if (nitems <= 0) return;
  hipLaunchKernelGGL(chol_inv_kernel, dim3((unsigned)nitems), dim3(256), 0, s, items, b);
}

}  // namespace adapm
