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

// r <= CH_MAX: right-looking by 16 x 16 blocks of the lower triangle, kept in LDS (row stride 17: a fragment's 16 rows fall on
// different banks), the rows and columns past r an identity.  One wave factorises a diagonal block and inverts it, a row per
// lane, whose columns reach the others by lane reads; the panel below it (P_i = A_i,p C_pp^-T), the trailing blocks and the inverse are
// products on the matrix cores.  What is serial, one pivot after the other, is 16 square roots and divisions per block;
// the trailing blocks of a panel are updated beside the next diagonal block, by the other waves.  78 KB of LDS, two workgroups per
// CU, so that the 288 matrices of the 1600 / 6400 table are all on chip at once: 0.83 -> 0.11 ms (element by element with three
// barriers per pivot, the whole square in LDS).  Pivots past r are skipped: a chain of sixteen for every block took the 85 matrices of
// r = 6 of a small model 9.1 us, element by element 6.8, now 6.1.
constexpr int CB = 16, CLD = 17, CBLK = CB * CLD, CNB = CH_MAX / CB;
__device__ __forceinline__ int block_at(int i, int j) { return (i * (i + 1) / 2 + j) * CBLK; }     // i >= j

__device__ __forceinline__ double lane_value(double x, int lane) {       // x of that lane; lane uniform
  const int lo = __builtin_amdgcn_readlane(__double2loint(x), lane), hi = __builtin_amdgcn_readlane(__double2hiint(x), lane);
  return __hiloint2double(hi, lo);
}

// operand fragment of a block: element [l % 16][4 v + l / 16], v = 0 .. 3
struct Frag { double v[4]; };
__device__ __forceinline__ Frag frag(const double* blk, int l16, int kq) {
  Frag f;
#pragma unroll
  for (int v = 0; v < 4; ++v) f.v[v] = blk[l16 * CLD + 4 * v + kq];
  return f;
}

// Between LDS writes and reads of the same places by other lanes of the same wave.  The hardware keeps a wave's LDS accesses in
// order; this tells the compiler, which sees one lane and may move accesses past each other that only lanes apart from it share.
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// diagonal block p, as it stands in LDS: its lower factor to global memory, its inverse in its place
__device__ __forceinline__ void diagonal(double* blk, double* A, int r, int p, int lane, int* bad) {
  const int i = lane & 15;                       // this lane's row (the four copies do the same)
  double row[CB];
#pragma unroll
  for (int k = 0; k < CB; ++k) row[k] = blk[i * CLD + k];
  bool wrong = false;
  const int real = r - CB * p;                   // pivots past the end are ones, with zeros beside them: nothing to do
#pragma unroll
  for (int j = 0; j < CB; ++j) {
    if (j < real) {
      const double piv = lane_value(row[j], j);
      wrong = wrong || !(piv > 0.0) || !isfinite(piv);
      const double d = sqrt(piv);
      row[j] = i == j ? d : row[j] / d;
#pragma unroll
      for (int k = j + 1; k < CB; ++k) row[k] -= row[j] * lane_value(row[j], k);
    }
  }
  // column i of the inverse by forward substitution
  double x[CB];
#pragma unroll
  for (int a = 0; a < CB; ++a) {
    double s = a == i ? 1.0 : 0.0;
    if (a < real) {
#pragma unroll
      for (int c = 0; c < a; ++c) s -= lane_value(row[c], a) * x[c];
      s /= lane_value(row[a], a);
    }
    x[a] = s;
  }
  wave_lds_order();                              // every lane has read its row
  if (wrong) *bad = 1;
  if (lane < CB) {
#pragma unroll
    for (int k = 0; k < CB; ++k) {
      if (CB * p + i < r && CB * p + k < r) A[(int64_t)(CB * p + i) * r + CB * p + k] = k <= i ? row[k] : 0.0;
      blk[k * CLD + i] = x[k];
    }
  }
}

__global__ __launch_bounds__(256, 2) void chol_inv_kernel(const CholItem* __restrict__ items, Bases b) {
  __shared__ double S[CNB * (CNB + 1) / 2 * CBLK];
  __shared__ int bad;
  const CholItem it = items[blockIdx.x];
  const int r = it.r, tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  double* A = reinterpret_cast<double*>(b.ws + it.off_gram);
  double* X = reinterpret_cast<double*>(b.ws + it.off_inv);
  if (r > CH_MAX) { chol_inv_global(A, X, r); return; }
  const int nb = (r + CB - 1) / CB;
  if (tid == 0) bad = 0;
  for (int e = tid; e < CB * nb * CB * nb; e += 256) {
    const int i = e / (CB * nb), k = e % (CB * nb), bi = i / CB, bk = k / CB;
    const bool in = i < r && k < r;
    if (bk <= bi) S[block_at(bi, bk) + (i % CB) * CLD + k % CB] = (in && k <= i) ? A[(int64_t)i * r + k] : (i == k ? 1.0 : 0.0);
    else if (in) A[(int64_t)i * r + k] = X[(int64_t)i * r + k] = 0.0;     // the blocks above the diagonal are not read
  }
  __syncthreads();
  // block (i, j) -= P_i P_j^T with the panel p
  auto trailing = [&](int i, int j, int p) {
    const Frag a = frag(S + block_at(i, p), l16, kq), c = frag(S + block_at(j, p), l16, kq);
    double* o = S + block_at(i, j) + kq * CLD + l16;
    f64x4 acc[1];
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[0][q] = o[4 * q * CLD];
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[0] = mfma_f64(-a.v[v], c.v[v], acc[0]);
    mfma_f64_results(acc);
#pragma unroll
    for (int q = 0; q < 4; ++q) o[4 * q * CLD] = acc[0][q];
  };
  for (int p = 0; p < nb; ++p) {
    if (wave == 0) {
      if (p > 0) trailing(p, p, p - 1);
      wave_lds_order();                              // its rows go to other lanes
      diagonal(S + block_at(p, p), A, r, p, lane, &bad);
    } else if (p > 0) {
      int n = 0;
      for (int i = p; i < nb; ++i)
        for (int j = p; j <= i; ++j) {
          if (i == p) continue;
          if (n++ % 3 == wave - 1) trailing(i, j, p - 1);
        }
    }
    __syncthreads();
    if (bad) break;                                  // uniform: set before the barrier, by one wave
    for (int i = p + 1 + wave; i < nb; i += 4) {     // P_i = A_i,p C_pp^-T, also to global memory
      double* blk = S + block_at(i, p);
      const Frag a = frag(blk, l16, kq), c = frag(S + block_at(p, p), l16, kq);
      f64x4 acc[1] = {f64x4{0.0, 0.0, 0.0, 0.0}};
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[0] = mfma_f64(a.v[v], c.v[v], acc[0]);
      mfma_f64_results(acc);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int row = 4 * q + kq;
        blk[row * CLD + l16] = acc[0][q];
        if (CB * i + row < r) A[(int64_t)(CB * i + row) * r + CB * p + l16] = acc[0][q];
      }
    }
    __syncthreads();
  }
  if (bad) {
    for (int e = tid; e < r * r; e += 256) A[e] = X[e] = (e / r == e % r) ? 1.0 : 0.0;
    return;
  }
  // columns of blocks of C^-1, two per wave, a long and a short one.  X_jj is in LDS; X_ij = -C_ii^-1 sum over k < i of
  // C_ik X_kj, where a block of X leaves the matrix cores as the operand of the next products (register q of lane l is its
  // element [4 q + l / 16][l % 16])
  for (int turn = 0; turn < 2; ++turn) {
    const int j = turn == 0 ? wave : 2 * 4 - 1 - wave;
    if (j >= nb) continue;
    f64x4 x[CNB];
#pragma unroll
    for (int n = 0; n < CNB; ++n) {
      if (j + n >= nb) continue;
      const double* inv = S + block_at(j + n, j + n);
      f64x4 acc[1] = {f64x4{0.0, 0.0, 0.0, 0.0}};
      if (n == 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[0][q] = inv[(4 * q + kq) * CLD + l16];
      } else {
        f64x4 sum[1] = {f64x4{0.0, 0.0, 0.0, 0.0}};
#pragma unroll
        for (int k = 0; k < n; ++k) {
          const Frag c = frag(S + block_at(j + n, j + k), l16, kq);
#pragma unroll
          for (int v = 0; v < 4; ++v) sum[0] = mfma_f64(c.v[v], x[k][v], sum[0]);
        }
        mfma_f64_results(sum);
        const Frag d = frag(inv, l16, kq);
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[0] = mfma_f64(-d.v[v], sum[0][v], acc[0]);
        mfma_f64_results(acc);
      }
      x[n] = acc[0];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int row = CB * (j + n) + 4 * q + kq, col = CB * j + l16;
        if (row < r && col < r) X[(int64_t)row * r + col] = acc[0][q];
      }
    }
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
