// fp64 batched GEMM on the fp64 matrix cores (the "F64" contraction mode and the re-expression of the factors):
//   Out = g X + s (a1 A1 B1 + a2 A2 B2 + a3 A3 B3),   optionally a second combination of X and the same sums
// One launch covers a list of output tiles drawn from many independent problems, so every thin product of Alg. 2 of every
// low-rank block runs in two launches per iteration (the r x r Gram matrices, then both factor updates with their
// products with G).  Operands (bf16 / fp32 / fp64) convert exactly to fp64; all sums run in fp64 in a fixed order.
//
// One workgroup (4 waves) per output tile of 16 tm x 16 tn (tm, tn = 1 or 2).  The products here are thin: a tile has a
// short free index and a contraction of 256 .. 6400, so what bounds the launch is the latency of one tile, and the four
// waves split the contraction (wave w takes every fourth step, neighbouring waves read neighbouring memory) and add
// their partial tiles through LDS in wave order.  Operands go from memory to the registers of the matrix instruction
// (k_f64_common.h); a step's loads are in flight while the previous step is multiplied.
// Measured against 64 x 64 tiles on the vector units with operands staged in LDS (one workgroup walking the whole
// contraction): G R^T, L^T G and the Gram matrices of one GD iteration with the factor updates, 56 blocks of 512 x 512 ..
// 1376 x 512 at r = 32: 454 -> 146 us (of which 115 us, 31 TFLOP/s, for the updates); 7 blocks of at most 256 x 1024 at
// r = 8: 157 -> 37 us; G R^T alone, with R held: 259 -> 61 us and 129 -> 13 us.
#include "k_f64_common.h"

namespace adapm {

namespace {

constexpr int NW = 4;                  // waves of a workgroup: they split the contraction

__device__ __forceinline__ double load_el(const char* base, int dtype, int64_t idx) {
  return dtype == DT_F32 ? (double)reinterpret_cast<const float*>(base)[idx] : reinterpret_cast<const double*>(base)[idx];
}

// acc += alpha * A B over this wave's share of k in [kb, ke)
template <int TM, int TN, int ADT, int BDT, int LAY>
__device__ __forceinline__ void product(const Mat& A, const Mat& B, double alpha, int M, int N, int kb, int ke, int i0, int j0,
                                        const Bases& bs, f64x4 (&acc)[TM][TN]) {
  constexpr bool AK = LAY != G64_IJ, BK_ = LAY == G64_KK;
  constexpr int V = (LAY == G64_KK && ADT == DT_BF16) ? 8 : 4, KS = 4 * V;     // bf16 rows: 16-byte loads
  typedef Operand<ADT, TM, V, AK> OA;
  typedef Operand<BDT, TN, V, BK_> OB;
  const int lane = threadIdx.x & 63, l16 = lane & 15, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const typename OA::Where wa = OA::where(resolve(A.ref, bs), A.s0, A.s1, i0, M, l16);
  const typename OB::Where wb = OB::where(resolve(B.ref, bs), B.s1, B.s0, j0, N, l16);
  OA a0, a1;
  OB b0, b1;
  auto mma = [&](const OA& a, const OB& b) {
#pragma unroll
    for (int v = 0; v < V; ++v) {
      double av[TM], bv[TN];
#pragma unroll
      for (int t = 0; t < TM; ++t) av[t] = alpha * a.get(wa, t, v);
#pragma unroll
      for (int t = 0; t < TN; ++t) bv[t] = b.get(wb, t, v);
#pragma unroll
      for (int t = 0; t < TM; ++t)
#pragma unroll
        for (int u = 0; u < TN; ++u) acc[t][u] = mfma_f64(av[t], bv[u], acc[t][u]);
    }
  };
  const int nfull = (ke - kb) / KS;
  const int k1 = kb + V * kq;
  if (wave < nfull) {
    a0.load(wa, k1 + wave * KS);
    b0.load(wb, k1 + wave * KS);
    for (int s = wave; s < nfull; s += NW) {
      const int nx = s + NW < nfull ? s + NW : s;      // past the end the last step is read again
      a1.load(wa, k1 + nx * KS);
      b1.load(wb, k1 + nx * KS);
      mma(a0, b0);
      a0 = a1;
      b0 = b1;
    }
    mfma_f64_results(acc);
  }
  if (kb + nfull * KS < ke && (nfull & (NW - 1)) == wave) {
    a0.load_edge(wa, k1 + nfull * KS, ke);
    b0.load_edge(wb, k1 + nfull * KS, ke);
    mma(a0, b0);
    mfma_f64_results(acc);
  }
}

// the operand types that occur, per layout and tile (the planner makes no others)
template <int TM, int TN, int LAY>
__device__ __forceinline__ void product_any(const Mat& A, const Mat& B, double alpha, int M, int N, int kb, int ke, int i0, int j0,
                                            const Bases& bs, f64x4 (&acc)[TM][TN]) {
#define ADAPM_CASE(ADT, BDT) \
  if (A.dtype == ADT && B.dtype == BDT) return product<TM, TN, ADT, BDT, LAY>(A, B, alpha, M, N, kb, ke, i0, j0, bs, acc)
  ADAPM_CASE(DT_F64, DT_F64);
  ADAPM_CASE(DT_F32, DT_F64);
  ADAPM_CASE(DT_F32, DT_F32);
  ADAPM_CASE(DT_F64, DT_F32);
  if constexpr (LAY == G64_KK) {
    ADAPM_CASE(DT_BF16, DT_F64);
    ADAPM_CASE(DT_BF16, DT_F32);
  }
  if constexpr (LAY == G64_IJ) {
    ADAPM_CASE(DT_F64, DT_BF16);
    ADAPM_CASE(DT_F32, DT_BF16);
  }
#undef ADAPM_CASE
}

template <int TM, int TN, int LAY>
__device__ __forceinline__ void tile_body(const GemmProblem& P, const GemmTile& t, const Bases& bs, double* red) {
  const int i0 = 16 * TM * t.ti, j0 = 16 * TN * t.tj;
  const int lane = threadIdx.x & 63, l16 = lane & 15, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  f64x4 acc[TM][TN];
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < TN; ++b) acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
  if (P.K1 > 0) {
    // a lower-triangular operand of the first product (tri = 1: A1, tri = 2: B1) leaves part of the contraction
    // identically zero for this tile: rows i0 .. of A1 end at column i0 + 16 TM - 1, columns j0 .. of B1 start at row j0
    const int ke = P.tri == 1 ? (P.K1 < i0 + 16 * TM ? P.K1 : i0 + 16 * TM) : P.K1;
    const int kb = P.tri == 2 ? j0 : 0;
    product_any<TM, TN, LAY>(P.A1, P.B1, P.a1 * (P.scale_g ? (double)grad_scale(bs) : 1.0), P.M, P.N, kb, ke, i0, j0, bs, acc);
  }
  if (P.K2 > 0) product_any<TM, TN, LAY>(P.A2, P.B2, P.a2, P.M, P.N, 0, P.K2, i0, j0, bs, acc);
  if (P.K3 > 0) product_any<TM, TN, LAY>(P.A3, P.B3, P.a3, P.M, P.N, 0, P.K3, i0, j0, bs, acc);
  // the waves' partial tiles, added in wave order; wave w finishes every NW-th result register
  constexpr int NR = TM * TN * 4;
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < TN; ++b)
#pragma unroll
      for (int q = 0; q < 4; ++q) red[(wave * NR + (a * TN + b) * 4 + q) * 64 + lane] = acc[a][b][q];
  __syncthreads();
  const char* Xb = P.X.ref.space != SP_NONE ? resolve(P.X.ref, bs) : nullptr;
  char* Ob = resolve(P.Out.ref, bs);
  // optional device scalar on everything but X (normalised step of Alg. 2)
  const double step_scale = P.off_s >= 0 ? *reinterpret_cast<const double*>(bs.ws + P.off_s) : P.s0;
  char* Ob2 = P.Out2.ref.space != SP_NONE ? resolve(P.Out2.ref, bs) : nullptr;
#pragma unroll
  for (int e = 0; e < NR / NW; ++e) {
    const int reg = e * NW + wave, q = reg & 3, b = (reg >> 2) % TN, a = (reg >> 2) / TN;
    double val = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) val += red[(w * NR + reg) * 64 + lane];
    const int row = 4 * q + kq;
    const int i = LAY == G64_IJ ? i0 + TM * row + a : i0 + 16 * a + row;
    const int j = LAY == G64_KK ? j0 + 16 * b + l16 : j0 + TN * l16 + b;
    if (i >= P.M || j >= P.N) continue;
    // the step with R held takes both D = b1 (L' - P) and L_t from one P = G R^T (three launches 62 + 19 + 13 -> 66 us)
    double val2 = P.s2 * val;
    val *= step_scale;
    if (Xb) {
      const double x = load_el(Xb, P.X.dtype, (int64_t)i * P.X.s0 + (int64_t)j * P.X.s1);
      val = fma(P.g, x, val);
      val2 = fma(P.g2, x, val2);
    }
    const int64_t o = (int64_t)i * P.Out.s0 + (int64_t)j * P.Out.s1;
    if (P.Out.dtype == DT_F64) reinterpret_cast<double*>(Ob)[o] = val;
    else reinterpret_cast<float*>(Ob)[o] = (float)val;
    if (Ob2) {
      const int64_t o2 = (int64_t)i * P.Out2.s0 + (int64_t)j * P.Out2.s1;
      if (P.Out2.dtype == DT_F64) reinterpret_cast<double*>(Ob2)[o2] = val2;
      else reinterpret_cast<float*>(Ob2)[o2] = (float)val2;
    }
  }
}

__global__ __launch_bounds__(64 * NW, 2) void gemm64_kernel(const GemmProblem* __restrict__ probs,
                                                         const GemmTile* __restrict__ tiles, Bases bs) {
  __shared__ double red[NW * 16 * 64];
  const GemmTile t = tiles[blockIdx.x];
  const GemmProblem& P = probs[t.prob];
  const int shape = 2 * P.tm + P.tn;     // 3: 16 x 16, 4: 16 x 32, 5: 32 x 16, 6: 32 x 32
  if (P.layout == G64_KK) {
    if (shape == 6) tile_body<2, 2, G64_KK>(P, t, bs, red);
    else if (shape == 5) tile_body<2, 1, G64_KK>(P, t, bs, red);
    else tile_body<1, 1, G64_KK>(P, t, bs, red);
  } else if (P.layout == G64_IJ) {
    if (shape == 6) tile_body<2, 2, G64_IJ>(P, t, bs, red);
    else if (shape == 4) tile_body<1, 2, G64_IJ>(P, t, bs, red);
    else tile_body<1, 1, G64_IJ>(P, t, bs, red);
  } else {
    if (shape == 6) tile_body<2, 2, G64_KJ>(P, t, bs, red);
    else tile_body<2, 1, G64_KJ>(P, t, bs, red);
  }
}

}  // namespace

void launch_gemm64(const GemmProblem* probs, const GemmTile* tiles, int64_t ntiles, Bases b, hipStream_t s) {
  if (ntiles <= 0) return;
  hipLaunchKernelGGL(gemm64_kernel, dim3((unsigned)ntiles), dim3(64 * NW), 0, s, probs, tiles, b);
}

}  // namespace adapm
