// fp64 batched GEMM on the fp64 matrix cores (the "F64" contraction mode and the re-expression of the factors):
//   Out = g X + s (a1 A1 B1 + a2 A2 B2 + a3 A3 B3),   optionally a second combination of X and the same sums
// One launch covers a list of output tiles drawn from many independent problems, so every thin product of Alg. 2 of every
// low-rank block runs in two launches per iteration (the r x r Gram matrices, then both factor updates with their
// products with G).  Operands (bf16 / fp32 / fp64) convert exactly to fp64; all sums run in fp64 in a fixed order.
//
// One workgroup per output tile.  The products here are thin: a tile has a short free index and a contraction of 256 .. 6400,
// so what bounds a launch is the latency of a tile, then the fp64 rate.  The waves of a workgroup split the contraction (wave
// w takes every NW-th step, neighbouring waves read neighbouring memory, the steps of up to three products are numbered
// through) and add their partial tiles through LDS in wave order.  Operands go from memory to the registers of the matrix
// instruction (k_f64_common.h); a step's loads are in flight while the previous step is multiplied.
//   4 waves, tiles of 16 tm x 16 tn (tm, tn = 1 or 2): launches of more tiles than the chip takes at once;
//   8 waves, 16 x 16: launches that leave compute units idle (waves64 in adapm_api.hip), whose contraction would otherwise
//   keep a few waves busy on a nearly empty chip: 7 blocks of at most 256 x 1024 at r = 8, Gram matrices of an iteration
//   11.6 -> 8.5 us, factor updates 16.8 -> 11.7, G R^T with R held 12.3 -> 7.7.  (16 waves were no better in any of 60 tables and 3 - 4 us a literal
//   step slower in most.)  What is left of such a launch is the look-up of its problem and a cold instruction cache.
// Measured against 64 x 64 tiles on the vector units with operands staged in LDS (one workgroup walking the whole
// contraction): G R^T, L^T G and the Gram matrices of one GD iteration with the factor updates, the 56 blocks: 454 -> 110 us
// (of which 86 us, 41 TFLOP/s, for the updates; the matrix cores are busy half of that; 24 us for the Gram matrices); the 7 small ones 157 -> 21 us.
#include "k_f64_common.h"

namespace adapm {

namespace {

__device__ __forceinline__ double load_el(const char* base, int dtype, int64_t idx) {
  return dtype == DT_F32 ? (double)reinterpret_cast<const float*>(base)[idx] : reinterpret_cast<const double*>(base)[idx];
}

// acc += alpha * A B over this wave's share of k in [kb, ke); `first`: the step that wave 0 would take if the steps of all
// products were numbered through (a short product then falls to the waves that the one before it left out)
template <int NW, bool AHEAD, int TM, int TN, int ADT, int BDT, int LAY>
__device__ __forceinline__ void product(const Mat& A, const Mat& B, double alpha, int M, int N, int kb, int ke, int i0, int j0,
                                        const Bases& bs, f64x4 (&acc)[TM][TN], int& first) {
  constexpr bool AK = LAY != G64_IJ, BK_ = LAY == G64_KK;
  constexpr int V = 4, KS = 4 * V;
  typedef Operand<ADT, TM, V, AK> OA;
  typedef Operand<BDT, TN, V, BK_> OB;
  const int lane = threadIdx.x & 63, l16 = lane & 15, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const typename OA::Where wa = OA::where(resolve(A.ref, bs), A.s0, A.s1, i0, M, l16);
  const typename OB::Where wb = OB::where(resolve(B.ref, bs), B.s1, B.s0, j0, N, l16);
  // steps in flight (three or four cost more in operands read twice at the end than they hide: 8 waves, 4 - 16 steps each,
  // 11.7 -> 13.2 us; 4 waves 98 -> 110 us)
  constexpr int PD = 2;
  OA a[PD];
  OB b[PD];
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
  const int nfull = (ke - kb) / KS, mine = (wave - first) & (NW - 1);
  const bool edge = kb + nfull * KS < ke;
  const int k1 = kb + V * kq;
  if constexpr (!AHEAD) {
    if (mine < nfull) {
      for (int t = mine; t < nfull; t += NW) {
        typename OA::Where pa = wa;
        typename OB::Where pb = wb;
        OA::step(pa, k1 + t * KS);
        OB::step(pb, k1 + t * KS);
        a[0].load(pa);
        b[0].load(pb);
        mma(a[0], b[0]);
      }
      mfma_f64_results(acc);
    }
  } else if (mine < nfull) {
    typename OA::Where pa = wa;
    typename OB::Where pb = wb;
    OA::step(pa, k1 + mine * KS);
    OB::step(pb, k1 + mine * KS);
    // where pa, pb stand now, then on by one of this wave's steps (past the end the last one is read again).  Without the
    // barrier the compiler reads operands where they are used: one load of either step's address for two loads
    auto request = [&](int s, OA& ao, OB& bo) {
      ao.load(pa);
      bo.load(pb);
      const int on = s + NW < nfull ? NW * KS : 0;
      OA::step(pa, on);
      OB::step(pb, on);
      __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int u = 0; u + 1 < PD; ++u) request(mine + u * NW, a[u], b[u]);
    for (int s0 = mine; s0 < nfull; s0 += PD * NW) {
#pragma unroll
      for (int u = 0; u < PD; ++u) {
        const int s = s0 + u * NW;
        if (u > 0 && s >= nfull) break;
        request(s + (PD - 1) * NW, a[(u + PD - 1) % PD], b[(u + PD - 1) % PD]);
        mma(a[u], b[u]);
      }
    }
    mfma_f64_results(acc);
  }
  if (edge && (nfull & (NW - 1)) == mine) {
    a[0].load_edge(wa, k1 + nfull * KS, ke);
    b[0].load_edge(wb, k1 + nfull * KS, ke);
    mma(a[0], b[0]);
    mfma_f64_results(acc);
  }
  first = (first + nfull + (edge ? 1 : 0)) & (NW - 1);
}

// the operand types that occur, per layout and tile (the planner makes no others)
template <int NW, bool AHEAD, int TM, int TN, int LAY>
__device__ __forceinline__ void product_any(const Mat& A, const Mat& B, double alpha, int M, int N, int kb, int ke, int i0, int j0,
                                            const Bases& bs, f64x4 (&acc)[TM][TN], int& first) {
#define ADAPM_CASE(ADT, BDT) \
  if (A.dtype == ADT && B.dtype == BDT) return product<NW, AHEAD, TM, TN, ADT, BDT, LAY>(A, B, alpha, M, N, kb, ke, i0, j0, bs, acc, first)
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

template <int NW, bool AHEAD, int TM, int TN, int LAY>
__device__ __forceinline__ void tile_body(const GemmProblem& P, const GemmTile& t, const Bases& bs, double* red) {
  const int i0 = 16 * TM * t.ti, j0 = 16 * TN * t.tj;
  const int lane = threadIdx.x & 63, l16 = lane & 15, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  f64x4 acc[TM][TN];
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < TN; ++b) acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
  // wave w finishes every NW-th result register; what it adds them to is requested ahead of the products
  constexpr int NR = TM * TN * 4, NE = (NR + NW - 1) / NW;
  auto place = [&](int e, int& i, int& j) {
    const int reg = e * NW + wave, q = reg & 3, b = (reg >> 2) % TN, a = (reg >> 2) / TN;
    const int row = 4 * q + kq;
    i = LAY == G64_IJ ? i0 + TM * row + a : i0 + 16 * a + row;
    j = LAY == G64_KK ? j0 + 16 * b + l16 : j0 + TN * l16 + b;
    return reg < NR && i < P.M && j < P.N;
  };
  const char* Xb = P.X.ref.space != SP_NONE ? resolve(P.X.ref, bs) : nullptr;
  double xs[NE];
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    int i, j;
    xs[e] = 0.0;
    if (Xb && place(e, i, j)) xs[e] = load_el(Xb, P.X.dtype, (int64_t)i * P.X.s0 + (int64_t)j * P.X.s1);
  }
  int first = 0;
  if (P.K1 > 0) {
    // a lower-triangular operand of the first product (tri = 1: A1, tri = 2: B1) leaves part of the contraction
    // identically zero for this tile: rows i0 .. of A1 end at column i0 + 16 TM - 1, columns j0 .. of B1 start at row j0
    const int ke = P.tri == 1 ? (P.K1 < i0 + 16 * TM ? P.K1 : i0 + 16 * TM) : P.K1;
    const int kb = P.tri == 2 ? j0 : 0;
    product_any<NW, AHEAD, TM, TN, LAY>(P.A1, P.B1, P.a1 * (P.scale_g ? (double)grad_scale(bs) : 1.0), P.M, P.N, kb, ke, i0, j0, bs, acc, first);
  }
  if (P.K2 > 0) product_any<NW, AHEAD, TM, TN, LAY>(P.A2, P.B2, P.a2, P.M, P.N, 0, P.K2, i0, j0, bs, acc, first);
  if (P.K3 > 0) product_any<NW, AHEAD, TM, TN, LAY>(P.A3, P.B3, P.a3, P.M, P.N, 0, P.K3, i0, j0, bs, acc, first);
  // the waves' partial tiles, added in wave order
#pragma unroll
  for (int a = 0; a < TM; ++a)
#pragma unroll
    for (int b = 0; b < TN; ++b)
#pragma unroll
      for (int q = 0; q < 4; ++q) red[(wave * NR + (a * TN + b) * 4 + q) * 64 + lane] = acc[a][b][q];
  __syncthreads();
  char* Ob = resolve(P.Out.ref, bs);
  // optional device scalar on everything but X (normalised step of Alg. 2)
  const double step_scale = P.off_s >= 0 ? *reinterpret_cast<const double*>(bs.ws + P.off_s) : P.s0;
  char* Ob2 = P.Out2.ref.space != SP_NONE ? resolve(P.Out2.ref, bs) : nullptr;
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    int i, j;
    if (!place(e, i, j)) continue;
    double val = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) val += red[(w * NR + e * NW + wave) * 64 + lane];
    // the step with R held takes both D = b1 (L' - P) and L_t from one P = G R^T (three launches 62 + 19 + 13 -> 66 us)
    // s2 = 0: the old factor is copied, whatever the sums are
    double val2 = P.s2 != 0.0 ? P.s2 * val : 0.0;
    val *= step_scale;
    if (Xb) {
      val = fma(P.g, xs[e], val);
      val2 = fma(P.g2, xs[e], val2);
    }
    if (P.dup) val2 = val;
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

template <int NW, bool AHEAD>
__global__ __launch_bounds__(64 * NW, NW == 4 ? 2 : 4) void gemm64_kernel(const GemmProblem* __restrict__ probs,
                                                                          const GemmTile* __restrict__ tiles, Bases bs) {
  __shared__ double red[NW * (NW == 4 ? 16 : 4) * 64];
  const GemmTile t = tiles[blockIdx.x];
  if (t.prob == GEMM_TILE_NONE) return;
  const GemmProblem& P = probs[t.prob];
  if constexpr (NW > 4) {
    if (P.layout == G64_KK) tile_body<NW, AHEAD, 1, 1, G64_KK>(P, t, bs, red);
    else tile_body<NW, AHEAD, 1, 1, G64_IJ>(P, t, bs, red);
  } else {
    const int shape = 2 * P.tm + P.tn;     // 3: 16 x 16, 4: 16 x 32, 5: 32 x 16, 6: 32 x 32
    if (P.layout == G64_KK) {
      if (shape == 6) tile_body<NW, AHEAD, 2, 2, G64_KK>(P, t, bs, red);
      else if (shape == 5) tile_body<NW, AHEAD, 2, 1, G64_KK>(P, t, bs, red);
      else tile_body<NW, AHEAD, 1, 1, G64_KK>(P, t, bs, red);
    } else if (P.layout == G64_IJ) {
      if (shape == 6) tile_body<NW, AHEAD, 2, 2, G64_IJ>(P, t, bs, red);
      else if (shape == 4) tile_body<NW, AHEAD, 1, 2, G64_IJ>(P, t, bs, red);
      else tile_body<NW, AHEAD, 1, 1, G64_IJ>(P, t, bs, red);
    } else {
      if (shape == 6) tile_body<NW, AHEAD, 2, 2, G64_KJ>(P, t, bs, red);
      else tile_body<NW, AHEAD, 2, 1, G64_KJ>(P, t, bs, red);
    }
  }
}

}  // namespace

void launch_gemm64(int waves, bool ahead, const GemmProblem* probs, const GemmTile* tiles, int64_t ntiles, Bases b, hipStream_t s) {
  if (ntiles <= 0) return;
  const dim3 grid((unsigned)ntiles);
  if (waves == 8) hipLaunchKernelGGL((gemm64_kernel<8, true>), grid, dim3(512), 0, s, probs, tiles, b);
  else if (ahead) hipLaunchKernelGGL((gemm64_kernel<4, true>), grid, dim3(256), 0, s, probs, tiles, b);
  else hipLaunchKernelGGL((gemm64_kernel<4, false>), grid, dim3(256), 0, s, probs, tiles, b);
}

}  // namespace adapm
