// Update of the low-rank blocks on the exact path, with the m x n term of eq. 3-4 built tile by tile in fp64 on the fp64
// matrix cores and never stored:
//   C = a1 A1 B1 + a2 A2 B2 (fp64, rounded once to fp32),   m^c = cG G + cC C,   then v and W as in the element-wise update.
//
// Contraction over the rank only (8 .. 128 and up), result as large as the block: bound by the streams of G, W and v, which
// are requested before the contraction starts.  One workgroup (4 waves) per 64 x 64 tile, a wave owns 16 rows x 64 columns:
// a lane's share of an operand row is one 16-byte load (four values of k of A, four columns of B), its results are four
// consecutive columns of four rows, so every stream moves 64 consecutive elements per row and nothing passes through LDS.
// Against a GEMM of 32 x 32 tiles that splits this short contraction over its waves and stores C, followed by the
// element-wise kernel (56 blocks of 512 x 512 .. 1376 x 512, 25 M elements, r = 32, fp32 W and v, bf16 G): one product (R held)
// 150 + 108 -> 153 us, two (after Alg. 2) 202 + 106 -> 202 us; its 0.45 GB take 87 us at 5.2 TB/s.
#include "k_f64_common.h"

namespace adapm {

namespace {

constexpr int UT = UPD64_TILE;

struct __attribute__((packed, aligned(2))) u32x2_a2 { uint32_t x, y; };

// four consecutive elements of a row as they lie in memory, at the alignment of their type
struct Raw4 {
  uint32_t r[4];
  __device__ __forceinline__ void load(const char* base, int dtype, int64_t e) {
    if (dtype == DT_BF16) {
      const u32x2_a2 q = *reinterpret_cast<const u32x2_a2*>(base + e * 2);
      r[0] = q.x; r[1] = q.y;
    } else {
      const u32x4_a2 q = *reinterpret_cast<const u32x4_a2*>(base + e * 4);
      r[0] = q.x; r[1] = q.y; r[2] = q.z; r[3] = q.w;
    }
  }
  __device__ __forceinline__ void get(int dtype, float (&x)[4]) const {
    if (dtype == DT_BF16) {
      x[0] = bf16lo(r[0]); x[1] = bf16hi(r[0]); x[2] = bf16lo(r[1]); x[3] = bf16hi(r[1]);
    } else {
#pragma unroll
      for (int t = 0; t < 4; ++t) x[t] = __uint_as_float(r[t]);
    }
  }
};

__device__ __forceinline__ float load_one(const char* base, int dtype, int64_t e) {
  return dtype == DT_BF16 ? bf16lo((uint32_t)reinterpret_cast<const uint16_t*>(base)[e]) : reinterpret_cast<const float*>(base)[e];
}

// acc[t] += alpha A(i0 + l16 .., k) B(k, column of the lane + t): rows of both operands are contiguous
template <int ADT, int BDT>
__device__ __forceinline__ void accumulate(const Mat& A, const Mat& B, double alpha, int K, int M, int N, int i0, int col,
                                           const Bases& bs, f64x4 (&acc)[4]) {
  constexpr int EA = elem_bytes(ADT), EB = elem_bytes(BDT);
  const int lane = threadIdx.x & 63, l16 = lane & 15, kq = lane >> 4;
  const int row = i0 + l16 < M ? i0 + l16 : M - 1;                 // rows past the end repeat the last one
  const char* pa = resolve(A.ref, bs) + (int64_t)row * A.s0 * EA;
  const char* pb = resolve(B.ref, bs) + (int64_t)col * EB;
  const int64_t sb = B.s0 * EB;
  const bool wide = N >= 4;
  for (int k0 = 0; k0 < K; k0 += 16) {
    const int k = k0 + 4 * kq;
    RawVec<ADT, 4> a;
    RawVec<BDT, 4> b[4];
    if (k0 + 16 <= K) a.load(pa + (int64_t)k * EA);
    else {
#pragma unroll
      for (int v = 0; v < 4; ++v) a.load1(v, pa + (int64_t)(k + v < K ? k + v : K - 1) * EA);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const char* p = pb + (int64_t)(k + v < K ? k + v : K - 1) * sb;
      if (wide) b[v].load(p);
      else {
#pragma unroll
        for (int t = 0; t < 4; ++t) b[v].load1(t, p + (t < N ? t : N - 1) * EB);
      }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const bool in = k + v < K;                                    // values of k past the end count as zero
      const double av = in ? alpha * a.get(v) : 0.0;
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[t] = mfma_f64(av, in ? b[v].get(t) : 0.0, acc[t]);
    }
  }
  mfma_f64_results(acc);
}

// the operand types that occur (the planner makes no others)
__device__ __forceinline__ void accumulate_any(const Mat& A, const Mat& B, double alpha, int K, int M, int N, int i0, int col,
                                               const Bases& bs, f64x4 (&acc)[4]) {
  if (A.dtype == DT_F32) accumulate<DT_F32, DT_F32>(A, B, alpha, K, M, N, i0, col, bs, acc);
  else if (B.dtype == DT_F32) accumulate<DT_F64, DT_F32>(A, B, alpha, K, M, N, i0, col, bs, acc);
  else accumulate<DT_F64, DT_F64>(A, B, alpha, K, M, N, i0, col, bs, acc);
}

__global__ __launch_bounds__(256, 2) void update64_kernel(const GemmProblem* __restrict__ probs, const GemmTile* __restrict__ tiles,
                                                       const BlockDev* __restrict__ blocks, Bases bs, StepScalars sc) {
  const GemmTile tile = tiles[blockIdx.x];
  const GemmProblem& P = probs[tile.prob];
  const int M = P.M, N = P.N, block = P.Out.ref.block;
  const BlockDev& blk = blocks[block];
  const int lane = threadIdx.x & 63, l16 = lane & 15, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i0 = UT * tile.ti + 16 * wave;
  if (i0 >= M) return;
  // this lane's four columns: j .. j + 3, or, across the end of a row, its last four (the first of which another lane
  // updates); fewer than four columns: `own` of them from column 0
  const int j = UT * tile.tj + 4 * l16;
  const int col = j + 4 <= N ? j : (N >= 4 ? N - 4 : 0);
  const int skip = j < N ? j - col : 4, own = N < 4 ? N : 4;        // columns skip .. own - 1 are this lane's to update
  const char* __restrict__ G = (const char*)bs.grads[block];
  char* __restrict__ W = (char*)bs.params[block];
  float* __restrict__ v = reinterpret_cast<float*>(bs.state + blk.off_v);
  const int gdt = blk.grad_dtype, wdt = blk.param_dtype;
  const bool vel = blk.v_mode == VM_ELEMENT, wide = N >= 4;
  const int vrows = vel ? 1 : (int)(blk.group_elems / N);           // rows that share one v
  // G, W and v of the lane's 4 x 4 elements are requested before the contraction and used behind it
  Raw4 gq[4], wq[4], vq[4];
  float vg[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int i = i0 + 4 * q + kq, ic = i < M ? i : M - 1;
    const int64_t e = (int64_t)ic * N + col;
    if (wide) {
      gq[q].load(G, gdt, e);
      wq[q].load(W, wdt, e);
      if (vel) vq[q].load((const char*)v, DT_F32, e);
    }
    vg[q] = vel ? 0.f : v[ic / vrows];
  }
  f64x4 acc[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
  accumulate_any(P.A1, P.B1, P.a1, P.K1, M, N, i0, col, bs, acc);
  if (P.K2 > 0) accumulate_any(P.A2, P.B2, P.a2, P.K2, M, N, i0, col, bs, acc);
  const UpdCoef cf = make_coef(sc.lr, blk.lr_scale, blk.wd, sc.clip);
  const float ob2 = 1.f - sc.beta2;
  const float gs = grad_scale(bs);                                  // global clipping: the method sees gs * G
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int i = i0 + 4 * q + kq;
    if (i >= M || skip >= own) continue;
    const int64_t e = (int64_t)i * N + col;
    float g[4], w[4], vv[4];
    if (wide) {
      gq[q].get(gdt, g);
      wq[q].get(wdt, w);
      if (vel) vq[q].get(DT_F32, vv);
    } else {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int64_t et = e + (t < own ? t : 0);
        g[t] = load_one(G, gdt, et);
        w[t] = load_one(W, wdt, et);
        if (vel) vv[t] = v[et];
      }
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      if (gs != 1.f) g[t] *= gs;
      vv[t] = vel ? sc.beta2 * vv[t] + ob2 * g[t] * g[t] : vg[q];
      const float inv = inv_denom_fast(vv[t], sc.inv_debias_v, sc.inv_debias_m, sc.eps);
      w[t] = apply_update(w[t], sc.cG * g[t] + sc.cC * (float)acc[t][q], inv, cf);
    }
    if (skip == 0 && own == 4) {
      if (vel) *reinterpret_cast<f32x4_a4*>(v + e) = f32x4_a4{vv[0], vv[1], vv[2], vv[3]};
      if (wdt == DT_BF16) *reinterpret_cast<u32x2_a2*>(W + e * 2) = u32x2_a2{pack_bf16x2(w[0], w[1]), pack_bf16x2(w[2], w[3])};
      else *reinterpret_cast<f32x4_a4*>(W + e * 4) = f32x4_a4{w[0], w[1], w[2], w[3]};
    } else {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        if (t < skip || t >= own) continue;
        if (vel) v[e + t] = vv[t];
        if (wdt == DT_BF16) reinterpret_cast<uint16_t*>(W)[e + t] = (uint16_t)pack_bf16x2(w[t], 0.f);
        else reinterpret_cast<float*>(W)[e + t] = w[t];
      }
    }
  }
}

}  // namespace

void launch_update64(const GemmProblem* probs, const GemmTile* tiles, int64_t ntiles, const BlockDev* blocks, Bases b,
                     StepScalars sc, hipStream_t s) {
  if (ntiles <= 0) return;
  hipLaunchKernelGGL(update64_kernel, dim3((unsigned)ntiles), dim3(256), 0, s, probs, tiles, blocks, b, sc);
}

}  // namespace adapm
