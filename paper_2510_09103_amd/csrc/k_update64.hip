// Update of the low-rank blocks on the exact path, with the m x n term of eq. 3-4 built tile by tile in fp64 on the fp64
// matrix cores and never stored:
//   C = a1 A1 B1 + a2 A2 B2 (fp64, rounded once to fp32),   m^c = cG G + cC C,   then v and W as in the element-wise update.
//
// Contraction over the rank only (8 .. 128 and up), result as large as the block: bound by the streams of G, W and v.  One
// workgroup (4 waves) owns 64 rows x a few chunks of 64 columns, a wave 16 of the rows: a lane's share of an operand row is one
// 16-byte load (four values of k of A, four columns of B), its results are four consecutive columns of four rows, so every
// stream moves 64 consecutive elements per row.  A lane multiplies the same values of A in every chunk: they wait in LDS,
// as fp64, each lane's own (no lane reads another's).  The streams of a chunk are requested ahead of its contraction; three
// workgroups per CU (168 registers; four spill) hide the rest.
// 25 M elements in 56 blocks of 512 x 512 .. 1376 x 512 at r = 32, fp32 W and v, bf16 G (0.45 GB, 87 us at 5.2 TB/s): one product
// (R held) 148 -> 101 us, two (after Alg. 2) 203 -> 135 us, against one 64 x 64 tile per workgroup whose types were switched
// on at run time and whose pointers were generic ones: 95 loads per wave where 42 would do, split into 4- and 8-byte pieces.
#include "k_f64_common.h"

namespace adapm {

namespace {

constexpr int UT = UPD64_TILE;
constexpr int UW = 4;                          // waves of a workgroup
constexpr int STEP_BYTES = 2 * 64 * 16;        // a wave's values of A for 16 values of k

// four consecutive elements of a row as they lie in memory, at the alignment of their type
template <int DT>
using Raw4 = RawVec<DT, 4>;
template <int DT>
__device__ __forceinline__ void floats(const Raw4<DT>& q, float (&x)[4]) {
  if constexpr (DT == DT_BF16) {
    x[0] = bf16lo(q.r[0]); x[1] = bf16hi(q.r[0]); x[2] = bf16lo(q.r[1]); x[3] = bf16hi(q.r[1]);
  } else {
#pragma unroll
    for (int t = 0; t < 4; ++t) x[t] = q.r[t];
  }
}
__device__ __forceinline__ void store_one(char* base, int dtype, int64_t e, float x) {
  if (dtype == DT_BF16) reinterpret_cast<uint16_t*>(base)[e] = (uint16_t)pack_bf16x2(x, 0.f);
  else reinterpret_cast<float*>(base)[e] = x;
}

// one product of the m x n term as a wave sees it
struct Factors {
  const char* a;          // this lane's row of A, from its first value of k on
  const char* b;          // first row of B
  unsigned sb;            // bytes from one row of B to the next
  double alpha;
  int K;
  bool a64, b64;          // fp64 (else fp32)
};
__device__ __forceinline__ Factors factors_of(const Mat& A, const Mat& B, double alpha, int K, int row, int kq, const Bases& bs) {
  Factors f;
  f.a64 = A.dtype == DT_F64; f.b64 = B.dtype == DT_F64;
  f.a = resolve(A.ref, bs) + ((int64_t)row * A.s0 + 4 * kq) * (f.a64 ? 8 : 4);
  f.b = resolve(B.ref, bs);
  f.sb = (unsigned)B.s0 * (f.b64 ? 8u : 4u);
  f.alpha = alpha; f.K = K;
  return f;
}

// alpha A for 16 values of k from k0 on -> this lane's place in LDS; values past the end count as zero
template <int ADT>
__device__ __forceinline__ void stage(const Factors& f, int k0, int kq, f64x2_a8* slot) {
  RawVec<ADT, 4> a;
  const char* p = f.a + (int64_t)k0 * elem_bytes(ADT);
  const int left = f.K - k0 - 4 * kq;
  if (k0 + 16 <= f.K) a.load(p);
  else {
#pragma unroll
    for (int v = 0; v < 4; ++v) a.load1(v, left > 0 ? p + (v < left ? v : left - 1) * elem_bytes(ADT) : f.a - 4 * kq * elem_bytes(ADT));
#pragma unroll
    for (int v = 0; v < 4; ++v)
      if (v >= left) a.zero(v);
  }
  slot[0] = f64x2_a8{f.alpha * a.get(0), f.alpha * a.get(1)};
  slot[64] = f64x2_a8{f.alpha * a.get(2), f.alpha * a.get(3)};
}

// acc[t] += A(.., k) B(k, column of the lane + t) for k in [kb, ke), kb a multiple of 16, A from LDS (values past K are zeros)
template <int BDT>
__device__ __forceinline__ void multiply(const Factors& f, int kb, int ke, int kq, int col, const f64x2_a8* slot, f64x4 (&acc)[4]) {
  constexpr unsigned EB = elem_bytes(BDT);
  RawVec<BDT, 4> b[4];
  auto mma = [&]() {
    const f64x2_a8 a0 = slot[0], a1 = slot[64];
    const double av[4] = {a0.x, a0.y, a1.x, a1.y};
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[t] = mfma_f64(av[v], b[v].get(t), acc[t]);
  };
  const unsigned ce = (unsigned)col * EB;
  int k0 = kb;
#pragma nounroll
  for (; k0 + 16 <= ke; k0 += 16) {
    const unsigned at = (unsigned)(k0 + 4 * kq) * f.sb + ce;
#pragma unroll
    for (int v = 0; v < 4; ++v) b[v].load(f.b + (at + (unsigned)v * f.sb));
    mma();
    slot += STEP_BYTES / 16;
  }
  if (k0 < ke) {                           // rows past the end read the last one and count as zero
    const int k = k0 + 4 * kq;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      b[v].load(f.b + ((uint64_t)(unsigned)(k + v < ke ? k + v : ke - 1) * f.sb + ce));
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (k + v >= ke) b[v].zero(t);
    }
    mma();
  }
}

// One body per type of G and W and kind of second moment.  cap: steps of A that a wave's part of the LDS holds; KEEP: they hold all of A of
// every block of the list, which is then staged once.
template <int GDT, int WDT, bool VEL, bool KEEP>
__device__ __forceinline__ void update64_body(const GemmProblem& P, const GemmTile& tile, const BlockDev& blk, const Bases& bs, const StepScalars& sc,
                                              int cap, f64x2_a8* lds) {
  const int M = P.M, N = P.N, block = P.Out.ref.block;
  const int lane = threadIdx.x & 63, l16 = lane & 15, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i0 = UT * tile.ti + 16 * wave;
  if (i0 >= M) return;
  // the wave's rows; offsets from here on are 32 bits (update64_class)
  const char* __restrict__ G = global_ptr((const char*)bs.grads[block] + (int64_t)i0 * N * elem_bytes(GDT));
  char* __restrict__ W = global_ptr((char*)bs.params[block] + (int64_t)i0 * N * elem_bytes(WDT));
  float* const vst = reinterpret_cast<float*>(bs.state + blk.off_v);
  char* __restrict__ V = global_ptr((char*)(vst + (VEL ? (int64_t)i0 * N : 0)));
  const int row = i0 + l16 < M ? i0 + l16 : M - 1;                 // rows past the end repeat the last one
  const Factors f1 = factors_of(P.A1, P.B1, P.a1, P.K1, row, kq, bs);
  const bool two = P.K2 > 0;
  const Factors f2 = two ? factors_of(P.A2, P.B2, P.a2, P.K2, row, kq, bs) : f1;
  const int s1 = (f1.K + 15) >> 4;
  f64x2_a8* const slots = lds + (wave * cap) * (STEP_BYTES / 16) + lane;
  auto stage_steps = [&](const Factors& f, int kb, int ke, f64x2_a8* slot) {
#pragma nounroll
    for (int k0 = kb; k0 < ke; k0 += 16, slot += STEP_BYTES / 16) {
      if (f.a64) stage<DT_F64>(f, k0, kq, slot); else stage<DT_F32>(f, k0, kq, slot);
    }
  };
  if (KEEP) {
    stage_steps(f1, 0, f1.K, slots);
    if (two) stage_steps(f2, 0, f2.K, slots + s1 * (STEP_BYTES / 16));
  }
  const UpdCoef cf = make_coef(sc.lr, blk.lr_scale, blk.wd, sc.clip);
  const float ob2 = 1.f - sc.beta2;
  const float gs = grad_scale(bs);                                  // global clipping: the method sees gs * G
  float vg[4];
  if (!VEL) {
    const int vrows = (int)(blk.group_elems / N);                   // rows that share one v
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = i0 + 4 * q + kq;
      vg[q] = inv_denom_fast(vst[(i < M ? i : M - 1) / vrows], sc.inv_debias_v, sc.inv_debias_m, sc.eps);
    }
  }
  for (int tj = tile.tj; tj < tile.tj + tile.nj; ++tj) {
    // this lane's four columns: j .. j + 3, or, across the end of a row, its last four (the first `skip` of which another
    // lane updates)
    const int j = UT * tj + 4 * l16;
    const int col = j + 4 <= N ? j : N - 4;
    const int skip = j < N ? j - col : 4;
    // G, W and v of the lane's 4 x 4 elements are requested before the contraction and used behind it
    Raw4<GDT> gq[4];
    Raw4<WDT> wq[4];
    Raw4<DT_F32> vq[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = 4 * q + kq, ic = i0 + i < M ? i : M - 1 - i0;
      const unsigned e = (unsigned)ic * (unsigned)N + (unsigned)col;
      gq[q].load(G + e * elem_bytes(GDT));
      wq[q].load(W + e * elem_bytes(WDT));
      if (VEL) vq[q].load(V + e * 4u);
    }
    __builtin_amdgcn_sched_barrier(0);
    f64x4 acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
    auto add = [&](const Factors& f, int kb, int ke, const f64x2_a8* slot) {
      if (f.b64) multiply<DT_F64>(f, kb, ke, kq, col, slot, acc); else multiply<DT_F32>(f, kb, ke, kq, col, slot, acc);
      mfma_f64_results(acc);
    };
    if (KEEP) {
      add(f1, 0, f1.K, slots);
      if (two) add(f2, 0, f2.K, slots + s1 * (STEP_BYTES / 16));
    } else {
      for (int p = 0; p < (two ? 2 : 1); ++p) {
        const Factors& f = p ? f2 : f1;
        for (int kb = 0; kb < f.K; kb += 16 * cap) {
          const int ke = kb + 16 * cap < f.K ? kb + 16 * cap : f.K;
          stage_steps(f, kb, ke, slots);
          add(f, kb, ke, slots);
        }
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = 4 * q + kq;
      if (i0 + i >= M || skip >= 4) continue;
      const unsigned e = (unsigned)i * (unsigned)N + (unsigned)col;
      float g[4], w[4], vv[4];
      floats<GDT>(gq[q], g);
      floats<WDT>(wq[q], w);
      if (VEL) floats<DT_F32>(vq[q], vv);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        if (gs != 1.f) g[t] *= gs;
        float inv;
        if (VEL) {
          vv[t] = sc.beta2 * vv[t] + ob2 * g[t] * g[t];
          inv = inv_denom_fast(vv[t], sc.inv_debias_v, sc.inv_debias_m, sc.eps);
        } else {
          inv = vg[q];
        }
        w[t] = apply_update(w[t], sc.cG * g[t] + sc.cC * (float)acc[t][q], inv, cf);
      }
      if (skip == 0) {
        if (VEL) *reinterpret_cast<f32x4_a4*>(V + e * 4u) = f32x4_a4{vv[0], vv[1], vv[2], vv[3]};
        if constexpr (WDT == DT_BF16) *reinterpret_cast<u32x2_a2*>(W + e * 2u) = u32x2_a2{pack_bf16x2(w[0], w[1]), pack_bf16x2(w[2], w[3])};
        else *reinterpret_cast<f32x4_a4*>(W + e * 4u) = f32x4_a4{w[0], w[1], w[2], w[3]};
      } else {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          if (t < skip) continue;
          if (VEL) reinterpret_cast<float*>(V)[e + t] = vv[t];
          store_one(W, WDT, e + t, w[t]);
        }
      }
    }
  }
}

// Blocks whose rows are shorter than a lane's four columns, or so long that a wave's rows or a factor pass 4 GiB: one thread per
// element, the sums in fp64 one product after the other
__device__ __forceinline__ void update64_elements(const GemmProblem& P, const GemmTile& tile, const BlockDev& blk, const Bases& bs, const StepScalars& sc) {
  const int N = P.N, block = P.Out.ref.block;
  const char* G = global_ptr((const char*)bs.grads[block]);
  char* W = global_ptr((char*)bs.params[block]);
  float* v = reinterpret_cast<float*>(bs.state + blk.off_v);
  const float gs = grad_scale(bs);
  const UpdCoef cf = make_coef(sc.lr, blk.lr_scale, blk.wd, sc.clip);
  auto at = [&](const Mat& m, const char* base, int64_t r, int64_t c) {
    return m.dtype == DT_F64 ? reinterpret_cast<const double*>(base)[r * m.s0 + c * m.s1]
                             : (double)reinterpret_cast<const float*>(base)[r * m.s0 + c * m.s1];
  };
  // the elements that there are: rows of two or three columns fill one turn of the threads instead of one lane in twenty of sixteen
  // turns, each of them a chain of loads (300 x 3 at r = 2 beside small blocks, R held, 31.8 -> 12.9 us)
  const int nc = UT * tile.nj < N - UT * tile.tj ? UT * tile.nj : N - UT * tile.tj, nr = UT < P.M - UT * tile.ti ? UT : P.M - UT * tile.ti;
  for (int id = threadIdx.x; id < nr * nc; id += 64 * UW) {
    const int i = UT * tile.ti + id / nc, j = UT * tile.tj + id % nc;
    auto dot = [&](const Mat& A, const Mat& B, double alpha, int K, double s) {
      const char *a = resolve(A.ref, bs), *b = resolve(B.ref, bs);
      for (int k = 0; k < K; ++k) s = fma(alpha * at(A, a, i, k), at(B, b, k, j), s);
      return s;
    };
    double c = dot(P.A1, P.B1, P.a1, P.K1, 0.0);
    if (P.K2 > 0) c = dot(P.A2, P.B2, P.a2, P.K2, c);
    const int64_t e = (int64_t)i * N + j;
    const float g = gs * (blk.grad_dtype == DT_BF16 ? bf16lo((uint32_t)reinterpret_cast<const uint16_t*>(G)[e]) : reinterpret_cast<const float*>(G)[e]);
    const float w = blk.param_dtype == DT_BF16 ? bf16lo((uint32_t)reinterpret_cast<const uint16_t*>(W)[e]) : reinterpret_cast<const float*>(W)[e];
    float x;
    if (blk.v_mode == VM_ELEMENT) {
      x = sc.beta2 * v[e] + (1.f - sc.beta2) * g * g;
      v[e] = x;
    } else {
      x = v[i / (int)(blk.group_elems / N)];
    }
    const float inv = inv_denom_fast(x, sc.inv_debias_v, sc.inv_debias_m, sc.eps);
    store_one(W, blk.param_dtype, e, apply_update(w, sc.cG * g + sc.cC * (float)c, inv, cf));
  }
}

// One kernel per class of blocks (a table of one class is one launch)
template <int GDT, int WDT, bool VEL, bool KEEP>
__global__ __launch_bounds__(64 * UW, 3) void update64_kernel(const GemmProblem* __restrict__ probs, const GemmTile* __restrict__ tiles,
                                                              const BlockDev* __restrict__ blocks, Bases bs, StepScalars sc, int cap) {
  extern __shared__ __attribute__((aligned(16))) unsigned char upd_lds[];
  const GemmTile tile = tiles[blockIdx.x];
  if (tile.prob == GEMM_TILE_NONE) return;
  const GemmProblem& P = probs[tile.prob];
  update64_body<GDT, WDT, VEL, KEEP>(P, tile, blocks[P.Out.ref.block], bs, sc, cap, reinterpret_cast<f64x2_a8*>(upd_lds));
}

__global__ __launch_bounds__(64 * UW) void update64_elements_kernel(const GemmProblem* __restrict__ probs, const GemmTile* __restrict__ tiles,
                                                                    const BlockDev* __restrict__ blocks, Bases bs, StepScalars sc) {
  const GemmTile tile = tiles[blockIdx.x];
  if (tile.prob == GEMM_TILE_NONE) return;
  const GemmProblem& P = probs[tile.prob];
  update64_elements(P, tile, blocks[P.Out.ref.block], bs, sc);
}

// ... and one for all of them, for few tiles of several classes (UPD64_MIXED).  Its workgroups walk one tile, so that staging A by and by
// costs nothing.
__global__ __launch_bounds__(64 * UW, 2) void update64_mixed_kernel(const GemmProblem* __restrict__ probs, const GemmTile* __restrict__ tiles,
                                                                    const BlockDev* __restrict__ blocks, Bases bs, StepScalars sc, int cap) {
  extern __shared__ __attribute__((aligned(16))) unsigned char upd_lds[];
  const GemmTile tile = tiles[blockIdx.x];
  if (tile.prob == GEMM_TILE_NONE) return;
  const GemmProblem& P = probs[tile.prob];
  const BlockDev& blk = blocks[P.Out.ref.block];
  f64x2_a8* const lds = reinterpret_cast<f64x2_a8*>(upd_lds);
  switch (P.cls) {
    case 0: update64_body<DT_F32, DT_F32, false, false>(P, tile, blk, bs, sc, cap, lds); break;
    case 1: update64_body<DT_BF16, DT_F32, false, false>(P, tile, blk, bs, sc, cap, lds); break;
    case 2: update64_body<DT_F32, DT_BF16, false, false>(P, tile, blk, bs, sc, cap, lds); break;
    case 3: update64_body<DT_BF16, DT_BF16, false, false>(P, tile, blk, bs, sc, cap, lds); break;
    case 4: update64_body<DT_F32, DT_F32, true, false>(P, tile, blk, bs, sc, cap, lds); break;
    case 5: update64_body<DT_BF16, DT_F32, true, false>(P, tile, blk, bs, sc, cap, lds); break;
    case 6: update64_body<DT_F32, DT_BF16, true, false>(P, tile, blk, bs, sc, cap, lds); break;
    case 7: update64_body<DT_BF16, DT_BF16, true, false>(P, tile, blk, bs, sc, cap, lds); break;
    default: update64_elements(P, tile, blk, bs, sc);
  }
}

constexpr int CAP = 8;                         // steps of A in LDS: 64 KB, two workgroups per CU

template <int GDT, int WDT, bool VEL>
void launch_class(dim3 grid, int steps, const GemmProblem* probs, const GemmTile* tiles, const BlockDev* blocks, Bases b, StepScalars sc,
                  hipStream_t s) {
  if (steps <= CAP) {
    const int cap = steps < 1 ? 1 : steps;
    hipLaunchKernelGGL((update64_kernel<GDT, WDT, VEL, true>), grid, dim3(64 * UW), (size_t)UW * cap * STEP_BYTES, s, probs, tiles, blocks, b, sc, cap);
  } else {
    hipLaunchKernelGGL((update64_kernel<GDT, WDT, VEL, false>), grid, dim3(64 * UW), (size_t)UW * CAP * STEP_BYTES, s, probs, tiles, blocks, b, sc, CAP);
  }
}

}  // namespace

// Class of a block's update: 1 = bf16 G, 2 = bf16 W, 4 = per-element second moment, added up; 8 = one thread per element
int update64_class(int64_t N, int64_t K, bool g16, bool w16, bool vel) {
  if (N < 4 || (K > 16 ? K : 16) * N * 8 >= (1ll << 32)) return 8;
  return (g16 ? 1 : 0) + (w16 ? 2 : 0) + (vel ? 4 : 0);
}

// steps: most steps of 16 values of k that a block of the list contracts over (both products together)
void launch_update64(int cls, const GemmProblem* probs, const GemmTile* tiles, int64_t ntiles, int steps, const BlockDev* blocks, Bases b,
                     StepScalars sc, hipStream_t s) {
  if (ntiles <= 0) return;
  const dim3 grid((unsigned)ntiles);
  switch (cls) {
    case 0: launch_class<DT_F32, DT_F32, false>(grid, steps, probs, tiles, blocks, b, sc, s); break;
    case 1: launch_class<DT_BF16, DT_F32, false>(grid, steps, probs, tiles, blocks, b, sc, s); break;
    case 2: launch_class<DT_F32, DT_BF16, false>(grid, steps, probs, tiles, blocks, b, sc, s); break;
    case 3: launch_class<DT_BF16, DT_BF16, false>(grid, steps, probs, tiles, blocks, b, sc, s); break;
    case 4: launch_class<DT_F32, DT_F32, true>(grid, steps, probs, tiles, blocks, b, sc, s); break;
    case 5: launch_class<DT_BF16, DT_F32, true>(grid, steps, probs, tiles, blocks, b, sc, s); break;
    case 6: launch_class<DT_F32, DT_BF16, true>(grid, steps, probs, tiles, blocks, b, sc, s); break;
    case 7: launch_class<DT_BF16, DT_BF16, true>(grid, steps, probs, tiles, blocks, b, sc, s); break;
    case UPD64_MIXED: {
      const int cap = steps < 1 ? 1 : (steps < CAP ? steps : CAP);
      hipLaunchKernelGGL(update64_mixed_kernel, grid, dim3(64 * UW), (size_t)UW * cap * STEP_BYTES, s, probs, tiles, blocks, b, sc, cap);
      break;
    }
    default: hipLaunchKernelGGL(update64_elements_kernel, grid, dim3(64 * UW), 0, s, probs, tiles, blocks, b, sc);
  }
}

}  // namespace adapm
