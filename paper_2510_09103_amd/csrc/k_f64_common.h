// Building blocks shared by the fp64 kernels of the exact contraction path (k_gemm64.hip, k_update64.hip) and of the
// re-expression of R (k_chol.hip): the fp64 matrix instruction, and operands that go from memory straight into its registers.
//
// v_mfma_f64_16x16x4_f64: lane l holds A[l % 16][l / 16] and B[l / 16][l % 16]; result register q of lane l is
// D[4 q + l / 16][l % 16].  One instruction is 64 cycles of a SIMD whatever the dependence on the previous one (measured:
// 68.5 TFLOP/s with one accumulator per wave, 72 with eight), the rate of the vector fp64 multiply-add, but its
// 2048 flop take one register pair per operand instead of a register tile fed from LDS.
//
// Which contraction index sits in which of the four slots of an instruction is free as long as A and B agree, and so is
// which free index sits in which lane as long as the store knows: a lane therefore takes V consecutive values of a
// contiguous contraction index (one wide load feeds V instructions: instruction v covers k0 + V (l / 16) + v), and T
// consecutive values of a contiguous free index (one load feeds T output tiles: tile t of lane l is index T (l % 16) + t).
// Every operand element is used once per wave, so nothing is staged in LDS; k_update64.hip, whose waves multiply the same rows of A
// with chunk after chunk of B, keeps those in LDS.
#pragma once
#include "adapm_plan.h"
#include "ew_math.h"

namespace adapm {
namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));
struct __attribute__((packed, aligned(8))) f64x2_a8 { double x, y; };
struct __attribute__((packed, aligned(4))) f32x2_a4 { float x, y; };
struct __attribute__((packed, aligned(2))) u32_a2 { uint32_t x; };
struct __attribute__((packed, aligned(2))) u32x2_a2 { uint32_t x, y; };

__device__ __forceinline__ f64x4 mfma_f64(double a, double b, f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Between the matrix instructions of a product and the first other use of its results.  The hardware does not interlock
// that read: it returns the registers' old contents until 19 wait states after the instruction.  The compiler is to fill them
// in, but has left 4 - 9 along branches from one matrix instruction to the next (rows 92 - 95 of a 96-row tile stale), so the
// source waits itself: 20 states, held in place by the two rows of ties.  What may still come before it are copies from
// register to register; tests/test_fp64_listings.py checks the distance of those in the listings of every build.
//
// The kernels ask for two or more waves per SIMD (two, three or four: 256, 168 or 128 registers at most), because the compiler
// lets the instruction work on ordinary registers up to 256.  With more it keeps the accumulators in the second half of the file and copies
// them there and back in every step of a loop, and every copy is such a read.
template <int N>
__device__ __forceinline__ void mfma_f64_tie(f64x4 (&acc)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) asm volatile("" : "+v"(acc[i]));
}
template <int M, int N>
__device__ __forceinline__ void mfma_f64_tie(f64x4 (&acc)[M][N]) {
#pragma unroll
  for (int i = 0; i < M; ++i) mfma_f64_tie(acc[i]);
}
template <class Acc>
__device__ __forceinline__ void mfma_f64_results(Acc& acc) {
  mfma_f64_tie(acc);
  asm volatile("; fp64 results\n\ts_nop 15\n\ts_nop 3");
  mfma_f64_tie(acc);
}

__host__ __device__ constexpr int elem_bytes(int dtype) { return dtype == DT_F64 ? 8 : (dtype == DT_F32 ? 4 : 2); }

// N consecutive elements as they lie in memory (raw: converted only where they are used, so that a load stays in flight)
template <int DT, int N>
struct RawVec;
template <int N>
struct RawVec<DT_F32, N> {
  float r[N];
  __device__ __forceinline__ void load(const char* p) {
    if constexpr (N % 4 == 0) {
#pragma unroll
      for (int i = 0; i < N / 4; ++i) {
        const f32x4_a4 q = reinterpret_cast<const f32x4_a4*>(p)[i];
        r[4 * i] = q.x; r[4 * i + 1] = q.y; r[4 * i + 2] = q.z; r[4 * i + 3] = q.w;
      }
    } else if constexpr (N == 2) {
      const f32x2_a4 q = *reinterpret_cast<const f32x2_a4*>(p);
      r[0] = q.x; r[1] = q.y;
    } else {
      r[0] = *reinterpret_cast<const float*>(p);
    }
  }
  __device__ __forceinline__ void load1(int i, const char* p) { r[i] = *reinterpret_cast<const float*>(p); }
  __device__ __forceinline__ double get(int i) const { return (double)r[i]; }
  __device__ __forceinline__ void zero(int i) { r[i] = 0.f; }
  __device__ __forceinline__ void move(int to, int from) { r[to] = r[from]; }
};
template <int N>
struct RawVec<DT_F64, N> {
  double r[N];
  __device__ __forceinline__ void load(const char* p) {
    if constexpr (N % 2 == 0) {
#pragma unroll
      for (int i = 0; i < N / 2; ++i) {
        const f64x2_a8 q = reinterpret_cast<const f64x2_a8*>(p)[i];
        r[2 * i] = q.x; r[2 * i + 1] = q.y;
      }
    } else {
      r[0] = *reinterpret_cast<const double*>(p);
    }
  }
  __device__ __forceinline__ void load1(int i, const char* p) { r[i] = *reinterpret_cast<const double*>(p); }
  __device__ __forceinline__ double get(int i) const { return r[i]; }
  __device__ __forceinline__ void zero(int i) { r[i] = 0.0; }
  __device__ __forceinline__ void move(int to, int from) { r[to] = r[from]; }
};
template <int N>
struct RawVec<DT_BF16, N> {
  static constexpr int W = (N + 1) / 2;
  uint32_t r[W];                       // packed pairs
  __device__ __forceinline__ void load(const char* p) {
    if constexpr (N % 8 == 0) {
#pragma unroll
      for (int i = 0; i < N / 8; ++i) {
        const u32x4_a2 q = reinterpret_cast<const u32x4_a2*>(p)[i];
        r[4 * i] = q.x; r[4 * i + 1] = q.y; r[4 * i + 2] = q.z; r[4 * i + 3] = q.w;
      }
    } else if constexpr (N == 4) {
      const u32x2_a2 q = *reinterpret_cast<const u32x2_a2*>(p);
      r[0] = q.x; r[1] = q.y;
    } else if constexpr (N == 2) {
      r[0] = reinterpret_cast<const u32_a2*>(p)->x;
    } else {
      static_assert(N == 1, "lengths that occur");
      r[0] = *reinterpret_cast<const uint16_t*>(p);
    }
  }
  // elements one at a time, in ascending order from 0
  __device__ __forceinline__ void load1(int i, const char* p) {
    const uint32_t h = *reinterpret_cast<const uint16_t*>(p);
    r[i / 2] = (i & 1) ? (r[i / 2] | (h << 16)) : h;
  }
  __device__ __forceinline__ double get(int i) const { return (double)((i & 1) ? bf16hi(r[i / 2]) : bf16lo(r[i / 2])); }
  __device__ __forceinline__ void zero(int i) { r[i / 2] &= (i & 1) ? 0x0000ffffu : 0xffff0000u; }
  __device__ __forceinline__ void move(int to, int from) {
    const uint32_t h = (from & 1) ? r[from / 2] >> 16 : r[from / 2] & 0xffffu;
    r[to / 2] = (to & 1) ? ((r[to / 2] & 0xffffu) | (h << 16)) : ((r[to / 2] & 0xffff0000u) | h);
  }
};

// One operand (free index u, contraction index k) of T tiles for one step of 4 V values of k: what one lane holds.
// KFAST: k is contiguous, tile t of lane l is u0 + 16 t + l % 16; otherwise u is contiguous and tile t is u0 + T (l % 16) + t.
template <int DT, int T, int V, bool KFAST>
struct Operand {
  static constexpr int ES = elem_bytes(DT);
  RawVec<DT, KFAST ? V : T> q[KFAST ? T : V];
  struct Where {                       // fixed per workgroup tile
    const char* p[KFAST ? T : 1];      // KFAST: row of each tile; otherwise the first of the lane's T columns; moved along by step()
    int64_t sk;                        // bytes from k to k + 1
    bool shift;                        // !KFAST, T = 2: the lane's last column is the last one that exists
  };
  static __device__ __forceinline__ Where where(const char* base, int64_t su, int64_t sk, int u0, int U, int l16) {
    Where w;
    w.shift = false;
    if constexpr (KFAST) {
      w.sk = ES;
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const int u = u0 + 16 * t + l16;
        w.p[t] = base + (int64_t)(u < U ? u : U - 1) * su * ES;
      }
    } else {
      // lanes beyond the edge repeat its last T columns; a lane that straddles it moves back by one and shifts
      w.sk = sk * ES;
      int u = u0 + T * l16;
      w.shift = T == 2 && u == U - 1;
      u = u > U - T ? (U - T > 0 ? U - T : 0) : u;
      w.p[0] = base + (int64_t)u * ES;
    }
    return w;
  }
  // on by k values
  static __device__ __forceinline__ void step(Where& w, int k) {
#pragma unroll
    for (int t = 0; t < (KFAST ? T : 1); ++t) w.p[t] += (int64_t)k * w.sk;
  }
  // from this lane's first value of the contraction index, where w stands
  __device__ __forceinline__ void load(const Where& w) {
    if constexpr (KFAST) {
#pragma unroll
      for (int t = 0; t < T; ++t) q[t].load(w.p[t]);
    } else {
#pragma unroll
      for (int v = 0; v < V; ++v) q[v].load(w.p[0] + v * w.sk);
    }
  }
  // a step that ends at or beyond ke, k: this lane's first value of it (w stands at the row's start): values past the end read
  // a valid element and become zero
  __device__ __forceinline__ void load_edge(const Where& w, int k, int ke) {
    if constexpr (KFAST) {
#pragma unroll
      for (int t = 0; t < T; ++t)
#pragma unroll
        for (int v = 0; v < V; ++v) q[t].load1(v, w.p[t] + (int64_t)(k + v < ke ? k + v : ke - 1) * ES);
#pragma unroll
      for (int t = 0; t < T; ++t)
#pragma unroll
        for (int v = 0; v < V; ++v)
          if (k + v >= ke) q[t].zero(v);
    } else {
#pragma unroll
      for (int v = 0; v < V; ++v) q[v].load(w.p[0] + (int64_t)(k + v < ke ? k + v : ke - 1) * w.sk);
#pragma unroll
      for (int v = 0; v < V; ++v)
        if (k + v >= ke) {
#pragma unroll
          for (int t = 0; t < T; ++t) q[v].zero(t);
        }
    }
  }
  __device__ __forceinline__ double get(const Where& w, int t, int v) const {
    if constexpr (KFAST) return q[t].get(v);
    else if constexpr (T == 2) return (t == 0 && w.shift) ? q[v].get(1) : q[v].get(t);
    else return q[v].get(t);
  }
};

}  // namespace
}  // namespace adapm
