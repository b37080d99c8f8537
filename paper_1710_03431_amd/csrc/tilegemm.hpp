// Tile products of the gradient sweep, and the operand layout that the fixed-step unraveling
// shares: a workgroup of kGW wavefronts holds TT trajectories as an LDS tile [NP][LD] (columns
// 2t, 2t + 1 = re, im of trajectory t) and multiplies it by NP x NP operands read from
// global memory on MFMA (FP32 or FP64 16x16x4).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>

namespace aqt {
namespace tile {

constexpr int kGW = 8;              // wavefronts per workgroup
constexpr int kGThreads = kGW * 64;

typedef float f4 __attribute__((ext_vector_type(4)));
typedef double d4 __attribute__((ext_vector_type(4)));

template <class T> struct Mfma;
template <> struct Mfma<float> {
  using acc_t = f4;
  __device__ static acc_t zero() { return f4{0.f, 0.f, 0.f, 0.f}; }
  __device__ static acc_t step(float a, float b, acc_t c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
  // element e of lane l holds output row 4 (l / 16) + e, column l % 16
  __device__ static int row(int lane, int e) { return 4 * (lane >> 4) + e; }
};
template <> struct Mfma<double> {
  using acc_t = d4;
  __device__ static acc_t zero() { return d4{0.0, 0.0, 0.0, 0.0}; }
  __device__ static acc_t step(double a, double b, acc_t c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
  // element e of lane l holds output row l / 16 + 4 e, column l % 16
  __device__ static int row(int lane, int e) { return (lane >> 4) + 4 * e; }
};

// Operand A of the products below: an NP x NP row-major matrix in the state precision
// (packed copies of O_g - I, its transpose and X_g), read straight into registers.  Each
// wave owns whole 16-row tiles; lane (r, q) of the 16 x 4 fragment grid loads VW
// consecutive entries A[row][k..k+VW) with one 16-byte load, so one MFMA step takes
// k = 4 VW j + VW q + e (e < VW) from lane q: any bijection of k onto (step, lane
// group) is a valid contraction as long as A and B use the same one.
template <class T> struct Vec;
template <> struct Vec<float> { using t = float __attribute__((ext_vector_type(4))); static constexpr int W = 4; };
template <> struct Vec<double> { using t = double __attribute__((ext_vector_type(2))); static constexpr int W = 2; };

// Products of A with NB LDS operands over the row tiles rt = wave (mod kGW) of each wave:
// done(i, rt, acc) takes the accumulators of its i-th row tile.  The panel comes in an even
// number of chunks and the next one (the next row tile's first at the end) is in flight while
// the current one is multiplied: loading a whole panel and waiting for it left the matrix
// cores idle for more than half of a product (256 levels FP32, one 16-trajectory product:
// 38000 cycles where the MFMAs take 16400).  With it, the wide tile copies and the sums read
// together, the gradient of 4096 FP32 trajectories over 500 points takes 44.0 ms against 52.6.
// The order in k is that of a plain loop.
template <int NP, int NC, int LD, class T, int NB, class Done>
__device__ __forceinline__ void panel_mma(const T* __restrict__ A, const T* const (&B)[NB], Done done) {
  constexpr int RT = NP / 16, CT = NC / 16;
  constexpr int VW = Vec<T>::W;
  constexpr int NJ = NP / (4 * VW);                // vector loads per lane for the whole panel
  constexpr int JCH = (NJ > 16) ? 8 : (NJ > 1 ? NJ / 2 : 1);
  constexpr int NCH = NJ / JCH, NBUF = NCH > 1 ? 2 : 1;
  static_assert(NCH == 1 || NCH % 2 == 0, "buffers alternate over whole panels");
  using V = typename Vec<T>::t;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, q = lane >> 4, c = lane & 15;
  V av[NBUF][JCH];
  auto load = [&](int rt, int ch, V* v) {
    const V* arow = reinterpret_cast<const V*>(A + static_cast<size_t>(rt * 16 + c) * NP) + q;
#pragma unroll
    for (int u = 0; u < JCH; ++u) v[u] = arow[(ch * JCH + u) * 4];
  };
  if (wave < RT) load(wave, 0, av[0]);
  int i = 0;
#pragma unroll 1
  for (int rt = wave; rt < RT; rt += kGW, ++i) {
    typename Mfma<T>::acc_t acc[NB][CT];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) acc[b][ct] = Mfma<T>::zero();
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
      const V* cur = av[ch % NBUF];
      if (NBUF == 2) {
        const bool last = ch + 1 == NCH;
        load(last ? (rt + kGW < RT ? rt + kGW : rt) : rt, last ? 0 : ch + 1, av[(ch + 1) % NBUF]);
        __builtin_amdgcn_sched_barrier(0);   // (else the loads sink to the products that use them)
      }
#pragma unroll
      for (int u = 0; u < JCH; ++u)
#pragma unroll
        for (int e = 0; e < VW; ++e) {
          const int k = (ch * JCH + u) * 4 * VW + q * VW + e;
#pragma unroll
          for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
              acc[b][ct] = Mfma<T>::step(cur[u][e], B[b][k * LD + ct * 16 + c], acc[b][ct]);
        }
    }
    if (NBUF == 1 && rt + kGW < RT) load(rt + kGW, 0, av[0]);
    done(i, rt, acc);
  }
}

// Y = (I + A) B over NP x NC (A = O_g - I or its transpose); B and Y in LDS, Y != B.
template <int NP, int NC, int LD, class T>
__device__ void gemm_kick(const T* __restrict__ A, const T* B, T* Y) {
  const int lane = threadIdx.x & 63, c = lane & 15;
  const T* const Bs[1] = {B};
  panel_mma<NP, NC, LD, T, 1>(A, Bs, [&](int, int rt, const typename Mfma<T>::acc_t (&acc)[1][NC / 16]) {
#pragma unroll
    for (int ct = 0; ct < NC / 16; ++ct)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = rt * 16 + Mfma<T>::row(lane, e), col = ct * 16 + c;
        Y[r * LD + col] = acc[0][ct][e] + B[r * LD + col];
      }
  });
}

// Y1 = (I + A) B1 and Y2 = (I + A) B2 with one pass over A (the panel loads are shared);
// each product is accumulated in the same order as gemm_kick's.
template <int NP, int NC, int LD, class T>
__device__ void gemm_kick2(const T* __restrict__ A, const T* B1, T* Y1, const T* B2, T* Y2) {
  const int lane = threadIdx.x & 63, c = lane & 15;
  const T* const Bs[2] = {B1, B2};
  panel_mma<NP, NC, LD, T, 2>(A, Bs, [&](int, int rt, const typename Mfma<T>::acc_t (&acc)[2][NC / 16]) {
#pragma unroll
    for (int ct = 0; ct < NC / 16; ++ct)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = rt * 16 + Mfma<T>::row(lane, e), col = ct * 16 + c;
        Y1[r * LD + col] = acc[0][ct][e] + B1[r * LD + col];
        Y2[r * LD + col] = acc[1][ct][e] + B2[r * LD + col];
      }
  });
}

// Copies between an LDS state tile (leading dimension LD) and a dense [NP][NC] block, 16
// bytes at a time in global memory, all of a thread's loads in flight at once (one value at
// a time took 18500 cycles of a 256-level step for 32 KB).
template <int NP, int NC, int LD, class T>
__device__ void tile_store(const T* src, T* __restrict__ dst) {
  using V = typename Vec<T>::t;
  constexpr int W = Vec<T>::W, N = NP * NC / W;
#pragma unroll
  for (int i = 0; i < (N + kGThreads - 1) / kGThreads; ++i) {
    const int f = threadIdx.x + i * kGThreads;
    if (N % kGThreads && f >= N) continue;
    const T* s = src + (f * W / NC) * LD + f * W % NC;
    V v;
#pragma unroll
    for (int e = 0; e < W; ++e) v[e] = s[e];
    reinterpret_cast<V*>(dst)[f] = v;
  }
}
template <int NP, int NC, int LD, class T>
__device__ void tile_load(const T* __restrict__ src, T* dst) {
  using V = typename Vec<T>::t;
  constexpr int W = Vec<T>::W, N = NP * NC / W, I = (N + kGThreads - 1) / kGThreads;
  V v[I];
#pragma unroll
  for (int i = 0; i < I; ++i) {
    const int f = threadIdx.x + i * kGThreads;
    v[i] = V{};
    if (N % kGThreads == 0 || f < N) v[i] = reinterpret_cast<const V*>(src)[f];
  }
#pragma unroll
  for (int i = 0; i < I; ++i) {
    const int f = threadIdx.x + i * kGThreads;
    if (N % kGThreads && f >= N) continue;
    T* d = dst + (f * W / NC) * LD + f * W % NC;
#pragma unroll
    for (int e = 0; e < W; ++e) d[e] = v[i][e];
  }
}

}  // namespace tile
}  // namespace aqt
