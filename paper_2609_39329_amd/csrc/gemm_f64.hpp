// fp64 product tile on MFMA 16x16x4 f64, shared by the fp64 statistics and the fp64 solve.
#pragma once

#include "common.hpp"

namespace pkv {
namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

// BM x BM output tile, 4 waves of BM/2 x BM/2; a K chunk of both operands is staged
// through registers into one of two [k][row] LDS buffers (the next chunk's loads are in
// flight while one is multiplied). Pitch BM + 1: a wave's fragment read touches 4 k rows
// of 16 consecutive doubles, the k-fastest stores land in different banks.
// Lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16] of each 16x16x4 step and holds
// D[4 e + l / 16][l % 16] in element e.
constexpr int kF64Kc = 32;
template <int BM>
struct F64Lds {
  static constexpr int P = BM + 1;
  double a[2][kF64Kc * P], b[2][kF64Kc * P];
};

// One operand of a tile: element (o, k), o < n, k < K, is (P - P2)[o * so + k * sk] (P2 may
// be null). Threads run along k when it is the contiguous index, else along o.
template <class T>
struct F64Operand {
  const T* P;
  const T* P2;
  int64_t so, sk;
  int n;  // valid outer indices from the tile's first (<= 0: none)
};
__device__ __forceinline__ double to_f64(double x) { return x; }
__device__ __forceinline__ double to_f64(float x) { return (double)x; }
__device__ __forceinline__ double to_f64(__bf16 x) { return (double)(float)x; }

// acc = sum over k < K of A(i, k) B(j, k) for the tile's rows i and columns j
template <int BM, class TA, class TB>
__device__ __forceinline__ void f64_tile(f64x4 (&acc)[BM / 32][BM / 32], int K,
                                         const F64Operand<TA>& A, const F64Operand<TB>& B,
                                         F64Lds<BM>& lds) {
  constexpr int KC = kF64Kc, P = F64Lds<BM>::P, W = BM / 32, NU = BM * KC / 256;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int wi = (wid >> 1) * (BM / 2), wj = (wid & 1) * (BM / 2);
  const int lk = lane >> 4, l16 = lane & 15;
#pragma unroll
  for (int a = 0; a < W; ++a)
#pragma unroll
    for (int b = 0; b < W; ++b) acc[a][b] = f64x4{};
  // element u of a thread: outer index o0 + u * ou, k index k0 + u * ku of the chunk
  // (one code path for both orders: the kernel is short, and its instruction fetch counts)
  const bool ak = A.sk == 1, bk = B.sk == 1;
  const int ao = ak ? tid / KC : tid % BM, aou = ak ? 256 / KC : 0;
  const int akk = ak ? tid % KC : tid / BM, aku = ak ? 0 : 256 / BM;
  const int bo = bk ? tid / KC : tid % BM, bou = bk ? 256 / KC : 0;
  const int bkk = bk ? tid % KC : tid / BM, bku = bk ? 0 : 256 / BM;
  const int64_t a0 = ao * A.so + akk * A.sk, au = aou * A.so + aku * A.sk;
  const int64_t b0 = bo * B.so + bkk * B.sk, bu = bou * B.so + bku * B.sk;
  // raw values, converted and masked at the LDS store: a chunk's loads are all issued
  // before the first is waited for (out-of-range elements load the tile's first one)
  TA ra[NU], ra2[NU];
  TB rb[NU], rb2[NU];
  bool ina[NU], inb[NU];
  auto fetch = [&](int kc) {
    const int64_t ca = a0 + (int64_t)kc * A.sk, cb = b0 + (int64_t)kc * B.sk;
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      ina[u] = ao + u * aou < A.n && kc + akk + u * aku < K;
      inb[u] = bo + u * bou < B.n && kc + bkk + u * bku < K;
      ra[u] = A.P[ina[u] ? ca + u * au : 0];
      rb[u] = B.P[inb[u] ? cb + u * bu : 0];
    }
    if (A.P2) {
#pragma unroll
      for (int u = 0; u < NU; ++u) ra2[u] = A.P2[ina[u] ? ca + u * au : 0];
    }
    if (B.P2) {
#pragma unroll
      for (int u = 0; u < NU; ++u) rb2[u] = B.P2[inb[u] ? cb + u * bu : 0];
    }
  };
  auto stash = [&](int buf) {
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const double v = to_f64(ra[u]) - (A.P2 ? to_f64(ra2[u]) : 0.0);
      const double w = to_f64(rb[u]) - (B.P2 ? to_f64(rb2[u]) : 0.0);
      lds.a[buf][(akk + u * aku) * P + ao + u * aou] = ina[u] ? v : 0.0;
      lds.b[buf][(bkk + u * bku) * P + bo + u * bou] = inb[u] ? w : 0.0;
    }
  };
  fetch(0);
  stash(0);
  __syncthreads();
  for (int kc = 0, buf = 0; kc < K; kc += KC, buf ^= 1) {
    if (kc + KC < K) fetch(kc + KC);
#pragma unroll
    for (int ks = 0; ks < KC; ks += 4) {
      double av[W], bv[W];
#pragma unroll
      for (int a = 0; a < W; ++a) av[a] = lds.a[buf][(ks + lk) * P + wi + 16 * a + l16];
#pragma unroll
      for (int b = 0; b < W; ++b) bv[b] = lds.b[buf][(ks + lk) * P + wj + 16 * b + l16];
#pragma unroll
      for (int a = 0; a < W; ++a)
#pragma unroll
        for (int b = 0; b < W; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a], bv[b], acc[a][b], 0, 0, 0);
    }
    // the other buffer was last read one barrier ago
    if (kc + KC < K) stash(buf ^ 1);
    __syncthreads();
  }
}

// f(i, j, v) for every element of the wave's part of the tile (tile coordinates)
template <int BM, class F>
__device__ __forceinline__ void f64_each(const f64x4 (&acc)[BM / 32][BM / 32], F f) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int wi = (wid >> 1) * (BM / 2), wj = (wid & 1) * (BM / 2);
#pragma unroll
  for (int a = 0; a < BM / 32; ++a)
#pragma unroll
    for (int b = 0; b < BM / 32; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        f(wi + 16 * a + 4 * e + (lane >> 4), wj + 16 * b + (lane & 15), acc[a][b][e]);
}

}  // namespace
}  // namespace pkv
