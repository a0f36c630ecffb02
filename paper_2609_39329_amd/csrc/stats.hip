// Targets and sufficient statistics (Eq. 5 and Eq. 9, row form):
//   T = (O_f - O_c) W + rho (O_f - O_c)
//   G (+)= X^T X,   C (+)= X^T (Yf - Yc)
// and the MLP-shaped block (Sec. 2.2; Alg. 1): SwiGLU features of the RMS-normed
// attention output, targets through the down-projection plus the attention
// residual, and the student state through the patched block.
//
// fp32-accumulate path: split pre-passes + bgemm_kernel (bf16 MFMA, fp32 accumulation).
// fp64-accumulate path (f64_gemm_kernel): fp64 MFMA tiles through LDS.
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "gemm_f64.hpp"
#include "kernels.hpp"

namespace pkv {

namespace {

// ---------------------------------------------------------------- fp32 path
//
// Every fp32 operand x is first split, once, into x_hi = bf16(x) and
// x_lo = bf16(x - x_hi) by a memory-bound pre-pass that also lays it out with the
// contraction index contiguous and zero-pads both dimensions (rows to 128, the
// contraction to 64). The products then run on one bf16 MFMA GEMM kernel that sums
// several (A_t, B_t) term pairs with fp32 accumulation:
//   x y ~ x_hi y_hi + x_hi y_lo + x_lo y_hi (+ x_lo y_lo for the Gram matrix).
// Dropping x_lo y_lo in G would subtract a PSD matrix L^T L whose diagonal grows
// with the number of rows (a systematic shift of the ridge), so G keeps all four
// products; C keeps three (its lo x lo cross term has no such bias). A bf16 operand
// (W) has no low part.

constexpr int G_BM = 256, G_KC = 64;  // row and contraction padding of the split planes

inline int64_t pad_to(int64_t x, int64_t m) { return (x + m - 1) / m * m; }

// dst[r][c] (r < rows_p, c < cols_p), hi and lo planes, = split(S1 - S2)[r][c] inside
// rows x cols, zero outside. One thread per 8 consecutive columns.
__global__ __launch_bounds__(256) void split_rows_kernel(const float* __restrict__ S1,
                                                         const float* __restrict__ S2, int rows,
                                                         int cols, int64_t ld, __bf16* __restrict__ hi,
                                                         __bf16* __restrict__ lo, int rows_p,
                                                         int cols_p) {
  const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int per_row = cols_p / 8;
  if (g >= (int64_t)rows_p * per_row) return;
  const int r = (int)(g / per_row), c0 = (int)(g % per_row) * 8;
  float v[8];
  const bool vec = (ld & 3) == 0 && (((uintptr_t)S1 | (uintptr_t)S2) & 15) == 0;
  if (r < rows && c0 + 7 < cols && vec) {
    const f32x4* p1 = (const f32x4*)(S1 + (int64_t)r * ld + c0);
    f32x4 a = p1[0], b = p1[1];
    if (S2) {
      const f32x4* p2 = (const f32x4*)(S2 + (int64_t)r * ld + c0);
      a -= p2[0];
      b -= p2[1];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[e] = a[e];
      v[4 + e] = b[e];
    }
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int c = c0 + e;
      v[e] = (r < rows && c < cols)
                 ? S1[(int64_t)r * ld + c] - (S2 ? S2[(int64_t)r * ld + c] : 0.f)
                 : 0.f;
    }
  }
  bf16x8 h, l;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    h[e] = to_bf16(v[e]);
    l[e] = to_bf16(v[e] - (float)h[e]);
  }
  const int64_t o = (int64_t)r * cols_p + c0;
  *(bf16x8*)(hi + o) = h;
  *(bf16x8*)(lo + o) = l;
}

// dst[c][r] (c < cols_p, r < rows_p) = split(S1 + s2 S2)[r][c] inside rows x cols,
// zero outside: the transpose, through a 128 x 64 LDS tile (s2 = -1: a difference,
// +1: a bf16 weight plus an fp32 patch). SRC float (hi and lo planes,
// lo may be null for a bf16 source) or bf16 (hi plane only). Each thread reads 4
// consecutive source columns (one vector load when vec is set: S1, S2 and ld allow
// it), and 16 threads write one 256-byte run of a destination row. pair >= 0: one of two
// matrices interleaved in blocks of 32 destination rows, 64 apart, from row pair on.
template <class SRC>
__global__ __launch_bounds__(256) void split_transpose_kernel(const SRC* __restrict__ S1,
                                                              const float* __restrict__ S2, float s2,
                                                              int rows, int cols, int64_t ld,
                                                              __bf16* __restrict__ hi,
                                                              __bf16* __restrict__ lo, int rows_p,
                                                              int cols_p, int vec, int pair) {
  constexpr int TR = 128, TC = 64;
  __shared__ float tile[TR][TC + 1];
  const int r0 = blockIdx.y * TR, c0 = blockIdx.x * TC;
  const int tid = threadIdx.x;
#pragma unroll
  for (int u = 0; u < TR * TC / 4 / 256; ++u) {
    const int e = u * 256 + tid;
    const int rr = e / 16, cc = (e % 16) * 4;
    const int r = r0 + rr, c = c0 + cc;
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    if (r < rows) {
      const int64_t o = (int64_t)r * ld + c;
      if (vec && c + 3 < cols) {
        if constexpr (std::is_same<SRC, float>::value) {
          const f32x4 x = *(const f32x4*)(S1 + o);
#pragma unroll
          for (int t = 0; t < 4; ++t) v[t] = x[t];
        } else {
          const bf16x4 x = *(const bf16x4*)(S1 + o);
#pragma unroll
          for (int t = 0; t < 4; ++t) v[t] = (float)x[t];
        }
        if (S2) {
          const f32x4 y = *(const f32x4*)(S2 + o);
#pragma unroll
          for (int t = 0; t < 4; ++t) v[t] = fmaf(s2, y[t], v[t]);
        }
      } else {
#pragma unroll
        for (int t = 0; t < 4; ++t)
          if (c + t < cols) {
            v[t] = (float)S1[o + t];
            if (S2) v[t] = fmaf(s2, S2[o + t], v[t]);
          }
      }
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) tile[rr][cc + t] = v[t];
  }
  __syncthreads();
  // row c of dst: 128 consecutive r as 16 chunks of 8 bf16
#pragma unroll
  for (int u = 0; u < TR * TC / 8 / 256; ++u) {
    const int e = u * 256 + tid;
    const int cc = e / 16, rr0 = (e % 16) * 8;
    const int c = c0 + cc;
    if (c >= cols_p || r0 + rr0 >= rows_p) continue;
    bf16x8 h, l;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const float v = tile[rr0 + t][cc];
      h[t] = to_bf16(v);
      l[t] = to_bf16(v - (float)h[t]);
    }
    const int row = pair < 0 ? c : (c / 32) * 64 + pair + c % 32;
    const int64_t o = (int64_t)row * rows_p + r0 + rr0;
    *(bf16x8*)(hi + o) = h;
    if (lo) *(bf16x8*)(lo + o) = l;
  }
}

// dst[c][r] = S[r][c] for a bf16 source of whole 16-byte row pieces (cols, ld multiples of 8,
// aligned), zero outside; destination rows as split_transpose_kernel's. Memory bound: a lane
// loads an 8 x 8 block (8 row pieces in flight), transposes it in registers and stores 8
// pieces of destination rows; a wave's 8 x 8 lanes read and write whole 128-byte lines.
// 4096 x 14336: 52 us (4.5 TB/s; 75 through a float tile in LDS).
__global__ __launch_bounds__(256) void transpose_bf16_kernel(const __bf16* __restrict__ S, int rows,
                                                             int cols, int64_t ld,
                                                             __bf16* __restrict__ dst, int rows_p,
                                                             int cols_p, int pair) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int r0 = blockIdx.y * 128 + (wid >> 1) * 64 + (lane >> 3) * 8;
  const int c0 = blockIdx.x * 128 + (wid & 1) * 64 + (lane & 7) * 8;
  if (r0 >= rows_p || c0 >= cols_p) return;
  u32x4 in[8];
#pragma unroll
  for (int i = 0; i < 8; ++i)
    in[i] = r0 + i < rows && c0 < cols ? *(const u32x4*)(S + (int64_t)(r0 + i) * ld + c0) : u32x4{};
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    u32x4 v;
#pragma unroll
    for (int k = 0; k < 4; ++k)  // rows 2 k, 2 k + 1 of column c
      v[k] = __builtin_amdgcn_perm(in[2 * k + 1][c / 2], in[2 * k][c / 2], c % 2 ? 0x07060302u : 0x05040100u);
    const int row = pair < 0 ? c0 + c : ((c0 + c) / 32) * 64 + pair + (c0 + c) % 32;
    *(u32x4*)(dst + (int64_t)row * rows_p + r0) = v;
  }
}

// Out[i][j] (+)= sum_t sum_k A_{a(t)}[i][k] B_{b(t)}[j][k] (+ rho (E1 - E2)[i][j]).
// The operands are up to two bf16 planes per side (hi, lo), each [rows_p][Kp] with
// the contraction index contiguous and zero padding (rows_p a multiple of G_BM, Kp of
// 64), so the main loop has no bounds checks. Each K chunk loads every plane once and
// applies all term products to it: term t multiplies plane a(t) = bit t of TA with
// plane b(t) = bit t of TB. The MFMA computes the transposed tile (rows = output
// columns), so a lane owns 4 consecutive output columns and the epilogue uses 16-byte
// accesses. SYM: only tiles with tile_i <= tile_j; the diagonal tiles keep their i <= j
// half and every tile is mirrored, so the result is exactly symmetric.
//
// Tile shapes (BgCfg), eight waves each. The products are bound by LDS reads and the barrier
// per chunk next to the MFMAs, so a wave's tile is wide on the side with fewer planes, and
// the next 16 k are read from LDS while the current ones are multiplied (u [Wg | Wu] of the
// MLP at M = 4096, 1.92 TFLOP of MFMA work: 1.57 -> 1.42 ms):
//   256 x 256, waves of 128 x 64 (64 x 128 with two A planes and one B plane), two or three
//     stages: one tile per CU fills the chip for a 4096 x 4096 output;
//   128 x 256 and 128 x 128, waves of 64 x 64 and 64 x 32: outputs of fewer tiles;
//   symmetric products, 192 x 192: two waves per 96 x 96 quadrant (nine accumulators
//     each): wave w takes the first 16 k of every 32-k chunk, wave w + 4 (on the same
//     SIMD) the second 16, and the two partial tiles are summed once at the end through
//     LDS. Three LDS stages; waves 0-3 load the A planes, waves 4-7 the B planes. A
//     4096-wide triangle is 253 tiles of 192 (one round on 256 CUs) against 136 of 256.
// A tile's K chunk goes from HBM straight into LDS (buffer_load ... lds; no staging
// registers) while earlier chunks are multiplied. Rows past a plane's end (the last
// 192-tile reaches past a 256-padded plane) read as zeros through the buffer range.
struct BGemm {
  const __bf16* A[2];  // planes of A [Ip][Kp]
  const __bf16* B[2];  // planes of B [Jp][Kp]; BNAT: the bf16 gate and up matrices, [K][ldb]
  int64_t ld;          // Kp
  int64_t ldb;         // BNAT: row length of B
  int K;               // BNAT: rows of B
  float* Out;
  int64_t ldo;
  const float* E1;
  const float* E2;
  int64_t lde;
  float rho;
  int I, J, Kp;
  int accumulate;
  int tiles_j, ntiles;
  int vec_out, vec_in;  // 16-byte accesses to Out, of E1 and E2
};

constexpr int BG_KC = 32;    // contraction chunk per LDS stage
constexpr int BG_GROUP = 4;  // tile rows per group of the non-symmetric tile order
// TI x TJ output tile of waves of WM x WN, S LDS stages, KSP waves per wave tile (each a
// part of the k range)
template <int TI_, int TJ_, int WM_, int WN_, int S_, int KSP_>
struct BgCfg {
  static constexpr int TI = TI_, TJ = TJ_, WM = WM_, WN = WN_, S = S_, KSP = KSP_;
  static constexpr int NTH = (TI / WM) * (TJ / WN) * KSP * 64;
};
using BgSym = BgCfg<192, 192, 96, 96, 3, 2>;

template <class CFG, int NA, int NB, int NT, int TA, int TB, bool SYM, bool BNAT, bool SWIGLU>
__global__ __launch_bounds__(CFG::NTH, 1) void bgemm_kernel(BGemm p) {
  static_assert(!BNAT || (SWIGLU && NB == 1 && CFG::KSP == 1 && CFG::NTH == 512), "gate and up as stored");
  static_assert(!SWIGLU || (!SYM && (CFG::WN / 32) % 2 == 0), "gate and up blocks side by side");
  constexpr int TI = CFG::TI, TJ = CFG::TJ, WM = CFG::WM, WN = CFG::WN, S = CFG::S;
  constexpr int KSP = CFG::KSP, NTH = CFG::NTH;
  constexpr int ROWS = NA * TI + NB * TJ;          // stacked plane rows per stage
  // KSP = 1: all threads load every plane; KSP = 2: threads [0, NTH/2) the A planes,
  // [NTH/2, NTH) the B planes
  constexpr int LTH = KSP == 1 ? NTH : NTH / 2;    // threads loading one plane
  constexpr int RPU = LTH / 4;                     // rows per load round (4 chunks per row)
  constexpr int PPA = TI / RPU, PPB = TJ / RPU;    // load rounds per A, B plane
  constexpr int LPT = ROWS * (BG_KC / 8) / NTH;    // 16-byte loads per thread per stage
  constexpr int MA = WM / 32, MB = WN / 32;
  static_assert(KSP == 1 || (KSP == 2 && NA == NB && TI == TJ), "split loads: as many A as B rows");
  static_assert(TI % RPU == 0 && TJ % RPU == 0, "whole load rounds per plane");
  static_assert(LPT == (KSP == 1 ? NA * PPA + NB * PPB : NA * PPA), "whole load rounds per stage");
  static_assert(BG_KC == 32 && (KSP == 1 || KSP == 2), "one or two 16-k halves per chunk");
  static_assert(WM % 16 == 0 && WN % 16 == 0 && TI % 16 == 0 && TJ % 16 == 0,
                "fragment rows aligned to the swizzle");
  static_assert(S * ROWS * BG_KC * 2 <= 160 * 1024, "the stages fit in LDS");
  __shared__ __attribute__((aligned(16))) __bf16 lds[S][ROWS * BG_KC];
  int ti, tj;
  {
    const int t = xcd_item((p.ntiles + kXcds - 1) / kXcds);
    if (t >= p.ntiles) return;
    if constexpr (SYM) {
      int r = 0, rem = t;
      while (rem >= p.tiles_j - r) {
        rem -= p.tiles_j - r;
        ++r;
      }
      ti = r;
      tj = r + rem;
    } else {
      // groups of BG_GROUP tile rows, column by column inside a group: the run of items
      // one XCD takes covers few tile rows and few tile columns, so its L2 serves more
      // of the operand re-reads
      const int tiles_i = p.ntiles / p.tiles_j;
      const int per_group = BG_GROUP * p.tiles_j;
      const int first = (t / per_group) * BG_GROUP;
      const int rows = min(BG_GROUP, tiles_i - first);
      const int r = t % per_group;
      ti = first + r % rows;
      tj = r / rows;
    }
  }
  const int i0 = ti * TI, j0 = tj * TJ;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int h32 = lane >> 5, l32 = lane & 31;
  constexpr int NQW = (TI / WM) * (TJ / WN);  // waves per k half
  const int wq = wid % NQW, kh = wid / NQW;  // output block, k half (KSP = 2)
  const int wi = (wq / (TJ / WN)) * WM, wj = (wq % (TJ / WN)) * WN;
  const int nq = p.Kp / BG_KC;

  f32x16 acc[MA][MB];
#pragma unroll
  for (int a = 0; a < MA; ++a)
#pragma unroll
    for (int b = 0; b < MB; ++b) acc[a][b] = f32x16{};

  // Stages of unpadded [stacked row][32 k] tiles. LDS position c of a stage (16 bytes)
  // holds stacked row c / 4, k chunk (c % 4) ^ ((row / 4) % 4): the 16 consecutive rows
  // an MFMA fragment read takes at one k chunk land in 16 different bank groups. Load u
  // (u < LPT) of thread tid fills stacked row u * RPU + tid / 4 (KSP = 1), or row
  // (u % PPA) * RPU + lt / 4 of plane (tid < NTH/2 ? 0 : NA) + u / PPA (KSP = 2;
  // lt = tid % (NTH/2)).
  // buffer descriptors of the planes' rows of this tile (unused ones repeat plane 0;
  // plain variables: the host pass drops the kernel if a descriptor is a temporary);
  // the planes hold pad(I) and pad(J) rows, pad = G_BM
  const int ip = (p.I + G_BM - 1) / G_BM * G_BM, jp = (p.J + G_BM - 1) / G_BM * G_BM;
  auto plane_base = [&](int pl) {
    return pl < NA ? p.A[pl] + (int64_t)i0 * p.ld : p.B[pl - NA] + (BNAT ? 0 : (int64_t)j0 * p.ld);
  };
  auto plane_bytes = [&](int pl) {
    return (uint32_t)((pl < NA ? min(TI, ip - i0) : min(TJ, jp - j0)) * p.ld * 2);
  };
  const __amdgpu_buffer_rsrc_t rs0 =
      __builtin_amdgcn_make_buffer_rsrc((void*)plane_base(0), 0, plane_bytes(0), 0x00020000);
  const __amdgpu_buffer_rsrc_t rs1 = __builtin_amdgcn_make_buffer_rsrc(
      (void*)plane_base(NA + NB > 1 ? 1 : 0), 0, plane_bytes(NA + NB > 1 ? 1 : 0), 0x00020000);
  const __amdgpu_buffer_rsrc_t rs2 = __builtin_amdgcn_make_buffer_rsrc(
      (void*)plane_base(NA + NB > 2 ? 2 : 0), 0, plane_bytes(NA + NB > 2 ? 2 : 0), 0x00020000);
  const __amdgpu_buffer_rsrc_t rs3 = __builtin_amdgcn_make_buffer_rsrc(
      (void*)plane_base(NA + NB > 3 ? 3 : 0), 0, plane_bytes(NA + NB > 3 ? 3 : 0), 0x00020000);
  static_assert(NA + NB <= 4, "at most four planes");
  const int lt = tid % LTH, lw = lt / 64;  // thread and wave within the loading group
  const uint32_t voff0 = (uint32_t)(((lt / 4) * p.ld + (((lt % 4) ^ ((lt / 16) % 4)) * 8)) * 2);
  // BNAT: B's chunk as stored, in sub-tiles [TJ / 32][32 k][32 columns] of 64-byte rows:
  // 16-byte chunk c of the stage's B part holds k (c / 4) % 32, columns 8 (c % 4) .. of
  // sub-tile c / 128. The sub-tiles alternate between gate and up (a wave's 64 chunks lie in
  // one sub-tile of fixed parity). Rows past K read as zeros through the
  // buffer range (the row offset is in the lane's offset: the range check leaves the scalar
  // offset out); columns past ldb run into the next row and are never stored.
  const int bw = BNAT ? (__builtin_amdgcn_readfirstlane(wid) >> 1) & 1 : 0;
  const int jcol = j0 / 2;  // first column of this tile in the stored matrices
  const __bf16* bn = p.B[bw] + jcol;
  const uint32_t bn_bytes = BNAT ? (uint32_t)(((int64_t)p.K * p.ldb - jcol) * 2) : 0;
  const __amdgpu_buffer_rsrc_t rsb =
      __builtin_amdgcn_make_buffer_rsrc((void*)bn, 0, bn_bytes, 0x00020000);
  const uint32_t voffb =
      (uint32_t)(((tid >> 2) & 31) * p.ldb + (tid >> 8) * 32 + (tid & 3) * 8) * 2;
  auto issue = [&](int q, int buf) {
    const uint32_t k0b = (uint32_t)(q * BG_KC * 2);
    static_for<LPT>([&](auto u_t) {
      constexpr int u = decltype(u_t)::value;
      // KSP = 1: the stacked rows of A's planes, then B's; KSP = 2: one side's planes
      constexpr bool in_a = u < NA * PPA;
      constexpr int ur = KSP == 1 && !in_a ? (u - NA * PPA) % PPB : u % PPA;  // round in the plane
      const uint32_t vo = voff0 + (uint32_t)(ur * RPU * p.ld * 2);
      if constexpr (BNAT && !in_a) {
        PKV_LDS void* dst = (PKV_LDS void*)&lds[buf][(u * NTH + wid * 64) * 8];
        const uint32_t vb = voffb + (uint32_t)((u - NA * PPA) * 2 * 64) +
                            (uint32_t)(q * BG_KC) * (uint32_t)(p.ldb * 2);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsb, dst, 16, vb, 0, 0, 0);
      } else if constexpr (KSP == 1) {
        constexpr int pl = in_a ? u / PPA : NA + (u - NA * PPA) / PPB;
        PKV_LDS void* dst = (PKV_LDS void*)&lds[buf][(u * NTH + wid * 64) * 8];
        if constexpr (pl == 0) __builtin_amdgcn_raw_ptr_buffer_load_lds(rs0, dst, 16, vo, k0b, 0, 0);
        else if constexpr (pl == 1) __builtin_amdgcn_raw_ptr_buffer_load_lds(rs1, dst, 16, vo, k0b, 0, 0);
        else if constexpr (pl == 2) __builtin_amdgcn_raw_ptr_buffer_load_lds(rs2, dst, 16, vo, k0b, 0, 0);
        else __builtin_amdgcn_raw_ptr_buffer_load_lds(rs3, dst, 16, vo, k0b, 0, 0);
      } else {
        // a wave's 64 lanes fill 16 rows (1 KB) of one plane; which plane is wave-uniform
        constexpr int pu = u / PPA;  // plane within the side (hi or lo)
        const int row = (u % PPA) * RPU + lw * 16;
        if (__builtin_amdgcn_readfirstlane(wid) < NTH / 128) {
          PKV_LDS void* dst = (PKV_LDS void*)&lds[buf][(pu * TI + row) * BG_KC];
          if constexpr (pu == 0) __builtin_amdgcn_raw_ptr_buffer_load_lds(rs0, dst, 16, vo, k0b, 0, 0);
          else __builtin_amdgcn_raw_ptr_buffer_load_lds(rs1, dst, 16, vo, k0b, 0, 0);
        } else {
          PKV_LDS void* dst = (PKV_LDS void*)&lds[buf][(NA * TI + pu * TJ + row) * BG_KC];
          if constexpr (pu == 0) __builtin_amdgcn_raw_ptr_buffer_load_lds(rs2, dst, 16, vo, k0b, 0, 0);
          else __builtin_amdgcn_raw_ptr_buffer_load_lds(rs3, dst, 16, vo, k0b, 0, 0);
        }
      }
    });
  };
  // at most N of this wave's loads still in flight (the chunks issued after the one
  // needed next), then a plain barrier (the workgroup fence of __syncthreads adds
  // nothing here)
  auto landed = [&](auto n_t) {
    constexpr int N = decltype(n_t)::value;
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
  };
  const int sw = (l32 / 4) % 4;
  const int bn_lane = (8 * h32 + ((lane & 15) >> 2)) * 32 + ((lane >> 4) & 1) * 16 + (lane & 3) * 4;
  // the fragments of the 16 k at ks of the chunk in stage st
  struct Frags {
    bf16x8 a[NA][MA], b[NB][MB];
  };
  auto read = [&](Frags& f, int st, int ks) {
    const __bf16* L0 = lds[st];
    const int ch = ((2 * (ks / 16) + h32) ^ sw) * 8;  // k chunk of this lane, swizzled
#pragma unroll
    for (int pa = 0; pa < NA; ++pa)
#pragma unroll
      for (int a = 0; a < MA; ++a)
        f.a[pa][a] = *(const bf16x8*)(L0 + (pa * TI + wi + 32 * a + l32) * BG_KC + ch);
#pragma unroll
    for (int pb = 0; pb < NB; ++pb)
#pragma unroll
      for (int b = 0; b < MB; ++b) {
        if constexpr (BNAT) {
          // two transposing reads: lane 4 r + q of a 16-lane group points at k row r,
          // columns 4 q .. of a 4 x 16 block; a half-wave reads 256 contiguous bytes
          const PKV_LDS __bf16* t = (const PKV_LDS __bf16*)(L0 + NA * TI * BG_KC + (wj / 32 + b) * (32 * 32) +
                                                            ks * 32 + bn_lane);
          f.b[pb][b] = cat8(lds_read_tr16(t), lds_read_tr16(t + 4 * 32));
        } else {
          f.b[pb][b] = *(const bf16x8*)(L0 + (NA * TI + pb * TJ + wj + 32 * b + l32) * BG_KC + ch);
        }
      }
  };
  auto mult = [&](const Frags& f) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int a = 0; a < MA; ++a)
#pragma unroll
        for (int b = 0; b < MB; ++b)
          acc[a][b] = mfma32(f.b[(TB >> t) & 1][b], f.a[(TA >> t) & 1][a], acc[a][b]);
  };

  // Chunk q in stage q % S; S chunks in flight at first. The fragments of the next 16 k are
  // read while the current ones are multiplied, across the barrier too: the barrier in
  // the middle of step q says that every wave has read chunk q (its stage takes chunk
  // q + S) and that chunk q + 1 has landed (the S - 2 chunks after it may be in flight).
  static_for<S>([&](auto q_t) {
    if (decltype(q_t)::value < nq) issue(decltype(q_t)::value, decltype(q_t)::value);
  });
  if (nq >= S) landed(std::integral_constant<int, (S - 1) * LPT>{});
  else landed(std::integral_constant<int, 0>{});
  Frags f[KSP == 1 ? 2 : 1];
  if constexpr (KSP == 1) read(f[0], 0, 0);
  auto step = [&](int q, auto st_t, auto tail_t) {
    constexpr int st = decltype(st_t)::value, sn = (st + 1) % S;
    constexpr bool TAIL = decltype(tail_t)::value;
    auto next = [&]() {
      if (!TAIL || q + S - 1 < nq) landed(std::integral_constant<int, (S - 2) * LPT>{});
      else landed(std::integral_constant<int, 0>{});
      if (!TAIL || q + S < nq) issue(q + S, st);
    };
    if constexpr (KSP == 1) {
      read(f[1], st, 16);
      mult(f[0]);
      next();
      // (past the last chunk too, unused: a branch around these reads would make the
      // products below wait for all of them)
      read(f[0], sn, 0);
      mult(f[1]);
    } else {
      read(f[0], st, 16 * kh);  // (a second set of fragments would not fit in registers)
      mult(f[0]);
      next();
    }
  };
  int q0 = 0;
  for (; q0 + 2 * S - 1 < nq; q0 += S)
    static_for<S>([&](auto s_t) { step(q0 + decltype(s_t)::value, s_t, std::false_type{}); });
  for (; q0 < nq; q0 += S)
    static_for<S>([&](auto s_t) {
      if (q0 + decltype(s_t)::value < nq) step(q0 + decltype(s_t)::value, s_t, std::true_type{});
    });
  // KSP = 2: the second k half's partial tile goes through the (now idle) stages,
  // lane-major per register (a wave's 64 lanes write and read 256 consecutive bytes),
  // and is added in the epilogue, four values at a time
  static_assert(KSP == 1 || NQW * MA * MB * 16 * 64 * 4 <= (int)sizeof(lds), "partial tiles fit the stages");
  const float* part = (const float*)&lds[0][0] + wq * (MA * MB * 16 * 64);
  if constexpr (KSP == 2) {
    if (kh == 1) {
      float* pw = (float*)&lds[0][0] + wq * (MA * MB * 16 * 64);
#pragma unroll
      for (int a = 0; a < MA; ++a)
#pragma unroll
        for (int b = 0; b < MB; ++b)
#pragma unroll
          for (int e = 0; e < 16; ++e) pw[((a * MB + b) * 16 + e) * 64 + lane] = acc[a][b][e];
    }
    __syncthreads();
    if (kh == 1) return;
  }

  if constexpr (SWIGLU) {
    // column blocks 2 b and 2 b + 1 of the tile hold gate and up of the same 32 features:
    // H = silu(g) u, silu(g) = g / (1 + e^-g)
#pragma unroll
    for (int a = 0; a < MA; ++a)
#pragma unroll
      for (int b = 0; b < MB; b += 2)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int i = i0 + wi + 32 * a + l32, j = (j0 + wj + 32 * b) / 2 + 8 * g + 4 * h32;
          if (i >= p.I || j >= p.J / 2) continue;
          f32x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float x = acc[a][b][4 * g + e];
            v[e] = x / (1.0f + expf(-x)) * acc[a][b + 1][4 * g + e];
          }
          *(f32x4*)(p.Out + (int64_t)i * p.ldo + j) = v;
        }
    return;
  }
  // Inside the matrix, what the epilogue adds (rho (E1 - E2), or Out) is loaded 16 bytes at a
  // time, a 32 x 32 block ahead of the one being stored. Element by element under bounds
  // checks, every load waited for the one before: targets, G and C of two chunks of 2,048
  // rows at d = 4096 1096 us, 1067 now; the MLP block at 4,096 x 14,336 5.33 ms, 5.24 now.
  if constexpr (!SYM && KSP == 1) {
    auto add_blocks = [&](const float* P1, const float* P2, int64_t ldp, float c, auto two_t) {
      constexpr bool TWO = decltype(two_t)::value;
      constexpr int NBLK = MA * MB;
      const int64_t r0 = i0 + wi + l32;
      const int c0 = j0 + wj + 4 * h32;
      f32x4 x[2][4], y[2][TWO ? 4 : 1];
      auto load = [&](int k, auto s_t) {
        constexpr int s = decltype(s_t)::value;
        const int64_t o = (r0 + 32 * (k / MB)) * ldp + c0 + 32 * (k % MB);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          x[s][g] = *(const f32x4*)(P1 + o + 8 * g);
          if constexpr (TWO) y[s][g] = *(const f32x4*)(P2 + o + 8 * g);
        }
      };
      load(0, std::integral_constant<int, 0>{});
      static_for<NBLK>([&](auto k_t) {
        constexpr int k = decltype(k_t)::value, a = k / MB, b = k % MB;
        if constexpr (k + 1 < NBLK) load(k + 1, std::integral_constant<int, (k + 1) % 2>{});
        float* o = p.Out + (r0 + 32 * a) * p.ldo + c0 + 32 * b;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          f32x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e)
            v[e] = acc[a][b][4 * g + e] + c * (TWO ? x[k % 2][g][e] - y[k % 2][g][e] : x[k % 2][g][e]);
          *(f32x4*)(o + 8 * g) = v;
        }
      });
    };
    if (p.vec_out && i0 + wi + WM <= p.I && j0 + wj + WN <= p.J) {
      if (p.E1 && !p.accumulate && p.vec_in) {
        if (p.E2) add_blocks(p.E1, p.E2, p.lde, p.rho, std::true_type{});
        else add_blocks(p.E1, nullptr, p.lde, p.rho, std::false_type{});
        return;
      }
      if (!p.E1 && p.accumulate) {
        add_blocks(p.Out, nullptr, p.ldo, 1.0f, std::false_type{});
        return;
      }
    }
  }
  // The same for a running symmetric sum, off the diagonal: a block of the tile and its mirror.
  if constexpr (SYM) {
    if (p.accumulate && p.vec_out && ti != tj && i0 + wi + WM <= p.I && j0 + wj + WN <= p.J) {
#pragma unroll
      for (int a = 0; a < MA; ++a)
#pragma unroll
        for (int b = 0; b < MB; ++b) {
          const int64_t i = i0 + wi + 32 * a + l32, j = j0 + wj + 32 * b + 4 * h32;
          f32x4 x[4], m[4];  // (a second set for the next block would not fit in registers)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            x[g] = *(const f32x4*)(p.Out + i * p.ldo + j + 8 * g);
#pragma unroll
            for (int e = 0; e < 4; ++e) m[g][e] = p.Out[(j + 8 * g + e) * p.ldo + i];
          }
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            f32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              v[e] = acc[a][b][4 * g + e];
              if constexpr (KSP == 2) v[e] += part[((a * MB + b) * 16 + 4 * g + e) * 64 + lane];
            }
            *(f32x4*)(p.Out + i * p.ldo + j + 8 * g) = v + x[g];
#pragma unroll
            for (int e = 0; e < 4; ++e) p.Out[(j + 8 * g + e) * p.ldo + i] = m[g][e] + v[e];
          }
        }
      return;
    }
  }
  // lane owns Out[i0+wi+32a+l32][j0+wj+32b+8g+4h32 .. +3]
#pragma unroll
  for (int a = 0; a < MA; ++a)
#pragma unroll
    for (int b = 0; b < MB; ++b)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int i = i0 + wi + 32 * a + l32, j = j0 + wj + 32 * b + 8 * g + 4 * h32;
        if (i >= p.I || j >= p.J) continue;
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = acc[a][b][4 * g + e];
        if constexpr (KSP == 2) {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] += part[((a * MB + b) * 16 + 4 * g + e) * 64 + lane];
        }
        if (p.E1) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (j + e < p.J)
              v[e] += p.rho * (p.E1[(int64_t)i * p.lde + j + e] -
                               (p.E2 ? p.E2[(int64_t)i * p.lde + j + e] : 0.f));
        }
        float* o = p.Out + (int64_t)i * p.ldo + j;
        const bool diag = SYM && ti == tj;
        if (p.vec_out && j + 3 < p.J && !diag) {
          // v stays this call's contribution: the mirror below adds it again
          *(f32x4*)o = p.accumulate ? v + *(const f32x4*)o : v;
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (j + e < p.J && !(diag && i > j + e)) o[e] = p.accumulate ? o[e] + v[e] : v[e];
        }
        if constexpr (SYM) {
          // mirror to (j + e, i): the 32 lanes of a half write 32 consecutive floats
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int jj = j + e;
            if (jj >= p.J || i >= jj) continue;
            float* o2 = p.Out + (int64_t)jj * p.ldo + i;
            *o2 = p.accumulate ? *o2 + v[e] : v[e];
          }
        }
      }
}

template <class CFG, int NA, int NB, int NT, int TA, int TB, bool SYM, bool BNAT, bool SWIGLU>
hipError_t launch_bgemm(BGemm& p, hipStream_t st) {
  p.tiles_j = (p.J + CFG::TJ - 1) / CFG::TJ;
  p.ntiles = SYM ? p.tiles_j * (p.tiles_j + 1) / 2 : (p.I + CFG::TI - 1) / CFG::TI * p.tiles_j;
  const dim3 grid((p.ntiles + kXcds - 1) / kXcds * kXcds), block(CFG::NTH);
  hipLaunchKernelGGL((bgemm_kernel<CFG, NA, NB, NT, TA, TB, SYM, BNAT, SWIGLU>), grid, block, 0, st, p);
  return hipGetLastError();
}

// The tile whose rounds over the 256 CUs are estimated shortest: 1, 0.62 and 0.42 are the
// measured times of one round of 256 x 256, 128 x 256 and 128 x 128 tiles. Targets of
// d = 4096 with all three (us): M = 1024 179 / 114 / 93, 2048 192 / 147 / 172, 3000
// 222 / 243 / 244, 4096 277 / 289 / 330. The same line suits more terms: fp32 weights (three)
// M = 1024 263 / 164 / 127, 2048 279 / 209 / 231, 4096 381 / 408 / 442, d = 1500, M = 2000
// 129 / 78 / 56; SwiGLU features of fp32 weights 4096 x 14336, M = 4096 2302 / 2560 / 2991; whole
// dual patches (X^T Y of four) of 512 rows, 1024 x 4096 277 / 261 / 251, of 4096, 14336 x 4096
// 4473 / 4482 / 4670 (4449 with the rest of the rounds on its own shape). Symmetric
// products: 128-tiles while one round of them holds the triangle (d = 1500, M = 2000, G and C:
// 222 us on large tiles, 100 now), else 192-tiles.
template <int NA, int NB, int NT, int TA, int TB, bool SYM, bool BNAT = false, bool SWIGLU = false>
hipError_t run_bgemm(BGemm p, hipStream_t st) {
  p.vec_out = (p.ldo & 3) == 0 && ((uintptr_t)p.Out & 15) == 0;
  p.vec_in = (p.lde & 3) == 0 && (((uintptr_t)p.E1 | (uintptr_t)p.E2) & 15) == 0;
  using Small = std::conditional_t<SWIGLU, BgCfg<128, 128, 32, 64, 4, 1>, BgCfg<128, 128, 64, 32, 4, 1>>;
  if constexpr (SYM) {
    const int64_t t = (p.J + 127) / 128;
    if (t * (t + 1) / 2 <= 256) return launch_bgemm<Small, NA, NB, NT, TA, TB, true, false, false>(p, st);
    return launch_bgemm<BgSym, NA, NB, NT, TA, TB, true, false, false>(p, st);
  } else {
    using Big = std::conditional_t<NA + NB == 3, BgCfg<256, 256, 64, 128, 3, 1>, BgCfg<256, 256, 128, 64, 2, 1>>;
    using Mid = BgCfg<128, 256, 64, 64, 3, 1>;
    // rows [r0, r0 + n) of the product on one tile shape; the estimated time of the best one
    auto best = [&](int64_t n, int& shape) {
      auto rounds = [&](int ti, int tj) { return (double)(((n + ti - 1) / ti * ((p.J + tj - 1) / tj) + 255) / 256); };
      const double t[3] = {rounds(256, 256), 0.62 * rounds(128, 256), 0.42 * rounds(128, 128)};
      shape = t[0] <= t[1] && t[0] <= t[2] ? 0 : t[1] <= t[2] ? 1 : 2;
      return t[shape];
    };
    auto run = [&](int64_t r0, int64_t n, int shape) {
      BGemm q = p;
      q.I = (int)n;
      for (auto& a : q.A)
        if (a) a += r0 * p.ld;
      q.Out += r0 * p.ldo;
      if (q.E1) q.E1 += r0 * p.lde;
      if (q.E2) q.E2 += r0 * p.lde;
      if (shape == 0) return launch_bgemm<Big, NA, NB, NT, TA, TB, false, BNAT, SWIGLU>(q, st);
      if (shape == 1) return launch_bgemm<Mid, NA, NB, NT, TA, TB, false, BNAT, SWIGLU>(q, st);
      return launch_bgemm<Small, NA, NB, NT, TA, TB, false, BNAT, SWIGLU>(q, st);
    };
    // whole rounds of 256 x 256 tiles, and the rest on the shape that suits it (as a second
    // launch) where that is estimated to save more than the launch (X^T Y of 14336 x 4096:
    // 3.5 rounds as 3 + 0.62: 1.43 -> 1.34 ms)
    int one, head, rest;
    const double all = best(p.I, one);
    const int64_t tj = (p.J + 255) / 256, full = ((int64_t)((p.I + 255) / 256) * tj / 256) * 256 / tj * 256;
    if (full > 0 && full < p.I) {
      const double parts = best(full, head) + best(p.I - full, rest);
      if (parts < 0.95 * all) {
        const hipError_t e = run(0, full, head);
        return e != hipSuccess ? e : run(full, p.I - full, rest);
      }
    }
    return run(0, p.I, one);
  }
}

// bf16 weights [K][J] that the GEMM reads as stored: 16-byte pieces of whole rows, the
// matrix within a buffer descriptor's range, and few rows M of the other operand. The
// transposing reads make the product about 18 % slower, the transposed copies cost the same
// whatever M is. SwiGLU features of d = 4096, d_ff = 14336, as stored against transposed, us:
// M = 128 101 / 203, 512 234 / 302, 1024 444 / 496, 1536 653 / 689, 2048 886 / 895,
// 4096 1678 / 1605; d = 1088, d_ff = 3456, M = 700 48 / 52, 3000 133 / 121.
constexpr int kStoredRows = 1536;
bool as_stored(const void* W, int64_t M, int64_t K, int64_t J) {
  return M <= kStoredRows && J % 8 == 0 && ((uintptr_t)W & 15) == 0 && (K + G_KC) * J * 2 < (int64_t)1 << 32;
}

hipError_t run_split_rows(const float* S1, const float* S2, int64_t rows, int64_t cols, int64_t ld,
                          __bf16* hi, __bf16* lo, int64_t rows_p, int64_t cols_p, hipStream_t st) {
  const int64_t n = rows_p * (cols_p / 8);
  hipLaunchKernelGGL(split_rows_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, S1, S2,
                     (int)rows, (int)cols, ld, hi, lo, (int)rows_p, (int)cols_p);
  return hipGetLastError();
}

template <class SRC>
hipError_t run_split_transpose(const SRC* S1, const float* S2, int64_t rows, int64_t cols,
                               int64_t ld, __bf16* hi, __bf16* lo, int64_t rows_p, int64_t cols_p,
                               hipStream_t st, float s2 = -1.f, int pair = -1) {
  // rows_p is a multiple of 8 (every caller pads it to 64), cols_p of 8: whole 16-byte chunks
  if constexpr (std::is_same<SRC, __bf16>::value) {
    if (!S2 && !lo && cols % 8 == 0 && ld % 8 == 0 && (uintptr_t)S1 % 16 == 0) {
      const dim3 grid((unsigned)((cols_p + 127) / 128), (unsigned)((rows_p + 127) / 128));
      hipLaunchKernelGGL(transpose_bf16_kernel, grid, dim3(256), 0, st, S1, (int)rows, (int)cols, ld, hi,
                         (int)rows_p, (int)cols_p, pair);
      return hipGetLastError();
    }
  }
  const dim3 grid((unsigned)((cols_p + 63) / 64), (unsigned)((rows_p + 127) / 128));
  const int vec = ld % 4 == 0 && (uintptr_t)S1 % (4 * sizeof(SRC)) == 0 &&
                  (S2 == nullptr || (uintptr_t)S2 % 16 == 0);
  hipLaunchKernelGGL((split_transpose_kernel<SRC>), grid, dim3(256), 0, st, S1, S2, s2, (int)rows,
                     (int)cols, ld, hi, lo, (int)rows_p, (int)cols_p, vec, pair);
  return hipGetLastError();
}

// u = z / sqrt(mean(z^2) + eps) per row, split into hi and lo planes [rows_p][cols_p]
// (zero outside rows x cols). One workgroup per row; the mean square in fp32. A thread
// owns 8 consecutive columns of every 2,048; the first kRmsKeep such pieces stay in
// registers between the two passes. Memory bound:
// 4096 x 4096 29 us (4.6 TB/s), 55 with scalar loads and a second read of z.
constexpr int kRmsKeep = 4;
__global__ __launch_bounds__(256) void rmsnorm_split_kernel(const float* __restrict__ Z, int rows,
                                                            int cols, float eps,
                                                            __bf16* __restrict__ hi,
                                                            __bf16* __restrict__ lo, int cols_p) {
  __shared__ float part[5];
  const int r = blockIdx.x, tid = threadIdx.x;
  const float* z = Z + (int64_t)r * cols;
  const bool vec = (cols & 3) == 0 && ((uintptr_t)Z & 15) == 0;
  auto load = [&](int c0, f32x4 (&v)[2]) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int c = c0 + 4 * h;
      v[h] = f32x4{};
      if (r < rows) {
        if (vec) {
          if (c < cols) v[h] = *(const f32x4*)(z + c);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (c + e < cols) v[h][e] = z[c + e];
        }
      }
    }
  };
  f32x4 keep[kRmsKeep][2], v[2];
  float ss = 0.f;
  auto square = [&](const f32x4 (&x)[2]) {
#pragma unroll
    for (int e = 0; e < 8; ++e) ss = fmaf(x[e >> 2][e & 3], x[e >> 2][e & 3], ss);
  };
#pragma unroll
  for (int u = 0; u < kRmsKeep; ++u) load(tid * 8 + u * 2048, keep[u]);
#pragma unroll
  for (int u = 0; u < kRmsKeep; ++u) square(keep[u]);
  for (int c0 = tid * 8 + kRmsKeep * 2048; c0 < cols; c0 += 2048) {
    load(c0, v);
    square(v);
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) ss += __shfl_xor(ss, o);
  if ((tid & 63) == 0) part[tid >> 6] = ss;
  __syncthreads();
  if (tid == 0) part[4] = 1.0f / sqrtf((part[0] + part[1] + part[2] + part[3]) / (float)cols + eps);
  __syncthreads();
  const float inv = r < rows ? part[4] : 0.f;
  auto store = [&](int c0, const f32x4 (&x)[2]) {
    if (c0 >= cols_p) return;
    bf16x8 h, l;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float u = x[e >> 2][e & 3] * inv;
      h[e] = to_bf16(u);
      l[e] = to_bf16(u - (float)h[e]);
    }
    *(bf16x8*)(hi + (int64_t)r * cols_p + c0) = h;
    *(bf16x8*)(lo + (int64_t)r * cols_p + c0) = l;
  };
#pragma unroll
  for (int u = 0; u < kRmsKeep; ++u) store(tid * 8 + u * 2048, keep[u]);
  for (int c0 = tid * 8 + kRmsKeep * 2048; c0 < cols_p; c0 += 2048) {
    load(c0, v);
    store(c0, v);
  }
}

struct TargetsWs {
  size_t Dh, Dl, Wh, Wl, total;
};
TargetsWs targets_layout(int64_t M, int64_t din, int64_t dout) {
  const int64_t Mp = pad_to(M, G_BM), Kp = pad_to(din, G_KC), Jp = pad_to(dout, G_BM);
  TargetsWs L{};
  size_t o = 0;
  L.Dh = o; o += align_up((size_t)Mp * Kp * 2);
  L.Dl = o; o += align_up((size_t)Mp * Kp * 2);
  L.Wh = o; o += align_up((size_t)Jp * Kp * 2);
  L.Wl = o; o += align_up((size_t)Jp * Kp * 2);
  L.total = o;
  return L;
}
struct NormalEqWs {
  size_t Xh, Xl, Yh, Yl, total;
};
NormalEqWs normal_eq_layout(int64_t rows, int64_t din, int64_t dout) {
  const int64_t Kp = pad_to(rows, G_KC), Ip = pad_to(din, G_BM), Jp = pad_to(dout, G_BM);
  NormalEqWs L{};
  size_t o = 0;
  L.Xh = o; o += align_up((size_t)Ip * Kp * 2);
  L.Xl = o; o += align_up((size_t)Ip * Kp * 2);
  L.Yh = o; o += align_up((size_t)Jp * Kp * 2);
  L.Yl = o; o += align_up((size_t)Jp * Kp * 2);
  L.total = o;
  return L;
}

struct MlpWs {
  size_t Uh, Ul, Wh, Wl, total;
  int64_t Mp, Kp, Jh;  // padded rows, padded d, padded d_ff (half of the interleaved gate and up rows)
};
MlpWs mlp_layout(int64_t M, int64_t d, int64_t d_ff) {
  MlpWs L{};
  L.Mp = pad_to(M, G_BM);
  L.Kp = pad_to(d, G_KC);
  L.Jh = pad_to(d_ff, G_BM / 2);
  size_t o = 0;
  L.Uh = o; o += align_up((size_t)L.Mp * L.Kp * 2);
  L.Ul = o; o += align_up((size_t)L.Mp * L.Kp * 2);
  L.Wh = o; o += align_up((size_t)2 * L.Jh * L.Kp * 2);
  L.Wl = o; o += align_up((size_t)2 * L.Jh * L.Kp * 2);
  L.total = o;
  return L;
}

// ---------------------------------------------------------------- fp64 path

template <class TA, class TB>
struct F64Params {
  const TA* A1;
  const TA* A2;
  int64_t sai, sak;
  const TB* B1;
  const TB* B2;
  int64_t sbj, sbk;
  double* Out;
  int64_t ldo;
  const float* E1;
  const float* E2;
  int64_t lde;
  double rho;
  int I, J, K;
  int accumulate;
  int tiles_j;
};

// Out[i][j] (+)= sum_k A(i,k) B(j,k) (+ rho E), all products and sums in fp64 (MFMA f64).
template <int BM, class TA, class TB>
__device__ __forceinline__ void f64_gemm_body(const F64Params<TA, TB>& p, int t, F64Lds<BM>& lds) {
  const int i0 = (t / p.tiles_j) * BM, j0 = (t % p.tiles_j) * BM;
  f64x4 acc[BM / 32][BM / 32];
  const F64Operand<TA> A{p.A1 + i0 * p.sai, p.A2 ? p.A2 + i0 * p.sai : nullptr, p.sai, p.sak, p.I - i0};
  const F64Operand<TB> B{p.B1 + j0 * p.sbj, p.B2 ? p.B2 + j0 * p.sbj : nullptr, p.sbj, p.sbk, p.J - j0};
  f64_tile<BM>(acc, p.K, A, B, lds);
  f64_each<BM>(acc, [&](int ti, int tj, double r) {
    const int i = i0 + ti, j = j0 + tj;
    if (i >= p.I || j >= p.J) return;
    if (p.E1)
      r += p.rho * ((double)p.E1[(int64_t)i * p.lde + j] - (double)p.E2[(int64_t)i * p.lde + j]);
    double* o = p.Out + (int64_t)i * p.ldo + j;
    *o = p.accumulate ? *o + r : r;
  });
}

// One or two problems per launch: workgroups [0, n0) work on p, the rest on q.
template <int BM, class TA, class TB, class TA1, class TB1>
__global__ __launch_bounds__(256) void f64_gemm_kernel(F64Params<TA, TB> p, F64Params<TA1, TB1> q,
                                                       int n0) {
  __shared__ F64Lds<BM> lds;
  const int t = blockIdx.x;
  if (t < n0) f64_gemm_body<BM>(p, t, lds);
  else f64_gemm_body<BM>(q, t - n0, lds);
}

// 64-tiles once they fill the 256 CUs, else 32-tiles (a call of few tiles is bound by the
// latency of its K loop). d = 256, 128 rows: the targets 12 us (48 on 64-tiles of fp64 FMA),
// G and C together 7 us (31 + 48).
template <class TA, class TB, class TA1, class TB1>
hipError_t run_f64(F64Params<TA, TB> p, F64Params<TA1, TB1> q, hipStream_t st) {
  auto tiles = [](auto& x, int bm) {
    x.tiles_j = (x.J + bm - 1) / bm;
    return (x.I + bm - 1) / bm * x.tiles_j;
  };
  int n0 = tiles(p, 64), n1 = tiles(q, 64);
  if (n0 + n1 >= 256) {
    hipLaunchKernelGGL((f64_gemm_kernel<64, TA, TB, TA1, TB1>), dim3(n0 + n1), dim3(256), 0, st, p, q,
                       n0);
  } else {
    n0 = tiles(p, 32);
    n1 = tiles(q, 32);
    hipLaunchKernelGGL((f64_gemm_kernel<32, TA, TB, TA1, TB1>), dim3(n0 + n1), dim3(256), 0, st, p, q,
                       n0);
  }
  return hipGetLastError();
}
template <class TA, class TB>
hipError_t run_f64(const F64Params<TA, TB>& p, hipStream_t st) {
  return run_f64(p, F64Params<TA, TB>{}, st);
}

}  // namespace

size_t targets_ws_bytes(int64_t M, int64_t din, int64_t dout) {
  return targets_layout(M, din, dout).total;
}
size_t mlp_features_ws_bytes(int64_t M, int64_t d, int64_t d_ff) {
  return mlp_layout(M, d, d_ff).total;
}

hipError_t launch_mlp_features(const float* Z, const void* Wg, const void* Wu, bool w_bf16,
                               int64_t M, int64_t d, int64_t d_ff, float eps, float* H, void* ws,
                               hipStream_t st) {
  const MlpWs L = mlp_layout(M, d, d_ff);
  char* w = (char*)ws;
  __bf16 *Uh = (__bf16*)(w + L.Uh), *Ul = (__bf16*)(w + L.Ul);
  __bf16 *Wh = (__bf16*)(w + L.Wh), *Wl = (__bf16*)(w + L.Wl);
  hipLaunchKernelGGL(rmsnorm_split_kernel, dim3((unsigned)L.Mp), dim3(256), 0, st, Z, (int)M, (int)d,
                     eps, Uh, Ul, (int)L.Kp);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // gate and up interleaved in blocks of 32 features, so a workgroup's tile holds both of
  // a feature and forms H itself
  BGemm p{};
  p.ld = L.Kp;
  p.Out = H;
  p.ldo = d_ff;
  p.I = (int)M;
  p.J = (int)(2 * d_ff);
  p.Kp = (int)L.Kp;
  p.A[0] = Uh; p.A[1] = Ul;
  if (w_bf16 && as_stored(Wg, M, d, d_ff) && as_stored(Wu, M, d, d_ff)) {
    p.B[0] = (const __bf16*)Wg; p.B[1] = (const __bf16*)Wu;
    p.ldb = d_ff;
    p.K = (int)d;
    return run_bgemm<2, 1, 2, 0b10, 0b00, false, true, true>(p, st);
  }
  for (int h = 0; h < 2; ++h) {
    const void* Wx = h ? Wu : Wg;
    if (w_bf16)
      e = run_split_transpose((const __bf16*)Wx, nullptr, d, d_ff, d_ff, Wh, nullptr, L.Kp, L.Jh, st,
                              -1.f, 32 * h);
    else
      e = run_split_transpose((const float*)Wx, nullptr, d, d_ff, d_ff, Wh, Wl, L.Kp, L.Jh, st, -1.f,
                              32 * h);
    if (e != hipSuccess) return e;
  }
  p.B[0] = Wh; p.B[1] = Wl;
  return w_bf16 ? run_bgemm<2, 1, 2, 0b10, 0b00, false, false, true>(p, st)
                : run_bgemm<2, 2, 3, 0b010, 0b100, false, false, true>(p, st);
}

size_t propagate_ws_bytes(int64_t M, int64_t d_ff, int64_t d) {
  return targets_layout(M, d_ff, d).total;
}

hipError_t launch_propagate(const float* Hc, const void* W, bool w_bf16, const float* dW,
                            const float* Zc, int64_t M, int64_t d_ff, int64_t d, float* Y, void* ws,
                            hipStream_t st) {
  const TargetsWs L = targets_layout(M, d_ff, d);
  const int64_t Mp = pad_to(M, G_BM), Kp = pad_to(d_ff, G_KC), Jp = pad_to(d, G_BM);
  char* w = (char*)ws;
  __bf16 *Hh = (__bf16*)(w + L.Dh), *Hl = (__bf16*)(w + L.Dl);
  __bf16 *Wh = (__bf16*)(w + L.Wh), *Wl = (__bf16*)(w + L.Wl);
  hipError_t e = run_split_rows(Hc, nullptr, M, d_ff, d_ff, Hh, Hl, Mp, Kp, st);
  if (e != hipSuccess) return e;
  // (W + dW) [d_ff][d] -> transposed [d][d_ff], split
  if (w_bf16)
    e = run_split_transpose((const __bf16*)W, dW, d_ff, d, d, Wh, Wl, Kp, Jp, st, 1.f);
  else
    e = run_split_transpose((const float*)W, dW, d_ff, d, d, Wh, Wl, Kp, Jp, st, 1.f);
  if (e != hipSuccess) return e;
  BGemm p{};  // Y = Hc (W + dW) + Zc: terms (0,0) (0,1) (1,0)
  p.ld = Kp;
  p.Out = Y;
  p.ldo = d;
  p.E1 = Zc;
  p.lde = d;
  p.rho = 1.f;
  p.I = (int)M;
  p.J = (int)d;
  p.Kp = (int)Kp;
  p.A[0] = Hh; p.A[1] = Hl;
  p.B[0] = Wh; p.B[1] = Wl;
  return run_bgemm<2, 2, 3, 0b100, 0b010, false>(p, st);
}
size_t normal_eq_ws_bytes(int64_t rows, int64_t din, int64_t dout) {
  return normal_eq_layout(rows, din, dout).total;
}

// ---------------------------------------------------------------- dual-form statistics
//
// For the ridge patch through the push-through identity (few rows, wide d_in):
// K = X X^T over the rows, and dW = X^T Y. Both sum all four hi/lo term pairs (the
// split of both operands loses only the lo x lo cross term otherwise; X^T Y's result
// can be much smaller than |X||Y| when the ridge is small, so it keeps every term).
struct DualWs {
  size_t Ah, Al, Bh, Bl, total;
};
DualWs dual_layout(int64_t rows, int64_t din, int64_t dout) {
  // K: planes of X [rows_p][din_p] (contraction d_in); X^T Y: planes of X^T and Y^T
  // [*][rows_p] (contraction rows)
  const int64_t rK = pad_to(rows, G_BM), cK = pad_to(din, G_KC);
  const int64_t kY = pad_to(rows, G_KC), iY = pad_to(din, G_BM), jY = pad_to(dout, G_BM);
  const size_t a = std::max((size_t)rK * cK, (size_t)iY * kY) * 2;
  const size_t b = (size_t)jY * kY * 2;
  DualWs L{};
  size_t o = 0;
  L.Ah = o; o += align_up(a);
  L.Al = o; o += align_up(a);
  L.Bh = o; o += align_up(b);
  L.Bl = o; o += align_up(b);
  L.total = o;
  return L;
}

hipError_t launch_gram_rows(const float* X, int64_t rows, int64_t din, float* K, void* ws,
                            hipStream_t st) {
  const DualWs L = dual_layout(rows, din, 1);
  const int64_t rK = pad_to(rows, G_BM), cK = pad_to(din, G_KC);
  char* w = (char*)ws;
  __bf16 *Xh = (__bf16*)(w + L.Ah), *Xl = (__bf16*)(w + L.Al);
  hipError_t e = run_split_rows(X, nullptr, rows, din, din, Xh, Xl, rK, cK, st);
  if (e != hipSuccess) return e;
  BGemm g{};
  g.ld = cK;
  g.Out = K;
  g.ldo = rows;
  g.I = (int)rows;
  g.J = (int)rows;
  g.Kp = (int)cK;
  g.A[0] = Xh; g.A[1] = Xl;
  g.B[0] = Xh; g.B[1] = Xl;
  return run_bgemm<2, 2, 4, 0b1100, 0b1010, true>(g, st);
}

hipError_t launch_xt_y(const float* X, const float* Y, int64_t rows, int64_t din, int64_t dout,
                       float* Out, void* ws, hipStream_t st) {
  const DualWs L = dual_layout(rows, din, dout);
  const int64_t kY = pad_to(rows, G_KC), iY = pad_to(din, G_BM), jY = pad_to(dout, G_BM);
  char* w = (char*)ws;
  __bf16 *Xh = (__bf16*)(w + L.Ah), *Xl = (__bf16*)(w + L.Al);
  __bf16 *Yh = (__bf16*)(w + L.Bh), *Yl = (__bf16*)(w + L.Bl);
  // X [rows][din] -> X^T [din][rows]; Y [rows][dout] -> Y^T [dout][rows]
  hipError_t e = run_split_transpose(X, (const float*)nullptr, rows, din, din, Xh, Xl, kY, iY, st);
  if (e != hipSuccess) return e;
  e = run_split_transpose(Y, (const float*)nullptr, rows, dout, dout, Yh, Yl, kY, jY, st);
  if (e != hipSuccess) return e;
  BGemm p{};
  p.ld = kY;
  p.Out = Out;
  p.ldo = dout;
  p.I = (int)din;
  p.J = (int)dout;
  p.Kp = (int)kY;
  p.A[0] = Xh; p.A[1] = Xl;
  p.B[0] = Yh; p.B[1] = Yl;
  return run_bgemm<2, 2, 4, 0b1100, 0b1010, false>(p, st);
}

size_t dual_stats_ws_bytes(int64_t rows, int64_t din, int64_t dout) {
  return dual_layout(rows, din, dout).total;
}

hipError_t launch_targets(const float* Of, const float* Oc, const void* W, bool w_bf16, int64_t M,
                          int64_t din, int64_t dout, int rho, float* T, void* ws, hipStream_t st,
                          const float* Zf, const float* Zc) {
  const TargetsWs L = targets_layout(M, din, dout);
  const int64_t Mp = pad_to(M, G_BM), Kp = pad_to(din, G_KC), Jp = pad_to(dout, G_BM);
  char* w = (char*)ws;
  __bf16 *Dh = (__bf16*)(w + L.Dh), *Dl = (__bf16*)(w + L.Dl);
  __bf16 *Wh = (__bf16*)(w + L.Wh), *Wl = (__bf16*)(w + L.Wl);
  hipError_t e = run_split_rows(Of, Oc, M, din, din, Dh, Dl, Mp, Kp, st);
  if (e != hipSuccess) return e;
  // W [din][dout] -> W^T [dout][din] (rows j, contraction k contiguous)
  if (w_bf16)
    e = run_split_transpose((const __bf16*)W, nullptr, din, dout, dout, Wh, nullptr, Kp, Jp, st);
  else
    e = run_split_transpose((const float*)W, nullptr, din, dout, dout, Wh, Wl, Kp, Jp, st);
  if (e != hipSuccess) return e;
  BGemm p{};
  p.ld = Kp;
  p.Out = T;
  p.ldo = dout;
  if (Zf) {  // residual pair of its own (width dout)
    p.E1 = Zf;
    p.E2 = Zc;
    p.lde = dout;
    p.rho = 1.f;
  } else if (rho) {
    p.E1 = Of;
    p.E2 = Oc;
    p.lde = din;
    p.rho = (float)rho;
  }
  p.I = (int)M;
  p.J = (int)dout;
  p.Kp = (int)Kp;
  p.A[0] = Dh; p.A[1] = Dl;
  p.B[0] = Wh; p.B[1] = Wl;
  // terms (a, b): bf16 W (0,0) (1,0); fp32 W (0,0) (1,0) (0,1)
  if (w_bf16) return run_bgemm<2, 1, 2, 0b10, 0b00, false>(p, st);
  return run_bgemm<2, 2, 3, 0b010, 0b100, false>(p, st);
}

hipError_t launch_normal_eq_f32(const float* X, const float* Yf, const float* Yc, int64_t rows,
                                int64_t din, int64_t dout, bool accumulate, float* G, float* C,
                                void* ws, hipStream_t st) {
  const NormalEqWs L = normal_eq_layout(rows, din, dout);
  const int64_t Kp = pad_to(rows, G_KC), Ip = pad_to(din, G_BM), Jp = pad_to(dout, G_BM);
  char* w = (char*)ws;
  __bf16 *Xh = (__bf16*)(w + L.Xh), *Xl = (__bf16*)(w + L.Xl);
  __bf16 *Yh = (__bf16*)(w + L.Yh), *Yl = (__bf16*)(w + L.Yl);
  // X [rows][din] -> X^T [din][rows]; (Yf - Yc) [rows][dout] -> [dout][rows]
  hipError_t e = run_split_transpose(X, (const float*)nullptr, rows, din, din, Xh, Xl, Kp, Ip, st);
  if (e != hipSuccess) return e;
  e = run_split_transpose(Yf, Yc, rows, dout, dout, Yh, Yl, Kp, Jp, st);
  if (e != hipSuccess) return e;
  {  // G = X^T X: terms (0,0) (0,1) (1,0) (1,1), upper block triangle, mirrored
    BGemm g{};
    g.ld = Kp;
    g.Out = G;
    g.ldo = din;
    g.I = (int)din;
    g.J = (int)din;
    g.Kp = (int)Kp;
    g.accumulate = accumulate;
    g.A[0] = Xh; g.A[1] = Xl;
    g.B[0] = Xh; g.B[1] = Xl;
    e = run_bgemm<2, 2, 4, 0b1100, 0b1010, true>(g, st);
    if (e != hipSuccess) return e;
  }
  BGemm p{};  // C = X^T (Yf - Yc): terms (0,0) (0,1) (1,0)
  p.ld = Kp;
  p.Out = C;
  p.ldo = dout;
  p.I = (int)din;
  p.J = (int)dout;
  p.Kp = (int)Kp;
  p.accumulate = accumulate;
  p.A[0] = Xh; p.A[1] = Xl;
  p.B[0] = Yh; p.B[1] = Yl;
  return run_bgemm<2, 2, 3, 0b100, 0b010, false>(p, st);
}

hipError_t launch_targets_f64(const float* Of, const float* Oc, const void* W, bool w_bf16,
                              int64_t M, int64_t din, int64_t dout, int rho, double* T,
                              hipStream_t st) {
  if (w_bf16) {
    F64Params<float, __bf16> p{};
    p.A1 = Of; p.A2 = Oc; p.sai = din; p.sak = 1;
    p.B1 = (const __bf16*)W; p.sbj = 1; p.sbk = dout;
    p.Out = T; p.ldo = dout;
    if (rho) { p.E1 = Of; p.E2 = Oc; p.lde = din; p.rho = rho; }
    p.I = (int)M; p.J = (int)dout; p.K = (int)din;
    return run_f64(p, st);
  }
  F64Params<float, float> p{};
  p.A1 = Of; p.A2 = Oc; p.sai = din; p.sak = 1;
  p.B1 = (const float*)W; p.sbj = 1; p.sbk = dout;
  p.Out = T; p.ldo = dout;
  if (rho) { p.E1 = Of; p.E2 = Oc; p.lde = din; p.rho = rho; }
  p.I = (int)M; p.J = (int)dout; p.K = (int)din;
  return run_f64(p, st);
}

hipError_t launch_normal_eq_f64(const float* X, const float* Yf, const float* Yc, const double* Yd,
                                int64_t rows, int64_t din, int64_t dout, bool accumulate,
                                double* G, double* C, hipStream_t st) {
  // G and C in one launch
  F64Params<float, float> g{};
  g.A1 = X; g.sai = 1; g.sak = din;
  g.B1 = X; g.sbj = 1; g.sbk = din;
  g.Out = G; g.ldo = din; g.accumulate = accumulate;
  g.I = (int)din; g.J = (int)din; g.K = (int)rows;
  if (Yd) {
    F64Params<float, double> p{};
    p.A1 = X; p.sai = 1; p.sak = din;
    p.B1 = Yd; p.sbj = 1; p.sbk = dout;
    p.Out = C; p.ldo = dout; p.accumulate = accumulate;
    p.I = (int)din; p.J = (int)dout; p.K = (int)rows;
    return run_f64(g, p, st);
  }
  F64Params<float, float> p{};
  p.A1 = X; p.sai = 1; p.sak = din;
  p.B1 = Yf; p.B2 = Yc; p.sbj = 1; p.sbk = dout;
  p.Out = C; p.ldo = dout; p.accumulate = accumulate;
  p.I = (int)din; p.J = (int)dout; p.K = (int)rows;
  return run_f64(g, p, st);
}

}  // namespace pkv
