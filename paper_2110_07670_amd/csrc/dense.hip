// Dense FP64 stages of the ACE build on gfx950 (arXiv 2110.07670, section
// "ACE Operator"): the overlap matrix M = dV Phi^T W, the Cholesky factor of
// -M, the projectors xi = W L^{-T} and their application
// V_ACE psi = -xi (dV xi^T psi).  The products run on the FP64 matrix cores
// (v_mfma_f64_16x16x4f64); the small factorisation runs in one workgroup.
//
// MFMA f64 16x16x4 operand layout (per wave, lane l):
//   A fragment: A[i = l % 16][k = l / 16]
//   B fragment: B[k = l / 16][j = l % 16]
//   D (4 doubles): D[i = l / 16 + 4 v][j = l % 16], v = 0..3
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>

#include "kernels.h"

namespace acex {

typedef double d4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ d4 mfma16x16x4(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// ------------------------------------------------------------------ C = A B^T, large tiles
// More than 64 rows on both sides: 256 threads (4 waves in 2 x 2), output
// tile 128 x 128, each wave 64 x 64 = 4 x 4 MFMA blocks.  K staged through
// two LDS buffers in slabs of KT: while the MFMAs read one slab, the next one
// (loaded into registers behind them) is stored into the other buffer, so
// each slab costs one barrier.  VEC (even K, 16-byte aligned operands): two
// consecutive k per load and per LDS store, rows padded to 18 (16-byte
// aligned, and the MFMA operand reads of 32 lanes still fall on distinct
// banks); else one k per access, rows padded to 17.  Whole 128-byte lines per
// row and each operand read once per workgroup: 556 us for 128 x 128 over
// 884,736 points against 545-700 us without LDS (the kernel below), 1094
// against 1378 us over 1,728,000.  sym: only the tiles on and below the
// diagonal (512 orbitals: 10 of 16).
constexpr int kAbtTile = 128;
constexpr int kAbtKT = 16;
constexpr int kAbtPer = kAbtTile * kAbtKT / 256;  // elements per thread per operand

template <bool VEC>
__global__ __launch_bounds__(256) void k_gemm_abt_tile(const double* __restrict__ A,
                                                  const double* __restrict__ B, int m, int n,
                                                  int64_t K, int64_t kchunk, int tiles_n, bool sym,
                                                  bool abs_in, double* __restrict__ partial,
                                                  const int* __restrict__ skip) {
  if (skip && *skip != 0) return;
  constexpr int kAbtPitch = VEC ? kAbtKT + 2 : kAbtKT + 1;
  __shared__ __align__(16) double sA[2][kAbtTile * kAbtPitch];
  __shared__ __align__(16) double sB[2][kAbtTile * kAbtPitch];
  const int split = blockIdx.y;
  int tm, tn;
  if (sym) {  // the tiles on and below the diagonal, row by row
    tm = 0;
    int t = blockIdx.x;
    while (t > tm) t -= ++tm;
    tn = t;
  } else {
    tm = blockIdx.x / tiles_n;
    tn = blockIdx.x % tiles_n;
  }
  const int m0 = tm * kAbtTile, n0 = tn * kAbtTile;
  const int64_t kbeg = (int64_t)split * kchunk;
  int64_t kend = kbeg + kchunk;
  if (kend > K) kend = K;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  d4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};

  double ra[kAbtPer], rb[kAbtPer];
  auto fetch = [&](int64_t k0) {
    if constexpr (VEC) {
      // element pairs (r, c), (r, c + 1), c even; kend is even
#pragma unroll
      for (int q = 0; q < kAbtPer / 2; ++q) {
        const int e = tid + q * 256;
        const int r = e / (kAbtKT / 2), c = 2 * (e % (kAbtKT / 2));
        const int64_t k = k0 + c;
        double2 va = {0.0, 0.0}, vb = {0.0, 0.0};
        if (k < kend) {
          if (m0 + r < m) va = *reinterpret_cast<const double2*>(A + (int64_t)(m0 + r) * K + k);
          if (n0 + r < n) vb = *reinterpret_cast<const double2*>(B + (int64_t)(n0 + r) * K + k);
        }
        ra[2 * q] = abs_in ? fabs(va.x) : va.x;
        ra[2 * q + 1] = abs_in ? fabs(va.y) : va.y;
        rb[2 * q] = abs_in ? fabs(vb.x) : vb.x;
        rb[2 * q + 1] = abs_in ? fabs(vb.y) : vb.y;
      }
    } else {
#pragma unroll
      for (int q = 0; q < kAbtPer; ++q) {
        const int e = tid + q * 256;
        const int r = e / kAbtKT, c = e % kAbtKT;
        const int64_t k = k0 + c;
        double va = 0.0, vb = 0.0;
        if (k < kend) {
          if (m0 + r < m) va = A[(int64_t)(m0 + r) * K + k];
          if (n0 + r < n) vb = B[(int64_t)(n0 + r) * K + k];
        }
        ra[q] = abs_in ? fabs(va) : va;
        rb[q] = abs_in ? fabs(vb) : vb;
      }
    }
  };
  auto stage = [&](int buf) {
    if constexpr (VEC) {
#pragma unroll
      for (int q = 0; q < kAbtPer / 2; ++q) {
        const int e = tid + q * 256;
        const int r = e / (kAbtKT / 2), c = 2 * (e % (kAbtKT / 2));
        *reinterpret_cast<double2*>(&sA[buf][r * kAbtPitch + c]) = double2{ra[2 * q], ra[2 * q + 1]};
        *reinterpret_cast<double2*>(&sB[buf][r * kAbtPitch + c]) = double2{rb[2 * q], rb[2 * q + 1]};
      }
    } else {
#pragma unroll
      for (int q = 0; q < kAbtPer; ++q) {
        const int e = tid + q * 256;
        const int r = e / kAbtKT, c = e % kAbtKT;
        sA[buf][r * kAbtPitch + c] = ra[q];
        sB[buf][r * kAbtPitch + c] = rb[q];
      }
    }
  };
  if (kbeg < kend) {
    fetch(kbeg);
    stage(0);
  }
  __syncthreads();
  int buf = 0;
  for (int64_t k0 = kbeg; k0 < kend; k0 += kAbtKT) {
    const bool more = k0 + kAbtKT < kend;
    if (more) fetch(k0 + kAbtKT);
#pragma unroll
    for (int kk = 0; kk < kAbtKT; kk += 4) {
      double af[4], bf[4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        af[i] = sA[buf][(wm * 64 + i * 16 + (lane & 15)) * kAbtPitch + kk + (lane >> 4)];
#pragma unroll
      for (int j = 0; j < 4; ++j)
        bf[j] = sB[buf][(wn * 64 + j * 16 + (lane & 15)) * kAbtPitch + kk + (lane >> 4)];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = mfma16x16x4(af[i], bf[j], acc[i][j]);
    }
    if (more) stage(buf ^ 1);
    __syncthreads();
    buf ^= 1;
  }
  double* out = partial + (int64_t)split * m * n;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = m0 + wm * 64 + i * 16 + (lane >> 4) + 4 * v;
        const int col = n0 + wn * 64 + j * 16 + (lane & 15);
        if (row < m && col < n) out[(int64_t)row * n + col] = acc[i][j][v];
      }
}

// ------------------------------------------------------------------ C = A B^T, few rows
// Both operands run along K, so a lane's MFMA operand (one row, one k) lies
// next to the following k's: the fragments are loaded straight into
// registers, 64 contiguous bytes of a row per four lanes, with no LDS and no
// barrier in the loop.  Within eight k, lane group g = lane / 16 takes k = 2 g
// and 2 g + 1: the same permutation of the sum on both sides.
//
// A workgroup's four waves cover WM x WN wave tiles of (16 RM) x (16 RN)
// outputs; the remaining factor WK = 4 / (WM WN) splits its K range (eight k
// per wave in turn), summed in LDS in a fixed order at the end.  The tile
// follows the output (abt_shape): in the 128 x 128 tile above a product of
// few rows spends its time on the matrix cores' padding rows (4 x 128 outputs
// over 884,736 points 553 us there, 190 us here, which is 4.8 TB/s of its
// operands; 36 x 36 over 110,592 83 and 26 us; 8 x 8 over 32,768 25 and 5).
// kAbtAhead eight-k steps are in flight per wave, which with the 128
// registers of a 64 x 64 wave tile leaves two waves per SIMD.
//
// VEC: K a multiple of 8 and 16-byte aligned operands; else scalar loads
// with a bounds check per k.
constexpr int kAbtAhead = 3;

template <int RM, int WM, int RN, int WN, bool VEC>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_gemm_abt(
    const double* __restrict__ A, const double* __restrict__ B, int m, int n, int64_t K,
    int64_t kchunk, int tiles_n, bool abs_in, double* __restrict__ partial,
    const int* __restrict__ skip) {
  if (skip && *skip != 0) return;
  constexpr int WK = 4 / (WM * WN), TM = 16 * RM * WM, TN = 16 * RN * WN, D = kAbtAhead;
  const int tm = blockIdx.x / tiles_n, tn = blockIdx.x % tiles_n;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wk = wave / (WM * WN), wmn = wave % (WM * WN), wm = wmn / WN, wn = wmn % WN;
  const int li = lane & 15, g = lane >> 4;
  const int64_t kbeg = (int64_t)blockIdx.y * kchunk;
  int64_t kend = kbeg + kchunk;
  if (kend > K) kend = K;
  // a wave's operand rows as a uniform base and 32-bit lane offsets (64 rows of
  // at most 192^3 doubles are under 4 GiB); rows past the end read the last
  // row, and their outputs are not stored
  const int ra = (tm * WM + wm) * RM * 16, rb = (tn * WN + wn) * RN * 16;
  const char* ba = reinterpret_cast<const char*>(A + (int64_t)min(ra, m - 1) * K);
  const char* bb = reinterpret_cast<const char*>(B + (int64_t)min(rb, n - 1) * K);
  unsigned oa[RM], ob[RN];
#pragma unroll
  for (int i = 0; i < RM; ++i)
    oa[i] = 8u * ((unsigned)max(min(16 * i + li, m - 1 - ra), 0) * (unsigned)K + 2 * g);
#pragma unroll
  for (int j = 0; j < RN; ++j)
    ob[j] = 8u * ((unsigned)max(min(16 * j + li, n - 1 - rb), 0) * (unsigned)K + 2 * g);
  d4 acc[RM][RN];
#pragma unroll
  for (int i = 0; i < RM; ++i)
#pragma unroll
    for (int j = 0; j < RN; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};
  double2 fa[D][RM], fb[D][RN];
  auto ld = [&](const char* p, unsigned o, int64_t k) __attribute__((always_inline)) {
    const double* q = reinterpret_cast<const double*>(p + 8 * k + o);
    if constexpr (VEC) {
      return *reinterpret_cast<const double2*>(q);
    } else {
      double2 v = {0.0, 0.0};
      if (k + 2 * g < kend) v.x = q[0];
      if (k + 2 * g + 1 < kend) v.y = q[1];
      return v;
    }
  };
  // this wave's steps: k = kbeg + 8 (wk + WK t), t < steps; a fetch past the
  // last one repeats it and is not multiplied
  const int steps =
      kbeg + 8 * wk < kend ? (int)((kend - kbeg - 8 * wk + 8 * WK - 1) / (8 * WK)) : 0;
  auto fetch = [&](int d, int t) __attribute__((always_inline)) {
    const int64_t k = kbeg + 8 * (wk + (int64_t)WK * min(t, steps - 1));
#pragma unroll
    for (int i = 0; i < RM; ++i) fa[d][i] = ld(ba, oa[i], k);
#pragma unroll
    for (int j = 0; j < RN; ++j) fb[d][j] = ld(bb, ob[j], k);
  };
  auto multiply = [&](int d) __attribute__((always_inline)) {
    if (abs_in) {
#pragma unroll
      for (int i = 0; i < RM; ++i) fa[d][i] = double2{fabs(fa[d][i].x), fabs(fa[d][i].y)};
#pragma unroll
      for (int j = 0; j < RN; ++j) fb[d][j] = double2{fabs(fb[d][j].x), fabs(fb[d][j].y)};
    }
#pragma unroll
    for (int i = 0; i < RM; ++i)
#pragma unroll
      for (int j = 0; j < RN; ++j) acc[i][j] = mfma16x16x4(fa[d][i].x, fb[d][j].x, acc[i][j]);
#pragma unroll
    for (int i = 0; i < RM; ++i)
#pragma unroll
      for (int j = 0; j < RN; ++j) acc[i][j] = mfma16x16x4(fa[d][i].y, fb[d][j].y, acc[i][j]);
  };
  if (steps > 0) {
#pragma unroll
    for (int d = 0; d < D - 1; ++d) fetch(d, d);
    for (int t = 0; t < steps; t += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        fetch((d + D - 1) % D, t + d + D - 1);
        if (t + d < steps) multiply(d);
      }
    }
  }
  double* out = partial + (int64_t)blockIdx.y * m * n;
  __shared__ double red[WK > 1 ? WK : 1][WK > 1 ? WM * WN * RN * 256 : 1];
#pragma unroll
  for (int i = 0; i < RM; ++i) {
    if constexpr (WK > 1) {
      if (i > 0) __syncthreads();
#pragma unroll
      for (int j = 0; j < RN; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[wk][((wmn * RN + j) * 4 + v) * 64 + lane] = acc[i][j][v];
      __syncthreads();
      if (wk > 0) continue;
#pragma unroll
      for (int j = 0; j < RN; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          double s = acc[i][j][v];
#pragma unroll
          for (int w = 1; w < WK; ++w) s += red[w][((wmn * RN + j) * 4 + v) * 64 + lane];
          acc[i][j][v] = s;
        }
    }
#pragma unroll
    for (int j = 0; j < RN; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = tm * TM + (wm * RM + i) * 16 + g + 4 * v;
        const int col = tn * TN + (wn * RN + j) * 16 + li;
        if (row < m && col < n) out[(int64_t)row * n + col] = acc[i][j][v];
      }
  }
}

// C[i] = scale * sum_s partial[s][i]: 256 / G outputs per workgroup, G
// threads per output each summing the splits s = g mod G in order, combined
// in a fixed order.  sym_tile > 0: only the tiles of that size on and below
// the diagonal were computed; an output above them is its mirror image.
template <int G>
__global__ __launch_bounds__(256) void k_reduce_splits(const double* __restrict__ partial,
                                                       int nsplit, int64_t count, int n,
                                                       int sym_tile, double scale,
                                                       double* __restrict__ C,
                                                       const int* __restrict__ skip) {
  if (skip && *skip != 0) return;
  constexpr int O = 256 / G;
  __shared__ double red[G][O];
  const int o = threadIdx.x % O, g = threadIdx.x / O;
  const int64_t i = (int64_t)blockIdx.x * O + o;
  int64_t src = i;
  if (sym_tile > 0 && i < count) {
    const int r = (int)(i / n), c = (int)(i % n);
    if (r / sym_tile < c / sym_tile) src = (int64_t)c * n + r;
  }
  double s = 0.0;
  if (i < count) {
#pragma unroll 4
    for (int k = g; k < nsplit; k += G) s += partial[(int64_t)k * count + src];
  }
  red[g][o] = s;
  __syncthreads();
  if (g == 0 && i < count) {
#pragma unroll
    for (int q = 1; q < G; ++q) s += red[q][o];
    C[i] = scale * s;
  }
}

namespace {

// Wave tile rows (in 16s) and wave rows of a product with m output rows: the
// smallest that covers them, up to 64 rows per wave and two wave rows.
struct AbtShape {
  int r, w;
};
AbtShape abt_shape(int m) {
  if (m <= 16) return {1, 1};
  if (m <= 32) return {2, 1};
  if (m <= 64) return {4, 1};
  return {4, 2};
}
int abt_tile(int m) {
  const AbtShape s = abt_shape(m);
  return 16 * s.r * s.w;
}

template <int RM, int WM, int RN, int WN>
void abt_launch(bool vec, dim3 grid, hipStream_t s, const double* A, const double* B, int m, int n,
                int64_t K, int64_t kchunk, int tiles_n, bool abs_in, double* partial,
                const int* skip) {
  if (vec)
    hipLaunchKernelGGL((k_gemm_abt<RM, WM, RN, WN, true>), grid, dim3(256), 0, s, A, B, m, n, K,
                       kchunk, tiles_n, abs_in, partial, skip);
  else
    hipLaunchKernelGGL((k_gemm_abt<RM, WM, RN, WN, false>), grid, dim3(256), 0, s, A, B, m, n, K,
                       kchunk, tiles_n, abs_in, partial, skip);
}

}  // namespace

// Workgroups along K: together two per CU for the large tiles (two are
// resident; 1024 instead of 512 workgroups took 13 us more at 128 x 128, and
// the reduction of twice the partial sums 10 us more) and four for the
// smaller ones; at least eight steps per wave; and no more partial sums than
// the operands themselves are large (each is written and read once more).
static int abt_splits(int m, int n, int64_t K, int64_t tiles) {
  const AbtShape sm = abt_shape(m), sn = abt_shape(n);
  const int wk = 4 / (sm.w * sn.w);
  const int64_t want = sm.r * sn.r * sm.w * sn.w >= 32 ? 512 : 1024;
  int64_t ns = want / tiles;
  ns = std::min(ns, (K + 64 * wk - 1) / (64 * wk));
  ns = std::min(ns, K * (m + n) / (2 * (int64_t)m * n));
  return (int)std::max<int64_t>(ns, 1);
}

// The most that a product of these sizes takes: a square one may be symmetric,
// whose fewer tiles (one triangle) are split further.
int gemm_abt_splits(int m, int n, int64_t K) {
  const int64_t tm = (m + abt_tile(m) - 1) / abt_tile(m), tn = (n + abt_tile(n) - 1) / abt_tile(n);
  return abt_splits(m, n, K, m == n ? tm * (tm + 1) / 2 : tm * tn);
}

hipError_t launch_gemm_abt(const double* A, const double* B, int m, int n, int64_t K,
                           double scale, double* C, double* partial, int nsplit, bool abs_inputs,
                           const int* skip, hipStream_t s) {
  const AbtShape sm = abt_shape(m), sn = abt_shape(n);
  const int tiles_m = (m + abt_tile(m) - 1) / abt_tile(m);
  const int tiles_n = (n + abt_tile(n) - 1) / abt_tile(n);
  const int wk = 4 / (sm.w * sn.w);
  // a product of one operand with itself is symmetric, bit for bit (the same
  // products in the same order): the tiles above the diagonal are mirrored.  More
  // than one tile: more than 128 rows, which are large tiles
  const bool sym = A == B && m == n && tiles_m > 1;
  const int tiles = sym ? tiles_m * (tiles_m + 1) / 2 : tiles_m * tiles_n;
  nsplit = std::min(nsplit, abt_splits(m, n, K, tiles));
  int64_t kchunk = (K + nsplit - 1) / nsplit;
  const int unit = m > 64 && n > 64 ? kAbtKT : 8 * wk;
  kchunk = ((kchunk + unit - 1) / unit) * unit;
  const bool vec = K % 8 == 0 && reinterpret_cast<uintptr_t>(A) % 16 == 0 &&
                   reinterpret_cast<uintptr_t>(B) % 16 == 0;
  const dim3 grid(tiles, nsplit);
#define ACEX_ABT(RM, WM, RN, WN)                                                              \
  if (sm.r == RM && sm.w == WM && sn.r == RN && sn.w == WN)                                   \
    abt_launch<RM, WM, RN, WN>(vec, grid, s, A, B, m, n, K, kchunk, tiles_n, abs_inputs,      \
                               partial, skip);
#define ACEX_ABT_ROW(RM, WM) \
  ACEX_ABT(RM, WM, 1, 1) ACEX_ABT(RM, WM, 2, 1) ACEX_ABT(RM, WM, 4, 1)
  ACEX_ABT_ROW(1, 1) ACEX_ABT_ROW(2, 1) ACEX_ABT_ROW(4, 1) ACEX_ABT_ROW(4, 2)
  ACEX_ABT(1, 1, 4, 2) ACEX_ABT(2, 1, 4, 2) ACEX_ABT(4, 1, 4, 2)
  if (m > 64 && n > 64) {
    if (vec)
      hipLaunchKernelGGL(k_gemm_abt_tile<true>, grid, dim3(256), 0, s, A, B, m, n, K, kchunk,
                         tiles_n, sym, abs_inputs, partial, skip);
    else
      hipLaunchKernelGGL(k_gemm_abt_tile<false>, grid, dim3(256), 0, s, A, B, m, n, K, kchunk,
                         tiles_n, sym, abs_inputs, partial, skip);
  }
#undef ACEX_ABT_ROW
#undef ACEX_ABT
  const int64_t count = (int64_t)m * n;
  const int sym_tile = sym ? abt_tile(m) : 0;
  if (count < 2048)
    hipLaunchKernelGGL(k_reduce_splits<64>, dim3((unsigned)((count + 3) / 4)), dim3(256), 0, s,
                       partial, nsplit, count, n, sym_tile, scale, C, skip);
  else
    hipLaunchKernelGGL(k_reduce_splits<16>, dim3((unsigned)((count + 15) / 16)), dim3(256), 0, s,
                       partial, nsplit, count, n, sym_tile, scale, C, skip);
  return hipGetLastError();
}

// ------------------------------------------------------------------ Out = A B (A small)
// A (16 RB rows of it) sits in LDS for the whole launch; every wave streams
// its own 32-column tiles of B past it, with no barrier after the first: B's
// MFMA operand (row k, 16 adjacent columns) is contiguous in memory, so it
// goes straight to registers, two columns per lane (256 contiguous bytes of a
// row), 32 rows ahead of the multiplication (16 ahead, the loads issued after
// a tile's stores waited for these: 708 against 588 us).  One wave's stores
// and loads run under the other waves' matrix instructions, and B is read once
// per 16 RB output rows.  128 x 128 over 884,736 columns: 588 us, 397 us with
// tri; staging B through LDS in 16-row slabs with two barriers each, and
// reading it twice, took 700 us.  4 rows: 199 against 332 us, 4.7 TB/s.
//
// LDS: sA[k][row], row fastest; an odd k's rows are stored with bit 4 flipped,
// which puts the 16 rows that adjacent lane groups read on different banks.
//
// tri: A is lower triangular; row block b needs only k < 16 (b + 1).
// VEC: R even, 16-byte aligned B and Out; else scalar accesses.
constexpr int kAbThreads = 512;
constexpr int kAbCols = 32;  // columns per wave tile

template <int RB, int KCAP, bool VEC>
__global__ __launch_bounds__(kAbThreads) __attribute__((amdgpu_waves_per_eu(2))) void k_gemm_ab(
    const double* __restrict__ A, const double* __restrict__ B, int m, int k, int64_t R,
    double scale, double* __restrict__ Out, bool tri, int nrb, const int* __restrict__ skip) {
  if (skip && *skip != 0) return;
  constexpr int P = 16 * RB;
  __shared__ double sA[KCAP * P];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, g = lane >> 4;
  // the row blocks of one column group are consecutive on one XCD
  // (workgroup b runs on XCD b mod 8): they find B's rows in its L2
  const int xcd = blockIdx.x & 7, q = blockIdx.x >> 3;
  const int rb0 = (q % nrb) * RB;  // first 16-row block
  const int group = (q / nrb) * 8 + xcd, groups = (gridDim.x / 8 / nrb) * 8;
  const int kblocks = tri ? min((k + 15) / 16, rb0 + RB) : (k + 15) / 16;
  auto place = [](int kk, int row) __attribute__((always_inline)) {
    return kk * P + (RB > 1 ? row ^ ((kk & 1) << 4) : row);
  };
  for (int e = tid; e < kblocks * 16 * P; e += kAbThreads) {
    // 16 rows x 4 k per 64 threads
    const int c = e >> 6, row = (c % RB) * 16 + (e & 15), kk = (c / RB) * 4 + ((e >> 4) & 3);
    const int r = rb0 * 16 + row;
    sA[place(kk, row)] = (r < m && kk < k) ? A[(int64_t)r * k + kk] : 0.0;
  }
  __syncthreads();
  const int nact = min(RB, (m - rb0 * 16 + 15) / 16);  // row blocks with a row
  const int64_t tiles = (R + kAbCols - 1) / kAbCols;
  const int64_t stride = (int64_t)groups * (kAbThreads / 64);
  double2 cur[4], nxt[4], far[4];
  auto load = [&](double2* v, int64_t tile, int kb) __attribute__((always_inline)) {
    const int64_t col = tile * kAbCols + 2 * li;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int kk = kb * 16 + 4 * s + g;
      v[s] = double2{0.0, 0.0};
      if constexpr (VEC) {
        if (kk < k && col < R) v[s] = *reinterpret_cast<const double2*>(B + (int64_t)kk * R + col);
      } else {
        if (kk < k && col < R) v[s].x = B[(int64_t)kk * R + col];
        if (kk < k && col + 1 < R) v[s].y = B[(int64_t)kk * R + col + 1];
      }
    }
  };
  int64_t tile = (int64_t)group * (kAbThreads / 64) + wave;
  if (tile >= tiles) return;
  // 16-row block kb + ahead of the wave's stream of blocks, past a tile's end
  // the next tile's
  auto load_ahead = [&](double2* v, int kb, int ahead) __attribute__((always_inline)) {
    int64_t t = tile;
    for (kb += ahead; kb >= kblocks; kb -= kblocks) t += stride;
    if (t < tiles) load(v, t, kb);
  };
  load(cur, tile, 0);
  load_ahead(nxt, 0, 1);
  for (; tile < tiles; tile += stride) {
    d4 acc[RB][2];
#pragma unroll
    for (int i = 0; i < RB; ++i) acc[i][0] = acc[i][1] = d4{0.0, 0.0, 0.0, 0.0};
    for (int kb = 0; kb < kblocks; ++kb) {
      load_ahead(far, kb, 2);
#pragma unroll
      for (int i = 0; i < RB; ++i) {
        if (i < nact && (!tri || rb0 + i >= kb)) {
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            const double a = sA[place(kb * 16 + 4 * s + g, i * 16 + li)];
            acc[i][0] = mfma16x16x4(a, cur[s].x, acc[i][0]);
            acc[i][1] = mfma16x16x4(a, cur[s].y, acc[i][1]);
          }
        }
      }
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        cur[s] = nxt[s];
        nxt[s] = far[s];
      }
    }
    const int64_t col = tile * kAbCols + 2 * li;
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = (rb0 + i) * 16 + g + 4 * v;
        const double2 o = {scale * acc[i][0][v], scale * acc[i][1][v]};
        if constexpr (VEC) {
          if (row < m && col < R) *reinterpret_cast<double2*>(Out + (int64_t)row * R + col) = o;
        } else {
          if (row < m && col < R) Out[(int64_t)row * R + col] = o.x;
          if (row < m && col + 1 < R) Out[(int64_t)row * R + col + 1] = o.y;
        }
      }
  }
}

namespace {

// workgroups resident per CU (LDS, registers), looked up once per kernel
template <int RB, int KCAP>
int ab_per_cu() {
  static std::atomic<int> cached{0};
  int occ = cached.load(std::memory_order_relaxed);
  if (occ > 0) return occ;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k_gemm_ab<RB, KCAP, true>, kAbThreads,
                                                   0) != hipSuccess ||
      occ < 1)
    occ = 1;
  cached.store(occ, std::memory_order_relaxed);
  return occ;
}

template <int RB, int KCAP>
hipError_t ab_launch(const double* A, const double* B, int m, int k, int64_t R, double scale,
                     double* Out, bool tri, const int* skip, hipStream_t s) {
  const int nrb = (m + 16 * RB - 1) / (16 * RB);
  const int64_t tiles = (R + kAbCols - 1) / kAbCols, waves = kAbThreads / 64;
  // column groups: as many as are resident, in eights, at most one per eight tiles
  int64_t groups = (int64_t)device_cus() * ab_per_cu<RB, KCAP>() / nrb / 8 * 8;
  groups = std::max<int64_t>(8, std::min(groups, ((tiles + waves - 1) / waves + 7) / 8 * 8));
  const dim3 grid((unsigned)(groups * nrb));
  const bool vec = R % 2 == 0 && reinterpret_cast<uintptr_t>(B) % 16 == 0 &&
                   reinterpret_cast<uintptr_t>(Out) % 16 == 0;
  if (vec)
    hipLaunchKernelGGL((k_gemm_ab<RB, KCAP, true>), grid, dim3(kAbThreads), 0, s, A, B, m, k, R,
                       scale, Out, tri, nrb, skip);
  else
    hipLaunchKernelGGL((k_gemm_ab<RB, KCAP, false>), grid, dim3(kAbThreads), 0, s, A, B, m, k, R,
                       scale, Out, tri, nrb, skip);
  return hipGetLastError();
}

}  // namespace

// Rows per workgroup: those of the output, up to what LDS holds of A (128 KB:
// 128 rows of 128, 64 of 256, 32 of 512).
hipError_t launch_gemm_ab(const double* A, const double* B, int m, int k, int64_t R, double scale,
                          double* Out, bool tri, const int* skip, hipStream_t s) {
  if (k < 1 || k > 512) return hipErrorInvalidValue;
#define ACEX_AB(RB, KCAP) return ab_launch<RB, KCAP>(A, B, m, k, R, scale, Out, tri, skip, s)
  if (m <= 16) {
    if (k <= 128) ACEX_AB(1, 128);
    ACEX_AB(1, 512);
  }
  if (m <= 32 || k > 256) {
    if (k <= 128) ACEX_AB(2, 128);
    ACEX_AB(2, 512);
  }
  if (m <= 64 || k > 128) {
    if (k <= 128) ACEX_AB(4, 128);
    ACEX_AB(4, 256);
  }
  ACEX_AB(8, 128);
#undef ACEX_AB
}

// ------------------------------------------------------------------ Cholesky and L^{-1}
// -M = L L^T (lower, positive diagonal), then X = L^{-1}, in blocks of 32
// columns (a partial last block when 32 does not divide n).
//
// k_chol_left: one workgroup of 1024 threads, left-looking, L built in place
// in the L buffer (at these sizes it stays in the CU's caches).  Block column
// J (columns j0 .. j0 + w - 1):
//   1. the finished columns 0 .. j0-1 of its rows are staged in LDS,
//      transposed: lj[k][c] = L[j0 + c][k];
//   2. every row i >= j0: A[i][j0 + c] -= sum_{k < j0} L[i][k] lj[k][c]
//      (thread = (row, c), k in increasing order);
//   3. the diagonal block is factored by one wave, a row per lane in registers,
//      the pivot column's values read across lanes (in LDS, with three barriers
//      per column, it took 1 us per column and most of the factorisation); a
//      non-positive (or NaN) pivot stops the factorisation with info = column + 1;
//   4. the rows below it are solved against it, L[i][J] = A[i][J] D^{-T}
//      (one thread per row, the row in registers).
// k_tri_inv: one workgroup per block column J of X; forward block
// substitution down the row blocks I >= J with the block column in LDS:
//   X[I][J] = D_I^{-1} (delta - sum_{J <= K < I} L[I][K] X[K][J]),
// the triangular solve by one thread per column with the column in
// registers.  Both are skipped after a failed factorisation (X undefined).  Up
// to 32 orbitals k_chol_left inverts its one block itself.
constexpr int kCholNB = 32;
constexpr int kCholMaxN = 512;

// v of lane l (uniform)
__device__ __forceinline__ double lane_of(double v, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                          __builtin_amdgcn_readlane(__double2loint(v), l));
}

__global__ __launch_bounds__(1024) void k_chol_left(const double* __restrict__ M, int n,
                                                    double* __restrict__ L,
                                                    int* __restrict__ info,
                                                    double* __restrict__ trace,
                                                    double* __restrict__ X) {
  __shared__ double lj[kCholMaxN - kCholNB][kCholNB];
  __shared__ double dblk[kCholNB][kCholNB + 1];
  __shared__ int bad;
  const int tid = threadIdx.x;
  const int c = tid % kCholNB, il = tid / kCholNB;
  for (int64_t e = tid; e < (int64_t)n * n; e += 1024) {
    const int i = (int)(e / n), j = (int)(e % n);
    L[e] = (j <= i) ? -M[e] : 0.0;
  }
  if (tid == 0) bad = 0;
  if (tid < 64) {
    // tr(M): lane sums, then across the wave, in a fixed order
    double t = 0.0;
    for (int i = tid; i < n; i += 64) t += M[(int64_t)i * n + i];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) t += __shfl_xor(t, off, 64);
    if (tid == 0) *trace = t;
  }
  __syncthreads();
  for (int j0 = 0; j0 < n; j0 += kCholNB) {
    const int w = min(kCholNB, n - j0);
    // 1. stage the block's rows of the finished columns
    for (int e = tid; e < j0 * kCholNB; e += 1024) {
      const int k = e / kCholNB, cc = e % kCholNB;
      lj[k][cc] = cc < w ? L[(int64_t)(j0 + cc) * n + k] : 0.0;
    }
    __syncthreads();
    // 2. left-looking update of the block column
    if (c < w) {
      for (int i = j0 + il; i < n; i += 1024 / kCholNB) {
        const double* __restrict__ li = L + (int64_t)i * n;
        double s = li[j0 + c];
#pragma unroll 8
        for (int k = 0; k < j0; ++k) s -= li[k] * lj[k][c];
        L[(int64_t)i * n + j0 + c] = s;
      }
    }
    __syncthreads();
    // 3. the diagonal block, factored in LDS
    for (int e = tid; e < w * w; e += 1024) {
      const int r = e / w, cc = e % w;
      dblk[r][cc] = L[(int64_t)(j0 + r) * n + j0 + cc];
    }
    __syncthreads();
    if (tid < 64) {
      const int r = tid;  // lanes past w hold zeros and never show
      double row[kCholNB];
#pragma unroll
      for (int cc = 0; cc < kCholNB; ++cc) row[cc] = r < w && cc < w ? dblk[r][cc] : 0.0;
      bool ok = true;
#pragma unroll
      for (int j = 0; j < kCholNB; ++j) {
        if (ok && j < w) {
          const double d = lane_of(row[j], j);
          if (!(d > 0.0)) {
            ok = false;
            if (tid == 0) bad = j0 + j + 1;
          } else {
            const double ljj = sqrt(d);
            row[j] = r == j ? ljj : r > j ? row[j] / ljj : row[j];
#pragma unroll
            for (int q = j + 1; q < kCholNB; ++q)
              if (q < w) row[q] -= row[j] * lane_of(row[j], q);
          }
        }
      }
#pragma unroll
      for (int cc = 0; cc < kCholNB; ++cc)
        if (r < w && cc < w) dblk[r][cc] = row[cc];
    }
    __syncthreads();
    if (bad) break;
    for (int e = tid; e < w * w; e += 1024) {
      const int r = e / w, cc = e % w;
      L[(int64_t)(j0 + r) * n + j0 + cc] = cc <= r ? dblk[r][cc] : 0.0;
    }
    // 4. rows below: forward substitution against the diagonal block (w = 32
    // whenever rows remain below it)
    const int i = j0 + kCholNB + tid;
    if (w == kCholNB && i < n) {
      double* __restrict__ li = L + (int64_t)i * n + j0;
      double x[kCholNB];
#pragma unroll
      for (int cc = 0; cc < kCholNB; ++cc) x[cc] = li[cc];
#pragma unroll
      for (int cc = 0; cc < kCholNB; ++cc) {
#pragma unroll
        for (int k = 0; k < cc; ++k) x[cc] -= x[k] * dblk[cc][k];
        x[cc] /= dblk[cc][cc];
      }
#pragma unroll
      for (int cc = 0; cc < kCholNB; ++cc) li[cc] = x[cc];
    }
    __syncthreads();
  }
  __syncthreads();
  if (tid == 0) *info = bad;
  // one block: its inverse right here, a column per thread
  if (X && !bad && tid < n) {
    double x[kCholNB];
#pragma unroll
    for (int r = 0; r < kCholNB; ++r) {
      if (r < n) {
        double v = r == tid ? 1.0 : 0.0;
#pragma unroll
        for (int k = 0; k < r; ++k) v -= dblk[r][k] * x[k];
        x[r] = v / dblk[r][r];
        X[(int64_t)r * n + tid] = r >= tid ? x[r] : 0.0;
      }
    }
  }
}

__global__ __launch_bounds__(1024) void k_tri_inv(const double* __restrict__ L, int n,
                                                  double* __restrict__ X,
                                                  const int* __restrict__ info) {
  __shared__ double xs[kCholMaxN][kCholNB];  // rows j0 .. n-1 of the block column
  __shared__ double dblk[kCholNB][kCholNB + 1];
  if (*info != 0) return;
  const int j0 = blockIdx.x * kCholNB;
  const int w = min(kCholNB, n - j0);
  const int tid = threadIdx.x, c = tid % kCholNB, il = tid / kCholNB;
  for (int i0 = j0; i0 < n; i0 += kCholNB) {
    const int h = min(kCholNB, n - i0);
    // right-hand sides of row block I
    if (il < h && c < w) {
      const int i = i0 + il;
      const double* __restrict__ li = L + (int64_t)i * n;
      double s = (i == j0 + c) ? 1.0 : 0.0;
#pragma unroll 8
      for (int k = j0; k < i0; ++k) s -= li[k] * xs[k - j0][c];
      xs[i - j0][c] = s;
    }
    for (int e = tid; e < h * h; e += 1024) {
      const int r = e / h, cc = e % h;
      dblk[r][cc] = L[(int64_t)(i0 + r) * n + i0 + cc];
    }
    __syncthreads();
    // X[I][J] = D_I^{-1} (right-hand sides): one thread per column
    if (tid < w) {
      double x[kCholNB];
#pragma unroll
      for (int r = 0; r < kCholNB; ++r) x[r] = r < h ? xs[i0 - j0 + r][tid] : 0.0;
#pragma unroll
      for (int r = 0; r < kCholNB; ++r) {
        if (r < h) {
#pragma unroll
          for (int k = 0; k < r; ++k) x[r] -= dblk[r][k] * x[k];
          x[r] /= dblk[r][r];
        }
      }
#pragma unroll
      for (int r = 0; r < kCholNB; ++r)
        if (r < h) xs[i0 - j0 + r][tid] = x[r];
    }
    __syncthreads();
  }
  for (int e = tid; e < n * kCholNB; e += 1024) {
    const int i = e / kCholNB, cc = e % kCholNB;
    if (cc >= w) continue;
    const int col = j0 + cc;
    X[(int64_t)i * n + col] = (i >= col) ? xs[i - j0][cc] : 0.0;
  }
}

hipError_t launch_cholesky_inv(const double* M, int n, double* L, double* Linv, int* info,
                               double* trace, hipStream_t s) {
  if (n > kCholMaxN || n < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_chol_left, dim3(1), dim3(1024), 0, s, M, n, L, info, trace,
                     n <= kCholNB ? Linv : (double*)nullptr);
  if (n > kCholNB)
    hipLaunchKernelGGL(k_tri_inv, dim3((n + kCholNB - 1) / kCholNB), dim3(1024), 0, s, L, n, Linv,
                     info);
  return hipGetLastError();
}

// ------------------------------------------------------------------ reductions
// Fixed-order weighted sum: 256 contiguous chunks, then the chunk sums in order.
__global__ __launch_bounds__(256) void k_weighted_sum(const double* __restrict__ e,
                                                      const double* __restrict__ w, int count,
                                                      double* __restrict__ out) {
  __shared__ double part[256];
  const int tid = threadIdx.x;
  const int per = (count + 255) / 256;
  double s = 0.0;
  const int b = tid * per;
  for (int i = b; i < b + per && i < count; ++i) s += w[i] * e[i];
  part[tid] = s;
  __syncthreads();
  if (tid == 0) {
    double t = 0.0;
    for (int i = 0; i < 256; ++i) t += part[i];
    *out = t;
  }
}

hipError_t launch_weighted_sum(const double* e, const double* w, int count, double* out,
                               hipStream_t s) {
  hipLaunchKernelGGL(k_weighted_sum, dim3(1), dim3(256), 0, s, e, w, count, out);
  return hipGetLastError();
}

__device__ __forceinline__ double pair_weight(int code, int n_orb, double wscale) {
  return wscale * (code / n_orb == code % n_orb ? 1.0 : 2.0);
}

// sum of w e in a fixed order: 1024 interleaved runs, then a tree over them
__global__ __launch_bounds__(1024) void k_pair_sum(const double* __restrict__ e,
                                                   const int* __restrict__ codes, int count,
                                                   int n_orb, double wscale,
                                                   double* __restrict__ out) {
  __shared__ double part[1024];
  const int tid = threadIdx.x;
  double s = 0.0;
#pragma unroll 4
  for (int i = tid; i < count; i += 1024)
    if (codes[i] >= 0) s += pair_weight(codes[i], n_orb, wscale) * e[i];
  part[tid] = s;
  for (int d = 512; d >= 1; d /= 2) {
    __syncthreads();
    if (tid < d) part[tid] += part[tid + d];
  }
  if (tid == 0) *out = part[0];
}

__global__ void k_scatter_pairs(const double* __restrict__ e, const int* __restrict__ codes,
                                int count, int n_orb, double wscale,
                                double* __restrict__ pair_e) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count || codes[i] < 0) return;
  pair_e[codes[i]] = pair_weight(codes[i], n_orb, wscale) * e[i];
}

hipError_t launch_pair_energies(const double* e, const int* codes, int count, int n_orb,
                                double weight_scale, double* ex, double* pair_e, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_pair_sum, dim3(1), dim3(1024), 0, s, e, codes, count, n_orb, weight_scale,
                     ex);
  hipLaunchKernelGGL(k_scatter_pairs, dim3((count + 255) / 256), dim3(256), 0, s, e, codes, count,
                     n_orb, weight_scale, pair_e);
  return hipGetLastError();
}

}  // namespace acex
