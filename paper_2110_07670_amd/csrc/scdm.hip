// SCDM localisation on gfx950 (arXiv 2110.07670, section "s-MTACE Method":
// a rank-revealing QR of Psi^* picks columns of the density matrix, which are
// orthonormalised; section "s'-MTACE Method": only grid points with
// rho > <rho> and |grad rho| < <|grad rho|> enter the QR).
//
//   preselection : k_density, k_grad_norm (central differences, periodic),
//                  fixed-order means, and an ordered compaction of the kept
//                  points (count per block, one scan, in-block prefix);
//   pivoted QR   : Businger-Golub column pivoting on the n_orb x m matrix,
//                  stored point-major (each column contiguous); one launch
//                  per step (k_qr_step);
//   orthonormalisation : Newton-Schulz iteration Y <- (3 Y - Y Y^T Y) / 2
//                  from Y = A_C^T / ||A_C||_F, which converges to the
//                  orthogonal polar factor; two small MFMA launches per
//                  iteration (k_ns_gram, k_ns_step).
#include <algorithm>

#include "kernels.h"

namespace acex {

namespace {

constexpr int kSelBlock = 1024;  // points per compaction block (256 threads x 4)
constexpr int kScdmSumBlocks = 1024;  // partial sums of the means

__device__ __forceinline__ double block_sum_1024(double v, double* red) {
  // fixed-order: wave tree, then the wave partials in order
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[wid] = v;
  __syncthreads();
  double s = 0.0;
  const int nw = (blockDim.x + 63) >> 6;
  for (int i = 0; i < nw; ++i) s += red[i];
  return s;
}

// v of the lane that the DPP control names (within rows of 16 lanes)
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double lane_value(double v, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                          __builtin_amdgcn_readlane(__double2loint(v), l));
}
// Sum over groups of G adjacent lanes, fixed order, the same value in every
// lane of a group: a butterfly (xor 1, xor 2, then the mirrors, which pair
// the quads and the halves of a row as xor 4 and xor 8 do).  Register moves up
// to a row of 16 lanes: a shuffle per step would go through LDS.
template <int G>
__device__ __forceinline__ double group_sum(double v) {
  v += dpp_move<0xB1>(v);                         // quad_perm 1 0 3 2
  v += dpp_move<0x4E>(v);                         // quad_perm 2 3 0 1
  v += dpp_move<0x141>(v);                        // row_half_mirror
  if constexpr (G >= 16) v += dpp_move<0x140>(v);  // row_mirror
  if constexpr (G >= 32) v += __shfl_xor(v, 16, 64);
  if constexpr (G >= 64) v += __shfl_xor(v, 32, 64);
  return v;
}

// rho(r) = sum_i phi_i(r)^2, products and sums rounded one by one, in order
__global__ void k_density(const double* __restrict__ phi, int k, int64_t npts,
                          double* __restrict__ rho) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= npts) return;
  double acc = 0.0;
  for (int i = 0; i < k; ++i) {
    const double f = phi[(int64_t)i * npts + r];
    acc = __dadd_rn(acc, __dmul_rn(f, f));
  }
  rho[r] = acc;
}

__global__ void k_grad_norm(const double* __restrict__ rho, int n, double two_h0, double two_h1,
                            double two_h2, double* __restrict__ g) {
  const int64_t npts = (int64_t)n * n * n;
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= npts) return;
  const int z = (int)(r % n), y = (int)((r / n) % n), x = (int)(r / ((int64_t)n * n));
  const int64_t nn = (int64_t)n * n;
  const int xp = x + 1 == n ? 0 : x + 1, xm = x == 0 ? n - 1 : x - 1;
  const int yp = y + 1 == n ? 0 : y + 1, ym = y == 0 ? n - 1 : y - 1;
  const int zp = z + 1 == n ? 0 : z + 1, zm = z == 0 ? n - 1 : z - 1;
  const int64_t base_x = (int64_t)y * n + z, base_y = (int64_t)x * nn + z,
                base_z = (int64_t)x * nn + (int64_t)y * n;
  const double dx = (rho[xp * nn + base_x] - rho[xm * nn + base_x]) / two_h0;
  const double dy = (rho[base_y + (int64_t)yp * n] - rho[base_y + (int64_t)ym * n]) / two_h1;
  const double dz = (rho[base_z + zp] - rho[base_z + zm]) / two_h2;
  double s = 0.0;
  s = __dadd_rn(s, __dmul_rn(dx, dx));
  s = __dadd_rn(s, __dmul_rn(dy, dy));
  s = __dadd_rn(s, __dmul_rn(dz, dz));
  g[r] = sqrt(s);
}

// per-block partial sums of a and b over a grid-stride range
__global__ __launch_bounds__(256) void k_sum2_partial(const double* __restrict__ a,
                                                      const double* __restrict__ b, int64_t n,
                                                      double* __restrict__ part) {
  __shared__ double red[4];
  double sa = 0.0, sb = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    sa += a[i];
    sb += b[i];
  }
  const double ta = block_sum_1024(sa, red);
  const double tb = block_sum_1024(sb, red);
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = ta;
    part[2 * blockIdx.x + 1] = tb;
  }
}

__global__ __launch_bounds__(256) void k_sum2_final(const double* __restrict__ part, int nblk,
                                                    int64_t n, double* __restrict__ means) {
  __shared__ double red[4];
  double sa = 0.0, sb = 0.0;
  for (int i = threadIdx.x; i < nblk; i += 256) {
    sa += part[2 * i];
    sb += part[2 * i + 1];
  }
  const double ta = block_sum_1024(sa, red);
  const double tb = block_sum_1024(sb, red);
  if (threadIdx.x == 0) {
    means[0] = ta / (double)n;
    means[1] = tb / (double)n;
  }
}

__device__ __forceinline__ bool kept(const double* rho, const double* g, const double* means,
                                     int64_t r) {
  return rho[r] > means[0] && g[r] < means[1];
}

// kept points per block of kSelBlock consecutive points
__global__ __launch_bounds__(256) void k_sel_count(const double* __restrict__ rho,
                                                   const double* __restrict__ g,
                                                   const double* __restrict__ means, int64_t npts,
                                                   int* __restrict__ cnt) {
  __shared__ int red[4];
  const int64_t r0 = (int64_t)blockIdx.x * kSelBlock;
  int c = 0;
  for (int q = 0; q < kSelBlock / 256; ++q) {
    const int64_t r = r0 + q * 256 + threadIdx.x;
    if (r < npts && kept(rho, g, means, r)) ++c;
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) c += __shfl_xor(c, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) cnt[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

// exclusive scan of the block counts: each of 1024 threads scans a run of
// blocks (a few thousand in all), the run totals are scanned in LDS
__global__ __launch_bounds__(1024) void k_sel_scan(const int* __restrict__ cnt, int nblk,
                                                   int* __restrict__ off,
                                                   int* __restrict__ total) {
  __shared__ int sums[1024];
  const int t = threadIdx.x;
  const int per = (nblk + 1023) / 1024, b0 = t * per, b1 = min(b0 + per, nblk);
  int own = 0;
  for (int i = b0; i < b1; ++i) own += cnt[i];
  sums[t] = own;
  __syncthreads();
  for (int d = 1; d < 1024; d *= 2) {
    const int v = t >= d ? sums[t - d] : 0;
    __syncthreads();
    sums[t] += v;
    __syncthreads();
  }
  int s = sums[t] - own;
  for (int i = b0; i < b1; ++i) {
    off[i] = s;
    s += cnt[i];
  }
  if (t == 1023) *total = sums[1023];
}

// write the kept points of each block, in increasing order
__global__ __launch_bounds__(256) void k_sel_write(const double* __restrict__ rho,
                                                   const double* __restrict__ g,
                                                   const double* __restrict__ means, int64_t npts,
                                                   const int* __restrict__ off,
                                                   int* __restrict__ points) {
  __shared__ int wsum[4];
  const int64_t r0 = (int64_t)blockIdx.x * kSelBlock;
  int base = off[blockIdx.x];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  for (int q = 0; q < kSelBlock / 256; ++q) {
    const int64_t r = r0 + q * 256 + threadIdx.x;
    const bool f = r < npts && kept(rho, g, means, r);
    const unsigned long long bal = __ballot(f);
    const int below = __popcll(bal & ((1ull << lane) - 1ull));
    if (lane == 0) wsum[wid] = __popcll(bal);
    __syncthreads();
    int before = 0;
    for (int w = 0; w < wid; ++w) before += wsum[w];
    if (f) points[base + before + below] = (int)r;
    const int tot = wsum[0] + wsum[1] + wsum[2] + wsum[3];
    __syncthreads();
    base += tot;
  }
}

// ---- Pivoted QR, one launch per step.
//
// Columns stay where they are; pos[j] is the place of column j in the pivoted
// order (the step that chose it, below s) and perm the column at each place
// still open, so that ties resolve as if the columns were swapped.  Every
// workgroup of a step finds the pivot by itself from the largest residual
// norm that each workgroup of the step before left in cand (a few KB), reads
// that one column (nobody writes it any more), forms the Householder vector in
// registers, and applies it to its own columns, one wave per column, while it
// looks for the largest residual norm of the next step.  A step takes 12 us at
// the 18,000 columns of 128 that the preselection leaves on the 96^3 grid, the
// same for the first and the last: it is the chain launch, candidates, pivot
// column, sums that bounds it, not the 9 MB it moves on average.  A pivot
// launch by one workgroup over all norms and an apply launch took 11.2 + 9.5.

// A column that may be the next pivot: squared residual norm, place, index.
struct __align__(16) QrCand {
  double norm;
  int pos, col;
};
static_assert(sizeof(QrCand) == kScdmCandBytes, "the workspace holds these");

__device__ __forceinline__ bool cand_less(const QrCand& a, const QrCand& b) {
  return b.norm > a.norm || (b.norm == a.norm && b.pos < a.pos);
}

__device__ __forceinline__ double wave_max(double v) {
  double o = dpp_move<0xB1>(v);
  v = o > v ? o : v;
  o = dpp_move<0x4E>(v);
  v = o > v ? o : v;
  o = dpp_move<0x141>(v);
  v = o > v ? o : v;
  o = dpp_move<0x140>(v);
  v = o > v ? o : v;
  const double a = lane_value(v, 0), b = lane_value(v, 16), c = lane_value(v, 32),
               d = lane_value(v, 48);
  const double ab = b > a ? b : a, cd = d > c ? d : c;
  return cd > ab ? cd : ab;
}

// The best of the workgroup's candidates, in every thread (NaN norms never
// win; col = -1 when there is none).  No candidate holds a NaN: cand_less
// keeps them out.
template <int NT>
__device__ __forceinline__ QrCand cand_best(QrCand c, QrCand* sh) {
  const double best = wave_max(c.norm);
  unsigned long long at = __ballot(c.norm == best);
  QrCand w = {best, 0, 0};
  int l = __ffsll((long long)at) - 1;
  w.pos = __builtin_amdgcn_readlane(c.pos, l);
  w.col = __builtin_amdgcn_readlane(c.col, l);
  for (at &= at - 1; at != 0; at &= at - 1) {  // a tie: the first place
    l = __ffsll((long long)at) - 1;
    const int pos = __builtin_amdgcn_readlane(c.pos, l);
    if (pos < w.pos) {
      w.pos = pos;
      w.col = __builtin_amdgcn_readlane(c.col, l);
    }
  }
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = w;
  __syncthreads();
  c = sh[0];
#pragma unroll
  for (int q = 1; q < NT / 64; ++q)
    if (cand_less(c, sh[q])) c = sh[q];
  return c;
}

constexpr int kQrThreads = 512;

// A (point-major, column j = point points[j], k values at pitch kp = k rounded
// up to even, zero beyond k), the places, and the candidates of the first step.
__global__ __launch_bounds__(kQrThreads) void k_qr_gather(const double* __restrict__ phi,
                                                          const int* __restrict__ points, int m,
                                                          int k, int kp, int64_t npts,
                                                          double* __restrict__ A,
                                                          int* __restrict__ pos,
                                                          int* __restrict__ perm,
                                                          QrCand* __restrict__ cand) {
  __shared__ QrCand sh[kQrThreads / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int waves = gridDim.x * (kQrThreads / 64);
  QrCand best = {-1.0, m, -1};
  for (int j = blockIdx.x * (kQrThreads / 64) + wave; j < m; j += waves) {
    const int64_t pt = points ? (int64_t)points[j] : (int64_t)j;
    double s = 0.0;
#pragma unroll 4
    for (int i = lane; i < kp; i += 64) {
      const double v = i < k ? phi[(int64_t)i * npts + pt] : 0.0;
      A[(int64_t)j * kp + i] = v;
      s += v * v;
    }
    s = group_sum<64>(s);
    if (lane == 0) pos[j] = perm[j] = j;
    const QrCand c = {s, j, j};
    if (cand_less(best, c)) best = c;
  }
  best = cand_best<kQrThreads>(best, sh);
  if (threadIdx.x == 0) cand[blockIdx.x] = best;
}

// Step s: pivot = the largest residual norm, first place on a tie;
// (I - tau v v^T) A[s:, p] = beta e_s; every open column
// A[s:, j] -= tau v (v^T A[s:, j]), its residual norm over rows s + 1 ...
// recomputed; info = s + 1 on a zero column.
// G lanes hold a column, two adjacent rows per lane in each of Q chunks of 2 G
// rows (whole 128-byte lines per column from G = 8 on): 64 / G columns per
// wave at a time, and a column's two sums cost log2(G) lane exchanges for all
// of them at once.  Chunks above row s are left alone.
template <int G, int Q>
__global__ __launch_bounds__(kQrThreads) void k_qr_step(int s, int m, int k, int kp,
                                                        double* __restrict__ A,
                                                        int* __restrict__ pos,
                                                        int* __restrict__ perm,
                                                        const QrCand* __restrict__ cand,
                                                        QrCand* __restrict__ next,
                                                        const int* __restrict__ points,
                                                        int* __restrict__ pivots,
                                                        int* __restrict__ info) {
  constexpr int C = 64 / G;  // columns per wave
  static_assert(2 * G * Q <= kQrThreads, "a thread per row");
  __shared__ QrCand sh[2][kQrThreads / 64];
  __shared__ __align__(16) double sv[kQrThreads];
  const int lane = threadIdx.x & 63, sub = lane % G;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int stride = gridDim.x * (kQrThreads / 64) * C;
  // rows 2 sub + 2 G q and the next of column j
  auto load = [&](double2* a, int j) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int row = 2 * (sub + G * q);
      a[q] = double2{0.0, 0.0};
      if (2 * G * (q + 1) > s && j < m && row < k)
        a[q] = *reinterpret_cast<const double2*>(A + (int64_t)j * kp + row);
    }
  };
  int j = (blockIdx.x * (kQrThreads / 64) + wave) * C + lane / G;
  double2 a[Q];
  load(a, j);  // in flight while the pivot is found
  int pj = j < m ? pos[j] : -1;
  QrCand c = {-1.0, m, -1};
  if (threadIdx.x < gridDim.x) c = cand[threadIdx.x];  // one per workgroup, at most kQrThreads
  c = cand_best<kQrThreads>(c, sh[0]);
  const int cs = __builtin_amdgcn_readfirstlane(perm[s]);
  // no column compares (NaN norms): the one at place s
  const int cj = __builtin_amdgcn_readfirstlane(c.col < 0 ? cs : c.col);
  const int p = __builtin_amdgcn_readfirstlane(c.col < 0 ? s : c.pos);
  // the Householder vector: the column in every group of lanes for its norm
  double2 v[Q];
  load(v, cj);
  const double xt = (int)threadIdx.x < k ? A[(int64_t)cj * kp + threadIdx.x] : 0.0;
  double x0 = 0.0, nx2 = 0.0;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int row = 2 * (sub + G * q);
    if (row < s) v[q].x = 0.0;
    if (row + 1 < s) v[q].y = 0.0;
    nx2 += v[q].x * v[q].x + v[q].y * v[q].y;
    if (s / (2 * G) == q) x0 = lane_value(s & 1 ? v[q].y : v[q].x, (s / 2) % G);
  }
  const double nx = sqrt(group_sum<G>(nx2));
  double tau = 0.0, beta = 0.0;
  if (nx != 0.0) {
    beta = x0 >= 0.0 ? -nx : nx;
    tau = (beta - x0) / beta;
  }
  // one row per thread: a division takes about 40 instructions, and one per
  // row in every wave was most of the step (14.5 us)
  sv[threadIdx.x] = beta == 0.0 || (int)threadIdx.x < s ? 0.0
                    : (int)threadIdx.x == s             ? 1.0
                                                        : xt / (x0 - beta);
  __syncthreads();
#pragma unroll
  for (int q = 0; q < Q; ++q) v[q] = *reinterpret_cast<const double2*>(&sv[2 * (sub + G * q)]);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    pivots[s] = points ? points[cj] : cj;
    if (p != s) perm[p] = cs;  // place s is read by no later step, p > s
    if (nx == 0.0 && *info == 0) *info = s + 1;
  }
  QrCand best = {-1.0, m, -1};
  while (j < m) {
    // the open column at place s moves to the pivot's place
    const int np = j == cj ? s : j == cs ? p : pj;
    if (np != pj && sub == 0) pos[j] = np;
    double w = 0.0;
#pragma unroll
    for (int q = 0; q < Q; ++q) w += v[q].x * a[q].x + v[q].y * a[q].y;
    w = group_sum<G>(w);
    double r = 0.0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int row = 2 * (sub + G * q);
      a[q].x -= tau * v[q].x * w;
      a[q].y -= tau * v[q].y * w;
      if (2 * G * (q + 1) > s && np > s && row < k)
        *reinterpret_cast<double2*>(A + (int64_t)j * kp + row) = a[q];
      if (row > s) r += a[q].x * a[q].x;
      if (row + 1 > s) r += a[q].y * a[q].y;
    }
    r = group_sum<G>(r);
    const QrCand o = {r, np, j};
    if (np > s && cand_less(best, o)) best = o;
    j += stride;
    if (j < m) {
      load(a, j);
      pj = pos[j];
    }
  }
  best = cand_best<kQrThreads>(best, sh[1]);
  if (threadIdx.x == 0) next[blockIdx.x] = best;
}

// ---- Newton-Schulz, two launches per iteration on 16 x 16 tiles, four waves
// each, operands straight from the caches (k <= 512: at most 2 MB a matrix).
// The general products took four launches per iteration (22 us at 128
// orbitals); these two take 3.4 us each on average over the iterations that
// work and those that find the iteration done.

typedef double d4 __attribute__((ext_vector_type(4)));

// acc[i][j] = sum_t X[i0 + i][t] Z(t, j0 + j), Z(t, j) = TRANS ? Z[j][t] : Z[t][j],
// over t in 16s from t0 in strides of dt
template <bool TRANS>
__device__ __forceinline__ d4 ns_tile(const double* X, const double* Z, int k, int i0, int j0,
                                      int t0 = 0, int dt = 16) {
  const int lane = threadIdx.x & 63, li = lane & 15, g = lane >> 4;
  const bool ri = i0 + li < k, rj = j0 + li < k;
  const int64_t xo = (int64_t)min(i0 + li, k - 1) * k;
  const int64_t zr = (int64_t)min(j0 + li, k - 1);
  d4 acc[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) acc[u] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
  for (; t0 < k; t0 += dt) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int t = t0 + 4 * u + g, tc = min(t, k - 1);
      const double x = X[xo + tc], z = TRANS ? Z[zr * k + tc] : Z[(int64_t)tc * k + zr];
      acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(ri && t < k ? x : 0.0,
                                                    rj && t < k ? z : 0.0, acc[u], 0, 0, 0);
    }
  }
  return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

// The same tile by four waves, a quarter of the sum each; the whole in wave 0.
template <bool TRANS>
__device__ __forceinline__ d4 ns_tile4(const double* X, const double* Z, int k, int i0, int j0,
                                       d4 (*red)[64]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  d4 acc = ns_tile<TRANS>(X, Z, k, i0, j0, 16 * wave, 64);
  if (wave > 0) red[wave - 1][lane] = acc;
  __syncthreads();
  if (wave == 0) acc = ((acc + red[0][lane]) + red[1][lane]) + red[2][lane];
  return acc;
}

// Stores tile (i0, j0), i0 >= j0, of G = Y Y^T and its mirror image; the
// tile's largest |G - I| in every lane (a NaN never compares).
__device__ __forceinline__ double ns_gram_tile(d4 acc, double* G, int k, int i0, int j0) {
  const int lane = threadIdx.x & 63, li = lane & 15, g = lane >> 4;
  double e = 0.0;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int i = i0 + g + 4 * v, j = j0 + li;
    if (i < k && j < k) {
      G[(int64_t)i * k + j] = acc[v];
      if (i0 != j0) G[(int64_t)j * k + i] = acc[v];
      const double d = fabs(acc[v] - (i == j ? 1.0 : 0.0));
      e = d > e ? d : e;
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const double o = __shfl_xor(e, off, 64);
    e = o > e ? o : e;
  }
  return e;
}

// Yn = (3 Y - z) / 2, tile (i0, j0), z = G Y
__device__ __forceinline__ void ns_step_tile(d4 z, const double* Y, double* Yn, int k, int i0,
                                             int j0) {
  const int lane = threadIdx.x & 63, li = lane & 15, g = lane >> 4;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int i = i0 + g + 4 * v, j = j0 + li;
    if (i < k && j < k) Yn[(int64_t)i * k + j] = 1.5 * Y[(int64_t)i * k + j] - 0.5 * z[v];
  }
}

// Below 1e-10 two more steps polish the result (the iteration converges
// quadratically there): iteration it is the last one, taking no step, when
// the errors of iterations 0 .. it hold a third value below it.
__device__ __forceinline__ bool ns_done(const double* err, int it) {
  const int lane = threadIdx.x & 63;
  int below = 0;
  for (int b = 0; b <= it; b += 64)
    below += __popcll(__ballot(b + lane <= it && err[min(b + lane, it)] < 1e-10));
  return below > 2;
}

// the largest of non-negative doubles: their bit patterns compare alike
__device__ __forceinline__ void max_into(double* p, double v) {
  atomicMax(reinterpret_cast<unsigned long long*>(p),
            (unsigned long long)__double_as_longlong(v));
}

// Y[j][i] = phi_i(pivot_j), one workgroup per pivot, and the row's square sum
__global__ __launch_bounds__(256) void k_ns_gather(const double* __restrict__ phi,
                                                   const int* __restrict__ pivots, int k,
                                                   int64_t npts, double* __restrict__ Y,
                                                   double* __restrict__ sq) {
  __shared__ double red[4];
  const int j = blockIdx.x;
  const int64_t pt = pivots[j];
  double s = 0.0;
  for (int i = threadIdx.x; i < k; i += 256) {
    const double x = phi[(int64_t)i * npts + pt];
    Y[(int64_t)j * k + i] = x;
    s += x * x;
  }
  s = block_sum_1024(s, red);
  if (threadIdx.x == 0) sq[j] = s;
}

// Y /= ||Y||_F (one workgroup per row); the iteration's state cleared
__global__ __launch_bounds__(256) void k_ns_init(int k, const double* __restrict__ sq,
                                                 double* __restrict__ Y, int iters,
                                                 double* __restrict__ err,
                                                 int* __restrict__ state) {
  __shared__ double red[4];
  double s = 0.0;
  for (int i = threadIdx.x; i < k; i += 256) s += sq[i];
  const double fro = sqrt(block_sum_1024(s, red));
  const double inv = fro > 0.0 ? 1.0 / fro : 0.0;
  for (int i = threadIdx.x; i < k; i += 256) Y[(int64_t)blockIdx.x * k + i] *= inv;
  if (blockIdx.x == 0) {
    for (int i = threadIdx.x; i < iters; i += 256) err[i] = 0.0;
    if (threadIdx.x == 0) {
      state[0] = 0;  // done: the launches below exit
      state[1] = 0;  // which of the two buffers holds the result
    }
  }
}

// tile t of the lower triangle, row by row
__device__ __forceinline__ void lower_tile(int t, int& i, int& j) {
  i = 0;
  while (t > i) t -= ++i;
  j = t;
}

__global__ __launch_bounds__(256) void k_ns_gram(const double* __restrict__ Y,
                                                double* __restrict__ G, int k, int it,
                                                double* __restrict__ err,
                                                const int* __restrict__ state) {
  if (state[0] != 0) return;
  __shared__ d4 red[3][64];
  int i, j;
  lower_tile(blockIdx.x, i, j);
  const d4 acc = ns_tile4<true>(Y, Y, k, 16 * i, 16 * j, red);
  if (threadIdx.x >= 64) return;
  const double e = ns_gram_tile(acc, G, k, 16 * i, 16 * j);
  if (threadIdx.x == 0) max_into(&err[it], e);
}

__global__ __launch_bounds__(256) void k_ns_step(const double* __restrict__ Y,
                                                const double* __restrict__ G,
                                                double* __restrict__ Yn, int k, int it,
                                                const double* __restrict__ err,
                                                int* __restrict__ state) {
  // after the last iteration err stays 0, so every later launch ends here too
  if (ns_done(err, it)) {
    if (blockIdx.x == 0 && threadIdx.x == 0 && state[0] == 0) {
      state[0] = 1;
      state[1] = it & 1;
    }
    return;
  }
  __shared__ d4 red[3][64];
  const int T = (k + 15) / 16;
  const int i0 = 16 * ((int)blockIdx.x / T), j0 = 16 * ((int)blockIdx.x % T);
  const d4 z = ns_tile4<false>(G, Y, k, i0, j0, red);
  if (threadIdx.x < 64) ns_step_tile(z, Y, Yn, k, i0, j0);
}

// Iterations it0 .. iters - 1 in one workgroup, for the rare matrix that the
// launched iterations leave unfinished (ns_launched); exits at once otherwise.
// Buffers and err are read and written by one workgroup only, with a barrier
// between.
__global__ __launch_bounds__(1024) void k_ns_tail(double* Y0, double* Y1, double* G, int k,
                                                  int it0, int iters, double* err, int* state) {
  if (state[0] != 0) return;
  const int T = (k + 15) / 16, wave = threadIdx.x >> 6;
  int below = 0;  // errors of the iterations so far below 1e-10 (ns_done)
  for (int q = 0; q < it0; ++q) below += err[q] < 1e-10;
  for (int it = it0; it < iters; ++it) {
    double* Y = (it & 1) ? Y1 : Y0;
    double* Yn = (it & 1) ? Y0 : Y1;
    for (int t = wave; t < T * (T + 1) / 2; t += 16) {
      int i, j;
      lower_tile(t, i, j);
      const double e =
          ns_gram_tile(ns_tile<true>(Y, Y, k, 16 * i, 16 * j), G, k, 16 * i, 16 * j);
      if ((threadIdx.x & 63) == 0) max_into(&err[it], e);
    }
    __threadfence();
    __syncthreads();
    // read past the caches, where the maximum was formed
    below += __hip_atomic_load(&err[it], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < 1e-10;
    if (below > 2) {
      if (threadIdx.x == 0) {
        state[0] = 1;
        state[1] = it & 1;
      }
      return;
    }
    for (int t = wave; t < T * T; t += 16)
      ns_step_tile(ns_tile<false>(G, Y, k, 16 * (t / T), 16 * (t % T)), Y, Yn, k, 16 * (t / T),
                   16 * (t % T));
    __syncthreads();
  }
}

__global__ void k_set_int(int* __restrict__ p, int v) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *p = v;
}

// the result into Y0; info = k + 1 if the iteration did not converge
__global__ __launch_bounds__(256) void k_ns_finish(const int* __restrict__ state, int iters, int k,
                                                   double* __restrict__ Y0,
                                                   const double* __restrict__ Y1,
                                                   int* __restrict__ info) {
  const int which = state[0] != 0 ? state[1] : iters & 1;
  if (which != 0)
    for (int i = threadIdx.x; i < k; i += 256)
      Y0[(int64_t)blockIdx.x * k + i] = Y1[(int64_t)blockIdx.x * k + i];
  if (threadIdx.x == 0 && blockIdx.x == 0 && *info == 0 && state[0] == 0) *info = k + 1;
}

}  // namespace

int64_t scdm_sel_blocks(int64_t npts) { return (npts + kSelBlock - 1) / kSelBlock; }
int scdm_sum_blocks() { return kScdmSumBlocks; }

hipError_t launch_set_int(int* p, int v, hipStream_t s) {
  hipLaunchKernelGGL(k_set_int, dim3(1), dim3(64), 0, s, p, v);
  return hipGetLastError();
}

hipError_t launch_scdm_preselect(const double* phi, int n, int k, const double* L, double* rho,
                                 double* g, double* part, double* means, int* cnt, int* off,
                                 int* points, int* count, hipStream_t s) {
  const int64_t npts = (int64_t)n * n * n;
  const unsigned blocks = (unsigned)((npts + 255) / 256);
  hipLaunchKernelGGL(k_density, dim3(blocks), dim3(256), 0, s, phi, k, npts, rho);
  const double h0 = L[0] / n, h1 = L[1] / n, h2 = L[2] / n;
  hipLaunchKernelGGL(k_grad_norm, dim3(blocks), dim3(256), 0, s, rho, n, 2.0 * h0, 2.0 * h1,
                     2.0 * h2, g);
  hipLaunchKernelGGL(k_sum2_partial, dim3(kScdmSumBlocks), dim3(256), 0, s, rho, g, npts, part);
  hipLaunchKernelGGL(k_sum2_final, dim3(1), dim3(256), 0, s, part, kScdmSumBlocks, npts, means);
  const int64_t nb = scdm_sel_blocks(npts);
  hipLaunchKernelGGL(k_sel_count, dim3((unsigned)nb), dim3(256), 0, s, rho, g, means, npts, cnt);
  hipLaunchKernelGGL(k_sel_scan, dim3(1), dim3(1024), 0, s, cnt, (int)nb, off, count);
  hipLaunchKernelGGL(k_sel_write, dim3((unsigned)nb), dim3(256), 0, s, rho, g, means, npts, off,
                     points);
  return hipGetLastError();
}

int scdm_qr_groups(int m) {
  // a wave per eight columns, up to two workgroups per CU (a candidate per
  // thread of a workgroup)
  return std::max(1, std::min((m + 63) / 64, kQrThreads));
}

template <int G, int Q>
static void qr_step(int s, int m, int k, double* A, int* pos, int* perm, const QrCand* cand,
                    QrCand* next, const int* points, int* pivots, int* info, hipStream_t st) {
  hipLaunchKernelGGL((k_qr_step<G, Q>), dim3(scdm_qr_groups(m)), dim3(kQrThreads), 0, st, s, m, k,
                     scdm_qr_pitch(k), A, pos, perm, cand, next, points, pivots, info);
}

hipError_t launch_scdm_qr(const double* phi, const int* points, int m, int k, int64_t npts,
                          double* A, int* pos, int* perm, void* cand, int* pivots, int* info,
                          hipStream_t s) {
  const int groups = scdm_qr_groups(m);
  QrCand* c[2] = {static_cast<QrCand*>(cand), static_cast<QrCand*>(cand) + groups};
  hipLaunchKernelGGL(k_qr_gather, dim3(groups), dim3(kQrThreads), 0, s, phi, points, m, k,
                     scdm_qr_pitch(k), npts, A, pos, perm, c[0]);
  for (int st = 0; st < k; ++st) {
    const QrCand* in = c[st & 1];
    QrCand* out = c[(st + 1) & 1];
    // up to 16 values of a column per lane: the registers of two columns (the
    // Householder vector's and the wave's own) leave four waves per SIMD
    if (k <= 32) qr_step<8, 2>(st, m, k, A, pos, perm, in, out, points, pivots, info, s);
    else if (k <= 64) qr_step<8, 4>(st, m, k, A, pos, perm, in, out, points, pivots, info, s);
    else if (k <= 128) qr_step<8, 8>(st, m, k, A, pos, perm, in, out, points, pivots, info, s);
    else if (k <= 256) qr_step<16, 8>(st, m, k, A, pos, perm, in, out, points, pivots, info, s);
    else if (k <= 512) qr_step<32, 8>(st, m, k, A, pos, perm, in, out, points, pivots, info, s);
    else return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Iterations issued as launches; the rest, up to max_iter, in k_ns_tail.  From
// Y = A / ||A||_F the smallest singular value grows by 1.5 per iteration until
// it nears 1, so 40 iterations reach a condition number of about 1e5.  An
// iteration that finds all done costs 3 us, one of the tail's 0.1 ms at 128
// orbitals, 0.45 at 192 and 7 at 512, where a launched one takes 10 to 50 us.
// Past 128 orbitals all are therefore launched (a whole localisation with 256:
// 3.58 -> 3.76 ms where 20 iterations do, 47.1 -> 4.6 at a condition number of
// 1e12, 12.7 -> 4.2 at 1e6; with 512 96.5 -> 12.8); from 65 on 44 of them (128
// at 1e12 7.4 -> 6.9 ms, at 1e6 2.9 -> 2.4, where 20 do 1.647 -> 1.659).
static int ns_launched(int k, int max_iter) {
  return std::min(k > 128 ? max_iter : k > 64 ? 44 : 40, max_iter);
}

hipError_t launch_scdm_polar(const double* phi, const int* pivots, int k, int64_t npts, double* Y,
                             double* G, double* Z, double* sq, double* err, int* state, int* info,
                             int max_iter, hipStream_t s) {
  const int T = (k + 15) / 16;
  hipLaunchKernelGGL(k_ns_gather, dim3(k), dim3(256), 0, s, phi, pivots, k, npts, Y, sq);
  hipLaunchKernelGGL(k_ns_init, dim3(k), dim3(256), 0, s, k, sq, Y, max_iter, err, state);
  const int launched = ns_launched(k, max_iter);
  for (int it = 0; it < launched; ++it) {
    double* in = (it & 1) ? Z : Y;
    double* out = (it & 1) ? Y : Z;
    hipLaunchKernelGGL(k_ns_gram, dim3(T * (T + 1) / 2), dim3(256), 0, s, in, G, k, it, err, state);
    hipLaunchKernelGGL(k_ns_step, dim3(T * T), dim3(256), 0, s, in, G, out, k, it, err, state);
  }
  if (launched < max_iter)
    hipLaunchKernelGGL(k_ns_tail, dim3(1), dim3(1024), 0, s, Y, Z, G, k, launched, max_iter, err,
                       state);
  hipLaunchKernelGGL(k_ns_finish, dim3(k), dim3(256), 0, s, state, max_iter, k, Y, Z, info);
  return hipGetLastError();
}

}  // namespace acex
