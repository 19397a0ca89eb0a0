// df.hip -- the density-fitting solve of Eq. M4 on gfx950:
//     sum_Q J^{k12}_PQ d^{k1k2}_{Q mu nu} = V^{k1k2}_{P mu nu}   for every k-pair,
// with J^k Hermitian positive definite (a Coulomb metric with q = 0 removed).
// Per k of the mesh, all k in the same launches, in blocks of 64:
//   1. Cholesky factor J = L L^H, right-looking: the diagonal block and its
//      inverse by one workgroup in LDS, the panel below it by substitution, the
//      trailing blocks as 64 x 64 x 64 complex products on the FP64 matrix cores;
//   2. W = L^{-1} block row by block row, a strip of 16 columns per workgroup.
// Bound by the chain of n / 64 steps, not by operations: 420 functions on a
// 2x2x2 mesh took 26.6 ms with one workgroup per k column by column and one
// thread per column of W, and take 1.2 ms in this form (0.8 ms of it the seven
// diagonal blocks, whose 64 dependent columns are the chain).
// Then for every k-pair Y = W V and d = W^H Y (the forward and backward
// substitutions of L L^H d = V as products with the substituted inverse, which
// keeps the error of two triangular solves) as complex FP64 matrix products on
// the matrix cores (v_mfma_f64_16x16x4f64), V row-major [naux][ncol] with the
// columns (mu, nu) contiguous.  A pivot below 1e-12 of its diagonal entry of
// J^k (J numerically singular: linearly dependent aux functions) sets a flag;
// the host reports it.
#include <hip/hip_runtime.h>

#include "kernels.h"

namespace rsgdf {

typedef double df_d4 __attribute__((ext_vector_type(4)));
constexpr int FB = 64;         // block of the factorisation
constexpr int FBP = FB + 1;    // LDS row stride (doubles): rows start in distinct banks

// L = lower triangle of J (strict upper zero), W = 0, bad = 0
__global__ __launch_bounds__(256) void df_init_kernel(const double2 *__restrict__ J, double2 *__restrict__ L,
                                                      double2 *__restrict__ W, int n, int64_t total,
                                                      int *__restrict__ bad, int nk) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < nk) bad[i] = 0;
  if (i >= total) return;
  const int64_t e = i % ((int64_t)n * n);
  const int r = (int)(e / n), c = (int)(e % n);
  double2 v = make_double2(0.0, 0.0);
  if (c <= r) v = J[i];
  if (c == r) v.y = 0.0;
  L[i] = v;
  W[i] = make_double2(0.0, 0.0);
}

// Diagonal block p of every k: Cholesky factor and its inverse in LDS (one
// workgroup per k).  A pivot below 1e-12 of its diagonal entry of J marks k.
// The imaginary part of a diagonal entry, zero by definition, holds the sum of
// |L_jc|^2 of the columns done so far, here and in the trailing update: the entry
// itself is rounded once, when the sum is taken off it (taken off column by
// column, the solve's error was 1.3 to 1.7 times as large for well-conditioned
// metrics of 33 to 160 functions).
__global__ __launch_bounds__(256) void df_diag_kernel(const double *__restrict__ J, double *__restrict__ L,
                                                      double *__restrict__ W, int n, int p, int *__restrict__ bad) {
  __shared__ double ar[FB][FBP], ai[FB][FBP], wr[FB][FBP], wi[FB][FBP], piv;
  const int k = blockIdx.x, tid = threadIdx.x;
  const int p0 = p * FB, nb = min(FB, n - p0);
  double *Lk = L + 2 * (size_t)k * n * n, *Wk = W + 2 * (size_t)k * n * n;
  const double *Jk = J + 2 * (size_t)k * n * n;
  for (int e = tid; e < FB * FB; e += 256) {
    const int r = e / FB, c = e % FB;
    const bool in = r < nb && c <= r;
    const size_t o = 2 * ((size_t)(p0 + r) * n + p0 + c);
    ar[r][c] = in ? Lk[o] : 0.0;
    ai[r][c] = in ? Lk[o + 1] : 0.0;
    wr[r][c] = wi[r][c] = 0.0;
  }
  int failed = 0;
  const int tx = tid & 15, ty = tid >> 4;
  // thread i < nb holds row i's sum of |L_ic|^2 with its rounding error
  double sum = 0.0, lo = 0.0;
  __syncthreads();
  if (tid < nb) sum = ai[tid][tid];
  if (tid == 0) piv = ar[0][0] - sum;
  for (int j = 0; j < nb; ++j) {
    __syncthreads();
    const double d = piv;
    if (tid == 0 && !(d > 1e-12 * Jk[2 * ((size_t)(p0 + j) * n + p0 + j)])) failed = 1;
    const double s = (d > 0.0) ? sqrt(d) : 1.0, inv = 1.0 / s;
    __syncthreads();
    if (tid > j && tid < nb) {
      const double xr = ar[tid][j] * inv, xi = ai[tid][j] * inv;
      ar[tid][j] = xr;
      ai[tid][j] = xi;
      const double x2 = xr * xr + xi * xi, t = sum + x2, b = t - sum;
      lo += (sum - (t - b)) + (x2 - b);
      sum = t;
      if (tid == j + 1) piv = ar[tid][tid] - (sum + lo);
    }
    if (tid == j) {
      ar[j][j] = s;
      ai[j][j] = 0.0;
    }
    __syncthreads();
    for (int i = j + 1 + ty; i < nb; i += 16)
      for (int c = j + 1 + tx; c < i; c += 16) {
        const double xr = ar[i][j], xi = ai[i][j], yr = ar[c][j], yi = ai[c][j];
        ar[i][c] -= xr * yr + xi * yi;  // L_ij conj(L_cj)
        ai[i][c] -= xi * yr - xr * yi;
      }
  }
  if (tid == 0 && failed) bad[k] = 1;
  // rows of the inverse: four threads per column share the sum over c
  const int j = tid >> 2, part = tid & 3;
  for (int i = 0; i < nb; ++i) {
    __syncthreads();
    double sr = 0.0, si = 0.0;
    for (int c = j + part; c < i; c += 4) {
      const double xr = ar[i][c], xi = ai[i][c], yr = wr[c][j], yi = wi[c][j];
      sr += xr * yr - xi * yi;
      si += xr * yi + xi * yr;
    }
#pragma unroll
    for (int o = 1; o < 4; o <<= 1) {
      sr += __shfl_xor(sr, o, 64);
      si += __shfl_xor(si, o, 64);
    }
    const double inv = 1.0 / ar[i][i];
    if (part == 0 && j <= i) {
      wr[i][j] = (j == i) ? inv : -sr * inv;
      wi[i][j] = (j == i) ? 0.0 : -si * inv;
    }
  }
  __syncthreads();
  for (int e = tid; e < FB * FB; e += 256) {
    const int r = e / FB, c = e % FB;
    if (r >= nb || c > r) continue;
    const size_t o = 2 * ((size_t)(p0 + r) * n + p0 + c);
    Lk[o] = ar[r][c];
    Lk[o + 1] = ai[r][c];
    Wk[o] = wr[r][c];
    Wk[o + 1] = wi[r][c];
  }
}

// v of lane src (a constant) of the four
__device__ __forceinline__ double quad_bcast(double v, int src) {
  int2 w = *reinterpret_cast<int2 *>(&v);
  auto at = [src](int x) {
    switch (src) {
      case 0: return __builtin_amdgcn_mov_dpp(x, 0x00, 0xf, 0xf, true);
      case 1: return __builtin_amdgcn_mov_dpp(x, 0x55, 0xf, 0xf, true);
      case 2: return __builtin_amdgcn_mov_dpp(x, 0xaa, 0xf, 0xf, true);
      default: return __builtin_amdgcn_mov_dpp(x, 0xff, 0xf, 0xf, true);
    }
  };
  w.x = at(w.x);
  w.y = at(w.y);
  return *reinterpret_cast<double *>(&w);
}

// Blocks below the diagonal block p: the rows of L_ip L_pp^H = A_ip by forward
// substitution.  (A product with the explicit inverse W_pp is not as accurate: it
// alone added a third to the solve's error at 100 to 160 functions.)  Grid (nk,
// row block); four lanes share a row, lane `part` holding its columns part, part +
// 4, ...: a chain of 64 scalings, each passed on within the quad.
__global__ __launch_bounds__(256) void df_panel_kernel(double *__restrict__ L, int n, int p) {
  __shared__ double lr[FB][FBP], li[FB][FBP], linv[FB];
  const int tid = threadIdx.x, p0 = p * FB, row = (p + 1 + (int)blockIdx.y) * FB + (tid >> 2), part = tid & 3;
  double *Lk = L + 2 * (size_t)blockIdx.x * n * n;
  for (int e = tid; e < FB * FB; e += 256) {  // block p is a whole one: a row block follows it
    const double2 v = *reinterpret_cast<const double2 *>(Lk + 2 * ((size_t)(p0 + e / FB) * n + p0 + e % FB));
    lr[e / FB][e % FB] = v.x;
    li[e / FB][e % FB] = v.y;
    if (e / FB == e % FB) linv[e / FB] = 1.0 / v.x;
  }
  double2 *x = reinterpret_cast<double2 *>(Lk) + (size_t)min(row, n - 1) * n + p0 + part;
  double xr[FB / 4], xi[FB / 4];
#pragma unroll
  for (int c = 0; c < FB / 4; ++c) {
    const double2 v = x[4 * c];
    xr[c] = v.x;
    xi[c] = v.y;
  }
  __syncthreads();
#pragma unroll
  for (int jb = 0; jb < FB / 4; ++jb)
#pragma unroll
    for (int jp = 0; jp < 4; ++jp) {
      const int j = 4 * jb + jp;
      const double inv = linv[j], yr = quad_bcast(xr[jb], jp) * inv, yi = quad_bcast(xi[jb], jp) * inv;
      if (part == jp) {
        xr[jb] = yr;
        xi[jb] = yi;
      }
#pragma unroll
      for (int c = 0; c < FB / 4; ++c) {
        if (c < jb) continue;
        const bool on = c > jb || part > jp;
        const double zr = lr[4 * c + part][j], zi = li[4 * c + part][j];
        const double re = yr * zr + yi * zi, im = yi * zr - yr * zi;  // y conj(L_qj)
        xr[c] -= on ? re : 0.0;
        xi[c] -= on ? im : 0.0;
      }
    }
  if (row >= n) return;
#pragma unroll
  for (int c = 0; c < FB / 4; ++c) x[4 * c] = make_double2(xr[c], xi[c]);
}

// Trailing blocks i >= k > p: A_ik -= L_ip L_kp^H.  Grid (nk, row block, column
// block); every block is read and written by one workgroup.  Wave w holds rows
// [16 w, 16 w + 16), its four 16-column tiles in cre/cim (result D[lg + 4 v][li]).
// The products of kUpdCols columns are summed from zero on the matrix cores, then
// taken off the block: the block's own rounding comes once per 8 columns, and the
// sums stay small beside it.  (Residual |L L^H - J| against a factorisation column
// by column, at 130 and 300 functions: 1.6 and 1.2 with all 64 columns in one sum,
// 1.3 and 1.3 with every product added to the block, 0.95 and 0.8 with 8.)
constexpr int kUpdCols = 8;

__global__ __launch_bounds__(256) void df_update_kernel(double *__restrict__ L, int n, int p) {
  __shared__ double xr[FB][FBP], xi[FB][FBP], yr[FB][FBP], yi[FB][FBP];
  const int tid = threadIdx.x, p0 = p * FB;
  const int ib = p + 1 + blockIdx.y, kb = p + 1 + (int)blockIdx.z;
  if (kb > ib) return;
  double *Lk = L + 2 * (size_t)blockIdx.x * n * n;
  for (int e = tid; e < FB * FB; e += 256) {
    const int r = e / FB, c = e % FB;
    const int ri = ib * FB + r, rk = kb * FB + r;
    const double2 x = ri < n ? *reinterpret_cast<const double2 *>(Lk + 2 * ((size_t)ri * n + p0 + c))
                             : make_double2(0.0, 0.0);
    const double2 y = rk < n ? *reinterpret_cast<const double2 *>(Lk + 2 * ((size_t)rk * n + p0 + c))
                             : make_double2(0.0, 0.0);
    xr[r][c] = x.x;
    xi[r][c] = x.y;
    yr[r][c] = y.x;
    yi[r][c] = y.y;
  }
  const int lane = tid & 63, wave = tid >> 6, li = lane & 15, lg = lane >> 4;
  df_d4 cre[4], cim[4];  // the block, less what has been summed
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = ib * FB + 16 * wave + lg + 4 * v, q = kb * FB + 16 * c + li;
      const double2 old = (r < n && q <= r) ? *reinterpret_cast<const double2 *>(Lk + 2 * ((size_t)r * n + q))
                                            : make_double2(0.0, 0.0);
      cre[c][v] = old.x;
      cim[c][v] = old.y;
    }
  __syncthreads();
#pragma unroll 2
  for (int t0 = 0; t0 < FB; t0 += kUpdCols) {
    df_d4 sre[4], sim[4];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int v = 0; v < 4; ++v) sre[c][v] = sim[c][v] = 0.0;
#pragma unroll
    for (int ks = 0; ks < kUpdCols / 4; ++ks) {
      const int t = t0 + 4 * ks + lg;
      const double a_r = xr[16 * wave + li][t], a_i = xi[16 * wave + li][t];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const double b_r = yr[16 * c + li][t], b_i = yi[16 * c + li][t];
        // (a_r + i a_i)(b_r - i b_i)
        sre[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a_r, b_r, sre[c], 0, 0, 0);
        sre[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a_i, b_i, sre[c], 0, 0, 0);
        sim[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a_i, b_r, sim[c], 0, 0, 0);
        sim[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a_r, b_i, sim[c], 0, 0, 0);
      }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const bool diag = ib * FB + 16 * wave + lg + 4 * v == kb * FB + 16 * c + li;
        cre[c][v] -= diag ? 0.0 : sre[c][v];
        cim[c][v] -= diag ? -sre[c][v] : sim[c][v];
      }
  }
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = ib * FB + 16 * wave + lg + 4 * v, q = kb * FB + 16 * c + li;
      if (r < n && q <= r)
        *reinterpret_cast<double2 *>(Lk + 2 * ((size_t)r * n + q)) = make_double2(cre[c][v], cim[c][v]);
    }
}

// W = L^{-1} below the diagonal blocks, a strip of 16 columns (of block j) per
// workgroup: W_i = -W_ii sum_{j <= k < i} L_ik W_k for i = j + 1, ...  The wave's
// operands come straight from memory (its 16 rows of L are its own, the strip's
// rows are 256 contiguous bytes); only the sum crosses LDS, from the result
// layout to the operand layout.
__global__ __launch_bounds__(256, 1) void df_inverse_kernel(const double *__restrict__ L, double *W, int n) {
  __shared__ double tr[FB][17], ti[FB][17];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, lg = lane >> 4;
  const int c0 = blockIdx.y * 16, jb = c0 / FB, nblk = (n + FB - 1) / FB;
  const double2 *Lk = reinterpret_cast<const double2 *>(L) + (size_t)blockIdx.x * n * n;
  double2 *Wk = reinterpret_cast<double2 *>(W) + (size_t)blockIdx.x * n * n;
  const int col = c0 + li;
  const double2 zero = make_double2(0.0, 0.0);
  for (int ib = jb + 1; ib < nblk; ++ib) {
    const int row = ib * FB + 16 * wave + li;
    df_d4 sr = {0.0, 0.0, 0.0, 0.0}, si = sr;
    for (int kb = jb; kb < ib; ++kb) {
      double2 a[FB / 4], b[FB / 4];
#pragma unroll
      for (int ks = 0; ks < FB / 4; ++ks) {
        const int t = kb * FB + 4 * ks + lg;  // kb < ib: inside the matrix
        a[ks] = row < n ? Lk[(size_t)row * n + t] : zero;
        b[ks] = col < n ? Wk[(size_t)t * n + col] : zero;
      }
#pragma unroll
      for (int ks = 0; ks < FB / 4; ++ks) {
        sr = __builtin_amdgcn_mfma_f64_16x16x4f64(a[ks].x, b[ks].x, sr, 0, 0, 0);
        sr = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[ks].y, b[ks].y, sr, 0, 0, 0);
        si = __builtin_amdgcn_mfma_f64_16x16x4f64(a[ks].x, b[ks].y, si, 0, 0, 0);
        si = __builtin_amdgcn_mfma_f64_16x16x4f64(a[ks].y, b[ks].x, si, 0, 0, 0);
      }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      tr[16 * wave + lg + 4 * v][li] = sr[v];
      ti[16 * wave + lg + 4 * v][li] = si[v];
    }
    __syncthreads();
    df_d4 dr = {0.0, 0.0, 0.0, 0.0}, di = dr;
#pragma unroll 4
    for (int ks = 0; ks < FB / 4; ++ks) {
      const int t = 4 * ks + lg, tc = ib * FB + t;
      const double2 a = (row < n && tc < n) ? Wk[(size_t)row * n + tc] : zero;
      const double b_r = tr[t][li], b_i = ti[t][li];
      dr = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.x, b_r, dr, 0, 0, 0);
      dr = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b_i, dr, 0, 0, 0);
      di = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.x, b_i, di, 0, 0, 0);
      di = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.y, b_r, di, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = ib * FB + 16 * wave + lg + 4 * v;
      if (r < n && col < n) Wk[(size_t)r * n + col] = make_double2(dr[v], di[v]);
    }
    __threadfence_block();
    __syncthreads();  // the strip's new rows are read by every wave in the next step
  }
}

hipError_t launch_df_factor(const double *J, double *L, double *W, int *bad, int nk, int n, hipStream_t stream) {
  if (nk == 0 || n == 0) return hipSuccess;
  const int64_t total = (int64_t)nk * n * n;
  const int64_t g = (total > nk ? total : nk) / 256 + 1;
  const int nblk = (n + FB - 1) / FB;
  if (g > 0x7fffffff || nblk > 65535) return hipErrorInvalidConfiguration;
  hipLaunchKernelGGL(df_init_kernel, dim3((unsigned)g), dim3(256), 0, stream, reinterpret_cast<const double2 *>(J),
                     reinterpret_cast<double2 *>(L), reinterpret_cast<double2 *>(W), n, total, bad, nk);
  for (int p = 0; p < nblk; ++p) {
    hipLaunchKernelGGL(df_diag_kernel, dim3((unsigned)nk), dim3(256), 0, stream, J, L, W, n, p, bad);
    const unsigned rest = (unsigned)(nblk - 1 - p);
    if (rest == 0) break;
    hipLaunchKernelGGL(df_panel_kernel, dim3((unsigned)nk, rest), dim3(256), 0, stream, L, n, p);
    hipLaunchKernelGGL(df_update_kernel, dim3((unsigned)nk, rest, rest), dim3(256), 0, stream, L, n, p);
  }
  if (nblk > 1)
    hipLaunchKernelGGL(df_inverse_kernel, dim3((unsigned)nk, (unsigned)((nblk - 1) * (FB / 16))), dim3(256), 0, stream,
                       L, W, n);
  return hipGetLastError();
}

// ---- Y = W V and d = W^H Y on the FP64 matrix cores -----------------------------
// C[t][m][n] = sum_q op(A)[cls[t]][m][q] B[t][q][n], complex, op(A) = A
// (CONJT = false) or A^H (CONJT = true, op(A)[m][q] = conj(A[q][m])); A
// [*][M][M] row-major, B and C [*][M][N] (n contiguous).  W is lower
// triangular: the q steps where op(A)'s tile is zero are skipped (q > m for W,
// q < m for W^H).  Workgroup tile 128 x 128, 8
// waves as 4 (rows of 32) x 2 (columns of 64); 16 q per step staged in LDS,
// the next step's loads in flight during the MFMAs.  Fragments (li = lane %
// 16, lg = lane / 16): A[li][lg], B[lg][li]; result D[lg + 4 v][li].
constexpr int DG_BM = 128, DG_BN = 128, DG_BK = 16, DG_NT = 512;

template <bool CONJT>
__global__ __launch_bounds__(DG_NT) void df_gemm_kernel(const double *__restrict__ A, const int32_t *__restrict__ cls,
                                                        const double *__restrict__ B, double *__restrict__ C, int M,
                                                        int64_t N) {
  __shared__ double sar[DG_BM][DG_BK + 1], sai[DG_BM][DG_BK + 1];
  __shared__ double sbr[DG_BK][DG_BN + 1], sbi[DG_BK][DG_BN + 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lg = lane >> 4;
  const int wm = wave >> 1, wn = wave & 1;
  const int t = blockIdx.z;
  const int M0 = blockIdx.y * DG_BM;
  const int64_t N0 = (int64_t)blockIdx.x * DG_BN;
  const double *At = A + 2 * (size_t)cls[t] * M * M;
  const double *Bt = B + 2 * (size_t)t * M * N;
  double *Ct = C + 2 * (size_t)t * M * N;
  // staging: A tile 128 x 16 (thread: row tid/4, 4 q), B tile 16 x 128 (thread: q tid/32, 4 columns)
  const int ar0 = tid >> 2, aq = (tid & 3) * 4;
  const int bq = tid >> 5, bc = (tid & 31) * 4;
  double ga[8], gb[8];
  auto gload = [&](int k0) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int m = M0 + ar0, k = k0 + aq + j;
      const bool ok = m < M && k < M;
      const size_t o = CONJT ? (size_t)k * M + m : (size_t)m * M + k;
      ga[2 * j] = ok ? At[2 * o] : 0.0;
      ga[2 * j + 1] = ok ? (CONJT ? -At[2 * o + 1] : At[2 * o + 1]) : 0.0;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int k = k0 + bq;
      const int64_t col = N0 + bc + j;
      const bool ok = k < M && col < N;
      gb[2 * j] = ok ? Bt[2 * ((size_t)k * N + col)] : 0.0;
      gb[2 * j + 1] = ok ? Bt[2 * ((size_t)k * N + col) + 1] : 0.0;
    }
  };
  df_d4 cre[2][4], cim[2][4];
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int v = 0; v < 4; ++v) cre[r][c][v] = cim[r][c][v] = 0.0;
  // non-zero q range of the row tile: W (lower) has q <= m, W^H has q >= m
  const int kbeg = CONJT ? (M0 / DG_BK) * DG_BK : 0;
  const int kend = CONJT ? M : (M0 + DG_BM < M ? M0 + DG_BM : M);
  gload(kbeg);
  for (int k0 = kbeg; k0 < kend; k0 += DG_BK) {
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      sar[ar0][aq + j] = ga[2 * j];
      sai[ar0][aq + j] = ga[2 * j + 1];
      sbr[bq][bc + j] = gb[2 * j];
      sbi[bq][bc + j] = gb[2 * j + 1];
    }
    __syncthreads();
    if (k0 + DG_BK < kend) gload(k0 + DG_BK);
#pragma unroll
    for (int ks = 0; ks < DG_BK / 4; ++ks) {
      const int k = ks * 4 + lg;
      double a_r[2], a_i[2], b_r[4], b_i[4];
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        a_r[r] = sar[wm * 32 + r * 16 + li][k];
        a_i[r] = sai[wm * 32 + r * 16 + li][k];
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        b_r[c] = sbr[k][wn * 64 + c * 16 + li];
        b_i[c] = sbi[k][wn * 64 + c * 16 + li];
      }
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          cre[r][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a_r[r], b_r[c], cre[r][c], 0, 0, 0);
          cre[r][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a_i[r], b_i[c], cre[r][c], 0, 0, 0);
          cim[r][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a_r[r], b_i[c], cim[r][c], 0, 0, 0);
          cim[r][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a_i[r], b_r[c], cim[r][c], 0, 0, 0);
        }
    }
  }
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int m = M0 + wm * 32 + r * 16 + lg + 4 * v;
        const int64_t col = N0 + wn * 64 + c * 16 + li;
        if (m < M && col < N) {
          Ct[2 * ((size_t)m * N + col)] = cre[r][c][v];
          Ct[2 * ((size_t)m * N + col) + 1] = cim[r][c][v];
        }
      }
}

hipError_t launch_df_gemm(bool conjt, const double *W, const int32_t *cls, const double *V, double *D, int naux,
                          int64_t ncol, int nkp, hipStream_t stream) {
  if (nkp == 0 || naux == 0 || ncol == 0) return hipSuccess;
  const int64_t gx = (ncol + DG_BN - 1) / DG_BN;
  if (gx > 0x7fffffff || nkp > 65535) return hipErrorInvalidConfiguration;
  const dim3 grid((unsigned)gx, (unsigned)((naux + DG_BM - 1) / DG_BM), (unsigned)nkp);
  if (conjt) hipLaunchKernelGGL(df_gemm_kernel<true>, grid, dim3(DG_NT), 0, stream, W, cls, V, D, naux, ncol);
  else hipLaunchKernelGGL(df_gemm_kernel<false>, grid, dim3(DG_NT), 0, stream, W, cls, V, D, naux, ncol);
  return hipGetLastError();
}

}  // namespace rsgdf
