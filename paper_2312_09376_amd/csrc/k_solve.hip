// Kernels around the solve: the residual B - A X with the row sums of |A|
// for ||A||_inf fused into the same pass over A, the backward error of
// Eq. 7, the column updates of iterative refinement (Sec. 5) and the
// outer product of the adjoint.
//
// These are HBM-bound (one read of the matrix, a few columns of output). The
// products with the matrix run on the matrix cores (k_rows_product), so that
// up to 16 right-hand sides cost about what one does; the GEMM is kept for
// many right-hand sides.
#include "internal.h"

namespace rbt {

namespace {

constexpr int kRows = 256;       // rows per workgroup
constexpr int64_t kChunk = 256;  // columns per split-K chunk of the residual

__device__ __forceinline__ double nanmax(double a, double b) {
  // NaN-propagating maximum: a NaN residual must never look converged
  return (b > a || b != b) ? b : a;
}

// Block-wide NaN-propagating max of one value per thread (kRows threads).
__device__ double block_nanmax(double v, double *sh) {
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int s = kRows / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) sh[threadIdx.x] = nanmax(sh[threadIdx.x], sh[threadIdx.x + s]);
    __syncthreads();
  }
  const double r = sh[0];
  __syncthreads();
  return r;
}

// O = G - op(A) X (G null: op(A) X) for op(A) = A or A^T (n x n) on the FP64
// matrix cores, in one pass over A. A workgroup forms 16 RT rows and 16 CT
// right-hand sides; its eight wavefronts take every eighth run of 32 columns
// of op(A), the next run's loads in flight, and their sums are added through LDS
// in a fixed order. Also per workgroup, for up to 16 right-hand sides:
// blockstat[blk (3 N + 1) + 3 c + 0..2] = max |O|, |X|, |G| over its rows, and
// (ABS) entry 3 N of it, or blockstat[blk] for more right-hand sides, the
// maximum over its rows of the row sums of |op(A)|.
// Bound by reading A once for up to 16 right-hand sides (n = 8191: 110 to 114 us,
// 4.8 TB/s, a copy's rate being 5.3) and by the matrix cores and the readings of
// X for more. With 8 right-hand sides at n = 8191 the product as partial sums over
// chunks of 256 columns and their sum by a second kernel, one workgroup per 256
// rows, took 111 and 95 us, the transposed one from LDS 357; with 64 at n = 5003 a
// GEMM of 79 tiles of 64 x 64 took 392 us, this 216.
constexpr int kRunK = 32;    // columns of op(A) per run of a wavefront
constexpr int kWaves = 8;
typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));
template <bool TRANS, int RT, int CT, bool ABS>
__global__ void __launch_bounds__(64 * kWaves)
    k_rows_product(int64_t n, int nrhs, const double *__restrict__ A, int64_t lda,
                   const double *__restrict__ X, int64_t ldx, const double *__restrict__ G,
                   int64_t ldg, double *__restrict__ O, int64_t ldo,
                   double *__restrict__ blockstat, const int32_t *gate) {
  if (gated(gate)) return;
  __shared__ double red[kWaves][RT][CT][4][64];
  __shared__ double absred[ABS ? kWaves : 1][RT][64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lk = lane >> 4;
  const int64_t m0 = int64_t(blockIdx.x) * (16 * RT);
  const int c0 = int(blockIdx.y) * (16 * CT);
  // operand rows and right-hand sides beyond the last repeat it (not stored)
  const double *ap[RT], *xp[CT];
#pragma unroll
  for (int i = 0; i < RT; ++i) {
    const int64_t m = m0 + 16 * i + l16 < n ? m0 + 16 * i + l16 : n - 1;
    ap[i] = TRANS ? A + m * lda : A + m;
  }
#pragma unroll
  for (int t = 0; t < CT; ++t) {
    const int c = c0 + 16 * t + l16 < nrhs ? c0 + 16 * t + l16 : nrhs - 1;
    xp[t] = X + int64_t(c) * ldx;
  }
  // the lane's columns of a run: k0 + 8 q + 2 lk + {0, 1}, q = 0..3
  double a[RT][8], x[CT][8], an[RT][8], xn[CT][8];
  auto load = [&](int64_t k0, double (&av)[RT][8], double (&xv)[CT][8]) {
    if (k0 + kRunK <= n) {
      const int64_t k = k0 + 2 * lk;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int i = 0; i < RT; ++i) {
          if constexpr (TRANS) {
            const d2u v = *reinterpret_cast<const d2u *>(ap[i] + k + 8 * q);
            av[i][2 * q] = v[0];
            av[i][2 * q + 1] = v[1];
          } else {
            av[i][2 * q] = ap[i][(k + 8 * q) * lda];
            av[i][2 * q + 1] = ap[i][(k + 8 * q + 1) * lda];
          }
        }
#pragma unroll
        for (int t = 0; t < CT; ++t) {
          const d2u v = *reinterpret_cast<const d2u *>(xp[t] + k + 8 * q);
          xv[t][2 * q] = v[0];
          xv[t][2 * q + 1] = v[1];
        }
      }
    } else {  // the last, partial run: clamped loads, zero beyond
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int64_t k = k0 + 8 * (e >> 1) + 2 * lk + (e & 1);
        const int64_t kc = k < n ? k : n - 1;
#pragma unroll
        for (int i = 0; i < RT; ++i) {
          const double v = TRANS ? ap[i][kc] : ap[i][kc * lda];
          av[i][e] = k < n ? v : 0.0;
        }
#pragma unroll
        for (int t = 0; t < CT; ++t) {
          const double v = xp[t][kc];
          xv[t][e] = k < n ? v : 0.0;
        }
      }
    }
  };
  d4 acc[RT][CT];
  double as[RT];
#pragma unroll
  for (int i = 0; i < RT; ++i) {
    as[i] = 0.0;
#pragma unroll
    for (int t = 0; t < CT; ++t) acc[i][t] = d4{0.0, 0.0, 0.0, 0.0};
  }
  int64_t k0 = int64_t(wave) * kRunK;
  if (k0 < n) load(k0, a, x);
  while (k0 < n) {
    const int64_t kn = k0 + kWaves * kRunK;
    if (kn < n) load(kn, an, xn);
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int i = 0; i < RT; ++i) {
        if constexpr (ABS) as[i] += fabs(a[i][e]);
#pragma unroll
        for (int t = 0; t < CT; ++t)
          acc[i][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i][e], x[t][e], acc[i][t], 0, 0, 0);
      }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
#pragma unroll
      for (int i = 0; i < RT; ++i) a[i][e] = an[i][e];
#pragma unroll
      for (int t = 0; t < CT; ++t) x[t][e] = xn[t][e];
    }
    k0 = kn;
  }
  // acc[i][t][v]: row 16 i + lk + 4 v, right-hand side 16 t + l16
#pragma unroll
  for (int i = 0; i < RT; ++i) {
#pragma unroll
    for (int t = 0; t < CT; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) red[wave][i][t][v][lane] = acc[i][t][v];
    if constexpr (ABS) absred[wave][i][lane] = as[i];
  }
  __syncthreads();
  constexpr int ROWS = 16 * RT;  // rows of a right-hand side stand in consecutive lanes
  const bool stats = nrhs <= kSkinnyMax;
  double *bs = blockstat + int64_t(blockIdx.x) * (stats ? 3 * nrhs + 1 : 1);
  for (int e = tid; e < ROWS * 16 * CT; e += 64 * kWaves) {
    const int r = e % ROWS, c = e / ROWS, i = r >> 4, t = c >> 4;
    const int src = (r & 3) * 16 + (c & 15), v = (r & 15) >> 2;
    double sum = 0.0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) sum += red[w][i][t][v][src];
    const int64_t m = m0 + r;
    const int col = c0 + c;
    double o = 0.0, xv = 0.0, g = 0.0;
    if (m < n && col < nrhs) {
      if (G != nullptr) {
        g = G[m + int64_t(col) * ldg];
        o = g - sum;
        xv = X[m + int64_t(col) * ldx];
      } else {
        o = sum;
      }
      O[m + int64_t(col) * ldo] = o;
    }
    if (stats && G != nullptr) {
      o = fabs(o);
      xv = fabs(xv);
      g = fabs(g);
#pragma unroll
      for (int d = 1; d < ROWS; d <<= 1) {
        o = nanmax(o, __shfl_xor(o, d));
        xv = nanmax(xv, __shfl_xor(xv, d));
        g = nanmax(g, __shfl_xor(g, d));
      }
      if (r == 0 && col < nrhs) {
        bs[3 * col] = o;
        bs[3 * col + 1] = xv;
        bs[3 * col + 2] = g;
      }
    }
  }
  if constexpr (ABS) {
    if (blockIdx.y == 0 && wave == 0) {
      double sum = 0.0;
      if (lane < ROWS && m0 + lane < n)
        for (int w = 0; w < kWaves; ++w)
          for (int h = 0; h < 4; ++h) sum += absred[w][lane >> 4][16 * h + (lane & 15)];
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) sum = nanmax(sum, __shfl_xor(sum, d));
      if (lane == 0) bs[stats ? 3 * nrhs : 0] = sum;
    }
  }
}

// Final reduction over the workgroups of k_rows_product, N <= 16 right-hand
// sides: anorm (ABS) and the backward error of Eq. 7. A wavefront takes every
// fourth right-hand side.
template <bool ABS>
__global__ void __launch_bounds__(kRows) k_berr_rows(int64_t nblk, int N,
                                                     const double *__restrict__ blockstat,
                                                     double *__restrict__ anorm,
                                                     double *__restrict__ berr, BerrHost host,
                                                     const int32_t *gate) {
  if (gated(gate)) return;
  __shared__ double sh[kRows / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int stride = 3 * N + 1;
  auto column = [&](int e) {  // maximum of entry e over the blocks, in every lane
    double v = 0.0;
    for (int64_t b = lane; b < nblk; b += 64) v = nanmax(v, blockstat[b * stride + e]);
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) v = nanmax(v, __shfl_xor(v, d));
    return v;
  };
  double an;
  if (ABS) {
    an = column(3 * N);
    if (threadIdx.x == 0) anorm[0] = an;
  } else {
    an = anorm[0];
  }
  double be = 0.0;
  for (int c = wave; c < N; c += kRows / 64) {
    const double r = column(3 * c), x = column(3 * c + 1), g = column(3 * c + 2);
    be = nanmax(be, r / (an * x + g));
  }
  if (lane == 0) sh[wave] = be;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kRows / 64; ++w) be = nanmax(be, sh[w]);
    berr[0] = be;
    host.store(be);
  }
}

// ---- wide right-hand sides (N > 16): GEMM residual, separate norms ----

// partial[c * n + i] = sum_{j in chunk c} |A[i, j]|
__global__ void __launch_bounds__(kRows) k_rowabs_partial(int64_t n, const double *__restrict__ A,
                                                         int64_t lda,
                                                         double *__restrict__ partial) {
  const int64_t i = int64_t(blockIdx.x) * kRows + threadIdx.x;
  if (i >= n) return;
  const int64_t j0 = int64_t(blockIdx.y) * kChunk;
  const int64_t j1 = j0 + kChunk < n ? j0 + kChunk : n;
  double s0 = 0.0, s1 = 0.0;
  int64_t j = j0;
  for (; j + 2 <= j1; j += 2) {
    s0 += fabs(A[i + j * lda]);
    s1 += fabs(A[i + (j + 1) * lda]);
  }
  for (; j < j1; ++j) s0 += fabs(A[i + j * lda]);
  partial[int64_t(blockIdx.y) * n + i] = s0 + s1;
}

// blockstat[blk] = max over the block's rows of sum_c partial
__global__ void __launch_bounds__(kRows) k_rowabs_reduce(int64_t n, int64_t chunks,
                                                        const double *__restrict__ partial,
                                                        double *__restrict__ blockstat) {
  __shared__ double sh[kRows];
  const int64_t i = int64_t(blockIdx.x) * kRows + threadIdx.x;
  double s = 0.0;
  if (i < n)
    for (int64_t c = 0; c < chunks; ++c) s += partial[c * n + i];
  const double m = block_nanmax(s, sh);
  if (threadIdx.x == 0) blockstat[blockIdx.x] = m;
}

__global__ void __launch_bounds__(kRows) k_max_reduce(int64_t nblk, const double *__restrict__ v,
                                                     double *__restrict__ out) {
  __shared__ double sh[kRows];
  double m = 0.0;
  for (int64_t b = threadIdx.x; b < nblk; b += kRows) m = nanmax(m, v[b]);
  m = block_nanmax(m, sh);
  if (threadIdx.x == 0) out[0] = m;
}

// colstat[3 c + {0,1,2}] = max |R[:, c]|, max |X[:, c]|, max |B[:, c]|
__global__ void __launch_bounds__(kRows) k_colmax(int64_t n, const double *__restrict__ R,
                                                 int64_t ldr, const double *__restrict__ X,
                                                 int64_t ldx, const double *__restrict__ B,
                                                 int64_t ldb, double *__restrict__ colstat) {
  __shared__ double sh[kRows];
  const int64_t c = blockIdx.x;
  double mr = 0.0, mx = 0.0, mb = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += kRows) {
    mr = nanmax(mr, fabs(R[i + c * ldr]));
    mx = nanmax(mx, fabs(X[i + c * ldx]));
    mb = nanmax(mb, fabs(B[i + c * ldb]));
  }
  mr = block_nanmax(mr, sh);
  mx = block_nanmax(mx, sh);
  mb = block_nanmax(mb, sh);
  if (threadIdx.x == 0) {
    colstat[3 * c] = mr;
    colstat[3 * c + 1] = mx;
    colstat[3 * c + 2] = mb;
  }
}

// berr = max_c colstat_r / (anorm * colstat_x + colstat_b)   (Eq. 7 per column)
__global__ void k_berr_final(int64_t nrhs, const double *__restrict__ colstat,
                             const double *__restrict__ anorm, double *__restrict__ berr,
                             BerrHost host) {
  if (threadIdx.x != 0) return;
  const double a = anorm[0];
  double m = 0.0;
  for (int64_t c = 0; c < nrhs; ++c)
    m = nanmax(m, colstat[3 * c] / (a * colstat[3 * c + 1] + colstat[3 * c + 2]));
  berr[0] = m;
  host.store(m);
}

__global__ void __launch_bounds__(kRows) k_axpy_cols(int64_t n, int64_t nrhs,
                                                    const double *__restrict__ D, int64_t ldd,
                                                    double *__restrict__ X, int64_t ldx,
                                                    const int32_t *gate) {
  if (gated(gate)) return;
  const int64_t i = int64_t(blockIdx.x) * kRows + threadIdx.x;
  if (i >= n) return;
  for (int64_t c = blockIdx.y; c < nrhs; c += gridDim.y) X[i + c * ldx] += D[i + c * ldd];
}

__global__ void __launch_bounds__(kRows) k_copy_cols(int64_t n, int64_t nrhs,
                                                    const double *__restrict__ S, int64_t lds,
                                                    double *__restrict__ D, int64_t ldd) {
  const int64_t i = int64_t(blockIdx.x) * kRows + threadIdx.x;
  if (i >= n) return;
  for (int64_t c = blockIdx.y; c < nrhs; c += gridDim.y) D[i + c * ldd] = S[i + c * lds];
}

// dA = -L X^T (n x n, rank nrhs), bound by the n^2 writes: a lane owns two
// consecutive rows of 16 columns, so every store instruction writes 1 KB of
// one column per wavefront (16-byte stores; the operands are only 8-byte
// aligned in general, which these stores accept), and the stores are
// non-temporal (dA is written once and not read back here, so it should not
// displace cached data). The X entries of a column chunk are the same for
// every lane (scalar loads). Each element sums l_k x_k in the order
// k = 0..nrhs-1.
typedef double d2s __attribute__((ext_vector_type(2), aligned(8)));
__global__ void __launch_bounds__(kRows) k_neg_outer(int64_t n, int64_t nrhs,
                                                    const double *__restrict__ Lm, int64_t ldl,
                                                    const double *__restrict__ X, int64_t ldx,
                                                    double *__restrict__ dA, int64_t ldda) {
  const int64_t i = (int64_t(blockIdx.x) * kRows + threadIdx.x) * 2;
  if (i >= n) return;
  const bool pair = i + 1 < n;
  for (int64_t j0 = int64_t(blockIdx.y) * 16; j0 < n; j0 += int64_t(gridDim.y) * 16) {
    double a0[16], a1[16];
#pragma unroll
    for (int jj = 0; jj < 16; ++jj) a0[jj] = a1[jj] = 0.0;
    for (int64_t k = 0; k < nrhs; ++k) {
      const double l0 = Lm[i + k * ldl];
      const double l1 = pair ? Lm[i + 1 + k * ldl] : 0.0;
#pragma unroll
      for (int jj = 0; jj < 16; ++jj) {
        const int64_t j = j0 + jj;
        const double x = (j < n) ? X[j + k * ldx] : 0.0;
        a0[jj] += l0 * x;
        a1[jj] += l1 * x;
      }
    }
#pragma unroll
    for (int jj = 0; jj < 16; ++jj) {
      const int64_t j = j0 + jj;
      if (j >= n) break;
      double *p = dA + i + j * ldda;
      if (pair) {
        const d2s v = {-a0[jj], -a1[jj]};
        __builtin_nontemporal_store(v, reinterpret_cast<d2s *>(p));
      } else {
        __builtin_nontemporal_store(-a0[jj], p);
      }
    }
  }
}

// out[i] = sum_k |A[k, i]| (column sums: ||A||_1 = ||A^T||_inf), one
// workgroup per column.
__global__ void __launch_bounds__(kRows) k_colabs(int64_t n, const double *__restrict__ A,
                                                 int64_t lda, double *__restrict__ out) {
  __shared__ double sh[kRows];
  const int64_t i = blockIdx.x;
  double acc = 0.0;
  for (int64_t k = threadIdx.x; k < n; k += kRows) acc += fabs(A[k + i * lda]);
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int st = kRows / 2; st > 0; st >>= 1) {
    if (threadIdx.x < st) sh[threadIdx.x] += sh[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[i] = sh[0];
}

__global__ void k_refine_step(const double *__restrict__ berr, double tol, int32_t *gate,
                              int32_t *iters) {
  if (threadIdx.x != 0 || *gate != 0) return;
  if (*berr <= tol)  // a NaN error never stops the steps
    *gate = 1;
  else
    *iters += 1;
}

__global__ void k_fill_i32(int32_t *p, int32_t v) {
  if (threadIdx.x == 0) p[0] = v;
}

__global__ void k_fill_f64(double *p, double v) {
  if (threadIdx.x == 0) p[0] = v;
}

// Krylov vector kernels (GMRES in FP64 on column blocks of <= kSkinnyMax
// independent columns; basis vector i of column c at V[i * vs + c * n + m]).
// out[i * N + c] = <V_i[:, c], W[:, c]>, one workgroup per (i, c).
__global__ void __launch_bounds__(kRows) k_coldots(int64_t n, int N, const double *__restrict__ V,
                                                   int64_t vs, const double *__restrict__ W,
                                                   int64_t ldw, double *__restrict__ out) {
  __shared__ double sh[kRows];
  const int i = blockIdx.x, c = blockIdx.y;
  const double *v = V + int64_t(i) * vs + int64_t(c) * n;
  const double *w = W + int64_t(c) * ldw;
  double acc = 0.0;
  for (int64_t m = threadIdx.x; m < n; m += kRows) acc += v[m] * w[m];
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int st = kRows / 2; st > 0; st >>= 1) {
    if (threadIdx.x < st) sh[threadIdx.x] += sh[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[i * N + c] = sh[0];
}

// W[:, c] += sign * sum_{i < J} coef[i * N + c] V_i[:, c]
__global__ void __launch_bounds__(kRows) k_colcombo(int64_t n, int N, int J,
                                                    const double *__restrict__ V, int64_t vs,
                                                    const double *__restrict__ coef, double sign,
                                                    double *__restrict__ W, int64_t ldw) {
  const int64_t m = int64_t(blockIdx.x) * kRows + threadIdx.x;
  const int c = blockIdx.y;
  if (m >= n) return;
  double acc = 0.0;
  for (int i = 0; i < J; ++i) acc += coef[i * N + c] * V[int64_t(i) * vs + int64_t(c) * n + m];
  W[m + int64_t(c) * ldw] += sign * acc;
}

// O[:, c] = W[:, c] / sqrt(nrm2[c]) (zero when nrm2[c] is not positive:
// a column whose Krylov space is exhausted contributes nothing more).
__global__ void __launch_bounds__(kRows) k_colscale(int64_t n, const double *__restrict__ W,
                                                    int64_t ldw, const double *__restrict__ nrm2,
                                                    double *__restrict__ O) {
  const int64_t m = int64_t(blockIdx.x) * kRows + threadIdx.x;
  const int c = blockIdx.y;
  if (m >= n) return;
  const double q = nrm2[c];
  O[m + int64_t(c) * n] = q > 0.0 ? W[m + int64_t(c) * ldw] / sqrt(q) : 0.0;
}

dim3 col_grid(int64_t n, int64_t nrhs) {
  return dim3(unsigned((n + kRows - 1) / kRows), unsigned(nrhs < 65535 ? nrhs : 65535));
}

// Whether k_rows_product takes a residual with more than 16 right-hand sides
// rather than a GEMM of 64 x 64 tiles: where those leave the device short of
// work, up to one tile per compute unit if all are whole, one and a half if some are
// partial, whose conditional loads are slower. On 256 compute units (n, right-hand
// sides, tiles: us as a GEMM / so), whole: 2048, 384, 192: 216 / 197; 4096, 192, 192:
// 280 / 264; 4096, 256, 256: 295 / 339; partial: 5003, 64, 79: 424 / 187; 5003, 256,
// 316: 576 / 460; 6000, 256, 376: 687 / 682; 8191, 192, 384: 890 / 975; 5003, 320, 395:
// 589 / 615; 4096, 400, 448: 502 / 555; 6000, 320, 470: 743 / 890.
bool few_gemm_tiles(int64_t n, int64_t nrhs) {
  const int64_t tiles = ((n + 63) / 64) * ((nrhs + 63) / 64);
  return 2 * tiles < (n % 64 == 0 && nrhs % 64 == 0 ? 2 : 3) * int64_t(device_cus());
}

// 16-row tiles per workgroup of k_rows_product for up to 16 right-hand sides:
// one until that makes a workgroup per compute unit, then two, which read
// longer runs of a column (one / two tiles, us: n = 4096 32 / 39, 4097 60 / 41,
// 8191 155 / 124).
int rows_tiles(int64_t n) { return n <= 16 * int64_t(device_cus()) ? 1 : 2; }

// O = G - op(A) X or op(A) X, and the workgroups' statistics; their number.
template <bool TRANS, bool ABS>
int64_t launch_rows_product(int64_t n, int64_t nrhs, const double *A, int64_t lda, const double *X,
                            int64_t ldx, const double *G, int64_t ldg, double *O, int64_t ldo,
                            double *blockstat, hipStream_t s) {
  const int rt = nrhs <= kSkinnyMax ? rows_tiles(n) : 1;
  const int ct = nrhs <= kSkinnyMax ? 1 : (nrhs <= 32 ? 2 : 4);
  const int64_t blocks = (n + 16 * rt - 1) / (16 * rt);
  const dim3 grid = dim3(unsigned(blocks), unsigned((nrhs + 16 * ct - 1) / (16 * ct)));
#define RBT_ROWS(RT, CT)                                                                         \
  if (rt == RT && ct == CT)                                                                      \
    hipLaunchKernelGGL((k_rows_product<TRANS, RT, CT, ABS>), grid, dim3(64 * kWaves), 0, s, n,   \
                       int(nrhs), A, lda, X, ldx, G, ldg, O, ldo, blockstat, refine_gate());
  RBT_ROWS(1, 1)
  RBT_ROWS(2, 1)
  RBT_ROWS(1, 2)
  RBT_ROWS(1, 4)
#undef RBT_ROWS
  return blocks;
}
template <bool TRANS>
hipError_t rows_residual(int64_t n, int64_t nrhs, const double *A, int64_t lda, const double *X,
                         int64_t ldx, const double *G, int64_t ldg, double *O, int64_t ldo,
                         bool with_anorm, double *blockstat, double *anorm, double *berr,
                         BerrHost host, hipStream_t s) {
  const int64_t blocks =
      with_anorm ? launch_rows_product<TRANS, true>(n, nrhs, A, lda, X, ldx, G, ldg, O, ldo, blockstat, s)
                 : launch_rows_product<TRANS, false>(n, nrhs, A, lda, X, ldx, G, ldg, O, ldo, blockstat, s);
  if (nrhs <= kSkinnyMax) {
    if (with_anorm)
      hipLaunchKernelGGL((k_berr_rows<true>), dim3(1), dim3(kRows), 0, s, blocks, int(nrhs), blockstat, anorm, berr, host, refine_gate());
    else
      hipLaunchKernelGGL((k_berr_rows<false>), dim3(1), dim3(kRows), 0, s, blocks, int(nrhs), blockstat, anorm, berr, host, refine_gate());
  } else if (with_anorm) {
    hipLaunchKernelGGL(k_max_reduce, dim3(1), dim3(kRows), 0, s, blocks, blockstat, anorm);
  }
  return hipGetLastError();
}

}  // namespace

// Of callers' workspaces, so the amount does not shrink: rbt_solve_ex_noalloc
// refuses the orders whose workspace exceeds its array. k_rows_product's
// statistics take blocks (3 N + 1) of it (blocks <= n / 16 + 1) for up to 16
// right-hand sides; more use abspart (chunks n), blockstat and colstat.
size_t resid_scratch_doubles(int64_t n, int64_t nrhs) {
  const int64_t chunks = (n + kChunk - 1) / kChunk;
  const int64_t nblk = (n + kRows - 1) / kRows;
  const int64_t nn = nrhs < 1 ? 1 : nrhs;
  const int64_t w = nn > kSkinnyMax ? 0 : nn;
  return size_t(chunks) * n * (w + 1) + size_t(nblk) * (3 * kSkinnyMax + 1) + 3 * size_t(nn) + 64;
}

hipError_t launch_residual_berr(int64_t n, int64_t nrhs, const double *A, int64_t lda,
                                const double *X, int64_t ldx, const double *B, int64_t ldb,
                                double *R, int64_t ldr, bool with_anorm, double *scratch,
                                double *anorm, double *berr, hipStream_t s, BerrHost host) {
  if (n <= 0 || nrhs <= 0) {
    hipLaunchKernelGGL(k_fill_f64, dim3(1), dim3(64), 0, s, berr, 0.0);
    return hipGetLastError();
  }
  const int64_t chunks = (n + kChunk - 1) / kChunk;
  const int64_t nblk = (n + kRows - 1) / kRows;
  if (nrhs <= kSkinnyMax)
    return rows_residual<false>(n, nrhs, A, lda, X, ldx, B, ldb, R, ldr, with_anorm, scratch, anorm, berr, host, s);
  double *abspart = scratch;
  double *blockstat = abspart + chunks * n;
  double *colstat = blockstat + nblk * (3 * kSkinnyMax + 1);
  if (few_gemm_tiles(n, nrhs)) {
    hipError_t e = rows_residual<false>(n, nrhs, A, lda, X, ldx, B, ldb, R, ldr, with_anorm, scratch, anorm, berr, host, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_colmax, dim3(unsigned(nrhs)), dim3(kRows), 0, s, n, R, ldr, X, ldx, B, ldb, colstat);
    hipLaunchKernelGGL(k_berr_final, dim3(1), dim3(64), 0, s, nrhs, colstat, anorm, berr, host);
    return hipGetLastError();
  }
  // wide: norms by their own pass, residual by the matrix-core GEMM
  if (with_anorm) {
    hipLaunchKernelGGL(k_rowabs_partial, dim3(unsigned(nblk), unsigned(chunks)), dim3(kRows), 0, s, n, A, lda, abspart);
    hipLaunchKernelGGL(k_rowabs_reduce, dim3(unsigned(nblk)), dim3(kRows), 0, s, n, chunks, abspart, blockstat);
    hipLaunchKernelGGL(k_max_reduce, dim3(1), dim3(kRows), 0, s, nblk, blockstat, anorm);
  }
  hipLaunchKernelGGL(k_copy_cols, col_grid(n, nrhs), dim3(kRows), 0, s, n, nrhs, B, ldb, R, ldr);
  hipError_t e = launch_dgemm(n, nrhs, n, A, lda, OpA::General, X, ldx, OpB::General, R, ldr,
                              Acc::Subtract, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_colmax, dim3(unsigned(nrhs)), dim3(kRows), 0, s, n, R, ldr, X, ldx, B, ldb, colstat);
  hipLaunchKernelGGL(k_berr_final, dim3(1), dim3(64), 0, s, nrhs, colstat, anorm, berr, host);
  return hipGetLastError();
}

hipError_t launch_axpy_cols(int64_t n, int64_t nrhs, const double *D, int64_t ldd, double *X,
                            int64_t ldx, hipStream_t s) {
  if (n == 0 || nrhs == 0) return hipSuccess;
  hipLaunchKernelGGL(k_axpy_cols, col_grid(n, nrhs), dim3(kRows), 0, s, n, nrhs, D, ldd, X, ldx, refine_gate());
  return hipGetLastError();
}

hipError_t launch_copy_cols(int64_t n, int64_t nrhs, const double *S, int64_t lds, double *D,
                            int64_t ldd, hipStream_t s) {
  if (n == 0 || nrhs == 0) return hipSuccess;
  hipLaunchKernelGGL(k_copy_cols, col_grid(n, nrhs), dim3(kRows), 0, s, n, nrhs, S, lds, D, ldd);
  return hipGetLastError();
}

hipError_t launch_neg_outer(int64_t n, int64_t nrhs, const double *Lm, int64_t ldl,
                            const double *X, int64_t ldx, double *dA, int64_t ldda,
                            hipStream_t s) {
  if (n == 0) return hipSuccess;
  const int64_t cols = (n + 15) / 16;
  const int64_t rows2 = (n + 1) / 2;  // two rows per lane
  const dim3 grid(unsigned((rows2 + kRows - 1) / kRows), unsigned(cols < 1024 ? cols : 1024));
  hipLaunchKernelGGL(k_neg_outer, grid, dim3(kRows), 0, s, n, nrhs, Lm, ldl, X, ldx, dA, ldda);
  return hipGetLastError();
}

namespace {
thread_local const int32_t *t_gate = nullptr;
}
const int32_t *refine_gate() { return t_gate; }
RefineGate::RefineGate(const int32_t *gate) : prev(t_gate) { t_gate = gate; }
RefineGate::~RefineGate() { t_gate = prev; }

hipError_t launch_refine_step(const double *berr, double tol, int32_t *gate, int32_t *iters,
                              hipStream_t s) {
  hipLaunchKernelGGL(k_refine_step, dim3(1), dim3(64), 0, s, berr, tol, gate, iters);
  return hipGetLastError();
}

hipError_t launch_fill_i32(int32_t *p, int32_t v, hipStream_t s) {
  hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, s, p, v);
  return hipGetLastError();
}

hipError_t launch_fill_f64(double *p, double v, hipStream_t s) {
  hipLaunchKernelGGL(k_fill_f64, dim3(1), dim3(64), 0, s, p, v);
  return hipGetLastError();
}

hipError_t launch_matvec(int64_t n, int64_t nrhs, const double *A, int64_t lda, const double *X,
                         int64_t ldx, double *Y, int64_t ldy, double *scratch, hipStream_t s) {
  if (n <= 0 || nrhs <= 0) return hipSuccess;
  if (nrhs > kSkinnyMax) return hipErrorInvalidValue;
  launch_rows_product<false, false>(n, nrhs, A, lda, X, ldx, nullptr, 0, Y, ldy, scratch, s);
  return hipGetLastError();
}

hipError_t launch_coldots(int64_t n, int N, int J, const double *V, int64_t vs, const double *W,
                          int64_t ldw, double *out, hipStream_t s) {
  if (J <= 0 || N <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_coldots, dim3(unsigned(J), unsigned(N)), dim3(kRows), 0, s, n, N, V, vs, W,
                     ldw, out);
  return hipGetLastError();
}

hipError_t launch_colcombo(int64_t n, int N, int J, const double *V, int64_t vs,
                           const double *coef, double sign, double *W, int64_t ldw,
                           hipStream_t s) {
  if (J <= 0 || N <= 0 || n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_colcombo, dim3(unsigned((n + kRows - 1) / kRows), unsigned(N)), dim3(kRows),
                     0, s, n, N, J, V, vs, coef, sign, W, ldw);
  return hipGetLastError();
}

hipError_t launch_colscale(int64_t n, int N, const double *W, int64_t ldw, const double *nrm2,
                           double *O, hipStream_t s) {
  if (N <= 0 || n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_colscale, dim3(unsigned((n + kRows - 1) / kRows), unsigned(N)), dim3(kRows),
                     0, s, n, W, ldw, nrm2, O);
  return hipGetLastError();
}

// R = G - A^T L (the residual of the adjoint system A^T L = G) and its Eq. 7
// backward error with ||A^T||_inf = ||A||_1 (with_anorm: computed here into
// *anorm, else read). scratch as launch_residual_berr.
hipError_t launch_residual_berr_T(int64_t n, int64_t nrhs, const double *A, int64_t lda,
                                  const double *L, int64_t ldl, const double *G, int64_t ldg,
                                  double *R, int64_t ldr, bool with_anorm, double *scratch,
                                  double *anorm, double *berr, hipStream_t s, BerrHost host) {
  if (n <= 0 || nrhs <= 0) {
    hipLaunchKernelGGL(k_fill_f64, dim3(1), dim3(64), 0, s, berr, 0.0);
    return hipGetLastError();
  }
  double *colabs = scratch;
  double *colstat = scratch + n;
  if (nrhs <= kSkinnyMax)
    return rows_residual<true>(n, nrhs, A, lda, L, ldl, G, ldg, R, ldr, with_anorm, scratch, anorm, berr, host, s);
  if (few_gemm_tiles(n, nrhs)) {
    hipError_t e = rows_residual<true>(n, nrhs, A, lda, L, ldl, G, ldg, R, ldr, with_anorm, scratch, anorm, berr, host, s);
    if (e != hipSuccess) return e;
  } else {
    if (with_anorm) {
      hipLaunchKernelGGL(k_colabs, dim3(unsigned(n)), dim3(kRows), 0, s, n, A, lda, colabs);
      hipLaunchKernelGGL(k_max_reduce, dim3(1), dim3(kRows), 0, s, n, colabs, anorm);
    }
    hipLaunchKernelGGL(k_copy_cols, col_grid(n, nrhs), dim3(kRows), 0, s, n, nrhs, G, ldg, R, ldr);
    hipError_t e = launch_dgemm(n, nrhs, n, A, lda, OpA::GeneralT, L, ldl, OpB::General, R, ldr,
                                Acc::Subtract, s);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_colmax, dim3(unsigned(nrhs)), dim3(kRows), 0, s, n, R, ldr, L, ldl, G, ldg,
                     colstat);
  hipLaunchKernelGGL(k_berr_final, dim3(1), dim3(64), 0, s, nrhs, colstat, anorm, berr, host);
  return hipGetLastError();
}

}  // namespace rbt
