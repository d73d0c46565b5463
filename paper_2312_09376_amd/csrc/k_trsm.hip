// Block triangular solves with a factored kb x kb diagonal block (kb <= 128)
// of the elimination, 16 rows (columns) at a time: the update from the
// blocks already solved runs on the FP64 matrix cores, and each 16 x 16
// diagonal block is solved by plain substitution, so the rounding behaviour
// is that of ordinary forward/back substitution except that a division by a
// pivot is a multiplication by its reciprocal (within one rounding of the
// quotient). (Multiplying by explicit inverses of the diagonal blocks, even
// 16 x 16 ones, raised the backward error several-fold on N(0,1) matrices
// with large growth.)
//
// The kernels are latency-bound chains of eight dependent steps, so every
// operand of the loop is staged in LDS once, with coalesced reads, before
// the first step: the 28 off-diagonal 16 x 16 blocks of the triangle in
// matrix-core operand order (56 KB), the eight diagonal blocks in the order
// the substitution reads them (16 KB), and each wavefront's right-hand-side
// strip (17 KB, padded rows). After that a wavefront only talks to its own
// strip, so the steps need no workgroup barrier (LDS accesses of one
// wavefront complete in issue order). 140 KB of LDS: one workgroup per CU.
//
// Substitution inside a diagonal block: lane l16 of each group of 16 lanes
// holds entry l16 of four right-hand sides, which is how the matrix-core
// product leaves them, and its 16 coefficients in registers. At pivot j lane j
// scales its entries and the update takes them as a DPP row broadcast inside
// the multiply-add: no LDS access and no shuffle in the chain of 16 pivots. The
// entries that a pivot does not update take a zero coefficient, which keeps
// them unless the pivot's entry is Inf or NaN (0 * Inf is NaN and stays so to the
// end of the tile); a tile that ends with a NaN is therefore solved again, those
// entries kept by a select. So every entry sees the same operations in the same
// order as in one-lane-per-right-hand-side substitution. (With four lanes per right-hand
// side, their coefficients read from LDS a pivot ahead: both solves of a panel
// step at n = 1000 18.2 us, now 17.7; the inverses of the diagonal blocks,
// where no pivot scales, 16.6 and 14.5.)
//
// Left solves, op(T) X = B in place (B: kb x N):
//   LN  T = L (unit lower)     forward  (panel U12 = L11^-1 A12, L y = b)
//   UN  T = U (upper)          backward (U x = y)
//   UT  T = U^T (lower)        forward  (U^T z = g, adjoint solves)
//   LT  T = L^T (unit upper)   backward (L^T w = z)
//   X_I = T_II \ (B_I - sum_{J before I} T_IJ X_J)
// Each wavefront owns 16 columns of B; a workgroup of four covers 64.
//
// Right solve, X U = B in place (B: M x kb) for the panel L21 = A21 U11^-1:
//   X_J = (B_J - sum_{I<J} X_I U_IJ) / U_JJ
// Each wavefront owns 16 rows of B.
//
// MFMA: 16 x 16 x 4 products in the arithmetic type C (mma16.h).
//
// The triangle (TT) and the right-hand sides (TB) may be stored in FP32
// (mixed-precision elimination). The arithmetic type C is FP64 for FP64
// factors; for FP32 factors it is FP32 (LDS, substitution and the FP32
// matrix cores), or FP64 as an option, in which case values are widened on
// load and rounded once on store.
#include "internal.h"
#include "mma16.h"
#include "row16.h"

namespace rbt {

namespace {

constexpr int NB = kNB;  // 128
constexpr int IB = 16;
constexpr int NBK = NB / IB;  // 8 diagonal blocks
constexpr int BLK = IB * IB;  // 256 doubles per block
constexpr int NOFF = NBK * (NBK - 1) / 2;  // 28 off-diagonal blocks on one side
// A wavefront's strip holds 128 vectors of 16 doubles, 17 apart: with a
// stride of 16 (128 bytes) the lanes that each own one vector hit the same
// LDS banks when staging and storing it back (65 % of the LDS cycles were
// bank conflicts).
constexpr int SLD = IB + 1;

template <TriMode MODE>
constexpr bool forward_order() {
  return MODE == TriMode::LN || MODE == TriMode::UT;
}
template <TriMode MODE>
constexpr bool unit_diag() {
  return MODE == TriMode::LN || MODE == TriMode::LT;
}

// op(T)(i, j) read from global memory (i, j < kb), in the stored type.
// Loads are issued unconditionally at clamped valid indices and masked
// afterwards, so that a batch of them is in flight together (a conditional
// load per element, or a widening right after it, serializes them).
template <TriMode MODE, typename TT>
__device__ __forceinline__ TT op_t(const TT *T, int64_t ldt, int i, int j) {
  if constexpr (MODE == TriMode::LN || MODE == TriMode::UN)
    return T[i + int64_t(j) * ldt];
  else
    return T[j + int64_t(i) * ldt];
}
__device__ __forceinline__ int clampi(int v, int hi) { return v < hi ? v : hi; }

// Orders the LDS accesses of the lanes of one wavefront (no instruction).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// In-place substitution with one 16 x 16 diagonal block: x[v] = entry l16 of
// four right-hand sides; m[j] = minus the coefficient of pivot j for entry l16,
// zero where it has none; rd = the reciprocal of the lane's own pivot. KEEP: the
// entries without a coefficient are kept by a select.
template <bool FWD, bool UNIT, bool KEEP, int S, typename C>
__device__ __forceinline__ void substitute(C (&x)[4], const C (&m)[IB], C rd, int l16) {
  if constexpr (S < IB) {
    constexpr int J = FWD ? S : IB - 1 - S;
    if constexpr (!UNIT) {
      const C f = l16 == J ? rd : C(1);
#pragma unroll
      for (int v = 0; v < 4; ++v) x[v] *= f;
    }
    if constexpr (KEEP) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const C nx = fma_c(m[J], row_bcast<J>(x[v]), x[v]);
        x[v] = (FWD ? l16 > J : l16 < J) ? nx : x[v];
      }
    } else {
      fmac_rows<J, 4>(x, m[J]);
    }
    substitute<FWD, UNIT, KEEP, S + 1>(x, m, rd, l16);
  }
}
template <bool FWD, bool UNIT, typename C>
__device__ __forceinline__ void substitute_tile(C (&x)[4], const C (&m)[IB], C rd, int l16) {
  C r[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) r[v] = x[v];
  substitute<FWD, UNIT, false, 0>(x, m, rd, l16);
  const bool nan = __builtin_isunordered(x[0], x[1]) || __builtin_isunordered(x[2], x[3]);
  if (__any(nan)) {
    substitute<FWD, UNIT, true, 0>(r, m, rd, l16);
#pragma unroll
    for (int v = 0; v < 4; ++v) x[v] = r[v];
  }
}

// BATCH: blockIdx.y selects diagonal block b of an n x n factor (T and B
// offset by b * kNB (1 + ldt) and b * bstride, kb = min(kNB, n - b kNB)), and
// the right-hand side is the identity (X = op(T_bb)^-1): used to form the
// inverses of the diagonal blocks once per factorization.
// LDS of one workgroup of either solve: diagonal blocks, off-diagonal
// blocks, four right-hand-side strips (136 KB).
template <typename C>
struct TrsmSmem {
  __attribute__((aligned(16))) C dblk[NBK * BLK];
  C drec[NB];  // reciprocals of the diagonal
  __attribute__((aligned(16))) C oblk[NOFF * BLK];
  __attribute__((aligned(16))) C strip[4][NB * SLD];
};

// Left solve of the 64 columns [64 bx, 64 bx + 64) of B.
template <TriMode MODE, bool BATCH, typename TT, typename TB, typename C>
__device__ __forceinline__ void trsm_left_body(int kb, int64_t N, const TT *T, int64_t ldt,
                                               TB *B, int64_t ldb, int64_t n, int64_t bstride,
                                               int64_t bx, TrsmSmem<C> &sm) {
  typedef Mma16<C> M;
  typedef typename M::v4 c4;
  typedef C c2 __attribute__((ext_vector_type(2)));
  if constexpr (BATCH) {
    const int64_t b = blockIdx.y;
    const int64_t r0 = b * NB;
    kb = int(n - r0 < NB ? n - r0 : NB);
    N = kb;
    T += r0 + r0 * ldt;
    B += b * bstride;
  }
  // dblk: -op(T)(i, j) of diagonal block b at b*256 + j*16 + i where pivot j
  // updates entry i, else zero; ablk: off-diagonal block (I, J), J before I, at
  // p*256 + lane*4 + kk = op(T)(16I + l16, 16J + 4kk + lk), p = I(I-1)/2 + J (forward) or J(J-1)/2 + I (backward)
  C *dblk = sm.dblk;
  C *ablk = sm.oblk;
  constexpr bool FWD = forward_order<MODE>();
  constexpr bool TRANS = MODE == TriMode::UT || MODE == TriMode::LT;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l16 = lane & 15, lk = lane >> 4;
  C *strip = sm.strip[wave];  // row-major 128 x 16
  const int64_t col0 = bx * 64 + wave * 16;

  TB sraw[BATCH ? 1 : 2][IB];  // the strip
  {  // stage the diagonal blocks and the off-diagonal operands, coalesced
     // (consecutive threads read consecutive addresses of the stored T), and the
     // strip: all loads are in flight before the first store waits
    const int f = threadIdx.x & 15, g = threadIdx.x >> 4;
    const int i = TRANS ? g : f, j = TRANS ? f : g;  // element (i, j) of a block of op(T)
    TT raw[NBK];
#pragma unroll
    for (int b = 0; b < NBK; ++b)
      raw[b] = op_t<MODE>(T, ldt, clampi(IB * b + i, kb - 1), clampi(IB * b + j, kb - 1));
    TT oraw[NOFF];
#pragma unroll
    for (int p = 0, I = 1; I < NBK; ++I)
#pragma unroll
      for (int J = 0; J < I; ++J, ++p) {
        // forward: block (I, J) below the diagonal; backward: (J, I) above it
        const int bi = FWD ? I : J, bj = FWD ? J : I;
        oraw[p] = op_t<MODE>(T, ldt, clampi(IB * bi + i, kb - 1), clampi(IB * bj + j, kb - 1));
      }
    if constexpr (!BATCH) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int64_t rr = clampi(lane + 64 * h, kb - 1);
#pragma unroll
        for (int cc = 0; cc < IB; ++cc)
          sraw[h][cc] = B[rr + (col0 + cc < N ? col0 + cc : N - 1) * ldb];
      }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int b = 0; b < NBK; ++b) {
      const int gi = IB * b + i, gj = IB * b + j;
      const C v = (gi < kb && gj < kb) ? C(raw[b]) : (i == j ? C(1) : C(0));
      if (!unit_diag<MODE>() && i == j) sm.drec[gi] = C(1) / v;
      dblk[b * BLK + j * IB + i] = (FWD ? i > j : i < j) ? -v : C(0);
    }
    const int slot = (16 * (j & 3) + i) * 4 + (j >> 2);  // lane (lk = j%4, l16 = i), kk = j/4
#pragma unroll
    for (int p = 0, I = 1; I < NBK; ++I)
#pragma unroll
      for (int J = 0; J < I; ++J, ++p) {
        const int bi = FWD ? I : J, bj = FWD ? J : I;
        const int gi = IB * bi + i, gj = IB * bj + j;
        ablk[p * BLK + slot] = (gi < kb && gj < kb) ? C(oraw[p]) : C(0);
      }
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {  // strip: lane = row (two halves), 16 columns
    const int row = lane + 64 * h;
#pragma unroll
    for (int c = 0; c < IB; ++c) {
      const int64_t col = col0 + c;
      if constexpr (BATCH)
        strip[row * SLD + c] = (row < kb && col < N && row == col) ? C(1) : C(0);
      else
        strip[row * SLD + c] = (row < kb && col < N) ? C(sraw[h][c]) : C(0);
    }
  }
  __syncthreads();

  const int nbk = (kb + IB - 1) / IB;
  for (int step = 0; step < nbk; ++step) {
    const int I = FWD ? step : nbk - 1 - step;
    C m[IB], x[4];
#pragma unroll
    for (int j = 0; j < IB; ++j) m[j] = dblk[I * BLK + j * IB + l16];
    const C rd = unit_diag<MODE>() ? C(1) : sm.drec[IB * I + l16];
    C *xs = strip + (IB * I + l16) * SLD + M::row(lk, 0);
    constexpr int RS = M::row(0, 1);  // right-hand sides between the lane's entries
#pragma unroll
    for (int v = 0; v < 4; ++v) x[v] = xs[RS * v];
    c4 acc0 = {C(0), C(0), C(0), C(0)}, acc1 = {C(0), C(0), C(0), C(0)};
#pragma unroll
    for (int s2 = 0; s2 < NBK - 1; ++s2) {
      if (s2 < step) {
        const int J = FWD ? s2 : nbk - 1 - s2;
        const int p = FWD ? I * (I - 1) / 2 + J : J * (J - 1) / 2 + I;
        const c2 a01 = *reinterpret_cast<const c2 *>(ablk + p * BLK + lane * 4);
        const c2 a23 = *reinterpret_cast<const c2 *>(ablk + p * BLK + lane * 4 + 2);
        const int k0 = IB * J + lk;
        // (right-hand sides x entries: the lane's column is its entry)
        acc0 = M::mma(strip[(k0) * SLD + l16], a01[0], acc0);
        acc1 = M::mma(strip[(k0 + 4) * SLD + l16], a01[1], acc1);
        acc0 = M::mma(strip[(k0 + 8) * SLD + l16], a23[0], acc0);
        acc1 = M::mma(strip[(k0 + 12) * SLD + l16], a23[1], acc1);
      }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) x[v] -= acc0[v] + acc1[v];
    substitute_tile<FWD, unit_diag<MODE>()>(x, m, rd, l16);
#pragma unroll
    for (int v = 0; v < 4; ++v) xs[RS * v] = IB * I + l16 < kb ? x[v] : C(0);
    wave_sync();
  }

#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int row = lane + 64 * h;
#pragma unroll
    for (int c = 0; c < IB; ++c) {
      const int64_t col = col0 + c;
      if (row < kb && col < N) B[row + col * ldb] = TB(strip[row * SLD + c]);
    }
  }
}

template <TriMode MODE, typename TT, typename TB, typename C>
__global__ void __launch_bounds__(256, 1) k_trsm_left(int kb, int64_t N, const TT *T,
                                                      int64_t ldt, TB *B, int64_t ldb) {
  __shared__ TrsmSmem<C> sm;
  trsm_left_body<MODE, false, TT, TB, C>(kb, N, T, ldt, B, ldb, int64_t(0), int64_t(0),
                                         int64_t(blockIdx.x), sm);
}

// Right solve of the 64 rows [64 bx, 64 bx + 64) of B.
template <typename TT, typename C>
__device__ __forceinline__ void trsm_right_upper_body(int kb, int64_t M, const TT *T, int64_t ldt,
                                                      TT *B, int64_t ldb, int64_t bx,
                                                      TrsmSmem<C> &sm) {
  typedef Mma16<C> Mm;
  typedef typename Mm::v4 c4;
  typedef C c2 __attribute__((ext_vector_type(2)));
  // dblk: -U(r, c) of diagonal block b at b*256 + r*16 + c for r < c, else
  // zero; ublk: block (I, J), I < J, at p*256 +
  // lane*4 + kk = U(16I + 4kk + lk, 16J + l16), p = J(J-1)/2 + I
  C *dblk = sm.dblk;
  C *ublk = sm.oblk;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l16 = lane & 15, lk = lane >> 4;
  C *strip = sm.strip[wave];  // column-major 16 x 128
  const int64_t row0 = bx * 64 + wave * 16;

  {  // stage the triangle, consecutive threads on consecutive rows of U, and the
     // strip (lane = row sr, column group cg: columns cg + 4 u): all loads are in
     // flight before the first store waits
    const int r = threadIdx.x % IB, c = threadIdx.x / IB;
    TT raw[NBK];
#pragma unroll
    for (int b = 0; b < NBK; ++b)
      raw[b] = T[clampi(IB * b + r, kb - 1) + int64_t(clampi(IB * b + c, kb - 1)) * ldt];
    TT uraw[NOFF];
#pragma unroll
    for (int p = 0, J = 1; J < NBK; ++J)
#pragma unroll
      for (int I = 0; I < J; ++I, ++p)
        uraw[p] = T[clampi(IB * I + r, kb - 1) + int64_t(clampi(IB * J + c, kb - 1)) * ldt];
    const int sr = lane % IB, cg = lane / IB;
    const int64_t row = row0 + sr;
    const int64_t rr = row < M ? row : M - 1;
    TT sraw[32];
#pragma unroll
    for (int u = 0; u < 32; ++u) sraw[u] = B[rr + int64_t(clampi(cg + 4 * u, kb - 1)) * ldb];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int b = 0; b < NBK; ++b) {
      const int gi = IB * b + r, gj = IB * b + c;
      const C v = (gi < kb && gj < kb) ? C(raw[b]) : (r == c ? C(1) : C(0));
      if (r == c) sm.drec[gi] = C(1) / v;
      dblk[b * BLK + r * IB + c] = r < c ? -v : C(0);
    }
    const int slot = (16 * (r & 3) + c) * 4 + (r >> 2);  // lane (lk = r%4, l16 = c), kk = r/4
#pragma unroll
    for (int p = 0, J = 1; J < NBK; ++J)
#pragma unroll
      for (int I = 0; I < J; ++I, ++p) {
        const int gi = IB * I + r, gj = IB * J + c;
        ublk[p * BLK + slot] = (gi < kb && gj < kb) ? C(uraw[p]) : C(0);
      }
#pragma unroll
    for (int u = 0; u < 32; ++u) {
      const int cu = cg + 4 * u;
      strip[cu * SLD + sr] = (row < M && cu < kb) ? C(sraw[u]) : C(0);
    }
  }
  __syncthreads();

  const int nbk = (kb + IB - 1) / IB;
  for (int J = 0; J < nbk; ++J) {
    C m[IB], x[4];
#pragma unroll
    for (int j = 0; j < IB; ++j) m[j] = dblk[J * BLK + j * IB + l16];
    const C rd = sm.drec[IB * J + l16];
    C *xs = strip + (IB * J + l16) * SLD + Mm::row(lk, 0);
    constexpr int RS = Mm::row(0, 1);  // rows between the lane's entries
#pragma unroll
    for (int v = 0; v < 4; ++v) x[v] = xs[RS * v];
    c4 acc0 = {C(0), C(0), C(0), C(0)}, acc1 = {C(0), C(0), C(0), C(0)};
#pragma unroll
    for (int I = 0; I < NBK - 1; ++I) {
      if (I < J) {
        const int p = J * (J - 1) / 2 + I;
        const c2 b01 = *reinterpret_cast<const c2 *>(ublk + p * BLK + lane * 4);
        const c2 b23 = *reinterpret_cast<const c2 *>(ublk + p * BLK + lane * 4 + 2);
        const int k0 = IB * I + lk;
        acc0 = Mm::mma(strip[(k0) * SLD + l16], b01[0], acc0);
        acc1 = Mm::mma(strip[(k0 + 4) * SLD + l16], b01[1], acc1);
        acc0 = Mm::mma(strip[(k0 + 8) * SLD + l16], b23[0], acc0);
        acc1 = Mm::mma(strip[(k0 + 12) * SLD + l16], b23[1], acc1);
      }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) x[v] -= acc0[v] + acc1[v];
    substitute_tile<true, false>(x, m, rd, l16);
#pragma unroll
    for (int v = 0; v < 4; ++v) xs[RS * v] = IB * J + l16 < kb ? x[v] : C(0);
    wave_sync();
  }

  {
    const int r = lane % IB, cg = lane / IB;
    const int64_t row = row0 + r;
#pragma unroll
    for (int u = 0; u < 32; ++u) {
      const int c = cg + 4 * u;
      if (row < M && c < kb) B[row + int64_t(c) * ldb] = TT(strip[c * SLD + r]);
    }
  }
}

// Both solves of a panel step with one factored diagonal block, which are
// independent: L21 = A21 U11^-1 (the first gr workgroups, 64 rows each) and
// U12 = L11^-1 A12 for the panel's columns to the right (the rest, 64
// columns each). One launch instead of two, and the short left solve runs
// beside the right one.
template <typename TT, typename C>
__global__ void __launch_bounds__(256, 1) k_panel_trsm(int kb, int64_t M, int64_t N, const TT *T,
                                                       int64_t ldt, TT *Br, TT *Bl, int64_t ldb,
                                                       int64_t gr) {
  __shared__ TrsmSmem<C> sm;
  const int64_t bx = blockIdx.x;
  if (bx < gr)
    trsm_right_upper_body<TT, C>(kb, M, T, ldt, Br, ldb, bx, sm);
  else
    trsm_left_body<TriMode::LN, false, TT, TT, C>(kb, N, T, ldt, Bl, ldb, int64_t(0),
                                                  int64_t(0), bx - gr, sm);
}

// Inverses of the diagonal blocks of L (blockIdx.z = 0) and of U, 64 of their
// columns per workgroup: one launch, the two side by side (n = 1000: 17 us, as two
// launches 29).
template <typename TT, typename C>
__global__ void __launch_bounds__(256, 1) k_diag_inverses(int64_t n, const TT *LU, int64_t ld, C *W) {
  __shared__ TrsmSmem<C> sm;
  // L^-1 at W + b * 2 kNB^2, U^-1 at W + b * 2 kNB^2 + kNB^2, each ld kNB
  if (blockIdx.z == 0)
    trsm_left_body<TriMode::LN, true, TT, C, C>(NB, int64_t(NB), LU, ld, W, int64_t(NB), n,
                                                int64_t(2 * NB * NB), int64_t(blockIdx.x), sm);
  else
    trsm_left_body<TriMode::UN, true, TT, C, C>(NB, int64_t(NB), LU, ld, W + NB * NB, int64_t(NB),
                                                n, int64_t(2 * NB * NB), int64_t(blockIdx.x), sm);
}

template <typename TT, typename TB, typename C>
hipError_t trsm_left_t(TriMode mode, int kb, int64_t N, const TT *T, int64_t ldt, TB *B,
                       int64_t ldb, hipStream_t s) {
  if (kb <= 0 || N <= 0) return hipSuccess;
  if (kb > kNB) return hipErrorInvalidValue;
  const dim3 grid(unsigned((N + 63) / 64));
  switch (mode) {
    case TriMode::LN: hipLaunchKernelGGL((k_trsm_left<TriMode::LN, TT, TB, C>), grid, dim3(256), 0, s, kb, N, T, ldt, B, ldb); break;
    case TriMode::UN: hipLaunchKernelGGL((k_trsm_left<TriMode::UN, TT, TB, C>), grid, dim3(256), 0, s, kb, N, T, ldt, B, ldb); break;
    case TriMode::UT: hipLaunchKernelGGL((k_trsm_left<TriMode::UT, TT, TB, C>), grid, dim3(256), 0, s, kb, N, T, ldt, B, ldb); break;
    case TriMode::LT: hipLaunchKernelGGL((k_trsm_left<TriMode::LT, TT, TB, C>), grid, dim3(256), 0, s, kb, N, T, ldt, B, ldb); break;
  }
  return hipGetLastError();
}

// Inverses of the diagonal blocks, in the arithmetic and storage type C of W.
template <typename TT, typename C>
hipError_t diag_inverses_t(int64_t n, const TT *LU, int64_t ld, C *W, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t nb = (n + NB - 1) / NB;
  if (nb > 65535) return hipErrorInvalidValue;
  // 2 x 64 columns of each 128 x 128 block
  hipLaunchKernelGGL((k_diag_inverses<TT, C>), dim3(2, unsigned(nb), 2), dim3(256), 0, s, n, LU, ld,
                     W);
  return hipGetLastError();
}

template <typename TT, typename C>
hipError_t panel_trsm_t(int kb, int64_t M, int64_t N, const TT *T, int64_t ldt, TT *Br, TT *Bl,
                        int64_t ldb, hipStream_t s) {
  if (kb <= 0 || (M <= 0 && N <= 0)) return hipSuccess;
  if (kb > kNB) return hipErrorInvalidValue;
  const int64_t gr = M > 0 ? (M + 63) / 64 : 0, gl = N > 0 ? (N + 63) / 64 : 0;
  if (gr + gl > 0x7fffffff) return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_panel_trsm<TT, C>), dim3(unsigned(gr + gl)), dim3(256), 0, s, kb, M, N, T,
                     ldt, Br, Bl, ldb, gr);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_trsm_left(TriMode mode, int kb, int64_t N, const double *T, int64_t ldt,
                            double *B, int64_t ldb, hipStream_t s) {
  return trsm_left_t<double, double, double>(mode, kb, N, T, ldt, B, ldb, s);
}
hipError_t launch_trsm_left(TriMode mode, int kb, int64_t N, const float *T, int64_t ldt, float *B,
                            int64_t ldb, bool fp64_arith, hipStream_t s) {
  return fp64_arith ? trsm_left_t<float, float, double>(mode, kb, N, T, ldt, B, ldb, s)
                    : trsm_left_t<float, float, float>(mode, kb, N, T, ldt, B, ldb, s);
}
hipError_t launch_diag_inverses(int64_t n, const double *LU, int64_t ld, double *W,
                                hipStream_t s) {
  return diag_inverses_t(n, LU, ld, W, s);
}
hipError_t launch_diag_inverses(int64_t n, const float *LU, int64_t ld, double *W, hipStream_t s) {
  return diag_inverses_t(n, LU, ld, W, s);
}
hipError_t launch_diag_inverses(int64_t n, const float *LU, int64_t ld, float *W, hipStream_t s) {
  return diag_inverses_t(n, LU, ld, W, s);
}
hipError_t launch_panel_trsm(int kb, int64_t M, int64_t N, const double *T, int64_t ldt,
                             double *Br, double *Bl, int64_t ldb, hipStream_t s) {
  return panel_trsm_t<double, double>(kb, M, N, T, ldt, Br, Bl, ldb, s);
}
hipError_t launch_panel_trsm(int kb, int64_t M, int64_t N, const float *T, int64_t ldt, float *Br,
                             float *Bl, int64_t ldb, bool fp64_arith, hipStream_t s) {
  return fp64_arith ? panel_trsm_t<float, double>(kb, M, N, T, ldt, Br, Bl, ldb, s)
                    : panel_trsm_t<float, float>(kb, M, N, T, ldt, Br, Bl, ldb, s);
}

}  // namespace rbt
