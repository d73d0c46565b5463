// Diagonal-block kernel of the blocked elimination without pivoting.
//
// One workgroup of 1024 threads factors a kb x kb diagonal block (kb <= 128)
// in place, A = L U with unit-lower L (Sec. 1, step 2: GENP), in eight
// 16-column steps on the block held in LDS (column-major, leading dimension
// 129 so that row-wise and column-wise lane patterns are both bank-conflict
// free). Every diagonal block is on the elimination's critical path and
// leaves the rest of the device idle, so what counts is the chain of 128
// pivots (a division, a multiplication, an update each); the rest is
// arranged to run beside it. In step p, columns c0 = 16 p .. c0 + 15:
//   - wavefronts 0 and 1 factor the panel right-looking, one row per lane;
//   - wavefronts 2 and 3 compute the 16-row block of U to its right, one row
//     per lane and four columns of each 16-column tile per group of 16 lanes;
//     all four keep a copy of the panel's top 16 rows in each group of 16
//     lanes, so a pivot row reaches its consumers as a DPP row broadcast
//     inside the multiply-add, and the 16 pivots need no barrier;
//   - wavefronts 4 to 15 meanwhile apply step p - 1 to the tiles right of and
//     below both, on the matrix cores, and store the finished columns;
//   - then all apply step p to the column tile and the row tile of step p + 1,
//     a 16 x 16 tile each (accumulators start from the LDS values, the L
//     operand is negated).
// Step 0 takes the panel and its row block straight from memory while
// wavefronts 4 to 15 stage the rest. Rows and columns beyond kb hold the
// identity, so they never disturb the active part. Measured for 128 columns:
// 36.7 -> 28.9 us (FP64) and 27.6 -> 23 us (FP32) against panel, row block and update
// one after the other on eight wavefronts with the pivot rows broadcast by
// readlane; a panel on its own takes 4200 cycles and 5000 to 7000 beside the
// products, which share the FP64 and FP32 units with it.
// The arithmetic type C is FP64 for FP64 factors; for the FP32
// factors of the mixed-precision elimination it is FP32 (LDS, broadcasts,
// the FP32 matrix cores), or FP64 as an option, in which case the block is
// widened on load and rounded once on store. A zero pivot is recorded in
// *info (first one, 1-based, offset gofs) and the arithmetic continues with
// IEEE Inf/NaN.
#include "internal.h"
#include "mma16.h"
#include "row16.h"

namespace rbt {

namespace {

constexpr int NB = kNB;  // 128
constexpr int LD = NB + 1;
constexpr int PW = 16;    // panel width
constexpr int NT = 1024;  // threads
constexpr int NW = NT / 64;
constexpr int UW0 = 2;    // first wavefront of the row block
constexpr int XW0 = 4;    // first wavefront of the trailing update
constexpr int XW = NW - XW0;

// Pivots K .. 15 of a panel: t holds the top 16 rows (a row per lane, in each
// group of 16 lanes), x what else the pivots update: PANEL, a row of the panel
// below the top per lane (its entry K becomes the multiplier); otherwise
// entries of the top's rows in 16 columns right of the panel. rp is the
// reciprocal of pivot K. The column of the next pivot is updated first, and its
// division (the chain) is issued between the other updates.
template <int K, bool PANEL, typename C>
__device__ __forceinline__ void pivot_steps(C (&t)[PW], C (&x)[PW], int l16, C rp) {
  // (rows up to the pivot's: a zero multiplier, also where their entry is not finite)
  const C mt = l16 > K ? -t[K] * rp : C(0);
  const C lx = PANEL ? x[K] * rp : C(0);
  if constexpr (K + 1 < PW) {
    fmac_rows<K, 1>(t + K + 1, mt);
    dpp_distance(t[K + 1]);
    const C q = row_bcast<K + 1>(t[K + 1]);
    C rn = C(1) / q;  // one division per pivot (scaling as in LAPACK's getf2)
    if constexpr (PANEL)
      fmac_rows<K, PW - 1 - K>(x + K + 1, t + K + 1, -lx);
    else
      fmac_rows<K, PW>(x, mt);
    fmac_rows<K, PW - 2 - K>(t + K + 2, mt);
    if constexpr (PANEL) x[K] = lx;
    t[K] = l16 > K ? -mt : t[K];
    __builtin_amdgcn_sched_barrier(0);
    pivot_steps<K + 1, PANEL>(t, x, l16, rn);
  } else {
    if constexpr (PANEL)
      x[K] = lx;
    else
      fmac_rows<K, PW>(x, mt);
    t[K] = l16 > K ? -mt : t[K];
  }
}

// The updates of one column right of the panel (v: its entry in the lane's row; l:
// the row of the panel's factored top), rows up to the pivot's kept by a select.
template <int K, typename C>
__device__ __forceinline__ void keep_steps(const C (&l)[PW], C &v, int l16) {
  if constexpr (K < PW) {
    const C nv = fma_c(-l[K], row_bcast<K>(v), v);
    v = l16 > K ? nv : v;
    keep_steps<K + 1>(l, v, l16);
  }
}

template <typename T, typename C>
__global__ void __launch_bounds__(NT) k_diag_lu(int kb, T *__restrict__ A, int64_t lda,
                                                 int64_t gofs, int32_t *__restrict__ info) {
  typedef Mma16<C> M;
  typedef typename M::v4 c4;
  __shared__ C S[NB * LD];
  // the top tile of the next panel (column-major): wavefronts 0 to 3 read it
  // from here, since wavefront 0 stores the factored one into S as soon as it
  // has it; written again only after the next barrier
  __shared__ C top[PW * (PW + 1)];
  __shared__ __attribute__((aligned(8))) int again[2];  // wavefronts 2 and 3

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lk = lane >> 4;
  const int nt = (kb + PW - 1) / PW;  // 16-column tiles
  if (tid >= 64 * UW0 && lane == 0 && tid < 64 * XW0) again[wave - UW0] = 0;

  // entry (r, c) of the block, identity beyond kb: the load is unconditional at
  // clamped indices, so that a batch of them is in flight together
  auto raw = [&](int r, int c) {
    return A[(r < kb ? r : kb - 1) + int64_t(c < kb ? c : kb - 1) * lda];
  };
  auto entry = [&](T v, int r, int c) {
    return (r < kb && c < kb) ? C(v) : (r == c ? C(1) : C(0));
  };
  // tile (i, j) -= (tile column q of L, row tile i) (tile row q of U, column tile j);
  // to_top: the result to `top`
  auto update_tile = [&](int q, int i, int j, bool to_top) {
    const C *pa = S + (PW * q + lk) * LD + PW * i + l16;
    const C *pb = S + (PW * j + l16) * LD + PW * q + lk;
    C *pc = S + (PW * j + l16) * LD + PW * i + M::row(lk, 0);
    constexpr int RS = M::row(0, 1);  // rows between the lane's results
    c4 acc;
    C a[4], b[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      a[kk] = -pa[4 * kk * LD];
      b[kk] = pb[4 * kk];
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[v] = pc[RS * v];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) acc = M::mma(a[kk], b[kk], acc);
    C *po = to_top ? top + l16 * (PW + 1) + M::row(lk, 0) : pc;
#pragma unroll
    for (int v = 0; v < 4; ++v) po[RS * v] = acc[v];
  };
  auto store_half = [&](int c, int h) {  // 64 rows of column c
    const int r = 64 * h + lane;
    if (r < kb && c < kb) A[r + int64_t(c) * lda] = T(S[c * LD + r]);
  };

  // Wavefronts 0 to 3: t, the top row of the step; x, on 0 and 1 the lane's row
  // below the panel, on 2 and 3 the top row's entries in column tiles
  // p + 1 + 4 (wave - 2) and the three after it, lane group lk columns 4 lk ..
  // 4 lk + 3 of each. A wavefront has a part in step p only where its rows or
  // tiles exist.
  C t[PW], x[PW];
  auto below = [&](int p) { return PW * (p + 1) + 64 * wave + lane; };
  auto tile0 = [&](int p) { return p + 1 + 4 * (wave - UW0); };
  auto panel = [&](int p) {
    return wave == 0 || (wave < UW0 && PW * (p + 1) + 64 * wave < PW * nt);
  };
  auto row_block = [&](int p) { return wave >= UW0 && wave < XW0 && tile0(p) < nt; };
  auto last = [](int i) { return i < NB ? i : NB - 1; };
  if (panel(0)) {
    T vt[PW], vx[PW];
    const int r = last(below(0));
#pragma unroll
    for (int j = 0; j < PW; ++j) {
      vt[j] = raw(l16, j);
      vx[j] = raw(r, j);
    }
#pragma unroll
    for (int j = 0; j < PW; ++j) {
      t[j] = entry(vt[j], l16, j);
      x[j] = entry(vx[j], r, j);
    }
  } else if (row_block(0)) {
    T vt[PW], vx[PW];
    auto col = [&](int j) { return last(PW * (tile0(0) + j / 4) + 4 * lk + j % 4); };
#pragma unroll
    for (int j = 0; j < PW; ++j) {
      vt[j] = raw(l16, j);
      vx[j] = raw(l16, col(j));
    }
#pragma unroll
    for (int j = 0; j < PW; ++j) {
      t[j] = entry(vt[j], l16, j);
      x[j] = entry(vx[j], l16, col(j));
      S[col(j) * LD + l16] = x[j];  // (for the case of a row that is not finite)
    }
  } else if (wave >= XW0) {
    // the rest of the block, rows and columns 16 .. 127 (indices beyond the
    // last repeat it)
    constexpr int NI = (NB - PW + XW - 1) / XW;
    T v[2 * NI];
    const int r0 = PW + lane, r1 = last(PW + 64 + lane);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = last(PW + (wave - XW0) + XW * i);
      v[2 * i] = raw(r0, c);
      v[2 * i + 1] = raw(r1, c);
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = last(PW + (wave - XW0) + XW * i);
      S[c * LD + r0] = entry(v[2 * i], r0, c);
      S[c * LD + r1] = entry(v[2 * i + 1], r1, c);
    }
  }
  if (wave < XW0) __builtin_amdgcn_s_setprio(3);  // the chain's wavefronts issue first
#pragma unroll 1
  for (int p = 0; p < nt; ++p) {
    const int c0 = PW * p, c1 = c0 + PW;
    if (panel(p)) {
      pivot_steps<0, true>(t, x, l16, C(1) / row_bcast<0>(t[0]));
      if (wave == 0) {  // first zero pivot of the panel: lane j holds pivot j in t[j]
        C d = t[0];
#pragma unroll
        for (int j = 1; j < PW; ++j) d = l16 == j ? t[j] : d;
        const unsigned long long z = __ballot(lane < PW && c0 + lane < kb && d == C(0));
        if (lane == 0 && z != 0 && info != nullptr)
          atomicCAS(info, 0, int32_t(gofs + c0 + __ffsll(z)));
        if (lane < PW) {
          C *q = S + c0 * LD + c0 + l16;
#pragma unroll
          for (int j = 0; j < PW; ++j) q[j * LD] = t[j];
        }
      }
      if (below(p) < NB) {
        C *q = S + c0 * LD + below(p);
#pragma unroll
        for (int j = 0; j < PW; ++j) q[j * LD] = x[j];
      }
    } else if (row_block(p)) {
      pivot_steps<0, false>(t, x, l16, C(1) / row_bcast<0>(t[0]));
      C *q = S + (PW * tile0(p) + 4 * lk) * LD + c0 + l16;
      bool nan = false;
#pragma unroll
      for (int j = 0; j < PW; j += 2) nan = nan || __builtin_isunordered(x[j], x[j + 1]);
      if (__any(nan)) {
        if (lane == 0) again[wave - UW0] = 1;  // (see after the barrier)
      } else {
#pragma unroll
        for (int h = 0; h < 4; ++h) {
          if (tile0(p) + h < nt) {
#pragma unroll
            for (int j = 0; j < 4; ++j) q[(PW * h + j) * LD] = x[4 * h + j];
          }
        }
      }
    } else if (wave >= XW0 && p > 0) {
      // step p - 1 on the tiles beyond step p's, and the columns that it
      // finished to memory
      // (from p = 3 on wavefronts 1 and 3 have no part: the products go to their
      // SIMDs, since one that issues them slows a chain beside it)
      const int m = nt - 1 - p;
      const bool odd = m <= 4;
      const int first = odd ? (wave - XW0) >> 1 : wave - XW0;
      const int step = odd ? XW / 2 : XW;
      for (int i = first, j = 0; m > 0 && !(odd && (wave & 1) == 0); i += step) {
        while (i >= m && j < m) {
          i -= m;
          ++j;
        }
        if (j >= m) break;
        update_tile(p - 1, p + 1 + i, p + 1 + j, false);
      }
      for (int e = wave - XW0; e < 2 * PW; e += XW) store_half(c0 - PW + (e >> 1), e & 1);
    }
    __syncthreads();
    // Where a pivot row is not finite, the zero multipliers of the rows up to it
    // have made NaN of finished entries of the row block (0 * Inf): then once more
    // from the entries before, with selects. Without a NaN the two are
    // bit-identical. (Here, where no wavefront holds a part of the block in
    // registers, the case costs the others none.)
    if ((again[0] | again[1]) != 0) {
      if (row_block(p) && again[wave - UW0] != 0) {
        C l[PW];
#pragma unroll
        for (int j = 0; j < PW; ++j) l[j] = S[(c0 + j) * LD + c0 + l16];
#pragma unroll 1
        for (int e = 0; e < PW && tile0(p) + (e >> 2) < nt; ++e) {
          C *q = S + (PW * (tile0(p) + (e >> 2)) + 4 * lk + (e & 3)) * LD + c0 + l16;
          C v = *q;
          keep_steps<0>(l, v, l16);
          *q = v;
        }
      }
      __syncthreads();
      if (tid < 2) again[tid] = 0;
    }
    // step p on the column tile and the row tile of step p + 1
    const int m = nt - 1 - p;
    if (wave < 2 * m - 1)
      update_tile(p, wave < m ? p + 1 + wave : p + 1, wave < m ? p + 1 : p + 2 + wave - m,
                  wave == 0);
    if (m == 0) break;
    __syncthreads();
    if (wave < XW0) {
#pragma unroll
      for (int j = 0; j < PW; ++j) t[j] = top[j * (PW + 1) + l16];
      if (wave < UW0) {
        const C *q = S + c1 * LD + last(below(p + 1));
#pragma unroll
        for (int j = 0; j < PW; ++j) x[j] = q[j * LD];
      } else {
        const C *q = S + (PW * tile0(p + 1) + 4 * lk) * LD + c1 + l16;
#pragma unroll
        for (int h = 0; h < 4; ++h) {
          const C *qh = tile0(p + 1) + h < nt ? q + PW * h * LD : S;  // (not used beyond nt)
#pragma unroll
          for (int j = 0; j < 4; ++j) x[4 * h + j] = qh[j * LD];
        }
      }
    } else {  // (no values to keep: without this the registers of both arrays stay taken)
      forget(t);
      forget(x);
    }
  }
  for (int e = wave; e < 2 * PW; e += NW) store_half(PW * (nt - 1) + (e >> 1), e & 1);
}

}  // namespace

template <typename T, typename C>
hipError_t diag_lu_t(int kb, T *A, int64_t lda, int64_t gofs, int32_t *info, hipStream_t s) {
  if (kb <= 0) return hipSuccess;
  if (kb > kNB) return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_diag_lu<T, C>), dim3(1), dim3(NT), 0, s, kb, A, lda, gofs, info);
  return hipGetLastError();
}

hipError_t launch_diag_lu(int kb, double *A, int64_t lda, int64_t gofs, int32_t *info,
                          hipStream_t s) {
  return diag_lu_t<double, double>(kb, A, lda, gofs, info, s);
}
hipError_t launch_diag_lu(int kb, float *A, int64_t lda, int64_t gofs, int32_t *info,
                          bool fp64_arith, hipStream_t s) {
  return fp64_arith ? diag_lu_t<float, double>(kb, A, lda, gofs, info, s)
                    : diag_lu_t<float, float>(kb, A, lda, gofs, info, s);
}

}  // namespace rbt
