// Gaussian elimination with partial pivoting (GEPP), the robust solver that
// the fallback of Sec. 5 re-solves with when the unpivoted RBT solve cannot
// be refined to the tolerance (the "responsibly reckless" pairing of a fast
// unpivoted solve with a check and a pivoted re-solve).
//
// Blocked right-looking, panels of kNB = 128 columns in slabs of kSlab = 32:
//   k_gepp_slab  factors a slab in one launch: its rows stay in registers over
//                all 32 columns, spread over at most kSlabGroups workgroups,
//                which exchange one pivot candidate each per column;
//   k_gepp_swap  applies the slab's 32 interchanges to all other columns at
//                once, as one gather per column;
//   then U = L11^-1 A12 of the panel's columns right of the slab (k_trsm.hip,
//   unit lower) and their update on the FP64 matrix cores (k_gemm.hip); after
//   the panel's last slab the same for the trailing matrix, with depth 128.
// Slabs of more rows than the workgroups can hold (and a workspace too small
// for the exchange) go column by column: k_pivot_partial (max |a_ij| over
// many workgroups), k_pivot_swap (pivot row, ipiv, interchange over all
// columns) and k_panel_column (multipliers and rank-1 update).
// Every path takes the first row among equal magnitudes (LAPACK's idamax) and
// records ipiv[j] = p + 1 (1-based, LAPACK's getrf convention).
// A zero pivot column (max |a_ij| = 0) is recorded in *info (first, 1-based)
// and left unswapped; the elimination goes on with IEEE Inf/NaN.
//
// Solves: ipiv is turned into the permutation it applies (one thread,
// sequential, in LDS), the rows of B are gathered through it in parallel, and
// the triangular solves reuse the sweeps of the unpivoted factors (the L\U
// layout is the same).
#include "internal.h"

namespace rbt {

namespace {

constexpr int TPB = 256;
constexpr int kPivotGroups = 256;  // workgroups of the pivot search

__device__ __forceinline__ bool better(double v, int64_t i, double bv, int64_t bi) {
  // larger magnitude wins; equal magnitudes: the smaller row index; NaN
  // never wins over a number (a NaN column then pivots on its first row)
  return v > bv || (v == bv && i < bi);
}

__global__ void __launch_bounds__(TPB)
    k_pivot_partial(int64_t n, const double *__restrict__ A, int64_t lda, int64_t j,
                    double *__restrict__ pval, int64_t *__restrict__ pidx) {
  __shared__ double sv[TPB / 64];
  __shared__ int64_t si[TPB / 64];
  double bv = -1.0;
  int64_t bi = INT64_MAX;
  const double *col = A + j * lda;
  for (int64_t i = j + int64_t(blockIdx.x) * TPB + threadIdx.x; i < n;
       i += int64_t(gridDim.x) * TPB) {
    const double v = fabs(col[i]);
    if (better(v, i, bv, bi)) {
      bv = v;
      bi = i;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const double ov = __shfl_xor(bv, o);
    const int64_t oi = __shfl_xor(bi, o);
    if (better(ov, oi, bv, bi)) {
      bv = ov;
      bi = oi;
    }
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) {
    sv[wave] = bv;
    si[wave] = bi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < TPB / 64; ++w)
      if (better(sv[w], si[w], bv, bi)) {
        bv = sv[w];
        bi = si[w];
      }
    pval[blockIdx.x] = bv;
    pidx[blockIdx.x] = bi;
  }
}

__global__ void __launch_bounds__(TPB)
    k_pivot_swap(int64_t n, double *__restrict__ A, int64_t lda, int64_t j, int groups,
                 const double *__restrict__ pval, const int64_t *__restrict__ pidx,
                 int64_t *__restrict__ ipiv, int32_t *__restrict__ info) {
  __shared__ int64_t p_sh;
  if (threadIdx.x == 0) {
    double bv = -1.0;
    int64_t bi = INT64_MAX;
    for (int g = 0; g < groups; ++g)
      if (better(pval[g], pidx[g], bv, bi)) {
        bv = pval[g];
        bi = pidx[g];
      }
    int64_t p = bi;
    if (!(bv > 0.0) || p >= n) {  // zero (or NaN) column: no interchange
      if (bv == 0.0 && info != nullptr && *info == 0) *info = int32_t(j + 1);
      p = j;
    }
    ipiv[j] = p + 1;
    p_sh = p;
  }
  __syncthreads();
  const int64_t p = p_sh;
  if (p == j) return;
  for (int64_t c = threadIdx.x; c < n; c += TPB) {
    double *a = A + j + c * lda, *b = A + p + c * lda;
    const double t = *a;
    *a = *b;
    *b = t;
  }
}

// Column j of the panel [k0, kend): multipliers below the pivot and the
// rank-1 update of the panel columns j+1 .. kend-1.
__global__ void __launch_bounds__(TPB)
    k_panel_column(int64_t n, double *__restrict__ A, int64_t lda, int64_t j, int64_t kend) {
  const int64_t i = j + 1 + int64_t(blockIdx.x) * TPB + threadIdx.x;
  if (i >= n) return;
  const double piv = A[j + j * lda];
  const double l = A[i + j * lda] / piv;
  A[i + j * lda] = l;
  for (int64_t c = j + 1; c < kend; ++c) A[i + c * lda] -= l * A[j + c * lda];
}

// ---- slab of kSlab columns in one launch ----
//
// What bounds it: one dependent chain per column, a reduction in each wavefront and
// one over the wavefronts, the candidate's row written by one lane, barriers, a
// division and the update. A column takes 2.1 us in one workgroup (up to 1024 rows)
// and 2.9 in several, whose exchange goes through the memory side of the XCDs' caches
// (a store and a load); column by column,
// in launches of their own, it took 46 us at n = 4000 (21 of them one
// workgroup's strided swap of two rows over all columns). The factorization
// went from 178 to 14 ms (0.2 of it the agreement below) at n = 4000 and from 3.78 s to 0.22 s at n = 20000.
// Publishing a candidate from LDS as one coalesced store instead of 34 stores
// of one lane took a column from 3.7 to 2.8 us.
//
// Workgroup g owns kSlabThreads * RPT consecutive rows, thread t the rows
// g * kSlabThreads * RPT + r * kSlabThreads + t. Per column every workgroup publishes
// its best candidate (magnitude, row and the row's 32 entries), workgroup 0
// also the diagonal row; every workgroup reads all of them, picks the same
// winner and has both rows of the interchange at hand. The publication buffer
// has a slot of its own for each column, preset to a signalling NaN that
// arithmetic never yields, so each 8-byte entry says by itself that it has
// arrived (as in the triangular sweeps): one store and one load per column.
//
// Progress: the workgroups wait for each other, so all of them must be resident,
// which other work on the device (other streams, other processes) may prevent for
// as long as it likes, or for good where it waits for this slab's CUs in turn. So
// they agree first: the exchange of column 0 decides, by one compare-and-swap on a
// word of the buffer, between "together" (some workgroup has seen every candidate, so
// all are resident and every later wait ends) and "alone" (some workgroup waited
// for longer than the sweeps' spin limit). Alone, the workgroup that decided it
// factors the slab by itself from memory, where nothing has been stored yet, and the
// others leave; the later slabs of the factorization are then taken alone at once.
// Either way the factors are the same. In the common case this is one
// compare-and-swap of one thread per slab, beside column 0's update (n = 4000: 15.3 ->
// 15.5 ms). Together, waits
// are bounded all the same (kSlabSpins, none after the first that expires); one that
// expires, or a negative limit, which makes every wait expire at once, leaves NaN in
// the slab, *info = -1 and *err set (both nullable). The workgroups take an eighth of
// the device's CUs at most (slab_max_groups): the four hardware queues of a process,
// each of which dispatches in order, then never hold more than half of it waiting.
//
// The column loop is unrolled over 8 columns only (32 copies of its body would
// not fit the instruction cache): after 8 columns the 32 registers of a row
// are rotated by 8, and the columns already done, then at the end, are
// skipped by a uniform branch.
constexpr int kSlab = 32;
constexpr int kSlabThreads = 512;
constexpr int kSlabGroups = 32;
constexpr int kSlabMaxRpt = 2;  // (three rows of 32 entries no longer fit the registers)
constexpr int kSlot = kSlab + 2;  // row entries, magnitude (-1: no candidate), row
constexpr uint64_t kSlabUnpublished = 0x7FF4B1A5C0DE0001ull;

__device__ __forceinline__ bool slab_unpublished(double v) {
  return __builtin_bit_cast(uint64_t, v) == kSlabUnpublished;
}
__device__ __forceinline__ void slab_publish(double *p, double v) {
  __hip_atomic_store(p, slab_unpublished(v) ? __builtin_nan("") : v, __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}

// Order-preserving key of a candidate magnitude: 0 for none (and NaN, which
// never wins over a number).
__device__ __forceinline__ uint64_t mag_key(double mag) {
  return mag >= 0.0 ? __builtin_bit_cast(uint64_t, mag) + 1 : 0;
}
__device__ __forceinline__ double key_mag(uint64_t key) {
  return key == 0 ? -1.0 : __builtin_bit_cast(double, key - 1);
}

template <int CTRL, int ROWS, bool MIN>
__device__ __forceinline__ uint32_t dpp_step(uint32_t v) {
  const uint32_t o = uint32_t(
      __builtin_amdgcn_update_dpp(MIN ? -1 : 0, int(v), CTRL, ROWS, 0xF, false));
  return MIN ? (o < v ? o : v) : (o > v ? o : v);
}
// Extreme of v over the wavefront (FULL), or over its first 8 lanes.
template <bool MIN, bool FULL>
__device__ __forceinline__ uint32_t wave_extreme(uint32_t v) {
  v = dpp_step<0x111, 0xF, MIN>(v);  // row_shr 1, 2, 4, 8
  v = dpp_step<0x112, 0xF, MIN>(v);
  v = dpp_step<0x114, 0xF, MIN>(v);
  if constexpr (!FULL) return uint32_t(__builtin_amdgcn_readlane(int(v), 7));
  v = dpp_step<0x118, 0xF, MIN>(v);
  v = dpp_step<0x142, 0xA, MIN>(v);  // row_bcast 15, 31
  v = dpp_step<0x143, 0xC, MIN>(v);
  return uint32_t(__builtin_amdgcn_readlane(int(v), 63));
}
// Largest key of the wavefront (or of its first 8 lanes, the others holding
// 0) and the smallest row among the lanes that hold it (uniform results), and
// the first lane that does. The upper halves of the keys nearly always decide.
template <bool FULL>
__device__ __forceinline__ int wave_argmax(uint64_t &key, uint32_t &row) {
  const uint32_t hi = uint32_t(key >> 32), lo = uint32_t(key);
  const uint32_t mh = wave_extreme<false, FULL>(hi);
  unsigned long long at = __ballot(hi == mh);
  if (!FULL) at &= 0xFF;
  int src;
  if ((at & (at - 1)) == 0) {
    src = __ffsll(at) - 1;
  } else {
    const uint32_t ml = wave_extreme<false, FULL>(hi == mh ? lo : 0u);
    const bool top = hi == mh && lo == ml;
    const uint32_t r = wave_extreme<true, FULL>(top ? row : 0xFFFFFFFFu);
    at = __ballot(top && row == r);
    if (!FULL) at &= 0xFF;
    src = __ffsll(at) - 1;
  }
  row = uint32_t(__builtin_amdgcn_readlane(int(row), src));
  key = (uint64_t(mh) << 32) | uint32_t(__builtin_amdgcn_readlane(int(lo), src));
  return src;
}

// Control words behind the publication buffer: the decision of a slab (preset with
// the buffer), and 1 + the first column of the last slab taken alone, 0 if none was.
constexpr int kSlabControl = 2;
constexpr uint64_t kSlabTogether = 1, kSlabAlone = 2;
constexpr int64_t kSlabSpins = int64_t(1) << 24;
__device__ __forceinline__ uint64_t look(const uint64_t *word) {
  return __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
constexpr int kLeaveSlab = 1, kTakeSlab = 2;  // what a workgroup of a slab taken alone does

template <int RPT>
__global__ void __launch_bounds__(kSlabThreads)
    k_gepp_slab(int64_t n, double *__restrict__ A, int64_t lda, int64_t k0, int w, int groups,
                double *pub, uint64_t *control, int64_t *__restrict__ ipiv,
                int32_t *__restrict__ info, int64_t spin_limit, int32_t *err) {
  constexpr int NWAVE = kSlabThreads / 64;
  // this workgroup's candidates, one per wavefront, and the diagonal row (two
  // columns' worth, so that a column needs no barrier after its last read)
  __shared__ __attribute__((aligned(16))) double sw[2][NWAVE + 1][kSlab];
  __shared__ __attribute__((aligned(16))) double sl[(kSlabGroups + 1) * kSlot];
  __shared__ uint64_t skey[2][NWAVE];
  __shared__ uint32_t srow[2][NWAVE];
  __shared__ int expired_sh, mode_sh;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g = blockIdx.x;
  const bool agree = groups > 1 && spin_limit >= 0;
  const uint32_t m = uint32_t(n - k0);
  const uint32_t first = uint32_t(g) * (kSlabThreads * RPT) + uint32_t(tid);
  double *S = A + k0 + k0 * lda;  // row r, column c of the slab at S[r + c lda]
  int64_t limit = spin_limit < 0 ? spin_limit : (spin_limit < kSlabSpins ? kSlabSpins : spin_limit);

  double x[RPT][kSlab];
#pragma unroll
  for (int r = 0; r < RPT; ++r) {
    const uint32_t row = first + uint32_t(r) * kSlabThreads;
    const uint32_t rc = row < m ? row : m - 1;  // clamped: never stored
#pragma unroll
    for (int c = 0; c < kSlab; ++c) x[r][c] = c < w ? S[rc + int64_t(c) * lda] : 0.0;
  }
  if (tid == 0) {
    expired_sh = mode_sh = 0;
    const uint64_t since = agree ? look(control + 1) : 0;
    if (since != 0)  // (this slab's own decision, or an earlier one's)
      mode_sh = g == 0 && since != uint64_t(k0) + 1 ? kTakeSlab : kLeaveSlab;
  }
  if (agree) __syncthreads();

  const int columns = agree && mode_sh != 0 ? 0 : w;
#pragma unroll 1
  for (int q = 0; q < kSlab / 8; ++q) {
    // position c of a row holds column (c + 8 q) mod kSlab
#pragma unroll
    for (int jj = 0; jj < 8; ++jj) {
      const int j = 8 * q + jj;
      if (j < columns) {
        // ---- this workgroup's candidate for column j ----
        uint64_t key = 0;
        uint32_t row = 0xFFFFFFFFu;
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
          const uint32_t rr = first + uint32_t(r) * kSlabThreads;
          const uint64_t kr = (rr >= uint32_t(j) && rr < m) ? mag_key(fabs(x[r][jj])) : 0;
          if (kr > key) {  // rows ascend with r: the first of equal ones stays
            key = kr;
            row = rr;
          }
        }
        const int buf = jj & 1;
        wave_argmax<true>(key, row);
        if (lane == 0) {
          skey[buf][wave] = key;
          srow[buf][wave] = row;
        }
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
          const uint32_t rr = first + uint32_t(r) * kSlabThreads;
          if (rr == row || rr == uint32_t(j)) {
            double *d = rr == row ? sw[buf][wave] : sw[buf][NWAVE];
#pragma unroll
            for (int c = 0; c < kSlab; ++c) d[c] = x[r][c];
            if (rr == row && rr == uint32_t(j)) {
#pragma unroll
              for (int c = 0; c < kSlab; ++c) sw[buf][NWAVE][c] = x[r][c];
            }
          }
        }
        __syncthreads();
        if (jj == 1 && q == 0 && mode_sh != 0) limit = -1;  // (column 0 decided: alone)
        key = lane < NWAVE ? skey[buf][lane] : 0;
        row = lane < NWAVE ? srow[buf][lane] : 0xFFFFFFFFu;
        const int ww = wave_argmax<false>(key, row);
        const double *drow = sw[buf][NWAVE], *prow = sw[buf][ww];
        if (groups > 1) {
          // ---- publish it (one coalesced store), and the diagonal row, which
          // workgroup 0 holds ----
          double *pj = pub + int64_t(j) * (groups + 1) * kSlot;
          if (wave == 0 && lane < kSlot) {
            const double v = lane < kSlab ? (key != 0 ? sw[buf][ww][lane] : 0.0)
                                          : (lane == kSlab ? key_mag(key) : double(row));
            slab_publish(pj + g * kSlot + lane, v);
          }
          if (g == 0 && wave == 1 && lane < kSlab)
            slab_publish(pj + groups * kSlot + lane, drow[lane]);
          // ---- all candidates and the diagonal row ----
          const int total = (groups + 1) * kSlot - 2;  // the diagonal row has no last two
          bool opening = jj == 0 && q == 0 && agree;
          for (;;) {
            const int64_t most = opening ? spin_limit : limit;
            bool expired = false;
            for (int e = tid; e < total; e += kSlabThreads) {
              double v = __hip_atomic_load(pj + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              int64_t spins = 0;
              while (slab_unpublished(v)) {
                if (spins >= most || (opening && spins % 64 == 63 && look(control) == kSlabAlone)) {
                  expired = true;
                  v = __builtin_nan("");
                  break;
                }
                __builtin_amdgcn_s_sleep(1);
                ++spins;
                v = __hip_atomic_load(pj + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              }
              sl[e] = v;
            }
            if (expired) expired_sh = 1;
            __syncthreads();
            if (!opening) break;
            // the decision: this workgroup's has all candidates, or has waited enough
            const bool all = expired_sh == 0;
            if (tid == 0) {
              uint64_t seen = kSlabUnpublished;
              const bool made = __hip_atomic_compare_exchange_strong(
                  control, &seen, all ? kSlabTogether : kSlabAlone, __ATOMIC_RELAXED,
                  __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              if (made ? !all : seen == kSlabAlone) mode_sh = made ? kTakeSlab : kLeaveSlab;
            }
            if (all) break;  // (what was decided is read at column 1)
            __syncthreads();
            if (mode_sh != 0) break;
            if (tid == 0) expired_sh = 0;  // together: the candidates are on their way
            __syncthreads();
            opening = false;
          }
          if (expired_sh != 0) limit = -1;
          // ---- the winner, the same in every workgroup ----
          key = 0;
          row = 0xFFFFFFFFu;
          if (lane < groups) {
            key = mag_key(sl[lane * kSlot + kSlab]);
            if (key != 0) row = uint32_t(sl[lane * kSlot + kSlab + 1]);
          }
          const int wg = wave_argmax<true>(key, row);
          drow = sl + groups * kSlot;
          prow = sl + wg * kSlot;
        }
        const bool pivot = key > 1;  // key 1 is magnitude zero: left unswapped
        const uint32_t p = pivot ? row : uint32_t(j);
        if (!pivot) prow = drow;
        if (g == 0 && tid == 0 && mode_sh == 0) {
          ipiv[k0 + j] = k0 + int64_t(p) + 1;
          if (key == 1 && info != nullptr && *info == 0) *info = int32_t(k0 + j + 1);
        }
        // ---- interchange, multipliers, rank-1 update ----
        const double piv = prow[jj];
        const bool moved = p != uint32_t(j);
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
          const uint32_t rr = first + uint32_t(r) * kSlabThreads;
          if (moved && (rr == p || rr == uint32_t(j))) {
            const double *src = rr == p ? drow : prow;
#pragma unroll
            for (int c = 0; c < kSlab; ++c) x[r][c] = src[c];
          }
        }
        double u[kSlab];
#pragma unroll
        for (int cq = 0; cq < kSlab / 8; ++cq) {
          if (cq + q < kSlab / 8) {  // later positions hold columns already done
#pragma unroll
            for (int ci = 0; ci < 8; ++ci)
              if (8 * cq + ci > jj) u[8 * cq + ci] = prow[8 * cq + ci];
          }
        }
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
          if (first + uint32_t(r) * kSlabThreads > uint32_t(j)) {
            const double l = x[r][jj] / piv;
            x[r][jj] = l;
#pragma unroll
            for (int cq = 0; cq < kSlab / 8; ++cq) {
              if (cq + q < kSlab / 8) {
#pragma unroll
                for (int ci = 0; ci < 8; ++ci) {
                  const int c = 8 * cq + ci;
                  if (c > jj) x[r][c] = __builtin_fma(-l, u[c], x[r][c]);
                }
              }
            }
          }
        }
      }
    }
    // rotate by 8 columns
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
      double t[8];
#pragma unroll
      for (int c = 0; c < 8; ++c) t[c] = x[r][c];
#pragma unroll
      for (int c = 0; c + 8 < kSlab; ++c) x[r][c] = x[r][c + 8];
#pragma unroll
      for (int c = 0; c < 8; ++c) x[r][kSlab - 8 + c] = t[c];
    }
  }

  if (agree) __syncthreads();
  if (mode_sh == 0) {
    const bool bad = expired_sh != 0;
    if (bad && tid == 0) {
      if (err != nullptr)
        __hip_atomic_fetch_or(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (info != nullptr)
        __hip_atomic_store(info, -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
      const uint32_t row = first + uint32_t(r) * kSlabThreads;
      if (row < m) {
#pragma unroll
        for (int c = 0; c < kSlab; ++c)
          if (c < w) S[row + int64_t(c) * lda] = bad ? __builtin_nan("") : x[r][c];
      }
    }
  }
  if (mode_sh != kTakeSlab) return;
  // The slab by one workgroup, in memory: the same operations column by column.
  if (tid == 0)
    __hip_atomic_store(control + 1, uint64_t(k0) + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  for (int j = 0; j < w; ++j) {
    __syncthreads();
    uint64_t key = 0;
    uint32_t row = 0xFFFFFFFFu;
    for (uint32_t r = uint32_t(j + tid); r < m; r += kSlabThreads) {
      const uint64_t kr = mag_key(fabs(S[r + int64_t(j) * lda]));
      if (kr > key) {
        key = kr;
        row = r;
      }
    }
    wave_argmax<true>(key, row);
    if (lane == 0) {
      skey[0][wave] = key;
      srow[0][wave] = row;
    }
    __syncthreads();
    key = lane < NWAVE ? skey[0][lane] : 0;
    row = lane < NWAVE ? srow[0][lane] : 0xFFFFFFFFu;
    wave_argmax<false>(key, row);
    const uint32_t p = key > 1 ? row : uint32_t(j);
    double *urow = sl;  // the pivot's row
    if (tid == 0) {
      ipiv[k0 + j] = k0 + int64_t(p) + 1;
      if (key == 1 && info != nullptr && *info == 0) *info = int32_t(k0 + j + 1);
    }
    if (tid < w) {
      const double a = S[j + int64_t(tid) * lda], b = S[p + int64_t(tid) * lda];
      if (p != uint32_t(j)) {
        S[j + int64_t(tid) * lda] = b;
        S[p + int64_t(tid) * lda] = a;
      }
      urow[tid] = b;
    }
    __syncthreads();
    const double piv = urow[j];
    for (uint32_t r = uint32_t(j + 1 + tid); r < m; r += kSlabThreads) {
      const double l = S[r + int64_t(j) * lda] / piv;
      S[r + int64_t(j) * lda] = l;
      for (int c = j + 1; c < w; ++c)
        S[r + int64_t(c) * lda] = __builtin_fma(-l, urow[c], S[r + int64_t(c) * lda]);
    }
  }
}

// A sequence of w <= 32 interchanges of rows k + e and p_e touches at most 64
// rows: lane e < 32 of a wavefront stands for row k + e, lane 32 + e for the
// pivot row of step e (if it is not one of the rows k .. k + w - 1 and not an
// earlier lane's). Runs the interchanges on the lanes' row numbers and returns
// whether the lane's row *pos takes another row's entry, that of row *cur.
// p: pivot row of step (lane % 32), any value for steps >= w.
__device__ __forceinline__ bool slab_moves(int64_t k, int w, int64_t p, int64_t *pos,
                                           int64_t *cur) {
  const int lane = threadIdx.x & 63, e = lane & 31;
  const int pe = int(p - k);
  // lane that stands for the pivot row of step e
  int home = 32 + e;
#pragma unroll
  for (int s = kSlab - 1; s >= 0; --s)
    if (s < w && __builtin_amdgcn_readlane(pe, s) == pe) home = 32 + s;
  if (pe >= 0 && pe < w) home = pe;
  if (e >= w) home = e;
  const bool live = e < w && (lane < 32 || home == lane);
  const int at = lane < 32 ? lane : pe;
  int from = at;
#pragma unroll
  for (int s = 0; s < kSlab; ++s) {  // (steps >= w: home = s, nothing moves)
    const int lp = __builtin_amdgcn_readlane(home, s);
    const int a = __builtin_amdgcn_readlane(from, s), b = __builtin_amdgcn_readlane(from, lp);
    from = lane == lp ? a : from;
    from = lane == s ? b : from;
  }
  *pos = k + at;
  *cur = k + from;
  return live && from != at;
}

// The slab's interchanges on every column outside [k0, k0 + w), and the
// publication buffer (count entries) preset for the next slab. Each wavefront
// moves a column with one gather and one scatter: every load of a column
// comes before its stores, so the move is in place. Strided by nature (a
// 64-byte line per entry); kSwapCols columns in flight per wavefront hide its
// latency.
constexpr int kSwapCols = 8;
__global__ void __launch_bounds__(TPB)
    k_gepp_swap(int64_t n, double *__restrict__ A, int64_t lda, int64_t k0, int w,
                const int64_t *__restrict__ ipiv, double *__restrict__ pub, int64_t count) {
  for (int64_t e = int64_t(blockIdx.x) * TPB + threadIdx.x; e < count;
       e += int64_t(gridDim.x) * TPB)
    pub[e] = __builtin_bit_cast(double, kSlabUnpublished);
  const int lane = threadIdx.x & 63;
  const int64_t wave = int64_t(blockIdx.x) * (TPB / 64) + (threadIdx.x >> 6);
  const int64_t cols = n - w;  // columns to move, the slab's own left out
  if (wave * kSwapCols >= cols) return;
  int64_t pos, cur;
  const bool move = slab_moves(k0, w, lane % 32 < w ? ipiv[k0 + lane % 32] - 1 : k0, &pos, &cur);
  double v[kSwapCols];
#pragma unroll
  for (int i = 0; i < kSwapCols; ++i) {
    const int64_t c0 = wave * kSwapCols + i;
    const int64_t c = c0 < k0 ? c0 : c0 + w;
    v[i] = (move && c0 < cols) ? A[cur + c * lda] : 0.0;
  }
  __builtin_amdgcn_wave_barrier();  // every gather before any scatter
#pragma unroll
  for (int i = 0; i < kSwapCols; ++i) {
    const int64_t c0 = wave * kSwapCols + i;
    const int64_t c = c0 < k0 ? c0 : c0 + w;
    if (move && c0 < cols) A[pos + c * lda] = v[i];
  }
}

__global__ void __launch_bounds__(TPB)
    k_slab_reset(double *__restrict__ pub, int64_t count, uint64_t *__restrict__ control) {
  if (blockIdx.x == 0 && threadIdx.x == 0) control[1] = 0;
  for (int64_t e = int64_t(blockIdx.x) * TPB + threadIdx.x; e < count;
       e += int64_t(gridDim.x) * TPB)
    pub[e] = __builtin_bit_cast(double, kSlabUnpublished);
}

// Workgroups that a slab may take: an eighth of the device's CUs (32 of 256).
int slab_max_groups() {
  const int g = device_cus() / 8;
  return g < 1 ? 1 : (g < kSlabGroups ? g : kSlabGroups);
}
// Workgroups of a slab with m rows (0: too many rows for one launch) and the
// rows per thread. Up to 1024 rows one workgroup takes all, with two rows per
// thread if need be: no exchange. Above, the fewest rows per thread that
// `most` workgroups allow (a thread's rows are updated one after another).
int slab_groups(int64_t m, int most, int *rpt) {
  if (m <= kSlabThreads * kSlabMaxRpt) {
    *rpt = m <= kSlabThreads ? 1 : kSlabMaxRpt;
    return 1;
  }
  for (int r = 1; r <= kSlabMaxRpt; ++r) {
    const int64_t g = (m + kSlabThreads * r - 1) / (kSlabThreads * r);
    if (g <= most) {
      *rpt = r;
      return int(g);
    }
  }
  return 0;
}
int64_t slab_pub_doubles(int groups) {
  return groups > 1 ? int64_t(kSlab) * (groups + 1) * kSlot : 0;
}

// perm[i] = original row that ends in row i after the interchanges
// ipiv[0..n) (1-based), applied in order. One workgroup: the interchanges are
// sequential, but each wavefront reduces 32 of them to the moves they amount to
// (slab_moves), kPermWaves slabs at a time, and the first then runs the slabs'
// moves on perm, one gather and one scatter each (one thread took 145 ns for
// each interchange: 580 us at n = 4000, now 49).
constexpr int kPermWaves = 16;
__global__ void __launch_bounds__(64 * kPermWaves)
    k_ipiv_to_perm(int64_t n, const int64_t *__restrict__ ipiv, int64_t *perm) {
  HIP_DYNAMIC_SHARED(int32_t, p_lds)
  __shared__ int64_t mpos[kPermWaves][64], mcur[kPermWaves][64];
  const bool in_lds = n <= kPermLdsMax;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int64_t i = threadIdx.x; i < n; i += 64 * kPermWaves) {
    if (in_lds)
      p_lds[i] = int32_t(i);
    else
      perm[i] = i;
  }
  for (int64_t k0 = 0; k0 < n; k0 += kPermWaves * kSlab) {
    const int64_t k = k0 + wave * kSlab;
    const int64_t left = n - k;
    const int w = left <= 0 ? 0 : int(left < kSlab ? left : kSlab);
    const int e = lane & 31;
    int64_t p = e < w ? ipiv[k + e] - 1 : k;
    if (p < 0 || p >= n) p = k + e;  // no interchange
    int64_t pos, cur;
    const bool move = slab_moves(k, w, p, &pos, &cur);
    mpos[wave][lane] = move ? pos : -1;
    mcur[wave][lane] = cur;
    __syncthreads();
    if (wave == 0) {
      for (int s = 0; s < kPermWaves; ++s) {
        const int64_t q = mpos[s][lane], c = mcur[s][lane];
        if (in_lds) {
          const int32_t v = q >= 0 ? p_lds[c] : 0;
          __builtin_amdgcn_wave_barrier();  // every gather before any scatter
          if (q >= 0) p_lds[q] = v;
          __builtin_amdgcn_wave_barrier();
        } else {
          const int64_t v = q >= 0 ? perm[c] : 0;
          __builtin_amdgcn_wave_barrier();
          if (q >= 0) perm[q] = v;
          __threadfence_block();
        }
      }
    }
    __syncthreads();
  }
  if (in_lds)
    for (int64_t i = threadIdx.x; i < n; i += 64 * kPermWaves) perm[i] = p_lds[i];
}

// Y[i, c] = B[perm[i], c]
__global__ void __launch_bounds__(TPB)
    k_gather_rows(int64_t n, int64_t nrhs, const int64_t *__restrict__ perm,
                  const double *__restrict__ B, int64_t ldb, double *__restrict__ Y,
                  int64_t ldy) {
  const int64_t i = int64_t(blockIdx.x) * TPB + threadIdx.x;
  if (i >= n) return;
  const int64_t r = perm[i];
  for (int64_t c = blockIdx.y; c < nrhs; c += gridDim.y) Y[i + c * ldy] = B[r + c * ldb];
}

}  // namespace

size_t gepp_scratch_bytes() {
  return align256(size_t(kPivotGroups) * sizeof(double)) +
         align256(size_t(kPivotGroups) * sizeof(int64_t));
}

// Workgroups of the largest slab of an n x n matrix that is one launch.
static int largest_slab_groups(int64_t n, int most) {
  const int64_t one = (n + kSlabThreads - 1) / kSlabThreads;  // (one row a thread)
  return one > most ? most : int(one);
}
size_t gepp_slab_bytes(int64_t n) {
  const int64_t count = slab_pub_doubles(largest_slab_groups(n, slab_max_groups()));
  return count == 0 ? 0 : size_t(count + kSlabControl) * sizeof(double);
}

hipError_t launch_gepp(int64_t n, double *A, int64_t lda, int64_t *ipiv, int32_t *info,
                       void *scratch, size_t scratch_bytes, int32_t *err, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  double *pval = static_cast<double *>(scratch);
  int64_t *pidx = reinterpret_cast<int64_t *>(static_cast<char *>(scratch) +
                                              align256(size_t(kPivotGroups) * sizeof(double)));
  double *pub = static_cast<double *>(scratch);
  const bool slabs = scratch_bytes >= gepp_slab_bytes(n);
  const int most = slab_max_groups();
  const int64_t count = slab_pub_doubles(largest_slab_groups(n, most));
  uint64_t *control = reinterpret_cast<uint64_t *>(pub + count);
  const int64_t preset = count == 0 ? 0 : count + 1;  // the buffer and the slab's decision
  bool fresh = false;  // the publication buffer is preset for the next slab
  for (int64_t k0 = 0; k0 < n; k0 += kNB) {
    const int64_t kend = k0 + kNB < n ? k0 + kNB : n;
    const int kb = int(kend - k0);
    for (int64_t k = k0; k < kend; k += kSlab) {
      const int w = int(kend - k < kSlab ? kend - k : kSlab);
      const int64_t m = n - k;
      int rpt = 1;
      const int groups = slabs ? slab_groups(m, most, &rpt) : 0;
      if (groups > 0) {
        if (groups > 1 && !fresh)
          hipLaunchKernelGGL(k_slab_reset, dim3(64), dim3(TPB), 0, s, pub, preset, control);
        const dim3 grid{unsigned(groups)}, block{kSlabThreads};
        const int64_t spin = sweep_spin_limit();
        if (rpt == 1)
          hipLaunchKernelGGL((k_gepp_slab<1>), grid, block, 0, s, n, A, lda, k, w, groups, pub,
                             control, ipiv, info, spin, err);
        else
          hipLaunchKernelGGL((k_gepp_slab<2>), grid, block, 0, s, n, A, lda, k, w, groups, pub,
                             control, ipiv, info, spin, err);
        const int64_t waves = (n - w + kSwapCols - 1) / kSwapCols;
        if (waves > 0) {
          const int64_t grid_swap = (waves + TPB / 64 - 1) / (TPB / 64);
          hipLaunchKernelGGL(k_gepp_swap, dim3(unsigned(grid_swap)), dim3(TPB), 0, s, n, A, lda,
                             k, w, ipiv, pub, preset);
          fresh = true;
        }
      } else {
        for (int64_t j = k; j < k + w; ++j) {
          const int64_t rows = n - j;
          const int pg = int(rows > int64_t(kPivotGroups) * TPB ? kPivotGroups
                                                                : (rows + TPB - 1) / TPB);
          hipLaunchKernelGGL(k_pivot_partial, dim3(unsigned(pg)), dim3(TPB), 0, s, n, A, lda, j,
                             pval, pidx);
          hipLaunchKernelGGL(k_pivot_swap, dim3(1), dim3(TPB), 0, s, n, A, lda, j, pg, pval, pidx,
                             ipiv, info);
          if (rows > 1)
            hipLaunchKernelGGL(k_panel_column, dim3(unsigned((rows - 1 + TPB - 1) / TPB)),
                               dim3(TPB), 0, s, n, A, lda, j, k + w);
        }
        fresh = false;
      }
      const int64_t pc = kend - k - w;  // panel columns right of the slab
      if (pc > 0) {
        hipError_t e = launch_trsm_left(TriMode::LN, w, pc, A + k + k * lda, lda,
                                        A + k + (k + w) * lda, lda, s);
        if (e != hipSuccess) return e;
        e = launch_dgemm(n - k - w, pc, w, A + (k + w) + k * lda, lda, OpA::General,
                         A + k + (k + w) * lda, lda, OpB::General, A + (k + w) + (k + w) * lda,
                         lda, Acc::Subtract, s);
        if (e != hipSuccess) return e;
      }
    }
    const int64_t rest = n - kend;
    if (rest > 0) {
      hipError_t e = launch_trsm_left(TriMode::LN, kb, rest, A + k0 + k0 * lda, lda,
                                      A + k0 + kend * lda, lda, s);
      if (e != hipSuccess) return e;
      e = launch_dgemm(rest, rest, kb, A + kend + k0 * lda, lda, OpA::General,
                       A + k0 + kend * lda, lda, OpB::General, A + kend + kend * lda, lda,
                       Acc::SubtractTrailing, s);
      if (e != hipSuccess) return e;
    }
  }
  return hipGetLastError();
}

hipError_t launch_ipiv_to_perm(int64_t n, const int64_t *ipiv, int64_t *perm, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const size_t lds = n <= kPermLdsMax ? size_t(n) * sizeof(int32_t) : 0;
  hipLaunchKernelGGL(k_ipiv_to_perm, dim3(1), dim3(64 * kPermWaves), lds, s, n, ipiv, perm);
  return hipGetLastError();
}

hipError_t launch_gather_rows(int64_t n, int64_t nrhs, const int64_t *perm, const double *B,
                              int64_t ldb, double *Y, int64_t ldy, hipStream_t s) {
  if (n <= 0 || nrhs <= 0) return hipSuccess;
  const dim3 grid(unsigned((n + TPB - 1) / TPB), unsigned(nrhs < 65535 ? nrhs : 65535));
  hipLaunchKernelGGL(k_gather_rows, grid, dim3(TPB), 0, s, n, nrhs, perm, B, ldb, Y, ldy);
  return hipGetLastError();
}

}  // namespace rbt
