// Triangular sweeps for few right-hand sides (groups of 4 to 16) as ONE persistent
// launch per sweep, for the solves after the elimination (Sec. 1, step 3:
// L y = b~, U x~ = y) and the adjoint solves.
//
// Each workgroup takes a ticket (atomic counter) and handles the block row
// of that rank in sweep order: it accumulates op(A)[b, j] x_j over the
// blocks j solved before it, then solves its diagonal block with the
// precomputed inverse (x = Di r; for FP64 factors and FP32 arithmetic one
// more step, x += Di (r - T x), keeps the backward error of substitution) and
// publishes x_b. The matrix entries of the next block are loaded before
// each wait, so the loads overlap it.
//
// Publication: every solution entry carries its own readiness. Before the
// sweep (for up to 8 right-hand sides, before the two of a solve) the launcher, or
// the transform before the solve, fills a publication buffer P (n x nrhs, in the sync
// area) with a signalling-NaN pattern that no arithmetic produces; a
// workgroup publishes x_b by storing its entries into P with agent-scope
// atomic stores (and into B, the output), and a workgroup that needs x_j
// polls its entries of P with agent-scope atomic loads until none holds the
// pattern. One 8-byte entry is written once per sweep and read whole, so a
// read value that is not the pattern is the published one: no fence, no
// counter and no second round trip sit between a block's solution and its
// consumers (the critical path of the sweep is one store and one load per
// block).
//
// Progress: a workgroup only waits for blocks of smaller tickets, which were
// taken by workgroups already running, so every wait ends. The spin is also
// bounded (spin_limit sleeps per entry, the library's option; a negative
// limit expires every wait at once, which tests use to reach this path): a
// workgroup whose wait expires uses NaN for that entry, sets the sticky
// error word sync[3] (which no sweep launch clears), stores NaN as its
// block's solution, so the result can never be a silently wrong finite
// vector, and goes on, so the grid always drains.
//
// Layout: 512 threads = 8 wavefronts of 16 rows each. A wavefront forms whole
// rows of a product of a 128 x 128 block with the x block, so nothing is
// reduced across wavefronts and each of the up to four products on the
// critical path (the last block's, and three with the diagonal block) costs
// one barrier. One right-hand side: a row belongs to a quad of lanes, 32
// columns each, summed over the quad by DPP. More: the matrix cores, a lane
// holding row l % 16 and every fourth group of columns of the block
// (16x16x4 products for groups of 16; for groups of 4 and 8 the 4x4x4 FP64 and
// 4x4x1 FP32 products on four row groups, whose cost goes with the right-hand
// sides: 16 and 8 cycles per four of them against 64 and 32 for sixteen). With
// lanes on 128 rows x 4 segments, FMA loops over x in LDS and a sum over the
// segments through LDS after each product, the step from block to block was
// LDS-bound for several right-hand sides. Microseconds per block then and now
// (FP64, n = 4096, not transposed / transposed): a group of 16 right-hand sides
// 43 / 48 and 12.6, of 8 of them 14.9 / 19.6 and 7.4, of 4 of them 9.0 / 13.7 and
// 4.2 / 4.9, one 5.2 / 7.9 and 3.2 / 3.4 (n = 20000: 5.8 / 10.0 and 4.0).
//
// Columns of a block are dealt to the lanes of a row in pairs (FP64; groups
// of four in FP32): step q = qq V + h takes column qq 4 V + sl V + h in lane
// group sl, so that the transposed modes, where a row is contiguous, read
// 64-byte runs with 16-byte loads.
//
// More right-hand sides than a group takes are several groups in the same
// launch, their tickets interleaved: the groups run side by side, each on its
// own chain, and share the blocks through the caches. group_width() chooses.
//
// Arithmetic type C: FP64 for FP64 factors. For the FP32 factors of the
// mixed-precision solve it is FP32: the right-hand side (FP64 storage, the
// transformed residual) is rounded to FP32 when loaded, the products, the
// diagonal-block inverses (FP32) and the reductions are FP32, and the FP32
// result is stored back widened; FP64 arithmetic with FP64 inverses is kept
// as an option.
#include <type_traits>

#include "internal.h"
#include "mma16.h"

namespace rbt {

namespace {

constexpr int TPB = 512;
constexpr int STEPS = 32;  // columns per lane of a 128-wide block

__device__ __forceinline__ double coherent_load(const double *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void coherent_store(double *p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// (a published entry with this pattern is stored as a quiet NaN)
__device__ __forceinline__ bool unpublished(double v) {
  return __builtin_bit_cast(uint64_t, v) == kUnpublished;
}

// Sums over the four lanes that share a row (the same in all four): a quad,
// or the lanes l, l + 16, l + 32, l + 48.
template <typename C>
__device__ __forceinline__ C quad_sum(C v) {
  const C a = quad_bcast_k<0>(v) + quad_bcast_k<1>(v);
  const C b = quad_bcast_k<2>(v) + quad_bcast_k<3>(v);
  return a + b;
}
// v[l] + v[l ^ 32], v[l] + v[l ^ 16]: swapping halves (rows) of two copies of v
// leaves one half (the even rows) in the first, the other in the second.
template <bool HALVES>
__device__ __forceinline__ uint2 swap_copies(unsigned v) {
  if constexpr (HALVES) {
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return uint2{r[0], r[1]};
  } else {
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return uint2{r[0], r[1]};
  }
}
template <bool HALVES>
__device__ __forceinline__ float add_swapped(float v) {
  const uint2 r = swap_copies<HALVES>(unsigned(__float_as_int(v)));
  return __int_as_float(int(r.x)) + __int_as_float(int(r.y));
}
template <bool HALVES>
__device__ __forceinline__ double add_swapped(double v) {
  const uint2 lo = swap_copies<HALVES>(unsigned(__double2loint(v)));
  const uint2 hi = swap_copies<HALVES>(unsigned(__double2hiint(v)));
  return __hiloint2double(int(hi.x), int(lo.x)) + __hiloint2double(int(hi.y), int(lo.y));
}

// Product of the wavefront's 16 rows of a 128 x 128 block (STEPS entries per
// lane: row rl, columns of lane group sl) with the x block in LDS. NT
// right-hand sides; the result has NV values per lane, value v at row
// row(v), right-hand side col(v). XN: values of x per LDS row.
template <int NT, bool TRANS, typename C>
struct Prod;

// One right-hand side: four lanes per row, such that consecutive lanes read
// consecutive memory: a quad where rows are contiguous (TRANS), else the lanes
// l, l + 16, l + 32, l + 48.
template <bool TRANS, typename C>
struct Prod<1, TRANS, C> {
  static constexpr int NV = 1, XN = 1;
  static __device__ __forceinline__ int rl(int lane) { return TRANS ? lane >> 2 : lane & 15; }
  static __device__ __forceinline__ int sl(int lane) { return TRANS ? lane & 3 : lane >> 4; }
  static __device__ __forceinline__ int row(int lane, int) { return rl(lane); }
  static __device__ __forceinline__ int col(int, int) { return 0; }
  static __device__ __forceinline__ bool owns(int lane) { return sl(lane) == 0; }
  template <int V>
  static __device__ __forceinline__ int slot(int k) { return k; }
  template <int V>
  static __device__ __forceinline__ void mul(const C (&e)[STEPS], const C *xs, int lane,
                                             C (&out)[NV]) {
    const C *x = xs + sl(lane) * V;
    C a[4] = {C(0), C(0), C(0), C(0)};
#pragma unroll
    for (int q = 0; q < STEPS; ++q)
      a[q & 3] = fma_c(e[q], x[(q / V) * 4 * V + q % V], a[q & 3]);
    const C v = (a[0] + a[1]) + (a[2] + a[3]);
    if constexpr (TRANS)
      out[0] = quad_sum(v);
    else
      out[0] = add_swapped<false>(add_swapped<true>(v));
  }
};

// Matrix cores, 16 x 16 x 4. LDS row of column k: the rows of one step's four
// lane groups are neighbours (conflict-free reads); 17 apart.
template <bool TRANS, typename C>
struct Prod<16, TRANS, C> {
  typedef Mma16<C> M;
  static constexpr int NV = 4, XN = 17;
  static __device__ __forceinline__ int rl(int lane) { return lane & 15; }
  static __device__ __forceinline__ int sl(int lane) { return lane >> 4; }
  static __device__ __forceinline__ int row(int lane, int v) { return M::row(lane >> 4, v); }
  static __device__ __forceinline__ int col(int lane, int) { return lane & 15; }
  static __device__ __forceinline__ bool owns(int) { return true; }
  template <int V>
  static __device__ __forceinline__ int slot(int k) {
    return 4 * ((k / (4 * V)) * V + k % V) + (k / V) % 4;
  }
  template <int V>
  static __device__ __forceinline__ void mul(const C (&e)[STEPS], const C *xs, int lane,
                                             C (&out)[NV]) {
    const C *x = xs + (lane >> 4) * XN + (lane & 15);
    typename M::v4 a0 = {C(0), C(0), C(0), C(0)}, a1 = a0;
#pragma unroll
    for (int q = 0; q < STEPS; q += 2) {
      a0 = M::mma(e[q], x[4 * q * XN], a0);
      a1 = M::mma(e[q + 1], x[4 * (q + 1) * XN], a1);
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) out[v] = a0[v] + a1[v];
  }
};

// FP64 matrix cores, 4 x 4 x 4 on four blocks of rows: lane l supplies
// A[row l % 16][l / 16] (as for 16 x 16 x 4) and B[l / 16][l % 4], and holds
// row 4 ((l / 4) % 4) + l / 16, column l % 4 of the result.
template <int NT>
struct Prod4 {
  static constexpr int NV = NT / 4, XN = NT + 1;
  static __device__ __forceinline__ int rl(int lane) { return lane & 15; }
  static __device__ __forceinline__ int sl(int lane) { return lane >> 4; }
  static __device__ __forceinline__ int row(int lane, int) {
    return 4 * ((lane >> 2) & 3) + (lane >> 4);
  }
  static __device__ __forceinline__ int col(int lane, int v) { return 4 * v + (lane & 3); }
  static __device__ __forceinline__ bool owns(int) { return true; }
  template <int V>
  static __device__ __forceinline__ int slot(int k) {
    return 4 * ((k / (4 * V)) * V + k % V) + (k / V) % 4;
  }
  template <int V>
  static __device__ __forceinline__ void mul(const double (&e)[STEPS], const double *xs, int lane,
                                             double (&out)[NV]) {
    constexpr int CH = 4 / NV;  // accumulation chains per column group
    const double *x = xs + (lane >> 4) * XN + (lane & 3);
    double a[NV][CH];
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
      for (int h = 0; h < CH; ++h) a[v][h] = 0.0;
#pragma unroll
    for (int q = 0; q < STEPS; ++q)
#pragma unroll
      for (int v = 0; v < NV; ++v)
        a[v][q % CH] = __builtin_amdgcn_mfma_f64_4x4x4f64(e[q], x[4 * q * XN + 4 * v], a[v][q % CH],
                                                          0, 0, 0);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      out[v] = a[v][0];
#pragma unroll
      for (int h = 1; h < CH; ++h) out[v] += a[v][h];
    }
  }
};
// Sums over the lanes l, l + 16, l + 32, l + 48 of four values, value l / 16 to
// lane l: each swap leaves one half (the even rows) of two values in the first
// result and the other in the second.
__device__ __forceinline__ float sum_and_scatter(float v0, float v1, float v2, float v3) {
  auto bits = [](float v) { return unsigned(__float_as_int(v)); };
  auto sum = [](auto r) { return __int_as_float(int(r[0])) + __int_as_float(int(r[1])); };
  const float s0 = sum(__builtin_amdgcn_permlane32_swap(bits(v0), bits(v2), false, false));
  const float s1 = sum(__builtin_amdgcn_permlane32_swap(bits(v1), bits(v3), false, false));
  return sum(__builtin_amdgcn_permlane16_swap(bits(s0), bits(s1), false, false));
}

// FP32 matrix cores, 4 x 4 x 1 on 16 blocks: four row blocks times four groups
// of columns of the block. Lane l supplies A[row l % 16] and B[column l % 4] of
// the group l / 16; its four results are rows 4 ((l / 4) % 4) + v of the group's
// partial sum, added over the groups at the end (row l / 16 of the four).
template <bool TRANS>
struct Prod<4, TRANS, float> {
  typedef float v4 __attribute__((ext_vector_type(4)));
  static constexpr int NV = 1, XN = 5;
  static __device__ __forceinline__ int rl(int lane) { return lane & 15; }
  static __device__ __forceinline__ int sl(int lane) { return lane >> 4; }
  static __device__ __forceinline__ int row(int lane, int) {
    return 4 * ((lane >> 2) & 3) + (lane >> 4);
  }
  static __device__ __forceinline__ int col(int lane, int) { return lane & 3; }
  static __device__ __forceinline__ bool owns(int) { return true; }
  template <int V>
  static __device__ __forceinline__ int slot(int k) {
    return 4 * ((k / (4 * V)) * V + k % V) + (k / V) % 4;
  }
  template <int V>
  static __device__ __forceinline__ void mul(const float (&e)[STEPS], const float *xs, int lane,
                                             float (&out)[NV]) {
    const float *x = xs + (lane >> 4) * XN + (lane & 3);
    v4 a[4] = {};
#pragma unroll
    for (int q = 0; q < STEPS; ++q)
      a[q & 3] = __builtin_amdgcn_mfma_f32_4x4x1f32(e[q], x[4 * q * XN], a[q & 3], 0, 0, 0);
    const v4 t = (a[0] + a[1]) + (a[2] + a[3]);
    out[0] = sum_and_scatter(t[0], t[1], t[2], t[3]);
  }
};
template <bool TRANS>
struct Prod<4, TRANS, double> : Prod4<4> {};
template <bool TRANS>
struct Prod<8, TRANS, double> : Prod4<8> {};

// The lane's STEPS entries of row m of op(A), columns c0 .. c0 + cb - 1 of the
// block (cb <= 128, FULL: cb = 128; entries beyond are zero).
template <bool FULL, TriMode MODE, int V, typename TF, typename C>
__device__ __forceinline__ void load_block(const TF *A, int64_t ld, int64_t m, int64_t c0, int cb,
                                           int sl, C (&e)[STEPS]) {
  constexpr bool TRANS = MODE == TriMode::UT || MODE == TriMode::LT;
  typedef TF vec __attribute__((ext_vector_type(V), aligned(sizeof(TF))));
  if constexpr (FULL) {
    if constexpr (TRANS) {
      const TF *p = A + c0 + m * ld + sl * V;
      vec w[STEPS / V];
#pragma unroll
      for (int qq = 0; qq < STEPS / V; ++qq) w[qq] = *reinterpret_cast<const vec *>(p + qq * 4 * V);
#pragma unroll
      for (int q = 0; q < STEPS; ++q) e[q] = C(w[q / V][q % V]);
    } else {
      const TF *p = A + m + (c0 + sl * V) * ld;
      TF w[STEPS];
#pragma unroll
      for (int q = 0; q < STEPS; ++q) w[q] = p[int64_t((q / V) * 4 * V + q % V) * ld];
#pragma unroll
      for (int q = 0; q < STEPS; ++q) e[q] = C(w[q]);
    }
    return;
  }
  TF w[STEPS];  // clamped, unconditional loads, masked afterwards
#pragma unroll
  for (int q = 0; q < STEPS; ++q) {
    const int k = (q / V) * 4 * V + sl * V + q % V;
    const int64_t kc = c0 + (k < cb ? k : cb - 1);
    w[q] = TRANS ? A[kc + m * ld] : A[m + kc * ld];
  }
#pragma unroll
  for (int q = 0; q < STEPS; ++q) {
    const int k = (q / V) * 4 * V + sl * V + q % V;
    e[q] = k < cb ? C(w[q]) : C(0);
  }
}

template <int NT, TriMode MODE, typename TF, bool REFINE, typename C>
__global__ void __launch_bounds__(TPB)
    k_sweep(int64_t n, int64_t nrhs, const TF *__restrict__ A, int64_t ld,
            const C *__restrict__ Winv, double *B, int64_t ldb, int32_t *sync, double *P,
            int64_t nb, int groups, int width, int ticket_word, bool keep, int64_t spin_limit,
            const int32_t *gate) {
  // (the gate is read before any ticket is taken: every workgroup of a gated
  // launch returns here)
  if (gated(gate)) return;
  constexpr bool FWD = (MODE == TriMode::LN || MODE == TriMode::UT);
  constexpr bool UNIT = (MODE == TriMode::LN || MODE == TriMode::LT);
  constexpr bool TRANS = (MODE == TriMode::UT || MODE == TriMode::LT);
  typedef Prod<NT, TRANS, C> Pr;
  constexpr int V = 16 / int(sizeof(TF));
  constexpr int NV = Pr::NV, XN = Pr::XN;
  __shared__ __attribute__((aligned(16))) C xs[2][kNB * XN];
  __shared__ int32_t tk;
  __shared__ int expired_sh, nonfinite_sh;

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int sl = Pr::sl(lane);
  const int i = 16 * wave + Pr::rl(lane);  // the lane's row as an operand
  if (tid == 0) {
    tk = atomicAdd(&sync[ticket_word], 1);
    expired_sh = nonfinite_sh = 0;
  }
  for (int e = tid; e < 2 * kNB * XN; e += TPB) xs[0][e] = C(0);  // unused columns stay zero
  __syncthreads();
  const int64_t ticket = __builtin_amdgcn_readfirstlane(tk);  // (block indices in scalar registers)
  if (ticket >= nb * groups) return;
  const int64_t t = ticket / groups;
  const int64_t g0 = (ticket - t * groups) * width;  // the group's first right-hand side
  const int N = int(nrhs - g0 < width ? nrhs - g0 : width);
  B += g0 * ldb;
  double *pub = P + g0 * n;  // entry (row, c) of the group at pub[row N + c]
  int32_t *err = sync + kSweepErrWord;  // sticky: cleared by the entry points, not per sweep
  const int64_t b = FWD ? t : nb - 1 - t;
  const int64_t r0 = b * kNB;
  const int kb = int(n - r0 < kNB ? n - r0 : kNB);
  const int64_t ri = r0 + (i < kb ? i : kb - 1);  // clamped row for loads

  // The diagonal block's inverse, the block itself (masked to its triangle)
  // and the block's right-hand side do not depend on other blocks: they are
  // loaded before any wait and leave the critical path of the sweep.
  C di[STEPS];
  {
    const C *Di = Winv + b * 2 * kNB * kNB + (UNIT ? 0 : kNB * kNB);
    load_block<true, MODE, V, C, C>(Di, int64_t(kNB), int64_t(i), int64_t(0), kNB, sl, di);
#pragma unroll
    for (int q = 0; q < STEPS; ++q) {
      // Di is a full kNB x kNB allocation; entries beyond kb are masked
      const int k = (q / V) * 4 * V + sl * V + q % V;
      di[q] = (i < kb && k < kb) ? di[q] : C(0);
    }
  }
  C td[REFINE ? STEPS : 1];
  if constexpr (REFINE) {
    if (kb == kNB)
      load_block<true, MODE, V, TF, C>(A, ld, ri, r0, kb, sl, td);
    else
      load_block<false, MODE, V, TF, C>(A, ld, ri, r0, kb, sl, td);
#pragma unroll
    for (int q = 0; q < STEPS; ++q) {
      const int k = (q / V) * 4 * V + sl * V + q % V;
      if (k >= kb || i >= kb) td[q] = C(0);
      else if (k == i) td[q] = UNIT ? C(1) : td[q];
      else if (FWD ? (k > i) : (k < i)) td[q] = C(0);
    }
  }
  // the lane's results: rows rv[v] of the block, right-hand sides cv[v]
  int rv[NV], cv[NV];
  bool in[NV];
  C bv[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    rv[v] = 16 * wave + Pr::row(lane, v);
    cv[v] = Pr::col(lane, v);
    in[v] = rv[v] < kb && cv[v] < N;
    bv[v] = in[v] ? C(B[(r0 + rv[v]) + int64_t(cv[v]) * ldb]) : C(0);
  }
  // writes the lane's values into an x block in LDS (zero outside)
  auto to_lds = [&](C *x, const C (&val)[NV]) {
    if (!Pr::owns(lane)) return;
#pragma unroll
    for (int v = 0; v < NV; ++v)
      if (NT == 1 || cv[v] < NT)
        x[Pr::template slot<V>(rv[v]) * XN + cv[v]] = in[v] ? val[v] : C(0);
  };

  // entries of P this thread polls: entry idx of block j sits at
  // P[c0 N + idx], row idx / N, right-hand side idx % N
  constexpr int PER = (kNB * NT + TPB - 1) / TPB;
  int prow[PER], pslot[PER];
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int idx = tid + q * TPB;
    prow[q] = NT == 1 ? idx : idx / N;
    pslot[q] = prow[q] < kNB
                   ? Pr::template slot<V>(prow[q]) * XN + (NT == 1 ? 0 : idx - prow[q] * N)
                   : 0;
  }

  // ---- accumulate op(A)[b, j] x_j over the blocks solved before b ----
  C acc[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) acc[v] = C(0);
  auto block = [&](int64_t s, auto full) {
    const int64_t j = FWD ? s : nb - 1 - s;
    const int64_t c0 = j * kNB;
    const int cb = full.value ? kNB : int(n - c0);
    C e[STEPS];
    load_block<full.value, MODE, V, TF, C>(A, ld, ri, c0, cb, sl, e);
    // x_j from P, each entry polled until published (bounded); a thread's
    // entries are all loaded before any is waited on, so a published block
    // costs one round trip. The two buffers of x alternate: a wavefront still
    // reading the last block's is at most one barrier behind.
    C *x = xs[s & 1];
    const double *pj = pub + c0 * N + tid;
    double xv[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) xv[q] = prow[q] < cb ? coherent_load(pj + q * TPB) : 0.0;
    bool expired = false;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      if (prow[q] >= kNB) continue;
      int64_t spins = 0;
      while (unpublished(xv[q])) {
        if (spins >= spin_limit) {  // expired: NaN for this entry, poison this block
          expired = true;
          xv[q] = __builtin_nan("");
          break;
        }
        __builtin_amdgcn_s_sleep(1);
        ++spins;
        xv[q] = coherent_load(pj + q * TPB);
      }
      x[pslot[q]] = C(xv[q]);
    }
    if (expired) {
      __hip_atomic_fetch_or(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      expired_sh = 1;
    }
    __syncthreads();
    C o[NV];
    Pr::template mul<V>(e, x, lane, o);
#pragma unroll
    for (int v = 0; v < NV; ++v) acc[v] += o[v];
  };
  // only the last block can be partial: the first one that a backward sweep
  // solves (its own step, so that the loop carries no column masks)
  int64_t s0 = 0;
  if (!FWD && t > 0 && n % kNB != 0) {
    block(0, std::false_type{});
    s0 = 1;
  }
  for (int64_t s = s0; s < t; ++s) block(s, std::true_type{});

  // ---- r = b_b - acc, x = Di r (and x += Di (r - T x)) ----
  C r[NV], x[NV];
  C *xa = xs[t & 1], *xb = xs[(t & 1) ^ 1];
#pragma unroll
  for (int v = 0; v < NV; ++v) r[v] = in[v] ? bv[v] - acc[v] : C(0);
  to_lds(xa, r);
  __syncthreads();
  Pr::template mul<V>(di, xa, lane, x);
  // KEEP (with `keep`): a block whose solution is not finite everywhere is solved
  // by substitution (below). Noted before the barriers that are there anyway.
  constexpr bool KEEP = NT > 1 && std::is_same<TF, double>::value;
  auto note = [&](const C (&val)[NV]) {
    if constexpr (KEEP) {
      if (!keep) return;
      bool bad = false;
#pragma unroll
      for (int v = 0; v < NV; ++v) bad = bad || (in[v] && !(fabs(val[v]) < C(INFINITY)));
      if (__any(bad) && lane == 0) nonfinite_sh = 1;
    }
  };
  if constexpr (REFINE) {
    note(x);
    to_lds(xb, x);
    __syncthreads();
    C tx[NV], dx[NV];
    Pr::template mul<V>(td, xb, lane, tx);
#pragma unroll
    for (int v = 0; v < NV; ++v) tx[v] = r[v] - tx[v];
    note(tx);
    to_lds(xa, tx);
    __syncthreads();
    Pr::template mul<V>(di, xa, lane, dx);
#pragma unroll
    for (int v = 0; v < NV; ++v) x[v] += dx[v];
  }
  if constexpr (KEEP) {
    // Products with the inverse make NaN of every entry of the block where the
    // inverse has one Inf or NaN (a zero on the diagonal) or r has (0 * Inf);
    // substitution, which more than kSkinnyMax right-hand sides take without a
    // publication buffer, keeps the entries solved before it. A pivot per barrier,
    // the next one's coefficients in flight.
    if (keep && nonfinite_sh != 0 && expired_sh == 0) {
      constexpr int ROWS = kNB * NT / TPB;  // rows per thread, of right-hand side tid % NT
      const int c = tid % NT, m0 = tid / NT;
      TF tn[ROWS], dn;
      auto load = [&](int jj) {
        const int j = FWD ? jj : kb - 1 - jj;
#pragma unroll
        for (int q = 0; q < ROWS; ++q) {
          const int m = m0 + q * (TPB / NT), mc = m < kb ? m : kb - 1;
          tn[q] = TRANS ? A[(r0 + j) + (r0 + mc) * ld] : A[(r0 + mc) + (r0 + j) * ld];
        }
        dn = A[(r0 + j) + (r0 + j) * ld];
      };
      load(0);
      __syncthreads();  // (every wavefront has read xa)
      to_lds(xa, r);
      for (int jj = 0; jj < kb; ++jj) {
        const int j = FWD ? jj : kb - 1 - jj;
        TF t[ROWS];
#pragma unroll
        for (int q = 0; q < ROWS; ++q) t[q] = tn[q];
        const C rd = UNIT ? C(1) : C(1) / C(dn);
        if (jj + 1 < kb) load(jj + 1);
        __syncthreads();
        const C xj = xa[Pr::template slot<V>(j) * XN + c] * rd;
#pragma unroll
        for (int q = 0; q < ROWS; ++q) {
          const int m = m0 + q * (TPB / NT);
          C *xm = xa + Pr::template slot<V>(m) * XN + c;
          if (m == j)
            xb[Pr::template slot<V>(m) * XN + c] = xj;
          else if (m < kb && (FWD ? m > j : m < j))
            *xm = fma_c(-C(t[q]), xj, *xm);
        }
      }
      __syncthreads();
#pragma unroll
      for (int v = 0; v < NV; ++v)
        if (in[v]) x[v] = xb[Pr::template slot<V>(rv[v]) * XN + cv[v]];
    }
  }

  // ---- publish x_b (NaN if a wait of this block expired): the consumers'
  // copy in P and the output B ----
  const bool poisoned = expired_sh != 0;
  if (Pr::owns(lane)) {
#pragma unroll
    for (int v = 0; v < NV; ++v)
      if (in[v]) {
        const double val = poisoned ? __builtin_nan("") : double(x[v]);
        coherent_store(&pub[(r0 + rv[v]) * N + cv[v]], unpublished(val) ? __builtin_nan("") : val);
      }
#pragma unroll
    for (int v = 0; v < NV; ++v)
      if (in[v])
        B[(r0 + rv[v]) + int64_t(cv[v]) * ldb] = poisoned ? __builtin_nan("") : double(x[v]);
  }
}

// Before a sweep, or the two of a solve: tickets cleared, P (count entries) set
// to the unpublished pattern.
__global__ void k_sweep_reset(int32_t *sync, double *P, int64_t count) {
  SweepPrep{sync, P, count}.run(int64_t(blockIdx.x) * blockDim.x + threadIdx.x,
                                int64_t(gridDim.x) * blockDim.x);
}

template <int NT, TriMode MODE, typename TF, typename C>
hipError_t sweep_t(int64_t n, int64_t nrhs, const TF *LU, int64_t ld, const C *Winv, double *B,
                   int64_t ldb, int32_t *sync, double *P, SweepOf of, hipStream_t s) {
  // one refinement step per diagonal block for FP64 factors and for FP32
  // arithmetic (a product with an explicit FP32 inverse alone is accurate to
  // kappa(block) u32 only); FP64 arithmetic on FP32 factors needs none
  constexpr bool REFINE = std::is_same<TF, double>::value || std::is_same<C, float>::value;
  const int64_t nb = (n + kNB - 1) / kNB;
  const int64_t width = nrhs < NT ? nrhs : NT;  // right-hand sides per group
  const int64_t groups = (nrhs + width - 1) / width;
  if (nb * groups > 0x7fffffff) return hipErrorInvalidValue;
  // the tickets and P; the sticky error word sync[3] is left alone
  const int64_t count = n * nrhs;
  if (of == SweepOf::Alone || of == SweepOf::First) {
    const int64_t entries = of == SweepOf::First ? 2 * count : count;
    const int64_t blocks = (entries + 255) / 256 < 1024 ? (entries + 255) / 256 : 1024;
    hipLaunchKernelGGL(k_sweep_reset, dim3(unsigned(blocks < 1 ? 1 : blocks)), dim3(256), 0, s,
                       sync, P, entries);
  } else if (of == SweepOf::Second) {
    P += count;
  }
  hipLaunchKernelGGL((k_sweep<NT, MODE, TF, REFINE, C>), dim3(unsigned(nb * groups)), dim3(TPB), 0,
                     s, n, nrhs, LU, ld, Winv, B, ldb, sync, P, nb, int(groups),
                     int(width), of == SweepOf::Second ? 1 : 0, nrhs > kSkinnyMax,
                     sweep_spin_limit(), refine_gate());
  return hipGetLastError();
}

template <int NT, typename TF, typename C>
hipError_t sweep_n(TriMode mode, int64_t n, int64_t nrhs, const TF *LU, int64_t ld, const C *Winv,
                   double *B, int64_t ldb, int32_t *sync, double *P, SweepOf of,
                   hipStream_t s) {
  switch (mode) {
    case TriMode::LN: return sweep_t<NT, TriMode::LN>(n, nrhs, LU, ld, Winv, B, ldb, sync, P, of, s);
    case TriMode::UN: return sweep_t<NT, TriMode::UN>(n, nrhs, LU, ld, Winv, B, ldb, sync, P, of, s);
    case TriMode::UT: return sweep_t<NT, TriMode::UT>(n, nrhs, LU, ld, Winv, B, ldb, sync, P, of, s);
    default: return sweep_t<NT, TriMode::LT>(n, nrhs, LU, ld, Winv, B, ldb, sync, P, of, s);
  }
}

// Right-hand sides per group (4, 8 or 16; FP32 arithmetic: 4 or 16). Narrow
// groups have short chains (microseconds per block below, measured at n = 5003 to
// 12000), and each group reads the factors once, at about 7.5 TB/s where many
// groups stream them through the caches. Both directions of one FP64 solve in ms with
// groups of 4 / 8 / 16: n = 1000, 16 right-hand sides 0.12 / 0.16 / 0.24; n = 5003, 64 of
// them 0.61 / 0.80 / 1.07 and 384 of them 2.01 / 1.60 / 1.35; n = 20000, 8 of them 2.25 / 2.62
// (one group), 32 of them 3.72 / 3.65 / 5.09 and 128 of them 12.4 / 7.9 / 5.9. FP32 at
// n = 8191, 8 right-hand sides: a sweep of two groups of 4 0.23, of one of 16 0.42.
template <typename TF, typename C>
int group_width(int64_t n, int64_t nrhs) {
  constexpr bool F32 = std::is_same<C, float>::value;
  constexpr bool REFINE = std::is_same<TF, double>::value || F32;
  const double chain[3] = {F32 ? 3.7 : (REFINE ? 4.7 : 3.0), REFINE ? 7.9 : 4.4,
                           F32 ? 6.6 : (REFINE ? 13.2 : 7.4)};
  const double blocks = double((n + kNB - 1) / kNB);
  const double read = double(n) * double(n) * sizeof(TF) / 2 / 7.5e6;
  int best = 4;
  double least = 0.0;
  for (int k = 0; k < 3; ++k) {
    const int w = 4 << k;
    if (w == 8 && F32) continue;
    const double cost = blocks * chain[k] + double((nrhs + w - 1) / w) * read;
    if (k == 0 || cost < least) {
      best = w;
      least = cost;
    }
  }
  return best;
}

template <typename TF, typename C>
hipError_t sweep_any(TriMode mode, int64_t n, int64_t nrhs, const TF *LU, int64_t ld,
                     const C *Winv, double *B, int64_t ldb, int32_t *sync, double *P,
                     SweepOf of, hipStream_t s) {
  if (n <= 0 || nrhs <= 0) return hipSuccess;
  if (sync == nullptr) return hipErrorInvalidValue;
  if (P != nullptr || nrhs > kSweepPairMax) of = SweepOf::Alone;  // room for one only
  if (P == nullptr) {
    if (nrhs > kSkinnyMax) return hipErrorInvalidValue;
    P = reinterpret_cast<double *>(sync + kSyncPubOffsetInts);
  }
  if (nrhs == 1) return sweep_n<1>(mode, n, nrhs, LU, ld, Winv, B, ldb, sync, P, of, s);
  switch (group_width<TF, C>(n, nrhs)) {
    case 4: return sweep_n<4>(mode, n, nrhs, LU, ld, Winv, B, ldb, sync, P, of, s);
    case 8:
      if constexpr (std::is_same<C, double>::value)
        return sweep_n<8>(mode, n, nrhs, LU, ld, Winv, B, ldb, sync, P, of, s);
      [[fallthrough]];
    default: return sweep_n<16>(mode, n, nrhs, LU, ld, Winv, B, ldb, sync, P, of, s);
  }
}

}  // namespace

hipError_t launch_sweep(TriMode mode, int64_t n, int64_t nrhs, const double *LU, int64_t ld,
                        const double *Winv, double *B, int64_t ldb, int32_t *sync,
                        hipStream_t s, double *pub, SweepOf of) {
  return sweep_any(mode, n, nrhs, LU, ld, Winv, B, ldb, sync, pub, of, s);
}
hipError_t launch_sweep(TriMode mode, int64_t n, int64_t nrhs, const float *LU, int64_t ld,
                        const double *Winv, double *B, int64_t ldb, int32_t *sync,
                        hipStream_t s, double *pub, SweepOf of) {
  return sweep_any(mode, n, nrhs, LU, ld, Winv, B, ldb, sync, pub, of, s);
}
hipError_t launch_sweep(TriMode mode, int64_t n, int64_t nrhs, const float *LU, int64_t ld,
                        const float *Winv, double *B, int64_t ldb, int32_t *sync,
                        hipStream_t s, double *pub, SweepOf of) {
  return sweep_any(mode, n, nrhs, LU, ld, Winv, B, ldb, sync, pub, of, s);
}

}  // namespace rbt
