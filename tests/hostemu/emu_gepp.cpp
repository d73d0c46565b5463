// Host build of the elimination with partial pivoting (k_gepp.hip, with the left
// solves of k_trsm.hip) for tests, driven from a file; the matrix-core GEMM is a
// plain loop here.
//
//   emu_gepp IN OUT
// IN (little-endian): int64 n, spin limit; then A (n x n, column-major FP64).
// OUT: L\\U; int64 ipiv[n]; int64 perm[n]; int32 info; int32 err.
// EMU_THREADS: workgroups that run at once; with fewer than a slab has, the others
// start only when those have left.
#include <cstdio>
#include <vector>

#include "internal.h"

namespace {
int64_t g_limit = 0;
}

namespace rbt {
int64_t sweep_spin_limit() { return g_limit; }
int device_cus() { return 256; }
hipError_t launch_dgemm(int64_t M, int64_t N, int64_t K, const double *A, int64_t lda, OpA,
                        const double *B, int64_t ldb, OpB, double *C, int64_t ldc, Acc,
                        hipStream_t) {
  for (int64_t j = 0; j < N; ++j)
    for (int64_t k = 0; k < K; ++k)
      for (int64_t i = 0; i < M; ++i) C[i + j * ldc] -= A[i + k * lda] * B[k + j * ldb];
  return hipSuccess;
}
}  // namespace rbt

int main(int argc, char **argv) {
  if (argc != 3) return 2;
  FILE *in = std::fopen(argv[1], "rb");
  FILE *out = std::fopen(argv[2], "wb");
  if (!in || !out) return 2;
  int64_t h[2];
  if (std::fread(h, 8, 2, in) != 2) return 2;
  const int64_t n = h[0];
  g_limit = h[1];
  std::vector<double> A(size_t(n * n));
  if (std::fread(A.data(), 8, A.size(), in) != A.size()) return 2;
  std::vector<int64_t> ipiv(size_t(n), -1), perm(size_t(n), -1);
  int32_t info = 0, err = 0;
  const size_t need = rbt::gepp_slab_bytes(n);
  const size_t bytes = need > rbt::gepp_scratch_bytes() ? need : rbt::gepp_scratch_bytes();
  std::vector<double> work(bytes / sizeof(double));
  hipError_t e = rbt::launch_gepp(n, A.data(), n, ipiv.data(), &info, work.data(), bytes, &err, nullptr);
  if (e == hipSuccess) e = rbt::launch_ipiv_to_perm(n, ipiv.data(), perm.data(), nullptr);
  if (e != hipSuccess) return 3;
  std::fwrite(A.data(), 8, A.size(), out);
  std::fwrite(ipiv.data(), 8, ipiv.size(), out);
  std::fwrite(perm.data(), 8, perm.size(), out);
  std::fwrite(&info, 4, 1, out);
  std::fwrite(&err, 4, 1, out);
  std::fclose(in);
  std::fclose(out);
  return 0;
}
