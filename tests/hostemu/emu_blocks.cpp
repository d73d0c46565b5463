// Host build of the elimination's block kernels for tests (k_getrf.hip,
// k_trsm.hip), driven from a file.
//
//   emu_blocks IN OUT
// IN (little-endian): int64 op, m, n, lda, ldb; then A (lda x m) and B
//   (ldb x n), column-major, in the operation's storage type.
//   op 0, 1, 2: diagonal block of order m, in FP64, FP32, and FP32 storage with
//     FP64 arithmetic; A -> L\U.
//   op 10 + mode, 20 + mode: left solve with A (m x m, FP64 / FP32) of the n
//     columns of B; mode: LN, UN, UT, LT in the order of TriMode.
//   op 30, 31: panel solves (FP64 / FP32): rows B (n x m, ldb) <- B U^-1, and
//     the n columns C (m x n, m) <- L^-1 C, read after B.
//   op 40: inverses of the diagonal blocks of A (order m, FP64).
// OUT: A, then B, then C (or the inverses); int32 info.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "internal.h"

namespace {

template <typename T>
T *rd(FILE *f, size_t n) {
  T *p = static_cast<T *>(std::malloc(n * sizeof(T) + 1));
  if (n && std::fread(p, sizeof(T), n, f) != n) {
    std::fprintf(stderr, "emu_blocks: short input\n");
    std::exit(2);
  }
  return p;
}

template <typename T>
int run(FILE *in, FILE *out, const int64_t *h) {
  const int64_t op = h[0], m = h[1], n = h[2], lda = h[3], ldb = h[4];
  T *A = rd<T>(in, size_t(lda * m));
  const size_t nb = op >= 30 && op < 40 ? size_t(ldb * m) : size_t(ldb * n);
  T *B = rd<T>(in, nb);
  size_t nc = 0;
  T *C = nullptr;
  int32_t info = 0;
  hipError_t e = hipSuccess;
  constexpr bool F64 = sizeof(T) == 8;
  if (op <= 2) {
    if constexpr (F64)
      e = rbt::launch_diag_lu(int(m), A, lda, 0, &info, nullptr);
    else
      e = rbt::launch_diag_lu(int(m), A, lda, 0, &info, op == 2, nullptr);
  } else if (op < 30) {
    const rbt::TriMode mode = rbt::TriMode(op % 10);
    if constexpr (F64)
      e = rbt::launch_trsm_left(mode, int(m), n, A, lda, B, ldb, nullptr);
    else
      e = rbt::launch_trsm_left(mode, int(m), n, A, lda, B, ldb, false, nullptr);
  } else if (op < 40) {
    // (one leading dimension for both: the block and its right neighbours)
    nc = size_t(ldb * n);
    C = rd<T>(in, nc);
    if constexpr (F64)
      e = rbt::launch_panel_trsm(int(m), n, n, A, lda, B, C, ldb, nullptr);
    else
      e = rbt::launch_panel_trsm(int(m), n, n, A, lda, B, C, ldb, false, nullptr);
  } else {
    if constexpr (F64) {
      nc = size_t(rbt::diag_inv_doubles(m));
      C = static_cast<T *>(std::calloc(nc, sizeof(T)));
      e = rbt::launch_diag_inverses(m, A, lda, C, nullptr);
    }
  }
  if (e != hipSuccess) return 3;
  std::fwrite(A, sizeof(T), size_t(lda * m), out);
  std::fwrite(B, sizeof(T), nb, out);
  if (nc) std::fwrite(C, sizeof(T), nc, out);
  std::fwrite(&info, sizeof(info), 1, out);
  std::free(A);
  std::free(B);
  std::free(C);
  return 0;
}

}  // namespace

int main(int argc, char **argv) {
  if (argc != 3) return 2;
  FILE *in = std::fopen(argv[1], "rb");
  FILE *out = std::fopen(argv[2], "wb");
  if (!in || !out) return 2;
  int64_t h[5];
  if (std::fread(h, 8, 5, in) != 5) return 2;
  const int64_t op = h[0];
  const bool f32 = op == 1 || op == 2 || (op >= 20 && op < 30) || op == 31;
  const int rc = f32 ? run<float>(in, out, h) : run<double>(in, out, h);
  std::fclose(in);
  std::fclose(out);
  return rc;
}
