// Host build of the batched solver's diagonal-block function (k_batched.hip's
// diag_block in FP64, as its FP64 fallback uses it), driven from a file.
//
//   emu_batched_diag IN OUT
// IN (little-endian): int64 n <= 64; then A (n x n, column-major FP64).
// OUT: L\U (n x n), then the inverses (64 x 64: L^-1 below the diagonal, U^-1 on
//   and above; identity beyond n).
#include <cstdio>
#include <vector>

#include "k_batched.hip"

namespace rbt {
int64_t butterfly_granule() { return 1; }
int butterfly_kind() { return 0; }
int butterfly_sides() { return 2; }

namespace {
void one_block(SoloSys *s, double *inv) {
  __shared__ double lds[kR0Doubles + kR1Doubles];
  __shared__ int info;
  if (threadIdx.x == 0) info = 0;
  __syncthreads();
  diag_block<double>(*s, 0, int(s->n), lds, lds + kR0Doubles, inv, &info);
}
}  // namespace
}  // namespace rbt

int main(int argc, char **argv) {
  if (argc != 3) return 2;
  FILE *in = std::fopen(argv[1], "rb");
  FILE *out = std::fopen(argv[2], "wb");
  if (!in || !out) return 2;
  int64_t n = 0;
  if (std::fread(&n, 8, 1, in) != 1 || n < 1 || n > rbt::BB) return 2;
  std::vector<double> F(size_t(n * n)), inv(size_t(rbt::BB * rbt::BB));
  if (std::fread(F.data(), 8, F.size(), in) != F.size()) return 2;
  rbt::SoloSys s{};
  s.n = n;
  s.F64 = F.data();
  rbt::SoloSys *sp = &s;
  double *ip = inv.data();
  hipLaunchKernelGGL(rbt::one_block, dim3(1), dim3(unsigned(rbt::BT)), 0, nullptr, sp, ip);
  std::fwrite(F.data(), 8, F.size(), out);
  std::fwrite(inv.data(), 8, inv.size(), out);
  std::fclose(in);
  std::fclose(out);
  return 0;
}
