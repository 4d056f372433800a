// The dispatch rules of the GEMM passes behind a C interface, for tests.
#include "pass_rules.hpp"

extern "C" {
int rule_pass(int dtype, int gateup, long long max_rows, long long likely_rows, int G, int ffn, int d,
              int cus) {
  return fs::pass_kind(dtype, gateup, max_rows, likely_rows, G, ffn, d, cus);
}
int rule_pass_fp8(int gateup, long long max_rows, int G, int ffn, int d, int cus) {
  return fs::pass_kind_fp8(gateup, max_rows, G, ffn, d, cus);
}
int rule_dense(int dtype, int m, int n, int kdim, int cus) {
  return fs::dense_kind(dtype, m, n, kdim, cus);
}
}
