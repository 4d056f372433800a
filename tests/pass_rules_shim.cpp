// The dispatch and tile rules of the GEMM passes behind a C interface, for tests.
#include "pass_rules.hpp"
#include "tall_tiles.hpp"

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
int rule_height(long long rows, int G, int n_tiles, int cus, int unit) {
  return fs::r192_height(rows, G, n_tiles, cus, unit);
}
int tall_height(int rows, int t192, int t160, int t128, int nn, int wgs) {
  return fs::tall_height(rows, t192, t160, t128, nn, wgs);
}
int tall_rows(int rows, int tiles, int unit) { return fs::tall_rows(rows, tiles, unit); }
// m-tile and n-tile of every item of a group of `tiles` m-tiles and nn n-tiles
void tall_order(int tiles, int nn, int* mt, int* nt) {
  for (int i = 0; i < tiles * nn; ++i) fs::tall_order(i, tiles, nn, mt[i], nt[i]);
}
}
