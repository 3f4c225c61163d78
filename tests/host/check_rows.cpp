// CPU check of what the real-space plane pass and the row kernels index with
// (paper_2506_21908_amd/csrc/nct_tables.hpp), built with AddressSanitizer and
// UndefinedBehaviorSanitizer by tests/test_host_rows.py: pmap and rnext lead from every grid point to
// exactly the sphere rows that lie on it, in atom order and without cycles, and to none elsewhere; and the grids
// that stride over the rows cover them within the launch limits.  Prints "ok <cases>" and returns 0, or
// names the first failure.
#include <cstdio>
#include <random>
#include <vector>

#include "../../paper_2506_21908_amd/csrc/nct_tables.hpp"

namespace {

int g_fail = 0;

std::vector<nct_channel> kb18() {
  return {{0, 1, 1.0, 0.7}, {1, 1, 0.45, 0.7}, {1, 3, 0.525, 0.7}, {2, 3, -0.375, 0.7}, {2, 5, -0.25, 0.7}};
}

bool check_case(const int n[3], const double cell[3], const std::vector<double>& pos, double rs) {
  nct::tables::ProjectorTables t;
  const auto ch = kb18();
  const std::string why = nct::tables::build_projector_tables(n, cell, int(pos.size() / 3), pos.data(), int(ch.size()),
                                                              ch.data(), rs, t);
  if (!why.empty()) return std::printf("FAIL: builder refused: %s\n", why.c_str()), false;
  const size_t NYZ = size_t(n[1]) * n[2], N = n[0] * NYZ;
  if (t.pmap.size() != N || t.rnext.size() != size_t(t.Jtot)) return std::printf("FAIL: sizes\n"), false;
  std::vector<char> seen(t.Jtot, 0);
  int multi = 0;
  for (size_t p = 0; p < N; ++p) {
    int prev = -1, len = 0;
    for (int J = t.pmap[p]; J >= 0; J = t.rnext[J]) {
      if (J >= t.Jtot) return std::printf("FAIL: point %zu leads to row %d of %d\n", p, J, t.Jtot), false;
      if (J <= prev) return std::printf("FAIL: chain of point %zu not in row order\n", p), false;
      if (size_t(t.ix_of_row[J]) * NYZ + t.pidx[J] != p) return std::printf("FAIL: row %d is not on point %zu\n", J, p), false;
      if (seen[J]++) return std::printf("FAIL: row %d reached twice\n", J), false;
      prev = J;
      ++len;
    }
    multi += len > 1;
  }
  for (int J = 0; J < t.Jtot; ++J)
    if (!seen[J]) return std::printf("FAIL: row %d not reached\n", J), false;
  std::printf("  %d rows, %d points with several\n", t.Jtot, multi);
  return true;
}

}  // namespace

int main() {
  int cases = 0;
  struct C { int n[3]; double L[3]; int atoms; double rs; };
  const C list[] = {{{8, 8, 8}, {6.0, 6.0, 6.0}, 1, 2.5},    {{12, 16, 12}, {6.0, 8.0, 6.0}, 3, 2.5},
                    {{16, 12, 16}, {8.0, 6.0, 8.0}, 8, 2.9}, {{24, 24, 24}, {12.0, 12.0, 12.0}, 20, 5.9},
                    {{8, 12, 16}, {6.0, 7.0, 9.0}, 40, 0.3}, {{32, 32, 32}, {13.44, 13.44, 13.44}, 2, 2.5}};
  for (const C& c : list) {
    std::mt19937_64 g(c.atoms);
    std::uniform_real_distribution<double> u(-1.0, 2.0);
    std::vector<double> pos;
    for (int a = 0; a < c.atoms; ++a)
      for (int d = 0; d < 3; ++d) pos.push_back(u(g) * c.L[d]);
    pos.push_back(0.0), pos.push_back(0.0), pos.push_back(0.0);  // the corner, twice
    pos.push_back(0.0), pos.push_back(0.0), pos.push_back(0.0);
    if (!check_case(c.n, c.L, pos, c.rs)) ++g_fail;
    ++cases;
  }
  for (const int J : {1, 255, 256, 257, 16776959, 16776960, 16776961, 1 << 30}) {
    const unsigned nb = nct::tables::row_blocks(J, 256);
    if (nb < 1 || nb > nct::tables::kMaxGridY) std::printf("FAIL: %u blocks for %d rows\n", nb, J), ++g_fail;
    // the last row belongs to a block of the first stride in which it lies; no index leaves int
    const long long stride = 256LL * nb, trips = (J + stride - 1) / stride;
    if (trips * stride < J || (trips + 1) * stride > 2147483647LL) std::printf("FAIL: stride over %d rows\n", J), ++g_fail;
    ++cases;
  }
  if (g_fail) return 1;
  std::printf("ok %d\n", cases);
  return 0;
}
