// Build step: writes the header of reference 1D coefficients used as
// compile-time constants by the operator kernels.
//
// On a uniform mesh with the default penalty gamma = k(k+1) applied as
// gamma / h, the rows of the periodic classes of the global 1D matrices
// (Sec. 4: mass M, stiffness L, and B with its point terms) scale exactly
// with the mesh size: M = h M^, L = L^ / h, B = B^ / h^3.  The header holds
// M^, L^, B^ of the periodic rows (cell position p = 0..k-1, offsets
// -2k..2k) for k = 2..7, printed as hexadecimal floating-point literals so
// that they are the float64 values computed by the set-up code.
//
// Near the boundary the rows of M and L are the periodic rows with the
// entries of boundary and outside nodes dropped.  Those of B differ further
// in the first (and last) cell only, by the point term at the boundary
// (one-sided mean with full weight): bl holds rows 1..k of B on columns
// 1..3k, and db[i - 1][j - 1] = B(i, j) - B^(i, j), i, j = 1..k; the last
// cell's are their mirror images.
//
// pt is the embedding table of the transfers (set-up's prolongation_table).
//
// Usage: gen_refcoef <output header>
#include <cmath>
#include <cstdio>
#include <vector>

#include "setup.h"

int main(int argc, char** argv) {
  if (argc != 2) {
    std::fprintf(stderr, "usage: %s <output header>\n", argv[0]);
    return 2;
  }
  std::FILE* f = std::fopen(argv[1], "w");
  if (!f) return 1;
  std::fprintf(f,
               "// Generated by gen_refcoef.cpp at build time: reference (h = 1) rows of the\n"
               "// periodic classes of M, L, B for gamma = k(k+1), [p][2k + offset].\n"
               "#pragma once\n\nnamespace c0ip {\ntemplate <int K> struct RefCoef;\n");
  const int N = 16;  // any mesh with periodic rows; the rows are scaled back to h = 1
  for (int k = 2; k <= 7; ++k) {
    const c0ip::Level1D lv = c0ip::build_level_1d(k, N, k * (k + 1.0));
    const c0ip::RowClasses rc = c0ip::row_classes(lv);
    if (!rc.periodic) return 1;
    const double h = lv.h;
    const double scale[3] = {1.0 / h, h, h * h * h};
    const c0ip::Band* mats[3] = {&lv.M, &lv.L, &lv.B};
    const char* names[3] = {"m", "l", "b"};
    std::fprintf(f, "template <> struct RefCoef<%d> {\n", k);
    for (int m = 0; m < 3; ++m) {
      std::fprintf(f, "  static constexpr double %s[%d][%d] = {\n", names[m], k, 4 * k + 1);
      for (int p = 0; p < k; ++p) {
        const int row = rc.row_of_class[2 * rc.left + p];
        std::fprintf(f, "      {");
        for (int o = -2 * k; o <= 2 * k; ++o) {
          const int j = row + o;
          const double v = (j < 0 || j >= lv.n1) ? 0.0 : mats[m]->get(row, j) * scale[m];
          std::fprintf(f, "%s%a", o == -2 * k ? "" : ", ", v);
        }
        std::fprintf(f, "}%s\n", p + 1 < k ? "," : "");
      }
      std::fprintf(f, "  };\n");
    }
    // every near-boundary row must be the periodic row plus db
    std::fprintf(f, "  static constexpr double db[%d][%d] = {\n", k, k);
    for (int i = 1; i <= 2 * k; ++i) {
      const int row = rc.row_of_class[2 * rc.left + i % k];
      if (i <= k) std::fprintf(f, "      {");
      for (int j = 1; j < lv.n1 - 1; ++j) {
        const int o = j - i;
        if (o < -2 * k || o > 2 * k) continue;
        for (int m = 0; m < 3; ++m) {
          const double d = (mats[m]->get(i, j) - mats[m]->get(row, row + o)) * scale[m];
          const double mirror =
              (mats[m]->get(lv.n1 - 1 - i, lv.n1 - 1 - j) - mats[m]->get(i, j)) * scale[m];
          const double tol = 1e-10 * std::fabs(mats[m]->get(row, row) * scale[m]);
          if (!(std::fabs(mirror) <= tol)) return 1;
          if (m == 2 && i <= k && j <= k)
            std::fprintf(f, "%s%a", j == 1 ? "" : ", ", d);
          else if (!(std::fabs(d) <= tol))
            return 1;
        }
      }
      if (i <= k) std::fprintf(f, "}%s\n", i < k ? "," : "");
    }
    std::fprintf(f, "  };\n");
    std::fprintf(f, "  static constexpr double bl[%d][%d] = {\n", k, 3 * k);
    for (int i = 1; i <= k; ++i) {
      std::fprintf(f, "      {");
      for (int j = 1; j <= 3 * k; ++j)
        std::fprintf(f, "%s%a", j == 1 ? "" : ", ", j - i <= 2 * k ? lv.B.get(i, j) * scale[2] : 0.0);
      std::fprintf(f, "}%s\n", i < k ? "," : "");
    }
    std::fprintf(f, "  };\n");
    // embedding table: value of coarse-cell basis a at position p of fine cell 2 cc + s
    const std::vector<double> pt = c0ip::prolongation_table(k);
    std::fprintf(f, "  static constexpr double pt[2][%d][%d] = {\n", k, k + 1);
    for (int s = 0; s < 2; ++s)
      for (int p = 0; p < k; ++p) {
        std::fprintf(f, "      %s{", p == 0 ? "{" : "");
        for (int a = 0; a <= k; ++a)
          std::fprintf(f, "%s%a", a == 0 ? "" : ", ", pt[(size_t)(s * k + p) * (k + 1) + a]);
        std::fprintf(f, "}%s\n", p + 1 < k ? "," : s == 0 ? "}," : "}");
      }
    std::fprintf(f, "  };\n");
    std::fprintf(f, "};\n");
  }
  std::fprintf(f, "}  // namespace c0ip\n");
  return std::fclose(f) == 0 ? 0 : 1;
}
