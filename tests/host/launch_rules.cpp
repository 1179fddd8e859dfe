// Asks the library's host rules (csrc/gemm_forms.h) in which form launches run; one question a line of standard input:
//   nt PLANES PADDED_N REVERSE ROWS PREFIX SUFFIX   a projection product of one width (rows, of them prefix and suffix spans)
//     -> tile rows, tile columns (0 0: tiles staged through registers), whole, parts
//   tn TILES STEPS                                   a rule-gradient product on one plane -> steps of a workgroup's share
#include <cstdio>
#include <cstring>

#include "gemm_forms.h"

int main() {
  char what[8];
  while (scanf("%7s", what) == 1) {
    if (strcmp(what, "nt") == 0) {
      int planes, Np, reverse, rows, pre, suf;
      if (scanf("%d %d %d %d %d %d", &planes, &Np, &reverse, &rows, &pre, &suf) != 6) return 1;
      const int kt = Np / 32, mid = rows - pre - suf;
      spcfg::NtArgs a{};
      a.planes3 = planes; a.a_bf16 = planes == 1; a.max_wgs = spcfg::kGemmWgs; a.rows = rows;
      a.K = reverse ? 2 * Np : Np; a.cols = reverse ? Np : 2 * Np;
      auto part = [&](int i, int row0, int n, int c0, int kbeg, int steps) {
        a.prt_row0[i] = row0; a.prt_rows[i] = n; a.prt_c0[i] = c0; a.prt_kbeg[i] = kbeg; a.prt_kt[i] = steps;
      };
      if (reverse) {
        a.parts = 3;
        part(0, 0, pre, 0, 0, kt); part(1, pre, mid, 0, 0, 2 * kt); part(2, pre + mid, suf, 0, kt, kt);
      } else if (Np % 128 == 0) {
        a.parts = 2; a.cols = Np;
        part(0, 0, pre + mid, 0, 0, kt); part(1, pre, mid + suf, Np, 0, kt);
      }
      const spcfg::nt::Form f = spcfg::nt::pick_form(a);
      const bool staged = f.shape == spcfg::nt::kStaged;
      printf("%d %d %d %d\n", staged ? 0 : spcfg::nt::kShapes3[f.shape].bm, staged ? 0 : spcfg::nt::kShapes3[f.shape].bn, f.whole,
             f.parts);
    } else {
      int tiles, steps;
      if (strcmp(what, "tn") != 0 || scanf("%d %d", &tiles, &steps) != 2) return 1;
      printf("%d\n", spcfg::nt::tn3_share(1, tiles, steps, spcfg::kGemmWgs));
    }
  }
  return 0;
}
