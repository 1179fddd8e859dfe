// Kernel launchers replaced by stubs: lets the host side of the library (argument checks, workspace layout, span
// plan, the width-synchronous schedule of both passes) run under AddressSanitizer / UBSan without a GPU.  The stubs check what the
// real launchers rely on: the panels that a product reads were packed, the sums of every width are taken once and before the
// product that reads them, operand planes end on whole steps, a launch of product and sums lies within its kernel's limits.
#include <cstdio>
#include <set>

#include "spcfg_internal.h"

#define REQUIRE(cond) do { if (!(cond)) { printf("stub launcher, line %d: %s\n", __LINE__, #cond); fflush(stdout); __builtin_trap(); } } while (0)

namespace spcfg {
static long g_launches = 0, g_steps = 0;
static std::set<const void*> g_packed;                        // panels that the call has packed
static int g_fwd[kMaxLen + 2], g_bwd[kMaxLen + 2];            // how often the sums of a width were taken
static Layout g_ly;
long stub_launch_count() { return g_launches; }
long stub_step_count() { return g_steps; }
void launch_plan(const Layout& ly, const Ptrs&, const LenArg&, hipStream_t) {
  ++g_launches;
  g_ly = ly;
  g_packed.clear();
  for (int& x : g_fwd) x = 0;
}
void launch_plan_sentrows(const Layout&, const Ptrs&, hipStream_t) { ++g_launches; }
void launch_pack_weights(const Layout&, const Ptrs& p, const float* L, const float* R, hipStream_t) {
  ++g_launches;
  REQUIRE(L != nullptr && R != nullptr);
  for (const void* w : {(const void*)p.Wn, (const void*)p.Wp, (const void*)p.Wtn, (const void*)p.Wtp, (const void*)p.Wn3,
                        (const void*)p.Wp3, (const void*)p.Wtn3, (const void*)p.Wtp3})
    if (w) g_packed.insert(w);
}
void launch_leaf_prep(const Layout&, const Ptrs&, const float*, bool, hipStream_t) { ++g_launches; }
void launch_split_fwd(const Layout&, const Ptrs&, int w, int64_t, int64_t, bool, hipStream_t) { ++g_launches; ++g_fwd[w]; }
void launch_root_fwd(const Layout& ly, const Ptrs&, const float*, float*, hipStream_t) {
  ++g_launches;
  for (int w = 2; w <= ly.n_long; ++w) REQUIRE(g_fwd[w] == 1);
}
void launch_root_bwd(const Layout&, const Ptrs&, const float*, const float*, float*, int, hipStream_t) {
  ++g_launches;
  for (int& x : g_bwd) x = 0;
}
void launch_split_bwd(const Layout&, const Ptrs&, int w, int64_t, int64_t, bool, hipStream_t) { ++g_launches; ++g_bwd[w]; }
void launch_zero_pad_emit(const Layout&, const Ptrs&, float*, hipStream_t) { ++g_launches; }
void launch_span_marginals(const Layout&, const Ptrs&, float*, int32_t*, hipStream_t) { ++g_launches; }
void launch_gemm_nt(const NtArgs& a, hipStream_t) {
  for (int p = 0; p < a.parts; ++p)
    REQUIRE(a.prt_row0[p] >= 0 && a.prt_rows[p] >= 0 && a.prt_row0[p] + a.prt_rows[p] <= a.rows);
  REQUIRE(a.rows > 0 && a.cols > 0 && a.K % (a.planes3 == 1 || a.b_bf16 ? 64 : 32) == 0);
  REQUIRE(g_packed.count(a.planes3 >= 2 && gemm_nt_reads_planes(a) ? a.Bm3 : a.Bm) == 1);
  if (a.step) {
    const StepArgs& s = *a.step;
    ++g_steps;
    REQUIRE(!gemm_nt_reads_planes(a) && !a.a_bf16 && !a.b_bf16 && a.fp32_mfma == 0 && s.Bm == a.Bm && s.K == a.K && s.K % 32 == 0);
    REQUIRE(s.w >= 1 && s.w <= s.n_long && s.n_long == g_ly.n_long && s.Np == g_ly.Np && s.Pp == g_ly.Pp && s.B == g_ly.B);
    REQUIRE(s.stride == (g_ly.n_max + 1) * s.B && s.Np % step_nonterminals(s.tall) == 0 && (s.forward || !s.tall));
    // bands: terms of the widths from w0 on (forward), of parents below w0 (reverse)
    const int next = s.forward ? s.w + 1 : s.w - 1;
    REQUIRE(next >= 1 && next <= s.n_long);
    REQUIRE(s.w0 == 0 || s.w0 == next / kBandW * kBandW + (s.forward ? 0 : kBandW));
    REQUIRE(s.w0 == 0 || (s.forward ? s.w0 < next && s.w0 >= 2 * kBandW : s.w0 > next));
    // one workgroup a CU, and few without work; sentences in the third dimension of the grid
    const int64_t tiles = (int64_t)s.B * ((s.n_long + step_spans(s.tall)) / step_spans(s.tall)) * (s.Np / step_nonterminals(s.tall));
    REQUIRE(s.B <= 65535 && tiles <= 4096);
    REQUIRE((s.UVb != nullptr) == (g_ly.tn3 != 0) && (s.UVb == nullptr || s.planes == g_ly.planes_bwd));
    REQUIRE((s.b_stride != 0) == (g_ly.G > 1));
    ++(s.forward ? g_fwd : g_bwd)[next];
  }
  ++g_launches;
}
static void all_parents_summed() {
  for (int w = 1; w <= g_ly.n_long && w < g_ly.n_max; ++w) REQUIRE(g_bwd[w] == 1);
}
void launch_gemm_tn(const TnArgs&, hipStream_t) { ++g_launches; all_parents_summed(); }
void launch_gemm_tn3(const Tn3Args& a, hipStream_t) {
  REQUIRE(a.KT > 0 && a.planes == g_ly.tn3);
  all_parents_summed();
  ++g_launches;
}
// (the product reads whole steps: 32 rows of three planes, 64 of one)
void launch_scaled_planes(const float*, int64_t, const float*, int64_t S, int64_t Srows, void*, int64_t plane_stride, hipStream_t) {
  REQUIRE(Srows >= S && Srows % (plane_stride ? 32 : 64) == 0);
  ++g_launches;
}
void launch_zero_plane_rows(void*, int64_t plane_stride, int64_t ld, int64_t row0, int64_t rows, hipStream_t) {
  REQUIRE(rows == (plane_stride ? 32 : 64) && (row0 + rows) * ld <= g_ly.uvb_plane);
  ++g_launches;
}
bool gemm_nt_keep_parts(NtArgs& a) { return a.parts != 0; }
bool gemm_nt_reads_planes(const NtArgs& a) { return a.planes3 != 0 && !a.grouped && (a.planes3 <= 2 || a.rows >= 380); }
int gemm_nt_tiles(int rows, int cols) { return ((rows + 31) / 32) * ((cols + 127) / 128); }
size_t gemm_nt_partial_bytes(int max_wgs) { return (size_t)2 * max_wgs * 128 * 128 * 4; }
}  // namespace spcfg
