// C ABI of libspcfg: argument checks, workspace layout, the width-synchronous schedule (Sec. 3.2,
// span-level parallelism: one launch handles every span of one width across the batch) and optional
// per-kernel-class timing with HIP events.
#include <cstdio>
#include <atomic>
#include <cstring>
#include <mutex>
#include <vector>

#include "spcfg_internal.h"

namespace spcfg {

namespace {

thread_local char g_hip_err[256] = "";
thread_local const char* g_refused = nullptr;  // set by a launcher that refused to launch

struct Plan {            // host-side copy of the span schedule
  std::vector<int64_t> off;   // off[w] = first row of width w (1-based), off[n_max+1] = Sall
  std::vector<int64_t> cnt;   // cnt[w] = number of spans of width w
  LenArg lens;
};

// When a band of widths pays (choose_bands): bytes of row reads saved, less kBandTables for every tile and value of s (its
// tables take eleven dependent lookups, whatever N is), against what another dependent launch costs.  Fitted to 930 forward and
// 1082 reverse bands timed with and without, N = 64 .. 2048, B = 8 .. 960, n = 36 .. 100: with this rule no batch's split sums take more
// than 2.3 % longer than without bands.  With 50 MB and no charge for the tables, which is right for N >= 512, batches of small
// grammars lost up to 17 % (B = 128, N = 128, n = 10 .. 60 forward: 568 us without bands, 662 us with, 562 us by this rule;
// B = 960, N = 64, n <= 40 reverse: 893, 1007 and 893 us); from kBandManyWaves wavefronts on (N = 2048, B = 64) 50 MB pay.
constexpr double kBandTables = 3072;
constexpr double kBandBytes = 100e6, kBandBytesMany = 50e6;
constexpr int64_t kBandManyWaves = 16384;
// Long chains of few spans are latency, not bytes: from this many split points (parents) on they pay while the band has fewer
// wavefronts than kBandFewWaves in the form with 64 nonterminals a wavefront.
constexpr int kBandChain = 48;
constexpr int64_t kBandFewWaves = 768;

size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

int check_cfg(const spcfg_config* c) {
  if (!c || c->struct_size != sizeof(spcfg_config)) return SPCFG_ERR_ARG;
  if (c->N < 1 || c->P < 1 || c->N > (1 << 16) || c->P > (1 << 16)) return SPCFG_ERR_SHAPE;
  if (c->max_B < 1 || c->max_B > kMaxB || c->max_n < 2 || c->max_n > kMaxLen) return SPCFG_ERR_SHAPE;
  if (c->precision != SPCFG_PRECISION_FP32 && c->precision != SPCFG_PRECISION_BF16) return SPCFG_ERR_UNSUPPORTED;
  if (c->flags & ~(uint32_t)(SPCFG_FLAG_ACCUMULATE_GRADS | SPCFG_FLAG_PER_SENTENCE_GRAMMAR | SPCFG_FLAG_FP32_MFMA |
                              SPCFG_FLAG_BF16_SINGLE_FORWARD)) return SPCFG_ERR_UNSUPPORTED;
  return SPCFG_OK;
}

// Byte layout of the workspace for a batch with S1 leaf rows and S2 rows of width >= 2.
Layout make_layout(int N, int P, int B, int n_max, int64_t S1, int64_t S2, int bf16, int per_sentence, int fp32_mfma,
                   int bf16_single, int gemm_wgs = kGemmWgs) {
  Layout ly{};
  ly.gemm_wgs = gemm_wgs;
  // Operand planes for the projection products.  fp32 mode with a shared grammar: the exact three-piece cut, forward
  // and reverse (the products then never cut operands themselves).  bf16 mode with a shared grammar: two pieces
  // (hi + lo) for the forward products, which decide log Z, the plain bf16 rounding for the reverse ones; with one
  // grammar per sentence the forward products run on fp32 operands instead (the grouped kernel cuts them itself; there
  // is no grouped kernel on planes), the reverse ones on one plane; one plane both ways when the caller asks for single
  // bf16 operands.
  const bool shared = !(per_sentence && B > 1);
  ly.fwd_fp32 = bf16 && !shared && !bf16_single;
  ly.planes = bf16 ? (bf16_single ? 1 : (shared ? 2 : 0)) : (!shared || fp32_mfma ? 0 : 3);
  ly.planes_bwd = bf16 ? 1 : ly.planes;
  ly.N = N; ly.P = P; ly.B = B; ly.n_max = n_max; ly.bf16 = bf16;
  ly.G = per_sentence ? B : 1;
  ly.Np = round_up(N, kPad);
  ly.Pp = round_up(P, kPad);
  ly.S1 = S1; ly.S2 = S2; ly.Sall = S1 + S2;
  size_t o = 0;
  auto take = [&](size_t bytes) { size_t at = o; o = align_up(o + bytes); return at; };
  const size_t i4 = sizeof(int32_t), f4 = sizeof(float);
  ly.lens = take(i4 * B);
  ly.rowbase = take(i4 * 3 * (size_t)(n_max + 1) * B);  // three tables, see the span plan kernel
  ly.rootrow = take(i4 * B);
  ly.ztil = take(f4 * B);
  ly.rmax = take(f4 * B);
  ly.row_b = take(i4 * ly.Sall);
  ly.row_i = take(i4 * ly.Sall);
  ly.rootmask = take(i4 * ly.Sall);
  ly.mexp = take(i4 * ly.Sall);
  ly.uexp = take(i4 * ly.Sall);
  ly.tmaxb = take(i4 * ly.Sall);
  ly.umaxb = take(i4 * ly.Sall);
  ly.hmaxb = take(i4 * ly.Sall);
  ly.zmaxb = take(i4 * ly.Sall);
  ly.colmax = take(f4 * 2 * (size_t)(ly.Np + ly.Pp) * ly.G);
  ly.gsc = take(f4 * ly.Sall);
  ly.xs = take(f4 * S1);
  // One arrival counter per output tile of the largest launch: at most max(S1, S2) rows (one width; grouped
  // launches round every sentence's rows up to whole row tiles, at most one extra tile per sentence) and
  // max(2Np, Pp) columns (the projections write 2Np columns, the leaf reverse product P of them).  A launch cut
  // into up to three row ranges rounds each of them up to whole row tiles: two extra tiles of 32 rows (also with
  // the per-sentence flag when the batch is a single sentence: that runs as a shared grammar).
  ly.n_counters = gemm_nt_tiles((int)(S1 > S2 ? S1 : S2) + 64 + (per_sentence ? 32 * B : 0),
                                2 * ly.Np > ly.Pp ? 2 * ly.Np : ly.Pp);
  {  // the bf16 rule-gradient product has 2Np rows and up to max(Np, Pp) columns
    const int g = (2 * ly.Np / 128 + 1) * ((ly.Np > ly.Pp ? ly.Np : ly.Pp) / 128 + 1);
    if (g > ly.n_counters) ly.n_counters = g;
  }
  ly.counters = take(i4 * (size_t)ly.n_counters);
  ly.partial = take(gemm_nt_partial_bytes(gemm_wgs));
  const size_t w4 = bf16 ? 2 : 4;  // bytes per packed weight
  const size_t w4f = (bf16 && !ly.fwd_fp32) ? 2 : 4;  // ... of the forward panels
  ly.Wn = take(w4f * 2 * (size_t)ly.Np * ly.Np * ly.G);
  ly.Wp = take(w4f * 2 * (size_t)ly.Np * ly.Pp * ly.G);
  ly.Wtn = take(w4 * 2 * (size_t)ly.Np * ly.Np * ly.G);
  ly.Wtp = take(w4 * 2 * (size_t)ly.Np * ly.Pp * ly.G);
  if (ly.planes >= 2) {
    ly.Wn3 = take(2 * (size_t)ly.planes * 2 * ly.Np * ly.Np); ly.Wp3 = take(2 * (size_t)ly.planes * 2 * ly.Np * ly.Pp);
  }
  if (ly.planes_bwd == 3) {
    ly.Wtn3 = take(6 * 2 * (size_t)ly.Np * ly.Np); ly.Wtp3 = take(6 * 2 * (size_t)ly.Np * ly.Pp);
  }
  if (per_sentence) { ly.sentrows = take(i4 * (size_t)S2); ly.sentoff = take(i4 * (size_t)B); }
  if (ly.planes > 0) {
    ly.Tb = take(2 * (size_t)ly.planes * S2 * ly.Np);
    ly.leafEb = take(2 * (size_t)ly.planes * S1 * ly.Pp);
  }
  // rule gradients on planes (shared grammar): the adjoint planes get the zeroed rows of a step behind the last row (the
  // product reads whole steps), and the scaled inside vectors get planes of their own, padded to whole steps
  ly.tn3 = shared ? ly.planes_bwd : 0;
  const int64_t step = ly.tn3 ? kTn3Rows(ly.tn3) : 1;
  ly.S1p = (S1 + step - 1) / step * step; ly.S2p = (S2 + step - 1) / step * step;
  ly.uvb_plane = (ly.Sall + (ly.tn3 ? step : 0)) * 2 * ly.Np;
  if (ly.planes_bwd > 0) ly.UVb = take(2 * (size_t)ly.planes_bwd * ly.uvb_plane);
  if (ly.tn3) {
    ly.Tg3 = take(2 * ly.tn3 * (size_t)ly.S2p * ly.Np);
    ly.Eg3 = take(2 * ly.tn3 * (size_t)ly.S1p * ly.Pp);
  }
  ly.leafE = take(f4 * (size_t)S1 * ly.Pp);
  ly.T = take(f4 * (size_t)S2 * ly.Np);
  ly.BH = take(f4 * (size_t)S2 * ly.Np);
  ly.HZ = take(f4 * (size_t)ly.Sall * 2 * ly.Np);
  ly.UV = take(f4 * (size_t)ly.Sall * 2 * ly.Np);
  ly.total = o;
  return ly;
}

Ptrs resolve(const Layout& ly, void* ws) {
  unsigned char* b = static_cast<unsigned char*>(ws);
  Ptrs p;
  p.lens = (int32_t*)(b + ly.lens); p.rowbase = (int32_t*)(b + ly.rowbase); p.rootrow = (int32_t*)(b + ly.rootrow);
  p.row_b = (int32_t*)(b + ly.row_b); p.row_i = (int32_t*)(b + ly.row_i); p.rootmask = (int32_t*)(b + ly.rootmask);
  p.mexp = (int32_t*)(b + ly.mexp); p.uexp = (int32_t*)(b + ly.uexp);
  p.tmaxb = (uint32_t*)(b + ly.tmaxb); p.umaxb = (uint32_t*)(b + ly.umaxb);
  p.hmaxb = (int32_t*)(b + ly.hmaxb); p.zmaxb = (int32_t*)(b + ly.zmaxb); p.colmax = (float*)(b + ly.colmax);
  p.gsc = (float*)(b + ly.gsc); p.xs = (float*)(b + ly.xs);
  p.ztil = (float*)(b + ly.ztil); p.rmax = (float*)(b + ly.rmax);
  p.leafE = (float*)(b + ly.leafE); p.T = (float*)(b + ly.T); p.HZ = (float*)(b + ly.HZ);
  p.UV = (float*)(b + ly.UV); p.BH = (float*)(b + ly.BH);
  p.partial = (float*)(b + ly.partial); p.counters = (int32_t*)(b + ly.counters);
  p.sentrows = (int32_t*)(b + ly.sentrows); p.sentoff = (int32_t*)(b + ly.sentoff);
  p.Tb = ly.planes ? b + ly.Tb : nullptr; p.UVb = ly.planes_bwd ? b + ly.UVb : nullptr; p.leafEb = ly.planes ? b + ly.leafEb : nullptr;
  p.Tg3 = b + ly.Tg3; p.Eg3 = b + ly.Eg3;
  p.Wn3 = b + ly.Wn3; p.Wp3 = b + ly.Wp3; p.Wtn3 = b + ly.Wtn3; p.Wtp3 = b + ly.Wtp3;
  p.Wn = (float*)(b + ly.Wn); p.Wp = (float*)(b + ly.Wp); p.Wtn = (float*)(b + ly.Wtn); p.Wtp = (float*)(b + ly.Wtp);
  return p;
}

// Which bands of widths sum together (k_split_band_fwd / _bwd).  A band saves rows read (of Np floats) and costs a launch
// of its own, the partial sums' rows written and read, rows read for spans that a tile lacks, and its tables; counted exactly
// here, per tile of four starts.
void choose_bands(const Plan& plan, Layout* ly) {
  ly->n_long = 2;
  for (int b = 0; b < ly->B; ++b) ly->n_long = plan.lens.v[b] > ly->n_long ? plan.lens.v[b] : ly->n_long;
  for (int k = 0; k * kBandW < ly->n_long; ++k) {
    const int w0 = k * kBandW, wt = w0 + kBandW;
    double fwd = 0, bwd = 0;              // rows saved
    double fwd_steps = 0, bwd_steps = 0;  // values of s, over all tiles
    for (int b = 0; b < ly->B; ++b) {
      const int n = plan.lens.v[b];
      if (n < w0 || n < 2) continue;
      const int tiles = (n - w0 + kBandI) / kBandI;
      ly->band_tiles[k] += tiles;
      fwd_steps += (double)tiles * (w0 + 2);
      bwd_steps += (double)tiles * (n - w0);
      for (int w = w0 > 0 ? w0 : 1; w < wt && w <= n; ++w) {
        const double spans = n - w + 1;
        fwd += spans * (2.0 * (w - 1) - 4.0 * (w - w0) - 2.0);
        const int near = wt - 1 - w < n - w ? wt - 1 - w : n - w;  // parents inside the band, at most, on either side
        bwd += spans * (2.0 * (n - w) - 4.0 * near - 4.0);
      }
    }
    fwd -= (kBandI + kBandQ) * fwd_steps;
    bwd -= (kBandI + kBandQ) * bwd_steps;
    const int64_t waves = (int64_t)ly->band_tiles[k] * (ly->Np / 64);
    auto pays = [&](double rows, double steps, int64_t launch_waves, bool chain) {
      return 4.0 * ly->Np * rows - kBandTables * steps >= (launch_waves >= kBandManyWaves ? kBandBytesMany : kBandBytes) ||
             (chain && launch_waves < kBandFewWaves);
    };
    // (below width 8 most split points have a child inside the band)
    ly->band_fwd[k] = w0 >= 2 * kBandW && pays(fwd, fwd_steps, waves, w0 >= kBandChain);
    ly->band_bwd[k] = pays(bwd, bwd_steps, 2 * waves, ly->n_long - w0 >= kBandChain);
  }
}

// Bytes of chart rows (N floats) that the split launches of a width read and write, for the profile: two rows a term and
// the sum's own row; with a band the terms inside it, the partial sum read and written once more, and at its first launch
// eleven rows for every tile and value of s.  (Rows that tiles have in common are counted for each: they may come from a cache.)
double split_fwd_bytes(const Plan& plan, const Layout& ly, int w) {
  const bool band = ly.band_fwd[w / kBandW] != 0;
  const int w0 = w / kBandW * kBandW;
  double rows = 0;
  for (int b = 0; b < ly.B; ++b) {
    const int n = plan.lens.v[b];
    if (n < w) continue;
    rows += (n - w + 1) * (band ? 4.0 * (w - w0) + 2.0 : 2.0 * (w - 1) + 1.0);
    if (!band || w != w0) continue;
    for (int i0 = 0; i0 + w0 <= n; i0 += kBandI) {
      const int last = i0 + kBandI + w0 - 2 < n - 1 ? i0 + kBandI + w0 - 2 : n - 1;
      rows += (double)(kBandI + kBandQ) * (last > i0 ? last - i0 : 0);
    }
    for (int v = w0; v < w0 + kBandW && v <= n; ++v) rows += n - v + 1;
  }
  return 4.0 * ly.N * rows;
}
double split_bwd_bytes(const Plan& plan, const Layout& ly, int w) {
  const bool band = ly.band_bwd[w / kBandW] != 0;
  const int w0 = w / kBandW * kBandW, wt = w0 + kBandW;
  double rows = 0;
  for (int b = 0; b < ly.B; ++b) {
    const int n = plan.lens.v[b];
    if (n > w) {  // (a root has no parents and no sums)
      const int most = band ? wt - 1 - w : n;
      for (int i = 0; i <= n - w; ++i) rows += 2.0 * ((n - w - i < most ? n - w - i : most) + (i < most ? i : most));
      rows += (band ? 4.0 : 2.0) * (n - w + 1);
    }
    if (!band || w != band_top(ly, w0)) continue;
    for (int i0 = 0; i0 + w0 <= n; i0 += kBandI)
      rows += (double)(kBandI + kBandQ) * ((n - i0 - wt >= 0 ? n - i0 - wt + 1 : 0) + i0 + kBandI - 1);
    for (int v = w0 > 0 ? w0 : 1; v < wt && v < n; ++v) rows += 2.0 * (n - v + 1);
  }
  return 4.0 * ly.N * rows;
}

int make_plan(const spcfg_config* cfg, const int32_t* lengths, int B, int n_max, Plan* plan, Layout* ly,
              int gemm_wgs = kGemmWgs) {
  if (!lengths) return SPCFG_ERR_ARG;
  if (B < 1 || B > cfg->max_B || n_max < 2 || n_max > cfg->max_n) return SPCFG_ERR_SHAPE;
  for (int b = 0; b < B; ++b)
    if (lengths[b] < 2 || lengths[b] > n_max) return SPCFG_ERR_LENGTH;
  plan->off.assign(n_max + 2, 0);
  plan->cnt.assign(n_max + 2, 0);
  for (int b = 0; b < B; ++b) {
    plan->lens.v[b] = lengths[b];
    for (int w = 1; w <= lengths[b]; ++w) plan->cnt[w] += lengths[b] - w + 1;
  }
  int64_t run = 0;
  for (int w = 1; w <= n_max + 1; ++w) {
    plan->off[w] = run;
    if (w <= n_max) run += plan->cnt[w];
  }
  const int64_t S1 = plan->cnt[1], Sall = run;
  if (Sall >= (int64_t)1 << 30) return SPCFG_ERR_SHAPE;
  *ly = make_layout(cfg->N, cfg->P, B, n_max, S1, Sall - S1, cfg->precision == SPCFG_PRECISION_BF16,
                    (cfg->flags & SPCFG_FLAG_PER_SENTENCE_GRAMMAR) != 0, (cfg->flags & SPCFG_FLAG_FP32_MFMA) != 0,
                    (cfg->flags & SPCFG_FLAG_BF16_SINGLE_FORWARD) != 0, gemm_wgs);
  choose_bands(*plan, ly);
  return SPCFG_OK;
}

// ---- profiling -------------------------------------------------------------------------------------
// A Scope names the kernel class of the launches made during its lifetime; every such launch gets its own
// start/stop event pair (see launch_k), so a class's time is the sum of its kernels' own durations.
// The counters are process-wide; a mutex guards them, and the class that a thread's launches are charged to is that
// thread's own, so concurrent callers do not corrupt the records (their launches simply add up).
// A launch of two classes at once (a product together with the sums that wait for it) counts in both and is charged to
// each with half its time; what comes from such launches is kept apart as well (spcfg_profile_read_shared).
thread_local int t_cur_cls = -1, t_cur_also = -1;
struct Prof {
  std::atomic<bool> on{false};
  std::mutex mu;
  struct Rec { hipEvent_t a, b; int cls, also; };
  std::vector<Rec> recs;
  std::vector<hipEvent_t> pool;
  struct Sums {
    double ms[SPCFG_PROF_CLASSES] = {0}, work[SPCFG_PROF_CLASSES] = {0};
    int64_t launches[SPCFG_PROF_CLASSES] = {0};
  };
  Sums all, shared;  // (ms: filled when the events are read)
  Sums last_shared;  // of the last spcfg_profile_read
  hipEvent_t get() {
    if (!pool.empty()) { hipEvent_t e = pool.back(); pool.pop_back(); return e; }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
  }
  void recycle() {
    for (auto& r : recs) { pool.push_back(r.a); pool.push_back(r.b); }
    recs.clear();
  }
} g_prof;

struct Scope {
  int prev, prev_also;
  Scope(int c, double work, int also = -1, double also_work = 0.0) : prev(t_cur_cls), prev_also(t_cur_also) {
    if (!g_prof.on) return;
    t_cur_cls = c;
    t_cur_also = also;
    std::lock_guard<std::mutex> lock(g_prof.mu);
    g_prof.all.work[c] += work;
    if (also < 0) return;
    g_prof.all.work[also] += also_work;
    g_prof.shared.work[c] += work;
    g_prof.shared.work[also] += also_work;
  }
  ~Scope() { t_cur_cls = prev; t_cur_also = prev_also; }
};

}  // namespace

void launch_refused(const char* what) { g_refused = what; }

LaunchEvents prof_launch_events() {
  LaunchEvents ev;
  if (!g_prof.on || t_cur_cls < 0) return ev;
  std::lock_guard<std::mutex> lock(g_prof.mu);
  ++g_prof.all.launches[t_cur_cls];
  if (t_cur_also >= 0) {
    ++g_prof.all.launches[t_cur_also];
    ++g_prof.shared.launches[t_cur_cls];
    ++g_prof.shared.launches[t_cur_also];
  }
  ev.start = g_prof.get();
  ev.stop = g_prof.get();
  if (!ev.start || !ev.stop) {
    if (ev.start) g_prof.pool.push_back(ev.start);
    if (ev.stop) g_prof.pool.push_back(ev.stop);
    return LaunchEvents{};
  }
  g_prof.recs.push_back({ev.start, ev.stop, t_cur_cls, t_cur_also});
  return ev;
}

namespace {

int hip_status() {
  if (g_refused) {
    snprintf(g_hip_err, sizeof(g_hip_err), "%s", g_refused);
    g_refused = nullptr;
    (void)hipGetLastError();
    return SPCFG_ERR_WORKSPACE;
  }
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) return SPCFG_OK;
  snprintf(g_hip_err, sizeof(g_hip_err), "%s", hipGetErrorString(e));
  return SPCFG_ERR_HIP;
}

int check_ws(const Layout& ly, void* ws, size_t bytes) {
  if (!ws) return SPCFG_ERR_ARG;
  if (((uintptr_t)ws & 255) != 0 || bytes < ly.total) return SPCFG_ERR_WORKSPACE;
  return SPCFG_OK;
}

// Shared grammar, fp32, width >= 2: the rows of a width are ordered [prefix spans | middle spans | suffix spans]
// (a span that is both, i.e. a root, counts as prefix).  A prefix span is never a right child and a suffix span
// never a left child, so one of their two projections (forward) resp. one half of their adjoint (reverse, it
// is zero) takes no part: the launch is cut into parts that leave those products out.
struct WidthBlocks { int nP, nM, nS; };
WidthBlocks width_blocks(const Plan& plan, const Layout& ly, int w) {
  WidthBlocks k{0, 0, 0};
  for (int b = 0; b < ly.B; ++b) {
    const int cnt = plan.lens.v[b] - w + 1;
    if (cnt >= 1) ++k.nP;
    if (cnt >= 2) ++k.nS;
    if (cnt >= 3) k.nM += cnt - 2;
  }
  return k;
}
bool use_parts(const Layout& ly, int w) { return ly.G == 1 && w >= 2; }
void set_part(NtArgs& a, int i, int row0, int rows, int c0, int kbeg, int kt) {
  a.prt_row0[i] = row0; a.prt_rows[i] = rows; a.prt_c0[i] = c0; a.prt_kbeg[i] = kbeg; a.prt_kt[i] = kt;
}

// One grammar per sentence: the launch for width w multiplies each sentence's rows with that sentence's panel.
void set_groups(NtArgs& a, const Plan& plan, const Layout& ly, const Ptrs& p, int w, int64_t row0, int64_t b_stride) {
  if (ly.G == 1) return;
  a.grouped = 1; a.ngroups = ly.B; a.grp_w = w;
  a.grp_lens = p.lens; a.grp_rowbase = p.rowbase + (size_t)w * ly.B; a.grp_row_first = row0; a.grp_b_stride = b_stride;
  a.grp_tiles_m[0] = a.grp_tiles_m[1] = a.grp_tiles_m[2] = 0;
  a.grp_max_rows = 0;
  for (int b = 0; b < ly.B; ++b) {
    const int cnt = plan.lens.v[b] - w + 1;
    if (cnt <= 0) continue;
    a.grp_tiles_m[0] += (cnt + 31) / 32; a.grp_tiles_m[1] += (cnt + 63) / 64; a.grp_tiles_m[2] += (cnt + 127) / 128;
    if (cnt > a.grp_max_rows) a.grp_max_rows = cnt;
  }
}

// The forward product of width w: [eta | zeta] = [L;R] * inside vectors (width 1: [L_P ; R_P] * emission vectors).
// *skipped: flop of the projections that the launch leaves out (w >= 2).
NtArgs forward_product(const Plan& plan, const Layout& ly, const Ptrs& p, int fp32_mfma, int w, double* skipped) {
  const int64_t Np = ly.Np, Pp = ly.Pp;
  NtArgs a{};
  if (w == 1) {
    a.partial = p.partial; a.counters = p.counters; a.max_wgs = ly.gemm_wgs; a.n_counters = ly.n_counters; a.b_bf16 = ly.bf16 && !ly.fwd_fp32; a.fp32_mfma = fp32_mfma;
    a.A = p.leafE; a.lda = Pp; a.Bm = p.Wp; a.ldb = Pp; a.C = p.HZ; a.ldc = 2 * Np;
    if (ly.bf16 && !ly.fwd_fp32) { a.A = p.leafEb; a.a_bf16 = 1; }
    if (ly.planes >= 2) {
      a.A3 = p.leafEb; a.Bm3 = p.Wp3; a.planes3 = ly.planes; a.a_plane = ly.S1 * Pp; a.b_plane = 2 * Np * Pp;
      a.a_bf16 = 0; a.b_bf16 = 0;
    } else if (ly.planes == 1 && ly.G == 1) {
      a.A3 = a.A; a.Bm3 = a.Bm; a.planes3 = 1; a.b_bf16 = 0;
    }
    a.rows = (int)ly.S1; a.cols = (int)(2 * Np); a.K = (int)Pp;
    a.epilogue = NT_EPI_ROWSCALE; a.rowmaxb = p.tmaxb;
    set_groups(a, plan, ly, p, 1, 0, 2 * Np * Pp);
    return a;
  }
  const int64_t row0 = plan.off[w], rows = plan.cnt[w];
  a.partial = p.partial; a.counters = p.counters; a.max_wgs = ly.gemm_wgs; a.n_counters = ly.n_counters; a.b_bf16 = ly.bf16 && !ly.fwd_fp32; a.fp32_mfma = fp32_mfma;
  a.A = p.T + (row0 - ly.S1) * Np; a.lda = Np; a.Bm = p.Wn; a.ldb = Np;
  if (ly.bf16 && !ly.fwd_fp32) { a.A = static_cast<const uint16_t*>(p.Tb) + (row0 - ly.S1) * Np; a.a_bf16 = 1; }
  if (ly.planes >= 2) {
    a.A3 = static_cast<const uint16_t*>(p.Tb) + (row0 - ly.S1) * Np; a.Bm3 = p.Wn3;
    a.planes3 = ly.planes; a.a_plane = ly.S2 * Np; a.b_plane = 2 * Np * Np;
    a.a_bf16 = 0; a.b_bf16 = 0;
  } else if (ly.planes == 1 && ly.G == 1) {
    a.A3 = a.A; a.Bm3 = a.Bm; a.planes3 = 1; a.b_bf16 = 0;
  }
  a.C = p.HZ + row0 * 2 * Np; a.ldc = 2 * Np;
  a.rows = (int)rows; a.cols = (int)(2 * Np); a.K = (int)Np;
  a.epilogue = NT_EPI_ROWSCALE; a.rowmaxb = p.tmaxb + row0;
  // eta for the prefix and middle rows, zeta for the middle and suffix rows (when Np is not a whole number of
  // 128-column tiles the two column blocks would each pad their last tile: one product of 2Np columns then)
  if (use_parts(ly, w) && Np % 128 == 0) {
    const WidthBlocks k = width_blocks(plan, ly, w);
    const int kt = (int)(Np / 32);
    a.parts = 2; a.cols = (int)Np;
    set_part(a, 0, 0, k.nP + k.nM, 0, 0, kt);
    set_part(a, 1, k.nP, k.nM + k.nS, (int)Np, 0, kt);
    // the profile counts the executed flop: one of the two projections is left out for k.nP + k.nS rows
    if (gemm_nt_keep_parts(a)) *skipped = 2.0 * ly.N * (double)ly.N * (k.nP + k.nS);
  }
  set_groups(a, plan, ly, p, w, row0, 2 * Np * Np);
  return a;
}

// The reverse product of width w; *flop: what it executes.
NtArgs reverse_product(const Plan& plan, const Layout& ly, const Ptrs& p, int fp32_mfma, int w, float* grad_log_emit,
                       double* flop) {
  const int64_t Np = ly.Np, Pp = ly.Pp, row0 = plan.off[w], rows = plan.cnt[w];
  NtArgs a{};
  a.partial = p.partial; a.counters = p.counters; a.max_wgs = ly.gemm_wgs; a.n_counters = ly.n_counters; a.b_bf16 = ly.bf16; a.fp32_mfma = fp32_mfma;
  a.A = p.UV + row0 * 2 * Np; a.lda = 2 * Np; a.K = (int)(2 * Np); a.rows = (int)rows;
  if (ly.bf16) { a.A = static_cast<const uint16_t*>(p.UVb) + row0 * 2 * Np; a.a_bf16 = 1; }
  if (ly.planes_bwd == 3) {
    a.A3 = static_cast<const uint16_t*>(p.UVb) + row0 * 2 * Np; a.Bm3 = w >= 2 ? p.Wtn3 : p.Wtp3;
    a.planes3 = 3; a.a_plane = ly.uvb_plane; a.b_plane = 2 * Np * (w >= 2 ? Np : Pp);
  }
  a.Bm = w >= 2 ? p.Wtn : p.Wtp;
  if (ly.bf16 && ly.G == 1) { a.A3 = a.A; a.Bm3 = a.Bm; a.planes3 = 1; a.b_bf16 = 0; }
  if (w >= 2) {
    *flop = 4.0 * ly.N * (double)ly.N * rows;
    a.ldb = 2 * Np; a.C = p.BH + (row0 - ly.S1) * Np; a.ldc = Np; a.cols = (int)Np;
    a.epilogue = NT_EPI_MASKROWS; a.rowmask = p.rootmask + row0; a.rowmaxb = p.umaxb + row0;
    if (use_parts(ly, w)) {  // prefix rows: only the eta adjoint (first half of K); suffix rows: only zeta's
      const WidthBlocks k = width_blocks(plan, ly, w);
      const int kt = (int)(Np / 32);
      a.parts = 3;
      set_part(a, 0, 0, k.nP, 0, 0, kt);
      set_part(a, 1, k.nP, k.nM, 0, 0, 2 * kt);
      set_part(a, 2, k.nP + k.nM, k.nS, 0, kt, kt);
      // (the profile counts the executed flop)
      if (gemm_nt_keep_parts(a)) *flop -= 2.0 * ly.N * (double)ly.N * (k.nP + k.nS);
    }
    set_groups(a, plan, ly, p, w, row0, 2 * Np * Np);
  } else {
    *flop = 4.0 * ly.N * (double)ly.P * rows;
    a.ldb = 2 * Np; a.C = grad_log_emit; a.ldc = ly.P; a.cols = ly.P;
    a.epilogue = NT_EPI_LEAF_EMIT; a.E = p.leafE; a.lde = Pp; a.rowexp = p.uexp;
    a.row_b = p.row_b; a.row_i = p.row_i; a.n_max = ly.n_max;
    set_groups(a, plan, ly, p, 1, 0, 2 * Np * Pp);
  }
  return a;
}

// Where the weight packing writes: the panels that some product of the pass reads, null for the others.  A panel of
// N = P = 2048 takes 33 MB as fp32 and 50 MB as planes: scoring needs none of the reverse ones, and launches that all have few
// rows no planes (scoring one sentence of 40 words: 700 -> 631 us, 64 treebank sentences 3044 -> 2985 us).
Ptrs panels_read(const Plan& plan, const Layout& ly, const Ptrs& p, int fp32_mfma, bool fwd, bool bwd) {
  Ptrs q = p;
  q.Wn = q.Wp = q.Wtn = q.Wtp = nullptr;
  q.Wn3 = q.Wp3 = q.Wtn3 = q.Wtp3 = nullptr;
  double flop;
  auto use = [](const NtArgs& a, float* W, void* W3, float** to, void** to3) {
    if (a.planes3 >= 2 && gemm_nt_reads_planes(a)) *to3 = W3;
    else *to = W;
  };
  if (fwd) use(forward_product(plan, ly, p, fp32_mfma, 1, &flop), p.Wp, p.Wp3, &q.Wp, &q.Wp3);
  if (bwd) use(reverse_product(plan, ly, p, fp32_mfma, 1, nullptr, &flop), p.Wtp, p.Wtp3, &q.Wtp, &q.Wtp3);
  bool f = fwd, r = bwd;  // some wider launch may read another form
  for (int w = 2; w < ly.n_max && plan.cnt[w] > 0 && (f || r); ++w) {
    if (f) {
      NtArgs a = forward_product(plan, ly, p, fp32_mfma, w, &flop);
      use(a, p.Wn, p.Wn3, &q.Wn, &q.Wn3);
      a.parts = 0; a.cols = (int)(2 * ly.Np);  // as one product: at least the work of every wider launch
      f = !(q.Wn && q.Wn3) && a.planes3 == 3 && (q.Wn3 || gemm_nt_reads_planes(a));  // (one or two planes: all read the same)
    }
    if (r) {
      NtArgs a = reverse_product(plan, ly, p, fp32_mfma, w, nullptr, &flop);
      use(a, p.Wtn, p.Wtn3, &q.Wtn, &q.Wtn3);
      a.parts = 0;
      r = !(q.Wtn && q.Wtn3) && a.planes3 == 3 && (q.Wtn3 || gemm_nt_reads_planes(a));
    }
  }
  if (!fwd) q.colmax = nullptr;
  return q;
}

// Whether the product of width w and the sums that wait for it go in one launch (gemm_step.hip): 0 not, 1 in small tiles, 2 in tall ones.
// Small tiles pay while all workgroups start at once, one a CU, and the product's K is short.  The grid has a tile for every
// start of the longest sentence in every sentence, and those without spans cost their dispatch (N = 512, B = 32, n = 10 .. 30
// training 937 us separate, 963 us with up to four grids of the chip, 935 us with two).  Tall tiles, forward only, where 64
// or 128 padded nonterminals leave most lanes of the separate sums idle: N = 64, B = 128, n = 30 scoring 381 -> 245 us; N = 128,
// B = 30, n = 20 .. 40 390 -> 310 us, but with two blocks of 64 and more than kStepTallTerms terms they fall behind (N = 124, B = 38,
// n = 25 .. 71: 915 us separate, 903 us so, 957 us without the limit), as with more nonterminals (N = 256, B = 12: 278, 289)
// and in reverse (N = 64, B = 128: 100 us slower).
constexpr int kStepWgs = 256, kStepGrid = 512, kStepK = 512, kStepTallNp = 64, kStepTallTerms = 24;
int step_form(const Plan& plan, const Layout& ly, const Ptrs& p, int fp32_mfma, int w, bool fwd) {
  if (ly.bf16 || fp32_mfma) return 0;
  const int next = fwd ? w + 1 : w - 1;
  if (next < 1 || next > ly.n_long || plan.cnt[w] == 0) return 0;
  // (a band's launch has to come between)
  if (fwd ? ly.band_fwd[next / kBandW] && next % kBandW == 0 : ly.band_bwd[next / kBandW] && next == band_top(ly, next / kBandW * kBandW))
    return 0;
  if ((fwd ? (w == 1 ? ly.Pp : ly.Np) : ly.Np) > kStepK) return 0;
  double flop;
  // (the forward launch writes no operand planes of the sums)
  if (fwd && next < ly.n_long && gemm_nt_reads_planes(forward_product(plan, ly, p, fp32_mfma, next, &flop))) return 0;
  const int terms = fwd && ly.band_fwd[next / kBandW] ? 2 * (next % kBandW) : next - 1;
  const bool tall_too = fwd && (ly.Np <= kStepTallNp || (ly.Np <= 2 * kStepTallNp && terms <= kStepTallTerms));
  for (int tall = 0; tall <= (tall_too ? 1 : 0); ++tall) {
    const int per = step_spans(tall);
    int64_t tiles = 0;
    for (int b = 0; b < ly.B; ++b) {
      const int sums = plan.lens.v[b] > next || (fwd && plan.lens.v[b] == next) ? plan.lens.v[b] - next + 1 : 0;
      tiles += (sums + per - 1) / per;
    }
    // (the grid has a tile for every start of the longest sentence in every sentence; those without spans end at once)
    const int64_t cols = ly.Np / step_nonterminals(tall), grid = (int64_t)ly.B * ((ly.n_long - next + per) / per);
    if (tiles * cols <= kStepWgs && grid * cols <= kStepGrid) return 1 + tall;
  }
  return 0;
}
StepArgs step_args(const Layout& ly, const Ptrs& p, int w, bool fwd, int tall) {
  StepArgs s{};
  s.forward = fwd; s.tall = tall; s.w = w;
  s.B = ly.B; s.Np = ly.Np; s.Pp = ly.Pp; s.n_long = ly.n_long; s.stride = (ly.n_max + 1) * ly.B; s.per_sentence = ly.G > 1;
  s.S1 = ly.S1; s.lens = p.lens; s.rowtab = p.rowbase;
  s.K = fwd ? (w == 1 ? ly.Pp : ly.Np) : 2 * ly.Np;
  s.A = fwd ? (w == 1 ? p.leafE : p.T) : p.UV;
  s.a_row0 = fwd && w > 1 ? ly.S1 : 0;
  s.Bm = fwd ? (w == 1 ? p.Wp : p.Wn) : p.Wtn;
  s.b_stride = ly.G > 1 ? 2 * (int64_t)ly.Np * (fwd && w == 1 ? ly.Pp : ly.Np) : 0;
  s.HZ = p.HZ; s.T = p.T; s.UV = p.UV; s.BH = p.BH;
  s.mexp = p.mexp; s.uexp = p.uexp; s.tmaxb = p.tmaxb; s.umaxb = p.umaxb; s.hmaxb = p.hmaxb; s.zmaxb = p.zmaxb;
  s.gsc = p.gsc; s.xs = p.xs; s.rootmask = p.rootmask; s.colmax = p.colmax;
  const int next = fwd ? w + 1 : w - 1, w0 = next / kBandW * kBandW;
  if (fwd) s.w0 = ly.band_fwd[next / kBandW] ? w0 : 0;
  else s.w0 = ly.band_bwd[next / kBandW] ? w0 + kBandW : 0;
  return s;
}

bool with_step(NtArgs& a, StepArgs* step, const Plan& plan, const Layout& ly, const Ptrs& p, int fp32_mfma, int w, bool fwd) {
  const int form = gemm_nt_reads_planes(a) ? 0 : step_form(plan, ly, p, fp32_mfma, w, fwd);
  if (form == 0) return false;
  *step = step_args(ly, p, w, fwd, form - 1);
  if (ly.tn3) { step->UVb = p.UVb; step->planes = ly.planes_bwd; step->plane_stride = ly.uvb_plane; }  // (rule gradients read them)
  a.step = step;
  return true;
}

int forward(const spcfg_config* cfg, const Plan& plan, const Layout& ly, const Ptrs& p, const float* log_root,
            const float* L, const float* R, const float* log_emit, float* logZ, bool with_backward, hipStream_t st) {
  const int n_max = ly.n_max;
  const int fp32_mfma = (cfg->flags & SPCFG_FLAG_FP32_MFMA) ? 1 : 0;
  NtArgs leaf = forward_product(plan, ly, p, fp32_mfma, 1, nullptr);
  {
    // (L and R read, the panels of the passes to come written)
    Scope s(SPCFG_PROF_SETUP, 4.0 * 2 * (double)ly.N * (ly.N + ly.P) * (with_backward ? 3 : 2) + 8.0 * ly.S1 * ly.P);
    launch_plan(ly, p, plan.lens, st);
    if (ly.G > 1) launch_plan_sentrows(ly, p, st);
    launch_pack_weights(ly, panels_read(plan, ly, p, fp32_mfma, true, with_backward), L, R, st);
    // operand planes are written only for the launches that read them (bf16 mode: all of them)
    launch_leaf_prep(ly, p, log_emit, (ly.bf16 && !ly.fwd_fp32) || gemm_nt_reads_planes(leaf), st);
  }
  StepArgs step;
  bool summed;  // the sums of the next width were taken in the launch of the last product
  {
    summed = with_step(leaf, &step, plan, ly, p, fp32_mfma, 1, true);
    Scope s(SPCFG_PROF_GEMM_FWD, 4.0 * ly.N * (double)ly.P * ly.S1, summed ? SPCFG_PROF_SPLIT_FWD : -1,
            summed && g_prof.on ? split_fwd_bytes(plan, ly, 2) : 0.0);
    launch_gemm_nt(leaf, st);
  }
  for (int w = 2; w <= n_max; ++w) {
    const int64_t row0 = plan.off[w], rows = plan.cnt[w];
    if (rows == 0) continue;
    const double split_bytes = g_prof.on ? split_fwd_bytes(plan, ly, w) : 0.0;
    if (w == n_max) {  // every span of the largest width is a root span: never a child, not projected
      if (!summed) {
        Scope s(SPCFG_PROF_SPLIT_FWD, split_bytes);
        launch_split_fwd(ly, p, w, row0, rows, false, st);
      }
      break;
    }
    double skipped = 0.0;  // flop of the projections that the launch leaves out
    NtArgs a = forward_product(plan, ly, p, fp32_mfma, w, &skipped);
    if (!summed) {
      Scope s(SPCFG_PROF_SPLIT_FWD, split_bytes);
      launch_split_fwd(ly, p, w, row0, rows, (ly.bf16 && !ly.fwd_fp32) || gemm_nt_reads_planes(a), st);
    }
    summed = with_step(a, &step, plan, ly, p, fp32_mfma, w, true);
    Scope s(SPCFG_PROF_GEMM_FWD, 4.0 * ly.N * (double)ly.N * rows - skipped, summed ? SPCFG_PROF_SPLIT_FWD : -1,
            summed && g_prof.on ? split_fwd_bytes(plan, ly, w + 1) : 0.0);
    launch_gemm_nt(a, st);
  }
  {
    Scope s(SPCFG_PROF_ROOT, 8.0 * ly.N * ly.B);
    launch_root_fwd(ly, p, log_root, logZ, st);
  }
  (void)cfg;
  return hip_status();
}

// (L, R: null where the forward call packed the reverse panels too)
int backward(const spcfg_config* cfg, const Plan& plan, const Layout& ly, const Ptrs& p, const float* log_root, const float* L,
             const float* R,
             const float* grad_logZ, float* grad_L, float* grad_R, float* grad_log_root, float* grad_log_emit,
             hipStream_t st) {
  const int n_max = ly.n_max;
  const int64_t Np = ly.Np, Pp = ly.Pp;
  const int fp32_mfma = (cfg->flags & SPCFG_FLAG_FP32_MFMA) ? 1 : 0;
  const int acc = (cfg->flags & SPCFG_FLAG_ACCUMULATE_GRADS) ? 1 : 0;
  if (L) {
    Scope s(SPCFG_PROF_SETUP, 4.0 * 2 * (double)ly.N * (ly.N + ly.P) * 2);
    launch_pack_weights(ly, panels_read(plan, ly, p, fp32_mfma, false, true), L, R, st);
  }
  {
    Scope s(SPCFG_PROF_ROOT, 16.0 * ly.N * ly.B);
    launch_root_bwd(ly, p, log_root, grad_logZ, grad_log_root, acc, st);
    launch_zero_pad_emit(ly, p, grad_log_emit, st);
  }
  StepArgs step;
  bool summed = false;  // the sums of this width were taken in the launch of the last product
  for (int w = n_max - 1; w >= 1; --w) {  // spans of width n_max are all roots
    const int64_t row0 = plan.off[w], rows = plan.cnt[w];
    if (rows == 0) continue;
    const double split_bytes = g_prof.on ? split_bwd_bytes(plan, ly, w) : 0.0;
    double gemm_flop;
    NtArgs a = reverse_product(plan, ly, p, fp32_mfma, w, grad_log_emit, &gemm_flop);
    if (!summed) {
      Scope s(SPCFG_PROF_SPLIT_BWD, split_bytes);
      // (the rule-gradient product on planes reads the adjoint planes of every row)
      launch_split_bwd(ly, p, w, row0, rows, ly.bf16 || ly.tn3 || gemm_nt_reads_planes(a), st);
    }
    {
      summed = w >= 2 && with_step(a, &step, plan, ly, p, fp32_mfma, w, false);
      Scope s(SPCFG_PROF_GEMM_BWD, gemm_flop, summed ? SPCFG_PROF_SPLIT_BWD : -1,
              summed && g_prof.on ? split_bwd_bytes(plan, ly, w - 1) : 0.0);
      launch_gemm_nt(a, st);
    }
  }
  {
    Scope s(SPCFG_PROF_GEMM_GRAD, 4.0 * ly.N * ((double)ly.N * ly.S2 + (double)ly.P * ly.S1));
    if (ly.G > 1) {
      // one reduction per sentence over its own spans of width >= 2 (listed in sentrows), one over its leaves
      int n_longest = 2;
      for (int b = 0; b < ly.B; ++b) n_longest = plan.lens.v[b] > n_longest ? plan.lens.v[b] : n_longest;
      TnArgs t{};
      t.fp32_mfma = fp32_mfma;
      t.Np = (int)Np; t.N = ly.N; t.gL = grad_L; t.gR = grad_R; t.ldg = ly.N + ly.P; t.accumulate = acc;
      t.ngroups = ly.B; t.grp_lens = p.lens; t.grp_gstride = (int64_t)ly.N * (ly.N + ly.P);
      t.A = p.UV; t.lda = 2 * Np; t.sc = p.gsc;
      t.grp_mode = 1; t.rowlist = p.sentrows; t.grp_off = p.sentoff; t.brow0 = ly.S1;
      t.Bm = p.T; t.ldb = Np; t.cols = ly.N; t.col0 = 0;
      t.grp_kt_max = (int)(((int64_t)n_longest * (n_longest - 1) / 2 + 31) / 32);
      launch_gemm_tn(t, st);
      t.grp_mode = 2; t.grp_base = p.rowbase + ly.B;  // first leaf row of every sentence
      t.Bm = p.leafE; t.ldb = Pp; t.cols = ly.P; t.col0 = ly.N;
      t.grp_kt_max = (n_longest + 31) / 32;
      launch_gemm_tn(t, st);
    } else if (ly.tn3) {
      // on planes: the adjoint rows as their producers cut them, the inside vectors times the span scale cut here
      const int64_t step = kTn3Rows(ly.tn3), planes = ly.tn3 == 3 ? 1 : 0;
      launch_scaled_planes(p.T, Np, p.gsc + ly.S1, ly.S2, ly.S2p, p.Tg3, planes * ly.S2p * Np, st);
      launch_scaled_planes(p.leafE, Pp, p.gsc, ly.S1, ly.S1p, p.Eg3, planes * ly.S1p * Pp, st);
      launch_zero_plane_rows(p.UVb, planes * ly.uvb_plane, 2 * Np, ly.Sall, step, st);
      Tn3Args t{};
      t.planes = ly.tn3;
      t.partial = p.partial; t.counters = p.counters; t.max_wgs = ly.gemm_wgs; t.n_counters = ly.n_counters;
      t.Np = (int)Np; t.N = ly.N; t.gL = grad_L; t.gR = grad_R; t.ldg = ly.N + ly.P; t.accumulate = acc;
      t.a_plane = ly.uvb_plane; t.lda = 2 * Np;
      t.A3 = static_cast<const uint16_t*>(p.UVb) + ly.S1 * 2 * Np; t.B3 = static_cast<const uint16_t*>(p.Tg3);
      t.b_plane = ly.S2p * Np; t.ldb = Np; t.KT = (int)(ly.S2p / step); t.cols = ly.N; t.col0 = 0;
      launch_gemm_tn3(t, st);
      t.A3 = static_cast<const uint16_t*>(p.UVb); t.B3 = static_cast<const uint16_t*>(p.Eg3);
      t.b_plane = ly.S1p * Pp; t.ldb = Pp; t.KT = (int)(ly.S1p / step); t.cols = ly.P; t.col0 = ly.N;
      launch_gemm_tn3(t, st);
    } else {
      TnArgs t{};
      t.fp32_mfma = fp32_mfma;
      t.partial = p.partial; t.counters = p.counters; t.max_wgs = ly.gemm_wgs; t.n_counters = ly.n_counters;
      t.Np = (int)Np; t.N = ly.N; t.gL = grad_L; t.gR = grad_R; t.ldg = ly.N + ly.P; t.accumulate = acc;
      t.A = p.UV + ly.S1 * 2 * Np; t.lda = 2 * Np; t.Bm = p.T; t.ldb = Np; t.sc = p.gsc + ly.S1; t.S = ly.S2;
      t.cols = ly.N; t.col0 = 0;
      launch_gemm_tn(t, st);
      t.A = p.UV; t.Bm = p.leafE; t.ldb = Pp; t.sc = p.gsc; t.S = ly.S1; t.cols = ly.P; t.col0 = ly.N;
      launch_gemm_tn(t, st);
    }
  }
  return hip_status();
}

}  // namespace
}  // namespace spcfg

using namespace spcfg;

// ---- static device scratch for the entry point that allocates nothing ---------------------------------------
// One array per GPU (every device that loads the library's code object holds its own copy at its own address).
// In host code the array's name only stands for the symbol: the device address comes from hipGetSymbolAddress,
// once per device, and that pointer is what the kernels get.
#ifndef SPCFG_HOST_CHECKS_BUILD  // (the host-only build of tests/sanitize has no device code object to hold it)
static __device__ __align__(256) unsigned char scratch[SPCFG_STATIC_SCRATCH_BYTES];
#endif

namespace {
constexpr int kStaticGemmWgs = 64;   // partial-tile scratch of the static buffer: 2 * 64 slots of 64 KiB = 8 MiB
constexpr int kMaxDevices = 64;
void* g_scratch_ptr[kMaxDevices] = {nullptr};
std::mutex g_scratch_mutex;

// Device address of this device's copy of `scratch` (looked up on the first call on a device, with that device
// current), or nullptr with the HIP error text recorded.
void* static_scratch() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    snprintf(g_hip_err, sizeof(g_hip_err), "no current HIP device below %d", kMaxDevices);
    (void)hipGetLastError();
    return nullptr;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
#ifndef SPCFG_HOST_CHECKS_BUILD
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
#else
    const hipError_t e = hipErrorNotSupported;
#endif
    if (e != hipSuccess || !ptr) {
      snprintf(g_hip_err, sizeof(g_hip_err), "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
      (void)hipGetLastError();
      return nullptr;
    }
    g_scratch_ptr[dev] = ptr;
  }
  return g_scratch_ptr[dev];
}
}  // namespace

extern "C" {

int spcfg_inside_static(const spcfg_config* cfg, const float* log_root, const float* L, const float* R,
                        const float* log_emit, const int32_t* lengths, int32_t B, int32_t n_max, float* logZ,
                        void* hip_stream) {
  int rc = check_cfg(cfg);
  if (rc) return rc;
  if (!log_root || !L || !R || !log_emit || !logZ) return SPCFG_ERR_ARG;
  Plan plan; Layout ly;
  rc = make_plan(cfg, lengths, B, n_max, &plan, &ly, kStaticGemmWgs);
  if (rc) return rc;
  if (ly.total > (size_t)SPCFG_STATIC_SCRATCH_BYTES) return SPCFG_ERR_STATIC_CAPACITY;
  void* ws = static_scratch();
  if (!ws) return SPCFG_ERR_HIP;
  return forward(cfg, plan, ly, resolve(ly, ws), log_root, L, R, log_emit, logZ, false, (hipStream_t)hip_stream);
}

int spcfg_workspace_bytes(const spcfg_config* cfg, size_t* out_bytes) {
  int rc = check_cfg(cfg);
  if (rc) return rc;
  if (!out_bytes) return SPCFG_ERR_ARG;
  const int64_t S1 = (int64_t)cfg->max_B * cfg->max_n;
  const int64_t Sall = (int64_t)cfg->max_B * cfg->max_n * (cfg->max_n + 1) / 2;
  if (Sall >= (int64_t)1 << 30) return SPCFG_ERR_SHAPE;
  *out_bytes = make_layout(cfg->N, cfg->P, cfg->max_B, cfg->max_n, S1, Sall - S1,
                           cfg->precision == SPCFG_PRECISION_BF16,
                           (cfg->flags & SPCFG_FLAG_PER_SENTENCE_GRAMMAR) != 0,
                           (cfg->flags & SPCFG_FLAG_FP32_MFMA) != 0,
                           (cfg->flags & SPCFG_FLAG_BF16_SINGLE_FORWARD) != 0).total;
  return SPCFG_OK;
}

int spcfg_workspace_bytes_for(const spcfg_config* cfg, const int32_t* lengths, int32_t B, int32_t n_max,
                              size_t* out_bytes) {
  int rc = check_cfg(cfg);
  if (rc) return rc;
  if (!out_bytes) return SPCFG_ERR_ARG;
  Plan plan; Layout ly;
  rc = make_plan(cfg, lengths, B, n_max, &plan, &ly);
  if (rc) return rc;
  *out_bytes = ly.total;
  return SPCFG_OK;
}

int spcfg_inside(const spcfg_config* cfg, const float* log_root, const float* L, const float* R,
                 const float* log_emit, const int32_t* lengths, int32_t B, int32_t n_max, float* logZ,
                 void* workspace, size_t workspace_bytes, void* hip_stream) {
  int rc = check_cfg(cfg);
  if (rc) return rc;
  if (!log_root || !L || !R || !log_emit || !logZ) return SPCFG_ERR_ARG;
  Plan plan; Layout ly;
  rc = make_plan(cfg, lengths, B, n_max, &plan, &ly);
  if (rc) return rc;
  rc = check_ws(ly, workspace, workspace_bytes);
  if (rc) return rc;
  return forward(cfg, plan, ly, resolve(ly, workspace), log_root, L, R, log_emit, logZ, false, (hipStream_t)hip_stream);
}

int spcfg_inside_backward(const spcfg_config* cfg, const float* log_root, const float* L, const float* R,
                          const float* log_emit, const int32_t* lengths, int32_t B, int32_t n_max,
                          const float* grad_logZ, float* grad_L, float* grad_R, float* grad_log_root,
                          float* grad_log_emit, void* workspace, size_t workspace_bytes, void* hip_stream) {
  int rc = check_cfg(cfg);
  if (rc) return rc;
  if (!log_root || !L || !R || !log_emit || !grad_L || !grad_R || !grad_log_root || !grad_log_emit)
    return SPCFG_ERR_ARG;
  Plan plan; Layout ly;
  rc = make_plan(cfg, lengths, B, n_max, &plan, &ly);
  if (rc) return rc;
  rc = check_ws(ly, workspace, workspace_bytes);
  if (rc) return rc;
  return backward(cfg, plan, ly, resolve(ly, workspace), log_root, L, R, grad_logZ, grad_L, grad_R, grad_log_root,
                  grad_log_emit, (hipStream_t)hip_stream);
}

int spcfg_inside_forward_backward(const spcfg_config* cfg, const float* log_root, const float* L,
                                  const float* R, const float* log_emit, const int32_t* lengths, int32_t B,
                                  int32_t n_max, const float* grad_logZ, float* logZ, float* grad_L,
                                  float* grad_R, float* grad_log_root, float* grad_log_emit, void* workspace,
                                  size_t workspace_bytes, void* hip_stream) {
  int rc = check_cfg(cfg);
  if (rc) return rc;
  if (!log_root || !L || !R || !log_emit || !logZ || !grad_L || !grad_R || !grad_log_root || !grad_log_emit)
    return SPCFG_ERR_ARG;
  Plan plan; Layout ly;
  rc = make_plan(cfg, lengths, B, n_max, &plan, &ly);
  if (rc) return rc;
  rc = check_ws(ly, workspace, workspace_bytes);
  if (rc) return rc;
  const Ptrs p = resolve(ly, workspace);
  rc = forward(cfg, plan, ly, p, log_root, L, R, log_emit, logZ, true, (hipStream_t)hip_stream);
  if (rc) return rc;
  return backward(cfg, plan, ly, p, log_root, nullptr, nullptr, grad_logZ, grad_L, grad_R, grad_log_root, grad_log_emit,
                  (hipStream_t)hip_stream);
}

int spcfg_span_marginals(const spcfg_config* cfg, const int32_t* lengths, int32_t B, int32_t n_max,
                         const void* workspace, size_t workspace_bytes, float* span_post, int32_t* span_label,
                         void* hip_stream) {
  int rc = check_cfg(cfg);
  if (rc) return rc;
  if (!span_post) return SPCFG_ERR_ARG;
  Plan plan; Layout ly;
  rc = make_plan(cfg, lengths, B, n_max, &plan, &ly);
  if (rc) return rc;
  rc = check_ws(ly, const_cast<void*>(workspace), workspace_bytes);
  if (rc) return rc;
  launch_span_marginals(ly, resolve(ly, const_cast<void*>(workspace)), span_post, span_label, (hipStream_t)hip_stream);
  return hip_status();
}

const char* spcfg_strerror(int code) {
  switch (code) {
    case SPCFG_OK: return "ok";
    case SPCFG_ERR_ARG: return "invalid argument (null pointer or bad struct_size)";
    case SPCFG_ERR_SHAPE: return "shape out of range or above the configured capacity";
    case SPCFG_ERR_LENGTH: return "sentence length below 2 or above n_max";
    case SPCFG_ERR_WORKSPACE: return "workspace misaligned or too small";
    case SPCFG_ERR_UNSUPPORTED: return "precision or flag not supported";
    case SPCFG_ERR_HIP: return "HIP runtime error";
    case SPCFG_ERR_STATIC_CAPACITY: return "batch needs more scratch than the static device buffer of spcfg_inside_static holds";
    default: return "unknown error code";
  }
}

const char* spcfg_last_hip_error(void) { return g_hip_err; }

int spcfg_profile_enable(int on) {
  std::lock_guard<std::mutex> lock(g_prof.mu);
  g_prof.on = on != 0;
  if (g_prof.on) {
    g_prof.recycle();
    g_prof.all = g_prof.shared = Prof::Sums{};
  }
  return SPCFG_OK;
}

int spcfg_profile_read(double* ms, int64_t* launches, double* work) {
  if (!ms || !launches || !work) return SPCFG_ERR_ARG;
  std::lock_guard<std::mutex> lock(g_prof.mu);
  int rc = SPCFG_OK;
  for (auto& r : g_prof.recs) {
    float t = 0.0f;
    if (hipEventSynchronize(r.b) != hipSuccess || hipEventElapsedTime(&t, r.a, r.b) != hipSuccess) rc = SPCFG_ERR_HIP;
    if (r.also < 0) { g_prof.all.ms[r.cls] += t; continue; }
    for (int c : {r.cls, r.also}) { g_prof.all.ms[c] += 0.5 * t; g_prof.shared.ms[c] += 0.5 * t; }
  }
  g_prof.recycle();
  for (int c = 0; c < SPCFG_PROF_CLASSES; ++c) {
    ms[c] = g_prof.all.ms[c];
    launches[c] = g_prof.all.launches[c];
    work[c] = g_prof.all.work[c];
  }
  g_prof.last_shared = g_prof.shared;
  g_prof.all = g_prof.shared = Prof::Sums{};
  return rc;
}

int spcfg_profile_read_shared(double* ms, int64_t* launches, double* work) {
  if (!ms || !launches || !work) return SPCFG_ERR_ARG;
  std::lock_guard<std::mutex> lock(g_prof.mu);
  for (int c = 0; c < SPCFG_PROF_CLASSES; ++c) {
    ms[c] = g_prof.last_shared.ms[c];
    launches[c] = g_prof.last_shared.launches[c];
    work[c] = g_prof.last_shared.work[c];
  }
  return SPCFG_OK;
}

const char* spcfg_profile_class_name(int cls) {
  static const char* names[SPCFG_PROF_CLASSES] = {"setup", "gemm_fwd", "split_fwd", "root", "split_bwd", "gemm_bwd",
                                                  "gemm_grad"};
  return (cls >= 0 && cls < SPCFG_PROF_CLASSES) ? names[cls] : "?";
}

}  // extern "C"
