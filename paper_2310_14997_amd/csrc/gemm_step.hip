// One launch for a width's projection product and the next width's split-point sums (forward), resp. for a width's reverse
// product and the parents' sums of the width below (reverse), where launches are short and a pass costs its chain of them.
//
// The sums are elementwise in the nonterminal: beta(i, i+w+1)[A] needs eta and zeta of nonterminal A only.  So a workgroup
// that owns a block of nonterminals - their columns of eta and of zeta - for a run of spans of one sentence can go on from
// its product to the sums of the next width without hearing from any other workgroup; only the next product needs all of
// a row.  And all terms but two of such a sum have children that earlier launches wrote: half of the wavefronts (the product's) split K
// between them, the other half sum those old terms in the meantime, and when both are done the new terms are added.
//  * A tile is 16 MI consecutive spans of one sentence and 16 NJ nonterminals.  Neighbouring tiles overlap by one span: a sum
//    needs the children at starts i and i + 1 (reverse: the parents at i - 1 and i).
//  * Operands go from memory to registers, 16 rows x 32 values a wavefront and load pair; each value is cut into three bf16
//    pieces by the one lane that multiplies it (nt::Split3), and the wavefronts' partial tiles are summed in wavefront order.
//  * The old terms' sum keeps a running largest exponent per span and wavefront (rescaling by powers of two is exact), so
//    its wavefronts need no word from each other before the one barrier.
//  * Everything that does not depend on the product is asked for before it: two dependent lookups (length and row tables,
//    then rows and exponents) lie before the first matrix instruction and before the first sum alike.
// A forward launch takes 6 us at N = 64 to 141 (product and sums apart 3.5 + 4.5 us and a launch more), 8 us at N = 512 (9 us), a
// reverse one 7.6 us at N = 141.  Whole calls,
// separate -> one launch a width, sentences of 30 words: scoring N = 64, B = 32 269 -> 199 us; N = 141, B = 1 238 -> 181; N = 256,
// B = 4 260 -> 206; a training step 647 -> 499, 524 -> 438 and 553 -> 488 us.  A second round of workgroups costs more than
// the launch that it saves (N = 141, B = 24: 284 -> 383 us if all widths went this way), long rows of K leave the form behind
// the separate product's finer tiles (N = 1024, B = 1: 299 -> 316 us): see step_form in spcfg_api.hip.
#include <type_traits>

#include "chart_device.h"

namespace spcfg {

namespace {

using namespace nt;

constexpr int kProdWaves = 8;  // wavefronts that split K
constexpr int kSumWaves = 8;   // wavefronts that share the old terms
constexpr int kStepThreads = 64 * (kProdWaves + kSumWaves);
constexpr int kTerms = 4;      // terms of a wavefront in flight

// A uniform read of a table that this launch does not write (through the scalar cache).
__device__ __forceinline__ int uniform(const int32_t* p, int at) {
#if defined(__HIP_DEVICE_COMPILE__)
  return reinterpret_cast<const __attribute__((address_space(4))) int32_t*>((uintptr_t)p)[at];
#else
  return p[at];
#endif
}
template <int MI, int NJ> struct StepGeo {
  static constexpr int R = 16 * MI;       // spans of the product in a tile
  static constexpr int NB = 16 * NJ;      // nonterminals
  static constexpr int Q = 4 * NJ;        // lanes that share a span's nonterminals (four each)
  static constexpr int SPW = 64 / Q;      // spans that a wavefront sums at a time
  static constexpr int PS = R / SPW;      // such groups of spans in a tile
  static constexpr int WP = kSumWaves / PS;  // wavefronts that share a group's terms
  static_assert(PS * WP == kSumWaves && R * Q <= 64 * kSumWaves, "the wavefronts that sum cover the tile");
};

__device__ __forceinline__ float4 load4(const float* p) { return *reinterpret_cast<const float4*>(p); }
__device__ __forceinline__ void axpy(float4& acc, float c, const float4& x, float cz, const float4& y) {
  acc.x = fmaf(c * x.x, cz * y.x, acc.x);
  acc.y = fmaf(c * x.y, cz * y.y, acc.y);
  acc.z = fmaf(c * x.z, cz * y.z, acc.z);
  acc.w = fmaf(c * x.w, cz * y.w, acc.w);
}
__device__ __forceinline__ float4 scaled(float c, const float4& x) { return make_float4(c * x.x, c * x.y, c * x.z, c * x.w); }
__device__ __forceinline__ float4 sum4(const float4& x, const float4& y) {
  return make_float4(x.x + y.x, x.y + y.y, x.z + y.z, x.w + y.w);
}
// The value that lane Q of this lane's four has, and the largest of the four.
template <int Q> __device__ __forceinline__ int quad(int v) {
  return __builtin_amdgcn_update_dpp(0, v, Q * 0x55, 0xf, 0xf, true);  // quad_perm [Q, Q, Q, Q]
}
template <int Q> __device__ __forceinline__ float quad(float v) { return __int_as_float(quad<Q>(__float_as_int(v))); }
__device__ __forceinline__ int quad_max(int v) {
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0xb1, 0xf, 0xf, true));  // quad_perm [1, 0, 3, 2]
  return max(v, __builtin_amdgcn_update_dpp(0, v, 0x4e, 0xf, 0xf, true));  // quad_perm [2, 3, 0, 1]
}
__device__ __forceinline__ float exp_coef(int d, int m) { return d == kExpZero ? 0.0f : pow2i(d - m); }

// The product of one wavefront: MI x NI tiles of 16 x 16 over its K-steps wave, wave + kProdWaves, ... of 32 values; partial
// tiles to `part` in the accumulators' layout (row 4 (l / 16) + v, column l % 16).
template <int MI, int NI, typename Rows>
__device__ __forceinline__ bool product(const float* const (&bp)[NI], int steps, int wave, int lane, float* part, Rows&& rows) {
  floatx4 acc[MI][NI];
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) acc[mi][ni] = floatx4{0.f, 0.f, 0.f, 0.f};
  constexpr int NF = MI + NI;
  constexpr int NBUF = NF <= 4 ? 2 : 1;  // steps whose operands fit in registers
  float4 u[NBUF][NF], v[NBUF][NF];
  const float* ap[MI];
  auto fetch_b = [&](int s, int buf) {
#pragma unroll
    for (int q = 0; q < NI; ++q) { u[buf][MI + q] = load4(bp[q] + s * 32); v[buf][MI + q] = load4(bp[q] + s * 32 + 16); }
  };
  auto fetch_a = [&](int s, int buf) {
#pragma unroll
    for (int q = 0; q < MI; ++q) { u[buf][q] = load4(ap[q] + s * 32); v[buf][q] = load4(ap[q] + s * 32 + 16); }
  };
  // the panel's operands of the first steps are asked for before the rows are known
#pragma unroll
  for (int f = 0; f < NBUF; ++f)
    if (wave + f * kProdWaves < steps) fetch_b(wave + f * kProdWaves, f);
  if (!rows(ap)) return false;
#pragma unroll
  for (int f = 0; f < NBUF; ++f)
    if (wave + f * kProdWaves < steps) fetch_a(wave + f * kProdWaves, f);
  __builtin_amdgcn_sched_barrier(0);
  for (int s0 = wave; s0 < steps; s0 += NBUF * kProdWaves) {
#pragma unroll
    for (int f = 0; f < NBUF; ++f) {
      const int s = s0 + f * kProdWaves;
      if (s >= steps) break;
      Split3 x[MI];
#pragma unroll
      for (int q = 0; q < MI; ++q) x[q].cut(u[f][q], v[f][q]);
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) {
        Split3 y;
        y.cut(u[f][MI + ni], v[f][MI + ni]);
#define SPCFG_T(X, Y)                                 \
  _Pragma("unroll") for (int mi = 0; mi < MI; ++mi)   \
    acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[mi].X(), y.Y(), acc[mi][ni], 0, 0, 0);
        SPCFG_T(l, h) SPCFG_T(h, l) SPCFG_T(m, m) SPCFG_T(m, h) SPCFG_T(h, m) SPCFG_T(h, h)
#undef SPCFG_T
      }
      if (s + NBUF * kProdWaves < steps) { fetch_b(s + NBUF * kProdWaves, f); fetch_a(s + NBUF * kProdWaves, f); }
    }
  }
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int e = 0; e < 4; ++e) part[((mi * NI + ni) * 4 + e) * 64 + lane] = acc[mi][ni][e];
  return true;
}

// Four neighbouring columns of the product: row `row` of the tile, column block ni, columns 4 c4 .. + 3; the wavefronts' parts in order.
template <int MI, int NI>
__device__ __forceinline__ float4 product_at(const float* part, int row, int ni, int c4) {
  const float* p = part + (((row >> 4) * NI + ni) * 4 + (row & 3)) * 64 + ((row >> 2) & 3) * 16 + 4 * c4;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int q = 0; q < kProdWaves; ++q) s = sum4(s, load4(p + q * (MI * NI * 256)));  // (a wavefront without a step has zeros)
  return s;
}

template <int MI, int NJ>
__global__ void __launch_bounds__(kStepThreads) k_step_fwd(StepArgs g) {
  using G = StepGeo<MI, NJ>;
  constexpr int NI = 2 * NJ;  // eta's column blocks, then zeta's
  extern __shared__ __align__(16) float smem[];
  float* s_part = smem;                                             // [kProdWaves][MI NI 256]
  float* s_sum = s_part + kProdWaves * MI * NI * 256;               // [kSumWaves][SPW][NB]
  int32_t* s_exp = reinterpret_cast<int32_t*>(s_sum + kSumWaves * 256);  // [kSumWaves][SPW]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = blockIdx.z, w = g.w, W = w + 1, B = g.B, Np = g.Np;
  const int32_t* tab = g.rowtab + b;
  const int32_t* tab1 = tab + g.stride;
  const int32_t* tab2 = tab1 + g.stride;
  const int i0 = blockIdx.y * (G::R - 1), a0 = blockIdx.x * G::NB;
  const int steps = g.K / 32;
  // split points of the next width: all, or (w0 > 0) those with a child of width w0 or more; the first and the last have a
  // child of width w
  const int nk = g.w0 > 0 ? 2 * (W - g.w0) : w;
  const int nold = max(nk - 2, 0);
  const int64_t ld = 2 * (int64_t)Np;
  if (wave < kProdWaves) {
    const int fr = lane & 15, kq = (lane >> 4) * 4;
    const float* bp[NI];
    const float* bm = static_cast<const float*>(g.Bm) + b * g.b_stride + kq;
#pragma unroll
    for (int q = 0; q < NI; ++q) bp[q] = bm + (int64_t)((q / NJ) * Np + a0 + (q % NJ) * 16 + fr) * g.K;
    const bool there = product<MI, NI>(bp, steps, wave, lane, s_part + wave * (MI * NI * 256), [&](const float* (&ap)[MI]) {
      const int pairs = uniform(g.lens, b) - w;
      const int w_first = uniform(tab, w * B), w_mid = uniform(tab1, w * B) - 1, w_last = uniform(tab2, w * B);
#pragma unroll
      for (int q = 0; q < MI; ++q) {
        const int i = min(i0 + 16 * q + fr, pairs);
        const int r = i == 0 ? w_first : (i == pairs ? w_last : w_mid + i);
        ap[q] = static_cast<const float*>(g.A) + (r - g.a_row0) * g.K + kq;
      }
      return i0 < pairs;  // (uniform: otherwise this sentence has fewer spans)
    });
    if (there) __syncthreads();
    return;
  }
  const int sw = wave - kProdWaves;
  // ---- what the last step needs, asked for first: thread u finishes span u / Q of the tile, nonterminals 4 (u % Q) .. + 3
  const int u = tid - 64 * kProdWaves, fs = u / G::Q, c4 = u % G::Q;
  const int fa = a0 + 4 * c4;
  const int fi = i0 + fs;                         // start of the span of width w, and of the span of width w + 1
  const int pass = sw / G::WP, at = sw % G::WP;
  const int si = i0 + pass * G::SPW + lane / G::Q;  // start of the span whose old terms this lane sums
  // the first kTerms terms' rows: lane % 4 looks up one of them, for every lane of the span
  int lr, rr, rr_end;
  auto lookup = [&](int t0) {  // (nothing here waits for the sentence's length)
    const int t = min(t0 + (lane & 3) * G::WP, max(nold - 1, 0)) + 1;
    const int k = min((g.w0 > 0 && t >= W - g.w0) ? t + 2 * g.w0 - W : t + 1, w);
    lr = (si == 0 ? tab : tab1)[k * B] + (si == 0 ? 0 : si - 1);
    rr = tab1[(W - k) * B] + si + k - 1;
    rr_end = tab2[(W - k) * B];
  };
  lookup(at);
  const int n = uniform(g.lens, b);
  const int w_first = uniform(tab, w * B), w_mid = uniform(tab1, w * B) - 1, w_last = uniform(tab2, w * B);  // rows of width w
  const int o_first = uniform(tab, W * B), o_mid = uniform(tab1, W * B) - 1, o_last = uniform(tab2, W * B), leaf0 = uniform(tab, B);  // of width w + 1, of width 1
  const int pairs = n - w;  // spans of width w + 1; the sentence has one more of width w
  if (i0 >= pairs) return;
  const bool fin = u < G::R * G::Q && fi <= pairs;  // there is such a span of width w
  const bool sum = fin && fs < G::R - 1 && fi < pairs;
  const int fl = min(fi, pairs), fc = min(fi, pairs - 1);
  const int r_l = fl == 0 ? w_first : (fl == pairs ? w_last : w_mid + fl), r_r = fc + 1 == pairs ? w_last : w_mid + fc + 1;
  const int r_out = fc == 0 ? o_first : (fc + W == n ? o_last : o_mid + fc);
  // exponents of the rows of width w, as eta of the left child and zeta of the right child, and of the two children of width 1
  int m_l = 0, m_r = 0, h_l = 0, z_r = 0, m_h = 0, m_z = 0, h_h = 0, z_z = 0, pe = kExpZero;
  uint32_t t_l = 0, t_r = 0, t_h = 0, t_z = 0;
  float4 h1, z1, wl, wr, first = make_float4(0.f, 0.f, 0.f, 0.f);
  h1 = z1 = wl = wr = first;
  if (u < G::R * G::Q) {
    m_l = g.mexp[r_l]; t_l = g.tmaxb[r_l]; h_l = g.hmaxb[r_l];
    m_r = g.mexp[r_r]; t_r = g.tmaxb[r_r]; z_r = g.zmaxb[r_r];
    if (w > 1) {  // the word before the right child, the word behind the left one
      const int lh = leaf0 + fc, lz = leaf0 + fc + w;
      m_h = g.mexp[lh]; t_h = g.tmaxb[lh]; h_h = g.hmaxb[lh];
      m_z = g.mexp[lz]; t_z = g.tmaxb[lz]; z_z = g.zmaxb[lz];
      h1 = load4(g.HZ + lh * ld + fa);
      z1 = load4(g.HZ + lz * ld + Np + fa);
    }
    if (g.w0 > 0) {
      pe = g.uexp[r_out];
      first = load4(g.T + (r_out - g.S1) * Np + fa);
    }
    const float* cm = g.colmax + (int64_t)(g.per_sentence ? b : 0) * 2 * (Np + g.Pp) + fa;
    wl = load4(cm);
    wr = load4(cm + Np + g.Pp);
  }
  // ---- the old terms
  {
    const float* hz = g.HZ + a0 + 4 * (lane % G::Q);
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    int mr = kExpZero;
    for (int t0 = at; t0 < nold; t0 += G::WP * kTerms) {
      if (t0 > at) lookup(t0);
      if (si + W == n) rr = rr_end;
      if (si >= pairs) lr = rr = 0;  // no such span: a row that exists; nothing of it is used
      float4 h[kTerms], z[kTerms];
      const uint32_t tl = g.tmaxb[lr], tr = g.tmaxb[rr];
      const int hl = g.hmaxb[lr], zr = g.zmaxb[rr], ml = g.mexp[lr], mrr = g.mexp[rr];
      static_for<0, kTerms>([&](auto q) {
        constexpr int qv = decltype(q)::value;
        h[qv] = load4(hz + quad<qv>(lr) * ld);
        z[qv] = load4(hz + quad<qv>(rr) * ld + Np);
      });
      int d = add_exp(proj_exp(ml, tl, hl), proj_exp(mrr, tr, zr));
      if (t0 + (lane & 3) * G::WP >= nold) d = kExpZero;
      const int mn = max(mr, quad_max(d));
      acc = scaled(exp_coef(mr, mn), acc);
      mr = mn;
      const float c = d == kExpZero ? 0.0f : pow2i(d - mr - proj_shift(tl, hl)), cz = pow2i(-proj_shift(tr, zr));
      static_for<0, kTerms>([&](auto q) {
        constexpr int qv = decltype(q)::value;
        axpy(acc, quad<qv>(c), h[qv], quad<qv>(cz), z[qv]);
      });
    }
    *reinterpret_cast<float4*>(s_sum + sw * 256 + lane * 4) = acc;
    if (lane % G::Q == 0) s_exp[sw * G::SPW + lane / G::Q] = mr;
  }
  __syncthreads();
  if (u >= (G::R * G::Q + 63) / 64 * 64) return;  // (whole wavefronts: the reductions below see every lane)
  const int jb = c4 / 4, cc = c4 % 4;
  const float f_l = norm_scale(t_l), f_r = norm_scale(t_r);
  const int gh_l = proj_shift(t_l, h_l), gz_r = proj_shift(t_r, z_r), gh_h = proj_shift(t_h, h_h), gz_z = proj_shift(t_z, z_z);
  const int e_l = proj_exp(m_l, t_l, h_l), e_r = proj_exp(m_r, t_r, z_r);
  const int e_h = proj_exp(m_h, t_h, h_h), e_z = proj_exp(m_z, t_z, z_z);
  float tmax = 0.0f;
  int hsum = 0, zsum = 0, m = kExpZero;
  if (fin) {
    const float4 h = scaled(f_l, product_at<MI, NI>(s_part, fs, jb, cc));
    const float4 z0 = scaled(f_l, product_at<MI, NI>(s_part, fs, NJ + jb, cc));
    if (fs < G::R - 1 || fi == pairs) {  // (the last span of a tile is the next tile's first)
      *reinterpret_cast<float4*>(g.HZ + r_l * ld + fa) = h;
      *reinterpret_cast<float4*>(g.HZ + r_l * ld + Np + fa) = z0;
    }
    if (sum) {
      const float4 z = scaled(f_r, product_at<MI, NI>(s_part, fs + 1, NJ + jb, cc));
      // the new terms: the left child (i, i + w) with a word or, at w = 1, with (i + 1, i + 2); a word with (i + 1, i + 1 + w)
      const int d1 = w > 1 ? add_exp(e_l, e_z) : add_exp(e_l, e_r), d2 = w > 1 ? add_exp(e_h, e_r) : kExpZero;
      const int fp = fs / G::SPW, slot = fs % G::SPW;
      m = max(max(d1, d2), pe);
#pragma unroll
      for (int q = 0; q < G::WP; ++q) m = max(m, s_exp[(fp * G::WP + q) * G::SPW + slot]);
      float4 acc = scaled(exp_coef(pe, m), first);
#pragma unroll
      for (int q = 0; q < G::WP; ++q) {
        const int fw = fp * G::WP + q;
        acc = sum4(acc, scaled(exp_coef(s_exp[fw * G::SPW + slot], m), load4(s_sum + fw * 256 + (slot * G::Q + c4) * 4)));
      }
      if (w > 1) {
        axpy(acc, d2 == kExpZero ? 0.0f : pow2i(d2 - m - gh_h), h1, pow2i(-gz_r), z);
        axpy(acc, d1 == kExpZero ? 0.0f : pow2i(d1 - m - gh_l), h, pow2i(-gz_z), z1);
      } else {
        axpy(acc, d1 == kExpZero ? 0.0f : pow2i(d1 - m - gh_l), h, pow2i(-gz_r), z);
      }
      *reinterpret_cast<float4*>(g.T + (r_out - g.S1) * Np + fa) = acc;
      tmax = fmaxf(fmaxf(acc.x, acc.y), fmaxf(acc.z, acc.w));
      hsum = max(max(bexp_sum(wl.x, acc.x), bexp_sum(wl.y, acc.y)), max(bexp_sum(wl.z, acc.z), bexp_sum(wl.w, acc.w)));
      zsum = max(max(bexp_sum(wr.x, acc.x), bexp_sum(wr.y, acc.y)), max(bexp_sum(wr.z, acc.z), bexp_sum(wr.w, acc.w)));
    }
  }
#pragma unroll
  for (int o = 1; o < G::Q; o <<= 1) {
    tmax = fmaxf(tmax, __shfl_xor(tmax, o, 64));
    hsum = max(hsum, __shfl_xor(hsum, o, 64));
    zsum = max(zsum, __shfl_xor(zsum, o, 64));
  }
  if (sum && c4 == 0) {
    if (tmax > 0.0f && m != kExpZero) atomicMax(&g.tmaxb[r_out], __float_as_uint(tmax));
    if (hsum > 0 && m != kExpZero) atomicMax(&g.hmaxb[r_out], hsum);
    if (zsum > 0 && m != kExpZero) atomicMax(&g.zmaxb[r_out], zsum);
    if (blockIdx.x == 0) g.mexp[r_out] = m;
  }
}

// Reverse: the product of the spans of width w (parents), then the sums over parents of the spans of width v = w - 1.  Slot x
// of a tile is the parent of start i0 - 1 + x; child y, of start i0 + y, is the right child of slot y and the left child of slot
// y + 1.  Where the parent is the root (a sentence of w words) its adjoint is there already and nothing is multiplied.
template <int MI, int NJ>
__global__ void __launch_bounds__(kStepThreads) k_step_bwd(StepArgs g) {
  using G = StepGeo<MI, NJ>;
  constexpr int NI = NJ;
  extern __shared__ __align__(16) float smem[];
  float* s_part = smem;                                                 // [kProdWaves][MI NI 256]
  float* s_sum = s_part + kProdWaves * MI * NI * 256;                   // [kSumWaves][2][SPW][NB]
  int32_t* s_exp = reinterpret_cast<int32_t*>(s_sum + kSumWaves * 512);  // [kSumWaves][SPW]
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = blockIdx.z, w = g.w, v = w - 1, B = g.B, Np = g.Np;
  const int32_t* tab = g.rowtab + b;
  const int32_t* tab1 = tab + g.stride;
  const int32_t* tab2 = tab1 + g.stride;
  const int i0 = blockIdx.y * (G::R - 1), a0 = blockIdx.x * G::NB;
  const int64_t ld = 2 * (int64_t)Np;
  if (wave < kProdWaves) {
    const int fr = lane & 15, kq = (lane >> 4) * 4;
    const float* bp[NI];
    const float* bm = static_cast<const float*>(g.Bm) + b * g.b_stride + kq;
#pragma unroll
    for (int q = 0; q < NI; ++q) bp[q] = bm + (int64_t)(a0 + q * 16 + fr) * g.K;
    const bool there = product<MI, NI>(bp, g.K / 32, wave, lane, s_part + wave * (MI * NI * 256), [&](const float* (&ap)[MI]) {
      const int last = uniform(g.lens, b) - w;
      const int w_first = uniform(tab, w * B), w_mid = uniform(tab1, w * B) - 1, w_last = uniform(tab2, w * B);
#pragma unroll
      for (int q = 0; q < MI; ++q) {
        const int p = min(max(i0 - 1 + 16 * q + fr, 0), last);
        const int r = p == 0 ? w_first : (p == last ? w_last : w_mid + p);
        ap[q] = static_cast<const float*>(g.A) + (r - g.a_row0) * g.K + kq;
      }
      return last >= 0 && i0 <= last + 1;  // (uniform: otherwise this sentence has no such spans)
    });
    if (there) __syncthreads();
    return;
  }
  const int sw = wave - kProdWaves;
  const int u = tid - 64 * kProdWaves, fs = u / G::Q, c4 = u % G::Q;
  const int fa = a0 + 4 * c4;
  const int fi = i0 + fs;
  // ---- the old terms: parents of width pw (> w), below w0 where a band has summed the wider ones.  Lane % 4 looks up one term
  // for every lane of its span: bit 0 its role (0: this span is the left child, sibling's zeta; 1: the right child, sibling's eta),
  // bit 1 which of two parent widths
  const int pass = sw / G::WP, at = sw % G::WP;
  const int si = i0 + pass * G::SPW + lane / G::Q, sj = si + v;
  const int role = lane & 1;
  constexpr int U = kTerms / 2;
  int pw, rp, rs, rp_end, rs_end;
  auto lookup = [&](int t0) {  // (nothing here waits for the sentence's length)
    pw = t0 + ((lane >> 1) & 1) * G::WP;
    const int pc = min(pw, g.n_long), sc = pc - v;
    const int ps = role ? sj - pc : si, ss = role ? ps : sj;  // starts of parent and sibling
    rp = ps <= 0 ? tab[pc * B] : tab1[pc * B] + ps - 1;
    rs = ss <= 0 ? tab[sc * B] : tab1[sc * B] + ss - 1;
    rp_end = tab2[pc * B];
    rs_end = tab2[sc * B];
  };
  lookup(w + 1 + at);
  const int n = uniform(g.lens, b);
  const int w_first = uniform(tab, w * B), w_mid = uniform(tab1, w * B) - 1, w_last = uniform(tab2, w * B);  // rows of width w
  const int o_first = uniform(tab, v * B), o_mid = uniform(tab1, v * B) - 1, o_last = uniform(tab2, v * B), leaf0 = uniform(tab, B);  // of width w - 1, of width 1
  const int last = n - w;  // start of the last parent; the last child starts one later
  if (last < 0 || i0 > last + 1) return;
  const bool root = last == 0;
  const int top = g.w0 > 0 ? min(g.w0 - 1, n) : n;
  const int fc = min(fi, last + 1), fj = fc + v;  // the child of this thread
  const bool fin = u < G::R * G::Q && fs < G::R - 1 && fi <= last + 1;
  const bool is_l = fin && fi <= last;  // left child of the parent (i, i + w)
  const bool is_r = fin && fi >= 1;     // right child of the parent (i - 1, i - 1 + w)
  const int sl = min(fc, last), sr = min(max(fc - 1, 0), last);
  const int p_l = sl == 0 ? w_first : (sl == last ? w_last : w_mid + sl), p_r = sr == 0 ? w_first : (sr == last ? w_last : w_mid + sr);
  const int r_c = fc == 0 ? o_first : (fj == n ? o_last : o_mid + fc);
  const int l_l = leaf0 + min(fj, n - 1), l_r = leaf0 + max(fc - 1, 0);  // siblings: the word behind, the word before
  int me = 0, ue_l = 0, ue_r = 0, m_l = 0, m_r = 0, z_l = 0, h_r = 0, peu = kExpZero, pev = kExpZero;
  uint32_t um_l = 0, um_r = 0, t_l = 0, t_r = 0;
  float4 z1 = make_float4(0.f, 0.f, 0.f, 0.f), h1 = z1, xl = z1, xr = z1, u0 = z1, v0 = z1;
  if (u < G::R * G::Q) {
    me = g.mexp[r_c];
    ue_l = g.uexp[p_l]; um_l = g.umaxb[p_l];
    ue_r = g.uexp[p_r]; um_r = g.umaxb[p_r];
    m_l = g.mexp[l_l]; t_l = g.tmaxb[l_l]; z_l = g.zmaxb[l_l];
    m_r = g.mexp[l_r]; t_r = g.tmaxb[l_r]; h_r = g.hmaxb[l_r];
    z1 = load4(g.HZ + l_l * ld + Np + fa);
    h1 = load4(g.HZ + l_r * ld + fa);
    if (root) xl = xr = load4(g.BH + (w_first - g.S1) * Np + fa);
    if (g.w0 > 0) {
      const int2 pe = bwd_part_exp(v, r_c, g.S1, Np, g.BH, g.xs, g.rootmask);
      peu = pe.x;
      pev = pe.y;
      u0 = load4(g.UV + r_c * ld + fa);
      v0 = load4(g.UV + r_c * ld + Np + fa);
    }
  }
  {
    const int aq = a0 + 4 * (lane % G::Q);
    const float* bh = g.BH + aq - g.S1 * Np;
    const float* hz = g.HZ + aq;
    float4 x[2];
    x[0] = x[1] = make_float4(0.f, 0.f, 0.f, 0.f);
    int mr = kExpZero;
    for (int t0 = w + 1 + at; t0 <= top; t0 += G::WP * U) {
      if (t0 > w + 1 + at) lookup(t0);
      const bool there = pw <= top && si <= last + 1 && (role ? sj >= pw : si + pw <= n);
      const bool end = (role ? sj : si + pw) == n;  // the parent ends the sentence; its left child's sibling too
      if (end && (role ? sj > pw : si > 0)) rp = rp_end;
      if (end && !role) rs = rs_end;
      if (!there) { rp = (int)g.S1; rs = 0; }  // rows that exist; nothing of them is used
      const uint32_t um = g.umaxb[rp], ts = g.tmaxb[rs];
      const int ue = g.uexp[rp], ms = g.mexp[rs], ps = (role ? g.hmaxb : g.zmaxb)[rs];
      float4 p[kTerms], q4[kTerms];
      static_for<0, kTerms>([&](auto q) {
        constexpr int qv = decltype(q)::value;
        p[qv] = q4[qv] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (quad<qv>((int)there)) {
          p[qv] = load4(bh + (int64_t)quad<qv>(rp) * Np);
          q4[qv] = load4(hz + quad<qv>(rs) * ld + ((qv & 1) ? 0 : Np));
        }
      });
      const int d = there ? add_exp(norm_exp(ue, um), proj_exp(ms, ts, ps)) : kExpZero;
      const int mn = max(mr, quad_max(d));
      const float f = exp_coef(mr, mn);
      x[0] = scaled(f, x[0]);
      x[1] = scaled(f, x[1]);
      mr = mn;
      const float c = exp_coef(d, mr), cs = pow2i(-proj_shift(ts, ps));
      static_for<0, kTerms>([&](auto q) {
        constexpr int qv = decltype(q)::value;
        axpy(x[qv & 1], quad<qv>(c), p[qv], quad<qv>(cs), q4[qv]);
      });
    }
    *reinterpret_cast<float4*>(s_sum + sw * 512 + lane * 4) = x[0];
    *reinterpret_cast<float4*>(s_sum + sw * 512 + 256 + lane * 4) = x[1];
    if (lane % G::Q == 0) s_exp[sw * G::SPW + lane / G::Q] = mr;
  }
  __syncthreads();
  if (u >= (G::R * G::Q + 63) / 64 * 64) return;
  const int jb = c4 / 4, cc = c4 % 4;
  const float f_l = norm_scale(um_l), f_r = norm_scale(um_r), c_l = pow2i(-proj_shift(t_l, z_l)), c_r = pow2i(-proj_shift(t_r, h_r));
  const int d_l = is_l ? add_exp(norm_exp(ue_l, um_l), proj_exp(m_l, t_l, z_l)) : kExpZero;
  const int d_r = is_r ? add_exp(norm_exp(ue_r, um_r), proj_exp(m_r, t_r, h_r)) : kExpZero;
  float amax = 0.0f;
  int m = kExpZero;
  if (fin) {
    if (!root) {
      if (is_l) {
        xl = scaled(f_l, product_at<MI, NI>(s_part, fs + 1, jb, cc));
        *reinterpret_cast<float4*>(g.BH + (p_l - g.S1) * Np + fa) = xl;
      }
      if (is_r) xr = scaled(f_r, product_at<MI, NI>(s_part, fs, jb, cc));
      else xr = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    const int fp = fs / G::SPW, slot = fs % G::SPW;
    m = max(max(d_l, d_r), max(peu, pev));
#pragma unroll
    for (int q = 0; q < G::WP; ++q) m = max(m, s_exp[(fp * G::WP + q) * G::SPW + slot]);
    float4 xu = scaled(exp_coef(peu, m), u0), xv = scaled(exp_coef(pev, m), v0);
#pragma unroll
    for (int q = 0; q < G::WP; ++q) {
      const int fw = fp * G::WP + q;
      const float f = exp_coef(s_exp[fw * G::SPW + slot], m);
      xu = sum4(xu, scaled(f, load4(s_sum + fw * 512 + (slot * G::Q + c4) * 4)));
      xv = sum4(xv, scaled(f, load4(s_sum + fw * 512 + 256 + (slot * G::Q + c4) * 4)));
    }
    axpy(xu, exp_coef(d_l, m), xl, c_l, z1);
    axpy(xv, exp_coef(d_r, m), xr, c_r, h1);
    *reinterpret_cast<float4*>(g.UV + r_c * ld + fa) = xu;
    *reinterpret_cast<float4*>(g.UV + r_c * ld + Np + fa) = xv;
    if (g.UVb) {
      store_planes4(g.UVb, g.planes, g.plane_stride, r_c * ld + fa, xu);
      store_planes4(g.UVb, g.planes, g.plane_stride, r_c * ld + Np + fa, xv);
    }
    amax = fmaxf(fmaxf(fmaxf(fabsf(xu.x), fabsf(xu.y)), fmaxf(fabsf(xu.z), fabsf(xu.w))),
                 fmaxf(fmaxf(fabsf(xv.x), fabsf(xv.y)), fmaxf(fabsf(xv.z), fabsf(xv.w))));
  }
#pragma unroll
  for (int o = 1; o < G::Q; o <<= 1) amax = fmaxf(amax, __shfl_xor(amax, o, 64));
  if (fin && c4 == 0) {
    if (amax > 0.0f && m != kExpZero) atomicMax(&g.umaxb[r_c], __float_as_uint(amax));
    if (blockIdx.x == 0) {
      g.uexp[r_c] = m;
      g.gsc[r_c] = (m == kExpZero || me == kExpZero) ? 0.0f : pow2i(max(m + me, -160));
    }
  }
}

template <int MI, int NJ, bool FWD>
void launch_cfg(const StepArgs& a, hipStream_t st) {
  using G = StepGeo<MI, NJ>;
  constexpr int NI = FWD ? 2 * NJ : NJ;
  constexpr size_t lds = sizeof(float) * (kProdWaves * MI * NI * 256 + kSumWaves * (FWD ? 256 : 512) + kSumWaves * G::SPW);
  void (*kernel)(StepArgs);
  if constexpr (FWD) kernel = &k_step_fwd<MI, NJ>;
  else kernel = &k_step_bwd<MI, NJ>;
  static const bool attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) == hipSuccess;
  (void)attr;
  const int spans = FWD ? a.n_long - a.w : a.n_long - a.w + 2;
  launch_k(kernel, dim3((unsigned)(a.Np / G::NB), (unsigned)((spans + G::R - 2) / (G::R - 1)), (unsigned)a.B), dim3(kStepThreads), lds,
           st, a);
}

}  // namespace

void launch_step(const StepArgs& a, hipStream_t st) {
  if (!a.forward) launch_cfg<1, 1, false>(a, st);
  else if (a.tall) launch_cfg<2, 2, true>(a, st);
  else launch_cfg<1, 1, true>(a, st);
}

}  // namespace spcfg
