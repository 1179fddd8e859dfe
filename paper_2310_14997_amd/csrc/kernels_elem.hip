// Span plan, weight packing, leaf preparation, split-point reductions (forward and reverse) and root
// reductions for the simple-PCFG inside pass on gfx950.  All kernels are deterministic (no atomics).
#include <type_traits>

#include "chart_device.h"

namespace spcfg {

namespace {


// ------------------------------------------------------------------------------------------ span plan
// Width-synchronous schedule (Sec. 3.2, span-level parallelism): rows are ordered by width.  Within a width the
// order is: the prefix spans (i = 0) of all sentences, then the other spans that do not end the sentence
// (sentence by sentence, by start), then the suffix spans (j = n, i > 0).  A prefix span is never a right
// child and a suffix span never a left child, so the first two blocks are exactly the rows whose left projection
// (eta) is used and the last two blocks those whose right projection (zeta) is used: each is one contiguous row
// range for the projection products.  Width 1, and every width when each sentence has its own grammar, keep the
// plain (sentence, start) order; the three tables then describe that order.
//   rowtab[0 * stride + w * B + b]  row of span (0, w) of sentence b (-1 if the sentence is shorter)
//   rowtab[1 * stride + w * B + b]  row of span (1, 1 + w) (the spans 1 .. n-w-1 follow each other)
//   rowtab[2 * stride + w * B + b]  row of span (n - w, n)
// One workgroup per width, four sentences per thread: the first row of a width is a closed sum over the sentences, the places
// within it four scans.  (One workgroup with a thread per width that walked the sentences took 22 us at B = 64, n_max = 40 and
// 4.8 us at B = 1; this one 3.8 and 3.2.)
constexpr int kPlanThreads = 256;
static_assert(4 * kPlanThreads >= kMaxB, "four sentences per thread");
__global__ void __launch_bounds__(kPlanThreads)
k_plan_rowbase(LenArg la, int B, int n_max, int by_sentence, int32_t* __restrict__ lens, int32_t* __restrict__ rowtab,
               int32_t* __restrict__ rootrow, int32_t* __restrict__ counters, int n_counters) {
  __shared__ int4 s_sum[kPlanThreads / 64];
  __shared__ int s_below[kPlanThreads / 64];
  const int w = blockIdx.x + 1, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int stride = (n_max + 1) * B;
  for (int t = blockIdx.x * kPlanThreads + tid; t < n_counters; t += gridDim.x * kPlanThreads) counters[t] = 0;  // GEMM arrival counters
  int cnt[4];
  int4 own = make_int4(0, 0, 0, 0);  // of this thread's sentences: spans, prefix spans, middle spans, suffix spans
  int below = 0;                     // their spans of smaller widths
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int b = 4 * tid + q;
    const int n = b < B ? la.v[b] : 0;
    if (b < B && blockIdx.x == 0) lens[b] = n;
    cnt[q] = max(0, n - w + 1);
    own.x += cnt[q];
    own.y += cnt[q] >= 1 ? 1 : 0;
    own.z += max(0, cnt[q] - 2);
    own.w += cnt[q] >= 2 ? 1 : 0;
    const int v = min(w - 1, n);  // sum of n - u + 1 over the widths u = 1 .. v
    below += v * n - v * (v - 1) / 2;
  }
  int4 x = own;  // inclusive scan over the wavefront, then over the workgroup
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int4 y = make_int4(__shfl_up(x.x, o, 64), __shfl_up(x.y, o, 64), __shfl_up(x.z, o, 64), __shfl_up(x.w, o, 64));
    if (lane >= o) x = make_int4(x.x + y.x, x.y + y.y, x.z + y.z, x.w + y.w);
    below += __shfl_xor(below, o, 64);
  }
  if (lane == 63) { s_sum[wave] = x; s_below[wave] = below; }
  __syncthreads();
  int base = 0;
  int4 at = make_int4(x.x - own.x, x.y - own.y, x.z - own.z, x.w - own.w), all = make_int4(0, 0, 0, 0);
#pragma unroll
  for (int q = 0; q < kPlanThreads / 64; ++q) {
    const int4 y = s_sum[q];
    base += s_below[q];
    if (q < wave) at = make_int4(at.x + y.x, at.y + y.y, at.z + y.z, at.w + y.w);
    all = make_int4(all.x + y.x, all.y + y.y, all.z + y.z, all.w + y.w);
  }
  int* tp = rowtab + w * B;
  int* tm = rowtab + stride + w * B;
  int* ts = rowtab + 2 * stride + w * B;
  // first rows of this thread's next sentence: plain order, or prefix, middle and suffix blocks
  int run = base + at.x, rp = base + at.y, rm = base + all.y + at.z, rs = base + all.y + all.z + at.w;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int b = 4 * tid + q;
    if (b >= B) break;
    const bool any = cnt[q] > 0;
    if (by_sentence || w == 1) {
      tp[b] = any ? run : -1;
      tm[b] = any ? run + 1 : -1;
      ts[b] = any ? run + cnt[q] - 1 : -1;
      if (cnt[q] == 1) rootrow[b] = run;
    } else {
      tp[b] = any ? rp : -1;
      tm[b] = any ? rm : -1;
      ts[b] = any ? (cnt[q] >= 2 ? rs : rp) : -1;  // a span that is the whole sentence is both: it sits in the prefix block
      if (cnt[q] == 1) rootrow[b] = rp;
    }
    run += cnt[q];
    rp += any ? 1 : 0;
    rm += max(0, cnt[q] - 2);
    rs += cnt[q] >= 2 ? 1 : 0;
  }
}

__global__ void k_plan_rows(int B, int stride, const int32_t* __restrict__ lens, const int32_t* __restrict__ rowtab,
                            int32_t* __restrict__ row_b, int32_t* __restrict__ row_i,
                            int32_t* __restrict__ rootmask, uint32_t* __restrict__ tmaxb,
                            uint32_t* __restrict__ umaxb, int32_t* __restrict__ hmaxb,
                            int32_t* __restrict__ zmaxb, uint32_t* __restrict__ colmax, int64_t n_colmax) {
  const int w = blockIdx.x + 1, b = blockIdx.y;
  // (the weight packing takes column maxima into these)
  for (int64_t c = ((int64_t)b * gridDim.x + blockIdx.x) * blockDim.x + threadIdx.x; c < n_colmax;
       c += (int64_t)gridDim.x * gridDim.y * blockDim.x)
    colmax[c] = 0u;
  const int n = lens[b];
  if (w > n) return;
  for (int i = threadIdx.x; i <= n - w; i += blockDim.x) {
    const int r = row_of(rowtab, stride, B, w, b, i, n);
    row_b[r] = b;
    row_i[r] = i;
    rootmask[r] = (w == n) ? 1 : 0;
    tmaxb[r] = 0u;
    umaxb[r] = 0u;
    hmaxb[r] = 0;
    zmaxb[r] = 0;
  }
}

// Rows of width >= 2 listed sentence by sentence (width, then start): the reduction order of the per-sentence
// rule gradients.  Sentence b owns entries [sum_{b'<b} n_b'(n_b'-1)/2, + n_b(n_b-1)/2).
__global__ void k_plan_sentrows(int B, int stride, const int32_t* __restrict__ lens,
                                const int32_t* __restrict__ rowtab, int32_t* __restrict__ sentrows,
                                int32_t* __restrict__ sentoff) {
  const int w = blockIdx.x + 2, b = blockIdx.y;
  const int n = lens[b];
  if (w > n) return;
  int64_t off = 0;
  for (int bb = 0; bb < b; ++bb) off += (int64_t)lens[bb] * (lens[bb] - 1) / 2;
  if (w == 2 && threadIdx.x == 0) sentoff[b] = (int32_t)off;
  // spans of widths 2..w-1 of this sentence: sum_{v=2}^{w-1} (n - v + 1)
  off += (int64_t)(w - 2) * (n + 1) - ((int64_t)w * (w - 1) / 2 - 1);
  for (int i = threadIdx.x; i <= n - w; i += blockDim.x) sentrows[off + i] = row_of(rowtab, stride, B, w, b, i, n);
}

// ------------------------------------------------------------------------------------------ weights
// Stacks [L;R] (Sec. 3.2, kernel fusion: one matrix product for both projections) into zero-padded,
// K-contiguous operands: Wn [2Np x Np] / Wp [2Np x Pp] for the forward products and their transposes
// Wtn [Np x 2Np] / Wtp [Pp x 2Np] for the reverse products.
// One kernel writes every panel of a call, so L and R are read once: a 64 x 64 tile of a factor goes out as it lies and,
// turned in LDS, transposed, four consecutive values per thread and store.  Panels of type FwdT / RevT (float or __bf16; the
// values rounded to it) and NPLF / NPLR bf16 planes (the first pieces of the cut nt::Split3, 2Np*Np resp. 2Np*Pp
// elements apart; shared grammars only); a null panel is left out.  Bound by HBM: N = P = 2048, fp32 panels and three planes
// both ways: 76 us (400 MB, 5.3 TB/s; two kernels with 2- and 4-byte stores took 151 us); the forward ones alone 41 us, without
// planes 22 us.
template <typename T> __device__ __forceinline__ void put_panel4(T* w, int64_t at, float4 v) {
  if (w == nullptr) return;
  if constexpr (sizeof(T) == 4) *reinterpret_cast<float4*>(w + at) = v;
  else store_bf16x4(w, at, v);
}
template <typename FwdT, int NPLF, typename RevT, int NPLR>
__global__ void __launch_bounds__(256)
k_pack_weights(const float* __restrict__ L, const float* __restrict__ R, int N, int P, int Np, int Pp, FwdT* __restrict__ Wn,
               FwdT* __restrict__ Wp, RevT* __restrict__ Wtn, RevT* __restrict__ Wtp, void* __restrict__ Wn3,
               void* __restrict__ Wp3, void* __restrict__ Wtn3, void* __restrict__ Wtp3, uint32_t* __restrict__ colmax) {
  __shared__ float tile[64][65];
  const int64_t M = (int64_t)N + P;
  const int gi = blockIdx.z >> 1, lr = blockIdx.z & 1;  // grammar, left / right factor
  const float* src = (lr ? R : L) + (int64_t)gi * N * M;
  const bool ppart = (int)blockIdx.x * 64 >= Np;  // padded columns: [0, Np) nonterminals, [Np, Np + Pp) preterminals
  const int K = ppart ? Pp : Np, cols = ppart ? P : N;
  const int c0 = (int)blockIdx.x * 64 - (ppart ? Np : 0), a0 = blockIdx.y * 64;
  const int64_t plane = 2 * (int64_t)Np * K, half = (int64_t)lr * Np;
  FwdT* W = ppart ? Wp : Wn;
  RevT* Wt = ppart ? Wtp : Wtn;
  if (W != nullptr) W += gi * plane;
  if (Wt != nullptr) Wt += gi * plane;
  const int x = (threadIdx.x & 15) * 4, y = threadIdx.x >> 4;
  if (ppart) src += N;
  const bool vec = ((uintptr_t)src & 15) == 0 && (M & 3) == 0;
  float4 v[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int a = a0 + y + 16 * q, c = c0 + x;
    const float* s = src + a * M + c;
    v[q] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (a < N) {
      if (vec && c + 4 <= cols) {
        v[q] = *reinterpret_cast<const float4*>(s);
      } else {
        if (c < cols) v[q].x = s[0];
        if (c + 1 < cols) v[q].y = s[1];
        if (c + 2 < cols) v[q].z = s[2];
        if (c + 3 < cols) v[q].w = s[3];
      }
    }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = y + 16 * q;
    tile[r][x] = v[q].x; tile[r][x + 1] = v[q].y; tile[r][x + 2] = v[q].z; tile[r][x + 3] = v[q].w;
    const int64_t at = (half + a0 + r) * K + c0 + x;
    put_panel4(W, at, v[q]);
    void* W3 = ppart ? Wp3 : Wn3;
    if (NPLF > 0 && W3 != nullptr) store_planes4(W3, NPLF, plane, at, v[q]);
  }
  void* Wt3 = ppart ? Wtp3 : Wtn3;
  const bool turned = Wt != nullptr || (NPLR > 0 && Wt3 != nullptr);
  if (!turned && colmax == nullptr) return;
  __syncthreads();
  if (threadIdx.x < 64 && colmax != nullptr) {
    // colmax[(g * 2 + lr) * (Np + Pp) + c] = max_A W[A, c] over the padded columns c (nonterminals [0, Np), then
    // preterminals): feeds the exponent bounds of the projections (see proj_shift).  Weights are non-negative, so the
    // maximum of the bit patterns is the maximum of the values; the array is zeroed by the span plan.
    float m = 0.0f;
#pragma unroll 16
    for (int q = 0; q < 64; ++q) m = fmaxf(m, tile[q][threadIdx.x]);
    if (m > 0.0f)
      atomicMax(colmax + (int64_t)blockIdx.z * (Np + Pp) + (int64_t)blockIdx.x * 64 + threadIdx.x, __float_as_uint(m));
  }
  if (!turned) return;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int c = y + 16 * q;
    const float4 t = make_float4(tile[x][c], tile[x + 1][c], tile[x + 2][c], tile[x + 3][c]);
    const int64_t at = (int64_t)(c0 + c) * (2 * Np) + half + a0 + x;
    put_panel4(Wt, at, t);
    if (NPLR > 0 && Wt3 != nullptr) store_planes4(Wt3, NPLR, plane, at, t);
  }
}

// Operand planes of the rule-gradient product on planes: the three bf16 pieces (or the rounding) of sc[s] * X[s][.] for s < S, zero
// for the rows up to the end of the last step (the product reads whole steps).  One thread per four columns.
__global__ void k_scaled_planes(const float* __restrict__ X, int64_t ld, const float* __restrict__ sc, int64_t S,
                                uint16_t* __restrict__ planes, int64_t plane_stride) {
  const int64_t s = blockIdx.x;
  const int c = (blockIdx.y * blockDim.x + threadIdx.x) * 4;
  if (c >= ld) return;
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  if (s < S) {
    const float f = sc[s];
    const float4 x = *reinterpret_cast<const float4*>(X + s * ld + c);
    v = make_float4(f * x.x, f * x.y, f * x.z, f * x.w);
  }
  store_planes4(planes, plane_stride ? 3 : 1, plane_stride, s * ld + c, v);
}

__global__ void k_zero_plane_rows(uint16_t* __restrict__ planes, int64_t plane_stride, int64_t first, int64_t count) {
  uint16_t* p = planes + (int64_t)blockIdx.y * plane_stride + first;
  for (int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 8; i < count; i += (int64_t)gridDim.x * blockDim.x * 8)
    *reinterpret_cast<uint4*>(p + i) = uint4{0u, 0u, 0u, 0u};  // count and first are multiples of 8 elements
}

// ------------------------------------------------------------------------------------------ leaves
// Base case (Sec. 3.1): the inside vector of token i is its emission vector; it is stored as
// exp(e - max e) with the maximum kept aside (it re-enters only in log Z).
// One workgroup per token.  Bound by its chain (indices, row, two block reductions): up to kLeafHeld * 1024 values stay in registers
// between the maximum and the exponentials, four consecutive ones a thread (P = 2048: 1442 tokens 14 us, 40 tokens
// 6.3 us; two passes over memory with 4-byte loads and 2-byte plane stores took 20 and 11).
constexpr int kLeafHeld = 4;
__device__ __forceinline__ float4 load_upto4(const float* p, int left, bool vec, float fill) {
  if (vec && left >= 4) return *reinterpret_cast<const float4*>(p);
  return make_float4(left > 0 ? p[0] : fill, left > 1 ? p[1] : fill, left > 2 ? p[2] : fill, left > 3 ? p[3] : fill);
}
__global__ void __launch_bounds__(256)
k_leaf_prep(const float* __restrict__ log_emit, int P, int Pp, int n_max, const int32_t* __restrict__ row_b,
            const int32_t* __restrict__ row_i, float* __restrict__ leafE, float* __restrict__ xs,
            int32_t* __restrict__ mexp, uint32_t* __restrict__ tmaxb, uint16_t* __restrict__ leafEb, int planes,
            int64_t plane_stride, const float* __restrict__ colmax, int Np, int per_sentence,
            int32_t* __restrict__ hmaxb, int32_t* __restrict__ zmaxb) {
  __shared__ float red[16];
  __shared__ int redi[16];
  const int r = blockIdx.x, t0 = threadIdx.x * 4;
  const float* e = log_emit + ((int64_t)row_b[r] * n_max + row_i[r]) * P;
  const bool vec = ((uintptr_t)e & 15) == 0;
  const float* cmL = colmax + (int64_t)(per_sentence ? row_b[r] : 0) * 2 * (Np + Pp) + Np;  // preterminal columns of L
  const float* cmR = cmL + (Np + Pp);
  float4 held[kLeafHeld], wl[kLeafHeld], wr[kLeafHeld];
  float mx = -INFINITY;
#pragma unroll
  for (int q = 0; q < kLeafHeld; ++q) {
    const int t = t0 + q * 1024;
    if (t >= Pp) continue;
    held[q] = load_upto4(e + t, P - t, vec, -INFINITY);
    wl[q] = *reinterpret_cast<const float4*>(cmL + t);
    wr[q] = *reinterpret_cast<const float4*>(cmR + t);
    mx = fmaxf(fmaxf(fmaxf(mx, held[q].x), fmaxf(held[q].y, held[q].z)), held[q].w);
  }
  for (int t = t0 + kLeafHeld * 1024; t < Pp; t += 1024) {
    const float4 x = load_upto4(e + t, P - t, vec, -INFINITY);
    mx = fmaxf(fmaxf(fmaxf(mx, x.x), fmaxf(x.y, x.z)), x.w);
  }
  mx = block_max(mx, red);
  const bool dead = !(mx > -INFINITY);
  const float x = dead ? 0.0f : mx;
  int hs = 0, zs = 0;
  auto finish = [&](int t, const float4& l, const float4& a, const float4& b) {
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (!dead) {
      if (t < P) v.x = expf(l.x - x);
      if (t + 1 < P) v.y = expf(l.y - x);
      if (t + 2 < P) v.z = expf(l.z - x);
      if (t + 3 < P) v.w = expf(l.w - x);
    }
    *reinterpret_cast<float4*>(leafE + (int64_t)r * Pp + t) = v;
    hs = max(hs, max(max(bexp_sum(a.x, v.x), bexp_sum(a.y, v.y)), max(bexp_sum(a.z, v.z), bexp_sum(a.w, v.w))));
    zs = max(zs, max(max(bexp_sum(b.x, v.x), bexp_sum(b.y, v.y)), max(bexp_sum(b.z, v.z), bexp_sum(b.w, v.w))));
    if (leafEb) store_planes4(leafEb, planes, plane_stride, (int64_t)r * Pp + t, v);
  };
#pragma unroll
  for (int q = 0; q < kLeafHeld; ++q)
    if (t0 + q * 1024 < Pp) finish(t0 + q * 1024, held[q], wl[q], wr[q]);
  for (int t = t0 + kLeafHeld * 1024; t < Pp; t += 1024)
    finish(t, load_upto4(e + t, P - t, vec, -INFINITY), *reinterpret_cast<const float4*>(cmL + t),
           *reinterpret_cast<const float4*>(cmR + t));
  hs = block_max_i(hs, redi);
  zs = block_max_i(zs, redi);
  if (threadIdx.x == 0) {
    xs[r] = x;
    mexp[r] = dead ? kExpZero : 0;
    tmaxb[r] = dead ? 0u : __float_as_uint(1.0f);  // the largest entry is exactly 1
    hmaxb[r] = hs;
    zmaxb[r] = zs;
  }
}

// ------------------------------------------------------------------------------------------ bands of widths
// Most of the split-point sums of kBandW consecutive widths w0 .. w0 + kBandW - 1 in one pass, before the first of them
// (forward), resp. before the last of them (reverse), is finished.  A launch per width reads two rows per term: span
// (i, j) needs the rows eta(i, .) and zeta(., j), and no other span of its width shares one.  Spans of neighbouring
// widths do: over a tile of kBandI starts x kBandW widths the sums are outer products
//   forward          beta(i, j)      = sum_s eta(i, s) * zeta(s, j)            both children narrower than w0
//   adjoint of eta   adj eta(i, j)   = sum_s adj beta(i, s) * zeta(j, s)       parents wider than the band
//   adjoint of zeta  adj zeta(i, j)  = sum_s adj beta(s, j) * eta(s, i)        parents wider than the band
// so for each s the wavefront loads 4 rows X(i, s) and 7 rows Y(s, j) and uses them for 16 terms: 0.69 rows a term
// instead of 2.  The few terms that touch the band itself (at most 2 * (w - w0) forward, w0 + kBandW - 1 - w a side
// in reverse) are left to the kernel of their width, which adds them to this partial sum; the partial sum lies in the row's
// place in T (UV) with an exponent of its own.  Every term is scaled by an exact power of two against the largest
// exponent of its own sum, as in the kernels of one width.
// A workgroup is one tile; with enough of them each of its up to four wavefronts has 64 nonterminals, with few of them (late
// widths of small batches) sixteen share 64 nonterminals, take every sixteenth group of four s and meet in LDS in wavefront
// order.  blockIdx.x is the block of nonterminals.  A tile shares three of its seven Y rows with its neighbour in blockIdx.y;
// both run on the same XCD, and find them in one L2, only where the grid is a multiple of eight wide (Np a multiple of 2048,
// in the shared form of 512); elsewhere those rows are read from the Infinity Cache or HBM by several XCDs.
// Bound by reading rows: asked for are 6.4 TB/s in reverse and 5.9 forward at B = 32, N = 4096, n = 40, 4.4 in reverse at B = 4, N = 1024,
// n = 137 .. 188.  Split-point sums of a whole pass before and
// after: B = 4, N = 1024, n <= 200: reverse 10.1 -> 6.2 ms, forward 5.6 -> 4.0 ms; B = 32, N = 4096, n = 40: 4.2 -> 2.7 and
// 2.7 -> 1.8 ms.  kBandShare wavefronts per 64 nonterminals: at n = 200 the launches of the last widths fall from 62 us (four
// wavefronts) to 25 us; above kBandMinWaves wavefronts in all a wavefront per 64 nonterminals is the faster form, because the
// tables are built once for four blocks of nonterminals (60 against 85 us there).
constexpr int kBandWaves = 4;    // wavefronts of a workgroup with 64 nonterminals each, at most
constexpr int kBandShare = 16;   // wavefronts of a workgroup that share 64 nonterminals
constexpr int kBandMinWaves = 1536;
enum { BAND_FWD = 0, BAND_ETA = 1, BAND_ZETA = 2 };

// LDS words of the tables for S (a multiple of 4) values of s, and of the wavefronts' partial sums
__host__ __device__ constexpr int band_words(int S) { return 3 * (kBandI + kBandQ) * S; }
constexpr int kBandSumWords = kBandShare * kBandI * kBandW * 64;
constexpr int band_threads(int KS) { return 64 * (KS > 1 ? KS : kBandWaves); }

template <int ROLE, int KS>
__device__ __forceinline__ void split_band(int w0, int b, int i0, int B, int Np, int64_t S1, int stride, int n, int S_max,
                                           const int32_t* __restrict__ rowtab, const float* __restrict__ HZ,
                                           const float* __restrict__ BH, const int32_t* __restrict__ mexp,
                                           const uint32_t* __restrict__ tmaxb, const int32_t* __restrict__ hmaxb,
                                           const int32_t* __restrict__ zmaxb, const int32_t* __restrict__ uexp,
                                           const uint32_t* __restrict__ umaxb, float* __restrict__ out, int64_t out_ld,
                                           int64_t out_row0, int32_t* __restrict__ fwd_exp, const BwdPartExp& bwd_exp, int32_t* lds,
                                           int32_t* s_m) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // KS == 1: every wavefront has 64 nonterminals of its own; KS > 1: KS of them share 64 and take turns in s
  const int waves = KS > 1 ? KS : (int)(blockDim.x >> 6);
  const int a = (KS > 1 ? (int)blockIdx.x : (int)blockIdx.x * waves + wave) * 64 + lane;
  const int al = min(a, Np - 1);  // (a last workgroup may have wavefronts past the end: they load, and store nothing)
  const int wt = w0 + kBandW;
  // the values of s that some span of the tile uses
  const int s_lo = ROLE == BAND_FWD ? i0 + 1 : (ROLE == BAND_ETA ? i0 + wt : 0);
  const int s_hi = ROLE == BAND_FWD ? min(i0 + kBandI + w0 - 2, n - 1) : (ROLE == BAND_ETA ? n : i0 + kBandI - 2);
  const int S = max(0, s_hi - s_lo + 1), S4 = (S + 3) & ~3;
  int32_t* x_row = lds;                        // [kBandI][S_max] row of X
  int32_t* x_max = x_row + kBandI * S_max;     // its exponent
  int32_t* x_app = x_max + kBandI * S_max;     // its exponent as stored (without the shift of a projected half)
  int32_t* y_row = x_app + kBandI * S_max;     // [kBandQ][S_max] row of Y
  int32_t* y_exp = y_row + kBandQ * S_max;
  float* y_sc = reinterpret_cast<float*>(y_exp + kBandQ * S_max);  // scale of its shift
  // a row that has been written, for the entries that take no part (their coefficient is zero)
  const int safe_hz = rowtab[B + b], safe_bh = rowtab[n * B + b];
  // one row of the tables at a time per wavefront; `count` strides of 64 values of s together, so that their two dependent
  // lookups (row, then its exponents) overlap
  auto fill_x = [&](int p, int k0, auto count) {
    constexpr int U = decltype(count)::value;
    const int i = i0 + p;
    int row[U];
    bool ok[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int s = s_lo + k0 + 64 * u;
      ok[u] = ROLE == BAND_FWD ? (s > i && s < i + w0 && s < n)
                               : (ROLE == BAND_ETA ? (s >= i + wt && s <= n) : (s < i && i < n));
      const int width = ROLE == BAND_ZETA ? i - s : s - i, start = ROLE == BAND_ZETA ? s : i;
      row[u] = ok[u] ? row_of(rowtab, stride, B, width, b, start, n) : (ROLE == BAND_ETA ? safe_bh : safe_hz);
    }
    int em[U], ea[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (ROLE == BAND_ETA) {
        em[u] = ea[u] = norm_exp(uexp[row[u]], umaxb[row[u]]);
      } else {
        em[u] = proj_exp(mexp[row[u]], tmaxb[row[u]], hmaxb[row[u]]);
        ea[u] = em[u] == kExpZero ? kExpZero : em[u] - proj_shift(tmaxb[row[u]], hmaxb[row[u]]);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = k0 + 64 * u;
      if (k >= S4) continue;
      x_row[p * S_max + k] = row[u];
      x_max[p * S_max + k] = ok[u] ? em[u] : kExpZero;
      x_app[p * S_max + k] = ok[u] ? ea[u] : kExpZero;
    }
  };
  auto fill_y = [&](int q, int k0, auto count) {
    constexpr int U = decltype(count)::value;
    const int j = i0 + w0 + q;
    int row[U];
    bool ok[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int s = s_lo + k0 + 64 * u;
      // (an end j = 0 exists in the lowest band only, for its width 0, which is no span)
      ok[u] = j <= n && (ROLE == BAND_FWD ? (s > j - w0 && s < j) : (ROLE == BAND_ETA ? (s > j && s <= n && j > 0) : (s <= j - wt)));
      const int width = ROLE == BAND_ETA ? s - j : j - s, start = ROLE == BAND_ETA ? j : s;
      row[u] = ok[u] ? row_of(rowtab, stride, B, width, b, start, n) : (ROLE == BAND_ZETA ? safe_bh : safe_hz);
    }
    int e[U];
    float sc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (ROLE == BAND_ZETA) {
        e[u] = norm_exp(uexp[row[u]], umaxb[row[u]]);
        sc[u] = 1.0f;
      } else {
        e[u] = proj_exp(mexp[row[u]], tmaxb[row[u]], zmaxb[row[u]]);
        sc[u] = pow2i(-proj_shift(tmaxb[row[u]], zmaxb[row[u]]));
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = k0 + 64 * u;
      if (k >= S4) continue;
      y_row[q * S_max + k] = row[u];
      y_exp[q * S_max + k] = ok[u] ? e[u] : kExpZero;
      y_sc[q * S_max + k] = ok[u] ? sc[u] : 0.0f;
    }
  };
  for (int pq = wave; pq < kBandI + kBandQ; pq += waves) {
    if (S4 <= 64) {
      if (pq < kBandI) fill_x(pq, lane, std::integral_constant<int, 1>{});
      else fill_y(pq - kBandI, lane, std::integral_constant<int, 1>{});
    } else {
      for (int k0 = lane; k0 < S4; k0 += 256) {
        if (pq < kBandI) fill_x(pq, k0, std::integral_constant<int, 4>{});
        else fill_y(pq - kBandI, k0, std::integral_constant<int, 4>{});
      }
    }
  }
  __syncthreads();
  for (int pair = tid >> 4; pair < kBandI * kBandW; pair += waves * 4) {  // largest exponent of a span's sum: sixteen threads
    const int p = pair / kBandW, q = p + pair % kBandW;
    int m = kExpZero;
    for (int k = tid & 15; k < S4; k += 16) m = max(m, add_exp(x_max[p * S_max + k], y_exp[q * S_max + k]));
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o, 64));
    if ((tid & 15) == 0) s_m[pair] = m;
  }
  __syncthreads();

  float acc[kBandI][kBandW];
  int neg_m[kBandI][kBandW];
#pragma unroll
  for (int p = 0; p < kBandI; ++p)
#pragma unroll
    for (int d = 0; d < kBandW; ++d) {
      acc[p][d] = 0.0f;
      const int m = __builtin_amdgcn_readfirstlane(s_m[p * kBandW + d]);
      neg_m[p][d] = m == kExpZero ? 0 : -m;
    }
  const int64_t ldx = ROLE == BAND_ETA ? Np : 2 * (int64_t)Np, ldy = ROLE == BAND_ZETA ? Np : 2 * (int64_t)Np;
  const float* xb = ROLE == BAND_ETA ? BH : HZ;                              // eta is the first half of a row of HZ
  const float* yb = ROLE == BAND_ZETA ? BH : HZ + Np;                        // zeta the second
  const int64_t xs = ROLE == BAND_ETA ? S1 : 0, ys = ROLE == BAND_ZETA ? S1 : 0;  // BH starts at the rows of width 2
  for (int k = KS > 1 ? wave * 4 : 0; k < S4; k += KS * 4) {
    float x[kBandI][4], y[kBandQ][4];
    int4 xa[kBandI], ye[kBandQ];
#pragma unroll
    for (int p = 0; p < kBandI; ++p) {
      const int4 r = *reinterpret_cast<const int4*>(x_row + p * S_max + k);
      xa[p] = *reinterpret_cast<const int4*>(x_app + p * S_max + k);
      x[p][0] = (xb + (__builtin_amdgcn_readfirstlane(r.x) - xs) * ldx)[al];
      x[p][1] = (xb + (__builtin_amdgcn_readfirstlane(r.y) - xs) * ldx)[al];
      x[p][2] = (xb + (__builtin_amdgcn_readfirstlane(r.z) - xs) * ldx)[al];
      x[p][3] = (xb + (__builtin_amdgcn_readfirstlane(r.w) - xs) * ldx)[al];
    }
#pragma unroll
    for (int q = 0; q < kBandQ; ++q) {
      const int4 r = *reinterpret_cast<const int4*>(y_row + q * S_max + k);
      ye[q] = *reinterpret_cast<const int4*>(y_exp + q * S_max + k);
      y[q][0] = (yb + (__builtin_amdgcn_readfirstlane(r.x) - ys) * ldy)[al];
      y[q][1] = (yb + (__builtin_amdgcn_readfirstlane(r.y) - ys) * ldy)[al];
      y[q][2] = (yb + (__builtin_amdgcn_readfirstlane(r.z) - ys) * ldy)[al];
      y[q][3] = (yb + (__builtin_amdgcn_readfirstlane(r.w) - ys) * ldy)[al];
    }
#pragma unroll
    for (int q = 0; q < kBandQ; ++q) {
      const float4 sc = *reinterpret_cast<const float4*>(y_sc + q * S_max + k);
      y[q][0] *= sc.x; y[q][1] *= sc.y; y[q][2] *= sc.z; y[q][3] *= sc.w;
    }
#pragma unroll
    for (int p = 0; p < kBandI; ++p)
#pragma unroll
      for (int d = 0; d < kBandW; ++d) {
        const int q = p + d;
        acc[p][d] = fmaf(__builtin_amdgcn_ldexpf(x[p][0], xa[p].x + ye[q].x + neg_m[p][d]), y[q][0], acc[p][d]);
        acc[p][d] = fmaf(__builtin_amdgcn_ldexpf(x[p][1], xa[p].y + ye[q].y + neg_m[p][d]), y[q][1], acc[p][d]);
        acc[p][d] = fmaf(__builtin_amdgcn_ldexpf(x[p][2], xa[p].z + ye[q].z + neg_m[p][d]), y[q][2], acc[p][d]);
        acc[p][d] = fmaf(__builtin_amdgcn_ldexpf(x[p][3], xa[p].w + ye[q].w + neg_m[p][d]), y[q][3], acc[p][d]);
      }
  }
  if (KS > 1) {
    __syncthreads();  // the tables have been read: their place holds the wavefronts' sums now
    float* sum = reinterpret_cast<float*>(lds);
#pragma unroll
    for (int p = 0; p < kBandI; ++p)
#pragma unroll
      for (int d = 0; d < kBandW; ++d) sum[((wave * kBandI + p) * kBandW + d) * 64 + lane] = acc[p][d];
    __syncthreads();
#pragma unroll
    for (int pair = 0; pair < kBandI * kBandW; ++pair) {
      if (pair % KS != wave) continue;  // each wavefront finishes its share of the spans
      float t = 0.0f;
#pragma unroll
      for (int q = 0; q < KS; ++q) t += sum[(q * kBandI * kBandW + pair) * 64 + lane];
      acc[pair / kBandW][pair % kBandW] = t;
    }
  }
#pragma unroll
  for (int p = 0; p < kBandI; ++p)
#pragma unroll
    for (int d = 0; d < kBandW; ++d) {
      const int i = i0 + p, w = w0 + d;
      if (KS > 1 && (p * kBandW + d) % KS != wave) continue;
      // no such span (the lowest band's width 0 among them); the root span has no parents
      if (w == 0 || i + w > n || (ROLE != BAND_FWD && w == n)) continue;
      const int r = row_of(rowtab, stride, B, w, b, i, n);
      if (a < Np) out[(r - out_row0) * out_ld + a] = acc[p][d];
      if (blockIdx.x == 0 && lane == 0 && (KS > 1 || wave == 0)) {
        if (ROLE == BAND_FWD) fwd_exp[r] = s_m[p * kBandW + d];
        else bwd_exp.put(ROLE == BAND_ZETA, r, S1, Np, s_m[p * kBandW + d]);
      }
    }
}

template <int KS>
__global__ void __launch_bounds__(band_threads(KS))
k_split_band_fwd(int w0, int B, int Np, int64_t S1, int stride, int S_max, const int32_t* __restrict__ lens,
                 const int32_t* __restrict__ rowtab, const float* __restrict__ HZ, const int32_t* __restrict__ mexp,
                 const uint32_t* __restrict__ tmaxb, const int32_t* __restrict__ hmaxb, const int32_t* __restrict__ zmaxb,
                 float* __restrict__ T, int32_t* __restrict__ part_exp) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int32_t s_m[kBandI * kBandW];
  const int b = blockIdx.z, n = lens[b], i0 = blockIdx.y * kBandI;
  if (i0 + w0 > n) return;
  split_band<BAND_FWD, KS>(w0, b, i0, B, Np, S1, stride, n, S_max, rowtab, HZ, nullptr, mexp,
                       tmaxb, hmaxb, zmaxb, nullptr, nullptr, T, Np, S1, part_exp, BwdPartExp{}, reinterpret_cast<int32_t*>(smem), s_m);
}

// blockIdx.z: sentence, and which of the two adjoints
template <int KS>
__global__ void __launch_bounds__(band_threads(KS))
k_split_band_bwd(int w0, int B, int Np, int64_t S1, int stride, int S_max, const int32_t* __restrict__ lens,
                 const int32_t* __restrict__ rowtab, const float* __restrict__ HZ, const float* __restrict__ BH,
                 const int32_t* __restrict__ mexp, const uint32_t* __restrict__ tmaxb, const int32_t* __restrict__ hmaxb,
                 const int32_t* __restrict__ zmaxb, const int32_t* __restrict__ uexp, const uint32_t* __restrict__ umaxb,
                 float* __restrict__ UV, BwdPartExp part_exp) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int32_t s_m[kBandI * kBandW];
  const int b = blockIdx.z >> 1, n = lens[b], i0 = blockIdx.y * kBandI;
  if (i0 + w0 > n) return;
  if ((blockIdx.z & 1) == 0)
    split_band<BAND_ETA, KS>(w0, b, i0, B, Np, S1, stride, n, S_max, rowtab, HZ, BH, mexp, tmaxb, hmaxb, zmaxb, uexp, umaxb, UV,
                         2 * (int64_t)Np, 0, nullptr, part_exp, reinterpret_cast<int32_t*>(smem), s_m);
  else
    split_band<BAND_ZETA, KS>(w0, b, i0, B, Np, S1, stride, n, S_max, rowtab, HZ, BH, mexp, tmaxb, hmaxb, zmaxb, uexp, umaxb,
                          UV + Np, 2 * (int64_t)Np, 0, nullptr, part_exp, reinterpret_cast<int32_t*>(smem), s_m);
}

// ------------------------------------------------------------------------------------------ forward split
// beta_ij = sum_k eta_ik * zeta_kj (Sec. 3.1 vector form) for every span of one width, in the scaled
// representation: T = sum_k 2^(d_k - m) etat_ik * zetat_kj with d_k = e_ik + e_kj, m = max_k d_k.
// One wavefront per (span, block of 256 nonterminals): split-point rows and coefficients are staged in
// LDS, eight split points (16 row loads) are in flight per lane, the per-span maximum that drives the
// rescaling of Sec. 3.2 is a wavefront reduction followed by one integer atomicMax, and nothing per split
// point goes to HBM.  The normalisation itself is applied by the projection GEMM's epilogue.
// KG = 4 is the shape for launches with few spans and more than 64 split points, which would leave most of the chip idle: the
// wavefront covers 64 nonterminals and its four groups of 16 lanes take every fourth split point, so four times as many
// wavefronts run and each walks a quarter of the split points.  Nearly all such widths lie in bands; what is left is mostly the
// last width of a batch whose longest sentence has a multiple of four words (choose_bands ends below it).  A band for that one
// width costs a launch more: split sums of one sentence of 72 words 371 instead of 362 us at N = 64, 501 instead of 491 at 2048.
constexpr int kChunk = 256;  // nonterminals per wavefront (4 per lane) when KG = 1

template <int KG>
__global__ void __launch_bounds__(64)
k_split_fwd(int w, int64_t row0, int B, int Np, int64_t S1, int stride, const int32_t* __restrict__ lens,
            const int32_t* __restrict__ rowtab, const int32_t* __restrict__ row_b,
            const int32_t* __restrict__ row_i, const float* __restrict__ HZ,
            float* __restrict__ T, int32_t* __restrict__ mexp, uint32_t* __restrict__ tmaxb, void* __restrict__ Tb,
            int planes, int64_t plane_stride, int32_t* __restrict__ hmaxb, int32_t* __restrict__ zmaxb,
            const float* __restrict__ colmax, int Pp, int per_sentence, int w0, const int32_t* __restrict__ part_exp) {
  extern __shared__ __align__(16) unsigned char smem[];
  // split points of this launch: all w - 1, or (w0 > 0) those with a child of width w0 or more, the rest lies summed in T
  const int nk = w0 > 0 ? 2 * (w - w0) : w - 1;
  float* s_c = reinterpret_cast<float*>(smem);             // [nk] coefficient of the left child's eta
  float* s_cz = s_c + nk;                                  // [nk] coefficient of the right child's zeta
  int32_t* s_l = reinterpret_cast<int32_t*>(s_cz + nk);    // [nk] row of the left child
  int32_t* s_r = s_l + nk;                                 // [nk] row of the right child
  const int lane = threadIdx.x;
  const int64_t r = row0 + blockIdx.x;
  const int b = row_b[r], i = row_i[r];
  const int n = lens[b];
  const int pe = w0 > 0 ? part_exp[r] : kExpZero;
  int dmax = pe;
  for (int t = lane; t < nk; t += 64) {
    const int k = (w0 > 0 && t >= w - w0) ? t + 2 * w0 - w : t + 1;
    const int lr = row_of(rowtab, stride, B, k, b, i, n);          // span (i, i+k)
    const int rr = row_of(rowtab, stride, B, w - k, b, i + k, n);  // span (i+k, i+w)
    s_l[t] = lr;
    s_r[t] = rr;
    const int d = add_exp(proj_exp(mexp[lr], tmaxb[lr], hmaxb[lr]), proj_exp(mexp[rr], tmaxb[rr], zmaxb[rr]));
    s_c[t] = __int_as_float(d);
    s_cz[t] = __int_as_float(proj_shift(tmaxb[lr], hmaxb[lr]));  // eta's shift, used once m is known
    dmax = max(dmax, d);
  }
  const int m = wave_max_i(dmax);
  __syncthreads();
  // the term of split point k is 2^(d_k - m) * (2^-gh eta) * (2^-gz zeta): the first two factors go with eta
  // (coefficient 2^(d_k - m - gh)), the last with zeta (coefficient 2^-gz); both products stay at or below 1
  for (int k = lane; k < nk; k += 64) {
    const int d = __float_as_int(s_c[k]);
    const int gh = __float_as_int(s_cz[k]);
    s_c[k] = (d == kExpZero) ? 0.0f : pow2i(d - m - gh);
    s_cz[k] = (d == kExpZero) ? 0.0f : pow2i(-proj_shift(tmaxb[s_r[k]], zmaxb[s_r[k]]));
  }
  __syncthreads();

  const int64_t ld = 2 * (int64_t)Np;
  constexpr int LG = 64 / KG;          // lanes per split-point group
  const int kg = lane / LG;            // this lane's group: it takes the split points kg, kg + KG, ...
  const int a = blockIdx.y * (LG * 4) + (lane % LG) * 4;
  float tmax = 0.0f;
  int hsum = 0, zsum = 0;
  if (a < Np) {  // always true for KG > 1 (the padded width is a multiple of 64): the shuffles below see every lane
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    if (w0 > 0 && kg == 0) {
      const float c = pe == kExpZero ? 0.0f : pow2i(pe - m);
      const float4 t = *reinterpret_cast<const float4*>(T + (r - S1) * Np + a);
      acc = make_float4(c * t.x, c * t.y, c * t.z, c * t.w);
    }
    const float* hz_l = HZ + a;
    const float* hz_r = HZ + Np + a;
    int k = 0;
    for (; k + 8 * KG <= nk; k += 8 * KG) {
      float4 h[8], z[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        h[u] = *reinterpret_cast<const float4*>(hz_l + s_l[k + u * KG + kg] * ld);
        z[u] = *reinterpret_cast<const float4*>(hz_r + s_r[k + u * KG + kg] * ld);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const float c = s_c[k + u * KG + kg], cz = s_cz[k + u * KG + kg];
        acc.x = fmaf(c * h[u].x, cz * z[u].x, acc.x);
        acc.y = fmaf(c * h[u].y, cz * z[u].y, acc.y);
        acc.z = fmaf(c * h[u].z, cz * z[u].z, acc.z);
        acc.w = fmaf(c * h[u].w, cz * z[u].w, acc.w);
      }
    }
    for (; k < nk; k += 4 * KG) {  // remainder in masked groups of four: no serial chain of dependent loads
      float4 h[4], z[4];
      float c[4], cz[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int idx = k + u * KG + kg;
        const int kk = min(idx, nk - 1);
        c[u] = (idx < nk) ? s_c[kk] : 0.0f;
        cz[u] = s_cz[kk];
        h[u] = *reinterpret_cast<const float4*>(hz_l + s_l[kk] * ld);
        z[u] = *reinterpret_cast<const float4*>(hz_r + s_r[kk] * ld);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        acc.x = fmaf(c[u] * h[u].x, cz[u] * z[u].x, acc.x);
        acc.y = fmaf(c[u] * h[u].y, cz[u] * z[u].y, acc.y);
        acc.z = fmaf(c[u] * h[u].z, cz[u] * z[u].z, acc.z);
        acc.w = fmaf(c[u] * h[u].w, cz[u] * z[u].w, acc.w);
      }
    }
    if (KG > 1) {  // sum of the groups' partial sums, in a fixed order
#pragma unroll
      for (int o = LG; o < 64; o <<= 1) {
        acc.x += __shfl_xor(acc.x, o, 64);
        acc.y += __shfl_xor(acc.y, o, 64);
        acc.z += __shfl_xor(acc.z, o, 64);
        acc.w += __shfl_xor(acc.w, o, 64);
      }
    }
    if (kg == 0) {
      *reinterpret_cast<float4*>(T + (r - S1) * Np + a) = acc;
      if (Tb) store_planes4(Tb, planes, plane_stride, (r - S1) * Np + a, acc);
    }
    tmax = fmaxf(fmaxf(acc.x, acc.y), fmaxf(acc.z, acc.w));
    // exponent bounds of this vector's two projections (see proj_shift)
    const float* cmL = colmax + (int64_t)(per_sentence ? b : 0) * 2 * (Np + Pp) + a;
    const float4 wl = *reinterpret_cast<const float4*>(cmL), wr = *reinterpret_cast<const float4*>(cmL + Np + Pp);
    hsum = max(max(bexp_sum(wl.x, acc.x), bexp_sum(wl.y, acc.y)), max(bexp_sum(wl.z, acc.z), bexp_sum(wl.w, acc.w)));
    zsum = max(max(bexp_sum(wr.x, acc.x), bexp_sum(wr.y, acc.y)), max(bexp_sum(wr.z, acc.z), bexp_sum(wr.w, acc.w)));
  }
  tmax = wave_max(tmax);
  hsum = wave_max_i(hsum);
  zsum = wave_max_i(zsum);
  if (lane == 0) {
    if (tmax > 0.0f && m != kExpZero) atomicMax(&tmaxb[r], __float_as_uint(tmax));
    if (hsum > 0 && m != kExpZero) atomicMax(&hmaxb[r], hsum);
    if (zsum > 0 && m != kExpZero) atomicMax(&zmaxb[r], zsum);
    if (blockIdx.y == 0) mexp[r] = m;
  }
}

// Sentence and start of a workgroup's span: from the block index alone (starts > 0: a workgroup for every start of the longest
// sentence, in every sentence), or from the row tables, one dependent load more and no workgroup without a span.
__device__ __forceinline__ void few_span(int starts, int64_t row0, const int32_t* __restrict__ row_b,
                                         const int32_t* __restrict__ row_i, int* b, int* i) {
  if (starts > 0) {
    *b = blockIdx.x / starts;
    *i = blockIdx.x % starts;
  } else {
    *b = row_b[row0 + blockIdx.x];
    *i = row_i[row0 + blockIdx.x];
  }
}

// The same sum for launches with too few spans to fill the chip, where a launch costs its chain of dependent loads and not
// its bytes: the split points of a (span, 256 nonterminals) are shared by the W wavefronts of one workgroup, U to each, and
// all row loads of the span are in flight at once (W * U >= split points, at most 64).  The staging needs no LDS: in
// every wavefront lane t holds split point t's rows and exponents, the row addresses go out (readlane) before the
// exponents are looked up, and the partial sums meet in LDS in a fixed order.  Every dependent load costs most of a
// microsecond here (what the launch before wrote is in no L2), so sentence and start come from the block index and row
// tables are read for both cases that the sentence's length decides: three loads deep instead of six.
template <int W, int U>
__global__ void __launch_bounds__(64 * W)
k_split_fwd_few(int w, int starts, int64_t row0, const int32_t* __restrict__ row_b, const int32_t* __restrict__ row_i,
                int B, int Np, int64_t S1, int stride, const int32_t* __restrict__ lens,
                const int32_t* __restrict__ rowtab, const float* __restrict__ HZ,
                float* __restrict__ T, int32_t* __restrict__ mexp, uint32_t* __restrict__ tmaxb, void* __restrict__ Tb,
                int planes, int64_t plane_stride, int32_t* __restrict__ hmaxb, int32_t* __restrict__ zmaxb,
                const float* __restrict__ colmax, int Pp, int per_sentence, int w0, const int32_t* __restrict__ part_exp) {
  static_assert(W * U <= 64, "one lane per split point");
  __shared__ float4 s_part[W > 1 ? W - 1 : 1][64];
  const int nk = w0 > 0 ? 2 * (w - w0) : w - 1;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  int b, i;
  few_span(starts, row0, row_b, row_i, &b, &i);
  const int n = lens[b];
  // (row_of with the length's part left for later: children (i, i+k) never end the sentence, (i+k, i+w) never begin it)
  const int* tab = rowtab + b;
  const int own0 = tab[(i == 0 ? 0 : stride) + w * B] + (i == 0 ? 0 : i - 1), own2 = tab[2 * stride + w * B];
  int lr = 0, rr = 0, rr2 = 0;
  if (nk > 0) {
    const int t = min(lane, nk - 1);
    const int k = (w0 > 0 && t >= w - w0) ? t + 2 * w0 - w : t + 1;
    lr = tab[(i == 0 ? 0 : stride) + k * B] + (i == 0 ? 0 : i - 1);
    rr = tab[stride + (w - k) * B] + i + k - 1;
    rr2 = tab[2 * stride + (w - k) * B];
  }
  if (i + w > n) return;  // (uniform over the workgroup: this sentence has fewer spans)
  const int64_t r = i > 0 && i + w == n ? own2 : own0;
  if (i + w == n) rr = rr2;
  const int64_t ld = 2 * (int64_t)Np;
  const int col = blockIdx.y * kChunk + lane * 4;
  const int a = min(col, Np - 4);  // lanes past the end load the last columns and store nothing
  float4 h[U], z[U];
  const bool some = wave < nk;  // (a wavefront without a split point of its own)
  if (some) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = min(wave + u * W, nk - 1);
      h[u] = *reinterpret_cast<const float4*>(HZ + (int64_t)__builtin_amdgcn_readlane(lr, t) * ld + a);
      z[u] = *reinterpret_cast<const float4*>(HZ + (int64_t)__builtin_amdgcn_readlane(rr, t) * ld + Np + a);
    }
  }
  const int pe = w0 > 0 ? part_exp[r] : kExpZero;
  float4 first = make_float4(0.f, 0.f, 0.f, 0.f), wl = first, wr = first;
  if (wave == 0) {
    if (w0 > 0) first = *reinterpret_cast<const float4*>(T + (r - S1) * Np + a);
    const float* cmL = colmax + (int64_t)(per_sentence ? b : 0) * 2 * (Np + Pp) + a;
    wl = *reinterpret_cast<const float4*>(cmL);
    wr = *reinterpret_cast<const float4*>(cmL + Np + Pp);
  }
  int d = kExpZero, gh = 0, gz = 0;
  if (nk > 0) {
    const uint32_t tl = tmaxb[lr], tr = tmaxb[rr];
    const int hl = hmaxb[lr], zr = zmaxb[rr];
    d = add_exp(proj_exp(mexp[lr], tl, hl), proj_exp(mexp[rr], tr, zr));
    gh = proj_shift(tl, hl);
    gz = proj_shift(tr, zr);
  }
  const int m = max(wave_max_i(d), pe);
  const int c = __float_as_int(d == kExpZero ? 0.0f : pow2i(d - m - gh));
  const int cz = __float_as_int(d == kExpZero ? 0.0f : pow2i(-gz));
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  if (wave == 0 && w0 > 0) {
    const float cp = pe == kExpZero ? 0.0f : pow2i(pe - m);
    acc = make_float4(cp * first.x, cp * first.y, cp * first.z, cp * first.w);
  }
  if (some) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = wave + u * W;
      if (t < nk) {
        const float ct = __int_as_float(__builtin_amdgcn_readlane(c, t)), czt = __int_as_float(__builtin_amdgcn_readlane(cz, t));
        acc.x = fmaf(ct * h[u].x, czt * z[u].x, acc.x);
        acc.y = fmaf(ct * h[u].y, czt * z[u].y, acc.y);
        acc.z = fmaf(ct * h[u].z, czt * z[u].z, acc.z);
        acc.w = fmaf(ct * h[u].w, czt * z[u].w, acc.w);
      }
    }
  }
  if (W > 1) {
    if (wave > 0) s_part[wave - 1][lane] = acc;
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int q = 0; q < W - 1; ++q) {
      const float4 o = s_part[q][lane];
      acc.x += o.x; acc.y += o.y; acc.z += o.z; acc.w += o.w;
    }
  }
  float tmax = 0.0f;
  int hsum = 0, zsum = 0;
  if (col < Np) {
    *reinterpret_cast<float4*>(T + (r - S1) * Np + a) = acc;
    if (Tb) store_planes4(Tb, planes, plane_stride, (r - S1) * Np + a, acc);
    tmax = fmaxf(fmaxf(acc.x, acc.y), fmaxf(acc.z, acc.w));
    hsum = max(max(bexp_sum(wl.x, acc.x), bexp_sum(wl.y, acc.y)), max(bexp_sum(wl.z, acc.z), bexp_sum(wl.w, acc.w)));
    zsum = max(max(bexp_sum(wr.x, acc.x), bexp_sum(wr.y, acc.y)), max(bexp_sum(wr.z, acc.z), bexp_sum(wr.w, acc.w)));
  }
  tmax = wave_max(tmax);
  hsum = wave_max_i(hsum);
  zsum = wave_max_i(zsum);
  if (lane == 0) {
    if (tmax > 0.0f && m != kExpZero) atomicMax(&tmaxb[r], __float_as_uint(tmax));
    if (hsum > 0 && m != kExpZero) atomicMax(&hmaxb[r], hsum);
    if (zsum > 0 && m != kExpZero) atomicMax(&zmaxb[r], zsum);
    if (blockIdx.y == 0) mexp[r] = m;
  }
}

// ------------------------------------------------------------------------------------------ root
// Z = sum_A pi(S->A) beta_0n[A] (rule S -> A, Sec. 2).
// Bound by its chain of lookups: up to kRootHeld * 256 values of the row and of the root's scores are asked for before the
// maximum of the scores is known (N = 2048: 5.3 us for 64 sentences, 4.1 for one; two loops one after the other took 15 and 9.8).
constexpr int kRootHeld = 8;
__global__ void __launch_bounds__(256)
k_root_fwd(int B, int N, int Np, int64_t S1, const int32_t* __restrict__ lens, const int32_t* __restrict__ rowbase,
           const int32_t* __restrict__ rootrow, const float* __restrict__ log_root, const float* __restrict__ T,
           const int32_t* __restrict__ mexp, const uint32_t* __restrict__ tmaxb, const float* __restrict__ xs,
           float* __restrict__ logZ, float* __restrict__ ztil, float* __restrict__ rmaxs, int64_t root_stride) {
  __shared__ float redf[16];
  __shared__ double redd[16], redx[16];
  const int b = blockIdx.x, tid = threadIdx.x;
  log_root += b * root_stride;
  const int64_t r = rootrow[b];
  const int n = lens[b];
  const int leaf0 = rowbase[1 * B + b];  // width 1 keeps the (sentence, start) order
  float lr[kRootHeld], th[kRootHeld];
  float rm = -INFINITY;
#pragma unroll
  for (int q = 0; q < kRootHeld; ++q) {
    const int a = tid + q * 256;
    lr[q] = a < N ? log_root[a] : -INFINITY;
    rm = fmaxf(rm, lr[q]);
  }
  for (int a = tid + kRootHeld * 256; a < N; a += 256) rm = fmaxf(rm, log_root[a]);
  const float* t = T + (r - S1) * Np;
#pragma unroll
  for (int q = 0; q < kRootHeld; ++q) th[q] = tid + q * 256 < N ? t[tid + q * 256] : 0.0f;
  const uint32_t tb = tmaxb[r];
  const int me = mexp[r];
  double sx = 0.0;
  for (int i = tid; i < n; i += 256) sx += (double)xs[leaf0 + i];
  rm = block_max(rm, redf);
  const bool deadroot = !(rm > -INFINITY);
  const float rmx = deadroot ? 0.0f : rm;
  const float fs = norm_scale(tb);
  double z = 0.0;
#pragma unroll
  for (int q = 0; q < kRootHeld; ++q)
    if (tid + q * 256 < N) z += (double)expf(lr[q] - rmx) * (double)(th[q] * fs);
  for (int a = tid + kRootHeld * 256; a < N; a += 256) z += (double)expf(log_root[a] - rmx) * (double)(t[a] * fs);
  z = block_sum_d(z, redd);
  sx = block_sum_d(sx, redx);
  if (tid == 0) {
    const int e = norm_exp(me, tb);
    const bool dead = deadroot || e == kExpZero || !(z > 0.0);
    logZ[b] = dead ? -INFINITY : (float)((double)rmx + log(z) + (double)e * 0.6931471805599453094 + sx);
    ztil[b] = dead ? 0.0f : (float)z;
    rmaxs[b] = rmx;
  }
}

// d logZ / d beta_0n[A] = pi(S->A) / Z.  Scaled adjoint of the root span: BH = g * r[A] / Zt, exponent -e_0n.
__global__ void k_root_bwd(int N, int Np, int64_t S1, const int32_t* __restrict__ rootrow,
                           const float* __restrict__ log_root, const float* __restrict__ grad_logZ,
                           const float* __restrict__ ztil, const float* __restrict__ rmaxs,
                           const int32_t* __restrict__ mexp, const uint32_t* __restrict__ tmaxb,
                           float* __restrict__ BH, float* __restrict__ UV, int32_t* __restrict__ uexp,
                           uint32_t* __restrict__ umaxb, float* __restrict__ gsc, int64_t root_stride,
                           uint16_t* __restrict__ UVb, int planes, int64_t plane_stride) {
  const int b = blockIdx.x;
  log_root += b * root_stride;
  const int64_t r = rootrow[b];
  const float g = grad_logZ ? grad_logZ[b] : 1.0f;
  const float zt = ztil[b];
  const bool dead = !(zt > 0.0f) || g == 0.0f;
  const float s = dead ? 0.0f : g / zt;
  const float rmx = rmaxs[b];
  float* bh = BH + (r - S1) * Np;
  float* uv = UV + r * 2 * (int64_t)Np;
  for (int a = threadIdx.x; a < Np; a += blockDim.x) {
    bh[a] = (a < N && !dead) ? s * expf(log_root[a] - rmx) : 0.0f;
    uv[a] = 0.0f;
    uv[Np + a] = 0.0f;
    if (UVb) {
      for (int pl = 0; pl < planes; ++pl) {  // bf16 zero is the all-zero bit pattern
        UVb[pl * plane_stride + r * 2 * (int64_t)Np + a] = 0;
        UVb[pl * plane_stride + r * 2 * (int64_t)Np + Np + a] = 0;
      }
    }
  }
  if (threadIdx.x == 0) {
    // consumers read the exponent of BH as uexp + norm_shift(umaxb); 0.5 has shift 0
    uexp[r] = dead ? kExpZero : -norm_exp(mexp[r], tmaxb[r]);
    umaxb[r] = dead ? 0u : __float_as_uint(0.5f);
    gsc[r] = 0.0f;
  }
}

// grad_log_root[A] = sum_b g_b * pi(S->A) beta_0n[A] / Z_b  (root posteriors); fixed summation order.
__global__ void k_grad_log_root(int B, int N, int Np, int64_t S1, const int32_t* __restrict__ rootrow,
                                const float* __restrict__ log_root, const float* __restrict__ grad_logZ,
                                const float* __restrict__ ztil, const float* __restrict__ rmaxs,
                                const float* __restrict__ T, const uint32_t* __restrict__ tmaxb,
                                float* __restrict__ grad_log_root, int accumulate, int per_sentence) {
  const int a = blockIdx.x * blockDim.x + threadIdx.x;
  if (a >= N) return;
  int b_lo = 0, b_hi = B;
  if (per_sentence) {  // one root vector and one gradient per sentence: no sum over the batch
    b_lo = blockIdx.y; b_hi = b_lo + 1;
    log_root += (int64_t)b_lo * N;
    grad_log_root += (int64_t)b_lo * N;
  }
  const float lr = log_root[a];
  float acc = 0.0f;
  for (int b0 = b_lo; b0 < b_hi; b0 += 8) {  // eight sentences' loads in flight; summed in sentence order
    float t[8], coef[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int b = min(b0 + u, b_hi - 1);
      const float zt = ztil[b];
      const int64_t r = rootrow[b];
      const float g = grad_logZ ? grad_logZ[b] : 1.0f;
      const bool on = b0 + u < b_hi && zt > 0.0f;
      t[u] = T[(r - S1) * Np + a] * norm_scale(tmaxb[r]);  // the root span's inside vector: always written, finite
      coef[u] = on ? g * expf(lr - rmaxs[b]) / zt : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) acc += coef[u] * t[u];
  }
  grad_log_root[a] = accumulate ? grad_log_root[a] + acc : acc;
}

// ------------------------------------------------------------------------------------------ reverse split
// Reverse of the split-point sum in gather form (Sec. 3.2 "Recomputation": the per-split products are
// recomputed from the stored projections, never saved).  For the span (i,j):
//   adjoint of eta_ij  = sum_{j'>j} adj(beta_ij') * zeta_jj'     (as the left child of (i,j'))
//   adjoint of zeta_ij = sum_{i'<i} adj(beta_i'j) * eta_i'i      (as the right child of (i',j))
// Both are written with one common exponent so that they can be projected back through [L;R] together;
// as in the forward pass one wavefront handles (span, 256 nonterminals) and the normalisation by the
// largest magnitude is left to the GEMM epilogue.
__global__ void __launch_bounds__(64)
k_split_bwd(int w, int64_t row0, int B, int Np, int64_t S1, int stride, const int32_t* __restrict__ lens,
            const int32_t* __restrict__ rowtab, const int32_t* __restrict__ row_b,
            const int32_t* __restrict__ row_i, const int32_t* __restrict__ rootmask,
            const float* __restrict__ HZ, const float* __restrict__ BH, const int32_t* __restrict__ mexp,
            const uint32_t* __restrict__ tmaxb, float* __restrict__ UV, int32_t* __restrict__ uexp,
            uint32_t* __restrict__ umaxb, float* __restrict__ gsc, void* __restrict__ UVb, int planes,
            int64_t plane_stride, const int32_t* __restrict__ hmaxb, const int32_t* __restrict__ zmaxb, int wt,
            const float* __restrict__ xs) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x;
  const int64_t r = row0 + blockIdx.x;
  // (asked for with the row's indices: the row's place in BH is in no cache yet)
  const int2 pe = wt > 0 ? bwd_part_exp(w, r, S1, Np, BH, xs, rootmask) : make_int2(kExpZero, kExpZero);
  if (w > 1 && rootmask[r]) return;  // the root span has no parent; its adjoint comes from k_root_bwd (no leaf is a root)
  const int b = row_b[r], i = row_i[r];
  const int n = lens[b];
  const int j = i + w;
  // parents of this launch: all, or (wt > 0) those narrower than wt, the rest lies summed in UV
  const int most = wt > 0 ? wt - 1 - w : n;
  const int nl = min(n - j, most);  // parents (i, j'), j' = j+1..   (this span is their left child)
  const int nr = min(i, most);      // parents (i', j), i' = ..i-1   (this span is their right child)
  const int nt = nl + nr;
  float* s_c = reinterpret_cast<float*>(smem);             // [nt] coefficient of the parent's adjoint
  float* s_cs = s_c + nt;                                  // [nt] coefficient of the sibling's projection
  int32_t* s_p = reinterpret_cast<int32_t*>(s_cs + nt);    // [nt] parent row (index into BH: row - S1)
  int32_t* s_s = s_p + nt;                                 // [nt] sibling row

  const int peu = pe.x, pev = pe.y;
  int dmax = max(peu, pev);
  for (int t = lane; t < nt; t += 64) {
    int pr, sr;
    if (t < nl) {
      const int jp = j + 1 + t;
      pr = row_of(rowtab, stride, B, jp - i, b, i, n);   // parent (i, j')
      sr = row_of(rowtab, stride, B, jp - j, b, j, n);   // sibling (j, j'), used through its zeta
    } else {
      const int ip = i - nr + (t - nl);
      pr = row_of(rowtab, stride, B, j - ip, b, ip, n);  // parent (i', j)
      sr = row_of(rowtab, stride, B, i - ip, b, ip, n);  // sibling (i', i), used through its eta
    }
    s_p[t] = pr - (int)S1;
    s_s[t] = sr;
    const int sb = t < nl ? zmaxb[sr] : hmaxb[sr];  // the sibling's zeta (this span is the left child) or eta
    const int d = add_exp(norm_exp(uexp[pr], umaxb[pr]), proj_exp(mexp[sr], tmaxb[sr], sb));
    s_c[t] = __int_as_float(d);
    s_cs[t] = pow2i(-proj_shift(tmaxb[sr], sb));
    dmax = max(dmax, d);
  }
  const int m = wave_max_i(dmax);
  __syncthreads();
  for (int t = lane; t < nt; t += 64) {
    const int d = __float_as_int(s_c[t]);
    s_c[t] = (d == kExpZero) ? 0.0f : pow2i(d - m);
    if (d == kExpZero) s_cs[t] = 0.0f;
  }
  __syncthreads();

  const int64_t ld = 2 * (int64_t)Np;
  const int a = blockIdx.y * kChunk + lane * 4;
  float amax = 0.0f;
  if (a < Np) {
    float4 u = make_float4(0.f, 0.f, 0.f, 0.f), v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (wt > 0) {
      const float cu = peu == kExpZero ? 0.0f : pow2i(peu - m), cv = pev == kExpZero ? 0.0f : pow2i(pev - m);
      u = *reinterpret_cast<const float4*>(UV + r * ld + a);
      v = *reinterpret_cast<const float4*>(UV + r * ld + Np + a);
      u = make_float4(cu * u.x, cu * u.y, cu * u.z, cu * u.w);
      v = make_float4(cv * v.x, cv * v.y, cv * v.z, cv * v.w);
    }
    const float* bh = BH + a;
    // left-child role: sibling zeta (second half of HZ); right-child role: sibling eta (first half)
#define SPCFG_GATHER(ACC, T0, T1, HZOFF)                                                        \
  {                                                                                             \
    int t = (T0);                                                                               \
    for (; t + 8 <= (T1); t += 8) {                                                             \
      float4 gq[8], sq[8];                                                                      \
      _Pragma("unroll") for (int q = 0; q < 8; ++q) {                                           \
        gq[q] = *reinterpret_cast<const float4*>(bh + (int64_t)s_p[t + q] * Np);                \
        sq[q] = *reinterpret_cast<const float4*>(HZ + s_s[t + q] * ld + (HZOFF) + a);           \
      }                                                                                         \
      _Pragma("unroll") for (int q = 0; q < 8; ++q) {                                           \
        const float c = s_c[t + q], cs = s_cs[t + q];                                           \
        ACC.x = fmaf(c * gq[q].x, cs * sq[q].x, ACC.x);                                         \
        ACC.y = fmaf(c * gq[q].y, cs * sq[q].y, ACC.y);                                         \
        ACC.z = fmaf(c * gq[q].z, cs * sq[q].z, ACC.z);                                         \
        ACC.w = fmaf(c * gq[q].w, cs * sq[q].w, ACC.w);                                         \
      }                                                                                         \
    }                                                                                           \
    for (; t < (T1); t += 4) {                                                                  \
      float4 gq[4], sq[4];                                                                      \
      float cq[4], cs[4];                                                                       \
      _Pragma("unroll") for (int q = 0; q < 4; ++q) {                                           \
        const int tt = min(t + q, (T1)-1);                                                      \
        cq[q] = (t + q < (T1)) ? s_c[tt] : 0.0f;                                                \
        cs[q] = s_cs[tt];                                                                       \
        gq[q] = *reinterpret_cast<const float4*>(bh + (int64_t)s_p[tt] * Np);                   \
        sq[q] = *reinterpret_cast<const float4*>(HZ + s_s[tt] * ld + (HZOFF) + a);              \
      }                                                                                         \
      _Pragma("unroll") for (int q = 0; q < 4; ++q) {                                           \
        ACC.x = fmaf(cq[q] * gq[q].x, cs[q] * sq[q].x, ACC.x);                                  \
        ACC.y = fmaf(cq[q] * gq[q].y, cs[q] * sq[q].y, ACC.y);                                  \
        ACC.z = fmaf(cq[q] * gq[q].z, cs[q] * sq[q].z, ACC.z);                                  \
        ACC.w = fmaf(cq[q] * gq[q].w, cs[q] * sq[q].w, ACC.w);                                  \
      }                                                                                         \
    }                                                                                           \
  }
    SPCFG_GATHER(u, 0, nl, Np)
    SPCFG_GATHER(v, nl, nt, 0)
#undef SPCFG_GATHER
    float* out = UV + r * ld;
    *reinterpret_cast<float4*>(out + a) = u;
    *reinterpret_cast<float4*>(out + Np + a) = v;
    if (UVb) {
      store_planes4(UVb, planes, plane_stride, r * ld + a, u);
      store_planes4(UVb, planes, plane_stride, r * ld + Np + a, v);
    }
    amax = fmaxf(fmaxf(fmaxf(fabsf(u.x), fabsf(u.y)), fmaxf(fabsf(u.z), fabsf(u.w))),
                 fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
  }
  amax = wave_max(amax);
  if (lane == 0) {
    if (amax > 0.0f && m != kExpZero) atomicMax(&umaxb[r], __float_as_uint(amax));
    if (blockIdx.y == 0) {
      uexp[r] = m;
      // scale that turns UV[r] (x) (stored inside vector of the row) into its contribution to dZ/d[L;R]
      const int me = mexp[r];
      gsc[r] = (m == kExpZero || me == kExpZero) ? 0.0f : pow2i(max(m + me, -160));
    }
  }
}

// The reverse sums for launches with few spans, shared by W wavefronts as in k_split_fwd_few: lane t of every wavefront
// holds parent t (right-child roles first: their number does not depend on the sentence's length), wavefront q takes the
// parents q, q + W, ...
template <int W, int U>
__global__ void __launch_bounds__(64 * W)
k_split_bwd_few(int w, int starts, int64_t row0, const int32_t* __restrict__ row_b, const int32_t* __restrict__ row_i,
                int n_long, int B, int Np, int64_t S1, int stride, const int32_t* __restrict__ lens,
                const int32_t* __restrict__ rowtab, const float* __restrict__ HZ, const float* __restrict__ BH, const int32_t* __restrict__ mexp,
                const uint32_t* __restrict__ tmaxb, float* __restrict__ UV, int32_t* __restrict__ uexp,
                uint32_t* __restrict__ umaxb, float* __restrict__ gsc, void* __restrict__ UVb, int planes,
                int64_t plane_stride, const int32_t* __restrict__ hmaxb, const int32_t* __restrict__ zmaxb, int wt,
                const float* __restrict__ xs, const int32_t* __restrict__ rootmask) {
  static_assert(W * U <= 64, "one lane per parent");
  __shared__ float4 s_part[W > 1 ? W : 1][2][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  int b, i;
  few_span(starts, row0, row_b, row_i, &b, &i);
  const int n = lens[b], j = i + w;
  const int most = wt > 0 ? wt - 1 - w : n_long;
  const int nr = min(i, most);  // parents (i', j), i' = i - nr .. i - 1; then the parents (i, j'), j' = j + 1 ..
  // row_of for parent and sibling with the length's part left for later: row 2 is that of a span that ends the sentence
  const int* tab = rowtab + b;
  const int own0 = tab[(i == 0 ? 0 : stride) + w * B] + (i == 0 ? 0 : i - 1), own2 = tab[2 * stride + w * B];
  const bool left = lane >= nr;
  const int ip = i - nr + lane, jp = j + 1 + lane - nr;
  const int p_at = left ? i : ip, p_w = min(left ? jp - i : j - ip, n_long);
  const int s_at = left ? j : ip, s_w = min(left ? jp - j : i - ip, n_long);
  int pr = tab[(p_at == 0 ? 0 : stride) + p_w * B] + (p_at == 0 ? 0 : p_at - 1);
  int sr = tab[(s_at == 0 ? 0 : stride) + s_w * B] + (s_at == 0 ? 0 : s_at - 1);
  const int pr2 = tab[2 * stride + p_w * B], sr2 = tab[2 * stride + s_w * B];
  if (i + w > n || w == n) return;  // (uniform) no such span, or a root: it has no parent, its adjoint comes from k_root_bwd
  const int64_t r = i > 0 && j == n ? own2 : own0;
  const int nl = min(n - j, most), nt = nl + nr;
  if (p_at > 0 && (left ? jp : j) == n) pr = pr2;
  if (left && jp == n) sr = sr2;
  if (lane >= nt) { pr = (int)S1; sr = 0; }
  const int64_t ld = 2 * (int64_t)Np;
  const int col = blockIdx.y * kChunk + lane * 4;
  const int a = min(col, Np - 4);
  float4 gq[U], sq[U];
  const bool some = wave < nt;
  if (some) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = min(wave + u * W, nt - 1);
      gq[u] = *reinterpret_cast<const float4*>(BH + ((int64_t)__builtin_amdgcn_readlane(pr, t) - S1) * Np + a);
      sq[u] = *reinterpret_cast<const float4*>(HZ + (int64_t)__builtin_amdgcn_readlane(sr, t) * ld + (t >= nr ? Np : 0) + a);
    }
  }
  const int2 pe = wt > 0 ? bwd_part_exp(w, r, S1, Np, BH, xs, rootmask) : make_int2(kExpZero, kExpZero);
  const int peu = pe.x, pev = pe.y;
  float4 u0 = make_float4(0.f, 0.f, 0.f, 0.f), v0 = u0;
  if (wave == 0 && wt > 0) {
    u0 = *reinterpret_cast<const float4*>(UV + r * ld + a);
    v0 = *reinterpret_cast<const float4*>(UV + r * ld + Np + a);
  }
  const int me = mexp[r];
  int d = kExpZero;
  float cs_lane = 0.0f;
  if (lane < nt) {
    const int sb = left ? zmaxb[sr] : hmaxb[sr];
    const uint32_t tb = tmaxb[sr];
    d = add_exp(norm_exp(uexp[pr], umaxb[pr]), proj_exp(mexp[sr], tb, sb));
    cs_lane = d == kExpZero ? 0.0f : pow2i(-proj_shift(tb, sb));
  }
  const int m = max(wave_max_i(d), max(peu, pev));
  const int c = __float_as_int(d == kExpZero ? 0.0f : pow2i(d - m)), cs = __float_as_int(cs_lane);
  float4 x[2] = {make_float4(0.f, 0.f, 0.f, 0.f), make_float4(0.f, 0.f, 0.f, 0.f)};
  if (wave == 0 && wt > 0) {
    const float cu = peu == kExpZero ? 0.0f : pow2i(peu - m), cv = pev == kExpZero ? 0.0f : pow2i(pev - m);
    x[0] = make_float4(cu * u0.x, cu * u0.y, cu * u0.z, cu * u0.w);
    x[1] = make_float4(cv * v0.x, cv * v0.y, cv * v0.z, cv * v0.w);
  }
  if (some) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = wave + u * W;
      if (t < nt) {
        const float ct = __int_as_float(__builtin_amdgcn_readlane(c, t)), cst = __int_as_float(__builtin_amdgcn_readlane(cs, t));
        const float4 p = make_float4(ct * gq[u].x, ct * gq[u].y, ct * gq[u].z, ct * gq[u].w);
        const float4 q = make_float4(cst * sq[u].x, cst * sq[u].y, cst * sq[u].z, cst * sq[u].w);
        if (t >= nr) {
          x[0].x = fmaf(p.x, q.x, x[0].x); x[0].y = fmaf(p.y, q.y, x[0].y);
          x[0].z = fmaf(p.z, q.z, x[0].z); x[0].w = fmaf(p.w, q.w, x[0].w);
        } else {
          x[1].x = fmaf(p.x, q.x, x[1].x); x[1].y = fmaf(p.y, q.y, x[1].y);
          x[1].z = fmaf(p.z, q.z, x[1].z); x[1].w = fmaf(p.w, q.w, x[1].w);
        }
      }
    }
  }
  if (W > 1) {
    s_part[wave][0][lane] = x[0];
    s_part[wave][1][lane] = x[1];
    __syncthreads();
    if (wave > 1) return;
  }
  float amax = 0.0f;
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    if (W > 1 && half != wave) continue;  // with several wavefronts the first writes adj eta, the second adj zeta
    float4 o = x[half];
    if (W > 1) {
      o = s_part[0][half][lane];
#pragma unroll
      for (int q = 1; q < W; ++q) {
        const float4 y = s_part[q][half][lane];
        o.x += y.x; o.y += y.y; o.z += y.z; o.w += y.w;
      }
    }
    if (col < Np) {
      *reinterpret_cast<float4*>(UV + r * ld + half * (int64_t)Np + a) = o;
      if (UVb) store_planes4(UVb, planes, plane_stride, r * ld + half * (int64_t)Np + a, o);
      amax = fmaxf(amax, fmaxf(fmaxf(fabsf(o.x), fabsf(o.y)), fmaxf(fabsf(o.z), fabsf(o.w))));
    }
  }
  amax = wave_max(amax);
  if (lane == 0) {
    if (amax > 0.0f && m != kExpZero) atomicMax(&umaxb[r], __float_as_uint(amax));
    if (blockIdx.y == 0 && wave == 0) {
      uexp[r] = m;
      gsc[r] = (m == kExpZero || me == kExpZero) ? 0.0f : pow2i(max(m + me, -160));
    }
  }
}

// grad_log_emit is zero at padded token positions.
__global__ void k_zero_pad_emit(int P, int n_max, const int32_t* __restrict__ lens, float* __restrict__ g) {
  const int b = blockIdx.x;
  const int n = lens[b];
  float* base = g + ((int64_t)b * n_max + n) * P;
  const int64_t cnt = (int64_t)(n_max - n) * P;
  for (int64_t t = threadIdx.x; t < cnt; t += blockDim.x) base[t] = 0.0f;
}

// ------------------------------------------------------------------------------------------ span posteriors
// mu(i,j) = sum_A beta_ij[A] * d logZ / d beta_ij[A]: the posterior probability that some nonterminal spans
// (i,j) (inside-outside by back-propagation, Sec. 3.2).  Both factors are still in the workspace after the
// reverse pass: beta = 2^mexp * T and its adjoint = 2^(uexp + f') * BH.  One wavefront per (sentence, i, j-1)
// entry of the dense output; entries that are no span get 0 / -1.  Width-1 spans carry the same mass as the
// root span (both are in every tree), so they read the root row.  label = first arg-max nonterminal.
__global__ void __launch_bounds__(64)
k_span_marginals(int B, int N, int Np, int n_max, int64_t S1, const int32_t* __restrict__ lens,
                 const int32_t* __restrict__ rowtab, const float* __restrict__ T, const float* __restrict__ BH,
                 const int32_t* __restrict__ mexp, const int32_t* __restrict__ uexp,
                 const uint32_t* __restrict__ umaxb, float* __restrict__ mu, int32_t* __restrict__ label) {
  const int lane = threadIdx.x;
  const int b = blockIdx.y;
  const int i = blockIdx.x / n_max, j = blockIdx.x % n_max + 1;
  const int n = lens[b];
  const int64_t out = ((int64_t)b * n_max + i) * n_max + (j - 1);
  if (j <= i || j > n) {
    if (lane == 0) {
      mu[out] = 0.0f;
      if (label) label[out] = -1;
    }
    return;
  }
  const int w = j - i;
  const int stride = (n_max + 1) * B;
  const int64_t r = (w == 1) ? rowtab[n * B + b] : row_of(rowtab, stride, B, w, b, i, n);
  const float* t = T + (r - S1) * Np;
  const float* h = BH + (r - S1) * Np;
  float sum = 0.0f, best = 0.0f;
  int arg = -1;
  for (int a = lane * 4; a < Np; a += 256) {
    const float4 x = *reinterpret_cast<const float4*>(t + a);
    const float4 y = *reinterpret_cast<const float4*>(h + a);
    const float p0 = x.x * y.x, p1 = x.y * y.y, p2 = x.z * y.z, p3 = x.w * y.w;
    sum += (p0 + p1) + (p2 + p3);
    if (p0 > best) { best = p0; arg = a; }
    if (p1 > best) { best = p1; arg = a + 1; }
    if (p2 > best) { best = p2; arg = a + 2; }
    if (p3 > best) { best = p3; arg = a + 3; }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    sum += __shfl_xor(sum, o, 64);
    const float ob = __shfl_xor(best, o, 64);
    const int oa = __shfl_xor(arg, o, 64);
    if (ob > best || (ob == best && oa >= 0 && (arg < 0 || oa < arg))) { best = ob; arg = oa; }
  }
  if (lane == 0) {
    const int d = add_exp(mexp[r], norm_exp(uexp[r], umaxb[r]));
    const float m = (d == kExpZero) ? 0.0f : pow2i(d) * sum;
    mu[out] = m;
    if (label) label[out] = (w >= 2 && m > 0.0f && arg < N) ? arg : -1;
  }
}

// the tables of a band over 1024-word sentences take 136 KB
bool set_band_lds(const void* kernel) {
  return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 4 * band_words(kMaxLen + 8)) == hipSuccess;
}

}  // namespace

void launch_plan(const Layout& ly, const Ptrs& p, const LenArg& lens, hipStream_t st) {
  launch_k(k_plan_rowbase, dim3((unsigned)ly.n_max), dim3(kPlanThreads), 0, st, lens, ly.B, ly.n_max, ly.G > 1 ? 1 : 0, p.lens,
           p.rowbase, p.rootrow, p.counters, ly.n_counters);
  launch_k(k_plan_rows, dim3(ly.n_max, ly.B), dim3(64), 0, st, ly.B, (ly.n_max + 1) * ly.B, p.lens, p.rowbase, p.row_b, p.row_i,
                     p.rootmask, p.tmaxb, p.umaxb, p.hmaxb, p.zmaxb, reinterpret_cast<uint32_t*>(p.colmax),
                     2 * (int64_t)(ly.Np + ly.Pp) * ly.G);
}

void launch_plan_sentrows(const Layout& ly, const Ptrs& p, hipStream_t st) {
  if (ly.n_max < 2) return;
  launch_k(k_plan_sentrows, dim3(ly.n_max - 1, ly.B), dim3(64), 0, st, ly.B, (ly.n_max + 1) * ly.B, p.lens, p.rowbase, p.sentrows,
                     p.sentoff);
}

void launch_pack_weights(const Layout& ly, const Ptrs& p, const float* L, const float* R, hipStream_t st) {
  const dim3 grid((ly.Np + ly.Pp) / 64, ly.Np / 64, 2 * ly.G), block(256);
  uint32_t* cm = reinterpret_cast<uint32_t*>(p.colmax);
  void* none = nullptr;
  float *Wn = p.Wn, *Wp = p.Wp, *Wtn = p.Wtn, *Wtp = p.Wtp;
  __bf16 *Wtn_b = reinterpret_cast<__bf16*>(Wtn), *Wtp_b = reinterpret_cast<__bf16*>(Wtp);
  if (ly.planes == 3)  // fp32 panels, and once more as three bf16 planes
    launch_k(k_pack_weights<float, 3, float, 3>, grid, block, 0, st, L, R, ly.N, ly.P, ly.Np, ly.Pp, Wn, Wp, Wtn, Wtp, p.Wn3,
             p.Wp3, p.Wtn3, p.Wtp3, cm);
  else if (ly.fwd_fp32)  // fp32 panels for the forward products, bf16 panels for the reverse ones
    launch_k(k_pack_weights<float, 0, __bf16, 0>, grid, block, 0, st, L, R, ly.N, ly.P, ly.Np, ly.Pp, Wn, Wp, Wtn_b, Wtp_b, none,
             none, none, none, cm);
  else if (ly.planes == 2)  // two bf16 planes for the forward products, single bf16 panels for the reverse ones
    launch_k(k_pack_weights<__bf16, 2, __bf16, 0>, grid, block, 0, st, L, R, ly.N, ly.P, ly.Np, ly.Pp, (__bf16*)nullptr,
             (__bf16*)nullptr, Wtn_b, Wtp_b, p.Wn3, p.Wp3, none, none, cm);
  else if (ly.bf16)
    launch_k(k_pack_weights<__bf16, 0, __bf16, 0>, grid, block, 0, st, L, R, ly.N, ly.P, ly.Np, ly.Pp,
             reinterpret_cast<__bf16*>(Wn), reinterpret_cast<__bf16*>(Wp), Wtn_b, Wtp_b, none, none, none, none, cm);
  else
    launch_k(k_pack_weights<float, 0, float, 0>, grid, block, 0, st, L, R, ly.N, ly.P, ly.Np, ly.Pp, Wn, Wp, Wtn, Wtp, none, none,
             none, none, cm);
}

void launch_scaled_planes(const float* X, int64_t ld, const float* sc, int64_t S, int64_t Srows, void* planes,
                          int64_t plane_stride, hipStream_t st) {
  if (Srows <= 0) return;
  const dim3 grid((unsigned)Srows, (unsigned)((ld / 4 + 255) / 256));
  launch_k(k_scaled_planes, grid, dim3(256), 0, st, X, ld, sc, S, static_cast<uint16_t*>(planes), plane_stride);
}

void launch_zero_plane_rows(void* planes, int64_t plane_stride, int64_t ld, int64_t row0, int64_t rows, hipStream_t st) {
  const int64_t count = rows * ld;  // ld is a multiple of 64
  launch_k(k_zero_plane_rows, dim3((unsigned)((count / 8 + 255) / 256 < 256 ? (count / 8 + 255) / 256 : 256), plane_stride ? 3 : 1), dim3(256), 0, st,
           static_cast<uint16_t*>(planes), plane_stride, row0 * ld, count);
}

void launch_leaf_prep(const Layout& ly, const Ptrs& p, const float* log_emit, bool write_planes, hipStream_t st) {
  launch_k(k_leaf_prep, dim3((unsigned)ly.S1), dim3(256), 0, st, log_emit, ly.P, ly.Pp, ly.n_max, p.row_b,
                     p.row_i, p.leafE, p.xs, p.mexp, p.tmaxb, static_cast<uint16_t*>(write_planes ? p.leafEb : nullptr), ly.planes,
                     (int64_t)ly.S1 * ly.Pp, p.colmax, ly.Np, ly.G > 1 ? 1 : 0, p.hmaxb, p.zmaxb);
}

namespace {
// Launches of few wavefronts (in the plain form) share each span among several: there a launch costs its chain of dependent
// loads (B = 7, N = 141, n <= 37: 6.4 us a forward and 6.8 us a reverse launch plain, 4.7 and 5.1 us shared; B = 1, N = 2048,
// n = 40: 7.2 and 5.4 us forward).  Every sharing wavefront looks all terms of the span up and keeps its rows in flight, so the
// form pays while few rows are requested in all: kFewLoads counts them as wavefronts times the form's terms.  Split sums
// of a pass in us, plain / up to this limit / up to twice as many / with a limit on wavefronts alone: forward B = 8, N = 64,
// n = 60 428 / 314 / 312 / 315; B = 4, N = 2048, n = 60 689 / 668 / 731 / 793; B = 1, N = 4096, n = 60 579 / 544 / 606 / 607.
// The reverse form pays up to 1024 nonterminals: B = 1, n = 60 with N = 64 426 / 310 / 316 / 317, N = 1024 488 / 404 / 383 /
// 393, but N = 2048 484 / 474 / 563 / 566 (B = 2: 640 / 649 / 651 / 825) and N = 4096 687 / 728 / 737 / 1073.
constexpr int64_t kFewWaves = 1024;
constexpr int64_t kFewLoads = 16384;
constexpr int kFewChunksBwd = 4;
// Terms that the form with room for `terms` has room for (launch_few_fwd, launch_few_bwd)
int few_slots(int terms) { return terms <= 4 ? 4 : (terms <= 8 ? 8 : (terms <= 16 ? 16 : (terms <= 32 ? 32 : 64))); }
bool few_pays(int64_t waves, int terms) {
  return terms <= 64 && waves <= kFewWaves && waves * few_slots(terms) <= kFewLoads;
}
// Spans by block index (see few_span) while the workgroups, with and without a span, are few enough to start at once.
int few_starts(const Layout& ly, int w, int chunks) {
  const int64_t starts = ly.n_long - w + 1;
  return starts * ly.B * chunks <= kFewWaves ? (int)starts : 0;
}
template <typename... A>
void launch_few_fwd(int terms, dim3 grid, hipStream_t st, A... args) {
  if (terms <= 4) launch_k(k_split_fwd_few<1, 4>, grid, dim3(64), 0, st, args...);
  else if (terms <= 8) launch_k(k_split_fwd_few<2, 4>, grid, dim3(128), 0, st, args...);
  else if (terms <= 16) launch_k(k_split_fwd_few<4, 4>, grid, dim3(256), 0, st, args...);
  else if (terms <= 32) launch_k(k_split_fwd_few<8, 4>, grid, dim3(512), 0, st, args...);
  else launch_k(k_split_fwd_few<8, 8>, grid, dim3(512), 0, st, args...);
}
template <typename... A>
void launch_few_bwd(int terms, dim3 grid, hipStream_t st, A... args) {
  if (terms <= 4) launch_k(k_split_bwd_few<1, 4>, grid, dim3(64), 0, st, args...);
  else if (terms <= 8) launch_k(k_split_bwd_few<2, 4>, grid, dim3(128), 0, st, args...);
  else if (terms <= 16) launch_k(k_split_bwd_few<4, 4>, grid, dim3(256), 0, st, args...);
  else if (terms <= 32) launch_k(k_split_bwd_few<8, 4>, grid, dim3(512), 0, st, args...);
  else launch_k(k_split_bwd_few<8, 8>, grid, dim3(512), 0, st, args...);
}
}  // namespace

namespace {
// The launch of one band: a grid of every tile of the longest sentence, in every sentence.  With enough tiles a wavefront
// per 64 nonterminals, up to four a workgroup and evenly dealt to the workgroups (at most one of these has a wavefront without
// nonterminals of its own: with four in each, B = 960, N = 64, n <= 40 spent 831 + 1443 us forward + reverse on split sums, and
// 694 + 989 us so); otherwise kBandShare wavefronts per 64.  What counts is the tiles that there are, not those of the grid:
// by the grid's, late bands of mixed lengths took the first form (B = 64, N = 512, n = 2 .. 100: 2187 us forward, 1875 us so).
struct BandGrid {
  bool share;
  dim3 grid, block;
  size_t lds;
  int S_max;
};
BandGrid band_grid(const Layout& ly, int w0, int S, int roles) {
  BandGrid g;
  const int blocks = ly.Np / 64, groups = (blocks + kBandWaves - 1) / kBandWaves;
  g.share = (int64_t)roles * ly.band_tiles[w0 / kBandW] * blocks < kBandMinWaves;
  g.grid = dim3((unsigned)(g.share ? blocks : groups), (unsigned)((ly.n_long - w0 + kBandI) / kBandI), (unsigned)(roles * ly.B));
  g.block = dim3(64u * (unsigned)(g.share ? kBandShare : (blocks + groups - 1) / groups));
  g.S_max = round_up(S, 4);
  g.lds = sizeof(int32_t) * (size_t)band_words(g.S_max);
  const size_t sums = sizeof(float) * (size_t)kBandSumWords;
  if (g.share && g.lds < sums) g.lds = sums;
  return g;
}
template <int KS>
void launch_band_fwd(const BandGrid& g, const Layout& ly, const Ptrs& p, int w0, hipStream_t st) {
  static const bool attr = set_band_lds(reinterpret_cast<const void*>(&k_split_band_fwd<KS>));
  (void)attr;
  launch_k(k_split_band_fwd<KS>, g.grid, g.block, g.lds, st, w0, ly.B, ly.Np, ly.S1, (ly.n_max + 1) * ly.B, g.S_max, p.lens,
           p.rowbase, p.HZ, p.mexp, p.tmaxb, p.hmaxb, p.zmaxb, p.T, p.uexp);
}
template <int KS>
void launch_band_bwd(const BandGrid& g, const Layout& ly, const Ptrs& p, int w0, hipStream_t st) {
  static const bool attr = set_band_lds(reinterpret_cast<const void*>(&k_split_band_bwd<KS>));
  (void)attr;
  launch_k(k_split_band_bwd<KS>, g.grid, g.block, g.lds, st, w0, ly.B, ly.Np, ly.S1, (ly.n_max + 1) * ly.B, g.S_max, p.lens,
           p.rowbase, p.HZ, p.BH, p.mexp, p.tmaxb, p.hmaxb, p.zmaxb, p.uexp, p.umaxb, p.UV, BwdPartExp{p.BH, p.xs, p.rootmask});
}
}  // namespace

void launch_split_fwd(const Layout& ly, const Ptrs& p, int w, int64_t row0, int64_t rows, bool write_planes,
                      hipStream_t st) {
  void* Tb = write_planes ? p.Tb : nullptr;
  const int stride = (ly.n_max + 1) * ly.B;
  const int w0 = ly.band_fwd[w / kBandW] ? w / kBandW * kBandW : 0;
  if (w == w0) {  // the first width of a band: all that its widths can do together
    const BandGrid g = band_grid(ly, w0, w0 + kBandI, 1);
    if (g.share) launch_band_fwd<kBandShare>(g, ly, p, w0, st);
    else launch_band_fwd<1>(g, ly, p, w0, st);
  }
  const int nk = w0 > 0 ? 2 * (w - w0) : w - 1;
  const size_t sh = (size_t)nk * 16;
  const int chunks = (ly.Np + kChunk - 1) / kChunk;
  const int starts = few_starts(ly, w, chunks);
  if (few_pays(rows * chunks, nk)) {
    launch_few_fwd(nk, dim3((unsigned)(starts > 0 ? starts * ly.B : rows), (unsigned)chunks), st, w, starts, row0, p.row_b, p.row_i, ly.B, ly.Np, ly.S1, stride, p.lens,
                   p.rowbase, p.HZ, p.T, p.mexp, p.tmaxb, Tb, ly.planes, (int64_t)ly.S2 * ly.Np, p.hmaxb, p.zmaxb, p.colmax, ly.Pp,
                   ly.G > 1 ? 1 : 0, w0, p.uexp);
    return;
  }
  if (rows * chunks < 1024 && nk >= 64) {  // fewer than one wavefront per SIMD, long chains of split points (see k_split_fwd)
    const dim3 grid((unsigned)rows, (unsigned)(ly.Np / 64));
    launch_k(k_split_fwd<4>, grid, dim3(64), sh, st, w, row0, ly.B, ly.Np, ly.S1, stride, p.lens, p.rowbase, p.row_b, p.row_i, p.HZ,
             p.T, p.mexp, p.tmaxb, Tb, ly.planes, (int64_t)ly.S2 * ly.Np, p.hmaxb, p.zmaxb, p.colmax, ly.Pp,
             ly.G > 1 ? 1 : 0, w0, p.uexp);
    return;
  }
  const dim3 grid((unsigned)rows, (unsigned)chunks);
  launch_k(k_split_fwd<1>, grid, dim3(64), sh, st, w, row0, ly.B, ly.Np, ly.S1, stride, p.lens, p.rowbase, p.row_b, p.row_i, p.HZ,
           p.T, p.mexp, p.tmaxb, Tb, ly.planes, (int64_t)ly.S2 * ly.Np, p.hmaxb, p.zmaxb, p.colmax, ly.Pp,
           ly.G > 1 ? 1 : 0, w0, p.uexp);
}

void launch_root_fwd(const Layout& ly, const Ptrs& p, const float* log_root, float* logZ, hipStream_t st) {
  launch_k(k_root_fwd, dim3(ly.B), dim3(256), 0, st, ly.B, ly.N, ly.Np, ly.S1, p.lens, p.rowbase,
                     p.rootrow, log_root, p.T, p.mexp, p.tmaxb, p.xs, logZ, p.ztil, p.rmax,
                     (int64_t)(ly.G > 1 ? ly.N : 0));
}

void launch_root_bwd(const Layout& ly, const Ptrs& p, const float* log_root, const float* grad_logZ,
                     float* grad_log_root, int accumulate, hipStream_t st) {
  launch_k(k_root_bwd, dim3(ly.B), dim3(256), 0, st, ly.N, ly.Np, ly.S1, p.rootrow, log_root, grad_logZ,
                     p.ztil, p.rmax, p.mexp, p.tmaxb, p.BH, p.UV, p.uexp, p.umaxb, p.gsc,
                     (int64_t)(ly.G > 1 ? ly.N : 0), static_cast<uint16_t*>(p.UVb), ly.planes_bwd,
                     ly.uvb_plane);
  launch_k(k_grad_log_root, dim3((ly.N + 255) / 256, ly.G > 1 ? ly.B : 1), dim3(256), 0, st, ly.B, ly.N,
                     ly.Np, ly.S1, p.rootrow, log_root, grad_logZ, p.ztil, p.rmax, p.T, p.tmaxb, grad_log_root,
                     accumulate, ly.G > 1 ? 1 : 0);
}

void launch_split_bwd(const Layout& ly, const Ptrs& p, int w, int64_t row0, int64_t rows, bool write_planes,
                      hipStream_t st) {
  const int stride = (ly.n_max + 1) * ly.B;
  const bool band = ly.band_bwd[w / kBandW] != 0;
  const int w0 = w / kBandW * kBandW, wt = band ? w0 + kBandW : 0;
  if (band && w == band_top(ly, w0)) {
    const BandGrid g = band_grid(ly, w0, ly.n_long - w0 + kBandI, 2);  // (adj eta: n - wt + 1 values of s, adj zeta: n - w0 + 3)
    if (g.share) launch_band_bwd<kBandShare>(g, ly, p, w0, st);
    else launch_band_bwd<1>(g, ly, p, w0, st);
  }
  const int most = band ? 2 * (wt - 1 - w) : ly.n_long - w;  // parents of a span
  const int chunks = (ly.Np + kChunk - 1) / kChunk;
  const int starts = few_starts(ly, w, chunks);
  if (chunks <= kFewChunksBwd && few_pays(rows * chunks, most)) {
    launch_few_bwd(most, dim3((unsigned)(starts > 0 ? starts * ly.B : rows), (unsigned)chunks), st, w, starts, row0, p.row_b, p.row_i, ly.n_long, ly.B, ly.Np, ly.S1, stride,
                   p.lens, p.rowbase, p.HZ, p.BH, p.mexp, p.tmaxb, p.UV, p.uexp, p.umaxb, p.gsc, write_planes ? p.UVb : nullptr,
                   ly.planes_bwd, ly.uvb_plane, p.hmaxb, p.zmaxb, wt, p.xs, p.rootmask);
    return;
  }
  const size_t sh = (size_t)(band ? 2 * (wt - 1 - w) : ly.n_max) * 16;
  const dim3 grid((unsigned)rows, (unsigned)((ly.Np + kChunk - 1) / kChunk));
  launch_k(k_split_bwd, grid, dim3(64), sh, st, w, row0, ly.B, ly.Np, ly.S1, stride, p.lens, p.rowbase, p.row_b,
                     p.row_i, p.rootmask, p.HZ, p.BH, p.mexp, p.tmaxb, p.UV, p.uexp, p.umaxb, p.gsc, write_planes ? p.UVb : nullptr, ly.planes_bwd,
                     ly.uvb_plane, p.hmaxb, p.zmaxb, wt, p.xs);
}

void launch_zero_pad_emit(const Layout& ly, const Ptrs& p, float* grad_log_emit, hipStream_t st) {
  launch_k(k_zero_pad_emit, dim3(ly.B), dim3(256), 0, st, ly.P, ly.n_max, p.lens, grad_log_emit);
}

void launch_span_marginals(const Layout& ly, const Ptrs& p, float* mu, int32_t* label, hipStream_t st) {
  const dim3 grid((unsigned)(ly.n_max * ly.n_max), (unsigned)ly.B);
  launch_k(k_span_marginals, grid, dim3(64), 0, st, ly.B, ly.N, ly.Np, ly.n_max, ly.S1, p.lens, p.rowbase,
                     p.T, p.BH, p.mexp, p.uexp, p.umaxb, mu, label);
}

}  // namespace spcfg
