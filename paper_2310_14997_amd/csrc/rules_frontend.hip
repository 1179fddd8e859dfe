// Rule-probability front-end and its backward: the four softmaxes that end the neural parameterisation
// (App. A) - root over the nonterminals, left and right productions over N u P children per parent,
// emissions over the vocabulary per preterminal - and the per-token gather of the emission table that the
// inside pass consumes.  All kernels are memory-bound row reductions or elementwise passes; results are
// deterministic (every entry of the emission gradient has one owner, which adds its tokens in order).
#include <cmath>

#include "spcfg_internal.h"

namespace spcfg {

namespace {

__device__ __forceinline__ float wmax(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ float wsum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float bmax(float v, float* red) {
  v = wmax(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  float r = red[0];
  for (int i = 1; i < (int)(blockDim.x >> 6); ++i) r = fmaxf(r, red[i]);
  return r;
}
__device__ __forceinline__ float bsum(float v, float* red) {
  v = wsum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  float r = 0.0f;
  for (int i = 0; i < (int)(blockDim.x >> 6); ++i) r += red[i];  // fixed order
  return r;
}

// ---- rows held in registers ------------------------------------------------------------------------------
// Every softmax row is read once: the 256 threads of a workgroup keep it in registers (up to 4 * kMostE4 values each)
// between the maximum, the sum and the write.  16-byte loads where base and row length allow it, 4-byte ones otherwise
// (the same values per workgroup, other columns per thread).  Longer rows are read once per pass instead.
constexpr int kMostE4 = 16;

template <bool VEC, int E4>
__device__ __forceinline__ void row_load(const float* __restrict__ row, int cols, float pad, float (&x)[4 * E4]) {
#pragma unroll
  for (int e = 0; e < E4; ++e) {
    if (VEC) {
      const int c = (e * 256 + (int)threadIdx.x) * 4;
      const float4 v = c < cols ? *reinterpret_cast<const float4*>(row + c) : make_float4(pad, pad, pad, pad);
      x[4 * e] = v.x; x[4 * e + 1] = v.y; x[4 * e + 2] = v.z; x[4 * e + 3] = v.w;
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int c = (e * 4 + u) * 256 + (int)threadIdx.x;
        x[4 * e + u] = c < cols ? row[c] : pad;
      }
    }
  }
}
template <bool VEC, int E4>
__device__ __forceinline__ void row_store(float* __restrict__ row, int cols, const float (&x)[4 * E4]) {
#pragma unroll
  for (int e = 0; e < E4; ++e) {
    if (VEC) {
      const int c = (e * 256 + (int)threadIdx.x) * 4;
      if (c < cols) *reinterpret_cast<float4*>(row + c) = make_float4(x[4 * e], x[4 * e + 1], x[4 * e + 2], x[4 * e + 3]);
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int c = (e * 4 + u) * 256 + (int)threadIdx.x;
        if (c < cols) row[c] = x[4 * e + u];
      }
    }
  }
}

// out = softmax(row), or with `lse` *out = logsumexp(row)
template <bool VEC, int E4>
__device__ __forceinline__ void row_softmax(const float* __restrict__ row, int cols, float* __restrict__ out, bool lse,
                                            float* red) {
  float x[4 * E4];
  row_load<VEC, E4>(row, cols, -INFINITY, x);
  float m = x[0];
#pragma unroll
  for (int e = 1; e < 4 * E4; ++e) m = fmaxf(m, x[e]);
  m = bmax(m, red);
  float s = 0.0f;
#pragma unroll
  for (int e = 0; e < 4 * E4; ++e) { x[e] = expf(x[e] - m); s += x[e]; }
  s = bsum(s, red);
  if (lse) {
    if (threadIdx.x == 0) *out = m + logf(s);
    return;
  }
  const float inv = 1.0f / s;
#pragma unroll
  for (int e = 0; e < 4 * E4; ++e) x[e] *= inv;
  row_store<VEC, E4>(out, cols, x);
}
__device__ void row_softmax_long(const float* __restrict__ row, int64_t cols, float* __restrict__ out, bool lse, float* red) {
  float m = -INFINITY;
  for (int64_t c = threadIdx.x; c < cols; c += 256) m = fmaxf(m, row[c]);
  m = bmax(m, red);
  float s = 0.0f;
  for (int64_t c = threadIdx.x; c < cols; c += 256) s += expf(row[c] - m);
  s = bsum(s, red);
  if (lse) {
    if (threadIdx.x == 0) *out = m + logf(s);
    return;
  }
  const float inv = 1.0f / s;
  for (int64_t c = threadIdx.x; c < cols; c += 256) out[c] = expf(row[c] - m) * inv;
}
// out = log_softmax(row) for the one row of root scores.  A rounding of the sum's logarithm would shift every entry alike (by up
// to 5e-7 at N = 2048, as large as all other errors of the pass): sum and logarithm are in 64 bits.
__device__ void row_log_softmax(const float* __restrict__ row, int cols, float* __restrict__ out, float* red) {
  __shared__ double part[4];
  float m = -INFINITY;
  for (int c = threadIdx.x; c < cols; c += 256) m = fmaxf(m, row[c]);
  m = bmax(m, red);
  double s = 0.0;
  for (int c = threadIdx.x; c < cols; c += 256) s += (double)expf(row[c] - m);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
  __syncthreads();
  const double ls = log(part[0] + part[1] + part[2] + part[3]);
  for (int c = threadIdx.x; c < cols; c += 256) out[c] = (float)(((double)row[c] - (double)m) - ls);
}

__device__ __forceinline__ bool aligned16(const void* a, const void* b, int64_t cols) {
  return ((((uintptr_t)a | (uintptr_t)b) & 15) == 0) && (cols & 3) == 0;
}

// All rows of the forward pass in one launch: the root (a chain), the P vocabulary rows (the longest), then L and R.
// Bound by HBM: every score is read once and L, R written once.  N = P = 2048, V = 10000: 53 us (4.0 TB/s); four launches
// that read each row two or three times took 104 us.
__global__ void __launch_bounds__(256) k_rows_forward(int N, int P, int64_t V, const float* __restrict__ root,
                                                      const float* __restrict__ Lz, const float* __restrict__ Rz,
                                                      const float* __restrict__ emis, float* __restrict__ log_root,
                                                      float* __restrict__ L, float* __restrict__ R, float* __restrict__ lse) {
  __shared__ float red[4];
  const int64_t M = (int64_t)N + P;
  int r = blockIdx.x;
  if (r == 0) {
    row_log_softmax(root, N, log_root, red);
    return;
  }
  r -= 1;
  const float* row;
  float* out;
  int64_t cols = M;
  const bool lse_row = r < P;
  if (lse_row) { row = emis + r * V; out = lse + r; cols = V; }
  else if ((r -= P) < N) { row = Lz + r * M; out = L + r * M; }
  else { r -= N; row = Rz + r * M; out = R + r * M; }
  const bool vec = aligned16(row, lse_row ? row : out, cols);
  if (cols <= 1024 * 4) {
    if (vec) row_softmax<true, 4>(row, (int)cols, out, lse_row, red);
    else row_softmax<false, 4>(row, (int)cols, out, lse_row, red);
  } else if (cols <= 1024 * kMostE4) {
    if (vec) row_softmax<true, kMostE4>(row, (int)cols, out, lse_row, red);
    else row_softmax<false, kMostE4>(row, (int)cols, out, lse_row, red);
  } else {
    row_softmax_long(row, cols, out, lse_row, red);
  }
}

// log_emit[b, i, T] = emis_logits[T, tok] - lse[T] for i < n_b, 0 on padding; an out-of-range token id gives NaN.
// A line of the table per token and preterminal, most of them from cache (tokens repeat and share lines): 26 us for 1400
// tokens at P = 2048, V = 10000.  Whole tiles of the table turned in LDS took 54 us, and twice as long at every size
// from 320 to 12800 tokens.
__global__ void __launch_bounds__(256) k_gather_emit(LenArg la, int n_max, int P, int V,
                                                     const float* __restrict__ emis, const float* __restrict__ lse,
                                                     const int32_t* __restrict__ tokens, float* __restrict__ out) {
  const int b = blockIdx.x / n_max, i = blockIdx.x % n_max;
  float* o = out + (int64_t)blockIdx.x * P;
  if (i >= la.v[b]) {
    for (int t = threadIdx.x; t < P; t += 256) o[t] = 0.0f;
    return;
  }
  const int tok = tokens[blockIdx.x];
  const bool ok = (unsigned)tok < (unsigned)V;
  for (int t = threadIdx.x; t < P; t += 256) o[t] = ok ? emis[(int64_t)t * V + tok] - lse[t] : NAN;
}

// ---- the emission table in tiles of 64 preterminals x kVChunk vocabulary entries ---------------------------
constexpr int kVChunk = 128;
constexpr int kSeg = 1024;        // token positions looked through at a time, four per thread
constexpr int kMaxVBlocks = 32768;  // workgroups along the vocabulary; longer tables take several chunks each
static_assert((int64_t)kMaxB * kMaxLen < (1 << 20), "a list entry holds a position in 20 bits");

// softmax backward per row: dz = p * (g - sum_j p_j g_j), both rows kept in registers
template <bool VEC, int E4>
__device__ __forceinline__ void row_softmax_bwd(const float* __restrict__ p, const float* __restrict__ g, int cols,
                                                float* __restrict__ dz, float* red) {
  float x[4 * E4], y[4 * E4];
  row_load<VEC, E4>(p, cols, 0.0f, x);
  row_load<VEC, E4>(g, cols, 0.0f, y);
  float d = 0.0f;
#pragma unroll
  for (int e = 0; e < 4 * E4; ++e) d = fmaf(x[e], y[e], d);
  d = bsum(d, red);
#pragma unroll
  for (int e = 0; e < 4 * E4; ++e) x[e] = x[e] * (y[e] - d);
  row_store<VEC, E4>(dz, cols, x);
}

// part[c][T] = sum of grad_log_emit[b, i, T] over the real token positions p = b * n_max + i with p % kColChunks == c
// (position order inside a chunk); tot[T] = sum_c part[c][T] in chunk order.  Deterministic two-level sum.
constexpr int kColChunks = 32;

// Everything of the backward pass that the emission tiles wait for or that they do not need, in one launch: column sums
// (a wavefront per 64 preterminals and chunk, eight positions in flight; chains, so they start first), then the rows of
// L and R, then the root (dz = g - exp(log_root) * sum_j g_j).  N = P = 2048, 1400 tokens: 61 us; five launches took 100 us.
__global__ void __launch_bounds__(256) k_rows_backward(LenArg la, int B, int n_max, int N, int P,
                                                       const float* __restrict__ log_root, const float* __restrict__ L,
                                                       const float* __restrict__ R, const float* __restrict__ g_root,
                                                       const float* __restrict__ gL, const float* __restrict__ gR,
                                                       const float* __restrict__ ge, float* __restrict__ d_root,
                                                       float* __restrict__ dL, float* __restrict__ dR,
                                                       float* __restrict__ part) {
  __shared__ float red[4];
  const int col_blocks = (P + 63) / 64 * (kColChunks / 4);
  int r = blockIdx.x;
  if (r < col_blocks) {
    const int t = r / (kColChunks / 4) * 64 + (threadIdx.x & 63);
    const int c = r % (kColChunks / 4) * 4 + (threadIdx.x >> 6);
    if (t >= P) return;
    float s = 0.0f;
    for (int p0 = c; p0 < B * n_max; p0 += 8 * kColChunks) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int p = p0 + u * kColChunks;
        const int b = p / n_max;
        v[u] = p < B * n_max && p - b * n_max < la.v[min(b, B - 1)] ? ge[(int64_t)p * P + t] : 0.0f;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) s += v[u];
    }
    part[(int64_t)c * P + t] = s;
    return;
  }
  r -= col_blocks;
  if (r == 2 * N) {
    float s = 0.0f;
    for (int c = threadIdx.x; c < N; c += 256) s += g_root[c];
    s = bsum(s, red);
    for (int c = threadIdx.x; c < N; c += 256) d_root[c] = g_root[c] - expf(log_root[c]) * s;
    return;
  }
  const int64_t cols = (int64_t)N + P, base = (int64_t)(r < N ? r : r - N) * cols;
  const float* p = (r < N ? L : R) + base;
  const float* g = (r < N ? gL : gR) + base;
  float* dz = (r < N ? dL : dR) + base;
  const bool vec = aligned16(p, g, cols) && aligned16(dz, dz, cols);
  if (cols <= 1024 * 4) {
    if (vec) row_softmax_bwd<true, 4>(p, g, (int)cols, dz, red);
    else row_softmax_bwd<false, 4>(p, g, (int)cols, dz, red);
  } else if (cols <= 1024 * 8) {
    if (vec) row_softmax_bwd<true, 8>(p, g, (int)cols, dz, red);
    else row_softmax_bwd<false, 8>(p, g, (int)cols, dz, red);
  } else {
    float d = 0.0f;
    for (int64_t c = threadIdx.x; c < cols; c += 256) d = fmaf(p[c], g[c], d);
    d = bsum(d, red);
    for (int64_t c = threadIdx.x; c < cols; c += 256) dz[c] = p[c] * (g[c] - d);
  }
}

// d emis[T, v] = sum_{(b,i): tok = v} grad_log_emit[b, i, T]  -  softmax(emis[T, :])[v] * tot[T].
// One workgroup owns a tile of 64 preterminals x kVChunk vocabulary entries and accumulates the token contributions in LDS.
// Deterministic: the tokens of a segment are listed in position order, in four lists by token id mod 4, one per
// wavefront, so every LDS word has one owner that adds in position order (eight positions' loads in flight).  The
// tile's part of the table is loaded before the tokens are looked through, and the tile is written once, coalesced along v.
// P = 2048, V = 10000, 1400 tokens: 73 us (36 us of traffic); one wavefront per tile, adding a token at a time, took 332 us.
__global__ void __launch_bounds__(256) k_emis_grad(LenArg la, int B, int n_max, int P, int V,
                                                   const int32_t* __restrict__ tokens, const float* __restrict__ ge,
                                                   const float* __restrict__ emis, const float* __restrict__ lse,
                                                   const float* __restrict__ part, float* __restrict__ d) {
  __shared__ float tile[kVChunk][65];
  __shared__ int list[kSeg];
  __shared__ int cnt[64], first[65];  // [list][quarter of the segment][wavefront]
  __shared__ float tot[64], ls[64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int t0 = blockIdx.x * 64, t = t0 + lane;
  const int positions = B * n_max, chunks = (V + kVChunk - 1) / kVChunk;
  if (wave == 0) {
    float s = 0.0f;
    if (t < P) {
#pragma unroll
      for (int c = 0; c < kColChunks; ++c) s += part[(int64_t)c * P + t];
    }
    tot[lane] = s;
    ls[lane] = t < P ? lse[t] : 0.0f;
  }
  for (int vc = blockIdx.y; vc < chunks; vc += gridDim.y) {
    const int v0 = vc * kVChunk, nv = min(kVChunk, V - v0);
    float ea[16], eb[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int tr = min(t0 + wave * 16 + r, P - 1);
      const float* row = emis + (int64_t)tr * V + v0;
      ea[r] = lane < nv ? row[lane] : 0.0f;
      eb[r] = lane + 64 < nv ? row[lane + 64] : 0.0f;
    }
    __syncthreads();  // the tile of the chunk before has been written out
    for (int v = wave; v < kVChunk; v += 4) tile[v][lane] = 0.0f;
    for (int seg = 0; seg < positions; seg += kSeg) {
      int rel[kSeg / 256];
#pragma unroll
      for (int j = 0; j < kSeg / 256; ++j) {
        const int p = seg + j * 256 + threadIdx.x;
        rel[j] = -1;
        if (p < positions) {
          const int b = p / n_max;
          const int tok = tokens[p];
          if (p - b * n_max < la.v[b] && tok >= v0 && tok < v0 + nv) rel[j] = tok - v0;
        }
      }
      int before[kSeg / 256];  // entries of the same list, quarter and wavefront before this one
#pragma unroll
      for (int j = 0; j < kSeg / 256; ++j) {
        before[j] = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const unsigned long long m = __ballot(rel[j] >= 0 && (rel[j] & 3) == q);
          if (lane == 0) cnt[q * 16 + j * 4 + wave] = __popcll(m);
          if ((rel[j] & 3) == q) before[j] = __popcll(m & ((1ull << lane) - 1));
        }
      }
      __syncthreads();  // counts (and, in the first segment, the cleared tile) are there; the list before has been used
      if (wave == 0) {
        int s = cnt[lane];
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const int below = __shfl_up(s, o, 64);
          if (lane >= o) s += below;
        }
        first[lane + 1] = s;
        if (lane == 0) first[0] = 0;
      }
      __syncthreads();
      if (first[64] == 0) continue;
#pragma unroll
      for (int j = 0; j < kSeg / 256; ++j)
        if (rel[j] >= 0)
          list[first[(rel[j] & 3) * 16 + j * 4 + wave] + before[j]] = ((seg + j * 256 + threadIdx.x) << 8) | rel[j];
      __syncthreads();
      const int end = first[wave * 16 + 16];
      for (int h = first[wave * 16]; h < end; h += 8) {
        int e[8];
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          e[u] = list[min(h + u, end - 1)];
          v[u] = t < P ? ge[(int64_t)(e[u] >> 8) * P + t] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (h + u < end) tile[e[u] & 255][lane] += v[u];
      }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = wave * 16 + r;
      if (t0 + row >= P) break;
      float* o = d + (int64_t)(t0 + row) * V + v0;
      if (lane < nv) o[lane] = tile[lane][row] - expf(ea[r] - ls[row]) * tot[row];
      if (lane + 64 < nv) o[lane + 64] = tile[lane + 64][row] - expf(eb[r] - ls[row]) * tot[row];
    }
  }
}

int check(int N, int P, int V, int B, int n_max, const int32_t* lengths, LenArg* la) {
  if (N < 1 || P < 1 || V < 1 || N > (1 << 16) || P > (1 << 16) || V > (1 << 24)) return SPCFG_ERR_SHAPE;
  if (B < 1 || B > kMaxB || n_max < 1 || n_max > kMaxLen) return SPCFG_ERR_SHAPE;
  if (!lengths) return SPCFG_ERR_ARG;
  for (int b = 0; b < B; ++b) {
    if (lengths[b] < 0 || lengths[b] > n_max) return SPCFG_ERR_LENGTH;
    la->v[b] = lengths[b];
  }
  return SPCFG_OK;
}

dim3 tile_grid(int P, int V) {
  const int chunks = (V + kVChunk - 1) / kVChunk;
  return dim3((P + 63) / 64, chunks < kMaxVBlocks ? chunks : kMaxVBlocks);
}

int status() { return hipGetLastError() == hipSuccess ? SPCFG_OK : SPCFG_ERR_HIP; }

}  // namespace
}  // namespace spcfg

using namespace spcfg;

extern "C" {

int spcfg_rules_forward(int32_t N, int32_t P, int32_t V, const float* root_logits, const float* L_logits,
                        const float* R_logits, const float* emis_logits, const int32_t* tokens, const int32_t* lengths,
                        int32_t B, int32_t n_max, float* log_root, float* L, float* R, float* log_emit, float* emis_lse,
                        void* hip_stream) {
  LenArg la;
  int rc = check(N, P, V, B, n_max, lengths, &la);
  if (rc) return rc;
  if (!root_logits || !L_logits || !R_logits || !emis_logits || !tokens || !log_root || !L || !R || !log_emit ||
      !emis_lse)
    return SPCFG_ERR_ARG;
  hipStream_t st = (hipStream_t)hip_stream;
  hipLaunchKernelGGL(k_rows_forward, dim3(P + 2 * N + 1), dim3(256), 0, st, N, P, (int64_t)V, root_logits, L_logits, R_logits,
                     emis_logits, log_root, L, R, emis_lse);
  hipLaunchKernelGGL(k_gather_emit, dim3(B * n_max), dim3(256), 0, st, la, n_max, P, V, emis_logits, emis_lse, tokens, log_emit);
  return status();
}

int spcfg_rules_backward(int32_t N, int32_t P, int32_t V, const float* log_root, const float* L, const float* R,
                         const float* emis_logits, const float* emis_lse, const int32_t* tokens,
                         const int32_t* lengths, int32_t B, int32_t n_max, const float* grad_log_root,
                         const float* grad_L, const float* grad_R, const float* grad_log_emit, float* grad_root_logits,
                         float* grad_L_logits, float* grad_R_logits, float* grad_emis_logits, float* scratch,
                         void* hip_stream) {
  LenArg la;
  int rc = check(N, P, V, B, n_max, lengths, &la);
  if (rc) return rc;
  if (!log_root || !L || !R || !emis_logits || !emis_lse || !tokens || !grad_log_root || !grad_L || !grad_R ||
      !grad_log_emit || !grad_root_logits || !grad_L_logits || !grad_R_logits || !grad_emis_logits || !scratch)
    return SPCFG_ERR_ARG;
  hipStream_t st = (hipStream_t)hip_stream;
  hipLaunchKernelGGL(k_rows_backward, dim3((P + 63) / 64 * (kColChunks / 4) + 2 * N + 1), dim3(256), 0, st, la, B, n_max, N, P,
                     log_root, L, R, grad_log_root, grad_L, grad_R, grad_log_emit, grad_root_logits, grad_L_logits,
                     grad_R_logits, scratch);
  hipLaunchKernelGGL(k_emis_grad, tile_grid(P, V), dim3(256), 0, st, la, B, n_max, P, V, tokens, grad_log_emit, emis_logits,
                     emis_lse, scratch, grad_emis_logits);
  return status();
}

}  // extern "C"
