// Projection products with few rows (the short widths' launches of small grammars, the last widths of large ones):
// C[r][c] = sum_k A[r][k] * Bm[c][k] on fp32 operands, as the split products of gemm_nt.hip.
//
// What bounds such a launch is latency, not the matrix rate: gemm_nt.hip shares (tile, K-step) units between workgroups
// and pays for a barrier pair per K-step, for the exchange of partial tiles through memory and for the arrival
// counters.  Here nothing leaves the workgroup: a workgroup owns one small output tile over its whole K range, its 8 or
// 16 wavefronts take every 8th or 16th K-step of 32 values, and their partial sums meet once, in LDS, in wavefront order.
//  * Each wavefront streams its own K-steps global -> LDS (1 KB per instruction, whole 128-byte lines: 8 rows x 32
//    values) into a ring of its own: the only waits are its own load counter, the only barrier is the one before the
//    final sum.  A stage is refilled as soon as its operands are in registers.
//  * LDS rows are 128 bytes; the 16-byte chunk index is XORed with a key of the row (chunk_key, on the global side of the
//    load), so the 16-byte operand reads meet no bank conflict.
//  * Every operand value is cut into its three bf16 pieces (nt::Split3) by the one lane that multiplies it; fp32 matrix
//    instructions instead of the cut were 5 % faster on 16 x 16 tiles and 10-60 % slower on all larger ones.
//  * blockIdx.x is the column tile: workgroups go to the eight XCDs in turn, so where the columns are a multiple of 128 * NI
//    the row tiles of one column tile read their share of the panel through the same L2; elsewhere through several.
// Measured against gemm_nt.hip (us per launch, N = 1024, forward shape 2N columns, K = N / reverse shape N columns, K = 2N):
// 16 rows 11.5 -> 4.1 / 13.3 -> 6.0; 64 rows 13.1 -> 5.8 / 16.4 -> 8.0; 200 rows 20.3 -> 10.4 / 21.8 -> 11.3;
// 600 rows 32.8 -> 26.7 / 31.6 -> 26.2.  N = 2048: 16 rows 15.7 -> 6.7 / 18.9 -> 10.2; 200 rows 37.1 -> 28.4 / 41.7 -> 30.9;
// 300 rows 46.2 -> 49.8 / 47.1 -> 45.8.
#include "gemm_nt_common.h"

namespace spcfg {

namespace {

using namespace nt;

// Both 16-byte chunks that this lane contributes to a 16-row operand of one 32-wide K-step (issued only: see wait_lds).
struct Raw { floatx4 u, v; };
// NF operands (16 rows = 2048 bytes apart) read and waited for in one block
template <int NF> __device__ __forceinline__ void read_frags(Raw (&f)[NF], unsigned a0, unsigned a1);
#define SPCFG_RD(D, A, O) "ds_read_b128 %" #D ", %" #A " offset:" #O "\n\t"
template <> __device__ __forceinline__ void read_frags<2>(Raw (&f)[2], unsigned a0, unsigned a1) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile(SPCFG_RD(0, 4, 0) SPCFG_RD(1, 5, 0) SPCFG_RD(2, 4, 2048) SPCFG_RD(3, 5, 2048) "s_waitcnt lgkmcnt(0)"
               : "=&v"(f[0].u), "=&v"(f[0].v), "=&v"(f[1].u), "=&v"(f[1].v) : "v"(a0), "v"(a1) : "memory");
#else
  (void)f; (void)a0; (void)a1;
#endif
}
template <> __device__ __forceinline__ void read_frags<3>(Raw (&f)[3], unsigned a0, unsigned a1) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile(SPCFG_RD(0, 6, 0) SPCFG_RD(1, 7, 0) SPCFG_RD(2, 6, 2048) SPCFG_RD(3, 7, 2048) SPCFG_RD(4, 6, 4096)
               SPCFG_RD(5, 7, 4096) "s_waitcnt lgkmcnt(0)"
               : "=&v"(f[0].u), "=&v"(f[0].v), "=&v"(f[1].u), "=&v"(f[1].v), "=&v"(f[2].u), "=&v"(f[2].v)
               : "v"(a0), "v"(a1) : "memory");
#else
  (void)f; (void)a0; (void)a1;
#endif
}
template <> __device__ __forceinline__ void read_frags<4>(Raw (&f)[4], unsigned a0, unsigned a1) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile(SPCFG_RD(0, 8, 0) SPCFG_RD(1, 9, 0) SPCFG_RD(2, 8, 2048) SPCFG_RD(3, 9, 2048) SPCFG_RD(4, 8, 4096)
               SPCFG_RD(5, 9, 4096) SPCFG_RD(6, 8, 6144) SPCFG_RD(7, 9, 6144) "s_waitcnt lgkmcnt(0)"
               : "=&v"(f[0].u), "=&v"(f[0].v), "=&v"(f[1].u), "=&v"(f[1].v), "=&v"(f[2].u), "=&v"(f[2].v),
                 "=&v"(f[3].u), "=&v"(f[3].v)
               : "v"(a0), "v"(a1) : "memory");
#else
  (void)f; (void)a0; (void)a1;
#endif
}
template <> __device__ __forceinline__ void read_frags<6>(Raw (&f)[6], unsigned a0, unsigned a1) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile(SPCFG_RD(0, 12, 0) SPCFG_RD(1, 13, 0) SPCFG_RD(2, 12, 2048) SPCFG_RD(3, 13, 2048) SPCFG_RD(4, 12, 4096)
               SPCFG_RD(5, 13, 4096) SPCFG_RD(6, 12, 6144) SPCFG_RD(7, 13, 6144) SPCFG_RD(8, 12, 8192)
               SPCFG_RD(9, 13, 8192) SPCFG_RD(10, 12, 10240) SPCFG_RD(11, 13, 10240) "s_waitcnt lgkmcnt(0)"
               : "=&v"(f[0].u), "=&v"(f[0].v), "=&v"(f[1].u), "=&v"(f[1].v), "=&v"(f[2].u), "=&v"(f[2].v),
                 "=&v"(f[3].u), "=&v"(f[3].v), "=&v"(f[4].u), "=&v"(f[4].v), "=&v"(f[5].u), "=&v"(f[5].v)
               : "v"(a0), "v"(a1) : "memory");
#else
  (void)f; (void)a0; (void)a1;
#endif
}
template <> __device__ __forceinline__ void read_frags<8>(Raw (&f)[8], unsigned a0, unsigned a1) {
  Raw lo[4], hi[4];
  read_frags<4>(lo, a0, a1);
  read_frags<4>(hi, a0 + 8192, a1 + 8192);
#pragma unroll
  for (int q = 0; q < 4; ++q) { f[q] = lo[q]; f[q + 4] = hi[q]; }
}
#undef SPCFG_RD

// What the 16-byte chunk index of an LDS row is XORed with.  The 64 lanes of a 16-byte read are served sixteen at a time, and
// not in order: rows 0-3 and 12-15 of one chunk go with rows 4-11 of the next.  With the row's pair number as the key these
// two sets fell on the same banks (LdsBankConflict 0.7 to 0.9 in every launch); moved on by two they fall on different
// ones (0.0000).  The launches take the same time either way: they wait for memory.
__device__ __forceinline__ int chunk_key(int row) { return ((row >> 1) + 2) & 7; }

template <int EPI>
__device__ __forceinline__ void store_one(const NtArgs& g, int r, int c, int c_shift, float acc) {
  float scale = 1.0f;
  int64_t drow = r;
  if (EPI == NT_EPI_MASKROWS && g.rowmask[r]) return;
  if (EPI == NT_EPI_LEAF_EMIT) {
    const int q = g.rowexp[r];
    scale = (q == kExpZero || q < -160) ? 0.0f : ldexpf(1.0f, min(q, 127));
    drow = (int64_t)g.row_b[r] * g.n_max + g.row_i[r];
  } else {  // normalising shift of the input row, as in nt::epilogue
    const uint32_t mb = g.rowmaxb[r];
    const int f = max((int)((mb >> 23) & 0xffu) - 126, -126);
    scale = mb == 0u ? 0.0f : ldexpf(1.0f, -f);
  }
  float val = acc * scale;
  if (EPI == NT_EPI_LEAF_EMIT) val *= g.E[(int64_t)r * g.lde + c];
  g.C[drow * g.ldc + c + c_shift] = val;
}

template <int EPI, int MI, int NI, int NW, int ST, int MODE>
__global__ void __launch_bounds__(NW * 64) k_gemm_short(NtArgs g) {
  constexpr int BMS = 16 * MI, BNS = 16 * NI, NF = MI + NI;
  constexpr int ND = 2 * NF;                 // 1 KB loads of a wavefront per K-step
  constexpr int kStageBytes = NF * 2048;
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int row0, row_end, c_shift = 0, kbeg = 0, steps = g.K / 32;
  const float* bmat = static_cast<const float*>(g.Bm);
  if (MODE == 1) {  // one grammar per sentence: blockIdx.z is the sentence
    const int b = blockIdx.z;
    const int cnt = g.grp_lens[b] - g.grp_w + 1;
    if ((int)blockIdx.y * BMS >= cnt) return;
    const int first = (int)(g.grp_rowbase[b] - g.grp_row_first);
    row0 = first + blockIdx.y * BMS;
    row_end = first + cnt;
    bmat += b * g.grp_b_stride;
  } else if (MODE == 2) {  // parts: blockIdx.y runs over the row tiles of all parts
    int p = 0, ty = blockIdx.y;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (p == q && q + 1 < g.parts) {
        const int tq = (g.prt_rows[q] + BMS - 1) / BMS;
        if (ty >= tq) { ty -= tq; p = q + 1; }
      }
    }
    row0 = g.prt_row0[p] + ty * BMS;
    row_end = g.prt_row0[p] + g.prt_rows[p];
    c_shift = g.prt_c0[p];
    kbeg = g.prt_kbeg[p] * 32;
    steps = g.prt_kt[p];
    bmat += (int64_t)c_shift * g.ldb;
  } else {
    row0 = blockIdx.y * BMS;
    row_end = g.rows;
  }
  const int col0 = blockIdx.x * BNS;

  // lane -> (row of eight, 16-byte chunk) of a load
  const int l8 = lane >> 3;
  const float* gp[ND];
#pragma unroll
  for (int q = 0; q < ND; ++q) {
    const int ch = (lane & 7) ^ chunk_key(((q & 1) << 3) | l8);
    if (q < 2 * MI)
      gp[q] = static_cast<const float*>(g.A) + (int64_t)min(row0 + q * 8 + l8, row_end - 1) * g.lda + kbeg + ch * 4;
    else
      gp[q] = bmat + (int64_t)min(col0 + (q - 2 * MI) * 8 + l8, g.cols - 1) * g.ldb + kbeg + ch * 4;
  }
  unsigned char* ring = smem + (size_t)wave * ST * kStageBytes;
  const unsigned ring_a = lds_address(ring);
  const int fr = lane & 15, kq = lane >> 4;
  const unsigned fa0 = ring_a + fr * 128 + (((2 * kq) ^ chunk_key(fr)) << 4);
  const unsigned fa1 = ring_a + fr * 128 + (((2 * kq + 1) ^ chunk_key(fr)) << 4);

  floatx4 acc[MI][NI];
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) acc[mi][ni] = floatx4{0.f, 0.f, 0.f, 0.f};

  const int n = (steps - wave + NW - 1) / NW;  // this wavefront's K-steps: wave, wave + NW, ... (may be none)
  auto issue = [&](int t, int stage) {
    const int k = (wave + t * NW) * 32;
#pragma unroll
    for (int q = 0; q < ND; ++q) dma16(gp[q] + k, ring_a + stage * kStageBytes + q * 1024);
  };
#pragma unroll
  for (int s = 0; s < ST; ++s)
    if (s < n) issue(s, s);
  int stage = 0;
  for (int t = 0; t < n; ++t) {
    const int left = n - t;  // steps in flight: min(ST, left)
    if (left >= ST) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(ND * (ST - 1)) : "memory");
    else if (ST > 3 && left == 3) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(ND * 2) : "memory");
    else if (ST > 2 && left == 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(ND) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    Raw f[NF];
    read_frags<NF>(f, fa0 + stage * kStageBytes, fa1 + stage * kStageBytes);
    if (t + ST < n) issue(t + ST, stage);  // the stage's operands are in registers
    stage = stage + 1 == ST ? 0 : stage + 1;
    Split3 x[NF];
#pragma unroll
    for (int q = 0; q < NF; ++q) x[q].cut(__builtin_bit_cast(float4, f[q].u), __builtin_bit_cast(float4, f[q].v));
#define SPCFG_T(X, Y)                                                                                         \
  _Pragma("unroll") for (int mi = 0; mi < MI; ++mi)                                                           \
    _Pragma("unroll") for (int ni = 0; ni < NI; ++ni)                                                         \
      acc[mi][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[mi].X(), x[MI + ni].Y(), acc[mi][ni], 0, 0, 0);
    SPCFG_T(l, h) SPCFG_T(h, l) SPCFG_T(m, m) SPCFG_T(m, h) SPCFG_T(h, m) SPCFG_T(h, h)
#undef SPCFG_T
  }
  // partial sums of the wavefronts, each in its own ring (nothing is in flight any more), summed in wavefront order
  constexpr int kTile = BMS * BNS;
  static_assert(kTile * 4 <= ST * kStageBytes, "a partial tile has to fit its wavefront's ring");
  float* part = reinterpret_cast<float*>(ring);
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int v = 0; v < 4; ++v) part[((mi * NI + ni) * 4 + v) * 64 + lane] = acc[mi][ni][v];
  __syncthreads();
#pragma unroll
  for (int e0 = 0; e0 < kTile; e0 += NW * 64) {
    const int e = e0 + tid;
    if (kTile < NW * 64 && e >= kTile) break;
    const float* src = reinterpret_cast<const float*>(smem) + e;
    float s = 0.0f;
#pragma unroll
    for (int q = 0; q < NW; ++q) s += src[q * (ST * kStageBytes / 4)];
    const int l = e & 63, v = (e >> 6) & 3, t = e >> 8;
    const int r = row0 + (t / NI) * 16 + 4 * (l >> 4) + v, c = col0 + (t % NI) * 16 + (l & 15);
    if (r < row_end && c < g.cols) store_one<EPI>(g, r, c, c_shift, s);
  }
}

template <int EPI, int MI, int NI, int NW, int ST, int MODE>
void launch_cfg(const NtArgs& a, hipStream_t st) {
  constexpr size_t lds = (size_t)NW * ST * (MI + NI) * 2048;
  static bool attr_set = false;
  if (!attr_set) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_short<EPI, MI, NI, NW, ST, MODE>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    attr_set = true;
  }
  const int tn = (a.cols + 16 * NI - 1) / (16 * NI);
  int tm = 0;
  if (MODE == 1) tm = (a.grp_max_rows + 16 * MI - 1) / (16 * MI);
  else if (MODE == 2) for (int p = 0; p < a.parts; ++p) tm += (a.prt_rows[p] + 16 * MI - 1) / (16 * MI);
  else tm = (a.rows + 16 * MI - 1) / (16 * MI);
  if (tm <= 0) return;
  launch_k(k_gemm_short<EPI, MI, NI, NW, ST, MODE>, dim3(tn, tm, MODE == 1 ? a.ngroups : 1), dim3(NW * 64), lds, st, a);
}

// Tile shapes: 16 * MI rows x 16 * NI columns, NW wavefronts, ST stages per ring.  One workgroup per CU except for the
// 32 x 32 tile (two).  Time of a launch, from sweeps at N = 192 .. 2048 and 5 .. 600 rows (within 10-15 %):
//   2 us + rounds * (fixed + slope * K / 1024),  rounds = workgroups / 256 rounded up.
// Tall tiles cost less per output (fewer loads and cuts), short ones finish a K range sooner while CUs are idle.
struct Shape { int mi, ni; double fixed, slope; };
constexpr Shape kShapes[] = {{1, 1, 0.2, 1.95}, {2, 1, 0.6, 2.6}, {2, 2, 0.7, 3.9}, {4, 2, 1.4, 6.2}, {4, 4, 3.0, 9.55}};
constexpr int kNumShapes = 5;

// Workgroups of a launch with this shape (grouped: an upper bound for 16-row tiles)
int64_t workgroups(const NtArgs& a, const Shape& s) {
  const int bm = 16 * s.mi;
  int64_t tm = 0;
  if (a.grouped) tm = bm == 16 ? 2 * (int64_t)a.grp_tiles_m[0] : a.grp_tiles_m[bm == 32 ? 0 : 1];
  else if (a.parts > 0) for (int p = 0; p < a.parts; ++p) tm += (a.prt_rows[p] + bm - 1) / bm;
  else tm = (a.rows + bm - 1) / bm;
  return tm * ((a.cols + 16 * s.ni - 1) / (16 * s.ni));
}

// The shape with the least estimated time, or -1 where gemm_nt.hip's kernels are faster: launches tall enough for their
// 128-row tiles, and those whose estimate is not below theirs (about 15 us + 12.5 us per 10^9 multiply-accumulates for the
// launches with 32- and 64-row tiles; 10 % off for the errors of both estimates).
int pick_shape(const NtArgs& a) {
  if (a.fp32_mfma || chosen_bm(a) == 128) return -1;
  int best = -1;
  double t_best = 0.9 * (15.0 + 12.5e-9 * work_of(a) * (a.grouped ? a.ngroups : 1));
  for (int i = 0; i < kNumShapes; ++i) {
    const double rounds = (double)((workgroups(a, kShapes[i]) + 255) / 256);
    const double t = 2.0 + rounds * (kShapes[i].fixed + kShapes[i].slope * a.K / 1024.0);
    if (t < t_best) { t_best = t; best = i; }
  }
  return best;
}

template <int EPI, int MODE>
void launch_shape(int shape, const NtArgs& a, hipStream_t st) {
  switch (shape) {
    case 0: launch_cfg<EPI, 1, 1, 16, 2, MODE>(a, st); break;
    case 1: launch_cfg<EPI, 2, 1, 16, 1, MODE>(a, st); break;
    case 2: launch_cfg<EPI, 2, 2, 8, 1, MODE>(a, st); break;
    case 3: launch_cfg<EPI, 4, 2, 8, 1, MODE>(a, st); break;
    default: launch_cfg<EPI, 4, 4, 8, 1, MODE>(a, st); break;
  }
}
template <int EPI>
void launch_mode(int shape, const NtArgs& a, hipStream_t st) {
  if (a.grouped) launch_shape<EPI, 1>(shape, a, st);
  else if (a.parts > 0) launch_shape<EPI, 2>(shape, a, st);
  else launch_shape<EPI, 0>(shape, a, st);
}

}  // namespace

bool launch_gemm_short(const NtArgs& a, hipStream_t st) {
  const int shape = pick_shape(a);
  if (shape < 0) return false;
  switch (a.epilogue) {
    case NT_EPI_ROWSCALE: launch_mode<NT_EPI_ROWSCALE>(shape, a, st); break;
    case NT_EPI_MASKROWS: launch_mode<NT_EPI_MASKROWS>(shape, a, st); break;
    default: launch_mode<NT_EPI_LEAF_EMIT>(shape, a, st); break;
  }
  return true;
}

}  // namespace spcfg
