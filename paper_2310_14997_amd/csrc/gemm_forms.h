// Host rules: in which form a product on bf16 planes runs.  Kept apart from the launchers so that a program without device code
// can ask them.
#pragma once
#include "gemm_nt_common.h"

namespace spcfg {
namespace nt {

constexpr int BK3 = 32;  // K values per step and plane: one 64-byte row

// Output tiles and (tile, K-step) units of a launch with this tile shape; kt: the steps of a tile, 0 where parts differ in them.
struct Units { int tiles, total, kt; };
inline Units units_of(const NtArgs& a, int bm, int bn, int ks) {
  const int tiles_n = (a.cols + bn - 1) / bn;
  Units u{0, 0, a.K / (BK3 * ks)};
  if (a.parts == 0) {
    u.tiles = ((a.rows + bm - 1) / bm) * tiles_n;
    u.total = u.tiles * u.kt;
    return u;
  }
  u.kt = -1;
  for (int p = 0; p < a.parts; ++p) {
    const int tp = ((a.prt_rows[p] + bm - 1) / bm) * tiles_n, kt = a.prt_kt[p] / ks;
    u.tiles += tp;
    u.total += tp * kt;
    if (tp > 0) u.kt = u.kt < 0 || u.kt == kt ? kt : 0;
  }
  if (u.kt < 0) u.kt = 0;
  return u;
}

// Forms of a projection product on one or two planes, and what a launch takes in each, in us (all but the turn-around that the
// forms have in common).  The form of least estimated time is taken: tile shape, whole tiles (a workgroup an output tile) or equal shares, and, on
// one plane, the kernel that stages tiles through registers (gemm_nt16.hip), for which a launch becomes one product without
// parts.
//  * Planes kernel (gemm_nt3.hip), per K-step of a workgroup: b + c * (share of the chip that is busy), since operands come from L2
//    and past it; `fixed` for the first stages of the ring and the epilogue.  Shares pay an exchange (`cut`) on top, unless they are tiles;
//    whole tiles their last, partly filled round.  More than one round of 64-row tiles reads the panel over and over, kShortRounds times as
//    long a step (N = 3072, 768 rows: 61.6 us, 50 by the steps of a single round).
//  * Register-staged kernel, with tiles of 32 rows only (its taller ones, 25 to 31 us for 112 to 480 rows at N = 3520, were never the
//    fastest): the same with two workgroups a CU, and kNextTile where a share goes on to another tile.
// Fitted to 684 launches on one and 323 on two planes (N = 64 .. 4096, 1 to 64 sentences, 6 to 2000 rows, both directions), every form
// timed with the caches' contents replaced between launches: on average a launch takes 1.008 (one plane) and 1.009 (two) times its fastest
// form's time.  With shapes fitted at N = 4096 only, 32-row tiles always in shares and the staged kernel for all of K <= 1024 it
// was 1.085 and 1.043 (N = 1280, 10 rows 11.2 us, 9.0 so; N = 768 reverse, 1984 rows 30.8, 15.9; N = 512 on two planes, 1984 rows
// 28.6, 17.3), with the staged kernel throughout 1.165 (N = 3072, 1056 rows 96.5 us, 46.4).
struct Shape3 { int bm, bn; double fixed[2], cut[2], b[2], c[2]; };  // (one plane, 64 values a step; two planes, 32)
constexpr Shape3 kShapes3[] = {
    {128, 256, {2.3, 3.2}, {16.0, 16.5}, {0.50, 0.64}, {0.41, 0.70}},
    {128, 128, {2.3, 3.2}, {12.5, 11.0}, {0.28, 0.35}, {0.27, 0.42}},
    {64, 128, {2.3, 3.2}, {7.3, 7.0}, {0.26, 0.277}, {0.05, 0.09}},
    {32, 128, {1.0, 1.0}, {4.5, 3.1}, {0.20, 0.25}, {0.08, 0.127}},
};
constexpr int kStaged = 4;  // (in the place of an index into kShapes3)
constexpr double kShortRounds = 1.2, kNextTile = 2.0;
constexpr double kStagedCut = 2.4, kStagedB = 0.34, kStagedC = 0.345;

struct Form { int shape; bool whole, parts; };

inline int least(int a, int b) { return a < b ? a : b; }

inline double planes_us(const NtArgs& a, const Units& u, const Shape3& s, bool whole) {
  const int pl = a.planes3 - 1;
  const double more = s.bm == 64 && u.tiles > 256 ? kShortRounds : 1.0, b = more * s.b[pl], c = more * s.c[pl];
  if (whole) {
    const int rest = u.tiles % 256;
    return s.fixed[pl] + u.kt * (u.tiles / 256 * (b + c) + (rest ? b + c * rest / 256.0 : 0.0));
  }
  // (the partial-tile scratch holds 2 * max_wgs slots of 128 x 128; at least two K-steps a share)
  const int wgs = least(least(256, a.max_wgs * (128 / s.bm) * 128 / s.bn), u.total > 3 ? u.total / 2 : 1);
  const int share = (u.total + wgs - 1) / wgs;
  if (u.kt > 0 && share % u.kt == 0)
    return s.fixed[pl] + share * (b + c * least(256, (u.total + share - 1) / share) / 256.0) + kNextTile * (share / u.kt - 1);
  return s.fixed[pl] + s.cut[pl] + share * (b + c);
}
inline double staged_us(const NtArgs& a) {  // (a: without parts)
  const int kt = a.K / 64, total = ((a.rows + 31) / 32) * ((a.cols + BN - 1) / BN) * kt;
  int wgs = least(least(pick_wgs(total, 64), a.max_wgs * 4), total > 3 ? total / 2 : 1);
  const int share = (total + wgs - 1) / wgs;
  wgs = (total + share - 1) / share;
  const double step = (wgs > 256 ? wgs / 256.0 : 1.0) * (kStagedB + kStagedC * least(wgs, 256) / 256.0);
  return (share % kt == 0 ? 0.0 : kStagedCut) + share * step + kNextTile * ((share - 1) / kt);
}
// The launch as one product: without the parts, whose left-out halves are zeros (reverse) or not read (forward).
inline void drop_parts(NtArgs& a) {
  if (a.parts == 2) a.cols += a.prt_c0[1];
  a.parts = 0;
}
inline Form pick_form(const NtArgs& a) {
  Form best{0, false, a.parts > 0};
  double t_best = 1e30;
  auto consider = [&](double t, int shape, bool whole, bool parts) {
    if (t < t_best) { t_best = t; best = Form{shape, whole, parts}; }
  };
  NtArgs one = a;
  drop_parts(one);
  if (a.planes3 == 1 && chosen_bm(one) == 32) consider(staged_us(one), kStaged, false, false);
  for (int i = 0; i < 4; ++i) {
    const Shape3& s = kShapes3[i];
    // (the reverse product's parts round their rows up to tiles each; where they save nothing it runs as one)
    for (int parts = a.parts == 2 ? 1 : 0; parts <= (a.parts > 0 ? 1 : 0); ++parts) {
      const NtArgs& l = parts ? a : one;
      const Units u = units_of(l, s.bm, s.bn, a.planes3 == 1 ? 2 : 1);
      if (u.total == 0) continue;
      consider(planes_us(l, u, s, false), i, false, parts != 0);
      if (s.bm > 32 && u.kt > 0) consider(planes_us(l, u, s, true), i, true, parts != 0);
    }
  }
  return best;
}

// Steps of a workgroup's share of a rule-gradient product (gemm_tn3.hip) of `tiles` output tiles and KT steps each; KT: whole tiles.
// A tile costs its share's steps in a row, then the last workgroup adds up KT / share partial tiles at about half a step's time
// each: shares of at least sqrt(KT / 2) steps balance the two when few tiles would be cut for the whole chip.
// B = 7, N = 141, n <= 37 (6 tiles of 66 steps): whole call 638 -> 620 us; larger outputs have longer shares anyway.
// On one plane a short reduction is not worth the exchange, and more than one round of whole tiles pays its last, partly filled round
// in full; estimated in us from 90 launches timed both ways (N = 192 .. 4096, 6 to 390 steps), with 64-row steps of b + c * (share
// of the chip that is busy): 1.007 times the faster way's time on average.  16 tiles of 6 steps 11.3 us whole, 19.0 in shares; 144 of
// 20 22.9, 33.0; 297 tiles (N = 2112) of 390 668, 452; 324 of 150 235, 194.  With whole tiles wherever a share comes within 14
// steps of a tile or past it, 1.061.  With three planes whole tiles would be faster for short reductions as well, but the longer sums
// are less accurate (N = 141, 7 sentences: 1.2e-7 from 64 bits instead of 8.5e-8).
constexpr double kTnB = 0.57, kTnC = 0.37, kTnRound = 2.0, kTnCut = 8.0, kTnPart = 2.0;
inline int tn3_share(int planes, int tiles, int KT, int max_wgs) {
  const int total = tiles * KT;
  // (one workgroup per CU; the partial-tile scratch holds 2 * max_wgs slots of 128 x 128, a tile on one plane is two of them)
  const int wgs = least(least(256, planes == 1 ? max_wgs / 2 : max_wgs), total > 3 ? total / 2 : 1);
  int share = (total + wgs - 1) / wgs;
  while (2 * (int64_t)share * share < KT) ++share;
  if (planes != 1) return share;
  const int busy = least(256, (total + share - 1) / share), rest = tiles % 256;
  const double whole = kTnRound * ((tiles + 255) / 256) + KT * (tiles / 256 * (kTnB + kTnC) + (rest ? kTnB + kTnC * rest / 256.0 : 0.0));
  const double cut = kTnCut + kTnPart * (share < KT ? (KT + share - 1) / share : 2) +
                     share * (kTnB + kTnC * busy / 256.0) + kTnRound * ((share + KT - 1) / KT);
  return whole < cut ? KT : share;
}

}  // namespace nt
}  // namespace spcfg
