// Which kernel runs a linear layer on fragment-packed operands, on the host: the wave-level kernel (wgemm.hip) or a tile shape and parts
// of K of the workgroup-tile kernel (bgemm.hip).  A decision on sizes and kinds alone, apart from the kernels so that it can be
// asked without them.
#pragma once
#include <cmath>

#include "wgemm.h"

namespace df {

// Tile shapes.  `slab` and `epi` are the microseconds of a round of workgroups per 64 of K and for prologue + epilogue
// (GEGLU, QKV, plain / residual, fused cross-attention), `base` those of a launch, `alone` the round of a workgroup that
// has a unit to itself where two would fit, `kf` the k-fragments of a stage; fitted to 38 token counts x 8 layers with weights
// that no cache holds.  Chosen by them (and the time of the wave-level kernel, below), those layers take 1.3 % more than with the
// best of 18 shapes.  The columns of GEGLU, QKV and cross-attention are from after the epilogues in the accumulators: GEGLU layers of 256 -
// 7200 tokens (18 counts x 2) take 1.4 % more than with the best of the nine shapes that have it, QKV and cross-attention layers in the
// step (7 images x 2 levels) were fitted to the step's time, cross-attention again (20 images) after the wave-level kernel spread it over
// its waves: 4096 tokens of 640 features 2.3 us less on 128 x 128 with a unit to itself, 1224 of 1280 about 3 less on the wave-level kernel.  The 96-, 160- and 192-wide tiles and 256 x 256 are there because a round of workgroups over 256 units is
// rarely full: 7200 x 640 x 2560 44.9 -> 33.2 us, 4096 x 1280 x 1280 28.8 -> 24.7, 1976 x 640 x 2560 23.3 -> 18.1, 4096 x 3840 x
// 1280 55.7 -> 44.2, 494 x 10240 x 1280 with GEGLU 27.3 -> 24.7, 1024 x 1280 x 1280 12.7 -> 12.0.
struct TileCfg { int bt, bf, occ, kf; double base, slab, epi[4], alone; };
constexpr TileCfg kTiles[] = {
    {8, 10, 1, 2, 1.51, 1.886, {8.5, 28.6, 19.2, 1e9}, 1.0},      // 256 x 320, eight waves of 64 x 160
    {4, 4, 2, 4, 3.00, 0.982, {2.2, 3.6, 8.0, 3.2}, 0.71},        // 128 x 128, eight waves of 32 x 64, two workgroups per unit
    {4, 4, 1, 4, 1.59, 0.468, {4.0, 3.6, 6.5, 5.2}, 1.0},         // 128 x 128, four ring stages
    {2, 4, 2, 4, 3.11, 0.602, {3.4, 3.0, 4.8, 8.3}, 0.63},        // 64 x 128, two k-groups, two workgroups per unit
    {2, 2, 2, 8, 2.52, 0.407, {1e9, 2.9, 2.4, 7.3}, 0.78},        // 64 x 64, two k-groups, two workgroups per unit
    {2, 2, 1, 8, 2.31, 0.224, {1e9, 2.8, 2.1, 6.6}, 1.0},         // 64 x 64, two k-groups, four stages of 128 (plain: kPlain64)
    {4, 10, 1, 2, 1.43, 1.056, {6.0, 7.5, 13.3, 1e9}, 1.0},       // 128 x 320, eight waves of 32 x 160
    {2, 3, 1, 8, 2.83, 0.281, {1e9, 4.3, 3.2, 1e9}, 1.0},         // 64 x 96, four k-groups of 32 x 96
    {4, 5, 1, 4, 1.88, 0.551, {1e9, 9.5, 8.6, 1e9}, 1.0},         // 128 x 160, two k-groups of 32 x 160
    {8, 8, 1, 2, 1.04, 1.429, {8.5, 10.0, 17.7, 1e9}, 1.0},       // 256 x 256, eight waves of 64 x 128
    {4, 3, 1, 4, 2.11, 0.412, {1e9, 4.5, 5.1, 1e9}, 1.0},         // 128 x 96, two k-groups of 32 x 96
    {4, 6, 1, 2, 2.24, 0.690, {5.3, 8.0, 7.6, 1e9}, 1.0},         // 128 x 192, eight waves of 32 x 96
};

// Parts of K, for plain layers whose tiles cover part of the chip: one round of workgroups in all.  `fixed` is the time of
// the second launch and of what the parts do beside their stages; each part's sums cost a write and a read.
// kCrowdUs is what parts lose that take more than kCrowd units.  All four are fitted with the wave-level kernel's times of plain layers
// (choose_tile).  By 0.9, 3.0 and a crowd from 200 units on, which one layer of 1280 x 5120 had given, narrower ones split that should not
// have: 224 x 1280 x 3840 11.6 -> 13.9 us, 288 x 960 x 3840 11.2 -> 13.0.
struct SplitCfg { int tile; double fixed; };
constexpr SplitCfg kSplits[] = {{2, 2.0}, {6, 2.2}};
constexpr int kMaxParts = 8, kSplitFamily = 7;          // (the first tiles: those that parts of K were weighed against)
constexpr double kPartUs = 1.9e-6;                     // microseconds per output value and part, and per value of the sums
constexpr double kCrowdUs = 2.0;
constexpr int kCrowd = 224;
constexpr double kPlain64 = 0.008;                     // more per slab of the 64 x 64 tile in a plain layer of the step
// Cross-attention on the 64 x 128 tile: 1224 tokens of 1280 features 11.5, 11.9, 15.2 and 13.7 us against one to four fragments of 32 text
// tokens.  With the third's time for all, the wave-level kernel had 13.8, 14.2, 14.5 and 15.1.
constexpr double kXaEpi64x128 = 6.3;

inline int max_parts(const TileCfg& t, long long MT, long long NF) {
  const long long n = ((MT + t.bt - 1) / t.bt) * ((NF + t.bf - 1) / t.bf);
  return n > 256 ? 1 : 256 / n > kMaxParts ? kMaxParts : (int)(256 / n);
}

// The tile shape with the least predicted time, if that is below the wave-level kernel's `other_us`; else -1.
inline int pick_bgemm(const WParams& p, double other_us, long long room, int* parts) {
  const int mode = p.xkv ? 3 : p.geglu ? 0 : p.nseg ? 1 : 2;
  const int MT = (p.M + 31) / 32, NF = p.N / 32;
  const double kt = p.K / 64.0;
  double best = other_us;
  int pick = -1;
  auto consider = [&](int c) {
    const TileCfg& t = kTiles[c];
    if ((p.K / 16) % t.kf) return;
    const int bfo = p.geglu ? t.bf / 2 : t.bf;
    const long long n = (long long)((MT + t.bt - 1) / t.bt) * ((NF + bfo - 1) / bfo);
    // rounds of workgroups; two workgroups of a unit share it, so their rounds are continuous beyond the first few
    double r = (double)((n + 255) / 256);
    if (t.occ == 2) {
      const long long rem = n % 512;
      r = n > 1536 ? n / 512.0 : (double)(n / 512) + (rem == 0 ? 0.0 : rem <= 256 ? t.alone : 1.0);
    }
    const double slab = c == 5 && mode == 2 && !p.ln_s ? t.slab + kPlain64 : t.slab;
    const double epi = c == 3 && mode == 3 && (p.xa_keys + 31) / 32 != 3 ? kXaEpi64x128 : t.epi[mode];
    const double us = t.base + r * (kt * slab + epi);
    if (us < best) { best = us; pick = c; *parts = 1; }
  };
  *parts = 1;
  for (int c = 0; c < kSplitFamily; ++c) consider(c);
  // Inputs written by the kernel before, weights cold: 494 x 1280 x 5120 21.9 us in five parts, 24.4 on the wave-level kernel; 224 15.7 in
  // eight against 18.1; 1024 32.1 in three against 33.4 on the best tile.  The error against 64 bits is that of the whole layer (494:
  // 1.19e-7 against 1.29e-7 relative).  At 640 features and K = 2560 and below the sums cost what the parts gain.
  if (mode == 2 && !p.ln_s && room > 1) {
    for (const SplitCfg& q : kSplits) {
      const TileCfg& t = kTiles[q.tile];
      const int most = max_parts(t, MT, NF);
      const long long tiles = (long long)((MT + t.bt - 1) / t.bt) * ((NF + t.bf - 1) / t.bf);
      for (int s = 2; s <= most && s <= room; ++s) {
        if (kt / s < 8) break;
        const double us = t.base + std::ceil(kt / s) * t.slab + q.fixed + kPartUs * (s + 1) * (32.0 * MT) * p.N + (tiles * s > kCrowd ? kCrowdUs : 0.0);
        if (us < best) { best = us; pick = q.tile; *parts = s; }
      }
    }
  }
  for (int c = kSplitFamily; c < (int)(sizeof(kTiles) / sizeof(kTiles[0])); ++c) consider(c);
  return pick;
}

// The wave-level kernel's form.  Measured with cold weights.  Up to 128 wave tiles of 32 tokens x 64 features the 32 x 32 tile (`few`)
// puts twice the workgroups on the chip: such a layer waits for its weights, which a compute unit pulls from HBM at no more than 25
// bytes per cycle (64 x 1280 x 5120 18.4 -> 13.1 us, 150 x 1280 x 1280 6.4 -> 5.2; at 140 tiles it loses).  Up to ~320
// the 32 x 64 tile keeps the most waves in flight; from there on the 64 x 64 tile's lower operand traffic per flop wins;
// and where a still larger tile (`wide`, 64 x 96 without GEGLU) covers the output with at most one workgroup per unit, its single
// round of workgroups wins again, provided the reduction is long enough to amortise the row-by-row epilogue.
struct WaveForm { long long tiles; bool few, wide; };
inline WaveForm wave_form(const WParams& p) {
  const int MT = (p.M + 31) / 32, nfrag = p.N / 32;
  const long long tiles = (long long)MT * (p.geglu ? nfrag : nfrag / 2);
  const bool wide = tiles >= 320 && p.K / 16 / 4 >= 16 && !p.geglu && nfrag % 3 == 0 && (long long)((MT + 1) / 2) * (nfrag / 3) <= 256 && !p.xkv;
  return {tiles, tiles <= 128, wide};
}

inline bool is_plain(const WParams& p) { return !p.ln_s && !p.geglu && !p.nseg && !p.xkv; }

// The tile shape, and the parts of K (at most `room`, which the caller's scratch holds), or -1 for the wave-level kernel: that keeps the
// problems whose token count does not fill the tiles.  Its predicted time is fitted like theirs (microseconds: launch + rounds of
// workgroups x (K loop + epilogue)).
inline int choose_tile(const WParams& p, const WaveForm& f, long long room, int* parts) {
  *parts = 1;
  if (f.few) return -1;
  const int MT = (p.M + 31) / 32, nfrag = p.N / 32;
  const double kt = p.K / 64.0;
  const bool two = f.tiles >= 320 && !p.xkv;
  const double n = f.wide ? 0.0 : two ? (double)((MT + 1) / 2) * (p.geglu ? nfrag : nfrag / 2) : (double)f.tiles;
  double us;
  if (is_plain(p)) {
    // Rounds of 256 workgroups, one per unit, whatever part of the units the last one covers: 1280 x 5120 14.6 - 15.2 us with 224 to 384
    // tokens, 19 - 20 with 494 to 768.  Every XCD reads all tokens, hence the term in M x K: inputs that the kernel before has just written
    // instead of ones read before take 1.5 us more at 1024 x 640 x 640 and 3 at 768 x 1280 x 5120.  Fitted to 41 layers (320 to 10240
    // features, K of 64 to 10240) of 130 to 7200 tokens, weights that no cache holds.  What this chooses takes 0.7 % more than the best of all
    // tiles and parts with inputs just written, 1.2 % with inputs read again and again, 1.5 % with K below 640.  Constants from 1280 x 5120
    // alone took 1.9, 1.7 and 2.0, and up to 18 % more than another tile (1500 x 640 x 2560 11.7 -> 13.8 us, 2400 x 320 x 1280 7.5 -> 8.4).
    const double q = n / 256.0;
    const double r = q <= 1.0 ? 0.65 : q > 2.0 ? 1.3 * q : two ? 1.2 + 0.5 * (q - 1.0) : 1.0 + 1.35 * (q - 1.0);
    us = (f.wide ? 6.2 + 0.21 * kt : two ? 4.95 + r * (0.26 * kt + 0.8) : 3.46 + r * (0.201 * kt + 0.34)) + 0.5e-6 * (32.0 * MT) * p.K;
  } else {
    const double r = n / 256.0 > 0.6 ? n / 256.0 : 0.6;
    us = f.wide ? 9.7 + 0.125 * kt
         : two ? 4.95 + r * (0.261 * kt + (p.geglu ? 0.34 : p.nseg ? 0.7 : 0.23))
         : p.xkv ? 5.3 + r * (0.165 * kt + 0.1)
                 : 3.46 + r * (0.201 * kt + (p.geglu ? 2.1 : p.nseg ? 2.2 : 0.49));
  }
  // (in the step the wave-level kernel keeps its time where the tiles lose a few per cent to what runs before them)
  return pick_bgemm(p, 0.98 * us, room, parts);
}

}  // namespace df
