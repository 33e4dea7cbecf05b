// Shared by the two kernels for linear layers on fragment-packed operands (wgemm.hip: wave-level, few tokens;
// bgemm.hip: workgroup tiles through LDS, many tokens): the kernel arguments and the store of one output unit.
#pragma once
#include "kernels.h"

namespace df {

struct WParams {
  const bf16x8* Xp;
  const bf16x8* Wp;
  int M, N, K;          // N: rows of W that produce outputs (geglu: F value rows; the gate rows follow at row F)
  const float* bias;
  const float* ln_s;
  const float* ln_t;
  float ln_eps;
  const float* residual;
  long long ldr;
  float* out_f32;
  long long ldo;
  bf16_t* out_packed;
  bf16_t* out_rows;
  long long ld_rows;
  int geglu;
  int nseg, seg_w;
  bf16_t* seg_out[3];
  long long seg_ld[3], seg_rows_out[3], seg_row0[3];
  int seg_rows_in[3];
  int seg_tr[3];
  int seg_pin[3], seg_pout[3];
  float seg0_scale;     // factor of segment 0 (the attention queries), 1 without one; segment 0 is never transposed
  // fused cross-attention (XA > 0): per (batch item, head) 8*XA key fragments then 4*XA value fragments
  const bf16x8* xkv;
  int xa_keys;          // valid text tokens
  long long xa_bstride; // fragments between batch items
  int xa_rows;          // token rows per batch item
  float xa_scale;
  f32x4* partials;      // bgemm with `parts` > 1 parts of K: their sums
  int parts;
  int group_m;          // bgemm: token tiles of a panel in the tile order (see there)
};

// One output unit: 8 consecutive features n .. n+7 of token m = mt*32 + lane%32, written in every requested form.
__device__ __forceinline__ void wg_store_unit(const WParams& p, int mt, int m, int n, int lane, const float* v) {
  const bool row_ok = m < p.M;
  if (p.out_f32 && row_ok) {
    st_vec(p.out_f32 + (long long)m * p.ldo + n, v);
    st_vec(p.out_f32 + (long long)m * p.ldo + n + 4, v + 4);
  }
  if (p.out_packed) {
    // fragment (mt, n/16) of the [M, N] result as the next layer's activation operand; padded token rows are
    // written too (they only ever feed padded rows)
    const int KFo = p.N >> 4;
    st_vec(p.out_packed + (((size_t)mt * KFo + (n >> 4)) * 64 + lane) * 8, v);
  }
  if (row_ok) {
    if (p.nseg > 0) {
      // 8 features never straddle a segment (seg_w % 32 == 0); at most three segments, usually one batch item:
      // comparisons instead of integer divisions
      const int sg = (n >= p.seg_w ? 1 : 0) + (n >= 2 * p.seg_w ? 1 : 0);
      const int bi = m < p.seg_rows_in[sg] ? 0 : m / p.seg_rows_in[sg];
      if (p.seg_tr[sg]) {
        // feature-major output: the 32 tokens of a half wave are consecutive in memory for each feature
        bf16_t* o = p.seg_out[sg] + ((long long)bi * p.seg_w + (n - sg * p.seg_w)) * p.seg_ld[sg] + p.seg_row0[sg] +
                    seg_pos(m - bi * p.seg_rows_in[sg], p.seg_pin[sg], p.seg_pout[sg]);
#pragma unroll
        for (int q = 0; q < 8; ++q) o[q * p.seg_ld[sg]] = f2bf(v[q]);
      } else {
        const long long orow = (long long)bi * p.seg_rows_out[sg] + p.seg_row0[sg] +
                               seg_pos(m - bi * p.seg_rows_in[sg], p.seg_pin[sg], p.seg_pout[sg]);
        const float sc = sg == 0 ? p.seg0_scale : 1.0f;
        const float w[8] = {v[0] * sc, v[1] * sc, v[2] * sc, v[3] * sc, v[4] * sc, v[5] * sc, v[6] * sc, v[7] * sc};
        st_vec(p.seg_out[sg] + orow * p.seg_ld[sg] + (n - sg * p.seg_w), w);
      }
    } else if (p.out_rows) {
      st_vec(p.out_rows + (long long)m * p.ld_rows + n, v);
    }
  }
}

// Workgroup-tile kernel (bgemm.hip), tile shape `cfg` of its table.
int launch_bgemm(const WParams& p, int cfg, hipStream_t st);
// Tile shape predicted to be faster than the wave-level kernel's `other_us`, or -1, and the parts to split K into: at most `room`,
// which the caller's scratch holds.
int pick_bgemm(const WParams& p, double other_us, long long room, int* parts);
int launch_part_sums(const WParams& p, hipStream_t st);

// Parts of K that the scratch handed to a plain layer (MT token rows of 32, NF feature rows of 32, K) has to hold; 1: any scratch
// will do.  This decides which calls return DF_ENOMEM and nothing else.  It is the choice of parts as it was when that became
// part of the entry point, with the predicted times of then (a launch, a round of workgroups per 64 of K, its prologue and
// epilogue, the round of a workgroup alone on a unit), so that a later fit of the tiles does not move the set of calls that
// are refused.  Layers that it leaves out split as far as their scratch allows.
inline int parts_due(int MT, int NF, int K) {
  struct Tile { int bt, bf, occ; double base, slab, epi, alone; };
  constexpr Tile tiles[] = {{8, 10, 1, 0.00, 1.603, 26.3, 1.0}, {4, 4, 2, 3.77, 1.078, 4.2, 0.70}, {4, 4, 1, 1.80, 0.474, 6.0, 1.0},
                            {2, 4, 2, 3.90, 0.620, 2.9, 0.62},  {2, 2, 2, 2.30, 0.432, 1.7, 0.86}, {2, 2, 1, 2.50, 0.227, 1.9, 1.0},
                            {4, 10, 1, 1.43, 0.947, 13.8, 1.0}};
  const double kt = K / 64.0;
  const long long wave_tiles = (long long)MT * (NF / 2), pairs = (MT + 1) / 2;
  if (wave_tiles <= 128) return 1;
  const bool two = wave_tiles >= 320, wide = two && K >= 1024 && NF % 3 == 0 && pairs * (NF / 3) <= 256;
  const double waves = (two ? (double)(pairs * (NF / 2)) : (double)wave_tiles) / 256.0, rw = waves > 0.6 ? waves : 0.6;
  double best = 0.94 * (wide ? 9.7 + 0.125 * kt : two ? 4.6 + rw * (0.286 * kt + 1.16) : 5.3 + rw * (0.189 * kt - 2.2));
  for (int c = 0; c < 7; ++c) {
    const Tile& t = tiles[c];
    if ((c == 4 || c == 5) && K / 64 % 2) continue;
    const long long n = (long long)((MT + t.bt - 1) / t.bt) * ((NF + t.bf - 1) / t.bf), rem = n % 512;
    const double r = t.occ == 1 ? (double)((n + 255) / 256)
                     : n > 1536 ? n / 512.0 : (double)(n / 512) + (rem == 0 ? 0.0 : rem <= 256 ? t.alone : 1.0);
    const double us = t.base + r * (kt * t.slab + t.epi);
    if (us < best) best = us;
  }
  int parts = 1;
  for (int c = 2; c <= 6; c += 4) {
    const Tile& t = tiles[c];
    const long long n = (long long)((MT + t.bt - 1) / t.bt) * ((NF + t.bf - 1) / t.bf);
    for (int s = 2; s <= 8 && n * s <= 256 && kt / s >= 8; ++s) {
      const double us = t.base + (K / 64 + s - 1) / s * t.slab + (c == 2 ? 4.3 : 5.0) + 2.2e-6 * s * (32.0 * MT) * (32.0 * NF);
      if (us < 0.97 * best) { best = us / 0.97; parts = s; }
    }
  }
  return parts;
}

}  // namespace df
