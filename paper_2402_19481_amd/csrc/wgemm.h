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
  int res_frag, f32_frag;
  bf16_t* out_packed;
  bf16_t* out_rows;
  long long ld_rows;
  int geglu;
  int nseg, seg_w;
  bf16_t* seg_out[3];
  long long seg_ld[3], seg_rows_out[3], seg_row0[3];
  int seg_rows_in[3];
  int seg_tr[3];        // 0: rows; 1: transposed; 2: transposed, token pairs stay together and 4-byte aligned
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
  int mgroups, kfw;     // wgemm: groups of token rows, k-fragments of a wave, and the reciprocals of both
  unsigned int mg_recip, kfw_recip;
  int group_m;          // bgemm: token tiles of a panel in the tile order (see there)
};

// Arguments of the segment that a fragment of 32 features lies in (seg_w % 32 == 0).  `n0`, its first feature, is the same for the
// whole wave and the three are chosen by scalar selects: indexed by a lane's feature number the arguments came by four dependent
// vector loads per unit, most of the 3.5 us that the epilogue of a 128 x 128 query / key / value tile took.
struct WSegment {
  bf16_t* out;
  long long ld, rows_out, row0;
  int rows_in, tr, pin, pout, first;   // first: feature 0 of the segment
  float scale;
};
__device__ __forceinline__ WSegment wg_segment(const WParams& p, int n0) {
  const bool s1 = n0 >= p.seg_w, s2 = n0 >= 2 * p.seg_w;
  auto pick = [&](const auto& v) { return s2 ? v[2] : s1 ? v[1] : v[0]; };
  return {pick(p.seg_out), pick(p.seg_ld),  pick(p.seg_rows_out), pick(p.seg_row0), pick(p.seg_rows_in),
          pick(p.seg_tr),  pick(p.seg_pin), pick(p.seg_pout),     s2 ? 2 * p.seg_w : s1 ? p.seg_w : 0,
          s1 ? 1.0f : p.seg0_scale};
}

// What the epilogues need of the arguments is requested while the first operands are on their way: fetched where it is first used, a
// batch of them costs that epilogue a round trip to memory (they are cold in every launch).  The outputs stay in registers from here on
// (left alone, the compiler fetches them again); the segments' are too many for that and come from the scalar cache later.
struct WOut {
  float* f32;
  bf16_t *packed, *rows;
  long long ldo, ld_rows;
  int f32_frag;
};
template <typename T>
__device__ __forceinline__ T wg_pin(T v) {
  asm volatile("" : "+s"(v));
  return v;
}
template <bool SEG>
__device__ __forceinline__ WOut wg_outputs(const WParams& p) {
  WOut o = {};
  if constexpr (SEG) {
    asm volatile("" ::"s"(p.seg_w), "s"(p.seg_out[0]), "s"(p.seg_out[1]), "s"(p.seg_out[2]), "s"(p.seg_ld[0]), "s"(p.seg_ld[1]), "s"(p.seg_ld[2]),
                 "s"(p.seg_rows_out[0]), "s"(p.seg_rows_out[1]), "s"(p.seg_rows_out[2]));
    asm volatile("" ::"s"(p.seg_row0[0]), "s"(p.seg_row0[1]), "s"(p.seg_row0[2]), "s"(p.seg_rows_in[0]), "s"(p.seg_rows_in[1]), "s"(p.seg_rows_in[2]),
                 "s"(p.seg_tr[0]), "s"(p.seg_tr[1]), "s"(p.seg_tr[2]), "s"(p.seg_pin[0]), "s"(p.seg_pin[1]), "s"(p.seg_pin[2]),
                 "s"(p.seg_pout[0]), "s"(p.seg_pout[1]), "s"(p.seg_pout[2]), "s"(p.seg0_scale));
  } else {
    o.f32 = wg_pin(p.out_f32); o.ldo = wg_pin(p.ldo); o.f32_frag = wg_pin(p.f32_frag);
    o.packed = wg_pin(p.out_packed); o.rows = wg_pin(p.out_rows); o.ld_rows = wg_pin(p.ld_rows);
  }
  return o;
}

// Eight consecutive floats of a unit (see wg_store_unit) of the residual or the float output: the first four, and how far on the others
// are.  Row-major, or in fragments [token row][feature row][4][64 lanes] of four, quarter 2 f + h of a fragment holding
// features 16 f + 8 (lane / 32) + 4 h .. of token lane % 32: the accumulators' own order, a kilobyte per access where a row-major one
// touches a line for every lane (the address unit takes one a cycle: 64 cycles against 16).
template <typename T>
__device__ __forceinline__ T* wg_float_unit(T* base, int frag, long long ld, int N, int mt, int m, int n0, int fo, int lane, int* next) {
  *next = frag ? 256 : 4;
  return frag ? base + (((size_t)mt * (N >> 5) + (n0 >> 5)) * 4 + 2 * (fo >> 4)) * 256 + lane * 4 : base + (long long)m * ld + n0 + fo;
}

// One output unit: features n0 + fo .. + 7 of token m, written in every requested form.  n0 is uniform, the first of a fragment; `lane`
// is the lane of that token and feature group in the packed layout (m % 32 + 32 (fo / 8 % 2)); lane ^ 1 of the wave holds token m ^ 1.
template <bool SEG>
__device__ __forceinline__ void wg_store_unit(const WParams& p, const WOut& o, int mt, int m, int n0, int fo, int lane, const float* v) {
  const bool row_ok = m < p.M;
  const int n = n0 + fo;
  if constexpr (SEG) {
    const WSegment s = wg_segment(p, n0);
    const int mp = s.tr > 1 ? m & ~1 : m;
    const int bi = mp < s.rows_in ? 0 : mp / s.rows_in;   // (usually one batch item: a comparison instead of a division)
    const long long pos = s.row0 + seg_pos(mp - bi * s.rows_in, s.pin, s.pout);
    if (s.tr > 1) {
      // feature-major, token pairs stay together and aligned (launcher): neighbouring lanes exchange, the even one keeps feature 2q of
      // both tokens and the odd one 2q + 1; a store covers the 32 tokens of four features
      bf16_t* d = s.out + ((long long)bi * p.seg_w + (n - s.first) + (m & 1)) * s.ld + pos;
      const unsigned int sel = m & 1 ? 0x07060302u : 0x01000504u;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const unsigned int u = pack_bf2(v[2 * q], v[2 * q + 1]);
        const unsigned int w = (unsigned int)__builtin_amdgcn_update_dpp(0, (int)u, 0xb1, 0xf, 0xf, true);   // lane ^ 1
        const unsigned int x = __builtin_amdgcn_perm(u, w, sel);
        if (row_ok) *reinterpret_cast<unsigned int*>(d + 2 * q * s.ld) = x;
      }
    } else if (s.tr) {
      bf16_t* d = s.out + ((long long)bi * p.seg_w + (n - s.first)) * s.ld + pos;
      if (row_ok) {
#pragma unroll
        for (int q = 0; q < 8; ++q) d[q * s.ld] = f2bf(v[q]);
      }
    } else if (row_ok) {
      const float w[8] = {v[0] * s.scale, v[1] * s.scale, v[2] * s.scale, v[3] * s.scale,
                          v[4] * s.scale, v[5] * s.scale, v[6] * s.scale, v[7] * s.scale};
      st_vec(s.out + ((long long)bi * s.rows_out + pos) * s.ld + (n - s.first), w);
    }
    return;
  }
  if (o.f32 && (row_ok || o.f32_frag)) {
    int next;
    float* d = wg_float_unit(o.f32, o.f32_frag, o.ldo, p.N, mt, m, n0, fo, lane, &next);
    st_vec(d, v);
    st_vec(d + next, v + 4);
  }
  if (o.packed) {
    // fragment (mt, n/16) of the [M, N] result as the next layer's activation operand; padded token rows are
    // written too (they only ever feed padded rows)
    const int KFo = p.N >> 4;
    st_vec(o.packed + (((size_t)mt * KFo + (n >> 4)) * 64 + lane) * 8, v);
  }
  if (o.rows && row_ok) st_vec(o.rows + (long long)m * o.ld_rows + n, v);
}

// Workgroup-tile kernel (bgemm.hip), tile shape `cfg` of kTiles (wchoice.h).
int launch_bgemm(const WParams& p, int cfg, hipStream_t st);
int launch_part_sums(const WParams& p, hipStream_t st);

// A segmented layer folds a LayerNorm and writes its segments: nothing is added to them and no other output comes with them.
inline bool segments_alone(const WGemmArgs& a) {
  return a.nseg <= 0 || (a.ln_s && !a.residual && !a.out_f32 && !a.out_packed && !a.out_rows && !a.geglu && !a.xa_kv);
}

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
