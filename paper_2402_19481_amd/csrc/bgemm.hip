#include <cmath>
#include <type_traits>

#include "wchoice.h"

namespace df {

namespace {

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_b;

template <int VM>
__device__ __forceinline__ void wait_vm_lds() {   // s_waitcnt vmcnt(VM) lgkmcnt(0)
  __builtin_amdgcn_s_waitcnt((VM & 0xF) | ((VM >> 4) << 14) | (0x7 << 4));
}
enum { EPI_PLAIN = 0, EPI_GEGLU = 1, EPI_QKV = 2, EPI_XA = 3, EPI_PART = 4 };

// Geometry of a tile's epilogue: the accumulators go through LDS in passes of R token fragment rows of the tile (row
// i * WT + wt of the order is row i of the waves at wt).
template <int WT, int WF, int TT, int TF, int KG, int OCC, bool LN>
struct Epi {
  static constexpr int BT = WT * TT, BF = WF * TF;
  static constexpr int kStats = LN ? (KG * WF + 1) * BT * 32 * 2 * 4 : 0;
  static constexpr int kVecs = (LN ? 2 : 1) * BF * 32 * 4;
  static constexpr int kCap = 160 * 1024 / OCC - kStats - kVecs;
  static constexpr int pass_bytes(int r) { return KG * r * BF * 4096; }
  static constexpr int pick() {
    for (int r = BT; r > 1; --r)
      if (BT % r == 0 && (r % WT == 0 || WT % r == 0) && pass_bytes(r) <= kCap) return r;
    return 1;
  }
  static constexpr int R = pick();
  static constexpr int kBytes = pass_bytes(R) + kStats + kVecs;
};

// Cross-attention of one head and 32 tokens (row mt) in one wave: S^T = K Q^T against XA 32-key tiles of packed text keys (lane = token),
// softmax over the valid keys, O^T = V^T P^T, packed output.  LATE: the values are requested here, behind the scores (they and the keys do
// not fit the registers of a unit's second workgroup).
template <int XA, bool LATE>
__device__ __forceinline__ void xa_head(const WParams& p, int mt, int head, int g, int lane, const bf16x8 (&qf)[4],
                                        const bf16x8 (&kf)[XA][4], const bf16x8 (*vpre)[2], const bf16x8* kv) {
  f32x16 sa[XA];
#pragma unroll
  for (int kt = 0; kt < XA; ++kt) {
#pragma unroll
    for (int e = 0; e < 16; ++e) sa[kt][e] = 0.f;
#pragma unroll
    for (int ds = 0; ds < 4; ++ds) sa[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kt][ds], qf[ds], sa[kt], 0, 0, 0);
  }
  bf16x8 vf[2 * XA][2];
#pragma unroll
  for (int ks = 0; ks < 2 * XA; ++ks)
#pragma unroll
    for (int dt = 0; dt < 2; ++dt) vf[ks][dt] = LATE ? kv[(size_t)(4 * XA + dt * 2 * XA + ks) * 64] : vpre[ks][dt];
  const float sc = p.xa_scale * 1.4426950408889634f;
  float mx = -INFINITY;
#pragma unroll
  for (int kt = 0; kt < XA; ++kt)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int key = kt * 32 + 16 * (e >> 3) + 8 * g + (e & 7);
      if (key >= p.xa_keys) sa[kt][e] = -INFINITY;
      mx = fmaxf(mx, sa[kt][e]);
    }
  mx = fmaxf(mx, __shfl_xor(mx, 32, 64)) * sc;
  float l = 0.f;
#pragma unroll
  for (int kt = 0; kt < XA; ++kt)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const float pv = __builtin_amdgcn_exp2f(fmaf(sa[kt][e], sc, -mx));
      sa[kt][e] = pv;
      l += pv;
    }
  l += __shfl_xor(l, 32, 64);
  f32x16 oa[2];
#pragma unroll
  for (int dt = 0; dt < 2; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) oa[dt][e] = 0.f;
#pragma unroll
  for (int ks = 0; ks < 2 * XA; ++ks) {
    const int kt = ks >> 1, hf = ks & 1;
    const u32x4 pk = {pack_bf2(sa[kt][8 * hf + 0], sa[kt][8 * hf + 1]), pack_bf2(sa[kt][8 * hf + 2], sa[kt][8 * hf + 3]),
                      pack_bf2(sa[kt][8 * hf + 4], sa[kt][8 * hf + 5]), pack_bf2(sa[kt][8 * hf + 6], sa[kt][8 * hf + 7])};
    const bf16x8 pf = __builtin_bit_cast(bf16x8, pk);
#pragma unroll
    for (int dt = 0; dt < 2; ++dt) oa[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[ks][dt], pf, oa[dt], 0, 0, 0);
  }
  const float inv = __builtin_amdgcn_rcpf(l);
  const int KFo = p.N >> 4;
#pragma unroll
  for (int dt = 0; dt < 2; ++dt)
#pragma unroll
    for (int f2 = 0; f2 < 2; ++f2) {
      float o8[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) o8[q] = oa[dt][8 * f2 + q] * inv;
      st_vec(p.out_packed + (((size_t)mt * KFo + head * 4 + dt * 2 + f2) * 64 + lane) * 8, o8);
    }
}

// LDS of the epilogue of one k-group, which leaves the accumulators where they are: the waves' partial row sums, the
// per-feature vectors, and (GEGLU on an odd number of fragments per wave) the halves that two waves exchange.
template <int WT, int WF, int TT, int TF, bool LN, bool GEGLU>
struct Direct {
  static constexpr int BT = WT * TT, BF = WF * TF;
  static constexpr int kXch = GEGLU && TF % 2 ? BT * 4096 : 0;
  static constexpr int kStats = LN ? WF * BT * 32 * 2 * 4 : 0;
  static constexpr int kVecs = (LN ? 2 : 1) * BF * 32 * 4;
  static constexpr int kBytes = kXch + kStats + kVecs;
};

// Linear layer on fragment-packed operands, a workgroup per output tile: BT x 32 tokens by BF x 32 features, the waves WT x WF
// over it and KG over the k-steps of a stage.  The operands' 1 KB fragments go from memory to an LDS ring of ST stages by direct
// loads, and from there to the waves without conflicts, since a fragment is in lane order.
// What bounds it: a compute unit receives 25 - 33 bytes per cycle by direct loads (128 x 320 tile, K = 1280: 1750 cycles
// per 64 of K by the loads alone, 1530 by the matrix instructions and LDS reads alone, 2230 together), so a tile is as fast
// as its operand bytes per flop and the number of compute units that have one; then the epilogue (with GEGLU a sixth of the time at
// K = 1280), which in the smaller tiles runs beside the other workgroup of the unit.  Hence a set of tiles, from 64 x 64 to
// 256 x 320 with 320 a divisor of most layers' widths, and the choice by predicted time (wchoice.h).  With the stages requested
// in parts between the matrix instructions and the 320-wide tiles, 1024 x 10240 x 1280 with GEGLU 46.6 -> 36.3 us, 1800
// x 10240 x 1280 68 -> 62, 4096 x 5120 x 640 43.5 -> 39.9, 14400 x 640 x 2560 with residual 78 -> 61.  Four waves of 64 x
// 160 instead of eight of 32 x 160: 40 us (one wave per SIMD issues the epilogue half as fast).  With loads that leave the waits
// for LDS reads exact (lds_load_buf): 1800 x 1280 x 5120 48.9 -> 41.4 us, 1800 x 3840 x 1280 30.4 -> 27.5, 4096 x 1280 x 1280 27.2
// -> 24.7.  With the epilogue of a single k-group in the accumulators and its arguments requested early: 1024 x 10240 x 1280 with GEGLU
// 35.4 -> 31.4 us, 1800 x 10240 x 1280 61 -> 53, 1024 x 3840 x 1280 split into queries, keys and values 20 -> 17.5.
// As in wgemm.hip the leading arguments come in scalar registers: operands, the per-feature vectors, the residual, sizes, and in `order` the token
// tiles of a panel, the parts of K (from bit 26) and whether the residual is in fragments (bit 30).  With attn_wave_d64's the same way, step of
// 1024 x 1024 with guidance 6467 -> 6351 us, 1280 x 1920 7140 -> 7070, 832 x 1216 8717 -> 8667, 1024 x 1024 full 11870 -> 11778.
template <int WT, int WF, int TT, int TF, int KG, int KS, int ST, int OCC, int EPI, bool LN, int XA>
__global__ __launch_bounds__(64 * WT * WF * KG, (WT * WF * KG * OCC + 3) / 4) void bgemm_kernel(const bf16x8* Xp, const bf16x8* Wp, const float* vec_s,
                                                                                              const float* vec_t, const float* residual, int M, int N, int K,
                                                                                              unsigned int order, WParams p) {
  using E = Epi<WT, WF, TT, TF, KG, OCC, LN>;
  constexpr int NW = WT * WF * KG;                     // waves
  constexpr int BT = WT * TT, BF = WF * TF;            // token / feature fragment rows of the workgroup tile
  constexpr int BKF = KS * KG;                         // k-fragments per stage
  constexpr int STAGE = (BT + BF) * BKF * 1024;
  constexpr int I = (BT + BF) * BKF;                   // 1 KB direct loads per stage
  constexpr int NL = (I + NW - 1) / NW;                // per wave (the last wave repeats the last fragment)
  static_assert(NL * (ST - 1) < 64, "vmcnt field is 6 bits");
  static_assert((WF & (WF - 1)) == 0, "");
  static_assert(EPI != EPI_QKV || LN, "the segmented epilogue applies the folded LayerNorm");
  extern __shared__ __attribute__((aligned(16))) char smem[];

  const int group_m = (int)(order & 0x3ffffff), parts = (int)(order >> 26 & 15);
  const bool res_frag = order >> 30;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tok = lane & 31, g = lane >> 5;
  const int kg = wave / (WT * WF), wq = wave % (WT * WF), wt = wq % WT, wf = wq / WT;
  const int MT = (M + 31) >> 5, NF = N >> 5;
  constexpr int BFO = EPI == EPI_GEGLU ? BF / 2 : BF;  // output fragments of the tile along the features
  const int MG = (MT + BT - 1) / BT, NG = (NF + BFO - 1) / BFO, nwg = MG * NG;
  int t = blockIdx.x;
  {
    const int xcd = t & 7, loc = t >> 3;
    const int base = nwg >> 3, rem = nwg & 7;
    t = xcd * base + (xcd < rem ? xcd : rem) + loc;
  }
  int mg, ng;
  {
    const int per = group_m * NG, pn = t / per, r = t - pn * per, m0 = pn * group_m;
    const int gh = MG - m0 < group_m ? MG - m0 : group_m;
    ng = r / gh;
    mg = m0 + r - ng * gh;
  }
  const int KF = K >> 4;
  int KT = KF / BKF, kt0 = 0;                          // stages of this workgroup, the first of them
  if constexpr (EPI == EPI_PART) {
    kt0 = (int)((long long)KT * blockIdx.y / parts);
    KT = (int)((long long)KT * (blockIdx.y + 1) / parts) - kt0;
  }

  // fragment row of the weights behind row r (0 .. BF-1) of the tile.  GEGLU, several k-groups: the first half are value rows, the
  // second half their gates.  GEGLU, one k-group: a wave holds pairs, values in front; an odd fragment in the middle is
  // the value (first wave) or the gate (second) of a pair that the two waves share.
  constexpr int HP = TF / 2;                           // pairs of a wave
  auto wrow = [&](int r) {
    int nt;
    if constexpr (EPI == EPI_GEGLU) {
      bool gate;
      if constexpr (KG == 1) {
        static_assert(TF % 2 == 0 || WF == 2, "two waves share the odd pair");
        const int w = r / TF, j = r - w * TF;
        gate = TF % 2 && j == HP ? w == 1 : j >= TF - HP;
        nt = ng * BFO + (TF % 2 && j == HP ? HP : w * (TF - HP) + (gate ? j - (TF - HP) : j));
      } else {
        gate = r >= BFO;
        nt = ng * BFO + (gate ? r - BFO : r);
      }
      if (nt > NF - 1) nt = NF - 1;
      return gate ? NF + nt : nt;
    }
    nt = ng * BF + r;
    return nt < NF ? nt : NF - 1;
  };
  const int lo = lane * 16;
  const char* src[NL];
#pragma unroll
  for (int q = 0; q < NL; ++q) {
    int i = wave * NL + q;
    if (i > I - 1) i = I - 1;
    const int row = i / BKF, kk = i - row * BKF;
    int mt = mg * BT + row;
    if (mt > MT - 1) mt = MT - 1;                      // ragged last tile: re-read, never stored
    src[q] = (row < BT ? (const char*)Xp + (size_t)mt * KF * 1024 : (const char*)Wp + (size_t)wrow(row - BT) * KF * 1024) +
             ((size_t)kt0 * BKF + kk) * 1024;
  }
  // Plain layers of whole 1024s of tokens, up to 31 of them missing: the XCDs walk K from different stages on, an eighth apart.  Their shares of
  // the tokens begin whole tiles apart there, and in step the eight ask the same channels of the last-level cache.  In step / apart, weights from
  // HBM: 1280 x 5120 1000 tokens 28.5 / 24.1 us, 1024 28.6 / 24.1, 2048 42.2 / 35.8, 3072 49.2 / 44.5, 4096 58.9 / 56.3, 5120 82.9 / 78.4; 640 x 2560
  // 3072 20.4 / 19.2, 4096 23.8 / 21.8, 5120 25.9 / 23.6; with a K of 640 or 1280 the same within 1 % (8192 x 640 x 640 3 % faster); 1024 x 1024 full
  // step 12.96 / 12.78 ms, 2048 x 2048 strips 15.54 / 15.36.  Multiples of 256 alone would gain with 5120 too (1536 35.8 / 32.8, 2304 44.1 / 39.0)
  // and keep their order; other counts lose (1800 35.6 / 36.1, 4000 55.3 / 56.1, 7200 91.7 / 93.4), the layers that fold a LayerNorm 0 - 3 %.
  // Within an XCD the workgroups stay in step, so that what one has fetched the others find in its L2 (an offset per tile: steps 2 - 5 % slower).
  const int rot = EPI == EPI_PLAIN && !LN && MT % 32 == 0 ? (int)((blockIdx.x & 7) * (unsigned int)KT >> 3) : 0;
  // loads of a stage: all (STEP < 0), or part STEP of KS
  auto issue = [&](int kt, int slot, auto stepc) {
    constexpr int STEP = decltype(stepc)::value;
    const int kr = EPI == EPI_PLAIN && !LN ? kt + rot : kt;
    const unsigned int ko = (unsigned int)(kr < KT ? kr : kr - KT) * (BKF * 1024);
#pragma unroll
    for (int q = 0; q < NL; ++q) {
      if (STEP >= 0 && q * KS / NL != STEP) continue;
      int i = wave * NL + q;
      if (i > I - 1) i = I - 1;
      lds_load_buf(src[q], lo, ko, smem + slot * STAGE + i * 1024);
    }
  };

  // per-feature vectors of the tile (norm scale / shift, or bias): requested now, parked in LDS for the epilogue
  constexpr int NV = (BF * 32 + 64 * NW - 1) / (64 * NW);
  float vs[NV], vt[NV];
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    const int r = tid + q * 64 * NW;
    vs[q] = vt[q] = 0.f;
    if (r < BF * 32) {
      const int n = wrow(r >> 5) * 32 + (r & 31);
      if constexpr (LN) { vs[q] = vec_s[n]; vt[q] = vec_t[n]; }
      else if (EPI != EPI_PART && vec_t) vt[q] = vec_t[n];
    }
  }
  f32x16 acc[TT][TF];
  constexpr bool kResInit = EPI == EPI_PLAIN && !LN;
  if (kResInit && residual && kg == 0) {
    // the residual is the accumulators' start value: its latency runs beside the first stages'
    long long ldr = 0;                                 // (not among the arguments that come in registers)
    if (!res_frag) { asm volatile(""); ldr = p.ldr; }
#pragma unroll
    for (int i = 0; i < TT; ++i) {
      const int m = (mg * BT + wt * TT + i) * 32 + tok;
#pragma unroll
      for (int j = 0; j < TF; ++j) {
        const int nt = ng * BF + wf * TF + j;
        f32x4 r[4];
#pragma unroll
        for (int f = 0; f < 4; ++f) r[f] = f32x4{0.f, 0.f, 0.f, 0.f};
        if ((res_frag ? m < MT * 32 : m < M) && nt < NF) {
          int next;
          const float* rp = wg_float_unit(residual, res_frag, ldr, N, m >> 5, m, nt * 32, 8 * g, lane, &next);
          const int half = res_frag ? 512 : 16;      // from the first eight features to the others
#pragma unroll
          for (int f = 0; f < 4; ++f) r[f] = *reinterpret_cast<const f32x4*>(rp + half * (f >> 1) + next * (f & 1));
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = r[e >> 2][e & 3];
      }
    }
  } else {
#pragma unroll
    for (int i = 0; i < TT; ++i)
#pragma unroll
      for (int j = 0; j < TF; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
  }
  float ln_sum[TT], ln_sq[TT];
#pragma unroll
  for (int i = 0; i < TT; ++i) { ln_sum[i] = 0.f; ln_sq[i] = 0.f; }

  bf16x8 xa[2][TT], wa[2][TF];
  auto rd = [&](int slot, int ks, auto bc) {
    constexpr int b = decltype(bc)::value;
    const char* s = smem + slot * STAGE + (kg * KS + ks) * 1024 + lo;
#pragma unroll
    for (int i = 0; i < TT; ++i) xa[b][i] = *reinterpret_cast<const bf16x8*>(s + (wt * TT + i) * (BKF * 1024));
#pragma unroll
    for (int j = 0; j < TF; ++j) wa[b][j] = *reinterpret_cast<const bf16x8*>(s + (BT + wf * TF + j) * (BKF * 1024));
  };
  auto mm = [&](int kidx, auto bc) {
    constexpr int b = decltype(bc)::value;
#pragma unroll
    for (int i = 0; i < TT; ++i)
#pragma unroll
      for (int j = 0; j < TF; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa[b][j], xa[b][i], acc[i][j], 0, 0, 0);
    if constexpr (LN) {
      // row sums of the tokens; the waves that share a token row take alternate k-steps
      if ((kidx & (WF - 1)) == wf) {
        const bf16x2_b ones = __builtin_bit_cast(bf16x2_b, 0x3f803f80u);
#pragma unroll
        for (int i = 0; i < TT; ++i) {
          const u32x4 raw = __builtin_bit_cast(u32x4, xa[b][i]);
          const unsigned int wds[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const bf16x2_b v2 = __builtin_bit_cast(bf16x2_b, wds[q]);
            ln_sum[i] = __builtin_amdgcn_fdot2_f32_bf16(v2, ones, ln_sum[i], false);
            ln_sq[i] = __builtin_amdgcn_fdot2_f32_bf16(v2, v2, ln_sq[i], false);
          }
        }
      }
    }
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
#define DF_SB __builtin_amdgcn_sched_barrier(0)
  using I2 = std::integral_constant<int, 2>;
  using All = std::integral_constant<int, -1>;
  constexpr bool SEG = EPI == EPI_QKV;
  WOut out = {};
  auto request_args = [&] {                            // (behind the first loads)
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (EPI != EPI_PART && EPI != EPI_XA) out = wg_outputs<SEG>(p);
    if constexpr (EPI == EPI_XA) asm volatile("" ::"s"(p.out_packed), "s"(p.ln_eps), "s"(p.xkv), "s"(p.xa_rows), "s"(p.xa_bstride));
  };
  // Cross-attention on a tile whose waves hold a head each: its keys and values are requested when nothing else is left to request.
  constexpr bool kDirectXa = EPI == EPI_XA && KG == 1 && TF == 2;
  bf16x8 xkf[XA > 0 ? XA : 1][4], xvf[XA > 0 ? 2 * XA : 1][2];
  const bf16x8* kv = nullptr;
  auto request_kv = [&] {
    const int mt = mg * BT + wt * TT, head = ng * WF + wf;
    const int bi = mt * 32 < p.xa_rows || mt >= MT ? 0 : mt * 32 / p.xa_rows;
    kv = p.xkv + (size_t)bi * p.xa_bstride + (size_t)(head * 2 < NF ? head : 0) * (12 * XA) * 64 + lane;
#pragma unroll
    for (int kt = 0; kt < XA; ++kt)
#pragma unroll
      for (int ds = 0; ds < 4; ++ds) xkf[kt][ds] = kv[(size_t)(kt * 4 + ds) * 64];
    if constexpr (OCC == 1)
#pragma unroll
      for (int ks = 0; ks < 2 * XA; ++ks)
#pragma unroll
        for (int dt = 0; dt < 2; ++dt) xvf[ks][dt] = kv[(size_t)(4 * XA + dt * 2 * XA + ks) * 64];
  };
  if constexpr (ST >= 4) {
    // Stage kt + ST - 1 is requested in parts between the matrix instructions of stage kt
    constexpr int LATE = NL - ((KS - 1) * NL + KS - 1) / KS;   // loads of the part behind the barrier
#pragma unroll
    for (int s = 0; s < ST - 1; ++s) issue(s < KT ? s : KT - 1, s, All{});   // past the end: the last stage again
    request_args();
    wait_vm_lds<NL * (ST - 2)>();
    block_sync();
    rd(0, 0, I0{});
    int slot = 0, pslot = ST - 1, kt = 0;
    for (; kt + ST - 1 < KT; ++kt) {
      const int nslot = slot + 1 == ST ? 0 : slot + 1, kn = kt + ST - 1;
      DF_SB; rd(slot, 1, I1{}); DF_SB; mm(kt * KS, I0{}); DF_SB; issue(kn, pslot, I0{});
      if constexpr (KS == 4) {
        DF_SB; rd(slot, 2, I0{}); DF_SB; mm(kt * KS + 1, I1{}); DF_SB; issue(kn, pslot, I1{});
        DF_SB; rd(slot, 3, I1{}); DF_SB; mm(kt * KS + 2, I0{}); DF_SB; issue(kn, pslot, I2{});
      }
      wait_vm_lds<NL * (ST - 2) - LATE>();
      block_sync();
      rd(nslot, 0, I0{});
      DF_SB; mm(kt * KS + KS - 1, I1{}); DF_SB; issue(kn, pslot, std::integral_constant<int, KS - 1>{});
      pslot = slot;
      slot = nslot;
    }
    // The last ST - 1 stages have been requested.  (With the last one requested again and again to keep the counts, the loop ended
    // with a wait for stages that nobody reads: 10 - 30 % of the loads.)
    auto last = [&](auto uc) {                           // stage kt, uc stages into the tail: false behind the last one
      constexpr int U = decltype(uc)::value;
      const int nslot = slot + 1 == ST ? 0 : slot + 1;
      if constexpr (kDirectXa && U == ST - 2) request_kv();   // (nothing is in flight any more)
      DF_SB; rd(slot, 1, I1{}); DF_SB; mm(kt * KS, I0{}); DF_SB;
      if constexpr (KS == 4) {
        rd(slot, 2, I0{}); DF_SB; mm(kt * KS + 1, I1{}); DF_SB;
        rd(slot, 3, I1{}); DF_SB; mm(kt * KS + 2, I0{}); DF_SB;
      }
      const bool more = U < ST - 2 && kt + 1 < KT;
      if (more) {
        wait_vm_lds<U < ST - 2 ? NL * (ST - 3 - U) : 0>();   // (stages of a short K that were requested twice count too)
        block_sync();
        rd(nslot, 0, I0{});
      }
      DF_SB; mm(kt * KS + KS - 1, I1{}); DF_SB;
      slot = nslot;
      ++kt;
      return more;
    };
    static_assert(ST <= 6, "");
    if (last(I0{}) && last(I1{}))
      if (last(I2{}))
        if constexpr (ST >= 5)
          if (last(std::integral_constant<int, 3>{}))
            if constexpr (ST >= 6) last(std::integral_constant<int, 4>{});
    if (KT < ST - 1) wait_vm_lds<0>();                   // the ring becomes the epilogue's (cross-attention has more stages, launch_one)
  } else {
#pragma unroll
  for (int s = 0; s < ST; ++s)
    if (s < KT) issue(s, s, All{});
  request_args();
  if (ST <= KT) wait_vm_lds<NL * (ST - 1)>();
  else wait_vm_lds<0>();
  block_sync();
  rd(0, 0, I0{});
  int slot = 0;
  for (int kt = 0; kt < KT; ++kt) {
    const int nslot = slot + 1 == ST ? 0 : slot + 1;
    DF_SB; rd(slot, 1, I1{}); DF_SB; mm(kt * KS, I0{}); DF_SB;
    if constexpr (KS == 4) {
      rd(slot, 2, I0{}); DF_SB; mm(kt * KS + 1, I1{}); DF_SB;
      rd(slot, 3, I1{}); DF_SB; mm(kt * KS + 2, I0{}); DF_SB;
    }
    if (kt + 1 < KT) {
      if (kt + ST <= KT) wait_vm_lds<NL * (ST - 2)>();
      else wait_vm_lds<0>();
      block_sync();
      rd(nslot, 0, I0{});
      if (kt + ST < KT) issue(kt + ST, slot, All{});
    }
    DF_SB; mm(kt * KS + KS - 1, I1{}); DF_SB;
    slot = nslot;
  }
  }

  if constexpr (EPI == EPI_PART) {
    // the part's sums as they are: [part][token row][feature row][quarter][lane], 1 KB per store
    static_assert(KG == 1, "one wave holds the sum of a part");
    f32x4* d = p.partials + (size_t)blockIdx.y * MT * NF * 256 + lane;
#pragma unroll
    for (int i = 0; i < TT; ++i)
#pragma unroll
      for (int j = 0; j < TF; ++j) {
        const int mt = mg * BT + wt * TT + i, nt = ng * BF + wf * TF + j;
        if (mt >= MT || nt >= NF) continue;
#pragma unroll
        for (int h = 0; h < 4; ++h)
          d[((size_t)mt * NF + nt) * 256 + h * 64] = f32x4{acc[i][j][4 * h], acc[i][j][4 * h + 1], acc[i][j][4 * h + 2], acc[i][j][4 * h + 3]};
      }
    return;
  }

  auto add_residual = [&](int mt, int m, int n0, int fo, int ln, float* v) {
    int next;
    const float* rp = wg_float_unit(p.residual, p.res_frag, p.ldr, N, mt, m, n0, fo, ln, &next);
    float r8[8];
    ld_vec(rp, r8); ld_vec(rp + next, r8 + 4);
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] += r8[q];
  };

  // ---- epilogue: the operand ring is free ----
  // One k-group: a wave finishes its own tile where it stands, in the accumulators.  A lane holds one token's 2 x 8 consecutive
  // features of every fragment, which is the unit of the packed output.  The folded LayerNorm, rstd (x - mean s) + t, is a
  // product with rstd and then one v_mfma_f32_32x32x2_f32 per fragment, whose two k's are s x (-mean rstd) and t x 1 (a plain layer:
  // bias x 1): float throughout, on the matrix unit beside the vector ALU, which bounds these epilogues, and two LDS reads per
  // fragment instead of four per eight values.  4096 x 5120 x 640 with GEGLU (256 x 320 tile): 11.1 us of epilogue through LDS as below
  // with the norm on the vector ALU, 5.2 now, which is what the vector ALU takes for the gates.
  if constexpr (KG == 1 && (EPI != EPI_XA || TF == 2)) {
    using D = Direct<WT, WF, TT, TF, LN, EPI == EPI_GEGLU>;
    constexpr bool kOdd = EPI == EPI_GEGLU && TF % 2;
    f32x4* xch = reinterpret_cast<f32x4*>(smem);       // [from wave row 0 / 1][BT][2][64 lanes]
    float* s_part = reinterpret_cast<float*>(smem + D::kXch);            // [WF][BT*32][2]
    float* s_t = reinterpret_cast<float*>(smem + D::kXch + D::kStats);   // [BF*32] shift / bias
    float* s_s = s_t + BF * 32;                        // [BF*32] scale sums
    if constexpr (kDirectXa && ST < 4) request_kv();
    block_sync();
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      const int r = tid + q * 64 * NW;
      if (r < BF * 32) { s_t[r] = vt[q]; if constexpr (LN) s_s[r] = vs[q]; }
    }
    if constexpr (LN) {
#pragma unroll
      for (int i = 0; i < TT; ++i) {
        const float sm = ln_sum[i] + __shfl_xor(ln_sum[i], 32, 64);
        const float sq = ln_sq[i] + __shfl_xor(ln_sq[i], 32, 64);
        if (g == 0) {
          float* d = s_part + ((wf * BT + wt * TT + i) * 32 + tok) * 2;
          d[0] = sm; d[1] = sq;
        }
      }
    }
    if constexpr (kOdd) {
      // of the shared pair the first wave finishes features 0 - 7 of either half, the second 8 - 15 (register order)
#pragma unroll
      for (int i = 0; i < TT; ++i) {
        const f32x16& a = acc[i][HP];
        f32x4* d = xch + ((wf * BT + wt * TT + i) * 2) * 64 + lane;
        if (wf == 0) {
          d[0] = f32x4{a[8], a[9], a[10], a[11]};
          d[64] = f32x4{a[12], a[13], a[14], a[15]};
        } else {
          d[0] = f32x4{a[0], a[1], a[2], a[3]};
          d[64] = f32x4{a[4], a[5], a[6], a[7]};
        }
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // (a barrier that leaves the keys and values on their way)
    block_sync();
    // weight row tok of a fragment is its feature sigma(tok) (bits 2 and 3 swapped)
    const int sig = (tok & 0x13) | ((tok & 4) << 1) | ((tok & 8) >> 1);
    auto vec_of = [&](int r) { return LN ? (g ? s_t : s_s)[r * 32 + sig] : g ? s_t[r * 32 + sig] : 0.f; };
    auto rows_out = [&](auto po) {
      constexpr bool packed_only = decltype(po)::value;  // (the step's GEGLU: short code, it is cold in every launch)
#pragma unroll
      for (int i = 0; i < TT; ++i) {
        const int mt = mg * BT + wt * TT + i, m = mt * 32 + tok;
        float rstd = 1.f, bm = g ? 1.f : 0.f;
        if constexpr (LN) {
          float sm = 0.f, sq = 0.f;
#pragma unroll
          for (int w = 0; w < WF; ++w) {
            const float* q = s_part + ((w * BT + wt * TT + i) * 32 + tok) * 2;
            sm += q[0]; sq += q[1];
          }
          const float inv_k = __builtin_amdgcn_rcpf((float)K);
          const float mean = sm * inv_k;
          const float var = fmaxf(fmaf(sq, inv_k, -mean * mean), 0.f);
          rstd = __builtin_amdgcn_rsqf(var + p.ln_eps);
          bm = g ? 1.f : -mean * rstd;
        }
        auto finish = [&](f32x16& a, int r) {            // tile row r: norm and shift, or bias
          if constexpr (LN) {
#pragma unroll
            for (int e = 0; e < 16; ++e) a[e] *= rstd;
          }
          a = __builtin_amdgcn_mfma_f32_32x32x2f32(vec_of(r), bm, a, 0, 0, 0);
        };
        auto store = [&](int nt, int f, float* v) {
          if (mt >= MT || nt >= NF) return;
          if constexpr (!kResInit) {
            if (p.residual && (m < M || p.res_frag)) add_residual(mt, m, nt * 32, 16 * f + 8 * g, lane, v);
          }
          wg_store_unit<SEG>(p, out, mt, m, nt * 32, 16 * f + 8 * g, lane, v);
        };
        if constexpr (EPI == EPI_GEGLU) {
          if (mt >= MT) continue;
          auto unit = [&](int nt, int f, const f32x16& a, const f32x16& gt) {
            if (nt >= NF) return;
            float v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = a[8 * f + q] * gelu_erf(gt[8 * f + q]);
            if (packed_only) st_vec(out.packed + (((size_t)mt * (N >> 4) + nt * 2 + f) * 64 + lane) * 8, v);
            else store(nt, f, v);
          };
#pragma unroll
          for (int j = 0; j < HP; ++j) {
            finish(acc[i][j], wf * TF + j);
            finish(acc[i][TF - HP + j], wf * TF + TF - HP + j);
#pragma unroll
            for (int f = 0; f < 2; ++f) unit(ng * BFO + wf * (TF - HP) + j, f, acc[i][j], acc[i][TF - HP + j]);
          }
          if constexpr (kOdd) {
            const f32x4* d = xch + (((1 - wf) * BT + wt * TT + i) * 2) * 64 + lane;
            const f32x4 lo = d[0], hi = d[64];
            f32x16 o;
#pragma unroll
            for (int e = 0; e < 16; ++e) o[e] = (e & 4 ? hi : lo)[e & 3];
            finish(acc[i][HP], wf * TF + HP);
            finish(o, (1 - wf) * TF + HP);
            if (wf == 0) unit(ng * BFO + HP, 0, acc[i][HP], o);
            else unit(ng * BFO + HP, 1, o, acc[i][HP]);
          }
        } else if constexpr (EPI == EPI_XA) {
          finish(acc[i][0], wf * TF);
          finish(acc[i][1], wf * TF + 1);
          const int head = ng * WF + wf;
          if (mt >= MT || head * 2 >= NF) continue;
          // the head's normalised, rounded query is the B operand of S^T = K Q^T
          bf16x8 qf[4];
#pragma unroll
          for (int ds = 0; ds < 4; ++ds) {
            const f32x16& a = acc[i][ds >> 1];
            const int e = 8 * (ds & 1);
            qf[ds] = __builtin_bit_cast(bf16x8, u32x4{pack_bf2(a[e], a[e + 1]), pack_bf2(a[e + 2], a[e + 3]), pack_bf2(a[e + 4], a[e + 5]),
                                                      pack_bf2(a[e + 6], a[e + 7])});
          }
          xa_head<XA, (OCC > 1)>(p, mt, head, g, lane, qf, xkf, xvf, kv);
        } else if constexpr (EPI == EPI_QKV) {
#pragma unroll
          for (int j = 0; j < TF; ++j) {
            finish(acc[i][j], wf * TF + j);
            const int nt = ng * BF + wf * TF + j;
            if (mt >= MT || nt >= NF) continue;
#pragma unroll
            for (int f = 0; f < 2; ++f) {
              float v[8];
#pragma unroll
              for (int q = 0; q < 8; ++q) v[q] = acc[i][j][8 * f + q];
              wg_store_unit<SEG>(p, out, mt, m, nt * 32, 16 * f + 8 * g, lane, v);
            }
          }
        } else {
#pragma unroll
          for (int j = 0; j < TF; ++j) {
            finish(acc[i][j], wf * TF + j);
#pragma unroll
            for (int f = 0; f < 2; ++f) {
              float v[8];
#pragma unroll
              for (int q = 0; q < 8; ++q) v[q] = acc[i][j][8 * f + q];
              store(ng * BF + wf * TF + j, f, v);
            }
          }
        }
      }
    };
    if (EPI == EPI_GEGLU && out.packed && !out.f32 && !out.rows && !p.residual) rows_out(std::true_type{});
    else rows_out(std::false_type{});
    return;
  }

  // Several k-groups: their accumulators meet in LDS.
  constexpr int R = E::R;
  f32x4* red = reinterpret_cast<f32x4*>(smem);         // [KG][R rows][BF][2 f][2 halves][64 lanes]
  float* s_part = reinterpret_cast<float*>(smem + E::pass_bytes(R));   // [KG*WF][BT*32][2] partial (sum, sum of squares)
  float* s_mr = s_part + (LN ? KG * WF * BT * 64 : 0);  // [BT*32][2] mean, rstd
  float* s_t = s_part + E::kStats / 4;                 // [BF*32] shift / bias
  float* s_s = s_t + BF * 32;                          // [BF*32] scale sums (folded LayerNorm)
  block_sync();
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    const int r = tid + q * 64 * NW;
    if (r < BF * 32) { s_t[r] = vt[q]; if constexpr (LN) s_s[r] = vs[q]; }
  }
  if constexpr (LN) {
#pragma unroll
    for (int i = 0; i < TT; ++i) {
      const float sm = ln_sum[i] + __shfl_xor(ln_sum[i], 32, 64);
      const float sq = ln_sq[i] + __shfl_xor(ln_sq[i], 32, 64);
      if (g == 0) {
        float* d = s_part + (((kg * WF + wf) * BT + wt * TT + i) * 32 + tok) * 2;
        d[0] = sm; d[1] = sq;
      }
    }
  }
#pragma unroll 1
  for (int pass = 0; pass < BT / R; ++pass) {
    if (pass > 0) __syncthreads();                     // the previous pass has been read
#pragma unroll
    for (int i = 0; i < TT; ++i) {
      const int row = i * WT + wt - pass * R;          // (uniform; accumulator indices stay compile-time)
      if (row < 0 || row >= R) continue;
#pragma unroll
      for (int j = 0; j < TF; ++j)
#pragma unroll
        for (int h = 0; h < 4; ++h)
          red[(((kg * R + row) * BF + wf * TF + j) * 4 + h) * 64 + lane] =
              f32x4{acc[i][j][4 * h], acc[i][j][4 * h + 1], acc[i][j][4 * h + 2], acc[i][j][4 * h + 3]};
    }
    __syncthreads();
    if constexpr (LN) {
      if (pass == 0) {
        for (int r = tid; r < BT * 32; r += 64 * NW) {
          float sm = 0.f, sq = 0.f;
#pragma unroll
          for (int w = 0; w < KG * WF; ++w) { sm += s_part[(w * BT * 32 + r) * 2]; sq += s_part[(w * BT * 32 + r) * 2 + 1]; }
          const float inv_k = __builtin_amdgcn_rcpf((float)K);
          const float mean = sm * inv_k;
          const float var = fmaxf(fmaf(sq, inv_k, -mean * mean), 0.f);
          s_mr[2 * r] = mean;
          s_mr[2 * r + 1] = __builtin_amdgcn_rsqf(var + p.ln_eps);
        }
        __syncthreads();
      }
    }
    // 8 consecutive features 16f + 8g .. of tile fragment (row r of the pass, weight row jf), token tk of the row
    auto value8 = [&](int r, int trow, int jf, int f, int gg, int tk, float* v) {
      f32x4 a, b;
#pragma unroll
      for (int k = 0; k < KG; ++k) {
        const f32x4* q = red + (((k * R + r) * BF + jf) * 4 + 2 * f) * 64 + tk + 32 * gg;
        a = k ? a + q[0] : q[0];
        b = k ? b + q[64] : q[64];
      }
      const float* tv = s_t + jf * 32 + 16 * f + 8 * gg;
      const f32x4 t0 = *reinterpret_cast<const f32x4*>(tv), t1 = *reinterpret_cast<const f32x4*>(tv + 4);
      if constexpr (LN) {
        const float* sv = s_s + jf * 32 + 16 * f + 8 * gg;
        const f32x4 s0 = *reinterpret_cast<const f32x4*>(sv), s1 = *reinterpret_cast<const f32x4*>(sv + 4);
        const float mean = s_mr[(trow * 32 + tk) * 2], rstd = s_mr[(trow * 32 + tk) * 2 + 1];
        a = (a - s0 * mean) * rstd + t0;
        b = (b - s1 * mean) * rstd + t1;
      } else {
        a += t0;
        b += t1;
      }
      v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    };

    if constexpr (EPI == EPI_XA) {
      // items (token row of the pass, head): the head's normalised, rounded query is the B operand of S^T = K Q^T
      constexpr int HW = BF / 2;
#pragma unroll 1
      for (int it = wave; it < R * HW; it += NW) {
        const int hd = it % HW, r = it / HW;
        const int q0 = pass * R + r, trow = (q0 % WT) * TT + q0 / WT, mt = mg * BT + trow, head = ng * HW + hd;
        if (mt >= MT || head * 2 >= NF) continue;
        const int bi = mt * 32 < p.xa_rows ? 0 : mt * 32 / p.xa_rows;
        const bf16x8* kv = p.xkv + (size_t)bi * p.xa_bstride + (size_t)head * (12 * XA) * 64 + lane;
        bf16x8 kf[XA][4];
#pragma unroll
        for (int kt = 0; kt < XA; ++kt)
#pragma unroll
          for (int ds = 0; ds < 4; ++ds) kf[kt][ds] = kv[(size_t)(kt * 4 + ds) * 64];
        bf16x8 qf[4];
#pragma unroll
        for (int ds = 0; ds < 4; ++ds) {
          float v[8];
          value8(r, trow, hd * 2 + (ds >> 1), ds & 1, g, tok, v);
          const u32x4 qv = {pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3]), pack_bf2(v[4], v[5]), pack_bf2(v[6], v[7])};
          qf[ds] = __builtin_bit_cast(bf16x8, qv);
        }
        xa_head<XA, true>(p, mt, head, g, lane, qf, kf, nullptr, kv);
      }
    } else {
      // items (token row, output fragment, half of the row's tokens): lane -> token it*16 + lane%16, features 8*(lane/16) ..
      const int tl = lane & 15, f = lane >> 5, gg = (lane >> 4) & 1;
#pragma unroll 1
      for (int it = wave; it < R * BFO * 2; it += NW) {
        const int half = it & 1, jo = (it >> 1) % BFO, r = (it >> 1) / BFO;
        const int q0 = pass * R + r, trow = (q0 % WT) * TT + q0 / WT, mt = mg * BT + trow, nt = ng * BFO + jo;
        if (mt >= MT || nt >= NF) continue;
        const int jf = jo;
        const int tk = half * 16 + tl;
        float v[8];
        value8(r, trow, jf, f, gg, tk, v);
        if constexpr (EPI == EPI_GEGLU) {
          float gt[8];
          value8(r, trow, jf + BFO, f, gg, tk, gt);
#pragma unroll
          for (int q = 0; q < 8; ++q) v[q] *= gelu_erf(gt[q]);
        }
        const int m = mt * 32 + tk;
        if constexpr (!kResInit) {
          if (p.residual && (m < M || p.res_frag)) add_residual(mt, m, nt * 32, 16 * f + 8 * gg, tk + 32 * gg, v);
        }
        wg_store_unit<SEG>(p, out, mt, m, nt * 32, 16 * f + 8 * gg, tk + 32 * gg, v);
      }
    }
  }
}

// Adds the parts of K in their order and finishes the layer: a wave per half of a fragment (token row, 16 features), all parts
// (at most eight) requested together with what is added to them.  1024 x 1280 in three parts 7.0 -> 6.8 us (a loop that requested
// the next part before it added one), bound by the 16 MB of sums; 64 x 1280 in four 4.7, a launch and two round trips to memory.
template <int NP>
__global__ __launch_bounds__(256) void bgemm_sum_kernel(WParams p) {
  asm volatile("" ::"s"(p.partials), "s"(p.M), "s"(p.N), "s"(p.bias), "s"(p.residual), "s"(p.ldr), "s"(p.out_f32), "s"(p.ldo), "s"(p.out_packed),
               "s"(p.out_rows), "s"(p.nseg), "s"(p.res_frag), "s"(p.f32_frag));   // (one batch of argument loads, see wgemm.hip)
  const int MT = (p.M + 31) >> 5, NF = p.N >> 5, lane = threadIdx.x & 63;
  const int u = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (u >= MT * NF * 2) return;
  const int fr = u >> 1, f = u & 1, mt = fr / NF, nt = fr - mt * NF;
  const int m = mt * 32 + (lane & 31), n = nt * 32 + 16 * f + 8 * (lane >> 5);
  const f32x4* s = p.partials + (size_t)fr * 256 + f * 128 + lane;
  f32x4 ta[NP], tb[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    ta[i] = s[0];
    tb[i] = s[64];
    s += (size_t)MT * NF * 256;
  }
  f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = a, ba = a, bb = a;
  if (p.bias) {
    ba = *reinterpret_cast<const f32x4*>(p.bias + n);
    bb = *reinterpret_cast<const f32x4*>(p.bias + n + 4);
  }
  if (p.residual && (m < p.M || p.res_frag)) {
    int next;
    const float* rp = wg_float_unit(p.residual, p.res_frag, p.ldr, p.N, mt, m, nt * 32, 16 * f + 8 * (lane >> 5), lane, &next);
    a = *reinterpret_cast<const f32x4*>(rp);
    b = *reinterpret_cast<const f32x4*>(rp + next);
  }
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    a += ta[i];
    b += tb[i];
  }
  if (p.bias) {
    a += ba;
    b += bb;
  }
  const float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
  wg_store_unit<false>(p, wg_outputs<false>(p), mt, m, nt * 32, 16 * f + 8 * (lane >> 5), lane, v);
}

template <int WT, int WF, int TT, int TF, int KG, int KS, int ST, int OCC, int EPI, bool LN, int XA>
int launch_one(const WParams& pin, hipStream_t st) {
  constexpr int BT = WT * TT, BF = WF * TF, BFO = EPI == EPI_GEGLU ? BF / 2 : BF, NW = WT * WF * KG;
  WParams p = pin;
  const int MT = (p.M + 31) / 32, NF = p.N / 32;
  const int MG = (MT + BT - 1) / BT, NG = (NF + BFO - 1) / BFO;
  const long long nwg = (long long)MG * NG;
  if ((p.K / 16) % (KS * KG)) return DF_ESHAPE;
  // a tile whose waves hold a head each requests keys and values beside the last of at least ST - 1 stages
  if (EPI == EPI_XA && KG == 1 && TF == 2 && ST >= 4 && p.K / (16 * KS * KG) < ST - 1) return DF_ESHAPE;
  const int parts = EPI == EPI_PART ? p.parts : 1;
  const double conc = std::fmin((double)nwg / 8.0, 32.0 * OCC / parts);
  int gm = (int)(std::sqrt(conc * BF / BT) + 0.5);
  if (gm < 1) gm = 1;
  if (gm > MG) gm = MG;
  const int np = (MG + gm - 1) / gm;
  p.group_m = (MG + np - 1) / np;
  constexpr int ring = ST * (BT + BF) * KS * KG * 1024;
  constexpr bool direct = KG == 1 && (EPI != EPI_XA || TF == 2);
  constexpr int fin = direct ? Direct<WT, WF, TT, TF, LN, EPI == EPI_GEGLU>::kBytes : Epi<WT, WF, TT, TF, KG, OCC, LN>::kBytes;
  constexpr int smem = ring > fin ? ring : fin;
  static_assert(smem <= 160 * 1024, "LDS of a compute unit");
  auto k = bgemm_kernel<WT, WF, TT, TF, KG, KS, ST, OCC, EPI, LN, XA>;
  static bool attr_set = false;
  if (!attr_set) {
    if (hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, smem) != hipSuccess) return DF_EHIP;
    attr_set = true;
  }
  const unsigned int order = (unsigned int)p.group_m | (unsigned int)parts << 26 | (p.res_frag ? 1u << 30 : 0u);   // (parts: at most eight)
  hipLaunchKernelGGL(k, dim3((unsigned)nwg, (unsigned)parts), dim3(64 * NW), smem, st, p.Xp, p.Wp, p.ln_s, LN ? p.ln_t : p.bias, p.residual,
                     p.M, p.N, p.K, order, p);
  DF_LAUNCH_CHECK();
  if constexpr (EPI == EPI_PART) {
    return launch_part_sums(p, st);
  }
  return DF_OK;
}

template <int WT, int WF, int TT, int TF, int KG, int KS, int ST, int OCC>
int launch_tile_cfg(const WParams& p, hipStream_t st) {
  constexpr int BF = WF * TF;
  if (p.xkv) {
    if constexpr (BF % 2 == 0 && WT * TT * BF <= 16) {   // (the registers of a larger tile's wave do not hold keys and values too)
      switch ((p.xa_keys + 31) / 32) {
        case 1: return launch_one<WT, WF, TT, TF, KG, KS, ST, OCC, EPI_XA, true, 1>(p, st);
        case 2: return launch_one<WT, WF, TT, TF, KG, KS, ST, OCC, EPI_XA, true, 2>(p, st);
        case 3: return launch_one<WT, WF, TT, TF, KG, KS, ST, OCC, EPI_XA, true, 3>(p, st);
        default: return launch_one<WT, WF, TT, TF, KG, KS, ST, OCC, EPI_XA, true, 4>(p, st);
      }
    }
    return DF_ESHAPE;
  }
  if (p.geglu) {
    if constexpr (BF % 2 == 0 && BF > 2) {               // (64 x 64 tiles: one value fragment per wave row, never the choice)
      if (p.ln_s) return launch_one<WT, WF, TT, TF, KG, KS, ST, OCC, EPI_GEGLU, true, 0>(p, st);
      return launch_one<WT, WF, TT, TF, KG, KS, ST, OCC, EPI_GEGLU, false, 0>(p, st);
    }
    return DF_ESHAPE;
  }
  if (p.nseg) {
    if (!p.ln_s) return DF_ESHAPE;                       // (the segmented projections of the step fold a LayerNorm)
    return launch_one<WT, WF, TT, TF, KG, KS, ST, OCC, EPI_QKV, true, 0>(p, st);
  }
  if (p.parts > 1) {
    if constexpr (TT == 1 && KG == 1 && OCC == 1 && TF != 3) return launch_one<WT, WF, TT, TF, KG, KS, ST, OCC, EPI_PART, false, 0>(p, st);
    return DF_ESHAPE;
  }
  if (p.ln_s) return launch_one<WT, WF, TT, TF, KG, KS, ST, OCC, EPI_PLAIN, true, 0>(p, st);
  return launch_one<WT, WF, TT, TF, KG, KS, ST, OCC, EPI_PLAIN, false, 0>(p, st);
}

}  // namespace

// Adds the parts of K, with bias and residual, and writes the layer's outputs.
int launch_part_sums(const WParams& p, hipStream_t st) {
  const int units = ((p.M + 31) / 32) * (p.N / 32) * 2;
  const dim3 grid((unsigned)((units + 3) / 4));
  switch (p.parts) {
#define DF_SUM(NP) case NP: hipLaunchKernelGGL(bgemm_sum_kernel<NP>, grid, dim3(256), 0, st, p); break
    DF_SUM(2); DF_SUM(3); DF_SUM(4); DF_SUM(5); DF_SUM(6); DF_SUM(7); DF_SUM(8);
#undef DF_SUM
    default: return DF_ESHAPE;
  }
  DF_LAUNCH_CHECK();
  return DF_OK;
}

int launch_bgemm(const WParams& p, int cfg, hipStream_t st) {
  switch (cfg) {
    case 0: return launch_tile_cfg<4, 2, 2, 5, 1, 2, 4, 1>(p, st);
    case 1: return launch_tile_cfg<4, 2, 1, 2, 1, 4, 2, 2>(p, st);
    case 2: return launch_tile_cfg<4, 2, 1, 2, 1, 4, 4, 1>(p, st);
    case 3: return launch_tile_cfg<2, 2, 1, 2, 2, 2, 3, 2>(p, st);
    case 4: return launch_tile_cfg<2, 2, 1, 1, 2, 4, 2, 2>(p, st);
    case 5: return launch_tile_cfg<2, 2, 1, 1, 2, 4, 4, 1>(p, st);
    case 6: return launch_tile_cfg<4, 2, 1, 5, 1, 2, 5, 1>(p, st);
    case 7: return launch_tile_cfg<2, 1, 1, 3, 4, 2, 4, 1>(p, st);
    case 8: return launch_tile_cfg<4, 1, 1, 5, 2, 2, 4, 1>(p, st);
    case 9: return launch_tile_cfg<4, 2, 2, 4, 1, 2, 4, 1>(p, st);
    case 10: return launch_tile_cfg<4, 1, 1, 3, 2, 2, 5, 1>(p, st);
    case 11: return launch_tile_cfg<4, 2, 1, 3, 1, 2, 6, 1>(p, st);
    default: return DF_ESHAPE;
  }
}

// bytes of scratch that a plain layer's parts of K may take
size_t wgemm_scratch_bytes(long long M, long long N) {
  const long long MT = (M + 31) / 32, NF = N / 32;
  int parts = 1;
  for (const SplitCfg& q : kSplits) {
    const int n = max_parts(kTiles[q.tile], MT, NF);
    if (n > parts) parts = n;
  }
  return kScratchCounterBytes + (parts > 1 ? (size_t)parts * MT * NF * 4096 : 0);
}

}  // namespace df
