#include <cmath>
#include <type_traits>

#include "tile.h"

namespace df {

namespace {

template <int VM>
__device__ __forceinline__ void wait_vm_lds() {   // s_waitcnt vmcnt(VM) lgkmcnt(0)
  __builtin_amdgcn_s_waitcnt((VM & 0xF) | ((VM >> 4) << 14) | (0x7 << 4));
}
template <int MOST>
__device__ __forceinline__ void wait_vm_lds(int n) {   // the same with a count (0 .. MOST) that unrolling makes known
  if (n == MOST) wait_vm_lds<MOST>();
  else if constexpr (MOST > 0) wait_vm_lds<MOST - 1>(n);
}
struct RcExtra {
  const bf16_t* zeros;
  float* partials;
  int th, tw;                 // output pixels of a tile: th rows x tw columns, th * tw <= BM
  int tiles_r, tiles_c;       // tiles of an image of the batch
  unsigned int tw_magic;      // ceil(2^16 / tw): s / tw for s < 256
  unsigned int rw_magic;      // ceil(2^20 / (tw + 2)): p / (tw + 2) for p < 512
  int group_m;
};

// Fragment rows of a tile that go through LDS at once in the epilogue
constexpr int pass_rows(int rows, int kg, int bn) {
  int r = rows;
  while (r > 1 && (rows % r || kg * r * 32 * (bn + 4) * 4 > 144 * 1024)) --r;
  return r;
}

// 3x3 convolution, stride 1, on a th x tw tile of output pixels by BN output channels per workgroup: the tile's input pixels
// with their border, (th + 2) x (tw + 2) of 64 channels, stay in LDS while the nine taps of those channels pass, so that they
// cross the load path once and not nine times; the weights go through a ring of ST stages of TAPS taps each.
// Eight waves of TM x TN blocks of 32 x 32 outputs: PM x PN of them over the tile and KG over the 16-deep steps of a tap, added
// through LDS at the end.  Two buffers of input pixels; the next 64 channels' are requested during the current ones'.
// What bounds it: with few tiles the barriers and the launch (128 x 64 outputs: 1.8 us per 64 channels against 0.96 of matrix
// instructions, 1.45 without any loads in the loop; 7 us for prologue, epilogue and kernel boundary), hence three taps per
// barrier where the weights' stages fit; with all compute units busy the clock under the power limit (256 x 160: 1100 TFLOP/s on
// 28800 pixels x 640 x 320 channels).
// Same machine, against the tiles of tgemm.hip: 4096 pixels x 320 x 320 21.0 -> 14.1 us, 300 x 1280 x 1280 25.1 -> 20.6,
// 1200 x 640 x 640 20.3 -> 16.1, 4800 x 960 x 320 43.5 -> 31.4, 28800 x 640 x 320 125 -> 96.5, 4096 x 1280 x 1280 133 -> 111.
// LDS rows of 128 bytes (a pixel's or an output channel's 64 values) hold 16-byte chunk c at slot c ^ ((row >> 1) & 7): 32
// neighbouring rows, wherever they start, meet no bank twice.  (Tile widths that are no multiple of 32 do meet some: forcing whole
// 32s removed every conflict and no time, and cost tiles.)
// Order: a stage's loads are requested ST - 1 stages ahead in parts between the matrix instructions, into the slot of the
// stage that ended at the last barrier; a stage ends with the wait for the next one's loads, lgkmcnt(0) and a barrier, and
// its last matrix instructions (operands in registers) run behind that barrier beside the next stage's first reads.  The other
// buffer of pixels was last read in the stage before the current channels' first, so its refill is behind a barrier too.
// What the requests of the first weights need are the leading arguments, which come in scalar registers (as in wgemm.hip): GroupNorm and
// convolution of 128 x 128 x 320 over four patches 19.9 -> 19.5 us, 512 x 512 step 4428 -> 4407, 1024 x 1024 with guidance 6361 -> 6329.
template <int PM, int PN, int TM, int TN, int KG, int TAPS, int ST, int NIN, typename OutT>
__global__ __launch_bounds__(512, 2) void rconv_kernel(const bf16_t* Wt, const bf16_t* A, int N, int Cin, int ldw, int MT, int group_m, int nsplit,
                                                       int per_img, int tiles_c, int R, int W, TileParams p, RcExtra x) {
  static_assert(PM * PN * KG == 8, "eight waves");
  constexpr int BN = PN * TN * 32;
  constexpr int NST = 9 / TAPS;                            // stages of 64 channels
  constexpr int NK = 4 / KG, NSUB = TAPS * NK;             // 16-deep steps of a tap / of a stage, per wave
  constexpr int NB = (NSUB * NST) % 2 == 0 ? 2 : 3;        // fragment buffers, used in turn
  static_assert((NSUB * NST) % NB == 0 && 4 % KG == 0 && 9 % TAPS == 0, "");
  constexpr int WJ = (BN / 8 + 7) / 8;                     // weight loads of a wave and tap (the last wave's repeat the last rows)
  constexpr int WL = WJ * TAPS;                            // and stage
  constexpr int IB = NIN * 8192;                           // bytes of a buffer of pixels
  constexpr int WB = TAPS * BN * 128;                      // bytes of a stage of weights
  constexpr int INS = NST - (ST - 2);                      // stages that may carry pixel loads (they must land with the channels)
  static_assert(INS >= 1, "");
  constexpr int IPS = (NIN + INS - 1) / INS;               // pixel loads of one of them
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave / (PM * PN), wq = wave % (PM * PN), wm = wq % PM, wn = wq / PM;
  const int NT = (N + BN - 1) / BN, nwg = MT * NT;
  int t = blockIdx.x;
  {
    const int xcd = t & 7, loc = t >> 3;
    const int base = nwg >> 3, rem = nwg & 7;
    t = xcd * base + (xcd < rem ? xcd : rem) + loc;
  }
  int mt, n0;
  {
    const int per = group_m * NT, pn = t / per, r = t - pn * per, mf = pn * group_m;
    const int gh = MT - mf < group_m ? MT - mf : group_m;
    n0 = r / gh;
    mt = mf + r - n0 * gh;
    n0 *= BN;
  }
  const int bi = mt / per_img, trc = mt - bi * per_img;
  const int r0 = trc / tiles_c * x.th, c0 = (trc - trc / tiles_c * tiles_c) * x.tw;
  const int slabs_all = Cin / 64;
  const int s_lo = (int)((long long)slabs_all * blockIdx.y / nsplit), s_hi = (int)((long long)slabs_all * (blockIdx.y + 1) / nsplit);

  // First channel of the slab that is being computed and of the one behind it.  The XCDs begin with different slabs, where the channels are not
  // split over workgroups or a tile has 64 pixels: all of them read the same weights, and in step they ask the same channels of the last-level
  // cache.  640 -> 640 of 32 x 32 19.2 -> 16.0 us, 960 -> 320 of 26 x 76 25.7 -> 21.1, 640 -> 1280 of 26 x 19 19.1 -> 17.5; 100 layers of 64 to 7904
  // pixels 0.974 on average, 1.019 at most.  Parts of the channels begin at different slabs already: with larger tiles the start costs up to 9 %
  // (300 x 2560 -> 1280 in four parts 33.5 -> 35.7 us, 1024 x 1920 -> 640 in three 30.4 -> 31.9; 76 layers 1.011).
  const int slabs = s_hi - s_lo, rot = nsplit == 1 || PM * TM == 2 ? (int)((blockIdx.x & 7) * (unsigned int)slabs >> 3) : 0;
  auto behind = [&](int c) { return c + 64 < s_hi * 64 ? c + 64 : s_lo * 64; };
  int ch = (s_lo + rot) * 64, chn = behind(ch);
  // weight loads: instruction j of a tap covers output channels wrow(j) .. +7 of the tile, lane / 8 one of them
  const int lr = lane >> 3;
  auto wrow = [&](int j) { return (j * 8 + wave < BN / 8 ? j * 8 + wave : BN / 8 - 1) * 8; };
  const char* const w_tile = (const char*)(Wt + (long long)n0 * ldw);
  unsigned int w_ofs[WJ];
#pragma unroll
  for (int j = 0; j < WJ; ++j) {
    const int row = wrow(j) + lr;
    const int n = (n0 + row < N ? n0 + row : N - 1) - n0;   // ragged last tile: re-read, never stored
    w_ofs[j] = 2u * ((unsigned int)n * (unsigned int)ldw + ((lane & 7) ^ ((row >> 1) & 7)) * 8);
  }
  auto load_w = [&](int ch, int st, int slot, int l) {     // load l of a stage: tap l / WJ, instruction l % WJ
    const int tp = l / WJ, j = l % WJ;
    lds_load_buf(w_tile, w_ofs[j], 2u * ((st * TAPS + tp) * Cin + ch), smem + 2 * IB + slot * WB + tp * (BN * 128) + wrow(j) * 128);
  };
  // the first stage's weights, the coldest of what the loop waits for, are requested before the pixels' addresses are known
#pragma unroll
  for (int l = 0; l < WL; ++l) load_w(ch, 0, 0, l);
  // pixel loads: instruction q of a wave covers rows (q * 8 + wave) * 8 + lane / 8 of the buffer, slot lane % 8
  const int RW = x.tw + 2, np = (x.th + 2) * RW;
  const bf16_t* in_ptr[NIN];
  bool in_zero[NIN];
#pragma unroll
  for (int q = 0; q < NIN; ++q) {
    const int px = (q * 8 + wave) * 8 + lr;
    const int pr = (int)(((unsigned)px * x.rw_magic) >> 20), pc = px - pr * RW;
    const int ri = r0 + pr - 1, ci = c0 + pc - 1;
    const bf16_t* src = nullptr;
    if (px < np && ri <= R && ci <= W)
      src = conv_tap_src(A, p.top, p.bot, p.halo_bs, p.left, p.right, p.side_bs, p.side_rs, bi, ri, ci, R, W, Cin);
    in_zero[q] = src == nullptr;
    in_ptr[q] = (src ? src : x.zeros) + ((lane & 7) ^ ((px >> 1) & 7)) * 8;
  }
  auto load_in = [&](int ch, int buf, int q) {
    const bf16_t* src = in_ptr[q] + (in_zero[q] ? 0 : ch);
    lds_load16(src, smem + buf * IB + (q * 8 + wave) * 1024);
  };

  // operand addresses.  Pixel s of the tile at tap (ky, kx): buffer row pix0 + ky * RW + kx
  const int lrow = lane & 31, g = lane >> 5;
  int pix0[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int s = (wm * TM + i) * 32 + lrow;
    const int tr = (int)(((unsigned)s * x.tw_magic) >> 16), tc = s - tr * x.tw;
    pix0[i] = tr < x.th ? tr * RW + tc : 0;                // slots beyond the tile: never stored
  }
  int wofs[NK];
#pragma unroll
  for (int k = 0; k < NK; ++k) {
    const int n = wn * TN * 32 + lrow;
    wofs[k] = 2 * IB + n * 128 + (((2 * (kg * NK + k) + g) ^ ((n >> 1) & 7)) * 16);
  }
  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
  bf16x8 xa[NB][TM], wa[NB][TN];
  int xofs[TM];                                            // of the tap being read, first step of the wave
  auto rd = [&](int slot, int buf, int st, int u, int b) { // step u of stage st (compile-time st, u, b)
    const int tap = st * TAPS + u / NK, k = u % NK;
    const char* ws = smem + slot * WB + (u / NK) * (BN * 128) + wofs[k];
#pragma unroll
    for (int j = 0; j < TN; ++j) wa[b][j] = *reinterpret_cast<const bf16x8*>(ws + j * 4096);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      if (k == 0) {
        // (computed anew for every tap: left alone, the compiler keeps all of a channel block's addresses in registers and spills)
        int pix = pix0[i];
        asm volatile("" : "+v"(pix));
        pix += (tap / 3) * RW + tap % 3;
        xofs[i] = buf * IB + pix * 128 + (((2 * kg * NK + g) ^ ((pix >> 1) & 7)) * 16);
      }
      xa[b][i] = *reinterpret_cast<const bf16x8*>(smem + (xofs[i] ^ (k * 32)));
    }
  };
  auto mm = [&](int b) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa[b][j], xa[b][i], acc[i][j], 0, 0, 0);
  };
  // part `part` of NSUB of the loads requested during stage st of the channels `slab`: the weights ST - 1 stages on, and the
  // next channels' pixels.  The last channels (LAST) request what is left of their own weights and nothing else: loaded once more to
  // keep the counts behind the waits they were a fifth of the loads of 320 channels.
  auto in_loads = [&](int st) { return st * IPS >= NIN ? 0 : (NIN - st * IPS < IPS ? NIN - st * IPS : IPS); };
  auto issue = [&](auto lastc, int buf, int wslot, int st, int part) {
    constexpr bool LAST = decltype(lastc)::value;
    const int ws = st + ST - 1, nw = LAST && ws >= NST ? 0 : WL, nin = LAST ? 0 : in_loads(st), n = nw + nin;
#pragma unroll
    for (int l = 0; l < WL + IPS; ++l) {
      if (l >= n || l * NSUB / n != part) continue;
      if (l < nw) load_w(ws / NST ? chn : ch, ws % NST, wslot, l);
      else load_in(chn, buf ^ 1, st * IPS + l - nw);
    }
  };
  // loads that may still be in flight at the end of stage st: those requested in the last ST - 2 stages
  constexpr int FLY = (ST - 2) * (WL + IPS);               // (at most)
  static_assert(FLY <= 63, "vmcnt");
  auto in_flight = [&](auto lastc, int st) {
    int n = 0;
#pragma unroll
    for (int k = 0; k < ST - 2; ++k) {
      const int j = st - k;
      n += decltype(lastc)::value ? (j < 0 || j + ST - 1 < NST ? WL : 0) : WL + in_loads((j + NST) % NST);
    }
    return n;
  };
#define DF_SB __builtin_amdgcn_sched_barrier(0)
  // prologue
#pragma unroll
  for (int q = 0; q < NIN; ++q) load_in(ch, 0, q);
#pragma unroll
  for (int s = 1; s < ST - 1; ++s) {
#pragma unroll
    for (int l = 0; l < WL; ++l) load_w(s / NST ? chn : ch, s % NST, s, l);
  }
  // the epilogue's arguments (cold in every launch) come beside the first operands
  asm volatile("" ::"s"(p.bias), "s"(p.chan_add), "s"(p.chan_ld), "s"(p.residual), "s"(p.ldr), "s"(p.out), "s"(p.ldo), "s"(p.act), "s"(x.partials));
  wait_vm_lds<(ST - 2) * WL>();
  block_sync();
  rd(0, 0, 0, 0, 0);
  int slot = 0, wslot = ST - 1, buf = 0;
  using Last = std::true_type;
  using More = std::false_type;
  if (s_lo + 1 < s_hi) issue(More{}, 0, wslot, 0, 0);
  else issue(Last{}, 0, wslot, 0, 0);
  auto channels = [&](auto lastc, int slab) {
    constexpr bool LAST = decltype(lastc)::value;
#pragma unroll
    for (int st = 0; st < NST; ++st) {
      const int nslot = slot + 1 == ST ? 0 : slot + 1;
#pragma unroll
      for (int u = 0; u < NSUB; ++u) {
        const int b = (st * NSUB + u) % NB, bn = (st * NSUB + u + 1) % NB;
        if (u + 1 < NSUB) {
          DF_SB; rd(slot, buf, st, u + 1, bn); DF_SB; mm(b); DF_SB;
          issue(lastc, buf, wslot, st, u + 1);
        } else if (LAST && st + 1 == NST) {
          DF_SB; mm(b); DF_SB;
        } else {
          wait_vm_lds<FLY>(in_flight(lastc, st));
          block_sync();
          const bool wrap = st + 1 == NST;
          rd(nslot, wrap ? buf ^ 1 : buf, wrap ? 0 : st + 1, 0, bn);
          DF_SB; mm(b); DF_SB;
          // the next stage's first part goes to the slot of the stage that has just ended
          if (!wrap) {
            issue(lastc, buf, slot, st + 1, 0);
          } else {
            ch = chn;
            chn = behind(ch);
            if (slab + 2 < s_hi) issue(More{}, buf ^ 1, slot, 0, 0);
            else issue(Last{}, buf ^ 1, slot, 0, 0);
          }
        }
      }
      wslot = slot;
      slot = nslot;
    }
    buf ^= 1;
  };
  for (int slab = s_lo; slab + 1 < s_hi; ++slab) channels(More{}, slab);
  // What the epilogue adds per channel is requested where only weights are left to request.
  constexpr int RS = 512 / (BN / 4);                       // rows per round of the epilogue; a thread keeps its columns
  const bool part = nsplit > 1;
  const int c4 = (tid % (BN / 4)) * 4, col = n0 + c4;
  const bool mine = tid < RS * (BN / 4) && col < N;
  f32x4 add = {0.f, 0.f, 0.f, 0.f}, add_image = add;
  if (!part && mine) {
    if (p.bias) add = *reinterpret_cast<const f32x4*>(p.bias + col);
    if (p.chan_add) add_image = *reinterpret_cast<const f32x4*>(p.chan_add + (long long)bi * p.chan_ld + col);
  }
  channels(Last{}, s_hi - 1);
#undef DF_SB

  // ---- epilogue: accumulators -> LDS in passes of RP fragment rows of the tile, k-groups added, rows of the output stored ----
  constexpr int RP = pass_rows(PM * TM, KG, BN), PT = BN + 4;
  float* tile = reinterpret_cast<float*>(smem);
  constexpr int U = 4;                                     // rows in flight per thread
#pragma unroll 1
  for (int f0 = 0; f0 < PM * TM; f0 += RP) {
    block_sync();                                          // the ring, or the previous pass, has been read
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int fr = wm * TM + i - f0;                     // (uniform)
      if (fr < 0 || fr >= RP) continue;
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<f32x4*>(tile + ((kg * RP + fr) * 32 + lrow) * PT + (wn * TN + j) * 32 + 8 * q + 4 * g) =
              f32x4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
    }
    __syncthreads();
    if (mine) {
#pragma unroll 1
      for (int l0 = tid / (BN / 4); l0 < RP * 32; l0 += RS * U) {
        long long row[U];
        f32x4 res[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
          const int s = f0 * 32 + l0 + k * RS;
          const int tr = (int)(((unsigned)s * x.tw_magic) >> 16), tc = s - tr * x.tw;
          const bool ok = l0 + k * RS < RP * 32 && tr < x.th && r0 + tr < R && c0 + tc < W;
          row[k] = ok ? ((long long)bi * R + r0 + tr) * W + c0 + tc : -1;
          res[k] = f32x4{0.f, 0.f, 0.f, 0.f};
          if (!part && p.residual && ok) res[k] = *reinterpret_cast<const f32x4*>(p.residual + row[k] * p.ldr + col);
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
          if (row[k] < 0) continue;
          const float* tp = tile + (l0 + k * RS) * PT + c4;
          f32x4 v = *reinterpret_cast<const f32x4*>(tp);
#pragma unroll
          for (int h = 1; h < KG; ++h) v += *reinterpret_cast<const f32x4*>(tp + h * RP * 32 * PT);
          if (part) {
            *reinterpret_cast<f32x4*>(x.partials + ((size_t)blockIdx.y * p.M + row[k]) * N + col) = v;
            continue;
          }
          v += add + add_image;
          v += res[k];
          if (p.act == 1) { v.x = silu_f(v.x); v.y = silu_f(v.y); v.z = silu_f(v.z); v.w = silu_f(v.w); }
          OutT* o = reinterpret_cast<OutT*>(p.out) + row[k] * p.ldo + col;
          if constexpr (sizeof(OutT) == 4) {
            *reinterpret_cast<f32x4*>(o) = v;
          } else {
            const u32x2 w = {pack_bf2(v.x, v.y), pack_bf2(v.z, v.w)};
            *reinterpret_cast<u32x2*>(o) = w;
          }
        }
      }
    }
  }
}

// Tile of th x tw pixels for a patch of R x W: the fewest tiles, then the fewest input pixels, over heights of up to 24 rows and
// the one that takes the whole width.  This runs at every launch: a height with as many rows of tiles as the one before it is
// left out, since it is never wider.
struct Geo { int th, tw, tr, tc; };
Geo pick_geo(int R, int W, int bm, int cap) {
  Geo best = {0, 0, 0, 0};
  unsigned int fewest = ~0u, pixels = 0;
  auto cd = [](unsigned int a, unsigned int b) { return (a + b - 1) / b; };
  auto consider = [&](unsigned int th, unsigned int tr) {
    unsigned int tw = (unsigned int)bm / th;
    if ((th + 2) * (tw + 2) > (unsigned int)cap) tw = (unsigned int)cap / (th + 2) > 2 ? cap / (th + 2) - 2 : 0;
    if (tw > (unsigned int)W) tw = W;
    if (tw < 1) return;
    const unsigned int tc = cd(W, tw), n = tr * tc;
    if (n > fewest) return;
    const unsigned int h = cd(R, tr), w = cd(W, tc), in = (h + 2) * (w + 2);
    if (n < fewest || in < pixels) { fewest = n; pixels = in; best = Geo{(int)h, (int)w, (int)tr, (int)tc}; }
  };
  unsigned int last = 0;
  for (int th = 1; th <= R && th <= 24; ++th) {
    const unsigned int tr = cd(R, th);
    if (tr != last) consider(th, tr);
    last = tr;
  }
  if (W < bm) {
    int th = bm / W;
    if ((th + 2) * (W + 2) > cap) th = cap / (W + 2) - 2;
    if (th > R) th = R;
    if (th > 24) consider(th, cd(R, th));
  }
  return best;
}

template <int PM, int PN, int TM, int TN, int KG, int TAPS, int ST, int NIN, typename OutT>
int launch_one(const TileParams& p, const Geo& g, int nsplit, hipStream_t st) {
  constexpr int BM = PM * TM * 32, BN = PN * TN * 32;
  const long long MT = (long long)g.tr * g.tc * (p.M / ((long long)p.R * p.W)), NT = cdiv(p.N, BN), nwg = MT * NT;
  if (nwg > 0x7fffffffLL) return DF_ESHAPE;
  if (nsplit > p.Cin / 64) nsplit = p.Cin / 64;
  if (nsplit > 1 && ((long long)p.M * p.N >= (1LL << 31))) return DF_ESHAPE;
  RcExtra x = {};
  char* scr = scratch_region(p.scr, kScratchCounterBytes + (nsplit > 1 ? (size_t)nsplit * p.M * p.N * sizeof(float) : 0));
  if (!scr) return DF_ENOMEM;
  x.zeros = (const bf16_t*)(scr + kScratchZeroPageOffset);
  x.partials = (float*)(scr + kScratchCounterBytes);
  x.th = g.th; x.tw = g.tw; x.tiles_r = g.tr; x.tiles_c = g.tc;
  x.tw_magic = ((1u << 16) + g.tw - 1) / g.tw;
  x.rw_magic = ((1u << 20) + g.tw + 1) / (g.tw + 2);
  // pixel tiles of a panel: the workgroups an XCD runs at once then cover a square of the output
  const double conc = std::fmin((double)nwg / 8.0, 32.0);
  int gm = (int)(std::sqrt(conc * BN / BM) + 0.5);
  if (gm < 1) gm = 1;
  if (gm > MT) gm = (int)MT;
  x.group_m = cdiv(MT, cdiv(MT, gm));
  constexpr int ring = 2 * NIN * 8192 + ST * TAPS * BN * 128, fin = KG * pass_rows(PM * TM, KG, BN) * 32 * (BN + 4) * 4;
  constexpr int smem = ring > fin ? ring : fin;
  static_assert(smem <= 160 * 1024, "LDS of a compute unit");
  auto k = rconv_kernel<PM, PN, TM, TN, KG, TAPS, ST, NIN, OutT>;
  static bool attr_set = false;
  if (!attr_set) {
    if (hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, smem) != hipSuccess) return DF_EHIP;
    attr_set = true;
  }
  hipLaunchKernelGGL(k, dim3((unsigned)nwg, (unsigned)nsplit), dim3(512), smem, st, p.Wt, p.A, p.N, p.Cin, (int)p.ldw, (int)MT,
                     x.group_m, (int)nsplit, x.tiles_r * x.tiles_c, x.tiles_c, p.R, p.W, p, x);
  DF_LAUNCH_CHECK();
  return nsplit > 1 ? launch_conv_reduce(p, x.partials, nsplit, sizeof(OutT) == 4 ? DF_F32 : DF_BF16, st) : DF_OK;
}

template <int PM, int PN, int TM, int TN, int KG, int TAPS, int ST, int NIN>
int launch_cfg(const TileParams& p, const Geo& g, int out_dtype, int nsplit, hipStream_t st) {
  if (g.th <= 0 || g.th * g.tw > PM * TM * 32 || (g.th + 2) * (g.tw + 2) > NIN * 64) return DF_ESHAPE;   // (the table's row is another tile's)
  return out_dtype == DF_BF16 ? launch_one<PM, PN, TM, TN, KG, TAPS, ST, NIN, bf16_t>(p, g, nsplit, st)
                              : launch_one<PM, PN, TM, TN, KG, TAPS, ST, NIN, float>(p, g, nsplit, st);
}

// Tile shapes with their predicted times: microseconds of a launch, of 64 input channels (nine taps) and of a workgroup's prologue
// and epilogue, times the rounds of workgroups over the chip; fitted to 32 layers (64 to 28800 pixels, 320 to 2560 channels, weights
// that no cache holds) with 1 to 16 parts of the channels each.  Chosen by them, those layers take 0.4 % more than with the best
// of all shapes, and 0.84 of what the tiles of tgemm.hip, which fetch every pixel nine times, took.
struct TileCfg { int bm, bn, nin; double base, slab, fixed; };
constexpr TileCfg kTiles[] = {
    {256, 160, 6, 3.25, 8.115, 3.95},
    {256, 128, 6, 2.70, 5.611, 4.66},
    {256, 64, 6, 2.38, 3.585, 2.91},
    {128, 160, 4, 3.88, 4.594, 4.17},
    {128, 128, 3, 2.64, 3.506, 3.36},
    {128, 64, 3, 1.64, 1.829, 2.85},
    {64, 160, 3, 3.48, 3.270, 4.10},
    {64, 64, 2, 1.30, 1.339, 2.67},
};
// A second kernel adds the parts: microseconds of it, and per output value and part.  Refitted to which tile and parts are best on 64 layers
// after the kernel's last change (by 4.98 and 1.07e-6 layers took too many parts: 24 x 24 pixels x 1280 x 1280 five of 128 x 128, where two of
// 128 x 64 are faster; one patch of 576 tokens at the deepest level, whole step, 9618 -> 9437 us).
constexpr double kSplitUs = 3.25, kPartUs = 1.8e-6;
constexpr int kMaxSplit = 16, kMaxSplitWgs = 640;

}  // namespace

int launch_rconv(const TileParams& p, int out_dtype, hipStream_t st) {
  const long long img = p.M / ((long long)p.R * p.W);
  const int slabs = p.Cin / 64;
  // parts of the channels that the scratch reserved for a layer of this size holds
  const long long room = (long long)((gemm_scratch_bytes(p.M, p.N) - kScratchCounterBytes) / ((size_t)p.M * p.N * sizeof(float)));
  int cfg = -1, ns = 1;
  double best = 1e30;
  Geo g = {}, chosen = {};
  for (int c = 0; c < (int)(sizeof(kTiles) / sizeof(kTiles[0])); ++c) {
    const TileCfg& t = kTiles[c];
    if (c == 0 || t.bm != kTiles[c - 1].bm || t.nin != kTiles[c - 1].nin) g = pick_geo(p.R, p.W, t.bm, t.nin * 64);
    if (g.th <= 0) continue;
    const long long n = (long long)g.tr * g.tc * img * cdiv(p.N, t.bn);
    for (int s = 1; s <= kMaxSplit && s <= slabs; ++s) {
      if (s > 1 && (n * s > kMaxSplitWgs || s > room)) break;
      const double us = t.base + std::ceil(n * s / 256.0) * (cdiv(slabs, s) * t.slab + t.fixed) +
                        (s > 1 ? kSplitUs + kPartUs * s * (double)p.M * p.N : 0.0);
      if (us < best) { best = us; cfg = c; ns = s; chosen = g; }
    }
  }
#ifdef DF_TUNING
  if (tune_env("DF_RC")) {
    cfg = atoi(tune_env("DF_RC"));
    if (cfg >= 0 && cfg < (int)(sizeof(kTiles) / sizeof(kTiles[0]))) chosen = pick_geo(p.R, p.W, kTiles[cfg].bm, kTiles[cfg].nin * 64);
  }
  if (tune_env("DF_RCS")) ns = atoi(tune_env("DF_RCS"));
#endif
  switch (cfg) {
    case 0: return launch_cfg<8, 1, 1, 5, 1, 1, 3, 6>(p, chosen, out_dtype, ns, st);
    case 1: return launch_cfg<4, 2, 2, 2, 1, 1, 3, 6>(p, chosen, out_dtype, ns, st);
    case 2: return launch_cfg<8, 1, 1, 2, 1, 3, 2, 6>(p, chosen, out_dtype, ns, st);
    case 3: return launch_cfg<4, 1, 1, 5, 2, 1, 4, 4>(p, chosen, out_dtype, ns, st);
    case 4: return launch_cfg<4, 2, 1, 2, 1, 1, 4, 3>(p, chosen, out_dtype, ns, st);
    case 5: return launch_cfg<4, 1, 1, 2, 2, 3, 3, 3>(p, chosen, out_dtype, ns, st);
    case 6: return launch_cfg<2, 1, 1, 5, 4, 1, 4, 3>(p, chosen, out_dtype, ns, st);
    case 7: return launch_cfg<2, 1, 1, 2, 4, 3, 3, 2>(p, chosen, out_dtype, ns, st);
    default: return DF_ESHAPE;
  }
}

}  // namespace df
