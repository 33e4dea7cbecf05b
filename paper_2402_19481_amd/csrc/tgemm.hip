#include <cmath>
#include <type_traits>

#include "tile.h"

namespace df {

namespace {

template <int VM>
__device__ __forceinline__ void wait_vm_lds() {   // s_waitcnt vmcnt(VM) lgkmcnt(0)
  __builtin_amdgcn_s_waitcnt((VM & 0xF) | ((VM >> 4) << 14) | (0x7 << 4));
}
// Epilogue of four consecutive columns of one output row: what is added, requested at once, and the rest
struct Added { f32x4 bias, chan, res; };
template <bool kConv>
__device__ __forceinline__ Added added4(const TileParams& p, int row, int col) {
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  Added a = {zero, zero, zero};
  if (p.bias) a.bias = *reinterpret_cast<const f32x4*>(p.bias + col);
  if constexpr (kConv) {
    if (p.chan_add) a.chan = *reinterpret_cast<const f32x4*>(p.chan_add + (long long)(row / (p.Ro * p.Wo)) * p.chan_ld + col);
  }
  if (p.residual) a.res = *reinterpret_cast<const f32x4*>(p.residual + (long long)row * p.ldr + col);
  return a;
}
template <bool kConv, typename OutT>
__device__ __forceinline__ void store4(const TileParams& p, int row, int col, f32x4 v, const Added& add) {
  if (p.bias) v += add.bias;
  if constexpr (kConv) {
    if (p.chan_add) v += add.chan;
  }
  if (p.residual) v += add.res;
  if (p.act == 1) { v.x = silu_f(v.x); v.y = silu_f(v.y); v.z = silu_f(v.z); v.w = silu_f(v.w); }
  OutT* o = reinterpret_cast<OutT*>(p.out) + (long long)row * p.ldo + col;
  if constexpr (sizeof(OutT) == 4) {
    *reinterpret_cast<f32x4*>(o) = v;
  } else {
    const u32x2 t = {pack_bf2(v.x, v.y), pack_bf2(v.z, v.w)};
    *reinterpret_cast<u32x2*>(o) = t;
  }
}

struct TgExtra {
  const bf16_t* zeros;
  float* partials;
  int group_m;
};

// BM x BN output tile per workgroup, (BM/WM) x (BN/WN) waves of WM x WN as 32 x 32 MFMA blocks, KG groups of such waves
// that take alternate 64-wide k-slabs and are added through LDS at the end.  Operands go global -> LDS with direct
// loads (8 rows of 128 B per instruction) into a ring of ST stages of KG slabs.  Rows beyond M / N are clamped to the last
// valid one (never stored); the convolution's zero padding is fetched from a page of zeros.
//   - What bounds it: the direct loads (45 bytes per cycle and compute unit measured with the matrix instructions taken
//     out) and the matrix pipe in about equal parts (128 x 128: 0.35 us of either per slab, 0.46 together; 256 x 128:
//     0.51 and 0.52, 0.77 together); HBM does not (weights cold or resident in L2: the same).
//   - A wave issues its loads in four parts between the matrix instructions: all of them right behind the barrier kept
//     every wave of the unit waiting for the load queue (256 x 128: 0.96 -> 0.77 us per slab).
//   - Waits for LDS reads are exact (see the direct loads in common.h): 4096 pixels x 320 x 320 channels 22.7 -> 21.3 us, 1200 x 640
//     x 640 22.7 -> 20.8, 4096 x 1280 x 1280 142 -> 134.
//   - Weights are the MFMA's row operand, so a lane holds four consecutive output channels of one pixel and the tile is
//     staged through LDS with 16-byte accesses.
//   - What the first requests need are the leading arguments, which come in scalar registers (see wgemm.hip): with attn_pipe_d64's the
//     same way the layer of 1024 of 4096 tokens of 640 features, six launches, 45.8 -> 44.4 us.
template <int BM, int BN, int WM, int WN, int KG, int ST, int OCC, bool kConv, typename OutT>
__global__ __launch_bounds__(64 * (BM / WM) * (BN / WN) * KG, ((BM / WM) * (BN / WN) * KG * OCC + 3) / 4)
void tgemm_kernel(const bf16_t* A, const bf16_t* Wt, int M, int N, int K, int lda, int ldw, int group_m, int nsplit, int packed_w,
                  TileParams p, TgExtra x) {
  constexpr int NWG = (BM / WM) * (BN / WN), NW = NWG * KG, NTHR = 64 * NW;
  constexpr int TM = WM / 32, TN = WN / 32;
  constexpr int AJ = BM / 8 / NWG, BJ = BN / 8 / NWG;     // 1 KB direct loads per wave and slab (its k-group's)
  static_assert(AJ * 8 * NWG == BM && BJ * 8 * NWG == BN, "whole loads");
  constexpr int L = AJ + BJ;
  constexpr int SLAB = (BM + BN) * 128, STAGE = SLAB * KG;
  static_assert(ST > 2 && L * (ST - 1) < 64, "part 3 is requested behind the barrier; the vmcnt field is 6 bits");
  constexpr int LATE = L - (3 * L + 3) / 4;               // loads of part 3
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave / NWG, wq = wave % NWG, wm = wq % (BM / WM), wn = wq / (BM / WM);
  const int MT = (M + BM - 1) / BM, NT = (N + BN - 1) / BN, nwg = MT * NT;
  int t = blockIdx.x;
  {
    const int xcd = t & 7, loc = t >> 3;
    const int base = nwg >> 3, rem = nwg & 7;
    t = xcd * base + (xcd < rem ? xcd : rem) + loc;
  }
  int m0, n0;
  {
    const int per = group_m * NT, pn = t / per, r = t - pn * per, mf = pn * group_m;
    const int gh = MT - mf < group_m ? MT - mf : group_m;
    n0 = r / gh;
    m0 = (mf + r - n0 * gh) * BM;
    n0 *= BN;
  }
  const int split = blockIdx.y;
  const int slabs_all = K / 64;
  const int stages_all = (slabs_all + KG - 1) / KG;
  const int per_split = (stages_all + nsplit - 1) / nsplit;
  const int s_lo = split * per_split * KG;                               // first slab of the split
  int s_hi = s_lo + per_split * KG;
  if (s_hi > slabs_all) s_hi = slabs_all;
  const int KT = (s_hi - s_lo + KG - 1) / KG;

  // direct loads: instruction j of a wave covers tile rows (wq*AJ + j)*8 + lane/8, LDS slot lane%8 of the row; row r keeps
  // its 16-byte chunk c at slot c ^ ((r >> 1) & 7)
  const int lr = lane >> 3;
  const bf16_t* a_base[AJ];                                              // convolution: channel 0 of the centre pixel
  const char* const a_tile = (const char*)(A + (long long)m0 * (kConv ? 0 : lda));   // linear layer: the tile's first row,
  unsigned int a_ofs[AJ];                                                // and the lane's bytes from there (launcher: below 2^31)
  int a_r[AJ], a_c[AJ], a_b[AJ];
#pragma unroll
  for (int j = 0; j < AJ; ++j) {
    const int row = (wq * AJ + j) * 8 + lr;
    int m = m0 + row;
    if (m >= M) m = M - 1;                                           // ragged last tile: re-read, never stored
    const int ch = ((lane & 7) ^ ((row >> 1) & 7)) * 8;
    if constexpr (kConv) {
      const int per = p.Ro * p.Wo;
      a_b[j] = m / per;
      const int rem = m - a_b[j] * per;
      a_r[j] = rem / p.Wo;
      a_c[j] = (rem - a_r[j] * p.Wo) * p.stride;
      a_r[j] *= p.stride;
      a_base[j] = A + (((long long)a_b[j] * p.R + a_r[j]) * p.W + a_c[j]) * p.Cin + ch;
      a_ofs[j] = 0;
    } else {
      a_base[j] = nullptr;
      a_b[j] = a_r[j] = a_c[j] = 0;
      a_ofs[j] = 2u * ((unsigned int)(m - m0) * (unsigned int)lda + (unsigned int)ch);
    }
  }
  const bool tiled = !kConv && packed_w;                              // (see tile.h)
  const char* const b_tile = (const char*)(Wt + w_tile_base(tiled, n0, slabs_all, ldw));
  unsigned int b_ofs[BJ];
#pragma unroll
  for (int j = 0; j < BJ; ++j) b_ofs[j] = w_lane_bytes(tiled, n0, (wq * BJ + j) * 8 + lr, lane & 7, N, slabs_all, ldw);
  const unsigned int b_step = w_slab_bytes(tiled);
  // Convolution: a lane's source pixel changes only with the filter tap, every Cin / 64 slabs
  const bf16_t* a_tap[AJ];
  bool a_pad[AJ];
  int tap_k0 = 0, tap_end = 0;                                           // k range of the tap the pointers are set for
  auto set_tap = [&](int k0) {
    const int tap = k0 / p.Cin;
    tap_k0 = tap * p.Cin;
    tap_end = tap_k0 + p.Cin;
    const int dy = tap / 3 - 1, dx = tap - (tap / 3) * 3 - 1;
    const long long off = ((long long)dy * p.W + dx) * p.Cin;
#pragma unroll
    for (int j = 0; j < AJ; ++j) {
      const int ri = a_r[j] + dy, ci = a_c[j] + dx;
      a_tap[j] = a_base[j] + off;
      a_pad[j] = false;
      if ((unsigned)ri >= (unsigned)p.R || (unsigned)ci >= (unsigned)p.W) {
        const bf16_t* src = conv_tap_src(A, p.top, p.bot, p.halo_bs, p.left, p.right, p.side_bs, p.side_rs, a_b[j], ri,
                                         ci, p.R, p.W, p.Cin);
        const int row = (wq * AJ + j) * 8 + lr;
        a_pad[j] = src == nullptr;
        a_tap[j] = (src ? src : x.zeros) + ((lane & 7) ^ ((row >> 1) & 7)) * 8;
      }
    }
  };
  // part STEP of 4 of a stage's loads (one part per 16 of K of the loop below: a wave that issues them all at once waits
  // for the queue of the load path, and every wave of the unit with it)
  auto issue = [&](int kt, int slot, auto stepc) {
    constexpr int STEP = decltype(stepc)::value;
    int slab = s_lo + kt * KG + kg;
    if (slab > slabs_all - 1) slab = slabs_all - 1;                      // a group's missing last slab: loaded, not used
    const int k0 = slab * 64;
    char* sa = smem + slot * STAGE + kg * SLAB + wq * AJ * 1024;
    char* sb = smem + slot * STAGE + kg * SLAB + BM * 128 + wq * BJ * 1024;
    if constexpr (kConv && STEP == 0) {
      if (k0 >= tap_end || k0 < tap_k0) set_tap(k0);                     // (uniform)
    }
#pragma unroll
    for (int q = 0; q < L; ++q) {
      if (q * 4 / L != STEP) continue;
      const int j = q < AJ ? q : q - AJ;
      if (q < AJ) {
        if constexpr (kConv) {
          lds_load16(a_pad[j < AJ ? j : 0] ? a_tap[j < AJ ? j : 0] : a_tap[j < AJ ? j : 0] + (k0 - tap_k0), sa + j * 1024);
        } else {
          lds_load_buf(a_tile, a_ofs[j < AJ ? j : 0], (unsigned int)k0 * 2u, sa + j * 1024);
        }
      } else {
        lds_load_buf(b_tile, b_ofs[j < BJ ? j : 0], (unsigned int)slab * b_step, sb + j * 1024);
      }
    }
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
  const int lrow = lane & 31, g = lane >> 5, sw = (lrow >> 1) & 7;
  bf16x8 xa[2][TM], wa[2][TN];
  auto rd = [&](int slot, int ks, auto bc) {
    constexpr int b = decltype(bc)::value;
    const char* s = smem + slot * STAGE + kg * SLAB + lrow * 128 + ((2 * ks + g) ^ sw) * 16;
#pragma unroll
    for (int i = 0; i < TM; ++i) xa[b][i] = *reinterpret_cast<const bf16x8*>(s + (wm * WM + i * 32) * 128);
#pragma unroll
    for (int j = 0; j < TN; ++j) wa[b][j] = *reinterpret_cast<const bf16x8*>(s + (BM + wn * WN + j * 32) * 128);
  };
  auto mm = [&](auto bc) {
    constexpr int b = decltype(bc)::value;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa[b][j], xa[b][i], acc[i][j], 0, 0, 0);
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
#define DF_SB __builtin_amdgcn_sched_barrier(0)
  using I2 = std::integral_constant<int, 2>;
  using I3 = std::integral_constant<int, 3>;
#pragma unroll
  for (int s = 0; s < ST - 1; ++s) {
    const int k = s < KT ? s : KT - 1;                                   // past the end: the last stage again (vmcnt stays uniform)
    issue(k, s, I0{}); issue(k, s, I1{}); issue(k, s, I2{}); issue(k, s, I3{});
  }
  // the epilogue's arguments (cold in every launch) come beside the first operands
  asm volatile("" ::"s"(p.bias), "s"(p.chan_add), "s"(p.chan_ld), "s"(p.residual), "s"(p.ldr), "s"(p.out), "s"(p.ldo), "s"(p.act), "s"(x.partials));
  wait_vm_lds<L * (ST - 2)>();
  block_sync();
  rd(0, 0, I0{});
  int slot = 0, pslot = ST - 1, kt = 0;
  auto has_slab = [&] { return KG == 1 || s_lo + kt * KG + kg < s_hi; };   // (uniform) the group has a slab in stage kt
  for (; kt + ST - 1 < KT; ++kt) {
    const int nslot = slot + 1 == ST ? 0 : slot + 1, kn = kt + ST - 1;
    const bool mine = has_slab();
    DF_SB; rd(slot, 1, I1{}); DF_SB; if (mine) mm(I0{}); DF_SB; issue(kn, pslot, I0{});
    DF_SB; rd(slot, 2, I0{}); DF_SB; if (mine) mm(I1{}); DF_SB; issue(kn, pslot, I1{});
    DF_SB; rd(slot, 3, I1{}); DF_SB; if (mine) mm(I0{}); DF_SB; issue(kn, pslot, I2{});
    wait_vm_lds<L * (ST - 2) - LATE>();
    block_sync();
    rd(nslot, 0, I0{});
    DF_SB; if (mine) mm(I1{}); DF_SB; issue(kn, pslot, I3{});
    pslot = slot;
    slot = nslot;
  }
  // the last ST - 1 stages have been requested (as in bgemm.hip)
  auto last = [&](auto uc) {                                             // stage kt, uc stages into the tail: false behind the last one
    constexpr int U = decltype(uc)::value;
    const int nslot = slot + 1 == ST ? 0 : slot + 1;
    const bool mine = has_slab(), more = U < ST - 2 && kt + 1 < KT;
    DF_SB; rd(slot, 1, I1{}); DF_SB; if (mine) mm(I0{}); DF_SB;
    rd(slot, 2, I0{}); DF_SB; if (mine) mm(I1{}); DF_SB;
    rd(slot, 3, I1{}); DF_SB; if (mine) mm(I0{}); DF_SB;
    if (more) {
      wait_vm_lds<U < ST - 2 ? L * (ST - 3 - U) : 0>();                  // (stages of a short K that were requested twice count too)
      block_sync();
      rd(nslot, 0, I0{});
    }
    DF_SB; if (mine) mm(I1{}); DF_SB;
    slot = nslot;
    ++kt;
    return more;
  };
  static_assert(ST == 3 || ST == 4, "");
  if (last(I0{}))
    if (last(I1{}))
      if constexpr (ST == 4) last(I2{});
  if (KT < ST - 1) wait_vm_lds<0>();                                     // the ring becomes the epilogue's
#undef DF_SB

  // ---- epilogue: accumulators -> LDS (the ring is free), k-groups added, whole rows stored ----
  constexpr int PT = BN + 4;
  float* tile = reinterpret_cast<float*>(smem);
  block_sync();
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<f32x4*>(tile + (kg * BM + wm * WM + i * 32 + lrow) * PT + wn * WN + j * 32 + 8 * q + 4 * g) =
            f32x4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
  __syncthreads();
  // (four rows' additions requested together: one by one each waited for the one before it)
  constexpr int ITEMS = BM * (BN / 4) / NTHR, U = ITEMS % 4 == 0 ? 4 : ITEMS % 2 == 0 ? 2 : 1;
  static_assert(ITEMS * NTHR == BM * (BN / 4), "");
#pragma unroll 1
  for (int i0 = 0; i0 < ITEMS; i0 += U) {
    Added add[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int idx = tid + (i0 + k) * NTHR, row = m0 + idx / (BN / 4), col = n0 + (idx % (BN / 4)) * 4;
      add[k] = nsplit > 1 || row >= M || col >= N ? Added{} : added4<kConv>(p, row, col);
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int idx = tid + (i0 + k) * NTHR, r = idx / (BN / 4), c4 = (idx % (BN / 4)) * 4;
      const int row = m0 + r, col = n0 + c4;
      if (row >= M || col >= N) continue;
      f32x4 v = *reinterpret_cast<const f32x4*>(tile + r * PT + c4);
#pragma unroll
      for (int h = 1; h < KG; ++h) v += *reinterpret_cast<const f32x4*>(tile + (h * BM + r) * PT + c4);
      if (nsplit > 1) *reinterpret_cast<f32x4*>(x.partials + ((size_t)split * M + row) * N + col) = v;
      else store4<kConv, OutT>(p, row, col, v, add[k]);
    }
  }
}

// Sum over the splits, in split order, then the epilogue; four columns per lane.  NS of them are requested together with what the
// epilogue adds: in a loop over the splits each load waited for the one before it (64 x 1280, five splits: 6.4 -> 4.6 us, of which
// a launch and two round trips to memory are some 4).
template <int NS, bool kConv, typename OutT>
__global__ __launch_bounds__(256) void tgemm_reduce_kernel(TileParams p, const float* __restrict__ partials, int nsplit) {
  // (every argument requested in one batch, see wgemm.hip)
  asm volatile("" ::"s"(partials), "s"(nsplit), "s"(p.M), "s"(p.N), "s"(p.bias), "s"(p.residual), "s"(p.ldr), "s"(p.chan_add), "s"(p.chan_ld),
               "s"(p.Ro), "s"(p.Wo), "s"(p.out), "s"(p.ldo), "s"(p.act));
  const unsigned int idx = blockIdx.x * 256 + threadIdx.x;               // M * N / 4 < 2^31 (launcher)
  const unsigned int n4 = (unsigned int)p.N / 4;
  if (idx >= (unsigned int)p.M * n4) return;
  const int row = (int)(idx / n4), col = (int)(idx - (unsigned int)row * n4) * 4;
  const float* src = partials + (size_t)row * p.N + col;
  const size_t pitch = (size_t)p.M * p.N;
  const Added add = added4<kConv>(p, row, col);
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < nsplit; s0 += NS) {                              // (one round up to eight splits)
    f32x4 t[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) t[s] = *reinterpret_cast<const f32x4*>(src + (s0 + s < nsplit ? s0 + s : nsplit - 1) * pitch);
#pragma unroll
    for (int s = 0; s < NS; ++s)
      if (s0 + s < nsplit) v += t[s];
  }
  store4<kConv, OutT>(p, row, col, v, add);
}

template <bool kConv, typename OutT>
void launch_reduce(const TileParams& p, const float* partials, int nsplit, hipStream_t st) {
  const long long n = (long long)p.M * (p.N / 4);
  const dim3 grid((unsigned)((n + 255) / 256));
  switch (nsplit) {
#define DF_RED(NS) hipLaunchKernelGGL((tgemm_reduce_kernel<NS, kConv, OutT>), grid, dim3(256), 0, st, p, partials, nsplit); break
    case 2: DF_RED(2);
    case 3: DF_RED(3);
    case 4: DF_RED(4);
    case 5: DF_RED(5);
    case 6: DF_RED(6);
    default: DF_RED(8);
#undef DF_RED
  }
}

template <int BM, int BN, int WM, int WN, int KG, int ST, int OCC, bool kConv, typename OutT>
int launch_one(const TileParams& p, int nsplit, hipStream_t st) {
  constexpr int NW = (BM / WM) * (BN / WN) * KG;
  const int MT = cdiv(p.M, BM), NT = cdiv(p.N, BN), stages = cdiv(p.K / 64, KG);
  const long long nwg = (long long)MT * NT;
  if (nwg > 0x7fffffffLL) return DF_ESHAPE;
  if (nsplit > stages) nsplit = stages;
  if (nsplit < 1) nsplit = 1;
  nsplit = cdiv(stages, cdiv(stages, nsplit));                           // no empty split
  if (nsplit > 1 && ((long long)p.M * p.N >= (1LL << 31))) return DF_ESHAPE;
  TgExtra x = {};
  if (kConv || nsplit > 1) {
    char* scr = scratch_region(p.scr, kScratchCounterBytes + (nsplit > 1 ? (size_t)nsplit * p.M * p.N * sizeof(float) : 0));
    if (!scr) return DF_ENOMEM;
    x.zeros = (const bf16_t*)(scr + kScratchZeroPageOffset);
    x.partials = (float*)(scr + kScratchCounterBytes);
  }
  // token tiles of a panel: the workgroups an XCD runs at once then cover a square of the output
  const double conc = std::fmin((double)nwg / 8.0, 32.0 * OCC);
  int gm = (int)(std::sqrt(conc * BN / BM) + 0.5);
  if (gm < 1) gm = 1;
  if (gm > MT) gm = MT;
  x.group_m = cdiv(MT, cdiv(MT, gm));
  constexpr int ring = ST * (BM + BN) * 128 * KG, fin = KG * BM * (BN + 4) * 4;
  constexpr int smem = ring > fin ? ring : fin;
  static_assert(smem * OCC <= 160 * 1024, "LDS of a compute unit");
  auto k = tgemm_kernel<BM, BN, WM, WN, KG, ST, OCC, kConv, OutT>;
  static bool attr_set = false;
  if (!attr_set) {
    if (hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, smem) != hipSuccess) return DF_EHIP;
    attr_set = true;
  }
  hipLaunchKernelGGL(k, dim3((unsigned)nwg, (unsigned)nsplit), dim3(64 * NW), smem, st, p.A, p.Wt, p.M, p.N, p.K, (int)p.lda, (int)p.ldw,
                     x.group_m, (int)nsplit, p.packed_w, p, x);
  DF_LAUNCH_CHECK();
  if (nsplit > 1) {
    launch_reduce<kConv, OutT>(p, x.partials, nsplit, st);
    DF_LAUNCH_CHECK();
  }
  return DF_OK;
}

template <int BM, int BN, int WM, int WN, int KG, int ST, int OCC>
int launch_cfg(const TileParams& p, bool conv, int out_dtype, int nsplit, hipStream_t st) {
  if (conv) return out_dtype == DF_BF16 ? launch_one<BM, BN, WM, WN, KG, ST, OCC, true, bf16_t>(p, nsplit, st)
                                        : launch_one<BM, BN, WM, WN, KG, ST, OCC, true, float>(p, nsplit, st);
  return out_dtype == DF_BF16 ? launch_one<BM, BN, WM, WN, KG, ST, OCC, false, bf16_t>(p, nsplit, st)
                              : launch_one<BM, BN, WM, WN, KG, ST, OCC, false, float>(p, nsplit, st);
}

// Tile shapes with their predicted times: microseconds of a launch, of a stage (KG slabs) and of a workgroup's prologue and
// epilogue.  They come from 28 convolutions, most of which are rconv.hip's now, and 11 linear layers with the loads of then; what still
// holds is which tile they choose, not the times (0.4 to 1.1 of a launch with nothing in a cache).  Measured so with the present
// loads, the chosen tile and parts against the best of these six in 1 to 16 parts: 54 linear layers (256 to 38400 tokens, 320 to
// 1920 features, K 320 to 5120) take 1.8 % more in the mean, 14 % at worst (2400 x 1920 x 640: 16.5 us, 14.4 on 256 x 128), nine
// convolutions of stride 2 0.9 %.
struct TileCfg { int bm, bn, kg, occ; double base, stage, fixed; };
constexpr TileCfg kTiles[] = {
    {128, 128, 1, 1, 2.96, 0.518, 1.99},
    {128, 64, 1, 2, 3.56, 0.708, 0.0},     // two workgroups per unit
    {64, 64, 2, 1, 2.03, 0.532, 1.42},
    {64, 128, 2, 1, 2.63, 0.789, 1.32},
    {128, 160, 1, 1, 4.56, 0.641, 2.59},   // channel counts are multiples of 320
    {256, 128, 1, 1, 3.48, 0.774, 2.48},   // sixteen waves
};
constexpr int kNumTiles = (int)(sizeof(kTiles) / sizeof(kTiles[0]));
// Parts of K: at least four slabs each, at most as many as the chip takes workgroups at once with some to spare
constexpr int kMaxSplit = 16, kMaxSplitWgs = 640;

long long tiles_of(const TileCfg& t, long long M, long long N) { return ((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn); }

}  // namespace

// bytes of library scratch a launch may ask for (plans reserve it up front); also covers a convolution with M output
// pixels, N = Cout
size_t gemm_scratch_bytes(long long M, long long N) {
  long long ns = 0;
  for (const TileCfg& t : kTiles) {
    long long n = kMaxSplitWgs / tiles_of(t, M, N);
    if (n > kMaxSplit) n = kMaxSplit;
    if (n > ns) ns = n;
  }
  return kScratchCounterBytes + (size_t)(ns > 1 ? ns * M * N * (long long)sizeof(float) : 0);
}

int launch_conv_reduce(const TileParams& p, const float* partials, int nsplit, int out_dtype, hipStream_t st) {
  if (out_dtype == DF_BF16) launch_reduce<true, bf16_t>(p, partials, nsplit, st);
  else launch_reduce<true, float>(p, partials, nsplit, st);
  DF_LAUNCH_CHECK();
  return DF_OK;
}

int launch_tgemm(const TileParams& p, bool conv, int out_dtype, hipStream_t st) {
  auto al = [](const void* ptr, int a) { return ((uintptr_t)ptr % a) == 0; };
  const bool ok = p.K % 64 == 0 && (!conv || p.Cin % 64 == 0) && p.N % 4 == 0 && p.ldo % 4 == 0 && al(p.out, 16) && al(p.bias, 16) &&
                  al(p.chan_add, 16) && p.chan_ld % 4 == 0 && (!p.residual || (p.ldr % 4 == 0 && al(p.residual, 16)));
  if (!ok || p.ldw >= (1 << 22) || (!conv && p.lda >= (1 << 22)) || p.K >= (1 << 22)) return DF_ESHAPE;   // 32-bit offsets inside a tile
  // (the tiles below serve linear layers and the convolutions of stride 2, where a pixel is used by a quarter of the taps)
#ifdef DF_TUNING
  const bool tap_wise = tune_env("DF_TG") != nullptr;
#else
  const bool tap_wise = false;
#endif
  if (conv && p.stride == 1 && !tap_wise) return launch_rconv(p, out_dtype, st);
  const int slabs = p.K / 64;
  int cfg = 0, ns = 1;
  double best = 1e30;
  for (int c = 0; c < kNumTiles; ++c) {
    const TileCfg& t = kTiles[c];
    const long long n = tiles_of(t, p.M, p.N);
    for (int s = 1; s <= kMaxSplit; ++s) {
      if (s > 1 && (n * s > kMaxSplitWgs || slabs / s < 4)) break;
      const int stages = cdiv(cdiv(slabs, t.kg), s);
      const double wgs = (double)n * s;
      // rounds of workgroups; two of a unit share it, and one alone is faster
      const double r = t.occ == 1 ? std::ceil(wgs / 256.0) : wgs <= 256.0 ? 0.6 : wgs > 1024.0 ? wgs / 512.0 : std::ceil(wgs / 512.0);
      const double us = t.base + r * (stages * t.stage + (conv ? t.fixed : 0.0)) +
                        (s > 1 ? 3.97 + 1.46e-6 * s * (double)p.M * p.N : 0.0);   // the partials and the kernel that adds them
      if (us < best) { best = us; cfg = c; ns = s; }
    }
  }
#ifdef DF_TUNING
  if (tune_env("DF_TG")) cfg = atoi(tune_env("DF_TG"));
  if (tune_env("DF_TGS")) ns = atoi(tune_env("DF_TGS"));
#endif
  switch (cfg) {
    case 0: return launch_cfg<128, 128, 32, 64, 1, 4, 1>(p, conv, out_dtype, ns, st);
    case 1: return launch_cfg<128, 64, 32, 32, 1, 3, 2>(p, conv, out_dtype, ns, st);
    case 2: return launch_cfg<64, 64, 32, 32, 2, 4, 1>(p, conv, out_dtype, ns, st);
    case 3: return launch_cfg<64, 128, 32, 64, 2, 3, 1>(p, conv, out_dtype, ns, st);
    case 4: return launch_cfg<128, 160, 32, 160, 1, 4, 1>(p, conv, out_dtype, ns, st);
    case 5: return launch_cfg<256, 128, 64, 32, 1, 3, 1>(p, conv, out_dtype, ns, st);
    default: return DF_ESHAPE;
  }
}

}  // namespace df
