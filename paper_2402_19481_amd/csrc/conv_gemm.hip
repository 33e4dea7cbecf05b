// bf16 MFMA tile kernel shared by the linear layers and the 3x3 convolution,
// plus the direct convolution kernels for shapes that are not worth a tile.
//
// Sparse convolution of one patch (Section 4, Sparse operations): an implicit
// GEMM over M = B*Ro*Wo output pixels of the patch, N = Cout, K = 9*Cin.  The
// A-operand loader gathers each 32- or 64-channel slice of a tap straight from the
// fresh patch, or - for the row above / below the patch - from the stale halo
// row (Section 5.3: only boundary rows come from other patches), or zero at the
// image border.  The scatter is never materialised.  Patches that are vertical
// strips take the column left / right of the patch from the stale buffer in the
// same way (one pixel per input row, strided).
//
// Two tile kernels: mfma_pipe_kernel (BM x BN x 64 slabs, operands loaded
// global -> LDS directly into a multi-stage ring, used whenever K % 64 == 0)
// and mfma_tile_kernel (BM x BN x 32, register-staged, any K % 32 == 0).  Both
// run 4 compute waves in a 2x2 grid, each owning (BM/2)x(BN/2) as 32x32 blocks
// of v_mfma_f32_32x32x16_bf16.
#include <cstdio>
#include <cstdlib>
#include <type_traits>

#include "kernels.h"

namespace df {

namespace {

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;

constexpr int BK = 32;
constexpr int LDS_PITCH = 40;  // bf16 elements per LDS row: 32 + 8 pad

struct TileParams {
  // GEMM view
  const bf16_t* A;
  const bf16_t* Wt;
  const float* bias;
  const float* residual;
  const float* chan_add;
  long long chan_ld;
  void* out;
  int M, N, K;
  long long lda, ldw, ldr, ldo;
  int act;
  // convolution geometry (kConv only)
  const bf16_t* top;
  const bf16_t* bot;
  long long halo_bs;
  const bf16_t* left;    // stale column left / right of a vertical strip: pixel (b, row) at left + b*side_bs + row*side_rs
  const bf16_t* right;
  long long side_bs, side_rs;
  int R, W, Cin, Ro, Wo, stride;
  // epilogue variants of the pipelined kernel (see GemmArgs)
  int geglu;      // F (half of N) or 0
  int nseg, seg_w;
  void* seg_out[3];
  long long seg_ld[3], seg_rows_out[3], seg_row0[3];
  int seg_rows_in[3];
  int seg_tr[3];
  int seg_pin[3], seg_pout[3];
  int packed_w;
  const float* ln_s;
  const float* ln_t;
  float ln_eps;
  bf16_t* out2;
  long long ldo2;
  int vec_epi;    // every epilogue pointer / stride allows 16-byte (float) and 8-byte (bf16) accesses
  const Scratch* scr;   // host side only: where split-K partials and the page of zeros live
};

// Source pixel (channel 0) of one filter tap: the fresh patch, a stale halo row (patches are horizontal strips) or
// halo column (vertical strips), or nullptr where the tap falls on the zero padding around the image.
template <typename T>
__device__ __forceinline__ const T* conv_tap_src(const T* x, const T* top, const T* bot, long long halo_bs, const T* left,
                                                 const T* right, long long side_bs, long long side_rs, int b, int ri,
                                                 int ci, int R, int W, int Cin) {
  if (ci < 0 || ci >= W) {
    const T* side = ci < 0 ? left : right;
    if (!side || ri < 0 || ri >= R) return nullptr;
    return side + b * side_bs + ri * side_rs;
  }
  if (ri < 0) return top ? top + b * halo_bs + (long long)ci * Cin : nullptr;
  if (ri >= R) return bot ? bot + b * halo_bs + (long long)ci * Cin : nullptr;
  return x + (((long long)b * R + ri) * W + ci) * Cin;
}

template <int BM, int BN, bool kConv, typename OutT>
__global__ __launch_bounds__(256) void mfma_tile_kernel(TileParams p) {
  constexpr int TM = BM / 64, TN = BN / 64;      // 32x32 blocks per wave in each direction
  constexpr int A_CH = BM * 4 / 256, B_CH = BN * 4 / 256;  // 16-byte chunks per lane per tile
  __shared__ __attribute__((aligned(16))) bf16_t As[2][BM * LDS_PITCH];
  __shared__ __attribute__((aligned(16))) bf16_t Bs[2][BN * LDS_PITCH];

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
  const int KT = p.K / BK;

  // ---- per-lane source description of its A and B chunks ----
  int a_row[A_CH], a_kc[A_CH];
  long long a_off[A_CH];          // GEMM: element offset of (row, kc*8); conv: unused
  int a_b[A_CH], a_ro[A_CH], a_co[A_CH];
  bool a_ok[A_CH];
#pragma unroll
  for (int i = 0; i < A_CH; ++i) {
    const int q = tid + i * 256;
    a_row[i] = q >> 2;
    a_kc[i] = q & 3;
    const int m = m0 + a_row[i];
    a_ok[i] = m < p.M;
    if constexpr (kConv) {
      const int per = p.Ro * p.Wo;
      const int mm = a_ok[i] ? m : 0;
      a_b[i] = mm / per;
      const int rem = mm - a_b[i] * per;
      a_ro[i] = rem / p.Wo;
      a_co[i] = rem - a_ro[i] * p.Wo;
      a_off[i] = 0;
    } else {
      a_off[i] = (long long)m * p.lda + a_kc[i] * 8;
      a_b[i] = a_ro[i] = a_co[i] = 0;
    }
  }
  long long b_off[B_CH];
  bool b_ok[B_CH];
  int b_row[B_CH], b_kc[B_CH];
#pragma unroll
  for (int i = 0; i < B_CH; ++i) {
    const int q = tid + i * 256;
    b_row[i] = q >> 2;
    b_kc[i] = q & 3;
    const int n = n0 + b_row[i];
    b_ok[i] = n < p.N;
    b_off[i] = (long long)n * p.ldw + b_kc[i] * 8;
  }

  u32x4 a_reg[A_CH], b_reg[B_CH];
  const u32x4 zero4 = {0u, 0u, 0u, 0u};

  auto load_tile = [&](int kt) {
    const int k0 = kt * BK;
    if constexpr (kConv) {
      const int tap = k0 / p.Cin;
      const int cin0 = k0 - tap * p.Cin;
      const int ky = tap / 3, kx = tap - ky * 3;
#pragma unroll
      for (int i = 0; i < A_CH; ++i) {
        const int ri = a_ro[i] * p.stride + ky - 1;
        const int ci = a_co[i] * p.stride + kx - 1;
        const bf16_t* src = a_ok[i] ? conv_tap_src(p.A, p.top, p.bot, p.halo_bs, p.left, p.right, p.side_bs, p.side_rs,
                                                   a_b[i], ri, ci, p.R, p.W, p.Cin)
                                    : nullptr;
        a_reg[i] = src ? *reinterpret_cast<const u32x4*>(src + cin0 + a_kc[i] * 8) : zero4;
      }
    } else {
#pragma unroll
      for (int i = 0; i < A_CH; ++i)
        a_reg[i] = a_ok[i] ? *reinterpret_cast<const u32x4*>(p.A + a_off[i] + k0) : zero4;
    }
#pragma unroll
    for (int i = 0; i < B_CH; ++i)
      b_reg[i] = b_ok[i] ? *reinterpret_cast<const u32x4*>(p.Wt + b_off[i] + k0) : zero4;
  };
  auto store_tile = [&](int buf) {
#pragma unroll
    for (int i = 0; i < A_CH; ++i)
      *reinterpret_cast<u32x4*>(&As[buf][a_row[i] * LDS_PITCH + a_kc[i] * 8]) = a_reg[i];
#pragma unroll
    for (int i = 0; i < B_CH; ++i)
      *reinterpret_cast<u32x4*>(&Bs[buf][b_row[i] * LDS_PITCH + b_kc[i] * 8]) = b_reg[i];
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  load_tile(0);
  store_tile(0);
  __syncthreads();
  const int lrow = lane & 31, lk = (lane >> 5) * 8;
  for (int kt = 0; kt < KT; ++kt) {
    const int buf = kt & 1;
    if (kt + 1 < KT) load_tile(kt + 1);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      bf16x8 af[TM], bfr[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i)
        af[i] = *reinterpret_cast<const bf16x8*>(&As[buf][(wm * (BM / 2) + i * 32 + lrow) * LDS_PITCH + ks * 16 + lk]);
#pragma unroll
      for (int j = 0; j < TN; ++j)
        bfr[j] = *reinterpret_cast<const bf16x8*>(&Bs[buf][(wn * (BN / 2) + j * 32 + lrow) * LDS_PITCH + ks * 16 + lk]);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
    }
    if (kt + 1 < KT) store_tile(buf ^ 1);
    __syncthreads();
  }

  // ---- epilogue: accumulator element 4*j+r of a 32x32 block sits at row 8*j + 4*(lane/32) + r, column lane%32 ----
  OutT* out = reinterpret_cast<OutT*>(p.out);
  const int per = kConv ? p.Ro * p.Wo : 1;
#pragma unroll
  for (int tn = 0; tn < TN; ++tn) {
    const int col = n0 + wn * (BN / 2) + tn * 32 + (lane & 31);
    if (col >= p.N) continue;
    const float bias = p.bias ? p.bias[col] : 0.f;
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int row = m0 + wm * (BM / 2) + tm * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3);
        if (row >= p.M) continue;
        float v = acc[tm][tn][e] + bias;
        if constexpr (kConv) {
          if (p.chan_add) v += p.chan_add[(long long)(row / per) * p.chan_ld + col];
        }
        if (p.residual) v += p.residual[(long long)row * p.ldr + col];
        if (p.act == 1) v = silu_f(v);
        Elem<OutT>::st(out + (long long)row * p.ldo + col, v);
      }
    }
  }
}


// ---- pipelined variant: global -> LDS direct loads (global_load_lds_dwordx4), multi-stage ring ----
//
// BM x BN x 64 tiles.  Every wave instruction moves 64 lanes x 16 B = 8 tile rows of 128 B straight
// into LDS (no registers), so several k-tiles of loads are in flight per workgroup; the oldest stage
// is awaited with an explicit vmcnt.  A direct load writes lane l at LDS offset 16*l, so the tile is
// row-major unpadded; bank conflicts are avoided by fetching, for LDS slot s of row r, the global
// 16-byte chunk s ^ ((r >> 1) & 7), and reading the MFMA operand for chunk c at slot c ^ ((r >> 1) & 7).
// Rows beyond M / N are clamped to the last valid row (never stored); zero padding of the
// convolution is fetched from a page of zeros.
#define DF_GPTR(p) ((const __attribute__((address_space(1))) void*)(p))
#define DF_LPTR(p) ((__attribute__((address_space(3))) void*)(p))

#ifdef DF_TUNING
// Tuning build only: cycle stamps of workgroup 0 / wave 0 at four points of every k-slab iteration.
__device__ long long g_pipe_trace[4 * 512 + 8];
#define DF_TRACE(slot)                                                                           \
  do {                                                                                           \
    if (blockIdx.x == 0 && blockIdx.y == 0 && wave == 0 && lane == 0 && (slot) < 4 * 512 + 8)    \
      g_pipe_trace[(slot)] = (long long)__builtin_readcyclecounter();                            \
  } while (0)
#else
#define DF_TRACE(slot) do {} while (0)
#endif

template <int VM>
__device__ __forceinline__ void wait_vm_and_lds() {
  // s_waitcnt vmcnt(VM) lgkmcnt(0): gfx9 encoding vmcnt[3:0]=imm[3:0], vmcnt[5:4]=imm[15:14], expcnt=imm[6:4], lgkmcnt=imm[11:8]
  __builtin_amdgcn_s_waitcnt((VM & 0xF) | ((VM >> 4) << 14) | (0x7 << 4));
}

// Split-K (gridDim.y > 1): every split accumulates a contiguous range of k-tiles and stores its float
// partial; splitk_reduce_kernel adds the partials in split order and runs the epilogue.
// KS = 64-wide k-slabs per ring stage: with two, the barrier and the first LDS round trip of an iteration are paid
// once per 128 of K, which is what bounds the short K loops of the patch-sized GEMMs.
// NW = waves per workgroup (4 or 8).  The first four compute; with eight, the other four only issue their share of the
// direct loads: measured fetch throughput of a compute unit is bounded per wave, so problems that put a single
// workgroup on a unit (the ~100-tile GEMMs of the patch step) stream their operands twice as fast with twice the waves.
template <int BM, int BN, int STAGES, bool kConv, typename OutT, int KS, int NW>
__global__ __launch_bounds__(64 * NW) void mfma_pipe_kernel(TileParams p, const bf16_t* __restrict__ zeros,
                                                            float* __restrict__ partials) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  constexpr int TM = BM / 64, TN = BN / 64;
  constexpr int A_BYTES = BM * 128, B_BYTES = BN * 128, SLAB = A_BYTES + B_BYTES, STAGE = SLAB * KS;
  constexpr int NTHR = 64 * NW;
  constexpr int AJ = BM / (8 * NW), BJ = BN / (8 * NW);   // direct-load instructions per wave per k-slab
  static_assert(AJ >= 1 && BJ >= 1, "every wave issues at least one load per operand");
  constexpr int L = (AJ + BJ) * KS;
  static_assert(KS == 1, "one k-slab per ring stage");
  static_assert((STAGES - 1) * L < 64, "vmcnt field is 6 bits");

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // scalar: LDS bases and the compute / load-only split
  const int wm = (wave >> 1) & 1, wn = wave & 1;
  const bool computes = wave < 4;
  // workgroups round-robin over the 8 XCDs; give each XCD a contiguous run of tiles, M-tile fastest, so that the
  // workgroups sharing a weight tile sit behind the same L2
  const int MT = (p.M + BM - 1) / BM, NT = (p.N + BN - 1) / BN;
  const int nwg = MT * NT;
  int t = blockIdx.x;
  {
    // XCD x (= workgroup id mod 8) receives the x-th contiguous chunk of tiles; chunk sizes differ by at most one
    const int xcd = t & 7, loc = t >> 3;
    const int base = nwg >> 3, rem = nwg & 7;
    t = xcd * base + (xcd < rem ? xcd : rem) + loc;
  }
  // consecutive tiles (same XCD, same time) share the larger operand: the weight tile when M is small (patch GEMMs),
  // the activation rows when M is large (convolutions)
  const bool m_fast = (long long)p.M <= (long long)p.N * 2;
  const int m0 = (m_fast ? t % MT : t / NT) * BM, n0 = (m_fast ? t / MT : t % NT) * BN;
  const int nsplit = gridDim.y, split = blockIdx.y;
  const int KT_all = p.K / (64 * KS);
  const int kt_per = (KT_all + nsplit - 1) / nsplit;
  const int kt_lo = split * kt_per;
  const int KT = (kt_lo + kt_per <= KT_all ? kt_per : KT_all - kt_lo);   // >= 1 by construction of nsplit

  const int lr = lane >> 3;                 // row within the 8-row group a wave instruction covers
  // LDS row r keeps global chunk c at slot c ^ ((r >> 1) & 7): with 64 banks a 16-byte read is served 16 lanes at a
  // time, i.e. 16 consecutive rows, which this spreads over all banks (rows r and r+1 differ by 128 B = 32 banks)
  // swizzle key of a tile row r is (r >> 1) & 7; BM / NW and BN / NW are multiples of 8, so the key is the same for
  // the A and B rows of instruction j when BM == BN, and is computed per operand otherwise
  auto kc_a = [&](int j) { return (lane & 7) ^ (((wave * (BM / NW) + j * 8 + lr) >> 1) & 7); };
  auto kc_b = [&](int j) { return (lane & 7) ^ (((wave * (BN / NW) + j * 8 + lr) >> 1) & 7); };
  const bf16_t* a_ptr[AJ];
  int a_b[AJ], a_ro[AJ], a_co[AJ];
  bool a_ok[AJ];
#pragma unroll
  for (int j = 0; j < AJ; ++j) {
    const int row = wave * (BM / NW) + j * 8 + lr;
    int m = m0 + row;
    a_ok[j] = m < p.M;
    if (m >= p.M) m = p.M - 1;
    if constexpr (kConv) {
      const int per = p.Ro * p.Wo;
      a_b[j] = m / per;
      const int rem = m - a_b[j] * per;
      a_ro[j] = rem / p.Wo;
      a_co[j] = rem - a_ro[j] * p.Wo;
      a_ptr[j] = nullptr;
    } else {
      a_ptr[j] = p.A + (long long)m * p.lda + kc_a(j) * 8;
      a_b[j] = a_ro[j] = a_co[j] = 0;
    }
  }
  const bf16_t* b_ptr[BJ];
#pragma unroll
  for (int j = 0; j < BJ; ++j) {
    const int tr = wave * (BN / NW) + j * 8 + lr;     // tile row of the weight operand
    int n = n0 + tr;
    if (p.geglu) {
      // tile columns come in (value, gate) pairs of 32: columns [64q, 64q+32) are value rows, [64q+32, 64q+64) the
      // gate rows of the same 32 outputs, so that one wave holds both in its two accumulator blocks
      const int q = tr >> 6, w32 = tr & 31, gate = (tr >> 5) & 1;
      n = (n0 >> 1) + q * 32 + w32 + gate * p.geglu;
    }
    if (n >= p.N) n = p.N - 1;
    if (p.packed_w)   // tile (n/64, kt) is 8 KB contiguous, rows and swizzled 16-byte slots exactly as they sit in LDS
      b_ptr[j] = p.Wt + ((long long)(n >> 6) * (p.K / 64) * 64 + (n & 63)) * 64 + (lane & 7) * 8;
    else
      b_ptr[j] = p.Wt + (long long)n * p.ldw + kc_b(j) * 8;
  }
  const int b_kstep = p.packed_w ? 4096 : 64;   // elements between consecutive k-tiles of the weight operand

  // Convolution: a lane's source row changes only with the filter tap, i.e. every Cin / 64 slabs; its pointer (channel
  // 0 of the tap's pixel in the fresh patch or a halo row, or the page of zeros for padding) is kept between slabs and
  // a slab only adds its scalar channel offset.  (Recomputed per slab, the gather's address arithmetic - two divisions
  // and a handful of 64-bit multiplies under divergent branches - outweighed the slab's four MFMAs.)
  const bf16_t* a_tap[AJ];
  bool a_pad[AJ];
  int tap_k0 = -1;                          // first k of the tap the pointers are set for
  auto set_tap = [&](int tap) {
    const int ky = tap / 3, kx = tap - ky * 3;
#pragma unroll
    for (int j = 0; j < AJ; ++j) {
      const int ri = a_ro[j] * p.stride + ky - 1;
      const int ci = a_co[j] * p.stride + kx - 1;
      const bf16_t* src = a_ok[j] ? conv_tap_src(p.A, p.top, p.bot, p.halo_bs, p.left, p.right, p.side_bs, p.side_rs,
                                                 a_b[j], ri, ci, p.R, p.W, p.Cin)
                                  : nullptr;
      a_pad[j] = src == nullptr;
      a_tap[j] = (src ? src : zeros) + kc_a(j) * 8;
    }
  };
  auto issue = [&](int kt, int stage) {
    if (kt > KT - 1) kt = KT - 1;           // past the end: reload the last tile into a free stage (keeps vmcnt uniform)
#pragma unroll
    for (int sl = 0; sl < KS; ++sl) {
      const int slab = (kt_lo + kt) * KS + sl;
      const int k0 = slab * 64;
      char* sa = smem + stage * STAGE + sl * SLAB + (wave * (BM / NW)) * 128;
      char* sb = smem + stage * STAGE + sl * SLAB + A_BYTES + (wave * (BN / NW)) * 128;
      if constexpr (kConv) {
        if (tap_k0 < 0 || k0 < tap_k0 || k0 >= tap_k0 + p.Cin) {     // (uniform) a new tap
          const int tap = k0 / p.Cin;
          tap_k0 = tap * p.Cin;
          set_tap(tap);
        }
        const int cin0 = k0 - tap_k0;
#pragma unroll
        for (int j = 0; j < AJ; ++j) {
          const bf16_t* src = a_pad[j] ? a_tap[j] : a_tap[j] + cin0;
          __builtin_amdgcn_global_load_lds(DF_GPTR(src), DF_LPTR(sa + j * 1024), 16, 0, 0);
        }
      } else {
#pragma unroll
        for (int j = 0; j < AJ; ++j)
          __builtin_amdgcn_global_load_lds(DF_GPTR(a_ptr[j] + k0), DF_LPTR(sa + j * 1024), 16, 0, 0);
      }
#pragma unroll
      for (int j = 0; j < BJ; ++j)
        __builtin_amdgcn_global_load_lds(DF_GPTR(b_ptr[j] + (long long)slab * b_kstep), DF_LPTR(sb + j * 1024), 16, 0, 0);
    }
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  DF_TRACE(0);
#pragma unroll
  for (int s = 0; s < STAGES; ++s) issue(s, s);
  DF_TRACE(1);

  const int lrow = lane & 31, g = lane >> 5;
  const int sw = (lrow >> 1) & 7;
  const bool ln_fold = !kConv && p.ln_s != nullptr;
  float ln_sum[TM], ln_sq[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) { ln_sum[i] = 0.f; ln_sq[i] = 0.f; }

  // The MFMA operands of a whole k-slab (four 16-wide k-steps) are held in registers, double-buffered over slabs:
  // the fragments of slab kt+1 are requested from LDS before the MFMAs of slab kt are issued, so neither the LDS
  // round trip nor the barrier sits between dependent matrix instructions.  (One fragment read per MFMA made the
  // K loop a chain of LDS latencies: 0.4 us per slab whatever the depth of the ring.)  A ring stage is free again
  // once every wave holds its fragments, so STAGES slabs of loads are in flight, not STAGES-1.
  bf16x8 af[2][4][TM], bfr[2][4][TN];
  auto read_frags = [&](int stage, auto bufc) {
    constexpr int buf = decltype(bufc)::value;
    const char* As = smem + stage * STAGE + (wm * (BM / 2) + lrow) * 128;
    const char* Bs = smem + stage * STAGE + A_BYTES + (wn * (BN / 2) + lrow) * 128;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const int slot = ((2 * ks + g) ^ sw) * 16;
#pragma unroll
      for (int i = 0; i < TM; ++i) af[buf][ks][i] = *reinterpret_cast<const bf16x8*>(As + i * 32 * 128 + slot);
#pragma unroll
      for (int j = 0; j < TN; ++j) bfr[buf][ks][j] = *reinterpret_cast<const bf16x8*>(Bs + j * 32 * 128 + slot);
    }
  };
  // with fewer than four accumulator blocks per wave, even and odd k-steps go to separate accumulators so that
  // consecutive MFMAs do not wait for each other's result
  constexpr int NACC = (TM * TN >= 4) ? 1 : 2;
  f32x16 acc2[NACC - 1 ? TM : 1][NACC - 1 ? TN : 1];
  if constexpr (NACC == 2) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc2[i][j][e] = 0.f;
  }
  auto slab_step = [&](int kt, int stage, auto curc, auto nxtc) {
    constexpr int cur = decltype(curc)::value;
    // own loads of slab kt+1 have landed (at most STAGES-2 younger slabs outstanding); own fragment reads of slab kt
    // are complete
    DF_TRACE(8 + 4 * kt);
    wait_vm_and_lds<(STAGES - 2) * L>();
    asm volatile("" ::: "memory");
    DF_TRACE(8 + 4 * kt + 1);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    DF_TRACE(8 + 4 * kt + 2);
    issue(kt + STAGES, stage);                // stage of slab kt: every wave holds its fragments in registers
    if (computes) {
      if (kt + 1 < KT) read_frags(stage + 1 == STAGES ? 0 : stage + 1, nxtc);
      __builtin_amdgcn_sched_barrier(0);
      DF_TRACE(8 + 4 * kt + 3);
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            if (NACC == 2 && (ks & 1))
              acc2[NACC - 1 ? i : 0][NACC - 1 ? j : 0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                  af[cur][ks][i], bfr[cur][ks][j], acc2[NACC - 1 ? i : 0][NACC - 1 ? j : 0], 0, 0, 0);
            else
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[cur][ks][i], bfr[cur][ks][j], acc[i][j], 0, 0, 0);
          }
        if constexpr (!kConv) {
          // row sums of the A operand for the folded LayerNorm: two v_dot2 per dword, the two waves that share
          // the rows take alternate k-steps (runs on the vector ALU beside the matrix pipe)
          if (ln_fold && (ks & 1) == wn) {
            const bf16x2_t ones = __builtin_bit_cast(bf16x2_t, 0x3f803f80u);
#pragma unroll
            for (int i = 0; i < TM; ++i) {
              const u32x4 raw = __builtin_bit_cast(u32x4, af[cur][ks][i]);
              const unsigned int wds[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                const bf16x2_t v2 = __builtin_bit_cast(bf16x2_t, wds[q]);
                ln_sum[i] = __builtin_amdgcn_fdot2_f32_bf16(v2, ones, ln_sum[i], false);
                ln_sq[i] = __builtin_amdgcn_fdot2_f32_bf16(v2, v2, ln_sq[i], false);
              }
            }
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // slab 0 has landed once at most STAGES-1 younger slabs are outstanding
  wait_vm_and_lds<(STAGES - 1) * L>();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  if (computes) read_frags(0, std::integral_constant<int, 0>());
  int stage = 0;
  for (int kt = 0; kt < KT; kt += 2) {
    slab_step(kt, stage, std::integral_constant<int, 0>(), std::integral_constant<int, 1>());
    stage = (stage + 1 == STAGES) ? 0 : stage + 1;
    if (kt + 1 < KT) {
      slab_step(kt + 1, stage, std::integral_constant<int, 1>(), std::integral_constant<int, 0>());
      stage = (stage + 1 == STAGES) ? 0 : stage + 1;
    }
  }
  if constexpr (NACC == 2) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] += acc2[i][j];
  }
  DF_TRACE(2);
  wait_vm_and_lds<0>();                      // drain the clamped tail loads before the workgroup ends
  DF_TRACE(3);

  // ---- epilogue ----
  // The accumulators are staged through LDS (the operand ring is free now) so that every lane then handles four
  // consecutive columns of one row: bias / norm vectors / residual are read and the result is written with 16-byte
  // (float) or 8-byte (bf16) accesses instead of 4- and 2-byte ones.
  constexpr int PT = (BM * (BN + 4) * 4 + BM * 24 <= STAGES * STAGE) ? BN + 4 : BN;   // LDS pitch of the staged tile
  float* tile = reinterpret_cast<float*>(smem);
  float* s_mr = tile + BM * PT;               // [BM][2] mean, rstd of the tile's rows (folded LayerNorm)
  if constexpr (!kConv) {
    if (ln_fold) {
      float* s_part = s_mr + BM * 2;          // [2][BM][2] partial (sum, sum of squares) of the two waves of a row
      __syncthreads();                        // every wave is done with the operand stages
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const float sm = ln_sum[i] + __shfl_xor(ln_sum[i], 32, 64);   // the two lane groups hold different k chunks
        const float sq = ln_sq[i] + __shfl_xor(ln_sq[i], 32, 64);
        if (g == 0 && computes) {
          const int r = wm * (BM / 2) + i * 32 + lrow;
          s_part[(wn * BM + r) * 2] = sm;
          s_part[(wn * BM + r) * 2 + 1] = sq;
        }
      }
      __syncthreads();
      if (tid < BM) {
        const float sm = s_part[tid * 2] + s_part[(BM + tid) * 2];
        const float sq = s_part[tid * 2 + 1] + s_part[(BM + tid) * 2 + 1];
        const float mean = sm / (float)p.K;
        const float var = fmaxf(sq / (float)p.K - mean * mean, 0.f);
        s_mr[tid * 2] = mean;
        s_mr[tid * 2 + 1] = 1.0f / sqrtf(var + p.ln_eps);
      }
    }
  }

  if (p.vec_epi) {
    __syncthreads();                          // operand stages no longer read by anyone
    if (computes)
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
      for (int tn = 0; tn < TN; ++tn)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int lr_ = wm * (BM / 2) + tm * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3);
          tile[lr_ * PT + wn * (BN / 2) + tn * 32 + (lane & 31)] = acc[tm][tn][e];
        }
    __syncthreads();
    const int per = kConv ? p.Ro * p.Wo : 1;
    if (nsplit > 1) {
      float* mine = partials + (size_t)split * p.M * p.N;
      for (int idx = tid; idx < BM * (BN / 4); idx += NTHR) {
        const int lr_ = idx / (BN / 4), c4 = (idx % (BN / 4)) * 4;
        const int row = m0 + lr_, col = n0 + c4;
        if (row < p.M && col < p.N)
          *reinterpret_cast<f32x4*>(mine + (size_t)row * p.N + col) = *reinterpret_cast<const f32x4*>(tile + lr_ * PT + c4);
      }
      return;
    }
    if constexpr (!kConv && TN == 2 && sizeof(OutT) == 2) {
      if (p.geglu) {
        // tile columns [64q, 64q+32) are value columns, [64q+32, 64q+64) the gate columns of the same outputs
        for (int idx = tid; idx < BM * (BN / 8); idx += NTHR) {
          const int lr_ = idx / (BN / 8), o = (idx % (BN / 8)) * 4;
          const int row = m0 + lr_, oc = (n0 >> 1) + o;
          if (row >= p.M || oc >= p.geglu) continue;
          const int tc = (o >> 5) * 64 + (o & 31);
          f32x4 val = *reinterpret_cast<const f32x4*>(tile + lr_ * PT + tc);
          f32x4 gte = *reinterpret_cast<const f32x4*>(tile + lr_ * PT + tc + 32);
          if (ln_fold) {
            const float mean = s_mr[lr_ * 2], rstd = s_mr[lr_ * 2 + 1];
            val = (val - *reinterpret_cast<const f32x4*>(p.ln_s + oc) * mean) * rstd + *reinterpret_cast<const f32x4*>(p.ln_t + oc);
            gte = (gte - *reinterpret_cast<const f32x4*>(p.ln_s + p.geglu + oc) * mean) * rstd +
                  *reinterpret_cast<const f32x4*>(p.ln_t + p.geglu + oc);
          } else if (p.bias) {
            val += *reinterpret_cast<const f32x4*>(p.bias + oc);
            gte += *reinterpret_cast<const f32x4*>(p.bias + p.geglu + oc);
          }
          float r4[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) r4[q] = val[q] * gelu_erf(gte[q]);
          u32x2 t = {pack_bf2(r4[0], r4[1]), pack_bf2(r4[2], r4[3])};
          *reinterpret_cast<u32x2*>(reinterpret_cast<bf16_t*>(p.out) + (long long)row * p.ldo + oc) = t;
        }
        return;
      }
    }
    if constexpr (!kConv && sizeof(OutT) == 2) {
      if (p.nseg > 0 && p.seg_tr[n0 / p.seg_w]) {
        // transposed segment (V^T for the attention kernel): feature-major output, rows contiguous.  Threads walk the
        // tile row-fastest so that neighbouring threads write neighbouring rows of one feature.
        const int sg = n0 / p.seg_w;
        bf16_t* obase = reinterpret_cast<bf16_t*>(p.seg_out[sg]);
        for (int idx = tid; idx < BM * BN; idx += NTHR) {
          const int lr_ = idx % BM, lc = idx / BM;
          const int row = m0 + lr_, col = n0 + lc;
          if (row >= p.M || col >= p.N) continue;
          float v = tile[lr_ * PT + lc];
          if (ln_fold) v = (v - p.ln_s[col] * s_mr[lr_ * 2]) * s_mr[lr_ * 2 + 1] + p.ln_t[col];
          else if (p.bias) v += p.bias[col];
          const int bi = row / p.seg_rows_in[sg];
          obase[((long long)bi * p.seg_w + (col - sg * p.seg_w)) * p.seg_ld[sg] + p.seg_row0[sg] +
                seg_pos(row - bi * p.seg_rows_in[sg], p.seg_pin[sg], p.seg_pout[sg])] = f2bf(v);
        }
        return;
      }
    }
    for (int idx = tid; idx < BM * (BN / 4); idx += NTHR) {
      const int lr_ = idx / (BN / 4), c4 = (idx % (BN / 4)) * 4;
      const int row = m0 + lr_, col = n0 + c4;
      if (row >= p.M || col >= p.N) continue;
      f32x4 v = *reinterpret_cast<const f32x4*>(tile + lr_ * PT + c4);
      if constexpr (kConv) {
        if (p.bias) v += *reinterpret_cast<const f32x4*>(p.bias + col);
        if (p.chan_add) v += *reinterpret_cast<const f32x4*>(p.chan_add + (long long)(row / per) * p.chan_ld + col);
      } else {
        if (ln_fold)
          v = (v - *reinterpret_cast<const f32x4*>(p.ln_s + col) * s_mr[lr_ * 2]) * s_mr[lr_ * 2 + 1] +
              *reinterpret_cast<const f32x4*>(p.ln_t + col);
        else if (p.bias)
          v += *reinterpret_cast<const f32x4*>(p.bias + col);
      }
      if (p.residual) v += *reinterpret_cast<const f32x4*>(p.residual + (long long)row * p.ldr + col);
      if (p.act == 1) { v.x = silu_f(v.x); v.y = silu_f(v.y); v.z = silu_f(v.z); v.w = silu_f(v.w); }
      OutT* obase = reinterpret_cast<OutT*>(p.out);
      long long old = p.ldo, orow = row;
      int ocol = col;
      if (p.nseg > 0) {                       // a group of four columns never straddles a segment (seg_w % 64 == 0)
        const int sg = col / p.seg_w;
        obase = reinterpret_cast<OutT*>(p.seg_out[sg]);
        old = p.seg_ld[sg];
        ocol = col - sg * p.seg_w;
        const int bi = row / p.seg_rows_in[sg];
        orow = (long long)bi * p.seg_rows_out[sg] + p.seg_row0[sg] +
               seg_pos(row - bi * p.seg_rows_in[sg], p.seg_pin[sg], p.seg_pout[sg]);
      }
      if constexpr (sizeof(OutT) == 4) {
        *reinterpret_cast<f32x4*>(obase + orow * old + ocol) = v;
      } else {
        u32x2 t = {pack_bf2(v.x, v.y), pack_bf2(v.z, v.w)};
        *reinterpret_cast<u32x2*>(obase + orow * old + ocol) = t;
      }
      if constexpr (!kConv) {
        if (p.out2) {
          u32x2 t = {pack_bf2(v.x, v.y), pack_bf2(v.z, v.w)};
          *reinterpret_cast<u32x2*>(p.out2 + (long long)row * p.ldo2 + col) = t;
        }
      }
    }
    return;
  }

  // ---- scalar epilogue: shapes or pointers that do not allow the vector accesses above ----
  __syncthreads();                            // the folded-norm statistics, if any, are visible
  if (!computes) return;                      // loader waves hold no accumulators
  if (nsplit > 1) {
    // float partial of this split, [split][M][N]; the epilogue runs in splitk_reduce_kernel
    float* mine = partials + (size_t)split * p.M * p.N;
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
      const int col = n0 + wn * (BN / 2) + tn * 32 + (lane & 31);
      if (col >= p.N) continue;
#pragma unroll
      for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int row = m0 + wm * (BM / 2) + tm * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3);
          if (row < p.M) mine[(size_t)row * p.N + col] = acc[tm][tn][e];
        }
    }
    return;
  }

  OutT* out = reinterpret_cast<OutT*>(p.out);
  const int per = kConv ? p.Ro * p.Wo : 1;
  if constexpr (!kConv && TN == 2 && sizeof(OutT) == 2) {
    if (p.geglu) {
      // accumulator block 0 holds the value columns, block 1 the gate columns of the same outputs
      const int oc = (n0 >> 1) + wn * 32 + (lane & 31);
      if (oc < p.geglu) {
        const float bv = p.bias ? p.bias[oc] : 0.f, bg = p.bias ? p.bias[p.geglu + oc] : 0.f;
        const float sv = ln_fold ? p.ln_s[oc] : 0.f, sg = ln_fold ? p.ln_s[p.geglu + oc] : 0.f;
        const float tv = ln_fold ? p.ln_t[oc] : 0.f, tg = ln_fold ? p.ln_t[p.geglu + oc] : 0.f;
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            const int lr_ = wm * (BM / 2) + tm * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3);
            const int row = m0 + lr_;
            if (row >= p.M) continue;
            float val = acc[tm][0][e] + bv, gte = acc[tm][1][e] + bg;
            if (ln_fold) {
              const float mean = s_mr[lr_ * 2], rstd = s_mr[lr_ * 2 + 1];
              val = rstd * (acc[tm][0][e] - mean * sv) + tv;
              gte = rstd * (acc[tm][1][e] - mean * sg) + tg;
            }
            const float gl = gelu_erf(gte);
            Elem<OutT>::st(out + (long long)row * p.ldo + oc, val * gl);
          }
      }
      return;
    }
  }
#pragma unroll
  for (int tn = 0; tn < TN; ++tn) {
    const int col = n0 + wn * (BN / 2) + tn * 32 + (lane & 31);
    if (col >= p.N) continue;
    const float bias = p.bias ? p.bias[col] : 0.f;
    const float ln_sc = ln_fold ? p.ln_s[col] : 0.f, ln_tc = ln_fold ? p.ln_t[col] : 0.f;
    // segmented output: the 32 columns of a block never straddle a segment (seg_w % 32 == 0)
    OutT* obase = out;
    long long old = p.ldo, orow0 = 0, orows_out = 0;
    int ocol = col, orows_in = 0x7fffffff, opin = 0, opout = 0;
    bool otr = false;
    if (p.nseg > 0) {
      const int sg = col / p.seg_w;
      obase = reinterpret_cast<OutT*>(p.seg_out[sg]);
      old = p.seg_ld[sg]; orow0 = p.seg_row0[sg]; orows_out = p.seg_rows_out[sg]; orows_in = p.seg_rows_in[sg];
      ocol = col - sg * p.seg_w;
      otr = p.seg_tr[sg] != 0;
      opin = p.seg_pin[sg]; opout = p.seg_pout[sg];
    }
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int lr_ = wm * (BM / 2) + tm * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3);
        const int row = m0 + lr_;
        if (row >= p.M) continue;
        float v = acc[tm][tn][e] + bias;
        if constexpr (kConv) {
          if (p.chan_add) v += p.chan_add[(long long)(row / per) * p.chan_ld + col];
        } else {
          if (ln_fold) v = s_mr[lr_ * 2 + 1] * (acc[tm][tn][e] - s_mr[lr_ * 2] * ln_sc) + ln_tc;
        }
        if (p.residual) v += p.residual[(long long)row * p.ldr + col];
        if (p.act == 1) v = silu_f(v);
        long long orow = row;
        if (p.nseg > 0) {
          const int bi = row / orows_in;
          const long long pos = seg_pos(row - bi * orows_in, opin, opout);
          orow = (long long)bi * orows_out + orow0 + pos;
          if (otr) {   // feature-major segment
            Elem<OutT>::st(obase + ((long long)bi * p.seg_w + ocol) * old + orow0 + pos, v);
            continue;
          }
        }
        Elem<OutT>::st(obase + orow * old + ocol, v);
        if constexpr (!kConv) {
          if (p.out2) p.out2[(long long)row * p.ldo2 + col] = f2bf(v);
        }
      }
    }
  }
}

// ---- direct convolutions for tiny or narrow shapes ----

// One lane per (output pixel, output channel).
template <typename T, typename OutT>
__global__ __launch_bounds__(256) void conv3x3_direct(const T* __restrict__ x, const T* __restrict__ top,
                                                      const T* __restrict__ bot, long long halo_bs,
                                                      const T* __restrict__ left, const T* __restrict__ right,
                                                      long long side_bs, long long side_rs,
                                                      const T* __restrict__ w, const float* __restrict__ bias,
                                                      const float* __restrict__ chan_add,
                                                      const float* __restrict__ residual, OutT* __restrict__ y, int B,
                                                      int R, int W, int Cin, int Cout, int Ro, int Wo, int stride,
                                                      int act) {
  const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long total = (long long)B * Ro * Wo * Cout;
  if (idx >= total) return;
  const int co = (int)(idx % Cout);
  long long pix = idx / Cout;
  const int c = (int)(pix % Wo);
  pix /= Wo;
  const int r = (int)(pix % Ro);
  const int b = (int)(pix / Ro);
  float acc = bias ? bias[co] : 0.f;
  for (int ky = 0; ky < 3; ++ky) {
    const int ri = r * stride + ky - 1;
    for (int kx = 0; kx < 3; ++kx) {
      const int ci = c * stride + kx - 1;
      const T* xp = conv_tap_src(x, top, bot, halo_bs, left, right, side_bs, side_rs, b, ri, ci, R, W, Cin);
      if (!xp) continue;
      const T* wp = w + (((long long)co * 3 + ky) * 3 + kx) * Cin;
      float s = 0.f;
      for (int i = 0; i < Cin; ++i) s = fmaf(Elem<T>::ld(xp + i), Elem<T>::ld(wp + i), s);
      acc += s;
    }
  }
  if (chan_add) acc += chan_add[(long long)b * Cout + co];
  if (residual) acc += residual[idx];
  if (act == 1) acc = silu_f(acc);
  Elem<OutT>::st(y + idx, acc);
}

// f32, Cin % 4 == 0: a workgroup owns 4 pixels x 32 output channels, its four waves every fourth 16-byte chunk of the channels
// of each tap; a lane owns one output channel of two pixels.  Latency-bound at the sizes it is used at: all loads of
// a tap are independent, and the weights of a channel are read along its row (one thread per output before, a serial
// loop over 9 x Cin with the lanes' weights a row apart: 128 pixels x 32 channels, Cin = 32: 37.9 -> 4 us).
__global__ __launch_bounds__(256) void conv3x3_f32(const float* __restrict__ x, const float* __restrict__ top,
                                                   const float* __restrict__ bot, long long halo_bs,
                                                   const float* __restrict__ left, const float* __restrict__ right,
                                                   long long side_bs, long long side_rs, const float* __restrict__ w,
                                                   const float* __restrict__ bias, const float* __restrict__ chan_add,
                                                   const float* __restrict__ residual, float* __restrict__ y, int B, int R,
                                                   int W, int Cin, int Cout, int Ro, int Wo, int stride, int act) {
  __shared__ float red[4][4][32];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int nct = (Cout + 31) >> 5;
  const long long total = (long long)B * Ro * Wo;
  const long long p0 = (long long)(blockIdx.x / nct) * 4;
  const int c0 = (int)(blockIdx.x % nct) * 32;
  const int co = c0 + (lane & 31) < Cout ? c0 + (lane & 31) : Cout - 1;
  int pr[2], pc[2], pb[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    long long pix = p0 + 2 * (lane >> 5) + i;
    if (pix >= total) pix = total - 1;
    pc[i] = (int)(pix % Wo) * stride;
    pr[i] = (int)((pix / Wo) % Ro) * stride;
    pb[i] = (int)(pix / ((long long)Wo * Ro));
  }
  float acc[2] = {0.f, 0.f};
#pragma unroll
  for (int tap = 0; tap < 9; ++tap) {
    const float* xp[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
      xp[i] = conv_tap_src(x, top, bot, halo_bs, left, right, side_bs, side_rs, pb[i], pr[i] + tap / 3 - 1,
                           pc[i] + tap % 3 - 1, R, W, Cin);
    const float* wp = w + ((long long)co * 9 + tap) * Cin;
    for (int k = wave * 4; k < Cin; k += 16) {
      const f32x4 wv = *reinterpret_cast<const f32x4*>(wp + k);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        f32x4 xv = {0.f, 0.f, 0.f, 0.f};
        if (xp[i]) xv = *reinterpret_cast<const f32x4*>(xp[i] + k);
        acc[i] = fmaf(xv.x, wv.x, acc[i]); acc[i] = fmaf(xv.y, wv.y, acc[i]);
        acc[i] = fmaf(xv.z, wv.z, acc[i]); acc[i] = fmaf(xv.w, wv.w, acc[i]);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) red[wave][2 * (lane >> 5) + i][lane & 31] = acc[i];
  __syncthreads();
  if (threadIdx.x < 128) {
    const int px = threadIdx.x >> 5, n = c0 + (threadIdx.x & 31);
    const long long pix = p0 + px;
    if (pix >= total || n >= Cout) return;
    float v = (red[0][px][threadIdx.x & 31] + red[1][px][threadIdx.x & 31]) +
              (red[2][px][threadIdx.x & 31] + red[3][px][threadIdx.x & 31]);
    if (bias) v += bias[n];
    if (chan_add) v += chan_add[pix / ((long long)Ro * Wo) * Cout + n];
    if (residual) v += residual[pix * Cout + n];
    if (act == 1) v = silu_f(v);
    y[pix * Cout + n] = v;
  }
}

// One wave per output pixel, lanes split the 9*Cin reduction; for wide inputs and few outputs (Cout <= 8).
template <typename T, typename OutT, int CO>
__global__ __launch_bounds__(256) void conv3x3_wave(const T* __restrict__ x, const T* __restrict__ top,
                                                    const T* __restrict__ bot, long long halo_bs,
                                                    const T* __restrict__ left, const T* __restrict__ right,
                                                    long long side_bs, long long side_rs,
                                                    const T* __restrict__ w, const float* __restrict__ bias,
                                                    const float* __restrict__ residual, OutT* __restrict__ y, int B,
                                                    int R, int W, int Cin, int Cout, int Ro, int Wo, int stride,
                                                    int act) {
  const int lane = threadIdx.x & 63;
  const long long pix = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (pix >= (long long)B * Ro * Wo) return;
  const int c = (int)(pix % Wo);
  const int r = (int)((pix / Wo) % Ro);
  const int b = (int)(pix / ((long long)Wo * Ro));
  float acc[CO];
#pragma unroll
  for (int o = 0; o < CO; ++o) acc[o] = 0.f;
  for (int ky = 0; ky < 3; ++ky) {
    const int ri = r * stride + ky - 1;
    for (int kx = 0; kx < 3; ++kx) {
      const int ci = c * stride + kx - 1;
      const T* xp = conv_tap_src(x, top, bot, halo_bs, left, right, side_bs, side_rs, b, ri, ci, R, W, Cin);
      if (!xp) continue;
      for (int i = lane; i < Cin; i += 64) {
        const float xv = Elem<T>::ld(xp + i);
#pragma unroll
        for (int o = 0; o < CO; ++o)
          if (o < Cout) acc[o] = fmaf(xv, Elem<T>::ld(w + (((long long)o * 3 + ky) * 3 + kx) * Cin + i), acc[o]);
      }
    }
  }
#pragma unroll
  for (int o = 0; o < CO; ++o) acc[o] = wave_sum(acc[o]);
  if (lane == 0) {
#pragma unroll
    for (int o = 0; o < CO; ++o) {
      if (o >= Cout) break;
      float v = acc[o] + (bias ? bias[o] : 0.f);
      if (residual) v += residual[pix * Cout + o];
      if (act == 1) v = silu_f(v);
      Elem<OutT>::st(y + pix * Cout + o, v);
    }
  }
}

// Four input channels (the latent entering the network): a thread owns one pixel and 8 consecutive output channels;
// the 9 x 4 inputs are loaded once with 8-byte accesses and reused for the 8 outputs, the 46 KB of weights stay in L1.
template <typename OutT>
__global__ __launch_bounds__(256) void conv3x3_cin4(const bf16_t* __restrict__ x, const bf16_t* __restrict__ top,
                                                    const bf16_t* __restrict__ bot, long long halo_bs,
                                                    const bf16_t* __restrict__ left, const bf16_t* __restrict__ right,
                                                    long long side_bs, long long side_rs,
                                                    const bf16_t* __restrict__ w, const float* __restrict__ bias,
                                                    const float* __restrict__ residual, OutT* __restrict__ y, int B, int R,
                                                    int W, int Cout, int Ro, int Wo, int stride, int act) {
  const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const int cg = Cout >> 3;
  const long long total = (long long)B * Ro * Wo * cg;
  if (idx >= total) return;
  const int co = (int)(idx % cg) * 8;
  long long pix = idx / cg;
  const int c = (int)(pix % Wo);
  const int r = (int)((pix / Wo) % Ro);
  const int b = (int)(pix / ((long long)Wo * Ro));
  float xin[9][4];
#pragma unroll
  for (int ky = 0; ky < 3; ++ky) {
    const int ri = r * stride + ky - 1;
#pragma unroll
    for (int kx = 0; kx < 3; ++kx) {
      const int ci = c * stride + kx - 1;
      const bf16_t* xp = conv_tap_src(x, top, bot, halo_bs, left, right, side_bs, side_rs, b, ri, ci, R, W, 4);
      u32x2 t = {0u, 0u};
      if (xp) t = *reinterpret_cast<const u32x2*>(xp);
      xin[ky * 3 + kx][0] = __uint_as_float(t.x << 16); xin[ky * 3 + kx][1] = __uint_as_float(t.x & 0xffff0000u);
      xin[ky * 3 + kx][2] = __uint_as_float(t.y << 16); xin[ky * 3 + kx][3] = __uint_as_float(t.y & 0xffff0000u);
    }
  }
  float acc[8];
#pragma unroll
  for (int o = 0; o < 8; ++o) {
    float a = bias ? bias[co + o] : 0.f;
    const bf16_t* wp = w + (long long)(co + o) * 36;
#pragma unroll
    for (int tp = 0; tp < 9; ++tp) {
      const u32x2 t = *reinterpret_cast<const u32x2*>(wp + tp * 4);
      a = fmaf(xin[tp][0], __uint_as_float(t.x << 16), a);
      a = fmaf(xin[tp][1], __uint_as_float(t.x & 0xffff0000u), a);
      a = fmaf(xin[tp][2], __uint_as_float(t.y << 16), a);
      a = fmaf(xin[tp][3], __uint_as_float(t.y & 0xffff0000u), a);
    }
    acc[o] = a;
  }
  const long long o0 = pix * Cout + co;
  if (residual) {
    float r8[8];
    ld_vec(residual + o0, r8); ld_vec(residual + o0 + 4, r8 + 4);
#pragma unroll
    for (int o = 0; o < 8; ++o) acc[o] += r8[o];
  }
  if (act == 1) {
#pragma unroll
    for (int o = 0; o < 8; ++o) acc[o] = silu_f(acc[o]);
  }
  if constexpr (sizeof(OutT) == 4) { st_vec(y + o0, acc); st_vec(y + o0 + 4, acc + 4); }
  else st_vec(y + o0, acc);
}

// Few output channels (the noise prediction leaving the network, Cout <= 4) and Cin % 8 == 0: a wave owns four
// neighbouring pixels of one row; lanes split the 9 x Cin reduction in 16-byte chunks, each weight chunk is used for
// the four pixels.
template <typename OutT, int CO>
__global__ __launch_bounds__(256) void conv3x3_fewout(const bf16_t* __restrict__ x, const bf16_t* __restrict__ top,
                                                      const bf16_t* __restrict__ bot, long long halo_bs,
                                                      const bf16_t* __restrict__ left, const bf16_t* __restrict__ right,
                                                      long long side_bs, long long side_rs,
                                                      const bf16_t* __restrict__ w, const float* __restrict__ bias,
                                                      const float* __restrict__ residual, OutT* __restrict__ y, int B,
                                                      int R, int W, int Cin, int Cout, int act) {
  const int lane = threadIdx.x & 63;
  const int wq = (W + 3) >> 2;                                  // pixel quads per row
  const long long quad = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (quad >= (long long)B * R * wq) return;
  const int c0 = (int)(quad % wq) * 4;
  const int r = (int)((quad / wq) % R);
  const int b = (int)(quad / ((long long)wq * R));
  const int cpt = Cin >> 3;                                     // 16-byte chunks per tap
  float acc[4][CO];
#pragma unroll
  for (int px = 0; px < 4; ++px)
#pragma unroll
    for (int o = 0; o < CO; ++o) acc[px][o] = 0.f;
  for (int ch = lane; ch < 9 * cpt; ch += 64) {
    const int tp = ch / cpt, k8 = (ch - tp * cpt) * 8;
    const int ky = tp / 3, kx = tp - ky * 3;
    const int ri = r + ky - 1;
    float wv[CO][8];
#pragma unroll
    for (int o = 0; o < CO; ++o) {
      if (o < Cout) ld_vec(w + ((long long)o * 9 + tp) * Cin + k8, wv[o]);
      else {
#pragma unroll
        for (int e = 0; e < 8; ++e) wv[o][e] = 0.f;
      }
    }
#pragma unroll
    for (int px = 0; px < 4; ++px) {
      // pixels beyond the row's end read its last pixel (nothing is stored for them)
      const int ci = (c0 + px < W ? c0 + px : W - 1) + kx - 1;
      const bf16_t* xp = conv_tap_src(x, top, bot, halo_bs, left, right, side_bs, side_rs, b, ri, ci, R, W, Cin);
      if (!xp) continue;
      float xv[8];
      ld_vec(xp + k8, xv);
#pragma unroll
      for (int o = 0; o < CO; ++o)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[px][o] = fmaf(xv[e], wv[o][e], acc[px][o]);
    }
  }
#pragma unroll
  for (int px = 0; px < 4; ++px)
#pragma unroll
    for (int o = 0; o < CO; ++o) acc[px][o] = wave_sum(acc[px][o]);
  if (lane < 4 && c0 + lane < W) {
    const long long pix = ((long long)b * R + r) * W + c0 + lane;
#pragma unroll
    for (int o = 0; o < CO; ++o) {
      if (o >= Cout) break;
      float v = 0.f;
#pragma unroll
      for (int px = 0; px < 4; ++px) if (px == lane) v = acc[px][o];
      v += bias ? bias[o] : 0.f;
      if (residual) v += residual[pix * Cout + o];
      if (act == 1) v = silu_f(v);
      Elem<OutT>::st(y + pix * Cout + o, v);
    }
  }
}

// ---- one-time weight re-layout for the pipelined kernel ----
// out tile (n/64, k/64) is 64 rows x 64 k, row r = n % 64 holds global 16-byte chunk c at slot c ^ ((r >> 1) & 7)
__global__ __launch_bounds__(256) void pack_weight_kernel(const bf16_t* __restrict__ w, const float* __restrict__ gamma,
                                                          bf16_t* __restrict__ out, int N, int K) {
  const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const int kch = K / 8;
  if (idx >= (long long)N * kch) return;
  const int n = (int)(idx / kch), c = (int)(idx % kch);
  float v[8];
  ld_vec(w + (long long)n * K + c * 8, v);
  if (gamma) {
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] *= gamma[c * 8 + i];
  }
  const int r = n & 63, kt = c >> 3, slot = (c & 7) ^ ((r >> 1) & 7);
  st_vec(out + (((long long)(n >> 6) * (K / 64) + kt) * 64 + r) * 64 + slot * 8, v);
}

// one wave per output row
__global__ __launch_bounds__(256) void fold_vectors_kernel(const bf16_t* __restrict__ w, const float* __restrict__ gamma,
                                                           const float* __restrict__ beta, const float* __restrict__ bias,
                                                           float* __restrict__ s, float* __restrict__ t, int N, int K) {
  const int lane = threadIdx.x & 63;
  const int n = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (n >= N) return;
  float a = 0.f, b = 0.f;
  for (int k = lane; k < K; k += 64) {
    const float wv = bf2f(w[(long long)n * K + k]);
    a += bf2f(f2bf(wv * gamma[k]));
    b = fmaf(wv, beta[k], b);
  }
  a = wave_sum(a);
  b = wave_sum(b);
  if (lane == 0) { s[n] = a; t[n] = b + (bias ? bias[n] : 0.f); }
}

template <int BM, int BN, bool kConv>
int launch_tile(const TileParams& p, int out_dtype, hipStream_t st) {
  dim3 grid(cdiv(p.N, BN), cdiv(p.M, BM));
  if (grid.y > 65535) return DF_ESHAPE;
  if (out_dtype == DF_BF16)
    hipLaunchKernelGGL((mfma_tile_kernel<BM, BN, kConv, bf16_t>), grid, dim3(256), 0, st, p);
  else
    hipLaunchKernelGGL((mfma_tile_kernel<BM, BN, kConv, float>), grid, dim3(256), 0, st, p);
  DF_LAUNCH_CHECK();
  return DF_OK;
}

// out[m, n] = sum over splits of partial[s][m][n] + bias + per-(batch,channel) add + residual, activation; 4 columns per lane
template <typename OutT>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(TileParams p, const float* __restrict__ partials, int nsplit,
                                                           int per) {
  // 32-bit index arithmetic (split launches have fewer than 1024 tiles of 64 x 64, far below 2^31 elements)
  const unsigned int idx = blockIdx.x * blockDim.x + threadIdx.x;
  const unsigned int n4 = (unsigned int)p.N / 4;
  if (idx >= (unsigned int)p.M * n4) return;
  const int row = (int)(idx / n4), col = (int)(idx - (idx / n4) * n4) * 4;
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  for (int s = 0; s < nsplit; ++s)
    v += *reinterpret_cast<const f32x4*>(partials + ((size_t)s * p.M + row) * p.N + col);
  if (p.bias) v += *reinterpret_cast<const f32x4*>(p.bias + col);
  if (p.chan_add) v += *reinterpret_cast<const f32x4*>(p.chan_add + (long long)(row / per) * p.chan_ld + col);
  if (p.residual) v += *reinterpret_cast<const f32x4*>(p.residual + (long long)row * p.ldr + col);
  if (p.act == 1) { v.x = silu_f(v.x); v.y = silu_f(v.y); v.z = silu_f(v.z); v.w = silu_f(v.w); }
  OutT* o = reinterpret_cast<OutT*>(p.out) + (long long)row * p.ldo + col;
  if constexpr (sizeof(OutT) == 4) {
    *reinterpret_cast<f32x4*>(o) = v;
  } else {
    u32x2 t = {pack_bf2(v.x, v.y), pack_bf2(v.z, v.w)};
    *reinterpret_cast<u32x2*>(o) = t;
  }
  if (p.out2) {
    u32x2 t = {pack_bf2(v.x, v.y), pack_bf2(v.z, v.w)};
    *reinterpret_cast<u32x2*>(p.out2 + (long long)row * p.ldo2 + col) = t;
  }
}

template <int BM, int BN, int STAGES, bool kConv, int KS = 1, int NW = 4>
int launch_pipe(const TileParams& p, int out_dtype, int nsplit, hipStream_t st) {
  const long long nwg = (long long)cdiv(p.M, BM) * cdiv(p.N, BN);
  if (nwg > 0x7fffffffLL) return DF_ESHAPE;
  if (p.K % (64 * KS)) return DF_ESHAPE;
  const int KT = p.K / (64 * KS);
  if (nsplit > KT) nsplit = KT;
  if (nsplit < 1 || p.N % 4 || p.ldr % 4 || p.ldo % 4 || p.ldo2 % 4 || p.ln_s || p.geglu || p.nseg) nsplit = 1;
  if (nsplit > 1) nsplit = cdiv(KT, cdiv(KT, nsplit));   // no empty split
  const size_t part_bytes = nsplit > 1 ? (size_t)nsplit * p.M * p.N * sizeof(float) : 0;
  char* scr = nullptr;
  if (kConv || nsplit > 1) {
    scr = scratch_region(p.scr, kScratchCounterBytes + part_bytes);
    if (!scr) return DF_ENOMEM;
  }
  const bf16_t* zeros = scr ? (const bf16_t*)(scr + kScratchZeroPageOffset) : nullptr;
  float* partials = scr ? (float*)(scr + kScratchCounterBytes) : nullptr;
  constexpr int smem = STAGES * (BM + BN) * 128 * KS;
  dim3 grid((unsigned)nwg, (unsigned)nsplit);
  TileParams q = p;
  {
    auto al = [](const void* ptr, int a) { return ((uintptr_t)ptr % a) == 0; };
    bool ok = p.N % 4 == 0 && p.ldo % 4 == 0 && al(p.out, 16) && al(p.bias, 16) && al(p.chan_add, 16) && p.chan_ld % 4 == 0 &&
              (!p.residual || (p.ldr % 4 == 0 && al(p.residual, 16))) && (!p.out2 || (p.ldo2 % 4 == 0 && al(p.out2, 8))) &&
              al(p.ln_s, 16) && al(p.ln_t, 16) && (!p.geglu || p.geglu % 4 == 0);
    for (int i = 0; i < p.nseg; ++i) ok = ok && (p.seg_tr[i] || (p.seg_ld[i] % 4 == 0 && al(p.seg_out[i], 8))) && p.seg_w % 4 == 0;
    if (p.ln_s && BM * (BN + 4) * 4 + BM * 24 > smem) return DF_ESHAPE;   // no room for the row statistics
    q.vec_epi = ok ? 1 : 0;
  }
  if (out_dtype == DF_BF16) {
    auto k = mfma_pipe_kernel<BM, BN, STAGES, kConv, bf16_t, KS, NW>;
    static bool attr_set = false;
    if (!attr_set) {
      if (hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, smem) != hipSuccess) return DF_EHIP;
      attr_set = true;
    }
    hipLaunchKernelGGL(k, grid, dim3(64 * NW), smem, st, q, zeros, partials);
  } else {
    auto k = mfma_pipe_kernel<BM, BN, STAGES, kConv, float, KS, NW>;
    static bool attr_set = false;
    if (!attr_set) {
      if (hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, smem) != hipSuccess) return DF_EHIP;
      attr_set = true;
    }
    hipLaunchKernelGGL(k, grid, dim3(64 * NW), smem, st, q, zeros, partials);
  }
  DF_LAUNCH_CHECK();
  if (nsplit > 1) {
    const long long n = (long long)p.M * (p.N / 4);
    const int per = kConv ? p.Ro * p.Wo : 1;
    if (out_dtype == DF_BF16)
      hipLaunchKernelGGL(splitk_reduce_kernel<bf16_t>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, partials, nsplit, per);
    else
      hipLaunchKernelGGL(splitk_reduce_kernel<float>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, partials, nsplit, per);
    DF_LAUNCH_CHECK();
  }
  return DF_OK;
}

// Tile choice.  DF_TILE=<BM>x<BN>x<STAGES> and DF_SPLITK=<n> in the environment override the heuristic (tuning
// aid); with DF_TUNE set they are re-read on every launch.
bool tune_mode() {
  static int v = -1;
  if (v < 0) v = tune_env("DF_TUNE") ? 1 : 0;
  return v == 1;
}

int parse_tile() {
  const char* e = tune_env("DF_TILE");
  int bm = 0, bn = 0, st = 4;
  if (e && sscanf(e, "%dx%dx%d", &bm, &bn, &st) >= 2) return (bm * 1000 + bn) * 10 + st;
  return 0;
}

int tile_override() {
  if (tune_mode()) return parse_tile();
  static int v = -1;
  if (v < 0) v = parse_tile();
  return v;
}

int split_override() {
  if (tune_mode()) { const char* e = tune_env("DF_SPLITK"); return e ? atoi(e) : 0; }
  static int v = -1;
  if (v < 0) { const char* e = tune_env("DF_SPLITK"); v = e ? atoi(e) : 0; }
  return v;
}

// Tile and split choice, measured on the patch step (kernel trace, weights cold).  A compute unit delivers operands
// to its waves at a fixed rate (about one 1 KB wave load per 32 cycles), so what counts is that every unit carries the
// same number of equally long workgroups: a problem with T 64x64 tiles is split along K into ns parts such that
// T * ns just fills the slots the chip offers for the chosen ring depth (two stages = 32 KB of LDS, three = 48 KB:
// three workgroups per unit, 768 slots; four stages with eight waves: two per unit, 512 slots).  Measured optima this
// reproduces: 375 tiles -> 2 parts, 190 tiles -> 4 parts, 100 tiles -> 5 parts; every part keeps at least 8 k-slabs.
// Only very large problems use 128x128.
template <bool kConv>
int launch_auto(const TileParams& p, int out_dtype, hipStream_t st) {
  const long long big = (long long)cdiv(p.M, 128) * cdiv(p.N, 128);
  const long long nwg = (long long)cdiv(p.M, 64) * cdiv(p.N, 64);
  const int KT = p.K / 64;
  auto parts_for = [&](long long slots) {
    int ns = (int)((slots + nwg / 2) / nwg);
    if (ns > 8) ns = 8;
    while (ns > 1 && KT / ns < 8) --ns;
    return ns < 1 ? 1 : ns;
  };
  if (split_override() > 0) return launch_pipe<64, 64, 4, kConv, 1, 8>(p, out_dtype, split_override(), st);
  if (big >= 1024 && !p.ln_s) return launch_pipe<128, 128, 3, kConv, 1, 8>(p, out_dtype, 1, st);   // eight waves: four only load
  if (nwg >= 512) return launch_pipe<64, 64, 2, kConv>(p, out_dtype, 1, st);
  if (nwg > 128) {
    const int ns = parts_for(768);
    if (ns <= 2) return launch_pipe<64, 64, 2, kConv>(p, out_dtype, ns, st);
    return launch_pipe<64, 64, 3, kConv>(p, out_dtype, ns, st);
  }
  return launch_pipe<64, 64, 4, kConv, 1, 8>(p, out_dtype, parts_for(512), st);   // few tiles: four stages, eight waves
}

template <bool kConv>
int pick_tile(const TileParams& p, int out_dtype, hipStream_t st) {
  const long long big = (long long)cdiv(p.M, 128) * cdiv(p.N, 128);
  const bool pipe = (p.K % 64 == 0) && (!kConv || p.Cin % 64 == 0) && p.K >= 128;
  if (pipe) {
    const int so = split_override() > 0 ? split_override() : 1;
    switch (tile_override()) {
      case 1281284: return launch_pipe<128, 128, 4, kConv>(p, out_dtype, so, st);
      case 1281283: return launch_pipe<128, 128, 3, kConv>(p, out_dtype, so, st);
      case 1281282: return launch_pipe<128, 128, 2, kConv>(p, out_dtype, so, st);
      case 1281286: return launch_pipe<128, 128, 4, kConv, 1, 8>(p, out_dtype, so, st);   // 'x6': four stages, eight waves
      case 1281287: return launch_pipe<128, 128, 3, kConv, 1, 8>(p, out_dtype, so, st);   // 'x7': three stages, eight waves
      case 1280647: return launch_pipe<128, 64, 3, kConv, 1, 8>(p, out_dtype, so, st);
      case 640647: return launch_pipe<64, 64, 3, kConv, 1, 8>(p, out_dtype, so, st);
      case 1280643: return launch_pipe<128, 64, 3, kConv>(p, out_dtype, so, st);
      case 640644: return launch_pipe<64, 64, 4, kConv>(p, out_dtype, so, st);
      case 640642: return launch_pipe<64, 64, 2, kConv>(p, out_dtype, so, st);
      case 640643: return launch_pipe<64, 64, 3, kConv>(p, out_dtype, so, st);
      case 640646: return launch_pipe<64, 64, 4, kConv, 1, 8>(p, out_dtype, so, st);   // 'x6': four stages, eight waves
      case 640648: return launch_pipe<64, 64, 8, kConv>(p, out_dtype, so, st);
      case 641282: return launch_pipe<64, 128, 2, kConv>(p, out_dtype, so, st);
      case 641284: return launch_pipe<64, 128, 4, kConv>(p, out_dtype, so, st);
      default: break;
    }
    return launch_auto<kConv>(p, out_dtype, st);
  }
  if (big >= 384) return launch_tile<128, 128, kConv>(p, out_dtype, st);
  return launch_tile<64, 64, kConv>(p, out_dtype, st);
}

}  // namespace

int launch_pack_weight(const bf16_t* w, const float* gamma, bf16_t* out, int N, int K, hipStream_t st) {
  if (N % 64 || K % 64 || N <= 0 || K <= 0) return DF_ESHAPE;
  const long long n = (long long)N * (K / 8);
  hipLaunchKernelGGL(pack_weight_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, w, gamma, out, N, K);
  DF_LAUNCH_CHECK();
  return DF_OK;
}

int launch_fold_vectors(const bf16_t* w, const float* gamma, const float* beta, const float* bias, float* s, float* t,
                        int N, int K, hipStream_t st) {
  hipLaunchKernelGGL(fold_vectors_kernel, dim3((unsigned)((N + 3) / 4)), dim3(256), 0, st, w, gamma, beta, bias, s, t, N, K);
  DF_LAUNCH_CHECK();
  return DF_OK;
}

// bytes of library scratch a tile launch may ask for (plans reserve it up front)
size_t gemm_scratch_bytes(long long M, long long N) {
  // split-K is only used below 1024 workgroups of 64x64 and with at most 8 splits
  const long long nwg = (long long)cdiv(M, 64) * cdiv(N, 64);
  return kScratchCounterBytes + (size_t)(nwg < 1024 ? 8 * M * N * sizeof(float) : 0);
}

int launch_gemm_bf16(const GemmArgs& a, hipStream_t st) {
  if (a.M <= 0 || a.N <= 0 || a.K <= 0 || a.K % BK) return DF_ESHAPE;
  if (a.lda % 8 || a.ldw % 8 || ((uintptr_t)a.A % 16) || ((uintptr_t)a.W % 16)) return DF_EINVAL;
  TileParams p = {};
  p.A = (const bf16_t*)a.A; p.Wt = (const bf16_t*)a.W; p.bias = a.bias; p.residual = a.residual; p.out = a.out;
  p.M = a.M; p.N = a.N; p.K = a.K; p.lda = a.lda; p.ldw = a.ldw; p.ldr = a.ldr; p.ldo = a.ldo; p.act = a.act;
  p.scr = a.scr;
  const bool special = a.packed_w || a.ln_s || a.out2;
  if (special) {
    if (a.K % 64 || a.K < 128) return DF_ESHAPE;
    if (a.packed_w && a.N % 64) return DF_ESHAPE;
    if (a.ln_s && (!a.ln_t || a.bias)) return DF_EINVAL;
    if (a.out2 && (a.geglu || a.nseg)) return DF_ESHAPE;
    p.packed_w = a.packed_w; p.ln_s = a.ln_s; p.ln_t = a.ln_t; p.ln_eps = a.ln_eps;
    p.out2 = (bf16_t*)a.out2; p.ldo2 = a.ldo2;
  }
  if (a.geglu || a.nseg > 0) {
    if (a.K % 64 || a.K < 128 || a.out_dtype != DF_BF16 || a.residual || a.act) return DF_ESHAPE;
    if (a.geglu) {
      if (a.N % 128 || a.nseg) return DF_ESHAPE;
      p.geglu = a.N / 2;
      // thousands of rows (the synchronous full-image step): the 128x128 tile with eight waves, half the operand bytes
      // per MFMA (4096 x 10240 x 1280: 220 -> 191 us)
      static const int big_geglu = tune_env("DF_GEGLU_BIG") ? atoi(tune_env("DF_GEGLU_BIG")) : 512;   // tuning aid
      if ((long long)cdiv(a.M, 128) * cdiv(a.N, 128) >= big_geglu)
        return launch_pipe<128, 128, 3, false, 1, 8>(p, DF_BF16, 1, st);
      return launch_pipe<64, 128, 2, false>(p, DF_BF16, 1, st);
    }
    if (a.nseg > 3 || a.seg_w % 64 || a.seg_w * a.nseg != a.N) return DF_ESHAPE;
    p.nseg = a.nseg; p.seg_w = a.seg_w;
    for (int i = 0; i < a.nseg; ++i) {
      if (!a.seg_out[i] || a.seg_rows_in[i] <= 0) return DF_EINVAL;
      p.seg_out[i] = a.seg_out[i]; p.seg_ld[i] = a.seg_ld[i]; p.seg_rows_out[i] = a.seg_rows_out[i];
      p.seg_row0[i] = a.seg_row0[i]; p.seg_rows_in[i] = a.seg_rows_in[i]; p.seg_tr[i] = a.seg_tr[i];
      p.seg_pin[i] = a.seg_pin[i]; p.seg_pout[i] = a.seg_pout[i];
    }
    if ((long long)cdiv(a.M, 64) * cdiv(a.N, 64) >= 512) return launch_pipe<64, 64, 2, false>(p, DF_BF16, 1, st);
    return launch_pipe<64, 64, 4, false, 1, 8>(p, DF_BF16, 1, st);
  }
  if (special) return launch_auto<false>(p, a.out_dtype, st);   // these epilogues exist in the pipelined kernel only
  return pick_tile<false>(p, a.out_dtype, st);
}

int launch_conv3x3(const ConvArgs& a, hipStream_t st) {
  if (a.stride != 1 && a.stride != 2) return DF_ESHAPE;
  if (a.stride == 2 && ((a.R & 1) || (a.W & 1))) return DF_ESHAPE;
  const int Ro = a.R / a.stride, Wo = a.W / a.stride;
  const long long M = (long long)a.B * Ro * Wo;
  if (M <= 0 || M > 0x7fffffffLL) return DF_ESHAPE;
  const bool sides = a.halo_left || a.halo_right;
  if (sides && (a.halo_top || a.halo_bot)) return DF_EINVAL;     // a patch is a strip along one direction
  const bool mfma = a.dtype == DF_BF16 && a.Cin % BK == 0 && a.Cout % 32 == 0 && ((uintptr_t)a.x % 16 == 0) &&
                    ((uintptr_t)a.w % 16 == 0) && ((uintptr_t)a.halo_top % 16 == 0) &&
                    ((uintptr_t)a.halo_bot % 16 == 0) && (a.halo_bstride % 8 == 0) && ((uintptr_t)a.halo_left % 16 == 0) &&
                    ((uintptr_t)a.halo_right % 16 == 0) && (a.side_bstride % 8 == 0) && (a.side_rstride % 8 == 0);
  if (mfma) {
    TileParams p = {};
    p.A = (const bf16_t*)a.x; p.Wt = (const bf16_t*)a.w; p.bias = a.bias; p.residual = a.residual;
    p.chan_add = a.chan_add; p.chan_ld = a.chan_ld ? a.chan_ld : a.Cout; p.out = a.y;
    p.M = (int)M; p.N = a.Cout; p.K = 9 * a.Cin; p.lda = 0; p.ldw = 9LL * a.Cin; p.ldr = a.Cout; p.ldo = a.Cout;
    p.act = a.act; p.scr = a.scr;
    p.top = (const bf16_t*)a.halo_top; p.bot = (const bf16_t*)a.halo_bot; p.halo_bs = a.halo_bstride;
    p.left = (const bf16_t*)a.halo_left; p.right = (const bf16_t*)a.halo_right; p.side_bs = a.side_bstride;
    p.side_rs = a.side_rstride;
    p.R = a.R; p.W = a.W; p.Cin = a.Cin; p.Ro = Ro; p.Wo = Wo; p.stride = a.stride;
    return pick_tile<true>(p, a.out_dtype, st);
  }
  if (a.chan_add && a.chan_ld && a.chan_ld != a.Cout) return DF_ESHAPE;   // the direct kernels assume a dense [B, Cout]
  const long long total = M * a.Cout;
#define DF_DIRECT(T, OT)                                                                                              \
  hipLaunchKernelGGL((conv3x3_direct<T, OT>), dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, (const T*)a.x, \
                     (const T*)a.halo_top, (const T*)a.halo_bot, a.halo_bstride, (const T*)a.halo_left,               \
                     (const T*)a.halo_right, a.side_bstride, a.side_rstride, (const T*)a.w, a.bias, a.chan_add,       \
                     a.residual, (OT*)a.y, a.B, a.R, a.W, a.Cin, a.Cout, Ro, Wo, a.stride, a.act)
#define DF_WAVE(T, OT)                                                                                                \
  hipLaunchKernelGGL((conv3x3_wave<T, OT, 8>), dim3((unsigned)((M + 3) / 4)), dim3(256), 0, st, (const T*)a.x,        \
                     (const T*)a.halo_top, (const T*)a.halo_bot, a.halo_bstride, (const T*)a.halo_left,               \
                     (const T*)a.halo_right, a.side_bstride, a.side_rstride, (const T*)a.w, a.bias, a.residual,       \
                     (OT*)a.y, a.B, a.R, a.W, a.Cin, a.Cout, Ro, Wo, a.stride, a.act)
  if ((total + 255) / 256 > 0x7fffffffLL) return DF_ESHAPE;
  // 16-byte loads; the pixels of four channels are loaded with 8-byte ones
  const int pa = a.Cin == 4 && a.dtype == DF_BF16 ? 8 : 16;
  const bool al16 = ((uintptr_t)a.x % 16 == 0) && ((uintptr_t)a.w % 16 == 0) && ((uintptr_t)a.halo_top % 16 == 0) &&
                    ((uintptr_t)a.halo_bot % 16 == 0) && ((uintptr_t)a.halo_left % pa == 0) && ((uintptr_t)a.halo_right % pa == 0);
  const int pe = pa / (a.dtype == DF_BF16 ? 2 : 4);              // elements per aligned access
  if (a.dtype == DF_BF16 && !a.chan_add && al16 && a.side_bstride % pe == 0 && a.side_rstride % pe == 0) {
    if (a.Cin == 4 && a.Cout % 8 == 0 && a.halo_bstride % 4 == 0 && ((uintptr_t)a.y % 16 == 0) &&
        ((uintptr_t)a.residual % 16 == 0)) {
      const long long n = M * (a.Cout / 8);
#define DF_C4(OT)                                                                                                  \
  hipLaunchKernelGGL((conv3x3_cin4<OT>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, (const bf16_t*)a.x,     \
                     (const bf16_t*)a.halo_top, (const bf16_t*)a.halo_bot, a.halo_bstride, (const bf16_t*)a.halo_left, \
                     (const bf16_t*)a.halo_right, a.side_bstride, a.side_rstride, (const bf16_t*)a.w, a.bias,         \
                     a.residual, (OT*)a.y, a.B, a.R, a.W, a.Cout, Ro, Wo, a.stride, a.act)
      if (a.out_dtype == DF_BF16) DF_C4(bf16_t); else DF_C4(float);
#undef DF_C4
      DF_LAUNCH_CHECK();
      return DF_OK;
    }
    if (a.Cout <= 4 && a.Cin % 8 == 0 && a.stride == 1 && a.halo_bstride % 8 == 0) {
      const long long quads = (long long)a.B * a.R * ((a.W + 3) / 4);
#define DF_FEW(OT)                                                                                                 \
  hipLaunchKernelGGL((conv3x3_fewout<OT, 4>), dim3((unsigned)((quads + 3) / 4)), dim3(256), 0, st, (const bf16_t*)a.x, \
                     (const bf16_t*)a.halo_top, (const bf16_t*)a.halo_bot, a.halo_bstride, (const bf16_t*)a.halo_left, \
                     (const bf16_t*)a.halo_right, a.side_bstride, a.side_rstride, (const bf16_t*)a.w, a.bias,         \
                     a.residual, (OT*)a.y, a.B, a.R, a.W, a.Cin, a.Cout, a.act)
      if (a.out_dtype == DF_BF16) DF_FEW(bf16_t); else DF_FEW(float);
#undef DF_FEW
      DF_LAUNCH_CHECK();
      return DF_OK;
    }
  }
  const bool wave = a.Cout <= 8 && a.Cin >= 64 && !a.chan_add;
  if (a.dtype == DF_F32) {
    if (a.out_dtype != DF_F32) return DF_ESHAPE;
    if (!wave && al16 && a.Cin % 4 == 0 && a.halo_bstride % 4 == 0 && a.side_bstride % 4 == 0 && a.side_rstride % 4 == 0) {
      // outputs per workgroup: 4 pixels x 32 channels
      const long long nwg = cdiv(M, 4) * (long long)cdiv(a.Cout, 32);
      if (nwg > 0x7fffffffLL) return DF_ESHAPE;
      hipLaunchKernelGGL(conv3x3_f32, dim3((unsigned)nwg), dim3(256), 0, st, (const float*)a.x, (const float*)a.halo_top,
                         (const float*)a.halo_bot, a.halo_bstride, (const float*)a.halo_left, (const float*)a.halo_right,
                         a.side_bstride, a.side_rstride, (const float*)a.w, a.bias, a.chan_add, a.residual, (float*)a.y, a.B,
                         a.R, a.W, a.Cin, a.Cout, Ro, Wo, a.stride, a.act);
    } else if (wave) DF_WAVE(float, float); else DF_DIRECT(float, float);
  } else {
    if (a.out_dtype == DF_BF16) { if (wave) DF_WAVE(bf16_t, bf16_t); else DF_DIRECT(bf16_t, bf16_t); }
    else { if (wave) DF_WAVE(bf16_t, float); else DF_DIRECT(bf16_t, float); }
  }
#undef DF_DIRECT
#undef DF_WAVE
  DF_LAUNCH_CHECK();
  return DF_OK;
}

#ifdef DF_TUNING
// Tuning build only: copies the cycle stamps of the last mfma_pipe_kernel launch to host memory (synchronises).
extern "C" __attribute__((visibility("default"))) int df_tune_pipe_trace(long long* out, int n) {
  if (!out || n <= 0 || n > 4 * 512 + 8) return DF_EINVAL;
  if (hipDeviceSynchronize() != hipSuccess) return DF_EHIP;
  if (hipMemcpyFromSymbol(out, HIP_SYMBOL(g_pipe_trace), (size_t)n * sizeof(long long)) != hipSuccess) return DF_EHIP;
  return DF_OK;
}
#endif

}  // namespace df
