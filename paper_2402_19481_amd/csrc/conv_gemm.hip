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
// Two tile kernels: tgemm.hip (operands global -> LDS directly into a ring of stages, used whenever K % 64 == 0) and
// mfma_tile_kernel (BM x BN x 32, register-staged, any K % 32 == 0) with 4 waves in a 2x2 grid, each owning
// (BM/2)x(BN/2) as 32x32 blocks of v_mfma_f32_32x32x16_bf16.
#include "tile.h"

namespace df {

namespace {

constexpr int BK = 32;
constexpr int LDS_PITCH = 40;  // bf16 elements per LDS row: 32 + 8 pad

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
// of each tap; a lane owns one output channel of two pixels.  Latency-bound at the sizes it is used at: the loads of a tap are
// independent and the weights of a channel are read along its row, but the branch around absent pixels keeps each tap behind the one
// before it.  128 pixels x 32 channels, Cin = 32: 9.9 us with its boundary in a graph (one thread per output, a serial loop over 9 x Cin with the
// lanes' weights a row apart: 37.9).
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
// Bound by the requests' round trips: with a branch per tap around each load they came one after another.  Three chunks of weights and
// pixels are requested together, and a lane's sums are added without LDS: 16 x 64 x 320 -> 4 16.5 -> 10.6 us, 256 x 480 140 -> 112.
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
  constexpr int NC = 3;                                         // chunks of a lane requested together
  auto unpack8 = [](const u32x4& t, float* v) {
    const unsigned int q[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) { v[2 * i] = __uint_as_float(q[i] << 16); v[2 * i + 1] = __uint_as_float(q[i] & 0xffff0000u); }
  };
  float acc[4][CO];
#pragma unroll
  for (int px = 0; px < 4; ++px)
#pragma unroll
    for (int o = 0; o < CO; ++o) acc[px][o] = 0.f;
  for (int ch0 = lane; ch0 < 9 * cpt; ch0 += 64 * NC) {
    u32x4 wv[NC][CO], xv[NC][4];
    bool ok[NC][4];
#pragma unroll
    for (int u = 0; u < NC; ++u) {
      const int ch = ch0 + 64 * u < 9 * cpt ? ch0 + 64 * u : ch0;
      const int tp = ch / cpt, k8 = (ch - tp * cpt) * 8;
      const int ky = tp / 3, kx = tp - ky * 3;
      const int ri = r + ky - 1;
#pragma unroll
      for (int o = 0; o < CO; ++o)
        wv[u][o] = *reinterpret_cast<const u32x4*>(w + ((long long)(o < Cout ? o : 0) * 9 + tp) * Cin + k8);
#pragma unroll
      for (int px = 0; px < 4; ++px) {
        // pixels beyond the row's end read its last pixel (nothing is stored for them)
        const int ci = (c0 + px < W ? c0 + px : W - 1) + kx - 1;
        const bf16_t* xp = conv_tap_src(x, top, bot, halo_bs, left, right, side_bs, side_rs, b, ri, ci, R, W, Cin);
        ok[u][px] = xp != nullptr && ch0 + 64 * u < 9 * cpt;
        xv[u][px] = *reinterpret_cast<const u32x4*>((xp ? xp : x) + k8);   // (requested without a branch, used only where ok)
      }
    }
#pragma unroll
    for (int u = 0; u < NC; ++u)
#pragma unroll
      for (int px = 0; px < 4; ++px) {
        if (!ok[u][px]) continue;
        float xf[8];
        unpack8(xv[u][px], xf);
#pragma unroll
        for (int o = 0; o < CO; ++o) {
          float wf[8];
          unpack8(wv[u][o], wf);
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[px][o] = fmaf(xf[e], wf[e], acc[px][o]);
        }
      }
  }
#pragma unroll
  for (int px = 0; px < 4; ++px)
#pragma unroll
    for (int o = 0; o < CO; ++o) acc[px][o] = wave_total(acc[px][o]);
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

// The register-staged tile is left with K % 64 != 0 and pointers or strides that do not allow 16-byte accesses.
template <bool kConv>
int pick_tile(const TileParams& p, int out_dtype, hipStream_t st) {
  const int rc = launch_tgemm(p, kConv, out_dtype, st);
  if (rc != DF_ESHAPE) return rc;
  if (p.packed_w) return DF_ESHAPE;
  if ((long long)cdiv(p.M, 128) * cdiv(p.N, 128) >= 384) return launch_tile<128, 128, kConv>(p, out_dtype, st);
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

int launch_gemm_bf16(const GemmArgs& a, hipStream_t st) {
  if (a.M <= 0 || a.N <= 0 || a.K <= 0 || a.K % BK) return DF_ESHAPE;
  if (a.lda % 8 || a.ldw % 8 || ((uintptr_t)a.A % 16) || ((uintptr_t)a.W % 16)) return DF_EINVAL;
  TileParams p = {};
  p.A = (const bf16_t*)a.A; p.Wt = (const bf16_t*)a.W; p.bias = a.bias; p.residual = a.residual; p.out = a.out;
  p.M = a.M; p.N = a.N; p.K = a.K; p.lda = a.lda; p.ldw = a.ldw; p.ldr = a.ldr; p.ldo = a.ldo; p.act = a.act;
  p.scr = a.scr;
  if (a.packed_w && (a.N % 64 || a.K % 64)) return DF_ESHAPE;
  p.packed_w = a.packed_w;
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

}  // namespace df
