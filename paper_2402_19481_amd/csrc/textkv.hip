#include <type_traits>

#include "tile.h"

namespace df {

namespace {

template <int VM>
__device__ __forceinline__ void wait_vm() {   // s_waitcnt vmcnt(VM)
  __builtin_amdgcn_s_waitcnt((VM & 0xF) | ((VM >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

struct TextKvParams {
  const bf16_t* text;
  int K, TL, B, passes, units, tiled, nseg;
  TextKvSeg seg[kTextKvSegs];
};

constexpr int text_kv_stage(int XA, int IT) { return (32 * XA * IT + 128) * 128; }
constexpr int text_kv_stages(int XA, int IT) { const int n = 160 * 1024 / text_kv_stage(XA, IT); return n < 6 ? n : 6; }

// The text tokens' keys and values of all transformer blocks, as the fragments of the cross-attention (launch_pack_text_kv).  A tile is 128
// columns (two heads' keys or values) of IT batch items, padded to XA * 32 tokens each; a wave has 32 columns of one item in registers.
//   - What bounds it: the weights, from HBM, once.  A workgroup per compute unit goes through its tiles as through one long K: the next
//     tile's loads are under way while this one's results are stored, and nothing of LDS is needed for that, because the operands are read in the
//     order (bits 2 and 3 of the row swapped) and the roles (tokens as the matrix instruction's columns for keys, as its rows for values)
//     that leave the accumulators as 16-byte pieces of the fragments.
//   - Four of the waves only load: a wave that issues its loads between the matrix instructions waits for the load path's queue, with one or
//     two such waves per SIMD nothing else ran meanwhile.  100 tiles of K = 2048 20.8 -> 14.4 us.
//   - The units begin K at different slabs (rot): in lockstep over tiles that lie powers of two apart they asked the same memory channels.
//     77 tokens, 1300 tiles of K = 2048 (682 MB of weights): 173 us in lockstep, 146 from different slabs; 140 with the same number of tiles for
//     every workgroup that has any, 5.1 TB/s with the results; a layer on 128 x 128 tiles and a launch that packs its result took 190.  Two batch
//     items 174 us (of 260): twice the matrix instructions and reads of LDS.
template <int XA, int IT>
__global__ __launch_bounds__(256 * (IT + 1), IT + 1) void text_kv_kernel(TextKvParams p) {
  constexpr int NC = 4 * IT, NW = 4, ST = text_kv_stages(XA, IT), STAGE = text_kv_stage(XA, IT), ROWS = 32 * XA * IT;
  constexpr int AJ = ROWS / 8 / NW, BJ = 16 / NW, L = AJ + BJ;           // 1 KB direct loads per wave and slab
  static_assert(AJ * 8 * NW == ROWS && ST > 2 && L * (ST - 1) < 64, "whole loads; the vmcnt field is 6 bits");
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int item = wave >> 2, cb = wave & 3, lw = wave - NC;   // batch item of the pass, 32 columns of the tile
  const int KT = p.K / 64;
  const int mine = (p.units - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x, NS = mine * KT;
  const int rot = (int)((blockIdx.x * (unsigned int)KT) / gridDim.x);
  const int last0 = p.B - IT;                                            // first item of the last pass (items before it: done already)

  // unit u: a tile of one of the segments and a pass of batch items
  struct Unit { int seg, tile, b0, first; };
  auto unit = [&](int i) {
    const int u = (int)blockIdx.x + i * (int)gridDim.x;
    Unit r;
    r.tile = u / p.passes;
    r.first = (u - r.tile * p.passes) * IT;
    r.b0 = r.first < last0 ? r.first : last0;
    r.seg = 0;
    while (r.seg + 1 < p.nseg && r.tile >= p.seg[r.seg].tiles) r.tile -= p.seg[r.seg++].tiles;
    return r;
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  if (wave >= NC) {                                                      // a loading wave
    const int lr = lane >> 3;
    unsigned int a_ofs[AJ], b_ofs[BJ];
#pragma unroll
    for (int j = 0; j < AJ; ++j) {
      const int row = (lw * AJ + j) * 8 + lr, it = row / (32 * XA), key = row - it * (32 * XA);
      const int src = it * p.TL + (key < p.TL ? key : p.TL - 1);           // (no such token: the last one again, zeroed when stored)
      a_ofs[j] = 2u * ((unsigned int)src * (unsigned int)p.K + (unsigned int)(((lane & 7) ^ ((row >> 1) & 7)) * 8));
    }
#pragma unroll
    for (int j = 0; j < BJ; ++j) b_ofs[j] = w_lane_bytes(p.tiled, 0, (lw * BJ + j) * 8 + lr, lane & 7, 128, KT, p.K);
    const unsigned int b_step = w_slab_bytes(p.tiled);
    const char *la = nullptr, *lb = nullptr;
    int li = 0, lk = 0;
    auto set_load = [&] {
      const Unit u = unit(li);
      la = (const char*)(p.text + (long long)u.b0 * p.TL * p.K);
      lb = (const char*)((const bf16_t*)p.seg[u.seg].w + w_tile_base(p.tiled, u.tile * 128, KT, p.K));
    };
    auto issue = [&](int slot) {
      int slab = lk + rot;
      if (slab >= KT) slab -= KT;
      char* sa = smem + slot * STAGE + lw * AJ * 1024;
      char* sb = smem + slot * STAGE + ROWS * 128 + lw * BJ * 1024;
#pragma unroll
      for (int q = 0; q < BJ; ++q) lds_load_buf(lb, b_ofs[q], (unsigned int)slab * b_step, sb + q * 1024);
#pragma unroll
      for (int q = 0; q < AJ; ++q) lds_load_buf(la, a_ofs[q], (unsigned int)slab * 128u, sa + q * 1024);
      if (++lk == KT) {
        lk = 0;
        if (++li < mine) set_load();
      }
    };
    set_load();
    for (int s = 0; s < ST - 1; ++s)
      if (s < NS) issue(s);
    if (NS >= ST - 1) wait_vm<L * (ST - 2)>();
    else wait_vm<0>();
    block_sync();
    int pslot = ST - 1;
    for (int s = 0; s < NS; ++s) {
      if (s + ST - 1 < NS) {
        issue(pslot);
        pslot = pslot + 1 == ST ? 0 : pslot + 1;
        wait_vm<L * (ST - 2)>();
      } else {
        wait_vm<0>();
      }
      block_sync();
    }
    return;
  }
  f32x16 acc[XA];
  const int lrow = lane & 31, g = lane >> 5;
  const int sig = (lrow & 0x13) | ((lrow & 4) << 1) | ((lrow & 8) >> 1), sw = (sig >> 1) & 7;
  bf16x8 xa[2][XA], wa[2];
  auto rd = [&](int slot, int ks, auto bc) {
    constexpr int b = decltype(bc)::value;
    const char* s = smem + slot * STAGE + sig * 128 + ((2 * ks + g) ^ sw) * 16;
#pragma unroll
    for (int i = 0; i < XA; ++i) xa[b][i] = *reinterpret_cast<const bf16x8*>(s + (item * XA + i) * 4096);
    wa[b] = *reinterpret_cast<const bf16x8*>(s + ROWS * 128 + cb * 4096);
  };
  auto mm = [&](auto bc, auto vc) {
    constexpr int b = decltype(bc)::value;
#pragma unroll
    for (int i = 0; i < XA; ++i)
      acc[i] = decltype(vc)::value ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(xa[b][i], wa[b], acc[i], 0, 0, 0)
                                   : __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa[b], xa[b][i], acc[i], 0, 0, 0);
  };
  block_sync();
  rd(0, 0, I0{});
  int slot = 0, s = 0;
#define DF_SB __builtin_amdgcn_sched_barrier(0)
  auto tile = [&](auto vc) {
#pragma unroll
    for (int i = 0; i < XA; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
    for (int k = 0; k < KT; ++k, ++s) {
      const int nslot = slot + 1 == ST ? 0 : slot + 1;
      DF_SB; rd(slot, 1, I1{}); DF_SB; mm(I0{}, vc);
      DF_SB; rd(slot, 2, I0{}); DF_SB; mm(I1{}, vc);
      DF_SB; rd(slot, 3, I1{}); DF_SB; mm(I0{}, vc); DF_SB;
      __builtin_amdgcn_s_waitcnt(0xc07f);                                 // lgkmcnt(0): the slab is read
      block_sync();
      if (s + 1 < NS) rd(nslot, 0, I0{});
      DF_SB; mm(I1{}, vc); DF_SB;
      slot = nslot;
    }
  };
#undef DF_SB
  for (int i = 0; i < mine; ++i) {
    const Unit u = unit(i);
    const int heads = p.seg[u.seg].heads, col = 2 * u.tile + (cb >> 1), dt = cb & 1;
    const int j = col / (2 * heads), hv = col - j * 2 * heads, b = u.b0 + item;
    const bool values = hv >= heads;
    bf16_t* out = (bf16_t*)p.seg[u.seg].out +
                  ((((long long)b * p.seg[u.seg].count + j) * heads + (values ? hv - heads : hv)) * (12 * XA) * 64 + lane) * 8;
    if (values) tile(std::true_type{});
    else tile(std::false_type{});
    if (b < u.first) continue;
#pragma unroll
    for (int kt = 0; kt < XA; ++kt)
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        const int key = kt * 32 + (values ? 16 * f + 8 * g : sig);
        float o[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) o[q] = key + (values ? q : 0) < p.TL ? acc[kt][8 * f + q] : 0.f;
        st_vec(out + (values ? 4 * XA + dt * 2 * XA + 2 * kt + f : 4 * kt + 2 * dt + f) * 512, o);
      }
  }
}

template <int XA, int IT>
int launch_one(const TextKvParams& p, hipStream_t st) {
  constexpr int smem = text_kv_stages(XA, IT) * text_kv_stage(XA, IT);
  static bool attr_set = false;
  if (!attr_set) {
    if (hipFuncSetAttribute((const void*)text_kv_kernel<XA, IT>, hipFuncAttributeMaxDynamicSharedMemorySize, smem) != hipSuccess) return DF_EHIP;
    attr_set = true;
  }
  const int each = cdiv(p.units, 256);                                   // (a unit less at most for some of the workgroups)
  hipLaunchKernelGGL((text_kv_kernel<XA, IT>), dim3((unsigned)cdiv(p.units, each)), dim3(256 * (IT + 1)), smem, st, p);
  DF_LAUNCH_CHECK();
  return DF_OK;
}

}  // namespace

int launch_text_kv(const TextKvArgs& a, hipStream_t st) {
  if (a.B <= 0 || a.TL <= 0 || a.TL > 128 || a.K <= 0 || a.K % 64 || a.nseg <= 0 || a.nseg > kTextKvSegs) return DF_ESHAPE;
  if (a.K >= (1 << 22)) return DF_ESHAPE;                                // 32-bit offsets inside a tile
  if (!a.text || (uintptr_t)a.text % 16) return DF_EINVAL;
  TextKvParams p = {};
  p.text = (const bf16_t*)a.text; p.K = a.K; p.TL = a.TL; p.B = a.B; p.tiled = a.packed_w; p.nseg = a.nseg;
  long long tiles = 0;
  for (int s = 0; s < a.nseg; ++s) {
    const TextKvSeg& g = a.seg[s];
    if (!g.w || !g.out || (uintptr_t)g.w % 16 || (uintptr_t)g.out % 16) return DF_EINVAL;
    if (g.heads <= 0 || g.count <= 0) return DF_ESHAPE;
    p.seg[s] = g;
    if ((long long)g.heads * g.count > (1 << 24)) return DF_ESHAPE;
    p.seg[s].tiles = g.heads * g.count;                                  // 2 * heads * count column blocks of 64
    tiles += p.seg[s].tiles;
  }
  const int IT = a.B > 1 ? 2 : 1, XA = (a.TL + 31) / 32;
  p.passes = (a.B + IT - 1) / IT;
  if (tiles * p.passes * (a.K / 64) > 0x7fffffffLL) return DF_ESHAPE;
  p.units = (int)(tiles * p.passes);
  switch (XA * 2 + IT) {
    case 3: return launch_one<1, 1>(p, st);
    case 4: return launch_one<1, 2>(p, st);
    case 5: return launch_one<2, 1>(p, st);
    case 6: return launch_one<2, 2>(p, st);
    case 7: return launch_one<3, 1>(p, st);
    case 8: return launch_one<3, 2>(p, st);
    case 9: return launch_one<4, 1>(p, st);
    default: return launch_one<4, 2>(p, st);
  }
}

}  // namespace df
