// Displaced self-attention (Section 4, Sparse operations): fresh queries of one
// patch against keys/values of the whole feature map, where the patch's own
// rows are read from the fresh tensors and every other row from the stale
// buffers.  The splice happens in the tile loader; no scattered copy exists.
//
// bf16 (head dim 64): attn_pipe_d64 and, for few queries, attn_wave_d64.  Both compute S^T = K Q^T with
// v_mfma_f32_32x32x16_bf16 so that a lane owns one query column: the softmax's row statistics are lane-local plus one
// exchange with lane^32.  The rows of the K tile are assigned to MFMA rows in a permuted order chosen so that the
// exponentiated accumulators are, without any data movement, the B operand (P^T) of O^T = V^T P^T.
// In the UNet step every key comes from the (already refreshed) stale buffers and V is stored transposed ([feature][key],
// written that way by the projection), so a V^T operand is one 16-byte read of an LDS tile.
// f32: d / 4 lanes share a key (attn_f32); for the small full-precision configuration only.
#include <cstdlib>
#include <type_traits>

#include "kernels.h"

namespace df {

namespace {

constexpr float kLog2e = 1.4426950408889634f;

struct AttnParams {
  const void* q; const void* kf; const void* vf; const void* ks; const void* vs;
  void* out;
  float* part_o;   // [nsplit][B][heads][Lq][d] float (split mode)
  float* part_ml;  // [nsplit][B][heads][Lq][2]
  int B, Lq, L, heads;
  int own_lo, own_n;
  int own_period;  // 0: keys [own_lo, own_lo + own_n) are fresh; P > 0: key j is fresh iff j % P lies in that range
                   // (a vertical strip of a token grid with P columns) and is row (j / P) * own_n + j % P - own_lo
  unsigned int own_magic;   // floor(2^32 / own_period), at most 2^32 - 1
  long long ldq, ldkf, ldvf, ldks, ldvs, ldo;
  long long bsq, bskf, bsvf, bsks, bsvs, bso;
  float scale;
  float sc_log2;   // factor of the scores in log2 units (transposed-V variants): scale * log2(e), or 1 for scaled queries
  int nsplit, keys_per_split;
  int out_packed;
  // transposed-V variant: vs is V^T [B][heads*64][vt_ld] (keys contiguous), every key comes from ks / vs
  long long vt_ld;
  NextReads next;
  int qblocks;     // attn_wave_d64: blocks of 32 queries; the rows of the grid beyond them read ahead
  unsigned int qb_recip;   // the reciprocal of qblocks, where the grid counts them head by head, an eighth for each XCD
};

// Row of the fresh tensor that holds key j, or -1 if the key comes from the stale buffer (Section 4: the keys and
// values are the scatter output; the scatter is resolved here, key by key).
__device__ __forceinline__ long long fresh_row(int own_lo, int own_n, int period, int j) {
  if (period > 0) {
    const int r = j / period, rel = j - r * period - own_lo;
    return (rel >= 0 && rel < own_n) ? (long long)r * own_n + rel : -1;
  }
  const int rel = j - own_lo;
  return (rel >= 0 && rel < own_n) ? (long long)rel : -1;
}

// physical key (0..31) loaded into MFMA row rho of a 32-key block
__device__ __forceinline__ int key_of_mfma_row(int rho) {
  const int j = rho >> 3, g = (rho >> 2) & 1, r = rho & 3;
  return 16 * (j >> 1) + 8 * g + 4 * (j & 1) + r;
}

#ifdef DF_TUNING
// Tuning build only: per workgroup (waves 0 and 5; wave 5's rows follow at +256), 32 stamps: the constant-rate clock at entry and exit, cycle stamps between.
__device__ long long g_attn_trace[512 * 32];
#define DF_ATRACE(slot, expr)                                                                             \
  do {                                                                                                    \
    const unsigned wg_ = blockIdx.x + gridDim.x * blockIdx.y;                                            \
    if ((threadIdx.x == 0 || threadIdx.x == 320) && wg_ < 256 && (slot) < 32)                             \
      g_attn_trace[(wg_ + (threadIdx.x ? 256 : 0)) * 32 + (slot)] = (long long)(expr);                    \
  } while (0)
#else
#define DF_ATRACE(slot, expr) do {} while (0)
#endif

#define DF_LPTR(p) ((__attribute__((address_space(3))) void*)(p))

// Self-attention of the UNet step for many queries: the matrix pipe and the vector ALU of a SIMD work at the same time only
// where one wave's instruction stream mixes the two (measured: 16 MFMAs then 64 exponentials 1030-1600 cycles with any
// number of waves, interleaved one by one 660), so the loop is software-pipelined inside the wave.  Iteration t issues the
// matrix instructions of S_{t+1} = K_{t+1} Q^T and of O += V_{t-1} P_{t-1} between the exponentials of tile t; nothing
// in an iteration waits for anything the same iteration started.
//   - PRE: the queries already carry scale * log2(e) (the projection applies it to its float accumulators before rounding).
//     S then starts from -m instead of zero (the first MFMA of a tile reads the register tuple that holds it), so the
//     exponential's argument is the accumulator itself; otherwise one fma per score.
//   - The running maximum m is that of a range's first tile and moves only when a tile has probabilities far above 1 (so P stays
//     far inside float and bf16 range; relative precision is that of any other scaling).  The sum of a lane's 32 probabilities,
//     which it needs anyway, tells: beyond 2^13 (32 of 2^8) the wave moves m by the power of two above the sum and scales what it has
//     by it, the tile's packed probabilities exactly; beyond 2^100, at the latest where one of them overflows, it drops them (nothing
//     has read them yet) and does the tile again from memory, in a branch beside the loop.  Watching the maximum of the scores
//     instead took 16 instructions per tile, and their latency between the last matrix instruction and the barrier.  A tile from memory
//     stalls the workgroup for some 2 us: with one for every sum beyond 256, peaked scores took 1024 x 4096 x 10 heads from 25 us
//     (standard deviation of 0.25 nats) to 33 (4) and 43 (8), 4096 x 16384 x 10 with the scale from 175 to 217 and 273; now 24.6, 25.1 and
//     30.7, 174, 186 and 222.
//   - Row sums add the float probabilities, not the rounded ones the matrix instructions take: the rounding of a heavy key
//     would otherwise enter every feature of the row (a key of weight 0.9 with values near zero: 2.0e-3 of error against 1.4e-3,
//     where the rounding of the result alone is 1.4e-3; random scores differ by less than 7 % in either direction).  Sums
//     of the packed pairs by v_dot2 are half the instructions and 0.6 % faster on the largest shape.
// K and V^T tiles go global -> LDS through a ring of three slots of an 8 KB tile of each; K_{t+3} and V_{t+1} are requested in
// iteration t.  Slot i holds K_i, K_{i+3}, .. and V_{i+1}, V_{i+4}, ..: what an iteration reads lies in one slot, in the same order
// in both tiles, so four address registers serve its sixteen reads.
// Order of a slot: iteration t reads K_{t+1} and V_{t-1} (S_0 before the loop reads K_0) and ends with a barrier that every wave
// reaches with its reads done (lgkmcnt(0)).  K_{t+3} goes to the slot of K_t, last read in iteration t-1; V_{t+1} to the slot of
// V_{t-2}, last read in iteration t-1: the barrier at that iteration's end lies between.  K_0 is read before the loop, so
// S_0 has a barrier of its own before iteration 0 requests K_3.  A tile done again reads no LDS and passes no barrier.
// Bound by the vector instructions of the softmax (85 per wave and tile: 32 exponentials of 8.3 cycles, 32 additions, 16 packings)
// beside 16 MFMAs of 32 cycles, and by what the power limit leaves of the clock (1.6 - 1.8 GHz): every instruction that goes
// counts.  Measured in the step (PRE), against 109 vector instructions per tile (maxima of the scores, separate addresses of K and
// V): 7200 queries x 57600 keys x 10 heads 1088 -> 1010 us (1050 TFLOP/s), 1800 x 14400 x 20 160 -> 147, 4096 x 16384 x 10 (strips)
// 189 -> 175; queries without the scale, fresh and stale rows: the layer of 1024 of 4096 tokens x 10 heads 51.3 -> 49.5.
// Fresh and stale rows (kSrcRows, kSrcPeriodic): the splice is resolved in the source addresses of the direct loads, lane by
// lane; V is transposed by ds_read_b64_tr_b16 on its way from LDS to the registers.
// 1024 of 4096 tokens x 10 heads: 35 -> 29 us with the merge, against staging through registers.
// Where K and V come from: all stale, V transposed (V^T); rows of the fresh and the stale tensors, the fresh ones a range of keys
// (kSrcRows) or periodic (kSrcPeriodic)
enum { kSrcVt = 0, kSrcRows = 1, kSrcPeriodic = 2 };

template <bool PRE, int SRC>
__global__ __launch_bounds__(256, 2) void attn_pipe_d64(const bf16_t* q, const bf16_t* ks, const bf16_t* vs, int Lq, int L, unsigned int heads_splits, int keys_per_split,
                                                        int ldq, int ldks, int ldv, int nwg, AttnParams p) {
  // (leading arguments come in scalar registers, see wgemm.hip; ldv: the pitch of V^T or of the stale V)
  const int heads = (int)(heads_splits & 0xffffff), nsplit = (int)(heads_splits >> 24);
  constexpr int D = 64, TK = 64, KB = TK * D * 2;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int xor32 = (lane ^ 32) << 2;
  const int g = lane >> 5, c = lane & 31;
  const int csig = (c & 0x13) | ((c & 4) << 1) | ((c & 8) >> 1);
  int t = blockIdx.x;
  {
    const int xcd = t & 7, loc = t >> 3;
    const int base = nwg >> 3, rem = nwg & 7;
    t = xcd * base + (xcd < rem ? xcd : rem) + loc;
  }
  const int nqb = (Lq + 127) / 128;
  const int qb = t % nqb;
  const int h = (t / nqb) % heads;
  const int zz = t / (nqb * heads);
  const int b = zz / nsplit, split = zz % nsplit;
  const int q0 = qb * 128 + wave * 32;
  const int kv_lo = split * keys_per_split;              // multiple of 64
  int kv_hi = kv_lo + keys_per_split;
  if (kv_hi > L) kv_hi = L;
  const int ntiles = (kv_hi - kv_lo + TK - 1) / TK;

  const bf16_t *kg = ks + h * D, *vg = vs + (SRC == kSrcVt ? (long long)h * D * ldv : (long long)h * D), *qg = q + h * D;
  if (b > 0) {
    asm volatile("");
    kg += (long long)b * p.bsks; vg += (long long)b * p.bsvs; qg += (long long)b * p.bsq;
  }
  const bf16_t* kfr = (const bf16_t*)p.kf + (long long)b * p.bskf + h * D;
  const bf16_t* vfr = (const bf16_t*)p.vf + (long long)b * p.bsvf + h * D;

  // direct loads: instruction j of a wave covers tile rows (2*wave + j)*8 + lane/8, 16-byte slot lane%8.  K tiles are
  // [key][d], row r holding chunk c at slot c ^ ((r >> 1) & 7).  V^T tiles are [d][key]; V tiles (fresh and stale rows) [key][d]
  // with a swizzle for the transposing reads.
  const int lr = lane >> 3, slot8 = lane & 7;
  int trow[2], kch[2], vch[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int row = (2 * wave + j) * 8 + lr;
    trow[j] = row;
    kch[j] = (slot8 ^ ((row >> 1) & 7)) * 8;
    vch[j] = SRC == kSrcVt ? kch[j] : (slot8 ^ (((row >> 1) & 1) * 2) ^ (((row >> 3) & 1) * 4)) * 8;
  }
  // offsets inside a tile whose rows are consecutive in one tensor (32-bit, the launcher bounds the pitches)
  unsigned int kofs[2], vofs[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    kofs[j] = (unsigned int)trow[j] * (unsigned int)ldks + (unsigned int)kch[j];
    vofs[j] = (unsigned int)trow[j] * (unsigned int)ldv + (unsigned int)vch[j];
  }
  // kSrcVt: kofr are the offsets inside the last tile when it is ragged
  unsigned int kofr[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int left = L - 1 - (kv_lo + (ntiles - 1) * TK);
    kofr[j] = (unsigned int)(trow[j] < left ? trow[j] : left) * (unsigned int)ldks + (unsigned int)kch[j];
  }
  // Byte offsets of the K loads (kSrcVt) of the tile requested next; those of the last tile from the iteration that requests it on
  unsigned int kcur[2];
  // Direct load j of the wave, of tile ti of K (V: of V or V^T), to LDS.  Fresh and stale rows are told apart lane by lane: with
  // branches for tiles that lie on one side the layer of 1024 of 4096 tokens took 52.1 us instead of 49.5 (a wave that has its
  // SIMD to itself waits out every branch).
  auto load_tile = [&](auto isv, int ti, int j, const char* to) {
    constexpr bool V = decltype(isv)::value;
    const int key0 = kv_lo + ti * TK;
    if constexpr (SRC == kSrcVt) {
      lds_load16(V ? vg + key0 : kg + (long long)key0 * ldks, V ? 2u * vofs[j] : kcur[j], to);
      return;
    }
    // rows beyond the last key re-read it (masked)
    unsigned int key = (unsigned int)(key0 + trow[j] < L ? key0 + trow[j] : L - 1), row = key - (unsigned int)p.own_lo;
    bool own = row < (unsigned int)p.own_n;
    if constexpr (SRC == kSrcPeriodic) {
      // key = q * P + r, q from the rounded-down reciprocal (at most one too small)
      unsigned int q = __umulhi(key, p.own_magic), rr = key - q * (unsigned int)p.own_period;
      if (rr >= (unsigned int)p.own_period) { ++q; rr -= (unsigned int)p.own_period; }
      row = rr - (unsigned int)p.own_lo;
      own = row < (unsigned int)p.own_n;
      row += q * (unsigned int)p.own_n;
    }
    row = own ? row : key;
    if constexpr (V) lds_load16((own ? vfr : vg) + (unsigned long long)row * (unsigned int)(own ? p.ldvf : ldv) + vch[j], to);
    else lds_load16((own ? kfr : kg) + (unsigned long long)row * (unsigned int)(own ? p.ldkf : ldks) + kch[j], to);
  };
  using IsK = std::false_type;
  using IsV = std::true_type;
  bf16x8 qreg[4];
  {
    const int qi = q0 + c;
    const bf16_t* qp = qg + (long long)qi * ldq;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      u32x4 tq = {0u, 0u, 0u, 0u};
      if (qi < Lq) tq = *reinterpret_cast<const u32x4*>(qp + 16 * s + 8 * g);
      qreg[s] = __builtin_bit_cast(bf16x8, tq);
    }
  }
  // LDS: a ring of three slots, a K tile and a V tile each.  Slot i % 3 takes K_i and V_{i+1}, so an iteration reads its K and its V
  // in one slot and refills another.
  constexpr int SLOT = 2 * KB;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const int ti = i < ntiles ? i : ntiles - 1;            // past the end: the last tile again (keeps vmcnt uniform)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      kcur[j] = 2u * (ti == ntiles - 1 ? kofr[j] : kofs[j]);
      load_tile(IsK{}, ti, j, smem + i * SLOT + (2 * wave + j) * 1024);
    }
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    load_tile(IsV{}, 0, j, smem + 2 * SLOT + KB + (2 * wave + j) * 1024);
    kcur[j] = 2u * (ntiles - 1 <= 3 ? kofr[j] : kofs[j]);
  }

  // LDS byte offsets of this lane's fragments inside a tile, the same for K (MFMA row c, which is key csig, of key block kb; k-step s)
  // and V^T (feature csig of feature block db; key step ts).  The second block is 4096 bytes on.
  int kof[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) kof[i] = csig * (D * 2) + (((2 * i + g) ^ ((csig >> 1) & 7)) * 16);
  // V rows: a transposing read hands 16 lanes four keys of 16 features: lane i supplies the address of key i / 4, features 4 * (i
  // % 4) .., and receives feature i.  Chunks 1 and 2 are exchanged (csig), key + 8 g; the second feature block is slot ^ 4.
  const int tri = lane & 15;
  const int vtr = (8 * g + (tri >> 2)) * (D * 2) + (((2 * (c >> 4) + (tri & 1)) ^ (2 * ((tri >> 3) & 1)) ^ (4 * g)) * 16) + ((tri >> 1) & 1) * 8;
  const char* const lds = smem;

  f32x16 o_acc[2], sa[2], cinit;
#pragma unroll
  for (int e = 0; e < 16; ++e) { o_acc[0][e] = 0.f; o_acc[1][e] = 0.f; cinit[e] = 0.f; }
  float m_run = -INFINITY, l_run = 0.f;
  const float sc = PRE ? 1.0f : p.sc_log2;
  u32x4 pk[4];                                             // packed probabilities of the previous tile
#pragma unroll
  for (int i = 0; i < 4; ++i) pk[i] = u32x4{0u, 0u, 0u, 0u};

  auto max8 = [&](const f32x16& s, int h, float a) {       // maximum with accumulators 8h .. 8h+7
    a = fmaxf(fmaxf(a, s[8 * h]), s[8 * h + 1]);
    a = fmaxf(fmaxf(a, s[8 * h + 2]), s[8 * h + 3]);
    a = fmaxf(fmaxf(a, s[8 * h + 4]), s[8 * h + 5]);
    return fmaxf(fmaxf(a, s[8 * h + 6]), s[8 * h + 7]);
  };
  auto vfrag = [&](int base, int ts, int db) { return *reinterpret_cast<const u32x4*>(lds + (base + kof[ts]) + KB + 4096 * db); };
  // The eight V fragments of a tile of rows ([2 * ts + db], low and high half), requested by vrequest() and there after
  // varrive<1>() (key steps 0 and 1) and varrive<2>() (2 and 3), which name every register again: the compiler's own
  // transposing read waits for all global loads in flight (it takes them for possible writers of the tile).
  struct VTile { u32x2 r[16]; };
  auto vrequest = [&](int base, VTile& v) {
    const unsigned int a0 = (unsigned int)(uintptr_t)DF_LPTR(lds + base + KB + vtr), a1 = (unsigned int)(uintptr_t)DF_LPTR(lds + base + KB + (vtr ^ 64));
#define DF_TR(o, a, off) "ds_read_b64_tr_b16 %" #o ", %" #a " offset:" #off "\n\t"
    asm volatile(DF_TR(0, 16, 0) DF_TR(1, 16, 512) DF_TR(2, 17, 0) DF_TR(3, 17, 512)
                 DF_TR(4, 16, 2048) DF_TR(5, 16, 2560) DF_TR(6, 17, 2048) DF_TR(7, 17, 2560)
                 DF_TR(8, 16, 4096) DF_TR(9, 16, 4608) DF_TR(10, 17, 4096) DF_TR(11, 17, 4608)
                 DF_TR(12, 16, 6144) DF_TR(13, 16, 6656) DF_TR(14, 17, 6144) DF_TR(15, 17, 6656)
                 : "=&v"(v.r[0]), "=&v"(v.r[1]), "=&v"(v.r[2]), "=&v"(v.r[3]), "=&v"(v.r[4]), "=&v"(v.r[5]), "=&v"(v.r[6]), "=&v"(v.r[7]),
                   "=&v"(v.r[8]), "=&v"(v.r[9]), "=&v"(v.r[10]), "=&v"(v.r[11]), "=&v"(v.r[12]), "=&v"(v.r[13]), "=&v"(v.r[14]), "=&v"(v.r[15])
                 : "v"(a0), "v"(a1) : "memory");
#undef DF_TR
  };
  auto varrive = [&](VTile& v, auto half) {
    if constexpr (decltype(half)::value == 1)
      asm volatile("s_waitcnt lgkmcnt(8)" : "+v"(v.r[0]), "+v"(v.r[1]), "+v"(v.r[2]), "+v"(v.r[3]), "+v"(v.r[4]), "+v"(v.r[5]), "+v"(v.r[6]), "+v"(v.r[7]) :: "memory");
    else
      asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(v.r[8]), "+v"(v.r[9]), "+v"(v.r[10]), "+v"(v.r[11]), "+v"(v.r[12]), "+v"(v.r[13]), "+v"(v.r[14]), "+v"(v.r[15]) :: "memory");
  };
  auto vof8 = [&](const VTile& v, int ts, int db) {
    const u32x2 lo = v.r[4 * ts + 2 * db], hi = v.r[4 * ts + 2 * db + 1];
    return u32x4{lo.x, lo.y, hi.x, hi.y};
  };
  using H1 = std::integral_constant<int, 1>;
  using H2 = std::integral_constant<int, 2>;
  auto kfrag = [&](int base, int s, int kb) { return *reinterpret_cast<const u32x4*>(lds + (base + kof[s]) + 4096 * kb); };
  auto pv_mfma = [&](u32x4 v, int ts, int db) {
    o_acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, v), __builtin_bit_cast(bf16x8, pk[ts]), o_acc[db], 0, 0, 0);
  };
  auto s_mfma = [&](u32x4 k, int s, int kb) {
    sa[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, k), qreg[s], s == 0 ? cinit : sa[kb], 0, 0, 0);
  };
  auto sync_tile = [&](auto vmc) {
    constexpr int VM = decltype(vmc)::value;
    __builtin_amdgcn_s_waitcnt((VM & 0xF) | ((VM >> 4) << 14) | (0x7 << 4) | (0 << 8));   // vmcnt(VM) lgkmcnt(0)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
#define DF_FENCE __builtin_amdgcn_sched_barrier(0)

  // S_0
  sync_tile(std::integral_constant<int, 0>{});
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) s_mfma(kfrag(0, s, kb), s, kb);
  sync_tile(std::integral_constant<int, 0>{});             // every wave has read K_0: its slot takes K_3

  int base = SLOT, dst = 0;                                // slots: of K_{tl+1} and V_{tl-1}, of K_{tl+3} and V_{tl+1}
  int tl = 0;
  auto advance = [&] {
    dst = base;
    base = base == 2 * SLOT ? 0 : base + SLOT;
    ++tl;
  };
  const bool ragged = (kv_hi - kv_lo) % TK != 0;
  const int nfull = ragged ? ntiles - 1 : ntiles;
  float m_base = 0.f;                                      // what the scores in sa are relative to (PRE)
  // Maximum of 32 scores per lane and of the other half of the query's: the running maximum that covers them.
  auto settle = [&](const f32x16& s0, const f32x16& s1) {
    const float mx = max8(s1, 1, max8(s1, 0, max8(s0, 1, max8(s0, 0, -INFINITY))));
    const float part = __int_as_float(__builtin_amdgcn_ds_bpermute(xor32, __float_as_int(mx)));
    return fmaxf(m_run, PRE ? fmaxf(mx, part) + m_base : fmaxf(mx, part) * sc);
  };
  // Everything to the new maximum; returns what is to be added to scores that are relative to the old one (PRE)
  auto move_to = [&](float m_new) {
    const float shift = m_base - m_new;
    if constexpr (PRE) {
#pragma unroll
      for (int e = 0; e < 16; ++e) { sa[0][e] += shift; sa[1][e] += shift; cinit[e] = -m_new; }
      m_base = m_new;
    }
    const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
#pragma unroll
    for (int e = 0; e < 16; ++e) { o_acc[0][e] *= alpha; o_acc[1][e] *= alpha; }
    l_run *= alpha;
    m_run = m_new;
    return shift;
  };

  // Tile tl: its probabilities from the scores in sa (in place: a key block's registers take S of tile tl+1 as soon as
  // its exponentials are done), O += V P of tile tl-1 (PV), S of tile tl+1.  One matrix instruction and its share of
  // vector instructions per slot; operand fragments are read from LDS five slots ahead.  Returns the tile's row sums.
  auto tile = [&](auto pvc) {
    constexpr bool PV = decltype(pvc)::value;
    u32x4 f[16];
    VTile vt;
    if constexpr (PV && SRC == kSrcVt) {
#pragma unroll
      for (int i = 0; i < 5; ++i) f[i] = vfrag(base, i >> 1, i & 1);
    }
    if constexpr (PV && SRC != kSrcVt) vrequest(base, vt);
    auto vread = [&](int ts, int db) { return PV && SRC == kSrcVt ? vfrag(base, ts, db) : u32x4{0u, 0u, 0u, 0u}; };
    auto pv = [&](const u32x4& ahead, int ts, int db) {
      if constexpr (PV) pv_mfma(SRC == kSrcVt ? ahead : vof8(vt, ts, db), ts, db);
    };
    float ex[2][8];
    auto E = [&](int u, int h) {                           // four exponentials of key step u
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float x = sa[u >> 1][8 * (u & 1) + 4 * h + q];
        ex[u & 1][4 * h + q] = __builtin_amdgcn_exp2f(PRE ? x : fmaf(x, sc, -m_run));
      }
    };
    unsigned int w[2][4];
    auto C = [&](int u) {                                  // packing (after the matrix instructions of key step u read pk[u])
#pragma unroll
      for (int q = 0; q < 4; ++q) w[u & 1][q] = pack_bf2(ex[u & 1][2 * q], ex[u & 1][2 * q + 1]);
      pk[u] = u32x4{w[u & 1][0], w[u & 1][1], w[u & 1][2], w[u & 1][3]};
      asm volatile("" : "+v"(pk[u]));                    // (stays here: the branch behind the tile may replace it)
    };
    float tsum = 0.f;
    auto S = [&](int u) {                                  // row sums
      const float* e = ex[u & 1];
      const float t = ((e[0] + e[1]) + (e[2] + e[3])) + ((e[4] + e[5]) + (e[6] + e[7]));
      tsum = u == 0 ? t : tsum + t;
      asm volatile("" : "+v"(tsum));
    };
    const int tk3 = tl + 3 < ntiles ? tl + 3 : ntiles - 1, tv1 = tl + 1 < ntiles ? tl + 1 : ntiles - 1;
    auto dma_k = [&](int j) { load_tile(IsK{}, tk3, j, smem + dst + (2 * wave + j) * 1024); };
    auto dma_v = [&](int j) { load_tile(IsV{}, tv1, j, smem + dst + KB + (2 * wave + j) * 1024); };
    DF_FENCE;
    if constexpr (SRC != kSrcVt && PV) { E(0, 0); E(0, 1); DF_FENCE; varrive(vt, H1{}); DF_FENCE; }
    pv(f[0], 0, 0); f[5] = vread(2, 1); if constexpr (SRC == kSrcVt || !PV) E(0, 0); DF_FENCE;
    pv(f[1], 0, 1); f[6] = kfrag(base, 0, 0); if constexpr (SRC == kSrcVt || !PV) E(0, 1); dma_k(0); DF_FENCE;
    pv(f[2], 1, 0); f[7] = vread(3, 0); C(0); dma_k(1); DF_FENCE;
    pv(f[3], 1, 1); f[8] = kfrag(base, 1, 0); E(1, 0); DF_FENCE;
    if constexpr (SRC != kSrcVt && PV) { varrive(vt, H2{}); DF_FENCE; }
    pv(f[4], 2, 0); f[9] = vread(3, 1); E(1, 1); DF_FENCE;
    pv(f[5], 2, 1); f[10] = kfrag(base, 2, 0); C(1); S(0); DF_FENCE;
    s_mfma(f[6], 0, 0); f[11] = kfrag(base, 3, 0); E(2, 0); DF_FENCE;
    pv(f[7], 3, 0); f[12] = kfrag(base, 0, 1); E(2, 1); S(1); DF_FENCE;
    s_mfma(f[8], 1, 0); f[13] = kfrag(base, 1, 1); C(2); dma_v(0); DF_FENCE;
    pv(f[9], 3, 1); f[14] = kfrag(base, 2, 1); E(3, 0); DF_FENCE;
    s_mfma(f[10], 2, 0); f[15] = kfrag(base, 3, 1); E(3, 1); dma_v(1); DF_FENCE;
    s_mfma(f[11], 3, 0); S(2); DF_FENCE;
    s_mfma(f[12], 0, 1); C(3); DF_FENCE;
    s_mfma(f[13], 1, 1); S(3); DF_FENCE;
    s_mfma(f[14], 2, 1); DF_FENCE;
    s_mfma(f[15], 3, 1);
    if (SRC == kSrcVt && tl + 4 == ntiles - 1) {           // the next iteration requests the last tile
#pragma unroll
      for (int j = 0; j < 2; ++j) { kcur[j] = 2u * kofr[j]; asm volatile("" : "+v"(kcur[j])); }
    }
    sync_tile(std::integral_constant<int, 4>{});           // K_{tl+1} and V_{tl-1} of the next tile have landed, for every wave
    return tsum;
  };
  constexpr float kMove = 0x1p13f, kRedo = 0x1p100f;
  // A tile with probabilities far above 1: its scores once more, from memory (K's slot is taken), and its probabilities and the
  // sums relative to a maximum that covers them.  Nothing has read them yet.
  auto redo = [&]() {
    f32x16 t[2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      const int key = kv_lo + tl * TK + 32 * kb + key_of_mfma_row(c);
      const long long fr = SRC == kSrcVt ? -1 : fresh_row(p.own_lo, p.own_n, SRC == kSrcPeriodic ? p.own_period : 0, key);
      const bf16_t* kr = (fr >= 0 ? kfr + fr * p.ldkf : kg + (long long)key * ldks) + 8 * g;
#pragma unroll
      for (int s = 0; s < 4; ++s)
        t[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(kr + 16 * s)), qreg[s],
                                                        s == 0 ? cinit : t[kb], 0, 0, 0);
    }
    const float shift = move_to(settle(t[0], t[1]));
    float tsum = 0.f;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      float e[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const float x = t[u >> 1][8 * (u & 1) + q];
        e[q] = __builtin_amdgcn_exp2f(PRE ? x + shift : fmaf(x, sc, -m_run));
        tsum += e[q];
      }
      pk[u] = u32x4{pack_bf2(e[0], e[1]), pack_bf2(e[2], e[3]), pack_bf2(e[4], e[5]), pack_bf2(e[6], e[7])};
    }
    return tsum;
  };

  // A tile with a large sum that its probabilities and the sum still hold: m up by the power of two above it, for the query's two lanes.
  // Returns the sum on the scale of the probabilities, by which m moves as well but for rounding (a whole step from 2^24 on).
  auto lower = [&](float tsum) {
    const float part = __int_as_float(__builtin_amdgcn_ds_bpermute(xor32, __float_as_int(tsum)));
    const float s = fmaxf(tsum, part);
    const int k = s > kMove ? __builtin_amdgcn_frexp_expf(s) : 0;
    const float scale = __builtin_amdgcn_ldexpf(1.0f, -k);
    move_to(m_run + (float)k);
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float lo = __uint_as_float(pk[u][q] << 16) * scale, hi = __uint_as_float(pk[u][q] & 0xffff0000u) * scale;
        pk[u][q] = __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
      }
    return tsum * scale;
  };

  bool again = false;                                      // tile tl has a large sum (NaN passes on as it is)
  float tsum = 0.f;
  auto values = [&](bool last) {                           // O += V P of the pending tile
    VTile vt;
    if constexpr (SRC != kSrcVt) { vrequest(base, vt); varrive(vt, H1{}); varrive(vt, H2{}); }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int ts = i >> 1;
      u32x4 v = SRC == kSrcVt ? vfrag(base, ts, i & 1) : vof8(vt, ts, i & 1);
      if (last && ragged) {                                // keys beyond the range: P is 0, V must be finite
        const int key = kv_lo + (ntiles - 1) * TK + (2 * ts + g) * 8;
        if (key + 0 >= kv_hi) v.x = 0u; else if (key + 1 >= kv_hi) v.x &= 0xffffu;
        if (key + 2 >= kv_hi) v.y = 0u; else if (key + 3 >= kv_hi) v.y &= 0xffffu;
        if (key + 4 >= kv_hi) v.z = 0u; else if (key + 5 >= kv_hi) v.z &= 0xffffu;
        if (key + 6 >= kv_hi) v.w = 0u; else if (key + 7 >= kv_hi) v.w &= 0xffffu;
      }
      pv_mfma(v, ts, i & 1);
    }
  };
  for (;;) {
    if (again) {
      // (the sums of the tiles before move with m, so this tile's is added behind)
      const float sum = __builtin_amdgcn_ballot_w64(tsum > kRedo) ? redo() : lower(tsum);
      l_run += sum;
      advance();
      if (tl >= ntiles) break;
    }
    if (tl == 0 || tl >= nfull) {
      // First tile, or the ragged last one: settle the pending tile's values, mask the keys beyond the range, move the running
      // maximum and rescale everything to it.
      if (ragged && tl == ntiles - 1) {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int e = 0; e < 16; ++e)
            if (kv_lo + tl * TK + 32 * kb + 16 * (e >> 3) + 8 * g + (e & 7) >= kv_hi) sa[kb][e] = -INFINITY;
      }
      if (tl > 0) values(false);
      move_to(settle(sa[0], sa[1]));
      l_run += tile(std::false_type{});
      advance();
    }
    again = false;
    while (tl < nfull) {
      tsum = tile(std::true_type{});
      again = __builtin_amdgcn_ballot_w64(tsum > kMove) != 0;
      if (again) break;
      l_run += tsum;
      advance();
    }
    if (!again && tl >= ntiles) break;
  }
  // the last tile's values
  sync_tile(std::integral_constant<int, 0>{});
  values(true);
#undef DF_FENCE
  l_run += __int_as_float(__builtin_amdgcn_ds_bpermute(xor32, __float_as_int(l_run)));

  const int qi = q0 + c;
  if (qi >= Lq) return;
  if (nsplit == 1) {
    const float inv = 1.0f / l_run;
    bf16_t* op = (bf16_t*)p.out + (long long)b * p.bso + (long long)qi * p.ldo + h * D;
    const long long m = (long long)b * Lq + qi;
    bf16_t* pp = (bf16_t*)p.out + (((m >> 5) * (long long)(heads * D / 16) + h * (D / 16)) * 64 + (m & 31) + 32 * g) * 8;
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        u32x4 tq;
        tq.x = pack_bf2(o_acc[db][8 * f + 0] * inv, o_acc[db][8 * f + 1] * inv);
        tq.y = pack_bf2(o_acc[db][8 * f + 2] * inv, o_acc[db][8 * f + 3] * inv);
        tq.z = pack_bf2(o_acc[db][8 * f + 4] * inv, o_acc[db][8 * f + 5] * inv);
        tq.w = pack_bf2(o_acc[db][8 * f + 6] * inv, o_acc[db][8 * f + 7] * inv);
        if (p.out_packed) *reinterpret_cast<u32x4*>(pp + (2 * db + f) * 512) = tq;
        else *reinterpret_cast<u32x4*>(op + 32 * db + 16 * f + 8 * g) = tq;
      }
  } else {
    const long long row = (((long long)split * p.B + b) * heads + h) * Lq + qi;
    float* po = p.part_o + row * D;
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        f32x4 t0 = {o_acc[db][8 * f], o_acc[db][8 * f + 1], o_acc[db][8 * f + 2], o_acc[db][8 * f + 3]};
        f32x4 t1 = {o_acc[db][8 * f + 4], o_acc[db][8 * f + 5], o_acc[db][8 * f + 6], o_acc[db][8 * f + 7]};
        *reinterpret_cast<f32x4*>(po + 32 * db + 16 * f + 8 * g) = t0;
        *reinterpret_cast<f32x4*>(po + 32 * db + 16 * f + 8 * g + 4) = t1;
      }
    if (g == 0) {
      p.part_ml[row * 2] = m_run;
      p.part_ml[row * 2 + 1] = l_run;
    }
  }
}

// Workgroups of attn_wave_d64's launch beyond its query blocks: each XCD's read that XCD's eighth of every region once and drop it.
template <int NW>
__device__ __forceinline__ void read_ahead(const AttnParams& p, int row) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int xcd = blockIdx.x & 7, rows = (int)gridDim.y - p.qblocks, cols = (int)gridDim.x >> 3;   // (gridDim.x: a multiple of 8)
  const int first = (((int)blockIdx.z * rows + row) * cols + ((int)blockIdx.x >> 3)) * NW + wave;
  const int stride = (int)gridDim.z * rows * cols * NW;
  for (int r = 0; r < p.next.n; ++r) {
    const long long kb = p.next.bytes[r] >> 10, lo = kb * xcd / 8;
    const int n = (int)(kb * (xcd + 1) / 8 - lo);
    const char* base = (const char*)p.next.p[r] + (lo << 10) + lane * 16;
    for (int i = first; i < n; i += 4 * stride) {
      u32x4 t[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = i + u * stride;
        t[u] = *reinterpret_cast<const u32x4*>(base + ((long long)(k < n ? k : i) << 10));
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) asm volatile("" ::"v"(t[u]));
    }
  }
}

// Self-attention of a patch with few queries (the deepest levels: 32-1024 query rows against the whole image's keys).
// One workgroup = one 32-query block of one head; its NW waves take contiguous runs of 64-key tiles and merge their
// (max, sum, O) states through LDS at the end, so nothing is split across workgroups and no second kernel runs.
// Nothing is shared between waves inside the loop: every wave stages its own K and V^T tiles (global -> LDS with
// direct loads, 1 KB contiguous per instruction; a wave reading its MFMA operands straight from the row-major buffers
// touches 32 cache lines per instruction and ran at a quarter of the rate) in a private 16 KB of LDS, so the loop has no
// barrier: the fragments of V of tile i and of K of tile i + 1 go LDS -> registers, then the loads of V of tile i + 1 and K
// of tile i + 2 are issued into the same LDS while the scores of tile i + 1 are on the matrix cores and the
// exponentials of tile i on the vector ALU.  Same operand conventions and swizzles as attn_pipe_d64.
// Two waves share a SIMD, and the one launched first took the issue slots: the later half carries the higher wave
// priority.  300 queries x 2400 keys x 20 heads, cold keys: 17.7 us; scores a tile ahead 16.5; priority 15.5.  Of these the
// launch takes 1.5, the first tiles' way from HBM 3 (12 MB of keys for all heads), the merge 1; a round of eight tiles takes
// 1.3 us where its 128 KB need 1.2 at the rate that L2 fills a compute unit (52 B per clock).
template <int NW, bool HEAD_BY_HEAD>
__global__ __launch_bounds__(64 * NW, 2) void attn_wave_d64(const bf16_t* q, const bf16_t* ks, const bf16_t* vs, int Lq, int L, int heads, int qblocks,
                                                             int ldq, int ldks, int vt_ld, unsigned int qb_recip, AttnParams p) {
  constexpr int D = 64, TK = 64;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  DF_ATRACE(0, wall_clock64());
  DF_ATRACE(1, __builtin_readcyclecounter());
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int xor32 = (lane ^ 32) << 2;
  const int g = lane >> 5, c = lane & 31;
  const int csig = (c & 0x13) | ((c & 4) << 1) | ((c & 8) >> 1);
  // Grid (heads rounded up to a multiple of 8, query blocks, batch): workgroups go round-robin over the 8 XCDs in
  // x-fastest order, so every query block of head h runs on XCD h % 8 and the blocks of a head, which read the same
  // K / V^T, share an L2 - without any index arithmetic (the divisions of a linear index were a tenth of this kernel).
  // That leaves the XCDs of the first heads % 8 a head more: where they do not hold it in one round, blocks are counted instead (700 queries x
  // 1400 keys x 20 heads, 66 of 64 places, 23.8 -> 16.1 us; 352 x 704 x 20, 33 of 32, 10.9 -> 8.5).
  int h = blockIdx.x, qb = blockIdx.y, b = blockIdx.z;
  if constexpr (HEAD_BY_HEAD) {
    const unsigned int xcd = blockIdx.x & 7, base = gridDim.x >> 3, rem = gridDim.x & 7;
    const unsigned int t = xcd * base + (xcd < rem ? xcd : rem) + (blockIdx.x >> 3);
    h = (int)quotient_u32(t, (unsigned int)qblocks, qb_recip);
    qb = (int)t - h * qblocks;
    b = h < heads ? 0 : h / heads;
    h -= b * heads;
  } else {
    if (qb >= qblocks) { read_ahead<NW>(p, qb - qblocks); return; }
    if (h >= heads) return;
  }
  const int q0 = qb * 32;
  const int NT = (L + TK - 1) / TK;
  const int t_lo = (int)((long long)wave * NT / NW), t_hi = (int)((long long)(wave + 1) * NT / NW);

  const bf16_t *kg = ks + h * D, *vg = vs + (long long)h * D * vt_ld, *qg = q + h * D;
  if (b > 0) {                                               // (the strides are not among the arguments that come in registers)
    asm volatile("");
    kg += (long long)b * p.bsks; vg += (long long)b * p.bsvs; qg += (long long)b * p.bsq;
  }

  bf16x8 qreg[4];
  {
    const int qi = q0 + c;
    const bf16_t* qp = qg + (long long)qi * ldq;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      u32x4 tq = {0u, 0u, 0u, 0u};
      if (qi < Lq) tq = *reinterpret_cast<const u32x4*>(qp + 16 * s + 8 * g);
      qreg[s] = __builtin_bit_cast(bf16x8, tq);
    }
  }
  // direct loads: instruction j of the wave covers tile rows j*8 + lane/8, 16-byte slot lane%8 (swizzled on the source
  // side); a lane's offsets inside a tile never change (32-bit, the launcher bounds the pitches)
  const int lr = lane >> 3, slot = lane & 7;
  unsigned int kofs[8], vofs[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int row = j * 8 + lr;
    kofs[j] = (unsigned int)row * (unsigned int)ldks + (unsigned int)((slot ^ ((row >> 1) & 7)) * 8);
    vofs[j] = (unsigned int)row * (unsigned int)vt_ld + (unsigned int)((slot ^ (row & 7) ^ (row >> 3)) * 8);
  }
  char* sk = smem + wave * (2 * TK * D * 2);                 // this wave's K tile [key][d], then its V^T tile [d][key]
  char* sv = sk + TK * D * 2;
  auto issue_k = [&](int tl) {
    const int key0 = tl * TK;
    if (key0 + TK <= L) {                                  // (uniform) every key row of the tile exists
      const bf16_t* kb0 = kg + (long long)key0 * ldks;
#pragma unroll
      for (int j = 0; j < 8; ++j) lds_load16(kb0, 2u * kofs[j], sk + j * 1024);
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int row = j * 8 + lr;
        int key = key0 + row;
        if (key > L - 1) key = L - 1;                    // rows beyond the last key are masked in the tile body
        lds_load16(kg + (long long)key * ldks + ((slot ^ ((row >> 1) & 7)) * 8), sk + j * 1024);
      }
    }
  };
  auto issue_v = [&](int tl) {
    const bf16_t* vb0 = vg + tl * TK;                        // the V^T buffer is padded to whole tiles
#pragma unroll
    for (int j = 0; j < 8; ++j) lds_load16(vb0, 2u * vofs[j], sv + j * 1024);
  };
  bf16x8 kfr[2][4];
  u32x4 vfr[4][2];
  auto read_k = [&]() {
    const bf16_t* Ks = reinterpret_cast<const bf16_t*>(sk);
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      const int row = 32 * kb + key_of_mfma_row(c);
      const int f = (row >> 1) & 7;
#pragma unroll
      for (int s = 0; s < 4; ++s) kfr[kb][s] = *reinterpret_cast<const bf16x8*>(&Ks[row * D + (((2 * s + g) ^ f) * 8)]);
    }
  };
  auto read_v = [&]() {
    const bf16_t* Vt = reinterpret_cast<const bf16_t*>(sv);
#pragma unroll
    for (int ts = 0; ts < 4; ++ts) {
      const int kchunk = 4 * (ts >> 1) + 2 * (ts & 1) + g;
#pragma unroll
      for (int db = 0; db < 2; ++db) {
        const int d = 32 * db + csig;
        vfr[ts][db] = *reinterpret_cast<const u32x4*>(&Vt[d * TK + (kchunk ^ (d & 7) ^ (d >> 3)) * 8]);
      }
    }
  };

  f32x16 o_acc[2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) o_acc[i][e] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  const float sc = p.sc_log2;

  auto scores = [&](f32x16 (&s_acc)[2]) {                    // S^T of the tile whose K fragments are in registers
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int e = 0; e < 16; ++e) s_acc[kb][e] = 0.f;
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
        s_acc[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kfr[kb][s], qreg[s], s_acc[kb], 0, 0, 0);
  };
  auto new_max = [&](const f32x16 (&s_acc)[2]) {
    float mx = -INFINITY;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int e = 0; e < 16; ++e) mx = fmaxf(mx, s_acc[kb][e]);
    const auto halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
    mx = fmaxf(__uint_as_float(halves[0]), __uint_as_float(halves[1])) * sc;
    return fmaxf(m_run, mx);                                 // finite: a tile holds at least one key
  };
  // P of 16 keys (MFMA operand) from their scores, the row sums on the way
  auto probs = [&](f32x16 (&s_acc)[2], int ts, float m_new, float& rs) {
    const int kb = ts >> 1, half = ts & 1;
    float e8[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      e8[i] = __builtin_amdgcn_exp2f(fmaf(s_acc[kb][8 * half + i], sc, -m_new));
      rs += e8[i];
    }
    const u32x4 pk = {pack_bf2(e8[0], e8[1]), pack_bf2(e8[2], e8[3]), pack_bf2(e8[4], e8[5]), pack_bf2(e8[6], e8[7])};
    return __builtin_bit_cast(bf16x8, pk);
  };
  auto rescale = [&](float m_new) {
    const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
    m_run = m_new;
    l_run *= alpha;                                          // this lane's half of the keys; the halves meet at the end
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) o_acc[i][e] *= alpha;     // (without a branch: a jump here costs copies of all 32)
  };
  // The query blocks of a head read the same keys; started on the same tile they would all wait for the same cache
  // lines while the rest of the head's K / V^T (cold: other patches' rows, last touched a step ago) is not even
  // requested.  Block qb therefore walks each wave's run of tiles from a different starting tile, wrapping around:
  // ten blocks keep ten tiles per wave slot in flight and find the others' tiles in L2.  The order is a fixed
  // function of the indices, so results stay reproducible.  A tile with fewer than 64 keys stays the last.
  const int nt = t_hi - t_lo;
  const int nrot = t_hi * TK > L ? nt - 1 : nt;
  const int rot = ((qb & 7) * nrot) >> 3;                    // < nrot, spread over the run
  auto tile_at = [&](int i) { const int k = i + rot; return t_lo + (i >= nrot ? i : k < nrot ? k : k - nrot); };
  // The scores run one tile ahead: while the exponentials and sums of tile i are on the vector ALU, the matrix cores take
  // the scores of tile i + 1 and the product with V of tile i.
  auto landed = [&]() {
    __builtin_amdgcn_s_waitcnt((0 & 0xF) | (0x7 << 4) | (0xF << 8));   // vmcnt(0): this wave's loads are in its LDS
    asm volatile("" ::: "memory");
  };
  auto in_registers = [&]() {
    __builtin_amdgcn_s_waitcnt((0x3F & 0xF) | ((0x3F >> 4) << 14) | (0x7 << 4) | (0 << 8));   // lgkmcnt(0)
    asm volatile("" ::: "memory");
  };
  auto step = [&](int i, f32x16 (&cur)[2], f32x16 (&nxt)[2]) {
    landed();                                                // V of tile i, K of tile i + 1
    DF_ATRACE(3 + 3 * i, __builtin_readcyclecounter());
    read_k();
    read_v();
    const float m_new = new_max(cur);
    in_registers();
    DF_ATRACE(4 + 3 * i, __builtin_readcyclecounter());
    issue_v(tile_at(i + 1));                                 // into the LDS just read, under this tile's work
    if (i + 2 < nt) issue_k(tile_at(i + 2));                 // (uniform)
    __builtin_amdgcn_sched_barrier(0);
    scores(nxt);
    rescale(m_new);
    float rs = 0.f;
#pragma unroll
    for (int ts = 0; ts < 4; ++ts) {
      const bf16x8 pfrag = probs(cur, ts, m_new, rs);
#pragma unroll
      for (int db = 0; db < 2; ++db)
        o_acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vfr[ts][db]), pfrag, o_acc[db], 0, 0, 0);
    }
    l_run += rs;
    asm volatile("" : "+v"(l_run));                        // (here, not sunk into a later block)
    __builtin_amdgcn_sched_barrier(0);
    DF_ATRACE(5 + 3 * i, __builtin_readcyclecounter());
  };
  f32x16 s_a[2], s_b[2];
  if (wave >= NW / 2) __builtin_amdgcn_s_setprio(1);
  if (nt > 0) {
    issue_k(tile_at(0));
    issue_v(tile_at(0));
    __builtin_amdgcn_s_waitcnt((8 & 0xF) | (0x7 << 4) | (0xF << 8));   // vmcnt(8): K is there
    asm volatile("" ::: "memory");
    read_k();
    in_registers();
    if (nt > 1) issue_k(tile_at(1));
    scores(s_a);
    DF_ATRACE(2, __builtin_readcyclecounter());
    int i = 0;
    for (; i + 2 < nt; i += 2) {
      step(i, s_a, s_b);
      step(i + 1, s_b, s_a);
    }
    if (i + 1 < nt) {
      step(i, s_a, s_b);
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) s_a[kb] = s_b[kb];
      ++i;
    }
    // the last tile: no scores ahead, and it may hold fewer than 64 keys
    const int tile_base = tile_at(i) * TK;
    landed();
    DF_ATRACE(3 + 3 * i, __builtin_readcyclecounter());
    read_v();
    if (tile_base + TK > L) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int j = e >> 2, r = e & 3;
          const int key = tile_base + 32 * kb + 16 * (j >> 1) + 8 * g + 4 * (j & 1) + r;
          if (key >= L) s_a[kb][e] = -INFINITY;
        }
#pragma unroll
      for (int ts = 0; ts < 4; ++ts)
#pragma unroll
        for (int db = 0; db < 2; ++db) {                     // keys beyond the range: P is 0, V must be finite
          const int key = tile_base + (4 * (ts >> 1) + 2 * (ts & 1) + g) * 8;
          u32x4& vraw = vfr[ts][db];
          if (key + 0 >= L) vraw.x = 0u; else if (key + 1 >= L) vraw.x &= 0xffffu;
          if (key + 2 >= L) vraw.y = 0u; else if (key + 3 >= L) vraw.y &= 0xffffu;
          if (key + 4 >= L) vraw.z = 0u; else if (key + 5 >= L) vraw.z &= 0xffffu;
          if (key + 6 >= L) vraw.w = 0u; else if (key + 7 >= L) vraw.w &= 0xffffu;
        }
    }
    const float m_new = new_max(s_a);
    DF_ATRACE(4 + 3 * i, __builtin_readcyclecounter());
    rescale(m_new);
    float rs = 0.f;
#pragma unroll
    for (int ts = 0; ts < 4; ++ts) {
      const bf16x8 pfrag = probs(s_a, ts, m_new, rs);
#pragma unroll
      for (int db = 0; db < 2; ++db)
        o_acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vfr[ts][db]), pfrag, o_acc[db], 0, 0, 0);
    }
    l_run += rs;
    DF_ATRACE(5 + 3 * i, __builtin_readcyclecounter());
  }
  l_run += __int_as_float(__builtin_amdgcn_ds_bpermute(xor32, __float_as_int(l_run)));

  // ---- merge the NW states in wave order ----
  __syncthreads();                                           // every wave is done with its tiles: the LDS is free
  float* mrg = reinterpret_cast<float*>(smem);               // [NW][34][64]: 32 accumulators, max, sum per lane
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) mrg[(wave * 34 + i * 16 + e) * 64 + lane] = o_acc[i][e];
  mrg[(wave * 34 + 32) * 64 + lane] = m_run;
  mrg[(wave * 34 + 33) * 64 + lane] = l_run;
  __syncthreads();
  DF_ATRACE(28, __builtin_readcyclecounter());
  DF_ATRACE(31, nt);
  const int qi = q0 + c;
  if (qi >= Lq) return;
  float mw[NW], m_all = -INFINITY;
#pragma unroll
  for (int w = 0; w < NW; ++w) { mw[w] = mrg[(w * 34 + 32) * 64 + lane]; m_all = fmaxf(m_all, mw[w]); }
  float l_all = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    mw[w] = __builtin_amdgcn_exp2f(mw[w] - m_all);           // a wave without keys has max -inf: weight 0
    l_all = fmaf(mw[w], mrg[(w * 34 + 33) * 64 + lane], l_all);
  }
  const float inv = __builtin_amdgcn_rcpf(l_all);
  // wave w finishes accumulators 4w .. 4w+3 (NW == 8) of every lane: 4 consecutive features of the lane's query
  constexpr int PER = 32 / NW;
  static_assert(PER == 4 || PER == 8, "four or eight waves");
  float o[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) v = fmaf(mw[w], mrg[(w * 34 + wave * PER + k) * 64 + lane], v);
    o[k] = v * inv;
  }
  const int e0 = wave * PER;                                 // accumulator index = 16 * db + 8 * f + e
  const int db = e0 >> 4, f = (e0 >> 3) & 1, eo = e0 & 7;
  bf16_t* dst;
  if (p.out_packed) {
    const long long m = (long long)b * Lq + qi;
    dst = (bf16_t*)p.out + (((m >> 5) * (long long)(heads * D / 16) + h * (D / 16)) * 64 + (m & 31) + 32 * g) * 8 +
          (2 * db + f) * 512 + eo;
  } else {
    dst = (bf16_t*)p.out + (long long)b * p.bso + (long long)qi * p.ldo + h * D + 32 * db + 16 * f + 8 * g + eo;
  }
  if constexpr (PER == 4) {
    u32x2 tq = {pack_bf2(o[0], o[1]), pack_bf2(o[2], o[3])};
    *reinterpret_cast<u32x2*>(dst) = tq;
  } else {
    u32x4 tq = {pack_bf2(o[0], o[1]), pack_bf2(o[2], o[3]), pack_bf2(o[4], o[5]), pack_bf2(o[6], o[7])};
    *reinterpret_cast<u32x4*>(dst) = tq;
  }
  DF_ATRACE(29, __builtin_readcyclecounter());
  DF_ATRACE(30, wall_clock64());
}

// Merges the partial results of NS (or, NS = 8, more) key ranges: eight lanes per query, eight features each, in the order of the
// ranges.  All of them are requested at once: in a loop over the ranges each load waited for the one before it (1800 queries x 20
// heads x 5 ranges 12.4 -> 9.0 us, 7200 x 10 x 4 17.1 -> 13.7, 1024 x 20 x 3 5.5 -> 5.0; a launch and two round trips to memory are some 4).
template <int NS>
__global__ __launch_bounds__(256) void attn_combine_d64(AttnParams p) {
  constexpr int D = 64;
  // 32-bit index arithmetic (the launcher bounds rows * 16 below 2^31): the 64-bit divisions below were a tenth of
  // this kernel's time
  asm volatile("" ::"s"(p.part_o), "s"(p.part_ml), "s"(p.B), "s"(p.heads), "s"(p.Lq), "s"(p.nsplit), "s"(p.out), "s"(p.bso), "s"(p.ldo),
               "s"(p.out_packed));                         // (one batch of argument loads, see wgemm.hip)
  const unsigned int idx = blockIdx.x * 256 + threadIdx.x;
  const unsigned int rows = (unsigned int)(p.B * p.heads * p.Lq);
  if (idx >= rows * (D / 8)) return;
  const unsigned int row = idx / (D / 8);
  const int d8 = (int)(idx % (D / 8)) * 8;
  const f32x2* ml = reinterpret_cast<const f32x2*>(p.part_ml) + row;
  const float* po = p.part_o + (size_t)row * D + d8;
  float m = -INFINITY, l = 0.f;
  f32x4 o0 = {0.f, 0.f, 0.f, 0.f}, o1 = o0;
  for (int s0 = 0; s0 < p.nsplit; s0 += NS) {              // (one round up to eight ranges)
    f32x2 sm[NS];
    f32x4 t0[NS], t1[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int k = s0 + s < p.nsplit ? s0 + s : p.nsplit - 1;
      sm[s] = ml[(size_t)k * rows];
      t0[s] = *reinterpret_cast<const f32x4*>(po + (size_t)k * rows * D);
      t1[s] = *reinterpret_cast<const f32x4*>(po + (size_t)k * rows * D + 4);
    }
    if (s0 == 0) {
#pragma unroll
      for (int s = 0; s < NS; ++s) m = fmaxf(m, sm[s].x);
      for (int s = NS; s < p.nsplit; ++s) m = fmaxf(m, ml[(size_t)s * rows].x);
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      if (s0 + s >= p.nsplit) continue;
      const float w = __builtin_amdgcn_exp2f(sm[s].x - m);
      l += w * sm[s].y;
      o0 += t0[s] * w;
      o1 += t1[s] * w;
    }
  }
  const float inv = __builtin_amdgcn_rcpf(l);
  const unsigned int bh = row / (unsigned int)p.Lq;
  const int qi = (int)(row - bh * (unsigned int)p.Lq);
  const int b = (int)(bh / (unsigned int)p.heads);
  const int h = (int)(bh - (unsigned int)b * (unsigned int)p.heads);
  bf16_t* op = (bf16_t*)p.out + (long long)b * p.bso + (long long)qi * p.ldo + h * D + d8;
  if (p.out_packed) {
    const long long q = (long long)b * p.Lq + qi;
    const int col = h * D + d8;
    op = (bf16_t*)p.out + (((q >> 5) * (long long)(p.heads * D / 16) + (col >> 4)) * 64 + (q & 31) + 32 * ((col >> 3) & 1)) * 8;
  }
  const float v[8] = {o0.x * inv, o0.y * inv, o0.z * inv, o0.w * inv, o1.x * inv, o1.y * inv, o1.z * inv, o1.w * inv};
  st_vec(op, v);
}

// ---- f32 ----
// One workgroup per QN neighbouring queries of a head; its four waves take every fourth step of the keys.  D/4 lanes share a
// key (16-byte loads, the score is summed over them), so a wave's step covers 256/D keys, four of them per lane in flight;
// every group of lanes keeps its own (max, sum, O) and the groups, then the waves, are merged at the end.
// Latency-bound at the sizes it is used at (whole keys per lane and 6 x D shuffles at the end before: 128 queries x
// 256 keys, d = 32: 18.3 -> 5.3 us; 2304 x 9216, d = 64: 513).  QN = 4 reuses the loads of a key for four queries and is taken where one query
// per workgroup would already give every compute unit eight workgroups.
template <int D, int QN>
__global__ __launch_bounds__(256) void attn_f32(AttnParams p) {
  constexpr int LPK = D / 4, KPS = 64 / LPK, U = 4;        // lanes per key, keys per wave step, steps in flight
  __shared__ float red[4][QN][D + 2];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int sub = lane % LPK, grp = lane / LPK;
  const int nqb = (p.Lq + QN - 1) / QN;
  const int q0 = (int)(blockIdx.x % nqb) * QN;
  const int h = (int)((blockIdx.x / nqb) % p.heads);
  const int b = (int)(blockIdx.x / (nqb * p.heads));
  const int col = h * D + 4 * sub;
  const float* kf = (const float*)p.kf + (long long)b * p.bskf + col;
  const float* vf = (const float*)p.vf + (long long)b * p.bsvf + col;
  const float* ks = p.ks ? (const float*)p.ks + (long long)b * p.bsks + col : nullptr;
  const float* vs = p.vs ? (const float*)p.vs + (long long)b * p.bsvs + col : nullptr;
  auto ld4 = [](const float* x) { return f32x4{x[0], x[1], x[2], x[3]}; };   // one 16-byte load where aligned, else four
  const bool al = !((((uintptr_t)p.q | (uintptr_t)p.kf | (uintptr_t)p.vf | (uintptr_t)p.ks | (uintptr_t)p.vs) & 15) ||
                    ((p.ldq | p.ldkf | p.ldvf | p.ldks | p.ldvs | p.bsq | p.bskf | p.bsvf | p.bsks | p.bsvs) & 3));
  auto ld = [&](const float* x) { return al ? *reinterpret_cast<const f32x4*>(x) : ld4(x); };
  f32x4 qv[QN], acc[QN];
  float m[QN], l[QN];
#pragma unroll
  for (int q = 0; q < QN; ++q) {
    const int qi = q0 + q < p.Lq ? q0 + q : p.Lq - 1;
    qv[q] = ld((const float*)p.q + (long long)b * p.bsq + (long long)qi * p.ldq + col);
    acc[q] = f32x4{0.f, 0.f, 0.f, 0.f};
    m[q] = -INFINITY; l[q] = 0.f;
  }
  for (int j0 = wave * (U * KPS); j0 < p.L; j0 += 4 * U * KPS) {
    f32x4 kv[U], vv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      int j = j0 + u * KPS + grp;
      if (j >= p.L) j = p.L - 1;
      const long long fr = fresh_row(p.own_lo, p.own_n, p.own_period, j);
      kv[u] = ld(fr >= 0 ? kf + fr * p.ldkf : ks + (long long)j * p.ldks);
      vv[u] = ld(fr >= 0 ? vf + fr * p.ldvf : vs + (long long)j * p.ldvs);
    }
    if (j0 + U * KPS > p.L) {                              // (uniform) keys beyond the last: weight 0, the value must be finite
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (j0 + u * KPS + grp >= p.L) vv[u] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int q = 0; q < QN; ++q) {
      float s[U], mn = m[q];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float t = fmaf(qv[q].w, kv[u].w, fmaf(qv[q].z, kv[u].z, fmaf(qv[q].y, kv[u].y, qv[q].x * kv[u].x)));
#pragma unroll
        for (int o = LPK / 2; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
        s[u] = j0 + u * KPS + grp < p.L ? t * p.scale : -INFINITY;
        mn = fmaxf(mn, s[u]);
      }
      // a maximum of -inf (no key in the group's first step, scores of -inf, or NaN, which fmaxf passes over) is no reference
      const float ref = mn == -INFINITY ? 0.f : mn, a = expf(m[q] - ref);
      l[q] *= a; acc[q] *= a;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float e = expf(s[u] - ref);
        l[q] += e;
        acc[q] += vv[u] * e;
      }
      m[q] = mn;
    }
  }
#pragma unroll
  for (int q = 0; q < QN; ++q) {                           // the groups of the wave
    float mg = m[q];
#pragma unroll
    for (int o = 32; o >= LPK; o >>= 1) mg = fmaxf(mg, __shfl_xor(mg, o, 64));
    const float w = m[q] == -INFINITY ? 0.f : expf(m[q] - mg);
    l[q] *= w; acc[q] *= w;
#pragma unroll
    for (int o = 32; o >= LPK; o >>= 1) {
      l[q] += __shfl_xor(l[q], o, 64);
      acc[q].x += __shfl_xor(acc[q].x, o, 64); acc[q].y += __shfl_xor(acc[q].y, o, 64);
      acc[q].z += __shfl_xor(acc[q].z, o, 64); acc[q].w += __shfl_xor(acc[q].w, o, 64);
    }
    if (grp == 0) {
      float* r = red[wave][q];
      r[4 * sub] = acc[q].x; r[4 * sub + 1] = acc[q].y; r[4 * sub + 2] = acc[q].z; r[4 * sub + 3] = acc[q].w;
      if (sub == 0) { r[D] = mg; r[D + 1] = l[q]; }
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < QN * D; i += 256) {        // the four waves
    const int q = i / D, d = i % D;
    if (q0 + q >= p.Lq) break;
    float mg = -INFINITY, lt = 0.f, o = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) mg = fmaxf(mg, red[w][q][D]);
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float e = red[w][q][D] == -INFINITY ? 0.f : expf(red[w][q][D] - mg);
      lt += e * red[w][q][D + 1];
      o += e * red[w][q][d];
    }
    ((float*)p.out)[(long long)b * p.bso + (long long)(q0 + q) * p.ldo + h * D + d] = o / lt;
  }
}

// Predicted time (microseconds) of attn_pipe_d64 with the keys in `ns` ranges, fitted on 22 shapes between 64 x 256 and
// 7200 x 57600 with 1 to 12 ranges each.  A compute unit works through its workgroups' 64-key tiles at nearly the same
// rate whether one or two are resident (0.65 and 0.53 us per tile; with the row gather, `rows`, 0.76 and 0.58), so the time
// follows the most loaded unit; ranges even out the load, and cost a second kernel and the float partials (written and read
// at 2.9 TB/s together).
double pipe_us(int B, int Lq, int L, int heads, bool rows, int ns) {
  const long long blocks = (long long)cdiv(Lq, 128) * heads * B;
  const long long per_cu = (blocks * ns + 255) / 256;
  const double tiles = cdiv(cdiv(L, ns), 64);
  return 4.5 + tiles * (per_cu == 1 ? (rows ? 0.76 : 0.65) : (rows ? 0.58 : 0.53) * per_cu) +
         (ns > 1 ? 2.5 + (double)B * heads * Lq * ns * 512.0 / 2.9e6 : 0.0);
}

// Number of key ranges
int pick_splits(int B, int Lq, int L, int heads, bool rows) {
#ifdef DF_TUNING
  const int forced = tune_env("DF_ATTN_SPLITS") ? atoi(tune_env("DF_ATTN_SPLITS")) : 0;
  if (forced > 0) return (L / forced >= 64) ? forced : 1;
#endif
  int best = 1;
  double best_us = 1e30;
  for (int ns = 1; ns <= 16; ++ns) {
    if (ns > 1 && L / ns < 128) break;
    const double us = pipe_us(B, Lq, L, heads, rows, ns);
    if (us < best_us - 1e-9) { best_us = us; best = ns; }
  }
  return best;
}

}  // namespace

#ifdef DF_TUNING
// Tuning build only: copies the stamps of the last attn_wave_d64 launch to host memory (synchronises).
extern "C" __attribute__((visibility("default"))) int df_tune_attn_trace(long long* out, int n) {
  if (!out || n <= 0 || n > 512 * 32) return DF_EINVAL;
  if (hipDeviceSynchronize() != hipSuccess) return DF_EHIP;
  if (hipMemcpyFromSymbol(out, HIP_SYMBOL(g_attn_trace), (size_t)n * sizeof(long long)) != hipSuccess) return DF_EHIP;
  return DF_OK;
}
#endif

size_t attention_scratch_bytes(int B, int Lq, int L, int heads, int d) {
  const int n0 = pick_splits(B, Lq, L, heads, false), n1 = pick_splits(B, Lq, L, heads, true), ns = n0 > n1 ? n0 : n1;
  if (ns == 1) return kScratchCounterBytes;
  return kScratchCounterBytes + (size_t)ns * B * heads * Lq * (d + 2) * sizeof(float) + 256;
}

int launch_attention(const AttnArgs& a, hipStream_t st) {
  if (a.B <= 0 || a.Lq <= 0 || a.L <= 0 || a.heads <= 0) return DF_ESHAPE;
  if (!(a.scale > 0.f) || !(a.scale < INFINITY)) return DF_EINVAL;   // the kernels fold the scale into exp2 arguments
  if (a.own_period < 0 || (a.own_period > 0 && (a.L % a.own_period || a.own_lo < 0 || a.own_lo + a.own_n > a.own_period)))
    return DF_ESHAPE;
  const bool own_all = a.own_lo <= 0 && a.own_lo + a.own_n >= (a.own_period > 0 ? a.own_period : a.L);
  if (!own_all && (!a.k_stale || !a.v_stale)) return DF_EINVAL;
  AttnParams p = {};
  p.q = a.q; p.kf = a.k_fresh; p.vf = a.v_fresh; p.ks = a.k_stale; p.vs = a.v_stale; p.out = a.out;
  p.B = a.B; p.Lq = a.Lq; p.L = a.L; p.heads = a.heads; p.own_lo = a.own_lo; p.own_n = a.own_n;
  p.own_period = a.own_period;
  p.own_magic = a.own_period > 1 ? (unsigned int)((1ULL << 32) / (unsigned int)a.own_period) : 0xffffffffu;
  p.ldq = a.ldq; p.ldkf = a.ldkf; p.ldvf = a.ldvf; p.ldks = a.ldks; p.ldvs = a.ldvs; p.ldo = a.ldo;
  p.bsq = a.bsq; p.bskf = a.bskf; p.bsvf = a.bsvf; p.bsks = a.bsks; p.bsvs = a.bsvs; p.bso = a.bso;
  p.scale = a.scale;
  p.sc_log2 = a.q_scaled ? 1.0f : a.scale * kLog2e;
  const bool scaled = a.v_transposed && p.sc_log2 == 1.0f;             // (a caller's own scaling and scale = ln 2 do as well)
  if (a.q_scaled && !a.v_transposed) return DF_EINVAL;
  p.nsplit = 1; p.keys_per_split = a.L;
  p.out_packed = a.out_packed;
  if (a.out_packed && (a.dtype != DF_BF16 || ((uintptr_t)a.out % 16))) return DF_EINVAL;
  if (a.dtype == DF_F32) {
    const long long heads = (long long)a.B * a.heads;
    const bool four = heads * a.Lq >= 8 * 256;
    const long long nwg = heads * cdiv(a.Lq, four ? 4 : 1);
    if (nwg > 0x7fffffffLL) return DF_ESHAPE;
    const dim3 grid((unsigned)nwg);
    if (a.d == 32 && four) hipLaunchKernelGGL((attn_f32<32, 4>), grid, dim3(256), 0, st, p);
    else if (a.d == 32) hipLaunchKernelGGL((attn_f32<32, 1>), grid, dim3(256), 0, st, p);
    else if (a.d == 64 && four) hipLaunchKernelGGL((attn_f32<64, 4>), grid, dim3(256), 0, st, p);
    else if (a.d == 64) hipLaunchKernelGGL((attn_f32<64, 1>), grid, dim3(256), 0, st, p);
    else return DF_ESHAPE;
    DF_LAUNCH_CHECK();
    return DF_OK;
  }
  if (a.d != 64) return DF_ESHAPE;
  const long long lds[] = {a.ldq, a.ldkf, a.ldvf, a.ldks, a.ldvs, a.ldo, a.bsq, a.bskf, a.bsvf, a.bsks, a.bsvs, a.bso};
  for (long long v : lds) if (v % 8) return DF_EINVAL;
  if (a.heads >= (1 << 24) || a.ldq >= (1LL << 31)) return DF_ESHAPE;   // (as the kernels' leading arguments hold them, beside at most 16 parts of the keys)
  const void* ptrs[] = {a.q, a.k_fresh, a.v_fresh, a.k_stale, a.v_stale, a.out};
  for (const void* q : ptrs) if ((uintptr_t)q % 16) return DF_EINVAL;
  // Few queries (the patch at the deepest levels): one workgroup per 32-query block and head whose eight waves split the
  // keys; no partials, no merge kernel.  Each block streams the head's whole K / V^T, so a compute unit pulls Lq / 32 x
  // the head's keys through its load path where the LDS-shared kernel pulls Lq / 128 x: it is only taken with its workgroups
  // in one round (at most one per compute unit), and where a wave's rounds of 64 keys are few.  The more query blocks share a
  // head's keys, the sooner they come from L2, and the more rounds it stays ahead: by measurement on 134 shapes, cold keys, up
  // to 3 + 3/4 of the blocks, at most 10 (beyond, where the model of the split form says that it is slower still).
  // Microseconds, split form against this: 64 queries x 256 keys x 10 heads 6.8 / 5.7, 128 x 512 x 20 10.7 / 7.4,
  // 256 x 1024 x 10 13.3 / 9.1, 300 x 2400 x 20 20.7 / 15.7, 256 x 4096 x 10 19.8 / 18.6, 128 x 3072 x 20 19.2 / 18.7; the other way
  // 32 x 2048 x 20 14.7 / 15.7, 128 x 4096 x 20 20.7 / 23.2, 300 x 9600 x 20 40.5 / 48.6.
#ifdef DF_TUNING
  const char* wave_env = tune_env("DF_ATTN_WAVE");
#else
  const char* wave_env = nullptr;
#endif
  const long long qblocks = cdiv(a.Lq, 32), rounds = cdiv(cdiv(a.L, 64), 8);
  const bool wave_fits = a.v_transposed && a.L >= 64 && qblocks * a.heads * a.B <= 256;
  const bool wave_over_split = wave_fits && a.L >= 512 && (wave_env ? atoi(wave_env) != 0
      : 4.7 + 1.93 * (double)rounds < pipe_us(a.B, a.Lq, a.L, a.heads, false, pick_splits(a.B, a.Lq, a.L, a.heads, false)));
  const bool wave_few_rounds = wave_fits && (wave_env ? atoi(wave_env) != 0 : rounds <= 3 + 3 * qblocks / 4 && rounds <= 10);
  // Up to twice as many blocks: four waves each, two workgroups per compute unit, where the keys are few for the number of blocks
  // (the split form has a workgroup per 128 queries on less than half of the units).  Microseconds, split form against this: 416 queries x 416
  // keys x 20 heads 10.2 / 8.5, 494 x 988 x 20 16.1 / 13.4, 608 x 1216 x 20 16.2 / 14.3, 960 x 960 x 10 12.7 / 11.7, two batch items of 300 x 1200 x 20
  // 17.9 / 14.5, 700 x 1400 x 20 19.8 / 16.1, 1600 x 1600 x 10 18.9 / 17.6; the other way 432 x 1728 x 20 16.6 / 17.1, 1024 x 2048 x 10 18.9 / 19.8.
  const bool four_waves = a.v_transposed && a.L >= 64 && qblocks * a.heads * a.B > 256 && qblocks * a.heads * a.B <= 512 &&
      (wave_env ? atoi(wave_env) != 0
                : 5.2 + 1.85 * (double)cdiv(cdiv(a.L, 64), 4) < pipe_us(a.B, a.Lq, a.L, a.heads, false, pick_splits(a.B, a.Lq, a.L, a.heads, false)));
  auto launch_wave = [&]() -> int {
    if (!a.k_stale || !a.v_stale || a.own_n != 0 || a.own_period != 0 || a.vt_ld % 8 || a.vt_ld < (long long)cdiv(a.L, 64) * 64) return DF_EINVAL;
    if (a.ldks <= 0 || a.ldks >= (1 << 23) || a.vt_ld >= (1 << 25)) return DF_ESHAPE;   // 32-bit offsets inside a tile
    p.vt_ld = a.vt_ld; p.nsplit = 1; p.keys_per_split = a.L;
    // Compute units without a workgroup read ahead what the next launches of the stream read (packed weights; from HBM into the
    // last-level cache).  A layer of few tokens waits for its weights: 64 x 1280 x 1280 5.4 us with them in HBM, 4.0 with them
    // read before.  The amount is what these units read (20 GB/s each, 3 TB/s together) while the others attend; more makes
    // this launch longer (26 MB: 5.9 -> 9.8 us), and with few idle units, or long keys that come from HBM themselves, it
    // takes more from them than it gives (300 x 2400 x 20, 48 units: 17.0 -> 23.5 us): nothing below 80 units.  512 x 512 step of
    // four patches 5150 -> 5000 us, 1024 x 1024 of eight with guidance 7205 -> 7135.
    const int cols = cdiv(a.heads, 8) * 8;
    const long long idle = 256 - qblocks * a.heads * a.B;
    long long rows = a.next.n > 0 ? idle / ((long long)cols * a.B) : 0;
    if (rows * cols * a.B < 80) rows = 0;
    const double us = 1.0 + 1.93 * (double)rounds, rate = 0.02e6 * (double)(rows * cols * a.B);
    long long kb = (long long)(us * (rate < 3.0e6 ? rate : 3.0e6) / 1024.0);
    p.next.n = 0;
    for (int i = 0; i < a.next.n && rows > 0 && kb > 0; ++i) {
      const long long n = a.next.bytes[i] >> 10 < kb ? a.next.bytes[i] >> 10 : kb;
      p.next.p[p.next.n] = a.next.p[i]; p.next.bytes[p.next.n++] = n << 10;
      kb -= n;
    }
    p.qblocks = (int)qblocks;
    const dim3 grid((unsigned)cols, (unsigned)(qblocks + (p.next.n ? rows : 0)), (unsigned)a.B);
    constexpr int NW = 8;
    constexpr int smem = NW * 2 * 64 * 64 * 2;          // a K and a V^T tile per wave; the merge reuses it
    static_assert(NW * 34 * 64 * 4 <= smem, "the merge fits");
    static bool attr_set = false;
    if (!attr_set) {
      if (hipFuncSetAttribute((const void*)attn_wave_d64<NW, false>, hipFuncAttributeMaxDynamicSharedMemorySize, smem) != hipSuccess ||
          hipFuncSetAttribute((const void*)attn_wave_d64<NW, true>, hipFuncAttributeMaxDynamicSharedMemorySize, smem) != hipSuccess)
        return DF_EHIP;
      attr_set = true;
    }
    // (the pitches of keys and values are bounded above; every caller's queries have heads * 64)
#define DF_WAVE_ARGS                                                                                                         \
  (const bf16_t*)p.q, (const bf16_t*)p.ks, (const bf16_t*)p.vs, p.Lq, p.L, p.heads, p.qblocks, (int)p.ldq, (int)p.ldks, (int)p.vt_ld, \
      p.qb_recip, p
    if (four_waves || (p.next.n == 0 && cols / 8 * qblocks * a.B > 32)) {
      p.next.n = 0;
      p.qb_recip = reciprocal_u32((unsigned int)qblocks);
      const dim3 blocks((unsigned)(qblocks * a.heads * a.B));
      if (four_waves) hipLaunchKernelGGL((attn_wave_d64<4, true>), blocks, dim3(256), smem / 2, st, DF_WAVE_ARGS);
      else hipLaunchKernelGGL((attn_wave_d64<NW, true>), blocks, dim3(64 * NW), smem, st, DF_WAVE_ARGS);
    } else {
      hipLaunchKernelGGL((attn_wave_d64<NW, false>), grid, dim3(64 * NW), smem, st, DF_WAVE_ARGS);
    }
#undef DF_WAVE_ARGS
    DF_LAUNCH_CHECK();
    return DF_OK;
  };
  if (wave_over_split) return launch_wave();
  int ns = pick_splits(a.B, a.Lq, a.L, a.heads, !a.v_transposed);
  if ((long long)a.B * ns > 65535) return DF_ESHAPE;
  if ((long long)a.B * a.heads * a.Lq * 16 >= (1LL << 31)) return DF_ESHAPE;   // the merge kernel indexes with 32 bits
  if (ns > 1) {
    const int kps = cdiv(cdiv(a.L, ns), 128) * 128;      // whole pairs of tiles
    ns = cdiv(a.L, kps);                                 // rounding up may leave the last ranges empty: drop them
    if (ns > 1) {
      char* scr = scratch_region(a.scr, attention_scratch_bytes(a.B, a.Lq, a.L, a.heads, a.d));
      if (!scr) return DF_ENOMEM;
      p.nsplit = ns;
      p.keys_per_split = kps;
      p.part_o = (float*)(scr + kScratchCounterBytes);
      p.part_ml = p.part_o + (size_t)ns * a.B * a.heads * a.Lq * 64;
    }
  }
  if (wave_few_rounds || four_waves) return launch_wave();   // (what the caller has to provide stays that of the split form)
  const long long nwg = (long long)cdiv(a.Lq, 128) * a.heads * a.B * p.nsplit;
#define DF_PIPE(KERNEL, LDV)                                                                                                      \
  hipLaunchKernelGGL(KERNEL, dim3((unsigned)nwg), dim3(256), smem, st, (const bf16_t*)p.q, (const bf16_t*)p.ks, (const bf16_t*)p.vs, p.Lq, \
                     p.L, (unsigned int)p.heads | (unsigned int)p.nsplit << 24, p.keys_per_split, (int)p.ldq, (int)p.ldks, (int)(LDV), (int)nwg, p)
  if (nwg > 0x7fffffffLL) return DF_ESHAPE;
  if (a.v_transposed) {
    // every key from k_stale (row-major) / v_stale (V^T, row pitch vt_ld >= L rounded up to whole 64-key tiles)
    if (!a.k_stale || !a.v_stale || a.own_n != 0 || a.own_period != 0 || a.vt_ld % 8 || a.vt_ld < (long long)cdiv(a.L, 64) * 64) return DF_EINVAL;
    if (a.ldks <= 0 || a.ldks >= (1 << 23) || a.vt_ld >= (1 << 25)) return DF_ESHAPE;   // 32-bit offsets inside a tile
    p.vt_ld = a.vt_ld;
    constexpr int smem = 6 * 64 * 64 * 2;                // three K and three V^T tiles
    if (scaled) DF_PIPE((attn_pipe_d64<true, kSrcVt>), p.vt_ld);
    else DF_PIPE((attn_pipe_d64<false, kSrcVt>), p.vt_ld);
  } else {
    // 32-bit row offsets inside a 64-key tile
    if (a.ldkf >= (1 << 24) || a.ldvf >= (1 << 24) || a.ldks >= (1 << 24) || a.ldvs >= (1 << 24)) return DF_ESHAPE;
    constexpr int smem = 6 * 64 * 64 * 2;                // three K and three V tiles
    if (a.own_period > 0) DF_PIPE((attn_pipe_d64<false, kSrcPeriodic>), p.ldvs);
    else DF_PIPE((attn_pipe_d64<false, kSrcRows>), p.ldvs);
  }
#undef DF_PIPE
  DF_LAUNCH_CHECK();
  if (ns > 1) {
    const long long n = (long long)a.B * a.heads * a.Lq * 8;
    const dim3 grid((unsigned)((n + 255) / 256));
    switch (ns) {
#define DF_MERGE(NS) hipLaunchKernelGGL(attn_combine_d64<NS>, grid, dim3(256), 0, st, p); break
      case 2: DF_MERGE(2);
      case 3: DF_MERGE(3);
      case 4: DF_MERGE(4);
      case 5: DF_MERGE(5);
      case 6: DF_MERGE(6);
      case 7: DF_MERGE(7);
      default: DF_MERGE(8);
#undef DF_MERGE
    }
    DF_LAUNCH_CHECK();
  }
  return DF_OK;
}

}  // namespace df
