// Corrected asynchronous GroupNorm (Section 4, Eq. 2) for channels-last patches.
//
// Large tensors take two launches, both streaming passes with 16-byte accesses:
//   gn_stats     every block sums a strip of pixels into per-group (sum, sum of
//                squares) partials; one block also snapshots the cached sums.
//   gn_apply     every block first adds all partials in the same fixed order (so
//                all blocks hold bit-identical statistics without a third launch or
//                a grid-wide wait: an in-kernel barrier across the eight XCDs costs
//                more than a kernel boundary here), combines them with the stale
//                sums of the other patches according to the statistic mode, then
//                y = (x - mean) * rstd * gamma + beta (+ SiLU) on the strip it summed
//                in the first launch; block 0 also emits the fresh per-patch sums.
// Small tensors take one launch, one workgroup per (group, batch item), and those between one whose workgroups hand each other
// their sums (gn_meet_kernel).
// A lane keeps a fixed channel offset for its whole strip, so gamma/beta and
// the statistics are fetched once per lane.
//
// Numerics: sums are taken of x - p, p being the group's first value of the batch
// item (its "pivot"), and turned into the sums of x in double only where a group's
// totals are known: E[x^2] - E[x]^2 of float sums loses (mean / sigma)^2 ulps, which
// a tensor whose mean is far from zero cannot afford at float32 tolerance.  The
// normalisation subtracts the mean as a (high, low) float pair before scaling.
#include <atomic>
#include <cstdlib>
#include <mutex>
#include "gnmeet.h"
#include "kernels.h"

namespace df {

namespace {

constexpr int kMaxG = 64;
constexpr long long kGnGroupMaxElems = 24 * 1024;   // per (group, batch item): above this the two-launch path (unless
                                                    // the patch fits the registers of one workgroup per group)
constexpr int kGnMaxPpb = 32;                      // pixels a block of that path handles per iteration, at most
constexpr int kGnMaxStrips = 256;                   // pixel strips (= blocks per launch) per batch item on that path

struct GnHalo {
  bf16_t* out;      // nullptr: no boundary-row copy
  int W, rpp, patch0, npatch;
  int single;       // the tensor holds exactly one patch (rpp rows): boundary rows follow from comparisons
  int cols, rows;   // cols != 0: vertical strips of rpp columns, the state holds boundary columns of `rows` pixels
};

// stores 2, 4 or 8 bf16 values of pixel p (within its batch item), channels c0.., into the boundary-row state if the
// pixel lies on the first or last row of its patch
template <int V>
__device__ __forceinline__ void halo_store(const GnHalo& h, int b, long long p, int C, int c0, const float* v) {
  // (this runs per pixel and lane: no 64-bit division, and none at all for the one-patch tensors of a displaced step)
  const unsigned int pi = (unsigned int)p;
  unsigned int row, col, pr, patch;
  if (h.cols) {
    row = pi / (unsigned int)h.W; col = pi - row * (unsigned int)h.W;
    const unsigned int q = col / (unsigned int)h.rpp;
    const unsigned int pc = col - q * (unsigned int)h.rpp;
#pragma unroll
    for (int which = 0; which < 2; ++which) {
      if ((int)pc != (which ? h.rpp - 1 : 0)) continue;
      bf16_t* o = h.out + ((((long long)b * h.npatch + (h.patch0 + q)) * 2 + which) * h.rows + row) * C + c0;
      if constexpr (V == 8) {
        st_vec(o, v);
      } else if constexpr (V == 4) {
        u32x2 t = {pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3])};
        *reinterpret_cast<u32x2*>(o) = t;
      } else {
        *reinterpret_cast<unsigned int*>(o) = pack_bf2(v[0], v[1]);
      }
    }
    return;
  }
  if (h.single) {
    const unsigned int last0 = (unsigned int)(h.rpp - 1) * (unsigned int)h.W;
    if (pi >= (unsigned int)h.W && pi < last0) return;           // an interior row
    pr = pi < (unsigned int)h.W ? 0u : (unsigned int)(h.rpp - 1);
    col = pi < (unsigned int)h.W ? pi : pi - last0;
    row = pr; patch = (unsigned int)h.patch0;
    if (h.rpp == 1) { pr = 0; col = pi; }
  } else {
    row = pi / (unsigned int)h.W; col = pi - row * (unsigned int)h.W;
    const unsigned int q = row / (unsigned int)h.rpp;
    pr = row - q * (unsigned int)h.rpp; patch = (unsigned int)h.patch0 + q;
  }
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    if ((int)pr != (which ? h.rpp - 1 : 0)) continue;
    bf16_t* o = h.out + ((((long long)b * h.npatch + patch) * 2 + which) * h.W + col) * C + c0;
    if constexpr (V == 8) {
      st_vec(o, v);
    } else if constexpr (V == 4) {
      u32x2 t = {pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3])};
      *reinterpret_cast<u32x2*>(o) = t;
    } else {
      *reinterpret_cast<unsigned int*>(o) = pack_bf2(v[0], v[1]);
    }
  }
}

// PAIR: x is the concatenation of two tensors along the channels, Ca of `x` and the rest of `b`, which is never stored as floats; the
// kernel that reads it first leaves the bf16 copy that the shortcut convolution takes.  A lane's channels lie on one side (Ca % 4 == 0).
// Of the 10 bytes per value that a concatenation kernel moves (floats and bf16 written, both tensors read) 2 remain; 832x1216 step 9703 ->
// 9637 us, 512x512 step 4654 -> 4644, 2048x2048 in strips 15770 -> 15686.
struct GnPair {
  const float* b;
  int Ca;
  bf16_t* cat;
};
// The kernels of one tensor take nothing in its place: with the pair's 24 bytes among their arguments a call of few pixels took 0.2 - 0.3 us
// longer (64 x 320 bf16 4.28 -> 4.55 us, 300 x 320 4.68 -> 4.98).
struct GnWhole {};
template <bool PAIR>
using GnFrom = std::conditional_t<PAIR, GnPair, GnWhole>;
// Where channel c of pixel 0 is, and the values from a pixel to the next
template <bool PAIR, typename Tin>
__device__ __forceinline__ const Tin* gn_source(const Tin* x, const GnFrom<PAIR>& pr, int C, int c, int* pitch) {
  if constexpr (PAIR) {
    *pitch = c < pr.Ca ? pr.Ca : C - pr.Ca;
    return c < pr.Ca ? x + c : pr.b + (c - pr.Ca);
  }
  *pitch = C;
  return x + c;
}
template <bool PAIR, typename Tin>
__device__ __forceinline__ float gn_value(const Tin* x, const GnFrom<PAIR>& pr, int C, long long pix, int c) {
  int pitch;
  const Tin* s = gn_source<PAIR>(x, pr, C, c, &pitch);
  return Elem<Tin>::ld(s + pix * pitch);
}

// NCH (template parameter of the two-launch kernels): 16-byte loads a lane keeps in flight, 1, 2, 4 or 8

// 16 bytes as loaded -> kVec float values
template <typename T>
__device__ __forceinline__ void unpack_vec(const u32x4& t, float* v) {
  if constexpr (sizeof(T) == 4) {
    v[0] = __uint_as_float(t.x); v[1] = __uint_as_float(t.y); v[2] = __uint_as_float(t.z); v[3] = __uint_as_float(t.w);
  } else {
    v[0] = __uint_as_float(t.x << 16); v[1] = __uint_as_float(t.x & 0xffff0000u);
    v[2] = __uint_as_float(t.y << 16); v[3] = __uint_as_float(t.y & 0xffff0000u);
    v[4] = __uint_as_float(t.z << 16); v[5] = __uint_as_float(t.z & 0xffff0000u);
    v[6] = __uint_as_float(t.w << 16); v[7] = __uint_as_float(t.w & 0xffff0000u);
  }
}

struct GnLayout {
  int tp;        // lanes per pixel (C / vec)
  int ppb;       // pixels per block iteration
  int threads;   // tp * ppb
  int nblk;      // blocks per segment
  int pix_per_blk;
};

template <typename Tin, int NCH, bool PAIR>
__global__ void gn_stats(const Tin* __restrict__ x, float* __restrict__ partial, int pix_seg, int C, int G, int tp,
                         int ppb, int pix_per_blk, int nseg, const float* stale, float* __restrict__ stale_copy,
                         int stale_n, GnFrom<PAIR> pr) {
  constexpr int V = Elem<Tin>::kVec;
  __shared__ float s_sum[kMaxG], s_sq[kMaxG], s_piv[kMaxG];
  const int blk = blockIdx.x, seg = blockIdx.y, b = blockIdx.z;
  const int nblk = gridDim.x;
  const int cg = C / G;
  const int tid = threadIdx.x;
  const int c0 = (tid % tp) * V;
  const int psub = tid / tp;
  const long long seg_base = ((long long)b * nseg + seg) * pix_seg;
  const int p_lo = blk * pix_per_blk;
  int p_hi = p_lo + pix_per_blk;
  if (p_hi > pix_seg) p_hi = pix_seg;
  // a lane requests NCH pixels at once (a strip is usually one chunk: the whole tensor is in flight together);
  // the first chunk goes out before anything else
  int pitch;
  const Tin* const xs = gn_source<PAIR>(x, pr, C, c0, &pitch);
  u32x4 raw[NCH];
#pragma unroll
  for (int k = 0; k < NCH; ++k) {
    const int p = p_lo + psub + k * ppb;
    raw[k] = *reinterpret_cast<const u32x4*>(xs + (seg_base + (p < p_hi ? p : p_lo)) * pitch);
  }
  if (tid < G) s_piv[tid] = gn_value<PAIR>(x, pr, C, (long long)b * nseg * pix_seg, tid * cg);   // the groups' pivots
  // The second launch may overwrite the patch's own slot of the cached sums (in-place refresh) while other blocks of
  // it still need the old value: it reads this snapshot instead.
  if (stale != nullptr && blk == 0 && seg == 0 && b == 0)
    for (int i = tid; i < stale_n; i += blockDim.x) stale_copy[i] = stale[i];
  __syncthreads();

  const int ga = c0 / cg;                       // group of the lane's first channel
  float s[V], q[V], piv[V];
#pragma unroll
  for (int i = 0; i < V; ++i) {
    s[i] = 0.f; q[i] = 0.f;
    piv[i] = s_piv[cg >= V ? (c0 + i >= (ga + 1) * cg ? ga + 1 : ga) : (c0 + i) / cg];
  }
  for (int p0 = p_lo + psub; p0 < p_hi; p0 += NCH * ppb) {
    if (p0 != p_lo + psub) {
#pragma unroll
      for (int k = 0; k < NCH; ++k) {
        const int p = p0 + k * ppb;
        raw[k] = *reinterpret_cast<const u32x4*>(xs + (seg_base + (p < p_hi ? p : p0)) * pitch);
      }
    }
#pragma unroll
    for (int k = 0; k < NCH; ++k) {
      if (p0 + k * ppb >= p_hi) break;
      float v[V];
      unpack_vec<Tin>(raw[k], v);
      if constexpr (PAIR) {
        const u32x2 t = {pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3])};
        *reinterpret_cast<u32x2*>(pr.cat + (seg_base + p0 + k * ppb) * C + c0) = t;
      }
#pragma unroll
      for (int i = 0; i < V; ++i) { const float d = v[i] - piv[i]; s[i] += d; q[i] = fmaf(d, d, q[i]); }
    }
  }
  // Ordered fold of the lanes' per-channel sums into groups (no atomics: the result must not depend on timing -
  // the UNet amplifies even one-ulp differences of a statistic to the level of its bf16 rounding noise).
  // Two levels: thread (g, ps) adds group g's channels over the lanes of pixel slot ps, then thread g adds the slots.
  extern __shared__ float s_lane[];            // fast path: float4 per lane; general path: [V][blockDim.x]
  __shared__ float s_lvl[2][kGnMaxPpb][kMaxG];
  const int nthr = blockDim.x;
  if (cg >= V) {
    // a lane's V consecutive channels touch at most two groups: it leaves (sum, sum of squares) of the part in its
    // first group and of the part in the next one
    f32x4 mine = {0.f, 0.f, 0.f, 0.f};
    const int nb = (ga + 1) * cg - c0;          // channels of the lane that belong to group ga
#pragma unroll
    for (int i = 0; i < V; ++i) {
      if (i < nb) { mine.x += s[i]; mine.y += q[i]; } else { mine.z += s[i]; mine.w += q[i]; }
    }
    reinterpret_cast<f32x4*>(s_lane)[tid] = mine;
    __syncthreads();
    for (int role = tid; role < G * ppb; role += nthr) {
      const int fg = role % G, fps = role / G;
      const int t_lo = (fg * cg) / V, t_hi = ((fg + 1) * cg - 1) / V;
      float as = 0.f, aq = 0.f;
      for (int tc = t_lo; tc <= t_hi; ++tc) {
        const f32x4 e = reinterpret_cast<const f32x4*>(s_lane)[fps * tp + tc];
        if ((tc * V) / cg == fg) { as += e.x; aq += e.y; } else { as += e.z; aq += e.w; }
      }
      s_lvl[0][fps][fg] = as;
      s_lvl[1][fps][fg] = aq;
    }
    __syncthreads();
  } else {
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
#pragma unroll
      for (int i = 0; i < V; ++i) s_lane[i * nthr + tid] = pass ? q[i] : s[i];
      __syncthreads();
      for (int role = tid; role < G * ppb; role += nthr) {
        const int fg = role % G, fps = role / G;
        float acc = 0.f;
        for (int ch = fg * cg; ch < (fg + 1) * cg; ++ch) acc += s_lane[(ch % V) * nthr + fps * tp + ch / V];
        s_lvl[pass][fps][fg] = acc;
      }
      __syncthreads();
    }
  }
  if (tid < G) {
    float ss = 0.f, qq = 0.f;
    for (int ps = 0; ps < ppb; ++ps) { ss += s_lvl[0][ps][tid]; qq += s_lvl[1][ps][tid]; }
    s_sum[tid] = ss;
    s_sq[tid] = qq;
  }
  __syncthreads();
  float* my = partial + ((((long long)b * nseg + seg) * nblk + blk) * G) * 2;
  if (tid < G) { my[2 * tid] = s_sum[tid]; my[2 * tid + 1] = s_sq[tid]; }
}

// Sums of x from the sums of x - piv over n values (double: this is where the cancellation would happen).
__device__ __forceinline__ void gn_unshift(float s, float q, double n, float piv, double& S, double& SS) {
  const double p = (double)piv;
  S = (double)s + n * p;
  SS = (double)q + 2.0 * p * (double)s + n * p * p;
}

struct GnMoments { float mean_hi, mean_lo, rstd; };

// Mean and variance of one (batch item, group) from the fresh sums of this launch and the cached per-patch sums,
// according to the statistic mode (Section 4, Eq. 2; Section 5.3).  Runs once per group, in double.
// `st_*`: sums of the cached entries of the other patches, `own_*`: the cached entry of this patch.
// The reciprocals come from the host: this runs on one wave while the others wait, and a division or a square root in double is some
// twenty dependent instructions.  The quotients are those of a division all the same (div_by).
struct GnCount { double n_loc, inv_loc, n_all, inv_all; };   // values of a group in the patch, and in the image
__device__ __forceinline__ GnMoments gn_combine_pre(double tot_s, double tot_q, const GnCount& n, int nseg, int N,
                                                    int stat_mode, double st_s, double st_q, double own_s,
                                                    double own_q, float eps) {
  auto loc = [&](double s) { return div_by(s, n.n_loc, n.inv_loc); };
  auto all = [&](double s) { return div_by(s, n.n_all, n.inv_all); };
  double mean, var;
  if (nseg > 1 || (N == 1 && stat_mode != DF_GN_STALE)) {
    // the whole image is fresh: exact statistics
    mean = all(tot_s);
    var = fmax(all(tot_q) - mean * mean, 0.0);
  } else {
    const double loc_m = loc(tot_s), loc_m2 = loc(tot_q);
    if (stat_mode == DF_GN_SUMS) {
      mean = all(tot_s + st_s);
      var = fmax(all(tot_q + st_q) - mean * mean, 0.0);
    } else if (stat_mode == DF_GN_EQ2) {
      mean = all(st_s + own_s) + (loc_m - loc(own_s));
      const double m2 = all(st_q + own_q) + (loc_m2 - loc(own_q));
      var = m2 - mean * mean;
      if (var < 0.0) var = loc_m2 - loc_m * loc_m;
    } else if (stat_mode == DF_GN_SEPARATE) {
      mean = loc_m;
      var = fmax(loc_m2 - loc_m * loc_m, 0.0);
    } else {
      mean = all(st_s + own_s);
      var = fmax(all(st_q + own_q) - mean * mean, 0.0);
    }
  }
  GnMoments m;
  m.mean_hi = (float)mean;
  m.mean_lo = (float)(mean - (double)m.mean_hi);
  const double v = var + (double)eps;
  // the hardware's float estimate (1 ulp), refined; outside float range the long way
  m.rstd = v > 1e-30 && v < 1e30 ? (float)rsqrt_from(v, __builtin_amdgcn_rsqf((float)v)) : (float)(1.0 / sqrt(v));
  return m;
}

__device__ __forceinline__ GnMoments gn_combine(double tot_s, double tot_q, const GnCount& n_loc, int nseg, int N, int stat_mode,
                                                const float* stale, int b, int g, int B, int G, int patch_idx,
                                                float eps) {
  double st_s = 0.0, st_q = 0.0, own_s = 0.0, own_q = 0.0;
  if (!(nseg > 1 || (N == 1 && stat_mode != DF_GN_STALE))) {
    for (int j = 0; j < N; ++j) {
      const float* sp = stale + (((long long)j * B + b) * G + g) * 2;
      const float a = sp[0], c = sp[1];
      if (j == patch_idx) { own_s = a; own_q = c; } else { st_s += a; st_q += c; }
    }
  }
  return gn_combine_pre(tot_s, tot_q, n_loc, nseg, N, stat_mode, st_s, st_q, own_s, own_q, eps);
}

// The cached sums of one (batch item, group) gathered by a whole wave: lane j fetches patch j's entry (one memory
// round trip for all patches instead of a chain of N), lane order fixes the order of the additions.
__device__ __forceinline__ void gn_stale_wave(const float* stale, int b, int g, int B, int G, int N,
                                              int patch_idx, int lane, double& st_s, double& st_q, double& own_s,
                                              double& own_q) {
  st_s = st_q = own_s = own_q = 0.0;
  if (stale == nullptr) return;
  for (int j0 = 0; j0 < N; j0 += 64) {
    float a = 0.f, c = 0.f;
    if (j0 + lane < N) {
      const float* sp = stale + (((long long)(j0 + lane) * B + b) * G + g) * 2;
      a = sp[0]; c = sp[1];
    }
    const int n = N - j0 < 64 ? N - j0 : 64;
    for (int j = 0; j < n; ++j) {
      const float aj = __shfl(a, j, 64), cj = __shfl(c, j, 64);
      if (j0 + j == patch_idx) { own_s = aj; own_q = cj; } else { st_s += aj; st_q += cj; }
    }
  }
}

// Second launch of the large path.  Every block adds the partials of its batch item in the same fixed order, combines
// them with the cached sums and normalises the strip of pixels it was given.
template <typename Tin, typename Tout, int NCH, bool PAIR>
__global__ __launch_bounds__(1024) void gn_apply(const Tin* __restrict__ x, Tout* __restrict__ y,
                                                 const float* __restrict__ partial, const float* __restrict__ stale_copy,
                                                 float* sums_out, const float* __restrict__ gamma,
                                                 const float* __restrict__ beta, int pix_seg, int C, int G, int nblk,
                                                 int nseg, int B, int patch_idx, int N, float eps, int stat_mode, int tp,
                                                 int ppb, int pix_per_blk, int silu, int packed, GnHalo halo, GnCount cnt,
                                                 GnFrom<PAIR> pr) {
  constexpr int V = Elem<Tin>::kVec;
  __shared__ float s_red[2][32][kMaxG];
  __shared__ float s_mom[kMaxG][3];
  const int blk = blockIdx.x, seg = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x;
  const int cg = C / G;
  // The lane's first NCH pixels are requested before anything else: the fold of the partials below then runs
  // while they are on their way (usually that is the lane's whole share of the strip).
  const bool works = tid < tp * ppb;
  const int c0 = (tid % tp) * V;
  const int psub = tid / tp;
  const long long base = ((long long)b * nseg + seg) * pix_seg;     // pixels before this segment
  const int p_lo = blk * pix_per_blk;
  int p_hi = p_lo + pix_per_blk;
  if (p_hi > pix_seg) p_hi = pix_seg;
  int pitch;
  const Tin* const xs = gn_source<PAIR>(x, pr, C, c0, &pitch);
  u32x4 raw[NCH];
  if (works) {
#pragma unroll
    for (int k = 0; k < NCH; ++k) {
      const int p = p_lo + psub + k * ppb;
      raw[k] = *reinterpret_cast<const u32x4*>(xs + (base + (p < p_hi ? p : p_lo)) * pitch);
    }
  }
  {
    const int parts = (int)blockDim.x / G < 32 ? (int)blockDim.x / G : 32;
    const int g = tid % G, part = tid / G;
    const bool folds = part < parts;
    double tot_s = 0.0, tot_q = 0.0;  // sums of x over all segments (valid where part == 0)
    // the partials are sums of x - pivot, the pivot being the group's first value of the batch item
    const float piv = folds ? gn_value<PAIR>(x, pr, C, (long long)b * nseg * pix_seg, g * cg) : 0.f;
    const double n_seg = cnt.n_loc;
    for (int sg = 0; sg < nseg; ++sg) {
      float a = 0.f, c = 0.f;
      if (folds) {
        const float* base = partial + (((long long)b * nseg + sg) * nblk) * G * 2;
        // 8 partials per trip are requested together (one memory round trip), then added in index order
        for (int k0 = part; k0 < nblk; k0 += 8 * parts) {
          float2 v[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const int k = k0 + i * parts;
            v[i] = k < nblk ? *reinterpret_cast<const float2*>(base + ((long long)k * G + g) * 2) : make_float2(0.f, 0.f);
          }
#pragma unroll
          for (int i = 0; i < 8; ++i) { a += v[i].x; c += v[i].y; }
        }
        s_red[0][part][g] = a;
        s_red[1][part][g] = c;
      }
      __syncthreads();
      if (part == 0) {
        float fs = 0.f, fq = 0.f;
        for (int k = 0; k < parts; ++k) { fs += s_red[0][k][g]; fq += s_red[1][k][g]; }
        double S, SS;
        gn_unshift(fs, fq, n_seg, piv, S, SS);
        tot_s += S; tot_q += SS;
        if (nseg > 1 && blk == 0 && seg == 0) {        // full image: the per-patch sums are the cache's new content
          float* o = sums_out + (((long long)sg * B + b) * G + g) * 2;
          o[0] = (float)S; o[1] = (float)SS;
        }
      }
      __syncthreads();
    }
    if (part == 0) {
      double st_s = 0.0, st_q = 0.0, own_s = 0.0, own_q = 0.0;
      if (!(nseg > 1 || (N == 1 && stat_mode != DF_GN_STALE))) {
        for (int j = 0; j < N; ++j) {                  // patch order fixes the order of the additions
          const float* sp = stale_copy + (((long long)j * B + b) * G + g) * 2;
          const float av = sp[0], cv = sp[1];
          if (j == patch_idx) { own_s = av; own_q = cv; } else { st_s += av; st_q += cv; }
        }
      }
      const GnMoments mo = gn_combine_pre(tot_s, tot_q, cnt, nseg, N, stat_mode, st_s, st_q, own_s, own_q, eps);
      if (nseg == 1 && sums_out != nullptr && blk == 0) {   // may alias the patch's slot of the cache: every block reads
        float* o = sums_out + ((long long)b * G + g) * 2;   // the snapshot, never the cache itself
        o[0] = (float)tot_s; o[1] = (float)tot_q;
      }
      s_mom[g][0] = mo.mean_hi; s_mom[g][1] = mo.mean_lo; s_mom[g][2] = mo.rstd;
    }
    __syncthreads();
  }
  if (!works) return;
  float sc[V], sh[V], mh[V], ml[V];
#pragma unroll
  for (int i = 0; i < V; ++i) {
    const int c = c0 + i;
    const int g = c / cg;
    mh[i] = s_mom[g][0]; ml[i] = s_mom[g][1];
    sc[i] = s_mom[g][2] * gamma[c];
    sh[i] = beta[c];
  }
  for (int p0 = p_lo + psub; p0 < p_hi; p0 += NCH * ppb) {
    if (p0 != p_lo + psub) {                   // further chunks of a long strip
#pragma unroll
      for (int k = 0; k < NCH; ++k) {
        const int p = p0 + k * ppb;
        raw[k] = *reinterpret_cast<const u32x4*>(xs + (base + (p < p_hi ? p : p0)) * pitch);
      }
    }
#pragma unroll
   for (int k = 0; k < NCH; ++k) {
    const int p = p0 + k * ppb;
    if (p >= p_hi) break;
    float v[V];
    unpack_vec<Tin>(raw[k], v);
#pragma unroll
    for (int i = 0; i < V; ++i) {
      float t = fmaf((v[i] - mh[i]) - ml[i], sc[i], sh[i]);
      v[i] = silu ? silu_f(t) : t;
    }
    const long long m = base + p;
    Tout* o = y + m * C + c0;
    if (packed) {
      // fragment-packed bf16 operand of the linear layers: pixel m is row m%32 of fragment row m/32, the
      // 8 channels from c0 & ~7 sit in slot (m%32) + 32*((c0/8)%2) of fragment column c0/16
      o = y + (((m >> 5) * (C >> 4) + (c0 >> 4)) * 64 + (m & 31) + 32 * ((c0 >> 3) & 1)) * 8 + (c0 & 7);
    }
    if constexpr (sizeof(Tout) == sizeof(Tin)) {
      st_vec(o, v);
    } else {  // float in, bf16 out: 4 values = 8 bytes
      u32x2 t = {pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3])};
      *reinterpret_cast<u32x2*>(o) = t;
    }
    if constexpr (sizeof(Tout) == 2) {
      if (halo.out) halo_store<V>(halo, b, (long long)seg * pix_seg + p, C, c0, v);
    }
   }
  }
}

// Small tensors (the patch at the deeper levels): one workgroup per (group, batch item) does the whole GroupNorm in
// one launch - sums over the group's channels of every pixel, ordered fold, statistic combination, then the
// normalisation on a second read that hits L2.  Groups are independent, so no workgroup waits for another.
template <typename Tin, typename Tout>
__global__ __launch_bounds__(1024) void gn_group_kernel(const Tin* __restrict__ x, Tout* __restrict__ y,
                                                        const float* stale, float* sums_out,
                                                        const float* __restrict__ gamma, const float* __restrict__ beta,
                                                        int pix_seg, int C, int G, int nseg, int B, int patch_idx, int N,
                                                        float eps, int stat_mode, int silu, int packed, GnHalo halo, GnCount cnt) {
  __shared__ float s_s[1024], s_q[1024];
  __shared__ float s_mr[3];
  const int g = blockIdx.x, b = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63;
  const int cg = C / G, cgv = cg >> 2;              // channel vectors of 4 per group
  const int ppass = blockDim.x / cgv;               // pixels per pass
  const int cv = tid % cgv, psub = tid / cgv;
  const bool active = psub < ppass;
  const int c0 = g * cg + cv * 4;
  const float piv = Elem<Tin>::ld(x + (long long)b * nseg * pix_seg * C + g * cg);   // sums are taken of x - piv
  const double n_seg = cnt.n_loc;
  double tot_s = 0.0, tot_q = 0.0;
  for (int sg = 0; sg < nseg; ++sg) {
    const long long base = ((long long)b * nseg + sg) * pix_seg;
    float a = 0.f, q = 0.f;
    if (active)
      for (int p = psub; p < pix_seg; p += ppass) {
        float v[4];
        const Tin* src = x + (base + p) * C + c0;
        if constexpr (sizeof(Tin) == 4) {
          ld_vec(src, v);
        } else {
          const u32x2 t = *reinterpret_cast<const u32x2*>(src);
          v[0] = __uint_as_float(t.x << 16); v[1] = __uint_as_float(t.x & 0xffff0000u);
          v[2] = __uint_as_float(t.y << 16); v[3] = __uint_as_float(t.y & 0xffff0000u);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) { const float d = v[i] - piv; a += d; q = fmaf(d, d, q); }
      }
    s_s[tid] = a; s_q[tid] = q;
    __syncthreads();
    if (tid < 64) {                                  // ordered fold: strided serial sums, then a fixed butterfly
      float fs = 0.f, fq = 0.f;
      for (int k = lane; k < (int)blockDim.x; k += 64) { fs += s_s[k]; fq += s_q[k]; }
      fs = wave_sum(fs); fq = wave_sum(fq);
      double S, SS;
      gn_unshift(fs, fq, n_seg, piv, S, SS);
      tot_s += S; tot_q += SS;
      if (nseg > 1 && lane == 0) {
        float* o = sums_out + (((long long)sg * B + b) * G + g) * 2;
        o[0] = (float)S; o[1] = (float)SS;
      }
    }
    __syncthreads();
  }
  if (tid == 0) {
    const GnMoments mo = gn_combine(tot_s, tot_q, cnt, nseg, N, stat_mode, stale, b, g, B, G, patch_idx, eps);
    if (nseg == 1 && sums_out != nullptr) {          // after the stale sums were read: may alias the own slot
      float* o = sums_out + ((long long)b * G + g) * 2;
      o[0] = (float)tot_s; o[1] = (float)tot_q;
    }
    s_mr[0] = mo.mean_hi; s_mr[1] = mo.mean_lo; s_mr[2] = mo.rstd;
  }
  __syncthreads();
  if (!active) return;
  const float mean = s_mr[0], mean_lo = s_mr[1], rstd = s_mr[2];
  float sc[4], sh[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    sc[i] = rstd * gamma[c0 + i];
    sh[i] = beta[c0 + i];
  }
  const long long pix_b = (long long)pix_seg * nseg;
  const long long base = (long long)b * pix_b;
  for (long long p = psub; p < pix_b; p += ppass) {
    float v[4];
    const Tin* src = x + (base + p) * C + c0;
    if constexpr (sizeof(Tin) == 4) {
      ld_vec(src, v);
    } else {
      const u32x2 t = *reinterpret_cast<const u32x2*>(src);
      v[0] = __uint_as_float(t.x << 16); v[1] = __uint_as_float(t.x & 0xffff0000u);
      v[2] = __uint_as_float(t.y << 16); v[3] = __uint_as_float(t.y & 0xffff0000u);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float t = fmaf((v[i] - mean) - mean_lo, sc[i], sh[i]);
      v[i] = silu ? silu_f(t) : t;
    }
    const long long m = base + p;
    Tout* o = y + m * C + c0;
    if (packed) o = y + (((m >> 5) * (C >> 4) + (c0 >> 4)) * 64 + (m & 31) + 32 * ((c0 >> 3) & 1)) * 8 + (c0 & 7);
    if constexpr (sizeof(Tout) == 4) {
      st_vec(o, v);
    } else {
      u32x2 t = {pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3])};
      *reinterpret_cast<u32x2*>(o) = t;
      if (halo.out) halo_store<4>(halo, b, p, C, c0, v);
    }
  }
}

// V consecutive channels from / to memory
template <int V, typename T>
__device__ __forceinline__ void ld_chan(const T* p, float* v) {
  if constexpr (sizeof(T) == 4) {
    if constexpr (V == 4) ld_vec(p, v);
    else { const float2 t = *reinterpret_cast<const float2*>(p); v[0] = t.x; v[1] = t.y; }
  } else if constexpr (V == 4) {
    const u32x2 t = *reinterpret_cast<const u32x2*>(p);
    v[0] = __uint_as_float(t.x << 16); v[1] = __uint_as_float(t.x & 0xffff0000u);
    v[2] = __uint_as_float(t.y << 16); v[3] = __uint_as_float(t.y & 0xffff0000u);
  } else {
    const unsigned int t = *reinterpret_cast<const unsigned int*>(p);
    v[0] = __uint_as_float(t << 16); v[1] = __uint_as_float(t & 0xffff0000u);
  }
}
template <int V, typename T>
__device__ __forceinline__ void st_chan(T* p, const float* v) {
  if constexpr (sizeof(T) == 4) {
    if constexpr (V == 4) st_vec(p, v);
    else *reinterpret_cast<float2*>(p) = make_float2(v[0], v[1]);
  } else if constexpr (V == 4) {
    const u32x2 t = {pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3])};
    *reinterpret_cast<u32x2*>(p) = t;
  } else {
    *reinterpret_cast<unsigned int*>(p) = pack_bf2(v[0], v[1]);
  }
}

// The same for one segment whose share per lane is at most NV pixels: every lane requests all its pixels at once
// (one memory round trip instead of one per pass) and keeps them in registers for the normalisation, so x is read
// once.  V channels per lane: 4, or 2 where the group's channel count allows no more (320 channels in 32 groups).
// Bound by two round trips, the kernel's start and a workgroup's share of the load path.  Requests carry no branch (a lane without
// a pixel repeats the last one and leaves it out of the sums), a wave adds its lanes without LDS, and the one wave that combines
// the moments multiplies where it divided: 300 x 1280 float32 6.4 -> 5.5 us, 64 x 1280 4.5 -> 3.9, 494 x 1280 bf16 8.2 -> 7.1, 1200 x 640
// float32 10.5 -> 9.4, 1024 x 1280 bf16 12.6 -> 11.0 (a launch after another, 1.5 us of each the boundary).  Two launches cost ~11 us however
// small the tensor is.
template <typename Tin, typename Tout, int NV, int V, bool PAIR>
__global__ __launch_bounds__(1024) void gn_group_reg_kernel(const Tin* __restrict__ x, Tout* __restrict__ y,
                                                            const float* stale, float* sums_out,
                                                            const float* __restrict__ gamma, const float* __restrict__ beta,
                                                            int pix, int C, int G, int B, int patch_idx, int N, float eps,
                                                            int stat_mode, int silu, int packed, GnHalo halo, GnCount cnt,
                                                            GnFrom<PAIR> pr) {
  __shared__ float s_s[16], s_q[16];
  __shared__ float s_mr[3];
  const int g = blockIdx.x, b = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = (int)blockDim.x >> 6;   // (16 waves)
  const int cg = C / G, cgv = cg / V;
  const int ppass = blockDim.x / cgv;
  const int cv = tid % cgv, psub = tid / cgv;
  const bool active = psub < ppass;
  const int c0 = g * cg + cv * V;
  const long long base = (long long)b * pix;
  const float piv = gn_value<PAIR>(x, pr, C, base, g * cg);   // sums are taken of x - piv
  int pitch;
  const Tin* const xs = gn_source<PAIR>(x, pr, C, c0, &pitch);
  // everything that does not depend on x is requested first: affine parameters and, in the first wave, the cached sums (lane j:
  // patch j; added only after x has been requested - waited for here they held up the wave's share of x)
  float gm[V], bt[V];
#pragma unroll
  for (int i = 0; i < V; ++i) { gm[i] = 0.f; bt[i] = 0.f; }
  if (active) { ld_chan<V>(gamma + c0, gm); ld_chan<V>(beta + c0, bt); }
  const bool cached = stale != nullptr && !(N == 1 && stat_mode != DF_GN_STALE);
  float2 st = make_float2(0.f, 0.f);
  if (cached && tid < 64 && lane < N) {
    const float* sp = stale + (((long long)lane * B + b) * G + g) * 2;
    st.x = sp[0]; st.y = sp[1];
  }
  float v[NV][V];
  float a = 0.f, q = 0.f;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int p = psub + k * ppass;
    ld_chan<V>(xs + (base + (p < pix ? p : pix - 1)) * pitch, v[k]);      // (without branches; absent pixels are not added)
  }
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const bool here = active && psub + k * ppass < pix;
#pragma unroll
    for (int i = 0; i < V; ++i) { const float d = here ? v[k][i] - piv : 0.f; a += d; q = fmaf(d, d, q); }
  }
  a = wave_total(a); q = wave_total(q);
  if (lane == 0) { s_s[wave] = a; s_q[wave] = q; }
  __syncthreads();
  if (tid < 64) {
    const float fs = wave_total(lane < nw ? s_s[lane] : 0.f), fq = wave_total(lane < nw ? s_q[lane] : 0.f);
    double st_s = 0.0, st_q = 0.0, own_s = 0.0, own_q = 0.0;
    if (cached && N > 64) {
      gn_stale_wave(stale, b, g, B, G, N, patch_idx, lane, st_s, st_q, own_s, own_q);
    } else if (cached) {
      for (int j = 0; j < N; ++j) {                             // patch order fixes the order of the additions
        const float aj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(st.x), j));
        const float cj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(st.y), j));
        if (j == patch_idx) { own_s = aj; own_q = cj; } else { st_s += aj; st_q += cj; }
      }
    }
    if (tid == 0) {
      double S, SS;
      gn_unshift(fs, fq, cnt.n_loc, piv, S, SS);
      const GnMoments mo = gn_combine_pre(S, SS, cnt, 1, N, stat_mode, st_s, st_q, own_s, own_q, eps);
      if (sums_out != nullptr) {                     // after the stale sums were read: may alias the own slot
        float* o = sums_out + ((long long)b * G + g) * 2;
        o[0] = (float)S; o[1] = (float)SS;
      }
      s_mr[0] = mo.mean_hi; s_mr[1] = mo.mean_lo; s_mr[2] = mo.rstd;
    }
  }
  __syncthreads();
  if (!active) return;
  const float mean = s_mr[0], mean_lo = s_mr[1], rstd = s_mr[2];
  float sc[V], sh[V];
#pragma unroll
  for (int i = 0; i < V; ++i) {
    sc[i] = rstd * gm[i];
    sh[i] = bt[i];
  }
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int p = psub + k * ppass;
    if (p >= pix) continue;
    float o4[V];
#pragma unroll
    for (int i = 0; i < V; ++i) {
      const float t = fmaf((v[k][i] - mean) - mean_lo, sc[i], sh[i]);
      o4[i] = silu ? silu_f(t) : t;
    }
    const long long m = base + p;
    if constexpr (PAIR) st_chan<V>(pr.cat + m * C + c0, v[k]);
    Tout* o = y + m * C + c0;
    if (packed) o = y + (((m >> 5) * (C >> 4) + (c0 >> 4)) * 64 + (m & 31) + 32 * ((c0 >> 3) & 1)) * 8 + (c0 & 7);
    st_chan<V>(o, o4);
    if constexpr (sizeof(Tout) == 2) {
      if (halo.out) halo_store<V>(halo, b, p, C, c0, o4);
    }
  }
}

// Larger patches in one launch: x is read once and stays in registers, as above, but P workgroups share the groups of an eighth of the
// channels (a slab), each with a range of pixels, and hand each other their sums.  The workgroups of a slab lie on one XCD
// (workgroups go round-robin over the eight, so blockIdx % 8 is the slab), and a sum goes through that XCD's L2 as an 8-byte word with the
// launch's number beside the float, so one store and one poll pass it on: 0.9 us with the wait for the slowest, where an exchange
// over all XCDs takes 5 and a second launch 2 and another read of x.
//   - The result depends neither on where the workgroups are nor on all of them being there at once: after `wait` polls (0.2 us each, all
//     together what a second launch costs; launches and steps with the chip to themselves are as fast with 8 as with 1024) a workgroup adds up the
//     ranges that are missing itself, in the same order, with the same bits, and hands them on.  So every wait ends.  Beside a kernel of another
//     stream on one unit of each XCD, 16384 x 960 bf16 45 us a launch (two launches 46); with 1024 polls, and every workgroup adding up all
//     ranges again, 361.  Where nobody waits for anybody 151 us, 4096 x 320 48.
//   - A word is of this launch and no other: gnmeet.h says how the number is chosen, also for replays of a recorded call and for calls that overlap.
// Bound by two round trips to memory and the exchange (32 x 128 x 320 bf16, us from the first start: requests out 1.6, sums 2.4, all
// there 3.3, moments 3.8, stored 4.4), by the rates of both beyond some 10 MB.  A launch after another, against two launches or (up to sixteen
// pixels per lane) a workgroup per group: 1024 x 320 float 7.3 -> 5.0 us, 4096 x 320 bf16 12.1 -> 6.5, 494 x 1280 float 6.5 -> 5.1,
// 1024 x 1280 bf16 10.8 -> 5.95, 4096 x 640 float 15.1 -> 8.4, 16384 x 960 bf16 27.1 -> 24.5.  One lane-ordered sum in LDS for the
// eight words of a workgroup (sums through LDS lane by lane, moments with the cached sums behind the exchange) took 2.5 us more.
constexpr int kGnMeetParts = 32, kGnMeetBatch = 8, kGnMeetGroups = 4, kGnMeetWait = 16;
// 8-byte words of a (batch item, slab): a line with the counters of tickets and of arrivals, then 8 per workgroup; and of a launch with P workgroups per slab
__host__ __device__ constexpr int gn_meet_stride(int P) { return 8 + 8 * P; }
constexpr size_t gn_meet_words(int P) { return (size_t)kGnMeetBatch * 8 * gn_meet_stride(P); }
// launches with 2, 4, .. 32 workgroups per slab have words of their own, one after the other
constexpr size_t gn_meet_offset(int P) {
  size_t o = 0;
  for (int q = 2; q < P; q *= 2) o += gn_meet_words(q);
  return o;
}
constexpr size_t kGnMeetWords = gn_meet_offset(2 * kGnMeetParts);
constexpr int kGnMeetCopies = 4;                         // of the library's own words, for calls that overlap
__device__ __align__(256) unsigned long long g_gn_words[kGnMeetCopies * kGnMeetWords];

// Indices come from shifts and reciprocals (P, the segments and a slab's groups are powers of two): tp lanes hold a pixel's channels of the
// slab, ppb pixels go through a workgroup at once.
struct GnMeet {
  unsigned long long* words;
  unsigned int id, tp_recip, cg_recip;
  int lgP, lgS, tp, ppb, pix_part, wait;                 // lgS: of the workgroups of a segment
};

// The wave's sums of eight words per lane: word 4 (lane / 32) + 2 (lane / 16 % 2) + lane / 8 % 2 in every eight lanes.  A step adds half of the
// words in half of the lanes.
__device__ __forceinline__ float swap_add32(float x, float y) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float swap_add16(float x, float y) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
template <int CTRL>
__device__ __forceinline__ float lane_move(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float wave_total8(const float (&w)[8], int lane) {
  float a[4], c[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) a[i] = swap_add32(w[i], w[i + 4]);
#pragma unroll
  for (int i = 0; i < 2; ++i) c[i] = swap_add16(a[i], a[i + 2]);
  const bool up = lane & 8;
  float t = (up ? c[1] : c[0]) + lane_move<0x128>(up ? c[0] : c[1]);   // row_ror:8
  t += lane_move<0x141>(t);                              // row_half_mirror
  t += lane_move<0xb1>(t);                               // quad_perm: lane ^ 1
  t += lane_move<0x4e>(t);                               // lane ^ 2
  return t;
}
// The sum over lanes lane % 8, + 8, + 16, ..: over 8 `over` of them (over = 1, 2, 4, 8)
__device__ __forceinline__ float eighth_total(float t, int over) {
  if (over > 1) t += lane_move<0x128>(t);
  if (over > 2) t = swap_add16(t, t);
  if (over > 4) t = swap_add32(t, t);
  return t;
}

template <typename Tin, typename Tout, int NV, bool PAIR>
__global__ __launch_bounds__(1024) void gn_meet_kernel(const Tin* __restrict__ x, Tout* __restrict__ y, const float* stale,
                                                       float* sums_out, const float* __restrict__ gamma,
                                                       const float* __restrict__ beta, int pix, int C, int G, int nseg, int B,
                                                       int patch_idx, int N, float eps, int stat_mode, int silu, int packed,
                                                       GnHalo halo, GnCount cnt, GnMeet mt, GnFrom<PAIR> pr) {
  constexpr int V = Elem<Tin>::kVec, NP = kGnMeetParts / 8;
  __shared__ float s_wave[16][8], s_all[kGnMeetParts][8], s_mom[kGnMeetGroups][3];
  __shared__ unsigned int s_missing;
  __shared__ int s_met;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int slab = blockIdx.x & 7, loc = blockIdx.x >> 3, P = 1 << mt.lgP;
  const int b = loc >> mt.lgP, part = loc & (P - 1), pps = 1 << mt.lgS;
  unsigned long long* const words = mt.words + (size_t)(b * 8 + slab) * gn_meet_stride(P);
  unsigned int ticket = 0;
  if (mt.id == 0 && tid == 0) ticket = __hip_atomic_fetch_add((unsigned int*)words, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const int Gs = G >> 3, g0 = slab * Gs, cg = C / G;
  const int psub = (int)quotient_u32(tid, mt.tp, mt.tp_recip), tc = tid - psub * mt.tp;
  const int cl = tc * V, la = (int)quotient_u32(cl, cg, mt.cg_recip), nb = (la + 1) * cg - cl;   // group of the slab, and its channels here
  const int c0 = slab * (C >> 3) + cl;
  const bool active = psub < mt.ppb;
  const long long item = (long long)b * nseg * pix;      // the batch item's first pixel
  const float pa = gn_value<PAIR>(x, pr, C, item, (g0 + la) * cg), pb = gn_value<PAIR>(x, pr, C, item, (g0 + (nb < V ? la + 1 : la)) * cg);
  // first wave: lane j * Gs + i holds patch j's cached sums of group g0 + i
  const bool cached = stale != nullptr && !(nseg > 1 || (N == 1 && stat_mode != DF_GN_STALE));
  float2 st = make_float2(0.f, 0.f);
  float gpiv = 0.f;
  if (wave == 0) {
    const int lg = Gs >> 1;                              // (Gs = 1, 2, 4)
    if (cached && lane < N * Gs) {
      const float* sp = stale + (((long long)(lane >> lg) * B + b) * G + g0 + (lane & (Gs - 1))) * 2;
      st.x = sp[0]; st.y = sp[1];
    }
    if (lane < Gs) gpiv = gn_value<PAIR>(x, pr, C, item, (g0 + lane) * cg);
  }
  int pitch;
  const Tin* xs;                                         // where the lane's channels of a batch item's pixels begin
  unsigned int xo = 0;
  if constexpr (PAIR) {
    xs = gn_source<PAIR>(x, pr, C, c0, &pitch);
    xs += item * pitch;
  } else {
    pitch = C;
    xs = x + item * C;                                   // (uniform: the lane's part is an offset)
    xo = (unsigned int)c0 * (unsigned int)sizeof(Tin);
  }
  u32x4 raw[NV];
  auto request = [&](int q) {                            // range q of the batch item; pixels that it does not have are others
    const unsigned int unit = (unsigned int)pitch * (unsigned int)sizeof(Tin), end = (unsigned int)(pix - 1) * unit + xo;
    const char* const base = (const char*)(xs + (long long)(q >> mt.lgS) * pix * pitch);
    unsigned int o = (unsigned int)((q & (pps - 1)) * mt.pix_part + psub) * unit + xo;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      raw[k] = *reinterpret_cast<const u32x4*>(base + (o < end ? o : end));
      o += (unsigned int)mt.ppb * unit;
    }
  };
  auto range = [&](int q, int& lo, int& hi) {
    lo = (q & (pps - 1)) * mt.pix_part;
    hi = lo + mt.pix_part < pix ? lo + mt.pix_part : pix;
  };
  // sums of range q, which is in the registers, to the first wave: word lane % 8 is the sum (0 - 3) or the sum of squares (4 - 7) of x - pivot
  // of group lane % 4
  auto sums = [&](int q) {
    int lo, hi;
    range(q, lo, hi);
    float s0 = 0.f, q0 = 0.f, s1 = 0.f, q1 = 0.f;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const bool here = active && lo + psub + k * mt.ppb < hi;
      float v[V];
      unpack_vec<Tin>(raw[k], v);
#pragma unroll
      for (int i = 0; i < V; ++i) {
        const bool first = i < nb;
        const float d = here ? v[i] - (first ? pa : pb) : 0.f;
        const float d0 = first ? d : 0.f, d1 = first ? 0.f : d;
        s0 += d0; q0 = fmaf(d0, d0, q0);
        s1 += d1; q1 = fmaf(d1, d1, q1);
      }
      if constexpr (NV > 4) __builtin_amdgcn_sched_barrier(0);          // (a pixel at a time: 128 registers per lane)
    }
    float w[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      w[i] = la == i ? s0 : la + 1 == i ? s1 : 0.f;
      w[i + 4] = la == i ? q0 : la + 1 == i ? q1 : 0.f;
    }
    const float t = wave_total8(w, lane);
    if ((lane & 7) == 0) s_wave[wave][lane >> 3] = t;
    __syncthreads();
    float r = 0.f;
    if (wave == 0) r = eighth_total(s_wave[lane >> 3][lane & 7] + s_wave[8 + (lane >> 3)][lane & 7], 8);
    return r;
  };
  request(part);
  const float mine = sums(part);
  float gm[V], bt[V];                                    // (beside the exchange)
  ld_vec(gamma + c0, gm); ld_vec(beta + c0, bt);
  if constexpr (V == 8) { ld_vec(gamma + c0 + 4, gm + 4); ld_vec(beta + c0 + 4, bt + 4); }
  __builtin_amdgcn_sched_barrier(0);
  bool met = false;
  float val[NP];                                         // word lane % 8 of range lane / 8 + 8 i
  unsigned int tag = 0;
  double st_s = 0.0, st_q = 0.0, own_s = 0.0, own_q = 0.0;
  bool writes = false;                                   // the patch's own sums
  auto hand = [&](int q, float t) {                      // the sums of range q
    if (lane < 8)
      __hip_atomic_store(words + 8 + q * 8 + lane, (unsigned long long)tag << 32 | __float_as_uint(t), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  // the words of the ranges in `missing` (a bit each) that have come, to s_all; those that have not
  auto look = [&](unsigned int missing) {
    unsigned int left = 0;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int q = (lane >> 3) + 8 * i;
      bool gone = missing >> q & 1u;
      if (gone) {
        const unsigned long long w = __hip_atomic_load(words + 8 + lane + 64 * i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        gone = (unsigned int)(w >> 32) != tag;
        if (!gone) s_all[q][lane & 7] = __uint_as_float((unsigned int)w);
      }
      unsigned long long m = __ballot(gone);             // a bit per word: gathered to one per range
      m |= m >> 4; m |= m >> 2; m |= m >> 1;
      left |= (unsigned int)((m & 0x0101010101010101ull) * 0x0102040810204080ull >> 56) << (8 * i);
    }
    return left;
  };
  if (wave == 0) {
    tag = gn_meet_number(mt.id, (unsigned int)__builtin_amdgcn_readfirstlane((int)ticket), mt.lgP);
    hand(part, mine);
    writes = gn_meet_writes(false, 0, P, part);
    unsigned int arrived = 0;
    const bool counted = mt.id == 0 && cached && gn_reads_own(stat_mode);   // (id 0: words that no other launch uses)
    if (counted) {
      // the cached sums are here before this workgroup counts itself: the last to do so overwrites the patch's own, which may lie among them
      unsigned int one = 1u;
      asm volatile("" : "+v"(one) : "v"(st.x), "v"(st.y));
      if (lane == 0) arrived = __hip_atomic_fetch_add((unsigned int*)words + 1, one, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (cached)
      for (int j = 0; j < N; ++j) {                      // patch order fixes the order of the additions
        const float aj = __shfl(st.x, j * Gs + (lane & (Gs - 1)), 64), cj = __shfl(st.y, j * Gs + (lane & (Gs - 1)), 64);
        if (j == patch_idx) { own_s = aj; own_q = cj; } else { st_s += aj; st_q += cj; }
      }
    for (int n = 0; n < mt.wait && !met; ++n) {
      bool ok = true;
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        unsigned long long w = (unsigned long long)tag << 32;
        if ((lane >> 3) + 8 * i < P) w = __hip_atomic_load(words + 8 + lane + 64 * i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        val[i] = __uint_as_float((unsigned int)w);
        ok &= (unsigned int)(w >> 32) == tag;
      }
      met = __all(ok);
    }
    if (lane == 0) s_met = met;
    if (counted) writes = gn_meet_writes(true, (unsigned int)__builtin_amdgcn_readfirstlane((int)arrived), P, part);
  }
  auto moments = [&] {                                   // of the slab's groups, by lanes 0 .. Gs - 1 of the first wave
    double tot_s = 0.0, tot_q = 0.0;
    auto segment = [&](float t, int sg) {                // a segment's words
      double S, SS;
      gn_unshift(t, lane_move<0x104>(t), cnt.n_loc, gpiv, S, SS);   // row_shl:4
      tot_s += S; tot_q += SS;
      if (nseg > 1 && writes && lane < Gs) {
        float* o = sums_out + (((long long)sg * B + b) * G + g0 + lane) * 2;
        o[0] = (float)S; o[1] = (float)SS;
      }
    };
    if (nseg == 1) {
      float t = val[0];
#pragma unroll
      for (int i = 1; i < NP; ++i) t += val[i];
      segment(eighth_total(t, 8), 0);
    } else {
#pragma unroll
      for (int i = 0; i < NP; ++i) val[i] = eighth_total(val[i], pps < 8 ? pps : 8);
      for (int sg = 0; sg < nseg; ++sg) {
        float t = 0.f;
#pragma unroll
        for (int i = 0; i < NP; ++i)
          if (i >= (sg * pps) >> 3 && 8 * i < (sg + 1) * pps) t += val[i];
        segment(__shfl(t, ((sg * pps) & 7) * 8 + (lane & 7), 64), sg);
      }
    }
    if (lane < Gs) {
      const GnMoments mo = gn_combine_pre(tot_s, tot_q, cnt, nseg, N, stat_mode, st_s, st_q, own_s, own_q, eps);
      s_mom[lane][0] = mo.mean_hi; s_mom[lane][1] = mo.mean_lo; s_mom[lane][2] = mo.rstd;
      if (nseg == 1 && sums_out != nullptr && writes) {
        float* o = sums_out + ((long long)b * G + g0 + lane) * 2;
        o[0] = (float)tot_s; o[1] = (float)tot_q;
      }
    }
  };
  if (met) moments();
  __syncthreads();
  if (__builtin_expect(!s_met, 0)) {
    // Some range did not appear.  Those that are missing are added up here, each workgroup beginning with another one.
    auto left = [&](unsigned int missing) {              // told to all waves
      if (wave == 0) {
        if (mt.wait > 0 && missing) missing = look(missing);
        if (lane == 0) s_missing = missing;
      }
      __syncthreads();
      return (unsigned int)__builtin_amdgcn_readfirstlane((int)s_missing);
    };
    unsigned int missing = left(P < 32 ? (1u << P) - 1u : ~0u);
    while (missing) {
      unsigned int rest = missing;
      for (int k = part % __popc(missing); k > 0; --k) rest &= rest - 1;
      const int q = __ffs(rest) - 1;
      request(q);
      const float t = sums(q);
      if (wave == 0) {
        if (lane < 8) s_all[q][lane] = t;
        if (mt.wait > 0) hand(q, t);
      }
      missing = left(missing & ~(1u << q));
    }
    int own = part;                                      // (the addresses of the first time kept until here did not fit the registers)
    asm volatile("" : "+s"(own));
    request(own);
    if (wave == 0) {
#pragma unroll
      for (int i = 0; i < NP; ++i) val[i] = (lane >> 3) + 8 * i < P ? s_all[(lane >> 3) + 8 * i][lane & 7] : 0.f;
      moments();
    }
    __syncthreads();
  }
  if (!active) return;
  const int lb = nb < V ? la + 1 : la;
  const float ma = s_mom[la][0], mla = s_mom[la][1], ra = s_mom[la][2], mb = s_mom[lb][0], mlb = s_mom[lb][1], rb = s_mom[lb][2];
  int lo, hi;
  range(part, lo, hi);
  const int seg = part >> mt.lgS;
#pragma unroll
  for (int i = 0; i < V; ++i) gm[i] *= i < nb ? ra : rb;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int p = lo + psub + k * mt.ppb;
    if (p >= hi) break;
    float v[V];
    unpack_vec<Tin>(raw[k], v);
    const long long m = item + (long long)seg * pix + p;
    if constexpr (PAIR) {
      const u32x2 t = {pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3])};
      *reinterpret_cast<u32x2*>(pr.cat + m * C + c0) = t;
    }
#pragma unroll
    for (int i = 0; i < V; ++i) {
      const float t = fmaf((v[i] - (i < nb ? ma : mb)) - (i < nb ? mla : mlb), gm[i], bt[i]);
      v[i] = silu ? silu_f(t) : t;
    }
    Tout* o = y + m * C + c0;
    if (packed) o = y + (((m >> 5) * (C >> 4) + (c0 >> 4)) * 64 + (m & 31) + 32 * ((c0 >> 3) & 1)) * 8 + (c0 & 7);
    if constexpr (sizeof(Tout) == sizeof(Tin)) {
      st_vec(o, v);
    } else {
      const u32x2 t = {pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3])};
      *reinterpret_cast<u32x2*>(o) = t;
    }
    if constexpr (sizeof(Tout) == 2) {
      if (halo.out) halo_store<V>(halo, b, (long long)seg * pix + p, C, c0, v);
    }
    if constexpr (NV > 4) __builtin_amdgcn_sched_barrier(0);
  }
}

// Strips of the two-launch path: as close to target_blocks strips as the pixel count allows (the chip has 256
// compute units and a strip is one block in either launch); a small tensor gets short strips and blocks with few
// pixel slots rather than few blocks.
GnLayout gn_layout(int C, int vec, long long pix, int target_blocks, int max_threads, int min_threads) {
  GnLayout L;
  L.tp = C / vec;
  long long per = (pix + target_blocks - 1) / target_blocks;
  L.ppb = max_threads / L.tp;
  if (L.ppb > kGnMaxPpb) L.ppb = kGnMaxPpb;
  if (L.ppb > per) L.ppb = (int)per;
  if (L.ppb * L.tp < min_threads) L.ppb = (min_threads + L.tp - 1) / L.tp;   // the kernels give every group a thread
  if (L.ppb < 1) L.ppb = 1;
  L.threads = L.tp * L.ppb;
  per = (per + L.ppb - 1) / L.ppb * L.ppb;
  L.pix_per_blk = (int)per;
  L.nblk = (int)((pix + per - 1) / per);
  return L;
}

}  // namespace

size_t groupnorm_meet_bytes() { return kGnMeetWords * sizeof(unsigned long long); }

size_t groupnorm_scratch_bytes(int B, int nseg, int G, int N) {
  // snapshot of the cached sums + partials of at most kGnMaxStrips strips per batch item
  (void)nseg;
  return kScratchCounterBytes + ((size_t)B * kGnMaxStrips * G * 2 + (size_t)N * B * G * 2 + 64) * sizeof(float) + 1024;
}

namespace {
// One launch that keeps its pixels in registers (nv > 0: that many per lane; P > 0: P workgroups per slab), one launch of a workgroup per
// group (`group`), or two.
struct GnForm { int v, nv; bool group; int P, tp, ppb, pix_part; };
// The form whose workgroups hand each other their sums (P = 0: it does not take the call).  As many workgroups as the compute units of
// an XCD while each has a pixel per lane: 64 x 64 x 640 float 8.8 us with 32 per slab, 10.5 with 16; two batch items 12.6 with 16 each, 15.6 with 32.
GnForm gn_meet_form(const GnArgs& a) {
  GnForm f = {};
  const int V = a.in_dtype == DF_BF16 ? 8 : 4, Gs = a.G / 8;
  const long long pix = (long long)a.Rseg * a.W;
  if (a.G % 8 || (Gs != 1 && Gs != 2 && Gs != 4) || a.C % (8 * V) || a.C / a.G < V || a.N > 16 || a.B > kGnMeetBatch) return f;
  if (a.nseg != 1 && a.nseg != 2 && a.nseg != 4 && a.nseg != 8) return f;
  // y over x: a workgroup that has to add up another's range would find results in it
  const size_t n = (size_t)a.B * a.nseg * pix * a.C;
  const uintptr_t x = (uintptr_t)a.x, y = (uintptr_t)a.y;
  if (x && x < y + n * (a.out_dtype == DF_BF16 ? 2 : 4) && y < x + n * (a.in_dtype == DF_BF16 ? 2 : 4)) return f;
  f.tp = a.C / 8 / V;
  if (f.tp > 1024) return f;
  f.ppb = 1024 / f.tp;
  int P = a.nseg;
  while (P < 2 || (2 * P <= kGnMeetParts / a.B && pix > (long long)f.ppb * (P / a.nseg))) P *= 2;
  if (const char* e = tune_env("DF_GN_MEET")) { if (atoi(e) > 1) P = atoi(e); if (P < 2 || P % a.nseg) return f; }
  const long long part = (pix + P / a.nseg - 1) / (P / a.nseg), nv = (part + f.ppb - 1) / f.ppb;
  if (nv > 8) return f;                                  // (sixteen do not fit the registers)
  f.nv = 1;
  while (f.nv < nv) f.nv *= 2;
  f.pix_part = (int)part;
  f.P = P;
  return f;
}
GnForm gn_form(const GnArgs& a) {
  const int cg = a.C / a.G;
  const long long pix_seg = (long long)a.Rseg * a.W, per_group = pix_seg * a.nseg * cg;
  static const bool no_fused = tune_env("DF_GN_3K") != nullptr;   // tuning aid
  // channels per lane of the form that keeps its pixels in registers, and pixels per pass of its 1024 lanes
  const int v = cg % 4 == 0 ? 4 : cg % 2 == 0 ? 2 : 0;
  const int ppass = (v && cg / v <= 1024) ? 1024 / (cg / v) : 0;
  // up to 16 pixels per lane (a workgroup's loads then take as long as the second launch would); the kernel requests nv of them
  // whether they are there or not, so nv is the power of two from 2 on that holds the lane's share
  int nv = a.nseg == 1 && ppass && pix_seg <= (long long)ppass * 16 ? 2 : 0;
  while (nv && (long long)ppass * nv < pix_seg) nv *= 2;
  if (no_fused) return {v, 0, false};
  // Handing over the sums costs 1 us, which a workgroup per group saves while its lanes have up to four pixels (300 x 1280 float 5.0 us both
  // ways, bf16 5.2 against 5.6; 494 x 960 5.9 against 5.1 and 6.2 against 5.9, 1024 x 320 7.3 against 5.0 and 6.6 against 5.7).
  // Of bf16 values, whose lanes hold twice as many channels, it takes more (300 x 960: 5.4 against 5.6).
  const char* e = tune_env("DF_GN_MEET");
  if (e ? atoi(e) != 0 : (nv == 0 || nv >= 8) && per_group >= (a.in_dtype == DF_BF16 ? 10000 : 8000)) {
    const GnForm m = gn_meet_form(a);
    if (m.P) return m;
  }
  return {v, nv, !nv && cg % 4 == 0 && cg / 4 <= 1024 && per_group <= kGnGroupMaxElems};
}
}  // namespace

namespace {
template <bool PAIR>
GnFrom<PAIR> gn_from(const GnArgs& a) {
  if constexpr (PAIR) return {a.x2, a.x2_from, (bf16_t*)a.cat_out};
  else return {};
}
}  // namespace

bool groupnorm_takes_pair(const GnArgs& a) {
  return a.G > 0 && a.C % a.G == 0 && a.in_dtype == DF_F32 && a.out_dtype == DF_BF16 && a.x2_from % 4 == 0 && !gn_form(a).group;
}

namespace {
__global__ __launch_bounds__(256) void gn_copy_sums(const float* __restrict__ stale, float* __restrict__ copy, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) copy[i] = stale[i];
}

int ilog2(int n) { return n > 1 ? 1 + ilog2(n / 2) : 0; }
__global__ __launch_bounds__(256) void gn_clear_words(unsigned long long* words, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) __hip_atomic_store(words + i, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
bool recording(hipStream_t st) {
  if (!st) return false;                                 // (the default stream cannot be recorded)
  hipStreamCaptureStatus s = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &s) != hipSuccess) { (void)hipGetLastError(); return true; }
  return s != hipStreamCaptureStatusNone;
}
// The words of a launch and its number (gnmeet.h): the caller's, or the library's on the current device
int gn_words(const GnArgs& a, int P, hipStream_t st, unsigned long long** words, unsigned int* id) {
  if (a.meet) {
    *words = (unsigned long long*)a.meet + gn_meet_offset(P);
    *id = 0;
    return DF_OK;
  }
  static std::atomic<unsigned long long*> at[64];
  static std::atomic<unsigned long long> calls[2];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return DF_EHIP;
  unsigned long long* w = at[dev].load(std::memory_order_relaxed);
  if (!w) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(g_gn_words)) != hipSuccess || !ptr) { (void)hipGetLastError(); return DF_EHIP; }
    w = (unsigned long long*)ptr;
    at[dev].store(w, std::memory_order_relaxed);
  }
  const bool rec = recording(st);
  const unsigned long long n = calls[rec].fetch_add(1, std::memory_order_relaxed);
  *id = gn_call_id(n, rec);
  *words = w + (n % kGnMeetCopies) * kGnMeetWords + gn_meet_offset(P);
  if (rec) {
    const int cleared = a.B * 8 * gn_meet_stride(P);
    hipLaunchKernelGGL(gn_clear_words, dim3(cdiv(cleared, 256)), dim3(256), 0, st, *words, cleared);
    DF_LAUNCH_CHECK();
  }
  return DF_OK;
}
}  // namespace

int launch_groupnorm(const GnArgs& a, hipStream_t st) {
  const int vec = a.in_dtype == DF_BF16 ? 8 : 4;
  if (a.C % a.G || a.C % vec || a.G > kMaxG || a.C / vec > 1024) return DF_ESHAPE;
  if (a.in_dtype == DF_BF16 && a.out_dtype != DF_BF16) return DF_ESHAPE;
  if (a.B > 1024) return DF_ESHAPE;
  if (a.y_packed && (a.out_dtype != DF_BF16 || a.C % 16)) return DF_ESHAPE;
  const long long pix_seg = (long long)a.Rseg * a.W;
  GnHalo halo = {};
  if (a.halo_out && a.halo_cols) {
    if (a.out_dtype != DF_BF16 || a.y_packed || a.halo_rpp <= 0 || a.W % a.halo_rpp || a.halo_patch0 < 0 ||
        a.halo_patch0 + a.W / a.halo_rpp > a.halo_npatch || ((uintptr_t)a.halo_out % 16))
      return DF_EINVAL;
    halo.out = (bf16_t*)a.halo_out; halo.W = a.W; halo.rpp = a.halo_rpp; halo.patch0 = a.halo_patch0;
    halo.npatch = a.halo_npatch; halo.cols = 1; halo.rows = a.Rseg * a.nseg;
  } else if (a.halo_out) {
    if (a.out_dtype != DF_BF16 || a.y_packed || a.halo_rpp <= 0 || ((long long)a.Rseg * a.nseg) % a.halo_rpp ||
        a.halo_patch0 < 0 || a.halo_patch0 + (a.Rseg * a.nseg) / a.halo_rpp > a.halo_npatch || ((uintptr_t)a.halo_out % 16))
      return DF_EINVAL;
    halo.out = (bf16_t*)a.halo_out; halo.W = a.W; halo.rpp = a.halo_rpp; halo.patch0 = a.halo_patch0;
    halo.npatch = a.halo_npatch;
    halo.single = ((long long)a.Rseg * a.nseg == a.halo_rpp) ? 1 : 0;
  }
  if (pix_seg <= 0 || pix_seg * a.nseg > 0x7fffffffLL) return DF_ESHAPE;
  if (a.x2 && (!a.cat_out || a.in_dtype != DF_F32 || a.out_dtype != DF_BF16 || a.x2_from % 4 || a.x2_from <= 0 || a.x2_from >= a.C ||
               ((uintptr_t)a.x2 % 16) || ((uintptr_t)a.cat_out % 16)))
    return DF_EINVAL;
  const double n_loc = (double)pix_seg * (double)(a.C / a.G);
  const double n_all = n_loc * (double)(a.nseg > 1 ? a.nseg : a.N > 1 ? a.N : 1);
  const GnCount cnt = {n_loc, 1.0 / n_loc, n_all, 1.0 / n_all};
  const bool need_stale = !(a.nseg > 1 || (a.N == 1 && a.stat_mode != DF_GN_STALE));
  if (need_stale && !a.stale) return DF_EINVAL;
  const int stale_n = need_stale ? a.N * a.B * a.G * 2 : 0;
  // small tensors: the whole GroupNorm in one launch, one workgroup per (group, batch item)
  {
    const GnForm form = gn_form(a);
    const int v = form.v, nv = form.nv;
    if (a.x2 && form.group) return DF_ESHAPE;
    if (form.P) {
      const float* stale = a.stale;
      if (need_stale && !a.meet && gn_meet_copies(stale, a.sums_out, (long long)a.B * a.G * 2, a.patch_idx, a.N, a.stat_mode)) {
        char* scr = scratch_region(a.scr, groupnorm_scratch_bytes(a.B, a.nseg, a.G, a.N));
        if (!scr) return DF_ENOMEM;
        float* copy = (float*)(scr + kScratchCounterBytes);
        hipLaunchKernelGGL(gn_copy_sums, dim3(cdiv(stale_n, 256)), dim3(256), 0, st, stale, copy, stale_n);
        DF_LAUNCH_CHECK();
        stale = copy;
      }
      unsigned long long* words = nullptr;
      unsigned int id = 0;
      if (const int rc = gn_words(a, form.P, st, &words, &id)) return rc;
      const GnMeet mt = {words, id, reciprocal_u32(form.tp), reciprocal_u32(a.C / a.G), ilog2(form.P),
                         ilog2(form.P / a.nseg), form.tp, form.ppb, form.pix_part, a.looks < 0 ? 0 : a.looks ? a.looks : kGnMeetWait};
#define DF_GN_MEET(TI, TO, NVV, PR)                                                                                         \
  hipLaunchKernelGGL((gn_meet_kernel<TI, TO, NVV, PR>), dim3(8 * form.P * a.B), dim3(1024), 0, st, (const TI*)a.x, (TO*)a.y, stale, \
                     a.sums_out, a.gamma, a.beta, (int)pix_seg, a.C, a.G, a.nseg, a.B, a.patch_idx, a.N, a.eps, a.stat_mode,      \
                     a.silu, a.y_packed, halo, cnt, mt, gn_from<PR>(a))
#define DF_GN_MEET_T(NVV)                                                                                                    \
  {                                                                                                                          \
    if (a.x2) DF_GN_MEET(float, bf16_t, NVV, true);                                                                          \
    else if (a.in_dtype == DF_BF16) DF_GN_MEET(bf16_t, bf16_t, NVV, false);                                                  \
    else if (a.out_dtype == DF_BF16) DF_GN_MEET(float, bf16_t, NVV, false);                                                  \
    else DF_GN_MEET(float, float, NVV, false);                                                                               \
  }
      if (form.nv == 1) DF_GN_MEET_T(1) else if (form.nv == 2) DF_GN_MEET_T(2) else if (form.nv == 4) DF_GN_MEET_T(4)
      else DF_GN_MEET_T(8)
#undef DF_GN_MEET_T
#undef DF_GN_MEET
      DF_LAUNCH_CHECK();
      return DF_OK;
    }
    if (nv || form.group) {
      dim3 grid(a.G, a.B);
      if (nv) {
        // one patch: single read of x
#define DF_GN_REG(TI, TO, NVV, VV, PR)                                                                                \
  hipLaunchKernelGGL((gn_group_reg_kernel<TI, TO, NVV, VV, PR>), grid, dim3(1024), 0, st, (const TI*)a.x, (TO*)a.y, a.stale, \
                     a.sums_out, a.gamma, a.beta, (int)pix_seg, a.C, a.G, a.B, a.patch_idx, a.N, a.eps, a.stat_mode,  \
                     a.silu, a.y_packed, halo, cnt, gn_from<PR>(a))
#define DF_GN_REG_T(NVV, VV)                                                                                          \
  {                                                                                                                   \
    if (a.x2) DF_GN_REG(float, bf16_t, NVV, VV, true);                                                                \
    else if (a.in_dtype == DF_BF16) DF_GN_REG(bf16_t, bf16_t, NVV, VV, false);                                        \
    else if (a.out_dtype == DF_BF16) DF_GN_REG(float, bf16_t, NVV, VV, false);                                        \
    else DF_GN_REG(float, float, NVV, VV, false);                                                                     \
  }
#define DF_GN_REG_V(VV)                                                                                               \
  {                                                                                                                   \
    if (nv == 2) DF_GN_REG_T(2, VV) else if (nv == 4) DF_GN_REG_T(4, VV)                                              \
    else if (nv == 8) DF_GN_REG_T(8, VV) else DF_GN_REG_T(16, VV)                                                     \
  }
        if (v == 4) DF_GN_REG_V(4) else DF_GN_REG_V(2)
#undef DF_GN_REG_V
#undef DF_GN_REG_T
#undef DF_GN_REG
        DF_LAUNCH_CHECK();
        return DF_OK;
      }
#define DF_GN_GROUP(TI, TO)                                                                                         \
  hipLaunchKernelGGL((gn_group_kernel<TI, TO>), grid, dim3(1024), 0, st, (const TI*)a.x, (TO*)a.y, a.stale, a.sums_out, \
                     a.gamma, a.beta, (int)pix_seg, a.C, a.G, a.nseg, a.B, a.patch_idx, a.N, a.eps, a.stat_mode, a.silu, \
                     a.y_packed, halo, cnt)
      if (a.in_dtype == DF_BF16) DF_GN_GROUP(bf16_t, bf16_t);
      else if (a.out_dtype == DF_BF16) DF_GN_GROUP(float, bf16_t);
      else DF_GN_GROUP(float, float);
#undef DF_GN_GROUP
      DF_LAUNCH_CHECK();
      return DF_OK;
    }
  }
  // Both launches use the same partition of the pixels into strips, at most kGnMaxStrips per batch item: every block
  // of the second launch reads all partials of its batch item, so their number is bounded, and a block normalises
  // the strip whose sums it (or a block on the same XCD) took, which is then still in that XCD's L2 for tensors of a
  // few MB per XCD.
  int target = kGnMaxStrips / a.nseg;
  if (target < 1) target = 1;
  GnLayout L = gn_layout(a.C, vec, pix_seg, target, 1024, a.G);
  if (L.threads > 1024 || L.ppb > kGnMaxPpb) return DF_ESHAPE;
  char* scr = scratch_region(a.scr, groupnorm_scratch_bytes(a.B, a.nseg, a.G, a.N));
  if (!scr) return DF_ENOMEM;
  float* stale_copy = (float*)(scr + kScratchCounterBytes);
  float* partial = stale_copy + (((size_t)a.N * a.B * a.G * 2 + 63) / 64) * 64;
  dim3 gs(L.nblk, a.nseg, a.B);
  const size_t lds = (size_t)vec * L.threads * sizeof(float);
  const int thr_apply = L.threads < a.G ? a.G : L.threads;   // the fold needs a lane per group
  const int iters = L.pix_per_blk / L.ppb;              // pixels per lane and strip
#define DF_GN_STATS(TI, NCHV, PR)                                                                                     \
  hipLaunchKernelGGL((gn_stats<TI, NCHV, PR>), gs, dim3(L.threads), lds, st, (const TI*)a.x, partial, (int)pix_seg, a.C,  \
                     a.G, L.tp, L.ppb, L.pix_per_blk, a.nseg, need_stale ? a.stale : nullptr, stale_copy, stale_n, gn_from<PR>(a))
#define DF_GN_APPLY(TI, TO, NCHV, PR)                                                                                 \
  hipLaunchKernelGGL((gn_apply<TI, TO, NCHV, PR>), gs, dim3(thr_apply), 0, st, (const TI*)a.x, (TO*)a.y, partial,         \
                     stale_copy, a.sums_out, a.gamma, a.beta, (int)pix_seg, a.C, a.G, L.nblk, a.nseg, a.B, a.patch_idx, \
                     a.N, a.eps, a.stat_mode, L.tp, L.ppb, L.pix_per_blk, a.silu, a.y_packed, halo, cnt, gn_from<PR>(a))
#define DF_GN_BOTH(NCHV)                                                                                              \
  {                                                                                                                   \
    if (a.x2) DF_GN_STATS(float, NCHV, true);                                                                         \
    else if (a.in_dtype == DF_BF16) DF_GN_STATS(bf16_t, NCHV, false);                                                 \
    else DF_GN_STATS(float, NCHV, false);                                                                             \
    DF_LAUNCH_CHECK();                                                                                                \
    if (a.x2) DF_GN_APPLY(float, bf16_t, NCHV, true);                                                                 \
    else if (a.in_dtype == DF_BF16) DF_GN_APPLY(bf16_t, bf16_t, NCHV, false);                                         \
    else if (a.out_dtype == DF_BF16) DF_GN_APPLY(float, bf16_t, NCHV, false);                                         \
    else DF_GN_APPLY(float, float, NCHV, false);                                                                      \
  }
  if (iters <= 1) DF_GN_BOTH(1) else if (iters <= 2) DF_GN_BOTH(2) else if (iters <= 4) DF_GN_BOTH(4) else DF_GN_BOTH(8)
#undef DF_GN_BOTH
#undef DF_GN_APPLY
#undef DF_GN_STATS
  DF_LAUNCH_CHECK();
  return DF_OK;
}

// Per-strip sums of a full image for vertical strips (the synchronous step only: not on the hot path).  One
// workgroup per (strip, group, batch item); sums of x minus the group's pivot, ordered fold, turned into sums of x
// in double.
template <typename Tin>
__global__ __launch_bounds__(256) void gn_strip_sums_kernel(const Tin* __restrict__ x, float* __restrict__ sums, int B,
                                                            int R, int W, int C, int G, int N) {
  __shared__ float s_s[256], s_q[256];
  const int j = blockIdx.x, g = blockIdx.y, b = blockIdx.z, tid = threadIdx.x;
  const int cg = C / G, Wp = W / N;
  const float piv = Elem<Tin>::ld(x + (long long)b * R * W * C + g * cg);
  const long long n = (long long)R * Wp * cg;
  float a = 0.f, q = 0.f;
  for (long long i = tid; i < n; i += 256) {
    const int ch = (int)(i % cg);
    const long long px = i / cg;
    const int c = (int)(px % Wp), r = (int)(px / Wp);
    const float d = Elem<Tin>::ld(x + (((long long)b * R + r) * W + j * Wp + c) * C + g * cg + ch) - piv;
    a += d; q = fmaf(d, d, q);
  }
  s_s[tid] = a; s_q[tid] = q;
  __syncthreads();
  if (tid == 0) {
    float fs = 0.f, fq = 0.f;
    for (int k = 0; k < 256; ++k) { fs += s_s[k]; fq += s_q[k]; }
    double S, SS;
    gn_unshift(fs, fq, (double)n, piv, S, SS);
    float* o = sums + (((long long)j * B + b) * G + g) * 2;
    o[0] = (float)S; o[1] = (float)SS;
  }
}

int launch_gn_strip_sums(const void* x, int in_dtype, float* sums, int B, int R, int W, int C, int G, int N, hipStream_t st) {
  if (B <= 0 || R <= 0 || W <= 0 || C <= 0 || G <= 0 || N <= 0 || C % G || W % N || G > 65535 || B > 65535) return DF_ESHAPE;
  dim3 grid(N, G, B);
  if (in_dtype == DF_BF16)
    hipLaunchKernelGGL(gn_strip_sums_kernel<bf16_t>, grid, dim3(256), 0, st, (const bf16_t*)x, sums, B, R, W, C, G, N);
  else
    hipLaunchKernelGGL(gn_strip_sums_kernel<float>, grid, dim3(256), 0, st, (const float*)x, sums, B, R, W, C, G, N);
  DF_LAUNCH_CHECK();
  return DF_OK;
}

// Argument validation shared by the two GroupNorm entry points of the C ABI.
int groupnorm_entry(const void* x_fresh, void* y, const float* stale_stats, float* fresh_stats_out, const float* gamma,
                    const float* beta, int B, int R, int W, int C, int G, int patch_idx, int N, float eps, int stat_mode,
                    int fuse_silu, int dtype, const Scratch* scr, hipStream_t st, int looks) {
  if (!x_fresh || !y || !gamma || !beta || (dtype != DF_F32 && dtype != DF_BF16)) return DF_EINVAL;
  if (stat_mode < DF_GN_SUMS || stat_mode > DF_GN_STALE) return DF_EINVAL;
  if (B <= 0 || R <= 0 || W <= 0 || C <= 0 || G <= 0 || N <= 0 || patch_idx < 0 || patch_idx >= N) return DF_ESHAPE;
  if ((N > 1 || stat_mode == DF_GN_STALE) && !stale_stats) return DF_EINVAL;
  if (((uintptr_t)x_fresh % 16) || ((uintptr_t)y % 16)) return DF_EINVAL;
  GnArgs a = {};
  a.x = x_fresh; a.y = y; a.stale = stale_stats; a.sums_out = fresh_stats_out; a.gamma = gamma; a.beta = beta;
  a.B = B; a.Rseg = R; a.W = W; a.C = C; a.G = G; a.nseg = 1; a.patch_idx = patch_idx; a.N = N; a.eps = eps;
  a.stat_mode = stat_mode; a.silu = fuse_silu ? 1 : 0; a.in_dtype = dtype; a.out_dtype = dtype;
  a.scr = scr; a.looks = looks;
  return launch_groupnorm(a, st);
}

}  // namespace df

// ---- the entry point for callers that cannot allocate ----
// Its kernels take their partial sums from this array instead of an allocated region.  Every GPU the library runs on
// holds its own copy until the process ends; host code reaches it only through the address hipGetSymbolAddress
// returns for the current device.
static constexpr size_t kStaticScratchBytes = DF_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {
void* g_static_scratch[64];            // per device: address of that device's copy of `scratch`
std::mutex g_static_scratch_mu;

int static_scratch_region(df::Scratch* out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return DF_EHIP;
  std::lock_guard<std::mutex> lock(g_static_scratch_mu);
  if (!g_static_scratch[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) { (void)hipGetLastError(); return DF_EHIP; }
    g_static_scratch[dev] = ptr;
  }
  out->ptr = (char*)g_static_scratch[dev];
  out->bytes = kStaticScratchBytes;
  return DF_OK;
}
}  // namespace

extern "C" {
#pragma GCC visibility push(default)

int df_groupnorm_stale_noalloc(const void* x_fresh, void* y, const float* stale_stats, float* fresh_stats_out,
                               const float* gamma, const float* beta, int B, int R, int W, int C, int G, int patch_idx,
                               int N, float eps, int stat_mode, int fuse_silu, int dtype, void* stream) {
  if (B <= 0 || G <= 0) return DF_ESHAPE;
  // the statistics pass keeps up to 256 partial (sum, sum of squares) pairs per batch item and group, plus a snapshot
  // of the cached sums
  if (N <= 0 || df::groupnorm_scratch_bytes(B, 1, G, N) > kStaticScratchBytes) return DF_ENOMEM;
  df::Scratch region = {nullptr, 0};
  const int rc = static_scratch_region(&region);
  if (rc != DF_OK) return rc;
  // nothing in the region has to start at zero: every partial and every statistic is written before it is read
  return df::groupnorm_entry(x_fresh, y, stale_stats, fresh_stats_out, gamma, beta, B, R, W, C, G, patch_idx, N, eps,
                             stat_mode, fuse_silu, dtype, &region, (hipStream_t)stream);
}

#pragma GCC visibility pop
}  // extern "C"
