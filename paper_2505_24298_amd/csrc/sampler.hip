// Fused vocabulary-wide sampler: temperature, fixed-point softmax mass,
// top-p nucleus, Philox draw, behaviour and full log-probabilities.
//
// One work-group of 16 wavefronts per row of logits.  The row is cut into
// segments of 256 consecutive token ids (one wavefront pass, 4 ids per lane,
// 16-byte loads); all order-sensitive steps work on per-segment integer sums
// in LDS, so the result does not depend on how the row was split.
//
// A row is spread over up to 64 work-groups instead, with partial results in a scratch
// buffer in device memory, where that is faster: few rows (fewer than half the compute
// units) with the whole vocabulary kept (top-p = 1), and every nucleus (top-p < 1) over a
// large vocabulary.  top-p = 1: partial maxima, per-segment masses, and a third launch scans
// the masses and picks the token.  top-p < 1: see sampler_split_hist_kernel.  The masses are
// integers and the maximum is exact, so the token is the same either way.
//
// Determinism contract (include/areal.h, areal_sample_logprob): the token id
// is a pure function of the float32 logits.  Every floating-point step that
// feeds an integer decision is a single IEEE float32 operation; contraction
// into fused multiply-add is switched off for this whole file.
#include <algorithm>
#include <type_traits>
#include <mutex>
#include <string>

#include "../../include/areal.h"
#include "kernels.hpp"

#pragma clang fp contract(off)

namespace areal {

constexpr int SEG = 256, MAX_SEG = 1024;       // ids per segment, segments per row at most
constexpr int SAMPLER_MAX_PARTS = 64;          // work-groups one row can be spread over
constexpr int SAMPLER_SPLIT_MAX_ROWS = AREAL_SAMPLE_STATIC_MAX_ROWS;   // rows the scratch buffer holds
constexpr size_t SAMPLER_SCRATCH_ROW = 55616;  // bytes of it per row
static_assert(AREAL_SAMPLE_STATIC_MAX_VOCAB == SEG * MAX_SEG, "header limit = segments x ids per segment");

namespace {

constexpr int TPB = 1024, NWAVES = 16;
// Segments from which the nucleus is spread: 32 (about 8,192 ids) up to 64 rows, 48 above.  Logits N(0, 0.4), top-p
// 0.95, one work-group per row / spread: 8,192 ids 27 / 24 us at 1 row, 28.4 / 27.7 at 64, 28.9 / 30.9 at 128; 10,240 ids
// 31.5 / 33.2 at 128 rows; 12,288 ids 36.7 / 33.2; 32,768 ids 71 / 24 at 1 row, 72 / 40 at 128.
constexpr int NUCLEUS_SPLIT_MIN_SEG = 32, NUCLEUS_SPLIT_MIN_SEG_MANY = 48, NUCLEUS_FEW_ROWS = 64;
constexpr int NBINS = 257;   // masses are 33-bit (0 .. 2^32); top level bins = c >> 24


typedef unsigned long long u64;

// ---- specified exponential -----------------------------------------------
// mass = floor(min(sexp(x), 1) * 2^32) with sexp as specified in include/areal.h and the oracle.
// The specified steps that cannot change the integer are not executed: the result p * 2^n is scaled
// by 2^32 in the exponent (p in [0.7, 1.42], n >= -36: no subnormal, the product is exact); below
// x = -25 the clamped argument gives 2^32 e^-25 = 0.06, which truncates to the specified 0; and
// min(w, 1) is the comparison with 2^32 below.
// The rounding to an integer is an addition of 1.5 * 2^23 + 32: in that range floats are integers, to nearest and
// ties to even like rint (the constant is even), and the low bits of the sum are n + 32, shifted into the exponent as they are.
__device__ __forceinline__ float scaled_sexp(float x) {
  const float xs = fmaxf(x, -25.0f);
  const float u = xs * 1.44269502162933349609375f + 12582944.0f;            // 0x3FB8AA3B
  const float n = u - 12582944.0f;                                          // exact
  float r = xs - n * 0.693359375f;                                          // exact product
  r = r - n * -2.12194442749023437500e-4f;                                  // 0xB95E8083
  float p = 1.98412701138295233249664306640625e-4f;                         // 1/7!
  p = p * r; p = p + 1.388888922519981861114501953125e-3f;                   // 1/6!
  p = p * r; p = p + 8.333333767950534820556640625e-3f;                      // 1/5!
  p = p * r; p = p + 4.16666679084300994873046875e-2f;                       // 1/4!
  p = p * r; p = p + 0.1666666716337203979492187500f;                        // 1/3!
  p = p * r; p = p + 0.5f;
  p = p * r; p = p + 1.0f;
  p = p * r; p = p + 1.0f;
  return __int_as_float(__float_as_int(p) + (__float_as_int(u) << 23));
}
__device__ __forceinline__ u64 mass_of_scaled(float w) {
  // below 2^32 the value fits the 32-bit truncating conversion; only w = 1 gives 2^32 itself
  return w >= 4294967296.0f ? (1ull << 32) : (u64)__float2uint_rz(w);
}
__device__ __forceinline__ u64 mass_of(float z, float m) { return mass_of_scaled(scaled_sexp(z - m)); }

// ---- Philox4x32-10 (Salmon et al., SC'11) ----------------------------------
__device__ __forceinline__ u64 philox_draw(u64 seed, uint32_t seq_id, uint32_t position) {
  uint32_t c0 = position, c1 = seq_id, c2 = 0, c3 = 0;
  uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint32_t hi0 = __umulhi(0xD2511F53u, c0), lo0 = 0xD2511F53u * c0;
    const uint32_t hi1 = __umulhi(0xCD9E8D57u, c2), lo1 = 0xCD9E8D57u * c2;
    const uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
    c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
    k0 += 0x9E3779B9u; k1 += 0xBB67AE85u;
  }
  return ((u64)c1 << 32) | c0;
}

// ---- wave / block primitives on 64-bit integers -----------------------------
// Scans run on DPP adds, which cost an instruction where an exchange through LDS costs a round trip: a 64-bit
// value as limbs of 24 bits, whose sums over 64 lanes fit 32.
__device__ __forceinline__ u64 shfl_u64(u64 v, int src) {
  uint32_t lo = __shfl((uint32_t)v, src), hi = __shfl((uint32_t)(v >> 32), src);
  return ((u64)hi << 32) | lo;
}
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t add_from(uint32_t x) {   // lanes without a source add 0
  return x + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xF, false);
}
__device__ __forceinline__ uint32_t wave_incl_scan_u32(uint32_t x) {
  x = add_from<0x111, 0xF>(x);           // row_shr:1, 2, 4, 8: inside each 16 lanes
  x = add_from<0x112, 0xF>(x);
  x = add_from<0x114, 0xF>(x);
  x = add_from<0x118, 0xF>(x);
  x = add_from<0x142, 0xA>(x);           // row_bcast:15 into rows 1 and 3
  return add_from<0x143, 0xC>(x);        // row_bcast:31 into rows 2 and 3
}
__device__ __forceinline__ uint32_t last_lane(uint32_t x) { return (uint32_t)__builtin_amdgcn_readlane((int)x, 63); }
constexpr uint32_t LIMB = (1u << 24) - 1;
__device__ __forceinline__ u64 wave_incl_scan_u64(u64 v) {
  const uint32_t a = wave_incl_scan_u32((uint32_t)v & LIMB), b = wave_incl_scan_u32((uint32_t)(v >> 24) & LIMB),
                 c = wave_incl_scan_u32((uint32_t)(v >> 48));
  return (u64)a + ((u64)b << 24) + ((u64)c << 48);
}
__device__ __forceinline__ u64 wave_sum_u64(u64 v) {         // v < 2^50 in every lane
  return (u64)last_lane(wave_incl_scan_u32((uint32_t)v & LIMB)) +
         ((u64)last_lane(wave_incl_scan_u32((uint32_t)(v >> 24))) << 24);
}
// Inclusive scan over the 1024 threads of the block; `total` = sum of all.
__device__ __forceinline__ u64 block_incl_scan_u64(u64 v, u64* wave_tot, u64& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  v = wave_incl_scan_u64(v);
  __syncthreads();                       // wave_tot may still be read from a previous use
  if (lane == 63) wave_tot[wave] = v;
  __syncthreads();
  u64 before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < NWAVES; ++w) {
    const u64 t = wave_tot[w];
    if (w < wave) before += t;
    all += t;
  }
  total = all;
  return v + before;
}

struct Row {
  const float* lp;
  int V;
  bool vec;            // rows are 16-byte aligned and V % 4 == 0
  float inv_t;
};
// z of ids id0 .. id0+3 (-inf beyond the vocabulary)
__device__ __forceinline__ void load_z4(const Row& r, int id0, float (&z)[4]) {
  if (r.vec) {
    if (id0 < r.V) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(r.lp + id0);
#pragma unroll
      for (int k = 0; k < 4; ++k) z[k] = v[k] * r.inv_t;
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) z[k] = -INFINITY;
    }
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k) z[k] = id0 + k < r.V ? r.lp[id0 + k] * r.inv_t : -INFINITY;
  }
}

// f(segment, z of this lane's four ids) for segments first, first + step, .. below nseg, U at a time and the loads of the next
// U ahead of them.  Buffer loads, which need no mask at the row's end, so that they go out in a run.  U = 1: `head` is the first.
template <bool VEC>
__device__ __forceinline__ f32x4 load_segment(const Row& r, int s, int lane) {
  const auto buf = buffer_rsrc(r.lp, (uint32_t)r.V * 4u);
  const int off = s * (SEG * 4) + lane * 16;
  if (VEC) return buf4f(buf, off);
  f32x4 v;
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] = __builtin_bit_cast(float, buf1(buf, off + 4 * k));
  return v;
}
// The first segment of a walk, for a caller that has something to wait for before it.
__device__ __forceinline__ f32x4 first_segment(const Row& r, int first, int lane) {
  first = __builtin_amdgcn_readfirstlane(first);
  return r.vec ? load_segment<true>(r, first, lane) : load_segment<false>(r, first, lane);
}
template <int U, bool VEC, class F>
__device__ __forceinline__ void walk_row(const Row& r, int first, int step, int nseg, int lane, f32x4 head, F f) {
  auto load = [&](int s) { return load_segment<VEC>(r, s, lane); };
  f32x4 cur[U], next[U];
  if constexpr (U == 1) cur[0] = head;
  else {
#pragma unroll
    for (int u = 0; u < U; ++u) cur[u] = load(first + u * step);
  }
  for (int s = first; s < nseg; s += U * step) {
#pragma unroll
    for (int u = 0; u < U; ++u) next[u] = load(s + (U + u) * step);     // past the end: zeros, not used
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int su = s + u * step;
      if (u > 0 && su >= nseg) break;
      float z[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) z[k] = cur[u][k] * r.inv_t;
      if ((su + 1) * SEG > r.V) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (su * SEG + lane * 4 + k >= r.V) z[k] = -INFINITY;
      }
      f(su, z);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) cur[u] = next[u];
  }
}
template <int U, class F>
__device__ __forceinline__ void walk_row(const Row& r, int first, int step, int nseg, int lane, f32x4 head, F f) {
  first = __builtin_amdgcn_readfirstlane(first);
  if (r.vec) walk_row<U, true>(r, first, step, nseg, lane, head, f);
  else walk_row<U, false>(r, first, step, nseg, lane, head, f);
}
__device__ __forceinline__ float max4(const float (&z)[4], float mx) {
  return fmaxf(fmaxf(mx, fmaxf(z[0], z[1])), fmaxf(z[2], z[3]));
}
// Masses of four scaled exponentials in 32 bits: the hardware's conversion truncates and stops at 2^32 - 1, which no
// float below 2^32 gives, so that this value stands for 2^32.  Returns whether any lane of the wave has one.
__device__ __forceinline__ bool masses4(const float (&w)[4], uint32_t (&c)[4]) {
#pragma unroll
  for (int k = 0; k < 4; ++k) asm("v_cvt_u32_f32 %0, %1" : "=v"(c[k]) : "v"(w[k]));
  // as integers, which order floats from 0 on as they are
  const int hi = max(max(__float_as_int(w[0]), __float_as_int(w[1])), max(__float_as_int(w[2]), __float_as_int(w[3])));
  return __any(hi >= 0x4F800000);
}
// Sum of the masses of a segment, in every lane.
__device__ __forceinline__ u64 segment_mass(const float (&z)[4], float m) {
  float w[4];
  uint32_t c[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) w[k] = scaled_sexp(z[k] - m);
  const bool whole = masses4(w, c);
  u64 sum = ((u64)c[0] + c[1]) + ((u64)c[2] + c[3]);
  if (whole) {
#pragma unroll
    for (int k = 0; k < 4; ++k) sum += c[k] == 0xFFFFFFFFu;
  }
  return wave_sum_u64(sum);
}

// Highest bin b with  sum_{b' >= b} hist[b'] >= need ; returns b and the mass
// strictly above it.  Executed by wave 0 (all 64 lanes), result in every lane.
__device__ __forceinline__ int find_bin(const u64* hist, u64 need, int lane, u64& above_out) {
  constexpr int PER = 5;                 // 64 * 5 >= 257
  u64 chunk = 0;
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int b = lane * PER + k;
    if (b < NBINS) chunk += hist[b];
  }
  // suffix[lane] = sum of chunks of lanes >= lane
  const u64 incl = wave_incl_scan_u64(chunk), suf = shfl_u64(incl, 63) - incl + chunk;
  const u64 ok = __ballot(suf >= need);
  const int L = 63 - __builtin_clzll(ok);        // ok != 0: total mass >= need
  int bsel = 0;
  u64 above = 0;
  if (lane == L) {
    above = suf - chunk;
    for (int k = PER - 1; k >= 0; --k) {
      const int b = lane * PER + k;
      if (b >= NBINS) continue;
      const u64 h = hist[b];
      if (above + h >= need) { bsel = b; break; }
      above += h;
    }
  }
  bsel = __shfl(bsel, L);
  above_out = shfl_u64(above, L);
  return bsel;
}

// The last step of both variants.  segmass[s] = kept mass of segment s (LDS), segtie[s] = ties
// at the threshold before segment s (top-p < 1 only); draws (or takes the forced token), walks
// the chosen segment in id order and writes the outputs of `row`.  A row without mass (its maximum is
// not finite: every mass is 0) has nothing to draw from: token 0, or the forced one, with a behaviour
// log-prob of -inf.
__device__ __forceinline__ void choose_token(const Row& R, int row, int nseg, float m, u64 S_total, u64 S_nuc,
                                             bool all_in, u64 tau, u64 n_take, const u64* segmass,
                                             const uint32_t* segtie, u64* wave_tot, u64* sh_u64, int* sh_int,
                                             u64 seed, const int32_t* __restrict__ seq_ids,
                                             const int32_t* __restrict__ positions,
                                             const int32_t* __restrict__ forced,
                                             int32_t* __restrict__ tokens_out, float* __restrict__ logp_behav,
                                             float* __restrict__ logp_full) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, V = R.V;
  int tok;
  u64 base = 0;          // kept mass before the chosen segment (draw path)
  u64 r = 0;
  if (forced) {
    tok = forced[row];
    tok = tok < 0 ? 0 : (tok >= V ? V - 1 : tok);
    if (tid == 0) sh_int[2] = tok / SEG;
  } else {
    const u64 Rbits = philox_draw(seed, (uint32_t)seq_ids[row], (uint32_t)positions[row]);
    r = __umul64hi(Rbits, S_nuc);
    if (tid == 0) { sh_int[2] = 0; sh_u64[1] = 0; }      // the scan's barriers order this before the one write below
    u64 tot;
    const u64 mine = tid < nseg ? segmass[tid] : 0;
    const u64 incl = block_incl_scan_u64(mine, wave_tot, tot);
    if (tid < nseg && incl > r && incl - mine <= r) { sh_int[2] = tid; sh_u64[1] = incl - mine; }
    tok = -1;
  }
  __syncthreads();
  const int sseg = sh_int[2];
  base = sh_u64[1];

  // wave 0 walks the chosen segment in id order
  if (wave == 0) {
    float z[4];
    load_z4(R, sseg * SEG + lane * 4, z);
    double log_nuc = log((double)S_nuc), log_total = log((double)S_total);
    asm volatile("" : "+v"(log_nuc), "+v"(log_total));   // while the segment is on its way
    u64 c[4], kept[4];
    uint32_t tie_lane = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      c[k] = mass_of(z[k], m);
      if (!all_in && sseg * SEG + lane * 4 + k < V && c[k] == tau) tie_lane += 1;
    }
    // ties before this lane's first id
    uint32_t tie_before = 0;
    if (!all_in) {
      tie_before = segtie[sseg] + wave_incl_scan_u32(tie_lane) - tie_lane;
    }
    u64 lane_sum = 0;
    bool member[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const bool in = sseg * SEG + lane * 4 + k < V;
      if (all_in) {
        member[k] = in;
      } else if (c[k] > tau) {
        member[k] = in;
      } else if (c[k] == tau && in) {
        member[k] = tie_before < n_take;
        tie_before += 1;
      } else {
        member[k] = false;
      }
      kept[k] = member[k] ? c[k] : 0;
      lane_sum += kept[k];
    }
    int k_sel = -1;
    if (forced) {
      if ((tok % SEG) / 4 == lane) k_sel = tok & 3;
    } else {
      const u64 incl = wave_incl_scan_u64(lane_sum);
      u64 run = base + incl - lane_sum;
      if (run <= r && r < run + lane_sum) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if (k_sel < 0) {
            run += kept[k];
            if (run > r) k_sel = k;
          }
        }
      }
      if (S_nuc == 0 && lane == 0) k_sel = 0;
    }
    if (k_sel >= 0) {
      const int t = sseg * SEG + lane * 4 + k_sel;
      u64 ct = 0;
      float zt = 0.f;
      bool mem = false;
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (k == k_sel) { ct = c[k]; zt = z[k]; mem = member[k]; }
      tokens_out[row] = t;
      logp_behav[row] = (mem && ct > 0) ? (float)(log((double)ct) - log_nuc) : -INFINITY;
      if (logp_full)
        logp_full[row] = (float)((double)(zt - m) - (log_total - 32.0 * 0.69314718055994530942));
    }
  }
}

// Shared memory of the nucleus selection.
struct NucleusLds {
  u64 segmass[MAX_SEG];            // kept mass per segment
  uint32_t segtie[MAX_SEG];        // ties at the threshold per segment, then their exclusive prefix
  u64 hist_mass[NBINS];
  uint32_t hist_cnt[NBINS];
  u64 wave_tot[NWAVES];
  u64 sh_u64[4];                   // broadcast slots
  int sh_int[4];
};

__device__ __forceinline__ u64 nucleus_target(float top_p, u64 S_total) {
  u64 target = (u64)ceil((double)top_p * (double)S_total);
  if (target < 1) target = 1;
  return target > S_total ? S_total : target;
}

// Mass above tau and number of ids at tau, per segment of a row.
__device__ __forceinline__ void segments_above(const Row& R, int nseg, float m, u64 tau, NucleusLds& L) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int s = wave; s < nseg; s += NWAVES) {
    float z[4];
    load_z4(R, s * SEG + lane * 4, z);
    u64 gt = 0;
    uint32_t tie = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const u64 c = mass_of(z[k], m);
      const bool in = s * SEG + lane * 4 + k < R.V;
      if (in && c > tau) gt += c;
      if (in && c == tau) tie += 1;
    }
    gt = wave_sum_u64(gt);
    tie = last_lane(wave_incl_scan_u32(tie));
    if (lane == 0) { L.segmass[s] = gt; L.segtie[s] = tie; }
  }
  __syncthreads();
}

// One work-group selects the nucleus of a whole row: threshold tau, number of ids at tau that
// are taken (in id order), mass S_nuc, and the kept mass / ties before each segment in `L`.
__device__ __forceinline__ void nucleus_of_row(const Row& R, int nseg, float m, float top_p, u64 S_total,
                                               NucleusLds& L, u64& tau, u64& n_take, u64& S_nuc) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, V = R.V;
  const u64 target = nucleus_target(top_p, S_total);
  u64 mass_above = 0, prefix = 0;
  uint32_t cnt_tau = 0;
  // radix select on the 33-bit masses
  for (int level = 0; level < 4; ++level) {
    const int shift = 24 - 8 * level;
    for (int b = tid; b < NBINS; b += TPB) { L.hist_mass[b] = 0; L.hist_cnt[b] = 0; }
    __syncthreads();
    for (int s = wave; s < nseg; s += NWAVES) {
      float z[4];
      load_z4(R, s * SEG + lane * 4, z);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const u64 c = mass_of(z[k], m);
        const bool in = (s * SEG + lane * 4 + k < V) && (level == 0 || (c >> (shift + 8)) == prefix);
        const int bin = level == 0 ? (int)(c >> 24) : (int)((c >> shift) & 255);
        // near-flat logits put most ids into one bin: add once per wave then
        const int bin0 = __builtin_amdgcn_readfirstlane(bin);
        if (__all(in && bin == bin0)) {
          const u64 tot = wave_sum_u64(c);
          if (lane == 0) {
            atomicAdd(&L.hist_mass[bin0], tot);
            atomicAdd(&L.hist_cnt[bin0], 64u);
          }
        } else if (in) {
          atomicAdd(&L.hist_mass[bin], c);
          atomicAdd(&L.hist_cnt[bin], 1u);
        }
      }
    }
    __syncthreads();
    if (wave == 0) {
      u64 above;
      const int b = find_bin(L.hist_mass, target - mass_above, lane, above);
      if (lane == 0) {
        L.sh_int[0] = b;
        L.sh_u64[0] = mass_above + above;
        L.sh_int[1] = (int)L.hist_cnt[b];
      }
    }
    __syncthreads();
    const int bsel = L.sh_int[0];
    mass_above = L.sh_u64[0];
    cnt_tau = (uint32_t)L.sh_int[1];
    __syncthreads();
    if (level == 0) {
      prefix = (u64)bsel;
      if (bsel == 256) { prefix = 1ull << 32; break; }   // only c = 2^32 lives in this bin
    } else {
      prefix = (prefix << 8) | (u64)bsel;
    }
  }
  tau = prefix;
  n_take = (target - mass_above + tau - 1) / tau;
  if (n_take > cnt_tau) n_take = cnt_tau;                 // cannot happen; keeps indices sane
  S_nuc = mass_above + n_take * tau;

  segments_above(R, nseg, m, tau, L);
}

// Fold the ties that are taken into the segments' kept mass; segtie becomes its exclusive prefix.
__device__ __forceinline__ void fold_ties(NucleusLds& L, int nseg, u64 tau, u64 n_take) {
  const int tid = threadIdx.x;
  u64 tot;
  const u64 mine = tid < nseg ? L.segtie[tid] : 0;
  const u64 incl = block_incl_scan_u64(mine, L.wave_tot, tot);
  const u64 excl = incl - mine;
  __syncthreads();
  if (tid < nseg) {
    const u64 takes = excl >= n_take ? 0 : (n_take - excl < mine ? n_take - excl : mine);
    L.segmass[tid] += takes * tau;
    L.segtie[tid] = (uint32_t)excl;                       // now: ties before this segment
  }
  __syncthreads();
}

__global__ __launch_bounds__(TPB) void sampler_kernel(
    int V, const float* __restrict__ logits, const int32_t* __restrict__ seq_ids,
    const int32_t* __restrict__ positions, float inv_t, float top_p, u64 seed,
    const int32_t* __restrict__ forced, int32_t* __restrict__ tokens_out,
    float* __restrict__ logp_behav, float* __restrict__ logp_full) {
  __shared__ NucleusLds L;
  __shared__ float wave_max_s[NWAVES];

  const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  Row R;
  R.lp = logits + (int64_t)row * V;
  R.V = V;
  R.vec = (V % 4 == 0) && (((uintptr_t)logits & 15) == 0);
  R.inv_t = inv_t;
  const int nseg = (V + SEG - 1) / SEG;
  const bool all_in = top_p >= 1.0f;

  // ---- pass A: m = max z ----------------------------------------------------
  float mx = -INFINITY;
  walk_row<4>(R, wave, NWAVES, nseg, lane, f32x4{}, [&](int, const float (&z)[4]) { mx = max4(z, mx); });
  f32x4 head = first_segment(R, wave, lane);
  mx = wave_max(mx);
  if (lane == 0) wave_max_s[wave] = mx;
  __syncthreads();
  float m = wave_max_s[0];
#pragma unroll
  for (int w = 1; w < NWAVES; ++w) m = fmaxf(m, wave_max_s[w]);

  // ---- pass B: per-segment mass, S = total mass --------------------------------
  walk_row<1>(R, wave, NWAVES, nseg, lane, head, [&](int s, const float (&z)[4]) {
    const u64 c = segment_mass(z, m);
    if (lane == 0) L.segmass[s] = c;
  });
  __syncthreads();
  u64 S_total;
  block_incl_scan_u64(tid < nseg ? L.segmass[tid] : 0, L.wave_tot, S_total);

  // ---- nucleus (top_p < 1) -----------------------------------------------------
  u64 tau = 0, n_take = 0, S_nuc = S_total;
  if (!all_in && S_total > 0) {
    nucleus_of_row(R, nseg, m, top_p, S_total, L, tau, n_take, S_nuc);
    fold_ties(L, nseg, tau, n_take);
  } else if (!all_in) {
    L.segtie[tid] = 0;                 // no mass, no nucleus (choose_token's barriers publish this)
  }

  choose_token(R, row, nseg, m, S_total, S_nuc, all_in, tau, n_take, L.segmass, L.segtie, L.wave_tot, L.sh_u64,
               L.sh_int, seed, seq_ids, positions, forced, tokens_out, logp_behav, logp_full);
}

// ---- a row spread over several work-groups -----------------------------------------
// Work-group (part, row) of 4 waves takes segments part*4 + wave, then every parts*4-th.
constexpr int SPLIT_TPB = 256, SPLIT_WAVES = 4;

// Bins of a mass for the nucleus: exact below 64, then 64 per octave (28 octaves up to 2^32), so that a
// bin holds masses within 1.6 % of each other wherever the threshold falls: at the flattest row of a
// full vocabulary (logits N(0, 0.8), T = 1) the fullest bin holds about 1,200 ids.
constexpr int LOG_BINS = 28 * 64;
constexpr int LIST_CAP = 4096;                 // ids of one bin that the scratch buffer holds per row
struct SplitScratch {                          // one row's share of the scratch buffer
  u64 segmass[MAX_SEG];                        // mass per segment (top-p < 1: of the bins above the threshold's)
  u64 hist[LOG_BINS];                          // mass per bin
  union {                                      // of the threshold's bin:
    uint32_t list[LIST_CAP][2];                // {id, low 32 bits of its mass}
    uint32_t segtie[MAX_SEG];                  // or, where the bin is one value, its ids per segment
  };
  float pmax[SAMPLER_MAX_PARTS];
  uint32_t n_list, pad[15];                    // ids in that bin (may exceed LIST_CAP)
};
static_assert(sizeof(SplitScratch) == SAMPLER_SCRATCH_ROW && sizeof(SplitScratch) % 16 == 0, "scratch layout");

// Bin of the mass of a scaled exponential w >= 0: c itself below 64, else octave and next six bits of c = trunc(w), which
// are exponent and leading fraction bits of w, for truncation leaves the leading seven bits of a number of 64 and more.
// The bits' bin is below c for w < 64 and equal to it or below from there on, so that the middle one of c, that bin and 64 is
// the one meant (c saturates at 2^31 - 1).
__device__ __forceinline__ int log_bin(float w) {
  const int top = (min(__float_as_int(w), 0x4F800000) >> 17) - ((127 + 5) << 6);
  int c, bin;
  asm("v_cvt_i32_f32 %0, %1" : "=v"(c) : "v"(w));
  asm("v_med3_i32 %0, %1, %2, 64" : "=v"(bin) : "v"(c), "v"(top));
  return bin;
}
__device__ __forceinline__ u64 log_bin_low(int b) {    // smallest mass of a bin
  return b < 64 ? (u64)b : (u64)(64 + (b & 63)) << ((b >> 6) - 1);
}

__device__ __forceinline__ int log_bin_width(int b) {  // bits of a mass's offset in its bin (the last bin holds 2^32 only)
  return b < 64 || b == LOG_BINS - 64 ? 0 : (b >> 6) - 1;
}

__device__ __forceinline__ Row make_row(const float* logits, int row, int V, float inv_t) {
  Row R;
  R.lp = logits + (int64_t)row * V;
  R.V = V;
  R.vec = (V % 4 == 0) && (((uintptr_t)logits & 15) == 0);
  R.inv_t = inv_t;
  return R;
}

__global__ __launch_bounds__(SPLIT_TPB) void sampler_split_max_kernel(int V, const float* __restrict__ logits,
                                                                      float inv_t, int parts, int clear_hist,
                                                                      SplitScratch* __restrict__ scratch) {
  __shared__ float wmax[SPLIT_WAVES];
  const int row = blockIdx.y, part = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const Row R = make_row(logits, row, V, inv_t);
  SplitScratch& sc = scratch[row];
  const int nseg = (V + SEG - 1) / SEG;
  if (clear_hist) {
    for (int b = part * SPLIT_TPB + threadIdx.x; b < LOG_BINS; b += parts * SPLIT_TPB) sc.hist[b] = 0;
    if (part == 0 && threadIdx.x == 0) sc.n_list = 0;
  }
  float mx = -INFINITY;
  walk_row<4>(R, part * SPLIT_WAVES + wave, parts * SPLIT_WAVES, nseg, lane, f32x4{}, [&](int, const float (&z)[4]) { mx = max4(z, mx); });
  mx = wave_max(mx);
  if (lane == 0) wmax[wave] = mx;
  __syncthreads();
  if (threadIdx.x == 0) sc.pmax[part] = fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]));
}

__device__ __forceinline__ float row_max_of_parts(const SplitScratch& sc, int parts) {
  const int lane = threadIdx.x & 63;                     // parts <= SAMPLER_MAX_PARTS = 64
  return wave_max(lane < parts ? sc.pmax[lane] : -INFINITY);
}

__global__ __launch_bounds__(SPLIT_TPB) void sampler_split_mass_kernel(int V, const float* __restrict__ logits,
                                                                       float inv_t, int parts,
                                                                       SplitScratch* __restrict__ scratch) {
  const int row = blockIdx.y, part = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const Row R = make_row(logits, row, V, inv_t);
  SplitScratch& sc = scratch[row];
  const int nseg = (V + SEG - 1) / SEG;
  const f32x4 head = first_segment(R, part * SPLIT_WAVES + wave, lane);
  const float m = row_max_of_parts(sc, parts);
  walk_row<1>(R, part * SPLIT_WAVES + wave, parts * SPLIT_WAVES, nseg, lane, head, [&](int sg, const float (&z)[4]) {
    const u64 c = segment_mass(z, m);
    if (lane == 0) sc.segmass[sg] = c;
  });
}

__global__ __launch_bounds__(TPB) void sampler_split_pick_kernel(
    int V, const float* __restrict__ logits, const int32_t* __restrict__ seq_ids,
    const int32_t* __restrict__ positions, float inv_t, u64 seed, const int32_t* __restrict__ forced, int parts,
    const SplitScratch* __restrict__ scratch, int32_t* __restrict__ tokens_out, float* __restrict__ logp_behav,
    float* __restrict__ logp_full) {
  __shared__ u64 segmass[MAX_SEG];
  __shared__ u64 wave_tot[NWAVES];
  __shared__ u64 sh_u64[4];
  __shared__ int sh_int[4];
  const int row = blockIdx.x, tid = threadIdx.x;
  const Row R = make_row(logits, row, V, inv_t);
  const SplitScratch& sc = scratch[row];
  const int nseg = (V + SEG - 1) / SEG;
  const float m = row_max_of_parts(sc, parts);
  const u64 mine = tid < nseg ? sc.segmass[tid] : 0;
  segmass[tid] = mine;
  u64 S_total;
  block_incl_scan_u64(mine, wave_tot, S_total);        // its barriers also publish segmass
  choose_token(R, row, nseg, m, S_total, S_total, true, 0, 0, segmass, nullptr, wave_tot, sh_u64, sh_int, seed,
               seq_ids, positions, forced, tokens_out, logp_behav, logp_full);
}

// ---- nucleus of a row spread over several work-groups ------------------------------
// One work-group per row walks the vocabulary seven times and evaluates the specified exponential in
// six of them, ~70 us each on one compute unit.  Spread: (1) partial maxima; (2) masses into a histogram
// of logarithmic bins, which locates the bin the threshold falls into to 1.6 % of its value; (3) the
// kept mass of the bins above, per segment, and the list of that one bin's ids; (4) per row, the exact
// threshold by radix select over the list, ties in id order, the draw.  The exponential is evaluated
// twice per id, on all compute units: 64 rows of 151,936 logits 566 -> 49 us, 1 row 530 -> 24, 128 rows
// 576 -> 69 (bound by the exponential's arithmetic and four launches).  On the way: 61 and 91 us (64, 128 rows) with exchanges
// through LDS for the wave sums and 64-bit shifts for the bins; 56 and 82 with 55 instructions an id, 64-bit masses among
// them; 50.3 and 71.0 with 37; 48.7 and 68.7 with a row's first segment and the list read ahead of what says which of
// them count, rounds of a bin a thread in the list, and the logarithms while the chosen segment is on its way.  More segments
// ahead: no change; ids above the bin packed before their exponentials: 48.2, but 49.7 for 48.9 where half of all are.  A bin of one value (every mass
// below 128, and 2^32: the maximum itself) needs no list but its ids per segment; for a bin with more
// ids than the list holds see nucleus_in_bin.
__global__ __launch_bounds__(SPLIT_TPB) void sampler_split_hist_kernel(int V, const float* __restrict__ logits,
                                                                       float inv_t, int parts,
                                                                       SplitScratch* __restrict__ scratch) {
  __shared__ u64 hist[LOG_BINS];
  const int row = blockIdx.y, part = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const Row R = make_row(logits, row, V, inv_t);
  SplitScratch& sc = scratch[row];
  const int nseg = (V + SEG - 1) / SEG;
  const f32x4 head = first_segment(R, part * SPLIT_WAVES + wave, lane);
  const float m = row_max_of_parts(sc, parts);
  for (int b = threadIdx.x; b < LOG_BINS; b += SPLIT_TPB) hist[b] = 0;
  __syncthreads();
  walk_row<1>(R, part * SPLIT_WAVES + wave, parts * SPLIT_WAVES, nseg, lane, head, [&](int, const float (&z)[4]) {
    float w[4];
    uint32_t c[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = scaled_sexp(z[k] - m);
    const bool whole = masses4(w, c);                  // masses are 0 beyond the vocabulary
    const int bin0 = log_bin(w[0]);
    if (whole || __all(bin0 == __builtin_amdgcn_readfirstlane(bin0))) {   // 2^32 among them, or heavily tied logits
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const u64 ck = mass_of_scaled(w[k]);
        const int b = log_bin(w[k]), b0 = __builtin_amdgcn_readfirstlane(b);
        if (__all(b == b0)) {                          // once per wave
          const u64 tot = wave_sum_u64(ck);
          if (lane == 0) atomicAdd(&hist[b0], tot);
        } else if (ck > 0) {
          atomicAdd(&hist[b], ck);
        }
      }
      return;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (c[k] > 0) atomicAdd(&hist[log_bin(w[k])], (u64)c[k]);
  });
  __syncthreads();
  for (int b = threadIdx.x; b < LOG_BINS; b += SPLIT_TPB)
    if (hist[b]) atomicAdd(&sc.hist[b], hist[b]);
}

// The bin in which the mass summed from the top reaches need(total mass), and the mass of the bins
// above it (bin 0 if there is no mass).  All NW * 64 threads of the work-group take part; results in
// every thread.
template <int NW, int BINS, class Need>
__device__ __forceinline__ int bin_from_top(const u64* hist, Need need_of, u64* wtot, u64* res_u64, int* res_int,
                                            u64& above) {
  constexpr int NT = NW * 64, PER = (BINS + NT - 1) / NT;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  u64 h[PER], mine = 0;
#pragma unroll
  for (int k = 0; k < PER; ++k) {                      // thread 0 holds the highest bins
    const int b = BINS - 1 - (tid * PER + k);
    h[k] = b >= 0 ? hist[b] : 0;
    mine += h[k];
  }
  const u64 incl_w = wave_incl_scan_u64(mine);
  if (lane == 63) wtot[wave] = incl_w;
  if (tid == 0) { *res_int = 0; *res_u64 = 0; }
  __syncthreads();
  u64 before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const u64 t = wtot[w];
    if (w < wave) before += t;
    all += t;
  }
  const u64 need = need_of(all), incl = before + incl_w;
  if (incl >= need && incl - mine < need) {            // exactly one thread (none if there is no mass)
    u64 a = incl - mine;
    int sel = 0;
    bool found = false;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      if (!found) {
        if (a + h[k] >= need) { sel = BINS - 1 - (tid * PER + k); found = true; }
        else a += h[k];
      }
    }
    *res_int = sel;
    *res_u64 = a;
  }
  __syncthreads();
  above = *res_u64;
  return *res_int;
}
// Total mass of a row, the nucleus's target, and the logarithmic bin its threshold falls into.
template <int NW>
__device__ __forceinline__ int threshold_bin(const SplitScratch& sc, float top_p, u64* wtot, u64* res_u64, int* res_int,
                                             u64& S_total, u64& target, u64& above) {
  return bin_from_top<NW, LOG_BINS>(sc.hist, [&](u64 all) {
    S_total = all;
    return target = nucleus_target(top_p, all);
  }, wtot, res_u64, res_int, above);
}

// The exact threshold in a bin with more ids than the list holds (flat rows: a spread of z below 0.23 over
// 152k ids or 0.4 over 262k, which a high temperature gives; or ties): one work-group walks the row again,
// 13 bits of the offset at a time, two passes at the widest bin, and once more for the segments.  Selecting
// over the whole row instead (four passes of 8 bits) took 331 / 546 us for 128 rows of 152k / 262k ids with a
// spread of 0.02, 322 / 539 without the spread launches; this way 232 / 374.
constexpr int OFFSET_BITS = 13, OFFSET_BINS = 1 << OFFSET_BITS;
__device__ __forceinline__ void nucleus_in_bin(const Row& R, int nseg, float m, int tb, u64 target, u64 mass_above,
                                               u64* hist, NucleusLds& L, u64& tau, u64& n_take, u64& S_nuc) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const u64 low = log_bin_low(tb);
  u64 prefix = 0;
  for (int top = log_bin_width(tb); top > 0;) {
    const int shift = max(0, top - OFFSET_BITS), bits = top - shift;
    for (int b = tid; b < OFFSET_BINS; b += TPB) hist[b] = 0;
    __syncthreads();
    for (int s = wave; s < nseg; s += NWAVES) {
      float z[4];
      load_z4(R, s * SEG + lane * 4, z);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const u64 c = mass_of(z[k], m), d = c - low;   // below the bin d wraps: its high bits are set
        const bool in = (d >> top) == prefix;          // (masses beyond the vocabulary are 0: below it)
        const int bin = (int)(d >> shift) & ((1 << bits) - 1);
        const int bin0 = __builtin_amdgcn_readfirstlane(bin);
        if (__all(in && bin == bin0)) {
          const u64 tot = wave_sum_u64(c);
          if (lane == 0) atomicAdd(&hist[bin0], tot);
        } else if (in) {
          atomicAdd(&hist[bin], c);
        }
      }
    }
    __syncthreads();
    u64 above;
    const int b = bin_from_top<NWAVES, OFFSET_BINS>(hist, [&](u64) { return target - mass_above; }, L.wave_tot,
                                                    &L.sh_u64[2], &L.sh_int[3], above);
    mass_above += above;
    prefix = (prefix << bits) | (u64)b;
    top = shift;
    __syncthreads();                                   // the histogram and the broadcast slots are free again
  }
  tau = low + prefix;
  n_take = (target - mass_above + tau - 1) / tau;
  S_nuc = mass_above + n_take * tau;
  segments_above(R, nseg, m, tau, L);
}

__global__ __launch_bounds__(SPLIT_TPB) void sampler_split_collect_kernel(int V, const float* __restrict__ logits,
                                                                          float inv_t, float top_p, int parts,
                                                                          SplitScratch* __restrict__ scratch) {
  __shared__ u64 wtot[SPLIT_WAVES], res_u64;
  __shared__ int res_int;
  __shared__ uint32_t list[LIST_CAP][2];
  __shared__ uint32_t n_list, base;
  const int row = blockIdx.y, part = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const Row R = make_row(logits, row, V, inv_t);
  SplitScratch& sc = scratch[row];
  const int nseg = (V + SEG - 1) / SEG;
  const int first = part * SPLIT_WAVES + wave, step = parts * SPLIT_WAVES;
  const f32x4 head = first_segment(R, first, lane);
  const float m = row_max_of_parts(sc, parts);
  if (threadIdx.x == 0) n_list = 0;
  u64 S_total, target, above;
  const int tb = threshold_bin<SPLIT_WAVES>(sc, top_p, wtot, &res_u64, &res_int, S_total, target, above);
  // Ids below the threshold's bin add nothing, and for a wave whose ids all are the exponential need not be
  // evaluated: below x_skip their masses are less than the bin's lowest by a thousandth at least, far beyond
  // the specified exponential's error.
  const float x_skip = (float)(log((double)log_bin_low(tb)) - 32.0 * 0.69314718055994530942) - 1e-3f;   // -inf for bin 0
  auto append = [&](int id, uint32_t mass) {
    const uint32_t at = atomicAdd(&n_list, 1u);
    if (at < LIST_CAP) { list[at][0] = id; list[at][1] = mass; }
  };
  if (log_bin_width(tb) == 0) {
    walk_row<1>(R, first, step, nseg, lane, head, [&](int sg, const float (&z)[4]) {
      u64 gt = 0;
      int ties = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (!__any(!(z[k] - m < x_skip))) continue;
        const float w = scaled_sexp(z[k] - m);
        const int bin = log_bin(w);
        if (bin > tb) gt += mass_of_scaled(w);
        ties += __popcll(__ballot(bin == tb && sg * SEG + lane * 4 + k < V));
      }
      gt = wave_sum_u64(gt);
      if (lane == 0) { sc.segmass[sg] = gt; sc.segtie[sg] = ties; }
    });
  } else {
    // The bin's masses [lo, hi) in 32 bits, lo >= 128: no id beyond the vocabulary, whose mass is 0, is among them.  2^32 - 1
    // stands for 2^32 (masses4) and lies above every such bin.
    const uint32_t lo = (uint32_t)log_bin_low(tb), hi = (uint32_t)min((u64)0xFFFFFFFFu, log_bin_low(tb + 1)), width = hi - lo;
    walk_row<1>(R, first, step, nseg, lane, head, [&](int sg, const float (&z)[4]) {
      u64 gt = 0;
      if (__any(!(max4(z, -INFINITY) - m < x_skip))) {
        float w[4];
        uint32_t c[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) w[k] = scaled_sexp(z[k] - m);
        const bool whole = masses4(w, c);
        bool in = false;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          gt += c[k] >= hi ? c[k] : 0;
          in |= c[k] - lo < width;
        }
        if (whole) {
#pragma unroll
          for (int k = 0; k < 4; ++k) gt += c[k] == 0xFFFFFFFFu;
        }
        if (in) {
#pragma unroll
          for (int k = 0; k < 4; ++k)
            if (c[k] - lo < width) append(sg * SEG + lane * 4 + k, c[k]);
        }
        gt = wave_sum_u64(gt);
      }
      if (lane == 0) sc.segmass[sg] = gt;
    });
  }
  __syncthreads();
  const uint32_t n = n_list;
  if (threadIdx.x == 0 && n) base = atomicAdd(&sc.n_list, n);
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < n && i < LIST_CAP; i += SPLIT_TPB) {
    const uint32_t at = base + i;
    if (at < LIST_CAP) { sc.list[at][0] = list[i][0]; sc.list[at][1] = list[i][1]; }
  }
}

__global__ __launch_bounds__(TPB) void sampler_split_nucleus_pick_kernel(
    int V, const float* __restrict__ logits, const int32_t* __restrict__ seq_ids,
    const int32_t* __restrict__ positions, float inv_t, float top_p, u64 seed, const int32_t* __restrict__ forced,
    int parts, const SplitScratch* __restrict__ scratch, int32_t* __restrict__ tokens_out,
    float* __restrict__ logp_behav, float* __restrict__ logp_full) {
  __shared__ NucleusLds L;
  __shared__ u64 offset_hist[OFFSET_BINS];
  constexpr int PER = LIST_CAP / TPB;
  const int row = blockIdx.x, tid = threadIdx.x;
  const Row R = make_row(logits, row, V, inv_t);
  const SplitScratch& sc = scratch[row];
  const int nseg = (V + SEG - 1) / SEG;
  const float m = row_max_of_parts(sc, parts);
  const uint32_t n = sc.n_list;
  // this thread's ids of the threshold's bin and their masses (then mass offsets), and its segment's mass: read ahead of the bin
  // that says whether they are in use, and of n (whatever lies behind the list is not used)
  uint32_t id[PER], d[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) { id[k] = sc.list[tid + k * TPB][0]; d[k] = sc.list[tid + k * TPB][1]; }
  const u64 seg_above = sc.segmass[tid];
  u64 S_total, target, mass_above;
  const int tb = threshold_bin<NWAVES>(sc, top_p, L.wave_tot, &L.sh_u64[2], &L.sh_int[3], S_total, target, mass_above);
  u64 tau = 0, n_take = 0, S_nuc = 0;
  if (S_total == 0) {                                  // uniform over the work-group, as is n
    L.segmass[tid] = 0;
    L.segtie[tid] = 0;
    __syncthreads();
  } else if (log_bin_width(tb) == 0) {                 // the bin's one value is the threshold
    tau = log_bin_low(tb);
    n_take = (target - mass_above + tau - 1) / tau;
    S_nuc = mass_above + n_take * tau;
    if (tid < nseg) { L.segmass[tid] = seg_above; L.segtie[tid] = sc.segtie[tid]; }
    __syncthreads();
  } else if (n > LIST_CAP) {
    nucleus_in_bin(R, nseg, m, tb, target, mass_above, offset_hist, L, tau, n_take, S_nuc);
  } else {
    const u64 low = log_bin_low(tb);
#pragma unroll
    for (int k = 0; k < PER; ++k) d[k] -= (uint32_t)low;         // < 2^26: the width of the widest bin
    if (tid < nseg) { L.segmass[tid] = seg_above; L.segtie[tid] = 0; }
    // radix select on the offsets, in rounds of up to 10 bits from the bin's own width down: a bin a thread, to clear and to
    // scan (3 rounds at the widest bin; 13 bits a round take two, of eight bins a thread)
    uint32_t prefix = 0;
    const int round = (log_bin_width(tb) + (log_bin_width(tb) + 9) / 10 - 1) / ((log_bin_width(tb) + 9) / 10);
    for (int top = log_bin_width(tb); top > 0;) {
      const int shift = max(0, top - round), bits = top - shift;
      offset_hist[tid] = 0;
      __syncthreads();
#pragma unroll
      for (int k = 0; k < PER; ++k)
        if (tid + k * TPB < n && (d[k] >> top) == prefix)
          atomicAdd(&offset_hist[(d[k] >> shift) & ((1u << bits) - 1u)], low + d[k]);
      __syncthreads();
      u64 above;
      const int b = bin_from_top<NWAVES, TPB>(offset_hist, [&](u64) { return target - mass_above; }, L.wave_tot,
                                                      &L.sh_u64[2], &L.sh_int[3], above);
      mass_above += above;
      prefix = (prefix << bits) | (uint32_t)b;
      top = shift;
      __syncthreads();                                 // the histogram and the broadcast slots are free again
    }
    tau = low + prefix;
    n_take = (target - mass_above + tau - 1) / tau;
    S_nuc = mass_above + n_take * tau;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      if (tid + k * TPB < n) {
        if (d[k] > prefix) atomicAdd(&L.segmass[id[k] / SEG], low + d[k]);
        else if (d[k] == prefix) atomicAdd(&L.segtie[id[k] / SEG], 1u);
      }
    }
    __syncthreads();
  }
  fold_ties(L, nseg, tau, n_take);
  choose_token(R, row, nseg, m, S_total, S_nuc, false, tau, n_take, L.segmass, L.segtie, L.wave_tot, L.sh_u64,
               L.sh_int, seed, seq_ids, positions, forced, tokens_out, logp_behav, logp_full);
}

}  // namespace

size_t sampler_scratch_bytes() { return SAMPLER_SPLIT_MAX_ROWS * SAMPLER_SCRATCH_ROW; }

hipError_t launch_sampler(hipStream_t s, int n, int vocab, const float* logits, const int32_t* seq_ids,
                          const int32_t* positions, float inv_temperature, float top_p, uint64_t seed,
                          const int32_t* forced, int32_t* tokens_out, float* logp_behav,
                          float* logp_full, void* scratch) {
  if (n <= 0 || vocab <= 0 || (vocab + SEG - 1) / SEG > MAX_SEG || !logits || !tokens_out ||
      !logp_behav || !(inv_temperature > 0.f) || !(top_p > 0.f))
    return hipErrorInvalidValue;
  if (!forced && (!seq_ids || !positions)) return hipErrorInvalidValue;
  // whole vocabulary kept, few rows: 2 .. 64 work-groups of four waves per row, about four per
  // compute unit (the specified exponential is arithmetic-bound: it wants every SIMD's wave slots)
  const int nseg = (vocab + SEG - 1) / SEG;
  int parts = std::min(SAMPLER_MAX_PARTS, 1024 / n);
  parts = std::min(parts, (nseg + SPLIT_WAVES - 1) / SPLIT_WAVES);
  if (scratch && ((uintptr_t)scratch & 15)) return hipErrorInvalidValue;
  SplitScratch* sc = reinterpret_cast<SplitScratch*>(scratch);
  if (scratch && top_p >= 1.0f && n <= SAMPLER_SPLIT_MAX_ROWS && parts >= 2) {
    const dim3 grid(parts, n);
    sampler_split_max_kernel<<<grid, SPLIT_TPB, 0, s>>>(vocab, logits, inv_temperature, parts, 0, sc);
    sampler_split_mass_kernel<<<grid, SPLIT_TPB, 0, s>>>(vocab, logits, inv_temperature, parts, sc);
    sampler_split_pick_kernel<<<n, TPB, 0, s>>>(vocab, logits, seq_ids, positions, inv_temperature, (u64)seed,
                                                forced, parts, sc, tokens_out, logp_behav, logp_full);
    return hipGetLastError();
  }
  if (scratch && top_p < 1.0f && nseg >= (n > NUCLEUS_FEW_ROWS ? NUCLEUS_SPLIT_MIN_SEG_MANY : NUCLEUS_SPLIT_MIN_SEG)) {
    for (int r0 = 0; r0 < n; r0 += SAMPLER_SPLIT_MAX_ROWS) {     // the scratch buffer's rows at a time
      const int rows = std::min(n - r0, SAMPLER_SPLIT_MAX_ROWS);
      const int pt = std::max(1, std::min(std::min(SAMPLER_MAX_PARTS, 1024 / rows), (nseg + SPLIT_WAVES - 1) / SPLIT_WAVES));
      const float* lg = logits + (int64_t)r0 * vocab;
      const dim3 grid(pt, rows);
      sampler_split_max_kernel<<<grid, SPLIT_TPB, 0, s>>>(vocab, lg, inv_temperature, pt, 1, sc);
      sampler_split_hist_kernel<<<grid, SPLIT_TPB, 0, s>>>(vocab, lg, inv_temperature, pt, sc);
      sampler_split_collect_kernel<<<grid, SPLIT_TPB, 0, s>>>(vocab, lg, inv_temperature, top_p, pt, sc);
      sampler_split_nucleus_pick_kernel<<<rows, TPB, 0, s>>>(
          vocab, lg, seq_ids ? seq_ids + r0 : nullptr, positions ? positions + r0 : nullptr, inv_temperature, top_p,
          (u64)seed, forced ? forced + r0 : nullptr, pt, sc, tokens_out + r0, logp_behav + r0,
          logp_full ? logp_full + r0 : nullptr);
    }
    return hipGetLastError();
  }
  sampler_kernel<<<n, TPB, 0, s>>>(vocab, logits, seq_ids, positions, inv_temperature, top_p,
                                   (u64)seed, forced, tokens_out, logp_behav, logp_full);
  return hipGetLastError();
}

}  // namespace areal

// ---- the entry point that allocates nothing -----------------------------------------
// Same sampler, for callers that cannot allocate or hand over a workspace: the scratch
// buffer of the spread variant is a file-scope device array.  Each GPU the library runs on
// holds its own copy (about 7 MiB) at its own address until the process ends; the address is
// looked up once per device, with that device current, and only that pointer (never the
// array's name, which in host code is a stand-in, not a device address) is handed to kernels.
namespace {

static __device__ __align__(256) unsigned char g_sampler_scratch[areal::SAMPLER_SPLIT_MAX_ROWS *
                                                                areal::SAMPLER_SCRATCH_ROW];
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of this GPU's copy of the array (null + message on failure).
void* static_scratch(std::string* why) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    *why = std::string("hipGetDevice: ") + (e != hipSuccess ? hipGetErrorString(e) : "device index out of range");
    return nullptr;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(g_sampler_scratch));
    if (e != hipSuccess || !p) {
      *why = std::string("hipGetSymbolAddress(sampler scratch): ") + hipGetErrorString(e);
      return nullptr;
    }
    g_scratch_ptr[dev] = p;
  }
  return g_scratch_ptr[dev];
}

}  // namespace

extern "C" int areal_sample_logprob_static(void* hip_stream, int32_t n, int32_t vocab, const float* logits,
                                           const int32_t* seq_ids, const int32_t* positions, float temperature,
                                           float top_p, uint64_t seed, const int32_t* forced,
                                           int32_t* tokens_out, float* logp_behav, float* logp_full) {
  if (n == 0) return AREAL_OK;
  if (n < 0 || vocab <= 0 || !logits || !tokens_out || !logp_behav || (!forced && (!seq_ids || !positions))) {
    areal::set_global_error("areal_sample_logprob_static: NULL argument, negative count or no vocabulary");
    return AREAL_E_INVAL;
  }
  if (n > AREAL_SAMPLE_STATIC_MAX_ROWS || vocab > AREAL_SAMPLE_STATIC_MAX_VOCAB) {
    areal::set_global_error("areal_sample_logprob_static: at most " +
                            std::to_string(AREAL_SAMPLE_STATIC_MAX_ROWS) + " rows of at most " +
                            std::to_string(AREAL_SAMPLE_STATIC_MAX_VOCAB) +
                            " logits fit the static scratch buffer: split the batch, or use areal_sample_logprob");
    return AREAL_E_NOMEM;
  }
  if (!(temperature > 0.f) || !(top_p > 0.f)) {
    areal::set_global_error("areal_sample_logprob_static: temperature and top_p must be > 0");
    return AREAL_E_INVAL;
  }
  std::string why;
  void* scratch = static_scratch(&why);
  if (!scratch) {
    areal::set_global_error(why);
    return AREAL_E_HIP;
  }
  const hipError_t e = areal::launch_sampler((hipStream_t)hip_stream, n, vocab, logits, seq_ids, positions,
                                             1.0f / temperature, top_p, seed, forced, tokens_out, logp_behav,
                                             logp_full, scratch);
  if (e != hipSuccess) {
    areal::set_global_error(std::string("areal_sample_logprob_static: ") + hipGetErrorString(e));
    return e == hipErrorInvalidValue ? AREAL_E_INVAL : AREAL_E_HIP;
  }
  return AREAL_OK;
}
