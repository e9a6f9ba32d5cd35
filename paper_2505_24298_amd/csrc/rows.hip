// Products of a handful of rows (the decode steps of a few sequences): C (+)= X W^T, with the RMSNorm that makes X inside.
//
// Bound by the stream of the weights and by what stands before and after it.  Matrix cores need 16 rows to pay, and a tile
// that passes its weights through LDS pays for barriers, for float32 atomics of K splits and, at 1 row, for 31 rows of
// nothing.  Here a lane takes 16 bytes of a weight row straight into registers, one instruction of a wave 1 KiB in a
// row, multiplies them with its part of the few input rows, which it holds in registers for the whole launch
// (v_dot2_f32_f16: exact products, float32 sums), and the lanes' sums are folded once per weight row.  One work-group of
// 4 waves per compute unit takes the same number of weight rows, and each output has one owner: no atomics, nothing to clear
// beforehand.  The first weights are in flight before the RMSNorm is computed, every work-group for itself, so that the norm
// has no launch of its own.
//
// Bytes in flight: a plain read of 108 (216) KB per compute unit, a launch after an empty one, takes 5.2 (9.7) us with 32 KB in
// flight on each, 5.7 (10.1) with 112 KB.  Two batches of 1 or 2 weight rows per wave (24 - 48 KB): step of one row 965 us, three
// batches 1,026, four 1,043.  The rows that all work-groups read at a time follow one another in memory (round b of work-group w:
// chunk b G + w): with a run of its own for each work-group, 256 places at once, 2 % more (7B shape 2 %).
// Against the tiles of gemm.hip and two RMSNorm launches per layer, steps of n rows, 1.5B shape, 700 tokens: 1 row 1,215 -> 965 us,
// 2 rows 1,234 -> 1,003, 4 rows 1,261 -> 1,046, 8 rows 1,279 -> 1,204; 7B shape, 2,000 tokens: 3,006 -> 2,731, 3,071 -> 2,872, 3 rows
// 3,043 -> 2,832, 4 rows 3,156 -> 2,988.  More rows do not fit a lane's registers at these K.  The output projection and its norm, which
// the tiles stream at 5.9 TB/s, gain 3 - 13 us (2, 4, 8 rows: 998 -> 992, 1,046 -> 1,038, 1,208 -> 1,194 us a step).
#include <algorithm>

#include "kernels.hpp"

namespace areal {

namespace {

constexpr int WAVES = 4, TPB = WAVES * 64;
constexpr int UNITS = 256;                       // compute units: work-groups of a launch
// Weight rows of a work-group at most (sums in LDS; an added output's old value is a lane's).
template <int MODE>
constexpr int max_cols() { return MODE == GEMM_SWIGLU_F16 ? 160 : MODE == GEMM_ADD_F32 ? 64 : 640; }

struct Late {
  void* C;
  int ldc;
  float eps;
};

// Sums over the wave of 4 (2) values at once: exchanged halves and rows of 16 lanes put one value into each row
// (half): folded_value.
template <int CB>
__device__ __forceinline__ float fold_values(const float (&v)[CB]) {
  static_assert(CB == 2 || CB == 4, "values per fold");
  auto swap32 = [](float a, float b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b), false, false);
    const uint32_t lo = r[0], hi = r[1];
    return __builtin_bit_cast(float, lo) + __builtin_bit_cast(float, hi);
  };
  float s = swap32(v[0], v[1]);
  if constexpr (CB == 4) {
    const float t = swap32(v[2], v[3]);
    const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, s), __builtin_bit_cast(uint32_t, t), false, false);
    const uint32_t lo = r[0], hi = r[1];
    s = __builtin_bit_cast(float, lo) + __builtin_bit_cast(float, hi);
  } else {
    s = xor_lanes<16>(s, [](float a, float b) { return a + b; });
  }
  s += dpp<0x128>(s);
  s += dpp<0x124>(s);
  s += dpp<0x4E>(s);
  s += dpp<0xB1>(s);
  return s;
}
// Which of four values a lane holds after fold_values (of two: lane >> 5).
__device__ __forceinline__ int folded_value(int lane) { return ((lane >> 5) & 1) | ((lane >> 3) & 2); }

// LDS only: the weights in flight stay in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The loads before this stay before it (a fence that costs no instruction): the compiler moves loads down to their first use, behind
// the weights' or into the loop, and then waits for all.
__device__ __forceinline__ void issue_here() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
  __builtin_amdgcn_sched_barrier(0);
}

// NR input rows (n of them exist); WPC waves share a weight row, a lane holds NCH times 16 bytes of it.
// NORM: x float32, normalised with `gain`; else halves.  The weights: one matrix, or (stored products) up to three row
// segments, of end8 & 0xFFFF and end8 >> 16 times 8 rows up to the second and third, or (SwiGLU) gate p0 and up p1.
template <int NR, int NCH, int WPC, int MODE, bool NORM>
__global__ __launch_bounds__(TPB) void rows_kernel(const void* __restrict__ x, const f16* __restrict__ gain,
                                                   const f16* __restrict__ p0, const f16* __restrict__ p1,
                                                   const f16* __restrict__ p2, uint32_t end8, int N, int K, uint32_t shape,
                                                   Late late) {
  constexpr int GROUPS = WAVES / WPC;
  constexpr int CB = NCH > 3 ? 1 : 2, DEPTH = 2;           // weight rows per batch of loads, batches in flight
  constexpr int KP = NCH * WPC * 512;                      // K and what is masked
  constexpr int COLS = max_cols<MODE>();
  __shared__ __attribute__((aligned(16))) f16 xs[NORM && NR > 1 ? NR * KP : 8];
  __shared__ float red[NR][WPC][COLS];

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = wave / WPC, sub = wave % WPC;
  const int n = shape & 255, rounds = (shape >> 8) & 255, G = shape >> 16;
  // weight rows in the order of their outputs (SwiGLU: gate and up of a feature side by side); round b of this work-group
  // takes RC of them from first(b) on
  constexpr int PER_OUT = MODE == GEMM_SWIGLU_F16 ? 2 : 1, RC = GROUPS * CB, RO = RC / PER_OUT;
  const int total = N * PER_OUT;
  auto first = [&](int b) { return (b * G + (int)blockIdx.x) * RC; };

  // the input rows first: they are needed first, and loads return in order
  // A single row is normalised by every wave for itself, in the order in which it holds it: nothing goes through LDS and no wave
  // waits for another (1,041 -> 1,015 us).  Of several rows, r = wave, wave + 4, .. are a wave's.
  constexpr bool ALONE = NORM && NR == 1 && WPC == 1;
  constexpr int NV = NORM ? KP / 256 : 1, RPW = (NR + WAVES - 1) / WAVES;
  f32x4 hv[RPW][NV];
  f16x4 gv[NV];
  f16x8 xr[NR][NCH];
  const int lane_off = (sub * 64 + lane) * 16;
  f16x8 g8[ALONE ? NCH : 1];
  if constexpr (ALONE) {
    const auto hr = buffer_rsrc(x, (uint32_t)K * 4u), gr = buffer_rsrc(gain, (uint32_t)K * 2u);
#pragma unroll
    for (int i = 0; i < NV; ++i) hv[0][i] = buf4f(hr, (i >> 1) * 2048 + lane * 32 + (i & 1) * 16);
#pragma unroll
    for (int c = 0; c < NCH; ++c) g8[c] = buf8(gr, lane_off + c * 1024);
  } else if constexpr (NORM) {
    const auto gr = buffer_rsrc(gain, wave < n ? (uint32_t)K * 2u : 0u);
#pragma unroll
    for (int k = 0; k < RPW; ++k) {
      const int r = wave + k * WAVES;
      const auto hr = buffer_rsrc((const float*)x + (int64_t)r * K, r < n ? (uint32_t)K * 4u : 0u);
#pragma unroll
      for (int i = 0; i < NV; ++i) hv[k][i] = buf4f(hr, (i * 64 + lane) * 16);
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) gv[i] = buf4(gr, (i * 64 + lane) * 8);
  } else {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const auto rr = buffer_rsrc((const f16*)x + (int64_t)r * K, r < n ? (uint32_t)K * 2u : 0u);
#pragma unroll
      for (int c = 0; c < NCH; ++c) xr[r][c] = buf8(rr, lane_off + c * WPC * 1024);
    }
  }
  issue_here();

  // column q of this work-group's; past the end: an empty range, which reads nothing
  const int mid = (int)(end8 & 0xFFFFu) * 8, last = (int)(end8 >> 16) * 8;
  auto load = [&](f16x8 (&w)[CB][NCH], int b) {
#pragma unroll
    for (int u = 0; u < CB; ++u) {
      const int c = first(b) + grp * CB + u;
      const f16* p;
      int64_t row;
      if (MODE == GEMM_SWIGLU_F16) {
        p = c & 1 ? p1 : p0;
        row = c >> 1;
      } else if (MODE == GEMM_STORE_F32) {
        p = c >= last ? p2 : (c >= mid ? p1 : p0);
        row = c - (c >= last ? last : (c >= mid ? mid : 0));
      } else {
        p = p0;
        row = c;
      }
      const auto wr = buffer_rsrc(p + row * K, b < rounds && c < total ? (uint32_t)K * 2u : 0u);
#pragma unroll
      for (int c = 0; c < NCH; ++c) w[u][c] = buf8(wr, lane_off + c * WPC * 1024);
    }
  };
  f16x8 w[DEPTH][CB][NCH];
#pragma unroll
  for (int d = 0; d < DEPTH; ++d) load(w[d], d);
  issue_here();
  void* const C = late.C;
  const int ldc = late.ldc;
  asm volatile("" : : "s"(C), "s"(ldc));                    // read here, not where the launch ends
  // output i of this work-group's
  auto output = [&](int i) { return ((i / RO) * G + (int)blockIdx.x) * RO + i % RO; };
  // the residual's old values: one owner per output, wave r has rows r, r + 4, ..
  float old[RPW];
  if constexpr (MODE == GEMM_ADD_F32) {
#pragma unroll
    for (int k = 0; k < RPW; ++k) {
      const int r = wave + k * WAVES;
      const auto cr = buffer_rsrc((const float*)C + (int64_t)r * ldc, r < n ? (uint32_t)N * 4u : 0u);
      old[k] = __builtin_bit_cast(float, buf1(cr, output(lane) * 4));
    }
  }

  if constexpr (ALONE) {
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i)
      ss += hv[0][i][0] * hv[0][i][0] + hv[0][i][1] * hv[0][i][1] + hv[0][i][2] * hv[0][i][2] + hv[0][i][3] * hv[0][i][3];
    ss = wave_sum(ss);
    const float rs = 1.0f / sqrtf(ss / (float)K + late.eps);
#pragma unroll
    for (int c = 0; c < NCH; ++c)
#pragma unroll
      for (int e = 0; e < 8; ++e) xr[0][c][e] = f2h_sat(hv[0][2 * c + (e >> 2)][e & 3] * rs * h2f(g8[c][e]));
  } else if constexpr (NORM) {
#pragma unroll
    for (int k = 0; k < RPW; ++k) {
      const f32x4(&v)[NV] = hv[k];
      float ss = 0.f;
#pragma unroll
      for (int i = 0; i < NV; ++i) ss += v[i][0] * v[i][0] + v[i][1] * v[i][1] + v[i][2] * v[i][2] + v[i][3] * v[i][3];
      ss = wave_sum(ss);
      const float rs = 1.0f / sqrtf(ss / (float)K + late.eps);
      const int r = wave + k * WAVES;
      if (r < NR) {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
          f16x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = f2h_sat(v[i][e] * rs * h2f(gv[i][e]));
          *reinterpret_cast<f16x4*>(&xs[r * KP + (i * 64 + lane) * 4]) = o;       // zeros from K on
        }
      }
    }
    lds_barrier();
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int c = 0; c < NCH; ++c) xr[r][c] = *reinterpret_cast<const f16x8*>(&xs[r * KP + lane_off / 2 + c * WPC * 512]);
  }

  auto compute = [&](const f16x8 (&wt)[CB][NCH], int b) {
    float acc[NR][CB];
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int u = 0; u < CB; ++u) acc[r][u] = 0.f;
#pragma unroll
    for (int c = 0; c < NCH; ++c)
#pragma unroll
      for (int e = 0; e < 8; e += 2)
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
          for (int u = 0; u < CB; ++u)
            acc[r][u] = __builtin_amdgcn_fdot2(f16x2{wt[u][c][e], wt[u][c][e + 1]}, f16x2{xr[r][c][e], xr[r][c][e + 1]},
                                               acc[r][u], false);
    const int q0 = (b * GROUPS + grp) * CB;
    if constexpr (NR == 1 && CB == 1) {
      const float s = wave_sum(acc[0][0]);
      if (lane == 0) red[0][sub][q0] = s;
    } else if constexpr (CB == 1) {
#pragma unroll
      for (int r = 0; r < NR; r += 2) {
        const float v[2] = {acc[r][0], acc[r + 1][0]};
        const float s = fold_values<2>(v);
        if ((lane & 31) == 0) red[r + (lane >> 5)][sub][q0] = s;
      }
    } else if constexpr (NR == 1) {
      const float s = fold_values<2>(acc[0]);
      const int q = q0 + (lane >> 5);
      if ((lane & 31) == 0) red[0][sub][q] = s;
    } else {
#pragma unroll
      for (int r = 0; r < NR; r += 2) {
        const float v[4] = {acc[r][0], acc[r][1], acc[r + 1][0], acc[r + 1][1]};
        const float s = fold_values<4>(v);
        const int k = folded_value(lane), q = q0 + (k & 1);
        if ((lane & 15) == 0) red[r + (k >> 1)][sub][q] = s;
      }
    }
  };
  static_assert(DEPTH == 2, "two batches in turn");
  // One way out after each half, so that the wait of a half always finds the other's loads behind its own.  (Left in the middle
  // for the loop's head instead, the first half waited for all loads: 1,010 us.)
  for (int b = 0;; b += 2) {
    compute(w[0], b);
    load(w[0], b + 2);
    if (b + 1 >= rounds) break;
    compute(w[1], b + 1);
    load(w[1], b + 3);
    if (b + 2 >= rounds) break;
  }
  lds_barrier();

#pragma unroll
  for (int k = 0; k < RPW; ++k) {
    const int r = wave + k * WAVES;
    if (r >= n) break;
    for (int i = lane; i < rounds * RO; i += 64) {
      const int o = output(i);
      if (o >= N) continue;
      auto sum = [&](int q) {
        float s = red[r][0][q];
#pragma unroll
        for (int p = 1; p < WPC; ++p) s += red[r][p][q];
        return s;
      };
      const int64_t at = (int64_t)r * ldc + o;
      if constexpr (MODE == GEMM_SWIGLU_F16) {
        ((f16*)C)[at] = f2h_sat(silu_f(sum(2 * i)) * sum(2 * i + 1));
      } else if constexpr (MODE == GEMM_ADD_F32) {
        ((float*)C)[at] = old[k] + sum(i);                  // one round of this loop
      } else {
        ((float*)C)[at] = sum(i);
      }
    }
  }
}

// Chunks of 16 bytes per lane and waves per weight row, by the largest K of each, and the most rows of it (measured at the head
// of this file).  A wave has a weight row to itself as long as its chunks fit: with four waves to a row of K = 3,584 every one of
// them folds every sum (7B shape, 1 row 2,913 us, with one 2,871; 4 rows 3,305 and 3,146).
struct Layout { int K, nch, wpc, rows; };
constexpr Layout kLayouts[] = {{512, 1, 1, 8},  {1536, 3, 1, 8},  {2048, 4, 1, 8}, {3584, 7, 1, 4},
                                {4096, 8, 1, 4}, {12288, 6, 4, 8}, {20480, 10, 4, 4}};
constexpr int kNormLayouts = 5;
int layout(int M, int K, bool norm) {
  for (int l = 0; l < (norm ? kNormLayouts : 7); ++l)
    if (K <= kLayouts[l].K) return M <= kLayouts[l].rows ? l : -1;
  return -1;
}

// Weight rows of a round of a work-group, and rounds of all.
int chunk(int lay) { return WAVES / kLayouts[lay].wpc * (kLayouts[lay].nch > 3 ? 1 : 2); }
int chunks_of(int N, GemmMode mode, int lay) { return (N * (mode == GEMM_SWIGLU_F16 ? 2 : 1) + chunk(lay) - 1) / chunk(lay); }

template <int NR, int MODE, bool NORM, int LAY>
void launch(int lay, int grid, hipStream_t s, const void* x, const f16* gain, const GemmW& W, uint32_t end8, int N, int K,
            uint32_t shape, Late late) {
  if constexpr (LAY < (NORM ? kNormLayouts : 7)) {
    if (lay != LAY) return launch<NR, MODE, NORM, LAY + 1>(lay, grid, s, x, gain, W, end8, N, K, shape, late);
    if constexpr (NR <= kLayouts[LAY].rows)
      rows_kernel<NR, kLayouts[LAY].nch, kLayouts[LAY].wpc, MODE, NORM>
          <<<grid, TPB, 0, s>>>(x, gain, W.ptr[0], W.ptr[1], W.ptr[2], end8, N, K, shape, late);
  }
}

}  // namespace

bool rows_product_serves(int M, int N, int K, GemmMode mode, bool norm) {
  if (M < 1 || N < 1 || K < 8 || K % 8 || layout(M, K, norm) < 0) return false;
  const int lay = layout(M, K, norm), most = mode == GEMM_SWIGLU_F16 ? max_cols<GEMM_SWIGLU_F16>()
                                               : mode == GEMM_ADD_F32 ? max_cols<GEMM_ADD_F32>() : max_cols<GEMM_STORE_F32>();
  return N <= UNITS * most && (chunks_of(N, mode, lay) + UNITS - 1) / UNITS * chunk(lay) <= most;
}

hipError_t launch_rows_product(hipStream_t s, const void* x, const f16* gain, float eps, GemmW W, void* C, int M, int N, int K,
                               int ldc, GemmMode mode) {
  const bool norm = gain != nullptr;
  if (!rows_product_serves(M, N, K, mode, norm) || !x || !C || ldc < N || !W.ptr[0]) return hipErrorInvalidValue;
  if (((uintptr_t)x | (uintptr_t)gain | (uintptr_t)W.ptr[0] | (uintptr_t)W.ptr[1] | (uintptr_t)W.ptr[2]) & 15 ||
      (uintptr_t)C & (mode == GEMM_SWIGLU_F16 ? 1 : 3))
    return hipErrorInvalidValue;
  if (mode == GEMM_ADD_F32 && W.end[0] != N) return hipErrorInvalidValue;
  // modes in use: the norm before stored and SwiGLU products, none before residual adds
  if (norm != (mode != GEMM_ADD_F32)) return hipErrorInvalidValue;
  uint32_t end8 = 0xFFFFFFFFu;                                                    // beyond any column
  if (mode == GEMM_SWIGLU_F16) {
    if (!W.ptr[1]) return hipErrorInvalidValue;
  } else if (mode == GEMM_STORE_F32 && W.ptr[1]) {
    if (!W.ptr[2] || W.end[0] % 8 || W.end[1] % 8 || W.end[0] < 0 || W.end[1] < W.end[0] || W.end[2] != N ||
        W.end[1] > N || N >= 0xFFFF * 8)
      return hipErrorInvalidValue;
    end8 = (uint32_t)(W.end[0] / 8) | (uint32_t)(W.end[1] / 8) << 16;
  }
  const int lay = layout(M, K, norm), chunks = chunks_of(N, mode, lay), grid = std::min(UNITS, chunks);
  const uint32_t shape = (uint32_t)M | (uint32_t)((chunks + grid - 1) / grid) << 8 | (uint32_t)grid << 16;
  const Late late{C, ldc, eps};
#define AREAL_MODE(NR)                                                                                               \
  (mode == GEMM_STORE_F32    ? launch<NR, GEMM_STORE_F32, true, 0>(lay, grid, s, x, gain, W, end8, N, K, shape, late)    \
   : mode == GEMM_SWIGLU_F16 ? launch<NR, GEMM_SWIGLU_F16, true, 0>(lay, grid, s, x, gain, W, end8, N, K, shape, late)   \
                             : launch<NR, GEMM_ADD_F32, false, 0>(lay, grid, s, x, gain, W, end8, N, K, shape, late))
  if (M == 1) AREAL_MODE(1);
  else if (M == 2) AREAL_MODE(2);
  else if (M <= 4) AREAL_MODE(4);
  else if (M <= 6) AREAL_MODE(6);
  else AREAL_MODE(8);
#undef AREAL_MODE
  return hipGetLastError();
}

}  // namespace areal
