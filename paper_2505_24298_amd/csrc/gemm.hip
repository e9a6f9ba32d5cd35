// f16 x f16 -> float32 GEMM on the gfx950 matrix cores.
//   C[M,N] (+)= A[M,K] * W[N,K]^T      (both operands K-contiguous)
// Work-group tile BM x BN x 64 staged through LDS with register prefetch of
// the next K-slab; WM x WN wavefronts, each computing (BM/WM) x (BN/WN) with
// v_mfma_f32_32x32x16_f16.  The K range can be split over work-groups
// (float32 atomic accumulation into C) so that skinny decode-shape products
// still fill 256 compute units; the block id -> tile map keeps the row tiles
// that share a weight panel on one XCD (one L2).
#include <algorithm>
#include <cmath>

#include "kernels.hpp"
#include "row_groups.hpp"
#include <cstdlib>
#include <type_traits>

namespace areal {

namespace {

constexpr int BK = 64;
constexpr int LDS_K = BK + 8;   // row stride in elements (144 B): conflict-free 16-B reads

// Row `b` of the W tile -> pointer to that row of the (segmented) weight, or
// null when it lies outside the matrix.
template <int BN, int MODE>
__device__ __forceinline__ const f16* w_row_ptr(const GemmW& W, int tile_n, int b, int N, int K) {
  if (MODE == GEMM_SWIGLU_F16) {
    // every 64 tile rows = 32 gate rows then 32 up rows of the same 32 features
    const int grp = b >> 6, within = b & 63;
    const int isup = within >> 5, c = within & 31;
    const int f = tile_n * (BN / 2) + grp * 32 + c;
    return f < N ? W.ptr[isup] + (int64_t)f * K : nullptr;
  } else {
    const int n = tile_n * BN + b;
    if (n >= N) return nullptr;
    if (n < W.end[0]) return W.ptr[0] + (int64_t)n * K;
    if (n < W.end[1]) return W.ptr[1] + (int64_t)(n - W.end[0]) * K;
    return W.ptr[2] + (int64_t)(n - W.end[1]) * K;
  }
}

// The weights as the direct-to-LDS kernels take them: scalar arguments, which arrive in registers with the launch.
// What comes before the first load counts in a decode step, whose products of a few microseconds cannot start before
// the kernel ahead of them ends: with the arguments read from memory (a struct, and one of its pointers again
// for every row group) and divisions in the tile map, a wave of the 32 x 80 gate/up tile ran some 300 instructions and
// ten dependent reads before its first load; with scalars and the map below about 110 and none (the resources of a wave's
// later row groups, some ten instructions each, are made while its first loads travel).  Decode step of one row 1,370 ->
// 1,251 us, of 24 rows 2,183 -> 2,066, of 88 3,107 -> 3,011, one prompt of 301 tokens 2,591 -> 2,525 (a part of it from the
// other kernels' arguments).
struct WRows {
  const f16 *p0, *p1, *p2;
  int end0, end1;
};

// Buffer resources of the row groups of a tile (row_groups.hpp).  Rows outside the matrix read as zero or as its last row and
// feed only accumulator rows / columns that are never stored.
template <int BM, int BN, int MODE>
struct TileRsrc {
  static constexpr int NC = MODE == GEMM_SWIGLU_F16 ? BN / 2 : BN;
  const char *pa, *pw0, *pw1;       // first rows of the tile
  uint32_t row_bytes, a_bytes, w_bytes;   // of a row, and of those of the matrix from there on, as far as the tile reaches
  uint64_t seg0, to1, to2;          // stored products: address of the first segment, and what leads on to the others
  int end0, end1, n0, N;
  __device__ __forceinline__ TileRsrc(const f16* A, WRows W, int M, int n, int K, int tile_m, int tile_n)
      : row_bytes((uint32_t)K * 2u), seg0((uint64_t)W.p0), to1((uint64_t)W.p1 ^ (uint64_t)W.p0),
        to2((uint64_t)W.p2 ^ (uint64_t)W.p1), end0(W.end0), end1(W.end1), n0(tile_n * NC), N(n) {
    pa = reinterpret_cast<const char*>(A + (int64_t)(tile_m * BM) * K);
    a_bytes = (uint32_t)min(M - tile_m * BM, BM) * row_bytes;
    w_bytes = (uint32_t)min(N - n0, NC) * row_bytes;
    if (MODE != GEMM_STORE_F32) pw0 = reinterpret_cast<const char*>(W.p0 + (int64_t)n0 * K);
    if (MODE == GEMM_SWIGLU_F16) pw1 = reinterpret_cast<const char*>(W.p1 + (int64_t)n0 * K);
  }
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const char* p, int row, uint32_t bytes) const {
    const RowRange g = row_range(row, row_bytes, bytes);
    return buffer_rsrc(p + g.first, g.bytes);
  }
  // The group that begins at row r of the A tile; all of its rows (and those of a W tile of one matrix).
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t a(int r) const { return rsrc(pa, r, a_bytes); }
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t a() const { return buffer_rsrc(pa, a_bytes); }
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t w() const { return buffer_rsrc(pw0, w_bytes); }
  // The group that begins at row r of the W tile, or at its feature r of gate or up.  Stored products: of up to three segments,
  // each of whole groups but the last; a group below the matrix takes its last one.
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t w(int r, bool is_up) const {
    if (MODE == GEMM_SWIGLU_F16) return rsrc(is_up ? pw1 : pw0, r, w_bytes);
    if (MODE != GEMM_STORE_F32) return rsrc(pw0, r, w_bytes);
    const int n = min(n0 + r, (N - 1) & ~7);
    const bool in1 = n >= end0, in2 = in1 && n >= end1;              // (one segment: end0 = N, end1 unset)
    const uint64_t p = seg0 ^ (in1 ? to1 : 0) ^ (in2 ? to2 : 0);
    const int start = in2 ? end1 : (in1 ? end0 : 0);
    return buffer_rsrc(reinterpret_cast<const char*>(p) + (int64_t)(n - start) * row_bytes, (uint32_t)min(8, N - n) * row_bytes);
  }
};

// Whether a group's place in its tile stands in the lanes' offsets (one register a load, one resource an operand) or in a base of its
// own (four scalar registers a load).  Residual adds take the former: where rows are a multiple of 4,096 bytes apart, so that all
// of a slab's lines lie on few memory channels, it is the faster one whatever the reason (128 x 96 tiles, 128 x 1,536 x 28,672 in 8 splits
// 48.0 us with bases, 38.4 with lanes; 128 x 4,128 x 14,336 43.2 and 41.5, x 18,944 52.0 and 50.9, x 11,008 33.4 and 34.2), except
// where the accumulators leave no register for it (256 x 256).  Gate/up and stored products take bases (8,960 features of K = 1,536,
// 128 rows 18.5 us with one resource and scalar places, 17.9; QKV 4.05 and 3.9 us at 8 rows, 9.15 and 9.0 at 256).
template <int BM, int BN, int NW, int MODE>
constexpr bool lane_rows() { return MODE == GEMM_ADD_F32 && BM * BN < 128 * 64 * NW; }

// Arguments that a kernel needs late: read from memory where they are used.
struct GemmLate {
  void* C;
  int ldc;
  GemmLse lse;
};

// Block -> (row tile, column tile, K split).  Work-groups are handed to the 8 XCDs round-robin in launch order, x fastest,
// so ids equal mod 8 share one L2.
//  * Up to 256 rows (decode): a unit = (column tile, K split) with all its
//    row tiles, so that the work-groups that read one W slab run side by side on
//    one XCD; units go to the XCDs round-robin, which keeps the XCDs evenly
//    loaded whatever the number of column tiles (1536 columns = 12 tiles).  The grid is (8, row tiles, units / 8), and the
//    one division left is a multiplication by `map` = 2^32 / column tiles, rounded up (0: one column tile): such a
//    launch is a few microseconds, and a wave needs about 0.1 us for each 64 instructions it runs before its first load.
//  * Above 256 rows (prefill), map = kLinearMap, a grid of one dimension: the tiles are numbered band by band (4 column
//    tiles), inside a band in blocks of 8 row tiles, one K split after the other, and XCD x
//    takes the x-th eighth of that row of tiles: every XCD gets the same number of
//    tiles whatever the shape, and the 32 work-groups resident on its compute units
//    are neighbours that share A and W slabs in its L2.  (Column tiles handed out
//    round-robin left XCDs idle where their number is not a multiple of 8: with 12
//    tiles of 128 columns, four XCDs did two thirds of the O projection.)
constexpr int BAND_N = 4, BAND_M = 8, DECODE_ROWS = 256;
constexpr uint32_t kLinearMap = 0xFFFFFFFFu;
struct Grid { dim3 dim; uint32_t map; };
static Grid make_grid(int M, int m_tiles, int n_tiles, int splits) {
  const int64_t units = (int64_t)n_tiles * splits, deep = (units + 7) / 8;
  // unit / column tiles by `map` is exact while (units + 8) * column tiles stays below 2^32
  if (M <= DECODE_ROWS && deep < 65536 && (units + 8) * n_tiles < (int64_t)1 << 32)
    return {dim3(8, m_tiles, (unsigned)deep), n_tiles == 1 ? 0u : (uint32_t)((((uint64_t)1 << 32) + n_tiles - 1) / n_tiles)};
  return {dim3((unsigned)(8 * ((units * m_tiles + 7) / 8))), kLinearMap};
}
__device__ __forceinline__ bool tile_of_block(uint32_t map, int m_tiles, int n_tiles, int nk, int sps, int& tile_m, int& tile_n,
                                              int& split) {
  if (map != kLinearMap) {
    const uint32_t unit = blockIdx.z * 8 + blockIdx.x;
    tile_m = blockIdx.y;
    split = map ? __umulhi(unit, map) : unit;   // the up to 7 padding units get split >= the split count: an empty
    tile_n = unit - split * n_tiles;            // K range, on which the kernels return before touching memory
    return true;
  }
  const int xcd = blockIdx.x & 7, q = blockIdx.x >> 3;
  const int tiles = m_tiles * n_tiles, splits = sps < nk ? (nk + sps - 1) / sps : 1;
  const int64_t units = (int64_t)tiles * splits;
  const int u = (int)(units * xcd / 8) + q;
  if (u >= (int)(units * (xcd + 1) / 8)) return false;
  split = splits == 1 ? 0 : u / tiles;
  const int t = u - split * tiles;
  const int band = t / (BAND_N * m_tiles), in_band = t - band * BAND_N * m_tiles;
  const int width = min(BAND_N, n_tiles - band * BAND_N);
  const int blk = in_band / (BAND_M * width), in_blk = in_band - blk * BAND_M * width;
  const int height = min(BAND_M, m_tiles - blk * BAND_M);
  // scalars, whatever unit the compiler divides on: a buffer resource in vector registers makes a loop of every load
  split = __builtin_amdgcn_readfirstlane(split);
  tile_m = __builtin_amdgcn_readfirstlane(blk * BAND_M + in_blk % height);
  tile_n = __builtin_amdgcn_readfirstlane(band * BAND_N + in_blk / height);
  return true;
}

template <int BM, int BN, int WM, int WN, int MODE, bool RAGGED_K>
__global__ __launch_bounds__(WM * WN * 64) void gemm_kernel(const f16* __restrict__ A, int M, int N, int K,
                                                            uint32_t map, int slabs_per_split, int ldc,
                                                            void* __restrict__ Cv, int atomic, GemmW W) {
  constexpr int NT = WM * WN * 64;
  constexpr int TM = BM / WM / 32, TN = BN / WN / 32;   // 32x32 MFMA tiles per wave
  constexpr int ACH = BM * 8 / NT, BCH = BN * 8 / NT;   // 16-B chunks per thread per slab
  static_assert(TM >= 1 && TN >= 1 && ACH >= 1 && BCH >= 1, "tile too small for the wave grid");
  static_assert(MODE != GEMM_SWIGLU_F16 || (TN % 2 == 0), "SwiGLU needs gate+up in one wave tile");
  __shared__ __attribute__((aligned(16))) f16 sA[2][BM * LDS_K];
  __shared__ __attribute__((aligned(16))) f16 sB[2][BN * LDS_K];

  constexpr int NC = MODE == GEMM_SWIGLU_F16 ? BN / 2 : BN;
  int tile_m, tile_n, split;
  if (!tile_of_block(map, (M + BM - 1) / BM, (N + NC - 1) / NC, (K + BK - 1) / BK, slabs_per_split, tile_m, tile_n, split))
    return;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int m0 = tile_m * BM;
  const int kc = tid & 7, r0 = tid >> 3;         // chunk column, first chunk row
  constexpr int RSTEP = NT / 8;                  // rows covered per chunk round

  // Rows outside the matrix are clamped to a valid row: they only feed
  // accumulator rows / columns that are never stored.
  const f16* pa[ACH];
  const f16* pb[BCH];
#pragma unroll
  for (int i = 0; i < ACH; ++i) {
    const int m = min(m0 + r0 + RSTEP * i, M - 1);
    pa[i] = A + (int64_t)m * K + kc * 8;
  }
#pragma unroll
  for (int i = 0; i < BCH; ++i) {
    const f16* p = w_row_ptr<BN, MODE>(W, tile_n, r0 + RSTEP * i, N, K);
    if (!p) p = w_row_ptr<BN, MODE>(W, 0, 0, N, K);
    pb[i] = p + kc * 8;
  }

  struct Slab { f16x8 a[ACH], b[BCH]; };
  // RAGGED_K (K % 64 != 0; K % 8 == 0 always): a 16-byte chunk is all inside or
  // all outside the row; outside chunks are fetched from the row start and zeroed.
  auto load_slab = [&](Slab& r, int k0) {
    if (RAGGED_K) {
      const f16x8 zero8 = {0, 0, 0, 0, 0, 0, 0, 0};
      const bool kin = k0 + kc * 8 < K;
      const int ko = kin ? k0 : -kc * 8;
#pragma unroll
      for (int i = 0; i < BCH; ++i) { const f16x8 v = ld8(pb[i] + ko); r.b[i] = kin ? v : zero8; }
#pragma unroll
      for (int i = 0; i < ACH; ++i) { const f16x8 v = ld8(pa[i] + ko); r.a[i] = kin ? v : zero8; }
    } else {
#pragma unroll
      for (int i = 0; i < BCH; ++i) r.b[i] = ld8(pb[i] + k0);
#pragma unroll
      for (int i = 0; i < ACH; ++i) r.a[i] = ld8(pa[i] + k0);
    }
  };
  auto store_slab = [&](const Slab& r, int buf) {
#pragma unroll
    for (int i = 0; i < ACH; ++i)
      *reinterpret_cast<f16x8*>(&sA[buf][(r0 + RSTEP * i) * LDS_K + kc * 8]) = r.a[i];
#pragma unroll
    for (int i = 0; i < BCH; ++i)
      *reinterpret_cast<f16x8*>(&sB[buf][(r0 + RSTEP * i) * LDS_K + kc * 8]) = r.b[i];
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  const int fr = lane & 31, fh = lane >> 5;      // fragment row, K half
  auto compute = [&](int buf) {
#pragma unroll
    for (int kk = 0; kk < BK / 16; ++kk) {
      f16x8 fa[TM], fb[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i)
        fa[i] = *reinterpret_cast<const f16x8*>(
            &sA[buf][(wm * (BM / WM) + i * 32 + fr) * LDS_K + kk * 16 + fh * 8]);
#pragma unroll
      for (int j = 0; j < TN; ++j)
        fb[j] = *reinterpret_cast<const f16x8*>(
            &sB[buf][(wn * (BN / WN) + j * 32 + fr) * LDS_K + kk * 16 + fh * 8]);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[i], fb[j], acc[i][j], 0, 0, 0);
    }
  };

  // Software pipeline, two slabs of global loads in flight: while slab kt is
  // multiplied out of LDS, slab kt+1 sits in one register set (already
  // requested) and slab kt+2 is requested into the other.
  const int nk_all = (K + BK - 1) / BK;
  const int kt0 = split * slabs_per_split;
  const int kt1 = min(nk_all, kt0 + slabs_per_split);
  if (kt0 >= kt1) return;
  Slab r0s, r1s;
  // Loads are issued unconditionally (past the end they re-read the last slab)
  // so that no branch separates a load from the wait that consumes it: the
  // wait counters then let two slabs stay in flight.
  const int k_last = (kt1 - 1) * BK;
  load_slab(r0s, kt0 * BK);
  load_slab(r1s, min((kt0 + 1) * BK, k_last));
  store_slab(r0s, 0);
  __syncthreads();
  for (int kt = kt0; kt < kt1; kt += 2) {
    // even step: LDS buffer 0 holds slab kt, r1s holds slab kt+1
    load_slab(r0s, min((kt + 2) * BK, k_last));
    compute(0);
    store_slab(r1s, 1);
    __syncthreads();
    if (kt + 1 >= kt1) break;
    // odd step: LDS buffer 1 holds slab kt+1, r0s holds slab kt+2
    load_slab(r1s, min((kt + 3) * BK, k_last));
    compute(1);
    store_slab(r0s, 0);
    __syncthreads();
  }

  // D layout of the 32x32 tile: lane (fh, fr) holds column fr, rows 8*(v/4) + 4*fh + v%4.
  if (MODE == GEMM_SWIGLU_F16) {
    f16* C = reinterpret_cast<f16*>(Cv);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; j += 2) {
        // wave columns [wn*BN/WN + j*32, +64) = gate | up of 32 features
        const int f = tile_n * (BN / 2) + (wn * (BN / WN) + j * 32) / 2 + fr;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int m = m0 + wm * (BM / WM) + i * 32 + 8 * (v >> 2) + 4 * fh + (v & 3);
          if (m < M && f < N)
            C[(int64_t)m * ldc + f] = f2h_sat(silu_f(acc[i][j][v]) * acc[i][j + 1][v]);
        }
      }
  } else {
    float* C = reinterpret_cast<float*>(Cv);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int n = tile_n * BN + wn * (BN / WN) + j * 32 + fr;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int m = m0 + wm * (BM / WM) + i * 32 + 8 * (v >> 2) + 4 * fh + (v & 3);
          if (m < M && n < N) {
            float* p = C + (int64_t)m * ldc + n;
            if (atomic) unsafeAtomicAdd(p, acc[i][j][v]);
            else if (MODE == GEMM_ADD_F32) *p += acc[i][j][v];
            else *p = acc[i][j][v];
          }
        }
      }
  }
}


// Epilogue of dma_tile: the wave's accumulators to C.  FULL: the tile lies wholly
// inside the matrix and no element is checked.  Row addresses are wave-uniform (scalar registers);
// a lane adds one 32-bit offset.  With bounds, 64-bit addresses and half-word stores instead, the two waves of a
// SIMD spend about a seventh of a gate/up tile of 24 slabs (K = 1,536) here: 8,192 x 17,920 x 1,536 in 256 x 256 tiles
// of dma_tile 454 us, 424 with this form.  The division in silu is 16 us of such a product: 422 us with an approximate
// reciprocal in its place, 437 with it.
template <int BM, int BN, int WM, int WN, int MODE, bool FULL>
__device__ __forceinline__ void store_tile_part(const f32x16 (&acc)[BM / WM / 32][BN / WN / 32],
                                                void* __restrict__ Cv, int M, int N, int ldc, int tile_m,
                                                int tile_n, int wm, int wn, int fr, int fh, int atomic) {
  constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
  const int m_wave = tile_m * BM + wm * (BM / WM);
  if (MODE == GEMM_SWIGLU_F16) {
    // A lane holds one feature of 16 rows; neighbouring lanes trade the odd rows of one for the even
    // rows of the other, so that each stores two features of a row as one word.
    const int odd = fr & 1;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; j += 2) {
        const int f0 = tile_n * (BN / 2) + (wn * (BN / WN) + j * 32) / 2;
        f16* Cw = reinterpret_cast<f16*>(Cv) + (int64_t)(m_wave + i * 32) * ldc + f0;
        const int lane_off = (4 * fh + odd) * ldc + (fr - odd);
#pragma unroll
        for (int v = 0; v < 16; v += 2) {
          const float y0 = silu_f(acc[i][j][v]) * acc[i][j + 1][v];
          const float y1 = silu_f(acc[i][j][v + 1]) * acc[i][j + 1][v + 1];
          const uint32_t h0 = __builtin_bit_cast(uint16_t, f2h_sat(y0)), h1 = __builtin_bit_cast(uint16_t, f2h_sat(y1));
          const uint32_t got = dpp_xor1(odd ? h0 : h1);
          const uint32_t w = odd ? (got | (h1 << 16)) : (h0 | (got << 16));
          const int r = 8 * (v >> 2) + (v & 3);
          f16* p = Cw + (int64_t)r * ldc + lane_off;
          if (FULL) {
            *reinterpret_cast<uint32_t*>(p) = w;
          } else if (m_wave + i * 32 + r + 4 * fh + odd < M && f0 + fr - odd < N) {   // N is even
            *reinterpret_cast<uint32_t*>(p) = w;
          }
        }
      }
  } else {
    const int lane_off = 4 * fh * ldc + fr;
    const int n_wave = tile_n * BN + wn * (BN / WN);
    float* Cw = reinterpret_cast<float*>(Cv) + (int64_t)m_wave * ldc + n_wave;
    auto inside = [&](int i, int j, int r) {
      return FULL || (m_wave + i * 32 + r + 4 * fh < M && n_wave + j * 32 + fr < N);
    };
    auto at = [&](int i, int j, int r, int ld) { return Cw + (int64_t)(i * 32 + r) * ld + j * 32 + lane_off; };
    if (MODE == GEMM_ADD_F32 && !atomic) {
      // Nobody else adds into this tile: the residual's values of 32 rows are fetched together, one
      // batch ahead of the stores (a plain += waits for every load in turn, an atomic is a read and
      // a write in the L2).  The O projection of 8,192 rows, 8,192 x 1,536 x 1,536, went from 82 us with
      // atomics to 55 inside a scoring pass, together with the even tile map and the buffer loads.
      // The opaque row strides keep one batch's addresses from staying in registers for another.
      float old[2][TN][16];
      auto fetch = [&](int i) {
        int ld = ldc;
        asm volatile("" : "+s"(ld));
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int r = 8 * (v >> 2) + (v & 3);
            old[i & 1][j][v] = inside(i, j, r) ? *at(i, j, r, ld) : 0.f;
          }
        __builtin_amdgcn_sched_barrier(0);
      };
      fetch(0);
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        if (i + 1 < TM) fetch(i + 1);
        int ld = ldc;
        asm volatile("" : "+s"(ld));
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int r = 8 * (v >> 2) + (v & 3);
            if (inside(i, j, r)) *at(i, j, r, ld) = old[i & 1][j][v] + acc[i][j][v];
          }
        __builtin_amdgcn_sched_barrier(0);
      }
      return;
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      int ld = ldc;
      asm volatile("" : "+s"(ld));
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int r = 8 * (v >> 2) + (v & 3);
          if (inside(i, j, r)) {
            if (atomic) unsafeAtomicAdd(at(i, j, r, ld), acc[i][j][v]);
            else *at(i, j, r, ld) = acc[i][j][v];
          }
        }
    }
  }
}

template <int BM, int BN, int WM, int WN, int MODE>
__device__ __forceinline__ void store_tile(const f32x16 (&acc)[BM / WM / 32][BN / WN / 32], void* __restrict__ Cv,
                                           int M, int N, int ldc, int tile_m, int tile_n, int wm, int wn,
                                           int fr, int fh, int atomic) {
  constexpr int NC = MODE == GEMM_SWIGLU_F16 ? BN / 2 : BN;
  if ((tile_m + 1) * BM <= M && (tile_n + 1) * NC <= N)
    store_tile_part<BM, BN, WM, WN, MODE, true>(acc, Cv, M, N, ldc, tile_m, tile_n, wm, wn, fr, fh, atomic);
  else
    store_tile_part<BM, BN, WM, WN, MODE, false>(acc, Cv, M, N, ldc, tile_m, tile_n, wm, wn, fr, fh, atomic);
}

constexpr int GEMM_LSE = 3;     // internal mode of the direct-to-LDS kernel: launch_gemm_lse

__device__ __forceinline__ void lse_pair_combine(float& m, float& s, float m2, float s2) {
  const float mn = fmaxf(m, m2);
  const float mu = mn == -INFINITY ? 0.f : mn;
  s = s * __expf(m - mu) + s2 * __expf(m2 - mu);
  m = mn;
}

// ---- direct-to-LDS variant ---------------------------------------------------
// Products of up to 32 rows, and 128 x 128 tiles.  Same tiling, but the K-slabs travel HBM -> LDS with buffer_load_dwordx4 ... lds
// (no register staging) into a ring of STAGES slab buffers, so STAGES-1 slabs
// of loads stay in flight per work-group.  One wavefront instruction moves a
// group of 8 tile rows x 128 B; lane s of the group lands at byte s*16 of the
// group's 1 KiB window, and fetches chunk (s&7) ^ (row&7) of row s>>3, an XOR
// swizzle that makes the later 16-byte fragment reads bank-conflict free.
// Requires K % 64 == 0.
constexpr int GROUP_BYTES = 1024 + 128;   // 8 rows x 128 B, + 128 B skew between groups

// One tile over the K slabs [kt0, kt1), through the ring in `lds` (STAGES * STAGE_BYTES bytes).
template <int BM, int BN, int WM, int WN, int STAGES, int MODE>
__device__ __forceinline__ void dma_tile(const f16* __restrict__ A, const WRows& W, void* __restrict__ Cv, int M,
                                         int N, int K, int ldc, int tile_m, int tile_n, int kt0, int kt1,
                                         int atomic, char* lds) {
  constexpr int NW = WM * WN;
  constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
  constexpr int GA = BM / 8, GB = BN / 8;              // row groups per slab
  constexpr int LPS = (GA + GB) / NW;                  // load instructions per wave per slab
  static_assert((GA + GB) % NW == 0 && GA % NW == 0, "row groups must divide over the waves");
  static_assert(MODE != GEMM_SWIGLU_F16 || (TN % 2 == 0), "SwiGLU needs gate+up in one wave tile");
  constexpr int STAGE_BYTES = (GA + GB) * GROUP_BYTES;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;

  // This wave's share of the row groups: GA/NW groups of A, then GB/NW of B.  The loads are buffer
  // loads (a scalar base, a lane's 32-bit offset and the slab's scalar offset), not global ones: these
  // are FLAT instructions to the compiler's wait insertion, which then waits for every LDS read in
  // flight wherever it has to wait for one.
  const TileRsrc<BM, BN, MODE> tile(A, W, M, N, K, tile_m, tile_n);
  // A lane holds its rows, of one resource, in residual adds (lane_rows) and, of A, where a wave has more than six groups: with
  // four scalar registers for each they do not fit.
  constexpr bool W_LANES = lane_rows<BM, BN, NW, MODE>(), A_LANES = LPS > 6 || W_LANES;
  __amdgpu_buffer_rsrc_t rsrc[LPS];
  int src[LPS], dst_off[LPS];
#pragma unroll
  for (int i = 0; i < LPS; ++i) {
    const bool is_a = i < GA / NW;
    const int gi = is_a ? wave * (GA / NW) + i : wave * (GB / NW) + (i - GA / NW);
    src[i] = (is_a ? A_LANES : W_LANES)
                 ? tile_lane_offset(lane, gi * 8, is_a ? min(M - tile_m * BM, BM) : min(N - tile_n * BN, BN), K * 2)
                 : group_lane_offset(lane, false, K * 2);
    if (is_a) rsrc[i] = A_LANES ? tile.a() : tile.a(gi * 8);
    else if (W_LANES) rsrc[i] = tile.w();
    else if (MODE == GEMM_SWIGLU_F16) rsrc[i] = tile.w((gi >> 3) * 32 + (gi & 3) * 8, (gi >> 2) & 1);
    else rsrc[i] = tile.w(gi * 8, false);
    dst_off[i] = ((is_a ? 0 : GA) + gi) * GROUP_BYTES;
    dma16(rsrc[i], src[i], kt0 * BK * 2, lds + dst_off[i]);     // the first slab: the later groups' addresses behind its loads
    __builtin_amdgcn_sched_barrier(0);
  }
  auto issue = [&](int stage, int k0) {
#pragma unroll
    for (int i = 0; i < LPS; ++i) dma16(rsrc[i], src[i], k0 * 2, lds + stage * STAGE_BYTES + dst_off[i]);
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  const int fr = lane & 31, fh = lane >> 5;
  // fragment addressing: tile row R -> group R>>3, slot (R&7)*8 + (chunk ^ (R&7))
  int a_base[TM], b_base[TN], koff[BK / 16];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int R = wm * (BM / WM) + i * 32 + fr;
    a_base[i] = (R >> 3) * GROUP_BYTES + (R & 7) * 128;
  }
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int R = wn * (BN / WN) + j * 32 + fr;
    b_base[j] = (GA + (R >> 3)) * GROUP_BYTES + (R & 7) * 128;
  }
#pragma unroll
  for (int kk = 0; kk < BK / 16; ++kk) koff[kk] = ((kk * 2 + fh) ^ (fr & 7)) << 4;

  // Fragment reads run one K-step ahead of the MFMAs that consume them, so the
  // LDS latency is covered by a full K-step of matrix work.
  struct Frags { f16x8 a[TM], b[TN]; };
  auto read_frags = [&](Frags& f, const char* base, int kk) {
#pragma unroll
    for (int i = 0; i < TM; ++i) f.a[i] = *reinterpret_cast<const f16x8*>(base + a_base[i] + koff[kk]);
#pragma unroll
    for (int j = 0; j < TN; ++j) f.b[j] = *reinterpret_cast<const f16x8*>(base + b_base[j] + koff[kk]);
  };
  auto mma = [&](const Frags& f) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(f.a[i], f.b[j], acc[i][j], 0, 0, 0);
  };
  // One slab's four K-steps are software-pipelined across the slab boundary: the barrier that frees
  // the stage stands in front of the last K-step's MFMAs, whose operands are in registers by then, and
  // the next slab's first fragments are read behind it, under those MFMAs.  In a 256 x 256 tile, whose slab is
  // 2,048 cycles of MFMAs and about as many of LDS traffic, a barrier at the slab's start and waits for all
  // fragments at once cost 5 - 7 % (gate/up of 8,192 rows 444 us, 423 in this order; of 2,048 rows 136 and 127).
  Frags f0, f1;
  const int k_last = (kt1 - 1) * BK;
  // prologue: STAGES slabs in flight (past the end: re-read the last slab, never consumed)
#pragma unroll
  for (int s = 1; s < STAGES; ++s) issue(s, min((kt0 + s) * BK, k_last));
  wait_vmcnt((STAGES - 1) * LPS);
  __builtin_amdgcn_s_barrier();
  read_frags(f0, lds, 0);
  for (int kt = kt0; kt < kt1; kt += STAGES) {
#pragma unroll
    for (int u = 0; u < STAGES; ++u) {
      if (kt + u < kt1) {
        // slab kt+u sits in stage u, its first K-step's fragments in (or on their way to) f0
        const char* base = lds + u * STAGE_BYTES;
        read_frags(f1, base, 1);
        __builtin_amdgcn_sched_barrier(0);
        mma(f0);
        __builtin_amdgcn_sched_barrier(0);
        read_frags(f0, base, 2);
        __builtin_amdgcn_sched_barrier(0);
        mma(f1);
        __builtin_amdgcn_sched_barrier(0);
        read_frags(f1, base, 3);
        __builtin_amdgcn_sched_barrier(0);
        mma(f0);
        __builtin_amdgcn_sched_barrier(0);
        wait_lgkmcnt0();      // this wave's reads of stage u are complete
        if (kt + u + 1 < kt1) {
          // and its part of slab kt+u+1 has landed (the STAGES-2 slabs requested after it may still be
          // in flight); plain barrier (no fence: a fence would drain every outstanding load): the
          // same holds for every wave
          wait_vmcnt((STAGES - 2) * LPS);
          __builtin_amdgcn_s_barrier();
          __builtin_amdgcn_sched_barrier(0);
          // (with two stages the wait above is for everything: nothing needs requesting past the end)
          if (STAGES > 2 || kt + u + STAGES < kt1) issue(u, min((kt + u + STAGES) * BK, k_last));
          read_frags(f0, lds + ((u + 1) % STAGES) * STAGE_BYTES, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
        mma(f1);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  // (all remaining in-flight loads target LDS only; the epilogue does not touch LDS)

  store_tile<BM, BN, WM, WN, MODE>(acc, Cv, M, N, ldc, tile_m, tile_n, wm, wn, fr, fh, atomic);
  // drain the loads that were requested past the end before the LDS is released
  wait_vmcnt(0);
}

// The first 14 words of the arguments (those before `late`) arrive in registers; nk_sps: K slabs | slabs per split << 16.
template <int BM, int BN, int WM, int WN, int STAGES, int MODE>
__global__ __launch_bounds__(WM * WN * 64) void gemm_dma_kernel(
    const f16* __restrict__ A, const f16* __restrict__ w0, const f16* __restrict__ w1, const f16* __restrict__ w2,
    int M, int N, uint32_t nk_sps, uint32_t map, int end0, int end1, GemmLate late) {
  __shared__ __attribute__((aligned(16))) char lds[STAGES * (BM / 8 + BN / 8) * GROUP_BYTES];
  constexpr int NC = MODE == GEMM_SWIGLU_F16 ? BN / 2 : BN;
  const int nk = nk_sps & 0xFFFF, sps = nk_sps >> 16;
  int tile_m, tile_n, split;
  if (!tile_of_block(map, (M + BM - 1) / BM, (N + NC - 1) / NC, nk, sps, tile_m, tile_n, split)) return;
  const int kt0 = split * sps, kt1 = min(nk, kt0 + sps);
  if (kt0 >= kt1) return;
  dma_tile<BM, BN, WM, WN, STAGES, MODE>(A, WRows{w0, w1, w2, end0, end1}, late.C, M, N, nk * BK, late.ldc, tile_m,
                                         tile_n, kt0, kt1, sps < nk, lds);
}

// ---- direct-to-LDS tiles on the 16x16x32 MFMA: the prefill sizes --------------
// What bounds a long run of the large products is the package's power: with operands drawn at random the
// 256 x 256 tile runs at 1.67 GHz, with zeros at 2.3 (407 against 294 us for 8,192 x 17,920 x 1,536 on the
// 32x32x16 MFMA).  Fed from registers alone, the 32x32x16 MFMA reaches 1.71 PFLOP/s on random operands
// and the 16x16x32 one, which adds into its accumulators half as often, 1.97; with the tile's
// fragment reads 1.58 and 1.78, and 1.86 in the order below (zeros: 2.45 all of them).
//
// Ring and swizzle are those of dma_tile, without the skew; the row groups of a slab are dealt to the waves in turn, so
// that a tile need not divide evenly over them.  A slab is two K-steps of 32; a wave's (BM/WM) x (BN/WN) part is
// TM x TN MFMAs of 16 x 16, taken in bands of two rows, column by column, there and back: of two MFMAs in a row
// one operand is always the same, and fewer bits toggle.
// Gate/up and scoring form W A^T: a lane then holds neighbouring columns of one row (lane & 15), which it stores as
// 16 bytes or folds by itself.  Stored and added float32 tiles are A W^T, column lane & 15 of four neighbouring
// rows in a lane: an atomic instruction then adds 64 contiguous bytes per row, not 16 (2.4 times the time for QKV
// of 301 rows in 3 K splits).
// Measured, 1.5B shape, inside scoring passes of 8,192 rows, against the 32x32x16 MFMA (two cards): gate/up 401 -> 370 us
// (1,218 TFLOP/s, matrix cores busy 70 % of the time at 1.75 GHz), down 206 -> 182 (with two barriers a slab, below),
// QKV 52 -> 49, O in 256 x 192 for 128 x 128 tiles 54 -> 46, output projection with its log-sum-exp 3,462 -> 3,035.  128 x 128 tiles of stored and added results gain nothing (their runs are short) and stay
// with dma_tile.
constexpr int WIDE_GROUP = 1024;        // 8 tile rows x 128 B: these reads have no bank conflicts without a skew
template <int TM, int TN>
struct Wide {
  f32x4 acc[TM][TN];
  struct Frags { f16x8 a[TM], b[TN]; };
  static constexpr int MFMAS = TM * TN, READS = TM + TN;
  // MFMA z of the walk -> its row and column: bands of two rows, column by column, there and back
  static constexpr int row(int z) {
    const int band = z / (2 * TN), h = TM - 2 * band < 2 ? 1 : 2, q = z - band * 2 * TN;
    return h == 1 ? 2 * band : 2 * band + ((q & 1) ^ ((q >> 1) & 1));
  }
  static constexpr int col(int z) {
    const int band = z / (2 * TN), h = TM - 2 * band < 2 ? 1 : 2, c = (z - band * 2 * TN) / h;
    return band & 1 ? TN - 1 - c : c;
  }
};

// Gate/up: which row of the weights LDS row `b` of a W tile holds, as feature of the tile and gate (0) or up (1).
//  * waves of whole 64-row groups (TN % 4 == 0): 32 gate rows, then the up rows of the same features, each as two MFMA
//    tiles whose rows 4g + v are the features 8g + v and 8g + 4 + v: a lane of group g ends up with eight
//    neighbouring features of a row;
//  * others: every MFMA tile of 16 rows is 8 gate rows, then the up rows of the same features; lanes trade
//    halves afterwards, and a tile can be any multiple of 8 features wide.
template <int TN>
__device__ __forceinline__ int wide_feature(int b) {
  if (TN % 4) return (b >> 4) * 8 + (b & 7);
  const int t = (b >> 4) & 1, r = b & 15;
  return (b >> 6) * 32 + 8 * (r >> 2) + 4 * t + (r & 3);
}
template <int TN>
__device__ __forceinline__ int wide_is_up(int b) { return TN % 4 ? (b >> 3) & 1 : (b >> 5) & 1; }

// ROWS, COLS: every row (column) of the tile lies inside the matrix; gate/up with COLS stores a lane's features at once,
// rows checked one by one where not all are inside.  Without that (every tile at the lower edge element by element)
// gate/up of 704 rows took 51.2 us, 46.4 with it; of 720 53.2 and 46.0, of 1,500 95.2 and 88.7, of 350 32.1 and 29.8.
template <int BM, int BN, int WM, int WN, int MODE, bool ROWS, bool COLS>
__device__ __forceinline__ void store_wide_part(const f32x4 (&acc)[BM / WM / 16][BN / WN / 16], void* __restrict__ Cv,
                                                int M, int N, int ldc, int tile_m, int tile_n, int wm, int wn,
                                                int fr, int fh, int atomic) {
  constexpr int TM = BM / WM / 16, TN = BN / WN / 16;
  const int m_wave = tile_m * BM + wm * (BM / WM);
  if constexpr (MODE == GEMM_SWIGLU_F16) {
    if constexpr (TN % 4 != 0) {
      // Gate in the lower half of the lanes, up in the upper: of two tiles, the lower lanes take the first and give their
      // part of the second for it, so that every lane holds four neighbouring features whole (a last odd tile: the
      // lower lanes do).
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; j += 2) {
          const bool two = j + 1 < TN;
          const int f = tile_n * (BN / 2) + (wn * TN + j + (two ? fh >> 1 : 0)) * 8 + (fh & 1) * 4, m = m_wave + i * 16 + fr;
          f16* p = reinterpret_cast<f16*>(Cv) + (int64_t)m * ldc + f;
          f16x4 y;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const float first = acc[i][j][v], second = acc[i][two ? j + 1 : j][v];
            const auto gu = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, first),
                                                             __builtin_bit_cast(uint32_t, second), false, false);
            const uint32_t gate = gu[0], up = gu[1];
            y[v] = f2h_sat(silu_f(__builtin_bit_cast(float, gate)) * __builtin_bit_cast(float, up));
          }
          if (two || fh < 2) {
            if (COLS) {
              if (ROWS || m < M) *reinterpret_cast<f16x4*>(p) = y;
            } else if (m < M) {
#pragma unroll
              for (int e = 0; e < 4; ++e)
                if (f + e < N) p[e] = y[e];
            }
          }
        }
      return;
    } else {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; j += 4) {
        const int f0 = tile_n * (BN / 2) + (wn * (BN / WN) + j * 16) / 2;
        f16* Cw = reinterpret_cast<f16*>(Cv) + (int64_t)(m_wave + i * 16) * ldc + f0;
        f16* p = Cw + fr * ldc + fh * 8;
        f16x8 y;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int v = 0; v < 4; ++v) y[4 * t + v] = f2h_sat(silu_f(acc[i][j + t][v]) * acc[i][j + 2 + t][v]);
        if (COLS) {
          if (ROWS || m_wave + i * 16 + fr < M) *reinterpret_cast<f16x8*>(p) = y;
        } else if (m_wave + i * 16 + fr < M) {
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (f0 + fh * 8 + e < N) p[e] = y[e];
        }
      }
    }
  } else {
    const int n_wave = tile_n * BN + wn * (BN / WN);
    float* Cw = reinterpret_cast<float*>(Cv) + (int64_t)m_wave * ldc + n_wave;
    // the opaque row stride keeps one batch's addresses from staying in registers for another
    auto stride = [&] { int ld = ldc; asm volatile("" : "+s"(ld)); return ld; };
    auto at = [&](int i, int j, int v, int ld) { return Cw + (int64_t)(i * 16 + v) * ld + j * 16 + (4 * fh * ld + fr); };
    auto inside = [&](int i, int j, int v) {
      return (ROWS && COLS) || (m_wave + i * 16 + 4 * fh + v < M && n_wave + j * 16 + fr < N);
    };
    if (MODE == GEMM_ADD_F32 && !atomic) {
      float old[2][TN][4];
      auto fetch = [&](int i) {
        const int ld = stride();
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int v = 0; v < 4; ++v) old[i & 1][j][v] = inside(i, j, v) ? *at(i, j, v, ld) : 0.f;
        __builtin_amdgcn_sched_barrier(0);
      };
      fetch(0);
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        if (i + 1 < TM) fetch(i + 1);
        const int ld = stride();
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            if (inside(i, j, v)) *at(i, j, v, ld) = old[i & 1][j][v] + acc[i][j][v];
        __builtin_amdgcn_sched_barrier(0);
      }
      return;
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int ld = stride();
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (inside(i, j, v)) {
            if (atomic) unsafeAtomicAdd(at(i, j, v, ld), acc[i][j][v]);
            else *at(i, j, v, ld) = acc[i][j][v];
          }
    }
  }
}

// Epilogue of launch_gemm_lse: nothing of the tile is stored but, per row, the (max, sum of exponentials) pair over
// the tile's columns and the value at the row's target column.  A lane holds 4 TN columns of one row per row tile,
// so a row is folded in the lane and over the four lanes that share it: its maximum first, then the
// exponentials once, against it.  The ring's LDS is reused (all its loads have landed and all waves are past their
// last read).
template <int BM, int BN, int WM, int WN>
__device__ __forceinline__ void store_wide_lse(const f32x4 (&acc)[BM / WM / 16][BN / WN / 16], char* lds,
                                               float2* __restrict__ part, int ld_rows, int M, int N, int tile_m,
                                               int tile_n, int wm, int wn, int fr, int fh, const GemmLse& lse) {
  constexpr int TM = BM / WM / 16, TN = BN / WN / 16, NT = WM * WN * 64;
  float2* red = reinterpret_cast<float2*>(lds);                       // [BM][WN]
  const int m0 = tile_m * BM;
  int tgt[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int m = m0 + wm * (BM / WM) + i * 16 + fr;
    tgt[i] = m < M ? lse.target[m] : -1;
  }
  wait_vmcnt(0);
  __syncthreads();                                                    // the ring is free
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int row = wm * (BM / WM) + i * 16 + fr;
    float z[TN][4], m = -INFINITY, sum = 0.f;
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int n = tile_n * BN + wn * (BN / WN) + j * 16 + fh * 4 + v;
        z[j][v] = n < N ? acc[i][j][v] * lse.inv_t : -INFINITY;
        if (n == tgt[i]) lse.target_z[m0 + row] = z[j][v];
        m = fmaxf(m, z[j][v]);
      }
    m = fmaxf(m, __shfl_xor(m, 16));
    m = fmaxf(m, __shfl_xor(m, 32));
    const float mu = m == -INFINITY ? 0.f : m;
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) sum += __expf(z[j][v] - mu);
    sum += __shfl_xor(sum, 16);
    sum += __shfl_xor(sum, 32);
    if (fh == 0) red[row * WN + wn] = float2{m, sum};
  }
  __syncthreads();
  for (int r = threadIdx.x; r < BM; r += NT) {
    if (m0 + r >= M) continue;
    float m = -INFINITY, sum = 0.f;
#pragma unroll
    for (int w = 0; w < WN; ++w) lse_pair_combine(m, sum, red[r * WN + w].x, red[r * WN + w].y);
    part[(int64_t)tile_n * ld_rows + m0 + r] = float2{m, sum};
  }
}

template <int BM, int BN, int WM, int WN, int STAGES, int MODE>
__device__ __forceinline__ void wide_tile(const f16* __restrict__ A, const WRows& W, void* __restrict__ Cv, int M,
                                          int N, int K, int ldc, int tile_m, int tile_n, int kt0, int kt1,
                                          int atomic, const GemmLse& lse, char* lds) {
  constexpr int NW = WM * WN;
  constexpr int TM = BM / WM / 16, TN = BN / WN / 16;
  constexpr int GA = BM / 8, GB = BN / 8;              // row groups per slab
  constexpr int LPS = (GA + GB + NW - 1) / NW;         // load instructions per slab of the first waves,
  constexpr int SHORT = (GA + GB) % NW;                // of which waves >= SHORT > 0 have one less
  static_assert(BM % (WM * 16) == 0 && BN % (WN * 16) == 0, "tile does not divide over the waves");
  constexpr int STAGE_BYTES = (GA + GB) * WIDE_GROUP;
  typedef Wide<TM, TN> WideT;
  constexpr bool TRANS = MODE == GEMM_SWIGLU_F16 || MODE == GEMM_LSE;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;

  // Groups of 8 rows are dealt to the waves in turn, A's first.
  const TileRsrc<BM, BN, MODE> tile(A, W, M, N, K, tile_m, tile_n);
  // Gate/up tiles of whole 64-row groups: the rows of a group are two runs of four features (wide_feature).
  constexpr bool SPREAD = MODE == GEMM_SWIGLU_F16 && TN % 4 == 0;
  __amdgpu_buffer_rsrc_t rsrc[LPS];
  int src[LPS], dst_off[LPS];
  auto issue1 = [&](int stage, int k0, int i) {
    if (SHORT == 0 || i < LPS - 1 || wave < SHORT)      // wave-uniform
      dma16(rsrc[i], src[i], k0 * 2, lds + stage * STAGE_BYTES + dst_off[i]);
  };
#pragma unroll
  for (int i = 0; i < LPS; ++i) {
    const int gi = i * NW + wave, b0 = (gi - GA) * 8;
    // all of the waves' i-th groups are A's, all W's, or (at one i, where they do not divide) this wave's decides
    const bool is_a = i * NW + NW <= GA || (i * NW < GA && gi < GA);
    if (lane_rows<BM, BN, NW, MODE>()) {
      rsrc[i] = is_a ? tile.a() : tile.w();
      src[i] = tile_lane_offset(lane, is_a ? gi * 8 : b0, is_a ? min(M - tile_m * BM, BM) : min(N - tile_n * BN, BN), K * 2);
    } else {
      if (is_a) rsrc[i] = tile.a(gi * 8);
      else if (MODE == GEMM_SWIGLU_F16) rsrc[i] = tile.w(wide_feature<TN>(b0), wide_is_up<TN>(b0));
      else rsrc[i] = tile.w(b0, false);
      src[i] = group_lane_offset(lane, SPREAD && !is_a, K * 2);
    }
    dst_off[i] = gi * WIDE_GROUP;
    issue1(0, kt0 * BK, i);          // the first slab: the later groups' addresses behind its loads
    __builtin_amdgcn_sched_barrier(0);
  }
  // waits until at most `slabs` slabs of this wave's loads are in flight
  auto wait_slabs = [&](auto slabs) {
    constexpr int S = decltype(slabs)::value;
    if (SHORT == 0 || S == 0 || wave < SHORT) wait_vmcnt(S * LPS);
    else wait_vmcnt(S * (LPS - 1));
  };

  WideT t;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) t.acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int fr = lane & 15, fh = lane >> 4;
  // fragment addresses inside a stage: tile row R -> group R>>3, slot (R&7)*8 + (chunk ^ (R&7)); the 16-row tiles of a
  // wave are two groups apart
  int a_at[2], b_at[2];
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) {
    const int ko = ((kk * 4 + fh) ^ (fr & 7)) << 4;
    const int ra = wm * (BM / WM) + fr, rb = wn * (BN / WN) + fr;
    a_at[kk] = (ra >> 3) * WIDE_GROUP + (ra & 7) * 128 + ko;
    b_at[kk] = (GA + (rb >> 3)) * WIDE_GROUP + (rb & 7) * 128 + ko;
  }
  typename WideT::Frags f0, f1;
  // the fragment reads of a K-step in the order in which the walk needs them: a0 a1 | b0 b1 .. | a2 a3 ..
  constexpr int A0 = TM < 2 ? TM : 2;
  auto read1 = [&](typename WideT::Frags& f, const char* base, int kk, int r) {
    const bool is_a = r < A0 || r >= A0 + TN;
    const int x = r < A0 ? r : (r < A0 + TN ? r - A0 : r - TN);
    if (is_a) f.a[x] = *reinterpret_cast<const f16x8*>(base + a_at[kk] + x * 2 * WIDE_GROUP);
    else f.b[x] = *reinterpret_cast<const f16x8*>(base + b_at[kk] + x * 2 * WIDE_GROUP);
  };
  auto mma1 = [&](const typename WideT::Frags& f, int i, int j) {
    t.acc[i][j] = TRANS ? __builtin_amdgcn_mfma_f32_16x16x32_f16(f.b[j], f.a[i], t.acc[i][j], 0, 0, 0)
                        : __builtin_amdgcn_mfma_f32_16x16x32_f16(f.a[i], f.b[j], t.acc[i][j], 0, 0, 0);
  };
  const int k_last = (kt1 - 1) * BK;
  // prologue: STAGES slabs in flight (past the end: re-read the last slab, never consumed)
#pragma unroll
  for (int s = 1; s < STAGES; ++s)
#pragma unroll
    for (int i = 0; i < LPS; ++i) issue1(s, min((kt0 + s) * BK, k_last), i);
  wait_slabs(std::integral_constant<int, STAGES - 1>{});
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int r = 0; r < WideT::READS; ++r) read1(f0, lds, 0, r);
  int cur = 0, kt = kt0;
  const std::true_type yes{};
  const std::false_type no{};
  // One slab: two K-steps of P pairs of MFMAs, everything else placed between them in a fixed order: fragment reads RPP a
  // pair, loads spread over the second K-step, or one every second pair (TWO).  LOAD: slab kt + STAGES exists; NEXT:
  // slab kt + 1 does.
  //   at FREE every wave has its last fragments of the stage (which the loads of slab kt + STAGES then refill),
  //   at LAND slab kt + 1 has landed for every wave, and its first fragments are read from there on.
  // Gate/up and scoring in 256 x 256 take both at one barrier between the K-steps.  Tried for gate/up of 8,192 rows, 365 us in
  // a long run: loads two, four or eight at a time 366, 373, 385; a barrier each, half a K-step apart, 382; a
  // ring of four or five stages of 32 along K, whose loads fetch half lines, 396 and 403.  The residual adds have
  // two, which leaves the loads between one and one and a half slabs of time instead of a half and one: down of 2,048
  // rows in 48 tiles 213 -> 195 us, of 8,192 229 -> 224, in the tiles of its choice 212 -> 186, in 192 x 256 tiles at
  // 6,768 rows 190 -> 157 inside a prefill.  So have tiles of 24 MFMAs a K-step everywhere (gate/up of 1,024 rows in
  // 192 x 256 75 -> 67 us, QKV of 4,096 40.3 -> 38.4) and stored 256 x 256 ones (QKV of 8,192 57.4 -> 55.7).
  constexpr int P = (WideT::MFMAS + 1) / 2;
  constexpr bool STORES = MODE == GEMM_ADD_F32 || MODE == GEMM_STORE_F32;
  constexpr bool TWO = (WideT::MFMAS == 24 || (STORES && WideT::MFMAS > 24)) && SHORT == 0 && STAGES == 2;
  constexpr int FREE = TWO ? P * 3 / 4 : P, LAND = TWO ? P + P / 2 : P;
  constexpr int RPP = TWO ? (WideT::READS * 2 + P - 1) / P : (WideT::READS * 4 + P * 3 - 1) / (P * 3);
  // pair behind which load d of a slab goes out, and how many go out ahead of LAND
  constexpr auto load_at = [](int d) { return TWO ? FREE + 2 * d : FREE + d * P / LPS; };
  constexpr int EARLY = TWO ? (LAND - FREE + 1) / 2 : 0;
  static_assert(load_at(LPS - 1) < 2 * P && (!TWO || (EARLY <= LPS && RPP * FREE >= WideT::READS && RPP * (2 * P - LAND) >= WideT::READS)),
                "a slab's loads and reads go out inside it");
  auto slab = [&](auto load, auto next) {
    constexpr bool LOAD = decltype(load)::value, NEXT = decltype(next)::value;
    const int nxt = cur + 1 == STAGES ? 0 : cur + 1, k_load = min((kt + STAGES) * BK, k_last);
    const char *base = lds + cur * STAGE_BYTES, *base_next = lds + nxt * STAGE_BYTES;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int z = 0; z < 2 * P; ++z) {
      const typename WideT::Frags& f = z < P ? f0 : f1;
      const int q = z < P ? z : z - P;
      // plain barriers: a fence would drain every outstanding load
      if (TWO && LOAD && z == FREE) {
        wait_lgkmcnt0();
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
      }
      if (NEXT && z == LAND) {
        if (!TWO) wait_lgkmcnt0();
        if constexpr (TWO) wait_vmcnt(LOAD ? EARLY : 0);
        else wait_slabs(std::integral_constant<int, STAGES - 2>{});
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
      }
      mma1(f, WideT::row(2 * q), WideT::col(2 * q));
      if (2 * q + 1 < WideT::MFMAS) mma1(f, WideT::row(2 * q + 1), WideT::col(2 * q + 1));
      if (LOAD) {
#pragma unroll
        for (int d = 0; d < LPS; ++d)
          if (load_at(d) == z) issue1(cur, k_load, d);
      }
#pragma unroll
      for (int r = 0; r < WideT::READS; ++r) {
        if (z < P && r / RPP == z) read1(f1, base, 1, r);
        if (NEXT && z >= LAND && r / RPP == z - LAND) read1(f0, base_next, 0, r);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    cur = nxt;
    ++kt;
  };
  // with two stages nothing is requested past the end
  const int n_load = kt1 - kt0 - (STAGES == 2 ? 2 : 1);
  for (int i = 0; i < n_load; ++i) slab(yes, yes);
  if (STAGES == 2 && kt1 - kt0 >= 2) slab(no, yes);
  slab(no, no);

  if constexpr (MODE == GEMM_LSE) {
    store_wide_lse<BM, BN, WM, WN>(t.acc, lds, reinterpret_cast<float2*>(Cv), ldc, M, N, tile_m, tile_n, wm, wn, fr, fh,
                                   lse);
  } else {
    constexpr int NC = MODE == GEMM_SWIGLU_F16 ? BN / 2 : BN;
    // gate/up: a lane's eight (four) features go out as 16 (8) bytes where rows start on 16 (8) bytes
    const bool whole = MODE != GEMM_SWIGLU_F16 ||
                       (TN % 4 ? ((ldc & 3) == 0 && ((uintptr_t)Cv & 7) == 0) : ((ldc & 7) == 0 && ((uintptr_t)Cv & 15) == 0));
    const bool rows = (tile_m + 1) * BM <= M, cols = whole && (tile_n + 1) * NC <= N;
    if (rows && cols)
      store_wide_part<BM, BN, WM, WN, MODE, true, true>(t.acc, Cv, M, N, ldc, tile_m, tile_n, wm, wn, fr, fh, atomic);
    else if (MODE == GEMM_SWIGLU_F16 && cols)   // rows below the matrix only
      store_wide_part<BM, BN, WM, WN, MODE, false, true>(t.acc, Cv, M, N, ldc, tile_m, tile_n, wm, wn, fr, fh, atomic);
    else
      store_wide_part<BM, BN, WM, WN, MODE, false, false>(t.acc, Cv, M, N, ldc, tile_m, tile_n, wm, wn, fr, fh, atomic);
  }
  // drain the loads that were requested past the end before the LDS is released
  wait_vmcnt(0);
}

template <int BM, int BN, int WM, int WN, int STAGES, int MODE>
__global__ __launch_bounds__(WM * WN * 64) void gemm_wide_kernel(
    const f16* __restrict__ A, const f16* __restrict__ w0, const f16* __restrict__ w1, const f16* __restrict__ w2,
    int M, int N, uint32_t nk_sps, uint32_t map, int end0, int end1, GemmLate late) {
  __shared__ __attribute__((aligned(16))) char lds[STAGES * (BM / 8 + BN / 8) * WIDE_GROUP];
  constexpr int NC = MODE == GEMM_SWIGLU_F16 ? BN / 2 : BN;
  const int nk = nk_sps & 0xFFFF, sps = nk_sps >> 16;
  int tile_m, tile_n, split;
  if (!tile_of_block(map, (M + BM - 1) / BM, (N + NC - 1) / NC, nk, sps, tile_m, tile_n, split)) return;
  const int kt0 = split * sps, kt1 = min(nk, kt0 + sps);
  if (kt0 >= kt1) return;
  wide_tile<BM, BN, WM, WN, STAGES, MODE>(A, WRows{w0, w1, w2, end0, end1}, late.C, M, N, nk * BK, late.ldc, tile_m,
                                          tile_n, kt0, kt1, sps < nk, late.lse, lds);
}

// Tiles, K split and grid of a launch.
struct Cut { int m_tiles, n_tiles, splits, sps; Grid grid; };
static Cut make_cut(int M, int N, int nk, int bm, int cols, int splits) {
  Cut c;
  c.n_tiles = (N + cols - 1) / cols;
  c.m_tiles = (M + bm - 1) / bm;
  splits = std::max(1, std::min(splits, nk));
  c.sps = (nk + splits - 1) / splits;
  c.splits = (nk + c.sps - 1) / c.sps;
  c.grid = make_grid(M, c.m_tiles, c.n_tiles, c.splits);
  return c;
}

template <int BM, int BN, int WM, int WN, int STAGES, int MODE>
hipError_t run_wide(hipStream_t s, const f16* A, const GemmW& W, void* C, int M, int N, int K, int ldc,
                    int splits, GemmLse lse = GemmLse{nullptr, nullptr, 1.f}) {
  if (K % BK || K / BK > 0xFFFF) return hipErrorInvalidValue;
  const Cut c = make_cut(M, N, K / BK, BM, MODE == GEMM_SWIGLU_F16 ? BN / 2 : BN, splits);
  gemm_wide_kernel<BM, BN, WM, WN, STAGES, MODE><<<c.grid.dim, WM * WN * 64, 0, s>>>(
      A, W.ptr[0], W.ptr[1], W.ptr[2], M, N, (uint32_t)(K / BK) | (uint32_t)c.sps << 16, c.grid.map, W.end[0], W.end[1],
      GemmLate{C, ldc, lse});
  return hipGetLastError();
}

// The same tiles with the last, partly filled round of work-groups evened out (one work-group
// per compute unit; the residual-add products only: the pieces of a cut tile add into C with float32
// atomics, a whole tile has one owner and adds without).
// XCD x takes the x-th eighth of the tiles (numbered row tile slowest: a block of neighbouring
// tiles, so its work-groups share A and W panels in one L2).  Its G work-groups take whole
// tiles G at a time; the `rem` tiles left over (rem < G) are cut along K: work-group j < rem walks
// the first S = ceil(rem nk / G) slabs of tile j, side by side with the others at the same K, and
// the work-groups j >= rem walk S-slab pieces of what is left of those tiles.  For shapes whose
// tile count leaves compute units idle in the last round (1,536 output columns: 192 tiles of
// 256 x 256 at 8,192 rows on 256 units).
template <int BM, int BN, int WM, int WN, int STAGES>
__global__ __launch_bounds__(WM * WN * 64) void gemm_even_kernel(const f16* __restrict__ A, const f16* __restrict__ w0,
                                                                     int M, int N, int K, int n_tiles, int tiles, int G,
                                                                     int ldc, float* __restrict__ C) {
  __shared__ __attribute__((aligned(16))) char lds[STAGES * (BM / 8 + BN / 8) * WIDE_GROUP];
  const int nk = K / BK;
  const WRows W{w0, nullptr, nullptr, N, N};
  const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
  const int t0 = (int)((int64_t)tiles * xcd / 8), t1 = (int)((int64_t)tiles * (xcd + 1) / 8);
  const int rounds = __builtin_amdgcn_readfirstlane((t1 - t0) / G), rem = t1 - t0 - rounds * G;
  const GemmLse none{nullptr, nullptr, 1.f};
  const int last = t0 + rounds * G;
  const int S = __builtin_amdgcn_readfirstlane((rem * nk + G - 1) / G);   // slabs per work-group in the last round, < nk
  const int tail = nk - S;                               // slabs left of each of the rem tiles
  int r = 0, u = (j - rem) * S;
  const int u_end = min((j - rem + 1) * S, rem * tail);
  // one call, so that the tile is compiled into the kernel once
  for (;;) {
    int tile, k0, k1;
    if (r < rounds) {
      tile = t0 + r * G + j;
      k0 = 0;
      k1 = nk;
    } else if (j < rem) {
      if (r > rounds) break;
      tile = last + j;
      k0 = 0;
      k1 = S;
    } else {
      if (u >= u_end) break;
      tile = last + u / tail;
      k0 = S + u % tail;
      k1 = min(nk, k0 + (u_end - u));
      u += k1 - k0;
    }
    ++r;
    // scalars, as in tile_of_block
    auto scalar = [](int x) { return __builtin_amdgcn_readfirstlane(x); };
    tile = scalar(tile), k0 = scalar(k0), k1 = scalar(k1);
    const int tile_m = scalar(tile / n_tiles);
    wide_tile<BM, BN, WM, WN, STAGES, GEMM_ADD_F32>(A, W, C, M, N, K, ldc, tile_m, tile - tile_m * n_tiles, k0,
                                                           k1, k1 - k0 < nk, none, lds);
    __syncthreads();            // every wave is done with the ring before the next piece refills it
  }
}

template <int BM, int BN, int WM, int WN, int STAGES>
hipError_t run_even(hipStream_t s, const f16* A, const GemmW& W, float* C, int M, int N, int K, int ldc,
                        int n_groups) {
  if (K % BK || n_groups <= 0 || n_groups % 8) return hipErrorInvalidValue;
  const int n_tiles = (N + BN - 1) / BN, m_tiles = (M + BM - 1) / BM;
  gemm_even_kernel<BM, BN, WM, WN, STAGES><<<n_groups, WM * WN * 64, 0, s>>>(A, W.ptr[0], M, N, K, n_tiles,
                                                                               n_tiles * m_tiles, n_groups / 8, ldc, C);
  return hipGetLastError();
}

template <int BM, int BN, int WM, int WN, int STAGES, int MODE>
hipError_t run_dma(hipStream_t s, const f16* A, const GemmW& W, void* C, int M, int N, int K, int ldc,
                   int splits) {
  if (K % BK || K / BK > 0xFFFF) return hipErrorInvalidValue;
  const Cut c = make_cut(M, N, K / BK, BM, MODE == GEMM_SWIGLU_F16 ? BN / 2 : BN, splits);
  gemm_dma_kernel<BM, BN, WM, WN, STAGES, MODE><<<c.grid.dim, WM * WN * 64, 0, s>>>(
      A, W.ptr[0], W.ptr[1], W.ptr[2], M, N, (uint32_t)(K / BK) | (uint32_t)c.sps << 16, c.grid.map, W.end[0], W.end[1],
      GemmLate{C, ldc, GemmLse{}});
  return hipGetLastError();
}

template <int BM, int BN, int WM, int WN, int MODE>
hipError_t run(hipStream_t s, const f16* A, const GemmW& W, void* C, int M, int N, int K, int ldc,
               int splits) {
  const Cut c = make_cut(M, N, (K + BK - 1) / BK, BM, MODE == GEMM_SWIGLU_F16 ? BN / 2 : BN, splits);
  const int atomic = c.splits > 1 || MODE == GEMM_ADD_F32;
  if (K % BK)
    gemm_kernel<BM, BN, WM, WN, MODE, true><<<c.grid.dim, WM * WN * 64, 0, s>>>(A, M, N, K, c.grid.map, c.sps,
                                                                                ldc, C, atomic, W);
  else
    gemm_kernel<BM, BN, WM, WN, MODE, false><<<c.grid.dim, WM * WN * 64, 0, s>>>(A, M, N, K, c.grid.map, c.sps,
                                                                                 ldc, C, atomic, W);
  return hipGetLastError();
}

// Prices of tiles and K splits above 256 rows.  No one rule holds from 257 to 8,192 rows: what decides is how the
// last round of work-groups fills 256 compute units, and below about 1,000 rows whether there is a
// round at all (36 tiles of 128 x 128 for the down projection of a 301-token prompt: 58 us with 2
// splits, 22 with 6).  So every candidate is priced in microseconds: a fixed part, the K slabs one
// compute unit walks (slower the fuller the chip: clocks and L2 are shared), and the adds into C per
// million elements (with atomics for every split, or read and written once).  Constants: fitted to sweeps of
// 8 products (1.5B and 7B shape) x 18 - 50 row counts from 257 to 8,192 x tiles x splits; over the last one (10,458 times
// on one card) the choice, small tiles, evened launch and whole tiles included, is 0.6 % from the best of these tiles on average.
// Tiles of 160 columns, gate/up's, would be better at some row counts (O 7B of 1,700 rows 58 us in 160 x 160, 65 chosen).
// Farthest off else are down of the 7B shape at 1,345 - 1,408 rows (212 us for 183 with a split that adds with atomics, see
// prefill_choose), its O at 317 - 320 (24.1 for 21.5), and QKV of 3,969 - 4,096 rows (37.4 for 34.7).
struct PrefillTile {
  int cfg, bm, bn, per_cu;        // work-groups of this tile a compute unit holds
  float fixed, slab_few, slab_all, add_split, add_whole;
};
constexpr PrefillTile TILE_256x192 = {26, 256, 192, 1, 12.54f, 0.715f, 1.157f, 1.758f, 0.846f};
constexpr PrefillTile prefill_tiles[] = {
    {19, 256, 256, 1, 15.0f, 0.878f, 1.549f, 1.691f, 0.911f}, {28, 192, 256, 1, 11.44f, 0.715f, 1.157f, 1.80f, 0.982f},
    TILE_256x192,                                             {27, 128, 192, 1, 8.62f, 0.471f, 0.711f, 1.682f, 0.968f},
    {21, 128, 128, 1, 7.57f, 0.368f, 0.58f, 1.297f, 0.599f},  {20, 128, 128, 2, 10.2f, 0.49f, 1.02f, 1.252f, 0.532f},
};
static float prefill_us(const PrefillTile& t, int M, int N, int K, int mode, int splits) {
  const int cols = mode == GEMM_SWIGLU_F16 ? t.bn / 2 : t.bn, nk = K / BK;
  const float melem = (float)M * (float)N * 1e-6f;
  const float n_wg = (float)((N + cols - 1) / cols) * (float)((M + t.bm - 1) / t.bm);
  const int sps = (nk + splits - 1) / splits, parts = (nk + sps - 1) / sps;
  const float load = n_wg * (float)parts / (256.0f * t.per_cu), rounds = ceilf(load);
  float us = t.fixed * (1.0f + 0.4f * (rounds - 1.0f)) +
             (float)sps * rounds * (t.slab_few + (t.slab_all - t.slab_few) * load / rounds);
  if (parts > 1) us += t.add_split * melem * (float)parts;
  else if (mode == GEMM_ADD_F32) us += t.add_whole * melem;
  return us;
}
// Residual adds with a long K: tiles of 256 x 256 with the last round evened out along K.  Below a round every tile is cut,
// into about 256 / tiles parts that all add.
constexpr int EVENED_MIN_K = 4096;
static float evened_us(int M, int N, int K) {
  const float tiles = (float)((N + 255) / 256) * (float)((M + 255) / 256);
  return 45.0f + tiles * (float)(K / BK) / 256.0f * 1.46f +
         1.87f * (float)M * (float)N * 1e-6f * std::max(1.0f, 256.0f / tiles);
}
// Configuration 24 takes tiles of 192 columns instead where these fill every round of 256 compute units, so that
// nothing is left to cut, and are the cheaper ones: 8,192 x 1,536 x 8,960 (256 tiles) 186 us, 219 in whole tiles of 256
// columns.
static bool evened_192(int M, int N, int K) {
  return K >= EVENED_MIN_K && (int64_t)((N + 191) / 192) * ((M + 255) / 256) % 256 == 0 &&
         prefill_us(TILE_256x192, M, N, K, GEMM_ADD_F32, 1) <= evened_us(M, N, K);
}

// Gate/up, and the narrow products of a decode step.  A launch of one round of work-groups lives on what a
// compute unit takes in: a stream of weights that come from memory stays at about 45 GB/s per compute unit, however
// many bytes are in flight (32, 64 or 128 KB: the same), and rows of A that come from L2 queue behind them, so
// that (rows + columns) of a tile times 2 K bytes at 41 GB/s is its time, where all weights at 5.9 TB/s do not take longer.
// So tiles are chosen whose work-groups come as close to 256 as the width allows (8,960 features: 224 of 40,
// 125 x 2 of 72; 18,944: 237 of 80), with no more rows than the launch has.  Measured against tiles of
// 64 features, 1.5B shape: 15.1 -> 13.3 us at 24 rows, 18.9 -> 15.4 at 64, 20.4 -> 17.4 at 88, 34.7 -> 24.7 at 256,
// 32.8 -> 27.7 at 300; 7B shape: 58.5 -> 48.4 at 24, 66 -> 49 at 64, 80 -> 57 at 128, 133 -> 93 at 256.  Over 65 + 30 row
// counts from 257 to 8,192 (1.5B and 7B shape) the choice is 0.5 % from the best of 14 tiles on average, 6 % at most.
struct StreamTile { int cfg, bm, bn; };
constexpr StreamTile stream_tiles[] = {{36, 32, 80},   {37, 64, 80},   {29, 96, 80},   {38, 128, 80},  {39, 128, 144},
                                       {30, 64, 160},  {31, 96, 160},  {32, 128, 160}, {33, 160, 160}, {34, 192, 160}};
static float stream_us(const StreamTile& t, int M, int N, int K) {
  const float load = (float)((2 * N + t.bn - 1) / t.bn) * (float)((M + t.bm - 1) / t.bm) / 256.0f;
  const float rounds = std::max(1.0f, 0.5f * (load + ceilf(load)));      // a last round that is partly filled
  return 4.5f + std::max(rounds * (float)(t.bm + t.bn) * (float)K * (2e-3f / 41.0f), (float)N * (float)K * (4e-6f / 5.9f));
}
// The tiles of a prefill pass by prefill_us, fitted to the same sweep.  128 x 128, two to a compute unit, where row tiles of
// 192 and 256 end badly: 769 - 896 rows of the 1.5B shape 64 us in 192 x 256, 59 in 128 x 128.
constexpr PrefillTile gateup_tiles[] = {
    {19, 256, 256, 1, 11.36f, 1.101f, 1.541f, 0.f, 0.f}, {28, 192, 256, 1, 9.03f, 0.833f, 1.17f, 0.f, 0.f},
    {26, 256, 192, 1, 9.83f, 0.724f, 1.211f, 0.f, 0.f},  {27, 128, 192, 1, 9.73f, 0.837f, 0.687f, 0.f, 0.f},
    {20, 128, 128, 2, 7.50f, 0.733f, 1.073f, 0.f, 0.f},
};
static int gateup_choose(int M, int N, int K) {
  int cfg = 0;
  float best = 1e30f;
  for (const StreamTile& t : stream_tiles) {
    const float us = stream_us(t, M, N, K);
    if (us < best) { best = us; cfg = t.cfg; }
  }
  if (M > DECODE_ROWS)
    for (const PrefillTile& t : gateup_tiles) {
      const float us = prefill_us(t, M, N, K, GEMM_SWIGLU_F16, 1);
      if (us < best) { best = us; cfg = t.cfg; }
    }
  return cfg;
}
// QKV, O and down projection at up to 256 rows: tile and K split by the same two streams (added as fourth powers: neither
// hides the other wholly) and the adds of all splits, fitted to sweeps of 6 products x 35 row counts; over the last one the
// choice is 0.3 % (down 7B) to 7 % (O of the 1.5B shape: half a microsecond) from the best measured.  64 x 96
// for 64 x 128 tiles: down of 88 rows 13.5 -> 11.9 us, of 256 rows 22.8 -> 20.6, O of the 7B shape at 128 rows 15.5 -> 13.6.
struct NarrowTile {
  int cfg, bm, bn;
  float fixed, cu_gbs, add;            // us, GB/s per compute unit, us per million elements added
};
constexpr NarrowTile narrow_tiles[] = {{22, 32, 128, 4.28f, 67.4f, 2.48f}, {23, 64, 96, 3.47f, 64.9f, 2.50f},
                                       {35, 128, 96, 4.50f, 70.0f, 3.05f}, {21, 128, 128, 2.69f, 58.2f, 3.19f}};
// Above 256 rows the tiles of one round of work-groups compete with those of a prefill pass: O of 301 rows 11.1 -> 9.7 us,
// of 768 19.8 -> 13.1, of 1,024 20.2 -> 13.7; QKV of 301 12.6 -> 10.5, of 512 18.5 -> 12.5, of 768 19.0 -> 13.8; down
// of 257 22.1 -> 19.8.  Over 114 (product, rows) from 257 to 1,024 the choice is 0.4 % from the best measured.
constexpr NarrowTile one_round_tiles[] = {{23, 64, 96, 3.68f, 64.0f, 2.60f}, {29, 96, 80, 3.90f, 67.0f, 2.71f},
                                          {35, 128, 96, 3.31f, 64.8f, 3.11f}};
static float narrow_load(const NarrowTile& t, int M, int N, int K, int splits) {
  const int nk = K / BK, sps = (nk + splits - 1) / splits, parts = (nk + sps - 1) / sps;
  return (float)((N + t.bn - 1) / t.bn) * (float)((M + t.bm - 1) / t.bm) * (float)parts / 256.0f;
}
static float narrow_us(const NarrowTile& t, int M, int N, int K, int splits) {
  const int nk = K / BK, sps = (nk + splits - 1) / splits, parts = (nk + sps - 1) / sps;
  const float load = narrow_load(t, M, N, K, splits), rounds = std::max(1.0f, 0.5f * (load + ceilf(load)));
  const float cu = rounds * (float)sps * (float)(t.bm + t.bn) * (0.128f / t.cu_gbs);
  const float mem = (float)N * (float)K * (2e-6f / 7.0f);
  return t.fixed + sqrtf(sqrtf(cu * cu * cu * cu + mem * mem * mem * mem)) +
         t.add * (float)M * (float)N * 1e-6f * (parts > 1 ? (float)parts : 0.4f);
}

// A number stands for one tile in every mode that it serves (26 and 27 deal it to the waves differently for gate/up).
// No choice returns 1, 3 and 5 to 18: areal_op_gemm serves them, as yardsticks for sweeps.
template <int MODE>
hipError_t dispatch(hipStream_t s, int cfg, const f16* A, const GemmW& W, void* C, int M, int N, int K,
                    int ldc, int splits) {
  switch (cfg) {
    case 0: return run<128, 128, 2, 2, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 1: return run<256, 128, 4, 2, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 2: return run<64, 128, 1, 2, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 3: return run<256, 64, 4, 1, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 4: return run<32, 128, 1, 2, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 5: return run<128, 64, 2, 1, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 6: return run<64, 64, 1, 1, MODE>(s, A, W, C, M, N, K, ldc, splits);
    // direct-to-LDS ring (K % 64 == 0)
    case 7: return run_dma<128, 128, 2, 2, 3, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 8: return run_dma<128, 128, 2, 2, 2, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 9: return run_dma<256, 128, 4, 2, 2, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 10: return run_dma<64, 128, 1, 2, 3, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 11: return run_dma<64, 128, 1, 2, 4, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 12: return run_dma<32, 128, 1, 2, 4, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 13: return run_dma<128, 64, 2, 1, 4, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 14: return run_dma<256, 64, 4, 1, 3, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 15: return run_dma<128, 128, 2, 2, 4, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 16: return run_dma<256, 256, 2, 2, 2, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 17: return run_dma<256, 128, 2, 2, 2, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 18: return run_wide<256, 256, 4, 2, 2, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 19: return run_wide<256, 256, 2, 4, 2, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 20: return run_dma<128, 128, 4, 2, 2, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 21: return run_dma<128, 128, 4, 2, 3, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 22:   // one 32-column panel per wave: no room for a gate/up pair
      if constexpr (MODE != GEMM_SWIGLU_F16) return run_dma<32, 128, 1, 4, 4, MODE>(s, A, W, C, M, N, K, ldc, splits);
      else return hipErrorInvalidValue;
    case 23:   // narrow products of a decode step
      if constexpr (MODE != GEMM_SWIGLU_F16) return run_wide<64, 96, 2, 2, 4, MODE>(s, A, W, C, M, N, K, ldc, splits);
      else return hipErrorInvalidValue;
    case 24:   // residual adds with the last round of work-groups evened out along K
      if constexpr (MODE == GEMM_ADD_F32) {
        if (evened_192(M, N, K))
          return run_even<256, 192, 4, 2, 2>(s, A, W, reinterpret_cast<float*>(C), M, N, K, ldc, 256);
        return run_even<256, 256, 2, 4, 2>(s, A, W, reinterpret_cast<float*>(C), M, N, K, ldc, 256);
      } else return hipErrorInvalidValue;
    case 25:   // 64-column tiles, one 32-column panel per wave (twice the work-groups of 22)
      if constexpr (MODE != GEMM_SWIGLU_F16) return run_dma<32, 64, 1, 2, 4, MODE>(s, A, W, C, M, N, K, ldc, splits);
      else return hipErrorInvalidValue;
    // 192-row and 192-column tiles: other shapes of the last round (1,536 columns = 8 x 192).  Gate/up
    // needs whole pairs of 32-column panels in a wave: there every wave takes all six panels.
    case 26:
      if constexpr (MODE != GEMM_SWIGLU_F16) return run_wide<256, 192, 4, 2, 2, MODE>(s, A, W, C, M, N, K, ldc, splits);
      else return run_wide<256, 192, 8, 1, 2, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 27:
      if constexpr (MODE != GEMM_SWIGLU_F16) return run_wide<128, 192, 4, 2, 3, MODE>(s, A, W, C, M, N, K, ldc, splits);
      else return run_wide<128, 192, 4, 1, 3, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 28: return run_wide<192, 256, 2, 4, 2, MODE>(s, A, W, C, M, N, K, ldc, splits);
    // gate/up by StreamTile; 29 and 35 also stored and added by NarrowTile, 30 to 34 the output projection
    case 29: return run_wide<96, 80, 6, 1, 4, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 30: return run_wide<64, 160, 4, 1, 4, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 31: return run_wide<96, 160, 6, 1, 4, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 32: return run_wide<128, 160, 4, 1, 4, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 33: return run_wide<160, 160, 5, 1, 3, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 34: return run_wide<192, 160, 6, 1, 3, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 35: return run_wide<128, 96, 4, 2, 4, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 36: return run_wide<32, 80, 2, 1, 4, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 37: return run_wide<64, 80, 4, 1, 4, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 38: return run_wide<128, 80, 8, 1, 4, MODE>(s, A, W, C, M, N, K, ldc, splits);
    case 39: return run_wide<128, 144, 8, 1, 4, MODE>(s, A, W, C, M, N, K, ldc, splits);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

int gemm_num_configs() { return 40; }

// Tile configuration and K split for a product of this shape: the cheapest by prices fitted to
// sweeps over the configurations on the MI355X at the decoder's shapes, a few rules by row count
// beside them (`cfg` / `splits` >= 0 in launch_gemm_cfg override them).
// Upper limit of the K split (tuning knob for sweeps: AREAL_GEMM_MAX_SPLITS, read once).
static int max_splits() {
  static const int v = [] {
    const char* e = getenv("AREAL_GEMM_MAX_SPLITS");
    const int x = e ? atoi(e) : 0;
    return (x >= 1 && x <= 64) ? x : 12;
  }();
  return v;
}

// Ragged K: the largest K split that keeps every XCD at one round of work-groups (32 CUs, one
// work-group each): units of (column tile, split) go to the XCDs round-robin, each with
// m_tiles work-groups.  Each split keeps at least 3 slabs.  Beyond 8 (12 with a single
// row tile) the atomic adds outweigh the shorter K walk.
static int split_for(int M, int bm, int n_tiles, int nk) {
  const int m_tiles = (M + bm - 1) / bm;
  const int cap = std::min(std::max(1, nk / 3), std::min(m_tiles == 1 ? 12 : 8, max_splits()));
  static const int steps[] = {12, 8, 6, 4, 3, 2, 1};
  for (int cand : steps) {
    if (cand > cap) continue;
    if (((n_tiles * cand + 7) / 8) * m_tiles <= 32 || cand == 1) return cand;
  }
  return 1;
}

// Tile and K split above 256 rows: the cheapest by prefill_us, narrow_us and evened_us, where a cut along K has to earn
// what it takes away.  Its parts add into C with float32 atomics in no fixed order, so that a pass no longer repeats
// itself bit for bit; whole tiles all give the same bits, whatever their size.  Where tiles of 128 x 128 leave a
// quarter of the compute units without work a cut is taken whenever it is the cheaper one (down of 1,024 rows 46 us,
// 58 in the best whole tiles).  Beyond that a split has to save a tenth by price, and so has the evened launch below a
// whole round of tiles, where it cuts them all; from a round on, a thirty-second.  Down of 2,304 rows 86 us split, 88
// whole; of 3,500 113 and 106; of 4,272 138 and 144; QKV of the 7B shape at 1,285 rows 70 and 59, its O at 1,700 71
// and 64, down at 1,600 211 and 222, at 4,000 507 and 483, at 6,500 766 and 755; but down at 1,500 rows 195 and 219, at
// 2,048 274 and 310, at 8,192 921 and 975.
static void prefill_choose(int M, int N, int K, GemmMode mode, int* cfg, int* splits) {
  static const int steps[] = {1, 2, 3, 4, 6, 8, 12};
  constexpr float SPLIT_SAVES = 1.0f - 1.0f / 10.0f, EVENED_SAVES = 1.0f - 1.0f / 32.0f;
  const int nk = K / BK;
  const bool filled = (int64_t)((N + 127) / 128) * ((M + 127) / 128) > 192;
  float whole = 1e30f, split = 1e30f;
  int split_cfg = -1, parts = 1;
  auto take = [&](int c, int sp, float us) {
    if (sp == 1 && us < whole) { whole = us; *cfg = c; }
    if (sp > 1 && us < split) { split = us; split_cfg = c; parts = sp; }
  };
  for (const PrefillTile& t : prefill_tiles)
    for (int sp : steps) {
      if (sp > 1 && (sp > max_splits() || 3 * sp > nk)) break;
      take(t.cfg, sp, prefill_us(t, M, N, K, mode, sp));
    }
  for (const NarrowTile& t : one_round_tiles)
    for (int sp : steps) {
      if ((sp > 1 && (sp > max_splits() || 3 * sp > nk)) || narrow_load(t, M, N, K, sp) > 1.0f) break;
      take(t.cfg, sp, narrow_us(t, M, N, K, sp));
    }
  float best = whole;
  *splits = 1;
  if (split < (filled ? whole * SPLIT_SAVES : whole)) {
    best = split;
    *cfg = split_cfg;
    *splits = parts;
  }
  const int64_t evened_tiles = (int64_t)((N + 255) / 256) * ((M + 255) / 256);
  if (mode == GEMM_ADD_F32 && K >= EVENED_MIN_K && evened_tiles >= 96) {
    // Configuration 24, by the price of the tiles that it launches: of 192 columns, the work of configuration 26
    // without a split; of 256, whose cut tiles add with atomics: not under a limit of one split.
    const float us = evened_us(M, N, K);
    if (evened_192(M, N, K) ? *cfg == 26 && *splits == 1
                            : us < best && us < whole * (evened_tiles < 256 ? SPLIT_SAVES : EVENED_SAVES) &&
                                  max_splits() > 1) {
      *cfg = 24;
      *splits = 1;
    }
  }
}

void gemm_choose(int M, int N, int K, GemmMode mode, int* cfg, int* splits) {
  const bool wide_out = (N + 127) / 128 >= 100;
  *splits = 1;
  if (K % BK) {                        // register-staged path (ragged K)
    *cfg = M <= 32 ? 4 : (M <= 64 ? 2 : 0);
    const int bm = M <= 32 ? 32 : (M <= 64 ? 64 : 128);
    if (mode != GEMM_SWIGLU_F16 && M <= DECODE_ROWS) *splits = split_for(M, bm, (N + 127) / 128, (K + BK - 1) / BK);
  } else if (mode == GEMM_SWIGLU_F16) {
    *cfg = gateup_choose(M, N, K);
  } else if (M > DECODE_ROWS) {        // prefill: MFMA-bound, large tiles
    prefill_choose(M, N, K, mode, cfg, splits);
  } else if (wide_out) {
    // output projection: one row tile where the rows fit one (152k columns, 160 rows: 135 us in tiles of 160 x 160,
    // 155 in 256 x 256)
    *cfg = M <= 32 ? 22 : (M <= 64 ? 30 : (M <= 96 ? 31 : (M <= 128 ? 21 : (M <= 160 ? 33 : (M <= 192 ? 34 : 19)))));
  } else if (mode == GEMM_ADD_F32 && M <= 32 && K >= 4096 && N <= 2048) {
    // down projection at few rows: 64-column tiles, 8 splits = twice the work-groups of the
    // 128-column tile at 12 splits (8.1 / 8.9 us against 8.7 / 9.8 at 16 / 32 rows of the 1.5B shape)
    *cfg = 25;
    *splits = std::min(8, max_splits());
  } else {
    static const int steps[] = {1, 2, 3, 4, 6, 8, 12};
    float best = 1e30f;
    *cfg = 22;
    for (const NarrowTile& t : narrow_tiles)
      for (int sp : steps) {
        // one row tile of 32 up to 32 rows: inside a decode step of 24 rows QKV takes 5.2 us with it, 5.9 in 64 rows
        if ((sp > 1 && (sp > max_splits() || 3 * sp > K / BK)) || t.bm > (M <= 32 ? 32 : 2 * M)) continue;
        const float us = narrow_us(t, M, N, K, sp);
        if (us < best) { best = us; *cfg = t.cfg; *splits = sp; }
      }
  }
}

__global__ __launch_bounds__(256) void clear_rows_kernel(float* __restrict__ C, int N, int ldc) {
  for (int n = threadIdx.x; n < N; n += 256) C[(int64_t)blockIdx.x * ldc + n] = 0.f;
}

// The forms a configuration is made for.  Asked before a shape is passed on to other tiles, so that what it does not
// serve is refused at every shape.
static bool config_serves(int cfg, GemmMode mode, int K) {
  if (cfg >= gemm_num_configs() || (cfg >= 7 && K % BK)) return false;
  if (mode == GEMM_SWIGLU_F16) return cfg != 22 && cfg != 23 && cfg != 24 && cfg != 25;
  return cfg != 24 || mode == GEMM_ADD_F32;
}

hipError_t launch_gemm_cfg(hipStream_t s, const f16* A, GemmW W, void* C, int M, int N, int K, int ldc,
                           GemmMode mode, int cfg, int splits, bool overwrite) {
  if (M <= 0 || N <= 0 || K <= 0 || K % 8 || ldc < N || !A || !C || !W.ptr[0]) return hipErrorInvalidValue;
  if (((uintptr_t)A | (uintptr_t)W.ptr[0] | (uintptr_t)W.ptr[1] | (uintptr_t)W.ptr[2]) & 15)
    return hipErrorInvalidValue;
  int c0, s0;
  gemm_choose(M, N, K, mode, &c0, &s0);
  if (cfg < 0) cfg = c0;
  if (!config_serves(cfg, mode, K)) return hipErrorInvalidValue;
  const bool clear = overwrite && splits < 0 && s0 > 1 && M > DECODE_ROWS;
  if (splits < 0) splits = s0;
  // the direct-to-LDS tiles load W in groups of 8 rows that lie in one segment, with 32-bit offsets
  // inside a row tile: other shapes go through the register-staged tiles
  const bool odd_segments = mode == GEMM_STORE_F32 && W.end[0] < N && ((W.end[0] | W.end[1]) & 7) != 0;
  if (cfg >= 7 && (odd_segments || K >= (1 << 22))) cfg = M <= 32 ? 4 : (M <= 64 ? 2 : 0);
  switch (mode) {
    case GEMM_STORE_F32:
      if (W.end[0] > N || (W.end[0] < N && (!W.ptr[1] || W.end[1] > N)) ||
          (W.end[0] < N && W.end[1] < N && (!W.ptr[2] || W.end[2] != N)))
        return hipErrorInvalidValue;
      if (clear) clear_rows_kernel<<<M, 256, 0, s>>>(reinterpret_cast<float*>(C), N, ldc);
      return dispatch<GEMM_STORE_F32>(s, cfg, A, W, C, M, N, K, ldc, splits);
    case GEMM_ADD_F32:
      if (W.end[0] != N) return hipErrorInvalidValue;
      return dispatch<GEMM_ADD_F32>(s, cfg, A, W, C, M, N, K, ldc, splits);
    case GEMM_SWIGLU_F16:
      if (!W.ptr[1]) return hipErrorInvalidValue;
      // the direct-to-LDS tiles store pairs of features as words: rows that do not start on one, or
      // end inside one, go through the register-staged tiles, which store single elements
      if (cfg >= 7 && ((N | ldc) & 1 || (uintptr_t)C & 3)) cfg = M <= 32 ? 4 : (M <= 64 ? 2 : 0);
      return dispatch<GEMM_SWIGLU_F16>(s, cfg, A, W, C, M, N, K, ldc, 1);
  }
  return hipErrorInvalidValue;
}

// Column tiles of launch_gemm_lse: 256 wide above 256 rows (the 256 x 256 tile), else 128.
int gemm_lse_tiles(int M, int N) { return M > 256 ? (N + 255) / 256 : (N + 127) / 128; }

hipError_t launch_gemm_lse(hipStream_t s, const f16* A, GemmW W, int M, int N, int K, void* part, int ld_rows,
                           GemmLse lse) {
  if (M <= 0 || N <= 0 || K <= 0 || K % BK || ld_rows < M || !A || !part || !W.ptr[0] || W.end[0] != N ||
      !lse.target || !lse.target_z || !(lse.inv_t > 0.f) ||
      (((uintptr_t)A | (uintptr_t)W.ptr[0]) & 15) || ((uintptr_t)part & 7))
    return hipErrorInvalidValue;
  if (M > 256) return run_wide<256, 256, 2, 4, 2, GEMM_LSE>(s, A, W, part, M, N, K, ld_rows, 1, lse);
  return run_wide<128, 128, 4, 2, 3, GEMM_LSE>(s, A, W, part, M, N, K, ld_rows, 1, lse);
}

hipError_t launch_gemm(hipStream_t s, const f16* A, GemmW W, void* C, int M, int N, int K, int ldc,
                       GemmMode mode) {
  // GEMM_STORE_F32 callers that did not zero C get no K split
  int cfg, splits;
  gemm_choose(M, N, K, mode, &cfg, &splits);
  if (mode == GEMM_STORE_F32) splits = 1;
  return launch_gemm_cfg(s, A, W, C, M, N, K, ldc, mode, cfg, splits);
}

}  // namespace areal
