// Grouped-query causal attention over the paged KV cache.
//
// One wavefront owns 16 "rows" (decode: the <=16 query heads that share one
// KV head, for one sequence; prefill: 16 consecutive query positions of one
// head) and walks KV blocks of 16 tokens with an online softmax:
//   S^T[token, row] = K_tile . Q^T      v_mfma_f32_16x16x32_f16, K straight
//                                       from HBM (tiles stored in operand order)
//   P = exp2(S^T - m)                   float32, per-row running max / sum
//   O[row, :] += P . V_tile             v_mfma_f32_16x16x16_f16; the 
//                                       accumulator layout of S^T is already
//                                       the A-operand layout of this product,
//                                       and the V tile is stored in its
//                                       B-operand layout, so nothing is
//                                       transposed or staged through LDS.
#include "kernels.hpp"
#include <algorithm>
#include <cstdlib>
#include <type_traits>

namespace areal {
namespace {

constexpr int NB = 2;   // KV blocks per softmax update (32 tokens)

template <int D>
struct KvFrag {
  f16x8 k[NB][D / 32];
  f16x8 v[NB][D / 32];
};

__device__ __forceinline__ f32x4 mfma_qk(f16x8 a, f16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma_pv(f16x4 p, f16x4 v, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x16f16(p, v, c, 0, 0, 0);
}

// Folded over the four lanes (lane & 15 the same) that share a row.
__device__ __forceinline__ float max_over_groups(float v) {
  auto f = [](float a, float b) { return fmaxf(a, b); };
  return xor_lanes<32>(xor_lanes<16>(v, f), f);
}
__device__ __forceinline__ float sum_over_groups(float v) {
  auto f = [](float a, float b) { return a + b; };
  return xor_lanes<32>(xor_lanes<16>(v, f), f);
}

// One online-softmax update over the NB blocks held in `f`.
//   qf     : this lane's slice of its row's query (row = lane & 15)
//   row_pos: last visible token position of this lane's row
//   m, l   : running max (log2 domain) and this lane's share of the running sum
//   o      : accumulator, lane (g, jj) holds rows 4g+v, dims 16n+jj
template <int D>
__device__ __forceinline__ void attend_group(const KvFrag<D>& f, const f16x8 (&qf)[D / 32], int b,
                                             int row_pos, float scale_log2, float& m, float& l,
                                             f32x4 (&o)[D / 16], int lane) {
  const int g = lane >> 4;
  float s[NB][4];
  float mx = -INFINITY;
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < D / 32; ++c) acc = mfma_qk(f.k[u][c], qf[c], acc);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int t = (b + u) * kBlockTokens + 4 * g + v;
      s[u][v] = t <= row_pos ? acc[v] * scale_log2 : -INFINITY;
      mx = fmaxf(mx, s[u][v]);
    }
  }
  mx = max_over_groups(mx);
  const float m_new = fmaxf(m, mx);
  const float m_use = m_new == -INFINITY ? 0.f : m_new;
  const float alpha = __builtin_amdgcn_exp2f(m - m_use);   // m = -inf -> 0
  m = m_new;
  float psum = 0.f;
  f16x4 p[NB];
#pragma unroll
  for (int u = 0; u < NB; ++u)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float e = __builtin_amdgcn_exp2f(s[u][v] - m_use);
      psum += e;
      p[u][v] = f2h(e);
    }
  l = l * alpha + psum;
  // rescale the accumulator rows: row 4g+v needs the alpha held by lanes with (lane&15)==4g+v
  float ao[4];
#pragma unroll
  for (int v = 0; v < 4; ++v) ao[v] = __shfl(alpha, 4 * g + v);
#pragma unroll
  for (int n = 0; n < D / 16; ++n)
#pragma unroll
    for (int v = 0; v < 4; ++v) o[n][v] *= ao[v];
#pragma unroll
  for (int u = 0; u < NB; ++u)
#pragma unroll
    for (int n = 0; n < D / 16; ++n) {
      const f16x8 vv = f.v[u][n >> 1];
      f16x4 vh;
      if (n & 1) vh = f16x4{vv[4], vv[5], vv[6], vv[7]}; else vh = f16x4{vv[0], vv[1], vv[2], vv[3]};
      o[n] = mfma_pv(p[u], vh, o[n]);
    }
}

// ------------------------------------------------------------------ decode
// Block ids of a segment, fetched once: lane l of every wave holds the ids of
// blocks b0 + l and b0 + 64 + l (a segment spans at most 128 blocks).  Entries past the table's end read as zero.
struct BlockIds { int lo, hi; };
__device__ __forceinline__ BlockIds load_ids(const int32_t* table, int n, int lane) {
  const auto r = buffer_rsrc(table, (uint32_t)n * 4u);
  return BlockIds{buf1(r, lane * 4), buf1(r, lane * 4 + 256)};
}
__device__ __forceinline__ int block_id(const BlockIds& t, int rel) {      // rel: the same in all lanes
  const int lo = __builtin_amdgcn_readlane(t.lo, rel & 63), hi = __builtin_amdgcn_readlane(t.hi, rel & 63);
  return rel < 64 ? lo : hi;
}

// K and V tiles of blocks b and b + 1 for this wave's next update.  A block past b_end is an empty buffer: it reads as
// zero.  `tiles`: the kv head's K tile in block 0.
template <int D>
__device__ __forceinline__ void load_group_ids(KvFrag<D>& f, const f16* tiles, int block_stride, const BlockIds& ids,
                                               int b0, int b, int b_end, int lane) {
  constexpr int TILE_B = kBlockTokens * D * 2;
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    const int blk = block_id(ids, b + u - b0);
    // both tiles are stored chunk-major in operand order: load c of a wave reads 1 KiB in a row
    const auto r = buffer_rsrc(tiles + (int64_t)blk * block_stride, b + u < b_end ? 2u * TILE_B : 0u);
#pragma unroll
    for (int c = 0; c < D / 32; ++c) {
      f.k[u][c] = buf8(r, lane * 16 + c * 1024);
      f.v[u][c] = buf8(r, lane * 16 + TILE_B + c * 1024);
    }
  }
}

// Bias, rotate-half RoPE and rounding to half of one head vector of the float32
// QKV row, delivered as this lane's MFMA fragments: lane group g gets dims
// [32c + 8g, +8) for c = 0 .. D/32-1.  For D >= 64 a lane holds both members of
// every rotation pair (dims x and x + D/2 sit in chunks c and c + D/64); for
// D = 32 the partner sits in lane ^ 32.  Loading and rotating are separate steps
// so that the caller can put other loads in flight between them.
template <int D>
struct RawHead {
  float x[D / 32][8];
};
template <int D>
struct RopeAngles {                       // cos / sin of this lane's rotation pairs
  float c[D >= 64 ? D / 64 : 1][8], s[D >= 64 ? D / 64 : 1][8];
};

template <int D>
__device__ __forceinline__ void load_raw(RawHead<D>& r, const float* __restrict__ src, int g) {
#pragma unroll
  for (int c = 0; c < D / 32; ++c) {
    const float4 a = *reinterpret_cast<const float4*>(src + 32 * c + 8 * g);
    const float4 b = *reinterpret_cast<const float4*>(src + 32 * c + 8 * g + 4);
    r.x[c][0] = a.x; r.x[c][1] = a.y; r.x[c][2] = a.z; r.x[c][3] = a.w;
    r.x[c][4] = b.x; r.x[c][5] = b.y; r.x[c][6] = b.z; r.x[c][7] = b.w;
  }
}
template <int D>
__device__ __forceinline__ void load_angles(RopeAngles<D>& a, const float* __restrict__ ct,
                                            const float* __restrict__ sn, int g) {
  constexpr int HC = D >= 64 ? D / 64 : 1;
#pragma unroll
  for (int c = 0; c < HC; ++c) {
    const int j0 = D >= 64 ? 32 * c + 8 * g : (8 * g) & 15;
    const float4 c0 = *reinterpret_cast<const float4*>(ct + j0), c1 = *reinterpret_cast<const float4*>(ct + j0 + 4);
    const float4 s0 = *reinterpret_cast<const float4*>(sn + j0), s1 = *reinterpret_cast<const float4*>(sn + j0 + 4);
    a.c[c][0] = c0.x; a.c[c][1] = c0.y; a.c[c][2] = c0.z; a.c[c][3] = c0.w;
    a.c[c][4] = c1.x; a.c[c][5] = c1.y; a.c[c][6] = c1.z; a.c[c][7] = c1.w;
    a.s[c][0] = s0.x; a.s[c][1] = s0.y; a.s[c][2] = s0.z; a.s[c][3] = s0.w;
    a.s[c][4] = s1.x; a.s[c][5] = s1.y; a.s[c][6] = s1.z; a.s[c][7] = s1.w;
  }
}
template <int D>
__device__ __forceinline__ void rotate(RawHead<D>& r, const f16* __restrict__ bias, const RopeAngles<D>& a,
                                       int g, f16x8 (&out)[D / 32]) {
  if (bias) {
#pragma unroll
    for (int c = 0; c < D / 32; ++c) {
      const f16x8 bb = ld8(bias + 32 * c + 8 * g);
#pragma unroll
      for (int e = 0; e < 8; ++e) r.x[c][e] += h2f(bb[e]);
    }
  }
  if constexpr (D >= 64) {
    constexpr int HC = D / 64;
#pragma unroll
    for (int c = 0; c < HC; ++c)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float x1 = r.x[c][e], x2 = r.x[c + HC][e];
        out[c][e] = f2h_sat(x1 * a.c[c][e] - x2 * a.s[c][e]);
        out[c + HC][e] = f2h_sat(x2 * a.c[c][e] + x1 * a.s[c][e]);
      }
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float xp = __shfl_xor(r.x[0][e], 32);
      out[0][e] = f2h_sat(g < 2 ? r.x[0][e] * a.c[0][e] - xp * a.s[0][e] : r.x[0][e] * a.c[0][e] + xp * a.s[0][e]);
    }
  }
}

// What a decode work-group needs besides its segment (read from memory while descriptor and block ids travel).
struct DecodeArgs {
  const float* qkv;
  const f16 *bq, *bk, *bv;
  const float *cos_tab, *sin_tab;
  f16* arena;
  int block_stride, nq, max_own;
  float scale_log2;
  float *part_o, *part_ml;
  f16* out;
  const int32_t* pos;
  DecodeGroups grp;
};
constexpr int kSegRows = 32768;      // most work-groups along a grid's second dimension

// The leading KV blocks that a set of rows has in common (the work-groups of the decode launch behind the
// segments': u = chunk of the shared part).  Wave w
// owns tile w of the set: 16 MFMA rows = floor(16 / G) sequences x their G query heads, so
// every lane has its own sequence, position and query head.  Each wave walks all blocks of the
// chunk (the four waves read the same tiles: one fetch from L2 per work-group) and writes
// its rows' partial (max, sum, accumulator) into slot n_own + u of those rows (n_own: the launch's most own segments); the
// merge kernel folds them into the rows' own partials.  Every shared position precedes every
// row's position, so nothing is masked but the tail of the last block pair.
template <int D>
__device__ __forceinline__ void decode_shared_set(const DecodeArgs& A, int nkv, int n_slots, int set, int kvh, int u) {
  const float* __restrict__ qkv = A.qkv;
  const int nq = A.nq, n_own = A.max_own;
  const float *__restrict__ cos_tab = A.cos_tab, *__restrict__ sin_tab = A.sin_tab;
  const f16* __restrict__ bq = A.bq;
  const float scale_log2 = A.scale_log2;
  float *__restrict__ part_o = A.part_o, *__restrict__ part_ml = A.part_ml;
  const DecodeGroups& grp = A.grp;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, j = lane & 15;
  const int G = nq / nkv, P = 16 / G;
  const int chunk = grp.sh_chunk;
  const int t0 = u * chunk, b0 = t0 / kBlockTokens;
  const BlockIds ids = load_ids(grp.set_table + (int64_t)set * grp.set_stride + b0,
                                max(0, min(chunk / kBlockTokens, grp.set_stride - b0)), lane);
  const int sq = j / G;                                  // sequence of this lane's row inside the tile
  const int r = sq < P ? grp.set_rows[((int64_t)set * kGroupTiles + wave) * 16 + sq] : -1;
  const int ts = grp.set_start[set];
  if (t0 >= ts) return;
  if (__ballot(r >= 0) == 0) return;                     // no tile for this wave
  const f16* tiles = A.arena + kvh * 2 * (kBlockTokens * D);
  const int t1 = min(ts, t0 + chunk);
  const int b1 = (t1 + kBlockTokens - 1) / kBlockTokens;
  const int rr = max(r, 0);                              // empty rows read row 0 and are zeroed below
  const int pos = A.pos[rr];
  const int head = kvh * G + (j - sq * G);
  RawHead<D> qraw;
  load_raw<D>(qraw, qkv + ((int64_t)rr * (nq + 2 * nkv) + head) * D, g);
  RopeAngles<D> ang;
  load_angles<D>(ang, cos_tab + (int64_t)pos * (D / 2), sin_tab + (int64_t)pos * (D / 2), g);
  int b = b0;
  KvFrag<D> cur, nxt;
  load_group_ids<D>(cur, tiles, A.block_stride, ids, b0, b, b1, lane);
  f16x8 qf[D / 32];
  rotate<D>(qraw, bq ? bq + head * D : nullptr, ang, g, qf);
  if (r < 0) {
    const f16x8 zero8 = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int c = 0; c < D / 32; ++c) qf[c] = zero8;
  }
  float m = -INFINITY, l = 0.f;
  f32x4 o[D / 16];
#pragma unroll
  for (int n = 0; n < D / 16; ++n) o[n] = f32x4{0.f, 0.f, 0.f, 0.f};
  while (b < b1) {
    const int bn = b + NB;
    if (bn < b1) load_group_ids<D>(nxt, tiles, A.block_stride, ids, b0, bn, b1, lane);
    attend_group<D>(cur, qf, b, t1 - 1, scale_log2, m, l, o, lane);
    cur = nxt;
    b = bn;
  }
  l = sum_over_groups(l);
  const int slot = n_own + u;
  if (g == 0 && r >= 0) {
    const int64_t pi = ((int64_t)r * nq + head) * n_slots + slot;
    part_ml[pi * 2] = m;
    part_ml[pi * 2 + 1] = l;
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {                          // accumulator row 4g+v belongs to lane 4g+v's row
    const int r_v = __shfl(r, 4 * g + v), head_v = __shfl(head, 4 * g + v);
    if (r_v >= 0) {
      const int64_t pi = ((int64_t)r_v * nq + head_v) * n_slots + slot;
#pragma unroll
      for (int n = 0; n < D / 16; ++n) part_o[pi * D + 16 * n + j] = o[n][v];
    }
  }
}

// One work-group per (segment, kv head); the partials of a row cut into several segments
// are combined by attn_merge_kernel.  Bound by HBM: work-groups are handed out by decode_plan.hpp (segments of
// about equal length, an eighth of the tokens to each XCD), and where a segment's block ids lie depends on the
// launch index alone, so that they travel together with its descriptor.  The row's query heads
// are taken from the float32 QKV row (bias, RoPE, rounding done here).  The
// cached positions 0 .. pos-1 come from the paged arena; the token being
// appended (position pos) is handled by the work-group whose segment contains
// pos: its last wave, which has the fewest blocks, rotates and rounds the new key and stores key and value into the
// sequence's block for later steps, and the new token is folded into the softmax
// state as one more (score, value) pair.
// The first arguments arrive in registers with the launch: where the segment's descriptor and block ids lie.  base x: first
// segment of XCD x (the first XCD's is 0).  A work-group lives for some 20 us, of which two round trips before its first
// K/V tile cannot be helped; the argument reads before them (a third one), divisions, exec masks around loads and block ids
// passed through LDS could.  With them gone, in the merge too, and the wave's index and block addresses in scalar
// registers: step of 24 rows 2,066 -> 2,007 us, 88 3,011 -> 2,927, 256 2,921 -> 2,796, 7B of 128 7,356 -> 7,074, 16 rows of
// 26,000 tokens 7,497 -> 7,333.
template <int D>
__global__ __launch_bounds__(256) void attn_decode_kernel(
    const int4* __restrict__ desc, const int32_t* __restrict__ seg_table, int base1, int base2, int base3, int base4,
    int base5, int base6, int base7, int base8, int depth, uint32_t shape, DecodeArgs) {
  typedef decltype(attn_decode_kernel<D>) Kernel;
  __shared__ float sm[4][16], sl[4][16];
  __shared__ float so[4][16][D];
  __shared__ float s_new[16], v_new[D];
  // grid (8 nkv, .., ..): work-groups 8 (q nkv .. q nkv + nkv - 1) + x are segment q of XCD x, one per kv head
  const int xcd = blockIdx.x & 7, kvh = blockIdx.x >> 3;
  const int stride = shape & 255, G = (shape >> 8) & 31, nkv = shape >> 13, nq = G * nkv;
  const int q_seg = blockIdx.z * kSegRows + blockIdx.y;
  if (q_seg >= depth) {                                  // the shared leading blocks of a set of rows
    const DecodeArgs A = late_args<Kernel>();
    const int n_shared = A.grp.n_shared, w = (q_seg - depth) * 8 + xcd;
    const int set = n_shared > 0 ? w / n_shared : 0;
    if (n_shared > 0 && set < A.grp.n_sets)
      decode_shared_set<D>(A, nkv, A.max_own + n_shared, set, kvh, w - set * n_shared);
    return;
  }
  // base of XCD x and of the next one, by the bits of x
  const bool x1 = xcd & 1, x2 = xcd & 2, x4 = xcd & 4;
  const int seg = (x4 ? (x2 ? (x1 ? base7 : base6) : (x1 ? base5 : base4)) : (x2 ? (x1 ? base3 : base2) : (x1 ? base1 : 0))) + q_seg;
  const int seg_end = x4 ? (x2 ? (x1 ? base8 : base7) : (x1 ? base6 : base5)) : (x2 ? (x1 ? base4 : base3) : (x1 ? base2 : base1));
  if (seg >= seg_end) return;                            // this XCD has fewer
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, j = lane & 15;
  const BlockIds ids = load_ids(seg_table + (int64_t)seg * stride, stride, lane);
  const int4 d = desc[seg];
  const DecodeArgs A = late_args<Kernel>();
  const float* __restrict__ qkv = A.qkv;
  const f16 *__restrict__ bq = A.bq, *__restrict__ bk = A.bk, *__restrict__ bv = A.bv;
  f16* __restrict__ arena = A.arena;
  const int n_slots = A.max_own + A.grp.n_shared;        // partial slots per (row, head)
  const float scale_log2 = A.scale_log2;
  const f16* tiles = arena + kvh * 2 * (kBlockTokens * D);
  // Token and block indices below are relative to the first position this row's own work-groups cover.
  const int i = d.x, pos_abs = d.y, pos = d.z, packed = d.w;
  const int t0 = (packed & 0xFFF) * 32, n_tok = ((packed >> 12) & 0x7F) * 32, slot = (packed >> 19) & 31;
  const bool single = (packed >> 24) & 1;              // the row has no other partial
  const int b0 = t0 / kBlockTokens;
  const bool owner = pos < t0 + n_tok;                 // this segment holds the appended position
  const int t1 = min(pos, t0 + n_tok);                 // cached tokens [t0, t1)
  const int b1 = (t1 + kBlockTokens - 1) / kBlockTokens;

  // Loads go out in dependency order (the query row needs nothing, the angles need pos,
  // the K/V tiles need the block ids) and the rotation runs while the tiles are in flight.
  const float* row = qkv + (int64_t)i * (nq + 2 * nkv) * D;
  const int head = kvh * G + min(j, G - 1);

  // wave w takes block groups w, w+4, ... of this segment
  int b = b0 + wave * NB;
  KvFrag<D> cur, nxt;
  if (b < b1) load_group_ids<D>(cur, tiles, A.block_stride, ids, b0, b, b1, lane);
  RawHead<D> qraw;
  load_raw<D>(qraw, row + head * D, g);
  RopeAngles<D> ang;
  load_angles<D>(ang, A.cos_tab + (int64_t)pos_abs * (D / 2), A.sin_tab + (int64_t)pos_abs * (D / 2), g);

  f16x8 qf[D / 32];
  rotate<D>(qraw, bq ? bq + head * D : nullptr, ang, g, qf);
  if (j >= G) {
    const f16x8 zero8 = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int c = 0; c < D / 32; ++c) qf[c] = zero8;
  }
  if (owner && wave == 3) {                            // wave-uniform
    RawHead<D> kraw;
    load_raw<D>(kraw, row + (nq + kvh) * D, g);
    f16x8 kf[D / 32];
    rotate<D>(kraw, bk ? bk + kvh * D : nullptr, ang, g, kf);
    float dot = 0.f;
#pragma unroll
    for (int c = 0; c < D / 32; ++c)
#pragma unroll
      for (int e = 0; e < 8; ++e) dot += h2f(qf[c][e]) * h2f(kf[c][e]);
    dot = sum_over_groups(dot);
    if (g == 0) s_new[j] = dot * scale_log2;
    const int blk = block_id(ids, pos / kBlockTokens - b0), tin = pos % kBlockTokens;
    f16* kt = arena + (int64_t)blk * A.block_stride + kvh * 2 * (kBlockTokens * D);
    if (j == 0) {
#pragma unroll
      for (int c = 0; c < D / 32; ++c) *reinterpret_cast<f16x8*>(kt + k_tile_index(tin, 32 * c + 8 * g)) = kf[c];
    }
    f16* vt = kt + kBlockTokens * D;
    const float* vrow = row + (nq + nkv + kvh) * D;
    for (int dim = lane; dim < D; dim += 64) {
      float v = vrow[dim];
      if (bv) v += h2f(bv[kvh * D + dim]);
      const f16 hv = f2h_sat(v);
      v_new[dim] = h2f(hv);
      vt[v_tile_index(D, tin, dim)] = hv;
    }
  }
  float m = -INFINITY, l = 0.f;
  f32x4 o[D / 16];
#pragma unroll
  for (int n = 0; n < D / 16; ++n) o[n] = f32x4{0.f, 0.f, 0.f, 0.f};

  while (b < b1) {
    const int bn = b + 4 * NB;
    if (bn < b1) load_group_ids<D>(nxt, tiles, A.block_stride, ids, b0, bn, b1, lane);
    attend_group<D>(cur, qf, b, pos - 1, scale_log2, m, l, o, lane);
    cur = nxt;
    b = bn;
  }
  l = sum_over_groups(l);

  if (g == 0) { sm[wave][j] = m; sl[wave][j] = l; }
#pragma unroll
  for (int n = 0; n < D / 16; ++n)
#pragma unroll
    for (int v = 0; v < 4; ++v) so[wave][4 * g + v][16 * n + j] = o[n][v];
  __syncthreads();
  for (int idx = threadIdx.x; idx < G * D; idx += 256) {
    const int h = idx / D, dd = idx - h * D;
    float M = fmaxf(fmaxf(sm[0][h], sm[1][h]), fmaxf(sm[2][h], sm[3][h]));
    const float Mu = M == -INFINITY ? 0.f : M;               // no cached token in this split
    float L = 0.f, O = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float sc = __builtin_amdgcn_exp2f(sm[w][h] - Mu);  // idle wave: m = -inf -> 0
      L += sl[w][h] * sc;
      O += so[w][h][dd] * sc;
    }
    if (owner) {                                             // the appended token
      const float sN = s_new[h];
      const float M2 = fmaxf(M, sN);
      const float a = __builtin_amdgcn_exp2f(M - M2), e = __builtin_amdgcn_exp2f(sN - M2);
      L = L * a + e;
      O = O * a + e * v_new[dd];
      M = M2;
    }
    const int head = kvh * G + h;
    if (single) {
      A.out[((int64_t)i * nq + head) * D + dd] = f2h_sat(O / L);
    } else {
      const int64_t pi = ((int64_t)i * nq + head) * n_slots + slot;
      A.part_o[pi * D + dd] = O;
      if (dd == 0) { A.part_ml[pi * 2] = M; A.part_ml[pi * 2 + 1] = L; }
    }
  }
}

// Combine the split partials of one (row, head): out = sum_s O_s 2^(M_s-M) / sum_s L_s 2^(M_s-M).
// Bound by latency, one round trip: every load address depends only on the launch shape, so the row's slot count, the
// statistics (lane s fetches (M_s, L_s)) and the first eight partial rows all go out
// together; which slots really exist for this row is applied afterwards by selection.  The
// other slots hold stale values of earlier launches: selected away, never multiplied.
template <int D>
__global__ __launch_bounds__(D < 64 ? 64 : D) void attn_merge_kernel(const float* __restrict__ part_o,
                                                       const float* __restrict__ part_ml,
                                                       const int32_t* __restrict__ own, int nq, int max_own,
                                                       int n_shared, int sh_chunk,
                                                       const int32_t* __restrict__ t_start, f16* __restrict__ out) {
  constexpr int BATCH = 8;
  const int n_slots = max_own + n_shared;                     // <= 32
  const int i = blockIdx.y;                                   // grid (heads, rows)
  const int64_t pair = (int64_t)i * nq + blockIdx.x;
  const int lane = threadIdx.x & 63;
  const int dd = min((int)threadIdx.x, D - 1);
  const auto po = buffer_rsrc(part_o + pair * n_slots * D, (uint32_t)(n_slots * D) * 4u);    // past its end: zero
  const auto pml = buffer_rsrc(part_ml + pair * n_slots * 2, (uint32_t)n_slots * 8u);
  auto row = [&](int slot) { return __builtin_bit_cast(float, buf1(po, (slot * D + dd) * 4)); };
  const b64_t mlb = __builtin_amdgcn_raw_buffer_load_b64(pml, lane * 8, 0, 0);
  const uint32_t mb = mlb[0], lb = mlb[1];
  float v[BATCH], vn[BATCH];
#pragma unroll
  for (int u = 0; u < BATCH; ++u) v[u] = row(u);
  const int ns = own[i];
  const int ts = t_start ? t_start[i] : 0;

  // slots of this row: its own segments 0 .. ns - 1, then the chunks of
  // the part it shares with its set (slot max_own + u exists while u * sh_chunk < ts)
  if (ns == 1 && ts == 0) return;                             // nothing to combine: `out` is written
  const bool mine = lane < max_own ? lane < ns : (lane < n_slots && (lane - max_own) * sh_chunk < ts);
  const uint64_t have = __ballot(mine);                       // slots live in lanes 0 .. 31
  const float ms = mine ? __builtin_bit_cast(float, mb) : -INFINITY, ls = mine ? __builtin_bit_cast(float, lb) : 0.f;
  const float M = wave_max(ms);                               // whole waves only: blockDim >= 64
  const float sc = __builtin_amdgcn_exp2f(ms - M);           // other lanes: 2^-inf = 0
  const float L = wave_sum(ls * sc);
  float O = 0.f;
  for (int s0 = 0; s0 < n_slots; s0 += BATCH) {
    const bool more = (have >> (s0 + BATCH)) != 0 && s0 + BATCH < n_slots;
    if (more) {                                               // next batch in flight while this one is used
#pragma unroll
      for (int u = 0; u < BATCH; ++u) vn[u] = row(s0 + BATCH + u);
    }
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
      const float w = __builtin_bit_cast(
          float, __builtin_amdgcn_readlane((int)__builtin_bit_cast(uint32_t, sc), (s0 + u) & 31));
      O += ((have >> (s0 + u)) & 1u) ? v[u] * w : 0.f;
    }
    if (!more) break;
#pragma unroll
    for (int u = 0; u < BATCH; ++u) v[u] = vn[u];
  }
  if (threadIdx.x < D) out[pair * D + dd] = f2h_sat(O / L);
}

// ----------------------------------------------------------------- prefill
// One work-group per (tile of 16 or 32 query positions, kv head): its rows are
// those positions x the G query heads that share the kv head, cut into
// row-groups of 16 (positions of one head), RGW row-groups per wave.  KV blocks
// travel HBM -> LDS once per work-group (buffer_load ... lds, a ring of PF_STAGES
// stages of two blocks each) and every wave multiplies all its row-groups
// against them, so each K/V byte fetched serves up to 32*G query rows.
// Both products use the 16x16x32 MFMA: for P.V the 32-deep contraction runs
// over the two blocks of a stage (slots 0-3: tokens 4g..4g+3 of the first
// block, slots 4-7: of the second), which is the order the S^T accumulators and
// the stored V tiles already have.
//
// A launch lives on its longest walks (122 steps of 32 tokens for the last tile of 3,900), whose waves have few
// others beside them, so a wave overlaps its own work: step p holds the scores of pair p and issues
//   A: the score MFMAs of pair p + 1, a score's exponential (of pair p) between two of them,
//   B: the value MFMAs of pair p, between them scale, mask and maximum of the scores of pair p + 1
// (one after another they are 768 cycles of MFMAs and about 650 of float32 arithmetic per step of three row-groups).
//
// Issue bounds the step: an MFMA takes 8 cycles of a SIMD's issue, an exponential 8, other vector instructions 4, a
// fragment read about 14, and with one wave to a SIMD nothing hides the barrier (170 cycles) and the step's loads (250):
// 1,240 cycles of A and B, some 1,900 in all.  In order of phases and with the mask for every pair it was 2,150: one launch
// of a prompt of 4,096 tokens 163 -> 136 us, two 166 -> 152, 4 of 2,048 91 -> 79, 8 of 1,024 50 -> 44, 32 of 256 22 -> 20.5
// (12 / 2 heads of 128); a prefill of 1,000 tokens 2,508 -> 2,486 us in whole.  Slower: the 32x32x16 MFMA with a wave's 32
// positions (156 us), ten stages (one work-group on a compute unit: 211), a barrier between A and B (149).
constexpr int PF_STAGES = 5;   // two work-groups of 80 KB on a compute unit at head_dim 128

// The running maximum is a reference, not an exact maximum: it is raised (two cross-lane exchanges and a rescale of
// the accumulator) only when some score of the wave exceeds it by more than 2^kMaxSlack, so
// probabilities stay below 2^kMaxSlack in half precision and the common step has no cross-lane traffic at all.
constexpr float kMaxSlack = 8.0f;

// A value that is computed where it stands in the program (not moved behind the barrier, next to its use).
template <class T>
__device__ __forceinline__ T stay(T x) {
  asm volatile("" : "+v"(x));
  return x;
}

template <int D, int RGW>
struct PfState {
  static constexpr int DC = D / 32, NO = D / 16, TILE_B = 16 * D * 2;
  f16x8 qf[RGW][DC];            // queries
  f32x4 o[RGW][NO];             // accumulators: lane (g, j) holds rows 4g + v, dims 16n + j
  float nm[RGW], l[RGW];        // minus the reference maximum (log2 domain), this lane's share of the sums
  float mx[RGW];                // largest scaled score of this lane relative to the reference
  int rpos[RGW];                // last token that this lane's row sees
  f32x4 s[RGW][2];              // raw scores q.k of the pair whose turn is next: lane (g, j) holds tokens 4g + v of row j
  f32x4 t[RGW][2];              // the same scaled, minus the reference: exponents of 2; -inf where masked
  // K fragments f = u * DC + c (MFMA c of block u) are read KD ahead of their use, V fragments VD ahead: few other waves
  // fill the time of an LDS read.
  static constexpr int KD = 2 * DC < 4 ? 2 * DC : 4, VD = DC < 2 ? DC : 2;
  int g;

  __device__ __forceinline__ f16x8 tile(const char* base, int c, int lane) const {
    return *reinterpret_cast<const f16x8*>(base + c * 1024 + lane * 16);
  }
  __device__ __forceinline__ f16x8 k_frag(const char* stage, int f, int lane) const {
    return tile(stage + (f / DC) * 2 * TILE_B, f % DC, lane);
  }
  // t from s for score z = r * 8 + u * 4 + v of pair `pair`
  template <bool MASK>
  __device__ __forceinline__ void scale_one(int z, int pair, float scale_log2) {
    const int r = z >> 3, u = (z >> 2) & 1, v = z & 3;
    const float x = __builtin_fmaf(s[r][u][v], scale_log2, nm[r]);
    t[r][u][v] = !MASK || (2 * pair + u) * kBlockTokens + 4 * g + v <= rpos[r] ? x : -INFINITY;
  }
  // Scores of row-group r, whose raw values are in s, against the reference -nm; raises it where t says so.
  __device__ __forceinline__ void raise(int r, float scale_log2, bool first) {
    float x = max_over_groups(mx[r]);                     // relative to the present reference
    const float up = first ? x : fmaxf(x, 0.f);
    const float by = up == -INFINITY ? 0.f : up;          // a wave without rows: nothing is visible
    const float alpha = first ? 0.f : __builtin_amdgcn_exp2f(-by);
    nm[r] -= by;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        t[r][u][v] = t[r][u][v] == -INFINITY ? -INFINITY : __builtin_fmaf(s[r][u][v], scale_log2, nm[r]);
    if (first) return;
    l[r] *= alpha;
    float ao[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) ao[v] = __shfl(alpha, 4 * g + v);
#pragma unroll
    for (int n = 0; n < NO; ++n)
#pragma unroll
      for (int v = 0; v < 4; ++v) o[r][n][v] *= ao[v];
  }
  // First pair: scores, scale, mask, reference; first fragments of the second.
  __device__ __forceinline__ void start(const char* stage, float scale_log2, int lane) {
#pragma unroll
    for (int c = 0; c < DC; ++c)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const f16x8 k = tile(stage + u * 2 * TILE_B, c, lane);
#pragma unroll
        for (int r = 0; r < RGW; ++r) s[r][u] = mfma_qk(k, qf[r][c], c ? s[r][u] : f32x4{0.f, 0.f, 0.f, 0.f});
      }
#pragma unroll
    for (int r = 0; r < RGW; ++r) {
      mx[r] = -INFINITY;
#pragma unroll
      for (int z = 0; z < 8; ++z) {
        scale_one<true>(r * 8 + z, 0, scale_log2);
        mx[r] = fmaxf(mx[r], t[r][z >> 2][z & 3]);
      }
      raise(r, scale_log2, true);
      mx[r] = 0.f;
    }
  }
  // Step of `pair`, whose scores are in t.  NEXT: pair + 1 exists, its K tiles in k_stage; MASK: some of its tokens may
  // lie behind a row of this wave.
  template <bool NEXT, bool MASK>
  __device__ __forceinline__ void step(const char* v_stage, const char* k_stage, int pair, float scale_log2, int lane) {
    bool over = false;
#pragma unroll
    for (int r = 0; r < RGW; ++r) over |= mx[r] > kMaxSlack;
    if (__any(over)) {                                    // wave-uniform, rare
#pragma unroll
      for (int r = 0; r < RGW; ++r) raise(r, scale_log2, false);
    }
    f16x8 p[RGW], v0[VD], v1[VD];
    float psum[RGW];
#pragma unroll
    for (int r = 0; r < RGW; ++r) psum[r] = 0.f;
    auto read_v = [&](int c) {
      v0[c % VD] = tile(v_stage + TILE_B, c, lane);
      v1[c % VD] = tile(v_stage + 3 * TILE_B, c, lane);
    };
    // A, block by block: exponential z of the present pair (block z / (4 RGW), row-group z / 4 % RGW) behind a score MFMA
    // of the same block of the next, its sum and its rounding one and two later, so that nothing waits for the
    // exponential's latency and the two pairs' scores hardly overlap in registers.
    constexpr int NS = RGW * 8, NQ = RGW * 2 * DC, PER = NS / NQ, LEAD = NS / 4;
    auto exp_part = [&](int z) {                          // z = 0 .. NS + 1
      if (z < NS) {
        f32x4& x = t[(z >> 2) % RGW][z / (4 * RGW)];
        x[z & 3] = stay(__builtin_amdgcn_exp2f(x[z & 3]));
      }
      if (z >= 2) {
        const int y = z - 2, r = (y >> 2) % RGW, u = y / (4 * RGW), v = y & 3;
        psum[r] = stay(psum[r] + t[r][u][v]);
        if (v & 1) {
          const f16x2 h = {f2h(t[r][u][v - 1]), f2h(t[r][u][v])};
          const uint32_t w = stay(__builtin_bit_cast(uint32_t, h));
          p[r][u * 4 + v - 1] = __builtin_bit_cast(f16x2, w)[0];
          p[r][u * 4 + v] = __builtin_bit_cast(f16x2, w)[1];
        }
      }
    };
    if (NEXT) {
      f16x8 k[KD + 1];
#pragma unroll
      for (int f = 0; f < KD; ++f) k[f] = k_frag(k_stage, f, lane);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int z = 0; z < LEAD; ++z) exp_part(z);         // while the first fragments travel
#pragma unroll
      for (int f = 0; f < 2 * DC; ++f) {
        if (f + KD < 2 * DC) k[(f + KD) % (KD + 1)] = k_frag(k_stage, f + KD, lane);
        if (f >= 2 * DC - 2 * VD && (f - (2 * DC - 2 * VD)) % 2 == 0) read_v((f - (2 * DC - 2 * VD)) / 2);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < RGW; ++r) {
          const int c = f % DC, u = f / DC;
          s[r][u] = mfma_qk(k[f % (KD + 1)], qf[r][c], c ? s[r][u] : f32x4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
          for (int e = 0; e < PER; ++e)
            if ((f * RGW + r) * PER + e + LEAD < NS) exp_part((f * RGW + r) * PER + e + LEAD);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    } else {
#pragma unroll
      for (int c = 0; c < VD; ++c) read_v(c);
#pragma unroll
      for (int z = 0; z < NS; ++z) exp_part(z);
    }
    exp_part(NS);
    exp_part(NS + 1);
#pragma unroll
    for (int r = 0; r < RGW; ++r) {
      l[r] += psum[r];
      mx[r] = -INFINITY;
    }
    __builtin_amdgcn_sched_barrier(0);
    // B.
    constexpr int NV = RGW * NO, PERV = NS / NV;
    auto scale_part = [&](int z) {
      if (!NEXT) return;
      scale_one<MASK>(z, pair + 1, scale_log2);
      if (z & 1) mx[z >> 3] = fmaxf(fmaxf(mx[z >> 3], t[z >> 3][(z >> 2) & 1][(z & 3) - 1]), t[z >> 3][(z >> 2) & 1][z & 3]);
    };
#pragma unroll
    for (int c = 0; c < DC; ++c) {
      const f16x8 a = v0[c % VD], b = v1[c % VD];
      const f16x8 ve = f16x8{a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
      const f16x8 vo = f16x8{a[4], a[5], a[6], a[7], b[4], b[5], b[6], b[7]};
      if (c + VD < DC) read_v(c + VD);
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int r = 0; r < RGW; ++r) {
          o[r][2 * c + h] = mfma_qk(p[r], h ? vo : ve, o[r][2 * c + h]);
#pragma unroll
          for (int e = 0; e < PERV; ++e) scale_part(((2 * c + h) * RGW + r) * PERV + e);
          __builtin_amdgcn_sched_barrier(0);
        }
    }
  }
};

// parts_magic: 2^32 / (kv heads x head parts), rounded up (0: one); shape: G | head parts << 5 | kv heads << 10;
// inv_g: 2^16 / heads of a part, rounded up.
template <int D, int RGW>
__global__ __launch_bounds__(256, (D == 128 && RGW == 3) ? 2 : 1) void attn_prefill_kernel(
    const AttnWork* __restrict__ work, const f16* __restrict__ q, const int32_t* __restrict__ tables,
    const f16* __restrict__ arena, uint32_t parts_magic, uint32_t shape, uint32_t inv_g, int tile_pos, int max_blocks,
    int block_stride, int n_wgs, float scale_log2, f16* __restrict__ out) {
  typedef PfState<D, RGW> State;
  constexpr int TILE_B = State::TILE_B;   // bytes of one K or V tile
  constexpr int STAGE_B = 4 * TILE_B;     // two blocks x (K, V)
  constexpr int NI = TILE_B / 1024;       // load instructions per tile = per wave per stage
  __shared__ __attribute__((aligned(16))) char lds[PF_STAGES * STAGE_B];

  // Work comes longest walk first, all KV heads of a tile in a row.  In a pass of 8,192 rows all 512 work-groups are
  // resident at once, two to a compute unit, and with the tiles in sequence order the two KV heads of the longest walk
  // shared one: 15 trajectories of 512 - 3,900 tokens 110.7 -> 108.1 ms in whole, attention 145 -> 123 us a launch.  Of two work-groups that share a compute unit the
  // second 256 are taken from the short end, so that long and short walks pair up; from then on a free place
  // takes the longest left.
  int rank = blockIdx.x;
  if (rank >= 256 && rank < 512) rank = min(511, n_wgs - 1) - (rank - 256);
  const int g_all = shape & 31, head_parts = (shape >> 5) & 31, nkv = shape >> 10, nq = g_all * nkv;
  int item = parts_magic ? __umulhi(rank, parts_magic) : rank;
  if (item * (nkv * head_parts) > rank) --item;          // (a rank beyond 2^32 / parts may round up to the next item)
  const int of_item = rank - item * (nkv * head_parts);
  const AttnWork wk = work[item];
  const int kvh = head_parts == 1 ? of_item : of_item >> 1, part = head_parts == 1 ? 0 : of_item & 1;   // one or two parts
  // this work-group's query heads: head0 .. head0 + n_heads - 1 of the G that share the kv head
  const int G = (g_all + head_parts - 1) >> (head_parts - 1);
  const int head0 = kvh * g_all + part * G, n_heads = min(G, g_all - part * G);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, j = lane & 15;
  const int n_rg = (tile_pos / 16) * G;
  const int last_pos = wk.pos0 + wk.n_rows - 1;
  const int b_end = last_pos / kBlockTokens + 1;
  const int n_pairs = (b_end + 1) >> 1;
  const auto table = buffer_rsrc(tables + (int64_t)wk.slot * max_blocks, (uint32_t)b_end * 4u);

  // ---- this wave's share of the loads: one tile of the stage (block u, K or V) ----
  const int u_ld = wave >> 1, isv_ld = wave & 1;
  // tiles are stored in operand order, chunk c of all lanes in a 1 KiB run: the copy into LDS
  // is verbatim and lane-linear, and so are the fragment reads (no bank conflicts, no swizzle)
  const f16* my_tiles = arena + (kvh * 2 + isv_ld) * (kBlockTokens * D);
  int id_chunk = 0, ids = buf1(table, lane * 4);
  auto issue = [&](int pair) {
    const int b = min(2 * pair + u_ld, b_end - 1);     // past the end: re-read the last block (masked anyway)
    if ((b >> 6) != id_chunk) {                        // wave-uniform
      id_chunk = b >> 6;
      ids = buf1(table, (id_chunk * 64 + lane) * 4);
      // used here, so that the wait for this load stands here: behind the branch the compiler would
      // have to wait in every step, for all loads in flight, the ring's among them
      asm volatile("" : "+v"(ids));
    }
    const int blk = __builtin_amdgcn_readlane(ids, b & 63);
    const auto tile = buffer_rsrc(my_tiles + (int64_t)blk * block_stride, TILE_B);
    char* dst = lds + (pair % PF_STAGES) * STAGE_B + (u_ld * 2 + isv_ld) * TILE_B;
#pragma unroll
    for (int t = 0; t < NI; ++t) dma16(tile, lane * 16, t * 1024, dst + t * 1024);
  };

  // ---- this wave's row-groups ----
  State w;
  w.g = g;
  int gmax[RGW];
#pragma unroll
  for (int r = 0; r < RGW; ++r) {
    const int rg = wave * RGW + r;
    const int pos_blk = (rg * inv_g) >> 16, hd = rg - pos_blk * G, head = head0 + hd;
    const int row_in = pos_blk * 16 + j;
    const bool active = rg < n_rg && hd < n_heads && pos_blk * 16 < wk.n_rows;
    const bool ok = active && row_in < wk.n_rows;
    gmax[r] = active ? wk.pos0 + min(wk.n_rows, pos_blk * 16 + 16) - 1 : -1;
    w.rpos[r] = ok ? wk.pos0 + row_in : gmax[r];
    // MFMA c contracts dims [32c, 32c+32), lane group g its slice [32c + 8g, +8): the order of the K tiles
    const auto qr = buffer_rsrc(q + ((int64_t)wk.row0 * nq + (active ? head : 0)) * D,
                                active ? (uint32_t)((wk.n_rows - 1) * nq + 1) * (D * 2u) : 0u);   // rows below: zero
#pragma unroll
    for (int c = 0; c < D / 32; ++c) w.qf[r][c] = buf8(qr, row_in * nq * (D * 2) + (c * 32 + g * 8) * 2);
    w.nm[r] = 0.f;
    w.l[r] = 0.f;
#pragma unroll
    for (int n = 0; n < D / 16; ++n) w.o[r][n] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  asm volatile("" : "+v"(ids));                        // (its wait here, not before every use)
#pragma unroll
  for (int s = 0; s < PF_STAGES - 1; ++s)
    if (s < n_pairs) issue(s);

  // pairs of blocks that lie wholly below the first query position of this wave need no mask
  // (row-group r = 0 holds the wave's earliest positions; a wave without rows masks everything)
  const int p_free = gmax[0] >= 0 ? (wk.pos0 + ((wave * RGW * inv_g) >> 16) * 16 + 1) / (2 * kBlockTokens) : 0;

  // waits until at most `pairs` of the pairs requested last are on their way
  auto wait_pairs = [&](int pairs) {
    static_assert(PF_STAGES == 5, "cases below");
    if (pairs >= 3) wait_vmcnt(3 * NI);
    else if (pairs == 2) wait_vmcnt(2 * NI);
    else if (pairs == 1) wait_vmcnt(NI);
    else wait_vmcnt(0);
  };
  // pair 0 has landed, for every wave
  wait_pairs(min(n_pairs, PF_STAGES - 1) - 1);
  __builtin_amdgcn_s_barrier();
  auto stage = [&](int pair) { return lds + (pair % PF_STAGES) * STAGE_B; };
  w.start(lds, scale_log2, lane);
  auto step = [&](int p, auto masked) {
    // the stage that is refilled below was read in the step before: those reads are complete, for every wave, and pair
    // p + 1 has landed for every wave (the pairs after it may still be on their way)
    wait_lgkmcnt0();
    if (p + PF_STAGES - 1 <= n_pairs) wait_vmcnt((PF_STAGES - 3) * NI);
    else wait_pairs(n_pairs - 2 - p);
    __builtin_amdgcn_s_barrier();
    if (p + PF_STAGES - 1 < n_pairs) issue(p + PF_STAGES - 1);
    w.template step<true, decltype(masked)::value>(stage(p), stage(p + 1), p, scale_log2, lane);
  };
  // all waves of the work-group run the same number of steps (the barrier is shared); each
  // wave's mask-free prefix is its own
  const int p_split = min(p_free, n_pairs) - 1;
  int p = 0;
  for (; p < p_split; ++p) step(p, std::false_type{});
  for (; p < n_pairs - 1; ++p) step(p, std::true_type{});
  w.template step<false, false>(stage(p), nullptr, p, scale_log2, lane);

#pragma unroll
  for (int r = 0; r < RGW; ++r) {
    const int rg = wave * RGW + r;
    const int pos_blk = (rg * inv_g) >> 16, head = head0 + rg - pos_blk * G;
    const float lr = sum_over_groups(w.l[r]);
    float lo[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) lo[v] = __shfl(lr, 4 * g + v);
    if (gmax[r] < 0) continue;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row_in = pos_blk * 16 + 4 * g + v;
      if (row_in < wk.n_rows) {
        f16* op = out + ((int64_t)(wk.row0 + row_in) * nq + head) * D;
        const float inv = 1.0f / lo[v];
#pragma unroll
        for (int n = 0; n < D / 16; ++n) op[16 * n + j] = f2h_sat(w.o[r][n][v] * inv);
      }
    }
  }
}

}  // namespace

static bool geom_ok(const KvGeom& g, int nq) {
  const int d = g.head_dim;
  if (d != 32 && d != 64 && d != 128) return false;
  if (g.n_kv_heads <= 0 || nq % g.n_kv_heads || nq / g.n_kv_heads > 16) return false;
  return true;
}

static bool groups_ok(const DecodeGroups& grp, int M, int max_own) {
  if (grp.n_sets == 0 && grp.n_shared == 0 && !grp.t_start) return true;
  return grp.n_sets > 0 && grp.n_sets <= M && grp.n_shared > 0 && max_own + grp.n_shared <= 32 &&
         grp.sh_chunk > 0 && grp.sh_chunk % (NB * kBlockTokens) == 0 && grp.sh_chunk <= 128 * kBlockTokens &&
         grp.t_start && grp.set_rows && grp.set_start && grp.set_table && grp.set_stride > 0;
}

hipError_t launch_attn_decode(hipStream_t s, const float* qkv, int M, RowMeta rm, const f16* bq, const f16* bk,
                              const f16* bv, const float* cos_tab, const float* sin_tab, f16* arena_layer, KvGeom geom,
                              int n_q_heads, DecodeSegs segs, float* part_o, float* part_ml, f16* out,
                              DecodeGroups grp) {
  bool base_ok = segs.base[0] == 0 && segs.base[8] > 0;
  for (int x = 0; x < 8; ++x) base_ok &= segs.base[x] <= segs.base[x + 1] && segs.base[x + 1] - segs.base[x] <= segs.depth;
  if (M <= 0 || !geom_ok(geom, n_q_heads) || !base_ok || segs.max_own < 1 || segs.max_own > 32 ||
      segs.stride <= 0 || segs.stride > 132 || !segs.desc || !segs.table || !segs.own ||
      ((uintptr_t)segs.desc & 15) || !groups_ok(grp, M, segs.max_own) ||
      (segs.max_own + grp.n_shared > 1 && (!part_o || !part_ml)) ||
      !qkv || !cos_tab || !sin_tab || (bq && (!bk || !bv)) ||
      (((uintptr_t)qkv | (uintptr_t)bq | (uintptr_t)bk | (uintptr_t)bv | (uintptr_t)arena_layer) & 15))
    return hipErrorInvalidValue;
  const float scale_log2 = 1.4426950408889634f / sqrtf((float)geom.head_dim);
  const int nkv = geom.n_kv_heads;
  const int64_t rows = segs.depth + ((int64_t)grp.n_sets * grp.n_shared + 7) / 8;
  if (rows > (int64_t)kSegRows * 65535 || nkv >= 1 << 19) return hipErrorInvalidValue;
  const dim3 grid(8 * nkv, (unsigned)std::min<int64_t>(rows, kSegRows), (unsigned)((rows + kSegRows - 1) / kSegRows));
  const DecodeArgs args{qkv, bq, bk, bv, cos_tab, sin_tab, arena_layer, geom.block_stride, n_q_heads, segs.max_own,
                        scale_log2, part_o, part_ml, out, rm.pos, grp};
  const int* base = segs.base;
  const uint32_t shape = (uint32_t)segs.stride | (uint32_t)(n_q_heads / nkv) << 8 | (uint32_t)nkv << 13;
#define AREAL_DEC(DD)                                                                              \
  attn_decode_kernel<DD><<<grid, 256, 0, s>>>(segs.desc, segs.table, base[1], base[2], base[3], base[4], base[5], base[6], \
                                               base[7], base[8], segs.depth, shape, args);
  switch (geom.head_dim) {
    case 32: AREAL_DEC(32) break;
    case 64: AREAL_DEC(64) break;
    default: AREAL_DEC(128) break;
  }
#undef AREAL_DEC
  return hipGetLastError();
}

hipError_t launch_attn_merge(hipStream_t s, int M, int head_dim, int n_q_heads, DecodeSegs segs, const float* part_o,
                             const float* part_ml, f16* out, DecodeGroups grp) {
  const int n_slots = segs.max_own + grp.n_shared;
  if (M <= 0 || segs.max_own < 1 || n_slots < 2 || n_slots > 32 || !segs.own || !part_o || !part_ml || !out ||
      (grp.n_shared > 0 && (!grp.t_start || grp.sh_chunk <= 0)) || (head_dim != 32 && head_dim != 64 && head_dim != 128))
    return hipErrorInvalidValue;
  const int64_t row_slots = (int64_t)n_q_heads * n_slots;
#define AREAL_MRG(DD)                                                                              \
  for (int r = 0; r < M; r += kSegRows)                                                            \
    attn_merge_kernel<DD><<<dim3(n_q_heads, std::min(M - r, kSegRows)), DD < 64 ? 64 : DD, 0, s>>>( \
        part_o + r * row_slots * DD, part_ml + r * row_slots * 2, segs.own + r, n_q_heads, segs.max_own, grp.n_shared, \
        grp.sh_chunk, grp.t_start ? grp.t_start + r : nullptr, out + (int64_t)r * n_q_heads * DD);
  switch (head_dim) {
    case 32: AREAL_MRG(32) break;
    case 64: AREAL_MRG(64) break;
    default: AREAL_MRG(128) break;
  }
#undef AREAL_MRG
  return hipGetLastError();
}

int attn_prefill_tile_rows(int n_q_heads, int n_kv_heads, int tiles32) {
  // tuning knob for sweeps: AREAL_PREFILL_TILE_ROWS=16|32 (read once)
  static const int forced = [] {
    const char* e = getenv("AREAL_PREFILL_TILE_ROWS");
    const int v = e ? atoi(e) : 0;
    return (v == 16 || v == 32) ? v : 0;
  }();
  // at most 3 row-groups per wave keep two work-groups resident per CU at head_dim 128
  // (7B shape, 7 query heads per KV head: 532 TFLOP/s with 16 positions against 377 with 32)
  const int G = n_q_heads / n_kv_heads;
  if (forced && (forced == 16 || G <= 8)) return forced;
  // Up to one 32-row work-group per compute unit: 16 rows where that leaves a wave fewer row-groups, one of 3 or 4 heads and
  // of 5 or 6 dealt to two work-groups (launch_attn_prefill).  One launch, head_dim 128, a prompt of 301 / 1,000 /
  // 2,000 tokens in 32 rows -> 16: 3 heads per KV head 16.9 / 37.4 / 67.2 -> 12.9 / 27.4 / 48.8 us, 4 heads 17.0 / 38.0 /
  // 67.6 -> 13.2 / 27.9 / 49.8, 6 heads 17.9 / 39.4 / 71.2 -> 13.0 / 28.1 / 52.5.  1 or 2 heads have one row-group a wave in
  // 32 rows too, and 16 only fetch every K/V tile twice as often: 12 prompts of 300 13.2 -> 14.0 and 13.9 -> 14.6.
  return G > 6 || (G > 2 && tiles32 * n_kv_heads <= 256) ? 16 : 32;
}

hipError_t launch_attn_prefill(hipStream_t s, const f16* q, const AttnWork* work, int n_work,
                               SeqState st, const f16* arena_layer, KvGeom geom, int n_q_heads, int tile,
                               f16* out) {
  if (n_work <= 0 || !geom_ok(geom, n_q_heads) || (tile != 16 && tile != 32) || (tile / 16) * (n_q_heads / geom.n_kv_heads) > 16)
    return hipErrorInvalidValue;
  const float scale_log2 = 1.4426950408889634f / sqrtf((float)geom.head_dim);
  const int G = n_q_heads / geom.n_kv_heads;
  // A launch of few work-groups lives on its longest walk: a tile's query heads go to two work-groups, whose
  // steps have one row-group a wave (32 rows: three, 16: two).  Whole prefill at the 1.5B shape, one head part of 32 or
  // 16 rows -> two of 16: one prompt of 301 tokens 2,766 -> 2,640 us, 600 3,886 -> 3,685, 1,000 5,769 -> 5,415, 2,000
  // 8,568 -> 8,020; 4 of 400 - 800 8,731 -> 8,598; 2 of 1,800 - 2,000 12,795 -> 12,406; beyond 512 work-groups of 16
  // rows it costs (8 of 500 - 700: 14,320 -> 14,390; a scoring pass of 8,192 rows 104.8 -> 107.4 ms).
  const int head_parts = tile == 16 && G >= 5 && G <= 8 && 2 * n_work * geom.n_kv_heads <= 1024 ? 2 : 1;
  const int rgw = ((tile / 16) * ((G + head_parts - 1) / head_parts) + 3) / 4;           // row-groups per wave: 1 .. 4
  const int grid = n_work * geom.n_kv_heads * head_parts;
  const int of_item = geom.n_kv_heads * head_parts, heads = (G + head_parts - 1) / head_parts;
  if ((int64_t)n_work * of_item >= (int64_t)1 << 31 || geom.n_kv_heads >= 1 << 22) return hipErrorInvalidValue;
  const uint32_t magic = of_item == 1 ? 0u : (uint32_t)((((uint64_t)1 << 32) + of_item - 1) / of_item);
  const uint32_t shape = (uint32_t)G | (uint32_t)head_parts << 5 | (uint32_t)geom.n_kv_heads << 10;
#define AREAL_PF(DD, RR)                                                                          \
  attn_prefill_kernel<DD, RR><<<grid, 256, 0, s>>>(work, q, st.table, arena_layer, magic, shape,  \
                                                   (65536u + heads - 1) / heads, tile, st.max_blocks, geom.block_stride, \
                                                   grid, scale_log2, out)
#define AREAL_PF_D(DD)                                                                            \
  switch (rgw) {                                                                                  \
    case 1: AREAL_PF(DD, 1); break;                                                               \
    case 2: AREAL_PF(DD, 2); break;                                                               \
    case 3: AREAL_PF(DD, 3); break;                                                               \
    default: AREAL_PF(DD, 4); break;                                                              \
  }
  switch (geom.head_dim) {
    case 32: AREAL_PF_D(32) break;
    case 64: AREAL_PF_D(64) break;
    default: AREAL_PF_D(128) break;
  }
#undef AREAL_PF_D
#undef AREAL_PF
  return hipGetLastError();
}

}  // namespace areal

