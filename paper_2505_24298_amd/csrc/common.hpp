// Shared device-side types and small helpers for the gfx950 kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace areal {

// Matrix-core operands (weights, activations, K/V) are IEEE half precision; all
// accumulation, the residual stream, softmax statistics and logits are float32.
typedef _Float16 f16;
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16_in;   // only as an input format of parameter sets
typedef float  f32x4 __attribute__((ext_vector_type(4)));
typedef float  f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kWave = 64;
constexpr int kBlockTokens = 16;   // tokens per KV block

__device__ __forceinline__ float h2f(f16 x) { return (float)x; }
__device__ __forceinline__ f16 f2h(float x) { return (f16)x; }   // round to nearest even
// Activations and K/V on their way to the matrix cores: magnitudes beyond the half range
// saturate to +-65504 instead of turning into infinities (NaN stays NaN).
__device__ __forceinline__ f16 f2h_sat(float x) {
  return (f16)__builtin_amdgcn_fmed3f(x, -65504.0f, 65504.0f);
}

// 16-byte global load of 8 halves
__device__ __forceinline__ f16x8 ld8(const f16* p) { return *reinterpret_cast<const f16x8*>(p); }

// f(value of this lane, value of lane ^ O), O = 32, 16 by a swap of lane halves or rows, without the LDS crossbar that
// __shfl_xor goes through (about 60 ns each); f has to be commutative.
template <int O, class F>
__device__ __forceinline__ float xor_lanes(float v, F f) {
  static_assert(O == 32 || O == 16, "lane distance");
  const uint32_t x = __builtin_bit_cast(uint32_t, v);
  if constexpr (O == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    const uint32_t a = r[0], b = r[1];
    return f(__builtin_bit_cast(float, a), __builtin_bit_cast(float, b));
  } else {
    const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    const uint32_t a = r[0], b = r[1];
    return f(__builtin_bit_cast(float, a), __builtin_bit_cast(float, b));
  }
}
// Value of the lane that a DPP control names (within the 16 lanes of a row; every lane reads an existing one).
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp((int)__builtin_bit_cast(uint32_t, v), CTRL, 0xF, 0xF, false));
}
// All 64 lanes folded by a commutative f, every lane gets the result, with the pairs (and so the roundings) of a butterfly
// over lane distances 32, 16, 8, 4, 2, 1: after a step both lanes of a pair hold the same value, so rotations of a
// row by 8 and 4 lanes stand for exchanges at these distances.
template <class F>
__device__ __forceinline__ float wave_fold(float v, F f) {
  v = xor_lanes<32>(v, f);
  v = xor_lanes<16>(v, f);
  v = f(v, dpp<0x128>(v));      // row_ror:8
  v = f(v, dpp<0x124>(v));      // row_ror:4
  v = f(v, dpp<0x4E>(v));       // quad_perm 2 3 0 1
  v = f(v, dpp<0xB1>(v));       // quad_perm 1 0 3 2
  return v;
}
__device__ __forceinline__ float wave_sum(float v) {
  return wave_fold(v, [](float a, float b) { return a + b; });
}
__device__ __forceinline__ float wave_max(float v) {
  return wave_fold(v, [](float a, float b) { return fmaxf(a, b); });
}

// Value of lane ^ 1 (DPP).
__device__ __forceinline__ uint32_t dpp_xor1(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xB1, 0xF, 0xF, false);
}

// A correctly rounded quotient, in every tile: the hardware's reciprocal (1 ulp) times z is another half now and then.
__device__ __forceinline__ float silu_f(float z) { return z / (1.0f + __expf(-z)); }

// Base and size of a range for buffer loads (raw, 32-bit offsets, reads past the end return zero).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00027000);
}
// 16 bytes per lane, HBM -> LDS: lane i of the wave fetches byte lane_off + wave_off of src and writes
// dst_wave_base + i*16.  Buffer loads, not global ones: those are FLAT instructions, after which the
// compiler's wait insertion waits for ALL LDS reads in flight (lgkmcnt(0)) wherever it needs one of
// them, so that fragment reads ahead of their use gain nothing.
__device__ __forceinline__ void dma16(__amdgpu_buffer_rsrc_t src, int lane_off, int wave_off, void* dst_wave_base) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(src, (__attribute__((address_space(3))) void*)dst_wave_base, 16,
                                           lane_off, wave_off, 0, 0);
}

// 16 (8) bytes per lane at byte `off` of a buffer; past its end: zero, no access.
typedef uint32_t b128_t __attribute__((ext_vector_type(4)));
typedef uint32_t b64_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ f16x8 buf8(__amdgpu_buffer_rsrc_t r, int off) {
  return __builtin_bit_cast(f16x8, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}
__device__ __forceinline__ f32x4 buf4f(__amdgpu_buffer_rsrc_t r, int off) {
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}
__device__ __forceinline__ f16x4 buf4(__amdgpu_buffer_rsrc_t r, int off) {
  return __builtin_bit_cast(f16x4, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}
__device__ __forceinline__ int buf1(__amdgpu_buffer_rsrc_t r, int off) {
  return (int)__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
}

// Where a kernel's last parameter lies in its arguments (one after the other, each at its own alignment), and its type.
template <class Kernel>
struct LastParam;
template <class... P>
struct LastParam<void(P...)> {
  template <class A, class... R>
  static constexpr int offset_of(int at) {
    at = (at + (int)alignof(A) - 1) / (int)alignof(A) * (int)alignof(A);
    if constexpr (sizeof...(R) == 0) return at;
    else return offset_of<R...>(at + (int)sizeof(A));
  }
  static constexpr int offset = offset_of<P...>(0);
  template <class A, class... R>
  struct Last : Last<R...> {};
  template <class A>
  struct Last<A> { typedef A type; };
  typedef typename Last<P...>::type type;
};
static_assert(LastParam<void(void*, int, double)>::offset == 16 && LastParam<void(void*, int, int, double)>::offset == 16 &&
              LastParam<void(void*, char, short, float)>::offset == 12, "an argument starts at its alignment");
// The last parameter of Kernel (the type of the kernel that calls this), a struct by value, read here and not on entry: the reads
// of a by-value parameter all start there, and a wave that needs few of them first waits for all.
template <class Kernel>
__device__ __forceinline__ typename LastParam<Kernel>::type late_args() {
  typedef typename LastParam<Kernel>::type T;
  typedef const __attribute__((address_space(4))) T* ptr;
  return *(const T*)(ptr)((const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr() +
                          LastParam<Kernel>::offset);
}

// Every LDS read of this wave has returned (s_waitcnt with only lgkmcnt constrained).
__device__ __forceinline__ void wait_lgkmcnt0() { __builtin_amdgcn_s_waitcnt(0xC07F); }

__device__ __forceinline__ void wait_vmcnt(int n) {
  // s_waitcnt with only vmcnt constrained (gfx9 encoding: vmcnt = [15:14]:[3:0]); the counter
  // has 6 bits, so a larger bound is tightened to 63
  switch (n < 63 ? n : 63) {
#define AREAL_W(N) case N: __builtin_amdgcn_s_waitcnt(((N) & 15) | (((N) >> 4) << 14) | 0x0F70); break;
#define AREAL_W8(B) AREAL_W(B) AREAL_W(B + 1) AREAL_W(B + 2) AREAL_W(B + 3) AREAL_W(B + 4) AREAL_W(B + 5) \
                    AREAL_W(B + 6) AREAL_W(B + 7)
    AREAL_W8(0) AREAL_W8(8) AREAL_W8(16) AREAL_W8(24) AREAL_W8(32) AREAL_W8(40) AREAL_W8(48) AREAL_W8(56)
#undef AREAL_W8
#undef AREAL_W
    default: __builtin_amdgcn_s_waitcnt(0x0F70); break;
  }
}

// ---- paged KV arena addressing --------------------------------------------
// arena = [layer][block][kv_head][K tile | V tile], tiles of 16*d halves.
//   K tile: [c 0..d/32-1][g 0..3][token 0..15][e 0..7] holding K[token][dim 32c+8g+e]:
//           the 16 bytes at (c, lane = g*16 + token) are lane's A-operand
//           registers of MFMA c of the 16x16x32 score product.
//   V tile: [c 0..d/32-1][lane 0..63][e 0..7] with lane = g*16 + j and
//           e = 4*(n&1) + t holding V[token 4g+t][dim 16n+j], n = 2c + (e>>2):
//           the 16 bytes at (c, lane) are lane's B-operand registers of the
//           16x16x16 MFMAs n = 2c, 2c+1 that multiply probabilities by values,
//           and one load instruction of a wave (fixed c) reads 1 KiB in a row.
struct KvGeom {
  int n_kv_heads, head_dim;
  int64_t layer_stride;   // elements between layers = n_blocks * block_stride
  int block_stride;       // elements per block of one layer = n_kv_heads * 2 * 16 * d
};
__device__ __forceinline__ int64_t kv_tile_off(const KvGeom& g, int block, int kvh, int is_v) {
  return (int64_t)block * g.block_stride + (int64_t)(kvh * 2 + is_v) * (kBlockTokens * g.head_dim);
}
__device__ __forceinline__ int k_tile_index(int token, int dim) {
  return (((dim >> 5) * 64 + ((dim >> 3) & 3) * 16 + token) * 8) + (dim & 7);
}
__device__ __forceinline__ int v_tile_index(int head_dim, int token, int dim) {
  (void)head_dim;
  int g = token >> 2, t = token & 3, n = dim >> 4, j = dim & 15;
  return (((n >> 1) * 64 + g * 16 + j) * 8) + (n & 1) * 4 + t;
}

}  // namespace areal
