// Device code shared by the attention kernels: element types and the layout of a block, matrix-core and cross-lane
// primitives, handle resolution, and the work of one wave on one block.
#pragma once

#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include "pie_attn_split.h"
#include "pie_internal.h"

namespace pie {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------------------------------
// element types and the layout of a block
//
// A block is [K tiles of the kv heads][V tiles of the kv heads]; a tile is 16 tokens x head_dim elements.
// With v = 16 / elem_bytes elements per 16-byte vector and w = v / 4:
//   K tile: element (token t, dim c) at  (c / v) * (16 v) + t v + c % v
//           -> a vector holds v consecutive dims of one token; lane i of a 64-lane load of 1 KiB gets
//              token i % 16, dims 8 (i / 16) .. of a 4-vector-wide slab: the A operand of a 16x16x32 MFMA.
//   V tile: element (t, c) at  (((c / (16 w)) * 4 + t / 4) * 16 + c % 16) * v + ((c / 16) % w) * 4 + t % 4
//           -> a vector holds 4 consecutive tokens of dim c (and, 16-bit, of dim c + 16); lane i of a 1 KiB
//              load gets tokens 4 (i / 16) .., dim i % 16 of a 16 w-dim slab: the A operand(s) of 16x16x16 MFMAs
//              whose contraction runs over the 16 tokens of the block.
// ---------------------------------------------------------------------------------------------------

struct F32 { static constexpr int kBytes = 4; };
struct F16 { static constexpr int kBytes = 2; };
struct BF16 { static constexpr int kBytes = 2; };

__host__ __device__ __forceinline__ int32_t k_tile_index(int32_t t, int32_t c, int32_t v) {
  return (c / v) * (16 * v) + t * v + c % v;
}
__host__ __device__ __forceinline__ int32_t v_tile_index(int32_t t, int32_t c, int32_t v) {
  const int32_t w = v / 4;
  return (((c / (16 * w)) * 4 + t / 4) * 16 + c % 16) * v + ((c / 16) % w) * 4 + t % 4;
}

__device__ __forceinline__ uint16_t f32_to_bf16_bits(float x) {
  uint32_t u = __float_as_uint(x);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);  // NaN stays NaN
  u += 0x7fffu + ((u >> 16) & 1u);                                            // nearest even
  return (uint16_t)(u >> 16);
}

template <typename E> __device__ __forceinline__ float load_elem(const void* base, size_t idx);
template <> __device__ __forceinline__ float load_elem<F32>(const void* base, size_t idx) {
  return reinterpret_cast<const float*>(base)[idx];
}
template <> __device__ __forceinline__ float load_elem<F16>(const void* base, size_t idx) {
  return __half2float(reinterpret_cast<const __half*>(base)[idx]);
}
template <> __device__ __forceinline__ float load_elem<BF16>(const void* base, size_t idx) {
  return __uint_as_float((uint32_t)reinterpret_cast<const uint16_t*>(base)[idx] << 16);
}

// two consecutive elements, idx even
template <typename E> __device__ __forceinline__ float2 load_elem2(const void* base, size_t idx);
template <> __device__ __forceinline__ float2 load_elem2<F32>(const void* base, size_t idx) {
  return *reinterpret_cast<const float2*>(reinterpret_cast<const float*>(base) + idx);
}
template <> __device__ __forceinline__ float2 load_elem2<F16>(const void* base, size_t idx) {
  return __half22float2(*reinterpret_cast<const __half2*>(reinterpret_cast<const __half*>(base) + idx));
}
template <> __device__ __forceinline__ float2 load_elem2<BF16>(const void* base, size_t idx) {
  const uint32_t u = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const uint16_t*>(base) + idx);
  return make_float2(__uint_as_float(u << 16), __uint_as_float(u & 0xffff0000u));
}

template <typename E> __device__ __forceinline__ void store_elem(void* base, size_t idx, float v);
template <> __device__ __forceinline__ void store_elem<F32>(void* base, size_t idx, float v) {
  reinterpret_cast<float*>(base)[idx] = v;
}
template <> __device__ __forceinline__ void store_elem<F16>(void* base, size_t idx, float v) {
  reinterpret_cast<__half*>(base)[idx] = __float2half_rn(v);
}
template <> __device__ __forceinline__ void store_elem<BF16>(void* base, size_t idx, float v) {
  reinterpret_cast<uint16_t*>(base)[idx] = f32_to_bf16_bits(v);
}

template <typename E> __device__ __forceinline__ void store_elem2(void* base, size_t idx, float2 v);
template <> __device__ __forceinline__ void store_elem2<F32>(void* base, size_t idx, float2 v) {
  *reinterpret_cast<float2*>(reinterpret_cast<float*>(base) + idx) = v;
}
template <> __device__ __forceinline__ void store_elem2<F16>(void* base, size_t idx, float2 v) {
  *reinterpret_cast<__half2*>(reinterpret_cast<__half*>(base) + idx) = __floats2half2_rn(v.x, v.y);
}
template <> __device__ __forceinline__ void store_elem2<BF16>(void* base, size_t idx, float2 v) {
  *reinterpret_cast<uint32_t*>(reinterpret_cast<uint16_t*>(base) + idx) =
      (uint32_t)f32_to_bf16_bits(v.x) | ((uint32_t)f32_to_bf16_bits(v.y) << 16);
}

// ---------------------------------------------------------------------------------------------------
// handle -> device slot, with the checks that keep a bad table from becoming a bad address
// ---------------------------------------------------------------------------------------------------

__device__ __forceinline__ int32_t resolve_slot(int32_t handle, const int32_t* __restrict__ map, int32_t n_handles,
                                                int32_t n_gpu_blocks, int32_t n_slots, bool stage_valid,
                                                uint32_t* __restrict__ err) {
  if (handle < 0 || handle >= n_handles) {
    atomicOr(err, PIE_DEVERR_BAD_HANDLE);
    return -1;
  }
  const int32_t slot = map[handle];
  if (slot < 0 || slot >= n_slots || (slot >= n_gpu_blocks && !stage_valid)) {
    atomicOr(err, PIE_DEVERR_NOT_PRESENT);
    return -1;
  }
  return slot;
}

// The same for a slot that has been looked up already, if the handle is one.
__device__ __forceinline__ int32_t check_slot(int32_t handle, int32_t slot, int32_t n_handles, int32_t n_gpu_blocks,
                                              int32_t n_slots, bool stage_valid, uint32_t* __restrict__ err) {
  const bool known = handle >= 0 && handle < n_handles;
  const bool present = known && slot >= 0 && slot < n_slots && (slot < n_gpu_blocks || stage_valid);
  if (!present) atomicOr(err, known ? PIE_DEVERR_NOT_PRESENT : PIE_DEVERR_BAD_HANDLE);
  return present ? slot : -1;
}

// The slot of the tail block a new row goes to, or -1: which tail blocks a launch writes is its kAppend* mode.
__device__ __forceinline__ int32_t append_slot(int32_t handle, const int32_t* __restrict__ map, int32_t n_handles,
                                               int32_t n_gpu_blocks, int32_t n_slots, int32_t mode, bool report,
                                               uint32_t* __restrict__ err) {
  if (handle < 0 || handle >= n_handles) {
    if (report) atomicOr(err, PIE_DEVERR_BAD_HANDLE);
    return -1;
  }
  const int32_t slot = map[handle];
  const bool gpu_homed = slot >= 0 && slot < n_gpu_blocks;
  const bool staged = slot >= n_gpu_blocks && slot < n_slots;
  bool take = false, missing = false;
  switch (mode) {
    case kAppendPresent: take = gpu_homed || staged; missing = !take; break;
    case kAppendGpuStrict: take = gpu_homed; missing = !take; break;
    case kAppendGpuHomed: take = gpu_homed; missing = !gpu_homed && !staged && slot != -1; break;
    default: take = staged; missing = !gpu_homed && !staged; break;                    // kAppendStaged
  }
  if (missing && report) atomicOr(err, PIE_DEVERR_NOT_PRESENT);
  return take ? slot : -1;
}

constexpr int kMaxGroup = 16;         // query heads per kv head the matrix-core kernels handle (their 16 columns)
constexpr float kNegBig = -1.0e30f;   // finite stand-in for -inf as the initial running max

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

template <typename TO, typename FROM>
__device__ __forceinline__ TO bits_as(const FROM& x) {
  static_assert(sizeof(TO) == sizeof(FROM), "size mismatch");
  TO y;
  __builtin_memcpy(&y, &x, sizeof(TO));
  return y;
}

template <typename E> struct Mfma;
template <> struct Mfma<F16> {
  __device__ static f32x4 qk(const uint4& a, const uint4& b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(bits_as<f16x8>(a), bits_as<f16x8>(b), c, 0, 0, 0);
  }
  __device__ static f32x4 pv(const uint2& a, const uint2& b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x16f16(bits_as<f16x4>(a), bits_as<f16x4>(b), c, 0, 0, 0);
  }
  __device__ static uint2 round(const f32x4& p) { return bits_as<uint2>(__builtin_convertvector(p, f16x4)); }
  __device__ static f32x4 widen(const uint2& r) { return __builtin_convertvector(bits_as<f16x4>(r), f32x4); }
  // values for a residue of weights, which is zero where a weight needs no rounding: an infinity times it must not be NaN
  __device__ static uint2 bounded(const uint2& v) {
    const f16x4 most = {(_Float16)65504.f, (_Float16)65504.f, (_Float16)65504.f, (_Float16)65504.f};
    return bits_as<uint2>(__builtin_elementwise_max(__builtin_elementwise_min(bits_as<f16x4>(v), most), -most));
  }
};
template <> struct Mfma<BF16> {
  __device__ static f32x4 qk(const uint4& a, const uint4& b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(bits_as<bf16x8>(a), bits_as<bf16x8>(b), c, 0, 0, 0);
  }
  __device__ static f32x4 pv(const uint2& a, const uint2& b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(bits_as<s16x4>(a), bits_as<s16x4>(b), c, 0, 0, 0);
  }
  __device__ static uint2 round(const f32x4& p) { return bits_as<uint2>(__builtin_convertvector(p, bf16x4)); }
  __device__ static f32x4 widen(const uint2& r) {
    f32x4 f;
    f[0] = __uint_as_float(r.x << 16);
    f[1] = __uint_as_float(r.x & 0xffff0000u);
    f[2] = __uint_as_float(r.y << 16);
    f[3] = __uint_as_float(r.y & 0xffff0000u);
    return f;
  }
  __device__ static uint2 bounded(const uint2& v) { return v; }   // (an infinity among bf16 values gives NaN)
};

// Two-element dot products on the vector ALU (v_dot2_f32_f16 / v_dot2_f32_bf16): c + a.x b.x + a.y b.y with the
// products and the sum in fp32.  Used by the variant of the decode kernel that keeps off the matrix cores.
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
template <typename E> struct Dot2;
template <> struct Dot2<F16> {
  __device__ static float fma2(uint32_t a, uint32_t b, float c) {
    return __builtin_amdgcn_fdot2(bits_as<f16x2>(a), bits_as<f16x2>(b), c, false);
  }
};
template <> struct Dot2<BF16> {
  __device__ static float fma2(uint32_t a, uint32_t b, float c) {
    return __builtin_amdgcn_fdot2_f32_bf16(bits_as<bf16x2>(a), bits_as<bf16x2>(b), c, false);
  }
};

// max / sum over the four lanes i, i ^ 16, i ^ 32, i ^ 48; every lane gets the result
__device__ __forceinline__ float quad16_max(float x) {
  auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float quad16_sum(float x) {
  auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// max / sum over the 16 lanes of a row (lanes 16 r .. 16 r + 15); every lane of the row gets the result
template <int CTRL>
__device__ __forceinline__ float dpp_get(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float row16_max(float x) {
  x = fmaxf(x, dpp_get<0xB1>(x));    // quad_perm [1,0,3,2]: lane ^ 1
  x = fmaxf(x, dpp_get<0x4E>(x));    // quad_perm [2,3,0,1]: lane ^ 2
  x = fmaxf(x, dpp_get<0x141>(x));   // row_half_mirror: the other quad of the 8
  x = fmaxf(x, dpp_get<0x140>(x));   // row_mirror: the other half of the 16
  return x;
}
__device__ __forceinline__ float row16_sum(float x) {
  x += dpp_get<0xB1>(x);
  x += dpp_get<0x4E>(x);
  x += dpp_get<0x141>(x);
  x += dpp_get<0x140>(x);
  return x;
}

// sum over the wave (every lane gets it) and inclusive prefix sum over its lanes
template <int CTRL, int ROWS>
__device__ __forceinline__ int32_t dpp_add(int32_t x) {
  return x + __builtin_amdgcn_update_dpp(0, x, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ int32_t wave_scan(int32_t x) {
  x = dpp_add<0x111, 0xf>(x);        // row_shr:1
  x = dpp_add<0x112, 0xf>(x);        // row_shr:2
  x = dpp_add<0x114, 0xf>(x);        // row_shr:4
  x = dpp_add<0x118, 0xf>(x);        // row_shr:8
  x = dpp_add<0x142, 0xa>(x);        // row_bcast:15 into rows 1 and 3
  return dpp_add<0x143, 0xc>(x);     // row_bcast:31 into rows 2 and 3
}
__device__ __forceinline__ int32_t wave_sum(int32_t x) { return __builtin_amdgcn_readlane(wave_scan(x), 63); }

__device__ __forceinline__ uint4 nt_load16(const char* p) {
  const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}

// The item sizes the planning kernel chooses from when none is set: multiples of one pass of a workgroup's waves.
constexpr int kAutoParts = 7;
__host__ __device__ constexpr int32_t auto_part(int i) {
  return i == 0 ? 512 : i == 1 ? 768 : i == 2 ? 1024 : i == 3 ? 1536 : i == 4 ? 2048 : i == 5 ? 3072 : 4096;
}

// Context length as the kernels use it: never beyond what the block table can name.
__device__ __forceinline__ int32_t clamp_ctx(int32_t ctx, int32_t max_blocks) {
  const int32_t cap = max_blocks * kBlockTokens;
  return ctx > cap ? cap : ctx;
}

// One block of one wave, 16-bit caches: scores of its sixteen tokens, online softmax, accumulation of the values.
// kr, vr: the block's K and V vectors as loaded (vr is masked in place where the block holds rows beyond `limit`);
// qreg: the B operand of the first product; lane (quad, col) holds S[t_first + 4 quad + r][head col].
template <typename E, int HD, bool SPLIT>
__device__ __forceinline__ void mfma_block(uint4 (&kr)[HD / 32], uint4 (&vr)[HD / 32], const uint4 (&qreg)[HD / 32],
                                           int32_t t_first, int32_t limit, int quad, float scale_log2e, float& m, float& l,
                                           f32x4 (&o)[HD / 16]) {
  using MM = Mfma<E>;
  constexpr int NKC = HD / 32, NO = HD / 16;
  f32x4 s = {0.f, 0.f, 0.f, 0.f};             // s[r]: token t_first + 4 quad + r, head col
#pragma unroll
  for (int kc = 0; kc < NKC; ++kc) s = MM::qk(kr[kc], qreg[kc], s);
#pragma unroll
  for (int r = 0; r < 4; ++r) s[r] *= scale_log2e;
  if (t_first + kBlockTokens > limit) {       // the block holds rows beyond the context
    const int32_t t_lane = t_first + 4 * quad;
    uint32_t keep_lo = 0, keep_hi = 0;        // 16-bit masks of tokens (0, 1) and (2, 3) of this lane's quad
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const bool valid = t_lane + r < limit;
      s[r] = valid ? s[r] : -INFINITY;
      const uint32_t bits = valid ? (0xffffu << (16 * (r & 1))) : 0u;
      if (r < 2) keep_lo |= bits; else keep_hi |= bits;
    }
#pragma unroll
    for (int i = 0; i < NKC; ++i) {           // garbage rows must not reach the sum
      vr[i].x &= keep_lo; vr[i].y &= keep_hi; vr[i].z &= keep_lo; vr[i].w &= keep_hi;
    }
  }
  const float mx = quad16_max(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])));
  const float m_new = fmaxf(m, mx);
  if (__builtin_amdgcn_ballot_w64(m_new > m) != 0) {              // some head's maximum moved: rescale
    const float corr = __builtin_amdgcn_exp2f(m - m_new);
    l *= corr;
#pragma unroll
    for (int n = 0; n < NO; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) o[n][r] *= corr;
    m = m_new;
  }
  f32x4 p;
#pragma unroll
  for (int r = 0; r < 4; ++r) p[r] = __builtin_amdgcn_exp2f(s[r] - m);
  l += (p[0] + p[1]) + (p[2] + p[3]);
  const uint2 p_hi = MM::round(p);
  uint2 p_lo = make_uint2(0, 0);
  if (SPLIT) {
    const f32x4 back = MM::widen(p_hi);
    f32x4 rest;
#pragma unroll
    for (int r = 0; r < 4; ++r) rest[r] = p[r] - back[r];
    p_lo = MM::round(rest);
  }
#pragma unroll
  for (int i = 0; i < NKC; ++i) {
    const uint2 v0 = make_uint2(vr[i].x, vr[i].y), v1 = make_uint2(vr[i].z, vr[i].w);
    o[2 * i] = MM::pv(v0, p_hi, o[2 * i]);
    o[2 * i + 1] = MM::pv(v1, p_hi, o[2 * i + 1]);
    if (SPLIT) {
      o[2 * i] = MM::pv(MM::bounded(v0), p_lo, o[2 * i]);
      o[2 * i + 1] = MM::pv(MM::bounded(v1), p_lo, o[2 * i + 1]);
    }
  }
}

// A wave's share of a part.
template <typename E_, int HD_, bool SPLIT>
struct Wave16 {              // 16-bit caches: all query heads of a kv head, on the matrix cores
  using E = E_;
  static constexpr int HD = HD_, NL = HD / 32, EB = 2, kWavesPerEu = HD == 128 ? 3 : 4;
  uint4 q[NL];
  float m, l;
  f32x4 o[HD / 16];
  __device__ __forceinline__ void load_q(const char* base, size_t row0, int G, int lane, float) {
    const int col = lane & 15, quad = lane >> 4;
#pragma unroll
    for (int kc = 0; kc < NL; ++kc) {
      q[kc] = make_uint4(0, 0, 0, 0);
      if (col < G) q[kc] = *reinterpret_cast<const uint4*>(base + ((row0 + col) * HD + 32 * kc + 8 * quad) * 2);
    }
  }
  __device__ __forceinline__ void reset() {
    m = kNegBig;
    l = 0.f;
#pragma unroll
    for (int n = 0; n < HD / 16; ++n) o[n] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  __device__ __forceinline__ void block(uint4 (&kr)[NL], uint4 (&vr)[NL], int32_t t_first, int32_t limit, int lane, float scale) {
    mfma_block<E, HD, SPLIT>(kr, vr, q, t_first, limit, lane >> 4, scale, m, l, o);
  }
  __device__ __forceinline__ void to_lds(float* s_m, float* s_l, float* s_acc, int row_floats, int wave, int G, int lane) {
    const int col = lane & 15, quad = lane >> 4;
    l = quad16_sum(l);
    if (col < G) {
      if (quad == 0) {
        s_m[wave * kMaxGroup + col] = m;
        s_l[wave * kMaxGroup + col] = l;
      }
      float* row = s_acc + ((size_t)wave * G + col) * row_floats + 4 * quad;
#pragma unroll
      for (int n = 0; n < HD / 16; ++n) *reinterpret_cast<f32x4*>(row + 16 * n) = o[n];
    }
  }
};

// One block of one wave and one query head, fp32 caches.  Lane (quad, row) holds, of the K tile, token `row`'s
// 4-dim vectors 4 i + quad; of the V tile, dim 16 n + row of the tokens 4 quad .. 4 quad + 3.  qf is scaled.
template <int HD>
__device__ __forceinline__ void f32_block(const uint4 (&kr)[HD / 16], const uint4 (&vr)[HD / 16], const float (&qf)[HD / 16][4],
                                          int32_t t_first, int32_t limit, int lane, float& m, float& l, float (&acc)[HD / 16]) {
  const int row = lane & 15, quad = lane >> 4;
  float d = 0.f;
#pragma unroll
  for (int i = 0; i < HD / 16; ++i) {
    d = fmaf(qf[i][0], __uint_as_float(kr[i].x), d);
    d = fmaf(qf[i][1], __uint_as_float(kr[i].y), d);
    d = fmaf(qf[i][2], __uint_as_float(kr[i].z), d);
    d = fmaf(qf[i][3], __uint_as_float(kr[i].w), d);
  }
  float s = quad16_sum(d);                      // score of token t_first + row, on all four lanes of the token
  if (t_first + row >= limit) s = -INFINITY;
  const float m_new = fmaxf(m, row16_max(s));
  const float corr = __builtin_amdgcn_exp2f(m - m_new);
  const float p = __builtin_amdgcn_exp2f(s - m_new);
  l = l * corr + p;                             // this lane's token only; summed over the row at the end
  m = m_new;
  float pt[4];
#pragma unroll
  for (int tt = 0; tt < 4; ++tt) pt[tt] = __shfl(p, 4 * quad + tt, 64);
#pragma unroll
  for (int n = 0; n < HD / 16; ++n) {
    const uint32_t w[4] = {vr[n].x, vr[n].y, vr[n].z, vr[n].w};
    float x = acc[n] * corr;
#pragma unroll
    for (int tt = 0; tt < 4; ++tt) {
      const bool valid = t_first + 4 * quad + tt < limit;        // garbage rows must not reach the sum
      x = fmaf(pt[tt], valid ? __uint_as_float(w[tt]) : 0.f, x);
    }
    acc[n] = x;
  }
}

// ---- storing a sequence's newest key and value rows into its tail block --------------------------------------

// by a workgroup
__device__ __forceinline__ void append_rows(const AppendArgs& a, int32_t b, int32_t layer) {
  const int32_t ctx = a.ctx[b];
  if (ctx <= 0) return;
  const int32_t pos = ctx - 1;
  const int32_t j = pos / a.block_tokens;
  if (j >= a.max_blocks) {
    if (threadIdx.x == 0) atomicOr(a.err, PIE_DEVERR_BAD_HANDLE);
    return;
  }
  __shared__ int32_t s_slot;
  if (threadIdx.x == 0)
    s_slot = append_slot(a.table[(size_t)b * a.max_blocks + j], a.map + (size_t)layer * a.map_stride, a.n_handles,
                         a.n_gpu_blocks, a.n_slots, a.mode, true, a.err);
  __syncthreads();
  const int32_t slot = s_slot;
  if (slot < 0) return;
  // one 16-byte vector of a key row goes to one vector of the K tile; a value row is scattered element by
  // element over the V tile's token-quad vectors
  const int32_t v = 16 / a.elem_bytes;
  const int32_t vec_per_row = a.head_dim / v;
  const int32_t tile_bytes = kBlockTokens * a.head_dim * a.elem_bytes;
  char* blk = a.kv_layer + layer * a.kv_layer_stride + (size_t)slot * a.block_bytes;
  const char* k_new = a.k_new + layer * a.new_layer_stride;
  const char* v_new = a.v_new + layer * a.new_layer_stride;
  const size_t v_off = a.block_bytes / 2;
  const int32_t t = pos % kBlockTokens;
  const int32_t n_vec = a.n_kv_heads * vec_per_row;
  for (int32_t i = threadIdx.x; i < n_vec; i += blockDim.x) {
    const int32_t g = i / vec_per_row, cv = i % vec_per_row;
    const size_t src = ((size_t)b * a.n_kv_heads + g) * a.head_dim * a.elem_bytes + (size_t)cv * 16;
    const size_t dst = (size_t)g * tile_bytes + (size_t)k_tile_index(t, cv * v, v) * a.elem_bytes;
    *reinterpret_cast<uint4*>(blk + dst) = *reinterpret_cast<const uint4*>(k_new + src);
  }
  const int32_t n_el = a.n_kv_heads * a.head_dim;
  for (int32_t i = threadIdx.x; i < n_el; i += blockDim.x) {
    const int32_t g = i / a.head_dim, c = i % a.head_dim;
    const size_t src = ((size_t)b * a.n_kv_heads + g) * a.head_dim + c;
    const size_t dst = v_off + (size_t)g * tile_bytes + (size_t)v_tile_index(t, c, v) * a.elem_bytes;
    if (a.elem_bytes == 2)
      *reinterpret_cast<uint16_t*>(blk + dst) = reinterpret_cast<const uint16_t*>(v_new)[src];
    else
      *reinterpret_cast<uint32_t*>(blk + dst) = reinterpret_cast<const uint32_t*>(v_new)[src];
  }
}

}  // namespace pie
