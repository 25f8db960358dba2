// What the GEMM kernels share: the swizzled LDS tile rows, FP8 weight widening, the row
// statistics of a folded LayerNorm and the epilogue of four consecutive output columns.
#pragma once
#include <type_traits>

#include "nt_common.h"
#include "nt_kernels.h"

namespace nt {
namespace {

constexpr int ROWB = 128;           // bytes of K per tile row per step
// Byte offset of 16-byte chunk `ch` of tile row `row` in a swizzled LDS tile.
__device__ __forceinline__ int swz(int row, int ch) { return row * ROWB + ((ch ^ (row & 7)) << 4); }
// Same for the 64-byte rows of an FP8 weight tile (64 k-values per step): rows r, r+4,
// r+8, r+12 fall on the same banks, so the chunk position is XORed with bits 2..3 of
// the row and 16 consecutive rows read at one chunk hit 16 distinct bank groups.
constexpr int ROWB8 = 64;
__device__ __forceinline__ int swz8(int row, int ch) { return row * ROWB8 + ((ch ^ ((row >> 2) & 3)) << 4); }

// Eight FP8 E4M3 weights (two 32-bit words, k in byte order) as eight fp16 values of an
// MFMA operand.  Every E4M3 value is exact in fp16, so the conversion loses nothing.
template <bool HI>
__device__ __forceinline__ unsigned f8x2(unsigned w) {
  return __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w, 1.0f, HI));
}
__device__ __forceinline__ u32x4 f8_to_f16x8(unsigned w0, unsigned w1) {
  return u32x4{f8x2<false>(w0), f8x2<true>(w0), f8x2<false>(w1), f8x2<true>(w1)};
}

// Sum and sum of squares of the eight (fp16/bf16) or four (fp32) values of one 16-byte
// operand fragment, each taken relative to the row's shift c (one of the row's own
// values), added into s and q in fp32: the row statistics of a folded LayerNorm.  With
// the shift, the variance (q/K - (s/K)^2) no longer cancels when the row's mean is large
// against its spread: the deviations from c are of the size of the spread.  For fp16 the
// deviation is formed in fp16 (exact whenever x and c are within a factor of two, which is
// where cancellation would matter), then squared and summed by fdot2 in fp32.
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
template <typename T>
__device__ __forceinline__ void frag_stats(const u32x4& a, T c, float& s, float& q) {
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    if constexpr (std::is_same<T, f16>::value) {
      // the word is copied out first: a bit_cast of the vector element itself read word 0
      const unsigned u = a[w];
      const half2v h = __builtin_bit_cast(half2v, u) - half2v{c, c};
      s = __builtin_amdgcn_fdot2(h, half2v{(_Float16)1.0f, (_Float16)1.0f}, s, false);
      q = __builtin_amdgcn_fdot2(h, h, q, false);
    } else if constexpr (std::is_same<T, bf16>::value) {
      const float cf = to_f32(c);
      const float lo = __uint_as_float(a[w] << 16) - cf, hi = __uint_as_float(a[w] & 0xffff0000u) - cf;
      s += lo;
      s += hi;
      q = fmaf(lo, lo, q);
      q = fmaf(hi, hi, q);
    } else {
      const float x = __uint_as_float(a[w]) - to_f32(c);
      s += x;
      q = fmaf(x, x, q);
    }
  }
}

// Applies the epilogue MODE to up to 4 consecutive columns n..n+3 of row m (n % 4 == 0).
// With OPS, it adds the bias (if any) and, for EPI_RESID, the residual itself; without,
// the caller has added both (an EPI_RESID group is then a plain store).  The mode is a
// template argument so that a tile's unrolled groups carry only their own mode's code.
// fp32 output (out_f32) goes with EPI_STORE only.  d, dh and ldc are multiples of 4 in
// every mode that scatters, so the 4 columns never straddle a head or a K/V boundary and
// land on 4 consecutive destination elements.
template <typename T, int MODE, bool OPS>
__device__ __forceinline__ void epilogue4(const GemmEpi& e, int m, int n, int N, float4 v4, int t_slot) {
  float v[4] = {v4.x, v4.y, v4.z, v4.w};
  const int cnt = min(4, N - n);
  if constexpr (OPS) {
    if (e.bias) {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (k < cnt) v[k] += e.bias[n + k];
    }
  }
  const bool vec = cnt == 4 && (e.ldc & 3) == 0;
  if constexpr (MODE == EPI_STORE) {
    if (e.out_f32) {
      const int mo = e.out_map ? e.sent_list[m / e.beam] * e.beam + m % e.beam : m;
      float* o = static_cast<float*>(e.out) + (size_t)mo * e.ldc + n;
      if (vec) {
        *reinterpret_cast<float4*>(o) = make_float4(v[0], v[1], v[2], v[3]);
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (k < cnt) o[k] = v[k];
      }
      return;
    }
  }
  T* o = nullptr;
  if constexpr (MODE == EPI_STORE) {
    o = static_cast<T*>(e.out) + (size_t)m * e.ldc + n;
  } else if constexpr (MODE == EPI_RELU) {
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = fmaxf(v[k], 0.f);
    o = static_cast<T*>(e.out) + (size_t)m * e.ldc + n;
  } else if constexpr (MODE == EPI_RESID) {
    if constexpr (OPS) {
      const T* r = static_cast<const T*>(e.resid) + (size_t)m * e.ldc + n;
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (k < cnt) v[k] += to_f32(r[k]);
    }
    o = static_cast<T*>(e.out) + (size_t)m * e.ldc + n;
  } else if constexpr (MODE == EPI_SELF_QKV) {
    if (n < e.d) {
      o = static_cast<T*>(e.out) + (size_t)m * e.ldc + n;
    } else {
      int c = n - e.d;
      const int kv = c >= e.d;
      c -= kv * e.d;
      const int h = c / e.dh, x = c - h * e.dh;
      const int p = e.sent_list[m / e.beam] * e.beam + m % e.beam;
      const size_t idx = ((size_t)(p * e.H + h) * e.Tcap + t_slot) * e.dh + x;
      if (e.kv_f8) {   // E4M3 cache: the 4 columns as 4 bytes, one 32-bit store (idx % 4 == 0)
        uint8_t* o8 = static_cast<uint8_t*>(kv ? e.vcache : e.kcache) + idx;
        if (cnt == 4) {
          *reinterpret_cast<uint32_t*>(o8) = (uint32_t)e4m3_rne(v[0]) | ((uint32_t)e4m3_rne(v[1]) << 8) |
                                             ((uint32_t)e4m3_rne(v[2]) << 16) | ((uint32_t)e4m3_rne(v[3]) << 24);
        } else {
#pragma unroll
          for (int k = 0; k < 4; ++k)
            if (k < cnt) o8[k] = e4m3_rne(v[k]);
        }
        return;
      }
      o = static_cast<T*>(kv ? e.vcache : e.kcache) + idx;
    }
  } else {
    static_assert(MODE == EPI_CROSS_KV, "epilogue mode");
    const int j = n / (2 * e.d);
    int c = n - j * 2 * e.d;
    const int kv = c >= e.d;
    c -= kv * e.d;
    const int h = c / e.dh, x = c - h * e.dh;
    const int b = m / e.S, s = m - b * e.S;
    o = static_cast<T*>(e.cross) + ((((size_t)j * 2 + kv) * e.B + b) * e.H + h) * (size_t)e.S * e.dh +
        (size_t)s * e.dh + x;
  }
  if (vec || (MODE >= EPI_SELF_QKV && cnt == 4)) {
    if constexpr (sizeof(T) == 2) {
      T t4[4] = {from_f32<T>(v[0]), from_f32<T>(v[1]), from_f32<T>(v[2]), from_f32<T>(v[3])};
      *reinterpret_cast<uint2*>(o) = *reinterpret_cast<const uint2*>(t4);
    } else {
      *reinterpret_cast<float4*>(o) = make_float4(v[0], v[1], v[2], v[3]);
    }
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (k < cnt) o[k] = from_f32<T>(v[k]);
  }
}

// s_waitcnt immediate that waits until at most `vm` vector-memory operations of this wave
// are outstanding (expcnt / lgkmcnt left unconstrained).
__host__ __device__ constexpr int vmcnt_imm(int vm) { return (vm & 0xF) | ((vm >> 4) << 14) | (0x7 << 4) | (0xF << 8); }

#define NT_LDS(p) ((__attribute__((address_space(3))) void*)(p))

}  // namespace
}  // namespace nt
