// Pieces of the fp32 kernels: 16-row tiles on the fp32 matrix instruction
// (v_mfma_f32_16x16x4_f32: fp32 products and sums, as the vector unit's FMA).
//
// A workgroup is F32_NW waves on one 16-row output tile; the waves take the
// tiles of the contracted side in turn and their partial results merge in LDS
// at the end, so that short sequences fill the chip too: 16 rows per workgroup
// instead of one row per thread of 64 brought the smallest shapes from 4
// workgroups to 64 waves.
//
// Register layouts (lane l: lq = l % 16, g = l / 16):
//   A (16 x 4): lane = row lq, k-index g;  B (4 x 16): lane = column lq, k-index g;
//   C (16 x 16): element r of lane l = row 4 g + r, column lq.
// A contraction over the head dimension gives lane group g the dimensions
// {g D/8 .. +D/8} and {D/2 + g D/8 .. +D/8}, D/4 in all, so that both partners
// of every rotation pair (either pairing) sit in one lane.  A contraction over
// tile rows gives step s the row 4 g + s, which is where the C layout of the
// scores already holds it.
#pragma once
#include "common.hpp"

namespace af {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int F32_NW = 4;    // waves per workgroup
constexpr int F32_T = 16;    // rows per tile

__device__ __forceinline__ f32x4 mfma16_f32(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// The lane's D/4 values of one row (16-byte loads).
template <int D>
__device__ __forceinline__ void f32_load_row(float (&x)[D / 4], const float* __restrict__ row, int g) {
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 0; i < D / 8; i += 4) {
      const float4 v = *reinterpret_cast<const float4*>(row + h * (D / 2) + g * (D / 8) + i);
      x[h * (D / 8) + i] = v.x;
      x[h * (D / 8) + i + 1] = v.y;
      x[h * (D / 8) + i + 2] = v.z;
      x[h * (D / 8) + i + 3] = v.w;
    }
}

// The (cos, sin) entries of the lane's pairs of one position.
template <int D, int ROPE>
__device__ __forceinline__ void f32_load_cs(float (&cs)[D / 4], const float2* __restrict__ trow, int g) {
  if constexpr (ROPE == ROPE_NONE) return;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    // NeoX: pairs g D/8 .. +D/8; interleaved: D/16 pairs in each half of the row
    const float* t = reinterpret_cast<const float*>(
        ROPE == ROPE_NEOX ? trow + g * (D / 8) + h * (D / 16) : trow + h * (D / 4) + g * (D / 16));
#pragma unroll
    for (int i = 0; i < D / 8; i += 4) {
      const float4 v = *reinterpret_cast<const float4*>(t + i);
      cs[h * (D / 8) + i] = v.x;
      cs[h * (D / 8) + i + 1] = v.y;
      cs[h * (D / 8) + i + 2] = v.z;
      cs[h * (D / 8) + i + 3] = v.w;
    }
  }
}

template <int D, int ROPE>
__device__ __forceinline__ void f32_rotate(float (&x)[D / 4], const float (&cs)[D / 4]) {
  if constexpr (ROPE == ROPE_NEOX) {
#pragma unroll
    for (int i = 0; i < D / 8; ++i) rotate_pair<false>(x[i], x[D / 8 + i], cs[2 * i], cs[2 * i + 1]);
  } else if constexpr (ROPE == ROPE_INTERLEAVED) {
#pragma unroll
    for (int i = 0; i < D / 4; i += 2) rotate_pair<false>(x[i], x[i + 1], cs[i], cs[i + 1]);
  }
}

// <a, b> over the head dimension for 16 x 16 rows: two chains of D/8 steps.
template <int D>
__device__ __forceinline__ f32x4 f32_dot(const float (&a)[D / 4], const float (&b)[D / 4]) {
  f32x4 s0 = f32x4{}, s1 = f32x4{};
#pragma unroll
  for (int i = 0; i < D / 4; i += 2) {
    s0 = mfma16_f32(a[i], b[i], s0);
    s1 = mfma16_f32(a[i + 1], b[i + 1], s1);
  }
  return s0 + s1;
}

// The transposed operand X^T (dims x tile rows) of a tile in global memory:
// element s MT + mt = row row0 + 4 g + s (clamped to S - 1), dim 16 mt + lq.
template <int D>
__device__ __forceinline__ void f32_load_t(float (&x)[D / 4], const float* __restrict__ X, int row0, int S, int lq,
                                           int g) {
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const float* r = X + (size_t)min(row0 + 4 * g + s, S - 1) * D + lq;
#pragma unroll
    for (int mt = 0; mt < D / 16; ++mt) x[s * (D / 16) + mt] = r[16 * mt];
  }
}

// The same operand of a tile held in the row layout (a rotated one), through
// this wave's F32_T * (D + 4) floats of LDS.  A wave's LDS accesses complete
// in order, so no barrier is needed, only that the compiler keeps them so.
template <int D>
__device__ __forceinline__ void f32_transpose(float (&t)[D / 4], const float (&x)[D / 4], float* __restrict__ lds,
                                              int lq, int g) {
  asm volatile("" ::: "memory");
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 0; i < D / 8; i += 4)
      *reinterpret_cast<float4*>(lds + lq * (D + 4) + h * (D / 2) + g * (D / 8) + i) =
          float4{x[h * (D / 8) + i], x[h * (D / 8) + i + 1], x[h * (D / 8) + i + 2], x[h * (D / 8) + i + 3]};
  __builtin_amdgcn_wave_barrier();
  asm volatile("" ::: "memory");
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int mt = 0; mt < D / 16; ++mt) t[s * (D / 16) + mt] = lds[(4 * g + s) * (D + 4) + 16 * mt + lq];
  asm volatile("" ::: "memory");
  __builtin_amdgcn_wave_barrier();
}

// acc^T (dims x 16) += X^T (dims x tile rows) P (tile rows x 16).
template <int D>
__device__ __forceinline__ void f32_accumulate(f32x4 (&acc)[D / 16], const float (&t)[D / 4], const float (&p)[4]) {
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int mt = 0; mt < D / 16; ++mt) acc[mt] = mfma16_f32(t[s * (D / 16) + mt], p[s], acc[mt]);
}

// Reductions over the four lane groups (the lanes that share lq).
__device__ __forceinline__ float groups_max(float x) {
  x = fmaxf(x, __shfl_xor(x, 16, 64));
  return fmaxf(x, __shfl_xor(x, 32, 64));
}
__device__ __forceinline__ float groups_sum(float x) {
  x += __shfl_xor(x, 16, 64);
  return x + __shfl_xor(x, 32, 64);
}

// Merging the waves' partial accumulators: every wave puts its own, and after
// a barrier wave w < D/32 gets the weighted sum of the dims tiles w and
// w + D/32 (NeoX partners: the inverse rotation needs both).
template <int D>
constexpr int F32_XCH = F32_NW * (D / 4) * 64;   // floats

template <int D>
__device__ __forceinline__ void f32_put(float* __restrict__ xch, const f32x4 (&acc)[D / 16], int wave, int lane) {
#pragma unroll
  for (int mt = 0; mt < D / 16; ++mt)
    *reinterpret_cast<f32x4*>(xch + ((wave * (D / 16) + mt) * 64 + lane) * 4) = acc[mt];
}

template <int D>
__device__ __forceinline__ void f32_get(f32x4 (&out)[2], const float* __restrict__ xch, const float (&w)[F32_NW],
                                        int wave, int lane) {
  out[0] = out[1] = f32x4{};
#pragma unroll
  for (int j = 0; j < F32_NW; ++j)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int mt = wave + h * (D / 32);
      out[h] += w[j] * *reinterpret_cast<const f32x4*>(xch + ((j * (D / 16) + mt) * 64 + lane) * 4);
    }
}

// Inverse rotation of the two dims tiles of f32_get: out[h][r] is dim
// 16 (wave + h D/32) + 4 g + r of the position whose table row is trow.
template <int D, int ROPE>
__device__ __forceinline__ void f32_rotate_back(f32x4 (&out)[2], const float2* __restrict__ trow, int wave, int g) {
  if constexpr (ROPE == ROPE_NEOX) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float2 cs = trow[16 * wave + 4 * g + r];
      float a = out[0][r], b = out[1][r];
      rotate_pair<true>(a, b, cs.x, cs.y);
      out[0][r] = a;
      out[1][r] = b;
    }
  } else if constexpr (ROPE == ROPE_INTERLEAVED) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int r = 0; r < 4; r += 2) {
        const float2 cs = trow[8 * (wave + h * (D / 32)) + 2 * g + r / 2];
        float a = out[h][r], b = out[h][r + 1];
        rotate_pair<true>(a, b, cs.x, cs.y);
        out[h][r] = a;
        out[h][r + 1] = b;
      }
  }
}

template <int D>
__device__ __forceinline__ void f32_store(float* __restrict__ row, const f32x4 (&out)[2], int wave, int g) {
#pragma unroll
  for (int h = 0; h < 2; ++h) *reinterpret_cast<f32x4*>(row + 16 * (wave + h * (D / 32)) + 4 * g) = out[h];
}

}  // namespace af
