// dK/dV pass, several workgroups per key block (dkdv_kernel.hpp), and the
// reduction of their partials.
#include "dkdv_kernel.hpp"

namespace af {

// ---------------------------------------------------------------- splits
// Sum the splits' partial dK' and dV, undo sigma and the rotation and store
// bf16: one thread per row and 4 + 4 dims (4c.. and D/2 + 4c.., NeoX
// partners).  Bound by reading the partials once.
template <int D, int ROPE>
__global__ __launch_bounds__(256) void bwd_dkdv_reduce_kernel(BwdParams p) {
  constexpr int TPR = D / 8;
  const long long rows = (long long)p.B * p.Hkv * p.S;
  const long long row = (long long)blockIdx.x * (256 / TPR) + threadIdx.x / TPR;
  if (row >= rows) return;
  const int c = threadIdx.x % TPR, d0 = 4 * c, d1 = D / 2 + 4 * c;
  const int pos = (int)(row % p.S);
  const float inv = 1.f / p.dscale[row / p.S];
  float x[2][8] = {};   // dK', dV: dims d0.. then d1..
  for (int sp = 0; sp < p.splits; ++sp)
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      const float* src = p.part + ((size_t)(2 * sp + m) * rows + row) * D;
      const float4 a = *reinterpret_cast<const float4*>(src + d0), b = *reinterpret_cast<const float4*>(src + d1);
      const float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
      for (int i = 0; i < 8; ++i) x[m][i] += v[i];
    }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    x[0][i] *= p.scale * inv;
    x[1][i] *= inv;
  }
  const float2* t = p.table + (size_t)pos * (D / 2);
  if constexpr (ROPE == ROPE_NEOX) {
#pragma unroll
    for (int i = 0; i < 4; ++i) rotate_pair<true>(x[0][i], x[0][4 + i], t[d0 + i].x, t[d0 + i].y);
  } else if constexpr (ROPE == ROPE_INTERLEAVED) {
#pragma unroll
    for (int i = 0; i < 4; i += 2) {
      rotate_pair<true>(x[0][i], x[0][i + 1], t[(d0 + i) / 2].x, t[(d0 + i) / 2].y);
      rotate_pair<true>(x[0][4 + i], x[0][5 + i], t[(d1 + i) / 2].x, t[(d1 + i) / 2].y);
    }
  }
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    uint16_t* dst = static_cast<uint16_t*>(m == 0 ? p.dk : p.dv) + row * D;
    *reinterpret_cast<u32x2*>(dst + d0) = u32x2{pack_bf16(x[m][0], x[m][1]), pack_bf16(x[m][2], x[m][3])};
    *reinterpret_cast<u32x2*>(dst + d1) = u32x2{pack_bf16(x[m][4], x[m][5]), pack_bf16(x[m][6], x[m][7])};
  }
}

template <int D>
static int reduce(int rope, const BwdParams& p, hipStream_t st) {
  constexpr int RPB = 256 / (D / 8);
  const long long rows = (long long)p.B * p.Hkv * p.S;
  const dim3 grid((unsigned)((rows + RPB - 1) / RPB));
  if (rope == ROPE_NEOX) hipLaunchKernelGGL((bwd_dkdv_reduce_kernel<D, ROPE_NEOX>), grid, dim3(256), 0, st, p);
  else if (rope == ROPE_INTERLEAVED)
    hipLaunchKernelGGL((bwd_dkdv_reduce_kernel<D, ROPE_INTERLEAVED>), grid, dim3(256), 0, st, p);
  else hipLaunchKernelGGL((bwd_dkdv_reduce_kernel<D, ROPE_NONE>), grid, dim3(256), 0, st, p);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

int launch_bwd_dkdv_split(int D, int rope, int mask, bool alibi, int ext, const BwdParams& p, hipStream_t st) {
  const int rc = bwd_dispatch<DkdvPass<true>>(D, rope, mask, alibi, ext, p, st);
  if (rc != 0) return rc;
  return D == 64 ? reduce<64>(rope, p, st) : reduce<128>(rope, p, st);
}

}  // namespace af
