// fp32 debug forward: the same method as the bf16 MFMA kernel (RoPE on the
// query once and on every key tile, post-matmul modifications, online softmax
// over key tiles, masked tiles skipped) in fp32 arithmetic throughout.
//
// One workgroup per 16 query rows; its waves take every F32_NW-th 16-key tile
// and merge their (max, sum, O) at the end (fp32_tiles.hpp).  Debug shapes are
// short, so what bounds it is the latency of the longest wave's chain of
// tiles; each tile's K, V and table loads are issued one tile ahead.
// Against one query row per thread of 64 with broadcast LDS reads: B1 H2 S128
// D64 (interleaved, causal) 95 -> 7.6 us; B1 H32/8 S2048 D128 (NeoX, causal)
// 9.4 -> 0.91 ms.
#include "fp32_tiles.hpp"
#include "launch.hpp"

namespace af {

template <int D, int ROPE, int MASK, bool ALIBI>
__global__ __launch_bounds__(64 * F32_NW) void fwd_fp32_kernel(FwdParams p) {
  constexpr int DL = D / 4, MT = D / 16;
  __shared__ __attribute__((aligned(16))) float xch[F32_XCH<D>];
  __shared__ float stat[2][F32_NW][16];
  const int tid = threadIdx.x, lane = tid & 63, lq = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int S = p.S;
  const int BH = p.B * p.H;
  const int nqb = (S + F32_T - 1) / F32_T;
  const int bh = blockIdx.x % BH;
  const int qb = nqb - 1 - (int)(blockIdx.x / BH);   // the longest causal rows first
  const int b = bh / p.H, h = bh % p.H;
  const size_t kv = (size_t)(b * p.Hkv + h / (p.H / p.Hkv)) * S * D;
  const int m0 = qb * F32_T, m = m0 + lq, mc = min(m, S - 1);
  const float* __restrict__ Q = static_cast<const float*>(p.q) + (size_t)bh * S * D;
  const float* __restrict__ K = static_cast<const float*>(p.k) + kv;
  const float* __restrict__ V = static_cast<const float*>(p.v) + kv;

  const float c2 = p.scale * kLog2e;
  const float slope2 = ALIBI ? p.slopes[h] * kLog2e : 0.f;
  const int W = p.window;
  int t = wave, t_end = nqb;
  if constexpr (MASK != MASK_NONE) t_end = qb + 1;
  if constexpr (MASK == MASK_SLIDING_WINDOW) t += max(0, m0 - W + 1) / F32_T;

  float k[DL], cs[DL], vt[DL];   // the tile in flight; rows past S: row S-1, masked
  auto load = [&](int tile) {
    const int n = min(tile * F32_T + lq, S - 1);
    f32_load_row<D>(k, K + (size_t)n * D, g);
    f32_load_cs<D, ROPE>(cs, p.table + (size_t)n * (D / 2), g);
    f32_load_t<D>(vt, V, tile * F32_T, S, lq, g);
  };
  if (t < t_end) load(t);
  float q[DL];
  {
    float qc[DL];
    f32_load_row<D>(q, Q + (size_t)mc * D, g);
    f32_load_cs<D, ROPE>(qc, p.table + (size_t)mc * (D / 2), g);
    f32_rotate<D, ROPE>(q, qc);
  }

  f32x4 acc[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) acc[i] = f32x4{};
  float m_run = -INFINITY, l_run = 0.f;   // l_run: this lane's part
  for (; t < t_end; t += F32_NW) {
    const int n0 = t * F32_T + 4 * g;     // key of element 0
    float kr[DL], v[DL];
#pragma unroll
    for (int i = 0; i < DL; ++i) {
      kr[i] = k[i];
      v[i] = vt[i];
    }
    f32_rotate<D, ROPE>(kr, cs);
    if (t + F32_NW < t_end) load(t + F32_NW);
    const f32x4 s = f32_dot<D>(kr, q);
    float x[4], mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int n = n0 + r;
      x[r] = ALIBI ? __builtin_fmaf(s[r], c2, slope2 * (float)(n - m)) : s[r] * c2;
      bool ok = n < S;
      if constexpr (MASK != MASK_NONE) ok = ok && (n <= m);
      if constexpr (MASK == MASK_SLIDING_WINDOW) ok = ok && (n > m - W);
      x[r] = ok ? x[r] : -INFINITY;
      mx = fmaxf(mx, x[r]);
    }
    const float m_new = fmaxf(m_run, groups_max(mx));
    const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
    const float alpha = exp2f(m_run - m_use);
    l_run *= alpha;
#pragma unroll
    for (int i = 0; i < MT; ++i) acc[i] *= alpha;
    float pr[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      pr[r] = exp2f(x[r] - m_use);
      l_run += pr[r];
    }
    f32_accumulate<D>(acc, v, pr);
    m_run = m_new;
  }

  f32_put<D>(xch, acc, wave, lane);
  l_run = groups_sum(l_run);
  if (g == 0) {
    stat[0][wave][lq] = m_run;
    stat[1][wave][lq] = l_run;
  }
  __syncthreads();
  if (wave < D / 32) {
    float w[F32_NW], mt = -INFINITY, l = 0.f;
#pragma unroll
    for (int j = 0; j < F32_NW; ++j) mt = fmaxf(mt, stat[0][j][lq]);
    const float m_use = (mt == -INFINITY) ? 0.f : mt;
#pragma unroll
    for (int j = 0; j < F32_NW; ++j) {
      w[j] = exp2f(stat[0][j][lq] - m_use);
      l = __builtin_fmaf(stat[1][j][lq], w[j], l);
    }
    const float inv = (l > 0.f) ? 1.f / l : 0.f;
    f32x4 o[2];
    f32_get<D>(o, xch, w, wave, lane);
    if (m < S) {
      o[0] *= inv;
      o[1] *= inv;
      f32_store<D>(static_cast<float*>(p.o) + ((size_t)bh * S + m) * D, o, wave, g);
      if (wave == 0 && g == 0) p.lse[(size_t)bh * S + m] = (l > 0.f) ? (mt + log2f(l)) * kLn2 : -INFINITY;
    }
  }
}

template <int D, int ROPE, int MASK, bool ALIBI>
static int launch_one(const FwdParams& p, hipStream_t st) {
  const int nqb = (p.S + F32_T - 1) / F32_T;
  hipLaunchKernelGGL((fwd_fp32_kernel<D, ROPE, MASK, ALIBI>), dim3((unsigned)(nqb * p.B * p.H)), dim3(64 * F32_NW),
                     0, st, p);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

template <int D, int ROPE>
static int dispatch_mask(int mask, bool alibi, const FwdParams& p, hipStream_t st) {
  switch (mask) {
    case MASK_NONE: return alibi ? launch_one<D, ROPE, MASK_NONE, true>(p, st) : launch_one<D, ROPE, MASK_NONE, false>(p, st);
    case MASK_CAUSAL: return alibi ? launch_one<D, ROPE, MASK_CAUSAL, true>(p, st) : launch_one<D, ROPE, MASK_CAUSAL, false>(p, st);
    case MASK_SLIDING_WINDOW: return alibi ? launch_one<D, ROPE, MASK_SLIDING_WINDOW, true>(p, st) : launch_one<D, ROPE, MASK_SLIDING_WINDOW, false>(p, st);
  }
  return -2;
}

template <int D>
static int dispatch_rope(int rope, int mask, bool alibi, const FwdParams& p, hipStream_t st) {
  switch (rope) {
    case ROPE_NONE: return dispatch_mask<D, ROPE_NONE>(mask, alibi, p, st);
    case ROPE_NEOX: return dispatch_mask<D, ROPE_NEOX>(mask, alibi, p, st);
    case ROPE_INTERLEAVED: return dispatch_mask<D, ROPE_INTERLEAVED>(mask, alibi, p, st);
  }
  return -2;
}

int launch_fwd_fp32(int D, int rope, int mask, bool alibi, const FwdParams& p, hipStream_t st) {
  if (D == 64) return dispatch_rope<64>(rope, mask, alibi, p, st);
  if (D == 128) return dispatch_rope<128>(rope, mask, alibi, p, st);
  return -2;
}

}  // namespace af
