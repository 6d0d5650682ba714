// fp32 debug backward: the passes of the bf16 backward (Section 4.4: dQ over
// key tiles; dK/dV over query tiles with the GQA group's heads summed; no
// atomics) in fp32 arithmetic throughout, the rotation recomputed on every
// tile.  It exists to check the backward at fp32 precision.
//
// With s_ij = scale <R_i q_i, R_j k_j> + bias_ij and P the softmax rows:
//   dV_j  = sum_i P_ij dO_i
//   dP_ij = <dO_i, v_j>,  delta_i = sum_d dO_id O_id,  dS_ij = P_ij (dP_ij - delta_i)
//   dQ_i  = R_i^T (scale sum_j dS_ij R_j k_j),  dK_j = R_j^T (scale sum_i dS_ij R_i q_i)
// P_ij is re-derived from the forward's LSE: P_ij = exp(s_ij - LSE_i).
//
// One workgroup per 16 output rows, its waves on the other side's 16-row tiles
// in turn (fp32_tiles.hpp).  The dQ pass forms delta for its own rows from
// registers and leaves it in the workspace for the dK/dV pass, so there is no
// pass of its own for it.  Bound, as the forward, by the chain of tiles of the
// longest wave.  Against one row per thread of 64: B1 H2 S128 D64 (interleaved,
// causal) dQ 139 -> 9.5 us, dK/dV 245 -> 9.2 us, and the row statistics' own
// pass (17 us) is gone; B1 H32/8 S2048 D128 (NeoX, causal) 210 -> 2.2 ms.
#include "fp32_tiles.hpp"
#include "launch.hpp"

namespace af {

// LDS: each wave's transposition tile, then the merge of the waves' partials.
template <int D>
constexpr int B32_LDS = F32_XCH<D> > F32_NW * F32_T * (D + 4) ? F32_XCH<D> : F32_NW * F32_T * (D + 4);

template <int D, int ROPE, int MASK, bool ALIBI>
__global__ __launch_bounds__(64 * F32_NW) void bwd_fp32_dq_kernel(BwdParams p) {
  constexpr int DL = D / 4, MT = D / 16;
  __shared__ __attribute__((aligned(16))) float lds[B32_LDS<D>];
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
  const size_t row = ((size_t)bh * S + mc) * D;
  const float* __restrict__ K = static_cast<const float*>(p.k) + kv;
  const float* __restrict__ V = static_cast<const float*>(p.v) + kv;

  const float c2 = p.scale * kLog2e;
  const float slope2 = ALIBI ? p.slopes[h] * kLog2e : 0.f;
  const int W = p.window;
  int t = wave, t_end = nqb;
  if constexpr (MASK != MASK_NONE) t_end = qb + 1;
  if constexpr (MASK == MASK_SLIDING_WINDOW) t += max(0, m0 - W + 1) / F32_T;

  float k[DL], cs[DL], vv[DL];   // the tile in flight; rows past S: row S-1, masked
  auto load = [&](int tile) {
    const int n = min(tile * F32_T + lq, S - 1);
    f32_load_row<D>(k, K + (size_t)n * D, g);
    f32_load_cs<D, ROPE>(cs, p.table + (size_t)n * (D / 2), g);
    f32_load_row<D>(vv, V + (size_t)n * D, g);
  };
  if (t < t_end) load(t);
  float q[DL], dov[DL];
  f32_load_row<D>(q, static_cast<const float*>(p.q) + row, g);
  f32_load_row<D>(dov, static_cast<const float*>(p.dout) + row, g);
  float dl = 0.f;
  {
    float x[DL];
    f32_load_cs<D, ROPE>(x, p.table + (size_t)mc * (D / 2), g);
    f32_rotate<D, ROPE>(q, x);
    f32_load_row<D>(x, static_cast<const float*>(p.o) + row, g);
#pragma unroll
    for (int i = 0; i < DL; ++i) dl = __builtin_fmaf(dov[i], x[i], dl);
    dl = groups_sum(dl);
  }
  const float l = p.lse[(size_t)bh * S + mc];
  const float l2 = (l == -INFINITY) ? INFINITY : l * kLog2e;
  if (wave == 0 && g == 0 && m < S) p.delta[(size_t)bh * S + m] = dl;

  f32x4 dq[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) dq[i] = f32x4{};
  for (; t < t_end; t += F32_NW) {
    const int n0 = t * F32_T + 4 * g;     // key of element 0
    float kr[DL], v[DL], kt[DL];
#pragma unroll
    for (int i = 0; i < DL; ++i) {
      kr[i] = k[i];
      v[i] = vv[i];
    }
    f32_rotate<D, ROPE>(kr, cs);
    if (t + F32_NW < t_end) load(t + F32_NW);
    f32_transpose<D>(kt, kr, lds + wave * F32_T * (D + 4), lq, g);
    const f32x4 s = f32_dot<D>(kr, q), dp = f32_dot<D>(v, dov);
    float ds[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int n = n0 + r;
      bool ok = n < S;
      if constexpr (MASK != MASK_NONE) ok = ok && (n <= m);
      if constexpr (MASK == MASK_SLIDING_WINDOW) ok = ok && (n > m - W);
      const float x = ALIBI ? __builtin_fmaf(s[r], c2, slope2 * (float)(n - m)) : s[r] * c2;
      ds[r] = ok ? exp2f(x - l2) * (dp[r] - dl) : 0.f;
    }
    f32_accumulate<D>(dq, kt, ds);
  }

  __syncthreads();   // every wave is past its transposition tile
  f32_put<D>(lds, dq, wave, lane);
  __syncthreads();
  if (wave < D / 32 && m < S) {
    const float w[F32_NW] = {p.scale, p.scale, p.scale, p.scale};
    f32x4 out[2];
    f32_get<D>(out, lds, w, wave, lane);
    f32_rotate_back<D, ROPE>(out, p.table + (size_t)m * (D / 2), wave, g);
    f32_store<D>(static_cast<float*>(p.dq) + ((size_t)bh * S + m) * D, out, wave, g);
  }
}

// 16 keys of one (batch, K/V head); the waves take the (query head of the
// group, query tile) pairs in turn.
template <int D, int ROPE, int MASK, bool ALIBI>
__global__ __launch_bounds__(64 * F32_NW) void bwd_fp32_dkdv_kernel(BwdParams p) {
  constexpr int DL = D / 4, MT = D / 16;
  __shared__ __attribute__((aligned(16))) float lds[B32_LDS<D>];
  const int tid = threadIdx.x, lane = tid & 63, lq = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int S = p.S;
  const int BG = p.B * p.Hkv;
  const int bg = blockIdx.x % BG;
  const int kb = (int)(blockIdx.x / BG);   // ascending: under a causal mask the first keys see the most queries
  const int b = bg / p.Hkv;
  const int G = p.H / p.Hkv;
  const int h0 = (bg % p.Hkv) * G;
  const int n0 = kb * F32_T, n = n0 + lq, nc = min(n, S - 1);

  const float c2 = p.scale * kLog2e;
  const int W = p.window;
  int tq = 0, tq_end = (S + F32_T - 1) / F32_T;
  if constexpr (MASK != MASK_NONE) tq = kb;
  if constexpr (MASK == MASK_SLIDING_WINDOW) tq_end = min(tq_end, (min(n0 + F32_T, S) - 1 + W - 1) / F32_T + 1);
  const int nt = tq_end - tq, items = G * nt;

  float q[DL], cs[DL], dor[DL], dot[DL], l4[4], d4[4];   // the tile in flight
  auto load = [&](int it) {
    const size_t bh = (size_t)b * p.H + h0 + it / nt;
    const int m0 = (tq + it % nt) * F32_T, m = min(m0 + lq, S - 1);
    f32_load_row<D>(q, static_cast<const float*>(p.q) + (bh * S + m) * D, g);
    f32_load_cs<D, ROPE>(cs, p.table + (size_t)m * (D / 2), g);
    f32_load_row<D>(dor, static_cast<const float*>(p.dout) + (bh * S + m) * D, g);
    f32_load_t<D>(dot, static_cast<const float*>(p.dout) + bh * S * D, m0, S, lq, g);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const size_t i = bh * S + min(m0 + 4 * g + r, S - 1);
      l4[r] = p.lse[i];
      d4[r] = p.delta[i];
    }
  };
  int it = wave;
  if (it < items) load(it);
  float k[DL], v[DL];
  {
    float x[DL];
    f32_load_row<D>(k, static_cast<const float*>(p.k) + ((size_t)bg * S + nc) * D, g);
    f32_load_cs<D, ROPE>(x, p.table + (size_t)nc * (D / 2), g);
    f32_rotate<D, ROPE>(k, x);
    f32_load_row<D>(v, static_cast<const float*>(p.v) + ((size_t)bg * S + nc) * D, g);
  }

  f32x4 dk[MT], dv[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) dk[i] = dv[i] = f32x4{};
  for (; it < items; it += F32_NW) {
    const int m0 = (tq + it % nt) * F32_T + 4 * g;   // query of element 0
    const float slope2 = ALIBI ? p.slopes[h0 + it / nt] * kLog2e : 0.f;
    float qr[DL], od[DL], ot[DL], qt[DL], l2[4], dl[4];
#pragma unroll
    for (int i = 0; i < DL; ++i) {
      qr[i] = q[i];
      od[i] = dor[i];
      ot[i] = dot[i];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      l2[r] = (l4[r] == -INFINITY) ? INFINITY : l4[r] * kLog2e;
      dl[r] = d4[r];
    }
    f32_rotate<D, ROPE>(qr, cs);
    if (it + F32_NW < items) load(it + F32_NW);
    f32_transpose<D>(qt, qr, lds + wave * F32_T * (D + 4), lq, g);
    const f32x4 s = f32_dot<D>(qr, k), dp = f32_dot<D>(od, v);
    float pr[4], ds[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = m0 + r;
      bool ok = n < S && m < S;
      if constexpr (MASK != MASK_NONE) ok = ok && (n <= m);
      if constexpr (MASK == MASK_SLIDING_WINDOW) ok = ok && (n > m - W);
      const float x = ALIBI ? __builtin_fmaf(s[r], c2, slope2 * (float)(n - m)) : s[r] * c2;
      pr[r] = ok ? exp2f(x - l2[r]) : 0.f;
      ds[r] = ok ? pr[r] * (dp[r] - dl[r]) : 0.f;
    }
    f32_accumulate<D>(dv, ot, pr);
    f32_accumulate<D>(dk, qt, ds);
  }

  const float one[F32_NW] = {1.f, 1.f, 1.f, 1.f}, sc[F32_NW] = {p.scale, p.scale, p.scale, p.scale};
  const size_t out_row = ((size_t)bg * S + nc) * D;
  const bool store = wave < D / 32 && n < S;
  f32x4 out[2];
  __syncthreads();   // every wave is past its transposition tile
  f32_put<D>(lds, dk, wave, lane);
  __syncthreads();
  if (store) {
    f32_get<D>(out, lds, sc, wave, lane);
    f32_rotate_back<D, ROPE>(out, p.table + (size_t)n * (D / 2), wave, g);
    f32_store<D>(static_cast<float*>(p.dk) + out_row, out, wave, g);
  }
  __syncthreads();
  f32_put<D>(lds, dv, wave, lane);
  __syncthreads();
  if (store) {
    f32_get<D>(out, lds, one, wave, lane);
    f32_store<D>(static_cast<float*>(p.dv) + out_row, out, wave, g);
  }
}

template <int D, int ROPE, int MASK, bool ALIBI>
static int launch_one(const BwdParams& p, hipStream_t st) {
  const int nb = (p.S + F32_T - 1) / F32_T;
  hipLaunchKernelGGL((bwd_fp32_dq_kernel<D, ROPE, MASK, ALIBI>), dim3((unsigned)(nb * p.B * p.H)), dim3(64 * F32_NW),
                     0, st, p);
  // after the dQ pass, which wrote delta
  hipLaunchKernelGGL((bwd_fp32_dkdv_kernel<D, ROPE, MASK, ALIBI>), dim3((unsigned)(nb * p.B * p.Hkv)),
                     dim3(64 * F32_NW), 0, st, p);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

template <int D, int ROPE>
static int dispatch_mask(int mask, bool alibi, const BwdParams& p, hipStream_t st) {
  switch (mask) {
    case MASK_NONE: return alibi ? launch_one<D, ROPE, MASK_NONE, true>(p, st) : launch_one<D, ROPE, MASK_NONE, false>(p, st);
    case MASK_CAUSAL: return alibi ? launch_one<D, ROPE, MASK_CAUSAL, true>(p, st) : launch_one<D, ROPE, MASK_CAUSAL, false>(p, st);
    case MASK_SLIDING_WINDOW: return alibi ? launch_one<D, ROPE, MASK_SLIDING_WINDOW, true>(p, st) : launch_one<D, ROPE, MASK_SLIDING_WINDOW, false>(p, st);
  }
  return -2;
}

template <int D>
static int dispatch_rope(int rope, int mask, bool alibi, const BwdParams& p, hipStream_t st) {
  switch (rope) {
    case ROPE_NONE: return dispatch_mask<D, ROPE_NONE>(mask, alibi, p, st);
    case ROPE_NEOX: return dispatch_mask<D, ROPE_NEOX>(mask, alibi, p, st);
    case ROPE_INTERLEAVED: return dispatch_mask<D, ROPE_INTERLEAVED>(mask, alibi, p, st);
  }
  return -2;
}

int launch_bwd_fp32(int D, int rope, int mask, bool alibi, const BwdParams& p, hipStream_t st) {
  if (D == 64) return dispatch_rope<64>(rope, mask, alibi, p, st);
  if (D == 128) return dispatch_rope<128>(rope, mask, alibi, p, st);
  return -2;
}

}  // namespace af
