// Fused RoPE + masked attention backward, bf16 MFMA with fp32 accumulation,
// for gfx950.
//
// The passes of Section 4.4, no atomics: every output tile has exactly one
// writer.
//   1. bwd_pre:   partial maxima of |dO| per (batch, K/V head), and with RoPE
//                 K' = R K rotated once into the workspace (fp16): the later
//                 kernels read every K' tile many times.  Under a block mask
//                 Q' = R Q too.
//   2. bwd_dq:    one workgroup per 128 or 256 query rows (GQA heads packed, as
//                 in the forward); it loops over visible key tiles:
//                 dQ' += scale dS K',  dQ = R^T dQ'.  Before the loop it forms
//                 what else the passes need of its rows from the registers that
//                 hold them: sigma (the power of two that brings the group's
//                 largest |dO| into [1, 2)), delta_i = rowsum(dO_i * O_i), and
//                 for the dK/dV pass sigma dO and (without a block mask)
//                 Q' = R Q in fp16 in the workspace.  Since it forms P and dP for every visible key of
//                 its rows, it also sums the softmax backward's row term
//                 delta_i = sum_j P_ij dP_ij in fp32 (with P renormalised by
//                 its own row sum) and leaves it, and the renormalised LSE.
//   3. bwd_dkdv:  (bwd_dkdv.hip) one workgroup per 128 keys of one (batch,
//                 K/V head); it loops over the query heads of the GQA group
//                 and their visible query tiles, re-deriving P = exp(S - LSE)
//                 tile by tile:  dV += P^T dO,  dS = P o (dO V^T - delta),
//                 dK' += scale dS^T Q';  dK = R^T dK'.
// delta from rowsum(dO o O) equals sum_j P_ij dP_ij only for the exact O;
// the bf16 O a forward stores moves it by O's rounding, which reaches dK and
// dQ through P_ij (dP_ij - delta_i).  The dK/dV pass therefore runs last, on
// the dQ pass's sum; the dQ pass itself uses rowsum(dO o O).
//
// Scaling: the fp16 MFMA operands dO and dS carry the factor sigma, so their
// magnitudes sit near 1 whatever the gradient's scale (unscaled bf16
// gradients of 1e-6 would fall into fp16's subnormals, 6e-8 apart); the
// gradients leave multiplied by 1/sigma.  Multiplying by a power of two is
// exact, so results do not depend on the scale of dO.
// Register layouts follow the forward: the operand held in registers is the
// MFMA B operand (lane = its row), tiles staged in LDS are the A operand, and
// contractions over queries/keys read a transposed LDS copy stored with the
// perm16 row order that matches the score tile's register order.
//
// Precision: Q', K' and dS are fp16 MFMA operands.  With RoPE the rotated
// Q' and K' are the fp16 values the forward's scores came from, so P is
// re-derived from the same rounded operands that produced its LSE; without
// RoPE, Q and K are converted exactly from bf16 as they are staged.  dS in
// fp16 (2^-12 relative rounding instead of bf16's 2^-9) keeps the sums
// dK = dS^T Q and dQ = dS K accurate when attention concentrates on a few
// keys and their gradients grow.  dV = P^T dO sums P over many queries
// without normalisation, so it also runs on fp16 operands (P and sigma dO,
// the latter converted exactly from bf16).  Range: the rotated |Q'|, |K'|
// and |V| must stay below the fp16 maximum 65504, and |sigma dS| <= 4 D
// max|V| below it too, i.e. max|V| < 16376 / D (128 at D = 128).  In the dQ
// pass dP = dO V^T uses the bf16 inputs as they are.
#include <type_traits>

#include "bwd_common.hpp"

namespace af {

// ---------------------------------------------------------------- before the dQ pass
// Blocks [0, B H_kv dmax_chunks): partial maxima of |dO| over chunks of each
// (batch, K/V head)'s G query heads (contiguous in [B, H, S, D]), as bf16
// magnitude bits: the bit patterns of non-negative bf16 values order like the
// values, so the maximum is an integer maximum.  With RoPE the blocks after
// them rotate the key rows, and under a block mask the query rows, one thread per
// chunk pair c (dims 8c.. and D/2 + 8c.., NeoX partners; interleaved pairs stay
// in-chunk).  One pass over dO and K (and Q), bound by HBM.  The rest of a preprocessing pass (delta, sigma dO,
// Q', sigma itself) happens in the dQ pass, which holds those rows anyway: as
// passes of their own they moved 370 MB more at B1 H32/8 S8192 D128 and cost
// 64 us of 2.56 ms, at B8 H16 S2048 D64 43 of 515, at B4 H12 S4096 D64
// block-sparse 16 of 293.  Q' alone is the exception under a block mask: there
// few tiles follow a workgroup's rotation, 5 us of VALU work at D = 128 with
// two waves per SIMD, nothing is in flight meanwhile (the tile list comes after),
// and this pass has the CUs to spare.  Whole backward, rotated there / in the dQ pass,
// us: B1 H8 S381 D128 10 % random 38 / 44, B1 H12/4 S5873 D128 band of three 106 / 114;
// over 200 drawn masks 1.11 times faster at the median.
template <int D, int ROPE>
__global__ __launch_bounds__(256) void bwd_pre_kernel(BwdParams p, int dmax_blocks) {
  if ((int)blockIdx.x < dmax_blocks) {
    const int nch = p.dmax_chunks;
    const int bg = blockIdx.x / nch, c = blockIdx.x - bg * nch;
    const long long n = (long long)(p.H / p.Hkv) * p.S * D;
    const long long per = ((n + nch - 1) / nch + 7) & ~7ll;   // elements per chunk (n % 8 == 0)
    const uint16_t* src = static_cast<const uint16_t*>(p.dout) + (long long)bg * n;
    const long long e1 = min(n, (c + 1) * per);
    uint32_t mx = 0;
    constexpr int U = 8, STRIDE = 8 * 256;   // loads in flight per thread
    long long e = c * per + 8 * threadIdx.x;
    for (; e + (U - 1) * STRIDE < e1; e += U * STRIDE) {
      u32x4 x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) x[u] = ld16(src + e + u * STRIDE);
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int w = 0; w < 4; ++w) mx = max(mx, max(x[u][w] & 0x7fffu, (x[u][w] >> 16) & 0x7fffu));
    }
    for (; e < e1; e += STRIDE) {
      const u32x4 x = ld16(src + e);
#pragma unroll
      for (int w = 0; w < 4; ++w) mx = max(mx, max(x[w] & 0x7fffu, (x[w] >> 16) & 0x7fffu));
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mx = max(mx, (uint32_t)__shfl_xor((int)mx, off, 64));
    __shared__ uint32_t part[4];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0) p.dmax[blockIdx.x] = max(max(part[0], part[1]), max(part[2], part[3]));
  } else if constexpr (ROPE != ROPE_NONE) {
    constexpr int TPR = D / 16;            // threads per row
    constexpr int RPB = 256 / TPR;         // rows per block
    const int c = threadIdx.x % TPR;
    const int d0 = 8 * c, d1 = D / 2 + 8 * c;
    const long long krows = (long long)p.B * p.Hkv * p.S, rows = krows + (p.bq_ptr ? (long long)p.B * p.H * p.S : 0);
    const long long at = (long long)(blockIdx.x - dmax_blocks) * RPB + threadIdx.x / TPR;
    if (at < rows) {   // key rows, then query rows
      const bool key = at < krows;
      const long long row = key ? at : at - krows;
      const int pos = (int)(row % p.S);
      const uint16_t* Kr = static_cast<const uint16_t*>(key ? p.k : p.q) + row * D;
      u32x4 k0 = ld16(Kr + d0), k1 = ld16(Kr + d1);
      if constexpr (ROPE == ROPE_NEOX) {
        rotate_neox8<false, true>(k0, k1, p.table + (size_t)pos * (D / 2) + 8 * c);
      } else {
        rotate_interleaved8<false, true>(k0, p.table + (size_t)pos * (D / 2) + 4 * c);
        rotate_interleaved8<false, true>(k1, p.table + (size_t)pos * (D / 2) + D / 4 + 4 * c);
      }
      uint16_t* kd = static_cast<uint16_t*>(key ? p.kr16 : p.qr16) + row * D;
      st16(kd + d0, k0);
      st16(kd + d1, k1);
    }
  }
}

// sigma of a (batch, K/V head) from its partial maxima (one wave, every lane
// gets it): 2^(127 - E) for the largest |dO| with biased exponent E, so that
// max |dO| * sigma lies in [1, 2); clamped to [2^-126, 2^126].  1 when the
// group's dO is all zero or holds an inf / NaN.
__device__ __forceinline__ float group_scale(const BwdParams& p, int bg, int lane) {
  static_assert(DMAX_PARTS == 4 * 64, "four partial maxima per lane");
  uint32_t part[4], mx = 0;   // (clamped rather than guarded: a guarded load waits for the one before it)
#pragma unroll
  for (int j = 0; j < 4; ++j) part[j] = p.dmax[(long long)bg * p.dmax_chunks + min(lane + 64 * j, p.dmax_chunks - 1)];
#pragma unroll
  for (int j = 0; j < 4; ++j) mx = max(mx, part[j]);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mx = max(mx, (uint32_t)__shfl_xor((int)mx, off, 64));
  const int E = (int)(mx >> 7);   // bf16 biased exponent (the sign bit is clear)
  if (mx == 0u || E == 255) return 1.f;
  return __uint_as_float((uint32_t)min(max(254 - max(E, 1), 1), 253) << 23);
}

// Convert a staged K tile's registers from bf16 to fp16 (exact for |k| < 65504).
template <int D>
__device__ __forceinline__ void k_to_f16(TileRegs<D, ROPE_NONE, 8>& R) {
  using C = TileCfg<D, ROPE_NONE>;
#pragma unroll
  for (int i = 0; i < C::KPT; ++i)
#pragma unroll
    for (int w = 0; w < 4; ++w) R.ka[i][w] = pack_f16(bf_lo(R.ka[i][w]), bf_hi(R.ka[i][w]));
}

// ---------------------------------------------------------------- dQ
// LDS layout of the dQ pass's key tiles: K' is read by rows (S^T = K' Q'^T)
// and transposed (dQ'^T += K'^T dS^T), so it is stored swizzled (swz_at, no
// padding); V is read by rows only, at a pitch of D + 8 (16-byte reads of 16
// rows fall in distinct banks).
template <int D>
struct DqTileCfg {
  static constexpr int K_ELEMS = 64 * D;
  static constexpr int VP = D + 8;
  static constexpr int STAGE = K_ELEMS + 64 * VP;
};

// Commit a staged key tile (tile_load layout of TileCfg<D, ROPE_NONE>) into
// the dQ pass's layout.
template <int D>
__device__ __forceinline__ void dq_tile_commit(const TileRegs<D, ROPE_NONE>& R, uint16_t* __restrict__ Ks,
                                               uint16_t* __restrict__ Vs, int tid) {
  using C = TileCfg<D, ROPE_NONE>;
#pragma unroll
  for (int i = 0; i < C::KPT; ++i) {
    const int it = tid + C::THREADS * i;
    if (C::K_ITEMS % C::THREADS != 0 && it >= C::K_ITEMS) break;
    const int r = it / C::K_UNITS, c = it % C::K_UNITS;
    *reinterpret_cast<u32x4*>(Ks + swz_at<D>(r, 8 * c)) = R.ka[i];
  }
#pragma unroll
  for (int i = 0; i < C::VPT; ++i) {
    const int it = tid + C::THREADS * i;
    if (C::V_ITEMS % C::THREADS != 0 && it >= C::V_ITEMS) break;
    const int r = it / (D / 8), c = it % (D / 8);
    *reinterpret_cast<u32x4*>(Vs + r * DqTileCfg<D>::VP + 8 * c) = R.v[i];
  }
}

// Same decomposition as the forward: GQA heads packed, double-buffered K'/V
// tiles; dQ'^T += K'^T dS^T with K'^T from transpose reads.  With RoPE the
// tiles (K' rotated, fp16, from the workspace; V) are copied straight to LDS
// by four waves, so that two workgroups share a CU and do not wait at each
// other's barriers; without it K is converted to fp16 as it is staged, eight
// waves sharing that work (layout above).  What bounds the pass is the chain
// S, dP -> softmax -> dQ of each tile, which the other waves of the SIMD hide.
// Against eight waves staging through registers: B1 H32/8 S8192 D128 causal
// 820 -> 788 us, window 1024 at B4 954 -> 854, B8 H16 S2048 D64 151 -> 139,
// B3 H16/4 S1777 D128 no mask 170 -> 138.
constexpr int dq_waves(int rope, bool sparse) { return (rope != ROPE_NONE && !sparse) ? 4 : 8; }

template <int D, int ROPE, int MASK, bool ALIBI, bool SPARSE, int EXT = EXT_NONE>
__global__ __launch_bounds__(64 * dq_waves(ROPE, SPARSE)) __attribute__((amdgpu_waves_per_eu(2)))
void bwd_dq_kernel(BwdParams p) {
  constexpr bool ASYNC = ROPE != ROPE_NONE && !SPARSE;
  using C = TileCfg<D, ROPE_NONE, dq_waves(ROPE, SPARSE)>;   // K' arrives rotated, or K is converted to fp16 at staging
  using AT = AsyncTile<D, C::NW>;
  using L = DqTileCfg<D>;
  constexpr bool ROT = ROPE != ROPE_NONE;    // Q' and K' come rotated (fp16) from the workspace
  constexpr bool TBIAS = EXT == EXT_BIAS || EXT == EXT_RELU_BIAS;
  constexpr bool RELU = EXT == EXT_RELU || EXT == EXT_RELU_BIAS;
  static_assert(TILE_LIST_SCRATCH_BYTES <= 2 * L::STAGE * (int)sizeof(uint16_t), "the tile-list scratch fits the stages");
  // the two key-tile stages, and at the end each wave's dQ rows on their way out
  constexpr int STAGES = ASYNC ? 4 * AT::ELEMS : 2 * L::STAGE;
  constexpr int SMEM = (STAGES > C::NW * OUT_ROWS_ELEMS<D>) ? STAGES : C::NW * OUT_ROWS_ELEMS<D>;
  __shared__ __attribute__((aligned(16))) uint16_t smem[SMEM];

  const int tid = threadIdx.x, lane = tid & 63, lq = lane & 31, lg = lane >> 5;
  const int wave = ASYNC ? __builtin_amdgcn_readfirstlane(tid >> 6) : tid >> 6;
  const int S = p.S;
  const int HP = p.heads_per_wg;
  const int WPH = C::NW / HP;
  const int P = 32 * WPH;
  const int G = p.H / p.Hkv;
  const int groups = G / HP;
  const int units = p.B * p.Hkv * groups;
  const int npb = (S + P - 1) / P;
  const int unit = blockIdx.x % units;
  // position blocks run backwards (the longest causal rows first); under a
  // block mask without an elementwise mask they run forwards, as the forward's
  // do, which starts global rows (conventionally the first) early
  const int pb = (SPARSE && MASK == MASK_NONE) ? (int)(blockIdx.x / units) : npb - 1 - (int)(blockIdx.x / units);
  const int hg = unit % groups, bg = unit / groups;
  const int b = bg / p.Hkv, g = bg % p.Hkv;
  const int h = g * G + hg * HP + wave / WPH;
  const int p0 = pb * P;
  const int mw = p0 + 32 * (wave % WPH);
  const int m = mw + lq;
  const int p_end = min(p0 + P, S);
  const size_t bh = (size_t)b * p.H + h;

  constexpr bool QROT = ROT && !SPARSE;      // this pass rotates its query rows (under a block mask the first one did)
  const uint16_t* Qh = static_cast<const uint16_t*>(ROT && SPARSE ? p.qr16 : p.q) + bh * S * D;
  const uint16_t* dOh = static_cast<const uint16_t*>(p.dout) + bh * S * D;
  const uint16_t* Kg = static_cast<const uint16_t*>(ROT ? p.kr16 : p.k) + (size_t)bg * S * D;
  const uint16_t* Vg = static_cast<const uint16_t*>(p.v) + (size_t)bg * S * D;

  const int W = p.window;
  const int ntiles = (S + C::BN - 1) / C::BN;
  int t_begin = 0, t_end = ntiles;
  if constexpr (MASK != MASK_NONE) t_end = min(ntiles, (p_end - 1) / C::BN + 1);
  if constexpr (MASK == MASK_SLIDING_WINDOW) t_begin = max(0, p0 - W + 1) / C::BN;
  // the first tile copied to LDS is in flight while the rows are loaded
  AT at(lane, wave);
  auto stage = [&](int t) { return smem + (t & 1) * 2 * AT::ELEMS; };   // K', then V
  if constexpr (ASYNC) {
    at.load(Kg, t_begin * C::BN, S, stage(0));
    at.load(Vg, t_begin * C::BN, S, stage(0) + AT::ELEMS);
  }

  u32x4 qreg[C::KS], oreg[C::KS];
  const int mc = min(m, S - 1);   // rows past S compute on row S-1 and are never stored
  load_row_operand<D, ROPE_NONE>(oreg, dOh, nullptr, mc, S, lg);   // dO as it is
  // delta_i from rowsum(dO o O), and LSE_i in log2 units (+inf for an empty row,
  // so its P is 0); relu attention has neither.  O's chunks are all in flight at
  // once, and gone before the rotation needs registers
  float lse2 = INFINITY, del = 0.f;
  if constexpr (!RELU) {
    const uint16_t* Oh = static_cast<const uint16_t*>(p.o) + bh * S * D + (size_t)mc * D + 8 * lg;
    u32x4 o[C::KS];
#pragma unroll
    for (int s = 0; s < C::KS; ++s) o[s] = ld16(Oh + 16 * s);
    const float l = p.lse[bh * S + mc];
#pragma unroll
    for (int s = 0; s < C::KS; ++s)
#pragma unroll
      for (int w = 0; w < 4; ++w) del += bf_lo(oreg[s][w]) * bf_lo(o[s][w]) + bf_hi(oreg[s][w]) * bf_hi(o[s][w]);
    lse2 = (m < S && l != -INFINITY) ? l * kLog2e : INFINITY;
  }
  const float sig = group_scale(p, bg, lane);
  if (tid == 0 && hg == 0 && p0 == 0) p.dscale[bg] = sig;   // for the dK/dV pass
  if constexpr (!RELU) del = pair_sum(del) * sig;
  load_row_operand<D, QROT ? ROPE : ROPE_NONE, !ROT>(qreg, Qh, p.table, mc, S, lg);   // Q' (fp16)
  // the dK/dV pass's operands of these rows: sigma dO, and Q' under RoPE
  if (m < S) {
    const size_t row = (bh * S + m) * D + 8 * lg;
    uint16_t* od = static_cast<uint16_t*>(p.do16) + row;
#pragma unroll
    for (int s = 0; s < C::KS; ++s) {
      u32x4 x;
#pragma unroll
      for (int w = 0; w < 4; ++w) x[w] = pack_f16(bf_lo(oreg[s][w]) * sig, bf_hi(oreg[s][w]) * sig);
      st16(od + 16 * s, x);
    }
    if constexpr (QROT) {
      uint16_t* qd = static_cast<uint16_t*>(p.qr16) + row;
#pragma unroll
      for (int s = 0; s < C::KS; ++s) st16(qd + 16 * s, qreg[s]);
    }
  }
  const float* __restrict__ brow = nullptr;       // this lane's row of the bias tensor
  if constexpr (TBIAS) brow = p.bias + b * p.bias_sb + h * p.bias_sh + mc * p.bias_sq;
  float dsum = 0.f;   // this lane's part of sum_j P_ij dP_ij (unscaled)
  float lsum = 0.f;   // and of sum_j P_ij

  f32x16 dq[C::MT];
#pragma unroll
  for (int i = 0; i < C::MT; ++i) dq[i] = f32x16{};

  const float c2 = p.scale * kLog2e;
  const float slope2 = ALIBI ? p.slopes[h] * kLog2e : 0.f;
  // Key tiles by position i: t_begin + i, or under a block-sparse mask the
  // union of the workgroup's query blocks' active key blocks (as the forward).
  __shared__ std::conditional_t<SPARSE, TileList<true>, int> tl;
  int ntl = t_end - t_begin;
  int jw = 0;
  if constexpr (SPARSE) {             // the staging memory serves as scratch: nothing is staged yet
    const int r0 = p0 / C::BN, r1 = (p_end - 1) / C::BN;
    ntl = __builtin_amdgcn_readfirstlane(build_tile_list<C::THREADS>(tl, smem, p.bq_ptr, p.bk_idx, r0, r1 - r0 + 1,
                                                                     ntiles, t_begin, t_end, tid));
    jw = mw / C::BN - r0;
  }
  auto tile_at = [&](int i) -> int {
    if constexpr (SPARSE) return __builtin_amdgcn_readfirstlane((int)tl.tile[i]);
    else return t_begin + i;
  };

  const SwzLane<D> zl(lane);
  TileRegs<D, ROPE_NONE, C::NW> R;
  if constexpr (ASYNC) {
    async_wait();
  } else if (ntl > 0) {
    tile_load<D, ROPE_NONE>(R, Kg, Vg, nullptr, tile_at(0) * C::BN, S, tid);
    if constexpr (!ROT) k_to_f16(R);
    dq_tile_commit<D>(R, smem, smem + L::K_ELEMS, tid);
  }
  __syncthreads();

  for (int t = 0; t < ntl; ++t) {
    const int n0 = tile_at(t) * C::BN;
    const SwzLane<D> z = ASYNC ? zl : zl.opaque();   // (AsyncTile has its own offsets)
    // (the lane offsets of AsyncTile carry the stage)
    const uint16_t* Ks = ASYNC ? smem : smem + (t & 1) * L::STAGE;
    const uint16_t* Vs = ASYNC ? smem + AT::ELEMS : Ks + L::K_ELEMS;
    const bool more = t + 1 < ntl;
    if constexpr (ASYNC) {
      const int next = tile_at(min(t + 1, ntl - 1)) * C::BN;   // past the last tile: into a stage nobody reads any more
      at.load(Kg, next, S, stage(t + 1));
      at.load(Vg, next, S, stage(t + 1) + AT::ELEMS);
    } else if (more) {
      tile_load<D, ROPE_NONE>(R, Kg, Vg, nullptr, tile_at(t + 1) * C::BN, S, tid);
    }

    bool visible = mw < S;
    if constexpr (SPARSE) visible = visible && ((tl.rows[t] >> jw) & 1);
    if constexpr (MASK != MASK_NONE) visible = visible && (n0 <= mw + 31);
    if constexpr (MASK == MASK_SLIDING_WINDOW) visible = visible && (n0 + C::BN - 1 > mw - W);
    if (visible) {
      bool need_mask = n0 + C::BN > S;
      if constexpr (MASK != MASK_NONE) need_mask = need_mask || (n0 + C::BN - 1 > mw);
      if constexpr (MASK == MASK_SLIDING_WINDOW) need_mask = need_mask || (n0 <= mw + 31 - W);
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        f32x16 sc = f32x16{}, dp = f32x16{};
#pragma unroll
        for (int k = 0; k < C::KS; ++k) {
          u32x4 ak, av;
          if constexpr (ASYNC) {
            ak = at.row(Ks, 32 * kt, k);
            av = at.row(Vs, 32 * kt, k);
          } else {
            ak = row_operand_swz<D>(Ks, z, 32 * kt, k);
            av = *reinterpret_cast<const u32x4*>(Vs + (32 * kt + lq) * L::VP + 16 * k + 8 * lg);
          }
          sc = mfma32<true>(ak, qreg[k], sc);
          dp = mfma32(av, oreg[k], dp);
        }
        // element r: key nn = n0 + 32 kt + 8 (r/4) + 4 lg + r%4, query m
        float ds[16];
        bool pos[16];   // relu attention: s > 0
        float bias[16] = {};
        if constexpr (TBIAS) load_bias16(bias, brow, n0 + 32 * kt, lg, S);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int nn = n0 + 32 * kt + 8 * (r >> 2) + 4 * lg + (r & 3);
          if constexpr (TBIAS || RELU) {
            const float bv = bias[r];
            if constexpr (RELU) {
              pos[r] = __builtin_fmaf(sc[r], p.scale, bv) > 0.f;
              ds[r] = 1.f;
            } else {
              ds[r] = fast_exp2(__builtin_fmaf(sc[r], c2, bv * kLog2e) - lse2);
            }
          } else {
            const float x = ALIBI ? __builtin_fmaf(sc[r], c2, slope2 * (float)(nn - m)) : sc[r] * c2;
            ds[r] = fast_exp2(x - lse2);
          }
        }
        if (need_mask) {   // wave-uniform
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int nn = n0 + 32 * kt + 8 * (r >> 2) + 4 * lg + (r & 3);
            bool ok = nn < S;
            if constexpr (MASK != MASK_NONE) ok = ok && (nn <= m);
            if constexpr (MASK == MASK_SLIDING_WINDOW) ok = ok && (nn > m - W);
            ds[r] = ok ? ds[r] : 0.f;
          }
        }
        if constexpr (RELU) {   // dS = dP where s > 0
#pragma unroll
          for (int r = 0; r < 16; ++r) ds[r] = pos[r] ? ds[r] * dp[r] * sig : 0.f;
        } else {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            lsum += ds[r];
            dsum = __builtin_fmaf(ds[r], dp[r], dsum);
            ds[r] *= __builtin_fmaf(dp[r], sig, -del);
          }
        }
        u32x4 db[2];
#pragma unroll
        for (int hf = 0; hf < 2; ++hf)
#pragma unroll
          for (int w = 0; w < 4; ++w) db[hf][w] = pack_f16(ds[8 * hf + 2 * w], ds[8 * hf + 2 * w + 1]);
#pragma unroll
        for (int mt = 0; mt < C::MT; ++mt)
#pragma unroll
          for (int hf = 0; hf < 2; ++hf) {
            u32x4 a;
            if constexpr (ASYNC) a = at.tr(Ks, 32 * kt + 16 * hf, mt);
            else a = tr_operand_swz<D>(Ks, z, 32 * kt + 16 * hf, mt);
            dq[mt] = mfma32<true>(a, db[hf], dq[mt]);
          }
      }
    }
    if constexpr (ASYNC) {
      async_wait();
      at.flip((t & 1) ? -2 * AT::ELEMS : 2 * AT::ELEMS);
    } else if (more) {
      uint16_t* Kn = smem + ((t + 1) & 1) * L::STAGE;
      if constexpr (!ROT) k_to_f16(R);
      dq_tile_commit<D>(R, Kn, Kn + L::K_ELEMS, tid);
    }
    __syncthreads();
  }
  // For the dK/dV pass: the row's probabilities as this pass formed them sum
  // to l = sum_j P_ij, which differs from 1 by the rounding of the LSE it was
  // given (noticeable when scores are large); LSE + log2 l renormalises them,
  // and delta = sum_j P_ij dP_ij / l is the softmax backward's row term of
  // the renormalised P.  Rows with no visible key keep LSE = +inf.
  if constexpr (!RELU) {
    const float ltot = pair_sum(lsum), dtot = pair_sum(dsum);   // the lane pair (l, l ^ 32) holds row m's keys
    if (m < S && lg == 0) {
      const bool any = ltot > 0.f;
      p.delta[bh * S + m] = any ? dtot / ltot * sig : 0.f;
      p.lse2[bh * S + m] = any ? lse2 + __log2f(ltot) : INFINITY;
    }
  }
  // the key loop ended on a barrier after every wave's last LDS read
  store_grad_rows<D, ROPE>(dq, p.scale / sig, static_cast<uint16_t*>(p.dq) + bh * S * D, p.table, mw, S,
                           smem + wave * OUT_ROWS_ELEMS<D>, lane);
}

// ---------------------------------------------------------------- launch
namespace {
struct BwdPasses {
  template <int D, int ROPE, int MASK, bool ALIBI, int EXT>
  static int run(const BwdParams& p, hipStream_t st) {
    constexpr int RPB = 256 / (D / 16);
    const long long rows = (ROPE != ROPE_NONE) ? (long long)p.B * (p.Hkv + (p.bq_ptr ? p.H : 0)) * p.S : 0;
    const int k_blocks = (int)((rows + RPB - 1) / RPB);
    const int d_blocks = p.B * p.Hkv * p.dmax_chunks;
    hipLaunchKernelGGL((bwd_pre_kernel<D, ROPE>), dim3((unsigned)(d_blocks + k_blocks)), dim3(256), 0, st, p, d_blocks);
    const int nw = (EXT == EXT_NONE && p.bq_ptr) ? dq_waves(ROPE, true) : dq_waves(ROPE, false);
    BwdParams pq = p;
    pq.heads_per_wg = heads_per_wg(p.H / p.Hkv) < nw ? heads_per_wg(p.H / p.Hkv) : nw;
    const int P = 32 * nw / pq.heads_per_wg;
    const long long qblocks = (long long)((p.S + P - 1) / P) * p.B * p.Hkv * ((p.H / p.Hkv) / pq.heads_per_wg);
    if (EXT == EXT_NONE && p.bq_ptr)
      hipLaunchKernelGGL((bwd_dq_kernel<D, ROPE, MASK, ALIBI, true>), dim3((unsigned)qblocks), dim3(64 * nw), 0,
                         st, pq);
    else
      hipLaunchKernelGGL((bwd_dq_kernel<D, ROPE, MASK, ALIBI, false, EXT>), dim3((unsigned)qblocks),
                         dim3(64 * nw), 0, st, pq);
    if (hipGetLastError() != hipSuccess) return -3;
    // after the dQ pass, which replaced delta by sum_j P_ij dP_ij
    return launch_bwd_dkdv_bf16(D, ROPE, MASK, ALIBI, EXT, p, st);
  }
};
}  // namespace

int launch_bwd_bf16(int D, int rope, int mask, bool alibi, int ext, const BwdParams& p, hipStream_t st) {
  return bwd_dispatch<BwdPasses>(D, rope, mask, alibi, ext, p, st);
}

}  // namespace af
