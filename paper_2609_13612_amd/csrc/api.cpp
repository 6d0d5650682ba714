// C-ABI entry points (declared in include/attnfuse.h): argument validation
// and dispatch to the kernel launchers.  Every argument is checked before the
// first HIP call; no exception leaves this file.  Nothing here allocates,
// synchronises or keeps state: the caller owns every buffer, the RoPE table
// included.
#include "attnfuse.h"

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstring>

#include "binding.h"
#include "launch.hpp"

namespace {

constexpr int kMaxS = 1 << 20;
static_assert(AF_DECODE_SCRATCH_BYTES == af::DECODE_SCRATCH_BYTES, "header and library agree on the static scratch");
constexpr int kAbiVersion = 3;

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
bool aligned4(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 3u) == 0; }

// Block-sparse masks: 64-position blocks, at most 2048 per side (the per-
// workgroup tile list lives in LDS).
constexpr int kMaxSparseS = 64 * 2048;


int map_launch(int rc) {
  if (rc == 0) return AF_OK;
  if (rc == -2) return AF_ERR_UNSUPPORTED;
  return AF_ERR_HIP;
}

// ---------------------------------------------------------------- caller-owned cos/sin table
// The table is [rows][D/2] (cos, sin) fp32 pairs; a RoPE call reads rows 0..S-1.
constexpr int kMaxTableRows = kMaxS;

size_t table_bytes(int rows, int D) { return (size_t)rows * (size_t)(D / 2) * 2 * sizeof(float); }

// Checks the table arguments of a call that rotates positions 0..S-1 (nothing
// without RoPE); a table given as an output would be a caller error too.
int check_table(int rope, const float* table, int rows, int S, const void* const* outs, int nouts) {
  if (rope == AF_ROPE_NONE) return AF_OK;
  if (!table || !aligned16(table) || rows < S || rows > kMaxTableRows) return AF_ERR_INVALID_ARG;
  for (int i = 0; i < nouts; ++i)
    if (outs[i] == static_cast<const void*>(table)) return AF_ERR_INVALID_ARG;
  return AF_OK;
}

// ---------------------------------------------------------------- validation
int check_common(int B, int H, int H_kv, int S, int D, int dtype, int rope, float rope_theta) {
  if (B < 1 || H < 1 || H_kv < 1 || S < 1 || S > kMaxS || D < 2 || (D & 1)) return AF_ERR_INVALID_ARG;
  if (H % H_kv != 0) return AF_ERR_INVALID_ARG;
  if (dtype != AF_DTYPE_BF16 && dtype != AF_DTYPE_FP32) return AF_ERR_INVALID_ARG;
  if (rope != AF_ROPE_NONE && rope != AF_ROPE_NEOX && rope != AF_ROPE_INTERLEAVED) return AF_ERR_INVALID_ARG;
  if (rope != AF_ROPE_NONE && !(std::isfinite(rope_theta) && rope_theta > 0.f)) return AF_ERR_INVALID_ARG;
  // grid sizes and element offsets must stay inside their integer types
  if ((long long)B * H * ((S + 63) / 64) >= (1LL << 31)) return AF_ERR_INVALID_ARG;
  return AF_OK;
}

int check_attn(int mask, int window, float scale) {
  if (mask != AF_MASK_NONE && mask != AF_MASK_CAUSAL && mask != AF_MASK_SLIDING_WINDOW) return AF_ERR_INVALID_ARG;
  if (mask == AF_MASK_SLIDING_WINDOW && window < 1) return AF_ERR_INVALID_ARG;
  if (!(std::isfinite(scale) && scale > 0.f)) return AF_ERR_INVALID_ARG;
  return AF_OK;
}

bool supported_d(int D) { return D == 64 || D == 128; }

// Workgroups that share one key block's (query head, query tile) steps in the
// dK/dV pass.  Few K/V heads or a short sequence leave CUs without one of its
// 128-key workgroups while each walks every query head of its group; splitting
// costs fp32 partials, written and read once at 4.5 TB/s, and a launch.  A step
// takes 2.2 us (64 queries, D = 128) or 3.0 (128 queries, D = 64).  Causal key
// blocks start longest first, so the pass ends with the longest or with the
// chip's share of the whole; equal ones run in rounds of 256.  Whole backward
// without / with, us: H32/8 D128 causal B1 S 256 / 512 / 1024 / 2048 / 4096 58 /
// 95 / 167 / 340 / 782 and 44 / 56 / 91 / 202 / 582; B3 H16/4 S1777 no mask 404 and
// 366; B2 H8/2 S4000 D64 causal 364 and 195.
double split_us(double units, int S, int D) { return units * S * D * 4.0 * 2 * 2 / 4.5e6; }   // a split's dK' and dV, out and in

int bwd_splits(int B, int H, int H_kv, int S, int D, int mask, int window) {
  const int G = H / H_kv, BQ = D == 64 ? 128 : 64;
  const double nkb = (S + 127) / 128, nt = (S + BQ - 1) / BQ, units = (double)B * H_kv;
  double longest = nt, sum = nkb * nt;   // query tiles of the longest key block, and of all
  if (mask == AF_MASK_CAUSAL) sum = nkb * (nt + 128.0 / BQ) / 2.0;
  if (mask == AF_MASK_SLIDING_WINDOW) {
    longest = std::fmin(nt, (128.0 + window) / BQ + 1.0);
    sum = nkb * longest;
  }
  longest *= G;
  const double share = sum * G * units / 256.0, step = D == 64 ? 3.0 : 2.2;
  double best = 0.0, first = 0.0;
  int n = 1;
  for (int k : {1, 2, 3, 4, 6, 8}) {
    if (k > longest) break;
    const double each = std::ceil(longest / k);
    double us = step * (mask == AF_MASK_CAUSAL ? std::fmax(each, share) : std::ceil(nkb * units * k / 256.0) * each);
    if (k == 1) best = first = us;
    else if ((us += 4.0 + k * split_us(units, S, D)) < best && us < 0.9 * first) best = us, n = k;
  }
  return n;
}

// The same under a block mask, from its lists: the 64-row query tiles that the
// longest 128-key block visits, and all of them, as af_bwd_blocksparse is told
// (0: not known).  Every workgroup spends 8 us on its list and resident rows, so
// the pass ends with the longest or with the chip's share of the steps and
// set-ups; at most `most`, what the dense call of the sizes takes.  All active:
// as the dense call, whose sums it then equals.  Whole backward unsplit / as the
// dense call / by the lists, us, causal: B1 H8 S2000 D128, diagonal blocks 55 / 81 /
// 55, 10 % random 87 / 96 / 87; B1 H32/8 S2048 D128 diagonal 73 / 90 / 73, BigBird
// (global block) 325 / 143 / 143; B1 H4/1 S8000 D128 10 % random 332 / 152 / 152.
int bwd_splits_sparse(int B, int H, int H_kv, int S, int D, int mask, int window, int longest_list, long long tiles,
                      int most) {
  if (longest_list < 1 || tiles < 1) return 1;
  const int G = H / H_kv;
  const long long nkb = (S + 127) / 128, nt = (S + 63) / 64;
  if (tiles == (mask == AF_MASK_NONE ? nkb * nt : nkb * nt - nkb * (nkb - 1))) return most;
  const double units = (double)B * H_kv, step = D == 64 ? 1.5 : 2.2, setup = 8.0;
  double longest = longest_list, sum = (double)tiles;
  if (mask == AF_MASK_SLIDING_WINDOW) {
    longest = std::fmin(longest, (128.0 + window) / 64.0 + 1.0);
    sum = std::fmin(sum, (double)nkb * longest);
  }
  double best = 0.0, first = 0.0;
  int n = 1;
  for (int k : {1, 2, 3, 4, 6, 8}) {
    if (k > longest * G || k > most) break;
    double us = std::fmax(setup + step * std::ceil(longest * G / k),
                          units * (nkb * k * setup + G * sum * step) / 256.0);
    if (k == 1) best = first = us;
    else if ((us += 4.0 + k * split_us(units, S, D)) < best && us < 0.9 * first) best = us, n = k;
  }
  return n;
}

// Backward workspace: [delta f32 | lse2 f32 | dO fp16 | dO scale f32 | partial
// max |dO| u32 | Q' fp16 | K' fp16 | partial dK' and dV f32], each section
// starting on a 256-byte boundary; Q' and K' only with RoPE, the partials only
// where some mask's dK/dV pass is split.  The partial maxima cover chunks of
// at least kDmaxChunk elements of each (batch, K/V head)'s dO.
constexpr long long kDmaxChunk = 16384;

struct BwdWorkspace {
  size_t delta, lse2, do16, dscale, dmax, qr16, kr16, part, total;
  int dmax_chunks;
  int splits;   // the partials there is room for
};

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

BwdWorkspace bwd_workspace(int B, int H, int H_kv, int S, int D, int rope) {
  const size_t rows = (size_t)B * H * S, krows = (size_t)B * H_kv * S;
  BwdWorkspace w{};
  size_t off = 0;
  w.delta = off; off += align256(rows * sizeof(float));
  w.lse2 = off;  off += align256(rows * sizeof(float));
  w.do16 = off;  off += align256(rows * D * 2);
  const size_t groups = (size_t)B * H_kv;
  w.dmax_chunks = (int)(((long long)(H / H_kv) * S * D + kDmaxChunk - 1) / kDmaxChunk);
  w.dscale = off; off += align256(groups * sizeof(float));
  w.dmax = off;   off += align256(groups * w.dmax_chunks * sizeof(uint32_t));
  if (rope != AF_ROPE_NONE) {
    w.qr16 = off; off += align256(rows * D * 2);
    w.kr16 = off; off += align256(krows * D * 2);
  }
  // the reported size does not know the mask or the type: room for the larger of
  // the two that fix the split by the sizes alone (a window takes at most that)
  w.splits = 1;
  if (supported_d(D)) {
    const int none = bwd_splits(B, H, H_kv, S, D, AF_MASK_NONE, 0), causal = bwd_splits(B, H, H_kv, S, D, AF_MASK_CAUSAL, 0);
    w.splits = none > causal ? none : causal;
  }
  w.part = off;
  if (w.splits > 1) off += align256((size_t)w.splits * 2 * krows * D * sizeof(float));
  w.total = off;
  return w;
}

// The splits (at most n) whose partials a workspace of `bytes` holds.  Everything
// before the partials is required; they are not, since the pass also runs unsplit: a
// workspace sized for a longer sequence, which splits less, serves a shorter one.
int splits_that_fit(int n, const BwdWorkspace& w, size_t bytes, size_t kv_elems) {
  const size_t room = (bytes - w.part) / (kv_elems * 2 * sizeof(float));
  return room < 2 ? 1 : room < (size_t)n ? (int)room : n;
}

// Decode workspace: per-wave partial (max, sum) pairs, then accumulators
// (four phase-1 waves per chunk, each writing its own partial).
struct DecodeLayout {
  int chunk, nsplit;
  size_t ml, acc, total;
};

// Keys per phase-1 workgroup: a power of two in [128, 4096] giving about 512
// workgroups (one resident round at two per CU, so each wave streams several
// tiles); the wave partials' (max, sum) pairs then accumulators, each
// 256-byte aligned.
DecodeLayout decode_layout(int B, int H, int H_kv, int S, int D) {
  const long long work = (long long)B * H_kv * S;
  DecodeLayout L{};
  L.chunk = 128;
  while (L.chunk < 4096 && (long long)L.chunk * 512 < work) L.chunk *= 2;
  L.nsplit = (S + L.chunk - 1) / L.chunk;
  const size_t parts = (size_t)B * H * L.nsplit * 4;
  L.ml = 0;
  L.acc = align256(parts * 2 * sizeof(float));
  L.total = L.acc + align256(parts * D * sizeof(float));
  return L;
}

// ---------------------------------------------------------------- shared bodies
// Dense bias tensor and normalisation of the extended entry points (EXT_NONE
// for the plain ones).
struct Ext {
  const float* bias = nullptr;
  long long sb = 0, sh = 0, sq = 0;
  int norm = AF_NORM_SOFTMAX;
  int kind() const {
    if (norm == AF_NORM_RELU) return bias ? af::EXT_RELU_BIAS : af::EXT_RELU;
    return bias ? af::EXT_BIAS : af::EXT_NONE;
  }
};

int check_ext(const Ext& e, const void* const* outs, int nouts) {
  if (e.norm != AF_NORM_SOFTMAX && e.norm != AF_NORM_RELU) return AF_ERR_INVALID_ARG;
  if (e.bias) {
    if ((reinterpret_cast<uintptr_t>(e.bias) & 3u) != 0) return AF_ERR_INVALID_ARG;
    if (e.sb < 0 || e.sh < 0 || e.sq < 0) return AF_ERR_INVALID_ARG;
    for (int i = 0; i < nouts; ++i) if (outs[i] == (const void*)e.bias) return AF_ERR_INVALID_ARG;
  }
  return AF_OK;
}

int fwd_impl(const void* Q, const void* K, const void* V, void* O, float* LSE, const int* q_block_ptr,
             const int* k_block_idx, const Ext& ext, int B, int H, int H_kv, int S, int D, int dtype, int rope,
             float rope_theta, const float* rope_table, int rope_table_rows, int mask, int window,
             const float* alibi_slopes, float softmax_scale, void* stream, void* k16 = nullptr, size_t k16_bytes = 0) {
  const bool relu = ext.norm == AF_NORM_RELU;   // no row statistic: LSE may be NULL
  if (!Q || !K || !V || !O || (!LSE && !relu)) return AF_ERR_INVALID_ARG;
  if (!aligned16(Q) || !aligned16(K) || !aligned16(V) || !aligned16(O) || !aligned16(LSE)) return AF_ERR_INVALID_ARG;
  if (O == Q || O == K || O == V || (const void*)LSE == Q || (const void*)LSE == K || (const void*)LSE == V)
    return AF_ERR_INVALID_ARG;
  const void* outs[] = {O, LSE};
  int rc0 = check_ext(ext, outs, 2);
  if (rc0 != AF_OK) return rc0;
  int rc = check_common(B, H, H_kv, S, D, dtype, rope, rope_theta);
  if (rc != AF_OK) return rc;
  if ((rc = check_attn(mask, window, softmax_scale)) != AF_OK) return rc;
  if ((rc = check_table(rope, rope_table, rope_table_rows, S, outs, 2)) != AF_OK) return rc;
  if (!supported_d(D)) return AF_ERR_UNSUPPORTED;
  if (q_block_ptr && dtype == AF_DTYPE_FP32) return AF_ERR_UNSUPPORTED;   // block-sparse: bf16 kernels only
  // the bias tensor and relu attention: bf16, without ALiBi or a block mask
  if (ext.kind() != af::EXT_NONE && (dtype == AF_DTYPE_FP32 || alibi_slopes || q_block_ptr))
    return AF_ERR_UNSUPPORTED;

  hipStream_t st = static_cast<hipStream_t>(stream);
  af::FwdParams p{};
  p.q = Q; p.k = K; p.v = V; p.o = O; p.lse = LSE;
  p.B = B; p.H = H; p.Hkv = H_kv; p.S = S;
  // a window of S or more keys is the causal mask; clamping keeps n + window in int range
  p.window = (mask == AF_MASK_SLIDING_WINDOW) ? (window < S ? window : S) : 0;
  p.slopes = alibi_slopes;
  p.scale = softmax_scale;
  p.table = (rope != AF_ROPE_NONE) ? reinterpret_cast<const float2*>(rope_table) : nullptr;
  p.bq_ptr = q_block_ptr;
  p.bk_idx = k_block_idx;
  p.bias = ext.bias;
  p.bias_sb = ext.sb; p.bias_sh = ext.sh; p.bias_sq = ext.sq;
  const bool alibi = alibi_slopes != nullptr;
  if (k16) {   // keys rotated once into the workspace
    const void* kin[] = {Q, K, V, O, LSE, ext.bias, q_block_ptr, k_block_idx, rope_table};
    for (const void* x : kin) if (x == k16) return AF_ERR_INVALID_ARG;
    if (!aligned16(k16) || dtype != AF_DTYPE_BF16 || rope == AF_ROPE_NONE) return AF_ERR_INVALID_ARG;
    if (k16_bytes < (size_t)B * H_kv * S * D * 2) return AF_ERR_INVALID_ARG;
    p.k16 = k16;
    return map_launch(af::launch_fwd_prerot(D, rope, mask, alibi, ext.kind(), p, st));
  }
  if (dtype == AF_DTYPE_BF16) return map_launch(af::launch_fwd_bf16(D, rope, mask, alibi, ext.kind(), p, st));
  return map_launch(af::launch_fwd_fp32(D, rope, mask, alibi, p, st));
}

// A block mask's four lists (none of a dense call) and the lengths of its column lists (0: not known).
struct Sparse {
  const int *q_block_ptr, *k_block_idx, *k_block_ptr, *q_block_idx;
  int longest = 0;
  long long tiles = 0;
};

int bwd_impl(const void* Q, const void* K, const void* V, const void* O, const void* dO, const float* LSE, void* dQ,
             void* dK, void* dV, const Sparse* sparse, const Ext& ext, void* workspace, size_t workspace_bytes,
             int B, int H, int H_kv, int S, int D, int dtype, int rope, float rope_theta, const float* rope_table,
             int rope_table_rows, int mask, int window, const float* alibi_slopes, float softmax_scale,
             void* stream) {
  const bool relu = ext.norm == AF_NORM_RELU;   // the LSE is not used: it may be NULL
  if (relu) LSE = nullptr;
  const void* ins[] = {Q, K, V, O, dO, LSE};
  void* outs[] = {dQ, dK, dV, workspace};
  for (const void* x : ins) if (!aligned16(x)) return AF_ERR_INVALID_ARG;
  if (!Q || !K || !V || !O || !dO || (!LSE && !relu)) return AF_ERR_INVALID_ARG;
  for (const void* x : outs) if (!x || !aligned16(x)) return AF_ERR_INVALID_ARG;
  for (const void* x : outs)
    for (const void* y : ins) if (y && x == y) return AF_ERR_INVALID_ARG;
  int rc0 = check_ext(ext, outs, 4);
  if (rc0 != AF_OK) return rc0;
  int rc = check_common(B, H, H_kv, S, D, dtype, rope, rope_theta);
  if (rc != AF_OK) return rc;
  if ((rc = check_attn(mask, window, softmax_scale)) != AF_OK) return rc;
  if ((rc = check_table(rope, rope_table, rope_table_rows, S, outs, 4)) != AF_OK) return rc;
  if (workspace_bytes < bwd_workspace(B, H, H_kv, S, D, rope).part) return AF_ERR_INVALID_ARG;
  if (!supported_d(D)) return AF_ERR_UNSUPPORTED;
  if (sparse && dtype == AF_DTYPE_FP32) return AF_ERR_UNSUPPORTED;        // block-sparse: bf16 kernels only
  if (ext.kind() != af::EXT_NONE && (dtype == AF_DTYPE_FP32 || alibi_slopes || sparse)) return AF_ERR_UNSUPPORTED;

  hipStream_t st = static_cast<hipStream_t>(stream);
  af::BwdParams p{};
  p.q = Q; p.k = K; p.v = V; p.o = O; p.dout = dO; p.lse = LSE;
  p.dq = dQ; p.dk = dK; p.dv = dV;
  const BwdWorkspace ws = bwd_workspace(B, H, H_kv, S, D, rope);
  char* wb = static_cast<char*>(workspace);
  p.delta = reinterpret_cast<float*>(wb + ws.delta);
  p.lse2 = reinterpret_cast<float*>(wb + ws.lse2);
  p.do16 = wb + ws.do16;
  p.dscale = reinterpret_cast<float*>(wb + ws.dscale);
  p.dmax = reinterpret_cast<uint32_t*>(wb + ws.dmax);
  p.splits = 1;
  if (dtype == AF_DTYPE_BF16) {
    const int w = window < S ? window : S, dense = bwd_splits(B, H, H_kv, S, D, mask, w);
    const int n = splits_that_fit(dense < ws.splits ? dense : ws.splits, ws, workspace_bytes, (size_t)B * H_kv * S * D);
    p.splits = sparse ? bwd_splits_sparse(B, H, H_kv, S, D, mask, w, sparse->longest, sparse->tiles, n) : n;
    p.part = reinterpret_cast<float*>(wb + ws.part);
  }
  p.dmax_chunks = ws.dmax_chunks < af::DMAX_PARTS ? ws.dmax_chunks : af::DMAX_PARTS;
  p.qr16 = (rope != AF_ROPE_NONE) ? wb + ws.qr16 : nullptr;
  p.kr16 = (rope != AF_ROPE_NONE) ? wb + ws.kr16 : nullptr;
  p.B = B; p.H = H; p.Hkv = H_kv; p.S = S;
  // a window of S or more keys is the causal mask; clamping keeps n + window in int range
  p.window = (mask == AF_MASK_SLIDING_WINDOW) ? (window < S ? window : S) : 0;
  p.slopes = alibi_slopes;
  p.scale = softmax_scale;
  p.table = (rope != AF_ROPE_NONE) ? reinterpret_cast<const float2*>(rope_table) : nullptr;
  if (sparse) {
    p.bq_ptr = sparse->q_block_ptr; p.bk_idx = sparse->k_block_idx;
    p.bk_ptr = sparse->k_block_ptr; p.bq_idx = sparse->q_block_idx;
  }
  p.bias = ext.bias;
  p.bias_sb = ext.sb; p.bias_sh = ext.sh; p.bias_sq = ext.sq;
  const bool alibi = alibi_slopes != nullptr;
  if (dtype == AF_DTYPE_FP32) return map_launch(af::launch_bwd_fp32(D, rope, mask, alibi, p, st));
  return map_launch(af::launch_bwd_bf16(D, rope, mask, alibi, ext.kind(), p, st));
}

// Query heads per workgroup, as the launchers pack them.
int heads_packed(int G, int max) {
  int hp = 1;
  while (hp < max && G % (2 * hp) == 0) hp *= 2;
  return hp;
}

}  // namespace

// Four waves (128 rows, two or three workgroups per CU that do not wait at each
// other's barriers) against eight (256 rows share each staged tile), us:
//   tiles copied to LDS, D = 128: B1 H32/8 causal S 500 / 2048 / 8192: 14.5 / 47.6 / 523 with four, 20.1 / 56.0 /
//   515 with eight; B4 H32/8 S8192 window 1024: 602 and 625; D = 64: B8 H16 S2048 causal 97 and 108, B4 H12 S2048
//   no mask 65 and 78.
// Past about 6000 keys per row at D = 128 the second copy of every tile costs
// more than the finer workgroups give.  So it does where the finer workgroups
// finish no sooner, all being equal without a mask: D = 64 B1 H12 S4096 76.1 with
// four, 73.3 with eight (staged through registers; 96.3 and 91.4 with a key bias),
// D = 128 with a key bias, whose loads wait for the copies, B1 H16/4 S3000 97.3 and 85.8,
// S2048 H32/8 77.0 and 71.9, causal S4096 159 and 145 (but with one head a workgroup four
// win: B3 H24/8 S4102 395 and 414).  (With a bias row per query
// four win: D = 64 B2 H16 S2048 72.5 and 93.)  Rotating in the loop doubles that work
// too.  There four waves win on short rows while their workgroups fit one round
// of the CUs (8 to 40 % at S 64 to 512 with D = 128, to 1024 with D = 64; from S
// 350 the interleaved form at D = 128 lost 1 to 9 %, its four-wave kernel spills).
// In more than a round they lose 10 to 28 % without a mask (B6 H16/2 S400 D128
// 29.9 and 38.0, B3 H12 S1000 D64 30.4 and 34.4), and win only
//   where all of them are resident, two to a CU, while eight waves need a second round (B6 H16 S616 D64 22.6 and 35.3);
//   with a causal mask at D = 64 (4 to 14 %) or, NeoX, over 128 to 256 rows (0 to 9 %);
//   under a window, whose edges the finer rows cut, by up to 60 % (B6 H16 S604 D64 window 66 15.2 and 24.6, B6 H24/8
//   S423 D128 window 23 26.5 and 40.0), but for packed heads of longer rows in one to two rounds (B3 H32/8 S512 D128
//   window 100 23.0 and 20.1).  There the keys that a workgroup visits stand in for the row's length.
int af::fwd_waves(int B, int H, int Hkv, int S, int D, int rope, int mask, int window, int bias) {
  const int G = H / Hkv, rows4 = 128 / heads_packed(G, 4), rows8 = 256 / heads_packed(G, 8);
  const bool cut = mask == AF_MASK_SLIDING_WINDOW;
  const long long n4 = (long long)((S + rows4 - 1) / rows4) * B * (H / heads_packed(G, 4));
  const long long n8 = (long long)((S + rows8 - 1) / rows8) * B * (H / heads_packed(G, 8));
  if (rope == AF_ROPE_NONE) {   // copied to LDS
    if (D == 64) return mask == AF_MASK_NONE && bias < 2 && n4 > 256 && n4 <= 512 && S >= (bias ? 1024 : 2048) ? 8 : 4;
    if (bias == 1 && mask == AF_MASK_NONE && (n4 + 255) / 256 >= 2 * ((n8 + 255) / 256)) return 8;
    if (bias == 1 && mask == AF_MASK_CAUSAL && n8 >= 512 && S >= 2048 && rows8 < 256) return 8;
    return S < 6144 ? 4 : 8;
  }
  const int keys = cut && window < S - rows8 ? rows8 + window : S;   // that a workgroup visits
  if (keys > (D == 64 ? 1024 : rope == AF_ROPE_INTERLEAVED && !cut ? 256 : 512)) return 8;
  if (n4 <= 256 || n4 == n8 || (n8 > 256 && n4 <= 512)) return 4;
  if (cut) return rows4 == 128 || n8 > 256 || S <= 256 || n4 <= 288 ? 4 : 8;
  if (n8 >= 256 || mask == AF_MASK_NONE) return 8;
  return D == 64 || (rope == AF_ROPE_NEOX && S >= 128 && S <= 256 && rows4 < rows8) ? 4 : 8;
}

extern "C" {

int attnfuse_version(void) { return kAbiVersion; }

size_t attnfuse_rope_table_bytes(int rows, int D) {
  if (rows < 1 || rows > kMaxTableRows || D < 2 || (D & 1)) return 0;
  return table_bytes(rows, D);
}

int attnfuse_rope_table_fill(float* table, int rows, int D, float rope_theta, void* stream) {
  if (!table || !aligned16(table) || rows < 1 || rows > kMaxTableRows || D < 2 || (D & 1)) return AF_ERR_INVALID_ARG;
  if (!(std::isfinite(rope_theta) && rope_theta > 0.f)) return AF_ERR_INVALID_ARG;
  if (!supported_d(D)) return AF_ERR_UNSUPPORTED;
  return map_launch(af::launch_rope_table(reinterpret_cast<float2*>(table), rows, D, (double)rope_theta,
                                          static_cast<hipStream_t>(stream)));
}

const char* attnfuse_strerror(int code) {
  switch (code) {
    case AF_OK: return "success";
    case AF_ERR_INVALID_ARG: return "invalid argument";
    case AF_ERR_UNSUPPORTED: return "unsupported variant (no compiled kernel)";
    case AF_ERR_HIP: return "HIP runtime error";
    case AF_ERR_TOO_LARGE: return "request needs more than the library's static scratch (use the workspace entry point)";
  }
  return "unknown error code";
}

int attnfuse_fwd(const void* Q, const void* K, const void* V, void* O, float* LSE,
                 int B, int H, int H_kv, int S, int D, int dtype,
                 int rope, float rope_theta, const float* rope_table, int rope_table_rows,
                 int mask, int window,
                 const float* alibi_slopes, float softmax_scale, void* stream) {
  return fwd_impl(Q, K, V, O, LSE, nullptr, nullptr, Ext{}, B, H, H_kv, S, D, dtype, rope, rope_theta, rope_table,
                  rope_table_rows, mask, window, alibi_slopes, softmax_scale, stream);
}

int attnfuse_fwd_blocksparse(const void* Q, const void* K, const void* V, void* O, float* LSE,
                             const int* q_block_ptr, const int* k_block_idx,
                             int B, int H, int H_kv, int S, int D, int dtype,
                             int rope, float rope_theta, const float* rope_table, int rope_table_rows,
                             int mask, int window,
                             const float* alibi_slopes, float softmax_scale, void* stream) {
  if (!q_block_ptr || !k_block_idx || !aligned4(q_block_ptr) || !aligned4(k_block_idx)) return AF_ERR_INVALID_ARG;
  const void* outs[] = {O, LSE};
  for (const void* x : outs)
    if (x == (const void*)q_block_ptr || x == (const void*)k_block_idx) return AF_ERR_INVALID_ARG;
  if (S < 1 || S > kMaxSparseS) return AF_ERR_INVALID_ARG;
  return fwd_impl(Q, K, V, O, LSE, q_block_ptr, k_block_idx, Ext{}, B, H, H_kv, S, D, dtype, rope, rope_theta,
                  rope_table, rope_table_rows, mask, window, alibi_slopes, softmax_scale, stream);
}

int attnfuse_fwd_bias_norm(const void* Q, const void* K, const void* V, void* O, float* LSE,
                           const float* bias, long long bias_stride_b, long long bias_stride_h,
                           long long bias_stride_q, int norm,
                           int B, int H, int H_kv, int S, int D, int dtype,
                           int rope, float rope_theta, const float* rope_table, int rope_table_rows,
                           int mask, int window,
                           const float* alibi_slopes, float softmax_scale, void* stream) {
  Ext e;
  e.bias = bias; e.sb = bias_stride_b; e.sh = bias_stride_h; e.sq = bias_stride_q; e.norm = norm;
  return fwd_impl(Q, K, V, O, LSE, nullptr, nullptr, e, B, H, H_kv, S, D, dtype, rope, rope_theta, rope_table,
                  rope_table_rows, mask, window, alibi_slopes, softmax_scale, stream);
}

// Rotating the keys once costs a launch and a pass over K (read bf16, write
// fp16: 2.6 us and 4.5 TB/s); rotating them in the loop costs every workgroup
// VALU work on every tile it visits, and keeps the tiles from being copied
// straight to LDS.  Measured on MI355X, in the loop / rotated once, us:
//   D = 128, H32/8 B1 causal, S 128 / 256 / 512 / 1024 / 2048 / 8192: 10.1 / 11.9, 14.6 / 13.9, 22.6 / 18.4,
//   38.5 / 26.8, 67 / 53, 605 / 528; B4 S8192 window 1024: 772 / 626; B16 H16 S512: 50.5 / 53.5;
//   D = 64, H12 B4 causal, S 512 / 1024 / 2048 / 4096: 13.4 / 15.7, 23.4 / 24.5, 48.5 / 49.5, 160 / 136; no mask 2048:
//   89.6 / 73.5; window 256 at 4096: 58.5 / 47.1; B32 H16 S512: 58.5 / 55.2;
//   block-sparse (9.2 % active) B4 H12 S4096 D64: 123 / 82; relu attention gains the rotation alone.
// Under a block mask the saving is the tiles' of an average workgroup while all
// run at once, then a part per workgroup that a CU takes in turn and per tile
// (fitted to 3000 drawn masks; a D = 64 mask of short lists without a causal range may
// hold a row far longer than the average, which hides that part in few turns).  With 0.6 us for
// every tile of all forms, as first, 30 of 222 calls that took it were slower by up to
// 25 % (B2 H32/8 S6316 D128 30 % random, window 25 72.5 / 86.8, B3 H8/2 S4910 D64 10 %
// random causal 27.9 / 31.3); now 5 of 157 by 3 to 9 %.
// An estimate in terms of 256-row workgroups, whichever form then runs: the
// saving follows the tiles of the longest workgroup while these leave CUs free,
// and otherwise the workgroups each CU takes in turn (5 us each) and the tiles of
// the busiest CU.  It is smaller where four waves rotate in the loop under a window (D = 64) and
// where the copied form's four-wave workgroups take more than a round, unless a
// causal mask or a window cuts their tiles: D = 64 B2 H16 S2048 no mask 49.4 / 52.8,
// B1 H12 S4096 83.0 / 85.6, B1 H8/2 S5066 window 827 26.2 / 27.7, but B2 H8/2 S4085 no
// mask 93.8 / 90.5; D = 128 B2 H16/4 S2048 window 300 26.2 / 28.1, but window 1024 45.1 / 44.1.
// With ALiBi or a bias the in-loop form has eight waves and fewer registers to
// spare, and more is saved: B1 H2 S1165 D64 window 538, bias row per query 37.8 / 26.2,
// B1 H8/1 S891 D64 ALiBi 26.1 / 19.0 (of 2500 drawn calls 3 are slower, by up to 16 %).
size_t af_fwd_workspace_bytes(int B, int H, int H_kv, int S, int D, int dtype, int rope, int mask, int window,
                              int norm, int extra, long long sparse_blocks) {
  if (B < 1 || H < 1 || H_kv < 1 || S < 1 || S > kMaxS || H % H_kv || !supported_d(D) || dtype != AF_DTYPE_BF16 ||
      rope == AF_ROPE_NONE)
    return 0;
  const size_t bytes = (size_t)B * H_kv * S * D * 2;
  const int G = H / H_kv;
  const int hp = heads_packed(G, sparse_blocks ? 4 : 8);
  const double units = (double)B * H_kv * (G / hp);
  const double nt = (S + 63) / 64;
  double saved;
  if (sparse_blocks) {
    // tiles visited, were the mask even: half of them under a causal mask, those of the band under a window
    double tiles = (double)sparse_blocks * (mask == AF_MASK_NONE ? 1.0 : 0.5);
    if (mask == AF_MASK_SLIDING_WINDOW) tiles = std::fmin(tiles, (double)sparse_blocks * std::fmin(1.0, (window / 64.0 + 1.5) / nt));
    const double turns = units * nt / 256.0, load = units * tiles / 256.0;
    if (turns <= 1.0) saved = 0.3 + (D == 128 ? 0.5 : 0.25) * tiles / nt;
    else if (D == 128) saved = 0.25 * (turns - 1.0) + 0.4 * load;
    else saved = (mask == AF_MASK_NONE && tiles < 8.0 * nt ? 2.0 * (turns - 3.0) : (hp == 1 ? 1.5 : 1.0) * turns - 0.7) + 0.22 * load;
  } else {
    const double rows = 256.0 / hp, wgs = std::ceil(S / rows);
    double longest = nt, tiles = wgs * nt;   // key tiles of the longest workgroup, and of all of a unit's
    if (mask == AF_MASK_CAUSAL) tiles = wgs * (nt + rows / 64.0) / 2.0;
    if (mask == AF_MASK_SLIDING_WINDOW) {
      longest = std::fmin(nt, (rows + window) / 64.0 + 1.0);
      tiles = std::fmin(wgs * (nt + rows / 64.0) / 2.0, wgs * longest);
    }
    const double turns = units * wgs / 256.0, load = std::fmax(longest, units * tiles / 256.0);
    if (norm == AF_NORM_RELU) {
      saved = (D == 128 ? 0.27 : 0.135) * load;
    } else if (turns <= 1.0) {
      const double rows4 = 128.0 / heads_packed(G, 4), n4 = std::ceil(S / rows4) * B * (H / heads_packed(G, 4));
      if (extra) saved = n4 > 256 ? (D == 128 ? 0.8 : 0.25) * longest : 1.2 + (D == 128 ? 0.75 : 0.4) * longest;
      else if (n4 > 256 && mask == AF_MASK_NONE) saved = D == 128 ? 2.0 + 0.22 * longest : 0.08 * longest;
      else if (n4 > 256 && mask == AF_MASK_SLIDING_WINDOW && hp > 1) saved = D == 128 ? 2.0 + 0.22 * longest : 0.2 * longest;
      else if (D == 128) saved = 0.8 * longest;
      else saved = (mask == AF_MASK_SLIDING_WINDOW && af::fwd_waves(B, H, H_kv, S, D, rope, mask, window, 0) == 4 ? 0.16 : 0.25) * longest;
    } else {
      saved = 5.0 * (turns - 1.0) + (D == 128 ? 0.3 : 0.2) * load;
    }
  }
  return saved > 2.6 + (double)bytes * 2.0 / 4.5e6 ? bytes : 0;
}

int af_fwd_waves(int B, int H, int H_kv, int S, int D, int rope, int mask, int window, int bias) {
  return af::fwd_waves(B, H, H_kv, S, D, rope, mask, window, bias);
}

int af_fwd_ws(const void* Q, const void* K, const void* V, void* O, float* LSE, const int* q_block_ptr,
              const int* k_block_idx, const float* bias, long long bias_stride_b, long long bias_stride_h,
              long long bias_stride_q, int norm, void* workspace, size_t workspace_bytes,
              int B, int H, int H_kv, int S, int D, int dtype,
              int rope, float rope_theta, const float* rope_table, int rope_table_rows, int mask, int window,
              const float* alibi_slopes, float softmax_scale, void* stream) {
  if (!workspace) return AF_ERR_INVALID_ARG;
  if ((q_block_ptr == nullptr) != (k_block_idx == nullptr) || !aligned4(q_block_ptr) || !aligned4(k_block_idx))
    return AF_ERR_INVALID_ARG;
  if (q_block_ptr) {
    const void* outs[] = {O, LSE};
    for (const void* x : outs)
      if (x == (const void*)q_block_ptr || x == (const void*)k_block_idx) return AF_ERR_INVALID_ARG;
    if (S < 1 || S > kMaxSparseS) return AF_ERR_INVALID_ARG;
  }
  Ext e;
  e.bias = bias; e.sb = bias_stride_b; e.sh = bias_stride_h; e.sq = bias_stride_q; e.norm = norm;
  return fwd_impl(Q, K, V, O, LSE, q_block_ptr, k_block_idx, e, B, H, H_kv, S, D, dtype, rope, rope_theta, rope_table,
                  rope_table_rows, mask, window, alibi_slopes, softmax_scale, stream, workspace, workspace_bytes);
}

size_t attnfuse_bwd_workspace_bytes(int B, int H, int H_kv, int S, int D, int rope) {
  if (B < 1 || H < 1 || H_kv < 1 || S < 1 || D < 2 || (D & 1) || H % H_kv) return 0;
  if (rope != AF_ROPE_NONE && rope != AF_ROPE_NEOX && rope != AF_ROPE_INTERLEAVED) return 0;
  return bwd_workspace(B, H, H_kv, S, D, rope).total;
}

int attnfuse_bwd(const void* Q, const void* K, const void* V, const void* O, const void* dO,
                 const float* LSE, void* dQ, void* dK, void* dV,
                 void* workspace, size_t workspace_bytes,
                 int B, int H, int H_kv, int S, int D, int dtype,
                 int rope, float rope_theta, const float* rope_table, int rope_table_rows,
                 int mask, int window,
                 const float* alibi_slopes, float softmax_scale, void* stream) {
  return bwd_impl(Q, K, V, O, dO, LSE, dQ, dK, dV, nullptr, Ext{}, workspace, workspace_bytes, B, H, H_kv, S, D,
                  dtype, rope, rope_theta, rope_table, rope_table_rows, mask, window, alibi_slopes, softmax_scale,
                  stream);
}

int af_bwd_blocksparse(const void* Q, const void* K, const void* V, const void* O, const void* dO,
                       const float* LSE, void* dQ, void* dK, void* dV,
                       const int* q_block_ptr, const int* k_block_idx,
                       const int* k_block_ptr, const int* q_block_idx, int longest_list, long long list_tiles,
                       void* workspace, size_t workspace_bytes,
                       int B, int H, int H_kv, int S, int D, int dtype,
                       int rope, float rope_theta, const float* rope_table, int rope_table_rows,
                       int mask, int window,
                       const float* alibi_slopes, float softmax_scale, void* stream) {
  const int* m[] = {q_block_ptr, k_block_idx, k_block_ptr, q_block_idx};
  for (const int* x : m) if (!x || !aligned4(x)) return AF_ERR_INVALID_ARG;
  const void* outs[] = {dQ, dK, dV, workspace};
  for (const void* x : outs)
    for (const int* y : m) if (x == (const void*)y) return AF_ERR_INVALID_ARG;
  if (S < 1 || S > kMaxSparseS) return AF_ERR_INVALID_ARG;
  const Sparse sp{q_block_ptr, k_block_idx, k_block_ptr, q_block_idx, longest_list, list_tiles};
  return bwd_impl(Q, K, V, O, dO, LSE, dQ, dK, dV, &sp, Ext{}, workspace, workspace_bytes, B, H, H_kv, S, D, dtype,
                  rope, rope_theta, rope_table, rope_table_rows, mask, window, alibi_slopes, softmax_scale, stream);
}

int attnfuse_bwd_blocksparse(const void* Q, const void* K, const void* V, const void* O, const void* dO,
                             const float* LSE, void* dQ, void* dK, void* dV,
                             const int* q_block_ptr, const int* k_block_idx,
                             const int* k_block_ptr, const int* q_block_idx,
                             void* workspace, size_t workspace_bytes,
                             int B, int H, int H_kv, int S, int D, int dtype,
                             int rope, float rope_theta, const float* rope_table, int rope_table_rows,
                             int mask, int window,
                             const float* alibi_slopes, float softmax_scale, void* stream) {
  return af_bwd_blocksparse(Q, K, V, O, dO, LSE, dQ, dK, dV, q_block_ptr, k_block_idx, k_block_ptr, q_block_idx, 0, 0,
                            workspace, workspace_bytes, B, H, H_kv, S, D, dtype, rope, rope_theta, rope_table,
                            rope_table_rows, mask, window, alibi_slopes, softmax_scale, stream);
}

void af_col_tiles(const unsigned char* active, int nb, long long* lengths) {
  long long longest[2] = {0, 0}, all[2] = {0, 0};
  for (int j0 = 0; j0 < nb; j0 += 64) {   // 64 columns (32 pairs) of every row at a time
    const int j1 = j0 + 64 < nb ? j0 + 64 : nb;
    long long n[2][32] = {};
    for (int i = 0; i < nb; ++i) {
      const unsigned char* row = active + (size_t)i * nb;
      for (int j = j0; j < j1; j += 2) {
        const int a = row[j], b = j + 1 < nb ? row[j + 1] : 0, p = (j - j0) / 2;
        n[0][p] += a | b;
        n[1][p] += (j <= i ? a : 0) | (j + 1 <= i ? b : 0);
      }
    }
    for (int m = 0; m < 2; ++m)
      for (long long x : n[m]) {
        all[m] += x;
        if (x > longest[m]) longest[m] = x;
      }
  }
  for (int m = 0; m < 2; ++m) { lengths[2 * m] = longest[m]; lengths[2 * m + 1] = all[m]; }
}

int af_bwd_splits(int B, int H, int H_kv, int S, int D, int mask, int window, int longest_list, long long list_tiles,
                  size_t partial_bytes) {
  const int w = window < S ? window : S;
  BwdWorkspace ws{};
  const int n = splits_that_fit(bwd_splits(B, H, H_kv, S, D, mask, w), ws, partial_bytes, (size_t)B * H_kv * S * D);
  return list_tiles < 0 ? n : bwd_splits_sparse(B, H, H_kv, S, D, mask, w, longest_list, list_tiles, n);
}

int attnfuse_bwd_bias_norm(const void* Q, const void* K, const void* V, const void* O, const void* dO,
                           const float* LSE, void* dQ, void* dK, void* dV,
                           const float* bias, long long bias_stride_b, long long bias_stride_h,
                           long long bias_stride_q, int norm,
                           void* workspace, size_t workspace_bytes,
                           int B, int H, int H_kv, int S, int D, int dtype,
                           int rope, float rope_theta, const float* rope_table, int rope_table_rows,
                           int mask, int window,
                           const float* alibi_slopes, float softmax_scale, void* stream) {
  Ext e;
  e.bias = bias; e.sb = bias_stride_b; e.sh = bias_stride_h; e.sq = bias_stride_q; e.norm = norm;
  return bwd_impl(Q, K, V, O, dO, LSE, dQ, dK, dV, nullptr, e, workspace, workspace_bytes, B, H, H_kv, S, D, dtype,
                  rope, rope_theta, rope_table, rope_table_rows, mask, window, alibi_slopes, softmax_scale, stream);
}

// ---------------------------------------------------------------- decode
size_t attnfuse_decode_workspace_bytes(int B, int H, int H_kv, int S_kv, int D) {
  if (B < 1 || H < 1 || H_kv < 1 || S_kv < 1 || S_kv > kMaxS || D < 2 || (D & 1) || H % H_kv) return 0;
  return decode_layout(B, H, H_kv, S_kv, D).total;
}

// The decode entry points share everything but where the partials live: the
// caller's workspace, or (workspace == nullptr) the library's static scratch.
static int decode_impl(const void* Q, const void* K, const void* V, const int* cache_lens, void* O, float* LSE,
                       void* workspace, size_t workspace_bytes, int B, int H, int H_kv, int S_kv, int D, int dtype,
                       int rope, float rope_theta, const float* rope_table, int rope_table_rows, int mask, int window,
                       const float* alibi_slopes, float softmax_scale, void* stream, bool static_scratch) {
  const void* ins[] = {Q, K, V};
  const void* outs[] = {O, LSE, workspace};
  const int nouts = static_scratch ? 2 : 3;
  for (const void* x : ins) if (!x || !aligned16(x)) return AF_ERR_INVALID_ARG;
  for (int i = 0; i < nouts; ++i) if (!outs[i] || !aligned16(outs[i])) return AF_ERR_INVALID_ARG;
  if (cache_lens && (reinterpret_cast<uintptr_t>(cache_lens) & 3u)) return AF_ERR_INVALID_ARG;
  for (int i = 0; i < nouts; ++i) {
    for (const void* y : ins) if (outs[i] == y) return AF_ERR_INVALID_ARG;
    if (outs[i] == static_cast<const void*>(cache_lens)) return AF_ERR_INVALID_ARG;
  }
  int rc = check_common(B, H, H_kv, S_kv, D, dtype, rope, rope_theta);
  if (rc != AF_OK) return rc;
  if ((rc = check_attn(mask, window, softmax_scale)) != AF_OK) return rc;
  if ((rc = check_table(rope, rope_table, rope_table_rows, S_kv, outs, nouts)) != AF_OK) return rc;
  const size_t need = attnfuse_decode_workspace_bytes(B, H, H_kv, S_kv, D);
  if (!static_scratch && workspace_bytes < need) return AF_ERR_INVALID_ARG;
  if (!supported_d(D) || dtype != AF_DTYPE_BF16 || H / H_kv > 32) return AF_ERR_UNSUPPORTED;
  if (static_scratch) {
    if (need > af::DECODE_SCRATCH_BYTES) return AF_ERR_TOO_LARGE;
    if (!(workspace = af::decode_scratch_ptr())) return AF_ERR_HIP;
  }

  hipStream_t st = static_cast<hipStream_t>(stream);
  const DecodeLayout L = decode_layout(B, H, H_kv, S_kv, D);
  af::DecodeParams p{};
  p.q = Q; p.k = K; p.v = V; p.lens = cache_lens; p.o = O; p.lse = LSE;
  char* wb = static_cast<char*>(workspace);
  p.part_ml = reinterpret_cast<float*>(wb + L.ml);
  p.part_acc = reinterpret_cast<float*>(wb + L.acc);
  p.B = B; p.H = H; p.Hkv = H_kv; p.S = S_kv;
  p.window = (mask == AF_MASK_SLIDING_WINDOW) ? (window < S_kv ? window : S_kv) : 0;
  p.chunk = L.chunk; p.nsplit = L.nsplit;
  p.slopes = alibi_slopes;
  p.scale = softmax_scale;
  p.table = (rope != AF_ROPE_NONE) ? reinterpret_cast<const float2*>(rope_table) : nullptr;
  return map_launch(af::launch_decode(D, rope, alibi_slopes != nullptr, p, st));
}

int attnfuse_decode(const void* Q, const void* K, const void* V, const int* cache_lens,
                    void* O, float* LSE, void* workspace, size_t workspace_bytes,
                    int B, int H, int H_kv, int S_kv, int D, int dtype,
                    int rope, float rope_theta, const float* rope_table, int rope_table_rows,
                    int mask, int window,
                    const float* alibi_slopes, float softmax_scale, void* stream) {
  if (!workspace) return AF_ERR_INVALID_ARG;
  return decode_impl(Q, K, V, cache_lens, O, LSE, workspace, workspace_bytes, B, H, H_kv, S_kv, D, dtype, rope,
                     rope_theta, rope_table, rope_table_rows, mask, window, alibi_slopes, softmax_scale, stream, false);
}

int attnfuse_decode_noalloc(const void* Q, const void* K, const void* V, const int* cache_lens,
                            void* O, float* LSE,
                            int B, int H, int H_kv, int S_kv, int D, int dtype,
                            int rope, float rope_theta, const float* rope_table, int rope_table_rows,
                            int mask, int window,
                            const float* alibi_slopes, float softmax_scale, void* stream) {
  return decode_impl(Q, K, V, cache_lens, O, LSE, nullptr, 0, B, H, H_kv, S_kv, D, dtype, rope, rope_theta,
                     rope_table, rope_table_rows, mask, window, alibi_slopes, softmax_scale, stream, true);
}

static int rope_common(const void* X0, const void* X1, void* Y0, void* Y1, int B, int H, int H_kv, int S, int D,
                       int dtype, int rope, float rope_theta, const float* rope_table, int rope_table_rows,
                       void* stream, bool inverse) {
  if (!X0 || !Y0 || !aligned16(X0) || !aligned16(Y0)) return AF_ERR_INVALID_ARG;
  if ((X1 == nullptr) != (Y1 == nullptr)) return AF_ERR_INVALID_ARG;
  if (X1 && (!aligned16(X1) || !aligned16(Y1))) return AF_ERR_INVALID_ARG;
  if (!X1) H_kv = 1;
  int rc = check_common(B, H, H_kv, S, D, dtype, rope, rope_theta);
  if (rc != AF_OK) return rc;
  if (rope == AF_ROPE_NONE) return AF_ERR_INVALID_ARG;
  const void* outs[] = {Y0, Y1};
  if ((rc = check_table(rope, rope_table, rope_table_rows, S, outs, 2)) != AF_OK) return rc;
  if (!supported_d(D)) return AF_ERR_UNSUPPORTED;
  hipStream_t st = static_cast<hipStream_t>(stream);
  af::RopeParams p{};
  p.x0 = X0; p.y0 = Y0; p.heads0 = H;
  p.x1 = X1; p.y1 = Y1; p.heads1 = X1 ? H_kv : 0;
  p.B = B; p.S = S;
  p.table = reinterpret_cast<const float2*>(rope_table);
  return map_launch(af::launch_rope(dtype == AF_DTYPE_FP32, D, rope, inverse, p, st));
}

int attnfuse_rope(const void* Q, const void* K, void* Qr, void* Kr, int B, int H, int H_kv, int S, int D,
                  int dtype, int rope, float rope_theta, const float* rope_table, int rope_table_rows,
                  void* stream) {
  return rope_common(Q, K, Qr, Kr, B, H, H_kv, S, D, dtype, rope, rope_theta, rope_table, rope_table_rows, stream,
                     false);
}

int attnfuse_rope_bwd(const void* dQr, const void* dKr, void* dQ, void* dK, int B, int H, int H_kv, int S, int D,
                      int dtype, int rope, float rope_theta, const float* rope_table, int rope_table_rows,
                      void* stream) {
  return rope_common(dQr, dKr, dQ, dK, B, H, H_kv, S, D, dtype, rope, rope_theta, rope_table, rope_table_rows, stream,
                     true);
}

}  // extern "C"
