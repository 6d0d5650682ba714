// Decode attention over a key/value cache, bf16 inputs, MFMA with fp32
// accumulation, for gfx950 (Section 4.2 "Flash Decoding"; Table tab:decode).
//
// One query per sequence makes the work a stream over the cache: each K/V
// element is used once per query head of its group, so the kernel is bound by
// HBM and is built to read the cache exactly once at full width.
//
// Phase 1 (decode_split_kernel): workgroup = 4 waves = one (sequence, K/V
//   head, chunk of `chunk` keys); the four waves take the chunk's 32-key
//   tiles in turn, so the workgroup streams its chunk front to back.  Scores
//   are formed transposed, S^T = K Q'^T: the 32 MFMA columns are the group's
//   query heads, replicated cyclically when the group has fewer than 32 (K and
//   V are then read once for all of them); every lane owns one head column, so
//   the softmax statistics stay in-lane as in the prefill kernel.  K tiles go
//   from HBM straight into registers as the A operand (lane = key row); V
//   tiles go through the wave's own LDS tile for the transpose read of
//   O^T += V^T P^T.  The first tile's loads are issued before the query is
//   loaded and rotated; each next tile's as soon as the current tile's score
//   MFMAs have consumed its keys, so one tile per wave is always in flight.
//   The register budget is held to two waves per SIMD so that two workgroups
//   stream on every CU at once.  Each wave then writes its own (m, l, acc)
//   partial for the group's G query heads straight from its registers (the
//   kernel has no barrier); chunks with no visible key return at once.
// Phase 2 (decode_combine_kernel): per (sequence, head), merge the wave
//   partials of the chunks that hold visible keys by log-sum-exp and write O
//   and LSE; the head's dims are spread over several workgroups so the merge
//   reads the partials with the whole chip, in one round trip to memory.
//
// Precision: without RoPE the bf16 query and keys meet exactly in a bf16
// MFMA.  With RoPE the query is rotated at position L-1 in fp32 and rounded to
// fp16, and the (already rotated) bf16 cache keys are widened to fp16 in
// registers (exact inside the fp16 range), as the prefill kernel does for its
// rotated operands.  P and V are bf16.
#include <atomic>

#include "common.hpp"
#include "launch.hpp"

// Device memory for the partials of callers that cannot allocate
// (attnfuse_decode_noalloc): one file-scope array, which every device the
// library runs on holds until the process ends.  In host code its name stands
// for a host-side shadow, not a device address; decode_scratch_ptr() looks the
// address up once per device and keeps it, and only that address is used.
static __device__ __align__(256) unsigned char scratch[af::DECODE_SCRATCH_BYTES];

namespace af {

namespace {
constexpr int kMaxScratchDevices = 64;
std::atomic<void*> g_scratch_ptr[kMaxScratchDevices];   // per device, resolved on first use
}  // namespace

void* decode_scratch_ptr() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxScratchDevices) return nullptr;
  void* ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (ptr) return ptr;
  if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return nullptr;
  g_scratch_ptr[dev].store(ptr, std::memory_order_release);
  return ptr;
}

template <int D>
struct DecCfg {
  static constexpr int NW = 4;                      // waves per workgroup
  static constexpr int KS = D / 16;                 // MFMA k-steps over the head dimension
  static constexpr int MT = D / 32;                 // 32-row output tiles over the head dimension
  static constexpr int VP = D + 16;                 // V tile pitch (transpose reads)
  static constexpr int VT = 32 * VP;                // one wave's V tile (elements)
  static constexpr int VPL = 32 * (D / 8) / 64;     // 16-byte V chunks per lane per tile
  static constexpr int SMEM = NW * VT;              // uint16 elements
};

__device__ __forceinline__ int seq_len(const DecodeParams& p, int b) {
  return p.lens ? min(p.lens[b], p.S) : p.S;
}

// First visible key of a sequence with L cached keys.
__device__ __forceinline__ int first_key(const DecodeParams& p, int L) {
  return (p.window > 0) ? max(0, L - p.window) : 0;
}

// ---------------------------------------------------------------- caches of different lengths
// With per-sequence lengths the even split of the longest possible cache
// leaves the workgroups of short sequences idle while others stream.  Here
// the pieces are sized from the lengths themselves: every sequence is cut into
// pieces of `c` 32-key tiles, c (a multiple of 4, the waves' step) the smallest
// (in steps of at most c / 16) for which all sequences together take at most
// p.slots pieces per K/V head: one round of resident workgroups.
// Every wave works this out for itself from the lengths (at most two loads per
// 64 sequences): the grid is fixed by the host at slots x H_kv, and the
// workgroups past the last piece return.  Even split / cut by length, us:
// B4 H64/8 cache 32768, lengths {32768, 16384, 8192, 24000} 78.9 / 68.7,
// {30000, 9000, 9000, 9000} 70.1 / 52.9; B6 H24/8, [8000, 32768] 122 / 80; B16
// H32/8 cache 8192, [2048, 8192] 75.7 / 68.2; B64 cache 4096, [100, 4096] 147 / 134.
__device__ __forceinline__ int visible_tiles(const DecodeParams& p, int b) {
  const int L = (b < p.B) ? seq_len(p, b) : 0;
  return L < 1 ? 0 : (L - (first_key(p, L) & ~31) + 31) / 32;
}

__device__ __forceinline__ int wave_sum(int x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}

// The wave's view of the plan: lane l holds sequence l's tiles (longer batches
// read the rest again each time).
struct Pieces {
  int own;   // tiles of sequence `lane`
  int c;     // tiles per piece
  __device__ __forceinline__ int tiles(const DecodeParams& p, int b0, int lane) const {
    return b0 == 0 ? own : visible_tiles(p, b0 + lane);
  }
  __device__ __forceinline__ int count(const DecodeParams& p, int b0, int lane) const {
    return (tiles(p, b0, lane) + c - 1) / c;
  }
  __device__ __forceinline__ Pieces(const DecodeParams& p, int lane) : own(visible_tiles(p, lane)) {
    int total = 0;
    for (int b0 = 0; b0 < p.B; b0 += 64) total += tiles(p, b0, lane);
    total = wave_sum(total);
    // c doubles at most: at ceil(total / (slots - B)) the pieces fit for certain
    const int sure = p.slots > p.B ? (total + p.slots - p.B - 1) / (p.slots - p.B) : 0x7ffffff0;
    for (c = max(4, ((total + p.slots - 1) / p.slots + 3) & ~3); c < sure; c += max(4, (c >> 4) & ~3)) {
      int n = 0;
      for (int b0 = 0; b0 < p.B; b0 += 64) n += count(p, b0, lane);
      if (wave_sum(n) <= p.slots) break;
    }
  }
  // The sequence that piece r belongs to (b = -1: past the last) and the
  // piece's index in it.
  __device__ __forceinline__ void find(const DecodeParams& p, int r, int lane, int& b, int& piece) const {
    int base = 0;
    for (int b0 = 0; b0 < p.B; b0 += 64) {
      const int n = count(p, b0, lane);
      int incl = n;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int x = __shfl_up(incl, o, 64);
        if (lane >= o) incl += x;
      }
      const unsigned long long hit = __ballot(base + incl > r);
      if (hit != 0ull) {
        const int l = __ffsll((long long)hit) - 1;
        b = b0 + l;
        piece = r - base - (__shfl(incl, l, 64) - __shfl(n, l, 64));
        return;
      }
      base += __shfl(incl, 63, 64);
    }
    b = -1;
    piece = 0;
  }
  // Pieces of the sequences before b.
  __device__ __forceinline__ int before(const DecodeParams& p, int b, int lane) const {
    int n = 0;
    for (int b0 = 0; b0 < b; b0 += 64) n += (b0 + lane < b) ? count(p, b0, lane) : 0;
    return wave_sum(n);
  }
};

template <int D, int ROPE, bool ALIBI, bool RAGGED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void decode_split_kernel(DecodeParams p) {
  using C = DecCfg<D>;
  constexpr bool QF16 = ROPE != ROPE_NONE;
  __shared__ __attribute__((aligned(16))) uint16_t smem[C::SMEM];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lq = lane & 31, lg = lane >> 5;
  const int G = p.H / p.Hkv;
  int b, g, split, chunk = p.chunk;
  if constexpr (RAGGED) {
    const Pieces pieces(p, lane);
    pieces.find(p, (int)(blockIdx.x / p.Hkv), lane, b, split);
    b = __builtin_amdgcn_readfirstlane(b);
    split = __builtin_amdgcn_readfirstlane(split);
    if (b < 0) return;                             // past the last piece (workgroup-uniform)
    g = (int)(blockIdx.x % p.Hkv);
    chunk = __builtin_amdgcn_readfirstlane(32 * pieces.c);
  } else {
    split = (int)(blockIdx.x % p.nsplit);
    const int u = (int)(blockIdx.x / p.nsplit);
    b = u / p.Hkv;
    g = u % p.Hkv;
  }
  const int unit = b * p.Hkv + g;
  const int L = seq_len(p, b);
  if (L < 1) return;
  const int lo = first_key(p, L);
  const int c0 = split * chunk + (RAGGED ? lo & ~31 : 0);
  if (c0 + chunk <= lo || c0 >= L) return;         // no visible key in this chunk (workgroup-uniform)
  const int pos = L - 1;                           // the query's position

  const int hc = lq % G;                           // head of this lane's column (cyclic replication)
  const int h = g * G + hc;
  const uint16_t* __restrict__ K = static_cast<const uint16_t*>(p.k) + (size_t)unit * p.S * D;
  const uint16_t* __restrict__ V = static_cast<const uint16_t*>(p.v) + (size_t)unit * p.S * D;

  const float c2 = p.scale * kLog2e;
  const float slope2 = ALIBI ? p.slopes[h] * kLog2e : 0.f;

  // This wave's tiles: every NW-th tile of the chunk from the wave's own,
  // starting at the first tile that holds a visible key.
  constexpr int STEP = 32 * C::NW;
  const int first = lo & ~31;
  const int kend = min(c0 + chunk, L);
  int kbeg = c0 + 32 * wave;
  if (kbeg < first) kbeg += (first - kbeg + STEP - 1) / STEP * STEP;

  uint16_t* Vw = smem + wave * C::VT;
  const int tr_key = 4 * lg + ((lane & 15) >> 2);
  const int tr_col = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);

  f32x16 acc[C::MT];
#pragma unroll
  for (int i = 0; i < C::MT; ++i) acc[i] = f32x16{};
  float m_run = -INFINITY, l_run = 0.f;

  u32x4 kreg[C::KS], vreg[C::VPL];
  auto load_tile = [&](int n0) {   // rows past L are clamped to L-1 (finite data, masked)
    const int n = min(n0 + lq, L - 1);
#pragma unroll
    for (int s = 0; s < C::KS; ++s) kreg[s] = ld16(K + (size_t)n * D + 16 * s + 8 * lg);
#pragma unroll
    for (int i = 0; i < C::VPL; ++i) {
      const int it = lane + 64 * i;
      const int r = it / (D / 8), c = it % (D / 8);
      vreg[i] = ld16(V + (size_t)min(n0 + r, L - 1) * D + 8 * c);
    }
  };

  if (kbeg < kend) load_tile(kbeg);
  // Query operand (B of S^T = K Q'^T): lane holds head column hc, dims 16s + 8lg .. +7.
  const uint16_t* __restrict__ Qh = static_cast<const uint16_t*>(p.q) + ((size_t)b * p.H + h) * D;
  u32x4 qreg[C::KS];
#pragma unroll
  for (int s = 0; s < C::KS; ++s) qreg[s] = ld16(Qh + 16 * s + 8 * lg);
  if constexpr (ROPE == ROPE_NEOX) {
#pragma unroll
    for (int s = 0; s < C::KS / 2; ++s)
      rotate_neox8<false, true>(qreg[s], qreg[s + C::KS / 2], p.table + (size_t)pos * (D / 2) + 16 * s + 8 * lg);
  } else if constexpr (ROPE == ROPE_INTERLEAVED) {
#pragma unroll
    for (int s = 0; s < C::KS; ++s)
      rotate_interleaved8<false, true>(qreg[s], p.table + (size_t)pos * (D / 2) + 8 * s + 4 * lg);
  }

  for (int n0 = kbeg; n0 < kend; n0 += STEP) {
    // V tile to this wave's LDS tile (the previous tile's transpose reads,
    // issued earlier by this wave, complete first: LDS is in order per wave)
#pragma unroll
    for (int i = 0; i < C::VPL; ++i) {
      const int it = lane + 64 * i;
      const int r = it / (D / 8), c = it % (D / 8);
      *reinterpret_cast<u32x4*>(Vw + r * C::VP + 8 * c) = vreg[i];
    }
    if constexpr (QF16) {   // cached keys bf16 -> fp16 to meet the fp16 query
#pragma unroll
      for (int s = 0; s < C::KS; ++s)
#pragma unroll
        for (int w = 0; w < 4; ++w) kreg[s][w] = pack_f16(bf_lo(kreg[s][w]), bf_hi(kreg[s][w]));
    }
    f32x16 st = f32x16{};
#pragma unroll
    for (int s = 0; s < C::KS; ++s) st = mfma32<QF16>(kreg[s], qreg[s], st);
    if (n0 + STEP < kend) load_tile(n0 + STEP);

    // element r: key n0 + 8 (r/4) + 4 lg + r%4 of head column lq
    if constexpr (ALIBI) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int n = n0 + 8 * (r >> 2) + 4 * lg + (r & 3);
        st[r] = __builtin_fmaf(st[r], c2, slope2 * (float)(n - pos));
      }
    }
    if (n0 + 32 > L || n0 < lo) {   // wave-uniform: edge tiles only
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int n = n0 + 8 * (r >> 2) + 4 * lg + (r & 3);
        st[r] = (n < L && n >= lo) ? st[r] : -INFINITY;
      }
    }
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, st[r]);
    mx = pair_max(mx);
    if constexpr (!ALIBI) mx *= c2;
    const float m_new = fmaxf(m_run, mx);
    if (__any(m_new > m_run + 8.f)) {   // raise the reference max (wave-uniform)
      const float alpha = (m_run == -INFINITY) ? 0.f : fast_exp2(m_run - m_new);
      l_run *= alpha;
#pragma unroll
      for (int i = 0; i < C::MT; ++i) acc[i] *= alpha;
      m_run = m_new;
    }
    const float m_use = (m_run == -INFINITY) ? 0.f : m_run;
    float pv[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      pv[r] = fast_exp2(ALIBI ? (st[r] - m_use) : __builtin_fmaf(st[r], c2, -m_use));
      l_run += pv[r];
    }
    u32x4 pop[2];
#pragma unroll
    for (int hf = 0; hf < 2; ++hf)
#pragma unroll
      for (int w = 0; w < 4; ++w) pop[hf][w] = pack_bf16(pv[8 * hf + 2 * w], pv[8 * hf + 2 * w + 1]);

    // O^T += V^T P^T (V^T from transpose reads of the row-major V tile)
#pragma unroll
    for (int hf = 0; hf < 2; ++hf)
#pragma unroll
      for (int mt = 0; mt < C::MT; ++mt) {
        const uint16_t* base = Vw + (16 * hf + tr_key) * C::VP + 32 * mt + tr_col;
        const u32x2 lo2 = lds_read_tr16(base);
        const u32x2 hi2 = lds_read_tr16(base + 8 * C::VP);
        const u32x4 a = {lo2[0], lo2[1], hi2[0], hi2[1]};
        acc[mt] = mfma32(a, pop[hf], acc[mt]);
      }
  }

  const float l_tot = pair_sum(l_run);
  if constexpr (RAGGED) {
    // One partial per piece (four times as many pieces fit the workspace as
    // with one per wave): the waves add theirs in LDS in turn, over the V
    // tiles, relative to the largest of their maxima.
    __shared__ float wm[C::NW][32], wl[C::NW][32];
    float* sum = reinterpret_cast<float*>(smem);   // [G][D]
    static_assert(32 * D * sizeof(float) <= C::SMEM * sizeof(uint16_t), "the sums fit the V tiles");
    if (lg == 0) {
      wm[wave][lq] = m_run;
      wl[wave][lq] = l_tot;
    }
    __syncthreads();
    float m_all = wm[0][lq];
#pragma unroll
    for (int w = 1; w < C::NW; ++w) m_all = fmaxf(m_all, wm[w][lq]);
    const float a = (m_run == -INFINITY) ? 0.f : fast_exp2(m_run - m_all);
#pragma unroll
    for (int w = 0; w < C::NW; ++w) {
      if (wave == w && lq < G) {
        float* dst = sum + lq * D + 4 * lg;
#pragma unroll
        for (int mt = 0; mt < C::MT; ++mt)
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) {
            float4* d = reinterpret_cast<float4*>(dst + 32 * mt + 8 * q4);
            float4 x = {a * acc[mt][4 * q4], a * acc[mt][4 * q4 + 1], a * acc[mt][4 * q4 + 2], a * acc[mt][4 * q4 + 3]};
            if (w > 0) {
              const float4 y = *d;
              x = float4{x.x + y.x, x.y + y.y, x.z + y.z, x.w + y.w};
            }
            *d = x;
          }
      }
      __syncthreads();
    }
    const int r = (int)(blockIdx.x / p.Hkv);
    for (int i = tid; i < G * (D / 4); i += 256) {
      const int hh = i / (D / 4), d4 = i % (D / 4);
      const size_t prow = (size_t)(g * G + hh) * p.slots + r;
      reinterpret_cast<float4*>(p.part_acc + prow * D)[d4] = reinterpret_cast<const float4*>(sum)[i];
    }
    if (tid < G) {
      float m = -INFINITY, l = 0.f;
#pragma unroll
      for (int w = 0; w < C::NW; ++w) m = fmaxf(m, wm[w][tid]);
#pragma unroll
      for (int w = 0; w < C::NW; ++w) l += (wm[w][tid] == -INFINITY) ? 0.f : wl[w][tid] * fast_exp2(wm[w][tid] - m);
      const size_t prow = (size_t)(g * G + tid) * p.slots + r;
      p.part_ml[prow * 2] = m;
      p.part_ml[prow * 2 + 1] = l;
    }
    return;
  }
  // One partial per wave, straight from registers: the first G head columns.
  const int nslot = p.nsplit * C::NW;
  if (lq < G) {
    const size_t prow = ((size_t)b * p.H + g * G + lq) * nslot + split * C::NW + wave;
    float* dst = p.part_acc + prow * D + 4 * lg;
#pragma unroll
    for (int mt = 0; mt < C::MT; ++mt)
#pragma unroll
      for (int a = 0; a < 4; ++a)
        *reinterpret_cast<float4*>(dst + 32 * mt + 8 * a) =
            float4{acc[mt][4 * a], acc[mt][4 * a + 1], acc[mt][4 * a + 2], acc[mt][4 * a + 3]};
    if (lg == 0) {
      p.part_ml[prow * 2] = m_run;
      p.part_ml[prow * 2 + 1] = l_tot;
    }
  }
}

// Fold the (max, sum) pair (m2, l2) into the running pair (m, l), log2 units.
__device__ __forceinline__ void merge_ml(float& m, float& l, float m2, float l2) {
  const float M = fmaxf(m, m2);
  if (M == -INFINITY) return;
  l = l * fast_exp2(m - M) + l2 * fast_exp2(m2 - M);
  m = M;
}

// Phase 2.  Workgroup = 256 threads = one (sequence, query head) and 32 of its
// dims, as eight groups of 32 threads that each take every eighth partial (4
// per chunk, one per wave).  Each thread loads its first PF partials'
// accumulators and maxima together with the statistics, so the merge costs
// one round trip to memory: each thread folds the (m, l) pairs it reads into
// a running pair, the pairs merge across the workgroup, and every thread
// weights its accumulators by 2^(m_s - M).
template <int D, int PF, bool RAGGED>
__global__ __launch_bounds__(256) void decode_combine_kernel(DecodeParams p) {
  __shared__ float red[256];
  __shared__ float wred[8];
  const int bh = blockIdx.x, t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int d = 32 * blockIdx.y + (t & 31), grp = t >> 5;
  const int b = bh / p.H;
  const int L = seq_len(p, b);
  uint16_t* O = static_cast<uint16_t*>(p.o) + (size_t)bh * D;
  if (L < 1) {   // workgroup-uniform
    if (grp == 0) O[d] = 0;
    if (t == 0 && blockIdx.y == 0) p.lse[bh] = -INFINITY;
    return;
  }
  int n;            // partials of this head, from row `row` of the workspace
  size_t row;
  if constexpr (RAGGED) {
    const Pieces pieces(p, lane);
    n = (visible_tiles(p, b) + pieces.c - 1) / pieces.c;
    row = (size_t)(bh % p.H) * p.slots + pieces.before(p, b, lane);
  } else {
    constexpr int NWV = DecCfg<D>::NW;   // partials per chunk
    const int s_lo = first_key(p, L) / p.chunk, s_hi = (L - 1) / p.chunk;
    n = (s_hi - s_lo + 1) * NWV;
    row = (size_t)bh * p.nsplit * NWV + s_lo * NWV;
  }
  const float* ml = p.part_ml + row * 2;
  const float* acc = p.part_acc + row * D + d;
  float a[PF], mm[PF];
#pragma unroll
  for (int j = 0; j < PF; ++j) {
    const int i = grp + 8 * j;
    a[j] = (i < n) ? acc[(size_t)i * D] : 0.f;
    mm[j] = (i < n) ? ml[2 * i] : -INFINITY;
  }
  float m = -INFINITY, l = 0.f;
  for (int i = t; i < n; i += 256) {
    const float2 v = *reinterpret_cast<const float2*>(ml + 2 * i);
    merge_ml(m, l, v.x, v.y);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) merge_ml(m, l, __shfl_xor(m, o), __shfl_xor(l, o));
  if (lane == 0) {
    wred[2 * wv] = m;
    wred[2 * wv + 1] = l;
  }
  __syncthreads();
  m = wred[0];
  l = wred[1];
#pragma unroll
  for (int w = 1; w < 4; ++w) merge_ml(m, l, wred[2 * w], wred[2 * w + 1]);
  float o = 0.f;
#pragma unroll
  for (int j = 0; j < PF; ++j) o += a[j] * fast_exp2(mm[j] - m);
  for (int i = grp + 8 * PF; i < n; i += 8) o += acc[(size_t)i * D] * fast_exp2(ml[2 * i] - m);
  red[t] = o;
  __syncthreads();
  if (grp == 0) {
    float sum = 0.f;
#pragma unroll
    for (int g = 0; g < 8; ++g) sum += red[32 * g + t];
    O[d] = static_cast<uint16_t>(pack_bf16(sum / l, 0.f) & 0xffffu);
    if (t == 0 && blockIdx.y == 0) p.lse[bh] = (m + __log2f(l)) * kLn2;
  }
}

template <int D, int ROPE, bool ALIBI>
static int launch_one(const DecodeParams& p, hipStream_t st) {
  const dim3 cgrid((unsigned)(p.B * p.H), D / 32);
  if (p.slots > 0) {   // sequences of different lengths
    hipLaunchKernelGGL((decode_split_kernel<D, ROPE, ALIBI, true>), dim3((unsigned)(p.slots * p.Hkv)), dim3(256), 0, st,
                       p);
    hipLaunchKernelGGL((decode_combine_kernel<D, 16, true>), cgrid, dim3(256), 0, st, p);
    return hipGetLastError() == hipSuccess ? 0 : -3;
  }
  const long long blocks = (long long)p.nsplit * p.B * p.Hkv;
  hipLaunchKernelGGL((decode_split_kernel<D, ROPE, ALIBI, false>), dim3((unsigned)blocks), dim3(256), 0, st, p);
  // preload depth: every partial of a head (8 groups x PF) when it fits
  if (p.nsplit * DecCfg<D>::NW <= 8 * 16)
    hipLaunchKernelGGL((decode_combine_kernel<D, 16, false>), cgrid, dim3(256), 0, st, p);
  else
    hipLaunchKernelGGL((decode_combine_kernel<D, 32, false>), cgrid, dim3(256), 0, st, p);
  return hipGetLastError() == hipSuccess ? 0 : -3;
}

// The mask is a runtime lower bound on the key index (p.window > 0 for a
// sliding window): NONE and CAUSAL see the same keys in decode.
template <int D>
static int dispatch_rope(int rope, bool alibi, const DecodeParams& p, hipStream_t st) {
  switch (rope) {
    case ROPE_NONE: return alibi ? launch_one<D, ROPE_NONE, true>(p, st) : launch_one<D, ROPE_NONE, false>(p, st);
    case ROPE_NEOX: return alibi ? launch_one<D, ROPE_NEOX, true>(p, st) : launch_one<D, ROPE_NEOX, false>(p, st);
    case ROPE_INTERLEAVED:
      return alibi ? launch_one<D, ROPE_INTERLEAVED, true>(p, st) : launch_one<D, ROPE_INTERLEAVED, false>(p, st);
  }
  return -2;
}

int launch_decode(int D, int rope, bool alibi, const DecodeParams& p, hipStream_t st) {
  if (D == 64) return dispatch_rope<64>(rope, alibi, p, st);
  if (D == 128) return dispatch_rope<128>(rope, alibi, p, st);
  return -2;
}

}  // namespace af
