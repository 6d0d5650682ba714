// Fused forward, bf16 (fwd_kernel.hpp), on keys rotated once: a launch of the
// rotation kernel writes K' = R K in fp16 to the workspace (the values the
// one-launch forward forms in its loop, so the results are the same bits),
// then the forward stages K' tiles as they are.
#include "fwd_kernel.hpp"

namespace af {

template <int D>
static int dispatch_rope(int rope, int mask, bool alibi, int ext, const FwdParams& p, hipStream_t st) {
  switch (rope) {
    case ROPE_NEOX: return fwd_dispatch_mask<D, ROPE_NEOX, true>(mask, alibi, ext, p, st);
    case ROPE_INTERLEAVED: return fwd_dispatch_mask<D, ROPE_INTERLEAVED, true>(mask, alibi, ext, p, st);
  }
  return -2;
}

int launch_fwd_prerot(int D, int rope, int mask, bool alibi, int ext, const FwdParams& p, hipStream_t st) {
  RopeParams r{};
  r.x0 = p.k;
  r.y0 = p.k16;
  r.heads0 = p.Hkv;
  r.B = p.B;
  r.S = p.S;
  r.table = p.table;
  const int rc = launch_rope_f16(D, rope, r, st);
  if (rc != 0) return rc;
  if (D == 64) return dispatch_rope<64>(rope, mask, alibi, ext, p, st);
  if (D == 128) return dispatch_rope<128>(rope, mask, alibi, ext, p, st);
  return -2;
}

}  // namespace af
