// Fused forward, bf16 (fwd_kernel.hpp), one launch: key tiles rotated as they
// are staged.
#include "fwd_kernel.hpp"

namespace af {

template <int D>
int launch_fwd_norope(int mask, bool alibi, int ext, const FwdParams& p, hipStream_t st);   // fwd_norope.hip

template <int D>
static int dispatch_rope(int rope, int mask, bool alibi, int ext, const FwdParams& p, hipStream_t st) {
  switch (rope) {
    case ROPE_NONE: return launch_fwd_norope<D>(mask, alibi, ext, p, st);
    case ROPE_NEOX: return fwd_dispatch_mask<D, ROPE_NEOX, false>(mask, alibi, ext, p, st);
    case ROPE_INTERLEAVED: return fwd_dispatch_mask<D, ROPE_INTERLEAVED, false>(mask, alibi, ext, p, st);
  }
  return -2;
}

int launch_fwd_bf16(int D, int rope, int mask, bool alibi, int ext, const FwdParams& p, hipStream_t st) {
  if (D == 64) return dispatch_rope<64>(rope, mask, alibi, ext, p, st);
  if (D == 128) return dispatch_rope<128>(rope, mask, alibi, ext, p, st);
  return -2;
}

}  // namespace af
