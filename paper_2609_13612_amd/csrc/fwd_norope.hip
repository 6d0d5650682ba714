// Fused forward, bf16 (fwd_kernel.hpp), without RoPE (a unit of its own so
// that the forward's instantiations compile in parallel).
#include "fwd_kernel.hpp"

namespace af {

template <int D>
int launch_fwd_norope(int mask, bool alibi, int ext, const FwdParams& p, hipStream_t st) {
  return fwd_dispatch_mask<D, ROPE_NONE, false>(mask, alibi, ext, p, st);
}

template int launch_fwd_norope<64>(int, bool, int, const FwdParams&, hipStream_t);
template int launch_fwd_norope<128>(int, bool, int, const FwdParams&, hipStream_t);

}  // namespace af
