// dK/dV pass, one workgroup per key block (dkdv_kernel.hpp).
#include "dkdv_kernel.hpp"

namespace af {

int launch_bwd_dkdv_bf16(int D, int rope, int mask, bool alibi, int ext, const BwdParams& p, hipStream_t st) {
  if (p.splits > 1) return launch_bwd_dkdv_split(D, rope, mask, alibi, ext, p, st);
  return bwd_dispatch<DkdvPass<false>>(D, rope, mask, alibi, ext, p, st);
}

}  // namespace af
