// The wide kernels with probabilities and partial sums in 32 bits (cb_attn_wide.h).
#include "cb_attn_wide.h"

namespace cb {

// (two tiles to a wave up to 128 rows at head_dim 128, whose sweeps are long: attn_wide_two_tiles in cb_attn_wide.hip)
hipError_t launch_attn_wide_px(hipStream_t st, const AttnParams& p, const SeqMeta& meta, int n_tiles, const LogitsWork* lw) {
  if (p.kv.block_size > 0) {
    return p.D == 64 ? launch_wide<64, true, true, 1>(st, p, meta, n_tiles, lw) : launch_wide<128, true, true, 2>(st, p, meta, n_tiles, lw);
  }
  return p.D == 64 ? launch_wide<64, true, false, 1>(st, p, meta, n_tiles, lw) : launch_wide<128, true, false, 2>(st, p, meta, n_tiles, lw);
}

}  // namespace cb
