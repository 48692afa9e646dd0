// The wide kernels with the compaction in the launch (cb_attn_wide.h).
#include "cb_attn_wide.h"

namespace cb {

template <int D, bool PX, bool PG, int R128>
static hipError_t launch(hipStream_t st, const AttnParams& p, const SeqMeta& meta, int n_tiles, const LogitsWork& lw) {
  hipLaunchKernelGGL((k_step_wide<D, PX, PG, R128>), dim3(n_tiles + lw.n_wgs), dim3(64 * kWideWaves), 0, st, p, meta, lw);
  return hipGetLastError();
}

// (the builds of one layer's launches: cb_attn_wide.hip, cb_attn_wide_px.hip)
hipError_t launch_attn_wide_step(hipStream_t st, const AttnParams& p, const SeqMeta& meta, int rows, int n_tiles, const LogitsWork* logits_work) {
  const LogitsWork lw = logits_work ? *logits_work : LogitsWork{};
  const bool paged = p.kv.block_size > 0;
  if (p.D == 64) return paged ? launch<64, true, true, 1>(st, p, meta, n_tiles, lw) : launch<64, true, false, 1>(st, p, meta, n_tiles, lw);
  if (p.precise) return paged ? launch<128, true, true, 2>(st, p, meta, n_tiles, lw) : launch<128, true, false, 2>(st, p, meta, n_tiles, lw);
  if (attn_wide_two_tiles(p, rows)) {
    return paged ? launch<128, false, true, 2>(st, p, meta, n_tiles, lw) : launch<128, false, false, 2>(st, p, meta, n_tiles, lw);
  }
  return paged ? launch<128, false, true, 1>(st, p, meta, n_tiles, lw) : launch<128, false, false, 1>(st, p, meta, n_tiles, lw);
}

}  // namespace cb
