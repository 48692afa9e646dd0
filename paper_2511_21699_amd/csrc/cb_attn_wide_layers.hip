// The wide kernels that serve several layers in a launch (cb_attn_wide.h).
#include "cb_attn_wide.h"

namespace cb {

template <int D, bool PX, bool PG, int R128>
static hipError_t launch(hipStream_t st, const AttnParams& p, const SeqMeta& meta, int n_tiles, const LogitsWork& lw, const LayerTable& layers) {
  hipLaunchKernelGGL((k_model_wide<D, PX, PG, R128>), dim3(n_tiles + lw.n_wgs), dim3(64 * kWideWaves), 0, st, p, meta, lw, layers);
  return hipGetLastError();
}

// (the builds of one layer's launches: cb_attn_wide.hip, cb_attn_wide_px.hip)
hipError_t launch_attn_wide_layers(hipStream_t st, const AttnParams& p, const SeqMeta& meta, int rows, int n_tiles, const LogitsWork& lw, const LayerTable& layers) {
  const bool paged = p.kv.block_size > 0;
  if (p.D == 64) return paged ? launch<64, true, true, 1>(st, p, meta, n_tiles, lw, layers) : launch<64, true, false, 1>(st, p, meta, n_tiles, lw, layers);
  if (p.precise) return paged ? launch<128, true, true, 2>(st, p, meta, n_tiles, lw, layers) : launch<128, true, false, 2>(st, p, meta, n_tiles, lw, layers);
  if (attn_wide_two_tiles(p, rows)) {
    return paged ? launch<128, false, true, 2>(st, p, meta, n_tiles, lw, layers) : launch<128, false, false, 2>(st, p, meta, n_tiles, lw, layers);
  }
  return paged ? launch<128, false, true, 1>(st, p, meta, n_tiles, lw, layers) : launch<128, false, false, 1>(st, p, meta, n_tiles, lw, layers);
}

}  // namespace cb
