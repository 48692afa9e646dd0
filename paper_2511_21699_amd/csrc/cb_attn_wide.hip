// The wide kernels with bf16 probabilities and partial sums (cb_attn_wide.h), and the choice among all of them.
#include "cb_attn_wide.h"

namespace cb {

// Tiles of 65 to 128 rows: four groups of one row tile, or two groups of two tiles with two key groups.  The two tiles read every operand
// for 64 rows -- a unit's operand reads are 64 KiB for four groups, 512 cycles of LDS beside 128 for its arrival, where its matrix
// instructions take 544 -- but a wave goes through them one behind the other, and the groups have states to combine.  So long sweeps
// take two.  A pass of the attention, two tiles -> four groups: 68 rows of 8 kv heads x 900 keys 12.2 -> 9.8 us, x 20000 29.0 -> 27.7; 128
// rows of 32 x 900 18.5 -> 14.9, x 20000 (2528 keys to a split) 73.8 -> 71.4, but paged 74.3 -> 75.8 and with 100 rows x 60000 187 -> 195;
// 70 rows x 60000 paged 184 -> 181; 8 sequences of up to 8000 paged keys in two splits 189 -> 186, of up to 16000 304 -> 308; 16 of up to
// 16384 in one split 401 -> 407.  With 32-bit sums at head_dim 128, whose slices are long, those take 586 -> 590.
bool attn_wide_two_tiles(const AttnParams& p, int rows) {
  return p.batch > 1 ? p.chunk > 4096 : p.kv.block_size > 0 && rows > 96 && p.chunk > 2048;
}

hipError_t launch_attn_wide(hipStream_t st, const AttnParams& p, const SeqMeta& meta, int rows, int n_tiles, const LogitsWork* lw) {
  if (p.move.words) return launch_attn_wide_step(st, p, meta, rows, n_tiles, lw);
  if (p.D == 64 || p.precise) return launch_attn_wide_px(st, p, meta, n_tiles, lw);
  const bool two = attn_wide_two_tiles(p, rows);
  if (p.kv.block_size > 0) {
    return two ? launch_wide<128, false, true, 2>(st, p, meta, n_tiles, lw) : launch_wide<128, false, true, 1>(st, p, meta, n_tiles, lw);
  }
  return two ? launch_wide<128, false, false, 2>(st, p, meta, n_tiles, lw) : launch_wide<128, false, false, 1>(st, p, meta, n_tiles, lw);
}

}  // namespace cb
