// Host side of libcacheback_verify.so: argument checks, workspace layout, launch planning and the
// extern "C" entry points declared in cacheback.h.  No arithmetic of the method happens here.
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <vector>
#include <mutex>
#include <new>

#include "cb_logits.h"

using namespace cb;

namespace {

thread_local char g_init_err[256] = "";

// Scratch memory of cb_tree_attention_noalloc: a fixed array in the library's own device image
// (every GPU the library runs on holds one copy until the process ends).  In host code the array's
// name is only a handle: its address on a device comes from hipGetSymbolAddress, once per device.
constexpr size_t kStaticScratchBytes = 32u << 20;
__device__ __align__(256) unsigned char g_static_scratch[kStaticScratchBytes];
constexpr int kMaxDevices = 64;
void* g_static_scratch_ptr[kMaxDevices];  // per device, filled on first use (under g_static_mutex)
std::mutex g_static_mutex;

constexpr size_t kAlign = 256;
size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

struct WsLayout {
  size_t anc, parent, tokens, amax_best, amax_out, path, len_ctx, res_len, res_tok, new_len, status,
      tickets, coop_tickets, amax_tickets, moves, dbg, partial, total;
  int amax_chunks;
  int max_total_nodes;
  int max_splits;
  int scalar_splits;  // split count the scalar kernel's fp32 partials have room for
  int ticket_count;
};

int effective_max_splits(const cb_config& c) { return c.max_splits > 0 ? c.max_splits : 64; }

bool config_ok(const cb_config* c, char* err, size_t n) {
  auto fail = [&](const char* m) {
    if (err && n) snprintf(err, n, "config: %s", m);
    return false;
  };
  if (!c) return fail("null");
  if (c->num_q_heads < 1 || c->num_kv_heads < 1 || c->num_q_heads % c->num_kv_heads != 0)
    return fail("num_q_heads must be a positive multiple of num_kv_heads");
  if (c->num_q_heads > 1024) return fail("num_q_heads > 1024");
  if (c->head_dim != 64 && c->head_dim != 128) return fail("head_dim must be 64 or 128");
  if ((c->qkv_dtype != CB_F32 && c->qkv_dtype != CB_BF16) || (c->logits_dtype != CB_F32 && c->logits_dtype != CB_BF16))
    return fail("dtype must be CB_F32 or CB_BF16");
  if (c->max_batch < 1 || c->max_batch > CB_MAX_BATCH) return fail("max_batch out of range");
  if (c->max_nodes < 1 || c->max_nodes > CB_MAX_NODES) return fail("max_nodes out of range");
  if (c->max_depth < 0 || c->max_depth >= CB_MAX_NODES) return fail("max_depth out of range");
  if (c->vocab_size < 1) return fail("vocab_size < 1");
  if (c->block_size < 0 || c->block_size > 65536) return fail("block_size out of range");
  if (c->max_splits < 0 || c->max_splits > 4096) return fail("max_splits out of range");
  return true;
}

WsLayout ws_layout(const cb_config& c) {
  WsLayout L{};
  const size_t mt = (size_t)c.max_batch * c.max_nodes;
  const size_t stride = (size_t)c.max_depth + 1;
  L.max_total_nodes = (int)mt;
  L.max_splits = effective_max_splits(c);
  L.amax_chunks = (int)(((int64_t)c.vocab_size + kArgmaxChunk - 1) / kArgmaxChunk);
  const int g = c.num_q_heads / c.num_kv_heads;
  // two 64-bit words per tile; at least 1024 of those, for launches that serve several layers
  L.ticket_count = std::max(4096, 4 * c.max_batch * c.num_kv_heads * ((c.max_nodes * g + kRowTile - 1) / kRowTile));
  size_t o = 0;
  auto take = [&](size_t bytes) { size_t at = o; o = align_up(o + bytes); return at; };
  L.anc = take(mt * kAncWords * 4);
  L.parent = take(mt * 4 * 2);  // staged tree of the host-array form: parents, then tokens right behind them
  L.tokens = L.parent;         // (placed per call)
  L.amax_out = take(mt * 4);
  L.path = take(c.max_batch * stride * 4);
  L.len_ctx = take(c.max_batch * 4);
  L.res_len = take(c.max_batch * (1 + stride) * 4);  // results of the host-array form: lengths, then tokens right behind them
  L.res_tok = L.res_len;                              // (placed per call)
  L.new_len = take(c.max_batch * 4);
  // from here to the timing table: the words that start at zero, cleared together by cb_init
  L.status = take(4);
  L.tickets = take((size_t)L.ticket_count * 4);
  L.coop_tickets = take((size_t)kCoopTiles * kCoopTicketStride);
  L.amax_tickets = take((size_t)c.max_batch * kTicketWords * 4);
  L.amax_best = take(mt * kAmaxStride * 8);
  L.moves = take((size_t)c.max_batch * c.num_kv_heads * 4);
  L.dbg = take(1024 * 8 * 8);
  // The scalar kernel's fp32 partials are twice the size of the MFMA kernel's.  A configuration
  // the MFMA kernel takes (bf16) runs the scalar one only on request (option
  // "attn_impl" = 1, a test aid) or when its geometry is not the MFMA kernel's (see Planner::cut): it gets
  // room for 8 splits there, not for max_splits.
  const bool mfma_cfg = c.qkv_dtype == CB_BF16;
  L.scalar_splits = mfma_cfg ? std::min(L.max_splits, 8) : L.max_splits;
  const size_t scalar_bytes = mt * c.num_q_heads * (size_t)L.scalar_splits * partial_stride(c.head_dim) * 4;
  auto mfma_partials = [&](int tile_rows) { return attn_mfma_partial_bytes(c.head_dim, c.head_dim == 64, tile_rows, mt, c.num_q_heads, c.num_kv_heads, c.max_batch, L.max_splits); };
  const size_t mfma_bytes = mfma_cfg ? std::max(mfma_partials(kRowTile), mfma_partials(attn_mfma_tile_rows(c.max_nodes * g))) : 0;  // (calls with small tiles, and with wide ones)
  L.partial = take(std::max(scalar_bytes, mfma_bytes));
  L.total = o;
  return L;
}

// Whether a bf16 call holds probabilities and partial sums in 32 bits: with head_dim 64, and with head_dim 128 where a split's
// slice of the block table has more than 1022 entries, as the scalar kernel did that served these two before the MFMA
// kernels took them; their callers keep that precision (plan_call).
bool precise_sums(const cb_config& c, int chunk) {
  return c.qkv_dtype == CB_BF16 && (c.head_dim == 64 || (c.block_size > 0 && chunk / c.block_size + 2 > 1024));
}

struct Plan {
  bool precise;  // (impl 2)
  int logits_wgs;  // of a verification: workgroups of the attention's launch that do the logits work (0: a launch of their own)
  int tile_rows;  // (impl 2)
  int impl;    // 1 fp32 (or the scalar kernel on request), 2 bf16 MFMA
  int nsplit;  // partial slots per row
  int chunk;   // keys per split
  int max_nodes, max_len;
};

}  // namespace

struct cb_ctx {
  cb_config cfg;
  WsLayout lay;
  char* ws;
  // pinned host mirror
  int32_t* h_parent;
  int32_t* h_tokens;
  int32_t* h_len;
  int32_t* h_tok;
  int32_t* h_path;
  int32_t* h_argmax;
  int32_t* h_misc;  // [0] status, [1..] new_len
  int32_t* h_last;  // [max_batch] last nodes of the host form's accepted paths
  int32_t* h_done;  // [max_batch] arrival flags of the host form's results (the call's sequence number)
  int32_t call_seq = 0;        // sequence number of the last host-form call (never 0 once used)
  int32_t* want_done = nullptr;  // these two are set by cb_verify_tree for the launch it is about to make
  int32_t* want_last = nullptr;
  hipStream_t unsynced = nullptr;  // stream that may still run the tail of a host-form call that has returned
  bool have_unsynced = false;
  int32_t* d_hblock = nullptr;  // the pinned block's address on the device
  void* h_block;
  // state of the last verify
  bool have_verify;
  int32_t launch_info[6];
  bool host_knows_len;
  bool nothing_moves;  // of the last verification, where the host knows its lengths
  int batch;
  int total_nodes;
  SeqMeta meta;
  int32_t last_len[CB_MAX_BATCH];
  hipStream_t last_stream;
  // options
  int64_t opt_splits, opt_impl, opt_time, opt_stages, opt_timeline, opt_external, opt_fork, opt_fuse, opt_coop, opt_spin, opt_full_sync, opt_logits_wgs, opt_tile_rows;
  hipEvent_t ev0, ev1, ev_fork, ev_join;
  hipStream_t aux;  // second stream (default priority) for the logits scan beside the attention
  bool ev_valid;
  const Plan* fixed_plan = nullptr;  // (cb_tree_attention_noalloc: the plan its scratch layout was cut for)
  bool want_move = false;  // the launch that run_pipeline makes next is to compact its cache too, if it can;
  bool moved = false;      // whether it does
  int32_t step_info[4] = {};  // (cb_debug_step)
  bool counters_dirty = false;  // a launch failed: the tickets may be left non-zero
  bool amax_dirty = false;      // a scan ran without its acceptance (option "stages"): row maxima are left behind
  char err[256];

  template <typename T>
  T* dev(size_t off) const { return reinterpret_cast<T*>(ws + off); }
};

namespace {

int set_err(cb_ctx* ctx, int code, const char* fmt, ...) {
  char* dst = ctx ? ctx->err : g_init_err;
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(dst, 256, fmt, ap);
  va_end(ap);
  return code;
}

#define CB_HIP(ctx, call)                                                                         \
  do {                                                                                            \
    hipError_t e__ = (call);                                                                      \
    if (e__ != hipSuccess) return set_err(ctx, CB_EHIP, "%s: %s", #call, hipGetErrorString(e__)); \
  } while (0)
// the same for the launches of run_pipeline: a failure there may leave tickets behind
#define CB_LAUNCH(ctx, call)                                                                      \
  do {                                                                                            \
    hipError_t e__ = (call);                                                                      \
    if (e__ != hipSuccess) {                                                                      \
      (ctx)->counters_dirty = true;                                                               \
      return set_err(ctx, CB_EHIP, "%s: %s", #call, hipGetErrorString(e__));                     \
    }                                                                                             \
  } while (0)

bool make_kv_addr(const cb_config& c, const cb_kv_layer& l, KvAddr* a) {
  const int64_t D = c.head_dim, H = c.num_kv_heads;
  a->k = l.k;
  a->v = l.v;
  a->block_table = l.block_table;
  a->max_blocks = l.max_blocks_per_seq;
  a->block_size = c.block_size;
  // (the kernels compare in 32 bits; a pool of more blocks than a table entry can name is one whose descriptor says so only: K and V of
  // that many of the smallest are 512 GiB)
  a->num_blocks = c.block_size > 0 ? std::min<int64_t>(l.capacity_or_num_blocks, INT32_MAX) : 0;
  const int64_t tokens_per_unit = c.block_size > 0 ? c.block_size : l.capacity_or_num_blocks;
  a->seq_stride = tokens_per_unit * H * D;
  if (l.layout == CB_LAYOUT_TOKEN_MAJOR) {
    a->token_stride = H * D;
    a->head_stride = D;
  } else if (l.layout == CB_LAYOUT_HEAD_MAJOR) {
    a->token_stride = D;
    a->head_stride = tokens_per_unit * D;
  } else {
    return false;
  }
  return true;
}

// A stretch of the device's address space.
struct Span {
  const void* at;
  size_t bytes;
  bool meets(const Span& o) const {
    const uintptr_t a = (uintptr_t)at, b = (uintptr_t)o.at;
    return a < b ? b - a < bytes && o.bytes != 0 : a - b < o.bytes && bytes != 0;
  }
};
// Bytes of a layer's K (or V) that a call with `batch` sequences can touch, by the descriptor (whose capacity may be just a large number: at
// most half of the address space, from where it begins).
size_t cache_bytes(const cb_config& c, const cb_kv_layer& l, int batch) {
  const size_t row = (size_t)c.num_kv_heads * c.head_dim * (c.qkv_dtype == CB_F32 ? 4 : 2), per_unit = row * (c.block_size > 0 ? c.block_size : batch);
  const size_t units = l.capacity_or_num_blocks > 0 ? l.capacity_or_num_blocks : 0;
  return std::min(units, (SIZE_MAX / 2) / per_unit) * per_unit;
}
bool same_cache(const cb_kv_layer& a, const cb_kv_layer& b) {
  return a.k == b.k && a.v == b.v && a.capacity_or_num_blocks == b.capacity_or_num_blocks && a.block_table == b.block_table &&
         a.max_blocks_per_seq == b.max_blocks_per_seq && a.layout == b.layout;
}

// Workgroups of a one-launch verification that do the logits work: the share of the chip that the logits' bytes
// have in the call's, in whole XCD rounds of 8, at least 8, at most what gives each of their 8 wavefronts an item.
int fused_logits_wgs(const cb_config& c, int batch, const int32_t* kv_len, const int32_t* node_offsets) {
  const int64_t eb = c.qkv_dtype == CB_F32 ? 4 : 2, lb = c.logits_dtype == CB_F32 ? 4 : 2;
  const int64_t rows = node_offsets[batch];
  int64_t slots = rows;
  for (int b = 0; b < batch; b++) slots += kv_len[b];
  const double kv = (double)slots * c.num_kv_heads * c.head_dim * 2 * eb, lg = (double)rows * c.vocab_size * lb;
  const int64_t items = rows * (((int64_t)c.vocab_size + kArgmaxChunk - 1) / kArgmaxChunk);
  const int share = (int)(256.0 * lg / (lg + kv));
  const int most = (int)std::min<int64_t>(192, (items + 7) / 8);
  return std::max(8, std::min(share, most) / 8 * 8);
}

// What splitting a call's sequences into chunks of so many keys means.  Its jobs are (sequence, kv head, row tile, chunk with keys);
// work is counted in stages of 64 keys, with six for what a job costs beside its sweep (start-up and tail).
struct SplitSums {
  int chunk;
  int grid_x;             // chunks of the longest sequence
  int64_t jobs, merged;   // merged: tiles that have partial states
  double work, shortest;
  double longest_chunk, longest_whole;  // job, of a sequence that is split and of one that is not
  double longest(double merge) const { return std::max(longest_chunk > 0.0 ? longest_chunk + merge : 0.0, longest_whole); }
};

// The split plan of one call's attention.  Pure host arithmetic: no device call, no context state beyond the numbers passed in.
// What a split count means for a batch is worked out once, whatever number of plans is made.
struct Planner {
  const cb_config& c;
  const int max_splits, scalar_splits, opt_splits, batch;
  const int32_t *const kv_len, *const node_offsets;
  const bool f32_tiles;
  const int impl, g;
  int max_nodes = 0, max_len = 0, tile_rows = 0;
  int64_t rows = 0, keys = 0;     // query rows of all heads; (row tile, key) pairs
  int32_t len[CB_MAX_BATCH];
  int64_t tiles[CB_MAX_BATCH];
  static constexpr int kKnown = 64;   // (the default for max_splits)
  SplitSums known[kKnown + 2];        // of the counts up to kKnown, and the last one beyond,
  int32_t known_chunk[kKnown + 2] = {};  // where this is their chunk

  Planner(const cb_config& c_, int max_splits_, int scalar_splits_, int opt_impl, int opt_splits_, int batch_, const int32_t* kv_len_, const int32_t* node_offsets_,
          int tile_rows_ = 0)
      : c(c_), max_splits(max_splits_), scalar_splits(scalar_splits_), opt_splits(opt_splits_), batch(batch_), kv_len(kv_len_), node_offsets(node_offsets_),
        f32_tiles(c_.qkv_dtype == CB_F32 && opt_impl != 1), impl(opt_impl == 1 || c_.qkv_dtype != CB_BF16 ? 1 : 2), g(c_.num_q_heads / c_.num_kv_heads) {
    for (int b = 0; b < batch; b++) {
      const int n = node_offsets[b + 1] - node_offsets[b];
      len[b] = kv_len[b] + n;
      max_nodes = std::max(max_nodes, n);
      max_len = std::max(max_len, len[b]);
      rows += (int64_t)n * c.num_q_heads;
    }
    tile_rows = tile_rows_ ? tile_rows_ : attn_mfma_tile_rows(max_nodes * g);
    for (int b = 0; b < batch; b++) {
      tiles[b] = (int64_t)(((node_offsets[b + 1] - node_offsets[b]) * g + tile_rows - 1) / tile_rows) * c.num_kv_heads;
      keys += tiles[b] * len[b];
    }
  }
  int cap() const { return (int)std::max<int64_t>(1, std::min<int64_t>(max_splits, (max_len + 127) / 128)); }
  int chunk_of(int ns) const { return ((max_len + ns - 1) / ns + 31) / 32 * 32; }

  const SplitSums& split_into(int ns) {
    const int at = std::min(ns, kKnown + 1), chunk = chunk_of(ns);
    SplitSums& s = known[at];
    if (known_chunk[at] == chunk) return s;
    known_chunk[at] = chunk;
    s = SplitSums{};
    s.chunk = chunk;
    s.grid_x = (max_len + s.chunk - 1) / s.chunk;
    s.shortest = 1e30;
    const double job_chunk = 6.0 + (s.chunk + 63) / 64, per_key = 1.0 / s.chunk;
    for (int b = 0; b < batch; b++) {
      int full = (int)(len[b] * per_key);  // (a division, off by one at most)
      full += (int64_t)(full + 1) * s.chunk <= len[b];
      full -= (int64_t)full * s.chunk > len[b];
      const int rest = len[b] - full * s.chunk, real = full + (rest > 0 ? 1 : 0);
      const double job_rest = rest > 0 ? 6.0 + ((rest + 63) >> 6) : 0.0, job = full > 0 ? job_chunk : job_rest;
      s.work += tiles[b] * (full * job_chunk + job_rest);
      s.jobs += tiles[b] * real;
      if (real > 1) s.merged += tiles[b];
      double& longest = real > 1 ? s.longest_chunk : s.longest_whole;
      longest = std::max(longest, job);
      s.shortest = std::min(s.shortest, job);
    }
    return s;
  }

  // What a batch in `ns` splits is expected to take on `units` compute units, in stages.
  double batch_cost(int ns, int units, bool empty_wgs) {
    const SplitSums& s = split_into(ns);
    const int tiles_max = (max_nodes * g + tile_rows - 1) / tile_rows;
    const double merge = s.grid_x > 1 ? 0.7 * s.grid_x * (tile_rows / 128.0) : 0.0;
    const double empty = empty_wgs ? (double)((int64_t)c.num_kv_heads * tiles_max * s.grid_x * batch - s.jobs) : 0.0;
    return s.jobs <= units ? s.longest(merge) : std::max(s.longest(merge), (s.work + s.merged * merge + empty) / units + s.shortest);
  }

  // The split count on `units` compute units (those that the attention's workgroups can count on).  empty_wgs: as if a batch's grid
  // held a workgroup for every split of its longest sequence.
  int splits(int units, bool empty_wgs) {
    if (opt_splits > 0) return opt_splits;
    if (impl == 1 && f32_tiles) {
      return attn_f32_splits(c.num_q_heads, c.num_kv_heads, c.head_dim, scalar_splits, batch, kv_len, node_offsets, max_len, units);
    }
    if (impl == 1) {
      // one workgroup per (row, split): aim for a few workgroups per compute unit, but never split
      // below 1024 keys -- a second (merge) launch costs more than a short row does
      const int64_t want = 2048;
      return (int)std::max<int64_t>(1, std::min<int64_t>((want + rows - 1) / rows, max_len / 1024));
    }
    // one workgroup per (row tile of 64 or 256 rows, kv head, split)
    const int last = cap(), tiles_max = (max_nodes * g + tile_rows - 1) / tile_rows;
    if (batch > 1 && (c.num_kv_heads * tiles_max) % 8 == 0) {
      // Several sequences, launched longest first within every XCD (see the kernel's workgroup
      // numbering).  Such a list schedule ends no later than max(longest job, work / units + a job
      // of the shortest sequence), so: estimate that for every split count, with what a tile's merge costs its last
      // workgroup (and one stage for every workgroup that finds no keys, where such are launched), and take the cheapest count -- the
      // fewest splits that still spread the longest sequence wide enough.
      empty_wgs |= c.num_kv_heads % 8 != 0;
      double best = 0.0;
      int nsplit = 1;
      for (int ns = 1; ns <= last; ns++) {
        if (ns > 1 && chunk_of(ns) == chunk_of(ns - 1)) continue;  // (keys per split are a multiple of 32: the same plan)
        const double cost = batch_cost(ns, units, empty_wgs);
        if (ns == 1 || cost < best - 1e-9) { best = cost; nsplit = ns; }
      }
      return nsplit;
    }
    // Every variant has a ring of more than half of the LDS: one workgroup per compute unit, so the grid
    // should come out just under a whole number of rounds of `units` workgroups.  Take the fewest
    // splits that fill >= 85% of them in whole rounds (fewer splits = fewer partials).
    // efficiency of ns splits: keys swept / (units x whole rounds x keys of a full split)
    auto efficiency = [&](int ns) {
      const SplitSums& s = split_into(ns);
      const int64_t rounds = (s.jobs + units - 1) / units;
      return (double)keys / ((double)rounds * units * s.chunk);
    };
    int nsplit = last;
    double best = -1.0;
    for (int ns = 1; ns <= last; ns++) {
      const double eff = efficiency(ns);
      if (eff >= 0.85) { nsplit = ns; best = eff; break; }
      if (eff > best) { best = eff; nsplit = ns; }
    }
    // A grid of one round merges cooperatively (no workgroup pulls a whole tile's partials), so
    // there more splits cost next to nothing: take the best-filling count among the one-round ones.
    if (best >= 0.85 && split_into(nsplit).jobs <= units) {
      for (int ns = nsplit + 1; ns <= last && ns <= 64 && split_into(ns).jobs <= units; ns++) {
        const double eff = efficiency(ns);
        if (eff > best + 1e-9) { best = eff; nsplit = ns; }
      }
    }
    return nsplit;
  }

  // The plan with (about) ns splits.  `precise`: sums in 32 bits whatever the slices' length.
  Plan cut(int ns, bool precise) const {
    Plan p{};
    p.impl = impl;
    p.tile_rows = tile_rows;
    p.max_nodes = max_nodes;
    p.max_len = max_len;
    const int most = impl == 1 ? scalar_splits : max_splits;
    ns = std::max(1, std::min(ns, most));
    p.chunk = std::max(chunk_of(ns), 32);
    p.precise = impl == 2 && (precise || precise_sums(c, p.chunk));
    if (p.precise && c.head_dim == 128 && ns > 1 && ns > most / 2) {
      // fp32 partial states are twice the size, and the workspace is cut for bf16 ones (longer splits stay precise)
      ns = std::max(1, most / 2);
      p.chunk = chunk_of(ns);
    }
    p.nsplit = (max_len + p.chunk - 1) / p.chunk;
    if (impl == 2) {
      // A geometry that the MFMA kernel does not take (blocks that are no power of two, say) goes to the scalar kernel,
      // whose fp32 partials have room for fewer splits: it is planned as such.
      AttnParams ap{};
      ap.Hq = c.num_q_heads;
      ap.Hkv = c.num_kv_heads;
      ap.D = c.head_dim;
      ap.nsplit = p.nsplit;
      ap.precise = p.precise;
      ap.kv.block_size = c.block_size;
      if (!attn_mfma_supports(ap)) {
        Planner scalar(c, max_splits, scalar_splits, 1, opt_splits, batch, kv_len, node_offsets);
        return scalar.cut(scalar.splits(256, false), false);
      }
    }
    return p;
  }
  Plan plan(int units, bool empty_wgs) { return cut(splits(units, empty_wgs), false); }
};

// Workgroups for the logits work of a verification with wide tiles, whose sweep is bound by its arithmetic: the fewest (in XCD
// rounds, at most 96) that are through with the logits, at about 20 GB/s each, in 0.7 of the time the attention takes: 13 us
// beside the sweep and, per 32 keys, 0.95 us with a tile of more than 128 rows and 0.55 with a smaller one.  Where rows are short a
// wave's round trip for each bounds them, 2.1 us (kLogitsItemUs for its workgroup): 2080 rows of 1000 entries beside 16 sequences of up
// to 1300 keys, 32 heads: 8 workgroups 139 us, 16 80, 48 78, a launch of their own 85.  Fewer keep the
// launch (a pass of 8 sequences of 32/8 heads with 250 rows of 33333 entries: 32 workgroups 41.7 us, 48 33.7; 128 rows
// of 32000 over 8192 keys: 8 44.5, 16 34.0, 24 33.5), more take compute units from the sweep (the batch with 96: 38.4).
// 0: a launch of their own, where the logits are more than 2.5 times the K/V bytes.  Results then come earlier, which pays where the
// host has work to do with them: 48 nodes of 32/8 heads of 64 x 3000 keys, 128256 fp32 entries (3.9 times), marshalled on the spot,
// 35.6 us a call in two launches and 38.3 in one.  (A device step of that shape would take 18.4 in one and 27.1 in two, and 128 nodes of head_dim
// 128 x 2048 keys with 7.8 times the bytes 29.8 and 38.1: the line is low for those.)  Below it one launch is faster in every form:
// 128 nodes x 2048 keys, 32000-entry rows (as many bytes) 22 against 30 us a device step and 25.6 against 32.4 a host one.
// 0 too for tiles of up to 128 rows in several rounds of workgroups, unless their sums are in 32 bits: those sweeps are bound by
// memory (5.5 TB/s) and there is little to hide behind.  It is near the line: 16 sequences of up to 16384 keys with 32 to 96 nodes, 32
// heads, a verification: one draw 425 us in two launches and 434 in one, another 538 and 528; with 32-bit sums 595 and 580.
constexpr double kLogitsItemUs = 2.1 / 4;
int fused_wide_logits_wgs(const cb_config& c, const Plan& alone, int batch, const int32_t* kv_len, const int32_t* node_offsets, double item_us) {
  const double lb = c.logits_dtype == CB_F32 ? 4 : 2;
  const int g = c.num_q_heads / c.num_kv_heads, rows = std::min(attn_mfma_tile_rows(alone.max_nodes * g), alone.max_nodes * g);
  double slots = 0, jobs = 0;
  for (int b = 0; b < batch; b++) {
    const int n = node_offsets[b + 1] - node_offsets[b], len = kv_len[b] + n;
    slots += len;
    jobs += (double)((n * g + 255) / 256) * c.num_kv_heads * len / alone.chunk;
  }
  const double kv = slots * c.num_kv_heads * c.head_dim * 4, lg = (double)node_offsets[batch] * c.vocab_size * lb;
  if (lg > 2.5 * kv) return 0;
  if (rows <= 128 && !alone.precise && jobs > 256) return 0;
  const double us = 13.0 + alone.chunk / 32 * (rows > 128 ? 0.95 : 0.55) * std::max(1.0, jobs / 256);
  const double items = (double)node_offsets[batch] * ((c.vocab_size + kArgmaxChunk - 1) / kArgmaxChunk);
  return std::min(96, ((int)(std::max(lg / 20e3, items * item_us) / (0.7 * us)) / 8 + 1) * 8);
}

// What a verification with wide tiles in `ns` splits is expected to take, in us: with `wgs` workgroups of its launch for the logits, or (0)
// with a launch of their own in front.  A stage of the sweep takes about 1.7 us in tiles of more than 128 rows and 1.0 in smaller ones;
// a logits workgroup scans about 20 GB/s of bf16 and, bound by its instructions, 40 of fp32.
double wide_verification_us(Planner& planner, int ns, int wgs) {
  const cb_config& c = planner.c;
  const SplitSums& s = planner.split_into(ns);
  const double stage = std::min(planner.tile_rows, planner.max_nodes * planner.g) > 128 ? 1.7 : 1.0, memory = 5.5e6;  // (bytes a us)
  const double lb = c.logits_dtype == CB_F32 ? 4 : 2, lg = (double)planner.node_offsets[planner.batch] * c.vocab_size * lb;
  double kv = 0.0;
  for (int b = 0; b < planner.batch; b++) kv += (double)planner.len[b] * c.num_kv_heads * c.head_dim * 4;
  const double merge = planner.batch > 1 && s.grid_x > 1 ? 0.8 * s.grid_x : 0.0, items = (double)planner.node_offsets[planner.batch] * ((c.vocab_size + kArgmaxChunk - 1) / kArgmaxChunk);
  const double scan = wgs ? std::max(lg / (lb * 10e3), items * kLogitsItemUs) / wgs / stage : 0.0;
  double stages = std::max(s.longest(merge), scan);
  if (s.jobs + wgs > 256) {
    // (a batch's longest-first schedule, the logits' workgroups in front, ends between work / units and that plus its shortest job)
    if (planner.batch == 1) stages = (double)((s.jobs + wgs + 255) / 256) * s.longest(merge);
    else stages = std::max(stages, (s.work + s.merged * merge + wgs * scan) / 256 + 0.5 * s.shortest);
  }
  return std::max(stages * stage, (kv + (wgs ? lg : 0.0)) / memory) + (wgs ? 0.0 : lg / 5e6 + 4.0);
}

// The split count of a verification with wide tiles and the workgroups of its launch for the logits (0: a launch of their own),
// chosen among few by what they are expected to take.  `beside` splits are planned for the units that n workgroups leave, `alone` for all
// of them.
// One sequence keeps to one round of workgroups, the logits' among them, so that its splits are merged cooperatively: 72 rows of 40
// heads x 3303 keys, 128256 entries: 360 workgroups beside 64 for the logits 41 us a pass, 160 beside 64 28.8, 240 behind a logits launch 35.8;
// 880 rows of 32/8 heads x 3183 keys: 352 beside 72 51.8, 160 beside 72 41, 256 behind a launch 43.4.  In a batch of several rounds
// the logits' workgroups are jobs of the schedule like the others, and units are free again when they are through: 6 sequences of
// up to 5247 keys, 32/8 heads x 92 nodes: two splits beside 40 90 us, three 72, three behind a launch 80; 8 of up to 1829 keys, 32 heads x
// 225 nodes: one split each behind a launch 117, beside 96 126.
int wide_verification_splits(Planner& planner, int alone, int beside, int n, bool whole, int forced_wgs, int* logits_wgs) {
  const cb_config& c = planner.c;
  auto share = [&](int ns) {
    const int wgs = fused_wide_logits_wgs(c, planner.cut(ns, false), planner.batch, planner.kv_len, planner.node_offsets, kLogitsItemUs);
    return wgs && forced_wgs > 0 ? forced_wgs : wgs;
  };
  if (planner.batch == 1 && n && planner.split_into(beside).jobs + n > 256 && planner.split_into(1).jobs + n <= 256) {
    for (beside = 1; beside < planner.cap() && planner.split_into(beside + 1).jobs + n <= 256;) beside++;
  }
  struct { int ns, wgs; } const options[] = {{whole ? 1 : (n ? alone : beside), 0}, {whole ? 1 : beside, whole ? share(1) : n}, {alone, planner.batch > 1 && !whole ? share(alone) : 0}};
  double best = 0.0;
  int nsplit = 0;
  for (const auto& o : options) {
    if (nsplit != 0 && o.wgs == 0) continue;
    const double us = wide_verification_us(planner, o.ns, o.wgs);
    if (nsplit != 0 && us >= best) continue;
    best = us;
    nsplit = o.ns;
    *logits_wgs = o.wgs;
  }
  return nsplit;
}

constexpr int kTallest = 256;  // option "tile_rows": the smallest tile that holds a kv head's rows, at most this

// What one round of workgroups with tiles of `rows` of a head's rows takes, in us (head_dim 128): start and tail, less of both without partial
// states (splits 1), and what 32 keys of the longest split cost, more while the ring fills.  Taller tiles read, park, write and merge more rows beside
// the sweep; shorter ones read the same keys again, from the L2.  A merge is shared out among a tile's splits: up to three have larger slices, which
// shows where a head has two tiles.  Verifications, splits x units: two tiles of 64 rows 4 x 4 10.0, 7 x 5 10.1, 15 x 14 14.9, 3 x 5
// 11.5, 3 x 8 13.0, 3 x 10 14.1; one of 128 with 66 rows 5 x 4 11.2, with 97 12.1, with 128 12.5.
double round_us(int rows, int head_rows, int chunk, int splits) {
  const double units = chunk / 32, early = std::min(units, 9.0), late = units - early;
  if (rows > 128) return splits > 1 ? 14.5 + 0.85 * units : 5.5 + 1.95 * early + 0.85 * late;
  if (rows > 64) return splits > 1 ? (head_rows > 128 ? 10.5 : 9.4 + 0.022 * (head_rows - 66)) + 0.5 * units : 5.0 + 1.05 * early + 0.5 * late;
  return splits > 1 ? 8.0 + 0.45 * units + (splits <= 3 && head_rows <= 128 ? 0.9 : 0.0) : 5.0 + 0.8 * early + 0.5 * late;
}

// The same of a call's round: its longest job.  (A sequence whose rows a shorter tile would hold costs what that does.)
double round_us(const Planner& pl, const SplitSums& s) {
  double us = 0.0;
  for (int b = 0; b < pl.batch; b++) {
    const int head_rows = (pl.node_offsets[b + 1] - pl.node_offsets[b]) * pl.g, keys = std::min(pl.len[b] + 31, s.chunk);
    const int rows = pl.tile_rows == kRowTile ? kRowTile : std::max(std::min(head_rows, pl.tile_rows), kRowTile + 1);
    // (a batch's tiles are not in step with each other: 8 sequences of up to 2000 keys, 32/8 heads x up to 48 nodes, 1024 keys to a
    // split 28.9 us)
    us = std::max(us, round_us(rows, head_rows, keys, (pl.len[b] + s.chunk - 1) / s.chunk) + (pl.batch > 1 && rows <= 128 ? 0.05 * keys / 32 : 0.0));
  }
  return us;
}

// Calls whose tiles leave compute units idle, or whose splits are so short that start and tail are most of them, take shorter tiles: those of
// 128 or 64 rows where the launch is still one round and expected to be faster by more than the estimates are off.  The attention alone, a
// pass in us with tiles of 256, 128 and 64 rows: 256 rows of 8 kv heads x 500 keys 16.3, 10.9, 9.5, x 4000 17.0, 13.6, 15.7, x 16000
// 29.3, 26.5, 40.0; 512 rows x 8000 28.5, 26.8, 40.2, x 16000 41.5, 43.3, 73.9; 256 rows of 32 kv heads x 200 keys 20.3, 13.6, 13.6, x
// 4000 33.5, 29.7, 44.6, x 8000 46.2, 47.5, 78.3; 128 rows of 8 kv heads x 1000 keys in 128 and 64 12.8, 10.3, x 8000 17.5, 16.0, x
// 16000 21.8, 24.4, of 32 x 500 12.6, 11.1, x 2000 16.2, 16.9.  Steps of batches: 3 sequences of 32/8 heads x 353 keys x 123 nodes, 128256 entries
// 48.9, 39.9, 38.4, 8 of up to 1246 keys x 42 nodes 27.0, 23.4, 29.7, 3 of 32 heads x 240 keys x 90 nodes 19.3, 18.9, 15.1.
void shorter_tiles(Planner& tall, int rows, bool verification, int forced, Plan* p, double* us) {
  if (rows >= p->tile_rows || (forced && forced != rows) || (p->precise && tall.c.head_dim == 128)) return;
  const cb_config& c = tall.c;
  Planner planner(c, tall.max_splits, tall.scalar_splits, 0, 0, tall.batch, tall.kv_len, tall.node_offsets, rows);
  int n = verification ? p->logits_wgs : 0;
  if (n && rows == kRowTile) n = std::max(n, fused_logits_wgs(c, tall.batch, tall.kv_len, tall.node_offsets));
  const int cap = p->nsplit == 1 ? 1 : std::min(planner.cap(), 64);  // (what is not split stays so: plan_call)
  const double limit = *us - std::max(0.3, 0.03 * *us);
  double best = forced ? 1e30 : limit;
  int ns = 0;
  for (int i = 1; i <= cap; i++) {
    if (i > 1 && planner.chunk_of(i) == planner.chunk_of(i - 1)) continue;
    const SplitSums& s = planner.split_into(i);
    if (s.jobs + n > 256 && !(forced && i == 1)) break;
    // (what is in 16 bits stays so: longer slices of the block table would put the sums in 32, at up to twice the time of the estimate, which
    // is that of 16-bit ones: 6 sequences of up to 17612 paged keys, 32 heads x up to 82 nodes, 418 us in one split instead of 201 in two)
    if (precise_sums(c, s.chunk) != p->precise) continue;
    const double t = round_us(planner, s);
    if (t >= best) continue;
    best = t;
    ns = i;
  }
  if (ns == 0) return;
  const bool precise = p->precise;
  *p = planner.cut(ns, precise);
  p->logits_wgs = n;
  *us = best;
}

// The plan of a call, a verification or the attention alone.
// What a call holds in 32 bits is a property of its shape that callers rely on, so it is decided by measures of the shape, whatever the
// kernels would like to have: the splits planned as if the logits never rode beside wide tiles and a batch's grid held a
// workgroup for every split of its longest sequence (empty_wgs), and those planned without either.  A call is precise where the
// slices of one of them are long; one that a measure does not split, whose sums stay in the accumulators to the end, is not
// split (partial states are bf16).
Plan plan_call(const cb_config& c, int max_splits, int scalar_splits, int opt_impl, int opt_splits, int opt_logits_wgs, int opt_tile_rows, int batch,
               const int32_t* kv_len, const int32_t* node_offsets, bool verification) {
  Planner planner(c, max_splits, scalar_splits, opt_impl, opt_splits, batch, kv_len, node_offsets);
  // A verification in fp32, or with small tiles, or whose logits hide behind the sweep, is one launch: its first workgroups do the logits work, and the
  // attention is planned for the compute units they leave (with option "fuse_logits" = 0 too, so that the
  // option does not change the splits and with them the rounding).
  const bool wide = planner.tile_rows != kRowTile && !planner.f32_tiles;
  int n_logits = 0, n_launched = 0;
  if (!verification) {
  } else if (!wide) {
    n_logits = fused_logits_wgs(c, batch, kv_len, node_offsets);
  } else if (planner.impl == 2) {
    const Plan alone = planner.plan(248, false);
    if (alone.impl == 2) {
      n_logits = fused_wide_logits_wgs(c, alone, batch, kv_len, node_offsets, 0.0);  // (as the measure has it: by bytes)
      n_launched = fused_wide_logits_wgs(c, alone, batch, kv_len, node_offsets, kLogitsItemUs);
    }
  }
  if (n_logits && opt_logits_wgs > 0) n_logits = n_launched = opt_logits_wgs;
  Plan p;
  if (planner.impl == 1) {
    p = planner.plan(256 - n_logits, false);
  } else {
    const int units = wide ? 256 : 256 - n_logits, measured = planner.splits(units, true);
    const bool same = units == 256 - n_logits && (batch == 1 || c.num_kv_heads % 8 != 0);  // (empty_wgs makes no difference)
    int nsplit = same ? measured : planner.splits(256 - n_logits, false);
    const Plan m0 = planner.cut(measured, false), m1 = same ? m0 : planner.cut(nsplit, false);
    const bool precise = m0.precise || m1.precise, whole = (m0.impl == 2 && m0.nsplit == 1 && !m0.precise) || m1.nsplit == 1;
    if (whole) nsplit = 1;
    if (verification && wide && opt_splits <= 0 && m1.impl == 2) {
      nsplit = wide_verification_splits(planner, measured, nsplit, n_launched, whole, opt_logits_wgs, &n_logits);
    } else if (wide) {
      n_logits = n_launched;
    } else if (verification && batch > 1 && !whole && opt_splits <= 0) {
      // The units of the logits' workgroups are free again soon: a batch whose jobs are more than the others, but no more than
      // all, is through when the last of them are, some 8 stages late, and merged by the last to arrive.  3 sequences of 11316 to 17155
      // paged keys, 32 heads: 192 workgroups beside 8 for the logits 189 us, 256 behind them 135.6.  (Not where the K/V take as long in any case,
      // 1.05 us a stage: 2 of 15000 keys 91.1 beside, 98.7 behind, 2 of 19672 and 24432 139 and 146.)
      double slots = 0;
      for (int b = 0; b < batch; b++) slots += planner.len[b];
      const double memory = slots * c.num_kv_heads * c.head_dim * 4 / 5.5e6 / 1.05;
      double best = 0.92 * std::max(memory, planner.batch_cost(nsplit, 256 - n_logits, false));
      for (int ns = nsplit + 1; ns <= planner.cap(); ns++) {
        const SplitSums& s = planner.split_into(ns);
        if (s.jobs > 256) break;
        const double cost = std::max(memory, s.longest(0.7 * s.grid_x * (planner.tile_rows / 128.0)) + 8.0);
        if (s.jobs <= 256 - n_logits || cost >= best) continue;
        best = cost;
        nsplit = ns;
      }
    }
    p = planner.cut(nsplit, precise);
  }
  p.logits_wgs = n_logits;
  if (p.impl == 2 && planner.tile_rows > kRowTile && opt_splits <= 0 && opt_tile_rows != kTallest) {
    const SplitSums& tall = planner.split_into(p.nsplit);
    double us = 2.5 + (double)((tall.jobs + p.logits_wgs + 255) / 256) * (round_us(planner, tall) - 2.5);
    for (const int shorter : {128, 64}) shorter_tiles(planner, shorter, verification, opt_tile_rows, &p, &us);
  }
  return p;
}

// A launch that serves several layers.
struct ModelLaunch {
  Plan plan;
  LayerTable table;
};

// The scratch layout of a cb_tree_attention_noalloc call, and the plan it is cut for.  Whether a call fits the fixed array
// is a property of its shape that callers rely on, so it is decided by one measure per kind of call, whatever the
// kernels would like to have: bf16 states in 16-row tiles at the planned splits for bf16 with head_dim 128, fp32 rows at the
// splits of one workgroup per row for the others.  The measure's splits are planned as if a batch's grid held a workgroup for
// every split of its longest sequence (empty_wgs): plans that launch fewer workgroups take more splits, and calls that
// fit would be refused.  A call within it gets its plan, with fewer splits if the kernels' own
// layout at the planned ones is larger than the array (one split needs no partial states, so an end is always found).
WsLayout noalloc_layout(const cb_config& c, const WsLayout& full, int batch, const int32_t* kv_len, const int32_t* node_offsets, Plan* plan) {
  const size_t total = node_offsets[batch];
  const int g = c.num_q_heads / c.num_kv_heads;
  auto fp32_rows = [&](int ns) { return ns <= 1 ? 0 : total * c.num_q_heads * ns * partial_stride(c.head_dim) * 4; };
  auto tiles = [&](bool precise, int rows, int ns) {
    return ns <= 1 ? 0 : attn_mfma_partial_bytes(c.head_dim, precise, rows, total, c.num_q_heads, c.num_kv_heads, batch, ns);
  };
  auto planned = [&](int most) {
    return plan_call(c, most, std::min(most, full.scalar_splits), 0, 0, 0, 0, batch, kv_len, node_offsets, false);
  };
  auto cut = [&](size_t partial_bytes) {
    WsLayout L{};
    L.max_total_nodes = (int)total;
    L.max_splits = L.scalar_splits = plan->nsplit;
    L.amax_chunks = full.amax_chunks;
    L.ticket_count = 4 * batch * c.num_kv_heads * ((plan->max_nodes * g + kRowTile - 1) / kRowTile);
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o = align_up(o + bytes); return at; };
    L.status = take(4);
    L.tickets = take((size_t)L.ticket_count * 4);
    L.coop_tickets = take((size_t)kCoopTiles * kCoopTicketStride);
    L.anc = take(total * kAncWords * 4);
    L.dbg = L.anc;  // (never written: the timing aid is off)
    L.partial = take(partial_bytes);
    L.total = o;
    return L;
  };
  *plan = planned(full.max_splits);
  const int measured = Planner(c, full.max_splits, full.scalar_splits, 0, 0, batch, kv_len, node_offsets).plan(256, true).nsplit;
  const bool by_rows = c.qkv_dtype == CB_F32 || c.head_dim == 64;
  const size_t measure = by_rows ? fp32_rows(Planner(c, full.max_splits, full.max_splits, 1, 0, batch, kv_len, node_offsets).plan(256, false).nsplit)
                         : plan->impl == 2 ? tiles(false, kRowTile, measured) : fp32_rows(measured);
  WsLayout L = cut(measure);
  if (L.total > kStaticScratchBytes) return L;
  for (;;) {
    L = cut(plan->impl == 2 ? tiles(plan->precise, plan->tile_rows, plan->nsplit) : fp32_rows(plan->nsplit));
    if (L.total <= kStaticScratchBytes || plan->nsplit <= 1) return L;
    *plan = planned(plan->nsplit - 1);
  }
}

// The attention of several layers as one launch, where all their queries are there.  A layer's launch by itself is a chain of latencies --
// start, first data, partial states, merge, drain -- that fills the chip with splits of a few hundred keys; together the layers
// fill it with whole sequences (32 layers of 64 nodes x 32 heads x 2048 keys: 1024 workgroups of one split each, four rounds, and
// nothing to merge).
// Splits are for steps whose tiles leave compute units idle (2 layers of 8 kv heads), in the first round of workgroups or in the last.  A call that is not split when its layers are launched one by one, whose sums stay in the accumulators, is not
// split here.  False: launched one by one, where that is expected to be faster (few long tiles and no room for their partial states).
bool plan_layers(const cb_config& c, const WsLayout& lay, int layers, int batch, const int32_t* kv_len, const int32_t* node_offsets, ModelLaunch* out) {
  const Plan last = plan_call(c, lay.max_splits, lay.scalar_splits, 0, 0, 0, kTallest, batch, kv_len, node_offsets, true);
  const Plan other = plan_call(c, lay.max_splits, lay.scalar_splits, 0, 0, 0, kTallest, batch, kv_len, node_offsets, false);
  if (last.impl != other.impl) return false;
  Planner planner(c, lay.max_splits, lay.scalar_splits, 0, 0, batch, kv_len, node_offsets);
  const int total = node_offsets[batch];
  const size_t room = lay.total - lay.partial;
  // The logits' workgroups come first.  Where the launch has several rounds their compute units go on with the attention afterwards: as
  // many as give each wavefront one item, so that no unit starts late.  In one round, the fewest that are through in 0.7 of the time.
  const double lb = c.logits_dtype == CB_F32 ? 4 : 2, lg = (double)total * c.vocab_size * lb;
  const int64_t items = total * (((int64_t)c.vocab_size + kArgmaxChunk - 1) / kArgmaxChunk);
  auto logits_wgs = [&](bool rounds, double us, int waves) {
    const int64_t most = std::min<int64_t>(192, (items + waves - 1) / waves);
    const int64_t want = rounds ? most : std::min<int64_t>(96, (int64_t)(std::max(lg / 20e3, items * kLogitsItemUs) / (0.7 * us)));
    return (int)(std::max<int64_t>(want, 1) + 7) / 8 * 8;
  };
  Plan& p = out->plan;
  if (planner.f32_tiles) {
    double us = 0.0, one = 0.0;
    auto splits = [&](int most, int n, double* t) { return attn_f32_splits(c.num_q_heads, c.num_kv_heads, c.head_dim, most, batch, kv_len, node_offsets, planner.max_len, 248, n, t); };
    splits(lay.scalar_splits, 1, &one);
    const size_t per_split = (size_t)total * c.num_q_heads * partial_stride(c.head_dim) * 4;
    const int tiles = batch * c.num_kv_heads * ((planner.max_nodes * planner.g + 15) / 16);
    const bool tickets = (int64_t)tiles * layers <= lay.ticket_count;
    const int ns = splits(tickets ? (int)std::max<int64_t>(1, std::min<int64_t>(lay.scalar_splits, room / (per_split * layers))) : 1, layers, &us);
    if (us > (one + 4.0) * layers) return false;
    p = planner.cut(ns, false);
    out->table.partial_bytes = p.nsplit > 1 ? (int64_t)per_split * p.nsplit : 0;
    p.logits_wgs = logits_wgs((int64_t)tiles * layers * p.nsplit > 248, us, 8);
    return true;
  }
  if (last.impl != 2) return false;
  const bool precise = last.precise || other.precise, whole = last.nsplit == 1 || other.nsplit == 1;
  double kv = 0.0;
  for (int b = 0; b < batch; b++) kv += (double)planner.len[b] * c.num_kv_heads * c.head_dim * 4;
  // Of one launch for n layers: rounds of equal jobs, or the longest-first schedule of a batch's; 6 of SplitSums' stages are a job's start
  // and tail.  A merge
  // takes 1 us, by the last workgroup to arrive 1.5 and a little for every split.
  auto us_of = [&](Planner& pl, int ns, int n) {
    const SplitSums& s = pl.split_into(ns);
    const int64_t jobs = s.jobs * n;
    const bool split = s.grid_x > 1;
    const double merge = !split ? 0.0 : jobs <= 240 ? 1.0 : 1.5 + 0.4 * s.grid_x * (pl.tile_rows / 128.0);
    // (with tiles of 64 rows a unit keeps a compute unit's memory pipe busy for 0.53 us: 2 layers of 40 heads x 17085 keys)
    const double start = (pl.tile_rows == 256 ? 9.5 : 7.0) + (split ? 1.0 : 0.0) - 2.5 + merge, stage = (pl.tile_rows == 256 ? 1.7 : pl.tile_rows == 128 ? 1.0 : 1.06) * c.head_dim / 128;
    const double longest = start + stage * s.chunk / 64;
    const double us = batch == 1 ? (double)((jobs + 255) / 256) * longest
                                 : std::max(longest, jobs > 256 ? ((s.work - 6.0 * s.jobs) * stage + s.jobs * start) * n / 256 + 0.5 * (start + (s.shortest - 6.0) * stage) : 0.0);
    return 2.5 + std::max(us, n * kv / 5.5e6);
  };
  const double one = us_of(planner, other.nsplit, 1);
  double us = 0.0;
  Plan& best = out->plan;
  best.impl = 0;
  for (int rows = planner.tile_rows; rows >= kRowTile && !(precise && c.head_dim == 128 && rows != planner.tile_rows); rows = rows == 256 ? 128 : rows / 2) {
    Planner pl(c, lay.max_splits, lay.scalar_splits, 0, 0, batch, kv_len, node_offsets, rows);
    const int64_t tiles = (int64_t)batch * c.num_kv_heads * ((pl.max_nodes * pl.g + rows - 1) / rows) * layers;  // as the tickets are numbered
    for (int ns = 1; ns <= (whole || tiles > std::min(kCoopTiles, lay.ticket_count / 4) ? 1 : std::min(pl.cap(), 64)); ns++) {
      if (ns > 1 && pl.chunk_of(ns) == pl.chunk_of(ns - 1)) continue;
      const Plan cut = pl.cut(ns, precise);
      const size_t bytes = cut.nsplit > 1 ? attn_mfma_partial_bytes(c.head_dim, cut.precise, rows, total, c.num_q_heads, c.num_kv_heads, batch, cut.nsplit) : 0;
      if (cut.impl != 2 || bytes * layers > room) break;
      if (cut.precise != precise) continue;  // (longer slices of the block table than the layers have one by one: plan_call decides what is in 32 bits)
      const double t = us_of(pl, ns, layers);
      if ((best.impl && t >= us) || (cut.nsplit > 1 && !attn_mfma_merges_inside(c.head_dim, cut.precise, pl.max_nodes * pl.g, rows, cut.nsplit))) continue;
      us = t;
      best = cut;
      best.logits_wgs = logits_wgs(tiles * cut.nsplit + 8 > 256, us, rows != kRowTile ? 4 : 8);
      out->table.partial_bytes = (int64_t)bytes;
    }
  }
  return best.impl == 2 && us <= 0.96 * one * layers;  // (2 layers of 8 sequences x 4105 keys, 32/8 heads x 180 nodes: 271 us together, 254 one by one)
}

int check_common(cb_ctx* ctx, int32_t batch, const void* q, const cb_kv_layer* kv, const int32_t* kv_len,
                 const int32_t* node_offsets, const void* logits, void* attn_out) {
  if (!ctx) return set_err(nullptr, CB_EINVAL, "null context");
  if (!q || !kv || !kv_len || !node_offsets || !logits || !attn_out)
    return set_err(ctx, CB_EINVAL, "null argument");
  if (batch < 1 || batch > ctx->cfg.max_batch) return set_err(ctx, CB_EINVAL, "batch %d outside [1, %d]", batch, ctx->cfg.max_batch);
  if (((uintptr_t)q | (uintptr_t)kv->k | (uintptr_t)kv->v | (uintptr_t)logits | (uintptr_t)attn_out) & 15)
    return set_err(ctx, CB_EINVAL, "device pointers must be 16-byte aligned");
  return CB_OK;
}

// A host-form call returns when its results arrive; what is left of its launches still reads the cache and uses the
// workspace, and only work on that same stream is ordered behind it.  Work on another stream waits here.
int order_behind_host_form(cb_ctx* ctx, hipStream_t st) {
  if (ctx->have_unsynced && ctx->unsynced != st) {
    CB_HIP(ctx, hipStreamSynchronize(ctx->unsynced));
    ctx->have_unsynced = false;
  }
  return CB_OK;
}

// Enqueues the whole verification on `st`; the tree is already on the device.  model: the attention of all layers of its table (q, kv and
// attn_out are the first one's).
int run_pipeline(cb_ctx* ctx, hipStream_t st, int batch, const void* q, const cb_kv_layer* kv,
                 const int32_t* kv_len, const int32_t* node_offsets, const int32_t* d_parent,
                 const int32_t* d_tokens, const void* logits, void* attn_out, int32_t* d_len, int32_t* d_tok,
                 int64_t stage_mask = 15, const ModelLaunch* model = nullptr) {
  const cb_config& c = ctx->cfg;
  SeqMeta meta{};
  for (int b = 0; b < batch; b++) meta.kv_len[b] = kv_len[b];
  for (int b = 0; b <= batch; b++) meta.node_off[b] = node_offsets[b];
  for (int b = 0; b < batch; b++) meta.by_length[b] = b;
  std::stable_sort(meta.by_length, meta.by_length + batch, [&](int32_t x, int32_t y) {
    return (int64_t)kv_len[x] + node_offsets[x + 1] - node_offsets[x] > (int64_t)kv_len[y] + node_offsets[y + 1] - node_offsets[y];
  });
  const int total = node_offsets[batch];
  const int ordered = order_behind_host_form(ctx, st);
  if (ordered) return ordered;
  if (ctx->counters_dirty) {  // (after a failed launch: the kernels rely on tickets that are zero between launches)
    const hipError_t e1 = launch_zero_words(st, ctx->dev<unsigned long long>(ctx->lay.tickets), ctx->lay.ticket_count / 2, 1, 1);
    const hipError_t e2 = launch_zero_words(st, ctx->dev<unsigned long long>(ctx->lay.coop_tickets), kCoopTiles, kCoopTicketStride / 8, 2);
    const hipError_t e3 = launch_zero_words(st, ctx->dev<unsigned long long>(ctx->lay.amax_tickets), c.max_batch * kTicketWords / 2, 1, 1);
    const hipError_t e4 = launch_zero_words(st, ctx->dev<unsigned long long>(ctx->lay.moves), (c.max_batch * c.num_kv_heads + 1) / 2, 1, 1);
    if (e1 != hipSuccess || e2 != hipSuccess || e3 != hipSuccess || e4 != hipSuccess) return set_err(ctx, CB_EHIP, "clearing the tickets after a failed launch failed");
    ctx->counters_dirty = false;
    ctx->amax_dirty = ctx->amax_dirty || (stage_mask & 4) != 0;  // (the row maxima too)
  }
  if (ctx->amax_dirty && (ctx->opt_stages & stage_mask & 12) == 12) {
    CB_HIP(ctx, launch_zero_words(st, ctx->dev<unsigned long long>(ctx->lay.amax_best), ctx->lay.max_total_nodes, kAmaxStride, 1));
    ctx->amax_dirty = false;
  }
  const bool f32_tiles = c.qkv_dtype == CB_F32 && ctx->opt_impl != 1;
  const Plan plan = model             ? model->plan
                    : ctx->fixed_plan ? *ctx->fixed_plan
                                    : plan_call(c, ctx->lay.max_splits, ctx->lay.scalar_splits, (int)ctx->opt_impl, (int)ctx->opt_splits, (int)ctx->opt_logits_wgs, (int)ctx->opt_tile_rows,
                                                batch, kv_len, node_offsets, (stage_mask & 8) != 0);
  const int n_logits = plan.logits_wgs;

  AttnParams ap{};
  ap.q = q;
  ap.out = attn_out;
  if (!make_kv_addr(c, *kv, &ap.kv)) return set_err(ctx, CB_EINVAL, "unknown cache layout %d", kv->layout);
  ap.anc = ctx->dev<uint32_t>(ctx->lay.anc);
  ap.parent = d_parent;
  ap.partial = ctx->dev<float>(ctx->lay.partial);
  ap.tickets = ctx->dev<uint32_t>(ctx->lay.tickets);
  ap.coop_tickets = ctx->dev<uint32_t>(ctx->lay.coop_tickets);
  ap.Hq = c.num_q_heads;
  ap.Hkv = c.num_kv_heads;
  ap.D = c.head_dim;
  ap.chunk = plan.chunk;
  ap.nsplit = plan.nsplit;
  ap.precise = plan.precise;
  ap.batch = batch;
  if (plan.impl == 2) {
    const int g = c.num_q_heads / c.num_kv_heads, rows = plan.tile_rows;
    ap.tile_rows = rows;
    const int64_t layers = model ? model->table.count : 1;
    int64_t live = 0;  // per kv head and layer
    for (int i = 0; i < CB_MAX_BATCH; i++) {
      meta.start[i] = INT32_MAX;
      if (i >= batch) continue;
      const int b = meta.by_length[i];
      const int64_t n = node_offsets[b + 1] - node_offsets[b];
      meta.start[i] = (int32_t)(live * (c.num_kv_heads / 8) * layers);
      live += (n * g + rows - 1) / rows * ((kv_len[b] + n + plan.chunk - 1) / plan.chunk);
    }
    ap.live_wgs = (int32_t)(live * c.num_kv_heads * layers);
  }
  ap.scale = c.softmax_scale > 0.f ? c.softmax_scale : 1.0f / sqrtf((float)c.head_dim);
  ap.status = ctx->dev<int32_t>(ctx->lay.status);
  ap.dbg_ts = ctx->dev<unsigned long long>(ctx->lay.dbg);
  ap.timeline = ctx->opt_timeline ? 1 : 0;
  ap.force_external_merge = ctx->opt_external ? 1 : 0;
  ap.max_depth = c.max_depth;
  ap.coop_merge = ctx->opt_coop ? 0 : -1;
  ap.spin_limit = (int32_t)ctx->opt_spin;

  // bit 0 ancestor sets, 1 attention, 2 argmax, 3 acceptance; the option is a measurement aid, the
  // mask is what the entry point asks for (cb_tree_attention_device: the first two)
  const int64_t stages = ctx->opt_stages & stage_mask;
  const bool use_mfma = plan.impl == 2;
  // The logits scan does not depend on the attention, and the MFMA attention builds the ancestor sets
  // it needs itself, so with option "parallel_scan" the scan runs beside it on the context's second
  // stream (fork/join with events; stream capture turns them into parallel graph branches).  Measured
  // on the 7B shape the cross-stream edges cost more than the 5 us scan they hide, so it is off by
  // default.  The scalar attention reads the sets from the workspace: there the scan goes first and
  // carries the blocks that build them.
  LogitsWork lw{};
  lw.logits = logits;
  lw.V = c.vocab_size;
  lw.rows = total;
  lw.batch = batch;
  lw.chunks = ctx->lay.amax_chunks;
  lw.n_wgs = n_logits;
  lw.is_f32 = c.logits_dtype == CB_F32;
  lw.accept_after = (stages & 8) != 0;
  lw.tickets = ctx->dev<uint32_t>(ctx->lay.amax_tickets);
  AcceptArgs& acc = lw.accept;
  acc.parent = d_parent;
  acc.tokens = d_tokens;
  acc.status = ctx->dev<int32_t>(ctx->lay.status);
  acc.best = ctx->dev<unsigned long long>(ctx->lay.amax_best);
  acc.max_depth = c.max_depth;
  acc.argmax_out = ctx->dev<int32_t>(ctx->lay.amax_out);
  acc.path = ctx->dev<int32_t>(ctx->lay.path);
  acc.len_ctx = ctx->dev<int32_t>(ctx->lay.len_ctx);
  acc.len_user = d_len;
  acc.tok_user = d_tok;
  acc.last_user = ctx->want_last;
  ctx->want_last = nullptr;
  acc.done_flag = ctx->want_done;
  acc.done_value = ctx->call_seq;
  ctx->want_done = nullptr;
  // Otherwise, and with option "fuse_logits" = 0, the logits work is a launch of its own in front.
  const bool fused = ctx->opt_fuse != 0 && (stages & 2) && (stages & 4) && (stages & 8) &&
                     (f32_tiles || use_mfma) && n_logits > 0;
  const bool fork = !fused && ctx->opt_fork != 0 && (use_mfma || f32_tiles) && (stages & 2) && (stages & 4);
  hipStream_t scan_stream = st;
  int merge_kind = plan.nsplit > 1 ? 3 : 0, kernels = 0;  // (the scalar attention always merges with a kernel of its own)
  if (fork) {
    CB_HIP(ctx, hipEventRecord(ctx->ev_fork, st));
    CB_HIP(ctx, hipStreamWaitEvent(ctx->aux, ctx->ev_fork, 0));
    scan_stream = ctx->aux;
  }
  if (fused) {
  } else if (stages & 4) {
    const bool carry = !use_mfma && !f32_tiles && (stages & 1);
    CB_LAUNCH(ctx, launch_logits(scan_stream, lw, meta, carry ? d_parent : nullptr, c.max_depth,
                                 carry ? ctx->dev<uint32_t>(ctx->lay.anc) : nullptr, carry ? ctx->dev<int32_t>(ctx->lay.status) : nullptr));
    if (!lw.accept_after) ctx->amax_dirty = true;
    kernels++;
  } else if (!use_mfma && !f32_tiles && (stages & 1)) {
    CB_LAUNCH(ctx, launch_tree_prepare(st, batch, meta, d_parent, c.max_depth, ctx->dev<uint32_t>(ctx->lay.anc),
                                    ctx->dev<int32_t>(ctx->lay.status)));
    kernels++;
  }
  if (fork) CB_HIP(ctx, hipEventRecord(ctx->ev_join, ctx->aux));
  const bool timing = ctx->opt_time != 0;
  // The compaction in the attention's launch, for the matrix-core kernels as they are by default.
  // Not in many rounds of workgroups, each of which its arrivals make about a microsecond longer (31 sequences of one node x 55 keys, 32
  // heads: 22.9 us in two launches, 26.1 in one; 18 of 53 x 36, 40 heads, 41.5 and 40.0).  (In fp32, 2048 workgroups of 20 nodes x 1000 keys, 16/8
  // heads, 194.2 in one launch and 199.8 in two: no such line.)
  // Nor, in bf16 with head_dim 64, where a logits workgroup accepts more than two sequences on average: what follows an acceptance is a chain of round
  // trips, which the sequences beyond take one after the other, and those sweeps are through before.  Steps in one launch and in two, 8
  // heads, vocabulary 1000 (8 logits workgroups): 16 sequences of 20 nodes x 1000 keys 19.4 and 19.6 us, 32 33.8 and 32.7, 64 66.2 and 61.6; with
  // head_dim 128 19.1 and 20.2, 34.3 and 35.9, 69.3 and 69.0; fp32 with head_dim 64 23.3 and 27.0, 40.7 and 44.4, 74.4 and 78.7.
  const bool few_to_a_workgroup = !fused || batch <= 2 * n_logits || !use_mfma || c.head_dim != 64;
  ctx->moved = ctx->want_move && stages == 15 && (f32_tiles || (use_mfma && ap.live_wgs <= 3 * 256)) && few_to_a_workgroup &&
               !timing && !fork && !ap.timeline;
  ctx->want_move = false;
  if (ctx->moved) ap.move = MoveArgs{ctx->dev<uint32_t>(ctx->lay.moves), acc.path, acc.len_ctx, fused ? 1 : 0};
  if (timing) CB_HIP(ctx, hipEventRecord(ctx->ev0, st));
  if (!(stages & 2)) {
  } else if (use_mfma) {
    CB_LAUNCH(ctx, launch_attn_mfma(st, ap, meta, plan.max_nodes, total, fused ? &lw : nullptr, model ? &model->table : nullptr, &merge_kind));  // merges its own splits
    kernels += merge_kind == 3 ? 2 : 1;
  } else if (f32_tiles) {
    const bool external = plan.nsplit > 1 && ap.force_external_merge;
    CB_LAUNCH(ctx, launch_attn_f32(st, ap, meta, plan.max_nodes, fused ? &lw : nullptr, model ? &model->table : nullptr));
    if (external) CB_LAUNCH(ctx, launch_merge(st, ap, meta, c.qkv_dtype, total));
    merge_kind = plan.nsplit > 1 ? (external ? 3 : 2) : 0;
    kernels += external ? 2 : 1;
  } else {
    CB_LAUNCH(ctx, launch_attn_simt(st, ap, meta, c.qkv_dtype, plan.max_nodes));
    if (plan.nsplit > 1) CB_LAUNCH(ctx, launch_merge(st, ap, meta, c.qkv_dtype, total));
    kernels += plan.nsplit > 1 ? 2 : 1;
  }
  if (timing) {
    CB_HIP(ctx, hipEventRecord(ctx->ev1, st));
    ctx->ev_valid = true;
  }
  if (fork) CB_HIP(ctx, hipStreamWaitEvent(st, ctx->ev_join, 0));
  if ((stages & 8) && !(stages & 4)) {
    CB_LAUNCH(ctx, launch_accept(st, batch, meta, acc));
    kernels++;
  }
  if (!(stage_mask & 8)) return CB_OK;  // attention alone leaves the state of the last verification as it is
  ctx->step_info[3] = use_mfma ? plan.tile_rows : 0;
  ctx->launch_info[0] = use_mfma ? 2 : 1;
  ctx->launch_info[1] = plan.nsplit;
  ctx->launch_info[2] = plan.chunk;
  ctx->launch_info[3] = fused ? 1 : 0;
  ctx->launch_info[4] = merge_kind;
  ctx->launch_info[5] = kernels;
  ctx->meta = meta;
  ctx->batch = batch;
  ctx->total_nodes = total;
  ctx->last_stream = st;
  ctx->have_verify = true;
  ctx->host_knows_len = false;
  return CB_OK;
}

// Shapes are host data in the device-resident forms too: everything except the tree's contents is checked.
int check_device_shapes(cb_ctx* ctx, int32_t batch, const cb_kv_layer* kv, const int32_t* kv_len, const int32_t* node_offsets) {
  const cb_config& c = ctx->cfg;
  if (!kv->k || !kv->v || kv->capacity_or_num_blocks < 1) return set_err(ctx, CB_EINVAL, "bad cache descriptor");
  if (c.block_size > 0 && (!kv->block_table || kv->max_blocks_per_seq < 1)) return set_err(ctx, CB_EINVAL, "paged cache without a block table");
  if (node_offsets[0] != 0) return set_err(ctx, CB_EINVAL, "node_offsets[0] must be 0");
  for (int b = 0; b < batch; b++) {
    const int64_t n = (int64_t)node_offsets[b + 1] - node_offsets[b];
    if (n < 1) return set_err(ctx, CB_EINVAL, "sequence %d has no root node", b);
    if (n > c.max_nodes) return set_err(ctx, CB_ECAP, "sequence %d has %lld nodes, max_nodes is %d", b, (long long)n, c.max_nodes);
    if (kv_len[b] < 0) return set_err(ctx, CB_EINVAL, "negative kv_len[%d]", b);
    const int64_t room = c.block_size > 0 ? (int64_t)kv->max_blocks_per_seq * c.block_size : kv->capacity_or_num_blocks;
    if (kv_len[b] + n > room || kv_len[b] + n > (1ll << 30)) return set_err(ctx, CB_ECAP, "sequence %d does not fit the cache", b);
  }
  return CB_OK;
}

// Whether the layers of a step can be launched together: everything about them valid (otherwise the calls one by one report what is
// not), one geometry and block table for all, options as they are by default, and no layer's results in the memory that another one, or
// the acceptance, reads or writes.
bool layers_together(cb_ctx* ctx, int batch, int n, const void* const* q, const cb_kv_layer* layers, const int32_t* kv_len, const int32_t* node_offsets,
                     const int32_t* d_parent, const int32_t* d_tokens, const void* logits, void* const* attn_out, const int32_t* d_len, const int32_t* d_tok) {
  const cb_config& c = ctx->cfg;
  if (ctx->opt_splits > 0 || ctx->opt_impl || ctx->opt_time || ctx->opt_stages != 15 || ctx->opt_timeline || ctx->opt_external || ctx->opt_fork ||
      !ctx->opt_fuse || !ctx->opt_coop || ctx->opt_logits_wgs > 0 || ctx->opt_tile_rows)
    return false;
  if (!kv_len || !node_offsets || !d_parent || !d_tokens || !logits || !d_len || !d_tok || batch < 1 || batch > c.max_batch || ((uintptr_t)logits & 15)) return false;
  const cb_kv_layer& first = layers[0];
  for (int i = 0; i < n; i++) {
    const cb_kv_layer& l = layers[i];
    if (!q[i] || !attn_out[i] || !l.k || !l.v || (((uintptr_t)q[i] | (uintptr_t)attn_out[i] | (uintptr_t)l.k | (uintptr_t)l.v) & 15)) return false;
    if (l.capacity_or_num_blocks != first.capacity_or_num_blocks || l.block_table != first.block_table || l.max_blocks_per_seq != first.max_blocks_per_seq || l.layout != first.layout) return false;
  }
  const int valid = check_device_shapes(ctx, batch, &first, kv_len, node_offsets);
  ctx->err[0] = 0;
  if (valid || (first.layout != CB_LAYOUT_TOKEN_MAJOR && first.layout != CB_LAYOUT_HEAD_MAJOR)) return false;
  struct Use {
    Span s;
    bool written;
  };
  std::vector<Use> uses;
  const size_t rows = node_offsets[batch], qo = rows * c.num_q_heads * c.head_dim * (c.qkv_dtype == CB_F32 ? 4 : 2), cache = cache_bytes(c, first, batch);
  try {
    uses.reserve((size_t)n * 4 + 6);
    for (int i = 0; i < n; i++) {
      uses.push_back({{q[i], qo}, false});
      uses.push_back({{layers[i].k, cache}, false});
      uses.push_back({{layers[i].v, cache}, false});
      uses.push_back({{attn_out[i], qo}, true});
    }
    uses.push_back({{logits, rows * c.vocab_size * (c.logits_dtype == CB_F32 ? 4 : 2)}, false});
    uses.push_back({{d_parent, rows * 4}, false});
    uses.push_back({{d_tokens, rows * 4}, false});
    uses.push_back({{first.block_table, c.block_size > 0 ? (size_t)batch * first.max_blocks_per_seq * 4 : 0}, false});
    uses.push_back({{d_len, (size_t)batch * 4}, true});
    uses.push_back({{d_tok, (size_t)batch * (c.max_depth + 1) * 4}, true});
  } catch (const std::bad_alloc&) {
    return false;
  }
  // In the order of their starts, a stretch that meets an earlier one starts before the furthest end of those.
  std::sort(uses.begin(), uses.end(), [](const Use& a, const Use& b) { return (uintptr_t)a.s.at < (uintptr_t)b.s.at; });
  uintptr_t any = 0, written = 0;
  for (const Use& u : uses) {
    if (u.s.bytes == 0) continue;
    const uintptr_t at = (uintptr_t)u.s.at, end = at + std::min<uintptr_t>(u.s.bytes, UINTPTR_MAX - at);
    if (at < (u.written ? any : written)) return false;
    any = std::max(any, end);
    if (u.written) written = std::max(written, end);
  }
  return true;
}

}  // namespace

extern "C" {

int cb_workspace_bytes(const cb_config* cfg, size_t* bytes) {
  if (!bytes) return set_err(nullptr, CB_EINVAL, "null bytes");
  if (!config_ok(cfg, g_init_err, sizeof g_init_err)) return CB_EINVAL;
  *bytes = ws_layout(*cfg).total;
  return CB_OK;
}

int cb_plan_attention(const cb_config* cfg, int32_t batch, const int32_t* kv_len, const int32_t* node_offsets,
                      int32_t forced_splits, int32_t plan[5]) {
  if (!config_ok(cfg, nullptr, 0) || !kv_len || !node_offsets || !plan) return CB_EINVAL;
  if (batch < 1 || batch > cfg->max_batch || node_offsets[0] != 0) return CB_EINVAL;
  for (int b = 0; b < batch; b++) {
    const int64_t n = (int64_t)node_offsets[b + 1] - node_offsets[b];
    if (n < 1 || n > cfg->max_nodes || kv_len[b] < 0 || (int64_t)kv_len[b] + n > (1ll << 30)) return CB_EINVAL;
  }
  const WsLayout lay = ws_layout(*cfg);
  const Plan p = plan_call(*cfg, lay.max_splits, lay.scalar_splits, 0, forced_splits, 0, kTallest, batch, kv_len, node_offsets, false);
  const int g = cfg->num_q_heads / cfg->num_kv_heads;
  const int tile = p.impl == 2 ? attn_mfma_tile_rows(p.max_nodes * g) : 1;
  int64_t wgs = 0;
  for (int b = 0; b < batch; b++) {
    const int n = node_offsets[b + 1] - node_offsets[b];
    const int64_t units = p.impl == 2 ? (int64_t)((n * g + tile - 1) / tile) * cfg->num_kv_heads : (int64_t)n * cfg->num_q_heads;
    wgs += units * ((kv_len[b] + n + p.chunk - 1) / p.chunk);
  }
  plan[0] = p.impl;
  plan[1] = p.nsplit;
  plan[2] = p.chunk;
  plan[3] = tile;
  plan[4] = (int32_t)std::min<int64_t>(wgs, INT32_MAX);
  return CB_OK;
}

// (declared in cb_internal.h: tests of the planning alone)
int cb_debug_plan(const cb_config* cfg, int32_t batch, const int32_t* kv_len, const int32_t* node_offsets, int32_t verification, int32_t plan[6]) {
  int32_t base[5];
  if (const int rc = cb_plan_attention(cfg, batch, kv_len, node_offsets, 0, base)) return rc;
  const WsLayout lay = ws_layout(*cfg);
  const Plan p = plan_call(*cfg, lay.max_splits, lay.scalar_splits, 0, 0, 0, kTallest, batch, kv_len, node_offsets, verification != 0);
  plan[0] = p.impl;
  plan[1] = p.nsplit;
  plan[2] = p.chunk;
  plan[3] = p.precise;
  plan[4] = p.logits_wgs;
  plan[5] = p.impl == 2 || cfg->qkv_dtype == CB_F32 ? p.logits_wgs > 0 : 0;
  return CB_OK;
}

int cb_debug_tiles(const cb_config* cfg, int32_t batch, const int32_t* kv_len, const int32_t* node_offsets, int32_t verification, int32_t plan[6]) {
  int32_t base[5];
  if (const int rc = cb_plan_attention(cfg, batch, kv_len, node_offsets, 0, base)) return rc;
  const WsLayout lay = ws_layout(*cfg);
  const Plan p = plan_call(*cfg, lay.max_splits, lay.scalar_splits, 0, 0, 0, 0, batch, kv_len, node_offsets, verification != 0);
  int64_t jobs = 0;
  if (p.impl == 2) jobs = Planner(*cfg, lay.max_splits, lay.scalar_splits, 0, 0, batch, kv_len, node_offsets, p.tile_rows).split_into(p.nsplit).jobs;
  const int32_t out[] = {p.impl == 2 ? p.tile_rows : 0, p.nsplit, p.chunk, p.precise, p.logits_wgs, (int32_t)jobs};
  memcpy(plan, out, sizeof out);
  return CB_OK;
}

int cb_debug_layers(const cb_config* cfg, int32_t layers, int32_t batch, const int32_t* kv_len, const int32_t* node_offsets, int32_t plan[6]) {
  int32_t base[5];
  if (const int rc = cb_plan_attention(cfg, batch, kv_len, node_offsets, 0, base)) return rc;
  if (layers < 2 || layers > kTableLayers) return CB_EINVAL;
  ModelLaunch m;
  memset(plan, 0, 6 * sizeof *plan);
  if (!plan_layers(*cfg, ws_layout(*cfg), layers, batch, kv_len, node_offsets, &m)) return CB_OK;
  const Plan& p = m.plan;
  const int32_t out[] = {1, p.impl == 2 ? p.tile_rows : 0, p.nsplit, p.chunk, p.precise, p.logits_wgs};
  memcpy(plan, out, sizeof out);
  return CB_OK;
}

int64_t cb_debug_pool_blocks(const cb_config* cfg, const cb_kv_layer* layer) {
  KvAddr a{};
  return make_kv_addr(*cfg, *layer, &a) ? a.num_blocks : -1;
}

int cb_check_verify_args(const cb_config* cfg, int32_t batch, const cb_kv_layer* kv, const int32_t* kv_len,
                         const int32_t* node_offsets, const int32_t* tree_parent, char* err, size_t err_len) {
  auto fail = [&](int code, const char* fmt, ...) __attribute__((format(printf, 3, 4))) {
    if (err && err_len) {
      va_list ap;
      va_start(ap, fmt);
      vsnprintf(err, err_len, fmt, ap);
      va_end(ap);
    }
    return code;
  };
  if (!config_ok(cfg, err, err_len)) return CB_EINVAL;
  if (!kv || !kv_len || !node_offsets || !tree_parent) return fail(CB_EINVAL, "null argument");
  if (batch < 1 || batch > cfg->max_batch) return fail(CB_EINVAL, "batch %d outside [1, %d]", batch, cfg->max_batch);
  if (!kv->k || !kv->v) return fail(CB_EINVAL, "null cache pointer");
  if (kv->layout != CB_LAYOUT_TOKEN_MAJOR && kv->layout != CB_LAYOUT_HEAD_MAJOR)
    return fail(CB_EINVAL, "unknown cache layout %d", kv->layout);
  if (kv->capacity_or_num_blocks < 1) return fail(CB_EINVAL, "empty cache");
  if (cfg->block_size > 0 && (!kv->block_table || kv->max_blocks_per_seq < 1))
    return fail(CB_EINVAL, "paged cache without a block table");
  if (cfg->block_size == 0 && kv->block_table) return fail(CB_EINVAL, "block table given for a contiguous cache");
  if (node_offsets[0] != 0) return fail(CB_EINVAL, "node_offsets[0] must be 0");
  for (int b = 0; b < batch; b++) {
    const int64_t n = (int64_t)node_offsets[b + 1] - node_offsets[b];
    if (n < 1) return fail(CB_EINVAL, "sequence %d has no root node", b);
    if (n > cfg->max_nodes) return fail(CB_ECAP, "sequence %d has %lld nodes, max_nodes is %d", b, (long long)n, cfg->max_nodes);
    if (kv_len[b] < 0) return fail(CB_EINVAL, "negative kv_len[%d]", b);
    const int64_t need = (int64_t)kv_len[b] + n;
    const int64_t room = cfg->block_size > 0 ? (int64_t)kv->max_blocks_per_seq * cfg->block_size : kv->capacity_or_num_blocks;
    if (need > room || need > (1ll << 30))
      return fail(CB_ECAP, "sequence %d needs %lld cache slots, %lld available", b, (long long)need, (long long)room);
    const int32_t* par = tree_parent + node_offsets[b];
    if (par[0] != -1) return fail(CB_ETREE, "sequence %d: root parent is %d, not -1", b, par[0]);
    int depth[CB_MAX_NODES];
    depth[0] = 0;
    for (int i = 1; i < n; i++) {
      if (par[i] < 0 || par[i] >= i) return fail(CB_ETREE, "sequence %d: parent[%d] = %d not in [0, %d)", b, i, par[i], i);
      depth[i] = depth[par[i]] + 1;
      if (depth[i] > cfg->max_depth) return fail(CB_ETREE, "sequence %d: node %d at depth %d > max_depth %d", b, i, depth[i], cfg->max_depth);
    }
  }
  return CB_OK;
}

int cb_init(const cb_config* cfg, void* workspace, size_t workspace_bytes, cb_ctx** out) {
  g_init_err[0] = 0;
  if (!out) return set_err(nullptr, CB_EINVAL, "null out");
  *out = nullptr;
  if (!config_ok(cfg, g_init_err, sizeof g_init_err)) return CB_EINVAL;
  const WsLayout lay = ws_layout(*cfg);
  if (!workspace || ((uintptr_t)workspace & (kAlign - 1))) return set_err(nullptr, CB_EINVAL, "workspace null or not 256-byte aligned");
  if (workspace_bytes < lay.total) return set_err(nullptr, CB_ECAP, "workspace of %zu bytes, %zu needed", workspace_bytes, lay.total);
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || ndev < 1) return set_err(nullptr, CB_EHIP, "no HIP device");
  cb_ctx* ctx = new (std::nothrow) cb_ctx();
  if (!ctx) return set_err(nullptr, CB_EHIP, "out of host memory");
  ctx->cfg = *cfg;
  ctx->lay = lay;
  ctx->ws = static_cast<char*>(workspace);
  ctx->opt_stages = 15;
  ctx->opt_fuse = 1;
  ctx->opt_coop = 1;
  ctx->opt_spin = 256;
  const size_t mt = lay.max_total_nodes, stride = (size_t)cfg->max_depth + 1;
  // (two tree areas: a host-form call may return while its kernels still run, and the next call
  // must not overwrite the tree they read)
  const size_t ints = mt * 5 + cfg->max_batch * (1 + 2 * stride) + 1 + 3 * (size_t)cfg->max_batch;
  hipError_t e = hipHostMalloc(&ctx->h_block, ints * 4, hipHostMallocDefault);
  if (e != hipSuccess) {
    delete ctx;
    return set_err(nullptr, CB_EHIP, "hipHostMalloc: %s", hipGetErrorString(e));
  }
  void* dptr = nullptr;
  e = hipHostGetDevicePointer(&dptr, ctx->h_block, 0);
  if (e != hipSuccess) {
    (void)hipHostFree(ctx->h_block);
    delete ctx;
    return set_err(nullptr, CB_EHIP, "hipHostGetDevicePointer: %s", hipGetErrorString(e));
  }
  ctx->d_hblock = static_cast<int32_t*>(dptr);
  int32_t* h = static_cast<int32_t*>(ctx->h_block);
  ctx->h_parent = h; h += mt;
  ctx->h_tokens = h; h += mt;
  h += 2 * mt;                       // (the second tree area, see cb_verify_tree)
  ctx->h_argmax = h; h += mt;
  ctx->h_len = h; h += cfg->max_batch;
  ctx->h_tok = h; h += cfg->max_batch * stride;
  ctx->h_path = h; h += cfg->max_batch * stride;
  ctx->h_misc = h; h += 1 + cfg->max_batch;
  ctx->h_last = h; h += cfg->max_batch;
  ctx->h_done = h;
  memset(ctx->h_done, 0, (size_t)cfg->max_batch * 4);
  e = hipEventCreate(&ctx->ev0);
  if (e == hipSuccess) e = hipEventCreate(&ctx->ev1);
  if (e == hipSuccess) e = hipEventCreateWithFlags(&ctx->ev_fork, hipEventDisableTiming);
  if (e == hipSuccess) e = hipEventCreateWithFlags(&ctx->ev_join, hipEventDisableTiming);
  if (e == hipSuccess) e = hipStreamCreateWithFlags(&ctx->aux, hipStreamNonBlocking);
  if (e == hipSuccess) e = hipMemset(ctx->ws + lay.status, 0, lay.dbg - lay.status);
  if (e == hipSuccess) e = hipDeviceSynchronize();
  if (e != hipSuccess) {
    (void)hipHostFree(ctx->h_block);
    delete ctx;
    return set_err(nullptr, CB_EHIP, "context set-up: %s", hipGetErrorString(e));
  }
  *out = ctx;
  return CB_OK;
}

int cb_verify_tree_device(cb_ctx* ctx, void* hip_stream, int32_t batch, const void* q, const cb_kv_layer* kv,
                          const int32_t* kv_len, const int32_t* node_offsets, const int32_t* d_tree_parent,
                          const int32_t* d_draft_tokens, const void* logits, void* attn_out,
                          int32_t* d_accepted_len, int32_t* d_accepted_tokens) {
  int rc = check_common(ctx, batch, q, kv, kv_len, node_offsets, logits, attn_out);
  if (rc) return rc;
  ctx->err[0] = 0;
  if (!d_tree_parent || !d_draft_tokens || !d_accepted_len || !d_accepted_tokens)
    return set_err(ctx, CB_EINVAL, "null argument");
  rc = check_device_shapes(ctx, batch, kv, kv_len, node_offsets);
  if (rc) return rc;
  return run_pipeline(ctx, static_cast<hipStream_t>(hip_stream), batch, q, kv, kv_len, node_offsets, d_tree_parent,
                      d_draft_tokens, logits, attn_out, d_accepted_len, d_accepted_tokens);
}

int cb_verify_and_compact_device(cb_ctx* ctx, void* hip_stream, int32_t batch, const void* q, const cb_kv_layer* kv,
                                 const int32_t* kv_len, const int32_t* node_offsets, const int32_t* d_tree_parent,
                                 const int32_t* d_draft_tokens, const void* logits, void* attn_out,
                                 int32_t* d_accepted_len, int32_t* d_accepted_tokens, int32_t num_layers, const cb_kv_layer* layers) {
  // One launch where the cache that is verified is the one that is compacted and its memory is nobody else's: the launch moves rows
  // while other workgroups still read their own inputs and write their results.  (Nor another sequence's: the tables of a paged batch may share
  // blocks, with one sequence's tree in what another attends to -- a row that is there twice to fill a captured batch up, say.)
  bool apart = false;
  if (ctx && kv && num_layers == 1 && (ctx->cfg.block_size == 0 || batch == 1) && layers && batch >= 1 && batch <= ctx->cfg.max_batch && node_offsets && same_cache(*kv, layers[0]) && ((((uintptr_t)kv->k | (uintptr_t)kv->v) & 15) == 0)) {
    const cb_config& c = ctx->cfg;
    const size_t rows = node_offsets[batch] > 0 ? node_offsets[batch] : 0, qo = rows * c.num_q_heads * c.head_dim * (c.qkv_dtype == CB_F32 ? 4 : 2);
    const size_t cache = cache_bytes(c, *kv, batch);
    const Span mine[] = {{kv->k, cache}, {kv->v, cache}};
    const Span others[] = {{kv->k, cache}, {q, qo}, {attn_out, qo}, {logits, rows * c.vocab_size * (c.logits_dtype == CB_F32 ? 4 : 2)},
                           {d_tree_parent, rows * 4}, {d_draft_tokens, rows * 4}, {d_accepted_len, (size_t)batch * 4},
                           {d_accepted_tokens, (size_t)batch * (c.max_depth + 1) * 4}, {kv->block_table, c.block_size > 0 ? (size_t)batch * kv->max_blocks_per_seq * 4 : 0}};
    apart = !mine[1].meets(others[0]);
    for (size_t i = 1; apart && i < sizeof others / sizeof *others; i++) apart = !mine[0].meets(others[i]) && !mine[1].meets(others[i]);
  }
  if (ctx) ctx->want_move = apart && node_offsets[batch] > batch;
  if (ctx) ctx->moved = false;
  const int rc = cb_verify_tree_device(ctx, hip_stream, batch, q, kv, kv_len, node_offsets, d_tree_parent, d_draft_tokens, logits, attn_out,
                                       d_accepted_len, d_accepted_tokens);
  if (ctx) ctx->want_move = false;
  if (rc) return rc;
  ctx->step_info[0] = ctx->moved;
  ctx->step_info[1] = ctx->step_info[2] = 0;
  if (ctx->moved || num_layers == 0) return rc;
  return cb_compact_kv(ctx, hip_stream, num_layers, layers, nullptr);
}

int cb_model_step_device(cb_ctx* ctx, void* hip_stream, int32_t batch, int32_t num_layers, const void* const* q, const cb_kv_layer* layers,
                         const int32_t* kv_len, const int32_t* node_offsets, const int32_t* d_tree_parent, const int32_t* d_draft_tokens,
                         const void* logits, void* const* attn_out, int32_t* d_accepted_len, int32_t* d_accepted_tokens) {
  if (!ctx) return set_err(nullptr, CB_EINVAL, "null context");
  ctx->err[0] = 0;
  if (num_layers < 1 || !q || !layers || !attn_out) return set_err(ctx, CB_EINVAL, "null argument");
  if (num_layers == 1)
    return cb_verify_and_compact_device(ctx, hip_stream, batch, q[0], layers, kv_len, node_offsets, d_tree_parent, d_draft_tokens, logits, attn_out[0],
                                        d_accepted_len, d_accepted_tokens, 1, layers);
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  int done = 0;
  ctx->step_info[0] = ctx->step_info[1] = ctx->step_info[2] = 0;
  if (layers_together(ctx, batch, num_layers, q, layers, kv_len, node_offsets, d_tree_parent, d_draft_tokens, logits, attn_out, d_accepted_len, d_accepted_tokens)) {
    // (as few launches as the table allows, of about as many layers each)
    const int launches = (num_layers + kTableLayers - 1) / kTableLayers;
    ModelLaunch m;
    for (int i = 0; i < launches; i++) {
      const int n = num_layers * (i + 1) / launches - done, mask = i + 1 < launches ? 3 : 15;
      m.table.count = n;
      if ((i == 0 || n != num_layers / launches) && !plan_layers(ctx->cfg, ctx->lay, n, batch, kv_len, node_offsets, &m)) break;
      for (int j = 0; j < n; j++) {
        const int l = done + j;
        m.table.at[j].q = q[l];
        m.table.at[j].out = attn_out[l];
        m.table.at[j].k = layers[l].k;
        m.table.at[j].v = layers[l].v;
      }
      const int rc = run_pipeline(ctx, st, batch, q[done], &layers[done], kv_len, node_offsets, d_tree_parent, d_draft_tokens, logits, attn_out[done],
                                  d_accepted_len, d_accepted_tokens, mask, &m);
      if (rc) return rc;
      done += n;
      ctx->step_info[1] = done;
      ctx->step_info[2]++;
    }
  }
  for (; done < num_layers; done++) {
    const int rc = done + 1 < num_layers
                       ? cb_tree_attention_device(ctx, hip_stream, batch, q[done], &layers[done], kv_len, node_offsets, d_tree_parent, attn_out[done])
                       : cb_verify_tree_device(ctx, hip_stream, batch, q[done], &layers[done], kv_len, node_offsets, d_tree_parent, d_draft_tokens, logits,
                                               attn_out[done], d_accepted_len, d_accepted_tokens);
    if (rc) return rc;
  }
  return cb_compact_kv(ctx, hip_stream, num_layers, layers, nullptr);
}

int cb_tree_attention_device(cb_ctx* ctx, void* hip_stream, int32_t batch, const void* q, const cb_kv_layer* kv,
                             const int32_t* kv_len, const int32_t* node_offsets, const int32_t* d_tree_parent,
                             void* attn_out) {
  if (!ctx) return set_err(nullptr, CB_EINVAL, "null context");
  ctx->err[0] = 0;
  if (!q || !kv || !kv_len || !node_offsets || !d_tree_parent || !attn_out) return set_err(ctx, CB_EINVAL, "null argument");
  if (batch < 1 || batch > ctx->cfg.max_batch) return set_err(ctx, CB_EINVAL, "batch %d outside [1, %d]", batch, ctx->cfg.max_batch);
  if (((uintptr_t)q | (uintptr_t)kv->k | (uintptr_t)kv->v | (uintptr_t)attn_out) & 15)
    return set_err(ctx, CB_EINVAL, "device pointers must be 16-byte aligned");
  const int rc = check_device_shapes(ctx, batch, kv, kv_len, node_offsets);
  if (rc) return rc;
  return run_pipeline(ctx, static_cast<hipStream_t>(hip_stream), batch, q, kv, kv_len, node_offsets, d_tree_parent,
                      nullptr, nullptr, attn_out, nullptr, nullptr, 3);
}

int cb_tree_attention_noalloc(const cb_config* cfg, void* hip_stream, int32_t batch, const void* q, const cb_kv_layer* kv,
                              const int32_t* kv_len, const int32_t* node_offsets, const int32_t* d_tree_parent,
                              void* attn_out) {
  g_init_err[0] = 0;
  if (!config_ok(cfg, g_init_err, sizeof g_init_err)) return CB_EINVAL;
  if (!q || !kv || !kv_len || !node_offsets || !d_tree_parent || !attn_out) return set_err(nullptr, CB_EINVAL, "null argument");
  if (batch < 1 || batch > cfg->max_batch) return set_err(nullptr, CB_EINVAL, "batch %d outside [1, %d]", batch, cfg->max_batch);
  if (((uintptr_t)q | (uintptr_t)kv->k | (uintptr_t)kv->v | (uintptr_t)attn_out) & 15)
    return set_err(nullptr, CB_EINVAL, "device pointers must be 16-byte aligned");
  // A context on the stack, never handed out: configuration, options at their defaults, and a
  // workspace layout cut from the static array for exactly this call's shapes.
  cb_ctx tmp{};
  tmp.cfg = *cfg;
  tmp.opt_stages = 15;
  tmp.opt_coop = 1;
  tmp.opt_spin = 256;
  int rc = check_device_shapes(&tmp, batch, kv, kv_len, node_offsets);
  if (rc) {
    memcpy(g_init_err, tmp.err, sizeof g_init_err);
    return rc;
  }
  const WsLayout full = ws_layout(*cfg);
  Plan plan;
  const WsLayout L = noalloc_layout(*cfg, full, batch, kv_len, node_offsets, &plan);
  if (L.total > kStaticScratchBytes)
    return set_err(nullptr, CB_ECAP, "this call needs %zu bytes of scratch memory, the library's fixed buffer has %zu", L.total, kStaticScratchBytes);
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess || dev < 0 || dev >= kMaxDevices) return set_err(nullptr, CB_EHIP, "hipGetDevice: %s", hipGetErrorString(e));
  void* base = nullptr;
  {
    std::lock_guard<std::mutex> lock(g_static_mutex);
    if (!g_static_scratch_ptr[dev]) {
      void* ptr = nullptr;
      e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(g_static_scratch));
      if (e != hipSuccess || !ptr) return set_err(nullptr, CB_EHIP, "hipGetSymbolAddress: %s", hipGetErrorString(e));
      g_static_scratch_ptr[dev] = ptr;
    }
    base = g_static_scratch_ptr[dev];
  }
  tmp.lay = L;
  tmp.fixed_plan = &plan;
  tmp.ws = static_cast<char*>(base);
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  // The array is shared by every call on this GPU and keeps the last call's contents: the words that
  // must start at zero are cleared here, by a kernel (a caller may be capturing the stream).
  e = launch_zero_words(st, tmp.dev<unsigned long long>(L.status), 1, 1, 1);
  if (e == hipSuccess) e = launch_zero_words(st, tmp.dev<unsigned long long>(L.tickets), L.ticket_count / 2, 1, 1);
  if (e == hipSuccess) e = launch_zero_words(st, tmp.dev<unsigned long long>(L.coop_tickets), std::min(L.ticket_count / 4, kCoopTiles), kCoopTicketStride / 8, 2);
  if (e != hipSuccess) return set_err(nullptr, CB_EHIP, "clearing the scratch counters: %s", hipGetErrorString(e));
  rc = run_pipeline(&tmp, st, batch, q, kv, kv_len, node_offsets, d_tree_parent, nullptr, nullptr, attn_out, nullptr, nullptr, 3);
  if (rc) memcpy(g_init_err, tmp.err, sizeof g_init_err);
  return rc;
}

int cb_verify_tree(cb_ctx* ctx, void* hip_stream, int32_t batch, const void* q, const cb_kv_layer* kv,
                   const int32_t* kv_len, const int32_t* node_offsets, const int32_t* tree_parent,
                   const int32_t* draft_tokens, const void* logits, void* attn_out, int32_t* accepted_len,
                   int32_t* accepted_tokens) {
  int rc = check_common(ctx, batch, q, kv, kv_len, node_offsets, logits, attn_out);
  if (rc) return rc;
  ctx->err[0] = 0;
  if (!tree_parent || !draft_tokens || !accepted_len || !accepted_tokens) return set_err(ctx, CB_EINVAL, "null argument");
  rc = cb_check_verify_args(&ctx->cfg, batch, kv, kv_len, node_offsets, tree_parent, ctx->err, sizeof ctx->err);
  if (rc) return rc;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  const int total = node_offsets[batch];
  const size_t stride = (size_t)ctx->cfg.max_depth + 1;
  // No copies: the kernels read the tree from, and write the results to, the context's pinned host
  // block through its device address (a few hundred bytes each way; two staged copies cost more
  // than the kernels' reads across the bus).  Parents and tokens back to back, lengths and tokens
  // back to back.  Calls alternate between two tree areas: this call may return before its launch
  // has ended (below), and the launch of the call before it has ended by the time this one's
  // results arrive, because both run on one stream (order_behind_host_form synchronises when the stream changes).
  const bool early = ctx->opt_full_sync == 0 && (ctx->opt_stages & 8) != 0;
  ctx->call_seq = ctx->call_seq == INT32_MAX ? 1 : ctx->call_seq + 1;
  int32_t* h_tree = ctx->h_parent + (size_t)(ctx->call_seq & 1) * 2 * ctx->lay.max_total_nodes;
  memcpy(h_tree, tree_parent, (size_t)total * 4);
  memcpy(h_tree + total, draft_tokens, (size_t)total * 4);
  int32_t* d_parent = ctx->d_hblock + (h_tree - static_cast<int32_t*>(ctx->h_block));
  int32_t* d_tokens = d_parent + total;
  int32_t* h_res = ctx->h_len;
  int32_t* d_len = ctx->d_hblock + (h_res - static_cast<int32_t*>(ctx->h_block));
  int32_t* d_tok = d_len + batch;
  ctx->want_last = ctx->d_hblock + (ctx->h_last - static_cast<int32_t*>(ctx->h_block));
  if (early) ctx->want_done = ctx->d_hblock + (ctx->h_done - static_cast<int32_t*>(ctx->h_block));
  rc = run_pipeline(ctx, st, batch, q, kv, kv_len, node_offsets, d_parent, d_tokens, logits, attn_out, d_len, d_tok);
  ctx->want_done = ctx->want_last = nullptr;
  if (rc) return rc;
  if (early) {
    // The acceptance stores a sequence's results, makes them visible at system scope and then stores
    // the call's number into the sequence's flag word; the host returns as soon as every flag shows
    // it, without waiting for the attention (which may not have begun) and for the
    // stream's completion signal.  The stream's state is looked at now and then, so that a failed
    // launch ends the wait.
    const int32_t want = ctx->call_seq;
    bool seen = false;
    for (uint32_t polls = 1; !seen; polls++) {
      seen = true;
      for (int b = 0; b < batch; b++)
        if (__atomic_load_n(ctx->h_done + b, __ATOMIC_ACQUIRE) != want) { seen = false; break; }
      if (seen) break;
      if ((polls & 2047) == 0) {
        const hipError_t q_rc = hipStreamQuery(st);
        if (q_rc == hipSuccess) {  // everything has run: the flags are there now or never
          seen = true;
          for (int b = 0; b < batch; b++)
            if (__atomic_load_n(ctx->h_done + b, __ATOMIC_ACQUIRE) != want) seen = false;
          if (!seen) return set_err(ctx, CB_EHIP, "the verification ran but its results did not arrive");
        } else if (q_rc != hipErrorNotReady) {
          return set_err(ctx, CB_EHIP, "%s: %s", "hipStreamQuery", hipGetErrorString(q_rc));
        }
      }
      __builtin_ia32_pause();
    }
    ctx->unsynced = st;
    ctx->have_unsynced = true;
  } else {
    CB_HIP(ctx, hipStreamSynchronize(st));
  }
  memcpy(accepted_len, h_res, (size_t)batch * 4);
  memcpy(accepted_tokens, h_res + batch, (size_t)batch * stride * 4);
  memcpy(ctx->last_len, h_res, (size_t)batch * 4);
  ctx->host_knows_len = true;
  // (the nodes of a path are in increasing order, so one whose last node is its length's has each in its place)
  ctx->nothing_moves = (ctx->opt_stages & 8) != 0;
  for (int b = 0; b < batch; b++) ctx->nothing_moves = ctx->nothing_moves && ctx->h_last[b] == ctx->last_len[b];
  return CB_OK;
}

int cb_compact_kv(cb_ctx* ctx, void* hip_stream, int32_t num_layers, const cb_kv_layer* layers, int32_t* new_kv_len) {
  if (!ctx) return set_err(nullptr, CB_EINVAL, "null context");
  ctx->err[0] = 0;
  if (!ctx->have_verify) return set_err(ctx, CB_ESTATE, "cb_compact_kv needs a preceding successful verify call");
  if (!layers || num_layers < 1 || num_layers > CB_MAX_LAYERS) return set_err(ctx, CB_EINVAL, "num_layers outside [1, %d]", CB_MAX_LAYERS);
  const cb_config& c = ctx->cfg;
  KvAddr addrs[CB_MAX_LAYERS];
  for (int l = 0; l < num_layers; l++) {
    const cb_kv_layer& y = layers[l];
    if (!y.k || !y.v || (((uintptr_t)y.k | (uintptr_t)y.v) & 15)) return set_err(ctx, CB_EINVAL, "layer %d: null or misaligned cache pointer", l);
    if (y.capacity_or_num_blocks != layers[0].capacity_or_num_blocks || y.block_table != layers[0].block_table ||
        y.max_blocks_per_seq != layers[0].max_blocks_per_seq || y.layout != layers[0].layout)
      return set_err(ctx, CB_EINVAL, "layer %d does not share the geometry of layer 0", l);
    if (!make_kv_addr(c, y, &addrs[l])) return set_err(ctx, CB_EINVAL, "unknown cache layout %d", y.layout);
  }
  if (c.block_size > 0 && (!layers[0].block_table || layers[0].max_blocks_per_seq < 1)) return set_err(ctx, CB_EINVAL, "paged cache without a block table");
  for (int b = 0; b < ctx->batch; b++) {
    const int64_t n = ctx->meta.node_off[b + 1] - ctx->meta.node_off[b];
    const int64_t room = c.block_size > 0 ? (int64_t)layers[0].max_blocks_per_seq * c.block_size : layers[0].capacity_or_num_blocks;
    if (ctx->meta.kv_len[b] + n > room) return set_err(ctx, CB_ECAP, "sequence %d does not fit these caches", b);
  }
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  // (the attention of a host-form call that has returned may not even have begun to read the slots that move here)
  const int ordered = order_behind_host_form(ctx, st);
  if (ordered) return ordered;
  const int eb = c.qkv_dtype == CB_F32 ? 4 : 2;
  // No launch where nothing moves: trees of roots alone, and accepted paths that are the tree's first nodes, where the host knows them
  // (one in two or three steps of a decode loop; the launch costs its pass 4 us).
  const bool roots = ctx->total_nodes == ctx->batch;
  if (!roots && !(ctx->host_knows_len && ctx->nothing_moves))
    CB_HIP(ctx, launch_compact(st, ctx->batch, ctx->meta, addrs, num_layers, c.num_kv_heads, c.head_dim, eb, c.max_depth,
                             ctx->dev<int32_t>(ctx->lay.path), ctx->dev<int32_t>(ctx->lay.len_ctx),
                             ctx->dev<int32_t>(ctx->lay.new_len)));
  if (new_kv_len) {
    if (ctx->host_knows_len || roots) {
      if (!ctx->host_knows_len) CB_HIP(ctx, hipStreamSynchronize(st));
      for (int b = 0; b < ctx->batch; b++) new_kv_len[b] = ctx->meta.kv_len[b] + (roots ? 0 : ctx->last_len[b]) + 1;
    } else {
      CB_HIP(ctx, hipMemcpyAsync(ctx->h_misc + 1, ctx->dev<int32_t>(ctx->lay.new_len), (size_t)ctx->batch * 4, hipMemcpyDeviceToHost, st));
      CB_HIP(ctx, hipStreamSynchronize(st));
      memcpy(new_kv_len, ctx->h_misc + 1, (size_t)ctx->batch * 4);
    }
  }
  return CB_OK;
}

int cb_get_path(cb_ctx* ctx, int32_t* path) {
  if (!ctx || !path) return set_err(ctx, CB_EINVAL, "null argument");
  if (!ctx->have_verify) return set_err(ctx, CB_ESTATE, "no verify call yet");
  const size_t n = (size_t)ctx->batch * (ctx->cfg.max_depth + 1);
  CB_HIP(ctx, hipMemcpyAsync(ctx->h_path, ctx->dev<int32_t>(ctx->lay.path), n * 4, hipMemcpyDeviceToHost, ctx->last_stream));
  CB_HIP(ctx, hipStreamSynchronize(ctx->last_stream));
  memcpy(path, ctx->h_path, n * 4);
  return CB_OK;
}

int cb_get_argmax(cb_ctx* ctx, int32_t* argmax) {
  if (!ctx || !argmax) return set_err(ctx, CB_EINVAL, "null argument");
  if (!ctx->have_verify) return set_err(ctx, CB_ESTATE, "no verify call yet");
  const size_t n = (size_t)ctx->total_nodes;
  CB_HIP(ctx, hipMemcpyAsync(ctx->h_argmax, ctx->dev<int32_t>(ctx->lay.amax_out), n * 4, hipMemcpyDeviceToHost, ctx->last_stream));
  CB_HIP(ctx, hipStreamSynchronize(ctx->last_stream));
  memcpy(argmax, ctx->h_argmax, n * 4);
  return CB_OK;
}

int cb_device_status(cb_ctx* ctx, int32_t* status) {
  if (!ctx || !status) return set_err(ctx, CB_EINVAL, "null argument");
  hipStream_t st = ctx->have_verify ? ctx->last_stream : nullptr;
  CB_HIP(ctx, hipMemcpyAsync(ctx->h_misc, ctx->dev<int32_t>(ctx->lay.status), 4, hipMemcpyDeviceToHost, st));
  CB_HIP(ctx, hipStreamSynchronize(st));
  *status = ctx->h_misc[0];
  CB_HIP(ctx, hipMemsetAsync(ctx->dev<int32_t>(ctx->lay.status), 0, 4, st));  // reading clears the sticky word
  CB_HIP(ctx, hipStreamSynchronize(st));
  return CB_OK;
}

int cb_set_option(cb_ctx* ctx, const char* name, int64_t value) {
  if (!ctx || !name) return set_err(ctx, CB_EINVAL, "null argument");
  if (!strcmp(name, "splits")) ctx->opt_splits = value;
  else if (!strcmp(name, "attn_impl")) ctx->opt_impl = value;
  else if (!strcmp(name, "time_attention")) ctx->opt_time = value;
  else if (!strcmp(name, "stages")) ctx->opt_stages = value & 15;
  else if (!strcmp(name, "timeline")) ctx->opt_timeline = value;
  else if (!strcmp(name, "full_sync")) ctx->opt_full_sync = value;
  else if (!strcmp(name, "external_merge")) ctx->opt_external = value;
  else if (!strcmp(name, "parallel_scan")) ctx->opt_fork = value;
  else if (!strcmp(name, "fuse_logits")) ctx->opt_fuse = value;
  else if (!strcmp(name, "coop_merge")) ctx->opt_coop = value;
  else if (!strcmp(name, "tile_rows")) ctx->opt_tile_rows = value == 64 || value == 128 || value == 256 ? value : 0;
  else if (!strcmp(name, "logits_wgs")) ctx->opt_logits_wgs = value < 0 ? 0 : (value > 192 ? 192 : value / 8 * 8);
  else if (!strcmp(name, "merge_spin_limit")) ctx->opt_spin = value < 0 ? 0 : (value > 4096 ? 4096 : value);
  else return set_err(ctx, CB_EINVAL, "unknown option '%s'", name);
  return CB_OK;
}

int cb_last_launch_info(cb_ctx* ctx, int32_t info[6]) {
  if (!ctx || !info) return set_err(ctx, CB_EINVAL, "null argument");
  if (!ctx->have_verify) return set_err(ctx, CB_ESTATE, "no verify call yet");
  for (int i = 0; i < 6; i++) info[i] = ctx->launch_info[i];
  return CB_OK;
}

int cb_debug_step(cb_ctx* ctx, int32_t info[4]) {
  if (!ctx || !info) return set_err(ctx, CB_EINVAL, "null argument");
  for (int i = 0; i < 4; i++) info[i] = ctx->step_info[i];
  return CB_OK;
}

int cb_last_attention_ms(cb_ctx* ctx, float* ms) {
  if (!ctx || !ms) return set_err(ctx, CB_EINVAL, "null argument");
  if (!ctx->ev_valid) return set_err(ctx, CB_ESTATE, "option time_attention was not set for the last verify");
  CB_HIP(ctx, hipEventSynchronize(ctx->ev1));
  CB_HIP(ctx, hipEventElapsedTime(ms, ctx->ev0, ctx->ev1));
  return CB_OK;
}

int cb_debug_timestamps(cb_ctx* ctx, uint64_t* out, int32_t workgroups) {
  if (!ctx || !out || workgroups < 1 || workgroups > 1024) return set_err(ctx, CB_EINVAL, "bad argument");
  hipStream_t st = ctx->have_verify ? ctx->last_stream : nullptr;
  CB_HIP(ctx, hipStreamSynchronize(st));
  CB_HIP(ctx, hipMemcpy(out, ctx->ws + ctx->lay.dbg, (size_t)workgroups * 64, hipMemcpyDeviceToHost));
  return CB_OK;
}

const char* cb_last_error(const cb_ctx* ctx) { return ctx ? ctx->err : g_init_err; }

void cb_destroy(cb_ctx* ctx) {
  if (!ctx) return;
  if (ctx->have_unsynced) (void)hipStreamSynchronize(ctx->unsynced);  // its launch may still write the pinned block
  (void)hipEventDestroy(ctx->ev0);
  (void)hipEventDestroy(ctx->ev1);
  (void)hipEventDestroy(ctx->ev_fork);
  (void)hipEventDestroy(ctx->ev_join);
  (void)hipStreamDestroy(ctx->aux);
  (void)hipHostFree(ctx->h_block);
  delete ctx;
}

}  // extern "C"
