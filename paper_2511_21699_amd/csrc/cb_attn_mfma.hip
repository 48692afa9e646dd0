// Tree attention on the matrix cores (bf16, head_dim 64 or 128), gfx950 only: tiles of up to 64 rows, the stand-alone
// merge, and the launch of both kinds of tile.
//
// Small tile: 4 row groups of 16 rows times two key groups.  Wave group gi takes the units 2s + gi of 32 keys (short of
// rows, long on keys: each SIMD still holds two waves whose MFMA, LDS and vector phases overlap); the groups'
// softmax states are combined through LDS at the end.  What bounds it is memory: a stage's arithmetic (17 MFMAs of 16
// cycles per wave) is a fifth of the time its 32 KiB take to arrive.
//
// Register layouts (v_mfma_f32_16x16x32_bf16; lane l, c = l%16, kg = l/16):
//   scores are computed transposed, S^T = K Q^T: A = K rows (key c of the 16-key sub-tile, dims
//   8kg..8kg+7 of the 32-dim step), B = Q^T (query c, same dims), D[v] = S^T[key 4kg+v][query c].
//   A lane therefore holds 4 keys x 1 query per 16-key sub-tile: softmax statistics are per-lane
//   scalars shared by the 4 lanes with equal c.
//   O^T = V^T P^T: B = P^T packs the lane's 8 probabilities of a 32-key tile (element e <-> key
//   16(e/4)+4kg+e%4), A = V^T must hold the same keys for dim c of the 16-dim tile; it is fetched
//   from the row-major V tile with ds_read_b64_tr_b16 (each 16-lane group reads a 4-key x 16-dim
//   block and receives it transposed).  D[v] = O^T[dim 4kg+v][query c].
#include <algorithm>

#include "cb_attn_tile.h"

namespace cb {

constexpr int kSmallRows = 64;

template <int D>
struct RowState {
  bf16x8 q[D / 32];    // B operands of QK^T: query c, dims 32*ds + 8kg ..
  floatx4 o[D / 16];   // O^T accumulators, dim tiles of 16
  floatx4 lacc;        // softmax denominator, accumulated by an MFMA against a tile of ones
  float mref;          // reference maximum of the raw scores (q.k, before the softmax scale)
};

// Maximum over the 4 lanes that share a query (lanes c, c+16, c+32, c+48): v_permlane16_swap exchanges odd 16-lane rows
// of one operand with even rows of the other, v_permlane32_swap the upper half of one with the lower half of the
// other, so two swaps of a value with itself bring every lane its partners.
__device__ __forceinline__ float quad_max(float x) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = maxn(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return maxn(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// 32-bit visibility word of the unit at key0 for one query: bit j <-> key key0 + j.
__device__ __forceinline__ uint32_t visible_keys(int key0, int S, int kend, const uint32_t* arow) {
  const int np = S - key0;     // prefix keys in the unit (may be <= 0 or >= 32)
  const int ne = kend - key0;  // keys before the split's end (>= 1)
  uint32_t vis = np >= 32 ? 0xffffffffu : (np <= 0 ? 0u : ((1u << np) - 1u));
  if (np < 32) {
    uint32_t tree;
    if (np > 0) {
      tree = arow[0] << np;  // tree node 0 sits at bit np
    } else {
      const int t0 = -np, w0 = t0 >> 5, sh = t0 & 31;
      const uint32_t lo = w0 < kAncWords ? arow[w0] : 0u;
      const uint32_t hi = (w0 + 1 < kAncWords) ? arow[w0 + 1] : 0u;
      tree = sh ? ((lo >> sh) | (hi << (32 - sh))) : lo;
    }
    vis |= tree;
  }
  if (ne < 32) vis &= (1u << ne) - 1u;  // keys past the split's end belong to the next split (or do not exist)
  return vis;
}

// One unit for the 16 rows of a wave.
//   scores  S^T = K Q^T
//   p = 2^(c*s - c*mref) with c = scale*log2(e); mref follows the running maximum lazily: it is
//   only raised (and O, l rescaled) when the maximum has grown by more than kRescaleSlack, so
//   probabilities stay below 2^8 and the accumulators are rarely touched by the vector ALU
//   O^T += V^T P^T, l += 1^T P^T
// All K and V operands are requested before the first MFMA, so that LDS latency hides behind the matrix and vector work.
template <int D, bool PX>
__device__ __forceinline__ void compute_unit(const uint4* __restrict__ ks, const uint4* __restrict__ vs, RowState<D>& st, float c2,
                                             int key0, int S, int kend, const uint32_t* arow, int l) {
  constexpr int VPR = D / 8;
  const int c = l & 15, kg = l >> 4;
  uint4 kraw[2][D / 32];
#pragma unroll
  for (int sub = 0; sub < 2; sub++) {
    const int row = 16 * sub + c;
#pragma unroll
    for (int ds = 0; ds < D / 32; ds++) kraw[sub][ds] = ks[row * VPR + ((kg + 4 * ds) ^ swizzle_k<D>(row))];
  }
  const char* vbytes = reinterpret_cast<const char*>(vs);
  bf16x4 va[D / 16][2];
#pragma unroll
  for (int dt = 0; dt < D / 16; dt++)
#pragma unroll
    for (int t = 0; t < 2; t++) {
      const int row = 16 * t + 4 * kg + (c >> 2);
      const int piece = 2 * dt + ((c & 3) >> 1);
      const char* addr = vbytes + row * (2 * D) + (piece ^ swizzle_v<D, 16>(row)) * 16 + (c & 1) * 8;
      va[dt][t] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((bf16x4 __attribute__((address_space(3)))*)(addr));
    }
  floatx4 s[2] = {floatx4{0.f, 0.f, 0.f, 0.f}, floatx4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
  for (int ds = 0; ds < D / 32; ds++)
#pragma unroll
    for (int sub = 0; sub < 2; sub++)
      s[sub] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kraw[sub][ds]), st.q[ds], s[sub], 0, 0, 0);
  float x[8];
#pragma unroll
  for (int e = 0; e < 8; e++) x[e] = s[e >> 2][e & 3];
  if (key0 + kUnitKeys > S || key0 + kUnitKeys > kend) {
    const uint32_t vis = visible_keys(key0, S, kend, arow);
#pragma unroll
    for (int e = 0; e < 8; e++) {
      const int j = 16 * (e >> 2) + 4 * kg + (e & 3);
      x[e] = ((vis >> j) & 1u) ? x[e] : -INFINITY;
    }
  }
  const float mx = quad_max(maxn(maxn(maxn(x[0], x[1]), maxn(x[2], x[3])), maxn(maxn(x[4], x[5]), maxn(x[6], x[7]))));
  // lazy reference update; the decision is identical in the 4 lanes of a query
  const bool raise = (mx - st.mref) * c2 > kRescaleSlack;  // false when both are -inf (NaN)
  if (__builtin_amdgcn_ballot_w64(raise) != 0ull) {
    const float alpha = raise ? __builtin_amdgcn_exp2f((st.mref - mx) * c2) : 1.0f;
    if (raise) st.mref = mx;
#pragma unroll
    for (int dt = 0; dt < D / 16; dt++) st.o[dt] *= alpha;
    st.lacc *= alpha;
  }
  const float nm = (st.mref == -INFINITY) ? 0.f : -st.mref * c2;
  union { bf16x8 v; __bf16 h[8]; } pk, rest;
#pragma unroll
  for (int e = 0; e < 8; e++) {
    const float pe = __builtin_amdgcn_exp2f(fmaf(x[e], c2, nm));
    pk.h[e] = (__bf16)pe;
    if (PX) rest.h[e] = (__bf16)(pe - (float)pk.h[e]);
  }
  const bf16x8 ones = __builtin_bit_cast(bf16x8, uint4{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u});
  st.lacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pk.v, st.lacc, 0, 0, 0);
  if (PX) st.lacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, rest.v, st.lacc, 0, 0, 0);
#pragma unroll
  for (int dt = 0; dt < D / 16; dt++) {
    const bf16x8 v = __builtin_shufflevector(va[dt][0], va[dt][1], 0, 1, 2, 3, 4, 5, 6, 7);
    st.o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v, pk.v, st.o[dt], 0, 0, 0);
    if (PX) st.o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v, rest.v, st.o[dt], 0, 0, 0);
  }
}

// One attention workgroup; `wg` is its number among those that do attention.  MOVE: the launch compacts its cache.
template <int D, bool PX, bool LEAN, bool MOVE, bool TS, typename Layers>
__device__ __forceinline__ void attn_tile(const AttnParams& p_arg, const SeqMetaLanes& ml, int wg, unsigned long long ts0,
                                          TileLds& sh, uint4* ring, unsigned long long* ts_sh, const Layers& layers) {
  using F = Feed<D, 8, 16, LEAN>;
  constexpr int NS = F::kSlots, PRO = F::kPrologue, P = PartialLayout<D, 16, PX>::P;
  AttnParams p = p_arg;
  pin_args(p);
  CB_LDS unsigned long long* ts = (CB_LDS unsigned long long*)ts_sh;
  first_stamps<TS>(ts, ts0);
  TileJob jb;
  if (!tile_job(p, ml, wg, kSmallRows, layers, jb)) return;
  take_layer(p, jb, layers);
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
  const int gi = w >> 2, wi = w & 3;
  const int c = l & 15, kg = l >> 4;
  const bool do_ts = TS && tid == 0;
#define CB_TS(i) do { if (do_ts) ts[i] = wall_clock64(); } while (0)
  const int S = jb.S, k0 = jb.k0, k1 = jb.k1;
  F feed(p, jb, sh.bt, ring);
  // Everything this workgroup needs from memory is requested up front, oldest first: the query rows (to registers),
  // then K/V units (to LDS).
  RowState<D> st;
  const bool has_rows = jb.row0 + 16 * wi < jb.M;
  int row = jb.row0 + 16 * wi + c;
  const bool valid = row < jb.M;
  row = valid ? row : jb.M - 1;
  const int node = row / jb.g, hg = row - node * jb.g;
  const int64_t gr = (int64_t)(jb.off + node) * p.Hq + jb.hk * jb.g + hg;
  const int64_t grow = valid ? gr : -1;  // global output row (node * Hq + head), or -1 past the end
  const CB_GLOBAL uintx4* qp = (const CB_GLOBAL uintx4*)((const CB_GLOBAL uint16_t*)p.q + gr * D);
#pragma unroll
  for (int ds = 0; ds < D / 32; ds++) st.q[ds] = __builtin_bit_cast(bf16x8, load_b128_untracked(qp + kg + 4 * ds));
#pragma unroll
  for (int dt = 0; dt < D / 16; dt++) st.o[dt] = floatx4{0.f, 0.f, 0.f, 0.f};
  st.lacc = floatx4{0.f, 0.f, 0.f, 0.f};
  st.mref = -INFINITY;
  const bool tree_split = k1 > S;  // this split reaches the tree nodes: masks needed
  // the tree itself: one parent entry per thread, requested before the K/V loads
  int my_parent = -1;
  if (tree_split && tid < jb.N && tid < CB_MAX_NODES) {
    if (tid > 0) {
      my_parent = ((const CB_GLOBAL int32_t*)p.parent)[jb.off + tid];
      if (my_parent < 0 || my_parent >= tid) my_parent = 0;  // (same repair as the acceptance, which reports it)
    }
  }
  const float c2 = p.scale * 1.4426950408889634f;  // softmax scale in the log2 domain
  const int nst = (k1 - k0 + 2 * kUnitKeys - 1) / (2 * kUnitKeys);  // stages
  const int nu = 2 * nst;                                           // units requested: whole stages
  // The prologue requests PRO units, and the rest of the ring goes out right behind the first stage's barrier.  (A
  // compute unit takes about 0.3 us to issue a unit's requests; with the whole ring in front of the first wait the
  // first stage's arithmetic starts that much later for every unit added.)  A split of up to 32 NS keys -- the
  // 7B-shaped workload's 288 -- is thereby requested in full before any of its arithmetic.
#pragma unroll
  for (int u = 0; u < PRO; u++) {
    if (u < nu) {
      feed.issue(u, u);
      feed.counted();
    }
  }
  CB_TS(2);
  if (tree_split) build_ancestor_sets(sh.anc, jb.N, my_parent, jump_rounds(p.max_depth));  // uniform in the workgroup; hidden behind the first K/V wait
  feed.wait_units(2);
#pragma unroll
  for (int ds = 0; ds < D / 32; ds++) asm volatile("" : "+v"(st.q[ds]));  // (older than every unit)
  CB_TS(3);
  int slot = gi;  // of this group's unit of the stage
  for (int s = 0; s < nst; s++) {
    if (s > 0) feed.wait_units(2 * s + 2);  // every wave's share of stage s has landed, and nobody reads stage s-1 any more
    feed.request_up_to(nu < 2 * s + NS ? nu : 2 * s + NS);
    const int key0 = k0 + (2 * s + gi) * kUnitKeys;
    if (key0 < k1 && has_rows) compute_unit<D, PX>(feed.k_at(slot), feed.v_at(slot), st, c2, key0, S, k1, &sh.anc.anc[node][0], l);
    slot = slot + 2 >= NS ? slot + 2 - NS : slot + 2;
  }
  CB_TS(4);

  // Each group finishes one half of the head dimension, the pieces from gi * P/2.  It parks the other half of its
  // accumulators and its (mref, l) in the ring, and adds the partner's parked half to its own.
  floatx4 f[P / 2];
  __syncthreads();  // every wave is done with the ring
  floatx4* const park = reinterpret_cast<floatx4*>(ring) + w * 64 * (P / 2) + l;
  float2* const park_ml = reinterpret_cast<float2*>(ring + 8 * 64 * (P / 2));
#pragma unroll
  for (int i = 0; i < P / 2; i++) {
    f[i] = gi == 0 ? st.o[i] : st.o[P / 2 + i];
    park[i * 64] = gi == 0 ? st.o[P / 2 + i] : st.o[i];
  }
  park_ml[tid] = float2{st.mref, st.lacc[0]};
  __syncthreads();
  const floatx4* const theirs = reinterpret_cast<const floatx4*>(ring) + (w ^ 4) * 64 * (P / 2) + l;
  const float2 ml2 = park_ml[tid ^ 256];
  const float m = fmaxf(st.mref, ml2.x);
  const float mu = (m == -INFINITY) ? 0.f : m;
  const float w0 = __builtin_amdgcn_exp2f((st.mref - mu) * c2), w1 = __builtin_amdgcn_exp2f((ml2.x - mu) * c2);
#pragma unroll
  for (int i = 0; i < P / 2; i++) f[i] = f[i] * w0 + theirs[i * 64] * w1;
  const float lsum = st.lacc[0] * w0 + ml2.y * w1;
#undef CB_TS
  HeadMove<row_pieces(D, 2), 1> move;
  if (MOVE && tree_split && w == 0) move.begin(jb.b, jb.hk, S, jb.N);
  write_rows<D, 16, PX, P / 2>(p, jb, wi, grow, f, gi * (P / 2), m, lsum, c2, gi == 0, l);
  auto finish_move = [&] { if (MOVE) move.finish(jb.b, jb.hk, S, jb.N); };
  if (jb.nsplit == 1 || p.external_merge) {  // (a following kernel merges: the kernel boundary orders the stores)
    finish_move();
    return;
  }
  split_merge<D, 16, PX, 8, kSmallRows, TS>(p, jb, kSmallRows, sh, ts, finish_move);
}

template <int D, bool PX, bool LEAN, bool TS>
__device__ __forceinline__ void attn_workgroup(const AttnParams& p, const SeqMeta& meta) {
  const unsigned long long ts0 = TS ? wall_clock64() : 0ull;
  const SeqMetaLanes ml = seq_meta_prefetch(meta);
  __shared__ uint4 ring[Feed<D, 8, 16, LEAN>::kRingVecs];
  __shared__ TileLds sh;
  __shared__ unsigned long long ts_sh[TS ? 16 : 1];
  attn_tile<D, PX, LEAN, false, TS>(p, ml, blockIdx.x, ts0, sh, ring, ts_sh, OneLayer{});
  flush_timestamps<TS>(p, blockIdx.x, ts_sh);
}

// The whole verification in one launch: the first lw.n_wgs workgroups do the logits work (they are dispatched
// first, so the acceptance is through long before the attention is, and a waiting host has its results then),
// the others the attention.  Neither waits for the other.
template <int D, bool PX, bool LEAN, bool MOVE, bool TS>
__device__ __forceinline__ void verify_workgroup(const AttnParams& p, const SeqMeta& meta, const LogitsWork& lw) {
  const unsigned long long ts0 = TS ? wall_clock64() : 0ull;
  const SeqMetaLanes ml = seq_meta_prefetch(meta);
  __shared__ uint4 ring[Feed<D, 8, 16, LEAN>::kRingVecs];
  __shared__ TileLds sh;
  __shared__ unsigned long long ts_sh[TS ? 16 : 1];
  static_assert(sizeof(ring) >= sizeof(AcceptWaveLds), "the acceptance's LDS is the ring's");
  const int wg = (int)blockIdx.x - lw.n_wgs;
  if (wg < 0) {
    logits_share<8, 16>(lw, ml, blockIdx.x, *reinterpret_cast<AcceptWaveLds*>(ring), after_acceptance<MOVE, row_pieces(D, 2), 1, 4>());
    return;
  }
  attn_tile<D, PX, LEAN, MOVE, TS>(p, ml, wg, ts0, sh, ring, ts_sh, OneLayer{});
  flush_timestamps<TS>(p, wg, ts_sh);
}

// The attention of several layers in one launch, with the logits work (of the last one) in its first workgroups where lw.n_wgs is not 0.
template <int D, bool PX, bool LEAN>
__global__ __launch_bounds__(512) void k_model_mfma(AttnParams p, SeqMeta meta, LogitsWork lw, LayerTable layers) {
  const SeqMetaLanes ml = seq_meta_prefetch(meta);
  __shared__ uint4 ring[Feed<D, 8, 16, LEAN>::kRingVecs];
  __shared__ TileLds sh;
  const int wg = (int)blockIdx.x - lw.n_wgs;
  if (wg < 0) logits_share<8, 16>(lw, ml, blockIdx.x, *reinterpret_cast<AcceptWaveLds*>(ring));
  else attn_tile<D, PX, LEAN, false, false>(p, ml, wg, 0ull, sh, ring, nullptr, layers);
}

// head_dim 64 always holds probabilities and partial sums in 32 bits, head_dim 128 in the precise builds.
template <int D, bool TS>
__global__ __launch_bounds__(512) void k_attn_mfma(AttnParams p, SeqMeta meta) { attn_workgroup<D, D == 64, false, TS>(p, meta); }
template <int D, bool TS>
__global__ __launch_bounds__(512) void k_attn_lean(AttnParams p, SeqMeta meta) { attn_workgroup<D, D == 64, true, TS>(p, meta); }
template <bool LEAN, bool TS>
__global__ __launch_bounds__(512) void k_attn_precise(AttnParams p, SeqMeta meta) { attn_workgroup<128, true, LEAN, TS>(p, meta); }
template <int D, bool TS>
__global__ __launch_bounds__(512) void k_verify_mfma(AttnParams p, SeqMeta meta, LogitsWork lw) { verify_workgroup<D, D == 64, false, false, TS>(p, meta, lw); }
template <int D, bool TS>
__global__ __launch_bounds__(512) void k_verify_lean(AttnParams p, SeqMeta meta, LogitsWork lw) { verify_workgroup<D, D == 64, true, false, TS>(p, meta, lw); }
template <bool LEAN, bool TS>
__global__ __launch_bounds__(512) void k_verify_precise(AttnParams p, SeqMeta meta, LogitsWork lw) { verify_workgroup<128, true, LEAN, false, TS>(p, meta, lw); }
// with the compaction (builds of their own: what follows the sweep takes scalar registers from it)
template <int D, bool PX, bool LEAN>
__global__ __launch_bounds__(512) void k_step_mfma(AttnParams p, SeqMeta meta, LogitsWork lw) { verify_workgroup<D, PX, LEAN, true, false>(p, meta, lw); }

// Launches for tiles of up to 64 rows.  (Steps and launches for several layers have no timeline build; their lw.n_wgs is 0 where the logits
// work has a launch of its own.)
template <bool LEAN>
static hipError_t launch_small(hipStream_t st, dim3 grid, const AttnParams& p, const SeqMeta& meta, const LogitsWork* logits_work, const LayerTable* layers) {
  const LogitsWork lw = logits_work ? *logits_work : LogitsWork{};
  auto launch = [&](auto* kernel, auto... args) { hipLaunchKernelGGL(kernel, grid, dim3(512), 0, st, p, meta, args...); };
  auto either = [&](auto* stamped, auto* plain, auto... args) { launch(p.timeline != 0 ? stamped : plain, args...); };
  if (p.move.words) {
    if (p.D == 64) launch(k_step_mfma<64, true, LEAN>, lw);
    else if (p.precise) launch(k_step_mfma<128, true, LEAN>, lw);
    else launch(k_step_mfma<128, false, LEAN>, lw);
  } else if (layers) {
    if (p.D == 64) launch(k_model_mfma<64, true, LEAN>, lw, *layers);
    else if (p.precise) launch(k_model_mfma<128, true, LEAN>, lw, *layers);
    else launch(k_model_mfma<128, false, LEAN>, lw, *layers);
  } else if (p.precise && p.D == 128) {
    if (logits_work) either(k_verify_precise<LEAN, true>, k_verify_precise<LEAN, false>, lw);
    else either(k_attn_precise<LEAN, true>, k_attn_precise<LEAN, false>);
  } else if (logits_work) {
    if (p.D == 64) LEAN ? either(k_verify_lean<64, true>, k_verify_lean<64, false>, lw) : either(k_verify_mfma<64, true>, k_verify_mfma<64, false>, lw);
    else LEAN ? either(k_verify_lean<128, true>, k_verify_lean<128, false>, lw) : either(k_verify_mfma<128, true>, k_verify_mfma<128, false>, lw);
  } else {
    if (p.D == 64) LEAN ? either(k_attn_lean<64, true>, k_attn_lean<64, false>) : either(k_attn_mfma<64, true>, k_attn_mfma<64, false>);
    else LEAN ? either(k_attn_lean<128, true>, k_attn_lean<128, false>) : either(k_attn_mfma<128, true>, k_attn_mfma<128, false>);
  }
  return hipGetLastError();
}

// Stand-alone merge of the partials, used when a tile's partials are too many for one
// workgroup to pull through its compute unit: one workgroup per TR-row tile, its four waves take a quarter of the
// pieces each.  grid: x = TR-row tile, y = kv head, z = sequence; block = 256 threads.
template <int D, int TR, bool PX>
__global__ __launch_bounds__(256) void k_merge_partials(AttnParams p, SeqMeta meta) {
  constexpr int NP = PartialLayout<D, TR, PX>::P / 4;
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  TileJob jb{};
  jb.b = blockIdx.z;
  jb.hk = blockIdx.y;
  jb.g = p.Hq / p.Hkv;
  jb.off = meta.node_off[jb.b];
  jb.N = meta.node_off[jb.b + 1] - jb.off;
  jb.M = jb.N * jb.g;
  const int ti = blockIdx.x;
  const int len = meta.kv_len[jb.b] + jb.N;
  const int ns = (len + p.chunk - 1) / p.chunk;
  if (ns <= 1 || ti * TR >= jb.M) return;  // (one split: the attention kernel already wrote the output)
  const int row = ti * TR + l % TR;
  const int node = row / jb.g, hg = row - node * jb.g;
  const int64_t gr = row < jb.M ? (int64_t)(jb.off + node) * p.Hq + jb.hk * jb.g + hg : -1;
  merge_pieces<D, TR, PX, NP, 0, 8>(partial_rsrc<D, TR, PX>(p, jb), gr, partial_byte<D, TR, PX>(p, jb, ti), (CB_GLOBAL uint16_t*)p.out, ns, w * NP, l);
}

static int block_bytes(int D, int tr, bool precise) { return tr * D * (precise ? 4 : 2) + tr * 8; }
static_assert(PartialLayout<128, 16, false>::kBytes == 16 * 128 * 2 + 16 * 8 && PartialLayout<64, 32, true>::kBytes == 32 * 64 * 4 + 32 * 8, "");

size_t attn_mfma_partial_bytes(int D, bool precise, int tile_rows, size_t max_total_nodes, int Hq, int Hkv, int max_batch, int max_splits) {
  // the last sequence's blocks end at or before tile max_total_nodes * Hq / TR + (Hkv + 1) * max_batch
  const int tr = tile_rows == kSmallRows ? 16 : 32;
  const size_t tiles = max_total_nodes * Hq / tr + (size_t)(Hkv + 1) * max_batch + 1;
  return tiles * (size_t)max_splits * block_bytes(D, tr, precise);
}

bool attn_mfma_supports(const AttnParams& p) {
  if (p.D != 128 && p.D != 64) return false;
  if (p.D == 64 && !p.precise) return false;  // (not built)
  if (p.kv.block_size > 0) {
    if (p.kv.block_size & (p.kv.block_size - 1)) return false;
  }
  if (p.nsplit > 4095) return false;  // the ticket counts arrivals in 12 bits
  // partial offsets inside one sequence are 32-bit byte offsets of a buffer descriptor
  if ((int64_t)p.Hkv * ((CB_MAX_NODES * (p.Hq / p.Hkv) + 31) / 32) * p.nsplit * block_bytes(128, 32, p.D == 128 && p.precise) >= (1ll << 31)) return false;
  return true;
}

// Rows per workgroup tile for a call whose largest sequence has `mrows` rows (g query heads x N nodes) per kv head.  Up
// to 64 rows one small tile holds them all; beyond, a second small tile would read the same K/V again, which costs
// more than the wide tile's longer start (two tiles of 64 against one of 128 rows, 32 kv heads x 8192 keys: 93 us against
// 58).
int attn_mfma_tile_rows(int mrows) { return mrows <= kSmallRows ? kSmallRows : 256; }

// One workgroup can pull about 50 GB/s of partials through its compute unit: beyond a few hundred
// KiB per tile a separate, fully parallel merge kernel is cheaper than the merge by a tile's last workgroup.
bool attn_mfma_merges_inside(int D, bool precise, int mrows, int rt_rows, int nsplit) {
  const int tr = rt_rows == kSmallRows ? 16 : 32;
  const int in_tile = (std::min(mrows, rt_rows) + tr - 1) / tr;
  return (int64_t)nsplit * in_tile * block_bytes(D, tr, precise) <= 320 * 1024;
}

hipError_t launch_attn_mfma(hipStream_t st, const AttnParams& p, const SeqMeta& meta, int max_nodes_in_call,
                            int total_nodes, const LogitsWork* logits_work, const LayerTable* layers, int* merge_kind) {
  if (!attn_mfma_supports(p)) return hipErrorInvalidValue;
  const int g = p.Hq / p.Hkv;
  const int M = max_nodes_in_call * g;
  const int rt_rows = p.tile_rows;
  if (rt_rows != kSmallRows && rt_rows != 128 && rt_rows != 256) return hipErrorInvalidValue;
  const int tiles = (M + rt_rows - 1) / rt_rows;
  AttnParams q = p;
  q.grid_x = p.nsplit;
  q.grid_y = p.Hkv * tiles;
  q.grid_z = p.batch;
  int64_t T = (int64_t)p.nsplit * p.Hkv * tiles * p.batch;
  // renumbering needs whole groups of splits inside each XCD's share of the grid
  q.xcd_remap = (T % 8 == 0 && (T / 8) % p.nsplit == 0) ? 1 : 0;
  if (p.Hkv % 8 == 0 && p.batch > 1) {  // (several sequences: longest first within every XCD)
    q.xcd_remap = 2;
    T = p.live_wgs;
  } else if (q.grid_y % 8 == 0 && p.batch > 1) {
    q.xcd_remap = 3;
  }
  LayerTable table;
  if (layers) {
    table = *layers;
    table.wgs = (int32_t)T;
    table.tiles = p.batch * p.Hkv * tiles;
    if (q.xcd_remap != 2) T *= table.count;
    if (T > INT32_MAX) return hipErrorInvalidValue;
  }
  const int n_layers = layers ? layers->count : 1;
  // (the logits' workgroups come first; a multiple of 8 of them leaves the others' XCDs as they are)
  const int n_logits = logits_work ? logits_work->n_wgs : 0;
  const dim3 grid((uint32_t)(n_logits + T));
  const int tr = rt_rows == kSmallRows ? 16 : 32;
  q.external_merge = p.nsplit > 1 && !attn_mfma_merges_inside(p.D, p.precise, M, rt_rows, p.nsplit) ? 1 : 0;
  // A grid that is resident in one round (one workgroup per compute unit) merges cooperatively:
  // every workgroup of a tile takes a slice, so the volume per compute unit does not grow with
  // the split count and no second launch is needed.
  static int compute_units = 0;
  if (compute_units == 0) {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0) compute_units = n;
    else compute_units = -1;
  }
  q.coop_merge = (p.coop_merge >= 0 && p.coop_tickets && p.nsplit > 1 && p.nsplit <= 64 && compute_units > 0 && T + n_logits <= compute_units &&
                  (int64_t)p.Hkv * tiles * p.batch * n_layers <= kCoopTiles) ? 1 : 0;
  if (q.coop_merge) q.external_merge = 0;
  if (p.force_external_merge && p.nsplit > 1) { q.external_merge = 1; q.coop_merge = 0; }  // (option "external_merge": a test aid)
  if (merge_kind) *merge_kind = p.nsplit <= 1 ? 0 : (q.coop_merge ? 1 : (q.external_merge ? 3 : 2));
  if (layers && q.external_merge) return hipErrorInvalidValue;  // (the merge kernel knows one layer)
  hipError_t e;
  if (rt_rows == kSmallRows) {
    // The lean builds (contiguous caches) where there are several rounds of workgroups, each of which starts 0.1 us sooner: 48 sequences of 8 nodes x
    // 200 keys, 32 heads, a verification 47.4 -> 45.7 us, 64 of 4 x 40 41.4 -> 39.3.  Not in one round: decoding from the host with 63 nodes of
    // 32 heads x 4111 keys takes 25.2 us a step with the others and 25.9 with these.
    const bool lean = p.kv.block_size == 0 && (int64_t)n_logits + T > 256;
    e = lean ? launch_small<true>(st, grid, q, meta, logits_work, layers ? &table : nullptr)
             : launch_small<false>(st, grid, q, meta, logits_work, layers ? &table : nullptr);
  } else if (layers) {
    e = launch_attn_wide_layers(st, q, meta, std::min(M, rt_rows), (int)T, logits_work ? *logits_work : LogitsWork{}, table);
  } else {
    e = launch_attn_wide(st, q, meta, std::min(M, rt_rows), (int)T, logits_work);
  }
  if (e != hipSuccess) return e;
  if (q.external_merge) {
    const dim3 mgrid((M + tr - 1) / tr, p.Hkv, p.batch);
#define CB_MERGE(D, PX)                                                                                            \
  do {                                                                                                              \
    if (tr == 16) hipLaunchKernelGGL((k_merge_partials<D, 16, PX>), mgrid, dim3(256), 0, st, q, meta);              \
    else hipLaunchKernelGGL((k_merge_partials<D, 32, PX>), mgrid, dim3(256), 0, st, q, meta);                       \
  } while (0)
    if (p.D == 64) CB_MERGE(64, true);
    else if (p.precise) CB_MERGE(128, true);
    else CB_MERGE(128, false);
#undef CB_MERGE
    e = hipGetLastError();
  }
  return e;
}

}  // namespace cb
