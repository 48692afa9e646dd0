// Tree attention in fp32 on the matrix cores (head_dim 64 or 128), gfx950 only.
//
// Tree attention, Section 3.2 of the paper: node i of a tree attends to the KV-cached prefix (slots 0..S-1) and to the
// tree nodes on its own ancestor chain (slots S+a, a in anc(i)).  For one kv head the g*N query rows (g query heads per
// kv head, N nodes) form a dense matrix, so both products are contractions for v_mfma_f32_16x16x4_f32, whose products
// and sums are plain fp32; the exponentials are the accurate expf.
//
// A workgroup of 8 wavefronts works on a (sequence, kv head, 16-row tile, split).  The wavefronts take units of 16 keys
// in turn and share nothing until the end, so K and V go straight from memory to the registers the MFMAs read: no LDS,
// no barrier in the sweep.  Their softmax states are combined through LDS, the splits' by the tile's last workgroup.
// What bounds it: a unit is D/2 MFMAs of 32 cycles, two wavefronts to a SIMD, against D * 128 bytes per wavefront from
// the L2 (a kv head's tiles share an XCD): 32 of the 64 bytes a clock that a compute unit can take, so the matrix cores
// for long sweeps, and the chain of a unit's loads and products for short ones.
// Step times (verification and compaction): 16/8 heads of 128, 40 nodes, 1500 keys 17.9 us, against 257 with the scalar
// kernel, which reads K and V once for every row; 8/8 heads of 64, 15 nodes, 256 keys 9.9 us against 26.8 (three
// launches fewer are most of that).  The values are requested at the head of their own unit's arithmetic: a unit ahead (32 registers more)
// the short calls took 11.4 us, the first unit's in front of the ancestor sets 10.4.
//
// Register layouts (lane l, r = l % 16, h = l / 16):
//   scores transposed, S^T = K Q^T: MFMA (j, e) contracts the dims 16j + 4h + e; A = K[key r], B = Q[query r], so both
//   are 16-byte pieces of a row, and D[v] = S^T[key 4h+v][query r].
//   O^T = V^T P^T: MFMA (v, n, e) contracts the keys 4h + v; B = the lane's own probability v, A = V[key 4h+v][dim
//   64n + 4r + e], again 16-byte pieces; D[i] = O^T[dim 64n + 16h + 4i + e][query r].
#include "cb_logits.h"

namespace cb {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

constexpr int kF32Rows = 16;   // rows per tile
constexpr int kF32Unit = 16;   // keys per unit
constexpr int kF32Waves = 8;
// Wavefronts that a SIMD has registers for: two whole workgroups at head_dim 64, and at 128 one and a half, so that a workgroup whose
// wavefronts end one by one makes room for the next before its last one has.  (Verifications at 128 with 169 registers instead of 168,
// where a workgroup waits for all of the one before it: 32 sequences of 4 nodes x 60 keys, 16/8 heads, 13.5 us for 11.7, 33 x 300 72.5 for 71.5.)
constexpr int f32_waves(int D) { return D == 64 ? 4 : 3; }

template <int D>
struct F32Lds {
  static constexpr int kStride = D + 4;   // (rows 16 bytes apart in the banks)
  AncScratch anc;
  float o[kF32Waves][kF32Rows * kStride];
  float2 ml[kF32Waves][kF32Rows];
  int last;
};

// Partial states are written through to memory and read past the reader's own L2 (the splits of a tile may run on
// different XCDs); 64-bit accesses, two floats each.
__device__ __forceinline__ void store_pair(float* p, float a, float b) {
  const unsigned long long x = (unsigned long long)__float_as_uint(a) | ((unsigned long long)__float_as_uint(b) << 32);
  __hip_atomic_store((CBL_GLOBAL unsigned long long*)p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 load_pair(const float* p) {
  const unsigned long long x = __hip_atomic_load((const CBL_GLOBAL unsigned long long*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return float2{__uint_as_float((uint32_t)x), __uint_as_float((uint32_t)(x >> 32))};
}
__device__ __forceinline__ float rows_max(float x) {  // over the four lanes with equal r
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float weight(float m, float ref) { return m == -INFINITY ? 0.f : expf(m - ref); }

template <int D, bool MOVE, typename Layers>
__device__ __forceinline__ void attn_f32_tile(const AttnParams& p_arg, const SeqMetaLanes& ml, int wg, F32Lds<D>& sh, const Layers& layers) {
  constexpr int NJ = D / 16, NB = D / 64;
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, r = l & 15, h = l >> 4;
  // The kv head runs fastest: with a multiple of 8 heads a head's tiles and splits meet in one XCD's L2.  Then row
  // tiles, splits, and the sequences from the longest to the shortest.
  AttnParams p = p_arg;
  if constexpr (Layers::kMany) {
    const int i = __builtin_amdgcn_readfirstlane(wg / layers.wgs);
    wg -= i * layers.wgs;
    p.q = layers.at[i].q;
    p.out = layers.at[i].out;
    p.kv.k = layers.at[i].k;
    p.kv.v = layers.at[i].v;
    p.partial = reinterpret_cast<float*>(reinterpret_cast<char*>(p.partial) + i * layers.partial_bytes);
    p.tickets += (int64_t)i * layers.tiles;
  }
  const int hk = wg % p.Hkv;
  int rest = wg / p.Hkv;
  const int rt = rest % p.grid_y;
  rest /= p.grid_y;
  const int split = rest % p.nsplit;
  const int b = __builtin_amdgcn_readlane(ml.ord, rest / p.nsplit);
  const SeqShape shp = seq_shape(ml, b);
  const int S = shp.S, N = shp.N, len = S + N, g = p.Hq / p.Hkv, M = N * g;
  const int k0 = split * p.chunk, row0 = rt * kF32Rows;
  if (row0 >= M || k0 >= len) return;
  const int k1 = k0 + p.chunk < len ? k0 + p.chunk : len;
  const int nsplit = (len + p.chunk - 1) / p.chunk;
  const int nu = (k1 - k0 + kF32Unit - 1) / kF32Unit;
  const CBL_GLOBAL float* const kb = (const CBL_GLOBAL float*)p.kv.k;
  const CBL_GLOBAL float* const vb = (const CBL_GLOBAL float*)p.kv.v;

  // The tree first: loads return in the order of their requests, and the ancestor sets are the longest chain of the start.
  const bool tree_split = k1 > S;
  int raw_parent = -1;
  if (tree_split && tid < N) raw_parent = as_global(p.parent)[shp.off + tid];

  const int row = row0 + r < M ? row0 + r : M - 1;   // (rows past the end repeat the last one and are not written)
  const int node = row / g;
  const CBL_GLOBAL f32x4* const qp = (const CBL_GLOBAL f32x4*)((const CBL_GLOBAL float*)p.q +
                                                               ((int64_t)(shp.off + node) * p.Hq + hk * g + (row - node * g)) * D);
  f32x4 q[NJ];
#pragma unroll
  for (int j = 0; j < NJ; j++) q[j] = qp[4 * j + h];
  // keys past the split's end repeat its last one (masked below), so every address stays inside the sequence
  auto load_k = [&](int u, f32x4 (&k)[NJ]) {
    int key = k0 + u * kF32Unit + r;
    key = key < k1 ? key : k1 - 1;
    const CBL_GLOBAL f32x4* const kp = (const CBL_GLOBAL f32x4*)(kb + slot_offset(p.kv, b, key, hk));
#pragma unroll
    for (int j = 0; j < NJ; j++) k[j] = kp[4 * j + h];
  };
  auto load_v = [&](int u, f32x4 (&v)[4][NB]) {
#pragma unroll
    for (int x = 0; x < 4; x++) {
      int key = k0 + u * kF32Unit + 4 * h + x;
      key = key < k1 ? key : k1 - 1;
      const CBL_GLOBAL f32x4* const vp = (const CBL_GLOBAL f32x4*)(vb + slot_offset(p.kv, b, key, hk));
#pragma unroll
      for (int n = 0; n < NB; n++) v[x][n] = vp[16 * n + r];
    }
  };
  f32x4 k[NJ];
  load_k(w, k);

  if (tree_split) {  // the tree's ancestor sets, behind the first loads; complete for any depth a tree of N nodes can have
    const bool report = hk == 0 && rt == 0;
    const bool odd = tid < N && (tid == 0 ? raw_parent != -1 : raw_parent < 0 || raw_parent >= tid);  // (as sanitized_parent)
    const int par = tid == 0 || tid >= N ? -1 : odd ? 0 : raw_parent;
    if (odd && report) atomicOr(p.status, 1);
    build_ancestor_sets(sh.anc, N, par, jump_rounds(N - 1));
    if (report && tid < N) {
      int depth = -1;
#pragma unroll
      for (int x = 0; x < kAncWords; x++) depth += __popc(sh.anc.anc[tid][x]);
      if (depth > p.max_depth) atomicOr(p.status, 2);
    }
  }

  f32x4 o[NB][4];
#pragma unroll
  for (int n = 0; n < NB; n++)
#pragma unroll
    for (int e = 0; e < 4; e++) o[n][e] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, lsum = 0.f;
  for (int u = w; u < nu; u += kF32Waves) {
    f32x4 v[4][NB], kn[NJ];
    load_v(u, v);
    load_k(u + kF32Waves, kn);
    f32x4 s = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < NJ; j += 2)
#pragma unroll
      for (int e = 0; e < 4; e++) {
        s = __builtin_amdgcn_mfma_f32_16x16x4f32(k[j][e], q[j][e], s, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(k[j + 1][e], q[j + 1][e], s1, 0, 0, 0);
      }
    s = (s + s1) * p.scale;
    const int key0 = k0 + u * kF32Unit;
    const bool masked = key0 + kF32Unit > (S < k1 ? S : k1);  // (uniform)
    bool odd_v = false;
    if (masked) {
#pragma unroll
      for (int x = 0; x < 4; x++) {
        const int key = key0 + 4 * h + x, t = key - S;
        const bool vis = key < k1 && (t < 0 || ((sh.anc.anc[node][t >> 5] >> (t & 31)) & 1u));
        s[x] = vis ? s[x] : -INFINITY;
      }
      // A value that a query must not see reaches its sum with weight 0, which hides it only if it is finite.
      bool bad = false;
#pragma unroll
      for (int x = 0; x < 4; x++)
#pragma unroll
        for (int n = 0; n < NB; n++)
#pragma unroll
          for (int e = 0; e < 4; e++) {
            const bool fin = (__float_as_uint(v[x][n][e]) & 0x7f800000u) != 0x7f800000u;
            bad |= !fin;
            v[x][n][e] = fin ? v[x][n][e] : 0.f;
          }
      odd_v = __builtin_amdgcn_ballot_w64(bad) != 0ull;
    }
    const float mn = fmaxf(m, rows_max(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]))));
    if (__builtin_amdgcn_ballot_w64(mn > m) != 0ull) {
      const float alpha = weight(m, mn);
#pragma unroll
      for (int n = 0; n < NB; n++)
#pragma unroll
        for (int e = 0; e < 4; e++) o[n][e] *= alpha;
      lsum *= alpha;
      m = mn;
    }
    float pr[4];
#pragma unroll
    for (int x = 0; x < 4; x++) {
      pr[x] = weight(s[x], m);
      lsum += pr[x];
    }
#pragma unroll
    for (int x = 0; x < 4; x++)
#pragma unroll
      for (int n = 0; n < NB; n++)
#pragma unroll
        for (int e = 0; e < 4; e++) o[n][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[x][n][e], pr[x], o[n][e], 0, 0, 0);
    if (odd_v) {  // (never in earnest: infinities or NaN among the unit's values, for the queries that do see them)
      for (int kk = 0; kk < kF32Unit && key0 + kk < k1; kk++) {
        const float mine = (kk & 2) ? ((kk & 1) ? pr[3] : pr[2]) : ((kk & 1) ? pr[1] : pr[0]);
        const float pk = __shfl(mine, (kk >> 2) * 16 + r, 64);
        const CBL_GLOBAL float* const vp = vb + slot_offset(p.kv, b, key0 + kk, hk);
#pragma unroll
        for (int n = 0; n < NB; n++)
#pragma unroll
          for (int e = 0; e < 4; e++)
#pragma unroll
            for (int i = 0; i < 4; i++) {
              const float x = vp[64 * n + 16 * h + 4 * i + e];
              const bool fin = (__float_as_uint(x) & 0x7f800000u) != 0x7f800000u;
              o[n][e][i] += (fin || pk == 0.f) ? 0.f : pk * x;
            }
      }
    }
#pragma unroll
    for (int j = 0; j < NJ; j++) k[j] = kn[j];
  }
  lsum += __shfl_xor(lsum, 16, 64);
  lsum += __shfl_xor(lsum, 32, 64);

  // The wavefronts' states into one.  Thread t then owns 4 dims of a row.
  constexpr int PS = partial_stride(D), LS = F32Lds<D>::kStride;
#pragma unroll
  for (int n = 0; n < NB; n++)
#pragma unroll
    for (int i = 0; i < 4; i++)
      *reinterpret_cast<f32x4*>(&sh.o[w][r * LS + 64 * n + 16 * h + 4 * i]) = f32x4{o[n][0][i], o[n][1][i], o[n][2][i], o[n][3][i]};
  if (h == 0) sh.ml[w][r] = float2{m, lsum};
  __syncthreads();
  HeadMove<row_pieces(D, 4), 2> move;
  if (MOVE && k1 > S && w == kF32Waves - 1) move.begin(b, hk, S, N);  // (nobody reads K or V any more)
  const int orow = tid / (D / 4), c = tid % (D / 4) * 4;
  const bool live = orow < kF32Rows && row0 + orow < M;
  const int onode = (row0 + orow) / g;
  const int64_t grow = (int64_t)(shp.off + onode) * p.Hq + hk * g + (row0 + orow - onode * g);
  float* const part = p.partial + grow * p.nsplit * PS;
  if (live) {
    float mm = -INFINITY, ll = 0.f;
    f32x4 oo = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int x = 0; x < kF32Waves; x++) mm = fmaxf(mm, sh.ml[x][orow].x);
#pragma unroll
    for (int x = 0; x < kF32Waves; x++) {
      const float2 st = sh.ml[x][orow];
      const float wgt = weight(st.x, mm);
      ll += st.y * wgt;
      oo += *reinterpret_cast<const f32x4*>(&sh.o[x][orow * LS + c]) * wgt;
    }
    if (nsplit == 1) {
      *(CBL_GLOBAL f32x4*)((CBL_GLOBAL float*)p.out + grow * D + c) = oo / ll;
    } else {
      float* const pp = part + split * PS;
      store_pair(pp + c, oo[0], oo[1]);
      store_pair(pp + c + 2, oo[2], oo[3]);
      if (c == 0) store_pair(pp + D, mm, ll);
    }
  }
  auto finish_move = [&] { if (MOVE) move.finish(b, hk, S, N); };
  if (nsplit == 1 || p.external_merge) {  // (k_merge follows: the kernel boundary orders the stores)
    finish_move();
    return;
  }
  // The stores are acknowledged before the ticket is drawn, so whoever completes the tile finds all of them in memory.
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) {
    CBL_GLOBAL uint32_t* const ticket = as_global(p.tickets) + ((int64_t)b * p.Hkv + hk) * p.grid_y + rt;
    const uint32_t n = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
    sh.last = n == (uint32_t)nsplit;
    if (n == (uint32_t)nsplit) __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // ready for the next launch
  }
  __syncthreads();
  finish_move();
  if (!sh.last || !live) return;
  constexpr int BS = 8;   // splits whose loads are in flight together
  float mm = -INFINITY, ll = 0.f;
  f32x4 oo = {0.f, 0.f, 0.f, 0.f};
  for (int t0 = 0; t0 < nsplit; t0 += BS) {
    float2 st[BS], x0[BS], x1[BS];
#pragma unroll
    for (int x = 0; x < BS; x++) {
      const float* const pp = part + (t0 + x < nsplit ? t0 + x : nsplit - 1) * PS;
      st[x] = load_pair(pp + D);
      x0[x] = load_pair(pp + c);
      x1[x] = load_pair(pp + c + 2);
    }
    float mn = mm;
#pragma unroll
    for (int x = 0; x < BS; x++) mn = fmaxf(mn, st[x].x);
    const float alpha = weight(mm, mn);
    oo *= alpha;
    ll *= alpha;
    mm = mn;
#pragma unroll
    for (int x = 0; x < BS; x++) {
      if (t0 + x >= nsplit) break;  // (a repeated split)
      const float wgt = weight(st[x].x, mm);
      ll += st[x].y * wgt;
      oo += f32x4{x0[x].x, x0[x].y, x1[x].x, x1[x].y} * wgt;
    }
  }
  *(CBL_GLOBAL f32x4*)((CBL_GLOBAL float*)p.out + grow * D + c) = oo / ll;
}

template <int D>
__global__ __launch_bounds__(64 * kF32Waves, f32_waves(D)) void k_attn_f32(AttnParams p, SeqMeta meta) {
  __shared__ F32Lds<D> sh;
  const SeqMetaLanes ml = seq_meta_prefetch(meta);
  attn_f32_tile<D, false>(p, ml, blockIdx.x, sh, OneLayer{});
}

// The whole verification in one launch: the first lw.n_wgs workgroups do the logits work, the others the attention.
template <int D, bool MOVE>
__device__ __forceinline__ void verify_f32(const AttnParams& p, const SeqMeta& meta, const LogitsWork& lw) {
  __shared__ union Lds {
    F32Lds<D> attn;
    AcceptWaveLds accept;
  } sh;
  const SeqMetaLanes ml = seq_meta_prefetch(meta);
  const int wg = (int)blockIdx.x - lw.n_wgs;
  if (wg < 0) logits_share<kF32Waves, 8>(lw, ml, blockIdx.x, sh.accept, after_acceptance<MOVE, row_pieces(D, 4), 2, 4>());
  else attn_f32_tile<D, MOVE>(p, ml, wg, sh.attn, OneLayer{});
}
template <int D>
__global__ __launch_bounds__(64 * kF32Waves, f32_waves(D)) void k_verify_f32(AttnParams p, SeqMeta meta, LogitsWork lw) { verify_f32<D, false>(p, meta, lw); }
// with the compaction (lw.n_wgs is 0 where the logits work has a launch of its own)
template <int D>
__global__ __launch_bounds__(64 * kF32Waves, f32_waves(D)) void k_step_f32(AttnParams p, SeqMeta meta, LogitsWork lw) { verify_f32<D, true>(p, meta, lw); }

// The attention of several layers in one launch, with the logits work (of the last one) in its first workgroups where lw.n_wgs is not 0.
template <int D>
__global__ __launch_bounds__(64 * kF32Waves, f32_waves(D)) void k_model_f32(AttnParams p, SeqMeta meta, LogitsWork lw, LayerTable layers) {
  __shared__ union Lds {
    F32Lds<D> attn;
    AcceptWaveLds accept;
  } sh;
  const SeqMetaLanes ml = seq_meta_prefetch(meta);
  const int wg = (int)blockIdx.x - lw.n_wgs;
  if (wg < 0) logits_share<kF32Waves, 8>(lw, ml, blockIdx.x, sh.accept);
  else attn_f32_tile<D, false>(p, ml, wg, sh.attn, layers);
}

// Splits of the longest sequence.  A workgroup costs about 3 us beside its sweep (start, combine, tail), every 128 keys
// it sweeps 1.7 us at head_dim 128 (a unit for each wavefront, two of them to a matrix core), a merge 2.5 us and a
// little for every split; `units` compute units run one workgroup each.  us: that
// estimate for the count returned.
int attn_f32_splits(int Hq, int Hkv, int D, int max_splits, int batch, const int32_t* kv_len, const int32_t* node_offsets, int max_len, int units, int layers, double* us) {
  const int cap = max_splits < (max_len + 127) / 128 ? max_splits : (max_len + 127) / 128;
  int best = 1;
  double best_cost = 0.0;
  for (int ns = 1; ns <= cap; ns++) {
    const int chunk = ((max_len + ns - 1) / ns + 31) / 32 * 32;
    int64_t jobs = 0;
    for (int b = 0; b < batch; b++) {
      const int n = node_offsets[b + 1] - node_offsets[b];
      jobs += (int64_t)((n * (Hq / Hkv) + kF32Rows - 1) / kF32Rows) * Hkv * ((kv_len[b] + n + chunk - 1) / chunk);
    }
    const double sweep = 1.7 * D / 128 * ((chunk + 127) / 128);
    const double cost = (double)((jobs * layers + units - 1) / units) * (3.0 + sweep) + (ns > 1 ? 2.5 + 0.15 * ns : 0.0);
    if (ns == 1 || cost < best_cost) { best = ns; best_cost = cost; }
  }
  if (us) *us = best_cost;
  return best;
}

hipError_t launch_attn_f32(hipStream_t st, const AttnParams& params, const SeqMeta& meta, int max_nodes_in_call, const LogitsWork* lw, const LayerTable* layers) {
  AttnParams p = params;
  p.grid_y = (max_nodes_in_call * (p.Hq / p.Hkv) + kF32Rows - 1) / kF32Rows;
  p.tile_rows = kF32Rows;
  p.external_merge = p.force_external_merge;
  const int64_t per_layer = (int64_t)p.Hkv * p.grid_y * p.nsplit * p.batch, wgs = per_layer * (layers ? layers->count : 1) + (lw ? lw->n_wgs : 0);
  if (wgs > INT32_MAX || (p.D != 64 && p.D != 128)) return hipErrorInvalidValue;
  const dim3 grid((uint32_t)wgs), block(64 * kF32Waves);
  if (layers) {
    if (p.external_merge) return hipErrorInvalidValue;  // (the merge kernel knows one layer)
    LayerTable table = *layers;
    table.wgs = (int32_t)per_layer;
    table.tiles = p.batch * p.Hkv * p.grid_y;
    const LogitsWork work = lw ? *lw : LogitsWork{};
    if (p.D == 64) hipLaunchKernelGGL(k_model_f32<64>, grid, block, 0, st, p, meta, work, table);
    else hipLaunchKernelGGL(k_model_f32<128>, grid, block, 0, st, p, meta, work, table);
    return hipGetLastError();
  }
  if (p.move.words) {
    const LogitsWork work = lw ? *lw : LogitsWork{};
    if (p.D == 64) hipLaunchKernelGGL(k_step_f32<64>, grid, block, 0, st, p, meta, work);
    else hipLaunchKernelGGL(k_step_f32<128>, grid, block, 0, st, p, meta, work);
    return hipGetLastError();
  }
  if (lw && p.D == 64) hipLaunchKernelGGL(k_verify_f32<64>, grid, block, 0, st, p, meta, *lw);
  else if (lw) hipLaunchKernelGGL(k_verify_f32<128>, grid, block, 0, st, p, meta, *lw);
  else if (p.D == 64) hipLaunchKernelGGL(k_attn_f32<64>, grid, block, 0, st, p, meta);
  else hipLaunchKernelGGL(k_attn_f32<128>, grid, block, 0, st, p, meta);
  return hipGetLastError();
}

}  // namespace cb
