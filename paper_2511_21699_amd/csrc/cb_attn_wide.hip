// Tree attention for tiles of 65 to 256 rows (bf16, head_dim 64 or 128), gfx950 only.
//
// A tile's rows decide how the 8 waves share it: RW row groups of 32 rows times KW = 8 / RW key groups (two key
// groups up to 128 rows, one beyond).  A unit of work is 32 keys; a stage is KW units, one for each key
// group, whose softmax states are combined through LDS at the end.
//
// Register layouts (v_mfma_f32_32x32x16_bf16; lane l, r = l % 32, h = l / 32):
//   scores are computed transposed, S^T = K Q^T: A = K rows (key r, dims 8h..8h+7 of the 16-dim step), B = Q^T
//   (query r, same dims), D[v] = S^T[key 8(v/4)+4h+v%4][query r].  A lane therefore holds 16 keys x 1 query:
//   softmax statistics are per-lane scalars shared by the 2 lanes with equal r.
//   O^T = V^T P^T: B = P^T packs the lane's 8 probabilities of a 16-key step j (element e <-> key
//   16j + 8(e/4) + 4h + e%4, which is what D holds), A = V^T must hold the same keys for dim r of the 32-dim
//   tile; it is fetched from the row-major V tile with ds_read_b64_tr_b16 (each 16-lane group reads a 4-key x
//   16-dim block and receives it transposed).  D[v] = O^T[dim 8(v/4)+4h+v%4][query r].
#include "cb_attn_tile.h"

namespace cb {

template <int D>
struct TileState {
  bf16x8 q[D / 16];     // B operands of QK^T: query r, dims 16 ds + 8h ..
  floatx16 o[D / 32];   // O^T accumulators, dim tiles of 32
  floatx4 lacc;         // softmax denominator of the lane's query (all four elements equal)
  float mref;           // reference maximum of the raw scores (q.k, before the softmax scale)
  float nm;             // -mref in log2 units (0 while mref is -inf)
};

__device__ __forceinline__ float half_swap_max(float x) {  // maximum over lanes l and l ^ 32
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return maxn(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

template <int D>
__device__ __forceinline__ uint4 read_k1(const uint4* ks, int ds, int l) {
  const int r = l & 31, h = l >> 5;
  return ks[r * (D / 8) + ((2 * ds + h) ^ swizzle_k<D>(r))];
}
template <int D>
__device__ __forceinline__ void read_k(const uint4* ks, uint4 (&k)[D / 16], int l) {
#pragma unroll
  for (int ds = 0; ds < D / 16; ds++) k[ds] = read_k1<D>(ks, ds, l);
}
// scores of a unit: S^T = K Q^T
template <int D>
__device__ __forceinline__ void scores(const uint4 (&k)[D / 16], const TileState<D>& st, floatx16& s) {
#pragma unroll
  for (int v = 0; v < 16; v++) s[v] = 0.f;
#pragma unroll
  for (int ds = 0; ds < D / 16; ds++) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, k[ds]), st.q[ds], s, 0, 0, 0);
}
// probabilities p = 2^(c*s - c*mref), packed as B operands of PV; with PX the roundings' rests behind them
template <int D, bool PX>
__device__ __forceinline__ void probs(const floatx16& s, const TileState<D>& st, float c2, bf16x8 (&p)[PX ? 4 : 2]) {
  const float nm = st.nm;
#pragma unroll
  for (int j = 0; j < 2; j++) {
    union { bf16x8 v; __bf16 e[8]; } pk, rest;
#pragma unroll
    for (int e = 0; e < 8; e++) {
      const float pe = __builtin_amdgcn_exp2f(fmaf(s[8 * j + e], c2, nm));
      pk.e[e] = (__bf16)pe;
      if (PX) rest.e[e] = (__bf16)(pe - (float)pk.e[e]);
    }
    p[j] = pk.v;
    if constexpr (PX) p[2 + j] = rest.v;
  }
}
template <int D>
__device__ __forceinline__ bf16x8 read_v(const uint4* vs, int dt, int j, int l) {
  const int c = l & 15, h = l >> 5, dh = (l >> 4) & 1;
  const int piece = 4 * dt + 2 * dh + ((c & 3) >> 1);
  bf16x4 x[2];
#pragma unroll
  for (int u = 0; u < 2; u++) {
    const int row = 16 * j + 8 * u + 4 * h + (c >> 2);
    const int slot = piece ^ swizzle_v<D, 32>(row);
    const char* addr = reinterpret_cast<const char*>(vs) + row * (D * 2) + slot * 16 + (c & 1) * 8;
    x[u] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((bf16x4 __attribute__((address_space(3)))*)(addr));
  }
  return __builtin_shufflevector(x[0], x[1], 0, 1, 2, 3, 4, 5, 6, 7);
}
// A operand of the denominator's MFMA (16x16x32 over the B operands of a 16-key step): ones where output row and
// key group belong to the same half of the queries, so that every lane's accumulator is its own query's sum
__device__ __forceinline__ bf16x8 half_ones(int l) {
  const uint32_t x = (((l >> 2) & 1) == ((l >> 4) & 1)) ? 0x3f803f80u : 0u;
  return __builtin_bit_cast(bf16x8, uint4{x, x, x, x});
}

// Keys the lane's query must not see get -inf: prefix keys below S are visible, tree keys by the ancestor word,
// keys at or past `kend` belong to the next split (or do not exist).
__device__ __forceinline__ void mask_scores(floatx16& s, int key0, int S, int kend, const uint32_t* arow, int h) {
  const int np = S - key0;     // prefix keys in the unit (may be <= 0 or >= 32)
  const int ne = kend - key0;  // keys before the split's end
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
  if (ne < 32) vis = ne <= 0 ? 0u : vis & ((1u << ne) - 1u);
  vis >>= 4 * h;
#pragma unroll
  for (int v = 0; v < 16; v++) s[v] = ((vis >> (8 * (v >> 2) + (v & 3))) & 1u) ? s[v] : -INFINITY;
}

__device__ __forceinline__ float row_max(const floatx16& s) {
  float m = maxn(maxn(s[0], s[1]), s[2]);
#pragma unroll
  for (int v = 3; v < 15; v += 2) m = maxn(maxn(m, s[v]), s[v + 1]);
  return half_swap_max(maxn(m, s[15]));
}
// Lazy reference: it is only raised (and O, l rescaled) when the maximum has grown by more than kRescaleSlack, so
// probabilities stay below 2^8 and the accumulators are rarely touched by the vector ALU.
template <int D>
__device__ __forceinline__ bool must_raise(const TileState<D>& st, float mx, float c2) {  // uniform
  return __builtin_amdgcn_ballot_w64((mx - st.mref) * c2 > kRescaleSlack) != 0ull;  // (false when both are -inf: NaN)
}
template <int D>
__device__ __forceinline__ void raise_reference(TileState<D>& st, float mx, float c2) {
  const bool raise = (mx - st.mref) * c2 > kRescaleSlack;
  const float alpha = raise ? __builtin_amdgcn_exp2f((st.mref - mx) * c2) : 1.0f;
  if (raise) {
    st.mref = mx;
    st.nm = -mx * c2;
  }
#pragma unroll
  for (int dt = 0; dt < D / 32; dt++) st.o[dt] *= alpha;
  st.lacc *= alpha;
}

// One steady step of a wave, in two halves: score_half scores a unit (its K operands in `k`, scores to sn) while the
// unit scored before it (sc) is exponentiated (to pb), add_half adds that unit's values (at vs) up while the maxima of sn
// are taken (to mx).  Written in issue order, pinned by the scheduling barriers: an MFMA occupies the matrix core for 32
// cycles in which the wave issues what belongs to the other unit (a v_exp_f32 takes 8 cycles, other vector
// instructions 4 to 5).  Left alone the compiler gathers each kind.
// score_half ends with the reads of add_half's first operands (v).  req(i), i = 0 .. NREQ - 1: memory requests to be
// spread over score_half.
// PREK: `k` is filled again in add_half, for the next score_half (its unit's K at kn).
template <int D, bool PX, int NREQ, typename Req>
__device__ __forceinline__ void score_half(const uint4 (&k)[D / 16], const TileState<D>& st, const floatx16& sc, floatx16& sn,
                                           uintx4 (&pb)[PX ? 4 : 2], const uint4* vs, bf16x8 (&v)[D / 32], float c2, int l, Req req) {
  constexpr int DS = D / 16, DT = D / 32;
  // The probabilities in three stages, each a slot behind the one before it, so that no instruction waits for the one
  // in front of it: argument, exponential, packing.  Slot i handles elements 2 i and 2 i + 1 (constant indices).
  constexpr int NP2 = 8;
  float x0[NP2], x1[NP2];
  auto arg = [&](int i) {
    if (i >= NP2) return;
    x0[i] = fmaf(sc[2 * i], c2, st.nm);
    x1[i] = fmaf(sc[2 * i + 1], c2, st.nm);
    asm volatile("" : "+v"(x0[i]), "+v"(x1[i]));
  };
  auto expo = [&](int i) {
    if (i < 0 || i >= NP2) return;
    x0[i] = __builtin_amdgcn_exp2f(x0[i]);
    x1[i] = __builtin_amdgcn_exp2f(x1[i]);
    asm volatile("" : "+v"(x0[i]), "+v"(x1[i]));
  };
  auto pack = [&](int i) {
    if (i < 0 || i >= NP2) return;
    typedef float float2v __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
    uint32_t z = __builtin_bit_cast(uint32_t, __builtin_convertvector((float2v){x0[i], x1[i]}, bf16x2v));
    asm volatile("" : "+v"(z));
    pb[i >> 2][i & 3] = z;
    if constexpr (PX) {
      const float r0 = x0[i] - __uint_as_float(z << 16), r1 = x1[i] - __uint_as_float(z & 0xffff0000u);
      uint32_t y = __builtin_bit_cast(uint32_t, __builtin_convertvector((float2v){r0, r1}, bf16x2v));
      asm volatile("" : "+v"(y));
      pb[2 + (i >> 2)][i & 3] = y;
    }
  };
  arg(0);
  arg(1);
  expo(0);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int x = 0; x < 16; x++) sn[x] = 0.f;
  constexpr int PER = 8 / DS;  // slots per MFMA
#pragma unroll
  for (int ds = 0; ds < DS; ds++) {
    sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, k[ds]), st.q[ds], sn, 0, 0, 0);
#pragma unroll
    for (int q = 0; q < PER; q++) {
      const int i = ds * PER + q;
      expo(i + 1);
      pack(i);
      arg(i + 2);
    }
    if (ds >= DS - DT) v[ds - (DS - DT)] = read_v<D>(vs, ds - (DS - DT), 0, l);
    if (NREQ > 0 && ds % (DS / (NREQ > 0 ? NREQ : 1)) == 0) req(ds / (DS / (NREQ > 0 ? NREQ : 1)));
    __builtin_amdgcn_sched_barrier(0);
  }
}
template <int D, bool PX, bool PREK>
__device__ __forceinline__ void add_half(uint4 (&k)[D / 16], const uint4* kn, const uint4* vs, bf16x8 (&v)[D / 32], TileState<D>& st,
                                         const uintx4 (&pb)[PX ? 4 : 2], const floatx16& sn, float& mx, const bf16x8& ones, int l) {
  constexpr int DS = D / 16, DT = D / 32;
  // the maxima of the new scores, then across the lanes, a few beside every MFMA from the second on
  float m;
  auto maxima = [&](int i) {  // (constant index)
    if (i < 0 || i >= 10) return;
    if (i == 0) m = maxn(maxn(sn[0], sn[1]), sn[2]);
    else if (i < 7) m = maxn(maxn(m, sn[2 * i + 1]), sn[2 * i + 2]);
    else if (i == 7) m = maxn(m, sn[15]);
    else if (i == 8) mx = half_swap_max(m);
    if (i < 8) asm volatile("" : "+v"(m));
    else asm volatile("" : "+v"(mx));
  };
  constexpr int NPV = 2 * DT;                        // PV MFMAs
  constexpr int MPER = (10 + NPV - 3) / (NPV - 2);   // maxima per MFMA
#pragma unroll
  for (int j = 0; j < 2; j++) {
#pragma unroll
    for (int dt = 0; dt < DT; dt++) {
      const int n = j * DT + dt;
      st.o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v[dt], __builtin_bit_cast(bf16x8, pb[j]), st.o[dt], 0, 0, 0);
      if constexpr (PX) st.o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v[dt], __builtin_bit_cast(bf16x8, pb[2 + j]), st.o[dt], 0, 0, 0);
      // (the operand's registers take the next thing from LDS)
      if (j == 0) v[dt] = read_v<D>(vs, dt, 1, l);
      else if (PREK) {
#pragma unroll
        for (int q = 0; q < DS / DT; q++) k[dt * (DS / DT) + q] = read_k1<D>(kn, dt * (DS / DT) + q, l);
      }
      if (dt == DT - 1) {
#pragma unroll
        for (int x = j; x < (PX ? 4 : 2); x += 2)
          st.lacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, __builtin_bit_cast(bf16x8, pb[x]), st.lacc, 0, 0, 0);
      }
#pragma unroll
      for (int q = 0; q < MPER; q++) maxima((n - 1) * MPER + q);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// The sweep of one workgroup whose tile has RW row groups, up to its output rows (a single split) or its partial
// state.
template <int D, bool PX, int RW, bool TS>
__device__ __forceinline__ void sweep_tile(const AttnParams& p, const TileJob& jb, TileLds& sh, uint4* ring,
                                           CB_LDS unsigned long long* ts) {
  using Part = PartialLayout<D, 32, PX>;
  using F = Feed<D, 8, 32>;
  constexpr int KW = 8 / RW;             // key groups
  constexpr int NS = F::kSlots, PRO = F::kPrologue;
  constexpr int NPB = PX ? 4 : 2;        // B operands of a unit's probabilities
  // (scores run one stage ahead of the softmax: two stages are resident while a third is requested)
  static_assert(3 * KW <= NS && KW <= PRO, "a stage is requested in full while the one before it is worked on");
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
  const int rw = w % RW, kw = w / RW;
  const int r = l & 31, h = l >> 5;
  const bool do_ts = TS && tid == 0;
#define CB_TS(i) do { if (do_ts) ts[i] = wall_clock64(); } while (0)
  const CB_GLOBAL uint16_t* gq = (const CB_GLOBAL uint16_t*)p.q;
  const int S = jb.S, k0 = jb.k0, k1 = jb.k1;
  F feed(p, jb, sh.bt, ring);
  // Everything the first stages need is requested up front, oldest first: the query rows (to registers), then K/V
  // units (to LDS).
  TileState<D> st;
  int row = jb.row0 + rw * 32 + r;
  const bool has_rows = row - r < jb.M, valid = row < jb.M;
  row = valid ? row : jb.M - 1;
  const int node = row / jb.g, hg = row - node * jb.g;  // tree node of the lane's query (indexes the ancestor sets)
  const int64_t gr = (int64_t)(jb.off + node) * p.Hq + jb.hk * jb.g + hg;
  const int64_t grow = valid ? gr : -1;                 // global output row (node * Hq + head), or -1 past the end
  const CB_GLOBAL uintx4* qp = (const CB_GLOBAL uintx4*)(gq + gr * D);
#pragma unroll
  for (int ds = 0; ds < D / 16; ds++) st.q[ds] = __builtin_bit_cast(bf16x8, load_b128_untracked(qp + 2 * ds + h));
#pragma unroll
  for (int dt = 0; dt < D / 32; dt++)
#pragma unroll
    for (int v = 0; v < 16; v++) st.o[dt][v] = 0.f;
  st.lacc = floatx4{0.f, 0.f, 0.f, 0.f};
  st.mref = -INFINITY;
  st.nm = 0.f;
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

  const int nst = (k1 - k0 + kUnitKeys * KW - 1) / (kUnitKeys * KW);  // stages
  const int nu = nst * KW;                                            // units requested: whole stages
  feed.request_up_to(nu < PRO ? nu : PRO);
  CB_TS(2);
  if (tree_split) build_ancestor_sets(sh.anc, jb.N, my_parent, jump_rounds(p.max_depth));  // uniform in the workgroup; hidden behind the first K/V wait
  feed.wait_units(KW);
#pragma unroll
  for (int ds = 0; ds < D / 16; ds++) asm volatile("" : "+v"(st.q[ds]));  // (older than every unit)
  CB_TS(3);

  auto top = [&](int s) {  // top of stage s: whatever fits is requested while stage s's units are still wanted
    const int want = (s + 2) * KW;
    feed.wait_units(want < nu ? want : nu);
    const int room = s * KW + NS;
    feed.request_up_to(nu < room ? nu : room);
  };
  // this wave's stages whose units are all prefix and all inside the split (rounds down; may be negative: none)
  auto fast_stages = [&] {
    const int n = ((S < k1 ? S : k1) - k0 - kw * kUnitKeys) / (kUnitKeys * KW);
    return nst < n ? nst : n;
  };
  int slot_cur = kw % NS;  // slot of this wave's unit of the current stage
  auto next_slot = [&](int x) { return x + KW >= NS ? x + KW - NS : x + KW; };
  const bf16x8 ones = half_ones(l);

  auto unit_scores = [&](int s, int slot, floatx16& sc) {
    uint4 k[D / 16];
    read_k<D>(feed.k_at(slot), k, l);
    scores<D>(k, st, sc);
    const int key0 = k0 + (s * KW + kw) * kUnitKeys;
    if (key0 + kUnitKeys > S || key0 + kUnitKeys > k1) mask_scores(sc, key0, S, k1, &sh.anc.anc[node][0], h);
  };
  auto add_unit = [&](const bf16x8(&pb)[NPB], int slot) {
    const uint4* vs = feed.v_at(slot);
#pragma unroll
    for (int j = 0; j < NPB; j++) st.lacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pb[j], st.lacc, 0, 0, 0);
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
      for (int dt = 0; dt < D / 32; dt++) {
        const bf16x8 a = read_v<D>(vs, dt, j, l);
#pragma unroll
        for (int x = j; x < NPB; x += 2) st.o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pb[x], st.o[dt], 0, 0, 0);
      }
  };
  auto sweep = [&] {
    floatx16 sc;
    bf16x8 pb[NPB];
    float mx;
    auto check = [&] {
      if (must_raise<D>(st, mx, c2)) raise_reference<D>(st, mx, c2);
    };
    unit_scores(0, slot_cur, sc);
    mx = row_max(sc);
    check();
    int s = 0;
    const int fast_end = fast_stages();
    floatx16 sd;
    uint4 k[D / 16];
    uintx4 pw[NPB];
    bf16x8 v[D / 32];
    if constexpr (KW == 1) {
      // Two steps per barrier, K operands a step ahead in registers, the units' requests spread over the steps (all
      // at once they hold up the wave that makes them).  At the barrier of the pair at s the units up to s + 3 have
      // landed, and everybody is done with those below s.
      const int whole_units = feed.even ? (k1 - k0) / kUnitKeys : 0;
      feed.request_up_to(nu < NS - 2 ? nu : NS - 2);
      if (s + 2 < fast_end) {
        feed.wait_units(s + 4 < nu ? s + 4 : nu);
        read_k<D>(feed.k_at(next_slot(slot_cur)), k, l);
        bool rq = false;
        auto score = [&](const floatx16& from, floatx16& to) {  // of unit s + 1; from: of unit s
          if (p.kv.block_size > 0) feed.bt_ahead(feed.requested);
          int64_t off[F::kParts];  // (worked out here: the paged form's branch would cut the instruction stream)
#pragma unroll
          for (int i = 0; i < F::kParts; i++) off[i] = feed.group_off(feed.requested, i);
          score_half<D, PX, F::kParts>(k, st, from, to, pw, feed.v_at(slot_cur), v, c2, l, [&](int i) { feed.issue_group(feed.slot_next, i, off[i], rq); });
          if (rq) feed.counted();
        };
        auto add = [&](const floatx16& scored) {  // unit s; scored: unit s + 1
          const int nx = next_slot(slot_cur);
          add_half<D, PX, true>(k, feed.k_at(next_slot(nx)), feed.v_at(slot_cur), v, st, pw, scored, mx, ones, l);
          check();
          slot_cur = nx;
          s++;
        };
        while (s + 2 < fast_end) {
          // The pair at s requests two units: in its score halves if both are whole, else here.
          feed.wait_units(s + 4 < nu ? s + 4 : nu);
          rq = feed.requested + 2 <= whole_units && feed.requested + 1 < s + NS;
          if (!rq) feed.request_up_to(nu < s + NS ? nu : s + NS);
          score(sc, sd);
          add(sd);
          score(sd, sc);
          add(sc);
        }
      }
    } else {
      auto step = [&](const floatx16& from, floatx16& to) {
        top(s);
        const int nx = next_slot(slot_cur);
        read_k<D>(feed.k_at(nx), k, l);
        score_half<D, PX, 0>(k, st, from, to, pw, feed.v_at(slot_cur), v, c2, l, [](int) {});
        add_half<D, PX, false>(k, nullptr, feed.v_at(slot_cur), v, st, pw, to, mx, ones, l);
        check();
        slot_cur = nx;
        s++;
      };
      while (s + 2 < fast_end) {  // (two at a time: the scores alternate between two sets of registers)
        step(sc, sd);
        step(sd, sc);
      }
    }
    for (; s + 1 < nst; s++) {
      top(s);
      floatx16 sn;
      unit_scores(s + 1, next_slot(slot_cur), sn);
      probs<D, PX>(sc, st, c2, pb);
      add_unit(pb, slot_cur);
      mx = row_max(sn);
      check();
      sc = sn;
      slot_cur = next_slot(slot_cur);
    }
    probs<D, PX>(sc, st, c2, pb);
    add_unit(pb, slot_cur);
  };
  if (has_rows) sweep();
  else {  // no rows of its own: it only brings its share, passing the same barriers
    int s = 0;
    if constexpr (KW == 1) {
      const int fast_end = fast_stages();
      feed.request_up_to(nu < NS - 2 ? nu : NS - 2);
      if (s + 2 < fast_end) feed.wait_units(s + 4 < nu ? s + 4 : nu);
      for (; s + 2 < fast_end; s += 2) {
        feed.wait_units(s + 4 < nu ? s + 4 : nu);
        feed.request_up_to(nu < s + NS ? nu : s + NS);
      }
    }
    for (; s + 1 < nst; s++) top(s);
  }
  CB_TS(4);

  // With two key groups each finishes one half of the pieces: all park their accumulators and (mref, l) in the
  // ring, then each adds up the groups' for its own pieces.
  constexpr int P = Part::P, PP = P / KW;
  floatx4 f[PP];
  float lsum, mfin;
  auto piece = [&](int pc) {
    return floatx4{st.o[pc >> 2][4 * (pc & 3)], st.o[pc >> 2][4 * (pc & 3) + 1], st.o[pc >> 2][4 * (pc & 3) + 2], st.o[pc >> 2][4 * (pc & 3) + 3]};
  };
  if constexpr (KW > 1) {
    __syncthreads();  // every wave is done with the ring
    floatx4* const park = reinterpret_cast<floatx4*>(ring);
    float2* const park_ml = reinterpret_cast<float2*>(ring + 8 * P * 64);
    static_assert(8 * P * 64 + 8 * 32 <= F::kRingVecs, "");
#pragma unroll
    for (int pc = 0; pc < P; pc++) park[(w * P + pc) * 64 + l] = piece(pc);  // (w = kw * RW + rw)
    park_ml[w * 64 + l] = float2{st.mref, st.lacc[0]};
    __syncthreads();
    float2 ml[KW];
    mfin = -INFINITY;
#pragma unroll
    for (int k = 0; k < KW; k++) {
      ml[k] = park_ml[(k * RW + rw) * 64 + l];
      mfin = fmaxf(mfin, ml[k].x);
    }
    const float mu = (mfin == -INFINITY) ? 0.f : mfin;
    lsum = 0.f;
#pragma unroll
    for (int i = 0; i < PP; i++) f[i] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < KW; k++) {
      const float wt = __builtin_amdgcn_exp2f((ml[k].x - mu) * c2);
      lsum += ml[k].y * wt;
#pragma unroll
      for (int i = 0; i < PP; i++) f[i] += park[((k * RW + rw) * P + kw * PP + i) * 64 + l] * wt;
    }
  } else {
    lsum = st.lacc[0];
    mfin = st.mref;
#pragma unroll
    for (int i = 0; i < PP; i++) f[i] = piece(i);
  }
  write_rows<D, 32, PX, PP>(p, jb, rw, grow, f, kw * PP, mfin, lsum, c2, kw == 0, l);
#undef CB_TS
}

// One attention workgroup of 8 waves whose tile has up to 256 rows; `wg` is its number among those that do attention.
template <int D, bool PX, bool TS>
__device__ __forceinline__ void attn_wide_tile(const AttnParams& p_arg, const SeqMetaLanes& ml, int wg, unsigned long long ts0,
                                               TileLds& sh, uint4* ring, unsigned long long* ts_sh) {
  AttnParams p = p_arg;
  pin_args(p);
  CB_LDS unsigned long long* ts = (CB_LDS unsigned long long*)ts_sh;
  first_stamps<TS>(ts, ts0);
  TileJob jb;
  if (!tile_job(p, ml, wg, 256, jb)) return;
  if (jb.M - jb.row0 <= 128) sweep_tile<D, PX, 4, TS>(p, jb, sh, ring, ts);
  else sweep_tile<D, PX, 8, TS>(p, jb, sh, ring, ts);
  if (jb.nsplit == 1 || p.external_merge) return;  // (a following kernel merges: the kernel boundary orders the stores)
  split_merge<D, 32, PX, 8, 256, TS>(p, jb, sh, ts);
}

template <int D, bool PX, bool TS>
__global__ __launch_bounds__(512) void k_attn_wide(AttnParams p, SeqMeta meta) {
  const unsigned long long ts0 = TS ? wall_clock64() : 0ull;
  const SeqMetaLanes ml = seq_meta_prefetch(meta);
  __shared__ uint4 ring[Feed<D, 8, 32>::kRingVecs];
  __shared__ TileLds sh;
  __shared__ unsigned long long ts_sh[TS ? 16 : 1];
  attn_wide_tile<D, PX, TS>(p, ml, blockIdx.x, ts0, sh, ring, ts_sh);
  flush_timestamps<TS>(p, blockIdx.x, ts_sh);
}

// The whole verification in one launch, as k_verify_mfma does it for small tiles: the first lw.n_wgs workgroups do the
// logits work, the others the attention.
template <int D, bool PX, bool TS>
__global__ __launch_bounds__(512) void k_verify_wide(AttnParams p, SeqMeta meta, LogitsWork lw) {
  const unsigned long long ts0 = TS ? wall_clock64() : 0ull;
  const SeqMetaLanes ml = seq_meta_prefetch(meta);
  __shared__ uint4 ring[Feed<D, 8, 32>::kRingVecs];
  __shared__ TileLds sh;
  __shared__ unsigned long long ts_sh[TS ? 16 : 1];
  static_assert(sizeof(ring) >= sizeof(AcceptWaveLds), "the acceptance's LDS is the ring's");
  const int wg = (int)blockIdx.x - lw.n_wgs;
  if (wg < 0) {
    logits_share<8, 16>(lw, ml, blockIdx.x, *reinterpret_cast<AcceptWaveLds*>(ring));
    return;
  }
  attn_wide_tile<D, PX, TS>(p, ml, wg, ts0, sh, ring, ts_sh);
  flush_timestamps<TS>(p, wg, ts_sh);
}

hipError_t launch_attn_wide(hipStream_t st, const AttnParams& p, const SeqMeta& meta, int n_tiles, const LogitsWork* lw) {
  const dim3 grid(n_tiles + (lw ? lw->n_wgs : 0)), block(512);
#define CB_LAUNCH(D, PX)                                                                                        \
  do {                                                                                                          \
    if (lw && p.timeline) hipLaunchKernelGGL((k_verify_wide<D, PX, true>), grid, block, 0, st, p, meta, *lw);   \
    else if (lw) hipLaunchKernelGGL((k_verify_wide<D, PX, false>), grid, block, 0, st, p, meta, *lw);           \
    else if (p.timeline) hipLaunchKernelGGL((k_attn_wide<D, PX, true>), grid, block, 0, st, p, meta);           \
    else hipLaunchKernelGGL((k_attn_wide<D, PX, false>), grid, block, 0, st, p, meta);                          \
  } while (0)
  if (p.D == 64) CB_LAUNCH(64, true);
  else if (p.precise) CB_LAUNCH(128, true);
  else CB_LAUNCH(128, false);
#undef CB_LAUNCH
  return hipGetLastError();
}

}  // namespace cb
