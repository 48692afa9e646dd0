// Tree attention for tiles of 65 to 256 rows (bf16, head_dim 64 or 128), gfx950 only.
//
// A tile's rows decide how the 8 waves share it: RW row groups of 32 * NVM rows times KW = 8 / RW key groups (two key
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

template <int D, int NVM>
struct TileState {
  bf16x8 q[NVM][D / 16];     // B operands of QK^T: query r, dims 16 ds + 8h ..
  floatx16 o[NVM][D / 32];   // O^T accumulators, dim tiles of 32
  floatx4 lacc[NVM];         // softmax denominator of the lane's query (all four elements equal)
  float mref[NVM];           // reference maximum of the raw scores (q.k, before the softmax scale)
  float nm[NVM];             // -mref in log2 units (0 while mref is -inf)
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
template <int D, int NV>
__device__ __forceinline__ void read_k(const uint4* ks, uint4 (&k)[D / 16], int l) {
#pragma unroll
  for (int ds = 0; ds < D / 16; ds++) k[ds] = read_k1<D>(ks, ds, l);
}
// scores of a unit: S^T = K Q^T
template <int D, int NVM, int NV>
__device__ __forceinline__ void scores(const uint4 (&k)[D / 16], const TileState<D, NVM>& st, floatx16 (&s)[NV]) {
#pragma unroll
  for (int t = 0; t < NV; t++)
#pragma unroll
    for (int v = 0; v < 16; v++) s[t][v] = 0.f;
#pragma unroll
  for (int ds = 0; ds < D / 16; ds++)
#pragma unroll
    for (int t = 0; t < NV; t++)
      s[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, k[ds]), st.q[t][ds], s[t], 0, 0, 0);
}
// probabilities p = 2^(c*s - c*mref), packed as B operands of PV; with PX the roundings' rests behind them
template <int D, int NVM, int NV, bool PX>
__device__ __forceinline__ void probs(const floatx16& s, const TileState<D, NVM>& st, int t, float c2, bf16x8 (&p)[PX ? 4 : 2]) {
  const float nm = st.nm[t];
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

template <int NV>
__device__ __forceinline__ void row_max(const floatx16 (&s)[NV], float (&mx)[NV]) {
#pragma unroll
  for (int t = 0; t < NV; t++) {
    float m = maxn(maxn(s[t][0], s[t][1]), s[t][2]);
#pragma unroll
    for (int v = 3; v < 15; v += 2) m = maxn(maxn(m, s[t][v]), s[t][v + 1]);
    mx[t] = half_swap_max(maxn(m, s[t][15]));
  }
}
// Lazy reference: it is only raised (and O, l rescaled) when the maximum has grown by more than kRescaleSlack, so
// probabilities stay below 2^8 and the accumulators are rarely touched by the vector ALU.
template <int NVM, int NV, typename State>
__device__ __forceinline__ bool must_raise(const State& st, const float (&mx)[NV], float c2) {  // uniform
  bool any = false;
#pragma unroll
  for (int t = 0; t < NV; t++) any |= (mx[t] - st.mref[t]) * c2 > kRescaleSlack;  // false when both are -inf (NaN)
  return __builtin_amdgcn_ballot_w64(any) != 0ull;
}
template <int D, int NVM, int NV>
__device__ __forceinline__ void raise_reference(TileState<D, NVM>& st, const float (&mx)[NV], float c2) {
#pragma unroll
  for (int t = 0; t < NV; t++) {
    const bool raise = (mx[t] - st.mref[t]) * c2 > kRescaleSlack;
    const float alpha = raise ? __builtin_amdgcn_exp2f((st.mref[t] - mx[t]) * c2) : 1.0f;
    if (raise) {
      st.mref[t] = mx[t];
      st.nm[t] = -mx[t] * c2;
    }
#pragma unroll
    for (int dt = 0; dt < D / 32; dt++) st.o[t][dt] *= alpha;
    st.lacc[t] *= alpha;
  }
}

// One steady step of a wave, in two halves: score_half scores a unit (its K operands in `k`, scores to sn) while the
// unit scored before it (sc) is exponentiated (to pb), add_half adds that unit's values (at vs) up while the maxima of sn
// are taken (to mx).  Written in issue order, pinned by the scheduling barriers: an MFMA occupies the matrix core for 32
// cycles in which the wave issues what belongs to the other unit (a v_exp_f32 takes 8 cycles, other vector
// instructions 4 to 5).  Left alone the compiler gathers each kind.
// score_half ends with the reads of add_half's first operands (v).  req(i), i = 0 .. NREQ - 1: memory requests to be
// spread over score_half.
// PREK: `k` is filled again in add_half, for the next score_half (its unit's K at kn).
template <int D, int NVM, int NV, bool PX, int NREQ, typename Req>
__device__ __forceinline__ void score_half(const uint4 (&k)[D / 16], const TileState<D, NVM>& st, const floatx16 (&sc)[NV], floatx16 (&sn)[NV],
                                           uintx4 (&pb)[NV][PX ? 4 : 2], const uint4* vs, bf16x8 (&v)[D / 32], float c2, int l, Req req) {
  constexpr int DS = D / 16, DT = D / 32;
  // The probabilities in three stages, each a slot behind the one before it, so that no instruction waits for the one
  // in front of it: argument, exponential, packing.  Slot i handles elements 2 i and 2 i + 1 (constant indices).
  constexpr int NP2 = 8 * NV;
  float x0[NP2], x1[NP2];
  auto arg = [&](int i) {
    if (i >= NP2) return;
    const int t = i >> 3, x = 2 * (i & 7);
    x0[i] = fmaf(sc[t][x], c2, st.nm[t]);
    x1[i] = fmaf(sc[t][x + 1], c2, st.nm[t]);
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
    pb[i >> 3][(i & 7) >> 2][i & 3] = z;
    if constexpr (PX) {
      const float r0 = x0[i] - __uint_as_float(z << 16), r1 = x1[i] - __uint_as_float(z & 0xffff0000u);
      uint32_t y = __builtin_bit_cast(uint32_t, __builtin_convertvector((float2v){r0, r1}, bf16x2v));
      asm volatile("" : "+v"(y));
      pb[i >> 3][2 + ((i & 7) >> 2)][i & 3] = y;
    }
  };
  arg(0);
  arg(1);
  expo(0);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int t = 0; t < NV; t++)
#pragma unroll
    for (int x = 0; x < 16; x++) sn[t][x] = 0.f;
  constexpr int PER = 8 / DS;  // slots per MFMA
#pragma unroll
  for (int ds = 0; ds < DS; ds++) {
#pragma unroll
    for (int t = 0; t < NV; t++) {
      sn[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, k[ds]), st.q[t][ds], sn[t], 0, 0, 0);
#pragma unroll
      for (int q = 0; q < PER; q++) {
        const int i = (ds * NV + t) * PER + q;
        expo(i + 1);
        pack(i);
        arg(i + 2);
      }
      if (t == 0 && ds >= DS - DT) v[ds - (DS - DT)] = read_v<D>(vs, ds - (DS - DT), 0, l);
      if (NREQ > 0 && t == NV - 1 && ds % (DS / (NREQ > 0 ? NREQ : 1)) == 0) req(ds / (DS / (NREQ > 0 ? NREQ : 1)));
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}
template <int D, int NVM, int NV, bool PX, bool PREK>
__device__ __forceinline__ void add_half(uint4 (&k)[D / 16], const uint4* kn, const uint4* vs, bf16x8 (&v)[D / 32], TileState<D, NVM>& st,
                                         const uintx4 (&pb)[NV][PX ? 4 : 2], const floatx16 (&sn)[NV], float (&mx)[NV], const bf16x8& ones, int l) {
  constexpr int DS = D / 16, DT = D / 32;
  // the maxima of the new scores, then across the lanes, a few beside every MFMA from the second on
  float m[NV];
  auto maxima = [&](int i) {  // (constant index)
    if (i < 0 || i >= 10 * NV) return;
    const int mt = i / 10, mi = i % 10;
    if (mi == 0) m[mt] = maxn(maxn(sn[mt][0], sn[mt][1]), sn[mt][2]);
    else if (mi < 7) m[mt] = maxn(maxn(m[mt], sn[mt][2 * mi + 1]), sn[mt][2 * mi + 2]);
    else if (mi == 7) m[mt] = maxn(m[mt], sn[mt][15]);
    else if (mi == 8) mx[mt] = half_swap_max(m[mt]);
    if (mi < 8) asm volatile("" : "+v"(m[mt]));
    else asm volatile("" : "+v"(mx[mt]));
  };
  constexpr int NPV = 2 * DT * NV;                        // PV MFMAs
  constexpr int MPER = (10 * NV + NPV - 3) / (NPV - 2);   // maxima per MFMA
#pragma unroll
  for (int j = 0; j < 2; j++) {
#pragma unroll
    for (int dt = 0; dt < DT; dt++) {
#pragma unroll
      for (int t = 0; t < NV; t++) {
        const int n = (j * DT + dt) * NV + t;
        st.o[t][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v[dt], __builtin_bit_cast(bf16x8, pb[t][j]), st.o[t][dt], 0, 0, 0);
        if constexpr (PX)
          st.o[t][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v[dt], __builtin_bit_cast(bf16x8, pb[t][2 + j]), st.o[t][dt], 0, 0, 0);
        if (t == NV - 1) {  // (the operand's registers take the next thing from LDS)
          if (j == 0) v[dt] = read_v<D>(vs, dt, 1, l);
          else if (PREK) {
#pragma unroll
            for (int q = 0; q < DS / DT; q++) k[dt * (DS / DT) + q] = read_k1<D>(kn, dt * (DS / DT) + q, l);
          }
        }
        if (dt == DT - 1) {
#pragma unroll
          for (int x = j; x < (PX ? 4 : 2); x += 2)
            st.lacc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, __builtin_bit_cast(bf16x8, pb[t][x]), st.lacc[t], 0, 0, 0);
        }
#pragma unroll
        for (int q = 0; q < MPER; q++) maxima((n - 1) * MPER + q);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
}

// The sweep of one workgroup whose tile has RW row groups, up to its output rows (a single split) or its partial
// state.
template <int D, bool PX, int NW, int NVM, int RW, bool TS>
__device__ __forceinline__ void sweep_tile(const AttnParams& p, const TileJob& jb, TileLds& sh, uint4* ring,
                                           CB_LDS unsigned long long* ts) {
  using Part = PartialLayout<D, 32, PX>;
  using F = Feed<D, NW, 32>;
  constexpr int KW = NW / RW;            // key groups
  constexpr int NS = F::kSlots, PRO = F::kPrologue;
  constexpr int NPB = PX ? 4 : 2;        // B operands of a unit's probabilities
  constexpr int LA = KW <= 2 ? 1 : 0;    // scores run one stage ahead of the softmax (needs two stages resident)
  static_assert((LA + 2) * KW <= NS && KW <= PRO, "a stage is requested in full while the one before it is worked on");
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
  TileState<D, NVM> st;
  int row_node[NVM];    // tree node of the lane's query (indexes the ancestor sets)
  int64_t grow[NVM];    // global output row (node * Hq + head), or -1 past the end
  int nvt = 0;          // this wave's row tiles that hold at least one real row (they come first)
#pragma unroll
  for (int t = 0; t < NVM; t++) {
    const int rl = (rw * NVM + t) * 32 + r;
    if (jb.row0 + rl - r < jb.M) nvt = t + 1;
    int row = jb.row0 + rl;
    const bool valid = row < jb.M;
    row = valid ? row : jb.M - 1;
    const int node = row / jb.g, hg = row - node * jb.g;
    row_node[t] = node;
    const int64_t gr = (int64_t)(jb.off + node) * p.Hq + jb.hk * jb.g + hg;
    grow[t] = valid ? gr : -1;
    const CB_GLOBAL uintx4* qp = (const CB_GLOBAL uintx4*)(gq + gr * D);
#pragma unroll
    for (int ds = 0; ds < D / 16; ds++) st.q[t][ds] = __builtin_bit_cast(bf16x8, load_b128_untracked(qp + 2 * ds + h));
#pragma unroll
    for (int dt = 0; dt < D / 32; dt++)
#pragma unroll
      for (int v = 0; v < 16; v++) st.o[t][dt][v] = 0.f;
    st.lacc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
    st.mref[t] = -INFINITY;
    st.nm[t] = 0.f;
  }
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
  for (int t = 0; t < NVM; t++)
#pragma unroll
    for (int ds = 0; ds < D / 16; ds++) asm volatile("" : "+v"(st.q[t][ds]));  // (older than every unit)
  CB_TS(3);

  auto top = [&](int s) {  // top of stage s: whatever fits is requested while stage s's units are still wanted
    const int want = (s + 1 + LA) * KW;
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

  auto sweep = [&](auto nvc) {
    constexpr int NV = decltype(nvc)::value;
    auto unit_scores = [&](int s, int slot, floatx16(&sc)[NV]) {
      uint4 k[D / 16];
      read_k<D, NV>(feed.k_at(slot), k, l);
      scores<D, NVM, NV>(k, st, sc);
      const int key0 = k0 + (s * KW + kw) * kUnitKeys;
      if (key0 + kUnitKeys > S || key0 + kUnitKeys > k1) {
#pragma unroll
        for (int t = 0; t < NV; t++) mask_scores(sc[t], key0, S, k1, &sh.anc.anc[row_node[t]][0], h);
      }
    };
    auto add_unit = [&](const bf16x8(&pb)[NV][NPB], int slot) {
      const uint4* vs = feed.v_at(slot);
#pragma unroll
      for (int t = 0; t < NV; t++)
#pragma unroll
        for (int j = 0; j < NPB; j++) st.lacc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pb[t][j], st.lacc[t], 0, 0, 0);
#pragma unroll
      for (int j = 0; j < 2; j++)
#pragma unroll
        for (int dt = 0; dt < D / 32; dt++) {
          const bf16x8 a = read_v<D>(vs, dt, j, l);
#pragma unroll
          for (int t = 0; t < NV; t++)
#pragma unroll
            for (int x = j; x < NPB; x += 2)
              st.o[t][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pb[t][x], st.o[t][dt], 0, 0, 0);
        }
    };
    floatx16 sc[NV];
    float mx[NV];
    bf16x8 pb[NV][NPB];
    if constexpr (LA == 0) {
      for (int s = 0; s < nst; s++) {
        top(s);
        unit_scores(s, slot_cur, sc);
        row_max<NV>(sc, mx);
        if (must_raise<NVM, NV>(st, mx, c2)) raise_reference<D, NVM, NV>(st, mx, c2);
#pragma unroll
        for (int t = 0; t < NV; t++) probs<D, NVM, NV, PX>(sc[t], st, t, c2, pb[t]);
        add_unit(pb, slot_cur);
        slot_cur = next_slot(slot_cur);
      }
    } else {
      unit_scores(0, slot_cur, sc);
      row_max<NV>(sc, mx);
      if (must_raise<NVM, NV>(st, mx, c2)) raise_reference<D, NVM, NV>(st, mx, c2);
      int s = 0;
      const int fast_end = fast_stages();
      floatx16 sd[NV];
      uint4 k[D / 16];
      uintx4 pw[NV][NPB];
      bf16x8 v[D / 32];
      auto check = [&] {
        if (must_raise<NVM, NV>(st, mx, c2)) raise_reference<D, NVM, NV>(st, mx, c2);
      };
      if constexpr (KW == 1) {
        // Two steps per barrier, K operands a step ahead in registers, the units' requests spread over the steps (all
        // at once they hold up the wave that makes them).  At the barrier of the pair at s the units up to s + 3 have
        // landed, and everybody is done with those below s.
        const int whole_units = feed.even ? (k1 - k0) / kUnitKeys : 0;
        feed.request_up_to(nu < NS - 2 ? nu : NS - 2);
        if (s + 2 < fast_end) {
          feed.wait_units(s + 4 < nu ? s + 4 : nu);
          read_k<D, NV>(feed.k_at(next_slot(slot_cur)), k, l);
          bool rq = false;
          auto score = [&](const floatx16(&from)[NV], floatx16(&to)[NV]) {  // of unit s + 1; from: of unit s
            if (p.kv.block_size > 0) feed.bt_ahead(feed.requested);
            int64_t off[F::kParts];  // (worked out here: the paged form's branch would cut the instruction stream)
#pragma unroll
            for (int i = 0; i < F::kParts; i++) off[i] = feed.group_off(feed.requested, i);
            score_half<D, NVM, NV, PX, F::kParts>(k, st, from, to, pw, feed.v_at(slot_cur), v, c2, l, [&](int i) { feed.issue_group(feed.slot_next, i, off[i], rq); });
            if (rq) feed.counted();
          };
          auto add = [&](const floatx16(&scored)[NV]) {  // unit s; scored: unit s + 1
            const int nx = next_slot(slot_cur);
            add_half<D, NVM, NV, PX, true>(k, feed.k_at(next_slot(nx)), feed.v_at(slot_cur), v, st, pw, scored, mx, ones, l);
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
        auto step = [&](const floatx16(&from)[NV], floatx16(&to)[NV]) {
          top(s);
          const int nx = next_slot(slot_cur);
          read_k<D, NV>(feed.k_at(nx), k, l);
          score_half<D, NVM, NV, PX, 0>(k, st, from, to, pw, feed.v_at(slot_cur), v, c2, l, [](int) {});
          add_half<D, NVM, NV, PX, false>(k, nullptr, feed.v_at(slot_cur), v, st, pw, to, mx, ones, l);
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
        floatx16 sn[NV];
        unit_scores(s + 1, next_slot(slot_cur), sn);
#pragma unroll
        for (int t = 0; t < NV; t++) probs<D, NVM, NV, PX>(sc[t], st, t, c2, pb[t]);
        add_unit(pb, slot_cur);
        row_max<NV>(sn, mx);
        if (must_raise<NVM, NV>(st, mx, c2)) raise_reference<D, NVM, NV>(st, mx, c2);
#pragma unroll
        for (int t = 0; t < NV; t++) sc[t] = sn[t];
        slot_cur = next_slot(slot_cur);
      }
#pragma unroll
      for (int t = 0; t < NV; t++) probs<D, NVM, NV, PX>(sc[t], st, t, c2, pb[t]);
      add_unit(pb, slot_cur);
    }
  };
  if (nvt == NVM) sweep(std::integral_constant<int, NVM>{});
  else if (NVM > 1 && nvt > 0) sweep(std::integral_constant<int, 1>{});
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
    for (; s + LA < nst; s++) top(s);
  }
  CB_TS(4);

  // With several key groups each finishes its share of the pieces: all park their accumulators and (mref, l) in the
  // ring, then each adds up the groups' for its own pieces.
  constexpr int P = Part::P, PP = P / KW;
  floatx4 f[NVM][PP];
  float lsum[NVM], mfin[NVM];
  if constexpr (KW > 1) {
    __syncthreads();  // every wave is done with the ring
    floatx4* const park = reinterpret_cast<floatx4*>(ring);
    float2* const park_ml = reinterpret_cast<float2*>(ring + NW * NVM * P * 64);
    static_assert(NW * NVM * P * 64 + NW * NVM * 32 <= F::kRingVecs, "");
#pragma unroll
    for (int t = 0; t < NVM; t++) {
      const int blk = (kw * RW + rw) * NVM + t;
#pragma unroll
      for (int pc = 0; pc < P; pc++)
        park[(blk * P + pc) * 64 + l] = floatx4{st.o[t][pc >> 2][4 * (pc & 3)], st.o[t][pc >> 2][4 * (pc & 3) + 1],
                                                st.o[t][pc >> 2][4 * (pc & 3) + 2], st.o[t][pc >> 2][4 * (pc & 3) + 3]};
      park_ml[blk * 64 + l] = float2{st.mref[t], st.lacc[t][0]};
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < NVM; t++) {
      float2 ml[KW];
      float m = -INFINITY;
#pragma unroll
      for (int k = 0; k < KW; k++) {
        ml[k] = park_ml[((k * RW + rw) * NVM + t) * 64 + l];
        m = fmaxf(m, ml[k].x);
      }
      const float mu = (m == -INFINITY) ? 0.f : m;
      lsum[t] = 0.f;
      mfin[t] = m;
#pragma unroll
      for (int i = 0; i < PP; i++) f[t][i] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < KW; k++) {
        const float wt = __builtin_amdgcn_exp2f((ml[k].x - mu) * c2);
        lsum[t] += ml[k].y * wt;
#pragma unroll
        for (int i = 0; i < PP; i++) f[t][i] += park[((((k * RW + rw) * NVM + t) * P) + kw * PP + i) * 64 + l] * wt;
      }
    }
  } else {
#pragma unroll
    for (int t = 0; t < NVM; t++) {
      lsum[t] = st.lacc[t][0];
      mfin[t] = st.mref[t];
#pragma unroll
      for (int i = 0; i < PP; i++)
        f[t][i] = floatx4{st.o[t][i >> 2][4 * (i & 3)], st.o[t][i >> 2][4 * (i & 3) + 1], st.o[t][i >> 2][4 * (i & 3) + 2], st.o[t][i >> 2][4 * (i & 3) + 3]};
    }
  }
#pragma unroll
  for (int t = 0; t < NVM; t++) write_rows<D, 32, PX, PP>(p, jb, rw * NVM + t, grow[t], f[t], kw * PP, mfin[t], lsum[t], c2, kw == 0, l);
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
  if (jb.M - jb.row0 <= 128) sweep_tile<D, PX, 8, 1, 4, TS>(p, jb, sh, ring, ts);
  else sweep_tile<D, PX, 8, 1, 8, TS>(p, jb, sh, ring, ts);
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

hipError_t launch_attn_wide(hipStream_t st, const AttnParams& p, const SeqMeta& meta, int n_tiles) {
  const dim3 grid(n_tiles), block(512);
#define CB_LAUNCH(D, PX)                                                                              \
  do {                                                                                                \
    if (p.timeline) hipLaunchKernelGGL((k_attn_wide<D, PX, true>), grid, block, 0, st, p, meta);      \
    else hipLaunchKernelGGL((k_attn_wide<D, PX, false>), grid, block, 0, st, p, meta);                \
  } while (0)
  if (p.D == 64) CB_LAUNCH(64, true);
  else if (p.precise) CB_LAUNCH(128, true);
  else CB_LAUNCH(128, false);
#undef CB_LAUNCH
  return hipGetLastError();
}

}  // namespace cb
