// Tree attention for tiles of 65 to 256 rows (bf16, head_dim 64 or 128), gfx950 only: the kernels, which cb_attn_wide.hip builds with
// bf16 probabilities and partial sums and cb_attn_wide_px.hip with 32-bit ones.
//
// Four waves, one to a SIMD, with 32 or 64 rows each.  A tile's rows decide how they share it: RW row groups times KW = 4 / RW
// key groups -- up to 64 rows two groups of one 32-row tile with two key groups, up to 128 four of one tile (or, see below, two of
// two), beyond four of two tiles.  A unit of work is 32 keys; a stage is KW units, one for each key group, whose softmax states are
// combined through LDS at the end.
//
// What bounds it: per unit of a 256-row tile the matrix cores have 1088 cycles of work; a wave issues 129 vector, 24 LDS and 22 scalar
// instructions beside it (the exponentials twice as long as the others), and takes 1870 with barrier, requests and
// waits, launch and tail included.  K and V operands serve two row tiles each: with eight waves of 32 rows (two to a SIMD) the LDS had 128 KiB of
// operand reads to deliver per unit, 1024 cycles, and the SIMDs twice the scalar and address instructions: 1890 cycles.
// Under long sweeps the chip's clock comes down (1.75 GHz of 2.4 at 40 heads x 65536 keys x 256 nodes: 641 k cycles a wave in 367
// us), so that work taken out counts there and stalls taken out do not.
// A pass with eight waves and with four: 128 nodes x 8192 keys of 32/8 heads 31.8 -> 31.3 us, 8 sequences of up to 2000 keys
// 42.6 -> 40.2, 16 paged sequences of up to 16384 keys, 32-bit sums, 629 -> 590, 256 nodes x 65536 keys of 40 heads 406 -> 383.
//
// Register layouts (v_mfma_f32_32x32x16_bf16; lane l, r = l % 32, h = l / 32):
//   scores are computed transposed, S^T = K Q^T: A = K rows (key r, dims 8h..8h+7 of the 16-dim step), B = Q^T
//   (query r, same dims), D[v] = S^T[key 8(v/4)+4h+v%4][query r].  A lane therefore holds 16 keys x 1 query:
//   softmax statistics are per-lane scalars shared by the 2 lanes with equal r.
//   O^T = V^T P^T: B = P^T packs the lane's 8 probabilities of a 16-key step j (element e <-> key
//   16j + 8(e/4) + 4h + e%4, which is what D holds), A = V^T must hold the same keys for dim r of the 32-dim
//   tile; it is fetched from the row-major V tile with ds_read_b64_tr_b16 (each 16-lane group reads a 4-key x
//   16-dim block and receives it transposed).  D[v] = O^T[dim 8(v/4)+4h+v%4][query r].
#pragma once
#include "cb_attn_tile.h"

namespace cb {

constexpr int kWideWaves = 4;

template <int D>
struct TileState {      // of one row tile of 32 rows
  bf16x8 q[D / 16];     // B operands of QK^T: query r, dims 16 ds + 8h ..
  floatx16 o[D / 32];   // O^T accumulators, dim tiles of 32
  floatx4 lacc;         // softmax denominator of the lane's query (all four elements equal)
  float mref;           // reference maximum of the raw scores (q.k, before the softmax scale)
  float top;            // the maximum up to which it stays
  float nm;             // -mref in log2 units (0 while mref is -inf)
};

__device__ __forceinline__ float half_swap_max(float x) {  // maximum over lanes l and l ^ 32
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return maxn(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// A lane's reads of a unit are at constant places from one address (a place in the ring plus what depends on the lane): the
// swizzles are XORs of bits that neither the row nor the place in the ring reaches, so a 16-byte piece further is the
// address XORed with a constant.
template <int D>
__device__ __forceinline__ uint32_t lane_k_byte(int l) {
  const int r = l & 31, h = l >> 5;
  return r * (2 * D) + ((h ^ swizzle_k<D>(r)) << 4);
}
template <int D>
__device__ __forceinline__ uint4 read_k1(uint32_t ka, int ds) {
  return __builtin_bit_cast(uint4, *(const CB_LDS uintx4*)(ka ^ (ds << 5)));
}
template <int D>
__device__ __forceinline__ void read_k(uint32_t ka, uint4 (&k)[D / 16]) {
#pragma unroll
  for (int ds = 0; ds < D / 16; ds++) k[ds] = read_k1<D>(ka, ds);
}
// scores of a unit: S^T = K Q^T
template <int D, int R>
__device__ __forceinline__ void scores(const uint4 (&k)[D / 16], const TileState<D> (&st)[R], floatx16 (&s)[R]) {
#pragma unroll
  for (int ds = 0; ds < D / 16; ds++)
#pragma unroll
    for (int t = 0; t < R; t++) {
      const floatx16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      s[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, k[ds]), st[t].q[ds], ds ? s[t] : zero, 0, 0, 0);
    }
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
__device__ __forceinline__ uint32_t lane_v_byte(int l) {
  const int c = l & 15, h = l >> 5, dh = (l >> 4) & 1, row = 4 * h + (c >> 2);
  return row * (2 * D) + (((2 * dh + ((c & 3) >> 1)) ^ swizzle_v<D, 32>(row)) << 4) + (c & 1) * 8;
}
template <int D>
__device__ __forceinline__ bf16x8 read_v(uint32_t va, int dt, int j) {
  bf16x4 x[2];
#pragma unroll
  for (int u = 0; u < 2; u++)
    x[u] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((CB_LDS bf16x4*)((va ^ (dt << 6)) + (16 * j + 8 * u) * (2 * D)));
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
__device__ __forceinline__ void raise_reference(TileState<D>& st, float mx, float c2) {
  const bool raise = mx > st.top;
  const float alpha = raise ? __builtin_amdgcn_exp2f((st.mref - mx) * c2) : 1.0f;
  if (raise) {
    st.mref = mx;
    st.top = mx + kRescaleSlack / c2;
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
// score_half also reads add_half's first operands (v), in front of its middle.  req(i), i = 0 .. NREQ - 1: memory requests to be
// spread over score_half.
// PREK: `k` is filled again in add_half, for the next score_half (its unit's K at kn).
template <int D, bool PX, int R, int NREQ, typename Req>
__device__ __forceinline__ void score_half(const uint4 (&k)[D / 16], const TileState<D> (&st)[R], const floatx16 (&sc)[R], floatx16 (&sn)[R],
                                           uintx4 (&pb)[R][PX ? 4 : 2], uint32_t va, bf16x8 (&v)[D / 32], float c2, Req req) {
  constexpr int DS = D / 16, DT = D / 32;
  // The probabilities in three stages, each a slot behind the one before it, so that no instruction waits for the one
  // in front of it: argument, exponential, packing.  Slot i handles elements 2 i and 2 i + 1 of tile i / 8 (constant indices).
  constexpr int NP2 = 8 * R;
  float x0[NP2], x1[NP2];
  auto arg = [&](int i) {
    if (i >= NP2) return;
    x0[i] = fmaf(sc[i / 8][2 * (i % 8)], c2, st[i / 8].nm);
    x1[i] = fmaf(sc[i / 8][2 * (i % 8) + 1], c2, st[i / 8].nm);
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
    const int t = i / 8, e = i % 8;
    pb[t][e >> 2][e & 3] = z;
    if constexpr (PX) {
      const float r0 = x0[i] - __uint_as_float(z << 16), r1 = x1[i] - __uint_as_float(z & 0xffff0000u);
      uint32_t y = __builtin_bit_cast(uint32_t, __builtin_convertvector((float2v){r0, r1}, bf16x2v));
      asm volatile("" : "+v"(y));
      pb[t][2 + (e >> 2)][e & 3] = y;
    }
  };
  arg(0);
  arg(1);
  expo(0);
  __builtin_amdgcn_sched_barrier(0);
  constexpr int PER = 8 / DS;  // slots per MFMA
  constexpr int NM = DS * R;   // MFMAs
#pragma unroll
  for (int n = 0; n < NM; n++) {
    const int ds = n / R, t = n % R;
    const floatx16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    sn[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, k[ds]), st[t].q[ds], ds ? sn[t] : zero, 0, 0, 0);
#pragma unroll
    for (int q = 0; q < PER; q++) {
      const int i = n * PER + q;
      expo(i + 1);
      pack(i);
      arg(i + 2);
    }
    if (n >= NM / 2 - DT && n < NM / 2) v[n - (NM / 2 - DT)] = read_v<D>(va, n - (NM / 2 - DT), 0);
    if (NREQ > 0 && n % (NM / (NREQ > 0 ? NREQ : 1)) == 0) req(n / (NM / (NREQ > 0 ? NREQ : 1)));
    __builtin_amdgcn_sched_barrier(0);
  }
}
template <int D, bool PX, int R, bool PREK>
__device__ __forceinline__ void add_half(uint4 (&k)[D / 16], uint32_t kn, uint32_t va, bf16x8 (&v)[D / 32], TileState<D> (&st)[R],
                                         const uintx4 (&pb)[R][PX ? 4 : 2], const floatx16 (&sn)[R], float (&mx)[R], const bf16x8& ones) {
  constexpr int DS = D / 16, DT = D / 32;
  // the maxima of the new scores, then across the lanes, a few beside every MFMA from the second on
  float m[R];
  auto maxima = [&](int i) {  // (constant index)
    if (i < 0 || i >= 10 * R) return;
    const int t = i / 10, e = i % 10;
    if (e == 0) m[t] = maxn(maxn(sn[t][0], sn[t][1]), sn[t][2]);
    else if (e < 7) m[t] = maxn(maxn(m[t], sn[t][2 * e + 1]), sn[t][2 * e + 2]);
    else if (e == 7) m[t] = maxn(m[t], sn[t][15]);
    else if (e == 8) mx[t] = half_swap_max(m[t]);
    if (e < 8) asm volatile("" : "+v"(m[t]));
    else asm volatile("" : "+v"(mx[t]));
  };
  constexpr int NPV = 2 * DT * R;                        // PV MFMAs
  constexpr int MPER = (10 * R + NPV - 3) / (NPV - 2);   // maxima per MFMA
#pragma unroll
  for (int n = 0; n < NPV; n++) {
    const int j = n / (DT * R), dt = n / R % DT, t = n % R;
    st[t].o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v[dt], __builtin_bit_cast(bf16x8, pb[t][j]), st[t].o[dt], 0, 0, 0);
    if constexpr (PX) st[t].o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v[dt], __builtin_bit_cast(bf16x8, pb[t][2 + j]), st[t].o[dt], 0, 0, 0);
    // (the operand's registers take the next thing from LDS)
    if (t == R - 1) {
      if (j == 0) v[dt] = read_v<D>(va, dt, 1);
      else if (PREK) {
#pragma unroll
        for (int q = 0; q < DS / DT; q++) k[dt * (DS / DT) + q] = read_k1<D>(kn, dt * (DS / DT) + q);
      }
    }
    if (dt == DT - 1) {
#pragma unroll
      for (int x = j; x < (PX ? 4 : 2); x += 2)
        st[t].lacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, __builtin_bit_cast(bf16x8, pb[t][x]), st[t].lacc, 0, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < MPER; q++) maxima((n - 1) * MPER + q);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// The memory side of the wide sweep.  A wavefront has its SIMD to itself here, so every instruction beside the arithmetic
// costs its four cycles in full: the ring's waits are constants and the addresses a few vector instructions.  For that,
// every barrier is followed by as many requests as units were finished in front of it, also when the split has no more:
// keys past its end are its last one, in the last unit too, so such a request brings one row and nobody reads it.
template <int D, bool PG>
struct WideFeed {
  using F = Feed<D, kWideWaves, 32>;
  static constexpr int NS = F::kSlots, P = F::kParts, RPR = F::RPR;
  static_assert(F::kReq == 2 * P, "a group is a request for K and one for V");
  F& f;
  int key[P];                      // the lane's row in the next unit's groups, at most the split's last key
  const int last;
  const CB_GLOBAL char *kb[P], *vb[P];   // what the row's offset is added to
  uint32_t place = 0;              // of the next unit in the ring, bytes
  int blk[P];                      // paged: the rows' entries of the block table
  __device__ __forceinline__ explicit WideFeed(F& feed) : f(feed), last(feed.jb.k1 - 1) {
    const AttnParams& p = f.p;
    const int lr = f.l / F::VPR, lc = f.l % F::VPR;
    const int64_t head = ((PG ? 0 : (int64_t)f.jb.b * p.kv.seq_stride) + (int64_t)f.jb.hk * p.kv.head_stride) * 2;
#pragma unroll
    for (int i = 0; i < P; i++) {
      const int rr = f.part_row(i) + lr;
      key[i] = f.jb.k0 + rr;
      key[i] = key[i] < last ? key[i] : last;
      kb[i] = f.kbase + head + (lc ^ swizzle_k<D>(rr)) * 16;
      vb[i] = f.vbase + head + (lc ^ swizzle_v<D, 32>(rr)) * 16;
      blk[i] = 0;
    }
    if (PG) look_up();
  }
  __device__ __forceinline__ void look_up() {
#pragma unroll
    for (int i = 0; i < P; i++) blk[i] = f.bt[((key[i] >> f.ka.bs_shift) - f.ka.bt_first) & (kBtLds - 1)];
  }
  // The next unit's addresses, and on to the one behind it (whose table entries are asked for here and looked at a step later).
  __device__ __forceinline__ void next(int64_t (&off)[P], uint32_t& dst) {
    const KvAddr& a = f.p.kv;
    if (PG) {
      if (f.long_slice) f.bt_ahead(f.requested);
#pragma unroll
      for (int i = 0; i < P; i++) {
        int b = blk[i];
        b = b < 0 ? 0 : (b >= (int)a.num_blocks ? (int)a.num_blocks - 1 : b);
        off[i] = (int64_t)(uint64_t)(uint32_t)b * (a.seq_stride * 2) + (int64_t)((uint64_t)(uint32_t)(key[i] & (a.block_size - 1)) * (uint32_t)f.ts2);
      }
    } else {
#pragma unroll
      for (int i = 0; i < P; i++) off[i] = (int64_t)((uint64_t)(uint32_t)key[i] * (uint32_t)f.ts2);
    }
#pragma unroll
    for (int i = 0; i < P; i++) {
      key[i] += kUnitKeys;
      key[i] = key[i] < last ? key[i] : last;
    }
    if (PG) look_up();
    dst = place + f.part_row(0) * (2 * D) + __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(CB_LDS uint4*)f.ring);
    place = place + F::kSlotBytes == NS * F::kSlotBytes ? 0 : place + F::kSlotBytes;
    f.requested++;
  }
  // request i of a unit's 2 P (a constant): group i / 2, K or V
  __device__ __forceinline__ void request(int i, const int64_t (&off)[P], uint32_t dst) const {
    const int part = i / 2;
    lds_dma_b128_at((i & 1 ? vb[part] : kb[part]) + off[part], dst + part * (RPR * 2 * D) + (i & 1 ? F::kSlotBytes / 2 : 0));
  }
  __device__ __forceinline__ void request_units(int n) {
    for (int u = 0; u < n; u++) {
      int64_t off[P];
      uint32_t dst;
      next(off, dst);
#pragma unroll
      for (int i = 0; i < 2 * P; i++) request(i, off, dst);
    }
  }
};

// The sweep of one workgroup whose tile has RW row groups of R row tiles each, up to its output rows (a single split) or its
// partial state.
template <int D, bool PX, bool PG, int R, int RW, bool TS>
__device__ __forceinline__ void sweep_tile(const AttnParams& p, const TileJob& jb, TileLds& sh, uint4* ring,
                                           CB_LDS unsigned long long* ts) {
  using Part = PartialLayout<D, 32, PX>;
  using F = Feed<D, kWideWaves, 32>;
  constexpr int KW = kWideWaves / RW;    // key groups
  constexpr int NS = F::kSlots, PRO = F::kPrologue;
  constexpr int NPB = PX ? 4 : 2;        // B operands of a unit's probabilities
  // (scores run one stage ahead of the softmax: two stages are resident while a third is requested)
  static_assert(3 * KW <= NS && KW <= PRO, "a stage is requested in full while the one before it is worked on");
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
  const int rw = w % RW, kw = w / RW;
  const int r = l & 31, h = l >> 5;
  const bool do_ts = TS && tid == 0;
#define CB_TS(i) do { if (do_ts) ts[i] = wall_clock64(); } while (0)
  const CB_GLOBAL uint16_t* gq = (const CB_GLOBAL uint16_t*)p.q;
  const int S = jb.S, k0 = jb.k0, k1 = jb.k1;
  F ring_feed(p, jb, sh.bt, ring);
  WideFeed<D, PG> feed(ring_feed);
  // Everything the first stages need is requested up front, oldest first: the query rows (to registers), then K/V
  // units (to LDS).
  TileState<D> st[R];
  int node[R];       // tree node of the lane's queries (indexes the ancestor sets)
  int64_t grow[R];   // their output rows (node * Hq + head), or -1 past the end
#pragma unroll
  for (int t = 0; t < R; t++) {
    int row = jb.row0 + (rw * R + t) * 32 + r;
    const bool valid = row < jb.M;
    row = valid ? row : jb.M - 1;
    node[t] = row / jb.g;
    const int64_t gr = (int64_t)(jb.off + node[t]) * p.Hq + jb.hk * jb.g + (row - node[t] * jb.g);
    grow[t] = valid ? gr : -1;
    const CB_GLOBAL uintx4* qp = (const CB_GLOBAL uintx4*)(gq + gr * D);
#pragma unroll
    for (int ds = 0; ds < D / 16; ds++) st[t].q[ds] = __builtin_bit_cast(bf16x8, load_b128_untracked(qp + 2 * ds + h));
#pragma unroll
    for (int dt = 0; dt < D / 32; dt++)
#pragma unroll
      for (int v = 0; v < 16; v++) st[t].o[dt][v] = 0.f;
    st[t].lacc = floatx4{0.f, 0.f, 0.f, 0.f};
    st[t].mref = st[t].top = -INFINITY;
    st[t].nm = 0.f;
  }
  const bool has_rows = jb.row0 + rw * R * 32 < jb.M;
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
  feed.request_units(nu < PRO ? nu : PRO);
  CB_TS(2);
  if (tree_split) build_ancestor_sets(sh.anc, jb.N, my_parent, jump_rounds(p.max_depth));  // uniform in the workgroup; hidden behind the first K/V wait
  ring_feed.wait_units(KW);
#pragma unroll
  for (int t = 0; t < R; t++)
#pragma unroll
    for (int ds = 0; ds < D / 16; ds++) {
      asm volatile("" : "+v"(st[t].q[ds]));  // (older than every unit)
#ifdef __HIP_DEVICE_COMPILE__
      if (R > 1) asm volatile("" : "+a"(st[t].q[ds]));  // (two tiles' queries live in accumulation registers)
#endif
    }
  CB_TS(3);

  // At the barrier in front of unit u NS - 2 units from u on have been requested.  It waits until those up to u + 3 have
  // landed; everybody is then done with those below u, whose places take the next requests.
  // (a split of fewer units waits for all of them at the first barrier)
  auto ready = [&] {
    wait_vmcnt<F::kReq * (NS - 6)>();
    bare_barrier();
  };
  auto first_ready = [&] {
    const int more = (nu < NS - 2 ? nu : NS - 2) - PRO;
    if (more > 0) feed.request_units(more);
    if (nu < NS - 2) wait_vmcnt<0>();
  };
  auto top = [&] {  // of a stage in the general loop, whose last reads may still be under way
    wait_vmcnt<F::kReq * (NS - 6)>();
    ring_barrier();
    feed.request_units(KW);
  };
  // this wave's stages whose units are all prefix and all inside the split (rounds down; may be negative: none)
  auto fast_stages = [&] {
    const int n = ((S < k1 ? S : k1) - k0 - kw * kUnitKeys) / (kUnitKeys * KW);
    return nst < n ? nst : n;
  };
  // Places in the ring, in bytes, of this wave's units of the current stage and the two behind it
  constexpr uint32_t kSlotBytes = F::kSlotBytes;
  auto next_place = [&](uint32_t x) { return x + KW * kSlotBytes >= NS * kSlotBytes ? x + KW * kSlotBytes - NS * kSlotBytes : x + KW * kSlotBytes; };
  uint32_t at = kw * kSlotBytes, at1 = next_place(at), at2 = next_place(at1);
  auto advance = [&] {
    at = at1;
    at1 = at2;
    at2 = next_place(at2);
  };
  const uint32_t lane_k = (uint32_t)(uintptr_t)(CB_LDS uint4*)ring + lane_k_byte<D>(l);
  const uint32_t lane_v = (uint32_t)(uintptr_t)(CB_LDS uint4*)ring + kSlotBytes / 2 + lane_v_byte<D>(l);
  const bf16x8 ones = half_ones(l);

  auto unit_scores = [&](int s, uint32_t place, floatx16 (&sc)[R]) {
    uint4 k[D / 16];
    read_k<D>(lane_k + place, k);
    scores<D, R>(k, st, sc);
    const int key0 = k0 + (s * KW + kw) * kUnitKeys;
    if (key0 + kUnitKeys > S || key0 + kUnitKeys > k1)
#pragma unroll
      for (int t = 0; t < R; t++) mask_scores(sc[t], key0, S, k1, &sh.anc.anc[node[t]][0], h);
  };
  auto add_unit = [&](const bf16x8 (&pb)[R][NPB], uint32_t place) {
    const uint32_t va = lane_v + place;
#pragma unroll
    for (int t = 0; t < R; t++)
#pragma unroll
      for (int j = 0; j < NPB; j++) st[t].lacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pb[t][j], st[t].lacc, 0, 0, 0);
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
      for (int dt = 0; dt < D / 32; dt++) {
        const bf16x8 a = read_v<D>(va, dt, j);
#pragma unroll
        for (int t = 0; t < R; t++)
#pragma unroll
          for (int x = j; x < NPB; x += 2) st[t].o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pb[t][x], st[t].o[dt], 0, 0, 0);
      }
  };
  auto sweep = [&] {
    floatx16 sc[R];
    bf16x8 pb[R][NPB];
    float mx[R];
    auto check = [&] {
      bool raise = mx[0] > st[0].top;  // (false for NaN)
      if (R > 1) raise |= mx[R - 1] > st[R - 1].top;
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(raise) != 0, 0)) {
#pragma unroll
        for (int t = 0; t < R; t++) raise_reference<D>(st[t], mx[t], c2);
      }
    };
    auto maxima = [&](const floatx16 (&x)[R]) {
#pragma unroll
      for (int t = 0; t < R; t++) mx[t] = row_max(x[t]);
    };
    unit_scores(0, at, sc);
    maxima(sc);
    check();
    int s = 0;
    const int fast_end = fast_stages();
    floatx16 sd[R];
    uint4 k[D / 16];
    uintx4 pw[R][NPB];
    bf16x8 v[D / 32];
    // Stages whose units are all prefix, two at a time (the scores alternate between two sets of registers), the requests
    // spread over the steps (all at once they hold up the wave that makes them).  One barrier per two units.
    auto step = [&](const floatx16 (&from)[R], floatx16 (&to)[R], bool barrier) {  // stage s; from: its scores, to: those of stage s + 1
      if (barrier) ready();
      int64_t off[KW][F::kParts];
      uint32_t dst[KW];
#pragma unroll
      for (int x = 0; x < KW; x++) feed.next(off[x], dst[x]);
      if (KW > 1) read_k<D>(lane_k + at1, k);
      score_half<D, PX, R, KW * F::kReq>(k, st, from, to, pw, lane_v + at, v, c2, [&](int i) {
        feed.request(i % F::kReq, off[i / F::kReq], dst[i / F::kReq]);
      });
      add_half<D, PX, R, KW == 1>(k, lane_k + at2, lane_v + at, v, st, pw, to, mx, ones);
      check();
      advance();
      s++;
    };
    first_ready();
    if (s + 2 < fast_end) {
      if (KW == 1) {  // (K operands are a step ahead in registers)
        ready();
        read_k<D>(lane_k + at1, k);
      }
      do {
        step(sc, sd, true);
        step(sd, sc, KW > 1);
      } while (s + 2 < fast_end);
    }
    for (; s + 1 < nst; s++) {
      top();
      floatx16 sn[R];
      unit_scores(s + 1, at1, sn);
#pragma unroll
      for (int t = 0; t < R; t++) probs<D, PX>(sc[t], st[t], c2, pb[t]);
      add_unit(pb, at);
      maxima(sn);
      check();
#pragma unroll
      for (int t = 0; t < R; t++) sc[t] = sn[t];
      advance();
    }
#pragma unroll
    for (int t = 0; t < R; t++) probs<D, PX>(sc[t], st[t], c2, pb[t]);
    add_unit(pb, at);
  };
  if (has_rows) sweep();
  else {  // no rows of its own: it only brings its share, passing the same barriers
    int s = 0;
    first_ready();
    if constexpr (KW == 1) {
      const int fast_end = fast_stages();
      if (s + 2 < fast_end) ready();
      for (; s + 2 < fast_end; s += 2) {
        ready();
        feed.request_units(2);
      }
    }
    for (; s + 1 < nst; s++) top();
  }
  wait_vmcnt<0>();  // (the requests past the split's end, before the ring serves anything else)
  CB_TS(4);
  // With two key groups each finishes one half of the pieces: all park their accumulators and (mref, l) in the
  // ring, then each adds up the groups' for its own pieces.
  constexpr int P = Part::P, PP = P / KW;
  auto piece = [&](int t, int pc) {
    const floatx16& o = st[t].o[pc >> 2];
    return floatx4{o[4 * (pc & 3)], o[4 * (pc & 3) + 1], o[4 * (pc & 3) + 2], o[4 * (pc & 3) + 3]};
  };
  floatx4* const park = reinterpret_cast<floatx4*>(ring);
  float2* const park_ml = reinterpret_cast<float2*>(ring + kWideWaves * R * P * 64);
  if constexpr (KW > 1) {
    __syncthreads();  // every wave is done with the ring
    static_assert(kWideWaves * R * (P * 64 + 32) <= F::kRingVecs, "");
#pragma unroll
    for (int t = 0; t < R; t++) {
#pragma unroll
      for (int pc = 0; pc < P; pc++) park[((w * R + t) * P + pc) * 64 + l] = piece(t, pc);  // (w = kw * RW + rw)
      park_ml[(w * R + t) * 64 + l] = float2{st[t].mref, st[t].lacc[0]};
    }
    __syncthreads();
  }
#pragma unroll
  for (int t = 0; t < R; t++) {
    floatx4 f[PP];
    float lsum, mfin;
    if constexpr (KW > 1) {
      float2 ml[KW];
      mfin = -INFINITY;
#pragma unroll
      for (int k = 0; k < KW; k++) {
        ml[k] = park_ml[((k * RW + rw) * R + t) * 64 + l];
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
        for (int i = 0; i < PP; i++) f[i] += park[(((k * RW + rw) * R + t) * P + kw * PP + i) * 64 + l] * wt;
      }
    } else {
      lsum = st[t].lacc[0];
      mfin = st[t].mref;
#pragma unroll
      for (int i = 0; i < PP; i++) f[i] = piece(t, i);
    }
    write_rows<D, 32, PX, PP>(p, jb, rw * R + t, grow[t], f, kw * PP, mfin, lsum, c2, kw == 0, l);
  }
#undef CB_TS
}

// One attention workgroup of four waves whose tile has up to 256 rows; `wg` is its number among those that do attention.
// R128: row tiles of a wave where the tile has 65 to 128 rows, four groups of one with one key group, or two of two with two key groups.
template <int D, bool PX, bool PG, int R128, bool MOVE, bool TS, typename Layers>
__device__ __forceinline__ void attn_wide_tile(const AttnParams& p_arg, const SeqMetaLanes& ml, int wg, unsigned long long ts0,
                                               TileLds& sh, uint4* ring, unsigned long long* ts_sh, const Layers& layers) {
  AttnParams p = p_arg;
  pin_args(p);
  CB_LDS unsigned long long* ts = (CB_LDS unsigned long long*)ts_sh;
  first_stamps<TS>(ts, ts0);
  TileJob jb;
  if (!tile_job(p, ml, wg, p.tile_rows, layers, jb)) return;
  take_layer(p, jb, layers);
  const int rows = jb.M - jb.row0 < p.tile_rows ? jb.M - jb.row0 : p.tile_rows;
  if (rows <= 64) sweep_tile<D, PX, PG, 1, 2, TS>(p, jb, sh, ring, ts);
  else if (rows <= 128) sweep_tile<D, PX, PG, R128, 4 / R128, TS>(p, jb, sh, ring, ts);
  else sweep_tile<D, PX, PG, 2, 4, TS>(p, jb, sh, ring, ts);
  HeadMove<row_pieces(D, 2), 1> move;
  if (MOVE && jb.k1 > jb.S) {  // (uniform)
    bare_barrier();  // (every wave's requests have landed)
    if (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) == 0) move.begin(jb.b, jb.hk, jb.S, jb.N);
  }
  auto finish_move = [&] { if (MOVE) move.finish(jb.b, jb.hk, jb.S, jb.N); };
  if (jb.nsplit == 1 || p.external_merge) {  // (a following kernel merges: the kernel boundary orders the stores)
    finish_move();
    return;
  }
  split_merge<D, 32, PX, kWideWaves, 256, TS>(p, jb, p.tile_rows, sh, ts, finish_move);
}

template <int D, bool PX, bool PG, int R128, bool TS>
__global__ __launch_bounds__(64 * kWideWaves, 1) void k_attn_wide(AttnParams p, SeqMeta meta) {
  const unsigned long long ts0 = TS ? wall_clock64() : 0ull;
  const SeqMetaLanes ml = seq_meta_prefetch(meta);
  __shared__ __align__(1024) uint4 ring[Feed<D, kWideWaves, 32>::kRingVecs];
  __shared__ TileLds sh;
  __shared__ unsigned long long ts_sh[TS ? 16 : 1];
  attn_wide_tile<D, PX, PG, R128, false, TS>(p, ml, blockIdx.x, ts0, sh, ring, ts_sh, OneLayer{});
  flush_timestamps<TS>(p, blockIdx.x, ts_sh);
}

// The whole verification in one launch, as k_verify_mfma does it for small tiles: the first lw.n_wgs workgroups do the
// logits work, the others the attention.
template <int D, bool PX, bool PG, int R128, bool TS>
__global__ __launch_bounds__(64 * kWideWaves, 1) void k_verify_wide(AttnParams p, SeqMeta meta, LogitsWork lw) {
  const unsigned long long ts0 = TS ? wall_clock64() : 0ull;
  const SeqMetaLanes ml = seq_meta_prefetch(meta);
  __shared__ __align__(1024) uint4 ring[Feed<D, kWideWaves, 32>::kRingVecs];
  __shared__ TileLds sh;
  __shared__ unsigned long long ts_sh[TS ? 16 : 1];
  static_assert(sizeof(ring) >= sizeof(AcceptWaveLds), "the acceptance's LDS is the ring's");
  const int wg = (int)blockIdx.x - lw.n_wgs;
  if (wg < 0) {
    logits_share<kWideWaves, 16>(lw, ml, blockIdx.x, *reinterpret_cast<AcceptWaveLds*>(ring));
    return;
  }
  attn_wide_tile<D, PX, PG, R128, false, TS>(p, ml, wg, ts0, sh, ring, ts_sh, OneLayer{});
  flush_timestamps<TS>(p, wg, ts_sh);
}

// The attention of several layers in one launch, with the logits work (of the last one) in its first workgroups where lw.n_wgs is not 0.
template <int D, bool PX, bool PG, int R128>
__global__ __launch_bounds__(64 * kWideWaves, 1) void k_model_wide(AttnParams p, SeqMeta meta, LogitsWork lw, LayerTable layers) {
  const SeqMetaLanes ml = seq_meta_prefetch(meta);
  __shared__ __align__(1024) uint4 ring[Feed<D, kWideWaves, 32>::kRingVecs];
  __shared__ TileLds sh;
  const int wg = (int)blockIdx.x - lw.n_wgs;
  if (wg < 0) logits_share<kWideWaves, 16>(lw, ml, blockIdx.x, *reinterpret_cast<AcceptWaveLds*>(ring));
  else attn_wide_tile<D, PX, PG, R128, false, false>(p, ml, wg, 0ull, sh, ring, nullptr, layers);
}

// A verification with the compaction in its launch; lw.n_wgs is 0 where the logits work has a launch of its own.
template <int D, bool PX, bool PG, int R128>
__global__ __launch_bounds__(64 * kWideWaves, 1) void k_step_wide(AttnParams p, SeqMeta meta, LogitsWork lw) {
  const SeqMetaLanes ml = seq_meta_prefetch(meta);
  __shared__ __align__(1024) uint4 ring[Feed<D, kWideWaves, 32>::kRingVecs];
  __shared__ TileLds sh;
  const int wg = (int)blockIdx.x - lw.n_wgs;
  if (wg < 0) logits_share<kWideWaves, 16>(lw, ml, blockIdx.x, *reinterpret_cast<AcceptWaveLds*>(ring), after_acceptance<true, row_pieces(D, 2), 1, 4>());
  else attn_wide_tile<D, PX, PG, R128, true, false>(p, ml, wg, 0ull, sh, ring, nullptr, OneLayer{});
}

template <int D, bool PX, bool PG, int R128>
inline hipError_t launch_wide(hipStream_t st, const AttnParams& p, const SeqMeta& meta, int n_tiles, const LogitsWork* lw) {
  const dim3 grid(n_tiles + (lw ? lw->n_wgs : 0)), block(64 * kWideWaves);
  if (lw && p.timeline) hipLaunchKernelGGL((k_verify_wide<D, PX, PG, R128, true>), grid, block, 0, st, p, meta, *lw);
  else if (lw) hipLaunchKernelGGL((k_verify_wide<D, PX, PG, R128, false>), grid, block, 0, st, p, meta, *lw);
  else if (p.timeline) hipLaunchKernelGGL((k_attn_wide<D, PX, PG, R128, true>), grid, block, 0, st, p, meta);
  else hipLaunchKernelGGL((k_attn_wide<D, PX, PG, R128, false>), grid, block, 0, st, p, meta);
  return hipGetLastError();
}

}  // namespace cb
