// Device code of the greedy acceptance check (Section 3.2 of the paper, last paragraphs): the
// vocabulary argmax of every tree node's logits row, and the longest accepted root-to-leaf path.
// Shared by the stand-alone logits kernel and by the attention kernels, whose first workgroups can
// do this work in the same launch.  gfx950 only.
#pragma once
#include "cb_move.h"

namespace cb {

// Wave-wide reductions that leave the result in every lane, without LDS traffic: four rotations
// inside each row of 16 lanes (DPP row_ror:1,2,4,8), then the gfx950 row swaps for the four rows
// (v_permlane16_swap exchanges odd rows of one operand with even rows of the other,
// v_permlane32_swap the upper half of one with the lower half of the other).
template <typename Op>
__device__ __forceinline__ uint32_t wave_allreduce_u32(uint32_t x, Op op) {
  x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x121, 0xf, 0xf, false));
  x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x122, 0xf, 0xf, false));
  x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x124, 0xf, 0xf, false));
  x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xf, 0xf, false));
  const auto a = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  x = op(a[0], a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  return op(b[0], b[1]);
}
__device__ __forceinline__ float wave_max_f32(float x) {
  return __uint_as_float(wave_allreduce_u32(__float_as_uint(x), [](uint32_t p, uint32_t q) {
    return __float_as_uint(fmaxf(__uint_as_float(p), __uint_as_float(q)));
  }));
}
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t x) {
  return wave_allreduce_u32(x, [](uint32_t p, uint32_t q) { return p < q ? p : q; });
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t x) {
  return wave_allreduce_u32(x, [](uint32_t p, uint32_t q) { return p > q ? p : q; });
}

// v_max3_f32 as such: fmaxf() costs a canonicalising instruction per operand first (the compiler cannot know that
// loaded values are not signalling NaNs; the inputs are finite by precondition).
__device__ __forceinline__ float max3(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// A row's first maximum as one 64-bit word that grows with the value and, among equal values, with
// falling index, so that workgroups combine their candidates with an atomic maximum: the value's bits
// made monotonic (-0 first made +0: the two compare equal) above the complement of the index.  Zero is
// below every candidate.
__device__ __forceinline__ unsigned long long amax_word(float v, int i) {
  const uint32_t u = __float_as_uint(v + 0.0f);
  const uint32_t key = u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
  return ((unsigned long long)key << 32) | (uint32_t)~(uint32_t)i;
}
__device__ __forceinline__ int amax_word_index(unsigned long long w) { return (int)~(uint32_t)w; }

struct AcceptArgs {
  const int32_t* parent;   // [sumN] local parent indices
  const int32_t* tokens;   // [sumN] draft tokens
  int32_t* status;
  unsigned long long* best;  // [sumN] row maxima (amax_word), kAmaxStride words apart; zero between launches
  int32_t max_depth;
  int32_t* argmax_out;     // [sumN]
  int32_t* path;           // [B][max_depth + 1] (these two are for the compaction; where it is part of the launch they are
  int32_t* len_ctx;        // [B] written through to memory)
  int32_t* len_user;       // [B]
  int32_t* tok_user;       // [B][max_depth + 1]
  int32_t* last_user;      // [B] or null: host-visible words for the path's last node (the path's length where nothing has to move)
  int32_t* done_flag;      // [B] or null: host-visible words that receive done_value once the sequence's
  int32_t done_value;      // user results are visible to the host (the host form polls them)
};

// Tells a polling host that sequence b's results have arrived.  Called by the wave that wrote the
// results, after its stores: the system-scope release fence makes the wave's earlier stores visible
// to the host before the flag store that follows can be.
__device__ __forceinline__ void publish_done(const AcceptArgs& g, int b, bool writer) {
  if (!g.done_flag) return;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");
  if (writer) __hip_atomic_store(as_global(g.done_flag) + b, g.done_value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

template <bool THROUGH>
__device__ __forceinline__ void store_result(int32_t* p, int x) {
  if (THROUGH) __hip_atomic_store(as_global(p), x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else *as_global(p) = x;
}

// Parent of node t as loaded -> as used (-1 at the root; an entry outside [0, t) becomes "child of the
// root" and is reported in the status word).
__device__ __forceinline__ int checked_parent(int raw, int t, int32_t* status) {
  const bool bad = t == 0 ? raw != -1 : (raw < 0 || raw >= t);
  if (bad) __hip_atomic_fetch_or(as_global(status), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return t == 0 ? -1 : (bad ? 0 : raw);
}
// The row's first maximum; the word is made zero again for the next launch.
__device__ __forceinline__ int take_argmax(const AcceptArgs& g, int row) {
  CBL_GLOBAL unsigned long long* const p = as_global(g.best) + (int64_t)row * kAmaxStride;
  const int a = amax_word_index(__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  __hip_atomic_store(p, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  as_global(g.argmax_out)[row] = a;
  return a;
}

// Greedy acceptance of one sequence's tree by ONE wavefront.  A node is accepted when every non-root
// node on its chain carries the token generated at that node's parent; the accepted node of greatest
// depth wins (lowest index among equals) and its chain is the path.  The other waves of the workgroup
// are not involved.  This form: at most 64 nodes, lane t owns node t, no LDS; the ancestor sets are
// 64-bit lane values combined with lane permutes, and "accepted" is "the set is a subset of the matching
// nodes".
__device__ __forceinline__ unsigned long long shfl_u64(unsigned long long x, int lane) {
  const uint32_t lo = __shfl((uint32_t)x, lane, 64), hi = __shfl((uint32_t)(x >> 32), lane, 64);
  return (unsigned long long)lo | ((unsigned long long)hi << 32);
}
template <bool THROUGH>
__device__ __forceinline__ void accept_small(const AcceptArgs& g, int b, int off, int N) {
  const int t = threadIdx.x & 63;
  const bool live = t < N;
  int par = -1, tok = 0, a = -1;
  if (live) {
    const int raw = as_global(g.parent)[off + t];
    tok = as_global(g.tokens)[off + t];
    a = take_argmax(g, off + t);
    par = checked_parent(raw, t, g.status);
  }
  const int a_par = __shfl(a, par < 0 ? 0 : par, 64);
  const bool match = live && (t == 0 || tok == a_par);
  const unsigned long long matched = __ballot(match);
  unsigned long long mine = live ? (1ull << t) : 0ull;
  int j = par;
  const int rounds = jump_rounds(g.max_depth);
  for (int r = 0; r < rounds && r < 6; r++) {  // six rounds complete any tree of 64 nodes
    const int src = j < 0 ? 0 : j;
    const unsigned long long other = shfl_u64(mine, src);
    const int jj = __shfl(j, src, 64);
    if (j >= 0) {
      mine |= other;
      j = jj;
    }
  }
  const int depth = __popcll(mine) - 1;
  bool acc = live && (mine & ~matched) == 0ull;
  if (live && (depth > g.max_depth || j >= 0)) {
    acc = false;
    __hip_atomic_fetch_or(as_global(g.status), 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  uint32_t key = acc ? ((uint32_t)(depth + 1) << 16) | (uint32_t)(0xffff - t) : 0u;
  key = wave_max_u32(key);
  const int best = 0xffff - (int)(key & 0xffff);  // the root is always accepted, so key != 0
  const int L = (int)(key >> 16) - 1;
  const unsigned long long on_path = shfl_u64(mine, best);
  const int stride = g.max_depth + 1;
  if (live && ((on_path >> t) & 1ull)) {
    store_result<THROUGH>(g.path + b * stride + depth, t);
    as_global(g.tok_user)[b * stride + depth] = a;
  }
  for (int d = t; d < stride; d += 64) {
    if (d > L) {
      store_result<THROUGH>(g.path + b * stride + d, -1);
      as_global(g.tok_user)[b * stride + d] = -1;
    }
  }
  if (t == 0) {
    store_result<THROUGH>(g.len_ctx + b, L);
    as_global(g.len_user)[b] = L;
    if (g.last_user) as_global(g.last_user)[b] = best;
  }
  publish_done(g, b, t == 0);
}

// The same for up to CB_MAX_NODES nodes, lane t owning nodes t, t + 64, t + 128, t + 192, with a few KiB
// of LDS of the wave's own.  Pointer jumping on one word per node -- ancestor pointer, depth collected,
// "all matched so far" --, every round's pointers kept so that the path can be marked afterwards: from
// the winner, the 2^r-th ancestors of all marked nodes for r from the last round down mark exactly its
// chain.  (The wave's LDS accesses execute in program order; the waits keep the compiler from moving
// them across.)
struct AcceptWaveLds {
  int32_t a[CB_MAX_NODES];
  uint32_t state[CB_MAX_NODES];      // bits 0-8 ancestor + 1 (0: none left), bit 9 matched, bits 16.. depth
  int16_t jump[8][CB_MAX_NODES];     // each round's ancestor pointers, -1 none
  uint32_t mark[CB_MAX_NODES];
  unsigned long long accepted;       // sequences that the workgroup accepted (logits_share)
};
__device__ __forceinline__ void wave_lds_sync() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

template <bool THROUGH>
__device__ __forceinline__ void accept_large(AcceptWaveLds& sh, const AcceptArgs& g, int b, int off, int N) {
  constexpr int KN = CB_MAX_NODES / 64;
  const int lane = threadIdx.x & 63;
  int par[KN], tok[KN], a[KN];
#pragma unroll
  for (int k = 0; k < KN; k++) {
    const int t = lane + 64 * k;
    par[k] = t < N ? as_global(g.parent)[off + t] : -1;
    tok[k] = t < N ? as_global(g.tokens)[off + t] : 0;
  }
#pragma unroll
  for (int k = 0; k < KN; k++) {
    const int t = lane + 64 * k;
    a[k] = -1;
    if (t < N) {
      a[k] = take_argmax(g, off + t);
      par[k] = checked_parent(par[k], t, g.status);
    }
    sh.a[t] = a[k];
    sh.mark[t] = 0;
  }
  wave_lds_sync();
  uint32_t st[KN];
#pragma unroll
  for (int k = 0; k < KN; k++) {
    const int t = lane + 64 * k;
    const bool match = t == 0 || (t < N && tok[k] == sh.a[par[k] < 0 ? 0 : par[k]]);
    st[k] = (uint32_t)(par[k] + 1) | (match ? 0x200u : 0u) | (par[k] >= 0 ? 0x10000u : 0u);
    sh.state[t] = st[k];
  }
  const int rounds = jump_rounds(g.max_depth);
  for (int r = 0; r < rounds; r++) {
    wave_lds_sync();
    uint32_t other[KN];
#pragma unroll
    for (int k = 0; k < KN; k++) {
      const int j = (int)(st[k] & 0x1ffu) - 1;
      sh.jump[r][lane + 64 * k] = (int16_t)j;
      other[k] = sh.state[j < 0 ? 0 : j];
    }
    wave_lds_sync();
#pragma unroll
    for (int k = 0; k < KN; k++) {
      if ((st[k] & 0x1ffu) != 0) {
        st[k] = (other[k] & 0x1ffu) | (st[k] & other[k] & 0x200u) | ((st[k] & 0xffff0000u) + (other[k] & 0xffff0000u));
        sh.state[lane + 64 * k] = st[k];
      }
    }
  }
  uint32_t key = 0;
#pragma unroll
  for (int k = 0; k < KN; k++) {
    const int t = lane + 64 * k;
    if (t >= N) continue;
    const int depth = (int)(st[k] >> 16);
    if (depth > g.max_depth || (st[k] & 0x1ffu) != 0) {  // (an unresolved node is deeper than the rounds reach, hence too deep)
      __hip_atomic_fetch_or(as_global(g.status), 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else if (st[k] & 0x200u) {
      const uint32_t kk = ((uint32_t)(depth + 1) << 16) | (uint32_t)(0xffff - t);
      key = kk > key ? kk : key;
    }
  }
  key = wave_max_u32(key);
  const int best = 0xffff - (int)(key & 0xffff);  // the root is always accepted, so key != 0
  const int L = (int)(key >> 16) - 1;
  if (lane == 0) sh.mark[best] = 1;
  for (int r = rounds - 1; r >= 0; r--) {
    wave_lds_sync();
#pragma unroll
    for (int k = 0; k < KN; k++) {
      const int t = lane + 64 * k;
      const int j = sh.jump[r][t];
      if (sh.mark[t] && j >= 0) sh.mark[j] = 1;
    }
  }
  wave_lds_sync();
  const int stride = g.max_depth + 1;
#pragma unroll
  for (int k = 0; k < KN; k++) {
    const int t = lane + 64 * k;
    if (t < N && sh.mark[t]) {
      const int depth = (int)(st[k] >> 16);
      store_result<THROUGH>(g.path + b * stride + depth, t);
      as_global(g.tok_user)[b * stride + depth] = a[k];
    }
  }
  for (int d = lane; d < stride; d += 64) {
    if (d > L) {
      store_result<THROUGH>(g.path + b * stride + d, -1);
      as_global(g.tok_user)[b * stride + d] = -1;
    }
  }
  if (lane == 0) {
    store_result<THROUGH>(g.len_ctx + b, L);
    as_global(g.len_user)[b] = L;
    if (g.last_user) as_global(g.last_user)[b] = best;
  }
  publish_done(g, b, lane == 0);
  wave_lds_sync();
}

template <bool THROUGH = false>
__device__ __forceinline__ void accept_wave(AcceptWaveLds& sh, const AcceptArgs& g, int b, int off, int N) {
  if (N <= 64) accept_small<THROUGH>(g, b, off, N);
  else accept_large<THROUGH>(sh, g, b, off, N > CB_MAX_NODES ? CB_MAX_NODES : N);
}

// The logits work of one verification call: items (row, chunk of kArgmaxChunk or kArgmaxShortChunk elements), item = row *
// chunks + chunk, shared out evenly, in order, among all wavefronts of the workgroups that do it.
struct LogitsWork {
  const void* logits;   // [rows][V]
  int64_t V;
  int32_t rows;         // total tree nodes of the call
  int32_t batch;
  int32_t chunks;       // per row
  int32_t n_wgs;        // workgroups that share the work (the first ones of the launch)
  int32_t is_f32;       // element type of the logits: bf16 or fp32
  int32_t accept_after;  // 1: the wave that completes a sequence's rows runs its acceptance
  uint32_t* tickets;    // [B][kTicketWords] items finished per sequence, zero between launches
  AcceptArgs accept;
};

// First maximum of elements [e0, e1) of one row by one wavefront; the result (a word of amax_word) is
// valid in every lane.  Bound by the loads: a wave requests up to 16 KiB at a time (kVecs loads of 16 bytes per
// lane, all in flight before the first is looked at) and spends about 12 vector instructions per load on the
// maximum alone; where in the block it is first attained is looked up only in blocks that raise it.  A row may
// start at any element: the elements in front of the first and behind the last whole 16-byte piece are taken
// one by one.
template <typename T, int KV>
struct WaveScan {
  static constexpr int VEC = 16 / sizeof(T);
  static constexpr int kVecs = KV;  // (even)
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

  static __device__ __forceinline__ float to_f32(T x) {
    if constexpr (sizeof(T) == 2) return __uint_as_float((uint32_t)x << 16);
    else return x;
  }
  static __device__ __forceinline__ float elem(const u32x4& u, int j) {  // (j: a constant)
    if constexpr (sizeof(T) == 2) return __uint_as_float((j & 1) ? (u[j >> 1] & 0xffff0000u) : (u[j >> 1] << 16));
    else return __uint_as_float(u[j]);
  }
  static __device__ __forceinline__ float vec_max(const u32x4& u) {
    if constexpr (sizeof(T) == 2) {
      const float m = max3(elem(u, 0), elem(u, 1), elem(u, 2));
      return max3(max3(m, elem(u, 3), elem(u, 4)), max3(elem(u, 5), elem(u, 6), elem(u, 7)), m);
    } else {
      const float m = max3(elem(u, 0), elem(u, 1), elem(u, 2));
      return max3(m, elem(u, 3), m);
    }
  }

  static __device__ __forceinline__ unsigned long long run(const T* row_base, int e0, int e1) {
    const int lane = threadIdx.x & 63;
    const CBL_GLOBAL T* const base = (const CBL_GLOBAL T*)row_base;
    // whole 16-byte pieces [v0, v1) of elements, and up to VEC - 1 single elements on either side
    const int skew = (int)(((uintptr_t)row_base / sizeof(T)) & (VEC - 1));
    int v0 = e0 + ((VEC - ((e0 + skew) & (VEC - 1))) & (VEC - 1));
    v0 = v0 < e1 ? v0 : e1;
    const int nv = (e1 - v0) / VEC;
    const int v1 = v0 + nv * VEC;
    const CBL_GLOBAL u32x4* const vp = (const CBL_GLOBAL u32x4*)(base + v0);
    float best = -INFINITY;  // (uniform)
    int bidx = 0x7fffffff;
    for (int i0 = 0; i0 < nv; i0 += 64 * kVecs) {
      u32x4 u[kVecs];
#pragma unroll
      for (int k = 0; k < kVecs; k++) {  // (pieces past the end repeat the last one, which changes nothing)
        const int i = i0 + 64 * k + lane;
        u[k] = vp[i < nv ? i : nv - 1];
      }
      __builtin_amdgcn_sched_barrier(0);  // (all requested before the first is waited for)
      float vm[kVecs];
#pragma unroll
      for (int k = 0; k < kVecs; k++) vm[k] = vec_max(u[k]);
      float lm = vm[0];
#pragma unroll
      for (int k = 1; k + 1 < kVecs; k += 2) lm = max3(lm, vm[k], vm[k + 1]);
      lm = max3(lm, vm[kVecs - 1], lm);
      const float m = wave_max_f32(lm);
      if (__builtin_amdgcn_ballot_w64(m > best) == 0ull) continue;  // (uniform; later blocks hold higher indices)
      best = m;
      // lowest index in the block: the lowest k that any lane attains the maximum with, its lowest lane, there
      // the lowest element
      uint32_t idx = 0x7fffffffu;
#pragma unroll
      for (int k = kVecs - 1; k >= 0; k--) {
        if (vm[k] == m) {
          const int i = i0 + 64 * k + lane;
          int j = VEC - 1;
#pragma unroll
          for (int q = VEC - 2; q >= 0; q--) j = elem(u[k], q) == m ? q : j;
          idx = (uint32_t)(v0 + (i < nv ? i : nv - 1) * VEC + j);
        }
      }
      bidx = (int)wave_min_u32(idx);
    }
    if (v0 != e0 || v1 != e1) {  // (uniform)
      const int head = v0 - e0, tail = e1 - v1;
      const int e = lane < head ? e0 + lane : v1 + (lane - head);
      const bool has = lane < head + tail;
      const float x = has ? to_f32(base[has ? e : e0]) : -INFINITY;
      const float m = wave_max_f32(x);
      const int mi = (int)wave_min_u32(has && x == m ? (uint32_t)e : 0x7fffffffu);
      if (m > best || (m == best && mi < bidx)) {
        best = m;
        bidx = mi;
      }
    }
    return amax_word(best, bidx);
  }
};

// One workgroup's share of the logits work: items [items * wg / n, items * (wg + 1) / n), its NW wavefronts
// taking them in turn.  Their candidates go into the rows' words with atomic maxima; once those are
// acknowledged (every wave waits for its own, then a barrier) the first wave counts the workgroup's items on
// their sequences' tickets, and the workgroup whose count completes a sequence -- all candidates are then in
// memory -- runs the acceptance with that wave.  Nobody waits for anybody, so the order in which workgroups
// run is irrelevant.
// Atomics on one word are served about 15 ns apart, so a sequence that many workgroups arrive at has its items
// counted in 16 groups first, each on a line of its own, and the groups that are full on a last word (one word for
// all of 512 wavefronts' arrivals: 13 us for a scan of 8 MB).
constexpr int kTicketGroups = 16;
constexpr int kTicketStride = 32;                                    // 32-bit words between them (128 bytes)
constexpr int kTicketWords = (kTicketGroups + 1) * kTicketStride;    // per sequence
constexpr int kTicketDirect = 48;  // arrivals up to which one word serves a sequence

// LOADS: loads of 16 bytes that a lane has in flight, as the kernel's registers allow.  EB: bytes of a logits element
// where the kernel is built for one type, else 0.  after(b, S, N, i, n): what the wavefronts of the workgroup that accepted sequence b do
// then, behind a barrier, the i-th of n that the sequence has.
struct NothingAfter {
  static constexpr bool kAny = false;
  __device__ __forceinline__ void operator()(int, int, int, int, int) const {}
};
template <int NW, int LOADS, bool SHORT = false, int EB = 0, typename After = NothingAfter>
__device__ __forceinline__ void logits_share(const LogitsWork& lw, const SeqMetaLanes& ml, int wg, AcceptWaveLds& sh, const After& after = After{}) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t items = (int64_t)lw.rows * lw.chunks;
  const int i0 = (int)(items * wg / lw.n_wgs), i1 = (int)(items * (wg + 1) / lw.n_wgs);
  for (int i = i0 + w; i < i1; i += NW) {
    const int row = i / lw.chunks, c = i - row * lw.chunks;
    constexpr int CH = SHORT ? kArgmaxShortChunk : kArgmaxChunk;
    constexpr int KB = LOADS < CH / 512 ? LOADS : CH / 512, KF = LOADS < CH / 256 ? LOADS : CH / 256;
    const int64_t e0 = (int64_t)c * CH;
    const int64_t e1 = e0 + CH < lw.V ? e0 + CH : lw.V;
    const unsigned long long word =
        EB == 4 || (EB == 0 && lw.is_f32) ? WaveScan<float, KF>::run((const float*)lw.logits + (int64_t)row * lw.V, (int)e0, (int)e1)
                  : WaveScan<uint16_t, KB>::run((const uint16_t*)lw.logits + (int64_t)row * lw.V, (int)e0, (int)e1);
    if (lane == 0)
      __hip_atomic_fetch_max(as_global(lw.accept.best) + (int64_t)row * kAmaxStride, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (!lw.accept_after) return;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (!After::kAny && w != 0) return;
  unsigned long long accepted = 0;
  auto count = [&](CBL_GLOBAL uint32_t* word, uint32_t n, uint32_t full) {  // true: this arrival completed it
    uint32_t old = 0;
    if (lane == 0) old = __hip_atomic_fetch_add(word, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const bool done = __builtin_amdgcn_readfirstlane(old) + n == full;
    if (done && lane == 0) __hip_atomic_store(word, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // ready for the next launch
    return done;
  };
  for (int i = w == 0 ? i0 : i1; i < i1;) {
    const int row = i / lw.chunks;
    // sequence of the row: the number of sequences that end at or before it
    const int b = __popcll(__ballot(lane < lw.batch - 1 && ml.o1 <= row));
    const int off = __builtin_amdgcn_readlane(ml.o0, b), N = __builtin_amdgcn_readlane(ml.o1, b) - off;
    const int first = off * lw.chunks, end = (off + N) * lw.chunks, nb = N * lw.chunks;
    const int seq_end = end < i1 ? end : i1;
    CBL_GLOBAL uint32_t* const words = as_global(lw.tickets) + b * kTicketWords;
    bool done;
    if ((int64_t)nb * lw.n_wgs <= items * kTicketDirect) {
      done = count(words, (uint32_t)(seq_end - i), (uint32_t)nb);
    } else {
      const int gs = (nb + kTicketGroups - 1) / kTicketGroups, ng = (nb + gs - 1) / gs;
      done = false;
      for (int j = i; j < seq_end;) {
        const int gr = (j - first) / gs;
        const int g0 = first + gr * gs, g1 = g0 + gs < end ? g0 + gs : end;
        const int n = (g1 < seq_end ? g1 : seq_end) - j;
        if (count(words + (1 + gr) * kTicketStride, (uint32_t)n, (uint32_t)(g1 - g0))) done = count(words, 1u, (uint32_t)ng);
        j += n;
      }
    }
    if (done) {
      accept_wave<After::kAny>(sh, lw.accept, b, off, N);
      accepted |= 1ull << b;
    }
    i = seq_end;
  }
  if constexpr (!After::kAny) return;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (the results are in memory before anybody is told)
  if (threadIdx.x == 0) sh.accepted = accepted;
  __syncthreads();
  // Several sequences side by side, each by its share of the wavefronts: what follows one is a chain of round trips to memory, about 2 us.
  constexpr int LOG = __builtin_ctz(NW);
  static_assert(NW == 1 << LOG, "");
  const int seqs = __builtin_amdgcn_readfirstlane(__popcll(sh.accepted)), wave = __builtin_amdgcn_readfirstlane(w);
  const int groups = seqs <= 1 ? 0 : seqs >= NW ? LOG : 32 - __builtin_clz(seqs - 1), log_n = LOG - groups;  // (logarithms)
  int i = 0;
  for (unsigned long long todo = sh.accepted; todo != 0; todo &= todo - 1, i++) {
    if ((i & ((1 << groups) - 1)) != wave >> log_n) continue;
    const int b = __builtin_amdgcn_readfirstlane(__builtin_ctzll(todo));
    const SeqShape s = seq_shape(ml, b);
    after(b, s.S, s.N, wave & ((1 << log_n) - 1), 1 << log_n);
  }
}

// What follows the acceptance in a launch that compacts its cache (MOVE), or in one that does not.
template <bool MOVE, int PIECES, int SHIFT, int HB>
__device__ __forceinline__ auto after_acceptance() {
  if constexpr (MOVE) return MoveAfter<PIECES, SHIFT, HB>{};
  else return NothingAfter{};
}

}  // namespace cb
