// Compaction (slot S+j <- slot S+path[j], j = 1..L) inside the launch that verifies: device code shared by the attention kernels,
// whose workgroups move the K/V of their kv head, and by the acceptance.  gfx950 only.
//
// As a launch of its own behind the verification the compaction cost 2 to 3 us of a step of 12 to 32 us, almost all of it start and
// drain of a kernel that moves a few rows per head (a step in two launches -> in one: 15 rows of 8 fp32 heads of 64 x 256 keys 12.2
// -> 10.1 us, 64 of 32 heads x 2048 keys 17.7 -> 14.8, 128 of 32/8 heads x 8192 keys 31.1 -> 29.9).  Here nobody waits either: what has to be
// over before a head's rows may move arrives at a word of the (sequence, kv head), and whoever completes the word moves them.  Arrivals are the
// workgroups whose split reaches the tree (their sweep has read the tree's K/V), every row tile's, and the acceptance where it is
// part of the launch.
// The workgroups with the tree end early, as the last split is the shortest, and move while they would wait for the other splits.
#pragma once
#include "cb_internal.h"

namespace cb {

// Pieces of 16 bytes in a head's row.
__host__ __device__ constexpr int row_pieces(int D, int elem_bytes) { return D * elem_bytes / 16; }

__device__ __forceinline__ int agent_load(const int32_t* p) {
  return __hip_atomic_load(as_global(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The kernel's first argument once more, from its memory: what follows a sweep would otherwise be kept in scalar registers all through
// it (35 of them spilled, 0.5 us a launch of the 64-row kernel).
typedef const __attribute__((address_space(4))) AttnParams* ArgsPtr;
__device__ __forceinline__ ArgsPtr fresh_args() {
  ArgsPtr a = (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
#ifdef __HIP_DEVICE_COMPILE__
  asm volatile("" : "+s"(a));
#endif
  return a;
}
__device__ __forceinline__ KvAddr fresh_kv(ArgsPtr a) {
  return KvAddr{a->kv.k, a->kv.v, a->kv.block_table, a->kv.seq_stride, a->kv.token_stride, a->kv.head_stride, a->kv.num_blocks, a->kv.max_blocks, a->kv.block_size};
}

// The accepted path of one sequence as a wavefront holds it: lane i has path[1 + i].
struct AcceptedPath {
  const int32_t* row;
  int max_depth, L, first;
  __device__ __forceinline__ AcceptedPath(ArgsPtr a, int b) : row(a->move.path + (int64_t)b * (a->max_depth + 1)), max_depth(a->max_depth) {
    L = agent_load(a->move.len + b);
    first = from(0);
    L = __builtin_amdgcn_readfirstlane(L < 0 ? 0 : (L > max_depth ? max_depth : L));
  }
  __device__ __forceinline__ int from(int j0) const {  // path[1 + j0 + lane]
    const int j = 1 + j0 + (threadIdx.x & 63);
    return agent_load(row + (j <= max_depth ? j : max_depth));
  }
  // whether any row has to move (the first of the root's children, and of its children's, are in place)
  __device__ __forceinline__ bool moves() const {
    const int lane = threadIdx.x & 63;
    return L > 64 || __builtin_amdgcn_ballot_w64(lane < L && first != lane + 1) != 0;
  }
};

__device__ __forceinline__ long long lane_value(long long x, int lane) {
  return (long long)(uint32_t)__shfl((int)x, lane, 64) | ((long long)__shfl((int)(x >> 32), lane, 64) << 32);
}

// Moves the rows of HB kv heads of one sequence and layer, K and V, by one wavefront whose lanes each own a 16-byte piece of K's or V's row
// for every JP-th step of the path.  All of a batch's reads are complete before its first write, and later batches read slots that no
// earlier one wrote (path[j] >= j, increasing), so the result is that of the steps in order.  (hk: a head may be there twice.)
// Where a step's rows lie is worked out by one lane for all: the block table's entries come in one round trip, and the code, of which every
// call has a copy, is a quarter of what a division for each row makes it.
template <int PIECES, int SHIFT, int HB>  // (SHIFT: log2 of the element's bytes)
__device__ __forceinline__ void move_heads(const KvAddr& geo, const AcceptedPath& path, int b, int S, int N, const int (&hk)[HB]) {
  constexpr int PER = 2 * PIECES, JP = 64 / PER;
  // (loads in flight: as many as the registers hold, which in fp32 with head_dim 64 are 128)
  constexpr int STEPS = PIECES == 16 && SHIFT == 2 ? 2 : (8 / JP < 4 ? 8 / JP : 4), kBatch = STEPS * JP;
  static_assert(64 % PER == 0 && 64 % kBatch == 0, "");
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  const int lane = threadIdx.x & 63, grp = lane / PER, vec = lane % PIECES;
  // (a choice between two members would put the struct into memory)
  const uintptr_t k = (uintptr_t)geo.k, to_v = (uintptr_t)geo.v - k;
  CBL_GLOBAL char* const base = (CBL_GLOBAL char*)(k + ((lane / PIECES) & 1) * to_v + vec * 16);
  int64_t head[HB];
#pragma unroll
  for (int i = 0; i < HB; i++) head[i] = (int64_t)hk[i] * geo.head_stride << SHIFT;
#pragma unroll 1
  for (int w0 = 0; w0 < path.L; w0 += 64) {
    const int to = w0 + 1 + lane, src = w0 == 0 ? path.first : path.from(w0);
    const bool mine = to <= path.L && src > to && src < N;  // (src == to: nothing to move)
    const unsigned long long any = __builtin_amdgcn_ballot_w64(mine);
    long long from_off = 0, to_off = 0;
    if (mine) {
      from_off = slot_offset(geo, b, S + src, 0) << SHIFT;
      to_off = slot_offset(geo, b, S + to, 0) << SHIFT;
    }
    const int steps = path.L - w0 < 64 ? path.L - w0 : 64;
#pragma unroll 1
    for (int j0 = 0; j0 < steps; j0 += kBatch) {
      u32x4 x[HB][STEPS];
#pragma unroll
      for (int s = 0; s < STEPS; s++) {
        const int j = j0 + s * JP + grp;
        const long long off = lane_value(from_off, j);
        if ((any >> j) & 1ull) {
#pragma unroll
          for (int i = 0; i < HB; i++) x[i][s] = *(const CBL_GLOBAL u32x4*)(base + (off + head[i]));
        }
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (lanes read what other lanes write)
#pragma unroll
      for (int s = 0; s < STEPS; s++) {
        const int j = j0 + s * JP + grp;
        const long long off = lane_value(to_off, j);
        if ((any >> j) & 1ull) {
#pragma unroll
          for (int i = 0; i < HB; i++) *(CBL_GLOBAL u32x4*)(base + (off + head[i])) = x[i][s];
        }
      }
    }
  }
}

// Arrivals that complete a head's word: the row tiles' workgroups whose split reaches the tree, and the acceptance.
__device__ __forceinline__ uint32_t move_arrivals(ArgsPtr a, int S, int N) {
  const int tiles = (N * (a->Hq / a->Hkv) + a->tile_rows - 1) / a->tile_rows, splits = (S + N + a->chunk - 1) / a->chunk - S / a->chunk;
  return (uint32_t)(tiles * splits + (a->move.own_acceptance ? 1 : 0));
}
__device__ __forceinline__ CBL_GLOBAL uint32_t* move_word(ArgsPtr a, int b, int hk) { return as_global(a->move.words) + (int64_t)b * a->Hkv + hk; }

// The arrival of an attention workgroup, by one of its wavefronts, in two halves: begin() once every wavefront's K/V requests have
// landed and been waited for, finish() where a round trip to memory does not hold up anything.
template <int PIECES, int SHIFT>
struct HeadMove {
  bool mine = false;  // (uniform in the wavefront)
  uint32_t all, old;
  __device__ __forceinline__ void begin(int b, int hk, int S, int N) {
    const ArgsPtr a = fresh_args();
    mine = true;
    all = move_arrivals(a, S, N);
    old = 0;
    if (all > 1 && (threadIdx.x & 63) == 0) old = __hip_atomic_fetch_add(move_word(a, b, hk), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ void finish(int b, int hk, int S, int N) {
    if (!mine) return;
    mine = false;
    if ((uint32_t)__builtin_amdgcn_readfirstlane((int)old) + 1 != all) return;
    const ArgsPtr a = fresh_args();
    const AcceptedPath path(a, b);
    if (all > 1 && (threadIdx.x & 63) == 0) __hip_atomic_store(move_word(a, b, hk), 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // ready for the next launch
    if (path.moves()) move_heads<PIECES, SHIFT, 1>(fresh_kv(a), path, b, S, N, {hk});
  }
};

// The acceptance's arrival for the heads of a sequence, by `nw` wavefronts of its workgroup (logits_share), this one the w-th of them, behind a
// barrier that follows the acknowledgement of its stores; the heads whose attention is through already are moved here, HB at a time.  (A short
// sweep is through before the acceptance is, and then all heads are: with wide tiles, whose workgroups have four wavefronts, 97 nodes of 40 heads x
// 790 keys took 17.2 us a step two heads at a time and 16.5 four, two launches 16.5; 64 fp32 sequences of 8 nodes x 200 keys 36.7 one at a
// time and 31.1 four, two launches 30.4.)
template <int PIECES, int SHIFT, int HB>
struct MoveAfter {
  static constexpr bool kAny = true;
  __device__ __forceinline__ void operator()(int b, int S, int N, int w, int nw) const {
    const ArgsPtr a = fresh_args();
    const int lane = threadIdx.x & 63, Hkv = a->Hkv;
    const uint32_t all = move_arrivals(a, S, N);
    auto arrive = [&](int hk) { return hk < Hkv ? __hip_atomic_fetch_add(move_word(a, b, hk), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u; };
    uint32_t old = arrive(w + lane * nw);
    const AcceptedPath path(a, b);  // (its loads and the first arrivals in one round trip)
    for (int h0 = w; h0 < Hkv; h0 += 64 * nw) {  // (lane i: head h0 + i nw, so that every wavefront has few to move)
      const int hk = h0 + lane * nw;
      if (h0 != w) old = arrive(hk);
      const bool last = hk < Hkv && old + 1 == all;
      if (last) __hip_atomic_store(move_word(a, b, hk), 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // ready for the next launch
      unsigned long long todo = __builtin_amdgcn_ballot_w64(last);
      if (!path.moves()) continue;
      while (todo != 0) {
        int heads[HB];
#pragma unroll
        for (int i = 0; i < HB; i++) {
          heads[i] = i > 0 && todo == 0 ? heads[0] : __builtin_amdgcn_readfirstlane(h0 + __builtin_ctzll(todo) * nw);
          todo &= todo - 1;
        }
        move_heads<PIECES, SHIFT, HB>(fresh_kv(a), path, b, S, N, heads);
      }
    }
  }
};

}  // namespace cb
