// Tree-masked flash-decode attention on the matrix cores (bf16), gfx950 only: what the kernels of cb_attn_mfma.hip
// (tiles of up to 64 rows) and cb_attn_wide.h (up to 256) share -- the workgroup's job, the K/V ring, the partial
// states and their merge.
//
// Tree attention, Section 3.2 of the paper: node i attends to the KV-cached prefix (slots 0..S-1)
// and to the tree nodes on its own ancestor chain (slots S+a, a in anc(i)).  For one kv head the
// g*N query rows (g query heads per kv head, N nodes) form a small dense matrix, so QK^T and PV are
// MFMA contractions; the KV sequence is split across workgroups and the partial softmax states
// (o, m, l) are merged afterwards.
//
// One workgroup of 8 wavefronts (4 in the wide kernel) works on a (sequence, kv head, row tile, split).  K/V is brought straight from HBM into
// an LDS ring by LDS-DMA (no registers held by loads in flight) and is shared by the waves.  All loads of the
// sweep -- the ring's requests and the query rows -- are issued as instructions the compiler does not interpret and are
// covered by the kernel's own counted waits.
#pragma once
#include <type_traits>

#include "cb_logits.h"

namespace cb {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;
typedef __attribute__((__vector_size__(4 * sizeof(unsigned)))) unsigned uintx4;
typedef __attribute__((__vector_size__(2 * sizeof(unsigned)))) unsigned uintx2;
#define CB_GLOBAL __attribute__((address_space(1)))
#define CB_LDS __attribute__((address_space(3)))
constexpr int kAgentCoherent = 16;  // buffer cache policy: sc1 = coherent at agent (device) scope

// Block-table entries of a split in LDS: a ring of kBtSegs segments (entry i of the split's slice sits at i % kBtLds).
// The first kBtLds entries are there before the first request; a later segment is requested, by LDS-DMA, when the
// refills come within two segments of it.  512 entries are at least 16 units of requests even with one token
// per block, and at most the ring's 16 units are in flight when a stage begins, so a segment has landed
// in every wave's share before the first address that needs it.
constexpr int kBtSeg = 256;
constexpr int kBtSegs = 4;
constexpr int kBtLds = kBtSeg * kBtSegs;

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  // s_waitcnt simm16 on gfx9: vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt[5:4] at [15:14]
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

// A 16-byte global load that the compiler does not know to be one.  It orders every load it tracks
// against the LDS-DMA requests of the ring as if the two kinds could overtake each other: the first
// use of a tracked load's result while ring requests are in flight costs a wait for all of them.
// Loads return in the order they were issued, so the ring's own counted waits cover these; the
// caller pins the result (asm "+v") behind such a wait before it touches it.
__device__ __forceinline__ uintx4 load_b128_untracked(const CB_GLOBAL void* p) {
  uintx4 r;
  asm volatile("global_load_dwordx4 %0, %1, off" : "=v"(r) : "v"(p) : "memory");
  return r;
}

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {  // rounded to nearest even (v_cvt_pk_bf16_f32)
  typedef float float2v __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((float2v){lo, hi}, bf16x2v));
}

template <bool CONTIGUOUS>
struct KeyAddr {  // resolves cache slots of one (sequence, kv head) to byte offsets
  const KvAddr* kv;
  const int* bt;   // LDS ring of this split's slice of the block table (paged caches)
  int bt_first;    // logical block of bt[0]
  int bs_shift;    // log2(block_size)
  int seq, head;
  __device__ __forceinline__ int64_t byte_off(int slot) const {
    const KvAddr& a = *kv;
    if (!CONTIGUOUS && a.block_size > 0) {
      const int lb = slot >> bs_shift;
      int64_t blk = bt[(lb - bt_first) & (kBtLds - 1)];
      blk = blk < 0 ? 0 : (blk >= a.num_blocks ? a.num_blocks - 1 : blk);
      return (blk * a.seq_stride + (int64_t)(slot - (lb << bs_shift)) * a.token_stride +
              (int64_t)head * a.head_stride) * 2;
    }
    return ((int64_t)seq * a.seq_stride + (int64_t)slot * a.token_stride + (int64_t)head * a.head_stride) * 2;
  }
};

// Workgroup barrier without the memory fence of __syncthreads(): the fence would wait for every
// outstanding global->LDS load (vmcnt 0) and serialise the ring.  Ordering of LDS traffic is by
// construction: a wave waits for its own loads of the stage (s_waitcnt vmcnt) before the barrier,
// and for its own LDS reads of the stage before.  The asm statements stop the compiler from moving memory
// accesses across.
__device__ __forceinline__ void ring_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// the same without a wait for the wave's own LDS reads, where those that are still under way read nothing that is about to be
// overwritten
__device__ __forceinline__ void bare_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// One LDS-DMA request: every lane's 16 bytes at `src` go to LDS at dst + lane * 16 (dst is the same
// in all lanes of the wave).  Written as an instruction the compiler does not interpret: for the
// builtin it keeps its own account of which request has landed, cannot relate the ring's counted
// waits to the conditional refills, and puts a wait for everything in flight in front of the
// stages' LDS reads (and in front of the loop, for the query registers).  Here every wait is the
// ring's own: a stage's wait and barrier come before any read of its slot, and each of these
// statements is a compiler barrier for memory accesses.
__device__ __forceinline__ void lds_dma_b128(const CB_GLOBAL char* src, CB_LDS uint4* dst) {
  const uint32_t base = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)dst);
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(base) : "memory");
}

// the same with the address as a uniform base and a 32-bit offset per lane; `lanes`: the lanes that take part, all or
// none (a request that is sometimes left out without a branch; called with all lanes of the wave active)
__device__ __forceinline__ void lds_dma_b128(const CB_GLOBAL char* base, uint32_t off, CB_LDS uint4* dst, bool lanes) {
  const uint32_t lds = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)dst);
  // (readfirstlane returns a signed int: the halves are made unsigned before they are put together)
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(uintptr_t)base);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uintptr_t)base >> 32));
  const uint64_t b64 = (uint64_t)lo | ((uint64_t)hi << 32);
  const int mask = __builtin_amdgcn_readfirstlane(lanes ? -1 : 0);
  // (a load may read a scalar register that a vector instruction wrote -- the base, where it comes from a readfirstlane --
  // five wait states later at the earliest, and inside an asm statement nobody else counts them: three moves and s_nop 1)
  asm volatile("s_mov_b32 m0, %2\n\ts_mov_b32 exec_lo, %3\n\ts_mov_b32 exec_hi, %3\n\ts_nop 1\n\tglobal_load_lds_dwordx4 %0, %1\n\ts_mov_b64 exec, -1"
               ::"v"(off), "s"(b64), "s"(lds), "s"(mask) : "memory");
}

// and with the address in LDS as a number, uniform
__device__ __forceinline__ void lds_dma_b128_at(const CB_GLOBAL char* src, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(lds) : "memory");
}

__device__ __forceinline__ void lds_dma_b32(const CB_GLOBAL int32_t* src, CB_LDS int* dst) {  // (dst + lane * 4)
  const uint32_t base = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)dst);
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off" ::"v"(src), "s"(base) : "memory");
}

// Forces every field of the argument block into scalar registers here and now: the empty asm
// statements take each value as an in/out operand, so the loads cannot be sunk past this point.  (Left to itself the
// compiler loads each near its first use, behind early exits, and the chain of dependent scalar loads then costs
// several microseconds before the first K/V request goes out.)
#define CB_PIN(x) asm volatile("" : "+s"(x))
__device__ __forceinline__ void pin_args(AttnParams& p) {
  CB_PIN(p.q); CB_PIN(p.out); CB_PIN(p.kv.k); CB_PIN(p.kv.v); CB_PIN(p.kv.block_table);
  CB_PIN(p.kv.seq_stride); CB_PIN(p.kv.token_stride); CB_PIN(p.kv.head_stride); CB_PIN(p.kv.num_blocks);
  CB_PIN(p.kv.max_blocks); CB_PIN(p.kv.block_size); CB_PIN(p.parent); CB_PIN(p.partial); CB_PIN(p.tickets); CB_PIN(p.coop_tickets);
  CB_PIN(p.Hq); CB_PIN(p.Hkv); CB_PIN(p.chunk); CB_PIN(p.nsplit); CB_PIN(p.batch); CB_PIN(p.scale);
  CB_PIN(p.external_merge); CB_PIN(p.max_depth); CB_PIN(p.xcd_remap); CB_PIN(p.grid_x); CB_PIN(p.grid_y); CB_PIN(p.grid_z); CB_PIN(p.coop_merge); CB_PIN(p.spin_limit);
  CB_PIN(p.status); CB_PIN(p.dbg_ts);
}
#undef CB_PIN

constexpr int kUnitKeys = 32;  // keys per unit: what one wave works on at a time, and the granularity of the LDS ring

// Partial softmax state, one block per (TR-row tile, split), laid out in the order the MFMA accumulators hold it (TR = 32
// or 16, the query columns of an accumulator tile).  Piece pc of the tile holds DP = 256 / TR dims from DP pc: lane (h, r),
// r = lane % TR, has o[row r][DP pc + 4 h + {0..3}], unnormalised, relative to the reference weight, as bf16 (8 bytes) or,
// PX, as fp32 (16 bytes).  A lane's pieces are stored in vectors of 16 bytes (one piece, or two as bf16), the lanes'
// vectors next to each other, so that a wave's store or load is 1024 contiguous bytes; then (m, l) as fp32 for each
// of the rows.  (With 8 bytes per lane, and rounded by integer
// instructions, the tail of a 256-row tile's workgroup from its sweep to its merge was 8.5 us at 15 splits, and is 7.0.)
// The blocks of sequence b start at tile block_tile0(b); kv head hk's row tile ti is block
// (hk * ceil(M_b / TR) + ti) * nsplit + split behind it.
//
// PX: the kernels' builds for calls that hold probabilities and partial sums in 32 bits (precise_sums() of the host side).
// A probability goes to the matrix cores as two bf16 terms, the rounded value and the rounded rest (together within 2^-17
// of the fp32 value), the denominator is the sum of both, and the partial states are fp32.
template <int D, int TR, bool PX>
struct PartialLayout {
  static constexpr int DP = 256 / TR;
  static constexpr int P = D / DP;  // pieces per tile
  static constexpr int kPer = PX ? 1 : 2;    // pieces to a vector
  static constexpr int kVec = 64 * 16;       // bytes of the lanes' vectors
  static constexpr int kMl = P / kPer * kVec;
  static constexpr int kBytes = kMl + TR * 8;
};
// first tile of a sequence whose nodes start at `off`: room for ceil(M_b / TR) tiles per kv
// head without a prefix sum over the sequences' tile counts
template <int TR>
__host__ __device__ __forceinline__ int64_t block_tile0(int64_t off, int Hq, int Hkv, int b) {
  return off * Hq / TR + (int64_t)(Hkv + 1) * b;
}

constexpr float kRescaleSlack = 8.0f;  // log2 units the running maximum may exceed the reference

// v_maximum3_f32: unlike fmaxf() it needs no canonicalised operands
__device__ __forceinline__ float maxn(float a, float b) { return __builtin_elementwise_maximum(a, b); }

// Which 16-byte piece of a row lands where is XORed with a value of the row so that the operand reads are free of
// bank conflicts (LDS serves 256 bytes per clock: 16 lanes of a ds_read_b128 -- K: 16 rows, one piece each -- or 32 of a
// ds_read_b64_tr_b16 -- V: 4 rows, 64 bytes of each, with the 32-row tiles; 8 rows, 32 bytes of each, with the 16-row ones).
template <int D>
__device__ __forceinline__ int swizzle_k(int row) { return D == 128 ? row & 15 : (row >> 1) & 7; }
template <int D, int TR>
__device__ __forceinline__ int swizzle_v(int row) {
  if (TR == 16) return D == 128 ? (row & 7) << 1 : ((row >> 1) & 3) << 1;
  return D == 128 ? (row & 3) << 2 : ((row >> 1) & 1) << 2;
}

// One workgroup's (tile, split) as the kernel's arguments and the workgroup's number give it; uniform.
struct TileJob {
  int b, hk, g;        // sequence, kv head, query heads per kv head
  int off, N, S, M;    // the sequence's first node, nodes, prefix; its rows per kv head
  int rt, tiles;       // row tile, row tiles per kv head of the launch
  int row0;            // first row of the tile
  int split, nsplit;   // and the sequence's number of splits
  int k0, k1;          // the split's keys
  int layer;           // of those that the launch serves
};

template <typename Layers>
__device__ __forceinline__ bool tile_job(const AttnParams& p, const SeqMetaLanes& ml, int d, int tile_rows, const Layers& layers, TileJob& j) {
  // Workgroups are handed to the 8 XCDs round-robin in dispatch order.  With xcd_remap the
  // dispatch index d is renumbered to j = (d % 8) * (T / 8) + d / 8, so that consecutive j --
  // in particular all splits of one (sequence, kv head, row tile) -- sit on the same XCD and
  // meet in its L2.  Tiles are numbered with the sequence running fastest: an XCD's share of the
  // tiles (a contiguous range of j) then holds a few heads of every sequence rather than every
  // head of a few sequences, so a batch of unequal lengths loads the XCDs equally.
  int by;
  j.tiles = p.grid_y / p.Hkv;
  j.g = p.Hq / p.Hkv;
  j.layer = 0;
  if constexpr (Layers::kMany) {  // (one layer behind the other; a layer's workgroups are a multiple of 8 where they are renumbered)
    if (p.xcd_remap != 2) {
      j.layer = d / layers.wgs;
      d -= j.layer * layers.wgs;
    }
  }
  if (p.xcd_remap == 2) {
    // XCD x = d % 8 works through position r = d / 8 of its own list: all splits of a tile together,
    // the tiles of one sequence together, the sequences from the longest to the shortest -- so the
    // workgroups that are dispatched last, and decide when the launch ends, are the short ones.  The
    // XCD's tiles are those of the same Hkv / 8 kv heads of every sequence.  Only workgroups that have keys are listed:
    // ones that leave at once still take their turn among the compute units, and the others then pile up on some (8 sequences
    // of 100 to 2000 keys in 192 workgroups and 64 empty ones, beside 56 that do logits: 49.5 us, without the empty ones 37).
    const int x = d & 7, r = d >> 3;
    const int i = __popcll(__builtin_amdgcn_ballot_w64(ml.start <= r)) - 1;  // (starts past the batch are INT_MAX)
    j.b = __builtin_amdgcn_readlane(ml.ord, i);
    const SeqShape s = seq_shape(ml, j.b);
    const int at = r - __builtin_amdgcn_readlane(ml.start, i);
    const int splits = (s.S + s.N + p.chunk - 1) / p.chunk, tiles = (s.N * j.g + tile_rows - 1) / tile_rows;
    j.split = at % splits;
    const int tile = at / splits;
    int head = tile / tiles;
    if constexpr (Layers::kMany) {  // (a sequence's tiles of all layers: the last workgroups are still the shortest)
      j.layer = head / (p.Hkv >> 3);
      head -= j.layer * (p.Hkv >> 3);
    }
    by = (x * (p.Hkv >> 3) + head) * j.tiles + tile % tiles;
  } else if (p.xcd_remap == 3) {
    const int x = d & 7, r = d >> 3, ypx = p.grid_y >> 3, tile = r / p.grid_x;
    j.split = r % p.grid_x;
    by = x * ypx + tile % ypx;
    j.b = __builtin_amdgcn_readlane(ml.ord, tile / ypx);
  } else {
    const int T = p.grid_x * p.grid_y * p.grid_z;
    const int n = p.xcd_remap ? (d & 7) * (T >> 3) + (d >> 3) : d;
    j.split = n % p.grid_x;
    const int rest = n / p.grid_x;
    j.b = rest % p.grid_z;
    by = rest / p.grid_z;
  }
  // (row tiles of one kv head are neighbours: they sweep the same K/V and then share an XCD's L2)
  j.rt = by % j.tiles;
  j.hk = by / j.tiles;
  const SeqShape shp = seq_shape(ml, j.b);
  j.off = shp.off;
  j.N = shp.N;
  j.S = shp.S;
  j.M = shp.N * j.g;
  j.row0 = j.rt * tile_rows;
  const int len = shp.S + shp.N;
  j.k0 = j.split * p.chunk;
  if (j.row0 >= j.M || j.k0 >= len) return false;
  j.k1 = (j.k0 + p.chunk < len) ? j.k0 + p.chunk : len;
  j.nsplit = (len + p.chunk - 1) / p.chunk;
  return true;
}

// The layer's pointers, scratch memory and tickets in the place of the launch's.
template <typename Layers>
__device__ __forceinline__ void take_layer(AttnParams& p, const TileJob& j, const Layers& layers) {
  if constexpr (Layers::kMany) {
    const int i = __builtin_amdgcn_readfirstlane(j.layer);
    p.q = layers.at[i].q;
    p.out = layers.at[i].out;
    p.kv.k = layers.at[i].k;
    p.kv.v = layers.at[i].v;
    p.partial = reinterpret_cast<float*>(reinterpret_cast<char*>(p.partial) + i * layers.partial_bytes);
    p.tickets += (int64_t)i * layers.tiles * 4;
    p.coop_tickets += (int64_t)i * layers.tiles * (kCoopTicketStride / 4);
    asm volatile("" : "+s"(p.q), "+s"(p.out), "+s"(p.kv.k), "+s"(p.kv.v), "+s"(p.partial), "+s"(p.tickets), "+s"(p.coop_tickets));
  }
}

// Timing aid: the stamps go to LDS and are copied out when the kernel ends -- a store to memory inside, even one that
// never executes, makes the compiler treat the loads in flight as unordered and wait for all of them wherever it needs
// one.  (TS: the timeline build of the kernels, a measurement aid; every stamp is compiled out of the kernels that ship
// as the default.)
template <bool TS>
__device__ __forceinline__ void first_stamps(CB_LDS unsigned long long* ts, unsigned long long ts0) {
  if (!TS || threadIdx.x != 0) return;
#pragma unroll
  for (int i = 2; i < 16; i++) ts[i] = 0;
  ts[0] = ts0;
  ts[1] = wall_clock64();
}

// Buffer descriptor over a sequence's partials (byte offsets fit 32 bits, checked by the launcher), and the byte
// offset of split 0's block of the tile's i-th TR-row tile.
template <int D, int TR, bool PX>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t partial_rsrc(const AttnParams& p, const TileJob& jb) {
  return __builtin_amdgcn_make_buffer_rsrc(
      reinterpret_cast<char*>(p.partial) + block_tile0<TR>(jb.off, p.Hq, p.Hkv, jb.b) * p.nsplit * PartialLayout<D, TR, PX>::kBytes, 0, 0x7fffffff, 0x00020000);
}
template <int D, int TR, bool PX>
__device__ __forceinline__ uint32_t partial_byte(const AttnParams& p, const TileJob& jb, int i) {
  return (uint32_t)(jb.hk * ((jb.M + TR - 1) / TR) + jb.row0 / TR + i) * (uint32_t)p.nsplit * (uint32_t)PartialLayout<D, TR, PX>::kBytes;
}

// LDS of a workgroup beside the ring
struct TileLds {
  int bt[kBtLds];
  AncScratch anc;  // ancestor sets of the whole tree, built here by the splits that reach the tree
  int flag, flag2;                    // merge verdicts (see split_merge)
  unsigned long long todo, todo2;
};

// The memory side of a workgroup's sweep: units of 32 keys (K and V) of one split, requested by LDS-DMA into a ring of
// kSlots, and what every wave brings of each.  Units are requested in order, unit u into slot u % kSlots.  CONTIGUOUS: the cache is, and
// nothing of a block table is in the code.
template <int D, int NW, int TR, bool CONTIGUOUS = false>
struct Feed {
  static constexpr int kVecs = kUnitKeys * D / 8;               // 16-byte pieces of a unit's K (or V)
  static constexpr int kSlots = D == 128 ? 9 : 16;              // ring depth in units (16 or 8 KiB each)
  static constexpr int kPrologue = D == 128 ? 6 : 10;           // units requested before the first wait
  static constexpr int kReq = 2 * kVecs / 64 / NW;              // requests per wave and unit
  static constexpr int kRingVecs = kSlots * 2 * kVecs;
  static constexpr uint32_t kSlotBytes = 2 * kVecs * 16;
  static constexpr int VPR = D / 8;                             // 16-byte pieces per row
  static constexpr int RPR = 64 / VPR;                          // rows per request
  static constexpr int kParts = kReq >= 2 ? kReq / 2 : 1;       // groups of RPR rows per wave and unit
  static_assert(kReq >= 1 && kReq * kSlots < 63, "");
  const AttnParams& p;
  const TileJob& jb;
  int* const bt;        // LDS ring of the split's block-table slice
  uint4* const ring;
  const int w, l;       // wave (uniform), lane
  const CB_GLOBAL char* const kbase;
  const CB_GLOBAL char* const vbase;
  const CB_GLOBAL int32_t* const gbt;
  KeyAddr<CONTIGUOUS> ka;
  int bt_seg = 1;       // furthest segment of the table slice that the requests have entered (the first kBtSegs are loaded at the start)
  bool even;            // see issue()
  bool long_slice = false;  // paged: more table entries than the LDS ring holds
  int64_t ts2;
  uint32_t lane_k[kParts], lane_v[kParts];
  int requested = 0, slot_next = 0;
  // Paged and `even`: the block-table entries (uniform) of the next two units' groups.  Read where they are needed, an LDS round trip held
  // up every request; with it and 64-bit scalars (group_off) 20 nodes of 32 heads x 9000 paged keys took 36.3 us a step, without 33.6, and
  // contiguous ones 29.9 and 29.0.
  int ahead[2][kParts];

  __device__ __forceinline__ Feed(const AttnParams& p_, const TileJob& jb_, int* bt_, uint4* ring_)
      : p(p_), jb(jb_), bt(bt_), ring(ring_), w(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)), l(threadIdx.x & 63),
        kbase((const CB_GLOBAL char*)p_.kv.k), vbase((const CB_GLOBAL char*)p_.kv.v), gbt((const CB_GLOBAL int32_t*)p_.kv.block_table) {
    ka.kv = &p.kv;
    ka.bt = bt;
    ka.bt_first = 0;
    ka.bs_shift = 0;
    ka.seq = jb.b;
    ka.head = jb.hk;
    if (paged()) {  // the launcher guarantees a power-of-two block size
      ka.bs_shift = 31 - __clz(p.kv.block_size);
      const int first = jb.k0 >> ka.bs_shift, last = (jb.k1 - 1) >> ka.bs_shift;
      for (int i = threadIdx.x; i <= last - first && i < kBtLds; i += 64 * NW)
        bt[i] = gbt[(int64_t)jb.b * p.kv.max_blocks + first + i];
      ka.bt_first = first;
      long_slice = last - first >= kBtLds;
      __syncthreads();  // the K/V addresses below depend on it
    }
    even = !paged() || p.kv.block_size >= RPR;
    ts2 = p.kv.token_stride * 2;
    const int lr = l / VPR, lc = l % VPR;
#pragma unroll
    for (int i = 0; i < kParts; i++) {
      const int rr = part_row(i) + lr;
      lane_k[i] = (uint32_t)(lr * (int)ts2) + (uint32_t)(lc ^ swizzle_k<D>(rr)) * 16;
      lane_v[i] = (uint32_t)(lr * (int)ts2) + (uint32_t)(lc ^ swizzle_v<D, TR>(rr)) * 16;
    }
#pragma unroll
    for (int i = 0; i < kParts; i++) ahead[0][i] = ahead[1][i] = 0;
    if (paged() && even) {
      look_up(0, ahead[0]);
      look_up(1, ahead[1]);
    }
  }
  __device__ __forceinline__ bool paged() const { return !CONTIGUOUS && p.kv.block_size > 0; }
  __device__ __forceinline__ const uint4* k_at(int slot) const { return ring + slot * (2 * kVecs); }
  __device__ __forceinline__ const uint4* v_at(int slot) const { return ring + slot * (2 * kVecs) + kVecs; }
  // Every wave brings the same rows of K and of V (of one of the two, where a wave makes a single request per unit).
  __device__ __forceinline__ int part_row(int part) const { return (kReq >= 2 ? w * kParts + part : w % (NW / 2)) * RPR; }
  __device__ __forceinline__ void look_up(int u, int (&entry)[kParts]) const {
#pragma unroll
    for (int i = 0; i < kParts; i++) entry[i] = bt[(((jb.k0 + u * kUnitKeys + part_row(i)) >> ka.bs_shift) - ka.bt_first) & (kBtLds - 1)];
  }
  __device__ __forceinline__ int64_t group_off(int u, int part) const {  // byte offset of the group's first row (uniform; `even` only)
    const int key = jb.k0 + u * kUnitKeys + part_row(part);
    // (pool sizes, keys and a row's stride have 32 bits: comparisons and products of 64-bit scalars are several instructions each)
    if (paged()) {
      int blk = __builtin_amdgcn_readfirstlane(ahead[0][part]);  // (of the unit that is next)
      blk = blk < 0 ? 0 : (blk >= (int)p.kv.num_blocks ? (int)p.kv.num_blocks - 1 : blk);
      return (int64_t)((uint64_t)(uint32_t)blk * (uint64_t)(p.kv.seq_stride * 2)) +
             (int64_t)((uint64_t)(uint32_t)(key & (p.kv.block_size - 1)) * (uint32_t)ts2) + (int64_t)jb.hk * p.kv.head_stride * 2;
    }
    return ((int64_t)jb.b * p.kv.seq_stride + (int64_t)jb.hk * p.kv.head_stride) * 2 + (int64_t)((uint64_t)(uint32_t)key * (uint32_t)ts2);
  }
  __device__ __forceinline__ void issue_group(int slot, int part, int64_t off, bool lanes) const {
    uint4* const kdst = ring + slot * (2 * kVecs) + part_row(part) * VPR;
    if (kReq >= 2 || w < NW / 2) lds_dma_b128(kbase + off, lane_k[part], (CB_LDS uint4*)kdst, lanes);
    if (kReq >= 2 || w >= NW / 2) lds_dma_b128(vbase + off, lane_v[part], (CB_LDS uint4*)kdst + kVecs, lanes);
  }
  // One unit's requests.  A group's rows are evenly spaced in memory in a contiguous cache, and in a paged one whose
  // blocks hold whole groups; then a request can be a uniform base and a lane offset that never changes.  Otherwise, and in
  // the unit that runs past the split's end, every lane works out its own row; keys past the end repeat the last one
  // (masked later), so every address stays inside the split's own range.
  // The uniform form is the faster one: 58 against 62 us at 32 heads x 16384 keys.  (The wide kernel has requests of its own.)
  __device__ __forceinline__ void issue(int u, int slot) const {
    const bool whole = jb.k0 + (u + 1) * kUnitKeys <= jb.k1;
    const int lr = l / VPR, lc = l % VPR;
#pragma unroll
    for (int i = 0; i < kParts; i++) {
      if (even && whole) {
        issue_group(slot, i, group_off(u, i), true);
      } else {
        const int rr = part_row(i) + lr;
        int key = jb.k0 + u * kUnitKeys + rr;
        key = key > jb.k1 - 1 ? jb.k1 - 1 : key;
        const int64_t off = ka.byte_off(key);
        uint4* const kdst = ring + slot * (2 * kVecs) + part_row(i) * VPR;
        if (kReq >= 2 || w < NW / 2) lds_dma_b128(kbase + off + (lc ^ swizzle_k<D>(rr)) * 16, (CB_LDS uint4*)kdst);
        if (kReq >= 2 || w >= NW / 2) lds_dma_b128(vbase + off + (lc ^ swizzle_v<D, TR>(rr)) * 16, (CB_LDS uint4*)kdst + kVecs);
      }
    }
  }
  // Before unit u of a paged cache is requested: entering segment q of the split's table slice requests
  // segment q + 2 (its ring place held q - 2), a dword per lane of the first waves.  (An extra request among those
  // in flight only makes the counted waits stricter.)
  __device__ __forceinline__ void bt_ahead(int u) {
    const int last_blk = (jb.k1 - 1) >> ka.bs_shift;
    int key = jb.k0 + (u + 1) * kUnitKeys - 1;
    key = key > jb.k1 - 1 ? jb.k1 - 1 : key;
    const int q = ((key >> ka.bs_shift) - ka.bt_first) / kBtSeg;
    if (q <= bt_seg) return;
    bt_seg = q;
    const int seg = q + 2;
    if (seg < kBtSegs || ka.bt_first + seg * kBtSeg > last_blk || w >= kBtSeg / 64) return;
    const int i = seg * kBtSeg + 64 * w + l;
    const int blk = ka.bt_first + i > last_blk ? last_blk : ka.bt_first + i;
    lds_dma_b32(gbt + (int64_t)jb.b * p.kv.max_blocks + blk, (CB_LDS int*)bt + ((seg * kBtSeg + 64 * w) & (kBtLds - 1)));
  }
  __device__ __forceinline__ void request_up_to(int limit) {
    while (requested < limit) {
      if (!CONTIGUOUS && long_slice) bt_ahead(requested);
      issue(requested, slot_next);
      counted();
    }
  }
  __device__ __forceinline__ void counted() {
    slot_next = slot_next + 1 == kSlots ? 0 : slot_next + 1;
    requested++;
    if (paged() && even) {
#pragma unroll
      for (int i = 0; i < kParts; i++) ahead[0][i] = ahead[1][i];
      look_up(requested + 1, ahead[1]);
    }
  }
  // Waits until the first `landed` units are in LDS, in this wave's share and, behind the barrier, in every wave's.
  // Requests complete in order, so "at most n requests outstanding" means that all but the youngest n have landed.
  __device__ __forceinline__ void wait_units(int landed) const {
    const int younger = requested - landed;
#define CB_W(n) if (younger >= n) { wait_vmcnt<kReq * n>(); break; }
    do {
      if constexpr (kSlots > 10) { CB_W(14) CB_W(12) CB_W(10) }
      CB_W(8) CB_W(7) CB_W(6) CB_W(5) CB_W(4) CB_W(3) CB_W(2) CB_W(1) wait_vmcnt<0>();
    } while (0);
#undef CB_W
    ring_barrier();
  }
};

// A lane's output row: NP pieces from pc0 (both even), scaled.  With 32-row tiles two lanes of a row exchange halves
// first, so that a lane has 8 dims in a row and stores 16 bytes.
template <int D, int TR, int NP>
__device__ __forceinline__ void store_row(CB_GLOBAL uint16_t* gout, int64_t grow, const floatx4 (&f)[NP], int pc0, float inv, int l) {
  constexpr int DP = 256 / TR;
  const int h = l / TR;
  uintx2 pk[NP];
#pragma unroll
  for (int n = 0; n < NP; n++) {
    pk[n][0] = pack_bf16(f[n][0] * inv, f[n][1] * inv);
    pk[n][1] = pack_bf16(f[n][2] * inv, f[n][3] * inv);
  }
  CB_GLOBAL uint16_t* orow = gout + grow * D;
  if constexpr (TR == 32) {
    static_assert(NP % 2 == 0, "");
#pragma unroll
    for (int n = 0; n < NP; n += 2) {
      // (swaps the first operand's upper 32 lanes with the second's lower ones)
      const auto a = __builtin_amdgcn_permlane32_swap(pk[n][0], pk[n + 1][0], false, false);
      const auto b = __builtin_amdgcn_permlane32_swap(pk[n][1], pk[n + 1][1], false, false);
      const uintx4 v = {a[0], b[0], a[1], b[1]};
      if (grow >= 0) *(CB_GLOBAL uintx4*)(orow + DP * (pc0 + n) + 8 * h) = v;
    }
  } else {
    if (grow < 0) return;
#pragma unroll
    for (int n = 0; n < NP; n++) *(CB_GLOBAL uintx2*)(orow + DP * (pc0 + n) + 4 * h) = pk[n];
  }
}

// Merge of NP pieces (from pc0) of one TR-row tile's partials by one wave: every lane merges the elements that the
// layout gives it, so each load of the wave is contiguous (`byte`: offset of slot 0's block).  Slots are
// combined online, BS per batch with all of a batch's loads in flight together: m = max m_t, w_t = 2^(m_t - m),
// o = sum w_t o_t / sum w_t l_t (m_t is stored in log2 units).  POL is the buffer cache policy of
// the loads.  A slot that saw no visible key carries m_t = -inf, l_t = 0 and gets weight 0; the
// reference is kept finite so that (-inf) - (-inf) never occurs.  grow: the lane's output row, or -1.
template <int D, int TR, bool PX, int NP, int POL, int BS>
__device__ __forceinline__ void merge_pieces(__amdgpu_buffer_rsrc_t prsrc, int64_t grow, uint32_t byte, CB_GLOBAL uint16_t* gout,
                                             int nslots, int pc0, int l) {
  using Part = PartialLayout<D, TR, PX>;
  constexpr int NV = NP / Part::kPer;  // vectors
  static_assert(NP % Part::kPer == 0, "");
  const int r = l % TR;
  floatx4 acc[NP];
#pragma unroll
  for (int i = 0; i < NP; i++) acc[i] = floatx4{0.f, 0.f, 0.f, 0.f};
  float lsum = 0.f, m_run = -3.0e38f;
  // (the slot's offset is the same in all lanes: it travels as the load's scalar offset, so a
  // load costs no vector arithmetic)
  const uint32_t vo_ml = byte + Part::kMl + r * 8, vo_v = byte + pc0 / Part::kPer * Part::kVec + l * 16;
  for (int t0 = 0; t0 < nslots; t0 += BS) {
    uintx4 v[BS][NV];
    uintx2 ml[BS];
#pragma unroll
    for (int u = 0; u < BS; u++) {
      const int t = (t0 + u < nslots) ? t0 + u : nslots - 1;  // (a repeated slot: weight 0 below)
      ml[u] = __builtin_amdgcn_raw_buffer_load_b64(prsrc, vo_ml, t * Part::kBytes, POL);
#pragma unroll
      for (int i = 0; i < NV; i++) v[u][i] = __builtin_amdgcn_raw_buffer_load_b128(prsrc, vo_v + i * Part::kVec, t * Part::kBytes, POL);
    }
    // (all of the batch's loads are requested before anything looks at a result: left alone, the
    // scheduler moves the first maxima up between the loads, and each then waits a round trip)
    __builtin_amdgcn_sched_barrier(0);
    float m_new = m_run;
#pragma unroll
    for (int u = 0; u < BS; u++) m_new = fmaxf(m_new, __uint_as_float(ml[u][0]));
    if (t0 > 0) {  // (uniform)
      const float resc = __builtin_amdgcn_exp2f(m_run - m_new);
#pragma unroll
      for (int i = 0; i < NP; i++) acc[i] *= resc;
      lsum *= resc;
    }
    m_run = m_new;
#pragma unroll
    for (int u = 0; u < BS; u++) {
      float wgt = __builtin_amdgcn_exp2f(__uint_as_float(ml[u][0]) - m_new);
      wgt = (t0 + u < nslots) ? wgt : 0.f;
      lsum = fmaf(__uint_as_float(ml[u][1]), wgt, lsum);
#pragma unroll
      for (int i = 0; i < NP; i++) {
        if constexpr (PX) {
#pragma unroll
          for (int x = 0; x < 4; x++) acc[i][x] = fmaf(__uint_as_float(v[u][i][x]), wgt, acc[i][x]);
        } else {
          const uint32_t lo = v[u][i / 2][2 * (i & 1)], hi = v[u][i / 2][2 * (i & 1) + 1];
          acc[i][0] = fmaf(__uint_as_float(lo << 16), wgt, acc[i][0]);
          acc[i][1] = fmaf(__uint_as_float(lo & 0xffff0000u), wgt, acc[i][1]);
          acc[i][2] = fmaf(__uint_as_float(hi << 16), wgt, acc[i][2]);
          acc[i][3] = fmaf(__uint_as_float(hi & 0xffff0000u), wgt, acc[i][3]);
        }
      }
    }
  }
  store_row<D, TR, NP>(gout, grow, acc, pc0, PX ? 1.0f / lsum : __builtin_amdgcn_rcpf(lsum), l);
}

// Split merge of a tile inside the launch.  The partials of the sweeps are write-through stores; once they have
// completed (vmcnt 0) the workgroup takes a ticket with a device-scope atomic.  No cache-wide write-back or
// invalidate is involved (a __threadfence() per workgroup costs a full L2 sweep on this chip).
//
// Ticket word of a tile (64 bits, zero between launches): arrivals in bits 0-11 and, to learn
// whether every split ran on one XCD, the sum (bits 24-39) and the sum of squares (bits 40-59)
// of the arrivals' XCC_ID (hardware register 20, bits 3:0): all ids equal mine  <=>
// sum = n*id and sumsq = n*id*id.  A second word per tile holds one bit per split whose
// workgroup gave up waiting (cooperative merge only).
// aside(): what the first wave has to do beside, where it would wait for the other splits, or, in the merge by the last to arrive, behind its
// share of that.
template <int D, int TR, bool PX, int NW, int MAXROWS, bool TS, typename Aside>
__device__ __forceinline__ void split_merge(const AttnParams& p, const TileJob& jb, int tile_rows, TileLds& sh, CB_LDS unsigned long long* ts, Aside aside) {
  constexpr int P = PartialLayout<D, TR, PX>::P;
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
  const bool do_ts = TS && tid == 0, do_ts64 = TS && tid == 64;
#define CB_TS(i) do { if (do_ts) ts[i] = wall_clock64(); } while (0)
  CB_GLOBAL uint16_t* gout = (CB_GLOBAL uint16_t*)p.out;
  const __amdgpu_buffer_rsrc_t prsrc = partial_rsrc<D, TR, PX>(p, jb);
  if (tid == 64) { sh.flag = 0; sh.flag2 = 0; }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  CB_TS(5);
  // (cooperative merge: the tiles' words are polled, so each tile has a 4 KiB stretch of its own
  // in a separate area -- neighbours in one line would all be served by one memory channel)
  const int64_t tile_id = ((int64_t)jb.b * p.Hkv + jb.hk) * jb.tiles + jb.rt;
  CB_GLOBAL unsigned long long* ticket = p.coop_merge ? (CB_GLOBAL unsigned long long*)p.coop_tickets + tile_id * (kCoopTicketStride / 8)
                                                      : (CB_GLOBAL unsigned long long*)p.tickets + 2 * tile_id;
  constexpr unsigned long long kArrivals = 0xfffull;
  const unsigned long long xcc = __builtin_amdgcn_s_getreg(20 | (0 << 6) | ((4 - 1) << 11)) & 15u;
  const unsigned long long arrive = 1ull | (xcc << 24) | ((xcc * xcc) << 40);
  const int nsplit = jb.nsplit, split = jb.split;
  auto one_xcd = [&](unsigned long long tot) {
    const unsigned long long n = tot & kArrivals, sum = (tot >> 24) & 0xffffull, sumsq = tot >> 40;
    return sum == n * xcc && sumsq == n * xcc * xcc;
  };
  // TR-row tile i of the tile: whether it holds rows, and the lane's output row (-1 past the end)
  auto tile_row = [&](int i, int64_t* gr) {
    const int row = jb.row0 + i * TR + l % TR;
    const int node = row / jb.g, hg = row - node * jb.g;
    *gr = row < jb.M ? (int64_t)(jb.off + node) * p.Hq + jb.hk * jb.g + hg : -1;
    return row - l % TR < jb.M && (MAXROWS <= 64 || i * TR < tile_rows);
  };

  if (!p.coop_merge) {
    // Merge by the last workgroup of the tile to arrive: the others leave at once and free their
    // compute units (grids of several rounds of workgroups).
    if (tid == 0) {
      const unsigned long long tot = __hip_atomic_fetch_add(ticket, arrive, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + arrive;
      int flag = ((tot & kArrivals) == (unsigned long long)nsplit) ? 1 : 0;
      if (flag) {
        if (!one_xcd(tot)) {
          flag = 2;  // some split ran on another XCD: its partials are not in this L2
          __hip_atomic_fetch_or((CB_GLOBAL int32_t*)p.status, 16, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __hip_atomic_store(ticket, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // ready for the next launch
      }
      sh.flag = flag;
    }
    __syncthreads();
    CB_TS(6);
    const int flag = sh.flag;
    // Same XCD: the write-through stores left the lines in this L2, plain (cached) loads are coherent
    // with them.  Otherwise read past the L2 with agent-coherent loads.
    constexpr int NP = 4, BS = PX ? 4 : 8;
    for (int u = flag ? w : MAXROWS; u < MAXROWS / TR * (P / NP); u += NW) {
      const int i = u / (P / NP);
      int64_t gr;
      if (!tile_row(i, &gr)) break;  // (nothing behind it either)
      const uint32_t byte = partial_byte<D, TR, PX>(p, jb, i);
      if (flag == 1) merge_pieces<D, TR, PX, NP, 0, BS>(prsrc, gr, byte, gout, nsplit, (u % (P / NP)) * NP, l);
      else merge_pieces<D, TR, PX, NP, kAgentCoherent, BS>(prsrc, gr, byte, gout, nsplit, (u % (P / NP)) * NP, l);
    }
    if (w == 0) aside();
    if (!flag) return;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    CB_TS(7);
    return;
  }

  // ---- cooperative merge (the whole grid is resident at once: one round of workgroups).  Every
  // workgroup of the tile merges a slice of it -- the (TR-row tile, piece) units u
  // with u % nsplit == split -- once all splits have arrived, so no compute unit has to pull the whole
  // tile's partials through its own memory pipe.  Thread 64 arrives and then polls the ticket, at
  // most spin_limit times: the tile is complete when the arrivals equal nsplit, or when the word
  // is zero again (the completing workgroup zeroes it for the next launch; after one's own arrival
  // it cannot be zero for any other reason).  A workgroup that gives up sets its bit in the tile's
  // second word, looks at the ticket once more and leaves if the tile is still incomplete: the
  // completing workgroup reads that word after its own arrival, so it finds the bit and merges the
  // slice.  (If the last look shows the tile complete after all, the workgroup merges its slice
  // itself: the completing workgroup may have read the word before the bit was there.  If both
  // merge it they write the same bytes.)
  CB_GLOBAL unsigned long long* gave_up = ticket + 1;
  if (tid == 64) {
    unsigned long long tot = __hip_atomic_fetch_add(ticket, arrive, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + arrive;
    const bool completes = (tot & kArrivals) == (unsigned long long)nsplit;
    auto complete = [&](unsigned long long t) { return (t & kArrivals) == (unsigned long long)nsplit || t == 0ull; };
    for (int spin = 0; !complete(tot) && spin < p.spin_limit; spin++) {
      __builtin_amdgcn_s_sleep(2);
      tot = __hip_atomic_load(ticket, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    unsigned long long todo = 1ull << split, todo2 = 0;
    bool own_bit = false;
    if (!complete(tot)) {
      // (the returning form: the bit is in memory before the ticket is looked at again)
      const unsigned long long before = __hip_atomic_fetch_or(gave_up, 1ull << split, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      asm volatile("s_waitcnt vmcnt(0)" ::"v"(before) : "memory");
      tot = __hip_atomic_load(ticket, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      own_bit = true;
      if (!complete(tot)) todo = 0;
      __hip_atomic_fetch_or((CB_GLOBAL int32_t*)p.status, 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // plain loads only when the ticket itself says that every split ran on this XCD
    int flag = (tot != 0ull && one_xcd(tot)) ? 1 : 2;
    if (todo != 0 && flag == 2) __hip_atomic_fetch_or((CB_GLOBAL int32_t*)p.status, 16, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    sh.todo = todo;
    __hip_atomic_store(&sh.flag, flag, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (do_ts64) ts[6] = wall_clock64();
    if (completes) {
      todo2 = __hip_atomic_load(gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & ~todo;
      if (todo2 != 0) __hip_atomic_store(gave_up, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(ticket, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // ready for the next launch
    } else if (own_bit && todo != 0) {
      __hip_atomic_fetch_and(gave_up, ~(1ull << split), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    sh.todo2 = todo2;
    __hip_atomic_store(&sh.flag2, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  // Unit u of the tile = pieces (u % (P / np)) * np .. of TR-row tile u / (P / np); this workgroup's own slice holds the
  // units split, split + nsplit, ...; its k-th unit goes to wave (k + 1) % NW.  What a wave needs
  // for its first unit -- the lane's output row, the partials' offsets -- is worked out before it
  // waits, so that the loads go out as soon as the verdict is in.  A unit is a round trip to memory for its wave, so
  // where two pieces each make more units than the workgroups have waves a unit is four (a tile of 256 rows has 128 pieces).
  const int rows = jb.M - jb.row0 < tile_rows ? jb.M - jb.row0 : tile_rows;
  const int pieces = (rows + TR - 1) / TR * P;
  // Tiles of up to 64 rows never do: a unit is what makes one 16-byte load, and 16 slots are in flight where there are more
  // than 8 splits (8 in flight: 4 rows over 3911 paged keys, 31 splits, 14.4 us a pass instead of 13.4).
  constexpr bool SMALL = MAXROWS <= 64;
  constexpr int NP0 = SMALL ? PartialLayout<D, TR, PX>::kPer : 2;
  const int np = SMALL || pieces <= 2 * NW * nsplit ? NP0 : 4;
  const int upt = P / np;                       // units of a TR-row tile
  const int NU = pieces / np;
  auto merge_one = [&](int u, int64_t gr, uint32_t byte, int flag) {
    const int pc = u % upt * np;
    auto go = [&](auto n, auto bs) {
      constexpr int NP = decltype(n)::value, BS = decltype(bs)::value;
      if (flag == 1) merge_pieces<D, TR, PX, NP, 0, BS>(prsrc, gr, byte, gout, nsplit, pc, l);
      else merge_pieces<D, TR, PX, NP, kAgentCoherent, BS>(prsrc, gr, byte, gout, nsplit, pc, l);
    };
    using std::integral_constant;
    constexpr int LONG = PX && !SMALL ? 8 : 16;  // (as many loads as the registers hold)
    if (nsplit <= 8) {  // (one batch in the common cases)
      if (np == NP0) go(integral_constant<int, NP0>{}, integral_constant<int, 8>{});
      else if constexpr (!SMALL) go(integral_constant<int, 4>{}, integral_constant<int, PX ? 4 : 8>{});
    } else {
      if (np == NP0) go(integral_constant<int, NP0>{}, integral_constant<int, LONG>{});
      else if constexpr (!SMALL) go(integral_constant<int, 4>{}, integral_constant<int, PX ? 4 : LONG>{});
    }
  };
  const int u_first = split + ((w + NW - 1) % NW) * nsplit;  // this wave's first unit of the own slice
  int64_t gr_first = -1;
  const bool have_first = u_first < NU && tile_row(u_first / upt, &gr_first);
  const uint32_t byte_first = partial_byte<D, TR, PX>(p, jb, u_first / upt);
  if (w == 0) aside();  // (the wave with the fewest units: it has one of its own only where they are at least NW)
  // the waves wait for thread 64's verdicts in LDS
  int flag;
  while ((flag = __hip_atomic_load(&sh.flag, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP)) == 0) __builtin_amdgcn_s_sleep(1);
  if (do_ts64) ts[8] = wall_clock64();
  auto merge_slices = [&](unsigned long long todo, bool first_done) {
    int k = 0;  // running number of the units of the slices in `todo`
    for (int s2 = 0; s2 < nsplit; s2++) {
      if (!((todo >> s2) & 1ull)) continue;
      for (int u = s2; u < NU; u += nsplit, k++) {
        if ((k + 1) % NW != w || (first_done && u == u_first)) continue;
        int64_t gr;
        if (tile_row(u / upt, &gr)) merge_one(u, gr, partial_byte<D, TR, PX>(p, jb, u / upt), flag);
      }
    }
  };
  const unsigned long long todo1 = sh.todo;
  if (todo1 == (1ull << split)) {  // the usual case: the own slice
    if (have_first) merge_one(u_first, gr_first, byte_first, flag);
    if (u_first + NW * nsplit < NU) merge_slices(todo1, true);
  } else if (todo1 != 0) {
    merge_slices(todo1, false);
  }
  if (do_ts64) ts[9] = wall_clock64();

  while (__hip_atomic_load(&sh.flag2, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) == 0) __builtin_amdgcn_s_sleep(1);
  if (sh.todo2 != 0) merge_slices(sh.todo2, false);
  if (do_ts64) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    ts[7] = wall_clock64();
  }
#undef CB_TS
}

// What a lane holds at the end of a sweep: its row's NP pieces from pc0, unnormalised, with the row's denominator and the
// reference maximum they are relative to.  Written out as the output row (a single split) or as the split's partial
// state (i: TR-row tile of the tile).
template <int D, int TR, bool PX, int NP>
__device__ __forceinline__ void write_rows(const AttnParams& p, const TileJob& jb, int i, int64_t grow, const floatx4 (&f)[NP], int pc0,
                                           float mref, float lsum, float c2, bool first, int l) {
  using Part = PartialLayout<D, TR, PX>;
  const int h = l / TR, r = l % TR;
  if (jb.nsplit == 1) {
    store_row<D, TR, NP>((CB_GLOBAL uint16_t*)p.out, grow, f, pc0, 1.0f / lsum, l);
    return;
  }
  if (grow < 0) return;
  // written through to memory (agent scope) so that the merging workgroup, possibly on another XCD with its own L2,
  // can read it without cache flushes
  const __amdgpu_buffer_rsrc_t prsrc = partial_rsrc<D, TR, PX>(p, jb);
  const uint32_t pbyte = partial_byte<D, TR, PX>(p, jb, i) + (uint32_t)jb.split * Part::kBytes;
#pragma unroll
  for (int n = 0; n < NP; n += Part::kPer) {
    const uint32_t at = pbyte + (pc0 + n) / Part::kPer * Part::kVec + l * 16;
    uintx4 v;
    if constexpr (PX) {
      v = __builtin_bit_cast(uintx4, f[n]);
    } else {
#pragma unroll
      for (int x = 0; x < 2; x++) {
        v[2 * x] = pack_bf16(f[n + x][0], f[n + x][1]);
        v[2 * x + 1] = pack_bf16(f[n + x][2], f[n + x][3]);
      }
    }
    if (p.external_merge) __builtin_amdgcn_raw_buffer_store_b128(v, prsrc, at, 0, 0);
    else __builtin_amdgcn_raw_buffer_store_b128(v, prsrc, at, 0, kAgentCoherent);
  }
  if (h == 0 && first) {
    // m = log2 of the reference weight 2^(c2*mref)
    const float mnat = (mref == -INFINITY) ? -INFINITY : mref * c2;
    const uintx2 ml = {__float_as_uint(mnat), __float_as_uint(lsum)};
    if (p.external_merge) __builtin_amdgcn_raw_buffer_store_b64(ml, prsrc, pbyte + Part::kMl + r * 8, 0, 0);
    else __builtin_amdgcn_raw_buffer_store_b64(ml, prsrc, pbyte + Part::kMl + r * 8, 0, kAgentCoherent);
  }
}

// Timing aid (timeline build): thread 0 copies the workgroup's stamps from LDS to the table, the
// first eight to row wg, the others (phases of the merge) to row wg + 512.
template <bool TS>
__device__ __forceinline__ void flush_timestamps(const AttnParams& p, int wg, const unsigned long long* ts_sh) {
  if constexpr (!TS) return;
  __syncthreads();  // (thread 64 stamps too)
  if (threadIdx.x != 0 || wg >= 1024) return;
  const CB_LDS unsigned long long* ts = (const CB_LDS unsigned long long*)ts_sh;
  CB_GLOBAL unsigned long long* out = (CB_GLOBAL unsigned long long*)p.dbg_ts;
  for (int i = 0; i < 8; i++) out[(int64_t)wg * 8 + i] = ts[i];
  if (wg < 512)
    for (int i = 0; i < 8; i++) out[(int64_t)(wg + 512) * 8 + i] = ts[8 + i];
}

}  // namespace cb
