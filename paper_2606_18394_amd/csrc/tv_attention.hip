// Tree-verification attention for CDNA4 (gfx950).
//
// Computes, for every draft-tree node v of every sequence and every query
// head, softmax(q_v K^T * scale + M_v) V over the sequence's cached prefix
// and the tree nodes, where the tree-causal mask M_v keeps only v's
// ancestors and v itself (Sec. 2.2, tree-causal mask and masked attention
// equations).  The ancestor relation is rebuilt inside each workgroup as a
// bitmask in LDS from the parent array; no dense mask ever exists (App. E).
//
// Work decomposition.  Rows of one (sequence b, KV head g) pair are the N*G
// (node, head-in-group) pairs, row r = node * G + head.  Keys are cut into
// 32-key tiles: ceil(kv_len/32) cache tiles, then the tree tiles up to the
// last node of the row block (a node never sees a later node because
// parents precede children).  The tiles are cut into contiguous chunks
// (split-KV) of one size for the whole batch, found on the device from the
// kv_lens (even_split), so that a capacity far above the lengths or a ragged
// batch still gives chunks of like size; a sequence of one chunk is written
// straight to the output.  A workgroup takes one block of 32*WR rows and
// one chunk with WR x WK wave64s: WR row groups of 32 rows, and WK key
// groups that share out the chunk's tiles, each streaming its tiles through
// an LDS ring of NS stages; key groups merge their softmax states in LDS at
// the end.  The host plan (tv_plan.h) picks WR, WK, NS and S per shape so
// that every CU holds 8 waves (two per SIMD).  The prologue requests the
// parents, the queries and every ring stage before it uses any of them;
// with several key groups on a full grid, key group 0 alone loads the
// queries and hands them to the others through LDS.
//
// Per tile.  K and V move HBM -> LDS with global_load_lds_dwordx4 (no
// register staging), rows XOR-swizzled in 16-byte chunks so the transposing
// V reads are free of bank conflicts and the K reads at most two-way (see
// TileLayout).  A wave computes S^T = K Q^T with
// v_mfma_f32_16x16x32_bf16 (keys on the M side, its 32 rows on the N side),
// runs an fp32 base-2 online softmax on the accumulators with a lazily moved
// reference maximum, and accumulates O^T += V^T P^T: P^T comes straight from
// the S^T accumulators (the 32 keys are ordered so the B operand needs no
// data movement) and V^T from ds_read_b64_tr_b16 transposing reads.
//
// Split-KV merge (sequences of several chunks).  Every chunk stores its (max,
// sum, O) partial.  The chunk that finishes last merges its row block inside
// this kernel (arrival counters in the workspace) when the plan prices that
// below a second kernel that merges all row blocks.
//
// The training mask of many small blocks has a kernel of its own (attn_packed).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <atomic>
#include <mutex>

#include "tv_plan.h"
#include "tv_walk.h"

namespace tv {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4 lds_i16x4;

struct AttnArgs {
  const __bf16* q;
  const __bf16* kc;
  const __bf16* vc;
  const __bf16* kt;
  const __bf16* vt;
  const int32_t* parent;
  const int32_t* kv_len;
  __bf16* out;
  f32x4* ws_o;
  float2* ws_ml;
  unsigned int* arrived;  // per row block: chunks that have stored partials
  int* tree_bad;          // per row block: invalid parent array seen
  int B, N, Hq, Hkv, Lmax, G, M, nRB, S, chunk, nwork;
  int fused;   // split-KV merge inside the main kernel (else a second kernel)
  int slots, min_chunk;  // even split (tv_plan.h): chunks per (KV head, row block), else 0
  float rslots, rslack;  // 1 / slots, 1 / (slots - B)
  int spread;  // work order of several sequences (tv_plan.h, work_item)
  float c;  // scale * log2(e): scores live in base-2 exponent units
  const int32_t* block_table;  // paged cache: [B, max_blocks], else NULL
  int block_shift, max_blocks, num_blocks;
  int tail;    // tree-tail layout: node i's K/V are cache row kv_len + i
  int cgroup;  // sequences sharing one cache (sequence b reads cache b / cgroup)
};

// The kernel's arguments, fetched (again) from where this is called on: what only
// the epilogue needs then holds no scalar registers during the tile loop, whose
// own would otherwise be spilled to vector lanes and read back at every tile.
typedef const __attribute__((address_space(4))) AttnArgs LateArgs;
__device__ __forceinline__ const LateArgs* late_args() {
  const LateArgs* p = (const LateArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return p;
}

// Context rows of sequence b: its kv_len clamped to what the cache holds (in
// the tree-tail layout behind room for the tree); a NULL kv_len means full.
__device__ __forceinline__ int context_rows(const AttnArgs& a, int b) {
  const int cap = a.tail ? a.Lmax - a.N : a.Lmax;
  const int kvl = a.kv_len ? a.kv_len[b] : cap;
  return kvl < 0 ? 0 : (kvl > cap ? cap : kvl);
}
// The same from a kv_len asked for earlier (any value for a NULL one).
__device__ __forceinline__ int context_rows_of(const AttnArgs& a, int asked) {
  const int cap = a.tail ? a.Lmax - a.N : a.Lmax;
  return a.kv_len && asked < cap ? max(asked, 0) : cap;
}

// The key tiles a row block attends over, behind kvl context rows and up to
// node i_hi.  Separate tree K/V: nct cache tiles (rows < kvl) then the tree
// tiles of nodes 0..i_hi.  Tree-tail layout: the tree rows follow the context
// in the cache and one run of nct = T tiles covers rows 0 .. kvl + i_hi.
struct Segment {
  int nct, T;
};
__device__ __forceinline__ Segment segment(const AttnArgs& a, int kvl, int i_hi) {
  if (a.tail) {
    const int t = (kvl + i_hi + kKeyTile) / kKeyTile;
    return Segment{t, t};
  }
  const int nct = (kvl + kKeyTile - 1) / kKeyTile;
  return Segment{nct, nct + i_hi / kKeyTile + 1};
}

// Longest-first order of a ragged batch (spread = 2).  XCD x serves one KV
// head and lane x / Hkv of L = 8 / Hkv lanes of chunks; pair p of the lane
// is sequence p / (S / L) and its (p % (S / L))-th chunk in that lane, as in
// work_item.  Each pair gets the distinct key (tile count << 16 | 0xFFFF - p)
// (longest first, lower pair index on ties), and the workgroup takes the
// pair whose key is the (i+1)-th largest, i its own pair index: with one
// pair per lane by counting larger keys over lane exchanges, else by
// bisection on the key value with wave-wide counts (each lane holds up to
// kRankPerLane pairs).  Every workgroup finds the same order, so this
// permutes the pairs: every work item is still covered once.
constexpr int kRankPerLane = 16;  // == kMaxRankPairs / 64 in tv_plan.h

__device__ __forceinline__ void longest_first(const AttnArgs& a, int bid, WorkItem& it) {
  const int lane = threadIdx.x & 63;
  const int L = kXcds / a.Hkv, per_b = a.S / L, npairs = a.B * per_b;  // L: a power of two
  const int x = bid % kXcds, target = (bid / kXcds) / a.nRB, ln = x / a.Hkv;
  const int nk = (npairs + 63) / 64;  // pair slots in use per lane
  // pair p's sequence (p < 2^10: the reciprocal is exact enough), and its chunk
  const float rper = __builtin_amdgcn_rcpf((float)per_b);
  auto seq = [&](int p) { return (int)(((float)p + 0.5f) * rper); };
  auto chunk_of = [&](int p, int b) { return ((ln - b) & (L - 1)) + L * (p - b * per_b); };
  int key[kRankPerLane];
  // all lengths are requested before any is used
#pragma unroll
  for (int k = 0; k < kRankPerLane; ++k)
    key[k] = k < nk ? context_rows(a, seq(min(lane + 64 * k, npairs - 1))) : -1;
#pragma unroll
  for (int k = 0; k < kRankPerLane; ++k) {
    const int p = lane + 64 * k;
    if (k < nk) {
      const int tiles = (key[k] + kKeyTile - 1) / kKeyTile + (a.N - 1) / kKeyTile + 1;
      const int work = max(0, min(a.chunk, tiles - chunk_of(p, seq(p)) * a.chunk));  // < 2^14 (plan)
      key[k] = p < npairs ? (work << 16) | (0xFFFF - p) : -1;
    }
  }
  int p;
  if (nk == 1) {
    // one pair per lane: every lane counts the larger keys by lane exchanges
    int rank = 0;
    for (int q = 0; q < 64; ++q) rank += __shfl(key[0], q) > key[0];
    const unsigned long long hit = __ballot(lane < npairs && rank == target);
    p = __builtin_amdgcn_readfirstlane(hit ? (int)__builtin_ctzll(hit) : 0);
  } else {
    // the largest v with at least target + 1 keys >= v is the wanted key (unused
    // slots count for none; four at a time, since a branch over each costs more
    // than it skips)
    int lo = 0, hi = 1 << 30;
    while (hi - lo > 1) {
      const int mid = lo + ((hi - lo) >> 1);
      int c = 0;
#pragma unroll
      for (int k4 = 0; k4 < kRankPerLane; k4 += 4) {
        if (k4 >= nk) break;
#pragma unroll
        for (int k = k4; k < k4 + 4; ++k) c += __popcll(__ballot(key[k] >= mid));
      }
      if (c >= target + 1) lo = mid;
      else hi = mid;
    }
    p = 0xFFFF - (lo & 0xFFFF);
  }
  it.b = seq(p);
  it.s = chunk_of(p, it.b);
}

__device__ __forceinline__ int wave_sum(int x) {
  x += (int)dpp_u32<0xB1>((unsigned)x);
  x += (int)dpp_u32<0x4E>((unsigned)x);
  x += (int)dpp_u32<0x141>((unsigned)x);
  x += (int)dpp_u32<0x140>((unsigned)x);
  return __builtin_amdgcn_readlane(x, 0) + __builtin_amdgcn_readlane(x, 16) +
         __builtin_amdgcn_readlane(x, 32) + __builtin_amdgcn_readlane(x, 48);
}

// Sums over the lanes up to each one (shifts by 1, 2, 4 and 8 lanes inside a
// row of 16, then row 0's and row 2's last lane into the next row and lane 31
// into rows 2 and 3), without the LDS crossbar.
__device__ __forceinline__ int wave_scan(int x) {
  x += (int)dpp_u32<0x111>((unsigned)x);
  x += (int)dpp_u32<0x112>((unsigned)x);
  x += (int)dpp_u32<0x114>((unsigned)x);
  x += (int)dpp_u32<0x118>((unsigned)x);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);
  return x;
}

// ceil(x / c) for 0 <= x < 2^20, 1 <= c < 2^20, rc = 1 / c to one ulp: the
// quotient's distance to the next whole number below, at least 1 / (2 c), is
// above the errors of the reciprocal and the product (together 1.5 * 2^-23 of a
// quotient of at most (x + c) / c)
__device__ __forceinline__ int ceil_div(int x, int c, float rc) {
  return (int)(((float)(x + c) - 0.5f) * rc);
}

// Even split of the batch (a.slots > 0): one chunk size for all sequences, the
// smallest for which they need at most a.slots chunks together.  Every wave
// finds it alike from the kv_lens, and with it the sequence b and the chunk s of
// it that a work item is (s < 0: past the work), the number `first` of that
// sequence's first chunk and its context rows kvl.  All of it comes before a
// workgroup's first load of keys, so it is kept short: a whole division is some
// 40 instructions and another look at kv_len a round trip to the cache, so the
// quotients are taken with reciprocals (the host's where the divisor is its) and
// kvl comes out of the lane that holds it.  (With whole divisions, a scan over the
// LDS crossbar and kv_len read twice: 33 nodes x 16 sequences of 300 to 4096 rows
// 54.7 us, now 53.6; 2 x 24 nodes over 4360 rows 18.5, now 17.7; 37 x 4 nodes over
// 271 rows 13.7, now 13.1; 64 nodes over 4096 rows 20.0, now 19.9.)
struct EvenItem {
  int chunk, b, s, first, kvl;
};

// One sequence: the item's number is the chunk's.
template <bool kAsked>
__device__ __forceinline__ EvenItem even_one(const AttnArgs& a, int item, int asked) {
  const int kvl = kAsked ? context_rows_of(a, asked) : context_rows(a, 0);
  const int t = segment(a, kvl, a.N - 1).T;
  const int chunk = max(a.min_chunk, ceil_div(t, a.slots, a.rslots));
  return EvenItem{chunk, 0, item * chunk < t ? item : -1, 0, kvl};
}

// Several, P consecutive ones per lane (all slots are computed, those past the
// batch hold no tiles: a branch over each costs more than it skips).  The tiles
// are those of the last row block: a chunk's row blocks read the same keys.  With
// item < 0 it is sequence b that is looked up (its s is then of no use).
template <int P>
__device__ __forceinline__ EvenItem even_lanes(const AttnArgs& a, int item, int b) {
  const int b0 = P * (threadIdx.x & 63);
  int kvl[P], t[P], n[P], sum = 0, most = 0;
#pragma unroll
  for (int k = 0; k < P; ++k) kvl[k] = context_rows(a, min(b0 + k, a.B - 1));
#pragma unroll
  for (int k = 0; k < P; ++k) {
    t[k] = b0 + k < a.B ? segment(a, kvl[k], a.N - 1).T : 0;
    sum += t[k];
    most = max(most, t[k]);
  }
  const float total = (float)wave_sum(sum);
  const int longest = (int)wave_max_u32((unsigned)most);
  // Chunks of less than total / slots tiles are too many, those of total /
  // (slots - B) few enough (the sum of ceil(t / c) is below total / c + B); the
  // margins cover the rounding.
  int lo = max(a.min_chunk - 1, (int)(total * a.rslots * 0.999999f) - 1);
  int hi = max(min(longest, (int)(total * a.rslack * 1.000001f) + 1), lo + 1);
  auto chunks = [&](int c) {
    const float rc = __builtin_amdgcn_rcpf((float)c);
    int s = 0;
#pragma unroll
    for (int k = 0; k < P; ++k) {
      n[k] = ceil_div(t[k], c, rc);
      s += n[k];
    }
    return s;
  };
  while (hi - lo > 1) {
    const int mid = lo + ((hi - lo) >> 1);
    if (wave_sum(chunks(mid)) <= a.slots) hi = mid;
    else lo = mid;
  }
  const int upto = wave_scan(chunks(hi));
  int first = upto;
#pragma unroll
  for (int k = 0; k < P; ++k) first -= n[k];
  // the last sequence that starts at or before the item: its lane, then its
  // place there (every sequence has a chunk, so places past the batch start with
  // the lane after them)
  const int owner = item < 0 ? b / P : __popcll(__ballot(b0 < a.B && first <= item)) - 1;
  int place = 0, kv = kvl[0], end = first + n[0];
#pragma unroll
  for (int k = 1; k < P; ++k) {
    const bool next = item < 0 ? b % P >= k : end <= item && b0 + k < a.B;
    place = next ? k : place;
    kv = next ? kvl[k] : kv;
    first = next ? end : first;
    end += n[k];
  }
  first = __builtin_amdgcn_readlane(first, owner);
  return EvenItem{hi, P * owner + __builtin_amdgcn_readlane(place, owner),
                  item < __builtin_amdgcn_readlane(upto, 63) ? item - first : -1, first,
                  __builtin_amdgcn_readlane(kv, owner)};
}

// Work item `item` of the batch, or (item < 0) what concerns sequence b; asked: the
// first sequence's kv_len where kAsked, else of no use.
template <bool kAsked>
__device__ __forceinline__ EvenItem even_split(const AttnArgs& a, int item, int b, int asked) {
  static_assert(kEvenSequences == 16 * 64, "sequences per lane");
  if (a.B == 1) return even_one<kAsked>(a, item, asked);
  if (a.B <= 64) return even_lanes<1>(a, item, b);
  return a.B <= 256 ? even_lanes<4>(a, item, b) : even_lanes<16>(a, item, b);
}

// Four output values, or four NaN when the sequence's tree is invalid (the
// NaN is written as a bit pattern: the kernels assume no NaN arithmetic).
__device__ __forceinline__ void store_out4(__bf16* p, const f32x4& acc, float inv, bool nan) {
  const bf16x4 v = {(__bf16)(acc[0] * inv), (__bf16)(acc[1] * inv), (__bf16)(acc[2] * inv),
                    (__bf16)(acc[3] * inv)};
  i16x4 bits = __builtin_bit_cast(i16x4, v);
  if (nan) bits = i16x4{0x7FC0, 0x7FC0, 0x7FC0, 0x7FC0};
  *reinterpret_cast<i16x4*>(p) = bits;
}

// Split-KV partials cross workgroups (and XCDs) through device-scope
// accesses: the sc1 bit makes a store complete only once it is visible at
// device scope and a load read at that level, which is how the compiler
// lowers relaxed agent-scope atomic loads and stores; these are their
// 8- and 16-byte forms.  Publishing then needs only vmcnt(0) before the
// arrival counter, where a release fence would write back the whole L2,
// and the merging workgroup needs no L2 invalidate (which would evict the
// keys that other workgroups are still reading).
__device__ __forceinline__ void store_dev(f32x4* p, f32x4 v) {
  asm volatile("global_store_dwordx4 %0, %1, off sc1" ::"v"(p), "v"(v) : "memory");
}
__device__ __forceinline__ void store_dev(float2* p, float2 v) {
  asm volatile("global_store_dwordx2 %0, %1, off sc1" ::"v"(p), "v"(v) : "memory");
}
__device__ __forceinline__ f32x4 load_dev(const f32x4* p) {
  f32x4 v;
  asm volatile("global_load_dwordx4 %0, %1, off sc1" : "=v"(v) : "v"(p) : "memory");
  return v;
}
__device__ __forceinline__ float2 load_dev(const float2* p) {
  float2 v;
  asm volatile("global_load_dwordx2 %0, %1, off sc1" : "=v"(v) : "v"(p) : "memory");
  return v;
}
// Plain 16- and 4-byte loads issued as inline assembly, for the prologue:
// the compiler does not track them, so it inserts no wait of its own that
// would also drain the tile DMAs issued after them.  Loads return in issue
// order, so an explicit vmcnt that leaves exactly the younger DMAs
// outstanding covers them; `loaded` then ties each value to that wait.
__device__ __forceinline__ bf16x8 load_b128(const __bf16* p) {
  bf16x8 v;
  asm volatile("global_load_dwordx4 %0, %1, off" : "=v"(v) : "v"(p) : "memory");
  return v;
}
__device__ __forceinline__ int load_i32(const int32_t* p) {
  int v;
  asm volatile("global_load_dword %0, %1, off" : "=v"(v) : "v"(p) : "memory");
  return v;
}
// Waits for every outstanding vector memory access; `loaded` values of
// load_dev are tied to the wait so no use is scheduled before it.
__device__ __forceinline__ void wait_all_vm() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
template <class T>
__device__ __forceinline__ void loaded(T& v) {
  asm volatile("" : "+v"(v));
}

__device__ __forceinline__ float wave_max_across_groups(float v) {
  v = fmaxf(v, __shfl_xor(v, 16));
  v = fmaxf(v, __shfl_xor(v, 32));
  return v;
}

// 16 bytes per lane from global memory straight into LDS: lane i reads
// sbase + voff (sbase wave-uniform, voff a per-lane byte offset) and its
// bytes land at lds_addr + 16 * i (lds_addr wave-uniform).  Issued as inline
// assembly so the compiler does not serialise every later LDS read behind
// it; completion is awaited with explicit vmcnt waits.
__device__ __forceinline__ void dma16(const void* sbase, uint32_t voff, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2"
               :
               : "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(voff), "s"(sbase)
               : "memory");
}

// A wave-uniform pointer the compiler cannot prove uniform, moved to SGPRs
// (the DMA's base address operand must be scalar).
__device__ __forceinline__ const char* uniform_ptr(const char* p) {
  const uint64_t u = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
  return (const char*)(((uint64_t)hi << 32) | lo);
}

// s_waitcnt vmcnt(n) with the other counters left alone (gfx9 encoding).
template <int n>
__device__ __forceinline__ void wait_vm() {
  static_assert(n >= 0 && n < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((n & 15) | ((n >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

// s_waitcnt vmcnt(n) for a wave-uniform n in 0..63 (the prologue's waits:
// queries and DMAs still in flight); anything else waits for everything.
__device__ __forceinline__ void wait_vm_any(int n) {
  switch (n) {
#define TV_WAIT_CASE(k) \
  case k:               \
    wait_vm<k>();       \
    break;
#define TV_WAIT_CASES8(k)                                                                    \
  TV_WAIT_CASE(k) TV_WAIT_CASE(k + 1) TV_WAIT_CASE(k + 2) TV_WAIT_CASE(k + 3) TV_WAIT_CASE(k + 4) \
      TV_WAIT_CASE(k + 5) TV_WAIT_CASE(k + 6) TV_WAIT_CASE(k + 7)
    TV_WAIT_CASES8(0) TV_WAIT_CASES8(8) TV_WAIT_CASES8(16) TV_WAIT_CASES8(24)
    TV_WAIT_CASES8(32) TV_WAIT_CASES8(40) TV_WAIT_CASES8(48) TV_WAIT_CASES8(56)
#undef TV_WAIT_CASES8
#undef TV_WAIT_CASE
    default: wait_vm<0>(); break;
  }
}

// s_waitcnt vmcnt(PW * min(n, T)): at most n tiles of PW DMAs in flight
template <int PW, int T>
__device__ __forceinline__ void wait_tiles(int n) {
  if constexpr (T == 0) {
    wait_vm<0>();
  } else {
    if (n >= T) wait_vm<T * PW>();
    else wait_tiles<PW, T - 1>(n);
  }
}

// Layout of one 32-key tile in LDS: row-major, D bf16 per row, 16-byte
// chunks XOR-swizzled by the row.  With reads served 256 bytes at a time
// (64 banks; 16 lanes of a ds_read_b128, 32 of a ds_read_b64_tr_b16) the
// swizzle is free of bank conflicts: 16 rows at one logical chunk (the K
// operand reads) land in 16 bank groups, and the transposing V reads (rows
// 8k..8k+7, two adjacent chunks) cover every bank once.  The hardware
// serves the K reads 128 bytes at a time (8 lanes), where rows r and r + 4
// collide: the K reads are 2-way, a third of the LDS-active cycles, as the
// bank-conflict counter shows.  A swizzle free of conflicts at both widths
// (((r & 3) << 1) | ((r >> 2) & 1) | (((r >> 2) ^ (r >> 3)) & 1) << 3 for
// D = 128) removed them and a third of the LDS-active cycles but not a
// cycle of the kernel (about 1% slower), so this one stays.
template <int D>
struct TileLayout {
  static constexpr int kRowBytes = 2 * D;
  static constexpr int kCPR = D / 8;               // 16-byte chunks per row
  static constexpr int kBytes = kKeyTile * kRowBytes;
  static constexpr int kDma = kBytes / 1024;       // 1 KB DMA instructions per tile
  static constexpr int kRowsPerDma = 64 / kCPR;
  __device__ static __forceinline__ int swz(int r) {
    return D == 128 ? (((r & 7) << 1) | ((r >> 3) & 1))
                    : ((((r >> 1) & 3) << 1) | ((r >> 3) & 1));
  }
  __device__ static __forceinline__ int off(int r, int chunk) {
    return r * kRowBytes + ((chunk ^ swz(r)) << 4);
  }
};

// Where a wave's K/V rows come from: the cache of one (sequence, KV head)
// pair, then its tree K/V.  The cache is either padded (row t at kcache +
// t * row_bytes) or paged (row t in pool block btab[t >> shift], whose rows
// are 2^shift apart from kcache + block * 2^shift * row_bytes; a 32-key
// tile never straddles blocks since blocks hold a power of two >= 32 rows).
// Block numbers are clamped into the pool.  Pointers are byte pointers.
struct TreeSrc {
  const char* kcache;
  const char* vcache;
  const char* ktree;
  const char* vtree;
  const int32_t* btab;  // this sequence's block table row, or NULL
  int shift, nblk;      // log2(block size), blocks in the pool
  int row_bytes;  // bytes between consecutive keys
  int rows;       // valid cache rows (the tree's too in the tree-tail layout)
  int nct;        // cache tiles
  int i_hi;       // last tree node the row block can see
};

// Issue this lane's DMA instructions for tile t into the stage at kdst (K
// tile, then V tile).  The scalar base is the tile's first row; rows past
// the valid range are clamped onto a valid row (the mask gives them zero
// weight, the clamp keeps reads in range).  dma_off is the per-lane byte
// offset of its chunk within a full tile.
template <int D, int PW, bool kPaged>
__device__ __forceinline__ void issue_tile(const TreeSrc& src, const uint32_t (&dma_off)[PW],
                                           int wr, int lane, int t, uint32_t kdst) {
  using TL = TileLayout<D>;
  const bool cache = t < src.nct;
  const int first = cache ? t * kKeyTile : (t - src.nct) * kKeyTile;
  const char* kb;
  const char* vb;
  if constexpr (kPaged) {
    size_t tofs = (size_t)first * src.row_bytes;
    if (cache) {
      // A scalar load through the constant address space (the table is
      // read-only here and the tile index wave-uniform): a vector load
      // would make the compiler wait for every DMA in flight.
      typedef const __attribute__((address_space(4))) int32_t ctab_t;
      int blk = ((ctab_t*)src.btab)[__builtin_amdgcn_readfirstlane(first >> src.shift)];
      blk = blk < 0 ? 0 : (blk >= src.nblk ? src.nblk - 1 : blk);
      tofs = (((size_t)blk << src.shift) + (first & ((1 << src.shift) - 1))) * src.row_bytes;
    }
    kb = uniform_ptr((cache ? src.kcache : src.ktree) + tofs);
    vb = uniform_ptr((cache ? src.vcache : src.vtree) + tofs);
  } else {
    kb = (cache ? src.kcache : src.ktree) + (size_t)first * src.row_bytes;
    vb = (cache ? src.vcache : src.vtree) + (size_t)first * src.row_bytes;
  }
  if (cache && (t + 1) * kKeyTile <= src.rows) {
#pragma unroll
    for (int k = 0; k < PW; ++k) {
      const int q = wr * PW + k;
      const bool isv = q >= TL::kDma;
      dma16(isv ? vb : kb, dma_off[k], kdst + (isv ? TL::kBytes : 0) + (q % TL::kDma) * 1024);
    }
    return;
  }
  const int last = cache ? src.rows - 1 : src.i_hi;  // >= first for every existing tile
#pragma unroll
  for (int k = 0; k < PW; ++k) {
    const int q = wr * PW + k;
    const bool isv = q >= TL::kDma;
    const int r = (q % TL::kDma) * TL::kRowsPerDma + lane / TL::kCPR;
    const int row = min(first + r, last) - first;
    const uint32_t off = (uint32_t)(row * src.row_bytes + ((lane % TL::kCPR) ^ TL::swz(r)) * 16);
    dma16(isv ? vb : kb, off, kdst + (isv ? TL::kBytes : 0) + (q % TL::kDma) * 1024);
  }
}

// Where a tile's scores need masking: the cache tail and the tree tiles.
struct MaskInfo {
  int t, nct, kvl, ntt, tail;
  const uint32_t* anc;
};

constexpr float kSlack = 8.f;  // log2 units a row's reference may lag its maximum

// Steps of one 32-key tile for a wave's 32 rows (two 16-row tiles nt).
//
// The compiler must not move instructions across this point: it would sink
// the LDS reads to just before their uses (fewer registers) and chain the
// score products, and the tile then waits for every LDS and matrix latency in
// turn.
__device__ __forceinline__ void pin_order() { __builtin_amdgcn_sched_barrier(0); }

// The tile's V^T operand from transposing LDS reads: lane (g4, l16) receives
// V[key 4*g4 + j (+16)][16*dt + l16], the key order of P^T.
template <int D>
__device__ __forceinline__ void read_values(const unsigned char* vt_lds, i16x4 (&vf)[D / 16][2],
                                            int g4, int l16) {
  using TL = TileLayout<D>;
#pragma unroll
  for (int dt = 0; dt < D / 16; ++dt) {
    const int rr = 4 * g4 + (l16 >> 2);
    const int chunk = 2 * dt + ((l16 & 3) >> 1);
    const int inb = 8 * (l16 & 1);
    vf[dt][0] =
        __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(vt_lds + TL::off(rr, chunk) + inb));
    vf[dt][1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (lds_i16x4*)(vt_lds + TL::off(rr + 16, chunk) + inb));
  }
}

// scores: S^T = K Q^T on the matrix cores; lane (g4, l16) holds
//   S^T[key 16*tt + 4*g4 + j][row 16*nt + l16].
template <int D, int NT>
__device__ __forceinline__ void tile_scores(const bf16x8 (&kf)[2][D / 32], const bf16x8 (&qf)[NT][D / 32],
                                            f32x4 (&sc)[2][NT]) {
  constexpr int NC = D / 32;
#pragma unroll
  for (int cc = 0; cc < NC; ++cc) {
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        sc[tt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[tt][cc], qf[nt][cc],
                                                             cc == 0 ? zero : sc[tt][nt], 0, 0, 0);
      }
    pin_order();
  }
}

// The first n keys of a tile (n < 0: none, n > 32: all) as a visibility word.
__device__ __forceinline__ uint32_t first_keys(int n) {
  n = n < 0 ? 0 : (n > kKeyTile ? kKeyTile : n);
  return (uint32_t)((1ull << n) - 1ull);
}

// The visible keys of tile mk.t for this lane's row of every 16-row tile, one
// bit per key: cache keys below kv_len, and tree keys of the row's
// ancestor-or-self set (one 32-bit word of its bitmask per tile).
template <int NT>
__device__ __forceinline__ void tile_bits(const MaskInfo& mk, const int (&node_rel)[NT],
                                          uint32_t (&bits)[NT]) {
  if (mk.tail) {
    // Tree-tail layout: key k of the tile is node s + k (s < 0: a context
    // row).  Its visibility bits are a 32-bit window of the row's ancestor
    // bitmask, words w0 and w0 + 1, with all-ones standing in for context
    // rows (word -1) and zeros past the last word.
    const int s = mk.t * kKeyTile - mk.kvl;  // > -kKeyTile in the masked tiles
    const int w0 = s >> 5, sh = s & 31;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const uint32_t* wp = mk.anc + node_rel[nt] * mk.ntt;
      const uint32_t lo = w0 < 0 ? 0xFFFFFFFFu : wp[w0];
      const uint32_t hi = w0 + 1 < mk.ntt ? wp[w0 + 1] : 0u;
      bits[nt] = (uint32_t)((((uint64_t)hi << 32) | lo) >> sh);
    }
  } else if (mk.t < mk.nct) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) bits[nt] = first_keys(mk.kvl - mk.t * kKeyTile);
  } else {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) bits[nt] = mk.anc[node_rel[nt] * mk.ntt + mk.t - mk.nct];
  }
}

// mask: -inf for the keys a row does not see.
template <int NT>
__device__ __forceinline__ void tile_mask(f32x4 (&sc)[2][NT], const uint32_t (&bits)[NT], int g4) {
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (!((bits[nt] >> (16 * tt + 4 * g4 + j)) & 1u)) sc[tt][nt][j] = -INFINITY;
}

// reference: online softmax in base 2 with a lazily moved reference.  A
//   row's reference m (log2 units) only moves when one of its scores
//   exceeds it by more than kSlack, so weights stay below 2^kSlack (far
//   inside the fp32 and bf16 ranges) and rescaling is rare.  Each lane
//   compares its raw scores with thr = (m + kSlack) / c; only a moving tile
//   pays for exact row maxima, and rows that move rescale O and l.
template <int DT, int NT>
__device__ __forceinline__ void tile_reference(const f32x4 (&sc)[2][NT], float (&m)[NT],
                                               float (&thr)[NT], f32x4 (&o)[DT][NT],
                                               f32x4 (&lacc)[NT], float c, float inv_c) {
  float mx[NT];
  bool move = false;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    float v = fmaxf(fmaxf(sc[0][nt][0], sc[0][nt][1]), sc[0][nt][2]);
    v = fmaxf(fmaxf(v, sc[0][nt][3]), sc[1][nt][0]);
    v = fmaxf(fmaxf(v, sc[1][nt][1]), sc[1][nt][2]);
    v = fmaxf(v, sc[1][nt][3]);
    mx[nt] = v;
    move |= v > thr[nt];
  }
  if (__any(move)) {
    // rare: a row that has not moved keeps its scale; its m may still be -inf
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      mx[nt] = wave_max_across_groups(mx[nt]) * c;
      const bool moved = mx[nt] > m[nt] + kSlack;
      const float alpha = moved ? __builtin_amdgcn_exp2f(m[nt] - mx[nt]) : 1.f;
      m[nt] = moved ? mx[nt] : m[nt];
      thr[nt] = (m[nt] + kSlack) * inv_c;
      lacc[nt] *= alpha;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) o[dt][nt] *= alpha;
    }
  }
}

// weights: the bf16 P^T operand, exactly as it lies in the accumulators.
template <int NT>
__device__ __forceinline__ void tile_weights(const f32x4 (&sc)[2][NT], const float (&m)[NT], float c,
                                             bf16x8 (&pf)[NT]) {
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const float mref = fmaxf(m[nt], -3.0e38f);  // rows with nothing visible yet: weights 0
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        pf[nt][4 * tt + j] = (__bf16)__builtin_amdgcn_exp2f(fmaf(sc[tt][nt][j], c, -mref));
  }
}

// values: row sums ones^T P^T into lacc (same rounded weights as the
//   numerator) and O^T += V^T P^T.
template <int D, int NT>
__device__ __forceinline__ void tile_values(const i16x4 (&vf)[D / 16][2], const bf16x8 (&pf)[NT],
                                            const bf16x8& ones, f32x4 (&o)[D / 16][NT],
                                            f32x4 (&lacc)[NT]) {
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
    lacc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pf[nt], lacc[nt], 0, 0, 0);
#pragma unroll
  for (int dt = 0; dt < D / 16; ++dt) {
    const bf16x4 lo = __builtin_bit_cast(bf16x4, vf[dt][0]), hi = __builtin_bit_cast(bf16x4, vf[dt][1]);
    const bf16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
      o[dt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v, pf[nt], o[dt][nt], 0, 0, 0);
  }
}

// The whole tile in order (the loop form without lookahead).
template <int D, int NT, bool kMasked>
__device__ __forceinline__ void attend_tile(const unsigned char* kt_lds, const bf16x8 (&qf)[NT][D / 32],
                                            f32x4 (&o)[D / 16][NT], f32x4 (&lacc)[NT],
                                            float (&m)[NT], float (&thr)[NT], const bf16x8& ones,
                                            float c, float inv_c, const uint32_t (&bits)[NT],
                                            int g4, int l16) {
  using TL = TileLayout<D>;
  constexpr int NC = D / 32;
  // All of the tile's LDS reads go out first, K before V.
  bf16x8 kf[2][NC];
#pragma unroll
  for (int cc = 0; cc < NC; ++cc)
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
      kf[tt][cc] = *reinterpret_cast<const bf16x8*>(kt_lds + TL::off(16 * tt + l16, 4 * cc + g4));
  i16x4 vf[D / 16][2];
  pin_order();
  f32x4 sc[2][NT];
  // The score products run at raised wave priority: the SIMD's other wave
  // is then mostly in its softmax (vector work) while these matrix
  // instructions issue back to back (measured 5-8% faster on matrix-bound
  // shapes than equal priority or raising it for the value products too).
  __builtin_amdgcn_s_setprio(1);
  tile_scores<D, NT>(kf, qf, sc);
  __builtin_amdgcn_s_setprio(0);
  read_values<D>(kt_lds + TL::kBytes, vf, g4, l16);
  pin_order();
  if (kMasked) tile_mask<NT>(sc, bits, g4);
  tile_reference<D / 16, NT>(sc, m, thr, o, lacc, c, inv_c);
  bf16x8 pf[NT];
  tile_weights<NT>(sc, m, c, pf);
  pin_order();
  tile_values<D, NT>(vf, pf, ones, o, lacc);
}

// Merge of the chunk partials of one row block, run by the workgroup whose
// chunk arrived last: out = sum_s e_s O_s / sum_s e_s l_s, e_s = 2^(m_s - m*),
// folded in online over s in batches of loads.  Wave w takes one 16-row
// tile and every WPN-th 16-column tile of it (or several row tiles when the
// block has more row tiles than the workgroup has waves), so each lane
// reads its rows' (m, l) once.
template <int D, int RB, int kWaves>
__device__ __forceinline__ void merge_chunks(const LateArgs* a, size_t part0, int nval, int b,
                                             int g, int r0, bool bad, int wave, int lane) {
  constexpr int DT = D / 16, NTG = RB / 16;
  constexpr bool kSplitCols = kWaves >= NTG;
  constexpr int WPN = kSplitCols ? kWaves / NTG : 1;  // waves per row tile
  constexpr int NPW = kSplitCols ? 1 : NTG / kWaves;  // row tiles per wave
  constexpr int DPW = DT / WPN;                       // column tiles per wave
  constexpr int UB = 32 / DPW;                        // chunks per batch of loads
  // every wave gets whole column tiles of one row tile, or whole row tiles
  static_assert(kSplitCols ? (kWaves % NTG == 0 && DT % WPN == 0) : (NTG % kWaves == 0),
                "merge split");
  const int g4 = lane >> 4, l16 = lane & 15;
#pragma unroll
  for (int k = 0; k < NPW; ++k) {
    const int ntg = kSplitCols ? wave % NTG : wave + k * kWaves;
    if (r0 + ntg * 16 >= a->M) continue;  // no rows
    const int dt0 = kSplitCols ? wave / NTG : 0;
    const int row = ntg * 16 + l16;
    float m = -INFINITY, l = 0.f;
    f32x4 acc[DPW];
#pragma unroll
    for (int j = 0; j < DPW; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < nval; s0 += UB) {
      float2 ml[UB];
      f32x4 ov[UB][DPW];
#pragma unroll
      for (int u = 0; u < UB; ++u)
        if (s0 + u < nval) {
          const size_t ps = part0 + s0 + u;
          ml[u] = load_dev(&a->ws_ml[ps * RB + row]);
#pragma unroll
          for (int j = 0; j < DPW; ++j)
            ov[u][j] = load_dev(&a->ws_o[(ps * DT * NTG + (dt0 + j * WPN) * NTG + ntg) * 64 + lane]);
        }
      wait_all_vm();
#pragma unroll
      for (int u = 0; u < UB; ++u)
        if (s0 + u < nval) {
          loaded(ml[u]);
#pragma unroll
          for (int j = 0; j < DPW; ++j) loaded(ov[u][j]);
        }
#pragma unroll
      for (int u = 0; u < UB; ++u)
        if (s0 + u < nval && ml[u].x != -INFINITY) {
          const float mn = fmaxf(m, ml[u].x);
          const float ea = __builtin_amdgcn_exp2f(m - mn);  // 0 while m = -inf
          const float eb = __builtin_amdgcn_exp2f(ml[u].x - mn);
          l = l * ea + eb * ml[u].y;
#pragma unroll
          for (int j = 0; j < DPW; ++j) acc[j] = acc[j] * ea + eb * ov[u][j];
          m = mn;
        }
    }
    const int r = r0 + row;
    if (r < a->M) {
      const int node = r / a->G, h = g * a->G + r % a->G;
      __bf16* op = a->out + ((size_t)(b * a->N + node) * a->Hq + h) * D + 4 * g4;
      const float inv = 1.f / l;
#pragma unroll
      for (int j = 0; j < DPW; ++j) store_out4(op + 16 * (dt0 + j * WPN), acc[j], inv, bad);
    }
  }
}

// A workgroup of WR x WK wave64s: WR row groups x WK key groups.  A wave owns 32 rows of its row group; the WR
// waves of a key group share one LDS ring and walk that group's tiles (every
// WK-th tile of the chunk) in lock step; WK > 1 groups merge their partial
// softmax states in LDS at the end.
template <int D, int WR, int WK, int NS, bool kPaged, bool kShareQ>
__global__ __launch_bounds__(64 * WR * WK) __attribute__((amdgpu_waves_per_eu(2, 2)))
void attn_main(AttnArgs a) {
  using TL = TileLayout<D>;
  constexpr int kThreads = 64 * WR * WK;
  constexpr int kWaves = WR * WK;
  constexpr int RB = kRowsPerWave * WR; // rows per workgroup
  constexpr int NT = kRowsPerWave / 16; // 16-row tiles per wave
  constexpr int NTG = RB / 16;          // 16-row tiles per workgroup
  constexpr int NC = D / 32;            // 32-wide head-dim chunks (QK^T)
  constexpr int DT = D / 16;            // 16-wide head-dim tiles (PV)
  constexpr int STAGE = 2 * TL::kBytes; // K tile + V tile
  constexpr int PW = 2 * TL::kDma / WR; // DMAs per wave per tile
  static_assert(PW >= 1 && PW * WR == 2 * TL::kDma, "DMA split");
  static_assert(NS >= 1, "ring does not fit");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

  WorkItem it{};
  int chunk = a.chunk, kvl, part0;  // part0: the row block's first chunk partial
  // One sequence's length is on its way while the work item is found (64 nodes over
  // 4096 rows 18.04 -> 17.80 us).  Not with one key group, whose plans have long
  // chunks: there 512 nodes over 8192 rows took 148.3 us so, and 147.7 without.
  int asked = 0;
  if constexpr (WK > 1) {
    if (a.kv_len) asked = a.kv_len[0];
    asm volatile("" ::: "memory");
  }
  if (a.slots > 0) {
    const int item = even_item(blockIdx.x, a.slots, a.nRB, a.Hkv, it);
    if (item < 0) return;
    const EvenItem ev = even_split<(WK > 1)>(a, item, 0, asked);
    if (ev.s < 0) return;
    it.b = ev.b;
    it.s = ev.s;
    chunk = ev.chunk;
    kvl = ev.kvl;
    part0 = (it.g * a.nRB + it.rb) * a.slots + ev.first;
  } else {
    if (!work_item(gridDim.x, a.nwork, a.S, a.nRB, a.spread, a.B, a.Hkv, blockIdx.x, it)) return;
    if (a.spread == 2) longest_first(a, blockIdx.x, it);
    kvl = context_rows(a, it.b);
    part0 = ((it.b * a.Hkv + it.g) * a.nRB + it.rb) * a.S;
  }
  const int s = it.s, rb = it.rb, g = it.g, b = it.b;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = wave % WR, wk = wave / WR;
  const int g4 = lane >> 4, l16 = lane & 15;

  const int r0 = rb * RB;
  const int rows = min(RB, a.M - r0);
  const int i_lo = r0 / a.G, i_hi = (r0 + rows - 1) / a.G;
  const Segment sg = segment(a, kvl, i_hi);
  const int nct = sg.nct, T = sg.T;
  const int ntt = i_hi / kKeyTile + 1;  // words of a node's ancestor bitmask
  const int t0 = s * chunk;
  const int t1 = min(T, t0 + chunk);
  if (t0 >= t1) return;  // empty chunk: the merge reads only chunks with tiles
  const bool has_tree = a.tail ? t1 * kKeyTile > kvl : t1 > nct;

  constexpr int RING = WK * NS * STAGE;
  const uint32_t ring = (uint32_t)(uintptr_t)smem + wk * NS * STAGE;
  const unsigned char* ring_ptr = smem + wk * NS * STAGE;
  // the block's queries (kShareQ) follow the rings, then the tree tables
  static_assert(!kShareQ || (WK > 1 && WR > 1), "queries are shared between key groups");
  constexpr bool qshare = kShareQ;
  const bool qload = !qshare || wk == 0;  // this wave loads its queries from memory
  unsigned char* qlds = smem + RING;
  uint32_t* anc = reinterpret_cast<uint32_t*>(smem + RING + (qshare ? RB * D * 2 : 0));
  const int anc_nodes = RB / a.G + 2;
  int32_t* par = reinterpret_cast<int32_t*>(anc + anc_nodes * ntt);
  int* flag = par + a.N;

  const size_t krow = (size_t)a.Hkv * D;  // elements between consecutive keys
  const size_t cache0 = kPaged ? 0 : (size_t)(b / a.cgroup) * a.Lmax * krow;  // paged: pool
  const __bf16* kcache = a.kc + cache0 + (size_t)g * D;
  const __bf16* vcache = a.vc + cache0 + (size_t)g * D;
  const size_t tree0 = (size_t)b * a.N * krow + (size_t)g * D;  // unused with a tree tail
  const __bf16* ktree = a.tail ? kcache : a.kt + tree0;
  const __bf16* vtree = a.tail ? vcache : a.vt + tree0;

  // This lane's share of the DMA instructions of one tile: instruction q
  // (q < kDma: K, else V) covers tile rows j*kRowsPerDma.. (j = q % kDma);
  // lane i fetches row j*kRowsPerDma + i/kCPR at the logical chunk that the
  // swizzle places at physical chunk i % kCPR.  dma_off is that byte offset
  // from the first row of a full tile.
  uint32_t dma_off[PW];
#pragma unroll
  for (int k = 0; k < PW; ++k) {
    const int q = wr * PW + k;
    const int r = (q % TL::kDma) * TL::kRowsPerDma + lane / TL::kCPR;
    dma_off[k] = (uint32_t)(r * (int)krow * 2 + ((lane % TL::kCPR) ^ TL::swz(r)) * 16);
  }
  const TreeSrc src{(const char*)kcache,
                    (const char*)vcache,
                    (const char*)ktree,
                    (const char*)vtree,
                    kPaged ? a.block_table + (size_t)b * a.max_blocks : nullptr,
                    a.block_shift,
                    a.num_blocks,
                    (int)krow * 2,
                    a.tail ? kvl + i_hi + 1 : kvl,
                    nct,
                    i_hi};

  // iteration i handles tile t0 + wk + WK*i of this wave's key group; all
  // waves run n_iter iterations so the per-iteration barriers line up
  const int n_iter = t1 > t0 ? (t1 - t0 + WK - 1) / WK : 0;
  const int n_mine = t0 + wk < t1 ? (t1 - t0 - wk + WK - 1) / WK : 0;  // valid tiles

  // Issue order: parents, queries, then the first tiles' DMAs, all before
  // any of them is used.  When the WR waves of a key group share its ring
  // (WR > 1) the prologue fills every stage: the ring's own refills come
  // after a workgroup barrier, and the first of them would otherwise wait
  // for the first tile's round trip.  A single-wave key group refills
  // before its waits and keeps one stage for that.  (Measured on the
  // Qwen3-8B-shaped 64-node, 4096-row call, together with the shared
  // queries below: 20.6 -> 19.6 us.)
  constexpr int kParPerThread = (kMaxNodes + kThreads - 1) / kThreads;
  constexpr int NQ = NT * NC;  // query loads per lane
  constexpr int kPro = WR > 1 ? NS : NS - 1;
  const int npro = min(kPro, n_mine);  // tiles the prologue issues
  int pv[kParPerThread];
  if (has_tree) {
    // indices clamped rather than branched on, so the loads stay in flight
    const int32_t* pr = a.parent + (size_t)b * a.N;
#pragma unroll
    for (int k = 0; k < kParPerThread; ++k) {
      const int i = tid + kThreads * k;
      pv[k] = a.parent ? load_i32(pr + (i < a.N ? i : a.N - 1)) : i - 1;  // NULL: a chain
    }
  }

  // ---- queries: B operand of S^T = K Q^T, lane holds Q[row l16][8*g4 .. +8]
  const int wrow0 = r0 + kRowsPerWave * wr;
  bf16x8 qf[NT][NC];
  bool qok[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int r = wrow0 + nt * 16 + l16;
    const bool ok = r < a.M;
    qok[nt] = ok;
    const int node = ok ? r / a.G : 0;
    const int h = g * a.G + (ok ? r % a.G : 0);
    const __bf16* qp = a.q + ((size_t)(b * a.N + node) * a.Hq + h) * D + 8 * g4;
    if (qload) {
#pragma unroll
      for (int c = 0; c < NC; ++c) qf[nt][c] = load_b128(qp + 32 * c);
    }
  }

#pragma unroll
  for (int i = 0; i < kPro; ++i)
    if (i < n_mine) issue_tile<D, PW, kPaged>(src, dma_off, wr, lane, t0 + wk + WK * i, ring + i * STAGE);

  // ---- tree structure: ancestor-or-self bitmask of this block's nodes
  if (has_tree) {
    // the parents are done once at most the queries and the DMAs are in flight
    wait_vm_any((qload ? NQ : 0) + npro * PW);
#pragma unroll
    for (int k = 0; k < kParPerThread; ++k) loaded(pv[k]);
    int bad = 0;
#pragma unroll
    for (int k = 0; k < kParPerThread; ++k) {
      const int i = tid + kThreads * k;
      if (i >= a.N) break;
      const int p = pv[k];
      par[i] = p;
      bad |= (i == 0) ? (p != -1) : (p < 0 || p >= i);
    }
    bad = __syncthreads_or(bad);
    const int nodes = i_hi - i_lo + 1;
    for (int t = tid; t < nodes; t += kThreads) {
      uint32_t* wd = anc + t * ntt;
      for (int k = 0; k < ntt; ++k) wd[k] = 0u;
      int u = i_lo + t;
      for (;;) {
        wd[u >> 5] |= 1u << (u & 31);
        if (u == 0) break;
        const int p = par[u];
        if (p < 0 || p >= u) break;  // invalid tree: the output becomes NaN
        u = p;
      }
    }
    if (tid == 0) *flag = bad;
    __syncthreads();
  }

  // the queries are done once at most the DMAs are in flight; rows past the
  // block's last row get zero queries.  Shared queries sit in LDS in the
  // tile layout, one 32-row tile per row group, read like the K operand.
  if (qload) {
    wait_vm_any(npro * PW);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        loaded(qf[nt][c]);
        if (!qok[nt]) qf[nt][c] = bf16x8{};
      }
  }
  // (the other key groups read them after the first ring step's barrier)
  unsigned char* qt = qlds + wr * TL::kBytes;
  if (qshare && wk == 0) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int c = 0; c < NC; ++c)
        *reinterpret_cast<bf16x8*>(qt + TL::off(16 * nt + l16, 4 * c + g4)) = qf[nt][c];
  }

  // O^T accumulators, and l: row sums of the bf16 weights, accumulated on
  // the matrix cores as ones^T P^T so numerator and denominator see the same
  // rounded weights (all 4 entries of lacc[nt] hold the lane's row sum)
  f32x4 o[DT][NT], lacc[NT];
  float m[NT];
  const bf16x8 ones = {(__bf16)1.f, (__bf16)1.f, (__bf16)1.f, (__bf16)1.f,
                       (__bf16)1.f, (__bf16)1.f, (__bf16)1.f, (__bf16)1.f};
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    m[nt] = -INFINITY;
    lacc[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[dt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // node of this lane's row in each 16-row tile, relative to i_lo
  int node_rel[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int r = wrow0 + nt * 16 + l16;
    node_rel[nt] = (r < a.M ? r : a.M - 1) / a.G - i_lo;
  }

  float thr[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) thr[nt] = -INFINITY;  // m = -inf: any visible score moves
  const float inv_c = 1.f / a.c;
  bf16x8 ones_v = ones;
  asm volatile("" : "+v"(ones_v));  // keep it in registers, not rebuilt every tile
  // Ring step of iteration i: wait for this key group's tile i and refill
  // the ring.  With WR > 1 the prologue issued tiles 0..NS-1 and step j >= 1
  // issues tile j+NS-1, so my DMAs of tile i are done once at most
  // min(later tiles, NS-1 at step 0, NS-2 after) tiles' DMAs are
  // outstanding; the barrier makes the whole group's visible and guarantees
  // the slot of tile i-1 is no longer read.
  auto ring_step = [&](int i) {
    const bool mine = i < n_mine;
    if (WR > 1) {
      if (mine) {
        if (i == 0) wait_tiles<PW, NS - 1>(n_mine - 1);
        else wait_tiles<PW, NS - 2>(n_mine - 1 - i);
      }
      __syncthreads();
      if (i >= 1 && i + NS - 1 < n_mine)
        issue_tile<D, PW, kPaged>(src, dma_off, wr, lane, t0 + wk + WK * (i + NS - 1),
                          ring + ((i + NS - 1) % NS) * STAGE);
    } else {
      if (i + NS - 1 < n_mine)
        issue_tile<D, PW, kPaged>(src, dma_off, wr, lane, t0 + wk + WK * (i + NS - 1),
                          ring + ((i + NS - 1) % NS) * STAGE);
      if (mine) wait_tiles<PW, NS - 1>(n_mine - 1 - i);
    }
  };
  // Full cache tiles first, without masking; the tiles that need a mask
  // (the cache tail, then the tree tiles) all come after them.  Shared
  // queries are read behind the first step's workgroup barrier: every
  // workgroup here has n_iter >= 1, so this loop always runs step 0.
  auto shared_queries = [&]() {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int c = 0; c < NC; ++c)
        qf[nt][c] = *reinterpret_cast<const bf16x8*>(qt + TL::off(16 * nt + l16, 4 * c + g4));
  };
  // a wave whose rows all lie past the last one only moves tiles
  const bool busy = wrow0 < a.M;
  uint32_t bits[NT] = {};
  int i = 0;
  for (; i < n_iter; ++i) {
    ring_step(i);
    if (i == 0 && qshare && wk != 0) shared_queries();
    const int t = t0 + wk + WK * i;
    if (i >= n_mine || t >= nct || (t + 1) * kKeyTile > kvl) break;
    if (!busy) continue;
    attend_tile<D, NT, false>(ring_ptr + (i % NS) * STAGE, qf, o, lacc, m, thr, ones_v, a.c, inv_c,
                              bits, g4, l16);
  }
  for (bool stepped = true; i < n_iter; ++i, stepped = false) {
    if (!stepped) ring_step(i);
    if (i >= n_mine || !busy) continue;
    const int t = t0 + wk + WK * i;
    tile_bits<NT>(MaskInfo{t, nct, kvl, ntt, a.tail, anc}, node_rel, bits);
    attend_tile<D, NT, true>(ring_ptr + (i % NS) * STAGE, qf, o, lacc, m, thr, ones_v, a.c, inv_c,
                             bits, g4, l16);
  }

  const LateArgs* z = late_args();
  float lsum[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) lsum[nt] = lacc[nt][0];
  const int invalid = has_tree ? *flag : 0;
  // Only chunks that hold tiles take part in a merge, nval of them; a row
  // block that is one chunk needs none and writes its output here.
  const int nval = (T + chunk - 1) / chunk;
  const bool whole = z->S == 1 || nval == 1;
  const int bg = b * z->Hkv + g;
  const size_t grp = (size_t)bg * z->nRB + rb;  // row block id

  // Final values of 16x16 fragments (dt, ntg) of this workgroup's rows: either
  // the normalised bf16 output (single chunk) or the chunk partial.  Fragments
  // wholly past the last row are neither stored here nor read by the merges,
  // which the plan's cost counts on (2 x 3 nodes, 32 heads on 8, 1361 rows: 19.0
  // -> 16.9 us; 64 x 2 nodes 55.5 -> 50.8; 16 x 33 nodes 53.0 -> 51.2).
  auto rows_at = [&](int ntg) { return r0 + ntg * 16 < z->M; };
  auto emit_out = [&](int dt, int ntg, const f32x4& acc, float l) {
    const int r = r0 + ntg * 16 + l16;
    if (r < z->M) {
      const int node = r / z->G, h = g * z->G + r % z->G;
      store_out4(z->out + ((size_t)(b * z->N + node) * z->Hq + h) * D + 16 * dt + 4 * g4, acc,
                 1.f / l, invalid != 0);
    }
  };
  auto emit_part = [&](bool dev, int dt, int ntg, const f32x4& acc, float mstar, float l) {
    f32x4* po = &z->ws_o[((size_t)(part0 + s) * DT * NTG + dt * NTG + ntg) * 64 + lane];
    float2* pml = &z->ws_ml[(size_t)(part0 + s) * RB + ntg * 16 + l16];
    if (dev) {  // read by another workgroup of this kernel
      store_dev(po, acc);
      if (dt == 0 && g4 == 0) store_dev(pml, make_float2(mstar, l));
    } else {    // read by the merge kernel
      *po = acc;
      if (dt == 0 && g4 == 0) *pml = make_float2(mstar, l);
    }
  };

  if (WK == 1) {
    // The kind of store is settled once per row tile, not at every fragment.
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const int ntg = wr * NT + nt;
      if (!rows_at(ntg)) break;
      if (whole) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) emit_out(dt, ntg, o[dt][nt], lsum[nt]);
      } else if (z->fused) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) emit_part(true, dt, ntg, o[dt][nt], m[nt], lsum[nt]);
      } else {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) emit_part(false, dt, ntg, o[dt][nt], m[nt], lsum[nt]);
      }
    }
  } else {
    // ---- merge the WK key groups of each row group (same rows, disjoint keys)
    __syncthreads();  // rings and tree tables are dead from here on
    f32x4* obuf = reinterpret_cast<f32x4*>(smem);
    float2* mlbuf = reinterpret_cast<float2*>(smem + (size_t)kWaves * kRowsPerWave * D * 4);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) obuf[((wave * DT + dt) * NT + nt) * 64 + lane] = o[dt][nt];
    if (g4 == 0) {
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
        mlbuf[wave * kRowsPerWave + nt * 16 + l16] = make_float2(m[nt], lsum[nt]);
    }
    __syncthreads();
    for (int f = wk; f < DT * NT; f += WK) {
      const int dt = f / NT, nt = f % NT;
      if (!rows_at(wr * NT + nt)) continue;
      const int rw = nt * 16 + l16;  // row within the wave's 32
      float mw[WK], mstar = -INFINITY;
#pragma unroll
      for (int k = 0; k < WK; ++k) {
        mw[k] = mlbuf[(k * WR + wr) * kRowsPerWave + rw].x;
        mstar = fmaxf(mstar, mw[k]);
      }
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
      float l = 0.f;
#pragma unroll
      for (int k = 0; k < WK; ++k) {
        const float e = mw[k] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mw[k] - mstar);
        l += e * mlbuf[(k * WR + wr) * kRowsPerWave + rw].y;
        acc += e * obuf[(((k * WR + wr) * DT + dt) * NT + nt) * 64 + lane];
      }
      if (whole) emit_out(dt, wr * NT + nt, acc, l);
      else if (z->fused) emit_part(true, dt, wr * NT + nt, acc, mstar, l);
      else emit_part(false, dt, wr * NT + nt, acc, mstar, l);
    }
  }
  if (whole || !z->fused) return;

  // ---- fused split-KV merge: the chunk that arrives last merges its row
  // block.  Every workgroup publishes its partial (device-scope stores,
  // completed before the count), then counts itself in; the one that
  // completes the count merges and resets the counter for the next call.
  __shared__ int s_last;
  if (has_tree && tid == 0)  // every row block has a chunk with tree tiles
    __hip_atomic_store(z->tree_bad + grp, invalid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  wait_all_vm();
  __syncthreads();
  if (tid == 0) {
    const unsigned int before =
        __hip_atomic_fetch_add(z->arrived + grp, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const bool last = before + 1 == (unsigned int)nval;
    if (last) __hip_atomic_store(z->arrived + grp, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_last = last;
  }
  __syncthreads();
  if (!s_last) return;
  const bool bad = __hip_atomic_load(z->tree_bad + grp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
  merge_chunks<D, RB, kWaves>(z, part0, nval, b, g, r0, bad, wave, lane);
}

// Training mask, several blocks to a workgroup.  The A blocks of an example read
// the same context up to their anchors.  With one block per workgroup a block of
// S * G <= 64 rows leaves a workgroup of four waves half empty, or (two waves)
// moves every tile through LDS for its few rows only, and what bounds it is the
// tiles' way into LDS.  So nb blocks with neighbouring anchors (pack_order sorts
// them, largest first) share a workgroup of 128 rows: row R belongs to block
// R / M of the pack.  The workgroup streams the context up to its largest anchor,
// then every block's own keys; a wave skips the tiles none of its rows sees, and
// a row's visible keys are counted per row (key < anchor in the context, key <=
// position in its own block).  A ring of four tiles (64 KB) lets two workgroups
// share a CU.  Now bound by the matrix products and the softmax between them.
// Measured (8 KV heads, D = 128 unless said, random anchors): one example of 512
// blocks of 16, G = 4, 4096 positions: 350 -> 292 us; 2 x 200 blocks of 8, G = 4,
// 2048: 185 -> 91; 3 x 223 blocks of 32, G = 1, 390: 183 -> 74; 3 x 300 of 16,
// G = 2, D = 64, 1000: 258 -> 87; pack_order 5-7 us of each.  When it is taken:
// tv_plan.h, pack_plan.
struct PackArgs {
  const __bf16* q;
  const __bf16* kc;
  const __bf16* vc;
  const __bf16* kt;
  const __bf16* vt;
  const int32_t* anchors;
  const int32_t* order;  // [B, A]: the example's blocks, largest anchor first
  __bf16* out;
  int B, A, S, Hq, Hkv, L, G, M, nb, packs;
  float c;
};

// Place of each of an example's blocks by anchor: kPackRank blocks per workgroup,
// every workgroup with all keys in LDS, four lanes per block on a quarter of them
// each, four at a time.
__global__ __launch_bounds__(4 * kPackRank) void pack_order(const int32_t* anchors, int32_t* order,
                                                            int A) {
  __shared__ __attribute__((aligned(16))) int key[kPackMaxBlocks];
  const int per = (A + kPackRank - 1) / kPackRank, b = blockIdx.x / per, A16 = (A + 15) & ~15;
  for (int i = threadIdx.x; i < A16; i += 4 * kPackRank)
    key[i] = i < A ? anchors[(size_t)b * A + i] : INT32_MIN;
  __syncthreads();
  const int i = (int)(blockIdx.x % per) * kPackRank + (int)(threadIdx.x >> 2);
  const int v = i < A ? key[i] : 0;
  int rank = 0;
  for (int j = 4 * (int)(threadIdx.x & 3); j < A16; j += 16) {
    const int4 k = *(const int4*)(key + j);
    rank += k.x > v || (k.x == v && j < i);
    rank += k.y > v || (k.y == v && j + 1 < i);
    rank += k.z > v || (k.z == v && j + 2 < i);
    rank += k.w > v || (k.w == v && j + 3 < i);
  }
  rank += __shfl_xor(rank, 1);
  rank += __shfl_xor(rank, 2);
  if (i < A && (threadIdx.x & 3) == 0) order[(size_t)b * A + rank] = i;
}

template <int D>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void attn_packed(PackArgs a) {
  using TL = TileLayout<D>;
  constexpr int WR = kPackRows / kRowsPerWave, NS = 4;
  constexpr int NT = kRowsPerWave / 16, NC = D / 32, DT = D / 16;
  constexpr int STAGE = 2 * TL::kBytes, PW = 2 * TL::kDma / WR, NQ = NT * NC;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int lane = threadIdx.x & 63, g4 = lane >> 4, l16 = lane & 15;
  const int wr = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  // KV heads in turn, then examples; the packs of the largest anchors come first.
  // Workgroups go to the XCDs in turn too, so an XCD reads the context of Hkv /
  // gcd(8, Hkv) heads: one with 8 of them, all where their number is odd.
  const int g = (int)blockIdx.x % a.Hkv, u = (int)blockIdx.x / a.Hkv;
  const int b = u % a.B, p = u / a.B;
  if (p >= a.packs) return;

  // the pack's blocks, one per lane
  const int nv = min(a.nb, a.A - p * a.nb);
  const int mine = lane < nv ? a.order[(size_t)b * a.A + p * a.nb + lane] : 0;
  int anchor = lane < nv ? a.anchors[(size_t)b * a.A + mine] : 0;
  anchor = anchor < 0 ? 0 : (anchor > a.L ? a.L : anchor);
  const int ntt = (a.S - 1) / kKeyTile + 1;

  // this lane's rows
  int blk[NT], node[NT];
  size_t orow[NT];
  bool ok[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int R = kRowsPerWave * wr + 16 * nt + l16, rr = R % a.M;
    blk[nt] = R / a.M;
    ok[nt] = blk[nt] < nv;
    node[nt] = rr / a.G;
    const int src = ok[nt] ? blk[nt] : 0;
    orow[nt] = (((size_t)b * a.A + __shfl(mine, src)) * a.S + node[nt]) * a.Hq + g * a.G + rr % a.G;
  }
  const int blk_lo = kRowsPerWave * wr / a.M, blk_hi = (kRowsPerWave * (wr + 1) - 1) / a.M;

  const size_t krow = (size_t)a.Hkv * D;
  const size_t cache0 = (size_t)b * a.L * krow + (size_t)g * D;
  uint32_t dma_off[PW];
#pragma unroll
  for (int k = 0; k < PW; ++k) {
    const int r = ((wr * PW + k) % TL::kDma) * TL::kRowsPerDma + lane / TL::kCPR;
    dma_off[k] = (uint32_t)(r * (int)krow * 2 + ((lane % TL::kCPR) ^ TL::swz(r)) * 16);
  }
  const char* kctx = uniform_ptr((const char*)(a.kc + cache0));
  const char* vctx = uniform_ptr((const char*)(a.vc + cache0));

  bf16x8 qf[NT][NC];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int cc = 0; cc < NC; ++cc) {
      const bf16x8 v =
          *reinterpret_cast<const bf16x8*>(a.q + orow[nt] * D + 8 * g4 + 32 * cc);
      qf[nt][cc] = ok[nt] ? v : bf16x8{};
    }
  // (the queries are in before the first tiles go out: the compiler's wait for
  // them would otherwise drain the tiles too)
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int cc = 0; cc < NC; ++cc) asm volatile("" : "+v"(qf[nt][cc]));
  // one pass over all blocks, or one per block (below)
  for (int j0 = 0, j1 = nv;;) {
    // the pass's tiles: the context up to its blocks' largest anchor, then their own
    const bool in = lane >= j0 && lane < j1;
    const int longest = (int)wave_max_u32(in ? (unsigned)anchor : 0u);
    const int nct = (longest + kKeyTile - 1) / kKeyTile, T = nct + (j1 - j0) * ntt;
    // its rows, and the smallest and largest of the wave's anchors
    bool on[NT];
    int kvl[NT], lo = a.L, hi = 0;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      on[nt] = ok[nt] && blk[nt] >= j0 && blk[nt] < j1;
      kvl[nt] = __shfl(anchor, blk[nt] & 63);
      if (!on[nt]) kvl[nt] = 0;
      else lo = min(lo, kvl[nt]);
      hi = max(hi, kvl[nt]);
    }
    lo = a.L - (int)wave_max_u32((unsigned)(a.L - lo));
    hi = (int)wave_max_u32((unsigned)hi);
    if (hi == 0) lo = 0;  // no context, or no rows
    // tile t: of the context, or of block j0 + (t - nct) / ntt's own keys
    auto issue = [&](int t) {
      TreeSrc src{kctx, vctx, kctx, vctx, nullptr, 0, 0, (int)krow * 2, longest, nct, a.S - 1};
      if (t >= nct) {
        const int j = j0 + (t - nct) / ntt;
        const size_t own =
            ((size_t)b * a.A + __builtin_amdgcn_readlane(mine, j)) * a.S * krow + (size_t)g * D;
        src.ktree = uniform_ptr((const char*)(a.kt + own));
        src.vtree = uniform_ptr((const char*)(a.vt + own));
        src.nct = nct + (j - j0) * ntt;
      }
      issue_tile<D, PW, false>(src, dma_off, wr, lane, t, (uint32_t)(uintptr_t)smem + (t % NS) * STAGE);
    };

#pragma unroll
    for (int t = 0; t < NS; ++t)
      if (t < T) issue(t);

    f32x4 o[DT][NT], lacc[NT];
    float m[NT], thr[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      m[nt] = thr[nt] = -INFINITY;
      lacc[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) o[dt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    bf16x8 ones = {(__bf16)1.f, (__bf16)1.f, (__bf16)1.f, (__bf16)1.f,
                   (__bf16)1.f, (__bf16)1.f, (__bf16)1.f, (__bf16)1.f};
    asm volatile("" : "+v"(ones));
    const float inv_c = 1.f / a.c;
    uint32_t bits[NT] = {};
    auto ring_step = [&](int t) {
      if (t == 0) wait_tiles<PW, NS - 1>(T - 1);
      else wait_tiles<PW, NS - 2>(T - 1 - t);
      __syncthreads();
      if (t >= 1 && t + NS - 1 < T) issue(t + NS - 1);
    };
    int t = 0;
    for (; t < T; ++t) {  // context tiles that all of the wave's rows see whole
      ring_step(t);
      if (t >= nct || (t + 1) * kKeyTile > lo) break;
      attend_tile<D, NT, false>(smem + (t % NS) * STAGE, qf, o, lacc, m, thr, ones, a.c, inv_c, bits,
                                g4, l16);
    }
    for (bool stepped = true; t < T; ++t, stepped = false) {
      if (!stepped) ring_step(t);
      const int j = t < nct ? 0 : j0 + (t - nct) / ntt;
      if (t < nct ? t * kKeyTile >= hi : (j < blk_lo || j > blk_hi)) continue;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
        bits[nt] = t < nct ? first_keys(kvl[nt] - t * kKeyTile)
                           : (blk[nt] == j ? first_keys(node[nt] + 1 - (t - nct) % ntt * kKeyTile) : 0u);
      attend_tile<D, NT, true>(smem + (t % NS) * STAGE, qf, o, lacc, m, thr, ones, a.c, inv_c, bits, g4,
                               l16);
    }
    // Non-finite outputs: a value that is an infinity or NaN reaches, times a
    // weight of zero, rows of the pack that do not see its key.  Then every block
    // is done again by itself.
    if (j0 == 0 && j1 == nv && nv > 1) {
      bool bad = false;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            uint32_t w = __float_as_uint(o[dt][nt][e]);
            asm("" : "+v"(w));  // (no assumption that it is a number)
            bad |= on[nt] && (w & 0x7f800000u) == 0x7f800000u;
          }
      if (__syncthreads_or(bad)) {
        j1 = 1;
        continue;
      }
      j1 = nv + 1;  // done after the store
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      if (!on[nt]) continue;
      const float inv = 1.f / lacc[nt][0];
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
        store_out4(a.out + orow[nt] * D + 16 * dt + 4 * g4, o[dt][nt], inv, false);
    }
    if (j1 >= nv) return;
    __syncthreads();  // the ring is free
    j0 = j1++;
  }
}

// Second kernel of the split-KV plans whose merge is too large for one
// workgroup: out = sum_s e_s O_s / sum_s e_s l_s with e_s = 2^(m_s - m*),
// folded in online over batches of U chunks.  Only chunks that hold tiles
// of this row block were written.  One wave per 16x16 fragment.  The
// parents (for the tree check), kv_len and the first batch of partials are
// all requested before any is used, so a merge of up to U chunks waits for
// one round of memory latency: the first batch reads the slots of the
// first min(S, U) chunks whether or not they were written by this call
// (they lie inside the workspace), and only the nval chunks that hold
// tiles, known once kv_len arrives, are folded in.
template <int D, int RB>
__global__ __launch_bounds__(256) void attn_combine(AttnArgs a) {
  constexpr int NTG = RB / 16, DT = D / 16, U = 16;
  constexpr int kParPerThread = kMaxNodes / 256;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g4 = lane >> 4, l16 = lane & 15;
  const int F = blockIdx.x * 4 + wave;  // fragment id; all 4 of a block share (b,g,rb)
  const int per_blk = DT * NTG;
  const int blk = F / per_blk, f = F % per_blk;
  const int rb = blk % a.nRB, bg = blk / a.nRB;
  const int b = bg / a.Hkv, g = bg % a.Hkv;
  int pv[kParPerThread];
#pragma unroll
  for (int k = 0; k < kParPerThread; ++k) {
    const int i = threadIdx.x + 256 * k;
    pv[k] = i >= a.N ? 0 : (a.parent ? a.parent[(size_t)b * a.N + i] : i - 1);
  }
  const int dt = f / NTG, ntg = f % NTG;
  const int row = ntg * 16 + l16, r = rb * RB + row;
  // chunks of this row block that hold tiles (the same count the main
  // kernel derives from kv_len and the block's last node)
  const int i_hi = (min(rb * RB + RB, a.M) - 1) / a.G;
  // the first chunk partial, and the partials from there on
  EvenItem ev{a.chunk, b, 0, 0, 0};
  size_t base = (size_t)(bg * a.nRB + rb) * a.S;
  int nslot = a.S;
  if (a.slots > 0) {
    if (a.B > 1) ev = even_split<false>(a, -1, b, 0);
    base = (size_t)(g * a.nRB + rb) * a.slots + ev.first;
    nslot = a.slots - ev.first;
  }
  float2 ml0[U];
  f32x4 ov0[U];
  const bool any = rb * RB + ntg * 16 < a.M;  // else no rows: nothing was stored
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (u < nslot && any) {
      ml0[u] = a.ws_ml[(base + u) * RB + row];
      ov0[u] = a.ws_o[((base + u) * DT * NTG + dt * NTG + ntg) * 64 + lane];
    }
  if (a.slots == 0) ev.kvl = context_rows(a, b);
  else if (a.B == 1) ev = even_one<false>(a, 0, 0);
  const int T = segment(a, ev.kvl, i_hi).T;
  int nval = (T + ev.chunk - 1) / ev.chunk;
  if (nval == 1) return;  // written by its only chunk
  if (!any) nval = 0;
  float m = -INFINITY, l = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < nval; s0 += U) {
    float2 ml[U];
    f32x4 ov[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (s0 + u < nval) {
        if (s0 == 0) {
          ml[u] = ml0[u];
          ov[u] = ov0[u];
        } else {
          ml[u] = a.ws_ml[(base + s0 + u) * RB + row];
          ov[u] = a.ws_o[((base + s0 + u) * DT * NTG + dt * NTG + ntg) * 64 + lane];
        }
      }
    float mb = m;
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (s0 + u < nval) mb = fmaxf(mb, ml[u].x);
    if (mb != -INFINITY) {  // else every chunk so far saw no key: nothing to add
      const float ea = __builtin_amdgcn_exp2f(m - mb);  // 0 while m = -inf
      l *= ea;
      acc *= ea;
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (s0 + u < nval && ml[u].x != -INFINITY) {
          const float e = __builtin_amdgcn_exp2f(ml[u].x - mb);
          l += e * ml[u].y;
          acc += e * ov[u];
        }
      m = mb;
    }
  }
  int bad = 0;
#pragma unroll
  for (int k = 0; k < kParPerThread; ++k) {
    const int i = threadIdx.x + 256 * k;
    if (i < a.N) bad |= (i == 0) ? (pv[k] != -1) : (pv[k] < 0 || pv[k] >= i);
  }
  bad = __syncthreads_or(bad);
  if (r >= a.M) return;
  const int node = r / a.G, h = g * a.G + r % a.G;
  store_out4(a.out + ((size_t)(b * a.N + node) * a.Hq + h) * D + 16 * dt + 4 * g4, acc, 1.f / l,
             bad != 0);
}

template <int D, int WR, int WK, int NS, bool kPaged, bool kShareQ>
static hipError_t launch_main(const AttnArgs& a, const AttnPlan& p, hipStream_t st) {
  // the kernel's LDS limit on each device, raised only when a call needs more
  constexpr int kDevices = 64;
  static std::atomic<int> limit[kDevices];
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kDevices) return hipErrorInvalidDevice;
  if (limit[dev].load(std::memory_order_acquire) < (int)p.lds_bytes) {
    static std::mutex raising;
    std::lock_guard<std::mutex> hold(raising);
    if (limit[dev].load(std::memory_order_relaxed) < (int)p.lds_bytes) {
      e = hipFuncSetAttribute((const void*)attn_main<D, WR, WK, NS, kPaged, kShareQ>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)p.lds_bytes);
      if (e != hipSuccess) return e;
      limit[dev].store((int)p.lds_bytes, std::memory_order_release);
    }
  }
  hipLaunchKernelGGL((attn_main<D, WR, WK, NS, kPaged, kShareQ>),
                     dim3(p.slots > 0 ? p.even_grid : p.grid), dim3(64 * WR * WK),
                     p.lds_bytes, st, a);
  return hipGetLastError();
}

template <int D, int ARR, bool kPaged>
static hipError_t launch_attn_t(const AttnArgs& a, const AttnPlan& p, hipStream_t st) {
  constexpr Arrangement ar = kArrangements[ARR];
  constexpr int NS = arr_stages(ar, D);
  if constexpr (NS == 0) {
    return hipErrorInvalidValue;  // never planned: the ring does not fit
  } else {
    // query sharing is a separate instantiation, so the kernels without it
    // carry none of its code or scalar registers
    hipError_t e;
    if constexpr (ar.WK > 1 && ar.WR > 1)
      e = p.qshare ? launch_main<D, ar.WR, ar.WK, NS, kPaged, true>(a, p, st)
                   : launch_main<D, ar.WR, ar.WK, NS, kPaged, false>(a, p, st);
    else
      e = launch_main<D, ar.WR, ar.WK, NS, kPaged, false>(a, p, st);
    if (e != hipSuccess || p.S == 1 || p.fused) return e;
    constexpr int RB = kRowsPerWave * ar.WR;
    const int frags = a.B * a.Hkv * p.nRB * (D / 16) * (RB / 16);
    hipLaunchKernelGGL((attn_combine<D, RB>), dim3(frags / 4), dim3(256), 0, st, a);
    return hipGetLastError();
  }
}

template <int D, int K = 0>
static hipError_t launch_attn_d(const AttnArgs& a, const AttnPlan& p, hipStream_t st) {
  if constexpr (K < kNumArrangements) {
    if (p.arr == K)
      return a.block_table ? launch_attn_t<D, K, true>(a, p, st)
                           : launch_attn_t<D, K, false>(a, p, st);
    return launch_attn_d<D, K + 1>(a, p, st);
  } else {
    return hipErrorInvalidValue;
  }
}

hipError_t launch_attention(const void* q, const void* kc, const void* vc, const void* kt,
                            const void* vt, const int32_t* parent, const int32_t* kv_len,
                            void* out, int B, int N, int Hq, int Hkv, int D, int Lmax,
                            float scale, void* ws, const AttnPlan& p, hipStream_t st,
                            const int32_t* block_table, int block_shift, int max_blocks,
                            int num_blocks, int cgroup) {
  AttnArgs a;
  a.tail = kt == nullptr;
  a.cgroup = cgroup;
  a.block_table = block_table;
  a.block_shift = block_shift;
  a.max_blocks = max_blocks;
  a.num_blocks = num_blocks;
  a.q = (const __bf16*)q;
  a.kc = (const __bf16*)kc;
  a.vc = (const __bf16*)vc;
  a.kt = (const __bf16*)kt;
  a.vt = (const __bf16*)vt;
  a.parent = parent;
  a.kv_len = kv_len;
  a.out = (__bf16*)out;
  a.arrived = (unsigned int*)ws;
  a.tree_bad = (int*)ws + kSyncGroups;
  a.ws_o = (f32x4*)((char*)ws + p.ws_sync_bytes);
  a.ws_ml = (float2*)((char*)ws + p.ws_sync_bytes + p.ws_o_bytes);
  a.B = B;
  a.N = N;
  a.Hq = Hq;
  a.Hkv = Hkv;
  a.Lmax = Lmax;
  a.G = p.G;
  a.M = p.M;
  a.nRB = p.nRB;
  a.S = p.S;
  a.chunk = p.chunk;
  a.nwork = p.nwork;
  a.fused = p.fused;
  a.spread = p.spread;
  a.slots = p.slots;
  a.min_chunk = p.min_chunk;
  a.rslots = p.slots > 0 ? 1.f / (float)p.slots : 0.f;
  a.rslack = p.slots > B ? 1.f / (float)(p.slots - B) : 1.f;
  a.c = scale * 1.4426950408889634f;
  return D == 128 ? launch_attn_d<128>(a, p, st) : launch_attn_d<64>(a, p, st);
}

template <int D>
static hipError_t launch_packed_d(const PackArgs& a, hipStream_t st) {
  constexpr int lds = 4 * 2 * TileLayout<D>::kBytes;  // at most 64 KB: no limit to raise
  static_assert(lds <= 64 * 1024, "the ring");
  const dim3 grid(kXcds * cdiv((long long)a.B * a.packs * a.Hkv, kXcds));
  hipLaunchKernelGGL(attn_packed<D>, grid, dim3(256), lds, st, a);
  return hipGetLastError();
}

hipError_t launch_packed(const void* q, const void* kc, const void* vc, const void* kt, const void* vt,
                         const int32_t* anchors, void* out, int B, int A, int S, int Hq, int Hkv, int D,
                         int L, float scale, void* ws, const PackPlan& p, hipStream_t st) {
  int32_t* order = (int32_t*)((char*)ws + kSyncBytes);
  hipLaunchKernelGGL(pack_order, dim3(B * cdiv(A, kPackRank)), dim3(4 * kPackRank), 0, st, anchors,
                     order, A);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  PackArgs a{(const __bf16*)q, (const __bf16*)kc, (const __bf16*)vc, (const __bf16*)kt,
             (const __bf16*)vt, anchors, order, (__bf16*)out, B, A, S, Hq, Hkv, L, Hq / Hkv,
             S * (Hq / Hkv), p.nb, p.packs, scale * 1.4426950408889634f};
  return D == 128 ? launch_packed_d<128>(a, st) : launch_packed_d<64>(a, st);
}

}  // namespace tv
