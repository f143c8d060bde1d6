// Host-side launch planning shared by the entry points and the kernels'
// launchers.  Pure C++ (no HIP): the plans depend only on host-known sizes.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace tv {

constexpr int kKeyTile = 32;       // keys one wave consumes per step
constexpr int kXcds = 8;           // MI355X accelerator complex dies
constexpr int kMaxRankPairs = 1024;  // longest-first ranking: pairs per XCD lane (16 per lane)
constexpr int kMaxNodes = 2048;    // == TV_MAX_NODES

inline int cdiv(long long a, long long b) { return (int)((a + b - 1) / b); }

// Attention work decomposition.  Rows of one (sequence, KV head) pair are the
// N*G (node, query-head-in-group) pairs, row r = node * G + head_in_group.
// A workgroup takes a block of RB = 32*WR consecutive rows and one
// fixed-size chunk of the key tiles (cache tiles first, then tree tiles).
// Its WR*WK waves form WR row groups (32 rows per wave) times WK key groups
// that split the chunk's tiles between them; each key group streams its
// tiles through an LDS ring of NS stages.  Arrangements are sized so that a
// CU holds 8 waves (two per SIMD), from one or more workgroups.
constexpr int kRowsPerWave = 32;
// Split-KV plans keep per-row-block sync words (arrival counter, tree flag)
// in a fixed region at the start of the workspace, the same place for every
// shape, so that one zero-filled workspace can serve calls of any sizes: a
// call's partials never overlap another call's counters, and each call
// leaves its counters at zero.  Plans with more row blocks do not split.
constexpr int kSyncGroups = 4096;
constexpr size_t kSyncBytes = (size_t)kSyncGroups * 8;
constexpr int kWavesPerCU = 8;
constexpr int kEvenSequences = 1024;  // batches the even split takes (up to 16 per lane)
constexpr int kEvenTiles = 1 << 20;   // key tiles a sequence of it has fewer than
constexpr size_t kMaxLds = 160 * 1024;

struct Arrangement {
  int WR, WK, NS128, NS64;
};
// WR x WK waves; ring stages for D = 128 and D = 64 (16 KB / 8 KB stages)
constexpr Arrangement kArrangements[] = {
    {8, 1, 4, 4}, {4, 2, 4, 4}, {2, 4, 2, 4}, {1, 8, 0, 2},
    {4, 1, 4, 4}, {2, 2, 2, 4}, {2, 1, 2, 4},
};
constexpr int kNumArrangements = sizeof(kArrangements) / sizeof(kArrangements[0]);

constexpr int arr_stages(const Arrangement& a, int D) { return D == 128 ? a.NS128 : a.NS64; }

struct AttnPlan {
  int arr;                     // index into kArrangements
  int WR, WK, NS, threads, wg_per_cu;
  int G, M, RB, nRB, S, chunk;
  int nwork, grid;             // work items, launched workgroups (x8 padded)
  int fused;                   // S > 1: merge in the main kernel's last chunk (else a second kernel)
  int spread;                  // work order of several sequences (below)
  int slots, min_chunk, even_grid;  // even split (below), else slots = 0
  size_t ws_o_bytes, ws_ml_bytes, ws_sync_bytes, ws_bytes;
  size_t lds_bytes;            // dynamic LDS of the main kernel
  int qshare;                  // key group 0 loads the queries, the others read them from LDS
};

// Dynamic LDS of the main kernel: the rings, then (qshare) the block's
// queries, then the tree tables; the key-group merge reuses it afterwards.
inline size_t attn_lds_bytes(int D, int WR, int WK, int NS, int G, int N, bool qshare) {
  const int RB = kRowsPerWave * WR;
  const size_t stage = 2 * (size_t)kKeyTile * 2 * D;
  const size_t ring = (size_t)WK * NS * stage + (qshare ? (size_t)RB * D * 2 : 0);
  const int words = cdiv(N, 32);
  const int nodes = RB / G + 2;
  const size_t tree = (size_t)nodes * words * 4 + (size_t)N * 4 + 16;
  const size_t waves = (size_t)WR * WK;
  const size_t merge = WK == 1 ? 0 : waves * kRowsPerWave * D * 4 + waves * kRowsPerWave * 8;
  const size_t a = ring + tree;
  return a > merge ? a : merge;
}

// The plan for one arrangement and `want` chunks per (KV head, row block) over
// all sequences (at least B; B: no split), of one size for the whole batch or
// (even = false) want / B of each sequence's capacity.
inline AttnPlan attn_plan_arr(int B, int N, int Hq, int Hkv, int D, int Lmax, int arr, long long want,
                              bool even = true) {
  const Arrangement& ar = kArrangements[arr];
  AttnPlan p{};
  p.arr = arr;
  p.WR = ar.WR;
  p.WK = ar.WK;
  p.NS = arr_stages(ar, D);
  p.threads = 64 * ar.WR * ar.WK;
  p.G = Hq / Hkv;
  p.wg_per_cu = kWavesPerCU / (ar.WR * ar.WK);
  p.lds_bytes = p.NS > 0 ? attn_lds_bytes(D, ar.WR, ar.WK, p.NS, p.G, N, false) : kMaxLds + 1;
  p.M = N * p.G;
  p.RB = kRowsPerWave * ar.WR;
  p.nRB = cdiv(p.M, p.RB);
  const int tiles = cdiv(Lmax, kKeyTile) + cdiv(N, kKeyTile);
  const long long base = (long long)B * Hkv * p.nRB;
  const int min_chunk = 2 * ar.WK;  // >= 2 tiles per key group
  const long long max_s = tiles / min_chunk > 1 ? tiles / min_chunk : 1;
  long long S = (want + B - 1) / B;
  if (S > max_s) S = max_s;
  if (S < 1 || base > kSyncGroups || (even && (B > kEvenSequences || tiles >= kEvenTiles))) S = 1;
  p.chunk = cdiv(tiles, S);
  p.S = cdiv(tiles, p.chunk);
  p.nwork = (int)(base * p.S);
  p.grid = cdiv(p.nwork, kXcds) * kXcds;
  if (p.S > 1 && even) {
    p.slots = (int)(want < (long long)B * p.S ? want : (long long)B * p.S);
    p.min_chunk = min_chunk;
    p.even_grid = kXcds * p.nRB * cdiv((long long)p.slots * Hkv, kXcds);
  }
  const int DT = D / 16, NTG = p.RB / 16;
  if (p.S > 1) {
    // sync region (counters, then tree flags), chunk partials: O fragments,
    // then (m, l) per row
    p.ws_sync_bytes = kSyncBytes;
    p.ws_o_bytes = (size_t)B * Hkv * p.nRB * p.S * DT * NTG * 64 * 16;
    p.ws_ml_bytes = (size_t)B * Hkv * p.nRB * p.S * p.RB * 8;
  }
  p.ws_bytes = p.ws_sync_bytes + p.ws_o_bytes + p.ws_ml_bytes;
  // With several key groups every one of them needs the block's queries.
  // When the grid fills every CU, key group 0 loads them and shares them
  // through LDS where that fits: the other groups' copies were 64 KB of
  // requests per workgroup ahead of the first tiles at the Qwen3-8B-shaped
  // 64-node call (2 x 4 waves; 2% faster shared).  On a GPU left mostly
  // idle the copies cost nothing and the LDS hop only adds latency (3%
  // slower for a grid of two workgroups).
  p.qshare = 0;
  if (p.NS > 0 && ar.WK > 1 && ar.WR > 1 && p.nwork >= 256LL * p.wg_per_cu) {
    const size_t with_q = attn_lds_bytes(D, ar.WR, ar.WK, p.NS, p.G, N, true);
    if (with_q * p.wg_per_cu <= kMaxLds) {
      p.qshare = 1;
      p.lds_bytes = with_q;
    }
  }
  // Workgroups go to the XCDs round-robin, and the row blocks of one
  // (sequence, KV head, chunk) read the same keys, so they stay on one XCD
  // (its L2).  With one sequence, XCD x takes a contiguous run of work
  // items.  With several sequences of different lengths that would give
  // each XCD whole sequences and very different work, so each XCD instead
  // takes one KV head and one of L = 8/Hkv lanes of chunks: chunk s of
  // sequence b goes to lane (b + s) % L.  Every XCD then sees every
  // sequence.  This needs Hkv to divide 8 and L to divide S.  (Plans with
  // an even split map their workgroups by its chunks instead.)
  p.spread = p.slots == 0 && B > 1 && kXcds % Hkv == 0 && p.S % (kXcds / Hkv) == 0;
  // Within an XCD workgroups start in index order as slots free up, so a
  // long chunk that starts in a late round sets the kernel's end.  When an
  // XCD's (sequence, chunk) pairs fit the ranking (kMaxRankPairs, tile
  // counts below 2^14), each workgroup ranks them by their tile counts (from
  // kv_len, on the device) and takes the pair whose rank is its position:
  // the longest chunks start first (spread = 2).
  if (p.spread && (long long)B * (p.S / (kXcds / Hkv)) <= kMaxRankPairs && p.chunk < (1 << 14))
    p.spread = 2;
  return p;
}

// The work item (sequence b, KV head g, row block rb, chunk s) of launched
// workgroup `bid`; false for padding workgroups past the work.  constexpr,
// so the kernels and the host checks decode with this same function.  With
// spread = 2 the kernel then replaces the (b, s) pair by the pair of the
// same XCD lane whose length rank is this one's index: a permutation of the
// lane's pairs, so every work item is still covered once.
struct WorkItem {
  int b, g, rb, s;
};
constexpr bool work_item(int grid, int nwork, int S, int nRB, int spread, int B, int Hkv, int bid,
                         WorkItem& it) {
  const int x = bid % kXcds, j = bid / kXcds;
  if (spread) {
    const int L = kXcds / Hkv, per_b = S / L;
    it.g = x % Hkv;
    it.rb = j % nRB;
    const int uu = j / nRB;
    it.b = uu / per_b;
    it.s = ((x / Hkv - it.b) % L + L) % L + L * (uu % per_b);
    return it.b < B;
  }
  int w = x * (grid / kXcds) + j;
  if (w >= nwork) return false;
  it.s = w % S;
  w /= S;
  it.rb = w % nRB;
  w /= nRB;
  it.g = w % Hkv;
  it.b = w / Hkv;
  return it.b < B;
}

// The even split (slots > 0): the chunks of all sequences are numbered in the
// order of the sequences, `count` in all (found on the device, at most slots).
// Every (chunk, KV head) pair is one pair of an XCD, the pairs going to the
// XCDs in turn, and its row blocks follow each other there, since they read
// the same keys.  Fills g and rb and returns the chunk's number, or -1 for a
// workgroup past the work; even_grid holds all pairs of slots chunks.
constexpr int even_item(int bid, int count, int nRB, int Hkv, WorkItem& it) {
  const int j = bid / kXcds, q = j / nRB * kXcds + bid % kXcds;
  it.rb = j % nRB;
  it.g = q % Hkv;
  return q / Hkv < count ? q / Hkv : -1;
}

inline bool attn_plan_fits(const AttnPlan& p) {
  return p.NS > 0 && p.lds_bytes * p.wg_per_cu <= kMaxLds;
}

// Relative time of a plan, roughly in microseconds.  The constants are fitted
// together so that the plan picked is the fastest measured one: 1537 shapes (1267 of
// 1 to 32 sequences, 8 to 512 nodes and 256 to 32768 cached rows of the head shapes
// of the models above and D = 64, or as many training blocks; 155 of 1 to 64
// sequences, 1 to 64 nodes, 1 to 32 KV heads and up to 120000 rows; 115 of 65 to 400
// sequences), each in every arrangement, up to five split counts and both merges.
// The plans picked are 3.0% slower than the fastest on average.  They stand close to
// each other, so a rounding of these constants moves some of them: time all of them
// again before changing one.
//
// A chunk's tiles take their turns at one time per tile and key group: the latency
// of a tile's chain of LDS reads, matrix and vector work, or the CU's share of that
// work.  A split plan's chunk has all its row blocks on one XCD, so what does not fit
// the XCDs at once queues there.  On top come the fixed costs at a workgroup's two
// ends, HBM as the floor of the streaming (also at what the CUs at work can ask for),
// and the split's partials.  The lengths of several sequences are unknown here: they
// are taken as spread over the capacity, kMeanFill of it on average.
constexpr double kMeanFill = 0.6284;

// Tile time of one key group with all 8 waves of a CU at work, per arrangement
// (its latency alone: 1.214, with two ring stages 1.34).
constexpr double kTileFull[] = {1.888, 1.349, 1.402, 1.433, 1.0, 1.112, 1.34};
static_assert(sizeof(kTileFull) / sizeof(kTileFull[0]) == kNumArrangements, "one per arrangement");

// Bytes per microsecond one CU can ask HBM for.  2 sequences of 80754 rows, 4
// nodes, 8 KV heads, D = 64: 128 workgroups of 8 waves 95 us, 256 75.
constexpr double kCuBytes = 88.5e3;

inline double attn_plan_cost(AttnPlan& p, int B, int Hkv, int D, int Lmax, int N) {
  const double longest = cdiv(Lmax, kKeyTile) + cdiv(N, kKeyTile);
  const double mean = B == 1 ? longest : kMeanFill * cdiv(Lmax, kKeyTile) + cdiv(N, kKeyTile);
  double chunk = longest, items = B;
  if (p.slots > 0) {
    chunk = B == 1 ? (double)cdiv((long long)longest, p.slots) : B * mean / (p.slots - 0.3277 * B);
    if (chunk < p.min_chunk) chunk = p.min_chunk;
    if (chunk > longest) chunk = longest;
    items = B == 1 ? (double)cdiv((long long)longest, (long long)chunk) : B * mean / chunk + 0.5163 * B;
    if (items > p.slots) items = p.slots;
  }
  const double wgs = items * Hkv * p.nRB, room = 256.0 * p.wg_per_cu;
  double per_cu = wgs / 256.0;
  per_cu = per_cu < 1.0 ? 1.0 : (per_cu > p.wg_per_cu ? p.wg_per_cu : per_cu);
  const double row_tiles = (double)cdiv(p.M, kRowsPerWave) / p.nRB;
  const double waves = per_cu * p.WK * (row_tiles < p.WR ? row_tiles : p.WR);
  double tile = p.NS == 2 ? 1.34 : 1.214;
  if (kTileFull[p.arr] * waves / 8.0 > tile) tile = kTileFull[p.arr] * waves / 8.0;
  if (D == 64) tile *= 0.4675;
  double t = chunk / p.WK * tile;
  // workgroups of the fullest XCD over what it holds at once (unsplit plans
  // spread their row blocks over all XCDs)
  const long long per_xcd = (long long)cdiv((long long)(items * Hkv + 0.999), kXcds) * p.nRB;
  const long long rounds = p.slots > 0 ? cdiv(per_xcd, 32LL * p.wg_per_cu)
                                       : cdiv((long long)wgs, (long long)room);
  if (rounds > 1) {
    double load = B * mean * Hkv * p.nRB / room;  // tiles a place takes, on average
    const double fullest = per_xcd * chunk / (32.0 * p.wg_per_cu);
    if (p.slots > 0 && fullest > load) load = fullest;
    const double queue = load / p.WK * tile + 0.3287 * t;
    const double turns = rounds * t;
    t = t > queue ? t : (queue < turns ? queue : turns);
  }
  // unsplit, whole sequences to an XCD, and no order that evens them out: the XCD
  // with the longest sets the end (64 x 234 nodes, 2 KV heads, D = 64, up to 6296
  // rows: 140 us unsplit, 122 in 2)
  if (p.slots == 0 && B >= kXcds && p.spread != 2) t *= 1.029;
  const double asked = (wgs < 256 ? wgs : 256) * kCuBytes;
  const double hbm = B * mean * kKeyTile * Hkv * D * 4.0 / (asked < 11.8e6 ? asked : 11.8e6);
  t = t > hbm ? t : hbm;
  t += 7.788 + (p.WK > 1 ? 0.9328 : 0.0) + (p.slots > 0 ? 17.69 : 17.86) * (rounds - 1);
  if (chunk < longest) {
    const double chunks = (double)cdiv((long long)longest, (long long)(chunk + 0.999));
    // A row block's partial in bytes (whole 16-row fragments), and all of them.
    // In the fused merge a wave folds one row tile's columns, or whole row tiles:
    // waves without rows are idle, and few waves read at less than the CU's rate
    // (one wave alone 33 to 44 KB/us: 1 node over 24503 rows, 383 chunks of 3 tiles,
    // 108 us where 42 chunks take 23).  The second kernel has one wave per
    // fragment, and waits for memory once per 16 chunks (the second time hardly: 1 node
    // over 24503 rows, 3 heads, in 77 chunks 26.6 us, in 41 21.7).
    const int NTG = p.RB / 16, waves_wg = p.WR * p.WK;
    const int nt = cdiv(p.M < p.RB ? p.M : p.RB, 16);
    const int active = waves_wg >= NTG ? waves_wg / NTG * nt : (nt < waves_wg ? nt : waves_wg);
    const double block = nt * 16.0 * D * 4.0, all = wgs / p.nRB * cdiv(p.M, 16) * 16.0 * D * 4.0;
    const double waits = chunks > 32 ? 1.6 * (cdiv((long long)chunks, 16) - 2) : 0.0;
    auto fold = [&](double per_wave, double per_cu) {
      return chunks * block / (active * per_wave < per_cu ? active * per_wave : per_cu);
    };
    const double fused = 0.935 + fold(49.5e3, 204.5e3), second = 3.894 + waits + all / 3.552e6;
    t += (fused < second ? fused : second) + all / 4.899e6 + 0.1181;
    // more than 64 sequences: several per lane in the search for a work item
    if (B > 64) t += B > 256 ? 5.0 : 2.0;
    // The kind of merge: by the workgroup whose chunk arrives last (one CU reads
    // 61 to 78 KB/us of partials), or by a second kernel that spreads it over
    // the GPU and starts when the slowest chunk is done (9 us for 33.5 MB).
    p.fused = 1.034 + fold(16.09e3, 66.53e3) <= 5.939 + waits + all / 3.4e6;
  }
  return t;
}

// The fixed split: S chunks of every sequence's capacity, in the arrangement that
// a rough price picks.  Calls that bring less workspace than the plan below asks
// for run on it where it asks for less: they were accepted before there was an
// even split, whose plans cut shapes that this one leaves whole (16 x 33 nodes, 32
// heads on 8, 4160 rows: 38 MB against none).
//
// Price: matrix work on padded rows, K/V traffic from L2 (each row block re-reads
// the keys), HBM, the split partials written and read back, a penalty when the two
// waves of a SIMD belong to one workgroup (its per-tile barriers keep them in
// phase, so their matrix and vector work overlap poorly), and a fixed cost per
// round of workgroups.
inline AttnPlan attn_plan_fixed(int B, int N, int Hq, int Hkv, int D, int Lmax) {
  AttnPlan best{};
  double best_cost = 0;
  bool have = false;
  for (int k = 0; k < kNumArrangements; ++k) {
    AttnPlan p = attn_plan_arr(B, N, Hq, Hkv, D, Lmax, k, B, false);
    const long long base = (long long)B * Hkv * p.nRB, target = 256LL * p.wg_per_cu;
    const int tiles = cdiv(Lmax, kKeyTile) + cdiv(N, kKeyTile);
    const long long max_s = tiles / (2 * p.WK) > 1 ? tiles / (2 * p.WK) : 1;
    long long S = (target + base - 1) / base;
    if (S > max_s) S = max_s;
    if (B > 1 && base < target && S < 4 && max_s >= 4) S = 4;  // ragged batches
    if (S > 1) p = attn_plan_arr(B, N, Hq, Hkv, D, Lmax, k, S * B, false);
    if (!attn_plan_fits(p)) continue;
    // the last chunk of a row block merges all of them when that takes at most two
    // batches of loads per lane, else a second kernel does
    p.fused = p.S > 1 && (size_t)p.S * p.RB * D * 4 <= (size_t)1024 * p.threads;
    const double keys = (double)Lmax + N;
    double mfma = (double)B * Hkv * p.nRB * p.RB * keys * 4.0 * D / 2.0e15;
    if (p.wg_per_cu == 1 && p.WR > 1) mfma *= 1.3;
    const double kv = (double)B * Hkv * keys * D * 4.0;
    const double l2 = kv * p.nRB / 20.0e12, hbm = kv / 6.0e12;
    double t = mfma > l2 ? mfma : l2;
    t = t > hbm ? t : hbm;
    t += (double)p.ws_bytes * 2.0 / 5.0e12 + cdiv(p.nwork, target) * 4.0e-6;
    if (!have || t < best_cost) {
      best = p;
      best_cost = t;
      have = true;
    }
  }
  return best;
}

// The cheapest plan of at most `most` bytes of workspace.
inline AttnPlan attn_plan_search(int B, int N, int Hq, int Hkv, int D, int Lmax, size_t most) {
  AttnPlan best{};
  double best_cost = 0;
  bool have = false;
  for (int k = 0; k < kNumArrangements; ++k) {
    AttnPlan one = attn_plan_arr(B, N, Hq, Hkv, D, Lmax, k, B);
    if (!attn_plan_fits(one)) continue;
    // one chunk per sequence, or as many as fill the XCDs once, a quarter, half or
    // twice that: a chunk's row blocks stay on one XCD
    const long long pairs = 32LL * one.wg_per_cu / one.nRB;  // (chunk, KV head) pairs per XCD
    const long long fill = kXcds * pairs / Hkv;
    const long long cand[5] = {B, fill / 4, fill / 2, fill, 2 * fill};
    for (int c = 0; c < 5; ++c) {
      // more chunks than sequences; of more than 64 sequences half as many again (a few
      // more split next to none of them)
      if (c > 0 && (B > 64 ? 2 * cand[c] < 3LL * B : cand[c] <= B)) continue;
      // (of more than 64 sequences only those whose row blocks leave CUs empty, half
      // of them where the longest go first (spread): 100 nodes, 32 heads on 8, D =
      // 64, up to 7273 rows 153 us unsplit, 201 in 2)
      const long long places = one.spread == 2 ? 128LL : 256LL;
      if (c > 0 && B > 64 && (long long)B * Hkv * one.nRB >= places * one.wg_per_cu) continue;
      AttnPlan p = c == 0 ? one : attn_plan_arr(B, N, Hq, Hkv, D, Lmax, k, cand[c]);
      if (p.ws_bytes > most) continue;
      const double t = attn_plan_cost(p, B, Hkv, D, Lmax, N);
      if (!have || t < best_cost) {
        best = p;
        best_cost = t;
        have = true;
      }
    }
  }
  return best;
}

inline bool attn_even_tiles(int N, int Lmax) {
  return cdiv(Lmax, kKeyTile) + cdiv(N, kKeyTile) < kEvenTiles;
}

inline AttnPlan attn_plan(int B, int N, int Hq, int Hkv, int D, int Lmax) {
  // (the even split's quotients hold below 2^20 tiles)
  return attn_even_tiles(N, Lmax) ? attn_plan_search(B, N, Hq, Hkv, D, Lmax, SIZE_MAX)
                                  : attn_plan_fixed(B, N, Hq, Hkv, D, Lmax);
}

// The plan of a call whose workspace is too small for attn_plan's: the fixed
// split's, or the cheapest within `bytes`, a smaller split or none.  That one
// serves workspaces that hold a split at all, and every size where no workspace
// was ever asked for (more than 64 sequences, caches of 2^20 tiles and more).
// False: the workspace is refused.
inline bool attn_plan_within(int B, int N, int Hq, int Hkv, int D, int Lmax, size_t bytes, AttnPlan& p) {
  p = attn_plan_fixed(B, N, Hq, Hkv, D, Lmax);
  if (p.ws_bytes <= bytes) return true;
  if (bytes < kSyncBytes && B <= 64 && attn_even_tiles(N, Lmax)) return false;
  p = attn_plan_search(B, N, Hq, Hkv, D, Lmax, bytes);
  return true;
}

// Training-mask calls with several blocks to a workgroup (tv_attention.hip,
// attn_packed): blocks of at most 64 rows (of more, a workgroup of 128 rows
// holds one), few enough for the sort, and enough of them that one block per
// workgroup would take well more than two rounds of the chip's 512 places; below
// that the packs are too few and their long tile chains cost more than they save.
// With n = examples x blocks x KV heads that is from 1280 on, for blocks of less
// than 16 rows (16 to a pack: the fewest packs) from 1800, and half a group more
// for every block of an example past 256, since the sort compares each with all.
// Measured on 260 shapes, one block each against packed: M = 16 rows, n = 1584,
// 186 positions 28.9 against 25.1 us, 2016, 1344 positions 95.5 against 54.1; M =
// 32, 1408, 245 positions 30.4 against 24.6; M = 64, 2048, 256 positions 40.4
// against 27.4; M = 8, 1677, 424 positions 33.5 against 41.8 (not packed), 2208,
// 247 positions 50.7 against 34.9; 1584 blocks of 16 rows of one head 25.5 against
// 33.6 (not packed).  The order of the blocks lies behind the sync words of the
// workspace.
constexpr int kPackRows = 128;
constexpr int kPackMaxBlocks = 2048;  // blocks per example the sort takes
constexpr int kPackMinGroups = 1280, kPackMinSmall = 1800;  // n, for M >= 16 and below
constexpr int kPackRank = 64;         // blocks a workgroup of the sort ranks
struct PackPlan {
  int nb, packs;  // blocks per workgroup (0: not packed), workgroups per (example, KV head)
  size_t ws_bytes;
};
inline PackPlan pack_plan(int B, int A, int S, int Hq, int Hkv) {
  PackPlan p{};
  const long long M = (long long)S * (Hq / Hkv);
  if (2 * M > kPackRows || A > kPackMaxBlocks) return p;
  const int nb = (int)(kPackRows / M) < 16 ? (int)(kPackRows / M) : 16;
  const int packs = cdiv(A, nb);
  const long long least = (M >= 16 ? kPackMinGroups : kPackMinSmall) + (A > 256 ? (A - 256) / 2 : 0);
  if (A < nb || (long long)B * A * Hkv < least) return p;
  p.nb = nb;
  p.packs = packs;
  p.ws_bytes = kSyncBytes + (size_t)B * A * 4;
  return p;
}

// Acceptance decomposition: a scan kernel runs one workgroup per (node row,
// vocabulary split) and stores one 64-bit key per pair; a second kernel runs
// one workgroup per sequence.  Splits give the scan >= ~2048 workgroups but
// each thread gets at least one full round of kAcceptScanLoads loads.
constexpr int kAcceptMaxSplit = 16;
constexpr int kScanThreads = 256;
constexpr int kScanLoadsPerThread = 8;   // 16-byte loads a thread keeps in flight
// The greedy acceptance scan moves the same bytes per round with twice the
// waves, each keeping half the loads in flight: measured 1-4% faster than
// 256 x 8, while 128 x 16 and 64 x 32 were 5-20% slower.
constexpr int kAcceptScanThreads = 512;
constexpr int kAcceptScanLoads = 4;
static_assert(kAcceptScanThreads * kAcceptScanLoads == kScanThreads * kScanLoadsPerThread,
              "same bytes per round as the other scans");
// The non-greedy acceptance's log-sum-exp scan takes the same shape: 512 x 4
// was 1.6 us faster than 256 x 8 per call at 512 rows of 151936 bf16 logits
// (together with the split rule of sample_plan), the same at 64 rows.
constexpr int kLseScanThreads = 512;
constexpr int kLseScanLoads = 4;
static_assert(kLseScanThreads * kLseScanLoads == kScanThreads * kScanLoadsPerThread,
              "same bytes per round as the other scans");

inline long long accept_split_cap(long long rows) {
  long long ns = (2048 + rows - 1) / rows;
  return ns < 1 ? 1 : (ns > kAcceptMaxSplit ? kAcceptMaxSplit : ns);
}

struct AcceptPlan {
  int nsplit;
  long long chunks_per_split;   // vector chunks (or scalars) per split
  int grid;
  size_t ws_bytes;
};

// Share of a workgroup's load slots that carry data when a row of `chunks`
// vector chunks is cut into ns splits (whole rounds of per_round chunks per
// workgroup; the last round is partly empty).
inline double accept_round_fill(long long chunks, long long ns, long long per_round) {
  const long long c = (chunks + ns - 1) / ns;
  const long long rounds = (c + per_round - 1) / per_round;
  return (double)c / (double)(rounds * per_round);
}

inline AcceptPlan accept_plan(int B, int N, int V, int esize, int vec_elems) {
  AcceptPlan p{};
  const long long rows = (long long)B * N;
  const long long chunks = (V + vec_elems - 1) / vec_elems;
  // at least one full round of loads per thread in every split
  long long ns = accept_split_cap(rows);
  const long long per_round = (long long)kAcceptScanThreads * kAcceptScanLoads;
  const long long by_size = (chunks + per_round - 1) / per_round;
  if (ns > by_size) ns = by_size;
  if (ns < 1) ns = 1;
  // Down to half as many splits, the count whose load slots are best used
  // (ties: more splits): a partly filled last round costs a whole round of
  // latency.  512 rows of 151936 bf16 logits in 4 splits take 2.3 rounds per
  // thread (77% of the slots used), in 2 splits 4.6 (93%), and the
  // acceptance ran 32.6 us in 4 against 31.7 us in 2; 128 rows stay at 10
  // splits (0.93 of one round), where 8 splits (1.16 rounds, 58%) were 5%
  // slower.
  {
    long long best = ns;
    double best_fill = accept_round_fill(chunks, ns, per_round);
    for (long long k = ns - 1; k >= 1 && 2 * k >= ns; --k) {
      const double f = accept_round_fill(chunks, k, per_round);
      if (f > best_fill + 1e-9) {
        best = k;
        best_fill = f;
      }
    }
    ns = best;
  }
  p.chunks_per_split = (chunks + ns - 1) / ns;
  p.nsplit = (int)((chunks + p.chunks_per_split - 1) / p.chunks_per_split);
  p.grid = (int)(rows * p.nsplit);
  p.ws_bytes = (size_t)rows * p.nsplit * 8;
  (void)esize;
  return p;
}

// Workspace bound valid for every dtype and alignment.
inline size_t accept_ws_bytes(int B, int N) {
  const long long rows = (long long)B * N;
  return (size_t)(rows * accept_split_cap(rows) * 8);
}

// Draft top-W (tree drafting's candidates): one workgroup per (draft-depth
// row, vocabulary split) reduces its slice to a running log-sum-exp state
// and its W best (value, token) pairs; a second kernel merges the splits of
// each row.  A slice is one round of loads wherever 16 splits allow it (the
// scan of more rounds keeps lists and runs several times longer), and where
// that leaves the GPU short of workgroups, up to 16 splits of fewer loads per
// thread.  Calls may bring less workspace than that takes, down to the acceptance
// scan's split cap (topw_min_bytes); they get as many splits as it holds.
constexpr int kTopwMax = 16;             // largest branching width W
constexpr int kMaxDraftDepth = 64;       // == TV_MAX_DRAFT_DEPTH
constexpr size_t kTopwPartBytes = 8 + 8 * kTopwMax;
constexpr int kTopwRound = 64;           // logits a thread reads in one round, at most

struct TopwPlan {
  int nsplit;
  long long chunks_per_split;
  int grid;
  size_t ws_bytes;
};

inline TopwPlan topw_plan(int B, int Nd, int V, int vec_elems,
                          long long most_splits = kAcceptMaxSplit) {
  TopwPlan p{};
  const long long rows = (long long)B * Nd;
  const long long chunks = (V + vec_elems - 1) / vec_elems;
  const long long per_round = (long long)kScanThreads * kTopwRound / vec_elems;
  long long ns = (chunks + per_round - 1) / per_round;
  const long long fill = (512 + rows - 1) / rows, whole = chunks / kScanThreads;  // >= 1 load each
  if (ns < fill) ns = fill < whole ? fill : whole;
  if (most_splits > kAcceptMaxSplit) most_splits = kAcceptMaxSplit;
  if (ns > most_splits) ns = most_splits;
  if (ns < 1) ns = 1;
  p.chunks_per_split = (chunks + ns - 1) / ns;
  p.nsplit = (int)((chunks + p.chunks_per_split - 1) / p.chunks_per_split);
  p.grid = (int)(rows * p.nsplit);
  p.ws_bytes = (size_t)rows * p.nsplit * kTopwPartBytes;
  return p;
}

// The least workspace a call is accepted with, and what the plan of either dtype
// asks for.
inline size_t topw_min_bytes(int B, int Nd) {
  const long long rows = (long long)B * Nd;
  return (size_t)(rows * accept_split_cap(rows)) * kTopwPartBytes;
}
inline size_t topw_ws_bytes(int B, int Nd, int V) {
  const size_t f32 = topw_plan(B, Nd, V, 4).ws_bytes, bf16 = topw_plan(B, Nd, V, 8).ws_bytes;
  const size_t most = f32 > bf16 ? f32 : bf16, least = topw_min_bytes(B, Nd);
  return most > least ? most : least;
}

// Non-greedy acceptance: an lse scan over the B*N target rows (splits as
// in the acceptance scan, in vocabulary entries that are multiples of 8),
// then one workgroup per (sequence, race split) that repeats the tests and
// races its vocabulary slice (about 512 workgroups in all, at least 8
// entries per thread, at most kRaceSlice entries so that the slice's token
// mask fits in LDS).
constexpr int kMaxRaceSplit = 64;
constexpr long long kRaceSlice = 131072;
constexpr long long kMaxSampledVocab = kRaceSlice * kMaxRaceSplit;

struct SamplePlan {
  int nsplit, nrace, lse_grid;
  long long eps, rps;  // vocabulary entries per lse / race split
  size_t race_bytes, ws_bytes;
};

inline SamplePlan sample_plan(int B, int N, int V) {
  SamplePlan p{};
  const long long rows = (long long)B * N;
  long long ns = accept_split_cap(rows);
  const long long per_round = (long long)kScanThreads * kScanLoadsPerThread * 8;
  const long long by_size = ((long long)V + per_round - 1) / per_round;
  if (ns > by_size) ns = by_size;
  if (ns < 1) ns = 1;
  {
    // the split count that uses the largest share of its load slots, down
    // to half the workgroup target (as in accept_plan)
    long long best = ns;
    double best_fill = accept_round_fill(V, ns, per_round);
    for (long long k = ns - 1; k >= 1 && 2 * k >= ns; --k) {
      const double f = accept_round_fill(V, k, per_round);
      if (f > best_fill + 1e-9) {
        best = k;
        best_fill = f;
      }
    }
    ns = best;
  }
  p.eps = ((V + ns - 1) / ns + 7) / 8 * 8;
  p.nsplit = (int)((V + p.eps - 1) / p.eps);
  p.lse_grid = (int)(rows * p.nsplit);
  long long nr = (512 + B - 1) / B;
  const long long by_v = ((long long)V + 8 * 256 - 1) / (8 * 256);
  if (nr > by_v) nr = by_v;
  const long long by_mask = ((long long)V + kRaceSlice - 1) / kRaceSlice;
  if (nr < by_mask) nr = by_mask;
  if (nr > kMaxRaceSplit) nr = kMaxRaceSplit;
  if (nr < 1) nr = 1;
  p.rps = ((V + nr - 1) / nr + 7) / 8 * 8;
  p.nrace = (int)((V + p.rps - 1) / p.rps);
  p.race_bytes = ((size_t)B * p.nrace * 16 + 255) / 256 * 256;
  p.ws_bytes = p.race_bytes + (size_t)rows * p.nsplit * 8;
  return p;
}

// LDS of the acceptance of one sequence of N nodes: per node the
// pointer-jumping state (two packed 32-bit words, double-buffered), the
// target argmax (int) and the parent (short).
constexpr size_t accept_lds_bytes(int N) { return (size_t)N * 14 + 16; }

}  // namespace tv
