// Host-side check of the launch plans (tv_plan.h is plain C++): for each
// shape on stdin ("B N Hq Hkv D Lmax V"), the plan a call gets, the fixed split's
// plan and those that calls with less workspace fall back to.  Every launched
// workgroup is enumerated exactly as the kernels decode it: the decoded work
// items are in range and cover every (b, g, rb, chunk) once, for the even split
// with the chunks that a host copy of the kernels' search finds for ragged,
// empty and full kv_lens; the workspace holds the largest index any workgroup
// writes, and the dynamic LDS fits the 160 KB of a CDNA4 CU.  Prints "OK ..." or
// "FAIL ...".
#include <algorithm>
#include <cstdio>
#include <vector>
#include "tv_plan.h"

using tv::AttnPlan;
using tv::cdiv;

static int B, N, Hq, Hkv, D, Lmax, V;

// what both kinds of plan keep
static bool check_common(const AttnPlan& p) {
  const int tiles = cdiv(Lmax, tv::kKeyTile) + cdiv(N, tv::kKeyTile);
  bool ok = p.grid % tv::kXcds == 0 && p.nwork == B * Hkv * p.nRB * p.S && p.grid >= p.nwork;
  ok = ok && (long long)p.S * p.chunk >= tiles && (long long)(p.S - 1) * p.chunk < tiles;
  ok = ok && p.WR >= 1 && p.RB == tv::kRowsPerWave * p.WR && tv::attn_plan_fits(p);
  ok = ok && p.lds_bytes <= 160 * 1024 && (p.fused == 0 || p.S > 1);
  // shared queries: several key groups of several waves, a grid that
  // fills every CU, and the queries' LDS counted in the kernel's
  if (p.qshare) ok = ok && p.WK >= 2 && p.WR >= 2 && p.nwork >= 256LL * p.wg_per_cu;
  ok = ok && p.lds_bytes == tv::attn_lds_bytes(D, p.WR, p.WK, p.NS, p.G, N, p.qshare != 0);
  if (p.S > 1) {
    // arrival counter + tree flag per row block; the workspace sections add up
    ok = ok && (size_t)B * Hkv * p.nRB <= (size_t)tv::kSyncGroups && p.ws_sync_bytes == tv::kSyncBytes;
    ok = ok && p.ws_bytes == p.ws_o_bytes + p.ws_ml_bytes + p.ws_sync_bytes;
  } else {
    ok = ok && p.ws_bytes == 0 && p.slots == 0;
  }
  return ok;
}

// the last element of chunk partial `part` lies in the workspace
static bool partial_fits(const AttnPlan& p, size_t part) {
  const int DT = D / 16, NT = p.RB / 16;
  const size_t last_o = ((part + 1) * DT * NT - 1) * 64 + 63, last_ml = part * p.RB + p.RB - 1;
  return (last_o + 1) * 16 <= p.ws_o_bytes && (last_ml + 1) * 8 <= p.ws_ml_bytes;
}

// key tiles of a sequence of kvl rows up to a row block's last node, and of its cache
static int seq_tiles(int kvl, int i_hi) { return cdiv(kvl, tv::kKeyTile) + i_hi / tv::kKeyTile + 1; }
static int last_node(const AttnPlan& p, int rb) {
  const int rows = std::min(p.RB, p.M - rb * p.RB);
  return (rb * p.RB + rows - 1) / p.G;
}

// the first ceil(T / chunk) chunks of a row block hold its tiles, every tile once,
// and one of them holds tree tiles
static bool check_chunks(const AttnPlan& p, int kvl, int chunk, int most) {
  const int nct = cdiv(kvl, tv::kKeyTile);
  for (int rb = 0; rb < p.nRB; ++rb) {
    const int T = seq_tiles(kvl, last_node(p, rb)), nval = cdiv(T, chunk);
    if (nval < 1 || nval > most) return false;
    int covered = 0, tree = 0;
    for (int s = 0; s < nval; ++s) {
      const int t0 = s * chunk, t1 = std::min(T, t0 + chunk);
      if (t0 >= t1) return false;
      covered += t1 - t0;
      tree += t1 > nct;
    }
    if (covered != T || tree < 1) return false;
  }
  return true;
}

// plans with one chunk size for the capacity (no split, or the fixed split)
static bool check_fixed(const AttnPlan& p) {
  bool ok = check_common(p) && p.slots == 0;
  // the spread order needs every workgroup to carry a work item
  if (p.spread && (p.grid != p.nwork || tv::kXcds % Hkv != 0 || p.S % (tv::kXcds / Hkv) != 0))
    ok = false;
  std::vector<int> seen((size_t)p.nwork, 0);
  int decoded = 0;
  for (int bid = 0; bid < p.grid && ok; ++bid) {
    tv::WorkItem it{};
    if (!tv::work_item(p.grid, p.nwork, p.S, p.nRB, p.spread, B, Hkv, bid, it)) continue;
    ++decoded;
    if (it.b < 0 || it.b >= B || it.g < 0 || it.g >= Hkv || it.rb < 0 || it.rb >= p.nRB ||
        it.s < 0 || it.s >= p.S || it.rb * p.RB >= p.M)
      return false;
    const size_t part = ((size_t)(it.b * Hkv + it.g) * p.nRB + it.rb) * p.S + it.s;
    seen[part]++;
    if (p.S > 1) ok = partial_fits(p, part);
  }
  for (int v : seen) ok = ok && v == 1;
  ok = ok && decoded == p.nwork;
  for (int kvl : {0, 1, Lmax / 2, Lmax})
    if (kvl <= Lmax) ok = ok && check_chunks(p, kvl, p.chunk, p.S);
  return ok;
}

// plans with an even split: chunks of one size, found from the kv_lens
static bool check_even(const AttnPlan& p) {
  if (!check_common(p) || p.S < 2 || p.slots <= B - (B == 1) || p.slots > B * p.S || p.spread ||
      p.min_chunk != 2 * p.WK || B > tv::kEvenSequences)
    return false;
  const int grid = tv::kXcds * p.nRB * cdiv((long long)p.slots * Hkv, tv::kXcds);
  if (p.even_grid != grid) return false;
  for (int kind = 0; kind < 6; ++kind) {
    std::vector<int> kvl(B), t(B);
    for (int b = 0; b < B; ++b) {
      const long long h = (long long)b * 977 + 31;
      kvl[b] = kind == 0 ? 0 : kind == 1 ? Lmax : kind == 2 ? (b ? 0 : Lmax)
               : kind == 3 ? (b == B - 1 ? Lmax : std::min(Lmax, 33))
               : kind == 4 ? (int)(h % (Lmax + 1LL)) : std::min(Lmax, 5);
      t[b] = seq_tiles(kvl[b], N - 1);
    }
    // the smallest chunk of which the sequences need at most slots together
    auto count = [&](int c) {
      long long n = 0;
      for (int x : t) n += cdiv(x, c);
      return n;
    };
    int chunk = p.min_chunk, hi = std::max(p.min_chunk, *std::max_element(t.begin(), t.end()));
    if (count(hi) > p.slots) return false;
    while (chunk < hi) {
      const int mid = chunk + (hi - chunk) / 2;
      if (count(mid) <= p.slots) hi = mid;
      else chunk = mid + 1;
    }
    const int chunks = (int)count(chunk);
    std::vector<int> first(B), seen((size_t)chunks * p.nRB * Hkv, 0);
    for (int b = 0, n = 0; b < B; ++b) {
      first[b] = n;
      n += cdiv(t[b], chunk);
      if (!check_chunks(p, kvl[b], chunk, cdiv(t[b], chunk))) return false;
    }
    for (int bid = 0; bid < p.even_grid; ++bid) {
      tv::WorkItem it{};
      const int item = tv::even_item(bid, p.slots, p.nRB, Hkv, it);
      if (item < 0 || item >= chunks) continue;
      if (it.g < 0 || it.g >= Hkv || it.rb < 0 || it.rb >= p.nRB) return false;
      seen[((size_t)item * Hkv + it.g) * p.nRB + it.rb]++;
      const int b = (int)(std::upper_bound(first.begin(), first.end(), item) - first.begin()) - 1;
      const int part0 = (it.g * p.nRB + it.rb) * p.slots + first[b];
      if (!partial_fits(p, (size_t)part0 + (item - first[b]))) return false;
    }
    for (int v : seen)
      if (v != 1) return false;
  }
  return true;
}

static bool check_plan(const AttnPlan& p) { return p.slots > 0 ? check_even(p) : check_fixed(p); }

// Calls with less workspace than the plan asks for: what is refused, and that the
// plans of the others stay within it.
static bool check_within(const AttnPlan& p, const AttnPlan& fixed) {
  const bool always = B > 64 || cdiv(Lmax, tv::kKeyTile) + cdiv(N, tv::kKeyTile) >= (1 << 20);
  for (size_t limit : {p.ws_bytes, fixed.ws_bytes, p.ws_bytes / 2, tv::kSyncBytes + 1, tv::kSyncBytes, (size_t)1}) {
    const size_t bytes = limit > 0 ? limit - 1 : 0;
    if (bytes >= p.ws_bytes) continue;
    AttnPlan q{};
    const bool ok = tv::attn_plan_within(B, N, Hq, Hkv, D, Lmax, bytes, q);
    if (ok != (fixed.ws_bytes <= bytes || bytes >= tv::kSyncBytes || always)) return false;
    if (ok && (q.ws_bytes > bytes || !check_plan(q))) return false;
  }
  return true;
}

static bool check_vocab() {
  bool ok = true;
  for (int esize : {2, 4}) {
    const int vec = 16 / esize;
    const tv::AcceptPlan ap = tv::accept_plan(B, N, V, esize, vec);
    const long long nch = ((long long)V + vec - 1) / vec;
    if (ap.ws_bytes > tv::accept_ws_bytes(B, N)) ok = false;
    if (ap.grid != (long long)B * N * ap.nsplit) ok = false;
    if ((long long)ap.nsplit * ap.chunks_per_split < nch) ok = false;
    if ((long long)(ap.nsplit - 1) * ap.chunks_per_split >= nch) ok = false;
    if (ap.nsplit < 1 || ap.nsplit > tv::kAcceptMaxSplit) ok = false;
    if (ap.ws_bytes != (size_t)B * N * ap.nsplit * 8) ok = false;
    if (tv::accept_lds_bytes(N) + (size_t)N * 8 > 64 * 1024) ok = false;
    // draft top-W over Nd = min(N, 64) depth rows, with the queried workspace
    // and the least: every chunk in one split, the workspace within its bound
    const int Nd = N < 64 ? N : 64;
    for (size_t bytes : {tv::topw_ws_bytes(B, Nd, V), tv::topw_min_bytes(B, Nd)}) {
      const tv::TopwPlan tp =
          tv::topw_plan(B, Nd, V, vec, (long long)(bytes / ((size_t)B * Nd * tv::kTopwPartBytes)));
      if (tp.grid != (long long)B * Nd * tp.nsplit) ok = false;
      if ((long long)tp.nsplit * tp.chunks_per_split < nch) ok = false;
      if ((long long)(tp.nsplit - 1) * tp.chunks_per_split >= nch) ok = false;
      if (tp.nsplit < 1 || tp.nsplit > tv::kAcceptMaxSplit) ok = false;
      if (tp.ws_bytes > bytes) ok = false;
    }
  }
  return ok;
}

int main() {
  int bad = 0, cases = 0;
  while (std::scanf("%d %d %d %d %d %d %d", &B, &N, &Hq, &Hkv, &D, &Lmax, &V) == 7) {
    ++cases;
    const AttnPlan p = tv::attn_plan(B, N, Hq, Hkv, D, Lmax);
    const AttnPlan fixed = tv::attn_plan_fixed(B, N, Hq, Hkv, D, Lmax);
    const bool ok = check_plan(p) && check_fixed(fixed) && check_within(p, fixed) && check_vocab();
    std::printf("%s B=%d N=%d Hq=%d Hkv=%d D=%d L=%d V=%d S=%d slots=%d fused=%d RB=%d nRB=%d grid=%d spread=%d lds=%zu ws=%zu\n",
                ok ? "OK" : "FAIL", B, N, Hq, Hkv, D, Lmax, V, p.S, p.slots, p.fused, p.RB, p.nRB,
                p.grid, p.spread, p.lds_bytes, p.ws_bytes);
    bad += !ok;
  }
  std::printf("%d cases, %d failed\n", cases, bad);
  return bad ? 1 : 0;
}
