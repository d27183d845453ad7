// Internal declarations shared by the library's translation units (not part of the C ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hstu {

// One unit of scheduled work: a tile of "owner" rows (query rows for the forward and dq
// passes, key rows for the dk/dv pass) plus up to two segments of "streamed" rows of the
// same sequence that the tile is computed against.  Rows index the caller's buffers;
// positions are in-sequence positions and drive the causal mask, so the same kernels serve
// whole-batch attention (one segment, row == offset + position) and a context-parallel
// rank's share (two mini-chunks per side, section 2.3 of the paper).
struct Item {
  int32_t row0;         // first owner row of the tile
  int32_t nrows;        // valid owner rows (0..tile)
  int32_t pos0;         // in-sequence position of row0
  int32_t nseg;         // streamed segments in use (0..2)
  int32_t seg_row0[2];  // first streamed row of each segment
  int32_t seg_len[2];   // rows in each segment
  int32_t seg_pos0[2];  // in-sequence position of each segment's first row
  int32_t seg_tcol0[2]; // column of each segment's first row in the transposed streamed copies
  int32_t cost;         // visible 32-row streamed blocks (the sort key)
  int32_t part;         // 0: the item writes its output rows; p > 0: it covers only a part of the
                        // streamed rows and writes an fp32 partial result into slot p - 1
  int32_t before;       // natural order of whole batches, key side: work of all items before this one
  int32_t pad;
};
static_assert(sizeof(Item) == 64, "Item is one 64-byte record");

// Blocks of `streamed` visible rows that the walking dk/dv kernel works through for an item: three at least.
constexpr int WALK_BLOCKS_MIN = 3;
// What an item costs besides, in blocks: its rows' loads, stores and masked blocks.  Backward of 1536 sequences of lognormal
// length (median 256), sorted by length, with 0, 1, 2 and 4: 5475, 4916, 4635 and 4552 us; 512 of median 300, not sorted:
// 1018, 1014, 992 and 1024 (H = 8 and 4, d = 128).
constexpr int WALK_ITEM_BLOCKS = 3;
__host__ __device__ inline int walk_blocks(int streamed) {
  const int n = streamed / 32 + (streamed % 32 ? 1 : 0);
  return n > WALK_BLOCKS_MIN ? n : WALK_BLOCKS_MIN;
}

// Device view of a built schedule.
struct Plan {
  const int32_t* header;  // [0] = number of items, [1] = number of 64-row streamed tiles,
                          // [2] = number of owner tiles whose partial results have to be summed,
                          // [3] = work of all items (where Item::before is filled in)
  const int32_t* red;     // per such tile: first owner row, rows, first partial slot, slots
  const int32_t* order;   // order[slot] = item index, non-increasing cost
  const Item* items;
  const int32_t* ttile;   // per 64-row streamed tile: first row, valid rows
  int32_t max_stiles;     // host bound on the streamed tiles; transposed copies have 64x this many columns
  int32_t direct;         // the items are in schedule order, every slot of the grid holds one (or one
                          // without rows): no count and no order to look up
};

// Byte offsets of one schedule's arrays inside the workspace.
struct PlanLayout {
  size_t header, owner_base, streamed_base, tile_base, stile_base, ttile, order, items, red, end;
};

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// max_items bounds the items the kernels see (parts included), max_tiles the owner tiles.
inline PlanLayout plan_layout(size_t base, int64_t batch, int64_t max_items, int64_t max_stiles,
                              int64_t max_tiles = 0) {
  PlanLayout l;
  size_t p = align_up(base, 256);
  l.header = p;        p += 64;
  l.owner_base = p;    p = align_up(p + (size_t)(batch + 1) * 4, 64);
  l.streamed_base = p; p = align_up(p + (size_t)(batch + 1) * 4, 64);
  l.tile_base = p;     p = align_up(p + (size_t)(batch + 1) * 4, 64);
  l.stile_base = p;    p = align_up(p + (size_t)(batch + 1) * 4, 64);
  l.ttile = p;         p = align_up(p + (size_t)max_stiles * 8, 64);
  l.order = p;         p = align_up(p + (size_t)max_items * 4, 64);
  l.items = p;         p = align_up(p + (size_t)max_items * sizeof(Item), 64);
  l.red = p;           p = align_up(p + (size_t)max_tiles * 16, 64);
  l.end = p;
  return l;
}

// Upper bound on the number of items when `rows` owner rows of `batch` sequences, each cut
// into at most `segs` segments, are tiled by `tile` rows.
inline int64_t max_items_bound(int64_t rows, int64_t batch, int segs, int tile) {
  return rows / tile + (int64_t)segs * batch + 1;
}

// The (up to two) segments one side of one sequence consists of.
struct Side {
  int nseg;
  int len[2];
  int pos[2];
  int rows;  // len[0] + len[1]
};

__device__ __forceinline__ Side make_side(int L, int cp, int rank) {
  Side s;
  if (rank < 0) {
    s.nseg = 1; s.len[0] = L; s.pos[0] = 0; s.len[1] = 0; s.pos[1] = 0;
  } else {
    // mini-chunk m covers positions [m*c, min((m+1)*c, L)), c = ceil(L / (2*cp))
    const uint32_t n = 2u * (uint32_t)cp;
    const long long c = (long long)((uint32_t)L / n + ((uint32_t)L % n ? 1u : 0u));
    const int m0 = rank, m1 = 2 * cp - 1 - rank;
    long long b0 = m0 * c, e0 = (m0 + 1) * c, b1 = m1 * c, e1 = (m1 + 1) * c;
    b0 = b0 < L ? b0 : L; e0 = e0 < L ? e0 : L; b1 = b1 < L ? b1 : L; e1 = e1 < L ? e1 : L;
    s.nseg = 2;
    s.len[0] = (int)(e0 - b0); s.pos[0] = (int)b0;
    s.len[1] = (int)(e1 - b1); s.pos[1] = (int)b1;
    if (s.len[1] > 0 && s.pos[1] == s.pos[0] + s.len[0]) {  // adjacent chunks: one segment
      s.len[0] += s.len[1]; s.len[1] = 0; s.nseg = 1;
    }
    if (s.len[1] == 0) s.nseg = 1;
  }
  s.rows = s.len[0] + s.len[1];
  return s;
}

__device__ __forceinline__ int clampi(long long x, int lo, int hi) {
  return x < lo ? lo : (x > hi ? hi : (int)x);
}

// Sanitised [start, end) of sequence b in the global layout: whatever the device array
// holds, 0 <= start <= end <= total_rows.
__device__ __forceinline__ void seq_range(const int32_t* off, int b, int total_rows, int& s, int& e) {
  s = clampi(off[b], 0, total_rows);
  e = clampi(off[b + 1], s, total_rows);
}

constexpr int STILE = 64;  // rows per tile of the streamed side (what the kernels stage in LDS)
__device__ __forceinline__ int blocks_of(int rows) { return (rows >> 5) + ((rows & 31) != 0); }  // of 32 rows

__device__ inline int tiles_of(const Side& s, int tile) {
  return (s.len[0] + tile - 1) / tile + (s.len[1] + tile - 1) / tile;
}

// The schedule item of owner tile t of segment u (0, 1) of one sequence: its rows, and the visible
// streamed segments, compacted to the front.  owner_base / streamed_base: first row of the sequence
// in the two sides' layouts; tcol0: first column in the transposed copy of the streamed side; pvis:
// visible rows of the (compacted) segments.
__device__ __forceinline__ Item describe_item(const Side& so, const Side& ss, int u, int t, int owner_base,
                                              int streamed_base, int tcol0, int tile, int causal, int side,
                                              int owner_rows, int streamed_rows, int (&pvis)[2]) {
  Item it;
  it.row0 = owner_base + (u ? so.len[0] : 0) + t * tile;
  it.nrows = (u ? so.len[1] : so.len[0]) - t * tile;
  if (it.nrows > tile) it.nrows = tile;
  it.pos0 = (u ? so.pos[1] : so.pos[0]) + t * tile;
  // never beyond the rows the caller declared for its buffers
  it.nrows = clampi((long long)owner_rows - it.row0, 0, it.nrows);
  // The visible streamed segments, compacted to the front.  Written without run-time array
  // indices so that the item stays in registers (indexed, it would live in scratch memory).
  int vrow[2] = {0, 0}, vlen[2] = {0, 0}, vpos[2] = {0, 0}, vcol[2] = {0, 0}, vcost[2] = {0, 0};
  int vvis[2] = {0, 0};
  bool von[2] = {false, false};
  int srow = streamed_base;
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    if (g < ss.nseg) {
      const int len = clampi((long long)streamed_rows - srow, 0, ss.len[g]);
      int vis;  // streamed rows that at least one owner row sees
      if (!causal) {
        vis = len;
      } else if (side == 0) {  // keys at positions <= last query position
        vis = clampi((long long)it.pos0 + it.nrows - ss.pos[g], 0, len);
      } else {                   // queries at positions >= first key position
        vis = len - clampi((long long)it.pos0 - ss.pos[g], 0, len);
      }
      von[g] = it.nrows > 0 && vis > 0;
      vrow[g] = srow; vlen[g] = len; vpos[g] = ss.pos[g];
      vcol[g] = tcol0 + (g ? (ss.len[0] + 63) / 64 * 64 : 0);
      vcost[g] = (vis + 31) >> 5;
      vvis[g] = vis;
      srow += ss.len[g];
    }
  }
  const bool first1 = !von[0] && von[1];  // only the second segment is visible: it moves to slot 0
  it.nseg = (von[0] ? 1 : 0) + (von[1] ? 1 : 0);
  it.cost = (von[0] ? vcost[0] : 0) + (von[1] ? vcost[1] : 0);
  it.seg_row0[0] = von[0] ? vrow[0] : (first1 ? vrow[1] : 0);
  it.seg_len[0] = von[0] ? vlen[0] : (first1 ? vlen[1] : 0);
  it.seg_pos0[0] = von[0] ? vpos[0] : (first1 ? vpos[1] : 0);
  it.seg_tcol0[0] = von[0] ? vcol[0] : (first1 ? vcol[1] : 0);
  const bool second = von[0] && von[1];
  it.seg_row0[1] = second ? vrow[1] : 0;
  it.seg_len[1] = second ? vlen[1] : 0;
  it.seg_pos0[1] = second ? vpos[1] : 0;
  it.seg_tcol0[1] = second ? vcol[1] : 0;
  it.part = 0;
  it.before = it.pad = 0;
  pvis[0] = von[0] ? vvis[0] : (first1 ? vvis[1] : 0);
  pvis[1] = second ? vvis[1] : 0;
  return it;
}

// Inclusive prefix sums over the wave's lanes on the vector pipe (no LDS round trips); lane 63 ends
// with the total.
__device__ __forceinline__ int wave_scan(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr:1, 2, 4, 8
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15, :31
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);
  return x;
}
__device__ __forceinline__ int wave_total(int x) { return __builtin_amdgcn_readlane(wave_scan(x), 63); }

// Minimum and maximum over the wave's lanes, on the vector pipe (a shuffle goes through LDS: six
// dependent round trips per reduction, and a packed item needs four of them).
template <class F>
__device__ __forceinline__ int wave_reduce(int x, const F& f) {
  x = f(x, __builtin_amdgcn_update_dpp(x, x, 0x111, 0xf, 0xf, false));  // row_shr:1, 2, 4, 8
  x = f(x, __builtin_amdgcn_update_dpp(x, x, 0x112, 0xf, 0xf, false));
  x = f(x, __builtin_amdgcn_update_dpp(x, x, 0x114, 0xf, 0xf, false));
  x = f(x, __builtin_amdgcn_update_dpp(x, x, 0x118, 0xf, 0xf, false));
  x = f(x, __builtin_amdgcn_update_dpp(x, x, 0x142, 0xa, 0xf, false));  // row_bcast:15, :31
  x = f(x, __builtin_amdgcn_update_dpp(x, x, 0x143, 0xc, 0xf, false));
  return __builtin_amdgcn_readlane(x, 63);
}
__device__ __forceinline__ int wave_min(int x) { return wave_reduce(x, [](int a, int b) { return a < b ? a : b; }); }
__device__ __forceinline__ int wave_max(int x) { return wave_reduce(x, [](int a, int b) { return a > b ? a : b; }); }

// Part k of ns of an item whose streamed segments have pvis visible rows: whole 64-row tiles of them;
// `part` is the item's Item::part.
__device__ __forceinline__ Item cut_item(const Item& it, const int (&pvis)[2], int k, int ns, int part) {
  const int nt0 = (pvis[0] + STILE - 1) / STILE, nt = nt0 + (pvis[1] + STILE - 1) / STILE;
  const int lo = (int)((long long)k * nt / ns), hi = (int)((long long)(k + 1) * nt / ns);
  Item sub = it;
  int srow2[2], slen2[2], spos2[2], scol2[2], scost = 0, n2 = 0;
  bool son[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int base = c ? nt0 : 0, ntc = c ? nt - nt0 : nt0;
    const int l = clampi(lo - base, 0, ntc), h = clampi(hi - base, 0, ntc);
    son[c] = h > l;
    const int skip = l * STILE;
    int len = it.seg_len[c] - skip;
    if (len > (h - l) * STILE) len = (h - l) * STILE;
    int vis = pvis[c] - skip;
    if (vis > (h - l) * STILE) vis = (h - l) * STILE;
    srow2[c] = it.seg_row0[c] + skip; slen2[c] = len; spos2[c] = it.seg_pos0[c] + skip;
    scol2[c] = it.seg_tcol0[c] + skip;
    if (son[c]) { scost += (vis + 31) >> 5; ++n2; }
  }
  const bool f1 = !son[0] && son[1], both = son[0] && son[1];
  sub.nseg = n2; sub.cost = scost; sub.part = part;
  sub.seg_row0[0] = son[0] ? srow2[0] : (f1 ? srow2[1] : 0);
  sub.seg_len[0] = son[0] ? slen2[0] : (f1 ? slen2[1] : 0);
  sub.seg_pos0[0] = son[0] ? spos2[0] : (f1 ? spos2[1] : 0);
  sub.seg_tcol0[0] = son[0] ? scol2[0] : (f1 ? scol2[1] : 0);
  sub.seg_row0[1] = both ? srow2[1] : 0;
  sub.seg_len[1] = both ? slen2[1] : 0;
  sub.seg_pos0[1] = both ? spos2[1] : 0;
  sub.seg_tcol0[1] = both ? scol2[1] : 0;
  return sub;
}

// What it takes to work an item out from the offsets (the fields are those of PlanArgs).
struct DirectPlan {
  const int32_t* off;
  int32_t batch, total_rows, cp, owner_rank, streamed_rank, side, tile, causal, owner_rows, streamed_rows;
  int32_t split_max, split_blocks;
};
// Where in the schedule an item is: its owner tile (counted in schedule order), which part of how many
// of that tile it is, and how many owner tiles of the schedule are cut.
struct DirectSlot { int tile, part, parts, cut_tiles; };

// Item `slot` of a schedule, worked out by one wave from the offsets: batches of at most 64 * K
// sequences, K per lane.  A slot beyond the last item gets no rows.
// The order is heaviest first, by the cost that describe_item gives a tile: the 32-row blocks it sees.  Along an
// owner segment (one per sequence, two in a rank's layout) that cost only grows (queries: each tile sees what the
// one before sees and more) or only shrinks (keys), so the tiles that cost at least v are the last or the
// first of the segment, and their number follows from the position at which the streamed segments have v blocks
// before it (after it).  A bisection over v finds the item's cost, a ballot the sequence.  About 0.5 us for K = 1.
// (With costs in whole tiles instead, launches of a few items per slot, which last as long as their worst
// combination, took up to 10 % longer: one of four ranks, 300 sequences of 500..1500 rows, H = 4, forward 221 ->
// 244, dq 244 -> 256 us.)
// Cut tiles: a tile of cost v has parts(v) = clamp(v / split_blocks, 1, split_max) items, neighbours in the
// order, so the items at or above a cost are sums of the same counts.
template <int K>
__device__ __forceinline__ DirectSlot direct_item(const DirectPlan& d, int slot, Item& it) {
  const int lane = threadIdx.x & 63;
  int s[K], e[K], n[K][2], pos[K][2], len[K][2];  // owner segments: tiles, first position, rows
  int spos[K][2], slen[K][2];                     // streamed segments
  const int tile_log2 = 31 - __builtin_clz(d.tile);  // (a power of two)
  const bool two = d.owner_rank >= 0;                // owner segments per sequence
  int most = 0;  // cost of a tile that sees all
#pragma unroll
  for (int k = 0; k < K; ++k) {
    s[k] = e[k] = 0;
    if (k * 64 + lane < d.batch) seq_range(d.off, k * 64 + lane, d.total_rows, s[k], e[k]);
    const Side so = make_side(e[k] - s[k], d.cp, d.owner_rank), ss = make_side(e[k] - s[k], d.cp, d.streamed_rank);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      pos[k][u] = so.pos[u]; len[k][u] = so.len[u];
      n[k][u] = (so.len[u] >> tile_log2) + ((so.len[u] & (d.tile - 1)) != 0);
      spos[k][u] = ss.pos[u]; slen[k][u] = ss.len[u];
    }
    const int all = blocks_of(ss.len[0]) + blocks_of(ss.len[1]);
    most = all > most ? all : most;
  }
  auto at_least = [&](int k, int u, int v) {  // tiles of the lane's segment (k, u) that cost v or more
    const int tiles = n[k][u];
    if (v <= 0) return tiles;
    const int b0 = blocks_of(slen[k][0]), b1 = blocks_of(slen[k][1]);
    if (!d.causal) return b0 + b1 >= v ? tiles : 0;
    if (d.side == 0) {  // the tile's end is beyond v - 1 blocks
      const bool g = v > b0;
      const int w = g ? v - b0 : v, x = (g ? spos[k][1] : spos[k][0]) + 32 * (w - 1) - pos[k][u];
      const int t = x > 0 ? x >> tile_log2 : 0;
      return (g && w > b1) || x >= len[k][u] ? 0 : tiles - t;
    }
    const bool g = v <= b1;  // more than v - 1 blocks begin at or after the tile
    const int w = g ? v : v - b1, x = (g ? spos[k][1] + slen[k][1] : spos[k][0] + slen[k][0]) - 32 * (w - 1) - 1 - pos[k][u];
    const int c = (x >> tile_log2) + 1;
    return (!g && w > b0) || x < 0 ? 0 : (c < tiles ? c : tiles);
  };
  auto lane_count = [&](int v) {
    int c = 0;
#pragma unroll
    for (int k = 0; k < K; ++k)
      if (k * 64 < d.batch) {
        c += at_least(k, 0, v);
        if (two) c += at_least(k, 1, v);
      }
    return c;
  };
  auto cut_cost = [&](int j) { return j * d.split_blocks; };  // the lowest cost of a tile cut into j parts
  auto count = [&](int v) {  // items of tiles that cost v or more
    int c = lane_count(v);
    for (int j = 2; j <= d.split_max; ++j) c += lane_count(v > cut_cost(j) ? v : cut_cost(j));
    return wave_total(c);
  };
  DirectSlot r = {0, 0, 1, 0};
  if (d.split_max > 1 && slot == 0) r.cut_tiles = wave_total(lane_count(cut_cost(2)));
  it = Item{};
  if (slot >= count(0)) return r;
  int lo = 0, hi = wave_max(most) + 1;  // count(lo) > slot >= count(hi)
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (count(mid) > slot) lo = mid; else hi = mid;
  }
  int rem = slot - count(lo + 1);
  if (d.split_max > 1) {
    while (r.parts < d.split_max && lo >= cut_cost(r.parts + 1)) ++r.parts;
    r.part = rem % r.parts;
    rem /= r.parts;
    r.tile = wave_total(lane_count(lo + 1)) + rem;
  }
  int b = 0, u = 0, t = 0, sb = 0, eb = 0;
  bool found = false;
#pragma unroll
  for (int k = 0; k < K; ++k)
#pragma unroll
    for (int g = 0; g < 2; ++g)
      if (!found && k * 64 < d.batch && (g == 0 || two)) {
        const int from = at_least(k, g, lo), above = at_least(k, g, lo + 1), mine = from - above;
        const int inc = wave_scan(mine), tot = __builtin_amdgcn_readlane(inc, 63);
        if (rem < tot) {
          const int l = (int)__builtin_ctzll(__ballot(rem >= inc - mine && rem < inc));
          b = k * 64 + l;
          u = g;
          sb = __builtin_amdgcn_readlane(s[k], l);
          eb = __builtin_amdgcn_readlane(e[k], l);
          const int first = d.side == 0 && d.causal ? n[k][g] - from : above;  // first tile of that cost
          t = __builtin_amdgcn_readlane(first - (inc - mine), l) + rem;
          found = true;
        } else {
          rem -= tot;
        }
      }
  const int rows = eb - sb;
  int ob = sb, stb = sb;  // first row of the sequence in the two sides' layouts
  if (d.owner_rank >= 0) {
    int c = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) c += k * 64 + lane < b ? len[k][0] + len[k][1] : 0;
    ob = wave_total(c);
  }
  if (d.streamed_rank >= 0) {
    int c = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) c += k * 64 + lane < b ? slen[k][0] + slen[k][1] : 0;
    stb = wave_total(c);
  }
  int pvis[2];
  it = describe_item(make_side(rows, d.cp, d.owner_rank), make_side(rows, d.cp, d.streamed_rank), u, t, ob, stb, 0,
                     d.tile, d.causal, d.side, d.owner_rows, d.streamed_rows, pvis);
  if (r.parts > 1) it = cut_item(it, pvis, r.part, r.parts, slot + 1);
  return r;
}

struct PlanArgs {
  const int32_t* off;     // device, batch + 1
  int32_t batch;
  int32_t total_rows;     // rows of the global layout
  int32_t cp;             // context-parallel size (1 for whole-batch attention)
  int32_t owner_rank;     // -1: owner side is in the global layout
  int32_t streamed_rank;  // -1: streamed side is in the global layout
  int32_t side;           // 0: owners are queries, 1: owners are keys
  int32_t tile;           // owner rows per item
  int32_t causal;
  int32_t owner_rows;     // rows the caller declared for the owner-side buffers
  int32_t streamed_rows;  // rows the caller declared for the streamed-side buffers
  int32_t max_items;      // bound on the items written (parts of split tiles included)
  int32_t max_stiles;     // bound on the 64-row tiles of the streamed side
  int32_t cost_shift;     // cost >> cost_shift selects the sort bin
  int32_t split_max;      // an owner tile is cut into at most this many parts along its streamed
                          // rows (1: never); side 0 only
  int32_t split_blocks;   // ... of at least this many visible 32-row blocks each
  int32_t* red;           // reduce table (see Plan), split_max > 1 only
  int32_t* header;
  int32_t* owner_base;
  int32_t* streamed_base;
  int32_t* tile_base;
  int32_t* stile_base;
  int32_t* ttile;
  int32_t want_ttile;     // the streamed side's tile table is needed (a transposed copy will be built from it)
  int32_t* order;
  Item* items;
};

// The schedules of batches of at most DIRECT_BATCH sequences in cost order: one wave per item (see
// direct_item), up to three schedules in one launch.  Every slot below max_items is written (no rows
// beyond the last item) and the list is in schedule order: Plan::direct.  (Beyond, the work per item grows with the
// batch and plan_kernel is faster: 300 sequences, one of four ranks, 25 us against 38 and more; 128 of median
// 150, forward and backward, 29 -> 18.)
constexpr int DIRECT_BATCH = 128;
struct ItemPlan {
  DirectPlan d;
  Item* items;
  int32_t* header;    // [2]: owner tiles that are cut (see Plan)
  int32_t* red;
  int32_t max_items;
};
struct ItemPlans { ItemPlan p[3]; };
hipError_t launch_item_plans(const ItemPlans& a, int count, hipStream_t stream);

// Builds up to three schedules in one launch (one workgroup each).
hipError_t launch_plans(const PlanArgs* a, int count, hipStream_t stream);
// Schedules of whole batches in natural order (uncut tiles, no table of streamed tiles) of at most that many sequences.
constexpr int NATURAL_BATCH = 1 << 16;
hipError_t launch_natural_plans(const PlanArgs* a, int count, hipStream_t stream);

// What the kernels need to know about a row's timestamp: the timestamp itself and the range of
// the timestamps of the (up to) 32 rows of the same sequence that start at this row, from which
// a 32-row block whose first row this is decides whether one bucket covers all its pairs.
struct TsRecord {
  int32_t ts, lo, hi, pad;
};
static_assert(sizeof(TsRecord) == 16, "one 16-byte record per row");
constexpr int MAX_TS_BUCKETS = 512;

// The bucket of a timestamp difference (the library's reading of section 2.1's sketch of the
// bias; see include/hstu_attn.h): 0 for delta <= 1, else min(nb - 1, e * 2^f + m) with
// e = floor(log2 delta) and m the f bits below delta's leading one.  Integer arithmetic only.
__device__ __forceinline__ int bias_bucket(uint32_t delta, int nb, int f) {
  const uint32_t d = delta > 2u ? delta : 2u;  // (no branch: the result for delta <= 1 is selected below)
  const int e = 31 - __builtin_clz(d);
  const uint32_t top = e >= f ? d >> (e - f) : d << (f - e);
  int b = (e << f) + (int)top - (1 << f);
  b = b < nb - 1 ? b : nb - 1;
  return delta <= 1u ? 0 : b;
}
// The same bucket for delta < 2^24, where the conversion to float is exact: the float's exponent
// and its top f mantissa bits are e and m.  (127 + e) * 2^f + m comes out of one shift of the bit
// pattern; delta = 0 and 1 land at or below zero and are clamped to bucket 0 like the rest.
constexpr uint32_t BIAS_SMALL_DELTA = 1u << 24;
__device__ __forceinline__ int bias_bucket_small(uint32_t delta, int nb, int f) {
  const int b = (int)(__builtin_bit_cast(uint32_t, (float)delta) >> (23 - f)) - (127 << f);
  const int lo = b > 0 ? b : 0;
  return lo < nb - 1 ? lo : nb - 1;
}
// |a - b| of two int32 values, exact up to 2^32 - 1.
__device__ __forceinline__ uint32_t abs_diff(int a, int b) {
  return (uint32_t)(a > b ? a : b) - (uint32_t)(a > b ? b : a);
}

// The gradient of the bias table is a sum of dS over all visible pairs of a bucket.  A workgroup
// of the dq pass sums its share in LDS as 64-bit fixed point with 32 fraction bits: LDS integer
// adds are served ten times faster than LDS float adds (measured: 8 against 80 ns per wave-wide
// instruction and CU), and the sum does not depend on the order of the additions.  Terms below
// 2^-32 are lost and a workgroup's sum for one bucket must stay below 2^31 in magnitude (128
// query rows against all their keys, dS unscaled: dP times SiLU').  The workgroups' sums are then
// added in double precision to a table of the call (acc), which a last small kernel scales and
// rounds to the caller's fp32 table.
constexpr float DW_FIXED_ONE = 4294967296.f;
__device__ __forceinline__ unsigned long long dw_to_fixed(float x) {
  return (unsigned long long)(long long)(x * DW_FIXED_ONE);
}
__device__ __forceinline__ double dw_from_fixed(unsigned long long q) {
  return (double)(long long)q * (1.0 / 4294967296.0);
}
// d_w[i] = (accumulate ? d_w[i] : 0) + scale * acc[i] for the nb buckets.
hipError_t launch_dw_finish(const double* acc, float* d_w, int nb, double scale, int accumulate,
                            hipStream_t stream);

// Builds the records of `total_rows` rows (rec has total_rows + 64 entries; the surplus is
// cleared) and, if acc is not null, clears the nb entries of the call's table of sums.  off: the
// offsets of the whole-batch layout (a row's range stops at the end of its sequence), or null for
// any other layout of rows (the range covers the next 32 rows whatever they belong to: a superset,
// which only makes the one-bucket test of a block more cautious).
hipError_t launch_ts_records(const int32_t* ts, const int32_t* off, int batch, int64_t total_rows,
                             TsRecord* rec, double* acc, int nb, hipStream_t stream);

// Packed tiles: schedules whose owner tiles are `tile` consecutive rows of the batch whatever
// sequences they belong to (item t = rows [t * tile, (t + 1) * tile), in natural order), for both
// sides at once, plus the per-row sequence bounds the kernels' windows come from.  Positions are
// row numbers.  Rows at or beyond off[batch] (clamped to total_rows) belong to no item.
struct PackedPlanArgs {
  const int32_t* off;
  int32_t batch, total_rows, tile, causal;
  int2* row_seq;                    // total_rows entries
  int32_t* header[2];               // per side (0: owners are queries, 1: keys): see Plan
  int32_t* order[2];
  Item* items[2];
};
hipError_t launch_packed_plan(const PackedPlanArgs& a, hipStream_t stream);

// Arguments of the attention kernels.
struct AttnArgs {
  const void* q;
  const void* k;
  const void* v;
  const void* d_o;
  const void* vt;   // transposed copy of v (bf16 forward; see launch_transpose_bf16)
  void* o;
  void* dq;
  void* dk;
  void* dv;
  Plan plan;
  DirectPlan self;  // off not null: every wave works its item out by itself (see direct_item), there is no schedule
  int32_t num_heads;
  int32_t causal;
  int32_t accumulate;
  int32_t max_items;
  int32_t waves;    // wavefronts per workgroup (bf16 kernels): owner tile = 32 * waves rows
  int32_t out_f32;  // outputs are fp32 (bf16 kernels only; the fp32 kernels always write fp32)
  int32_t item_parts;  // fp32 kernels: workgroups an item's rows are shared by, 32 rows each
  float* partial;   // partial results of split tiles: [slot][head][tile row][d] fp32 (or null)
  float* partial2;  // the same of the second result (forward and dq pass in one)
  float alpha;
  float inv_n;
  // Timestamp bias (ts_rec == null: no bias).
  const TsRecord* ts_rec;      // per row of the streamed side's buffers, built by launch_ts_records
  const TsRecord* ts_rec_own;  // per row of the owner side's buffers (the same array for whole batches)
  const float* ts_w;       // bucket table, nb entries
  double* d_ts_acc;        // the call's sums of dS per bucket (dq pass: added with atomics), or null
  int32_t nb;              // buckets
  int32_t fbits;           // log2 of the groups per octave
  int32_t bias_per_pair;   // no block takes the one-bucket path (HSTU_FLAG_BIAS_PER_PAIR)
  // Packed tiles (bf16 kernels, whole-batch layout, batches of short sequences; null: not packed):
  // per row the first row and the end row of its sequence, built by launch_packed_plan.
  const int2* row_seq;
  // Large batch (many items, none of them a large share of the whole): kernels that run one
  // workgroup per CU may launch as many workgroups as CUs and let each walk over its share.
  int32_t large_batch;
  // Schedules in natural order (the items of a sequence are neighbours in the list) with a head
  // count that divides 8: the hardware hands workgroup i to XCD i % 8, each XCD with an L2 of
  // its own, so the unit -> (item, head) map gives every XCD one head and one contiguous part
  // of the list (8 / heads parts) and the tiles of a sequence, which stream the same rows, meet
  // in one L2.  1: the plain map, unit = item * heads + head (with 8 heads that already is one
  // head per XCD).
  int32_t xcd_parts;
  // Walking workgroups take contiguous runs of their XCD's units instead of every n-th unit
  // (natural order with a head count that divides 8).
  int32_t walk_chunks;
  // ... of equal work instead of equal numbers of units (Item::before and header[3] are filled in).
  int32_t walk_costs;
  int32_t single_segment;  // every item has one streamed segment at most (the streamed side is the whole batch's)
  // dk/dv pass: keep to the kernel with one wave per 32 keys where the two-wave kernel would serve.
  int32_t dkdv_one_wave;
};

// Owner rows per item each kernel family expects (pass: 0 forward, 1 dk/dv, 2 dq); the
// schedule must be built with the same value.
enum { PASS_FWD = 0, PASS_DKDV = 1, PASS_DQ = 2 };
// Wavefronts per workgroup (32 owner rows each) the bf16 kernels of a pass use for a problem
// with `owner_rows` owner rows and `heads` heads: large problems take the wider workgroup, which
// halves the traffic of streamed tiles; small ones keep enough workgroups to fill the chip.
int waves_bf16(int pass, int64_t owner_rows, int heads);
int tile_rows_f32(int pass);

// Transposed copy of a streamed bf16 tensor: src [rows, H, D] -> dst [H, D, 64 * max_stiles], one
// 64-column group per streamed tile, columns permuted inside each group of 16 into the order
// the matrix instructions consume them, zero beyond the valid rows.
hipError_t launch_transpose_bf16(const void* src, void* dst, const Plan& plan, int num_heads, int d,
                                 hipStream_t stream);

// Load-balance reorder (section 2.3): copies the 64-row tiles of a rank's local layout from / to
// their place in the global layout, for `count` tensors whose rows are row_bytes[i] long.
struct ReorderArgs {
  const char* src[4];
  char* dst[4];
  int64_t row_bytes[4];
  const int32_t* off;
  int32_t count;
  int32_t scatter;  // 0: dst is local, src global (gather); 1: dst is global, src local
  int32_t batch, total_rows, local_rows, cp, rank;
  int32_t split;    // workgroups per 64-row tile (a divisor of 64)
};
// max_tiles: an upper bound on the 64-row tiles of the local layout (the grid's first dimension).
hipError_t launch_reorder(const ReorderArgs& a, int64_t max_tiles, hipStream_t stream);

// Sums the partial results of split owner tiles (in slot order: deterministic) into `out`
// [rows, H, d] with the output conventions of the attention kernels.
hipError_t launch_reduce_partials(const Plan& plan, int64_t max_tiles, const float* partial, void* out,
                                  int num_heads, int d, int tile_rows, int accumulate, int out_f32,
                                  hipStream_t stream);

hipError_t launch_fwd_bf16(const AttnArgs& a, int d_qk, int d_v, hipStream_t stream);
hipError_t launch_dkdv_bf16(const AttnArgs& a, int d_qk, int d_v, hipStream_t stream);
// The dk/dv pass with two waves per 32 keys (plain per-sequence schedules at d_qk = d_v = 128).
bool dkdv_pair_supported(const AttnArgs& a, int d_qk, int d_v);
hipError_t launch_dkdv_pair_bf16(const AttnArgs& a, int d_qk, int d_v, hipStream_t stream);
// Forward and dq pass in one kernel, d_qk = d_v = 128, no bias (a: its fields as hstu_fwd_dq_pair_bf16 names them).
hipError_t launch_fwd_dq_pair_bf16(const AttnArgs& a, int d_qk, int d_v, hipStream_t stream);
bool dkdv_walk_supported(const AttnArgs& a, int d_qk, int d_v);
hipError_t launch_dkdv_walk_bf16(const AttnArgs& a, int d_qk, int d_v, hipStream_t stream);
hipError_t launch_dq_bf16(const AttnArgs& a, int d_qk, int d_v, hipStream_t stream);
// dq, dk and dv of batches of short sequences in one kernel; a.self gives offsets, batch and rows.
bool bwd_short_supported(int d_qk, int d_v);
hipError_t launch_bwd_short_bf16(const AttnArgs& a, int d_qk, int d_v, hipStream_t stream);
hipError_t launch_fwd_f32(const AttnArgs& a, int d_qk, int d_v, hipStream_t stream);
hipError_t launch_dkdv_f32(const AttnArgs& a, int d_qk, int d_v, hipStream_t stream);
// dk/dv and dq pass in one launch (k, q: their arguments), for small calls without bias.
bool bwd_f32_supported(const AttnArgs& k, const AttnArgs& q, int d_qk, int d_v, int max_len);
hipError_t launch_bwd_f32(const AttnArgs& k, const AttnArgs& q, int d_qk, int d_v, int max_len, hipStream_t stream);
hipError_t launch_dq_f32(const AttnArgs& a, int d_qk, int d_v, hipStream_t stream);

// Measurement kernels (hstu_probe.hip): a loop of matrix instructions only (flops per launch
// returned), and fp32 atomic adds in the pattern of a dq produced by the dk/dv pass (payload
// bytes per launch returned).
hipError_t launch_mfma_loop(int iters, int random, float* sink, double* flops, hipStream_t stream);
hipError_t launch_dq_atomic(float* buf, int64_t rows, int heads, int nblk, int local, double* bytes,
                            hipStream_t stream);

}  // namespace hstu
