// Kernel work list of the prefix-shared decode attention.
//
// The attention kernel runs one persistent workgroup per compute unit; each
// workgroup walks a chain of unit records. A unit is a set of query rows
// (whole beams, consecutive in the canonical order, one KV head) and a list
// of KV blocks, each applying to a contiguous range of those rows. Two kinds
// of unit cover every (beam, used block) exactly once per KV head:
//
// * Wide units. A segment of more rows than one wave group of a narrow unit
//   takes (kGroupRows) is cut into row chunks of whole beams (up to
//   kMaxWideRows rows, or a smaller cap the cost model picks; the eight waves
//   of the workgroup share every block through LDS, each computing one or
//   two row tiles) and, along its blocks, into pieces; every (piece, chunk)
//   is a unit whose blocks apply to all of its rows. (Short pieces may go to
//   narrow-mode units instead, and fp32 caches use only those.) The chunks
//   of one piece read the same blocks and are placed on one XCD.
// * Narrow units. Everything else -- segments of few beams and every beam's
//   private tail -- is listed depth-first over the prefix tree (a segment's
//   blocks, then its subtrees and the tails of the beams ending at it, in
//   canonical order). Consecutive entries of that list always cover a
//   contiguous range of beams, so the list is cut into units of at most
//   kMaxUnitBeams beams / kMaxRows rows (kGroupRows in streaming batches) /
//   kMaxUnitEntries entries and about equal cost: a small subtree with its
//   tails becomes one unit and one partial state per beam instead of one per
//   segment.
//
// Units are replicated per KV head, grouped, spread over the XCDs longest
// first and then over each XCD's workgroups longest first.
#include <algorithm>
#include <cmath>
#include <numeric>

#include "tts_meta.h"

namespace tts {
namespace {

// Cost model (microseconds of one workgroup, all compute units busy),
// fitted to per-unit clock marks of the kernel at the 7B-shaped batches
// (D 128, g 7; bf16: the 64-beam trees, the straggler batch and the
// verification of four tokens; fp8: the long-chain batch). Every unit pays
// a fixed part (its first memory round trips, the end of its loop, the
// partial writes).
// * Narrow: 3.0 us + 0.26 us per 8 KiB block (fp8: 0.225 us per 4 KiB one) +
//   0.05 us per query row; with more than 32 rows, whose waves work in two
//   groups, 1.5 us more, and blocks with rows of both groups count twice.
// * Wide, up to eight row tiles (each half of the waves takes every other
//   pair): 5.3 us + (0.27 + 0.011 tiles) us per 8 KiB block; more tiles:
//   5.3 us + (0.12 + 0.029 tiles) us. fp8: 5.3 us + (0.175 + 0.0325 tiles)
//   us per block, in both forms.
// * fp32 (16 rows to a wave group, four groups of two waves above 32 rows):
//   the larger of 0.26 us per 8 KiB of blocks and of the matrix cores' time,
//   0.24 us per block and row tile (D 128; four times the largest tile's
//   blocks with four groups, whose waves do not help each other out); 1.5 us
//   more with several groups. Fitted to whole calls: 36 drawn decode and
//   verification batches of both head sizes take 0.945 times as long as with
//   the bf16 terms scaled by the bytes, 40 of D 64 0.940 times.
// Every shape scales the tile term by the head size.
constexpr double kNarrowFixedUs = 3.0, kNarrowBlockUs = 0.26, kRowUs = 0.05, kGroupsUs = 1.5;
constexpr double kWideFixedUs = 5.3;
constexpr double kHalvesBlockUs = 0.27, kHalvesTileUs = 0.011;
constexpr double kFullBlockUs = 0.12, kFullTileUs = 0.029;
constexpr double kFp8NarrowBlockUs = 0.225;
constexpr double kFp8WideBlockUs = 0.175, kFp8WideTileUs = 0.0325;
constexpr double kF32NarrowBlockUs = 0.26, kF32TileBlockUs = 0.24;
// Where the batch holds many bytes per workgroup the narrow units' blocks
// come at the rate of the memory, not of one workgroup's round trips: 0.33
// us per block with every workgroup streaming (straggler batch) against 0.26
// where half of them run wide units (64-beam tree). Above this many KV bytes
// per workgroup the bf16 narrow block term is scaled by 1.3.
constexpr double kStreamBytesPerGroup = 400e3, kStreamScale = 1.3;
constexpr int kGroupRows = 32;  // rows of a narrow unit whose waves work in one group
constexpr int kXcds = 8;  // workgroup k of a launch runs on XCD k % 8
constexpr int kFewWideRows = 192, kStreamWideRows = 128;  // wide-unit row caps tried besides kMaxWideRows
constexpr double kCapGain = 0.97;
// Units of a chain beyond this many per workgroup are weighed against fewer,
// larger ones, with this much more for each of them than the terms above say
// (fitted to 40 batches of 600 to 3,072 beams in both plans: 2.5 us, the
// fewest wrong choices at 3).
constexpr double kLongChain = 4, kChainUnitUs = 3.0;
constexpr double kSmallWorkUs = 1.5;  // modelled block time per workgroup (half of a unit's fixed part)
// The merge (a second launch): a fixed cost, and for the beam with the most
// partial states their writing and reading.
constexpr double kMergeFixedUs = 3.2;
constexpr double kMergeSlotUs = 0.06;

int tiles_of(int rows) { return (rows + 15) / 16; }

// The blocks of a narrow unit: how many, how many with rows of both wave
// groups, which both read; for fp32 caches also how many reads the busiest row
// tile and the first two tiles need.
struct NarrowLoad {
  int blocks = 0, span = 0;
  int most = 0, low = 0;
};

struct CostModel {
  double blk_bytes, q_row_bytes, part_row_bytes, d_scale;
  bool fp8 = false, f32 = false;
  double narrow_scale = 1.0;  // kStreamScale where the batch is bound by streaming
  double row_us() const { return kRowUs * (q_row_bytes + part_row_bytes) / 800.0; }
  // Narrow units: the waves split the block pairs, every wave runs every tile.
  double narrow_us(const NarrowLoad& x, int rows) const {
    if (f32) {
      const int tiles = rows > 32 ? 4 * x.most : x.low;
      return kNarrowFixedUs + (rows > 16 ? kGroupsUs : 0.0) +
             std::max(x.blocks * narrow_block_us(), tiles * f32_tile_us()) + rows * row_us();
    }
    return kNarrowFixedUs + (rows > kGroupRows ? kGroupsUs : 0.0) + (x.blocks + x.span) * narrow_block_us() +
           rows * row_us();
  }
  double f32_tile_us() const { return kF32TileBlockUs * d_scale; }
  double narrow_block_us() const {
    if (f32) return blk_bytes * (kF32NarrowBlockUs / 8192);
    return fp8 ? kFp8NarrowBlockUs : narrow_scale * blk_bytes * (kNarrowBlockUs / 8192);
  }
  // Wide units: one block, all tiles.
  double wide_block_us(int rows) const {
    const int nt = tiles_of(rows);
    if (fp8) return kFp8WideBlockUs + nt * kFp8WideTileUs * d_scale;
    if (nt <= kUnitWaves) return blk_bytes * (kHalvesBlockUs / 8192) + nt * kHalvesTileUs * d_scale;
    return blk_bytes * (kFullBlockUs / 8192) + nt * kFullTileUs * d_scale;
  }
  double wide_us(int blocks, int rows) const { return kWideFixedUs + blocks * wide_block_us(rows); }
};

// A unit of one KV head: a run [a, b) of the narrow list's items, or (seg >=
// 0) of the blocks of a segment that is cut into units of its own. Its
// entries are written out only for the plan that is taken (Entries).
struct Tmpl {
  int32_t lo = 0, hi = 0;  // beam positions [lo, hi)
  int32_t mode = kModeNarrow;
  int32_t seg = -1;
  int32_t a = 0, b = 0;
  double cost = 0;
  int32_t group = -1;  // units of a segment: index of their piece
};

struct Entries {
  std::vector<int32_t> ids;
  std::vector<uint32_t> info;
  int32_t nstatic = 0;   // narrow: static entries of the first window; wide: all entries
  int32_t nstatic2 = 0;  // narrow: entries of the second window (after the extension entries)
};

struct NItem {
  int32_t id;
  int32_t p0, p1;
  int32_t valid;
  uint32_t flags;
  int32_t run = 1;  // from here, plain blocks of the same beams (they follow each other)
};

struct Work {
  int32_t t, kvh;
  double cost;
};

// Which of a unit's beams (t.lo + i) it writes partial states for: all of
// a segment's unit; of a narrow run those that some item covers.
void touched_beams(const Tmpl& t, const std::vector<NItem>& items, std::vector<char>* out) {
  out->assign(t.hi - t.lo, t.seg >= 0 ? 1 : 0);
  for (int32_t k = t.a; t.seg < 0 && k < t.b; ++k)
    for (int32_t i = items[k].p0 - t.lo; i < items[k].p1 - t.lo; ++i) (*out)[i] = 1;
}

}  // namespace

void build_work_plan(const HostMeta& m, const PlanShape& shape, WorkPlan* plan, const WorkPlan* warm) {
  WorkPlan& P = *plan;
  P = WorkPlan();
  const int32_t S = m.num_seqs;
  const int32_t g = shape.num_q_heads / shape.num_kv_heads;
  const int32_t hkv = shape.num_kv_heads;
  const int32_t bs = m.block_size;
  // Beams per narrow unit: set per candidate row cap below.
  auto narrow_beams = [&](int32_t cap_rows) { return std::max(1, std::min(kMaxUnitBeams, cap_rows / g)); };
  int32_t RB = narrow_beams(kMaxRows);
  // Beams per wide unit (bf16 and fp8 caches; segments of fp32 caches are cut
  // into chunks of as many rows as a narrow unit holds, whatever the cap of
  // the narrow list): set per candidate row cap below.
  const bool wide_mode = shape.kv_bytes <= 2;
  int32_t RW = RB;
  auto wide_beams = [&](int32_t cap_rows) {
    return wide_mode ? std::max(1, std::min(kMaxWideBeams, cap_rows / g)) : narrow_beams(kMaxRows);
  };
  const int32_t nseg = static_cast<int32_t>(m.seg_req.size());
  const int32_t nbins = std::max(1, shape.num_bins);
  P.num_bins = nbins;
  P.build_len.assign(m.seq_lens.begin(), m.seq_lens.end());

  CostModel cm;
  cm.blk_bytes = 2.0 * bs * shape.head_dim * shape.kv_bytes;
  cm.q_row_bytes = shape.head_dim * (shape.kv_bytes == 4 ? 4.0 : 2.0);
  // A partial state is written once and read once by the merge.
  cm.part_row_bytes = 2.0 * (shape.head_dim * (shape.kv_bytes == 4 ? 4.0 : 2.0) + 4 * kPartMl);
  cm.d_scale = shape.head_dim / 128.0;
  cm.fp8 = shape.kv_bytes == 1;
  cm.f32 = shape.kv_bytes == 4;

  const bool streaming = static_cast<double>(m.unique_blocks) * hkv * cm.blk_bytes > kStreamBytesPerGroup * nbins;
  if (streaming) cm.narrow_scale = kStreamScale;

  // ---- tree structure ----------------------------------------------------
  std::vector<std::vector<int32_t>> children(nseg), leaves(nseg);
  std::vector<std::vector<std::pair<int32_t, int32_t>>> top(std::max<size_t>(1, m.req_off.size()) - 1);
  auto req_of_pos = [&](int32_t pos) {
    return static_cast<int32_t>(std::upper_bound(m.req_off.begin(), m.req_off.end(), pos) - m.req_off.begin()) - 1;
  };
  for (int32_t s = 0; s < nseg; ++s) {
    if (m.seg_parent[s] >= 0)
      children[m.seg_parent[s]].push_back(s);
    else
      top[m.seg_req[s]].push_back({m.seg_beam_begin[s], s});
  }
  for (int32_t pos = 0; pos < S; ++pos) {
    const int32_t b = m.perm[pos];
    const int32_t k0 = m.path_seg_off[b], k1 = m.path_seg_off[b + 1];
    if (k1 > k0)
      leaves[m.path_seg[k1 - 1]].push_back(pos);
    else
      top[req_of_pos(pos)].push_back({pos, -1 - pos});
  }
  std::vector<char> wide(nseg, 0);
  auto seg_block = [&](int32_t s, int32_t j) {
    const int32_t b = m.perm[m.seg_beam_begin[s]];
    return m.tables[static_cast<size_t>(b) * m.max_blocks + m.seg_lblock_begin[s] + j];
  };

  // ---- depth-first list of the narrow work --------------------------------
  std::vector<NItem> items;
  auto emit_tail = [&](int32_t pos) {
    const int32_t b = m.perm[pos];
    const int32_t L = m.seq_lens[b];
    const int32_t nb = (L + bs - 1) / bs;
    for (int32_t j = m.tail_lblock[b]; j < nb; ++j) {
      const int32_t v = std::min(bs, L - j * bs);
      const uint32_t fl = (j == nb - 1 && v < bs) ? kEntLive : 0u;
      items.push_back({m.tables[static_cast<size_t>(b) * m.max_blocks + j], pos, pos + 1, v, fl});
    }
    items.push_back({0, pos, pos + 1, 1, kEntExt});
  };
  // Iterative walk: a stack of (segment, or -1 - leaf position).
  std::vector<int32_t> stack;
  auto push_sorted = [&](std::vector<std::pair<int32_t, int32_t>>& v) {
    std::sort(v.begin(), v.end());
    for (auto it = v.rbegin(); it != v.rend(); ++it) stack.push_back(it->second);
  };
  std::vector<std::pair<int32_t, int32_t>> tmp;
  auto list_items = [&]() {
    // A segment of more rows than one wave group takes is cut into units of
    // its own (left to narrow units of two groups, its blocks are read twice:
    // 7B 64-beam tree 24.4 us per call against 23.1; fp32 caches, and plans
    // of few units: of more than a narrow unit takes, beams' blocks beside
    // their segment's need no unit and no state of their own).
    const int32_t most = wide_mode && !P.few_units ? narrow_beams(kGroupRows) : RB;
    for (int32_t s = 0; s < nseg; ++s) wide[s] = (m.seg_beam_end[s] - m.seg_beam_begin[s]) > most;
    items.clear();
    for (auto& t : top) {
      push_sorted(t);
      while (!stack.empty()) {
        const int32_t x = stack.back();
        stack.pop_back();
        if (x < 0) {
          emit_tail(-1 - x);
          continue;
        }
        const int32_t bb = m.seg_beam_begin[x], be = m.seg_beam_end[x];
        if (!wide[x]) {
          for (int32_t j = 0; j < m.seg_nblocks[x]; ++j)
            items.push_back({seg_block(x, j), bb, be, bs, 0u});
        }
        tmp.clear();
        for (int32_t c : children[x]) tmp.push_back({m.seg_beam_begin[c], c});
        for (int32_t pos : leaves[x]) tmp.push_back({pos, -1 - pos});
        push_sorted(tmp);
      }
    }
    for (size_t k = items.size(); k-- > 1;) {
      NItem& x = items[k - 1];
      const NItem& y = items[k];
      if (x.flags == 0 && y.flags == 0 && x.p0 == y.p0 && x.p1 == y.p1) x.run = y.run + 1;
    }
  };

  // ---- units for a target unit time T ------------------------------------
  // A wide segment of G beams and n blocks is cut into C row chunks and P
  // pieces, in the wide mode (chunks of up to RW beams) or the narrow mode
  // (up to RB beams): among the choices whose units fit T the one with the
  // least share of the modelled time, its units' time over the workgroups
  // plus the merge of its pieces' states (else the fastest). The narrow list
  // is cut greedily into units that fit T.
  auto narrow_us = [&](int32_t blocks, int32_t rows) {  // every block for all rows
    return cm.narrow_us({blocks, rows > kGroupRows ? blocks : 0, blocks, std::min(2, tiles_of(rows)) * blocks}, rows);
  };
  auto make_templates = [&](double T, std::vector<Tmpl>& tm) {
    tm.clear();
    int32_t ngroups = 0;
    for (int32_t s = 0; s < nseg; ++s) {  // preorder: ancestors first
      if (!wide[s]) continue;
      const int32_t bb = m.seg_beam_begin[s], G = m.seg_beam_end[s] - bb;
      const int32_t n = m.seg_nblocks[s], np = (n + 1) / 2;
      struct Choice {
        int32_t mode, C, P;
        double share, us;
      } best{kModeNarrow, 0, 0, 0, 0};
      bool have = false, best_fits = false;
      for (int32_t mode : {kModeWide, kModeNarrow}) {
        if (mode == kModeWide && !wide_mode) continue;
        const int32_t cap = mode == kModeWide || !wide_mode ? RW : RB;
        for (int32_t C = (G + cap - 1) / cap; C <= std::min(G, 4 * ((G + cap - 1) / cap)); ++C) {
          const int32_t rows = ((G + C - 1) / C) * g;
          const int32_t max_ent = mode == kModeWide ? kMaxUnitEntries : kMaxEntries;
          for (int32_t P = std::max(1, (n + max_ent - 1) / max_ent); P <= np; ++P) {
            const int32_t blocks = std::min(n, 2 * ((np + P - 1) / P));
            const double us = mode == kModeWide ? cm.wide_us(blocks, rows) : narrow_us(blocks, rows);
            const double share = C * P * us * hkv / nbins + kMergeSlotUs * P;
            const bool fits = us <= T;
            const bool better = !have || (fits && !best_fits) ||
                                (fits == best_fits && (fits ? share < best.share : us < best.us));
            if (better) {
              best = {mode, C, P, share, us};
              best_fits = fits;
              have = true;
            }
            if (fits) break;  // more pieces only add fixed parts
          }
        }
      }
      const int32_t C = best.C, pieces = best.P;
      for (int32_t j = 0; j < pieces; ++j) {
        const int32_t a = 2 * static_cast<int32_t>(static_cast<int64_t>(np) * j / pieces);
        const int32_t e = std::min(n, 2 * static_cast<int32_t>(static_cast<int64_t>(np) * (j + 1) / pieces));
        for (int32_t c = 0; c < C; ++c) {
          Tmpl t;
          t.lo = bb + static_cast<int32_t>(static_cast<int64_t>(G) * c / C);
          t.hi = bb + static_cast<int32_t>(static_cast<int64_t>(G) * (c + 1) / C);
          const int32_t rows = (t.hi - t.lo) * g;
          t.mode = best.mode;
          t.seg = s;
          t.a = a;
          t.b = e;
          t.cost = t.mode == kModeWide ? cm.wide_us(e - a, rows) : narrow_us(e - a, rows);
          t.group = ngroups;
          tm.push_back(t);
        }
        ++ngroups;
      }
    }
    Tmpl cur;
    // The open unit's static items, and its LIVE and extension items.
    NarrowLoad load;
    int32_t tile[kMaxRows / 16] = {};  // fp32: blocks of each row tile
    int32_t nlive_ext = 0;
    auto with = [&](const NItem& it, int32_t lo, int32_t n) {  // n blocks of the item's beams more
      NarrowLoad x = load;
      if (it.flags & kEntExt) return x;
      const int32_t r0 = (it.p0 - lo) * g, r1 = (it.p1 - lo) * g;
      x.blocks += n;
      if (r0 < kGroupRows && r1 > kGroupRows) x.span += n;
      for (int32_t t = r0 / 16; cm.f32 && 16 * t < r1; ++t) {
        x.most = std::max(x.most, tile[t] + n);
        x.low += t < 2 ? n : 0;
      }
      return x;
    };
    auto flush = [&]() {
      if (cur.b == cur.a) return;
      cur.cost = cm.narrow_us(load, (cur.hi - cur.lo) * g);
      tm.push_back(cur);
      cur.a = cur.b;
      load = NarrowLoad();
      std::fill(tile, tile + kMaxRows / 16, 0);
      nlive_ext = 0;
    };
    // (Costs grow with the blocks: a run whose last block fits, fits.)
    for (int32_t k = 0, n = 0; k < static_cast<int32_t>(items.size()); k += n) {
      const NItem& it = items[k];
      const int32_t live = (it.flags & (kEntLive | kEntExt)) ? 1 : 0;
      const bool open = cur.b > cur.a;
      const int32_t lo = open ? std::min(cur.lo, it.p0) : it.p0, hi = open ? std::max(cur.hi, it.p1) : it.p1;
      auto fits = [&](int32_t m) {
        return hi - lo <= RB && cur.b - cur.a + m <= kMaxUnitEntries && nlive_ext + live <= kMaxEntries &&
               cm.narrow_us(with(it, lo, m), (hi - lo) * g) <= T;
      };
      n = it.run;
      if (n > 1 && !fits(n)) n = 1;
      if (n == 1 && open && !fits(1)) {
        flush();
        n = 0;  // the item opens the next unit
        continue;
      }
      cur.lo = lo;
      cur.hi = hi;
      cur.b = k + n;
      load = with(it, lo, n);
      for (int32_t t = (it.p0 - lo) * g / 16; cm.f32 && !(it.flags & kEntExt) && 16 * t < (it.p1 - lo) * g; ++t)
        tile[t] += n;
      nlive_ext += live;
    }
    flush();
  };

  // A unit's entries: the first window holds its LIVE entries, static
  // entries up to 64 with the extension entries, which come last; the
  // second window the remaining static entries (the order of a unit's
  // blocks does not change its result beyond rounding).
  auto write_entries = [&](const Tmpl& t, Entries* out) {
    Entries& x = *out;
    x.ids.clear();
    x.info.clear();
    if (t.seg >= 0) {
      const uint32_t info = t.mode == kModeWide ? 0u : ent_info(0, (t.hi - t.lo) * g, bs, 0u);
      for (int32_t k = t.a; k < t.b; ++k) x.ids.push_back(seg_block(t.seg, k));
      x.info.assign(x.ids.size(), info);
      x.nstatic = t.b - t.a;
      x.nstatic2 = 0;
      return;
    }
    auto push = [&](const NItem& it) {
      const bool is_ext = (it.flags & kEntExt) != 0;
      x.ids.push_back(is_ext ? it.p0 - t.lo : it.id);
      x.info.push_back(ent_info((it.p0 - t.lo) * g, (it.p1 - t.lo) * g, it.valid, it.flags));
    };
    int32_t room = kMaxEntries;  // plain static entries the first window takes
    for (int32_t k = t.a; k < t.b; ++k) room -= (items[k].flags & (kEntLive | kEntExt)) ? 1 : 0;
    int32_t plain = 0;
    for (int32_t k = t.a; k < t.b; ++k) {
      if (items[k].flags & kEntExt) continue;
      if ((items[k].flags & kEntLive) || plain++ < room) push(items[k]);
    }
    x.nstatic = static_cast<int32_t>(x.ids.size());
    for (int32_t k = t.a; k < t.b; ++k)
      if (items[k].flags & kEntExt) push(items[k]);
    plain = 0;
    for (int32_t k = t.a; k < t.b; ++k)
      if (!(items[k].flags & (kEntLive | kEntExt)) && plain++ >= room) push(items[k]);
    x.nstatic2 = std::max(0, plain - room);
  };

  // ---- placement: groups -> XCDs -> workgroups ------------------------------
  // Units are replicated per KV head. The wide chunks of one piece (same
  // KV head) form a group that stays on one XCD, so they share its L2;
  // groups go to the XCDs longest first, then each XCD's units to its
  // workgroups longest first. Returns the largest workgroup load.
  // bins: each workgroup's units, or null for the load alone.
  struct Group {  // templates [t0, t1) of one KV head
    int32_t t0, t1, kvh;
    double cost;
  };
  std::vector<Group> groups;
  auto place = [&](const std::vector<Tmpl>& tm, std::vector<std::vector<Work>>* bins) {
    groups.clear();
    for (int32_t kvh = 0; kvh < hkv; ++kvh) {
      for (int32_t t = 0; t < static_cast<int32_t>(tm.size()); ++t) {
        if (tm[t].group >= 0 && t > 0 && tm[t].group == tm[t - 1].group) {
          groups.back().t1 = t + 1;
          groups.back().cost += tm[t].cost;
        } else {
          groups.push_back({t, t + 1, kvh, tm[t].cost});
        }
      }
    }
    std::vector<int32_t> gorder(groups.size());
    std::iota(gorder.begin(), gorder.end(), 0);
    std::stable_sort(gorder.begin(), gorder.end(),
                     [&](int32_t a, int32_t b) { return groups[a].cost > groups[b].cost; });
    const int32_t nx = std::min(kXcds, nbins);
    std::vector<int32_t> xbins(nx, 0);
    for (int32_t k = 0; k < nbins; ++k) xbins[k % nx]++;
    std::vector<double> xload(nx, 0);
    std::vector<std::vector<Work>> xunits(nx);
    for (int32_t gi : gorder) {
      int32_t x = 0;
      for (int32_t k = 1; k < nx; ++k)
        if (xload[k] / xbins[k] < xload[x] / xbins[x]) x = k;
      xload[x] += groups[gi].cost;
      for (int32_t t = groups[gi].t0; t < groups[gi].t1; ++t) xunits[x].push_back({t, groups[gi].kvh, tm[t].cost});
    }
    if (bins) bins->assign(nbins, {});
    double makespan = 0;
    for (int32_t x = 0; x < nx; ++x) {
      auto& v = xunits[x];
      std::stable_sort(v.begin(), v.end(), [](const Work& a, const Work& b) { return a.cost > b.cost; });
      std::vector<int32_t> mine;
      for (int32_t k = x; k < nbins; k += nx) mine.push_back(k);
      std::vector<double> load(mine.size(), 0);
      for (const Work& w : v) {
        size_t best = 0;
        for (size_t k = 1; k < mine.size(); ++k)
          if (load[k] < load[best]) best = k;
        load[best] += w.cost;
        if (bins) (*bins)[mine[best]].push_back(w);
      }
      for (double l : load) makespan = std::max(makespan, l);
    }
    // Within a workgroup, wide units first (their chunks run concurrently on
    // the XCD's other workgroups and share its L2), then in creation order.
    if (bins)
      for (auto& v : *bins)
        std::stable_sort(v.begin(), v.end(), [](const Work& a, const Work& b) { return a.t < b.t; });
    return makespan;
  };

  // ---- target search ---------------------------------------------------------
  // Units of about equal cost: the smallest target T whose units (times the
  // KV heads) fit in the workgroups, one each, is found by bisection (the
  // unit count only falls as T grows). From there a few smaller targets,
  // whose units are chained several to a workgroup, and larger ones, whose
  // longer units leave fewer partial states to merge, are placed too, and
  // the one with the least modelled time (the largest workgroup load plus
  // the merge) is taken. When even the largest units outnumber the
  // workgroups, the targets are taken around the average work.
  std::vector<Tmpl> tm;
  // Units (of one KV head) that fit the workgroups one each. Where there is
  // little work per workgroup (kSmallWorkUs), a batch with enough beams to
  // fill half of them at four units per beam and head gets no more than that,
  // and one with fewer beams no chained units: few partial states per beam.
  // With more work the bound lengthens the units instead: in trees with long
  // private tails, 10 beams of 7B shape over fp8 took 49.3 us per call with
  // it and 30.4 without, 16 of 1.5B shape 21.8 and 18.1. Below the line its
  // cost is the smaller one (1.5B 16-beam tree 12.4 us per call against
  // 11.2, 7B shape with 8 beams 12.5 against 11.6; most batches within 1%).
  const int32_t all_units = std::max(1, nbins / hkv);
  const int32_t few_units = 4 * S >= all_units / 2 ? std::min(all_units, 4 * S) : all_units;
  int32_t fit_units = all_units;
  const double target0 = kNarrowFixedUs;  // a unit's fixed part: targets scale what is above it
  auto units_at = [&](double T) {
    make_templates(T, tm);
    return static_cast<int32_t>(tm.size());
  };
  std::vector<char> touched;
  std::vector<int32_t> slot_cnt;
  auto merge_us = [&](const std::vector<Tmpl>& t) {
    slot_cnt.assign(S, 0);
    for (const Tmpl& x : t) {
      touched_beams(x, items, &touched);
      for (int32_t i = 0; i < x.hi - x.lo; ++i)
        if (touched[i]) ++slot_cnt[m.perm[x.lo + i]];
    }
    const int32_t slots = S > 0 ? *std::max_element(slot_cnt.begin(), slot_cnt.end()) : 0;
    return kMergeFixedUs + kMergeSlotUs * slots;
  };
  // Whether the templates' partial states outgrow the library's own scratch
  // array (counted in whole rows, with room for the two arrays' alignment).
  const double state_bytes = shape.head_dim * (shape.kv_bytes == 4 ? 4.0 : 2.0) + 4 * kPartMl;
  auto outgrows = [&](double rows_per_head) {
    return rows_per_head * hkv * state_bytes + 512 > static_cast<double>(kScratchBytes);
  };
  auto rows_of = [&](const std::vector<Tmpl>& t) {
    double rows = 0;
    for (const Tmpl& x : t) rows += static_cast<double>(x.hi - x.lo) * g;
    return rows;
  };
  auto over = [&](const std::vector<Tmpl>& t) { return outgrows(rows_of(t)); };
  // One search at the current RW: fills tm and the plan's target, work and
  // chaining; returns the modelled time.
  auto search = [&]() {
    double est = -1;
    double work = 0;
    for (const NItem& it : items)
      if (!(it.flags & kEntExt)) work += cm.narrow_block_us();
    for (int32_t s = 0; s < nseg; ++s)
      if (wide[s])
        work += m.seg_nblocks[s] * (cm.f32 ? tiles_of((m.seg_beam_end[s] - m.seg_beam_begin[s]) * g) * cm.f32_tile_us()
                                           : cm.wide_block_us(RW * g));
    work = work * hkv / nbins;
    P.work_us = work;
    P.chained = false;
    const bool small = work < kSmallWorkUs;
    fit_units = small ? few_units : all_units;
    if (warm && warm->target_us > 0 && warm->work_us > 0) {
      // Warm re-plan: the earlier target, scaled with the work, raised while
      // its units outnumber the workgroups (unless that plan was chained);
      // one placement, no search.
      double T = target0 + (warm->target_us - target0) * (work / warm->work_us);
      T = std::max(T, target0 + 1e-3);
      if (!warm->chained)
        for (int it = 0; it < 12 && units_at(T) > fit_units; ++it) T = target0 + 1.15 * (T - target0);
      units_at(T);
      P.target_us = T;
      P.chained = warm->chained;
      return 0.0;
    }
    // Upper bound of the bisection: a few times the average work per unit,
    // raised while the units do not fit (one entry of many rows can cost
    // more than that bound by its row term alone).
    double base = work;
    double hi = target0 + 4.0 * work + 4.0;
    for (int it = 0; it < 6 && units_at(hi) > fit_units; ++it) hi *= 2.0;
    const bool fits = static_cast<int32_t>(tm.size()) <= fit_units;
    if (fits) {
      double lo = target0;
      for (int it = 0; it < 12; ++it) {
        const double mid = 0.5 * (lo + hi);
        if (units_at(mid) <= fit_units)
          hi = mid;
        else
          lo = mid;
      }
      base = hi - target0;
    }
    std::vector<Tmpl> cand;
    auto try_target = [&](double T) {
      make_templates(T, cand);
      if (small && static_cast<int32_t>(cand.size()) > fit_units && 4 * S < all_units && est >= 0) return;
      const double e = place(cand, nullptr) + merge_us(cand);
      const bool fit = P.few_states && !over(cand), had_fit = P.few_states && !over(tm);
      if (est >= 0 && (fit != had_fit ? had_fit : e >= est)) return;
      est = e;
      P.chained = static_cast<int32_t>(cand.size()) * hkv > nbins;
      tm.swap(cand);
      P.target_us = T;
    };
    if (fits)
      for (double f : {1.0, 0.5, 0.6, 0.75, 1.15, 1.3, 1.5, 1.75, 2.0, 2.5, 3.0, 4.0}) try_target(target0 + f * base);
    else
      for (double f : {0.35, 0.5, 0.65, 0.8, 1.0, 1.2, 1.45, 1.75, 2.1, 2.5, 3.0, 4.0}) try_target(target0 + f * base);
    return est;
  };

  // Row caps of wide and of narrow units; the model picks, and a second
  // choice has to model faster by the model's own error (kCapGain).
  // * A streaming batch takes narrow units of up to 32 rows (one wave group;
  //   straggler batch 86 us per call against 92 to 100 with 64 rows) and wide
  //   units of up to 128, or of up to 256 where that models faster (long
  //   chain 289 us per call with 256-row units, 302 with 192, 325 with 128).
  // * Other batches take narrow units of up to 64 rows (7B 64-beam tree 23.1
  //   us per call against 24.2 with 32) and wide units of up to 192 rows, or
  //   256.
  // * fp32 caches try 64, 32 and 16 rows: streaming tails are fastest in one
  //   or two wave groups (28 heads of 4, 4 requests of 5 beams of 8k tokens:
  //   125 us per call against 166 to 176 with 64 rows), heavy segments in
  //   units of 64 rows (verification of three tokens, 2 x 24 beams: 429
  //   against 535 with 32).
  // A warm re-plan keeps the earlier plan's caps.
  // Smaller units write more partial states. The call that keeps them in the
  // library's scratch array refuses a plan that outgrows it, so a plan that
  // does is replaced by one of larger units where that fits (512 to 3072
  // beams: up to 1.3 times the bytes without this rule). Callers with a
  // workspace of their own lose nothing by it: of five batches of 1,920 to
  // 3,072 beams, 202, 246, 258, 173 and 234 us per call with the larger units
  // and 227, 268, 277, 228 and 242 with those they replace.
  auto set_caps = [&](int32_t wide_rows, int32_t narrow_rows) {
    P.wide_rows = wide_rows;
    P.narrow_rows = narrow_rows;
    RB = narrow_beams(narrow_rows);
    RW = wide_beams(wide_rows);
    list_items();
  };
  // The same larger units are weighed wherever many units are chained to a
  // workgroup (237 requests of 8 beams, 7B shape: 107 us per call against
  // 121; 44 of 48 beams, 14 heads of 2: 69 against 77).
  // A warm re-plan keeps the choice too, unless the other one would now fit
  // (judged by few_ratio): a batch that shrank gets its fastest plan back,
  // and one whose plan outgrows the array is planned anew where larger units
  // may fit.
  if (warm && warm->target_us > 0 && warm->work_us > 0 && warm->wide_rows > 0) {
    P.few_units = warm->few_units;
    P.few_states = warm->few_states;
    P.few_ratio = warm->few_ratio;
    set_caps(warm->wide_rows, warm->narrow_rows);
    search();
    const double rows = rows_of(tm);
    const bool anew = P.few_states ? !outgrows(rows / P.few_ratio) || (outgrows(rows) && !outgrows(warm->rows_per_head))
                                   : outgrows(rows) && !outgrows(rows * P.few_ratio);
    if (anew) warm = nullptr;
  } else {
    warm = nullptr;
  }
  if (!warm) {
    P.few_units = P.few_states = false;
    P.few_ratio = 0;
    set_caps(streaming ? kStreamWideRows : kFewWideRows, streaming && wide_mode ? kGroupRows : kMaxRows);
    double best = search();
    // Runs the search at other caps and keeps its plan if keep (of its
    // modelled time) says so, else restores the plan at hand.
    auto try_caps = [&](int32_t wide_rows, int32_t narrow_rows, bool few_units, auto keep) {
      std::vector<Tmpl> tm0 = tm;
      const bool few0 = P.few_units;
      const int32_t wide0 = P.wide_rows, narrow0 = P.narrow_rows;
      const double target0 = P.target_us, work0 = P.work_us;
      const bool chained0 = P.chained;
      P.few_units = few_units;
      set_caps(wide_rows, narrow_rows);
      const double alt = search();
      if (keep(alt)) {
        best = alt;
        return;
      }
      P.few_states = false;
      P.few_units = few0;
      set_caps(wide0, narrow0);
      tm.swap(tm0);
      P.target_us = target0;
      P.work_us = work0;
      P.chained = chained0;
    };
    // (A cap under which every segment is cut into as many chunks as under
    // the other gives the same plan.)
    bool chunks_differ = false;
    const int32_t most = wide_beams(kMaxWideRows);
    for (int32_t s = 0; s < nseg && wide_mode; ++s) {
      const int32_t G = m.seg_beam_end[s] - m.seg_beam_begin[s];
      if (wide[s] && (G + RW - 1) / RW != (G + most - 1) / most) chunks_differ = true;
    }
    if (chunks_differ) try_caps(kMaxWideRows, P.narrow_rows, false, [&](double us) { return us < kCapGain * best; });
    for (int32_t rows : {kGroupRows, kGroupRows / 2})
      if (cm.f32) try_caps(P.wide_rows, rows, false, [&](double us) { return us < kCapGain * best; });
    // Long chains of units: fewer, larger ones where they model faster with
    // what the model leaves out per unit of a chain.
    const double chain = static_cast<double>(tm.size()) * hkv / nbins;
    if (wide_mode && streaming && chain > kLongChain)
      try_caps(kMaxWideRows, kMaxRows, true, [&](double us) {
        return us + kChainUnitUs * tm.size() * hkv / nbins < best + kChainUnitUs * chain;
      });
    if (over(tm)) {
      const double rows = rows_of(tm);
      P.few_states = true;
      try_caps(kMaxWideRows, kMaxRows, true, [&](double) {
        P.few_ratio = rows_of(tm) / rows;
        return !over(tm);
      });
    }
  }

  std::vector<std::vector<Work>> bins;
  place(tm, &bins);

  // ---- partial rows and merge lists ----------------------------------------
  std::vector<int32_t> prow0(tm.size());
  std::vector<std::vector<int32_t>> per_beam(S);
  int32_t rows = 0;
  for (size_t t = 0; t < tm.size(); ++t) {
    prow0[t] = rows;
    const int32_t nb = tm[t].hi - tm[t].lo;
    std::vector<char> touched;
    touched_beams(tm[t], items, &touched);
    for (int32_t i = 0; i < nb; ++i)
      if (touched[i]) per_beam[m.perm[tm[t].lo + i]].push_back(rows + i * g);
    rows += nb * g;
  }
  P.rows_per_head = rows;
  P.slot_off.assign(S + 1, 0);
  for (int32_t b = 0; b < S; ++b) P.slot_off[b + 1] = P.slot_off[b] + static_cast<int32_t>(per_beam[b].size());
  P.slot_rows.reserve(P.slot_off[S]);
  for (int32_t b = 0; b < S; ++b) P.slot_rows.insert(P.slot_rows.end(), per_beam[b].begin(), per_beam[b].end());
  P.num_slots = static_cast<int64_t>(P.slot_rows.size());
  size_t most = 0;
  for (const auto& v : per_beam) most = std::max(most, v.size());
  P.slot_stride = static_cast<int32_t>((most + 1 + 15) / 16 * 16);
  P.slot_tab.assign(static_cast<size_t>(S) * P.slot_stride, 0);
  for (int32_t b = 0; b < S; ++b) {
    int32_t* row = P.slot_tab.data() + static_cast<size_t>(b) * P.slot_stride;
    row[0] = static_cast<int32_t>(per_beam[b].size());
    std::copy(per_beam[b].begin(), per_beam[b].end(), row + 1);
  }

  // ---- records ---------------------------------------------------------------
  // Waves of the first of a narrow unit's two wave groups (UnitRec::mode;
  // rows 0 .. 31 and the rest, for fp32 caches 0 .. 15): in proportion to
  // the block entries with rows of each group.
  auto first_group_waves = [&](const Tmpl& t, const Entries& x) {
    const int32_t cut = wide_mode ? kGroupRows : kGroupRows / 2;
    int32_t c0 = 0, c1 = 0;
    for (size_t k = 0; t.mode == kModeNarrow && k < x.ids.size(); ++k) {
      if (x.info[k] & kEntExt) continue;
      const int32_t r0 = x.info[k] & 63, r1 = ((x.info[k] >> 6) & 63) + 1;
      c0 += r0 < cut;
      c1 += r1 > cut;
    }
    const int32_t n = c0 + c1 > 0 ? (kUnitWaves * c0 + (c0 + c1) / 2) / (c0 + c1) : kUnitWaves / 2;
    return std::min(kUnitWaves - 1, std::max(1, n));
  };
  Entries x;
  auto make_rec = [&](const Work& w) {
    UnitRec r{};
    const Tmpl& t = tm[w.t];
    write_entries(t, &x);
    r.kvh = w.kvh;
    r.nrows = (t.hi - t.lo) * g;
    r.nstatic = x.nstatic;
    r.nent = static_cast<int32_t>(x.ids.size());
    r.prow0 = prow0[w.t];
    r.next = -1;
    r.mode = t.mode | first_group_waves(t, x) << 8;
    for (int32_t i = 0; i < t.hi - t.lo; ++i) r.beams[i] = m.perm[t.lo + i];
    // First window: entries [0, n1); second window: the rest.
    const size_t n1 = x.ids.size() - static_cast<size_t>(t.mode == kModeWide ? std::max(0, x.nstatic - kMaxEntries)
                                                                                : x.nstatic2);
    r.nstatic2 = static_cast<int32_t>(x.ids.size() - n1);
    if (t.mode == kModeNarrow) r.nent = static_cast<int32_t>(n1);
    if (r.nstatic2 > 0) P.two_windows = true;
    for (size_t k = 0; k < x.ids.size(); ++k) {
      if (k < n1) {
        r.ent_id[k] = x.ids[k];
        r.ent_info[k] = x.info[k];
      } else {
        r.ent_id2[k - n1] = x.ids[k];
        r.ent_info2[k - n1] = x.info[k];
      }
    }
    return r;
  };
  P.recs.assign(nbins, UnitRec{});
  for (int32_t k = 0; k < nbins; ++k) P.recs[k].next = -1;
  for (int32_t k = 0; k < nbins; ++k) {
    int32_t prev = -1;
    for (size_t i = 0; i < bins[k].size(); ++i) {
      int32_t idx;
      if (i == 0) {
        idx = k;
        P.recs[k] = make_rec(bins[k][i]);
      } else {
        idx = static_cast<int32_t>(P.recs.size());
        P.recs.push_back(make_rec(bins[k][i]));
      }
      if (prev >= 0) P.recs[prev].next = idx;
      prev = idx;
      P.num_units++;
    }
  }
}

}  // namespace tts
