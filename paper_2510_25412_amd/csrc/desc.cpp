// Batch-descriptor builder (host, integer work only).  See desc.hpp.
#include "desc.hpp"

#include <algorithm>
#include <cstring>

#include "../../include/symphony_kv.h"

namespace symkv {

namespace {
// How many steps over its keys one tile of a batch should take at most, when few tiles would leave compute units idle or a
// long one would be the batch's tail.  lens: (steps of a tile, number of such tiles).  A batch of `rounds` workgroups per
// slot, all of b steps, ends after rounds * (b + start) steps; b is the smallest size with which the pieces fit into that many
// slots.  Cutting costs a partial result per row and chunk and a merge launch (`merge` steps).  0 = leave the tiles whole.
// bf16, 32 query / 8 kv heads, whole calls cut / whole: 512 tokens on 8000: 102 / 276 us; 64 on 60 000: 100 / 1820; 32 on
// 2000: 25 / 61; three prompts of 100..700 on 200..4000: 76 / 117; 1024 on nothing: 43 / 53; 512 on nothing stays whole
// (36.1 / 35.5).
// beside: work of other kinds in the same launch, in steps: nothing ends before the chip has done all of it.  per_piece: partials that a piece
// of a cut tile leaves at most; all pieces leave no more than `budget`.
int64_t chunk_steps(const std::vector<std::pair<int32_t, int32_t>>& lens, int64_t slots, int64_t start, int64_t merge, int64_t max_chunks, int64_t unit,
                    int64_t beside, int64_t per_piece, int64_t budget) {
  int64_t n = 0, longest = 0, total = 0;
  for (auto& t : lens) {
    n += t.second;
    longest = std::max<int64_t>(longest, t.first);
    total += (int64_t)t.first * t.second;
  }
  if (n == 0 || n > 3 * slots) return 0;
  const int64_t rounds0 = (n + slots - 1) / slots;
  int64_t best = rounds0 == 1 ? longest + start : std::max(longest + start, std::min(rounds0 * (longest + start), total / slots + rounds0 * start + longest / 2));
  best = std::max(best, (total + beside) / slots);
  best -= best / 8;                              // a cut has to promise an eighth
  int64_t b_best = 0;
  int64_t pieces = 0, partials = 0;
  auto cut = [&](int64_t b) {
    pieces = partials = 0;
    for (auto& t : lens) {
      const int64_t nc = (t.first + b - 1) / b;
      pieces += nc * t.second;
      if (nc > 1) partials += nc * t.second * per_piece;
    }
  };
  for (int64_t rounds = rounds0; rounds <= rounds0 + 2; ++rounds) {
    int64_t lo = (longest + max_chunks - 1) / max_chunks, hi = longest;       // smallest b in [lo, hi] whose pieces fit
    lo = std::max((lo + unit - 1) / unit, (int64_t)1);
    hi = std::max((hi + unit - 1) / unit, lo);
    while (lo < hi) {
      const int64_t mid = (lo + hi) / 2;
      cut(mid * unit);
      if (pieces <= rounds * slots && partials <= budget) hi = mid;
      else lo = mid + 1;
    }
    if (lo * unit >= longest) continue;          // whole tiles
    const int64_t est = std::max(rounds * (lo * unit + start), (total + beside) / slots) + merge;
    if (est < best) {
      best = est;
      b_best = lo * unit;
    }
  }
  return b_best;
}
// Longest range (pages) that a small decode batch leaves to one workgroup of four wavefronts, and to one of eight.  Per layer, 32 query
// heads, cut at four pages per wavefront and merged / whole: 32 files of 100 tokens 13.6 / 9.1 us, sixteen of 200 12.8 / 9.7, eight of
// 300 12.5 / 10.6, one of 400 12.1 / 12.2; whole ranges of eight wavefronts, 1..14 files of 400..510 tokens, 0.69..0.85 of such a cut.
// Against a cut at one or two pages per wavefront, as longer ranges have it, a single file of 500 tokens is slower whole (13.6 / 9.2 us):
// the lines are where they were for the coarser cut, and have not been weighed against the finer one over numbers of files and heads.
constexpr int64_t kWholePages = 24, kWholePagesWide = 32;
// A small batch of long ranges is cut finer than min_units only where that saves more in the layers of the step than the longer plan
// costs once (1 to 4 us of planning and upload).  Matrix cores: layers x query columns (heads x tokens of a row) x kSpreadUnits reach the
// pages of the batch.  Vector units: layers x query heads per kv head, the work per page, reach kSpreadLayers or a 16th of the pages.
// Whole steps, four pages per wavefront / the finer cut: 1 head per kv head, 10 files of 600 tokens on 2 kv heads, 1 layer 18.9 / 21.7
// us, 4 layers 46.8 / 50.5, 16 layers 133.7 / 130.8; 4 heads, a file of 1000 tokens on 8 kv heads 17.9 / 20.0, 2 layers 29.4 / 31.3, 3 layers
// 41.0 / 39.0, 4 layers 53.2 / 47.3, on 1 kv head 2 layers, alone, 43.3 / 39.8; 8 heads, 600 tokens on 8 kv heads 19.1 / 18.3, 2000 tokens
// 19.5 / 20.1, four of 900 20.3 / 22.5; 4 tokens of 4 heads on 700 19.9 / 18.7, on four of 900 21.0 / 22.7, 4 layers 73.2 / 71.6.
constexpr int64_t kSpreadLayers = 12, kSpreadUnits = 64;
// bf16 tiles, in steps of a 32-key block: what the start and the end of a tile cost, and the merge launch.  196 random prompt batches
// whose plan some setting changes, attention and merge together, against whole tiles: 0.82 of the time, one more than 4 % slower (6 %).  A
// start of 6: 0.81, five slower, by up to 12 %; a merge of 8: 0.79, ten slower.
// Units (token, kv head, page) of decode rows that take as long as a step: 111 batches of prompts beside 4..224 decode files 0.652 of
// the time with whole tiles, three slower, by up to 12 % (3: 0.653, three; 6: 0.653, five; not counted: 0.654, thirteen, by up to 44 %: two
// prompts of 64 tokens beside 200 files of 1000..3000 tokens 292 us whole, 421 cut).
constexpr int64_t kTileStart = 10, kTileMerge = 11, kUnitsPerStep = 4;
// A segment record, and what is added to get from a kv head's to the next one's (plus G in S_QROW).
typedef int32_t SegRecord __attribute__((vector_size(SEG_WORDS * sizeof(int32_t))));
constexpr SegRecord kNextHead = {0, 1, 0, 0, 0, 0, 0, 0};
// A row tile's record.
typedef int32_t RtileRecord __attribute__((vector_size(RTILE_WORDS * sizeof(int32_t))));
// Most key chunks of a row tile: a token's chunks are merged one group of four after the other.  Kernel time over 525 shapes (4..200
// new tokens on 0..8000) against 64: 0.985 (16: 0.986); one file of 8000 tokens, 8 new ones, 8 heads: 24.7 -> 18.5 us.
constexpr int64_t kRowTileChunks = 32;
// With 8 query heads per kv head: fewest (token, kv head, page) units of a batch that go to row tiles, if a file has more pages than this.
constexpr int64_t kRowTileUnits = 2048, kRowTilePages = 24;
}  // namespace

int build_desc(const DescParams& prm, int32_t n_lips, const int32_t* n_tokens, const int64_t* len_after,
               const int32_t* const* tables, BatchDesc* out) {
  const int32_t P = prm.page_tokens, H = prm.n_kv_heads, G = prm.n_q_heads / H;
  // Row tiles, unless there is little to do on long files with 8 heads per kv head: such a tile has 4 tokens in two column tiles, so a
  // page costs it twice the matrix instructions for half the sharing, and few tiles leave the chip idle.  Whole calls, tiles /
  // rows, 8 heads per kv head, files of 500 tokens on: 1.05..1.15 up to 2047 units (token, kv head, page), 0.92 from there to 16 000,
  // then 0.7 and less; files of up to 250 tokens 0.85 (fewer heads: 0.9 and less at any size).
  bool row_tiles = prm.row_tile_rows > 0;
  if (row_tiles && G == 8) {
    int64_t units = 0, longest = 0;
    for (int32_t b = 0; b < n_lips; ++b)
      if (n_tokens[b] >= prm.prefill_min) {
        const int64_t pages = (len_after[b] + P - 1) / P;
        units += std::min(pages, kRowTileUnits) * std::min<int64_t>(n_tokens[b], kRowTileUnits) * H;
        longest = std::max(longest, pages);
      }
    row_tiles = units >= kRowTileUnits || longest <= kRowTilePages;
  }
  auto is_rtile = [&](int32_t b) { return row_tiles && n_tokens[b] >= prm.prefill_min; };
  auto is_prefill = [&](int32_t b) { return (prm.tile_tokens > 0 && n_tokens[b] >= prm.prefill_min) || is_rtile(b); };   // no decode rows
  // Tiles of a batch with prefill chunks have prm.tile_tokens new tokens (256 query rows by default:
  // eight wavefronts share one staging of K/V); a batch whose only tiles are shared prefixes (few
  // members per group) keeps 128-row tiles, two workgroups per CU.
  bool any_prefill = false;
  for (int32_t b = 0; b < n_lips && !any_prefill; ++b) any_prefill = n_tokens[b] >= 1 && is_prefill(b) && !is_rtile(b);
  const int32_t TQ = any_prefill ? prm.tile_tokens : std::min(prm.tile_tokens, 128 / G);
  // A decode row holds up to RT consecutive new tokens of one LIP (a short draft to verify):
  // they share one pass over the file's pages.
  const int32_t RT = std::max(1, std::min(prm.row_tokens, (int32_t)ROW_TOKENS_MAX));
  int32_t max_nt = 1;
  int64_t n_rows = 0, entries = 0, n_tiles = 0, n_tok_total = 0, n_rrows = 0;
  auto& rorder = out->rtile_order;
  rorder.clear();
  for (int32_t b = 0; b < n_lips; ++b) {
    if (n_tokens[b] < 1 || len_after[b] < n_tokens[b] || len_after[b] > (int64_t)0x7fffffff) return SYM_EINVAL;
    if (is_rtile(b)) {
      n_rrows += n_tokens[b];
      rorder.push_back(b);
    } else if (is_prefill(b)) n_tiles += (int64_t)((n_tokens[b] + TQ - 1) / TQ) * H;
    else {
      n_rows += (n_tokens[b] + RT - 1) / RT;
      max_nt = std::max(max_nt, std::min(RT, n_tokens[b]));
    }
    n_tok_total += n_tokens[b];
    entries += (len_after[b] + P - 1) / P;
  }
  if (n_tok_total > 0x7fffffff / (2 * H) || entries > 0x3fffffff || n_tiles > 0x0fffffff) return SYM_EINVAL;

  // ---- sharing groups: single-token LIPs whose files begin with the same pages.  Same page id
  // means same bytes, so the group's common FULL pages can be read once for all members.
  std::vector<int32_t>& share_start = out->share_start;   // per LIP: pages covered by the group (0 = none)
  std::vector<int32_t>& share_base = out->share_base;     // per LIP: first shared partial of its member tile
  std::vector<int32_t>& share_k = out->share_k;           // per LIP: members in its tile
  std::vector<int32_t>& share_ml = out->share_ml;         // per LIP: its index among them
  std::vector<int32_t>& share_nc = out->share_nc;         // per LIP: key chunks of the common prefix
  std::vector<int32_t>& member_rows = out->member_rows;   // q rows of the members, tile after tile
  std::vector<int32_t>& stiles = out->shared_tiles;       // (first lip, member offset, K, C, NC, partial base) per member tile
  share_start.assign(n_lips, 0);
  share_base.assign(n_lips, 0);
  share_k.assign(n_lips, 0);
  share_ml.assign(n_lips, 0);
  share_nc.assign(n_lips, 0);
  member_rows.clear();
  stiles.clear();
  int64_t n_shared_partials = 0, n_shared_tiles = 0;
  // Partial slots: a wave boundary cuts one (row, head), whose two pieces leave a partial per token
  // of the row; the rest is split between the prefix partials of sharing groups and the
  // members' own ranges (one partial per (member, head), never more than the former).
  const int64_t shared_budget = std::max<int64_t>(0, ((int64_t)prm.max_partials - 2 * (int64_t)RT * prm.max_waves) / 2);
  int64_t one_round = 0;                                    // workgroups that tiles and bins together may have (0: no matter)
  const int32_t tile_lips = TQ;                             // members of a shared-prefix tile (rows = members x G)
  if (prm.share_min_lips > 0 && tile_lips > 0) {
    auto& cand = out->by_first_page;
    cand.clear();
    std::vector<int32_t>& qrow_of = out->qrow_of;            // token index of each LIP's first row
    qrow_of.resize(n_lips);
    int64_t tok = 0;
    for (int32_t b = 0; b < n_lips; tok += n_tokens[b], ++b) {
      qrow_of[b] = (int32_t)tok;
      if (n_tokens[b] == 1 && (len_after[b] - 1) / P >= prm.share_min_pages) cand.emplace_back(tables[b][0], b);
    }
    std::sort(cand.begin(), cand.end());
    // First pass: groups and their common page counts (the second pass sizes the key chunks).
    // Files that start with the same page are candidates; inside such a run, take the first
    // unassigned file as representative, measure how many leading pages every other one has in
    // common with it (limited to full pages), and keep the k closest files that maximise the
    // pages saved, (k - 1) * common pages.  Files left over get another round among themselves.
    auto& groups = out->groups;                               // (offset into grp_members, count, C) triples
    auto& gm = out->grp_members;
    auto& lcp = out->lcp;                                     // (common pages, index into cand) of the round
    groups.clear();
    gm.clear();
    int64_t base_tiles = 0;
    for (size_t lo = 0; lo < cand.size();) {
      size_t hi = lo + 1;
      while (hi < cand.size() && cand[hi].first == cand[lo].first) ++hi;
      size_t left = hi - lo;                                  // unassigned files of the run
      for (size_t rep = lo; rep < hi && (int32_t)left >= prm.share_min_lips; ++rep) {
        if (cand[rep].first < 0) continue;                    // already assigned
        const int32_t b0 = cand[rep].second;
        const int64_t full0 = (len_after[b0] - 1) / P;        // full pages of the file before the call
        lcp.clear();
        for (size_t i = rep; i < hi; ++i) {
          if (cand[i].first < 0) continue;
          const int32_t b = cand[i].second;
          const int64_t lim = std::min<int64_t>(full0, (len_after[b] - 1) / P);
          const int32_t* t = tables[b];
          const int64_t c = i == rep ? lim : std::mismatch(t, t + lim, tables[b0]).first - t;
          lcp.emplace_back((int32_t)(c & ~(int64_t)1), (int32_t)i);      // whole 32-token blocks
        }
        std::sort(lcp.begin(), lcp.end(), [](const std::pair<int32_t, int32_t>& x, const std::pair<int32_t, int32_t>& y) {
          return x.first != y.first ? x.first > y.first : x.second < y.second;
        });
        int64_t best = 0;
        size_t best_k = 0;
        for (size_t k = (size_t)prm.share_min_lips; k <= lcp.size(); ++k) {
          const int64_t c = lcp[k - 1].first;
          if (c < prm.share_min_pages) break;
          if ((int64_t)(k - 1) * c > best) {
            best = (int64_t)(k - 1) * c;
            best_k = k;
          }
        }
        if (best_k == 0) {                                    // nothing worth sharing with this file
          cand[rep].first = -1;
          --left;
          continue;
        }
        const int32_t C = lcp[best_k - 1].first;
        std::sort(lcp.begin(), lcp.begin() + best_k, [](const std::pair<int32_t, int32_t>& x, const std::pair<int32_t, int32_t>& y) { return x.second < y.second; });
        groups.insert(groups.end(), {(int32_t)gm.size(), (int32_t)best_k, C});
        for (size_t k = 0; k < best_k; ++k) {
          gm.push_back(cand[lcp[k].second].second);
          cand[lcp[k].second].first = -1;
        }
        left -= best_k;
        base_tiles += (int64_t)((best_k + tile_lips - 1) / tile_lips) * H;
      }
      lo = hi;
    }
    if (!groups.empty()) {
      int64_t target = std::max(1, prm.share_tiles);          // default 512: about two workgroups per CU
      // Tiles and the bins of the members' own pages (workgroups of four, two per compute unit) in one round, where whole chunks
      // leave neither of them more than 15 % above its share: a second round starts with a memory latency of its own.  512 tiles
      // and 512 bins / in one round: 16 roots x 16 members, 2048 tokens shared and up to 256 own, 80.0 / 70.0 us (1 head per kv head
      // 67.8 / 61.0); 8 x 24 on 1000 51.4 / 44.5; 9 x 24 on 2200 79.9 / 61.7; 10 x 20 on 4000 89.3 / 74.0.  At 25..31 % of imbalance, 16 query
      // heads, 4 to 7 % slower.
      int64_t tile_units = 0, own_units = 0;
      for (size_t gi = 0; gi < groups.size(); gi += 3) {
        tile_units += (int64_t)((groups[gi + 1] + tile_lips - 1) / tile_lips) * groups[gi + 2] * H;
        own_units -= (int64_t)groups[gi + 1] * groups[gi + 2] * H;
      }
      bool prompts = false;
      for (int32_t b = 0; b < n_lips; ++b) {
        prompts |= is_prefill(b);
        own_units += (len_after[b] + P - 1) / P * H;
      }
      const int64_t round = 2 * (int64_t)prm.cus, bins_then = std::min<int64_t>(own_units / (4 * (int64_t)prm.min_units_per_wave) + 1, prm.max_waves / 4);
      if (prm.one_round && prm.bin_waves > 0 && max_nt == 1 && !prompts && own_units > 0 &&
          (target + base_tiles - 1) / base_tiles * base_tiles + bins_then > round) {
        const int64_t tiles = std::max<int64_t>(1, (round * tile_units / (tile_units + own_units) + base_tiles / 2) / base_tiles) * base_tiles;
        const int64_t most = (tile_units + own_units) * 115 / 100;      // x 1 / round
        if (tiles < round && tile_units * round <= most * tiles && own_units * round <= most * (round - tiles)) {
          target = std::min(target, tiles);                   // fewer tiles than share_tiles, never more
          one_round = round;
        }
      }
      int32_t nc_want = (int32_t)std::max<int64_t>(1, std::min<int64_t>(8, (target + base_tiles - 1) / base_tiles));
      // every member leaves one partial per kv head and key chunk: the same number of chunks for all groups
      // that the partial slots can hold (not the wanted number for the first groups and none for the last)
      int64_t members_total = 0;
      for (size_t gi = 0; gi < groups.size(); gi += 3) members_total += groups[gi + 1];
      nc_want = (int32_t)std::max<int64_t>(1, std::min<int64_t>(nc_want, shared_budget / std::max<int64_t>(1, members_total * H)));
      for (size_t gi = 0; gi < groups.size(); gi += 3) {
        const int32_t lo = groups[gi], K = groups[gi + 1], C = groups[gi + 2];
        // pages per key chunk are even (whole 32-token blocks): rounding up can leave the last chunks empty
        // (66 pages in 8 chunks of 10: the 8th would be [66, 66)), so the count follows from the size
        auto chunks_of = [C](int32_t n) { const int32_t cp = ((C + n - 1) / n + 1) & ~1; return (C + cp - 1) / cp; };
        int32_t nc = chunks_of(std::max(1, std::min(nc_want, C / 8)));
        while (nc > 1 && n_shared_partials + (int64_t)K * H * nc > shared_budget) nc = chunks_of(nc - 1);   // partial slots must fit
        if (n_shared_partials + (int64_t)K * H * nc > shared_budget) continue;            // no room: plain rows
        for (int32_t i = 0; i < K; i += tile_lips) {
          const int32_t k = std::min(tile_lips, K - i);
          const int32_t moff = (int32_t)member_rows.size();
          for (int32_t j = 0; j < k; ++j) {
            const int32_t b = gm[lo + i + j];
            member_rows.push_back(qrow_of[b]);
            share_start[b] = C;
            share_base[b] = (int32_t)n_shared_partials;
            share_k[b] = k;
            share_ml[b] = j;
            share_nc[b] = nc;
          }
          stiles.insert(stiles.end(), {gm[lo + i], moff, k, C, nc, (int32_t)n_shared_partials});
          n_shared_partials += (int64_t)k * H * nc;
          n_shared_tiles += (int64_t)H * nc;
        }
      }
    }
  }
  n_tiles += n_shared_tiles;

  // ---- row tiles: RQ new tokens of a LIP x one kv head; the workgroup's eight wavefronts take every eighth page each, so a
  // step over the keys is eight pages.  Two workgroups of 512 threads fit on a compute unit.
  const int32_t RQ = std::max(1, prm.row_tile_rows / G);
  // partial slots left for tiles that are cut into key chunks
  int64_t chunk_budget = (int64_t)prm.max_partials - 2 * (int64_t)RT * prm.max_waves - 2 * n_shared_partials;
  int64_t n_rtiles = 0, n_rtile_split = 0, n_chunk_partials = 0, rsteps = 0;
  constexpr int32_t kRowTileWaves = 8;
  auto& rpages = out->rtile_pages;                          // pages every tile reads, file by file in the order of rorder, first tokens first
  auto rchunks = [&](int32_t pages) { return rsteps > 0 ? (pages + (int32_t)rsteps * kRowTileWaves - 1) / ((int32_t)rsteps * kRowTileWaves) : 1; };
  auto count_rtiles = [&]() {
    n_rtiles = n_rtile_split = n_chunk_partials = 0;
    if (rsteps == 0) {                                      // whole tiles
      n_rtiles = (int64_t)rpages.size() * H;
      return;
    }
    const int32_t* pages = rpages.data();
    for (int32_t b : rorder)
      for (int32_t t0 = 0; t0 < n_tokens[b]; t0 += RQ) {
        const int32_t nc = rchunks(*pages++);
        n_rtiles += (int64_t)nc * H;
        if (nc > 1) {
          n_rtile_split += H;
          n_chunk_partials += (int64_t)nc * H * std::min(RQ, n_tokens[b] - t0);
        }
      }
  };
  if (!rorder.empty()) {
    std::stable_sort(rorder.begin(), rorder.end(), [&](int32_t x, int32_t y) { return len_after[x] > len_after[y]; });
    auto& lens = out->tile_lens;
    lens.clear();
    rpages.clear();
    for (int32_t b : rorder) {
      const int64_t len0 = len_after[b] - n_tokens[b];
      int64_t pages = (len0 + P - 1) / P;
      for (int32_t t0 = 0; t0 < n_tokens[b]; t0 += RQ) {
        while (pages * P < len0 + std::min(t0 + RQ, n_tokens[b])) ++pages;
        rpages.push_back((int32_t)pages);
        lens.emplace_back((int32_t)((pages + kRowTileWaves - 1) / kRowTileWaves), H);
      }
    }
    rsteps = chunk_steps(lens, 2 * (int64_t)prm.cus, 4, 4, kRowTileChunks, 1, 0, RQ, chunk_budget);
    count_rtiles();
    chunk_budget -= n_chunk_partials;
  }

  // ---- prefill tiles of a small batch: their keys are cut into chunks until the batch fills the compute units.  A step
  // is a block of 32 keys; a tile of 256 rows has a compute unit to itself, two of 128 rows share one.
  int64_t bsteps = 0, n_btile_split = 0, n_btile_extra = 0, n_btile_partials = 0;
  auto bblocks = [&](int32_t b, int32_t t0) { return (int32_t)((len_after[b] - n_tokens[b] + std::min(t0 + TQ, n_tokens[b]) + 31) / 32); };
  auto bchunks = [&](int32_t blocks) { return bsteps > 0 ? (blocks + (int32_t)bsteps - 1) / (int32_t)bsteps : 1; };
  auto count_btiles = [&]() {
    n_btile_split = n_btile_extra = n_btile_partials = 0;
    if (bsteps == 0) return;
    for (int32_t b = 0; b < n_lips; ++b) {
      if (!is_prefill(b) || is_rtile(b)) continue;
      for (int32_t t0 = 0; t0 < n_tokens[b]; t0 += TQ) {
        const int32_t nc = bchunks(bblocks(b, t0));
        if (nc == 1) continue;
        n_btile_split += H;
        n_btile_extra += (int64_t)(nc - 1) * H;
        n_btile_partials += (int64_t)nc * H * std::min(TQ, n_tokens[b] - t0);
      }
    }
  };
  if (any_prefill) {
    const int64_t slots = (int64_t)prm.cus * (TQ * G == 256 ? 1 : 2);
    if (n_tiles - n_shared_tiles <= 3 * slots) {
      auto& lens = out->tile_lens;
      lens.clear();
      for (int32_t b = 0; b < n_lips; ++b)
        if (is_prefill(b) && !is_rtile(b))
          for (int32_t t0 = 0; t0 < n_tokens[b]; t0 += TQ) lens.emplace_back(bblocks(b, t0), H);
      int64_t units = 0;                                   // decode work in the same launch (plain decode rows)
      for (int32_t b = 0; b < n_lips; ++b)
        if (!is_prefill(b)) units += ((len_after[b] + P - 1) / P - share_start[b]) * H * ((n_tokens[b] + RT - 1) / RT);
      bsteps = chunk_steps(lens, slots, kTileStart, kTileMerge, 64, 3, units / kUnitsPerStep, TQ, chunk_budget);      // tiles of 128 rows walk blocks by threes; for 256 rows pieces of any size measured the same
      count_btiles();
    }
  }

  // ---- units of the decode kernel
  int64_t total_units = 0, longest_range = 0;
  for (int32_t b = 0; b < n_lips; ++b) {
    if (is_prefill(b)) continue;
    for (int32_t i = 0; i < n_tokens[b]; i += RT) {
      const int64_t vis_last = len_after[b] - n_tokens[b] + std::min(i + RT, n_tokens[b]);   // what the row's last token sees
      const int64_t pages = (vis_last + P - 1) / P - share_start[b];
      total_units += pages * H;
      longest_range = std::max(longest_range, pages);
    }
  }
  // bins (whole ranges per workgroup, pieces combined through LDS) for the vector-unit kernel, and for the matrix-core decode
  // kernel (which rows of several tokens need) in a batch without tiles; otherwise its launch takes the global cut
  const bool mfma_bins = prm.mfma_bins && (prm.decode_mfma || max_nt > 1) && n_tiles == 0 && total_units > 0;
  const bool bins = mfma_bins || (prm.bin_waves > 0 && max_nt == 1 && total_units > 0);
  // a bin is a workgroup: eight wavefronts, or four when the launch has tiles of 128 query rows (four-wavefront workgroups)
  // A batch that gives no compute unit more than a workgroup of four: workgroups of four instead of eight, so that twice as many
  // compute units share it, and plain loads.  One compute unit draws about 40 GB/s with nontemporal loads, 60 with plain ones, and
  // that is what bounds such a launch (a page per wavefront: 1.65 us with eight wavefronts, 0.93 with four, 0.68 with plain loads).
  // Per layer, 32 query heads, before / after: a file of 2000 tokens 15.7 / 12.3 us, four of 200 15.6 / 12.2, sixteen of 400
  // 16.9 / 14.5, 64 of 100 18.0 / 15.9; past the line, sixteen of 1000 tokens (8064 units): 21.0 / 22.9.
  const bool small_decode = bins && prm.spread_small && n_tiles == 0 && total_units <= (int64_t)prm.cus * 4 * prm.min_units_per_wave;
  // ... and if there are no more ranges than compute units and all are short, a workgroup per range: nothing is divided between
  // workgroups, so the merge launch is saved, which is worth about four pages of a wavefront's time.
  // (the longer of such ranges need eight wavefronts for it, four pages each)
  const bool whole_wide = small_decode && prm.bin_waves == 8 && n_rows * H <= prm.cus && longest_range > kWholePages && longest_range <= kWholePagesWide;
  const bool whole_small = whole_wide || (small_decode && n_rows * H <= prm.cus && longest_range <= kWholePages);
  const int32_t W = !bins ? 0 : n_tiles > 0 ? (TQ * G != 256 ? 4 : 8) : (prm.bin_waves == 4 || (small_decode && !whole_wide) ? 4 : 8);
  const int64_t max_bins = std::max<int64_t>(1, std::min<int64_t>(prm.max_waves / std::max(W, 1), one_round > 0 && W == 4 ? one_round - n_tiles : prm.max_waves));
  int64_t nw = (total_units + prm.min_units_per_wave - 1) / prm.min_units_per_wave;
  nw = std::max<int64_t>(1, std::min<int64_t>(nw, prm.max_waves));
  if (total_units == 0) nw = 0;
  int64_t n_bins = 0;
  if (bins) {
    // A small batch with long ranges: a wavefront takes as few pages as give every compute unit one workgroup (both of two are in
    // flight from the start), but no fewer than leave a range in the pieces that a merge of four wavefronts reads in one round trip
    // (16), in two where a piece has more than one page and its merge is short (the vector-unit kernel); and two at least on the
    // matrix cores.  32 layers, four pages per wavefront / by this rule: a file of 600 tokens 362 / 298 us, of 1000 361 / 299, of
    // 2000 389 / 354, of 4000 414 / 390; four of 800..1200 400 / 360, eight of 400..700 397 / 381; 2000 tokens with 16 query heads
    // 293 / 272.  Per layer, 4 heads of one kv head, a file of 2000 tokens 12.1 / 10.6, of 4800 12.0 / 11.8; 8 heads of one, 2000
    // tokens 15.1 / 13.8, 2550 tokens 15.1 / 14.2.  Past these lines, two pages against four: 4 heads of one kv head, 8000 tokens
    // 12.6 / 12.2, 24 000 19.6 / 16.5; 8 heads of one, 8000 tokens 18.5 / 16.0, 20 000 26.2 / 19.8; 3 tokens on 20 000 22.2 / 18.0.
    // Short ranges in more than one per compute unit stay at four: there is no latency of a long range to divide.  So does a plan that
    // serves few layers (kSpreadLayers).
    int64_t upw = prm.min_units_per_wave;
    const int64_t gain = (int64_t)prm.layers * G * (mfma_bins ? max_nt : 1);
    if (small_decode && longest_range > kWholePagesWide && (gain * (mfma_bins ? kSpreadUnits : kSpreadUnits / 4) >= total_units || (!mfma_bins && gain >= kSpreadLayers))) {
      const int64_t trip = 16 * W, most = mfma_bins ? trip : 2 * trip;
      int64_t fewest = (longest_range + most - 1) / most;
      if (mfma_bins || longest_range > trip) fewest = std::max<int64_t>(fewest, 2);
      upw = std::min(upw, std::max(fewest, (total_units + prm.cus * 4 - 1) / (prm.cus * 4)));
    }
    // No more wavefronts than the batch's cost has steps: the starts of the cut (plan B) are then apart, and no wavefront without a
    // page begins inside a range.  (With the default settings a wavefront's share never falls below one.)
    n_bins = std::min((total_units + upw * W - 1) / (upw * W), (total_units + (int64_t)prm.range_cost * n_rows * H) / W);
    n_bins = std::max<int64_t>(1, std::min<int64_t>(n_bins, max_bins));
    if (whole_small) n_bins = n_rows * H;
    nw = n_bins * W;
  }
  const int64_t n_members = (int64_t)member_rows.size();

  // A member of a shared-prefix group reads only the pages after the common ones; those are read by
  // the group's tiles through the table of each tile's first member.  So the common pages of every
  // other member stay out of the descriptor (256 forks of 128-page prefixes: 128 KB that would
  // cross PCIe for nothing); its table offset is moved back by the pages left out, so that page
  // index i >= its first own page still finds entry i.
  std::vector<uint8_t>& full_table = out->full_table;
  full_table.assign((size_t)n_lips, 1);
  for (int32_t b = 0; b < n_lips; ++b)
    if (share_start[b] > 0) full_table[b] = 0;
  for (size_t s = 0; s < stiles.size(); s += 6) full_table[stiles[s]] = 1;
  for (int32_t b = 0; b < n_lips; ++b)
    if (!full_table[b]) entries -= share_start[b];

  // ---- rows, planned before the allocation (the bins are made of them)
  std::vector<int32_t>& rows_tmp = out->rows_tmp;
  rows_tmp.resize((size_t)n_rows * ROW_WORDS);
  out->fused.assign((size_t)n_lips, 0);
  int32_t n_fused = 0;
  {
    int64_t r = 0, e = 0, tok = 0;
    for (int32_t b = 0; b < n_lips; ++b) {
      const int64_t skip = full_table[b] ? 0 : share_start[b];
      const int64_t e_lip = e - skip;
      e += (len_after[b] + P - 1) / P - skip;
      if (!is_prefill(b)) {
        for (int32_t i = 0; i < n_tokens[b]; i += RT, ++r) {
          const int32_t nt = std::min(RT, n_tokens[b] - i);
          rows_tmp[r * ROW_WORDS + 0] = (int32_t)e_lip;                                    // page-table offset
          rows_tmp[r * ROW_WORDS + 1] = (int32_t)(len_after[b] - n_tokens[b] + i + 1);   // tokens the row's first token sees
          rows_tmp[r * ROW_WORDS + 2] = (int32_t)(tok + i);                               // q / out row of its first token
          rows_tmp[r * ROW_WORDS + 3] = share_start[b] | ((nt - 1) << ROW_NT_SHIFT);      // first page of the row's own range; tokens - 1
        }
        // the attention kernel can append a LIP's token itself when it is the LIP's only one (nobody else reads it in this launch)
        if (bins && !mfma_bins && prm.fuse_append && n_tokens[b] == 1) {
          out->fused[b] = 1;
          ++n_fused;
        }
      }
      tok += n_tokens[b];
    }
  }
  out->row_lip.clear();
  if (bins && n_fused > 0) {
    out->row_lip.reserve((size_t)n_rows);
    for (int32_t b = 0; b < n_lips; ++b)
      if (!is_prefill(b))
        for (int32_t i = 0; i < n_tokens[b]; i += RT) out->row_lip.push_back(b);
  }
  auto trow_nt = [&](int64_t rr) { return (rows_tmp[rr * ROW_WORDS + 3] >> ROW_NT_SHIFT) + 1; };
  auto trow_pages = [&](int64_t rr) { return (rows_tmp[rr * ROW_WORDS + 1] + trow_nt(rr) - 1 + P - 1) / P; };   // pages its last token sees
  auto trow_first = [&](int64_t rr) { return rows_tmp[rr * ROW_WORDS + 3] & ROW_PAGE_MASK; };

  // record of kv head 0 of a row as one segment, destination the output
  auto seg_record = [&](int64_t row) {
    const int32_t* rw = rows_tmp.data() + row * ROW_WORDS;
    const int32_t app = (!out->row_lip.empty() && out->fused[out->row_lip[row]]) ? (rw[1] - 1) % P : -1;
    return SegRecord{rw[0], rw[3] & ~ROW_PAGE_MASK, trow_first(row), trow_pages(row), rw[1], rw[2] * prm.n_q_heads, -1, app};
  };

  // ---- bins: segments (whole ranges, or pieces of ranges too long for a bin), handed to the bins longest first
  std::vector<int32_t>& seg_tmp = out->seg_tmp;          // SEG_WORDS per segment, in (row, head, page) order
  std::vector<int32_t>& item_bin = out->item_bin;        // bin of every segment
  int64_t n_segs = 0, n_split_partials = 0, n_split_merge = 0;
  bool whole = false;                                    // every range is one segment, in the bin that item_bin says
  const int64_t alpha = prm.range_cost;
  if (bins) {
    const int64_t total_cost = total_units + alpha * n_rows * H;
    auto& order = out->item_order;
    auto& heap = out->bin_heap;
    // no more segments than ranges and cuts at bin boundaries; the vectors only ever grow
    const size_t seg_cap = (size_t)(n_rows * H + n_bins + 1);
    if (seg_tmp.size() < seg_cap * SEG_WORDS) seg_tmp.resize(seg_cap * SEG_WORDS);
    if (item_bin.size() < (size_t)(n_rows * H)) item_bin.resize((size_t)(n_rows * H));
    auto emit = [&](SegRecord rec, int32_t pb, int32_t pe) {
      if (pe != rec[S_PE]) rec[S_APPEND] = -1;
      rec[S_PB] = pb;
      rec[S_PE] = pe;
      std::memcpy(seg_tmp.data() + n_segs++ * SEG_WORDS, &rec, sizeof rec);
    };
    // Plan A, when there are several ranges per bin (short files, the members of forked prefixes): whole ranges, handed to
    // the bins longest first; nothing is split, so no range leaves partials in device memory because of the bins.  Only the
    // bin of every range is found here; the records are written straight into the descriptor, bin by bin, further down (planning
    // 256 files of 100..260 tokens, 8 kv heads: 35 -> 25 us; 16 x 16 forks 55 -> 44; one-page ranges of 147 files 15.6 -> 10).
    bool planned = false;
    if (whole_small || n_rows * H >= 3 * n_bins) {
      int32_t longest = 0, shortest = 0x7fffffff;
      auto& own = out->row_pages;                              // pages of every row's own range
      own.resize((size_t)n_rows);
      for (int64_t row = 0; row < n_rows; ++row) {
        own[row] = trow_pages(row) - trow_first(row);
        longest = std::max(longest, own[row]);
        shortest = std::min(shortest, own[row]);
      }
      int64_t worst = 0;
      if (longest == shortest) {                               // of one length: neighbours together, which is the cheapest to write down
        const int64_t n = n_rows * H, per = n / n_bins, more = n % n_bins;      // `more` bins get one range more
        int32_t* bin_of = item_bin.data();
        for (int64_t b = 0; b < n_bins; ++b)
          for (int64_t i = 0; i < per + (b < more); ++i) *bin_of++ = (int32_t)b;
        worst = (per + (more > 0)) * std::max<int64_t>(1, longest + alpha);
      } else {
        // longest first by counting sort on the page count (rows come in, the H ranges of a row are equal)
        order.assign((size_t)longest + 2, 0);                  // order[c] = rows with more than c pages, after the prefix sum
        for (int64_t row = 0; row < n_rows; ++row) ++order[longest - own[row] + 1];
        for (int32_t c = 0; c <= longest; ++c) order[c + 1] += order[c];
        auto& sorted = out->tile_tmp;                            // rows, longest first (scratch that the tile list reuses later)
        sorted.resize((size_t)n_rows);
        for (int64_t row = 0; row < n_rows; ++row) sorted[order[longest - own[row]]++] = (int32_t)row;
        // The bin of least load, the lowest of equals, takes the next range.  Loads are small whole numbers: one bit per bin and
        // load says which bins carry it, and the least load only rises.  Ranges of one length come together, so where a word of
        // bins has no more members than ranges are left, they are all served at once, lowest first.
        const int64_t max_load = total_cost / n_bins + longest + alpha + 1, wpl = (n_bins + 63) / 64;
        if (max_load * wpl <= (1 << 16)) {
          auto& bits = out->bin_bits;
          auto& cnt = out->bin_count;
          bits.assign((size_t)((max_load + 1) * wpl), 0);
          cnt.assign((size_t)max_load + 1, 0);
          for (int64_t b = 0; b < n_bins; ++b) bits[b >> 6] |= 1ull << (b & 63);
          cnt[0] = (int32_t)n_bins;
          int64_t lo = 0, word = 0;
          for (int64_t i = 0; i < n_rows;) {
            const int32_t pages = own[sorted[i]];
            const int64_t c = std::max<int64_t>(1, pages + alpha);
            int64_t j = i + 1;                                   // rows i .. j are of one length
            while (j < n_rows && own[sorted[j]] == pages) ++j;
            int32_t row = sorted[i], g = 0;                      // the range that is next
            for (int64_t left = (j - i) * H; left > 0;) {
              if (cnt[lo] == 0) {
                while (cnt[lo] == 0) ++lo;
                word = 0;
              }
              uint64_t* from = bits.data() + lo * wpl;
              while (!from[word]) ++word;
              uint64_t set = from[word];
              int32_t n = __builtin_popcountll(set);
              if (n > left) {                                    // the lowest `left` of them
                n = (int32_t)left;
                uint64_t rest = set;
                for (int32_t k = 0; k < n; ++k) rest &= rest - 1;
                set ^= rest;
              }
              from[word] ^= set;
              bits[(lo + c) * wpl + word] |= set;
              cnt[lo] -= n;
              cnt[lo + c] += n;
              worst = std::max(worst, lo + c);
              left -= n;
              for (; set; set &= set - 1) {
                item_bin[(size_t)row * H + g] = (int32_t)(word * 64 + __builtin_ctzll(set));
                if (++g == H) {
                  g = 0;
                  if (++i < j) row = sorted[i];
                }
              }
            }
            i = j;
          }
        } else {
          heap.clear();
          for (int64_t b = 0; b < n_bins; ++b) heap.emplace_back(0, (int32_t)b);
          auto worse = [](const std::pair<int64_t, int32_t>& x, const std::pair<int64_t, int32_t>& y) { return x > y; };   // min-heap on (load, bin)
          for (int32_t row : sorted) {
            const int64_t c = own[row] + alpha;
            for (int32_t g = 0; g < H; ++g) {
              std::pop_heap(heap.begin(), heap.end(), worse);
              heap.back().first += c;
              item_bin[(size_t)row * H + g] = heap.back().second;
              worst = std::max(worst, heap.back().first);
              std::push_heap(heap.begin(), heap.end(), worse);
            }
          }
        }
      }
      planned = whole = whole_small || worst * n_bins * 100 <= total_cost * (100 + prm.bin_tolerance);
    }
    // One bin (a small batch): every range is a segment of it, cut between its wavefronts only.
    if (!planned && n_bins == 1) {
      planned = whole = true;
      std::fill(item_bin.begin(), item_bin.begin() + n_rows * H, 0);
    }
    if (whole) {
      n_segs = n_rows * H;
      for (int64_t row = 0; row < n_rows; ++row)
        if (trow_first(row) > 0) n_split_partials += H;        // the members of a shared prefix always leave partials
      n_split_merge = n_split_partials;
    }
    // Plan B: the units in (row, head, page) order are cut into n_bins * W contiguous ranges of equal cost, one per wavefront,
    // exactly like the global cut (on a virtual axis where every range occupies range_cost + pages, wavefront k starts at
    // total * k / (n_bins * W); a start inside the overhead part of a range snaps to its first page), and every W consecutive
    // wavefronts are a bin.  A range that a BIN boundary divides becomes one segment per part, each leaving a partial in
    // device memory (at most n_bins - 1 ranges); what the wavefront boundaries inside a bin divide is combined through LDS.
    if (!planned) {
      out->wave_pos.resize((size_t)nw * 3);              // (segment, page, units before it) where every wavefront starts
      auto& seg_end = out->bin_first;                    // first segment of every bin
      seg_end.assign((size_t)n_bins + 1, 0);
      int32_t* wpos = out->wave_pos.data();
      int64_t k = 0, vstart = 0, cut = 0;                // cut: where wavefront k starts, total_cost * k / nw ...
      const int64_t step = total_cost / nw, over = total_cost % nw;
      int64_t rem = 0, units_before = 0;                 // ... and what that leaves: total_cost * k % nw
      SegRecord next_head = kNextHead;
      next_head[S_QROW] = G;
      for (int64_t row = 0; row < n_rows; ++row) {
        SegRecord rec = seg_record(row);
        const int32_t np = rec[S_PE], p0 = rec[S_PB];
        for (int32_t g = 0; g < H; ++g, rec += next_head) {
          const int64_t vend = vstart + alpha + (np - p0);
          const size_t first_seg = (size_t)n_segs;
          int32_t pb = p0;
          while (k < nw && cut < vend) {
            const int32_t at = p0 + (int32_t)std::max<int64_t>(0, cut - vstart - alpha);
            if (k % W == 0) {                            // a bin begins here
              if (at > pb) {
                emit(rec, pb, at);
                pb = at;
              }
              seg_end[k / W] = (int32_t)n_segs;
            }
            wpos[0] = (int32_t)n_segs;                   // the segment that is emitted next holds page `at`
            wpos[1] = at;
            wpos[2] = (int32_t)(uint32_t)(units_before + at - p0);      // (differences of neighbours count, modulo 2^32)
            wpos += 3;
            ++k;
            cut += step;
            if ((rem += over) >= nw) {
              rem -= nw;
              ++cut;
            }
          }
          emit(rec, pb, np);
          const size_t n_here = (size_t)n_segs - first_seg;
          if (n_here > 1 || p0 > 0) {
            const int32_t nt = trow_nt(row);             // a part leaves one partial per token of the row
            for (size_t i = 0; i < n_here; ++i) seg_tmp[(first_seg + i) * SEG_WORDS + S_DEST] = (int32_t)(n_split_partials + i * nt);
            n_split_partials += (int64_t)n_here * nt;
            n_split_merge += nt;
          }
          vstart = vend;
          units_before += np - p0;
        }
      }
      seg_end[n_bins] = (int32_t)n_segs;
    }
  }

  const int64_t off_rows = DESC_HEADER_WORDS;
  const int64_t off_waves = off_rows + (n_rows + n_rrows) * ROW_WORDS;      // the rows of row tiles follow the decode rows
  const int64_t off_merge = off_waves + nw * WAVE_WORDS;
  // a merge entry per token of a cut (row, head) (at most one cut per wave boundary) and per (member row, head)
  // (a cut (row, head) has a wave boundary inside it, and there are no more of them than (row, head)s);
  // with bins: one per (row, head) that is split between bins or belongs to a shared prefix
  const int64_t merge_cap = bins ? n_split_merge : std::min<int64_t>(nw, n_rows * H) * max_nt + n_members * H;
  const int64_t off_pt = off_merge + merge_cap * MERGE_WORDS;
  const int64_t off_ptoff = off_pt + entries;
  const int64_t off_tiles = off_ptoff + n_lips + 1;
  {
    // words without and with the tiles' chunks (a tile record and a place in the order table each, a merge entry per tile)
    const int64_t base = off_tiles + n_tiles * TILE_WORDS + n_members + (bins ? (n_segs + 2) * SEG_WORDS + n_bins * LMERGE_WORDS : 0) +
                         ((bins && n_tiles > 0) ? n_tiles + (n_bins + 7) / 8 : 0);
    if (rsteps > 0 && base + n_rtiles * RTILE_WORDS + n_rtile_split * TMERGE_WORDS > prm.max_words) {
      rsteps = 0;                                 // no room for the chunks: whole tiles
      count_rtiles();
    }
    if (bsteps > 0 && base + n_btile_extra * (TILE_WORDS + 1) + n_btile_split * TMERGE_WORDS > prm.max_words) {
      bsteps = 0;
      count_btiles();
    }
    n_tiles += n_btile_extra;
  }
  const int64_t off_members = off_tiles + n_tiles * TILE_WORDS;
  const int64_t off_segs = off_members + n_members;
  const int64_t off_lmerge = off_segs + (bins ? (n_segs + 2) * SEG_WORDS : 0);       // two spare records: the kernel looks ahead
  // the order table of a launch with tiles and bins: a word per group of 8 workgroups (no more tile groups than tiles)
  const int64_t off_groups = off_lmerge + (bins ? n_bins * LMERGE_WORDS : 0);
  const int64_t groups_cap = (bins && n_tiles > 0) ? n_tiles + (n_bins + 7) / 8 : 0;
  const int64_t off_rtiles = off_groups + groups_cap;
  const int64_t off_tmerge = off_rtiles + n_rtiles * RTILE_WORDS;
  const int64_t total = off_tmerge + (n_rtile_split + n_btile_split) * TMERGE_WORDS;
  if (total > 0x7fffffff) return SYM_EINVAL;
  int32_t* const w = out->alloc ? out->alloc(total) : nullptr;   // the caller's buffer (pinned staging memory on the GPU path)
  if (!w) return SYM_ENOSPC;
  out->words = w;
  out->n_words = total;
  std::memset(w, 0, DESC_HEADER_WORDS * sizeof(int32_t));

  // ---- rows, prefill tiles, page table
  int32_t* rows = w + off_rows;
  int32_t* pt = w + off_pt;
  int32_t* ptoff = w + off_ptoff;
  int32_t* tiles = w + off_tiles;
  int64_t e = 0, tok = 0, ti = 0;
  int32_t n_tmerge = 0, tmerge_tokens = 0;                // tiles cut into key chunks
  int32_t* tm_next = w + off_tmerge;
  int64_t n_btile_done = 0;                               // partials handed to chunks of prefill tiles so far
  std::vector<int32_t>& tok_of = out->qrow_of;             // token index of each LIP's first row
  tok_of.resize(n_lips);
  for (int32_t b = 0; b < n_lips; ++b) {
    tok_of[b] = (int32_t)tok;
    const int64_t skip = full_table[b] ? 0 : share_start[b];      // leading pages left out (see above)
    const int64_t e_lip = e - skip;
    ptoff[b] = (int32_t)e_lip;
    int64_t np = (len_after[b] + P - 1) / P;
    if (np > skip) std::memcpy(pt + e, tables[b] + skip, (size_t)(np - skip) * sizeof(int32_t));
    e += np - skip;
    if (is_prefill(b) && !is_rtile(b)) {
      // order (kv head, token tile): the tiles that read the same K/V are neighbours
      for (int32_t g = 0; g < H; ++g)
        for (int32_t t0 = 0; t0 < n_tokens[b]; t0 += TQ) {
          const int32_t blocks = bblocks(b, t0), nc = bchunks(blocks), per = ((blocks + nc - 1) / nc + 2) / 3 * 3;
          const int32_t count = std::min<int32_t>(TQ, n_tokens[b] - t0);
          for (int32_t c = 0; c < nc; ++c, ++ti) {
            int32_t* t = tiles + ti * TILE_WORDS;
            std::memset(t, 0, TILE_WORDS * sizeof(int32_t));
            t[T_TBL] = (int32_t)e_lip;                                // page-table offset
            t[T_LEN] = (int32_t)(len_after[b] - n_tokens[b]);         // file length before the call
            t[T_QROW] = (int32_t)(tok + t0);                          // q / out row of the tile's first token
            t[T_COUNT] = count;                                       // tokens in the tile
            t[T_HEAD] = g;
            t[T_AUX] = t0;                                            // token offset inside the chunk
            t[T_KIND] = nc > 1 ? TILE_CHUNK : TILE_PREFILL;
            if (nc > 1) {
              t[T_PAGE0] = 2 * std::min(c * per, blocks);
              t[T_PAGE1] = 2 * std::min((c + 1) * per, blocks);
              t[T_DEST] = (int32_t)(n_btile_done + (int64_t)c * count);      // + the first of these partials, added below
            }
          }
          if (nc > 1) {
            tm_next[TM_FIRST] = (int32_t)n_btile_done;
            tm_next[TM_CHUNKS] = nc;
            tm_next[TM_COUNT] = count;
            tm_next[TM_QROW] = (int32_t)(tok + t0) * prm.n_q_heads + g * G;
            tm_next += TMERGE_WORDS;
            ++n_tmerge;
            tmerge_tokens = std::max(tmerge_tokens, count);
            n_btile_done += (int64_t)nc * count;
          }
        }
    }
    tok += n_tokens[b];
  }
  ptoff[n_lips] = (int32_t)e;
  if (n_rows > 0) std::memcpy(rows, rows_tmp.data(), (size_t)n_rows * ROW_WORDS * sizeof(int32_t));

  // ---- cut the unit sequence into nw ranges of equal cost; number the partial results.
  // Cost of a range = its units + range_cost per (row, head) it starts in (the end-of-range
  // combine and the restart of the pipeline are not free).  On a virtual axis where every
  // (row, head) occupies range_cost + pages, wave k ends at total * (k+1) / nw; a cut that
  // falls into the overhead part of a (row, head) snaps to its first page.
  int32_t* waves = w + off_waves;
  int32_t* merge = w + off_merge;
  auto row_nt = [&](int64_t rr) { return (rows[rr * ROW_WORDS + 3] >> ROW_NT_SHIFT) + 1; };
  auto row_pages = [&](int64_t rr) { return (rows[rr * ROW_WORDS + 1] + row_nt(rr) - 1 + P - 1) / P; };   // pages its last token sees
  auto row_first = [&](int64_t rr) { return rows[rr * ROW_WORDS + 3] & ROW_PAGE_MASK; };
  int32_t part = 0;
  int32_t n_merge = 0;        // (row, head) ranges that need a merge
  if (bins) {
    // ---- bins: segment list bin by bin, wave records, in-bin merge lists, merge entries of split ranges
    int32_t* segs = w + off_segs;
    int32_t* lmerge = w + off_lmerge;
    std::memset(lmerge, 0, (size_t)n_bins * LMERGE_WORDS * sizeof(int32_t));
    auto& first = out->bin_first;                         // first segment of every bin in the final order
    auto& bin_units = out->bin_units;                     // units of every bin of whole ranges
    if (whole) {                                          // (row, head, page) order is kept inside a bin
      first.assign((size_t)n_bins + 1, 0);
      for (int64_t i = 0; i < n_segs; ++i) ++first[item_bin[i] + 1];
      for (int64_t b = 0; b < n_bins; ++b) first[b + 1] += first[b];
      auto& pos = out->item_order;                        // reused: next free place of every bin
      pos.assign(first.begin(), first.end() - 1);
      bin_units.assign((size_t)n_bins, 0);
      for (int64_t row = 0; row < n_rows; ++row) {
        SegRecord rec = seg_record(row);
        const int32_t units = rec[S_PE] - rec[S_PB], qh = rec[S_QROW];
        const int32_t dest = rec[S_PB] > 0 ? n_merge : -1;      // a member of a shared prefix leaves a partial and has a merge entry
        rec[S_DEST] = dest;
        SegRecord next_head = kNextHead;
        next_head[S_QROW] = G;
        next_head[S_DEST] = dest < 0 ? 0 : 1;
        const int32_t* bin_of = item_bin.data() + (size_t)row * H;
        for (int32_t g = 0; g < H; ++g, rec += next_head) {
          const int32_t bin = bin_of[g];
          bin_units[bin] += units;
          std::memcpy(segs + (int64_t)pos[bin]++ * SEG_WORDS, &rec, sizeof rec);
        }
        for (int32_t g = 0; g < H && dest >= 0; ++g) {
          int32_t* it = merge + (int64_t)n_merge++ * MERGE_WORDS;
          std::memset(it, 0, MERGE_WORDS * sizeof(int32_t));
          it[0] = dest + g;
          it[1] = 1;
          it[2] = qh + g * G;
          it[6] = 1;
        }
      }
    } else {
      std::memcpy(segs, seg_tmp.data(), (size_t)n_segs * SEG_WORDS * sizeof(int32_t));      // bins are contiguous
    }
    std::memset(segs + n_segs * SEG_WORDS, 0, 2 * SEG_WORDS * sizeof(int32_t));
    // merge entries of the ranges that leave partials, in (row, head) order = the order of their partial numbers
    for (int64_t i = 0; i < n_segs && !whole; ++i) {
      const int32_t* sg = seg_tmp.data() + i * SEG_WORDS;
      if (sg[S_DEST] < 0) continue;
      const bool first_piece = i == 0 || sg[-SEG_WORDS + S_DEST] < 0 || sg[-SEG_WORDS + S_QROW] != sg[S_QROW];
      const int32_t nt = (sg[S_HEAD] >> ROW_NT_SHIFT) + 1;
      if (first_piece)
        for (int32_t t = 0; t < nt; ++t) {
          int32_t* it = merge + (int64_t)n_merge++ * MERGE_WORDS;
          std::memset(it, 0, MERGE_WORDS * sizeof(int32_t));
          it[0] = sg[S_DEST] + t;
          it[2] = sg[S_QROW] + t * prm.n_q_heads;
          it[6] = nt;                                     // distance between the token's pieces
        }
      for (int32_t t = 0; t < nt; ++t) ++merge[(int64_t)(n_merge - 1 - t) * MERGE_WORDS + 1];
    }
    part = (int32_t)n_split_partials;
    // Inside a bin the wavefronts cut the bin's segments like the global cut does the batch: on a virtual axis where every
    // segment occupies range_cost + pages, wavefront k of the Wb that get work starts at total * k / Wb (snapped to the
    // segment's first page inside the overhead part).  Wb <= pages of the bin, so no two cuts fall on one page and the
    // pieces of a cut segment lie in consecutive wavefronts.  A piece that is not its whole segment goes to an LDS slot:
    // 2 * wavefront for a wavefront's first piece, 2 * wavefront + 1 for its last; the list of cut segments (segment,
    // slot of the first piece, its wavefront, pieces) tells the workgroup what to combine when all are done.
    for (int64_t b = 0; b < n_bins; ++b) {
      const int64_t s0 = first[b], s1 = first[b + 1];
      int32_t* bw = waves + b * W * WAVE_WORDS;
      std::memset(bw, 0, (size_t)W * WAVE_WORDS * sizeof(int32_t));
      int32_t* lm = lmerge + b * LMERGE_WORDS;
      lm[1] = (int32_t)s0;                              // the bin's segments
      lm[2] = (int32_t)s1;
      int64_t Wb = W, total;                            // wavefronts that get work; units of the bin (plan B: of the batch up to its end)
      if (whole) {
        total = bin_units[b];
        Wb = std::min<int64_t>(W, total);
        if (Wb == 0) continue;
        const int64_t vt = total + alpha * (s1 - s0), step = vt / Wb, over = vt - step * Wb;
        int64_t k = 0, vstart = 0, units = 0, cut = 0, rem = 0;      // wavefront k starts at cut = vt * k / Wb, rem = vt * k % Wb
        for (int64_t i = s0; i < s1 && k < Wb; ++i) {
          const int32_t pb = segs[i * SEG_WORDS + S_PB], n = segs[i * SEG_WORDS + S_PE] - pb;
          const int64_t vend = vstart + alpha + n;
          while (k < Wb && cut < vend) {
            int32_t* ww = bw + k * WAVE_WORDS;
            const int32_t in = (int32_t)std::max<int64_t>(0, cut - vstart - alpha);
            ww[0] = (int32_t)i;
            ww[1] = pb + in;
            ww[2] = (int32_t)(uint32_t)(units + in);    // units before it, for now
            ++k;
            cut += step;
            if ((rem += over) >= Wb) {
              rem -= Wb;
              ++cut;
            }
          }
          vstart = vend;
          units += n;
        }
      } else {                                          // the wavefronts' starts come from the cut of the whole batch
        const int32_t* wp = out->wave_pos.data() + b * W * 3;
        for (int64_t k = 0; k < W; ++k) std::memcpy(bw + k * WAVE_WORDS, wp + 3 * k, 3 * sizeof(int32_t));
        total = b + 1 < n_bins ? (uint32_t)wp[3 * W + 2] : total_units;
      }
      for (int64_t k = 0; k < Wb; ++k) {
        int32_t* ww = bw + k * WAVE_WORDS;
        const int32_t* sg = segs + (int64_t)ww[0] * SEG_WORDS;
        const int32_t p = ww[1], last = sg[S_PE] - 1;
        const int32_t* ids = pt + sg[S_TBL];            // of the first pages: their loads need no table lookup
        for (int t = 0; t < 3; ++t) ww[4 + t] = ids[std::min(p + t, last)];
        ww[7] = sg[S_HEAD];
        ww[2] = (int32_t)((k + 1 < Wb ? (uint32_t)ww[WAVE_WORDS + 2] : (uint32_t)total) - (uint32_t)ww[2]);
        if (p == sg[S_PB]) continue;
        // it continues a segment: of the wavefront before it, whose last piece is either the segment's first or continues it too
        const int32_t* wb = ww - WAVE_WORDS;
        if (wb[0] != ww[0] || wb[1] == sg[S_PB]) {
          int32_t* en = lm + 4 + 4 * lm[0]++;
          en[0] = ww[0];
          en[1] = (int32_t)(wb[0] == ww[0] ? 2 * (k - 1) : 2 * (k - 1) + 1);
          en[2] = (int32_t)(k - 1);
          en[3] = 1;
        }
        ++lm[4 + 4 * (lm[0] - 1) + 3];
      }
    }
  } else {
    const int64_t vtotal = total_units + alpha * n_rows * H;
    {
      int64_t k = 0, vstart = 0;     // next boundary to place; virtual start of the current (row, head)
      for (int64_t row = 0; row < n_rows && k < nw; ++row) {
        const int32_t np = row_pages(row), p0 = row_first(row);
        for (int32_t g = 0; g < H && k < nw; ++g) {
          const int64_t vend = vstart + alpha + (np - p0);
          while (k < nw && vtotal * k / nw < vend) {
            const int64_t o = vtotal * k / nw - vstart;
            int32_t* ww = waves + k * WAVE_WORDS;
            ww[0] = (int32_t)row;
            ww[1] = g;
            ww[2] = p0 + (int32_t)std::max<int64_t>(0, o - alpha);
            ++k;
          }
          vstart = vend;
        }
      }
    }
    for (int64_t k = 0; k < nw; ++k) {
      int32_t* ww = waves + k * WAVE_WORDS;
      int64_t row = ww[0];
      int32_t g = ww[1], p = ww[2];
      // the range ends where the next one starts (or at the end of the batch)
      const int64_t erow = k + 1 < nw ? ww[WAVE_WORDS + 0] : n_rows;
      const int32_t eg = k + 1 < nw ? ww[WAVE_WORDS + 1] : 0, ep = k + 1 < nw ? ww[WAVE_WORDS + 2] : 0;
      ww[4] = part;
      {                                   // ids of the first pages: their loads need no table lookup
        const int32_t np0 = row_pages(row);
        const int32_t* t0 = pt + rows[row * ROW_WORDS + 0];
        for (int i = 0; i < 3; ++i) ww[5 + i] = t0[std::min(p + i, np0 - 1)];
      }
      int64_t units = 0;
      while (row < erow || (row == erow && (g < eg || (g == eg && p < ep)))) {
        const int32_t np = row_pages(row), p0 = row_first(row);
        const int32_t cnt = (row == erow && g == eg) ? ep - p : np - p;
        if (!(p == 0 && cnt == np)) {                            // a whole (row, g) needs no partial
          const int32_t nt = row_nt(row);                        // a piece leaves one partial per token of the row
          if (p == p0) {                                         // first piece of this (row, g)
            for (int32_t t = 0; t < nt; ++t, ++n_merge) {
              int32_t* it = merge + (int64_t)n_merge * MERGE_WORDS;
              std::memset(it, 0, MERGE_WORDS * sizeof(int32_t));
              it[0] = part + t;
              it[2] = (rows[row * ROW_WORDS + 2] + t) * prm.n_q_heads + g * G;
              it[6] = nt;                                        // distance between the token's pieces
            }
          }
          for (int32_t t = 0; t < nt; ++t) ++merge[(int64_t)(n_merge - 1 - t) * MERGE_WORDS + 1];
          part += nt;
        }
        units += cnt;
        p += cnt;
        if (p == np) {
          if (++g == H) {
            g = 0;
            ++row;
          }
          p = row < n_rows ? row_first(row) : 0;
        }
      }
      ww[3] = (int32_t)units;
    }

  }

  // ---- shared-prefix tiles and the extra partials of their members' merge entries
  const int32_t shared_base = part;
  int32_t max_shared_rows = 0;
  if (!stiles.empty()) {
    int32_t* members = w + off_members;
    std::memcpy(members, member_rows.data(), member_rows.size() * sizeof(int32_t));
    for (size_t s = 0; s < stiles.size(); s += 6) {
      const int32_t b0 = stiles[s], moff = stiles[s + 1], k = stiles[s + 2], C = stiles[s + 3], nc = stiles[s + 4], base = stiles[s + 5];
      const int32_t cp = ((C + nc - 1) / nc + 1) & ~1;        // pages per key chunk, even
      for (int32_t g = 0; g < H; ++g)
        for (int32_t c = 0; c < nc; ++c, ++ti) {
          int32_t* t = tiles + ti * TILE_WORDS;
          std::memset(t, 0, TILE_WORDS * sizeof(int32_t));
          t[T_TBL] = ptoff[b0];
          t[T_QROW] = moff;                                    // offset into the member list
          t[T_COUNT] = k;
          max_shared_rows = std::max(max_shared_rows, k * G);
          t[T_HEAD] = g;
          t[T_AUX] = shared_base + base + (g * nc + c) * k;    // first partial of this tile
          t[T_KIND] = TILE_SHARED;
          t[T_PAGE0] = std::min(c * cp, C);
          t[T_PAGE1] = std::min((c + 1) * cp, C);
        }
    }
  }
  // ---- row tiles: the longest file first, from its last tokens down (more than the compute units hold at once: the longest piece
  // first, below); the kv heads of a token tile are neighbours, so that with 8 of them (workgroup b runs on XCD b % 8) the tiles that
  // read one (file, kv head) share an L2
  if (n_btile_partials > 0) {                            // the partials of the prefill tiles' chunks follow those of the shared prefixes
    const int32_t first = shared_base + (int32_t)n_shared_partials;
    for (int64_t i = 0; i < n_tiles; ++i)
      if (tiles[i * TILE_WORDS + T_KIND] == TILE_CHUNK) tiles[i * TILE_WORDS + T_DEST] += first;
    for (int32_t i = 0; i < n_tmerge; ++i) w[off_tmerge + (int64_t)i * TMERGE_WORDS + TM_FIRST] += first;
  }
  if (!rorder.empty()) {
    // Two workgroups share a compute unit, and its matrix cores bound the launch.  More workgroups than compute units: pieces go
    // longest first over all files; if all start at once, the second ones of the compute units (handed out in the same order as the
    // first) go shortest first, so that the longest gets the shortest beside it.  Four prompts of 64..512 tokens on new files, 8 heads,
    // file by file / longest first / paired: 32.5 / 28.7 / 26.6 us; three of 400..512 32.5 / 28.0 / 26.1.
    const int64_t pieces = n_rtiles / H, alone = prm.cus / H;
    const bool by_length = n_rtiles > prm.cus, paired = n_rtiles <= 2 * (int64_t)prm.cus;
    auto& place = out->tile_order;                         // per piece length, longest first: place of the next such piece
    if (by_length) {
      int32_t longest = *std::max_element(rpages.begin(), rpages.end());
      if (rsteps > 0) longest = (int32_t)std::min<int64_t>(longest, rsteps * kRowTileWaves);
      place.assign((size_t)longest + 2, 0);
      for (int32_t pages : rpages) {
        if (rsteps == 0) {
          ++place[(size_t)(longest - pages) + 1];
          continue;
        }
        const int32_t nc = rchunks(pages), per = (pages + nc - 1) / nc;
        for (int32_t c = 0; c < nc; ++c) ++place[(size_t)(longest - (std::min((c + 1) * per, pages) - std::min(c * per, pages))) + 1];
      }
      for (int32_t i = 0; i <= longest; ++i) place[i + 1] += place[i];
    }
    const int32_t longest = (int32_t)place.size() - 2;
    int64_t next = 0;
    int32_t* tm = tm_next;
    int64_t chunk_base = shared_base + n_shared_partials + n_btile_partials;
    int32_t* rr = rows + n_rows * ROW_WORDS;
    const int32_t* file_pages = rpages.data();             // of the file's first tile
    for (int32_t b : rorder) {
      const int32_t len0 = (int32_t)(len_after[b] - n_tokens[b]), tok0 = tok_of[b], file_tiles = (n_tokens[b] + RQ - 1) / RQ;
      const int32_t* tile_pages = file_pages + file_tiles;
      file_pages += file_tiles;
      for (int32_t t = 0; t < n_tokens[b]; ++t, rr += ROW_WORDS) {
        rr[0] = ptoff[b];
        rr[1] = len0 + t + 1;
        rr[2] = tok0 + t;
        rr[3] = 0;
      }
      for (int32_t t0 = (file_tiles - 1) * RQ; t0 >= 0; t0 -= RQ) {
        const int32_t count = std::min(RQ, n_tokens[b] - t0), pages = *--tile_pages, nc = rchunks(pages);
        const int32_t per = nc == 1 ? pages : (pages + nc - 1) / nc;
        for (int32_t c = 0; c < nc; ++c) {
          int64_t at = next++;
          if (by_length) {
            at = place[longest - (std::min((c + 1) * per, pages) - std::min(c * per, pages))]++;
            if (paired && at >= alone) at = alone + pieces - 1 - at;
          }
          const int32_t p0 = c * per, p1 = std::min(p0 + per, pages);
          RtileRecord rec = {ptoff[b], len0 + t0 + 1, tok0 + t0, count, 0, std::min(p0, pages), p1, nc > 1 ? (int32_t)(chunk_base + (int64_t)c * count) : -1};
          RtileRecord next_head = {0, 0, 0, 0, 1, 0, 0, nc > 1 ? nc * count : 0};
          int32_t* rt = w + off_rtiles + at * H * RTILE_WORDS;
          for (int32_t g = 0; g < H; ++g, rec += next_head) std::memcpy(rt + g * RTILE_WORDS, &rec, sizeof rec);
        }
        if (nc > 1) {
          for (int32_t g = 0; g < H; ++g, tm += TMERGE_WORDS, ++n_tmerge) {
            tm[TM_FIRST] = (int32_t)(chunk_base + (int64_t)g * nc * count);
            tm[TM_CHUNKS] = nc;
            tm[TM_COUNT] = count;
            tm[TM_QROW] = (tok0 + t0) * prm.n_q_heads + g * G;
          }
          tmerge_tokens = std::max(tmerge_tokens, count);
          chunk_base += (int64_t)nc * H * count;
        }
      }
    }
  }
  // ---- ids of the pages of a tile's first block (the page after its last one stands in by the last)
  for (int64_t i = 0; i < n_tiles; ++i) {
    int32_t* t = tiles + i * TILE_WORDS;
    const int32_t p0 = t[T_KIND] == TILE_PREFILL ? 0 : t[T_PAGE0];
    const int64_t rows_end = ((int64_t)t[T_LEN] + t[T_AUX] + t[T_COUNT] + P - 1) / P;      // pages the tile's last row sees
    const int32_t end = t[T_KIND] == TILE_SHARED ? t[T_PAGE1] : t[T_KIND] == TILE_CHUNK ? (int32_t)std::min<int64_t>(rows_end, t[T_PAGE1]) : (int32_t)rows_end;
    t[T_ID0] = pt[t[T_TBL] + std::min(p0, std::max(end - 1, 0))];
    t[T_ID1] = pt[t[T_TBL] + std::min(p0 + 1, std::max(end - 1, 0))];
  }
  // ---- the tile list in 8 shares of equal cost, one per XCD
  int32_t tile_blocks = 0;
  {
    int32_t* xo = w + H_XCD_OFF;
    for (int x = 0; x <= 8; ++x) xo[x] = 0;
    if (n_tiles > 0) {
      auto cost = [&](const int32_t* t) -> int64_t {
        return t[T_KIND] != TILE_PREFILL ? (t[T_PAGE1] - t[T_PAGE0] + 1) / 2 + 1
                                        : ((int64_t)t[T_LEN] + t[T_AUX] + t[T_COUNT] + 31) / 32 + 1;
      };
      // A batch of prompts whose tiles were cut into chunks fills the chip in a known number of rounds of about equal pieces: shares
      // of equal COUNT, neighbours (same keys) together.  Otherwise, also where shared prefixes (of other lengths, last in the list)
      // are computed beside the pieces, shares of equal cost (48 batches of forks and prompts, attention launch: 0.85 of the time
      // with equal counts; the fork tree of 16 x 16 beside 512 tokens on 8000: 280 -> 154 us):
      // groups = runs of tiles with the same page table and kv head, split so that none exceeds 1/16 of the work
      const bool equal_count = bsteps > 0 && n_shared_tiles == 0;
      int64_t total = 0;
      for (int64_t i = 0; i < n_tiles; ++i) total += cost(tiles + i * TILE_WORDS);
      const int64_t cap = std::max<int64_t>(1, total / 16);
      auto& groups = out->tile_groups;                    // (cost, first tile); the next group's first tile ends it
      groups.clear();
      int64_t acc = 0;
      for (int64_t i = 0; i < n_tiles; ++i) {
        const int32_t* t = tiles + i * TILE_WORDS;
        const bool same = !equal_count && i > 0 && t[T_TBL] == t[-TILE_WORDS + T_TBL] && t[T_HEAD] == t[-TILE_WORDS + T_HEAD] && t[T_KIND] == t[-TILE_WORDS + T_KIND];
        if (!same || acc >= cap) {
          groups.emplace_back(0, (int32_t)i);
          acc = 0;
        }
        acc += cost(t);
        groups.back().first += cost(t);
      }
      const size_t ng = groups.size();
      auto& order = out->tile_order;                      // group indices, heaviest first
      order.resize(ng);
      for (size_t i = 0; i < ng; ++i) order[i] = (int32_t)i;
      if (!equal_count) std::stable_sort(order.begin(), order.end(), [&](int32_t x, int32_t y) { return groups[x].first > groups[y].first; });
      int64_t load[8] = {0, 0, 0, 0, 0, 0, 0, 0};
      std::vector<int32_t> share_of(ng);
      int32_t count[8] = {0, 0, 0, 0, 0, 0, 0, 0};
      for (int32_t gi : order) {
        int best = 0;
        if (equal_count) best = (int)((int64_t)gi * 8 / (int64_t)ng);
        else
          for (int x = 1; x < 8; ++x)
            if (load[x] < load[best]) best = x;
        share_of[gi] = best;
        load[best] += groups[gi].first;
        const int32_t gend = (size_t)gi + 1 < ng ? groups[gi + 1].second : (int32_t)n_tiles;
        count[best] += gend - groups[gi].second;
      }
      for (int x = 0; x < 8; ++x) xo[x + 1] = xo[x] + count[x];
      // rewrite the list share by share (groups in heaviest-first order inside a share)
      auto& tmp = out->tile_tmp;
      tmp.assign(tiles, tiles + n_tiles * TILE_WORDS);
      int32_t pos[8];
      for (int x = 0; x < 8; ++x) pos[x] = xo[x];
      for (int32_t gi : order) {
        const int32_t gend = (size_t)gi + 1 < ng ? groups[gi + 1].second : (int32_t)n_tiles;
        const int32_t n = gend - groups[gi].second;
        std::memcpy(tiles + (int64_t)pos[share_of[gi]] * TILE_WORDS, tmp.data() + (int64_t)groups[gi].second * TILE_WORDS,
                    (size_t)n * TILE_WORDS * sizeof(int32_t));
        pos[share_of[gi]] += n;
      }
      for (int x = 0; x < 8; ++x) tile_blocks = std::max(tile_blocks, 8 * count[x]);
    }
    w[H_TILE_BLOCKS] = tile_blocks;
  }
  if (groups_cap > 0) {
    // Tiles come longest first and decode groups all cost the same.  Default: the decode groups go among the first
    // half of the tile groups, so that some CUs stream K/V from HBM for decode ranges while the others keep the
    // matrix cores busy, and no decode group starts late and becomes the tail of the grid.
    const int64_t T = tile_blocks / 8, D = (n_bins + 7) / 8;
    const int64_t lead = T * std::min(std::max(prm.mix_lead, 0), 100) / 100;
    const int64_t spread = std::min(T - lead, (T * std::min(std::max(prm.mix_spread, 0), 100) + 99) / 100);
    const int64_t gs = spread + D;                       // groups of the mixed stretch
    int32_t* gm = w + off_groups;
    int64_t t = 0, d = 0;
    for (int64_t j = 0; j < T + D; ++j) {
      const int64_t jj = j - lead;
      const bool dec = jj >= 0 && jj < gs && (jj + 1) * D / gs > jj * D / gs;
      gm[j] = dec ? ~(int32_t)d++ : (int32_t)t++;
    }
    w[H_N_GROUPS] = (int32_t)(T + D);
    w[H_OFF_GROUPS] = (int32_t)off_groups;
  }

  // every (member row, head): extra partials first + i * stride, i < count
  if (n_members > 0) {
    // merge entries are sorted by word 2 (q row * Hq + first head), as are the LIPs by q row
    int64_t tk = 0;
    int32_t mi = 0;
    for (int32_t b = 0; b < n_lips; tk += n_tokens[b], ++b) {
      if (share_start[b] == 0) continue;
      for (int32_t g = 0; g < H; ++g) {
        const int32_t key = (int32_t)tk * prm.n_q_heads + g * G;
        while (mi < n_merge && merge[(int64_t)mi * MERGE_WORDS + 2] < key) ++mi;
        int32_t* it = merge + (int64_t)mi * MERGE_WORDS;     // exists: a member row never writes final output itself
        it[3] = shared_base + share_base[b] + g * share_nc[b] * share_k[b] + share_ml[b];
        it[4] = share_k[b];
        it[5] = share_nc[b];
      }
    }
  }
  const int32_t n_partials = shared_base + (int32_t)(n_shared_partials + n_btile_partials + n_chunk_partials);
  if (n_partials > prm.max_partials) return SYM_ENOSPC;

  w[H_N_ROWS] = (int32_t)(n_rows + n_rrows);
  w[H_N_RTILES] = (int32_t)n_rtiles;
  w[H_OFF_RTILES] = (int32_t)off_rtiles;
  w[H_N_TMERGE] = n_tmerge;
  w[H_OFF_TMERGE] = (int32_t)off_tmerge;
  out->n_rtiles = (int32_t)n_rtiles;
  out->n_tmerge = n_tmerge;
  out->tmerge_tokens = tmerge_tokens;
  out->merge_pieces = 0;
  if (n_merge <= kWideMergeItems)                 // (more entries never use it)
    for (int32_t i = 0; i < n_merge; ++i) out->merge_pieces = std::max(out->merge_pieces, merge[(int64_t)i * MERGE_WORDS + 1] + merge[(int64_t)i * MERGE_WORDS + 5]);
  w[H_N_WAVES] = (int32_t)nw;
  w[H_N_PARTIALS] = n_partials;
  w[H_N_LIPS] = n_lips;
  w[H_N_TILES] = (int32_t)n_tiles;
  w[H_N_MERGE] = n_merge;
  w[H_OFF_ROWS] = (int32_t)off_rows;
  w[H_OFF_WAVES] = (int32_t)off_waves;
  w[H_OFF_MERGE] = (int32_t)off_merge;
  w[H_OFF_PT] = (int32_t)off_pt;
  w[H_OFF_PTOFF] = (int32_t)off_ptoff;
  w[H_OFF_TILES] = (int32_t)off_tiles;
  w[H_OFF_MEMBERS] = (int32_t)off_members;
  w[H_N_MEMBERS] = (int32_t)n_members;
  w[H_N_SHARED_TILES] = (int32_t)n_shared_tiles;
  w[H_TOTAL_WORDS] = (int32_t)total;
  w[H_TOTAL_UNITS_LO] = (int32_t)(total_units & 0xffffffff);
  w[H_TOTAL_UNITS_HI] = (int32_t)(total_units >> 32);
  w[H_N_SEGS] = (int32_t)(bins ? n_segs : 0);
  w[H_OFF_SEGS] = (int32_t)off_segs;
  w[H_N_BINS] = (int32_t)n_bins;
  w[H_BIN_WAVES] = W;
  w[H_OFF_LMERGE] = (int32_t)off_lmerge;
  out->n_bins = (int32_t)n_bins;
  out->bin_waves = W;
  out->small_decode = small_decode ? 1 : 0;
  out->n_segs = (int32_t)(bins ? n_segs : 0);
  out->n_fused = n_fused;
  out->n_rows = (int32_t)n_rows;
  out->n_waves = (int32_t)nw;
  out->n_partials = n_partials;
  out->n_merge = n_merge;
  out->n_lips = n_lips;
  out->n_tiles = (int32_t)n_tiles;
  out->total_units = total_units;
  out->max_row_tokens = max_nt;
  out->tile_blocks = tile_blocks;
  out->tile_rows = TQ * G;
  out->small_shared_only = (n_tiles > 0 && !any_prefill && max_shared_rows > 0 && max_shared_rows <= 64) ? 1 : 0;
  return SYM_OK;
}

}  // namespace symkv
