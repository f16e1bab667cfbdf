// Host construction of the split-KV work plan (rule documented in include/libra.h).
#include <algorithm>
#include <array>
#include <cstring>
#include <queue>

#include "internal.h"

namespace libra {
namespace {

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

using Unit = std::array<int32_t, kUnitInts>;

// Rule step 4: split counts that cut the single rows into at most R pieces per KV head
// with the smallest possible largest piece.  Each extra split goes to the row with the
// largest share pages_b / n_b (exact cross-multiplied comparison, ties to the smaller b)
// among the rows that can still be split; a row that cannot be split now never can, as
// only its own split count would change that.  Not balanced when the rows do not fit in R or
// the largest piece exceeds 1.5 times the mean share.  For ascending budgets R: each one's
// splits are those of the one before and some more.
struct Apportionment {
  int64_t R;
  bool balanced = false;
  std::vector<int64_t> n;  // split counts (1 for other rows), if balanced
  int64_t largest = 0;     // pages of the largest piece
};

void one_wave_splits(const std::vector<int64_t>& pages, const std::vector<int64_t>& single,
                     const libra_plan_params& p, std::vector<Apportionment>& budgets) {
  if (single.empty()) return;
  std::vector<int64_t> n(pages.size(), 1);
  auto before = [&](int64_t a, int64_t b) {  // true if row a's share is served after b's
    const int64_t lhs = pages[a] * n[b], rhs = pages[b] * n[a];
    if (lhs != rhs) return lhs < rhs;
    return a > b;
  };
  std::priority_queue<int64_t, std::vector<int64_t>, decltype(before)> heap(before);
  for (int64_t b : single) heap.push(b);
  int64_t total = int64_t(single.size()), sum = 0;
  for (int64_t b : single) sum += pages[b];
  for (Apportionment& a : budgets) {
    if (int64_t(single.size()) > a.R) continue;
    while (total < a.R && !heap.empty()) {
      const int64_t b = heap.top();
      heap.pop();
      if (n[b] >= p.max_splits || pages[b] < (n[b] + 1) * int64_t(p.min_split_pages)) continue;
      ++n[b];
      ++total;
      heap.push(b);
    }
    for (int64_t b : single) a.largest = std::max(a.largest, ceil_div(pages[b], n[b]));
    a.balanced = __int128(2) * a.largest * a.R <= __int128(3) * sum;
    if (a.balanced) a.n = n;
  }
}

// Rule step 11: the units (in step 9's order) are dealt to S slots, each to the slot with
// room that minimises (load + cost) / weight; the r-th unit of slot c is listed at position
// c + r * S.  Slots of one XCD share a weight, so one min-heap of (load, c) per XCD yields
// that XCD's best slot and the eight candidates are compared exactly; this picks the same
// slot as a scan over all of them.
std::vector<Unit> place_on_slots(const std::vector<Unit>& units, const libra_plan_params& p,
                                 int64_t S) {
  const int64_t n = int64_t(units.size());
  auto weight = [&](int64_t c) -> int64_t {
    const int32_t x = p.xcd_weight[c % kNumXcds];
    return x > 0 ? x : 1000;
  };
  auto cap = [&](int64_t c) { return c < n ? (n - 1 - c) / S + 1 : int64_t(0); };
  using Entry = std::pair<int64_t, int64_t>;  // (load, slot)
  bool equal = true;
  for (int x = 1; x < kNumXcds; ++x) equal = equal && weight(x) == weight(0);
  const int nheaps = equal ? 1 : kNumXcds;  // equal weights: the least (load, slot) of all
  std::array<std::priority_queue<Entry, std::vector<Entry>, std::greater<Entry>>, kNumXcds> heaps;
  for (int64_t c = 0; c < std::min(S, n); ++c) heaps[size_t(c % nheaps)].push({0, c});
  std::vector<int64_t> taken(size_t(std::min(S, n)), 0);
  std::vector<Unit> out(units.size());
  for (const Unit& u : units) {
    const int64_t cost = ceil_div(u[U_KV1], kPage) - u[U_KV0] / kPage;
    int best = -1;
    Entry be{0, 0};
    for (int k = 0; k < nheaps; ++k) {
      if (heaps[k].empty()) continue;
      const Entry e = heaps[k].top();
      if (best >= 0) {
        const __int128 lhs = __int128(e.first + cost) * weight(be.second);
        const __int128 rhs = __int128(be.first + cost) * weight(e.second);
        if (lhs > rhs || (lhs == rhs && e.second > be.second)) continue;
      }
      best = k;
      be = e;
    }
    heaps[best].pop();
    const int64_t c = be.second;
    out[size_t(c + taken[c] * S)] = u;
    if (++taken[c] < cap(c)) heaps[best].push({be.first + cost, c});
  }
  return out;
}

size_t place(size_t& off, size_t bytes) {
  const size_t at = off;
  off = align256(off + bytes);
  return at;
}

// Places the tables and the single rows' partial results in the workspace.
void workspace_layout(Plan& P) {
  size_t off = 0;
  P.off_units = place(off, size_t(P.info.n_units) * kUnitInts * sizeof(int32_t));
  P.off_writes = place(off, P.writes.size() * sizeof(int32_t));
  P.off_merges = place(off, size_t(P.info.n_merge_groups) * kMergeInts * sizeof(int32_t));
  P.upload_bytes = off;
  const size_t rows = size_t(P.info.n_partial_slots) * size_t(P.group);
  P.off_part_o = place(off, rows * kDim * sizeof(float));
  P.off_part_lse = place(off, rows * sizeof(float));
  P.ws_bytes = std::max<size_t>(off, 256);
}

// Places the tables of Q's fine tiles and their chunk_slots partial results (of kTileRows
// rows) behind the workspace of the plan it is a form of.
void fine_layout(Plan& Q, const Plan& P, int64_t chunk_slots) {
  Q.base = &P;
  Q.off_units = P.off_units;
  Q.off_writes = P.off_writes;
  Q.off_merges = P.off_merges;
  Q.off_part_o = P.off_part_o;
  Q.off_part_lse = P.off_part_lse;
  size_t off = P.ws_bytes;
  Q.upload_off = off;
  Q.off_tiles = place(off, Q.tiles.size() * sizeof(int32_t));
  Q.off_chunk_merges = place(off, Q.chunk_merges.size() * sizeof(int32_t));
  Q.upload_bytes = off - Q.upload_off;
  const size_t rows = size_t(chunk_slots) * kTileRows;
  Q.off_chunk_o = place(off, rows * kDim * sizeof(float));
  Q.off_chunk_lse = place(off, rows * sizeof(float));
  Q.ws_bytes = off;
}

// A plan of the same batch, whose tables and launch are still to be set.
std::unique_ptr<Plan> sibling(const Plan& P) {
  auto Q = std::make_unique<Plan>();
  Q->mode = P.mode;
  Q->batch = P.batch;
  Q->num_q_heads = P.num_q_heads;
  Q->num_kv_heads = P.num_kv_heads;
  Q->group = P.group;
  Q->params = P.params;
  Q->info = P.info;
  Q->pages_needed = P.pages_needed;
  return Q;
}

// Chooses the form of the chunk launch: chunk units on workgroups of kChunkRows rows (eight
// waves, one per CU), or fine tiles of kTileRows rows (four waves, two workgroups per CU)
// where that is faster.  Whole fine tiles in many waves are the halves of the units, in their
// queues' order, read from the unit table, with a list of them where some units have only one;
// those of a single wave, whose keys may be split, get records of their own.  Built without a
// record for each of many thousand tiles, a plan costs the host about what one of units does
// (80 prompts of 510 tokens 154 us as units, 158 as halves, 314 with records).
// single_pages: pages of the decode rows beside them, over the KV heads; longest_queue: units
// of the longest queue.
//
// At most S = 2 num_cus fine tiles are resident at once and their longest sets the launch's
// time, so their keys may be split as well: into ceil(steps / t) near-equal ranges, t being
// the smallest piece (at least kMinPieceSteps) for which the pieces fit in S.  The pieces
// write float32 partials, which a merge combines.  The forms are compared by the times
// below, in 10 ns, measured over appends of 8 to 1,600 tokens to 1 to 128 requests (256 CUs):
// * a 64-key step of a wide workgroup takes 1.25 us while half of the CUs are idle, 1.67 us
//   when all are busy, and a workgroup 8-9 us besides (dispatch, first loads, stores); CUs
//   whose unit is short are idle towards the end, so half of the units count by their length
//   (236 of unequal lengths, at most 20,500 keys, 457 us, cut tiles 528 us);
// * a 32-key step of a fine tile takes 0.65 us alone on a CU and 0.93-0.96 us beside
//   another, a tile 3.5 us of its CU besides (7 us by itself), a split launch and its merge
//   13 us more (496 tokens on 431, at most 29 steps: 25 us whole, 35 us split in four).
// So full tiles in many waves stay wide from about 12 steps on (20 prompts of 2,040 tokens
// 974 us against 984 us, 10 of 4,080 1,642 and 1,716 us, 40,960-token prefill 13.8 and
// 15.0 ms), and fine tiles take shorter ones (80 prompts of 510 tokens 470 us against 515 us,
// 16 of 230-911 99 and 109 us) and query tiles of at most 128 rows (128 x 20 tokens on 2,000,
// 4 heads per KV head: 218 and 266 us); over 140 appends of 8-1,024 tokens to 4-128 requests
// whose modelled times differ by less than 12%, the form chosen takes 0.3% more than the
// better one on average, at most 4%.  Launches that leave CUs idle are cut (333 tokens on
// 16,001: 129 and 326 us; 800 on 16,000: 267 and 340 us; 4 x 8 on 30,000: 54 and 583 us).
// Decode rows run beside the chunk launch, which is dispatched first: they take about 330 ns
// per page of a CU, start up to 12 us later (the fork) and find the share of the CUs that the
// chunk workgroups leave, so a form ends after max(t, lag + decode + t * share it fills).  A
// fine tile shares its CU with them (steps of 0.65 us become 0.93 us meanwhile), a wide
// workgroup's LDS keeps them off.  Tiles cut to fill the chip then only pay where whole units
// would outlast the decode rows, and where units would not, they are taken up to 5% above, as
// their CUs serve the decode rows' last wave better.  Such a call also takes the host 45-50 us
// (fork and join), and the launch that merges cut tiles 5 more, so what ends before is not cut
// (4 x 26 tokens on 330 beside 12 rows 45.7 us, cut 51.3 us; from a graph 39 and 30 us; the
// floor stands at 35 us, above which cutting gains more in a graph than it costs outside).
// Measured with 32 heads on 8 KV heads, cut tiles and units: 333 tokens on 4,000 alone 45 and
// 94 us, beside 16 rows of 1,000 78 and 107 us, beside 127 of them 149 and 121 us; on 16,000
// beside 127 of 1,000 206 and 335 us, of 4,000 441 and 379 us (whole tiles 411 us); 20 tokens
// on 430 beside 16 rows of 16,000 206 us as whole tiles, 189 us as units.  Over 287 random
// batches of 1-64 chunk rows beside 1-128 decode rows, launched from a graph, the form chosen
// takes 0.9% more than the best of the three on average (1.8% if they are left out of view).
constexpr int64_t kMinPieceSteps = 8;
constexpr int64_t kMaxFineSlots = 2048;  // bounds the partial results (64.5 KiB each)

// A row of an append with its tokens and KV length before them; its chunk units and their
// halves are the same for every KV head.
struct ChunkRow { int64_t b, tokens, prior, row0; };
// Half h (rows [128 h, 128 h + 128)) of the unit of tokens [q0, q1): it sees `keys` keys,
// cut into n pieces (set, with the pieces' running partial slot and step, as they are cut).
struct Tile { int64_t q0, q1, h, keys, steps, n, slot, step; };

// Calls f(tile, first half of its unit) on the halves of a chunk row's units.
template <class F>
void each_tile(const ChunkRow& r, int64_t T, int64_t G, F f) {
  const int64_t half = (kTileRows - 1) / G + 1;  // tokens that a unit's first half touches
  for (int64_t q0 = 0; q0 < r.tokens; q0 += T) {
    const int64_t q1 = std::min(q0 + T, r.tokens);
    const int64_t k0 = r.prior + std::min(q1, q0 + half), k1 = r.prior + q1;
    f(Tile{q0, q1, 0, k0, ceil_div(k0, kTileStepKeys), 1, -1, 0});
    if ((q1 - q0) * G > kTileRows) f(Tile{q0, q1, 1, k1, ceil_div(k1, kTileStepKeys), 1, -1, 0});
  }
}

void build_fine(const std::vector<ChunkRow>& rows, int64_t T, int64_t single_pages,
                int64_t longest_queue, Plan& P) {
  const int64_t cus = P.params.num_cus, Hkv = P.num_kv_heads, G = P.group;
  const int64_t S = std::min<int64_t>(2 * cus, kMaxFineSlots);
  int64_t n = 0, units = 0, longest = 0, total = 0, longest_unit = 0, unit_total = 0;
  for (const ChunkRow& r : rows) {
    each_tile(r, T, G, [&](const Tile& t) {
      n += Hkv;
      longest = std::max(longest, t.steps);
      total += Hkv * t.steps;
      if (t.h) return;
      const int64_t unit_steps = ceil_div(r.prior + t.q1, kChunkStepKeys);
      units += Hkv;
      longest_unit = std::max(longest_unit, unit_steps);
      unit_total += Hkv * unit_steps;
    });
  }
  if (n == 0) return;
  if (n > S) {
    if (167 * unit_total + 840 * units <= 48 * total + 350 * n) return;
    if (n == units || n == 2 * units) {  // the units' queues and tables serve as they are
      P.chunk_form = n == units ? kFirstHalves : kBothHalves;
      P.chunk_grid = kNumXcds * longest_queue * (n / units);
      return;
    }
    // A list of the halves that there are: workgroups without one would take their turn in the
    // dispatch over the shader engines, and where every fourth has none a quarter of the CUs
    // waits (25-73 tokens of 40/8 heads on 5,500-14,500 for 32 requests: 477 us with such
    // workgroups, 437 us with a list and 436 us from full records).
    auto Q = sibling(P);
    Q->chunk_form = kListedHalves;
    Q->tiles.reserve(size_t(n));
    const int32_t* u = P.units.data() + size_t(P.info.n_single) * kUnitInts;
    int64_t longest_run = 0;
    for (size_t x = 0; x < kNumXcds; ++x) {
      const int32_t first = int32_t(Q->tiles.size());
      const int32_t end = P.xcd_map[2 * x] + P.xcd_map[2 * x + 1];
      for (int32_t i = P.xcd_map[2 * x]; i < end; ++i, u += kUnitInts) {
        Q->tiles.push_back(i << 1);
        if ((u[U_Q1] - u[U_Q0]) * G > kTileRows) Q->tiles.push_back(i << 1 | 1);
      }
      Q->xcd_map.push_back(first);
      Q->xcd_map.push_back(int32_t(Q->tiles.size()) - first);
      longest_run = std::max<int64_t>(longest_run, Q->xcd_map.back());
    }
    Q->chunk_grid = kNumXcds * longest_run;
    fine_layout(*Q, P, 0);
    P.fine = std::move(Q);
    return;
  }

  // One wave: the tiles' keys may be split.
  std::vector<Tile> tiles;  // of one KV head
  std::vector<size_t> row_end;
  tiles.reserve(size_t(n / Hkv));
  for (const ChunkRow& r : rows) {
    each_tile(r, T, G, [&](const Tile& t) { tiles.push_back(t); });
    row_end.push_back(tiles.size());
  }
  auto pieces = [&](int64_t t) {
    int64_t k = 0;
    for (const Tile& x : tiles) k += ceil_div(x.steps, t);
    return k * Hkv;
  };
  int64_t piece = longest, t = std::min(kMinPieceSteps, longest);
  for (int64_t hi = longest; t < hi;) {
    const int64_t mid = (t + hi) / 2;
    if (pieces(mid) <= S) hi = mid;
    else t = mid + 1;
  }
  const int64_t single_time = 33 * single_pages / cus;
  const int64_t lag = std::min<int64_t>(1200, 8 * single_time);
  const int64_t host = single_pages ? 3500 : 0;
  auto beside = [&](int64_t time, int64_t groups, int64_t room, int64_t least) {
    return std::max({time, lag + single_time + time * std::min(groups, room) / room, least});
  };
  auto fine_time = [&](int64_t steps, int64_t groups, int64_t fixed, int64_t least) {
    const int64_t time = steps * (groups <= cus ? 65 : 93) + fixed;
    const int64_t shared = groups <= cus ? 43 * std::min(time, single_time) / 100 : 0;
    return beside(time + shared, groups, 2 * cus, least);
  };
  const int64_t whole_time = fine_time(longest, n, 700, host);
  const int64_t split_time = fine_time(t, pieces(t), 2000, host ? host + 500 : 0);
  if (split_time < whole_time) piece = t;
  const int64_t busy = (units + unit_total / longest_unit) / 2;
  const int64_t unit_step = std::max<int64_t>(125, 80 + 90 * busy / cus);
  const int64_t unit_time = longest_unit * unit_step + 800;
  const int64_t bias = single_time > unit_time ? 95 : 100;
  if (units <= cus &&
      beside(unit_time, units, cus, host) * bias < 100 * std::min(whole_time, split_time))
    return;

  // Pieces that read the same keys next to each other (by row, KV head and key range), the
  // list cut into eight runs of equal cost, one per XCD, so that they share an L2; each
  // queue its longest piece first.
  auto Q = sibling(P);
  Q->chunk_form = kFineTiles;
  struct Piece { int32_t rec[kTileInts]; int64_t steps; };
  std::vector<std::vector<Piece>> queues(kNumXcds);
  for (auto& q : queues) q.reserve(size_t(S / kNumXcds + 1));
  int64_t slots = 0, before = 0, x = 0;
  for (Tile& t : tiles) t.n = ceil_div(t.steps, piece);
  for (size_t i = 0; i < rows.size(); ++i) {
    const ChunkRow& r = rows[i];
    Tile* const first = tiles.data() + (i ? row_end[i - 1] : 0);
    Tile* const last = tiles.data() + row_end[i];
    int64_t most = 1;
    for (const Tile* t = first; t < last; ++t) most = std::max(most, t->n);
    for (int64_t g = 0; g < Hkv; ++g) {
      for (Tile* t = first; t < last; ++t) {
        t->step = 0;
        if (t->n == 1) continue;
        const int32_t rec[kMergeInts] = {int32_t(g | t->h << 16), int32_t(t->q0), int32_t(t->n),
                                         int32_t(slots), int32_t(r.row0), int32_t(t->q1), 0, 0};
        Q->chunk_merges.insert(Q->chunk_merges.end(), rec, rec + kMergeInts);
        t->slot = slots;
        slots += t->n;
      }
      for (int64_t j = 0; j < most; ++j) {
        for (Tile* t = first; t < last; ++t) {
          if (j >= t->n) continue;
          const int64_t s0 = t->step, s1 = (j + 1) * t->steps / t->n;
          t->step = s1;
          // the eighth of the total that the middle of the piece lies in
          while ((2 * before + s1 - s0) * kNumXcds >= 2 * total * (x + 1)) ++x;
          before += s1 - s0;
          queues[size_t(x)].push_back(
              {{int32_t(r.b), int32_t(g | t->h << 16), int32_t(t->q0), int32_t(t->q1),
                int32_t(r.row0), int32_t(r.prior), int32_t(s0 * kTileStepKeys),
                int32_t(std::min(s1 * kTileStepKeys, t->keys)),
                t->n > 1 ? int32_t(t->slot + j) : -1, int32_t(t->n)}, s1 - s0});
        }
      }
    }
  }
  size_t all = 0, done = 0, longest_run = 0;
  for (const auto& q : queues) all += q.size();
  Q->tiles.resize(all * kTileInts);
  for (const auto& q : queues) {
    Q->xcd_map.push_back(int32_t(done));
    Q->xcd_map.push_back(int32_t(q.size()));
    longest_run = std::max(longest_run, q.size());
    // In order of 64 buckets of length: sizes differ by a step or two where keys are cut.
    int64_t most = 0, least = INT64_MAX;
    for (const Piece& p : q) most = std::max(most, p.steps), least = std::min(least, p.steps);
    int shift = 0;
    while (!q.empty() && (most - least) >> shift > 63) ++shift;
    std::array<size_t, 65> at{};
    for (const Piece& p : q) ++at[size_t((most - p.steps) >> shift) + 1];
    for (size_t i = 1; i < at.size(); ++i) at[i] += at[i - 1];
    for (const Piece& p : q)
      std::memcpy(Q->tiles.data() + (done + at[size_t((most - p.steps) >> shift)]++) * kTileInts, p.rec,
                  sizeof(p.rec));
    done += q.size();
  }
  Q->chunk_grid = kNumXcds * int64_t(longest_run);
  fine_layout(*Q, P, slots);
  P.fine = std::move(Q);
}

}  // namespace

libra_status build_plan(const libra_plan_desc& d, const int32_t* seq_lens, const int32_t* q_lens,
                        const libra_plan_params& p, Plan* out, bool fewer_units) {
  const int64_t B = d.batch;
  const int64_t Hkv = d.num_kv_heads;
  const int64_t G = d.num_q_heads / d.num_kv_heads;
  const bool append = d.mode == LIBRA_MODE_APPEND;

  std::vector<int64_t> L(B), C(B), pages(B), row0(B);
  int64_t rows = 0;
  for (int64_t b = 0; b < B; ++b) {
    L[b] = seq_lens[b];
    C[b] = append ? q_lens[b] : 1;
    if (L[b] < 0) return set_error(LIBRA_E_INVAL, "seq_lens must be >= 0");
    if (append && (C[b] < 1 || C[b] > L[b]))
      return set_error(LIBRA_E_INVAL, "append needs 1 <= q_lens[b] <= seq_lens[b]");
    pages[b] = ceil_div(L[b], kPage);
    row0[b] = rows;
    rows += C[b];
  }
  if (rows > INT32_MAX) return set_error(LIBRA_E_INVAL, "too many query rows");

  // Steps 3-5: one wave of S units per KV head if the single rows can fill it evenly,
  // else the chunk rule.
  std::vector<int64_t> single;
  int64_t W = 0;
  for (int64_t b = 0; b < B; ++b)
    if (C[b] == 1) {
      single.push_back(b);
      W += pages[b] * Hkv;
    }
  const int64_t S = int64_t(p.num_cus) * p.units_per_cu;
  const int64_t chunk = W > 0 ? std::max<int64_t>(p.min_split_pages, ceil_div(W, S))
                              : int64_t(p.min_split_pages);
  std::vector<int64_t> nsplit(B, 1), slot_base(B, -1);
  // The last budget is the rule's; the others are of fewer units per CU (see the end).
  const int64_t cus = p.num_cus;
  std::vector<Apportionment> budgets;
  if (fewer_units && int64_t(single.size()) == B && p.units_per_cu == 3) {
    if (W <= 100 * cus) budgets.push_back({cus / Hkv});
    if (W <= 400 * cus) budgets.push_back({2 * cus / Hkv});
  }
  budgets.push_back({S / Hkv});
  one_wave_splits(pages, single, p, budgets);
  const bool balanced = budgets.back().balanced;
  if (balanced)
    nsplit = budgets.back().n;
  else
    for (int64_t b : single)
      nsplit[b] = std::min<int64_t>(p.max_splits, std::max<int64_t>(1, ceil_div(pages[b], chunk)));

  // Step 10: partial slots in ascending (b, g).
  auto place_slots = [&](const std::vector<int64_t>& n, std::vector<int64_t>& base) {
    int64_t slots = 0;
    for (int64_t b : single) {
      base[size_t(b)] = n[size_t(b)] > 1 ? slots : -1;
      if (n[size_t(b)] > 1) slots += n[size_t(b)] * Hkv;
    }
    return slots;
  };
  const int64_t slots = place_slots(nsplit, slot_base);
  if (slots > INT32_MAX) return set_error(LIBRA_E_INVAL, "too many partial slots");

  // Steps 6, 8, 9 and 11: the single units of split counts n, on S slots.
  auto single_units = [&](const std::vector<int64_t>& nsplit, const std::vector<int64_t>& slot_base,
                          int64_t S) {
    std::vector<Unit> units;
    for (int64_t b : single) {
      const int64_t n = nsplit[b];
      for (int64_t g = 0; g < Hkv; ++g) {
        for (int64_t j = 0; j < n; ++j) {
          const int64_t p0 = (j * pages[b]) / n, p1 = ((j + 1) * pages[b]) / n;
          Unit u{};
          u[U_B] = int32_t(b);
          u[U_G] = int32_t(g);
          u[U_KV0] = int32_t(kPage * p0);
          u[U_KV1] = int32_t(std::min<int64_t>(kPage * p1, L[b]));
          u[U_Q0] = 0;
          u[U_Q1] = 1;
          u[U_SPLIT] = int32_t(j);
          u[U_NSPLIT] = int32_t(n);
          u[U_PART] = n > 1 ? int32_t(slot_base[b] + g * n) : -1;
          u[U_ROW0] = int32_t(row0[b]);
          u[U_KIND] = kKindSingle;
          u[U_PRIOR] = int32_t(L[b] - 1);
          units.push_back(u);
        }
      }
    }
    // Built in ascending (b, g, j), so equal token counts stay in that order.
    std::vector<std::pair<int32_t, int32_t>> order(units.size());  // (-tokens, index)
    for (size_t i = 0; i < units.size(); ++i)
      order[i] = {units[i][U_KV0] - units[i][U_KV1], int32_t(i)};
    std::sort(order.begin(), order.end());
    std::vector<Unit> sorted;
    sorted.reserve(units.size());
    for (const auto& o : order) sorted.push_back(units[size_t(o.second)]);
    return sorted.empty() ? sorted : place_on_slots(sorted, p, S);
  };
  // Fewer single units, where there are no chunk rows beside them and the default three units
  // per CU (as many as are resident) were asked for; the public unit table stays the rule's,
  // and the form is taken only if it needs no more workspace.  While the rows hold at most 400 pages
  // per CU, what a unit costs besides its pages (start, wait for its slowest wave, partial
  // result) and an uneven last few units weigh more than the third unit's loads in flight:
  // the rows are then cut for one wave of two units per CU if step 4 can balance it, and of
  // one if they hold at most 100 pages per CU and its largest piece is within 15% of the
  // mean.  Measured, decode and merge, caches cold: 64 rows of ~2,048 tokens (7 heads per KV
  // head, 217 pages per CU) 80.5 us with three units, 76.2 with two; 128 rows of 300-700
  // tokens (64 pages) 31.2 and 26.2; 16 rows of ~2,048 (43 pages) 23.4, 22.5 and 22.2 with
  // one; one of 40,959 (80 pages) 34.5, 34.2 and 33.5; but 32 rows (85 pages, largest piece
  // 1.3 times the mean) 37.5, 36.5 and 38.8, and 16 of 20,000-32,000 (810 pages) 271.7,
  // 273.8 and 296.1.
  auto count_units = [&](const std::vector<int64_t>& n) {
    int64_t count = 0;
    for (int64_t b : single) count += n[size_t(b)] * Hkv;
    return count;
  };
  auto count_merges = [&](const std::vector<int64_t>& n) {
    int64_t count = 0;
    for (int64_t b : single) count += n[size_t(b)] > 1 ? Hkv : 0;
    return count;
  };
  const Apportionment* fewer = nullptr;
  std::vector<int64_t> fewer_base(B, -1);
  int64_t fewer_slots = 0;
  for (size_t i = 0; i + 1 < budgets.size() && !fewer; ++i) {
    const Apportionment& a = budgets[i];
    if (!a.balanced || (a.R == cus / Hkv && 100 * a.largest * cus > 115 * W)) continue;
    fewer_slots = place_slots(a.n, fewer_base);
    if (count_units(a.n) < count_units(nsplit) && count_merges(a.n) <= count_merges(nsplit) &&
        fewer_slots <= slots)
      fewer = &a;
  }
  // Step 11: CU slots for one wave, else the XCD queues.
  std::vector<Unit> singles;
  if (!fewer)
    singles = single_units(nsplit, slot_base, balanced ? int64_t(p.num_cus) : int64_t(kNumXcds));
  std::vector<Unit> chunks;
  std::vector<ChunkRow> chunk_rows;

  // Step 7: query tiles of chunk rows.
  const int64_t T = p.q_tile > 0 ? p.q_tile : int64_t(kChunkRows) / G;
  for (int64_t b = 0; b < B; ++b) {
    if (C[b] == 1) continue;
    const int64_t P = L[b] - C[b];
    chunk_rows.push_back({b, C[b], P, row0[b]});
    for (int64_t g = 0; g < Hkv; ++g) {
      for (int64_t q0 = 0; q0 < C[b]; q0 += T) {
        const int64_t q1 = std::min(q0 + T, C[b]);
        Unit u{};
        u[U_B] = int32_t(b);
        u[U_G] = int32_t(g);
        u[U_KV0] = 0;
        u[U_KV1] = int32_t(P + q1);
        u[U_Q0] = int32_t(q0);
        u[U_Q1] = int32_t(q1);
        u[U_SPLIT] = 0;
        u[U_NSPLIT] = 1;
        u[U_PART] = -1;
        u[U_ROW0] = int32_t(row0[b]);
        u[U_KIND] = kKindChunk;
        u[U_PRIOR] = int32_t(P);
        chunks.push_back(u);
      }
    }
  }
  // Step 9 (chunk units): XCD-affine order.  Tiles of one (b, g) read the same keys, so
  // they are kept on one XCD (workgroup w runs on XCD w % kNumXcds) to share its L2,
  // unless the group costs more than an eighth of the launch: it is then cut into
  // contiguous, cost-balanced parts so that every XCD gets work.  Parts by descending
  // cost (ties ascending (b, g, part)) are dealt to the XCD queue with the least
  // accumulated cost (ties to the lowest queue); each queue then lists its parts by
  // descending cost of their longest tile, a part's tiles together and longest first (so
  // the last tiles a CU takes are short, and the tiles that read the same keys run
  // together); queues are listed one after another.  A tile costs its key-loop steps: the kernel spends the
  // same time on a step whatever the number of the tile's query tokens.
  auto cost = [](const Unit& u) { return ceil_div(u[U_KV1] - u[U_KV0], kChunkStepKeys); };
  int64_t total_cost = 0;
  for (const Unit& u : chunks) total_cost += cost(u);
  const int64_t fair = std::max<int64_t>(1, ceil_div(total_cost, kNumXcds));
  struct Part { int64_t cost; int32_t b, g, idx; size_t first, last; };  // [first, last) in part_tiles
  std::vector<Part> parts;
  std::vector<Unit> part_tiles;  // chunks regrouped part by part
  part_tiles.reserve(chunks.size());
  for (size_t i = 0; i < chunks.size();) {  // chunks are built in ascending (b, g, q_begin)
    size_t j = i + 1;
    while (j < chunks.size() && chunks[j][U_B] == chunks[i][U_B] && chunks[j][U_G] == chunks[i][U_G]) ++j;
    int64_t c = 0;
    for (size_t k = i; k < j; ++k) c += cost(chunks[k]);
    const int64_t n = std::min<int64_t>(int64_t(j - i), ceil_div(c, fair));
    int64_t before = 0, cur = -1;
    for (size_t k = i; k < j; ++k) {
      const int64_t idx = int64_t(__int128(before) * n / c);
      if (idx != cur) {
        parts.push_back(Part{0, chunks[k][U_B], chunks[k][U_G], int32_t(idx), part_tiles.size(),
                             part_tiles.size()});
        cur = idx;
      }
      parts.back().cost += cost(chunks[k]);
      parts.back().last += 1;
      part_tiles.push_back(chunks[k]);
      before += cost(chunks[k]);
    }
    i = j;
  }
  std::vector<size_t> porder(parts.size());
  for (size_t k = 0; k < porder.size(); ++k) porder[k] = k;
  std::sort(porder.begin(), porder.end(), [&](size_t a, size_t b) {
    const Part &x = parts[a], &y = parts[b];
    if (x.cost != y.cost) return x.cost > y.cost;
    if (x.b != y.b) return x.b < y.b;
    if (x.g != y.g) return x.g < y.g;
    return x.idx < y.idx;
  });
  // Deal the parts; then each queue lists its parts by descending cost of their longest
  // tile (ties ascending (b, g, part)), a part's tiles together, by descending cost (ties
  // ascending q_begin).
  std::vector<std::vector<size_t>> qparts(kNumXcds);
  int64_t qcost[kNumXcds] = {0};
  for (size_t k : porder) {
    int x = 0;
    for (int y = 1; y < kNumXcds; ++y)
      if (qcost[y] < qcost[x]) x = y;
    qcost[x] += parts[k].cost;
    qparts[x].push_back(k);
  }
  auto tile_order = [&](const Unit& a, const Unit& b) {
    const int64_t ca = cost(a), cb = cost(b);
    if (ca != cb) return ca > cb;
    return a[U_Q0] < b[U_Q0];
  };
  std::vector<int64_t> longest_tile(parts.size(), 0);
  for (size_t k = 0; k < parts.size(); ++k) {
    std::sort(part_tiles.begin() + parts[k].first, part_tiles.begin() + parts[k].last, tile_order);
    longest_tile[k] = cost(part_tiles[parts[k].first]);
  }
  std::vector<std::vector<Unit>> queues(kNumXcds);
  for (int x = 0; x < kNumXcds; ++x) {
    std::sort(qparts[x].begin(), qparts[x].end(), [&](size_t a, size_t b) {
      if (longest_tile[a] != longest_tile[b]) return longest_tile[a] > longest_tile[b];
      const Part &pa = parts[a], &pb = parts[b];
      if (pa.b != pb.b) return pa.b < pb.b;
      if (pa.g != pb.g) return pa.g < pb.g;
      return pa.idx < pb.idx;
    });
    for (size_t k : qparts[x])
      queues[x].insert(queues[x].end(), part_tiles.begin() + parts[k].first,
                       part_tiles.begin() + parts[k].last);
  }
  chunks.clear();
  int32_t xcd_map[2 * kNumXcds];
  int32_t longest = 0;
  for (int x = 0; x < kNumXcds; ++x) {
    xcd_map[2 * x] = int32_t(chunks.size());
    xcd_map[2 * x + 1] = int32_t(queues[x].size());
    longest = std::max<int32_t>(longest, int32_t(queues[x].size()));
    chunks.insert(chunks.end(), queues[x].begin(), queues[x].end());
  }

  Plan& P = *out;
  P.mode = d.mode;
  P.batch = d.batch;
  P.num_q_heads = d.num_q_heads;
  P.num_kv_heads = d.num_kv_heads;
  P.group = int32_t(G);
  P.params = p;
  P.units.clear();
  P.units.reserve((singles.size() + chunks.size()) * kUnitInts);
  for (const Unit& u : singles) P.units.insert(P.units.end(), u.begin(), u.end());
  for (const Unit& u : chunks) P.units.insert(P.units.end(), u.begin(), u.end());

  // Cache-write table (append): every (sequence, page) holding new positions [P_b, L_b).
  P.writes.clear();
  if (append) {
    for (int64_t b = 0; b < B; ++b) {
      const int64_t P0 = L[b] - C[b];
      for (int64_t pg = P0 / kPage; pg * kPage < L[b]; ++pg) {
        const int64_t s0 = std::max<int64_t>(P0, pg * kPage) - pg * kPage;
        const int64_t s1 = std::min<int64_t>(L[b], pg * kPage + kPage) - pg * kPage;
        const int32_t rec[kWriteInts] = {int32_t(b), int32_t(pg), int32_t(s0), int32_t(s1),
                                         int32_t(row0[b] + pg * kPage + s0 - P0), 0, 0, 0};
        P.writes.insert(P.writes.end(), rec, rec + kWriteInts);
      }
    }
  }

  P.xcd_map.assign(xcd_map, xcd_map + 2 * kNumXcds);
  P.chunk_grid = int64_t(kNumXcds) * longest;

  // Split-merge table: every single row with n_b > 1, per KV head, ascending (b, g).
  auto merge_table = [&](const std::vector<int64_t>& n, const std::vector<int64_t>& base) {
    std::vector<int32_t> merges;
    for (int64_t b : single) {
      if (n[b] <= 1) continue;
      for (int64_t g = 0; g < Hkv; ++g) {
        const int32_t rec[kMergeInts] = {int32_t(b), int32_t(g), int32_t(n[b]),
                                         int32_t(base[b] + g * n[b]), int32_t(row0[b]), 0, 0, 0};
        merges.insert(merges.end(), rec, rec + kMergeInts);
      }
    }
    return merges;
  };
  if (!fewer) P.merges = merge_table(nsplit, slot_base);

  // Block-table columns the kernels read: every unit's pages and every written page.
  P.pages_needed = 0;
  for (int64_t b = 0; b < B; ++b) P.pages_needed = std::max(P.pages_needed, pages[b]);
  for (size_t i = 0; i < P.writes.size(); i += kWriteInts)
    P.pages_needed = std::max<int64_t>(P.pages_needed, int64_t(P.writes[i + W_PAGE]) + 1);

  libra_plan_info& I = P.info;
  std::memset(&I, 0, sizeof(I));
  I.n_single = int32_t(count_units(nsplit));
  I.n_chunk = int32_t(chunks.size());
  I.n_units = I.n_single + I.n_chunk;
  I.n_partial_slots = int32_t(slots);
  I.chunk_pages = chunk;
  I.q_tile = int32_t(T);
  I.n_rows = int32_t(rows);
  I.n_write_tiles = int32_t(P.writes.size() / kWriteInts);
  I.num_cus = p.num_cus;
  I.n_merge_groups = int32_t(count_merges(nsplit));
  I.balanced = balanced ? 1 : 0;

  workspace_layout(P);
  build_fine(chunk_rows, T, W, longest, P);
  if (fewer) {
    auto Q = sibling(P);
    for (const Unit& u : single_units(fewer->n, fewer_base, cus))
      Q->units.insert(Q->units.end(), u.begin(), u.end());
    Q->merges = merge_table(fewer->n, fewer_base);
    Q->info.n_units = Q->info.n_single = int32_t(Q->units.size() / kUnitInts);
    Q->info.n_partial_slots = int32_t(fewer_slots);
    Q->info.n_merge_groups = int32_t(Q->merges.size() / kMergeInts);
    Q->writes = P.writes;
    Q->xcd_map = P.xcd_map;
    workspace_layout(*Q);  // every part is at most as large as P's
    Q->ws_bytes = P.ws_bytes;
    P.lens.assign(seq_lens, seq_lens + B);
    P.upload_bytes = 0;
    P.fine = std::move(Q);
  }
  return LIBRA_OK;
}

libra_status build_units(Plan& P) {
  libra_plan_desc d{};
  d.mode = P.mode;
  d.batch = P.batch;
  d.num_q_heads = P.num_q_heads;
  d.num_kv_heads = P.num_kv_heads;
  const std::vector<int32_t> ones(P.lens.size(), 1);
  Plan whole;
  const libra_status st = build_plan(d, P.lens.data(), d.mode == LIBRA_MODE_APPEND ? ones.data() : nullptr,
                                     P.params, &whole, false);
  if (st == LIBRA_OK) P.units = std::move(whole.units);
  return st;
}

}  // namespace libra
