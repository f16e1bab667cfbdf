// The launched forms of plans, checked and printed.  Reads one plan per line from stdin:
//   mode batch num_q_heads num_kv_heads num_cus units_per_cu min_split_pages max_splits q_tile
//   then the KV lengths and, for append (mode 1), the new tokens,
// builds it with the library's planner alone and checks that the launch covers every (token,
// head, key) once: the decode units' key ranges and partial slots with their merge records,
// the chunk workgroups' rows and key ranges as the kernel takes them from units, halves of
// units or fine tiles, their queues, partial slots and merge records, and that the tables and
// partials lie in the workspace without overlap.  Prints one line per plan:
//   <chunk form> <chunk workgroups> <most key ranges of a tile> <most pages of a workgroup>
//   <decode units> <decode units of the table> <most splits of a row> <workspace> <plain>
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <set>
#include <string>
#include <tuple>

#include "internal.h"

using namespace libra;

namespace libra {
libra_status set_error(libra_status s, const std::string&) { return s; }
libra_status hip_error(hipError_t, const char*) { return LIBRA_E_HIP; }
}  // namespace libra

#define CHECK(cond)                                                          \
  do {                                                                       \
    if (!(cond)) {                                                           \
      std::fprintf(stderr, "check failed: %s (line %d)\n", #cond, __LINE__); \
      std::exit(1);                                                          \
    }                                                                        \
  } while (0)

namespace {

// A chunk workgroup: tile rows [first, first + rows) of (b, g, q0, q1), keys [kv0, kv1).
struct Group {
  int b, g, q0, q1, first, rows, row0, prior, kv0, kv1, part, n;
};

// The chunk workgroups of a launch, in the kernel's terms.
std::vector<Group> chunk_groups(const Plan& P, const Plan& base) {
  std::vector<Group> out;
  const std::vector<int32_t>& units = base.units;
  const size_t first = size_t(P.info.n_single);
  int64_t longest = 0;
  for (int x = 0; x < kNumXcds; ++x) {
    const int f = P.xcd_map[size_t(2 * x)], c = P.xcd_map[size_t(2 * x + 1)];
    CHECK(x == 0 ? f == 0 : f == P.xcd_map[size_t(2 * x - 2)] + P.xcd_map[size_t(2 * x - 1)]);
    const int per = P.chunk_form == kBothHalves ? 2 : 1;
    longest = std::max<int64_t>(longest, int64_t(c) * per);
    for (int slot = 0; slot < c * per; ++slot) {
      if (P.chunk_form == kFineTiles) {
        CHECK(size_t(f + slot + 1) * kTileInts <= P.tiles.size());
        const int32_t* t = P.tiles.data() + size_t(f + slot) * kTileInts;
        out.push_back({t[T_B], t[T_GH] & 0xFFFF, t[T_Q0], t[T_Q1], (t[T_GH] >> 16) * kTileRows,
                       kTileRows, t[T_ROW0], t[T_PRIOR], t[T_KV0], t[T_KV1], t[T_PART],
                       t[T_NSPLIT]});
        continue;
      }
      int unit = f + slot / per, h = slot % per;
      if (P.chunk_form == kListedHalves) {
        CHECK(size_t(f + slot) < P.tiles.size());
        unit = P.tiles[size_t(f + slot)] >> 1, h = P.tiles[size_t(f + slot)] & 1;
      }
      CHECK((first + size_t(unit) + 1) * kUnitInts <= units.size());
      const int32_t* u = units.data() + (first + size_t(unit)) * kUnitInts;
      CHECK(u[U_KIND] == kKindChunk);
      const bool narrow = P.chunk_form != kUnits;
      const int rows = narrow ? kTileRows : kChunkRows;
      CHECK(h * rows < (u[U_Q1] - u[U_Q0]) * P.group);  // no workgroup without rows
      const int kv1 = narrow && h == 0
                          ? std::min(u[U_KV1], u[U_PRIOR] + u[U_Q0] + (kTileRows - 1) / P.group + 1)
                          : u[U_KV1];
      out.push_back({u[U_B], u[U_G], u[U_Q0], u[U_Q1], h * rows, rows, u[U_ROW0], u[U_PRIOR], 0, kv1,
                     -1, 1});
    }
  }
  CHECK(P.chunk_grid == kNumXcds * longest);
  return out;
}

}  // namespace

int main() {
  int mode;
  libra_plan_desc d{};
  libra_plan_params p{};
  while (std::scanf("%d %d %d %d %d %d %d %d %d", &mode, &d.batch, &d.num_q_heads, &d.num_kv_heads,
                    &p.num_cus, &p.units_per_cu, &p.min_split_pages, &p.max_splits,
                    &p.q_tile) == 9) {
    d.mode = mode;
    const int G = d.num_q_heads / d.num_kv_heads;
    std::vector<int32_t> L(size_t(d.batch)), C(size_t(d.batch), 1);
    for (auto& x : L) CHECK(std::scanf("%d", &x) == 1);
    if (mode)
      for (auto& x : C) CHECK(std::scanf("%d", &x) == 1);
    Plan plan;
    CHECK(build_plan(d, L.data(), mode ? C.data() : nullptr, p, &plan) == LIBRA_OK);
    const Plan& P = plan.fine ? *plan.fine : plan;
    const Plan& T = P.base ? *P.base : P;  // whose unit, write and merge tables the launch reads
    std::vector<int> row0(L.size() + 1, 0);
    for (size_t b = 0; b < L.size(); ++b) row0[b + 1] = row0[b] + C[b];

    // Decode units: every (row, KV head) once over its keys.
    std::map<std::pair<int, int>, std::vector<const int32_t*>> singles;
    int most_splits = 0, widest = 0;
    CHECK(T.units.size() >= size_t(P.info.n_single) * kUnitInts);
    for (int i = 0; i < P.info.n_single; ++i) {
      const int32_t* u = T.units.data() + size_t(i) * kUnitInts;
      singles[{u[U_B], u[U_G]}].push_back(u);
    }
    std::set<int> slots;
    std::map<std::pair<int, int>, const int32_t*> merges;
    CHECK(T.merges.size() == size_t(P.info.n_merge_groups) * kMergeInts);
    for (size_t i = 0; i < T.merges.size(); i += kMergeInts)
      CHECK(merges.insert({{T.merges[i + M_B], T.merges[i + M_G]}, &T.merges[i]}).second);
    size_t want = 0;
    for (size_t b = 0; b < L.size(); ++b) {
      if (C[b] != 1) continue;
      for (int g = 0; g < d.num_kv_heads; ++g, ++want) {
        auto& us = singles[{int(b), g}];
        std::sort(us.begin(), us.end(), [](auto* x, auto* y) { return x[U_SPLIT] < y[U_SPLIT]; });
        const int n = int(us.size());
        CHECK(n >= 1 && us[0][U_KV0] == 0 && us.back()[U_KV1] == L[b]);
        const bool split = n > 1;
        CHECK(merges.count({int(b), g}) == (split ? 1u : 0u));
        most_splits = std::max(most_splits, n);
        for (int j = 0; j < n; ++j) {
          const int32_t* u = us[size_t(j)];
          CHECK(u[U_SPLIT] == j && u[U_NSPLIT] == n && u[U_ROW0] == row0[b] && u[U_KIND] == kKindSingle);
          CHECK(j == 0 || (u[U_KV0] == us[size_t(j - 1)][U_KV1] && u[U_KV0] % kPage == 0));
          if (!split) CHECK(u[U_PART] == -1);
          if (!split) continue;
          const int32_t* m = merges[{int(b), g}];
          CHECK(u[U_PART] == m[M_PART] && m[M_N] == n && m[M_ROW] == row0[b]);
          CHECK(m[M_PART] + j < P.info.n_partial_slots && slots.insert(m[M_PART] + j).second);
        }
      }
    }
    CHECK(singles.size() == want);

    // Chunk workgroups: every row of (b, g) over the keys it sees, each key range once.
    const std::vector<Group> groups = chunk_groups(P, T);
    using Key = std::tuple<int, int, int, int>;  // (b, g, q0, first row)
    std::map<Key, std::vector<Group>> tiles;
    std::map<std::pair<int, int>, int64_t> rows_done;
    int most_parts = 0;
    for (const Group& t : groups) tiles[{t.b, t.g, t.q0, t.first}].push_back(t);
    std::set<int> parts;
    std::map<Key, const int32_t*> chunk_merges;
    for (size_t i = 0; i < P.chunk_merges.size(); i += kMergeInts) {
      const int32_t* m = &P.chunk_merges[i];
      bool found = false;  // its sequence is the one with its first row
      for (size_t b = 0; b < L.size(); ++b)
        if (row0[b] == m[CM_ROW0] && C[b] > 1)
          found = chunk_merges.insert({Key{int(b), m[CM_GH] & 0xFFFF, m[CM_Q0], (m[CM_GH] >> 16) * kTileRows}, m}).second;
      CHECK(found);
    }
    size_t merged = 0;
    for (auto& [key, ts] : tiles) {
      std::sort(ts.begin(), ts.end(), [](const Group& x, const Group& y) { return x.kv0 < y.kv0; });
      const Group& t = ts[0];
      const int n = int(ts.size());
      const int tokens = std::min(t.q1, t.q0 + (t.first + t.rows - 1) / G + 1);
      CHECK(t.b >= 0 && t.b < d.batch && t.g >= 0 && t.g < d.num_kv_heads && C[size_t(t.b)] > 1);
      CHECK(t.q1 > t.q0 && t.q1 <= C[size_t(t.b)] && (t.q1 - t.q0) * G <= kChunkRows);
      CHECK(t.kv0 == 0 && ts.back().kv1 == t.prior + tokens);
      rows_done[{t.b, t.g}] += std::min((t.q1 - t.q0) * G - t.first, t.rows);
      most_parts = std::max(most_parts, n);
      for (int j = 0; j < n; ++j) {
        const Group& x = ts[size_t(j)];
        CHECK(x.n == n && x.row0 == row0[size_t(t.b)] && x.prior == L[size_t(t.b)] - C[size_t(t.b)] && x.q1 == t.q1);
        CHECK(j == 0 || x.kv0 == ts[size_t(j - 1)].kv1);
        CHECK(x.kv0 % kTileStepKeys == 0 && x.kv1 > x.kv0);
        widest = std::max(widest, int((x.kv1 - x.kv0 + kPage - 1) / kPage));
        CHECK((x.part >= 0) == (n > 1));
        if (n > 1) CHECK(parts.insert(x.part).second && x.part == ts[0].part + j);
      }
      if (n > 1) {
        const auto it = chunk_merges.find(key);
        CHECK(it != chunk_merges.end());
        CHECK(it->second[CM_N] == n && it->second[CM_PART] == ts[0].part && it->second[CM_Q1] == t.q1);
        ++merged;
      }
    }
    CHECK(merged * kMergeInts == P.chunk_merges.size());
    for (size_t b = 0; b < L.size(); ++b)
      for (int g = 0; g < d.num_kv_heads && C[b] > 1; ++g)
        CHECK((rows_done[{int(b), g}]) == int64_t(C[b]) * G);

    // Workspace: the launch's tables and partials within it, behind one another.
    std::vector<std::pair<size_t, size_t>> at = {
        {P.off_units, T.units.size() * 4}, {P.off_writes, T.writes.size() * 4},
        {P.off_merges, T.merges.size() * 4},
        {P.off_part_o, size_t(P.info.n_partial_slots) * G * kDim * 4},
        {P.off_part_lse, size_t(P.info.n_partial_slots) * G * 4},
        {P.off_tiles, P.tiles.size() * 4}, {P.off_chunk_merges, P.chunk_merges.size() * 4},
        {P.off_chunk_o, parts.size() * kTileRows * kDim * 4},
        {P.off_chunk_lse, parts.size() * kTileRows * 4}};
    std::sort(at.begin(), at.end());
    size_t end = 0;
    for (const auto& [off, bytes] : at) {
      if (bytes == 0) continue;
      CHECK(off % 256 == 0 && off >= end);
      end = off + bytes;
    }
    CHECK(end <= P.ws_bytes && plan.ws_bytes <= P.ws_bytes);
    if (P.base) CHECK(P.upload_off >= plan.ws_bytes && P.off_tiles >= plan.ws_bytes);
    CHECK(parts.empty() || *parts.rbegin() + 1 == int(parts.size()));

    const char* const names[] = {"units", "halves", "halves", "listed", "tiles"};
    const char* form = groups.empty() ? "none" : names[P.chunk_form];
    std::printf("%s %zu %d %d %d %d %d %zu %zu\n", form, groups.size(), most_parts, widest,
                P.info.n_single, plan.info.n_single, most_splits, P.ws_bytes, plan.ws_bytes);
  }
  return 0;
}
