// How the units of a plan go to the GPU: which way a launch takes them, and the records and lists the unit kernel reads.
// Host only, worked out from the plan alone; the plan a caller sees (xy_attn_plan_get) does not change with it.
#include <algorithm>
#include <cstdint>
#include <cstring>
#include <vector>

#include "plan_internal.h"
#include "xy_probe.h"

namespace {

constexpr int32_t kXcds = 8;
constexpr int64_t kWavefronts = 4;          // per worker
// How a launch processes its units of at most 32 rows, by what they are on average over the
// launch; wavefronts are four per worker.  A unit on two slices costs some 200 instructions more than a short one, which
// a lone wavefront pays for with 0.1 us and a busy CU with more, and gains where it waits for memory in every slice, with its
// neighbours idle.  Unit kernel, us short / two slices, decodes of 32 heads in 8, each a unit of its own, caches cold:
//   units   1 slice          2               3               4               5               8
//   8       4.9 / 5.0        5.8 / 5.9       6.9 / 6.9       7.7 / 7.7       8.8 / 8.6       11.6 / 11.3
//   512     6.1 / 6.3        7.3 / 8.2       8.7 / 9.1       10.0 / 10.2     11.7 / 11.6     15.0 / 14.7
//   1024    7.5 / 7.9        9.8 / 10.9      12.1 / 12.6     14.6 / 14.8     17.6 / 17.7     24.7 / 24.9
//   2048    12.5 / 13.1      16.5 / 18.8     21.6 / 22.4     25.5 / 26.1     31.4 / 31.7     46.8 / 46.3
//   4096    20.3 / 21.8      29.0 / 32.5     38.2 / 38.9     47.9 / 49.0     59.4 / 60.4     90.5 / 90.9
// so up to four slices a unit are short, up to eight (level there, 1 to 2 % at five) where there are more units than wavefronts.
// Units of 32 rows, whose Q is eight times as much, 512 / 2048 / 4096 of them: 8.7 / 9.8, 22.9 / 25.4, 42.2 / 44.6 with 2 slices,
// 10.0 / 10.7, 28.2 / 29.4, 52.7 / 53.1 with 3, 11.2 / 11.7, 32.5 / 33.7, 63.4 / 64.2 with 4.  The line of two slices above 16 rows
// a unit was drawn when 4096 units of 4 slices took 66.4 / 65.7; with both ways as they are now it is on the safe side of where they meet.
constexpr int64_t kShortSlices = 4, kShortSlicesManyUnits = 8, kShortSlicesManyRows = 2, kManyRows = 16;
// Longer ones: two slices in flight up to kDeepTiles tiles a wavefront, one beyond (see process_solo; two are 1 to 3 % faster at
// 7.5 tiles and half a percent at 11.6, one is 2 % faster at 14 and 1 % at 15.5).
constexpr int64_t kDeepTiles = 10;
// Units of more than kHalfRows rows that go to the GPU as two, by their tokens, for a worker each: all of them or none.
// The kernel then holds one row tile a wavefront instead of two, which takes two thirds of the time for units that are
// alone, but reads the K/V twice and keeps two workers busy: only where there are idle workers for all second halves, with a
// wavefront left for every narrow unit.  Unit kernel, us, whole / halves, 64 tokens x 4 heads, caches cold:
//   units   1 K/V tile       4              16             64
//   8       14.3 / 10.3      21.5 / 15.0    49.1 / 34.5    161 / 114
//   64      14.7 / 11.0      22.2 / 16.4    51.0 / 37.5    166 / 119
//   112     15.5 / 11.8      23.4 / 17.9    53.2 / 41.4    170 / 131
//   128     15.6 / 12.1      23.9 / 18.7    53.8 / 42.6    170 / 142    (every worker busy)
// and with fewer wavefronts left than narrow units the other way round (whole / halves: a suffix of 160 tokens beside 536
// narrow units 244.0 / 259.7 us for eight layers, a chunk of 512 beside 1184 156.5 / 163.3).  The plan the caller sees stays as it is.
// A half is at most kHalfRows rows, so the tokens of a unit must divide: with 3, 5, 10, 12 and some other heads a group the
// default tile (256 / heads tokens: 85, 51, 25, 21) has a first half of 129 to 132 rows, and one such unit keeps the whole
// launch on two row tiles, without teams.
int32_t first_half(const xy_work_unit& u) { return (u.q_count + 1) / 2; }
// Wavefronts that share a narrow unit, for launches that have fewer such units than wavefronts: four while every unit can
// have a worker without wide units to itself, two while half of one, else none.  Unit kernel, us, one wavefront a unit / team (decodes of 32 heads
// in 8, caches cold):
//   units   2 slices (64 keys)   3             4             8             16            63
//   8       6.0 / 5.7            6.6 / 6.1     7.8 / 6.4     11.3 / 8.2    18.4 / 10.0   59.8 / 23.1
//   224     6.2 / 6.5            7.3 / 7.1     8.2 / 7.7     12.1 / 10.4   19.2 / 13.7   61.5 / 38.0
//   256     6.4 / 6.6            7.3 / 7.3     8.5 / 8.0     12.2 / 10.9   19.4 / 14.7   61.9 / 43.0
//   264     6.6 / 6.9 (two)      7.9 / 8.5     8.8 / 9.4     12.6 / 11.7   20.4 / 18.4   64.3 / 58.8
//   512     7.4 / 8.0            8.8 / 9.8     10.3 / 10.9   15.7 / 15.2   26.1 / 24.6   87.1 / 83.7
// so a team of four takes units of three slices and more on average, a team of two those of eight.  XY_SPLIT_AUTO cuts such
// batches into more pieces than that; teams of two are for plans with a split size of the caller's or none.
constexpr int64_t kTeamOf4Slices = 3, kTeamOf2Slices = 8;

int32_t rows_of(const xy_work_unit& u) { return u.q_count * u.head_count; }
bool is_narrow(const xy_work_unit& u) { return rows_of(u) <= 32; }

}  // namespace

XyLayout xy_plan_layout(const xy_attn_plan* plan) {
  const int64_t units = plan->narrow_units, slices = plan->narrow_slices, W = plan->cfg.num_workers, large = plan->large_units;
  XyLayout l;
  l.records = (int32_t)plan->units.size();
  l.row_tiles = plan->most_rows > kHalfRows ? 2 : 1;
  const int64_t wavefronts = kWavefronts * W, wide = l.records - units;
  const int64_t short_slices = plan->narrow_rows > kManyRows * units ? kShortSlicesManyRows
                               : units > wavefronts ? kShortSlicesManyUnits : kShortSlices;
  l.short_units = units > 0 && slices <= short_slices * units;
  l.depth = plan->narrow_tiles <= kDeepTiles * wavefronts ? 2 : 1;
  const int32_t* const lists = plan->worker_offsets.data();
  int64_t free = W;             // workers without wide units
  if (wide > 0) {
    int32_t busy = 0;
    for (int64_t w = 0; w < W; ++w) busy += lists[w] != lists[w + 1];
    const int64_t idle = W - busy;
    if (large > 0 && (plan->half_rows > kHalfRows || large > idle || units > kWavefronts * (idle - large))) return l;
    free = idle;
    if (units > 0 && lists[W] > wide)           // narrow units on the workers' lists
      for (int64_t w = 0; w < W; ++w)
        free += lists[w] != lists[w + 1] && std::all_of(&plan->units[lists[w]], &plan->units[lists[w + 1] - 1] + 1, is_narrow);
    free -= large;
  }
  l.halved = (int32_t)large;
  l.records += l.halved;
  l.row_tiles = 1;
  // (the kernels with teams hold one row tile: no unit has more than kHalfRows rows here)
  l.team = units == 0 ? 0 : units <= free ? (slices >= kTeamOf4Slices * units ? 4 : 0)
           : units <= 2 * free && slices >= kTeamOf2Slices * units ? 2 : 0;
  if (l.team) l.depth = 2;
  return l;
}

int32_t xy_plan_hand_out(xy_attn_plan* plan, const XyLayout& l, XyDevUnit* du, int32_t* offsets) {
  const int32_t group = plan->cfg.num_q_heads / plan->cfg.num_kv_heads;
  const int32_t W = plan->cfg.num_workers, per_chip = W % kXcds == 0 ? W / kXcds : W;
  int32_t* const rank = offsets + W + 1;
  const xy_work_unit* const units = plan->units.data();
  const xy_seq_desc* const descs = plan->descs.data();
  const int32_t *const starts = plan->token_start.data(), *const lists = plan->worker_offsets.data();
  std::vector<int32_t>& second_of = plan->scratch.cursor;      // worker -> the unit whose second half it gets, or -1
  if (l.halved) {
    second_of.assign(W, -1);                                    // (the planner left room for W)
    // the second half goes to an idle worker of the same chiplet if there is one: both read the same K/V
    int32_t at[kXcds] = {};                                     // the next worker to look at, per chiplet
    auto next_idle = [&](const int32_t chip) {
      const int32_t* const of_chip = lists + chip * per_chip;
      int32_t& n = at[chip];
      while (n < per_chip && of_chip[n] != of_chip[n + 1]) ++n;
      return n < per_chip ? chip * per_chip + n++ : -1;
    };
    for (int32_t w = 0; w < W; ++w)
      for (int32_t i = lists[w]; i < lists[w + 1]; ++i) {
        if (rows_of(units[i]) <= kHalfRows) continue;
        int32_t to = next_idle(w / per_chip);
        for (int32_t chip = 0; to < 0; ++chip) to = next_idle(chip);     // there are as many idle workers as halves
        second_of[to] = i;
      }
  }
  int32_t emitted = 0, free_workers = 0;
  auto record = [=](const xy_work_unit& u, const int32_t q_begin, const int32_t q_count, const int32_t flags) {
    const xy_seq_desc& sd = descs[u.seq];
    return XyDevUnit{u.seq, u.head_begin, u.head_count, q_begin, q_count, u.kv_block_begin, u.kv_block_end, flags, u.ws_offset,
                     sd.mask_word_offset, sd.query_len, sd.context_len, starts[u.seq], u.head_begin / group};
  };
  const int32_t all = (int32_t)plan->units.size();
  if (l.team || (l.row_tiles == 1 && plan->most_rows > 32)) {
    auto emit = [&](const xy_work_unit& u, const int32_t first_token, const int32_t tokens) {
      const int32_t flags = u.kind_flags | rows_of(u) << kSlabRowsShift | (first_token * u.head_count) << kSlabFirstShift;
      du[emitted++] = record(u, u.q_begin + first_token, tokens, flags);
    };
    const int32_t* const second = l.halved ? second_of.data() : nullptr;
    for (int32_t w = 0; w < W; ++w) {
      offsets[w] = emitted;
      for (int32_t i = lists[w]; i < lists[w + 1]; ++i) {
        if (l.team && is_narrow(units[i])) continue;
        emit(units[i], 0, l.halved && rows_of(units[i]) > kHalfRows ? first_half(units[i]) : units[i].q_count);
      }
      if (second && second[w] >= 0) {
        const xy_work_unit& u = units[second[w]];
        emit(u, first_half(u), u.q_count - first_half(u));
      }
    }
    offsets[W] = emitted;
    // the shared list; with teams every narrow unit is on it
    if (l.team) {
      for (int32_t i = 0; i < all; ++i)
        if (is_narrow(units[i])) emit(units[i], 0, units[i].q_count);
    } else {
      for (int32_t i = lists[W]; i < all; ++i) du[emitted++] = record(units[i], units[i].q_begin, units[i].q_count, units[i].kind_flags);
    }
  } else {
    emitted = all;
    for (int32_t i = 0; i < emitted; ++i) du[i] = record(units[i], units[i].q_begin, units[i].q_count, units[i].kind_flags);
    memcpy(offsets, lists, plan->worker_offsets.size() * sizeof(int32_t));
  }
  for (int32_t w = 0; w < W; ++w) rank[w] = offsets[w + 1] == offsets[w] ? free_workers++ : -1;
  if (l.team && per_chip < W && free_workers < W) {
    // Team i is the worker of rank i: the chiplets in turn, or a short launch would run on one or two of them (unit kernel, eight
    // wide units beside 32 / 128 / 192 decodes of 2000 keys, caches cold, us: ranks in the workers' order 34.8 / 44.4 / 46.4,
    // in turn 29.1 / 34.9 / 41.2; where a launch is bound by one unit, the same).  The shared list keeps the workers' order: units
    // that stand next to each other there may read the same K/V.
    int32_t at[kXcds] = {};
    for (int32_t given = 0; given < free_workers;)
      for (int32_t chip = 0; chip < kXcds; ++chip) {
        const int32_t* const of_chip = rank + chip * per_chip;
        while (at[chip] < per_chip && of_chip[at[chip]] < 0) ++at[chip];
        if (at[chip] < per_chip) rank[chip * per_chip + at[chip]++] = given++;
      }
  }
  return free_workers;
}

extern "C" int xy_probe_plan_layout(xy_attn_plan* plan, xy_probe_layout* out, void* records, int64_t capacity, int32_t* lists) {
  if (!plan || !out || !records != !lists) return XY_ERR_ARG;
  const XyLayout l = xy_plan_layout(plan);
  *out = xy_probe_layout{l.row_tiles, l.halved, l.team, l.short_units, l.depth, l.records};
  if (!records) return XY_OK;
  if (capacity < l.records) return XY_ERR_CAPACITY;
  xy_plan_hand_out(plan, l, static_cast<XyDevUnit*>(records), lists);
  return XY_OK;
}
