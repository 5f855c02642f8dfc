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
// a lone wavefront pays for with 0.3 us, and gains where it waits for memory in every slice, with its neighbours idle.
// Decodes of 32 heads in 8, each a unit of its own, us short / two slices: 4 slices 7.1 / 7.3 (8 units), 9.3 / 9.2 (512),
// 24.4 / 24.7 (2048), 47.9 / 49.2 (4096); 1 and 2 slices 2 to 13 % less short; 8 slices 11.3 / 10.8, 14.5 / 13.6 up to a
// unit for every second wavefront, 22.4 / 22.5 at one each, 89.4 / 91.6 at four: so up to four slices a unit are short,
// up to eight where there are more units than wavefronts.  Units of 32 rows, whose Q is eight times as much: 4096 of them
// 42.1 / 44.8 with 2 slices, 66.4 / 65.7 with 4: up to two slices above 16 rows a unit.
constexpr int64_t kShortSlices = 4, kShortSlicesManyUnits = 8, kShortSlicesManyRows = 2, kManyRows = 16;
// Longer ones: two slices in flight up to kDeepTiles tiles a wavefront, one beyond (see process_solo; measured at 7.5
// tiles, 3 % in favour of two, and at 14, 1 % against).
constexpr int64_t kDeepTiles = 10;
// Units of more than kHalfRows rows that go to the GPU as two, by their tokens, for a worker each: all of them or none.
// The kernel then holds one row tile a wavefront instead of two, which takes two thirds of the time for units that are
// alone, but reads the K/V twice and keeps two workers busy: only where there are idle workers for all second halves, with a
// wavefront left for every narrow unit.  Unit kernel, us, whole / halves, 64 tokens x 4 heads, caches cold:
//   units   1 K/V tile       4              16             64
//   8       20.4 / 13.0      25.5 / 17.0    53.1 / 36.0
//   64      18.6 / 12.3      27.5 / 18.2    56.2 / 40.8    170 / 125
//   112     20.2 / 14.5      26.7 / 21.6    58.9 / 52.5    177 / 149
//   128     18.5 / 15.2      29.9 / 22.9    63.4 / 58.1    185 / 162    (every worker busy)
// and with fewer wavefronts left than narrow units the other way round (a suffix of 150-250 tokens beside 472 narrow units
// 254.9 -> 266.0 us for eight layers, a chunk of 512 beside 1184 157 -> 164 us).  The plan the caller sees stays as it is.
// A half is at most kHalfRows rows, so the tokens of a unit must divide: with 3, 5, 10, 12 and some other heads a group the
// default tile (256 / heads tokens: 85, 51, 25, 21) has a first half of 129 to 132 rows, and one such unit keeps the whole
// launch on two row tiles, without teams.
int32_t first_half(const xy_work_unit& u) { return (u.q_count + 1) / 2; }
// Wavefronts that share a narrow unit, for launches that have fewer such units than wavefronts: four while every unit can
// have a worker without wide units to itself, two while half of one, else none.  Unit kernel, us, one wavefront a unit / team (decodes of 32 heads
// in 8, caches cold):
//   units   2 slices (64 keys)    4            8            16           63
//   8       5.7 / 5.8             8.3 / 6.5    11.2 / 8.4   18.2 / 10.4  60.2 / 23.7
//   224     6.8 / 6.8             8.6 / 8.1    12.2 / 10.6  19.4 / 14.1  61.4 / 39.1
//   256     6.0 / 6.9             8.3 / 8.4    12.4 / 11.2  19.5 / 15.5  62.0 / 43.9
//   264     7.1 / 7.4 (two)       9.1 / 9.8    12.9 / 12.4  20.1 / 19.2  62.2 / 59.0
//   512     7.5 / 8.3             10.2 / 11.4  15.6 / 15.1  25.9 / 24.8  85.3 / 84.5
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
