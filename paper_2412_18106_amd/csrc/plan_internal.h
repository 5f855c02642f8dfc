// Private layout of a plan object, shared by the host planner and the launcher.
#pragma once
#include <cstdint>
#include <utility>
#include <vector>

#include "xy_attn.h"

// Per-unit record read by the persistent kernel: the unit and what it has to know of its sequence, so that a
// wavefront goes from the unit's number to addresses with one 64-byte scalar load.
struct XyDevUnit {
  int32_t seq, head_begin, head_count, q_begin, q_count, kv_begin, kv_end, flags;
  int64_t ws_offset, mask_off;
  int32_t q_len, ctx_len, token_start, kv_head;
};
static_assert(sizeof(XyDevUnit) == 64, "one aligned scalar load");
// XyDevUnit::flags: kind and mask in the low bits; where wide units are on one row tile also the rows of the family's partial
// results and the unit's first row among them
constexpr int kSlabRowsShift = 8, kSlabFirstShift = 20;

constexpr int32_t kHalfRows = 128;          // most rows of a wide unit that four wavefronts of one row tile hold

// How a launch takes the units of a plan (layout.cpp).
struct XyLayout {
  int32_t records = 0;                      // units as they are handed out, second halves among them
  int32_t halved = 0;                       // units handed out as two halves
  int32_t row_tiles = 2;                    // of a wavefront on a wide unit
  int32_t team = 0;                         // wavefronts that share a narrow unit, 2 or 4; else 0
  int32_t depth = 2;                        // slices a wavefront keeps in flight on a narrow unit that is not short
  bool short_units = false;                 // narrow units are processed as short ones
};

// Per-sequence record read by the append kernel.
struct XyDevSeq {
  int32_t ctx_len, token_start;
};

// Up to kMergeRows rows of one K/V-split family, merged by one workgroup of the merge pass.
struct XyDevMergeRows {
  int64_t ws_offset;                        // the family's first partial
  int32_t rows, row_begin;                  // rows of the family; the first of this workgroup
  int32_t num_splits, token_begin;          // pieces; packed token index of the family's first token
  int32_t head_begin, head_count;
};

// Working arrays of the planner, kept between rebuilds so that planning a step allocates nothing once the
// object has seen a batch of that size.
struct XyPlanScratch {
  std::vector<xy_work_unit> fam;            // the units in the order they are made
  std::vector<int64_t> place;               // a unit's place in the order that breaks ties of the sort
  std::vector<uint64_t> key;                // a unit's cost, complemented
  std::vector<int32_t> order_tmp;
  std::vector<int32_t> order, worker_of, other_worker_of, count, cursor, chip_of_group;
  std::vector<int64_t> group_cost, by_cost;
  std::vector<std::pair<int64_t, int32_t>> heap;
  struct TileClass {
    int64_t nb, count, rows;                // K/V tiles; families (head groups); rows of a family
    bool prefill;
  };
  std::vector<TileClass> wide, narrow, may_cut;     // token tiles of more than 32 rows, of at most 32, those of them that may be cut
  std::vector<std::pair<int64_t, int64_t>> sizes, loads;
};

struct xy_attn_plan {
  xy_attn_config cfg;
  int32_t num_seqs = 0;
  int64_t total_tokens = 0;
  std::vector<xy_seq_desc> descs;
  std::vector<int32_t> token_start;
  std::vector<xy_work_unit> units;          // grouped by worker
  std::vector<int32_t> worker_offsets;      // W + 1
  std::vector<xy_merge_item> merges;
  int64_t workspace_floats = 0;
  int64_t merge_groups = 0;                 // workgroups of the merge pass (of the tables last copied to the GPU)
  int32_t free_workers = 0;                 // workers without units of their own (of the tables last copied to the GPU)
  XyLayout layout;                          // of the tables last copied to the GPU
  int32_t most_rows = 0;                    // most rows of a unit
  int64_t large_units = 0;                  // units of more than kHalfRows rows
  int32_t half_rows = 0;                    // most rows of the first half of one (half of its tokens, rounded up)
  int64_t narrow_units = 0, narrow_rows = 0, narrow_tiles = 0, narrow_slices = 0;     // units of at most 32 rows, their rows, K/V tiles and 32-key slices
  bool has_tree = false;
  XyPlanScratch scratch;
  // Device copy of the tables (owned): one arena on one device and a pinned staging buffer of the same size,
  // both kept and reused when the plan is rebuilt; the table pointers point into the arena.
  int device = -1;                          // device of the arena, -1 while there is none
  bool device_stale = true;                 // the host tables changed since they were last copied
  void* d_arena = nullptr;
  void* h_stage = nullptr;                  // pinned host memory the copy kernel reads from
  void* h_stage_dev = nullptr;              // the same memory as the device sees it
  size_t arena_capacity = 0;
  void* copied = nullptr;                   // hipEvent_t recorded behind the last copy: the staging buffer is free again after it
  void* d_units = nullptr;
  void* d_offsets = nullptr;
  void* d_seqs = nullptr;
  void* d_merges = nullptr;
  void* d_counters = nullptr;               // XY_ASSIGN_DYNAMIC: shared-list cursor and finished-workgroup counts (null without a shared list)
};

// layout.cpp; host only.  xy_plan_hand_out fills the tables of the unit kernel for the layout xy_plan_layout has just worked
// out: the records, and behind each other the workers' offsets (W + 1; the shared list follows the last worker's) and ranks
// (W; a worker's number among those that have no units of their own, -1 where it has some).  Returns how many have none.
XyLayout xy_plan_layout(const xy_attn_plan* plan);
int32_t xy_plan_hand_out(xy_attn_plan* plan, const XyLayout& layout, XyDevUnit* records, int32_t* offsets);
// Implemented in the HIP translation unit; frees the arena, the staging buffer and the event.
void xy_plan_free_device(xy_attn_plan* plan);
