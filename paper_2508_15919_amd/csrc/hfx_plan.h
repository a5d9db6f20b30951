// Host planner interface (internal).  See hfx_plan.cpp.
#pragma once
#include <stddef.h>

#include <vector>

#include "../../include/hfxattn.h"
#include "hfx_desc.h"

namespace hfx {

// What the queue order needs of an item, side by side (the records themselves are 80 bytes apart).
struct ItemNote {
  uint32_t cost;
  uint32_t unit;     // of items that read the same keys (see the queue order in plan_step)
  float frac;        // of a prefill item: its row tile's place in the chunk, in [0, 1)
};

// The (request, kv-head) pairs of the prompts, as the queue per die cuts them.
struct Stream {
  uint32_t first, pieces;      // its pieces
  double work;                 // of one of them
};

struct Plan {
  std::vector<HfxReq> reqs;
  std::vector<HfxItem> items;
  std::vector<HfxGroup> groups;
  std::vector<HfxUnit> units;
  int32_t total_q = 0, n_bt = 0, n_partial_rows = 0, n_decode_items = 0, n_prefill_items = 0, n_runs = 0;
  int32_t queue_classes = 1;            // 1: plain queue; HFX_QUEUE_CLASSES: one list per die, interleaved by position
  int32_t die_items = 0;                // see HfxHeader
  int32_t deal_balanced = 0;            // see HfxHeader
  // scratch of plan_step, kept so that a reused Plan allocates nothing once it has grown
  std::vector<uint64_t> sort_keys;
  std::vector<uint32_t> order;          // queue position -> index into items
  std::vector<int32_t> split_cost;
  std::vector<uint32_t> order_dec, order_pre;
  std::vector<ItemNote> notes;          // of each item
  std::vector<int64_t> unit_cost;
  std::vector<uint32_t> unit_fill, unit_start;
  std::vector<uint64_t> unit_keys;
  std::vector<double> stream_ns;        // of each request with a prompt: time of the items that read the keys of one of its kv-heads
  std::vector<Stream> streams;          // of those, each kv-head
  std::vector<uint32_t> die_lists[HFX_QUEUE_CLASSES];
  std::vector<int32_t> queue;           // order in which items are taken, if it is not theirs; as many as items, or none
  std::vector<float> cut_cost, cut_sort, cut_load;   // trial of a cut: item times, sort scratch, CU loads
};

hfx_status check_shape(const hfx_shape* shape);
// sizes_only: the plan is good for layout_blob alone, its items are not put in order.
hfx_status plan_step(const hfx_shape* shape, int32_t num_requests, const int32_t* kind, const int32_t* q_len,
                     const int32_t* ctx_len, Plan* out, bool sizes_only = false);
void layout_blob(const hfx_shape* shape, const Plan& plan, HfxHeader* header);
hfx_status fill_blob(const hfx_shape* shape, Plan& plan, const int32_t* bt_indptr, const int32_t* bt_pages,
                     void* host_desc, size_t host_desc_bytes);

}  // namespace hfx
