// Internal host-side structures shared by the layout/planner and the launch code.
#pragma once
#include <cstdint>
#include <deque>
#include <vector>

#include "prefillshare.h"

struct ps_pool {
  int32_t num_blocks = 0;
  std::deque<int32_t> free_list;
  std::vector<int32_t> refcount;
};

// One unit of attention work: a token range of one KV segment for one KV head, applied to the
// query rows of n_req requests (all G q heads of the head's group each).
struct ps_item {
  int32_t blk_off;      // index of the segment's first block in the concatenated block array
  int32_t tok_begin;
  int32_t tok_end;
  int32_t req_off;      // index of the first request in the request list
  int32_t n_req;
  int32_t kv_head;
  int32_t split_local;  // partial-state slot of request r is slot_base[r] + split_local
  int32_t kind;         // bit 0: 0 prefix, 1 suffix; bit 1: some row of the item sees less than tok_end
};
// bit 2: up to 256 rows, split over the waves of a workgroup by rows instead of by tokens (partial prefill)
// bit 3: a root segment (a context several prompts begin with), read by every request below the root
// bit 4: other items (further row groups of the same sharing group) read the same K/V range: keep it cacheable
constexpr int32_t kPsItemSuffix = 1, kPsItemMasked = 2, kPsItemRowSplit = 4, kPsItemRoot = 8, kPsItemReread = 16;
static_assert(sizeof(ps_item) == 32, "ps_item is 8 int32");

struct ps_layout {
  ps_geometry geo{};
  int32_t num_prompts = 0, num_requests = 0;
  std::vector<int32_t> prefix_len, suffix_len, req_prompt, req_model;
  std::vector<int32_t> prefix_blk_indptr, prefix_blk, group_indptr, group_req, suffix_blk_indptr, suffix_blk;
  // blocks adopted from another layout (the cached beginning of a prompt's prefix): adopt_indptr[P+1], ids; empty
  // when nothing is adopted.  They are the first blocks of the prompt's prefix list and are not written by ingest.
  std::vector<int32_t> adopt_indptr, adopt_blk;
  // parked: the blocks were handed back to the pool (their contents staged elsewhere by the caller); the block
  // arrays keep their shape but name no blocks until ps_layout_resume
  bool parked = false;
  // optional third level: roots (contexts several prompts begin with); prompt_root[p] = -1: none
  int32_t num_roots = 0;
  std::vector<int32_t> root_len, prompt_root, root_blk_indptr, root_blk, root_group_indptr, root_group_req;
  // per request: how many leading tokens of its prompt's prefix it attends to; empty = all of them
  std::vector<int32_t> visible;
  bool any_masked = false;           // the plan holds an item with kPsItemMasked
  // request list the items index into: group_req, then the identity list (suffix items), then root_group_req,
  // then the subsets of a sharing group that see into a prefix chunk (only where visible lengths cut a group)
  std::vector<int32_t> req_list;

  // split plan
  ps_plan_options opt{};
  int32_t num_cus = 0;               // compute units the plan spreads the work over
  int32_t prefix_variant = PS_VARIANT_WAVE, suffix_variant = PS_VARIANT_WAVE;
  int32_t prefix_chunk = 0, suffix_chunk = 0;
  int32_t max_rows_prefix = 0;       // largest n_req * G over prefix items
  std::vector<ps_item> items;        // row-split shared items, then the other shared (root, prefix) items, then suffix items
  int32_t rowsplit_rows = 256;       // most rows of a row-split item: the prefill kernel's workgroup takes 32 a wave
  int32_t num_rowsplit_items = 0;    // launched one workgroup each by the prefill kernel, outside the schedules
  bool tile_spread = true;           // tile kernel: row groups of more than 16 rows go a row tile to a wave
  int32_t solo_limit = 0;            // tile kernel: most tokens of a private item that a wave takes alone; 0: none does
  int32_t num_solo_items = 0;        // tile kernel: the last items, those within it
  int32_t num_prefix_items = 0;      // all shared items: root and prefix, row-split ones included
  // K/V loads of a launch over the shared / private / all items are non-temporal (little of its K/V is read by several)
  bool stream_prefix = true, stream_suffix = true, stream_all = true;
  std::vector<int32_t> slot_base;    // [R+1]
  int64_t num_slots = 0;
  int32_t max_states = 0;            // most slots of a request
  int64_t coarser_slots = -1;        // slots by the rules for fewer states (at least); -1: nothing to gain or no need
  // requests whose partial states ps_decode_attention has to merge: all but those with a single one that the prefill
  // kernel writes out itself; only filled (and in the blob) where there are such
  std::vector<int32_t> merge_req;
  bool any_direct = false;

  // persistent-kernel schedules: for a set of items, the items regrouped by workgroup (8 int32 each,
  // workgroup w owns [indptr[w], indptr[w+1])) -- one schedule per launchable set
  struct schedule {
    int64_t off_items = 0, off_indptr = 0;  // blob offsets in words
    int64_t off_solo = -1;  // int32[num_wg]: the workgroup's first item that a wave takes alone; -1: no such items
    int32_t num_wg = 0, max_rows = 0;
    bool stream = true;   // K/V loads of the launch are non-temporal (little of the set's K/V is read by several items)
  };
  schedule sched_prefix, sched_suffix, sched_all;
  // the schedules' contents as packed by the planner (copied into the blob; kept so that a decode step that changes
  // no chunk structure can patch token counts and block offsets instead of planning again)
  struct packed_set {
    std::vector<ps_item> items;
    std::vector<int32_t> indptr;
    std::vector<int32_t> solo;       // empty, or per workgroup where its solo items begin (see kPsSoloTokens)
    int64_t heaviest = 0, all = 0;   // cost of the heaviest workgroup, and of all, when it was packed (whole step's only)
    int32_t max_rows = 0, occ = 1;   // occ: workgroups per compute unit (ps_mfma_occupancy)
    bool stream = true;
  };
  packed_set pk_prefix, pk_suffix, pk_all;
  // per request: tokens per suffix chunk and number of suffix chunks in the current plan; where the root blocks
  // started in the concatenated block array when the plan was made
  std::vector<int32_t> suffix_chunk_size, suffix_chunks;
  int32_t planned_root_blk0 = 0;
  // upload staging (abi.hip): two pinned host buffers used alternately, so that ps_layout_upload returns as soon as
  // its copy is enqueued and the tables may change again right away; given to later layouts, or freed, with the layout
  struct upload_staging;
  mutable upload_staging* staging = nullptr;
  mutable void (*staging_free)(upload_staging*) = nullptr;
  ~ps_layout() {
    if (staging && staging_free) staging_free(staging);
  }
  // directory entries (first source token, valid tokens) of the shared segments' blocks: prefixes, then roots
  std::vector<int32_t> ent_fixed_tok0, ent_fixed_valid;
  // ... and the order in which an ingest walks them: by physical block, within each kind
  std::vector<int32_t> ent_fixed_order;

  // where the token of the most recent ps_layout_append went: block * B + slot per request, -1 = none
  std::vector<int32_t> append_dest;

  // device table blob (int32 words) and section offsets in words
  std::vector<int32_t> blob;
  int64_t off_blk = 0, off_req = 0, off_items = 0, off_slot = 0;
  int64_t off_merge = 0;             // merge_req
  int64_t off_visible = 0;           // int32[R]: effective visible prefix length of every request
  // for the cache-writing kernels, per entry of the concatenated block array: index of its first token in the
  // ragged source tensor of its kind (prefixes back to back / suffixes back to back) and its number of valid
  // tokens; then append_dest; then, per entry position, the entry an ingest or a stage-in takes there (every kind
  // keeps its range of positions)
  int64_t off_ent_tok0 = 0, off_ent_valid = 0, off_dest = 0, off_ent_order = 0;
};

// Waves per SIMD the MFMA kernel is built for, by the widest row group it must carry.
constexpr int ps_mfma_occupancy(int max_rows, int kv_dtype) {
  // two workgroups per compute unit where the kernel fits in 256 VGPRs: one 16-row tile, or e4m3 KV
  // (half-size tile buffers) with up to two
  if (max_rows <= 16) return 2;
  if (max_rows <= 32 && kv_dtype == PS_FP8_E4M3) return 2;
  return 1;
}
constexpr int kPsMfmaMaxChunk = 8192;  // tokens per MFMA work item (64 tiles per wave: their block ids fill two registers)
// Items short enough for one wave, four at a time in a workgroup, in the persistent and in the tile kernel (the rules and
// their figures are in build_plan).  Appends make private ones longer: in the tile kernel one that passes its limit is shared out
// over four waves again; a schedule of the persistent kernel is planned anew where a workgroup has come to have too much to do,
// and at the latest when such an item is half as long again as this (60 contexts of 200 to 1000 tokens under six models, 768 /
// 1000 private tokens: 236 / 298 us without such items, 240 / 303 with), well inside the 64 tiles of a wave.
constexpr int kPsSoloTokens = 512, kPsSoloTokensTile = 256;
static_assert(kPsSoloTokens * 3 / 2 <= kPsMfmaMaxChunk / 4, "a wave's own item holds up to 64 tiles of 32 tokens");
// Rows of such an item in the persistent kernel: what a wave fetches of the queries, by the row tiles the launch carries.
inline int ps_solo_rows(int max_rows) { return max_rows <= 32 ? 8 : 16; }

// A launch takes fewer than 2^32 threads a dimension: workgroups of 256.  The copies of whole blocks go out in ranges of entries
// that stay under it (a block's tile of a little over a piece is two pieces, so that a pool of 140 GB would pass it).
constexpr int64_t kMaxWorkgroups = (int64_t(1) << 24) - 1;
inline int64_t entries_per_launch(int64_t entries, int64_t pieces_per_entry, int64_t pieces_per_workgroup) {
  const int64_t most = kMaxWorkgroups * pieces_per_workgroup / pieces_per_entry;
  return entries <= most ? entries : most > 0 ? most : 1;
}

// Compute units of the current device, or 0 if none can be asked.  Null in a build without the device side of the
// library (the planner then assumes kPsDefaultNumCus); abi.hip installs it when the library is loaded.
extern int32_t (*ps_device_num_cus_hook)();
constexpr int32_t kPsDefaultNumCus = 256;   // MI355X
// Called when the last block pool is destroyed (abi.hip gives back what it keeps between layouts); null as above.
extern void (*ps_last_pool_hook)();

// layout.cpp
int32_t ps_plan_build(ps_layout* lay, const ps_plan_options* opt);
int32_t ps_blob_build(ps_layout* lay);
bool ps_mfma_supported(const ps_geometry& g);
