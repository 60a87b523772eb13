// The order in which an ingest or a stage-in walks a layout's blocks, read from the table blob: by physical block within
// each shared kind, as stored for the private segments -- through park, replan or set_visible while parked, and resume.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <numeric>
#include <vector>

#include "ps_internal.h"

static void require(bool ok, const char* what, int blocks, int via) {
  if (ok) return;
  std::printf("FAILED: %s (blocks %d, via %d)\n", what, blocks, via);
  std::exit(1);
}

static std::vector<int32_t> order_of(const ps_layout* lay) {
  const int32_t* at = lay->blob.data() + lay->off_ent_order;
  return std::vector<int32_t>(at, at + lay->prefix_blk.size() + lay->suffix_blk.size() + lay->root_blk.size());
}

static std::vector<int32_t> expected(const ps_layout* lay) {
  std::vector<int32_t> out;
  auto by_id = [&](const std::vector<int32_t>& blk, bool sorted) {
    const int32_t first = int32_t(out.size());
    std::vector<int32_t> idx(blk.size());
    std::iota(idx.begin(), idx.end(), 0);
    if (sorted) std::stable_sort(idx.begin(), idx.end(), [&](int32_t a, int32_t b) { return blk[size_t(a)] < blk[size_t(b)]; });
    for (int32_t i : idx) out.push_back(first + i);
  };
  by_id(lay->prefix_blk, true);
  by_id(lay->suffix_blk, false);
  by_id(lay->root_blk, true);
  return out;
}

int main() {
  // 11 and 60 shared blocks on pools that they fill closely (laid out by id) and thinly (sorted)
  for (int32_t shared : {11, 60})
    for (int32_t pool_blocks : {4 * shared, 200 * shared})
      for (int via = 0; via < 3; ++via) {   // 0: nothing, 1: replan, 2: set_visible, while parked
        std::vector<int32_t> free_order(static_cast<size_t>(pool_blocks));
        for (int32_t i = 0; i < pool_blocks; ++i) free_order[size_t(i)] = int32_t((int64_t(i) * 7919 + 13) % pool_blocks);
        if (std::gcd(7919, pool_blocks) != 1) return 2;
        ps_pool* pool = nullptr;
        ps_layout* lay = nullptr;
        require(ps_pool_create(pool_blocks, free_order.data(), &pool) == PS_OK, "pool", shared, via);
        ps_geometry g{8, 2, 128, 16, PS_BF16, PS_BF16, 2 * 2 * 16 * 128, 2 * 16 * 128, 16 * 128, 128};
        const int32_t root_len[1] = {16 * 3 - 5}, prompt_root[2] = {0, -1}, prefix_len[2] = {16 * (shared / 2), 16 * (shared - shared / 2) - 3};
        const int32_t req_prompt[3] = {0, 0, 1}, req_model[3] = {0, 1, 0}, suffix_len[3] = {20, 0, 33}, visible[3] = {16, 5, 16};
        require(ps_kv_layout_tree(pool, &g, 1, root_len, 2, prompt_root, prefix_len, 3, req_prompt, req_model, suffix_len, &lay) == PS_OK,
                "layout", shared, via);
        require(order_of(lay) == expected(lay), "order of a fresh layout", shared, via);
        for (int round = 0; round < 2; ++round) {
          require(ps_layout_park(pool, lay) == PS_OK, "park", shared, via);
          if (via == 1) require(ps_layout_replan(lay, nullptr) == PS_OK, "replan", shared, via);
          if (via == 2) require(ps_layout_set_visible(lay, round ? nullptr : visible) == PS_OK, "set_visible", shared, via);
          if (via) {
            std::vector<int32_t> parked = order_of(lay);
            std::sort(parked.begin(), parked.end());
            for (size_t i = 0; i < parked.size(); ++i) require(parked[i] == int32_t(i), "parked order is no permutation", shared, via);
          }
          require(ps_layout_resume(pool, lay) == PS_OK, "resume", shared, via);
          require(order_of(lay) == expected(lay), "order after resume", shared, via);
        }
        require(ps_layout_release(pool, lay) == PS_OK && ps_pool_destroy(pool) == PS_OK, "release", shared, via);
      }
  std::puts("ok");
  return 0;
}
