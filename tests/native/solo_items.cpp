// Short items that a wave takes alone: which ones the schedules and the tile kernel's tail hold, and that appends never let one
// outgrow its limit.
#include <cstdio>
#include <vector>

#include "ps_internal.h"

static int fail(const char* what, int at) {
  std::printf("FAILED: %s (%d)\n", what, at);
  return 1;
}

// limit: of the tile kernel's items
static int run(int32_t q_heads, int32_t kv_heads, int32_t head_dim, int32_t dtype, const std::vector<int32_t>& contexts, int32_t models,
               const std::vector<int32_t>& lens, int32_t num_cus, bool want_solo, int32_t limit = kPsSoloTokens * 3 / 2) {
  const bool mfma = dtype != PS_F32 && head_dim == 128;
  const int32_t group = q_heads / kv_heads, n = int32_t(contexts.size()) * models;
  const int64_t tile = int64_t(16) * head_dim;
  ps_geometry g{q_heads, kv_heads, head_dim, 16, dtype == PS_F32 ? PS_F32 : PS_BF16, dtype, kv_heads * 2 * tile, 2 * tile, tile, head_dim};
  std::vector<int32_t> prompt, model, suffix, active(size_t(n), 1);
  int32_t blocks = 0;
  for (size_t p = 0; p < contexts.size(); ++p)
    for (int32_t m = 0; m < models; ++m) {
      prompt.push_back(int32_t(p));
      model.push_back(m);
      suffix.push_back(lens[suffix.size() % lens.size()]);
    }
  for (int32_t l : contexts) blocks += (l + 15) / 16;
  ps_pool* pool = nullptr;
  ps_layout* lay = nullptr;
  if (ps_pool_create(blocks + n * 140, nullptr, &pool) != PS_OK ||
      ps_kv_layout(pool, &g, int32_t(contexts.size()), contexts.data(), n, prompt.data(), model.data(), suffix.data(), &lay) != PS_OK)
    return fail("layout", 0);
  ps_plan_options opt{};
  opt.num_cus = num_cus;
  if (ps_layout_replan(lay, &opt) != PS_OK) return fail("plan", 0);
  for (int step = 0; step < 1300; ++step) {
    const auto& pk = lay->pk_all;
    if (mfma) {
      if (pk.solo.empty() == want_solo && step == 0) return fail("solo items", step);
      // (the kernel with four row tiles over e4m3 has no form for them)
      if (dtype == PS_FP8_E4M3 && !pk.solo.empty() && pk.max_rows > 32) return fail("four row tiles", step);
      for (size_t w = 0; w < pk.solo.size(); ++w) {
        if (pk.solo[w] < pk.indptr[w] || pk.solo[w] > pk.indptr[w + 1]) return fail("bounds", step);
        for (int32_t i = pk.solo[w]; i < pk.indptr[w + 1]; ++i) {
          const ps_item& it = pk.items[size_t(i)];
          if (it.tok_end - it.tok_begin > limit || it.n_req * group > ps_solo_rows(pk.max_rows) || (it.kind & kPsItemMasked)) return fail("item", step);
        }
      }
    } else {
      if ((lay->num_solo_items == 0) == want_solo && step == 0) return fail("solo items", step);
      for (size_t i = lay->items.size() - size_t(lay->num_solo_items); i < lay->items.size(); ++i) {
        const ps_item& it = lay->items[i];
        if (!(it.kind & kPsItemSuffix) || it.tok_end - it.tok_begin > limit || it.n_req * group > 16) return fail("item", step);
      }
      // (and all that are within it, whatever order the appends have left)
      for (size_t i = size_t(lay->num_prefix_items); i < lay->items.size() - size_t(lay->num_solo_items); ++i) {
        const ps_item& it = lay->items[i];
        if (it.tok_end - it.tok_begin <= lay->solo_limit) return fail("missed", step);
      }
    }
    // (every seventh request never grows)
    for (int32_t r = 0; r < n; ++r) active[size_t(r)] = r % 7 != 3;
    if (ps_layout_append(pool, lay, active.data(), nullptr) != PS_OK) return fail("append", step);
  }
  ps_layout_release(pool, lay);
  ps_pool_destroy(pool);
  return 0;
}

int main() {
  const std::vector<int32_t> lens{0, 1, 31, 32, 33, 255, 256, 257, 511, 512, 513, 700};
  if (int rc = run(32, 8, 128, PS_BF16, {2000, 600, 40}, 4, lens, 4, true)) return rc;
  if (int rc = run(64, 8, 128, PS_BF16, {2000, 600, 40}, 4, lens, 4, true)) return rc;
  if (int rc = run(28, 4, 128, PS_BF16, {2000, 600, 40}, 7, lens, 4, true)) return rc;
  if (int rc = run(64, 8, 128, PS_FP8_E4M3, {2000, 600, 40}, 12, lens, 4, true)) return rc;   // groups of more than 64 rows
  if (int rc = run(32, 2, 128, PS_FP8_E4M3, {2000, 600, 40}, 5, lens, 4, false)) return rc;
  if (int rc = run(48, 1, 128, PS_FP8_E4M3, {2000, 600, 40}, 5, lens, 1, false)) return rc;   // four row tiles
  if (int rc = run(16, 8, 128, PS_BF16, {300, 40, 520}, 1, lens, 4, true)) return rc;     // shared items of two rows
  if (int rc = run(32, 2, 128, PS_BF16, {300, 40, 520}, 1, lens, 1, false)) return rc;    // sixteen rows: more than a wave fetches
  if (int rc = run(32, 8, 128, PS_BF16, {2000}, 2, lens, 256, false)) return rc;          // fewer items than workgroups
  if (int rc = run(32, 8, 64, PS_BF16, {2000, 600, 40}, 4, lens, 4, true, 1024)) return rc;          // fours for every workgroup
  if (int rc = run(32, 8, 64, PS_BF16, {6000, 600, 40}, 4, lens, 16, true, 256)) return rc;
  if (int rc = run(16, 4, 256, PS_BF16, {2000, 600, 40}, 4, lens, 8, true, 512)) return rc;
  if (int rc = run(16, 4, 256, PS_F32, {2000, 600, 40}, 4, lens, 4, true, 128)) return rc;
  std::vector<int32_t> many_contexts;
  for (int32_t i = 0; i < 24; ++i) many_contexts.push_back(533 + 467 * i % 1600);
  if (int rc = run(8, 4, 256, PS_F32, many_contexts, 3, {40, 1, 64, 65, 128}, 256, true, 64)) return rc;   // 288 private items
  if (int rc = run(32, 1, 64, PS_F32, {2000, 600, 40}, 4, lens, 1, false)) return rc;     // thirty-two rows
  std::puts("ok");
  return 0;
}
