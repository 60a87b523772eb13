// What the plan of a batch on standard input holds of short items that a wave takes alone.  Words: q heads, KV heads, head size, block,
// query and cache format, compute units, kernel families of the shared and the private segments, contexts, requests, the contexts'
// lengths, the requests' contexts, their private lengths.  Prints how many such items the whole step's schedule holds, how many the
// tile kernel's launch, and whether its row tiles are spread.
#include <cstdio>
#include <vector>

#include "ps_internal.h"

int main() {
  auto word = [] {
    int v = 0;
    if (std::scanf("%d", &v) != 1) v = -1;
    return v;
  };
  const int32_t q_heads = word(), kv_heads = word(), d = word(), block = word(), q = word(), kv = word();
  ps_plan_options opt{};
  opt.num_cus = word();
  opt.prefix_variant = word();
  opt.suffix_variant = word();
  const int32_t contexts = word(), requests = word();
  std::vector<int32_t> len, prompt, model, suffix;
  int64_t blocks = 1;
  for (int32_t p = 0; p < contexts; ++p) len.push_back(word());
  for (int32_t r = 0; r < requests; ++r) prompt.push_back(word());
  for (int32_t r = 0; r < requests; ++r) suffix.push_back(word());
  for (int32_t r = 0; r < requests; ++r) model.push_back(r);
  for (int32_t l : len) blocks += (l + block - 1) / block;
  for (int32_t l : suffix) blocks += (l + block - 1) / block;
  const int64_t tile = int64_t(block) * d;
  ps_geometry g{q_heads, kv_heads, d, block, q, kv, kv_heads * 2 * tile, 2 * tile, tile, d};
  ps_pool* pool = nullptr;
  ps_layout* lay = nullptr;
  if (ps_pool_create(int32_t(blocks), nullptr, &pool) != PS_OK ||
      ps_kv_layout(pool, &g, contexts, len.data(), requests, prompt.data(), model.data(), suffix.data(), &lay) != PS_OK ||
      ps_layout_replan(lay, &opt) != PS_OK)
    return 1;
  int64_t packed = 0;
  for (size_t w = 0; w < lay->pk_all.solo.size(); ++w) packed += lay->pk_all.indptr[w + 1] - lay->pk_all.solo[w];
  std::printf("%lld %d %d\n", (long long)packed, lay->num_solo_items, int(lay->tile_spread));
  ps_layout_release(pool, lay);
  ps_pool_destroy(pool);
  return 0;
}
