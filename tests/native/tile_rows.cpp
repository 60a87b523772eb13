// How the plan asks the tile kernel for row groups of more than 16 rows: all row tiles in every wave only where there is such a
// kernel (one format for queries and cache, no e4m3, heads of 64 or, in bf16, of 128) and where it measured faster, by the bytes of
// the batch and the rows of its widest group.
#include <cstdio>
#include <vector>

#include "ps_internal.h"

static int check(int32_t head_dim, int32_t q, int32_t kv, int32_t requests, int64_t megabytes, bool want_spread, double share = 1) {
  const int64_t tile = int64_t(16) * head_dim, bytes = kv == PS_F32 ? 4 : kv == PS_BF16 ? 2 : 1;
  ps_geometry g{32, 8, head_dim, 16, q, kv, 16 * tile, 2 * tile, tile, head_dim};
  const double all = double(megabytes) * 1e6 / double(2 * 8 * head_dim * bytes);   // tokens, `share` of them in the context
  const int32_t tokens = int32_t(all * share);
  std::vector<int32_t> prompt(size_t(requests), 0), model, suffix(size_t(requests), int32_t(all * (1 - share) / requests));
  for (int32_t r = 0; r < requests; ++r) model.push_back(r);
  ps_pool* pool = nullptr;
  ps_layout* lay = nullptr;
  ps_plan_options opt{};
  opt.prefix_variant = opt.suffix_variant = PS_VARIANT_WAVE;
  bool ok = ps_pool_create(int32_t(all / 16) + requests + 2, nullptr, &pool) == PS_OK &&
            ps_kv_layout(pool, &g, 1, &tokens, requests, prompt.data(), model.data(), suffix.data(), &lay) == PS_OK &&
            ps_layout_replan(lay, &opt) == PS_OK;
  ok = ok && lay->tile_spread == want_spread;
  if (!ok) std::printf("FAILED: d = %d, formats %d / %d, %d rows, %lld MB\n", head_dim, q, kv, 4 * requests, (long long)megabytes);
  if (lay) ps_layout_release(pool, lay);
  if (pool) ps_pool_destroy(pool);
  return !ok;
}

int main() {
  int bad = 0;
  for (int32_t requests : {5, 8, 9, 16})   // 20 to 64 rows
    for (int64_t mb : {20, 60, 100, 135, 200, 500, 1500}) {
      const bool wide = requests > 8;
      for (int32_t d : {64, 128, 256})
        for (int32_t q : {PS_F32, PS_BF16})
          for (int32_t kv : {PS_F32, PS_BF16, PS_FP8_E4M3}) {
            bool spread = true;
            if (q == kv && d == 64) spread = kv == PS_F32 ? wide || mb <= 400 : mb <= (wide ? 45 : 65);
            if (q == kv && d == 128 && kv == PS_BF16) spread = mb <= 140;
            bad += check(d, q, kv, requests, mb, spread);
          }
    }
  for (int32_t d : {64, 128}) bad += check(d, PS_BF16, PS_BF16, 4, 1500, true);   // 16 rows
  // private segments beside the group
  bad += check(64, PS_BF16, PS_BF16, 8, 300, true, 0.3) + check(64, PS_BF16, PS_BF16, 8, 300, false, 0.36);
  bad += check(128, PS_BF16, PS_BF16, 16, 600, true, 0.3) + check(128, PS_BF16, PS_BF16, 16, 600, false, 0.36);
  bad += check(64, PS_F32, PS_F32, 8, 600, false, 0.2) + check(64, PS_F32, PS_F32, 16, 600, false, 0.4) + check(64, PS_F32, PS_F32, 16, 600, true, 0.6);
  bad += check(64, PS_F32, PS_F32, 8, 300, true, 0.2) + check(64, PS_BF16, PS_F32, 8, 300, true, 0.4);
  if (bad) return 1;
  std::puts("ok");
  return 0;
}
