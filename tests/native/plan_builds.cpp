// How often a batch is planned: once, and a second time only where that brings its partial states into the static workspace.
// (The planner asks for the compute units once per plan.)
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "ps_internal.h"

static int plans = 0;
static int32_t count_plans() {
  ++plans;
  return 256;
}

struct Batch {
  const char* what;
  int32_t q_heads, kv_heads, head_dim, block, q_dtype, kv_dtype, contexts, length, requests;
  bool causal;               // visible lengths: the last `requests` tokens of a context, one request each
  int32_t chunk;             // asked for, both kinds
  bool fits;
  int want;
};

int main() {
  ps_device_num_cus_hook = count_plans;
  const Batch batches[] = {
      {"a decode batch that fits", 32, 8, 128, 16, PS_BF16, PS_BF16, 8, 4096, 4, false, 0, true, 1},
      {"a float32 batch that fits", 32, 8, 128, 16, PS_F32, PS_F32, 8, 4096, 4, false, 0, true, 1},
      {"a partial prefill over the limit, cut coarsest already", 64, 8, 128, 16, PS_BF16, PS_FP8_E4M3, 20, 4100, 100, true, 0, false, 1},
      {"a float32 batch over the limit in chunks asked for", 32, 1, 128, 16, PS_F32, PS_F32, 8, 8000, 24, false, 128, false, 1},
      {"blocks of 24 tokens over the limit", 32, 1, 128, 24, PS_F32, PS_F32, 8, 8000, 64, false, 0, false, 1},
      {"a float32 batch over the limit either way", 32, 1, 128, 16, PS_F32, PS_F32, 8, 8000, 64, false, 0, false, 1},
      {"a float32 batch inside it with larger chunks", 32, 1, 128, 16, PS_F32, PS_F32, 8, 8000, 12, false, 0, true, 2},
  };
  for (const Batch& b : batches) {
    ps_pool* pool = nullptr;
    ps_layout* lay = nullptr;
    const int64_t tile = int64_t(b.block) * b.head_dim;
    ps_geometry g{b.q_heads, b.kv_heads, b.head_dim, b.block, b.q_dtype, b.kv_dtype, b.kv_heads * 2 * tile, 2 * tile, tile, b.head_dim};
    std::vector<int32_t> len(size_t(b.contexts), b.length), prompt, model, suffix(size_t(b.contexts) * size_t(b.requests), 0), visible;
    for (int32_t p = 0; p < b.contexts; ++p)
      for (int32_t m = 0; m < b.requests; ++m) {
        prompt.push_back(p);
        model.push_back(m);
        visible.push_back(b.length - b.requests + m + 1);
      }
    bool ok = ps_pool_create(b.contexts * (b.length / b.block + 2), nullptr, &pool) == PS_OK &&
              ps_kv_layout(pool, &g, b.contexts, len.data(), int32_t(prompt.size()), prompt.data(), model.data(), suffix.data(), &lay) == PS_OK;
    if (ok && b.causal) ok = ps_layout_set_visible(lay, visible.data()) == PS_OK;
    ps_plan_options opt{};
    opt.prefix_chunk_tokens = opt.suffix_chunk_tokens = b.chunk;
    plans = 0;
    ok = ok && ps_layout_replan(lay, &opt) == PS_OK;
    const bool fits = ps_workspace_bytes(lay) <= PS_STATIC_WORKSPACE_BYTES;
    if (!ok || fits != b.fits || plans != b.want) {
      std::printf("FAILED: %s: planned %d times, %.1f MiB\n", b.what, plans, double(ps_workspace_bytes(lay)) / (1 << 20));
      return 1;
    }
    ps_layout_release(pool, lay);
    ps_pool_destroy(pool);
  }
  std::puts("ok");
  return 0;
}
