// The schedule of a whole step is even: what its heaviest workgroup has to do, in half tiles -- an item of four waves takes
// ceil(tokens / 128) tiles and two more, four that a wave each takes half a tile for every 16 tokens of the longest and one more, two
// behind something else -- is what dealing them out heaviest first, each to the workgroup with the least to do, comes to.  And it stays so through a long turn: while every step
// makes the private segments longer the heaviest workgroup has no more than a quarter more to do than in a plan made afresh, and
// batch is not planned anew at every step for it.
#include <algorithm>
#include <cstdio>
#include <functional>
#include <queue>
#include <vector>

#include "ps_internal.h"

static int plans = 0;   // (the planner asks for the compute units once per plan)
static int32_t count_plans() {
  ++plans;
  return 256;
}

struct Turn {
  const char* what;
  int32_t q_heads, kv_heads, kv_dtype, contexts, shortest, longest, models;
};

// (lengths spread evenly, in an order that is not sorted)
static std::vector<int32_t> context_lengths(const Turn& t) {
  std::vector<int32_t> len;
  for (int32_t p = 0; p < t.contexts; ++p)
    len.push_back(t.shortest + int32_t(int64_t(t.longest - t.shortest) * ((7 * p) % t.contexts) / std::max(1, t.contexts - 1)));
  return len;
}

// Most half tiles of a workgroup; dealt: the same of these items and fours when dealt out by their half tiles.
static int64_t heaviest(const ps_layout* lay, int64_t* dealt) {
  const auto& pk = lay->pk_all;
  auto tiles = [](const ps_item& it, int64_t per) { return (it.tok_end - it.tok_begin + per - 1) / per; };
  struct unit { int64_t cost; bool four; };
  std::vector<unit> units;
  int64_t most = 0;
  for (size_t w = 0; w + 1 < pk.indptr.size(); ++w) {
    const int32_t first_solo = pk.solo.empty() ? pk.indptr[w + 1] : pk.solo[w];
    int64_t load = 0;
    for (int32_t i = pk.indptr[w]; i < first_solo; ++i) {
      units.push_back({2 * tiles(pk.items[size_t(i)], 128) + 4, false});
      load += units.back().cost;
    }
    for (int32_t i = first_solo; i < pk.indptr[w + 1]; i += 4) {
      int64_t longest = 0;
      for (int32_t k = i; k < std::min(i + 4, pk.indptr[w + 1]); ++k) longest = std::max(longest, tiles(pk.items[size_t(k)], 16));
      units.push_back({longest + 2, true});
      load += longest + (load ? 4 : 2);
    }
    most = std::max(most, load);
  }
  std::sort(units.begin(), units.end(), [](const unit& a, const unit& b) { return a.cost > b.cost; });
  std::priority_queue<int64_t, std::vector<int64_t>, std::greater<int64_t>> load;
  for (int w = 0; w < 256 * pk.occ; ++w) load.push(0);
  *dealt = 0;
  for (const unit& u : units) {
    const int64_t sum = load.top() + u.cost + (u.four && load.top() ? 2 : 0);
    load.pop();
    load.push(sum);
    *dealt = std::max(*dealt, sum);
  }
  return most;
}

static int fail(const Turn& t, int step, int64_t have, int64_t want) {
  std::printf("FAILED: %s: step %d: heaviest workgroup %lld half tiles, dealt out evenly %lld\n", t.what, step, (long long)have, (long long)want);
  return 1;
}

struct Batch {
  ps_pool* pool = nullptr;
  ps_layout* lay = nullptr;
  // `grow`: room for as many more tokens per request
  int make(const Turn& t, const std::vector<int32_t>& suffix, int32_t grow) {
    const int32_t n = t.contexts * t.models;
    const int64_t tile = 16 * 128;
    ps_geometry g{t.q_heads, t.kv_heads, 128, 16, PS_BF16, t.kv_dtype, t.kv_heads * 2 * tile, 2 * tile, tile, 128};
    const std::vector<int32_t> len = context_lengths(t);
    std::vector<int32_t> prompt, model;
    int32_t blocks = 0;
    for (int32_t p = 0; p < t.contexts; ++p) {
      blocks += (len[size_t(p)] + 15) / 16;
      for (int32_t m = 0; m < t.models; ++m) {
        blocks += (suffix[prompt.size()] + grow + 15) / 16 + 1;
        prompt.push_back(p);
        model.push_back(m);
      }
    }
    return ps_pool_create(blocks, nullptr, &pool) == PS_OK &&
           ps_kv_layout(pool, &g, t.contexts, len.data(), n, prompt.data(), model.data(), suffix.data(), &lay) == PS_OK;
  }
  ~Batch() {
    if (lay) ps_layout_release(pool, lay);
    if (pool) ps_pool_destroy(pool);
  }
};

// every: a request appends at every `every`-th step only, each at its own (1: all at every step)
static int run(const Turn& t, int every) {
  const int kSteps = 1100;
  const int32_t n = t.contexts * t.models;
  std::vector<int32_t> len(size_t(n), 0), active(size_t(n), 1);
  Batch batch;
  if (!batch.make(t, len, kSteps)) return fail(t, -1, 0, 0);
  int planned = 0;
  for (int step = 1; step <= kSteps; ++step) {
    for (int32_t r = 0; r < n; ++r) {
      active[size_t(r)] = (step + r) % every == 0 || step == 1;
      len[size_t(r)] += active[size_t(r)];
    }
    plans = 0;
    if (ps_layout_append(batch.pool, batch.lay, active.data(), nullptr) != PS_OK) return fail(t, step, 0, 0);
    planned += plans;
    int64_t dealt = 0, dealt_afresh = 0;
    const int64_t most = heaviest(batch.lay, &dealt);
    if (step == 1 && 10 * most > 11 * dealt) return fail(t, step, most, dealt);
    if (step % 50 && step > 8) continue;
    Batch afresh;
    if (!afresh.make(t, len, 0)) return fail(t, -1, 0, 0);
    const int64_t even = heaviest(afresh.lay, &dealt_afresh);
    if (4 * most > 5 * (even + 2)) return fail(t, step, most, even);   // (costs are rounded to tiles)
  }
  if (planned > 40) {
    std::printf("FAILED: %s: planned %d times in %d steps\n", t.what, planned, kSteps);
    return 1;
  }
  return 0;
}

// Lengths that hardly change: one request appends at a step.  No plan is due, also where the schedule could be more even.
static int stands_still(const Turn& t, int32_t shortest, int32_t longest) {
  const int32_t n = t.contexts * t.models;
  std::vector<int32_t> len, active(size_t(n), 0);
  for (int32_t r = 0; r < n; ++r) len.push_back(shortest + 37 * r % (longest - shortest + 1));
  Batch batch;
  if (!batch.make(t, len, 16)) return fail(t, -1, 0, 0);
  plans = 0;
  for (int step = 0; step < 40; ++step) {
    active[size_t(step % n)] = 1;
    if (ps_layout_append(batch.pool, batch.lay, active.data(), nullptr) != PS_OK) return fail(t, step, 0, 0);
    active[size_t(step % n)] = 0;
  }
  if (plans <= 4) return 0;
  std::printf("FAILED: %s: planned %d times in 40 steps of one request each\n", t.what, plans);
  return 1;
}

int main() {
  ps_device_num_cus_hook = count_plans;
  const Turn turns[] = {
      {"16 contexts, four models", 32, 8, PS_BF16, 16, 1024, 6144, 4},
      {"24 contexts, four models", 32, 8, PS_BF16, 24, 2000, 8000, 4},
      {"40 contexts, four models", 32, 8, PS_BF16, 40, 1024, 6144, 4},
      {"17 contexts, two models", 32, 8, PS_BF16, 17, 990, 3960, 2},
      {"16 contexts, four models, e4m3 under groups of eight", 64, 8, PS_FP8_E4M3, 16, 1024, 6144, 4},
      {"60 short contexts, six models", 32, 8, PS_BF16, 60, 200, 1000, 6},
      {"8 long contexts, four models", 32, 8, PS_BF16, 8, 8000, 16000, 4},
  };
  int bad = 0;
  for (const Turn& t : turns) bad += run(t, 1) + run(t, 3);
  bad += stands_still({"69 contexts, three models", 16, 4, PS_BF16, 69, 370, 542, 3}, 114, 280);
  bad += stands_still({"70 contexts, two models", 16, 4, PS_BF16, 70, 190, 1535, 2}, 180, 425);
  bad += stands_still({"37 contexts, three models, e4m3", 32, 4, PS_FP8_E4M3, 37, 360, 1885, 3}, 106, 422);
  bad += stands_still({"30 contexts, two models", 64, 8, PS_BF16, 30, 91, 1026, 2}, 102, 453);
  if (bad) return 1;
  std::puts("ok");
  return 0;
}
