// Host side of the library: block pool, the refcounted two-segment block table (ps_kv_layout) and
// the split plan.  Pure C++ -- no HIP calls -- so it is testable without a GPU.
//
// Sharing rule implemented here: a prompt's prefix blocks are allocated once and referenced by every
// request on that prompt (each decode module starts from the same base cache, Method Eq. 6), and
// only the model-specific segment is private (Efficiency Analysis Eq. 9).
#include <algorithm>
#include <atomic>
#include <cstdlib>
#include <cstring>
#include <map>
#include <tuple>
#include <new>
#include <numeric>
#include <queue>
#include <utility>

#include "ps_internal.h"

namespace {

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline int64_t round_up(int64_t a, int64_t b) { return ceil_div(a, b) * b; }

int32_t check_geometry(const ps_geometry& g) {
  if (g.num_q_heads <= 0 || g.num_kv_heads <= 0 || g.head_dim <= 0 || g.block_size <= 0) return PS_ERR_SHAPE;
  if (g.num_q_heads % g.num_kv_heads != 0) return PS_ERR_SHAPE;
  if (g.q_dtype != PS_F32 && g.q_dtype != PS_BF16) return PS_ERR_UNSUPPORTED;
  if (g.kv_dtype != PS_F32 && g.kv_dtype != PS_BF16 && g.kv_dtype != PS_FP8_E4M3) return PS_ERR_UNSUPPORTED;
  const int64_t esz = g.kv_dtype == PS_F32 ? 4 : (g.kv_dtype == PS_BF16 ? 2 : 1);
  const int64_t strides[4] = {g.kv_stride_block, g.kv_stride_head, g.kv_stride_kv, g.kv_stride_tok};
  for (int64_t s : strides)
    if (s <= 0 || (s * esz) % 16 != 0) return PS_ERR_SHAPE;
  if (g.kv_stride_tok < g.head_dim) return PS_ERR_SHAPE;
  return PS_OK;
}

}  // namespace

int32_t (*ps_device_num_cus_hook)() = nullptr;
void (*ps_last_pool_hook)() = nullptr;
static std::atomic<int64_t> live_pools{0};

bool ps_mfma_supported(const ps_geometry& g) {
  // The matrix-core kernels address a (block, head) slice through a buffer descriptor with 32-bit byte offsets
  // (V plane + token row + column), so the slice must span less than 2 GiB; a pool with K and V planes further
  // apart than that goes to the float32-probability family, which addresses the planes separately.
  const int64_t esz = g.kv_dtype == PS_BF16 ? 2 : 1;
  const int64_t slice_span = (g.kv_stride_kv + int64_t(g.block_size) * g.kv_stride_tok) * esz;
  return g.q_dtype == PS_BF16 && (g.kv_dtype == PS_BF16 || g.kv_dtype == PS_FP8_E4M3) && g.head_dim == 128 &&
         g.block_size % 16 == 0 && ((g.block_size / 16) & (g.block_size / 16 - 1)) == 0 &&  // 16, 32, 64, ...
         (g.num_q_heads / g.num_kv_heads) <= 64 && slice_span < (int64_t(1) << 31);
}

// What a workgroup of a schedule spends on an item that its waves share, in 64ths of a token, and on four that a wave each takes, by
// the longest of them, behind `before`.  Where there are fours, costs in time: an item of t tokens takes t / 128 + 2 tiles; a four, of
// whole 16-token blocks since a wave spends one on a single token, t / 32 + 1 and one more behind something else (the start of the
// first is one that the launch waits for anyway).  By tokens + 64 alone the fours looked like whole chunks (47 requests on 7
// contexts of 383 to 4074 tokens 24.8 us, 22.4 now; 54 on 11 of 136 to 1659 33.3, 28.1 now).  Four by their tokens, with one tile
// more for all of them or none / as here: 64 requests on 16 contexts of 1024 to 6144 tokens with one private token each 54.1 /
// 42.6 us, e4m3 under groups of eight 48.1 / 33.0, the 47 22.0 / 22.4, 160 on 40 contexts 99.7 / 101.4; no tile more for any, 301
// requests with up to 11 private tokens 206 against 201.6; for all, 46 on 13 of 173 to 564 21.2 against 17.5.  Equal ones by their
// tokens (155 requests on as many contexts of 9 to 157 tokens, 620 fours on 512 workgroups, 22.7 us, the first of the equal 26.2).
static int64_t shared_cost(bool fours, int64_t tokens) { return fours ? 64 * (round_up(tokens, 32) + 256) + tokens : 64 * (tokens + 64); }
static int64_t four_cost(int64_t longest, int64_t before) { return 64 * (4 * round_up(longest, 16) + (before ? 256 : 128)) + 4 * longest; }

// What a schedule comes to with its items as long as they are now: its heaviest workgroup, all together, the longest item that a
// wave takes alone, and what no schedule of these items avoids in some workgroup.
struct schedule_work { int64_t most = 0, all = 0, longest_solo = 0, unavoidable = 0; };
static schedule_work work_of(const ps_layout::packed_set& pk, int64_t num_cus) {
  schedule_work out;
  auto tokens = [&](int32_t i) { return int64_t(pk.items[size_t(i)].tok_end - pk.items[size_t(i)].tok_begin); };
  const bool fours = !pk.solo.empty();
  for (size_t w = 0; w + 1 < pk.indptr.size(); ++w) {
    const int32_t last = pk.indptr[w + 1], first_solo = fours ? pk.solo[w] : last;
    int64_t load = 0;
    for (int32_t i = pk.indptr[w]; i < first_solo; ++i) {
      load += shared_cost(fours, tokens(i));
      out.unavoidable = std::max(out.unavoidable, shared_cost(fours, tokens(i)));
    }
    for (int32_t i = first_solo; i < last; i += 4) {
      int64_t longest = 0;
      for (int32_t k = i; k < std::min(i + 4, last); ++k) longest = std::max(longest, tokens(k));
      load += four_cost(longest, load);
      out.longest_solo = std::max(out.longest_solo, longest);
      out.unavoidable = std::max(out.unavoidable, shared_cost(fours, longest));
    }
    out.most = std::max(out.most, load);
    out.all += load;
  }
  out.unavoidable = std::max(out.unavoidable, ceil_div(out.all, num_cus * pk.occ));
  return out;
}

// Whether the private segments have grown so far since the whole step's schedule was packed that it is worth planning anew: its
// heaviest workgroup has a quarter more to do than any schedule of these items makes unavoidable, and it has got a sixteenth more, or
// all together a hundredth, since (so that a batch that cannot be had more even is not planned at every step).  16 contexts
// of 1024 to 6144 tokens under four models, the plan of the first token kept / planned anew, after 128, 512 and 768 tokens 83 / 44,
// 202 / 58 and 281 / 72 us a launch (72, 121 and 159 with four waves on every item); a plan takes some 0.2 ms on the host.
static bool outgrown(const ps_layout* lay) {
  const ps_layout::packed_set& pk = lay->pk_all;
  const schedule_work now = work_of(pk, lay->num_cus);
  if (now.longest_solo > kPsSoloTokens * 3 / 2) return true;
  return 4 * now.most > 5 * now.unavoidable && (16 * now.most >= 17 * pk.heaviest || 100 * now.all >= 101 * pk.all);
}

// The tile kernel's short private items, which a wave takes alone, are the last of all; those that have grown past their limit go
// in front of them.
static void find_solo_items(ps_layout* lay) {
  auto too_long = [&](const ps_item& it) { return it.tok_end - it.tok_begin > lay->solo_limit; };
  if (std::any_of(lay->items.end() - lay->num_solo_items, lay->items.end(), too_long))
    std::stable_partition(lay->items.end() - lay->num_solo_items, lay->items.end(), too_long);
  lay->num_solo_items = 0;
  if (lay->solo_limit > 0)
    for (size_t i = lay->items.size(); i-- > size_t(lay->num_prefix_items) && !too_long(lay->items[i]);) ++lay->num_solo_items;
}

// ---------------------------------------------------------------------------------------------------
// Split plan: cut every segment into token chunks of (nearly) equal size, one workgroup each; a
// request's partial states are numbered prefix chunks first, then its suffix chunks.
// fewer_states: without the rules below that choose another chunk than a compute unit's share of the tokens for speed
// alone (see ps_plan_build).
static int32_t build_plan(ps_layout* lay, const ps_plan_options* user, bool fewer_states) {
  ps_plan_options opt{};
  if (user) opt = *user;
  if (opt.prefix_chunk_tokens < 0 || opt.suffix_chunk_tokens < 0 || opt.num_cus < 0) return PS_ERR_INVALID_ARG;
  auto bad_variant = [](int32_t v) { return v != PS_VARIANT_AUTO && v != PS_VARIANT_WAVE && v != PS_VARIANT_MFMA; };
  if (bad_variant(opt.prefix_variant) || bad_variant(opt.suffix_variant)) return PS_ERR_INVALID_ARG;
  if (opt.kv_cache_policy < PS_KV_POLICY_AUTO || opt.kv_cache_policy > PS_KV_POLICY_CACHEABLE) return PS_ERR_INVALID_ARG;
  const ps_geometry& g = lay->geo;
  const bool mfma_ok = ps_mfma_supported(g);
  if ((opt.prefix_variant == PS_VARIANT_MFMA || opt.suffix_variant == PS_VARIANT_MFMA) && !mfma_ok)
    return PS_ERR_UNSUPPORTED;
  const int32_t group = g.num_q_heads / g.num_kv_heads;
  // compute units to spread the work over: the caller's figure, else the current device's, else MI355X's
  int32_t num_cus = opt.num_cus;
  if (num_cus == 0 && ps_device_num_cus_hook) num_cus = ps_device_num_cus_hook();
  if (num_cus <= 0) num_cus = kPsDefaultNumCus;
  lay->num_cus = num_cus;

  // chunk boundaries fall on block boundaries and on the 32-token MFMA tile
  const int64_t granule = std::lcm<int64_t>(g.block_size, 32);
  int64_t total = 0;
  for (int32_t l : lay->prefix_len) total += l;
  for (int32_t l : lay->suffix_len) total += l;
  for (int32_t l : lay->root_len) total += l;
  total *= g.num_kv_heads;
  // Aim for about one full-size chunk per compute unit: long items amortise the per-item merge and keep
  // the number of partial states (workspace traffic) low; the many small suffix items fill the gaps.  Where the
  // kernel runs two workgroups per compute unit the aim is 0.6 of that, 1.2 times a workgroup's share: with
  // segments of unequal lengths the heaviest workgroups otherwise run on alone at the end of the launch (measured on
  // 20 to 60 concurrent sessions with contexts of 1024 to 6144 tokens: 2 to 10 % faster, none slower by more than
  // 0.5 %; any factor from 0.5 to 0.8 does about as well).
  // Shared segments of (nearly) equal lengths are cut as before: whole segments then pair up evenly on the compute
  // units by themselves, and the 4096-token prefixes of the 8B-shaped configuration are 2-3 % slower in halves.
  int32_t widest = group;   // rows of the widest item per KV head, for the kernel's residency
  {
    const int32_t cap = (g.kv_dtype == PS_FP8_E4M3 ? 32 : 64) / group;   // requests per item (see max_req below)
    for (size_t p = 0; p + 1 < lay->group_indptr.size(); ++p)
      widest = std::max(widest, std::min(std::max(1, cap), lay->group_indptr[p + 1] - lay->group_indptr[p]) * group);
    for (size_t t = 0; t + 1 < lay->root_group_indptr.size(); ++t)
      widest = std::max(widest, std::min(std::max(1, cap), lay->root_group_indptr[t + 1] - lay->root_group_indptr[t]) * group);
  }
  const bool two_per_cu = mfma_ok && ps_mfma_occupancy(widest, g.kv_dtype) == 2;
  int32_t shortest = INT32_MAX, longest = 0;   // of the shared segments
  for (int32_t l : lay->prefix_len) { shortest = std::min(shortest, l); longest = std::max(longest, l); }
  const bool unequal = longest > 0 && int64_t(longest) * 10 > int64_t(shortest) * 11;
  auto share_of = [&](bool two) { return std::max<int64_t>(1, ceil_div(two && unequal ? total * 3 / 5 : total, int64_t(num_cus))); };
  const int64_t ideal = share_of(two_per_cu);
  int64_t aim = ideal;   // of the persistent kernel's chunks: another where its items turn out narrower (see most_rows below)
  auto resolve = [&](int32_t v) { return v == PS_VARIANT_AUTO ? (mfma_ok ? PS_VARIANT_MFMA : PS_VARIANT_WAVE) : v; };
  // Row groups of more than 16 rows in the tile kernel: a wave per row tile (spread), where the waves of a tile's row groups
  // fetch it one after the other out of the caches, or all row tiles in every wave.  The first carries no more registers than
  // the 16-row kernel, so that two workgroups share a compute unit, and walks 64 rows in one pass; the second fetches every
  // line once, which pays where the launch streams from HBM and the products are cheap.  All row tiles a wave / spread, us
  // (batch, MB): d = 256 (passes of 16 rows there), bf16 276 MB 130 / 99, 1.5 GB 559 / 357, float32 552 MB 312 / 238, 267 MB 144 /
  // 144; d = 128, float32 463 MB 141 / 127, 555 MB 153 / 152, 1.2 GB 303 / 297, 279 MB 152 / 108, float32 queries over bf16 139 /
  // 119, 310 / 262, over e4m3 128 / 108; d = 64, e4m3 45 / 40, 35 / 34.
  // The other formats by the bytes of the whole batch, 24 or 32 rows and 56 or 64 rows a group on 8 to 40 contexts, spread against
  // all row tiles a wave: bf16, d = 128, 80 MB -11 to -8 and -14 to -11 %, 110 MB -4 to -2 and -9 to -3, 140 MB +1 to +3 and -2 to +6,
  // 170 MB +2 to +6 and -2 to +12, 280 MB +10 to +15 and +11 to +24; d = 64, 40 MB -13 to -11 and -5, 55 MB -5 to -3 and +3 to +4, 70 MB
  // +1 to +4 and +9 to +16, 140 MB +13 to +19 and +29 to +46; float32, d = 64, 300 MB -12 to -10 and -17 to -13, 400 MB -3 to +2 and
  // -15 to -13, 650 MB +1 to +6 and -16 to -13 (two passes in the form with all row tiles).
  // Where such groups hold under a quarter of the tokens (a short root, or private segments beside them), under a third in bf16,
  // the rest decides: 16-row items, two workgroups a compute unit and chunks for them (14 contexts of 2999 to 11998 tokens with
  // 64-wide heads under a root of 32: 44.0 -> 40.2 us).  Bf16 batches of 70 to 600 MB with private segments of 30 to 2000 tokens, d =
  // 64 and 128, against all row tiles a wave: 24 % of the tokens in such groups -38 to +5 %, 30 % -38 to +17, 39 % -35 to +21, 53 % -33 to
  // +32.  Float32 with 64-wide heads of more than 400 MB, 24 % -10 to +14 %, 30 % -12 to +21, 39 % -12 to +12; 53 % and more than 32 rows -11 to -1.
  int64_t wide_group_tokens = 0;
  for (size_t p = 0; p + 1 < lay->group_indptr.size(); ++p)
    if (int64_t(lay->group_indptr[p + 1] - lay->group_indptr[p]) * group > 16) wide_group_tokens += lay->prefix_len[p];
  for (size_t t = 0; t + 1 < lay->root_group_indptr.size(); ++t)
    if (int64_t(lay->root_group_indptr[t + 1] - lay->root_group_indptr[t]) * group > 16) wide_group_tokens += lay->root_len[t];
  const bool tile_bf16 = g.kv_dtype == PS_BF16 && g.q_dtype == PS_BF16;
  const bool tile_narrow = group <= 16 && (tile_bf16 ? 3 : 4) * wide_group_tokens * g.num_kv_heads < total;
  const int64_t kv_mb = total * 2 * g.head_dim * (g.kv_dtype == PS_F32 ? 4 : g.kv_dtype == PS_BF16 ? 2 : 1) / 1000000;
  if (tile_bf16 && g.head_dim != 256)
    lay->tile_spread = tile_narrow || kv_mb <= (g.head_dim != 64 ? 140 : widest <= 32 ? 65 : 45);
  else if (g.kv_dtype == PS_F32 && g.q_dtype == PS_F32 && g.head_dim == 64)
    lay->tile_spread = kv_mb <= 400 || (widest > 32 && 2 * wide_group_tokens * g.num_kv_heads >= total);
  else
    lay->tile_spread = true;   // (there is no other form)
  // The tile kernel (PS_VARIANT_WAVE, blocks of 16 k tokens) has a workgroup per item.  Heads of up to 128 with up to 16 rows
  // a wave leave room for two and more of them per compute unit: half a compute unit's share (measured, chunks of 1 / 0.5 / 0.25
  // of it: 36 float32 requests on 12 contexts of 512 to 4096 tokens 47.9 / 44.7 / 48.7 us, 72 bf16 requests with 64-wide
  // heads on 24 contexts of 1024 to 6144 tokens 51.2 / 44.5 / 43.1 us).  Where one is resident -- more rows a wave, or 256-wide
  // heads -- a second round only adds starts and states, and the share is a whole one (whole / half: bf16 queries over bf16
  // or e4m3 KV, groups of 20 to 64 rows on 8 to 60 contexts, d = 64 60.2 / 68.1, 31.0 / 34.9, 56.9 / 65.9, d = 128 84.1 /
  // 93.1, 42.9 / 45.3, 78.6 / 90.8 us; d = 256 26.8 / 34.7, 52.2 / 62.2, 85.0 / 92.9, in float32 44.7 / 56.3, 96.9 / 112,
  // 147 / 142, 236 / 229 us), but not with float32 products of up to 128: those are bound by the matrix cores, and the
  // finer cut evens the ends out (groups of 20 to 64 rows, d = 64 99.8 / 90.2, 50.5 / 40.9, 161 / 140, 114 / 122, d = 128 101 /
  // 83.3, 144 / 134, 296 / 291, 181 / 187, 172 / 187 us).  The vector kernel, which takes a pool that starts off a 16-byte
  // boundary with the same chunks, is faster with halves too (426 / 364, 170 / 134, 280 / 254, 280 / 230, 116 / 92 us).  At
  // least 128 tokens, one or two tiles per wave (two requests on one 256-token prompt, launches alone: chunks of 256 /
  // 128 / 64 tokens 9.4 / 7.9 / 7.7 us; contexts of some thousand tokens lose more in the merge than they gain).
  const bool tile_halves = g.head_dim < 256 && (widest <= 16 || tile_narrow || g.q_dtype == PS_F32 || g.kv_dtype == PS_F32);
  const int64_t tile_ideal = std::max<int64_t>(1, ceil_div(total, (tile_halves ? 2 : 1) * int64_t(num_cus)));
  auto pick = [&](int32_t asked, int32_t variant, bool fewer) -> int64_t {
    if (asked > 0) return round_up(asked, granule);
    const bool tiles = variant == PS_VARIANT_WAVE && g.block_size % 16 == 0 && !fewer;
    return std::min<int64_t>(std::max<int64_t>(round_up(tiles ? tile_ideal : fewer ? ideal : aim, granule), round_up(tiles ? 128 : 256, granule)),
                             round_up(kPsMfmaMaxChunk, granule));
  };
  const int64_t mfma_cap = std::max<int64_t>(granule, kPsMfmaMaxChunk / granule * granule);
  auto chunk_for = [&](int32_t asked, int32_t variant, bool fewer) {
    const int64_t chunk = pick(asked, variant, fewer);
    return variant == PS_VARIANT_MFMA ? std::min(chunk, mfma_cap) : chunk;
  };
  int64_t prefix_chunk = chunk_for(opt.prefix_chunk_tokens, resolve(opt.prefix_variant), fewer_states);
  int64_t suffix_chunk = chunk_for(opt.suffix_chunk_tokens, resolve(opt.suffix_variant), fewer_states);

  lay->opt = opt;
  lay->prefix_variant = resolve(opt.prefix_variant);
  lay->suffix_variant = resolve(opt.suffix_variant);

  // equal-sized chunks of a segment of `len` tokens: returns the chunk size used
  auto chunking = [&](int64_t len, int64_t chunk, int32_t* n) -> int64_t {
    if (len <= 0) { *n = 0; return chunk; }
    const int64_t count = ceil_div(len, chunk);
    const int64_t size = round_up(ceil_div(len, count), granule);
    *n = int32_t(ceil_div(len, size));
    return size;
  };
  // ... of a shared segment that goes to the prefill kernel: one that is only a little longer than a number of chunks
  // (by up to a quarter chunk) is not cut once more -- two halves of a context just over the aim cost an item, a
  // partial state per row and a merge more than they balance (partial-prefill batches whose contexts straddle the
  // aim: 7 % faster whole; decode batches of 60-80 sessions 1-2 % slower with the same rule, so they keep the plain
  // one).
  // (the prefill kernel walks a range of any length -- one scalar block id per tile -- so its items are not held to
  // the persistent kernel's 64 tiles per wave: the aim for them is the uncapped share, at most 32768 tokens)
  // The share is one of the work, which counts a range once per row group that walks it, wherever such groups hold most of
  // the batch's tokens: 160 new tokens with eight query rows each make five items per KV head and range, and cut by their
  // tokens alone the contexts went out in pieces of 256 tokens, each costing twelve tiles on top of its eight (batches of 1
  // to 44 contexts of 300 to 8500 tokens: 73.9 -> 42.8, 80.3 -> 48.7, 352 -> 276, 507 -> 441, 525 -> 432 us a step; shares of
  // 0.6 of this are slower again).
  int64_t wide_tokens = 0;
  for (size_t p = 0; p < lay->prefix_len.size(); ++p)
    if (int64_t(lay->group_indptr[p + 1] - lay->group_indptr[p]) * group > 64) wide_tokens += lay->prefix_len[p];
  for (size_t t = 0; t < lay->root_len.size(); ++t)
    if (int64_t(lay->root_group_indptr[t + 1] - lay->root_group_indptr[t]) * group > 64) wide_tokens += lay->root_len[t];
  wide_tokens *= g.num_kv_heads;
  const bool wide_shares = !lay->visible.empty() && resolve(opt.prefix_variant) == PS_VARIANT_MFMA &&
                           opt.prefix_chunk_tokens == 0 && 2 * wide_tokens > total && !fewer_states;
  auto wide_work = [&](int64_t rows_per_item, int64_t chunk) {   // tokens (chunk 0) or items of the wide groups, per KV head
    int64_t sum = 0;
    auto add = [&](int64_t len, int64_t reqs) {
      if (reqs * group <= 64 || len <= 0) return;
      const int64_t walks = ceil_div(reqs, std::max<int64_t>(1, rows_per_item / group));
      sum += walks * (chunk ? std::max<int64_t>(1, ceil_div(len - chunk / 4, chunk)) : len);   // (as chunking_shared cuts)
    };
    for (size_t p = 0; p < lay->prefix_len.size(); ++p) add(lay->prefix_len[p], lay->group_indptr[p + 1] - lay->group_indptr[p]);
    for (size_t t = 0; t < lay->root_len.size(); ++t) add(lay->root_len[t], lay->root_group_indptr[t + 1] - lay->root_group_indptr[t]);
    return sum;
  };
  auto wide_aim = [&](int64_t rows_per_item) {
    const int64_t share = std::max<int64_t>(1, ceil_div(wide_work(rows_per_item, 0) * g.num_kv_heads, int64_t(num_cus)));
    int64_t aim = std::max<int64_t>(round_up(share, granule), round_up(256, granule));
    // a few items more than compute units make a second round of the launch: larger pieces instead, up to half as large
    // again (264 items on 256 compute units 80.8 us, 168 larger ones 72.4 us)
    for (int64_t most = aim * 3 / 2; aim < most; aim = round_up(aim + aim / 16, granule)) {
      const int64_t items = wide_work(rows_per_item, aim) * g.num_kv_heads;
      if (items <= num_cus || 2 * items > 3 * int64_t(num_cus)) break;
    }
    return std::min<int64_t>(aim, round_up(32768, granule));
  };
  // Rows per item: 256, or 128 where the batch is nothing but wide groups and even those, in pieces of at most 512 tokens,
  // leave every item a compute unit of its own -- four waves, one per SIMD, then take a tile in less time than eight that
  // share the SIMDs (32 / 120 / 96 / 88 / 176 / 232 items of 256 rows against 56 / 224 / 176 / 136 / 256 / 236 of 128: 13.5 /
  // 14.6 / 15.1 / 23.6 / 27.8 / 30.9 us against 11.6 / 11.6 / 12.6 / 19.4 / 23.4 / 27.0).  With more items, or longer ones,
  // the tiles are fetched twice as often for nothing (376 items of 256 rows 29.6 us, 624 of 128 rows 31.1 us; 240 items of 28
  // tiles 47.1, 216 of 55 tiles 56.8 us).
  lay->rowsplit_rows = 256;
  if (wide_shares && wide_tokens == total && wide_aim(128) <= 512 && wide_work(128, wide_aim(128)) * g.num_kv_heads <= num_cus)
    lay->rowsplit_rows = 128;
  const int64_t token_share = std::min<int64_t>(std::max<int64_t>(round_up(ideal, granule), round_up(256, granule)), round_up(32768, granule));
  const int64_t wide_chunk = opt.prefix_chunk_tokens > 0 ? prefix_chunk : wide_shares ? wide_aim(lay->rowsplit_rows) : token_share;
  auto chunking_shared = [&](int64_t len, int64_t chunk, int32_t* n) -> int64_t {
    if (len <= 0) { *n = 0; return chunk; }
    if (opt.prefix_chunk_tokens > 0) return chunking(len, chunk, n);   // a chunk size the caller asked for is taken as it is
    const int64_t count = std::max<int64_t>(1, ceil_div(len - chunk / 4, chunk));
    const int64_t size = round_up(ceil_div(len, count), granule);
    *n = int32_t(ceil_div(len, size));
    return size;
  };

  const int32_t P = lay->num_prompts, R = lay->num_requests;
  // Visible prefix lengths (partial prefill: a query row may see only the leading part of its prompt's shared
  // prefix).  A request takes part in the prefix chunks that begin below its visible length, so its prefix splits
  // are the first ceil(visible / chunk size) of its prompt's; an item's token range ends at the largest visible
  // length among its rows, and it is marked where some row sees less than that.
  const bool limited = !lay->visible.empty();
  auto visible_of = [&](int32_t r) { return limited ? lay->visible[size_t(r)] : lay->prefix_len[size_t(lay->req_prompt[size_t(r)])]; };
  std::vector<int32_t> nsplit_root(R, 0), nsplit_prefix(R), nsplit_suffix(R);
  lay->suffix_chunk_size.assign(size_t(R), 0);
  lay->suffix_chunks.assign(size_t(R), 0);
  std::vector<ps_item> prefix_items, suffix_items;
  const bool prefix_mfma = resolve(opt.prefix_variant) == PS_VARIANT_MFMA;
  // The prefill kernel runs one workgroup per item, one item per compute unit at a time, and its items are long: with
  // a few items per compute unit the last round of the launch is badly filled (704 items of 132 tiles on 256 compute
  // units: three rounds for the work of 2.75).  The contexts whose items come last -- the shortest, the launch goes
  // heaviest first -- are therefore cut into more pieces, as many as fill the last round best; the others stay whole
  // (one partial state per row).
  std::vector<int32_t> tail_cut(size_t(P), 1);
  if (limited && prefix_mfma && opt.prefix_chunk_tokens == 0) {
    struct wide_prompt { int32_t p; int64_t items, tiles; };
    std::vector<wide_prompt> wp;
    int64_t n_items = 0, work = 0;
    for (int32_t p = 0; p < P; ++p) {
      const int64_t reqs = lay->group_indptr[p + 1] - lay->group_indptr[p];
      if (reqs * group <= 64 || lay->prefix_len[p] <= 0) continue;
      int32_t n0 = 0;
      const int64_t size0 = chunking_shared(lay->prefix_len[p], wide_chunk, &n0);
      const int64_t per_item = std::max(1, lay->rowsplit_rows / group);
      const wide_prompt e{p, ceil_div(reqs, per_item) * g.num_kv_heads * n0, ceil_div(std::min<int64_t>(size0, lay->prefix_len[p]), 32)};
      wp.push_back(e);
      n_items += e.items;
      work += e.items * e.tiles;
    }
    if (n_items > 0) {
      const int64_t mean_tiles = std::max<int64_t>(1, work / n_items);
      const int64_t rounds = work / num_cus / mean_tiles;          // rounds the whole items fill completely
      const int64_t rest = n_items - rounds * num_cus;             // items of the last, partly filled round
      // time of the last round in tiles, an item costing about twelve tiles beyond its own (launch, the dependent
      // reads of its start, filling the ring, its stores; measured: pieces of 33 tiles gained nothing on 132-tile items)
      constexpr int64_t kItemOverheadTiles = 12;
      int64_t best_cut = 1, best_cost = INT64_MAX, whole_cost = 0;
      for (int64_t cut : {1, 2, 3, 4, 6, 8}) {
        if (mean_tiles / cut < 16) break;                          // pieces of at least 512 tokens
        const int64_t cost = ceil_div(rest * cut, int64_t(num_cus)) * (ceil_div(mean_tiles, cut) + kItemOverheadTiles);
        if (cut == 1) whole_cost = cost;
        if (cost < best_cost) { best_cost = cost; best_cut = cut; }
      }
      // (worth it from 3 % of a compute unit's work on: the pieces cost their rows a partial state and a merge each)
      if (rest > 0 && best_cut > 1 && (whole_cost - best_cost) * 100 >= 3 * (work / num_cus)) {
        std::stable_sort(wp.begin(), wp.end(), [](const wide_prompt& x, const wide_prompt& y) { return x.tiles < y.tiles; });
        int64_t taken = 0;
        for (size_t i = 0; i < wp.size() && taken < rest; ++i) {
          tail_cut[size_t(wp[i].p)] = int32_t(best_cut);
          taken += wp[i].items;
        }
      }
    }
  }
  auto seen_by = [&](int32_t p, int64_t token) {   // requests that see past a token of their prompt's prefix
    int64_t count = 0;
    for (int32_t i = lay->group_indptr[p]; i < lay->group_indptr[p + 1]; ++i) count += visible_of(lay->group_req[size_t(i)]) > token;
    return count;
  };
  // how a prompt's prefix is cut: the tokens of a chunk, and how many there are
  auto cut_prefix = [&](int32_t p, int32_t* n) -> int64_t {
    const int32_t g0 = lay->group_indptr[p], g1 = lay->group_indptr[p + 1];
    const bool wide = limited && prefix_mfma && int64_t(g1 - g0) * group > 64;   // goes to the prefill kernel
    int64_t size = wide ? chunking_shared(lay->prefix_len[p], wide_chunk, n) : chunking(lay->prefix_len[p], prefix_chunk, n);
    if (wide && tail_cut[size_t(p)] > 1 && *n > 0) {
      size = round_up(ceil_div(int64_t(lay->prefix_len[p]), int64_t(*n) * tail_cut[size_t(p)]), granule);
      *n = int32_t(ceil_div(int64_t(lay->prefix_len[p]), size));
    }
    if (size > mfma_cap && prefix_mfma) {
      // chunks longer than the persistent kernel's items hold are fine only while every one of them goes to the
      // prefill kernel: a chunk that too few requests see into (64 rows or fewer) would be an ordinary item
      for (int32_t c = 0; c < *n && size > mfma_cap; ++c)
        if (seen_by(p, c * size) * group <= 64) size = chunking(lay->prefix_len[p], prefix_chunk, n);
    }
    return size;
  };
  // Rows an item carries per KV head: up to 64 (four row tiles).  With e4m3 KV a sharing group is cut at 32 rows where
  // the matrix-core kernel runs: the two-tile kernel keeps two workgroups per compute unit and measured 19 % faster
  // on 64-row groups than the four-tile one (bf16 KV the other way round: the four-tile kernel is 9-12 % faster).
  const bool narrow_items = g.kv_dtype == PS_FP8_E4M3 && prefix_mfma;
  int32_t most_rows = narrow_items ? 32 : 64;
  // Where a batch leaves the chip idle its row groups go out in narrower items: an item is one workgroup, and what bounds a small
  // launch is that workgroup's time, which the rows make longer -- in the tile kernel a row tile to a wave, so that each wave walks
  // all of the tokens (four of them share the tokens of a 16-row item), in the persistent kernel all row tiles in every wave, and
  // above 16 (e4m3: 32) rows only one workgroup on a compute unit.  The K/V is then read once per 16 rows, out of the caches.  64 (e4m3
  // on the persistent kernel: 32) / 16 rows, us a step: float32, 256-wide heads, 3 contexts of 85 to 171 tokens, 6 to 26 new ones
  // 42.5 / 18.5; float32, 1 of 262 to 525, 76 rows 25.0 / 12.3; 256-wide, 2 of 264 to 528, 60 rows 21.6 / 12.4; 64-wide, 3 of 94 to
  // 188, 160 rows 12.0 / 8.8; persistent kernel, 28 query on 4 KV heads, 56 and 30 rows on small contexts 17.0 / 9.9, 17.1 / 10.2, 64 on 8,
  // 64 rows on 4 15.4 / 9.9, e4m3, 24 rows 13.0 / 11.0.
  // The line lies where the items of 16 rows, private ones too, still have a compute unit each: 256-wide heads, 256 items 23.5 /
  // 14.1, 244 16.4 / 13.5, 360 19.6 / 20.6, 364 24.6 / 22.1 (32 rows: 18.5), 432 27.7 / 36.0; 64-wide, 228 12.3 / 9.2, 492 20.2 / 22.1, 526
  // 19.2 / 21.3; two of them with float32 products of up to 128, which are bound by the matrix cores (272 items 24.0 / 14.1, 352 24.8 /
  // 16.5, 560 25.3 / 20.4, 608 26.6 / 22.7); in the persistent kernel, where short private ones go four to a workgroup, five to four
  // (280 items 13.0 / 11.0, 312 13.4 / 11.8, 328 17.1 / 18.6, 424 20.1 / 20.7, 888 18.1 / 20.1).  32 rows by the same line, in the persistent
  // kernel up to two a compute unit (352 items 20.3 / 16.1, 464 66.2 / 62.4, 552 62.3 / 63.6).
  // And where the wide groups are few of the tokens (a short root), whatever the size: a launch without them runs the 16-row form
  // everywhere (19 contexts of 1733 tokens under a root of 1030, 256-wide heads 59.9 / 40.4; 5 of 17613, 64-wide 25.7 / 20.9; e4m3, 13.9 /
  // 11.8; not float32 of up to 128: 92.4 / 93.5).
  // Groups of 2 to 8 query heads were measured, and groups of one (20 to 64 requests a context, 40 batches of the three kinds 7 to 46 %
  // faster: bf16, 8 heads, 48 on one of 340 16.0 / 12.3; float32, 48 on one of 660 23.9 / 13.0); a request of 16 rows fills a tile alone.
  if (opt.prefix_chunk_tokens == 0 && group <= 8 && (prefix_mfma || g.block_size % 16 == 0)) {
    // What goes out in ordinary items: in a batch with visible lengths the prefill kernel takes the groups of more than 64 rows,
    // but not their chunks that few requests see into.
    struct shared_range { int64_t tokens, chunks, reqs; };
    std::vector<shared_range> ranges;
    ranges.reserve(size_t(lay->num_roots) + size_t(P));
    int64_t longest_item = 0;   // tokens
    for (int32_t t = 0; t < lay->num_roots; ++t) {
      const int64_t reqs = lay->root_group_indptr[size_t(t) + 1] - lay->root_group_indptr[size_t(t)];
      int32_t n = 0;
      const int64_t size = chunking(lay->root_len[size_t(t)], prefix_chunk, &n);
      if (limited && prefix_mfma && reqs * group > 64) continue;
      ranges.push_back({lay->root_len[size_t(t)], n, reqs});
      longest_item = std::max(longest_item, std::min<int64_t>(size, lay->root_len[size_t(t)]));
    }
    for (int32_t p = 0; p < P; ++p) {
      const int64_t reqs = lay->group_indptr[size_t(p) + 1] - lay->group_indptr[size_t(p)], len = lay->prefix_len[size_t(p)];
      int32_t n = 0;
      const int64_t size = cut_prefix(p, &n);
      if (!limited) {
        ranges.push_back({len, n, reqs});
        longest_item = std::max(longest_item, std::min(size, len));
        continue;
      }
      for (int32_t c = 0; c < n; ++c) {
        const int64_t count = seen_by(p, c * size);
        if (count == 0 || (prefix_mfma && count * group > 64)) continue;
        ranges.push_back({std::min(size, len - c * size), 1, count});
        longest_item = std::max(longest_item, ranges.back().tokens);
      }
    }
    struct shared_work { int64_t items = 0, tokens = 0; };   // with items of at most that many rows
    auto shared_at = [&](int32_t rows) {
      shared_work w;
      for (const shared_range& s : ranges) {
        const int64_t walks = ceil_div(s.reqs, std::max(1, rows / group)) * g.num_kv_heads;
        w.items += s.chunks * walks;
        w.tokens += s.tokens * walks;
      }
      return w;
    };
    int64_t own = 0;
    for (int32_t r = 0; r < R; ++r) own += ceil_div(lay->suffix_len[size_t(r)], suffix_chunk) * g.num_kv_heads;
    const bool float_products = !prefix_mfma && g.head_dim < 256 && (g.q_dtype == PS_F32 || g.kv_dtype == PS_F32);
    const int64_t room16 = prefix_mfma ? int64_t(num_cus) * 5 / 4 : int64_t(num_cus) * (float_products ? 2 : 1);
    const int64_t room32 = prefix_mfma ? int64_t(num_cus) * 2 : room16;
    const shared_work as_is = shared_at(most_rows), at16 = shared_at(16);
    const bool few_tokens = !float_products && as_is.tokens > 0 && 8 * at16.tokens <= 9 * as_is.tokens;
    // Not into a second round that the wide items do not need: where the persistent kernel's narrow ones outnumber the compute units
    // and the wide ones do not, the launch lasts two items (or one that shares its compute unit) instead of one.  Shared items wide /
    // narrow, us a step wide / narrow: 24 rows in 16, 256 / 288 of 2656 tokens 57.9 / 79.8, 252 / 294 of 832 23.8 / 29.9, 240 / 280 of 352
    // 14.9 / 17.7, of 256 and less the other way round (92 / 276 18.1 / 14.0); 35 to 64 rows in 32, 204 / 408 of 256 18.7 / 21.9, 240 / 300 of
    // 832 27.5 / 34.6, 256 / 320 of 3840 88.7 / 115.5; partial prefill, the prefill kernel's items counted in, 464 / 712 of 8100 252 / 418, 376
    // / 544 of 6208 182 / 251.  For 32 rows the line lies where the wide items and the private ones are no more than 9/8 of the compute
    // units (118 batches 15 % slower narrow, none faster), and a sixteenth of these is idle (256 and 32 private ones 30.7 / 17.8): beyond
    // it the narrow form gains about as often as it loses, but with items of more than 2048 tokens, and so it does in a partial prefill.
    // (What counts there is the rows that see into a chunk, not those of the whole group.)
    auto second_round = [&](const shared_work& narrow, int32_t rows) {
      if (!prefix_mfma || narrow_items || narrow.items <= num_cus || as_is.items > num_cus) return false;
      if (rows == 16) return longest_item > round_up(256, granule);
      return longest_item > 2048 || (!limited && 8 * (as_is.items + own) <= 9 * int64_t(num_cus) && 16 * as_is.items <= 15 * int64_t(num_cus));
    };
    // (few tokens of a batch with many private items beside them: the 16-row form everywhere gains more than the round costs; 256 /
    // 264 shared items, 536 / 544 in all 34.8 / 27.8, 256 / 320, 656 / 720 32.6 / 25.6; 282 / 314 39.2 / 47.9, 304 / 336 57.9 / 79.8)
    const bool again16 = second_round(at16, 16);
    if ((few_tokens && !(again16 && !unequal && 4 * (as_is.items + own) <= 5 * int64_t(num_cus))) || (at16.items + own <= room16 && !again16)) {
      most_rows = 16;
    } else if (most_rows > 32) {
      const shared_work at32 = shared_at(32);
      if (at32.items + own <= room32 && !second_round(at32, 32)) most_rows = 32;
    }
    // Two workgroups of the persistent kernel on a compute unit where the wide items had left room for one: chunks for two, as above.
    // Cut for the wide items / for two, us a step: under a root, 10 contexts of 2857 to 11430 tokens and eight models 55.3 / 45.2, 44 of 752
    // to 12047 153.7 / 141.3, 6 of 5357 to 21428 81.7 / 61.4; 405 batches with a share of 2048 tokens and more 11 % faster in the mean
    // (7 of them 1 to 6 % slower).  With a smaller share only where the items are few, up to nine to four compute units (45 batches 0 to
    // 25 % faster) or three to two: many small segments even out by themselves, and a finer cut adds states (43 of 160 to 2566 under a
    // root of 49, 40.2 / 42.8; 132 of 23 to 378 21.7 / 24.3).
    const int64_t share = ceil_div(total, int64_t(num_cus)), items16 = at16.items + own;
    const bool coarse = share >= 2048 || (share >= 1200 && 4 * items16 <= 9 * int64_t(num_cus)) || (share >= 800 && 2 * items16 <= 3 * int64_t(num_cus));
    if (most_rows == 16 && prefix_mfma && !limited && !fewer_states && !two_per_cu && ps_mfma_occupancy(most_rows, g.kv_dtype) == 2 && coarse) {
      aim = share_of(true);
      prefix_chunk = chunk_for(opt.prefix_chunk_tokens, resolve(opt.prefix_variant), false);
      suffix_chunk = chunk_for(opt.suffix_chunk_tokens, resolve(opt.suffix_variant), false);
    }
  }
  lay->prefix_chunk = int32_t(prefix_chunk);
  lay->suffix_chunk = int32_t(suffix_chunk);
  const int32_t max_req = std::max(1, most_rows / group);
  const int32_t total_prefix_blocks = int32_t(lay->prefix_blk.size());
  lay->max_rows_prefix = 0;
  lay->any_masked = false;
  lay->req_list.assign(lay->group_req.begin(), lay->group_req.end());
  for (int32_t r = 0; r < R; ++r) lay->req_list.push_back(r);
  lay->req_list.insert(lay->req_list.end(), lay->root_group_req.begin(), lay->root_group_req.end());
  // Root segments: read whole by every request below the root (all models of all its prompts), so the sharing group
  // is large.  In a decode batch it goes out in ordinary items of at most 64 rows, packed into the one persistent
  // launch with everything else (the root's K/V is then fetched once per 64 rows, mostly from the last-level cache;
  // a separate launch for a handful of root items would leave most of the chip idle while it runs).  In a
  // partial-prefill batch (visible lengths set) large groups go to the prefill kernel, roots included.
  const int32_t root_blk0 = int32_t(lay->prefix_blk.size() + lay->suffix_blk.size());   // roots close the block array
  lay->planned_root_blk0 = root_blk0;
  for (int32_t t = 0; t < lay->num_roots; ++t) {
    int32_t n = 0;
    const int32_t g0 = lay->root_group_indptr[size_t(t)], count = lay->root_group_indptr[size_t(t) + 1] - g0;
    const bool wide = limited && prefix_mfma && int64_t(count) * group > 64;
    // (a root is seen whole by every request below it, so all its chunks go the same way)
    const int64_t size = wide ? chunking_shared(lay->root_len[size_t(t)], wide_chunk, &n) : chunking(lay->root_len[size_t(t)], prefix_chunk, &n);
    for (int32_t i = 0; i < count; ++i) nsplit_root[size_t(lay->root_group_req[size_t(g0 + i)])] = n;
    const bool row_split = limited && prefix_mfma && int64_t(count) * group > 64;
    const int32_t per_item = row_split ? std::max(1, lay->rowsplit_rows / group) : max_req;
    // Row groups outside, KV heads inside: items of equal cost reach the workgroups in this order (LPT, lowest
    // index on ties) and workgroup i runs on XCD i mod 8, so with a multiple of eight KV heads the row groups that
    // read one (range, head) start together on one XCD and share its L2.
    for (int32_t c = 0; c < n; ++c)
      for (int32_t m0 = 0; m0 < count; m0 += per_item)
        for (int32_t h = 0; h < g.num_kv_heads; ++h) {
          ps_item it{};
          it.blk_off = root_blk0 + lay->root_blk_indptr[size_t(t)];
          it.tok_begin = int32_t(c * size);
          it.tok_end = int32_t(std::min<int64_t>(lay->root_len[size_t(t)], (c + 1) * size));
          it.req_off = 2 * R + g0 + m0;
          it.n_req = std::min(per_item, count - m0);
          it.kv_head = h;
          it.split_local = c;
          it.kind = kPsItemRoot | (row_split ? kPsItemRowSplit : 0) | (count > per_item ? kPsItemReread : 0);
          if (!row_split) lay->max_rows_prefix = std::max(lay->max_rows_prefix, it.n_req * group);
          prefix_items.push_back(it);
        }
  }
  std::vector<int32_t> members;
  for (int32_t p = 0; p < P; ++p) {
    int32_t n = 0;
    const int32_t g0 = lay->group_indptr[p], g1 = lay->group_indptr[p + 1];
    const int64_t size = cut_prefix(p, &n);
    for (int32_t i = g0; i < g1; ++i) {
      const int32_t r = lay->group_req[size_t(i)];
      nsplit_prefix[size_t(r)] = int32_t(ceil_div(visible_of(r), size));
    }
    for (int32_t c = 0; c < n; ++c) {
      // the requests that see into this chunk, in group order: the whole group unless lengths were limited
      int32_t list0 = g0, count = g1 - g0;
      if (limited) {
        members.clear();
        for (int32_t i = g0; i < g1; ++i)
          if (visible_of(lay->group_req[size_t(i)]) > c * size) members.push_back(lay->group_req[size_t(i)]);
        count = int32_t(members.size());
        if (count != g1 - g0) {
          list0 = int32_t(lay->req_list.size());
          lay->req_list.insert(lay->req_list.end(), members.begin(), members.end());
        }
      }
      // Partial prefill on the matrix cores: a sharing group with more rows than one 64-row item holds (the new
      // tokens of a context) goes out in items of up to 256 rows, which the prefill kernel splits over its waves
      // by rows, so that a K/V tile is fetched once per 256 rows instead of once per 64.
      const bool row_split = limited && prefix_mfma && int64_t(count) * group > 64;
      const int32_t per_item = row_split ? std::max(1, lay->rowsplit_rows / group) : max_req;
      for (int32_t m0 = 0; m0 < count; m0 += per_item)      // row groups outside, heads inside (see the roots)
        for (int32_t h = 0; h < g.num_kv_heads; ++h) {
          ps_item it{};
          it.blk_off = lay->prefix_blk_indptr[p];
          it.tok_begin = int32_t(c * size);
          it.req_off = list0 + m0;
          it.n_req = std::min(per_item, count - m0);
          int32_t v_max = 0, v_min = INT32_MAX;
          for (int32_t i = 0; i < it.n_req; ++i) {
            const int32_t v = visible_of(lay->req_list[size_t(it.req_off + i)]);
            v_max = std::max(v_max, v);
            v_min = std::min(v_min, v);
          }
          it.tok_end = int32_t(std::min<int64_t>(std::min<int64_t>(lay->prefix_len[p], (c + 1) * size), v_max));
          it.kv_head = h;
          it.split_local = c;   // the root's splits are added below, once every request's count is known
          it.kind = (v_min < it.tok_end ? kPsItemMasked : 0) | (row_split ? kPsItemRowSplit : 0) |
                    (count > per_item ? kPsItemReread : 0);
          if (it.kind & kPsItemMasked) lay->any_masked = true;
          if (!row_split) lay->max_rows_prefix = std::max(lay->max_rows_prefix, it.n_req * group);
          prefix_items.push_back(it);
        }
    }
  }
  for (int32_t r = 0; r < R; ++r) {
    int32_t n = 0;
    const int64_t size = chunking(lay->suffix_len[r], suffix_chunk, &n);
    nsplit_suffix[r] = n;
    lay->suffix_chunk_size[size_t(r)] = int32_t(size);
    lay->suffix_chunks[size_t(r)] = n;
    for (int32_t c = 0; c < n; ++c)
      for (int32_t h = 0; h < g.num_kv_heads; ++h) {
        ps_item it{};
        it.blk_off = total_prefix_blocks + lay->suffix_blk_indptr[r];
        it.tok_begin = int32_t(c * size);
        it.tok_end = int32_t(std::min<int64_t>(lay->suffix_len[r], (c + 1) * size));
        it.req_off = R + r;  // identity part of the request list
        it.n_req = 1;
        it.kv_head = h;
        it.split_local = nsplit_root[size_t(r)] + nsplit_prefix[size_t(r)] + c;
        it.kind = kPsItemSuffix;
        suffix_items.push_back(it);
      }
  }
  // a request's partial states: root splits, then prefix splits, then suffix splits (every request of a prefix item
  // is on the same prompt, hence below the same root)
  for (ps_item& it : prefix_items)
    if (!(it.kind & kPsItemRoot)) it.split_local += nsplit_root[size_t(lay->req_list[size_t(it.req_off)])];
  auto by_cost = [](const ps_item& a, const ps_item& b) { return (a.tok_end - a.tok_begin) > (b.tok_end - b.tok_begin); };
  auto rs_first = [&](const ps_item& a, const ps_item& b) {   // row-split items lead, heaviest (tokens x rows) first
    const bool ra = a.kind & kPsItemRowSplit, rb = b.kind & kPsItemRowSplit;
    if (ra != rb) return ra;
    if (ra) return int64_t(a.tok_end - a.tok_begin) * a.n_req > int64_t(b.tok_end - b.tok_begin) * b.n_req;
    return by_cost(a, b);
  };
  if (!std::is_sorted(prefix_items.begin(), prefix_items.end(), rs_first)) std::stable_sort(prefix_items.begin(), prefix_items.end(), rs_first);
  if (!std::is_sorted(suffix_items.begin(), suffix_items.end(), by_cost)) std::stable_sort(suffix_items.begin(), suffix_items.end(), by_cost);
  lay->num_rowsplit_items = 0;
  for (const ps_item& it : prefix_items) lay->num_rowsplit_items += (it.kind & kPsItemRowSplit) ? 1 : 0;
  if (lay->num_rowsplit_items > 8) {
    // XCD-aware launch order of the prefill kernel.  Workgroup i of a launch runs on XCD i mod 8, and each XCD has
    // its own L2.  The row groups that read the same K/V range (same segment, token begin and KV head: a family)
    // are therefore placed eight apart, on one XCD, and next to each other in that XCD's sequence, so that they run
    // at the same time and the range comes out of HBM once instead of once per row group.  Families go, heaviest
    // first, to the XCD with the fewest items so far.
    const int n_rs = lay->num_rowsplit_items;
    typedef std::tuple<int32_t, int32_t, int32_t> range_key;             // (segment, token begin, KV head)
    std::map<range_key, size_t> family_of;
    std::vector<std::vector<ps_item>> family;                             // in order of first (= heaviest) member
    for (int i = 0; i < n_rs; ++i) {
      const ps_item& it = prefix_items[size_t(i)];
      const auto at = family_of.emplace(range_key{it.blk_off, it.tok_begin, it.kv_head}, family.size());
      if (at.second) family.emplace_back();
      family[at.first->second].push_back(it);
    }
    std::vector<std::vector<ps_item>> column(8);
    for (const auto& members : family) {
      size_t target = 0;
      for (size_t c = 1; c < 8; ++c)
        if (column[c].size() < column[target].size()) target = c;
      column[target].insert(column[target].end(), members.begin(), members.end());
    }
    int out = 0;
    for (size_t row = 0; out < n_rs; ++row)
      for (size_t c = 0; c < 8; ++c)
        if (row < column[c].size()) prefix_items[size_t(out++)] = column[c][row];
  }
  // (what the persistent kernel is given must fit its per-wave tile directory; the cuts above see to it)
  if (prefix_mfma)
    for (const ps_item& it : prefix_items)
      if (!(it.kind & kPsItemRowSplit) && it.tok_end - it.tok_begin > mfma_cap) return PS_ERR_INVALID_ARG;
  // Short private items of the tile kernel go four to a workgroup as well, a wave each, where the items are more than two
  // rounds of the workgroups that are resident together (their last waves would otherwise end the launch: 736 items in 1.4
  // rounds, float32, private segments of 1 to 256 tokens, 44.7 us without, 46 / 47.8 / 55.7 with those of up to 64 / 128 /
  // 256).  Without and with (longest 64 / 128 / 256 tokens): 64-wide heads, 310 requests with up to 12 private tokens 21.9 /
  // 14.7 / 14.7 / 14.7 us, 72 with up to 256 43.5 / 43.9 / 43.7 / 42.2; 256-wide, 659 with up to 119 163 / 143 / 131 / 131, in
  // float32 147 with up to 142 56.0 / 54.8 / 48.9 / 50.4.  Float32 tokens are twice the bytes: half as many (171 requests with up
  // to 190 on 70 short contexts 45.8 / 45.4 / 46.0 / 54.2, 159 with up to 514 72.0 / 72.3 / 73.2 / 76.5; 525 with up to 160 127 /
  // 120 / 116 / 111).
  // Bf16 queries, longer ones, without / with: beyond 256 tokens only where the fours alone fill the resident workgroups (64-wide
  // heads, 60 contexts of 200 to 1000 tokens under six models, 384 / 512 / 1000 private tokens 97.6 / 76.2, 114 / 91.4, 163 / 148
  // us, with e4m3 43.3 / 39.1, 52.7 / 46.5, 89.7 / 88.3; 256-wide heads 168 / 158, 201 / 193, 296 / 311), since they end a shorter
  // launch (64-wide heads, 24 contexts of 1024 to 6144 tokens under four models 42.8 / 48.0, 48.7 / 55.0, 62.8 / 77.6, 90 of 300 to
  // 1500 with sixteen rows 37.4 / 40.5, 40.4 / 44.6, 55.8 / 56.2; though 12 of 500 to 3000 under eight 30.4 / 25.4, 36.5 / 29.0).
  // Half as long with 256-wide heads where the private items are not many more than the resident workgroups, which would have one
  // each and be done sooner (without / 64 / 128 / 256: float32, 72 requests with up to 145 on 24 contexts of 533 to 2132 tokens 70.2 /
  // 68.2 / 81.2, bf16, 71 with up to 188 on 18 46.1 / 45.6 / 44.8 / 48.3; but 64-wide heads, the 72 with up to 256 40.0 / 38.8).
  lay->solo_limit = 0;
  {
    const int rows = std::max(group, lay->max_rows_prefix);
    const int resident = g.head_dim == 256 || (rows > 16 && !lay->tile_spread) ? 1 : 2;
    if (lay->suffix_variant == PS_VARIANT_WAVE && g.block_size % 16 == 0 && group <= 16 &&
        int64_t(prefix_items.size() + suffix_items.size()) > 2 * int64_t(num_cus) * resident) {
      const bool many = g.q_dtype == PS_BF16 && int64_t(suffix_items.size()) >= 4 * int64_t(num_cus) * resident;
      lay->solo_limit = g.kv_dtype == PS_F32 ? kPsSoloTokensTile / 2 : !many ? kPsSoloTokensTile : g.head_dim == 64 ? 1024 : 512;
      if (g.head_dim == 256 && 3 * int64_t(suffix_items.size()) < 4 * int64_t(num_cus) * resident) lay->solo_limit /= 2;
    }
  }
  lay->num_prefix_items = int32_t(prefix_items.size());
  lay->items = std::move(prefix_items);
  lay->items.insert(lay->items.end(), suffix_items.begin(), suffix_items.end());
  lay->num_solo_items = 0;
  find_solo_items(lay);

  lay->slot_base.assign(R + 1, 0);
  lay->max_states = 0;
  int64_t slots = 0;
  for (int32_t r = 0; r < R; ++r) {
    slots += nsplit_root[r] + nsplit_prefix[r] + nsplit_suffix[r];
    if (slots > INT32_MAX) return PS_ERR_INVALID_ARG;
    lay->slot_base[r + 1] = int32_t(slots);
    lay->max_states = std::max(lay->max_states, lay->slot_base[r + 1] - lay->slot_base[r]);
  }
  lay->num_slots = slots;
  // What the rules for fewer states would leave, where they are others than the ones that were followed: the states by
  // their chunk sizes alone (the last round's extra cut of the prefill launch can only add to them).
  lay->coarser_slots = -1;
  const int64_t coarse_prefix = chunk_for(opt.prefix_chunk_tokens, lay->prefix_variant, true);
  const int64_t coarse_suffix = chunk_for(opt.suffix_chunk_tokens, lay->suffix_variant, true);
  if (!fewer_states && (wide_shares || coarse_prefix != prefix_chunk || coarse_suffix != suffix_chunk) &&
      ps_workspace_bytes(lay) > PS_STATIC_WORKSPACE_BYTES) {
    const int64_t coarse_wide = opt.prefix_chunk_tokens > 0 ? coarse_prefix : token_share;
    lay->coarser_slots = 0;
    int32_t n = 0;
    for (int32_t t = 0; t < lay->num_roots; ++t) {
      const int64_t count = lay->root_group_indptr[size_t(t) + 1] - lay->root_group_indptr[size_t(t)];
      if (limited && prefix_mfma && count * group > 64) chunking_shared(lay->root_len[size_t(t)], coarse_wide, &n);
      else chunking(lay->root_len[size_t(t)], coarse_prefix, &n);
      lay->coarser_slots += n * count;
    }
    for (int32_t p = 0; p < P; ++p) {
      const int32_t g0 = lay->group_indptr[p], g1 = lay->group_indptr[p + 1];
      const bool wide = limited && prefix_mfma && int64_t(g1 - g0) * group > 64;
      const int64_t size = wide ? chunking_shared(lay->prefix_len[p], coarse_wide, &n) : chunking(lay->prefix_len[p], coarse_prefix, &n);
      for (int32_t i = g0; i < g1; ++i) lay->coarser_slots += ceil_div(visible_of(lay->group_req[size_t(i)]), size);
    }
    for (int32_t r = 0; r < R; ++r) {
      chunking(lay->suffix_len[r], coarse_suffix, &n);
      lay->coarser_slots += n;
    }
  }
  // A request whose only partial state comes from the prefill kernel needs no merge in a whole step: the kernel rounds
  // and stores the row itself.
  std::vector<char> direct(size_t(R), 0);
  lay->any_direct = false;
  for (int32_t i = 0; i < lay->num_rowsplit_items; ++i) {
    const ps_item& it = lay->items[size_t(i)];
    for (int32_t m = 0; m < it.n_req; ++m) {
      const int32_t r = lay->req_list[size_t(it.req_off + m)];
      if (lay->slot_base[size_t(r) + 1] - lay->slot_base[size_t(r)] == 1) direct[size_t(r)] = 1;
    }
  }
  lay->merge_req.clear();
  for (char d : direct) lay->any_direct |= d != 0;
  if (lay->any_direct)
    for (int32_t r = 0; r < R; ++r)
      if (!direct[size_t(r)]) lay->merge_req.push_back(r);

  // Schedules for the persistent MFMA kernel: longest-processing-time-first packing of a set of items
  // onto the resident workgroups (cost = tokens + a fixed per-item charge), each list longest first.
  typedef ps_layout::packed_set packed;
  // Cache policy of a launch: K/V that one item reads is best streamed past the caches, K/V that several row
  // groups read (kPsItemReread) should stay in them.  The policy is per launch, so it goes by the share of the
  // set's tokens that lie in re-read items: streaming while that is under a quarter (measured: a root shared by 8
  // row groups next to 3/4 of ordinary traffic gains 1.5 % from streaming, two row groups per prompt at 46 % of
  // the tokens lose 5 %).
  // In the tile kernel so is a range that several row tiles fetch, or several passes (24-row groups, 256-wide heads, streamed /
  // cacheable 37.0 / 29.9, 128 / 114, 50.4 / 39.8 us; where they hold a few of the tokens beside private segments, float32, 110 /
  // 121, 132 / 144 us).
  const int32_t rows_at_once = lay->tile_spread ? 16 : g.head_dim == 64 && g.kv_dtype == PS_BF16 ? 64 : 32;
  auto fetched_again = [&](const ps_item& it) {
    const int32_t variant = (it.kind & kPsItemSuffix) ? lay->suffix_variant : lay->prefix_variant;
    return (it.kind & kPsItemReread) != 0 || (variant == PS_VARIANT_WAVE && it.n_req * group > rows_at_once);
  };
  auto streams = [&](int begin, int end) {
    int64_t tokens_all = 0, tokens_reread = 0;
    for (int i = begin; i < end; ++i) {
      const ps_item& it = lay->items[size_t(i)];
      tokens_all += it.tok_end - it.tok_begin;
      if (fetched_again(it)) tokens_reread += it.tok_end - it.tok_begin;
    }
    return opt.kv_cache_policy == PS_KV_POLICY_AUTO ? 4 * tokens_reread < tokens_all
                                                     : opt.kv_cache_policy == PS_KV_POLICY_STREAM;
  };
  auto pack = [&](int begin, int end, bool solo_allowed) {
    packed out;
    const int count = end - begin;
    for (int i = begin; i < end; ++i) out.max_rows = std::max(out.max_rows, lay->items[size_t(i)].n_req * group);
    out.occ = ps_mfma_occupancy(out.max_rows, g.kv_dtype);
    out.stream = streams(begin, end);
    std::vector<int> order(size_t(count), 0);
    std::iota(order.begin(), order.end(), begin);
    auto cost = [&](int i) { return int64_t(lay->items[size_t(i)].tok_end - lay->items[size_t(i)].tok_begin) + 64; };
    auto heavier = [&](int a, int b) { return cost(a) > cost(b); };
    // the shared items and the suffix items are each in descending cost already; a range that spans both is the
    // stable merge of two sorted runs
    const int split = std::min(std::max(lay->num_prefix_items, begin), end) - begin;
    if (!std::is_sorted(order.begin(), order.begin() + split, heavier)) std::stable_sort(order.begin(), order.begin() + split, heavier);
    if (!std::is_sorted(order.begin() + split, order.end(), heavier)) std::stable_sort(order.begin() + split, order.end(), heavier);
    if (split > 0 && split < count) std::inplace_merge(order.begin(), order.begin() + split, order.end(), heavier);
    // Short items go four to a workgroup, one per wave (which fetches up to ps_solo_rows of query rows): the waves then neither
    // share out a few tiles each nor meet to merge them, and a workgroup passes a quarter of the item boundaries.  Only where
    // the items outnumber the workgroups: where each has one, a wave alone takes longer (four models on one context of 2741
    // tokens, private segments of 1 to 256: 15.1 -> 18.8 us).  Measured, whole steps, longest such item 0 / 256 / 512 / 1024
    // tokens: 256 prompts of 512 to 16384 tokens under 2 to 6 models, private 1 to 1024, 1179 / 1170 / 1160 / 1155 us; 52 of
    // 20843, private 1 to 537, 739 / 722 / 703 / 705; 40 of 1024 to 6144, private 1 to 256, 118.2 / 115.6 / 115.5 / 115.5; e4m3,
    // 64 of 8192, private 1 to 512, 219.3 / 217.8 / 215.5 / 215.7; 162 requests with up to 7 private tokens on 114 contexts
    // 78.4 / 71.9; 87 requests on as many contexts of 147 tokens (two rows: the shared items too) 22.7 / 18.0.
    // A short launch takes shorter ones only: a wave's time with an item (some t / 32 + 1 tiles) is to stay under 7/8 of what a
    // workgroup has to do (t / 128 + 2 tiles for an item of four waves; 32 requests on 17 contexts of 990 to 3960 tokens, 0 / 64 /
    // 128 / 512: 33.2 / 32.4 / 29.4 / 41.4 us; 46 on 13 of 141 to 566 24.1 / 21.7 / 18.3 / 21.2).  And the
    // four-row-tile kernel, whose registers this overflows further, only where the short items are a good part of the work or
    // the launch is a long one (205 requests with a few private tokens on 31 contexts 34.0 -> 31.0 us a launch; 81 on 52 contexts
    // of 20843 tokens 723 -> 702 a step, 174 on 53 of 1180 to 18892 370 -> 351; but 39 on 16 of 2015 to 8060 68.7 -> 72.9).
    int64_t work = 0, solo_tokens = 0;
    for (int i = begin; i < end; ++i) work += cost(i) + 192;
    // (nor where one item is more than 5/4 of a workgroup's share of the work, and the launch waits for it whatever becomes of
    // the rest: its tiles take a little longer in the kernel that has both forms; 32 contexts of 4096 tokens on 512 workgroups,
    // an item each and 16 tokens of private ones, 108.6 -> 111.3)
    if (solo_allowed && !lay->any_masked && count > num_cus * out.occ && 4 * (cost(order[0]) + 192) <= 5 * (work / (num_cus * out.occ)))
      solo_tokens = std::min<int64_t>(kPsSoloTokens, std::max<int64_t>(32, (work / (num_cus * out.occ) * 7 / 8 - 128) / 4));
    auto solo = [&](int i) {
      const ps_item& it = lay->items[size_t(i)];
      return it.tok_end - it.tok_begin <= solo_tokens && it.n_req * group <= ps_solo_rows(out.max_rows);
    };
    if (out.max_rows > 32 && work < int64_t(kPsMfmaMaxChunk) * num_cus * out.occ && 4 * 256 * std::count_if(order.begin(), order.end(), solo) < work) solo_tokens = 0;
    const int n_full = solo_tokens == 0 ? count : int(std::stable_partition(order.begin(), order.end(), [&](int i) { return !solo(i); }) - order.begin());
    struct unit { int64_t cost; int first, count; };   // of `order`
    std::vector<unit> units;
    units.reserve(size_t(count));
    for (int n = 0; n < n_full; ++n) units.push_back({shared_cost(n_full < count, cost(order[size_t(n)]) - 64), n, 1});
    for (int n = n_full; n < count; n += 4) units.push_back({four_cost(cost(order[size_t(n)]) - 64, 0), n, std::min(4, count - n)});
    auto heavier_unit = [](const unit& a, const unit& b) { return a.cost > b.cost; };
    if (n_full > 0 && n_full < count) std::inplace_merge(units.begin(), units.begin() + n_full, units.end(), heavier_unit);
    const int num_wg = std::max(1, std::min(int(units.size()), num_cus * out.occ));
    // Least-loaded workgroup first, lowest index on ties.  As long as there are workgroups without a unit that is the next of them;
    // from then on the root of a min-heap of (assigned cost, workgroup), whose new load sinks to its place (640 items a step on 512
    // workgroups: with every unit through a queue the three schedules took 60 % of the plan).
    typedef unsigned __int128 slot;   // cost above, workgroup below: one comparison, and no branch, for both
    auto slot_of = [](int64_t assigned, int wg) { return slot(uint64_t(assigned)) << 32 | uint32_t(wg); };
    std::vector<int> wg_of(units.size(), 0), fill(size_t(num_wg) + 1, 0), full(size_t(num_wg), 0);
    std::vector<slot> load;
    load.reserve(size_t(num_wg));
    auto take = [&](size_t n, int64_t assigned, int wg) {
      const unit& u = units[n];
      wg_of[n] = wg;
      fill[size_t(wg) + 1] += u.count;
      if (u.first < n_full) ++full[size_t(wg)];
      return slot_of(assigned + (u.first < n_full ? u.cost : four_cost(cost(order[size_t(u.first)]) - 64, assigned)), wg);
    };
    const size_t direct = std::min(units.size(), size_t(num_wg));
    for (size_t n = 0; n < direct; ++n) load.push_back(take(n, 0, int(n)));
    if (units.size() > direct) std::make_heap(load.begin(), load.end(), std::greater<slot>());
    for (size_t n = direct; n < units.size(); ++n) {
      const slot sinking = take(n, int64_t(uint64_t(load[0] >> 32)), int(uint32_t(load[0])));
      size_t at = 0;
      for (size_t child = 1; child < load.size(); child = 2 * at + 1) {
        child += child + 1 < load.size() && load[child + 1] < load[child];
        if (load[child] > sinking) break;
        load[at] = load[child];
        at = child;
      }
      load[at] = sinking;
    }
    for (int w = 0; w < num_wg; ++w) fill[size_t(w) + 1] += fill[size_t(w)];
    out.indptr.assign(fill.begin(), fill.end());
    if (count > n_full)
      for (int w = 0; w < num_wg; ++w) out.solo.push_back(out.indptr[size_t(w)] + full[size_t(w)]);
    // a workgroup's items keep the order in which they were assigned, a wave's own ones after the others
    out.items.resize(size_t(count));
    std::vector<int> at_full(out.indptr.begin(), out.indptr.end()), at_solo(out.solo);
    for (size_t n = 0; n < units.size(); ++n) {
      const unit& u = units[n];
      int& at = (u.first < n_full ? at_full : at_solo)[size_t(wg_of[n])];
      for (int i = 0; i < u.count; ++i) out.items[size_t(at++)] = lay->items[size_t(order[size_t(u.first + i)])];
    }
    if (count == 0) out.indptr.assign(1, 0);
    if (solo_allowed) {   // the whole step's
      const schedule_work packed_work = work_of(out, num_cus);
      out.heaviest = packed_work.most;
      out.all = packed_work.all;
    }
    return out;
  };
  const int n_items = int(lay->items.size());
  const bool pre_mfma = lay->prefix_variant == PS_VARIANT_MFMA, suf_mfma = lay->suffix_variant == PS_VARIANT_MFMA;
  lay->stream_prefix = streams(0, lay->num_prefix_items);
  lay->stream_suffix = streams(lay->num_prefix_items, n_items);
  lay->stream_all = streams(0, n_items);
  const int first_packed = lay->num_rowsplit_items;   // row-split items run in the prefill kernel, one workgroup each
  lay->pk_prefix = pre_mfma ? pack(first_packed, lay->num_prefix_items, false) : packed{};
  lay->pk_suffix = suf_mfma ? pack(lay->num_prefix_items, n_items, false) : packed{};
  lay->pk_all = (pre_mfma && suf_mfma) ? pack(first_packed, n_items, true) : packed{};
  return ps_blob_build(lay);
}

// The plan by the rules for speed; where its partial states outgrow the static workspace and those by the rules for fewer
// states (a compute unit's whole share of the tokens per chunk) would not, the plan by these: ps_decode_attention_static
// serves such a batch, and callers with a workspace of their own lose nothing by it, since
// that many states cost more in the merge than the finer cut brings (float32, fewer / more states: 96 requests on 8 contexts
// of 8000 tokens and one KV head 248 / 319 us, 160 with 64-wide heads 152 / 195, 54 on 6 contexts and two KV heads 228 / 304).
int32_t ps_plan_build(ps_layout* lay, const ps_plan_options* user) {
  if (int32_t rc = build_plan(lay, user, false)) return rc;
  const int64_t slot_bytes = int64_t(lay->geo.num_q_heads) * (lay->geo.head_dim + 1) * 4;
  if (lay->coarser_slots < 0 || lay->coarser_slots * slot_bytes > PS_STATIC_WORKSPACE_BYTES) return PS_OK;
  const ps_plan_options opt = lay->opt;
  if (int32_t rc = build_plan(lay, &opt, true)) return rc;
  return ps_workspace_bytes(lay) <= PS_STATIC_WORKSPACE_BYTES ? PS_OK : build_plan(lay, &opt, false);
}

// Lays the tables out for the device: everything the kernels read, as one int32 blob.
int32_t ps_blob_build(ps_layout* lay) {
  typedef ps_layout::packed_set packed;
  const ps_geometry& g = lay->geo;
  const int32_t R = lay->num_requests;
  const int32_t total_prefix_blocks = int32_t(lay->prefix_blk.size());
  const int32_t root_blk0 = int32_t(lay->prefix_blk.size() + lay->suffix_blk.size());
  const packed &pk_prefix = lay->pk_prefix, &pk_suffix = lay->pk_suffix, &pk_all = lay->pk_all;
  const bool limited = !lay->visible.empty();
  auto visible_of = [&](int32_t r) { return limited ? lay->visible[size_t(r)] : lay->prefix_len[size_t(lay->req_prompt[size_t(r)])]; };
  // device blob: [block ids: prefix ++ suffix ++ root][request list: group_req ++ identity ++ root groups ++ per-chunk
  // subsets][items]
  // [slot_base][visible][requests to merge][schedules]
  // [per-block source offsets and valid counts][destinations of the last append]
  auto pad4 = [](int64_t n) { return (n + 3) / 4 * 4; };
  lay->off_blk = 0;
  lay->off_req = pad4(lay->off_blk + int64_t(lay->prefix_blk.size() + lay->suffix_blk.size() + lay->root_blk.size()));
  lay->off_items = pad4(lay->off_req + int64_t(lay->req_list.size()));
  lay->off_slot = pad4(lay->off_items + 8 * int64_t(lay->items.size()));
  lay->off_visible = pad4(lay->off_slot + R + 1);
  lay->off_merge = pad4(lay->off_visible + R);
  int64_t words = pad4(lay->off_merge + int64_t(lay->merge_req.size()));
  auto place = [&](ps_layout::schedule& s, const packed& pk) {
    s = ps_layout::schedule{};
    if (pk.items.empty()) return;
    s.num_wg = int32_t(pk.indptr.size()) - 1;
    s.max_rows = pk.max_rows;
    s.stream = pk.stream;
    s.off_items = words;
    words = pad4(words + 8 * int64_t(pk.items.size()));
    s.off_indptr = words;
    words = pad4(words + int64_t(pk.indptr.size()));
    if (!pk.solo.empty()) {
      s.off_solo = words;
      words = pad4(words + int64_t(pk.solo.size()));
    }
  };
  place(lay->sched_prefix, pk_prefix);
  place(lay->sched_suffix, pk_suffix);
  place(lay->sched_all, pk_all);
  // per-block directory for the cache-writing kernels
  const int64_t num_blk_entries = int64_t(lay->prefix_blk.size() + lay->suffix_blk.size() + lay->root_blk.size());
  lay->off_ent_tok0 = words;
  lay->off_ent_valid = pad4(lay->off_ent_tok0 + num_blk_entries);
  lay->off_dest = pad4(lay->off_ent_valid + num_blk_entries);
  lay->off_ent_order = pad4(lay->off_dest + R);
  words = pad4(lay->off_ent_order + num_blk_entries);
  // (the tables grow by a few words per decode step: room to spare keeps the buffer -- and its mapped pages -- in
  // place instead of taking a fresh allocation every step)
  const size_t blob_words = size_t(std::max<int64_t>(words, 4));
  if (lay->blob.capacity() < blob_words) lay->blob.reserve(blob_words + blob_words / 4 + 1024);
  lay->blob.resize(blob_words);   // (every word that a kernel reads is written below)
  int32_t* b = lay->blob.data();
  {
    const int32_t B = g.block_size;
    // skip: per segment, leading blocks that are not to be written (adopted from another layout); the ragged source
    // then holds only the tokens after them
    auto fill_entries = [&](const std::vector<int32_t>& indptr, const std::vector<int32_t>& len, int32_t* tok0_out,
                            int32_t* valid_out, const std::vector<int32_t>* skip) {
      int64_t tok = 0;
      for (size_t s = 0; s + 1 < indptr.size(); ++s) {
        const int64_t skipped = skip ? int64_t((*skip)[s + 1] - (*skip)[s]) * B : 0;
        for (int32_t i = indptr[s]; i < indptr[s + 1]; ++i) {
          const int64_t first = int64_t(i - indptr[s]) * B;
          if (tok + first > INT32_MAX) return false;
          const bool kept = first < skipped;
          tok0_out[i] = kept ? 0 : int32_t(tok + first - skipped);
          valid_out[i] = kept ? 0 : int32_t(std::min<int64_t>(B, len[s] - first));
        }
        tok += len[s] - skipped;
      }
      return true;
    };
    // The shared segments (prefixes, roots) never change after the layout is made, so their part of the directory is
    // worked out once and copied from then on; the private part follows the appends.
    const size_t n_fixed = lay->prefix_blk.size() + lay->root_blk.size();
    if (lay->ent_fixed_tok0.size() != n_fixed) {
      lay->ent_fixed_tok0.assign(n_fixed, 0);
      lay->ent_fixed_valid.assign(n_fixed, 0);
      int32_t* root_tok0 = lay->ent_fixed_tok0.data() + lay->prefix_blk.size();
      int32_t* root_valid = lay->ent_fixed_valid.data() + lay->prefix_blk.size();
      if (!fill_entries(lay->prefix_blk_indptr, lay->prefix_len, lay->ent_fixed_tok0.data(), lay->ent_fixed_valid.data(),
                        lay->adopt_indptr.empty() ? nullptr : &lay->adopt_indptr) ||
          (lay->num_roots && !fill_entries(lay->root_blk_indptr, lay->root_len, root_tok0, root_valid, nullptr))) {
        lay->ent_fixed_tok0.clear();
        lay->ent_fixed_valid.clear();
        return PS_ERR_INVALID_ARG;
      }
      // An ingest walks the shared blocks in the order of their addresses in the pool, not of the tokens: the pool's
      // blocks are scattered, and scattered reads (the source, now) cost less than scattered writes (measured on the
      // staging copies: 5.8 against 5.2 TB/s).
      auto by_block = [&](const std::vector<int32_t>& blk, int32_t* order) {
        if (blk.empty()) return;
        // (where the ids fill a good part of their range they are laid out by id, otherwise sorted; a permutation either
        // way, also of ids that repeat -- a parked layout's are all -1)
        const auto range = std::minmax_element(blk.begin(), blk.end());
        const int32_t lowest = *range.first;
        const size_t span = size_t(int64_t(*range.second) - lowest + 1);
        if (span <= 16 * blk.size()) {
          std::vector<int32_t> at(span, 0);      // entries with a smaller id, then the next position of an id
          for (int32_t b2 : blk) ++at[size_t(b2 - lowest)];
          std::exclusive_scan(at.begin(), at.end(), at.begin(), 0);
          for (size_t i = 0; i < blk.size(); ++i) order[at[size_t(blk[i] - lowest)]++] = int32_t(i);
        } else {
          std::iota(order, order + blk.size(), 0);
          std::sort(order, order + blk.size(), [&](int32_t a, int32_t b2) { return blk[size_t(a)] < blk[size_t(b2)]; });
        }
      };
      lay->ent_fixed_order.resize(n_fixed);
      by_block(lay->prefix_blk, lay->ent_fixed_order.data());
      by_block(lay->root_blk, lay->ent_fixed_order.data() + lay->prefix_blk.size());
    }
    std::copy(lay->ent_fixed_tok0.begin(), lay->ent_fixed_tok0.begin() + total_prefix_blocks, b + lay->off_ent_tok0);
    std::copy(lay->ent_fixed_valid.begin(), lay->ent_fixed_valid.begin() + total_prefix_blocks, b + lay->off_ent_valid);
    std::copy(lay->ent_fixed_tok0.begin() + total_prefix_blocks, lay->ent_fixed_tok0.end(), b + lay->off_ent_tok0 + root_blk0);
    std::copy(lay->ent_fixed_valid.begin() + total_prefix_blocks, lay->ent_fixed_valid.end(), b + lay->off_ent_valid + root_blk0);
    if (!fill_entries(lay->suffix_blk_indptr, lay->suffix_len, b + lay->off_ent_tok0 + total_prefix_blocks,
                      b + lay->off_ent_valid + total_prefix_blocks, nullptr))
      return PS_ERR_INVALID_ARG;
    lay->append_dest.resize(size_t(R), -1);
    std::copy(lay->append_dest.begin(), lay->append_dest.end(), b + lay->off_dest);
    // (entries of the concatenated block array: the shared kinds by block, the private segments as stored)
    std::copy(lay->ent_fixed_order.begin(), lay->ent_fixed_order.begin() + total_prefix_blocks, b + lay->off_ent_order);
    std::iota(b + lay->off_ent_order + total_prefix_blocks, b + lay->off_ent_order + root_blk0, total_prefix_blocks);
    for (size_t i = 0; i < lay->root_blk.size(); ++i)
      b[lay->off_ent_order + root_blk0 + int64_t(i)] = root_blk0 + lay->ent_fixed_order[size_t(total_prefix_blocks) + i];
  }
  auto fill = [&](const ps_layout::schedule& s, const packed& pk) {
    if (pk.items.empty()) return;
    std::memcpy(b + s.off_items, pk.items.data(), pk.items.size() * sizeof(ps_item));
    std::copy(pk.indptr.begin(), pk.indptr.end(), b + s.off_indptr);
    if (s.off_solo >= 0) std::copy(pk.solo.begin(), pk.solo.end(), b + s.off_solo);
  };
  fill(lay->sched_prefix, pk_prefix);
  fill(lay->sched_suffix, pk_suffix);
  fill(lay->sched_all, pk_all);
  std::copy(lay->prefix_blk.begin(), lay->prefix_blk.end(), b + lay->off_blk);
  std::copy(lay->suffix_blk.begin(), lay->suffix_blk.end(), b + lay->off_blk + lay->prefix_blk.size());
  std::copy(lay->root_blk.begin(), lay->root_blk.end(), b + lay->off_blk + root_blk0);
  std::copy(lay->req_list.begin(), lay->req_list.end(), b + lay->off_req);
  for (int32_t r = 0; r < R; ++r) b[lay->off_visible + r] = visible_of(r);
  std::copy(lay->merge_req.begin(), lay->merge_req.end(), b + lay->off_merge);
  if (!lay->items.empty()) std::memcpy(b + lay->off_items, lay->items.data(), lay->items.size() * sizeof(ps_item));
  std::copy(lay->slot_base.begin(), lay->slot_base.end(), b + lay->off_slot);
  return PS_OK;
}

namespace {

// Drops every reference the layout holds; blocks that reach zero join the free-list tail in ascending id.
// PS_ERR_REFCOUNT leaves the pool unchanged.
int32_t drop_references(ps_pool* pool, const ps_layout* lay) {
  std::vector<int64_t> drop(size_t(pool->num_blocks), 0);
  for (int32_t t = 0; t < lay->num_roots; ++t) {
    const int32_t k = lay->root_group_indptr[size_t(t) + 1] - lay->root_group_indptr[size_t(t)];
    for (int32_t i = lay->root_blk_indptr[size_t(t)]; i < lay->root_blk_indptr[size_t(t) + 1]; ++i) {
      const int32_t b = lay->root_blk[size_t(i)];
      if (b < 0 || b >= pool->num_blocks) return PS_ERR_REFCOUNT;
      drop[size_t(b)] += k;
    }
  }
  for (int32_t p = 0; p < lay->num_prompts; ++p) {
    const int32_t k = lay->group_indptr[size_t(p) + 1] - lay->group_indptr[size_t(p)];
    for (int32_t i = lay->prefix_blk_indptr[size_t(p)]; i < lay->prefix_blk_indptr[size_t(p) + 1]; ++i) {
      const int32_t b = lay->prefix_blk[size_t(i)];
      if (b < 0 || b >= pool->num_blocks) return PS_ERR_REFCOUNT;
      drop[size_t(b)] += k;
    }
  }
  for (int32_t b : lay->suffix_blk) {
    if (b < 0 || b >= pool->num_blocks) return PS_ERR_REFCOUNT;
    drop[size_t(b)] += 1;
  }
  for (int32_t b = 0; b < pool->num_blocks; ++b)
    if (pool->refcount[size_t(b)] < drop[size_t(b)]) return PS_ERR_REFCOUNT;
  for (int32_t b = 0; b < pool->num_blocks; ++b) {
    if (!drop[size_t(b)]) continue;
    pool->refcount[size_t(b)] -= int32_t(drop[size_t(b)]);
    if (pool->refcount[size_t(b)] == 0) pool->free_list.push_back(b);
  }
  return PS_OK;
}

// Takes the blocks of every segment by the canonical policy (roots, prompts, requests; head of the free list).  The
// caller has checked that the free list is long enough.
void take_blocks(ps_pool* pool, ps_layout* lay) {
  const int32_t B = lay->geo.block_size;
  auto take = [&](int32_t refs) {
    const int32_t blk = pool->free_list.front();
    pool->free_list.pop_front();
    pool->refcount[size_t(blk)] += refs;
    return blk;
  };
  lay->root_blk.clear();
  lay->prefix_blk.clear();
  lay->suffix_blk.clear();
  lay->root_blk_indptr.assign(size_t(lay->num_roots) + 1, 0);
  for (int32_t t = 0; t < lay->num_roots; ++t) {
    const int32_t k = lay->root_group_indptr[size_t(t) + 1] - lay->root_group_indptr[size_t(t)];
    const int64_t n = ceil_div(lay->root_len[size_t(t)], B);
    for (int64_t i = 0; i < n; ++i) lay->root_blk.push_back(take(k));
    lay->root_blk_indptr[size_t(t) + 1] = int32_t(lay->root_blk.size());
  }
  lay->prefix_blk_indptr.assign(size_t(lay->num_prompts) + 1, 0);
  const bool adopting = !lay->adopt_indptr.empty();
  for (int32_t p = 0; p < lay->num_prompts; ++p) {
    const int32_t k = lay->group_indptr[size_t(p) + 1] - lay->group_indptr[size_t(p)];
    const int64_t n = ceil_div(lay->prefix_len[size_t(p)], B);
    const int32_t a0 = adopting ? lay->adopt_indptr[size_t(p)] : 0, a1 = adopting ? lay->adopt_indptr[size_t(p) + 1] : 0;
    for (int64_t i = 0; i < n; ++i) {
      if (i < a1 - a0) {   // a cached block another layout holds: one more reference per request, like a fresh one
        const int32_t blk = lay->adopt_blk[size_t(a0 + i)];
        pool->refcount[size_t(blk)] += k;
        lay->prefix_blk.push_back(blk);
      } else {
        lay->prefix_blk.push_back(take(k));
      }
    }
    lay->prefix_blk_indptr[size_t(p) + 1] = int32_t(lay->prefix_blk.size());
  }
  lay->suffix_blk_indptr.assign(size_t(lay->num_requests) + 1, 0);
  for (int32_t r = 0; r < lay->num_requests; ++r) {
    const int64_t n = ceil_div(lay->suffix_len[size_t(r)], B);
    for (int64_t i = 0; i < n; ++i) lay->suffix_blk.push_back(take(1));
    lay->suffix_blk_indptr[size_t(r) + 1] = int32_t(lay->suffix_blk.size());
  }
}

int64_t blocks_of(const ps_layout* lay) {   // blocks the layout references, adopted ones included
  const int32_t B = lay->geo.block_size;
  int64_t n = 0;
  for (int32_t l : lay->root_len) n += ceil_div(l, B);
  for (int32_t l : lay->prefix_len) n += ceil_div(l, B);
  for (int32_t l : lay->suffix_len) n += ceil_div(l, B);
  return n;
}

}  // namespace

// ---------------------------------------------------------------------------------------------------
extern "C" {

int32_t ps_pool_create(int32_t num_blocks, const int32_t* free_order, ps_pool** out) {
  if (!out || num_blocks < 0) return PS_ERR_INVALID_ARG;
  ps_pool* p = new (std::nothrow) ps_pool();
  if (!p) return PS_ERR_OOM;
  p->num_blocks = num_blocks;
  p->refcount.assign(size_t(num_blocks), 0);
  if (free_order) {
    std::vector<char> seen(size_t(num_blocks), 0);
    for (int32_t i = 0; i < num_blocks; ++i) {
      const int32_t b = free_order[i];
      if (b < 0 || b >= num_blocks || seen[size_t(b)]) { delete p; return PS_ERR_INVALID_ARG; }
      seen[size_t(b)] = 1;
      p->free_list.push_back(b);
    }
  } else {
    for (int32_t i = 0; i < num_blocks; ++i) p->free_list.push_back(i);
  }
  live_pools.fetch_add(1);
  *out = p;
  return PS_OK;
}

int32_t ps_pool_destroy(ps_pool* pool) {
  if (!pool) return PS_OK;
  delete pool;
  if (live_pools.fetch_sub(1) == 1 && ps_last_pool_hook) ps_last_pool_hook();
  return PS_OK;
}

int32_t ps_pool_num_free(const ps_pool* pool, int32_t* out) {
  if (!pool || !out) return PS_ERR_INVALID_ARG;
  *out = int32_t(pool->free_list.size());
  return PS_OK;
}

int32_t ps_pool_free_list(const ps_pool* pool, int32_t* out, int32_t capacity, int32_t* count) {
  if (!pool || !count || capacity < 0 || (capacity > 0 && !out)) return PS_ERR_INVALID_ARG;
  *count = int32_t(pool->free_list.size());
  if (capacity < *count) return PS_ERR_INVALID_ARG;
  std::copy(pool->free_list.begin(), pool->free_list.end(), out);
  return PS_OK;
}

int32_t ps_pool_refcounts(const ps_pool* pool, const int32_t** refcount) {
  if (!pool || !refcount) return PS_ERR_INVALID_ARG;
  *refcount = pool->refcount.data();
  return PS_OK;
}

}  // extern "C"

namespace {

int32_t build_layout(ps_pool* pool, const ps_geometry* geometry, int32_t num_roots, const int32_t* root_len,
                     int32_t num_prompts, const int32_t* prompt_root, const int32_t* prefix_len,
                     const int32_t* adopt_indptr, const int32_t* adopt_blk, int32_t num_requests,
                     const int32_t* req_prompt, const int32_t* req_model, const int32_t* suffix_len, ps_layout** out) {
  if (!pool || !geometry || !out || num_roots < 0 || num_prompts < 0 || num_requests < 0) return PS_ERR_INVALID_ARG;
  if ((num_prompts && !prefix_len) || (num_requests && (!req_prompt || !req_model || !suffix_len)))
    return PS_ERR_INVALID_ARG;
  if (num_roots && (!root_len || !prompt_root)) return PS_ERR_INVALID_ARG;
  if (int32_t st = check_geometry(*geometry)) return st;
  const int32_t B = geometry->block_size;

  std::vector<int32_t> members_count(size_t(num_prompts), 0);
  std::vector<uint64_t> seen;      // (prompt, model) of every request
  seen.reserve(size_t(num_requests));
  for (int32_t r = 0; r < num_requests; ++r) {
    if (req_prompt[r] < 0 || req_prompt[r] >= num_prompts || req_model[r] < 0 || suffix_len[r] < 0)
      return PS_ERR_INVALID_ARG;
    seen.push_back(uint64_t(uint32_t(req_prompt[r])) << 32 | uint32_t(req_model[r]));
    ++members_count[size_t(req_prompt[r])];
  }
  if (!std::is_sorted(seen.begin(), seen.end())) std::sort(seen.begin(), seen.end());
  if (std::adjacent_find(seen.begin(), seen.end()) != seen.end()) return PS_ERR_INVALID_ARG;
  // requests below every root: all requests of the prompts that begin with it
  std::vector<int32_t> below_count(size_t(num_roots), 0), root_prompts(size_t(num_roots), 0);
  for (int32_t p = 0; p < num_prompts && num_roots; ++p) {
    const int32_t t = prompt_root[p];
    if (t < -1 || t >= num_roots) return PS_ERR_INVALID_ARG;
    if (t >= 0) {
      below_count[size_t(t)] += members_count[size_t(p)];
      ++root_prompts[size_t(t)];
    }
  }
  int64_t needed = 0;
  for (int32_t t = 0; t < num_roots; ++t) {
    if (root_len[t] < 0 || root_prompts[size_t(t)] == 0) return PS_ERR_INVALID_ARG;
    needed += ceil_div(root_len[t], B);
  }
  for (int32_t p = 0; p < num_prompts; ++p) {
    if (prefix_len[p] < 0 || members_count[size_t(p)] == 0) return PS_ERR_INVALID_ARG;
    needed += ceil_div(prefix_len[p], B);
  }
  for (int32_t r = 0; r < num_requests; ++r) needed += ceil_div(suffix_len[r], B);
  if (adopt_indptr) {
    // adopted blocks: full blocks of the prompt's prefix, alive (referenced by some layout) and named once
    if (adopt_indptr[0] != 0 || (adopt_indptr[num_prompts] > 0 && !adopt_blk)) return PS_ERR_INVALID_ARG;
    std::vector<char> named(size_t(pool->num_blocks), 0);
    for (int32_t p = 0; p < num_prompts; ++p) {
      const int32_t n = adopt_indptr[p + 1] - adopt_indptr[p];
      if (n < 0 || int64_t(n) * B > prefix_len[p]) return PS_ERR_INVALID_ARG;
      for (int32_t i = adopt_indptr[p]; i < adopt_indptr[p + 1]; ++i) {
        const int32_t blk = adopt_blk[i];
        if (blk < 0 || blk >= pool->num_blocks || pool->refcount[size_t(blk)] <= 0 || named[size_t(blk)])
          return PS_ERR_INVALID_ARG;
        named[size_t(blk)] = 1;
      }
      needed -= n;
    }
  }
  if (needed > int64_t(pool->free_list.size())) return PS_ERR_OOM;

  ps_layout* lay = new (std::nothrow) ps_layout();
  if (!lay) return PS_ERR_OOM;
  lay->geo = *geometry;
  lay->num_prompts = num_prompts;
  lay->num_requests = num_requests;
  lay->prefix_len.assign(prefix_len, prefix_len + num_prompts);
  lay->suffix_len.assign(suffix_len, suffix_len + num_requests);
  lay->req_prompt.assign(req_prompt, req_prompt + num_requests);
  lay->req_model.assign(req_model, req_model + num_requests);
  if (adopt_indptr && adopt_indptr[num_prompts] > 0) {
    lay->adopt_indptr.assign(adopt_indptr, adopt_indptr + num_prompts + 1);
    lay->adopt_blk.assign(adopt_blk, adopt_blk + adopt_indptr[num_prompts]);
  }
  lay->num_roots = num_roots;
  if (num_roots) {
    lay->root_len.assign(root_len, root_len + num_roots);
    lay->prompt_root.assign(prompt_root, prompt_root + num_prompts);
  }

  // sharing groups: a prompt's requests in ascending request index; a root's likewise
  lay->group_indptr.assign(size_t(num_prompts) + 1, 0);
  for (int32_t p = 0; p < num_prompts; ++p) lay->group_indptr[size_t(p) + 1] = lay->group_indptr[size_t(p)] + members_count[size_t(p)];
  lay->group_req.assign(size_t(num_requests), 0);
  {
    std::vector<int32_t> cursor(lay->group_indptr.begin(), lay->group_indptr.end() - 1);
    for (int32_t r = 0; r < num_requests; ++r) lay->group_req[size_t(cursor[size_t(req_prompt[r])]++)] = r;
  }
  lay->root_group_indptr.assign(size_t(num_roots) + 1, 0);
  for (int32_t t = 0; t < num_roots; ++t)
    lay->root_group_indptr[size_t(t) + 1] = lay->root_group_indptr[size_t(t)] + below_count[size_t(t)];
  lay->root_group_req.assign(size_t(lay->root_group_indptr.back()), 0);
  if (num_roots) {
    std::vector<int32_t> cursor(lay->root_group_indptr.begin(), lay->root_group_indptr.end() - 1);
    for (int32_t r = 0; r < num_requests; ++r) {
      const int32_t t = prompt_root[req_prompt[r]];
      if (t >= 0) lay->root_group_req[size_t(cursor[size_t(t)]++)] = r;
    }
  }

  take_blocks(pool, lay);

  if (int32_t st = ps_plan_build(lay, nullptr)) {
    // cannot fail with default options, but never leave references behind
    ps_layout_release(pool, lay);
    return st;
  }
  *out = lay;
  return PS_OK;
}

}  // namespace

extern "C" {

int32_t ps_kv_layout_tree(ps_pool* pool, const ps_geometry* geometry, int32_t num_roots, const int32_t* root_len,
                          int32_t num_prompts, const int32_t* prompt_root, const int32_t* prefix_len,
                          int32_t num_requests, const int32_t* req_prompt, const int32_t* req_model,
                          const int32_t* suffix_len, ps_layout** out) {
  return build_layout(pool, geometry, num_roots, root_len, num_prompts, prompt_root, prefix_len, nullptr, nullptr,
                      num_requests, req_prompt, req_model, suffix_len, out);
}

int32_t ps_kv_layout(ps_pool* pool, const ps_geometry* geometry, int32_t num_prompts, const int32_t* prefix_len,
                     int32_t num_requests, const int32_t* req_prompt, const int32_t* req_model,
                     const int32_t* suffix_len, ps_layout** out) {
  return build_layout(pool, geometry, 0, nullptr, num_prompts, nullptr, prefix_len, nullptr, nullptr, num_requests,
                      req_prompt, req_model, suffix_len, out);
}

int32_t ps_kv_layout_adopt(ps_pool* pool, const ps_geometry* geometry, int32_t num_prompts, const int32_t* prefix_len,
                           const int32_t* adopt_indptr, const int32_t* adopt_blk, int32_t num_requests,
                           const int32_t* req_prompt, const int32_t* req_model, const int32_t* suffix_len,
                           ps_layout** out) {
  if (num_prompts > 0 && !adopt_indptr) return PS_ERR_INVALID_ARG;
  return build_layout(pool, geometry, 0, nullptr, num_prompts, nullptr, prefix_len, adopt_indptr, adopt_blk,
                      num_requests, req_prompt, req_model, suffix_len, out);
}

int32_t ps_layout_root_tables(const ps_layout* lay, int32_t* num_roots, const int32_t** root_blk_indptr,
                              const int32_t** root_blk, const int32_t** root_group_indptr,
                              const int32_t** root_group_req) {
  if (!lay) return PS_ERR_INVALID_ARG;
  if (num_roots) *num_roots = lay->num_roots;
  if (root_blk_indptr) *root_blk_indptr = lay->root_blk_indptr.data();
  if (root_blk) *root_blk = lay->root_blk.data();
  if (root_group_indptr) *root_group_indptr = lay->root_group_indptr.data();
  if (root_group_req) *root_group_req = lay->root_group_req.data();
  return PS_OK;
}

int32_t ps_layout_release(ps_pool* pool, ps_layout* lay) {
  if (!pool || !lay) return PS_ERR_INVALID_ARG;
  if (!lay->parked)
    if (int32_t st = drop_references(pool, lay)) return st;
  delete lay;
  return PS_OK;
}

int32_t ps_blocks_needed(int32_t block_size, int32_t num_roots, const int32_t* root_len, int32_t num_prompts,
                         const int32_t* prefix_len, int32_t num_requests, const int32_t* suffix_len, int64_t* out) {
  if (!out || block_size <= 0 || num_roots < 0 || num_prompts < 0 || num_requests < 0) return PS_ERR_INVALID_ARG;
  if ((num_roots && !root_len) || (num_prompts && !prefix_len) || (num_requests && !suffix_len)) return PS_ERR_INVALID_ARG;
  int64_t n = 0;
  auto add = [&](const int32_t* len, int32_t count) {
    for (int32_t i = 0; i < count; ++i) {
      if (len[i] < 0) return false;
      n += ceil_div(len[i], block_size);
    }
    return true;
  };
  if (!add(root_len, num_roots) || !add(prefix_len, num_prompts) || !add(suffix_len, num_requests)) return PS_ERR_INVALID_ARG;
  *out = n;
  return PS_OK;
}

int32_t ps_layout_park(ps_pool* pool, ps_layout* lay) {
  if (!pool || !lay || lay->parked) return PS_ERR_INVALID_ARG;
  if (int32_t st = drop_references(pool, lay)) return st;
  lay->parked = true;
  lay->adopt_indptr.clear();   // a resumed layout holds fresh blocks only: its image carries the adopted contents
  lay->ent_fixed_tok0.clear();   // ... so the directory of the shared segments is worked out again
  lay->ent_fixed_valid.clear();
  lay->ent_fixed_order.clear();
  lay->adopt_blk.clear();
  std::fill(lay->root_blk.begin(), lay->root_blk.end(), -1);
  std::fill(lay->prefix_blk.begin(), lay->prefix_blk.end(), -1);
  std::fill(lay->suffix_blk.begin(), lay->suffix_blk.end(), -1);
  std::fill(lay->append_dest.begin(), lay->append_dest.end(), -1);
  return PS_OK;
}

int32_t ps_layout_resume(ps_pool* pool, ps_layout* lay) {
  if (!pool || !lay || !lay->parked) return PS_ERR_INVALID_ARG;
  if (blocks_of(lay) > int64_t(pool->free_list.size())) return PS_ERR_OOM;
  take_blocks(pool, lay);
  lay->parked = false;
  lay->ent_fixed_tok0.clear();   // a plan made while parked worked the directory out without blocks
  lay->ent_fixed_valid.clear();
  lay->ent_fixed_order.clear();
  return ps_plan_build(lay, &lay->opt);   // options that were accepted before cannot fail
}

int32_t ps_layout_state(const ps_layout* lay, int64_t* num_blocks, int32_t* parked) {
  if (!lay) return PS_ERR_INVALID_ARG;
  if (num_blocks) *num_blocks = blocks_of(lay);
  if (parked) *parked = lay->parked ? 1 : 0;
  return PS_OK;
}

int32_t ps_stage_layout(const ps_layout* lay, int64_t* block_bytes, int64_t* scales_offset_bytes, int64_t* total_bytes) {
  if (!lay) return PS_ERR_INVALID_ARG;
  const ps_geometry& g = lay->geo;
  const int64_t esz = g.kv_dtype == PS_F32 ? 4 : (g.kv_dtype == PS_BF16 ? 2 : 1);
  const int64_t per_block = int64_t(g.num_kv_heads) * 2 * g.block_size * g.head_dim * esz;
  const int64_t n = blocks_of(lay);
  const int64_t scales_off = round_up(n * per_block, 256);
  if (block_bytes) *block_bytes = per_block;
  if (scales_offset_bytes) *scales_offset_bytes = scales_off;
  if (total_bytes) *total_bytes = g.kv_dtype == PS_FP8_E4M3 ? scales_off + n * g.num_kv_heads * 2 * 4 : std::max<int64_t>(n * per_block, 16);
  return PS_OK;
}

int32_t ps_layout_tables(const ps_layout* lay, const int32_t** prefix_blk_indptr, const int32_t** prefix_blk,
                         const int32_t** group_indptr, const int32_t** group_req,
                         const int32_t** suffix_blk_indptr, const int32_t** suffix_blk) {
  if (!lay) return PS_ERR_INVALID_ARG;
  if (prefix_blk_indptr) *prefix_blk_indptr = lay->prefix_blk_indptr.data();
  if (prefix_blk) *prefix_blk = lay->prefix_blk.data();
  if (group_indptr) *group_indptr = lay->group_indptr.data();
  if (group_req) *group_req = lay->group_req.data();
  if (suffix_blk_indptr) *suffix_blk_indptr = lay->suffix_blk_indptr.data();
  if (suffix_blk) *suffix_blk = lay->suffix_blk.data();
  return PS_OK;
}

int32_t ps_layout_lengths(const ps_layout* lay, const int32_t** prefix_len, const int32_t** suffix_len) {
  if (!lay) return PS_ERR_INVALID_ARG;
  if (prefix_len) *prefix_len = lay->prefix_len.data();
  if (suffix_len) *suffix_len = lay->suffix_len.data();
  return PS_OK;
}

int32_t ps_layout_append(ps_pool* pool, ps_layout* lay, const int32_t* active, const int32_t** dest) {
  if (!pool || !lay || lay->parked) return PS_ERR_INVALID_ARG;
  const int32_t R = lay->num_requests, B = lay->geo.block_size;
  if (int64_t(pool->num_blocks) * B > INT32_MAX) return PS_ERR_INVALID_ARG;  // slot indices are int32
  auto is_active = [&](int32_t r) { return !active || active[r] != 0; };
  int64_t needed = 0;
  for (int32_t r = 0; r < R; ++r) {
    if (!is_active(r)) continue;
    if (lay->suffix_len[size_t(r)] == INT32_MAX) return PS_ERR_INVALID_ARG;
    if (lay->suffix_len[size_t(r)] % B == 0) ++needed;
  }
  if (needed > int64_t(pool->free_list.size())) return PS_ERR_OOM;
  // requests in ascending index; one whose private length is a multiple of the block size (none yet, or the
  // last block is full) takes the block at the head of the free list
  std::vector<int32_t> blk, indptr(size_t(R) + 1, 0);
  blk.reserve(lay->suffix_blk.size() + size_t(needed));
  lay->append_dest.assign(size_t(R), -1);
  for (int32_t r = 0; r < R; ++r) {
    const size_t first = blk.size();
    blk.insert(blk.end(), lay->suffix_blk.begin() + lay->suffix_blk_indptr[size_t(r)],
               lay->suffix_blk.begin() + lay->suffix_blk_indptr[size_t(r) + 1]);
    if (is_active(r)) {
      const int32_t pos = lay->suffix_len[size_t(r)];
      if (pos % B == 0) {
        const int32_t b = pool->free_list.front();
        pool->free_list.pop_front();
        pool->refcount[size_t(b)] += 1;
        blk.push_back(b);
      }
      lay->append_dest[size_t(r)] = blk[first + size_t(pos / B)] * B + pos % B;
      lay->suffix_len[size_t(r)] = pos + 1;
    }
    indptr[size_t(r) + 1] = int32_t(blk.size());
  }
  lay->suffix_blk.swap(blk);
  lay->suffix_blk_indptr.swap(indptr);
  // A step that leaves the chunk structure of every private segment as it is (same number of chunks, same chunk
  // size where there are several) only moves token ends and block offsets: the plan -- items, their order, the
  // packing onto workgroups -- is kept and patched, and only the tables are laid out again.  Anything else (a first
  // token, a segment outgrowing its chunks, a schedule its balance) plans afresh.
  bool same_structure = lay->suffix_chunks.size() == size_t(R) && lay->suffix_chunk > 0;
  const int64_t granule = std::lcm<int64_t>(B, 32);
  for (int32_t r = 0; r < R && same_structure; ++r) {
    if (!is_active(r)) continue;
    const int64_t len = lay->suffix_len[size_t(r)];
    const int64_t count = ceil_div(len, lay->suffix_chunk);
    const int64_t size = round_up(ceil_div(len, count), granule);
    const int64_t n = ceil_div(len, size);
    if (len <= 1 || n != lay->suffix_chunks[size_t(r)] || (n > 1 && size != lay->suffix_chunk_size[size_t(r)]))
      same_structure = false;
    else
      lay->suffix_chunk_size[size_t(r)] = int32_t(size);
  }
  if (same_structure) {
    const int32_t prefix_blocks = int32_t(lay->prefix_blk.size());
    const int32_t root_shift = int32_t(lay->prefix_blk.size() + lay->suffix_blk.size()) - lay->planned_root_blk0;
    auto patch = [&](std::vector<ps_item>& items) {
      for (ps_item& it : items) {
        if (it.kind & kPsItemSuffix) {
          const int32_t r = it.req_off - R;   // private-suffix items index the identity part of the request list
          it.blk_off = prefix_blocks + lay->suffix_blk_indptr[size_t(r)];
          it.tok_end = std::min(lay->suffix_len[size_t(r)], it.tok_begin + lay->suffix_chunk_size[size_t(r)]);
        } else if (it.kind & kPsItemRoot) {
          it.blk_off += root_shift;
        }
      }
    };
    patch(lay->items);
    patch(lay->pk_prefix.items);
    patch(lay->pk_suffix.items);
    patch(lay->pk_all.items);
    lay->planned_root_blk0 += root_shift;
    find_solo_items(lay);
    same_structure = !outgrown(lay);
  }
  if (int32_t st = same_structure ? ps_blob_build(lay) : ps_plan_build(lay, &lay->opt)) return st;
  if (dest) *dest = lay->append_dest.data();
  return PS_OK;
}

int32_t ps_layout_set_visible(ps_layout* lay, const int32_t* prefix_visible) {
  if (!lay) return PS_ERR_INVALID_ARG;
  std::vector<int32_t> v;
  if (prefix_visible) {
    v.assign(prefix_visible, prefix_visible + lay->num_requests);
    for (int32_t r = 0; r < lay->num_requests; ++r)
      if (v[size_t(r)] < 0 || v[size_t(r)] > lay->prefix_len[size_t(lay->req_prompt[size_t(r)])]) return PS_ERR_INVALID_ARG;
  }
  lay->visible.swap(v);
  if (int32_t st = ps_plan_build(lay, &lay->opt)) {
    lay->visible.swap(v);              // cannot fail with options that were accepted before; keep the old state
    ps_plan_build(lay, &lay->opt);
    return st;
  }
  return PS_OK;
}

int32_t ps_layout_request_list(const ps_layout* lay, int32_t* count, const int32_t** list) {
  if (!lay) return PS_ERR_INVALID_ARG;
  if (count) *count = int32_t(lay->req_list.size());
  if (list) *list = lay->req_list.data();
  return PS_OK;
}

int32_t ps_layout_replan(ps_layout* lay, const ps_plan_options* options) {
  if (!lay) return PS_ERR_INVALID_ARG;
  return ps_plan_build(lay, options);
}

int32_t ps_layout_plan(const ps_layout* lay, int32_t* num_items, const int32_t** items, const int32_t** slot_base,
                       int32_t* prefix_variant, int32_t* suffix_variant) {
  if (!lay) return PS_ERR_INVALID_ARG;
  if (num_items) *num_items = int32_t(lay->items.size());
  if (items) *items = reinterpret_cast<const int32_t*>(lay->items.data());
  if (slot_base) *slot_base = lay->slot_base.data();
  if (prefix_variant) *prefix_variant = lay->prefix_variant;
  if (suffix_variant) *suffix_variant = lay->suffix_variant;
  return PS_OK;
}

int32_t ps_layout_schedule(const ps_layout* lay, int32_t which, int32_t* num_workgroups, const int32_t** items,
                           const int32_t** indptr) {
  if (!lay || which < 0 || which > 2) return PS_ERR_INVALID_ARG;
  const ps_layout::schedule& s = which == 0 ? lay->sched_prefix : (which == 1 ? lay->sched_suffix : lay->sched_all);
  if (num_workgroups) *num_workgroups = s.num_wg;
  if (items) *items = s.num_wg ? lay->blob.data() + s.off_items : nullptr;
  if (indptr) *indptr = s.num_wg ? lay->blob.data() + s.off_indptr : nullptr;
  return PS_OK;
}

int64_t ps_layout_device_bytes(const ps_layout* lay) { return lay ? int64_t(lay->blob.size()) * 4 : -1; }

int64_t ps_workspace_bytes(const ps_layout* lay) {
  if (!lay) return -1;
  const int64_t rows = lay->num_slots * lay->geo.num_q_heads;
  return std::max<int64_t>(16, rows * (lay->geo.head_dim + 1) * 4);
}

int32_t ps_workspace_layout(const ps_layout* lay, int64_t* num_slots, int64_t* lse_offset_bytes) {
  if (!lay) return PS_ERR_INVALID_ARG;
  if (num_slots) *num_slots = lay->num_slots;
  if (lse_offset_bytes) *lse_offset_bytes = lay->num_slots * lay->geo.num_q_heads * int64_t(lay->geo.head_dim) * 4;
  return PS_OK;
}

const char* ps_strerror(int32_t status) {
  switch (status) {
    case PS_OK: return "ok";
    case PS_ERR_INVALID_ARG: return "invalid argument";
    case PS_ERR_SHAPE: return "geometry cannot be addressed (head counts, strides or alignment)";
    case PS_ERR_OOM: return "not enough free KV blocks (or host memory); nothing was allocated";
    case PS_ERR_REFCOUNT: return "refcount underflow or double release";
    case PS_ERR_UNSUPPORTED: return "no kernel for this dtype / head_dim / block_size combination";
    case PS_ERR_DEVICE: return "HIP call failed (see ps_last_hip_error)";
    case PS_ERR_TOO_LARGE: return "the batch's partial states exceed the library's static workspace (PS_STATIC_WORKSPACE_BYTES)";
    default: return "unknown status";
  }
}

}  // extern "C"
