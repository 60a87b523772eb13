// Partial-prefill attention on the gfx950 matrix cores: many query rows per KV head against the cached context.
//
// When a context grows by a segment, only the new tokens are prefilled (System Design, execution pipeline step 1):
// every new token is a query row on its context's shared KV, the token at position t seeing the first t + 1
// tokens.  With G q heads per KV head a chunk of c new tokens is c * G rows per KV head -- hundreds, where a decode
// step has a few dozen -- so the work is a dense contraction and the matrix cores, not HBM, are the bound.
//
// One workgroup of eight waves takes one work item: a token range of one context and KV head, and up to 256 query
// rows that see into it (four waves and 128 rows where the planner finds that enough, each then fetching two eighths of
// a tile, in a loop of its own: a wave alone on its SIMD has nobody to take turns with, and there the eight-wave loop is 6 to 13 %
// slower).  The rows are split over the waves, 32 each (the query rows resident in registers as MFMA
// B operands), and every wave walks the token range.  Two waves share a SIMD, so that the vector work of one
// (exponentials, conversions) runs under the matrix instructions of the other.
//
// The products are v_mfma_f32_32x32x16_bf16: 32 tokens x 32 rows per instruction.  On this chip it keeps the matrix
// core busy for 32 cycles and the SIMD's vector port for 8 of them, so six plain vector instructions fit into its
// shadow, where the 16x16x32 form (16 cycles, 8 of them on the port) leaves room for two: the same flops take half
// the issue slots.
//
// K and V reach the waves through LDS, as ready-made A operands: per 32-token tile the eight waves fetch one eighth
// of it each (K straight in operand layout; V as pairs of token rows, transposed inside the lane with one byte
// permute per operand register; e4m3 codes converted to bf16 once), write it to a ring of four tiles, and every wave reads the
// 8 K and 8 V operands of a tile back, 16 bytes per lane and operand, each lane exactly the slot of its own lane index (no bank
// conflicts).  A tile is thus fetched, transposed and converted once per 256 rows.  Global loads run five tiles ahead of the
// products (two tiles in registers, the others in LDS).
//
// Bound: power.  The chip holds 1.6 to 1.8 GHz here (2.4 without matrix work), and what takes cycles out of a tile gives about half
// of them back in clock.  What the loop is built for is thus fewer cycles and fewer instructions a tile, in this order:
// the two waves of a SIMD take turns at the matrix core (see the loop), nothing but the softmax stands between their turns, and
// addresses are a scalar base and a 32-bit lane offset.  Before / now, whole launches under the profiler, the stores below
// included: 32 contexts of 4096 tokens with 64 to 256 new ones, 32 heads, bf16 842 / 652 thousand cycles at 1.86 / 1.64 GHz, 452 / 398 us,
// matrix cores 38 / 49 % busy; 64 of 8192, 64 heads, e4m3 5.81 / 4.58 million at 2.11 / 1.82, 2753 / 2513, 44 / 56 %.  A tile is 138 / 127
// instructions a wave (bf16), 155 / 150 (e4m3).  The loop alone, without the profiler: 449 -> 417 us and 3031 -> 2800;
// 17 of 5626 to 11253, 32 heads, e4m3: 230 -> 197; short contexts, whose items are
// mostly their start and their states, alike (22 of 65 to 130, 62 to 251 new ones: 107 / 108).  With half the operand reads left out
// (a timing build) it would be another 3 %, which is what two row tiles a wave could gain.
//
// Per wave and tile: S^T = K Q^T (A = K: lane (m, g) holds elements 16 st + 8 g .. + 7 of token m for k-step st; B =
// Q^T likewise for query row n), whose result leaves lane (n, g) with the scores of row n against tokens
// 8 (r / 4) + 4 g + r % 4, r = 0 .. 15; online softmax with a lazily moving reference; O^T += V^T P^T with the
// probabilities as B operand exactly as they lie (registers 8 ks .. 8 ks + 7 for the 16-token step ks), V^T written
// to the ring so that position j of lane group g in step ks is token 16 ks + 8 (j / 4) + 4 g + j % 4.  A wave skips
// the tiles past what its own rows see; the per-row limit is applied only to tiles that reach past the wave's
// shortest row.  Nothing but the ring is shared between waves: no cross-wave merge, every wave writes the partial
// states of its own rows.
#include <type_traits>

#include "device_common.h"
#include "launch.h"
#include "mfma_common.h"

namespace psdev {

namespace {

constexpr int kD = kHeadDim;
constexpr int kRowsPerWave = 32;  // one 32-row tile per wave
constexpr int kTile = kTileTokens;
constexpr float kLazy = kLazyRescale;
constexpr float kLazyTop = 256.f;   // 2^kLazy
static_assert(kLazyRescale == 8.f, "kLazyTop is 2^kLazyRescale");
constexpr int kLdsDone = 0xc07f;     // s_waitcnt: LDS and scalar loads to zero (or to n: | n << 8), the other counters as they are
constexpr int kScalarMayPass = 4;    // sched_barrier: only scalar instructions

typedef __attribute__((ext_vector_type(16))) float f32x16;

// largest of eight scores, folded from the constant -inf so that three-input maxima do (see max_of4)
__device__ __forceinline__ float max_of8(const f32x16& s, int first) {
  float m = -__builtin_inff();
#pragma unroll
  for (int i = 0; i < 8; ++i) m = fmaxf(m, s[first + i]);
  return m;
}

__device__ __forceinline__ int wave_max(int x) {
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) x = max(x, __builtin_amdgcn_ds_bpermute(((int(threadIdx.x) & 63) ^ m) << 2, x));
  return __builtin_amdgcn_readfirstlane(x);
}

}  // namespace

// W: waves, eight or four.
template <int KVT, int W>
__global__ __launch_bounds__(64 * W, 2) void prefill_attention_kernel(AttnParams p, const ps_item* __restrict__ items) {
  constexpr int kStages = W == 8 ? 4 : 3;   // tiles of the ring
  __shared__ u32x4 sm_k[kStages][8][64];   // [stage][k-step][lane]: K as that lane's A operand
  __shared__ u32x4 sm_v[kStages][8][64];   // [stage][2 * column class + 16-token step][lane]: V^T as that lane's A operand
  __shared__ f32x4 sm_sc[kStages][2];      // e4m3: [stage][block] = (score scale in log2 units, log2 of the V scale, 1 / V scale, -)
  __shared__ int sm_see[W];
  struct RowPlace { int64_t state, out; };   // row of the workspace and, for a request's only state, of the output (else -1); -1: no row
  __shared__ RowPlace sm_place[W][kRowsPerWave];   // looked up ahead
  constexpr int kShares = 8 / W;   // eighths of a tile a wave fetches: one, or the same place of both 16-token blocks
  const ps_item* it = items + blockIdx.x;
  const int blk_off = __builtin_amdgcn_readfirstlane(it->blk_off);
  const int tok_begin = __builtin_amdgcn_readfirstlane(it->tok_begin);
  const int tok_end = __builtin_amdgcn_readfirstlane(it->tok_end);
  const int req_off = __builtin_amdgcn_readfirstlane(it->req_off);
  const int n_req = __builtin_amdgcn_readfirstlane(it->n_req);
  const int kv_head = __builtin_amdgcn_readfirstlane(it->kv_head);
  const int split_local = __builtin_amdgcn_readfirstlane(it->split_local);
  // visible lengths apply to a prompt's own prefix, and only where the plan found a row that sees less
  const bool limited = (__builtin_amdgcn_readfirstlane(it->kind) & kPsItemMasked) != 0;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  const int n = lane & 15;   // fetching: token within a 16-token block
  const int kg = lane >> 4;  // fetching: 8-element chunk of a 32-element piece (K), row / column class (V)
  const int g = lane >> 5;   // products: half of a k-step's 16 contraction indices
  const int G = p.group;
  const int rows = n_req * G;
  const int row_base = kRowsPerWave * wave;
  const bool has_rows = rows > row_base;   // a wave without rows only fetches
  const float neg_inf = -__builtin_inff();

  // ---- addressing: block base in SGPRs, loop-invariant lane offsets
  const int sub_shift = __builtin_ctz(unsigned(p.block_size >> 4));
  const int sub_mask = (p.block_size >> 4) - 1;
  constexpr int kEsz = KVT == PS_BF16 ? 2 : 1;
  const int tok_bytes = int(p.s_tok) * kEsz;
  const int kv_bytes = int(p.s_kv) * kEsz;
  const int64_t head_base = reinterpret_cast<int64_t>(p.kv) + int64_t(kv_head) * p.s_head * kEsz;
  const uint32_t blk_bytes = uint32_t(p.s_block * kEsz);
  const int sub_bytes = 16 * tok_bytes;
  const int sub0 = tok_begin >> 4;
  // What this wave fetches of every tile, all of it from one 16-token block (fblk) so that one block id and one
  // address per tile do.  K: token n of the block, elements 32 kst + 8 kg .. + 7 -- that is lane
  // (16 fblk + n, kg % 2) of the operand of k-step 2 kst + kg / 2.  V: the pair of token rows (vrow, vrow + 1), columns
  // 8 n + 4 (kg % 2) + x, x = 0 .. 3 -- the pair is register wave % 4 of lane (n + 16 (kg % 2), kg / 2) = this very
  // lane in the operand of column class x and step fblk; the operand's row lane % 32 is thus column
  // 8 (lane % 16) + 4 (lane / 16 % 2) + x, which the epilogue undoes.
  const int kst = wave & 3;
  auto fblk = [&](int s) __attribute__((always_inline)) { return W == 8 ? wave >> 2 : s; };   // block of the wave's share s
  const int vreg = wave & 3;
  const int vrow = 4 * (kg >> 1) + 8 * ((wave >> 1) & 1) + 2 * (wave & 1);
  const int k_lane_off = n * tok_bytes + (32 * kst + 8 * kg) * kEsz;
  const int v_lane_off = kv_bytes + vrow * tok_bytes + (8 * n + 4 * (kg & 1)) * kEsz;
  const int k_op = 2 * kst + (kg >> 1), k_slot = n + 32 * (kg & 1);
  // (constant address space: the table is read-only for the kernel's lifetime, which keeps the load a scalar one
  // whatever stands around it)
  typedef const __attribute__((address_space(4))) int32_t* const_i32_ptr;
  const const_i32_ptr blk_seg = (const_i32_ptr)(p.blk + blk_off);

  // Where this wave's block(s) of a tile lie: the physical block, and the byte offset of the 16 tokens in it.  The index is
  // clamped into the range (last_sub), so that nothing here branches around a load: a tile past the range repeats its last block,
  // which is never multiplied or masked out.
  struct Place { int id[kShares], off[kShares]; };
  int last_sub = max(sub0, ((tok_end + 15) >> 4) - 1);   // (narrowed below to what some row of the workgroup sees)
  auto locate = [&](int k) __attribute__((always_inline)) {   // wave-uniform
    Place r;
#pragma unroll
    for (int s = 0; s < kShares; ++s) {
      const int sub = min(sub0 + 2 * k + fblk(s), last_sub);
      r.id[s] = *(const_i32_ptr)((const __attribute__((address_space(4))) char*)blk_seg + (uint32_t(sub >> sub_shift) << 2));
      r.off[s] = (sub & sub_mask) * sub_bytes;
    }
    return r;
  };
  // this wave's share(s) of a tile, as loaded
  struct Fetched {
    std::conditional_t<KVT == PS_BF16, u32x4, u32x2> k[kShares];         // 8 elements of one token
    std::conditional_t<KVT == PS_BF16, u32x2, uint32_t> v[kShares][2];   // 4 columns of two token rows
    f32x2 sc[kShares];                                                   // e4m3: K and V scale of the block
  };
  auto fetch = [&](Fetched& f, const Place& pl) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < kShares; ++s) {
      typedef const __attribute__((address_space(1))) char* global_ptr;
      const global_ptr at = (global_ptr)(uint64_t(head_base) + uint64_t(uint32_t(pl.id[s])) * blk_bytes + uint32_t(pl.off[s]));
      typedef std::remove_reference_t<decltype(f.k[s])> k_word;
      typedef std::remove_reference_t<decltype(f.v[s][0])> v_word;
      f.k[s] = *(const __attribute__((address_space(1))) k_word*)(at + uint32_t(k_lane_off));
      f.v[s][0] = *(const __attribute__((address_space(1))) v_word*)(at + uint32_t(v_lane_off));
      f.v[s][1] = *(const __attribute__((address_space(1))) v_word*)(at + uint32_t(v_lane_off + tok_bytes));
      if constexpr (KVT == PS_FP8_E4M3)
        f.sc[s] = *(const __attribute__((address_space(1))) f32x2*)((global_ptr)p.scales + (int64_t(pl.id[s]) * p.num_kv_heads + kv_head) * 8);
    }
  };
  // The first two tiles and the block ids of the next two are requested at once, from the item's header alone: what
  // the rows see (request list -> visible lengths) is another two round trips to memory, which these need not wait for.
  Fetched fa, fb, fc;
  fetch(fa, locate(0));
  fetch(fb, locate(1));
  if constexpr (W == 8) fetch(fc, locate(2));
  constexpr int kAhead = W == 8 ? 3 : 2;   // tiles in the ring or about to be, ahead of the one multiplied
  const Place at0 = locate(kAhead), at1 = locate(kAhead + 1);

  // ---- this lane's query row (row lane % 32 of the wave): request, visible length, and the row itself as the
  // eight B operands of S^T = K Q^T (k-step st, lane group g: elements 16 st + 8 g .. + 7)
  int lim = 0;   // a padding row sees nothing
  bf16x8 qb[8];
#pragma unroll
  for (int st = 0; st < 8; ++st) qb[st] = as_bf16x8(u32x4{0, 0, 0, 0});
  int lim_hi = 0, lim_lo = 0x7fffffff;
  {
    const int row = row_base + (lane & 31);
    RowPlace place = {-1, -1};
    if (row < rows) {
      const int req = p.req_list[req_off + row / G];
      const int first_slot = p.slot_base[req], slots_end = p.slot_base[req + 1];
      lim = limited ? min(tok_end, p.visible[req]) : tok_end;
      const uint16_t* qrow = static_cast<const uint16_t*>(p.q) + (int64_t(req) * p.num_q_heads + kv_head * G + row % G) * kD;
#pragma unroll
      for (int st = 0; st < 8; ++st) qb[st] = as_bf16x8(*reinterpret_cast<const u32x4*>(qrow + 16 * st + 8 * g));
      lim_hi = lim;
      lim_lo = lim;
      const int h = kv_head * G + row % G;
      place.state = (int64_t(first_slot) + split_local) * p.num_q_heads + h;
      if (slots_end - first_slot == 1) place.out = int64_t(req) * p.num_q_heads + h;
    }
    if (lane < kRowsPerWave) sm_place[wave][lane] = place;
  }
  const int see_end = max(tok_begin, wave_max(lim_hi));   // no row of this wave sees a token at or past this one
  const int see_all = -wave_max(-lim_lo);                 // every row of this wave sees every token before this one
  if (lane == 0) sm_see[wave] = see_end;
  __syncthreads();
  int see_end_wg = tok_begin;
#pragma unroll
  for (int w = 0; w < W; ++w) see_end_wg = max(see_end_wg, sm_see[w]);
  see_end_wg = __builtin_amdgcn_readfirstlane(see_end_wg);
  const int n_tiles_wg = (see_end_wg - tok_begin + kTile - 1) / kTile;   // tiles the workgroup fetches
  const int n_tiles = has_rows ? (see_end - tok_begin + kTile - 1) / kTile : 0;   // tiles this wave multiplies
  const int n_whole = min(n_tiles, max(0, (see_all - tok_begin) / kTile));   // ... of which these need no per-row limit

  last_sub = max(sub0, ((see_end_wg + 15) >> 4) - 1);   // blocks past it are not fetched: nobody sees them

  // ... and its way into the ring: K as it is (e4m3: converted), V transposed -- register vreg of this lane's slot
  // in the operand of column class x holds column 8 n + 4 (kg % 2) + x of the token rows (vrow, vrow + 1)
  auto publish_k = [&](const Fetched& f, int stage) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < kShares; ++s) {
      const int b = fblk(s);
      if constexpr (KVT == PS_BF16) {
        sm_k[stage][k_op][16 * b + k_slot] = f.k[s];
      } else {
        sm_k[stage][k_op][16 * b + k_slot] = e4m3x8_to_bf16x8(f.k[s].x, f.k[s].y);
        // the block's scales, once per workgroup: the K scale folded into the score scale, the V scale as the exponent
        // offset of the probabilities and as the factor that takes it out of the row sums again
        if (kst == 0 && lane == 0) {
          const float lv = __builtin_amdgcn_logf(f.sc[s].y);
          sm_sc[stage][b] = f32x4{p.scale_log2 * f.sc[s].x, lv, fast_exp2(-lv), 0.f};
        }
      }
    }
  };
  // ragged_tag: std::true_type = the tile may be the item's last, which can reach past its range
  auto publish_v = [&](const Fetched& f, int stage, int k, auto ragged_tag) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < kShares; ++s) {
      const int b = fblk(s);
      // slots of tokens past the item's range may hold anything: zero them (their probabilities are zero)
      auto v0 = f.v[s][0], v1 = f.v[s][1];
      if (decltype(ragged_tag)::value && tok_begin + kTile * (k + 1) > tok_end) {   // (only the item's last tile can)
        const int tok = tok_begin + kTile * k + 16 * b + vrow;
        if (tok >= tok_end) v0 = decltype(v0){};
        if (tok + 1 >= tok_end) v1 = decltype(v1){};
      }
      uint32_t* dst = reinterpret_cast<uint32_t*>(&sm_v[stage][b][lane]) + vreg;   // operand 2 x + b
      if constexpr (KVT == PS_BF16) {
#pragma unroll
        for (int x = 0; x < 4; ++x)   // low (even column) or high (odd column) halves of the two rows: one byte permute
          dst[x * 2 * 64 * 4] = __builtin_amdgcn_perm(v1[x >> 1], v0[x >> 1], (x & 1) ? 0x07060302u : 0x05040100u);
      } else {
#pragma unroll
        for (int cp = 0; cp < 2; ++cp) {   // the codes of columns (2 cp, 2 cp + 1) of the two rows, then converted
          const uint32_t pair = __builtin_amdgcn_perm(v1, v0, cp ? 0x07030602u : 0x05010400u);
          dst[(2 * cp) * 2 * 64 * 4] = e4m3x2_to_bf16x2(pair, false);
          dst[(2 * cp + 1) * 2 * 64 * 4] = e4m3x2_to_bf16x2(pair, true);
        }
      }
    }
  };

  float m_run = neg_inf, l_run = 0.f;
  f32x16 acc[4];   // O^T, one block of 32 columns per column class
#pragma unroll
  for (int x = 0; x < 4; ++x)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[x][r] = 0.f;

  // One tile for this wave's rows, operands from the ring.
  // limited_tag: std::true_type applies the per-row limits (and guards rows that have seen nothing yet);
  // std::false_type promises that every row of the wave sees the whole tile.
  struct KOperands { u32x4 a[8]; };
  auto read_k = [&](int stage) __attribute__((always_inline)) {   // the 8 K operands of a stage, requested in one go
    KOperands ka;
#pragma unroll
    for (int st = 0; st < 8; ++st) ka.a[st] = sm_k[stage][st][lane];
    __builtin_amdgcn_sched_barrier(0);
    return ka;
  };
  struct Probabilities { bf16x8 b[2]; };
  struct VOperands { u32x4 a[8]; };
  auto read_v = [&](int stage) __attribute__((always_inline)) {   // the 8 V operands of a stage
    VOperands vt;
#pragma unroll
    for (int op = 0; op < 8; ++op) vt.a[op] = sm_v[stage][op][lane];
    return vt;
  };
  // raw scores S^T = K Q^T: register r of this lane = its row against token 8 (r / 4) + 4 g + r % 4 of the tile
  // (registers 0 .. 7 the first 16-token block, 8 .. 15 the second)
  auto scores = [&](const KOperands& ka) __attribute__((always_inline)) {
    f32x16 s;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
    for (int st = 0; st < 8; ++st) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(ka.a[st]), qb[st], s, 0, 0, 0);
    return s;
  };
  // softmax of a tile's scores: the probabilities as the operand of P V
  struct TileScales { f32x4 b[2]; };
  auto read_sc = [&](int stage) __attribute__((always_inline)) {
    TileScales r{};
    if constexpr (KVT == PS_FP8_E4M3) {
      r.b[0] = sm_sc[stage][0];
      r.b[1] = sm_sc[stage][1];
    }
    return r;
  };
  auto softmax = [&](f32x16 s, const TileScales& sc, int k, auto limited_tag) __attribute__((always_inline)) {
    constexpr bool kLimited = decltype(limited_tag)::value;
    const int tok0 = tok_begin + kTile * k;
    float sc_k[2], lvs[2], inv_v[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      if constexpr (KVT == PS_FP8_E4M3) {
        const f32x4 q4 = sc.b[b];
        sc_k[b] = q4.x;
        lvs[b] = q4.y;
        inv_v[b] = q4.z;
      } else {
        sc_k[b] = p.scale_log2;
        lvs[b] = 0.f;
        inv_v[b] = 1.f;
      }
    }
    if constexpr (kLimited) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (tok0 + 8 * (r >> 2) + 4 * g + (r & 3) >= lim) s[r] = neg_inf;
    }
    // The softmax reference m_run follows the row maximum lazily: it moves (and the accumulators are rescaled)
    // only when some score gets far ahead of it, so probabilities stay below 2^kLazy instead of below 1 -- the same
    // result by shift invariance of softmax.  The test is local to the lane and one wave vote decides; only when it
    // fires somewhere in the wave is the maximum of the row put together across the row's two lanes, which must
    // agree on m_run.  A row that has seen nothing yet has m_run = -inf and stays there until a score arrives.
    auto raw_max = [&]() { return fmaxf(max_of8(s, 0) * sc_k[0], max_of8(s, 8) * sc_k[1]); };
    auto move_reference = [&](float mx, float ahead_by) __attribute__((always_inline)) {
      const float row_mx = fmaxf(mx, lane_xor(mx, 32));
      const float m_new = (row_mx > m_run + ahead_by) ? row_mx : m_run;
      const float alpha = (m_new == m_run) ? 1.f : fast_exp2(m_run - m_new);   // -inf -> finite gives 0
      l_run *= alpha;
#pragma unroll
      for (int x = 0; x < 4; ++x) acc[x] *= alpha;
      m_run = m_new;
    };
    f32x16 e;   // exponents: score in log2 units, plus log2 of the block's V scale, minus the reference
    float pw[16], lsum[2];   // probabilities times the V scale; their sums per block
    auto probabilities = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        lsum[b] = 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          pw[8 * b + j] = fast_exp2(e[8 * b + j]);
          lsum[b] += pw[8 * b + j];
        }
      }
    };
    float total;   // this lane's 16 probabilities, summed
    if constexpr (kLimited) {
      // per-row limits: the test is made on the raw scores (in log2 units; the scales are positive, so a block's
      // maximum scales like its scores)
      const float mx = raw_max();
      if (__builtin_amdgcn_ballot_w64(mx > m_run + kLazy) != 0) move_reference(mx, kLazy);
      const float m_ref = (m_run == neg_inf) ? 0.f : m_run;   // keeps (-inf) - (-inf) out of the exponents
#pragma unroll
      for (int r = 0; r < 16; ++r) e[r] = __builtin_fmaf(s[r], sc_k[r >> 3], lvs[r >> 3] - m_ref);
      probabilities();
      total = (KVT == PS_FP8_E4M3) ? lsum[0] * inv_v[0] + lsum[1] * inv_v[1] : lsum[0] + lsum[1];
    } else {
      // Every row sees the whole tile: the test is made on the sum of the lane's probabilities, which the row sum
      // needs anyway -- a probability above 2^kLazy (or an infinite one: a row that has seen nothing yet has the
      // reference -inf) shows in it, and a sum above 2^kLazy means that one of its 16 terms is above 2^(kLazy - 4),
      // so in the rare branch the reference moves for every row that is that far ahead, after which the row's
      // probabilities are at most 1 and the test is quiet again.  No maximum is taken on the common path.
#pragma unroll
      for (int r = 0; r < 16; ++r) e[r] = __builtin_fmaf(s[r], sc_k[r >> 3], lvs[r >> 3] - m_run);
      probabilities();
      total = (KVT == PS_FP8_E4M3) ? lsum[0] * inv_v[0] + lsum[1] * inv_v[1] : lsum[0] + lsum[1];
      if (__builtin_amdgcn_ballot_w64(!(total <= kLazyTop)) != 0) {
        move_reference(raw_max(), kLazy - 4.f);
#pragma unroll
        for (int r = 0; r < 16; ++r) e[r] = __builtin_fmaf(s[r], sc_k[r >> 3], lvs[r >> 3] - m_run);
        probabilities();
        total = (KVT == PS_FP8_E4M3) ? lsum[0] * inv_v[0] + lsum[1] * inv_v[1] : lsum[0] + lsum[1];
      }
    }
    l_run += total;
    Probabilities pb;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int j = 0; j < 8; ++j) pb.b[b][j] = (__bf16)pw[8 * b + j];
    return pb;
  };

  // ---- stream the token range.  No branch surrounds a load, so that the counting of outstanding loads stays exact; every wave runs
  // every iteration (and every barrier), whether it has rows or not.  Two tiles per round at least, so that the fetch registers keep
  // their roles.  A loop each rather than tests inside one (a branch around the products would have the accumulators copied
  // where its sides meet): the tiles every row of the wave sees whole (eight waves: by fours, then a pair), then the rest of what the
  // wave sees with the per-row limits (a tile past it is masked out entirely), then the tiles only other waves need.  Every wave
  // passes the same number of barriers.
  publish_k(fa, 0);
  publish_v(fa, 0, 0, std::true_type{});
  fetch(fa, at0);
  publish_k(fb, 1);
  publish_v(fb, 1, 1, std::true_type{});
  fetch(fb, at1);
  Place at_nxt = locate(kAhead + 2);   // of the tile fetched next, asked for one iteration ahead
  __syncthreads();
  const int n_complete = (tok_end - tok_begin) / kTile;
  int k = 0;
  if constexpr (W == 8) {
    // Eight waves: a wave's work on a tile is two phases of about the same length, and the two waves of a SIMD take turns
    // in them: while one multiplies, the other has its softmax, and a barrier ends each phase.
    //   softmax phase k: the probabilities of tile k from its scores, nothing else
    //   product phase k: P V of tile k and the scores of tile k + 1, sixteen matrix instructions, and in their shadows
    //     everything else: each operand register is refilled from the ring right behind its product (V of tile k + 1, K of
    //     tile k + 2), tile k + 3 goes into the ring and tile k + 5 is requested from memory
    // Waves 4 .. 7 run one phase behind waves 0 .. 3.  A tile written in product phase k - 3 is complete when the later waves end
    // that phase, one before the earlier ones read its K in product phase k - 2; its place is taken by tile k + 4 in product phase
    // k + 1 of the earlier ones, after the later ones had its V in registers for product phase k: a ring of four tiles.
    // (With everything but the products in the softmax phase that phase is twice as long as the other: 3970 us against 3006 on the
    // 64 contexts above.  The product phase without its priority: 437 / 460 and 2942 / 3530.)
    KOperands ka = read_k(0);
    f32x16 s_cur = scores(ka);
    ka = read_k(1);
    VOperands vt = read_v(0);
    TileScales sc = read_sc(0);
    publish_k(fc, 2);
    publish_v(fc, 2, 2, std::true_type{});
    const bool second = wave >= 4;
    __builtin_amdgcn_s_waitcnt(kLdsDone);   // (the first barrier of the loop does not wait for the writes)
    if (second) __syncthreads();
    auto one_tile = [&](int k, auto stage, Fetched& f_pub, auto what_tag, auto ragged_tag) __attribute__((always_inline)) {
      constexpr bool kMultiply = !std::is_pointer<decltype(what_tag)>::value;
      Probabilities pb;
      if constexpr (kMultiply) pb = softmax(s_cur, sc, k, what_tag);
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_barrier();   // (nothing to wait for: the wave has written nothing since the last one)
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (kMultiply) {
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int x = i & 3, ks = i >> 2;
          acc[x] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(vt.a[2 * x + ks]), pb.b[ks], acc[x], 0, 0, 0);
          vt.a[2 * x + ks] = sm_v[(stage + 1) & 3][2 * x + ks][lane];
          if (i == 1) publish_k(f_pub, (stage + 3) & 3);
          if (i == 2) publish_v(f_pub, (stage + 3) & 3, k + 3, ragged_tag);
          if (i == 3) {
            asm volatile("" ::: "memory");   // the writes stand in front of the reads below, at least eight
            fetch(f_pub, at_nxt);
          }
          if (i == 5) at_nxt = locate(k + 6);
          __builtin_amdgcn_sched_barrier(kScalarMayPass);
        }
        f32x16 s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
        for (int st = 0; st < 8; ++st) {
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(ka.a[st]), qb[st], s, 0, 0, 0);
          ka.a[st] = sm_k[(stage + 2) & 3][st][lane];
          if (st == 1) sc = read_sc((stage + 1) & 3);
          __builtin_amdgcn_sched_barrier(kScalarMayPass);
        }
        s_cur = s;
        __builtin_amdgcn_s_setprio(0);
        // The wave's writes to the ring are done, the eight reads of K behind them need not be.
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(kLdsDone | 8 << 8);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
      } else {
        publish_k(f_pub, (stage + 3) & 3);
        publish_v(f_pub, (stage + 3) & 3, k + 3, ragged_tag);
        fetch(f_pub, at_nxt);
        at_nxt = locate(k + 6);
        __syncthreads();
      }
    };
    // (the first loops also stop short of the item's last complete tiles, so that the tiles they write, three ahead, are complete
    // ones and need no zeroing of rows past the range)
    const int n_fast = min(n_whole, n_complete - 3);
    for (; k + 4 <= n_fast; k += 4) {
      one_tile(k, std::integral_constant<int, 0>{}, fa, std::false_type{}, std::false_type{});
      one_tile(k + 1, std::integral_constant<int, 1>{}, fb, std::false_type{}, std::false_type{});
      one_tile(k + 2, std::integral_constant<int, 2>{}, fa, std::false_type{}, std::false_type{});
      one_tile(k + 3, std::integral_constant<int, 3>{}, fb, std::false_type{}, std::false_type{});
    }
    if (k + 2 <= n_fast) {
      one_tile(k, std::integral_constant<int, 0>{}, fa, std::false_type{}, std::false_type{});
      one_tile(k + 1, std::integral_constant<int, 1>{}, fb, std::false_type{}, std::false_type{});
      k += 2;
    }
    for (; k < n_tiles; k += 2) {
      one_tile(k, k, fa, std::true_type{}, std::true_type{});
      one_tile(k + 1, k + 1, fb, std::true_type{}, std::true_type{});
    }
    for (; k < n_tiles_wg; k += 2) {
      one_tile(k, k, fa, static_cast<void*>(nullptr), std::true_type{});
      one_tile(k + 1, k + 1, fb, static_cast<void*>(nullptr), std::true_type{});
    }
    if (!second) __syncthreads();
  } else {
    // Four waves: in iteration k the wave multiplies tile k (its K operands already in registers, requested during iteration
    // k - 1), requests the K operands of tile k + 1, writes its shares of tile k + 2 into the ring of three tiles, requests tile
    // k + 4 from memory, and meets the others at the barrier.
    int st_cur = 0, st_nxt = 1, st_wr = 2;   // tiles of the ring: the one multiplied, the next one, the one written
    KOperands ka_even, ka_odd;               // K operands of the even / odd tile in flight
    if (n_tiles > 0) ka_even = read_k(0);
    auto one_tile = [&](int k, Fetched& f_pub, const KOperands& ka, KOperands& ka_next, auto what_tag,
                        auto ragged_tag) __attribute__((always_inline)) {
      constexpr bool kMultiply = !std::is_pointer<decltype(what_tag)>::value;
      // (the fetching stands in front of the score products in program order and the compiler weaves it into them)
      if constexpr (kMultiply) ka_next = read_k(st_nxt);
      publish_k(f_pub, st_wr);
      publish_v(f_pub, st_wr, k + 2, ragged_tag);
      fetch(f_pub, at_nxt);
      at_nxt = locate(k + 5);
      if constexpr (kMultiply) {
        const f32x16 s = scores(ka);
        // the V operands are requested now, all eight, so that they arrive under the softmax (left to itself the
        // compiler requests each one right before its products, and the wave sits out the LDS latency eight times)
        const VOperands vt = read_v(st_cur);
        __builtin_amdgcn_sched_barrier(0);
        const Probabilities pb = softmax(s, read_sc(st_cur), k, what_tag);
#pragma unroll
        for (int i = 0; i < 8; ++i)
          acc[i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(vt.a[2 * (i & 3) + (i >> 2)]), pb.b[i >> 2], acc[i & 3], 0, 0, 0);
      }
      const int st_free = st_cur;
      st_cur = st_nxt;
      st_nxt = st_wr;
      st_wr = st_free;
      __syncthreads();
    };
    const int n_fast = min(n_whole, n_complete - 2);
    for (; k + 2 <= n_fast; k += 2) {
      one_tile(k, fa, ka_even, ka_odd, std::false_type{}, std::false_type{});
      one_tile(k + 1, fb, ka_odd, ka_even, std::false_type{}, std::false_type{});
    }
    for (; k < n_tiles; k += 2) {
      one_tile(k, fa, ka_even, ka_odd, std::true_type{}, std::true_type{});
      one_tile(k + 1, fb, ka_odd, ka_even, std::true_type{}, std::true_type{});
    }
    for (; k < n_tiles_wg; k += 2) {
      one_tile(k, fa, ka_even, ka_odd, static_cast<void*>(nullptr), std::true_type{});
      one_tile(k + 1, fb, ka_odd, ka_even, static_cast<void*>(nullptr), std::true_type{});
    }
  }

  // ---- one partial state per row: register r of column class x is column
  // 64 (r / 4 % 2) + 32 g + 8 (r % 4) + 4 (r / 8) + x of this lane's row.  The rows go through the ring, which is free now (8 KiB a
  // wave, 16-byte pieces at their index xor the row's against bank conflicts), so that a store covers 256 bytes of four rows
  // instead of 16 bytes of 64 places: 32 contexts of 4096 tokens 426 -> 408 us; where items are a few tiles and mostly their start and
  // their stores, 22 contexts of 65 to 130 with 62 to 251 new tokens, 64 heads, e4m3 106 -> 84, 11 of 165 to 331 33 -> 26.
  if (has_rows) {
    float l = l_run;
    l += lane_xor(l, 32);
    const float inv = l > 0.f ? 1.f / l : 0.f;
    const float lse = l > 0.f ? (m_run + __builtin_amdgcn_logf(l)) * kLn2 : neg_inf;
    u32x4* const turn = wave < kStages ? &sm_k[wave][0][0] : &sm_v[wave - kStages][0][0];
    const int my_row = lane & 31;
    // piece c (of 16) of row r; and what a lane reads back: row 4 i + lane / 16, piece lane % 16
    auto piece = [&](int r, int c) __attribute__((always_inline)) { return turn + 16 * r + (c ^ (r & 15)); };
    auto row_at = [&](int i) __attribute__((always_inline)) { return 4 * i + (lane >> 4); };
    const RowPlace mine = sm_place[wave][my_row];
    const bool final_row = p.out && mine.out >= 0;
    if (mine.state >= 0 && g == 0) {
      if (!final_row || p.keep_states) p.ws_lse[mine.state] = lse;
      if (final_row && p.out_lse) p.out_lse[mine.out] = lse;
    }
    if (__builtin_amdgcn_ballot_w64(mine.state >= 0 && (!final_row || p.keep_states)) != 0) {
#pragma unroll
      for (int half = 0; half < 2; ++half) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {   // columns 64 half ..: registers r with r / 4 % 2 == half
          const int r = 4 * half + 8 * (i >> 2) + (i & 3);
          *reinterpret_cast<f32x4*>(piece(my_row, 8 * g + 2 * (r & 3) + (r >> 3))) = f32x4{acc[0][r], acc[1][r], acc[2][r], acc[3][r]} * inv;
        }
        wave_lds_order();
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int r = row_at(i);
          const f32x4 v = *reinterpret_cast<const f32x4*>(piece(r, lane & 15));
          const RowPlace at = sm_place[wave][r];
          if (at.state >= 0 && (at.out < 0 || !p.out || p.keep_states))
            *reinterpret_cast<f32x4*>(p.ws_o + at.state * kD + 64 * half + 4 * (lane & 15)) = v;
        }
        wave_lds_order();
      }
    }
    if (__builtin_amdgcn_ballot_w64(final_row) != 0) {
      // The request's only partial state is the result: rounded and stored here as well, so
      // that no merge has to read it back (32 contexts of 4096 + 64..256 tokens, a step with state and merge / state and
      // row / row alone 415 / 403 / 383 us; 64 contexts of 8192 tokens, 64 query heads, e4m3 KV 2763 / 2704 / 2641 us).
      const bool some = l > 0.f;   // a row that saw nothing is zero
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        bf16x8 w;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          w[x] = (__bf16)(some ? acc[x][r] * inv : 0.f);
          w[4 + x] = (__bf16)(some ? acc[x][r + 8] * inv : 0.f);
        }
        *reinterpret_cast<bf16x8*>(piece(my_row, 8 * (r >> 2) + 4 * g + (r & 3))) = w;
      }
      wave_lds_order();
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int r = row_at(i);
        const u32x4 v = *piece(r, lane & 15);
        const RowPlace at = sm_place[wave][r];
        if (at.out >= 0) *reinterpret_cast<u32x4*>(static_cast<uint16_t*>(p.out) + at.out * kD + 8 * (lane & 15)) = v;
      }
    }
  }
}

int32_t launch_prefill_attention(const AttnParams& p, const ps_geometry& g, const ps_item* items, int num_items,
                                 int rows, hipStream_t st) {
  if (num_items <= 0) return PS_OK;
  const int spb = g.block_size / 16;
  if (g.head_dim != kD || g.q_dtype != PS_BF16 || g.block_size % 16 != 0 || (spb & (spb - 1)) != 0)
    return PS_ERR_UNSUPPORTED;
  const dim3 grid(num_items);
  if (g.kv_dtype == PS_BF16) {
    if (rows <= 128) hipLaunchKernelGGL((prefill_attention_kernel<PS_BF16, 4>), grid, dim3(256), 0, st, p, items);
    else hipLaunchKernelGGL((prefill_attention_kernel<PS_BF16, 8>), grid, dim3(512), 0, st, p, items);
  } else if (g.kv_dtype == PS_FP8_E4M3) {
    if (rows <= 128) hipLaunchKernelGGL((prefill_attention_kernel<PS_FP8_E4M3, 4>), grid, dim3(256), 0, st, p, items);
    else hipLaunchKernelGGL((prefill_attention_kernel<PS_FP8_E4M3, 8>), grid, dim3(512), 0, st, p, items);
  }
  else
    return PS_ERR_UNSUPPORTED;
  return PS_OK;
}

}  // namespace psdev
