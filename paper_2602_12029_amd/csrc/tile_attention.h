// Grouped-query attention over KV token ranges with float32 probabilities, on the gfx950 matrix cores: the kernel of
// the PS_VARIANT_WAVE family for paged pools with blocks of 16 tokens or a multiple of that.  Every storage format and
// head size of the library runs here (KV float32 / bf16 / e4m3, queries float32 / bf16, d = 64, 128, 256).
//
// One workgroup (4 waves) takes one work item: a token range of one KV segment and one KV head, applied to every query
// row that reads it.  The waves take 16- or 32-token tiles of the range in turn, stream K and V straight into matrix
// operand registers, keep an online softmax per row and merge through LDS at the end; one partial state per row leaves
// the workgroup.  (Short private items go four to a workgroup, a wave each, with nothing to merge: 748 items of 1 to 257 tokens
// 19.9 -> 12.8 us a launch, 3076 of 256-wide heads 159 -> 126.)  As in the bf16 decode kernel the products are the transposed ones,
//   S^T[token, row] = K[token, :] . Q[row, :]        A = K, B = Q^T
//   O^T[dcol, row] += V^T[dcol, token] . P^T[token, row]        A = V^T, B = P^T
// so that a lane's scores are, in place, its operand of the second product, and no cross-lane traffic is needed but
// the (rare) move of the softmax reference.
//
// Two forms of the products, both with probabilities that keep all of their 24 bits:
//   * float32 operands (KV or queries in float32): v_mfma_f32_16x16x4_f32.  Lane (n, kg) of a wave owns 16 bytes per
//     64-byte piece of token n (K: four k-steps per load, the contraction index permuted alike in K and Q) and of
//     tokens 4 kg .. 4 kg + 3 (V: a 16-lane group covers a whole row, and element e of the load is the operand of the
//     column group {columns congruent e}), so nothing is transposed; narrower formats are widened in the registers.
//   * bf16 queries over bf16 or e4m3 KV: v_mfma_f32_16x16x32_bf16.  K . Q is exact in the products as it is; a
//     probability goes in as the sum of three bf16 terms (8 + 8 + 8 bits: the split is exact), three products instead
//     of one, on an instruction of sixteen times the rate.  V is transposed inside the lane as in the decode kernel.
//
// Bound: HBM with up to 16 rows per KV head, and with bf16 products up to 32 rows of heads up to 128 (float32: 64 products
// of 32 cycles per 16 KiB tile and wave let 19.6 TB/s through at 16 rows); the vector form this replaces repeats its softmax on
// every lane of a row and walks the tokens once
// per 8 query rows.  Measured, whole step with the merge: 36 float32 requests on 12 contexts of 512 to 4096 tokens, d = 128,
// 214 MB, 137 -> 42.7 us (5.0 TB/s); 72 bf16 requests with 64-wide heads on 24 contexts of 1024 to 6144 tokens, 193 MB,
// 319 -> 38.9 us (5.0 TB/s); two requests on one 256-token prompt 18.3 -> 8.4 us.  K comes in whole 128-byte lines, as in the
// decode kernel: with half a line per token and load the two batches took 44.9 and 42.3 us.
// More rows are spread over the waves (SPREAD): two or four of them take a row tile each of the same tokens, and what the first
// fetches the others find in the caches.  That keeps the registers of the 16-row form -- two workgroups a compute unit with heads
// of up to 128 -- and walks the tokens once for 64 rows: 480 requests on 60 contexts with 256-wide heads 559 -> 357 us against
// passes of 16 rows.  Where a launch streams from HBM with bf16 products the form with all row tiles in a wave is faster (the
// planner's rule has both sides).  Error of float32 outputs against 64
// bits, mean over sixteen batches: 3.4e-7 -> 3.1e-7 (with the products in one chain per score it was 4.8e-7).
#pragma once
#include "device_common.h"
#include "launch.h"
#include "mfma_common.h"

namespace psdev {

namespace tile {

constexpr int kWaves = 4;
// log2 units a score may run ahead of a row's softmax reference before the reference moves
constexpr float kLazy = kLazyRescale;

template <int KVT>
constexpr int elem_bytes() { return KVT == PS_F32 ? 4 : (KVT == PS_BF16 ? 2 : 1); }

// Shape of a tile for a head size and a pair of formats.
template <int D, int KVT, int QT>
struct Shape {
  static constexpr int kEsz = elem_bytes<KVT>();
  static constexpr bool kSplit = QT == PS_BF16 && KVT != PS_F32;   // bf16 products, probabilities in three terms
  // 16-token blocks per tile: two (the bf16 product contracts over 32 tokens), one where a block alone fills 32 or
  // more registers of a wave
  static constexpr int kBlocks = (!kSplit && D * kEsz >= 256) ? 1 : 2;
  static constexpr int kTokens = 16 * kBlocks;
  static constexpr int kKLoads = D * kEsz / 64;                    // 16-byte loads per lane and block of K
  static constexpr int kKElems = 16 / kEsz;                        // elements per such load
  static constexpr bool kLines = kKLoads % 2 == 0;                 // K is fetched in whole 128-byte lines (rows of 64 bytes: no)
  static constexpr int kVBytes = (D / 16) * kEsz;                  // bytes of a V row per lane
  static constexpr int kVChunk = kVBytes < 16 ? kVBytes : 16;      // ... fetched in loads of this size
  static constexpr int kVLoads = kVBytes / kVChunk;
  static constexpr int kVElems = kVChunk / kEsz;                   // columns per such load
  static constexpr int kVWords = kVChunk / 4;
  static constexpr int kGroups = D / 16;                           // column groups of the accumulator (kVLoads * kVElems)
  static constexpr int kBufferRegs = kBlocks * (D * kEsz / 8);     // registers of one tile buffer
  // tile buffers in flight: 16 KiB and more per wave and buffer need no third one
  static constexpr int kRing = kBufferRegs >= 64 ? 2 : 3;
  static constexpr int kQRow = kSplit ? D + 8 : D + 4;             // padded query row in LDS, elements
};

template <int WORDS>
struct LoadWords;
template <> struct LoadWords<4> {
  typedef u32x4 type;
  template <int POLICY>
  static __device__ __forceinline__ type load(__amdgpu_buffer_rsrc_t rs, int voff, int soff) { return __builtin_amdgcn_raw_buffer_load_b128(rs, voff, soff, POLICY); }
};
template <> struct LoadWords<2> {
  typedef u32x2 type;
  template <int POLICY>
  static __device__ __forceinline__ type load(__amdgpu_buffer_rsrc_t rs, int voff, int soff) { return __builtin_amdgcn_raw_buffer_load_b64(rs, voff, soff, POLICY); }
};
template <> struct LoadWords<1> {
  typedef __attribute__((ext_vector_type(1))) uint32_t type;
  template <int POLICY>
  static __device__ __forceinline__ type load(__amdgpu_buffer_rsrc_t rs, int voff, int soff) { return type{__builtin_amdgcn_raw_buffer_load_b32(rs, voff, soff, POLICY)}; }
};

// element e of a few packed words, as float32 (exact)
template <int KVT, typename V>
__device__ __forceinline__ float widen(const V& w, int e) {
  if constexpr (KVT == PS_F32) return __uint_as_float(w[e]);
  else if constexpr (KVT == PS_BF16) return (e & 1) ? __uint_as_float(w[e >> 1] & 0xffff0000u) : __uint_as_float(w[e >> 1] << 16);
  else {
    const f32x2 pair = (e & 2) ? __builtin_amdgcn_cvt_pk_f32_fp8(w[e >> 2], true) : __builtin_amdgcn_cvt_pk_f32_fp8(w[e >> 2], false);
    return (e & 1) ? pair.y : pair.x;
  }
}

// raw K/V of one tile as loaded
template <int D, int KVT, int QT>
struct Regs {
  typedef Shape<D, KVT, QT> S;
  u32x4 k[S::kBlocks][S::kKLoads];
  typename LoadWords<S::kVWords>::type v[S::kBlocks][4][S::kVLoads];   // [block][token 4 kg + j][piece of the row]
};

// LDS of a workgroup: query rows (of a wave's own item: 16 each), then what the waves of a shared item merge.
template <int D, int KVT, int QT, int ROW_TILES>
struct Lds {
  typedef Shape<D, KVT, QT> S;
  typedef std::conditional_t<S::kSplit, uint16_t, float> q_elem;
  union {
    struct {
      __attribute__((aligned(16))) q_elem q[16 * ROW_TILES][S::kQRow];
      __attribute__((aligned(16))) float o[kWaves][16][D + 4];
      float m[kWaves][16], l[kWaves][16];
    };
    __attribute__((aligned(16))) q_elem q_own[kWaves][16][S::kQRow];
  };
};

// One item: by the four waves of a workgroup, or (SOLO, up to 16 rows) by one wave alone.
// NT: 16-row tiles a pass over the tokens carries at most (an item with fewer rows takes the narrowest of 1, 2, 4
// that holds them; one with more walks its tokens again).
// STREAM: K/V loads are non-temporal (the launch's ranges are read by one item each, or nearly so).
// SPREAD: items of more than 16 rows go a row tile to a wave (NT is 1).
template <int D, int KVT, int QT, int NT, bool STREAM, bool SOLO, bool SPREAD, typename LDS>
__device__ __forceinline__ void attend_item(const AttnParams& p, int item, LDS& lds) {
  typedef Shape<D, KVT, QT> S;
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  auto* sm_q = SOLO ? lds.q_own[wave] : lds.q;
  auto* sm_o = lds.o;
  auto* sm_m = lds.m;
  auto* sm_l = lds.l;
  const ps_item* ip = p.items + item;
  const int blk_off = __builtin_amdgcn_readfirstlane(ip->blk_off);
  const int tok_begin = __builtin_amdgcn_readfirstlane(ip->tok_begin);
  const int tok_end = __builtin_amdgcn_readfirstlane(ip->tok_end);
  const int req_off = __builtin_amdgcn_readfirstlane(ip->req_off);
  const int rows = __builtin_amdgcn_readfirstlane(ip->n_req) * p.group;
  const int kv_head = __builtin_amdgcn_readfirstlane(ip->kv_head);
  const int split_local = __builtin_amdgcn_readfirstlane(ip->split_local);
  const bool masked = (__builtin_amdgcn_readfirstlane(ip->kind) & kPsItemMasked) != 0;

  const int lane = threadIdx.x & 63;
  const int n = lane & 15;   // query row of a row tile / token of a block (K) / column lane (V), by role
  const int kg = lane >> 4;
  const int G = p.group;
  const float neg_inf = -__builtin_inff();

  // ---- addressing: a descriptor per 16-token block and plane (scalar), loop-invariant lane offsets
  const int spb = p.block_size >> 4;                  // 16-token blocks per physical block (>= 1)
  const int tok_bytes = int(p.s_tok) * S::kEsz;
  const int64_t head_k = reinterpret_cast<int64_t>(p.kv) + int64_t(kv_head) * p.s_head * S::kEsz;
  const int64_t plane_bytes = p.s_kv * S::kEsz;
  const int64_t blk_bytes = p.s_block * S::kEsz;
  const int sub_bytes = 16 * tok_bytes;
  const int k_lane_off = S::kLines ? (n & 7) * tok_bytes + 16 * ((n >> 3) + 2 * kg) : n * tok_bytes + 16 * kg;
  const int v_lane_off = 4 * kg * tok_bytes + n * S::kVChunk;
  const int sub0 = tok_begin >> 4, sub_end = (tok_end + 15) >> 4;
  typedef const __attribute__((address_space(4))) int32_t* const_i32_ptr;
  const const_i32_ptr blk_seg = (const_i32_ptr)(p.blk + blk_off);
  const int tiles_total = (sub_end - sub0 + S::kBlocks - 1) / S::kBlocks;

  // where a tile's blocks lie (scalar): physical block, and byte offset of the 16 tokens in it (-1: past the range)
  struct Place { int id[S::kBlocks], off[S::kBlocks]; };
  constexpr int kPolicy = STREAM ? kNonTemporal : 0;
  auto fetch = [&](Regs<D, KVT, QT>& r, const Place& pl) __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < S::kBlocks; ++b) {
      const int64_t addr = head_k + int64_t(pl.id[b]) * blk_bytes + max(pl.off[b], 0);
      const int size = pl.off[b] >= 0 ? 0x7fffffff : 0;
      const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(addr), 0, size, 0x00020000);
      const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(addr + plane_bytes), 0, size, 0x00020000);
#pragma unroll
      for (int s = 0; s < S::kKLoads; ++s)   // kLines: tokens 8 (s % 2) .., line s / 2 of their rows
        r.k[b][s] = S::kLines ? __builtin_amdgcn_raw_buffer_load_b128(rk, k_lane_off + 128 * (s >> 1), 8 * (s & 1) * tok_bytes, kPolicy)
                              : __builtin_amdgcn_raw_buffer_load_b128(rk, k_lane_off + 64 * s, 0, kPolicy);
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int c = 0; c < S::kVLoads; ++c)
          r.v[b][j][c] = LoadWords<S::kVWords>::template load<kPolicy>(rv, v_lane_off + 16 * S::kVChunk * c, j * tok_bytes);
    }
  };

  // One pass over the tokens for rows [row0, row0 + 16 M), or, SPREAD, [row0, row0 + (16 << spread)).
  auto pass = [&](int row0, auto tiles_tag, int spread) __attribute__((always_inline)) {
    constexpr int M = decltype(tiles_tag)::value;
    const int row_tile = SPREAD ? wave & ((1 << spread) - 1) : 0;
    // the wave's tiles of the item: tile0 + (k << step_shift)
    const int step_shift = SOLO ? 0 : SPREAD ? 2 - spread : 2, tile0 = SOLO ? 0 : SPREAD ? wave >> spread : wave;
    const int my_tiles = tiles_total > tile0 ? ((tiles_total - tile0 - 1) >> step_shift) + 1 : 0;
    // The table entry is read without a branch (index clamped into the range), so that outstanding loads are counted
    // exactly in the streaming loop; a block past the range gets a descriptor of size zero and is not fetched.
    auto locate = [&](int k) __attribute__((always_inline)) {
      Place pl;
#pragma unroll
      for (int b = 0; b < S::kBlocks; ++b) {
        const int sub = sub0 + S::kBlocks * (tile0 + (k << step_shift)) + b;
        const int c = min(sub, sub_end - 1);
        const int block = spb == 1 ? c : c / spb;
        pl.id[b] = blk_seg[block];
        pl.off[b] = sub < sub_end ? (c - block * spb) * sub_bytes : -1;
      }
      return pl;
    };
    // the first tiles go out from the header and the block table alone; the query rows follow while they fly
    Regs<D, KVT, QT> buf[S::kRing];
    Place at[S::kRing];
#pragma unroll
    for (int u = 0; u < S::kRing - 1; ++u) {
      at[u] = locate(u);
      fetch(buf[u], at[u]);
    }
    at[S::kRing - 1] = locate(S::kRing - 1);
    // e4m3: score scale and V scale of a tile's blocks.  A K scale may be anything finite that a caller's own quantiser
    // writes: zero (a tile of zeros by amax / 448) goes in as 2^-100, which leaves the scores 0 to the last digit and a masked
    // slot -inf; the sign of a negative one is moved to the scores (`flip`, scalar).
    struct Scales { float k[S::kBlocks], v[S::kBlocks]; bool flip[S::kBlocks]; };
    auto scales_of = [&](const Place& pl) __attribute__((always_inline)) {
      Scales sc;
#pragma unroll
      for (int b = 0; b < S::kBlocks; ++b) {
        sc.k[b] = p.scale_log2;
        sc.v[b] = 1.f;
        sc.flip[b] = false;
        if constexpr (KVT == PS_FP8_E4M3) {
          typedef const __attribute__((address_space(4))) float* const_f32_ptr;
          const const_f32_ptr s2 = (const_f32_ptr)(p.scales + (int64_t(pl.id[b]) * p.num_kv_heads + kv_head) * 2);
          const uint32_t bits = __float_as_uint(s2[0]), size = bits & 0x7fffffffu;
          sc.k[b] *= __uint_as_float(size ? size : __float_as_uint(0x1p-100f));
          sc.flip[b] = (bits >> 31) != 0;
          sc.v[b] = s2[1];
        }
      }
      return sc;
    };
    Scales scl[S::kRing];
#pragma unroll
    for (int u = 0; u < S::kRing - 1; ++u) scl[u] = scales_of(at[u]);

    // query rows -> LDS (float32 form: widened; rows past the item: zero).  A wave with an item of its own fills those
    // that the item has (the others' sums go nowhere).
    {
      constexpr int kQEsz = QT == PS_F32 ? 4 : 2;
      constexpr int kPieces = D * kQEsz / 16;          // 16-byte pieces of a query row
      const int pieces = (SOLO ? rows : SPREAD ? 16 << spread : 16 * M) * kPieces;
      for (int i = SOLO ? lane : int(threadIdx.x); i < pieces; i += SOLO ? 64 : 256) {
        const int r = i / kPieces, c = i % kPieces;
        u32x4 w = {0, 0, 0, 0};
        if (row0 + r < rows) {
          const int row = row0 + r;
          const int64_t at_row = int64_t(p.req_list[req_off + row / G]) * p.num_q_heads + kv_head * G + row % G;
          w = *reinterpret_cast<const u32x4*>(static_cast<const char*>(p.q) + (at_row * D) * kQEsz + 16 * c);
        }
        if constexpr (S::kSplit) {
          *reinterpret_cast<u32x4*>(&sm_q[r][8 * c]) = w;
        } else if constexpr (QT == PS_F32) {
          *reinterpret_cast<u32x4*>(&sm_q[r][4 * c]) = w;
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e) sm_q[r][8 * c + e] = widen<PS_BF16>(w, e);
        }
      }
    }
    int lim[M];   // first token the lane's row does not see
#pragma unroll
    for (int t = 0; t < M; ++t) {
      lim[t] = tok_end;
      const int row = row0 + 16 * (row_tile + t) + n;
      if (masked && row < rows) lim[t] = min(tok_end, p.visible[p.req_list[req_off + row / G]]);
    }
    if constexpr (SOLO) wave_lds_order();
    else __syncthreads();

    float m_run[M], l_run[M];
    f32x4 acc[M][S::kGroups];
#pragma unroll
    for (int t = 0; t < M; ++t) {
      m_run[t] = neg_inf;
      l_run[t] = 0.f;
#pragma unroll
      for (int c = 0; c < S::kGroups; ++c) acc[t][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    auto multiply = [&](Regs<D, KVT, QT>& r, const Scales& sc, int k) __attribute__((always_inline)) {
      const int tok0 = tok_begin + S::kTokens * (tile0 + (k << step_shift));
      const bool whole = !masked && tok0 + S::kTokens <= tok_end;   // every row sees the whole tile
      if constexpr (S::kLines) {   // every lane its own token: chunks 2 kg and 2 kg + 1 of line s / 2
#pragma unroll
        for (int b = 0; b < S::kBlocks; ++b)
#pragma unroll
          for (int s = 0; s < S::kKLoads; s += 2) {
            const u32x4 even = k_even(r.k[b][s], r.k[b][s + 1]), odd = k_odd(r.k[b][s], r.k[b][s + 1]);
            r.k[b][s] = even;
            r.k[b][s + 1] = odd;
          }
      }
      auto k_elem = [&](int st) { return (S::kLines ? 128 * (st >> 1) + 32 * kg + 16 * (st & 1) : 64 * st + 16 * kg) / S::kEsz; };
      // ---- scores of every row tile
      // (float32 form: the products are summed as a tree -- four chains over two 64-byte pieces, their pairs, the pieces of
      // each half of the row, the halves -- since long runs of roundings at the magnitude of a large score would cost the
      // softmax its last digits)
      constexpr int kChains = S::kSplit ? 1 : 4;
      constexpr int kSegment = KVT == PS_F32 ? 2 : 1;   // loads per run of the chains
      f32x4 s[M][S::kBlocks], part[M][S::kBlocks][kChains], first_half[M][S::kBlocks];
#pragma unroll
      for (int t = 0; t < M; ++t)
#pragma unroll
        for (int b = 0; b < S::kBlocks; ++b) {
          s[t][b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int e = 0; e < kChains; ++e) part[t][b][e] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
      for (int st = 0; st < S::kKLoads; ++st) {
        if constexpr (S::kSplit) {
          // a 16-byte load is one k-step of bf16, two of e4m3
#pragma unroll
          for (int half = 0; half < (KVT == PS_BF16 ? 1 : 2); ++half) {
            bf16x8 ka[S::kBlocks];
#pragma unroll
            for (int b = 0; b < S::kBlocks; ++b)
              ka[b] = KVT == PS_BF16 ? as_bf16x8(r.k[b][st]) : as_bf16x8(e4m3x8_to_bf16x8(r.k[b][st][2 * half], r.k[b][st][2 * half + 1]));
#pragma unroll
            for (int t = 0; t < M; ++t) {
              const bf16x8 qb = as_bf16x8(*reinterpret_cast<const u32x4*>(&sm_q[16 * (row_tile + t) + n][k_elem(st) + 8 * half]));
#pragma unroll
              for (int b = 0; b < S::kBlocks; ++b) s[t][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[b], qb, s[t][b], 0, 0, 0);
            }
          }
        } else {
#pragma unroll
          for (int e4 = 0; e4 < S::kKElems; e4 += 4) {
            float kf[S::kBlocks][4];
#pragma unroll
            for (int b = 0; b < S::kBlocks; ++b)
#pragma unroll
              for (int e = 0; e < 4; ++e) kf[b][e] = widen<KVT>(r.k[b][st], e4 + e);
#pragma unroll
            for (int t = 0; t < M; ++t) {
              const f32x4 qf = *reinterpret_cast<const f32x4*>(&sm_q[16 * (row_tile + t) + n][k_elem(st) + e4]);
#pragma unroll
              for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int b = 0; b < S::kBlocks; ++b) part[t][b][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[b][e], qf[e], part[t][b][e], 0, 0, 0);
            }
          }
          if ((st + 1) % kSegment == 0) {
#pragma unroll
            for (int t = 0; t < M; ++t)
#pragma unroll
              for (int b = 0; b < S::kBlocks; ++b) {
                s[t][b] += (part[t][b][0] + part[t][b][1]) + (part[t][b][2] + part[t][b][3]);
                if (st + 1 == S::kKLoads / 2) {
                  first_half[t][b] = s[t][b];
                  s[t][b] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
                if (st + 1 == S::kKLoads && S::kKLoads > kSegment) s[t][b] += first_half[t][b];
#pragma unroll
                for (int e = 0; e < kChains; ++e) part[t][b][e] = f32x4{0.f, 0.f, 0.f, 0.f};
              }
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
      if constexpr (KVT == PS_FP8_E4M3) {
#pragma unroll
        for (int b = 0; b < S::kBlocks; ++b)
          if (sc.flip[b])
#pragma unroll
            for (int t = 0; t < M; ++t) s[t][b] = -s[t][b];
      }
      // ---- slots past the range may hold anything: their scores are -inf and their V rows zero
      if (!whole) {
#pragma unroll
        for (int b = 0; b < S::kBlocks; ++b)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int tok = tok0 + 16 * b + 4 * kg + j;
#pragma unroll
            for (int t = 0; t < M; ++t)
              if (tok >= lim[t]) s[t][b][j] = neg_inf;
            if (tok >= tok_end)
#pragma unroll
              for (int c = 0; c < S::kVLoads; ++c) r.v[b][j][c] = decltype(r.v[b][j][c] + r.v[b][j][c]){};
          }
      }
      // ---- online softmax, the reference following the row maximum lazily (see the bf16 decode kernel)
#pragma unroll
      for (int t = 0; t < M; ++t) {
        float mx = neg_inf;
#pragma unroll
        for (int b = 0; b < S::kBlocks; ++b) mx = fmaxf(mx, max_of4(s[t][b]) * sc.k[b]);
        if (__builtin_amdgcn_ballot_w64(mx > m_run[t] + kLazy) != 0) {
          mx = fmaxf(mx, lane_xor(mx, 16));
          mx = fmaxf(mx, lane_xor(mx, 32));
          const float m_new = (mx > m_run[t] + kLazy) ? mx : m_run[t];
          const float alpha = (m_new == m_run[t]) ? 1.f : fast_exp2(m_run[t] - m_new);
          l_run[t] *= alpha;
#pragma unroll
          for (int c = 0; c < S::kGroups; ++c) acc[t][c] *= alpha;
          m_run[t] = m_new;
        }
        const float m_ref = m_run[t] == neg_inf ? 0.f : m_run[t];   // a row that has seen nothing yet: exponents stay -inf
#pragma unroll
        for (int b = 0; b < S::kBlocks; ++b)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float w = fast_exp2(__builtin_fmaf(s[t][b][j], sc.k[b], -m_ref));
            l_run[t] += w;
            s[t][b][j] = KVT == PS_FP8_E4M3 ? w * sc.v[b] : w;
          }
      }
      // ---- O^T += V^T P^T
      if constexpr (S::kSplit) {
        // The probability as an exact sum of three bf16 terms, by truncation: its upper eight bits, the next eight, the
        // rest, none negative (or none positive, where e4m3's V scale is negative: no infinities there).  Terms that would be zero are 2^-126 (lost in the sums) where the probability is not:
        // an infinite V then gives the infinity it should and no 0 * inf.
        bf16x8 pb[M][3];
        constexpr float kTiny = 0x1p-126f;
#pragma unroll
        for (int t = 0; t < M; ++t)
#pragma unroll
          for (int b = 0; b < S::kBlocks; ++b) {
            uint32_t word[3][2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
              float mid[2], low[2];
#pragma unroll
              for (int j = 0; j < 2; ++j) {
                const float w = s[t][b][2 * i + j], floor = fminf(w, kTiny);
                mid[j] = w - __uint_as_float(__float_as_uint(w) & 0xffff0000u);
                low[j] = fmaxf(mid[j] - __uint_as_float(__float_as_uint(mid[j]) & 0xffff0000u), floor);
                mid[j] = fmaxf(mid[j], floor);
              }
              word[0][i] = __builtin_amdgcn_perm(__float_as_uint(s[t][b][2 * i + 1]), __float_as_uint(s[t][b][2 * i]), 0x07060302u);
              word[1][i] = __builtin_amdgcn_perm(__float_as_uint(mid[1]), __float_as_uint(mid[0]), 0x07060302u);
              word[2][i] = __builtin_amdgcn_perm(__float_as_uint(low[1]), __float_as_uint(low[0]), 0x07060302u);
            }
#pragma unroll
            for (int term = 0; term < 3; ++term) {
              u32x4 w4 = __builtin_bit_cast(u32x4, pb[t][term]);
              w4[2 * b] = word[term][0];
              w4[2 * b + 1] = word[term][1];
              pb[t][term] = as_bf16x8(w4);
            }
          }
#pragma unroll
        for (int c = 0; c < S::kVLoads; ++c)
#pragma unroll
          for (int pair = 0; pair < S::kVElems / 2; ++pair) {
            // columns (2 pair, 2 pair + 1) of this lane's eight token rows
            uint32_t w0[4], w1[4];
#pragma unroll
            for (int i2 = 0; i2 < 4; ++i2) {
              const auto& lo = r.v[i2 >> 1][2 * (i2 & 1)][c];
              const auto& hi = r.v[i2 >> 1][2 * (i2 & 1) + 1][c];
              if constexpr (KVT == PS_BF16) {
                w0[i2] = __builtin_amdgcn_perm(hi[pair], lo[pair], 0x05040100u);
                w1[i2] = __builtin_amdgcn_perm(hi[pair], lo[pair], 0x07060302u);
              } else {
                const uint32_t codes = __builtin_amdgcn_perm(hi[pair >> 1], lo[pair >> 1], (pair & 1) ? 0x07030602u : 0x05010400u);
                w0[i2] = e4m3x2_to_bf16x2(codes, false);
                w1[i2] = e4m3x2_to_bf16x2(codes, true);
              }
            }
            const bf16x8 v0 = as_bf16x8(u32x4{w0[0], w0[1], w0[2], w0[3]}), v1 = as_bf16x8(u32x4{w1[0], w1[1], w1[2], w1[3]});
            const int g0 = c * S::kVElems + 2 * pair;
#pragma unroll
            for (int t = 0; t < M; ++t)
#pragma unroll
              for (int term = 2; term >= 0; --term) {   // the smallest terms first
                acc[t][g0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v0, pb[t][term], acc[t][g0], 0, 0, 0);
                acc[t][g0 + 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v1, pb[t][term], acc[t][g0 + 1], 0, 0, 0);
              }
          }
      } else {
        // (a block's sixteen tokens are summed by themselves and then added to the row's sum: fewer roundings at the
        // magnitude of the whole)
        constexpr int kCols = 4;   // column groups at a time
#pragma unroll
        for (int b = 0; b < S::kBlocks; ++b)
#pragma unroll
          for (int c = 0; c < S::kVLoads; ++c)
#pragma unroll
            for (int e4 = 0; e4 < S::kVElems; e4 += kCols) {
              f32x4 sum[M][kCols];
#pragma unroll
              for (int t = 0; t < M; ++t)
#pragma unroll
                for (int e = 0; e < kCols; ++e) sum[t][e] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
              for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int e = 0; e < kCols; ++e) {
                  const float vf = widen<KVT>(r.v[b][j][c], e4 + e);
#pragma unroll
                  for (int t = 0; t < M; ++t) sum[t][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf, s[t][b][j], sum[t][e], 0, 0, 0);
                }
#pragma unroll
              for (int t = 0; t < M; ++t)
#pragma unroll
                for (int e = 0; e < kCols; ++e) acc[t][c * S::kVElems + e4 + e] += sum[t][e];
              // (left to itself the compiler starts every group at once and spills, and scratch traffic is counted with the
              // tile loads: 51.4 us against 45.5 on the float32 batch above)
              __builtin_amdgcn_sched_barrier(0);
            }
      }
    };

    // ---- stream: tile k is multiplied while tile k + kRing - 1 is requested and tile k + kRing is looked up
    for (int k0 = 0; k0 < my_tiles; k0 += S::kRing) {
#pragma unroll
      for (int u = 0; u < S::kRing; ++u) {
        constexpr int R = S::kRing;
        const int ahead = (u + R - 1) % R;
        fetch(buf[ahead], at[ahead]);
        scl[ahead] = scales_of(at[ahead]);
        at[u] = locate(k0 + u + R);
        if (k0 + u < my_tiles) multiply(buf[u], scl[u], k0 + u);
      }
    }

    // ---- a wave's own item: nothing to merge
    if constexpr (SOLO) {
      float l = l_run[0];
      l += lane_xor(l, 16);
      l += lane_xor(l, 32);
      if (n < rows) {
        const float inv = l > 0.f ? 1.f / l : 0.f;
        const int64_t slot = int64_t(p.slot_base[p.req_list[req_off + n / G]]) + split_local;
        const int64_t row = slot * p.num_q_heads + kv_head * G + n % G;
        float* o = p.ws_o + row * D;
#pragma unroll
        for (int c = 0; c < S::kVLoads; ++c)
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < S::kVElems; e += 4)
              *reinterpret_cast<f32x4*>(o + 16 * S::kVElems * c + (4 * kg + j) * S::kVElems + e) =
                  f32x4{acc[0][c * S::kVElems + e][j], acc[0][c * S::kVElems + e + 1][j], acc[0][c * S::kVElems + e + 2][j],
                        acc[0][c * S::kVElems + e + 3][j]} * inv;
        if (kg == 0) p.ws_lse[row] = l > 0.f ? (m_run[0] + __builtin_amdgcn_logf(l)) * kLn2 : neg_inf;
      }
      return;
    }

    // ---- merge the four waves and write one partial state per row
    // (SPREAD: the waves of every row tile hand in theirs at once)
#pragma unroll
    for (int t = 0; t < M; ++t) {
      if (row0 + 16 * t >= rows) break;
      float l = l_run[t];
      l += lane_xor(l, 16);
      l += lane_xor(l, 32);
      if (kg == 0) {
        sm_m[wave][n] = m_run[t];
        sm_l[wave][n] = l;
      }
      // register j of group c * kVElems + e: column 16 kVElems c + (4 kg + j) kVElems + e of row n
#pragma unroll
      for (int c = 0; c < S::kVLoads; ++c)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int e = 0; e < S::kVElems; e += 4)
            *reinterpret_cast<f32x4*>(&sm_o[wave][n][16 * S::kVElems * c + (4 * kg + j) * S::kVElems + e]) =
                f32x4{acc[t][c * S::kVElems + e][j], acc[t][c * S::kVElems + e + 1][j], acc[t][c * S::kVElems + e + 2][j],
                      acc[t][c * S::kVElems + e + 3][j]};
      __syncthreads();
      const int rr = threadIdx.x >> 4;
      for (int tile = t; tile < (SPREAD ? 1 << spread : t + 1); ++tile) {
        const int row = row0 + 16 * tile + rr;
        if (row < rows) {
          float mw[kWaves], mn = neg_inf;
#pragma unroll
          for (int w = 0; w < kWaves; ++w) {
            mw[w] = !SPREAD || (w & ((1 << spread) - 1)) == tile ? sm_m[w][rr] : neg_inf;
            mn = fmaxf(mn, mw[w]);
          }
          float coef[kWaves], lsum = 0.f;
#pragma unroll
          for (int w = 0; w < kWaves; ++w) {
            coef[w] = (mw[w] == neg_inf) ? 0.f : fast_exp2(mw[w] - mn);
            lsum += coef[w] * sm_l[w][rr];
          }
          const float inv = lsum > 0.f ? 1.f / lsum : 0.f;
          const int req = p.req_list[req_off + row / G];
          const int h = kv_head * G + row % G;
          const int64_t slot = int64_t(p.slot_base[req]) + split_local;
          float* o = p.ws_o + (slot * p.num_q_heads + h) * D;
#pragma unroll
          for (int c0 = 0; c0 < D; c0 += 64) {
            const int col = c0 + 4 * (threadIdx.x & 15);
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < kWaves; ++w)
              if (!SPREAD || coef[w] != 0.f) v += coef[w] * *reinterpret_cast<const f32x4*>(&sm_o[w][rr][col]);
            *reinterpret_cast<f32x4*>(o + col) = v * inv;
          }
          if ((threadIdx.x & 15) == 0)
            p.ws_lse[slot * p.num_q_heads + h] = lsum > 0.f ? (mn + __builtin_amdgcn_logf(lsum)) * kLn2 : neg_inf;
        }
      }
      __syncthreads();
    }
  };

  if constexpr (SPREAD) {
    for (int row0 = 0; row0 < rows;) {
      const int spread = rows - row0 <= 16 ? 0 : rows - row0 <= 32 ? 1 : 2;
      pass(row0, std::integral_constant<int, 1>{}, spread);
      row0 += 16 << spread;
    }
    return;
  }
  for (int row0 = 0; row0 < rows; row0 += 16 * NT) {
    const int left = rows - row0;
    if constexpr (NT == 1) {
      pass(row0, std::integral_constant<int, 1>{}, 0);
    } else {
      if (left <= 16) pass(row0, std::integral_constant<int, 1>{}, 0);
      else if (NT == 2 || left <= 32) pass(row0, std::integral_constant<int, 2>{}, 0);
      else pass(row0, std::integral_constant<int, NT>{}, 0);
    }
  }
}

}  // namespace tile

// Which workgroups of a launch take which items: those from `solo_block` on, `solo_blocks` of them, the items from `solo_item`
// to `item_end`, a wave each; the others one item each, from `item_begin` on.
struct TileGrid { int item_begin, item_end, solo_item, solo_block, solo_blocks; };

// OCC: waves per SIMD the registers are budgeted for.  SOLO: the launch has short items that a wave takes alone (a body of their
// own: as a branch inside the other one they cost its items 3 to 9 %).
template <int D, int KVT, int QT, int NT, int OCC, bool STREAM, bool SOLO, bool SPREAD>
__global__ __launch_bounds__(256, OCC) void tile_attention_kernel(AttnParams p, TileGrid grid) {
  __shared__ tile::Lds<D, KVT, QT, SPREAD ? tile::kWaves : NT> lds;
  int block = int(blockIdx.x);
  if constexpr (SOLO) {
    const int ahead = block - grid.solo_block;
    if (ahead >= 0 && ahead < grid.solo_blocks) {
      const int item = grid.solo_item + ahead * tile::kWaves + __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
      if (item < grid.item_end) tile::attend_item<D, KVT, QT, 1, STREAM, true, false>(p, item, lds);
      return;
    }
    if (ahead >= 0) block -= grid.solo_blocks;
  }
  tile::attend_item<D, KVT, QT, NT, STREAM, false, SPREAD>(p, grid.item_begin + block, lds);
}

}  // namespace psdev
