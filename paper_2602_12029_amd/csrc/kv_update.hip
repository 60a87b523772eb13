// Writing KV into the paged pool: whole-segment ingest (a prefill worker's shared prefix cache, or a private
// segment produced elsewhere, handed over as contiguous [token][kv_head][d] tensors) and the per-step append
// of one new token per request.  bf16 / float32 pools store the source bits; e4m3 pools quantise per
// (block, kv head) tile with one float32 scale for K and one for V.
//
// Quantiser (every decision in float32 so that results are reproducible bit for bit): a = max |x| over the
// tile's valid tokens, scale = a / 448 (1 if a = 0), code = round-to-nearest-even e4m3fn of x / scale.  An
// append whose token raises the tile's scale re-encodes the tokens already stored from their stored values:
// y = (decode(code) * scale_old) / scale_new.
//
// Both kernels are plain streaming code: one wavefront per (block, kv head, K|V) tile or 4 KiB of one (ingest) or per
// (request, kv head, K|V) row (append); HBM-bound, no matrix work.
#include <algorithm>
#include <type_traits>

#include "device_common.h"
#include "launch.h"

namespace psdev {

namespace {

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

// Bulk K/V passes through these kernels once and is far larger than the caches: loads and stores are non-temporal,
// so the lines neither displace what the caches hold nor wait there for a reader that never comes.
template <typename V>
__device__ __forceinline__ V stream_load(const V* p) { return __builtin_nontemporal_load(p); }
template <typename V>
__device__ __forceinline__ void stream_store(V* p, V v) { __builtin_nontemporal_store(v, p); }

// e4m3fn code -> float32 (exact)
__device__ __forceinline__ float e4m3_to_f32(uint32_t code) {
  const uint32_t e = (code >> 3) & 0xf, m = code & 7;
  const float mag = e ? __uint_as_float(((e + 120u) << 23) | (m << 20)) : float(m) * 0x1p-9f;
  return (code & 0x80) ? -mag : mag;
}

// two float32 -> two e4m3fn codes in the low 16 bits (v_cvt_pk_fp8_f32: nearest even).  Inputs never reach the
// midpoint above 448 here (|x| <= tile maximum), so saturation behaviour is not relied upon.
__device__ __forceinline__ uint32_t f32x2_to_e4m3(float a, float b) {
  return uint32_t(__builtin_amdgcn_cvt_pk_fp8_f32(a, b, 0, false)) & 0xffffu;
}

__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) x = fmaxf(x, lane_xor(x, m));
  return x;
}

struct KvWriteParams {
  const int32_t* blk;        // concatenated block array
  const int32_t* ent_tok0;   // per entry: its first token in the ragged source of its kind
  const int32_t* ent_valid;  // per entry: tokens stored in the block
  const int32_t* ent_order;  // per entry position: the entry an ingest or stage-in takes there (shared kinds by physical block)
  const int32_t* dest;       // [R] block * B + slot of the token being appended, -1 = none
  void* kv;
  float* scales;
  int32_t num_kv_heads, head_dim, block_size;
  int64_t s_block, s_head, s_kv, s_tok;  // pool strides, elements
};

// ---- ingest, storage formats that keep the source bits (T = uint16_t for bf16, float) --------------------
// One wavefront per piece of an (entry, head, K|V) tile: 256 16-byte chunks, four a lane, all fetched before the first
// store; `ppt` pieces a tile.  HBM-bound; with a wave per tile a batch of a few hundred larger blocks left most of the chip
// idle (25 contexts of 3130 tokens in blocks of 32, two launches: 36.3 -> 34.1 us).  The four loads of a small launch stand without
// branches: a chunk past the tile's end reads the last one again, which costs less than the wait that a branch leaves behind each
// (one context of 10366 tokens in blocks of 16: 15.0 -> 13.2 us).  PACED: a large one keeps them, HBM bounds it anyway and takes
// shorter bursts better (43 contexts in blocks of 64 90.7 us, without 91.5; 134 thousand pieces 209.7 / 210.3).
template <typename T, bool PACED>
__global__ __launch_bounds__(256) void ingest_copy_kernel(KvWriteParams p, const T* __restrict__ src_k,
                                                          const T* __restrict__ src_v, int64_t src_s_tok,
                                                          int64_t src_s_head, int entry0, uint32_t num_tiles, uint32_t ppt) {
  constexpr int kVec = 16 / int(sizeof(T));
  const int lane = threadIdx.x & 63;
  const uint64_t piece = uint64_t(blockIdx.x) * 4 + uint32_t(__builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6));
  const uint32_t tile = ppt == 1 ? uint32_t(piece) : uint32_t(piece / ppt);
  if (piece >= uint64_t(num_tiles) * ppt) return;
  const int cpt = p.head_dim / kVec;   // 16-byte chunks per token
  const int which = int(tile & 1u);
  const int h = int((tile >> 1) % uint32_t(p.num_kv_heads));
  const int e = p.ent_order[entry0 + int((tile >> 1) / uint32_t(p.num_kv_heads))];
  // a block adopted from another layout has no valid tokens here: its contents are already there
  const int valid = max(0, p.ent_valid[e]), chunks = valid * cpt;
  const int c0 = int(piece - uint64_t(tile) * ppt) * 256 + lane;
  const T* src = (which ? src_v : src_k) + int64_t(p.ent_tok0[e]) * src_s_tok + int64_t(h) * src_s_head;
  T* dst = static_cast<T*>(p.kv) + int64_t(p.blk[e]) * p.s_block + int64_t(h) * p.s_head + int64_t(which) * p.s_kv;
  if (c0 - lane >= chunks) return;
  // (rows of a power of two of chunks: the lane keeps its column from chunk to chunk, which saves the divisions in front of the loads;
  // the context above 13.3 -> 12.9 us, 100 thousand pieces of float32 136.0 -> 134.5)
  const int tok0 = c0 / cpt, col0 = c0 - tok0 * cpt, tok_step = 64 / cpt;
  const bool same_column = 64 % cpt == 0;
  u32x4 v[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int c = PACED ? c0 + 64 * u : min(c0 + 64 * u, chunks - 1);
    int tok = PACED ? tok0 + u * tok_step : min(tok0 + u * tok_step, valid - 1), col = col0;
    if (!same_column) {
      tok = c / cpt;
      col = c % cpt;
    }
    if (!PACED || c < chunks) v[u] = stream_load(reinterpret_cast<const u32x4*>(src + int64_t(tok) * src_s_tok + col * kVec));
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int c = c0 + 64 * u;
    int tok = tok0 + u * tok_step, col = col0;
    if (!same_column) {
      tok = c / cpt;
      col = c % cpt;
    }
    if (c < chunks) stream_store(reinterpret_cast<u32x4*>(dst + int64_t(tok) * p.s_tok + col * kVec), v[u]);
  }
}

// ---- ingest, bf16 source -> e4m3 pool.  CH: 16-byte source chunks a lane keeps in registers; SHIFT >= 0:
// head_dim / 8 chunks per token is 2^SHIFT (index math by shifts), -1: any multiple of 8 ------------------------
template <int CH, int SHIFT>
__global__ __launch_bounds__(256) void ingest_e4m3_kernel(KvWriteParams p, const uint16_t* __restrict__ src_k,
                                                          const uint16_t* __restrict__ src_v, int64_t src_s_tok,
                                                          int64_t src_s_head, int entry0, int num_entries) {
  const int lane = threadIdx.x & 63;
  // wave-uniform tile coordinates (the launcher keeps the tile count under 2^31)
  const uint32_t tile = blockIdx.x * 4u + uint32_t(__builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6));
  if (tile >= uint32_t(num_entries) * uint32_t(p.num_kv_heads) * 2u) return;
  const int which = int(tile & 1u);
  const int h = int((tile >> 1) % uint32_t(p.num_kv_heads));
  const int e = p.ent_order[entry0 + int((tile >> 1) / uint32_t(p.num_kv_heads))];
  const int n_valid = p.ent_valid[e];
  if (n_valid <= 0) return;   // a block adopted from another layout: contents and scale are already there
  const uint16_t* src = (which ? src_v : src_k) + int64_t(p.ent_tok0[e]) * src_s_tok + int64_t(h) * src_s_head;
  const int id = p.blk[e];
  uint8_t* dst = static_cast<uint8_t*>(p.kv) + int64_t(id) * p.s_block + int64_t(h) * p.s_head + int64_t(which) * p.s_kv;
  const int cpt = p.head_dim / 8;
  const int total = n_valid * cpt;
  auto token_of = [&](int c) { return SHIFT >= 0 ? c >> SHIFT : c / cpt; };
  auto column_of = [&](int c) { return (SHIFT >= 0 ? c & ((1 << SHIFT) - 1) : c % cpt) * 8; };
  // every load goes out before anything waits: chunks past the tile re-read its last chunk and are zeroed after
  u32x4 raw[CH];
#pragma unroll
  for (int i = 0; i < CH; ++i) {
    const int c = min(lane + 64 * i, total - 1);
    raw[i] = stream_load(reinterpret_cast<const u32x4*>(src + int64_t(token_of(c)) * src_s_tok + column_of(c)));
  }
  float amax = 0.f;
#pragma unroll
  for (int i = 0; i < CH; ++i) {
    if (lane + 64 * i >= total) raw[i] = u32x4{0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      amax = fmaxf(amax, fabsf(bf16_bits_to_f32(raw[i][j] & 0xffffu)));
      amax = fmaxf(amax, fabsf(bf16_bits_to_f32(raw[i][j] >> 16)));
    }
  }
  amax = wave_max(amax);
  const float scale = amax > 0.f ? amax / 448.f : 1.f;
  if (lane == 0) p.scales[(int64_t(id) * p.num_kv_heads + h) * 2 + which] = scale;
  // x / scale without a division per element.  q0 = x * RN(1 / scale) is within 2 ulp of the exact quotient and
  // the correctly rounded quotient within 0.5 ulp, so both lie on the same side of every rounding boundary of
  // e4m3 -- and get the same code -- unless q0 is within a few ulp of one.  Boundaries (midpoints of neighbouring
  // e4m3 values) have the float32 pattern "3 mantissa bits, then 1000...0" in the normal range; a chunk in which
  // any lane is that close to one, or may fall into the subnormal range of e4m3 (an absolute grid), is redone with
  // the real division.  The stored codes are therefore exactly those of RN(x / scale) everywhere.
  const float rinv = 1.f / scale;
  const float subnormal_below = scale * 0x1.000002p-6f;   // |x| under this: the quotient may be under 2^-6
#pragma unroll
  for (int i = 0; i < CH; ++i) {
    const int c = lane + 64 * i;
    float x[8], q[8];
    bool risky = false;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      x[2 * j] = bf16_bits_to_f32(raw[i][j] & 0xffffu);
      x[2 * j + 1] = bf16_bits_to_f32(raw[i][j] >> 16);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      q[j] = x[j] * rinv;
      // low 20 mantissa bits within [0x7fffc, 0x80004]: shifted to the top of the word, offset so the window starts at 0
      risky |= (__float_as_uint(q[j]) << 12) + 0x80004000u <= 0x8000u;
      risky |= fabsf(x[j]) < subnormal_below;               // subnormal range of e4m3 (also catches exact zeros)
    }
    risky = risky && c < total;                               // lanes past the tile hold zeros: no say
    if (__builtin_amdgcn_ballot_w64(risky) != 0) {
      // second look: a quotient near a boundary that is exact (zero residual x - q0 * scale; ties of short
      // mantissas are common with bf16 inputs) is the correctly rounded quotient already
      bool divide = false;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const bool near = (__float_as_uint(q[j]) << 12) + 0x80004000u <= 0x8000u;
        divide |= near && __builtin_fmaf(-q[j], scale, x[j]) != 0.f;
        divide |= fabsf(x[j]) < subnormal_below;
      }
      divide = divide && c < total;
      if (__builtin_amdgcn_ballot_w64(divide) != 0) {
#pragma unroll
        for (int j = 0; j < 8; ++j) q[j] = x[j] / scale;
      }
    }
    if (c < total) {
      u32x2 out;
      out[0] = uint32_t(__builtin_amdgcn_cvt_pk_fp8_f32(q[2], q[3], __builtin_amdgcn_cvt_pk_fp8_f32(q[0], q[1], 0, false), true));
      out[1] = uint32_t(__builtin_amdgcn_cvt_pk_fp8_f32(q[6], q[7], __builtin_amdgcn_cvt_pk_fp8_f32(q[4], q[5], 0, false), true));
      stream_store(reinterpret_cast<u32x2*>(dst + int64_t(token_of(c)) * p.s_tok + column_of(c)), out);
    }
  }
}

// ---- append: one wavefront per (request, kv head, K|V) ----------------------------------------------------
template <typename T>
__device__ __forceinline__ void append_copy_row(const KvWriteParams& p, const T* __restrict__ new_k, const T* __restrict__ new_v, int dest,
                                                int r, int h, int which) {
  const int lane = threadIdx.x & 63;
  const int id = dest / p.block_size, slot = dest % p.block_size;
  const T* src = (which ? new_v : new_k) + (int64_t(r) * p.num_kv_heads + h) * p.head_dim;
  T* dst = static_cast<T*>(p.kv) + int64_t(id) * p.s_block + int64_t(h) * p.s_head + int64_t(which) * p.s_kv +
           int64_t(slot) * p.s_tok;
  for (int c = lane; c < p.head_dim; c += 64) dst[c] = src[c];
}

template <typename T>
__global__ __launch_bounds__(256) void append_copy_kernel(KvWriteParams p, const T* __restrict__ new_k,
                                                          const T* __restrict__ new_v, int num_requests) {
  const int64_t row = int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (row >= int64_t(num_requests) * p.num_kv_heads * 2) return;
  const int r = int((row >> 1) / p.num_kv_heads);
  const int dest = p.dest[r];
  if (dest >= 0) append_copy_row(p, new_k, new_v, dest, r, int((row >> 1) % p.num_kv_heads), int(row & 1));
}

// e4m3 with rows of 2^row_shift eight-element pieces: one wavefront per (request, kv head, K|V), eight elements a lane.  The
// stored tokens of a tile whose scale has grown are rewritten 64 >> row_shift at a time, and four of those rounds are fetched
// together: a block of sixteen 128-wide tokens in one round trip (a byte at a time the launch was bound by the chain of those
// rewrites: 64 requests, eight heads, tokens of changing magnitude 8.5 -> 5.2 us).
__device__ __forceinline__ void append_e4m3x8_row(const KvWriteParams& p, const u32x4* __restrict__ new_k, const u32x4* __restrict__ new_v,
                                                  int row_shift, int dest, int r, int h, int which) {
  const int lane = threadIdx.x & 63;
  const int id = dest / p.block_size, slot = dest % p.block_size;
  uint8_t* tile = static_cast<uint8_t*>(p.kv) + int64_t(id) * p.s_block + int64_t(h) * p.s_head + int64_t(which) * p.s_kv;
  float* scale_ptr = p.scales + (int64_t(id) * p.num_kv_heads + h) * 2 + which;
  const int c = lane & ((1 << row_shift) - 1), tok0 = lane >> row_shift, toks = 64 >> row_shift;
  // (every token group of the wave holds the whole row)
  const u32x4 raw = (which ? new_v : new_k)[((int64_t(r) * p.num_kv_heads + h) << row_shift) + c];
  const float old = *scale_ptr;   // (of a fresh block: anything, and not used)
  float x[8], amax = 0.f;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    x[2 * j] = bf16_bits_to_f32(raw[j] & 0xffffu);
    x[2 * j + 1] = bf16_bits_to_f32(raw[j] >> 16);
    amax = fmaxf(amax, fmaxf(fabsf(x[2 * j]), fabsf(x[2 * j + 1])));
  }
  amax = wave_max(amax);
  const float cand = amax / 448.f;
  float scale;
  auto encode = [](const float (&y)[8]) {
    u32x2 out;
    out[0] = uint32_t(__builtin_amdgcn_cvt_pk_fp8_f32(y[2], y[3], __builtin_amdgcn_cvt_pk_fp8_f32(y[0], y[1], 0, false), true));
    out[1] = uint32_t(__builtin_amdgcn_cvt_pk_fp8_f32(y[6], y[7], __builtin_amdgcn_cvt_pk_fp8_f32(y[4], y[5], 0, false), true));
    return out;
  };
  if (slot == 0) {
    scale = amax > 0.f ? cand : 1.f;
  } else {
    scale = fmaxf(old, cand);
    if (scale != old) {   // the tile's scale grew: re-encode what is stored, from the stored values
      for (int t0 = tok0; t0 < slot; t0 += 4 * toks) {
        u32x2 code[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (t0 + u * toks < slot) code[u] = *reinterpret_cast<const u32x2*>(tile + int64_t(t0 + u * toks) * p.s_tok + 8 * c);
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (t0 + u * toks < slot) {
            float y[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) y[j] = (e4m3_to_f32((code[u][j >> 2] >> (8 * (j & 3))) & 0xffu) * old) / scale;
            *reinterpret_cast<u32x2*>(tile + int64_t(t0 + u * toks) * p.s_tok + 8 * c) = encode(y);
          }
      }
    }
  }
  if (lane == 0) *scale_ptr = scale;
  if (tok0 == 0) {
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = x[j] / scale;
    *reinterpret_cast<u32x2*>(tile + int64_t(slot) * p.s_tok + 8 * c) = encode(x);
  }
}

__global__ __launch_bounds__(256) void append_e4m3x8_kernel(KvWriteParams p, const u32x4* __restrict__ new_k,
                                                            const u32x4* __restrict__ new_v, int row_shift) {
  const int r = blockIdx.x;
  const int row = int(blockIdx.y) * 4 + __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);   // of the token: (head, K|V)
  if (row >= 2 * p.num_kv_heads) return;
  const int dest = p.dest[r];
  if (dest >= 0) append_e4m3x8_row(p, new_k, new_v, row_shift, dest, r, row >> 1, row & 1);
}

// The tables on their way to the device and the tokens of the same decode step, which do not wait for them: a wave per row of a token
// reads where it goes from the pinned buffer, across PCIe like the tables themselves.
// Bound: that link and its latency; two launches in a row cost a turn's step a launch on the host and the gap between them (16
// contexts under four models, a turn of eight steps 520 -> 504 us; 25 of one, five steps 324 -> 294).  A row is a chain of dependent
// reads: with all rows of a request in one workgroup its waves walk them one after the other (bf16, 64 requests, a call with two
// launches / so / with a wave per row: 8 KV heads 11.5 / 9.3 / 9.1 us, 32 heads 16.5 / 17.9 / 14.6; 32 requests, 64 heads 16.0 / 21.9 /
// 14.3; float32, 64 requests, 64 heads 14.2 / 19.7 / 12.3; e4m3, where a row's tile may be rewritten, a turn of twelve steps 5 % longer so
// than with two launches).
template <int KVT>
__global__ __launch_bounds__(256) void upload_append_kernel(const u32x4* __restrict__ tables, u32x4* __restrict__ dev_tables, uint32_t pieces,
                                                            uint32_t upload_wgs, KvWriteParams p, const void* __restrict__ new_k,
                                                            const void* __restrict__ new_v, int row_shift) {
  if (blockIdx.x < upload_wgs) {
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    if (i < pieces) dev_tables[i] = tables[i];
    return;
  }
  const int wgs = (2 * p.num_kv_heads + 3) / 4;   // of a token
  const int wg = int(blockIdx.x - upload_wgs), r = wg / wgs, dest = p.dest[r];
  const int row = (wg - r * wgs) * 4 + __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);   // of the token: (head, K|V)
  if (dest < 0 || row >= 2 * p.num_kv_heads) return;
  typedef std::conditional_t<KVT == PS_F32, float, std::conditional_t<KVT == PS_BF16, uint16_t, u32x4>> word;
  const word *k = static_cast<const word*>(new_k), *v = static_cast<const word*>(new_v);
  if constexpr (KVT == PS_FP8_E4M3) append_e4m3x8_row(p, k, v, row_shift, dest, r, row >> 1, row & 1);
  else append_copy_row(p, k, v, dest, r, row >> 1, row & 1);
}

// Any head size and alignment.
__global__ __launch_bounds__(256) void append_e4m3_kernel(KvWriteParams p, const uint16_t* __restrict__ new_k,
                                                          const uint16_t* __restrict__ new_v, int num_requests) {
  const int lane = threadIdx.x & 63;
  const int64_t row = int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (row >= int64_t(num_requests) * p.num_kv_heads * 2) return;
  const int which = int(row & 1);
  const int h = int((row >> 1) % p.num_kv_heads);
  const int r = int((row >> 1) / p.num_kv_heads);
  const int dest = p.dest[r];
  if (dest < 0) return;
  const int id = dest / p.block_size, slot = dest % p.block_size;
  const uint16_t* src = (which ? new_v : new_k) + (int64_t(r) * p.num_kv_heads + h) * p.head_dim;
  uint8_t* tile = static_cast<uint8_t*>(p.kv) + int64_t(id) * p.s_block + int64_t(h) * p.s_head + int64_t(which) * p.s_kv;
  float* scale_ptr = p.scales + (int64_t(id) * p.num_kv_heads + h) * 2 + which;
  float amax = 0.f;
  for (int c = lane; c < p.head_dim; c += 64) amax = fmaxf(amax, fabsf(bf16_bits_to_f32(src[c])));
  amax = wave_max(amax);
  const float cand = amax / 448.f;
  float scale;
  if (slot == 0) {
    scale = amax > 0.f ? cand : 1.f;
  } else {
    const float old = *scale_ptr;
    scale = fmaxf(old, cand);
    if (scale != old) {   // the tile's scale grew: re-encode what is stored, from the stored values
      for (int c = lane; c < slot * p.head_dim; c += 64) {
        uint8_t* at = tile + int64_t(c / p.head_dim) * p.s_tok + c % p.head_dim;
        *at = uint8_t(f32x2_to_e4m3((e4m3_to_f32(*at) * old) / scale, 0.f) & 0xffu);
      }
    }
  }
  if (lane == 0) *scale_ptr = scale;
  uint8_t* dst = tile + int64_t(slot) * p.s_tok;
  for (int c = lane; c < p.head_dim; c += 64) dst[c] = uint8_t(f32x2_to_e4m3(bf16_bits_to_f32(src[c]) / scale, 0.f) & 0xffu);
}

// ---- staging of whole blocks (cold KV parked in host memory and reloaded, Appendix B.2) -------------------
// One wavefront per TILES consecutive pieces of (entry, KV head, K|V) tiles of B x d elements -- 256 16-byte chunks of a
// tile, `ppt` pieces a tile --; the image is dense,
// [entry][head][K|V][slot][d] in table order, followed by the e4m3 scales [entry][head][K|V].  TO_IMAGE: pool ->
// image, else image -> pool.  Bits are copied, 16 bytes per lane, four loads per piece before the first store.
// (A wave used to walk whole tiles: ten requests' blocks of 64 tokens, 54 MB there and back, in 103 workgroups 85.8 us, in
// 1648 23.2; 16-token blocks of bf16, 2.55 GB, where a tile is a piece, 451 -> 439 from the shorter index arithmetic.)
// LOADS: chunks a lane has of a piece (two for the 2 KiB tiles of e4m3 in blocks of 16).
template <bool TO_IMAGE, int TILES, int LOADS>
__global__ __launch_bounds__(256) void stage_copy_kernel(KvWriteParams p, uint8_t* __restrict__ image,
                                                         float* __restrict__ image_scales, int entry0, uint32_t num_tiles,
                                                         uint32_t ppt, int elem_bytes) {
  const int lane = threadIdx.x & 63;
  const uint64_t num_pieces = uint64_t(num_tiles) * ppt;
  // (tile = (entry, head, which), piece), TILES in a row
  const uint64_t piece0 = (uint64_t(blockIdx.x) * 4 + uint32_t(__builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6))) * TILES;
  if (piece0 >= num_pieces) return;
  const int row_bytes = p.head_dim * elem_bytes;
  const int row_chunks = row_bytes >> 4;
  const int chunks = p.block_size * row_chunks;
  const int64_t tok_bytes = p.s_tok * elem_bytes;
  uint8_t* pool_tile[TILES];
  uint8_t* image_tile[TILES];
  int first[TILES], last[TILES];   // chunks of the tile
#pragma unroll
  for (int i = 0; i < TILES; ++i) {
    const uint64_t piece = min(piece0 + i, num_pieces - 1);
    const uint32_t tile = ppt == 1 ? uint32_t(piece) : uint32_t(piece / ppt);
    const int part = int(piece - uint64_t(tile) * ppt);
    const bool live = piece0 + i < num_pieces;
    first[i] = 256 * part;
    last[i] = live ? min(chunks, first[i] + 256) : 0;
    const int which = int(tile & 1);
    const int h = int((tile >> 1) % uint32_t(p.num_kv_heads));
    // Into the pool the shared blocks are walked in the order of their addresses there, so that the scattered side of
    // the copy is the read of the image (scattered writes cost more); out of it in table order, for the same reason.
    const int pos = entry0 + int((tile >> 1) / uint32_t(p.num_kv_heads));
    const int e = TO_IMAGE ? pos : p.ent_order[pos];
    const int64_t image_tile_index = (int64_t(e) * p.num_kv_heads + h) * 2 + which;
    const int id = p.blk[e];
    pool_tile[i] = static_cast<uint8_t*>(p.kv) +
                   (int64_t(id) * p.s_block + int64_t(h) * p.s_head + int64_t(which) * p.s_kv) * elem_bytes;
    image_tile[i] = image + image_tile_index * int64_t(p.block_size) * row_bytes;
    if (image_scales && lane == 0 && live && part == 0) {
      float* pool_scale = p.scales + (int64_t(id) * p.num_kv_heads + h) * 2 + which;
      if (TO_IMAGE) image_scales[image_tile_index] = *pool_scale;
      else *pool_scale = image_scales[image_tile_index];
    }
  }
  // every load goes out before the first store
  {
    u32x4 v[TILES][LOADS];
#pragma unroll
    for (int i = 0; i < TILES; ++i)
#pragma unroll
      for (int u = 0; u < LOADS; ++u) {
        // (a piece a wave: no branch around a load, as in the ingest; with four the waits between them pace a launch that HBM
        // bounds anyway: 16-token blocks of bf16, 2.55 GB, 437 us, all sixteen loads at once 450)
        const int at = first[i] + 64 * u + lane, c = TILES == 1 ? min(at, chunks - 1) : at;
        if (TILES == 1 || c < last[i]) {
          const int slot = c / row_chunks, col = c % row_chunks;
          const uint8_t* src = TO_IMAGE ? pool_tile[i] + slot * tok_bytes + 16 * col : image_tile[i] + 16 * int64_t(c);
          v[i][u] = stream_load(reinterpret_cast<const u32x4*>(src));
        }
      }
#pragma unroll
    for (int i = 0; i < TILES; ++i)
#pragma unroll
      for (int u = 0; u < LOADS; ++u) {
        const int c = first[i] + 64 * u + lane;
        if (c < last[i]) {
          const int slot = c / row_chunks, col = c % row_chunks;
          uint8_t* dst = TO_IMAGE ? image_tile[i] + 16 * int64_t(c) : pool_tile[i] + slot * tok_bytes + 16 * col;
          stream_store(reinterpret_cast<u32x4*>(dst), v[i][u]);
        }
      }
  }
}

KvWriteParams make_write_params(const ps_layout* lay, const void* dev_tables, void* kv, float* scales) {
  const int32_t* t = static_cast<const int32_t*>(dev_tables);
  const ps_geometry& g = lay->geo;
  KvWriteParams p{};
  p.blk = t + lay->off_blk;
  p.ent_tok0 = t + lay->off_ent_tok0;
  p.ent_valid = t + lay->off_ent_valid;
  p.ent_order = t + lay->off_ent_order;
  p.dest = t + lay->off_dest;
  p.kv = kv;
  p.scales = scales;
  p.num_kv_heads = g.num_kv_heads;
  p.head_dim = g.head_dim;
  p.block_size = g.block_size;
  p.s_block = g.kv_stride_block;
  p.s_head = g.kv_stride_head;
  p.s_kv = g.kv_stride_kv;
  p.s_tok = g.kv_stride_tok;
  return p;
}

}  // namespace

int32_t launch_kv_ingest(const ps_layout* lay, const void* dev_tables, int which, const void* src_k, const void* src_v,
                         int64_t src_s_tok, int64_t src_s_head, void* kv, float* scales, hipStream_t st) {
  const ps_geometry& g = lay->geo;
  const int n_prefix = int(lay->prefix_blk.size());
  const int n_suffix = int(lay->suffix_blk.size());
  // entries follow the concatenated block array: prefixes, suffixes, roots
  const int entry0 = which == 0 ? 0 : (which == 1 ? n_prefix : n_prefix + n_suffix);
  const int num_entries = which == 0 ? n_prefix : (which == 1 ? n_suffix : int(lay->root_blk.size()));
  if (num_entries == 0) return PS_OK;
  const int64_t tiles = int64_t(num_entries) * g.num_kv_heads * 2;
  const int64_t grid64 = (tiles + 3) / 4;
  if (tiles > INT32_MAX) return PS_ERR_INVALID_ARG;
  const dim3 grid{unsigned(grid64)}, block{256};
  const KvWriteParams p = make_write_params(lay, dev_tables, kv, scales);
  if (g.kv_dtype != PS_FP8_E4M3) {   // formats that keep the source bits: pieces of 4 KiB
    const int vec = g.kv_dtype == PS_F32 ? 4 : 8;
    if (g.head_dim % vec) return PS_ERR_UNSUPPORTED;
    const int64_t ppt = (int64_t(g.block_size) * (g.head_dim / vec) + 255) / 256;
    if (ppt > INT32_MAX / 256) return PS_ERR_INVALID_ARG;
    const int64_t per_entry = int64_t(g.num_kv_heads) * 2, step = entries_per_launch(num_entries, per_entry * ppt, 4);
    const bool paced = tiles * ppt > 8 * 4096;
    for (int64_t first = 0; first < num_entries; first += step) {
      const int64_t n = std::min<int64_t>(step, num_entries - first) * per_entry;
      const dim3 copy_grid{unsigned((n * ppt + 3) / 4)};
#define PS_COPY(T, PACED)                                                                                              \
  hipLaunchKernelGGL((ingest_copy_kernel<T, PACED>), copy_grid, block, 0, st, p, static_cast<const T*>(src_k),         \
                     static_cast<const T*>(src_v), src_s_tok, src_s_head, entry0 + int(first), uint32_t(n), uint32_t(ppt))
      if (g.kv_dtype == PS_F32) {
        if (paced) PS_COPY(float, true); else PS_COPY(float, false);
      } else {
        if (paced) PS_COPY(uint16_t, true); else PS_COPY(uint16_t, false);
      }
#undef PS_COPY
    }
  } else {
    if (g.head_dim % 8) return PS_ERR_UNSUPPORTED;
    const int64_t chunks = (int64_t(g.block_size) * (g.head_dim / 8) + 63) / 64;   // per lane, whole tile in registers
#define PS_INGEST(CH, SHIFT)                                                                                     \
  hipLaunchKernelGGL((ingest_e4m3_kernel<CH, SHIFT>), grid, block, 0, st, p, static_cast<const uint16_t*>(src_k), \
                     static_cast<const uint16_t*>(src_v), src_s_tok, src_s_head, entry0, num_entries)
    if (g.head_dim == 128) {   // 16 chunks per token
      if (chunks <= 4) PS_INGEST(4, 4);
      else if (chunks <= 8) PS_INGEST(8, 4);
      else if (chunks <= 16) PS_INGEST(16, 4);
      else if (chunks <= 32) PS_INGEST(32, 4);
      else return PS_ERR_UNSUPPORTED;
    } else {
      if (chunks <= 4) PS_INGEST(4, -1);
      else if (chunks <= 8) PS_INGEST(8, -1);
      else if (chunks <= 16) PS_INGEST(16, -1);
      else if (chunks <= 32) PS_INGEST(32, -1);
      else return PS_ERR_UNSUPPORTED;
    }
#undef PS_INGEST
  }
  return PS_OK;
}

namespace {

// e4m3: eight elements a lane where a row is a power of two of such pieces and every address a multiple of one (pool
// strides are multiples of 16 bytes).  The copying formats gain nothing from wider stores: their launch is its dependent reads.
bool whole_pieces(const ps_layout* lay, const void* new_k, const void* new_v, const void* kv) {
  const ps_geometry& g = lay->geo;
  const int pieces = g.head_dim / 8;
  return g.kv_dtype == PS_FP8_E4M3 && g.head_dim % 8 == 0 && pieces <= 64 && (pieces & (pieces - 1)) == 0 &&
         (2 * g.num_kv_heads + 3) / 4 <= 65535 && lay->num_requests <= kMaxWorkgroups &&
         (reinterpret_cast<uintptr_t>(new_k) | reinterpret_cast<uintptr_t>(new_v) | reinterpret_cast<uintptr_t>(kv)) % 16 == 0;
}

}  // namespace

bool launch_upload_append(const ps_layout* lay, const void* host_tables, void* dev_tables, size_t bytes, const void* new_k,
                          const void* new_v, void* kv, float* scales, hipStream_t st) {
  const ps_geometry& g = lay->geo;
  const uint32_t pieces = uint32_t(bytes / 16), upload_wgs = (pieces + 255) / 256;
  const int64_t append_wgs = int64_t(lay->num_requests) * ((2 * g.num_kv_heads + 3) / 4);
  if (append_wgs == 0 || upload_wgs + append_wgs > kMaxWorkgroups) return false;
  if (g.kv_dtype == PS_FP8_E4M3 && !whole_pieces(lay, new_k, new_v, kv)) return false;
  KvWriteParams p = make_write_params(lay, dev_tables, kv, scales);
  p.dest = static_cast<const int32_t*>(host_tables) + lay->off_dest;
  const dim3 grid{upload_wgs + uint32_t(append_wgs)}, block{256};
  const auto *from = static_cast<const u32x4*>(host_tables);
  auto* to = static_cast<u32x4*>(dev_tables);
  const int row_shift = g.kv_dtype == PS_FP8_E4M3 ? __builtin_ctz(unsigned(g.head_dim / 8)) : 0;
#define PS_LAUNCH(KVT) hipLaunchKernelGGL((upload_append_kernel<KVT>), grid, block, 0, st, from, to, pieces, upload_wgs, p, new_k, new_v, row_shift)
  if (g.kv_dtype == PS_F32) PS_LAUNCH(PS_F32);
  else if (g.kv_dtype == PS_BF16) PS_LAUNCH(PS_BF16);
  else PS_LAUNCH(PS_FP8_E4M3);
#undef PS_LAUNCH
  return true;
}

int32_t launch_kv_append(const ps_layout* lay, const void* dev_tables, const void* new_k, const void* new_v, void* kv,
                         float* scales, hipStream_t st) {
  const ps_geometry& g = lay->geo;
  if (lay->num_requests == 0) return PS_OK;
  const int64_t rows = int64_t(lay->num_requests) * g.num_kv_heads * 2;
  const dim3 grid{unsigned((rows + 3) / 4)}, block{256};
  const KvWriteParams p = make_write_params(lay, dev_tables, kv, scales);
  if (whole_pieces(lay, new_k, new_v, kv))
    hipLaunchKernelGGL(append_e4m3x8_kernel, dim3(unsigned(lay->num_requests), unsigned((2 * g.num_kv_heads + 3) / 4)), block, 0, st, p,
                       static_cast<const u32x4*>(new_k), static_cast<const u32x4*>(new_v), __builtin_ctz(unsigned(g.head_dim / 8)));
  else if (g.kv_dtype == PS_F32)
    hipLaunchKernelGGL(append_copy_kernel<float>, grid, block, 0, st, p, static_cast<const float*>(new_k),
                       static_cast<const float*>(new_v), lay->num_requests);
  else if (g.kv_dtype == PS_BF16)
    hipLaunchKernelGGL(append_copy_kernel<uint16_t>, grid, block, 0, st, p, static_cast<const uint16_t*>(new_k),
                       static_cast<const uint16_t*>(new_v), lay->num_requests);
  else
    hipLaunchKernelGGL(append_e4m3_kernel, grid, block, 0, st, p, static_cast<const uint16_t*>(new_k),
                       static_cast<const uint16_t*>(new_v), lay->num_requests);
  return PS_OK;
}

int32_t launch_kv_stage(const ps_layout* lay, const void* dev_tables, bool to_image, void* kv, float* scales,
                        void* image, int64_t scales_offset_bytes, hipStream_t st) {
  const ps_geometry& g = lay->geo;
  const int64_t entries = int64_t(lay->prefix_blk.size() + lay->suffix_blk.size() + lay->root_blk.size());
  if (entries == 0) return PS_OK;
  const int esz = g.kv_dtype == PS_F32 ? 4 : (g.kv_dtype == PS_BF16 ? 2 : 1);
  if ((g.head_dim * esz) % 16) return PS_ERR_UNSUPPORTED;
  const int64_t tiles = entries * g.num_kv_heads * 2;
  if (tiles > INT32_MAX) return PS_ERR_INVALID_ARG;
  const KvWriteParams p = make_write_params(lay, dev_tables, kv, scales);
  uint8_t* img = static_cast<uint8_t*>(image);
  float* img_scales = g.kv_dtype == PS_FP8_E4M3 ? reinterpret_cast<float*>(img + scales_offset_bytes) : nullptr;
  // Tiles per wave: four consecutive tiles are K and V of two neighbouring heads, 16 KiB in a row on the pool side
  // for bf16 -- measured on scattered blocks, stage_in (dense reads, scattered writes) gains 9 % from the longer
  // runs (5.16 -> 5.65 TB/s), stage_out is unchanged; with the 2 KiB tiles of e4m3 more tiles per wave only lose.
  // A small batch keeps to one piece a wave, so that it fills the chip.
  const int64_t tile_chunks = int64_t(g.block_size) * g.head_dim * esz / 16, ppt = (tile_chunks + 255) / 256;
  if (ppt > INT32_MAX / 256) return PS_ERR_INVALID_ARG;
  const int per_wave = esz >= 2 && tiles * ppt > 4 * 4096 ? 4 : 1;
  const int64_t per_entry = int64_t(g.num_kv_heads) * 2, step = entries_per_launch(entries, per_entry * ppt, 4 * per_wave);
#define PS_STAGE(TO, N, LOADS)                                                                                               \
  hipLaunchKernelGGL((stage_copy_kernel<TO, N, LOADS>), dim3{unsigned((n * ppt + 4 * N - 1) / (4 * N))}, dim3{256}, 0, st, p, img, \
                     img_scales, int(first), uint32_t(n), uint32_t(ppt), esz)
  for (int64_t first = 0; first < entries; first += step) {
    const int64_t n = std::min<int64_t>(step, entries - first) * per_entry;
    if (to_image) {
      if (per_wave == 4) PS_STAGE(true, 4, 4); else if (tile_chunks > 128) PS_STAGE(true, 1, 4); else PS_STAGE(true, 1, 2);
    } else {
      if (per_wave == 4) PS_STAGE(false, 4, 4); else if (tile_chunks > 128) PS_STAGE(false, 1, 4); else PS_STAGE(false, 1, 2);
    }
  }
#undef PS_STAGE
  return PS_OK;
}

}  // namespace psdev
