// Instantiations and dispatch of the tile kernel (tile_attention.h).
#include <type_traits>

#include "tile_attention.h"

namespace psdev {

namespace {

// Row tiles that a wave carries where an item's rows are not spread over the waves (the plan says which, see build_plan): the
// pairs of formats and head size for which that is the faster form somewhere.  Four row tiles of a 128-wide head spill.
template <int D, int KVT, int QT>
constexpr int wide_tiles() { return D == 256 || KVT != QT ? 1 : KVT == PS_BF16 ? (D == 64 ? 4 : 2) : KVT == PS_F32 && D == 64 ? 2 : 1; }

template <int D, int KVT, int QT, bool STREAM, bool SOLO>
int32_t launch_as(const AttnParams& p, int max_rows, bool spread, const TileGrid& items, hipStream_t st) {
  constexpr int kWide = wide_tiles<D, KVT, QT>(), kOcc = D == 256 ? 1 : 2;
  const dim3 grid(items.solo_item - items.item_begin + items.solo_blocks), block(256);
  if (max_rows <= 16) {
    hipLaunchKernelGGL((tile_attention_kernel<D, KVT, QT, 1, kOcc, STREAM, SOLO, false>), grid, block, 0, st, p, items);
  } else if (spread) {
    hipLaunchKernelGGL((tile_attention_kernel<D, KVT, QT, 1, kOcc, STREAM, SOLO, true>), grid, block, 0, st, p, items);
  } else {
    if constexpr (kWide > 1) hipLaunchKernelGGL((tile_attention_kernel<D, KVT, QT, kWide, 1, STREAM, SOLO, false>), grid, block, 0, st, p, items);
    else return PS_ERR_UNSUPPORTED;
  }
  return PS_OK;
}

template <int D>
int32_t dispatch(const AttnParams& p, const ps_geometry& g, int max_rows, bool spread, bool stream, const TileGrid& items, hipStream_t st) {
#define PS_CASE(KVT, QT)                                                                              \
  if (g.kv_dtype == KVT && g.q_dtype == QT) {                                                         \
    if (items.solo_blocks)                                                                            \
      return stream ? launch_as<D, KVT, QT, true, true>(p, max_rows, spread, items, st)               \
                    : launch_as<D, KVT, QT, false, true>(p, max_rows, spread, items, st);             \
    return stream ? launch_as<D, KVT, QT, true, false>(p, max_rows, spread, items, st)                \
                  : launch_as<D, KVT, QT, false, false>(p, max_rows, spread, items, st);              \
  }
  PS_CASE(PS_F32, PS_F32)
  PS_CASE(PS_BF16, PS_BF16)
  PS_CASE(PS_FP8_E4M3, PS_BF16)
  PS_CASE(PS_BF16, PS_F32)
  PS_CASE(PS_F32, PS_BF16)
  PS_CASE(PS_FP8_E4M3, PS_F32)
#undef PS_CASE
  return PS_ERR_UNSUPPORTED;
}

}  // namespace

bool tile_supported(const AttnParams& p, const ps_geometry& g) {
  // whole 16-token blocks, one descriptor with 32-bit offsets each; 16-byte loads of K and of query rows
  const int64_t esz = g.kv_dtype == PS_F32 ? 4 : (g.kv_dtype == PS_BF16 ? 2 : 1);
  return (g.head_dim == 64 || g.head_dim == 128 || g.head_dim == 256) && g.block_size % 16 == 0 &&
         int64_t(g.block_size) * g.kv_stride_tok * esz < (int64_t(1) << 31) && reinterpret_cast<uintptr_t>(p.kv) % 16 == 0 &&
         reinterpret_cast<uintptr_t>(p.q) % 16 == 0;
}

int32_t launch_tile_attention(const AttnParams& p, const ps_geometry& g, int max_rows, bool spread, bool stream, int item_begin,
                              int n_items, int n_solo, int solo_block, hipStream_t st) {
  if (n_items <= 0) return PS_OK;
  const TileGrid items{item_begin, item_begin + n_items, item_begin + n_items - n_solo, solo_block, (n_solo + 3) / 4};
  switch (g.head_dim) {
    case 64: return dispatch<64>(p, g, max_rows, spread, stream, items, st);
    case 128: return dispatch<128>(p, g, max_rows, spread, stream, items, st);
    case 256: return dispatch<256>(p, g, max_rows, spread, stream, items, st);
    default: return PS_ERR_UNSUPPORTED;
  }
}

}  // namespace psdev
