// Instantiations and dispatch of the tile kernel (tile_attention.h).
#include <type_traits>

#include "tile_attention.h"

namespace psdev {

namespace {

// Row tiles a launch carries, by the widest item: one, or up to kWide.  float32 products over more than 32 rows are
// bound by the matrix cores, where two walks over the tokens cost what one wider walk would; four row tiles of a
// 128-wide head spill (63 registers), and a 256-wide head leaves room for one next to two tile buffers.
template <int D, int KVT, int QT>
constexpr int wide_tiles() { return D == 256 ? 1 : (tile::Shape<D, KVT, QT>::kSplit && D == 64 ? 4 : 2); }

template <int D, int KVT, int QT, bool STREAM, bool SOLO>
void launch_as(const AttnParams& p, int max_rows, const TileGrid& items, hipStream_t st) {
  constexpr int kWide = wide_tiles<D, KVT, QT>();
  const dim3 grid(items.solo_item - items.item_begin + items.solo_blocks), block(256);
  if (kWide == 1 || max_rows <= 16)
    hipLaunchKernelGGL((tile_attention_kernel<D, KVT, QT, 1, D == 256 ? 1 : 2, STREAM, SOLO>), grid, block, 0, st, p, items);
  else
    hipLaunchKernelGGL((tile_attention_kernel<D, KVT, QT, kWide, 1, STREAM, SOLO>), grid, block, 0, st, p, items);
}

template <int D>
bool dispatch(const AttnParams& p, const ps_geometry& g, int max_rows, bool stream, const TileGrid& items, hipStream_t st) {
#define PS_CASE(KVT, QT)                                                              \
  if (g.kv_dtype == KVT && g.q_dtype == QT) {                                         \
    /* an item with more rows than a pass carries walks its tokens again: they should still be in the caches then */ \
    const bool streams = stream && max_rows <= 16 * wide_tiles<D, KVT, QT>();         \
    if (items.solo_blocks) {                                                          \
      if (streams) launch_as<D, KVT, QT, true, true>(p, max_rows, items, st);         \
      else launch_as<D, KVT, QT, false, true>(p, max_rows, items, st);                \
    } else {                                                                          \
      if (streams) launch_as<D, KVT, QT, true, false>(p, max_rows, items, st);        \
      else launch_as<D, KVT, QT, false, false>(p, max_rows, items, st);               \
    }                                                                                 \
    return true;                                                                      \
  }
  PS_CASE(PS_F32, PS_F32)
  PS_CASE(PS_BF16, PS_BF16)
  PS_CASE(PS_FP8_E4M3, PS_BF16)
  PS_CASE(PS_BF16, PS_F32)
  PS_CASE(PS_F32, PS_BF16)
  PS_CASE(PS_FP8_E4M3, PS_F32)
#undef PS_CASE
  return false;
}

}  // namespace

bool tile_supported(const AttnParams& p, const ps_geometry& g) {
  // whole 16-token blocks, one descriptor with 32-bit offsets each; 16-byte loads of K and of query rows
  const int64_t esz = g.kv_dtype == PS_F32 ? 4 : (g.kv_dtype == PS_BF16 ? 2 : 1);
  return (g.head_dim == 64 || g.head_dim == 128 || g.head_dim == 256) && g.block_size % 16 == 0 &&
         int64_t(g.block_size) * g.kv_stride_tok * esz < (int64_t(1) << 31) && reinterpret_cast<uintptr_t>(p.kv) % 16 == 0 &&
         reinterpret_cast<uintptr_t>(p.q) % 16 == 0;
}

int32_t launch_tile_attention(const AttnParams& p, const ps_geometry& g, int max_rows, bool stream, int item_begin,
                              int n_items, int n_solo, int solo_block, hipStream_t st) {
  if (n_items <= 0) return PS_OK;
  const TileGrid items{item_begin, item_begin + n_items, item_begin + n_items - n_solo, solo_block, (n_solo + 3) / 4};
  bool ok = false;
  switch (g.head_dim) {
    case 64: ok = dispatch<64>(p, g, max_rows, stream, items, st); break;
    case 128: ok = dispatch<128>(p, g, max_rows, stream, items, st); break;
    case 256: ok = dispatch<256>(p, g, max_rows, stream, items, st); break;
    default: break;
  }
  return ok ? PS_OK : PS_ERR_UNSUPPORTED;
}

}  // namespace psdev
