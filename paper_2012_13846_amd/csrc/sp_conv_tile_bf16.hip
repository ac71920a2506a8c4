// gather_tile_kernel for bf16 features.
#include "sp_conv_tile.h"

namespace sp {

int conv_tile_bf16(const TileArgs& a, int kc, int ncs, int tr, hipStream_t s) {
    if (a.big) {
        if (ncs == kBigNcs && kc == 64) return launch_tile<uint16_t, 64, kBigNcs, 128, true>(a, s);
        if (ncs == kBigNcs && kc == 32) return launch_tile<uint16_t, 32, kBigNcs, 128, true>(a, s);
        return fail(SP_ERR_UNSUPPORTED, "internal: no tile kernel for slices of %d x %d beyond 32 bits", kc, ncs);
    }
#define SP_TILE(KC, NCS) /* 128-row tiles for three and more groups of channels only (conv_gather_tile) */ \
    if (kc == KC && ncs == NCS)                                                                        \
    return NCS >= 3 && tr == 128 ? launch_tile<uint16_t, KC, NCS, NCS >= 3 ? 128 : 64>(a, s) : launch_tile<uint16_t, KC, NCS, 64>(a, s)
#define SP_TILES(KC)  \
    SP_TILE(KC, 1);   \
    SP_TILE(KC, 2);   \
    SP_TILE(KC, 3);   \
    SP_TILE(KC, 4);   \
    SP_TILE(KC, 8)
    SP_TILES(32);
    SP_TILES(64);
#undef SP_TILES
#undef SP_TILE
    return fail(SP_ERR_UNSUPPORTED, "internal: no bf16 tile kernel for slices of %d x %d", kc, ncs);
}

}  // namespace sp
