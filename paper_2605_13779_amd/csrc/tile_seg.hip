// Prefill in tiles whose workgroups sum for themselves (see tile_seg.h).
#include "tile_seg.h"

namespace mlora {

int tile_max_rows() { return kTileSegRows; }

hipError_t launch_tile_seg(const TileArgs &a, const uint32_t *inl, hipStream_t st)
{
    if (a.n_tiles <= 0) return hipSuccess;
    if (a.xch) return launch_tile_seg_trade(a, inl, st);
    if (!tile_seg_args_ok(a)) return hipErrorInvalidValue;
    switch (a.r_pad) {
        case 1:  return launch_tile_seg_rp<1, false>(a, inl, st);
        case 2:  return launch_tile_seg_rp<2, false>(a, inl, st);
        case 4:  return launch_tile_seg_rp<4, false>(a, inl, st);
        case 8:  return launch_tile_seg_rp<8, false>(a, inl, st);
        case 16: return launch_tile_seg_rp<16, false>(a, inl, st);
        case 32: return launch_tile_seg_rp<32, false>(a, inl, st);
        case 64: return launch_tile_seg_rp<64, false>(a, inl, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace mlora
