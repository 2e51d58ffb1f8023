// Prefill in tiles whose parts trade partial sums (see tile_seg.h): batches of few rows.  Bound by what one CU moves, a part's share
// of the adapter and of the rows, behind the chain launch -> first loads -> trade -> expand: 512 rows of 4 prompts, rank 32,
// 7168 -> 7168, 18.9 us in 256 tiles of two rows, 12.3 in 42 of 13 rows and 6 parts (26 MB).
#include "tile_seg.h"

namespace mlora {

hipError_t launch_tile_seg_trade(const TileArgs &a, const uint32_t *inl, hipStream_t st)
{
    if (!tile_seg_args_ok(a) || !a.xch || !a.ctrl || a.parts < 2) return hipErrorInvalidValue;
    switch (a.r_pad) {
        case 8:  return launch_tile_seg_rp<8, true>(a, inl, st);
        case 16: return launch_tile_seg_rp<16, true>(a, inl, st);
        case 32: return launch_tile_seg_rp<32, true>(a, inl, st);
        case 64: return launch_tile_seg_rp<64, true>(a, inl, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace mlora
