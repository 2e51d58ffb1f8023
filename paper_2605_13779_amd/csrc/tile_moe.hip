// Packed MoE gate / up in tiles (see tile_body.h).  Bound by bytes: 64000 pairs over 32 x 128 groups of rank 8,
// 2048 -> 768, move 795 MB in 165 us (4.8 TB/s) for both sites, 250 us in the chunks of rows.hip.
#include "tile_body.h"

namespace mlora {

// Packed MoE: two sites on one x (gate and up), or one, four waves per workgroup -- the launches have
// thousands of tiles, and what hides a tile's round trips are the other workgroups of its CU.
// Tiles are dealt to the XCDs in runs of four.
template <int RP, int TM, int NS, int CP>
__global__ __launch_bounds__(256, (RP == 16 && TM == 16 && NS == 2 ? 3 : 4))
void tile_moe_kernel(const TileArgs a, const TileArgs b)
{
    __shared__ __attribute__((aligned(16))) unsigned char lds[TileCfg<RP, 4, TM, NS>::LDS];
    const int idx = (int)blockIdx.x >> 3, tile = ((idx >> 2) * 8 + ((int)blockIdx.x & 7)) * 4 + (idx & 3);
    if (tile >= a.n_tiles) return;
    TileRows<TM> t;
    if (!tile_from_plan<TM>((const int4 *)a.tiles, a.sorted, a.top_k, tile, (int)threadIdx.x & 63, t)) return;
    tile_body<RP, 4, TM, false, NS, CP>(a, b, t, lds, 0, (a.d_out + 63) >> 6);
}

template <int RP, int TM, int NS>
static hipError_t launch_tile_moe_cp(const TileArgs &a, const TileArgs &b, hipStream_t st)
{
    const dim3 grid((unsigned)((a.n_tiles + 31) / 32 * 32)), block(256);
    // y is pair-major: every row is touched once.  The adapters are too where a (slot, expert) group is about a tile.
    if (a.one_tile) tile_moe_kernel<RP, TM, NS, kStreamY | kStreamAB><<<grid, block, 0, st>>>(a, b);
    else tile_moe_kernel<RP, TM, NS, kStreamY><<<grid, block, 0, st>>>(a, b);
    return hipGetLastError();
}

template <int RP>
static hipError_t launch_tile_moe_rp(const TileArgs *sites, int n, hipStream_t st)
{
    const TileArgs &a = sites[0], &b = sites[n - 1];
    if (a.tile_rows <= 8) return n == 2 ? launch_tile_moe_cp<RP, 8, 2>(a, b, st) : launch_tile_moe_cp<RP, 8, 1>(a, b, st);
    return n == 2 ? launch_tile_moe_cp<RP, 16, 2>(a, b, st) : launch_tile_moe_cp<RP, 16, 1>(a, b, st);
}

// One packed MoE site, or two that take the same x and have the same widths, rank and row strides.
hipError_t launch_tile_moe(const TileArgs *sites, int n, hipStream_t st)
{
    if (n < 1 || n > 2 || sites[0].tile_rows < kChunk || sites[0].tile_rows > 16) return hipErrorInvalidValue;
    if (n == 2 && (sites[0].x != sites[1].x || sites[0].ldx != sites[1].ldx || sites[0].ldy != sites[1].ldy || sites[0].d_in != sites[1].d_in ||
                   sites[0].d_out != sites[1].d_out || sites[0].r_pad != sites[1].r_pad)) return hipErrorInvalidValue;
    if (sites[0].n_tiles <= 0) return hipSuccess;
    switch (sites[0].r_pad) {
        case 2:  return launch_tile_moe_rp<2>(sites, n, st);
        case 4:  return launch_tile_moe_rp<4>(sites, n, st);
        case 8:  return launch_tile_moe_rp<8>(sites, n, st);
        case 16: return launch_tile_moe_rp<16>(sites, n, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace mlora
