// Prefill in tiles (see tile_body.h): the batch's segments, cut into tiles of up to 48 rows.
#pragma once
#include "tile_body.h"

namespace mlora {

// The tile's segment: segs holds, per segment, its first tile, first row, rows and slot, in tile order.  The wave
// looks for the last segment that starts at or before the tile, 64 of them at equal distances at a time: one
// round trip for up to 64 segments, two for 4096 (walking the table takes one for every 64 of them).
template <int TM>
__device__ __forceinline__ bool tile_from_segments(const TileArgs &a, const uint32_t *segs, int tile, int lane, TileRows<TM> &t)
{
    int first = 0, row0 = 0, rows = 0, slot = -1;
    for (int lo = 0, len = a.n_segs;;) {
        const int step = (len + 63) >> 6, at = lane * step;
        int4 v = make_int4(0x7fffffff, 0, 0, 0);
        if (at < len) v = ((const int4 *)segs)[lo + at];
        const uint64_t hit = __ballot(v.x <= tile);          // (lane 0 always: segment lo starts at or before the tile)
        const int l = hit ? 63 - __builtin_clzll(hit) : 0;
        if (step <= 1) {
            first = __shfl(v.x, l, 64); row0 = __shfl(v.y, l, 64); rows = __shfl(v.z, l, 64); slot = __shfl(v.w, l, 64);
            break;
        }
        lo += l * step;
        len = min(step, len - l * step);
    }
    first = __builtin_amdgcn_readfirstlane(first); row0 = __builtin_amdgcn_readfirstlane(row0);
    rows = __builtin_amdgcn_readfirstlane(rows);
    t.key = __builtin_amdgcn_readfirstlane(slot);
    const int r0 = (tile - first) * a.tile_rows;
    t.cnt = min(a.tile_rows, rows - r0);
    if (t.cnt <= 0) return false;
#pragma unroll
    for (int g = 0; g < TM / 8; ++g) {
        t.xrow[g] = row0 + r0 + min(8 * g + ((lane >> 1) & 7), t.cnt - 1);
        t.yrow[g] = row0 + r0 + min(8 * g + (lane >> 3), t.cnt - 1);
    }
    return true;
}

struct TileSegInline { uint32_t w[kTileInline]; };

// TRADE: a tile's parts also divide d_in and trade partial sums; they run at the same time, one workgroup per CU.
template <int RP, int NW, int TM, int CP = 0, bool TRADE = false>
__global__ __launch_bounds__(NW * 64, 2)
void tile_seg_kernel(const TileArgs a, const TileSegInline inl)
{
    __shared__ __attribute__((aligned(16))) unsigned char lds[TileCfg<RP, NW, TM>::LDS];
    // an XCD gets a contiguous range of tiles (workgroups are dealt round-robin): neighbours share an adapter, in its L2
    const int n8 = (int)gridDim.x >> 3, item = ((int)blockIdx.x & 7) * n8 + ((int)blockIdx.x >> 3);
    const int tile = a.parts > 1 ? item / a.parts : item, part = item - tile * a.parts, blk0 = part * a.part_blocks;
    if constexpr (!TRADE) {
        if (tile >= a.n_tiles) return;
        TileRows<TM> t;
        if (!tile_from_segments<TM>(a, a.segs ? (const uint32_t *)a.segs : inl.w, tile, (int)threadIdx.x & 63, t)) return;
        tile_body<RP, NW, TM, false, 1, CP>(a, a, t, lds, blk0, min(a.part_blocks, ((a.d_out + 63) >> 6) - blk0));
    } else {
        // (see tile_multi_body: the last workgroup advances the launch tag when those with a tile have signed in)
        const bool last = item == (int)gridDim.x - 1;
        if (tile >= a.n_tiles && !last) return;
        TileTrade trade{true, item, a.parts, 0u};
        if (threadIdx.x == 0) trade.tag = tag_read(a.ctrl);
        if (tile < a.n_tiles) {
            TileRows<TM> t;
            if (tile_from_segments<TM>(a, a.segs ? (const uint32_t *)a.segs : inl.w, tile, (int)threadIdx.x & 63, t))
                tile_body<RP, NW, TM, true, 1, CP>(a, a, t, lds, blk0, min(a.part_blocks, ((a.d_out + 63) >> 6) - blk0), tile, part, trade);
            else if (threadIdx.x == 0) tag_sign_in(a.ctrl, item, trade.tag);
        }
        if (last && threadIdx.x < 64) {
            const uint32_t tag = __builtin_amdgcn_readfirstlane(trade.tag);
            if (tag != kTagPoison) tag_advance(a.ctrl, a.n_tiles * a.parts, tag, (int)threadIdx.x);
        }
    }
}

template <int RP, int TM, bool TRADE>
static hipError_t launch_tile_seg_tm(const TileArgs &a, const TileSegInline &table, hipStream_t st)
{
    const dim3 grid((unsigned)(((int64_t)a.n_tiles * a.parts + 7) / 8 * 8)), block(512);
    constexpr bool kHas = RP >= 8 && TM > 8 && !TRADE;             // (batches with as much y as that have tall tiles, and whole ones)
    if (kHas && a.stream) tile_seg_kernel<RP, 8, TM, kHas ? kStreamY : 0, TRADE><<<grid, block, 0, st>>>(a, table);
    else tile_seg_kernel<RP, 8, TM, 0, TRADE><<<grid, block, 0, st>>>(a, table);
    return hipGetLastError();
}

template <int RP, bool TRADE>
static hipError_t launch_tile_seg_rp(const TileArgs &a, const uint32_t *inl, hipStream_t st)
{
    TileSegInline table;
    if (!a.segs) for (int i = 0; i < 4 * a.n_segs; ++i) table.w[i] = inl[i];
    switch ((a.tile_rows + 7) / 8) {
        case 1: return launch_tile_seg_tm<RP, 8, TRADE>(a, table, st);
        case 2: return launch_tile_seg_tm<RP, 16, TRADE>(a, table, st);
        case 3: return launch_tile_seg_tm<RP, 24, TRADE>(a, table, st);
        case 4: return launch_tile_seg_tm<RP, 32, TRADE>(a, table, st);
        case 5: return launch_tile_seg_tm<RP, 40, TRADE>(a, table, st);
        case 6: return launch_tile_seg_tm<RP, 48, TRADE>(a, table, st);
    }
    return hipErrorInvalidValue;
}

constexpr int kTileSegRows = 48;
inline bool tile_seg_args_ok(const TileArgs &a)
{
    return a.tile_rows >= 1 && a.tile_rows <= kTileSegRows && a.parts >= 1 && (a.segs || 4 * a.n_segs <= kTileInline);
}

}  // namespace mlora
