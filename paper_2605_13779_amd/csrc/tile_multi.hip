// Dense decode in tiles (see tile_body.h): one or several sites that share a batch plan.
// Bound by the chain launch -> plan -> first loads -> (trade) -> expand, one or two tiles per CU.  Measured
// against the chunk launches of rows.hip: 93 rows at rank 64, 7168 -> 7168, 40.8 -> 14.5 us (33 MB); the seven
// projections of a 2560-wide layer at rank 16, 256 rows 58.6 -> 53.4 us (123 MB), 1001 rows 130.5 -> 93.4 us
// (261 MB).
#include "tile_body.h"

namespace mlora {

// Tiles of a plan, several sites of one rank in a launch: site s owns workgroups [first[s], first[s + 1]).
struct TileMultiArgs {
    int32_t n;
    int32_t first[kMaxMulti + 1];
    TileArgs site[kMaxMulti];
};
// The launch plans for itself (see rows_multi_plan_kernel); workgroup 0 leaves the plan for the launches behind it.
struct TilePlanArgs {
    const int32_t *token_slot, *ready_rank;
    int32_t T, n_slots, rec_bound;
    PlanView pv;
};

// The site this workgroup works on, its launch tag (XCH) and the tile.
template <int RP, int NW, int TM, bool XCH, typename Plan>
__device__ __forceinline__ void tile_multi_body(const TileMultiArgs &m, unsigned char *lds, Plan &&plan)
{
    const int b = (int)blockIdx.x, lane = (int)threadIdx.x & 63;
    int s = 0;
#pragma unroll
    for (int k = 1; k < kMaxMulti; ++k) s += (k < m.n && b >= m.first[k]) ? 1 : 0;
    const TileArgs &a = m.site[s];
    const int wg = b - m.first[s], n_wg = m.first[s + 1] - m.first[s];
    uint32_t tag = 0;
    const bool trade = XCH && a.xch != nullptr;
    if (trade) tag = tag_read(a.ctrl);                           // (every wave by itself: no barrier)
    const int4 *tiles = (const int4 *)a.tiles;
    const int32_t *sorted = a.sorted;
    plan(tiles, sorted);
    // the parts of one tile share its x and A and trade partial sums: on one XCD (workgroups are dealt round-robin)
    const int q = wg >> 3, g8 = q / a.parts, part = q - g8 * a.parts, tile = g8 * 8 + (wg & 7);
    TileRows<TM> t;
    const bool live = tile < a.n_tiles && tile_from_plan<TM>(tiles, sorted, a.top_k, tile, lane, t);
    if (trade) {
        tag = __builtin_amdgcn_readfirstlane(tag);
        if (threadIdx.x == 0) tag_sign_in(a.ctrl, wg, tag);
    }
    if (live) {
        const int blk0 = part * a.part_blocks, n_blk = min(a.part_blocks, ((a.d_out + 63) >> 6) - blk0);
        if constexpr (XCH) {
            tile_body<RP, NW, TM, true>(a, a, t, lds, blk0, n_blk, tile, part, trade ? tag : kTagPoison);
        } else {
            tile_body<RP, NW, TM>(a, a, t, lds, blk0, n_blk);
        }
    }
    if (trade && wg == n_wg - 1 && threadIdx.x < 64 && tag != kTagPoison) tag_advance(a.ctrl, n_wg, tag, lane);
}

template <int RP, int NW, int TM, bool XCH>
__global__ __launch_bounds__(NW * 64, 4)
void tile_multi_kernel(const TileMultiArgs m)
{
    __shared__ __attribute__((aligned(16))) unsigned char lds[TileCfg<RP, NW, TM>::LDS];
    tile_multi_body<RP, NW, TM, XCH>(m, lds, [](const int4 *&, const int32_t *&) {});
}

constexpr int kTilePlanRows = 256;
template <int RP, int NW, int TM, bool XCH>
__global__ __launch_bounds__(NW * 64, 4)
void tile_multi_plan_kernel(const TileMultiArgs m, const TilePlanArgs pl)
{
    // (the planner's tables are dead before the tile's LDS is written: plan_dense_local ends with a barrier)
    __shared__ __attribute__((aligned(16))) unsigned char lds[TileCfg<RP, NW, TM>::LDS];
    static_assert(sizeof(PlanLocalLds) <= TileCfg<RP, NW, TM>::LDS, "the planner's tables fit the tile's LDS");
    __shared__ int4 p_tiles[kTilePlanRows];
    __shared__ int32_t p_sorted[kTilePlanRows];
    tile_multi_body<RP, NW, TM, XCH>(m, lds, [&](const int4 *&tiles, const int32_t *&sorted) {
        plan_dense_local(pl.token_slot, pl.T, pl.n_slots, pl.ready_rank, pl.rec_bound, (int)threadIdx.x, NW * 64, *(PlanLocalLds *)lds, nullptr,
                         blockIdx.x == 0, pl.pv, m.site[0].tile_rows, m.site[0].n_tiles, p_tiles, p_sorted);
        tiles = p_tiles; sorted = p_sorted;
    });
}

template <int RP, int TM, bool XCH>
static hipError_t launch_tile_multi_tm(const TileMultiArgs &m, const TilePlanArgs *pl, hipStream_t st)
{
    const dim3 grid((unsigned)m.first[m.n]), block(512);
    if (pl) tile_multi_plan_kernel<RP, 8, TM, XCH><<<grid, block, 0, st>>>(m, *pl);
    else tile_multi_kernel<RP, 8, TM, XCH><<<grid, block, 0, st>>>(m);
    return hipGetLastError();
}

template <int RP>
static hipError_t launch_tile_multi_rp(const TileMultiArgs &m, const TilePlanArgs *pl, hipStream_t st)
{
    bool xch = false;
    for (int k = 0; k < m.n; ++k) xch = xch || m.site[k].xch;
    if (m.site[0].tile_rows <= 8) return xch ? launch_tile_multi_tm<RP, 8, true>(m, pl, st) : launch_tile_multi_tm<RP, 8, false>(m, pl, st);
    return xch ? launch_tile_multi_tm<RP, 16, true>(m, pl, st) : launch_tile_multi_tm<RP, 16, false>(m, pl, st);
}

static hipError_t launch_tile_multi_any(const TileArgs *sites, int n, const TilePlanArgs *pl, hipStream_t st)
{
    if (n < 1 || n > kMaxMulti || sites[0].tile_rows < kChunk || sites[0].tile_rows > 16) return hipErrorInvalidValue;
    if (sites[0].n_tiles <= 0) return hipSuccess;
    TileMultiArgs m;
    m.n = n;
    m.first[0] = 0;
    for (int k = 0; k < n; ++k) {
        if (sites[k].r_pad != sites[0].r_pad || sites[k].parts < 1) return hipErrorInvalidValue;
        m.site[k] = sites[k];
        m.first[k + 1] = m.first[k] + (sites[k].n_tiles + 7) / 8 * 8 * sites[k].parts;
    }
    for (int k = n; k < kMaxMulti; ++k) { m.site[k] = m.site[0]; m.first[k + 1] = m.first[n]; }
    switch (sites[0].r_pad) {
        case 4:  return launch_tile_multi_rp<4>(m, pl, st);
        case 8:  return launch_tile_multi_rp<8>(m, pl, st);
        case 16: return launch_tile_multi_rp<16>(m, pl, st);
        case 32: return launch_tile_multi_rp<32>(m, pl, st);
        case 64: return launch_tile_multi_rp<64>(m, pl, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_tile_multi(const TileArgs *sites, int n, hipStream_t st) { return launch_tile_multi_any(sites, n, nullptr, st); }

hipError_t launch_tile_multi_plan(const TileArgs *sites, int n, const PlanView &pv, const int32_t *token_slot, int T,
                                  int n_slots, const int32_t *ready_rank, hipStream_t st)
{
    TilePlanArgs pl;
    pl.token_slot = token_slot; pl.ready_rank = ready_rank; pl.T = T; pl.n_slots = n_slots;
    pl.rec_bound = (int)max_chunks(T, n_slots);
    pl.pv = pv;
    if (T < 1 || T > kTilePlanRows || n_slots > kLocalPlanSlots || pl.rec_bound > kTilePlanRows || sites[0].n_tiles > kTilePlanRows) return hipErrorInvalidValue;
    return launch_tile_multi_any(sites, n, &pl, st);
}

}  // namespace mlora
