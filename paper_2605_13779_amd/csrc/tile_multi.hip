// Dense decode in tiles (see tile_body.h): one or several sites that share a batch plan.
// Bound by the chain launch -> plan -> first loads -> (trade) -> expand, one or two tiles per CU.  Measured
// against the chunk launches of rows.hip: 93 rows at rank 64, 7168 -> 7168, 40.9 -> 14.5 us (33 MB); the seven
// projections of a 2560-wide layer at rank 16, 256 rows 58.5 -> 54.7 us (123 MB), 1001 rows 131.5 -> 92.8 us
// (261 MB).
#include "tile_body.h"

namespace mlora {

// Tiles of a plan, several sites of one rank in a launch: site s owns workgroups [first[s], first[s + 1]).
struct TileMultiArgs {
    int32_t n;
    int32_t first[kMaxMulti + 1];
    TileArgs site[kMaxMulti];
};
// The launch plans for itself: every workgroup finds its own tile in the batch (tile_from_batch); where launches behind
// it want the plan, workgroup 0 of kTilePlanner in front of the others writes it and does nothing else.
constexpr int kTilePlanSlots = 1024, kTilePlanner = 8;      // (8: the workgroups behind keep their XCDs)
struct TilePlanArgs {
    const int32_t *token_slot, *ready_rank;
    int32_t T, n_slots, rec_bound, write;
    PlanView pv;
};

struct TileBatchLds {
    __attribute__((aligned(16))) int32_t cnt[kTilePlanSlots];     // rows of the slot (far below zero: the slot is not ready)
    int32_t key[kSortMax];                                        // the rows' slots (-1: none)
    int32_t rows[8][kMaxTileRows];                                // per wave: the tile's rows
};

// Tile `tile` of the plan that plan_dense_count would write, found by a workgroup of eight waves for itself: one round trip
// for all slots, two barriers around their count, then every wave by itself: a scan over the slots' tiles, and the rows
// of the one slot by ballots.  The places of other tiles' rows, chunk records and their scans, which took two thirds of
// the time of a launch in which everybody built the whole plan, are not needed for that.  One token, 2560 -> 2560, rank 16
// 6.8 -> 6.2 us (the host's call takes as long), 93 rows, 7168 -> 7168, rank 64 14.5 -> 12.7; the 1001-row layer, whose plan had a
// launch of its own (7.8 us), 93.5 -> 87.9.
template <int TM>
__device__ __forceinline__ bool tile_from_batch(const TilePlanArgs &pl, int tile_rows, int tile, TileBatchLds &L, TileRows<TM> &t)
{
    constexpr int NT = 512, kNotReady = -(1 << 20);
    const int tid = (int)threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int T = pl.T, n_slots = pl.n_slots;
    const int per = n_slots <= 64 ? 1 : (n_slots + 255) / 256 * 4;      // slots per lane in the scan
    int v[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) v[r] = tid + r * NT < T ? pl.token_slot[tid + r * NT] : -1;
    for (int k = tid; k < 64 * per; k += NT) L.cnt[k] = pl.ready_rank && k < n_slots && pl.ready_rank[k] <= 0 ? kNotReady : 0;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        if (v[r] >= n_slots) v[r] = -1;
        L.key[tid + r * NT] = v[r];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 2; ++r) if (v[r] >= 0) atomicAdd(&L.cnt[v[r]], 1);
    __syncthreads();
    const uint32_t magic = (65536u + (uint32_t)tile_rows - 1) / (uint32_t)tile_rows;       // c / tile_rows, exact for c below 4096
    auto tiles_of = [&](int c) { return c > 0 ? (int)((uint32_t)(c + tile_rows - 1) * magic >> 16) : 0; };
    int slot = 0, first = 0, cnt = 0;
    uint64_t hit;
    if (per == 1) {
        const int c = L.cnt[lane], n = tiles_of(c), inc = wave_scan<false>(n);
        hit = __ballot(tile >= inc - n && tile < inc);
        slot = lane;
        first = (tile - (inc - n)) * tile_rows;
        cnt = c - first;
    } else {
        int n = 0;
        for (int u = 0; u < per; u += 4) {
            const int4 c = *(const int4 *)(L.cnt + lane * per + u);
            n += tiles_of(c.x) + tiles_of(c.y) + tiles_of(c.z) + tiles_of(c.w);
        }
        const int inc = wave_scan<false>(n);
        hit = __ballot(tile >= inc - n && tile < inc);
        int at = tile - (inc - n);                                     // the tile's number among the lane's
        for (int u = 0; u < per; ++u) {
            const int c = L.cnt[lane * per + u], m = tiles_of(c);
            if (at >= 0 && at < m) { slot = lane * per + u; first = at * tile_rows; cnt = c - first; }
            at -= m;
        }
    }
    if (hit == 0) return false;
    const int l = (int)__builtin_ctzll(hit);
    t.key = __builtin_amdgcn_readlane(slot, l);
    const int first_s = __builtin_amdgcn_readlane(first, l);
    t.cnt = min(tile_rows, __builtin_amdgcn_readlane(cnt, l));
    int base = -first_s;
    const int n_groups = (T + 63) >> 6;
    for (int g = 0; g < n_groups; ++g) {
        const uint64_t m = __ballot(L.key[64 * g + lane] == t.key);
        const int r = base + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        if ((m >> lane & 1u) && r >= 0 && r < t.cnt) L.rows[w][r] = 64 * g + lane;
        base += __popcll(m);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");             // (the wave's own words: LDS serves a wave in order)
#pragma unroll
    for (int g = 0; g < TM / 8; ++g) {
        t.xrow[g] = L.rows[w][min(8 * g + ((lane >> 1) & 7), t.cnt - 1)];
        t.yrow[g] = L.rows[w][min(8 * g + (lane >> 3), t.cnt - 1)];
    }
    return true;
}

// The site this workgroup works on, its launch tag (XCH) and the tile.
template <int RP, int NW, int TM, bool XCH, typename Find>
__device__ __forceinline__ void tile_multi_body(const TileMultiArgs &m, const int b, unsigned char *lds, Find &&find)
{
    const int lane = (int)threadIdx.x & 63;
    int s = 0;
#pragma unroll
    for (int k = 1; k < kMaxMulti; ++k) s += (k < m.n && b >= m.first[k]) ? 1 : 0;
    const TileArgs &a = m.site[s];
    const int wg = b - m.first[s], n_wg = m.first[s + 1] - m.first[s];
    // One thread reads the tag; tile_body hands it to the others through LDS, where they first need it.  (A wave that read it
    // by itself could come after the launch's last workgroup has advanced it -- nothing but this workgroup's sign-in
    // holds that up -- and would publish this launch's sums under the next one's tag.)
    TileTrade trade{XCH && a.xch != nullptr, wg, 0u};
    if (trade.on && threadIdx.x == 0) trade.tag = tag_read(a.ctrl);
    // the parts of one tile share its x and A and trade partial sums: on one XCD (workgroups are dealt round-robin)
    const int q = wg >> 3, g8 = q / a.parts, part = q - g8 * a.parts, tile = g8 * 8 + (wg & 7);
    TileRows<TM> t;
    const bool live = tile < a.n_tiles && find(a, tile, t);
    if (live) {
        const int blk0 = part * a.part_blocks, n_blk = min(a.part_blocks, ((a.d_out + 63) >> 6) - blk0);
        if constexpr (XCH) {
            tile_body<RP, NW, TM, true>(a, a, t, lds, blk0, n_blk, tile, part, trade);
        } else {
            tile_body<RP, NW, TM>(a, a, t, lds, blk0, n_blk);
        }
    } else if (trade.on && threadIdx.x == 0) {
        tag_sign_in(a.ctrl, wg, trade.tag);                      // (a live tile's workgroup does so in tile_body)
    }
    if (trade.on && wg == n_wg - 1 && threadIdx.x < 64) {
        const uint32_t tag = __builtin_amdgcn_readfirstlane(trade.tag);
        if (tag != kTagPoison) tag_advance(a.ctrl, n_wg, tag, lane);
    }
}

template <int RP, int NW, int TM, bool XCH>
__global__ __launch_bounds__(NW * 64, 4)
void tile_multi_kernel(const TileMultiArgs m)
{
    __shared__ __attribute__((aligned(16))) unsigned char lds[TileCfg<RP, NW, TM>::LDS];
    tile_multi_body<RP, NW, TM, XCH>(m, (int)blockIdx.x, lds, [](const TileArgs &a, int tile, TileRows<TM> &t) __attribute__((always_inline)) {
        return tile_from_plan<TM>((const int4 *)a.tiles, a.sorted, a.top_k, tile, (int)threadIdx.x & 63, t);
    });
}

template <int RP, int NW, int TM, bool XCH>
__global__ __launch_bounds__(NW * 64, 4)
void tile_multi_plan_kernel(const TileMultiArgs m, const TilePlanArgs pl)
{
    static_assert(NW == 8 && sizeof(PlanCountLds<kTilePlanSlots>) <= TileCfg<RP, NW, TM>::LDS, "the planner's tables fit the tile's LDS");
    __shared__ __attribute__((aligned(16))) unsigned char lds[TileCfg<RP, NW, TM>::LDS];
    __shared__ TileBatchLds batch;
    const int b = (int)blockIdx.x - (pl.write ? kTilePlanner : 0);
    if (b < 0) {
        if (b == -kTilePlanner)
            plan_dense_count<2, kTilePlanSlots>(pl.pv, pl.token_slot, pl.T, pl.n_slots, pl.ready_rank, pl.rec_bound, m.site[0].tile_rows, m.site[0].n_tiles,
                                                (int)threadIdx.x, NW * 64, *(PlanCountLds<kTilePlanSlots> *)lds);
        return;
    }
    tile_multi_body<RP, NW, TM, XCH>(m, b, lds, [&](const TileArgs &a, int tile, TileRows<TM> &t) __attribute__((always_inline)) {
        return tile_from_batch<TM>(pl, a.tile_rows, tile, batch, t);
    });
}

template <int RP, int TM, bool XCH>
static hipError_t launch_tile_multi_tm(const TileMultiArgs &m, const TilePlanArgs *pl, hipStream_t st)
{
    const dim3 grid((unsigned)m.first[m.n] + (pl && pl->write ? kTilePlanner : 0)), block(512);
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
    if (n < 1 || n > kMaxMulti || sites[0].tile_rows < kChunk || sites[0].tile_rows > kMaxTileRows) return hipErrorInvalidValue;
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

int tile_plan_rows() { return kSortMax; }
int tile_plan_slots() { return kTilePlanSlots; }

hipError_t launch_tile_multi_plan(const TileArgs *sites, int n, const PlanView &pv, const int32_t *token_slot, int T,
                                  int n_slots, const int32_t *ready_rank, bool write_plan, hipStream_t st)
{
    if (T < 1 || T > tile_plan_rows() || n_slots < 1 || n_slots > tile_plan_slots()) return hipErrorInvalidValue;
    TilePlanArgs pl;
    pl.token_slot = token_slot; pl.ready_rank = ready_rank; pl.T = T; pl.n_slots = n_slots;
    pl.rec_bound = (int)max_chunks(T, n_slots);
    pl.write = write_plan;
    pl.pv = pv;
    return launch_tile_multi_any(sites, n, &pl, st);
}

}  // namespace mlora
