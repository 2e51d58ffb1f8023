// Dense decode in tiles (see tile_body.h): one or several sites that share a batch plan.
// Bound by the chain launch -> plan -> first loads -> (trade) -> expand, one or two tiles per CU.  Measured
// against the chunk launches of rows.hip: 93 rows at rank 64, 7168 -> 7168, 40.9 -> 12.9 us (33 MB); the seven
// projections of a 2560-wide layer at rank 16, 256 rows 58.5 -> 46.5 us (123 MB), 1001 rows 131.5 -> 86 us
// (261 MB).  Before every workgroup found its own tile and tiles were cut by the live ones: 14.7, 54.7, 92.6.
#include "tile_body.h"

namespace mlora {

// Tiles of a plan, several sites of one rank in a launch.  How many parts a tile is cut in depends on the live tiles (split).
// (What a workgroup needs for its place comes first, in one line.)
struct TileMultiArgs {
    uint64_t split[kSplitEighths / 8];
    int32_t parts[kMaxMulti];                          // (0: no such site)
    const int4 *tiles;
    int32_t n_tiles, n;
    TileArgs site[kMaxMulti];
};
struct TileSplitRegs {
    uint64_t lo, hi;
    int32_t p0, p1, p2, p3;
};
// (Read by name and together: an array subscript that differs between lanes makes the compiler fetch the arguments with vector
// loads, and one at a time.  A line of them that is new to the scalar cache takes about a microsecond, so one word of each line of the
// first site's is read in the same breath.)
__device__ __forceinline__ TileSplitRegs tile_split(const TileMultiArgs &m)
{
    static_assert(kMaxMulti == 4 && kSplitEighths == 16, "");
    const TileSplitRegs r{m.split[0], m.split[1], m.parts[0], m.parts[1], m.parts[2], m.parts[3]};
    asm volatile("" :: "s"(r.lo), "s"(r.hi), "s"(r.p0), "s"(r.p1), "s"(r.p2), "s"(r.p3), "s"(m.tiles), "s"(m.n), "s"(m.n_tiles),
                       "s"(m.site[0].d_in), "s"(m.site[0].tiles), "s"(m.site[0].poll_limit));
    return r;
}

// Workgroup b's place: site s owns the workgroups behind those of the sites before it, eight for every eight tiles and part.
// The parts of one tile share its x and A and trade partial sums: they sit on one XCD (workgroups are dealt round-robin).
struct TilePlace {
    int site, wg, n_wg, parts, part, tile;             // (site -1: none)
};
__device__ __forceinline__ TilePlace tile_place(const TileSplitRegs &r, int b, int eighths)
{
    int p = 1;
    if (eighths <= kSplitEighths) p = (int)((eighths > 8 ? r.hi : r.lo) >> (((eighths - 1) & 7) * 8)) & 0xff;
    TilePlace t{-1, 0, 0, 1, 0, 0};
    auto site = [&](int k, int most) __attribute__((always_inline)) {
        const int pk = min(p, most), nk = 8 * eighths * pk;
        if (b >= 0 && b < nk) { t.site = k; t.wg = b; t.n_wg = nk; t.parts = pk; }
        b -= nk;
    };
    site(0, r.p0); site(1, r.p1); site(2, r.p2); site(3, r.p3);
    const int q = t.wg >> 3, g8 = (int)(((float)q + 0.5f) * __builtin_amdgcn_rcpf((float)t.parts));     // q / parts, exact below 2^20
    t.part = q - g8 * t.parts;
    t.tile = g8 * 8 + (t.wg & 7);
    return t;
}
__device__ __forceinline__ TilePlace tile_place_of_lane(const TilePlace &t, int l)
{
    auto get = [&](int v) { return __builtin_amdgcn_readlane(v, l); };
    return {get(t.site), get(t.wg), get(t.n_wg), get(t.parts), get(t.part), get(t.tile)};
}

// Lines of all sites' arguments into the scalar cache, while the workgroup waits to know its place and with it its site.
__device__ __forceinline__ void tile_args_ahead(const TileMultiArgs &m)
{
    static_assert(kMaxMulti == 4, "four sites' arguments");
    if (m.n > 1)
        asm volatile("" :: "s"(m.site[0].x), "s"(m.site[0].d_in), "s"(m.site[0].top_k), "s"(m.site[1].x), "s"(m.site[1].d_in), "s"(m.site[1].top_k),
                           "s"(m.site[2].x), "s"(m.site[2].d_in), "s"(m.site[2].top_k), "s"(m.site[3].x), "s"(m.site[3].d_in), "s"(m.site[3].top_k), "s"(m.site[3].poll_limit));
}

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
// 6.8 -> 6.2 us (the host's call takes as long), 93 rows, 7168 -> 7168, rank 64 14.5 -> 12.7 by this alone; the 1001-row layer, whose plan had a
// launch of its own (7.8 us), 93.5 -> 87.9.
struct TileBatch {
    int per, n, inc;               // slots per lane, tiles of the lane's slots, tiles up to and with them
    int live;                      // the batch's tiles
};
__device__ __forceinline__ uint32_t tile_magic(int tile_rows) { return (65536u + (uint32_t)tile_rows - 1) / (uint32_t)tile_rows; }
__device__ __forceinline__ int tiles_of(int c, int tile_rows, uint32_t magic)          // exact for c below 4096
{
    return c > 0 ? (int)((uint32_t)(c + tile_rows - 1) * magic >> 16) : 0;
}

template <typename Ahead>
__device__ __forceinline__ TileBatch count_batch(const TilePlanArgs &pl, int tile_rows, TileBatchLds &L, Ahead &&ahead)
{
    constexpr int NT = 512, kNotReady = -(1 << 20);
    const int tid = (int)threadIdx.x, lane = tid & 63, T = pl.T, n_slots = pl.n_slots;
    const int per = n_slots <= 64 ? 1 : (n_slots + 255) / 256 * 4;      // slots per lane in the scan
    int v[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) v[r] = tid + r * NT < T ? pl.token_slot[tid + r * NT] : -1;
    ahead();
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
    const uint32_t magic = tile_magic(tile_rows);
    int n = 0;
    if (per == 1) n = tiles_of(L.cnt[lane], tile_rows, magic);
    else for (int u = 0; u < per; u += 4) {
        const int4 c = *(const int4 *)(L.cnt + lane * per + u);
        n += tiles_of(c.x, tile_rows, magic) + tiles_of(c.y, tile_rows, magic) + tiles_of(c.z, tile_rows, magic) + tiles_of(c.w, tile_rows, magic);
    }
    const int inc = wave_scan<false>(n);
    return {per, n, inc, __builtin_amdgcn_readlane(inc, 63)};
}

template <int TM>
__device__ __forceinline__ bool tile_from_batch(const TileBatch &bt, int T, int tile_rows, int tile, TileBatchLds &L, TileRows<TM> &t)
{
    const int lane = (int)threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const uint64_t hit = __ballot(tile >= bt.inc - bt.n && tile < bt.inc);
    if (hit == 0) return false;
    int at = tile - (bt.inc - bt.n);                                   // the tile's number among the lane's
    int slot = lane, first = at * tile_rows, cnt;
    if (bt.per == 1) cnt = L.cnt[lane] - first;
    else {
        const uint32_t magic = tile_magic(tile_rows);
        cnt = 0;
        for (int u = 0; u < bt.per; ++u) {
            const int c = L.cnt[lane * bt.per + u], m = tiles_of(c, tile_rows, magic);
            if (at >= 0 && at < m) { slot = lane * bt.per + u; first = at * tile_rows; cnt = c - first; }
            at -= m;
        }
    }
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

// The workgroup's tile, one of `live`, found by `find` once its place is known.
template <int RP, int NW, int TM, bool XCH, typename Find>
__device__ __forceinline__ void tile_multi_body(const TileMultiArgs &m, const TilePlace &at, int live, unsigned char *lds, Find &&find)
{
    const int lane = (int)threadIdx.x & 63;
    if (at.site < 0) return;
    const TileArgs &a = m.site[at.site];
    // The site's last workgroup, mostly one without a tile, advances the launch tag when those with a tile have signed in.  (The
    // others without one do not: sign-ins, a handful of lines, wait for each other at the memory side.)
    const bool last = at.wg == at.n_wg - 1;
    if (at.tile >= live && !last) return;
    // One thread reads the tag; tile_body hands it to the others through LDS, where they first need it.  (A wave that read it
    // by itself could come after the launch's last workgroup has advanced it -- nothing but this workgroup's sign-in
    // holds that up -- and would publish this launch's sums under the next one's tag.)
    TileTrade trade{XCH && a.xch != nullptr && at.parts > 1, at.wg, at.parts, 0u};
    if (trade.on && threadIdx.x == 0) trade.tag = tag_read(a.ctrl);
    TileRows<TM> t;
    if (at.tile < live && find(a, t)) {
        const int n_blk = (a.d_out + 63) >> 6;
        const int blk0 = (int)((uint32_t)(at.part * n_blk) / (uint32_t)at.parts), blk1 = (int)((uint32_t)((at.part + 1) * n_blk) / (uint32_t)at.parts);
        if constexpr (XCH) {
            tile_body<RP, NW, TM, true>(a, a, t, lds, blk0, blk1 - blk0, at.tile, at.part, trade);
        } else {
            tile_body<RP, NW, TM>(a, a, t, lds, blk0, blk1 - blk0);
        }
    }
    if (trade.on && last && threadIdx.x < 64) {
        const uint32_t tag = __builtin_amdgcn_readfirstlane(trade.tag);
        if (tag != kTagPoison) tag_advance(a.ctrl, live * at.parts, tag, lane);
    }
}

template <int RP, int NW, int TM, bool XCH>
__global__ __launch_bounds__(NW * 64, 4)
void tile_multi_kernel(const TileMultiArgs m)
{
    __shared__ __attribute__((aligned(16))) unsigned char lds[TileCfg<RP, NW, TM>::LDS];
    // How many tiles are live is in every record of them, so a lane fetches the record that the workgroup would have for 8 * lane
    // + 1 to 8 * lane + 8 of them, and the count says whose it is: one round trip.
    const int lane = (int)threadIdx.x & 63;
    const int4 *tiles = m.tiles;
    const int bound = m.n_tiles;
    const TileSplitRegs split = tile_split(m);
    TilePlace at = tile_place(split, (int)blockIdx.x, min(lane, kSplitEighths - 1) + 1);
    int4 r = tiles[at.tile < bound ? at.tile : 0];
    tile_args_ahead(m);
    const int live = __builtin_amdgcn_readfirstlane(r.w), eighths = (live + 7) >> 3;
    if (live <= 0) return;
    if (eighths <= kSplitEighths) {
        at = tile_place_of_lane(at, eighths - 1);
        r.x = __builtin_amdgcn_readlane(r.x, eighths - 1); r.y = __builtin_amdgcn_readlane(r.y, eighths - 1); r.z = __builtin_amdgcn_readlane(r.z, eighths - 1);
    } else {
        at = tile_place(split, (int)blockIdx.x, eighths);
        r = tiles[at.tile < bound ? at.tile : 0];
    }
    tile_multi_body<RP, NW, TM, XCH>(m, at, live, lds, [&](const TileArgs &a, TileRows<TM> &t) __attribute__((always_inline)) {
        return tile_from_record<TM>(r, a.sorted, a.top_k, lane, t);
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
    const TileSplitRegs split = tile_split(m);
    const TileBatch bt = count_batch(pl, m.site[0].tile_rows, batch, [&]() __attribute__((always_inline)) { tile_args_ahead(m); });
    if (bt.live <= 0) return;
    const TilePlace at = tile_place_of_lane(tile_place(split, b, (bt.live + 7) >> 3), 0);
    tile_multi_body<RP, NW, TM, XCH>(m, at, bt.live, lds, [&](const TileArgs &a, TileRows<TM> &t) __attribute__((always_inline)) {
        return tile_from_batch<TM>(bt, pl.T, a.tile_rows, at.tile, batch, t);
    });
}

template <int RP, int TM, bool XCH>
static hipError_t launch_tile_multi_tm(const TileMultiArgs &m, int wgs, const TilePlanArgs *pl, hipStream_t st)
{
    const dim3 grid((unsigned)wgs + (pl && pl->write ? kTilePlanner : 0)), block(512);
    if (pl) tile_multi_plan_kernel<RP, 8, TM, XCH><<<grid, block, 0, st>>>(m, *pl);
    else tile_multi_kernel<RP, 8, TM, XCH><<<grid, block, 0, st>>>(m);
    return hipGetLastError();
}

template <int RP>
static hipError_t launch_tile_multi_rp(const TileMultiArgs &m, int wgs, const TilePlanArgs *pl, hipStream_t st)
{
    bool xch = false;
    for (int k = 0; k < m.n; ++k) xch = xch || m.site[k].xch;
    if (m.site[0].tile_rows <= 8) return xch ? launch_tile_multi_tm<RP, 8, true>(m, wgs, pl, st) : launch_tile_multi_tm<RP, 8, false>(m, wgs, pl, st);
    return xch ? launch_tile_multi_tm<RP, 16, true>(m, wgs, pl, st) : launch_tile_multi_tm<RP, 16, false>(m, wgs, pl, st);
}

static hipError_t launch_tile_multi_any(const TileArgs *sites, int n, const TileSplit &split, const TilePlanArgs *pl, hipStream_t st)
{
    if (n < 1 || n > kMaxMulti || sites[0].tile_rows < kChunk || sites[0].tile_rows > kMaxTileRows) return hipErrorInvalidValue;
    if (sites[0].n_tiles <= 0) return hipSuccess;
    TileMultiArgs m;
    m.n = n;
    m.n_tiles = sites[0].n_tiles;
    m.tiles = (const int4 *)sites[0].tiles;
    for (int k = 0; k < kSplitEighths / 8; ++k) m.split[k] = split.table[k];
    for (int k = 0; k < kMaxMulti; ++k) {
        const TileArgs &s = sites[k < n ? k : 0];
        if (s.r_pad != sites[0].r_pad || s.parts < 1 || s.n_tiles != sites[0].n_tiles || s.tiles != sites[0].tiles) return hipErrorInvalidValue;
        m.site[k] = s;
        m.parts[k] = k < n ? s.parts : 0;
    }
    switch (sites[0].r_pad) {
        case 4:  return launch_tile_multi_rp<4>(m, split.wgs, pl, st);
        case 8:  return launch_tile_multi_rp<8>(m, split.wgs, pl, st);
        case 16: return launch_tile_multi_rp<16>(m, split.wgs, pl, st);
        case 32: return launch_tile_multi_rp<32>(m, split.wgs, pl, st);
        case 64: return launch_tile_multi_rp<64>(m, split.wgs, pl, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_tile_multi(const TileArgs *sites, int n, const TileSplit &split, hipStream_t st)
{
    return launch_tile_multi_any(sites, n, split, nullptr, st);
}

int tile_plan_rows() { return kSortMax; }
int tile_plan_slots() { return kTilePlanSlots; }

hipError_t launch_tile_multi_plan(const TileArgs *sites, int n, const TileSplit &split, const PlanView &pv, const int32_t *token_slot, int T,
                                  int n_slots, const int32_t *ready_rank, bool write_plan, hipStream_t st)
{
    if (T < 1 || T > tile_plan_rows() || n_slots < 1 || n_slots > tile_plan_slots()) return hipErrorInvalidValue;
    TilePlanArgs pl;
    pl.token_slot = token_slot; pl.ready_rank = ready_rank; pl.T = T; pl.n_slots = n_slots;
    pl.rec_bound = (int)max_chunks(T, n_slots);
    pl.write = write_plan;
    pl.pv = pv;
    return launch_tile_multi_any(sites, n, split, &pl, st);
}

}  // namespace mlora
