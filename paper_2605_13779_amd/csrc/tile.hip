// LoRA apply over tiles of up to 16 or 32 rows that share one adapter (and expert), on the matrix cores:
//   shrink  h[row][j] = sum_i x[row, i] * A[j, i]
//   scale   h *= alpha / r, then a bf16 head and tail (16 bits of h reach the expand)
//   expand  y[row, o] = bf16_rne(float(y[row, o]) + sum_j h[row][j] * B[o, j])      in place
// h stays in LDS.  Used where many rows share an adapter; a chunk of four rows (rows.hip) fetches the
// adapter's rows again for every four, and what a CU can pull through its L1 then bounds the launch.
//
// Shrink operands go to v_mfma_f32_16x16x32_bf16 as whole-line loads leave them: one load covers the same
// 128 bytes of eight rows, lane l holding 16 bytes of row (l/2)%8 at piece 2*(l/16) + l%2.  To the instruction
// lane l%16 = (row, parity of the piece), l/16 the contraction group; products of A and x pieces of equal
// parity are the meant ones, half of what it computes.  They end in accumulators l%2 and 2 + l%2 of lane l
// (adapter rows 2*(l/16) and 2*(l/16) + 1, x row (l%16)/2), to be added over lane pairs once per tile.
// The operand layout proper (a lane per row) would touch four rows with every four neighbouring lanes,
// and the L1's look-ups, one line per four lanes and cycle, become the bound.
#include "plan_device.h"
#include "wave_ops.h"

namespace mlora {

namespace {
constexpr int ST_LD = 68;         // padded row stride of a wave's 16 x 64 staging tile, in floats

__device__ __forceinline__ f32x4_t mfma16(const uint4 &a, const uint4 &b, f32x4_t c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

template <int RP, int NW, int TM>
struct TileCfg {
    static constexpr int NT = NW * 64;
    static constexpr int RPE = RP < 8 ? 8 : RP;                // ranks as the expand sees them (zeros behind RP)
    static constexpr int RGN = RP < 16 ? 1 : 2;                // groups of eight adapter rows per wave
    static constexpr int RGW = RP <= 16 ? 1 : RP / 16;         // waves side by side over the adapter's rows
    static constexpr int KSW = NW / RGW;                       // waves side by side over d_in
    static constexpr int TG = TM / 8;                          // groups of eight x rows
    static constexpr int DP = TM <= 8 ? (RP <= 16 ? 6 : 4) : (TM <= 16 ? 4 : (TM <= 32 ? 3 : 2));                // shrink steps in flight per wave
    static constexpr bool K16 = RP <= 16;                      // expand on 16x16x16 (4 ranks per lane), else 16x16x32 (8)
    static constexpr int KC = RP <= 32 ? 1 : 2;                // pieces of B per lane and output
    static constexpr int HF = RP <= 8 ? 1 : 2 * KC;            // h operands per 16 rows
    static constexpr int BW = K16 ? 2 : 4;                     // words of a piece of B
    static constexpr int TH = (TM + 15) / 16;                  // halves of 16 rows in the expand
    static constexpr int ED = TM <= 8 ? (RP < 16 ? 6 : (RP == 16 ? 5 : (RP == 32 ? 4 : 2))) : TM <= 16 ? (RP <= 16 ? 4 : (RP == 32 ? 3 : 2)) : (TM <= 32 && RP <= 32 ? 3 : 2);   // expand blocks in flight per wave
    static constexpr int H_LD = RPE + 8;                       // padded row stride of h in LDS, in elements
    static constexpr int H_BYTES = 2 * TH * 16 * H_LD * 2;
    static constexpr int PART_BYTES = KSW * TM * RPE * 4, STG_BYTES = NW * 16 * ST_LD * 4;
    static constexpr int LDS = H_BYTES + (PART_BYTES > STG_BYTES ? PART_BYTES : STG_BYTES);
};
}  // namespace

// What a tile is made of: the adapter, and for this lane the rows it loads x from and adds y to.
template <int TM>
struct TileRows {
    int key, cnt;
    int xrow[TM / 8];              // row 8 * g + (lane / 2) % 8 of the tile
    int yrow[TM / 8];              // row 8 * g + lane / 8
};

// The tile's segment: segs holds, per segment, its first tile, first row, rows and slot.
template <int TM>
__device__ __forceinline__ bool tile_from_segments(const TileArgs &a, const uint32_t *segs, int tile, int lane, TileRows<TM> &t)
{
    int first = 0, row0 = 0, rows = 0, slot = -1;
    for (int s0 = 0; s0 < a.n_segs; s0 += 64) {
        const int si = s0 + lane;
        int4 v = make_int4(0x7fffffff, 0, 0, 0);
        if (si < a.n_segs) v = ((const int4 *)segs)[si];
        const uint64_t hit = __ballot(v.x <= tile);          // segments in tile order: the last one that starts at or before it
        if (hit) {
            const int l = 63 - __builtin_clzll(hit);
            first = __shfl(v.x, l, 64); row0 = __shfl(v.y, l, 64); rows = __shfl(v.z, l, 64); slot = __shfl(v.w, l, 64);
        }
        if (hit != ~0ull) break;
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

// Tile `tile` of a plan: its record and rows (in global memory, or in LDS where the launch planned for itself).
template <int TM>
__device__ __forceinline__ bool tile_from_plan(const int4 *tiles, const int32_t *sorted, int top_k, int tile, int lane, TileRows<TM> &t)
{
    const int4 r = tiles[tile];
    t.key = __builtin_amdgcn_readfirstlane(r.x);
    t.cnt = __builtin_amdgcn_readfirstlane(r.y);
    if (t.cnt <= 0) return false;
    const int32_t *rows = sorted + __builtin_amdgcn_readfirstlane(r.z);
#pragma unroll
    for (int g = 0; g < TM / 8; ++g) {
        t.xrow[g] = rows[min(8 * g + ((lane >> 1) & 7), t.cnt - 1)];
        t.yrow[g] = rows[min(8 * g + (lane >> 3), t.cnt - 1)];
    }
    if (top_k > 1) {                               // (at once: the division waits for the rows)
#pragma unroll
        for (int g = 0; g < TM / 8; ++g) t.xrow[g] /= top_k;
    }
    return true;
}

// blk0, n_blk: the blocks of 64 outputs to expand.  XCH: the tile's a.parts workgroups also divide d_in; each
// publishes the sums of its slice as words (value, launch tag) and adds everybody's in slice order.  A wait
// for a partner's words is bounded: on giving up the workgroup sums all of d_in itself.  A launch tag that says
// so (kTagPoison) makes every part sum all of d_in from the start.
template <int RP, int NW, int TM, bool XCH = false>
__device__ __forceinline__ void tile_body(const TileArgs &a, const TileRows<TM> &t, unsigned char *lds, const int blk0, const int n_blk,
                                          const int tile = 0, const int part_i = 0, const uint32_t tag = 0)
{
    using C = TileCfg<RP, NW, TM>;
    uint16_t *const hs_hi = (uint16_t *)lds, *const hs_lo = hs_hi + C::TH * 16 * C::H_LD;
    float *const part = (float *)(lds + C::H_BYTES);              // [KSW][TM][RPE]
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int slot = t.key / a.n_experts;
    const int U = a.d_in >> 3;                                   // 16-byte units per row of x / A

    // ---- shrink: wave w takes adapter rows [16 * (w % RGW), ..) and every KSW-th step of 8 units ----
    const int rgw = w % C::RGW, ksw = w / C::RGW;
    const int lr = (lane >> 1) & 7;
    const int lu = (lane >> 4) * 2 + (lane & 1);
    const int n_steps = (U + 7) >> 3;
    const char *Ag = (const char *)(a.a_tab + (int64_t)t.key * RP * a.d_in);
    const uint32_t row_bytes = (uint32_t)a.d_in * 2u;
    uint32_t a_off[C::RGN];
#pragma unroll
    for (int j = 0; j < C::RGN; ++j) a_off[j] = (uint32_t)min(rgw * 16 + j * 8 + lr, RP - 1) * row_bytes;
    const char *xp[C::TG];
    const bool solo = !XCH || tag == kTagPoison;
    __shared__ int s_missing;
    if (XCH && tid == 0) s_missing = 0;                          // (first looked at behind a barrier)
    // steps [st0, st1) of d_in; this wave's i-th is st0 + ksw + i * KSW
    const int st0 = solo ? 0 : part_i * n_steps / a.parts, st1 = solo ? n_steps : (part_i + 1) * n_steps / a.parts;
    const int n = (st1 - st0 - ksw + C::KSW - 1) / C::KSW;
    auto unit_of = [&](int i) { return (st0 + i * C::KSW + ksw) * 8 + lu; };
    uint4 av[C::DP][C::RGN], xv[C::DP][C::TG];
    auto load_a = [&](int i, auto slot_c) __attribute__((always_inline)) {
        constexpr int d = decltype(slot_c)::value;
        const uint32_t u16 = (uint32_t)min(unit_of(i), U - 1) * 16u;
#pragma unroll
        for (int j = 0; j < C::RGN; ++j) av[d][j] = *(const uint4 *)(Ag + (size_t)(a_off[j] + u16));
    };
    auto load_x = [&](int i, auto slot_c) __attribute__((always_inline)) {
        constexpr int d = decltype(slot_c)::value;
        const uint32_t u16 = (uint32_t)min(unit_of(i), U - 1) * 16u;
#pragma unroll
        for (int g = 0; g < C::TG; ++g) xv[d][g] = ld_stream(xp[g] + u16);
    };
    auto load = [&](int i, auto slot_c) __attribute__((always_inline)) { load_a(i, slot_c); load_x(i, slot_c); };
    f32x4_t acc[C::RGN][C::TG];
    auto consume = [&](int i, auto slot_c) __attribute__((always_inline)) {
        constexpr int d = decltype(slot_c)::value;
        const bool in = unit_of(i) < U;
#pragma unroll
        for (int g = 0; g < C::TG; ++g) {
            const uint4 xz = in ? xv[d][g] : make_uint4(0, 0, 0, 0);
#pragma unroll
            for (int j = 0; j < C::RGN; ++j) acc[j][g] = mfma16(av[d][j], xz, acc[j][g]);
        }
    };
    auto shrink = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < C::RGN; ++j)
#pragma unroll
            for (int g = 0; g < C::TG; ++g) acc[j][g] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        if (n <= 0) return;
        // (A does not depend on the tile's row list, which may still be on its way.  No step is requested twice:
        // the loads under a condition only stand where the pipeline ends, where a wait for all of them costs little.)
        auto open_x = [&]() {
#pragma unroll
            for (int g = 0; g < C::TG; ++g) xp[g] = (const char *)(a.x + (int64_t)t.xrow[g] * a.ldx);
        };
        if (n < C::DP) {
            static_for<C::DP>([&](auto d) { if (d.value < n) load_a(d.value, d); });
            open_x();
            static_for<C::DP>([&](auto d) { if (d.value < n) load_x(d.value, d); });
            static_for<C::DP>([&](auto d) { if (d.value < n) consume(d.value, d); });
            return;
        }
        static_for<C::DP>([&](auto d) { load_a(d.value, d); });
        open_x();
        static_for<C::DP>([&](auto d) { load_x(d.value, d); });
        int i = 0;
        for (; i + 2 * C::DP <= n; i += C::DP)
            static_for<C::DP>([&](auto d) { consume(i + d.value, d); load(i + C::DP + d.value, d); });
        static_for<C::DP>([&](auto d) { consume(i + d.value, d); if (i + C::DP + d.value < n) load(i + C::DP + d.value, d); });
        static_for<C::DP>([&](auto d) { if (i + C::DP + d.value < n) consume(i + C::DP + d.value, d); });
    };
    int rank = 0;
    float scale = 0.f;

    // ---- the first outputs' B and y travel while the partial sums meet ----
    const int mm = lane & 15, kq = lane >> 4, tr = lane >> 3, og = lane & 7;
    const int nb = (n_blk - w + NW - 1) / NW, w_blk = blk0 + w;          // this wave's blocks of 64 outputs: every NW-th
    const char *Bg = (const char *)(a.b_tab + (int64_t)t.key * a.d_out * RP);
    char *yp[C::TG];
#pragma unroll
    for (int g = 0; g < C::TG; ++g) yp[g] = (char *)(a.y + (int64_t)t.yrow[g] * a.ldy);
    uint32_t bv[C::ED][4][C::KC][C::BW];
    uint4 yv[C::ED][C::TG];
    auto fetch = [&](int b, auto buf_c) __attribute__((always_inline)) {
        constexpr int d = decltype(buf_c)::value;
        const int o_w = (b * NW + w_blk) * 64;
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
            const uint32_t o = (uint32_t)min(o_w + cb * 16 + mm, a.d_out - 1);
#pragma unroll
            for (int k = 0; k < C::KC; ++k) {
                uint32_t (&v)[C::BW] = bv[d][cb][k];
                if constexpr (RP >= 32) {
                    const uint4 q = *(const uint4 *)(Bg + (o * (uint32_t)(RP * 2) + (uint32_t)(k * 64 + kq * 16)));
                    v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
                } else if constexpr (RP >= 8) {                     // (rank 8: lane groups 2 and 3 load what 0 and 1 load)
                    const uint2 q = *(const uint2 *)(Bg + (o * (uint32_t)(RP * 2) + (uint32_t)((RP == 8 ? kq & 1 : kq) * 8)));
                    v[0] = q.x; v[1] = q.y;
                } else if constexpr (RP == 4) {
                    const uint2 q = *(const uint2 *)(Bg + o * 8u);
                    v[0] = q.x; v[1] = q.y;
                } else if constexpr (RP == 2) {
                    v[0] = *(const uint32_t *)(Bg + o * 4u); v[1] = 0u;
                } else {
                    v[0] = *(const uint16_t *)(Bg + o * 2u); v[1] = 0u;
                }
            }
        }
        const uint32_t oc = (uint32_t)min(o_w + og * 8, a.d_out - 8) * 2u;
#pragma unroll
        for (int g = 0; g < C::TG; ++g) yv[d][g] = *(const uint4 *)(yp[g] + oc);
    };
    auto first_fetch = [&]() __attribute__((always_inline)) {
        rank = a.rank[slot];
        scale = a.scale[slot];
        if (nb >= C::ED) static_for<C::ED>([&](auto d) { fetch(d.value, d); });
        else static_for<C::ED>([&](auto d) { if (d.value < nb) fetch(d.value, d); });
    };

    // ---- partial sums of the waves -> h ----
    auto sums_to_lds = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < C::RGN; ++j) {
            if (rgw * 16 + j * 8 >= C::RPE) continue;
#pragma unroll
            for (int g = 0; g < C::TG; ++g) {
                const bool odd = lane & 1;
                float v0 = odd ? acc[j][g][1] : acc[j][g][0], v1 = odd ? acc[j][g][3] : acc[j][g][2];
                v0 += lane_xor<1>(v0);
                v1 += lane_xor<1>(v1);
                // lane (row pair kq of the eight, x row (lane % 16) / 2): even lanes keep the first, odd ones the second
                part[(ksw * TM + g * 8 + (mm >> 1)) * C::RPE + rgw * 16 + j * 8 + kq * 2 + (lane & 1)] = odd ? v1 : v0;
            }
        }
        __syncthreads();
    };
    auto own_sum = [&](int e) {
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < C::KSW; ++k) s += part[k * (TM * C::RPE) + e];
        return s;
    };
    auto put_h = [&](int e, float s) {
        const int m = e / C::RPE, j = e % C::RPE;
        s = j < RP ? s * scale : 0.f;
        const uint32_t hi = f2bf(s);
        hs_hi[m * C::H_LD + j] = (uint16_t)hi;
        hs_lo[m * C::H_LD + j] = (uint16_t)f2bf(s - __uint_as_float(hi << 16));
    };
    shrink();
    first_fetch();
    sums_to_lds();
    if (!XCH || solo) {
        for (int e = tid; e < TM * C::RPE; e += C::NT) put_h(e, own_sum(e));
    } else {
        const int n_e = t.cnt * C::RPE;                          // rows past the count are nobody's
        uint64_t *const xw = a.xch + (int64_t)tile * a.parts * (TM * C::RPE);
        for (int e = tid; e < n_e; e += C::NT) xch_put(xw + (int64_t)part_i * (TM * C::RPE) + e, own_sum(e), tag);
        bool gave_up = false;
        for (int e = tid; e < n_e; e += C::NT) {
            float s = 0.f;
            for (int p0 = 0; p0 < a.parts; p0 += 4) {            // four words in flight, added in slice order
                uint64_t wv[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) if (p0 + k < a.parts) wv[k] = xch_get(xw + (int64_t)(p0 + k) * (TM * C::RPE) + e);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if (p0 + k >= a.parts) break;
                    if (p0 + k == part_i) { s += own_sum(e); continue; }
                    int spins = 0;
                    while ((uint32_t)(wv[k] >> 32) != tag) {
                        if (++spins > a.poll_limit) { gave_up = true; break; }
                        __builtin_amdgcn_s_sleep(1);
                        wv[k] = xch_get(xw + (int64_t)(p0 + k) * (TM * C::RPE) + e);
                    }
                    s += __uint_as_float((uint32_t)wv[k]);
                }
            }
            put_h(e, s);
        }
        if (gave_up) atomicOr(&s_missing, 1);
        __syncthreads();
        if (s_missing) {
            // Never expected: every element as a plain dot product (slow, but it needs nothing of what is in flight).
#pragma unroll
            for (int g = 0; g < C::TG; ++g) {
                for (int e0 = 0; e0 < 8 * C::RPE; e0 += C::NT) {
                    const int e = e0 + tid, m = min(e / C::RPE, 7), j = min(e % C::RPE, RP - 1);
                    const char *xr = (const char *)(a.x + (int64_t)__shfl(t.xrow[g], 2 * m, 64) * a.ldx), *ar = Ag + (size_t)((uint32_t)j * row_bytes);
                    float s = 0.f;
                    for (uint32_t u = 0; u < (uint32_t)U * 16u; u += 16u) s = dot8(*(const uint4 *)(xr + u), *(const uint4 *)(ar + u), s);
                    if (e < 8 * C::RPE) put_h(g * 8 * C::RPE + e, s);
                }
            }
        }
    }
    __syncthreads();
    if (rank <= 0) return;                                       // empty slot: rows stay untouched

    // ---- h as operand: rows m of each half of 16 ----
    // 16 x 16 x 16: lane group kq holds 4 ranks.  Rank 16: heads in one instruction, tails in a second; rank 8
    // and below: heads in groups 0 and 1 (what lies behind the rank is zero), tails in 2 and 3.
    uint4 hv[C::TH][C::HF];
#pragma unroll
    for (int half = 0; half < C::TH; ++half) {
        const uint16_t *ph = hs_hi + (half * 16 + mm) * C::H_LD, *pl = hs_lo + (half * 16 + mm) * C::H_LD;
        if constexpr (RP == 8) {
            const uint2 v = *(const uint2 *)((kq < 2 ? ph : pl) + (kq & 1) * 4);
            hv[half][0] = make_uint4(v.x, v.y, 0u, 0u);
        } else if constexpr (RP < 8) {                              // all groups load the same B: heads in 0, tails in 1, zeros
            const uint2 v = *(const uint2 *)((kq & 1) ? pl : ph);
            hv[half][0] = kq < 2 ? make_uint4(v.x, v.y, 0u, 0u) : make_uint4(0u, 0u, 0u, 0u);
        } else if constexpr (RP == 16) {
            const uint2 v = *(const uint2 *)(ph + kq * 4), u = *(const uint2 *)(pl + kq * 4);
            hv[half][0] = make_uint4(v.x, v.y, 0u, 0u); hv[half][1] = make_uint4(u.x, u.y, 0u, 0u);
        } else {
#pragma unroll
            for (int k = 0; k < C::KC; ++k) {
                hv[half][2 * k] = *(const uint4 *)(ph + k * 32 + kq * 8);
                hv[half][2 * k + 1] = *(const uint4 *)(pl + k * 32 + kq * 8);
            }
        }
    }
    // ---- expand: the accumulators pass through a staging tile of the wave so that y moves in row pieces ----
    float *stg = (float *)(lds + C::H_BYTES) + w * (16 * ST_LD);
    auto block = [&](int b, auto buf_c) __attribute__((always_inline)) {
        constexpr int d = decltype(buf_c)::value;
        const int o_w = (b * NW + w_blk) * 64;
        const bool col_ok = o_w + og * 8 < a.d_out;
        const uint32_t oc = (uint32_t)(o_w + og * 8) * 2u;
#pragma unroll
        for (int half = 0; half < C::TH; ++half) {
            if (half * 16 >= t.cnt) break;
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) {
                f32x4_t c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int f = 0; f < C::HF; ++f) {
                    const uint32_t *v = bv[d][cb][f / 2];
                    if constexpr (C::K16)
                        c = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4_t, make_uint2(hv[half][f].x, hv[half][f].y)),
                                                                      __builtin_bit_cast(s16x4_t, make_uint2(v[0], v[1])), c, 0, 0, 0);
                    else
                        c = mfma16(hv[half][f], make_uint4(v[0], v[1], v[2], v[C::BW - 1]), c);
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) stg[(4 * kq + i) * ST_LD + cb * 16 + mm] = c[i];
            }
            // (the staging tile is the wave's own and LDS serves a wave in order: compiler-level fences are enough)
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int trow = tr + 8 * q, g = half * 2 + q;
                if (g >= C::TG) break;
                const float4 d0 = *(const float4 *)(stg + trow * ST_LD + og * 8), d1 = *(const float4 *)(stg + trow * ST_LD + og * 8 + 4);
                const uint4 yo = yv[d][g];
                uint4 o;
                o.x = pack_bf2(bf_lo(yo.x) + d0.x, bf_hi(yo.x) + d0.y);
                o.y = pack_bf2(bf_lo(yo.y) + d0.z, bf_hi(yo.y) + d0.w);
                o.z = pack_bf2(bf_lo(yo.z) + d1.x, bf_hi(yo.z) + d1.y);
                o.w = pack_bf2(bf_lo(yo.w) + d1.z, bf_hi(yo.w) + d1.w);
                if (half * 16 + trow < t.cnt && col_ok) st_quiet(yp[g] + oc, o);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
    };
    int b = 0;
    for (; b + 2 * C::ED <= nb; b += C::ED)
        static_for<C::ED>([&](auto d) { block(b + d.value, d); fetch(b + C::ED + d.value, d); });
    static_for<C::ED>([&](auto d) {
        if (b + d.value < nb) block(b + d.value, d);
        if (b + C::ED + d.value < nb) fetch(b + C::ED + d.value, d);
    });
    static_for<C::ED>([&](auto d) { if (b + C::ED + d.value < nb) block(b + C::ED + d.value, d); });
}

struct TileSegInline { uint32_t w[kTileInline]; };

template <int RP, int NW, int TM>
__global__ __launch_bounds__(NW * 64, 2)
void tile_seg_kernel(const TileArgs a, const TileSegInline inl)
{
    __shared__ __attribute__((aligned(16))) unsigned char lds[TileCfg<RP, NW, TM>::LDS];
    // an XCD gets a contiguous range of tiles (workgroups are dealt round-robin): neighbours share an adapter, in its L2
    const int n8 = (int)gridDim.x >> 3, tile = ((int)blockIdx.x & 7) * n8 + ((int)blockIdx.x >> 3);
    if (tile >= a.n_tiles) return;
    TileRows<TM> t;
    if (!tile_from_segments<TM>(a, a.segs ? (const uint32_t *)a.segs : inl.w, tile, (int)threadIdx.x & 63, t)) return;
    tile_body<RP, NW, TM>(a, t, lds, 0, (a.d_out + 63) >> 6);
}

template <int RP>
static hipError_t launch_tile_seg_rp(const TileArgs &a, const uint32_t *inl, hipStream_t st)
{
    TileSegInline table;
    if (!a.segs) for (int i = 0; i < 4 * a.n_segs; ++i) table.w[i] = inl[i];
    const dim3 grid((unsigned)((a.n_tiles + 7) / 8 * 8)), block(512);
    switch ((a.tile_rows + 7) / 8) {
        case 1: tile_seg_kernel<RP, 8, 8><<<grid, block, 0, st>>>(a, table); break;
        case 2: tile_seg_kernel<RP, 8, 16><<<grid, block, 0, st>>>(a, table); break;
        case 3: tile_seg_kernel<RP, 8, 24><<<grid, block, 0, st>>>(a, table); break;
        case 4: tile_seg_kernel<RP, 8, 32><<<grid, block, 0, st>>>(a, table); break;
        case 5: tile_seg_kernel<RP, 8, 40><<<grid, block, 0, st>>>(a, table); break;
        case 6: tile_seg_kernel<RP, 8, 48><<<grid, block, 0, st>>>(a, table); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

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
            tile_body<RP, NW, TM, true>(a, t, lds, blk0, n_blk, tile, part, trade ? tag : kTagPoison);
        } else {
            tile_body<RP, NW, TM>(a, t, lds, blk0, n_blk);
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

int tile_max_rows() { return 48; }

hipError_t launch_tile_seg(const TileArgs &a, const uint32_t *inl, hipStream_t st)
{
    if (a.n_tiles <= 0) return hipSuccess;
    if (a.tile_rows < 1 || a.tile_rows > tile_max_rows() || (!a.segs && 4 * a.n_segs > kTileInline)) return hipErrorInvalidValue;
    switch (a.r_pad) {
        case 1:  return launch_tile_seg_rp<1>(a, inl, st);
        case 2:  return launch_tile_seg_rp<2>(a, inl, st);
        case 4:  return launch_tile_seg_rp<4>(a, inl, st);
        case 8:  return launch_tile_seg_rp<8>(a, inl, st);
        case 16: return launch_tile_seg_rp<16>(a, inl, st);
        case 32: return launch_tile_seg_rp<32>(a, inl, st);
        case 64: return launch_tile_seg_rp<64>(a, inl, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace mlora
