// LoRA apply over tiles of up to 16 (decode, MoE) or 48 rows (prefill) that share one adapter (and expert), on the
// matrix cores:
//   shrink  h[row][j] = sum_i x[row, i] * A[j, i]
//   scale   h *= alpha / r, then three bf16 terms (all 24 bits of h reach the expand)
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
#pragma once
#include "plan_device.h"
#include "wave_ops.h"

namespace mlora {

constexpr int ST_LD = 68;         // padded row stride of a wave's 16 x 64 staging tile, in floats

__device__ __forceinline__ f32x4_t mfma16(const uint4 &a, const uint4 &b, f32x4_t c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

// NS: sites that take the same x and share the workgroup (gate and up of an expert layer).
// DP and ED, what is in flight, are as many as the registers of the kernels' launch bounds hold (128 per lane at four waves
// per SIMD in decode and MoE, 256 at two in prefill): a step of the shrink is RGN + TG 16-byte loads per lane, a block of
// the expand 4 * KC pieces of B and TG of y, and the shrink's registers are free again in the expand.
template <int RP, int NW, int TM, int NS = 1>
struct TileCfg {
    static constexpr int NT = NW * 64;
    static constexpr int RPE = RP < 8 ? 8 : RP;                // ranks as the expand sees them (zeros behind RP)
    static constexpr int RGS = RP < 16 ? 1 : 2;                // groups of eight adapter rows per wave and site
    static constexpr int RGN = NS * RGS;
    static constexpr int RGW = RP <= 16 ? 1 : RP / 16;         // waves side by side over the adapter's rows
    static constexpr int KSW = NW / RGW;                       // waves side by side over d_in
    static constexpr int TG = TM / 8;                          // groups of eight x rows
    static constexpr int DP = TM <= 8 ? (RP <= 16 && NS == 1 ? 6 : 4) : (TM <= 16 ? 4 : (TM <= 32 ? 3 : 2));                // shrink steps in flight per wave
    static constexpr bool K16 = RP <= 16;                      // the expand takes 4 ranks per lane, else 8
    static constexpr int KC = RP <= 32 ? 1 : 2;                // pieces of B per lane and output
    static constexpr int HF = RP < 8 ? 1 : (RP == 8 ? 2 : 3 * KC);    // h operands per 16 rows
    static constexpr int HT = RP <= 8 ? 4 : 3;                 // terms of h
    static constexpr int BW = K16 ? 2 : 4;                     // words of a piece of B
    static constexpr int TH = (TM + 15) / 16;                  // halves of 16 rows in the expand
    static constexpr int ED = TM <= 8 ? (RP < 16 ? 6 : (RP == 16 ? 5 : (RP == 32 ? 4 : 2))) : TM <= 16 ? (RP <= 16 ? 4 : (RP == 32 ? 3 : 2)) : (TM <= 32 && RP <= 32 ? 3 : 2);   // expand blocks in flight per wave
    static constexpr int RT = NS * RPE;                        // ranks of all sites side by side
    static constexpr int H_LD = RT + 8;                        // padded row stride of h in LDS, in elements
    static constexpr int H_BYTES = HT * TH * 16 * H_LD * 2;
    static constexpr int PART_BYTES = KSW * TM * RT * 4, STG_BYTES = NW * 16 * ST_LD * 4;
    static constexpr int LDS = H_BYTES + (PART_BYTES > STG_BYTES ? PART_BYTES : STG_BYTES);
};

// What a tile is made of: the adapter, and for this lane the rows it loads x from and adds y to.
template <int TM>
struct TileRows {
    int key, cnt;
    int xrow[TM / 8];              // row 8 * g + (lane / 2) % 8 of the tile
    int yrow[TM / 8];              // row 8 * g + lane / 8
};

// A tile of a plan from its record, which every lane holds.
template <int TM>
__device__ __forceinline__ bool tile_from_record(const int4 &r, const int32_t *sorted, int top_k, int lane, TileRows<TM> &t)
{
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

template <int TM>
__device__ __forceinline__ bool tile_from_plan(const int4 *tiles, const int32_t *sorted, int top_k, int tile, int lane, TileRows<TM> &t)
{
    return tile_from_record<TM>(tiles[tile], sorted, top_k, lane, t);
}

// A launch whose parts trade partial sums, as a workgroup sees it.
struct TileTrade {
    bool on;                       // this site trades
    int wg;                        // the workgroup's number among the site's
    int parts;                     // workgroups of a tile
    uint32_t tag;                  // the launch tag (thread 0 only)
};

// blk0, n_blk: the blocks of 64 outputs to expand.  XCH: the tile's trade.parts workgroups also divide d_in; each
// publishes the sums of its slice as words (value, launch tag) and adds everybody's in slice order.  A wait
// for a partner's words is bounded: on giving up the workgroup sums all of d_in itself.  A launch tag that says
// so (kTagPoison) makes every part do that without waiting.
// NS = 2: `b2` is the second site; it has a's x, widths, row strides and experts.
// Cache policy (non-temporal: what is touched once leaves the caches to what is not): kStreamY for y where the
// launch's y is far larger than the caches, kStreamAB for adapters of one tile each.  x is never streamed:
// other sites, parts and experts come back for it (with x streamed the packed MoE launch of 64000 pairs took
// 207 instead of 170 us).
constexpr int kStreamY = 1, kStreamAB = 2;
template <bool NT> __device__ __forceinline__ uint4 ld16(const void *p) { if constexpr (NT) return ld_stream(p); else return *(const uint4 *)p; }

template <int RP, int NW, int TM, bool XCH = false, int NS = 1, int CP = 0, bool RB = false>
__device__ __forceinline__ void tile_body(const TileArgs &a, const TileArgs &b2, const TileRows<TM> &t, unsigned char *lds, const int blk0,
                                          const int n_blk, const int tile = 0, const int part_i = 0, const TileTrade &trade = TileTrade{false, 0, 1, 0u})
{
    static_assert(NS == 1 || (!XCH && RP <= 16), "two sites: small ranks, nothing traded");
    using C = TileCfg<RP, NW, TM, NS>;
    uint16_t *const hs = (uint16_t *)lds;                         // [term][row][rank]
    constexpr int H_TERM = C::TH * 16 * C::H_LD;
    float *const part = (float *)(lds + C::H_BYTES);              // [KSW][TM][RT]
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int slot = t.key / a.n_experts;
    const int U = a.d_in >> 3;                                   // 16-byte units per row of x / A

    // ---- shrink: wave w takes adapter rows [16 * (w % RGW), ..) and every KSW-th step of 8 units ----
    const int rgw = w % C::RGW, ksw = w / C::RGW;
    const int lr = (lane >> 1) & 7;
    const int lu = (lane >> 4) * 2 + (lane & 1);
    const int n_steps = (U + 7) >> 3;
    const char *Ag[NS];
    Ag[0] = (const char *)(a.a_tab + (int64_t)t.key * RP * a.d_in);
    if constexpr (NS == 2) Ag[1] = (const char *)(b2.a_tab + (int64_t)t.key * RP * a.d_in);
    const uint32_t row_bytes = (uint32_t)a.d_in * 2u;
    // Rank-bounded reads (slots of different true rank in one padded table): rows of A past the slot's rank are not
    // fetched, their lanes take the last real row again; what they sum meets zero columns of B.
    uint32_t a_off[RB ? NS : 1][C::RGS];
#pragma unroll
    for (int si = 0; si < (RB ? NS : 1); ++si) {
        int a_last = RP - 1;
        if constexpr (RB) a_last = min(max(__builtin_amdgcn_readfirstlane((si ? b2 : a).rank[slot]), 1), RP) - 1;
#pragma unroll
        for (int j = 0; j < C::RGS; ++j) a_off[si][j] = (uint32_t)min(rgw * 16 + j * 8 + lr, a_last) * row_bytes;
    }
    const char *xp[C::TG];
    const bool solo = !XCH || !trade.on;
    __shared__ int s_missing;
    __shared__ uint32_t s_tag;
    // steps [st0, st1) of d_in; this wave's i-th is st0 + ksw + i * KSW
    const int st0 = solo ? 0 : part_i * n_steps / trade.parts, st1 = solo ? n_steps : (part_i + 1) * n_steps / trade.parts;
    const int n = (st1 - st0 - ksw + C::KSW - 1) / C::KSW;
    auto unit_of = [&](int i) { return (st0 + i * C::KSW + ksw) * 8 + lu; };
    uint4 av[C::DP][C::RGN], xv[C::DP][C::TG];
    auto load_a = [&](int i, auto slot_c) __attribute__((always_inline)) {
        constexpr int d = decltype(slot_c)::value;
        const uint32_t u16 = (uint32_t)min(unit_of(i), U - 1) * 16u;
#pragma unroll
        for (int j = 0; j < C::RGN; ++j) av[d][j] = ld16<(CP & kStreamAB) != 0>(Ag[j / C::RGS] + (size_t)(a_off[RB ? j / C::RGS : 0][j % C::RGS] + u16));
    };
    auto load_x = [&](int i, auto slot_c) __attribute__((always_inline)) {
        constexpr int d = decltype(slot_c)::value;
        const uint32_t u16 = (uint32_t)min(unit_of(i), U - 1) * 16u;
#pragma unroll
        for (int g = 0; g < C::TG; ++g) xv[d][g] = *(const uint4 *)(xp[g] + u16);
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
    int rank[NS];
    float scale[NS];

    // ---- the first outputs' B and y travel while the partial sums meet ----
    const int mm = lane & 15, kq = lane >> 4, tr = lane >> 3, og = lane & 7;
    const int nb = (NS * n_blk - w + NW - 1) / NW;               // this wave's blocks of 64 outputs (the sites' one after the other): every NW-th
    const char *Bg[NS];
    char *yg[NS];
    Bg[0] = (const char *)(a.b_tab + (int64_t)t.key * a.d_out * RP);
    yg[0] = (char *)a.y;
    if constexpr (NS == 2) { Bg[1] = (const char *)(b2.b_tab + (int64_t)t.key * a.d_out * RP); yg[1] = (char *)b2.y; }
    int64_t y_off[C::TG];
#pragma unroll
    for (int g = 0; g < C::TG; ++g) y_off[g] = (int64_t)t.yrow[g] * a.ldy * 2;
    // block b of this wave: its site and its first output
    auto site_of = [&](int b) { return NS == 2 && b * NW + w >= n_blk ? 1 : 0; };
    auto out_of = [&](int b) { return (blk0 + b * NW + w - (NS == 2 ? site_of(b) * n_blk : 0)) * 64; };
    uint32_t bv[C::ED][4][C::KC][C::BW];
    uint4 yv[C::ED][C::TG];
    auto fetch = [&](int b, auto buf_c) __attribute__((always_inline)) {
        constexpr int d = decltype(buf_c)::value;
        const int o_w = out_of(b);
        const char *B = NS == 2 && site_of(b) ? Bg[NS - 1] : Bg[0];
        const char *yb = NS == 2 && site_of(b) ? yg[NS - 1] : yg[0];
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
            const uint32_t o = (uint32_t)min(o_w + cb * 16 + mm, a.d_out - 1);
#pragma unroll
            for (int k = 0; k < C::KC; ++k) {
                uint32_t (&v)[C::BW] = bv[d][cb][k];
                if constexpr (RP >= 32) {
                    const uint4 q = *(const uint4 *)(B + (o * (uint32_t)(RP * 2) + (uint32_t)(k * 64 + kq * 16)));
                    v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
                } else if constexpr (RP >= 8) {                     // (rank 8: lane groups 2 and 3 load what 0 and 1 load)
                    const char *src = B + (o * (uint32_t)(RP * 2) + (uint32_t)((RP == 8 ? kq & 1 : kq) * 8));
                    typedef __attribute__((ext_vector_type(2))) unsigned int u32x2_t;
                    const u32x2_t q = (CP & kStreamAB) ? __builtin_nontemporal_load((const u32x2_t *)src) : *(const u32x2_t *)src;
                    v[0] = q.x; v[1] = q.y;
                } else if constexpr (RP == 4) {
                    const uint2 q = *(const uint2 *)(B + o * 8u);
                    v[0] = q.x; v[1] = q.y;
                } else if constexpr (RP == 2) {
                    v[0] = *(const uint32_t *)(B + o * 4u); v[1] = 0u;
                } else {
                    v[0] = *(const uint16_t *)(B + o * 2u); v[1] = 0u;
                }
            }
        }
        const uint32_t oc = (uint32_t)min(o_w + og * 8, a.d_out - 8) * 2u;
#pragma unroll
        for (int g = 0; g < C::TG; ++g) yv[d][g] = ld16<(CP & kStreamY) != 0>(yb + (y_off[g] + oc));
    };
    auto first_fetch = [&]() __attribute__((always_inline)) {
        rank[0] = a.rank[slot];
        scale[0] = a.scale[slot];
        if constexpr (NS == 2) { rank[1] = b2.rank[slot]; scale[1] = b2.scale[slot]; }
        if (nb >= C::ED) static_for<C::ED>([&](auto d) { fetch(d.value, d); });
        else static_for<C::ED>([&](auto d) { if (d.value < nb) fetch(d.value, d); });
    };

    // ---- partial sums of the waves -> h ----
    auto sums_to_lds = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < C::RGN; ++j) {
            const int col = (j / C::RGS) * C::RPE + rgw * 16 + (j % C::RGS) * 8;
#pragma unroll
            for (int g = 0; g < C::TG; ++g) {
                const bool odd = lane & 1;
                float v0 = odd ? acc[j][g][1] : acc[j][g][0], v1 = odd ? acc[j][g][3] : acc[j][g][2];
                v0 += lane_xor<1>(v0);
                v1 += lane_xor<1>(v1);
                // lane (row pair kq of the eight, x row (lane % 16) / 2): even lanes keep the first, odd ones the second
                part[(ksw * TM + g * 8 + (mm >> 1)) * C::RT + col + kq * 2 + (lane & 1)] = odd ? v1 : v0;
            }
        }
        __syncthreads();
    };
    auto own_sum = [&](int e) {
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < C::KSW; ++k) s += part[k * (TM * C::RT) + e];
        return s;
    };
    // h as the sum of three bf16 terms: the bits of its mantissa cut in three, so they add up to h and share its sign.
    // A term with nothing left gets 2^-40 of the first one, an infinity stays one in all of them, and the matrix
    // instruction is given no zero in a term's place: where B is infinite, every product is then the infinity
    // that h * B is, and no 0 * inf or inf - inf makes a NaN of it.
    auto put_h = [&](int e, float s) {
        const int m = e / C::RT, j = e % C::RT;
        s = j % C::RPE < RP ? s * (j < C::RPE ? scale[0] : scale[NS - 1]) : 0.f;
        const bool finite = (__float_as_uint(s) & 0x7f800000u) != 0x7f800000u;
        float left = s;
#pragma unroll
        for (int k = 0; k < C::HT; ++k) {
            if (left == 0.f) left = s * 0x1p-40f;
            const uint32_t b = __float_as_uint(left) & 0xffff0000u;
            hs[k * H_TERM + m * C::H_LD + j] = (uint16_t)(s == s ? b >> 16 : 0x7fc0u);
            if (finite) left -= __uint_as_float(b);
        }
    };
    shrink();
    first_fetch();
    if (XCH && !solo && tid == 0) {                              // (looked at behind the barrier of sums_to_lds)
        s_tag = trade.tag;
        s_missing = 0;
        tag_sign_in(a.ctrl, trade.wg, trade.tag);
    }
    sums_to_lds();
    if (!XCH || solo) {
        for (int e = tid; e < TM * C::RT; e += C::NT) put_h(e, own_sum(e));
    } else {
        const int n_e = t.cnt * C::RPE;                          // rows past the count are nobody's
        uint64_t *const xw = a.xch + (int64_t)tile * trade.parts * (TM * C::RPE);
        const uint32_t tag = __builtin_amdgcn_readfirstlane(s_tag);
        bool gave_up = tag == kTagPoison;
        if (!gave_up)
            for (int e = tid; e < n_e; e += C::NT) xch_put(xw + (int64_t)part_i * (TM * C::RPE) + e, own_sum(e), tag);
        int spins = 0;                                           // (one allowance for all of the thread's words)
        // EB elements at once, W words of each in flight, added in slice order.  (All asked for, past the last part or element its
        // own again: behind a condition each waited for the one before it, 2 us of 16 parts.)
        constexpr int W = 4, EB = TM <= 16 ? 1 : 4;
        for (int e0 = tid; e0 < n_e && !gave_up; e0 += EB * C::NT) {
            float s[EB];
#pragma unroll
            for (int u = 0; u < EB; ++u) s[u] = 0.f;
            for (int p0 = 0; p0 < trade.parts; p0 += W) {
                uint64_t wv[EB][W];
                auto word = [&](int u, int k) __attribute__((always_inline)) { return xw + (int64_t)min(p0 + k, trade.parts - 1) * (TM * C::RPE) + min(e0 + u * C::NT, n_e - 1); };
#pragma unroll
                for (int u = 0; u < EB; ++u)
#pragma unroll
                    for (int k = 0; k < W; ++k) wv[u][k] = xch_get(word(u, k));
#pragma unroll
                for (int u = 0; u < EB; ++u)
#pragma unroll
                    for (int k = 0; k < W; ++k) {
                        if (p0 + k >= trade.parts || gave_up) break;
                        if (p0 + k == part_i) { s[u] += own_sum(min(e0 + u * C::NT, n_e - 1)); continue; }
                        while ((uint32_t)(wv[u][k] >> 32) != tag) {
                            if (++spins > a.poll_limit) { gave_up = true; break; }
                            __builtin_amdgcn_s_sleep(1);
                            wv[u][k] = xch_get(word(u, k));
                        }
                        s[u] += __uint_as_float((uint32_t)wv[u][k]);
                    }
            }
#pragma unroll
            for (int u = 0; u < EB; ++u) if (EB == 1 || e0 + u * C::NT < n_e) put_h(e0 + u * C::NT, s[u]);
        }
        if (gave_up) atomicOr(&s_missing, 1);
        __syncthreads();
        if (s_missing) {
            // Not expected: every element as a plain dot product (slow, but it needs nothing of what is in flight).
            if (tid == 0 && tag != kTagPoison) gave_up_count(a.ctrl);
#pragma unroll
            for (int g = 0; g < C::TG; ++g) {
                for (int e0 = 0; e0 < 8 * C::RPE; e0 += C::NT) {
                    const int e = e0 + tid, m = min(e / C::RPE, 7), j = min(e % C::RPE, RP - 1);
                    const char *xr = (const char *)(a.x + (int64_t)__shfl(t.xrow[g], 2 * m, 64) * a.ldx), *ar = Ag[0] + (size_t)((uint32_t)j * row_bytes);
                    float s = 0.f;
                    for (uint32_t u = 0; u < (uint32_t)U * 16u; u += 16u) s = dot8(*(const uint4 *)(xr + u), *(const uint4 *)(ar + u), s);
                    if (e < 8 * C::RPE) put_h(g * 8 * C::RPE + e, s);
                }
            }
        }
    }
    __syncthreads();
    if (NS == 1 && rank[0] <= 0) return;                         // empty slot: rows stay untouched

    // ---- h as operand: rows m of each half of 16 ----
    // Ranks up to 16 go through 16 x 16 x 16, four ranks of B per lane: a lane group per four ranks and an instruction
    // per term (16); terms 0 and 1 in the groups' two halves, then 2 and 3 (8); every group the same B and a term
    // of its own (below).  (Two terms at once through 16 x 16 x 32 with B twice in a row, and the third through
    // 16 x 16 x 16 behind it: the registers of the second B spilled, and where the two instructions followed
    // each other directly the second did not see the first one's sums.)
    uint4 hv[NS][C::TH][C::HF];
#pragma unroll
    for (int si = 0; si < NS; ++si)
#pragma unroll
    for (int half = 0; half < C::TH; ++half) {
        const uint16_t *ph = hs + (half * 16 + mm) * C::H_LD + si * C::RPE;
        if constexpr (C::K16) {
#pragma unroll
            for (int f = 0; f < C::HF; ++f) {
                const int term = RP == 16 ? f : (RP == 8 ? 2 * f + (kq >> 1) : kq), r0 = RP == 16 ? kq * 4 : (RP == 8 ? (kq & 1) * 4 : 0);
                const uint2 v = *(const uint2 *)(ph + term * H_TERM + r0);
                hv[si][half][f] = make_uint4(v.x, v.y, 0u, 0u);
            }
        } else {
#pragma unroll
            for (int f = 0; f < C::HF; ++f) hv[si][half][f] = *(const uint4 *)(ph + (f % 3) * H_TERM + (f / 3) * 32 + kq * 8);
        }
    }
    // ---- expand: the accumulators pass through a staging tile of the wave so that y moves in row pieces ----
    float *stg = (float *)(lds + C::H_BYTES) + w * (16 * ST_LD);
    auto block = [&](int b, auto buf_c) __attribute__((always_inline)) {
        constexpr int d = decltype(buf_c)::value;
        const int o_w = out_of(b), si = site_of(b);
        if (NS == 2 && (si ? rank[NS - 1] : rank[0]) <= 0) return;   // empty slot at this site
        char *yb = NS == 2 && si ? yg[NS - 1] : yg[0];
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
                    const uint32_t *v = bv[d][cb][C::K16 ? 0 : f / 3];
                    uint4 h = hv[0][half][f];
                    if constexpr (NS == 2) if (si) h = hv[NS - 1][half][f];
                    if constexpr (C::K16)
                        c = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4_t, make_uint2(h.x, h.y)),
                                                                      __builtin_bit_cast(s16x4_t, make_uint2(v[0], v[1])), c, 0, 0, 0);
                    else
                        c = mfma16(h, make_uint4(v[0], v[1], v[2], v[C::BW - 1]), c);
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
                if (half * 16 + trow < t.cnt && col_ok) {
                    if constexpr (CP & kStreamY) st_quiet_stream(yb + (y_off[g] + oc), o);
                    else st_quiet(yb + (y_off[g] + oc), o);
                }
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

}  // namespace mlora
