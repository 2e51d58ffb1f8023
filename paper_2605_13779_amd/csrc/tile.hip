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
#include "internal.h"
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
    static constexpr int DP = TM <= 16 ? 4 : (TM <= 32 ? 3 : 2);                // shrink steps in flight per wave
    static constexpr bool K16 = RP <= 16;                      // expand on 16x16x16 (4 ranks per lane), else 16x16x32 (8)
    static constexpr int KC = RP <= 32 ? 1 : 2;                // pieces of B per lane and output
    static constexpr int HF = RP <= 8 ? 1 : 2 * KC;            // h operands per 16 rows
    static constexpr int BW = K16 ? 2 : 4;                     // words of a piece of B
    static constexpr int TH = (TM + 15) / 16;                  // halves of 16 rows in the expand
    static constexpr int ED = TM <= 16 ? (RP <= 16 ? 4 : (RP == 32 ? 3 : 2)) : (TM <= 32 && RP <= 32 ? 3 : 2);   // expand blocks in flight per wave
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

template <int RP, int NW, int TM>
__device__ __forceinline__ void tile_body(const TileArgs &a, const TileRows<TM> &t, unsigned char *lds)
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
    const int lr = (lane >> 1) & 7, lu = (lane >> 4) * 2 + (lane & 1);
    const int n_steps = (U + 7) >> 3, n = (n_steps - ksw + C::KSW - 1) / C::KSW;
    const char *Ag = (const char *)(a.a_tab + (int64_t)t.key * RP * a.d_in);
    const uint32_t row_bytes = (uint32_t)a.d_in * 2u;
    uint32_t a_off[C::RGN];
#pragma unroll
    for (int j = 0; j < C::RGN; ++j) a_off[j] = (uint32_t)min(rgw * 16 + j * 8 + lr, RP - 1) * row_bytes;
    const char *xp[C::TG];
#pragma unroll
    for (int g = 0; g < C::TG; ++g) xp[g] = (const char *)(a.x + (int64_t)t.xrow[g] * a.ldx);
    auto unit_of = [&](int i) { return (min(i, n - 1) * C::KSW + ksw) * 8 + lu; };
    uint4 av[C::DP][C::RGN], xv[C::DP][C::TG];
    auto load = [&](int i, auto slot_c) __attribute__((always_inline)) {
        constexpr int d = decltype(slot_c)::value;
        const uint32_t u16 = (uint32_t)min(unit_of(i), U - 1) * 16u;
#pragma unroll
        for (int j = 0; j < C::RGN; ++j) av[d][j] = *(const uint4 *)(Ag + (size_t)(a_off[j] + u16));
#pragma unroll
        for (int g = 0; g < C::TG; ++g) xv[d][g] = ld_stream(xp[g] + u16);
    };
    f32x4_t acc[C::RGN][C::TG];
#pragma unroll
    for (int j = 0; j < C::RGN; ++j)
#pragma unroll
        for (int g = 0; g < C::TG; ++g) acc[j][g] = f32x4_t{0.f, 0.f, 0.f, 0.f};
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
    if (n > 0) {
        static_for<C::DP>([&](auto d) { load(d.value, d); });
        int i = 0;
        for (; i + C::DP < n; i += C::DP)                            // (the refill past the end repeats the last step: a cache hit)
            static_for<C::DP>([&](auto d) { consume(i + d.value, d); load(i + C::DP + d.value, d); });
        static_for<C::DP>([&](auto d) { if (i + d.value < n) consume(i + d.value, d); });
    }
    const int rank = a.rank[slot];
    const float scale = a.scale[slot];

    // ---- the first outputs' B and y travel while the partial sums meet ----
    const int mm = lane & 15, kq = lane >> 4, tr = lane >> 3, og = lane & 7;
    const int n_blocks = (a.d_out + 63) >> 6, nb = (n_blocks - w + NW - 1) / NW;    // blocks of 64 outputs: every NW-th
    const char *Bg = (const char *)(a.b_tab + (int64_t)t.key * a.d_out * RP);
    char *yp[C::TG];
#pragma unroll
    for (int g = 0; g < C::TG; ++g) yp[g] = (char *)(a.y + (int64_t)t.yrow[g] * a.ldy);
    uint32_t bv[C::ED][4][C::KC][C::BW];
    uint4 yv[C::ED][C::TG];
    auto fetch = [&](int b, auto buf_c) __attribute__((always_inline)) {
        constexpr int d = decltype(buf_c)::value;
        const int o_w = (min(b, nb - 1) * NW + w) * 64;
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
    if (nb > 0) static_for<C::ED>([&](auto d) { fetch(d.value, d); });

    // ---- partial sums of the waves -> h ----
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
    for (int e = tid; e < TM * C::RPE; e += C::NT) {
        const int m = e / C::RPE, j = e % C::RPE;
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < C::KSW; ++k) s += part[k * (TM * C::RPE) + e];
        s = j < RP ? s * scale : 0.f;
        const uint32_t hi = f2bf(s);
        hs_hi[m * C::H_LD + j] = (uint16_t)hi;
        hs_lo[m * C::H_LD + j] = (uint16_t)f2bf(s - __uint_as_float(hi << 16));
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
        const int o_w = (b * NW + w) * 64;
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
    for (; b + C::ED < nb; b += C::ED)
        static_for<C::ED>([&](auto d) { block(b + d.value, d); fetch(b + C::ED + d.value, d); });
    static_for<C::ED>([&](auto d) { if (b + d.value < nb) block(b + d.value, d); });
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
    tile_body<RP, NW, TM>(a, t, lds);
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

int tile_max_rows() { return 48; }

hipError_t launch_tile_seg(const TileArgs &a, int r_pad, const uint32_t *inl, hipStream_t st)
{
    if (a.n_tiles <= 0) return hipSuccess;
    if (a.tile_rows < 1 || a.tile_rows > tile_max_rows() || (!a.segs && 4 * a.n_segs > kTileInline)) return hipErrorInvalidValue;
    switch (r_pad) {
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
