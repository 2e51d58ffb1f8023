// MoE down projection with the routing-weight combine: token by token in one launch where the batch has few pairs per
// adapter (moe_down_token_kernel), else a shrink per chunk or tile of a (slot, expert) group and an expand + combine
// on the matrix cores.
//
// Per-expert LoRA tensors sit on the expert down projection too (Sections 3.4 and 4.4): pair
// p = (t, k) has its own input row and its delta is added, times the routing weight, into the ONE
// output row of token t.  The first launch (one wave per chunk of up to four pairs of a (slot, expert)
// group; ranks above 16 go through the chunk kernels of rows.hip) leaves,
// per pair, the rank-r vector  h[p] = w[p] * (alpha / r) * A_{s,e} x[p]  (fp32 split into a bf16
// head and tail).  What is left is, per slot s,
//
//     Y_s [tokens of s, d_out]  +=  H_s [tokens of s, E * r]  x  Bcat_s [E * r, d_out]
//
// where row t of H_s holds h[(t, k)] in the r columns of expert e(t, k) and zeros elsewhere, and
// Bcat_s stacks the slot's per-expert B tensors along the contraction axis -- exactly how the packed
// tables store them.  That is a dense contraction per slot (H_s is block sparse, but with a few
// tokens per (slot, expert) group nearly every expert's block is touched), so it runs on
// v_mfma_f32_32x32x16_bf16, and it has what the row-by-row form lacks: every output row has ONE
// writer (no fp32 [pairs, d_out] workspace to write and read back, no atomics, a fixed summation
// order), and a slot's B tensors are streamed once per 96 tokens.  Of a contraction step whose experts
// received no pair of the slot no B is fetched, and half chunks of four such steps are skipped, so sparse
// routing pays little for the dense form.
//
// A workgroup owns a tile of up to 96 tokens of one slot and 128 outputs; each of its 4 waves owns
// 32 outputs and streams its rows of B straight from the tables in operand layout (lane = output,
// 8 consecutive ranks: one 16-byte load), half a chunk of 8 contraction steps ahead (see the contraction).  H is never
// written out densely.  The tile's h vectors are fetched once into LDS, split into bf16 head and
// tail in operand layout (K vectors per token, plus one vector of zeros), beside a byte table
// inv[token][expert] = which of the token's K pairs went to that expert (0xff: none).  A lane's
// operand for a contraction step is then one table byte and two 16-byte LDS reads -- the pair's
// vector or the zeros -- so that after the prologue the waves run without a barrier until the
// epilogue.  Ranks below 8 are padded to 8 in the contraction (zeros in both operands; the loads
// fetch the real ranks only).
#include <algorithm>
#include <atomic>
#include <cmath>
#include "plan_device.h"
#include "wave_ops.h"

namespace mlora {

namespace {
constexpr int TN = 128;            // outputs per tile
constexpr int NWD = 4;             // waves: 32 outputs each
constexpr int NTD = NWD * 64;
constexpr int CHK = 128;           // contraction values per chunk (8 steps of 16)
constexpr int NST = CHK / 16;
constexpr int HST = NST / 2;       // steps whose B rows are fetched together
constexpr int KMAX = 16;           // largest top-k (a pair's index fits the table byte)
constexpr int STG_LD = TN + 4;     // padded row stride of the output staging block, in floats
constexpr int kStageBytes = 32 * STG_LD * 4;
constexpr int kLdsTwo = 80 * 1024 - 1024;     // dynamic LDS that leaves room for two workgroups per CU
constexpr int kLdsOne = 160 * 1024 - 2048;    // ... for one

// Where the tile's tables sit in dynamic LDS (byte offsets), for a padded rank rpe >= 8 and tm tokens.
struct DownLayout {
    int n_chunks;      // chunks of the padded contraction axis E * rpe
    int inv_half;      // rank 8: a step holds two experts, one per lane half; odd experts start here in a row
    int inv_ld;        // bytes per token row of inv
    int lo_off, inv_off, live_off, total;
};

__host__ __device__ inline DownLayout down_layout(int rpe, int tm, int K, int E)
{
    DownLayout L;
    L.n_chunks = (E * rpe + CHK - 1) / CHK;
    L.inv_half = rpe == 8 ? L.n_chunks * 8 : 0;
    const int row = L.n_chunks * (CHK / rpe);
    L.inv_ld = ((row + 7) & ~7) + 8;                         // (+8: rows do not start on the same banks)
    const int hb = ((tm * K + 1) * rpe * 2 + 15) & ~15;      // the vectors, one of zeros behind them
    L.lo_off = hb;
    L.inv_off = 2 * hb;
    L.live_off = (L.inv_off + tm * L.inv_ld + 15) & ~15;
    L.total = L.live_off + ((L.n_chunks + 15) & ~15);
    return L;
}

inline int down_dyn_bytes(int rpe, int tm, int K, int E)
{
    const int t = down_layout(rpe, tm, K, E).total;
    return t > kStageBytes ? t : kStageBytes;
}

// 32-row blocks per tile: the most that leaves two workgroups per CU, else the most that fits at all (0: none).
inline int down_blocks(int r_pad, int K, int E)
{
    const int rpe = r_pad < 8 ? 8 : r_pad;
    if ((int64_t)E * rpe > (1 << 21)) return 0;
    for (int mb = 3; mb >= 1; --mb) if (down_dyn_bytes(rpe, 32 * mb, K, E) <= kLdsTwo) return mb;
    for (int mb = 3; mb >= 1; --mb) if (down_dyn_bytes(rpe, 32 * mb, K, E) <= kLdsOne) return mb;
    return 0;
}
}  // namespace

__device__ __forceinline__ f32x16_t mfma32d(const uint4 &a, const uint4 &b, f32x16_t c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

// 16 bytes of B (or the ranks there are) at a byte offset; zeros, and nothing moved, at an offset behind the descriptor's range.
template <int RP>
__device__ __forceinline__ uint4 load_b_or_zero(__amdgpu_buffer_rsrc_t rsrc, uint32_t off)
{
    if constexpr (RP >= 8) return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)off, 0, 0));
    else if constexpr (RP == 4) { const uint2 v = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)off, 0, 0)); return make_uint4(v.x, v.y, 0u, 0u); }
    else if constexpr (RP == 2) return make_uint4(__builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)off, 0, 0), 0u, 0u, 0u);
    else return make_uint4(__builtin_amdgcn_raw_buffer_load_b16(rsrc, (int)off, 0, 0), 0u, 0u, 0u);
}

// SHORT: with a loop of its own for tiles of up to 32 rows (see launch_moe_down_rp).
template <int RP, int MB, bool SHORT>
__global__ __launch_bounds__(NTD, 3)
void moe_down_kernel(const MoeDownArgs a)
{
    constexpr int RPE = RP < 8 ? 8 : RP, TM = 32 * MB;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    __shared__ int32_t tokM[TM];                  // the tile's tokens

    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = (int)blockIdx.x / a.n_ntiles, nt = (int)blockIdx.x - g * a.n_ntiles;

    // ---- which slot, which tile of its tokens: tile g of the list of all slots' tiles (every wave
    //      finds it by itself: 64 slots per step, no barrier) ----
    int s = -1, t_lo = 0, rows = 0, r_s = 0;
    for (int s0 = 0, base = 0; s0 < a.n_slots; s0 += 64) {
        const int si = s0 + lane;
        const int lo = si < a.n_slots ? a.tok_off[si] : 0, hi = si < a.n_slots ? a.tok_off[si + 1] : 0;
        const int r_i = si < a.n_slots ? a.rank[si] : 0;
        const int tiles = (hi - lo + TM - 1) / TM;
        const int inc = wave_scan<false>(tiles), excl = base + inc - tiles;
        const uint64_t hit = __ballot(tiles > 0 && g >= excl && g < excl + tiles);
        if (hit) {
            const int l = __ffsll((long long)hit) - 1;
            s = s0 + l;
            r_s = __shfl(r_i, l, 64);
            t_lo = __shfl(lo, l, 64) + (g - __shfl(excl, l, 64)) * TM;
            rows = min(TM, __shfl(hi, l, 64) - t_lo);
            break;
        }
        base += __shfl(inc, 63, 64);
        if (g < base) break;
    }
    s = __builtin_amdgcn_readfirstlane(s);
    if (s < 0 || __builtin_amdgcn_readfirstlane(r_s) <= 0) return;   // no such tile, or the slot holds no adapter at this site
    t_lo = __builtin_amdgcn_readfirstlane(t_lo);
    rows = __builtin_amdgcn_readfirstlane(rows);

    const int E = a.E, K = a.K;
    const DownLayout L = down_layout(RPE, TM, K, E);
    uint16_t *const hch = (uint16_t *)lds, *const hcl = (uint16_t *)(lds + L.lo_off);
    uint8_t *const inv = lds + L.inv_off, *const live_l = lds + L.live_off;
    const int n_chunks = L.n_chunks, zero_row = TM * K;
    const char *Bs = (const char *)(a.b_tab + (int64_t)s * E * a.d_out * RP);
    const int am = lane & 31, kg = lane >> 5;
    const uint32_t o_b = (uint32_t)min(nt * TN + w * 32 + am, a.d_out - 1);   // this lane's output as B operand

    // (B is read through a descriptor of the slot's tables: a dead step's offset lies behind them and gives zeros)
    const __amdgpu_buffer_rsrc_t b_rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)Bs, 0, (int)((uint32_t)E * (uint32_t)a.d_out * (RP * 2u)), 0x00020000);
    // B rows of one contraction step: ranks [j0, j0 + 8) of expert e (the real ranks when there are fewer)
    auto load_b = [&](int c, int st, bool live) __attribute__((always_inline)) -> uint4 {
        const int kv0 = c * CHK + st * 16 + kg * 8;
        const uint32_t e = (uint32_t)(kv0 / RPE), j0 = (uint32_t)(kv0 % RPE);
        live = live && (int)e < E;
        const uint32_t off = ((e * (uint32_t)a.d_out + o_b) * (uint32_t)RP + (RP >= 8 ? j0 : 0u)) * 2u;
        return load_b_or_zero<RP>(b_rsrc, live ? off : 0xfffffff0u);
    };
    uint4 bq[2][HST];
    auto load_steps_b = [&](int c, int st0, auto bufc, uint32_t mask) __attribute__((always_inline)) {
        constexpr int bi = decltype(bufc)::value;
#pragma unroll
        for (int i = 0; i < HST; ++i) bq[bi][i] = load_b(c, st0 + i, (mask >> (st0 + i) & 1u) != 0);   // (every load is issued: the waits count them)
    };
    auto range_mask = [&](int c) { const int left = E * RPE - c * CHK; return left >= CHK ? 0xffu : (left <= 0 ? 0u : (1u << ((left + 15) >> 4)) - 1u); };

    // ---- the tile's tokens; live contraction steps per chunk (bit st: some expert of step st received
    //      a pair of this slot), from the slot's group offsets; inv cleared ----
    if (tid < TM) tokM[tid] = tid < rows ? a.tok_sorted[t_lo + tid] : -1;
    const int32_t *goff = a.group_off + (int64_t)s * E;
    for (int i0 = w * 64; i0 < n_chunks * NST; i0 += NTD) {
        const int i = i0 + lane, c = i >> 3, st = i & 7;
        bool live = false;
        if (c < n_chunks) {
            const int kv = c * CHK + st * 16;
            const int e0 = kv / RPE, e1 = min(E, (kv + 15) / RPE + 1);
            live = e0 < E && goff[e1] > goff[e0];
        }
        const uint64_t bits = __ballot(live);
        if (st == 0 && c < n_chunks) live_l[c] = (uint8_t)(bits >> (lane & 56));
    }
    load_steps_b(0, 0, IntC<0>{}, range_mask(0));     // on their way while the tile's tables are built
    for (int i = tid; i < TM * L.inv_ld / 8; i += NTD) ((uint2 *)inv)[i] = make_uint2(0xffffffffu, 0xffffffffu);
    if (tid < RPE / 8) { ((uint4 *)(hch + zero_row * RPE))[tid] = make_uint4(0, 0, 0, 0); ((uint4 *)(hcl + zero_row * RPE))[tid] = make_uint4(0, 0, 0, 0); }
    __syncthreads();

    // ---- the tile's pairs: which expert (as the plan saw it) -> inv; the h vector -> head and tail.
    //      Several pairs per thread at a time, so that their loads travel together. ----
    constexpr int NB = RP <= 16 ? 4 : (RP == 32 ? 2 : 1);
    for (int q0 = tid; q0 < TM * K; q0 += NB * NTD) {
        int key[NB];
        uint32_t hv[NB][RP];
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int q = q0 + i * NTD;
            const int t = q < TM * K ? tokM[q / K] : -1;
            key[i] = -1;
            if (t < 0) continue;
            const int64_t p = (int64_t)t * K + (q - (q / K) * K);
            key[i] = a.key_of[p];                                       // (-1: not in the plan)
            const uint32_t *hp = a.h + p * RP;
            if constexpr (RP >= 4) {
#pragma unroll
                for (int u = 0; u < RP / 4; ++u) { const uint4 v = ((const uint4 *)hp)[u]; hv[i][4 * u] = v.x; hv[i][4 * u + 1] = v.y; hv[i][4 * u + 2] = v.z; hv[i][4 * u + 3] = v.w; }
            } else {
#pragma unroll
                for (int j = 0; j < RP; ++j) hv[i][j] = hp[j];
            }
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int q = q0 + i * NTD, m = q / K, k = q - m * K;
            const int e = key[i] - s * E;
            if (key[i] < 0 || e < 0 || e >= E) continue;                // (its vector is never looked at)
            inv[m * L.inv_ld + (RPE == 8 ? (e & 1) * L.inv_half + (e >> 1) : e)] = (uint8_t)k;
            uint16_t *dh = hch + q * RPE, *dl = hcl + q * RPE;
            if constexpr (RP >= 8) {
#pragma unroll
                for (int u = 0; u < RP / 8; ++u) {
                    const uint32_t *v = hv[i] + 8 * u;
                    ((uint4 *)dh)[u] = make_uint4((v[0] & 0xffffu) | (v[1] << 16), (v[2] & 0xffffu) | (v[3] << 16),
                                                  (v[4] & 0xffffu) | (v[5] << 16), (v[6] & 0xffffu) | (v[7] << 16));
                    ((uint4 *)dl)[u] = make_uint4((v[0] >> 16) | (v[1] & 0xffff0000u), (v[2] >> 16) | (v[3] & 0xffff0000u),
                                                  (v[4] >> 16) | (v[5] & 0xffff0000u), (v[6] >> 16) | (v[7] & 0xffff0000u));
                }
            } else {
                uint32_t ph[4] = {0u, 0u, 0u, 0u}, pl[4] = {0u, 0u, 0u, 0u};
#pragma unroll
                for (int j = 0; j < RP; ++j) { ph[j >> 1] |= (hv[i][j] & 0xffffu) << (16 * (j & 1)); pl[j >> 1] |= (hv[i][j] >> 16) << (16 * (j & 1)); }
                *(uint4 *)dh = make_uint4(ph[0], ph[1], ph[2], ph[3]);
                *(uint4 *)dl = make_uint4(pl[0], pl[1], pl[2], pl[3]);
            }
        }
    }
    __syncthreads();

    // ---- the contraction: no barrier from here to the epilogue ----
    f32x16_t acc[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) acc[mb] = f32x16_t{0};
    const uint8_t *inv_lane = inv + am * L.inv_ld + (RPE == 8 ? kg * L.inv_half : 0);
    auto chunk_mask = [&](int c) __attribute__((always_inline)) { return __builtin_amdgcn_readfirstlane(c < n_chunks ? (uint32_t)live_l[c] : 0u); };
    // which of the token's pairs each step's expert is, for this lane's token of every block
    uint64_t sel[MB];
    auto load_sel = [&](int c) __attribute__((always_inline)) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const uint8_t *p = inv_lane + mb * 32 * L.inv_ld;
            if constexpr (RPE <= 16) { const uint2 v = *(const uint2 *)(p + 8 * c); sel[mb] = (uint64_t)v.y << 32 | v.x; }
            else if constexpr (RPE == 32) sel[mb] = *(const uint32_t *)(p + 4 * c);
            else sel[mb] = *(const uint16_t *)(p + 2 * c);
        }
    };
    auto operand = [&](int mb, int st, uint4 &ah, uint4 &al) __attribute__((always_inline)) {
        constexpr int per = RPE <= 16 ? 1 : RPE / 16;                         // steps per expert
        const int j0 = RPE == 8 ? 0 : (RPE == 16 ? kg * 8 : (st % per) * 16 + kg * 8);
        const uint32_t kb = (uint32_t)(sel[mb] >> (8 * (st / per))) & 0xffu;
        const int row = kb == 0xffu ? zero_row : (mb * 32 + am) * K + (int)kb;
        ah = *(const uint4 *)(hch + row * RPE + j0);
        al = *(const uint4 *)(hcl + row * RPE + j0);
    };
    // Half a chunk is straight code, the operands PD (block, step) pairs ahead of the matrix instructions.  With a branch per
    // step and per block the LDS reads of each pair stayed behind it: a workgroup alone on its CU took 20 us for 5 us of
    // matrix instructions.  Rows of B of a dead step are zeros, blocks without a token read the vector of zeros; tiles of up
    // to 32 rows, where that would be two thirds of the work, may have their own loop.  Fetching half a chunk and y only
    // behind the loop leaves 147 registers at rank 8, three workgroups per CU, or 128 and four without that loop (a whole
    // chunk and y in front: 230, two; the loop held to 128 spills 14 and is 4 % slower).  The down call on cold
    // tables, us before / after, 128 experts, top-8, rank 8, 768 -> 2048: 32 slots 2048 tokens 55.7 / 53.4, 4000 76.0 / 65.8, 8000 103.6 /
    // 88.6; 8 slots 512 tokens 28.6 / 23.6, 4000 61.1 / 47.1; 16 slots, rank 16, 8000 tokens 161.8 / 140.5; 8 slots of 64 experts,
    // top-4, rank 64, 1024 -> 2048, 512 tokens 68.0 / 54.6.
    constexpr int PD = 2;
    auto consume = [&](auto nbc, auto st0c, auto bufc, uint32_t mask) __attribute__((always_inline)) {
        constexpr int NB = decltype(nbc)::value, st0 = decltype(st0c)::value, N = HST * NB, bi = decltype(bufc)::value;
        if ((mask >> st0 & ((1u << HST) - 1u)) == 0u) return;
        uint4 ah[PD], al[PD];
        static_for<PD>([&](auto n) { operand(n.value % NB, st0 + n.value / NB, ah[n.value], al[n.value]); });
        static_for<N>([&](auto n) {
            constexpr int mb = n.value % NB, i = n.value / NB, d = n.value % PD;
            acc[mb] = mfma32d(ah[d], bq[bi][i], acc[mb]);
            acc[mb] = mfma32d(al[d], bq[bi][i], acc[mb]);
            if constexpr (n.value + PD < N) operand((n.value + PD) % NB, st0 + (n.value + PD) / NB, ah[d], al[d]);
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    auto contract = [&](auto nbc) __attribute__((always_inline)) {
        uint32_t mask = chunk_mask(0);
        // (the first steps' B were fetched before it was known which of them are dead)
#pragma unroll
        for (int i = 0; i < HST; ++i) if (!(mask >> i & 1u)) bq[0][i] = make_uint4(0, 0, 0, 0);
        for (int c = 0; c < n_chunks; ++c) {
            const uint32_t next = chunk_mask(c + 1);
            load_sel(c);
            load_steps_b(c, HST, IntC<1>{}, mask);
            consume(nbc, IntC<0>{}, IntC<0>{}, mask);
            load_steps_b(c + 1, 0, IntC<0>{}, next);
            consume(nbc, IntC<HST>{}, IntC<1>{}, mask);
            mask = next;
        }
    };
    if (SHORT && rows <= 32) contract(IntC<1>{});
    else contract(IntC<MB>{});

    // ---- this thread's pieces of the tile's y rows (16 bytes each) ----
    constexpr int YP = 32 * (TN / 8) / NTD;                          // pieces per thread and block of 32 rows
    uint4 yv[MB][YP];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int i = 0; i < YP; ++i) {
            const int q = tid + i * NTD, m = mb * 32 + q / (TN / 8), o = nt * TN + (q % (TN / 8)) * 8;
            const int t = tokM[m];
            yv[mb][i] = make_uint4(0, 0, 0, 0);
            if (t >= 0 && o < a.d_out) yv[mb][i] = *(const uint4 *)(a.y + (int64_t)t * a.ldy + o);
        }

    // ---- accumulators -> staging block (the tables are dead) -> y, whole 16-byte row pieces ----
    float *stg = (float *)lds;
    __syncthreads();
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
        if (mb * 32 >= rows) break;
#pragma unroll
        for (int i = 0; i < 16; ++i) stg[((i >> 2) * 8 + kg * 4 + (i & 3)) * STG_LD + w * 32 + am] = acc[mb][i];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < YP; ++i) {
            const int q = tid + i * NTD, m = q / (TN / 8), oc = (q - m * (TN / 8)) * 8, o = nt * TN + oc;
            if (mb * 32 + m >= rows || o >= a.d_out) continue;
            const uint4 y0 = yv[mb][i];
            const float4 d0 = *(const float4 *)(stg + m * STG_LD + oc), d1 = *(const float4 *)(stg + m * STG_LD + oc + 4);
            uint4 out;
            out.x = pack_bf2(bf_lo(y0.x) + d0.x, bf_hi(y0.x) + d0.y);
            out.y = pack_bf2(bf_lo(y0.y) + d0.z, bf_hi(y0.y) + d0.w);
            out.z = pack_bf2(bf_lo(y0.z) + d1.x, bf_hi(y0.z) + d1.y);
            out.w = pack_bf2(bf_lo(y0.w) + d1.z, bf_hi(y0.w) + d1.w);
            *(uint4 *)(a.y + (int64_t)tokM[mb * 32 + m] * a.ldy + o) = out;
        }
        __syncthreads();
    }
}

// First launch for padded ranks up to 16: one wave per chunk record of the plan (up to four pairs of
// one (slot, expert) group, their ids inside the record).  The lanes split d_in in 16-byte units; the
// chunk's x rows go against the adapter's A rows (fp32 sums per lane, one transposing reduction over
// the wave), and pair p's  h = w[p] * (alpha / r) * A x[p]  is left as bf16 head | tail words.  What a
// wave costs is its dependent round trips (record -> rows; a second flight when d_in is above 512);
// with a wave per chunk they all travel at once and the launch runs at the memory system's rate.
// A group of more than four pairs is several neighbouring records, hence neighbouring waves that run
// at the same time and find the adapter's rows in L2 after the first of them.  (One wave per GROUP,
// walking the group's pairs four at a time, came back for A a few microseconds later, when the rows
// had left L2 again: 18 MB of 94 MB fetched at the c4 shapes, 21.3 against 17.5 us.)
// Workgroup b sits on XCD b % 8: two workgroups of an XCD share a run of 8 records.
template <int RP>
__global__ __launch_bounds__(256)
void moe_down_shrink_kernel(const MoeDownArgs a)
{
    constexpr int CB = kChunk, NV = CB * RP;
    static_assert(kChunk == 4 && kRec == 8, "record layout: two 16-byte loads");
    const int lane = (int)threadIdx.x & 63;
    const int b = (int)blockIdx.x, q = b >> 3;
    const int c = __builtin_amdgcn_readfirstlane((((q >> 1) * 8 + (b & 7)) * 2 + (q & 1)) * 4 + ((int)threadIdx.x >> 6));
    if (c >= a.chunk_bound) return;
    const int4 *rec = (const int4 *)(a.chunks + (int64_t)c * kRec);
    const int4 r0 = rec[0], r1 = rec[1];
    const int key = __builtin_amdgcn_readfirstlane(r0.x), cnt = __builtin_amdgcn_readfirstlane(r0.y);
    if (cnt <= 0) return;                                                 // past the live chunks
    int p[CB];
    p[0] = __builtin_amdgcn_readfirstlane(r1.x); p[1] = __builtin_amdgcn_readfirstlane(r1.y);
    p[2] = __builtin_amdgcn_readfirstlane(r1.z); p[3] = __builtin_amdgcn_readfirstlane(r1.w);
#pragma unroll
    for (int i = 1; i < CB; ++i) p[i] = i < cnt ? p[i] : p[0];
    const int U = a.d_in >> 3;
    const int s = key / a.E;
    const uint4 *Ag = (const uint4 *)(a.a_tab + (int64_t)key * RP * a.d_in);
    const uint4 *xp[CB];
#pragma unroll
    for (int i = 0; i < CB; ++i) xp[i] = (const uint4 *)(a.x + (int64_t)p[i] * a.ldx);
    uint4 av[RP], xv[CB];
    auto load_flight = [&](int u0) __attribute__((always_inline)) {
        const int u = u0 + lane, uc = u < U ? u : 0;
#pragma unroll
        for (int j = 0; j < RP; ++j) av[j] = Ag[(int64_t)j * U + uc];
#pragma unroll
        for (int i = 0; i < CB; ++i) if (i < cnt) xv[i] = xp[i][uc];
    };
    load_flight(0);
    const int p_l = lane == 1 ? p[1] : (lane == 2 ? p[2] : (lane == 3 ? p[3] : p[0]));
    const float w_l = lane < cnt ? a.pair_w[p_l] : 0.f;
    const int r_s = a.rank[s];
    const float scale = a.scale[s];
    float acc[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) acc[i] = 0.f;
    for (int u0 = 0; u0 < U; u0 += 64) {
        if (u0 > 0) load_flight(u0);
        const bool in = u0 + lane < U;
#pragma unroll
        for (int i = 0; i < CB; ++i) {
            if (i >= cnt) continue;
            const uint4 xz = in ? xv[i] : make_uint4(0, 0, 0, 0);
#pragma unroll
            for (int j = 0; j < RP; ++j) acc[i * RP + j] = dot8(xz, av[j], acc[i * RP + j]);
        }
    }
    if (r_s <= 0) return;                                                 // the slot holds no adapter at this site
    wave_sum_transpose<NV>(acc, lane);
    const int idx = bitrev<Log2<NV>::v>(lane & (NV - 1)), ci = idx / RP, j = idx - ci * RP;
    const int pc = __shfl(p_l, ci, 64);
    const float wc = __shfl(w_l, ci, 64);
    if (lane < NV && ci < cnt) {
        const float f = acc[0] * scale * wc;
        const uint32_t hi = __float_as_uint(f) & 0xffff0000u;                 // head truncated, tail rounded
        a.h[(int64_t)pc * RP + j] = (hi >> 16) | (f2bf(f - __uint_as_float(hi)) << 16);
    }
}

// The same where the plan holds tiles of 8 or 16 pairs (several pairs per (slot, expert)): one wave per tile, the sums
// on the matrix cores with operands as whole-line loads leave them (lane l: 16 bytes of row (l/2)%8 at piece
// 2*(l/16) + l%2; only products of pieces of equal parity are meant, see tile_body.h).  Bound by what a CU pulls
// through its L1, and a chunk of four pairs pulls the adapter's A once per four
// rows of x.  Expert layer of 8000 tokens (16 pairs per group, rank 8, 768 -> 2048) 296.9 -> 293.0 us, this launch 32.4 us for 150 MB;
// of 2048 tokens (4 per group) 158.7 -> 157.6 us, 17.6 us for 75 MB.
template <int RP, int TG>
__global__ __launch_bounds__(256)
void moe_down_shrink_tile_kernel(const MoeDownArgs a)
{
    constexpr int RG = RP <= 8 ? 1 : 2;            // groups of eight adapter rows
    constexpr int DP = RG + TG <= 3 ? 6 : 4;       // steps of 64 inputs in flight
    const int lane = (int)threadIdx.x & 63;
    const int tile = __builtin_amdgcn_readfirstlane((int)blockIdx.x * 4 + ((int)threadIdx.x >> 6));
    if (tile >= a.n_tiles) return;
    const int4 r = ((const int4 *)a.tiles)[tile];
    const int key = __builtin_amdgcn_readfirstlane(r.x), cnt = __builtin_amdgcn_readfirstlane(r.y);
    if (cnt <= 0) return;                                                 // past the live tiles
    const int32_t *pairs = a.sorted + __builtin_amdgcn_readfirstlane(r.z);
    const int lr = (lane >> 1) & 7, kq = lane >> 4, lu = kq * 2 + (lane & 1);
    const int s = key / a.E, U = a.d_in >> 3, n = (U + 7) >> 3;
    int p[TG];
#pragma unroll
    for (int g = 0; g < TG; ++g) p[g] = pairs[min(8 * g + lr, cnt - 1)];
    const char *Ag = (const char *)(a.a_tab + (int64_t)key * RP * a.d_in);
    uint32_t a_off[RG];
#pragma unroll
    for (int j = 0; j < RG; ++j) a_off[j] = (uint32_t)min(j * 8 + lr, RP - 1) * ((uint32_t)a.d_in * 2u);
    uint4 av[DP][RG], xv[DP][TG];
    const char *xp[TG];
    auto load_a = [&](int i, auto slot_c) __attribute__((always_inline)) {
        constexpr int d = decltype(slot_c)::value;
        const uint32_t u16 = (uint32_t)min(i * 8 + lu, U - 1) * 16u;
#pragma unroll
        for (int j = 0; j < RG; ++j) av[d][j] = *(const uint4 *)(Ag + (size_t)(a_off[j] + u16));
    };
    auto load_x = [&](int i, auto slot_c) __attribute__((always_inline)) {
        constexpr int d = decltype(slot_c)::value;
        const uint32_t u16 = (uint32_t)min(i * 8 + lu, U - 1) * 16u;
#pragma unroll
        for (int g = 0; g < TG; ++g) xv[d][g] = *(const uint4 *)(xp[g] + u16);
    };
    f32x4_t acc[RG][TG];
#pragma unroll
    for (int j = 0; j < RG; ++j)
#pragma unroll
        for (int g = 0; g < TG; ++g) acc[j][g] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    auto consume = [&](int i, auto slot_c) __attribute__((always_inline)) {
        constexpr int d = decltype(slot_c)::value;
        const bool in = i * 8 + lu < U;
#pragma unroll
        for (int g = 0; g < TG; ++g) {
            const uint4 xz = in ? xv[d][g] : make_uint4(0, 0, 0, 0);
#pragma unroll
            for (int j = 0; j < RG; ++j)
                acc[j][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, av[d][j]), __builtin_bit_cast(bf16x8_t, xz), acc[j][g], 0, 0, 0);
        }
    };
    // (A does not depend on the pair ids, which are still on their way)
    static_for<DP>([&](auto d) { if (d.value < n) load_a(d.value, d); });
#pragma unroll
    for (int g = 0; g < TG; ++g) xp[g] = (const char *)(a.x + (int64_t)p[g] * a.ldx);
    static_for<DP>([&](auto d) { if (d.value < n) load_x(d.value, d); });
    float w[TG];
#pragma unroll
    for (int g = 0; g < TG; ++g) w[g] = a.pair_w[p[g]];
    const int r_s = a.rank[s];
    const float scale = a.scale[s];
    int i = 0;
    for (; i + 2 * DP <= n; i += DP)
        static_for<DP>([&](auto d) { consume(i + d.value, d); load_a(i + DP + d.value, d); load_x(i + DP + d.value, d); });
    static_for<DP>([&](auto d) {
        if (i + d.value < n) consume(i + d.value, d);
        if (i + DP + d.value < n) { load_a(i + DP + d.value, d); load_x(i + DP + d.value, d); }
    });
    static_for<DP>([&](auto d) { if (i + DP + d.value < n) consume(i + DP + d.value, d); });
    if (r_s <= 0) return;                                                 // the slot holds no adapter at this site
    const bool odd = lane & 1;
#pragma unroll
    for (int j = 0; j < RG; ++j)
#pragma unroll
        for (int g = 0; g < TG; ++g) {
            float v0 = odd ? acc[j][g][1] : acc[j][g][0], v1 = odd ? acc[j][g][3] : acc[j][g][2];
            v0 += lane_xor<1>(v0);
            v1 += lane_xor<1>(v1);
            const int row = j * 8 + lu;                                   // (2 * kq + parity: even lanes keep the first)
            const float f = (odd ? v1 : v0) * scale * w[g];
            const uint32_t hi = __float_as_uint(f) & 0xffff0000u;         // head truncated, tail rounded
            if (row < RP && 8 * g + lr < cnt) a.h[(int64_t)p[g] * RP + row] = (hi >> 16) | (f2bf(f - __uint_as_float(hi)) << 16);
        }
}

template <int RP>
static void launch_moe_down_shrink_tile(const MoeDownArgs &a, hipStream_t st)
{
    const dim3 grid((unsigned)((a.n_tiles + 3) / 4)), block(256);
    if (a.tile_rows <= 8) moe_down_shrink_tile_kernel<RP, 1><<<grid, block, 0, st>>>(a);
    else moe_down_shrink_tile_kernel<RP, 2><<<grid, block, 0, st>>>(a);
}

// ---------------------------------------------------------------------------------------------------------
// Both halves in one launch, token by token, for batches with few pairs per adapter (decode steps; see
// moe_down_takes_tokens).  A workgroup owns one token and a range of outputs: its waves take the token's pairs,
// h = w * (alpha / r) * A x per pair (dot products, one transposing reduction over the wave) meets in LDS, and a
// thread per output adds the K deltas in fp32, in order of expert id.  Of the plan it needs the pairs' keys only.  It is bound
// by one chain, launch -> keys -> rows of A, x and the first B -> sums -> outputs, where the two launches pay two
// and a dense form whose tiles hold a token or two each.  Parts of a token sum its A again; they sit on one XCD and
// find it in L2.  Expert layers of 128 experts x 32 slots, rank 8, 768 -> 2048, top-8, the down call on cold tables, two
// launches / token by token: 1 token 11.3 / 5.1 us, 48 tokens (17 MB of adapters) 17.6 / 7.0, 200 tokens (72 MB) 27.8 / 15.3.
// (Registers: what is in flight, the rows of A of two pieces and the B rows of eight pairs, is 110 of them at rank 8.
// Held to 128 the kernel spills 83 and the 48 tokens take 13.7 us, so ranks 8 and 16 run one workgroup per CU.)
// ---------------------------------------------------------------------------------------------------------
constexpr int kTokThreads = 512;

// KB: pairs whose B rows are in flight together (K rounded up to 2, 4 or 8; more pairs than that follow in turn).
template <int RP, int KB>
__global__ __launch_bounds__(kTokThreads, RP >= 8 ? 2 : 4)
void moe_down_token_kernel(const MoeDownArgs a, const int parts, const int part_out)
{
    constexpr int NW = kTokThreads / 64;
    constexpr int F = RP <= 8 ? 2 : 1;             // 16-byte units of d_in per lane and flight
    constexpr int BW = (RP + 1) / 2;               // words of an output's B row
    __shared__ float hs[KMAX * RP];
    __shared__ float hp[NW * RP], hw[NW];
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = (int)blockIdx.x >> 3, g8 = q / parts, part = q - g8 * parts, t = g8 * 8 + ((int)blockIdx.x & 7);
    if (t >= a.T) return;
    const int K = a.K;
    const int64_t p0 = (int64_t)t * K;
    const int key_l = lane < K ? a.key_of[p0 + lane] : -1;
    const int key_i = lane >> 3 < K ? a.key_of[p0 + (lane >> 3)] : -1, key_j = (lane & 7) < K ? a.key_of[p0 + (lane & 7)] : -1;
    const float w_l = lane < K ? a.pair_w[p0 + lane] : 0.f;
    const uint32_t valid = (uint32_t)__ballot(key_l >= 0);               // (K <= 16)
    if (valid == 0) return;                                              // the plan left the token out
    const int key_v = __builtin_amdgcn_readlane(key_l, __builtin_ctz(valid)), s = key_v / a.E;      // (a token's pairs share its slot)
    // (a pair that the plan left out, or that the token has not, loads a valid one's rows: every load is issued)
    auto key_at = [&](int k) __attribute__((always_inline)) { const int v = __builtin_amdgcn_readlane(key_l, k); return v < 0 ? key_v : v; };

    // ---- shrink: wave w takes pair w % K and slice w / K of d_in (pairs w, w + 8, .. where K is above 8) ----
    const int n_sl = K < NW ? NW / K : 1, slice = w / K;
    const bool busy = w < (K < NW ? n_sl * K : NW);
    const uint32_t row = (uint32_t)a.d_in * 2u, step = (uint32_t)n_sl * 1024u;
    uint4 av[F][RP], xv[F];
    float acc[RP];
    auto load_ax = [&](int k, uint32_t u0) __attribute__((always_inline)) {
        const char *A = (const char *)(a.a_tab + (int64_t)key_at(k) * RP * a.d_in), *x = (const char *)(a.x + (p0 + k) * a.ldx);
#pragma unroll
        for (int f = 0; f < F; ++f) {
            const uint32_t u = min(u0 + f * step, row - 16u);
#pragma unroll
            for (int j = 0; j < RP; ++j) av[f][j] = *(const uint4 *)(A + (j * row + u));
            xv[f] = *(const uint4 *)(x + u);
        }
    };
    auto dot_ax = [&](uint32_t u0) __attribute__((always_inline)) {
#pragma unroll
        for (int f = 0; f < F; ++f) {
            const uint4 xz = u0 + f * step < row ? xv[f] : make_uint4(0, 0, 0, 0);
#pragma unroll
            for (int j = 0; j < RP; ++j) acc[j] = dot8(xz, av[f][j], acc[j]);
        }
    };
    int key_o;                                     // lane i: the key of the pair that is added i-th
    const int o_lo = part * part_out, o_hi = min(a.d_out, o_lo + part_out);
    uint32_t bv[KB][BW];
    uint16_t yv = 0;
    // (threads past the part's end share its last row of B; y there is another workgroup's to write, and is left alone)
    auto load_b = [&](int o, int kb) __attribute__((always_inline)) {
        const uint32_t ob = (uint32_t)min(o, o_hi - 1) * (uint32_t)(RP * 2);
#pragma unroll
        for (int i = 0; i < KB; ++i) {
            const char *src = (const char *)a.b_tab + (int64_t)__builtin_amdgcn_readlane(key_o, min(kb + i, KMAX - 1)) * a.d_out * (RP * 2) + ob;
            if constexpr (RP >= 8) {
#pragma unroll
                for (int u = 0; u < RP / 8; ++u) { const uint4 v = ((const uint4 *)src)[u]; bv[i][4 * u] = v.x; bv[i][4 * u + 1] = v.y; bv[i][4 * u + 2] = v.z; bv[i][4 * u + 3] = v.w; }
            } else if constexpr (RP == 4) { const uint2 v = *(const uint2 *)src; bv[i][0] = v.x; bv[i][1] = v.y; }
            else if constexpr (RP == 2) bv[i][0] = *(const uint32_t *)src;
            else bv[i][0] = *(const uint16_t *)src;
        }
        if (kb == 0 && o < o_hi) yv = a.y[(int64_t)t * a.ldy + o];
    };
    const uint32_t u_first = (uint32_t)(slice * 64 + lane) * 16u;
    load_ax(w % K, u_first);
    // The deltas are added in order of expert id, and of pairs of one expert the first alone, as in the two launches: lane i
    // takes the pair whose key comes i-th (pairs left out last).  On the way of A's first rows, which take longer; up to
    // eight pairs meet in one comparison, lane 8 * i + j with j-th against i-th key.
    int at = lane, key_once = -1;
    if (K <= 8) {
        const int i = lane >> 3, j = lane & 7;
        const bool twin = key_j == key_i && j < i;
        const uint64_t less = __ballot((uint32_t)key_j < (uint32_t)key_i || twin), twins = __ballot(twin);
        if (lane < 8) {
            at = __popc((uint32_t)(less >> (8 * lane)) & 0xffu);
            if (!((uint32_t)(twins >> (8 * lane)) & 0xffu)) key_once = key_l;
        }
    } else {
        if (lane < K) { at = 0; key_once = key_l; }
        for (int j = 0; j < K; ++j) {
            const int kj = __builtin_amdgcn_readlane(key_l, j);
            const bool twin = kj == key_l && j < lane;
            if (lane < K && ((uint32_t)kj < (uint32_t)key_l || twin)) ++at;
            if (twin) key_once = -1;
        }
    }
    key_o = __builtin_amdgcn_ds_permute(at * 4, key_once);
    const uint32_t added = (uint32_t)__ballot(key_o >= 0);
    if (key_o < 0) key_o = key_v;
    if constexpr (RP <= 8) load_b(o_lo + tid, 0);
    const int r_s = a.rank[s];
    const float scale = a.scale[s];
    for (int k = busy ? w % K : K; k < K; k += NW) {
#pragma unroll
        for (int j = 0; j < RP; ++j) acc[j] = 0.f;
        uint32_t u = u_first;
        if (k != w % K) load_ax(k, u);
        dot_ax(u);
        for (u += F * step; u - (uint32_t)lane * 16u < row; u += F * step) { load_ax(k, u); dot_ax(u); }
        wave_sum_transpose<RP>(acc, lane);
        const float wk = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(w_l), k));
        if (lane < RP) {
            const int j = bitrev<Log2<RP>::v>(lane);
            const int pos = __builtin_amdgcn_readlane(at, k);
            if (n_sl == 1) hs[pos * RP + j] = acc[0] * scale * wk;
            else { hp[(slice * K + pos) * RP + j] = acc[0]; hw[pos] = wk; }
        }
    }
    if constexpr (RP > 8) load_b(o_lo + tid, 0);
    if (r_s <= 0) return;                                                // the slot holds no adapter at this site
    __syncthreads();
    if (n_sl > 1) {
        if (tid < K * RP) {
            const int k = tid / RP, j = tid - k * RP;
            float v = 0.f;
            for (int i = 0; i < n_sl; ++i) v += hp[(i * K + k) * RP + j];
            hs[tid] = v * scale * hw[k];
        }
        __syncthreads();
    }
    // ---- expand: a thread per output ----
    for (int o = o_lo + tid; o - tid < o_hi; o += kTokThreads) {
        float sum = 0.f;
        const uint16_t y0 = yv;
        for (int kb = 0; kb < K; kb += KB) {
            if (kb > 0) load_b(o, kb);
#pragma unroll
            for (int i = 0; i < KB; ++i) {
                if (!(added >> (kb + i) & 1u)) continue;
                const float *h = hs + (kb + i) * RP;
#pragma unroll
                for (int j = 0; j < RP; ++j) sum += h[j] * (j & 1 ? bf_hi(bv[i][j >> 1]) : bf_lo(bv[i][j >> 1]));
            }
        }
        if (o - tid + kTokThreads < o_hi) load_b(o + kTokThreads, 0);
        if (o < o_hi) a.y[(int64_t)t * a.ldy + o] = (uint16_t)f2bf(__uint_as_float((uint32_t)y0 << 16) + sum);
    }
}

// Parts of a token and the outputs of each: one workgroup per CU (48 tokens in 2, 4, 5 and 6 parts: 7.4, 7.5, 7.6 and 10.4 us), at
// least two waves of outputs each.
struct TokenParts { int parts, outs; };
static TokenParts token_parts(int T, int d_out, int cus)
{
    const int want = std::max(1, std::min(cus / T, (d_out + 127) / 128));
    const int outs = ((d_out + want - 1) / want + 63) / 64 * 64;
    return {(d_out + outs - 1) / outs, outs};
}

template <int RP, int KB>
static hipError_t launch_moe_down_token_kb(const MoeDownArgs &a, int cus, hipStream_t st)
{
    const TokenParts p = token_parts(a.T, a.d_out, cus);
    moe_down_token_kernel<RP, KB><<<dim3((unsigned)((a.T + 7) / 8 * 8 * p.parts)), dim3(kTokThreads), 0, st>>>(a, p.parts, p.outs);
    return hipGetLastError();
}

template <int RP>
static hipError_t launch_moe_down_token_rp(const MoeDownArgs &a, int cus, hipStream_t st)
{
    if (a.K <= 2) return launch_moe_down_token_kb<RP, 2>(a, cus, st);
    if (a.K <= 4 || RP == 16) return launch_moe_down_token_kb<RP, 4>(a, cus, st);
    return launch_moe_down_token_kb<RP, (RP == 16 ? 4 : 8)>(a, cus, st);
}

// Whether a down call goes token by token: the estimated time of both forms, in us, fitted to 1960 pairs of calls on cold tables
// (140 sites of ranks 1 to 16, 1 to 128 experts, top-1 to top-12, 1 to 32 slots, 1 to 1000 tokens).  Token by token: a round per workgroup
// that a CU runs at a time (two up to rank 4), a flight of B per 512 outputs, the distinct adapters and, from the caches,
// those of every pair; one chain, so little where tokens are few.  In two launches: two chains, a chunk of the contraction
// after the other, distinct adapters and rows.  Beyond a token per CU the estimate of the rounds is coarser, and the new form
// has to be 8 % ahead.  Over these calls the choice takes 0.6 % more than the better form each time (at most 5 % more
// in 97 of 100; slower than two launches by more than 3 % in 18, at most 1.34 times, 1000 tokens on one expert).  Two launches / token by
// token: 128 experts x 32 slots, top-8, 768 -> 2048, rank 8, 1 token 11.3 / 5.1, 48 17.6 / 7.0, 200 27.8 / 15.3, 300 33.0 / 27.0, 800
// 46.0 / 54.0; rank 16, 100 tokens 23.9 / 13.4, 300 36.6 / 42.5; 16 experts, top-4, rank 8, 1024 -> 4096, 64 tokens 11.0 / 7.5,
// 200 11.6 / 12.3.
bool moe_down_takes_tokens(int T, int K, int E, int n_slots, int r_pad, int d_in, int d_out, int cus)
{
    const int form = tuning(kMoeDownForm);
    if (r_pad > 16 || form < 0) return false;
    if (form > 0) return true;
    if (tuning(kTileMoeRows) > 0) return false;                          // (tiles asked for)
    const TokenParts p = token_parts(T, d_out, cus);
    const int per_cu = r_pad <= 4 ? 2 : 1, chunks = (E * std::max(r_pad, 8) + CHK - 1) / CHK;
    const double rounds = std::ceil((double)T * p.parts / (cus * per_cu)), flights = (p.outs + kTokThreads - 1) / kTokThreads;
    const double pairs = (double)T * K, keys = (double)n_slots * E;
    const double adapter_mb = 2e-6 * r_pad * ((double)d_in + d_out), distinct_mb = adapter_mb * keys * -std::expm1(-pairs / keys);
    const double x_mb = 2e-6 * pairs * d_in, y_mb = 4e-6 * T * d_out;
    const double token = 3.5 + rounds * (1.9 + 0.2 * flights) + 0.115 * distinct_mb + 0.062 * (pairs * adapter_mb + x_mb);
    const double two = 7.3 + 0.8 * chunks + 0.1 * distinct_mb + 0.35 * (x_mb + y_mb) + 1.7e-4 * r_pad * d_in;
    return token < (T <= cus ? 1.0 : 0.92) * two;
}

hipError_t launch_moe_down_token(const MoeDownArgs &a, int cus, hipStream_t st)
{
    if (a.T <= 0) return hipSuccess;
    if (a.K < 1 || a.K > KMAX) return hipErrorInvalidValue;
    switch (a.r_pad) {
        case 1:  return launch_moe_down_token_rp<1>(a, cus, st);
        case 2:  return launch_moe_down_token_rp<2>(a, cus, st);
        case 4:  return launch_moe_down_token_rp<4>(a, cus, st);
        case 8:  return launch_moe_down_token_rp<8>(a, cus, st);
        case 16: return launch_moe_down_token_rp<16>(a, cus, st);
    }
    return hipErrorInvalidValue;
}

bool moe_down_shrinks_by_wave(int r_pad) { return r_pad <= 16; }

hipError_t launch_moe_down_shrink(const MoeDownArgs &a, hipStream_t st)
{
    const int64_t groups = (int64_t)a.n_slots * a.E;
    if (groups <= 0 || a.T <= 0) return hipSuccess;
    if (!a.chunks || a.chunk_bound <= 0) return hipErrorInvalidValue;
    if (a.tiles && a.n_tiles > 0 && a.tile_rows <= 16) {
        switch (a.r_pad) {
            case 2:  launch_moe_down_shrink_tile<2>(a, st); return hipGetLastError();
            case 4:  launch_moe_down_shrink_tile<4>(a, st); return hipGetLastError();
            case 8:  launch_moe_down_shrink_tile<8>(a, st); return hipGetLastError();
            case 16: launch_moe_down_shrink_tile<16>(a, st); return hipGetLastError();
        }
    }
    // 64 records per round of the eight XCDs (two workgroups of four waves each per XCD)
    const dim3 grid((unsigned)(((int64_t)a.chunk_bound + 63) / 64 * 16)), block(256);
    switch (a.r_pad) {
        case 1:  moe_down_shrink_kernel<1><<<grid, block, 0, st>>>(a); break;
        case 2:  moe_down_shrink_kernel<2><<<grid, block, 0, st>>>(a); break;
        case 4:  moe_down_shrink_kernel<4><<<grid, block, 0, st>>>(a); break;
        case 8:  moe_down_shrink_kernel<8><<<grid, block, 0, st>>>(a); break;
        case 16: moe_down_shrink_kernel<16><<<grid, block, 0, st>>>(a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

int moe_down_tile_rows(int r_pad, int K, int E) { return 32 * down_blocks(r_pad, K, E); }
int moe_down_tile_cols() { return TN; }
int moe_down_max_k() { return KMAX; }

template <int RP, int MB, bool SHORT>
static hipError_t launch_moe_down_mb(const MoeDownArgs &a, hipStream_t st)
{
    const int dyn = down_dyn_bytes(RP < 8 ? 8 : RP, 32 * MB, a.K, a.E);
    // (a kernel may use more than 64 KB of dynamic LDS only after this call, per device; devices are few)
    static std::atomic<uint64_t> allowed{0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    if (!(allowed.load(std::memory_order_acquire) >> dev & 1u)) {
        if (hipFuncSetAttribute((const void *)moe_down_kernel<RP, MB, SHORT>, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsOne) != hipSuccess)
            return hipErrorUnknown;
        allowed.fetch_or(1ull << dev, std::memory_order_release);
    }
    const dim3 grid((unsigned)((int64_t)a.n_mtiles * a.n_ntiles)), block(NTD);
    moe_down_kernel<RP, MB, SHORT><<<grid, block, (size_t)dyn, st>>>(a);
    return hipGetLastError();
}

template <int RP>
static hipError_t launch_moe_down_rp(const MoeDownArgs &a, hipStream_t st)
{
    // The loop for short tiles is left out where slots average 112 tokens, so that few tiles are short: up to rank 8, where it costs
    // the fourth workgroup per CU, that gives a few percent, above 8 it is even.  Below, popular slots leave many short
    // tiles behind.  The down call on cold tables with / without it, us, 32 slots of Zipf(1.1) popularity and all alike, top-8, 768 -> 2048:
    // 64 experts, rank 8, 64 tokens per slot 32.0 / 33.7 and 31.8 / 32.0, 94 39.3 / 37.8 and 37.5 / 37.4, 125 44.4 / 41.8 and
    // 44.2 / 42.1, 250 66.7 / 64.7 and 63.1 / 63.3; 128 experts, rank 4, 94 44.3 / 50.2 and 43.7 / 44.1; rank 16, 64 78.1 / 89.9 and
    // 88.7 / 88.9, 94 96.7 / 100.4 and 107.2 / 104.4, 188 145.5 / 143.1 and 138.3 / 135.2.  8 slots of 64 experts, top-4, rank 64, alike, 64
    // 56.1 / 56.2, 125 96.7 / 92.3.
    const bool shorts = a.T < 112 * (int64_t)a.n_slots;
    switch (down_blocks(RP, a.K, a.E)) {
        case 3: return shorts ? launch_moe_down_mb<RP, 3, true>(a, st) : launch_moe_down_mb<RP, 3, false>(a, st);
        case 2: return shorts ? launch_moe_down_mb<RP, 2, true>(a, st) : launch_moe_down_mb<RP, 2, false>(a, st);
        case 1: return launch_moe_down_mb<RP, 1, false>(a, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_moe_down(const MoeDownArgs &a, hipStream_t st)
{
    if (a.T <= 0) return hipSuccess;
    if (a.K > KMAX || a.n_ntiles != (a.d_out + TN - 1) / TN) return hipErrorInvalidValue;
    if ((int64_t)a.E * a.d_out * a.r_pad * 2 >= ((int64_t)1 << 32)) return hipErrorInvalidValue;   // 32-bit offsets inside a slot's B
    switch (a.r_pad) {
        case 1:  return launch_moe_down_rp<1>(a, st);
        case 2:  return launch_moe_down_rp<2>(a, st);
        case 4:  return launch_moe_down_rp<4>(a, st);
        case 8:  return launch_moe_down_rp<8>(a, st);
        case 16: return launch_moe_down_rp<16>(a, st);
        case 32: return launch_moe_down_rp<32>(a, st);
        case 64: return launch_moe_down_rp<64>(a, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace mlora
