// Batch grouping kernels: which rows use which adapter.
//
// Dense decode (at most 64 distinct adapters share one decoding step, Section 4 cache-tier
// table) and the packed-MoE route index build (per-expert LoRA tensors keyed by expert id,
// Section 3.4).  All integer work; every output is uniquely determined by the inputs.
#include "plan_device.h"

namespace mlora {

constexpr int kOneRange = 256;     // one-launch route index build: pairs owned by a workgroup
constexpr int kOneKeys = 4096;     // ... largest key space (LDS: three int32 tables of this size, four with tile records)
constexpr int kOnePairs = 32768;   // ... largest batch (each workgroup walks all of it)
constexpr int kOneThreads = 1024;
// ... up to so many pairs a thread takes single ones, beyond whole tokens: 384 pairs, 48 threads of eight LDS adds each before,
// 7.1 -> 6.4 us, 2048 pairs 7.2 -> 6.6; with eight per thread 8000 pairs 8.9 -> 9.3.  (Half of the gain is that all workgroups write the
// group offsets, which the first did alone.)
constexpr int kFewPairs = 2048;
constexpr int kBigRange = 1024;    // three-launch form: items owned by a workgroup
constexpr int kBigKeys = 16384;    // ... largest key space (LDS: two int32 tables of this size)

// Words of ONE count table of the three-launch form (0: such a plan never takes it).
static int64_t plan_big_words(int64_t M, int64_t NK)
{
    if ((M <= kOnePairs && NK <= kOneKeys) || NK > kBigKeys) return 0;
    return ((M + kBigRange - 1) / kBigRange + 1) * NK;
}

// sum over groups of ceil(n_g / tile_rows), at most
int64_t max_tiles(int64_t items, int64_t n_keys, int tile_rows)
{
    const int64_t touched = n_keys < items ? n_keys : items;
    return (items + (tile_rows - 1) * touched) / tile_rows;
}

size_t plan_words(int64_t M, int64_t NK)
{
    return 8 + 3 * (NK + 1) + 4 * M + (kRec + 4) * max_chunks(M, NK) + 64 + 4    // the grouping of the items, its chunk and tile records
         + 8 + 2 * (NK + 1) + 4 * M                                        // the grouping of the tokens (route plans)
         + 2 * plan_big_words(M, NK);
}

PlanView plan_view(void *base, int64_t M, int64_t NK)
{
    PlanView v;
    int32_t *p = (int32_t *)base;
    v.hdr = p;            p += 8;
    v.count = p;          p += NK + 1;
    v.group_off = p;      p += NK + 1;
    v.chunk_base = p;     p += NK + 1;
    v.key_of = p;         p += M;
    v.ticket = p;         p += M;
    v.tmp = p;            p += M;
    v.sorted = p;         p += M;
    v.chunks = p;         p += kRec * max_chunks(M, NK) + 64;
    v.tok_hdr = p;        p += 8;
    v.tok_count = p;      p += NK + 1;
    v.tok_off = p;        p += NK + 1;
    v.tok_key_of = p;     p += M;
    v.tok_ticket = p;     p += M;
    v.tok_tmp = p;        p += M;
    v.tok_sorted = p;     p += M;
    const int64_t bw = plan_big_words(M, NK);
    v.big = bw ? p : nullptr;
    v.tok_big = bw ? p + bw : nullptr;
    p += 2 * bw;
    v.tiles = (int32_t *)(((uintptr_t)p + 15) & ~(uintptr_t)15);
    return v;
}

__global__ void fill_i32_kernel(int32_t *p, int32_t v, int64_t n)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

hipError_t launch_fill_i32(int32_t *p, int32_t v, int64_t n, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    fill_i32_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st>>>(p, v, n);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Small dense batches (up to kSortMax rows) over up to kSmallSlots slots: one workgroup, one row per thread (see
// plan_dense_count).  (The sorting network below, which larger slot tables take, has fifty exchange steps: 8.9
// against 7.9 us for 1001 rows over 64 slots.)
// ---------------------------------------------------------------------------------------------
constexpr int kSmallSlots = 4096;
__global__ __launch_bounds__(kSortMax)
void plan_dense_count_kernel(PlanView pv, const int32_t *__restrict__ token_slot, int T, int n_slots,
                             const int32_t *__restrict__ ready_rank, int rec_bound, int tile_rows, int tile_bound)
{
    __shared__ PlanCountLds<kSmallSlots> lds;
    plan_dense_count<1, kSmallSlots>(pv, token_slot, T, n_slots, ready_rank, rec_bound, tile_rows, tile_bound, (int)threadIdx.x, (int)blockDim.x, lds);
}

// ---------------------------------------------------------------------------------------------
// The same for any number of slots: one workgroup, one key (slot, row) per thread, sorted
// with a bitonic network -- keys are distinct, so the result is the stable sort by slot.  Exchanges
// at distance < 64 stay inside a wave (DPP / swizzle), only the few longer ones go through LDS.
// Group starts and chunk numbers then come from two scans, and the chunk records are written.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(1024)
void plan_dense_small_kernel(PlanView pv, const int32_t *__restrict__ token_slot, int T, int n_slots,
                             const int32_t *__restrict__ ready_rank, int rec_bound, int tile_rows, int tile_bound, int N)
{
    __shared__ uint2 xch[kSortMax + 2];          // long-distance exchanges, then sorted slots / chunk and tile starts
    __shared__ __attribute__((aligned(16))) int32_t wave_tot[16];
    __shared__ int32_t s_rows, s_chunks, s_tiles;
    const int i = threadIdx.x;                   // blockDim.x == N, a power of two in [64, 1024]
    const uint32_t kNone = 0xffffffffu;
    if (i == 0) { s_rows = 0; s_chunks = 0; s_tiles = 0; }
    uint32_t ks = kNone, kt = (uint32_t)i;
    if (i < T) {
        const int s = token_slot[i];
        if (s >= 0 && s < n_slots && !(ready_rank && ready_rank[s] <= 0)) ks = (uint32_t)s;
    }
    BitonicSort<kSortMax>::run(ks, kt, i, N, xch);

    // neighbours' slots through LDS: group starts, number of usable rows
    int32_t *ss = (int32_t *)xch;
    ss[i] = (int32_t)ks;
    __syncthreads();
    const bool live = ks != kNone;
    const bool start = live && (i == 0 || (uint32_t)ss[i - 1] != ks);
    if (live && (i == N - 1 || (uint32_t)ss[i + 1] == kNone)) s_rows = i + 1;
    __syncthreads();
    const int n_rows = s_rows;
    const int gs = block_scan<true>(start ? i : 0, i, N >> 6, wave_tot);
    const int r = i - gs;
    const bool cstart = live && (r % kChunk) == 0;
    const bool tstart = live && tile_rows > 0 && (r % tile_rows) == 0;
    const int both = block_scan<false>((cstart ? 1 : 0) | (tstart ? 0x10000 : 0), i, N >> 6, wave_tot);
    const int c = (both & 0xffff) - 1, tl = (both >> 16) - 1;                       // chunk and tile of this row
    if (live && i == n_rows - 1) { s_chunks = c + 1; s_tiles = tl + 1; }
    int32_t *cs = (int32_t *)xch;                // chunk c starts at sorted position cs[c]
    int32_t *tls = cs + kSortMax + 1;            // tile t at tls[t] (at most kSortMax - 1 of them: tiles have room for kChunk rows)
    __syncthreads();
    const int n_chunks = s_chunks, n_tiles = s_tiles;
    if (cstart) cs[c] = i;
    if (tstart) tls[tl] = i;
    if (i == 0) { cs[n_chunks] = n_rows; tls[n_tiles] = n_rows; }
    __syncthreads();
    if (tstart) ((int4 *)pv.tiles)[tl] = make_int4((int)ks, tls[tl + 1] - i, i, n_tiles);
    if (tile_rows > 0)
        for (int d = n_tiles + i; d < tile_bound; d += N) ((int4 *)pv.tiles)[d] = make_int4(0, 0, 0, n_tiles);
    if (live) {
        pv.sorted[i] = (int32_t)kt;
        int32_t *rec = pv.chunks + (int64_t)c * kRec;
        rec[4 + (r % kChunk)] = (int32_t)kt;
        if (cstart) { rec[0] = (int32_t)ks; rec[1] = cs[c + 1] - cs[c]; rec[2] = i; rec[3] = 0; }
    }
    if (i == 0) { pv.hdr[0] = n_chunks; pv.hdr[1] = n_rows; }
    // records past the live chunks are marked empty (count 0): the apply kernels read only records
    for (int d = n_chunks + i; d < rec_bound; d += N) pv.chunks[(int64_t)d * kRec + 1] = 0;
}

hipError_t launch_plan_dense_small(const PlanView &pv, const int32_t *token_slot, int T, int n_slots,
                                   const int32_t *ready_rank, int tile_rows, hipStream_t st)
{
    int N = 64;
    while (N < T) N <<= 1;
    if (N > kSortMax) return hipErrorInvalidValue;
    if (n_slots <= kSmallSlots) {
        plan_dense_count_kernel<<<dim3(1), dim3((unsigned)(T + 63) / 64 * 64), 0, st>>>(
            pv, token_slot, T, n_slots, ready_rank, (int)max_chunks(T, n_slots), tile_rows,
            tile_rows > 0 ? (int)max_tiles(T, n_slots, tile_rows) : 0);
        return hipGetLastError();
    }
    plan_dense_small_kernel<<<dim3(1), dim3(N), 0, st>>>(pv, token_slot, T, n_slots, ready_rank,
                                                         (int)max_chunks(T, n_slots), tile_rows,
                                                         tile_rows > 0 ? (int)max_tiles(T, n_slots, tile_rows) : 0, N);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// General pipeline (MoE pairs, large dense batches): histogram with tickets, scan, scatter, and
// an in-group rank that restores ascending order, so the result is the stable counting sort.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256)
void plan_hist_kernel(PlanView pv, const int32_t *__restrict__ topk, const int32_t *__restrict__ token_slot,
                      int P, int K, int E, int n_slots, const int32_t *__restrict__ ready_rank)
{
    int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= P) return;
    int t = p / K;
    int s = token_slot[t];
    int e = topk ? topk[p] : 0;
    int key = -1;
    if (s >= 0 && s < n_slots && e >= 0 && e < E && !(ready_rank && ready_rank[s] <= 0)) key = s * E + e;
    pv.key_of[p] = key;
    if (key >= 0) pv.ticket[p] = atomicAdd(&pv.count[key], 1);
}

// One workgroup: exclusive scans of the group sizes and of the per-group chunk counts.
__global__ __launch_bounds__(1024)
void plan_scan_kernel(PlanView pv, int NK, int32_t *__restrict__ out_group_off)
{
    __shared__ __attribute__((aligned(16))) int32_t wave_tot[16];
    const int tid = threadIdx.x;
    const int per = (NK + 1023) / 1024;
    const int lo = min(NK, tid * per), hi = min(NK, lo + per);
    int items = 0, chunks = 0;
    for (int k = lo; k < hi; ++k) {
        int c = pv.count[k];
        items += c;
        chunks += (c + kChunk - 1) / kChunk;
    }
    const int inc_i = block_scan<false>(items, tid, 16, wave_tot);
    const int inc_c = block_scan<false>(chunks, tid, 16, wave_tot);
    int run_i = inc_i - items, run_c = inc_c - chunks;
    for (int k = lo; k < hi; ++k) {
        int c = pv.count[k];
        pv.group_off[k] = run_i;
        if (out_group_off) out_group_off[k] = run_i;
        if (pv.chunk_base) pv.chunk_base[k] = run_c;
        pv.count[k] = 0;                           // leave the histogram clean for the next call
        run_i += c;
        run_c += (c + kChunk - 1) / kChunk;
    }
    if (tid == 1023) {
        pv.group_off[NK] = inc_i;
        if (out_group_off) out_group_off[NK] = inc_i;
        if (pv.chunk_base) pv.chunk_base[NK] = inc_c;
        pv.hdr[0] = inc_c;
        pv.hdr[1] = inc_i;
    }
}

__global__ __launch_bounds__(256)
void plan_scatter_kernel(PlanView pv, int P)
{
    int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= P) return;
    int key = pv.key_of[p];
    if (key >= 0) pv.tmp[pv.group_off[key] + pv.ticket[p]] = p;
}

__global__ __launch_bounds__(256)
void plan_fix_kernel(PlanView pv, int P, int32_t *__restrict__ out_sorted, int rec_bound)
{
    int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= P) return;
    const int n_rows = pv.hdr[1];
    const bool records = pv.chunks != nullptr;            // (the token-level grouping of a route plan has none)
    if (records && j >= pv.hdr[0] && j < rec_bound) pv.chunks[(int64_t)j * kRec + 1] = 0;   // empty record past the live chunks
    if (j >= n_rows) {
        pv.sorted[j] = -1;
        if (out_sorted) out_sorted[j] = -1;
        return;
    }
    int p = pv.tmp[j];
    int key = pv.key_of[p];
    int off = pv.group_off[key], n = pv.group_off[key + 1] - off;
    int r = 0;
    for (int m = 0; m < n; ++m) r += (pv.tmp[off + m] < p);
    pv.sorted[off + r] = p;
    if (out_sorted) out_sorted[off + r] = p;
    if (!records) return;
    int32_t *rec = pv.chunks + (int64_t)(pv.chunk_base[key] + r / kChunk) * kRec;
    rec[4 + (r % kChunk)] = p;
    if (r % kChunk == 0) { rec[0] = key; rec[1] = min(kChunk, n - r); rec[2] = off + r; rec[3] = 0; }
}

// ---------------------------------------------------------------------------------------------
// The same result in one launch, for batches of moderate size (MoE decode / prefill steps of a
// few thousand tokens).  Every workgroup owns kOneRange consecutive pairs and builds, in LDS, the
// histogram of ALL pairs and the histogram of the pairs in front of its range; a scan of the first
// gives the group starts and chunk numbers, the second is the stable rank of the range's first
// member of each group.  Position of pair p = group start + pairs of its key in front of the
// range + pairs of its key in front of it inside the range.  Every workgroup reads all keys
// (P * 4 bytes from L2 each), which is what replaces the three dependent launches and the global
// atomics of the pipeline above; the result is the unique stable counting sort either way.
// ---------------------------------------------------------------------------------------------
// k_magic = ceil(2^32 / K) (0 for K = 1): p / K is then the high word of p * k_magic, exact while
// p * K < 2^32.  A wave instruction takes four cycles on the 16-lane SIMDs, every workgroup walks
// all pairs, and the general division is some forty instructions per pair.
__device__ __forceinline__ int route_key(const int32_t *__restrict__ topk, const int32_t *__restrict__ token_slot,
                                         const int32_t *__restrict__ ready_rank, int p, uint32_t k_magic, int E, int n_slots)
{
    const int s = token_slot[k_magic ? (int)__umulhi((uint32_t)p, k_magic) : p];
    const int e = topk ? topk[p] : 0;
    if (s >= 0 && s < n_slots && e >= 0 && e < E && !(ready_rank && ready_rank[s] <= 0)) return s * E + e;
    return -1;
}

// TILED: tile records too, and with them a fourth LDS table (without it a CU holds one workgroup more).
template <bool TILED>
__device__ __forceinline__
void plan_route_one_body(const PlanView &pv, const int32_t *__restrict__ topk, const int32_t *__restrict__ token_slot,
                         int P, int K, uint32_t k_magic, int E, int n_slots, const int32_t *__restrict__ ready_rank,
                         int32_t *__restrict__ out_sorted, int32_t *__restrict__ out_group_off, int rec_bound, const int block,
                         const int n_blocks, const int tile_rows, const int tile_bound)
{
    __shared__ int32_t tbase[TILED ? kOneKeys + 1 : 1];      // first tile of each group
    __shared__ int32_t goff[kOneKeys + 1];       // exclusive group starts
    __shared__ uint32_t cnt2[kOneKeys];          // per key: pairs in the batch (low half) | pairs in front of this range (high half)
    __shared__ int32_t cbase[kOneKeys + 1];      // first chunk of each group
    __shared__ __attribute__((aligned(16))) int32_t lkey[kOneRange];
    __shared__ int32_t lrank[kOneRange];
    __shared__ __attribute__((aligned(16))) int32_t wave_tot[16];
    static_assert(kOneThreads == 4 * kOneRange, "four threads per pair in the in-range rank");
    static_assert(kOnePairs <= 32768, "two 16-bit counts per word");
    const int tid = threadIdx.x, NK = n_slots * E;
    const int p0 = block * kOneRange;
    const bool records = pv.chunks != nullptr;   // (the token-level grouping of a route plan has none)
    for (int k = tid; k < NK; k += kOneThreads) cnt2[k] = 0u;
    if (tid < kOneRange) lkey[tid] = -1;         // positions past the batch
    __syncthreads();
    // one visit per pair: both counts in one LDS add, and the keys of this range kept
    auto visit = [&](int q, int key) __attribute__((always_inline)) {
        if (key >= 0) atomicAdd(&cnt2[key], q < p0 ? 0x10001u : 1u);
        if (q >= p0 && q < p0 + kOneRange) lkey[q - p0] = key;
    };
    if (topk && K > 1 && P > kFewPairs) {
        // a thread takes whole tokens: the slot (and whether it is ready) once, the token's K experts
        // as 16-byte pieces where K allows -- an eighth of the loads of a pair-by-pair walk at K = 8
        const int T = P / K;
        const bool vec = K <= 16 && !(K & 3) && !((uintptr_t)topk & 15);    // a token's experts as 16-byte pieces
        constexpr int kT = 2;                                   // tokens per thread in flight
        for (int t0 = 0; t0 < T; t0 += kT * kOneThreads) {
            int sl[kT];
            int4 ex[kT][4];
#pragma unroll
            for (int u = 0; u < kT; ++u) {
                const int t = t0 + u * kOneThreads + tid;
                sl[u] = t < T ? token_slot[t] : -1;
                if (t < T && vec) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) if (4 * v < K) ex[u][v] = *(const int4 *)(topk + (int64_t)t * K + 4 * v);
                }
            }
#pragma unroll
            for (int u = 0; u < kT; ++u) {
                const int t = t0 + u * kOneThreads + tid;
                if (t >= T) continue;
                const int s = sl[u];
                const bool ok = s >= 0 && s < n_slots && !(ready_rank && ready_rank[s] <= 0);
                if (vec) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        if (4 * v >= K) break;
                        const int e4[4] = {ex[u][v].x, ex[u][v].y, ex[u][v].z, ex[u][v].w};
#pragma unroll
                        for (int i = 0; i < 4; ++i) visit(t * K + 4 * v + i, ok && e4[i] >= 0 && e4[i] < E ? s * E + e4[i] : -1);
                    }
                } else {
                    for (int k = 0; k < K; ++k) {
                        const int e = topk[(int64_t)t * K + k];
                        visit(t * K + k, ok && e >= 0 && e < E ? s * E + e : -1);
                    }
                }
            }
        }
    } else {
        constexpr int kU = 16;                                  // keys per thread in flight
        if (P <= kFewPairs) {
            int key[kFewPairs / kOneThreads];
#pragma unroll
            for (int u = 0; u < kFewPairs / kOneThreads; ++u) {
                const int q = u * kOneThreads + tid;
                key[u] = q < P ? route_key(topk, token_slot, ready_rank, q, k_magic, E, n_slots) : -1;
            }
#pragma unroll
            for (int u = 0; u < kFewPairs / kOneThreads; ++u) visit(u * kOneThreads + tid, key[u]);
        } else for (int q0 = 0; q0 < P; q0 += kU * kOneThreads) {
            int key[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int q = q0 + u * kOneThreads + tid;
                key[u] = q < P ? route_key(topk, token_slot, ready_rank, q, k_magic, E, n_slots) : -1;
            }
#pragma unroll
            for (int u = 0; u < kU; ++u) visit(q0 + u * kOneThreads + tid, key[u]);
        }
    }
    if (tid < kOneRange) lrank[tid] = 0;
    __syncthreads();
    // Members of the same group in front of a pair inside the range: pair i = tid % 256 against the
    // quarter tid / 256 of the range, four keys per LDS read; the quarters' counts meet in lrank.
    {
        const int i = tid & (kOneRange - 1), m0 = (tid / kOneRange) * (kOneRange / 4);
        const int key = lkey[i];
        int r = 0;
        if (key >= 0) {
#pragma unroll 4
            for (int m = m0; m < m0 + kOneRange / 4; m += 4) {
                const int4 k4 = *(const int4 *)(lkey + m);
                r += (m < i && k4.x == key) + (m + 1 < i && k4.y == key) + (m + 2 < i && k4.z == key) + (m + 3 < i && k4.w == key);
            }
            if (r) atomicAdd(&lrank[i], r);
        }
    }
    // exclusive scans of the group sizes and of the groups' chunk counts: one scan of both, 16 bits
    // each (at most kOnePairs = 2^15 pairs, and no more chunks than pairs)
    const int per = (NK + kOneThreads - 1) / kOneThreads;       // <= 4
    const int lo = min(NK, tid * per), hi = min(NK, lo + per);
    int cnt[kOneKeys / kOneThreads], both = 0;
#pragma unroll
    for (int u = 0; u < kOneKeys / kOneThreads; ++u) {
        cnt[u] = lo + u < hi ? (int)(cnt2[lo + u] & 0xffffu) : 0;
        both += cnt[u] | ((cnt[u] + kChunk - 1) / kChunk) << 16;
    }
    const int inc = block_scan<false>(both, tid, 16, wave_tot);
    const int inc_i = inc & 0xffff, inc_c = (int)((uint32_t)inc >> 16);
    int run_i = inc_i - (both & 0xffff), run_c = inc_c - (int)((uint32_t)both >> 16);
#pragma unroll
    for (int u = 0; u < kOneKeys / kOneThreads; ++u) {
        if (lo + u < hi) {
            goff[lo + u] = run_i;
            cbase[lo + u] = run_c;
            run_i += cnt[u];
            run_c += (cnt[u] + kChunk - 1) / kChunk;
        }
    }
    if (tid == kOneThreads - 1) { goff[NK] = inc_i; cbase[NK] = inc_c; }
    const bool tiled = TILED && records;
    if (tiled) {                                 // (uniform)
        int tiles = 0;
#pragma unroll
        for (int u = 0; u < kOneKeys / kOneThreads; ++u) tiles += (cnt[u] + tile_rows - 1) / tile_rows;
        const int inc_t = block_scan<false>(tiles, tid, 16, wave_tot);
        int run_t = inc_t - tiles;
#pragma unroll
        for (int u = 0; u < kOneKeys / kOneThreads; ++u)
            if (lo + u < hi) { tbase[lo + u] = run_t; run_t += (cnt[u] + tile_rows - 1) / tile_rows; }
        if (tid == kOneThreads - 1) tbase[NK] = inc_t;
    }
    __syncthreads();
    const int n_rows = goff[NK], n_chunks = cbase[NK], n_tiles = tiled ? tbase[NK] : 0;
    // group offsets: each workgroup writes a share
    for (int k = block * kOneThreads + tid; k <= NK; k += n_blocks * kOneThreads) {
        pv.group_off[k] = goff[k];
        if (out_group_off) out_group_off[k] = goff[k];
        if (records) pv.chunk_base[k] = cbase[k];
    }
    if (block == 0 && tid == 0) { pv.hdr[0] = n_chunks; pv.hdr[1] = n_rows; }
    if (tid < kOneRange) {
        const int j = p0 + tid;                  // this range also owns positions / records [p0, p0 + kOneRange)
        if (j < P) {
            if (records && j >= n_chunks && j < rec_bound) pv.chunks[(int64_t)j * kRec + 1] = 0;   // empty record past the live chunks
            if (tiled && j >= n_tiles && j < tile_bound) ((int4 *)pv.tiles)[j] = make_int4(0, 0, 0, n_tiles);
            if (j >= n_rows) {
                pv.sorted[j] = -1;
                if (out_sorted) out_sorted[j] = -1;
            }
            const int key = lkey[tid];
            pv.key_of[j] = key;                      // (the key as this plan saw it: the MoE down projection asks per pair)
            if (key >= 0) {
                const int r = (int)(cnt2[key] >> 16) + lrank[tid];
                const int off = goff[key], n = goff[key + 1] - off;
                pv.sorted[off + r] = j;
                if (out_sorted) out_sorted[off + r] = j;
                if (records) {
                    int32_t *rec = pv.chunks + (int64_t)(cbase[key] + r / kChunk) * kRec;
                    rec[4 + (r % kChunk)] = j;
                    if (r % kChunk == 0) { rec[0] = key; rec[1] = min(kChunk, n - r); rec[2] = off + r; rec[3] = 0; }
                }
                if (tiled && r % tile_rows == 0) ((int4 *)pv.tiles)[tbase[key] + r / tile_rows] = make_int4(key, min(tile_rows, n - r), off + r, n_tiles);
            }
        }
    }
}

// Workgroups [0, pair_blocks) group the routed pairs by (slot, expert); the workgroups behind them
// (route plans only) group the tokens by slot with the same code: key = slot, one item per token.
template <bool TILED>
__global__ __launch_bounds__(kOneThreads)
void plan_route_one_kernel(PlanView pv, const int32_t *__restrict__ topk, const int32_t *__restrict__ token_slot,
                           int P, int K, uint32_t k_magic, int E, int n_slots, const int32_t *__restrict__ ready_rank,
                           int32_t *__restrict__ out_sorted, int32_t *__restrict__ out_group_off, int rec_bound,
                           int pair_blocks, int T, int tile_rows, int tile_bound)
{
    const int b = (int)blockIdx.x;
    if (b < pair_blocks) {
        plan_route_one_body<TILED>(pv, topk, token_slot, P, K, k_magic, E, n_slots, ready_rank, out_sorted, out_group_off, rec_bound, b, pair_blocks, tile_rows, tile_bound);
    } else {
        const PlanView tv = plan_token_view(pv);
        plan_route_one_body<TILED>(tv, nullptr, token_slot, T, 1, 0u, 1, n_slots, ready_rank, nullptr, nullptr, 0, b - pair_blocks, (int)gridDim.x - pair_blocks, 0, 0);
    }
}

// ---------------------------------------------------------------------------------------------
// Large batches (more than kOnePairs items, or more than kOneKeys keys, up to kBigKeys): three launches,
// no global atomics, every step parallel over the batch.
//   count   a workgroup owns kBigRange consecutive items: each one's rank among the range's earlier items
//           of its key (-> ticket), and the range's count of every key (-> a row of the count table).
//           Inside a wave the rank comes from the lanes of equal key, found by one ballot per bit of the keys;
//           the sixteen waves then take turns adding their counts to the LDS table, which keeps the order stable.
//           (Comparing with the wave's 64 keys through LDS, whose broadcast reads of sixteen waves bound the launch: 64000 pairs on 4096
//           keys, all three launches, 18.1 us, now 16.7; 60000 rows on 32 slots 14.3, now 12.4.)
//   scan    per key, an exclusive prefix over the ranges, in place; the totals go to the last row.
//   place   every workgroup scans the totals of all keys (group starts, chunk numbers) and puts its items
//           at  group start + items of the key in earlier ranges + ticket.
// The tokens of a route plan are grouped by slot in further workgroups of the same launches.
// (The pipeline above in its place -- hist with one global atomic per item, one workgroup that scans all
// keys, scatter, and a rank by counting over the whole group, pairs and tokens one after the other, eight
// launches -- took 75 us for 64000 pairs on 4096 keys: groups of several hundred tokens alone 26 us.)
// ---------------------------------------------------------------------------------------------
struct BigSide {                   // one grouping: the pairs, or the tokens
    PlanView pv;
    const int32_t *topk;
    int32_t P, E, NK, blocks;      // items, experts, keys, ranges
    uint32_t k_magic;
};

__global__ __launch_bounds__(kBigRange)
void plan_big_count_kernel(const BigSide pairs, const BigSide toks, const int32_t *__restrict__ token_slot, int n_slots,
                           const int32_t *__restrict__ ready_rank)
{
    __shared__ uint16_t cnt[kBigKeys];
    const bool is_tok = (int)blockIdx.x >= pairs.blocks;
    const BigSide &d = is_tok ? toks : pairs;
    const int block = (int)blockIdx.x - (is_tok ? pairs.blocks : 0);
    const int tid = (int)threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int p = block * kBigRange + tid;
    const int key = p < d.P ? route_key(d.topk, token_slot, ready_rank, p, d.k_magic, d.E, n_slots) : -1;
    for (int k = tid; k < d.NK; k += kBigRange) cnt[k] = 0;
    uint64_t equal = __ballot(key >= 0);
    for (int bit = 0; d.NK - 1 >> bit; ++bit) {
        const bool one = key >> bit & 1;
        const uint64_t ones = __ballot(one);
        equal &= one ? ones : ~ones;
    }
    const int rank = __popcll(equal & (((uint64_t)1 << lane) - 1)), same = __popcll(equal);
    __syncthreads();
    int base = 0;
    for (int v = 0; v < kBigRange / 64; ++v) {
        if (v == w && key >= 0) {
            base = cnt[key];
            if (rank == 0) cnt[key] = (uint16_t)(base + same);
        }
        __syncthreads();
    }
    if (p < d.P) {
        d.pv.key_of[p] = key;
        d.pv.ticket[p] = base + rank;
    }
    int32_t *row = d.pv.big + (int64_t)block * d.NK;
    for (int k = tid; k < d.NK; k += kBigRange) row[k] = cnt[k];
}

// A workgroup takes 64 keys; its sixteen waves divide the ranges, each keeps its part in registers.
constexpr int kScanSeg = 8;        // ranges per wave and pass
__global__ __launch_bounds__(1024)
void plan_big_scan_kernel(const BigSide pairs, const BigSide toks, int pair_blocks)
{
    __shared__ int32_t seg[16][64];
    const bool is_tok = (int)blockIdx.x >= pair_blocks;
    const BigSide &d = is_tok ? toks : pairs;
    const int lane = (int)threadIdx.x & 63, w = (int)threadIdx.x >> 6;
    const int k = ((int)blockIdx.x - (is_tok ? pair_blocks : 0)) * 64 + lane;
    const bool on = k < d.NK;
    int32_t *col = d.pv.big + (on ? k : 0);
    int run = 0;                                 // items of the key in the passes before
    for (int b0 = 0; b0 < d.blocks; b0 += 16 * kScanSeg) {
        const int lo = b0 + w * kScanSeg;
        int c[kScanSeg], sum = 0;
#pragma unroll
        for (int i = 0; i < kScanSeg; ++i) c[i] = lo + i < d.blocks ? col[(int64_t)(lo + i) * d.NK] : 0;
#pragma unroll
        for (int i = 0; i < kScanSeg; ++i) sum += c[i];
        seg[w][lane] = sum;
        __syncthreads();
        int before = run, all = 0;
#pragma unroll
        for (int v = 0; v < 16; ++v) { const int s = seg[v][lane]; before += v < w ? s : 0; all += s; }
        run += all;
#pragma unroll
        for (int i = 0; i < kScanSeg; ++i) {
            if (on && lo + i < d.blocks) col[(int64_t)(lo + i) * d.NK] = before;
            before += c[i];
        }
        __syncthreads();
    }
    if (on && w == 0) col[(int64_t)d.blocks * d.NK] = run;
}

// TILED: tile records too, for half as many keys (a third LDS table).
template <bool TILED>
__global__ __launch_bounds__(kBigRange)
void plan_big_place_kernel(const BigSide pairs, const BigSide toks, int32_t *__restrict__ out_sorted,
                           int32_t *__restrict__ out_group_off, int rec_bound, int tile_rows, int tile_bound)
{
    constexpr int kKeys = TILED ? kBigKeys / 2 : kBigKeys;
    __shared__ int32_t goff[kKeys + 1];
    __shared__ int32_t cbase[kKeys + 1];
    __shared__ int32_t tbase[TILED ? kKeys + 1 : 1];
    __shared__ __attribute__((aligned(16))) int32_t wave_tot[16];
    const bool is_tok = (int)blockIdx.x >= pairs.blocks;
    const BigSide &d = is_tok ? toks : pairs;
    const PlanView &pv = d.pv;
    const int block = (int)blockIdx.x - (is_tok ? pairs.blocks : 0);
    const int tid = (int)threadIdx.x, NK = d.NK;
    const bool records = !is_tok;
    const int j = block * kBigRange + tid;
    // this item's own words travel while the totals are scanned
    const int key = j < d.P ? pv.key_of[j] : -1, ticket = j < d.P ? pv.ticket[j] : 0;
    const int earlier = key >= 0 ? pv.big[(int64_t)block * NK + key] : 0;
    const int32_t *total = pv.big + (int64_t)d.blocks * NK;
    const int per = (NK + kBigRange - 1) / kBigRange;           // <= 16 keys per thread
    const int lo = min(NK, tid * per), hi = min(NK, lo + per);
    constexpr int kPer = kKeys / kBigRange;
    int cnt[kPer], items = 0, chunks = 0;
#pragma unroll
    for (int u = 0; u < kPer; ++u) cnt[u] = lo + u < hi ? total[lo + u] : 0;
#pragma unroll
    for (int u = 0; u < kPer; ++u) { items += cnt[u]; chunks += (cnt[u] + kChunk - 1) / kChunk; }
    const int inc_i = block_scan<false>(items, tid, 16, wave_tot), inc_c = block_scan<false>(chunks, tid, 16, wave_tot);
    int run_i = inc_i - items, run_c = inc_c - chunks;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        if (lo + u < hi) {
            goff[lo + u] = run_i; cbase[lo + u] = run_c;
            run_i += cnt[u];
            run_c += (cnt[u] + kChunk - 1) / kChunk;
        }
    }
    if (tid == kBigRange - 1) { goff[NK] = inc_i; cbase[NK] = inc_c; }
    if constexpr (TILED) {
        int tiles = 0;
#pragma unroll
        for (int u = 0; u < kPer; ++u) tiles += (cnt[u] + tile_rows - 1) / tile_rows;
        const int inc_t = block_scan<false>(tiles, tid, 16, wave_tot);
        int run_t = inc_t - tiles;
#pragma unroll
        for (int u = 0; u < kPer; ++u)
            if (lo + u < hi) { tbase[lo + u] = run_t; run_t += (cnt[u] + tile_rows - 1) / tile_rows; }
        if (tid == kBigRange - 1) tbase[NK] = inc_t;
    }
    __syncthreads();
    const int n_rows = goff[NK], n_chunks = cbase[NK], n_tiles = TILED ? tbase[NK] : 0;
    // group offsets: each workgroup writes a share
    for (int k = block * kBigRange + tid; k <= NK; k += d.blocks * kBigRange) {
        pv.group_off[k] = goff[k];
        if (records) {
            pv.chunk_base[k] = cbase[k];
            if (out_group_off) out_group_off[k] = goff[k];
        }
    }
    if (block == 0 && tid == 0) { pv.hdr[0] = n_chunks; pv.hdr[1] = n_rows; }
    if (j >= d.P) return;
    if (records && j >= n_chunks && j < rec_bound) pv.chunks[(int64_t)j * kRec + 1] = 0;      // empty record past the live chunks
    if (TILED && records && j >= n_tiles && j < tile_bound) ((int4 *)pv.tiles)[j] = make_int4(0, 0, 0, n_tiles);
    if (j >= n_rows) {
        pv.sorted[j] = -1;
        if (records && out_sorted) out_sorted[j] = -1;
    }
    if (key < 0) return;
    const int r = earlier + ticket, off = goff[key], n = goff[key + 1] - off;
    pv.sorted[off + r] = j;
    if (!records) return;
    if (out_sorted) out_sorted[off + r] = j;
    int32_t *rec = pv.chunks + (int64_t)(cbase[key] + r / kChunk) * kRec;
    rec[4 + (r % kChunk)] = j;
    if (r % kChunk == 0) { rec[0] = key; rec[1] = min(kChunk, n - r); rec[2] = off + r; rec[3] = 0; }
    if (TILED && r % tile_rows == 0) ((int4 *)pv.tiles)[tbase[key] + r / tile_rows] = make_int4(key, min(tile_rows, n - r), off + r, n_tiles);
}

bool plan_route_in_one_launch(int64_t P, int64_t NK)
{
    return P <= kOnePairs && NK <= kOneKeys && !tuning(kPlanPipeline);
}

static bool plan_route_in_three_launches(const PlanView &pv, int64_t P, int64_t NK, int K)
{
    return pv.big && NK <= kBigKeys && P * K < ((int64_t)1 << 32) && !tuning(kPlanPipeline);     // (P * K: the bound of k_magic)
}

// Whether a plan of this size can hold tile records (the pipeline writes none).
bool plan_can_tile(const PlanView &pv, int64_t P, int64_t NK, int K)
{
    return plan_route_in_one_launch(P, NK) || (plan_route_in_three_launches(pv, P, NK, K) && NK <= kBigKeys / 2 && P < (1 << 24));
}

hipError_t launch_plan_general(const PlanView &pv, const int32_t *topk, const int32_t *token_slot,
                               int T, int K, int E, int n_slots, const int32_t *ready_rank,
                               int32_t *out_sorted, int32_t *out_group_off, int tile_rows, hipStream_t st)
{
    const int P = T * K, NK = n_slots * E;
    const int tile_bound = tile_rows > 0 ? (int)max_tiles(P, NK, tile_rows) : 0;
    const bool route = topk != nullptr;            // a route plan also groups the tokens by slot
    const uint32_t magic = K > 1 ? (uint32_t)((0x100000000ull + (uint64_t)K - 1) / (uint64_t)K) : 0u;
    if (plan_route_in_one_launch(P, NK)) {
        const int pair_blocks = (P + kOneRange - 1) / kOneRange, tok_blocks = route ? (T + kOneRange - 1) / kOneRange : 0;
        const auto kernel = tile_rows > 0 ? plan_route_one_kernel<true> : plan_route_one_kernel<false>;
        kernel<<<dim3((unsigned)(pair_blocks + tok_blocks)), dim3(kOneThreads), 0, st>>>(
            pv, topk, token_slot, P, K, magic, E, n_slots,
            ready_rank, out_sorted, out_group_off, (int)max_chunks(P, NK), pair_blocks, T, tile_rows, tile_bound);
        return hipGetLastError();
    }
    if (plan_route_in_three_launches(pv, P, NK, K)) {
        const BigSide pairs{pv, topk, P, E, NK, (P + kBigRange - 1) / kBigRange, magic};
        BigSide toks{plan_token_view(pv), nullptr, T, 1, n_slots, route ? (T + kBigRange - 1) / kBigRange : 0, 0u};
        const unsigned nb = (unsigned)(pairs.blocks + toks.blocks);
        const int pair_scans = (NK + 63) / 64, tok_scans = route ? (n_slots + 63) / 64 : 0;
        plan_big_count_kernel<<<dim3(nb), dim3(kBigRange), 0, st>>>(pairs, toks, token_slot, n_slots, ready_rank);
        plan_big_scan_kernel<<<dim3((unsigned)(pair_scans + tok_scans)), dim3(1024), 0, st>>>(pairs, toks, pair_scans);
        if (tile_rows > 0)
            plan_big_place_kernel<true><<<dim3(nb), dim3(kBigRange), 0, st>>>(pairs, toks, out_sorted, out_group_off, (int)max_chunks(P, NK), tile_rows, tile_bound);
        else
            plan_big_place_kernel<false><<<dim3(nb), dim3(kBigRange), 0, st>>>(pairs, toks, out_sorted, out_group_off, (int)max_chunks(P, NK), 0, 0);
        return hipGetLastError();
    }
    const unsigned nb = (unsigned)((P + 255) / 256);
    plan_hist_kernel<<<dim3(nb), dim3(256), 0, st>>>(pv, topk, token_slot, P, K, E, n_slots, ready_rank);
    plan_scan_kernel<<<dim3(1), dim3(1024), 0, st>>>(pv, NK, out_group_off);
    plan_scatter_kernel<<<dim3(nb), dim3(256), 0, st>>>(pv, P);
    plan_fix_kernel<<<dim3(nb), dim3(256), 0, st>>>(pv, P, out_sorted, (int)max_chunks(P, NK));
    if (route) {
        const PlanView tv = plan_token_view(pv);
        const unsigned tb = (unsigned)((T + 255) / 256);
        plan_hist_kernel<<<dim3(tb), dim3(256), 0, st>>>(tv, nullptr, token_slot, T, 1, 1, n_slots, ready_rank);
        plan_scan_kernel<<<dim3(1), dim3(1024), 0, st>>>(tv, n_slots, nullptr);
        plan_scatter_kernel<<<dim3(tb), dim3(256), 0, st>>>(tv, T);
        plan_fix_kernel<<<dim3(tb), dim3(256), 0, st>>>(tv, T, nullptr, 0);
    }
    return hipGetLastError();
}

}  // namespace mlora
