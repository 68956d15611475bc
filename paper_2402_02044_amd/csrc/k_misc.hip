// k_misc.hip -- per-query precompute (Sec. 3.2), store maintenance (lazy
// deletes and batched consolidation, App. A), top-k merge, the global mean
// (Sec. 2.3) and k-means for the M-LVQ centres (Sec. 3.2).
#include <float.h>

#include <algorithm>

#include "k_common.h"

namespace lvq {
namespace {

__device__ __forceinline__ float wave_sum_f32(float v)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// ---- query precompute: the query in kernel order, sum(q), <q, mu_m> -------
// One 256-lane workgroup per query; wave w reduces the means w, w+4, ...
__global__ __launch_bounds__(256) void k_prep(PrepArgs a)
{
    const int64_t i = blockIdx.x;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const float *q = reinterpret_cast<const float *>(a.q) + i * a.dim;
    for (int s = tid; s < a.kpos; s += 256) {
        int j = a.kdim[s];
        a.qk[i * a.kpos + s] = j >= 0 ? q[j] : 0.0f;
    }
    if (wave == 0) {
        float s = 0.0f;
        for (int j = lane; j < a.dim; j += 64) s += q[j];
        s = wave_sum_f32(s);
        if (lane == 0) a.qsum[i] = s;
    }
    if (a.metric == LVQ_IP) {
        for (int m = wave; m < a.n_means; m += 4) {
            const float *mu = a.means + (int64_t)m * a.dim;
            float s = 0.0f;
            for (int j = lane; j < a.dim; j += 64) s = fmaf(q[j], mu[j], s);
            s = wave_sum_f32(s);
            if (lane == 0) a.cm[i * a.n_means + m] = s;
        }
    }
}

// The vector scan's queries (see launch_prep_rows): a lane per value below
// tab_blocks, then a wave per (query, four means) for the sums.
__global__ __launch_bounds__(256) void k_prep_rows(PrepArgs a, const float *muk, int tq, int pair_chunk, unsigned tab_blocks,
                                                   int64_t n_tab, uint32_t *gthr)
{
    const float *q = reinterpret_cast<const float *>(a.q);
    if (blockIdx.x < tab_blocks) {
        const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
        if (e >= n_tab) return;
        const int64_t i = e / ((int64_t)a.kpos * tq) * tq + e % tq;
        int p = (int)(e / tq % a.kpos);
        if (pair_chunk) {
            const int r = p % pair_chunk;
            p = p - r + (r & 1) * (pair_chunk / 2) + (r >> 1);
        }
        const int j = a.kdim[p];
        float v = 0.0f;
        if (i < a.nq) {
            if (j >= 0) v = q[i * a.dim + j];
            if (a.metric == LVQ_L2) v -= muk[p];
            if (p == 0) gthr[i] = 0xFFFFFFFFu;
        }
        a.qk[e] = v;
        return;
    }
    const int groups = (a.n_means + 3) / 4, lane = threadIdx.x & 63;
    const int64_t unit = (int64_t)(blockIdx.x - tab_blocks) * 4 + (threadIdx.x >> 6);
    const int64_t i = unit / groups;
    const int m0 = (int)(unit % groups) * 4;
    if (i >= a.nq) return;
    q += i * a.dim;
    if (m0 == 0) {
        float s = 0.0f;
        for (int j = lane; j < a.dim; j += 64) s += q[j];
        s = wave_sum_f32(s);
        if (lane == 0) a.qsum[i] = s;
    }
    for (int m = m0; m < min(m0 + 4, a.n_means); ++m) {
        const float *mu = a.means + (int64_t)m * a.dim;
        float s = 0.0f;
        for (int j = lane; j < a.dim; j += 64) s = fmaf(q[j], mu[j], s);
        s = wave_sum_f32(s);
        if (lane == 0) a.cm[i * a.n_means + m] = s;
    }
}

__global__ void k_fill_i32(int32_t *p, int32_t v, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void k_fill_u32(uint32_t *p, uint32_t v, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// fp32 -> bf16 (upper half, round to nearest even; NaN stays a quiet NaN) or
// fp16 (the hardware conversion, round to nearest even).
__global__ void k_cast16(const float *x, int64_t n, int prec, uint16_t *out)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const float v = x[i];
        uint16_t h;
        if (prec == LVQ_BF16) {
            const uint32_t u = __float_as_uint(v);
            h = (u & 0x7FFFFFFFu) > 0x7F800000u ? (uint16_t)((u >> 16) | 0x40u)
                                                 : (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
        } else {
            const _Float16 f = (_Float16)v;
            h = __builtin_bit_cast(uint16_t, f);
        }
        out[i] = h;
    }
}

// ---- list order for the persistent launch ---------------------------------
// Lists are bucketed by floor(log2(length)), longest bucket first, so the
// work counter hands out long lists before short ones (longest-first
// scheduling).  The order inside a bucket does not affect any result.
// The work counter is reset beside it.
__global__ __launch_bounds__(1024) void k_list_order(const int64_t *offsets, int64_t nq, int32_t *order,
                                                     int32_t *queue)
{
    __shared__ int hist[64];
    __shared__ int base[64];
    const int tid = threadIdx.x;
    if (tid == 0) *queue = 0;
    if (tid < 64) hist[tid] = 0;
    __syncthreads();
    for (int64_t i = tid; i < nq; i += 1024) {
        int64_t len = offsets[i + 1] - offsets[i];
        int b = len > 0 ? 63 - __clzll((unsigned long long)len) : 0;
        atomicAdd(&hist[63 - b], 1);
    }
    __syncthreads();
    if (tid == 0) {
        int acc = 0;
        for (int b = 0; b < 64; ++b) {
            base[b] = acc;
            acc += hist[b];
        }
    }
    __syncthreads();
    for (int64_t i = tid; i < nq; i += 1024) {
        int64_t len = offsets[i + 1] - offsets[i];
        int b = len > 0 ? 63 - __clzll((unsigned long long)len) : 0;
        int pos = atomicAdd(&base[63 - b], 1);
        order[pos] = (int32_t)i;
    }
}

// ---- merge of per-part top-k keys -----------------------------------------
// One workgroup of W waves per query folds the parts' sorted key lists (k
// keys each, kNoKey past the valid ones) into the KS = 64 E >= k smallest,
// kept sorted in registers.  A wave takes every W-th piece: with k <= 64 a
// piece is 64 consecutive keys, whatever lists they belong to, sorted first;
// with more it is one list.  A piece with no key below the wave's k-th best
// is passed over, which after the first few pieces is nearly all of them.
// The waves' lists then meet in LDS, halving the waves each time.  The
// selection this replaces scanned all keys once per result (178 us for 4,096
// queries of 8 parts x 100 keys, 43 us for one query of 246 parts x 10
// keys); this form takes 16 us and 10 us.
template <int E>
__global__ __launch_bounds__(1024) void k_topk_merge(const uint64_t *keys, int n_parts, int k, int metric,
                                                     int32_t *ids, float *dist)
{
    extern __shared__ __align__(16) unsigned char smem[];
    uint64_t *lists = reinterpret_cast<uint64_t *>(smem);   // W x KS, W > 1
    const int64_t qi = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, W = blockDim.x >> 6;
    const int64_t n = (int64_t)n_parts * k;
    const uint64_t *src = keys + qi * n;
    const int piece = E == 1 ? 64 : k;                       // keys per piece
    const int n_pieces = E == 1 ? (int)((n + 63) / 64) : n_parts;
    uint64_t top[E], nx[E];
    auto load = [&](int p) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int i = e * 64 + lane;
            const int64_t at = (int64_t)p * piece + i;
            nx[e] = p < n_pieces && i < piece && at < n ? src[at] : kNoKey;
        }
    };
    auto fold = [&](const uint64_t (&v)[E]) {                // v sorted
        uint64_t r[E];
#pragma unroll
        for (int e = 0; e < E; ++e) r[e] = shfl_u64(v[E - 1 - e], 63 - lane);
#pragma unroll
        for (int e = 0; e < E; ++e) top[e] = min_u64(top[e], r[e]);
        wave_bitonic_merge<E>(top);
    };
    auto kth = [&]() {
        uint64_t b = kNoKey;
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (e == ((k - 1) >> 6)) b = top[e];
        return readlane_u64(b, (k - 1) & 63);
    };
#pragma unroll
    for (int e = 0; e < E; ++e) top[e] = kNoKey;
    uint64_t bound = kNoKey;
    load(wave);
    for (int p = wave; p < n_pieces; p += W) {
        uint64_t v[E];
#pragma unroll
        for (int e = 0; e < E; ++e) v[e] = nx[e];
        load(p + W);
        // (E > 1: a list's smallest key is its first)
        if (!__ballot(v[0] < bound)) continue;
        if constexpr (E == 1) wave_bitonic_sort<1>(v);
        fold(v);
        bound = kth();
    }
    for (int h = W >> 1; h > 0; h >>= 1) {
        if (wave >= h && wave < 2 * h)
#pragma unroll
            for (int e = 0; e < E; ++e) lists[(size_t)wave * 64 * E + e * 64 + lane] = top[e];
        __syncthreads();
        if (wave < h) {
            uint64_t v[E];
#pragma unroll
            for (int e = 0; e < E; ++e) v[e] = lists[(size_t)(wave + h) * 64 * E + e * 64 + lane];
            fold(v);
        }
    }
    if (wave != 0) return;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int i = e * 64 + lane;
        if (i >= k) continue;
        const bool got = top[e] != kNoKey;
        ids[qi * k + i] = got ? (int32_t)(uint32_t)top[e] : -1;
        dist[qi * k + i] = got ? key_score(top[e], metric)
                               : __uint_as_float(metric == LVQ_L2 ? 0x7F800000u : 0xFF800000u);
    }
}

// ---- store maintenance ----------------------------------------------------
__global__ void k_delete(StoreArgs a, const int32_t *slots, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        int32_t s = slots[i];
        if (s < 0 || (int64_t)s >= a.capacity) {
            atomicOr(a.err, kErrBadSlot);
            continue;
        }
        uint8_t *row = a.rows + (int64_t)s * a.row_bytes;
        uint32_t flags = row[13];
        uint32_t *del = reinterpret_cast<uint32_t *>(row + 20);
        if (!(flags & 1u) || *del != kLiveEpoch) {
            atomicOr(a.err, kErrBadSlot);
            continue;
        }
        *del = a.epoch;
    }
}

// Consolidation with the list of occupied slots, in three passes.  Pass 1 reads
// every slot's header once (one sector per slot: what bounds it; 10^6 slots
// take 19 us, 64 MB of sectors) and keeps what the others need as a bit per slot: reclaimable
// (tombstoned at an epoch no running query precedes) and still occupied; it
// counts both per block of 1024 slots.  (Four passes over the headers before:
// 76 us, 35 us now with the scan and the writes.)  Where there is no room for
// the bits (a memory budget), the passes run twice over the headers, for the
// reclaimable and then for the occupied, with one count per block in all.
struct SlotBits {
    uint64_t *gone, *kept;        // a word per 64 slots; NULL: not kept
    int32_t *n_gone, *n_kept;     // a count per 1024; NULL: the other round's
};

__device__ __forceinline__ void slot_state(const StoreArgs &a, int64_t s, uint32_t safe_epoch, bool *gone, bool *kept)
{
    bool used = false;
    *gone = false;
    if (s < a.capacity) {
        const uint8_t *row = a.rows + s * a.row_bytes;
        const uint32_t w = *reinterpret_cast<const uint32_t *>(row + 12);   // mean id, flags
        const uint32_t del = *reinterpret_cast<const uint32_t *>(row + 20);
        used = (w >> 8) & 1u;
        *gone = used && del != kLiveEpoch && del <= safe_epoch;
    }
    *kept = used && !*gone;
}

__global__ __launch_bounds__(1024) void k_consolidate_count(StoreArgs a, uint32_t safe_epoch, SlotBits b)
{
    __shared__ int wsum[2][16];
    const int64_t s = (int64_t)blockIdx.x * 1024 + threadIdx.x;
    bool gone, kept;
    slot_state(a, s, safe_epoch, &gone, &kept);
    const uint64_t mg = __ballot(gone), mk = __ballot(kept);
    if ((threadIdx.x & 63) == 0) {
        const int w = threadIdx.x >> 6;
        if (b.gone && s < a.capacity) {
            b.gone[s >> 6] = mg;
            b.kept[s >> 6] = mk;
        }
        wsum[0][w] = __popcll(mg);
        wsum[1][w] = __popcll(mk);
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        int t = 0;
        for (int w = 0; w < 16; ++w) t += wsum[threadIdx.x][w];
        int32_t *n = threadIdx.x == 0 ? b.n_gone : b.n_kept;
        if (n) n[blockIdx.x] = t;
    }
}

// Exclusive prefix sums of counts[0..nb) in place, in ascending block order
// or (descending) from the last block down; returns the total.  One
// workgroup of 1024 threads: each thread sums a run of blocks, the run
// totals are scanned across the workgroup, then each thread writes its run.
__device__ int64_t block_exclusive_scan(int32_t *counts, int nb, bool descending)
{
    __shared__ int64_t wtot[16];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int per = (nb + 1023) / 1024;
    const int b0 = t * per, b1 = min(nb, b0 + per);
    auto at = [&](int i) -> int32_t & { return counts[descending ? nb - 1 - i : i]; };
    int64_t run = 0;
    for (int i = b0; i < b1; ++i) run += at(i);
    // inclusive scan of run totals within the wave, then across waves
    int64_t inc = run;
    for (int o = 1; o < 64; o <<= 1) {
        const int64_t v = __shfl_up(inc, o, 64);
        if (lane >= o) inc += v;
    }
    if (lane == 63) wtot[wave] = inc;
    __syncthreads();
    int64_t before = 0, total = 0;
    for (int w = 0; w < 16; ++w) {
        if (w < wave) before += wtot[w];
        total += wtot[w];
    }
    int64_t acc = before + inc - run;
    for (int i = b0; i < b1; ++i) {
        const int32_t c = at(i);
        at(i) = (int32_t)acc;
        acc += c;
    }
    return total;
}

// pass 2: exclusive offsets, of the reclaimable in descending block order and of
// the occupied in ascending (a workgroup each); out: new stack top, list length
__global__ __launch_bounds__(1024) void k_consolidate_scan(SlotBits b, int nblocks, int64_t free_top, int64_t *out)
{
    const bool gone = blockIdx.x == 0;
    int32_t *n = gone ? b.n_gone : b.n_kept;
    if (!n) return;
    const int64_t total = block_exclusive_scan(n, nblocks, gone);
    if (threadIdx.x == 0) out[blockIdx.x] = gone ? free_top + total : total;
}

// pass 3: push the reclaimable slots (descending slot order) and clear their
// headers; write the occupied ones in ascending order
template <bool BITS>
__global__ __launch_bounds__(1024) void k_consolidate_write(StoreArgs a, uint32_t safe_epoch, SlotBits b, int32_t *stack,
                                                            int64_t free_top, int32_t *list)
{
    const int64_t s = (int64_t)blockIdx.x * 1024 + threadIdx.x;
    const int lane = threadIdx.x & 63;
    uint64_t mg, mk;
    int above = 0, below = 0;   // in the block's other waves
    if constexpr (BITS) {
        if (s >= a.capacity) return;
        const int64_t w0 = (int64_t)blockIdx.x * 16, w = s >> 6, words = (a.capacity + 63) >> 6;
        mg = b.gone[w];
        mk = b.kept[w];
        if (!(mg | mk)) return;
        for (int64_t v = w0; v < min(words, w0 + 16); ++v) {
            if (v > w) above += __popcll(b.gone[v]);
            if (v < w) below += __popcll(b.kept[v]);
        }
    } else {
        __shared__ int wsum[2][16];
        const int wave = threadIdx.x >> 6;
        bool gone, kept;
        slot_state(a, s, safe_epoch, &gone, &kept);
        mg = __ballot(gone);
        mk = __ballot(kept);
        if (lane == 0) {
            wsum[0][wave] = __popcll(mg);
            wsum[1][wave] = __popcll(mk);
        }
        __syncthreads();
        if (s >= a.capacity) return;
        for (int w = 0; w < 16; ++w) {
            if (w > wave) above += wsum[0][w];
            if (w < wave) below += wsum[1][w];
        }
    }
    above += __popcll(lane == 63 ? 0ull : mg >> (lane + 1));
    below += __popcll(mk & ((1ull << lane) - 1ull));
    if (b.n_gone && ((mg >> lane) & 1)) {
        stack[free_top + b.n_gone[blockIdx.x] + above] = (int32_t)s;
        uint4 *h = reinterpret_cast<uint4 *>(a.rows + s * a.row_bytes);
        h[0] = make_uint4(0u, 0u, 0u, 0u);
        h[1] = make_uint4(0u, 0u, 0u, 0u);
    }
    if (b.n_kept && ((mk >> lane) & 1)) list[b.n_kept[blockIdx.x] + below] = (int32_t)s;
}

__global__ void k_gather_rows(StoreArgs a, const int32_t *slots, int64_t n, uint8_t *rows_out,
                              uint8_t *resid_out)
{
    const int64_t i = blockIdx.x;
    int32_t s = slots[i];
    if (s < 0 || (int64_t)s >= a.capacity) {
        if (threadIdx.x == 0) atomicOr(a.err, kErrBadSlot);
        return;
    }
    const uint32_t *src = reinterpret_cast<const uint32_t *>(a.rows + (int64_t)s * a.row_bytes);
    uint32_t *dst = reinterpret_cast<uint32_t *>(rows_out + i * a.row_bytes);
    for (int w = threadIdx.x; w < a.row_bytes / 4; w += blockDim.x) dst[w] = src[w];
    if (resid_out && a.resid) {
        src = reinterpret_cast<const uint32_t *>(a.resid + (int64_t)s * a.resid_bytes);
        dst = reinterpret_cast<uint32_t *>(resid_out + i * a.resid_bytes);
        for (int w = threadIdx.x; w < a.resid_bytes / 4; w += blockDim.x) dst[w] = src[w];
    }
}

// ---- global mean: binary64 column sums over row chunks, then a fixed-order
// sum of the chunk partials --------------------------------------------------
constexpr int kMeanRows = 4096;

__global__ __launch_bounds__(256) void k_mean_partial(const float *x, int64_t n, int dim, double *part)
{
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= dim) return;
    const int64_t r0 = (int64_t)blockIdx.y * kMeanRows;
    const int64_t r1 = r0 + kMeanRows < n ? r0 + kMeanRows : n;
    double s = 0.0;
    for (int64_t r = r0; r < r1; ++r) s += (double)x[r * dim + j];
    part[(int64_t)blockIdx.y * dim + j] = s;
}

__global__ __launch_bounds__(256) void k_mean_final(const double *part, int nchunks, int64_t n, int dim, float *out)
{
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= dim) return;
    double s = 0.0;
    for (int c = 0; c < nchunks; ++c) s += part[(int64_t)c * dim + j];
    out[j] = (float)(s / (double)n);
}

// ---- k-means ----------------------------------------------------------------
__global__ __launch_bounds__(256) void k_km_assign(const float *x, int64_t n, int dim, const float *c, int k,
                                                   int32_t *assign)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const float *xi = x + i * dim;
    float best = FLT_MAX;
    int bm = 0;
    for (int m = 0; m < k; ++m) {
        const float *cm = c + (int64_t)m * dim;
        float s = 0.0f;
        for (int j = 0; j < dim; ++j) {
            float e = xi[j] - cm[j];
            s = fmaf(e, e, s);
        }
        if (s < best) {
            best = s;
            bm = m;
        }
    }
    assign[i] = bm;
}

// one workgroup per (centre, 256-dim block): binary64 sums in row order
__global__ __launch_bounds__(256) void k_km_update(const float *x, int64_t n, int dim, const int32_t *assign,
                                                   int k, float *c)
{
    const int m = blockIdx.y;
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= dim) return;
    double s = 0.0;
    int64_t cnt = 0;
    for (int64_t i = 0; i < n; ++i)
        if (assign[i] == m) {
            s += (double)x[i * dim + j];
            ++cnt;
        }
    if (cnt > 0) c[(int64_t)m * dim + j] = (float)(s / (double)cnt);
}

// ---- bandwidth probes (measurement): the loads of an access pattern with
// no arithmetic; each lane folds the words it read into one, and each block
// XORs its lanes' words into *sink, so no load can be dropped and the result
// is the XOR of every 32-bit word read.
__device__ __forceinline__ void block_xor_into(uint32_t acc, uint32_t *sink)
{
    __shared__ uint32_t part[4];
    for (int o = 32; o > 0; o >>= 1) acc ^= (uint32_t)__shfl_xor((int)acc, o, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) atomicXor(sink, part[0] ^ part[1] ^ part[2] ^ part[3]);
}

__global__ __launch_bounds__(256) void k_bw_stream(const uint4 *src, int64_t n, uint32_t *sink)
{
    // workgroup b streams the contiguous range [b * chunk, (b + 1) * chunk),
    // eight coalesced 16-byte loads in flight per lane
    const int64_t chunk = (n + gridDim.x - 1) / gridDim.x;
    const int64_t lo = (int64_t)blockIdx.x * chunk;
    const int64_t hi = min(n, lo + chunk);
    uint32_t acc = 0;
    int64_t i = lo + threadIdx.x;
    for (; i + 7 * 256 < hi; i += 8 * 256) {
        uint4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = src[i + u * 256];
#pragma unroll
        for (int u = 0; u < 8; ++u) acc ^= v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
    }
    for (; i < hi; i += 256) {
        const uint4 v = src[i];
        acc ^= v.x ^ v.y ^ v.z ^ v.w;
    }
    block_xor_into(acc, sink);
}

// GL lanes per listed slot (GL in {4, 8, 16}, the smallest covering the
// pieces): the header and first-level code bytes the similarity kernels read
// (code16 pieces of 16 bytes) and, when resid is set, the residual row
// (res16 pieces).
template <int GL>
__global__ __launch_bounds__(256) void k_bw_gather(const uint8_t *rows, int row_bytes, int code16, const uint8_t *resid,
                                                    int resid_bytes, int res16, const int32_t *ids, int64_t n,
                                                    int64_t capacity, uint32_t *sink)
{
    const int g = threadIdx.x % GL;
    const int64_t stride = (int64_t)gridDim.x * (256 / GL);
    uint32_t acc = 0;
    for (int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) / GL; i < n; i += stride) {
        const int32_t s = ids[i];
        if (s < 0 || s >= capacity) continue;
        const uint4 *r = reinterpret_cast<const uint4 *>(rows + (int64_t)s * row_bytes);
        for (int p = g; p < code16; p += GL) {
            const uint4 v = r[p];
            acc ^= v.x ^ v.y ^ v.z ^ v.w;
        }
        if (resid) {
            const uint4 *q = reinterpret_cast<const uint4 *>(resid + (int64_t)s * resid_bytes);
            for (int p = g; p < res16; p += GL) {
                const uint4 v = q[p];
                acc ^= v.x ^ v.y ^ v.z ^ v.w;
            }
        }
    }
    block_xor_into(acc, sink);
}

}  // namespace

hipError_t launch_prep(const PrepArgs &a, hipStream_t s)
{
    if (a.nq <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_prep, dim3((unsigned)a.nq), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_prep_rows(const PrepArgs &a, const float *muk, int tq, int pair_chunk, uint32_t *gthr,
                            hipStream_t s)
{
    if (a.nq <= 0) return hipSuccess;
    const int64_t n_tab = (a.nq + tq - 1) / tq * tq * a.kpos;
    const int64_t tb = (n_tab + 255) / 256;
    const int64_t sb = a.metric == LVQ_IP ? (a.nq * ((a.n_means + 3) / 4) + 3) / 4 : 0;
    hipLaunchKernelGGL(k_prep_rows, dim3((unsigned)(tb + sb)), dim3(256), 0, s, a, muk, tq, pair_chunk, (unsigned)tb,
                       n_tab, gthr);
    return hipGetLastError();
}

static unsigned fill_blocks(int64_t n)
{
    int64_t b = (n + 255) / 256;
    return (unsigned)(b < 4096 ? (b > 0 ? b : 1) : 4096);
}

hipError_t launch_fill_i32(int32_t *p, int32_t v, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_i32, dim3(fill_blocks(n)), dim3(256), 0, s, p, v, n);
    return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t *p, uint32_t v, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_u32, dim3(fill_blocks(n)), dim3(256), 0, s, p, v, n);
    return hipGetLastError();
}

hipError_t launch_bw_stream(const void *src, int64_t n16, uint32_t *sink, hipStream_t s)
{
    hipError_t e = launch_fill_u32(sink, 0u, 1, s);
    if (e != hipSuccess || n16 <= 0) return e;
    hipLaunchKernelGGL(k_bw_stream, dim3(8192), dim3(256), 0, s, reinterpret_cast<const uint4 *>(src), n16, sink);
    return hipGetLastError();
}

hipError_t launch_bw_gather(const uint8_t *rows, int row_bytes, int code16, const uint8_t *resid, int resid_bytes,
                            int res16, const int32_t *ids, int64_t n, int64_t capacity, uint32_t *sink, hipStream_t s)
{
    hipError_t e = launch_fill_u32(sink, 0u, 1, s);
    if (e != hipSuccess || n <= 0) return e;
    const int pieces = std::max(code16, resid ? res16 : 0);
    const int gl = pieces > 8 ? 16 : (pieces > 4 ? 8 : 4);
    const int64_t blocks = std::min<int64_t>((n * gl + 255) / 256, 16384);
    auto kern = gl == 16 ? k_bw_gather<16> : (gl == 8 ? k_bw_gather<8> : k_bw_gather<4>);
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), 0, s, rows, row_bytes, code16, resid, resid_bytes,
                       res16, ids, n, capacity, sink);
    return hipGetLastError();
}

hipError_t launch_cast16(const float *x, int64_t n, int prec, void *out, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_cast16, dim3(fill_blocks(n)), dim3(256), 0, s, x, n, prec, reinterpret_cast<uint16_t *>(out));
    return hipGetLastError();
}

hipError_t launch_list_order(const int64_t *offsets, int64_t nq, int32_t *order, int32_t *queue, hipStream_t s)
{
    if (nq <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_list_order, dim3(1), dim3(1024), 0, s, offsets, nq, order, queue);
    return hipGetLastError();
}

hipError_t launch_topk_merge(const uint64_t *keys, int64_t nq, int n_parts, int k, int metric, int32_t *ids,
                             float *dist, hipStream_t s)
{
    if (nq <= 0) return hipSuccess;
    if (k < 1 || k > kMaxTopK || n_parts < 1) return hipErrorInvalidValue;
    int E = 1;
    while (64 * E < k) E *= 2;
    // waves per query: while each has two pieces to fold and the batch leaves
    // wave slots idle (a full chip holds 8,192 waves; the halving steps cost
    // about two pieces each), within 64 KB of LDS
    const int64_t pieces = E == 1 ? ((int64_t)n_parts * k + 63) / 64 : n_parts;
    int W = 1;
    while (W < 16 && 4 * W <= pieces && nq * W < 2048 && (size_t)2 * W * 64 * E * sizeof(uint64_t) <= 65536) W *= 2;
    const size_t lds = W > 1 ? (size_t)W * 64 * E * sizeof(uint64_t) : 0;
    auto kern = E == 1 ? k_topk_merge<1> : E == 2 ? k_topk_merge<2> : E == 4 ? k_topk_merge<4>
              : E == 8 ? k_topk_merge<8> : k_topk_merge<16>;
    hipLaunchKernelGGL(kern, dim3((unsigned)nq), dim3(64 * W), lds, s, keys, n_parts, k, metric, ids, dist);
    return hipGetLastError();
}

hipError_t launch_delete(const StoreArgs &a, const int32_t *slots, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_delete, dim3(fill_blocks(n)), dim3(256), 0, s, a, slots, n);
    return hipGetLastError();
}

size_t consolidate_scratch(int64_t capacity, bool bits)
{
    const size_t words = (size_t)(capacity + 63) / 64, nb = (size_t)(capacity + 1023) / 1024;
    return bits ? 2 * words * sizeof(uint64_t) + 2 * nb * sizeof(int32_t) : nb * sizeof(int32_t);
}

hipError_t launch_consolidate(const StoreArgs &a, uint32_t safe_epoch, int32_t *free_stack, int64_t free_top,
                              int32_t *list, void *scratch, bool bits, int64_t *out, hipStream_t s)
{
    const int nb = (int)((a.capacity + 1023) / 1024);
    if (nb == 0) return hipSuccess;
    auto passes = [&](const SlotBits &b) {
        hipLaunchKernelGGL(k_consolidate_count, dim3(nb), dim3(1024), 0, s, a, safe_epoch, b);
        hipLaunchKernelGGL(k_consolidate_scan, dim3(2), dim3(1024), 0, s, b, nb, free_top, out);
        hipLaunchKernelGGL(b.gone ? k_consolidate_write<true> : k_consolidate_write<false>, dim3(nb), dim3(1024), 0, s,
                           a, safe_epoch, b, free_stack, free_top, list);
        return hipGetLastError();
    };
    if (bits) {
        const size_t words = (size_t)(a.capacity + 63) / 64;
        SlotBits b;
        b.gone = reinterpret_cast<uint64_t *>(scratch);
        b.kept = b.gone + words;
        b.n_gone = reinterpret_cast<int32_t *>(b.kept + words);
        b.n_kept = b.n_gone + nb;
        return passes(b);
    }
    int32_t *counts = reinterpret_cast<int32_t *>(scratch);
    const hipError_t e = passes({nullptr, nullptr, counts, nullptr});
    return e != hipSuccess ? e : passes({nullptr, nullptr, nullptr, counts});
}

hipError_t launch_gather_rows(const StoreArgs &a, const int32_t *slots, int64_t n, uint8_t *rows_out,
                              uint8_t *resid_out, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_gather_rows, dim3((unsigned)n), dim3(64), 0, s, a, slots, n, rows_out, resid_out);
    return hipGetLastError();
}

hipError_t launch_mean(const float *x, int64_t n, int dim, float *out, double *scratch, hipStream_t s)
{
    const int nchunks = (int)((n + kMeanRows - 1) / kMeanRows);
    dim3 g1((dim + 255) / 256, nchunks);
    hipLaunchKernelGGL(k_mean_partial, g1, dim3(256), 0, s, x, n, dim, scratch);
    hipLaunchKernelGGL(k_mean_final, dim3((dim + 255) / 256), dim3(256), 0, s, scratch, nchunks, n, dim, out);
    return hipGetLastError();
}

hipError_t launch_kmeans_assign(const float *x, int64_t n, int dim, const float *c, int k, int32_t *assign,
                                hipStream_t s)
{
    hipLaunchKernelGGL(k_km_assign, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, x, n, dim, c, k, assign);
    return hipGetLastError();
}

hipError_t launch_kmeans_update(const float *x, int64_t n, int dim, const int32_t *assign, int k, float *c,
                                hipStream_t s)
{
    hipLaunchKernelGGL(k_km_update, dim3((dim + 255) / 256, k), dim3(256), 0, s, x, n, dim, assign, k, c);
    return hipGetLastError();
}

}  // namespace lvq

#include "k_cand_inst.h"
#include "k_scan_impl.h"

namespace lvq {

int num_tile_shapes() { return kNumCandShapes; }
TileShape tile_shape(int i) { return kCandShapes[i]; }
size_t cand_lds_bytes(int kpos, int ntab, bool mask, int n_means_ip, int k, int cw, bool map, int nseg)
{
    return cand_lds_bytes_impl(kpos, ntab, mask, n_means_ip, k, cw, map, nseg);
}
int scan_tile_queries(int g, int ch, int bits1, bool few) { return few ? kScanTQSmall : scan_tq(g, ch, bits1); }
int scan_sorted_keys(int k) { return scan_sorted(k); }
size_t scan_lds_bytes(int tq, int n_means_ip, int k, int g, int bits1, int bits2)
{
    return scan_lds_bytes_impl(tq, (n_means_ip + 3) & ~3, k, scan_staged(g) ? scan_slab(g, bits1, bits2) * (bits1 + bits2) / bits1 : 0);
}

}  // namespace lvq
