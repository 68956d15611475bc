// k_scan_impl.h -- exhaustive top-k over every live slot (the k-NN problem of
// Sec. 2.1), FP32 vector-ALU form.
//
// Grid: (tile of TQ queries) x (part of the slot list).  A lane owns one row
// of the store per round (256 rows per workgroup round) and scores it against
// all TQ queries, whose values are uniform and come through scalar loads, TQ
// of them per code position.  The row is decoded piece by piece into registers
//   IP: y_p = Delta c1_p [+ Delta2 c2_p]          (score = c_m + l' sum q + <q, y>)
//   L2: x'_p = l' + Delta c1_p [+ Delta2 c2_p]    (score = sum (q' - x')^2,
//       padding positions forced to 0 so they contribute nothing)
// and each decoded value feeds TQ independent accumulation chains.
//
// Bound: vector-ALU issue, 2 instructions (IP: 1) per query, row and position;
// the decode (about 2 per position) is shared by the TQ queries.  A group of
// four lanes per row with the queries in LDS, which this replaces, issued
// about 1.9 times as many (a reduction over the lanes and a bound test per
// query and row) and waited on its LDS reads: 600 queries over 300,000 rows of
// d = 96, Euclidean, took 2,794 us, this form 970 us (1.8e13 position
// differences squared and summed per second: 0.91 of the issue rate at 2.4 GHz).
//
// Order of sums.  Values are added up as G lanes per row would add them: leaf
// g of the G takes pieces g, g + G, ... in order, and the G sums meet in a
// binary tree.  Here one lane runs all G chains.
//
// Top-k.  Per query, LDS holds the KS best keys so far (sorted; KS = k rounded
// up to a power of two >= 64) and room for a round's keys.  A score that can
// still enter is appended; queries with 64 or more pending keys are merged
// by their owner wave, 64 at a time, while the next round's products run.
// The parts share each query's bound through gthr.
#pragma once

#include "k_cand_impl.h"

// lambdas that keep arrays of their kernel in registers
#define LVQ_INLINE __attribute__((always_inline))

namespace lvq {

// Queries per tile: rows of up to four leaves (lanes g) run their leaves one
// after the other, 16 chains each; rows of sixteen leaves run all of them side
// by side, 8 chains each, so that the row's bytes are read in order (leaf by
// leaf, 8 bytes of a line at a time, every line came back from memory many
// times: 100 queries of 4x8 d = 768 took 4.3 ms, the four-lane form 2.5 ms,
// this 2.1 ms).  kScanTQSmall: few queries, or long key lists.
// (Pieces of 32 positions -- 4-bit codes, 16 bytes -- always take the few: with
// 8 chains the unrolled leaves spill.)
constexpr int kScanPairs = 1;     // "G" of the matrix cores' order of sums
constexpr int kScanTQSmall = 4;
constexpr int scan_tq(int g, int ch, int bits1)
{
    return g == 4 ? 16 : g == 16 && ch == 16 && bits1 == 4 ? kScanTQSmall : 8;
}
constexpr int kScanRows = 256;    // rows per workgroup round
constexpr int kScanPend = kScanRows + 64;   // pending keys: under 64 carried, a round's appends

inline int scan_sorted(int k)
{
    int ks = 64;
    while (ks < k) ks *= 2;
    return ks;
}

// Rows of sixteen leaves, or in the matrix cores' order, pass through LDS: a
// wave reads a slab of codes of its 64 rows (and the residual codes of the same
// positions) in runs of consecutive bytes, and its lanes take their own row's.
// Beside sixteen leaves' sums a slab of 64 bytes of 4-bit codes with twice the
// residual bytes leaves one wave per SIMD (100 queries of 4x8 d = 768 over
// 300,000 rows 3,992 us, 32 bytes 2,098 us); one chain has the registers and gains
// from the longer runs (one query over 10^6 rows 326 us against 466 us).
constexpr int scan_slab(int g, int bits1, int bits2) { return g == 16 && bits1 == 4 && bits2 == 8 ? 32 : 64; }
constexpr bool scan_staged(int g) { return g == 16 || g == kScanPairs; }

inline size_t scan_lds_bytes_impl(int tq, int n_means_ip, int k, int stage_bytes)
{
    return (size_t)kScanRows * stage_bytes + (size_t)tq * (scan_sorted(k) + kScanPend) * 8 + (size_t)tq * 16 +
           (size_t)tq * n_means_ip * 4;
}

// Words of a lane's own row from the wave's slab: U 16-byte units per row,
// unit u kept at u ^ f so that eight consecutive rows' reads cover all banks.
template <int U>
__device__ __forceinline__ int slab_swizzle(int row)
{
    return U >= 8 ? row & 7 : U == 4 ? (row >> 1) & 3 : U == 2 ? (row >> 2) & 1 : 0;
}

template <int N, int U>
__device__ __forceinline__ Words<N> slab_words(const uint4 *buf, int row, int f, int off)
{
    if constexpr (N == 8) {
        const Words<4> a = slab_words<4, U>(buf, row, f, off), b = slab_words<4, U>(buf, row, f, off + 16);
        Words<8> r;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            r.w[i] = a.w[i];
            r.w[i + 4] = b.w[i];
        }
        return r;
    } else {
        const uint8_t *p = reinterpret_cast<const uint8_t *>(buf + row * U + ((off >> 4) ^ f)) + (off & 15);
        return load_words<N>(p);
    }
}

// A float of device memory read through the scalar cache (uniform addresses).
typedef const __attribute__((address_space(4))) float ScalarF;
__device__ __forceinline__ ScalarF *scalar_ptr(const float *p)
{
    return (ScalarF *)(uintptr_t)p;
}

// The sums of LV leaves from g0 on, as a binary tree; leaves from n on are
// empty (0).  One copy of the leaf's code: the levels are loops.  (A leaf's
// sum starts at +0, so it is never -0 and 0 + sum is the sum.)
template <int LV, int TQ, class Leaf>
__device__ __forceinline__ void scan_tree(int g0, int n, Leaf &leaf, float (&out)[TQ])
{
    if constexpr (LV == 1) {
        leaf(g0, out);
    } else {
#pragma unroll
        for (int q = 0; q < TQ; ++q) out[q] = 0.0f;
        for (int h = 0; h < LV && g0 + h < n; h += LV / 2) {
            float t[TQ];
            scan_tree<LV / 2, TQ>(g0 + h, n, leaf, t);
#pragma unroll
            for (int q = 0; q < TQ; ++q) out[q] += t[q];
        }
    }
}

template <int B1, int B2, int METRIC, bool MASK, int G, int CH, int NCH, int TQ>
__global__ __launch_bounds__(256) void k_scan(ScanArgs a)
{
    using Geo = CandGeom<B1, CH>;
    using RGeo = ResGeom<B1, B2, CH>;
    constexpr int SLOTS = Geo::kSlots;        // code positions per piece

    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int npieces = a.kchunks * 16 / CH;
    const int leaves = npieces < G ? npieces : G;
    const int cm_n = a.n_means;               // (IP)
    const int k = a.k, ks = a.mks, cap = ks + kScanPend;

    uint64_t *region = reinterpret_cast<uint64_t *>(smem);            // TQ x (KS best, pending)
    uint64_t *thr = region + (size_t)TQ * cap;                        // k-th best key of this part
    float *thr_f = reinterpret_cast<float *>(thr + TQ);               // score bound (NaN: none yet)
    int *cnt = reinterpret_cast<int *>(thr_f + TQ);                   // pending keys
    float *cmt = reinterpret_cast<float *>(cnt + TQ);                 // [query][mean] c_m

    const int64_t q0 = (int64_t)blockIdx.x * TQ;
    const int nqt = (int)min<int64_t>(TQ, a.nq - q0);
    const int64_t r0 = (int64_t)blockIdx.y * a.rows_per_part;
    const int64_t r1 = min<int64_t>(a.n_rows, r0 + a.rows_per_part);
    auto out_keys = [&](int qi) { return a.part_keys + ((q0 + qi) * a.n_parts + blockIdx.y) * (int64_t)k; };
    if (r0 >= r1) {   // an empty part contributes no keys
        for (int qi = wave; qi < nqt; qi += 4)
            for (int i = lane; i < k; i += 64) out_keys(qi)[i] = kNoKey;
        return;
    }
    for (int t = tid; t < TQ * ks; t += 256) region[(size_t)(t / ks) * cap + t % ks] = kNoKey;
    if (tid < TQ) {
        thr[tid] = kNoKey;
        thr_f[tid] = __builtin_nanf("");
        cnt[tid] = 0;
    }
    if constexpr (METRIC == LVQ_IP)
        for (int t = tid; t < TQ * cm_n; t += 256) {
            const int qi = t / cm_n, m = t % cm_n;
            cmt[t] = qi < nqt ? a.cm[(q0 + qi) * cm_n + m] : 0.0f;
        }
    __syncthreads();

    ScalarF *qt = scalar_ptr(a.qk + (int64_t)blockIdx.x * a.kpos * TQ);   // [position][query]
    ScalarF *qs = scalar_ptr(a.qsum);
    ScalarF *mask = scalar_ptr(a.kmask);

    struct Piece {
        Words<Geo::kWords> w;
        Words<RGeo::kWords> r;
    };
    // a lane past the part reads the row at r0 (valid) and is not scored
    auto slot_at = [&](int64_t base) -> int64_t {
        const int64_t pos = base + tid;
        return a.list[pos < r1 ? pos : r0];
    };
    int64_t slot = slot_at(r0), slot_n = slot_at(r0 + kScanRows);
    constexpr int BS = 32 / TQ;               // positions per block of query values (32 scalar registers)
    float qv[BS * TQ];
#pragma unroll
    for (int i = 0; i < BS * TQ; ++i) qv[i] = qt[i];
    // staged: the wave's slab, the next one in flight in registers, and the
    // slots of the rows this lane loads units of
    constexpr bool ST = scan_staged(G);
    constexpr int SB = scan_slab(G, B1, B2);
    constexpr int CU = SB / 16, RU = ST && B2 ? SB * B2 / B1 / 16 : 1;   // units per row
    uint4 *const scode = reinterpret_cast<uint4 *>(cmt + (METRIC == LVQ_IP ? (TQ * cm_n + 3) / 4 * 4 : 0)) +
                      wave * 64 * (CU + (B2 ? RU : 0));
    uint4 *const sres = scode + 64 * CU;
    const int nslab = (a.kchunks + CU - 1) / CU;
    const int fc = slab_swizzle<CU>(lane), fr = slab_swizzle<RU>(lane);
    typedef uint32_t Unit __attribute__((ext_vector_type(4)));
    Unit pc[ST ? CU : 1], pr[RU];
    int32_t lc[ST ? CU : 1], lr[RU];
    auto rows_of = [&](int64_t s) LVQ_INLINE {
#pragma unroll
        for (int i = 0; i < CU; ++i) lc[i] = __shfl((int)s, i * (64 / CU) + lane / CU, 64);
        if constexpr (B2 != 0) {
#pragma unroll
            for (int i = 0; i < RU; ++i) lr[i] = __shfl((int)s, i * (64 / RU) + lane / RU, 64);
        }
    };
    // (units past the row's end read its last one and are not used)
    auto load_slab = [&](int s) LVQ_INLINE {
        const int c = min(s * CU + lane % CU, a.kchunks - 1);
#pragma unroll
        for (int i = 0; i < CU; ++i)
            pc[i] = *reinterpret_cast<const Unit *>(a.rows + (int64_t)lc[i] * a.row_bytes + kHeaderBytes + c * 16);
        if constexpr (B2 != 0) {
            const int r = min(s * RU + lane % RU, a.resid_bytes / 16 - 1);
#pragma unroll
            for (int i = 0; i < RU; ++i)
                pr[i] = *reinterpret_cast<const Unit *>(a.resid + (int64_t)lr[i] * a.resid_bytes + r * 16);
        }
    };
    // slab s into LDS (it is in registers), the one after it on its way
    auto next_slab = [&](int s) LVQ_INLINE {
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < CU; ++i) {
            const int row = i * (64 / CU) + lane / CU;
            reinterpret_cast<Unit *>(scode)[row * CU + ((lane % CU) ^ slab_swizzle<CU>(row))] = pc[i];
        }
        if constexpr (B2 != 0) {
#pragma unroll
            for (int i = 0; i < RU; ++i) {
                const int row = i * (64 / RU) + lane / RU;
                reinterpret_cast<Unit *>(sres)[row * RU + ((lane % RU) ^ slab_swizzle<RU>(row))] = pr[i];
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const bool more = s + 1 < nslab;
        if (!more) rows_of(slot_n);
        load_slab(more ? s + 1 : 0);
    };
    // four lanes' order: a leaf's pieces in flight
    auto load_piece = [&](int64_t s, int u) LVQ_INLINE {
        Piece P;
        P.w = load_words<Geo::kWords>(a.rows + s * a.row_bytes + kHeaderBytes + u * CH);
        if constexpr (B2 != 0) P.r = load_words<RGeo::kWords>(a.resid + s * a.resid_bytes + u * RGeo::kBytes);
        return P;
    };
    Piece ring[ST ? 1 : NCH];
    if constexpr (ST) {
        rows_of(slot);
        load_slab(0);
    } else {
#pragma unroll
        for (int i = 0; i < NCH; ++i) ring[i] = load_piece(slot, i * G < npieces ? i * G : 0);
    }

    for (int64_t base = r0; base < r1; base += kScanRows) {
        const bool last = base + kScanRows >= r1;
        const uint8_t *row = a.rows + slot * a.row_bytes;
        const float4 hdr = *reinterpret_cast<const float4 *>(row);
        const uint2 ep = *reinterpret_cast<const uint2 *>(row + 16);
        const int64_t slot_a = slot_at(base + 2 * kScanRows);
        const uint32_t gb = a.gthr[q0 + (lane < nqt ? lane : 0)];   // the other parts' bound of query `lane`
        const float l = hdr.x, dl = hdr.y, dl2 = hdr.z;
        const float lp = B2 ? l - 0.5f * dl : l;
        const float base_v = METRIC == LVQ_L2 ? lp : 0.0f;

        // N decoded values from table position p on, into TQ chains.  qv holds
        // the query values of the next BS positions: those of the block after
        // are loaded once the block's first position has been used (scalar
        // loads return out of order, so a wait is for all of them: a load
        // issued earlier would be waited for at once), position pn's after the
        // last.
        auto feed = [&](const auto &x, int p, int pn, float (&acc)[TQ]) LVQ_INLINE {
            constexpr int N = sizeof(x) / sizeof(float);
#pragma unroll
            for (int b = 0; b < N / BS; ++b) {
                auto pos = [&](int s) LVQ_INLINE {
#pragma unroll
                    for (int q = 0; q < TQ; ++q) {
                        if constexpr (METRIC == LVQ_IP) {
                            acc[q] = fmaf(qv[s * TQ + q], x[b * BS + s], acc[q]);
                        } else {
                            const float t = qv[s * TQ + q] - x[b * BS + s];
                            acc[q] = fmaf(t, t, acc[q]);
                        }
                    }
                };
                pos(0);
                __builtin_amdgcn_sched_barrier(0);
                ScalarF *qp = qt + (b + 1 < N / BS ? p + (b + 1) * BS : pn) * TQ;
                float qn[BS * TQ];
#pragma unroll
                for (int i = 0; i < BS * TQ; ++i) qn[i] = qp[i];
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int s = 1; s < BS; ++s) pos(s);
#pragma unroll
                for (int i = 0; i < BS * TQ; ++i) qv[i] = qn[i];
            }
        };
        // piece u of the row, decoded; piece un is the next
        auto piece = [&](const Piece &P, int u, int un, float (&acc)[TQ]) LVQ_INLINE {
            float x[SLOTS];
#pragma unroll
            for (int wi = 0; wi < Geo::kWords; ++wi) {
                const uint32_t w = P.w.w[wi];
                constexpr int QW = B1 == 4 ? 8 : 4;
                float c1[QW], c2[QW], s1[QW], s2[QW];
                if constexpr (B1 == 4) {
                    const uint32_t lo = w & 0x0F0F0F0Fu, hi = w & 0xF0F0F0F0u;
                    c1[0] = ub<0>(lo); c1[1] = ub<1>(lo); c1[2] = ub<2>(lo); c1[3] = ub<3>(lo);
                    c1[4] = ub<0>(hi); c1[5] = ub<1>(hi); c1[6] = ub<2>(hi); c1[7] = ub<3>(hi);
                    for (int s = 0; s < 4; ++s) { s1[s] = dl; s1[s + 4] = dl * 0.0625f; }
                    for (int s = 0; s < 8; ++s) { c2[s] = 0.f; s2[s] = dl2; }
                    if constexpr (B2 == 8) {
                        const uint32_t q0w = P.r.w[2 * wi], q1w = P.r.w[2 * wi + 1];
                        c2[0] = ub<0>(q0w); c2[1] = ub<2>(q0w); c2[2] = ub<0>(q1w); c2[3] = ub<2>(q1w);
                        c2[4] = ub<1>(q0w); c2[5] = ub<3>(q0w); c2[6] = ub<1>(q1w); c2[7] = ub<3>(q1w);
                    } else if constexpr (B2 == 4) {
                        const uint32_t r = P.r.w[wi];
                        const uint32_t rl = r & 0x0F0F0F0Fu, rh = r & 0xF0F0F0F0u;
                        c2[0] = ub<0>(rl); c2[1] = ub<1>(rl); c2[2] = ub<2>(rl); c2[3] = ub<3>(rl);
                        c2[4] = ub<0>(rh); c2[5] = ub<1>(rh); c2[6] = ub<2>(rh); c2[7] = ub<3>(rh);
                        for (int s = 4; s < 8; ++s) s2[s] = dl2 * 0.0625f;
                    }
                } else {
                    c1[0] = ub<0>(w); c1[1] = ub<1>(w); c1[2] = ub<2>(w); c1[3] = ub<3>(w);
                    for (int s = 0; s < 4; ++s) { s1[s] = dl; c2[s] = 0.f; s2[s] = dl2; }
                    if constexpr (B2 == 8) {
                        const uint32_t r = P.r.w[wi];
                        c2[0] = ub<0>(r); c2[1] = ub<1>(r); c2[2] = ub<2>(r); c2[3] = ub<3>(r);
                    } else if constexpr (B2 == 4) {
                        const uint32_t h = (P.r.w[wi >> 1] >> (16 * (wi & 1))) & 0xFFFFu;
                        const uint32_t rl = h & 0x0F0Fu, rh = h & 0xF0F0u;
                        c2[0] = ub<0>(rl); c2[2] = ub<1>(rl); c2[1] = ub<0>(rh); c2[3] = ub<1>(rh);
                        s2[1] = dl2 * 0.0625f; s2[3] = dl2 * 0.0625f;
                    }
                }
#pragma unroll
                for (int s = 0; s < QW; ++s) {
                    float v = fmaf(s1[s], c1[s], base_v);
                    if constexpr (B2 != 0) v = fmaf(s2[s], c2[s], v);
                    if constexpr (MASK) v *= mask[u * SLOTS + wi * QW + s];
                    x[wi * QW + s] = v;
                }
            }
            feed(x, u * SLOTS, un * SLOTS, acc);
        };
        float tot[TQ];
        if constexpr (G == 16) {
            constexpr int PPS = SB / CH;   // pieces per slab
            float acc[G][TQ];
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int q = 0; q < TQ; ++q) acc[g][q] = 0.0f;
#pragma unroll 1
            for (int u0 = 0; u0 < npieces; u0 += G) {
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    if (u0 + g < npieces) {
                        if (g % PPS == 0) next_slab((u0 + g) / PPS);
                        Piece P;
                        P.w = slab_words<Geo::kWords, CU>(scode, lane, fc, g % PPS * CH);
                        if constexpr (B2 != 0) P.r = slab_words<RGeo::kWords, RU>(sres, lane, fr, g % PPS * RGeo::kBytes);
                        piece(P, u0 + g, u0 + g + 1 < npieces ? u0 + g + 1 : 0, acc[g]);
                    }
                }
            }
#pragma unroll
            for (int o = 1; o < G; o *= 2)
#pragma unroll
                for (int g = 0; g < G; g += 2 * o)
#pragma unroll
                    for (int q = 0; q < TQ; ++q) acc[g][q] += acc[g + o][q];
#pragma unroll
            for (int q = 0; q < TQ; ++q) tot[q] = acc[0][q];
        } else if constexpr (G == kScanPairs) {
            // The FP32 matrix cores' order: one chain, through the chunks of
            // 32 bytes of codes, taking a position of the first half of a
            // chunk and one of the second in turn (what lanes l and l + 32
            // feed one product), each product fused into the sum.  The values
            // are theirs too: the code alone at the first level.
            constexpr int QW = B1 == 4 ? 8 : 4, CP = B1 == 4 ? 64 : 32;   // positions per word and chunk
            constexpr int RW = B2 ? B2 / B1 : 1;                          // residual words per code word
            constexpr int CPS = SB / 32;                                  // chunks per slab
#pragma unroll
            for (int q = 0; q < TQ; ++q) tot[q] = 0.0f;
            const int nchunk = a.kpos / CP;
#pragma unroll 1
            for (int s = 0; s < nslab; ++s) {
                next_slab(s);
#pragma unroll 1
                for (int c = CPS * s; c < min(CPS * s + CPS, nchunk); ++c) {
                    Words<4> w[2];
                    Words<4 * RW> r[2];
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        w[h] = slab_words<4, CU>(scode, lane, fc, (c % CPS * 2 + h) * 16);
                        if constexpr (B2 != 0)
                            r[h] = slab_words<4 * RW, RU>(sres, lane, fr, (c % CPS * 2 + h) * 16 * RW);
                    }
#pragma unroll
                    for (int wi = 0; wi < 4; ++wi) {
                        float x[2 * QW];
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            uint32_t cw[QW / 4], rw[QW / 4];
                            if constexpr (B1 == 4) {
                                cw[0] = w[h].w[wi] & 0x0F0F0F0Fu;
                                cw[1] = (w[h].w[wi] >> 4) & 0x0F0F0F0Fu;
                                if constexpr (B2 == 8) {
                                    rw[0] = __builtin_amdgcn_perm(r[h].w[2 * wi + 1], r[h].w[2 * wi], 0x06040200u);
                                    rw[1] = __builtin_amdgcn_perm(r[h].w[2 * wi + 1], r[h].w[2 * wi], 0x07050301u);
                                }
                            } else {
                                cw[0] = w[h].w[wi];
                                if constexpr (B2 == 8) rw[0] = r[h].w[wi];
                            }
#pragma unroll
                            for (int e = 0; e < QW; ++e) {
                                const float c1 = (float)((cw[e / 4] >> (8 * (e % 4))) & 0xFFu);
                                if constexpr (B2 == 8) {
                                    const float c2 = (float)((rw[e / 4] >> (8 * (e % 4))) & 0xFFu);
                                    x[2 * e + h] = fmaf(dl2, c2, dl * c1);
                                } else {
                                    x[2 * e + h] = c1;
                                }
                            }
                        }
                        const int p = c * CP + wi * 2 * QW;
                        feed(x, p, p + 2 * QW < a.kpos ? p + 2 * QW : 0, tot);
                    }
                }
            }
        } else {
            // one leaf: its pieces in order
            auto leaf = [&](int g, float (&acc)[TQ]) LVQ_INLINE {
                const bool more = g + 1 < leaves;
                Piece cur[NCH];
#pragma unroll
                for (int c = 0; c < NCH; ++c) {
                    cur[c] = ring[c];
                    const int u = c * G + (more ? g + 1 : 0);
                    ring[c] = load_piece(more ? slot : slot_n, u < npieces ? u : 0);
                }
#pragma unroll
                for (int q = 0; q < TQ; ++q) acc[q] = 0.0f;
#pragma unroll
                for (int c = 0; c < NCH; ++c) {
                    const int u = c * G + g;
                    if (u < npieces) piece(cur[c], u, u + G < npieces && c + 1 < NCH ? u + G : more ? g + 1 : 0, acc);
                }
            };
            scan_tree<G, TQ>(0, leaves, leaf, tot);
        }

        // the previous round's merges are done: their bounds are in LDS
        __syncthreads();
        float bnd = thr_f[lane < TQ ? lane : 0];   // bound of query `lane`; NaN admits everything
        if (gb != 0xFFFFFFFFu) {
            const float o = key_score((uint64_t)gb << 32, METRIC);
            bnd = METRIC == LVQ_L2 ? fminf(bnd, o) : fmaxf(bnd, o);
        }
        const bool live = base + tid < r1 && ((__float_as_uint(hdr.w) >> 8) & 1u) && ep.x <= a.epoch &&
                          a.epoch < ep.y;
        const int mid = (int)(__float_as_uint(hdr.w) & 0xFFu);
        const int mrow = mid < a.n_means ? mid : 0;
#pragma unroll
        for (int q = 0; q < TQ; ++q) {
            if (q >= nqt) break;
            float sc = tot[q];
            const float b = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(bnd), q));
            bool pass;
            if constexpr (G == kScanPairs) {
                // the matrix-core scans' score; they never return a NaN one
                sc = fmaf(B2 ? 1.0f : dl, sc, fmaf(lp, qs[q0 + q], cmt[q * cm_n + mrow]));
                pass = live && sc == sc && !(sc < b);
            } else {
                if constexpr (METRIC == LVQ_IP) sc = fmaf(lp, qs[q0 + q], cmt[q * cm_n + mrow]) + sc;
                // (a NaN score passes here and ranks last by its key)
                pass = live && !(METRIC == LVQ_L2 ? sc > b : sc < b);
            }
            if (__ballot(pass)) {
                const uint64_t key = make_key(sc, (int32_t)slot, METRIC);
                if (pass && key < thr[q]) region[(size_t)q * cap + ks + atomicAdd(&cnt[q], 1)] = key;
            }
        }
        // the round's appends are done
        __syncthreads();
        for (int q = wave; q < nqt; q += 4) {
            const int n = cnt[q];
            if (!last && n < 64) continue;
            uint64_t kth;
            const int got = merge_region_ks(ks, region + (size_t)q * cap, 0, n, k, last ? out_keys(q) : nullptr, &kth);
            if (lane == 0) {
                cnt[q] = 0;
                if (got == k) {
                    // this part holds k candidates at least as good as kth,
                    // so no worse score can enter the final top k
                    thr[q] = kth;
                    thr_f[q] = key_score(kth, METRIC);
                    __hip_atomic_fetch_min(&a.gthr[q0 + q], (uint32_t)(kth >> 32), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        }
        slot = slot_n;
        slot_n = slot_a;
    }
}

}  // namespace lvq
