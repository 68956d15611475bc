// k_mfma.hip -- matrix-core scan: first-level instantiations, the preparation
// of the queries, and the host-side launch helpers.
#include "k_mfma_impl.h"

namespace lvq {
namespace {

// Fragment order: [tile][block][chunk][step][lane], 16 bytes per lane: lane l
// holds query 32 block + (l & 31) (zero past nq) at the POS positions from
// CHUNK_POS c + (CHUNK_POS / 2)(l >> 5) + POS s on (zero at padding): those of
// the codes that b_fragment (16-bit) or code_words (FP32, one MFMA per
// position) hands that lane.
//
// The queries of a matrix-core scan as MFMA fragments, their sum(q) and c_m,
// and the shared bounds reset.  PREC picks the query type.  Workgroups below
// frag_blocks write one 16-byte fragment per lane (8 positions of a 16-bit
// query, 4 of an FP32 one; one fragment is what one lane feeds one MFMA step,
// or four FP32 ones); the others sum, one wave per (query, group of four
// means).  Both are latency-bound for a served batch, so the work is spread
// over as many lanes as there are fragments: one workgroup per query tile
// took 506 us for 300 queries of d = 768 with 16 means (five tiles) and 197
// us for 4,096 of d = 512; this form takes 23 us and 10 us.
template <int B1, int PREC>
__global__ __launch_bounds__(256) void k_prep_scan(const void *qv, int64_t nq, int dim, int kpos, int qb,
                                                   const int32_t *kdim, const float *means, int n_means, uint4 *frag,
                                                   int64_t n_frag, unsigned frag_blocks, float *qsum, float *cm,
                                                   uint32_t *gthr)
{
    constexpr bool F32 = PREC == LVQ_FP32;
    constexpr int CHUNK_POS = B1 == 8 ? 32 : 64;
    constexpr int POS = F32 ? 4 : 8;                      // positions per fragment
    constexpr int STEPS = CHUNK_POS / (2 * POS);          // fragments per chunk and lane
    const uint16_t *q16 = reinterpret_cast<const uint16_t *>(qv);
    const float *q32 = reinterpret_cast<const float *>(qv);
    if (blockIdx.x < frag_blocks) {
        const int64_t f = (int64_t)blockIdx.x * 256 + threadIdx.x;
        if (f >= n_frag) return;
        const int nchunk = kpos / CHUNK_POS;
        const int l = (int)(f & 63);
        const int64_t r = f >> 6;                          // ((tile * qb + b) * nchunk + c) * STEPS + s
        const int s = (int)(r % STEPS);
        const int c = (int)(r / STEPS % nchunk);
        const int64_t gq = r / (STEPS * nchunk) * 32 + (l & 31);
        const int p = c * CHUNK_POS + (l >> 5) * (CHUNK_POS / 2) + POS * s;
        uint32_t w[4] = {0u, 0u, 0u, 0u};
        if (gq < nq) {
#pragma unroll
            for (int j = 0; j < POS; ++j) {
                const int d = kdim[p + j];
                if constexpr (F32) {
                    w[j] = d >= 0 ? __float_as_uint(q32[gq * dim + d]) : 0u;
                } else {
                    const uint32_t v = d >= 0 ? q16[gq * dim + d] : 0u;
                    w[j >> 1] |= v << (16 * (j & 1));
                }
            }
        }
        frag[f] = make_uint4(w[0], w[1], w[2], w[3]);
        return;
    }
    const int groups = (n_means + 3) / 4;
    const int64_t unit = (int64_t)(blockIdx.x - frag_blocks) * 4 + (threadIdx.x >> 6);
    const int64_t gq = unit / groups;
    const int m0 = (int)(unit % groups) * 4, lane = threadIdx.x & 63;
    if (gq >= nq) return;
    auto val = [&](int d) -> float {
        if constexpr (F32) return q32[gq * dim + d];
        const uint16_t h = q16[gq * dim + d];
        if constexpr (PREC == LVQ_FP16) return (float)__builtin_bit_cast(_Float16, h);
        return __uint_as_float((uint32_t)h << 16);
    };
    if (m0 == 0) {
        float s = 0.0f;
        for (int d = lane; d < dim; d += 64) s += val(d);
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
        if (lane == 0) {
            qsum[gq] = s;
            gthr[gq] = 0xFFFFFFFFu;
        }
    }
    const int m1 = m0 + 4 < n_means ? m0 + 4 : n_means;
    for (int m = m0; m < m1; ++m) {
        float t = 0.0f;
        for (int d = lane; d < dim; d += 64) t = fmaf(val(d), means[(int64_t)m * dim + d], t);
        for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
        if (lane == 0) cm[gq * n_means + m] = t;
    }
}

template <int B1, int PREC>
hipError_t prep_scan(const void *q, int64_t nq, int dim, int kpos, int qb, const int32_t *kdim, const float *means,
                     int n_means, void *frag, float *qsum, float *cm, uint32_t *gthr, hipStream_t s)
{
    const int64_t tiles = (nq + 32 * qb - 1) / (32 * qb);
    const int64_t n_frag = tiles * 32 * qb * kpos * (PREC == LVQ_FP32 ? 4 : 2) / 16;
    const int64_t fb = (n_frag + 255) / 256, sb = (nq * ((n_means + 3) / 4) + 3) / 4;
    hipLaunchKernelGGL((k_prep_scan<B1, PREC>), dim3((unsigned)(fb + sb)), dim3(256), 0, s, q, nq, dim, kpos, qb, kdim,
                       means, n_means, reinterpret_cast<uint4 *>(frag), n_frag, (unsigned)fb, qsum, cm, gthr);
    return hipGetLastError();
}

}  // namespace

MfmaKernelPtr mfma_kernel_first(int bits1, int kpos, int fp16, int *qb)
{
    if (bits1 == 8) return fp16 ? (MfmaKernelPtr)mfma_lookup<8, 0, true>(kpos, qb) : (MfmaKernelPtr)mfma_lookup<8, 0, false>(kpos, qb);
    if (bits1 == 4) return fp16 ? (MfmaKernelPtr)mfma_lookup<4, 0, true>(kpos, qb) : (MfmaKernelPtr)mfma_lookup<4, 0, false>(kpos, qb);
    return nullptr;
}
int mfma_query_block(int bits1, int bits2, int kpos)
{
    if (bits1 != 4 && bits1 != 8) return 0;
    if (kpos % (bits1 == 8 ? 32 : 64)) return 0;
    int qb = 0;
    const MfmaKernelPtr k = bits2 == 0 ? mfma_kernel_first(bits1, kpos, 0, &qb)
                                       : bits2 == 8 ? mfma_kernel_full(bits1, kpos, 0, &qb) : nullptr;
    return k ? qb : 0;
}

size_t mfma_lds_bytes(int qb, int n_means, int k, int capq)
{
    const int tq = 32 * qb;
    size_t b = (size_t)tq * 4 + (size_t)tq * n_means * 4;
    b = (b + 15) & ~(size_t)15;
    b += (size_t)tq * (8 + 4 + 4) + (tq & 1) * 4 + 8;
    b += (size_t)tq * capq * 8;
    b += (size_t)kWaves * k * 8;
    return b;
}

// Largest per-query key buffer (<= 512 keys, the register sort's reach, or
// k + one round when k is larger) that fits lds_max; 0 if even k + one round
// does not.
int mfma_capq(int qb, int n_means, int k, size_t lds_max)
{
    const int need = k + kRowsPerIter;
    int cap = need > 512 ? need : 512;
    while (cap > need && mfma_lds_bytes(qb, n_means, k, cap) > lds_max) cap -= 16;
    if (cap < need) cap = need;
    return mfma_lds_bytes(qb, n_means, k, cap) <= lds_max ? cap : 0;
}

hipError_t launch_prep_scan(const void *q, int64_t nq, int dim, int kpos, int bits1, int qb, int prec,
                            const int32_t *kdim, const float *means, int n_means, void *frag, float *qsum, float *cm,
                            uint32_t *gthr, hipStream_t s)
{
    if (qb < 1 || n_means < 1 || (bits1 != 4 && bits1 != 8) || kpos % (bits1 == 8 ? 32 : 64)) return hipErrorInvalidValue;
    if (nq <= 0) return hipSuccess;
    auto run = [&](auto kern) {
        return kern(q, nq, dim, kpos, qb, kdim, means, n_means, frag, qsum, cm, gthr, s);
    };
    if (prec == LVQ_FP32) return bits1 == 8 ? run(prep_scan<8, LVQ_FP32>) : run(prep_scan<4, LVQ_FP32>);
    if (prec == LVQ_BF16) return bits1 == 8 ? run(prep_scan<8, LVQ_BF16>) : run(prep_scan<4, LVQ_BF16>);
    if (prec == LVQ_FP16) return bits1 == 8 ? run(prep_scan<8, LVQ_FP16>) : run(prep_scan<4, LVQ_FP16>);
    return hipErrorInvalidValue;
}

hipError_t launch_scan_mfma(const ScanArgs &a, int bits1, int bits2, int prec, hipStream_t s)
{
    int qb = 0;
    const int fp16 = prec == LVQ_FP16 ? 1 : 0;
    MfmaKernelPtr kern = bits2 == 0 ? mfma_kernel_first(bits1, a.kpos, fp16, &qb)
                                    : bits2 == 8 ? mfma_kernel_full(bits1, a.kpos, fp16, &qb) : nullptr;
    if (!kern) return hipErrorInvalidValue;
    const int64_t qtiles = (a.nq + 32 * qb - 1) / (32 * qb);
    const int64_t ntiles = qtiles * a.n_parts;
    const int64_t grid = (ntiles + 7) / 8 * 8;
    const size_t lds = mfma_lds_bytes(qb, a.n_means, a.k, a.capq);
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(256), lds, s, a);
    return hipGetLastError();
}

}  // namespace lvq
