// k_scan_inst.h -- instantiation table of k_scan for one first-level width.
#pragma once

#include "k_cand_inst.h"
#include "k_scan_impl.h"

namespace lvq {

using ScanKernel = void (*)(ScanArgs);

// variant: 0 = IP, 1 = L2, 2 = L2 masked (generic shape only)
// (queries per tile: scan_tq, or kScanTQSmall when `few`)
template <int B1, int B2, int S, int TQ>
constexpr ScanKernel scan_kernel_tq(int variant)
{
    constexpr CandShape sh = kCandShapes[S];
    if (variant == 0) return k_scan<B1, B2, LVQ_IP, false, sh.g, sh.ch, sh.nch, TQ>;
    if (variant == 1) return k_scan<B1, B2, LVQ_L2, false, sh.g, sh.ch, sh.nch, TQ>;
    if constexpr (S == 0)
        if (variant == 2) return k_scan<B1, B2, LVQ_L2, true, sh.g, sh.ch, sh.nch, TQ>;
    return nullptr;
}

template <int B1, int B2, int S>
constexpr ScanKernel scan_kernel_for(int variant, bool few)
{
    return few ? scan_kernel_tq<B1, B2, S, kScanTQSmall>(variant) : scan_kernel_tq<B1, B2, S, scan_tq(kCandShapes[S].g, kCandShapes[S].ch, B1)>(variant);
}

// Inner product in the matrix cores' order of sums, at the first level or with
// 8-bit residual codes.
template <int B1>
inline ScanKernel scan_pairs_lookup(int bits2, bool few)
{
    constexpr int T = scan_tq(kScanPairs, 16, B1), F = kScanTQSmall;
    if (bits2 == 0) return few ? k_scan<B1, 0, LVQ_IP, false, kScanPairs, 16, 1, F> : k_scan<B1, 0, LVQ_IP, false, kScanPairs, 16, 1, T>;
    if (bits2 == 8) return few ? k_scan<B1, 8, LVQ_IP, false, kScanPairs, 16, 1, F> : k_scan<B1, 8, LVQ_IP, false, kScanPairs, 16, 1, T>;
    return nullptr;
}

template <int B1, int B2>
inline ScanKernel scan_lookup(int variant, int shape, bool few)
{
    switch (shape) {
    case 0: return scan_kernel_for<B1, B2, 0>(variant, few);
    case 1: return B2 == 4 ? nullptr : scan_kernel_for<B1, B2, 1>(variant, few);
    case 3: return B2 == 4 ? nullptr : scan_kernel_for<B1, B2, 3>(variant, few);
    case 4: return B2 == 4 ? nullptr : scan_kernel_for<B1, B2, 4>(variant, few);
    default: return nullptr;
    }
}

}  // namespace lvq
