// Workgroup shapes of the persistent decode kernels (host code).
#pragma once

#include <algorithm>

#include "dtans_core.hpp"

namespace dtans {

// waves per SIMD the registers admit: the row-layout SpMV kernels, and those of
// the nonzero-balanced layout, which also track rows
constexpr int kRowWavesPerSimd = 8, kNnzWavesPerSimd = 6;

// Default workgroup shape of the decode kernels: LDS admits 160 KiB /
// table_bytes workgroups per CU (2 for FP64 and FP32); the registers admit
// `per_simd` waves per SIMD.  A workgroup's waves are dealt to the CU's 4
// SIMDs, so its size is kept a multiple of 4: with 9-wave workgroups, three
// per CU did not all fit and the third started only when another ended.
// Among workgroup counts, the most resident waves win (then the most
// workgroups).
inline void default_shape(bool f64, int per_simd, int &wpw, int &wgcu) {
    const int table_bytes = kSlots * (8 + (f64 ? 12 : 8));
    const int maxwg = std::max(1, 160 * 1024 / table_bytes);
    wpw = 4;
    wgcu = 1;
    for (int g = maxwg; g >= 1; --g) {
        const int w = std::min(16, (4 * per_simd / g) & ~3);
        if (w >= 4 && w * g > wpw * wgcu) {
            wpw = w;
            wgcu = g;
        }
    }
}

struct ShapePlan {
    int waves_per_wg, wg_per_cu;
    bool fixed;  // the caller's shape; otherwise each kernel may choose another
};

// The shape for the options waves_per_wg and wg_per_cu (0: automatic).  The
// default shape given as options is the automatic one: the autotuner returns
// shapes, its first candidate being the default, and what it timed fastest has
// to include the kernels and grids that only the automatic choice runs.
inline ShapePlan plan_shape(bool f64, bool row_layout, int waves_per_wg, int wg_per_cu) {
    const int per_simd = row_layout ? kRowWavesPerSimd : kNnzWavesPerSimd;
    int dw = 0, dg = 0;
    default_shape(f64, per_simd, dw, dg);
    ShapePlan p{dw, dg, false};
    if (wg_per_cu > 0) {
        p.wg_per_cu = wg_per_cu;
        p.waves_per_wg = std::max(4, std::min(16, (4 * per_simd / wg_per_cu) & ~3));
    }
    if (waves_per_wg > 0) p.waves_per_wg = waves_per_wg;
    p.fixed = p.waves_per_wg != dw || p.wg_per_cu != dg;
    return p;
}

}  // namespace dtans
