// The plan of the windowed product: what window_plan.cpp lays out for a space and the
// kernels of window_impl.h read.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace pd {

// One class of lanes of a pass: the lanes of workgroups first_block onwards, all
// with the same pair counts.
struct WinClass {
    uint32_t first_block, lanes;
    uint32_t NL;      // states of nl pairs on the orbits below the window
    uint32_t reach;   // largest rank count below the window that a lane reads
    int32_t K, m, nl; // pairs in the window, above it, below it
    int32_t pad;
};
struct WinPass {
    const WinClass *cls;     // device
    const int64_t *off;      // device: rank offset of each window state, per pair count
    int nclass, W, w0, qmin;
    uint32_t nblocks;
};
constexpr int kSegW = 7, kSegL = 9, kSeg = kSegW + kSegL;   // segment pass: window over low orbits
constexpr int kSegGroup = 128;
// Window pair counts in the order a group takes them, the longest lanes first.
__host__ __device__ constexpr int seg_order(int t) {
    return t < 6 ? (0x615243 >> (4 * t)) & 15 : t == 6 ? 0 : 7;
}
// The segments with q pairs, len elements each: nseg of them, in groups of
// `group` numbered from `first` on.  items[t]: the end of the items (64 lanes
// each) of window pair count seg_order(t); nl[K] low states, listed from
// first_pat[K] on.  magic, lane_magic: e / len and f / nl[K] as the upper half
// of a product (exact below 2^32 / len, 2^32 / nl[K]).
struct SegClass {
    uint32_t first, nseg;
    int32_t q, len, group;
    uint32_t magic;
    int32_t items[kSegW + 1], nl[kSegW + 1], first_pat[kSegW + 1];
    uint32_t lane_magic[kSegW + 1];
};
struct SegPass {
    const SegClass *cls;     // device
    const int32_t *off;      // device: place in the segment of each window state, per pair count
    int nclass, qmin, cap;   // cap: elements of a group
    uint32_t ngroup;
};
constexpr int kMaxWinPasses = 3;
constexpr int kMaxWinOmega = 40;
struct WinPlan {
    SegPass seg;
    WinPass pass[kMaxWinPasses];
    int npass;
};
// Spaces whose products go by windows: kMinWinDim states with 8 pairs (or
// holes) and more, kMinWinDim7 with 7.  A lane does the work of up to C(W, K) rows, so
// a small space leaves the chip idle, and with few pairs most lanes own one
// or two window states.  Measured, windows against a row per lane, us in FP64 / FP32
// (23 orbits with two waves to a lane group, kSplitBlocks in window_impl.h):
// Omega = 22, n = 11 (705,432 states) 56 / 44 against 46 / 31; Omega = 25, n = 8 (1.08e6)
// 90 / 59 against 76 / 49; Omega = 23, n = 10 (1.14e6) 66 / 54 against 76 / 50, n = 11 (1.35e6)
// 67 / 54 against 90 / 64; Omega = 27, n = 8 (2.2e6) 144 / 94 against 168 / 105; with 7 pairs Omega = 30 (2.0e6) 255 / 158 against 174 / 109, Omega = 33 (4.3e6)
// 402 / 237 against 414 / 253; with 6, Omega = 40 (3.8e6) 717 / 449 against 476 / 281.
constexpr uint64_t kMinWinDim = 1200000, kMinWinDim7 = 4200000;
// Bytes of a space's plan on the device, 0 when its products take a row per lane.
size_t window_plan_bytes(int omega, int n);
// The plan with device pointers into dev, and in host the window_plan_bytes
// bytes to put there.
bool window_plan_build(int omega, int n, void *dev, WinPlan *plan, unsigned char *host);
hipError_t window_product_f64(const WinPlan &plan, int omega, int n, const double *d, const double *V,
                              const double *x, double *y, hipStream_t s);
hipError_t window_product_f32(const WinPlan &plan, int omega, int n, const float *d, const float *V, const float *x,
                              float *y, hipStream_t s);

}  // namespace pd
