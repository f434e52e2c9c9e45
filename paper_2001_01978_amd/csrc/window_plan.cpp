// Plan of the windowed product (window_impl.h) for one space: how the orbits
// are cut, the classes of lanes of each pass, and the offset tables.
#include <algorithm>
#include <cstring>

#include "pd_internal.h"

namespace pd {
namespace {

constexpr int kMinW = 4, kMaxW = 8;
constexpr int kWinBlock = 256;
constexpr uint64_t kMinGroups = 512;       // two for each CU
// Eight orbits above the segments can be one window or two (fewer cannot be two, more are
// two at least): one of 8 from here on, two of 4 below: 24 orbits, 9 pairs (1.3e6
// states) 78.6 / 58.3 us (FP64 / FP32) with two and 92.9 / 72.8 with one; 10 pairs (2.0e6)
// 93.5 / 74.8 and 94.1 / 74.4; 12 pairs (2.7e6) 120 / 90 and 97.8 / 77.7.
constexpr uint64_t kMinWideDim = 2000000;

// Windows from the top: as few as possible, of nearly equal width, the wider
// ones first (the top window has the most orbits below it, and an element it
// loads serves the more states the wider it is).
int cut_orbits(int omega, uint64_t dim, int *W) {
    const int rest = omega - kSeg;
    if (rest < kMinW) return 0;
    const int np = rest == kMaxW && dim < kMinWideDim ? 2 : (rest + kMaxW - 1) / kMaxW;
    if (np > kMaxWinPasses || rest < np * kMinW) return 0;
    for (int i = 0; i < np; ++i) W[i] = rest / np + (i < rest % np ? 1 : 0);
    return np;
}

uint64_t lanes_of(int U, int m, int w0, int nl) { return binom_host(U, m) * binom_host(w0, nl); }

struct Pass {
    int W, w0, U, qmin, qmax;
    int ncls;
    uint32_t nblocks;
    WinClass cls[(kMaxW + 1) * (kMaxWinOmega + 1)];
};
struct SegPlan {
    int ncls, qmin, qmax, cap;
    uint32_t ngroup;
    SegClass cls[kSeg + 1];
};
// The plan of a space, host side (no heap: the C entry points call this).
struct Passes {
    int np;
    SegPlan seg;
    Pass win[kMaxWinPasses];
};

// Classes of the window pass; false when a count does not fit the kernel's 32-bit fields.
bool window_classes(int omega, int n, Pass &p) {
    const int m0 = std::max(0, n - p.w0 - p.W), m1 = std::min(n, p.U);
    p.qmin = n - m1;
    p.qmax = n - m0;
    double cost[(kMaxW + 1) * (kMaxWinOmega + 1)];
    p.ncls = 0;
    for (int m = m0; m <= m1; ++m)
        for (int K = 0; K <= p.W; ++K) {
            const int nl = n - m - K;
            if (nl < 0 || nl > p.w0) continue;
            const uint64_t lanes = lanes_of(p.U, m, p.w0, nl);
            uint64_t reach = 0;
            for (int l = std::max(nl - 1, 0); l <= std::min(nl + 1, p.w0); ++l)
                reach = std::max<uint64_t>(reach, binom_host(p.w0, l));
            if (lanes > 0xFFFF0000ull || reach * 8 > 0xFFFFFFFFull) return false;
            if ((K == 0 && nl == 0) || (K == p.W && nl == p.w0)) continue;   // no hops
            WinClass c;
            std::memset(&c, 0, sizeof(c));
            c.lanes = (uint32_t)lanes;
            c.NL = (uint32_t)binom_host(p.w0, nl);
            c.reach = (uint32_t)reach;
            c.K = K;
            c.m = m;
            c.nl = nl;
            const double t = 3.0 * binom_host(p.W, K) + nl * (double)binom_host(p.W, K + 1) +
                             (p.w0 - nl) * (K > 0 ? (double)binom_host(p.W, K - 1) : 0.0);
            // the longest lanes first, so that the last workgroups are short ones
            int at = p.ncls++;
            for (; at > 0 && cost[at - 1] < t; --at) {
                p.cls[at] = p.cls[at - 1];
                cost[at] = cost[at - 1];
            }
            p.cls[at] = c;
            cost[at] = t;
        }
    uint64_t nb = 0;
    for (int i = 0; i < p.ncls; ++i) {
        p.cls[i].first_block = (uint32_t)nb;
        nb += (p.cls[i].lanes + (uint64_t)kWinBlock - 1) / kWinBlock;
    }
    if (nb > 0x7FFFFFFFull) return false;
    p.nblocks = (uint32_t)nb;
    return true;
}

uint32_t magic_of(int d) { return d > 1 ? (uint32_t)(((uint64_t(1) << 32) + d - 1) / d) : 0; }

// The segments, longest first.
bool segment_classes(int omega, int n, SegPlan &p) {
    const int U = omega - kSeg;
    uint64_t groups = 0;
    p.ncls = p.cap = 0;
    p.qmin = std::max(0, n - U);
    p.qmax = std::min(n, kSeg);
    for (int q = p.qmin; q <= p.qmax; ++q) p.cap = std::max(p.cap, (int)binom_host(kSeg, q));
    // A group fills LDS unless the space is too small to give every CU two of them.
    const uint64_t rows = std::min<uint64_t>(p.cap, binom_host(omega, n) / kMinGroups);
    bool done[kSeg + 1] = {};
    for (int t = p.qmin; t <= p.qmax; ++t) {
        int q = -1;
        for (int i = p.qmin; i <= p.qmax; ++i)
            if (!done[i] && (q < 0 || binom_host(kSeg, i) > binom_host(kSeg, q))) q = i;
        done[q] = true;
        SegClass &c = p.cls[p.ncls++];
        std::memset(&c, 0, sizeof(c));
        c.first = (uint32_t)groups;
        c.nseg = (uint32_t)binom_host(U, n - q);
        c.q = q;
        c.len = (int)binom_host(kSeg, q);
        c.group = std::max(1, std::min<int>(kSegGroup, (int)(rows / c.len)));
        c.magic = magic_of(c.len);
        groups += (c.nseg + (uint64_t)c.group - 1) / c.group;
        int items = 0;
        for (int s = 0; s <= kSegW; ++s) {
            const int K = seg_order(s), kl = q - K;
            if (kl >= 0 && kl <= kSegL) {
                c.nl[K] = (int)binom_host(kSegL, kl);
                c.lane_magic[K] = magic_of(c.nl[K]);
                for (int i = 0; i < kl; ++i) c.first_pat[K] += (int)binom_host(kSegL, i);
                items += (c.group * c.nl[K] + 63) / 64;
            }
            c.items[s] = items;
        }
    }
    if (groups > 0x3FFFFFFFull) return false;
    p.ngroup = (uint32_t)groups;
    return true;
}

bool all_passes(int omega, int n, Passes &ps) {
    const int pairs = std::min(n, omega - n);
    if (omega > kMaxWinOmega || pairs < 7) return false;
    const uint64_t dim = binom_host(omega, n);
    if (dim < (pairs == 7 ? kMinWinDim7 : kMinWinDim)) return false;
    int W[kMaxWinPasses];
    const int np = cut_orbits(omega, dim, W);
    if (np == 0) return false;
    int top = omega;
    for (int i = 0; i < np; ++i) {
        Pass &p = ps.win[i];
        p.W = W[i];
        p.w0 = top - W[i];
        p.U = omega - top;
        top = p.w0;
        if (!window_classes(omega, n, p)) return false;
    }
    ps.np = np;
    return segment_classes(omega, n, ps.seg);
}

size_t off_bytes(int qmin, int qmax, int W, size_t entry) {
    return align256(((size_t)(qmax - qmin + 1) << W) * entry);
}
size_t pass_bytes(const Pass &p) {
    return align256((size_t)p.ncls * sizeof(WinClass)) + off_bytes(p.qmin, p.qmax, p.W, sizeof(int64_t));
}

// Place of each state g of the window [w0, w0 + W) among the states of q
// pairs on its orbits and those below, its low part's rank left out.
template <typename I>
void fill_offsets(I *t, int qmin, int qmax, int w0, int W) {
    for (int q = qmin; q <= qmax; ++q) {
        size_t pos = (size_t)(q - qmin) << W;
        for (int K = 0; K <= W; ++K)
            for (unsigned g = 0; g < (1u << W); ++g) {
                if (__builtin_popcount(g) != K) continue;
                int64_t v = 0;
                int idx = q - K;   // pairs below the window (no such state when negative)
                for (int b = 0; b < W; ++b)
                    if ((g >> b) & 1u) v += (int64_t)binom_host(w0 + b, ++idx);
                t[pos++] = q >= K ? (I)v : 0;
            }
    }
}

}  // namespace

size_t window_plan_bytes(int omega, int n) {
    Passes ps;
    if (!all_passes(omega, n, ps)) return 0;
    size_t b = align256((size_t)ps.seg.ncls * sizeof(SegClass)) +
               off_bytes(ps.seg.qmin, ps.seg.qmax, kSegW, sizeof(int32_t));
    for (int i = 0; i < ps.np; ++i) b += pass_bytes(ps.win[i]);
    return b;
}

bool window_plan_build(int omega, int n, void *dev, WinPlan *plan, unsigned char *host) {
    Passes ps;
    if (!all_passes(omega, n, ps)) return false;
    unsigned char *d = static_cast<unsigned char *>(dev);
    size_t off = 0;
    auto put = [&](const void *from, size_t bytes) {   // at the next free place; returns its device address
        if (from) std::memcpy(host + off, from, bytes);
        const unsigned char *at = d + off;
        off += align256(bytes);
        return at;
    };
    std::memset(plan, 0, sizeof(*plan));
    const SegPlan &sg = ps.seg;
    plan->seg.nclass = sg.ncls;
    plan->seg.qmin = sg.qmin;
    plan->seg.cap = sg.cap;
    plan->seg.ngroup = sg.ngroup;
    plan->seg.cls = reinterpret_cast<const SegClass *>(put(sg.cls, (size_t)sg.ncls * sizeof(SegClass)));
    fill_offsets(reinterpret_cast<int32_t *>(host + off), sg.qmin, sg.qmax, kSegL, kSegW);
    plan->seg.off = reinterpret_cast<const int32_t *>(put(nullptr, ((size_t)(sg.qmax - sg.qmin + 1) << kSegW) * 4));
    for (int i = 0; i < ps.np; ++i) {
        const Pass &p = ps.win[i];
        WinPass &o = plan->pass[plan->npass++];
        o.nclass = p.ncls;
        o.nblocks = p.nblocks;
        o.W = p.W;
        o.w0 = p.w0;
        o.qmin = p.qmin;
        o.cls = reinterpret_cast<const WinClass *>(put(p.cls, (size_t)p.ncls * sizeof(WinClass)));
        fill_offsets(reinterpret_cast<int64_t *>(host + off), p.qmin, p.qmax, p.w0, p.W);
        o.off = reinterpret_cast<const int64_t *>(put(nullptr, ((size_t)(p.qmax - p.qmin + 1) << p.W) * 8));
    }
    return true;
}

}  // namespace pd
