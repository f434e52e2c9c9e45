// y = H x by orbit windows (Sec. 3.3): the product of large full spaces.
//
// The orbits are cut, from the top, into windows of W = 4..8 neighbouring
// orbits and the kSeg = 16 lowest ones.  One pass per window takes every hop
// with at least one end in the window and none above it, and the segment pass takes
// the hops inside the lowest orbits and the diagonal, so each hop is taken once.
//
// Window pass.  A state is (s, g, l): the occupation of the orbits above the
// window, in it, and below it.  Colex ranks add up over the three parts:
//     rank = base(s) + off(g) + r(l),
// r(l) the rank of l among the states of its pair count on the low orbits.
// One lane owns (s, l) and all C(W, K) window states g of K pairs, whose
// results stay in its registers.  An element x(s, g', l') then serves
// every window state one hop away from it:
//   * l' = l: the hops inside the window, K (W - K) per element.  Element,
//     result and coupling are fixed at compile time and the coupling is the
//     same for all lanes (a scalar register);
//   * l' = l without j: K + 1 hops per element, l' = l with j: W - K + 1.
//     r(l') is found once per j and serves all window states; off(g') is the
//     same for all lanes, so a load's address is a scalar plus one register.
// An element is loaded once for up to 16 hops, where a product with a
// row per lane loads one per hop, and no address is computed per hop.
//
// Measured against a row per lane (32 orbits, 16 pairs, 6.0e8 rows x 256 hops, FP64):
// 82.9 -> 26.4 ms; 28 orbits, 14 pairs (4.0e7 rows) 3.98 -> 1.57 ms; 31 orbits, 17 pairs
// FP32 20.7 -> 6.25 ms.  Of the 26.4 ms the upper window takes 12.9, the next one 8.6
// and the segments 4.9.  The windows are bound by the address path of the L1: 26 and
// 18 loads per row and 27 and 25 cycles per load (a contiguous 8-byte load of 64
// lanes takes 16), 85% and 80% of the time; at the same time 65 and 26 GB come from below
// the L2s, 5 and 3 TB/s.  The arithmetic alone would take 4 ms.  In FP32 (14.5 ms) no
// unit is as busy, the addresser 66% and the VALU 46% of the time: three waves per SIMD
// leave latency bare.
#pragma once

#include <type_traits>
#include <utility>

#include "pd_internal.h"

namespace pd {
namespace win {

constexpr int cbinom(int a, int b) {
    if (b < 0 || b > a) return 0;
    long v = 1;
    for (int i = 0; i < b; ++i) v = v * (a - i) / (i + 1);
    return (int)v;
}
constexpr int cpop(unsigned v) {
    int c = 0;
    for (; v; v &= v - 1) ++c;
    return c;
}

// The states of K pairs on W orbits, ascending (colex) order, and the hops
// from and to them, grouped by the state they read.
template <int W, int K>
struct Tile {
    static constexpr int N = cbinom(W, K);
    struct List {
        int pat[N > 0 ? N : 1];
        int index[1 << W];
    };
    static constexpr List make() {
        List t{};
        int c = 0;
        for (int p = 0; p < (1 << W); ++p) {
            t.index[p] = 0;
            if (cpop(p) == K) {
                t.pat[c] = p;
                t.index[p] = c++;
            }
        }
        return t;
    }
    static constexpr List list = make();
    // position of the tile in a window's offset table (tiles of fewer pairs first)
    static constexpr int first() {
        int f = 0;
        for (int k = 0; k < K; ++k) f += cbinom(W, k);
        return f;
    }
};

// Hops of a window: element src of the tile of KP pairs adds coupling cpl times
// itself to result dst of the tile of K pairs.  KP == K: a hop inside the
// window, cpl = a * W + b; KP = K + 1: the pair leaves the window's orbit cpl;
// KP = K - 1: it enters orbit cpl.
template <int W, int K, int KP>
struct Hops {
    static constexpr int per = KP == K ? K * (W - K) : KP == K + 1 ? KP : W - KP;   // per element
    static constexpr int NS = cbinom(W, KP);
    static constexpr int N = NS * per;
    struct List {
        int dst[N > 0 ? N : 1], cpl[N > 0 ? N : 1];
    };
    static constexpr List make() {
        List t{};
        int c = 0;
        for (int s = 0; s < NS; ++s) {
            const int pat = Tile<W, KP>::list.pat[s];
            for (int o = 0; o < W; ++o) {
                if (KP == K) {
                    if (!((pat >> o) & 1)) continue;
                    for (int e = 0; e < W; ++e)
                        if (!((pat >> e) & 1)) {
                            t.dst[c] = Tile<W, K>::list.index[(pat & ~(1 << o)) | (1 << e)];
                            t.cpl[c++] = o < e ? o * W + e : e * W + o;
                        }
                } else if (((pat >> o) & 1) == (KP > K ? 1 : 0)) {
                    t.dst[c] = Tile<W, K>::list.index[pat ^ (1 << o)];
                    t.cpl[c++] = o;
                }
            }
        }
        return t;
    }
    static constexpr List list = make();
};

template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F &&f) {
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}
#define PD_INLINE __attribute__((always_inline))

// Read-only memory that the kernel does not write: a uniform address is read
// through the scalar cache, also after stores to y.
template <typename T>
using Const = const T __attribute__((address_space(4))) *;
template <typename T>
__device__ __forceinline__ Const<T> as_const(const T *p) {
    return (Const<T>)(uintptr_t)p;
}

// The same pointer (or number), which the compiler may not look through: what
// is read through it is read here, and not kept in registers from further up.
template <typename P>
__device__ __forceinline__ P here(P p) {
    asm volatile("" : "+s"(p));
    return p;
}

constexpr int kBlock = 256;

template <typename T>
struct WinArgs {
    int omega, n, w0, U;     // low orbits 0..w0-1, window w0..w0+W-1, U orbits above
    int nclass, qmin;
    const WinClass *__restrict__ cls;
    const int64_t *__restrict__ off;   // off[(q - qmin) << W | tile position]
    const T *__restrict__ x;
    T *__restrict__ y;
    const T *__restrict__ V;
};

// The first active lane's value, in scalar registers.
__device__ __forceinline__ int64_t first_lane64(int64_t v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ int64_t lane64(int64_t v, int lane) {
    const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)v, lane);
    const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), lane);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ int first_lane(int v) { return __builtin_amdgcn_readfirstlane(v); }
template <typename T>
using Global = T __attribute__((address_space(1))) *;
template <typename T>
__device__ __forceinline__ Global<T> first_lane_ptr(T *p) {
    return (Global<T>)first_lane64((int64_t)(uintptr_t)p);
}

// The element at a uniform address plus a lane's offset.  The sum of the
// uniform parts is kept out of sight, so that it is formed in scalar registers
// (the compiler would add the lane's part first, in vector ones).
template <typename T>
__device__ __forceinline__ Global<T> at(Global<T> uniform, uint32_t byte_off) {
    asm("" : "+s"(uniform));
    return (Global<T>)((Global<const char>)uniform + byte_off);
}

// Elements of a batch: a batch is asked for before the one ahead of it is
// multiplied.  Two batches make a chunk of a tile.  As many as the registers
// hold beside the results without spilling (FP64, W = 8: 140 registers of results);
// 7 or 12 instead of 10 were within 1% at 32 orbits.
template <typename T, int W>
constexpr int batch() {
    return sizeof(T) == 4 ? 14 : W == 8 ? 10 : W == 7 ? 9 : W == 6 ? 8 : 5;
}

// Batch b of the tile of KP pairs on W orbits, of elements at xb + off[] + voff.
template <typename T, int W, int KP, int B0, int NB>
__device__ __forceinline__ void load_batch(Global<const T> xb, Const<int64_t> off, uint32_t voff, T (&xv)[batch<T, W>()]) {
    constexpr int first = Tile<W, KP>::first();
#pragma unroll
    for (int i = 0; i < NB; ++i) xv[i] = *at<const T>(xb + off[first + B0 + i], voff);
}

// acc += couplings times the batch.
template <typename T, int W, int K, int KP, int B0, int NB, int NC>
__device__ __forceinline__ void take_batch(const T (&xv)[batch<T, W>()], const T (&v)[NC], T (&acc)[cbinom(W, K)]) {
    using H = Hops<W, K, KP>;
#pragma unroll
    for (int i = 0; i < NB * H::per; ++i)
        acc[H::list.dst[B0 * H::per + i]] += v[H::list.cpl[B0 * H::per + i]] * xv[i / H::per];
}

// One tile at one offset (the hops inside the window).
template <typename T, int W, int K>
__device__ __forceinline__ void take_tile(Global<const T> xb, Const<int64_t> off, uint32_t voff, const T (&v)[W * W],
                                          T (&acc)[cbinom(W, K)]) {
    constexpr int kBatch = batch<T, W>(), N = cbinom(W, K), NB = (N + kBatch - 1) / kBatch;
    T xv[2][kBatch];
    off = here(off);
    load_batch<T, W, K, 0, (N < kBatch ? N : kBatch)>(xb, off, voff, xv[0]);
    static_for<NB>([&](auto bc) PD_INLINE {
        constexpr int b = decltype(bc)::value, b0 = b * kBatch, b1 = b0 + kBatch;
        constexpr int nb = N - b0 < kBatch ? N - b0 : kBatch, nn = N - b1 < kBatch ? N - b1 : kBatch;
        if constexpr (nn > 0) load_batch<T, W, K, b1, nn>(xb, off, voff, xv[(b + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);
        take_batch<T, W, K, K, b0, nb>(xv[b & 1], v, acc);
        __builtin_amdgcn_sched_barrier(0);
    });
}

// The hops between the window and the low orbits of one kind: low orbits
// number from..to - 1, found one by one by next(j, r'), each with the tile of KP pairs.  The
// tile is taken in chunks, all steps for one chunk before the next: the lanes
// in flight then keep to kChunk rows of x for a while, which their XCD's L2 can
// hold, and an element is read from it for most of its uses (32 orbits FP64, before
// the segment pass took the lowest orbits: 44 ms tile by tile, 40 by chunks).
template <typename T, int W, int K, int KP, typename Start, typename Next>
__device__ __forceinline__ void take_steps(Global<const T> xb, Const<int64_t> off, uint32_t rel, int from, int to,
                                           const T *Vs, T (&acc)[cbinom(W, K)], Start &&start, Next &&next) {
    constexpr int kBatch = batch<T, W>(), kChunk = 2 * kBatch, N = cbinom(W, KP), NCH = (N + kChunk - 1) / kChunk;
    if (from >= to) return;
    static_for<NCH>([&](auto cc) PD_INLINE {
        constexpr int b0 = decltype(cc)::value * kChunk, b1 = b0 + kBatch;
        constexpr int n0 = N - b0 < kBatch ? N - b0 : kBatch;
        constexpr int n1 = N - b1 < 0 ? 0 : N - b1 < kBatch ? N - b1 : kBatch;
        T xv[2][kBatch];
        int j;
        uint32_t rp;
        start();
        for (int a = 0; a < from; ++a) next(a, j, rp);
        next(from, j, rp);
        load_batch<T, W, KP, b0, n0>(xb, here(off), (rel + rp) * (uint32_t)sizeof(T), xv[0]);
        for (int a = from; a < to; ++a) {
            T v[W];
#pragma unroll
            for (int i = 0; i < W; ++i) v[i] = Vs[j * W + i];
            const uint32_t voff = (rel + rp) * (uint32_t)sizeof(T);
            if constexpr (n1 > 0) {
                load_batch<T, W, KP, b1, n1>(xb, here(off), voff, xv[1]);
                __builtin_amdgcn_sched_barrier(0);
                take_batch<T, W, K, KP, b0, n0>(xv[0], v, acc);
                __builtin_amdgcn_sched_barrier(0);
                if (a + 1 < to) {
                    next(a + 1, j, rp);
                    load_batch<T, W, KP, b0, n0>(xb, here(off), (rel + rp) * (uint32_t)sizeof(T), xv[0]);
                }
                __builtin_amdgcn_sched_barrier(0);
                take_batch<T, W, K, KP, b1, n1>(xv[1], v, acc);
            } else {
                T xc[kBatch];
#pragma unroll
                for (int i = 0; i < n0; ++i) xc[i] = xv[0][i];
                take_batch<T, W, K, KP, b0, n0>(xc, v, acc);
                if (a + 1 < to) {
                    next(a + 1, j, rp);
                    load_batch<T, W, KP, b0, n0>(xb, here(off), (rel + rp) * (uint32_t)sizeof(T), xv[0]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    });
}

// The lane's (s, l): s as its base rank relative to xb / yb (a scalar base of
// the wave), l as its rank r and its word.  With PARTS = 2 two waves share the lanes'
// work, as evenly as whole steps allow; the second (part 1) hands its sums over
// in LDS, ex, which the slots of pre are a part of.
template <typename T, int W, int K, int PARTS>
__device__ __forceinline__ void window_rows(const WinArgs<T> &A, int nl, int q, int64_t ub, uint32_t rel, uint32_t r,
                                            uint32_t lw, const uint32_t *Ct, int ks, const T *Vs, uint32_t *pre,
                                            int part, bool write, T *ex) {
    using TK = Tile<W, K>;
    constexpr int N = TK::N;
    T acc[N];
#pragma unroll
    for (int i = 0; i < N; ++i) acc[i] = T(0);
    const Const<int64_t> off = as_const(A.off) + ((int64_t)(q - A.qmin) << W);
    const Global<const T> xb = first_lane_ptr(A.x + ub);

    // the steps of this part; the cost of a step is its tile's number of elements
    const int ne = A.w0 - nl;
    int o0 = 0, o1 = nl, e0 = 0, e1 = ne;
    if constexpr (PARTS == 2) {
        constexpr int inside = K > 0 && K < W ? N : 0, co = cbinom(W, K + 1), ce = cbinom(W, K - 1);
        int left = ((inside + nl * co + ne * ce) >> 1) - inside;
        const int ho = co > 0 ? max(0, min(nl, (left + co / 2) / (co > 0 ? co : 1))) : 0;
        left -= ho * co;
        const int he = ce > 0 && (ho == nl || co == 0) ? max(0, min(ne, (left + ce / 2) / (ce > 0 ? ce : 1))) : 0;
        if (part == 0) o1 = ho, e1 = he;
        else o0 = ho, e0 = he;
    }

    // hops inside the window
    if constexpr (K > 0 && K < W) if (part == 0) {
        const Const<T> V = as_const(A.V);
        T vw[W * W];
#pragma unroll
        for (int i = 0; i < W; ++i)
#pragma unroll
            for (int j = i + 1; j < W; ++j) vw[i * W + j] = V[(A.w0 + i) * A.omega + A.w0 + j];
        take_tile<T, W, K>(xb, off, (rel + r) * (uint32_t)sizeof(T), vw, acc);
    }

    // l' = l without its occupied orbit j (from the top; j is the idx-th
    // occupied orbit from below): r' = r - C(j, idx) - sum over the occupied p
    // above j of C(p, i) - C(p, i - 1).  The sums that the empty orbits need,
    // one per count a of occupied orbits above, go to the lane's LDS slots.
    {
        uint32_t occ = lw, up = 0;
        pre[0] = 0;
        for (int a = 0; a < nl; ++a) {
            const int j = 31 - __clz((int)occ);
            occ &= ~(1u << j);
            const uint32_t *c = Ct + j * ks + (nl - a);
            up += c[1] - c[0];
            pre[(a + 1) * (PARTS * kBlock)] = up;
        }
    }
    if constexpr (K < W) {
        uint32_t occ, down;
        take_steps<T, W, K, K + 1>(
            xb, off, rel, o0, o1, Vs, acc,
            [&]() PD_INLINE {
                occ = lw;
                down = 0;
            },
            [&](int a, int &j, uint32_t &rp) PD_INLINE {
                j = 31 - __clz((int)occ);
                occ &= ~(1u << j);
                const uint32_t *c = Ct + j * ks + (nl - a);
                const uint32_t c0 = c[0], cm = c[-1];
                rp = r - c0 - down;
                down += c0 - cm;
            });
    }
    // l' = l with its empty orbit j
    if constexpr (K > 0) {
        uint32_t emp;
        take_steps<T, W, K, K - 1>(
            xb, off, rel, e0, e1, Vs, acc,
            [&]() PD_INLINE { emp = ~lw & (A.w0 >= 32 ? ~0u : (1u << A.w0) - 1); },
            [&](int e, int &j, uint32_t &rp) PD_INLINE {
                j = 31 - __clz((int)emp);
                emp &= ~(1u << j);
                const int a = A.w0 - 1 - j - e;   // occupied orbits above j
                rp = r + Ct[j * ks + nl - a + 1] + pre[a * (PARTS * kBlock)];
            });
    }

    if constexpr (PARTS == 2) {
        __syncthreads();
        if (part == 1) {
#pragma unroll
            for (int i = 0; i < N; ++i) ex[i * kBlock] = acc[i];
        }
        __syncthreads();
        if (part == 1 || !write) return;
#pragma unroll
        for (int i = 0; i < N; ++i) acc[i] += ex[i * kBlock];
    }
    const Global<T> yb = first_lane_ptr(A.y + ub);
    const uint32_t vo = (rel + r) * (uint32_t)sizeof(T);
    constexpr int first = TK::first();
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const Global<T> p = at<T>(yb + off[first + i], vo);
        *p += acc[i];
    }
}

// Workgroups go to the eight XCDs in turn; each XCD's are given a run of
// kXcdRun neighbouring blocks, as many as it holds at once, so that the lanes
// that share its L2 have neighbouring low states and read the same elements
// (32 orbits: runs of 1, 32, 64 and 128 took 40.6, 39.8, 40.2 and 41.1 ms, then).
constexpr uint32_t kXcdRun = 64;
__device__ __forceinline__ uint32_t xcd_block(uint32_t b, uint32_t grid) {
    constexpr uint32_t group = 8 * kXcdRun;
    const uint32_t g0 = b / group * group;
    if (g0 + group > grid) return b;
    const uint32_t i = b - g0;
    return g0 + (i & 7) * kXcdRun + (i >> 3);
}

// LDS of a window workgroup: binomials of the low orbits, ranks and bases of
// the upper ones, couplings between low orbits and window, the lanes' slots.
struct WinLds {
    int ks, us;
    size_t vs, ur, ub, pre, total;
};
template <typename T>
__host__ __device__ inline WinLds win_lds(int n, int w0, int U, int W, int parts) {
    WinLds L;
    const int nl = n < w0 ? n : w0, m = n < U ? n : U;
    L.ks = nl + 2;
    L.us = m + 1;
    size_t o = 0;
    L.vs = o;
    o += (size_t)w0 * W * sizeof(T);
    o = (o + 15) & ~size_t(15);
    L.ub = o;
    o += (size_t)U * L.us * 8;
    L.ur = o;
    o += (size_t)U * L.us * 4;
    L.pre = o;   // binomials of the low orbits, then the slots
    o += (size_t)w0 * L.ks * 4 + (size_t)(nl + 1) * parts * kBlock * 4;
    if (parts == 2) {   // the sums handed over, in the same place
        const size_t e = L.pre + (size_t)cbinom(W, W / 2) * kBlock * sizeof(T);
        if (o < e) o = e;
    }
    L.total = o;
    return L;
}

template <typename T, int W, int PARTS>
__global__ __launch_bounds__(kBlock * PARTS, PARTS == 2 || (sizeof(T) == 8 && W == 8) ? 2
                                             : sizeof(T) == 8 && W == 7 || W == 8     ? 3
                                                                                      : 4) void window_kernel(WinArgs<T> A) {
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t block = xcd_block(blockIdx.x, gridDim.x);
    // class of this workgroup
    int c = 0;
    {
        int hi = A.nclass;
        while (hi - c > 1) {
            const int mid = (c + hi) >> 1;
            if (as_const(A.cls)[mid].first_block <= block) c = mid;
            else hi = mid;
        }
    }
    const Const<WinClass> cp = as_const(A.cls) + c;
    const WinClass C = {cp->first_block, cp->lanes, cp->NL, cp->reach, cp->K, cp->m, cp->nl, 0};
    const int nl = C.nl, m = C.m, q = A.n - m;
    const WinLds L = win_lds<T>(A.n, A.w0, A.U, W, PARTS);
    T *Vs = reinterpret_cast<T *>(smem + L.vs);
    uint64_t *Ub = reinterpret_cast<uint64_t *>(smem + L.ub);
    uint32_t *Ur = reinterpret_cast<uint32_t *>(smem + L.ur);
    uint32_t *Ct = reinterpret_cast<uint32_t *>(smem + L.pre);
    uint32_t *pre = Ct + A.w0 * L.ks + threadIdx.x;
    for (int i = threadIdx.x; i < A.w0 * W; i += kBlock * PARTS) Vs[i] = A.V[(A.w0 + i % W) * A.omega + i / W];
    for (int i = threadIdx.x; i < A.U * L.us; i += kBlock * PARTS) {
        const int p = i / L.us, k = i - p * L.us;
        Ur[i] = (uint32_t)g_binom.v[p][k];
        Ub[i] = g_binom.v[A.w0 + W + p][q + k];
    }
    for (int i = threadIdx.x; i < A.w0 * L.ks; i += kBlock * PARTS) {
        const int p = i / L.ks, k = i - p * L.ks;
        Ct[i] = (uint32_t)g_binom.v[p][k];
    }
    __syncthreads();
    const int part = PARTS == 2 ? first_lane((int)(threadIdx.x / kBlock)) : 0;
    uint32_t f = (block - C.first_block) * kBlock + threadIdx.x % kBlock;
    const bool write = f < C.lanes;
    if (PARTS == 2) f = write ? f : C.lanes - 1;   // barriers ahead
    else if (!write) return;
    const uint32_t si = f / C.NL, r = f - si * C.NL;
    // base of the upper state of rank si
    int64_t base = 0;
    {
        uint32_t rem = si;
        int k = m;
        for (int p = A.U - 1; p >= 0; --p) {
            const uint32_t cc = Ur[p * L.us + k];
            if (k > 0 && cc <= rem) {
                rem -= cc;
                base += (int64_t)Ub[p * L.us + k];
                --k;
            }
        }
    }
    uint32_t lw = 0;
    {
        uint32_t rem = r;
        int k = nl;
        for (int p = A.w0 - 1; p >= 0; --p) {
            const uint32_t cc = Ct[p * L.ks + k];
            const bool take = cc <= rem && k > 0;
            rem -= take ? cc : 0u;
            k -= take ? 1 : 0;
            lw |= take ? (1u << p) : 0u;
        }
    }
    T *ex = reinterpret_cast<T *>(smem + L.pre) + threadIdx.x % kBlock;
    auto rows = [&](int64_t ub, uint32_t rel) PD_INLINE {
        switch (C.K) {
#define PD_WIN_CASE(KK)                                                                                             \
    case KK:                                                                                                        \
        if constexpr (KK <= W)                                                                                      \
            window_rows<T, W, KK, PARTS>(A, nl, q, ub, rel, r, lw, Ct, L.ks, Vs, pre, part, write, ex);             \
        break;
            PD_WIN_CASE(0) PD_WIN_CASE(1) PD_WIN_CASE(2) PD_WIN_CASE(3) PD_WIN_CASE(4) PD_WIN_CASE(5)
            PD_WIN_CASE(6) PD_WIN_CASE(7) PD_WIN_CASE(8)
#undef PD_WIN_CASE
        }
    };
    if constexpr (PARTS == 2) {
        rows(0, (uint32_t)base);   // fewer than kSplitBlocks * 256 * 70 states
    } else {
        // Lanes whose base lies within 32 bits of the first one's go together
        // (all of them except at the ends of very large spaces).  The loop's condition is
        // the wave's, not the lane's: a loop that each lane left behind its own rows
        // could have the rows moved behind it, where lanes of different ub meet again.
        uint64_t pending = __ballot(1);
        const int lane = threadIdx.x & 63;
        while (pending) {
            const int64_t ub = lane64(base, __builtin_ctzll(pending));
            const uint64_t rel = (uint64_t)(base - ub);
            const bool mine = ((pending >> lane) & 1) && (rel + C.reach) * sizeof(T) <= 0xFFFFFFFFull;
            const uint64_t taken = __ballot(mine);
            if (mine) rows(ub, (uint32_t)rel);
            pending &= ~taken;
        }
    }
}

// ---------------------------------------------------------------- segment pass
// The kSeg lowest orbits: their own hops and the whole diagonal.  The states
// that share the occupation u of the orbits above are one run of x, a segment
// of at most C(16, 8) = 12870 elements, which a workgroup keeps in LDS.  The
// segment is a window of kSegW orbits over kSegL low ones, taken as in
// the window pass: a lane owns a low state l and all window states g of K pairs.
// The hops inside the low orbits read C(kSegW, K) elements each at one rank.
// Short segments of one pair count go through LDS together, as a group.
// While an FP64 segment is worked on, the next one is on its way into registers;
// in FP32 two workgroups share a CU, and one loads while the other works.
// Bound by LDS reads: 45 per row, 4 cycles per wave and FP64 read, 2.8 of 4.9 ms at 32
// orbits.  It replaced a third window of 8 and an 8-orbit pass: 40 -> 28.8 ms at
// 32 orbits (FP64), and groups of short segments made that 26.3.
constexpr int kSegThreads = 512;
constexpr int kSegFetch = (12870 + kSegThreads - 1) / kSegThreads;

template <typename T>
struct SegArgs {
    int omega, n, nclass, qmin, cap;
    uint32_t ngroup;
    const SegClass *__restrict__ cls;
    const int32_t *__restrict__ off;   // off[(q - qmin) << kSegW | tile position]
    const T *__restrict__ x;
    T *__restrict__ y;
    const T *__restrict__ V;
    const T *__restrict__ d;
};

struct SegLds {
    int us;
    size_t ur, vw, vl, dw, dl, du, gd, gb, rank, pat, total;
};
template <typename T>
__host__ __device__ inline SegLds seg_lds(int omega, int n, int cap) {
    SegLds L;
    const int U = omega - kSeg;
    L.us = (n < U ? n : U) + 1;
    size_t o = ((size_t)cap * sizeof(T) + 15) & ~size_t(15);
    L.vw = o;
    o += (size_t)kSegL * 8 * sizeof(T);
    L.ur = o;
    o += ((size_t)U * L.us * 4 + 15) & ~size_t(15);
    L.vl = o;
    o += (size_t)kSegL * 16 * sizeof(T);
    L.dw = o;
    o += (size_t)(1 << kSegW) * sizeof(T);
    L.dl = o;
    o += (size_t)(1 << kSegL) * sizeof(T);
    L.du = o;
    o += 64 * sizeof(T);
    L.gd = o;
    o += 3 * kSegGroup * sizeof(T);
    o = (o + 15) & ~size_t(15);
    L.gb = o;
    o += 3 * kSegGroup * sizeof(int64_t);
    L.rank = o;
    o += (size_t)(1 << kSegL) * 2;
    L.pat = o;
    o += (size_t)(1 << kSegL) * 2;
    L.total = o;
    return L;
}

// What a lane of the segment pass works with.
template <typename T>
struct SegLane {
    const T *xs, *vw, *vl, *dw;
    const uint16_t *rank;
    uint32_t seg0, r, lw;   // the segment's place in LDS, the low state's rank and word
    T *y;          // the segment's results
    T diag;        // of the orbits above the window and the low ones
    bool write;
};

template <typename T, int K>
__device__ __forceinline__ void segment_rows(const SegArgs<T> &A, const SegLane<T> &S, Const<int32_t> off) {
    constexpr int W = kSegW;
    using TK = Tile<W, K>;
    constexpr int N = TK::N;
    T acc[N];
    {
        const Const<int32_t> o = here(off) + TK::first();
        const Const<T> V = as_const(A.V);
        T vw[W * W];
#pragma unroll
        for (int i = 0; i < W; ++i)
#pragma unroll
            for (int j = i + 1; j < W; ++j) vw[i * W + j] = V[(kSegL + i) * A.omega + kSegL + j];
        T xv[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            xv[i] = S.xs[o[i] + (S.seg0 + S.r)];
            acc[i] = (S.diag + S.dw[TK::list.pat[i]]) * xv[i];
        }
        using H = Hops<W, K, K>;
#pragma unroll
        for (int h = 0; h < H::N; ++h) acc[H::list.dst[h]] += vw[H::list.cpl[h]] * xv[h / (H::per > 0 ? H::per : 1)];
    }
    __builtin_amdgcn_sched_barrier(0);
    // window to low orbits and back
    if constexpr (K < W) {
        using H = Hops<W, K, K + 1>;
        const Const<int32_t> o = here(off) + Tile<W, K + 1>::first();
        for (uint32_t occ = S.lw; occ;) {
            const int j = 31 - __clz((int)occ);
            occ &= ~(1u << j);
            const uint32_t rp = S.seg0 + S.rank[S.lw ^ (1u << j)];
            T v[W], xv[H::NS];
#pragma unroll
            for (int i = 0; i < W; ++i) v[i] = S.vw[j * 8 + i];
#pragma unroll
            for (int i = 0; i < H::NS; ++i) xv[i] = S.xs[o[i] + rp];
#pragma unroll
            for (int h = 0; h < H::N; ++h) acc[H::list.dst[h]] += v[H::list.cpl[h]] * xv[h / H::per];
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    const uint32_t full = (1u << kSegL) - 1;
    if constexpr (K > 0) {
        using H = Hops<W, K, K - 1>;
        const Const<int32_t> o = here(off) + Tile<W, K - 1>::first();
        for (uint32_t emp = ~S.lw & full; emp;) {
            const int j = 31 - __clz((int)emp);
            emp &= ~(1u << j);
            const uint32_t rp = S.seg0 + S.rank[S.lw ^ (1u << j)];
            T v[W], xv[H::NS];
#pragma unroll
            for (int i = 0; i < W; ++i) v[i] = S.vw[j * 8 + i];
#pragma unroll
            for (int i = 0; i < H::NS; ++i) xv[i] = S.xs[o[i] + rp];
#pragma unroll
            for (int h = 0; h < H::N; ++h) acc[H::list.dst[h]] += v[H::list.cpl[h]] * xv[h / H::per];
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    // inside the low orbits
    const Const<int32_t> o = here(off) + TK::first();
    for (uint32_t occ = S.lw; occ;) {
        const int j = 31 - __clz((int)occ);
        occ &= ~(1u << j);
        for (uint32_t emp = ~S.lw & full; emp;) {
            const int e = 31 - __clz((int)emp);
            emp &= ~(1u << e);
            const uint32_t rp = S.seg0 + S.rank[S.lw ^ (1u << j) ^ (1u << e)];
            const T c = S.vl[j * 16 + e];
            T xv[N];
#pragma unroll
            for (int i = 0; i < N; ++i) xv[i] = S.xs[o[i] + rp];
#pragma unroll
            for (int i = 0; i < N; ++i) acc[i] += c * xv[i];
        }
    }
    if (S.write) {
        T *y = S.y + S.r;
#pragma unroll
        for (int i = 0; i < N; ++i) y[o[i]] = acc[i];
    }
}

template <typename T>
__global__ __launch_bounds__(kSegThreads, sizeof(T) == 8 ? 2 : 4) void segment_kernel(SegArgs<T> A) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int next_item;
    const int tid = threadIdx.x, U = A.omega - kSeg;
    const SegLds L = seg_lds<T>(A.omega, A.n, A.cap);
    T *xs = reinterpret_cast<T *>(smem);
    T *vw = reinterpret_cast<T *>(smem + L.vw), *vl = reinterpret_cast<T *>(smem + L.vl);
    T *dw = reinterpret_cast<T *>(smem + L.dw), *dl = reinterpret_cast<T *>(smem + L.dl);
    T *du = reinterpret_cast<T *>(smem + L.du);
    uint32_t *Ur = reinterpret_cast<uint32_t *>(smem + L.ur);
    uint16_t *rank = reinterpret_cast<uint16_t *>(smem + L.rank), *pat = reinterpret_cast<uint16_t *>(smem + L.pat);
    for (int i = tid; i < kSegL * 8; i += kSegThreads)
        vw[i] = (i & 7) < kSegW ? A.V[(kSegL + (i & 7)) * A.omega + (i >> 3)] : T(0);
    for (int i = tid; i < kSegL * 16; i += kSegThreads)
        vl[i] = (i & 15) < kSegL ? A.V[(i >> 4) * A.omega + (i & 15)] : T(0);
    for (int i = tid; i < (1 << kSegW); i += kSegThreads) {
        T s = T(0);
        for (int p = 0; p < kSegW; ++p)
            if ((i >> p) & 1) s += A.d[kSegL + p];
        dw[i] = s;
    }
    if (tid < U) du[tid] = A.d[kSeg + tid];
    for (int i = tid; i < (1 << kSegL); i += kSegThreads) {
        // pattern i: its rank among those with as many bits, and where that one's list begins
        T s = T(0);
        int k = 0, r = 0, first = 0;
        for (int p = 0; p < kSegL; ++p)
            if ((i >> p) & 1) {
                s += A.d[p];
                r += (int)g_binom.v[p][++k];
            }
        for (int c = 0; c < k; ++c) first += (int)g_binom.v[kSegL][c];
        dl[i] = s;
        rank[i] = (uint16_t)r;
        pat[first + r] = (uint16_t)i;
    }
    for (int i = tid; i < U * L.us; i += kSegThreads) Ur[i] = (uint32_t)g_binom.v[i / L.us][i % L.us];
    __syncthreads();

    T *gd = reinterpret_cast<T *>(smem + L.gd);
    int64_t *gb = reinterpret_cast<int64_t *>(smem + L.gb);
    const Const<SegClass> classes = as_const(A.cls);
    auto class_of = [&](uint32_t g) PD_INLINE {
        int c = 0;
        while (c + 1 < A.nclass && classes[c + 1].first <= g) ++c;
        return classes + c;
    };
    auto count_of = [&](Const<SegClass> c, uint32_t g) PD_INLINE {   // segments of group g
        const uint32_t left = c->nseg - (g - c->first) * c->group;
        return (int)(left < (uint32_t)c->group ? left : (uint32_t)c->group);
    };
    // Where group g's segments begin in x, and the diagonal of their upper orbits.
    auto find = [&](uint32_t g, int slot) PD_INLINE {
        const Const<SegClass> c = class_of(g);
        if (tid >= count_of(c, g)) return;
        uint32_t rem = (g - c->first) * c->group + tid;
        int k = A.n - c->q;
        int64_t base = 0;
        T dup = T(0);
        for (int p = U - 1; p >= 0 && k > 0; --p) {
            const uint32_t cc = Ur[p * L.us + k];
            if (cc <= rem) {
                rem -= cc;
                base += (int64_t)g_binom.v[p + kSeg][c->q + k];
                dup += du[p];
                --k;
            }
        }
        gb[slot * kSegGroup + tid] = base;
        gd[slot * kSegGroup + tid] = dup;
    };
    constexpr bool kAhead = sizeof(T) == 8;
    T fetch[kSegFetch];
    int total = 0;   // elements asked for
    auto ask = [&](uint32_t g, int slot) PD_INLINE {
        const Const<SegClass> c = class_of(g);
        const int len = c->len, count = count_of(c, g);
        total = count * len;
        if (count == 1) {
            const Global<const T> xb = first_lane_ptr(A.x + gb[slot * kSegGroup]);
#pragma unroll
            for (int f = 0; f < kSegFetch; ++f)
                if (f * kSegThreads < total) {
                    const int left = total - f * kSegThreads;   // beyond the end: the run's last element again
                    fetch[f] = *at<const T>(xb + f * kSegThreads,
                                            (uint32_t)(tid < left ? tid : left - 1) * (uint32_t)sizeof(T));
                }
        } else {
            const uint32_t magic = c->magic;
#pragma unroll
            for (int f = 0; f < kSegFetch; ++f)
                if (f * kSegThreads < total) {
                    const int e0 = f * kSegThreads + tid, e = e0 < total ? e0 : total - 1;
                    const int sg = len == 1 ? e : (int)__umulhi((uint32_t)e, magic);
                    fetch[f] = A.x[gb[slot * kSegGroup + sg] + (e - sg * len)];
                }
        }
    };
    uint32_t g = blockIdx.x;
    if (g < A.ngroup) find(g, 0);
    if (g + gridDim.x < A.ngroup) find(g + gridDim.x, 1);
    __syncthreads();
    if (kAhead && g < A.ngroup) ask(g, 0);
    for (int slot = 0; g < A.ngroup; g += gridDim.x, slot = slot == 2 ? 0 : slot + 1) {
        const int slot1 = slot == 2 ? 0 : slot + 1, slot2 = slot1 == 2 ? 0 : slot1 + 1;
        if (!kAhead) ask(g, slot);
        // this group into LDS
#pragma unroll
        for (int f = 0; f < kSegFetch; ++f)
            if (tid < total - f * kSegThreads) xs[f * kSegThreads + tid] = fetch[f];
        if (tid == 0) next_item = 0;
        __syncthreads();
        if (kAhead && g + gridDim.x < A.ngroup) ask(g + gridDim.x, slot1);
        if (g + 2 * gridDim.x < A.ngroup) find(g + 2 * gridDim.x, slot2);
        const Const<SegClass> c = class_of(g);
        const int count = count_of(c, g);
        const Const<int32_t> off = as_const(A.off) + ((c->q - A.qmin) << kSegW);
        for (;;) {
            int it = 0;
            if ((tid & 63) == 0) it = atomicAdd(&next_item, 1);
            it = first_lane(it);
            if (it >= c->items[7]) break;
            int t = 0;
            while (it >= c->items[t]) ++t;
            if (t > 0) it -= c->items[t - 1];
            const int K = seg_order(t), NL = c->nl[K];
            const int f0 = it * 64 + (tid & 63), lanes = count * NL;
            const int f = f0 < lanes ? f0 : lanes - 1;
            const int sg = NL == 1 ? f : (int)__umulhi((uint32_t)f, c->lane_magic[K]);
            SegLane<T> S;
            S.write = f0 < lanes;
            S.seg0 = (uint32_t)(sg * c->len);
            S.r = (uint32_t)(f - sg * NL);
            S.lw = pat[c->first_pat[K] + S.r];
            S.xs = xs;
            S.vw = vw;
            S.vl = vl;
            S.dw = dw;
            S.rank = rank;
            S.diag = gd[slot * kSegGroup + sg] + dl[S.lw];
            S.y = A.y + gb[slot * kSegGroup + sg];
            switch (K) {
#define PD_SEG_CASE(KK) \
    case KK: segment_rows<T, KK>(A, S, off); break;
                PD_SEG_CASE(0) PD_SEG_CASE(1) PD_SEG_CASE(2) PD_SEG_CASE(3) PD_SEG_CASE(4) PD_SEG_CASE(5)
                PD_SEG_CASE(6) PD_SEG_CASE(7)
#undef PD_SEG_CASE
            }
        }
        __syncthreads();
    }
}

// A pass of fewer workgroups leaves wave slots empty (a CU holds two of W = 8 in
// FP64): two waves then share the lanes of each.  24 orbits, 12 pairs (257 workgroups): the
// product takes 97.9 / 77.6 us (FP64 / FP32) so and 104 / 87 without; 23 orbits, 11 pairs
// 66.7 / 54.4 and 71.8 / 60.3.  From 512 on, the slots are taken either way.  Built for the
// one window of 7 or 8 of spaces of 23 (11, 12 pairs) and 24 orbits (11 to 13); smaller ones take
// a row per lane, larger ones have more workgroups, and windows of 5 and 6 with it are untried.
constexpr uint32_t kSplitBlocks = 512;

template <typename T, int W>
hipError_t launch_window(const WinPass &ps, int omega, int n, const T *x, T *y, const T *V, hipStream_t s) {
    WinArgs<T> A;
    A.omega = omega;
    A.n = n;
    A.w0 = ps.w0;
    A.U = omega - ps.w0 - W;
    A.nclass = ps.nclass;
    A.qmin = ps.qmin;
    A.cls = ps.cls;
    A.off = ps.off;
    A.x = x;
    A.y = y;
    A.V = V;
    if constexpr (W >= 7) {
        if (ps.nblocks < kSplitBlocks) {
            const size_t lds = win_lds<T>(n, A.w0, A.U, W, 2).total;
            hipError_t e = hipSuccess;
            if (lds > 64 * 1024)
                e = hipFuncSetAttribute(reinterpret_cast<const void *>(&window_kernel<T, W, 2>),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 1024);
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL((window_kernel<T, W, 2>), dim3(ps.nblocks), dim3(2 * kBlock), lds, s, A);
            return hipGetLastError();
        }
    }
    const size_t lds = win_lds<T>(n, A.w0, A.U, W, 1).total;
    hipLaunchKernelGGL((window_kernel<T, W, 1>), dim3(ps.nblocks), dim3(kBlock), lds, s, A);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_product(const WinPlan &plan, int omega, int n, const T *d, const T *V, const T *x, T *y,
                          hipStream_t s) {
    SegArgs<T> A;
    A.omega = omega;
    A.n = n;
    A.nclass = plan.seg.nclass;
    A.qmin = plan.seg.qmin;
    A.cap = plan.seg.cap;
    A.ngroup = plan.seg.ngroup;
    A.cls = plan.seg.cls;
    A.off = plan.seg.off;
    A.x = x;
    A.y = y;
    A.V = V;
    A.d = d;
    const size_t lds = seg_lds<T>(omega, n, A.cap).total;
    // as many workgroups as the CUs hold at once
    const int per_cu = lds <= 80 * 1024 - 512 ? 2 : 1;
    const uint32_t grid = A.ngroup < (uint32_t)(256 * per_cu) ? A.ngroup : (uint32_t)(256 * per_cu);
    hipError_t e = hipSuccess;
    if (lds > 64 * 1024)
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(&segment_kernel<T>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 1024);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((segment_kernel<T>), dim3(grid), dim3(kSegThreads), lds, s, A);
    e = hipGetLastError();
    for (int i = 0; i < plan.npass && e == hipSuccess; ++i) {
        const WinPass &ps = plan.pass[i];
        switch (ps.W) {
            case 4: e = launch_window<T, 4>(ps, omega, n, x, y, V, s); break;
            case 5: e = launch_window<T, 5>(ps, omega, n, x, y, V, s); break;
            case 6: e = launch_window<T, 6>(ps, omega, n, x, y, V, s); break;
            case 7: e = launch_window<T, 7>(ps, omega, n, x, y, V, s); break;
            case 8: e = launch_window<T, 8>(ps, omega, n, x, y, V, s); break;
            default: e = hipErrorInvalidValue;
        }
    }
    return e;
}

}  // namespace win
}  // namespace pd
