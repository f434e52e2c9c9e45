// Many independent ground-state problems in one persistent launch.
//
// Each workgroup takes the next instance from a device work queue (one
// atomic counter over instances sorted largest-first by the host, i.e. the
// longest-processing-time order) and runs the whole restarted Lanczos
// iteration of Sec. 3.4 for it: the product (the same per-row hop code as
// the single-instance sigma, with its per-lane slots in dynamic LDS), Gram-Schmidt against all stored vectors
// (a second pass only when needed), the tridiagonal eigensolver (multisection by the 64
// lanes of a wave, inverse iteration by one), the restart, the convergence test of Eq. convergence
// and the occupation numbers -- all without returning to the host.  The
// Krylov vectors of an instance live in a per-workgroup slot of the caller's
// workspace and stay in L2 / the Infinity Cache for all but the largest
// instances.  The queue reset and the solver launch are captured into one
// HIP graph.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <map>
#include <mutex>
#include <numeric>
#include <vector>

#include "pd_internal.h"
#include "sigma_impl.h"
#include "tridiag.h"

namespace pd {
namespace batched {

constexpr int kMaxPairs = 12;    // min(n, omega - n) of a batched instance
constexpr int kMaxOmegaB = 32;   // orbits of a batched instance
constexpr int kMaxKrylovB = 32;  // Krylov vectors per cycle

struct Instance {
    int omega, n, nn, comp;
    int64_t dim;
    int64_t coef;     // offset (doubles) of d[omega] then V[omega*omega] in the coefficient array
    int64_t occ_off;  // offset (doubles) of this instance's occupations in the output
    uint64_t seed;
    int orig;         // index in the caller's order
    int m;            // Krylov vectors per cycle: min(krylov, dim)
    double dsum;      // sum of the pair energies
    double dscale;    // max |pair energy| (denominator guard of the residual)
    double eshift;    // energy of the original problem = eigenvalue here + eshift
};

struct Result {
    double E0, residual;
    int iterations, restarts, converged, pad;
    long long ticks;  // wall_clock64() ticks spent on the instance
};

struct Args {
    const Instance *inst;
    int count;
    int *counter;         // queue of the instances left to single workgroups (from level[1].end on)
    // The sorted table's first instances are solved by teams of workgroups: up to
    // level[0].end by the large ones, up to level[1].end by those of kMidTeam.
    struct Level {
        int teams, team_size;   // the grid is teams * team_size workgroups (teams = 0: no instances)
        int end;
        int *counter;           // queue
        int *flag;              // per team: one flag per member (Team::flag), zero at the start
        double *part;           // per team: 2 buffers x team_size x kMaxSums partial sums
        double *slots;          // per team: one slot
        int64_t slot_doubles;
    } level[2];
    int *error;           // set when a team barrier times out
    long long spin_limit;
    const double *coef;
    double *slots2;         // one slot per workgroup for the rest
    int64_t slot2_doubles;
    double tol;
    int max_restarts;
    Result *res;
    double *occ;
};

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    return v;
}

struct Shared {
    uint32_t Ct[kMaxOmegaB * (kMaxPairs + 2)];
    double Vs[kMaxOmegaB * kMaxOmegaB];
    double ds[kMaxOmegaB];
    double scratch[8 * (kMaxKrylovB + 2)];
    double alpha[kMaxKrylovB], beta[kMaxKrylovB], y[kMaxKrylovB];
    double c[kMaxKrylovB + 8], red[8];
    double sc[kMaxKrylovB + 1];   // column scales: q_j = sc[j] * (stored column j)
    double cs[kMaxKrylovB + 8];   // update coefficients of the stored columns
    double A[3 * kMaxKrylovB], v[kMaxKrylovB];
    double theta;
    int idx, flag, abort;
};

// The workgroups that solve one instance together (size 1 for small ones).
struct Team {
    int G, g;             // team size, member index
    int64_t r0, r1;       // rows owned by this member
    int *flag;            // flag[q]: the last exchange that member q has entered
    double *part;         // 2 x G x kMaxSums partial sums
    uint32_t *pre;        // the workgroup's per-lane LDS slots of the sigma
    int epoch;            // exchanges so far, the same for all members
    int one_xcd;          // all members share an L2
};

constexpr int kMaxSums = kMaxKrylovB + 2;
// s_getreg operand of the hardware register XCC_ID (20): the wave's XCD, 4 bits from bit 0.
constexpr int kXccId = 20 | (4 - 1) << 11;

// Values that members pass to each other go past the caches that the XCDs do
// not share, and are complete before the flag that announces them.
__device__ __forceinline__ void put(double *p, double v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double get(const double *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Sums nv values over the team, in the order of its members: sh.scratch
// [wave * kMaxSums + j] holds every wave's part, the totals land in out[0..nv)
// of every member.  With VISIBLE everything the members wrote before is also
// seen by all of them afterwards (a full barrier, nv may be 0).
// Each member announces its sums with a flag of its own and waits for all
// the others', so an exchange is one store and one load away; the fences, which
// write an XCD's L2 back, are left to the exchanges that pass vectors on.
// The wait is bounded: on a time-out the error flag is raised and every
// member abandons the instance, so the kernel always drains.
template <bool VISIBLE>
__device__ bool team_exchange(const Args &A, Team &T, int nv, Shared &sh, double *out) {
    const int tid = threadIdx.x, nw = blockDim.x >> 6;
    __syncthreads();
    double s = 0.0;
    if (tid < nv)
        for (int w = 0; w < nw; ++w) s += sh.scratch[w * kMaxSums + tid];
    if (T.G == 1) {
        if (tid < nv) out[tid] = s;
        __syncthreads();
        return true;
    }
    const int epoch = ++T.epoch;
    double *part = T.part + (int64_t)(epoch & 1) * T.G * kMaxSums;
    if (tid < nv) put(part + (int64_t)T.g * kMaxSums + tid, s);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (tid == 0) sh.abort = 0;
    __syncthreads();
    if (tid == 0) {
        if (VISIBLE && !T.one_xcd) __threadfence();
        __hip_atomic_store(T.flag + T.g, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    for (int q = tid; q < T.G; q += blockDim.x) {
        long long spins = 0;
        while (__hip_atomic_load(T.flag + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < epoch) {
            __builtin_amdgcn_s_sleep(1);
            if (++spins > A.spin_limit || ((spins & 63) == 0 && atomicAdd(A.error, 0) != 0)) {
                atomicExch(A.error, 1);
                sh.abort = 1;
                break;
            }
        }
    }
    __syncthreads();
    if (VISIBLE) {
        if (tid == 0) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        __syncthreads();
    }
    const bool ok = sh.abort == 0;
    if (tid < nv) {
        double t = 0.0;
        for (int q = 0; q < T.G; ++q) t += get(part + (int64_t)q * kMaxSums + tid);
        out[tid] = t;
    }
    __syncthreads();
    return ok;
}

// Every wave's sum of v into sum j of the next exchange.
__device__ __forceinline__ void put_sum(Shared &sh, int j, double v) {
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) sh.scratch[(threadIdx.x >> 6) * kMaxSums + j] = v;
}

template <int NN, bool COMP>
__device__ void wg_sigma_nn(const Instance &I, const Team &T, const Shared &sh, const double *x, double *y) {
    const int ks = I.nn + 2;
    for (int64_t row = T.r0 + threadIdx.x; row < T.r1; row += blockDim.x)
        y[row] = sigma_detail::sigma_row<uint32_t, double, NN, COMP, false, 0, true>(
            row, I.dim, I.omega, ks, sh.Ct, sh.Vs, sh.ds, I.dsum, x, T.pre, (int)blockDim.x,
            sigma_detail::x_resource<double>(x, I.dim));
}

// Instances arrive with n <= omega - n (the host maps the others to their
// particle-hole complement), so only the unmirrored kernels are needed.
__device__ void wg_sigma(const Instance &I, const Team &T, const Shared &sh, const double *x, double *y) {
    switch (I.nn) {
#define PD_B_CASE(K) \
    case K: wg_sigma_nn<K, false>(I, T, sh, x, y); break;
        PD_B_CASE(0) PD_B_CASE(1) PD_B_CASE(2) PD_B_CASE(3) PD_B_CASE(4) PD_B_CASE(5) PD_B_CASE(6) PD_B_CASE(7)
        PD_B_CASE(8) PD_B_CASE(9) PD_B_CASE(10) PD_B_CASE(11) PD_B_CASE(12)
#undef PD_B_CASE
        default: break;
    }
}

// One step of put_sums: of v[0..2 H) a lane keeps half and passes the other half
// on to its partner, OFF lanes away, which keeps that one.
template <int H, int OFF>
__device__ __forceinline__ double halve_sums(double (&v)[2 * H]) {
    const bool up = (threadIdx.x & OFF) != 0;
    double w[H];
#pragma unroll
    for (int i = 0; i < H; ++i) {
        const double keep = up ? v[i + H] : v[i], pass = up ? v[i] : v[i + H];
        w[i] = keep + __shfl_xor(pass, OFF, 64);
    }
    if constexpr (H > 1) {
        double (&half)[2 * (H / 2)] = w;
        return halve_sums<H / 2, OFF / 2>(half);
    } else {
        double t = w[0];
#pragma unroll
        for (int o = OFF / 2; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
        return t;
    }
}

// Every wave's sums of all[FIRST..FIRST + N) into those sums of the next exchange
// (N a power of two).  Halving the number of values with every step takes about
// N shuffles where a tree for each value takes 6 N.
template <int N, int FIRST, int LEN>
__device__ __forceinline__ void put_sums(Shared &sh, const double (&all)[LEN]) {
    const int lane = threadIdx.x & 63;
    double v[N];
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = all[FIRST + i];
    const double t = halve_sums<N / 2, 32>(v);
    if (lane % (64 / N) == 0) sh.scratch[(threadIdx.x >> 6) * kMaxSums + FIRST + lane / (64 / N)] = t;
}

// With ps = sp * p - da * qa - db * qb (the recurrence terms known before the
// projection): p = ps, sh.c[j] = Q[j] . ps for j < nc <= N, then sh.c[N] = ||ps||^2 and
// sh.c[N + 1] = ||sp * p||^2, all in one pass and one exchange.  Columns beyond nc repeat the last, so that all loads are unconditional.
template <int N>
__device__ __forceinline__ bool wg_project_n(const Args &A, Team &T, const double *Q, int64_t ld, int nc, double *p,
                                          double sp, const double *qa, double da, const double *qb, double db,
                                          Shared &sh) {
    double acc[N], nrm[2] = {0.0, 0.0};
#pragma unroll
    for (int j = 0; j < N; ++j) acc[j] = 0.0;
    for (int64_t i = T.r0 + threadIdx.x; i < T.r1; i += blockDim.x) {
        double ps = p[i];
        constexpr int H = N < 16 ? N : 16;
        double q[H];
        const double *qp = Q + i;
#pragma unroll
        for (int j = 0; j < H; ++j) {
            q[j] = *qp;
            qp += j + 1 < nc ? ld : 0;
        }
        const double pf = sp * ps;
        ps = pf - da * qa[i] - db * qb[i];
        p[i] = ps;
        nrm[0] += ps * ps;
        nrm[1] += pf * pf;
#pragma unroll
        for (int j = 0; j < H; ++j) acc[j] += q[j] * ps;
        if constexpr (N > H) {
#pragma unroll
            for (int j = H; j < N; ++j) {
                q[j - H] = *qp;
                qp += j + 1 < nc ? ld : 0;
            }
#pragma unroll
            for (int j = H; j < N; ++j) acc[j] += q[j - H] * ps;
        }
    }
    if constexpr (N == 24) {
        put_sums<16, 0>(sh, acc);
        put_sums<8, 16>(sh, acc);
    } else {
        put_sums<N, 0>(sh, acc);
    }
    put_sum(sh, N, nrm[0]);
    put_sum(sh, N + 1, nrm[1]);
    return team_exchange<false>(A, T, N + 2, sh, sh.c);
}

// The bound N of wg_project for nc columns.
__device__ __forceinline__ int project_bound(int nc) { return nc <= 8 ? 8 : nc <= 16 ? 16 : nc <= 24 ? 24 : 32; }

__device__ bool wg_project(const Args &A, Team &T, const double *Q, int64_t ld, int nc, double *p, double sp,
                           const double *qa, double da, const double *qb, double db, Shared &sh) {
    switch (project_bound(nc)) {
        case 8: return wg_project_n<8>(A, T, Q, ld, nc, p, sp, qa, da, qb, db, sh);
        case 16: return wg_project_n<16>(A, T, Q, ld, nc, p, sp, qa, da, qb, db, sh);
        case 24: return wg_project_n<24>(A, T, Q, ld, nc, p, sp, qa, da, qb, db, sh);
        default: return wg_project_n<32>(A, T, Q, ld, nc, p, sp, qa, da, qb, db, sh);
    }
}

// out = p - sum_{j < nc} (q_j . p) q_j with q_j = sc_j Qt_j and the raw dot
// products Qt_j . p in sh.c; ||out||^2 to sh.red[0], and out is seen by the whole
// team (it is the next product's input).  out may equal p.
__device__ bool wg_update_to(const Args &A, Team &T, const double *Q, int64_t ld, int nc, const double *p,
                             double *out, Shared &sh) {
    if ((int)threadIdx.x < kMaxKrylovB + 8)
        sh.cs[threadIdx.x] = (int)threadIdx.x < nc ? sh.sc[threadIdx.x] * sh.sc[threadIdx.x] * sh.c[threadIdx.x]
                                                   : 0.0;
    __syncthreads();
    double acc = 0.0;
    for (int64_t i = T.r0 + threadIdx.x; i < T.r1; i += blockDim.x) {
        double v = p[i];
        for (int j0 = 0; j0 < nc; j0 += 8) {
            double q[8];
#pragma unroll
            for (int jj = 0; jj < 8; ++jj) q[jj] = Q[(int64_t)(j0 + jj < nc ? j0 + jj : nc - 1) * ld + i];
#pragma unroll
            for (int jj = 0; jj < 8; ++jj) v -= q[jj] * sh.cs[j0 + jj];
        }
        out[i] = v;
        acc += v * v;
    }
    put_sum(sh, 0, acc);
    return team_exchange<true>(A, T, 1, sh, sh.red);
}

// out = a * in over the member's rows, seen by the whole team (out is read whole next).
__device__ bool wg_scale(const Args &A, Team &T, const double *in, double a, double *out, Shared &sh) {
    for (int64_t i = T.r0 + threadIdx.x; i < T.r1; i += blockDim.x) out[i] = a * in[i];
    return team_exchange<true>(A, T, 0, sh, sh.red);
}

__device__ void solve_instance(const Args &A, const Instance &I, double *slot, Team &T, Shared &sh) {
    const long long t_start = wall_clock64();
    const int omega = I.omega, ks = I.nn + 2;
    // stage tables (a barrier precedes any use)
    for (int i = threadIdx.x; i < omega * ks; i += blockDim.x) {
        int p = i / ks, k = i - p * ks;
        sh.Ct[i] = (uint32_t)g_binom.v[p][k];
    }
    const double *d = A.coef + I.coef;
    const double *V = d + kMaxOmegaB;
    for (int i = threadIdx.x; i < omega * omega; i += blockDim.x) sh.Vs[i] = V[i];
    for (int i = threadIdx.x; i < omega; i += blockDim.x) sh.ds[i] = d[i];

    const int64_t dim = I.dim;
    const int64_t ld = (dim + 63) & ~int64_t(63);
    {
        const int64_t chunk = ((dim + T.G - 1) / T.G + 63) & ~int64_t(63);
        T.r0 = (int64_t)T.g * chunk < dim ? (int64_t)T.g * chunk : dim;
        T.r1 = T.r0 + chunk < dim ? T.r0 + chunk : dim;
    }
    const int m = I.m;
    double *Q = slot;
    double *p = Q + (int64_t)m * ld;
    double *w = p + ld;

    int iterations = 0, cycle = 0;
    bool converged = false, final_check = false, ok = true;
    double residual = INFINITY, e0 = 0.0;

    // start: x_k = 2 u_k - 1 with u_k from SplitMix64 (seed, k)
    {
        double acc = 0.0;
        for (int64_t i = T.r0 + threadIdx.x; i < T.r1; i += blockDim.x) {
            uint64_t z = I.seed + (uint64_t)(i + 1) * 0x9E3779B97F4A7C15ull;
            z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
            z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
            z = z ^ (z >> 31);
            double v = 2.0 * ((double)(z >> 11) * 0x1.0p-53) - 1.0;
            w[i] = v;
            acc += v * v;
        }
        put_sum(sh, 0, acc);
        ok = team_exchange<false>(A, T, 1, sh, sh.red) && wg_scale(A, T, w, 1.0 / sqrt(sh.red[0]), Q, sh);
    }

    // Gram-Schmidt as in the single-instance solver: the recurrence terms
    // sigma q_k + beta_{k-1} q_{k-1} (sigma = alpha_{k-1}, or the previous
    // Ritz value) are subtracted first, one classical pass follows, and a
    // second one only when ||v|| < ||ps|| / sqrt(2) or ||v|| < ||H q_k|| / 128.
    // Columns are stored unnormalised with their scales in sh.sc.
    constexpr double kEta2 = 0.5, kTau2 = 1.0 / (128.0 * 128.0);
    double theta = 0.0;
    if (threadIdx.x == 0) sh.sc[0] = 1.0;
    __syncthreads();
    for (cycle = 0; ok; ++cycle) {
        int m_eff = m;
        double tnorm = 0.0;
        for (int k = 0; k < m; ++k) {
            const double *qk = Q + (int64_t)k * ld;
            wg_sigma(I, T, sh, qk, p);   // p: the member's rows, each by the thread that reads it next
            ++iterations;
            const double sigma = k > 0 ? sh.alpha[k - 1] : theta;
            const double da = sigma * sh.sc[k];
            const double db = k > 0 ? sh.beta[k - 1] * sh.sc[k - 1] : 0.0;
            if (!(ok = wg_project(A, T, Q, ld, k + 1, p, sh.sc[k], qk, da, k > 0 ? qk - ld : qk, db, sh))) break;
            const int at = project_bound(k + 1);
            const double nrm_ps = sh.c[at], nrm_hq = sh.c[at + 1];
            const double alpha = sigma + sh.sc[k] * sh.c[k];
            const bool store = k + 1 < m;
            double nrm_v = 0.0;
            if (store || k == 0) {
                double *out = store ? Q + (int64_t)(k + 1) * ld : w;
                if (!(ok = wg_update_to(A, T, Q, ld, k + 1, p, out, sh))) break;
                nrm_v = sh.red[0];
                if (!(nrm_v >= kEta2 * nrm_ps && nrm_v >= kTau2 * nrm_hq)) {
                    if (!(ok = wg_project(A, T, Q, ld, k + 1, out, 1.0, out, 0.0, out, 0.0, sh))) break;
                    if (!(ok = wg_update_to(A, T, Q, ld, k + 1, out, out, sh))) break;
                    nrm_v = sh.red[0];
                }
            }
            const double beta = sqrt(fmax(nrm_v, 0.0));
            if (threadIdx.x == 0) {
                sh.alpha[k] = alpha;
                sh.beta[k] = beta;
                if (store && beta > 0.0) sh.sc[k + 1] = 1.0 / beta;
            }
            // The next step reads these at once: a wave without rows has no product to
            // do first.  (Nobody reads them between the last exchange and here.)
            __syncthreads();
            if (k == 0) {
                e0 = alpha + I.eshift;
                residual = beta / fmax(fabs(e0), 1e-3 * I.dscale);
                if (residual <= A.tol) converged = true;
                if (converged || final_check) break;
            }
            if (!store) break;
            tnorm = fmax(tnorm, fabs(alpha) + beta);
            if (beta <= 1e-14 * fmax(tnorm, 1e-300)) {
                m_eff = k + 1;
                break;
            }
        }
        if (!ok || converged || final_check) break;
        __syncthreads();
        if (threadIdx.x < 64) {
#ifdef __HIP_DEVICE_COMPILE__
            const int st = tridiag_lowest_wave(m_eff, sh.alpha, sh.beta, &sh.theta, sh.y, sh.A, sh.v);
            if (threadIdx.x == 0) sh.flag = st;
#endif
        }
        __syncthreads();
        if (sh.flag != 0) break;
        theta = sh.theta;
        // psi = Q y, normalised, becomes q_1
        {
            double acc = 0.0;
            for (int64_t i = T.r0 + threadIdx.x; i < T.r1; i += blockDim.x) {
                double v = 0.0;
                for (int j = 0; j < m_eff; ++j) v += Q[(int64_t)j * ld + i] * (sh.y[j] * sh.sc[j]);
                w[i] = v;
                acc += v * v;
            }
            put_sum(sh, 0, acc);
            ok = team_exchange<false>(A, T, 1, sh, sh.red) && wg_scale(A, T, w, 1.0 / sqrt(sh.red[0]), Q, sh);
        }
        if (threadIdx.x == 0) sh.sc[0] = 1.0;
        __syncthreads();
        if (cycle >= A.max_restarts) final_check = true;
    }

    // occupations of q_1: <N_i> = 2 sum_k q_k^2 [orbit i occupied]
    for (int i0 = 0; ok && i0 < omega; i0 += 8) {
        double acc[8];
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) acc[jj] = 0.0;
        for (int64_t r = T.r0 + threadIdx.x; r < T.r1; r += blockDim.x) {
            uint64_t s = 0, rem = (uint64_t)r;
            int kk = I.n;
            for (int q = omega - 1; q >= 0; --q) {
                uint64_t c = g_binom.v[q][kk];
                if (kk > 0 && c <= rem) {
                    s |= 1ull << q;
                    rem -= c;
                    --kk;
                }
            }
            const double wq = Q[r] * Q[r];
#pragma unroll
            for (int jj = 0; jj < 8; ++jj) acc[jj] += ((s >> (i0 + jj)) & 1ull) ? wq : 0.0;
        }
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) put_sum(sh, jj, acc[jj]);
        if (!(ok = team_exchange<false>(A, T, 8, sh, sh.red))) break;
        if (T.g == 0 && (int)threadIdx.x < 8 && i0 + (int)threadIdx.x < omega)
            A.occ[I.occ_off + i0 + threadIdx.x] = 2.0 * sh.red[threadIdx.x];
        __syncthreads();
    }
    if (threadIdx.x == 0 && T.g == 0) {
        Result r;
        r.E0 = e0;
        r.residual = residual;
        r.iterations = iterations;
        r.restarts = cycle;
        r.converged = (ok && converged) ? 1 : 0;
        r.pad = ok ? 0 : 1;
        r.ticks = wall_clock64() - t_start;
        A.res[I.orig] = r;
    }
    __syncthreads();
}

// Dynamic LDS of the solver: the sigma's per-lane slots, 2 (kMaxPairs + 1)
// words per thread.
inline size_t batched_dyn_lds(int block) { return (size_t)2 * (kMaxPairs + 1) * block * sizeof(uint32_t); }

__global__ __launch_bounds__(512) void batched_kernel(Args A) {
    __shared__ Shared sh;
    extern __shared__ __align__(16) unsigned char bdyn[];
    // Levels 0 and 1: instances solved by a team of workgroups each (team =
    // workgroup id mod teams, member = id / teams: the members of a smaller team
    // all come from one larger team, and workgroup ids that are equal modulo 8 lie on
    // one XCD).  Level 2: the rest, one workgroup each.  A single call site of
    // solve_instance keeps one copy of the solver in the kernel.
    Team T;
    T.pre = reinterpret_cast<uint32_t *>(bdyn);
    T.epoch = 0;
    T.one_xcd = 0;
    int level = 0;
    for (;;) {
        int idx;
        double *slot;
        if (level < 2) {
            const Args::Level &L = A.level[level];
            if (L.teams == 0) {
                ++level;
                continue;
            }
            const int t = blockIdx.x % L.teams;
            T.G = L.team_size;
            T.g = blockIdx.x / L.teams;
            T.flag = L.flag + (int64_t)t * L.team_size;
            T.part = L.part + (int64_t)t * 2 * L.team_size * kMaxSums;
            // Member 0 takes the next instance and tells the others (the sum has no
            // other terms); whether they all run on one XCD is told by the mean and
            // the mean square of their XCD numbers.
            for (int w = threadIdx.x; w < (int)(blockDim.x >> 6); w += blockDim.x) {
                const int xcd = __builtin_amdgcn_s_getreg(kXccId);
                double *sum = sh.scratch + w * kMaxSums;
                sum[0] = T.g == 0 && w == 0 ? (double)atomicAdd(L.counter, 1) : 0.0;
                sum[1] = w == 0 ? (double)xcd : 0.0;
                sum[2] = w == 0 ? (double)(xcd * xcd) : 0.0;
            }
            T.one_xcd = 0;
            if (!team_exchange<false>(A, T, 3, sh, sh.red)) break;
            T.one_xcd = __builtin_amdgcn_readfirstlane(T.G * sh.red[2] == sh.red[1] * sh.red[1] ? 1 : 0);
            // uniform across the workgroup: keep it (and the instance record) in scalar registers
            idx = __builtin_amdgcn_readfirstlane((int)sh.red[0]);
            __syncthreads();
            if (idx >= L.end) {
                ++level;
                T.epoch = 0;
                continue;
            }
            slot = L.slots + (int64_t)t * L.slot_doubles;
        } else {
            T.G = 1;
            T.g = 0;
            T.flag = nullptr;
            T.part = nullptr;
            T.one_xcd = 0;
            if (threadIdx.x == 0) sh.idx = atomicAdd(A.counter, 1);
            __syncthreads();
            idx = __builtin_amdgcn_readfirstlane(sh.idx);
            __syncthreads();
            if (idx >= A.count) break;
            slot = A.slots2 + (int64_t)blockIdx.x * A.slot2_doubles;
        }
        solve_instance(A, A.inst[idx], slot, T, sh);
        if (level < 2) {
            if (threadIdx.x == 0) sh.flag = atomicAdd(A.error, 0);
            __syncthreads();
            if (sh.flag != 0) break;
        }
    }
}

__global__ void reset_queue(int *counter, int start, int *large, int *mid, int mid_start, int *flags, int nflags,
                            int *error) {
    for (int i = threadIdx.x; i < nflags; i += blockDim.x) flags[i] = 0;
    if (threadIdx.x == 0) {
        *counter = start;
        *large = 0;
        *mid = mid_start;
        *error = 0;
    }
}

}  // namespace batched
}  // namespace pd

// ------------------------------------------------------------------ host side
namespace pd {
namespace batched {
namespace {

int device_cus() {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 256;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) return 256;
    return cus;
}

constexpr int kSample = 32;

// Work of one restart cycle of instance i (products plus Gram-Schmidt).
double instance_cost(int omega, int n, int krylov) {
    const int nn = std::min(n, omega - n);
    const double dim = (double)binom_host(omega, n);
    const double m = std::min<double>(krylov, dim);
    return dim * ((double)nn * (omega - nn) + 1.0 + 2.0 * m);
}

// Schedule: with a full grid (a multiple of 64 workgroups), 8 teams of grid/8
// workgroups (fewer and larger ones when fewer than 5 instances go to teams)
// first solve the costliest instances (sorted order), then grid/kMidTeam teams of
// kMidTeam the next ones, and then every workgroup drains the rest alone.  Cost
// units are those of instance_cost (work of one product).  A team runs an
// instance at 93% of its workgroups' combined rate plus a fixed overhead per
// product (its exchanges), about 23 us for 32 workgroups and 13 us for 8 against
// the ~4.3e9 units/s of one, all measured.  A level takes the sum of its
// instances over its teams, and its costliest instance once more for
// teams that end at different times.  The split with the lowest predicted time is
// taken: small instances stay on single workgroups, where the exchanges would
// cost more than the work.  Measured, products of 64 instances at once: 3432
// states 22-25 us on teams of 8, 72-75 us alone; 12870 states 53-59 us on teams of 8,
// 38-41 us on teams of 32 of which there are a quarter as many (14.7 against 32.8 ms);
// 184756 states 735-880 against 201-209 us (304 against 223 ms).  128 instances of
// 45 to 184,756 states: 81 ms without the teams of 8, 67 ms with them.
constexpr double kTeamEff = 0.93;
constexpr double kTeamOverhead = 1.0e5, kMidOverhead = 5.5e4;
constexpr int kMidTeam = 8;
// The teams of 8 hold grid / 8 slots: up to this size (1.5 GB of them at krylov 20)
// their vectors stay in the Infinity Cache's reach and the workspace small.
constexpr int64_t kMidMaxDim = int64_t(1) << 18;
constexpr int kMaxCandidates = 256;
struct Schedule {
    int teams = 0, n_large = 0;      // the large teams and their instances [0, n_large)
    int mid_teams = 0, n_mid = 0;    // teams of kMidTeam: [n_large, n_large + n_mid)
};
Schedule plan_schedule(int count, const int *omega, const int *n, int krylov, int grid, const std::vector<int> &order) {
    Schedule S;
    if (grid < 64 || grid % 64 != 0) return S;
    const int nteams = 8, G = grid / nteams, nmid = grid / kMidTeam;
    std::vector<double> sum(count + 1, 0.0), cost(count + 1, 0.0);
    for (int i = 0; i < count; ++i) {
        cost[i] = instance_cost(omega[order[i]], n[order[i]], krylov);
        sum[i + 1] = sum[i] + cost[i];
    }
    const double rate = G * kTeamEff, mid_rate = kMidTeam * kTeamEff;
    std::vector<int64_t> dim(count + 1, 0);   // the largest of the instances from i on
    for (int i = count - 1; i >= 0; --i)
        dim[i] = std::max<int64_t>(dim[i + 1], (int64_t)binom_host(omega[order[i]], n[order[i]]));
    // candidates for the two splits: every count up to kMaxCandidates, evenly spread ones beyond
    const int step = (count + kMaxCandidates - 1) / kMaxCandidates;
    double best = 1e300;
    for (int a = 0;; a = std::min(a + step, count)) {
        const double t1 = a == 0 ? 0.0
                                 : (sum[a] / rate + a * kTeamOverhead) / nteams + cost[0] / rate + kTeamOverhead;
        for (int b = a;; b = std::min(b + step, count)) {
            if (b > a && dim[a] > kMidMaxDim) break;
            const double t2 = b == a ? 0.0
                                     : ((sum[b] - sum[a]) / mid_rate + (b - a) * kMidOverhead) / nmid +
                                           cost[a] / mid_rate + kMidOverhead;
            const double t = t1 + t2 + (sum[count] - sum[b]) / grid + cost[b];
            if (t < best) {
                best = t;
                S.n_large = a;
                S.n_mid = b - a;
            }
            if (b == count) break;
        }
        if (a == count) break;
    }
    // Fewer large instances than teams: the fewest teams (a power of two, so
    // it divides the grid) that still start every large instance at once;
    // idle teams would only hold their slots.  Measured: one instance of
    // 8.6e7 states 26.0 s on one of 8 teams of 32 workgroups, 3.9 s on one
    // team of all 256 (and 122 -> 15 GB of workspace); two of 3.0e7 states
    // 10.4 -> 2.8 s on two teams of 128.
    if (S.n_large > 0) {
        S.teams = 1;
        while (S.teams < S.n_large && S.teams < nteams) S.teams <<= 1;
    }
    if (S.n_mid > 0) S.mid_teams = nmid;
    return S;
}

struct Layout {
    size_t inst = 0, sample = 0, coef = 0, counter = 0, team_flag = 0, team_part = 0, res = 0, occ = 0, slots = 0,
           total = 0;
    int64_t slot_doubles = 0, mid_doubles = 0, slot2_doubles = 0, coef_doubles = 0, occ_doubles = 0;
    int grid = 0, m_max = 0;
    size_t slots_mid = 0, slots2 = 0;
    Schedule plan;
};


std::vector<int> cost_order(int count, const int *omega, const int *n, int krylov) {
    std::vector<double> cost(count);
    for (int i = 0; i < count; ++i) cost[i] = instance_cost(omega[i], n[i], krylov);
    std::vector<int> order(count);
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return cost[a] > cost[b]; });
    return order;
}

// Krylov columns and two more vectors of an instance of d states.
int64_t slot_for(int krylov, int64_t d) {
    const int64_t m = std::min<int64_t>(krylov, d), ld = (d + 63) & ~int64_t(63);
    return ((m + 2) * ld + 31) & ~int64_t(31);
}

Layout layout_for(int count, const int *omega, const int *n, int krylov) {
    Layout L;
    int64_t dmax = 1;
    for (int i = 0; i < count; ++i) {
        dmax = std::max<int64_t>(dmax, (int64_t)binom_host(omega[i], n[i]));
        L.coef_doubles += kMaxOmegaB + (int64_t)omega[i] * omega[i];
        L.occ_doubles += omega[i];
    }
    L.m_max = (int)std::min<int64_t>(krylov, dmax);
    // The whole device when teams are planned (a few large instances still
    // fill every compute unit); one workgroup per instance otherwise.
    L.grid = device_cus();
    const std::vector<int> order = cost_order(count, omega, n, krylov);
    L.plan = plan_schedule(count, omega, n, krylov, L.grid, order);
    const int n_large = L.plan.n_large, n_teams = n_large + L.plan.n_mid;
    if (n_teams == 0) L.grid = std::min(count, L.grid);
    // Slots fit the largest instance that they may hold (sorted costliest first).
    auto dim_of = [&](int q) { return (int64_t)binom_host(omega[order[q]], n[order[q]]); };
    int64_t d1 = 0, d2 = 0;
    for (int q = n_large; q < n_teams; ++q) d1 = std::max(d1, dim_of(q));
    for (int q = n_teams; q < count; ++q) d2 = std::max(d2, dim_of(q));
    L.slot_doubles = n_large > 0 ? slot_for(krylov, dmax) : 0;
    L.mid_doubles = d1 > 0 ? slot_for(krylov, d1) : 0;
    L.slot2_doubles = d2 > 0 ? slot_for(krylov, d2) : 0;
    size_t off = 0;
    L.inst = off;
    off += align256(sizeof(Instance) * (size_t)count);
    L.sample = off;
    off += align256(sizeof(Instance) * kSample);
    L.coef = off;
    off += align256(sizeof(double) * (size_t)L.coef_doubles);
    L.counter = off;    // single-workgroup queue at +0, large teams' at +64, error flag at +128, the others' at +192
    off += 256;
    L.team_flag = off;
    off += align256(sizeof(int) * 2 * (size_t)std::max(L.grid, 1));   // flags of both levels
    L.team_part = off;
    off += align256(sizeof(double) * 4 * kMaxSums * (size_t)std::max(L.grid, 1));   // sums of both levels
    L.res = off;
    off += align256(sizeof(Result) * (size_t)count);
    L.occ = off;
    off += align256(sizeof(double) * (size_t)L.occ_doubles);
    L.slots = off;
    off += align256(sizeof(double) * (size_t)L.slot_doubles * (size_t)L.plan.teams);
    L.slots_mid = off;
    off += align256(sizeof(double) * (size_t)L.mid_doubles * (size_t)L.plan.mid_teams);
    L.slots2 = off;
    off += sizeof(double) * (size_t)L.slot2_doubles * (size_t)L.grid;
    L.total = off;
    return L;
}

std::mutex g_tune_mu;
std::map<std::vector<int64_t>, int> g_tuned;

}  // namespace
}  // namespace batched

size_t batched_workspace_bytes(int count, const int *omega, const int *n, const pd_lanczos_opts *o) {
    return batched::layout_for(count, omega, n, o->krylov).total;
}

pd_status batched_validate(int count, const int *omega, const int *n, const pd_lanczos_opts *o) {
    if (count < 1) return fail(PD_EINVAL, "count must be >= 1");
    if (!omega || !n) return fail(PD_EINVAL, "omega and n must be host arrays");
    if (o->krylov < 2 || o->krylov > batched::kMaxKrylovB)
        return fail(PD_EINVAL, "batched krylov=%d outside [2, %d]", o->krylov, batched::kMaxKrylovB);
    for (int i = 0; i < count; ++i) {
        if (omega[i] < 1 || omega[i] > batched::kMaxOmegaB || n[i] < 0 || n[i] > omega[i])
            return fail(PD_EINVAL, "instance %d: omega=%d n=%d outside [1, %d] x [0, omega]", i, omega[i], n[i],
                        batched::kMaxOmegaB);
        if (std::min(n[i], omega[i] - n[i]) > batched::kMaxPairs)
            return fail(PD_ERANGE, "instance %d: min(n, omega-n) > %d", i, batched::kMaxPairs);
    }
    return PD_OK;
}

pd_status batched_run(int count, const int *omega, const int *n, const double *eps_packed, const double *V_packed,
                      const pd_lanczos_opts *o, int block, void *work, size_t work_bytes, double *E0_out,
                      double *occ_out, pd_lanczos_info *info_out, pd_batch_info *binfo, hipStream_t stream) {
    using namespace batched;
    auto t0 = std::chrono::steady_clock::now();
    {
        // static Shared plus the sigma's dynamic slots exceed the default 64 KB
        static bool raised = false;
        if (!raised) {
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&batched_kernel),
                                               hipFuncAttributeMaxDynamicSharedMemorySize,
                                               (int)batched_dyn_lds(512));
            if (e != hipSuccess) return fail(PD_EDEVICE, "batched kernel LDS: %s", hipGetErrorString(e));
            raised = true;
        }
    }
    Layout L = layout_for(count, omega, n, o->krylov);
    if (work_bytes < L.total) return fail(PD_ENOMEM, "workspace %zu bytes, need %zu", work_bytes, L.total);
    unsigned char *base = static_cast<unsigned char *>(work);

    // instances and coefficients (validated while packing)
    std::vector<Instance> inst(count);
    std::vector<char> flipped(count, 0);
    std::vector<double> coef((size_t)L.coef_doubles, 0.0);
    int64_t coff = 0, ooff = 0, eoff = 0, voff = 0;
    CoefBlock blk;
    for (int i = 0; i < count; ++i) {
        pd_status st = pack_coefficients(omega[i], n[i], eps_packed + eoff, V_packed + voff, &blk);
        if (st != PD_OK) return fail(st, "instance %d: %s", i, last_error());
        Instance &I = inst[i];
        // n > omega - n: solve the particle-hole complement (omega - n pairs,
        // pair energies -d_i, same V): H = (sum d) 1 + P H' P^T, so E0 = E0' + sum d
        // and <N_i> = 2 - <N_i>'.
        const bool flip = n[i] > omega[i] - n[i];
        flipped[i] = flip;
        I.omega = omega[i];
        I.n = flip ? omega[i] - n[i] : n[i];
        I.comp = 0;
        I.nn = I.n;
        I.dim = (int64_t)binom_host(omega[i], n[i]);
        I.eshift = flip ? blk.dsum64 : 0.0;
        I.coef = coff;
        I.occ_off = ooff;
        I.seed = o->seed + (uint64_t)i;
        I.orig = i;
        I.m = (int)std::min<int64_t>(o->krylov, I.dim);
        I.dsum = flip ? -blk.dsum64 : blk.dsum64;
        double sc = 0.0;
        for (int q = 0; q < omega[i]; ++q) {
            coef[coff + q] = flip ? -blk.d64[q] : blk.d64[q];
            sc = std::max(sc, std::fabs(blk.d64[q]));
        }
        I.dscale = sc > 0.0 ? sc : 1.0;
        for (int q = 0; q < omega[i] * omega[i]; ++q) coef[coff + kMaxOmegaB + q] = blk.V64[q];
        coff += kMaxOmegaB + (int64_t)omega[i] * omega[i];
        ooff += omega[i];
        eoff += omega[i];
        voff += (int64_t)omega[i] * omega[i];
    }
    const std::vector<int> order = cost_order(count, omega, n, o->krylov);
    std::vector<Instance> sorted(count);
    for (int i = 0; i < count; ++i) sorted[i] = inst[order[i]];

    Instance *d_inst = reinterpret_cast<Instance *>(base + L.inst);
    Instance *d_sample = reinterpret_cast<Instance *>(base + L.sample);
    double *d_coef = reinterpret_cast<double *>(base + L.coef);
    int *d_counter = reinterpret_cast<int *>(base + L.counter);
    int *d_large = reinterpret_cast<int *>(base + L.counter + 64);
    int *d_error = reinterpret_cast<int *>(base + L.counter + 128);
    int *d_mid = reinterpret_cast<int *>(base + L.counter + 192);
    int *d_team_flag = reinterpret_cast<int *>(base + L.team_flag);
    double *d_team_part = reinterpret_cast<double *>(base + L.team_part);
    Result *d_res = reinterpret_cast<Result *>(base + L.res);
    double *d_occ = reinterpret_cast<double *>(base + L.occ);
    double *d_slots = reinterpret_cast<double *>(base + L.slots);
    PD_HIP(hipMemcpyAsync(d_inst, sorted.data(), sizeof(Instance) * count, hipMemcpyHostToDevice, stream));
    PD_HIP(hipMemcpyAsync(d_coef, coef.data(), sizeof(double) * coef.size(), hipMemcpyHostToDevice, stream));
    PD_HIP(hipStreamSynchronize(stream));

    const Schedule &plan = L.plan;
    Args A;
    A.inst = d_inst;
    A.count = count;
    A.counter = d_counter;
    Args::Level &large = A.level[0], &mid = A.level[1];
    large.teams = plan.teams;
    large.team_size = plan.teams ? L.grid / plan.teams : 1;
    large.end = plan.n_large;
    large.counter = d_large;
    large.flag = d_team_flag;
    large.part = d_team_part;
    large.slots = d_slots;
    large.slot_doubles = L.slot_doubles;
    mid.teams = plan.mid_teams;
    mid.team_size = kMidTeam;
    mid.end = plan.n_large + plan.n_mid;
    mid.counter = d_mid;
    mid.flag = d_team_flag + L.grid;
    mid.part = d_team_part + (size_t)2 * kMaxSums * L.grid;
    mid.slots = reinterpret_cast<double *>(base + L.slots_mid);
    mid.slot_doubles = L.mid_doubles;
    A.error = d_error;
    A.spin_limit = 1ll << 25;
    A.coef = d_coef;
    A.slots2 = reinterpret_cast<double *>(base + L.slots2);
    A.slot2_doubles = L.slot2_doubles;
    A.tol = o->tol;
    A.max_restarts = o->max_restarts;
    A.res = d_res;
    A.occ = d_occ;

    // ---- autotune the workgroup size on a sample spread over the cost range
    double tune_seconds = 0.0;
    int tuned = 0;
    if (block == 0 && count <= kSample) {
        // The tuning sample would be the whole batch, solved once per
        // candidate: take the size the tuner picks on large batches.
        block = 512;
    } else if (block == 0) {
        std::vector<int64_t> key = {count, L.grid, o->krylov};
        for (int i = 0; i < count; ++i) key.push_back(sorted[i].dim);
        std::lock_guard<std::mutex> lk(g_tune_mu);
        auto it = g_tuned.find(key);
        if (it != g_tuned.end()) {
            block = it->second;
        } else {
            auto ts = std::chrono::steady_clock::now();
            const int S = std::min(count, kSample);
            // The sample runs on the largest teams there are (short trials); without
            // teams, on single workgroups.  The slots of the teams of 8 hold the
            // instances planned for them, the costliest ones: one further down the
            // cost order may have more states (4 of 32 orbits and 3 pairs, 4960
            // states, are costlier than 400 of 15 and 6, 5005) and then gives way to
            // the next costlier one that fits.
            const bool on_teams = plan.teams > 0 || plan.mid_teams > 0;
            const int64_t slot = plan.teams > 0 ? L.slot_doubles : on_teams ? L.mid_doubles : L.slot2_doubles;
            std::vector<Instance> sample(S);
            for (int q = 0; q < S; ++q) {
                // quantiles 5% .. 100% of the cost order (largest excluded)
                int pos = (int)((double)(q + 1) / (S + 1) * (count - 1));
                pos = std::min(count - 1, pos + count / 20);
                while (pos > 0 && slot_for(o->krylov, sorted[pos].dim) > slot) --pos;
                sample[q] = sorted[pos];
            }
            PD_HIP(hipMemcpyAsync(d_sample, sample.data(), sizeof(Instance) * S, hipMemcpyHostToDevice, stream));
            Args As = A;
            As.inst = d_sample;
            As.count = S;
            As.level[0].end = plan.teams > 0 ? S : 0;
            As.level[1].end = on_teams ? S : 0;
            if (plan.teams > 0) As.level[1].teams = 0;
            const int trial_grid = on_teams ? L.grid : std::min(S, L.grid);
            double best = 1e300;
            const int cands[3] = {128, 256, 512};
            struct Events {
                hipEvent_t a = nullptr, b = nullptr;
                ~Events() {
                    if (a) (void)hipEventDestroy(a);
                    if (b) (void)hipEventDestroy(b);
                }
            } ev;
            PD_HIP(hipEventCreate(&ev.a));
            PD_HIP(hipEventCreate(&ev.b));
            block = 0;
            for (int c : cands) {
                hipLaunchKernelGGL(reset_queue, dim3(1), dim3(64), 0, stream, d_counter, As.level[1].end, d_large,
                                   d_mid, 0, d_team_flag, 2 * L.grid, d_error);
                PD_HIP(hipEventRecord(ev.a, stream));
                hipLaunchKernelGGL(batched_kernel, dim3(trial_grid), dim3(c), batched_dyn_lds(c), stream, As);
                PD_HIP(hipGetLastError());
                PD_HIP(hipEventRecord(ev.b, stream));
                PD_HIP(hipEventSynchronize(ev.b));
                float ms = 0.0f;
                PD_HIP(hipEventElapsedTime(&ms, ev.a, ev.b));
                // A trial whose team barrier timed out drained early: its time
                // means nothing, so the candidate is not eligible.
                int trial_err = 0;
                PD_HIP(hipMemcpy(&trial_err, d_error, sizeof(int), hipMemcpyDeviceToHost));
                if (!trial_err && ms < best) {
                    best = ms;
                    block = c;
                }
            }
            if (block == 0)
                return fail(PD_EDEVICE, "every autotuner trial hit a team barrier time-out (is another kernel "
                                        "occupying the GPU?)");
            g_tuned[key] = block;
            tuned = 1;
            tune_seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - ts).count();
        }
    }
    if (block != 128 && block != 256 && block != 512) return fail(PD_EINVAL, "block must be 0, 128, 256 or 512");

    // ---- one graph: queue reset (a kernel, no memset node) + the persistent solver
    hipStream_t cap = nullptr;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    PD_HIP(hipStreamCreateWithFlags(&cap, hipStreamNonBlocking));
    hipError_t e = hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(reset_queue, dim3(1), dim3(64), 0, cap, d_counter, mid.end, d_large, d_mid, plan.n_large,
                           d_team_flag, 2 * L.grid, d_error);
        hipLaunchKernelGGL(batched_kernel, dim3(L.grid), dim3(block), batched_dyn_lds(block), cap, A);
        e = hipStreamEndCapture(cap, &graph);
    }
    if (e == hipSuccess) e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
    auto tk = std::chrono::steady_clock::now();
    if (e == hipSuccess) e = hipGraphLaunch(exec, stream);
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    const double kernel_seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - tk).count();
    if (exec) (void)hipGraphExecDestroy(exec);
    if (graph) (void)hipGraphDestroy(graph);
    (void)hipStreamDestroy(cap);
    if (e != hipSuccess) return fail(PD_EDEVICE, "batched solve: %s", hipGetErrorString(e));
    int err_flag = 0;
    PD_HIP(hipMemcpy(&err_flag, d_error, sizeof(int), hipMemcpyDeviceToHost));
    if (err_flag) return fail(PD_EDEVICE, "a workgroup team barrier timed out (is another kernel occupying the GPU?)");

    int wall_khz = 0, dev = 0;
    (void)hipGetDevice(&dev);
    if (hipDeviceGetAttribute(&wall_khz, hipDeviceAttributeWallClockRate, dev) != hipSuccess || wall_khz <= 0)
        wall_khz = 100000;
    const double wall_hz = 1e3 * wall_khz;
    std::vector<Result> res(count);
    PD_HIP(hipMemcpy(res.data(), d_res, sizeof(Result) * count, hipMemcpyDeviceToHost));
    if (occ_out) {
        PD_HIP(hipMemcpy(occ_out, d_occ, sizeof(double) * L.occ_doubles, hipMemcpyDeviceToHost));
        for (int i = 0; i < count; ++i)
            if (flipped[i])
                for (int q = 0; q < omega[i]; ++q) occ_out[inst[i].occ_off + q] = 2.0 - occ_out[inst[i].occ_off + q];
    }
    int nconv = 0;
    long long total_it = 0;
    for (int i = 0; i < count; ++i) {
        E0_out[i] = res[i].E0;
        nconv += res[i].converged;
        total_it += res[i].iterations;
        if (info_out) {
            pd_lanczos_info &f = info_out[i];
            std::memset(&f, 0, sizeof(f));
            f.iterations = res[i].iterations;
            f.restarts = res[i].restarts;
            f.converged = res[i].converged;
            f.residual = res[i].residual;
            f.seconds = (double)res[i].ticks / wall_hz;
        }
    }
    if (binfo) {
        binfo->block = block;
        binfo->grid = L.grid;
        binfo->tuned = tuned;
        binfo->tune_seconds = tune_seconds;
        binfo->kernel_seconds = kernel_seconds;
        binfo->seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
        binfo->converged = nconv;
        const Args::Level &first = plan.teams > 0 || plan.mid_teams == 0 ? large : mid;
        binfo->teams = first.teams;
        binfo->team_size = first.teams > 0 ? first.team_size : 1;
        binfo->large = plan.teams > 0 ? plan.n_large : plan.n_mid;
        binfo->total_iterations = total_it;
    }
    if (nconv < count) return fail(PD_ENOCONV, "%d of %d instances did not converge", count - nconv, count);
    return PD_OK;
}

}  // namespace pd
