// The batched solver (batched.hip) on the CPU: its kernel's code runs with one
// fiber per lane and one host thread per workgroup, its host code runs over host
// memory, and launches are looked at instead of made.
//
//   batched_host solve BLOCK TEAM SEED        one instance read from stdin
//   batched_host tune                         a batch's shape read from stdin
//
// A wave runs until all of its lanes wait at a workgroup barrier, then another
// one is chosen by SEED: 0 the first wave first, 1 the last wave first, else at
// random.  Between two barriers any order of the waves is allowed on the GPU, so results
// may not depend on it.  LDS starts with large numbers in it.
#include <hip/hip_runtime.h>
#include <ucontext.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <random>
#include <thread>
#include <vector>

asm(".macro s_waitcnt what\n.endm");   // every store is complete at once here

// ---------------------------------------------------------------- lanes, waves, barriers
struct Fiber {
    ucontext_t ctx;
    std::vector<char> stack;
    enum { Ready, Barrier, Wave, Done } at = Ready;
    long barriers = 0;
    int parity = 0;
};
struct Workgroup {
    ucontext_t main;
    std::vector<Fiber> lanes;
    std::vector<double> box[2];   // values that the lanes of a wave pass to each other
    std::function<void()> body;
    int now = 0;
};
static thread_local Workgroup *g_wg;
struct Dim {
    unsigned x, y, z;
};
static thread_local Dim threadIdx, blockIdx;
static Dim blockDim;

static void leave(decltype(Fiber::at) why) {
    Workgroup *W = g_wg;
    Fiber &F = W->lanes[W->now];
    F.at = why;
    swapcontext(&F.ctx, &W->main);
}
static void fiber_main() {
    g_wg->body();
    leave(Fiber::Done);
}
static void run_workgroup(int block, unsigned seed, std::function<void()> body) {
    Workgroup W;
    g_wg = &W;
    W.body = body;
    W.lanes.resize(block);
    for (auto &b : W.box) b.resize(block);
    for (auto &F : W.lanes) {
        F.stack.resize(256 << 10);
        getcontext(&F.ctx);
        F.ctx.uc_stack.ss_sp = F.stack.data();
        F.ctx.uc_stack.ss_size = F.stack.size();
        F.ctx.uc_link = nullptr;
        makecontext(&F.ctx, fiber_main, 0);
    }
    std::mt19937 rng(seed);
    std::vector<int> order(block / 64);
    for (size_t i = 0; i < order.size(); ++i) order[i] = seed == 1 ? (int)(order.size() - 1 - i) : (int)i;
    for (;;) {
        if (seed > 1) std::shuffle(order.begin(), order.end(), rng);
        for (int w : order)
            for (bool more = true; more;) {
                more = false;
                int meet = 0;
                for (int l = w * 64; l < w * 64 + 64; ++l) {
                    Fiber &F = W.lanes[l];
                    if (F.at == Fiber::Ready) {
                        more = true;
                        W.now = l;
                        threadIdx = {(unsigned)l, 0, 0};
                        swapcontext(&W.main, &F.ctx);
                    }
                    meet += F.at == Fiber::Wave;
                }
                if (meet == 64) {
                    more = true;
                    for (int l = w * 64; l < w * 64 + 64; ++l) W.lanes[l].at = Fiber::Ready;
                }
            }
        int barrier = 0, done = 0;
        for (auto &F : W.lanes) barrier += F.at == Fiber::Barrier, done += F.at == Fiber::Done;
        if (done == block) return;
        if (barrier != block) {
            std::printf("lanes do not meet: %d at a barrier, %d at an end, of %d\n", barrier, done, block);
            std::fflush(stdout);
            std::_Exit(3);
        }
        for (auto &F : W.lanes) F.at = Fiber::Ready;
    }
}

static void __syncthreads() { leave(Fiber::Barrier); }
static void __threadfence() { __atomic_thread_fence(__ATOMIC_SEQ_CST); }
template <typename T>
static T from_lane(T v, int lane) {
    Workgroup *W = g_wg;
    const int me = W->now, p = W->lanes[me].parity ^= 1;
    std::memcpy(&W->box[p][me], &v, sizeof(T));
    leave(Fiber::Wave);
    T r;
    std::memcpy(&r, &W->box[p][(me & ~63) + (lane & 63)], sizeof(T));
    return r;
}
template <typename T>
static T __shfl_xor(T v, int mask, int) { return from_lane(v, (int)threadIdx.x ^ mask); }
template <typename T>
static T __shfl_down(T v, int by, int) {
    const int lane = threadIdx.x & 63;
    return from_lane(v, lane + by < 64 ? lane + by : lane);
}
template <typename T>
static T __shfl(T v, int lane, int) { return from_lane(v, lane); }
// waiting for another workgroup: every other lane and workgroup goes on
static void pause_lane() {
    std::this_thread::yield();
    leave(Fiber::Ready);
}

static int atomicAdd(int *p, int v) { return __atomic_fetch_add(p, v, __ATOMIC_SEQ_CST); }
static int atomicExch(int *p, int v) { return __atomic_exchange_n(p, v, __ATOMIC_SEQ_CST); }
template <typename T>
static void atomic_store(T *p, T v) { __atomic_store(p, &v, __ATOMIC_SEQ_CST); }
template <typename T>
static T atomic_load(const T *p) {
    T v;
    __atomic_load(p, &v, __ATOMIC_SEQ_CST);
    return v;
}
static long long wall_clock64() { return 0; }
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_store(p, v, order, scope) atomic_store(p, v)
#define __hip_atomic_load(p, order, scope) atomic_load(p)
#define __builtin_amdgcn_s_sleep(n) pause_lane()
#define __builtin_amdgcn_fence(order, scope) __threadfence()
#define __builtin_amdgcn_readfirstlane(v) (v)
#define __builtin_amdgcn_s_getreg(r) (0)
#define __HIP_DEVICE_COMPILE__ 1
#undef __shared__
#define __shared__ thread_local
#undef __align__
#define __align__(n) __attribute__((aligned(n)))
#undef __launch_bounds__
#define __launch_bounds__(...)

template <typename F, typename... A>
static void launched(F kernel, A... args);
#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(kernel, grid, block, lds, stream, ...) launched(kernel, __VA_ARGS__)

#include "batched.hip"

namespace pd {
namespace batched {
thread_local unsigned char bdyn[64 << 10];

// Every instance that a launch may hand to a level has to fit that level's slots.
static int g_launches, g_bad;
static void look(const Args &A) {
    ++g_launches;
    for (int i = 0; i < A.count; ++i) {
        const Instance &I = A.inst[i];
        const int64_t need = (I.m + 2) * ((I.dim + 63) & ~int64_t(63));
        const bool l0 = A.level[0].teams > 0 && i < A.level[0].end, l1 = A.level[1].teams > 0 && i < A.level[1].end;
        const int64_t have = l0 ? A.level[0].slot_doubles : l1 ? A.level[1].slot_doubles : A.slot2_doubles;
        if (need > have) {
            ++g_bad;
            std::printf("launch %d, instance %d of %d: %lld doubles in a slot of %lld\n", g_launches, i, A.count,
                        (long long)need, (long long)have);
        }
        Result r = {};
        r.converged = 1;
        A.res[I.orig] = r;
    }
}

struct Problem {
    int omega, n, krylov;
    double tol;
    std::vector<double> d, V;
};

// One instance on a team of `team` workgroups.
static void solve(const Problem &P, int block, int team, unsigned seed) {
    Instance I = {};
    I.omega = P.omega;
    I.n = I.nn = P.n;
    I.dim = (int64_t)binom_host(P.omega, P.n);
    I.seed = 7;
    I.m = (int)std::min<int64_t>(P.krylov, I.dim);
    I.dscale = 1.0;
    std::vector<double> coef(kMaxOmegaB + P.V.size());
    std::copy(P.d.begin(), P.d.end(), coef.begin());
    std::copy(P.V.begin(), P.V.end(), coef.begin() + kMaxOmegaB);
    for (double d : P.d) I.dsum += d;
    std::vector<double> slot((I.m + 2) * ((I.dim + 63) & ~int64_t(63))), occ(P.omega), part(2 * team * kMaxSums);
    std::vector<int> flag(team);
    int error = 0;
    Result res = {};
    Args A = {};
    A.inst = &I;
    A.count = 1;
    A.error = &error;
    A.spin_limit = 1ll << 40;
    A.coef = coef.data();
    A.tol = P.tol;
    A.max_restarts = 200;
    A.res = &res;
    A.occ = occ.data();
    blockDim = {(unsigned)block, 1, 1};
    std::vector<std::thread> threads;
    for (int g = 0; g < team; ++g)
        threads.emplace_back([&, g] {
            blockIdx = {(unsigned)g, 0, 0};
            static thread_local Shared sh;
            std::vector<double> fill(sizeof(sh) / sizeof(double), 1e300);
            std::memcpy(&sh, fill.data(), fill.size() * sizeof(double));
            run_workgroup(block, seed, [&, g] {
                Team T = {};
                T.G = team;
                T.g = g;
                T.flag = flag.data();
                T.part = part.data();
                T.pre = reinterpret_cast<uint32_t *>(bdyn);
                solve_instance(A, I, slot.data(), T, sh);
            });
        });
    for (auto &t : threads) t.join();
    std::printf("%.17g %.17g %d %d %d", res.E0, res.residual, res.iterations, res.restarts, res.converged);
    for (double o : occ) std::printf(" %.17g", o);
    std::printf("\n");
}
}  // namespace batched

// Stands in for the library's functions that batched.hip calls.
pd_status fail(pd_status s, const char *fmt, ...) {
    std::printf("status %d: %s\n", (int)s, fmt);
    return s;
}
const char *last_error() { return ""; }
pd_status pack_coefficients(int, int, const double *, const double *, CoefBlock *out) {
    std::memset((void *)out, 0, sizeof(*out));
    return PD_OK;
}
}  // namespace pd

template <typename F, typename... A>
static void launched(F, A... args) {
    if constexpr (sizeof...(A) == 1) pd::batched::look(args...);
}

// The HIP calls of the host code, over host memory.
#define STUB(name, args) \
    hipError_t name args { return hipSuccess; }
hipError_t hipMemcpyAsync(void *to, const void *from, size_t n, hipMemcpyKind, hipStream_t) {
    std::memcpy(to, from, n);
    return hipSuccess;
}
hipError_t hipMemcpy(void *to, const void *from, size_t n, hipMemcpyKind) {
    std::memcpy(to, from, n);
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) {
    *v = 256;
    return hipSuccess;
}
hipError_t hipGetDevice(int *d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
    *ms = 1.0f;
    return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return ""; }
STUB(hipFuncSetAttribute, (const void *, hipFuncAttribute, int))
STUB(hipStreamSynchronize, (hipStream_t))
STUB(hipEventCreate, (hipEvent_t *))
STUB(hipEventDestroy, (hipEvent_t))
STUB(hipEventRecord, (hipEvent_t, hipStream_t))
STUB(hipEventSynchronize, (hipEvent_t))
STUB(hipGetLastError, (void))
STUB(hipStreamCreateWithFlags, (hipStream_t *, unsigned))
STUB(hipStreamBeginCapture, (hipStream_t, hipStreamCaptureMode))
STUB(hipStreamEndCapture, (hipStream_t, hipGraph_t *))
STUB(hipGraphInstantiate, (hipGraphExec_t *, hipGraph_t, hipGraphNode_t *, char *, size_t))
STUB(hipGraphLaunch, (hipGraphExec_t, hipStream_t))
STUB(hipGraphExecDestroy, (hipGraphExec_t))
STUB(hipGraphDestroy, (hipGraph_t))
STUB(hipStreamDestroy, (hipStream_t))

int main(int argc, char **argv) {
    if (argc == 5 && !std::strcmp(argv[1], "solve")) {
        pd::batched::Problem P;
        if (std::scanf("%d %d %d %lf", &P.omega, &P.n, &P.krylov, &P.tol) != 4) return 2;
        P.d.resize(P.omega);
        P.V.resize(P.omega * P.omega);
        for (double &v : P.d) if (std::scanf("%lf", &v) != 1) return 2;
        for (double &v : P.V) if (std::scanf("%lf", &v) != 1) return 2;
        pd::batched::solve(P, std::atoi(argv[2]), std::atoi(argv[3]), (unsigned)std::atoi(argv[4]));
        return 0;
    }
    if (argc == 2 && !std::strcmp(argv[1], "tune")) {
        int kinds, krylov;
        std::vector<int> omega, n;
        if (std::scanf("%d %d", &krylov, &kinds) != 2) return 2;
        size_t ne = 0, nv = 0;
        for (int k = 0, o, p, c; k < kinds; ++k) {
            if (std::scanf("%d %d %d", &o, &p, &c) != 3) return 2;
            for (int i = 0; i < c; ++i) {
                omega.push_back(o), n.push_back(p);
                ne += o, nv += (size_t)o * o;
            }
        }
        const int count = (int)omega.size();
        pd_lanczos_opts o = {};
        o.krylov = krylov;
        o.tol = 1e-10;
        o.max_restarts = 10;
        std::vector<unsigned char> work(pd::batched_workspace_bytes(count, omega.data(), n.data(), &o));
        std::vector<double> eps(ne), V(nv), E0(count), occ(ne);
        pd_batch_info info = {};
        const pd_status st = pd::batched_run(count, omega.data(), n.data(), eps.data(), V.data(), &o, 0, work.data(),
                                             work.size(), E0.data(), occ.data(), nullptr, &info, nullptr);
        std::printf("status %d launches %d teams %d of %d tuned %d bad %d\n", (int)st, pd::batched::g_launches,
                    info.teams, info.team_size, info.tuned, pd::batched::g_bad);
        return 0;
    }
    return 2;
}
