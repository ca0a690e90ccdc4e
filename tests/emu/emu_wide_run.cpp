// CPU emulation of the wide path's cooperative run (fw_wide_run.hip) against its launch-by-launch
// kernels (test infrastructure only). A process per workgroup, so that each has its own LDS, over
// shared memory with an inaccessible page behind every buffer; the threads of a workgroup in lockstep.
//
//   emu_wide_run NS ROWS d N R T M steps missing
//
// runs T iterations in launches of `steps`, without workgroup `missing` when it is not negative, and
// prints "same", "different" or, after a wait gave up, "gave up" with whether the counts are untouched.
#include <hip/hip_runtime.h>
thread_local Dim3emu threadIdx;
thread_local Dim3emu blockIdx;
EmuBlock *g_block = nullptr;

#include <sched.h>
#include <stdio.h>
#include <stdlib.h>
#include <sys/mman.h>
#include <sys/wait.h>
#include <unistd.h>

template <class T> inline T emu_load(T *p)
{
    sched_yield();                       // a poll gives way to the workgroups it waits for
    return std::atomic_ref<T>(*p).load();
}
#define __hip_atomic_load(p, o, s) emu_load(p)
template <class T> inline T atomicMin(T *p, T v)
{
    std::atomic_ref<T> a(*p);
    T o = a.load();
    while (v < o && !a.compare_exchange_weak(o, v)) {}
    return o;
}
#define hipDeviceGetAttribute(a, b, c) (*(a) = 1, hipSuccess)
#define hipDeviceAttributeMultiprocessorCount 0
#define hipDeviceAttributeCooperativeLaunch 0
#define hipLaunchCooperativeKernel(...) hipSuccess

#include "../../paper_2404_11631_amd/csrc/fw_wide.hip"
#include "../../paper_2404_11631_amd/csrc/fw_wide_run.hip"

using namespace fw;

static char *guarded(size_t n)
{
    const size_t page = 4096, m = (n + page - 1) / page * page;
    char *p = static_cast<char *>(mmap(nullptr, m + page, PROT_READ | PROT_WRITE, MAP_SHARED | MAP_ANONYMOUS, -1, 0));
    mprotect(p + m, page, PROT_NONE);
    return p + (m - n) / 16 * 16;
}

template <class T> T *filled(size_t n, T v = T())
{
    T *p = reinterpret_cast<T *>(guarded(n * sizeof(T)));
    std::fill(p, p + n, v);
    return p;
}

int main(int argc, char **argv)
{
    if (argc != 10) return 2;
    const int ns = atoi(argv[1]), rows = atoi(argv[2]);
    const uint32_t d = atoi(argv[3]), N = atoi(argv[4]), R = atoi(argv[5]), M = atoi(argv[7]);
    const uint64_t T = atoi(argv[6]), steps = atoi(argv[8]);
    const int missing = atoi(argv[9]);
    const uint32_t nq = d / 4, nwg = (nq + 31) / 32;
    WideArgs A{};
    A.d = d, A.nq = nq, A.N = N, A.nwg = nwg, A.R = R, A.k0 = 7, A.k1 = 9, A.gap_eps = 0.5f, A.lambda = 0.5, A.T = T;
    float *af = filled<float>(5 * d);
    srand(5);
    for (uint32_t j = 0; j < d; ++j) {
        const float sz = 1.17741f * (rand() / (float)RAND_MAX * 0.5f);
        af[j] = rand() / (float)RAND_MAX * 2 - 1;
        af[d + j] = sz;
        af[2 * d + j] = sz / N;
        af[3 * d + j] = sz / (N - 1);
        af[4 * d + j] = 0.5f / d;
    }
    A.mu_f = af, A.sz_f = af + d, A.c1_f = af + 2 * d, A.c2_f = af + 3 * d, A.w0_f = af + 4 * d;
    auto state = [&](WideArgs &B) {
        B.S = filled<uint64_t>(R * d);
        B.cnt = filled<uint32_t>(R * (d + 1));
        B.tau = filled<uint32_t>(R, kTauNone);
        B.dec = filled<uint32_t>(R * T, 0xEEEEEEEEu);
    };
    WideArgs B = A;
    state(A);
    state(B);
    if (missing < 0) {                   // the launch-by-launch run
        B.s1 = filled<float>(R * d);
        B.part_dot = filled<float>(R * N * nwg);
        B.part_qn = filled<float>(R * nwg);
        B.dot = filled<float>(R * N);
        B.qn = filled<float>(R);
        B.wg_g = filled<float>(2 * R * nwg);
        B.wg_gw = filled<float>(2 * R * nwg);
        B.wg_j = filled<uint32_t>(2 * R * nwg);
        auto grid = [&](uint32_t nx, const std::function<void()> &f) {
            for (uint32_t r = 0; r < R; ++r)
                for (uint32_t b = nx; b-- > 0;) emu_run_block(kWideBlock, b, f, r);
        };
        wide_sequence(
            N, nullptr, M, T, true, 0, nullptr,
            [&](uint64_t t, uint32_t e, const WideEpoch &E, float cw, bool w0, bool fold) {
                const int64_t prev = fold ? static_cast<int64_t>(t) - 1 : -1;
                grid(nwg, [&] { wide_sample_kernel(B, e, E.n, cw, w0, prev, E.par); });
                grid(E.n + 1, [&] { wide_dot_kernel(B, E.n); });
                grid(nwg, [&] { wide_gradient_kernel(B, e, E, cw, w0); });
                return 0;
            },
            [&](uint64_t t) {
                for (uint32_t r = 0; r < R; ++r)
                    emu_run_block(kWideBlock, r, [&] { wide_step_kernel(B, t, static_cast<uint32_t>(t & 1)); });
                return 0;
            },
            [&](double, uint32_t) { return 0; });
    }
    const size_t slots = wide_run_slot_bytes(R, nwg, N), total = wide_run_bytes(R, nwg, N, std::min(T, steps));
    char *w = guarded(total);
    std::memset(w, 0, slots);
    std::memset(w + slots, 0xAB, total - slots);
    WideRunArgs Q{};
    Q.M = M, Q.from_w0 = 1, Q.inv_n = static_cast<float>(1.0 / N), Q.words = reinterpret_cast<uint64_t *>(w);
    Q.fail = reinterpret_cast<uint32_t *>(w + slots - 8);
    Q.gw_log = reinterpret_cast<float *>(w + slots);
    Q.best_log = Q.gw_log + std::min(T, steps) * R * nwg;
    auto body = [&] {
        if (ns == 2 && rows == 0) wide_run_kernel<2, 0>(A, Q);
        if (ns == 4 && rows == 0) wide_run_kernel<4, 0>(A, Q);
        if (ns == 2 && rows == 3) wide_run_kernel<2, 3>(A, Q);
    };
    while (Q.t1 < T) {
        Q.t0 = Q.t1;
        Q.t1 = std::min(T, Q.t0 + steps);
        std::vector<pid_t> children;
        for (uint32_t r = 0; r < R; ++r)
            for (uint32_t g = 0; g < nwg; ++g) {
                if (static_cast<int>(g) == missing) continue;
                const pid_t c = fork();
                if (c == 0) {
                    emu_run_block(kWideBlock, g, body, r);
                    _exit(0);
                }
                children.push_back(c);
            }
        for (pid_t c : children) {
            int st = 0;
            waitpid(c, &st, 0);
            if (st) {
                printf("a workgroup ended with %x\n", st);
                return 1;
            }
        }
        const RunLog L{Q.gw_log, Q.best_log, nwg, R, d, 1.0f, A.gap_eps, Q.t0, T, Q.fail, A.dec, A.tau, A.cnt};
        for (uint32_t r = 0; r < R; ++r)
            for (uint32_t i = 0; i < Q.t1 - Q.t0; ++i) emu_run_block(256, i, [&] { run_log_kernel(L); }, r);
    }
    if (*Q.fail) {
        printf("gave up, counts %s\n", std::count(A.cnt, A.cnt + R * (d + 1), 0u) == R * (d + 1) ? "untouched" : "touched");
        return 0;
    }
    const bool same = !std::memcmp(A.S, B.S, 8 * R * d) && !std::memcmp(A.cnt, B.cnt, 4 * R * (d + 1)) &&
                      !std::memcmp(A.tau, B.tau, 4 * R) && !std::memcmp(A.dec, B.dec, 4 * R * T);
    printf("%s\n", same ? "same" : "different");
    return 0;
}
