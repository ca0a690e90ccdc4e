// emu_host.cpp -- the other half of the CPU runtime (emu_runtime.hpp), and what the emulated library
// leaves out: the path kernels of sim_run and the quasi-Newton replications, which these tests do not
// launch, and the loss of a quasi-Newton run's snapshots, in plain loops here.
#include "emu_runtime.hpp"

#include <sys/mman.h>
#include <sys/wait.h>
#include <unistd.h>

#include <cstdio>
#include <cstdlib>
#include <map>
#include <string>

#include "../../paper_2404_11631_amd/csrc/engine.hpp"
#include "../../paper_2404_11631_amd/csrc/sqn_split.hpp"
#include "../../paper_2404_11631_amd/csrc/wide.hpp"

thread_local Dim3emu threadIdx;
thread_local Dim3emu blockIdx;
EmuBlock *g_block = nullptr;

namespace fw {
bool paths_split_applies(const InstanceDesc &, bool, bool, int) { return true; }
int launch_fw_paths(const InstanceDesc &, const InstanceDesc *, const RunBuffers &, bool, hipStream_t, int *) { return 0; }
int launch_fw_dense(const InstanceDesc &, const InstanceDesc *, const RunBuffers &, hipStream_t) { return -3; }
int launch_sqn_run(const SqnArgs &, hipStream_t) { return -1; }
int launch_sqn_hessian(const SqnArgs &, uint32_t, uint32_t, uint32_t, double *, double *, uint32_t, hipStream_t) { return -1; }
int launch_sqn_loss(const SqnArgs &A, hipStream_t)
{
    if (!emu_launch()) return emu_last_error() == hipSuccess ? 0 : -1;
    const uint32_t ns = 1 + 2 * A.n_ckpt;
    for (uint32_t s = 0; s < (A.n_ckpt + 1) * A.R; ++s) {
        double f = 0.0;
        for (uint32_t i = 0; i < A.N; ++i) {
            double u = 0.0;
            for (uint32_t j = 0; j < A.n; ++j)
                if (A.X[static_cast<size_t>(i) * A.xw + j / 32] >> (j % 32) & 1u) u += A.wsnap[static_cast<size_t>(s) * A.ld + j];
            f += std::log1p(std::exp(-std::fabs(u))) + std::max(u, 0.0) - (A.z[i] ? u : 0.0);
        }
        A.fval[s] = f / A.N;
    }
    std::fill(A.stats, A.stats + kMaxStreams * kStreamFields + 2, 0.0);
    const double *Y = A.fval + static_cast<size_t>(A.n_ckpt) * A.R;
    for (uint32_t r = 0; r < A.R; ++r) A.stats[0] += Y[r], A.stats[2] += Y[r] * Y[r];
    for (uint32_t s = 0; s < ns; ++s) A.stats[s * kStreamFields + 4] = A.R;
    if (A.fail && *A.fail) A.stats[4] = -1.0;           // as the statistics kernel marks it
    A.stats[ns * kStreamFields] = *std::min_element(Y, Y + A.R);
    A.stats[ns * kStreamFields + 1] = *std::max_element(Y, Y + A.R);
    return 0;
}
}  // namespace fw

extern "C" {
// What goes wrong, by the number of the launch among those of its kind since the last emu_reset (0: the
// first; -1: none), and the launches there were.
struct EmuFaults {
    int refuse = -1;         // this cooperative launch is refused
    int missing = -1;        // in this cooperative launch the last workgroup is missing
    int failed = -1;         // before this cooperative launch the run's failure word is up
    int fail_launch = -1;    // from this ordinary launch on they fail
    int none = 0;            // 1: the device has no cooperative launches
    int cooperative = 0, launches = 0;
} emu;
char emu_events[1 << 16];    // calls in order, one per line
void emu_reset() { emu = EmuFaults{}, emu_events[0] = 0; }
EmuFaults *emu_faults() { return &emu; }
const char *emu_log() { return emu_events; }
}

namespace {

hipError_t g_last = hipSuccess;
std::map<void *, size_t> g_size;     // mapped bytes of a buffer's pages, by its first page
std::map<void *, void *> g_page;

void note(const std::string &s)
{
    const size_t n = std::strlen(emu_events);
    if (n + s.size() + 2 < sizeof(emu_events)) std::snprintf(emu_events + n, sizeof(emu_events) - n, "%s\n", s.c_str());
}

// the failure word of a run's arguments, by the type of its kernel's second argument
template <class Run> uint32_t *fail_word(void **args) { return static_cast<Run *>(args[1])->fail; }

}  // namespace

template <class Args, class Run> static void call_kernel(const void *fn, void **args)
{
    reinterpret_cast<void (*)(Args, Run)>(const_cast<void *>(fn))(*static_cast<Args *>(args[0]), *static_cast<Run *>(args[1]));
}

static int g_kind = 0;               // which run the next cooperative launches belong to: 1 wide, 2 newsvendor, 3 constraints, 4 SQN
extern "C" void emu_kind(int kind) { g_kind = kind; }

hipError_t hipMalloc(void **p, size_t n)
{
    note("malloc");
    const size_t page = 4096, m = (n + page - 1) / page * page;
    char *base = static_cast<char *>(mmap(nullptr, m + page, PROT_READ | PROT_WRITE, MAP_SHARED | MAP_ANONYMOUS, -1, 0));
    if (base == MAP_FAILED) return hipErrorOutOfMemory;
    mprotect(base + m, page, PROT_NONE);
    std::memset(base, 0xEE, m);
    *p = base + (m - n) / 16 * 16;
    g_size[*p] = m + page;
    g_page[*p] = base;
    return hipSuccess;
}

hipError_t hipFree(void *p)
{
    if (!p) return hipSuccess;
    note("free");
    munmap(g_page.at(p), g_size.at(p));
    g_page.erase(p);
    g_size.erase(p);
    return hipSuccess;
}

hipError_t hipMemcpy(void *d, const void *s, size_t n, int) { return std::memcpy(d, s, n), hipSuccess; }
hipError_t hipMemset(void *d, int v, size_t n) { return std::memset(d, v, n), hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return note("event"), hipSuccess; }
hipError_t emu_last_error()
{
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
hipError_t hipFuncSetAttribute(const void *fn, int, int value)
{
    char s[64];
    std::snprintf(s, sizeof(s), "attribute %p %d", fn, value);
    return note(s), hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, int what, int) { return *v = what == hipDeviceAttributeMultiprocessorCount ? 256 : !emu.none, hipSuccess; }

bool emu_launch()
{
    if (emu.fail_launch >= 0 && emu.launches >= emu.fail_launch) g_last = hipErrorLaunchFailure;
    return emu.launches++, g_last == hipSuccess;
}

hipError_t emu_cooperative(const void *fn, dim3 g, dim3 b, void **args, unsigned)
{
    const int k = emu.cooperative++;
    note("cooperative");
    if (k == emu.refuse) return g_last = hipErrorCooperativeLaunchTooLarge;
    if (k == emu.failed) {
        uint32_t *f = g_kind == 1   ? fail_word<fw::WideRunArgs>(args)
                      : g_kind == 2 ? fail_word<fw::NvRunArgs>(args)
                      : g_kind == 3 ? fail_word<fw::NvLpRunArgs>(args)
                                    : fail_word<fw::SqnSplitRun>(args);
        *f = 1;
    }
    auto body = [&] {
        if (g_kind == 1) call_kernel<fw::WideArgs, fw::WideRunArgs>(fn, args);
        else if (g_kind == 2) call_kernel<fw::NvArgs, fw::NvRunArgs>(fn, args);
        else if (g_kind == 3) call_kernel<fw::NvLpArgs, fw::NvLpRunArgs>(fn, args);
        else call_kernel<fw::SqnSplit, fw::SqnSplitRun>(fn, args);
    };
    std::vector<pid_t> children;
    for (unsigned y = 0; y < g.y; ++y)
        for (unsigned x = 0; x < g.x; ++x) {
            if (k == emu.missing && y + 1 == g.y && x + 1 == g.x) continue;
            const pid_t c = fork();
            if (c == 0) {
                emu_run_block(static_cast<int>(b.x), x, body, y);
                _exit(0);
            }
            children.push_back(c);
        }
    for (pid_t c : children) {
        int st = 0;
        waitpid(c, &st, 0);
        if (st) {
            std::fprintf(stderr, "a workgroup of cooperative launch %d ended with %x\n", k, st);
            std::abort();
        }
    }
    return hipSuccess;
}
