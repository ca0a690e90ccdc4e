// newsvendor.hpp -- Algorithm 2 (Section 3.2, Task 2): the multi-product newsvendor by stochastic
// Frank-Wolfe. Device arguments shared by the kernels (fw_newsvendor.hip) and the host driver
// (nv_api.hip).
#pragma once

#include <stddef.h>
#include <stdint.h>

#include "run_shape.hpp"

namespace fw {

constexpr int kNvBlock = 256;                   // threads per workgroup: kNvBlock / P quads of products
constexpr uint32_t kNvMaxLanes = 16;            // lanes per quad at most

// Lanes per quad for n/4 quads and R replications: the smallest power of two that gives ~65536
// threads (a wavefront per SIMD on every compute unit), at most kNvMaxLanes and at most S.
inline uint32_t nv_lanes_per_quad(uint32_t nq, uint64_t R, uint32_t S)
{
    uint32_t P = 1;
    while (P < kNvMaxLanes && 2 * P <= S && static_cast<uint64_t>(nq) * R * P < 65536u) P *= 2;
    return P;
}
constexpr uint32_t kNvMaxR = 64;
constexpr uint32_t kNvMaxS = 1024;
constexpr uint64_t kNvMaxN = 1ull << 24;
constexpr uint32_t kNvDomain = 4u;              // Philox stream domain of the demand samples
constexpr uint32_t kNvCostChunk = 4096;         // products per workgroup of the cost evaluation

struct NvArgs {
    uint32_t n, nq, S, nwg, R;                  // products, quads, samples per product, workgroups
    uint32_t P;                                 // lanes per quad (a power of two <= kNvMaxLanes), splitting its samples
    uint32_t k0, k1, dom;                       // Philox key; counter word 3 (domain 4 | instance)
    float C, gap_eps;
    // per product, binary32: threshold scale 1/(sqrt(2 ln 2) sigma), k - v, (h + v)/S, 1/c, C/c, x_0
    const float *mu_f, *isk_f, *a_f, *b_f, *ic_f, *xs_f, *x0_f;
    // per product, binary64, for the cost Eq. (6)
    const double *mu_d, *sig_d, *k_d, *h_d, *v_d, *xs_d;
    // state of each replication
    uint64_t *S_sig;                            // [R][n] sum of (t+1) over steps choosing vertex j
    uint32_t *cnt;                              // [R][n+1] decision counts, origin first
    uint32_t *tau;                              // [R]
    uint32_t *dec;                              // [R][T]
    uint64_t T;
    // per-iteration scratch
    // two buffers by iteration parity: a sample launch may read the previous iteration's partials
    float *wg_r;                                // [2][R][nwg] smallest g_j / c_j of the workgroup
    uint32_t *wg_j;                             // [2][R][nwg] its product
    float *wg_gx;                               // [2][R][nwg] the workgroup's part of g'x
    // outcomes
    double *cost_part;                          // [R][ceil(n / kNvCostChunk)][2] double-double partials
    double *fval;                               // [n_ckpt + 1][R]
    double *stats;                              // kMaxStreams x kStreamFields + 2
    uint64_t *origin_total;                     // kNvFailed after a cooperative run that gave up
    const uint32_t *fail;                       // its failure word (NULL: launch by launch)
};

constexpr uint64_t kNvFailed = ~0ull;

// Iteration t's samples and workgroup partials; with fold_prev it first takes the step of iteration
// t - 1 (whose partials the previous launch left in the other buffer).
int launch_nv_sample(const NvArgs &A, uint64_t t, uint32_t epoch, float cw, bool from_x0, bool fold_prev, hipStream_t s);
// The step of iteration t on its own.
int launch_nv_step(const NvArgs &A, uint64_t t, hipStream_t s);
int launch_nv_cost(const NvArgs &A, double c, uint32_t slot, hipStream_t s);
int launch_nv_finalize(const NvArgs &A, uint32_t n_ckpt, hipStream_t s);

// ---- many iterations in one cooperative launch (fw_newsvendor_run.hip) --------------------------
// A run takes this form when its workgroups fit twice per compute unit and a lane's samples of an
// epoch fit in registers (16 of them leave two wavefronts per SIMD, 32 one), which holds up to
// n = 130,000 at S = 50 on one replication. Past that an iteration's samples outweigh its launch (n = 1e6:
// 32 us against 2.7 us), and the launch-per-iteration kernels keep the chip full without an exchange.
// Measured (S = 25, K = 1500): n = 1e4 7.7 -> 3.7 ms a call, n = 872 2.3 times, n = 48,000 (S = 30) 1.8 times.
constexpr uint32_t kNvRunMaxNs = 16;            // samples per lane
struct NvRunArgs {
    uint64_t t0, t1;                            // the iterations of this launch
    uint32_t M;                                 // iterations per resample
    uint32_t from_x0;                           // iteration 0 starts from x0_f
    uint64_t *words;                            // [R][nwg][kRunLine] exchange slots, cleared before the run
    uint32_t *fail;                             // raised by a wait that gave up; cleared before the run
    float *gx_log;                              // [t1 - t0][R][nwg] parts of g'x
    float *best_log;                            // [t1 - t0][R] smallest ratios
};

// Bytes of the slots and the failure word (cleared before a run), and of all the form's scratch.
inline size_t nv_run_slot_bytes(uint64_t R, uint32_t nwg) { return sizeof(uint64_t) * (kRunLine * R * nwg + 1); }
inline size_t nv_run_bytes(uint64_t R, uint32_t nwg, uint64_t T)
{
    return nv_run_slot_bytes(R, nwg) + sizeof(float) * (T < kRunSteps ? T : kRunSteps) * R * (nwg + 1);
}

bool nv_run_fits(uint32_t nwg, uint32_t R, uint32_t S, uint32_t P, int device);
int launch_nv_run(const NvArgs &A, const NvRunArgs &Q, hipStream_t s);         // kRunRefused: the runtime would not

// ---- Algorithm 2 over X = {A x <= C, x >= 0} with M resource rows (Eq. (7)) --------------------
// threads of the subproblem workgroup (one per replication): few products leave a pricing pass
// short, and then four wavefronts' barriers cost less than sixteen's
constexpr int kNvLpBlockSmall = 256;
constexpr int kNvLpBlockLarge = 1024;
constexpr uint32_t kNvLpSmallN = 2048;          // products up to which the small workgroup runs
constexpr uint32_t kNvLpMaxM = 8;

struct NvLpArgs {
    uint32_t n, nq, S, nwg, R, M;
    uint32_t P;                                 // lanes per quad in the gradient launch (nv_lanes_per_quad)
    uint32_t k0, k1, dom;                       // Philox key; counter word 3 (domain 4 | instance)
    uint32_t max_pivots;
    double gap_eps;
    double eps_r, eps_d;                        // reduced-cost and pivot-element tolerances
    // per product, binary64
    const double *mu_d, *isk_d;                 // mean; 1/(sqrt(2 ln 2) sigma) (infinite for sigma = 0)
    const double *km_d, *hv_d;                  // k - v; h + v
    const double *sig_d, *k_d, *h_d, *v_d;      // for the cost Eq. (6)
    const double *x0_d;                         // starting point (zeros for the origin)
    const double *Am;                           // [M][n] resource use
    const double *Cv;                           // [M] resource levels
    // state of each replication
    double *x;                                  // [R][n] the iterate
    double *g;                                  // [R][n] the iteration's gradient Eq. (9)
    uint32_t *rec_basis;                        // [R][T][M] each iteration's basis
    double *rec_value;                          // [R][T][M] and its basic variables
    uint32_t *rec_piv;                          // [R][T] pivots taken (max_pivots + 1: not solved)
    uint32_t *tau;                              // [R]
    uint32_t *origin;                           // [R] iterations whose vertex is the origin
    uint64_t T;
    // outcomes
    double *cost_part;                          // [R][ceil(n / kNvCostChunk)][2]
    double *fval;                               // [n_ckpt + 1][R]
    double *stats;                              // kMaxStreams x kStreamFields + 2
    uint64_t *origin_total;                     // kNvFailed after a cooperative run that gave up
    const uint32_t *fail;                       // its failure word (NULL: launch by launch)
};

// ---- many iterations in one cooperative launch (fw_newsvendor_lp_run.hip) ------------------------
// A run takes this form when g fits in LDS, the samples of an epoch in a lane's registers, and the
// sample workgroups and the simplex workgroup have a compute unit each. Faster at every such size.
// 1,500 iterations, S = 25, launch by launch -> one launch, ms: n = 100, 3 rows 28.2 -> 10.8; n = 1,000
// with 1 row 21.6 -> 8.0, 3 rows 45.6 -> 14.7, 6 rows 97.9 -> 26.3, 3 rows and 7 replications 59.5 ->
// 14.9; n = 4,000, 3 rows 67.9 -> 32.0; n = 10,000, 3 rows 104.3 -> 61.9.
constexpr uint32_t kLpRunMaxNs = 8;             // samples per lane
constexpr uint32_t kLpRunSteps = 256;           // iterations per launch at most (the length of the LDS logs)
constexpr uint32_t kLpVertexWords = 24;         // three words for each of up to 8 basic columns
constexpr size_t kLpRunLds = 120 * 1024;        // g, and A where it fits: n (M + 1) <= 15,360

struct NvLpRunArgs {
    uint64_t t0, t1;                            // the iterations of this launch
    uint32_t Mr;                                // iterations per resample
    uint64_t *words;                            // [R][2][nq] counts, then [R][2][kLpVertexWords]; cleared before the run
    uint32_t *fail;                             // raised by a wait that gave up; cleared before the run
    double *gx_log;                             // [t1 - t0][R][nwg] parts of g'x
    double *gs_log;                             // [t1 - t0][R] g's
};

// Bytes of the slots and the failure word (cleared before a run), and of all the form's scratch.
inline size_t nv_lp_run_slot_bytes(uint64_t R, uint32_t nq) { return sizeof(uint64_t) * (R * 2 * (nq + kLpVertexWords) + 1); }
inline size_t nv_lp_run_bytes(uint64_t R, uint32_t nq, uint32_t nwg, uint64_t T)
{
    return nv_lp_run_slot_bytes(R, nq) + sizeof(double) * (T < kLpRunSteps ? T : kLpRunSteps) * R * (nwg + 1);
}

// The launches of a run of T iterations (resample every M): for each t, gradient(t, epoch, fold_prev)
// and subproblem(t); update(t) where the update cannot wait for the next gradient launch (a cost
// evaluation follows, or t is the last iteration); cost(slot) for every checkpoint equal to t + 1.
// Each callback returns 0 or an error, which ends the sequence and is returned.
template <class Gradient, class Subproblem, class Update, class Cost>
int nv_lp_sequence(uint64_t M, uint64_t T, uint32_t n_ckpt, const uint64_t *checkpoints, Gradient gradient,
                   Subproblem subproblem, Update update, Cost cost)
{
    uint32_t ck = 0;
    bool pending = false;
    for (uint64_t t = 0; t < T; ++t) {
        if (int rc = gradient(t, static_cast<uint32_t>(t / M), pending)) return rc;
        if (int rc = subproblem(t)) return rc;
        const bool cost_next = ck < n_ckpt && checkpoints[ck] == t + 1;
        pending = !(cost_next || t + 1 == T);
        if (!pending)
            if (int rc = update(t)) return rc;
        while (ck < n_ckpt && checkpoints[ck] == t + 1) {
            if (int rc = cost(ck)) return rc;
            ++ck;
        }
    }
    return 0;
}

bool nv_lp_run_fits(const NvLpArgs &A, int device);
int launch_nv_lp_run(const NvLpArgs &A, const NvLpRunArgs &Q, hipStream_t s);  // kRunRefused: the runtime would not
// Iteration t's gradient at x_t; with fold_prev it first moves x to x_t = x_{t-1} + gamma (s - x_{t-1})
// with the vertex the previous subproblem launch recorded.
int launch_nv_lp_gradient(const NvLpArgs &A, uint64_t t, uint32_t epoch, bool fold_prev, hipStream_t s);
// Iteration t's linear subproblem, its records and the Frank-Wolfe gap.
int launch_nv_lp_subproblem(const NvLpArgs &A, uint64_t t, hipStream_t s);
// The update of iteration t on its own (before a cost evaluation and after the last iteration).
int launch_nv_lp_update(const NvLpArgs &A, uint64_t t, hipStream_t s);
int launch_nv_lp_cost(const NvLpArgs &A, uint32_t slot, hipStream_t s);
int launch_nv_lp_finalize(const NvLpArgs &A, uint32_t n_ckpt, hipStream_t s);

}  // namespace fw
