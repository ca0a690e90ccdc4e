// fw_sqn_split_run.hip -- Algorithms 3-4 (Section 3.3, Task 3), one replication over many workgroups,
// many iterations in one launch.
//
// The kernels of fw_sqn_split.hip take two dependent launches per iteration (8.2 us and 9.8 us at
// n = 5,000, M = 25) and three per window (44 us, most of it one workgroup's small matrices). Here a
// cooperative launch runs iterations [k0, k1), a workgroup per slice, and the per-slice partial sums
// travel as tagged words (exchange.hpp; a binary64 value as two). The slice of w, of the window sum and
// of the previous average stays in registers, as do the stored pairs between two windows; every
// workgroup keeps the small matrices in LDS and rebuilds them for itself. The rows of iteration k + 1
// are fetched while iteration k waits for its sums.
//
// An iteration past 2L is two exchanges, the rows' dot products and S'g, Y'g; each workgroup reads the
// sums of all slices. From 65 rows on (and for the Hessian rows) that would be more than a wavefront's
// loads, so each workgroup sums a contiguous share of the rows, and the rows' coefficients take a
// second exchange.
//
// What bounds it (cycles of an iteration at n = 5,000, of 30,000): no unit, a chain of short steps with one
// wavefront per SIMD, 3,200 instructions each: the two exchanges with their sums over slices 9,300, the
// rows' coefficients summed into g 3,900, S'g and Y'g within the slice 2,000, the small products 2,200, the
// direction 2,500, the next rows' dot products 2,300, and per window 75,000 (small matrices 30,000).
// Bytes: the slice's pairs are read once per window, not twice per iteration.
//
// Every sum is taken in the order of fw_sqn_split.hip (a quad, the slice's 64 quads, the slices; the rows
// in four quarters; the pairs by wavefront), so a run's iterates and pairs are the same bits.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "exchange.hpp"
#include "sqn.hpp"
#include "sqn_device.hpp"
#include "sqn_slice.hpp"
#include "sqn_split.hpp"
#include "wave_dpp.hpp"

namespace fw {

namespace {

constexpr uint32_t kPitch = kSqnMaxM + 1;               // LDS pitch of the small matrices: a column's rows in different banks
constexpr uint32_t kSolve = 16;                         // terms of the triangular solve loaded together
constexpr uint32_t kPitchSY = kSqnMaxM + kSolve + 1;    // S'Y's rows and R^-1's columns are read that far past the end
constexpr uint32_t kRowsRi = kSqnMaxM + kSolve;
constexpr uint32_t kRedPitch = kSplitQuads + 1;         // the same for the quads' products
constexpr uint32_t kSlicesPerWave = kSplitMaxSlices / kSplitWaves;

// Bytes of the kernel's LDS, all of it dynamic.
struct Lds {
    double *xs;             // [kSplitMaxSlices][64] the sums one gather reads
    double *tot;            // [max(64, 3 M, 2 ceil(b_H / W))] what it makes of them
    double *sv, *sv_s;      // [257] the slice of a vector, zero in the last place
    double *part;           // [kSplitWaves][64][4]
    double *cs;             // [3][kSqnMaxM]
    double *SY, *YY, *Ri, *C;   // [kSqnMaxM][kPitchSY]; [kSqnMaxM], [kRowsRi] and [kSqnMaxM][kPitch]: zero past the pairs held
    double *coef;           // [max(b, b_H)]
    double *red;            // [3 M][kRedPitch]; the Hessian rows' bits before; T after
    uint32_t *bits;         // [b][kSliceWords]
    uint8_t *z;             // [b] labels
    uint32_t *fail;
    size_t bytes;
};

__host__ __device__ inline Lds lds_of(char *base, uint32_t M, uint32_t b, uint32_t bH, uint32_t W)
{
    Lds l;
    size_t at = 0;
    auto take = [&](size_t bytes) {
        char *p = base + at;
        at += (bytes + 15) / 16 * 16;
        return p;
    };
    auto doubles = [&](size_t n) { return reinterpret_cast<double *>(take(sizeof(double) * n)); };
    const uint32_t own = 2 * ((bH + W - 1) / W), most = 3 * M > own ? 3 * M : own;
    l.xs = doubles(kSplitMaxSlices * kSplitQuads);
    l.tot = doubles(most > 64 ? most : 64);
    l.sv = doubles(4 * kSplitQuads + 2);
    l.sv_s = doubles(4 * kSplitQuads + 2);
    l.part = doubles(kSplitWaves * kSplitQuads * 4);
    l.cs = doubles(3 * kSqnMaxM);
    l.SY = doubles(kSqnMaxM * kPitchSY);
    l.YY = doubles(kSqnMaxM * kPitch);
    l.Ri = doubles(kRowsRi * kPitch);
    l.C = doubles(kSqnMaxM * kPitch);
    l.coef = doubles(b > bH ? b : bH);
    const uint32_t quads = 3 * M * kRedPitch;
    const size_t red = sizeof(double) * (quads > kSqnMaxM * kPitch ? quads : kSqnMaxM * kPitch), hb = sizeof(uint32_t) * bH * kSliceWords;
    l.red = reinterpret_cast<double *>(take(red > hb ? red : hb));
    l.bits = reinterpret_cast<uint32_t *>(take(sizeof(uint32_t) * b * kSliceWords));
    l.z = reinterpret_cast<uint8_t *>(take(b));
    l.fail = reinterpret_cast<uint32_t *>(take(16));
    l.bytes = at;
    return l;
}

// A binary64 value as two tagged words, lo_off apart.
__device__ __forceinline__ void put2(uint64_t *slot, uint32_t lo_off, double v, uint32_t tag)
{
    const uint64_t b = static_cast<uint64_t>(__double_as_longlong(v));
    exchange_put(slot, static_cast<uint32_t>(b >> 32), tag);
    exchange_put(slot + lo_off, static_cast<uint32_t>(b), tag);
}

__device__ __forceinline__ double join2(uint64_t hi, uint64_t lo)
{
    return __longlong_as_double(static_cast<long long>((hi & 0xFFFFFFFF00000000ull) | (lo >> 32)));
}

// use(i, sum) for i < count: the sum over the W slices, in order, of the values at index index(i) of the
// slices' blocks (2 pad words each, high halves first). Wavefront wv reads slices wv, wv + 4, ..., all its
// loads in flight together; a chunk of 64 values at a time. xs holds zeros past slice W. What `use`
// writes to LDS is visible after it; past count it is called with 0.0, up to fill (at most the end of
// the last chunk). The other wavefronts take `meanwhile` beside the first chunk's sums. A value that
// does not come sets *fail.
template <class Index, class Use, class Meanwhile>
__device__ __forceinline__ void gather(const Slice &c, const uint64_t *blocks, uint32_t pad, uint32_t W, uint32_t tag,
                                       uint32_t count, uint32_t fill, double *xs, uint32_t *fail, Index index, Use use, Meanwhile meanwhile)
{
    FW_PIN_SGPR(pad);                                   // or every address of every gather stays in registers
    for (uint32_t base = 0; base < count; base += kSplitQuads) {
        const uint32_t i = base + c.ql, at = index(i < count ? i : count - 1);
        uint64_t hi[kSlicesPerWave], lo[kSlicesPerWave];
        bool seen;
        uint32_t polls = 0;
        do {
            seen = true;
#pragma unroll
            for (uint32_t j = 0; j < kSlicesPerWave; ++j) {
                const uint32_t u = c.wv + kSplitWaves * j;
                hi[j] = lo[j] = tag;
                if (u < W) {
                    const uint64_t *p = blocks + static_cast<size_t>(u) * 2 * pad;
                    hi[j] = exchange_get(p + at);
                    lo[j] = exchange_get(p + pad + at);
                }
            }
#pragma unroll
            for (uint32_t j = 0; j < kSlicesPerWave; ++j)
                seen = seen && static_cast<uint32_t>(hi[j]) == tag && static_cast<uint32_t>(lo[j]) == tag;
        } while (!seen && ++polls < kPollLimit);
        if (!seen) *fail = 1u;
#pragma unroll
        for (uint32_t j = 0; j < kSlicesPerWave; ++j) {
            const uint32_t u = c.wv + kSplitWaves * j;
            if (u < W) xs[u * kSplitQuads + c.ql] = join2(hi[j], lo[j]);
        }
        __syncthreads();
        if (c.wv == 0) {
            double a = 0.0;
            for (uint32_t u = 0; u < W; u += 8) {
                double v[8];
#pragma unroll
                for (uint32_t j = 0; j < 8; ++j) v[j] = xs[(u + j) * kSplitQuads + c.ql];
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (uint32_t j = 0; j < 8; ++j) a += v[j];
            }
            if (i < fill) use(i, i < count ? a : 0.0);
        } else if (base == 0) {
            meanwhile();
        }
        __syncthreads();
    }
}

// coef[0..count) from the workgroups that own the rows.
__device__ __forceinline__ void gather_coef(const Slice &c, const uint64_t *slots, uint32_t pad, uint32_t tag,
                                            uint32_t count, double *coef, uint32_t *fail)
{
    constexpr uint32_t kEach = kSqnMaxB / kSplitThreads;
    uint64_t hi[kEach], lo[kEach];
    bool seen;
    uint32_t polls = 0;
    do {
        seen = true;
#pragma unroll
        for (uint32_t j = 0; j < kEach; ++j) {
            hi[j] = lo[j] = tag;
            if (j * kSplitThreads < count) {
                const uint32_t i = min(j * kSplitThreads + c.tid, count - 1);
                hi[j] = exchange_get(slots + i);
                lo[j] = exchange_get(slots + pad + i);
            }
        }
#pragma unroll
        for (uint32_t j = 0; j < kEach; ++j)
            seen = seen && static_cast<uint32_t>(hi[j]) == tag && static_cast<uint32_t>(lo[j]) == tag;
    } while (!seen && ++polls < kPollLimit);
    if (!seen) *fail = 1u;
#pragma unroll
    for (uint32_t j = 0; j < kEach; ++j) {
        const uint32_t i = j * kSplitThreads + c.tid;
        if (i < count) coef[i] = join2(hi[j], lo[j]);
    }
    __syncthreads();
}

// The slice's bits of an iteration's sampled rows: word u is half u & 1 (16 bytes) of row u / 2, with LABELS
// the row's label beside it. The threads from FIRST on take the words in turn; AHEAD words of a thread are
// on their way from start (which the threads before FIRST may skip) to finish, the others are read in finish.
template <bool LABELS, uint32_t AHEAD, uint32_t FIRST>
struct RowFetch {
    static constexpr uint32_t kThreads = kSplitThreads - FIRST;
    uint4 v[AHEAD];
    uint8_t z[AHEAD];

    __device__ __forceinline__ void load(const SqnSplit &P, const Slice &c, uint64_t k, uint32_t dom, uint32_t u, uint4 &x,
                                         uint8_t &label)
    {
        const SqnArgs &A = P.A;
        const uint32_t n4 = A.xw / 4, i = u >> 1, e = i & 3u;
        const Words4 r = philox4x32_10(i >> 2, static_cast<uint32_t>(k), c.rep, (dom << 24) | A.inst, A.k0, A.k1);
        const uint32_t row = __umulhi(e < 2 ? (e == 0 ? r.x0 : r.x1) : (e == 2 ? r.x2 : r.x3), A.N);
        const uint32_t u4 = 2 * c.s + (u & 1u);
        x = reinterpret_cast<const uint4 *>(A.X + static_cast<size_t>(row) * A.xw)[u4 < n4 ? u4 : n4 - 1];
        if (u4 >= n4) x.x = x.y = x.z = x.w = 0u;
        if constexpr (LABELS) label = A.z[row];
    }

    __device__ __forceinline__ void start(const SqnSplit &P, const Slice &c, uint64_t k, uint32_t dom, uint32_t count)
    {
        if (c.wv * kSplitQuads < FIRST) return;
        const uint32_t first = c.wv * kSplitQuads - FIRST;
#pragma unroll
        for (uint32_t j = 0; j < AHEAD; ++j)
            if (j * kThreads + first < 2 * count)
                load(P, c, k, dom, min(j * kThreads + c.tid - FIRST, 2 * count - 1), v[j], z[j]);
    }

    __device__ __forceinline__ void finish(const SqnSplit &P, const Slice &c, uint64_t k, uint32_t dom, uint32_t count,
                                           uint32_t *bits, uint8_t *labels)
    {
        if (c.wv * kSplitQuads < FIRST) return;
#pragma unroll
        for (uint32_t j = 0; j < AHEAD; ++j) {
            const uint32_t u = j * kThreads + c.tid - FIRST;
            if (u >= 2 * count) continue;
            reinterpret_cast<uint4 *>(bits)[u] = v[j];
            if constexpr (LABELS) labels[u >> 1] = z[j];
        }
        for (uint32_t u = AHEAD * kThreads + c.tid - FIRST; u < 2 * count; u += kThreads) {
            uint4 x;
            uint8_t label = 0;
            load(P, c, k, dom, u, x, label);
            reinterpret_cast<uint4 *>(bits)[u] = x;
            if constexpr (LABELS) labels[u >> 1] = label;
        }
    }
};

// word_dot, four bits at a time: a place past the last bit adds the zero at v[256].
__device__ __forceinline__ double word_dot4(uint32_t bits, const double *v, uint32_t j0)
{
    double a = 0.0;
    while (bits) {
        double x[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            x[e] = v[bits ? j0 + static_cast<uint32_t>(__builtin_ctz(bits)) : 4 * kSplitQuads];
            bits &= bits - 1;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) a += x[e];
    }
    return a;
}

// 0.0 + x + the next seven lanes' x, in order; the first lane of each eight has it.
__device__ __forceinline__ double sum_words(double x)
{
    double a = 0.0;
    a += x;
    a += dpp_move<0x12F>(x);
    a += dpp_move<0x12E>(x);
    a += dpp_move<0x12D>(x);
    a += dpp_move<0x12C>(x);
    a += dpp_move<0x12B>(x);
    a += dpp_move<0x12A>(x);
    a += dpp_move<0x129>(x);
    return a;
}

// This slice's part of x_i'v for the staged rows (v's slice in sv) into the block's value i: a lane per
// bitmap word, a row's eight words in order.
__device__ __forceinline__ void put_row_dots(const Slice &c, const uint32_t *bits, uint32_t count, const double *sv,
                                             uint64_t *block, uint32_t pad, uint32_t tag)
{
    for (uint32_t base = 0; base < kSliceWords * count; base += kSplitThreads) {
        const uint32_t u = base + c.tid;
        const uint32_t w = u < kSliceWords * count ? bits[u] : 0u;
        const double a = sum_words(word_dot4(w, sv, 32u * (u % kSliceWords)));
        if (u % kSliceWords == 0 && u < kSliceWords * count) put2(block + u / kSliceWords, pad, a, tag);
    }
}

// The sums over the slice's 64 quads, in order, of red[v][.] into the block's value v.
__device__ __forceinline__ void put_column_sums(const Slice &c, const double *red, uint32_t count, uint64_t *block,
                                                uint32_t pad, uint32_t tag)
{
    if (c.tid < count) {
        double a = 0.0;
        for (uint32_t l = 0; l < kSplitQuads; l += 32) {
            double v[32];
#pragma unroll
            for (uint32_t j = 0; j < 32; ++j) v[j] = red[c.tid * kRedPitch + l + j];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (uint32_t j = 0; j < 32; ++j) a += v[j];
        }
        put2(block + c.tid, pad, a, tag);
    }
}

// The sum over q in [0, n) of x(q) y(q), in order, sixteen terms' loads together; the terms up to the next
// multiple of 16 have to be 0.
template <class X, class Y>
__device__ __forceinline__ double dot_in_order(uint32_t n, X x, Y y)
{
    double a = 0.0;
    for (uint32_t q = 0; q < n; q += 16) {
        double u[16], v[16];
#pragma unroll
        for (uint32_t j = 0; j < 16; ++j) {
            u[j] = x(q + j);
            v[j] = y(q + j);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (uint32_t j = 0; j < 16; ++j) a += u[j] * v[j];
    }
    return a;
}

// The small matrices with the new pair (sums s_i'y, y_i'y in tot[2i], tot[2i + 1], s'y_i in
// tot[2m + i]): S'Y and Y'Y extended, the oldest dropped when the ring was full, gamma, R^-1 and
// C = R^-T (D + gamma Y'Y) R^-1; T is scratch. Sums as sqn_split_small. Column c of R^-1 follows from
// rows and columns up to c, so the columns held before keep their values and only the last is solved
// for, by one thread (each entry's sum begins with the entry before it), while three wavefronts form
// T's other columns.
__device__ __forceinline__ double rebuild_small(const Slice &c, const Lds &l, uint32_t m, bool full)
{
    const uint32_t tid = c.tid, n1 = m - 1, col = tid % 32, row0 = tid / 32;
    double *SY = l.SY, *YY = l.YY, *Ri = l.Ri, *T = l.red;
    if (full) {
        constexpr uint32_t kRows = kSqnMaxM / 8;
        double a[kRows], b[kRows], d[kRows];
#pragma unroll
        for (uint32_t j = 0; j < kRows; ++j) {
            const uint32_t i = row0 + 8 * j, at = (i + 1) * kPitch + col + 1;
            if (i < n1 && col < n1) a[j] = SY[(i + 1) * kPitchSY + col + 1], b[j] = YY[at], d[j] = Ri[at];
        }
        __syncthreads();
#pragma unroll
        for (uint32_t j = 0; j < kRows; ++j) {
            const uint32_t i = row0 + 8 * j, at = i * kPitch + col;
            if (i < n1 && col < n1) SY[i * kPitchSY + col] = a[j], YY[at] = b[j], Ri[at] = d[j];
        }
    }
    if (tid < m) {
        if (tid < n1) SY[n1 * kPitchSY + tid] = l.tot[2 * m + tid], Ri[n1 * kPitch + tid] = 0.0;
        SY[tid * kPitchSY + n1] = l.tot[2 * tid];
        YY[tid * kPitch + n1] = l.tot[2 * tid + 1];
        YY[n1 * kPitch + tid] = l.tot[2 * tid + 1];
    }
    __syncthreads();
    const double gamma = SY[n1 * kPitchSY + n1] / YY[n1 * kPitch + n1];
    // T = (D + gamma Y'Y) R^-1; a thread has a column and every STEP-th row
    auto t_column = [&](auto rows, uint32_t j, uint32_t i0, uint32_t step) {
        constexpr uint32_t ROWS = decltype(rows)::value;
        double a[ROWS] = {}, dii[ROWS];
#pragma unroll
        for (uint32_t e = 0; e < ROWS; ++e) dii[e] = SY[min(i0 + step * e, n1) * (kPitchSY + 1)];
#pragma unroll 4
        for (uint32_t q = 0; q <= n1; ++q) {
            const double x = Ri[q * kPitch + j];
#pragma unroll
            for (uint32_t e = 0; e < ROWS; ++e) {
                const uint32_t i = min(i0 + step * e, n1);
                const double dl = gamma * YY[i * kPitch + q] + (i == q ? dii[e] : 0.0);
                a[e] += (q <= j ? dl : 0.0) * x;        // x is 0 from row j + 1 on
            }
        }
#pragma unroll
        for (uint32_t e = 0; e < ROWS; ++e)
            if (i0 + step * e < m) T[(i0 + step * e) * kPitch + j] = a[e];
    };
    if (c.wv > 0) {
        if (col < n1) t_column(std::integral_constant<uint32_t, (kSqnMaxM + 5) / 6>{}, col, row0 - 2, 6);
    } else if (tid == 0) {
        // R x = e_n1 from the last entry up; an entry's first loads go out before the division before it
        double last = 1.0 / SY[n1 * kPitchSY + n1], s[kSolve], x[kSolve], first = 0.0, dii = 1.0;
        Ri[n1 * kPitch + n1] = last;
        auto load = [&](const double *row, uint32_t q) {
#pragma unroll
            for (uint32_t j = 0; j < kSolve; ++j) {
                s[j] = row[q + j];
                x[j] = Ri[(q + j) * kPitch + n1];
            }
        };
        auto begin = [&](int i) {
            const double *row = SY + i * kPitchSY;
            dii = row[i];
            first = row[i + 1];
            load(row, i + 2);
        };
        if (n1 > 0) begin(static_cast<int>(n1) - 1);
        for (int i = static_cast<int>(n1) - 1; i >= 0; --i) {
            double a = 0.0;
            a += first * last;
            for (uint32_t q = i + 2; q <= n1;) {
#pragma unroll
                for (uint32_t j = 0; j < kSolve; ++j) a += s[j] * x[j];
                q += kSolve;
                if (q <= n1) {
                    load(SY + i * kPitchSY, q);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            const double d = dii;
            if (i > 0) begin(i - 1);
            __builtin_amdgcn_sched_barrier(0);
            last = -a / d;
            Ri[i * kPitch + n1] = last;
        }
    }
    __syncthreads();
    if (tid < m) t_column(std::integral_constant<uint32_t, 1>{}, n1, tid, 1);
    __syncthreads();
    if (col < m) {
        constexpr uint32_t kRows = kSqnMaxM / 8;
        double a[kRows] = {};
#pragma unroll 4
        for (uint32_t q = 0; q <= n1; ++q) {
            const double t = T[q * kPitch + col];
#pragma unroll
            for (uint32_t e = 0; e < kRows; ++e) {      // R^-1 is 0 from row i + 1 on
                const uint32_t i = min(row0 + 8 * e, n1);
                a[e] += Ri[q * kPitch + i] * (q <= i ? t : 0.0);
            }
        }
#pragma unroll
        for (uint32_t e = 0; e < kRows; ++e)
            if (row0 + 8 * e < m) l.C[(row0 + 8 * e) * kPitch + col] = a[e];
    }
    __syncthreads();
    return gamma;
}

// [small matrices of P.small] <-> LDS, m x m each
template <bool STORE>
__device__ __forceinline__ void move_small(const Slice &c, const Lds &l, double *small, uint32_t m)
{
    double *const at[4] = {l.SY, l.YY, l.Ri, l.C};
    for (uint32_t v = c.tid; v < m * m; v += kSplitThreads) {
        const uint32_t i = v / m, j = v % m;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            double *g = small + a * kSqnMaxM * kSqnMaxM + i * kSqnMaxM + j, *e = at[a] + i * (a == 0 ? kPitchSY : kPitch) + j;
            if constexpr (STORE) *g = *e;
            else *e = *g;
        }
    }
}

}  // namespace

// 256 threads, a workgroup per slice and replication, at most one per compute unit.
template <typename PT>
__global__ __launch_bounds__(kSplitThreads) void sqn_split_run_kernel(SqnSplit P, SqnSplitRun Q)
{
    HIP_DYNAMIC_SHARED(double, lds)
    const SqnArgs &A = P.A;
    Slice c = slice_of(P);
    const uint32_t W = P.W, M = A.M, b = A.b, bH = A.bH;
    const Lds l = lds_of(reinterpret_cast<char *>(lds), M, b, bH, W);
    const size_t ld = A.ld;
    if (failure_get(Q.fail)) return;                    // an earlier launch of the run gave up

    const SqnSplitSlots sl = sqn_split_slots(M, b, bH, W);
    uint64_t *words = Q.words + c.rep * sl.total;
    auto x_blocks = [&](uint64_t k) { return words + sl.x + (k & 1) * static_cast<size_t>(W) * 2 * sl.bp; };
    uint64_t *d_blocks = words + sl.d, *h_blocks = words + sl.h, *y_blocks = words + sl.y;
    uint64_t *cx = words + sl.cx, *ch = words + sl.ch;
    const bool shared_rows = b > kSplitQuads;           // the rows' sums are shared out

    PT *S = static_cast<PT *>(A.S) + static_cast<size_t>(c.rep) * M * ld + 4 * c.qc;
    PT *Y = static_cast<PT *>(A.Y) + static_cast<size_t>(c.rep) * M * ld + 4 * c.qc;
    double *small = P.small + static_cast<size_t>(c.rep) * kSqnSmall;
    const size_t at = c.rep * ld + 4 * c.qc;

    // the state between launches
    const uint64_t windows = (Q.k0 - 1) / A.L;
    uint64_t formed = windows > 0 ? windows - 1 : 0;    // pairs formed before iteration k
    uint32_t m = formed < M ? static_cast<uint32_t>(formed) : M;
    uint32_t head = formed < M ? 0u : static_cast<uint32_t>(formed % M);
    auto ring = [&](uint32_t i) { return head + i < M ? head + i : head + i - M; };     // slot of pair i, oldest first
    double w4[4] = {0.0, 0.0, 0.0, 0.0}, a4[4] = {0.0, 0.0, 0.0, 0.0}, pv[4] = {0.0, 0.0, 0.0, 0.0};
    double sq[kPairPerWave][4], yq[kPairPerWave][4];
    double gamma = 0.0;
    for (uint32_t v = c.tid; v < kSplitMaxSlices * kSplitQuads; v += kSplitThreads) l.xs[v] = 0.0;
    for (uint32_t v = c.tid; v < kSqnMaxM * kPitch; v += kSplitThreads) l.YY[v] = l.C[v] = 0.0;
    for (uint32_t v = c.tid; v < kSqnMaxM * kPitchSY; v += kSplitThreads) l.SY[v] = 0.0;
    for (uint32_t v = c.tid; v < kRowsRi * kPitch; v += kSplitThreads) l.Ri[v] = 0.0;
    __syncthreads();
    if (c.tid == 0) {
        l.sv[4 * kSplitQuads] = l.sv_s[4 * kSplitQuads] = 0.0;
        *l.fail = 0u;
    }
    RowFetch<true, 2, kSplitQuads> rows;
    rows.start(P, c, Q.k0, kSqnDomGrad, b);
    if (Q.k0 > 1) {
        load4(P.w + at, w4);
        load4(A.acc + at, a4);
        load4(A.wprev + at, pv);
#pragma unroll
        for (uint32_t j = 0; j < kPairPerWave; ++j) {
            const uint32_t i = c.wv + kSplitWaves * j;
            if (i < m) {
                load4(S + ring(i) * ld, sq[j]);
                load4(Y + ring(i) * ld, yq[j]);
            }
        }
        move_small<false>(c, l, small, m);
        gamma = small[4 * kSqnMaxM * kSqnMaxM];
    }
    rows.finish(P, c, Q.k0, kSqnDomGrad, b, l.bits, l.z);
    stage_slice(c, w4, l.sv);
    __syncthreads();
    put_row_dots(c, l.bits, b, l.sv, x_blocks(Q.k0) + static_cast<size_t>(c.s) * 2 * sl.bp, sl.bp,
                 static_cast<uint32_t>(Q.k0));

    uint32_t left = A.L - static_cast<uint32_t>((Q.k0 - 1) % A.L);     // iterations to the window's end
    for (uint64_t k = Q.k0; k < Q.k1; ++k) {
        // or every address and condition that follows from them is kept in registers over the iterations
        FW_PIN_VGPR(c.tid);
        FW_PIN_VGPR(c.ql);
        FW_PIN_SGPR(c.wv);
        FW_PIN_SGPR(m);
        const uint32_t tag = static_cast<uint32_t>(k);
        const bool qn = k > 2ull * A.L, more = k + 1 < Q.k1;
        auto fetch = [&] {
            if (more) rows.start(P, c, k + 1, kSqnDomGrad, b);
        };
        // the residuals of the rows
        if (!shared_rows) {
            gather(c, x_blocks(k), sl.bp, W, tag, b, b, l.xs, l.fail, [](uint32_t i) { return i; },
                   [&](uint32_t i, double a) { l.coef[i] = sigmoid(a) - static_cast<double>(l.z[i]); }, fetch);
        } else {
            const uint32_t per = (b + W - 1) / W, i0 = min(b, c.s * per), i1 = min(b, i0 + per);
            gather(c, x_blocks(k), sl.bp, W, tag, i1 - i0, i1 - i0, l.xs, l.fail, [&](uint32_t i) { return i0 + i; },
                   [&](uint32_t i, double a) { put2(cx + i0 + i, sl.bp, sigmoid(a) - static_cast<double>(l.z[i0 + i]), tag); }, [] {});
            fetch();
            gather_coef(c, cx, sl.bp, tag, b, l.coef, l.fail);
        }
        if (*l.fail) break;
        double g[4];
        slice_bit_sum(c, l.bits, l.coef, b, reinterpret_cast<double (*)[kSplitQuads][4]>(l.part), g);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            g[e] /= static_cast<double>(b);
            a4[e] += w4[e];
        }
        const double alpha = A.beta / static_cast<double>(k);
        if (!qn) {
#pragma unroll
            for (int e = 0; e < 4; ++e) w4[e] -= alpha * g[e];
            __syncthreads();                            // the rows' bits and labels are read
        } else {
            // s_i'g and y_i'g, pair i oldest first
#pragma unroll
            for (uint32_t j = 0; j < kPairPerWave; ++j) {
                const uint32_t i = c.wv + kSplitWaves * j;
                if (i < m) {
                    l.red[(2 * i) * kRedPitch + c.ql] = c.own ? dot4(sq[j], g) : 0.0;
                    l.red[(2 * i + 1) * kRedPitch + c.ql] = c.own ? dot4(yq[j], g) : 0.0;
                }
            }
            __syncthreads();
            put_column_sums(c, l.red, 2 * m, d_blocks + static_cast<size_t>(c.s) * 2 * sl.dp, sl.dp, tag);
            gather(c, d_blocks, sl.dp, W, tag, 2 * m, kSplitQuads, l.xs, l.fail, [](uint32_t i) { return i; },
                   [&](uint32_t i, double a) { l.tot[i] = a; }, [] {});
            if (*l.fail) break;
            // the compact representation's coefficients: cs = C S'g - gamma R^-T Y'g, cy = -gamma R^-1 S'g
            if (c.ql < m) {
                const uint32_t i = c.ql;
                double a = 0.0;
                if (c.wv == 0)
                    a = dot_in_order(m, [&](uint32_t q) { return l.C[i * kPitch + q]; }, [&](uint32_t q) { return l.tot[2 * q]; });
                else if (c.wv == 1)                     // zero from row i + 1 on
                    a = dot_in_order(m, [&](uint32_t q) { return l.Ri[q * kPitch + i]; },
                                     [&](uint32_t q) { return q <= i ? l.tot[2 * q + 1] : 0.0; });
                else if (c.wv == 2)
                    a = dot_in_order(m, [&](uint32_t q) { return l.Ri[i * kPitch + q]; },
                                     [&](uint32_t q) { return q >= i ? l.tot[2 * q] : 0.0; });
                if (c.wv < 3) l.cs[c.wv * kSqnMaxM + i] = a;
            }
            __syncthreads();
            double pd[4] = {0.0, 0.0, 0.0, 0.0};
            double cs[kPairPerWave], cy[kPairPerWave];
#pragma unroll
            for (uint32_t j = 0; j < kPairPerWave; ++j) {
                const uint32_t i = c.wv + kSplitWaves * j;
                cs[j] = l.cs[i] - gamma * l.cs[kSqnMaxM + i];
                cy[j] = -gamma * l.cs[2 * kSqnMaxM + i];
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (uint32_t j = 0; j < kPairPerWave; ++j)
                if (c.wv + kSplitWaves * j < m) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) pd[e] += sq[j][e] * cs[j] + yq[j][e] * cy[j];
                }
            double(*s_pd)[kSplitQuads][4] = reinterpret_cast<double (*)[kSplitQuads][4]>(l.part);
#pragma unroll
            for (int e = 0; e < 4; ++e) s_pd[c.wv][c.ql][e] = pd[e];
            __syncthreads();
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                double dir = gamma * g[e];
                for (uint32_t u = 0; u < kSplitWaves; ++u) dir += s_pd[u][c.ql][e];
                w4[e] -= alpha * dir;
            }
        }
        if (c.owner) {
            for (uint32_t q = 0; q < A.n_ckpt; ++q)
                if (A.ckpt[q] == k) store4(A.wsnap + static_cast<size_t>(q) * A.R * ld + at, w4);
            if (k == A.K) store4(A.wsnap + static_cast<size_t>(A.n_ckpt) * A.R * ld + at, w4);
        }
        const bool window = --left == 0, pair = window && k > A.L;
        if (window) left = A.L;
        if (more) {
            stage_slice(c, w4, l.sv);
            rows.finish(P, c, k + 1, kSqnDomGrad, b, l.bits, l.z);
            __syncthreads();
            put_row_dots(c, l.bits, b, l.sv, x_blocks(k + 1) + static_cast<size_t>(c.s) * 2 * sl.bp, sl.bp, tag + 1);
        }
        if (!window) continue;

        // the window average, s, and y = Eq. (13) applied to s
        RowFetch<false, 3, 0> hrows;
        if (pair) hrows.start(P, c, k, kSqnDomHess, bH);
        double wb[4], s_new[4], y[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            wb[e] = a4[e] / static_cast<double>(A.L);
            s_new[e] = wb[e] - pv[e];
            pv[e] = wb[e];
            a4[e] = 0.0;
        }
        if (!pair) continue;
        const bool full = m == M;
        const uint32_t slot = full ? head : ring(m);
        if (c.owner) store4(S + slot * ld, s_new);
        // s as stored (rounded to the pairs' type)
#pragma unroll
        for (int e = 0; e < 4; ++e) s_new[e] = static_cast<double>(static_cast<PT>(s_new[e]));
        if (full) head = ring(1);
        else ++m;
        ++formed;
        uint32_t *hbits = reinterpret_cast<uint32_t *>(l.red);
        __syncthreads();                                // sv's readers are done
        stage_slice(c, wb, l.sv);
        stage_slice(c, s_new, l.sv_s);
        hrows.finish(P, c, k, kSqnDomHess, bH, hbits, nullptr);
        __syncthreads();
        uint64_t *hb = h_blocks + static_cast<size_t>(c.s) * 2 * sl.hp;
        put_row_dots(c, hbits, bH, l.sv, hb, sl.hp, tag);            // x_i'wbar
        put_row_dots(c, hbits, bH, l.sv_s, hb + bH, sl.hp, tag);     // x_i's
        {
            const uint32_t per = (bH + W - 1) / W, i0 = min(bH, c.s * per), i1 = min(bH, i0 + per), own = i1 - i0;
            gather(c, h_blocks, sl.hp, W, tag, 2 * own, 2 * own, l.xs, l.fail,
                   [&](uint32_t i) { return i < own ? i0 + i : bH + i0 + i - own; },
                   [&](uint32_t i, double a) { l.tot[i] = a; }, [] {});
            for (uint32_t i = c.tid; i < own; i += kSplitThreads) {
                const double sg = sigmoid(l.tot[i]);
                put2(ch + i0 + i, sl.cp, sg * (1.0 - sg) * l.tot[own + i], tag);
            }
        }
        gather_coef(c, ch, sl.cp, tag, bH, l.coef, l.fail);
        if (*l.fail) break;
        // the pairs by their new ages
#pragma unroll
        for (uint32_t j = 0; j < kPairPerWave; ++j) {
            const uint32_t i = c.wv + kSplitWaves * j;
            if (i + 1 < m) {
                load4(S + ring(i) * ld, sq[j]);
                load4(Y + ring(i) * ld, yq[j]);
            }
        }
        slice_bit_sum(c, hbits, l.coef, bH, reinterpret_cast<double (*)[kSplitQuads][4]>(l.part), y);
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = static_cast<double>(static_cast<PT>(y[e] / static_cast<double>(bH)));
        if (c.owner) store4(Y + slot * ld, y);
#pragma unroll
        for (uint32_t j = 0; j < kPairPerWave; ++j) {
            const uint32_t i = c.wv + kSplitWaves * j;
            if (i < m) {
                if (i + 1 == m) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) sq[j][e] = s_new[e], yq[j][e] = y[e];
                }
                l.red[(2 * i) * kRedPitch + c.ql] = c.own ? dot4(sq[j], y) : 0.0;
                l.red[(2 * i + 1) * kRedPitch + c.ql] = c.own ? dot4(yq[j], y) : 0.0;
                l.red[(2 * m + i) * kRedPitch + c.ql] = c.own ? dot4(yq[j], s_new) : 0.0;
            }
        }
        __syncthreads();
        put_column_sums(c, l.red, 3 * m, y_blocks + static_cast<size_t>(c.s) * 2 * sl.yp, sl.yp, tag);
        gather(c, y_blocks, sl.yp, W, tag, 3 * m, 3 * m, l.xs, l.fail, [](uint32_t i) { return i; },
               [&](uint32_t i, double a) { l.tot[i] = a; }, [] {});
        if (*l.fail) break;
        gamma = rebuild_small(c, l, m, full);
    }
    if (*l.fail) {
        if (c.tid == 0) failure_raise(Q.fail);
        return;
    }
    if (c.owner) {
        store4(P.w + at, w4);
        store4(A.acc + at, a4);
        store4(A.wprev + at, pv);
    }
    if (c.s == 0) {
        move_small<true>(c, l, small, m);
        if (c.tid == 0) {
            small[4 * kSqnMaxM * kSqnMaxM] = gamma;
            A.pairs[c.rep] = static_cast<uint32_t>(formed);
        }
    }
}

namespace {

const void *run_fn(const SqnSplit &P)
{
    return P.A.pairs_fp32 ? reinterpret_cast<const void *>(&sqn_split_run_kernel<float>)
                          : reinterpret_cast<const void *>(&sqn_split_run_kernel<double>);
}

size_t run_lds(const SqnSplit &P) { return lds_of(nullptr, P.A.M, P.A.b, P.A.bH, P.W).bytes; }

}  // namespace

bool sqn_split_run_fits(const SqnSplit &P, int device)
{
    int cus = 0, coop = 0, per_cu = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess ||
        hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, device) != hipSuccess || !coop ||
        static_cast<uint64_t>(P.W) * P.A.R > static_cast<uint64_t>(cus))
        return false;
    const size_t lds = run_lds(P);
    if (lds > kSqnLdsPerCu) return false;
    // the form's largest size, not this run's: the attribute is the function's, for every context and thread
    if (hipFuncSetAttribute(run_fn(P), hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(kSqnLdsPerCu)) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, run_fn(P), kSplitThreads, lds) == hipSuccess && per_cu >= 1;
}

int launch_sqn_split_run(const SqnSplit &P, const SqnSplitRun &Q, hipStream_t s)
{
    SqnSplit p = P;
    SqnSplitRun q = Q;
    void *args[] = {&p, &q};
    return launch_cooperative(run_fn(P), dim3(P.W, P.A.R), kSplitThreads, args, run_lds(P), s);
}

}  // namespace fw
