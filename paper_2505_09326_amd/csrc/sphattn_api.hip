// Host side of the C ABI declared in include/sphattn.h: argument checks, kernel
// selection by (dtype, d), launch on the caller's stream.  Allocates nothing and
// never synchronises.
#include "sphattn_device.hpp"
#include "sphattn_pipelined.hpp"
#include "sphattn_keysplit.hpp"
#include "sphattn_f32.hpp"
#include "sphattn_softmax32.hpp"
#include "sphattn_backward.hpp"
#include "sphattn_fp8.hpp"
#include "sphattn_choice.hpp"
#include "../../include/sphattn.h"

#include <stdint.h>

#include <atomic>

namespace {

using namespace sphattn;

constexpr int kVersion = 510;   // 0.5.1

static_assert(kBC == kChoiceTile && kF32Tile == kChoiceF32Tile, "times per tile of the kernels' tiles");

// [a, a+an) and [b, b+bn) share a byte.  Written with differences, so that a range reaching the
// top of the address space cannot wrap the comparison.
bool overlaps(const void* a, size_t an, const void* b, size_t bn)
{
    const uintptr_t a0 = (uintptr_t)a, b0 = (uintptr_t)b;
    return a0 <= b0 ? b0 - a0 < an : a0 - b0 < bn;
}

// a buffer of `bytes` bytes at p would run past the end of the address space
bool wraps(const void* p, size_t bytes)
{
    return (uintptr_t)p + bytes < (uintptr_t)p;
}

int check_shape(int B, int H, int H_kv, int Nq, int Nk, int d, int dtype)
{
    if (B <= 0 || H <= 0 || Nq <= 0 || Nk <= 0 || H_kv <= 0 || H % H_kv != 0) return SPHATTN_ERR_SHAPE;
    if (d != 64 && d != 128) return SPHATTN_ERR_HEAD_DIM;
    if (dtype != SPHATTN_F32 && dtype != SPHATTN_BF16 && dtype != SPHATTN_FP8QK_BF16V &&
        dtype != SPHATTN_F16)
        return SPHATTN_ERR_DTYPE;
    const unsigned __int128 nmax = Nq > Nk ? Nq : Nk;
    // B*H*N*d elements must be addressable with 64-bit offsets and B*H*tiles with int
    if ((unsigned __int128)B * H * nmax * d > ((unsigned __int128)1 << 40)) return SPHATTN_ERR_SHAPE;
    if ((unsigned __int128)B * H * ((nmax + 31) / 32) > 0x7fffffff) return SPHATTN_ERR_SHAPE;
    // one head of one tensor is addressed through a 32-bit buffer range
    if (nmax * d * 4 > 0x7fffffff) return SPHATTN_ERR_SHAPE;
    return SPHATTN_OK;
}

// `out` is what the call writes (out_bytes of it); it must not overlap anything the call reads.
int check_args(const void* Q, const void* K, const void* V, const void* out, size_t out_bytes,
               const float* mult, const float* Z,
               int B, int H, int H_kv, int Nq, int Nk, int d, int dtype)
{
    if (!Q || !K || !V || !out) return SPHATTN_ERR_NULL;
    const int rc = check_shape(B, H, H_kv, Nq, Nk, d, dtype);
    if (rc != SPHATTN_OK) return rc;
    if (((uintptr_t)Q | (uintptr_t)K | (uintptr_t)V | (uintptr_t)out) & 15) return SPHATTN_ERR_ALIGN;
    if (((uintptr_t)mult | (uintptr_t)Z) & 3) return SPHATTN_ERR_ALIGN;
    const size_t nq = (size_t)B * H * Nq * d, nkv = (size_t)B * H_kv * Nk * d;
    const size_t qk = dtype == SPHATTN_F32 ? 4 : dtype == SPHATTN_FP8QK_BF16V ? 1 : 2;
    const size_t vo = dtype == SPHATTN_F32 ? 4 : 2;
    const size_t zb = (size_t)B * H * Nq * 4;
    if (wraps(out, out_bytes) || wraps(Q, nq * qk) || wraps(K, nkv * qk) || wraps(V, nkv * vo) ||
        (Z && wraps(Z, zb)) || (mult && wraps(mult, (size_t)B * Nk * 4)))
        return SPHATTN_ERR_SHAPE;
    if (overlaps(out, out_bytes, Q, nq * qk) || overlaps(out, out_bytes, K, nkv * qk) ||
        overlaps(out, out_bytes, V, nkv * vo) ||
        (mult && overlaps(out, out_bytes, mult, (size_t)B * Nk * 4)))
        return SPHATTN_ERR_ALIAS;
    if (Z && (overlaps(Z, zb, Q, nq * qk) || overlaps(Z, zb, K, nkv * qk) || overlaps(Z, zb, V, nkv * vo) ||
              overlaps(Z, zb, out, out_bytes) || (mult && overlaps(Z, zb, mult, (size_t)B * Nk * 4))))
        return SPHATTN_ERR_ALIAS;
    return SPHATTN_OK;
}

size_t out_bytes_of(int B, int H, int N, int d, int dtype)
{
    return (size_t)B * H * N * d * (dtype == SPHATTN_F32 ? 4 : 2);
}

// Kernels that use more than 64 KB of LDS need their limit raised once per device; `done` is
// that kernel's bit mask of devices already configured (the only state the library keeps).
long long cu_count();

// How many consecutive workgroups of one XCD's range run at the same time: that XCD's share of
// the compute units times the workgroups of this kernel that fit one unit.  Feeds the kernels'
// key-stream direction (see fwd_pipelined_kernel); asked once per kernel and device.
template <typename Kern>
int stream_period(Kern kern, int lds_bytes, std::atomic<int> (&cached)[64], int threads = kThreads)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
        (void)hipGetLastError();
        return 0;
    }
    int p = cached[dev].load(std::memory_order_relaxed);
    if (p == 0) {
        int per_cu = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)kern, threads, (size_t)lds_bytes) != hipSuccess ||
            per_cu <= 0) {
            (void)hipGetLastError();
            return 0;                              // 0: never reverse
        }
        p = (int)(cu_count() / kXcds) * per_cu;
        cached[dev].store(p, std::memory_order_relaxed);
    }
    return p;
}

template <typename Kern>
bool raise_lds_limit(Kern kern, int lds_bytes, std::atomic<uint64_t>& done)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
        (void)hipGetLastError();
        return false;
    }
    const uint64_t bit = 1ull << dev;
    if (done.load(std::memory_order_acquire) & bit) return true;
    if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                            lds_bytes) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    done.fetch_or(bit, std::memory_order_release);
    return true;
}

// A launch.  Whole problem: O is the output tensor, Z the optional row aggregates, n_splits 1.
// Partial accumulators: O is the fp32 slice-major o buffer, Z the z buffer, and the key axis
// is cut into n_splits slices of keys_per_split rows.
struct Problem {
    const void* Q; const void* K; const void* V; void* O; const float* mult; float* Z;
    int B, H, H_kv, Nq, Nk;
    hipStream_t stream;
    int n_splits = 1, keys_per_split = 0;
    int tile_rows = 0;          // query rows per workgroup: 0 = the library's choice, else 128 or 256
    bool one_key_order = false; // a launch below one round adds every row's terms in the 256-row kernel's order
};

// Query heads that share a K/V head lie next to each other, so their rows are one block of
// H / H_kv * Nq rows against that K/V head (Q, O, Z and the partial buffers alike, and the
// multiplicities belong to the batch entry): the launch sees H_kv heads of so many rows.  Whole
// tiles then run across the heads of a group: 4 heads of 64 queries are one tile of 256 rows
// instead of four quarter-filled ones that each stream the same K and V.  Not where one head's
// buffer range would pass 32 bits.
Problem packed_group(Problem p, int d)
{
    const long long group = p.H / p.H_kv;
    if (group > 1 && group * p.Nq * d * 4 <= 0x7fffffff) {
        p.Nq = (int)(group * p.Nq);
        p.H = p.H_kv;
    }
    return p;
}

// Key slices are whole 64-key tiles.  Asking for more slices than there are tiles, or for a
// count that does not divide them evenly, yields fewer, equally sized slices (the last may be
// shorter).
struct SplitPlan { int n_splits, keys_per_split; };
SplitPlan plan_splits(int Nk, int requested)
{
    const int tiles = (int)(((long long)Nk + kBC - 1) / kBC);   // >= 1: every caller has checked Nk >= 1
    requested = requested < 1 ? 1 : requested > tiles ? tiles : requested;
    const int per = (tiles + requested - 1) / requested;   // >= 1, and no overflow: requested <= tiles
    return SplitPlan{(tiles + per - 1) / per, per * kBC};
}

// Compute units of the current device, asked once per device; 256 (MI355X) when there is no
// device to ask.
long long cu_count()
{
    static std::atomic<int> cached[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
        (void)hipGetLastError();
        return 256;
    }
    int n = cached[dev].load(std::memory_order_relaxed);
    if (n <= 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) {
            (void)hipGetLastError();
            return 256;
        }
        cached[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

// Persistent workgroups for n_items work items when `resident` workgroups run at once (a multiple
// of the XCD count; 0 = unknown).  The items take ceil(n_items / resident) rounds; when the last
// round would be partly filled, the same number of rounds is run with fewer workgroups, all
// rounds equally full: the part is power-bound, so CUs left idle in every round give their
// share of the budget to the others as clock, while a last round of a few items runs alone at
// almost its usual duration (measured, 8 heads of d = 128, N = 41472: 162 query tiles per head on
// 32 CUs, 5.06 rounds; the 2 tiles of the sixth round cost 0.9 of a full round).
long long balanced_grid(long long n_items, long long resident)
{
    if (resident <= 0 || n_items <= resident) return n_items;
    const long long rounds = (n_items + resident - 1) / resident;
    long long grid = (n_items + rounds - 1) / rounds;
    grid = (grid + kXcds - 1) / kXcds * kXcds;
    return grid < resident ? grid : resident;
}

// The key-split kernel over a launch's items of 16 NQ RG query rows.
template <int D, int NQ, QKType QKT, bool MULT, bool PARTIAL, int RG, int KG, int CS = 1>
int launch_keysplit(const Problem& p)
{
    constexpr int BR = 16 * NQ * RG, threads = 64 * keysplit_waves<RG, KG>(), lds_bytes = keysplit_lds_bytes<D, NQ, RG, KG, QKT, MULT, D / CS>();
    auto kern = fwd_keysplit_kernel<D, NQ, QKT, MULT, PARTIAL, CS, RG, KG>;
    static std::atomic<uint64_t> done{0};
    static std::atomic<int> period[64];
    if (!raise_lds_limit(kern, lds_bytes, done)) return SPHATTN_ERR_LAUNCH;
    const int n_qtiles = (p.Nq + BR - 1) / BR;
    const long long n_wg = (long long)p.B * p.H * n_qtiles * p.n_splits * CS;
    if (n_wg > 0x7fffffff) return SPHATTN_ERR_SHAPE;
    const long long grid = balanced_grid(n_wg, (long long)kXcds * stream_period(kern, lds_bytes, period, threads));
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(threads), lds_bytes, p.stream,
                       p.Q, p.K, p.V, p.O, p.mult, p.Z, p.Nq, p.Nk, p.H, p.H / p.H_kv, n_qtiles, (int)n_wg,
                       p.n_splits, p.keys_per_split, 0, (int)n_wg, 0);
    return hipGetLastError() == hipSuccess ? SPHATTN_OK : SPHATTN_ERR_LAUNCH;
}

// The 128-row kernel on the remainder of a launch whose items do not fill their last round
// (launch_pipelined): items item_begin .. n_items - 1 of the 256-row numbering, one half of an
// item per workgroup.  resident_only: configure the kernel and return how many of its
// workgroups run at once (0: unknown) without launching.
template <int D, QKType QKT>
long long launch_halves(const Problem& p, int n_qtiles, int n_items, int item_begin, bool backwards, bool resident_only)
{
    constexpr int lds_bytes = keysplit_lds_bytes<D, 4, 2, 2, QKT, false>();
    auto kern = fwd_keysplit_kernel<D, 4, QKT, false, false, 1, 2, 2>;
    static std::atomic<uint64_t> done{0};
    static std::atomic<int> period[64];
    if (!raise_lds_limit(kern, lds_bytes, done)) return 0;
    const long long resident = (long long)kXcds * stream_period(kern, lds_bytes, period);
    if (resident_only) return resident;
    const int rest = n_items - item_begin;
    const unsigned grid = 2u * kXcds * (unsigned)((rest + kXcds - 1) / kXcds);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(kThreads), lds_bytes, p.stream,
                       p.Q, p.K, p.V, p.O, p.mult, p.Z, p.Nq, p.Nk, p.H, p.H / p.H_kv, n_qtiles, n_items,
                       1, 0, item_begin, n_items, backwards ? 2 : 1);
    return hipGetLastError() == hipSuccess ? resident : -1;
}

template <int D, int NQ, QKType QKT, Norm NORM, bool MULT, bool PARTIAL = false, int WAVES = kWaves>
int launch_pipelined(const Problem& p)
{
    constexpr int BR = WAVES * 16 * NQ, threads = 64 * WAVES;
    constexpr int lds_bytes = pipelined_lds_bytes<D, NQ, QKT, MULT, WAVES>();
    auto kern = fwd_pipelined_kernel<D, NQ, QKT, NORM, MULT, PARTIAL, WAVES>;
    static std::atomic<uint64_t> done{0};
    static std::atomic<int> period[64];
    if (!raise_lds_limit(kern, lds_bytes, done)) return SPHATTN_ERR_LAUNCH;
    const int n_qtiles = (p.Nq + BR - 1) / BR;
    const long long n_wg = (long long)p.B * p.H * n_qtiles * p.n_splits;
    if (n_wg > 0x7fffffff) return SPHATTN_ERR_SHAPE;
    const float scale_log2 = 1.4426950408889634f / __builtin_sqrtf((float)D);
    // persistent workgroups: as many as the chip runs at once (a multiple of the XCD count), or
    // one per item if that is fewer
    const long long resident = (long long)kXcds * stream_period(kern, lds_bytes, period, threads);
    // d = 64, a remainder of at most half a round behind at least one full round: the full rounds
    // run here and the remaining tiles as two 128-row halves each in a launch of their own, which
    // fills twice as many CUs for 0.6 of the time.  In full rounds, with f = remainder / resident:
    // rounds + 0.3 + 0.6 f against 0.5 (rounds + 1) + 0.5 (rounds + f) for the balanced grid (a
    // round filled to the fraction x takes about 0.5 + 0.5 x of a full one).  Measured: 20 heads of
    // 8192 x 64 (640 tiles, 1.25 rounds) 273 against 306 us, 12 x 12345 x 64 387 against 425 us.
    // At d = 128 the 128-row kernel is too much slower per row for this (8 x 41472 x 128: 4.84
    // against 4.66 ms, 4 x 20000 x 128: 649 against 632 us), and the balanced grid stays.
    constexpr bool HAS_HALVES = D == 64 && NQ == 4 && WAVES == kWaves && !PARTIAL && !MULT && NORM == Norm::Spherical && QKT != QKType::Fp8;
    if constexpr (HAS_HALVES) {
        const long long full = resident > 0 ? n_wg / resident : 0, rem = resident > 0 ? n_wg % resident : 0;
        if (p.tile_rows == 0 && full >= 1 && rem > 0) {
            const long long narrow = launch_halves<D, QKT>(p, n_qtiles, (int)n_wg, 0, false, true);
            const double f = (double)rem / (double)resident;
            if (2 * rem <= narrow && (double)full + 0.3 + 0.6 * f < 0.97 * ((double)full + 0.5 + 0.5 * f)) {
                const int n_main = (int)(full * resident);
                hipLaunchKernelGGL(kern, dim3((unsigned)resident), dim3(kThreads), lds_bytes, p.stream,
                                   p.Q, p.K, p.V, p.O, p.mult, p.Z,
                                   p.Nq, p.Nk, p.H, p.H / p.H_kv, n_qtiles, (int)n_wg,
                                   p.n_splits, p.keys_per_split, scale_log2, 0, n_main);
                if (hipGetLastError() != hipSuccess) return SPHATTN_ERR_LAUNCH;
                return launch_halves<D, QKT>(p, n_qtiles, (int)n_wg, n_main, full % 2 == 1, false) >= 0 ? SPHATTN_OK : SPHATTN_ERR_LAUNCH;
            }
        }
    }
    const long long grid = balanced_grid(n_wg, resident);
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(threads), lds_bytes, p.stream,
                       p.Q, p.K, p.V, p.O, p.mult, p.Z,
                       p.Nq, p.Nk, p.H, p.H / p.H_kv, n_qtiles, (int)n_wg,
                       p.n_splits, p.keys_per_split, scale_log2, 0, (int)n_wg);
    return hipGetLastError() == hipSuccess ? SPHATTN_OK : SPHATTN_ERR_LAUNCH;
}

// ROWS query rows per workgroup: 32 (four waves) or 16, of which CS workgroups share the columns of V
template <int D, int ROWS, bool MULT, bool PARTIAL, int CS = 1>
int launch_f32(const Problem& p)
{
    static_assert(ROWS == kF32SmallRows || CS == 1, "shares of the columns: 16 rows");
    constexpr bool SMALL = ROWS == kF32SmallRows;
    constexpr int waves = SMALL ? f32_small_waves<D>() : kWaves;
    constexpr int lds_bytes = SMALL ? f32_small_lds_bytes<D>() : waves * 2 * 32 * (D + 4) * 4;
    constexpr auto kern = SMALL ? fwd_f32_small_kernel<D, MULT, PARTIAL, CS> : fwd_f32_kernel<D, MULT, PARTIAL>;
    static std::atomic<uint64_t> done{0};
    if (!raise_lds_limit(kern, lds_bytes, done)) return SPHATTN_ERR_LAUNCH;
    const int n_qtiles = (p.Nq + ROWS - 1) / ROWS;
    const long long n_wg = (long long)p.B * p.H * n_qtiles * p.n_splits * CS;
    if (n_wg > 0x7fffffff) return SPHATTN_ERR_SHAPE;
    hipLaunchKernelGGL(kern, dim3((unsigned)n_wg), dim3(64 * waves), lds_bytes, p.stream,
                       (const float*)p.Q, (const float*)p.K, (const float*)p.V, (float*)p.O, p.mult, p.Z,
                       p.Nq, p.Nk, p.H, p.H / p.H_kv, n_qtiles, (int)n_wg,
                       p.n_splits, p.keys_per_split);
    return hipGetLastError() == hipSuccess ? SPHATTN_OK : SPHATTN_ERR_LAUNCH;
}

template <int D, int NQ, bool MULT, bool PARTIAL, bool TWO>
int launch_f32_parts(const Problem& p)
{
    constexpr int BR = kF32Waves * 16 * NQ, lds_bytes = f32_lds_bytes<D>();
    constexpr auto kern = TWO ? fwd_f32x2_kernel<D, NQ, MULT, PARTIAL> : fwd_f32x3_kernel<D, NQ, MULT, PARTIAL>;
    static std::atomic<uint64_t> done{0};
    if (!raise_lds_limit(kern, lds_bytes, done)) return SPHATTN_ERR_LAUNCH;
    const int n_qtiles = (p.Nq + BR - 1) / BR;
    const long long n_wg = (long long)p.B * p.H * n_qtiles * p.n_splits;
    if (n_wg > 0x7fffffff) return SPHATTN_ERR_SHAPE;
    hipLaunchKernelGGL(kern, dim3((unsigned)n_wg), dim3(64 * kF32Waves), lds_bytes, p.stream,
                       (const float*)p.Q, (const float*)p.K, (const float*)p.V, (float*)p.O, p.mult, p.Z,
                       p.Nq, p.Nk, p.H, p.H / p.H_kv, n_qtiles, (int)n_wg, p.n_splits, p.keys_per_split);
    return hipGetLastError() == hipSuccess ? SPHATTN_OK : SPHATTN_ERR_LAUNCH;
}

template <int D, bool MULT, bool PARTIAL>
int launch_f32_any(const Problem& p)
{
    const int rows = choose_f32((long long)p.B * p.H, p.Nq, PARTIAL ? p.keys_per_split : p.Nk, p.n_splits, D, cu_count()).rows;
    const bool two = f32_two_parts(PARTIAL ? p.keys_per_split : p.Nk, D);
    if (rows == 128) return two ? launch_f32_parts<D, 1, MULT, PARTIAL, true>(p) : launch_f32_parts<D, 1, MULT, PARTIAL, false>(p);
    if (rows == 256) return two ? launch_f32_parts<D, 2, MULT, PARTIAL, true>(p) : launch_f32_parts<D, 2, MULT, PARTIAL, false>(p);
    if (rows == 32) return launch_f32<D, 32, MULT, PARTIAL>(p);
    switch (f32_small_column_shares((long long)p.B * p.H * p.n_splits, p.Nq, cu_count())) {
    case 4: return launch_f32<D, 16, MULT, PARTIAL, 4>(p);
    case 2: return launch_f32<D, 16, MULT, PARTIAL, 2>(p);
    default: return launch_f32<D, 16, MULT, PARTIAL>(p);
    }
}

template <int D>
int launch_softmax32(const Problem& p)
{
    constexpr int BR = 256;
    constexpr int lds_bytes = kNBuf * kBC * (D * 2 + kKPad + D * 2 + kVPad);
    auto kern = softmax32_kernel<D>;
    static std::atomic<uint64_t> done{0};
    if (!raise_lds_limit(kern, lds_bytes, done)) return SPHATTN_ERR_LAUNCH;
    const int n_qtiles = (p.Nq + BR - 1) / BR;
    const long long n_wg = (long long)p.B * p.H * n_qtiles;
    if (n_wg > 0x7fffffff) return SPHATTN_ERR_SHAPE;
    const float scale_log2 = 1.4426950408889634f / __builtin_sqrtf((float)D);
    hipLaunchKernelGGL(kern, dim3((unsigned)n_wg), dim3(kThreads), lds_bytes, p.stream,
                       p.Q, p.K, p.V, p.O, p.Nq, n_qtiles, (int)n_wg, scale_log2);
    return hipGetLastError() == hipSuccess ? SPHATTN_OK : SPHATTN_ERR_LAUNCH;
}

template <int D, QKType QKT, bool MULT, bool PARTIAL>
int launch_spherical(const Problem& p)
{
    constexpr bool FP8 = QKT == QKType::Fp8, BF16 = QKT == QKType::Bf16;
    const long long slices = (long long)p.B * p.H * p.n_splits, tiles = ((PARTIAL ? p.keys_per_split : p.Nk) + kBC - 1) / kBC, cus = cu_count();
    const Storage st{BF16 && !PARTIAL, FP8, MULT};
    const FormChoice choice = p.tile_rows != 0 ? FormChoice{p.tile_rows == 128 ? kRows128 : kRows256, 0.0} : choose_form(slices, p.Nq, tiles, D, st, cus);
    if constexpr (!FP8) {
        const int shares = p.one_key_order ? 1 : column_shares(choice, slices, p.Nq, tiles, D, st, cus);
        if constexpr (D == 128)
            if (shares == 4) return launch_keysplit<D, 2, QKT, MULT, PARTIAL, 2, 4, 4>(p);
        if (shares == 2) return launch_keysplit<D, 2, QKT, MULT, PARTIAL, 2, 4, 2>(p);
    }
    Form form = choice.form;
    if (p.one_key_order) form = in_one_key_order(form, tiles, BF16 && !MULT && !PARTIAL);
    if constexpr (BF16 && !MULT && !PARTIAL)
        if (form == kNarrow) return launch_pipelined<D, 2, QKT, Norm::Spherical, MULT, PARTIAL>(p);
    if constexpr (!(FP8 && D == 128)) {
        if (form == kRows64) return launch_keysplit<D, 2, QKT, MULT, PARTIAL, 2, 2>(p);
        if (form == kRows64Wide) return launch_keysplit<D, 2, QKT, MULT, PARTIAL, 2, 4>(p);
    }
    if constexpr (D == 128) {
        if (form == kRows64Own) return launch_keysplit<D, 4, QKT, MULT, PARTIAL, 1, 4>(p);
    } else {
        if (form == kRows128Wide) return launch_keysplit<D, 4, QKT, MULT, PARTIAL, 2, 4>(p);
        if (form == kRows256Wide) return launch_keysplit<D, 4, QKT, MULT, PARTIAL, 4, 2>(p);
    }
    if (form == kRows128) return launch_keysplit<D, 4, QKT, MULT, PARTIAL, 2, 2>(p);
    if constexpr (D == 64 && !(FP8 && MULT))
        if (p.tile_rows == 0 && rows512_pay(slices, p.Nq, tiles, Storage{BF16, FP8, MULT}, !PARTIAL, cus)) return launch_pipelined<D, 4, QKT, Norm::Spherical, MULT, PARTIAL, 8>(p);
    return launch_pipelined<D, 4, QKT, Norm::Spherical, MULT, PARTIAL>(p);
}

// Spherical attention in any storage type; PARTIAL: accumulators over key slices.
template <bool MULT, bool PARTIAL = false>
int dispatch_spherical(const Problem& call, int d, int dtype)
{
    const Problem p = packed_group(call, d);
    switch (dtype) {
    case SPHATTN_BF16:
        return d == 128 ? launch_spherical<128, QKType::Bf16, MULT, PARTIAL>(p) : launch_spherical<64, QKType::Bf16, MULT, PARTIAL>(p);
    case SPHATTN_F16:
        return d == 128 ? launch_spherical<128, QKType::F16, MULT, PARTIAL>(p) : launch_spherical<64, QKType::F16, MULT, PARTIAL>(p);
    case SPHATTN_FP8QK_BF16V:
        return d == 128 ? launch_spherical<128, QKType::Fp8, MULT, PARTIAL>(p) : launch_spherical<64, QKType::Fp8, MULT, PARTIAL>(p);
    case SPHATTN_F32:
        return d == 128 ? launch_f32_any<128, MULT, PARTIAL>(p) : launch_f32_any<64, MULT, PARTIAL>(p);
    default:
        return SPHATTN_ERR_DTYPE;
    }
}

// The other normalizers: bf16, and the SoftMax twin also with fp8 Q/K.
template <Norm NORM>
int dispatch_normalizer(const Problem& p, int d, int dtype)
{
    if (dtype == SPHATTN_BF16)
        return d == 128 ? launch_pipelined<128, 4, QKType::Bf16, NORM, false>(p) : launch_pipelined<64, 4, QKType::Bf16, NORM, false>(p);
    if constexpr (NORM == Norm::Softmax) {
        if (dtype == SPHATTN_FP8QK_BF16V)
            return d == 128 ? launch_pipelined<128, 4, QKType::Fp8, NORM, false>(p) : launch_pipelined<64, 4, QKType::Fp8, NORM, false>(p);
    }
    return SPHATTN_ERR_DTYPE;
}

template <int D>
int launch_combine(const float* o_parts, const float* z_parts, int n_parts, void* O, float* Z,
                   size_t rows, int dtype, hipStream_t stream)
{
    const size_t threads = rows * (D / 4);
    const size_t blocks = (threads + 255) / 256;
    if (blocks > 0x7fffffff) return SPHATTN_ERR_SHAPE;
    const bool resident = parts_resident((size_t)n_parts, rows * D * 4);
    const auto kern = dtype == SPHATTN_F32 ? (resident ? combine_kernel<D, 0, true> : combine_kernel<D, 0, false>)
                    : dtype == SPHATTN_F16 ? (resident ? combine_kernel<D, 2, true> : combine_kernel<D, 2, false>)
                                           : (resident ? combine_kernel<D, 1, true> : combine_kernel<D, 1, false>);
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), 0, stream, o_parts, z_parts, n_parts, O, Z, rows);
    return hipGetLastError() == hipSuccess ? SPHATTN_OK : SPHATTN_ERR_LAUNCH;
}

struct BwdProblem {
    const void* Q; const void* K; const void* V; const float* mult; const void* O; const void* dO;
    const float* Z; void* dQ; void* dK; void* dV; float* delta;
    int B, H, H_kv, N;
    hipStream_t stream;
};

// Slices of the two backward kernels' streamed axes, and where their partial sums go.
struct BwdPlan {
    int sq = 1, keys_per_split = 0;                // dQ: slices of the keys
    int sk = 1, tiles_per_split = 0;               // dK, dV: slices of the 64-query tiles
    size_t bytes = 0;                              // of workspace: sq parts of dQ, then sk of dK, then sk of dV
};

// A backward problem as launched: shared K/V heads packed like the forward's (packed_group), one query head
// of Nq = kv_group N rows per K/V head.
struct BwdShape { int H, kv_group, Nq; };
BwdShape bwd_shape(int H, int H_kv, int N, int d)
{
    const long long group = H / H_kv;
    if (group > 1 && group * N * d * 4 <= 0x7fffffff) return BwdShape{H_kv, 1, (int)(group * N)};
    return BwdShape{H, (int)group, N};
}

template <int D, bool HALF, bool MULT, bool PARTQ, bool PARTK>
int launch_bwd(const BwdProblem& p, const BwdPlan& plan, float* parts)
{
    constexpr int NK = 2, tile = kBC * D * 2;
    constexpr int lds_dq = bwd_dq_lds_bytes<D, MULT>(), lds_dkv = 2 * (2 * tile + 2 * kBC * 4) + (MULT ? kWaves * NK * 16 * 4 : 0);
    auto kq = bwd_dq_kernel<D, HALF, MULT, PARTQ>;
    auto kkv = bwd_dkv_kernel<D, HALF, MULT, NK, PARTK>;
    static std::atomic<uint64_t> done_q{0}, done_kv{0};
    if (!raise_lds_limit(kq, lds_dq, done_q) || !raise_lds_limit(kkv, lds_dkv, done_kv)) return SPHATTN_ERR_LAUNCH;
    const BwdShape sh = bwd_shape(p.H, p.H_kv, p.N, D);
    const int n_qtiles = (sh.Nq + 255) / 256, n_ktiles = (p.N + 64 * NK - 1) / (64 * NK);
    const long long wg_q = (long long)p.B * sh.H * n_qtiles * plan.sq, wg_kv = (long long)p.B * p.H_kv * n_ktiles * plan.sk;
    if (wg_q > 0x7fffffff || wg_kv > 0x7fffffff) return SPHATTN_ERR_SHAPE;
    // the two planes of delta (delta_i r_i^2, then r_i) are written by the first kernel and read
    // by the second, in stream order
    float* rnorm = p.delta + (size_t)p.B * p.H * p.N;
    const size_t nq = (size_t)p.B * p.H * p.N * D, nk = (size_t)p.B * p.H_kv * p.N * D;
    float *parts_k = nullptr, *parts_v = nullptr;
    if constexpr (PARTK) {
        parts_k = parts + (PARTQ ? plan.sq * nq : 0);
        parts_v = parts_k + plan.sk * nk;
    }
    hipLaunchKernelGGL(kq, dim3((unsigned)wg_q), dim3(kThreads), lds_dq, p.stream,
                       p.Q, p.K, p.V, p.mult, p.O, p.dO, p.Z, PARTQ ? (void*)parts : p.dQ, p.delta, rnorm,
                       sh.Nq, p.N, sh.H, sh.kv_group, n_qtiles, (int)wg_q, plan.sq, plan.keys_per_split);
    if (hipGetLastError() != hipSuccess) return SPHATTN_ERR_LAUNCH;
    hipLaunchKernelGGL(kkv, dim3((unsigned)wg_kv), dim3(kThreads), lds_dkv, p.stream,
                       p.Q, p.K, p.V, p.mult, p.dO, (const float*)rnorm, (const float*)p.delta,
                       PARTK ? (void*)parts_k : p.dK, PARTK ? (void*)parts_v : p.dV,
                       sh.Nq, p.N, sh.H, sh.kv_group, n_ktiles, (int)wg_kv, plan.sk, plan.tiles_per_split);
    if (hipGetLastError() != hipSuccess) return SPHATTN_ERR_LAUNCH;
    if constexpr (PARTQ || PARTK) {
        const size_t n4q = PARTQ ? nq / 4 : 0, n4k = PARTK ? nk / 4 : 0, blocks = (n4q + 2 * n4k + 255) / 256;
        if (blocks > 0x7fffffff) return SPHATTN_ERR_SHAPE;
        const size_t most = (size_t)(plan.sq > plan.sk ? plan.sq : plan.sk);
        const bool resident = parts_resident(most, plan.bytes / most);
        const auto kern = resident ? bwd_combine_kernel<HALF, true> : bwd_combine_kernel<HALF, false>;
        hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), 0, p.stream,
                           (const float*)parts, plan.sq, n4q, p.dQ, (const float*)parts_k, (const float*)parts_v, plan.sk, n4k, p.dK, p.dV);
        if (hipGetLastError() != hipSuccess) return SPHATTN_ERR_LAUNCH;
    }
    return SPHATTN_OK;
}

template <int D, bool HALF, bool MULT>
int launch_bwd_plan(const BwdProblem& p, const BwdPlan& plan, void* workspace)
{
    float* parts = (float*)workspace;
    if (plan.sq > 1 && plan.sk > 1) return launch_bwd<D, HALF, MULT, true, true>(p, plan, parts);
    if (plan.sq > 1) return launch_bwd<D, HALF, MULT, true, false>(p, plan, parts);
    if (plan.sk > 1) return launch_bwd<D, HALF, MULT, false, true>(p, plan, parts);
    return launch_bwd<D, HALF, MULT, false, false>(p, plan, parts);
}

template <bool MULT>
int dispatch_bwd(const BwdProblem& p, int d, int dtype, const BwdPlan& plan, void* workspace)
{
    if (dtype == SPHATTN_F16) return d == 128 ? launch_bwd_plan<128, true, MULT>(p, plan, workspace) : launch_bwd_plan<64, true, MULT>(p, plan, workspace);
    return d == 128 ? launch_bwd_plan<128, false, MULT>(p, plan, workspace) : launch_bwd_plan<64, false, MULT>(p, plan, workspace);
}

size_t workspace_bytes(int B, int H, int N, int d, int n_splits)
{
    const size_t rows = (size_t)B * H * N;
    return ((size_t)n_splits * rows * (d + 1) * 4 + 255) & ~(size_t)255;
}

// The two launches of the split-key forward on checked arguments: partial pairs of every slice
// into `workspace` (o parts, then z parts), then their sum and the tail.  Every partial the
// second launch reads is written by the first (every planned slice holds at least one tile),
// so the workspace needs no clearing.
int run_splitkv(Problem p, int d, int dtype, int requested, SplitPlan plan, void* workspace)
{
    if (plan.n_splits == 1) {                      // nothing to combine: the unsplit launch
        p.one_key_order = requested == 1;          // one slice asked for by name (as the header says)
        return p.mult ? dispatch_spherical<true>(p, d, dtype) : dispatch_spherical<false>(p, d, dtype);
    }
    const size_t rows = (size_t)p.B * p.H * p.Nq;
    void* O = p.O;
    float* Z = p.Z;
    float* o_parts = (float*)workspace;
    float* z_parts = o_parts + (size_t)plan.n_splits * rows * d;
    p.O = o_parts;
    p.Z = z_parts;
    p.n_splits = plan.n_splits;
    p.keys_per_split = plan.keys_per_split;
    const int r1 = p.mult ? dispatch_spherical<true, true>(p, d, dtype) : dispatch_spherical<false, true>(p, d, dtype);
    if (r1 != SPHATTN_OK) return r1;
    return d == 128 ? launch_combine<128>(o_parts, z_parts, plan.n_splits, O, Z, rows, dtype, p.stream)
                    : launch_combine<64>(o_parts, z_parts, plan.n_splits, O, Z, rows, dtype, p.stream);
}

struct Fp8Problem {
    const unsigned char* Q; const unsigned char* K; const unsigned char* VT; const float* kmax; const float* mult; unsigned short* O;
    int B, H, H_kv, N, n_tiles;
    hipStream_t stream;
};

template <int D, bool SOFTMAX, bool MULT, int NQ, int WAVES>
int launch_fp8_shape(const Fp8Problem& p)
{
    constexpr int lds_bytes = 4 * (2 * kFp8Tile * D + (MULT ? kFp8Tile * 4 : 0)), BR = 16 * NQ * WAVES;
    static std::atomic<uint64_t> done{0};
    static std::atomic<int> period[64];
    auto kern = fwd_fp8_kernel<D, SOFTMAX, MULT, NQ, WAVES>;
    if (!raise_lds_limit(kern, lds_bytes, done)) return SPHATTN_ERR_LAUNCH;
    const int n_qtiles = (p.N + BR - 1) / BR;
    const long long n_wg = (long long)p.B * p.H * n_qtiles;   // (fits: check_shape counts 32-row tiles)
    hipLaunchKernelGGL(kern, dim3((unsigned)n_wg), dim3(64 * WAVES), lds_bytes, p.stream,
                       p.Q, p.K, p.VT, p.kmax, p.mult, p.O, p.N, p.H, p.H / p.H_kv, p.n_tiles, n_qtiles, (int)n_wg,
                       stream_period(kern, lds_bytes, period, 64 * WAVES), fp8_chunks((long long)p.B * p.H_kv, p.n_tiles));
    return hipGetLastError() == hipSuccess ? SPHATTN_OK : SPHATTN_ERR_LAUNCH;
}

template <int D, bool MULT>
int launch_fp8(const Fp8Problem& p)
{
    const Fp8Shape shape = choose_fp8((long long)p.B * p.H, p.N, D, MULT, cu_count());
    if (shape.nq == 1) return shape.waves == 4 ? launch_fp8_shape<D, false, MULT, 1, 4>(p) : launch_fp8_shape<D, false, MULT, 1, 8>(p);
    if constexpr (D == 64) {
        if (shape.waves == 4 && shape.nq == 2) return launch_fp8_shape<D, false, MULT, 2, 4>(p);
        if constexpr (!MULT)
            if (shape.nq == 4) return launch_fp8_shape<D, false, MULT, 4, 4>(p);
    }
    return launch_fp8_shape<D, false, MULT, 2, 8>(p);
}

int fp8_forward(const void* Q, const void* K, const void* V, const float* mult, void* O, void* workspace,
                       size_t workspace_bytes, int B, int H, int H_kv, int N, int d, void* stream, bool softmax)
{
    if (d != 64 && d != 128) return SPHATTN_ERR_HEAD_DIM;
    if (!Q || !K || !V || !O) return SPHATTN_ERR_NULL;
    const int rc = check_shape(B, H, H_kv, N, N, d, SPHATTN_FP8QK_BF16V);
    if (rc != SPHATTN_OK) return rc;
    if (((uintptr_t)Q | (uintptr_t)K | (uintptr_t)V | (uintptr_t)O) & 15) return SPHATTN_ERR_ALIGN;
    if ((uintptr_t)mult & 3) return SPHATTN_ERR_ALIGN;
    const size_t in_bytes = (size_t)B * H * N * d, kv_bytes = (size_t)B * H_kv * N * d, m_bytes = (size_t)B * N * 4;
    if (wraps(O, in_bytes * 2) || wraps(Q, in_bytes) || wraps(K, kv_bytes) || wraps(V, kv_bytes) ||
        (mult && wraps(mult, m_bytes)))
        return SPHATTN_ERR_SHAPE;
    if (overlaps(O, in_bytes * 2, Q, in_bytes) || overlaps(O, in_bytes * 2, K, kv_bytes) ||
        overlaps(O, in_bytes * 2, V, kv_bytes) || (mult && overlaps(O, in_bytes * 2, mult, m_bytes)))
        return SPHATTN_ERR_ALIAS;
    const size_t need = sphattn_fp8_workspace_bytes(B, H_kv, N, d);
    if (!workspace || ((uintptr_t)workspace & 15) || workspace_bytes < need || wraps(workspace, need))
        return SPHATTN_ERR_WORKSPACE;
    if (overlaps(workspace, need, Q, in_bytes) || overlaps(workspace, need, K, kv_bytes) ||
        overlaps(workspace, need, V, kv_bytes) || overlaps(workspace, need, O, in_bytes * 2) ||
        (mult && overlaps(workspace, need, mult, m_bytes)))
        return SPHATTN_ERR_ALIAS;
    const int heads = B * H_kv;                    // K/V heads: what the preparation pass covers
    const int n_tiles = (N + kFp8Tile - 1) / kFp8Tile;
    const size_t kmax_bytes = ((size_t)heads * 4 + 255) & ~(size_t)255;
    float* kmax = (float*)workspace;
    unsigned char* VT = (unsigned char*)workspace + kmax_bytes;
    hipStream_t st = (hipStream_t)stream;
    if ((long long)heads * n_tiles > 0x7fffffff) return SPHATTN_ERR_SHAPE;
    if ((long long)B * H * ((N + 255) / 256) > 0x7fffffff) return SPHATTN_ERR_SHAPE;
    if ((unsigned __int128)d * n_tiles * kFp8Tile > 0x7fffffff) return SPHATTN_ERR_SHAPE;   // one head of V^T: a 32-bit range
    // two or three launches; the attention kernel's attribute (the one thing that can fail without a
    // launch) is set by its launcher before it enqueues anything, so a refusal there leaves the
    // workspace written and nothing else
    const int n_chunks = fp8_chunks(heads, n_tiles);
    if (n_chunks == 0) {
        hipLaunchKernelGGL(fp8_clear_kernel, dim3((heads + 255) / 256), dim3(256), 0, st, kmax, heads);
        if (hipGetLastError() != hipSuccess) return SPHATTN_ERR_LAUNCH;
    }
    const long long prep_wg = (long long)heads * (n_tiles + n_chunks);
    if (prep_wg > 0x7fffffff) return SPHATTN_ERR_SHAPE;
    auto prepare = d == 128 ? (n_chunks ? fp8_prepare_kernel<128, true> : fp8_prepare_kernel<128, false>)
                            : (n_chunks ? fp8_prepare_kernel<64, true> : fp8_prepare_kernel<64, false>);
    hipLaunchKernelGGL(prepare, dim3((unsigned)prep_wg), dim3(256), 0, st,
                       (const unsigned char*)K, (const unsigned char*)V, mult, VT, kmax, N, n_tiles, H_kv, heads, n_chunks);
    if (hipGetLastError() != hipSuccess) return SPHATTN_ERR_LAUNCH;
    const Fp8Problem p{(const unsigned char*)Q, (const unsigned char*)K, VT, kmax, mult, (unsigned short*)O, B, H, H_kv, N, n_tiles, st};
    if (softmax)                                   // (the shape of the spherical kernel's large launches)
        return d == 128 ? launch_fp8_shape<128, true, false, 2, 8>(p) : launch_fp8_shape<64, true, false, 4, 4>(p);
    if (d == 128) return mult ? launch_fp8<128, true>(p) : launch_fp8<128, false>(p);
    return mult ? launch_fp8<64, true>(p) : launch_fp8<64, false>(p);
}

// Key slices for `heads` heads of Nq query rows against Nk keys, as sphattn_splitkv_fwd chooses them: 1 where
// cutting is not expected to gain at least 3 %, otherwise the count with the lowest estimated run time.  The
// estimate is of 256-row workgroups (32-row ones in fp32) and of an unsplit launch from before there were 64-row ones;
// plan_cross below prices the shapes that launches take.  In us, unsplit / this choice / plan_cross's: 1 x 8192 x 128 54 / 50 / 38,
// 1 x 8192 x 64 36 / 34 / 23, 1 x 2048 x 128 17 / 12.7 / 14, fp32 1 x 8192 x 128 348 / 348 / 151, fp32 4 x 1000 x 64 15.7 / 20.1 / 15.7; only this one
// cuts 16-bit launches above one round (1 x 40000 x 128 642 / 532).
int choose_splits(long long heads, long long Nq, long long Nk, int d, int dtype)
{
    const long long cus = cu_count();
    const long long tiles = (Nk + kBC - 1) / kBC;
    const long long most = (tiles + 7) / 8;        // no slice shorter than 8 tiles
    if (dtype == SPHATTN_F32) {
        // workgroups of 32 query rows: enough slices to give every CU one
        const long long wg = heads * ((Nq + 31) / 32);
        if (wg >= cus) return 1;
        const long long want = (cus + wg - 1) / wg;
        return plan_splits((int)Nk, (int)(want < most ? want : most)).n_splits;
    }
    // 256-row workgroups, `resident` of them at once (two per CU at d = 64).  A launch of wg S
    // items takes rounds = ceil(wg S / resident) rounds, run equally full (balanced_grid); a round
    // filled to the fraction f of the chip takes about 0.5 + 0.5 f of a full round's time (the
    // part is power-bound: idle CUs give their share of the budget to the rest), and an item
    // spends about 3.5 tile times on its prologue and tail.  In units of one full round over all
    // keys: main(S) = (0.5 rounds / S + 0.5 wg / resident) (1 + 3.5 / tiles per slice); the combine
    // step adds its launch (about 3 tile times) and S passes over wg / resident of the rows, 300 / Nk
    // of a round each.  Unsplit, a launch of at most `resident` 128-row workgroups costs
    // 0.6 (0.5 + wg / resident) on the same scale.  Measured against these (bf16, one GPU, unsplit as it was then):
    // 1 x 8192 x 128: S = 8 44 us (4: 57, unsplit 99); 2 x 8192 x 128: S = 4; 1 x 32768 x 128: S = 2;
    // 8 x 4096 x 128: unsplit; 1 x 40000 x 128 (157 tiles): S = 3 533 us (2: 645, unsplit 629);
    // 3 x 16384 x 128 (192 tiles): S = 4 291 us (2: 300, unsplit 298); 5 x 16384 x 64: S = 3 251 (unsplit 285).
    // The same holds above one round: 8 x 20000 x 128 (632 tiles, 2.47 rounds): S = 2 1080 us, unsplit 1174.
    const long long wg = heads * ((Nq + 255) / 256);
    const long long resident = cus * (d == 64 ? 2 : 1);
    const double share = (double)wg / (double)resident;
    const double edge = 3.5;
    const long long rounds1 = (wg + resident - 1) / resident;
    double best = (0.5 * (double)rounds1 + 0.5 * share) * (1.0 + edge / (double)tiles);
    if (d == 64 && (dtype == SPHATTN_BF16 || dtype == SPHATTN_F16) && wg > resident && wg % resident != 0 &&
        2 * (wg % resident) <= resident) {
        // the unsplit launch runs this remainder as 128-row halves (launch_pipelined)
        const double halves = ((double)(wg / resident) + 0.3 + 0.6 * (double)(wg % resident) / (double)resident) *
                              (1.0 + edge / (double)tiles);
        best = halves < best ? halves : best;
    }
    if (wg < resident && heads * ((Nq + 127) / 128) <= resident) {
        const double narrow = 0.6 * (0.5 + share) * (1.0 + edge / (double)tiles);
        best = narrow < best ? narrow : best;
    }
    best *= 0.97;                                  // split only for a gain of at least 3 %
    int pick = 1;
    for (long long S = 2; S <= most && S <= 32; ++S) {
        const SplitPlan plan = plan_splits((int)Nk, (int)S);
        if (plan.n_splits != S) continue;          // this count does not divide the tiles: same as a smaller one
        const long long rounds = (wg * S + resident - 1) / resident;
        const double per = (double)(plan.keys_per_split / kBC);
        const double cost = (0.5 * (double)rounds / (double)S + 0.5 * share) * (1.0 + edge / per)
                            + 3.0 / (double)tiles + (double)S * share * 300.0 / (double)Nk;
        // above one round the workspace is large: more slices only for more than 1 %
        if (cost < (wg >= resident ? 0.99 : 1.0) * best) {
            best = cost;
            pick = (int)S;
        }
    }
    return pick;
}

// The library's choice of slices for a rectangular problem, in the launch's terms (packed_group).
// A launch is cut only while all its slices still run at once as workgroups of 128 rows or fewer, one
// per CU (1 x 8192 x 64 in 4 slices, 256 workgroups, 23.8 us; 6: 26.6; 12: 34.8).  Either side is priced as the launch it would be
// (choose_form, choose_f32; shares of the columns, which both sides may be launched in, change no more than the two's difference on short
// axes: priced, 1 x 2048 x 128 13.9 -> 12.5 us, with counts 14.2 -> 14.4, 1 x 4000 x 64 12.2 -> 14.0), as without counts, which the plan does not know and which raise both, and without Narrow, which parts have not
// and with which no plan over 2535 shapes differs; the second launch costs 4 us, and each part is written and read at 6 TB/s together.
// Measured with the slices this picks against one: 1 x 8192 x 128 38 against 44 us, 1 x 8192 x 64 24 against 27.5; not cut:
// 4 x 1999 x 128 (22.7 at best against 15.7), 8 x 1000 x 128 (18.1 against 10.9).
SplitPlan plan_cross(int B, int H, int H_kv, int Nq, int Nk, int d, int dtype)
{
    Problem p{};
    p.B = B; p.H = H; p.H_kv = H_kv; p.Nq = Nq; p.Nk = Nk;
    p = packed_group(p, d);
    const long long heads = (long long)p.B * p.H, cus = cu_count();
    const long long items = heads * ((p.Nq + kSplitRows - 1) / kSplitRows);
    const int tiles = (Nk + kBC - 1) / kBC;
    const double part_us = (double)heads * (double)p.Nq * (d + 1) * 8.0 / 6e6;
    SplitPlan best = plan_splits(Nk, 1);
    double best_us = 0.0;
    // (fp32 also above one round, whose remainder cutting recovers: choose_f32 counts rounds;
    // 1 x 21694 x 128, 170 workgroups of 128 rows, 1464 us uncut, 951 in 3 slices of 256-row workgroups)
    const long long most = dtype == SPHATTN_F32 ? 4 * cus : cus;
    long long last = 0;
    // (every count up to 16, then in steps of an eighth: this runs on every call that may be cut)
    for (long long want = 1; (want * items <= most || want == 1) && want <= tiles; want += want < 16 ? 1 : want / 8) {
        const SplitPlan plan = plan_splits(Nk, (int)want);
        const long long S = plan.n_splits;
        if (S == last) continue;                   // the same slices as a smaller count
        last = S;
        const double per = (double)(S == 1 ? tiles : plan.keys_per_split / kBC);
        double us;
        if (dtype == SPHATTN_F32) {
            us = 6.0 + choose_f32(heads, p.Nq, S == 1 ? Nk : plan.keys_per_split, S, d, cus).us;
        } else {
            us = choose_form(S * heads, p.Nq, (long long)per, d, Storage{false, dtype == SPHATTN_FP8QK_BF16V, false}, cus).us;
        }
        if (S > 1) us += 4.0 + (double)S * part_us;
        if (S == 1) best_us = 0.9 * us;            // cut only for a gain of at least 10 %
        else if (us < best_us) { best_us = us; best = plan; }
    }
    return best;
}

// How many slices a backward kernel's streamed axis of `tiles` 64-row tiles is cut into, for `items` tiles of
// the other axis, `per_cu` workgroups at once on a CU, tau us per streamed tile in a full round and
// part_us for writing and reading one slice's partial sums (6 TB/s).  A slice costs what its tiles and
// about 5 more cost.  Where a round does not give every CU its `per_cu` the fullest CU counts: one of two workgroups
// alone takes 0.62 of the time of both, one or two of three 0.48 and 0.74.  Below one round an emptier chip
// also clocks higher (power-bound part); a last round of one workgroup per CU behind full ones costs 0.85 + 0.15 f
// of one if it fills the share f.  Cut for a gain of at least 5 % below one round and 2 % above it, into slices
// of 4 tiles or more and at most 256 MB of sums.  Whole backward in us, bf16, uncut / this choice: below one
// round 8 heads on 2 K/V heads of 1500 x 64 126 / 41, of 1500 x 128 207 / 62; 4 x 1000 x 128 68 / 44; 2 x 8192 x 128
// 438 / 210; 12 on 3 of 4096 x 64 325 / 168; 12 x 4096 x 128 (0.75 of a round in both) stays uncut: 304, 332 in 4
// slices of the keys, 330 in 4 of the queries.  Above it 3 x 25243 x 128 (1.16 rounds in both kernels) 3255 / 2560,
// 9 x 8192 x 128 1077 / 945, 17 x 8192 x 64 895 / 840 (dQ alone, 1.06 rounds); left alone where the
// remainder is a workgroup more on most CUs: dK/dV of 16 x 8192 x 64 (1.33 rounds of three per CU) 708, in two
// slices 725, and of 16 x 5200 x 128 (1.28 of two) 696, 729.
long long choose_bwd_slices(long long items, int per_cu, long long tiles, double tau, double part_us, size_t part_bytes)
{
    const double alone[3][3] = {{1.0, 1.0, 1.0}, {0.62, 1.0, 1.0}, {0.48, 0.74, 1.0}};
    const long long cus = cu_count(), resident = cus * per_cu;
    long long best = 1;
    double best_us = 0.0;
    for (long long S = 1; S <= 64 && (S == 1 || (tiles / S >= 4 && (size_t)S * part_bytes <= ((size_t)256 << 20))); S += S < 16 ? 1 : S / 8) {
        const long long per = (tiles + S - 1) / S, n = items * S, full = n / resident;
        const double f = (double)(n % resident) / (double)resident;
        double rounds;
        if (full == 0) rounds = alone[per_cu - 1][(n + cus - 1) / cus - 1] * (n < cus ? 0.75 + 0.25 * (double)n / (double)cus : 1.0);
        else rounds = (double)full + (f == 0.0 ? 0.0 : per_cu == 1 ? 0.85 + 0.15 * f : alone[per_cu - 1][(n % resident + cus - 1) / cus - 1]);
        const double us = rounds * ((double)per + 5.0) * tau + (S > 1 ? 2.0 + (double)S * part_us : 0.0);
        if (S == 1) best_us = (full == 0 ? 0.95 : 0.98) * us;
        else if (us < best_us) { best_us = us; best = S; }
    }
    return best;
}

BwdPlan plan_bwd(int B, int H, int H_kv, int N, int d)
{
    const BwdShape sh = bwd_shape(H, H_kv, N, d);
    BwdPlan plan;
    const long long key_tiles = ((long long)N + kBC - 1) / kBC, query_tiles = (long long)sh.kv_group * ((sh.Nq + kBC - 1) / kBC);
    const long long items_q = (long long)B * sh.H * (((long long)sh.Nq + 255) / 256), items_k = (long long)B * H_kv * (((long long)N + 127) / 128);
    const size_t bytes_q = (size_t)B * H * N * d * 4, bytes_k = 2 * (size_t)B * H_kv * N * d * 4;
    // workgroups per CU: dQ one (d = 128) or two, dK/dV two or three; tau from launches of many rounds
    const long long sq = choose_bwd_slices(items_q, d == 128 ? 1 : 2, key_tiles, d == 128 ? 2.2 : 1.96, (double)bytes_q * 2.0 / 6e6, bytes_q);
    const long long sk = choose_bwd_slices(items_k, d == 128 ? 2 : 3, query_tiles, d == 128 ? 3.06 : 2.27, (double)bytes_k * 2.0 / 6e6, bytes_k);
    if (sq > 1) {
        const SplitPlan s = plan_splits(N, (int)sq);
        plan.sq = s.n_splits;
        plan.keys_per_split = s.keys_per_split;
    }
    if (sk > 1) {
        plan.tiles_per_split = (int)((query_tiles + sk - 1) / sk);
        plan.sk = (int)((query_tiles + plan.tiles_per_split - 1) / plan.tiles_per_split);
    }
    plan.bytes = ((plan.sq > 1 ? (size_t)plan.sq * bytes_q : 0) + (plan.sk > 1 ? (size_t)plan.sk * bytes_k : 0) + 255) & ~(size_t)255;
    return plan;
}

// The workspace of a split launch against its size and the other arguments.
int check_workspace(const Problem& p, int d, int dtype, SplitPlan plan, const void* workspace, size_t size)
{
    const size_t need = sphattn_splitkv_workspace_bytes(p.B, p.H, p.Nq, d, plan.n_splits);
    if (!workspace || need == 0 || size < need || ((uintptr_t)workspace & 15)) return SPHATTN_ERR_WORKSPACE;
    if (wraps(workspace, need)) return SPHATTN_ERR_WORKSPACE;
    const size_t nq = (size_t)p.B * p.H * p.Nq * d, nkv = (size_t)p.B * p.H_kv * p.Nk * d;
    const size_t qk = dtype == SPHATTN_F32 ? 4 : dtype == SPHATTN_FP8QK_BF16V ? 1 : 2;
    const size_t vo = dtype == SPHATTN_F32 ? 4 : 2;
    if (overlaps(workspace, need, p.Q, nq * qk) || overlaps(workspace, need, p.K, nkv * qk) ||
        overlaps(workspace, need, p.V, nkv * vo) || overlaps(workspace, need, p.O, out_bytes_of(p.B, p.H, p.Nq, d, dtype)) ||
        (p.mult && overlaps(workspace, need, p.mult, (size_t)p.B * p.Nk * 4)) ||
        (p.Z && overlaps(workspace, need, p.Z, (size_t)p.B * p.H * p.Nq * 4)))
        return SPHATTN_ERR_ALIAS;
    return SPHATTN_OK;
}

// Argument checks of the backward entry points.
int check_bwd(const void* Q, const void* K, const void* V, const float* mult, const void* O, const void* dO, const float* Z,
              void* dQ, void* dK, void* dV, float* delta, int B, int H, int H_kv, int N, int d, int dtype)
{
    if (!Q || !K || !V || !O || !dO || !Z || !dQ || !dK || !dV || !delta) return SPHATTN_ERR_NULL;
    const int rc = check_shape(B, H, H_kv, N, N, d, dtype);
    if (rc != SPHATTN_OK) return rc;
    if (dtype != SPHATTN_BF16 && dtype != SPHATTN_F16) return SPHATTN_ERR_DTYPE;
    if (((uintptr_t)Q | (uintptr_t)K | (uintptr_t)V | (uintptr_t)O | (uintptr_t)dO |
         (uintptr_t)dQ | (uintptr_t)dK | (uintptr_t)dV) & 15)
        return SPHATTN_ERR_ALIGN;
    if (((uintptr_t)Z | (uintptr_t)delta | (uintptr_t)mult) & 3) return SPHATTN_ERR_ALIGN;
    const size_t tq = (size_t)B * H * N * d * 2, tkv = (size_t)B * H_kv * N * d * 2, rb = (size_t)B * H * N * 4;
    const void* ins[7] = {Q, K, V, O, dO, Z, mult};
    const size_t in_bytes[7] = {tq, tkv, tkv, tq, tq, rb, mult ? (size_t)B * N * 4 : 0};
    void* outs[4] = {dQ, dK, dV, delta};
    const size_t out_bytes[4] = {tq, tkv, tkv, 2 * rb};
    for (int o = 0; o < 4; ++o) {
        for (int i = 0; i < 7; ++i)
            if (ins[i] && overlaps(outs[o], out_bytes[o], ins[i], in_bytes[i])) return SPHATTN_ERR_ALIAS;
        for (int q = o + 1; q < 4; ++q)
            if (overlaps(outs[o], out_bytes[o], outs[q], out_bytes[q])) return SPHATTN_ERR_ALIAS;
    }
    return SPHATTN_OK;
}

// Scratch memory of sphattn_splitkv_fwd_noalloc: one array per GPU, part of the library's code
// object, alive until the process ends.  Host code never uses the array's name as an address:
// its device address is asked for once per device (scratch_address) and kept.
static __device__ __align__(256) unsigned char scratch[SPHATTN_NOALLOC_SCRATCH_BYTES];

// Device address of `scratch` on the current device, or nullptr if the runtime cannot give it.
void* scratch_address()
{
    static std::atomic<void*> known[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
        (void)hipGetLastError();
        return nullptr;
    }
    void* p = known[dev].load(std::memory_order_acquire);
    if (p == nullptr) {
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) {
            (void)hipGetLastError();
            return nullptr;
        }
        known[dev].store(p, std::memory_order_release);
    }
    return p;
}

}  // namespace

extern "C" {

int sphattn_fwd(const void* Q, const void* K, const void* V, void* O,
                int B, int H, int N, int d, int dtype, void* stream)
{
    return sphattn_fwd_z(Q, K, V, O, nullptr, B, H, N, d, dtype, stream);
}

int sphattn_fwd_z(const void* Q, const void* K, const void* V, void* O, float* Z,
                  int B, int H, int N, int d, int dtype, void* stream)
{
    return sphattn_fwd_tile_rows(Q, K, V, O, Z, B, H, N, d, dtype, 0, stream);
}

int sphattn_fwd_tile_rows(const void* Q, const void* K, const void* V, void* O, float* Z,
                          int B, int H, int N, int d, int dtype, int tile_rows, void* stream)
{
    const int rc = check_args(Q, K, V, O, out_bytes_of(B, H, N, d, dtype), nullptr, Z, B, H, H, N, N, d, dtype);
    if (rc != SPHATTN_OK) return rc;
    if (tile_rows != 0 && tile_rows != 128 && tile_rows != 256) return SPHATTN_ERR_SHAPE;
    Problem p{Q, K, V, O, nullptr, Z, B, H, H, N, N, (hipStream_t)stream};
    p.tile_rows = tile_rows;
    return dispatch_spherical<false>(p, d, dtype);
}

int sphattn_grn_fwd(const void* Q, const void* K, const void* V, const float* mult, void* O,
                    int B, int H, int H_kv, int N, int d, int dtype, void* stream)
{
    const int rc = check_args(Q, K, V, O, out_bytes_of(B, H, N, d, dtype), mult, nullptr, B, H, H_kv, N, N, d, dtype);
    if (rc != SPHATTN_OK) return rc;
    const Problem p{Q, K, V, O, mult, nullptr, B, H, H_kv, N, N, (hipStream_t)stream};
    return mult ? dispatch_spherical<true>(p, d, dtype)
                : dispatch_spherical<false>(p, d, dtype);
}

int sphattn_cross_fwd(const void* Q, const void* K, const void* V, const float* mult, void* O, float* Z,
                      int B, int H, int H_kv, int N_q, int N_k, int d, int dtype, void* stream)
{
    const int rc = check_args(Q, K, V, O, out_bytes_of(B, H, N_q, d, dtype), mult, Z, B, H, H_kv, N_q, N_k, d, dtype);
    if (rc != SPHATTN_OK) return rc;
    const Problem p{Q, K, V, O, mult, Z, B, H, H_kv, N_q, N_k, (hipStream_t)stream};
    return mult ? dispatch_spherical<true>(p, d, dtype)
                : dispatch_spherical<false>(p, d, dtype);
}

int sphattn_normalized_fwd(const void* Q, const void* K, const void* V, void* O,
                           int B, int H, int N, int d, int dtype, int normalizer, void* stream)
{
    const int rc = check_args(Q, K, V, O, out_bytes_of(B, H, N, d, dtype), nullptr, nullptr, B, H, H, N, N, d, dtype);
    if (rc != SPHATTN_OK) return rc;
    if (normalizer < SPHATTN_NORM_L2 || normalizer > SPHATTN_NORM_SQRELU) return SPHATTN_ERR_NORMALIZER;
    if (normalizer != SPHATTN_NORM_L2 && dtype != SPHATTN_BF16 &&
        !(normalizer == SPHATTN_NORM_SOFTMAX && dtype == SPHATTN_FP8QK_BF16V))
        return SPHATTN_ERR_DTYPE;
    const Problem p{Q, K, V, O, nullptr, nullptr, B, H, H, N, N, (hipStream_t)stream};
    switch (normalizer) {
    case SPHATTN_NORM_L2: return dispatch_spherical<false>(p, d, dtype);
    case SPHATTN_NORM_SOFTMAX: return dispatch_normalizer<Norm::Softmax>(p, d, dtype);
    case SPHATTN_NORM_L1: return dispatch_normalizer<Norm::L1>(p, d, dtype);
    default: return dispatch_normalizer<Norm::SqRelu>(p, d, dtype);
    }
}

int sphattn_softmax_fwd(const void* Q, const void* K, const void* V, void* O,
                        int B, int H, int N, int d, int dtype, void* stream)
{
    const int rc = check_args(Q, K, V, O, out_bytes_of(B, H, N, d, dtype), nullptr, nullptr, B, H, H, N, N, d, dtype);
    if (rc != SPHATTN_OK) return rc;
    if (dtype != SPHATTN_BF16) return SPHATTN_ERR_DTYPE;
    const Problem p{Q, K, V, O, nullptr, nullptr, B, H, H, N, N, (hipStream_t)stream};
    return d == 128 ? launch_softmax32<128>(p) : launch_softmax32<64>(p);
}

int sphattn_partial_fwd(const void* Q, const void* K, const void* V, const float* mult,
                        float* o_part, float* z_part,
                        int B, int H, int H_kv, int N_q, int N_k, int d, int dtype, void* stream)
{
    if (!z_part) return SPHATTN_ERR_NULL;
    const int rc = check_args(Q, K, V, o_part, (size_t)B * H * N_q * d * 4, mult, z_part,
                              B, H, H_kv, N_q, N_k, d, dtype);
    if (rc != SPHATTN_OK) return rc;
    Problem p{Q, K, V, o_part, mult, z_part, B, H, H_kv, N_q, N_k, (hipStream_t)stream};
    p.n_splits = 1;
    p.keys_per_split = plan_splits(N_k, 1).keys_per_split;
    return mult ? dispatch_spherical<true, true>(p, d, dtype) : dispatch_spherical<false, true>(p, d, dtype);
}

int sphattn_combine(const float* o_parts, const float* z_parts, int n_parts, void* O, float* Z,
                    int B, int H, int N, int d, int dtype, void* stream)
{
    if (!o_parts || !z_parts || !O) return SPHATTN_ERR_NULL;
    const int rc = check_shape(B, H, H, N, N, d, dtype);
    if (rc != SPHATTN_OK) return rc;
    if (n_parts <= 0 || n_parts > 65536) return SPHATTN_ERR_SHAPE;
    if (((uintptr_t)o_parts | (uintptr_t)O) & 15) return SPHATTN_ERR_ALIGN;
    if (((uintptr_t)z_parts | (uintptr_t)Z) & 3) return SPHATTN_ERR_ALIGN;
    const size_t rows = (size_t)B * H * N, ob = out_bytes_of(B, H, N, d, dtype);
    const size_t pob = (size_t)n_parts * rows * d * 4, pzb = (size_t)n_parts * rows * 4;
    if (overlaps(O, ob, o_parts, pob) || overlaps(O, ob, z_parts, pzb) ||
        (Z && (overlaps(Z, rows * 4, o_parts, pob) || overlaps(Z, rows * 4, z_parts, pzb) ||
               overlaps(Z, rows * 4, O, ob))))
        return SPHATTN_ERR_ALIAS;
    return d == 128 ? launch_combine<128>(o_parts, z_parts, n_parts, O, Z, rows, dtype, (hipStream_t)stream)
                    : launch_combine<64>(o_parts, z_parts, n_parts, O, Z, rows, dtype, (hipStream_t)stream);
}

size_t sphattn_splitkv_workspace_bytes(int B, int H, int N, int d, int n_splits)
{
    if (B <= 0 || H <= 0 || N <= 0 || (d != 64 && d != 128) || n_splits <= 0) return 0;
    if ((unsigned __int128)B * H * (unsigned __int128)N * (d + 1) * 4 * n_splits > ((unsigned __int128)1 << 46)) return 0;
    return workspace_bytes(B, H, N, d, n_splits);
}

int sphattn_splitkv_heuristic(int B, int H, int N, int d, int dtype)
{
    if (B <= 0 || H <= 0 || N <= 0 || (d != 64 && d != 128)) return 1;
    return choose_splits((long long)B * H, N, N, d, dtype);
}

int sphattn_splitkv_fwd(const void* Q, const void* K, const void* V, const float* mult, void* O, float* Z,
                        int B, int H, int H_kv, int N, int d, int dtype, int n_splits,
                        void* workspace, size_t workspace_size, void* stream)
{
    const int rc = check_args(Q, K, V, O, out_bytes_of(B, H, N, d, dtype), mult, Z, B, H, H_kv, N, N, d, dtype);
    if (rc != SPHATTN_OK) return rc;
    if (n_splits < 0) return SPHATTN_ERR_SHAPE;
    const int requested = n_splits;
    if (n_splits == 0) n_splits = sphattn_splitkv_heuristic(B, H, N, d, dtype);
    const SplitPlan plan = plan_splits(N, n_splits);
    const Problem p{Q, K, V, O, mult, Z, B, H, H_kv, N, N, (hipStream_t)stream};
    const int wrc = check_workspace(p, d, dtype, plan, workspace, workspace_size);
    return wrc != SPHATTN_OK ? wrc : run_splitkv(p, d, dtype, requested, plan, workspace);
}

size_t sphattn_cross_splitkv_workspace_bytes(int B, int H, int H_kv, int N_q, int N_k, int d, int dtype)
{
    if (check_shape(B, H, H_kv, N_q, N_k, d, dtype) != SPHATTN_OK) return 0;
    const SplitPlan plan = plan_cross(B, H, H_kv, N_q, N_k, d, dtype);
    return plan.n_splits == 1 ? 0 : sphattn_splitkv_workspace_bytes(B, H, N_q, d, plan.n_splits);
}

int sphattn_cross_splitkv_fwd(const void* Q, const void* K, const void* V, const float* mult, void* O, float* Z,
                              int B, int H, int H_kv, int N_q, int N_k, int d, int dtype,
                              void* workspace, size_t workspace_size, void* stream)
{
    const int rc = check_args(Q, K, V, O, out_bytes_of(B, H, N_q, d, dtype), mult, Z, B, H, H_kv, N_q, N_k, d, dtype);
    if (rc != SPHATTN_OK) return rc;
    const SplitPlan plan = plan_cross(B, H, H_kv, N_q, N_k, d, dtype);
    const Problem p{Q, K, V, O, mult, Z, B, H, H_kv, N_q, N_k, (hipStream_t)stream};
    if (plan.n_splits > 1) {
        const int wrc = check_workspace(p, d, dtype, plan, workspace, workspace_size);
        if (wrc != SPHATTN_OK) return wrc;
    }
    return run_splitkv(p, d, dtype, 0, plan, workspace);
}

int sphattn_splitkv_fwd_noalloc(const void* Q, const void* K, const void* V, const float* mult, void* O, float* Z,
                                int B, int H, int H_kv, int N, int d, int dtype, int n_splits, void* stream)
{
    const int rc = check_args(Q, K, V, O, out_bytes_of(B, H, N, d, dtype), mult, Z, B, H, H_kv, N, N, d, dtype);
    if (rc != SPHATTN_OK) return rc;
    if (n_splits < 0) return SPHATTN_ERR_SHAPE;
    const int requested = n_splits;
    if (n_splits == 0) {                           // the library's choice, if the array holds it
        n_splits = sphattn_splitkv_heuristic(B, H, N, d, dtype);
        if (sphattn_splitkv_workspace_bytes(B, H, N, d, plan_splits(N, n_splits).n_splits) > (size_t)SPHATTN_NOALLOC_SCRATCH_BYTES)
            n_splits = 1;
    }
    const SplitPlan plan = plan_splits(N, n_splits);
    // one slice is the unsplit launch and needs no scratch
    const Problem p{Q, K, V, O, mult, Z, B, H, H_kv, N, N, (hipStream_t)stream};
    if (plan.n_splits == 1) return run_splitkv(p, d, dtype, requested, plan, nullptr);
    const size_t need = sphattn_splitkv_workspace_bytes(B, H, N, d, plan.n_splits);
    if (need == 0 || need > (size_t)SPHATTN_NOALLOC_SCRATCH_BYTES) return SPHATTN_ERR_SCRATCH;
    void* ws = scratch_address();
    if (ws == nullptr) return SPHATTN_ERR_LAUNCH;
    // the caller's buffers are allocations of their own and cannot overlap the library's array
    return run_splitkv(p, d, dtype, requested, plan, ws);
}

int sphattn_grn_bwd(const void* Q, const void* K, const void* V, const float* mult,
                    const void* O, const void* dO, const float* Z,
                    void* dQ, void* dK, void* dV, float* delta,
                    int B, int H, int H_kv, int N, int d, int dtype, void* stream)
{
    const int rc = check_bwd(Q, K, V, mult, O, dO, Z, dQ, dK, dV, delta, B, H, H_kv, N, d, dtype);
    if (rc != SPHATTN_OK) return rc;
    const BwdProblem p{Q, K, V, mult, O, dO, Z, dQ, dK, dV, delta, B, H, H_kv, N, (hipStream_t)stream};
    return mult ? dispatch_bwd<true>(p, d, dtype, BwdPlan{}, nullptr) : dispatch_bwd<false>(p, d, dtype, BwdPlan{}, nullptr);
}

size_t sphattn_bwd_workspace_bytes(int B, int H, int H_kv, int N, int d, int dtype)
{
    if (check_shape(B, H, H_kv, N, N, d, dtype) != SPHATTN_OK || (dtype != SPHATTN_BF16 && dtype != SPHATTN_F16)) return 0;
    return plan_bwd(B, H, H_kv, N, d).bytes;
}

int sphattn_grn_bwd_split(const void* Q, const void* K, const void* V, const float* mult,
                          const void* O, const void* dO, const float* Z,
                          void* dQ, void* dK, void* dV, float* delta,
                          int B, int H, int H_kv, int N, int d, int dtype,
                          void* workspace, size_t workspace_size, void* stream)
{
    const int rc = check_bwd(Q, K, V, mult, O, dO, Z, dQ, dK, dV, delta, B, H, H_kv, N, d, dtype);
    if (rc != SPHATTN_OK) return rc;
    const BwdPlan plan = plan_bwd(B, H, H_kv, N, d);
    if (plan.bytes) {
        if (!workspace || workspace_size < plan.bytes || ((uintptr_t)workspace & 15) || wraps(workspace, plan.bytes)) return SPHATTN_ERR_WORKSPACE;
        const size_t tq = (size_t)B * H * N * d * 2, tkv = (size_t)B * H_kv * N * d * 2, rb = (size_t)B * H * N * 4;
        const void* others[11] = {Q, K, V, O, dO, Z, mult, dQ, dK, dV, delta};
        const size_t bytes[11] = {tq, tkv, tkv, tq, tq, rb, (size_t)B * N * 4, tq, tkv, tkv, 2 * rb};
        for (int i = 0; i < 11; ++i)
            if (others[i] && overlaps(workspace, plan.bytes, others[i], bytes[i])) return SPHATTN_ERR_ALIAS;
    }
    const BwdProblem p{Q, K, V, mult, O, dO, Z, dQ, dK, dV, delta, B, H, H_kv, N, (hipStream_t)stream};
    return mult ? dispatch_bwd<true>(p, d, dtype, plan, workspace) : dispatch_bwd<false>(p, d, dtype, plan, workspace);
}

int sphattn_bwd(const void* Q, const void* K, const void* V, const void* O, const void* dO, const float* Z,
                void* dQ, void* dK, void* dV, float* delta,
                int B, int H, int N, int d, int dtype, void* stream)
{
    return sphattn_grn_bwd(Q, K, V, nullptr, O, dO, Z, dQ, dK, dV, delta, B, H, H, N, d, dtype, stream);
}

size_t sphattn_fp8_workspace_bytes(int B, int H_kv, int N, int d)
{
    if (B <= 0 || H_kv <= 0 || N <= 0 || (d != 64 && d != 128)) return 0;
    const size_t tiles = ((size_t)N + kFp8Tile - 1) / kFp8Tile;
    return (size_t)B * H_kv * d * tiles * kFp8Tile + (((size_t)B * H_kv * 4 + 255) & ~(size_t)255);
}

int sphattn_fp8_fwd(const void* Q, const void* K, const void* V, void* O, void* workspace,
                    size_t workspace_bytes, int B, int H, int H_kv, int N, int d, void* stream)
{
    return fp8_forward(Q, K, V, nullptr, O, workspace, workspace_bytes, B, H, H_kv, N, d, stream, false);
}

int sphattn_fp8_grn_fwd(const void* Q, const void* K, const void* V, const float* mult, void* O, void* workspace,
                        size_t workspace_bytes, int B, int H, int H_kv, int N, int d, void* stream)
{
    return fp8_forward(Q, K, V, mult, O, workspace, workspace_bytes, B, H, H_kv, N, d, stream, false);
}

int sphattn_fp8_softmax_fwd(const void* Q, const void* K, const void* V, void* O, void* workspace,
                            size_t workspace_bytes, int B, int H, int H_kv, int N, int d, void* stream)
{
    return fp8_forward(Q, K, V, nullptr, O, workspace, workspace_bytes, B, H, H_kv, N, d, stream, true);
}

const char* sphattn_strerror(int code)
{
    switch (code) {
    case SPHATTN_OK: return "success";
    case SPHATTN_ERR_NULL: return "a required pointer is NULL";
    case SPHATTN_ERR_SHAPE: return "B, H, N must be positive, H_kv must divide H, and sizes must not overflow";
    case SPHATTN_ERR_HEAD_DIM: return "head dimension d must be 64 or 128";
    case SPHATTN_ERR_DTYPE: return "unsupported dtype for this entry point";
    case SPHATTN_ERR_ALIGN: return "Q, K, V and O must be 16-byte aligned";
    case SPHATTN_ERR_LAUNCH: return "the HIP runtime refused the kernel launch";
    case SPHATTN_ERR_ALIAS: return "O must not overlap Q, K or V";
    case SPHATTN_ERR_NORMALIZER: return "normalizer is not a sphattn_normalizer value";
    case SPHATTN_ERR_WORKSPACE: return "workspace is NULL, misaligned or smaller than the entry point's *_workspace_bytes";
    case SPHATTN_ERR_SCRATCH: return "the problem needs more scratch than the library's own array holds (SPHATTN_NOALLOC_SCRATCH_BYTES)";
    default: return "unknown sphattn error code";
    }
}

int sphattn_version(void) { return kVersion; }


}  // extern "C"
