// Forward for fp32 storage on the bf16 matrix instructions.
//
// The fp32 matrix instruction (v_mfma_f32_32x32x2_f32) runs at 1/16 of the bf16 one's rate.  An fp32
// value is the exact sum of three bf16 values, x = x0 + x1 + x2 (each the rest before it, rounded to bf16), so
//     x y = x0 y0 + (x0 y1 + x1 y0) + (x1 y1 + x0 y2 + x2 y0) + (x1 y2 + x2 y1 + x2 y2),
// six bf16 products, each exact in fp32, summed by the matrix cores in fp32.  |x1| <= 2^-8 and |x2| <= 2^-17 of
// x0's power of two, so the three left out come to at most 2^-24 |x y| and measure 5.5e-8 at most and 5.8e-9 in
// the root mean square over random mantissas, where one fp32 rounding of the product has 6.0e-8 and 2.5e-8 (an x0
// that is cut and not rounded doubles x1 and x2: 2.1e-7 and 2.3e-8).  Against 64 bits the results
// are no further off than those of the fp32 instruction, and closer at length, for two reasons: a score takes
// 24 additions at full size instead of 64, and o receives a 32-key tile as one sum that was formed from zero (one
// rounding at the size of o per 32 keys instead of 16).
//
// That holds while no part is lost to bf16's range.  x2 is formed as an fp32 value of at most seven significant
// bits, a multiple of 2^-23 of x's power of two, and is short of bits only below bf16's subnormal step of 2^-133, i.e. only
// where it is itself subnormal (an x1 that is cut there leaves such an x2); from 2^-103 on no x has a subnormal x2.
// So each wave watches whether any x2 that it forms, of Q, K and V elements and of scores, is subnormal (one
// instruction per value), and at the end whether o and z are finite (an x0 that rounds to infinity
// leaves NaN) and no o is below 2^-100.  If any wave of a workgroup saw one, for Q and the first tile before
// the loop, the workgroup does its rows again with the fp32 instruction (f32_exact_rows): V scaled by 1e-36,
// Q by 1e-36 against K by 1e36, infinities, subnormals and the largest fp32 values come out as they do there.
// The watch costs 2 % (8 x 4096 x 128 282.3 us without it, 288.7 with; 16 x 4096 x 64 283.8, 289.1).
// Done again from the first tile on, 8 x 4096 x 128 takes 707 us (702 on fwd_f32_kernel); from the last tile, 953.
//
// A workgroup is 8 waves (two per SIMD) x 16 NQ query rows; Q's three parts stay in registers.
// K and V tiles of 32 keys arrive as they are through direct global -> LDS copies (each wave's share in
// a region of its own), are split by the wave that copied them, a unit at a time between its matrix
// instructions, and go to LDS as three bf16 images in
// the block formats of the other kernels: K as 16 x 64-byte blocks with permuted pieces (row-major
// reads), V as 16 x 32-byte blocks (transposing reads).  Two image buffers, one barrier per tile.
#pragma once
#include "sphattn_pipelined.hpp"

namespace sphattn {

constexpr int kF32Waves = 8;
constexpr int kF32Tile = 32;           // keys per tile

// Two sets of six images, one tile as copied, and a word per wave.
template <int D>
constexpr int f32_flags_at() { return 2 * 6 * kF32Tile * D * 2 + 2 * kF32Tile * D * 4; }
template <int D>
constexpr int f32_lds_bytes() { return f32_flags_at<D>() + kF32Waves * 4; }

// Byte of a head's K or V at which row `row` of tile `tile` starts.  Heads are at most 2^31 - 1 bytes (the entry
// points refuse longer ones), which a tile past the last one may pass: such a tile is not asked for.
template <int D>
constexpr int f32_tile_byte(int tile, int row) { return (tile * kF32Tile + row) * D * 4; }
constexpr int kF32MostKeys128 = 0x7fffffff / (128 * 4), kF32MostKeys64 = 0x7fffffff / (64 * 4);
static_assert(f32_tile_byte<128>((kF32MostKeys128 - 1) / kF32Tile, kF32Tile - 1) > 0 &&
              f32_tile_byte<64>((kF32MostKeys64 - 1) / kF32Tile, kF32Tile - 1) > 0, "offsets of the longest head's last tile fit");

__device__ __forceinline__ uint32_t doubled_bits(float x) { return __builtin_bit_cast(uint32_t, x) << 1; }

// The lanes whose x is subnormal.  (The compiler's form of this goes through a vector register.)
__device__ __forceinline__ uint64_t subnormal_lanes(float x)
{
    uint64_t lanes;
    asm("v_cmp_class_f32 %0, %1, %2" : "=s"(lanes) : "v"(x), "s"(0x90));
    return lanes;
}

// A pair of fp32 values as three packed pairs of bf16 whose sums are the values, except in the lanes added to `outside`.
struct Split3 { int p0, p1, p2; };
__device__ __forceinline__ Split3 split3(float a, float b, uint64_t& outside)
{
    Split3 r;
    r.p0 = pack2<false>(a, b);
    a -= __builtin_bit_cast(float, (unsigned)r.p0 << 16);
    b -= __builtin_bit_cast(float, (unsigned)r.p0 & 0xffff0000u);
    r.p1 = pack2<false>(a, b);
    a -= __builtin_bit_cast(float, (unsigned)r.p1 << 16);
    b -= __builtin_bit_cast(float, (unsigned)r.p1 & 0xffff0000u);
    outside |= subnormal_lanes(a) | subnormal_lanes(b);
    r.p2 = pack2<false>(a, b);
    return r;
}

// One wave's 16 query rows from q0 on against N keys with the fp32 instruction, k-steps as in
// fwd_f32_small_kernel, K and V straight from memory; a tile's sums are formed from zero.  For the values
// that have no three parts, so few registers and no LDS rather than time.  Qh, Oh, Zh (null: not wanted): the
// head's rows; ks, vs, ms: the keys' buffers, zeros past the last.
template <int D, bool MULT, bool PARTIAL>
__device__ __forceinline__
void f32_exact_rows(const float* __restrict__ Qh, __amdgpu_buffer_rsrc_t ks, __amdgpu_buffer_rsrc_t vs, __amdgpu_buffer_rsrc_t ms,
                    float* __restrict__ Oh, float* __restrict__ Zh, int Nq, int N, int q0)
{
    constexpr int DB = D / 16, M = D / 16;
    const int lane = __lane_id(), n16 = lane & 15, g = lane >> 4;   // (not from threadIdx, which would hold a register till here)
    const int row = q0 + n16;
    const float* src = Qh + (size_t)(row < Nq ? row : Nq - 1) * D + 4 * g;
    f32x4 qf[M], oacc[DB];
#pragma unroll
    for (int m = 0; m < M; ++m) {
        qf[m] = *reinterpret_cast<const f32x4*>(src + 16 * m);
        oacc[m] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    float z[2] = {0.f, 0.f};
#pragma unroll 1
    for (uint32_t j0 = 0; j0 < (uint32_t)N; j0 += kF32Tile) {
        f32x4 s[2] = {f32x4{0, 0, 0, 0}, f32x4{0, 0, 0, 0}};
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
            for (int m = 0; m < M; ++m) {
                const f32x4 kf = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(ks, ((j0 + 16 * kb + n16) * D + 16 * m + 4 * g) * 4, 0, 0));
#pragma unroll
                for (int e = 0; e < 4; ++e) s[kb] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[e], qf[m][e], s[kb], 0, 0, 0);
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                if constexpr (MULT) s[kb][t] *= __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(ms, (j0 + 16 * kb + 4 * g + t) * 4, 0, 0));
                z[t & 1] = __builtin_fmaf(s[kb][t], s[kb][t], z[t & 1]);
            }
        }
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const float v = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(vs, ((j0 + 16 * kb + 4 * g + t) * D + db * 16 + n16) * 4, 0, 0));
                    sum = __builtin_amdgcn_mfma_f32_16x16x4f32(v, s[kb][t], sum, 0, 0, 0);
                }
            oacc[db] += sum;
        }
    }
    const float zt = sum_across_groups(z[0] + z[1]);
    const float inv = PARTIAL ? 1.f : zt > 0.f ? 1.0f / __builtin_sqrtf(zt) : 0.f;
    if (row < Nq) {
        if (g == 0 && (PARTIAL || Zh != nullptr)) Zh[row] = zt;
#pragma unroll
        for (int db = 0; db < DB; ++db) *reinterpret_cast<f32x4*>(Oh + (size_t)row * D + db * 16 + 4 * g) = oacc[db] * inv;
    }
}

// Nq, Nk, Zv, PARTIAL, n_splits and keys_per_split as in fwd_pipelined_kernel.
template <int D, int NQ, bool MULT, bool PARTIAL>
__global__ __launch_bounds__(64 * kF32Waves, 2)
void fwd_f32x3_kernel(const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
                      float* __restrict__ O, const float* __restrict__ mult, float* __restrict__ Zv,
                      int Nq, int Nk, int H, int kv_group, int n_qtiles, int n_wg, int n_splits, int keys_per_split)
{
    constexpr int BC = kF32Tile, BR = kF32Waves * 16 * NQ;
    constexpr int KK = D / 32, DB = D / 16;
    constexpr int IMG = BC * D * 2;                // one bf16 image of a K or V tile
    constexpr int SET = 6 * IMG;                   // K0 K1 K2 V0 V1 V2
    constexpr int RAW = 2 * SET, FLAGS = f32_flags_at<D>();
    constexpr int UNITS = 2 * 4 * KK;              // 1 KB units (8 rows x 32 columns of fp32) of K and V
    constexpr int UPW = UNITS / kF32Waves;         // per wave
    static_assert(UNITS % kF32Waves == 0, "units are dealt evenly");

    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    SPH_LDS unsigned char* smem = (SPH_LDS unsigned char*)smem_raw;

    const int tid = threadIdx.x, lane = tid & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n16 = lane & 15, g = lane >> 4;
    const int lid = xcd_contiguous_id(blockIdx.x, n_wg);
    const int qt = lid % n_qtiles;
    const int split = PARTIAL ? (lid / n_qtiles) % n_splits : 0;
    const int bh = PARTIAL ? lid / (n_qtiles * n_splits) : lid / n_qtiles;
    const int bidx = bh / H;
    const int k0 = PARTIAL ? split * keys_per_split : 0;
    const int N = PARTIAL ? min(Nk - k0, keys_per_split) : Nk;
    const size_t kv_off = ((size_t)(bidx * (H / kv_group) + (bh % H) / kv_group) * Nk + k0) * D;
    const int q0 = qt * BR + (int)wave * 16 * NQ;

    // ---- tile copies: unit u of this wave, rows past the last key as zeros
    const i32x4 krw = rsrc_words(K + kv_off, (uint32_t)N * D * 4);
    const i32x4 vrw = rsrc_words(V + kv_off, (uint32_t)N * D * 4);
    const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
    const int ld_lane = (lane >> 3) * D * 4 + (lane & 7) * 16;
    const int n_tiles = (N + BC - 1) / BC;
    auto copy_tile = [&](int t) {                  // past the last tile: that one again, which nothing uses
        const int tile = min(t, n_tiles - 1);
#pragma unroll
        for (int u = 0; u < UPW; ++u) {
            const int idx = wave * UPW + u, in = idx % (4 * KK);   // row group in / KK, column group in % KK
            copy_to_lds(idx < 4 * KK ? krw : vrw, lds0 + RAW + idx * 1024, ld_lane, f32_tile_byte<D>(tile, in / KK * 8) + in % KK * 128);
        }
    };
    uint64_t outside = 0;                          // lanes that met a value out of the parts' range
    // whether any wave of the workgroup says so (a barrier between the two)
    auto say = [&](bool yes) { *reinterpret_cast<SPH_LDS int*>(smem + FLAGS + wave * 4) = __any(yes); };
    auto anyone = [&]() -> bool {
        const i32x4 a = lds_read_b128(smem + FLAGS), b = lds_read_b128(smem + FLAGS + 16);
        return __builtin_amdgcn_readfirstlane(a[0] | a[1] | a[2] | a[3] | b[0] | b[1] | b[2] | b[3]) != 0;
    };
    // the same units split into the three images of set `set`
    const int rowin = lane >> 3, c4 = lane & 7;    // row and float4 of the unit
    auto split_unit = [&](int u, int set) {
            const int idx = wave * UPW + u, in = idx % (4 * KK), rg = in / KK, c = in % KK;
            const f32x4 x = __builtin_bit_cast(f32x4, lds_read_b128(smem + RAW + idx * 1024 + lane * 16));
            const Split3 lo = split3(x[0], x[1], outside), hi = split3(x[2], x[3], outside);
            const int row = (rg & 1) * 8 + rowin;
            const bool is_k = idx < 4 * KK;
            const int koff = ((rg >> 1) * KK + c) * 1024 + block_piece_offset(row, c4 >> 1) + (c4 & 1) * 8;
            const int voff = 3 * IMG + ((rg >> 1) * DB + 2 * c + (c4 >> 2)) * 512 + row * 32 + (c4 & 3) * 8;
            SPH_LDS unsigned char* dst = smem + set * SET + (is_k ? koff : voff);
            *reinterpret_cast<SPH_LDS i32x2*>(dst) = i32x2{lo.p0, hi.p0};
            *reinterpret_cast<SPH_LDS i32x2*>(dst + IMG) = i32x2{lo.p1, hi.p1};
            *reinterpret_cast<SPH_LDS i32x2*>(dst + 2 * IMG) = i32x2{lo.p2, hi.p2};
    };
    auto wait_copies = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0x0F70);        // vmcnt(0)
        asm volatile("" ::: "memory");
    };
    copy_tile(0);

    // ---- Q in three parts as B operands: row n16 of the block, elements 32 kk + 8 g .. + 7
    i32x4 qf[NQ][KK][3];
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb) {
        int row = q0 + qb * 16 + n16;
        row = row < Nq ? row : Nq - 1;             // rows past the end are computed and dropped
        const float* src = Q + ((size_t)bh * Nq + row) * D + 8 * g;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            const f32x4 a = *reinterpret_cast<const f32x4*>(src + 32 * kk), b = *reinterpret_cast<const f32x4*>(src + 32 * kk + 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const f32x4& ab = e < 2 ? a : b;
                const Split3 s = split3(ab[2 * (e & 1)], ab[2 * (e & 1) + 1], outside);
                qf[qb][kk][0][e] = s.p0;
                qf[qb][kk][1][e] = s.p1;
                qf[qb][kk][2][e] = s.p2;
            }
        }
    }
    f32x4 oacc[DB][NQ];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int qb = 0; qb < NQ; ++qb) oacc[db][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
    float zacc[NQ][2];
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb) zacc[qb][0] = zacc[qb][1] = 0.f;

    const __amdgpu_buffer_rsrc_t mrs = make_rsrc(MULT ? mult + (size_t)bidx * Nk + k0 : nullptr, MULT ? (uint32_t)N * 4 : 0);
    wait_copies();
#pragma unroll
    for (int u = 0; u < UPW; ++u) split_unit(u, 0);
    say(outside != 0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);            // lgkmcnt(0): the copied bytes are read, the images written
    copy_tile(1);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    bool in_range = !anyone();

    // which part of the left and of the right operand each of the six products takes, smallest first
    constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
    const int klane = block_piece_offset(n16, g), vlane = 3 * IMG + lane * 8;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    for (int j = 0; in_range && j < n_tiles; ++j) {
        const SPH_LDS unsigned char* set = smem + (j & 1) * SET;
        f32x4 mk[2];
        if constexpr (MULT) {                      // of the lane's keys 16 kb + 4 g + t; past the last key 0
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    mk[kb][t] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(mrs, (j * BC + 16 * kb + 4 * g + t) * 4, 0, 0));
        }
        // Steps of 12 NQ matrix instructions on six fragments, which are read a step ahead: KK score
        // steps (both 16-key blocks of a k-step), then DB / 2 output steps (two 16-column blocks).
        // The next tile is split a unit at a time in between; its copied bytes have had most of a
        // tile's time to land, and their successors are asked for when the last unit is read.
        constexpr int STEPS = KK + DB / 2, EVERY = STEPS / UPW;
        i32x4 fr[2][2][3];
        auto load_step = [&](int st) {
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int p = 0; p < 3; ++p) {
                    if (st < KK) {
                        fr[st & 1][u][p] = lds_read_b128(set + p * IMG + (u * KK + st) * 1024 + klane);
                    } else {
                        const SPH_LDS unsigned char* a = set + vlane + p * IMG + (2 * (st - KK) + u) * 512;
                        const i32x2 lo = lds_read_tr64(a), hi = lds_read_tr64(a + DB * 512);
                        fr[st & 1][u][p] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3);
                    }
                }
        };
        f32x4 s[2][NQ];
        i32x4 pf[NQ][3];
        load_step(0);
        wait_copies();
#pragma unroll
        for (int st = 0; st < STEPS; ++st) {
            if (st + 1 < STEPS) load_step(st + 1);
            if (st % EVERY == 0) split_unit(st / EVERY, (j + 1) & 1);
            if (st < KK) {
                // S^T = K Q^T
#pragma unroll
                for (int m = 0; m < 6; ++m)
#pragma unroll
                    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                        for (int qb = 0; qb < NQ; ++qb)
                            s[kb][qb] = mfma16x16<false>(fr[st & 1][kb][PA[m]], qf[qb][st][PB[m]], st == 0 && m == 0 ? zero : s[kb][qb]);
                if (st == KK - 1) {
                    // z, and the scores in three parts: registers 2 kb, 2 kb + 1 of the B operands
#pragma unroll
                    for (int qb = 0; qb < NQ; ++qb) {
#pragma unroll
                        for (int kb = 0; kb < 2; ++kb) {
                            if constexpr (MULT) s[kb][qb] *= mk[kb];
#pragma unroll
                            for (int c = 0; c < 2; ++c) {
                                const float a = s[kb][qb][2 * c], b = s[kb][qb][2 * c + 1];
                                zacc[qb][0] = __builtin_fmaf(a, a, zacc[qb][0]);
                                zacc[qb][1] = __builtin_fmaf(b, b, zacc[qb][1]);
                                const Split3 x = split3(a, b, outside);
                                pf[qb][0][2 * kb + c] = x.p0;
                                pf[qb][1][2 * kb + c] = x.p1;
                                pf[qb][2][2 * kb + c] = x.p2;
                            }
                        }
                    }
                }
            } else {
                // O^T += V^T P; the tile's sum is formed from zero and added once
                f32x4 t[2][NQ];
#pragma unroll
                for (int m = 0; m < 6; ++m)
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int qb = 0; qb < NQ; ++qb)
                            t[u][qb] = mfma16x16<false>(fr[st & 1][u][PA[m]], pf[qb][PB[m]], m == 0 ? zero : t[u][qb]);
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int qb = 0; qb < NQ; ++qb) oacc[2 * (st - KK) + u][qb] += t[u][qb];
            }
            __builtin_amdgcn_sched_barrier(0);
            if (st == (UPW - 1) * EVERY) {
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_waitcnt(0xC07F);    // lgkmcnt(0): the copied bytes have been read
                copy_tile(j + 2);
            }
        }
        // the other set is whole, this one may be overwritten
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xC07F);        // lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);            // the copies past the end must not outlive the workgroup's LDS

    const size_t rows0 = PARTIAL ? ((size_t)split * (n_wg / (n_qtiles * n_splits)) + bh) * Nq : (size_t)bh * Nq;
    if (in_range) {
        constexpr uint32_t LEAST = (27u << 24) - 1, INFINITE = 0xff000000u;   // doubled bits: of 2^-100, less one; of infinity
        uint32_t least = ~0u, most = 0;            // a zero becomes the largest of all by the subtraction
#pragma unroll
        for (int qb = 0; qb < NQ; ++qb) {
            most = max(most, doubled_bits(zacc[qb][0] + zacc[qb][1]));
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const uint32_t bits = doubled_bits(oacc[db][qb][t]);
                    least = min(least, bits - 1);
                    most = max(most, bits);
                }
        }
        say(outside != 0 || least < LEAST || most >= INFINITE);
        __syncthreads();
        in_range = !anyone();
    }
    if (!in_range) {
        const __amdgpu_buffer_rsrc_t ks = make_rsrc(K + kv_off, (uint32_t)N * D * 4), vs = make_rsrc(V + kv_off, (uint32_t)N * D * 4);
#pragma unroll 1
        for (int qb = 0; qb < NQ; ++qb)
            f32_exact_rows<D, MULT, PARTIAL>(Q + (size_t)bh * Nq * D, ks, vs, mrs, O + rows0 * D,
                                             Zv != nullptr ? Zv + rows0 : nullptr, Nq, N, q0 + qb * 16);
        return;
    }
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb) {
        const float z = sum_across_groups(zacc[qb][0] + zacc[qb][1]);
        const float inv = PARTIAL ? 1.f : z > 0.f ? 1.0f / __builtin_sqrtf(z) : 0.f;
        const int row = q0 + qb * 16 + n16;
        if (row < Nq) {
            if (g == 0 && (PARTIAL || Zv != nullptr)) Zv[rows0 + row] = z;
            float* dst = O + (rows0 + row) * D + 4 * g;
#pragma unroll
            for (int db = 0; db < DB; ++db) *reinterpret_cast<f32x4*>(dst + db * 16) = oacc[db][qb] * inv;
        }
    }
}

}  // namespace sphattn
