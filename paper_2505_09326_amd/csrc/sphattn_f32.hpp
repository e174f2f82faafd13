// Forward for fp32 storage on the bf16 matrix instructions.
//
// The fp32 matrix instruction (v_mfma_f32_32x32x2_f32) runs at 1/16 of the bf16 one's rate.  An fp32
// value is the exact sum of three bf16 values, x = x0 + x1 + x2 (x0 the upper 16 bits, x1 the
// remainder rounded to bf16, x2 what is left: 8 + 8 + 8 significant bits; no x0 overflows, because
// it is cut and not rounded), so
//     x y = x0 y0 + (x0 y1 + x1 y0) + (x1 y1 + x0 y2 + x2 y0) + terms below 2^-23 |x y|,
// six bf16 products, each exact in fp32, summed by the matrix cores in fp32.  The terms left out are
// of the size of one fp32 rounding and of random sign.  Against 64 bits the results are no further off
// than those of the fp32 instruction, and closer at length, for two reasons: a score takes 24 additions at
// full size instead of 64, and o receives a 32-key tile as one sum that was formed from zero (one rounding
// at the size of o per 32 keys instead of 16).  Values below 2^-110 in magnitude lose low bits (bf16
// subnormals), far below what a score's square can hold in fp32.
//
// A workgroup is 8 waves (two per SIMD) x 16 NQ query rows; Q's three parts stay in registers.
// K and V tiles of 32 keys arrive as they are through direct global -> LDS copies (each wave's share in
// a region of its own), are split by the wave that copied them, and go to LDS as three bf16 images in
// the block formats of the other kernels: K as 16 x 64-byte blocks with permuted pieces (row-major
// reads), V as 16 x 32-byte blocks (transposing reads).  Two image buffers, one barrier per tile; the
// waves 0..3 split the next tile before they work on the current one and the waves 4..7 after it, so
// that on every SIMD one wave's vector work falls into the other's matrix work.
#pragma once
#include "sphattn_pipelined.hpp"

namespace sphattn {

constexpr int kF32Waves = 8;
constexpr int kF32Tile = 32;           // keys per tile

template <int D>
constexpr int f32_lds_bytes()
{
    return 2 * 6 * kF32Tile * D * 2 + 2 * kF32Tile * D * 4;   // two sets of six images, one tile as copied
}

// A pair of fp32 values as three packed pairs of bf16 whose sums are the values.
struct Split3 { int p0, p1, p2; };
__device__ __forceinline__ Split3 split3(float a, float b)
{
    const unsigned ua = __builtin_bit_cast(unsigned, a), ub = __builtin_bit_cast(unsigned, b);
    Split3 r;
    r.p0 = (int)__builtin_amdgcn_perm(ub, ua, 0x07060302);
    a -= __builtin_bit_cast(float, ua & 0xffff0000u);
    b -= __builtin_bit_cast(float, ub & 0xffff0000u);
    r.p1 = pack2<false>(a, b);
    a -= __builtin_bit_cast(float, (unsigned)r.p1 << 16);
    b -= __builtin_bit_cast(float, (unsigned)r.p1 & 0xffff0000u);
    r.p2 = pack2<false>(a, b);
    return r;
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
    constexpr int RAW = 2 * SET;
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
    auto copy_tile = [&](int t) {
#pragma unroll
        for (int u = 0; u < UPW; ++u) {
            const int idx = wave * UPW + u, in = idx % (4 * KK);   // row group in / KK, column group in % KK
            copy_to_lds(idx < 4 * KK ? krw : vrw, lds0 + RAW + idx * 1024, ld_lane, (t * BC + in / KK * 8) * D * 4 + in % KK * 128);
        }
    };
    // the same units split into the three images of set `set`
    const int rowin = lane >> 3, c4 = lane & 7;    // row and float4 of the unit
    auto split_unit = [&](int u, int set) {
            const int idx = wave * UPW + u, in = idx % (4 * KK), rg = in / KK, c = in % KK;
            const f32x4 x = __builtin_bit_cast(f32x4, lds_read_b128(smem + RAW + idx * 1024 + lane * 16));
            const Split3 lo = split3(x[0], x[1]), hi = split3(x[2], x[3]);
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
                const Split3 s = e < 2 ? split3(a[2 * e], a[2 * e + 1]) : split3(b[2 * e - 4], b[2 * e - 3]);
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
    const int n_tiles = (N + BC - 1) / BC;
    wait_copies();
#pragma unroll
    for (int u = 0; u < UPW; ++u) split_unit(u, 0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);            // lgkmcnt(0): the copied bytes are read, the images written
    copy_tile(1);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    // which part of the left and of the right operand each of the six products takes, smallest first
    constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
    const int klane = block_piece_offset(n16, g), vlane = 3 * IMG + lane * 8;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    for (int j = 0; j < n_tiles; ++j) {
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
                    for (int qb = 0; qb < NQ; ++qb)
#pragma unroll
                        for (int kb = 0; kb < 2; ++kb) {
                            if constexpr (MULT) s[kb][qb] *= mk[kb];
#pragma unroll
                            for (int c = 0; c < 2; ++c) {
                                const float a = s[kb][qb][2 * c], b = s[kb][qb][2 * c + 1];
                                zacc[qb][0] = __builtin_fmaf(a, a, zacc[qb][0]);
                                zacc[qb][1] = __builtin_fmaf(b, b, zacc[qb][1]);
                                const Split3 x = split3(a, b);
                                pf[qb][0][2 * kb + c] = x.p0;
                                pf[qb][1][2 * kb + c] = x.p1;
                                pf[qb][2][2 * kb + c] = x.p2;
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
