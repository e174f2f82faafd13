// Forward kernel for launches that 256-row workgroups cannot spread over the chip: 32 NQ query rows
// per workgroup (128 or 64), the key axis dealt to two pairs of wavefronts.
//
// Same slot pipeline, layouts and matrix instructions as fwd_pipelined_kernel (read that first);
// what differs is who does what.  Wave w owns the 16 NQ query rows of row group w % 2 and, of every
// 64-key tile, the 32 keys of key group w / 2: one sub-step per wave and tile.  At NQ = 4 a wave still
// feeds every K and V^T fragment it reads to four query blocks.  (The other way to 128 rows, four waves
// of 32 rows over all keys, reads every fragment for two blocks only: twice the LDS reads per
// matrix instruction, which then bound it.)  The accumulator of Lemma 1 is a plain sum, so the two
// key groups' partial (o, z) are added once, through LDS, before the tail.
//
// What bounds it, measured while the chip is not full (d = 128, bf16, 2.4 GHz): 128 rows 0.55 us per tile
// = 1310 cycles, 1024 of them matrix instructions; 64 rows 0.42 us = 1000 cycles, 512 of them matrix
// instructions: there the copy of the tile, 32 KB at 33 bytes per cycle and CU, is the bound.
// 1 x 32768 x 64 281 us (four waves of 32 rows) to 217; 4 x 1999 x 128 23.4 to 17.8 (64 rows), fp16 38.6 to 18.0.
//
// Per tile a workgroup copies 32 KB (d = 128, bf16) for half the matrix work of a 256-row one,
// about 28 bytes per cycle and CU, near what direct copies reach (30 to 38); K and V therefore
// have rings of their own, each tile's buffer free again as soon as its one reader iteration is
// over, and copies run three iterations ahead of their use:
//     iteration t reads    K_{t+1} (stage A), V_{t-1} (stage C)
//     iteration t issues   K_{t+5} and V_{t+3}, into the buffers of K_{t+1} and V_{t-1}
// with group G_t = {K_{t+2}, V_t, multiplicities of t+2} needed from slot SLOTS - PD of iteration t on.
// There a wave waits until only the copies of the two younger groups are outstanding, and for its
// own LDS reads of the buffers about to be overwritten, and meets the others at the tile's barrier.
#pragma once
#include "sphattn_pipelined.hpp"

namespace sphattn {

constexpr int kSplitRows = 128;        // query rows per workgroup at NQ = 4; 64 at NQ = 2
constexpr int kSplitMultRing = 8;      // multiplicities outlive their K tile: a longer ring

template <int D, QKType QKT, bool MULT>
constexpr int keysplit_lds_bytes()
{
    return kNBuf * kBC * (D * (QKT == QKType::Fp8 ? 1 : 2) + D * 2) + (MULT ? kSplitMultRing * kBC * 4 : 0);
}

// One work item; arguments as fwd_pipelined_item, and: query tiles are tile_rows apart (the workgroup's rows, or
// twice as many when the item is one half, starting at row_off, of a wider tile).
template <int D, int NQ, QKType QKT, bool MULT, bool PARTIAL>
__device__ __forceinline__
void fwd_keysplit_item(const void* __restrict__ Qv, const void* __restrict__ Kv,
                       const void* __restrict__ Vv, void* __restrict__ Ov,
                       const float* __restrict__ mult, float* __restrict__ Zv,
                       int Nq, int Nk, int H, int kv_group, int n_qtiles, int n_items,
                       int n_splits, int keys_per_split,
                       int item, bool backwards, bool stream_out, int tile_rows, int row_off)
{
    constexpr bool FP8 = QKT == QKType::Fp8;
    constexpr bool HALF = QKT == QKType::F16;
    constexpr int BC = kBC, NBUF = kNBuf;
    constexpr int EQ = FP8 ? 1 : 2;
    constexpr int KROWB = D * EQ, KTILE = BC * KROWB;
    constexpr int VROWB = D * 2, VTILE = BC * VROWB;
    constexpr int DB = D / 16, KBLK = KROWB / 64, KK = D / 32;
    constexpr int VLDS = NBUF * KTILE;             // V ring behind the K ring
    constexpr int MLDS = VLDS + NBUF * VTILE;      // multiplicities behind both
    constexpr int LDK = KBLK, LDV = DB / 2;        // 1 KB copies per wave per K and per V tile
    constexpr int NST = LDK + LDV + (MULT ? 1 : 0);
    constexpr int SLOTS = DB, PD = 3, RING = 4;
    constexpr int QKM = FP8 ? 2 * NQ / SLOTS : NQ; // score matrix instructions per slot
    constexpr int PAIRS = 4 * NQ / SLOTS;          // score register pairs of stage B per slot
    constexpr int VALU_PER_MFMA = (MULT || D == 64) ? 2 : 1;
    static_assert(NQ == 4 || NQ == 2, "128 or 64 query rows per workgroup");
    static_assert(!FP8 || (2 * NQ) % SLOTS == 0, "fp8: whole score instructions per slot");
    static_assert(NBUF == 4 && SLOTS % RING == 0 && PD < RING && PD < SLOTS, "ring indices repeat every iteration");
    static_assert(LDK + LDV <= SLOTS, "one copy per slot (the multiplicities ride with the first)");
    static_assert(FP8 || 2 * KK == SLOTS, "16-bit: one K fragment per slot");
    static_assert(2 * NST < 64, "outstanding copies fit the counter");

    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    SPH_LDS unsigned char* smem = (SPH_LDS unsigned char*)smem_raw;

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int n16 = lane & 15, g = lane >> 4;
    const uint32_t wave_u = __builtin_amdgcn_readfirstlane(wave);
    const int rg = wave_u & 1, kg = wave_u >> 1;   // row group, key group

    const int lid = xcd_contiguous_id(item, n_items);
    const int qt = lid % n_qtiles;
    const int split = PARTIAL ? (lid / n_qtiles) % n_splits : 0;
    const int bh = PARTIAL ? lid / (n_qtiles * n_splits) : lid / n_qtiles;
    const size_t head_off = (size_t)bh * Nq * D;
    const int bidx = bh / H;
    const int k0 = PARTIAL ? split * keys_per_split : 0;
    const int N = PARTIAL ? min(Nk - k0, keys_per_split) : Nk;
    const size_t kv_off = ((size_t)(bidx * (H / kv_group) + (bh % H) / kv_group) * Nk + k0) * D;
    const unsigned char* Qh = (const unsigned char*)Qv + head_off * EQ;
    const int q0 = qt * tile_rows + row_off + rg * 16 * NQ;

    // fragment offsets inside a tile as in fwd_pipelined_item, at this wave's half of the tile
    // (row blocks 2 kg and 2 kg + 1)
    const int klane = kg * 2 * KBLK * 1024 + block_piece_offset(n16, g);
    const int vlane = VLDS + kg * 2 * DB * 512 + lane * 8;
    const int kld_lane = (16 * wave + (lane >> 2)) * KROWB + block_piece_in_slot(lane) * 16;
    const int vld_lane = (16 * wave + ((lane & 31) >> 1)) * VROWB + (lane >> 5) * 32 + (lane & 1) * 16;

    const int n_tiles = (N + BC - 1) / BC;
    auto src_tile = [&](int t) { return t >= n_tiles ? n_tiles : backwards ? n_tiles - 1 - t : t; };
    const i32x4 krw = rsrc_words((const unsigned char*)Kv + kv_off * EQ, (uint32_t)N * KROWB);
    const i32x4 vrw = rsrc_words((const unsigned short*)Vv + kv_off, (uint32_t)N * VROWB);
    const i32x4 mrw = rsrc_words(MULT ? mult + (size_t)bidx * Nk + k0 : nullptr, MULT ? (uint32_t)N * 4 : 0);
    const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
    auto copy_k = [&](int c, int t) {
        copy_to_lds(krw, lds0 + (t & (NBUF - 1)) * KTILE + (wave_u * KBLK + c) * 1024, kld_lane, src_tile(t) * KTILE + c * 64);
    };
    auto copy_v = [&](int c, int t) {
        copy_to_lds(vrw, lds0 + VLDS + (t & (NBUF - 1)) * VTILE + (wave_u * DB + 2 * c) * 512, vld_lane, src_tile(t) * VTILE + c * 64);
    };
    auto copy_m = [&](int t) {                     // the tile's 64 multiplicities, by every wave
        if constexpr (MULT)
            copy_to_lds_b32(mrw, lds0 + MLDS + (t & (kSplitMultRing - 1)) * BC * 4, lane * 4, src_tile(t) * BC * 4);
    };
    // copies number `c` (0 .. SLOTS - 1) of group G_t
    auto copy_group = [&](int c, int t) {
        if (c == 0) copy_m(t + 2);
        if (c < LDK) copy_k(c, t + 2);
        else if (c < LDK + LDV) copy_v(c - LDK, t);
    };

    // ---- prologue.  Q goes through LDS as well: read straight into registers, 16 rows x 64 bytes an
    // instruction with consecutive lanes in different rows, it arrives at 16 bytes per cycle and CU,
    // and both key groups would fetch it (64 KB = 1.8 us at d = 128); as 1 KB block copies, once, it
    // takes a quarter of that.  It waits in the buffers of V_1 and V_2, in K's block format.
    constexpr int QTILE = 32 * NQ * KROWB, QLDS = VLDS + VTILE;
    constexpr int QCOPIES = QTILE / 1024 / kWaves;
    static_assert(QTILE <= 2 * VTILE && QTILE % (1024 * kWaves) == 0, "Q fits the buffers of V_1 and V_2, in whole copies per wave");
    const int tile_row0 = qt * tile_rows + row_off;
    // (byte offsets of one head fit 32 bits; rows past the last query arrive as zeros)
    const i32x4 qrw = rsrc_words(Qh, (uint32_t)Nq * KROWB);
    const int qld_lane = (lane >> 2) * KROWB + block_piece_in_slot(lane) * 16;
    copy_m(0);
#pragma unroll
    for (int c = 0; c < LDK; ++c) copy_k(c, 0);
#pragma unroll
    for (int c = 0; c < QCOPIES; ++c) {            // blocks (row block, 64-byte column) of the workgroup's rows
        const int blk = wave_u * QCOPIES + c;
        copy_to_lds(qrw, lds0 + QLDS + blk * 1024, qld_lane, (tile_row0 + blk / KBLK * 16) * KROWB + blk % KBLK * 64);
    }
    copy_m(1);
#pragma unroll
    for (int c = 0; c < LDK; ++c) copy_k(c, 1);
#pragma unroll
    for (int c = 0; c < SLOTS; ++c) copy_group(c, 0);
    {                                              // V_{-1}, which the first stage C multiplies with P = 0: zeros
        const i32x4 zero4 = {0, 0, 0, 0};
        for (int i = tid; i < VTILE / 16; i += kThreads)
            *reinterpret_cast<SPH_LDS i32x4*>(smem + VLDS + (NBUF - 1) * VTILE + i * 16) = zero4;
    }
    asm volatile("" ::: "memory");
    {                                              // K_0 and Q have landed; K_1 and group 0 may be under way
        constexpr int VM = LDK + (MULT ? 1 : 0) + NST;
        __builtin_amdgcn_s_waitcnt(0x0070 | (VM & 15) | ((VM >> 4) << 14));
    }
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    constexpr int QREGS = FP8 ? 8 : 4;
    constexpr int QSTEPS = FP8 ? 1 : KK;
    typedef __attribute__((ext_vector_type(QREGS))) int qfrag_t;
    qfrag_t qf[NQ][QSTEPS];
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb) {
        const SPH_LDS unsigned char* src = smem + QLDS + (rg * NQ + qb) * KBLK * 1024 + block_piece_offset(n16, g);
#pragma unroll
        for (int kk = 0; kk < QSTEPS; ++kk) {
            if constexpr (FP8) {
                const i32x4 lo = lds_read_b128(src);
                i32x4 hi = {0, 0, 0, 0};
                if constexpr (D == 128) hi = lds_read_b128(src + 1024);
                qf[qb][kk] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            } else {
                qf[qb][kk] = lds_read_b128(src + kk * 1024);
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

    f32x4 mreg[2];
    auto mload = [&](int kb, int t) {
        if constexpr (MULT)
            mreg[kb] = __builtin_bit_cast(f32x4, lds_read_b128(smem + MLDS + (t & (kSplitMultRing - 1)) * BC * 4 + (32 * kg + 16 * kb + 4 * g) * 4));
    };
    mload(0, 0);

    f32x4 S0[2][NQ], S1[2][NQ];
    i32x4 P0[NQ], P1[NQ];
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb) {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) { S0[kb][qb] = f32x4{0, 0, 0, 0}; S1[kb][qb] = f32x4{0, 0, 0, 0}; }
        P0[qb] = i32x4{0, 0, 0, 0};
        P1[qb] = i32x4{0, 0, 0, 0};
    }
    auto mfma_qk = [&](qfrag_t a, qfrag_t b, f32x4 c) -> f32x4 {
        if constexpr (FP8)
            return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c, 0, 0, 0, 0, 0, 0);
        else
            return mfma16x16<HALF>(a, b, c);
    };
    auto k8frag = [&](i32x4 lo, i32x4 hi) -> i32x8 { return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7); };
    auto k8hi = [&](const SPH_LDS unsigned char* a) -> i32x4 {
        if constexpr (D == 128) return lds_read_b128(a + 1024);
        else return i32x4{0, 0, 0, 0};
    };

    // S0 = scores of tile 0
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
        if constexpr (FP8) {
            const SPH_LDS unsigned char* a = smem + klane + kb * KBLK * 1024;
            const qfrag_t kfr = k8frag(lds_read_b128(a), k8hi(a));
#pragma unroll
            for (int qb = 0; qb < NQ; ++qb) S0[kb][qb] = mfma_qk(kfr, qf[qb][0], S0[kb][qb]);
        } else {
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                const qfrag_t kfr = lds_read_b128(smem + klane + (kb * KBLK + kk) * 1024);
#pragma unroll
                for (int qb = 0; qb < NQ; ++qb) S0[kb][qb] = mfma_qk(kfr, qf[qb][kk], S0[kb][qb]);
            }
        }
    }
    // K_1 has landed, everywhere; every wave has read Q, where V_1 and V_2 go, and K_0, where K_4
    // goes.  The rest of group 2 follows in slots 0 .. SLOTS - PD - 1 of iteration 0.
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0070 | (NST & 15) | ((NST >> 4) << 14));   // vmcnt(NST), lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int c = 0; c < SLOTS; ++c) copy_group(c, 1);
#pragma unroll
    for (int c = 0; c < PD; ++c) copy_group(c, 2);

    i32x4 kf[FP8 ? 1 : RING];
    i32x4 kf8[FP8 ? 2 : 1][2][2];                  // fp8: the two fragments of a sub-step; sets alternate by tile
    i32x4 vf[RING];
    // reads for slot u of iteration t, of parity par: u < SLOTS: K_{t+1} and V_{t-1}; u >= SLOTS:
    // slot u - SLOTS of the next iteration
    auto issue_reads = [&](int u, int t, int par) {
        const int i = u % SLOTS;
        const int tt = u < SLOTS ? t : t + 1, set = u < SLOTS ? par : par ^ 1;
        const SPH_LDS unsigned char* kp = smem + ((tt + 1) & (NBUF - 1)) * KTILE + klane;
        const SPH_LDS unsigned char* a = smem + ((tt - 1) & (NBUF - 1)) * VTILE + vlane + i * 512;
        const i32x2 lo = lds_read_tr64(a);
        const i32x2 hi = lds_read_tr64(a + DB * 512);
        vf[i % RING] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3);
        if constexpr (FP8) {
            if (i % (SLOTS / 2) == 0) {
                const int kb = i / (SLOTS / 2);
                kf8[set][kb][0] = lds_read_b128(kp + kb * KBLK * 1024);
                kf8[set][kb][1] = k8hi(kp + kb * KBLK * 1024);
            }
        } else {
            const int kb = i / KK, kk = i % KK;
            kf[i % RING] = lds_read_b128(kp + (kb * KBLK + kk) * 1024);
        }
    };
#pragma unroll
    for (int u = 0; u < PD; ++u) issue_reads(u, 0, 0);

    // tiles in pairs, so that the score and P registers alternate statically; a tile past the end
    // has zero keys and adds nothing
    const int n_run = (n_tiles + 1) & ~1;
    for (int j = 0; j < n_run; j += 2) {
#pragma unroll
        for (int s = 0; s < 2 * SLOTS; ++s) {
            const int par = s / SLOTS, i = s % SLOTS;
            const int t = j + par;
            f32x4 (&Sn)[2][NQ] = par == 0 ? S1 : S0;
            f32x4 (&Sc)[2][NQ] = par == 0 ? S0 : S1;
            i32x4 (&Pc)[NQ] = par == 0 ? P0 : P1;
            i32x4 (&Pp)[NQ] = par == 0 ? P1 : P0;
            __builtin_amdgcn_sched_barrier(0);
            // Group G_t becomes readable.  This wave's reads of K_{t+1} and V_{t-1} (the last of them
            // issued in the slot before) have returned, so past the barrier their buffers may be
            // overwritten.
            if (i == SLOTS - PD) {
                constexpr int VM = 2 * NST;
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_waitcnt(0x0070 | (VM & 15) | ((VM >> 4) << 14));   // vmcnt(VM), lgkmcnt(0)
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            }
            issue_reads(i + PD, t, par);

            // A: next tile's scores
            if constexpr (FP8) {
#pragma unroll
                for (int u = 0; u < QKM; ++u) {
                    const int idx = i * QKM + u, kb = idx / NQ, qb = idx % NQ;
                    const qfrag_t kfr = k8frag(kf8[par][kb][0], kf8[par][kb][1]);
                    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
                    Sn[kb][qb] = mfma_qk(kfr, qf[qb][0], zero);
                }
            } else {
                const int kb = i / KK, kk = i % KK;
#pragma unroll
                for (int qb = 0; qb < NQ; ++qb) {
                    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
                    Sn[kb][qb] = mfma_qk(kf[i % RING], qf[qb][kk], kk == 0 ? zero : Sn[kb][qb]);
                }
            }
            // C: V^T fragment i against the previous tile's P
#pragma unroll
            for (int qb = 0; qb < NQ; ++qb)
                oacc[i][qb] = mfma16x16<HALF>(vf[i % RING], Pp[qb], oacc[i][qb]);
            // B: PAIRS register pairs of the current tile's scores
#pragma unroll
            for (int u = 0; u < PAIRS; ++u) {
                const int p = i * PAIRS + u;
                const int blkid = p / 2, c = p % 2, kb = blkid / NQ, qb = blkid % NQ;
                float a = Sc[kb][qb][2 * c], b = Sc[kb][qb][2 * c + 1];
                if constexpr (MULT) {
                    a *= mreg[kb][2 * c];
                    b *= mreg[kb][2 * c + 1];
                }
                zacc[qb][0] = __builtin_fmaf(a, a, zacc[qb][0]);
                zacc[qb][1] = __builtin_fmaf(b, b, zacc[qb][1]);
                Pc[qb][2 * kb + c] = pack2<HALF>(a, b);
            }
#pragma unroll
            for (int qb = 0; qb < NQ; ++qb) asm volatile("" : "+v"(zacc[qb][0]), "+v"(zacc[qb][1]));
            if (MULT && i == 0) mload(1, t);
            if (MULT && i == SLOTS / 2) mload(0, t + 1);
            // one copy per slot: group t + 3 from this iteration's barrier to the next one's
            if (i >= SLOTS - PD) copy_group(i - (SLOTS - PD), t + 3);
            else copy_group(i + PD, t + 2);
            {
                constexpr int NM = QKM + NQ;
#pragma unroll
                for (int m = 0; m < NM; ++m) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // MFMA
                    if (m < 4) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // DS read
                    __builtin_amdgcn_sched_group_barrier(0x002, VALU_PER_MFMA, 0);   // VALU
                    if (m == NM - 1) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);   // VMEM read (the copy)
                }
            }
        }
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- drain: stage C of the last tile
    {
        const SPH_LDS unsigned char* vp = smem + ((n_run - 1) & (NBUF - 1)) * VTILE + vlane;
#pragma unroll
        for (int i = 0; i < SLOTS; ++i) {
            const i32x2 lo = lds_read_tr64(vp + i * 512);
            const i32x2 hi = lds_read_tr64(vp + i * 512 + DB * 512);
            const i32x4 vfr = __builtin_shufflevector(lo, hi, 0, 1, 2, 3);
#pragma unroll
            for (int qb = 0; qb < NQ; ++qb) oacc[i][qb] = mfma16x16<HALF>(vfr, P1[qb], oacc[i][qb]);
        }
    }

    // ---- add the two key groups: each wave hands half of its query blocks to the other wave of
    // its row group and finishes the other half (blocks HQ kg .. HQ kg + HQ - 1)
    constexpr int HQ = NQ / 2, EXB = HQ * DB * 1024 + HQ * 256;   // bytes one wave receives
    static_assert(kWaves * EXB <= NBUF * (KTILE + VTILE), "the exchange fits the rings");
    __builtin_amdgcn_s_waitcnt(0x0F70);            // the copies past the end must not land in what follows
    __syncthreads();
    SPH_LDS unsigned char* give = smem + (wave ^ 2) * EXB;
    const SPH_LDS unsigned char* take = smem + wave * EXB;
    f32x4 own[DB][HQ];
    float z[HQ];
#pragma unroll
    for (int q = 0; q < HQ; ++q) {
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            own[db][q] = kg ? oacc[db][HQ + q] : oacc[db][q];
            *reinterpret_cast<SPH_LDS f32x4*>(give + (q * DB + db) * 1024 + lane * 16) = kg ? oacc[db][q] : oacc[db][HQ + q];
        }
        const float za = zacc[q][0] + zacc[q][1], zb = zacc[HQ + q][0] + zacc[HQ + q][1];
        z[q] = kg ? zb : za;
        *reinterpret_cast<SPH_LDS float*>(give + HQ * DB * 1024 + q * 256 + lane * 4) = kg ? za : zb;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < HQ; ++q) {
#pragma unroll
        for (int db = 0; db < DB; ++db)
            own[db][q] += *reinterpret_cast<const SPH_LDS f32x4*>(take + (q * DB + db) * 1024 + lane * 16);
        z[q] = sum_across_groups(z[q] + *reinterpret_cast<const SPH_LDS float*>(take + HQ * DB * 1024 + q * 256 + lane * 4));
    }
    const int row0 = q0 + kg * HQ * 16;

    if constexpr (PARTIAL) {
        const size_t rows0 = ((size_t)split * (n_items / (n_qtiles * n_splits)) + bh) * Nq;
        float* Op = (float*)Ov + rows0 * D;
        float* Zp = Zv + rows0;
#pragma unroll
        for (int q = 0; q < HQ; ++q) {
            const int row = row0 + q * 16 + n16;
            if (row < Nq) {
                if (g == 0) Zp[row] = z[q];
                float* dst = Op + (size_t)row * D + 4 * g;
#pragma unroll
                for (int db = 0; db < DB; ++db) *reinterpret_cast<f32x4*>(dst + db * 16) = own[db][q];
            }
        }
        return;
    }

    const __amdgpu_buffer_rsrc_t orw = make_rsrc((unsigned short*)Ov + head_off, (uint32_t)Nq * D * 2);
    constexpr int ROWS = 16 * HQ;
    static_assert(kWaves * ROWS * (D * 2 + 16) <= NBUF * (KTILE + VTILE), "the output stage fits the rings");
    SPH_LDS unsigned char* stage = smem + wave * ROWS * (D * 2 + 16);
    __syncthreads();                               // every wave has taken its half
#pragma unroll
    for (int q = 0; q < HQ; ++q) {
        const float inv = z[q] > 0.f ? 1.0f / __builtin_sqrtf(z[q]) : 0.f;
        const int row = row0 + q * 16 + n16;
        if (Zv != nullptr && g == 0 && row < Nq) Zv[(size_t)bh * Nq + row] = z[q];
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            const i32x2 o4 = {pack2<HALF>(own[db][q][0] * inv, own[db][q][1] * inv),
                              pack2<HALF>(own[db][q][2] * inv, own[db][q][3] * inv)};
            put_piece<D * 2>(stage, q * 16 + n16, db * 32 + 8 * g, o4);
        }
    }
    store_tile<ROWS, D * 2>(stage, orw, row0, Nq, lane, stream_out);
}

// Persistent workgroups over the items, every other batch streaming the keys backwards, and the
// remainder launch of half tiles: as fwd_pipelined_kernel.
template <int D, int NQ, QKType QKT, bool MULT, bool PARTIAL>
__global__ __launch_bounds__(kThreads, D == 64 ? 2 : 1)
void fwd_keysplit_kernel(const void* __restrict__ Qv, const void* __restrict__ Kv,
                         const void* __restrict__ Vv, void* __restrict__ Ov,
                         const float* __restrict__ mult, float* __restrict__ Zv,
                         int Nq, int Nk, int H, int kv_group, int n_qtiles, int n_items,
                         int n_splits, int keys_per_split, int item_begin, int item_end, int halves)
{
    constexpr int BR = 32 * NQ;
    if (halves) {
        // Remainder launch: the items item_begin .. item_end - 1 of a launch whose tiles are
        // 2 BR rows (n_qtiles and n_items count those), one half of an item per workgroup.
        // Workgroups 16u .. 16u+7 take the first halves of items item_begin + 8u .. +7,
        // workgroups 16u+8 .. 16u+15 the second halves: a workgroup stays on the XCD that owns
        // its item's range (item_begin is a multiple of the XCD count).
        const int t = blockIdx.x, half = (t / kXcds) & 1;
        const int item = item_begin + (t / (2 * kXcds)) * kXcds + t % kXcds;
        if (item >= item_end) return;
        const int qt = xcd_contiguous_id(item, n_items) % n_qtiles;
        if (qt * 2 * BR + half * BR >= Nq) return;     // the tile's second half lies past the last row
        fwd_keysplit_item<D, NQ, QKT, MULT, PARTIAL>(Qv, Kv, Vv, Ov, mult, Zv, Nq, Nk, H, kv_group, n_qtiles, n_items,
                                                 n_splits, keys_per_split, item, halves == 2, true, 2 * BR, half * BR);
        return;
    }
    const bool several_batches = item_end - item_begin > (int)gridDim.x || item_end < n_items;
    int batch = 0;
    for (int item = item_begin + blockIdx.x; item < item_end; item += gridDim.x, ++batch) {
        if (batch > 0) __syncthreads();            // every wave is done with the previous item's LDS
        fwd_keysplit_item<D, NQ, QKT, MULT, PARTIAL>(Qv, Kv, Vv, Ov, mult, Zv, Nq, Nk, H, kv_group, n_qtiles, n_items,
                                                 n_splits, keys_per_split, item, batch % 2 == 1, several_batches, BR, 0);
    }
}

}  // namespace sphattn
