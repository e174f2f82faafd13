// Forward kernel for launches that leave CUs without a 256-row workgroup, or with one (d = 64): 16 NQ RG query rows
// per workgroup, the key axis dealt to KG groups of RG wavefronts.
//
// Same slot pipeline, layouts and matrix instructions as fwd_pipelined_kernel (read that first);
// what differs is who does what.  Wave w owns the 16 NQ query rows of row group w % RG and, of every tile of
// 32 KG keys, the 32 keys of key group w / RG: one sub-step per wave and tile.  The accumulator of Lemma 1 is a plain
// sum, so the key groups' partial (o, z) are added once, through LDS, before the tail: two groups by an
// exchange of halves of the query blocks, four by a second exchange (of the remaining blocks, or of halves of the columns).
//
// Forms, and what bounds them (bf16; us per 64-key tile with few CUs busy, one more per share of the CUs: kFormCost):
//   NQ RG KG
//   4  2  2   128 rows, one wave per SIMD: 0.52 (d = 128) for 0.43 of matrix instructions at 2.4 GHz.
//   2  2  2   64 rows: 0.37 (0.25 at d = 64), 0.21 (0.11) of matrix instructions.  The wave, alone on its SIMD, stops for
//             every LDS read, copy and barrier.  Starts fastest (128 keys resident): short key axes.
//   2  2  4   64 rows, two waves per SIMD: 0.28 (0.16).  At d = 128 a tile is 64 KB and the copies (64 bytes per cycle and CU at
//             most) and the fragment reads, both of the LDS, take 0.64 us of the 0.55 to 0.65 of 128 keys.
//             1 x 12000 x 64 55.8 -> 41.1, 4 x 1999 x 128 17.0 -> 15.6 us.
//   2  2  4   with CS = 2 or 4, that part of the columns of V and O per workgroup, where it leaves no more than one on a CU: 0.255 (0.141) with two, the
//             copies 48 KB of a tile's 64, 40 with four (column_shares in sphattn_choice.hpp).  4 x 1999 x 128 15.6 -> 14.3, 8 x 1000 x 128 10.8 -> 9.5 us.
//   4  1  4   64 rows, d = 128: every wave holds all rows, so each byte of K and V is read from LDS once and
//             by the wave that copied it; no barrier in the loop.  0.28, less where many CUs stream (1 x 8192 x 128 53.5 -> 44.4) and
//             with counts (61 -> 54); and the 64-row form of fp8 Q/K, whose score instruction wants four query blocks
//             (0.22 against 0.45 of 128 rows: 5 x 3000 with counts 31.6 -> 21.6).
//   4  2  4   128 rows, two waves per SIMD, d = 64: 0.26 against 0.34 (4 x 8192 58.5 -> 54.5, 6 x 4000 with counts 33.9 -> 28.3).
//   4  4  2   256 rows, two waves per SIMD, d = 64: 0.45 against 0.54 of fwd_pipelined_kernel alone on its CU (3 x 12000
//             115.6 -> 94.7, 8 x 6000 with counts 75 -> 69, 32 x 2048 29.5 -> 28 with the call, 27.4 -> 26.2 of the kernel).
//
// Copies.  K and V have rings of their own, each tile's buffer free again as soon as its one reader iteration is
// over.  With NBUF buffers of K and NVB of V:
//     iteration t reads    K_{t+1} (stage A), V_{t-1} (stage C)
//     iteration t issues   K_{t+NBUF+1} and V_{t+NVB-1}, into the buffers of K_{t+1} and V_{t-1}
// and K_{t+2}, V_t (and the multiplicities of t+2) are needed from slot SLOTS - PD of iteration t on.
// There a wave waits until only copies of younger tiles are outstanding, and for its
// own LDS reads of the buffers about to be overwritten, and meets the others at the tile's barrier.  Four
// buffers, but of 64 KB tiles (four key groups, d = 128) two of K and three of V, all 160 KB of a CU: V's copies
// then have two iterations to land, and K's, issued first, most of one (two of each, as there is room for with counts, 1 x 8192 x 128
// 58.7 us, with the third 47.7).
// V's blocks: where an iteration is bound by the copies (d = 128 beyond the 2 2 2 and 4 2 2 forms) blocks of 16 rows x
// 64 bytes like K's, whose copies take 16 cycles of the copy path; elsewhere 16 x 32 bytes, whose copies
// take 32 (a lane quad then fetches two separate 32-byte pieces) but whose reads need one address
// register instead of two: d = 128 60.1 against 62.2 us (2 x 8192, four key groups), d = 64 9.8 against 9.7 (3 x 2000).
#pragma once
#include "sphattn_pipelined.hpp"

namespace sphattn {

constexpr int kSplitRows = 128;        // query rows of the widest form that calls are cut for

// Waves, keys per tile and tile buffers of a launch with RG row groups and KG key groups.
template <int RG, int KG> constexpr int keysplit_waves() { return RG * KG; }
template <int KG> constexpr int keysplit_keys() { return 32 * KG; }
template <int D, int KG> constexpr int keysplit_buffers() { return KG == 4 && D == 128 ? 2 : kNBuf; }
template <int D, int KG, bool MULT> constexpr int keysplit_v_buffers() { return keysplit_buffers<D, KG>() == 2 && !MULT ? 3 : keysplit_buffers<D, KG>(); }

// LDS: the rings of K, V (DV columns of it) and the multiplicities; Q behind them where it does not fit V's ring.
template <int D, int NQ, int RG, int KG, QKType QKT, bool MULT, int DV = D>
constexpr int keysplit_ring_bytes()
{
    return keysplit_keys<KG>() * (keysplit_buffers<D, KG>() * D * (QKT == QKType::Fp8 ? 1 : 2) + keysplit_v_buffers<D, KG, MULT>() * DV * 2) +
           (MULT ? 2 * keysplit_buffers<D, KG>() * (RG == 1 ? KG * 64 : keysplit_keys<KG>()) * 4 : 0);
}
template <int D, int NQ, int RG, int KG, QKType QKT, int DV = D>
constexpr bool keysplit_q_behind()
{
    return 16 * NQ * RG * D * (QKT == QKType::Fp8 ? 1 : 2) > (keysplit_buffers<D, KG>() == 2 ? 1 : 2) * keysplit_keys<KG>() * DV * 2;
}
// What a wave receives when the key groups are added up, and the output stage.
template <int DV, int NQ> constexpr int keysplit_exchange_bytes() { return NQ / 2 * (DV / 16 * 1024 + 256); }
template <int DV, int NQ, int RG> constexpr int keysplit_stage_bytes() { return 16 * NQ * RG * (DV * 2 + 16); }
template <int D, int NQ, int RG, int KG, QKType QKT, bool MULT, int DV = D>
constexpr int keysplit_lds_bytes()
{
    constexpr int loop = keysplit_ring_bytes<D, NQ, RG, KG, QKT, MULT, DV>() +
                         (keysplit_q_behind<D, NQ, RG, KG, QKT, DV>() ? 16 * NQ * RG * D * (QKT == QKType::Fp8 ? 1 : 2) : 0);
    constexpr int exchange = keysplit_waves<RG, KG>() * keysplit_exchange_bytes<DV, NQ>(), stage = keysplit_stage_bytes<DV, NQ, RG>();
    return loop > exchange ? (loop > stage ? loop : stage) : (exchange > stage ? exchange : stage);
}

// One work item; arguments as fwd_pipelined_item, and: query tiles are tile_rows apart (the workgroup's rows, or
// twice as many when the item is one half, starting at row_off, of a wider tile).  CS > 1: an item is a share of V's and O's columns
// (items go through the shares).
template <int D, int NQ, QKType QKT, bool MULT, bool PARTIAL, int CS, int RG, int KG>
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
    constexpr int WAVES = keysplit_waves<RG, KG>(), THREADS = 64 * WAVES;
    constexpr int BC = keysplit_keys<KG>(), NBUF = keysplit_buffers<D, KG>();
    constexpr bool V32 = D == 64 || (RG == 2 && KG == 2);
    constexpr int NVB = keysplit_v_buffers<D, KG, MULT>();
    constexpr int MRING = 2 * NBUF;                // multiplicities outlive their K tile: a longer ring
    constexpr int EQ = FP8 ? 1 : 2;
    constexpr int KROWB = D * EQ, KTILE = BC * KROWB;
    constexpr int DV = D / CS;                     // columns of V and O of an item
    constexpr int VROWB = D * 2, VTILE = BC * DV * 2;   // row of V in HBM, its tile in LDS
    constexpr int DB = DV / 16, KBLK = KROWB / 64, VBLK = DV * 2 / 64, KK = D / 32;
    constexpr int VLDS = NBUF * KTILE;             // V ring behind the K ring
    constexpr int MLDS = VLDS + NVB * VTILE;       // multiplicities behind both
    constexpr int LDK = (BC / 16 * KBLK + WAVES - 1) / WAVES, LDV = BC / 16 * VBLK / WAVES;   // 1 KB copies per wave per K and per V tile
    constexpr int NST = LDK + LDV + (MULT ? 1 : 0);
    constexpr int SLOTS = D / 16, PD = 3, RING = 4;
    constexpr int VSTEP = SLOTS / DB;              // slots per V^T fragment
    constexpr int QKM = FP8 ? 2 * NQ / SLOTS : NQ; // score matrix instructions per slot
    constexpr int PAIRS = 4 * NQ / SLOTS;          // score register pairs of stage B per slot
    constexpr int VALU_PER_MFMA = (MULT || D == 64 || CS > 1) ? 2 : 1;
    static_assert(NQ == 4 || NQ == 2, "64 or 32 query rows per wave");
    static_assert(CS == 1 || ((CS == 2 || (CS == 4 && D == 128)) && !FP8 && RG == 2 && KG == 4 && NQ == 2), "shares of the columns: the form that has them");
    static_assert(KG == 2 || KG == 4, "two or four key groups");
    constexpr int KSHARES = BC / 16 * KBLK / LDK;  // (fewer than waves: the same blocks twice)
    static_assert(KSHARES * LDK * 16 == BC * KBLK && WAVES % KSHARES == 0 && LDV * WAVES * 16 == BC * VBLK && (LDK % KBLK == 0 || KBLK % LDK == 0) && (LDV % VBLK == 0 || VBLK % LDV == 0),
                  "blocks are dealt evenly, whole row blocks or shares of one");
    // one row group: every wave reads the keys it copied itself, and no other wave does
    constexpr bool OWN = RG == 1;
    static_assert(!OWN || (LDK == 2 * KBLK && LDV == 2 * VBLK), "a wave's two row blocks");
    static_assert(!FP8 || (2 * NQ) % SLOTS == 0, "fp8: whole score instructions per slot");
    static_assert((NBUF == 4 || NBUF == 2) && (NVB == NBUF || (NBUF == 2 && NVB == 3)) && SLOTS % RING == 0 && PD < RING && PD < SLOTS, "ring indices repeat every iteration");
    // copies per slot: with two buffers in the first half of the slots, so that they have the second half to land
    constexpr int CPSK = (NBUF == 2 ? 2 : 1) * (OWN ? 2 : 1), CPSV = (NVB == 2 ? 2 : 1) * (OWN ? 2 : 1), KSLOTS = (LDK + CPSK - 1) / CPSK, CPS = CPSK;
    static_assert(KSLOTS + (LDV + CPSV - 1) / CPSV <= SLOTS, "the multiplicities ride with the first copy");
    static_assert(FP8 || 2 * KK == SLOTS, "16-bit: one K fragment per slot");
    static_assert(NBUF * NST < 64, "outstanding copies fit the counter");

    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    SPH_LDS unsigned char* smem = (SPH_LDS unsigned char*)smem_raw;

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int n16 = lane & 15, g = lane >> 4;
    const uint32_t wave_u = __builtin_amdgcn_readfirstlane(wave);
    const int rg = wave_u % RG, kg = wave_u / RG;  // row group, key group

    const int id = xcd_contiguous_id(item, n_items), lid = id / CS, cs = id % CS;
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
    const int vbase = VLDS + kg * 2 * DB * 512;
    const int vlane[2] = {vbase + (V32 ? lane * 8 : block_tr_offset(lane, 0)), vbase + (V32 ? 0 : block_tr_offset(lane, 1))};
    auto vfrag = [&](int i) { return V32 ? vlane[0] + i * 512 : vlane[i & 1] + (i >> 1) * 1024; };   // V^T fragment i of the wave's keys
    const int kshare = wave % KSHARES;
    const int kld_lane = (kshare * LDK / KBLK * 16 + (lane >> 2)) * KROWB + kshare * LDK % KBLK * 64 + block_piece_in_slot(lane) * 16;
    const int vld_lane = cs * DV * 2 + wave * LDV / VBLK * 16 * VROWB + wave * LDV % VBLK * 64 +
                         (V32 ? ((lane & 31) >> 1) * VROWB + (lane >> 5) * 32 + (lane & 1) * 16 : (lane >> 2) * VROWB + block_piece_in_slot(lane) * 16);

    const int n_tiles = (N + BC - 1) / BC;
    auto src_tile = [&](int t) { return t >= n_tiles ? n_tiles : backwards ? n_tiles - 1 - t : t; };
    const i32x4 krw = rsrc_words((const unsigned char*)Kv + kv_off * EQ, (uint32_t)N * KROWB);
    const i32x4 vrw = rsrc_words((const unsigned short*)Vv + kv_off, (uint32_t)N * VROWB);
    const i32x4 mrw = rsrc_words(MULT ? mult + (size_t)bidx * Nk + k0 : nullptr, MULT ? (uint32_t)N * 4 : 0);
    const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
    auto copy_k = [&](int c, int t) {
        copy_to_lds(krw, lds0 + (t & (NBUF - 1)) * KTILE + (wave_u % KSHARES * LDK + c) * 1024, kld_lane, src_tile(t) * KTILE + c / KBLK * 16 * KROWB + c % KBLK * 64);
    };
    // V tile t + r, seen from iteration t, r = -1 .. 2: a ring of three rotates, others go by the tile's number
    uint32_t rot[3] = {2 * VTILE, 0, VTILE};
    auto v_buffer = [&](int t, int r) -> uint32_t { return NVB == 3 ? rot[(r + 1) % 3] : (uint32_t)((t + r) & (NBUF - 1)) * VTILE; };
    auto copy_v = [&](int c, int t, uint32_t buffer) {
        copy_to_lds(vrw, lds0 + VLDS + buffer + (wave_u * LDV + c) * 1024, vld_lane, src_tile(t) * (BC * VROWB) + c / VBLK * 16 * VROWB + c % VBLK * 64);
    };
    constexpr int MSLOT = OWN ? WAVES * 256 : BC * 4;
    auto copy_m = [&](int t) {                     // 64 of the tile's multiplicities, by every other or by every wave
        if constexpr (MULT) {
            const int off = BC == 64 ? 0 : (OWN ? kg >> 1 : wave_u & 1) * 256;
            copy_to_lds_b32(mrw, lds0 + MLDS + (t & (MRING - 1)) * MSLOT + (OWN ? (int)wave_u * 256 : off), lane * 4, src_tile(t) * BC * 4 + off);
        }
    };
    // copies that go with slot `i` (0 .. SLOTS - 1 from iteration t's barrier on): K_{t+NBUF+1} and V_{t+NVB-1}, into the
    // buffers of K_{t+1} and V_{t-1}.  v: V's buffer
    auto copy_group = [&](int i, int t, uint32_t v) {
        if (i == 0) copy_m(t + NBUF + 1);
#pragma unroll
        for (int c = 0; c < LDK; ++c)
            if (c / CPSK == i) copy_k(c, t + NBUF + 1);
#pragma unroll
        for (int c = 0; c < LDV; ++c)
            if (KSLOTS + c / CPSV == i) copy_v(c, t + NVB - 1, v);
    };

    // ---- prologue.  Q goes through LDS as well: read straight into registers, 16 rows x 64 bytes an
    // instruction with consecutive lanes in different rows, it arrives at 16 bytes per cycle and CU,
    // and both key groups would fetch it (64 KB = 1.8 us at d = 128); as 1 KB block copies, once, it
    // takes a quarter of that.  It waits in the buffers of V_1 and V_2 (V_0 where there are two), or behind the rings, in
    // K's block format.
    constexpr bool QBEHIND = keysplit_q_behind<D, NQ, RG, KG, QKT, DV>();
    constexpr int QTILE = 16 * NQ * RG * KROWB;
    constexpr int QLDS = QBEHIND ? keysplit_ring_bytes<D, NQ, RG, KG, QKT, MULT, DV>() : NVB == 2 ? VLDS : VLDS + VTILE;
    constexpr int QBLOCKS = QTILE / 1024, QCOPIES = (QBLOCKS + WAVES - 1) / WAVES;
    static_assert(QBLOCKS % WAVES == 0 || WAVES % QBLOCKS == 0, "every wave copies as many blocks (where there are few, the same ones)");
    const int tile_row0 = qt * tile_rows + row_off;
    // (byte offsets of one head fit 32 bits; rows past the last query arrive as zeros)
    const i32x4 qrw = rsrc_words(Qh, (uint32_t)Nq * KROWB);
    const int qld_lane = (lane >> 2) * KROWB + block_piece_in_slot(lane) * 16;
    constexpr int YOUNGER = NBUF > 2 ? NST : NVB == 3 ? LDV : 0;   // copies of V_0 (and K_2) under way meanwhile
    copy_m(0);
#pragma unroll
    for (int c = 0; c < LDK; ++c) copy_k(c, 0);
#pragma unroll
    for (int c = 0; c < QCOPIES; ++c) {            // blocks (row block, 64-byte column) of the workgroup's rows
        const int blk = (wave_u * QCOPIES + c) % QBLOCKS;
        copy_to_lds(qrw, lds0 + QLDS + blk * 1024, qld_lane, (tile_row0 + blk / KBLK * 16) * KROWB + blk % KBLK * 64);
    }
    copy_m(1);
#pragma unroll
    for (int c = 0; c < LDK; ++c) copy_k(c, 1);
    if constexpr (NBUF > 2) {
#pragma unroll
        for (int i = 0; i < SLOTS; ++i) copy_group(i, 1 - NBUF, v_buffer(0, 0));
    } else if constexpr (NVB == 3) {
#pragma unroll
        for (int c = 0; c < LDV; ++c) copy_v(c, 0, v_buffer(0, 0));
    }
    {                                              // V_{-1}, which the first stage C multiplies with P = 0: zeros
        const i32x4 zero4 = {0, 0, 0, 0};
        for (int i = tid; i < VTILE / 16; i += THREADS)
            *reinterpret_cast<SPH_LDS i32x4*>(smem + VLDS + (NVB - 1) * VTILE + i * 16) = zero4;
    }
    asm volatile("" ::: "memory");
    {                                              // K_0 and Q have landed; K_1 and group 0 may be under way
        constexpr int VM = LDK + (MULT ? 1 : 0) + YOUNGER;
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
            mreg[kb] = __builtin_bit_cast(f32x4, lds_read_b128(smem + MLDS + (t & (MRING - 1)) * MSLOT + (OWN ? (int)wave_u * 256 + (kg & 1) * 128 : kg * 128) + (16 * kb + 4 * g) * 4));
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
    // K_1 has landed, everywhere; every wave has read Q, where V_0, or V_1 and V_2, go (QLDS), and K_0, where K_NBUF
    // goes.  The copies that follow here are those of iterations 1 - NBUF .. -1 that the prologue has not issued, the last of them in
    // part: the rest goes with slots 0 .. SLOTS - PD - 1 of iteration 0.
    asm volatile("" ::: "memory");
    {
        constexpr int VM = YOUNGER;
        __builtin_amdgcn_s_waitcnt(0x0070 | (VM & 15) | ((VM >> 4) << 14));   // vmcnt(VM), lgkmcnt(0)
    }
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if constexpr (NBUF > 2) {
#pragma unroll
        for (int i = 0; i < SLOTS; ++i) copy_group(i, 2 - NBUF, v_buffer(0, 1));
    }
#pragma unroll
    for (int i = 0; i < PD; ++i) copy_group(i, -1, v_buffer(0, NVB - 2));

    i32x4 kf[FP8 ? 1 : RING];
    i32x4 kf8[FP8 ? 2 : 1][2][2];                  // fp8: the two fragments of a sub-step; sets alternate by tile
    i32x4 vf[RING];
    // reads for slot u of iteration t, of parity par: u < SLOTS: K_{t+1} and V_{t-1}; u >= SLOTS:
    // slot u - SLOTS of the next iteration
    auto issue_reads = [&](int u, int t, int par) {
        const int i = u % SLOTS;
        const int tt = u < SLOTS ? t : t + 1, set = u < SLOTS ? par : par ^ 1;
        const SPH_LDS unsigned char* kp = smem + ((tt + 1) & (NBUF - 1)) * KTILE + klane;
        // (named by the tile read where that schedules the loop better: two key groups with counts 4 to 5 % on short key axes; not with four,
        // 1 x 12000 x 64 39.2 us for 38.2, nor in 256 rows with counts, 1 %)
        constexpr bool BY_TILE = KG == 2 && (RG == 2 || !MULT);
        if (VSTEP == 1 || i % VSTEP == 0) {
            const SPH_LDS unsigned char* a = smem + (BY_TILE ? v_buffer(tt, -1) : v_buffer(t, u < SLOTS ? -1 : 0)) + vfrag(i / VSTEP);
            const i32x2 lo = lds_read_tr64(a);
            const i32x2 hi = lds_read_tr64(a + DB * 512);
            vf[i % RING] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3);
        }
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
    // (one slot's after the other's, as in the loop: a wait at its top for the first slot's would else be for all.  With counts
    // the compiler's own order is the better one, but for the register moves that it costs at 128 rows of d = 128)
#pragma unroll
    for (int u = 0; u < PD; ++u) {
        issue_reads(u, 0, 0);
        if constexpr (!MULT || (D == 128 && NQ == 4)) __builtin_amdgcn_sched_barrier(0);
    }

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
                constexpr int VM = NVB == 3 ? LDV : (NBUF - 2) * NST;
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_waitcnt(0x0070 | (VM & 15) | ((VM >> 4) << 14));   // vmcnt(VM), lgkmcnt(0)
                if constexpr (!OWN) __builtin_amdgcn_s_barrier();
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
            // C: V^T fragment i (one in VSTEP slots) against the previous tile's P
            if (VSTEP == 1 || i % VSTEP == 0) {
#pragma unroll
                for (int qb = 0; qb < NQ; ++qb)
                    oacc[i / VSTEP][qb] = mfma16x16<HALF>(vf[i % RING], Pp[qb], oacc[i / VSTEP][qb]);
            }
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
            if (i >= SLOTS - PD) copy_group(i - (SLOTS - PD), t, v_buffer(t, NVB - 1));
            else copy_group(i + PD, t - 1, v_buffer(t, NVB - 2));
            {
                const int NM = QKM + (i % VSTEP == 0 ? NQ : 0);
#pragma unroll
                for (int m = 0; m < NM; ++m) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // MFMA
                    if (m < 4) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // DS read
                    __builtin_amdgcn_sched_group_barrier(0x002, VALU_PER_MFMA, 0);   // VALU
                    if (m >= NM - CPS) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);   // VMEM read (the copy)
                }
            }
            if (NVB == 3 && i == SLOTS - 1) {      // iteration t + 1's view
                const uint32_t first = rot[0];
                rot[0] = rot[1];
                rot[1] = rot[2];
                rot[2] = first;
            }
        }
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- drain: stage C of the last tile
    {
        const SPH_LDS unsigned char* vp = smem + v_buffer(n_run, -1);
#pragma unroll
        for (int i = 0; i < DB; ++i) {
            const i32x2 lo = lds_read_tr64(vp + vfrag(i));
            const i32x2 hi = lds_read_tr64(vp + vfrag(i) + DB * 512);
            const i32x4 vfr = __builtin_shufflevector(lo, hi, 0, 1, 2, 3);
#pragma unroll
            for (int qb = 0; qb < NQ; ++qb) oacc[i][qb] = mfma16x16<HALF>(vfr, P1[qb], oacc[i][qb]);
        }
    }

    // ---- add the key groups.  First the two of a pair (kg, kg ^ 1): each wave hands half of its query blocks to the other
    // and adds up the other half; with four groups then the two pairs, halving the query blocks once more or, where one
    // is left, its columns.
    constexpr int HQ = NQ / 2;
    constexpr bool FOUR = KG == 4, DSPLIT = FOUR && HQ == 1;
    constexpr int EXB = keysplit_exchange_bytes<DV, NQ>();
    __builtin_amdgcn_s_waitcnt(0x0F70);            // the copies past the end must not land in what follows
    __syncthreads();
    const bool odd = kg & 1, high = FOUR && kg >= 2;
    f32x4 own[DB][HQ];
    float z[HQ];
    {
        SPH_LDS unsigned char* give = smem + (((kg ^ 1) * RG) + rg) * EXB;
        const SPH_LDS unsigned char* take = smem + wave * EXB;
#pragma unroll
        for (int q = 0; q < HQ; ++q) {
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                own[db][q] = odd ? oacc[db][HQ + q] : oacc[db][q];
                *reinterpret_cast<SPH_LDS f32x4*>(give + (q * DB + db) * 1024 + lane * 16) = odd ? oacc[db][q] : oacc[db][HQ + q];
            }
            const float za = zacc[q][0] + zacc[q][1], zb = zacc[HQ + q][0] + zacc[HQ + q][1];
            z[q] = odd ? zb : za;
            *reinterpret_cast<SPH_LDS float*>(give + HQ * DB * 1024 + q * 256 + lane * 4) = odd ? za : zb;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < HQ; ++q) {
#pragma unroll
            for (int db = 0; db < DB; ++db)
                own[db][q] += *reinterpret_cast<const SPH_LDS f32x4*>(take + (q * DB + db) * 1024 + lane * 16);
            z[q] += *reinterpret_cast<const SPH_LDS float*>(take + HQ * DB * 1024 + q * 256 + lane * 4);
        }
    }
    constexpr int FQ = FOUR && !DSPLIT ? HQ / 2 : HQ, FD = DSPLIT ? DB / 2 : DB;   // blocks this wave finishes
    f32x4 fin[FD][FQ];
    float zf[FQ];
    if constexpr (FOUR) {
        constexpr int EX2 = FQ * FD * 1024 + FQ * 256;
        SPH_LDS unsigned char* give = smem + (((kg ^ 2) * RG) + rg) * EX2;
        const SPH_LDS unsigned char* take = smem + wave * EX2;
        __syncthreads();                           // every wave has taken its half
#pragma unroll
        for (int q = 0; q < FQ; ++q) {
#pragma unroll
            for (int db = 0; db < FD; ++db) {
                const f32x4 lo = own[db][q], hi = own[DSPLIT ? FD + db : db][DSPLIT ? q : FQ + q];
                fin[db][q] = high ? hi : lo;
                *reinterpret_cast<SPH_LDS f32x4*>(give + (q * FD + db) * 1024 + lane * 16) = high ? lo : hi;
            }
            const float lo = z[q], hi = z[DSPLIT ? q : FQ + q];
            zf[q] = high ? hi : lo;
            *reinterpret_cast<SPH_LDS float*>(give + FQ * FD * 1024 + q * 256 + lane * 4) = high ? lo : hi;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < FQ; ++q) {
#pragma unroll
            for (int db = 0; db < FD; ++db)
                fin[db][q] += *reinterpret_cast<const SPH_LDS f32x4*>(take + (q * FD + db) * 1024 + lane * 16);
            zf[q] += *reinterpret_cast<const SPH_LDS float*>(take + FQ * FD * 1024 + q * 256 + lane * 4);
        }
    } else {
#pragma unroll
        for (int q = 0; q < FQ; ++q) {
#pragma unroll
            for (int db = 0; db < FD; ++db) fin[db][q] = own[db][q];
            zf[q] = z[q];
        }
    }
#pragma unroll
    for (int q = 0; q < FQ; ++q) zf[q] = sum_across_groups(zf[q]);
    // the wave's rows of the workgroup's, and its first column block
    const int wrow = rg * 16 * NQ + ((odd ? HQ : 0) + (high && !DSPLIT ? FQ : 0)) * 16, db0 = high && DSPLIT ? FD : 0;
    const int row0 = tile_row0 + wrow;

    if constexpr (PARTIAL) {
        const size_t rows0 = ((size_t)split * (n_items / (CS * n_qtiles * n_splits)) + bh) * Nq;
        float* Op = (float*)Ov + rows0 * D;
        float* Zp = Zv + rows0;
#pragma unroll
        for (int q = 0; q < FQ; ++q) {
            const int row = row0 + q * 16 + n16;
            if (row < Nq) {
                if (g == 0 && db0 == 0 && cs == 0) Zp[row] = zf[q];
                float* dst = Op + (size_t)row * D + cs * DV + db0 * 16 + 4 * g;
#pragma unroll
                for (int db = 0; db < FD; ++db) *reinterpret_cast<f32x4*>(dst + db * 16) = fin[db][q];
            }
        }
        return;
    }

    // the rows go through LDS, so that every store instruction writes whole rows: the wave's own, with four key groups (a wave may
    // have parts of rows) the workgroup's
    const __amdgpu_buffer_rsrc_t orw = make_rsrc((unsigned short*)Ov + head_off, (uint32_t)Nq * D * 2);
    constexpr int ROWS = 16 * NQ * RG, WROWS = ROWS / WAVES;
    static_assert(FOUR || WROWS == 16 * FQ, "a wave's rows");
    __syncthreads();                               // every wave has taken its share
#pragma unroll
    for (int q = 0; q < FQ; ++q) {
        const float inv = zf[q] > 0.f ? 1.0f / __builtin_sqrtf(zf[q]) : 0.f;
        const int row = row0 + q * 16 + n16;
        if (Zv != nullptr && g == 0 && db0 == 0 && cs == 0 && row < Nq) Zv[(size_t)bh * Nq + row] = zf[q];
#pragma unroll
        for (int db = 0; db < FD; ++db) {
            const i32x2 o4 = {pack2<HALF>(fin[db][q][0] * inv, fin[db][q][1] * inv),
                              pack2<HALF>(fin[db][q][2] * inv, fin[db][q][3] * inv)};
            put_piece<DV * 2>(smem, wrow + q * 16 + n16, (db0 + db) * 32 + 8 * g, o4);
        }
    }
    if constexpr (FOUR) {
        __syncthreads();
        store_tile<WROWS, DV * 2, D * 2>(smem + wave_u * WROWS * (DV * 2 + 16), orw, tile_row0 + (int)wave_u * WROWS, Nq, lane, stream_out, cs * DV * 2);
    } else {                                       // (whole rows, the wave's own)
        store_tile<WROWS, DV * 2, D * 2>(smem + wrow * (DV * 2 + 16), orw, row0, Nq, lane, stream_out, cs * DV * 2);
    }
}

// Persistent workgroups over the items, every other batch streaming the keys backwards, and the
// remainder launch of half tiles: as fwd_pipelined_kernel.
template <int D, int NQ, QKType QKT, bool MULT, bool PARTIAL, int CS, int RG, int KG>
__global__ __launch_bounds__(64 * RG * KG, D == 64 || KG * RG == 8 ? 2 : 1)
void fwd_keysplit_kernel(const void* __restrict__ Qv, const void* __restrict__ Kv,
                         const void* __restrict__ Vv, void* __restrict__ Ov,
                         const float* __restrict__ mult, float* __restrict__ Zv,
                         int Nq, int Nk, int H, int kv_group, int n_qtiles, int n_items,
                         int n_splits, int keys_per_split, int item_begin, int item_end, int halves)
{
    constexpr int BR = 16 * NQ * RG;
    constexpr bool HALVES = D == 64 && CS == 1 && NQ == 4 && RG == 2 && KG == 2 && !MULT && !PARTIAL && QKT != QKType::Fp8;   // launch_halves
    if constexpr (HALVES) {
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
            fwd_keysplit_item<D, NQ, QKT, MULT, PARTIAL, CS, RG, KG>(Qv, Kv, Vv, Ov, mult, Zv, Nq, Nk, H, kv_group, n_qtiles, n_items,
                                                     n_splits, keys_per_split, item, halves == 2, true, 2 * BR, half * BR);
            return;
        }
    }
    const bool several_batches = item_end - item_begin > (int)gridDim.x || item_end < n_items;
    int batch = 0;
    for (int item = item_begin + blockIdx.x; item < item_end; item += gridDim.x, ++batch) {
        if (batch > 0) __syncthreads();            // every wave is done with the previous item's LDS
        fwd_keysplit_item<D, NQ, QKT, MULT, PARTIAL, CS, RG, KG>(Qv, Kv, Vv, Ov, mult, Zv, Nq, Nk, H, kv_group, n_qtiles, n_items,
                                                 n_splits, keys_per_split, item, batch % 2 == 1, several_batches, BR, 0);
    }
}

}  // namespace sphattn
