// Forward for fp32 storage on the 16-bit matrix instructions, in two fp16 parts or three bf16 parts.
//
// The fp32 matrix instruction (v_mfma_f32_32x32x2_f32) runs at 1/16 of the 16-bit ones' rate, so an fp32 product is
// taken apart.
//
// Two parts.  x = x0 + x1, each the rest before it rounded to fp16.  The rest has 12 bits and x1 holds 11, so x is off by
// 2^-23 of its power of two in one value of four and exact in the others: 2^-24 in the root mean square.
// x y = x0 y0 + (x0 y1 + x1 y0), three products; the one left out is at most 2^-22 |x y| and 2^-25 in the
// root mean square.  x1 has steps of 2^-24 at least, so all values are brought near the top of fp16's range by powers of two,
// which cost no bit: each row of Q to a largest element below 2^14, K to a mean exponent of 6 over 32 keys spread over the axis, each
// column of V likewise (zeros not counted), and a score with its count by 2^-17 and the power of two of the mean count.  The end takes
// them back.  What makes up for the parts' rounding is sums from zero: a score takes 12 additions at full size where three
// parts take 24 and the fp32 instruction 64; z receives four squares at a time, o 64 keys.  Error of O against 64 bits
// (relative 2-norm, normal values, d = 128) with three / two parts: 2.0e-7 / 1.9e-7 at 1000 keys, 3.0 / 2.5 at 5000,
// 5.2 / 3.8 at 20000; of z a half to two thirds.  Below 512 keys (d = 64: 1792) three parts are as close or closer, and such
// launches take them (f32_two_parts).
//
// The scales come from 32 keys and P has one for all of them, so the end asks what each element of O was formed of.  Below a
// power of two of 2^-2 a part's last bit is 2^-24 whatever the value.  So P is off by up to 2^-25 and, through K's last bits,
// 2^-17 2^-25 |row of Q|, 2^-24.5 at most; V by 2^-25; and an element of O by 2^-24.5 |column of V| and 2^-25 sqrt(z), all scaled, at random
// signs.  It is in doubt unless o^2 >= 2^-6 |column|^2 + 2^-8 z, above which that is 2^-21 of it in the worst case and 2^-22.5 in the
// root mean square.  Of normal values 0.4 to 1 % are in doubt, by chance, of one-hot V 2 to 5 %.  More than three eighths of a wave's rows of one
// column, or an eighth (and four) of a row's columns, are not chance but keys whose scores or values the scales do not fit and which
// carry that column or row: a key with 1e4 times the others' scores, say, and no value in some columns, which are then
// formed of the other keys.  (So that every wave has rows to count, rows past the last query are the head's first ones again; and a
// column whose squares come to zero is looked at a second time, as those of values below 2^-75 do: with a quarter of
// the columns zeros 1.5 to 3 % of the time, 6 % with zeros in all places.  Told apart in the loop by a second instruction per value: 1.6 % of every call.)
// Also asked: every row has z >= N / 16 in scaled scores (or is a row of zeros in Q); z without the scales is in
// [2^-100, 2^100]; no element is NaN (a value beyond fp16 leaves inf - inf).  If any wave of a workgroup sees one of these fail, after
// 512 keys (columns not yet; not on axes below 1024 keys) or at the end, the workgroup does its rows again in three parts, and from there with the fp32
// instruction.
//
// 8 x 4096 x 128: 284 us in three parts, 178 in two; 8 x 4096 x 64 171 and 109, 16 x 4000 x 128 534 and 324.  Given up after 512
// keys and done in three parts 10 to 13 % more than three parts alone; given up at the end, as is everything below 1024 keys, 60 to 65 %.  The products
// alone are 82 us of the 178 at 2.5 PFLOP/s; between them each SIMD splits the next tile and the scores.
//
// Three parts.  An fp32 value is the exact sum of three bf16 values, x = x0 + x1 + x2 (each the rest before it, rounded to bf16), so
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
// The watch costs 2 % (8 x 4096 x 128 in three parts 282.3 us without it, 288.7 with; 16 x 4096 x 64 283.8, 289.1).
// Done again from the first tile on, 8 x 4096 x 128 takes 707 us (702 on fwd_f32_kernel); from the last tile, 953.
//
// A workgroup is 8 waves (two per SIMD) x 16 NQ query rows; Q's parts stay in registers.
// K and V tiles of 32 keys arrive as they are through direct global -> LDS copies (each wave's share in
// a region of its own), are split by the wave that copied them, a unit at a time between its matrix
// instructions, and go to LDS as 16-bit images in
// the block formats of the other kernels: K as 16 x 64-byte blocks with permuted pieces (row-major
// reads), V as 16 x 32-byte blocks (transposing reads).  One barrier per tile.  Three parts: two buffers of six
// images.  Two parts: tiles go in pairs, the scores of both and then o from both, so K has two buffers and V
// three, and copies run two tiles ahead.
#pragma once
#include "sphattn_pipelined.hpp"

namespace sphattn {

constexpr int kF32Waves = 8;
constexpr int kF32Tile = 32;           // keys per tile

// LDS, in images of one part of a K or V tile.  Three parts: two sets of six, and one tile as copied (four).  Two parts: two
// tiles of K and three of V, two images each, and two tiles as copied.  Then a word per wave, sums over the
// first tile (of K per wave, of V per column in two halves) and the columns' powers of two.
template <int D>
constexpr int f32_flags_at() { return 18 * kF32Tile * D * 2; }
template <int D>
constexpr int f32_lds_bytes() { return f32_flags_at<D>() + 2 * kF32Waves * 4 + 3 * D * 4; }

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

// The same pair, already scaled, as two packed pairs of fp16.
struct Split2 { int p0, p1; };
__device__ __forceinline__ Split2 split2(float a, float b)
{
    Split2 r;
    r.p0 = pack2<true>(a, b);
    const f16x2 h = __builtin_bit_cast(f16x2, r.p0);
    r.p1 = pack2<true>(a - (float)h[0], b - (float)h[1]);
    return r;
}

// 2^e for an e that keeps it a normal number, and the e that brings a positive x to [2^(to - 1), 2^to); 0 for zero.
__device__ __forceinline__ float power_of_two(int e) { return __builtin_bit_cast(float, (uint32_t)(e + 127) << 23); }
__device__ __forceinline__ int exponent_to(float x, int to)
{
    const int e = to - __builtin_amdgcn_frexp_expf(x);
    return x > 0.f ? max(-126, min(126, e)) : 0;
}

// x of the lane N further on in the lane's row of 16.
template <int N>
__device__ __forceinline__ int lane_rotated(int x) { return __builtin_amdgcn_update_dpp(0, x, 0x120 + N, 0xf, 0xf, true); }

// One more bit at the low end of `bits`: whether a >= b does not hold.
__device__ __forceinline__ void append_unless(uint32_t& bits, float a, float b)
{
    asm("v_cmp_nge_f32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc" : "+v"(bits) : "v"(a), "v"(b) : "vcc");
}

// What a workgroup works on: its head's rows of Q, O and Z (null: not wanted), its keys, and its first row.
struct F32Rows {
    const float* Q; const float* K; const float* V; const float* mult; float* O; float* Z;
    int Nq, N, q0;
};

// Two parts: 8 waves x 16 NQ rows from p.q0 on; false, with nothing stored, where the values do not allow it.
// Every thread of the workgroup calls it and gets the same answer.
template <int D, int NQ, bool MULT, bool PARTIAL>
__device__ __forceinline__
bool f32_two_part_rows(const F32Rows& p)
{
    constexpr int BC = kF32Tile;
    constexpr int KK = D / 32, DB = D / 16;
    constexpr int IMG = BC * D * 2;                // one 16-bit image of a K or V tile
    constexpr int VRING = 4 * IMG;                 // V behind two tiles of K
    constexpr int RAW = 10 * IMG, FLAGS = f32_flags_at<D>(), SUMS = FLAGS + kF32Waves * 4, COLS = SUMS + kF32Waves * 4, POWERS = COLS + 2 * D * 4;
    constexpr int UNITS = 2 * 4 * KK;              // 1 KB units (8 rows x 32 columns of fp32) of K and V
    constexpr int UPW = UNITS / kF32Waves;         // per wave
    static_assert(UNITS % kF32Waves == 0, "units are dealt evenly");

    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    SPH_LDS unsigned char* smem = (SPH_LDS unsigned char*)smem_raw;

    const int Nq = p.Nq, N = p.N;
    const int tid = threadIdx.x, lane = tid & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n16 = lane & 15, g = lane >> 4;
    const int q0 = p.q0 + (int)wave * 16 * NQ;

    // ---- tile copies: unit u of this wave, rows past the last key as zeros.  Waves 0 to 3 have K, the others V; a
    // wave's units are one group of 32 columns, so that a lane has the same four columns in all of them
    const i32x4 krw = rsrc_words(p.K, (uint32_t)N * D * 4);
    const i32x4 vrw = rsrc_words(p.V, (uint32_t)N * D * 4);
    const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
    const int ld_lane = (lane >> 3) * D * 4 + (lane & 7) * 16;
    const int n_tiles = (N + BC - 1) / BC;
    const bool is_k = wave < 4;
    const int cg = (wave & 3) % KK, rg0 = (wave & 3) / KK * UPW;   // column group, first row group
    auto copy_tile = [&](int t) {                  // past the last tile zeros: no byte is in range
#pragma unroll
        for (int u = 0; u < UPW; ++u)
            copy_to_lds(is_k ? krw : vrw, lds0 + RAW + (t & 1) * 4 * IMG + (wave * UPW + u) * 1024, ld_lane,
                        t >= n_tiles ? N * D * 4 : f32_tile_byte<D>(t, (rg0 + u) * 8) + cg * 128);
    };
    auto raw_unit = [&](int u, int buffer) {
        return __builtin_bit_cast(f32x4, lds_read_b128(smem + RAW + buffer * 4 * IMG + (wave * UPW + u) * 1024 + lane * 16));
    };
    // what the waves of the workgroup say, together (a barrier between the two)
    auto say = [&](int what) { *reinterpret_cast<SPH_LDS int*>(smem + FLAGS + wave * 4) = what; };
    auto heard = [&]() -> int {
        const i32x4 a = lds_read_b128(smem + FLAGS), b = lds_read_b128(smem + FLAGS + 16);
        return __builtin_amdgcn_readfirstlane(a[0] | a[1] | a[2] | a[3] | b[0] | b[1] | b[2] | b[3]);
    };
    constexpr int OUTSIDE = 1, ZEROS = 2;
    // factors of the lane's four columns (of K: all the same), and the squares of V's columns, scaled
    f32x4 scale = {1.f, 1.f, 1.f, 1.f}, colsq = {0.f, 0.f, 0.f, 0.f};
    // The same units split into the images of the set at `set` (K's, V's): a row group is 8 rows of a 16-row block, whose other 8 rows lie 512 bytes
    // on in a K block (the same permutation of pieces) and 256 in a V block; the next block row D * 32.
    static_assert(UPW % 2 == 0, "rg0 is even");
    const int rowin = lane >> 3, c4 = lane & 7;    // row and float4 of the unit
    const int odd_rows = is_k ? 512 : 256;
    const int at = cg * 1024 + (is_k ? block_piece_offset(rowin, c4 >> 1) + (c4 & 1) * 8 : (c4 >> 2) * 512 + rowin * 32 + (c4 & 3) * 8);
    auto split_unit = [&](int u, int buffer, int kset, int vset) {
            f32x4 x = raw_unit(u, buffer);
            SPH_LDS unsigned char* dst = smem + (is_k ? kset : vset) + at + ((rg0 + u) >> 1) * D * 32 + (u & 1) * odd_rows;
            x *= scale;
#pragma unroll
            for (int e = 0; e < 4; ++e) colsq[e] = __builtin_fmaf(x[e], x[e], colsq[e]);
            const Split2 lo = split2(x[0], x[1]), hi = split2(x[2], x[3]);
            *reinterpret_cast<SPH_LDS i32x2*>(dst) = i32x2{lo.p0, hi.p0};
            *reinterpret_cast<SPH_LDS i32x2*>(dst + IMG) = i32x2{lo.p1, hi.p1};
    };
    auto wait_copies = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0x0F70);        // vmcnt(0)
        asm volatile("" ::: "memory");
    };
    // 32 keys spread over the axis, this wave's columns of K or V of 8 UPW of them: what the powers of two are taken from
    auto sampled_key = [&](int i) -> int { return (int)((uint32_t)i * (uint32_t)N >> 5); };
    f32x4 sample[UPW];
    {
        const float* src = is_k ? p.K : p.V;
#pragma unroll
        for (int u = 0; u < UPW; ++u)
            sample[u] = *reinterpret_cast<const f32x4*>(src + (size_t)sampled_key((rg0 + u) * 8 + rowin) * D + cg * 32 + c4 * 4);
    }
    copy_tile(0);
    copy_tile(1);

    // ---- Q in parts as B operands: row n16 of the block, elements 32 kk + 8 g .. + 7
    i32x4 qf[NQ][KK][2];
    int eq[NQ];                                    // the row's power of two
    bool qzero[NQ];
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb) {
        int row = q0 + qb * 16 + n16;
        if (p.q0 + kF32Waves * 16 * NQ > Nq)       // past the end the head's first rows again: computed, asked like any other, and dropped
            row = row < Nq ? row : row % Nq;
        const float* src = p.Q + (size_t)row * D + 8 * g;
        f32x4 x[KK][2];
        float most = 0.f;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                x[kk][h] = *reinterpret_cast<const f32x4*>(src + 32 * kk + 4 * h);
#pragma unroll
                for (int e = 0; e < 4; ++e) most = fmaxf(most, __builtin_fabsf(x[kk][h][e]));
            }
        most = max_across_groups(most);
        eq[qb] = exponent_to(most, 14);
        qzero[qb] = most == 0.f;
        const float f = power_of_two(eq[qb]);
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float a = x[kk][e >> 1][2 * (e & 1)], b = x[kk][e >> 1][2 * (e & 1) + 1];
                const Split2 s = split2(a * f, b * f);
                qf[qb][kk][0][e] = s.p0;
                qf[qb][kk][1][e] = s.p1;
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

    const __amdgpu_buffer_rsrc_t mrs = make_rsrc(p.mult, MULT ? (uint32_t)N * 4 : 0);
    auto load_counts = [&](int j, int kb) -> f32x4 {   // of the lane's keys 16 kb + 4 g + t; past the last key 0
        f32x4 m;
#pragma unroll
        for (int t = 0; t < 4; ++t)
            m[t] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(mrs, (j * BC + 16 * kb + 4 * g + t) * 4, 0, 0));
        return m;
    };
    wait_copies();
    int ek, ep = -17;                              // K's power of two; P = 2^ep (Q' K'), Q' and K' scaled
    {
        // Powers of two from the mean exponent of the sample's elements other than zero, which neither an outlier nor zeros
        // (padding, one-hot values, values cut at zero) move far: of K, and of each column of V.  Sums in one word:
        // the elements, from bit 20 on, and their exponents + 256, of 1024 at most.
        auto exponent_word = [](float x) -> int { return x != 0.f ? (1 << 20) + 256 + __builtin_amdgcn_frexp_expf(x) : 0; };
        auto mean_exponent = [](int elements, int sum) -> int {   // of at least one element
            return (int)__builtin_rintf((float)sum * __builtin_amdgcn_rcpf((float)elements)) - 256;
        };
        i32x4 word = {0, 0, 0, 0};
#pragma unroll
        for (int u = 0; u < UPW; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) word[e] += exponent_word(sample[u][e]);
#pragma unroll
        for (int w = 8; w < 64; w *= 2)            // over the unit's rows
#pragma unroll
            for (int e = 0; e < 4; ++e) word[e] += __shfl_xor(word[e], w);
        int all = word[0] + word[1] + word[2] + word[3];
#pragma unroll
        for (int w = 1; w < 8; w *= 2) all += __shfl_xor(all, w);
        if (lane == 0) *reinterpret_cast<SPH_LDS int*>(smem + SUMS + wave * 4) = all;
        if (!is_k && lane < 8) *reinterpret_cast<SPH_LDS i32x4*>(smem + COLS + ((wave & 3) / KK * D + cg * 32 + c4 * 4) * 4) = word;
        __syncthreads();
        const i32x4 ks = lds_read_b128(smem + SUMS), vs = lds_read_b128(smem + SUMS + 16);
        constexpr int LOW = (1 << 20) - 1;
        int kn = 0, ksum = 0, vn = 0, vsum = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            kn += ks[e] >> 20;
            ksum += ks[e] & LOW;
            vn += vs[e] >> 20;
            vsum += vs[e] & LOW;
        }
        ek = __builtin_amdgcn_readfirstlane(kn > 0 ? max(-126, min(126, 6 - mean_exponent(kn, ksum))) : 0);
        if constexpr (MULT) {
            const int key = sampled_key(lane & 31);
            int m = exponent_word(__builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(mrs, key * 4, 0, 0)));
#pragma unroll
            for (int w = 1; w < 32; w *= 2) m += __shfl_xor(m, w);
            if (m != 0) ep = max(-126, min(126, ep + 1 - mean_exponent(m >> 20, m & LOW)));
            ep = __builtin_amdgcn_readfirstlane(ep);
        }
        if (is_k) {
            const float f = power_of_two(ek);
            scale = f32x4{f, f, f, f};
        } else {
            const SPH_LDS unsigned char* sums = smem + COLS + (cg * 32 + c4 * 4) * 4;
            i32x4 cs = lds_read_b128(sums);
            if constexpr (KK == 2) cs += lds_read_b128(sums + D * 4);
            // A column with few values in the sample is not brought up further than the others (one small value says little of the
            // rest), one with none not brought down either, so that no value of it becomes zero.
            const int others = vn > 0 ? 6 - mean_exponent(vn, vsum) : 0;
            i32x4 ev;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int elements = cs[e] >> 20, own = elements > 0 ? 6 - mean_exponent(elements, cs[e] & LOW) : max(0, others);
                ev[e] = max(-126, min(126, elements > 0 && elements < 8 ? min(own, others) : own));
                scale[e] = power_of_two(ev[e]);
            }
            if (lane < 8) *reinterpret_cast<SPH_LDS i32x4*>(smem + POWERS + (cg * 32 + c4 * 4) * 4) = ev;   // (at KK = 2 by two waves, the same)
        }
    }
#pragma unroll
    for (int u = 0; u < UPW; ++u) split_unit(u, 0, 0, VRING);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);            // lgkmcnt(0): the copied bytes are read, the images written
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    // which part of the left and of the right operand each product takes, smallest first
    constexpr int PRODUCTS = 3, PA[3] = {1, 0, 0}, PB[3] = {0, 1, 0};
    const int klane = block_piece_offset(n16, g);
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    // Steps of a few fragments, read a step ahead, and their matrix instructions: KK score steps (both 16-key blocks of a
    // k-step), then output steps.  The next tile is split a unit at a time in between.
    // Tiles in pairs: the scores of both, then o += V^T P of both as one sum that is formed from zero, so o is rounded once
    // in 64 keys.  Copies run two tiles ahead; the second tile of a pair may be one past the end, all zeros.
    const float pscale = power_of_two(ep);
    int vring[3] = {VRING, VRING + 2 * IMG, VRING + 4 * IMG};   // V of the pair's tiles and of the next one
    i32x4 pf[2][NQ][2];
    auto tile_phase = [&](auto second, int j) __attribute__((always_inline)) {
        constexpr int SECOND = decltype(second)::value;
        constexpr int STEPS = KK + (SECOND ? DB : 0);
        // units from this step on, so many steps apart: the second tile's copies were asked for in the short first phase
        constexpr int FROM = SECOND ? 2 : 0, EVERY = SECOND ? (STEPS - FROM) / UPW : KK / UPW;
        static_assert(EVERY >= 1 && FROM + (UPW - 1) * EVERY < STEPS, "every unit has its step");
        const SPH_LDS unsigned char* kset = smem + SECOND * 2 * IMG;
        f32x4 mk[2];
        if constexpr (MULT) {
            mk[0] = load_counts(j, 0);
            mk[1] = load_counts(j, 1);
        }
        copy_tile(j + 2);
        i32x4 fr[2][2][2];                     // [step][key block, or tile of the pair][part]
        auto load_step = [&](int st) {
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    if (st < KK) {
                        fr[st & 1][u][q] = lds_read_b128(kset + q * IMG + (u * KK + st) * 1024 + klane);
                    } else {
                        const SPH_LDS unsigned char* a = smem + vring[u] + lane * 8 + q * IMG + (st - KK) * 512;
                        const i32x2 lo = lds_read_tr64(a), hi = lds_read_tr64(a + DB * 512);
                        fr[st & 1][u][q] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3);
                    }
                }
        };
        f32x4 s[2][NQ];
        load_step(0);
#pragma unroll
        for (int st = 0; st < STEPS; ++st) {
            if (st + 1 < STEPS) load_step(st + 1);
            if (st == FROM) {                  // the next tile has landed; the one after it may be under way
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_waitcnt(0x0F70 | UPW);
                asm volatile("" ::: "memory");
            }
            if (st >= FROM && (st - FROM) % EVERY == 0 && (st - FROM) / EVERY < UPW)
                split_unit((st - FROM) / EVERY, 1 - SECOND, (1 - SECOND) * 2 * IMG, vring[1 + SECOND]);
            if (st < KK) {
                // S^T = K Q^T
#pragma unroll
                for (int m = 0; m < PRODUCTS; ++m)
#pragma unroll
                    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                        for (int qb = 0; qb < NQ; ++qb)
                            s[kb][qb] = mfma16x16<true>(fr[st & 1][kb][PA[m]], qf[qb][st][PB[m]], st == 0 && m == 0 ? zero : s[kb][qb]);
                if (st == KK - 1) {
                    // z, and the scores in parts: registers 2 kb, 2 kb + 1 of the B operands
#pragma unroll
                    for (int qb = 0; qb < NQ; ++qb) {
                        float zt[2] = {0.f, 0.f};      // (from zero as well: one rounding of z in four squares)
#pragma unroll
                        for (int kb = 0; kb < 2; ++kb) {
                            if constexpr (MULT) s[kb][qb] *= mk[kb] * pscale;
                            else s[kb][qb] *= pscale;
#pragma unroll
                            for (int c = 0; c < 2; ++c) {
                                const float a = s[kb][qb][2 * c], b = s[kb][qb][2 * c + 1];
                                zt[0] = __builtin_fmaf(a, a, zt[0]);
                                zt[1] = __builtin_fmaf(b, b, zt[1]);
                                const Split2 x = split2(a, b);
                                pf[SECOND][qb][0][2 * kb + c] = x.p0;
                                pf[SECOND][qb][1][2 * kb + c] = x.p1;
                            }
                        }
                        zacc[qb][0] += zt[0];
                        zacc[qb][1] += zt[1];
                    }
                }
            } else {
                // O^T += V^T P over the pair's 64 keys
                f32x4 t[NQ];
#pragma unroll
                for (int m = 0; m < PRODUCTS; ++m)
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int qb = 0; qb < NQ; ++qb)
                            t[qb] = mfma16x16<true>(fr[st & 1][u][PA[m]], pf[u][qb][PB[m]], m == 0 && u == 0 ? zero : t[qb]);
#pragma unroll
                for (int qb = 0; qb < NQ; ++qb) oacc[st - KK][qb] += t[qb];
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        // the other K set and the next V are whole, this K set and the copied bytes may be overwritten
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xC07F);    // lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    // For the workgroup: OUTSIDE where the sums over the first `keys` keys are not what two parts hold, ZEROS where squares of V came to zero.  Before the end a row without any score (left
    // padding) is not asked yet.
    float z[NQ];
    auto in_range = [&](int keys, bool end) __attribute__((always_inline)) -> int {
        bool bad = false, zero = false;
        if (!is_k) {
            f32x4 all;
#pragma unroll
            for (int e = 0; e < 4; ++e) {          // over the unit's rows
                const float sum = colsq[e];        // (a bit cast of the vector's element itself takes element 0)
                all[e] = sum_across_groups(sum + __builtin_bit_cast(float, lane_rotated<8>(__builtin_bit_cast(int, sum))));
                zero |= all[e] == 0.f;
            }
            if (lane < 8) *reinterpret_cast<SPH_LDS f32x4*>(smem + COLS + ((wave & 3) / KK * D + cg * 32 + c4 * 4) * 4) = all;
        }
        __syncthreads();
        // An element of O is in doubt where it is not well above what the last bits of P (2^-25, times the column) and of V (times the row's
        // scores) come to.  Rows of zeros and columns of zeros have none.
        constexpr float NONE = -__builtin_inff();
        float zmin[NQ], finite = 0.f;
        int rows = 0;
        uint32_t zeros = 0;
        uint32_t doubts[NQ];                       // of the lane's columns, a bit each
#pragma unroll
        for (int qb = 0; qb < NQ; ++qb) {
            z[qb] = sum_across_groups(zacc[qb][0] + zacc[qb][1]);
            // the row's scores against the parts' resolution, and z as it is without the powers of two
            const float whole = __builtin_ldexpf(z[qb], -2 * (ep + eq[qb] + ek));
            const bool asked = !qzero[qb] && (end || z[qb] != 0.f);
            bad |= asked && !(z[qb] >= 0x1p-4f * (float)keys && whole >= 0x1p-100f && whole <= 0x1p100f);
            zmin[qb] = asked ? 0x1p-8f * z[qb] : NONE;
            finite += z[qb];
            rows += __builtin_popcountll(__ballot(asked) & 0xffff);
            doubts[qb] = 0;
        }
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            const SPH_LDS unsigned char* sums = smem + COLS + (db * 16 + 4 * g) * 4;
            f32x4 cs = __builtin_bit_cast(f32x4, lds_read_b128(sums));
            if constexpr (KK == 2) cs += __builtin_bit_cast(f32x4, lds_read_b128(sums + D * 4));
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float above_zero = cs[t] == 0.f ? -NONE : -0x1p-6f * cs[t];
                append_unless(zeros, cs[t], 0x1p-149f);
#pragma unroll
                for (int qb = 0; qb < NQ; ++qb) {
                    const float above = __builtin_fmaf(oacc[db][qb][t], oacc[db][qb][t], above_zero);
                    append_unless(doubts[qb], above, zmin[qb]);
                    // (a value that fp16 does not hold leaves NaN in its column of every row, a score in its whole row)
                    if (qb == 0 || (db == 0 && t == 0)) finite += above;
                }
            }
        }
        bad |= finite != finite;
        // In doubt at most: an eighth of a row's columns and four, and three eighths of the wave's rows of a column, counted bit by bit over the rows
        const float most = ((float)D - sum_across_groups((float)__builtin_popcount(zeros))) * 0.125f + 4.f;
        uint32_t n[6] = {doubts[0], 0, 0, 0, 0, 0};
#pragma unroll
        for (int qb = 0; qb < NQ; ++qb) bad |= sum_across_groups((float)__builtin_popcount(doubts[qb])) > most;
        if constexpr (NQ == 2) {
            n[1] = doubts[0] & doubts[1];
            n[0] = doubts[0] ^ doubts[1];
        }
        auto add_rotated = [&](auto by, int digits) __attribute__((always_inline)) {
            uint32_t carry = 0;
#pragma unroll
            for (int i = 0; i < 6; ++i) {
                if (i >= digits) { n[i] = i == digits ? carry : 0; continue; }
                const uint32_t m = lane_rotated<decltype(by)::value>(n[i]), x = n[i] ^ m;
                const uint32_t c = (n[i] & m) | (carry & x);
                n[i] = x ^ carry;
                carry = c;
            }
        };
        add_rotated(std::integral_constant<int, 8>{}, NQ);
        add_rotated(std::integral_constant<int, 4>{}, NQ + 1);
        add_rotated(std::integral_constant<int, 2>{}, NQ + 2);
        add_rotated(std::integral_constant<int, 1>{}, NQ + 3);
        // (not before the end: the squares of V are a tile ahead, and a column may have its first values there)
        const int limit = end ? rows * 3 / 8 : 16 * NQ;
        uint32_t more = 0, same = ~0u;             // columns whose count is above the limit, or equal so far
#pragma unroll
        for (int i = NQ + 3; i >= 0; --i) {
            const uint32_t bit = (limit >> i) & 1 ? ~0u : 0u;
            more |= same & n[i] & ~bit;
            same &= ~(n[i] ^ bit);
        }
        bad |= more != 0;
        say((__any(bad) ? OUTSIDE : 0) | (__any(zero) ? ZEROS : 0));
        __syncthreads();
        return heard();
    };
    // Asked at the end, and on long key axes once early, so that values that two parts cannot hold cost little more than
    // three parts do (a loop in a loop: asked inside one, d = 64 lost 4 %).
    constexpr int EARLY = 16;                      // tiles
    int found;
    for (int j = 0, stop = n_tiles < 2 * EARLY ? n_tiles : EARLY;; stop = n_tiles) {
        for (; j < stop; j += 2) {
            tile_phase(std::integral_constant<int, 0>{}, j);
            tile_phase(std::integral_constant<int, 1>{}, j + 1);
            const int next = vring[2];
            vring[2] = vring[1];
            vring[1] = vring[0];
            vring[0] = next;
        }
        found = in_range(min(N, stop * BC), stop == n_tiles);
        if ((found & OUTSIDE) || stop == n_tiles) break;
        __syncthreads();                           // the answer is read
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);            // the copies past the end must not land in what follows
    // Squares of values below 2^-75 vanish: are these columns zeros?  All waves look at the 32 columns around each again.
    if (found == ZEROS) {
        __syncthreads();                           // the answer is read
        bool values = false;
#pragma unroll 1
        for (int group = 0; group < KK; ++group) {
            const int column = group * 32 + c4 * 4;
            f32x4 sums = __builtin_bit_cast(f32x4, lds_read_b128(smem + COLS + column * 4));
            if constexpr (KK == 2) sums += __builtin_bit_cast(f32x4, lds_read_b128(smem + COLS + (D + column) * 4));
            if (!__any(sums[0] == 0.f || sums[1] == 0.f || sums[2] == 0.f || sums[3] == 0.f)) continue;
            uint32_t bits[4] = {0, 0, 0, 0};
#pragma unroll 8
            for (int key = wave * 8 + rowin; key < N; key += 64) {
                const f32x4 x = *reinterpret_cast<const f32x4*>(p.V + (size_t)key * D + column);
#pragma unroll
                for (int e = 0; e < 4; ++e) bits[e] |= doubled_bits(x[e]);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) values |= sums[e] == 0.f && bits[e] != 0;
        }
        say(__any(values) ? OUTSIDE : 0);
        __syncthreads();
        found = heard();
    }
    if (found & OUTSIDE) {
        __syncthreads();                           // the flags are read, the LDS is free
        return false;
    }
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb) {
        const int back = -(ep + eq[qb] + ek);      // a score is 2^back of what z and o were summed of
        const float inv = PARTIAL ? 1.f : z[qb] > 0.f ? 1.0f / __builtin_sqrtf(z[qb]) : 0.f;
        const int row = q0 + qb * 16 + n16;
        if (row < Nq) {
            if (g == 0 && (PARTIAL || p.Z != nullptr)) p.Z[row] = __builtin_ldexpf(z[qb], 2 * back);
            float* dst = p.O + (size_t)row * D + 4 * g;
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                f32x4 o = oacc[db][qb] * inv;
                const i32x4 ev = __builtin_bit_cast(i32x4, lds_read_b128(smem + POWERS + (db * 16 + 4 * g) * 4));
#pragma unroll
                for (int t = 0; t < 4; ++t) o[t] = __builtin_ldexpf(o[t], (PARTIAL ? back : 0) - ev[t]);
                *reinterpret_cast<f32x4*>(dst + db * 16) = o;
            }
        }
    }
    return true;
}

// Three parts.  Nq, Nk, Zv, PARTIAL, n_splits and keys_per_split as in fwd_pipelined_kernel.
template <int D, int NQ, bool MULT, bool PARTIAL>
__global__ __launch_bounds__(64 * kF32Waves, 2)
void fwd_f32x3_kernel(const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
                      float* __restrict__ O, const float* __restrict__ mult, float* __restrict__ Zv,
                      int Nq, int Nk, int H, int kv_group, int n_qtiles, int n_wg, int n_splits, int keys_per_split)
{
#include "sphattn_f32_three.inc"
}

// The same for a call from a kernel.
template <int D, int NQ, bool MULT, bool PARTIAL>
__device__ __forceinline__
void f32_three_part_rows(const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
                         float* __restrict__ O, const float* __restrict__ mult, float* __restrict__ Zv,
                         int Nq, int Nk, int H, int kv_group, int n_qtiles, int n_wg, int n_splits, int keys_per_split)
{
#include "sphattn_f32_three.inc"
}

// Two parts, and three where two do not hold the values.
template <int D, int NQ, bool MULT, bool PARTIAL>
__global__ __launch_bounds__(64 * kF32Waves, 2)
void fwd_f32x2_kernel(const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
                      float* __restrict__ O, const float* __restrict__ mult, float* __restrict__ Zv,
                      int Nq, int Nk, int H, int kv_group, int n_qtiles, int n_wg, int n_splits, int keys_per_split)
{
    {
        const int lid = xcd_contiguous_id(blockIdx.x, n_wg), qt = lid % n_qtiles;
        const int split = PARTIAL ? (lid / n_qtiles) % n_splits : 0;
        const int bh = PARTIAL ? lid / (n_qtiles * n_splits) : lid / n_qtiles, bidx = bh / H;
        const int k0 = PARTIAL ? split * keys_per_split : 0;
        const size_t kv_off = ((size_t)(bidx * (H / kv_group) + (bh % H) / kv_group) * Nk + k0) * D;
        const size_t rows0 = PARTIAL ? ((size_t)split * (n_wg / (n_qtiles * n_splits)) + bh) * Nq : (size_t)bh * Nq;
        const F32Rows p{Q + (size_t)bh * Nq * D, K + kv_off, V + kv_off, MULT ? mult + (size_t)bidx * Nk + k0 : nullptr, O + rows0 * D,
                        Zv != nullptr ? Zv + rows0 : nullptr, Nq, PARTIAL ? min(Nk - k0, keys_per_split) : Nk, qt * (kF32Waves * 16 * NQ)};
        if (f32_two_part_rows<D, NQ, MULT, PARTIAL>(p)) return;
    }
    // (All rows at once, which keeps 20 bytes a lane in scratch for 256 rows of d = 128: 128 at a time, without, took 18 % longer.)
    f32_three_part_rows<D, NQ, MULT, PARTIAL>(Q, K, V, O, mult, Zv, Nq, Nk, H, kv_group, n_qtiles, n_wg, n_splits, keys_per_split);
}

}  // namespace sphattn
