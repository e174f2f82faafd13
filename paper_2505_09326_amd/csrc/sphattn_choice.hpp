// Which kernel and how many query rows a launch takes, from its sizes: plain C++ that the library and its tests compile.
#pragma once
#include <initializer_list>

namespace sphattn {

constexpr int kChoiceTile = 64, kChoiceF32Tile = 32;   // keys that the times below are per

// How a launch of 16-bit or fp8-Q/K storage is laid out.  256 query rows (fwd_pipelined_kernel) is the shape of a full chip; the
// others (sphattn_keysplit.hpp) deal the keys of a tile to groups of waves, and pay while all their workgroups run at
// once, one per CU (two in Rows64 and Narrow at d = 64).  Rows64 has two key groups of two waves; Rows64Wide four of two, so two
// waves per SIMD; Rows64Own four of one wave with all 64 rows, which reads every K and V byte from LDS once (d = 128, where LDS and
// copies are the bound); Rows128 two of two, Rows128Wide four of two (d = 64); Rows256Wide two key groups of four waves
// (d = 64).  Narrow: 128 rows in four waves of 32 over all keys (bf16 without counts), which reads every fragment for
// two query blocks only, but starts with less.
enum Form { kRows64, kRows64Wide, kRows64Own, kRows128, kRows128Wide, kNarrow, kRows256Wide, kRows256, kForms };
constexpr int kFormRowsLog2[kForms] = {6, 6, 6, 7, 7, 7, 8, 8};

// Time of a launch that runs at once, in us: start + tiles (tile + share f of the CUs), the tiles of 64 keys rounded up to what the
// form's loop does at a time.  Fitted to 928 launches of bf16 and fp8 Q/K with and without counts (1 to 128 heads of 100 to 12000
// keys, every form timed on each; profiles/forward_forms_launches.txt): 1 to 4 % off in the root mean square, and what this picks is 0.0 to
// 0.3 % slower than the best form in the mean, 23 % at most (128 x 500 x 64).  Of Rows256Wide with fp8 Q/K, timed on 56 launches later, only the start is a fit (100 x 500
// with counts 12.0 us, 11.5 of Rows256; 24 x 2000 27.7, 28.7), the rest is bf16's.  tile 0: the form does not exist.  f16 measures like bf16.
struct FormCost { float start, tile, share; };
constexpr FormCost kFormCost[2][2][2][kForms] = {   // [d = 128][fp8 Q/K][counts]
    {{{{3.7f, .253f, .04f}, {4.5f, .162f, .05f}, {0, 0, 0}, {4.3f, .341f, .06f}, {5.5f, .262f, .08f}, {3.8f, .383f, .07f}, {5.0f, .453f, .15f}, {4.8f, .536f, .15f}},
      {{3.7f, .343f, .04f}, {4.7f, .228f, .05f}, {0, 0, 0}, {4.6f, .473f, .05f}, {5.8f, .324f, .07f}, {0, 0, 0}, {5.2f, .631f, .10f}, {4.7f, .728f, .09f}}},
     {{{3.6f, .230f, .04f}, {4.4f, .159f, .04f}, {0, 0, 0}, {4.5f, .322f, .05f}, {5.9f, .247f, .07f}, {0, 0, 0}, {5.4f, .453f, .15f}, {4.9f, .561f, .07f}},
      {{3.7f, .304f, .03f}, {4.6f, .197f, .04f}, {0, 0, 0}, {5.4f, .440f, .05f}, {6.1f, .313f, .08f}, {0, 0, 0}, {6.0f, .631f, .10f}, {4.9f, .729f, .07f}}}},
    {{{{4.7f, .370f, .09f}, {5.7f, .277f, .13f}, {6.5f, .276f, .11f}, {5.9f, .519f, .14f}, {0, 0, 0}, {4.7f, .506f, .20f}, {0, 0, 0}, {6.6f, .927f, .35f}},
      {{4.7f, .447f, .09f}, {5.7f, .334f, .14f}, {6.6f, .318f, .11f}, {6.1f, .616f, .11f}, {0, 0, 0}, {0, 0, 0}, {0, 0, 0}, {6.6f, 1.06f, .31f}}},
     {{{0, 0, 0}, {0, 0, 0}, {5.9f, .224f, .07f}, {5.5f, .446f, .10f}, {0, 0, 0}, {0, 0, 0}, {0, 0, 0}, {6.0f, .692f, .24f}},
      {{0, 0, 0}, {0, 0, 0}, {6.1f, .263f, .07f}, {5.6f, .533f, .09f}, {0, 0, 0}, {0, 0, 0}, {0, 0, 0}, {6.0f, .813f, .23f}}}}};

struct FormChoice { Form form; double us; };
struct Storage { bool bf16, fp8, counts; };
inline FormChoice choose_form(long long slices, long long Nq, long long tiles, int d, Storage st, long long cus)
{
    FormChoice best{kRows256, 0.0};
    if (slices * ((Nq + 255) / 256) > cus) return best;    // a full chip: rounds of 256 rows
    best.us = 1e30;
    const double per_cu = 1.0 / (double)cus;   // (no divisions by variables: this runs on every call)
    for (int form = 0; form < kForms; ++form) {
        const FormCost c = kFormCost[d == 128][st.fp8][st.counts][form];
        const long long items = slices * ((Nq + (1 << kFormRowsLog2[form]) - 1) >> kFormRowsLog2[form]);
        // two on a CU at d = 64: Narrow, and Rows64 for what has no Narrow.  They take 1.5 and 1.8 times as long as one (100 x 300 x 64
        // bf16 7.5 us, 8.5 on 256 rows; 64 x 500 x 64 fp8 7.6, 8.0 on 128 rows; 12 x 3000 x 64 fp8 with counts 34.8, 39.4)
        const double both = d != 64 ? 0.0 : form == kNarrow ? 1.5 : form == kRows64 && !(st.bf16 && !st.counts) ? 1.8 : 0.0;
        if (c.tile == 0 || (form == kNarrow && !st.bf16) || items > (both > 0.0 ? 2 * cus : cus)) continue;
        const long long step = form == kRows64Wide || form == kRows64Own || form == kRows128Wide ? 4 : form == kNarrow || form == kRows256 ? 1 : 2;
        const double n = (double)((tiles + step - 1) & -step), f = items > cus ? 1.0 : (double)items * per_cu;
        const double us = c.start + n * (c.tile + c.share * f) * (items > cus ? both : 1.0);
        if (us < best.us) best = FormChoice{(Form)form, us};
    }
    return best;
}

// Workgroups that share the columns of V and O of a row tile.  Where the 64-row workgroups of four key groups leave half of the CUs idle, two can have a
// row tile: each all of its scores and half of the columns, three quarters of the work and of the copies, and nothing to add up afterwards.  Form and
// figures as kFormCost, [d = 128][counts], fitted to 192 launches of 9 and more key tiles, 0.84 of the time in the mean at d = 128 and 0.95 at d = 64:
// 4 x 1999 x 128 15.6 -> 14.3 us, 8 x 1000 x 128 10.8 -> 9.4, with counts 2 x 3000 22.9 -> 20.5, 4 x 1999 x 64 9.9 -> 9.5.  On long key axes with most
// CUs busy K, then read twice, costs more than it gives (1 x 8000 x 128 43.8 us, 47.8 with halves; d = 64, 4 x 1999 of 4000, with counts 19.0 and 19.3).
// In place of Rows64 with two key groups from 3 tiles (d = 64: 7) on, 0.85 to 0.99 of the time there; below, halves take up to 8 % longer.
// At d = 128 four have quarters on axes of up to 64 tiles (on longer ones 0.91 to 1.27 of the halves' time): 64 x 1000 8.45 -> 7.93 us, 2 x 500
// 6.92 -> 6.60, with counts 9.43 -> 8.63 and 7.45 -> 7.00.  With nearly every CU busy K's copies, four times over, cost it again from 13 tiles on: 52 row
// tiles x 3000 16.7 -> 16.6 us, 60 17.3 -> 17.7, 64 17.8 -> 18.4; with counts, more work to hide them, 19.1 -> 18.0, 19.8 -> 19.2, 19.6 -> 19.6.
constexpr FormCost kHalfColumnsCost[2][2] = {{{4.28f, .141f, .045f}, {4.27f, .209f, .035f}}, {{4.32f, .255f, .115f}, {4.68f, .296f, .115f}}};
inline int column_shares(FormChoice c, long long slices, long long Nq, long long tiles, int d, Storage st, long long cus)
{
    if (st.fp8 || (c.form != kRows64 && c.form != kRows64Wide && c.form != kRows64Own)) return 1;
    const long long items = 2 * slices * ((Nq + 63) / 64);
    const FormCost h = kHalfColumnsCost[d == 128][st.counts];
    const double us = h.start + (double)((tiles + 3) & -4) * (h.tile + h.share * (double)items / (double)cus);
    if (items > cus || (d == 64 && tiles > 48) || (c.form == kRows64 ? tiles < (d == 128 ? 3 : 7) : us >= c.us)) return 1;
    const long long sixteenths = tiles <= 12 ? 16 : st.counts ? 15 : 13;
    return d == 128 && 32 * items <= sixteenths * cus && tiles <= 64 ? 4 : 2;
}

// d = 64, launches of more 256-row workgroups than CUs: 512 rows in eight waves, one workgroup per CU, in place of two of 256 rows in four
// waves, which share nothing: each byte of K and V is copied to LDS once per CU and not twice, and the waves of a SIMD stay at one tile by
// themselves.  8 x 32768 1415 -> 1384 us, 32 x 8192 370 -> 350, 9 x 8192 (one round, half filled) 152 -> 135, with counts 20 x 8192 358 -> 332,
// fp8 Q/K 289 -> 266.  Lines from 2200 launches of 257 to 5000 workgroups of 256 rows and 20 to 33000 keys, both forms timed on each (512 over
// 256 rows; taken: 0.96 in one round, 0.97 in several, 1.026 at most, 9 past 1.01):
//   fp8 Q/K with counts    spills, 1.02 to 1.05
//   from 129 key tiles on  256 rows have wave priorities by tile there.  Counts and fp8 Q/K 0.99 to 1.10 (fp8 Q/K 16 x 11180 374 and 394 us, with
//                          counts 20 x 10795 481 and 492); 16-bit storage 0.95 to 1.02, but in one round of heads of up to 3072 rows 0.96 to 1.07, as
//                          where K and V are past the 256 MB of the last-level cache (48 x 1333 of 29898 480 and 514)
//   fp8 Q/K past 256 MB    from 65 tiles on 0.97 to 1.03 (286 x 420 of 7777 273 and 281 us), below 0.98
//   short key axes         one round: 1 and 2 tiles 0.94 to 1.02 on heads of up to 1024 rows, else 0.95 to 1.04; several: up to 16 tiles 0.93 to 1.05
//                          (216 x 3519 of 581 124 and 127)
// Several rounds otherwise as they are filled: a round filled to f costs 0.5 + 0.5 f, and 256-row launches of 16-bit storage without counts may run
// their last one as halves (launch_pipelined): 8 x 17000 481 us, 547 with this, 8 x 24576 856 and 879.  Up to eight workgroups behind one round of
// 256 rows take one more item each on eight CUs, not a round (14 x 9470 with counts 327 and 366, 260 x 341 of 3124 99 and 129).
// In a launch of one round rows are added up in the same order either way; in several, every other one of which streams the keys
// backwards, a row may be in another kind of round.
inline bool rows512_pay(long long slices, long long Nq, long long tiles, Storage st, bool whole, long long cus)
{
    const long long n256 = slices * ((Nq + 255) / 256), n512 = slices * ((Nq + 511) / 512);
    const bool one_round = n512 <= cus;
    if (n256 <= cus || (st.fp8 && st.counts)) return false;
    if (tiles > 128 && (st.fp8 || st.counts || (one_round && Nq <= 3072))) return false;
    if (tiles > (st.fp8 ? 64 : 128) && slices * tiles * (kChoiceTile * 64 * (st.fp8 ? 3 : 4)) > (256ll << 20)) return false;
    if (one_round) return tiles >= 3 || Nq <= 1024;
    const long long full = n256 / (2 * cus), rest = n256 % (2 * cus);
    if (tiles < 17 || (full == 1 && rest > 0 && rest <= 8)) return false;
    double cost256 = 0.5 * (double)(full + (rest != 0)) + 0.25 * (double)n256 / (double)cus;
    if (whole && !st.fp8 && !st.counts && full >= 1 && rest > 0 && rest <= cus) {
        const double halves = (double)full + 0.3 + 0.3 * (double)rest / (double)cus;
        cost256 = halves < cost256 ? halves : cost256;
    }
    const double cost512 = 0.5 * (double)((n512 + cus - 1) / cus) + 0.5 * (double)n512 / (double)cus;
    return cost512 <= (tiles > 128 ? 1.0 : 1.02) * cost256;
}

// The same for a launch that has to add a row's terms in the order of kRows256, as Narrow does too (where the launch has it).  Narrow where it is one
// workgroup per CU (4 x 1999 x 128 22.3 us, 38.2 on 256 rows); two on a CU in place of kRows256Wide, on short key axes only (Narrow / 256 rows,
// d = 64: 32 x 2048 30.7 / 31.6, 24 x 2500 35.5 / 36.1, then 20 x 3000 39.2 / 37.1, 8 x 6000 65.2 / 60.3, 3 x 20000 235 / 226).
inline Form in_one_key_order(Form form, long long tiles, bool has_narrow)
{
    if (form == kRows256 || !has_narrow) return kRows256;
    return form != kRows256Wide || tiles <= 40 ? kNarrow : kRows256;
}

// fp32 storage has four workgroup shapes: 16 or 32 rows on the fp32 matrix instruction with the keys dealt
// to the waves (the least latency: the launches that cannot give every CU more than that), and 128
// or 256 rows in two fp16 or three bf16 parts.  Time of one round per 32-key tile, in us, as measured on launches
// that fill a small and the whole part of the CUs (f): d = 128 0.9, 1.42 on the fp32 instruction, 1.4 to 1.7, 2.0 to 2.6 in two
// parts, 2.05 to 2.55, 3.5 to 4.3 in three (without the watch that adds 2 %); d = 64 0.35, 0.68; 0.69 to 0.87, 1.0 to 1.38; 1.1 to 1.3, 1.85 to 2.25.
// Rounds times that picks the shape (32 rows, 128 and 256 in two parts, in three: 8 heads of 4096 x 128 704, 217 and
// 275, 328 and 452 us; 16 heads 1396, 433 and 333, 652 and 551; 4 heads of 4096 x 64 167, 99 and 150, 150 and 243; in three parts 1 x 8192 x
// 128 352, 553, 888, 16 rows 467; 4 x 1000 x 128 52, 73, 119, 16 rows 33).  S slices: S times the items, 1 / S of the tiles.
//
// Two parts wherever the results are then no further from 64 bits.  Error of O (relative 2-norm) with three / two parts:
// d = 128 1.73e-7 / 1.79e-7 at 200 keys, 1.85 / 1.84 at 500, 2.01 / 1.92 at 1000, 2.98 / 2.45 at 5000; d = 64
// 1.62 / 1.71 at 1000, 1.77 / 1.79 at 1500, 2.10 / 1.95 at 2500; z from 200 keys on closer with two.
inline bool f32_two_parts(long long keys, int d) { return keys >= (d == 128 ? 512 : 1792); }
struct F32Choice { int rows; double us; };
inline F32Choice choose_f32(long long heads, long long Nq, long long keys_per_slice, long long S, int d, long long n_cus)
{
    const double cus = (double)n_cus, tiles = (double)((keys_per_slice + kChoiceF32Tile - 1) / kChoiceF32Tile);
    const bool two = f32_two_parts(keys_per_slice, d);
    F32Choice best{32, 1e30};
    for (const int rows : {16, 32, 128, 256}) {
        const double items = (double)(heads * ((Nq + rows - 1) / rows) * S);
        const double f = items < cus ? items / cus : 1.0;
        double tau = d == 128 ? (rows == 16 ? 0.9 : rows == 32 ? 1.42 : rows == 128 ? 2.05 + 0.5 * f : 3.5 + 0.8 * f)
                              : (rows == 16 ? 0.35 : rows == 32 ? 0.68 : rows == 128 ? 1.1 + 0.2 * f : 1.85 + 0.4 * f);
        if (two && rows == 128) tau = d == 128 ? 1.4 + 0.28 * f : 0.69 + 0.18 * f;
        if (two && rows == 256) tau = d == 128 ? 2.0 + 0.6 * f : 1.0 + 0.38 * f;
        const double us = __builtin_ceil(items / cus) * tiles * tau;
        if (us < best.us) best = F32Choice{rows, us};
    }
    return best;
}

// Workgroups that share the columns of V of 16 rows on the fp32 instruction, as long as all have a CU of their own: such launches wait for one
// wave's chain of matrix instructions, half of which are V's.  Four shares, 1 x 256 x 64 6.5 -> 5.3 us, of 128 10.6 -> 8.1; two, 4 x 300 x 64 7.6 -> 6.8, of 128
// 14.1 -> 11.7.
inline int f32_small_column_shares(long long slices, long long Nq, long long cus)
{
    const long long items = slices * ((Nq + 15) / 16);
    return 4 * items <= cus ? 4 : 2 * items <= cus ? 2 : 1;
}

// The all-E4M3 forward's workgroup (sphattn_fp8.hpp): query blocks of 16 rows per wave, and waves.  64 rows while every CU gets at most
// one such workgroup, else 128 likewise, else 256: over 300 launches of 1 to 64 heads of 190 to 23000 keys, every shape timed on each, that is 0 to
// 0.5 % slower than the best shape in the mean and 4 % at most, and 0.68 to 0.76 of 256 rows in four waves (geometric mean; nowhere slower).  On 243
// launches of 65 to 800 heads of 60 to 16000 keys 0.81 of 256 rows in four waves (d = 128 0.92 at most, 64 1.01); other shapes were not timed there.
// At d = 64 above one round of 256 rows two workgroups share a CU, but not two of eight waves: the shape follows from rounds of two and a last
// round of one or two, in the units of a tile's time measured for them.  Without counts 256 rows in four waves, two on a CU 1.84, one 1.08,
// or 128 rows, 0.985 and 0.66 (8 x 9000 131.8 and 126.4 us, 12 x 5725 101.5 and 109.6; for a gain of 4 %); with counts 256 rows in eight waves, 1.11
// alone, or 128 rows, 1.16 and 0.74 (8 x 9000 165.3 and 138.5, 48 x 2149 57.6 and 58.2).
struct Fp8Shape { int nq, waves; };
inline Fp8Shape choose_fp8(long long heads, long long N, int d, bool counts, long long cus)
{
    if (heads * ((N + 63) / 64) <= cus) return Fp8Shape{1, 4};
    const long long n128 = heads * ((N + 127) / 128), n256 = heads * ((N + 255) / 256);
    if (n128 <= cus) return Fp8Shape{1, 8};
    if (d == 128 || n256 <= cus) return Fp8Shape{2, 8};
    auto cost = [cus](long long n, double two, double one) {   // rounds of two workgroups per CU and what is left
        const long long rest = n % (2 * cus);
        return (double)(n / (2 * cus)) * two + (rest == 0 ? 0.0 : rest <= cus ? one : two);
    };
    if (counts) return cost(n128, 1.16, 0.74) < 1.11 * (double)((n256 + cus - 1) / cus) ? Fp8Shape{2, 4} : Fp8Shape{2, 8};
    return cost(n128, 0.985, 0.66) < 0.96 * cost(n256, 1.84, 1.08) ? Fp8Shape{2, 4} : Fp8Shape{4, 4};
}

}  // namespace sphattn
