// SpDM kernel in which the sixteen waves of a workgroup share the rows of B through LDS (Algorithm 2 of the paper re-cut
// for CDNA4; the schedule it reads is described in gcoo_band.hpp).
//
// Work unit = (block of 16 h rows of A, column tile of 256 columns).  A lane keeps (24 + 1) x 4 partial sums (its four
// columns of the wave's rows, and the sink row; the tall cut: (48 + 1) x 2, tiles of 128 columns) in v[28:127], so four waves share a SIMD: what one wave waits for - LDS, scalar
// loads, the barrier - the other three fill.  With 48 rows per wave and two waves per SIMD nothing hid behind
// anything: every instruction of a wave took six to eight clocks.
//
// Per entry:   v_and_or_b32    LDS address of the B row (the record's place | lane * 16)
//              ds_read_b128    the lane's four columns of it, four entries ahead of their use
//              s_set_gpr_idx   the entry's row selects the partial sums (index mode, M0)
//              4 x v_fmac_f32  sum[row][c] += value * b[c]
// and for the second entry of a pair only the last two.  Value and row are scalar operands: the records come through the
// scalar cache, a unit of 16 at a time into one of two register banks while the other is multiplied, so no vector instruction
// moves them.  A multiply-add with a scalar (or DPP) operand or in index mode takes 1.8 ns per SIMD, the other vector
// instructions too: five of them per single entry, 9 ns, are what bounds dense bands; 10.1 measured in a loop of nothing else.
// By the counters a SIMD issues a vector instruction every 2.2 ns at 8000 x 8000, 10 %, and every 2.7 at 14000 x 14000, 2 % (15 and 14 of 16 waves resident).
// Sparser matrices have few entries per (wave, band), 3.5 ns at 4000 x 4000, 2 %: there the bands by themselves weigh.  No bank conflicts anywhere.
//
// The tall cut (V = 2): the same registers and the same LDS hold twice the rows of A and of B, half as wide.  A row of B is fetched for twice as
// many rows of A, and a launch has half as many bands, each with four times the entries of a wave; an entry costs a multiply-add
// less than half but the same address, read and index (7.5 ns in a loop of nothing else, where the wide cut takes 10.2 for twice the columns): the unit that reads LDS takes
// as long for 8 bytes per lane as for 16, and is the bound of dense matrices.  For sparse ones what is fetched and the bands are: 8000 x 8000, 0.5 %: 333 -> 294 us (a vector
// instruction every 4.1 ns, rows of B and entries from L2 at 9.7 TB/s),
// where the same launch without its multiply-adds takes 290, without its requests 240, and with neither requests nor
// entries 68: a band is a chain of waits (rows of B from L2, LDS, barrier) that fifteen other waves in the same phase do not fill.
//
// B: two bands of 80 rows x 1 KB in LDS.  While band b is multiplied, the rows of band b + 1 are requested, five per wave, straight
// to LDS; their columns come with the band's head, and the address is formed by the scalar unit.  One barrier per band, no rows of B
// in flight across it.  Rows of B that are aligned to 4 bytes only are fetched by the same requests of 16 bytes per lane, a line more for each: 8000 x 8000, N = 7999 (us, four requests of
// 4 bytes per lane instead, so, and N = 8000): 0.5 % 358 317 288; 2 % 677 646 630; 10 % 2335 2295 2287.
//
// When the rows are requested.  A request holds the one address path of the compute unit for 16 clocks, and a wave that finds it taken
// stands still: with all five requests of all waves at the band's start nobody multiplied for the first 0.5 us.  Four ways (SPREAD, LATE):
//   true, false     every wave asks for two rows at the start and one behind each of its first three steps; a band of few entries per
//                   wave would end before the late half's rows have landed
//   true, true      (the wide cut only) waves 0 - 7 at the start, waves 8 - 15 behind the second step of their first unit (or at the end of the band): one half
//                   multiplies while the other asks
//   false, false    as that, waves 8 - 15 behind their first unit
//   false, true     as that, waves 8 - 15 behind their second unit: where a band has units enough, the later the better
// Product alone, all at the start -> behind the first unit (us): 14000 x 14000, 2 % 3460 -> 3165; 8000 x 8000, 2 % 672 -> 633; 10 % 2323 -> 2284; 6001 x 6001,
// 1 % 290 -> 254; spread: 8000 x 8000, 0.5 % 366 -> 345; 10000 x 10000, 0.4 % 667 -> 590 (by halves 371 and 670).  A quarter of the
// waves at a time, a unit apart, is slower (1 % and more below 60 entries of a (wave, band), up to 10 % at 20); so is asking a row at a time and step everywhere (3365 for the first),
// the late half behind the first step (1 to 4 % slower than behind the first unit), and the early half behind its first step (2 %).  Where each is taken: launch_spdm_band().
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gcoo_band.hpp"
#include "gcoo_spdm_launch.hpp"
#include "gcoo_spdm_rows_kernel.hpp"

namespace gcoo {

constexpr int kBandFillBytes = kBandFetches * 1024;                // what a wave fetches of a band
constexpr int kBandBufferBytes = kBandWaves * kBandFillBytes;
constexpr int kBandLdsBytes = 2 * kBandBufferBytes;
static_assert(sizeof(RowsAllLds) <= kBandLdsBytes && kRowsAllLong <= 64 * kBandWaves, "uneven rows");
static_assert(kBandFetches == 5 && BandCut<4>::kRows * 1024 == kBandBufferBytes && BandCut<2>::kRows * 512 == kBandBufferBytes, "the asm text below uses these numbers");

typedef float band_f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t band_u32x4 __attribute__((ext_vector_type(4)));
typedef float band_f32x32 __attribute__((ext_vector_type(32)));

// sum(c, r) = v[28 + 25 * c + r], c = 0..3, r = 0..24 (wide); v[28 + 49 * c + r], c = 0..1, r = 0..48 (tall)
struct BandAcc {
    band_f32x4 t0;                    // v[28:31]
    band_f32x32 t1, t2, t3;           // v[32:127]
};
__device__ __forceinline__ float band_acc_get(const BandAcc& a, int s)
{
    if (s < 4) return a.t0[s];
    const int t = (s - 4) >> 5, i = (s - 4) & 31;
    return t == 0 ? a.t1[i] : t == 1 ? a.t2[i] : a.t3[i];
}

// ---- asm text -----------------------------------------------------------------------------------
// Registers of the main loop:
//   v0 lane * 16    v1 0x3fc00, the place field of a record    v2 the lane's byte offset in a row of B (lane * 16)
//   v3        LDS address of the next read    v[4:27] six sets of B values
//   s[36:67]  bank A: the unit that is multiplied, s[68:99]  bank B: the next one (or the other way round): value, place and row of record i
//   s12 s13   byte offsets of the head after next and of the next unit    s14  where the wave's rows of the next band go in LDS
//   s15 bands left   s[16:22]  head of this band: five columns, pair steps, single steps    s[24:30] of the next one    s23 scratch
//   s[32:35]  buffer descriptor of B, from the tile's first column on
//   vcc       not 0: rows of the next band are still to be requested (spread: 1 + how often it was done behind a step; halves: 1 or 2, the units behind which they will be);
//             all 64 bits are written each time, as a write to a half need not reach what s_cbranch_vccnz looks at
//   tall only: v126 scratch, v127 all ones in the upper half of the wave, s100 scratch
// What differs between the cuts: BD_FMAC_T<i> (the entry's partial sums += value x set i), BD_READ_T<i>, BD_MASK, BD_BEGIN, BD_FILL.
#define BD_FMAC_WIDE(val, b0, b1, b2, b3)              \
    "v_fmac_f32 v28, " #val ", " #b0 "\n\t"             \
    "v_fmac_f32 v53, " #val ", " #b1 "\n\t"             \
    "v_fmac_f32 v78, " #val ", " #b2 "\n\t"             \
    "v_fmac_f32 v103, " #val ", " #b3 "\n\t"
#define BD_FMAC_TALL(val, b0, b1)                      \
    "v_fmac_f32 v28, " #val ", " #b0 "\n\t"             \
    "v_fmac_f32 v77, " #val ", " #b1 "\n\t"
#define BD_READ_WIDE(meta, set) "v_and_or_b32 v3, " #meta ", v1, v0\n\tds_read_b128 " set ", v3\n\t"
#define BD_READ_TALL(meta, set) "v_and_or_b32 v3, " #meta ", v1, v0\n\tds_read_b64 " set ", v3\n\t"
// two entries, of sets A and B; index mode is off before and after
#define BD_TWO(val0, meta0, A, val1, meta1, B)                    \
    "s_set_gpr_idx_on " #meta0 ", gpr_idx(SRC2,DST)\n\t"           \
    BD_FMAC_##A(val0)                                              \
    "s_set_gpr_idx_idx " #meta1 "\n\t"                             \
    BD_FMAC_##B(val1)                                              \
    "s_set_gpr_idx_off\n\t"
// Step i of a unit at priority i, so that the waves of a SIMD go through their entries at one pace.  Among waves of one priority a SIMD serves the oldest first: the
// others had what was left, and the youngest went through the last of its entries alone, one instruction in six clocks (clocks from a barrier to the end of a wave's entries,
// waves 0 - 3, 4 - 7, 8 - 11 and 12 - 15, 8000 x 8000, 10 %: 9800 11400 14100 16500).  Product alone (us): 8000 x 8000, 10 % 2300 -> 2030,
// 4000 x 4000, 5 % 198 -> 183, 2 % 111 -> 108; 14000 x 14000, 2 % 3180 -> 2990; 8000 x 8000, 0.5 % 296 -> 286 (a whole step of it, conversion and product in turn, is level: 323).  Falling with the steps as fast; two priorities in turn 2170 to 2220 for the first.
#define BD_TURN(i) "s_setprio " #i "\n\t"
#define BD_WAIT(n) "s_waitcnt lgkmcnt(" #n ")\n\t"

// Request t of the five of a wave for the next band: one row of B (wide) or two, one per half of the wave (tall); the column, or both, in s<16 + t>.
#define BD_FILL_WIDE(col, at)                   \
    "s_add_u32 m0, s14, " #at "\n\t"             \
    "s_mul_i32 s23, " #col ", %[ldb4]\n\t"       \
    BD_LOAD_ROW
#define BD_FILL_TALL(cols, at)                                                                                          \
    "s_add_u32 m0, s14, " #at "\n\ts_and_b32 s23, " #cols ", 0xffff\n\ts_lshr_b32 s100, " #cols ", 16\n\t"            \
    "s_mul_i32 s23, s23, %[ldb4]\n\ts_mul_i32 s100, s100, %[ldb4]\n\t"                                                 \
    "v_and_b32 v126, s100, v127\n\tv_add_u32 v126, v126, v2\n\tbuffer_load_dwordx4 v126, s[32:35], s23 offen lds\n\t"
#define BD_FILL_BAND BD_FILL(s16, 0) BD_FILL(s17, 0x400) BD_FILL(s18, 0x800) BD_FILL(s19, 0xc00) BD_FILL(s20, 0x1000)
// The places where rows are requested; T = p (pair steps) or s (single steps).  BD_ASK_START behind the first reads of a band, BD_ASK_STEP behind
// step I of its first unit, BD_ASK_UNIT in front of a further unit, BD_ASK_END at its end; what is done there stands out of line (BD_ASK_REST).
#define BD_ASK_HERE(L, X) "s_cbranch_vccnz .Lbd_" #L "_" #X "_%=\n.Lbd_" #L "back_" #X "_%=:\n\t"
#define BD_ASK_THERE(L, X, STATE, FILLS) ".Lbd_" #L "_" #X "_%=:\n\ts_mov_b64 vcc, " #STATE "\n\t" FILLS "s_branch .Lbd_" #L "back_" #X "_%=\n"
#define BD_ASK_END(X) BD_ASK_HERE(fe, X)
// by halves, waves 8 - 15 behind unit LATE (STEP1: behind the second step of the first one)
#define BD_HALVES_START(T, X, LATE) "s_cmp_ge_u32 %[fillw], 0xa000\n\ts_cselect_b64 vcc, " #LATE ", 0\n\ts_cbranch_scc1 .Lbd_late" #T "_" #X "_%=\n\t" BD_FILL_BAND ".Lbd_late" #T "_" #X "_%=:\n\t"
#define BD_HALVES_STEP(T, I, X)
#define BD_HALVES_UNIT(T, X) BD_ASK_HERE(f##T, X)
#define BD_FIRST_START(T, X) BD_HALVES_START(T, X, 1)
#define BD_FIRST_REST(X) BD_ASK_THERE(fp, X, 0, BD_FILL_BAND) BD_ASK_THERE(fs, X, 0, BD_FILL_BAND) BD_ASK_THERE(fe, X, 0, BD_FILL_BAND)
#define BD_STEP1_STEP(T, I, X) BD_STEP1_STEP_##I(T, X)
#define BD_STEP1_STEP_0(T, X)
#define BD_STEP1_STEP_1(T, X) BD_ASK_HERE(f##T##1, X)
#define BD_STEP1_STEP_2(T, X)
#define BD_STEP1_UNIT(T, X)
#define BD_STEP1_REST(X) BD_ASK_THERE(fp1, X, 0, BD_FILL_BAND) BD_ASK_THERE(fs1, X, 0, BD_FILL_BAND) BD_ASK_THERE(fe, X, 0, BD_FILL_BAND)
#define BD_SECOND_START(T, X) BD_HALVES_START(T, X, 2)
#define BD_SECOND_UNIT(L, X) ".Lbd_" #L "_" #X "_%=:\n\ts_lshr_b64 vcc, vcc, 1\n\ts_cbranch_scc1 .Lbd_" #L "back_" #X "_%=\n\t" BD_FILL_BAND "s_branch .Lbd_" #L "back_" #X "_%=\n"
#define BD_SECOND_REST(X) BD_SECOND_UNIT(fp, X) BD_SECOND_UNIT(fs, X) BD_ASK_THERE(fe, X, 0, BD_FILL_BAND)
// spread
#define BD_SPREAD_START(T, X) "s_mov_b64 vcc, 1\n\t" BD_FILL(s16, 0) BD_FILL(s17, 0x400)
#define BD_SPREAD_STEP(T, I, X) BD_ASK_HERE(f##T##I, X)
#define BD_SPREAD_UNIT(T, X)
#define BD_SPREAD_REST(X)                                                                              \
    BD_ASK_THERE(fp0, X, 2, BD_FILL(s18, 0x800)) BD_ASK_THERE(fp1, X, 3, BD_FILL(s19, 0xc00)) BD_ASK_THERE(fp2, X, 0, BD_FILL(s20, 0x1000))    \
    BD_ASK_THERE(fs0, X, 2, BD_FILL(s18, 0x800)) BD_ASK_THERE(fs1, X, 3, BD_FILL(s19, 0xc00)) BD_ASK_THERE(fs2, X, 0, BD_FILL(s20, 0x1000))    \
    ".Lbd_fe_" #X "_%=:\n\t"                                                                           \
    "s_cmp_gt_u32 vcc_lo, 1\n\ts_cbranch_scc1 .Lbd_fe1_" #X "_%=\n\t" BD_FILL(s18, 0x800) ".Lbd_fe1_" #X "_%=:\n\t"     \
    "s_cmp_gt_u32 vcc_lo, 2\n\ts_cbranch_scc1 .Lbd_fe2_" #X "_%=\n\t" BD_FILL(s19, 0xc00) ".Lbd_fe2_" #X "_%=:\n\t"     \
    BD_FILL(s20, 0x1000) "s_mov_b64 vcc, 0\n\ts_branch .Lbd_feback_" #X "_%=\n"

#define BD_LOAD_UNIT(lo, hi)                                      \
    "s_load_dwordx16 s[" lo "], %[units], s13\n\t"                 \
    "s_load_dwordx16 s[" hi "], %[units], s13 offset:0x40\n\t"     \
    "s_add_u32 s13, s13, 0x80\n\t"
#define BD_LOAD_A BD_LOAD_UNIT("36:51", "52:67")
#define BD_LOAD_B BD_LOAD_UNIT("68:83", "84:99")

// One bank's half of the loop.  X = the bank whose unit is multiplied, Y = the other one, into which the next unit is loaded meanwhile;
// a<i>, m<i> = value and meta word of record i of bank X.  Labels: end_X (the band before has ended, its next unit is in X), band_X (a
// band begins), unitp_X / units_X (a band goes on in X, with pairs / with singles), p<i>_X, s<i>_X (step i of the unit).
#define BD_HALF(X, Y, a0, m0, a1, m1, a2, m2, a3, m3, a4, m4, a5, m5, a6, m6, a7, m7, a8, m8, a9, m9, a10, m10, a11, m11, a12, m12, a13, m13, a14, m14, a15, m15) \
    ".Lbd_unitp_" #X "_%=:\n\t"                                                                 \
    BD_ASK_UNIT(p, X)                                                                           \
    BD_WAIT(0) BD_LOAD_##Y                                                                      \
    BD_READ_T0(m0) BD_READ_T1(m2) BD_READ_T2(m4) BD_READ_T3(m6)                                 \
    "s_branch .Lbd_p0_" #X "_%=\n"                                                              \
    ".Lbd_units_" #X "_%=:\n\t"                                                                 \
    BD_ASK_UNIT(s, X)                                                                           \
    BD_WAIT(0) BD_LOAD_##Y                                                                      \
    BD_READ_T0(m0) BD_READ_T1(m1) BD_READ_T2(m2) BD_READ_T3(m3)                                 \
    "s_branch .Lbd_s0_" #X "_%=\n"                                                              \
    ".Lbd_ps1_" #X "_%=:\n\t"                                                                   \
    "s_cmp_eq_u32 s22, 0\n\ts_cbranch_scc1 .Lbd_end_" #Y "_%=\n\t"                              \
    BD_READ_T4(m4) BD_READ_T5(m5) BD_READ_T0(m6) BD_READ_T1(m7)                                 \
    "s_branch .Lbd_s1_" #X "_%=\n"                                                              \
    ".Lbd_ps2_" #X "_%=:\n\t"                                                                   \
    "s_cmp_eq_u32 s22, 0\n\ts_cbranch_scc1 .Lbd_end_" #Y "_%=\n\t"                              \
    BD_READ_T2(m8) BD_READ_T3(m9) BD_READ_T4(m10) BD_READ_T5(m11)                               \
    "s_branch .Lbd_s2_" #X "_%=\n"                                                              \
    ".Lbd_ps3_" #X "_%=:\n\t"                                                                   \
    "s_cmp_eq_u32 s22, 0\n\ts_cbranch_scc1 .Lbd_end_" #Y "_%=\n\t"                              \
    BD_READ_T0(m12) BD_READ_T1(m13) BD_READ_T2(m14) BD_READ_T3(m15)                             \
    "s_branch .Lbd_s3_" #X "_%=\n"                                                              \
    /* the end of a band: its last row requests, then the rows of the next band have landed and all waves are done with this one; its second unit is asked for in front of the barrier, whose wait \
       hides what it can of that (product alone, us, behind it and so: 4000 x 4000, 2 % 92.0 91.0, 5 % 158.7 157.3; 8000 x 8000, 0.5 % 274.4 273.7 (about 300 behind a conversion), 10 % 2023 2012; 14000 x 14000, 2 % 2985 2969) */ \
    ".Lbd_end_" #X "_%=:\n\t"                                                                   \
    BD_ASK_END(X)                                                                               \
    "s_sub_u32 s14, %[flip], s14\n\t"                                                           \
    BD_WAIT_BAND                                                                                \
    "s_mov_b64 s[16:17], s[24:25]\n\t"                                                          \
    "s_mov_b64 s[18:19], s[26:27]\n\t"                                                          \
    "s_mov_b64 s[20:21], s[28:29]\n\t"                                                          \
    "s_mov_b32 s22, s30\n\t"                                                                    \
    "s_load_dwordx8 s[24:31], %[head], s12\n\t"                                                 \
    "s_add_u32 s12, s12, 32\n\t"                                                                \
    BD_LOAD_##Y                                                                                 \
    "s_barrier\n\t"                                                                             \
    "s_sub_u32 s15, s15, 1\n\t"                                                                 \
    "s_cbranch_scc1 .Lbd_done_%=\n"                                                             \
    ".Lbd_band_" #X "_%=:\n\t"                                                                  \
    "s_cmp_eq_u32 s21, 0\n\ts_cbranch_scc1 .Lbd_bs_" #X "_%=\n\t"                               \
    BD_READ_T0(m0) BD_READ_T1(m2) BD_READ_T2(m4) BD_READ_T3(m6)                                 \
    BD_ASK_START(p, X)                                                                          \
    ".Lbd_p0_" #X "_%=:\n\t"                                                                    \
    BD_TURN(0) "s_sub_u32 s21, s21, 1\n\t"                                                      \
    BD_READ_T4(m8) BD_WAIT(4) BD_TWO(a0, m0, T0, a1, m1, T0)                                    \
    BD_READ_T5(m10) BD_WAIT(4) BD_TWO(a2, m2, T1, a3, m3, T1)                                   \
    BD_ASK_STEP(p, 0, X)                                                                        \
    "s_sub_u32 s21, s21, 1\n\ts_cbranch_scc1 .Lbd_ps1_" #X "_%=\n\t"                            \
    BD_TURN(1) BD_READ_T0(m12) BD_WAIT(4) BD_TWO(a4, m4, T2, a5, m5, T2)                        \
    BD_READ_T1(m14) BD_WAIT(4) BD_TWO(a6, m6, T3, a7, m7, T3)                                   \
    BD_ASK_STEP(p, 1, X)                                                                        \
    "s_sub_u32 s21, s21, 1\n\ts_cbranch_scc1 .Lbd_ps2_" #X "_%=\n\t"                            \
    BD_TURN(2) BD_WAIT(3) BD_TWO(a8, m8, T4, a9, m9, T4)                                        \
    BD_WAIT(2) BD_TWO(a10, m10, T5, a11, m11, T5)                                               \
    BD_ASK_STEP(p, 2, X)                                                                        \
    "s_sub_u32 s21, s21, 1\n\ts_cbranch_scc1 .Lbd_ps3_" #X "_%=\n\t"                            \
    BD_TURN(3) BD_WAIT(1) BD_TWO(a12, m12, T0, a13, m13, T0)                                    \
    BD_WAIT(0) BD_TWO(a14, m14, T1, a15, m15, T1)                                               \
    "s_cmp_lg_u32 s21, 0\n\ts_cbranch_scc1 .Lbd_unitp_" #Y "_%=\n\t"                            \
    "s_cmp_lg_u32 s22, 0\n\ts_cbranch_scc1 .Lbd_units_" #Y "_%=\n\t"                            \
    "s_branch .Lbd_end_" #Y "_%=\n"                                                             \
    ".Lbd_empty_" #X "_%=:\n\t"                                                                 \
    BD_FILL_BAND                                                                                \
    "s_branch .Lbd_end_" #Y "_%=\n"                                                             \
    BD_ASK_REST(X)                                                                              \
    ".Lbd_bs_" #X "_%=:\n\t"                                                                    \
    "s_cmp_eq_u32 s22, 0\n\ts_cbranch_scc1 .Lbd_empty_" #X "_%=\n\t"                            \
    BD_READ_T0(m0) BD_READ_T1(m1) BD_READ_T2(m2) BD_READ_T3(m3)                                 \
    BD_ASK_START(s, X)                                                                          \
    ".Lbd_s0_" #X "_%=:\n\t"                                                                    \
    BD_TURN(0) "s_sub_u32 s22, s22, 1\n\t"                                                      \
    BD_READ_T4(m4) BD_READ_T5(m5) BD_WAIT(4) BD_TWO(a0, m0, T0, a1, m1, T1)                     \
    BD_READ_T0(m6) BD_READ_T1(m7) BD_WAIT(4) BD_TWO(a2, m2, T2, a3, m3, T3)                     \
    BD_ASK_STEP(s, 0, X)                                                                        \
    ".Lbd_s1_" #X "_%=:\n\t"                                                                    \
    BD_TURN(1) "s_sub_u32 s22, s22, 1\n\ts_cbranch_scc1 .Lbd_end_" #Y "_%=\n\t"                 \
    BD_READ_T2(m8) BD_READ_T3(m9) BD_WAIT(4) BD_TWO(a4, m4, T4, a5, m5, T5)                     \
    BD_READ_T4(m10) BD_READ_T5(m11) BD_WAIT(4) BD_TWO(a6, m6, T0, a7, m7, T1)                   \
    BD_ASK_STEP(s, 1, X)                                                                        \
    ".Lbd_s2_" #X "_%=:\n\t"                                                                    \
    BD_TURN(2) "s_sub_u32 s22, s22, 1\n\ts_cbranch_scc1 .Lbd_end_" #Y "_%=\n\t"                 \
    BD_READ_T0(m12) BD_READ_T1(m13) BD_WAIT(4) BD_TWO(a8, m8, T2, a9, m9, T3)                   \
    BD_READ_T2(m14) BD_READ_T3(m15) BD_WAIT(4) BD_TWO(a10, m10, T4, a11, m11, T5)               \
    BD_ASK_STEP(s, 2, X)                                                                        \
    ".Lbd_s3_" #X "_%=:\n\t"                                                                    \
    BD_TURN(3) "s_sub_u32 s22, s22, 1\n\ts_cbranch_scc1 .Lbd_end_" #Y "_%=\n\t"                 \
    BD_WAIT(2) BD_TWO(a12, m12, T0, a13, m13, T1)                                               \
    BD_WAIT(0) BD_TWO(a14, m14, T2, a15, m15, T3)                                               \
    "s_cmp_lg_u32 s22, 0\n\ts_cbranch_scc1 .Lbd_units_" #Y "_%=\n\t"                            \
    "s_branch .Lbd_end_" #Y "_%=\n"
#define BD_HALF_A BD_HALF(A, B, s36, s37, s38, s39, s40, s41, s42, s43, s44, s45, s46, s47, s48, s49, s50, s51, s52, s53, s54, s55, s56, s57, s58, s59, s60, s61, s62, s63, s64, s65, s66, s67)
#define BD_HALF_B BD_HALF(B, A, s68, s69, s70, s71, s72, s73, s74, s75, s76, s77, s78, s79, s80, s81, s82, s83, s84, s85, s86, s87, s88, s89, s90, s91, s92, s93, s94, s95, s96, s97, s98, s99)

#define BD_CLEAR \
    "v_mov_b32 v28, 0\n\tv_mov_b32 v29, 0\n\tv_mov_b32 v30, 0\n\tv_mov_b32 v31, 0\n\tv_mov_b32 v32, 0\n\tv_mov_b32 v33, 0\n\tv_mov_b32 v34, 0\n\tv_mov_b32 v35, 0\n\tv_mov_b32 v36, 0\n\tv_mov_b32 v37, 0\n\t" \
    "v_mov_b32 v38, 0\n\tv_mov_b32 v39, 0\n\tv_mov_b32 v40, 0\n\tv_mov_b32 v41, 0\n\tv_mov_b32 v42, 0\n\tv_mov_b32 v43, 0\n\tv_mov_b32 v44, 0\n\tv_mov_b32 v45, 0\n\tv_mov_b32 v46, 0\n\tv_mov_b32 v47, 0\n\t" \
    "v_mov_b32 v48, 0\n\tv_mov_b32 v49, 0\n\tv_mov_b32 v50, 0\n\tv_mov_b32 v51, 0\n\tv_mov_b32 v52, 0\n\tv_mov_b32 v53, 0\n\tv_mov_b32 v54, 0\n\tv_mov_b32 v55, 0\n\tv_mov_b32 v56, 0\n\tv_mov_b32 v57, 0\n\t" \
    "v_mov_b32 v58, 0\n\tv_mov_b32 v59, 0\n\tv_mov_b32 v60, 0\n\tv_mov_b32 v61, 0\n\tv_mov_b32 v62, 0\n\tv_mov_b32 v63, 0\n\tv_mov_b32 v64, 0\n\tv_mov_b32 v65, 0\n\tv_mov_b32 v66, 0\n\tv_mov_b32 v67, 0\n\t" \
    "v_mov_b32 v68, 0\n\tv_mov_b32 v69, 0\n\tv_mov_b32 v70, 0\n\tv_mov_b32 v71, 0\n\tv_mov_b32 v72, 0\n\tv_mov_b32 v73, 0\n\tv_mov_b32 v74, 0\n\tv_mov_b32 v75, 0\n\tv_mov_b32 v76, 0\n\tv_mov_b32 v77, 0\n\t" \
    "v_mov_b32 v78, 0\n\tv_mov_b32 v79, 0\n\tv_mov_b32 v80, 0\n\tv_mov_b32 v81, 0\n\tv_mov_b32 v82, 0\n\tv_mov_b32 v83, 0\n\tv_mov_b32 v84, 0\n\tv_mov_b32 v85, 0\n\tv_mov_b32 v86, 0\n\tv_mov_b32 v87, 0\n\t" \
    "v_mov_b32 v88, 0\n\tv_mov_b32 v89, 0\n\tv_mov_b32 v90, 0\n\tv_mov_b32 v91, 0\n\tv_mov_b32 v92, 0\n\tv_mov_b32 v93, 0\n\tv_mov_b32 v94, 0\n\tv_mov_b32 v95, 0\n\tv_mov_b32 v96, 0\n\tv_mov_b32 v97, 0\n\t" \
    "v_mov_b32 v98, 0\n\tv_mov_b32 v99, 0\n\tv_mov_b32 v100, 0\n\tv_mov_b32 v101, 0\n\tv_mov_b32 v102, 0\n\tv_mov_b32 v103, 0\n\tv_mov_b32 v104, 0\n\tv_mov_b32 v105, 0\n\tv_mov_b32 v106, 0\n\tv_mov_b32 v107, 0\n\t" \
    "v_mov_b32 v108, 0\n\tv_mov_b32 v109, 0\n\tv_mov_b32 v110, 0\n\tv_mov_b32 v111, 0\n\tv_mov_b32 v112, 0\n\tv_mov_b32 v113, 0\n\tv_mov_b32 v114, 0\n\tv_mov_b32 v115, 0\n\tv_mov_b32 v116, 0\n\tv_mov_b32 v117, 0\n\t" \
    "v_mov_b32 v118, 0\n\tv_mov_b32 v119, 0\n\tv_mov_b32 v120, 0\n\tv_mov_b32 v121, 0\n\tv_mov_b32 v122, 0\n\tv_mov_b32 v123, 0\n\tv_mov_b32 v124, 0\n\tv_mov_b32 v125, 0\n\tv_mov_b32 v126, 0\n\tv_mov_b32 v127, 0\n\t"

#define BD_MAIN                                                                                         \
    asm volatile(                                                                                       \
        BD_CLEAR                                                                                        \
        "s_cmp_eq_u32 %[nb], 0\n\ts_cbranch_scc1 .Lbd_done_%=\n\t"                                   \
        BD_BEGIN                                                                                        \
        "s_mov_b32 s12, 0x60\n\t"                                                                       \
        "s_mov_b32 s13, 0\n\t"                                                                          \
        "s_mov_b64 vcc, 0\n\t"                                                                          \
        "s_sub_u32 s15, %[nb], 1\n\t"                                                                   \
        "s_load_dwordx8 s[16:23], %[head], 0x0\n\t"                                                     \
        "s_load_dwordx8 s[24:31], %[head], 0x40\n\t"                                                    \
        BD_LOAD_A                                                                                       \
        "s_waitcnt lgkmcnt(0)\n\t"                                                                      \
        "s_mov_b32 s14, %[fillw]\n\t"                                                                   \
        BD_FILL_BAND                                                                                    \
        "s_sub_u32 s14, %[flip], s14\n\t"                                                               \
        "s_load_dwordx8 s[16:23], %[head], 0x20\n\t"                                                    \
        BD_WAIT_BAND                                                                                    \
        BD_LOAD_B                                                                                       \
        "s_barrier\n\t"                                                                                 \
        "s_branch .Lbd_band_A_%=\n\t"                                                                   \
        /* (where the loop lies in the cache lines of the instructions makes up to 1 %: the same place in every build, 36 bytes behind a multiple of 256, so that no change in \
           front of it moves it; 14000 x 14000, 2 %: 3167 - 3177 us so, 3194 - 3201 without any alignment, as at multiples of 32; 8000 x 8000, 10 %: 2285 - 2295 and 2303 - 2310) */ \
        ".p2align 8\n.fill 9, 4, 0xbf800000\n"                                                           \
        BD_HALF_A                                                                                       \
        BD_HALF_B                                                                                       \
        /* the rows requested for the bands beyond the last one arrive before the wave gives up its LDS */ \
        ".Lbd_done_%=:\n\t"                                                                             \
        "s_waitcnt vmcnt(0) lgkmcnt(0)\n\t" \
        : "={v[28:31]}"(acc.t0), "={v[32:63]}"(acc.t1), "={v[64:95]}"(acc.t2), "={v[96:127]}"(acc.t3), "+{v0}"(lane_at), [fillw] "+s"(fillw) \
        : [head] "s"(head), [units] "s"(units), [nb] "s"(nb), [ldb4] "s"(ldb4), [flip] "s"(flip), "{s[32:35]}"(rsrc), "{v2}"(lane_b) \
        : "m0", "scc", "vcc", "memory",  \
          "v1", "v3", "v4", "v5", "v6", "v7", "v8", "v9", "v10", "v11", "v12", "v13", "v14", "v15", "v16", "v17", "v18", "v19",  \
          "v20", "v21", "v22", "v23", "v24", "v25", "v26", "v27", "s12", "s13", "s14", "s15", "s16", "s17", "s18", "s19", "s20",  \
          "s21", "s22", "s23", "s24", "s25", "s26", "s27", "s28", "s29", "s30", "s31", "s36", "s37", "s38", "s39", "s40", "s41",  \
          "s42", "s43", "s44", "s45", "s46", "s47", "s48", "s49", "s50", "s51", "s52", "s53", "s54", "s55", "s56", "s57", "s58",  \
          "s59", "s60", "s61", "s62", "s63", "s64", "s65", "s66", "s67", "s68", "s69", "s70", "s71", "s72", "s73", "s74", "s75",  \
          "s76", "s77", "s78", "s79", "s80", "s81", "s82", "s83", "s84", "s85", "s86", "s87", "s88", "s89", "s90", "s91", "s92",  \
          "s93", "s94", "s95", "s96", "s97", "s98", "s99" BD_MORE_SCALARS)

// How the launch works row by row instead (rows_all()), by tiles of 64 columns.
struct BandRowsGrid { int32_t tiles, rpw, wave_row; };

// A matrix with a list of far more entries than the others (take_rows and band_mark say so on the device, where the
// row lengths are) has no schedule: the waves would wait for that list in every band.  Its rows are multiplied one by one, by the
// workgroups of this launch.
template <int V, bool SPREAD, bool LATE>            // V = 4: the wide cut, 2: the tall one; when the rows of the next band are requested
__global__ __launch_bounds__(64 * kBandWaves) void spdm_band(BandArgs a, RowsArgs by_rows, BandRowsGrid rg)
{
    static_assert(V == 4 || !(SPREAD && LATE), "");
    extern __shared__ __attribute__((aligned(16))) uint32_t band_smem[];
    if (*a.uneven != 0u) {
        rows_all<16>(by_rows, rg.tiles, rg.rpw, rg.wave_row, *reinterpret_cast<RowsAllLds*>(band_smem));
        return;
    }
    // XCD-aware order: XCD x walks the contiguous slice [x*per, (x+1)*per) of the tile-major list, so the blocks that run on
    // it together read the same column tile of B.
    const int32_t per = (int32_t)(a.grid >> 3);
    const int32_t item = (int32_t)(blockIdx.x & 7u) * per + (int32_t)(blockIdx.x >> 3);
    if (item >= a.total || (int32_t)(blockIdx.x >> 3) >= per) return;    // the whole workgroup
    const int32_t tile = item / a.blocks, Q = item - tile * a.blocks;
    // the last tile of a B that is no multiple of a tile wide begins where it can hold a whole one
    constexpr int32_t kTile = BandCut<V>::kTile;
    const int32_t n = (int32_t)a.N, j0 = tile * kTile, jb = j0 > n - kTile && n >= kTile ? n - kTile : j0;

    BandAcc acc;
    uint32_t lane_at = (threadIdx.x & 63u) * (4u * V);           // the lane's columns in a row of B in LDS
    uint32_t fillw = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * (uint32_t)kBandFillBytes;       // the wave's rows inside a band buffer
    const int32_t nb = (__builtin_amdgcn_readfirstlane(a.count[Q]) + BandCut<V>::kRows - 1) / BandCut<V>::kRows;
    {
        const int64_t list = (int64_t)Q * kBandWaves + fillw / (uint32_t)kBandFillBytes;
        const uint32_t* head = a.head + list * a.head_stride * kBandHeadWords;
        const uint32_t* units = a.units + (int64_t)__builtin_amdgcn_readfirstlane(a.first[list]) * kBandUnitWords;
        // B from the tile's first column on; a load outside it would return zero
        const uint64_t bt = (uint64_t)(a.B + jb), bytes = (uint64_t)(a.k - 1) * (uint64_t)a.ldb * 4u + (uint64_t)(n - jb) * 4u;
        const band_u32x4 rsrc = {(uint32_t)bt, (uint32_t)(bt >> 32) & 0xffffu, (uint32_t)bytes, 0x00027000u};
        const uint32_t flip = 2u * fillw + kBandBufferBytes;
        const uint32_t ldb4 = (uint32_t)a.ldb * 4u;                // the launcher checks that every row offset fits 32 bits
#define BD_WAIT_BAND "s_waitcnt vmcnt(0) lgkmcnt(0)\n\t"
        // the lane's byte offset in what a request fetches; lanes beyond N fetch the first columns of the tile
        const uint32_t lane = threadIdx.x & 63u;
        if constexpr (V == 4) {
#define BD_FMAC_T0(val) BD_FMAC_WIDE(val, v4, v5, v6, v7)
#define BD_FMAC_T1(val) BD_FMAC_WIDE(val, v8, v9, v10, v11)
#define BD_FMAC_T2(val) BD_FMAC_WIDE(val, v12, v13, v14, v15)
#define BD_FMAC_T3(val) BD_FMAC_WIDE(val, v16, v17, v18, v19)
#define BD_FMAC_T4(val) BD_FMAC_WIDE(val, v20, v21, v22, v23)
#define BD_FMAC_T5(val) BD_FMAC_WIDE(val, v24, v25, v26, v27)
#define BD_READ_T0(meta) BD_READ_WIDE(meta, "v[4:7]")
#define BD_READ_T1(meta) BD_READ_WIDE(meta, "v[8:11]")
#define BD_READ_T2(meta) BD_READ_WIDE(meta, "v[12:15]")
#define BD_READ_T3(meta) BD_READ_WIDE(meta, "v[16:19]")
#define BD_READ_T4(meta) BD_READ_WIDE(meta, "v[20:23]")
#define BD_READ_T5(meta) BD_READ_WIDE(meta, "v[24:27]")
#define BD_BEGIN "v_mov_b32 v1, 0x3fc00\n\t"
#define BD_MORE_SCALARS
#define BD_FILL BD_FILL_WIDE
            const uint32_t lane_b = jb + (int32_t)(lane * 4u) < n ? lane * 16u : 0u;
#define BD_LOAD_ROW "buffer_load_dwordx4 v2, s[32:35], s23 offen lds\n\t"
            if constexpr (SPREAD && !LATE) {
#define BD_ASK_START BD_SPREAD_START
#define BD_ASK_STEP BD_SPREAD_STEP
#define BD_ASK_UNIT BD_SPREAD_UNIT
#define BD_ASK_REST BD_SPREAD_REST
                BD_MAIN;
#undef BD_ASK_START
#undef BD_ASK_STEP
#undef BD_ASK_UNIT
#undef BD_ASK_REST
            } else if constexpr (SPREAD) {
#define BD_ASK_START BD_FIRST_START
#define BD_ASK_STEP BD_STEP1_STEP
#define BD_ASK_UNIT BD_STEP1_UNIT
#define BD_ASK_REST BD_STEP1_REST
                BD_MAIN;
#undef BD_ASK_START
#undef BD_ASK_STEP
#undef BD_ASK_UNIT
#undef BD_ASK_REST
            } else if constexpr (LATE) {
#define BD_ASK_START BD_SECOND_START
#define BD_ASK_STEP BD_HALVES_STEP
#define BD_ASK_UNIT BD_HALVES_UNIT
#define BD_ASK_REST BD_SECOND_REST
                BD_MAIN;
#undef BD_ASK_START
#undef BD_ASK_STEP
#undef BD_ASK_UNIT
#undef BD_ASK_REST
            } else {
#define BD_ASK_START BD_FIRST_START
#define BD_ASK_STEP BD_HALVES_STEP
#define BD_ASK_UNIT BD_HALVES_UNIT
#define BD_ASK_REST BD_FIRST_REST
                BD_MAIN;
#undef BD_ASK_START
#undef BD_ASK_STEP
#undef BD_ASK_UNIT
#undef BD_ASK_REST
            }
#undef BD_LOAD_ROW
#undef BD_FILL
#undef BD_MORE_SCALARS
#undef BD_BEGIN
#undef BD_FMAC_T0
#undef BD_READ_T0
#undef BD_FMAC_T1
#undef BD_READ_T1
#undef BD_FMAC_T2
#undef BD_READ_T2
#undef BD_FMAC_T3
#undef BD_READ_T3
#undef BD_FMAC_T4
#undef BD_READ_T4
#undef BD_FMAC_T5
#undef BD_READ_T5
        } else {
#define BD_FMAC_T0(val) BD_FMAC_TALL(val, v4, v5)
#define BD_FMAC_T1(val) BD_FMAC_TALL(val, v6, v7)
#define BD_FMAC_T2(val) BD_FMAC_TALL(val, v8, v9)
#define BD_FMAC_T3(val) BD_FMAC_TALL(val, v10, v11)
#define BD_FMAC_T4(val) BD_FMAC_TALL(val, v12, v13)
#define BD_FMAC_T5(val) BD_FMAC_TALL(val, v14, v15)
#define BD_READ_T0(meta) BD_READ_TALL(meta, "v[4:5]")
#define BD_READ_T1(meta) BD_READ_TALL(meta, "v[6:7]")
#define BD_READ_T2(meta) BD_READ_TALL(meta, "v[8:9]")
#define BD_READ_T3(meta) BD_READ_TALL(meta, "v[10:11]")
#define BD_READ_T4(meta) BD_READ_TALL(meta, "v[12:13]")
#define BD_READ_T5(meta) BD_READ_TALL(meta, "v[14:15]")
#define BD_BEGIN "v_mov_b32 v1, 0x3fe00\n\tv_bfe_i32 v127, v0, 8, 1\n\t"
#define BD_MORE_SCALARS , "s100"
            const uint32_t lane_b = jb + (int32_t)((lane & 31u) * 4u) < n ? (lane & 31u) * 16u : 0u;
#define BD_FILL BD_FILL_TALL
            if constexpr (SPREAD) {
#define BD_ASK_START BD_SPREAD_START
#define BD_ASK_STEP BD_SPREAD_STEP
#define BD_ASK_UNIT BD_SPREAD_UNIT
#define BD_ASK_REST BD_SPREAD_REST
                BD_MAIN;
#undef BD_ASK_START
#undef BD_ASK_STEP
#undef BD_ASK_UNIT
#undef BD_ASK_REST
            } else if constexpr (LATE) {
#define BD_ASK_START BD_SECOND_START
#define BD_ASK_STEP BD_HALVES_STEP
#define BD_ASK_UNIT BD_HALVES_UNIT
#define BD_ASK_REST BD_SECOND_REST
                BD_MAIN;
#undef BD_ASK_START
#undef BD_ASK_STEP
#undef BD_ASK_UNIT
#undef BD_ASK_REST
            } else {
#define BD_ASK_START BD_FIRST_START
#define BD_ASK_STEP BD_HALVES_STEP
#define BD_ASK_UNIT BD_HALVES_UNIT
#define BD_ASK_REST BD_FIRST_REST
                BD_MAIN;
#undef BD_ASK_START
#undef BD_ASK_STEP
#undef BD_ASK_UNIT
#undef BD_ASK_REST
            }
#undef BD_FILL
#undef BD_MORE_SCALARS
#undef BD_BEGIN
#undef BD_FMAC_T0
#undef BD_READ_T0
#undef BD_FMAC_T1
#undef BD_READ_T1
#undef BD_FMAC_T2
#undef BD_READ_T2
#undef BD_FMAC_T3
#undef BD_READ_T3
#undef BD_FMAC_T4
#undef BD_READ_T4
#undef BD_FMAC_T5
#undef BD_READ_T5
        }
#undef BD_WAIT_BAND
    }

    // What the stores need is made again from the kernel's arguments: the loop leaves the compiler no vector register and eighteen
    // scalar ones, too few to carry it across.
    typedef const __attribute__((address_space(4))) char* arg_ptr;
    arg_ptr args = (arg_ptr)__builtin_amdgcn_kernarg_segment_ptr();
    uint32_t bid = blockIdx.x;
    asm volatile("" : "+s"(args), "+s"(bid));
    const __attribute__((address_space(4))) BandArgs* z = (const __attribute__((address_space(4))) BandArgs*)args;
    const int32_t item2 = (int32_t)(bid & 7u) * (int32_t)(z->grid >> 3) + (int32_t)(bid >> 3);
    const int32_t tile2 = item2 / z->blocks, Q2 = item2 - tile2 * z->blocks;
    const int32_t N = (int32_t)z->N, first = tile2 * kTile, base = first > N - kTile && N >= kTile ? N - kTile : first;
    const int32_t jc = base + (int32_t)(lane_at >> 2);             // the lane's first column; it stores those from `first` on
    if (jc + V > first && jc < N) {
        const int own = first > jc ? first - jc : 0;
        const int32_t h = z->h;
        const int64_t row0 = ((int64_t)Q2 * kBandWaves + fillw / (uint32_t)kBandFillBytes) * h, ldc = z->ldc;
        const int64_t rows = z->m - row0 < h ? z->m - row0 : h;
        float* __restrict__ dst = z->C + jc + row0 * ldc;
        constexpr int kStride = BandCut<V>::kMaxH + 1;
        typedef float vec __attribute__((ext_vector_type(V), aligned(4)));         // rows of C are aligned to 4 bytes only
#pragma unroll
        for (int r = 0; r < BandCut<V>::kMaxH; ++r) {
            if (r < rows) {
                vec o;
#pragma unroll
                for (int v = 0; v < V; ++v) o[v] = band_acc_get(acc, v * kStride + r);
                if (own == 0) {
                    __builtin_nontemporal_store(o, reinterpret_cast<vec*>(dst));
                } else {
#pragma unroll
                    for (int v = 1; v < V; ++v)
                        if (v >= own) __builtin_nontemporal_store(o[v], dst + v);
                }
            }
            dst += ldc;
        }
    }
}

}  // namespace gcoo
