// interp_gfx950.h -- handler tables of the threaded interpreter (threaded.h
// has the word format and the reasons), in gfx950 assembly.
//
// Registers (fixed; the caller's asm statement lists them all):
//   s[84:85] code of the program   s86 byte offset of the word after next
//   s[88:89] next word             s[90:91] table       s[92:93] jump target
//   s[94:95] return address        s87 resume offset    s83 result code
//   s82 staged cases / 256 (the scale of a row's byte offset)
//   s[68:75] compare masks         s[96:98] scratch     vcc, m0
//   v22..v25 constants             v31 LDS address of the lane's first case
//   v4..v18 temporaries (v4..v7 carry values to and from the caller, v12..v15
//   a second operand to it)
//   v36..v67 stack cells, K registers each (case j of cell i: v[36 + K i + j])
// A handler takes its payload (s89), loads the next word into s[88:89] and
// ends in GP_NEXT.  Temporaries and cells of one case sit in different
// register banks (number mod 4), so three-operand forms read without a
// conflict.
//
// Wait states (gfx940 and later): one instruction between a transcendental
// instruction and a user of its result, two between a compare's mask and the
// select that reads it, four between v_div_scale's vcc and v_div_fmas.  Other
// cases' instructions lie between where there are enough cases.
//
// Hot and cold code: the handlers that ordinary values take lie together;
// range checks that failed, the forms for any operand and the commands beyond
// the benchmark set lie in the cold blocks.  With both interleaved in blocks of
// a power of two, and eight cases per lane, the 100,000-program call missed the
// instruction cache 2.3 million times, now 0.5.
//
// Values outside a fast range (sin and cos beyond 2^17, exp beyond 87, square
// roots of magnitudes below 2^-100) and the library commands: the handler
// hands the top's K values to the caller (result code kCall...), which
// applies the out-of-line function and resumes at the block's finish code.
#pragma once

// (the tables are text of their own section: the function only carries them)
__device__ __attribute__((used, noinline)) void gp_threads_tables()
{
#ifdef __HIP_DEVICE_COMPILE__
asm volatile(R"(
.pushsection .text.gp_threads,"ax",@progbits
.set GP_CB, 36

.macro GP_LOADNEXT last
 .if !\last
  s_load_dwordx2 s[88:89], s[84:85], s86
  s_add_u32 s86, s86, 8
 .endif
.endm
// (lgkmcnt must be zero)
.macro GP_JUMP last
 .if \last
  s_mov_b32 s83, 0
  s_setpc_b64 s[94:95]
 .else
  s_add_u32 s92, s90, s88
  s_addc_u32 s93, s91, 0
  s_setpc_b64 s[92:93]
 .endif
.endm
.macro GP_NEXT last
  s_waitcnt lgkmcnt(0)
  GP_JUMP \last
.endm

// cell \c = the input row at payload offset s89
.macro GP_ROW K, c
  s_mul_i32 s89, s89, s82
  v_add_u32_e32 v4, s89, v31
 .if \K == 1
  ds_read_b32 v[GP_CB+\c], v4
 .else
  ds_read2st64_b32 v[GP_CB+\K*\c:GP_CB+\K*\c+1], v4 offset0:0 offset1:1
 .if \K == 4
  ds_read2st64_b32 v[GP_CB+4*\c+2:GP_CB+4*\c+3], v4 offset0:2 offset1:3
 .endif
 .endif
.endm
// cell \c = the constant s89
.macro GP_CONST_CELL K, c
  v_mov_b32_e32 v[GP_CB+\K*\c], s89
 .irp j,1,2,3
 .if \j < \K
  v_mov_b32_e32 v[GP_CB+\K*\c+\j], v[GP_CB+\K*\c]
 .endif
 .endr
.endm
// cell \d = cell \s
.macro GP_COPY_CELL K, d, s
 .irp j,0,1,2,3
 .if \j < \K
  v_mov_b32_e32 v[GP_CB+\K*\d+\j], v[GP_CB+\K*\s+\j]
 .endif
 .endr
.endm
// v\r = the largest (op max) or smallest (min) magnitude of cell \c
.macro GP_MAGNITUDE K, c, op, r
 .if \K == 1
  v_\op\()_f32_e64 v\r, |v[GP_CB+\c]|, |v[GP_CB+\c]|
 .elseif \K == 2
  v_\op\()_f32_e64 v\r, |v[GP_CB+2*\c]|, |v[GP_CB+2*\c+1]|
 .else
  v_\op\()3_f32 v\r, |v[GP_CB+4*\c]|, |v[GP_CB+4*\c+1]|, |v[GP_CB+4*\c+2]|
  v_\op\()_f32_e64 v\r, v\r, |v[GP_CB+4*\c+3]|
 .endif
.endm
// vcc = the magnitudes of cell \c may pass \limit, or hold a NaN: the sum of
// the magnitudes against it (adds issue twice as fast as maxima)
.macro GP_SUMTEST K, c, limit
 .if \K == 1
  v_and_b32_e32 v4, 0x7fffffff, v[GP_CB+\c]
 .else
  v_add_f32_e64 v4, |v[GP_CB+\K*\c]|, |v[GP_CB+\K*\c+1]|
 .if \K == 4
  v_add_f32_e64 v5, |v[GP_CB+4*\c+2]|, |v[GP_CB+4*\c+3]|
  v_add_f32_e32 v4, v4, v5
 .endif
 .endif
  v_cmp_nge_f32_e32 vcc, \limit, v4
.endm
// Each operator over the K cases.
// sin after t (v4..v7) and k (v8..v11) are set: reduction by three parts of
// pi, odd polynomial, sign flip by t's low bit
.macro GP_SINBODY K, c
 .irp j,0,1,2,3
 .if \j < \K
  v_fmac_f32_e32 v[GP_CB+\K*\c+\j], 0xc0490fdb, v[8+((\j+1)&3)]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_fmac_f32_e32 v[GP_CB+\K*\c+\j], 0x33bbbd2e, v[8+((\j+1)&3)]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_fmac_f32_e32 v[GP_CB+\K*\c+\j], 0x27772ced, v[8+((\j+1)&3)]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_mul_f32_e32 v[8+((\j+1)&3)], v[GP_CB+\K*\c+\j], v[GP_CB+\K*\c+\j]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_fmaak_f32 v[12+((\j+2)&3)], v[8+((\j+1)&3)], v23, 0xb94fb78c
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_fmaak_f32 v[12+((\j+2)&3)], v[8+((\j+1)&3)], v[12+((\j+2)&3)], 0x3c08876a
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_fmaak_f32 v[12+((\j+2)&3)], v[8+((\j+1)&3)], v[12+((\j+2)&3)], 0xbe2aaaa6
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_mul_f32_e32 v[8+((\j+1)&3)], v[GP_CB+\K*\c+\j], v[8+((\j+1)&3)]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_fmac_f32_e32 v[GP_CB+\K*\c+\j], v[8+((\j+1)&3)], v[12+((\j+2)&3)]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_lshl_add_u32 v[GP_CB+\K*\c+\j], v[4+((\j+3)&3)], 31, v[GP_CB+\K*\c+\j]
 .endif
 .endr
.endm
.macro GP_SIN K, c
 .irp j,0,1,2,3
 .if \j < \K
  v_fmaak_f32 v[4+((\j+3)&3)], v[GP_CB+\K*\c+\j], v22, 0x4b400000
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_add_f32_e32 v[8+((\j+1)&3)], 0xcb400000, v[4+((\j+3)&3)]
 .endif
 .endr
  GP_SINBODY \K, \c
.endm
.macro GP_COS K, c
 .irp j,0,1,2,3
 .if \j < \K
  v_fma_f32 v[4+((\j+3)&3)], v[GP_CB+\K*\c+\j], v22, -0.5
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_add_f32_e32 v[4+((\j+3)&3)], 0x4b400001, v[4+((\j+3)&3)]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_add_f32_e32 v[8+((\j+1)&3)], 0xcb400001, v[4+((\j+3)&3)]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_add_f32_e32 v[8+((\j+1)&3)], 0.5, v[8+((\j+1)&3)]
 .endif
 .endr
  GP_SINBODY \K, \c
.endm
// exp: 2^n through the exponent field, t = h + 1.5 * 2^23 holds n in its low
// bits (no NaN comes here: its low bits could be anything)
.macro GP_EXP K, c
 .irp j,0,1,2,3
 .if \j < \K
  v_mul_f32_e32 v[8+((\j+1)&3)], 0x3fb8aa3b, v[GP_CB+\K*\c+\j]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_fma_f32 v[12+((\j+2)&3)], v[GP_CB+\K*\c+\j], v24, -v[8+((\j+1)&3)]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_add_f32_e32 v[4+((\j+3)&3)], 0x4b400000, v[8+((\j+1)&3)]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_fmac_f32_e32 v[12+((\j+2)&3)], 0x32a57060, v[GP_CB+\K*\c+\j]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_add_f32_e32 v[GP_CB+\K*\c+\j], 0xcb400000, v[4+((\j+3)&3)]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_sub_f32_e32 v[8+((\j+1)&3)], v[8+((\j+1)&3)], v[GP_CB+\K*\c+\j]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_add_f32_e32 v[8+((\j+1)&3)], v[8+((\j+1)&3)], v[12+((\j+2)&3)]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_exp_f32_e32 v[8+((\j+1)&3)], v[8+((\j+1)&3)]
 .endif
 .endr
 .if \K == 1
  s_nop 0
 .endif
 .irp j,0,1,2,3
 .if \j < \K
  v_lshl_add_u32 v[GP_CB+\K*\c+\j], v[4+((\j+3)&3)], 23, v[8+((\j+1)&3)]
 .endif
 .endr
.endm
// ln |value|
.macro GP_LOG K, c
 .irp j,0,1,2,3
 .if \j < \K
  v_log_f32_e64 v[4+((\j+3)&3)], |v[GP_CB+\K*\c+\j]|
 .endif
 .endr
 .if \K == 1
  s_nop 0
 .endif
 .irp j,0,1,2,3
 .if \j < \K
  v_mul_f32_e32 v[GP_CB+\K*\c+\j], 0x3377d1cf, v[4+((\j+3)&3)]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_fmac_f32_e32 v[GP_CB+\K*\c+\j], 0x3f317217, v[4+((\j+3)&3)]
 .endif
 .endr
.endm
// the same with the protected range: 0 where |value| <= 0.001
.macro GP_LOGP K, c
 .irp j,0,1,2,3
 .if \j < \K
  v_log_f32_e64 v[4+((\j+3)&3)], |v[GP_CB+\K*\c+\j]|
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_cmp_nle_f32_e64 s[68+2*\j:69+2*\j], |v[GP_CB+\K*\c+\j]|, v25
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_mul_f32_e32 v[8+((\j+1)&3)], 0x3377d1cf, v[4+((\j+3)&3)]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_fmac_f32_e32 v[8+((\j+1)&3)], 0x3f317217, v[4+((\j+3)&3)]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_cndmask_b32_e64 v[GP_CB+\K*\c+\j], 0, v[8+((\j+1)&3)], s[68+2*\j:69+2*\j]
 .endif
 .endr
.endm
// cell \a = cell \a / cell \a+1 inside the range of GP_DIVRANGE: reciprocal, one
// Newton step, quotient, one residual correction.  Inside the range no step
// overflows, no residual is denormal, and the reciprocal scales exactly with its
// operand's exponent, so the quotient's rounding depends on the significands
// alone.  It is the IEEE quotient: found once for every pair of significands (2^46)
// on an MI355X by comparing the residual a - b q with half a unit in the last
// place of q; the tests cover every divisor significand under seven dividends and
// 2^23 random pairs six times over.  (The general form: 50 clocks of vector
// issue per case; this one: 20, and 6 for the range.)
.macro GP_DIV K, a
 .irp j,0,1,2,3
 .if \j < \K
  v_rcp_f32_e32 v[8+((\j+1)&3)], v[GP_CB+\K*(\a+1)+\j]
 .endif
 .endr
 .if \K == 1
  s_nop 0
 .endif
 .irp j,0,1,2,3
 .if \j < \K
  v_fma_f32 v[12+((\j+2)&3)], -v[GP_CB+\K*(\a+1)+\j], v[8+((\j+1)&3)], 1.0
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_fmac_f32_e32 v[8+((\j+1)&3)], v[12+((\j+2)&3)], v[8+((\j+1)&3)]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_mul_f32_e32 v[4+((\j+3)&3)], v[GP_CB+\K*\a+\j], v[8+((\j+1)&3)]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_fma_f32 v[12+((\j+2)&3)], -v[GP_CB+\K*(\a+1)+\j], v[4+((\j+3)&3)], v[GP_CB+\K*\a+\j]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_fma_f32 v[GP_CB+\K*\a+\j], v[12+((\j+2)&3)], v[8+((\j+1)&3)], v[4+((\j+3)&3)]
 .endif
 .endr
.endm
// cell \a = cell \a+1 / cell \a
.macro GP_DIVR K, a
 .irp j,0,1,2,3
 .if \j < \K
  v_rcp_f32_e32 v[8+((\j+1)&3)], v[GP_CB+\K*\a+\j]
 .endif
 .endr
 .if \K == 1
  s_nop 0
 .endif
 .irp j,0,1,2,3
 .if \j < \K
  v_fma_f32 v[12+((\j+2)&3)], -v[GP_CB+\K*\a+\j], v[8+((\j+1)&3)], 1.0
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_fmac_f32_e32 v[8+((\j+1)&3)], v[12+((\j+2)&3)], v[8+((\j+1)&3)]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_mul_f32_e32 v[4+((\j+3)&3)], v[GP_CB+\K*(\a+1)+\j], v[8+((\j+1)&3)]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_fma_f32 v[12+((\j+2)&3)], -v[GP_CB+\K*\a+\j], v[4+((\j+3)&3)], v[GP_CB+\K*(\a+1)+\j]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_fma_f32 v[GP_CB+\K*\a+\j], v[12+((\j+2)&3)], v[8+((\j+1)&3)], v[4+((\j+3)&3)]
 .endif
 .endr
.endm
// cell \r = cell \n / cell \d, any operands: the IEEE quotient (scaled reciprocal, one Newton step, two
// residual corrections, fix-up), 1 where |divisor| <= 0.001
.macro GP_DIVP K, n, d, r
 .irp j,0,1,2,3
 .if \j < \K
  v_div_scale_f32 v[4+((\j+3)&3)], s[96:97], v[GP_CB+\K*\d+\j], v[GP_CB+\K*\d+\j], v[GP_CB+\K*\n+\j]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_rcp_f32_e32 v[8+((\j+1)&3)], v[4+((\j+3)&3)]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_cmp_nle_f32_e64 s[68+2*\j:69+2*\j], |v[GP_CB+\K*\d+\j]|, v25
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_fma_f32 v[12+((\j+2)&3)], -v[4+((\j+3)&3)], v[8+((\j+1)&3)], 1.0
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_fmac_f32_e32 v[8+((\j+1)&3)], v[12+((\j+2)&3)], v[8+((\j+1)&3)]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_div_scale_f32 v16, vcc, v[GP_CB+\K*\n+\j], v[GP_CB+\K*\d+\j], v[GP_CB+\K*\n+\j]
  v_mul_f32_e32 v17, v16, v[8+((\j+1)&3)]
  v_fma_f32 v18, -v[4+((\j+3)&3)], v17, v16
  v_fmac_f32_e32 v17, v18, v[8+((\j+1)&3)]
  v_fma_f32 v18, -v[4+((\j+3)&3)], v17, v16
  v_div_fmas_f32 v[12+((\j+2)&3)], v18, v[8+((\j+1)&3)], v17
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_div_fixup_f32 v[12+((\j+2)&3)], v[12+((\j+2)&3)], v[GP_CB+\K*\d+\j], v[GP_CB+\K*\n+\j]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_cndmask_b32_e64 v[GP_CB+\K*\r+\j], 1.0, v[12+((\j+2)&3)], s[68+2*\j:69+2*\j]
 .endif
 .endr
.endm
// beyond the benchmark set: a cube formed in 64 bits, the square root with NaN
// below zero
.macro GP_CUBE K, c
 .irp j,0,1,2,3
 .if \j < \K
  v_cvt_f64_f32_e32 v[4:5], v[GP_CB+\K*\c+\j]
  v_mul_f64 v[6:7], v[4:5], v[4:5]
  v_mul_f64 v[6:7], v[6:7], v[4:5]
  v_cvt_f32_f64_e32 v[GP_CB+\K*\c+\j], v[6:7]
 .endif
 .endr
.endm
.macro GP_SQRTRAW K, c
 .irp j,0,1,2,3
 .if \j < \K
  v_sqrt_f32_e64 v[4+((\j+3)&3)], |v[GP_CB+\K*\c+\j]|
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_cmp_ngt_f32_e64 s[68+2*\j:69+2*\j], 0, v[GP_CB+\K*\c+\j]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_mov_b32_e32 v[8+((\j+1)&3)], 0x7fc00000
 .endif
 .endr
 .if \K == 1
  s_nop 0
 .endif
 .irp j,0,1,2,3
 .if \j < \K
  v_cndmask_b32_e64 v[GP_CB+\K*\c+\j], v[8+((\j+1)&3)], v[4+((\j+3)&3)], s[68+2*\j:69+2*\j]
 .endif
 .endr
.endm
.macro GP_ALL2 op, K, dst, s0, s1
 .irp j,0,1,2,3
 .if \j < \K
  \op v[GP_CB+\K*\dst+\j], v[GP_CB+\K*\s0+\j], v[GP_CB+\K*\s1+\j]
 .endif
 .endr
.endm
// The handlers of block \blk whose instruction starts with \d elements (a
// binary operator's cells start at \a, a unary's or leaf operand's top is
// cell \c); \last: the forms that end a program.  \target: the block one
// element deeper, whose operators a fused leaf runs on.  (Of two NaN operands
// the first decides the result's sign: the top is the first source of + and
// *, a constant the first of all.)
.macro GP_PUSHES tab, K, blk, d, last
 .org \tab + 81600 + 3776*(\blk) + 0
  GP_CONST_CELL \K, \d
  GP_LOADNEXT \last
  GP_NEXT \last
 .org \tab + 81600 + 3776*(\blk) + 64
  GP_ROW \K, \d
  GP_LOADNEXT \last
  GP_NEXT \last
.endm
// vcc / branch to the cold division unless every |operand| <= 2^60, every
// |dividend| > 2^-60 and every |divisor| > 0.001 (then nothing overflows, no
// step is denormal and no case is protected)
.macro GP_DIVRANGE tab, K, blk, a, num, den, cold
 .if \K == 4
  v_max3_f32 v4, |v[GP_CB+4*\a]|, |v[GP_CB+4*\a+1]|, |v[GP_CB+4*\a+2]|
  v_max3_f32 v4, v4, |v[GP_CB+4*\a+3]|, |v[GP_CB+4*\a+4]|
  v_max3_f32 v4, v4, |v[GP_CB+4*\a+5]|, |v[GP_CB+4*\a+6]|
  v_max_f32_e64 v4, v4, |v[GP_CB+4*\a+7]|
 .elseif \K == 2
  v_max3_f32 v4, |v[GP_CB+2*\a]|, |v[GP_CB+2*\a+1]|, |v[GP_CB+2*\a+2]|
  v_max_f32_e64 v4, v4, |v[GP_CB+2*\a+3]|
 .else
  v_max_f32_e64 v4, |v[GP_CB+\a]|, |v[GP_CB+\a+1]|
 .endif
  v_cmp_nge_f32_e32 vcc, 0x5d800000, v4
  GP_MAGNITUDE \K, \num, min, 5
  s_cbranch_vccnz \tab\()_\blk\()_\cold
  GP_MAGNITUDE \K, \den, min, 6
  v_mul_f32_e32 v5, 0x5883126f, v5
  v_min_f32_e32 v5, v5, v6
  v_cmp_nlt_f32_e32 vcc, 0x3a83126f, v5
  s_cbranch_vccnz \tab\()_\blk\()_\cold
.endm
.macro GP_CELLS tab, K, blk, a, last
 .org \tab + 81600 + 3776*(\blk) + 128
  GP_LOADNEXT \last
  GP_ALL2 v_add_f32_e32, \K, \a, (\a+1), \a
  GP_NEXT \last
 .org \tab + 81600 + 3776*(\blk) + 192
  GP_LOADNEXT \last
  GP_ALL2 v_sub_f32_e32, \K, \a, \a, (\a+1)
  GP_NEXT \last
 .org \tab + 81600 + 3776*(\blk) + 256
  GP_LOADNEXT \last
  GP_ALL2 v_mul_f32_e32, \K, \a, (\a+1), \a
  GP_NEXT \last
 .org \tab + 81600 + 3776*(\blk) + 320
  GP_LOADNEXT \last
\tab\()_\blk\()_div:
  GP_DIVRANGE \tab, \K, \blk, \a, \a, (\a+1), cdiv
  GP_DIV \K, \a
  GP_NEXT \last
// top minus, top over the element below
 .org \tab + 81600 + 3776*(\blk) + 608
  GP_LOADNEXT \last
  GP_ALL2 v_sub_f32_e32, \K, \a, (\a+1), \a
  GP_NEXT \last
 .org \tab + 81600 + 3776*(\blk) + 672
  GP_LOADNEXT \last
\tab\()_\blk\()_divr:
  GP_DIVRANGE \tab, \K, \blk, \a, (\a+1), \a, cdivr
  GP_DIVR \K, \a
  GP_NEXT \last
.endm
.macro GP_CONSTOP tab, K, blk, c, last, off, op
 .org \tab + 81600 + 3776*(\blk) + 0+\off
  v_mov_b32_e32 v4, s89
  GP_LOADNEXT \last
 .irp j,0,1,2,3
 .if \j < \K
  \op v[GP_CB+\K*\c+\j], v4, v[GP_CB+\K*\c+\j]
 .endif
 .endr
  GP_NEXT \last
.endm
.macro GP_ROWOP tab, K, blk, c, last, off, op
 .org \tab + 81600 + 3776*(\blk) + 0+\off
  GP_ROW \K, (\c+1)
  GP_LOADNEXT \last
  s_waitcnt lgkmcnt(0)
  GP_ALL2 \op, \K, \c, \c, (\c+1)
  GP_JUMP \last
.endm
.macro GP_LEAFOPS tab, K, blk, c, last, target
  GP_CONSTOP \tab, \K, \blk, \c, \last, 960, v_add_f32_e32
  GP_CONSTOP \tab, \K, \blk, \c, \last, 1024, v_subrev_f32_e32
  GP_CONSTOP \tab, \K, \blk, \c, \last, 1088, v_mul_f32_e32
 .org \tab + 81600 + 3776*(\blk) + 1152
  GP_CONST_CELL \K, (\c+1)
  GP_LOADNEXT \last
  s_branch \tab\()_\target\()_div
  GP_ROWOP \tab, \K, \blk, \c, \last, 1184, v_add_f32_e32
  GP_ROWOP \tab, \K, \blk, \c, \last, 1280, v_sub_f32_e32
  GP_ROWOP \tab, \K, \blk, \c, \last, 1376, v_mul_f32_e32
 .org \tab + 81600 + 3776*(\blk) + 1472
  GP_ROW \K, (\c+1)
  GP_LOADNEXT \last
  s_waitcnt lgkmcnt(0)
  s_branch \tab\()_\target\()_div
// a constant, a row minus or over the top
  GP_CONSTOP \tab, \K, \blk, \c, \last, 1536, v_sub_f32_e32
 .org \tab + 81600 + 3776*(\blk) + 1600
  GP_CONST_CELL \K, (\c+1)
  GP_LOADNEXT \last
  s_branch \tab\()_\target\()_divr
 .org \tab + 81600 + 3776*(\blk) + 1632
  GP_ROW \K, (\c+1)
  GP_LOADNEXT \last
  s_waitcnt lgkmcnt(0)
  GP_ALL2 v_sub_f32_e32, \K, \c, (\c+1), \c
  GP_JUMP \last
 .org \tab + 81600 + 3776*(\blk) + 1728
  GP_ROW \K, (\c+1)
  GP_LOADNEXT \last
  s_waitcnt lgkmcnt(0)
  s_branch \tab\()_\target\()_divr
.endm
.macro GP_UN tab, blk, u, off, last
 .org \tab + 81600 + 3776*(\blk) + 0+\off
  GP_LOADNEXT \last
\tab\()_\blk\()_un\u:
.endm
.macro GP_UNARIES tab, K, blk, c, last
  GP_UN \tab, \blk, 0, 1792, \last
  GP_SUMTEST \K, \c, 0x48000000
  s_cbranch_vccnz \tab\()_\blk\()_chk1
\tab\()_\blk\()_go1:
  GP_SIN \K, \c
  GP_NEXT \last
 .if \K == 1
  GP_CHECKS \tab, \K, \blk, \c
\tab\()_\blk\()_clog:
  GP_LOGP \K, \c
  GP_NEXT \last
 .endif
  GP_UN \tab, \blk, 1, 2208, \last
  GP_SUMTEST \K, \c, 0x48000000
  s_cbranch_vccnz \tab\()_\blk\()_chk2
\tab\()_\blk\()_go2:
  GP_COS \K, \c
  GP_NEXT \last
 .if (\K == 1) && ((\blk == 0) || (\c >= 1))
\tab\()_\blk\()_cdiv:
 .if \blk == 0
  GP_DIVP \K, 0, 1, 0
 .else
  GP_DIVP \K, (\c-1), \c, (\c-1)
 .endif
  GP_NEXT \last
\tab\()_\blk\()_cdivr:
 .if \blk == 0
  GP_DIVP \K, 1, 0, 0
 .else
  GP_DIVP \K, \c, (\c-1), (\c-1)
 .endif
  GP_NEXT \last
 .endif
  GP_UN \tab, \blk, 2, 2688, \last
  GP_SUMTEST \K, \c, 0x42ae0000
  s_cbranch_vccnz \tab\()_\blk\()_chk3
\tab\()_\blk\()_go3:
  GP_EXP \K, \c
  GP_NEXT \last
 .if \K == 1
  GP_TOCALLER \tab, \K, \blk, \c
 .endif
  GP_UN \tab, \blk, 3, 3008, \last
  GP_MAGNITUDE \K, \c, min, 4
  v_cmp_nlt_f32_e32 vcc, 0x3a83126f, v4
  s_cbranch_vccnz \tab\()_\blk\()_clog
  GP_LOG \K, \c
  GP_NEXT \last
  GP_UN \tab, \blk, 4, 3200, \last
  GP_MAGNITUDE \K, \c, min, 4
  v_cmp_nle_f32_e32 vcc, 0x0d800000, v4
  s_cbranch_vccnz \tab\()_\blk\()_slow4
 .irp j,0,1,2,3
 .if \j < \K
  v_sqrt_f32_e64 v[GP_CB+\K*\c+\j], |v[GP_CB+\K*\c+\j]|
 .endif
 .endr
  GP_NEXT \last
  GP_UN \tab, \blk, 5, 3296, \last
 .irp j,0,1,2,3
 .if \j < \K
  v_and_b32_e32 v[GP_CB+\K*\c+\j], 0x7fffffff, v[GP_CB+\K*\c+\j]
 .endif
 .endr
  GP_NEXT \last
.endm
.macro GP_PUSHUNS tab, K, blk, d, last, target
 .irp u,0,1,2,3,4,5
 .org \tab + 81600 + 3776*(\blk) + 3360+64*\u
  GP_ROW \K, \d
  GP_LOADNEXT \last
  s_waitcnt lgkmcnt(0)
  s_branch \tab\()_\target\()_un\u
 .endr
.endm

// ---- cold code.  With one case per lane, what a hot handler branches to lies in
// the unused part of its neighbours' slots (a branch would not reach the cold
// blocks of so deep a table).
// The top to the caller: code 1..4 (sin, cos, exp, sqrt beyond the fast
// range), 5..10 the library commands, 11 the square root with NaN below zero.
.macro GP_TOP K, c
 .irp j,0,1,2,3
 .if \j < \K
  v_mov_b32_e32 v[4+\j], v[GP_CB+\K*\c+\j]
 .endif
 .endr
.endm
.macro GP_LEAVE blk
  s_mov_b32 s87, 2400*(33-\blk) + 0
  s_waitcnt lgkmcnt(0)
  s_setpc_b64 s[94:95]
.endm
.macro GP_TOCALLER tab, K, blk, c
 .irp n,1,2,3,4
\tab\()_\blk\()_slow\n:
  s_mov_b32 s83, \n
  s_branch \tab\()_\blk\()_slow
 .endr
\tab\()_\blk\()_slow:
  GP_TOP \K, \c
  GP_LEAVE \blk
.endm
// the sum test failed: the largest magnitude decides (and a NaN, for exp)
.macro GP_CHECKS tab, K, blk, c
 .irp n,1,2
\tab\()_\blk\()_chk\n:
  GP_MAGNITUDE \K, \c, max, 5
  v_cmp_lt_f32_e32 vcc, 0x48000000, v5
  s_cbranch_vccnz \tab\()_\blk\()_slow\n
  s_branch \tab\()_\blk\()_go\n
 .endr
\tab\()_\blk\()_chk3:
  GP_MAGNITUDE \K, \c, max, 5
  v_cmp_lt_f32_e32 vcc, 0x42ae0000, v5
  s_cbranch_vccnz \tab\()_\blk\()_slow3
  v_cmp_u_f32_e32 vcc, v4, v4
  s_cbranch_vccnz \tab\()_\blk\()_slow3
  s_branch \tab\()_\blk\()_go3
.endm
.macro GP_SLOW tab, K, blk, c, last
// after a call: the values back into the top
 .org \tab + 2400*(33-\blk) + 0
 .irp j,0,1,2,3
 .if \j < \K
  v_mov_b32_e32 v[GP_CB+\K*\c+\j], v[4+\j]
 .endif
 .endr
  GP_JUMP \last
 .if \K > 1
 .org \tab + 2400*(33-\blk) + 32
  GP_TOCALLER \tab, \K, \blk, \c
 .org \tab + 2400*(33-\blk) + 96
  GP_CHECKS \tab, \K, \blk, \c
 .endif
.endm
.macro GP_COLDDIV tab, K, blk, a, last
 .if \K > 1
 .org \tab + 2400*(33-\blk) + 224
\tab\()_\blk\()_cdiv:
  GP_DIVP \K, \a, (\a+1), \a
  GP_NEXT \last
 .org \tab + 2400*(33-\blk) + 608
\tab\()_\blk\()_cdivr:
  GP_DIVP \K, (\a+1), \a, \a
  GP_NEXT \last
 .endif
.endm
.macro GP_COLDLOG tab, K, blk, c, last
 .if \K > 1
 .org \tab + 2400*(33-\blk) + 992
\tab\()_\blk\()_clog:
  GP_LOGP \K, \c
  GP_NEXT \last
 .endif
.endm
.macro GP_DUP tab, K, blk, d
 .org \tab + 2400*(33-\blk) + 1184
  GP_LOADNEXT 0
  GP_COPY_CELL \K, \d, (\d-1)
  GP_NEXT 0
.endm
.macro GP_SWAPDEL tab, K, blk, d
 .org \tab + 2400*(33-\blk) + 1248
  GP_LOADNEXT 0
 .irp j,0,1,2,3
 .if \j < \K
  v_swap_b32 v[GP_CB+\K*(\d-1)+\j], v[GP_CB+\K*(\d-2)+\j]
 .endif
 .endr
  GP_NEXT 0
 .org \tab + 2400*(33-\blk) + 1312
  GP_LOADNEXT 0
  GP_NEXT 0
.endm
// a held variable's cell: payload byte, numbered to 31 (the class has \maxd)
.macro GP_VARCELL K, maxd, dst, shift
  s_bfe_u32 \dst, s89, 0x50000+\shift
  s_sub_u32 \dst, \dst, 32-\maxd
  s_mul_i32 \dst, \dst, \K
.endm
// COPY: the variable's cell = the top
.macro GP_COPYVAR tab, K, maxd, blk, c
 .org \tab + 2400*(33-\blk) + 1344
  GP_VARCELL \K, \maxd, s96, 0
  GP_LOADNEXT 0
  s_set_gpr_idx_on s96, gpr_idx(DST)
 .irp j,0,1,2,3
 .if \j < \K
  v_mov_b32_e32 v[GP_CB+\j], v[GP_CB+\K*\c+\j]
 .endif
 .endr
  s_set_gpr_idx_off
  GP_NEXT 0
.endm
// PASTE: push the variable in cell byte 0; then the cell of byte 1 moves into
// it (the same cell when nothing moves)
.macro GP_PASTE tab, K, maxd, blk, d, last
 .org \tab + 2400*(33-\blk) + 1440
  GP_VARCELL \K, \maxd, s96, 0
  GP_VARCELL \K, \maxd, s97, 8
  GP_LOADNEXT \last
  s_set_gpr_idx_on s96, gpr_idx(SRC0)
 .irp j,0,1,2,3
 .if \j < \K
  v_mov_b32_e32 v[4+\j], v[GP_CB+\j]
 .endif
 .endr
  s_set_gpr_idx_off
  s_set_gpr_idx_on s97, gpr_idx(SRC0)
 .irp j,0,1,2,3
 .if \j < \K
  v_mov_b32_e32 v[12+\j], v[GP_CB+\j]
 .endif
 .endr
  s_set_gpr_idx_off
  s_set_gpr_idx_on s96, gpr_idx(DST)
 .irp j,0,1,2,3
 .if \j < \K
  v_mov_b32_e32 v[GP_CB+\j], v[12+\j]
 .endif
 .endr
  s_set_gpr_idx_off
 .irp j,0,1,2,3
 .if \j < \K
  v_mov_b32_e32 v[GP_CB+\K*\d+\j], v[4+\j]
 .endif
 .endr
  GP_NEXT \last
.endm
.macro GP_EXTUN tab, K, blk, c, last
 .org \tab + 2400*(33-\blk) + 1600
  GP_LOADNEXT \last
  GP_ALL2 v_mul_f32_e32, \K, \c, \c, \c
  GP_NEXT \last
 .org \tab + 2400*(33-\blk) + 1664
  GP_LOADNEXT \last
 .irp j,0,1,2,3
 .if \j < \K
  v_xor_b32_e32 v[GP_CB+\K*\c+\j], 0x80000000, v[GP_CB+\K*\c+\j]
 .endif
 .endr
  GP_NEXT \last
 .org \tab + 2400*(33-\blk) + 1728
  GP_LOADNEXT \last
  GP_CUBE \K, \c
  GP_NEXT \last
 .org \tab + 2400*(33-\blk) + 1856
  GP_LOADNEXT \last
  GP_MAGNITUDE \K, \c, min, 4
  v_cmp_nle_f32_e32 vcc, 0x0d800000, v4
  s_cbranch_vccnz \tab\()_\blk\()_slow11
  GP_SQRTRAW \K, \c
  GP_NEXT \last
 .org \tab + 2400*(33-\blk) + 2048
 .irp n,5,6,7,8,9,10
  s_mov_b32 s83, \n
  s_branch \tab\()_\blk\()_lib
 .endr
\tab\()_\blk\()_slow11:
  s_mov_b32 s83, 11
  s_branch \tab\()_\blk\()_cslow
\tab\()_\blk\()_lib:
  GP_LOADNEXT \last
\tab\()_\blk\()_cslow:
  GP_TOP \K, \c
  GP_LEAVE \blk
.endm
// POW of the cells \a, \a+1 (the top): both to the caller, the result into \a
// (the finish code of the block one element less deep)
.macro GP_POWCELLS tab, K, blk, a, last, lower
 .org \tab + 2400*(33-\blk) + 2176
  GP_LOADNEXT \last
\tab\()_\blk\()_pow:
 .irp j,0,1,2,3
 .if \j < \K
  v_mov_b32_e32 v[4+\j], v[GP_CB+\K*\a+\j]
  v_mov_b32_e32 v[12+\j], v[GP_CB+\K*(\a+1)+\j]
 .endif
 .endr
  s_mov_b32 s83, 12
  GP_LEAVE \lower
.endm
.macro GP_POWLEAF tab, K, blk, c, last, target
 .org \tab + 2400*(33-\blk) + 2272
  GP_CONST_CELL \K, (\c+1)
  GP_LOADNEXT \last
  s_branch \tab\()_\target\()_pow
 .org \tab + 2400*(33-\blk) + 2336
  GP_ROW \K, (\c+1)
  GP_LOADNEXT \last
  s_waitcnt lgkmcnt(0)
  s_branch \tab\()_\target\()_pow
.endm

// block \b = \d + 1: \d elements on the stack, at most \maxd; \n = \b + 1
.macro GP_HOTBLOCK tab, K, maxd, d, b, n
 .if \d < \maxd
  GP_PUSHES \tab, \K, \b, \d, 0
 .endif
 .if \d >= 2
  GP_CELLS \tab, \K, \b, (\d-2), 0
 .endif
 .if (\d >= 1) && (\d < \maxd)
  GP_LEAFOPS \tab, \K, \b, (\d-1), 0, \n
 .endif
 .if \d >= 1
  GP_UNARIES \tab, \K, \b, (\d-1), 0
 .endif
 .if \d < \maxd
  GP_PUSHUNS \tab, \K, \b, \d, 0, \n
 .endif
.endm
.macro GP_COLDBLOCK tab, K, maxd, d, b, n
 .if \d >= 1
  GP_SLOW \tab, \K, \b, (\d-1), 0
 .endif
 .if \d >= 2
  GP_COLDDIV \tab, \K, \b, (\d-2), 0
 .endif
 .if \d >= 1
  GP_COLDLOG \tab, \K, \b, (\d-1), 0
 .endif
 .if (\d >= 1) && (\d < \maxd)
  GP_DUP \tab, \K, \b, \d
 .endif
 .if \d >= 2
  GP_SWAPDEL \tab, \K, \b, \d
 .endif
 .if (\d >= 1) && (\d < \maxd)
  GP_COPYVAR \tab, \K, \maxd, \b, (\d-1)
 .endif
 .if \d < \maxd
  GP_PASTE \tab, \K, \maxd, \b, \d, 0
 .endif
 .if \d >= 1
  GP_EXTUN \tab, \K, \b, (\d-1), 0
 .endif
 .if \d >= 2
  GP_POWCELLS \tab, \K, \b, (\d-2), 0, (\b-1)
 .endif
 .if (\d >= 1) && (\d < \maxd)
  GP_POWLEAF \tab, \K, \b, (\d-1), 0, \n
 .endif
.endm
.macro GP_EIGHT kind, tab, K, maxd, d0, d1, d2, d3, d4, d5, d6, d7, d8, d9
  \kind \tab, \K, \maxd, \d0, \d1, \d2
  \kind \tab, \K, \maxd, \d1, \d2, \d3
  \kind \tab, \K, \maxd, \d2, \d3, \d4
  \kind \tab, \K, \maxd, \d3, \d4, \d5
  \kind \tab, \K, \maxd, \d4, \d5, \d6
  \kind \tab, \K, \maxd, \d5, \d6, \d7
  \kind \tab, \K, \maxd, \d6, \d7, \d8
  \kind \tab, \K, \maxd, \d7, \d8, \d9
.endm
.macro GP_EIGHTDOWN kind, tab, K, maxd, d0, d1, d2, d3, d4, d5, d6, d7, d8, d9
  \kind \tab, \K, \maxd, \d7, \d8, \d9
  \kind \tab, \K, \maxd, \d6, \d7, \d8
  \kind \tab, \K, \maxd, \d5, \d6, \d7
  \kind \tab, \K, \maxd, \d4, \d5, \d6
  \kind \tab, \K, \maxd, \d3, \d4, \d5
  \kind \tab, \K, \maxd, \d2, \d3, \d4
  \kind \tab, \K, \maxd, \d1, \d2, \d3
  \kind \tab, \K, \maxd, \d0, \d1, \d2
.endm
.macro GP_TABLE tab, K, maxd
 .p2align 8
 .skip 32
\tab\()_first:
 .set \tab, \tab\()_first - 2400*(33 - \maxd - 1)
 .if \maxd == 32
  GP_COLDBLOCK \tab, \K, 32, 32, 33, 34
  GP_EIGHTDOWN GP_COLDBLOCK, \tab, \K, \maxd, 24, 25, 26, 27, 28, 29, 30, 31, 32, 33
  GP_EIGHTDOWN GP_COLDBLOCK, \tab, \K, \maxd, 16, 17, 18, 19, 20, 21, 22, 23, 24, 25
 .endif
 .if \maxd == 16
  GP_COLDBLOCK \tab, \K, 16, 16, 17, 18
 .endif
 .if \maxd > 8
  GP_EIGHTDOWN GP_COLDBLOCK, \tab, \K, \maxd, 8, 9, 10, 11, 12, 13, 14, 15, 16, 17
 .else
  GP_COLDBLOCK \tab, \K, 8, 8, 9, 10
 .endif
  GP_EIGHTDOWN GP_COLDBLOCK, \tab, \K, \maxd, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9
  GP_SLOW \tab, \K, 0, 0, 1
  GP_COLDDIV \tab, \K, 0, 0, 1
  GP_COLDLOG \tab, \K, 0, 0, 1
 .org \tab + 2400*(33-0) + 1312
  GP_NEXT 1
  GP_PASTE \tab, \K, \maxd, 0, 0, 1
  GP_EXTUN \tab, \K, 0, 0, 1
  GP_POWCELLS \tab, \K, 0, 0, 1, 0
  GP_POWLEAF \tab, \K, 0, 0, 1, 0
  GP_PUSHES \tab, \K, 0, 0, 1
  GP_CELLS \tab, \K, 0, 0, 1
  GP_LEAFOPS \tab, \K, 0, 0, 1, 0
  GP_UNARIES \tab, \K, 0, 0, 1
  GP_PUSHUNS \tab, \K, 0, 0, 1, 0
  GP_EIGHT GP_HOTBLOCK, \tab, \K, \maxd, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9
 .if \maxd > 8
  GP_EIGHT GP_HOTBLOCK, \tab, \K, \maxd, 8, 9, 10, 11, 12, 13, 14, 15, 16, 17
 .endif
 .if \maxd > 16
  GP_EIGHT GP_HOTBLOCK, \tab, \K, \maxd, 16, 17, 18, 19, 20, 21, 22, 23, 24, 25
  GP_EIGHT GP_HOTBLOCK, \tab, \K, \maxd, 24, 25, 26, 27, 28, 29, 30, 31, 32, 33
 .endif
 .if \maxd == 8
  GP_HOTBLOCK \tab, \K, 8, 8, 9, 10
 .elseif \maxd == 16
  GP_HOTBLOCK \tab, \K, 16, 16, 17, 18
 .else
  GP_HOTBLOCK \tab, \K, 32, 32, 33, 34
 .endif
 .fill 64, 4, 0xbf9f0000
.endm

GP_TABLE gp_threads_d8, 4, 8
GP_TABLE gp_threads_d16, 2, 16
GP_TABLE gp_threads_d32, 1, 32
.popsection
)");
#endif
}
