// interp_gfx950.h -- handler tables of the threaded interpreter (threaded.h
// has the word format and the reasons), in gfx950 assembly.
//
// Registers (fixed; the caller's asm statement lists them all):
//   s[84:85] code of the program   s86 byte offset of the word after next
//   s[88:89] next word             s[90:91] table       s[92:93] jump target
//   s[94:95] return address        s87 resume offset    s83 result code
//   s[68:75] compare masks         s[96:97] scratch     vcc
//   v22..v25 constants             v31 LDS address of the lane's first case
//   v4..v19 temporaries (v4..v7 carry values to and from the caller)
//   v36.. stack cells, K registers each (case j of cell i: v[36 + K i + j])
// A handler takes its payload (s89), loads the next word into s[88:89] and
// ends in GP_NEXT.  Temporaries and cells of one case sit in different
// register banks (number mod 4), so three-operand forms read without a
// conflict.
//
// Wait states (gfx940 and later): one instruction between a transcendental
// instruction and a user of its result, two between a compare's mask and the
// select that reads it, four between v_div_scale's vcc and v_div_fmas.  The
// cases are interleaved so that these are other cases' instructions.
//
// Out-of-range values (sin and cos beyond 2^17, exp beyond 87, square roots
// of magnitudes below 2^-100): the handler hands the top's K values to the
// caller (result code 1..4), which applies the out-of-line
// function and resumes at the block's finish code.
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
.macro GP_JUMP tab, last
 .if \last
  s_mov_b32 s83, 0
  s_setpc_b64 s[94:95]
 .else
  s_add_u32 s92, s90, s88
  s_addc_u32 s93, s91, 0
  s_setpc_b64 s[92:93]
 .endif
.endm
.macro GP_NEXT tab, last
  s_waitcnt lgkmcnt(0)
  GP_JUMP \tab, \last
.endm

// cell \c = the input row at payload offset s89
.macro GP_ROW K, c
 .if \K == 4
  v_add_u32_e32 v4, s89, v31
  ds_read2st64_b32 v[GP_CB+4*\c:GP_CB+4*\c+1], v4 offset0:0 offset1:1
  ds_read2st64_b32 v[GP_CB+4*\c+2:GP_CB+4*\c+3], v4 offset0:2 offset1:3
 .else
  s_lshr_b32 s89, s89, 1
  v_add_u32_e32 v4, s89, v31
  ds_read2st64_b32 v[GP_CB+2*\c:GP_CB+2*\c+1], v4 offset0:0 offset1:1
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

// the fast-range test of the top cell \c: vcc = some |value| > \limit
.macro GP_RANGE K, c, limit
 .if \K == 4
  v_max3_f32 v4, |v[GP_CB+4*\c]|, |v[GP_CB+4*\c+1]|, |v[GP_CB+4*\c+2]|
  v_max_f32_e64 v4, v4, |v[GP_CB+4*\c+3]|
 .else
  v_max_f32_e64 v4, |v[GP_CB+2*\c]|, |v[GP_CB+2*\c+1]|
 .endif
  v_cmp_lt_f32_e32 vcc, \limit, v4
.endm

// sin after t (v4+j) and k (U) are set: reduction by three parts of pi,
// odd polynomial, sign flip by t's low bit
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

// unary operators of top cell \c; \blk: this block (for the slow path)
.macro GP_SIN tab, K, c, blk
  GP_RANGE \K, \c, 0x48000000
  s_cbranch_vccnz \tab\()_\blk\()_slow1
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
.macro GP_COS tab, K, c, blk
  GP_RANGE \K, \c, 0x48000000
  s_cbranch_vccnz \tab\()_\blk\()_slow2
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
.macro GP_EXP tab, K, c, blk
  GP_RANGE \K, \c, 0x42ae0000
  s_cbranch_vccnz \tab\()_\blk\()_slow3
 .irp j,0,1,2,3
 .if \j < \K
  v_mul_f32_e32 v[4+((\j+3)&3)], 0x3fb8aa3b, v[GP_CB+\K*\c+\j]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_rndne_f32_e32 v[8+((\j+1)&3)], v[4+((\j+3)&3)]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_fma_f32 v[12+((\j+2)&3)], v[GP_CB+\K*\c+\j], v24, -v[4+((\j+3)&3)]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_sub_f32_e32 v[4+((\j+3)&3)], v[4+((\j+3)&3)], v[8+((\j+1)&3)]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_fmac_f32_e32 v[12+((\j+2)&3)], 0x32a57060, v[GP_CB+\K*\c+\j]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_add_f32_e32 v[4+((\j+3)&3)], v[4+((\j+3)&3)], v[12+((\j+2)&3)]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_cvt_i32_f32_e32 v[8+((\j+1)&3)], v[8+((\j+1)&3)]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_exp_f32_e32 v[4+((\j+3)&3)], v[4+((\j+3)&3)]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_ldexp_f32 v[GP_CB+\K*\c+\j], v[4+((\j+3)&3)], v[8+((\j+1)&3)]
 .endif
 .endr
.endm
.macro GP_LOG K, c
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
.macro GP_SQRT tab, K, c, blk
 .if \K == 4
  v_min3_f32 v4, |v[GP_CB+4*\c]|, |v[GP_CB+4*\c+1]|, |v[GP_CB+4*\c+2]|
  v_min_f32_e64 v4, v4, |v[GP_CB+4*\c+3]|
 .else
  v_min_f32_e64 v4, |v[GP_CB+2*\c]|, |v[GP_CB+2*\c+1]|
 .endif
  v_cmp_nle_f32_e32 vcc, 0x0d800000, v4
  s_cbranch_vccnz \tab\()_\blk\()_slow4
 .irp j,0,1,2,3
 .if \j < \K
  v_sqrt_f32_e64 v[GP_CB+\K*\c+\j], |v[GP_CB+\K*\c+\j]|
 .endif
 .endr
.endm
.macro GP_ABS K, c
 .irp j,0,1,2,3
 .if \j < \K
  v_and_b32_e32 v[GP_CB+\K*\c+\j], 0x7fffffff, v[GP_CB+\K*\c+\j]
 .endif
 .endr
.endm
// cell \a = cell \a OP cell \a+1
.macro GP_OP3 K, op, a
 .irp j,0,1,2,3
 .if \j < \K
  \op v[GP_CB+\K*\a+\j], v[GP_CB+\K*\a+\j], v[GP_CB+\K*(\a+1)+\j]
 .endif
 .endr
.endm
// the same with the first source taken from cell \a+1 (of two NaN operands
// the first decides the result's sign: the order is the flag form's)
.macro GP_OP3R K, op, a
 .irp j,0,1,2,3
 .if \j < \K
  \op v[GP_CB+\K*\a+\j], v[GP_CB+\K*(\a+1)+\j], v[GP_CB+\K*\a+\j]
 .endif
 .endr
.endm
// protected division: the IEEE quotient (scaled reciprocal, one Newton step,
// two residual corrections, fix-up), 1 where |divisor| <= 0.001
.macro GP_DIV K, a
 .irp j,0,1,2,3
 .if \j < \K
  v_div_scale_f32 v[4+((\j+3)&3)], s[96:97], v[GP_CB+\K*(\a+1)+\j], v[GP_CB+\K*(\a+1)+\j], v[GP_CB+\K*\a+\j]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_rcp_f32_e32 v[8+((\j+1)&3)], v[4+((\j+3)&3)]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_cmp_nle_f32_e64 s[68+2*\j:69+2*\j], |v[GP_CB+\K*(\a+1)+\j]|, v25
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
  v_div_scale_f32 v16, vcc, v[GP_CB+\K*\a+\j], v[GP_CB+\K*(\a+1)+\j], v[GP_CB+\K*\a+\j]
  v_mul_f32_e32 v17, v16, v[8+((\j+1)&3)]
  v_fma_f32 v18, -v[4+((\j+3)&3)], v17, v16
  v_fmac_f32_e32 v17, v18, v[8+((\j+1)&3)]
  v_fma_f32 v18, -v[4+((\j+3)&3)], v17, v16
  v_div_fmas_f32 v[12+((\j+2)&3)], v18, v[8+((\j+1)&3)], v17
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_div_fixup_f32 v[12+((\j+2)&3)], v[12+((\j+2)&3)], v[GP_CB+\K*(\a+1)+\j], v[GP_CB+\K*\a+\j]
 .endif
 .endr
 .irp j,0,1,2,3
 .if \j < \K
  v_cndmask_b32_e64 v[GP_CB+\K*\a+\j], 1.0, v[12+((\j+2)&3)], s[68+2*\j:69+2*\j]
 .endif
 .endr
.endm

.macro GP_UN tab, blk, u, off, last
 .org \tab + 4096*(\blk) + \off
  GP_LOADNEXT \last
\tab\()_\blk\()_un\u:
.endm

// the handlers of block \blk whose instruction starts with \d elements;
// \last: the ones that end a program
.macro GP_PUSHES tab, K, blk, d, last
 .org \tab + 4096*(\blk)
  GP_CONST_CELL \K, \d
  GP_LOADNEXT \last
  GP_NEXT \tab, \last
 .org \tab + 4096*(\blk) + 64
  GP_ROW \K, \d
  GP_LOADNEXT \last
  GP_NEXT \tab, \last
.endm
.macro GP_PUSHUNS tab, K, blk, d, last, target
 .irp u,0,1,2,3,4,5
 .org \tab + 4096*(\blk) + 2816 + 64*\u
  GP_ROW \K, \d
  GP_LOADNEXT \last
  s_waitcnt lgkmcnt(0)
  s_branch \tab\()_\target\()_un\u
 .endr
.endm
.macro GP_CELLS tab, K, blk, a, last
 .org \tab + 4096*(\blk) + 128
  GP_LOADNEXT \last
  GP_OP3R \K, v_add_f32_e32, \a
  GP_NEXT \tab, \last
 .org \tab + 4096*(\blk) + 192
  GP_LOADNEXT \last
  GP_OP3 \K, v_sub_f32_e32, \a
  GP_NEXT \tab, \last
 .org \tab + 4096*(\blk) + 256
  GP_LOADNEXT \last
  GP_OP3R \K, v_mul_f32_e32, \a
  GP_NEXT \tab, \last
 .org \tab + 4096*(\blk) + 320
  GP_LOADNEXT \last
\tab\()_\blk\()_div:
  GP_DIV \K, \a
  GP_NEXT \tab, \last
.endm
// top cell \c OP a constant
.macro GP_CONSTOP tab, K, blk, c, last, n, op
 .org \tab + 4096*(\blk) + 704 + 64*\n
  v_mov_b32_e32 v4, s89
  GP_LOADNEXT \last
 .irp j,0,1,2,3
 .if \j < \K
  \op v[GP_CB+\K*\c+\j], v4, v[GP_CB+\K*\c+\j]
 .endif
 .endr
  GP_NEXT \tab, \last
.endm
// top cell \c OP an input row (taken into cell \c + 1)
.macro GP_ROWOP tab, K, blk, c, last, n, op
 .org \tab + 4096*(\blk) + 960 + 64*\n
  GP_ROW \K, (\c+1)
  GP_LOADNEXT \last
  s_waitcnt lgkmcnt(0)
  GP_OP3 \K, \op, \c
  GP_JUMP \tab, \last
.endm
.macro GP_LEAFOPS tab, K, blk, c, last, target
  GP_CONSTOP \tab, \K, \blk, \c, \last, 0, v_add_f32_e32
  GP_CONSTOP \tab, \K, \blk, \c, \last, 1, v_subrev_f32_e32
  GP_CONSTOP \tab, \K, \blk, \c, \last, 2, v_mul_f32_e32
 .org \tab + 4096*(\blk) + 704 + 192
  GP_CONST_CELL \K, (\c+1)
  GP_LOADNEXT \last
  s_branch \tab\()_\target\()_div
  GP_ROWOP \tab, \K, \blk, \c, \last, 0, v_add_f32_e32
  GP_ROWOP \tab, \K, \blk, \c, \last, 1, v_sub_f32_e32
  GP_ROWOP \tab, \K, \blk, \c, \last, 2, v_mul_f32_e32
 .org \tab + 4096*(\blk) + 960 + 192
  GP_ROW \K, (\c+1)
  GP_LOADNEXT \last
  s_waitcnt lgkmcnt(0)
  s_branch \tab\()_\target\()_div
.endm
.macro GP_UNARIES tab, K, blk, c, last
  GP_UN \tab, \blk, 0, 1216, \last
  GP_SIN \tab, \K, \c, \blk
  GP_NEXT \tab, \last
  GP_UN \tab, \blk, 1, 1664, \last
  GP_COS \tab, \K, \c, \blk
  GP_NEXT \tab, \last
  GP_UN \tab, \blk, 2, 2112, \last
  GP_EXP \tab, \K, \c, \blk
  GP_NEXT \tab, \last
  GP_UN \tab, \blk, 3, 2432, \last
  GP_LOG \K, \c
  GP_NEXT \tab, \last
  GP_UN \tab, \blk, 4, 2624, \last
  GP_SQRT \tab, \K, \c, \blk
  GP_NEXT \tab, \last
  GP_UN \tab, \blk, 5, 2752, \last
  GP_ABS \K, \c
  GP_NEXT \tab, \last
.endm
// values for the caller: code 1 + operator (sin, cos, exp, sqrt), the top in
// v4.., resume at the finish code
.macro GP_SLOW tab, K, blk, c, last
 .org \tab + 4096*(\blk) + 3200
 .irp n,1,2,3,4
\tab\()_\blk\()_slow\n:
  s_mov_b32 s83, \n
  s_branch \tab\()_\blk\()_slow
 .endr
\tab\()_\blk\()_slow:
 .irp j,0,1,2,3
 .if \j < \K
  v_mov_b32_e32 v[4+\j], v[GP_CB+\K*\c+\j]
 .endif
 .endr
  s_mov_b32 s87, 4096*\blk + 3328
  s_waitcnt lgkmcnt(0)
  s_setpc_b64 s[94:95]
 .org \tab + 4096*(\blk) + 3328
 .irp j,0,1,2,3
 .if \j < \K
  v_mov_b32_e32 v[GP_CB+\K*\c+\j], v[4+\j]
 .endif
 .endr
  GP_JUMP \tab, \last
.endm
// block \b = \d + 1: \d elements on the stack, at most \maxd; \n = \b + 1
.macro GP_BLOCK tab, K, maxd, d, b, n
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
 .if \d >= 1
  GP_SLOW \tab, \K, \b, (\d-1), 0
 .endif
.endm
.macro GP_BLOCKS8 tab, K, maxd, d0, d1, d2, d3, d4, d5, d6, d7, d8, d9
  GP_BLOCK \tab, \K, \maxd, \d0, \d1, \d2
  GP_BLOCK \tab, \K, \maxd, \d1, \d2, \d3
  GP_BLOCK \tab, \K, \maxd, \d2, \d3, \d4
  GP_BLOCK \tab, \K, \maxd, \d3, \d4, \d5
  GP_BLOCK \tab, \K, \maxd, \d4, \d5, \d6
  GP_BLOCK \tab, \K, \maxd, \d5, \d6, \d7
  GP_BLOCK \tab, \K, \maxd, \d6, \d7, \d8
  GP_BLOCK \tab, \K, \maxd, \d7, \d8, \d9
.endm
.macro GP_TABLE tab, K, maxd
 .p2align 8
\tab:
  GP_PUSHES \tab, \K, 0, 0, 1
  GP_CELLS \tab, \K, 0, 0, 1
  GP_LEAFOPS \tab, \K, 0, 0, 1, 0
  GP_UNARIES \tab, \K, 0, 0, 1
  GP_PUSHUNS \tab, \K, 0, 0, 1, 0
  GP_SLOW \tab, \K, 0, 0, 1
  GP_BLOCKS8 \tab, \K, \maxd, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9
 .if \maxd > 8
  GP_BLOCKS8 \tab, \K, \maxd, 8, 9, 10, 11, 12, 13, 14, 15, 16, 17
 .endif
 .if \maxd > 16
  GP_BLOCKS8 \tab, \K, \maxd, 16, 17, 18, 19, 20, 21, 22, 23, 24, 25
  GP_BLOCKS8 \tab, \K, \maxd, 24, 25, 26, 27, 28, 29, 30, 31, 32, 33
 .endif
 .if \maxd == 8
  GP_BLOCK \tab, \K, 8, 8, 9, 10
 .elseif \maxd == 16
  GP_BLOCK \tab, \K, 16, 16, 17, 18
 .else
  GP_BLOCK \tab, \K, 32, 32, 33, 34
 .endif
 .fill 64, 4, 0xbf9f0000
.endm

GP_TABLE gp_threads_d8, 4, 8
GP_TABLE gp_threads_d16, 4, 16
GP_TABLE gp_threads_d32, 2, 32
.popsection
)");
#endif
}
