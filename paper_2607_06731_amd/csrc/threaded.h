// threaded.h -- the benchmark-set interpreter as threaded code for gfx950.
//
// Each staged word names the address of the code that runs it: a handler
// specialised for one operator at one stack depth, so every stack cell is a
// fixed group of registers and no operand is moved or indexed.  A handler
// loads the next word, does its arithmetic on K cases per lane and jumps to
// the next handler; nothing is decoded.
//
// What it was built for (MI355X, clocks at 2.4 GHz per 64-lane instruction
// and SIMD, eight wavefronts per SIMD, measured): fp32 add, multiply, fma,
// moves and bit operations on vector registers, inline constants or literals
// issue every 2.2-2.5 clocks; the same with a scalar-register operand, and
// compares, selects, minima, conversions, division steps and every
// instruction in register-index mode, every 4.2-4.4; they pair with the
// first kind (1:1 mixes 2.4-2.9 per instruction), not with each other.  A
// scalar instruction costs 4.2 (one per clock for the four SIMDs of a CU).
// A loop that decodes flag bits spent 19 scalar and branch instructions and
// a register-indexed move per case on each word (101 clocks of vector and 77
// of scalar issue per word); this form spends six per word and none,
// and uses literal or vector-register constants throughout.  100,000 programs
// x 4,096 cases: a whole scoring call 1.74 -> 1.32 ms, 200,000 uneven programs
// x 16,384 cases 9.69 -> 7.26 ms, same bits.
//
// Cases per lane (K): 4 where the stack class holds at most 8 elements, 2 up
// to 16, 1 up to 32 -- 32 registers of stack in every class, so one kernel
// runs all three at six wavefronts per SIMD.  Eight, four and two cases spend
// 6% fewer vector instructions (a word's scalar work serves twice the cases)
// but leave four wavefronts and twice the code: the 100,000-program call took
// 1.34 ms against 1.32.
//
// Handler table (one per depth class): two blocks per stack depth, the hot
// one with the handlers that ordinary values take and the cold one with the
// rest; hot blocks lie together.  Block 0 holds the forms that end a program
// (the stack ends with one element, so only one depth each); block d + 1
// those that start with d elements on the stack.  Inside a block every
// operator has a fixed offset, so a word is the same for every class.  Word:
// x = the handler's offset from the table, y = constant bits, or variable
// index * 1024 (scaled to a byte offset by the number of cases staged / 256),
// or the cells of a variable move.
#pragma once

constexpr uint32_t kThHot = 3776u, kThCold = 2400u;     // bytes of a block
constexpr uint32_t kThHot0 = 34u * kThCold;             // hot blocks start here, upwards
constexpr uint32_t kThPushC = 0u;            // push a constant
constexpr uint32_t kThPushV = 64u;           // push an input row
constexpr uint32_t kThBin = 128u;            // + - * /: two stack cells (64 bytes each, / longer)
constexpr uint32_t kThBinC = 960u;           // top OP constant (64 bytes each)
constexpr uint32_t kThBinV = 1184u;          // top OP input row (96 bytes each)
// - and / with the top as the left operand: two cells; a constant; a row
constexpr uint32_t kThSubR = 608u, kThDivR = 672u, kThSubCR = 1536u, kThDivCR = 1600u;
constexpr uint32_t kThSubVR = 1632u, kThDivVR = 1728u;
constexpr uint32_t kThPushUn = 3360u;        // push f(input row) (64 bytes each)
// sin cos exp ln sqrt abs of the top: offsets in units of 32, one byte each
constexpr uint64_t kThUnary = 0x67645E544538ull;
// beyond the benchmark set: offsets in the cold block, marked
constexpr uint32_t kThColdBit = 0x8000u;
constexpr uint32_t kThDup = kThColdBit + 1184u, kThSwap = kThColdBit + 1248u, kThDel = kThColdBit + 1312u;
constexpr uint32_t kThCopy = kThColdBit + 1344u, kThPaste = kThColdBit + 1440u;
constexpr uint32_t kThSquare = kThColdBit + 1600u, kThSign = kThColdBit + 1664u, kThCube = kThColdBit + 1728u;
constexpr uint32_t kThSqrtRaw = kThColdBit + 1856u;
constexpr uint32_t kThLibrary = kThColdBit + 2048u;     // cbrt tan asin acos atan tanh: 8 bytes each
constexpr uint32_t kThPow = kThColdBit + 2176u, kThPowC = kThColdBit + 2272u, kThPowV = kThColdBit + 2336u;

// Result codes of a handler that hands values to the caller (0: the program
// has ended).
enum : uint32_t {
    kCallSin = 1, kCallCos, kCallExp, kCallSqrt, kCallCbrt, kCallTan, kCallAsin, kCallAcos,
    kCallAtan, kCallTanh, kCallSqrtRaw, kCallPow
};

// Words of the threaded form, made from the runtime depth `rt` before the
// instruction.
struct ThreadedWords {
    static __host__ __device__ uint32_t at(int rt, uint32_t off)
    {
        return off < kThColdBit ? kThHot0 + (uint32_t)(rt + 1) * kThHot + off
                                : (uint32_t)(32 - rt) * kThCold + off - kThColdBit;
    }
    static __host__ __device__ uint32_t un(uint32_t sel)
    {
        if (sel < kUnSquare) return ((uint32_t)(kThUnary >> (8u * sel)) & 0xFFu) * 32u;
        const uint32_t e = sel - kUnSquare;
        if (e == 0u) return kThSquare;
        if (e == 1u) return kThSign;
        if (e == 2u) return kThCube;
        return e == 9u ? kThSqrtRaw : kThLibrary + 8u * (e - 3u);
    }
    static __host__ __device__ uint2 push_const(int rt, uint32_t bits) { return make_uint2(at(rt, kThPushC), bits); }
    static __host__ __device__ uint2 push_row(int rt, uint32_t payload) { return make_uint2(at(rt, kThPushV), payload); }
    static __host__ __device__ uint2 push_unary(int rt, uint32_t sel, uint32_t payload)
    {
        return make_uint2(at(rt, kThPushUn + 64u * sel), payload);
    }
    static __host__ __device__ uint2 top_row(int rt, uint32_t sel, uint32_t payload)
    {
        return make_uint2(at(rt, sel == kBinPow ? kThPowV : kThBinV + 96u * sel), payload);
    }
    static __host__ __device__ uint2 top_const(int rt, uint32_t sel, uint32_t bits)
    {
        return make_uint2(at(rt, sel == kBinPow ? kThPowC : kThBinC + 64u * sel), bits);
    }
    static __host__ __device__ uint2 cells(int rt, uint32_t sel)
    {
        return make_uint2(at(rt, sel == kBinPow ? kThPow : kThBin + 64u * sel), 0u);
    }
    // the same with the operands exchanged: the row, the constant, the top is
    // the left one (sel 1: -, else /; + and * do not tell)
    static __host__ __device__ uint2 row_top(int rt, uint32_t sel, uint32_t payload)
    {
        return make_uint2(at(rt, sel == 1u ? kThSubVR : kThDivVR), payload);
    }
    static __host__ __device__ uint2 const_top(int rt, uint32_t sel, uint32_t bits)
    {
        return make_uint2(at(rt, sel == 1u ? kThSubCR : kThDivCR), bits);
    }
    static __host__ __device__ uint2 cells_top(int rt, uint32_t sel)
    {
        return make_uint2(at(rt, sel == 1u ? kThSubR : kThDivR), 0u);
    }
    static __host__ __device__ uint2 unary(int rt, uint32_t sel) { return make_uint2(at(rt, un(sel)), 0u); }
    // DUP, SWAP, DEL: `off` is the command's; COPY and PASTE with their cells
    // (numbered to 31, the class's own cells are the last of them)
    static __host__ __device__ uint2 move(int rt, uint32_t off, uint32_t cells = 0u)
    {
        return make_uint2(at(rt, off), cells);
    }
    // the same word as the program's last
    static __host__ __device__ uint2 last(uint2 w)
    {
        const uint32_t x = w.x < kThHot0 ? 33u * kThCold + w.x % kThCold : kThHot0 + (w.x - kThHot0) % kThHot;
        return make_uint2(x, w.y);
    }
};
