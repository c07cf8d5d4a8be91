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
// of scalar issue per word); this form spends six and none, and uses literal
// or vector-register constants throughout.  100,000 programs x 4,096 cases:
// a whole scoring call 1.74 -> 1.32 ms, 200,000 uneven programs x 16,384
// cases 9.69 -> 7.26 ms, same bits.
//
// Handler table (one per depth class): a 4,096-byte block per stack depth.
// Block 0 holds the forms that end a program (the stack ends with one
// element, so only one depth each); block d + 1 those that start with d
// elements on the stack.  Inside a block every operator has a fixed offset,
// so a word is the same for every class.  Word: x = block * 4096 + offset,
// y = constant bits, or the LDS byte offset of an input row at four cases
// per lane.
#pragma once

constexpr uint32_t kThBlock = 4096u;
constexpr uint32_t kThPushC = 0u;            // push a constant
constexpr uint32_t kThPushV = 64u;           // push an input row
constexpr uint32_t kThBin = 128u;            // + - * /: two stack cells (64 bytes each, / longer)
constexpr uint32_t kThBinC = 704u;           // top OP constant
constexpr uint32_t kThBinV = 960u;           // top OP input row
constexpr uint32_t kThPushUn = 2816u;        // push f(input row)
constexpr uint32_t kThSlow = 3200u;          // out-of-range values: leave to the caller
// sin cos exp ln sqrt abs of the top: offsets in units of 64, one byte each
constexpr uint64_t kThUnary = 0x2B2926211A13ull;

// Words of the threaded form, made from the runtime depth `rt` before the
// instruction (staging.h's walk asks for them through this interface).
struct ThreadedWords {
    static __host__ __device__ uint32_t at(int rt, uint32_t off) { return (uint32_t)(rt + 1) * kThBlock + off; }
    static __host__ __device__ uint32_t un(uint32_t sel) { return ((uint32_t)(kThUnary >> (8u * sel)) & 0xFFu) * 64u; }
    static __host__ __device__ uint2 push_const(int rt, uint32_t bits) { return make_uint2(at(rt, kThPushC), bits); }
    static __host__ __device__ uint2 push_row(int rt, uint32_t payload) { return make_uint2(at(rt, kThPushV), payload); }
    static __host__ __device__ uint2 push_unary(int rt, uint32_t sel, uint32_t payload)
    {
        return make_uint2(at(rt, kThPushUn + 64u * sel), payload);
    }
    static __host__ __device__ uint2 top_row(int rt, uint32_t sel, uint32_t payload)
    {
        return make_uint2(at(rt, kThBinV + 64u * sel), payload);
    }
    static __host__ __device__ uint2 top_const(int rt, uint32_t sel, uint32_t bits)
    {
        return make_uint2(at(rt, kThBinC + 64u * sel), bits);
    }
    static __host__ __device__ uint2 cells(int rt, uint32_t sel) { return make_uint2(at(rt, kThBin + 64u * sel), 0u); }
    static __host__ __device__ uint2 unary(int rt, uint32_t sel) { return make_uint2(at(rt, un(sel)), 0u); }
    // the same word as the program's last
    static __host__ __device__ uint2 last(uint2 w) { return make_uint2(w.x & (kThBlock - 1u), w.y); }
};
