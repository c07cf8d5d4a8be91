// staging.h -- the command table's operator kinds and the GCL stack and variable
// discipline (GclCheck), shared by the host validator and the device's staging
// (stage_waves.h), so that both accept the same programs.
//
// The includer provides, before this header: gpeval.h, __host__ and __device__.
#pragma once

// A variable's payload in a staged word is its input row's byte offset at 256
// staged cases (threaded.h).
constexpr uint32_t kVarPayload = 1024u;

// Op kinds of the command table.  Unary selectors: the benchmark set's six
// (SIN..ABS) first, then SQUARE..SQRT_RAW; POW's selector follows ADD..DIV.
// (bit tables over the 28 opcodes: one shift per test)
constexpr uint32_t kUnaryOps = 0xFC0u | (((1u << 10) - 1u) << GP_SQUARE);  // SIN..ABS, SQUARE..SQRT_RAW
__host__ __device__ constexpr bool op_is_unary(uint32_t op)
{
    return op < 32u && ((kUnaryOps >> op) & 1u);
}
__host__ __device__ constexpr uint32_t uop_sel(uint32_t op)
{
    return op <= GP_ABS ? op - GP_SIN : op - GP_SQUARE + 6u;
}
constexpr uint32_t kUnSquare = 6u;      // first selector beyond the benchmark set
constexpr uint32_t kBinPow = 4u;

// The GCL stack and variable discipline, one node at a time; the host
// validator and the device staging passes share it, so both accept the
// same programs.  Held variables fill the storage cells from the top:
// variable k sits `pos` cells below the top cell; a PASTE frees its cell
// and the variable in the lowest held cell moves into it, so the held
// variables always occupy the top `live` cells.
struct GclCheck {
    int depth = 0, live = 0, maxd = 0;
    uint32_t held = 0u;                 // bit k: variable k holds a value
    uint64_t pos = 0ull;                // 4 bits per variable

    __host__ __device__ int var_pos(uint32_t k) const { return (int)((pos >> (4u * k)) & 15ull); }
    __host__ __device__ void set_pos(uint32_t k, int p)
    {
        pos = (pos & ~(15ull << (4u * k))) | ((uint64_t)p << (4u * k));
    }
    // COPY @k of a free variable: its cell position.
    __host__ __device__ int copy(uint32_t k)
    {
        held |= 1u << k;
        set_pos(k, live);
        return live++;
    }
    // PASTE @k of a held variable: the position of the variable that moves
    // into k's freed cell, or -1.
    __host__ __device__ int paste(uint32_t k)
    {
        const int p = var_pos(k);
        held &= ~(1u << k);
        --live;
        if (p == live) return -1;
        for (uint32_t m = 0; m < GP_GCL_VARS; ++m)
            if (((held >> m) & 1u) && var_pos(m) == live) set_pos(m, p);
        return live;
    }
    // Applies one node; returns its GP_PROG_* status (checks in the order
    // op, operand range, underflow, pairing, depth).
    __host__ __device__ int step(uint32_t op, uint32_t arg, uint32_t allowed, int32_t n_vars,
                                 int64_t n_consts)
    {
        if (op < GP_DUP) {
            // the benchmark set: leaves push, binary ops pop one, unary ops
            // keep the depth
            if (!((allowed >> op) & 1u)) return GP_PROG_BAD_OP;
            if (op == GP_LOAD && (int64_t)arg >= (int64_t)n_vars) return GP_PROG_BAD_VAR;
            if (op == GP_CONST && (int64_t)arg >= n_consts) return GP_PROG_BAD_CONST;
            if (depth < (op <= GP_CONST ? 0 : (op <= GP_DIV ? 2 : 1))) return GP_PROG_UNDERFLOW;
            depth += op <= GP_CONST ? 1 : (op <= GP_DIV ? -1 : 0);
        } else {
            if (op >= GP_N_OPS || !((allowed >> op) & 1u)) return GP_PROG_BAD_OP;
            const int need = op == GP_SWAP || op == GP_POW ? 2 : (op == GP_PASTE ? 0 : 1);
            if (depth < need) return GP_PROG_UNDERFLOW;
            if (op == GP_COPY) {
                if (arg >= GP_GCL_VARS || ((held >> arg) & 1u)) return GP_PROG_BAD_PAIR;
                copy(arg);
            } else if (op == GP_PASTE) {
                if (arg >= GP_GCL_VARS || !((held >> arg) & 1u)) return GP_PROG_BAD_PAIR;
                paste(arg);
            }
            if (op == GP_PASTE || op == GP_DUP) ++depth;
            else if (op == GP_POW || op == GP_DEL) --depth;
        }
        if (depth + live > GP_MAX_STACK) return GP_PROG_TOO_DEEP;
        if (depth + live > maxd) maxd = depth + live;
        return GP_PROG_OK;
    }
    __host__ __device__ int finish() const
    {
        return depth != 1 ? GP_PROG_FINAL_DEPTH : (live != 0 ? GP_PROG_BAD_PAIR : GP_PROG_OK);
    }
};
