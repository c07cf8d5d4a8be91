// stage_waves.h -- staging by wavefronts: validation, constant folding,
// Sethi-Ullman order and the threaded words (threaded.h) of one program by one
// wavefront.
//
// The includer provides, before this header: staging.h and threaded.h with what
// they ask for, the wavefront primitives __ballot, __shfl_up, __popcll,
// atomicMax (LDS), lanes_below, lane_value, prefix_min and wave_settle, and the
// folding functions binary_value and unary_value.  (A host build gives them 64
// lanes that run in turn between them, so the walk is tested without a GPU.)
#pragma once

// One wavefront stages one program: lane l holds node l of a 64-node chunk
// (longer programs take several chunks), and what a serial walk (stage_lane)
// decides node by node has a form over lanes.
//   depth after a node   pushes minus pops up to it (two ballots)
//   elements that depend on a variable (the runtime depth)
//                        the smallest depth since the last variable or
//                        command that is not folded: a prefix minimum, made
//                        one scan over the whole chunk by subtracting 64 per
//                        such node passed
//   held constants       depth minus runtime depth
// From those each node knows the word it emits, if any, and the words before
// it.  Serial, uniform in the wavefront, are only the folded operators (their
// operands are the values at the last node of each depth) and, with the
// whole command table (EXT), the named variables' cells.  (A serial walk, a
// program per lane, cost 275 instructions a node for every wavefront, the
// union of what its 64 lanes were doing: 33 us for 32 programs, 70 us for
// 10,000; with the whole table 64 + 75 us for 2,000.)  Statuses, depths and
// values are the serial walk's; constants are held without a limit.
//
// LDS per wavefront: for each depth, one past the last node that left the
// stack there in the chunks before, and the constant at it.
constexpr int kDepthSlots = GP_MAX_STACK + 1;
struct WaveTables {
    uint32_t last[kDepthSlots];
    float value[kDepthSlots];
};

// Operands in Sethi-Ullman order: a binary operator whose right operand needs
// more stack cells than the left one takes it first, so an operator over
// operands of equal need is the only one that takes a cell more, and a program
// of 128 nodes needs at most 7.  (In the order written, an eighth of the
// programs of up to 64 nodes need more than 8 cells, a third of those of up to
// 128 -- half of all nodes -- and run at two or one cases per lane.)  The results
// are the same: no operator's operands change, only which of them is ready first.
// The walk takes a wavefront 4 us, which short datasets do not give back.  (us per
// call with and without it, programs of 3-64 nodes: 50,000 x 1,024 cases 265 and
// 256, x 2,048 401 and 417, x 8,192 1,083 and 1,238; 10,000 x 1,024 104 and 127,
// x 2,048 154 and 147, x 8,192 368 and 390; 1,000 x 1,024 50 and 44, x 2,048 62
// and 52, x 8,192 89 and 97; of 3-128 nodes 50,000 x 1,024 469 and 466, x 2,048 719
// and 787, x 8,192 1,998 and 2,523; 1,000 x 2,048 85 and 90.  Calls of few programs
// would gain from a higher limit, those of 10,000 from a lower one; the limit
// looks at the dataset alone, so that a program is staged the same way in any
// population.)
constexpr int kReorderMax = 128;         // nodes: two per lane
constexpr int64_t kReorderCases = 2048;
constexpr uint32_t kReversed = 1u << 8;  // on - and / of the reordered program: the top is the left operand

// Reorders a valid program; false: nothing to gain, or the program moves stack
// elements.  The walk keeps (first node, need) of the subtrees on the stack in
// the lanes of one register and visits neither unary operators nor leaves right
// before their operator; a node's place moves by the other operand's size for
// each reordered operator above it.
// (Node by node, 60,000 programs of up to 128 nodes x 16,384 cases took 1,598 us a
// call; like this 1,560.)
template <bool EXT>
__device__ __forceinline__ bool reorder(const uint32_t* __restrict__ nodes, int len, int lane, uint32_t* out)
{
    uint32_t w[2];
    int pos[2];
    uint64_t leaves[2], bins[2], may[2], rev[2];
    bool moves = false;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int k = h * 64 + lane;
        w[h] = k < len ? nodes[k] : 0xFFu;
        pos[h] = k;
        const uint32_t op = w[h] & 0xFFu;
        leaves[h] = __ballot(op <= GP_CONST);
        may[h] = __ballot(op - GP_ADD < 4u);
        bins[h] = may[h] | (EXT ? __ballot(op == GP_POW) : 0ull);
        rev[h] = 0ull;
        if (EXT)
            moves |= __ballot(k < len && op >= GP_DUP && op != GP_POW && !op_is_unary(op)) != 0ull;
    }
    if (moves) return false;
    // leaves right before their operator, and those operators
    const uint64_t fl[2] = {leaves[0] & (bins[0] >> 1 | bins[1] << 63), leaves[1] & bins[1] >> 1};
    const uint64_t fb[2] = {fl[0] << 1, fl[1] << 1 | fl[0] >> 63};
    int st = 0, sp = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        for (uint64_t todo = (leaves[h] & ~fl[h]) | bins[h]; todo != 0ull; todo &= todo - 1ull) {
            const int b = __builtin_ctzll(todo), i = h * 64 + b;
            const uint64_t bit = todo & (0ull - todo);
            if ((leaves[h] & bit) != 0ull) {
                st = lane == sp ? i << 8 | 1 : st;
                ++sp;
                continue;
            }
            const int r = lane_value(st, sp - 1);
            if ((fb[h] & bit) != 0ull) {
                // the right operand is a leaf: at least two cells
                if ((r & 255) == 1) st += lane == sp - 1 ? 1 : 0;
                continue;
            }
            const int l = lane_value(st, sp - 2);
            const int sr = i - (r >> 8), sl = (r >> 8) - (l >> 8), nr = r & 255, nl = l & 255;
            int need = nl > nr ? nl : nr + 1;
            if (nr > nl && (may[h] & bit) != 0ull) {
                need = nr;
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const uint32_t k = (uint32_t)(q * 64 + lane - (l >> 8));
                    pos[q] += k < (uint32_t)sl ? sr : (k - (uint32_t)sl < (uint32_t)sr ? -sl : 0);
                }
                rev[h] |= bit;
            }
            --sp;
            st = lane == sp - 1 ? (l & ~255) | need : st;
        }
    }
    if ((rev[0] | rev[1]) == 0ull) return false;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint32_t op = w[h] & 0xFFu;
        const bool turned = ((rev[h] >> lane) & 1ull) != 0ull && (op == GP_SUB || op == GP_DIV);
        if (h * 64 + lane < len) out[pos[h]] = op - GP_ADD < 4u ? op | (turned ? kReversed : 0u) : w[h];
    }
    return true;
}

// Stages program nodes[0, len) into dst; with `turned` the nodes are those of
// reorder() (in LDS).  Every argument is uniform in the wavefront.  status, cls (depth class) and the word count come back; dst
// holds the words when the status is GP_PROG_OK (else nothing useful), never
// more than len of them.  PACKED: a null dst stores nothing.
template <bool EXT, bool PACKED>
__device__ __forceinline__ int stage_wave(const uint32_t* __restrict__ nodes, const uint32_t* turned, int32_t len,
                                          const float* __restrict__ consts, int64_t n_consts,
                                          uint32_t allowed, int32_t n_vars,
                                          uint2* __restrict__ dst, WaveTables* tb, int lane,
                                          int* cls, int* n_words, int* cost)
{
    int extra = 0;                         // what the operators take beyond a word each
    int depth = 0, rt_in = 0, n = 0;       // after the chunks before: stack, runtime, words
    int live_in = 0;                       // held variables
    bool prev_load = false;
    float prev_value = 0.f;                // value at the chunk's previous node
    int over8 = 0, over16 = 0;
    const bool store = !PACKED || dst != nullptr;
    uint2 held = make_uint2(0u, 0u);       // the last word so far, not yet stored
    int held_at = -1;
    GclCheck gc;                           // the named variables' cells (EXT)
    const bool many = len > 64;
    if (many && lane < kDepthSlots) tb->last[lane] = 0u;
    for (int32_t c0 = 0; c0 < len; c0 += 64) {
        const int32_t k = c0 + lane;
        const bool live = k < len;
        uint32_t w = 0xFFu, nw = 0xFFu;
        if (turned) {
            if (live) w = turned[k];
            if (k + 1 < len) nw = turned[k + 1];
        } else {
            if (live) w = nodes[k];
            if (k + 1 < len) nw = nodes[k + 1];
        }
        const uint32_t op = w & 0xFFu, arg = w >> 8, nx = nw & 0xFFu;
        const bool leaf = op <= GP_CONST, load = op == GP_LOAD, cst = op == GP_CONST;
        const bool bin = op - GP_ADD < 4u, un = op - GP_SIN < 6u;       // folded operators
        const bool rev = turned && bin && arg != 0u, next_rev = turned && nx - GP_ADD < 4u && nw > 0xFFu;
        const bool pw = EXT && op == GP_POW;
        const bool copy = EXT && op == GP_COPY, paste = EXT && op == GP_PASTE;
        const bool push = leaf || (EXT && op == GP_DUP) || paste;
        const bool pop = bin || pw || (EXT && op == GP_DEL);
        const uint64_t pushes = __ballot(push), pops = __ballot(pop);
        const int d0 = depth + (int)lanes_below(pushes) - (int)lanes_below(pops);
        const int d1 = d0 + (push ? 1 : 0) - (pop ? 1 : 0);
        int used = d1;                           // cells in use after the node
        uint32_t cells = 0u;                     // a variable move's cells
        bool unpaired = false;
        int copies = 0, pastes = 0;
        if constexpr (EXT) {
            const uint64_t cm = __ballot(copy), pm = __ballot(paste);
            used += live_in + (int)lanes_below(cm) - (int)lanes_below(pm) + (copy ? 1 : 0) - (paste ? 1 : 0);
            copies = (int)__popcll(cm);
            pastes = (int)__popcll(pm);
            // (past a program's first broken node the state means nothing)
            for (uint64_t mv = cm | pm; mv != 0ull; mv &= mv - 1ull) {
                const int l = __builtin_ctzll(mv);
                const uint32_t name = (uint32_t)lane_value((int)arg, l);
                const bool is_copy = ((cm >> l) & 1ull) != 0ull;
                const bool held_var = name < GP_GCL_VARS && ((gc.held >> name) & 1u);
                const bool ok = name < GP_GCL_VARS && held_var != is_copy;
                uint32_t c = 0u;
                if (ok && is_copy) {
                    c = 31u - (uint32_t)gc.copy(name);
                } else if (ok) {
                    const int q = gc.var_pos(name), from = gc.paste(name);
                    c = (31u - (uint32_t)q) | ((31u - (uint32_t)(from >= 0 ? from : q)) << 8);
                }
                cells = lane == l ? c : cells;
                unpaired = lane == l ? !ok : unpaired;
            }
        }
        // the checks of the serial walk; the first failing node names the status
        int need = leaf || paste ? 0 : (bin || pw || (EXT && op == GP_SWAP) ? 2 : 1);
        int code = used > GP_MAX_STACK ? GP_PROG_TOO_DEEP : GP_PROG_OK;
        code = unpaired ? GP_PROG_BAD_PAIR : code;
        code = d0 < need ? GP_PROG_UNDERFLOW : code;
        code = cst && (int64_t)arg >= n_consts ? GP_PROG_BAD_CONST : code;
        code = load && (int64_t)arg >= (int64_t)n_vars ? GP_PROG_BAD_VAR : code;
        code = op < 32u && ((allowed >> (op & 31u)) & 1u) ? code : GP_PROG_BAD_OP;
        const uint64_t bad = __ballot(live && code != GP_PROG_OK);
        if (bad != 0ull) return lane_value(code, __builtin_ctzll(bad));
        // (clocks per word and four cases: 24 for the cheapest, division, sine and
        // cosine four to five times that, the other functions two to three)
        extra += 3 * (int)__popcll(__ballot(op == GP_DIV)) + 4 * (int)__popcll(__ballot(op - GP_SIN < 2u)) +
                 2 * (int)__popcll(__ballot(op - GP_SIN - 2u < 3u));
        if constexpr (EXT) extra += 12 * (int)__popcll(__ballot(pw || (live && op >= GP_CBRT && op_is_unary(op))));
        over8 |= __ballot(live && used > 8) != 0ull;
        over16 |= __ballot(live && used > 16) != 0ull;

        // runtime depth after and before each node
        const bool beyond = EXT && live && op >= GP_DUP;
        const uint64_t loads = __ballot(load), solid = EXT ? __ballot(load || beyond) : loads;
        const int sigma = (int)lanes_below(solid) + (load || beyond ? 1 : 0);
        const int r1 = min(rt_in, prefix_min(live ? d1 - 64 * sigma : INT_MAX)) + 64 * sigma;
        const int rp = __shfl_up(r1, 1);        // (every lane takes part)
        const int r0 = lane == 0 ? rt_in : rp;
        const int np = d0 - r0;
        const bool after_load = lane == 0 ? prev_load : ((loads >> (lane - 1)) & 1ull) != 0ull;
        const bool fused = after_load && (bin || un || pw);
        bool own = load || (!fused && ((bin && np < 2) || (un && np < 1)));
        if constexpr (EXT) own = own || (beyond && !fused && !(op == GP_DEL && d0 < 2));
        own = own && live;

        // constants, then the folded operators in order
        float val = cst ? consts[arg] : 0.f;
        // value at the last node before lane l that left the stack at depth d
        auto at_depth = [&](int d, int l) {
            const uint64_t m = __ballot(live && d1 == d) & ((1ull << l) - 1ull);
            return m != 0ull ? lane_value(val, 63 - __builtin_clzll(m)) : tb->value[d];
        };
        const uint64_t revs = __ballot(rev);
        uint64_t folds = __ballot(live && !fused && ((bin && np >= 2) || (un && np >= 1)));
        while (folds != 0ull) {
            const int l = __builtin_ctzll(folds);
            folds &= folds - 1ull;
            const uint32_t fo = (uint32_t)lane_value((int)op, l);
            const float b = l > 0 ? lane_value(val, l - 1) : prev_value;
            float r;
            if (fo <= GP_DIV) {
                const float a = at_depth(lane_value(d0, l) - 1, l > 0 ? l - 1 : 0);
                const bool t = ((revs >> l) & 1ull) != 0ull;
                r = binary_value(fo, t ? b : a, t ? a : b);
            } else {
                r = unary_value(fo, b);
            }
            val = lane == l ? r : val;
        }

        // words: a variable (or a command that is not folded) flushes the
        // constants held below it, then each node's own word
        int pos = n + (int)lanes_below(__ballot(own));
        int flushed = 0;
        uint64_t flushes = __ballot(live && np > 0 && (load || (beyond && !(pw && np == 1))));
        while (flushes != 0ull) {
            const int l = __builtin_ctzll(flushes);
            flushes &= flushes - 1ull;
            const int cnt = lane_value(np, l), rt = lane_value(r0, l);
            const int at = lane_value(pos, l);
            for (int i = 0; i < cnt; ++i) {
                const float v = at_depth(rt + 1 + i, l);
                if (lane == 0 && store) dst[at + i] = ThreadedWords::push_const(rt + i, __float_as_uint(v));
            }
            pos += lane >= l ? cnt : 0;
            flushed += cnt;
        }
        const float pv = __shfl_up(val, 1);
        const float top = lane == 0 ? prev_value : pv;
        uint2 word;
        if (load) {
            const uint32_t payload = arg * kVarPayload;
            const int rt = d0;                   // everything below is on the stack now
            word = next_rev                    ? ThreadedWords::row_top(rt, nx - GP_ADD, payload)
                   : nx - GP_ADD < 4u          ? ThreadedWords::top_row(rt, nx - GP_ADD, payload)
                   : EXT && nx == GP_POW       ? ThreadedWords::top_row(rt, kBinPow, payload)
                   : nx - GP_SIN < 6u          ? ThreadedWords::push_unary(rt, nx - GP_SIN, payload)
                                               : ThreadedWords::push_row(rt, payload);
        } else if (bin || pw) {
            const uint32_t sel = pw ? kBinPow : op - GP_ADD;
            if (rev)
                word = np == 1 ? ThreadedWords::const_top(r0, sel, __float_as_uint(top))
                               : ThreadedWords::cells_top(r0, sel);
            else
                word = np == 1 ? ThreadedWords::top_const(r0, sel, __float_as_uint(top))
                               : ThreadedWords::cells(pw ? d0 : r0, sel);
        } else if (EXT && beyond && !op_is_unary(op)) {
            const uint32_t off = op == GP_DUP    ? kThDup
                                 : op == GP_SWAP ? kThSwap
                                 : op == GP_DEL  ? kThDel
                                 : copy          ? kThCopy
                                                 : kThPaste;
            word = ThreadedWords::move(d0, off, cells);
        } else {
            word = ThreadedWords::unary(beyond ? d0 : r0, un || beyond ? uop_sel(op) : 0u);
        }
        // the chunk's last own word is stored once it is known whether
        // another follows
        const uint64_t owns = __ballot(own);
        if (owns != 0ull) {
            if (held_at >= 0 && lane == 0 && store) dst[held_at] = held;
            const int l = 63 - __builtin_clzll(owns);
            if (own && lane != l && store) dst[pos] = word;
            held = make_uint2((uint32_t)lane_value((int)word.x, l), (uint32_t)lane_value((int)word.y, l));
            held_at = lane_value(pos, l);
        }
        n += (int)__popcll(owns) + flushed;
        const int end = min(63, len - 1 - c0);
        depth = lane_value(d1, end);
        rt_in = lane_value(r1, end);
        prev_value = lane_value(val, end);
        prev_load = ((loads >> end) & 1ull) != 0ull;
        live_in += copies - pastes;
        if (many && c0 + 64 < len) {
            // the last node of each depth, for the chunks that follow
            atomicMax(&tb->last[d1], (uint32_t)k + 1u);
            if (tb->last[d1] == (uint32_t)k + 1u) tb->value[d1] = val;
        }
    }
    if (depth != 1) return GP_PROG_FINAL_DEPTH;
    if (live_in != 0) return GP_PROG_BAD_PAIR;
    if (rt_in == 0) {
        // what is left is a constant: its value is pushed
        if (held_at >= 0 && lane == 0 && store) dst[held_at] = held;
        held = ThreadedWords::push_const(0, __float_as_uint(prev_value));
        held_at = n;
        ++n;
    }
    if (lane == 0 && store) dst[held_at] = ThreadedWords::last(held);
    *cls = over16 ? 2 : over8;
    *n_words = n;
    *cost = n + extra;
    return GP_PROG_OK;
}

// The same program by one lane, node by node: the words, class and cost of
// stage_wave, a lane's worth of time instead of a wavefront's.  Returns
// kLeftToWave for a program that holds back more than kLaneHeld constants or
// that stage_program may reorder.  Else dst holds the words that come back and
// none beyond them; a null dst stores nothing.  held: this lane's constants,
// kLaneStride floats apart.
constexpr int kLaneHeld = 8, kLaneStride = 64;
constexpr int kLeftToWave = -1;
template <bool EXT>
__device__ __forceinline__ int stage_lane(const uint32_t* __restrict__ nodes, int32_t len,
                                          const float* __restrict__ consts, int64_t n_consts,
                                          uint32_t allowed, int32_t n_vars, uint2* __restrict__ dst,
                                          lds_f32* held, int64_t n_cases, int* cls, int* n_words, int* cost)
{
    const bool store = dst != nullptr;
    GclCheck gc;
    int rt = 0, np = 0, n = 0, extra = 0;   // runtime depth, held constants, words, cost beyond a word each
    uint2 last = make_uint2(0u, 0u);
    bool joined = false;                   // the node before was a variable that took this operator
    uint32_t w = nodes[0];
    for (int32_t k = 0; k < len; ++k) {
        const uint32_t nw = k + 1 < len ? nodes[k + 1] : 0xFFu;
        const uint32_t op = w & 0xFFu, arg = w >> 8, nx = nw & 0xFFu;
        w = nw;
        uint32_t cells = 0u;                 // PASTE: where the variable was, and what moves there
        if (EXT && op == GP_PASTE) {
            const int q = gc.var_pos(arg & (GP_GCL_VARS - 1u)), low = gc.live - 1;
            cells = (31u - (uint32_t)q) | (31u - (uint32_t)low) << 8;
        }
        const int code = gc.step(op, arg, allowed, n_vars, n_consts);
        if (code != GP_PROG_OK) return code;
        const bool bin = op - GP_ADD < 4u, un = op - GP_SIN < 6u, pw = EXT && op == GP_POW;
        extra += op == GP_DIV ? 3 : (op - GP_SIN < 2u ? 4 : (op - GP_SIN - 2u < 3u ? 2 : 0));
        if (EXT) extra += pw || (op >= GP_CBRT && op_is_unary(op)) ? 12 : 0;
        if (joined) {
            joined = false;
            continue;
        }
        if (op == GP_CONST) {
            if (np == kLaneHeld) return kLeftToWave;
            held[np * kLaneStride] = consts[arg];
            ++np;
            continue;
        }
        if (bin && np >= 2) {
            --np;
            held[(np - 1) * kLaneStride] = binary_value(op, held[(np - 1) * kLaneStride], held[np * kLaneStride]);
            continue;
        }
        if (un && np >= 1) {
            held[(np - 1) * kLaneStride] = unary_value(op, held[(np - 1) * kLaneStride]);
            continue;
        }
        if (!bin && !(pw && np == 1)) {      // (a folded function over no constant flushes none)
            for (int i = 0; i < np; ++i) {
                if (store) dst[n] = ThreadedWords::push_const(rt, __float_as_uint(held[i * kLaneStride]));
                ++n;
                ++rt;
            }
            np = 0;
        }
        int change = 0;
        if (op == GP_LOAD) {
            const uint32_t payload = arg * kVarPayload;
            joined = true;
            if (nx - GP_ADD < 4u) {
                last = ThreadedWords::top_row(rt, nx - GP_ADD, payload);
            } else if (EXT && nx == GP_POW) {
                last = ThreadedWords::top_row(rt, kBinPow, payload);
            } else {
                joined = nx - GP_SIN < 6u;
                last = joined ? ThreadedWords::push_unary(rt, nx - GP_SIN, payload)
                              : ThreadedWords::push_row(rt, payload);
                change = 1;
            }
        } else if (bin || pw) {
            const uint32_t sel = pw ? kBinPow : op - GP_ADD;
            last = np == 1 ? ThreadedWords::top_const(rt, sel, __float_as_uint(held[0])) : ThreadedWords::cells(rt, sel);
            change = np == 1 ? 0 : -1;
            np = 0;
        } else if (EXT && op >= GP_DUP && !op_is_unary(op)) {
            const uint32_t off = op == GP_DUP    ? kThDup
                                 : op == GP_SWAP ? kThSwap
                                 : op == GP_DEL  ? kThDel
                                 : op == GP_COPY ? kThCopy
                                                 : kThPaste;
            if (op == GP_COPY) cells = 31u - (uint32_t)gc.var_pos(arg);
            change = op == GP_DUP || op == GP_PASTE ? 1 : (op == GP_DEL ? -1 : 0);
            if (op == GP_DEL && rt < 2) {    // the only element: nothing to move
                --rt;
                continue;
            }
            last = ThreadedWords::move(rt, off, cells);
        } else {
            last = ThreadedWords::unary(rt, uop_sel(op));
        }
        if (store) dst[n] = last;
        ++n;
        rt += change;
    }
    const int code = gc.finish();
    if (code != GP_PROG_OK) return code;
    const int c = gc.maxd > 16 ? 2 : (gc.maxd > 8 ? 1 : 0);
    if (c != 0 && n_cases >= kReorderCases && len <= kReorderMax) return kLeftToWave;
    if (np != 0) {
        // what is left is a constant: its value is pushed
        last = ThreadedWords::push_const(0, __float_as_uint(held[0]));
        ++n;
    }
    if (store) dst[n - 1] = ThreadedWords::last(last);
    *cls = c;
    *n_words = n;
    *cost = n + extra;
    return GP_PROG_OK;
}

// Stages one program: in the order written, and where that needs more than 8
// cells again in Sethi-Ullman order.  cls: the depth class by the order written
// decides the unit in which cases are summed (class_k), so the class of a
// program with more than 16 cells stays, and *narrow says that its words fit
// the first class's handlers.
// dst has room for len words, and holds what the order written needs on the
// way.  PACKED: it has room for the words that come back only (the order written
// can need nearly twice as many: a leaf right before its operator joins it), so
// a program that may be reordered is walked without stores until its order is
// known.
template <bool EXT, bool PACKED>
__device__ __forceinline__ int stage_program(const uint32_t* __restrict__ nodes, int32_t len,
                                             const float* __restrict__ consts, int64_t n_consts,
                                             uint32_t allowed, int32_t n_vars, uint2* __restrict__ dst,
                                             WaveTables* tb, int64_t n_cases, uint32_t* turned, int lane, int* cls,
                                             int* n_words, int* cost, bool* narrow)
{
    const uint32_t* from = nullptr;
    int first = -1;
    const bool may_turn = n_cases >= kReorderCases && len <= kReorderMax;
    bool known = !may_turn;                // the order to store
    *narrow = false;
    for (;;) {
        int c = 0;
        const int status = stage_wave<EXT, PACKED>(nodes, from, len, consts, n_consts, allowed, n_vars,
                                                   PACKED && !known ? nullptr : dst, tb, lane, &c, n_words, cost);
        if (first >= 0) {
            *cls = first == 2 ? 2 : c;
            *narrow = first == 2 && c == 0;
            return status;
        }
        *cls = c;
        if (status != GP_PROG_OK || (PACKED && known)) return status;
        if (c == 0 || !may_turn || !reorder<EXT>(nodes, len, lane, turned)) {
            if (!PACKED) return status;
            known = true;
            continue;
        }
        first = c;
        from = turned;
        known = true;
        // the words are written again, the nodes read back by other lanes
        wave_settle();
    }
}
