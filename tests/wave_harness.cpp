// Host harness for the staging of one program by one wavefront
// (paper_2607_06731_amd/csrc/stage_waves.h), built by tests/test_wave_staging.py
// with the host compiler (also under ASan and UBSan).
//
// TEST INFRASTRUCTURE.  The wavefront's 64 lanes are 64 contexts that run in
// turn; a wavefront operation (a ballot, a lane's value, a scan, an LDS atomic)
// hands over to the next lane and goes on when every lane has come to it, and
// fails when two lanes meet at different operations.  The words are run by an
// evaluator written here (one value per cell and case), the nodes by a plain
// stack machine with the same host functions, and the two compared bit for bit.
//
// Per program: stage_program stores words in the program's own range of
// `nodes` words only, and names the class, the words' count and their depths.
// Then all programs again as after offsets that decrease: packed one after the
// other in a buffer of exactly the words counted, in an order of `seed`; every
// program's words have to be those of the first time.
//
// Input (binary, little endian): int64 P, n_nodes, n_consts, n_vars, n_cases
// (evaluated), data_cases (what the staging is told), ext, mask, seed; uint32
// nodes[n_nodes]; int64 offsets[P + 1]; float consts[n_consts];
// float X[n_vars][n_cases].
// Output: per program int64 {status, class, words, narrow, kept_range,
// words_ok, cases_differing, same_when_packed, by_lane}; then float
// out[P][n_cases].  by_lane: 1 where stage_lane gives the same status, words,
// class and cost, 2 where it leaves the program to a wavefront.
#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>

#include <ucontext.h>
#if defined(__SANITIZE_ADDRESS__)
#include <sanitizer/common_interface_defs.h>
#endif

#define __host__
#define __device__
#define __forceinline__ inline
#include "gpeval.h"

using std::max;
using std::min;

// ------------------------------------------------------------- the lanes
static constexpr int kLanes = 64;
static constexpr size_t kStack = 256 * 1024;

struct Lane {
    ucontext_t ctx;
    std::vector<char> stack;
    void* fake = nullptr;
    bool done = false;
    int at = 0;                         // the operation it waits in
    unsigned turn = 0;
};
static Lane g_lanes[kLanes];
static ucontext_t g_main;
static void* g_main_fake = nullptr;
static const void* g_main_stack = nullptr;
static size_t g_main_size = 0;
static int g_lane = 0;
static uint64_t g_slot[2][kLanes];

static void hand_over(bool last)
{
    const int l = g_lane;
#if defined(__SANITIZE_ADDRESS__)
    __sanitizer_start_switch_fiber(last ? nullptr : &g_lanes[l].fake, g_main_stack, g_main_size);
#endif
    if (last) setcontext(&g_main);
    swapcontext(&g_lanes[l].ctx, &g_main);
#if defined(__SANITIZE_ADDRESS__)
    __sanitizer_finish_switch_fiber(g_lanes[l].fake, &g_main_stack, &g_main_size);
#endif
}

// Every lane's `v` at this operation.
static const uint64_t* together(int op, uint64_t v)
{
    Lane& L = g_lanes[g_lane];
    const unsigned t = L.turn++ & 1u;
    g_slot[t][g_lane] = v;
    L.at = op;
    hand_over(false);
    return g_slot[t];
}

static void (*g_body)();
static void lane_main()
{
#if defined(__SANITIZE_ADDRESS__)
    __sanitizer_finish_switch_fiber(nullptr, &g_main_stack, &g_main_size);
#endif
    g_body();
    g_lanes[g_lane].done = true;
    hand_over(true);
}

static void run_wave(void (*body)())
{
    g_body = body;
    for (Lane& L : g_lanes) {
        L.stack.resize(kStack);
        getcontext(&L.ctx);
        L.ctx.uc_stack.ss_sp = L.stack.data();
        L.ctx.uc_stack.ss_size = kStack;
        L.ctx.uc_link = nullptr;
        makecontext(&L.ctx, lane_main, 0);
        L.done = false;
        L.at = 0;
        L.turn = 0;
    }
    for (bool any = true; any;) {
        for (g_lane = 0; g_lane < kLanes; ++g_lane) {
            Lane& L = g_lanes[g_lane];
            if (L.done) continue;
#if defined(__SANITIZE_ADDRESS__)
            __sanitizer_start_switch_fiber(&g_main_fake, L.stack.data(), kStack);
#endif
            swapcontext(&g_main, &L.ctx);
#if defined(__SANITIZE_ADDRESS__)
            __sanitizer_finish_switch_fiber(g_main_fake, nullptr, nullptr);
#endif
        }
        any = !g_lanes[0].done;
        for (const Lane& L : g_lanes)
            if (L.done != g_lanes[0].done || L.turn != g_lanes[0].turn || L.at != g_lanes[0].at) {
                std::fprintf(stderr, "lanes meet at different operations\n");
                std::exit(3);
            }
    }
}

// ------------------------------------------------- wavefront operations
static inline uint32_t __float_as_uint(float f)
{
    uint32_t u;
    memcpy(&u, &f, 4);
    return u;
}
static inline float __uint_as_float(uint32_t u)
{
    float f;
    memcpy(&f, &u, 4);
    return f;
}
static inline int __popcll(uint64_t v) { return __builtin_popcountll(v); }
static uint64_t __ballot(bool b)
{
    const uint64_t* v = together(1, b);
    uint64_t m = 0;
    for (int l = 0; l < kLanes; ++l) m |= v[l] << l;
    return m;
}
static uint32_t lanes_below(uint64_t m) { return (uint32_t)__popcll(m & ((1ull << g_lane) - 1ull)); }
static int lane_value(int v, int l)
{
    const uint64_t* a = together(2, (uint64_t)(uint32_t)v | (uint64_t)(uint32_t)l << 32);
    for (int k = 0; k < kLanes; ++k)
        if ((int)(a[k] >> 32) != l || l < 0 || l >= kLanes) {
            std::fprintf(stderr, "lane_value of lane %d, %d\n", l, (int)(a[k] >> 32));
            std::exit(3);
        }
    return (int)(uint32_t)a[l];
}
static float lane_value(float v, int l) { return __uint_as_float((uint32_t)lane_value((int)__float_as_uint(v), l)); }
static int __shfl_up(int v, int n)
{
    const uint64_t* a = together(3, (uint32_t)v);
    return (int)(uint32_t)a[g_lane >= n ? g_lane - n : g_lane];
}
static float __shfl_up(float v, int n) { return __uint_as_float((uint32_t)__shfl_up((int)__float_as_uint(v), n)); }
static int prefix_min(int v)
{
    const uint64_t* a = together(4, (uint32_t)v);
    int m = INT_MAX;
    for (int k = 0; k <= g_lane; ++k) m = min(m, (int)(uint32_t)a[k]);
    return m;
}
static uint32_t atomicMax(uint32_t* p, uint32_t v)
{
    const uint32_t old = *p;
    *p = max(old, v);
    together(5, 0);
    return old;
}
static void wave_settle() { together(6, 0); }

// ------------------------------------------------------ host operators
static inline float div_protected(float a, float b) { return fabsf(b) <= 0.001f ? 1.f : a / b; }
static inline float binary_value(uint32_t op, float a, float b)
{
    switch (op) {
    case GP_ADD: return a + b;
    case GP_SUB: return a - b;
    case GP_MUL: return a * b;
    case GP_POW: return powf(a, b);
    default: return div_protected(a, b);
    }
}
static inline float unary_value(uint32_t op, float x)
{
    switch (op) {
    case GP_SIN: return sinf(x);
    case GP_COS: return cosf(x);
    case GP_EXP: return expf(x);
    case GP_LOG: return fabsf(x) <= 0.001f ? 0.f : logf(fabsf(x));
    case GP_SQRT: return sqrtf(fabsf(x));
    case GP_ABS: return fabsf(x);
    case GP_SQUARE: return x * x;
    case GP_SIGN: return -x;
    case GP_CUBE: return (float)((double)x * (double)x * (double)x);
    case GP_CBRT: return cbrtf(x);
    case GP_TAN: return tanf(x);
    case GP_ASIN: return asinf(x);
    case GP_ACOS: return acosf(x);
    case GP_ATAN: return atanf(x);
    case GP_TANH: return tanhf(x);
    default: return x < 0.f ? NAN : sqrtf(x);
    }
}

typedef float lds_f32;
constexpr int kHeldConsts = 16, kBucketBlock = 1;       // of the serial walks, not run here
#define GP_STAGING_FN
#include "staging.h"
#include "threaded.h"
#include "stage_waves.h"

// ---------------------------------------------------- the words' evaluator
struct Words {
    const uint2* code;
    int n, maxd;                        // words; cells of the class's handlers
};
// Runs the words on one case; false: a word that no handler of the class has.
static bool run_words(const Words& w, const float* X, int64_t n_cases, int64_t n_vars, int64_t c, float* result)
{
    float cell[33], var[32];
    for (float& v : cell) v = NAN;
    for (float& v : var) v = NAN;
    int d = 0, live = 0;
    for (int k = 0; k < w.n; ++k) {
        const uint32_t x = w.code[k].x, y = w.code[k].y;
        const bool cold = x < kThHot0;
        const uint32_t off = cold ? x % kThCold : (x - kThHot0) % kThHot;
        const int start = cold ? 32 - (int)(x / kThCold) : (int)((x - kThHot0) / kThHot) - 1;
        const bool last = k == w.n - 1;
        if (start != (last ? -1 : d)) return false;
        float leaf = __uint_as_float(y);
        auto row = [&] {
            if (y % kVarPayload != 0u || (int64_t)(y / kVarPayload) >= n_vars) return false;
            leaf = X[(int64_t)(y / kVarPayload) * n_cases + c];
            return true;
        };
        // op: 0..3 the binary operators, 4 POW; `turned`: the top is the left operand
        auto with_leaf = [&](uint32_t sel, bool turned) {
            if (d < 1 || d + 1 > w.maxd) return false;
            const uint32_t op = sel == 4u ? (uint32_t)GP_POW : GP_ADD + sel;
            cell[d - 1] = turned ? binary_value(op, leaf, cell[d - 1]) : binary_value(op, cell[d - 1], leaf);
            return true;
        };
        auto with_cells = [&](uint32_t sel, bool turned) {
            if (d < 2) return false;
            const uint32_t op = sel == 4u ? (uint32_t)GP_POW : GP_ADD + sel;
            cell[d - 2] = turned ? binary_value(op, cell[d - 1], cell[d - 2]) : binary_value(op, cell[d - 2], cell[d - 1]);
            --d;
            return true;
        };
        auto push = [&](float v) {
            if (d + live + 1 > w.maxd) return false;
            cell[d++] = v;
            return true;
        };
        bool ok = false;
        if (!cold) {
            if (off == kThPushC) ok = push(leaf);
            else if (off == kThPushV) ok = row() && push(leaf);
            else if (off >= kThBin && off < kThBin + 256u && off % 64u == 0u) ok = with_cells((off - kThBin) / 64u, false);
            else if (off == kThSubR || off == kThDivR) ok = with_cells(off == kThSubR ? 1u : 3u, true);
            else if (off >= kThBinC && off <= kThBinC + 192u && (off - kThBinC) % 64u == 0u) ok = with_leaf((off - kThBinC) / 64u, false);
            else if (off >= kThBinV && off <= kThBinV + 288u && (off - kThBinV) % 96u == 0u) ok = row() && with_leaf((off - kThBinV) / 96u, false);
            else if (off == kThSubCR || off == kThDivCR) ok = with_leaf(off == kThSubCR ? 1u : 3u, true);
            else if (off == kThSubVR || off == kThDivVR) ok = row() && with_leaf(off == kThSubVR ? 1u : 3u, true);
            else if (off >= kThPushUn && (off - kThPushUn) % 64u == 0u && off - kThPushUn < 384u)
                ok = row() && push(unary_value(GP_SIN + (off - kThPushUn) / 64u, leaf));
            else
                for (uint32_t u = 0; u < 6u; ++u)
                    if (off == ((uint32_t)(kThUnary >> (8u * u)) & 0xFFu) * 32u && d >= 1) {
                        cell[d - 1] = unary_value(GP_SIN + u, cell[d - 1]);
                        ok = true;
                    }
        } else {
            const uint32_t o = off + kThColdBit;
            if (o == kThDup) ok = d >= 1 && push(cell[d - 1]);
            else if (o == kThSwap) {
                ok = d >= 2;
                if (ok) std::swap(cell[d - 1], cell[d - 2]);
            } else if (o == kThDel) {
                ok = d >= 2;
                --d;
            } else if (o == kThCopy) {
                ok = d >= 1 && d + live + 1 <= w.maxd && (y & 31u) == 31u - (uint32_t)live;
                if (ok) var[live++] = cell[d - 1];
            } else if (o == kThPaste) {
                const int q = 31 - (int)(y & 31u), from = 31 - (int)((y >> 8) & 31u);
                ok = live >= 1 && q < live && (from == q || from == live - 1);
                if (ok) {
                    const float v = var[q];
                    var[q] = var[from];
                    --live;
                    ok = push(v);
                }
            } else if (o == kThPow) ok = with_cells(4u, false);
            else if (o == kThPowC) ok = with_leaf(4u, false);
            else if (o == kThPowV) ok = row() && with_leaf(4u, false);
            else if (d >= 1) {
                uint32_t op = 0;
                if (o == kThSquare) op = GP_SQUARE;
                else if (o == kThSign) op = GP_SIGN;
                else if (o == kThCube) op = GP_CUBE;
                else if (o == kThSqrtRaw) op = GP_SQRT_RAW;
                else if (o >= kThLibrary && o < kThLibrary + 48u && (o - kThLibrary) % 8u == 0u)
                    op = GP_CBRT + (o - kThLibrary) / 8u;
                ok = op != 0u;
                if (ok) cell[d - 1] = unary_value(op, cell[d - 1]);
            }
        }
        if (!ok || d > w.maxd) return false;
    }
    *result = cell[0];
    return d == 1 && live == 0;
}

// The nodes by a plain stack machine.
static float run_nodes(const uint32_t* nodes, int64_t len, const float* consts, const float* X, int64_t n_cases,
                       int64_t c)
{
    std::vector<float> st;
    float held[GP_GCL_VARS] = {};
    for (int64_t k = 0; k < len; ++k) {
        const uint32_t op = nodes[k] & 0xFFu, arg = nodes[k] >> 8;
        if (op == GP_LOAD) st.push_back(X[(int64_t)arg * n_cases + c]);
        else if (op == GP_CONST) st.push_back(consts[arg]);
        else if (op == GP_DUP) st.push_back(st.back());
        else if (op == GP_SWAP) std::swap(st[st.size() - 1], st[st.size() - 2]);
        else if (op == GP_DEL) st.pop_back();
        else if (op == GP_COPY) held[arg] = st.back();
        else if (op == GP_PASTE) st.push_back(held[arg]);
        else if (op_is_binary(op)) {
            const float b = st.back();
            st.pop_back();
            st.back() = binary_value(op, st.back(), b);
        } else st.back() = unary_value(op, st.back());
    }
    return st.back();
}

// ------------------------------------------------------- one staging call
struct Call {
    const uint32_t* nodes;
    int32_t len;
    const float* consts;
    int64_t n_consts, data_cases;
    uint32_t mask;
    int32_t n_vars;
    uint2* dst;
    WaveTables* tb;
    uint32_t* turned;
    bool ext, packed;
    int status[kLanes], cls[kLanes], n[kLanes], cost[kLanes];
    bool narrow[kLanes];
};
static Call g_call;
template <bool EXT, bool PACKED> static void stage()
{
    Call& c = g_call;
    const int l = g_lane;
    int cls = 0, n = 0, cost = 0;
    bool narrow = false;
    const int status = stage_program<EXT, PACKED>(c.nodes, c.len, c.consts, c.n_consts, c.mask, c.n_vars, c.dst,
                                                  c.tb, c.data_cases, c.turned, l, &cls, &n, &cost, &narrow);
    c.status[l] = status;
    c.cls[l] = cls;
    c.n[l] = n;
    c.cost[l] = cost;
    c.narrow[l] = narrow;
}
static void stage_call()
{
    Call& c = g_call;
    // (LDS holds what the program before left there)
    static WaveTables tables;
    static uint32_t turned[kReorderMax];
    c.tb = &tables;
    c.turned = turned;
    if (c.ext) run_wave(c.packed ? stage<true, true> : stage<true, false>);
    else run_wave(c.packed ? stage<false, true> : stage<false, false>);
    for (int l = 1; l < kLanes; ++l)
        if (c.status[l] != c.status[0] || (c.status[0] == GP_PROG_OK &&
            (c.cls[l] != c.cls[0] || c.n[l] != c.n[0] || c.cost[l] != c.cost[0] || c.narrow[l] != c.narrow[0]))) {
            std::fprintf(stderr, "lanes disagree\n");
            std::exit(3);
        }
}

template <class T> static bool rd(FILE* f, T* p, size_t n) { return fread(p, sizeof(T), n, f) == n; }
static bool same(float a, float b) { return __float_as_uint(a) == __float_as_uint(b) || (std::isnan(a) && std::isnan(b)); }

int main(int argc, char** argv)
{
    if (argc != 3) return 2;
    FILE* in = fopen(argv[1], "rb");
    if (!in) return 2;
    int64_t hd[9];
    if (!rd(in, hd, 9)) return 2;
    const int64_t P = hd[0], NN = hd[1], NCo = hd[2], NV = hd[3], NC = hd[4];
    std::vector<uint32_t> nodes(NN);
    std::vector<int64_t> off(P + 1);
    std::vector<float> consts(NCo), X(NV * NC);
    if (!rd(in, nodes.data(), NN) || !rd(in, off.data(), P + 1) || !rd(in, consts.data(), NCo) ||
        !rd(in, X.data(), NV * NC))
        return 2;
    fclose(in);
    Call& c = g_call;
    c.consts = consts.data();
    c.n_consts = NCo;
    c.n_vars = (int32_t)NV;
    c.data_cases = hd[5];
    c.ext = hd[6] != 0;
    c.mask = (uint32_t)hd[7];
    const uint2 blank = make_uint2(0xDEADBEEFu, 0xDEADBEEFu);
    auto is_blank = [&](const uint2& w) { return w.x == blank.x && w.y == blank.y; };
    std::vector<int64_t> info(P * 9, 0);
    std::vector<float> out(P * NC, NAN);
    std::vector<std::vector<uint2>> words((size_t)P);
    std::vector<int64_t> start((size_t)P + 1, 0);
    for (int64_t p = 0; p < P; ++p) {
        const int64_t len = off[p + 1] - off[p];
        int64_t* I = &info[p * 9];
        start[p + 1] = start[p];
        if (len <= 0) {
            I[0] = GP_PROG_EMPTY;
            continue;
        }
        // exactly the program's range: ASan sees a word beyond it
        std::vector<uint2> dst((size_t)len, blank);
        c.nodes = nodes.data() + off[p];
        c.len = (int32_t)len;
        c.dst = dst.data();
        c.packed = false;
        stage_call();
        I[0] = c.status[0];
        if (c.status[0] != GP_PROG_OK) {
            std::vector<float> held(kLaneHeld * kLaneStride, NAN);
            int cl, nw, co;
            const int st = c.ext ? stage_lane<true>(c.nodes, c.len, c.consts, NCo, c.mask, c.n_vars, dst.data(),
                                                    held.data(), c.data_cases, &cl, &nw, &co)
                                 : stage_lane<false>(c.nodes, c.len, c.consts, NCo, c.mask, c.n_vars, dst.data(),
                                                     held.data(), c.data_cases, &cl, &nw, &co);
            I[8] = st == kLeftToWave ? 2 : st == c.status[0];
            continue;
        }
        const int n = c.n[0];
        I[1] = c.cls[0];
        I[2] = n;
        I[3] = c.narrow[0];
        I[4] = n >= 1 && n <= len;
        if (!I[4]) continue;
        words[(size_t)p].assign(dst.begin(), dst.begin() + n);
        // the same by one lane, where it takes the program
        {
            std::vector<uint2> one((size_t)len, blank);
            std::vector<float> held(kLaneHeld * kLaneStride, NAN);
            int cl = -1, nw = -1, co = -1;
            const int st = c.ext ? stage_lane<true>(c.nodes, c.len, c.consts, NCo, c.mask, c.n_vars, one.data(),
                                                    held.data(), c.data_cases, &cl, &nw, &co)
                                 : stage_lane<false>(c.nodes, c.len, c.consts, NCo, c.mask, c.n_vars, one.data(),
                                                     held.data(), c.data_cases, &cl, &nw, &co);
            I[8] = st == kLeftToWave ? 2 : (st == GP_PROG_OK && cl == c.cls[0] && nw == n && co == c.cost[0]);
            for (int k = 0; k < n && I[8] == 1; ++k)
                I[8] = one[(size_t)k].x == dst[(size_t)k].x && one[(size_t)k].y == dst[(size_t)k].y;
            // no word beyond those, and without stores the same answer
            for (int64_t k = n; k < len && I[8] == 1; ++k) I[8] = is_blank(one[(size_t)k]);
            int c2 = -1, n2 = -1, o2 = -1;
            const int s2 = c.ext ? stage_lane<true>(c.nodes, c.len, c.consts, NCo, c.mask, c.n_vars, nullptr,
                                                    held.data(), c.data_cases, &c2, &n2, &o2)
                                 : stage_lane<false>(c.nodes, c.len, c.consts, NCo, c.mask, c.n_vars, nullptr,
                                                     held.data(), c.data_cases, &c2, &n2, &o2);
            if (s2 != st || (st == GP_PROG_OK && (c2 != cl || n2 != nw || o2 != co))) I[8] = 0;
        }
        const Words w{words[(size_t)p].data(), n, c.narrow[0] ? 8 : 8 << c.cls[0]};
        I[5] = 1;
        for (int64_t k = 0; k < NC; ++k) {
            float v = NAN;
            if (!run_words(w, X.data(), NC, NV, k, &v)) I[5] = 0;
            out[p * NC + k] = v;
            I[6] += !same(v, run_nodes(c.nodes, len, consts.data(), X.data(), NC, k));
        }
        start[p + 1] += n;
    }
    // packed, in any order: what one program's staging writes beyond its words
    // spoils another's
    std::vector<int64_t> turn;
    for (int64_t p = 0; p < P; ++p)
        if (!words[(size_t)p].empty()) turn.push_back(p);
    std::mt19937_64 rng((uint64_t)hd[8]);
    std::shuffle(turn.begin(), turn.end(), rng);
    std::vector<uint2> all((size_t)start[P] + 4096, blank);
    for (const int64_t p : turn) {
        c.nodes = nodes.data() + off[p];
        c.len = (int32_t)(off[p + 1] - off[p]);
        c.dst = all.data() + start[p];
        c.packed = true;
        stage_call();
        if (c.n[0] != (int)words[(size_t)p].size()) return 4;
    }
    bool beyond = false;
    for (size_t k = (size_t)start[P]; k < all.size(); ++k) beyond = beyond || !is_blank(all[k]);
    for (const int64_t p : turn) {
        const std::vector<uint2>& w = words[(size_t)p];
        bool eq = !beyond;
        for (size_t k = 0; k < w.size(); ++k) {
            const uint2& v = all[(size_t)start[p] + k];
            eq = eq && v.x == w[k].x && v.y == w[k].y;
        }
        info[p * 9 + 7] = eq;
    }
    FILE* o = fopen(argv[2], "wb");
    if (!o) return 2;
    fwrite(info.data(), sizeof(int64_t), info.size(), o);
    fwrite(out.data(), sizeof(float), out.size(), o);
    fclose(o);
    return 0;
}
