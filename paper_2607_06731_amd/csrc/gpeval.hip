// gpeval.hip -- gfx950 kernels and C ABI of the batched fitness evaluator.
//
// Path of one scoring call (all on the caller's stream):
//   k_tables         calls of several requests: one workgroup checks the
//                    dataset and request tables, lays the requests out back
//                    to back and derives tile shapes (a single request's
//                    entries travel as kernel arguments).
//   k_stage_lanes    calls of many short programs: one lane per program does
//                    what k_stage_waves does with a wavefront, and leaves long
//                    and deep programs to it.
//   k_stage_waves    one wavefront per program: validate (GCL stack
//                    discipline, 32-cell limit, opcode/operand ranges,
//                    allowed ops) and stage each instruction as one 8-byte
//                    word (the address of its handler and a payload,
//                    threaded.h) in the program's own node range, folding
//                    constant subtrees and a leaf into the operator after
//                    it; depth class and partition key; key counts per block.
//   k_order          stable scatter of program ids by (depth class, length
//                    band), longest first; class ranges and (for a single
//                    request) its per-class work-item tables.
//   k_seg_tables     several requests: per (class, request) program counts,
//                    positions and work-item prefixes.
//   k_run<FIT, SPLIT>       persistent workgroups take (program chunk, case tiles)
//                    items of every depth class (max depth <= 8, <= 16,
//                    <= 32) from an atomic counter; the tiles' inputs and
//                    targets are staged in LDS; each wavefront takes the
//                    chunk's programs one at a time and runs one over
//                    sub-tiles of cases (4, 2 or 1 per lane) with the value
//                    stack in VGPRs (threaded code, interp_gfx950.h); the
//                    fitness epilogue is fused (MSE: scaled square with Kahan
//                    accumulation; correlation: shifted fp64 sums over valid
//                    pairs; integer reward: int64 per case; gp_predict: the
//                    outputs themselves) and a wave shuffle tree gives one
//                    partial per (program, tile).
//   k_reduce[_corr|_reward]  one thread per program: its tile partials in
//                    fixed order, then the score.
// gp_mc_rank runs k_rank, or k_rank_sample and k_rank_assign for samples
// beyond 256.
//
// Semantics follow the paper's GCL section (RPN stack machine, 32-element
// stack, command table operand order) and the protected-operator readings
// stated in gpeval.h.  One program per wavefront keeps the opcode stream
// wave-uniform (the paper's divergence argument, Sec. "Avoiding Thread
// Divergence", moved from a block to a wavefront).

#include "gpeval.h"

#include <hip/hip_runtime.h>

#include <cfloat>
#include <climits>
#include <cmath>
#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <array>
#include <map>
#include <vector>
#include <mutex>
#include <string>
#include <utility>

namespace {

// ------------------------------------------------------------------ errors
thread_local std::string g_last_error;

int set_error(int code, const char* fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_last_error = buf;
    return code;
}

}  // namespace

// Shared with the other translation units of the library (not exported).
__attribute__((visibility("hidden"))) void gp_internal_set_error(int code, const char* msg)
{
    (void)code;
    g_last_error = msg;
}

namespace {

#define GP_HIP_TRY(expr)                                                      \
    do {                                                                      \
        hipError_t e_ = (expr);                                               \
        if (e_ != hipSuccess)                                                 \
            return set_error(GP_E_HIP, "%s failed: %s", #expr,                \
                             hipGetErrorString(e_));                          \
    } while (0)

// ------------------------------------------------------------------ layout
#include "run_shape.h"

// Bands of a program's cost, four per octave from 8 to 128 words' worth: an
// item's programs are of one band, so its wavefronts end together.  (Eight
// bands of one octave of length each: at 10,000 programs x 4,096 cases the
// wavefronts waited 14% of the time at barriers for the longest.)
constexpr int kLenBuckets = 16;
constexpr int kKeys = kClasses * kLenBuckets;
constexpr int kMaxRequests = 4096;       // requests per batched call (tables are scanned by one workgroup)

// Per-program record written by the staging passes.
struct ProgMeta {
    int64_t start;      // first staged instruction
    int32_t len;        // node count (the length taxed)
    int32_t slen;       // staged instructions (0: not staged), and kNarrow
};
constexpr int32_t kNarrow = INT32_MIN;   // class 2, but the words need at most 8 cells
static_assert(sizeof(ProgMeta) == 16, "ProgMeta layout");

// Power-of-two pre-scale s = 2^-e with 4^e >= n: every scaled partial sum
// of squared residuals is then <= MSE, so it overflows fp32 only when the
// MSE itself is beyond FLT_MAX.
__host__ __device__ inline int scale_exponent(int64_t n)
{
    int e = 0;
    while ((int64_t(1) << (2 * e)) < n) ++e;
    return e;
}

// ---------------------------------------------------- datasets, segments
// Dataset entry as the kernels use it (derived on the device each call).
struct DevDataset {
    const float* X;
    const float* y;
    int64_t ld_x;
    int64_t n_cases;
    double tax;
    double unscale;                 // 4^e / n_cases
    float scale;                    // 2^-e
    int32_t n_vars;
    int32_t passes[kClasses];
    int32_t n_tiles[kClasses];
    int32_t window[kClasses];
};

// A dataset's derived entry (n_cases >= 1).
__host__ __device__ inline DevDataset make_dataset(const gp_dataset& in, int32_t tile_lds, int32_t tile_max)
{
    DevDataset o;
    const int e = scale_exponent(in.n_cases);
    o.X = in.X;
    o.y = in.y;
    o.ld_x = in.ld_x;
    o.n_cases = in.n_cases;
    o.tax = in.tax_on_length;
    o.unscale = ldexp(1.0, 2 * e) / (double)in.n_cases;
    o.scale = ldexpf(1.0f, -e);
    o.n_vars = in.n_vars;
    for (int c = 0; c < kClasses; ++c) {
        const TileShape t = tile_shape(in.n_cases, class_k(c, in.n_vars), in.n_vars, tile_lds, tile_max);
        o.passes[c] = t.passes;
        o.n_tiles[c] = t.n_tiles;
        o.window[c] = t.window;
    }
    return o;
}

// Request entry as the kernels use it: the caller's entry with its
// program and node offsets inside the whole call (derived each call).
struct DevRequest {
    const uint32_t* nodes;
    const int64_t* offsets;
    const float* consts;
    int64_t n_programs;
    int64_t n_nodes;
    int64_t n_consts;
    int64_t node_base;              // first staged slot of this request
    double* out;
    int32_t* out_status;
    int32_t dataset;
};

// One workgroup: check the dataset and request tables, derive each
// dataset's tile shapes and scales, and lay the requests out one after the
// other (program starts seg_start[], staged-node bases).  With ds_in == NULL
// the single dataset `one` is used; with req_in == NULL the single request
// `one_req`.  *bad becomes 1 for inconsistent tables; then no program is
// staged and sizes are clamped so that every later index stays in range.
__global__ __launch_bounds__(256) void k_tables(
    const gp_dataset* __restrict__ ds_in, int32_t n_ds, gp_dataset one,
    const gp_request* __restrict__ req_in, int32_t n_req, gp_request one_req,
    int64_t n_programs, int64_t n_nodes, int32_t max_vars, int64_t max_cases, int32_t need_out,
    int32_t tile_lds, int32_t tile_max, DevDataset* __restrict__ ds_out, DevRequest* __restrict__ req_out,
    int32_t* __restrict__ seg_ds, int64_t* __restrict__ seg_start, int32_t* __restrict__ bad)
{
    __shared__ int s_bad;
    __shared__ int64_t s_prog[256], s_node[256];
    if (threadIdx.x == 0) s_bad = 0;
    __syncthreads();
    for (int d = threadIdx.x; d < n_ds; d += blockDim.x) {
        gp_dataset in = ds_in ? ds_in[d] : one;
        const bool ok = in.n_cases >= 1 && in.n_cases <= max_cases && in.n_vars >= 0 &&
                        in.n_vars <= max_vars && in.y != nullptr &&
                        (in.n_vars == 0 || (in.X != nullptr && in.ld_x >= in.n_cases)) &&
                        __builtin_isfinite(in.tax_on_length);
        if (!ok) {
            atomicOr(&s_bad, 1);
            in.n_cases = 1;
            in.n_vars = 0;
        }
        ds_out[d] = make_dataset(in, tile_lds, tile_max);
    }
    // each thread takes a contiguous chunk of requests: check, clamp, sum
    const int chunk = (n_req + 255) / 256;
    const int r0 = min(n_req, (int)threadIdx.x * chunk), r1 = min(n_req, r0 + chunk);
    int64_t sp = 0, sn = 0;
    for (int r = r0; r < r1; ++r) {
        const gp_request q = req_in ? req_in[r] : one_req;
        const bool ok = q.n_programs >= 0 && q.n_programs <= n_programs && q.n_nodes >= 0 &&
                        q.n_nodes <= n_nodes && q.n_consts >= 0 && q.n_consts <= GP_MAX_CONSTS &&
                        (q.n_programs == 0 || q.offsets != nullptr) &&
                        (q.n_nodes == 0 || q.nodes != nullptr) &&
                        (q.n_consts == 0 || q.consts != nullptr) &&
                        (!need_out || q.n_programs == 0 || q.out_fitness != nullptr) &&
                        q.dataset >= 0 && q.dataset < n_ds;
        if (!ok) atomicOr(&s_bad, 1);
        sp += q.n_programs >= 0 && q.n_programs <= n_programs ? q.n_programs : 0;
        sn += q.n_nodes >= 0 && q.n_nodes <= n_nodes ? q.n_nodes : 0;
    }
    s_prog[threadIdx.x] = sp;
    s_node[threadIdx.x] = sn;
    __syncthreads();
    // inclusive Hillis-Steele scan of the chunk sums
    for (int off = 1; off < 256; off <<= 1) {
        const int64_t vp = threadIdx.x >= off ? s_prog[threadIdx.x - off] : 0;
        const int64_t vn = threadIdx.x >= off ? s_node[threadIdx.x - off] : 0;
        __syncthreads();
        s_prog[threadIdx.x] += vp;
        s_node[threadIdx.x] += vn;
        __syncthreads();
    }
    if (threadIdx.x == 0 && (s_prog[255] != n_programs || s_node[255] != n_nodes))
        atomicOr(&s_bad, 1);
    int64_t pp = s_prog[threadIdx.x] - sp, pn = s_node[threadIdx.x] - sn;
    for (int r = r0; r < r1; ++r) {
        const gp_request q = req_in ? req_in[r] : one_req;
        const int64_t np = q.n_programs >= 0 && q.n_programs <= n_programs ? q.n_programs : 0;
        const int64_t nn = q.n_nodes >= 0 && q.n_nodes <= n_nodes ? q.n_nodes : 0;
        DevRequest o;
        o.nodes = q.nodes;
        o.offsets = q.offsets;
        o.consts = q.consts;
        o.n_programs = np;
        o.n_nodes = nn;
        o.n_consts = q.n_consts;
        o.node_base = pn;
        o.out = q.out_fitness;
        o.out_status = q.out_status;
        o.dataset = q.dataset >= 0 && q.dataset < n_ds ? q.dataset : 0;
        req_out[r] = o;
        seg_ds[r] = o.dataset;
        // starts beyond the call's programs are clamped: such a table is bad
        seg_start[r] = pp < n_programs ? pp : n_programs;
        pp += np;
        pn += nn;
    }
    if (threadIdx.x == 0) seg_start[n_req] = n_programs;
    __syncthreads();
    if (threadIdx.x == 0) *bad = s_bad;
}

// ------------------------------------------------------------------ sin/cos
// Constants from gen_sin_poly.py: minimax odd polynomial of degree 9 for sin
// on |r| <= pi/2 + 0.01 (relative error 6.8e-9 before fp32 evaluation) and
// a three-part fp32 split of pi for Cody-Waite reduction.  Measured against
// correctly rounded results: <= 1.75 ulp for |x| <= 2^17, including inputs
// next to multiples of pi; larger or non-finite inputs take the library
// path (which carries a Payne-Hanek reduction).
constexpr float kSinC0 = -1.666665971e-01f;
constexpr float kSinC1 = 8.333066478e-03f;
constexpr float kSinC2 = -1.980943489e-04f;
constexpr float kSinC3 = 2.605112741e-06f;
constexpr float kPiA = 3.141592741e+00f;
constexpr float kPiB = -8.742277657e-08f;
constexpr float kPiC = -3.430249020e-15f;
constexpr float kInvPi = 3.183098733e-01f;
constexpr float kTrigFastLimit = 131072.0f;
// 1.5 * 2^23: adding it to |v| < 2^22 rounds v to an integer n (the value's
// spacing there is 1) and leaves n's parity in the lowest significand bit.
constexpr float kRoundInt = 12582912.0f;

// sin(r) for |r| <= pi/2 (+ margin)
__device__ __forceinline__ float sin_poly(float r)
{
    const float u = r * r;
    float q = fmaf(u, kSinC3, kSinC2);
    q = fmaf(u, q, kSinC1);
    q = fmaf(u, q, kSinC0);
    return fmaf(u * r, q, r);
}

// r = x - kh * pi in three fused steps (exact first step for |x| <= 2^17)
__device__ __forceinline__ float reduce_pi(float x, float kh)
{
    float r = fmaf(-kh, kPiA, x);
    r = fmaf(-kh, kPiB, r);
    return fmaf(-kh, kPiC, r);
}

// Flips the sign of s when the integer held in the low bit of t's
// significand is odd (adding the bit at position 31 flips the sign bit).
__device__ __forceinline__ float flip_if_odd(float s, float t)
{
    return __uint_as_float(__float_as_uint(s) + (__float_as_uint(t) << 31));
}

// sin x = (-1)^k sin(x - k pi), k = the integer nearest x / pi
__device__ __forceinline__ float sin_fast(float x)
{
    const float t = fmaf(x, kInvPi, kRoundInt);
    const float k = t - kRoundInt;
    return flip_if_odd(sin_poly(reduce_pi(x, k)), t);
}

// cos x = (-1)^(k+1) sin(x - (k + 1/2) pi), k = the integer nearest
// x / pi - 1/2; t carries k + 1 (the offset is odd, so the parity is k+1's)
__device__ __forceinline__ float cos_fast(float x)
{
    const float t = fmaf(x, kInvPi, -0.5f) + (kRoundInt + 1.0f);
    const float k = t - (kRoundInt + 1.0f);
    return flip_if_odd(sin_poly(reduce_pi(x, k + 0.5f)), t);
}

// ---------------------------------------------------------------------- exp
// e^x = 2^(x log2 e): h = fp32(x log2 e), n = the integer nearest h, and
// 2^((h - n) + (x log2 e - h)) from the hardware exp2 on |f| <= 1/2 + tiny,
// scaled by 2^n; log2 e is split into an fp32 head and tail so the product
// keeps about 48 bits.  For |x| <= 87 no step overflows or underflows (the
// scaled result stays a normal number); other inputs take ROCm's expf.
constexpr float kLog2eHi = 1.442695022e+00f;   // fp32(log2 e), 0x3fb8aa3b
constexpr float kLog2eLo = 1.925963034e-08f;   // fp32(log2 e - kLog2eHi), 0x32a57060
constexpr float kExpFastLimit = 87.0f;

__device__ __forceinline__ float exp_fast(float x)
{
    const float h = x * kLog2eHi;
    const float n = rintf(h);
    const float f = (h - n) + fmaf(x, kLog2eLo, fmaf(x, kLog2eHi, -h));
    return ldexpf(__builtin_amdgcn_exp2f(f), (int)n);
}

// --------------------------------------------------------- sqrt|a|, ln|a|
// sqrt|a| with the hardware square root (faithful, <= 1 ulp); magnitudes
// below 2^-100 are scaled by 2^64 first (and the root by 2^-32 after), so
// no denormal reaches the instruction.
constexpr float kSqrtTiny = 0x1p-100f;
__device__ __forceinline__ float sqrt_abs(float a)
{
    const float x = fabsf(a);
    const bool tiny = x < kSqrtTiny;
    const float r = __builtin_amdgcn_sqrtf(tiny ? x * 0x1p64f : x);
    return tiny ? r * 0x1p-32f : r;
}

// Protected logarithm: 0 for |a| <= fp32(0.001), else ln|a| =
// log2|a| * ln 2 with ln 2 split into an fp32 head (rounded toward zero)
// and a positive fp32 tail, so log2|a| = +inf gives +inf + +inf = +inf.
// The hardware log2 only ever sees |a| > 0.001 (never a denormal); NaN
// propagates (the comparison with the threshold is false for NaN).
constexpr float kLn2Hi = 6.931471229e-01f;    // fp32 below ln 2
constexpr float kLn2Lo = 5.769998879e-08f;    // fp32(ln 2 - kLn2Hi) > 0
__device__ __forceinline__ float log_protected(float a)
{
    const float x = fabsf(a);
    const float l2 = __builtin_amdgcn_logf(x);
    const float ln = fmaf(l2, kLn2Hi, l2 * kLn2Lo);
    return x <= 0.001f ? 0.f : ln;
}

// ------------------------------------------------------ scalar op values
// Protected division (the divisor threshold is fp32(0.001)); shared by the
// interpreter and by constant folding, so both give the same bits.
__device__ __forceinline__ float div_protected(float a, float b)
{
    return fabsf(b) <= 0.001f ? 1.f : a / b;
}

// Per-case values of the elementary functions: the fast formula inside its
// range, the library function outside.  Constant folding uses the inline
// forms.  The interpreter calls the out-of-line forms, only when some case
// of a wavefront is outside a fast range (it takes the fast formulas
// directly otherwise): out of line, their per-case range tests are not
// merged into the interpreter's wavefront-wide tests (which would keep the
// per-case results live across the branch) and their library reductions
// do not raise the interpreter's register count.  Both forms run the same
// arithmetic, so they give the same bits.
__device__ __forceinline__ float sin_value_inl(float x)
{
    return fabsf(x) <= kTrigFastLimit ? sin_fast(x) : sinf(x);
}
__device__ __forceinline__ float cos_value_inl(float x)
{
    return fabsf(x) <= kTrigFastLimit ? cos_fast(x) : cosf(x);
}
__device__ __forceinline__ float exp_value_inl(float x)
{
    return fabsf(x) <= kExpFastLimit ? exp_fast(x) : expf(x);
}
__attribute__((noinline)) __device__ float sin_value(float x) { return sin_value_inl(x); }
__attribute__((noinline)) __device__ float cos_value(float x) { return cos_value_inl(x); }
__attribute__((noinline)) __device__ float exp_value(float x) { return exp_value_inl(x); }
__attribute__((noinline)) __device__ float sqrt_value(float x) { return sqrt_abs(x); }

// The rest of the command table: ROCm's fp32 library functions, out of
// line (the full-table interpreter calls them per case; constant folding
// calls the same functions, so both give the same bits).  SQRT_RAW is the
// benchmark set's root with NaN below zero.
__attribute__((noinline)) __device__ float cbrt_value(float x) { return cbrtf(x); }
__attribute__((noinline)) __device__ float tan_value(float x) { return tanf(x); }
__attribute__((noinline)) __device__ float asin_value(float x) { return asinf(x); }
__attribute__((noinline)) __device__ float acos_value(float x) { return acosf(x); }
__attribute__((noinline)) __device__ float atan_value(float x) { return atanf(x); }
__attribute__((noinline)) __device__ float tanh_value(float x) { return tanhf(x); }
__attribute__((noinline)) __device__ float pow_value(float a, float b) { return powf(a, b); }
__attribute__((noinline)) __device__ float sqrt_raw_value(float x)
{
    return x < 0.f ? __builtin_nanf("") : sqrt_abs(x);
}

// One operator of the benchmark set on one value, exactly as the
// interpreter computes it for a case (used to fold constant subtrees while
// staging; the commands beyond the set are not folded, so staging makes no
// calls).
__device__ __forceinline__ float binary_value(uint32_t op, float a, float b)
{
    switch (op) {
    case GP_ADD: return a + b;
    case GP_SUB: return a - b;
    case GP_MUL: return a * b;
    default: return div_protected(a, b);
    }
}

__device__ __forceinline__ float unary_value(uint32_t op, float x)
{
    switch (op) {
    case GP_SIN: return sin_value_inl(x);
    case GP_COS: return cos_value_inl(x);
    case GP_EXP: return exp_value_inl(x);
    case GP_LOG: return log_protected(x);
    case GP_SQRT: return sqrt_abs(x);
    default: return fabsf(x);
    }
}

// Pointers to memory that is constant while a kernel runs: loads at uniform
// addresses are scalar loads, also past an asm statement (which the compiler
// takes as writing any ordinary memory).
template <class T> using const_ptr = const __attribute__((address_space(4))) T*;
template <class T> __device__ __forceinline__ const_ptr<T> as_const(const T* p)
{
    return (const_ptr<T>)(uintptr_t)p;
}

// ------------------------------------------------------------- staging
typedef __attribute__((address_space(3))) float lds_f32;
#include "staging.h"
#include "threaded.h"
#include "interp_gfx950.h"

// ------------------------------------------------ wavefront primitives
__device__ __forceinline__ uint32_t lanes_below(uint64_t mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}
__device__ __forceinline__ int lane_value(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ __forceinline__ float lane_value(float v, int l)
{
    return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(v), l));
}

// Minimum over lanes 0..own (row shifts inside 16 lanes, then two row
// broadcasts).
__device__ __forceinline__ int prefix_min(int v)
{
    constexpr int big = INT_MAX;
    v = min(v, __builtin_amdgcn_update_dpp(big, v, 0x111, 0xf, 0xf, false));   // row_shr:1
    v = min(v, __builtin_amdgcn_update_dpp(big, v, 0x112, 0xf, 0xf, false));   // row_shr:2
    v = min(v, __builtin_amdgcn_update_dpp(big, v, 0x114, 0xf, 0xf, false));   // row_shr:4
    v = min(v, __builtin_amdgcn_update_dpp(big, v, 0x118, 0xf, 0xf, false));   // row_shr:8
    v = min(v, __builtin_amdgcn_update_dpp(big, v, 0x142, 0xa, 0xf, false));   // row_bcast:15
    v = min(v, __builtin_amdgcn_update_dpp(big, v, 0x143, 0xc, 0xf, false));   // row_bcast:31
    return v;
}

// Everything a lane has written is there for the wavefront's other lanes.
__device__ __forceinline__ void wave_settle()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
}

#include "stage_waves.h"

// Per staging block: programs per partition key, and whether some program's
// offsets decrease.
struct StageRow {
    uint16_t cnt[kKeys];
    uint16_t down, pad;
};
static_assert(sizeof(StageRow) == 100, "StageRow layout");
constexpr int kStageWaves = 8;
constexpr int kStageBlocks = 1024;       // two workgroups of 8 wavefronts on every SIMD pair
constexpr int kStageRound = 1024;        // programs that a block looks through for those left to it
constexpr int kLaneWG = 256;
// Keys beyond the partition's: an invalid program, one whose offsets decrease,
// one that k_stage_lanes leaves to k_stage_waves.
constexpr uint8_t kKeyInvalid = 0xFF, kKeyDown = 0xFE, kKeyLeft = 0xFD;

// Programs per staging block: one per wavefront up to 8,192 programs, then
// as many as keep the grid at 1,024 blocks (a count fits 16 bits).
inline int64_t stage_share(int64_t n_programs)
{
    const int64_t c = (n_programs + kStageBlocks - 1) / kStageBlocks;
    return c < kStageWaves ? kStageWaves : (c > 32768 ? 32768 : c);
}

inline int64_t stage_blocks(int64_t n_programs)
{
    const int64_t share = stage_share(n_programs);
    return (n_programs + share - 1) / share;
}

// Nodes of a program that one lane stages, at most (0: every program takes a
// wavefront).  A wavefront's walk costs about the same for any program of up to 64
// nodes, 64 lanes' walks the time of the longest: lanes win where programs are
// short, but only when there are enough of them to fill the GPU with lanes, from
// about 4,000 per node of mean length.  (us per call over 100 cases by
// wavefronts and by lanes; programs of 1-3 nodes: 10,000 53.8 and 51.7, 1,000,000
// 1,101 and 430; of 3-8: 20,000 76.5 and 73.3, 10,000 54.7 and 60.7; of 3-20: 50,000
// 125 and 115, 20,000 79 and 91; of 3-64: 200,000 453 and 396, 100,000 266 and 266,
// 50,000 172 and 215.)
constexpr int32_t kLaneNodes = 64;
inline int32_t lane_nodes(int64_t n_programs, int64_t n_nodes)
{
    return (double)n_programs * (double)n_programs >= 4000.0 * (double)n_nodes ? kLaneNodes : 0;
}

// What the staging kernels share.  A call of one request brings its
// request and dataset entries by value (block 0 writes the tables that the
// later kernels read); a call of several has them in memory (k_tables).
struct StageArgs {
    int64_t n_programs, share;
    uint32_t allowed;
    int32_t single, lpt, n_seg;
    int32_t lane_nodes;             // nodes of a program that one lane stages, at most
    DevRequest one_req;
    DevDataset one_ds;
    DevDataset* ds;
    DevRequest* reqs;
    int32_t* seg_ds;
    int64_t* seg_start;
    int32_t* bad;
    ProgMeta* meta;
    uint8_t* cls;
    int32_t* pds;                   // request of each program (NULL: one request)
    int32_t* order;
    uint2* code;
    StageRow* rows;
    unsigned long long* words;      // staged words of each staging block
};

struct ProgRange {
    const uint32_t* nodes;
    const float* consts;
    int64_t n_consts, node_base, s, e;
    int32_t* out_status;
    int64_t n_nodes;
    int64_t n_cases;
    int32_t n_vars;
    int r;
};
// Program p's request fields and node range (all uniform).
template <class Args>
__device__ __forceinline__ ProgRange program_range(Args a, int64_t p, bool tab_ok)
{
    ProgRange g;
    g.s = g.e = 0;
    if (a->single) {
        g.r = 0;
        g.nodes = a->one_req.nodes;
        g.consts = a->one_req.consts;
        g.n_consts = a->one_req.n_consts;
        g.node_base = 0;
        g.n_nodes = a->one_req.n_nodes;
        g.n_vars = a->one_ds.n_vars;
        g.n_cases = a->one_ds.n_cases;
        g.out_status = a->one_req.out_status ? a->one_req.out_status + p : nullptr;
        g.s = as_const(a->one_req.offsets)[p];
        g.e = as_const(a->one_req.offsets)[p + 1];
        return g;
    }
    const const_ptr<int64_t> start = as_const((const int64_t*)a->seg_start);
    int lo = 0, hi = a->n_seg - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (start[mid] <= p) lo = mid; else hi = mid - 1;
    }
    const const_ptr<DevRequest> R = as_const((const DevRequest*)a->reqs) + lo;
    const int64_t q = p - start[lo];
    g.r = lo;
    g.nodes = R->nodes;
    g.consts = R->consts;
    g.n_consts = R->n_consts;
    g.node_base = R->node_base;
    g.n_nodes = R->n_nodes;
    g.n_vars = as_const((const DevDataset*)a->ds)[R->dataset].n_vars;
    g.n_cases = as_const((const DevDataset*)a->ds)[R->dataset].n_cases;
    g.out_status = R->out_status && q < R->n_programs ? R->out_status + q : nullptr;
    if (tab_ok) {
        g.s = as_const(R->offsets)[q];
        g.e = as_const(R->offsets)[q + 1];
    }
    return g;
}

// The same pointer, opaque to the optimizer: what is read through it is read
// there, not kept in scalar registers from the loop's start.
template <class T> __device__ __forceinline__ const_ptr<T> again(const_ptr<T> p)
{
    asm volatile("" : "+s"(p));
    return p;
}

// Nodes of a program, at most: the interpreter's offset of the word after the next
// (8 bytes each, never more words than nodes) has 32 bits.
constexpr int64_t kMaxNodes = (int64_t(1) << 29) - 16;

// The status that program g's range alone gives (GP_PROG_OK: look at its nodes).
__device__ __forceinline__ int range_status(const ProgRange& g, bool tab_ok)
{
    const bool ok = g.s >= 0 && g.e >= g.s && g.e <= g.n_nodes && g.e - g.s <= kMaxNodes;
    return !tab_ok ? GP_PROG_BAD_TABLE : (!ok ? GP_PROG_BAD_OFFSETS : (g.e == g.s ? GP_PROG_EMPTY : GP_PROG_OK));
}

// Program p's record and status, by one lane; returns its partition key: depth
// class, then (single-request calls) cost band from dearest to cheapest; with
// several requests the order inside a class stays the input order, so each
// request's programs stay together.
template <class Args>
__device__ __forceinline__ int put_program(Args a, int64_t p, const ProgRange& g, int status, int c,
                                           int n, int cost, bool narrow)
{
    if (status != GP_PROG_OK) {
        c = -1;
        n = 0;
    }
    ProgMeta m;
    m.start = g.node_base + g.s;
    m.len = (int32_t)(status == GP_PROG_BAD_OFFSETS || status == GP_PROG_BAD_TABLE ? 0 : g.e - g.s);
    m.slen = narrow ? n | kNarrow : n;
    a->meta[p] = m;
    if (a->pds) a->pds[p] = g.r;
    const uint32_t w = (uint32_t)(cost > 1 ? cost : 1), z = __clz(w);
    int lb = (int)(((31u - z) << 2) + ((w << z) >> 29 & 3u)) - 12;      // 4 log2(w / 8)
    lb = lb < 0 ? 0 : (lb < kLenBuckets ? lb : kLenBuckets - 1);
    const int key = c >= 0 ? c * kLenBuckets + (a->lpt ? kLenBuckets - 1 - lb : 0) : kKeyInvalid;
    a->cls[p] = (uint8_t)key;
    if (g.out_status) *g.out_status = status;
    return key;
}

// Pass 1 of calls of many programs, before k_stage_waves: a lane stages a program
// of up to a.lane_nodes nodes (stage_lane) and leaves others to it.
template <bool EXT>
__global__ __launch_bounds__(kLaneWG) void k_stage_lanes(StageArgs a)
{
    __shared__ float held[kLaneWG / 64][kLaneHeld * kLaneStride];
    const int64_t p = (int64_t)blockIdx.x * kLaneWG + threadIdx.x;
    if (p >= a.n_programs) return;
    const bool tab_ok = a.single || as_const((const int32_t*)a.bad)[0] == 0;
    const ProgRange g = program_range(&a, p, tab_ok);
    int status = range_status(g, tab_ok), c = -1, n = 0, cost = 0;
    if (status == GP_PROG_OK)
        status = g.e - g.s > a.lane_nodes
                     ? kLeftToWave
                     : stage_lane<EXT>(g.nodes + g.s, (int32_t)(g.e - g.s), g.consts, g.n_consts, a.allowed,
                                       g.n_vars, a.code + g.node_base + g.s,
                                       (lds_f32*)&held[threadIdx.x >> 6][threadIdx.x & 63], g.n_cases, &c, &n, &cost);
    if (status == kLeftToWave) a.cls[p] = kKeyLeft;
    else (void)put_program(&a, p, g, status, c, n, cost, false);
    if (g.e < g.s) a.cls[p] = kKeyDown;
}

// Pass 1, one wavefront per program: validate and
// stage each program at its own node offset in the request's part of `code`
// (its words never outnumber its nodes, so while offsets never decrease the
// programs' ranges are disjoint), and count the partition keys per block.
// The block's wavefronts take its programs one by one: a reordered program takes
// several times a plain one's time.  64 registers, so that all 1,024 blocks are
// resident (at 80 a quarter of them waited for a second round).  A call of
// 100,000 programs x 4,096 cases: 1,137 us without the two, 1,099 with them.
// LANES: k_stage_lanes has run; what it left is listed and staged here.
template <bool EXT, bool LANES>
__global__ __launch_bounds__(64 * kStageWaves, 8) void k_stage_waves(StageArgs a)
{
    __shared__ int cnt[kKeys];
    __shared__ int s_down;
    __shared__ unsigned long long s_words;
    __shared__ uint32_t s_taken, s_left;
    __shared__ uint16_t left[LANES ? kStageRound : 1];
    __shared__ WaveTables tables[kStageWaves];
    __shared__ uint32_t turned[kStageWaves][kReorderMax];
    const const_ptr<StageArgs> args = (const_ptr<StageArgs>)__builtin_amdgcn_kernarg_segment_ptr();
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (threadIdx.x < kKeys) cnt[threadIdx.x] = 0;
    if (threadIdx.x == 0) {
        s_down = 0;
        s_words = 0ull;
        s_taken = s_left = 0u;
    }
    if (a.single && blockIdx.x == 0 && threadIdx.x == 0) {
        a.ds[0] = a.one_ds;
        a.reqs[0] = a.one_req;
        a.seg_ds[0] = 0;
        a.seg_start[0] = 0;
        a.seg_start[1] = a.n_programs;
        a.bad[0] = 0;
    }
    __syncthreads();
    const bool tab_ok = a.single || as_const((const int32_t*)a.bad)[0] == 0;
    const int64_t p0 = (int64_t)blockIdx.x * a.share;
    const int64_t p1 = min(p0 + a.share, a.n_programs);
    for (int64_t r0 = p0, r1; r0 < p1; r0 = r1) {
        r1 = LANES ? min(r0 + kStageRound, p1) : p1;
        if (LANES) {
            if (r0 != p0) {
                __syncthreads();
                if (threadIdx.x == 0) s_taken = s_left = 0u;
                __syncthreads();
            }
            unsigned long long words = 0;
            for (int64_t p = r0 + threadIdx.x; p < r1; p += 64 * kStageWaves) {
                const int key = a.cls[p];
                if (key < kKeys) {
                    atomicAdd(&cnt[key], 1);
                    words += (unsigned long long)a.meta[p].slen;
                }
                if (key == kKeyDown) s_down = 1;
                if (key == kKeyLeft) left[atomicAdd(&s_left, 1u)] = (uint16_t)(p - r0);
            }
            if (words != 0ull) atomicAdd(&s_words, words);
            __syncthreads();
        }
        const int64_t todo = LANES ? (int64_t)s_left : r1 - r0;
        for (;;) {
            // (all lanes add one, as in k_run's claims)
            const int64_t t = (int64_t)(__builtin_amdgcn_readfirstlane(atomicAdd(&s_taken, 1u)) >> 6);
            if (t >= todo) break;
            const int64_t p = r0 + (LANES ? (int64_t)__builtin_amdgcn_readfirstlane((int)left[t]) : t);
            const const_ptr<StageArgs> ka = again(args);
            const ProgRange g = program_range(ka, p, tab_ok);
            int status = range_status(g, tab_ok), c = -1, n = 0, cost = 0;
            bool narrow = false;
            if (status == GP_PROG_OK)
                status = stage_program<EXT, false>(g.nodes + g.s, (int32_t)(g.e - g.s), g.consts, g.n_consts, ka->allowed,
                                                   g.n_vars, ka->code + g.node_base + g.s, &tables[wave], g.n_cases,
                                                   turned[wave], lane, &c, &n, &cost, &narrow);
            if (lane == 0) {
                if (g.e < g.s) s_down = 1;
                const int key = put_program(again(args), p, g, status, c, n, cost, narrow);
                if (key < kKeys) {
                    atomicAdd(&cnt[key], 1);
                    atomicAdd(&s_words, (unsigned long long)n);
                }
            }
        }
    }
    __syncthreads();
    StageRow* row = a.rows + blockIdx.x;
    if (threadIdx.x < kKeys) row->cnt[threadIdx.x] = (uint16_t)cnt[threadIdx.x];
    if (threadIdx.x == 0) {
        row->down = (uint16_t)s_down;
        a.words[blockIdx.x] = s_words;
    }
}

// Pass 2, same blocks: every block sums the key counts of the blocks before
// it (and of all), so the partition needs no scan of its own; program ids are
// scattered stably by (depth class, cost band); block 0 writes the class
// ranges, clears the work counter and, for a single request, writes its
// per-class tables (k_seg_tables' for one segment).
// Offsets that decrease somewhere let programs' node ranges overlap: then
// every program is staged again here, packed in program order, unless the
// staged programs need more than n_nodes words in total (no program of the
// call is staged then).  (us per call of 1,000,000 programs of 3-19 nodes x 100
// cases, without and with one pair that decreases: 732 and 1,025.)
struct SegOut {
    int32_t g_max, target_items, lds_floats, split, free_outputs;
    int32_t* seg_cnt;
    int32_t* seg_pos;
    uint32_t* item_pre;
    int32_t* class_g;
    int32_t* class_info;
    uint32_t* counter;
};

constexpr int kOrderWG = 256;
template <bool EXT, bool LANES>
__global__ __launch_bounds__(kOrderWG, 4) void k_order(StageArgs a, int32_t n_blk, int64_t code_capacity,
                                                    SegOut so)
{
    constexpr int kCols = (int)(sizeof(StageRow) / 4);        // pairs of counts
    constexpr int kRowStep = kOrderWG / kCols;
    __shared__ int s_all[2 * kCols], s_pre[2 * kCols];
    __shared__ int s_base[kKeys];
    __shared__ int s_chunk[kOrderWG / 64][kKeys];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    if (t < 2 * kCols) s_all[t] = s_pre[t] = 0;
    __syncthreads();
    if (t < kRowStep * kCols) {
        const uint32_t* __restrict__ rows = reinterpret_cast<const uint32_t*>(a.rows);
        const int c = t % kCols;
        int all0 = 0, all1 = 0, pre0 = 0, pre1 = 0;
        const int b = (int)blockIdx.x;
#pragma unroll 8
        for (int r = t / kCols; r < n_blk; r += kRowStep) {
            const uint32_t v = rows[(int64_t)r * kCols + c];
            all0 += (int)(v & 0xFFFFu);
            all1 += (int)(v >> 16);
            pre0 += r < b ? (int)(v & 0xFFFFu) : 0;
            pre1 += r < b ? (int)(v >> 16) : 0;
        }
        atomicAdd(&s_all[2 * c], all0);
        atomicAdd(&s_all[2 * c + 1], all1);
        atomicAdd(&s_pre[2 * c], pre0);
        atomicAdd(&s_pre[2 * c + 1], pre1);
    }
    __syncthreads();
    const bool restage = s_all[kKeys] != 0;          // StageRow::down
    const int64_t p0 = (int64_t)blockIdx.x * a.share;
    const int64_t p1 = min(p0 + a.share, a.n_programs);
    bool overflow = false;
    if (restage) {
        // staged words of all programs, and of those before this block
        __shared__ unsigned long long s_words, s_before;
        if (t == 0) s_words = s_before = 0ull;
        __syncthreads();
        unsigned long long all = 0, before = 0;
        for (int r = t; r < n_blk; r += kOrderWG) {
            const unsigned long long v = a.words[r];
            all += v;
            if (r < (int)blockIdx.x) before += v;
        }
        atomicAdd(&s_words, all);
        atomicAdd(&s_before, before);
        __syncthreads();
        overflow = (int64_t)s_words > code_capacity;
        if (!overflow) {
            __shared__ WaveTables tables[kOrderWG / 64];
            __shared__ uint32_t turned[kOrderWG / 64][kReorderMax];
            __shared__ unsigned long long s_wave[kOrderWG / 64];
            __shared__ float held[LANES ? kOrderWG / 64 : 1][kLaneHeld * kLaneStride];
            __shared__ int32_t left[kOrderWG];
            __shared__ uint32_t s_left;
            unsigned long long base = s_before;
            for (int64_t c0 = p0; c0 < p1; c0 += kOrderWG) {
                // where each of 256 programs starts now
                const int64_t p = c0 + t;
                const bool staged = p < p1 && a.cls[p] < kKeys;
                const unsigned long long v = staged ? (unsigned long long)(a.meta[p].slen & ~kNarrow) : 0ull;
                unsigned long long sum = v;
#pragma unroll
                for (int off = 1; off < 64; off <<= 1) {
                    const unsigned long long u = __shfl_up(sum, off);
                    sum += lane >= off ? u : 0ull;
                }
                if (lane == 63) s_wave[wave] = sum;
                if (t == 0) s_left = 0u;
                __syncthreads();
                unsigned long long chunk = 0;
                for (int w2 = 0; w2 < kOrderWG / 64; ++w2) {
                    if (w2 == wave) sum += base + chunk;
                    chunk += s_wave[w2];
                }
                base += chunk;
                if (staged) {
                    const int64_t start = (int64_t)(sum - v);
                    a.meta[p].start = start;
                    // as in pass 1: by this lane, or by a wavefront
                    int status = kLeftToWave;
                    if constexpr (LANES) {
                        const ProgRange g = program_range(&a, p, true);
                        int c = 0, n = 0, cost = 0;
                        if (g.e - g.s <= a.lane_nodes)
                            for (int pass = 0; pass < 2; ++pass) {
                                status = stage_lane<EXT>(g.nodes + g.s, (int32_t)(g.e - g.s), g.consts, g.n_consts,
                                                         a.allowed, g.n_vars, pass ? a.code + start : nullptr,
                                                         (lds_f32*)&held[wave][lane], g.n_cases, &c, &n, &cost);
                                if (status == kLeftToWave) break;
                            }
                    }
                    if (status == kLeftToWave) left[atomicAdd(&s_left, 1u)] = (int32_t)p;
                }
                __syncthreads();
                const int todo = (int)s_left;
                for (int q = __builtin_amdgcn_readfirstlane(wave); q < todo; q += kOrderWG / 64) {
                    const int64_t pw = __builtin_amdgcn_readfirstlane(left[q]);
                    const ProgRange g = program_range(&a, pw, true);
                    int c = 0, n = 0, cost = 0;
                    bool narrow = false;
                    (void)stage_program<EXT, true>(g.nodes + g.s, (int32_t)(g.e - g.s), g.consts, g.n_consts,
                                                   a.allowed, g.n_vars, a.code + a.meta[pw].start, &tables[wave],
                                                   g.n_cases, turned[wave], lane, &c, &n, &cost, &narrow);
                }
                __syncthreads();
            }
        }
    }
    if (t == 0) {
        int run = 0;
        for (int k = 0; k < kKeys; ++k) {
            s_base[k] = run + s_pre[k];
            run += s_all[k];
        }
    }
    if (blockIdx.x == 0 && t < kClasses) {
        int start = 0, count = 0;
        for (int k = 0; k < kKeys; ++k) {
            if (k / kLenBuckets < t) start += s_all[k];
            if (k / kLenBuckets == t) count += s_all[k];
        }
        if (overflow) count = 0;
        so.class_info[2 * t] = start;
        so.class_info[2 * t + 1] = count;
        if (t == 0) *so.counter = 0u;
        if (a.single) {
            const ClassCut cut = class_cut(t, count, a.one_ds.passes[t], a.one_ds.n_tiles[t], a.one_ds.n_cases,
                                           staged_rows(so.free_outputs != 0, a.one_ds.n_vars), so.g_max, so.target_items, so.lds_floats,
                                           so.split != 0, so.free_outputs != 0);
            so.seg_cnt[t] = count;
            so.class_g[t] = cut.G;
            so.class_g[kClasses + t] = cut.m_cap;
            so.class_g[2 * kClasses + t] = cut.split;
            so.seg_pos[t] = 0;
            so.item_pre[2 * t] = 0u;
            so.item_pre[2 * t + 1] = cut.items;
        }
    }
    if (overflow) {
        for (int64_t p = p0 + t; p < p1; p += kOrderWG) {
            if (a.cls[p] >= kKeys) continue;
            a.cls[p] = kKeyInvalid;
            const int r = a.pds ? a.pds[p] : 0;
            int32_t* st = a.single ? a.one_req.out_status : a.reqs[r].out_status;
            const int64_t q = a.single ? p : p - a.seg_start[r];
            if (st && (a.single || q < a.reqs[r].n_programs)) st[q] = GP_PROG_BAD_OFFSETS;
        }
        return;
    }
    // stable scatter, one chunk of the block's programs at a time
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    for (int64_t c0 = p0; c0 < p1; c0 += kOrderWG) {
        const int64_t p = c0 + t;
        const int key = p < p1 ? (int)a.cls[p] : 0xFF;
        if (lane < kKeys) s_chunk[wave][lane] = 0;
        int rank = 0;
        // one pass per distinct key in the wavefront
        for (uint64_t todo = __ballot(key < kKeys); todo != 0ull;) {
            const int first = __ffsll((unsigned long long)todo) - 1;
            const int k0 = __shfl(key, first);
            const uint64_t bm = __ballot(key == k0);
            if (lane == first) s_chunk[wave][k0] = __popcll(bm);
            if (key == k0) rank = __popcll(bm & below);
            todo &= ~bm;
        }
        __syncthreads();
        if (key < kKeys) {
            for (int w2 = 0; w2 < wave; ++w2) rank += s_chunk[w2][key];
            a.order[s_base[key] + rank] = (int32_t)p;
        }
        __syncthreads();
        if (t < kKeys) {
            for (int w2 = 0; w2 < kOrderWG / 64; ++w2) s_base[t] += s_chunk[w2][t];
        }
        __syncthreads();
    }
}

// Sum over the workgroup's threads (every thread gets it), and over the threads
// before this one.
constexpr int kSegWG = 256;
struct SegScan {
    unsigned long long sum[kSegWG / 64];
    uint32_t before[kSegWG / 64];
};
__device__ __forceinline__ double seg_sum(SegScan& sc, unsigned long long v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sc.sum[threadIdx.x >> 6] = v;
    __syncthreads();
    unsigned long long t = 0;
#pragma unroll
    for (int w = 0; w < kSegWG / 64; ++w) t += sc.sum[w];
    return (double)t;
}
__device__ __forceinline__ uint32_t seg_scan(SegScan& sc, uint32_t v)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t t = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t u = __shfl_up(t, off);
        t += lane >= off ? u : 0u;
    }
    __syncthreads();
    if (lane == 63) sc.before[wave] = t;
    __syncthreads();
    t -= v;
    for (int w = 0; w < wave; ++w) t += sc.before[w];
    return t;
}

// Calls of several requests, a workgroup per depth class c: the programs
// inside each segment (seg_cnt[c * n_seg + s]; the partition keeps each class in
// program order, so they are the class's entries between two lower bounds of the
// segment's program range), the cut (class_g[c], class_g[kClasses + c];
// class_g[2 kClasses + c]: cases are split), and per segment where its programs
// start inside the class's range of `order` (seg_pos) and the prefix of work
// items.  A thread takes a run of consecutive segments.  (One thread per class
// took 4,776 us for 4,096 requests of 5 programs, now 94, and 37 for 24; a single request's
// tables come from k_order.)
__global__ __launch_bounds__(kSegWG) void k_seg_tables(
    const int32_t* __restrict__ order, const int32_t* __restrict__ class_info,
    const int64_t* __restrict__ seg_start, int32_t n_seg, const int32_t* __restrict__ tables_bad,
    const int32_t* __restrict__ seg_ds, const DevDataset* __restrict__ ds, int32_t g_max,
    int32_t target_items, int32_t lds_floats, int32_t* __restrict__ seg_cnt,
    int32_t* __restrict__ seg_pos, uint32_t* __restrict__ item_pre, int32_t* __restrict__ class_g)
{
    __shared__ SegScan sc;
    const int c = blockIdx.x;
    const bool bad = *tables_bad != 0;              // then no program was staged
    const int32_t* __restrict__ ord = order + class_info[2 * c];
    const int32_t total = bad ? 0 : class_info[2 * c + 1];
    int32_t* __restrict__ pos = seg_pos + (int64_t)c * n_seg;
    // the lower bounds
    for (int s = threadIdx.x; s < n_seg; s += kSegWG) {
        const int64_t v = seg_start[s];
        int lo = 0, hi = total;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if ((int64_t)ord[mid] < v) lo = mid + 1; else hi = mid;
        }
        pos[s] = lo;
    }
    __syncthreads();
    const int chunk = (n_seg + kSegWG - 1) / kSegWG;
    const int s0 = min(n_seg, (int)threadIdx.x * chunk), s1 = min(n_seg, s0 + chunk);
    auto programs = [&](int s) { return (s + 1 < n_seg ? pos[s + 1] : total) - pos[s]; };
    unsigned long long v = 0;
    for (int s = s0; s < s1; ++s) v += (unsigned long long)programs(s) * (unsigned long long)ds[seg_ds[s]].n_tiles[c];
    const int32_t m_cap = cut_tiles(seg_sum(sc, v));
    auto groups = [&](int s) {
        const DevDataset& D = ds[seg_ds[s]];
        const int32_t m = item_tiles(D.passes[c], D.n_tiles[c], c, staged_rows(false, D.n_vars), lds_floats, m_cap);
        return item_groups(D.n_tiles[c], m);
    };
    v = 0;
    for (int s = s0; s < s1; ++s) v += (unsigned long long)programs(s) * (unsigned long long)groups(s);
    const int32_t G = cut_programs(seg_sum(sc, v), g_max, target_items);
    uint32_t items = 0;
    for (int s = s0; s < s1; ++s) items += (uint32_t)((programs(s) + G - 1) / G) * (uint32_t)groups(s);
    items = seg_scan(sc, items);
    uint32_t* __restrict__ pre = item_pre + (int64_t)c * (n_seg + 1);
    for (int s = s0; s < s1; ++s) {
        const int n = programs(s);
        seg_cnt[c * n_seg + s] = n;
        pre[s] = items;
        items += (uint32_t)((n + G - 1) / G) * (uint32_t)groups(s);
    }
    if (s0 < s1 && s1 == n_seg) pre[n_seg] = items;
    if (threadIdx.x == 0) {
        class_g[c] = G;
        class_g[kClasses + c] = m_cap;
        class_g[2 * kClasses + c] = 0;
    }
}

// ------------------------------------------------------------ evaluation
// Error-free sum: s + e == a + b exactly (Knuth's TwoSum).
__device__ __forceinline__ void two_sum(float a, float b, float& s, float& e)
{
    s = a + b;
    const float bp = s - a;
    e = (a - (s - bp)) + (b - bp);
}

// Compensated pair (hi, lo) += (h2, l2).
__device__ __forceinline__ void acc_pair(float& hi, float& lo, float h2, float l2)
{
    float s, e;
    two_sum(hi, h2, s, e);
    hi = s;
    lo = (lo + l2) + e;
}

// One case of the MSE fitness into a lane's Kahan pair (the represented sum
// is hi + lo).  ys is the target pre-scaled by the dataset's power of two s,
// so fma(f, s, -ys) is the scaled residual (f - y) s rounded once: the same
// value as rounding f - y and scaling it.  CHECK: the targets may hold NaN
// or +-inf (Sec. "Fitness Functions": invalid values in the dataset are
// handled as in Eq. 2): a case whose output and target are both invalid is
// a matched pair and adds nothing, a case where exactly one of them is
// invalid marks the program (worst fitness).  Without CHECK (every target
// finite) an invalid output needs no mark: its residual is NaN or +-inf and
// so is the lane's sum from then on, which the reduction turns into the
// worst fitness, as it does a sum that overflows.
template <bool CHECK>
__device__ __forceinline__ void mse_case(float f, float ys, float s, float& hi, float& lo,
                                         bool& bad)
{
    const float d = fmaf(f, s, -ys);
    float t = d * d;
    if constexpr (CHECK) {
        const bool fv = __builtin_isfinite(f), yv = __builtin_isfinite(ys);
        bad |= fv != yv;
        t = fv && yv ? t : 0.f;
    }
    // Kahan's compensated step (every term is >= 0, so the running sum
    // dominates the term after the first few cases)
    const float yk = t + lo;
    const float u = hi + yk;
    lo = yk - (u - hi);
    hi = u;
}

// ------------------------------------------------- threaded interpreter
// The constants its handlers read from vector registers v22..v25, made once
// per kernel: opaque to the optimizer, which would otherwise rebuild them at
// every run.
struct ThreadConsts {
    float inv_pi, sin_c3, log2e_hi, theta;
};
__device__ __forceinline__ float opaque(float v)
{
    asm volatile("" : "+v"(v));
    return v;
}
__device__ __forceinline__ ThreadConsts thread_consts()
{
    return {opaque(kInvPi), opaque(kSinC3), opaque(kLog2eHi), opaque(0.001f)};
}

// Runs one program staged as threaded words (threaded.h) on K cases per
// lane; `xl` is this lane's first case of the staged inputs, whose rows are
// `scale` * 256 cases long; the result is the stack's one element.  Handlers
// that meet a value outside their fast range, and the library commands,
// return with a code; the out-of-line function is applied here, per case,
// and the run resumes.
typedef float f32x32 __attribute__((ext_vector_type(32)));

#define GP_THREAD_TABLE(table)                                                             \
    "s_getpc_b64 s[90:91]\n"                                                              \
    "s_add_u32 s90, s90, " table "@rel32@lo+4\n"                                          \
    "s_addc_u32 s91, s91, " table "@rel32@hi+12\n"
// Loads still in flight when the statement starts would land in registers that
// the handlers use: the compiler does not wait for a load whose result is not
// read (a spilled value read back and not needed on this path), and takes the
// register as free.
#define GP_THREAD_SETTLE "s_waitcnt vmcnt(0) lgkmcnt(0)\n"
// the first word, then its handler
#define GP_THREAD_ENTER(table)                                                             \
    GP_THREAD_SETTLE "s_load_dwordx2 s[88:89], s[84:85], 0x0\n" GP_THREAD_TABLE(table)                      \
    "s_mov_b32 s86, 8\n"                                                                  \
    "s_waitcnt lgkmcnt(0)\n"                                                              \
    "s_add_u32 s92, s90, s88\n"                                                           \
    "s_addc_u32 s93, s91, 0\n"                                                            \
    "s_swappc_b64 s[94:95], s[92:93]\n"
// after a value was replaced: the finish code of the block that asked for it
#define GP_THREAD_RESUME(table)                                                            \
    GP_THREAD_SETTLE GP_THREAD_TABLE(table)                                                                 \
    "s_add_u32 s92, s90, s87\n"                                                           \
    "s_addc_u32 s93, s91, 0\n"                                                            \
    "s_swappc_b64 s[94:95], s[92:93]\n"
#define GP_THREAD_ASM(kind, table, io)                                                     \
    asm volatile(GP_THREAD_##kind(table)                                                   \
                 : "+{v[36:67]}"(cells), io "{v4}"(t[0]), io "{v5}"(t[1]), io "{v6}"(t[2]),    \
                   io "{v7}"(t[3]), "={v12}"(u[0]), "={v13}"(u[1]), "={v14}"(u[2]),         \
                   "={v15}"(u[3]), io "{s[88:89]}"(w), io "{s86}"(off), io "{s87}"(resume), \
                   "={s83}"(rc)                                                            \
                 : "{s[84:85]}"(pc), "{s82}"(scale), "{v31}"(lane_addr),                   \
                   "{v22}"(tc.inv_pi), "{v23}"(tc.sin_c3), "{v24}"(tc.log2e_hi),           \
                   "{v25}"(tc.theta)                                                       \
                 : "v8", "v9", "v10", "v11", "v16", "v17", "v18", "s68", "s69", "s70",     \
                   "s71", "s72", "s73", "s74", "s75", "s90", "s91", "s92", "s93", "s94",   \
                   "s95", "s96", "s97", "s98", "m0", "vcc", "scc", "memory")

// The function a result code asks for, on the K values v (u: the exponents).
template <int K>
__device__ __forceinline__ void threaded_call(uint32_t rc, float (&v)[4], const float (&u)[4])
{
#define GP_CALL(code, expr)                                                                \
    case code:                                                                             \
        _Pragma("unroll") for (int j = 0; j < K; ++j) v[j] = expr;                         \
        break;
    switch (rc) {
        GP_CALL(kCallSin, sin_value(v[j]))
        GP_CALL(kCallCos, cos_value(v[j]))
        GP_CALL(kCallExp, exp_value(v[j]))
        GP_CALL(kCallSqrt, sqrt_value(v[j]))
        GP_CALL(kCallCbrt, cbrt_value(v[j]))
        GP_CALL(kCallTan, tan_value(v[j]))
        GP_CALL(kCallAsin, asin_value(v[j]))
        GP_CALL(kCallAcos, acos_value(v[j]))
        GP_CALL(kCallAtan, atan_value(v[j]))
        GP_CALL(kCallTanh, tanh_value(v[j]))
        GP_CALL(kCallSqrtRaw, sqrt_raw_value(v[j]))
    default:
        _Pragma("unroll") for (int j = 0; j < K; ++j) v[j] = pow_value(v[j], u[j]);
        break;
    }
#undef GP_CALL
}

template <int MAXD, int K>
__device__ __forceinline__ void run_threaded(const uint2* code, const float* xl, uint32_t scale,
                                             const ThreadConsts& tc, float (&tos)[K])
{
    static_assert((MAXD == 8 && K == 4) || (MAXD == 16 && K == 2) || (MAXD == 32 && K == 1),
                  "the tables of interp_gfx950.h");
    const uint64_t pa = (uint64_t)(uintptr_t)code;
    const uint64_t pc = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(pa >> 32)) << 32 |
                        (uint32_t)__builtin_amdgcn_readfirstlane((int)pa);
    const uint32_t lane_addr =
        (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) float*)xl;
    f32x32 cells;                              // the stack
    float t[4], u[4];
    uint64_t w;
    uint32_t off, resume, rc;
    if constexpr (MAXD == 8) GP_THREAD_ASM(ENTER, "gp_threads_d8", "=");
    else if constexpr (MAXD == 16) GP_THREAD_ASM(ENTER, "gp_threads_d16", "=");
    else GP_THREAD_ASM(ENTER, "gp_threads_d32", "=");
    while (__builtin_expect(rc != 0u, 0)) {
        threaded_call<K>(rc, t, u);
        // (uniform; said again where the loop made them look otherwise)
        w = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(w >> 32)) << 32 |
            (uint32_t)__builtin_amdgcn_readfirstlane((int)w);
        off = (uint32_t)__builtin_amdgcn_readfirstlane((int)off);
        resume = (uint32_t)__builtin_amdgcn_readfirstlane((int)resume);
        if constexpr (MAXD == 8) GP_THREAD_ASM(RESUME, "gp_threads_d8", "+");
        else if constexpr (MAXD == 16) GP_THREAD_ASM(RESUME, "gp_threads_d16", "+");
        else GP_THREAD_ASM(RESUME, "gp_threads_d32", "+");
    }
#pragma unroll
    for (int j = 0; j < K; ++j) tos[j] = cells[j];
}

// ------------------------------------------------- correlation fitness
// Per (program, tile) sums of the correlation fitness (Eq. 1-2) over the
// valid pairs (output and target both finite), kept about a shift (s, t)
// that is itself one valid pair of the data, so a large mean cancels before
// anything is squared: n valid pairs, Sd = sum (f - s), Sdd = sum (f - s)^2,
// Se = sum (y - t), See = sum (y - t)^2, Sde = sum (f - s)(y - t) in fp64,
// and the pairs with one (c1) or both (c2) sides invalid.  A wavefront
// shares one shift per (program, window), so its lanes add plainly; windows
// and tiles merge by the exact shift-change identities, in a fixed order.
struct CorrPart {
    double s, t, sd, sdd, se, see, sde;
    int64_t n, c1, c2;
};
static_assert(sizeof(CorrPart) == 80, "CorrPart layout");

// one lane's sums over its cases of a window (the shift is the wavefront's)
struct CorrLane {
    double sd, sdd, se, see, sde;
    int32_t n, c1, c2;
};

enum : int { kFitMse = 0, kFitCorr = 1, kFitReward = 2, kFitPredict = 3 };
constexpr int kCorrMaxG = 32;            // programs per work item in correlation mode (LDS)

__device__ __forceinline__ void corr_zero(CorrPart& c)
{
    c.s = c.t = c.sd = c.sdd = c.se = c.see = c.sde = 0.0;
    c.n = c.c1 = c.c2 = 0;
}
__device__ __forceinline__ void corr_zero(CorrLane& c)
{
    c.sd = c.sdd = c.se = c.see = c.sde = 0.0;
    c.n = c.c1 = c.c2 = 0;
}

// one case: f the program's output, y the target, (s, t) the shift
__device__ __forceinline__ void corr_case(CorrLane& c, float f, float y, double s, double t)
{
    const bool fv = __builtin_isfinite(f), yv = __builtin_isfinite(y);
    if (fv && yv) {
        const double d = (double)f - s, e = (double)y - t;
        c.sd += d;
        c.sdd = fma(d, d, c.sdd);
        c.se += e;
        c.see = fma(e, e, c.see);
        c.sde = fma(d, e, c.sde);
        ++c.n;
    } else if (fv != yv) {
        ++c.c1;
    } else {
        ++c.c2;
    }
}

// Integer point-to-point reward of one case (StdFitFunc, Eq. 5, and its
// Square/Cube/Hyper variants: the ratio raised to `power`), in fp32 as the
// paper's reward function takes fp32 values: M when both are zero, else
// rint(M ratio^p), less M/11 for opposite signs; an invalid pair gives -M
// (one side invalid) or +M (both).  rint rounds half to even.
__device__ __forceinline__ long long pair_reward(float o, float y, float M, int power)
{
    const bool ov = __builtin_isfinite(o), yv = __builtin_isfinite(y);
    if (!(ov && yv)) return (ov || yv) ? -(long long)M : (long long)M;
    const float ao = fabsf(o), ay = fabsf(y);
    const float mx = ao > ay ? ao : ay, mn = ao > ay ? ay : ao;
    if (mx == 0.0f) return (long long)M;
    const float r = mn / mx;
    float rp = r;
    if (power == 2) rp = r * r;
    else if (power == 3) rp = (r * r) * r;
    else if (power == 8) { const float r2 = r * r, r4 = r2 * r2; rp = r4 * r4; }
    float v = M * rp;
    if ((o < 0.0f && y > 0.0f) || (o > 0.0f && y < 0.0f)) v = v - M / 11.0f;
    return (long long)rintf(v);
}

// a += b (fixed order: the result depends only on the two operands).  b's
// sums move to a's shift: with dl = b.s - a.s and el = b.t - a.t,
// sum (f - a.s) = Sd + n dl, sum (f - a.s)^2 = Sdd + dl (2 Sd + n dl),
// sum (f - a.s)(y - a.t) = Sde + dl Se + el (Sd + n dl), and likewise in y.
__device__ __forceinline__ void corr_merge(CorrPart& a, const CorrPart& b)
{
    a.c1 += b.c1;
    a.c2 += b.c2;
    if (b.n == 0) return;
    if (a.n == 0) {
        a.s = b.s; a.t = b.t;
        a.sd = b.sd; a.sdd = b.sdd; a.se = b.se; a.see = b.see; a.sde = b.sde;
        a.n = b.n;
        return;
    }
    const double dl = b.s - a.s, el = b.t - a.t, nb = (double)b.n;
    a.sdd += b.sdd + dl * (2.0 * b.sd + nb * dl);
    a.see += b.see + el * (2.0 * b.se + nb * el);
    a.sde += b.sde + dl * b.se + el * (b.sd + nb * dl);
    a.sd += b.sd + nb * dl;
    a.se += b.se + nb * el;
    a.n += b.n;
}

// wavefront tree: every lane ends with the same sums (one shared shift,
// and fp64 addition is commutative, so both lanes of a pair agree)
__device__ __forceinline__ void corr_wave_reduce(CorrLane& c)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        c.sd += __shfl_xor(c.sd, off);
        c.sdd += __shfl_xor(c.sdd, off);
        c.se += __shfl_xor(c.se, off);
        c.see += __shfl_xor(c.see, off);
        c.sde += __shfl_xor(c.sde, off);
        c.n += __shfl_xor(c.n, off);
        c.c1 += __shfl_xor(c.c1, off);
        c.c2 += __shfl_xor(c.c2, off);
    }
}

// ------------------------------------------------------------------ k_run
// Arguments of the evaluation kernel.
struct RunArgs {
    const uint2* code;
    const ProgMeta* meta;
    const int32_t* order;
    const int32_t* class_info;
    uint32_t* work_counter;
    const DevDataset* ds;
    const int32_t* seg_ds;
    const int32_t* seg_cnt;
    const int32_t* seg_pos;
    const uint32_t* item_pre;
    const int32_t* class_g;
    float2* part;
    uint8_t* part_bad;
    CorrPart* part_corr;    // the same memory as part, correlation mode
    float* out;             // gp_predict: per-case outputs
    int64_t ld_out;
    int32_t part_stride;    // partial of (program p, tile t) at t * part_stride + p
    int32_t n_seg;
    int32_t lds_floats;     // staged inputs and targets, at most
    int32_t reward_power;
    float reward_M, reward_less;    // M and M / 11
};

// One workgroup's item as its wavefronts see it (uniform).
struct Item {
    int64_t first;          // first case staged
    int32_t cases;          // cases staged (the last sub-tile may be partial)
    int32_t stride;         // cases per row of the staged memory (multiple of 256)
    int32_t n_vars;
    int32_t window;         // cases summed before each wavefront tree
    int32_t tile_cases;     // cases per partial; 0: the tile goes on past this piece
    int32_t tile;           // first tile
    int32_t obase, count;   // programs: order[obase .. obase + count)
    int32_t ynf;            // some staged target is NaN or infinite
    float scale;
};

// What a wavefront accumulates for one program.
template <int FIT> struct Sums;
template <> struct Sums<kFitMse> {
    float hi, lo;           // this lane's Kahan pair of the window
    float H, L;             // the tile's windows, added in order
    bool bad, tile_bad;
};
template <> struct Sums<kFitCorr> {
    CorrLane cl;
    double cs, ct;          // the window's shift
    bool have_shift;
};
template <> struct Sums<kFitReward> {
    long long rl;
};
template <> struct Sums<kFitPredict> {};

// (Per-case branches and an IEEE division each: 9,973 programs x 4,096 cases
// 255 us; this 244, and 237 with the 6 wavefronts per SIMD it leaves room for.)
// The reward of NJ ordinary cases per lane: both values nonzero, the larger
// magnitude within 2^-10 .. 2^60 and the smaller above 2^-60 (no case is
// invalid, and the ratio is formed as the interpreter's division: its steps
// are exact there), M at most 2^21 (a reward rounds by adding 1.5 * 2^23).
// False: some case is not ordinary.
template <int NJ>
__device__ __forceinline__ bool rewards(const float (&f)[NJ], const float* y, const RunArgs& a, int32_t& sum)
{
    float yv[NJ], mx[NJ], r[NJ];
    float all = 0.f, top = __builtin_inff(), low = __builtin_inff();
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        yv[j] = y[j * 64];
        const float fo = fabsf(f[j]), fy = fabsf(yv[j]);
        all += fo + fy;                                        // (NaN and infinities too)
        mx[j] = __builtin_amdgcn_fmed3f(fo, fy, __builtin_inff());
        r[j] = __builtin_amdgcn_fmed3f(fo, fy, 0.f);
        top = __builtin_amdgcn_fmed3f(top, mx[j], 0.f);        // the smallest of each
        low = __builtin_amdgcn_fmed3f(low, r[j], 0.f);
    }
    if (!(fabsf(a.reward_M) <= 0x1p21f) ||
        __ballot(!(all <= 0x1p60f && top >= 0x1p-10f && low > 0x1p-60f)) != 0ull)
        return false;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const float b = mx[j];
        float z = __builtin_amdgcn_rcpf(b);
        z = fmaf(fmaf(-b, z, 1.f), z, z);
        const float q = r[j] * z;
        r[j] = fmaf(fmaf(-b, q, r[j]), z, q);
    }
    if (a.reward_power == 2) {
#pragma unroll
        for (int j = 0; j < NJ; ++j) r[j] = r[j] * r[j];
    } else if (a.reward_power == 3) {
#pragma unroll
        for (int j = 0; j < NJ; ++j) r[j] = (r[j] * r[j]) * r[j];
    } else if (a.reward_power == 8) {
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const float r2 = r[j] * r[j], r4 = r2 * r2;
            r[j] = r4 * r4;
        }
    }
    const float M = a.reward_M, less = a.reward_less;
    sum = 0;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const uint32_t opposite = (uint32_t)((int32_t)(__float_as_uint(f[j]) ^ __float_as_uint(yv[j])) >> 31);
        const float v = M * r[j] - __uint_as_float(__float_as_uint(less) & opposite);
        sum += (int32_t)__float_as_uint(v + 0x1.8p23f) - 0x4B400000;
    }
    return true;
}

// NJ cases per lane from case `pos` of the staged piece: the fitness
// epilogue (MSE: scaled square with Kahan accumulation; correlation: shifted
// fp64 sums over valid pairs; integer reward: int64 per case), or the
// outputs themselves.
template <int FIT, int NJ>
__device__ __forceinline__ void add_cases(const float (&f)[NJ], const float* yt, int left, int lane,
                                          const RunArgs& a, const Item& it, Sums<FIT>& s, float* out)
{
    if constexpr (FIT == kFitPredict) {
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            if (lane + j * 64 < left) out[lane + j * 64] = f[j];
    } else if constexpr (FIT == kFitMse) {
        // a whole sub-tile in range with finite targets: no per-case tests
        // (wave-uniform branches)
        if (left >= NJ * 64 && !it.ynf) {
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                mse_case<false>(f[j], yt[lane + j * 64], it.scale, s.hi, s.lo, s.bad);
        } else {
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                if (lane + j * 64 < left)
                    mse_case<true>(f[j], yt[lane + j * 64], it.scale, s.hi, s.lo, s.bad);
        }
    } else if constexpr (FIT == kFitCorr) {
        // the shift: the window's first valid pair, in the order (sub-tile,
        // case, lane)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            if (!s.have_shift) {
                const float yj = yt[lane + j * 64];
                const bool v = lane + j * 64 < left && __builtin_isfinite(f[j]) && __builtin_isfinite(yj);
                const unsigned long long mk = __ballot(v);
                if (mk != 0ull) {
                    const int src = __builtin_ctzll(mk);
                    s.cs = (double)lane_value(f[j], src);
                    s.ct = (double)lane_value(yj, src);
                    s.have_shift = true;
                }
            }
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            if (lane + j * 64 < left) corr_case(s.cl, f[j], yt[lane + j * 64], s.cs, s.ct);
    } else {
        int32_t v;
        if (left >= NJ * 64 && rewards<NJ>(f, yt + lane, a, v)) {
            s.rl += v;
            return;
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j)
            if (lane + j * 64 < left)
                s.rl += pair_reward(f[j], yt[lane + j * 64], a.reward_M, a.reward_power);
    }
}

enum : int { kAll = 0, kKeep = 1, kSum = 2 };
// Runs one program of depth class C (3: of class 2, with the first class's
// handlers) over cases [from, to) of the staged piece, or keeps their outputs
// (kKeep) or sums the kept ones (kSum); acc is its
// running tile sum in LDS (correlation always; the others only when a tile
// goes on past the piece).
template <int FIT, int C, bool SPLIT>
__device__ __forceinline__ void run_piece(const uint2* pc, int pid, const float* xt, const RunArgs& a,
                                          const Item& it, const ThreadConsts& tc, int lane, void* acc,
                                          uint32_t* acc_bad, int from, int to, int mode, float* kept)
{
    if (!SPLIT || FIT == kFitPredict) mode = kAll;
    if (!SPLIT) {
        from = 0;
        to = it.cases;
    }

    constexpr int SUB = sub_cases(C == 3 ? 2 : C);
    constexpr int NJ = SUB / 64;
    const float* yt = xt + (int64_t)it.n_vars * it.stride;
    Sums<FIT> s;
    const bool goes_on = it.tile_cases == 0;
    if constexpr (FIT == kFitMse) {
        s.hi = s.lo = 0.f;
        s.bad = s.tile_bad = false;
        s.H = s.L = 0.f;
        if (goes_on) {
            const float2 v = *static_cast<const float2*>(acc);
            s.H = v.x;
            s.L = v.y;
            s.tile_bad = *acc_bad != 0u;
        }
    } else if constexpr (FIT == kFitCorr) {
        corr_zero(s.cl);
        s.cs = s.ct = 0.0;
        s.have_shift = false;
        if (!goes_on) corr_zero(*static_cast<CorrPart*>(acc));
    } else if constexpr (FIT == kFitReward) {
        s.rl = 0;
    }
    int wleft = it.window;
    int tleft = goes_on ? INT_MAX : it.tile_cases;
    int tile = it.tile;
    float* out = nullptr;
    if constexpr (FIT == kFitPredict) out = a.out + (int64_t)pid * a.ld_out + it.first;

    // after `SUB` cases ending at case `end`: close the window and the tile
    auto close = [&](int end) {
        if constexpr (FIT == kFitPredict) return;
        wleft -= SUB;
        tleft -= SUB;
        const bool stop = end >= it.cases;
        const bool tile_end = tleft == 0 || (stop && !goes_on);
        if (wleft == 0 || tile_end || stop) {
            wleft = it.window;
            if constexpr (FIT == kFitMse) {
                // wavefront tree: every lane ends with the same pair
#pragma unroll
                for (int off = 32; off >= 1; off >>= 1) {
                    const float h2 = __shfl_xor(s.hi, off);
                    const float l2 = __shfl_xor(s.lo, off);
                    acc_pair(s.hi, s.lo, h2, l2);
                }
                s.tile_bad = s.tile_bad || __ballot(s.bad) != 0ull;
                acc_pair(s.H, s.L, s.hi, s.lo);
                s.hi = s.lo = 0.f;
                s.bad = false;
            } else if constexpr (FIT == kFitCorr) {
                corr_wave_reduce(s.cl);
                // (every lane holds the same sums and writes the same value)
                CorrPart w;
                w.s = s.cs; w.t = s.ct;
                w.sd = s.cl.sd; w.sdd = s.cl.sdd; w.se = s.cl.se; w.see = s.cl.see;
                w.sde = s.cl.sde;
                w.n = s.cl.n; w.c1 = s.cl.c1; w.c2 = s.cl.c2;
                corr_merge(*static_cast<CorrPart*>(acc), w);
                corr_zero(s.cl);
                s.cs = s.ct = 0.0;
                s.have_shift = false;
            }
        }
        if (tile_end) {
            const int64_t slot = (int64_t)tile * a.part_stride + pid;
            if constexpr (FIT == kFitMse) {
                if (lane == 0) {
                    a.part[slot] = make_float2(s.H, s.L);
                    a.part_bad[slot] = (uint8_t)s.tile_bad;
                }
                s.H = s.L = 0.f;
                s.tile_bad = false;
            } else if constexpr (FIT == kFitCorr) {
                if (lane == 0) a.part_corr[slot] = *static_cast<const CorrPart*>(acc);
                corr_zero(*static_cast<CorrPart*>(acc));
            } else if constexpr (FIT == kFitReward) {
                // integers: exact in any order
#pragma unroll
                for (int off = 32; off >= 1; off >>= 1) s.rl += __shfl_xor(s.rl, off);
                if (lane == 0) reinterpret_cast<long long*>(a.part)[slot] = s.rl;
                s.rl = 0;
            }
            ++tile;
            tleft = it.tile_cases;
            wleft = it.window;
        }
    };

    for (int pos = from; pos < to;) {
        const float* xl = xt + pos + lane;
        float* kl = kept + pos + lane;
        if constexpr (C == 3) {
            // two sub-tiles at once (pos is a multiple of 256, like a row)
            float f[4];
            if (mode != kSum) run_threaded<8, 4>(pc, xl, it.stride >> 8, tc, f);
            else {
#pragma unroll
                for (int j = 0; j < 4; ++j) f[j] = kl[j * 64];
            }
            if (mode == kKeep) {
#pragma unroll
                for (int j = 0; j < 4; ++j) kl[j * 64] = f[j];
                pos += 2 * SUB;
                continue;
            }
            const float f0[2] = {f[0], f[1]}, f1[2] = {f[2], f[3]};
            add_cases<FIT, 2>(f0, yt + pos, it.cases - pos, lane, a, it, s, out + pos);
            close(pos + SUB);
            pos += SUB;
            if (pos >= it.cases) break;
            add_cases<FIT, 2>(f1, yt + pos, it.cases - pos, lane, a, it, s, out + pos);
            close(pos + SUB);
            pos += SUB;
            continue;
        }
        float f[NJ];
        constexpr int K = C == 0 ? 4 : (C == 1 ? 2 : 1);
        if (mode != kSum) {
#pragma unroll
            for (int h = 0; h < NJ; h += K) {
                float v[K];
                run_threaded<C == 0 ? 8 : (C == 1 ? 16 : 32), K>(pc, xl + h * 64, it.stride >> 8, tc, v);
#pragma unroll
                for (int j = 0; j < K; ++j) f[h + j] = v[j];
            }
        } else {
#pragma unroll
            for (int j = 0; j < NJ; ++j) f[j] = kl[j * 64];
        }
        if (mode == kKeep) {
#pragma unroll
            for (int j = 0; j < NJ; ++j) kl[j * 64] = f[j];
            pos += SUB;
            continue;
        }
        add_cases<FIT, NJ>(f, yt + pos, it.cases - pos, lane, a, it, s, out + pos);
        close(pos + SUB);
        pos += SUB;
    }
    if (goes_on) {
        if constexpr (FIT == kFitMse) {
            *static_cast<float2*>(acc) = make_float2(s.H, s.L);
            *acc_bad = s.tile_bad ? 1u : 0u;
        } else if constexpr (FIT == kFitReward) {
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) s.rl += __shfl_xor(s.rl, off);
            *static_cast<long long*>(acc) += s.rl;
        }
    }
}

// Loads the first lines (64 bytes, 8 words) of a program's code into the
// scalar cache together; met one by one they cost a wavefront a wait each.
__device__ __forceinline__ void warm_code(const uint2* pc, int words)
{
    const const_ptr<uint2> code = as_const(pc);
    const int top = words - 1;
    uint32_t w[kWarmLines];
#pragma unroll
    for (int l = 0; l < kWarmLines; ++l) w[l] = code[min(8 * l, top)].x;
#pragma unroll
    for (int l = 0; l < kWarmLines; ++l) asm volatile("" ::"s"(w[l]));
}

// LDS bytes of a workgroup's running sums: one per program of a chunk (a tile
// in pieces), or per wavefront.
constexpr int chunk_max(int fit, bool wide) { return wide ? kRunWaves : (fit == kFitCorr ? kCorrMaxG : kChunkMax); }
constexpr size_t acc_bytes(int fit, bool wide)
{
    return (size_t)chunk_max(fit, wide) *
           (fit == kFitCorr     ? sizeof(CorrPart)
            : fit == kFitReward ? sizeof(long long)
            : fit == kFitMse    ? sizeof(float2) + sizeof(uint32_t)
                                : 0);
}

// Lists programs order[obase .. obase + count) of a chunk (count <= G <= 64) in
// LDS, by one wavefront: looked up one by one, a wavefront would wait for
// three loads in turn before each.  The lanes left over touch the programs'
// code, a cache line each, so it is in this XCD's L2.
__device__ __forceinline__ uint32_t list_chunk(const RunArgs& a, int obase, int count, int G, int lane, uint4* list)
{
    const int per = 64 / G, g = lane / per, k = lane - g * per;
    uint32_t touched = 0;
    if (g < count) {
        const int pid = a.order[obase + g];
        const ProgMeta pm = a.meta[pid];
        const uint64_t at = (uint64_t)(uintptr_t)(a.code + pm.start);
        if (k == 0) list[g] = make_uint4((uint32_t)at, (uint32_t)(at >> 32), (uint32_t)pid, (uint32_t)pm.slen);
        const int words = pm.slen & ~kNarrow;
        for (int l = k; l * 16 < words; l += per) touched ^= a.code[pm.start + l * 16].x;
    }
    return touched;     // (to be consumed where the wait for it does no harm)
}

// Evaluation of every depth class in one launch.  Persistent workgroups take
// items (a chunk of programs of one class x a run of its case tiles) from a
// counter, the deepest class first and inside a class the longest programs
// first, so the launch ends on short ones.  The item's inputs and targets are
// staged in LDS, and each wavefront takes programs one at a time and runs
// each over all staged cases.  The wavefront that takes a chunk's first
// program claims the workgroup's next item and, when that is over the same
// cases, lists its programs behind the chunk's: wavefronts go on without
// meeting, up to kListed programs between two barriers.  (Barriers after
// every item left 44% of the wavefronts' time waiting; a class's kernel of its
// own left the GPU to each tail in turn and cost 13 us when it was empty.)
// WIDE: datasets of so many variables that a sub-tile leaves no room for the
// long list.
// Bound by vector issue (threaded.h).  80 registers leave six wavefronts per SIMD:
// 32 of stack, 16 of temporaries and the epilogue's; the compiler spills 23 for MSE
// and 46 for the reward, which still measured faster than fewer wavefronts
// (reward, 9,973 programs x 4,096 cases: 244 -> 237 us).  The correlation sums take
// 128 registers, four wavefronts.
template <int FIT, bool SPLIT, bool WIDE>
__global__ __launch_bounds__(kRunWG, FIT == kFitCorr ? 4 : 6) void k_run(RunArgs a)
{
    extern __shared__ __align__(16) float lds[];
    float* xt = lds;                              // [n_vars + 1][stride]: inputs, then targets
    char* accs = reinterpret_cast<char*>(lds + a.lds_floats);
    __shared__ uint32_t s_next, s_end, s_pending; // programs taken and listed; the next item
    constexpr int kList = WIDE ? 2 * kRunWaves : kListed, kChunk = chunk_max(FIT, WIDE);
    constexpr bool kNoTargets = FIT == kFitPredict;
    __shared__ uint4 s_prog[kList];             // listed programs: code, id, words
    __shared__ uint32_t s_done[kSplitMax];        // units of a program that are done
    const ThreadConsts tc = thread_consts();
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const const_ptr<uint32_t> pre = as_const(a.item_pre);
    const int ns = a.n_seg;
    const uint32_t n2 = pre[2 * (ns + 1) + ns], n1 = pre[(ns + 1) + ns], n0 = pre[ns];
    const uint32_t n_items = n2 + n1 + n0;
    int staged_d = -1, staged_n = 0, ynf = 0;     // what the staged memory holds
    int64_t staged = -1;

    for (uint32_t item = blockIdx.x; item < n_items;) {
        const int c = item < n2 ? 2 : (item < n2 + n1 ? 1 : 0);
        const uint32_t c0 = c == 2 ? 0u : (c == 1 ? n2 : n2 + n1);
        const uint32_t ci = item - c0;
        // segment of this item: last s with pre_c[s] <= ci
        const const_ptr<uint32_t> pre_c = pre + c * (ns + 1);
        int sl = 0, sh = ns - 1;
        while (sl < sh) {
            const int mid = (sl + sh + 1) >> 1;
            if (pre_c[mid] <= ci) sl = mid; else sh = mid - 1;
        }
        const int d = as_const(a.seg_ds)[sl];
        const const_ptr<DevDataset> D = as_const(a.ds) + d;
        const int G = as_const(a.class_g)[c], m_cap = as_const(a.class_g)[kClasses + c];
        const bool split = SPLIT && as_const(a.class_g)[2 * kClasses + c] != 0;
        const int passes = D->passes[c], n_tiles = D->n_tiles[c], n_vars = D->n_vars;
        const int sub = sub_cases(c);
        const int64_t n_cases = D->n_cases;
        const int m = item_tiles(passes, n_tiles, c, staged_rows(kNoTargets, n_vars), a.lds_floats, m_cap);
        const int count = as_const(a.seg_cnt)[c * ns + sl];
        const uint32_t groups = (uint32_t)((count + G - 1) / G);
        const uint32_t local = ci - pre_c[sl];
        // Run by run: the next item is mostly over the same cases.  A class of
        // few items with many runs of tiles takes them group by group instead,
        // all runs of the longest programs first, so the launch ends on short
        // programs.  (us per call run by run and group by group: 300 programs x
        // 65,536 cases 203 and 170, 3,000 x 65,536 714 and 626, 10,000 x 262,144
        // 7,530 and 6,232, 2,000 x 1,048,576 7,470 and 6,670; with many items
        // the staging of each costs more: 30,000 x 16,384 1,321 and 1,442, x 65,536
        // 4,706 and 5,435.  With 4 and 5 runs it goes either way: 10,000 x 4,099
        // correlations 267 and 312, 10,000 x 10,000 443 and 397.)
        const uint32_t n_class = c == 2 ? n2 : (c == 1 ? n1 : n0), tile_runs = (uint32_t)item_groups(n_tiles, m);
        const bool by_group = ns == 1 && tile_runs >= kManyRuns && n_class < kFewItems * gridDim.x;
        const uint32_t inner = by_group ? tile_runs : groups, o = local / inner, i = local - o * inner;
        const int tg = (int)(by_group ? i : o), grp = (int)(by_group ? o : i);
        // items of the same programs' segment, class and cases: [item0, item1)
        const uint32_t item0 = by_group ? item : item - (uint32_t)grp, item1 = by_group ? item : item0 + groups;
        const int seg0 = as_const(a.class_info)[2 * c] + as_const(a.seg_pos)[c * ns + sl];
        Item it;
        it.n_vars = n_vars;
        it.scale = D->scale;
        it.window = D->window[c] * sub;
        it.tile = tg * m;
        it.count = min(G, count - grp * G);
        it.obase = seg0 + grp * G;
        // the item's cases, and how many of them are staged at once
        const int64_t tile_cases = (int64_t)passes * sub;
        const int64_t first = tile_cases * it.tile;
        const int64_t last = min(first + tile_cases * min(m, n_tiles - it.tile), n_cases);
        const int64_t cap = staged_cases(a.lds_floats, staged_rows(kNoTargets, n_vars));
        const bool whole = tile_cases <= cap;
        const int64_t step = whole ? last - first : piece_cases(cap, it.window);
        it.tile_cases = whole ? (int)tile_cases : 0;
        if (!whole && FIT != kFitPredict) {
            // running sums of the chunk's programs over the tile's pieces
            for (int g = tid; g < it.count; g += kRunWG) {
                if constexpr (FIT == kFitCorr) corr_zero(reinterpret_cast<CorrPart*>(accs)[g]);
                else if constexpr (FIT == kFitReward) reinterpret_cast<long long*>(accs)[g] = 0;
                else {
                    reinterpret_cast<float2*>(accs)[g] = make_float2(0.f, 0.f);
                    reinterpret_cast<uint32_t*>(reinterpret_cast<float2*>(accs) + kChunk)[g] = 0u;
                }
            }
        }
        uint32_t touched = 0;
        if (wave == kRunWaves - 1) touched = list_chunk(a, it.obase, it.count, G, lane, s_prog);
        for (int64_t f0 = first; f0 < last; f0 += step) {
            it.first = f0;
            it.cases = (int)min(step, last - f0);
            it.stride = (it.cases + 255) & ~255;
            if (tid == 0) {
                s_next = 0u;
                s_end = (uint32_t)it.count;
            }
            if (split && tid < kSplitMax) s_done[tid] = 0u;
            if (f0 != staged || d != staged_d || it.cases != staged_n) {
                // one wavefront per 256 cases of a row; MSE mode stores the
                // targets pre-scaled (an exact power of two)
                const float* __restrict__ X = D->X;
                const float* __restrict__ y = D->y;
                const int64_t ld_x = D->ld_x;
                const int nb = it.stride >> 8, units = staged_rows(kNoTargets, n_vars) * nb;
                int nf = 0;
                for (int u = wave; u < units; u += kRunWaves) {
                    const int v = u / nb, b = u - v * nb;
                    const bool target = !kNoTargets && v == n_vars;
                    const float* __restrict__ src = (target ? y : X + (int64_t)v * ld_x) + f0 + b * 256;
                    const int left = it.cases - b * 256;
                    float val[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) val[j] = lane + j * 64 < left ? src[lane + j * 64] : 0.f;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        if (target) {
                            if (FIT == kFitMse) val[j] *= it.scale;
                            nf |= !__builtin_isfinite(val[j]);
                        }
                        xt[u * 256 + lane + j * 64] = val[j];
                    }
                }
                // (block-uniform branch: every thread reaches the barrier)
                ynf = __syncthreads_or(nf);
                staged = f0;
                staged_d = d;
                staged_n = it.cases;
            } else {
                __syncthreads();
            }
            asm volatile("" ::"v"(touched));
            it.ynf = ynf;
            // The claim has no lane-0-only region: every lane adds one to the
            // counter (a wavefront's 64 claims are one block of 64, so the
            // block index is the program).  A lane-0-only claim followed by a
            // lane-0-only update lets the optimizer rotate the two into one
            // region that lane 0 alone runs between iterations, so the other
            // lanes would re-read a stale claim.
            auto claim = [&] { return (int)(__builtin_amdgcn_readfirstlane(atomicAdd(&s_next, 1u)) >> 6); };
            auto listed = [&] {
                return (int)__builtin_amdgcn_readfirstlane(
                    __hip_atomic_load(&s_end, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
            };
            // the program at place g of the list, over cases [from, to)
            auto run_cases = [&](int g, int from, int to, int mode, float* kept) {
                const uint4 pr = s_prog[g];
                const int pid = __builtin_amdgcn_readfirstlane((int)pr.z);
                const int slen = __builtin_amdgcn_readfirstlane((int)pr.w);
                const uint2* pc = reinterpret_cast<const uint2*>(
                    (uintptr_t)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)pr.y) << 32 |
                                (uint32_t)__builtin_amdgcn_readfirstlane((int)pr.x)));
                warm_code(pc, slen & ~kNarrow);
                const int slot = whole ? wave : g;
                void* acc = nullptr;
                uint32_t* acc_bad = nullptr;
                if constexpr (FIT == kFitCorr) acc = reinterpret_cast<CorrPart*>(accs) + slot;
                else if constexpr (FIT == kFitReward) acc = reinterpret_cast<long long*>(accs) + slot;
                else if constexpr (FIT == kFitMse) {
                    acc = reinterpret_cast<float2*>(accs) + slot;
                    acc_bad = reinterpret_cast<uint32_t*>(reinterpret_cast<float2*>(accs) + kChunk) + slot;
                }
                if (c == 0) run_piece<FIT, 0, SPLIT>(pc, pid, xt, a, it, tc, lane, acc, acc_bad, from, to, mode, kept);
                else if (c == 1) run_piece<FIT, 1, SPLIT>(pc, pid, xt, a, it, tc, lane, acc, acc_bad, from, to, mode, kept);
                else if (slen < 0) run_piece<FIT, 3, SPLIT>(pc, pid, xt, a, it, tc, lane, acc, acc_bad, from, to, mode, kept);
                else run_piece<FIT, 2, SPLIT>(pc, pid, xt, a, it, tc, lane, acc, acc_bad, from, to, mode, kept);
            };
            auto take_next = [&] {
                uint32_t next = n_items;
                if (n_items > gridDim.x) {
                    if (lane == 0) next = gridDim.x + atomicAdd(a.work_counter, 1u);
                    next = __builtin_amdgcn_readfirstlane(next);
                }
                return next;
            };
            // the chunk's first program: the workgroup's next item, listed behind
            // the chunk when it is over the same cases
            auto follow = [&](int g, bool more) {
                const uint32_t next = take_next();
                if (more && whole && next < item1 && g + 2 * G <= kList) {
                    const int at = (int)(next - item0) * G, n = min(G, count - at);
                    const uint32_t t = list_chunk(a, seg0 + at, n, G, lane, s_prog + g + G);
                    asm volatile("" ::"v"(t));
                    // (a wavefront's LDS writes land in order)
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                    if (lane == 0)
                        __hip_atomic_store(&s_end, (uint32_t)(g + G + n), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
                } else if (lane == 0) {
                    s_pending = next;
                }
            };
            // A claim is a program, or with split cases one of its units of 256
            // cases (and the sum, for the wavefront that ends the last unit).
            // A wavefront that comes to the end of the list waits at the
            // barrier; a program listed meanwhile under its number is still
            // its own, run after the barrier (nothing is listed any more
            // then: a wavefront that lists goes on to the list's end).
            const int units = it.stride >> 8;
            bool after = false, sum = false;
            int t = claim();
            for (;;) {
                int g = t, from = 0, to = it.cases, mode = kAll;
                float* kept = xt;
                if (split) {
                    if (t >= it.count * units) break;
                    if (t == 0 && !sum) follow(0, false);
                    g = t / units;
                    if (FIT != kFitPredict) kept += (int64_t)(n_vars + 1 + g) * it.stride;
                    if (sum) {
                        mode = kSum;
                    } else {
                        from = (t - g * units) * 256;
                        to = min(from + 256, it.cases);
                        mode = FIT == kFitPredict ? kAll : kKeep;
                    }
                } else {
                    const int end = listed();
                    if (t >= end) {
                        if (after) break;
                        __syncthreads();
                        after = true;
                        continue;
                    }
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                    if (f0 == first && t % G == 0) follow(t, !after);
                }
                run_cases(g, from, to, mode, kept);
                if (SPLIT && mode == kKeep) {
                    // (every lane adds one, as in the claims)
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                    const int done = (int)(__builtin_amdgcn_readfirstlane(atomicAdd(&s_done[g], 1u)) >> 6);
                    sum = done == units - 1;
                    if (sum) {
                        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                        continue;
                    }
                }
                sum = false;
                if (after) break;
                t = claim();
            }
            __syncthreads();
        }
        if (!whole && FIT != kFitPredict) {
            for (int g = tid; g < it.count; g += kRunWG) {
                // tile-major partials: the reduction reads neighbours' together
                const int64_t slot = (int64_t)it.tile * a.part_stride + s_prog[g].z;
                if constexpr (FIT == kFitCorr) a.part_corr[slot] = reinterpret_cast<CorrPart*>(accs)[g];
                else if constexpr (FIT == kFitReward)
                    reinterpret_cast<long long*>(a.part)[slot] = reinterpret_cast<long long*>(accs)[g];
                else {
                    a.part[slot] = reinterpret_cast<float2*>(accs)[g];
                    a.part_bad[slot] =
                        (uint8_t)(reinterpret_cast<uint32_t*>(reinterpret_cast<float2*>(accs) + kChunk)[g] != 0u);
                }
            }
        }
        item = __builtin_amdgcn_readfirstlane(s_pending);
        if (!whole) __syncthreads();
    }
}

// Timed calls: the next k_run takes depth class c alone.  The classes' item counts
// (the ends of their prefixes) are kept in `counts` from the first of the three on.
__global__ __launch_bounds__(64) void k_pick_class(int32_t c, int32_t n_seg, uint32_t* __restrict__ item_pre,
                                                   int32_t* __restrict__ counts, uint32_t* __restrict__ counter)
{
    const int k = threadIdx.x;
    if (k == 0) *counter = 0u;
    if (k >= kClasses) return;
    uint32_t* end = item_pre + k * (n_seg + 1) + n_seg;
    if (c == 0) counts[k] = (int32_t)*end;
    *end = k == c ? (uint32_t)counts[k] : 0u;
}

// NaN rows for programs that failed validation (one workgroup per program).
__global__ __launch_bounds__(256) void k_fill_invalid(const uint8_t* __restrict__ cls,
                                                      int64_t n_cases, float* __restrict__ out,
                                                      int64_t ld_out)
{
    const int64_t p = blockIdx.x;
    if (cls[p] < kKeys) return;
    for (int64_t i = threadIdx.x; i < n_cases; i += 256) out[p * ld_out + i] = __builtin_nanf("");
}

// ------------------------------------------------------------ k_reduce
struct ReduceArgs {
    const ProgMeta* meta;
    const uint8_t* cls;
    const int32_t* pds;             // request of each program (NULL: one request)
    const DevRequest* reqs;
    const int64_t* seg_start;
    const DevDataset* ds;
    const float2* part;
    const uint8_t* part_bad;
    const CorrPart* part_corr;
    int64_t n_programs;
    int32_t part_stride;    // tile stride of the partials (the program count)
    double max_score;
};

__global__ __launch_bounds__(256) void k_reduce(ReduceArgs a)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= a.n_programs) return;
    const int r = a.pds ? a.pds[p] : 0;
    const DevRequest& R = a.reqs[r];
    const int64_t q = p - a.seg_start[r];
    if (!R.out || q >= R.n_programs) return;     // only for inconsistent tables
    const int c = a.cls[p];
    if (c >= kKeys) { R.out[q] = __builtin_nan(""); return; }
    const ProgMeta m = a.meta[p];
    const DevDataset& D = a.ds[R.dataset];
    const int nt = D.n_tiles[c / kLenBuckets];
    double s = 0.0;
    bool bad = false;
    for (int t = 0; t < nt; ++t) {
        const float2 v = a.part[(int64_t)t * a.part_stride + p];
        s += (double)v.x + (double)v.y;
        bad |= a.part_bad[(int64_t)t * a.part_stride + p] != 0;
    }
    const double mse = s * D.unscale;
    R.out[q] = (bad || !(mse <= (double)FLT_MAX)) ? __builtin_inf() : mse + D.tax * (double)m.len;
}

// Correlation score per program (Eq. 2 with r of Eq. 1 over the valid
// pairs): the tiles' shifted sums merged in order, then the centred sums
// Sxx = Sdd - Sd^2/n, Sxy = Sde - Sd Se/n, Syy = See - Se^2/n.  r = 0 below
// two valid pairs, or when a centred sum of squares is not positive (a
// constant output or target gives exactly zero: every shifted value is 0).
__global__ __launch_bounds__(256) void k_reduce_corr(ReduceArgs a)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= a.n_programs) return;
    const int r = a.pds ? a.pds[p] : 0;
    const DevRequest& R = a.reqs[r];
    const int64_t q = p - a.seg_start[r];
    if (!R.out || q >= R.n_programs) return;     // only for inconsistent tables
    const int c = a.cls[p];
    if (c >= kKeys) { R.out[q] = __builtin_nan(""); return; }
    const DevDataset& D = a.ds[R.dataset];
    const int nt = D.n_tiles[c / kLenBuckets];
    CorrPart acc;
    corr_zero(acc);
    for (int t = 0; t < nt; ++t) corr_merge(acc, a.part_corr[(int64_t)t * a.part_stride + p]);
    const int64_t n = acc.n, c1 = acc.c1, c2 = acc.c2;
    double rr = 0.0;
    if (n >= 2) {
        // centred sums from the shifted ones (the shift is a data value, so
        // these subtract quantities of the size of the spread)
        const double dn = (double)n;
        const double vx = acc.sdd - acc.sd * (acc.sd / dn);
        const double vy = acc.see - acc.se * (acc.se / dn);
        const double vxy = acc.sde - acc.sd * (acc.se / dn);
        if (vx > 0.0 && vy > 0.0) rr = vxy / sqrt(vx * vy);
    }
    const double r2 = rr * rr;
    R.out[q] = a.max_score * r2 * r2 * (double)n - a.max_score * (double)(c1 - c2);
}

// Integer reward per program (Eq. 5 and its power variants): the tiles'
// int64 totals added exactly, returned as a double (exact below 2^53).
__global__ __launch_bounds__(256) void k_reduce_reward(ReduceArgs a)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= a.n_programs) return;
    const int r = a.pds ? a.pds[p] : 0;
    const DevRequest& R = a.reqs[r];
    const int64_t q = p - a.seg_start[r];
    if (!R.out || q >= R.n_programs) return;     // only for inconsistent tables
    const int c = a.cls[p];
    if (c >= kKeys) { R.out[q] = __builtin_nan(""); return; }
    const DevDataset& D = a.ds[R.dataset];
    const int nt = D.n_tiles[c / kLenBuckets];
    const long long* part = reinterpret_cast<const long long*>(a.part);
    long long s = 0;
    for (int t = 0; t < nt; ++t) s += part[(int64_t)t * a.part_stride + p];
    R.out[q] = (double)s;
}

// ----------------------------------------------------------- workspaces
struct Layout {
    size_t code, meta, cls, order, class_info, class_g, counter, rows, words;
    size_t part, part_bad;
    size_t ds, req, seg_ds, seg_start, seg_cnt, seg_pos, item_pre, pds, bad, total;
    bool many;                      // several requests: each program's is kept (pds)
};

size_t align_up(size_t v) { return (v + 255) & ~size_t(255); }

Layout make_layout(int64_t n_programs, int64_t n_nodes, int32_t part_stride, int32_t n_ds,
                   int32_t n_seg, int fit = kFitMse)
{
    Layout L;
    size_t off = 0;
    L.many = n_seg > 1;
    // a staged program never holds more instructions than nodes
    L.code = off;       off = align_up(off + (size_t)(n_nodes + 1) * sizeof(uint2));
    L.meta = off;       off = align_up(off + (size_t)n_programs * sizeof(ProgMeta));
    L.cls = off;        off = align_up(off + (size_t)n_programs);
    L.order = off;      off = align_up(off + (size_t)n_programs * 4);
    L.class_info = off; off = align_up(off + 2 * kClasses * 4);
    L.class_g = off;    off = align_up(off + 4 * kClasses * 4);      // (k_pick_class: the last three)
    L.counter = off;    off = align_up(off + 4);
    // per (program, tile) partials: a compensated pair and a bad flag
    // (MSE), the correlation sums, or an int64 reward total
    const size_t part_elem = fit == kFitCorr ? sizeof(CorrPart) : sizeof(float2);
    L.part = off;       off = align_up(off + (size_t)n_programs * part_stride * part_elem);
    L.part_bad = off;   off = align_up(off + (fit != kFitMse ? 0 : (size_t)n_programs * part_stride));
    // the staging blocks' counts are read for the last time before the first
    // partial is written: the same memory
    L.rows = L.part;
    L.words = align_up(L.rows + (size_t)stage_blocks(n_programs) * sizeof(StageRow));
    const size_t rows_end = align_up(L.words + (size_t)stage_blocks(n_programs) * 8);
    off = off < rows_end ? rows_end : off;
    L.ds = off;         off = align_up(off + (size_t)n_ds * sizeof(DevDataset));
    L.req = off;        off = align_up(off + (size_t)n_seg * sizeof(DevRequest));
    L.seg_ds = off;     off = align_up(off + (size_t)n_seg * 4);
    L.seg_start = off;  off = align_up(off + (size_t)(n_seg + 1) * 8);
    L.seg_cnt = off;    off = align_up(off + (size_t)kClasses * n_seg * 4);
    L.seg_pos = off;    off = align_up(off + (size_t)kClasses * n_seg * 4);
    L.item_pre = off;   off = align_up(off + (size_t)kClasses * (n_seg + 1) * 4);
    L.pds = off;        off = align_up(off + (n_seg > 1 ? (size_t)n_programs * 4 : 0));
    L.bad = off;        off = align_up(off + 4);
    L.total = off;
    return L;
}

// Device views of one call's workspace.
struct Staged {
    uint2* code;
    ProgMeta* meta;
    uint8_t* cls;
    int32_t* order;
    int32_t* class_info;
    int32_t* class_g;
    uint32_t* counter;
    StageRow* rows;
    unsigned long long* words;
    float2* part;
    uint8_t* part_bad;
    CorrPart* part_corr;            // the same memory as part, correlation mode
    DevDataset* ds;
    DevRequest* req;
    int32_t* seg_ds;
    int64_t* seg_start;
    int32_t* seg_cnt;
    int32_t* seg_pos;
    uint32_t* item_pre;
    int32_t* pds;
    int32_t* bad;
};

Staged carve(void* base, const Layout& L)
{
    char* ws = static_cast<char*>(base);
    Staged st;
    st.code = reinterpret_cast<uint2*>(ws + L.code);
    st.meta = reinterpret_cast<ProgMeta*>(ws + L.meta);
    st.cls = reinterpret_cast<uint8_t*>(ws + L.cls);
    st.order = reinterpret_cast<int32_t*>(ws + L.order);
    st.class_info = reinterpret_cast<int32_t*>(ws + L.class_info);
    st.class_g = reinterpret_cast<int32_t*>(ws + L.class_g);
    st.counter = reinterpret_cast<uint32_t*>(ws + L.counter);
    st.rows = reinterpret_cast<StageRow*>(ws + L.rows);
    st.words = reinterpret_cast<unsigned long long*>(ws + L.words);
    st.part = reinterpret_cast<float2*>(ws + L.part);
    st.part_corr = reinterpret_cast<CorrPart*>(ws + L.part);
    st.part_bad = reinterpret_cast<uint8_t*>(ws + L.part_bad);
    st.ds = reinterpret_cast<DevDataset*>(ws + L.ds);
    st.req = reinterpret_cast<DevRequest*>(ws + L.req);
    st.seg_ds = reinterpret_cast<int32_t*>(ws + L.seg_ds);
    st.seg_start = reinterpret_cast<int64_t*>(ws + L.seg_start);
    st.seg_cnt = reinterpret_cast<int32_t*>(ws + L.seg_cnt);
    st.seg_pos = reinterpret_cast<int32_t*>(ws + L.seg_pos);
    st.item_pre = reinterpret_cast<uint32_t*>(ws + L.item_pre);
    st.pds = L.many ? reinterpret_cast<int32_t*>(ws + L.pds) : nullptr;
    st.bad = reinterpret_cast<int32_t*>(ws + L.bad);
    return st;
}

// Per-(device, caller stream) state of gp_eval / gp_predict.
struct Workspace {
    void* ptr = nullptr;
    size_t bytes = 0;
};

std::mutex g_ws_mutex;
std::map<std::pair<int, hipStream_t>, Workspace> g_ws;

int get_workspace(hipStream_t stream, size_t bytes, Workspace** out)
{
    int dev = 0;
    GP_HIP_TRY(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(g_ws_mutex);
    Workspace& w = g_ws[std::make_pair(dev, stream)];
    if (w.bytes < bytes) {
        if (w.ptr) {
            // earlier work on this stream may still use the old buffer
            GP_HIP_TRY(hipStreamSynchronize(stream));
            GP_HIP_TRY(hipFree(w.ptr));
            w.ptr = nullptr;
            w.bytes = 0;
        }
        size_t want = bytes + bytes / 4;
        if (hipMalloc(&w.ptr, want) != hipSuccess) {
            (void)hipGetLastError();
            w.ptr = nullptr;
            return set_error(GP_E_NO_MEMORY, "workspace allocation of %zu bytes failed", want);
        }
        w.bytes = want;
    }
    *out = &w;
    return GP_OK;
}

struct DeviceInfo {
    int cus = 0;
};
std::mutex g_dev_mutex;
std::map<int, DeviceInfo> g_dev;

int device_cus(int* cus)
{
    int dev = 0;
    GP_HIP_TRY(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(g_dev_mutex);
    DeviceInfo& di = g_dev[dev];
    if (di.cus == 0) GP_HIP_TRY(hipDeviceGetAttribute(&di.cus, hipDeviceAttributeMultiprocessorCount, dev));
    *cus = di.cus;
    return GP_OK;
}

// ---------------------------------------------------------------- timing
struct Timing {
    bool on = false;
    // events of calls not yet read: GP_TIMING_PHASES boundaries per call
    std::vector<std::array<hipEvent_t, GP_TIMING_PHASES>> pending;
    double ms[GP_TIMING_PHASES] = {0, 0, 0, 0, 0, 0};
    int64_t calls = 0;
};
thread_local Timing g_timing;

// boundaries: b0 before prepare, b1 before class 0, b2 before class 1,
// b3 before class 2, b4 before reduce, b5 after reduce
struct CallEvents {
    std::array<hipEvent_t, GP_TIMING_PHASES> ev{};
    bool on = false;
    int begin(bool enable)
    {
        on = enable && g_timing.on;
        if (!on) return GP_OK;
        for (auto& e : ev) GP_HIP_TRY(hipEventCreate(&e));
        return GP_OK;
    }
    int mark(int i, hipStream_t s)
    {
        if (on) GP_HIP_TRY(hipEventRecord(ev[i], s));
        return GP_OK;
    }
    void commit()
    {
        if (on) g_timing.pending.push_back(ev);
    }
};

// ------------------------------------------------------------- problem
// Everything one evaluation needs (device pointers, sizes, scoring).  A
// single-population call carries its request and dataset inline (req_dev
// and ds_dev NULL); a batched call points at device tables.
struct Problem {
    gp_request one_req;             // inline request ...
    const gp_request* req_dev;      // ... or a device table of n_req
    int32_t n_req;
    gp_dataset one;                 // inline dataset ...
    const gp_dataset* ds_dev;       // ... or a device table of n_ds
    int32_t n_ds;
    int64_t n_programs;             // over all requests
    int64_t n_nodes;
    int32_t max_vars;
    int64_t max_cases;
    uint32_t allowed;
    int32_t need_out;               // fitness outputs required (not for gp_predict)
    int32_t fit;                    // kFitMse, kFitCorr or kFitReward
    double max_score;               // M of the correlation score or the reward
    int32_t reward_power;           // 1, 2, 3 or 8 (reward mode)
};

int check_common(int64_t n_programs, int64_t n_nodes, int64_t n_consts, int32_t n_vars,
                 int64_t ld_x, int64_t n_cases)
{
    if (n_programs < 0) return set_error(GP_E_INVALID_ARG, "n_programs < 0");
    if (n_programs > INT32_MAX - 1) return set_error(GP_E_TOO_LARGE, "n_programs > 2^31-2");
    if (n_nodes < 0) return set_error(GP_E_INVALID_ARG, "n_nodes < 0");
    if (n_nodes > (int64_t(1) << 40)) return set_error(GP_E_TOO_LARGE, "n_nodes > 2^40");
    if (n_consts < 0) return set_error(GP_E_INVALID_ARG, "n_consts < 0");
    if (n_consts > GP_MAX_CONSTS) return set_error(GP_E_TOO_LARGE, "n_consts > 2^24");
    if (n_vars < 0) return set_error(GP_E_INVALID_ARG, "n_vars < 0");
    if (n_vars > 4096) return set_error(GP_E_TOO_LARGE, "n_vars > 4096 (inputs are staged in LDS)");
    if (n_cases < 1) return set_error(GP_E_INVALID_ARG, "n_cases < 1");
    if (n_cases > (int64_t(1) << 40)) return set_error(GP_E_TOO_LARGE, "n_cases > 2^40");
    if (n_vars > 0 && ld_x < n_cases) return set_error(GP_E_INVALID_ARG, "ld_x < n_cases");
    return GP_OK;
}

int check_pointers(const uint32_t* nodes, int64_t n_nodes, const float* consts, int64_t n_consts,
                   const float* X, int32_t n_vars)
{
    if (n_nodes > 0 && !nodes) return set_error(GP_E_INVALID_ARG, "nodes is NULL");
    if (n_consts > 0 && !consts) return set_error(GP_E_INVALID_ARG, "consts is NULL");
    if (n_vars > 0 && !X) return set_error(GP_E_INVALID_ARG, "X is NULL");
    return GP_OK;
}

int check_problem(const Problem& pb)
{
    const bool batched = pb.req_dev != nullptr;
    int rc = check_common(pb.n_programs, pb.n_nodes, batched ? 0 : pb.one_req.n_consts,
                          pb.max_vars, batched ? pb.max_cases : pb.one.ld_x, pb.max_cases);
    if (rc != GP_OK) return rc;
    if (pb.allowed & ~GP_ALL_OPS)
        return set_error(GP_E_INVALID_ARG, "allowed_op_mask has bits beyond GP_ALL_OPS");
    if (batched) {
        if (!pb.ds_dev) return set_error(GP_E_INVALID_ARG, "datasets_dev is NULL");
        if (pb.n_ds < 1) return set_error(GP_E_INVALID_ARG, "n_datasets < 1");
        if (pb.n_req < 1) return set_error(GP_E_INVALID_ARG, "n_requests < 1");
        if (pb.n_req > kMaxRequests) return set_error(GP_E_TOO_LARGE, "more than %d requests", kMaxRequests);
        return GP_OK;
    }
    if (pb.n_programs == 0) return GP_OK;
    const gp_request& q = pb.one_req;
    if (!q.offsets) return set_error(GP_E_INVALID_ARG, "offsets is NULL");
    if (pb.need_out && !q.out_fitness) return set_error(GP_E_INVALID_ARG, "out_fitness is NULL");
    if ((rc = check_pointers(q.nodes, q.n_nodes, q.consts, q.n_consts, nullptr, 0)) != GP_OK) return rc;
    if (!pb.one.y) return set_error(GP_E_INVALID_ARG, "y is NULL");
    if (pb.one.n_vars > 0 && !pb.one.X) return set_error(GP_E_INVALID_ARG, "X is NULL");
    if (!std::isfinite(pb.one.tax_on_length)) return set_error(GP_E_INVALID_ARG, "tax_on_length is not finite");
    return GP_OK;
}

// --------------------------------------------------- launch configuration
// Launch knobs.  G, wg_per_cu and concurrent change no result.  The tile
// knobs (the LDS budget of an input window and the cap on case tiles per
// program) set how a program's cases are grouped into windows and tiles,
// so they fix its summation order together with (n_cases, its depth class,
// n_vars): every call with the same knobs gives the same bits, and the
// defaults are those of gp_eval, gp_eval_batched and the server.
struct Tuning {
    int G = 64;             // programs per work item, at most (small classes use fewer)
    int wg_per_cu = 0;      // persistent workgroups per CU (0: occupancy limit)
    int concurrent = 0;     // accepted and reported; every class runs in one launch
    int tile_lds = kTileLds;    // LDS bytes of an input window
    int tile_max = kMaxTiles;   // case tiles per program, at most
};

// Whether a call's op mask reaches beyond the benchmark set (its staging then
// follows named variables and stack moves).
inline bool pb_ext(uint32_t allowed) { return (allowed & ~GP_BASE_OPS) != 0u; }


struct EvalLaunch {
    int32_t stride = 1;
    int32_t target_items = 1;   // work items per class worth keeping large groups for
    int32_t lds_floats = 0;     // staged inputs and targets
    int32_t split = 0;          // cases may be split over wavefronts
    int32_t wide = 0;           // a sub-tile takes nearly all LDS (k_run's WIDE)
    int32_t chunk = 0;          // programs per work item, at most
    int grid = 0;
    size_t lds = 0;
    Layout layout;
};

// Programs per work item at most: the tuning's value, capped by the LDS of the
// running sums.
int group_capacity(const Tuning& tu, const EvalLaunch& el) { return std::min(tu.G, el.chunk); }

// Grid and LDS of the evaluation kernel (LDS attribute set outside any
// capture).
template <int FIT, bool SPLIT, bool WIDE>
int run_grid(const Problem& pb, const Tuning& tu, int cus, EvalLaunch* el)
{
    el->wide = WIDE;
    el->chunk = chunk_max(FIT, WIDE);
    el->lds_floats = run_lds_floats(staged_rows(FIT == kFitPredict, pb.max_vars), tu.tile_lds);
    el->lds = (size_t)el->lds_floats * sizeof(float) + acc_bytes(FIT, WIDE);
    if (el->lds > 64 * 1024) {
        GP_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_run<FIT, SPLIT, WIDE>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)el->lds));
    }
    int per_cu = 0;
    GP_HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_run<FIT, SPLIT, WIDE>, kRunWG, el->lds));
    if (per_cu < 1)
        return set_error(GP_E_TOO_LARGE, "n_vars=%d needs %zu bytes of LDS per workgroup", pb.max_vars, el->lds);
    if (tu.wg_per_cu > 0 && tu.wg_per_cu < per_cu) per_cu = tu.wg_per_cu;
    el->grid = cus * per_cu;
    return GP_OK;
}

// (Classes are split one by one, see split_programs; a kernel of its own, as
// the forms for units cost the ordinary ones 3% in registers.)
template <int FIT>
int run_grid_for(const Problem& pb, const Tuning& tu, int cus, EvalLaunch* el)
{
    if (pb.max_vars >= kWideVars) {
        el->split = 0;
        return run_grid<FIT, false, true>(pb, tu, cus, el);
    }
    return el->split ? run_grid<FIT, true, false>(pb, tu, cus, el) : run_grid<FIT, false, false>(pb, tu, cus, el);
}

int configure_eval(const Problem& pb, const Tuning& tu, EvalLaunch* el)
{
    int cus = 0;
    int rc = device_cus(&cus);
    if (rc != GP_OK) return rc;
    el->stride = 1;
    for (int c = 0; c < kClasses; ++c) {
        // tile counts grow with n_cases, so the largest dataset sizes the
        // partial buffer
        const int32_t t = max_tiles(pb.max_cases, class_k(c, pb.max_vars), tu.tile_max);
        if (t > el->stride) el->stride = t;
    }
    el->target_items = 4 * 3 * cus;     // ~4 items per workgroup slot
    const int32_t tiles =
        tile_shape(pb.max_cases, class_k(0, pb.max_vars), pb.max_vars, tu.tile_lds, tu.tile_max).n_tiles;
    el->split = pb.req_dev == nullptr && pb.max_cases > 256 &&
                (pb.fit == kFitPredict || (double)pb.n_programs * (double)tiles <= kGpuWaves);
    if (pb.fit == kFitPredict) el->stride = 0;      // no partials
    if (pb.fit == kFitCorr) rc = run_grid_for<kFitCorr>(pb, tu, cus, el);
    else if (pb.fit == kFitReward) rc = run_grid_for<kFitReward>(pb, tu, cus, el);
    else if (pb.fit == kFitPredict) rc = run_grid_for<kFitPredict>(pb, tu, cus, el);
    else rc = run_grid_for<kFitMse>(pb, tu, cus, el);
    if (rc != GP_OK) return rc;
    el->layout = make_layout(pb.n_programs, pb.n_nodes, el->stride, pb.n_ds, pb.n_req, pb.fit);
    return GP_OK;
}

// Dataset/segment tables, validation, staging and the stable (depth class,
// cost) partition.
int enqueue_tables(const Problem& pb, const Tuning& tu, const Staged& st, hipStream_t stream)
{
    hipLaunchKernelGGL(k_tables, dim3(1), dim3(256), 0, stream, pb.ds_dev, pb.n_ds, pb.one,
                       pb.req_dev, pb.n_req, pb.one_req, pb.n_programs, pb.n_nodes, pb.max_vars,
                       pb.max_cases, pb.need_out, tu.tile_lds, tu.tile_max, st.ds, st.req,
                       st.seg_ds, st.seg_start, st.bad);
    GP_HIP_TRY(hipGetLastError());
    return GP_OK;
}

template <bool EXT, bool LANES>
int launch_stage(const StageArgs& a, int32_t n_blk, int64_t n_nodes, const SegOut& so, hipStream_t stream)
{
    if (LANES) {
        hipLaunchKernelGGL((k_stage_lanes<EXT>), dim3((unsigned)((a.n_programs + kLaneWG - 1) / kLaneWG)), dim3(kLaneWG),
                           0, stream, a);
        GP_HIP_TRY(hipGetLastError());
    }
    hipLaunchKernelGGL((k_stage_waves<EXT, LANES>), dim3(n_blk), dim3(64 * kStageWaves), 0, stream, a);
    GP_HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL((k_order<EXT, LANES>), dim3(n_blk), dim3(kOrderWG), 0, stream, a, n_blk, n_nodes, so);
    GP_HIP_TRY(hipGetLastError());
    return GP_OK;
}

// Validation, staging and partition (a single request brings its tables by
// value; several have them derived by k_tables first).
int enqueue_stage(const Problem& pb, const Tuning& tu, const EvalLaunch& el, const Staged& st,
                  hipStream_t stream)
{
    int rc = GP_OK;
    StageArgs a{};
    a.n_programs = pb.n_programs;
    a.share = stage_share(pb.n_programs);
    a.allowed = pb.allowed;
    a.single = pb.req_dev ? 0 : 1;
    a.lpt = pb.n_req == 1 ? 1 : 0;
    a.lane_nodes = lane_nodes(pb.n_programs, pb.n_nodes);
    a.n_seg = pb.n_req;
    a.ds = st.ds; a.reqs = st.req; a.seg_ds = st.seg_ds; a.seg_start = st.seg_start; a.bad = st.bad;
    a.meta = st.meta; a.cls = st.cls; a.pds = st.pds; a.order = st.order; a.code = st.code;
    a.rows = st.rows; a.words = st.words;
    if (a.single) {
        const gp_request& q = pb.one_req;
        a.one_req = DevRequest{q.nodes, q.offsets, q.consts, q.n_programs, q.n_nodes, q.n_consts, 0,
                               q.out_fitness, q.out_status, 0};
        a.one_ds = make_dataset(pb.one, tu.tile_lds, tu.tile_max);
    } else if ((rc = enqueue_tables(pb, tu, st, stream)) != GP_OK) {
        return rc;
    }
    const int32_t n_blk = (int32_t)stage_blocks(pb.n_programs);
    const SegOut so{group_capacity(tu, el), el.target_items, el.lds_floats, el.split, pb.fit == kFitPredict, st.seg_cnt, st.seg_pos,
                    st.item_pre, st.class_g, st.class_info, st.counter};
    if (pb_ext(pb.allowed))
        rc = a.lane_nodes > 0 ? launch_stage<true, true>(a, n_blk, pb.n_nodes, so, stream)
                              : launch_stage<true, false>(a, n_blk, pb.n_nodes, so, stream);
    else
        rc = a.lane_nodes > 0 ? launch_stage<false, true>(a, n_blk, pb.n_nodes, so, stream)
                              : launch_stage<false, false>(a, n_blk, pb.n_nodes, so, stream);
    if (rc != GP_OK) return rc;
    if (pb.req_dev) {
        hipLaunchKernelGGL(k_seg_tables, dim3(kClasses), dim3(kSegWG), 0, stream, st.order, st.class_info,
                           st.seg_start, pb.n_req, st.bad, st.seg_ds, st.ds, group_capacity(tu, el),
                           el.target_items, el.lds_floats, st.seg_cnt, st.seg_pos, st.item_pre,
                           st.class_g);
        GP_HIP_TRY(hipGetLastError());
    }
    return GP_OK;
}

template <int FIT>
void launch_run(const EvalLaunch& el, dim3 g, dim3 b, hipStream_t stream, const RunArgs& a)
{
    if (el.wide) hipLaunchKernelGGL((k_run<FIT, false, true>), g, b, el.lds, stream, a);
    else if (el.split) hipLaunchKernelGGL((k_run<FIT, true, false>), g, b, el.lds, stream, a);
    else hipLaunchKernelGGL((k_run<FIT, false, false>), g, b, el.lds, stream, a);
}

// The evaluation kernel (out: gp_predict's per-case outputs).
int enqueue_run(const Problem& pb, const EvalLaunch& el, const Staged& st, hipStream_t stream,
                float* out = nullptr, int64_t ld_out = 0)
{
    RunArgs a{};
    a.code = st.code; a.meta = st.meta; a.order = st.order; a.class_info = st.class_info;
    a.work_counter = st.counter; a.ds = st.ds; a.seg_ds = st.seg_ds; a.seg_cnt = st.seg_cnt;
    a.seg_pos = st.seg_pos; a.item_pre = st.item_pre; a.class_g = st.class_g;
    a.part = st.part; a.part_bad = st.part_bad; a.part_corr = st.part_corr;
    a.out = out; a.ld_out = ld_out;
    a.part_stride = (int32_t)pb.n_programs;       // tile stride of the partials
    a.n_seg = pb.n_req;
    a.lds_floats = el.lds_floats;
    a.reward_power = pb.reward_power;
    a.reward_M = (float)pb.max_score;
    a.reward_less = a.reward_M / 11.0f;
    const dim3 g(el.grid), b(kRunWG);
    if (pb.fit == kFitCorr) launch_run<kFitCorr>(el, g, b, stream, a);
    else if (pb.fit == kFitReward) launch_run<kFitReward>(el, g, b, stream, a);
    else if (pb.fit == kFitPredict) launch_run<kFitPredict>(el, g, b, stream, a);
    else launch_run<kFitMse>(el, g, b, stream, a);
    GP_HIP_TRY(hipGetLastError());
    return GP_OK;
}

// The whole evaluation as stream work (no allocation, no synchronization:
// safe to capture into a graph).
int enqueue_eval(const Problem& pb, const Tuning& tu, const EvalLaunch& el, const Staged& st,
                 hipStream_t stream, CallEvents& ce)
{
    int rc;
    if ((rc = ce.mark(0, stream)) != GP_OK) return rc;
    if ((rc = enqueue_stage(pb, tu, el, st, stream)) != GP_OK) return rc;
    if (ce.on) {
        // timed: a launch per depth class, so that each has its phase
        for (int c = 0; c < kClasses; ++c) {
            if ((rc = ce.mark(1 + c, stream)) != GP_OK) return rc;
            hipLaunchKernelGGL(k_pick_class, dim3(1), dim3(64), 0, stream, c, pb.n_req, st.item_pre,
                               st.class_g + 3 * kClasses, st.counter);
            GP_HIP_TRY(hipGetLastError());
            if ((rc = enqueue_run(pb, el, st, stream)) != GP_OK) return rc;
        }
        if ((rc = ce.mark(4, stream)) != GP_OK) return rc;
    } else if ((rc = enqueue_run(pb, el, st, stream)) != GP_OK) {
        return rc;
    }
    ReduceArgs ra{};
    ra.meta = st.meta; ra.cls = st.cls; ra.pds = st.pds; ra.reqs = st.req;
    ra.seg_start = st.seg_start; ra.ds = st.ds;
    ra.part = st.part; ra.part_bad = st.part_bad; ra.part_corr = st.part_corr;
    ra.n_programs = pb.n_programs; ra.part_stride = (int32_t)pb.n_programs;
    ra.max_score = pb.max_score;
    const dim3 g((unsigned)((pb.n_programs + 255) / 256)), b(256);
    if (pb.fit == kFitCorr) hipLaunchKernelGGL(k_reduce_corr, g, b, 0, stream, ra);
    else if (pb.fit == kFitReward) hipLaunchKernelGGL(k_reduce_reward, g, b, 0, stream, ra);
    else hipLaunchKernelGGL(k_reduce, g, b, 0, stream, ra);
    GP_HIP_TRY(hipGetLastError());
    if ((rc = ce.mark(5, stream)) != GP_OK) return rc;
    return GP_OK;
}

// ----------------------------------------------------------------- autotune
// In-process cache of tuned scheduling knobs, optionally mirrored in a
// text file named by GPEVAL_TUNE_CACHE (one "key G wg_per_cu concurrent"
// line per entry).  Keys describe the workload shape, not its values.
std::mutex g_tune_mutex;
std::map<std::string, Tuning> g_tune;
bool g_tune_loaded = false;

std::string tune_key(const Problem& pb)
{
    int dev = 0;
    (void)hipGetDevice(&dev);
    char name[64] = {0};
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, dev) == hipSuccess) snprintf(name, sizeof name, "%s", prop.gcnArchName);
    for (char* c = name; *c; ++c) if (*c == ' ' || *c == ':') *c = '_';
    const double mean_len = pb.n_programs ? (double)pb.n_nodes / (double)pb.n_programs : 0.0;
    int lp = 0;
    while ((int64_t(1) << (lp + 1)) <= pb.n_programs) ++lp;
    int lc = 0;
    while ((int64_t(1) << (lc + 1)) <= pb.max_cases) ++lc;
    char buf[160];
    snprintf(buf, sizeof buf, "%s/cases2^%d/vars%d/progs2^%d/len%d/reqs%d", name, lc,
             pb.max_vars, lp, (int)(mean_len + 0.5), pb.n_req);
    return buf;
}

void tune_load_locked()
{
    if (g_tune_loaded) return;
    g_tune_loaded = true;
    const char* path = getenv("GPEVAL_TUNE_CACHE");
    if (!path) return;
    FILE* f = fopen(path, "r");
    if (!f) return;
    char key[200];
    Tuning t;
    while (fscanf(f, "%199s %d %d %d %d %d", key, &t.G, &t.wg_per_cu, &t.concurrent, &t.tile_lds,
                  &t.tile_max) == 6)
        g_tune[key] = t;
    fclose(f);
}

void tune_store_locked(const std::string& key, const Tuning& t)
{
    g_tune[key] = t;
    const char* path = getenv("GPEVAL_TUNE_CACHE");
    if (!path) return;
    FILE* f = fopen(path, "a");
    if (!f) return;
    fprintf(f, "%s %d %d %d %d %d\n", key.c_str(), t.G, t.wg_per_cu, t.concurrent, t.tile_lds,
            t.tile_max);
    fclose(f);
}

}  // namespace

// ================================================================== plans
struct gp_plan {
    Problem pb;
    Tuning tu;
    EvalLaunch el;
    void* ws = nullptr;
    size_t ws_bytes = 0;
    Staged st;
    hipStream_t cap = nullptr;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    int device = 0;
    double tuned_ms = 0.0;
    int tune_trials = 0;
};

namespace {

void plan_release_graph(gp_plan* p)
{
    if (p->exec) (void)hipGraphExecDestroy(p->exec);
    if (p->graph) (void)hipGraphDestroy(p->graph);
    p->exec = nullptr;
    p->graph = nullptr;
}

// (Re)size the plan's workspace and capture its graph.
int plan_build(gp_plan* p)
{
    int rc = configure_eval(p->pb, p->tu, &p->el);
    if (rc != GP_OK) return rc;
    if (p->ws_bytes < p->el.layout.total) {
        if (p->ws) {
            GP_HIP_TRY(hipDeviceSynchronize());
            GP_HIP_TRY(hipFree(p->ws));
            p->ws = nullptr;
            p->ws_bytes = 0;
        }
        if (hipMalloc(&p->ws, p->el.layout.total) != hipSuccess) {
            (void)hipGetLastError();
            return set_error(GP_E_NO_MEMORY, "plan workspace of %zu bytes", p->el.layout.total);
        }
        p->ws_bytes = p->el.layout.total;
    }
    p->st = carve(p->ws, p->el.layout);
    // replays of a previous graph may still read the workspace
    if (p->exec) GP_HIP_TRY(hipDeviceSynchronize());
    plan_release_graph(p);
    GP_HIP_TRY(hipStreamBeginCapture(p->cap, hipStreamCaptureModeThreadLocal));
    CallEvents none;
    (void)none.begin(false);
    rc = enqueue_eval(p->pb, p->tu, p->el, p->st, p->cap, none);
    hipGraph_t g = nullptr;
    const hipError_t ec = hipStreamEndCapture(p->cap, &g);
    if (rc != GP_OK) {
        if (g) (void)hipGraphDestroy(g);
        return rc;
    }
    if (ec != hipSuccess) return set_error(GP_E_HIP, "hipStreamEndCapture: %s", hipGetErrorString(ec));
    p->graph = g;
    GP_HIP_TRY(hipGraphInstantiate(&p->exec, p->graph, nullptr, nullptr, 0));
    return GP_OK;
}

// Median of `runs` timed runs of one configuration (after one warm-up when
// `warm`), or a negative value when it does not fit the plan's workspace.
int time_config(gp_plan* p, const Tuning& t, hipStream_t stream, hipEvent_t e0, hipEvent_t e1,
                float* ms_out, int runs = 5, bool warm = true)
{
    *ms_out = -1.f;
    EvalLaunch el;
    int rc = configure_eval(p->pb, t, &el);
    if (rc != GP_OK) return rc;
    if (el.layout.total > p->ws_bytes) return GP_OK;
    const Staged st = carve(p->ws, el.layout);
    CallEvents none;
    (void)none.begin(false);
    float ms[8];
    runs = std::min(std::max(runs, 1), 8);
    if (warm && (rc = enqueue_eval(p->pb, t, el, st, stream, none)) != GP_OK) return rc;
    for (int r = 0; r < runs; ++r) {
        GP_HIP_TRY(hipEventRecord(e0, stream));
        if ((rc = enqueue_eval(p->pb, t, el, st, stream, none)) != GP_OK) return rc;
        GP_HIP_TRY(hipEventRecord(e1, stream));
        GP_HIP_TRY(hipEventSynchronize(e1));
        GP_HIP_TRY(hipEventElapsedTime(&ms[r], e0, e1));
    }
    std::sort(ms, ms + runs);
    *ms_out = ms[runs / 2];
    return GP_OK;
}

// Time candidate knobs on the real inputs and keep the fastest: coordinate
// descent over the axes (programs per work item, workgroups per CU, the LDS
// budget of an input window, the cap on case tiles per program), at values that
// differ (an item holds at most 64 programs, a CU three workgroups, and a window of
// up to 36 KB costs none of them), each axis tried in turn with the others at their
// best so far, two sweeps, each candidate the median of five runs; then the
// three fastest candidates are timed again in turns (five rounds, one run
// each per round, so drift hits them alike) and the lowest median wins.
// The tile axes set a program's summation order, so the chosen plan is
// deterministic for its problem shape (the tuning is cached by it) but may
// differ from gp_eval in the last bits.
int plan_autotune(gp_plan* p, hipStream_t stream)
{
    const std::string key = tune_key(p->pb);
    {
        std::lock_guard<std::mutex> lk(g_tune_mutex);
        tune_load_locked();
        auto it = g_tune.find(key);
        if (it != g_tune.end()) {
            p->tu = it->second;
            return GP_OK;
        }
    }
    hipEvent_t e0, e1;
    GP_HIP_TRY(hipEventCreate(&e0));
    GP_HIP_TRY(hipEventCreate(&e1));
    const int kAxes = 4;
    const std::vector<int> values[kAxes] = {{16, 32, 64}, {0, 2}, {12 * 1024, 24 * 1024, 36 * 1024}, {2, 8, 32}};
    auto field = [](Tuning& t, int a) -> int& {
        return a == 0 ? t.G : a == 1 ? t.wg_per_cu : a == 2 ? t.tile_lds : t.tile_max;
    };
    Tuning best = p->tu;
    float best_ms = 1e30f;
    int rc = time_config(p, best, stream, e0, e1, &best_ms);
    if (rc == GP_OK && best_ms < 0.f) best_ms = 1e30f;
    int tried = 1;
    std::vector<std::pair<float, Tuning>> seen;
    if (best_ms < 1e30f) seen.push_back({best_ms, best});
    for (int sweep = 0; sweep < 2 && rc == GP_OK; ++sweep) {
        for (int a = 0; a < kAxes && rc == GP_OK; ++a) {
            for (int v : values[a]) {
                Tuning t = best;
                if (field(t, a) == v) continue;
                field(t, a) = v;
                float ms = -1.f;
                if ((rc = time_config(p, t, stream, e0, e1, &ms)) != GP_OK) break;
                ++tried;
                if (ms >= 0.f) seen.push_back({ms, t});
                if (ms >= 0.f && ms < best_ms) {
                    best_ms = ms;
                    best = t;
                }
            }
        }
    }
    // run-off among the three fastest distinct candidates
    if (rc == GP_OK && seen.size() > 1) {
        std::stable_sort(seen.begin(), seen.end(),
                         [](const std::pair<float, Tuning>& x, const std::pair<float, Tuning>& y) {
                             return x.first < y.first;
                         });
        auto same = [](const Tuning& x, const Tuning& y) {
            return x.G == y.G && x.wg_per_cu == y.wg_per_cu && x.concurrent == y.concurrent &&
                   x.tile_lds == y.tile_lds && x.tile_max == y.tile_max;
        };
        std::vector<Tuning> top;
        for (const auto& c : seen) {
            bool dup = false;
            for (const auto& u : top) dup = dup || same(u, c.second);
            if (!dup) top.push_back(c.second);
            if (top.size() == 3) break;
        }
        std::vector<std::vector<float>> smp(top.size());
        for (int round = 0; round < 5 && rc == GP_OK; ++round)
            for (size_t i = 0; i < top.size() && rc == GP_OK; ++i) {
                float ms = -1.f;
                if ((rc = time_config(p, top[i], stream, e0, e1, &ms, 1, round == 0)) == GP_OK)
                    smp[i].push_back(ms);
            }
        if (rc == GP_OK) {
            for (size_t i = 0; i < top.size(); ++i) {
                std::sort(smp[i].begin(), smp[i].end());
                const float med = smp[i][smp[i].size() / 2];
                if (i == 0 || med < best_ms) {
                    best_ms = med;
                    best = top[i];
                }
            }
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc != GP_OK) return rc;
    p->tu = best;
    p->tuned_ms = best_ms;
    p->tune_trials = tried;
    std::lock_guard<std::mutex> lk(g_tune_mutex);
    tune_store_locked(key, best);
    return GP_OK;
}

Problem make_problem(const gp_problem* d)
{
    Problem pb{};
    pb.one_req.nodes = d->nodes; pb.one_req.offsets = d->offsets; pb.one_req.consts = d->consts;
    pb.one_req.n_programs = d->n_programs; pb.one_req.n_nodes = d->n_nodes;
    pb.one_req.n_consts = d->n_consts;
    pb.one_req.out_fitness = d->out_fitness; pb.one_req.out_status = d->out_status;
    pb.one_req.dataset = 0;
    pb.req_dev = nullptr; pb.n_req = 1;
    pb.one.X = d->X; pb.one.y = d->y; pb.one.ld_x = d->ld_x; pb.one.n_cases = d->n_cases;
    pb.one.tax_on_length = d->tax_on_length; pb.one.n_vars = d->n_vars; pb.one.reserved = 0;
    pb.ds_dev = nullptr; pb.n_ds = 1;
    pb.n_programs = d->n_programs; pb.n_nodes = d->n_nodes;
    pb.max_vars = d->n_vars; pb.max_cases = d->n_cases;
    pb.allowed = d->allowed_op_mask ? d->allowed_op_mask : GP_BASE_OPS;
    pb.need_out = 1;
    return pb;
}

int eval_problem(const Problem& pb, hipStream_t stream)
{
    int rc = check_problem(pb);
    if (rc != GP_OK || pb.n_programs == 0) return rc;
    Tuning tu;
    EvalLaunch el;
    if ((rc = configure_eval(pb, tu, &el)) != GP_OK) return rc;
    Workspace* w = nullptr;
    if ((rc = get_workspace(stream, el.layout.total, &w)) != GP_OK) return rc;
    const Staged st = carve(w->ptr, el.layout);
    CallEvents ce;
    if ((rc = ce.begin(true)) != GP_OK) return rc;
    if ((rc = enqueue_eval(pb, tu, el, st, stream, ce)) != GP_OK) return rc;
    ce.commit();
    return GP_OK;
}

// ------------------------------------------------- no-allocation form
// gp_eval_noalloc keeps its workspace in one fixed device array per GPU
// instead of memory the library allocates.  In host code `scratch` names a
// host-side stand-in, never the device memory: its device address is taken
// with hipGetSymbolAddress once per device (with that device current, each
// GPU holding its own copy) and only that address reaches kernels.  Every
// kernel of the call initializes what it reads (counters, flags, partials),
// so no clearing is needed between calls; calls that overlap in time on one
// GPU share the array and race.
constexpr size_t kScratchBytes = GP_NOALLOC_WORKSPACE_BYTES;
__device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxScratchDevices] = {};

// This device's scratch address; the first call on a device takes it and
// also caches the device's CU count (the only set-up that may touch host
// containers).
int scratch_for_device(void** out)
{
    int dev = 0;
    GP_HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxScratchDevices)
        return set_error(GP_E_INVALID_ARG, "device %d: the fixed workspace covers devices 0..%d", dev,
                         kMaxScratchDevices - 1);
    std::lock_guard<std::mutex> lk(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            (void)hipGetLastError();
            return set_error(GP_E_HIP, "hipGetSymbolAddress(scratch): %s", hipGetErrorString(e));
        }
        int cus = 0;
        const int rc = device_cus(&cus);
        if (rc != GP_OK) return rc;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return GP_OK;
}

// gp_eval's work on the fixed array: every depth class on the caller's
// stream (no side streams), no timing events, no allocation.
int eval_problem_noalloc(const Problem& pb, hipStream_t stream)
{
    int rc = check_problem(pb);
    if (rc != GP_OK || pb.n_programs == 0) return rc;
    void* base = nullptr;
    if ((rc = scratch_for_device(&base)) != GP_OK) return rc;
    Tuning tu;
    tu.concurrent = 0;
    EvalLaunch el;
    if ((rc = configure_eval(pb, tu, &el)) != GP_OK) return rc;
    if (el.layout.total > kScratchBytes)
        return set_error(GP_E_TOO_LARGE, "the call needs %zu bytes of workspace; the fixed array holds %zu",
                         el.layout.total, kScratchBytes);
    const Staged st = carve(base, el.layout);
    CallEvents ce;
    if ((rc = ce.begin(false)) != GP_OK) return rc;
    return enqueue_eval(pb, tu, el, st, stream, ce);
}

// ------------------------------------------------- Monte-Carlo ranking
// The paper's ranking without a sort (Sec. "Monte-Carlo Ranking", Table 2):
// a random sample of the population's fitness values estimates the
// percentiles, then one pass places every individual in its percentile
// band and gives the band's expected number of children.
//
// key(v): larger is better; NaN (a program that could not be scored) is
// the worst value and ties with -inf (an invalid MSE of +inf).
__device__ __forceinline__ double rank_key(double v, int higher_is_better)
{
    if (v != v) return -__builtin_inf();
    return higher_is_better ? v : -v;
}

// SplitMix64 (Steele, Lea, Flood 2014): the k-th output of the sequence
// started at `seed`, computed directly from the counter.
__device__ __forceinline__ uint64_t splitmix64_at(uint64_t seed, uint64_t k)
{
    uint64_t z = seed + (k + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

constexpr int kMaxRankSample = 1024;

// One workgroup: draw the sample (index k = high 64 bits of h_k * n), read
// the keys, sort them ascending by counting (ties by sample position, so
// the order is a function of the keys only), store them.
__global__ __launch_bounds__(1024) void k_rank_sample(const double* __restrict__ fitness,
                                                      int64_t n, int32_t higher, uint64_t seed,
                                                      int32_t S, double* __restrict__ sorted)
{
    __shared__ double keys[kMaxRankSample];
    const int t = threadIdx.x;
    if (t < S) {
        const uint64_t h = splitmix64_at(seed, (uint64_t)t);
        const int64_t idx = (int64_t)__umul64hi(h, (uint64_t)n);
        keys[t] = rank_key(fitness[idx], higher);
    }
    __syncthreads();
    if (t < S) {
        const double v = keys[t];
        int pos = 0;
        for (int j = 0; j < S; ++j) {
            const double u = keys[j];
            pos += (u < v) || (u == v && j < t);
        }
        sorted[pos] = v;
    }
}

// Expected children per percentile band (Table 2), band b = 10 b ... 10 b + 9.
__constant__ float kChildrenByBand[10] = {0.01f, 0.03f, 0.06f, 0.15f, 0.25f,
                                          0.5f, 1.0f, 1.5f, 2.5f, 4.0f};

// An individual's percentile is 100 x (sampled keys strictly below its key) /
// S, rounded down; its band is that percentile's tens digit (90 and above is
// the top band).  Band b is reached with 10 b S / 100 keys below, rounded up,
// that is when the sorted key before that place is below: nine comparisons.
__device__ __forceinline__ int band_place(int b, int S) { return (10 * b * S + 99) / 100 - 1; }

__device__ __forceinline__ void put_band(double v, const double (&at)[9], int64_t i, int32_t* __restrict__ out_band,
                                         float* __restrict__ out_children)
{
    int band = 0;
#pragma unroll
    for (int b = 0; b < 9; ++b) band += at[b] < v ? 1 : 0;
    out_band[i] = band * 10;
    if (out_children) out_children[i] = kChildrenByBand[band];
}

// One thread per individual.
__global__ __launch_bounds__(256) void k_rank_assign(const double* __restrict__ fitness, int64_t n,
                                                     int32_t higher, int32_t S,
                                                     const double* __restrict__ sorted,
                                                     int32_t* __restrict__ out_band,
                                                     float* __restrict__ out_children)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double at[9];
#pragma unroll
    for (int b = 0; b < 9; ++b) at[b] = sorted[band_place(b + 1, S)];
    put_band(rank_key(fitness[i], higher), at, i, out_band, out_children);
}

// A sample of up to 256: every workgroup draws and sorts it again (100 reads
// that hit L2 and 100 comparisons per thread) while its own individuals are
// on their way, which costs less than a launch before it.  1,000,000
// individuals, sample of 100: 8.4 us, two kernels 12.9; 16 bytes an
// individual are 3 us of memory.
constexpr int kRankWG = 256, kRankEach = 4;
__global__ __launch_bounds__(kRankWG) void k_rank(const double* __restrict__ fitness, int64_t n,
                                                  int32_t higher, uint64_t seed, int32_t S,
                                                  double* __restrict__ sorted, int32_t* __restrict__ out_band,
                                                  float* __restrict__ out_children)
{
    __shared__ double keys[kRankWG];
    __shared__ double places[9];
    const int t = threadIdx.x;
    const int64_t first = (int64_t)blockIdx.x * (kRankWG * kRankEach) + t;
    double mine = 0.0, v[kRankEach];
    if (t < S) {
        const uint64_t h = splitmix64_at(seed, (uint64_t)t);
        mine = fitness[(int64_t)__umul64hi(h, (uint64_t)n)];
    }
#pragma unroll
    for (int k = 0; k < kRankEach; ++k)
        v[k] = first + k * kRankWG < n ? fitness[first + k * kRankWG] : 0.0;
    mine = rank_key(mine, higher);
    if (t < S) keys[t] = mine;
    __syncthreads();
    if (t < S) {
        int pos = 0;
        for (int j = 0; j < S; ++j) {
            const double u = keys[j];
            pos += (u < mine) || (u == mine && j < t);
        }
#pragma unroll
        for (int b = 0; b < 9; ++b)
            if (pos == band_place(b + 1, S)) places[b] = mine;
        if (sorted && blockIdx.x == 0) sorted[pos] = mine;
    }
    __syncthreads();
    double at[9];
#pragma unroll
    for (int b = 0; b < 9; ++b) at[b] = places[b];
#pragma unroll
    for (int k = 0; k < kRankEach; ++k)
        if (first + k * kRankWG < n)
            put_band(rank_key(v[k], higher), at, first + k * kRankWG, out_band, out_children);
}

}  // namespace

// ================================================================ C ABI
extern "C" {

const char* gp_last_error(void) { return g_last_error.c_str(); }

int gp_version(void) { return GPEVAL_VERSION; }

int gp_validate(const uint32_t* nodes, const int64_t* offsets, int64_t n_programs,
                int64_t n_consts, int32_t n_vars, uint32_t allowed_op_mask,
                int32_t* status, int32_t* max_depth, int64_t* first_bad)
{
    if (n_programs < 0 || n_consts < 0 || n_vars < 0)
        return set_error(GP_E_INVALID_ARG, "negative size");
    if (n_programs > 0 && (!offsets)) return set_error(GP_E_INVALID_ARG, "offsets is NULL");
    const uint32_t allowed = allowed_op_mask ? allowed_op_mask : GP_ALL_OPS;
    int64_t bad_at = -1;
    for (int64_t p = 0; p < n_programs; ++p) {
        const int64_t s = offsets[p], e = offsets[p + 1];
        int st = GP_PROG_OK, md = 0;
        if (s < 0 || e < s) st = GP_PROG_BAD_OFFSETS;
        else if (e == s) st = GP_PROG_EMPTY;
        else if (!nodes) st = GP_PROG_BAD_OFFSETS;
        else {
            GclCheck gc;
            for (int64_t k = s; k < e && st == GP_PROG_OK; ++k)
                st = gc.step(nodes[k] & 0xFFu, nodes[k] >> 8, allowed, n_vars, n_consts);
            if (st == GP_PROG_OK) st = gc.finish();
            md = gc.maxd;
        }
        if (status) status[p] = st;
        if (max_depth) max_depth[p] = md;
        if (st != GP_PROG_OK && bad_at < 0) bad_at = p;
    }
    if (first_bad) *first_bad = bad_at;
    if (bad_at >= 0) return set_error(GP_E_BAD_PROGRAM, "program %lld is invalid", (long long)bad_at);
    return GP_OK;
}

int gp_eval(const uint32_t* nodes, const int64_t* offsets, int64_t n_programs,
            int64_t n_nodes, const float* consts, int64_t n_consts,
            const float* X, int32_t n_vars, int64_t ld_x,
            const float* y, int64_t n_cases,
            double tax_on_length, uint32_t allowed_op_mask,
            double* out_fitness, int32_t* out_status, hipStream_t stream)
{
    const gp_problem d{nodes, offsets, n_programs, n_nodes, consts, n_consts, X, n_vars, ld_x,
                       y, n_cases, tax_on_length, allowed_op_mask, out_fitness, out_status};
    return eval_problem(make_problem(&d), stream);
}

int gp_eval_noalloc(const uint32_t* nodes, const int64_t* offsets, int64_t n_programs,
                    int64_t n_nodes, const float* consts, int64_t n_consts,
                    const float* X, int32_t n_vars, int64_t ld_x,
                    const float* y, int64_t n_cases,
                    double tax_on_length, uint32_t allowed_op_mask,
                    double* out_fitness, int32_t* out_status, hipStream_t stream)
{
    const gp_problem d{nodes, offsets, n_programs, n_nodes, consts, n_consts, X, n_vars, ld_x,
                       y, n_cases, tax_on_length, allowed_op_mask, out_fitness, out_status};
    return eval_problem_noalloc(make_problem(&d), stream);
}

int gp_eval_correlation(const uint32_t* nodes, const int64_t* offsets, int64_t n_programs,
                        int64_t n_nodes, const float* consts, int64_t n_consts,
                        const float* X, int32_t n_vars, int64_t ld_x,
                        const float* y, int64_t n_cases, double max_score,
                        uint32_t allowed_op_mask, double* out_score, int32_t* out_status,
                        hipStream_t stream)
{
    if (!std::isfinite(max_score)) return set_error(GP_E_INVALID_ARG, "max_score is not finite");
    const gp_problem d{nodes, offsets, n_programs, n_nodes, consts, n_consts, X, n_vars, ld_x,
                       y, n_cases, 0.0, allowed_op_mask, out_score, out_status};
    Problem pb = make_problem(&d);
    pb.fit = kFitCorr;
    pb.max_score = max_score;
    return eval_problem(pb, stream);
}

int gp_eval_reward(const uint32_t* nodes, const int64_t* offsets, int64_t n_programs,
                   int64_t n_nodes, const float* consts, int64_t n_consts,
                   const float* X, int32_t n_vars, int64_t ld_x,
                   const float* y, int64_t n_cases, double max_score, int32_t power,
                   uint32_t allowed_op_mask, double* out_reward, int32_t* out_status,
                   hipStream_t stream)
{
    if (!(std::fabs(max_score) <= GP_MAX_REWARD_SCORE) || max_score != std::trunc(max_score))
        return set_error(GP_E_INVALID_ARG, "max_score is not an integer of magnitude <= 2^24");
    if (power != 1 && power != 2 && power != 3 && power != 8)
        return set_error(GP_E_INVALID_ARG, "power %d is not 1, 2, 3 or 8", (int)power);
    const gp_problem d{nodes, offsets, n_programs, n_nodes, consts, n_consts, X, n_vars, ld_x,
                       y, n_cases, 0.0, allowed_op_mask, out_reward, out_status};
    Problem pb = make_problem(&d);
    pb.fit = kFitReward;
    pb.max_score = max_score;
    pb.reward_power = power;
    return eval_problem(pb, stream);
}

int gp_mc_rank(const double* fitness, int64_t n, int32_t higher_is_better, uint64_t seed,
               int32_t sample_size, int32_t* out_band, float* out_children,
               double* out_sample_keys, hipStream_t stream)
{
    if (n < 0) return set_error(GP_E_INVALID_ARG, "n < 0");
    if (sample_size < 1 || sample_size > kMaxRankSample)
        return set_error(GP_E_INVALID_ARG, "sample_size must be 1..%d", kMaxRankSample);
    if (n == 0) return GP_OK;
    if (!fitness || !out_band) return set_error(GP_E_INVALID_ARG, "NULL fitness or out_band");
    const int32_t hb = higher_is_better ? 1 : 0;
    if (sample_size <= kRankWG) {
        const int64_t share = kRankWG * kRankEach;
        hipLaunchKernelGGL(k_rank, dim3((unsigned)((n + share - 1) / share)), dim3(kRankWG), 0, stream, fitness, n,
                           hb, seed, sample_size, out_sample_keys, out_band, out_children);
        GP_HIP_TRY(hipGetLastError());
        return GP_OK;
    }
    double* sorted = out_sample_keys;
    if (!sorted) {
        Workspace* w = nullptr;
        const int rc = get_workspace(stream, (size_t)sample_size * sizeof(double), &w);
        if (rc != GP_OK) return rc;
        sorted = static_cast<double*>(w->ptr);
    }
    hipLaunchKernelGGL(k_rank_sample, dim3(1), dim3(kMaxRankSample), 0, stream, fitness, n, hb,
                       seed, sample_size, sorted);
    GP_HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(k_rank_assign, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream,
                       fitness, n, hb, sample_size, sorted, out_band, out_children);
    GP_HIP_TRY(hipGetLastError());
    return GP_OK;
}

int gp_eval_batched(const gp_request* requests_dev, int32_t n_requests,
                    const gp_dataset* datasets_dev, int32_t n_datasets,
                    int64_t total_programs, int64_t total_nodes,
                    int32_t max_n_vars, int64_t max_n_cases, uint32_t allowed_op_mask,
                    hipStream_t stream)
{
    if (!requests_dev) return set_error(GP_E_INVALID_ARG, "requests_dev is NULL");
    Problem pb{};
    pb.req_dev = requests_dev; pb.n_req = n_requests;
    pb.ds_dev = datasets_dev; pb.n_ds = n_datasets;
    pb.n_programs = total_programs; pb.n_nodes = total_nodes;
    pb.max_vars = max_n_vars; pb.max_cases = max_n_cases;
    pb.allowed = allowed_op_mask ? allowed_op_mask : GP_BASE_OPS;
    pb.need_out = 1;
    return eval_problem(pb, stream);
}

int gp_predict(const uint32_t* nodes, const int64_t* offsets, int64_t n_programs,
               int64_t n_nodes, const float* consts, int64_t n_consts,
               const float* X, int32_t n_vars, int64_t ld_x, int64_t n_cases,
               uint32_t allowed_op_mask, float* out, int64_t ld_out, int32_t* out_status,
               hipStream_t stream)
{
    int rc = check_common(n_programs, n_nodes, n_consts, n_vars, ld_x, n_cases);
    if (rc != GP_OK) return rc;
    if (n_programs == 0) return GP_OK;
    if (!offsets || !out) return set_error(GP_E_INVALID_ARG, "NULL offsets or out");
    if (ld_out < n_cases) return set_error(GP_E_INVALID_ARG, "ld_out < n_cases");
    if ((rc = check_pointers(nodes, n_nodes, consts, n_consts, X, n_vars)) != GP_OK) return rc;
    // work items (program, sub-tile) are counted in 32 bits
    if ((double)n_programs * (double)((n_cases + 511) / 512) > 2.0e9)
        return set_error(GP_E_TOO_LARGE, "n_programs * n_cases too large for one gp_predict call");
    Problem pb{};
    pb.one_req.nodes = nodes; pb.one_req.offsets = offsets; pb.one_req.consts = consts;
    pb.one_req.n_programs = n_programs; pb.one_req.n_nodes = n_nodes;
    pb.one_req.n_consts = n_consts; pb.one_req.out_status = out_status;
    pb.n_req = 1;
    pb.one.X = X; pb.one.y = nullptr;
    pb.one.ld_x = ld_x; pb.one.n_cases = n_cases; pb.one.tax_on_length = 0.0;
    pb.one.n_vars = n_vars;
    pb.n_ds = 1;
    pb.n_programs = n_programs; pb.n_nodes = n_nodes;
    pb.max_vars = n_vars; pb.max_cases = n_cases;
    pb.allowed = allowed_op_mask ? allowed_op_mask : GP_ALL_OPS;
    pb.need_out = 0;
    pb.fit = kFitPredict;
    Tuning tu;
    tu.tile_max = predict_tiles(n_programs);
    EvalLaunch el;
    if ((rc = configure_eval(pb, tu, &el)) != GP_OK) return rc;
    Workspace* w = nullptr;
    if ((rc = get_workspace(stream, el.layout.total, &w)) != GP_OK) return rc;
    const Staged st = carve(w->ptr, el.layout);
    if ((rc = enqueue_stage(pb, tu, el, st, stream)) != GP_OK) return rc;
    if ((rc = enqueue_run(pb, el, st, stream, out, ld_out)) != GP_OK) return rc;
    hipLaunchKernelGGL(k_fill_invalid, dim3((unsigned)n_programs), dim3(256), 0, stream, st.cls,
                       n_cases, out, ld_out);
    GP_HIP_TRY(hipGetLastError());
    return GP_OK;
}

int gp_plan_create(gp_plan** plan, const gp_problem* problem, const gp_tuning* tuning,
                   int autotune, hipStream_t stream)
{
    if (!plan || !problem) return set_error(GP_E_INVALID_ARG, "NULL plan or problem");
    *plan = nullptr;
    const Problem pb = make_problem(problem);
    int rc = check_problem(pb);
    if (rc != GP_OK) return rc;
    if (pb.n_programs == 0) return set_error(GP_E_INVALID_ARG, "a plan needs n_programs >= 1");
    gp_plan* p = new gp_plan();
    p->pb = pb;
    if (tuning) {
        if (tuning->programs_per_item < 0 || tuning->programs_per_item > 128 || tuning->wg_per_cu < 0 ||
            tuning->tile_lds_bytes < 0 || (tuning->tile_lds_bytes > 0 && (tuning->tile_lds_bytes < 4096 ||
                                                                         tuning->tile_lds_bytes > 65536)) ||
            tuning->max_tiles < 0 || tuning->max_tiles > kMaxTiles ||
            tuning->concurrent_classes < 0 || tuning->concurrent_classes > 2) {
            delete p;
            return set_error(GP_E_INVALID_ARG, "tuning out of range");
        }
        if (tuning->programs_per_item > 0) p->tu.G = tuning->programs_per_item;
        p->tu.wg_per_cu = tuning->wg_per_cu;
        p->tu.concurrent = tuning->concurrent_classes;
        if (tuning->tile_lds_bytes > 0) p->tu.tile_lds = tuning->tile_lds_bytes;
        if (tuning->max_tiles > 0) p->tu.tile_max = tuning->max_tiles;
    }
    if (hipGetDevice(&p->device) != hipSuccess ||
        hipStreamCreateWithFlags(&p->cap, hipStreamNonBlocking) != hipSuccess) {
        gp_plan_destroy(p);
        return set_error(GP_E_HIP, "plan stream setup failed");
    }
    // workspace for the largest candidate configuration (the most programs
    // per item and the most tiles per program)
    EvalLaunch el;
    Tuning big = p->tu;
    big.G = 128;
    big.tile_max = kMaxTiles;
    if ((rc = configure_eval(pb, big, &el)) != GP_OK ||
        hipMalloc(&p->ws, el.layout.total) != hipSuccess) {
        (void)hipGetLastError();
        gp_plan_destroy(p);
        return rc != GP_OK ? rc : set_error(GP_E_NO_MEMORY, "plan workspace");
    }
    p->ws_bytes = el.layout.total;
    if (autotune && (rc = plan_autotune(p, stream)) != GP_OK) {
        gp_plan_destroy(p);
        return rc;
    }
    if ((rc = plan_build(p)) != GP_OK) {
        gp_plan_destroy(p);
        return rc;
    }
    *plan = p;
    return GP_OK;
}

int gp_plan_launch(gp_plan* plan, hipStream_t stream)
{
    if (!plan || !plan->exec) return set_error(GP_E_INVALID_ARG, "plan is not built");
    GP_HIP_TRY(hipGraphLaunch(plan->exec, stream));
    return GP_OK;
}

int gp_plan_update(gp_plan* plan, const gp_problem* problem)
{
    if (!plan || !problem) return set_error(GP_E_INVALID_ARG, "NULL plan or problem");
    const Problem pb = make_problem(problem);
    int rc = check_problem(pb);
    if (rc != GP_OK) return rc;
    if (pb.n_programs == 0) return set_error(GP_E_INVALID_ARG, "a plan needs n_programs >= 1");
    plan->pb = pb;
    return plan_build(plan);
}

int gp_plan_get_tuning(const gp_plan* plan, gp_tuning* out)
{
    if (!plan || !out) return set_error(GP_E_INVALID_ARG, "NULL plan or out");
    out->programs_per_item = plan->tu.G;
    out->wg_per_cu = plan->tu.wg_per_cu;
    out->concurrent_classes = plan->tu.concurrent;
    out->tile_lds_bytes = plan->tu.tile_lds;
    out->max_tiles = plan->tu.tile_max;
    return GP_OK;
}

void gp_plan_destroy(gp_plan* plan)
{
    if (!plan) return;
    if (plan->cap) (void)hipStreamSynchronize(plan->cap);
    (void)hipDeviceSynchronize();
    plan_release_graph(plan);
    if (plan->cap) (void)hipStreamDestroy(plan->cap);
    if (plan->ws) (void)hipFree(plan->ws);
    delete plan;
}

int gp_timing_enable(int on)
{
    g_timing.on = on != 0;
    return GP_OK;
}

int gp_timing_reset(void)
{
    for (auto& evs : g_timing.pending)
        for (auto& e : evs) (void)hipEventDestroy(e);
    g_timing.pending.clear();
    for (double& m : g_timing.ms) m = 0.0;
    g_timing.calls = 0;
    return GP_OK;
}

int gp_timing_read(double* ms, int64_t* n_calls)
{
    int rc = GP_OK;
    for (auto& evs : g_timing.pending) {
        if (hipEventSynchronize(evs[GP_TIMING_PHASES - 1]) != hipSuccess) {
            rc = set_error(GP_E_HIP, "hipEventSynchronize failed");
            break;
        }
        float t = 0.f;
        for (int i = 0; i + 1 < GP_TIMING_PHASES; ++i) {
            if (hipEventElapsedTime(&t, evs[i], evs[i + 1]) == hipSuccess) g_timing.ms[i] += t;
        }
        if (hipEventElapsedTime(&t, evs[0], evs[GP_TIMING_PHASES - 1]) == hipSuccess)
            g_timing.ms[GP_TIMING_PHASES - 1] += t;
        g_timing.calls += 1;
        for (auto& e : evs) (void)hipEventDestroy(e);
    }
    g_timing.pending.clear();
    if (ms)
        for (int i = 0; i < GP_TIMING_PHASES; ++i) ms[i] = g_timing.ms[i];
    if (n_calls) *n_calls = g_timing.calls;
    return rc;
}

int gp_workspace_size(int64_t n_programs, int64_t n_nodes, int32_t n_requests,
                      int32_t n_datasets, int32_t max_n_vars, int64_t max_n_cases,
                      size_t* bytes)
{
    if (!bytes) return set_error(GP_E_INVALID_ARG, "bytes is NULL");
    if (n_programs < 0 || n_nodes < 0 || n_requests < 1 || n_datasets < 1 || max_n_vars < 0 ||
        max_n_cases < 1)
        return set_error(GP_E_INVALID_ARG, "sizes out of range");
    int32_t stride = 1;
    for (int c = 0; c < kClasses; ++c) {
        const int32_t t = max_tiles(max_n_cases, class_k(c, max_n_vars), kMaxTiles);
        if (t > stride) stride = t;
    }
    const size_t need = make_layout(n_programs, n_nodes, stride, n_datasets, n_requests).total;
    *bytes = need + need / 4;      // the growth slack get_workspace adds
    return GP_OK;
}

}  // extern "C"

// Drops the cached workspace of one stream (the server calls it before it
// destroys its streams).  Not exported.
__attribute__((visibility("hidden"))) void gp_internal_release_stream_workspace(hipStream_t stream)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return;
    std::lock_guard<std::mutex> lk(g_ws_mutex);
    auto it = g_ws.find(std::make_pair(dev, stream));
    if (it == g_ws.end()) return;
    (void)hipStreamSynchronize(stream);
    if (it->second.ptr) (void)hipFree(it->second.ptr);
    g_ws.erase(it);
}

extern "C" {

void gp_release_workspaces(void)
{
    std::lock_guard<std::mutex> lk(g_ws_mutex);
    for (auto& kv : g_ws) {
        (void)hipStreamSynchronize(kv.first.second);
        if (kv.second.ptr) (void)hipFree(kv.second.ptr);
    }
    g_ws.clear();
}

}  // extern "C"
