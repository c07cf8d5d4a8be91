// Host harness for the threaded words (paper_2607_06731_amd/csrc/threaded.h),
// built by tests/test_threaded_words.py with the host compiler.
//
// TEST INFRASTRUCTURE.  Stages every program of an input population twice
// with the library's benchmark-set walk (staging.h), in the flag form and in
// the threaded form, and checks the two word by word: the threaded word of
// each instruction names the block of its stack depth (block 0 for the last
// word only), the offset of its operator, and the same payload; the depth
// stays within the program's depth class, so the handler exists in the
// class's table.
//
// Input (binary, little endian): int64 P, n_nodes, n_consts, n_vars; uint32
// nodes[n_nodes]; int64 offsets[P + 1]; float consts[n_consts].
// Output (text): valid programs, words checked, first differing program or -1.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <vector>

#define __host__
#define __device__
#include "gpeval.h"

static inline uint32_t __float_as_uint(float f)
{
    uint32_t u;
    memcpy(&u, &f, 4);
    return u;
}
typedef float lds_f32;
constexpr int kHeldConsts = 16;
constexpr int kBucketBlock = 1;

static inline float binary_value(uint32_t op, float a, float b)
{
    switch (op) {
    case GP_ADD: return a + b;
    case GP_SUB: return a - b;
    case GP_MUL: return a * b;
    default: return fabsf(b) <= 0.001f ? 1.f : a / b;
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
    default: return fabsf(x);
    }
}

#define GP_STAGING_FN
#include "staging.h"
#include "threaded.h"

struct Reader {
    const uint32_t* p;
    const float* c;
    int64_t nc;
    uint32_t op(int64_t k) const
    {
        const uint32_t o = (p[k] & 0xFFu) < 32u ? (p[k] & 0xFFu) : 0xFFu;
        return o == GP_CONST && (int64_t)(p[k] >> 8) >= nc ? kOpBadConst : o;
    }
    uint32_t pay(int64_t k) const { return p[k] >> 8; }
    float cval(int64_t, uint32_t pay) const { return c[pay]; }
};

// offset of a flag word's operator in its block, and its change of depth
static uint32_t offset_of(uint32_t f, int* change)
{
    static const uint32_t un[6] = {1792, 2208, 2688, 3008, 3200, 3296};
    const uint32_t sel = (f >> 8) & 0xFu;
    *change = 0;
    if (f & kFUn) {
        if (!(f & kFPush)) return un[sel];
        *change = 1;
        return kThPushUn + 64u * sel;
    }
    if (f & kFSBin) {
        *change = -1;
        return kThBin + 64u * sel;
    }
    if (f & kFLBin) return f & kFConst ? kThBinC + 64u * sel : kThBinV + 96u * sel;
    *change = 1;
    return f & kFConst ? kThPushC : kThPushV;
}

template <class T> static bool rd(FILE* f, T* p, size_t n) { return fread(p, sizeof(T), n, f) == n; }

int main(int argc, char** argv)
{
    if (argc != 2) return 2;
    FILE* in = fopen(argv[1], "rb");
    if (!in) return 2;
    int64_t hd[4];
    if (!rd(in, hd, 4)) return 2;
    const int64_t P = hd[0], NN = hd[1], NC = hd[2], NV = hd[3];
    std::vector<uint32_t> nodes(NN + 1);
    std::vector<int64_t> off(P + 1);
    std::vector<float> consts(NC + 1);
    if (!rd(in, nodes.data(), NN) || !rd(in, off.data(), P + 1) || !rd(in, consts.data(), NC)) return 2;
    fclose(in);
    long long valid = 0, words = 0, bad = -1;
    for (int64_t p = 0; p < P && bad < 0; ++p) {
        const int64_t s = off[p], e = off[p + 1];
        std::vector<uint2> a(e - s + 1), b(e - s + 1);
        float pv[kHeldConsts];
        const Reader r{nodes.data(), consts.data(), NC};
        int st1 = 0, md1 = 0, st2 = 0, md2 = 0;
        const int64_t n1 = stage_check_base(r, s, e, GP_BASE_OPS, (int32_t)NV, a.data(), pv, st1, md1);
        const int64_t n2 = stage_check_base<ThreadedWords>(r, s, e, GP_BASE_OPS, (int32_t)NV, b.data(),
                                                           pv, st2, md2);
        if (st1 != st2 || md1 != md2 || (st1 == GP_PROG_OK && n1 != n2)) bad = p;
        if (st1 != GP_PROG_OK || bad >= 0) continue;
        ++valid;
        const int maxd = md1 <= 8 ? 8 : (md1 <= 16 ? 16 : 32);
        int d = 0;
        for (int64_t k = 0; k < n1; ++k, ++words) {
            int change = 0;
            const uint32_t want = offset_of(a[k].x, &change);
            const bool last = (a[k].x & kFLast) != 0;
            // (the benchmark set has no cold words)
            const uint32_t at = b[k].x - kThHot0, blk = at / kThHot, o = at % kThHot;
            const int need = change < 0 ? 2 : (change > 0 ? 0 : 1);
            // a leaf taken as an operand sits in the cell above the top
            const bool leaf_op = o >= kThBinC && o < kThSubCR;
            if (o != want || b[k].y != a[k].y || blk != (last ? 0u : (uint32_t)(d + 1)) ||
                last != (k == n1 - 1) || d < need || d + (change > 0) > maxd ||
                (leaf_op && d + 1 > maxd))
                bad = p;
            d += change;
        }
        if (d != 1) bad = p;
    }
    printf("%lld %lld %lld\n", valid, words, bad);
    return 0;
}
