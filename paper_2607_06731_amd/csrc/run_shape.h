// run_shape.h -- how a scoring call's work is cut: case tiles and windows of a
// dataset (and so a program's summation order), and the evaluation kernel's work
// items and LDS.  Host and device share it, so that the cut can be checked
// without a GPU.
//
// The includer provides __host__, __device__ and <cstdint>.
#pragma once

constexpr int kClasses = 3;              // max depth <= 8, <= 16, <= 32
constexpr int kMaxTiles = 32;            // case tiles per program (cap)

// Cases per lane of a class's sub-tile, the unit in which its cases are
// grouped into windows and tiles (and so its summation order).  Depends only
// on the class, never on the rest of the population.  (Lane t holds cases t,
// t + 64, t + 128, ... whatever the unit, so the interpreter may run two
// sub-tiles at once.)
__host__ __device__ inline int class_k(int c, int n_vars) { return c == 2 ? 2 : 4; }

// Tile geometry for one class.  A sub-tile is 64*K cases (one wavefront, K
// per lane).  The inputs and targets of `window` sub-tiles fit the LDS tile
// budget together ((n_vars + 1) rows of 64*K floats each), so a wavefront
// runs a program over a whole window without a barrier.  A tile is `passes`
// consecutive sub-tiles (a whole number of windows where the case count
// allows, at most 32 tiles per program); a work item covers one tile of G
// programs.  Depends only on (n_cases, K, n_vars) -- the dataset -- so a
// program's summation order never depends on the rest of the population or
// the batch.
constexpr int kTileLds = 24 * 1024;      // LDS bytes for input windows (6 workgroups per CU)
constexpr int kMaxWindow = 8;

struct TileShape {
    int32_t sub;        // cases per sub-tile (64 * K)
    int32_t passes;     // sub-tiles per tile
    int32_t n_tiles;    // tiles covering n_cases
    int32_t window;     // sub-tiles staged in LDS at once
};

__host__ __device__ inline int32_t tile_window(int k, int n_vars, int32_t lds_bytes)
{
    const int64_t block = (int64_t)(n_vars + 1) * 64 * k * 4;
    int64_t w = lds_bytes / block;
    return (int32_t)(w < 1 ? 1 : (w > kMaxWindow ? kMaxWindow : w));
}

__host__ __device__ inline TileShape tile_shape(int64_t n_cases, int k, int n_vars,
                                               int32_t lds_bytes, int32_t max_t)
{
    TileShape t;
    t.sub = 64 * k;
    const int64_t n_sub = (n_cases + t.sub - 1) / t.sub;
    t.window = tile_window(k, n_vars, lds_bytes);
    int64_t passes = (n_sub + max_t - 1) / max_t;
    if (passes < t.window) passes = t.window < n_sub ? t.window : n_sub;
    if (passes < 1) passes = 1;
    t.passes = (int32_t)passes;
    t.n_tiles = (int32_t)((n_sub + passes - 1) / passes);
    return t;
}

// Partial slots per program that any dataset of at most max_cases cases
// can need: n_tiles never exceeds kMaxTiles or the sub-tile count, and the
// sub-tile count grows with n_cases, so a smaller dataset can need more
// tiles than the largest one (33 sub-tiles make 17 tiles, 32 make 32).
__host__ __device__ inline int32_t max_tiles(int64_t max_cases, int k, int32_t max_t)
{
    const int64_t n_sub = (max_cases + 64 * k - 1) / (64 * k);
    return (int32_t)(n_sub < max_t ? (n_sub < 1 ? 1 : n_sub) : max_t);
}

// How a class's work is cut into items.  An item is G programs over m
// consecutive case tiles, one workgroup's work between two barriers.
// m is as large as the workgroup's LDS holds (item_tiles), capped so that at
// least four (program, tiles) runs remain per wavefront of the GPU.
// G (programs) is as large as g_max allows while the class still has about
// target_items items, and at least one program per wavefront: larger groups
// balance a workgroup's wavefronts (each takes the next program).  Neither
// changes a result.
constexpr int kRunWaves = 8;             // wavefronts of an evaluation workgroup
constexpr int kRunWG = 64 * kRunWaves;
constexpr double kGpuWaves = 6144.0;     // evaluation wavefronts resident on the GPU
constexpr int kListed = 192;             // programs a workgroup lists between two barriers
constexpr uint32_t kManyRuns = 8u, kFewItems = 8u;      // runs of tiles; items per workgroup
// Programs of an item that the next one may follow, at least; up to 64 where they
// run over few cases each: the next items' programs are listed meanwhile, which
// takes about 5 us, and 16 programs over one sub-tile are over before that
// (1,000,000 programs of 3-8 nodes x 100 cases: k_run 730 us with 16, 433 with 64;
// x 1,000 cases 823 and 811).
constexpr int kRunOn = 16;
constexpr int64_t kRunOnCases = 64 * 256;    // an item's programs times their cases
constexpr int kChunkMax = 64;            // programs of an item, at most
constexpr int kWarmLines = 6;
// prog_tiles: the class's (program, tile) pairs
__host__ __device__ inline int32_t cut_tiles(double prog_tiles)
{
    const double cap = prog_tiles / (4.0 * kGpuWaves);
    return cap >= (double)kMaxTiles ? kMaxTiles : (cap < 1.0 ? 1 : (int32_t)cap);
}
// runs: the class's (program, m tiles) pairs
__host__ __device__ inline int32_t cut_programs(double runs, int32_t g_max, int32_t target_items)
{
    int32_t G = g_max;
    while (G > kRunWaves && runs / (double)G < (double)target_items) G >>= 1;
    return G < 1 ? 1 : G;
}

// Cases of a class's sub-tile (64 per case held by a lane).
__host__ __device__ constexpr int sub_cases(int c) { return c == 2 ? 128 : 256; }

// Rows of the staged memory: the inputs, and the targets where there are any
// (gp_predict has none).
__host__ __device__ constexpr int32_t staged_rows(bool outputs_only, int32_t n_vars)
{
    return n_vars + (outputs_only ? 0 : 1);
}

// Cases (a multiple of 256) whose rows (the inputs, and the targets) fit the
// staged memory.
__host__ __device__ inline int64_t staged_cases(int32_t lds_floats, int32_t rows)
{
    const int64_t n = lds_floats / (rows < 1 ? 1 : rows) / 256 * 256;
    return n < 256 ? 256 : n;
}

// Case tiles per item of one dataset: what the staged memory holds, spread
// evenly over the dataset's tiles; 1 when a tile is larger than that (the
// item then stages it piece by piece).
__host__ __device__ inline int32_t item_tiles(int32_t passes, int32_t n_tiles, int c, int32_t rows,
                                              int32_t lds_floats, int32_t m_cap)
{
    int64_t m = staged_cases(lds_floats, rows) / ((int64_t)passes * sub_cases(c));
    m = m < m_cap ? m : m_cap;
    m = m < 1 ? 1 : (m < n_tiles ? m : n_tiles);
    const int32_t groups = (int32_t)((n_tiles + m - 1) / m);
    return (n_tiles + groups - 1) / groups;
}
__host__ __device__ inline int32_t item_groups(int32_t n_tiles, int32_t m) { return (n_tiles + m - 1) / m; }

// A class of fewer (program, tile) pairs than the GPU holds wavefronts ends
// with its longest program: its pairs are split into units of 256 cases, which
// wavefronts take one by one, leaving the program's outputs in LDS; the one
// that finishes a program's last unit sums them up, in the order of a whole
// run.  gp_predict has nothing to sum and splits always.  Returns the programs
// per item, 0 for no split.  (us per call: 1,000 programs x 1,024 cases 44 ->
// 35; the whole command table, 2,000 x 2,048, 94 -> 74; outputs of 1,000 x 16,384
// 110 -> 101.  10,000 x 4,096, 6.5 pairs per wavefront: 268 either way.)
constexpr int kSplitMax = 8;             // programs per item
__host__ __device__ inline int32_t split_programs(int64_t tile_cases, int64_t n_cases, int32_t n_tiles, int32_t rows,
                                                  int32_t count, int32_t g_max, int32_t target_items,
                                                  int32_t lds_floats, bool free_outputs)
{
    const int64_t tile = tile_cases < n_cases ? tile_cases : n_cases;
    const int32_t stride = (int32_t)((tile + 255) & ~(int64_t)255), units = stride >> 8;
    if (units < 2) return 0;
    int32_t most = g_max < kSplitMax ? g_max : kSplitMax;
    if (!free_outputs) {
        if ((double)count * (double)n_tiles > kGpuWaves) return 0;
        const int32_t room = (lds_floats - rows * stride) / stride;
        most = most < room ? most : room;
        if (most < 1) return 0;
    }
    int32_t G = kRunWaves / units > 1 ? kRunWaves / units : 1;
    while (G > most) G >>= 1;
    while (2 * G <= most && (double)count * (double)n_tiles / G > (double)(target_items / 4)) G *= 2;
    return G;
}

// The cut of one class of a call of one request.
struct ClassCut {
    int32_t G, m_cap;       // programs per item; case tiles per item, at most
    int32_t split;          // cases are split
    uint32_t items;
};
__host__ __device__ inline ClassCut class_cut(int c, int32_t count, int32_t passes, int32_t n_tiles, int64_t n_cases,
                                              int32_t rows, int32_t g_max, int32_t target_items, int32_t lds_floats,
                                              bool may_split, bool free_outputs)
{
    ClassCut r;
    const int64_t tile = (int64_t)passes * sub_cases(c);
    r.m_cap = cut_tiles((double)count * (double)n_tiles);
    const int32_t m = item_tiles(passes, n_tiles, c, rows, lds_floats, r.m_cap);
    const int32_t groups = item_groups(n_tiles, m);
    // (items over the same cases follow each other without a barrier, so
    // small ones cost nothing and end the launch evenly)
    const bool whole = tile <= staged_cases(lds_floats, rows);
    int32_t most = g_max;
    if (whole) {
        const int64_t all = (n_cases + 255) & ~(int64_t)255;
        const int64_t cases = m * tile < all ? m * tile : all;
        int32_t on = kRunOn;
        while (2 * on * cases <= kRunOnCases) on *= 2;
        most = most < on ? most : on;
    }
    r.G = cut_programs((double)count * (double)groups, most, target_items);
    const int32_t split = may_split && whole && m == 1
                              ? split_programs(tile, n_cases, n_tiles, rows, count, g_max, target_items, lds_floats,
                                               free_outputs)
                              : 0;
    if (split) r.G = split;
    r.split = split != 0;
    r.items = (uint32_t)((count + r.G - 1) / r.G) * (uint32_t)groups;
    return r;
}

// Cases of a tile that are staged at once, where it is larger than the staged
// memory: whole windows.
__host__ __device__ inline int64_t piece_cases(int64_t cap, int32_t window)
{
    return (cap / window > 1 ? cap / window : 1) * window;
}

// LDS for staged inputs that leaves room for three workgroups per CU (160 KB).
constexpr int kRunLds = 48 * 1024;
// Floats of staged inputs and targets: at least a sub-tile of the widest dataset,
// and every window (a window of sub-tiles of 128 cases may round up by a third).
// A multiple of four: the running sums behind them hold 64-bit values.
inline int32_t run_lds_floats(int32_t rows, int32_t tile_lds)
{
    const int64_t one = (int64_t)(rows < 1 ? 1 : rows) * 256;
    const int64_t want = kRunLds / 4 > tile_lds / 3 ? kRunLds / 4 : tile_lds / 3;
    return (int32_t)(((one > want ? one : want) + 3) & ~(int64_t)3);
}

// Variables from which a sub-tile takes most of the LDS (k_run's WIDE).
constexpr int32_t kWideVars = 128;

// Case tiles per program of gp_predict, at most.  Outputs are not summed, so a tile
// can be as small as a window, and few programs over many cases need that to fill
// the GPU: about four (program, tile) pairs per wavefront (32 tiles: 1 program x
// 1,000,000 cases 310 us, 8 programs 728; so many: 36 and 69.  As many as
// windows whatever the programs: 1,000 x 10,000 with 20 variables 95 -> 111).
inline int32_t predict_tiles(int64_t n_programs)
{
    const int64_t t = 4 * (int64_t)kGpuWaves / (n_programs < 1 ? 1 : n_programs);
    return (int32_t)(t < kMaxTiles ? kMaxTiles : t);
}
