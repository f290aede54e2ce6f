// Declarations shared by the library's own translation units (not part of the
// C ABI and not used by the CPU oracle).
#ifndef AMULET_INTERNAL_H
#define AMULET_INTERNAL_H

#include <hip/hip_runtime.h>
#include <atomic>
#include <stdint.h>
#include <stdlib.h>

namespace amulet {

enum { TASK_IDENTITY = 0, TASK_DISCOUNT = 1, TASK_BOOST = 2, TASK_COUNT_GT = 3 };
// form of the threshold operand (paper Sec. 6.3): thres[j], thres[i], a constant, thres[i][j]
enum { THRES_COL = 0, THRES_ROW = 1, THRES_CONST = 2, THRES_ELEM = 3 };

// XCD-aware tile order, shared by every tiled kernel.  Workgroups are handed to the 8 XCDs
// round-robin (workgroup b runs on XCD b % 8) and each XCD has its own L2.  The tile grid of R
// is cut into 8 rectangular parts, px column parts by 8 / px row parts, and XCD x walks its
// part row tile by row tile: the workgroups resident on an XCD at any moment form a compact
// block of R that shares A rows and B columns through that L2.  px is the one of 8, 4, 2, 1
// whose largest part is smallest (ties go to more column parts), so that narrow grids and
// column counts that are not multiples of 8 still give every XCD a part.  (Used as the tile order
// when the parts cover the grid exactly, see below.)
struct XcdParts {
    int px;   // column parts
    int cw;   // column tiles per part
    int rh;   // row tiles per part
};
__host__ __device__ inline XcdParts xcd_parts(int64_t tiles_m, int64_t tiles_n)
{
    XcdParts best = {8, 0, 0};
    int64_t best_size = -1;
    for (int px = 8; px >= 1; px >>= 1) {
        const int py = 8 / px;
        const int64_t cw = (tiles_n + px - 1) / px, rh = (tiles_m + py - 1) / py;
        if (best_size < 0 || cw * rh < best_size) {
            best_size = cw * rh;
            best.px = px;
            best.cw = (int)cw;
            best.rh = (int)rh;
        }
    }
    return best;
}
// The parts cover the grid exactly (no padding) when both tile counts divide.  Otherwise some
// XCDs would get less than others, up to nothing (33 column tiles in 8 parts of 5: the last XCD
// idle, the one before it at 3 / 5), and the launch takes as long as its fullest XCD.  Then the
// tiles are put in one order instead -- column panels as wide as a part would be, row tile by
// row tile inside a panel -- and that order is cut into 8 runs of equal length (to within one
// tile): XCD x takes run x, still a compact block of R, and every XCD has the same number of tiles.
__host__ __device__ inline bool xcd_parts_exact(const XcdParts &g, int64_t tiles_m, int64_t tiles_n)
{
    return 8LL * g.cw * g.rh == tiles_m * tiles_n;
}
// places of one XCD's share of the order (the last of them may hold no tile)
__host__ __device__ inline int64_t xcd_places(int64_t tiles_m, int64_t tiles_n)
{
    const XcdParts g = xcd_parts(tiles_m, tiles_n);
    if (xcd_parts_exact(g, tiles_m, tiles_n)) return (int64_t)g.cw * g.rh;
    return (tiles_m * tiles_n + 7) / 8;
}
// tile rows and columns that an XCD's tiles lie in: lines of both operands that it reads (to within one)
inline int64_t xcd_lines(int64_t tiles_m, int64_t tiles_n)
{
    const XcdParts g = xcd_parts(tiles_m, tiles_n);
    if (xcd_parts_exact(g, tiles_m, tiles_n)) return g.cw + g.rh;
    const int64_t run = xcd_places(tiles_m, tiles_n), pw = (tiles_n + 7) / 8, down = (run + pw - 1) / pw;
    return (down < tiles_m ? down : tiles_m) + pw * (run > tiles_m * pw ? 2 : 1);
}
// workgroups to launch for a tile grid
inline int64_t xcd_grid(int64_t tiles_m, int64_t tiles_n) { return 8 * xcd_places(tiles_m, tiles_n); }
// tile of workgroup `block`; false when the workgroup is padding
__host__ __device__ inline bool xcd_tile(int block, int tiles_m, int tiles_n, int &tm, int &tn)
{
    const XcdParts g = xcd_parts(tiles_m, tiles_n);
    const int xcd = block & 7, slot = block >> 3;
    if (xcd_parts_exact(g, tiles_m, tiles_n)) {
        tn = (xcd % g.px) * g.cw + slot % g.cw;
        tm = (xcd / g.px) * g.rh + slot / g.cw;
        return tn < tiles_n && tm < tiles_m;
    }
    const int64_t tiles = (int64_t)tiles_m * tiles_n;
    const int64_t first = tiles * xcd / 8, next = tiles * (xcd + 1) / 8;   // XCD x: places [first, next)
    tm = 0;
    tn = 0;
    if (slot >= next - first) return false;
    const int64_t idx = first + slot;
    const int pw = (tiles_n + 7) / 8;                      // panel width, column tiles
    const int64_t per_panel = (int64_t)pw * tiles_m;
    const int full = tiles_n / pw;                         // panels of that width; one narrower may follow
    const int64_t p = idx / per_panel;
    if (p < full) {
        const int64_t rem = idx - p * per_panel;
        tm = (int)(rem / pw);
        tn = (int)(p * pw + rem % pw);
    } else {
        const int wl = tiles_n - full * pw;
        const int64_t rem = idx - (int64_t)full * per_panel;
        tm = (int)(rem / wl);
        tn = (int)(full * pw + rem % wl);
    }
    return true;
}

// Compute units of the current device (256 on MI355X), asked once per device.
inline int compute_units()
{
    static std::atomic<int> cached[16];   // zero-initialised; several host threads may ask at once
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 16) return 256;
    int n = cached[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
        cached[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

// Rows `ld` elements of `elem_bytes` apart collide in the memory system (same L2 sets, same
// channel) when their pitch is a multiple of 32 KiB of at least 64 KiB (measured on the vector-ALU
// kernels; the exported amulet_pitch_collides is this rule).
inline bool pitch_collides(int64_t ld, int elem_bytes)
{
    const int64_t pitch = ld * elem_bytes;
    return ld > 0 && pitch >= 65536 && pitch % 32768 == 0;
}

// A grid dimension holds at most 2^32 - 1 work-items (workgroups x threads), fewer than the
// 2^31 - 1 workgroups a tile order can have: a longer row of workgroups goes out as several
// launches, each told in `args.block_base` where in the row it starts (the kernels add it to
// blockIdx.x).  `launch(n)` enqueues n workgroups with the current args.  Returns the first
// launch error (later parts are then not sent).
// Test seam (amulet_debug_fail_launches): while positive, each launch attempt is refused on the
// host, counted down, and reported as hipErrorLaunchFailure; nothing reaches the device.
inline std::atomic<int> g_forced_launch_failures{0};
inline bool forced_launch_failure()
{
    int n = g_forced_launch_failures.load(std::memory_order_relaxed);
    while (n > 0)
        if (g_forced_launch_failures.compare_exchange_weak(n, n - 1, std::memory_order_relaxed)) return true;
    return false;
}

template <typename Args, typename Launch>
inline hipError_t launch_row_of_blocks(Args &args, int64_t blocks, int threads, Launch launch)
{
    const int64_t max_blocks = 0xFFFFFFFFLL / threads;
    for (int64_t base = 0; base < blocks; base += max_blocks) {
        if (forced_launch_failure()) return hipErrorLaunchFailure;
        args.block_base = (int)base;
        launch((unsigned)(blocks - base < max_blocks ? blocks - base : max_blocks));
        // a refused launch (bad grid, LDS not granted, a stream in error) ends the row: the error is
        // read, and so reset, exactly once, here, and handed up as the call's status
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Reproducible floating-point results (amulet_set_deterministic, or AMULET_DETERMINISTIC=1 in the
// environment when the library is first used): no launch splits K, so no tile is summed by
// several workgroups through float atomics, whose order of arrival differs from run to run.
inline std::atomic<int> g_deterministic{-1};   // -1: not asked yet, read the environment
inline bool k_split_allowed()
{
    int d = g_deterministic.load(std::memory_order_relaxed);
    if (d < 0) {
        const char *e = getenv("AMULET_DETERMINISTIC");
        d = (e && e[0] && e[0] != '0') ? 1 : 0;
        g_deterministic.store(d, std::memory_order_relaxed);
    }
    return d == 0;
}

// Tail split of the vector-ALU launchers.  The chip holds `round` workgroups at once (4 waves
// per SIMD) and workgroups take equally long, so a launch runs in rounds, and a last round with
// few workgroups leaves most of the chip idle for a whole K loop.  The tiles of the last round
// (or of the last two, or all of them when there is less than one round) are therefore launched
// once per k range, s ranges, when that shortens the launch: x rounds' worth of tiles then take
// ceil(x s) / s rounds.  They add their parts to R with hardware atomics and follow the whole
// tiles in the same grid, so they start as the last whole tiles finish.  Counted in real tiles:
// the blocks that pad the XCD parts to equal length come last in launch order and leave at once.
// A k range per workgroup for the streamed identity kernels: `chunk` (a multiple of the stage,
// `gran` k) made longer until the last range, K mod chunk, is empty or holds a whole stage too: the
// kernels multiply the k past a range's last whole stage from values fetched per lane, after
// streaming at least one stage.
inline int64_t chunk_with_a_whole_last_stage(int64_t K, int64_t chunk, int gran)
{
    while (chunk < K && K % chunk != 0 && K % chunk < gran) chunk += gran;
    return chunk;
}

struct TailSplit {
    int64_t base;     // first block (place in the tile order) of the split region
    int64_t blocks;   // places from there to the end of the padded order
    int splits;       // k ranges per tile
    int chunk;        // k per range, a multiple of k_align
    int64_t grid;     // blocks to launch: base + blocks * splits
};
inline bool choose_tail_split(int64_t real, int64_t wgs, int64_t round, int64_t K, int k_align, TailSplit &t)
{
    if (K < 512 || round <= 0 || real % round == 0 || !k_split_allowed()) return false;
    const int64_t tail = real % round;
    const int max_s = K / 256 < 8 ? (int)(K / 256) : 8;
    double best_cost = (double)((real + round - 1) / round);   // rounds of the plain launch
    int64_t best_region = 0;
    int best_s = 1;
    for (int two = 0; two < 2; ++two) {
        const int64_t region = tail + (two ? round : 0);
        if (region > real) break;
        for (int sp = 2; sp <= max_s; ++sp) {
            const int64_t parts = (region * sp + round - 1) / round;      // ceil(x s)
            // a k range costs a little more than its share of the K loop (set-up, atomics)
            const double cost = (double)((real - region) / round) + (double)parts / sp * (1.0 + 0.01 * sp);
            if (cost < best_cost - 0.03) { best_cost = cost; best_region = region; best_s = sp; }
        }
    }
    if (best_s <= 1) return false;
    const int64_t chunk = ((K + best_s - 1) / best_s + k_align - 1) / k_align * k_align;
    t.splits = (int)((K + chunk - 1) / chunk);
    t.chunk = (int)chunk;
    t.base = real - best_region;
    t.blocks = wgs - t.base;
    t.grid = t.base + t.blocks * t.splits;
    return t.splits > 1 && t.grid <= 0x7fffffffLL;
}

// K split of every tile for the matrix-core kernels when the tiles are few (at most four per
// compute unit).  One workgroup does not keep a compute unit's matrix cores busy: measured on
// the fp32 kernel, a unit with 1 / 2 / 3+ resident workgroups runs at 0.72 / 0.81 / 1.0 of its
// full rate (fp64, 8 waves per workgroup: 0.86 / 1.0).  With every tile launched once per k
// range, s ranges, the busiest unit of the busiest XCD (each XCD walks its own part of the tile
// grid, `part_tiles` places, on its own `units_per_xcd` units) gets n = ceil(part_tiles s /
// units_per_xcd) workgroups of 1/s of a tile each.  The estimate (n / s) / rate(n), plus 1 %
// per range for set-up and the atomic adds into R (mostly hidden behind other workgroups'
// K loops), is minimised over s <= 8 with at least 256 k per range.  Returns s (1: do not
// split).  Checked against sweeps of s = 1..8 at 144 ... 1024 tiles (fp32, K = 2048 ... 8192):
// the chosen s is within 4 % of the best one measured.
inline int choose_full_split(int64_t part_tiles, int64_t units_per_xcd, int64_t K, const double *rate,
                             int n_rates)
{
    if (!k_split_allowed()) return 1;
    const int max_s = K / 256 < 8 ? (int)(K / 256) : 8;
    int best_s = 1;
    double best = 0.0;
    for (int sp = 1; sp <= max_s; ++sp) {
        const int64_t n = (part_tiles * sp + units_per_xcd - 1) / units_per_xcd;
        const double r = rate[(n < n_rates ? n : n_rates) - 1];
        const double cost = (double)n / sp / r * (sp > 1 ? 1.0 + 0.01 * sp : 1.0);
        if (sp == 1 || cost < best - 0.02) { best = cost; best_s = sp; }
    }
    return best_s;
}

// K split of every tile for the streamed identity kernels (identity_mfma_dma.hip,
// identity_mfma_f64_dma.hip), whose workgroups hold `cap` to a compute unit and run at
// rate[c - 1] of the unit's full rate with c of them resident (fp32, measured: 0.92 / 0.985 /
// 1.0).  An XCD's `part_tiles` tiles, each launched once per k range, s ranges, are W =
// part_tiles s workgroups of K / s k each on S = units cap slots.  They run in W / S full rounds
// of cap K / s each, and the remainder either is the whole launch (spread evenly, c = ceil(W /
// units) per unit: c (K / s) / rate(c)) or follows full rounds, where the dispatcher refills the
// units that free first, so that a remainder piles up on a few units instead of spreading: after
// one full round it costs at least two workgroups' time, after two or more (the units have
// drifted apart by then) a whole round's (fp32, 1280 tiles: unsplit 123, in 3 ranges = five full
// rounds 142 TFLOP/s).  Costs are in units of one k of a tile at full rate (fp32 57.5 ns, fp64
// 115 ns).  A workgroup's set-up and write-back add `ovh_alone` (3 us: 50 / 30); a split launch
// adds its atomic adds, which the L2s retire at about 0.42 T per second for the whole chip:
// `atom_per_tile` (16384 adds: 0.68 / 0.34) x tiles x s (measured: 256 tiles in 2 ranges + 20 us,
// 64 tiles in 8 ranges + 23 us).  The s <= 1024 with at least 128 k per range and the lowest
// estimate is returned (1: do not split), the estimate in `lowest`.  Checked against sweeps of s = 1..8 at 64 ... 1536 tiles
// (K = 512 ... 4096): the chosen s is the best or within 3 % of the best one measured.
inline int choose_stream_split(int64_t part_tiles, int64_t units, int64_t K, int cap, const double *rate,
                               double ovh_alone = 50.0, double atom_per_tile = 0.68, double *lowest = nullptr)
{
    if (part_tiles <= 0 || units <= 0) return 1;
    const int max_s = !k_split_allowed() || K < 256 ? 1 : K / 128 < 1024 ? (int)(K / 128) : 1024;
    int best_s = 1;
    double best = 0.0;
    // every s up to 16, then a coarser ladder (problems of a tile or two with a very long K)
    for (int sp = 1; sp <= max_s; sp = sp < 16 ? sp + 1 : sp < 64 ? sp + 8 : sp < 256 ? sp + 32 : sp + 128) {
        const int64_t W = part_tiles * sp, S = units * cap;
        const int64_t q = W / S, r = W % S;
        const double work = (double)K / sp;
        double cost = (double)q * cap * work;
        if (r > 0) {
            const int64_t c = (r + units - 1) / units;
            double left = (double)c / rate[c - 1];
            if (q == 1 && left < 2.0) left = 2.0;
            if (q >= 2) left = (double)cap;
            cost += left * work;
        }
        cost += ovh_alone;
        if (sp > 1) cost += atom_per_tile * (double)(part_tiles * 8) * sp;
        if (sp == 1 || cost < best * 0.99) { best = cost; best_s = sp; }
    }
    if (lowest) *lowest = best;
    return best_s;
}

// K split of every tile in the wide vector-ALU kernels (mmlike_valu_impl.h, mmlike_valu_f64.hip): the k range of one
// workgroup, K where it is not split.  Tiles for at most half of the waves the chip holds at once (small
// M x N, e.g. an aggregation over a long K): as many workgroups per tile as still fit, at least 64 k each; each
// adds its part to R with hardware float atomics (the sum order is free, Sec. 4.1).  A SIMD with two waves
// runs a wave's work 20 % slower than one with four.
// fp32: as many parts as fill the chip to three waves per SIMD (four when the tiles alone fill one),
// of at least 64 k each and, from K = 512 on, of about 192: every part pays a first load of
// B, a pipeline fill and a tile of atomic adds, and parts of one tile that finish together
// queue on the same lines of R.  Measured over forced counts 1 ... 64, us, this rule / as many
// parts of 64 k as fit at four waves per SIMD (the earlier rule) / best forced: 512^3 40 / 55 / 40,
// 640^3 49 / 55 / 46, 768^3 63 / 73 / 61, 512^2 x 1024 58 / 86 / 54, 768^2 x 384 43 / 59 / 43,
// 128 x 4096 x 512 42 / 64 / 42, 256^2 x 4096 56 / 85 / 55, 512^2 x 2048 80 / 93 / 78,
// 1024^2 x 512 71 / 76 / 65; 256^3, 384^3, 896^3, 1024^3 unchanged (17, 24, 78, 97).
inline int64_t wide_k_range(int64_t waves, int64_t K)
{
    if (!k_split_allowed() || waves > 2048 || K < 128) return K;
    int64_t want = (waves >= 1024 ? 4096 : 3072) / waves;
    const int64_t most = K < 512 ? K / 64 : (K + 96) / 192;
    if (want > most) want = most;
    if (want < 1) want = 1;
    if (want > 1024) want = 1024;
    const int64_t range = ((K + want - 1) / want + 63) / 64 * 64;   // whole partial-sum periods
    return range < K ? range : K;
}
// us of a launch over tiles of 32 x 256 by workgroups of 8 waves, two to a compute unit, with the K split and the tail split
// they choose: a pair on a unit takes `pair` us per k, one alone `alone`, a last round of parts in between `between`.  Where
// neither split applies (one round and a bit, of a short K) the bit takes as long as the round.
// (`units`: the device's, as the launchers ask for it too)
inline double wide_launch_us(int64_t M, int64_t N, int64_t K, double pair, double alone, double between, int64_t units = compute_units())
{
    const int64_t tiles = ((M + 31) / 32) * ((N + 255) / 256), range = wide_k_range(tiles * 8, K), parts = (K + range - 1) / range;
    const int64_t round = 2 * units, W = (tiles + 7) / 8 * 8 * parts, rest = W % round;     // (an XCD's share is what its units have to take)
    const double us = 6.0 + 1.5 * (double)W / (double)units;
    if (parts > 1) return us + (double)range * (pair * (double)(W / round) + (rest == 0 ? 0.0 : rest <= units ? alone : between)) + (double)M * (double)N * (double)parts / 1.6e6;
    TailSplit t;
    if (!choose_tail_split(tiles, tiles, round, K, 64, t)) return us + (double)K * (pair * (double)(W / round) + (rest == 0 ? 0.0 : rest <= units ? alone : pair));
    const int64_t region = (tiles - t.base) * t.splits;
    return us + (double)K * pair * ((double)(t.base / round) + (double)((region + round - 1) / round) / t.splits * (1.0 + 0.01 * t.splits));
}
// fp64: as many parts as fill the chip, in ranges of whole stages
inline int64_t wide_k_range_f64(int64_t waves, int64_t K, int stage)
{
    if (!k_split_allowed() || waves > 2048 || K < 128) return K;
    int64_t want = 4096 / waves;
    if (want > K / 64) want = K / 64;
    if (want > 1024) want = 1024;
    const int64_t range = ((K + want - 1) / want + stage - 1) / stage * stage;
    return range < K ? range : K;
}

// Arguments of an fp32 task launch, already validated on the host.
struct MmlikeArgs {
    const float *A;
    const float *B;
    const float *thres;  // indexed as the launch's threshold form says; unused by the identity task
    const float *dis;    // dis[0..N), discount task only
    float *R;
    int64_t lda, ldb, ldr, ldt;   // ldt: row pitch of thres[i][j]
    int M, N, K;
    int transA, transB;  // operand stored transposed: a(i,k) = A[k*lda+i], b(k,j) = B[j*ldb+k]
    int vec;   // identity: 1 when B, R and their row pitches allow 16-byte vector accesses
    int vecA;  // 1 when A and its row pitch do
    int kchunk;  // k range of one workgroup when a launch splits K (set by the launcher)
    // Tail split: blocks from tail_base on are the launch's last `tail_blocks` places of the tile
    // order, each present tail_splits times, once per k range (tail_splits <= 1: no such blocks).
    int tail_base, tail_blocks, tail_splits;
    int block_base;   // added to blockIdx.x (launch_row_of_blocks)
    int force_splits; // > 1: every tile's K in this many parts (a k-axis point of the shape grid); 0: the launcher's rule
};

// Arguments of a mmlike_tile_kernel launch (mmlike_tile_impl.h).
template <typename T>
struct TileArgs {
    const T *A;
    const T *B;
    const T *thres;
    const T *dis;
    T *R;
    int64_t lda, ldb, ldr, ldt;
    int M, N, K;
    int kpart;       // k range of one of the gridDim.y parts of K
    int kgroup;      // of which each of a workgroup's groups of waves sums this many k
    int block_base;  // added to blockIdx.x (launch_row_of_blocks)
};

// A kernel's arguments (its first parameter) and its thread's number, opaque: for a second way of forming a tile after a first one
// that failed.  What both ways compute alike would else be held in registers through the first one's loop (BOOST's, 42 registers
// more than there are); so would the thread's number itself, but for its wave's, in a scalar register.
__device__ __forceinline__ unsigned own_wave() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }
template <typename Args>
__device__ __forceinline__ const __attribute__((address_space(4))) Args &opaque_args(unsigned wave, unsigned &tid)
{
    auto at = (const __attribute__((address_space(4))) Args *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(at), "+s"(wave));
    tid = wave * 64 + __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    return *at;
}

// How a tile-kernel launch covers its problem: tiles of 32 x 64 whose K four groups of two waves
// share, or of 16 x 64 shared by eight waves, and the k ranges that follow.
struct TilePlan {
    int wide;           // 1: 32 x 64, 0: 16 x 64
    int parts;          // workgroups per tile, each over kpart k (more than one: atomic adds into R)
    int kpart, kgroup;
    double us;          // the estimate it was chosen by
    // instead of a tile kernel, a kernel that shares its sums with the bf16 matrix cores: the identity task's
    // (identity_split.hip), rows of its tile; BOOST's (mmlike_boost_impl.h), 32; 0: neither
    int pieces;
    // fp64 tasks by mmlike_critical_f64_impl.h: rows of its tile, 0: not so; the rows from `rest` on
    // are the tile kernels', whose K has at most rest_parts parts
    int critical;
    int64_t rest, rest_parts;
};

// The plan with the lowest estimated time.  A compute unit holds two workgroups (16 waves) and is
// as fast per workgroup with two as with many; with one its SIMDs have two waves each and a
// workgroup takes 1.15 of the half share.  So W workgroups, counted with the padding of the tile
// order (an XCD's share is what its units have to take), are W / 512 pairs' time each `us_per_k`
// per k a group sums -- the time per k of one of two resident workgroups, which is the task's
// arithmetic -- and a last round of at most 256 is half a round and 15 % more.  Launch, first
// loads and write-back: 2.1 us and 1.3 per round; a tile in parts: 0.3 us and the atomic adds at
// 1.6 T (fp64 0.8 T) per second beside other workgroups' arithmetic.  Checked against the fastest of all plans at
// 240 drawn sizes (64 ... 8192 each way, both element types): 1.1 % behind it on average, 12 % at most (with any
// number of parts).
// (`alone`: the form that holds one workgroup to a unit, fp64 with thres[i][j]; nothing covers the loads of
// a tile's thresholds there, 3.5 us per round.)
// `max_parts`: the parts the wide kernel would add for the same call.  Every part is one more rounding of R, so a
// plan has no more of them: with ranges down to 32 k it had up to eight times as many (64 x 64 x 1024 in 32
// instead of 4: rms error 8.4e-8 against 4.9e-8 of the sums; now 4.5e-8), and split calls whose bits used to repeat.
// Unrestricted the estimate is 2.7 % lower on average over drawn sizes (fp64 1.7 %), 40 % at a few tiles.
template <typename T>
inline TilePlan choose_tile_plan(int64_t M, int64_t N, int64_t K, double us_per_k, int64_t max_parts, bool alone = false)
{
    constexpr int V = 16 / (int)sizeof(T);
    auto up = [](int64_t n, int64_t to) { return (n + to - 1) / to * to; };
    TilePlan best = {0, 0, 0, 0, 0.0, 0, 0, 0, 0};
    for (int wide = 0; wide < 2; ++wide) {
        const int rows = wide ? 32 : 16, groups = wide ? 4 : 8;
        const int64_t grid = xcd_grid((M + rows - 1) / rows, (N + 63) / 64);
        for (int64_t p = 1; p <= max_parts; p = p < 4 ? p + 1 : p % 3 ? p / 2 * 3 : p / 3 * 4) {   // 1 2 3 4 6 8 12 16 24 ...
            if (p > 1 && (K / p < 32 || grid * p > 12288)) break;
            const int64_t kpart = up((K + p - 1) / p, V), parts = (K + kpart - 1) / kpart;
            const int64_t kgroup = up((kpart + groups - 1) / groups, V);
            const int64_t W = grid * parts, rem = W % 512;
            const double rounds = alone ? 1.15 * (double)((W + 255) / 256) : 2.0 * (double)(W / 512) + (rem == 0 ? 0.0 : rem <= 256 ? 1.15 : 2.0);
            double us = rounds * (double)kgroup * us_per_k + 2.1 + (alone ? 3.5 : 1.3) * rounds;
            if (parts > 1) us += 0.3 + (double)M * (double)N * (double)parts / (sizeof(T) == 4 ? 1.6e6 : 0.8e6);
            if (best.parts == 0 || us < best.us) {
                best.wide = wide; best.parts = (int)parts; best.kpart = (int)kpart; best.kgroup = (int)kgroup; best.us = us;
            }
        }
    }
    return best;
}

// us of mmlike_critical_f64_impl.h's kernels: tiles of 64 x 128 (DISCOUNT, BOOST) or 128 x 128 (COUNT), two workgroups to a compute
// unit, a pair of which takes `pair` us per k and one alone `alone`, with `ends` per round for first loads and write-back; or DISCOUNT
// on 128 x 128, one.  A count transposed as it is added to R takes 0.036 more per tile: a lane's eight outputs, not the wave's, lie next
// to each other.  Within 3 to 4 % (rms) of 35 to 130 drawn calls per task of 2^26 to 2^35 products, all layouts.
inline double critical_f64_us(int task, int64_t M, int64_t N, int64_t K, int rows, int64_t units, bool transposed)
{
    struct Cost { double pair, alone, ends; };
    static const Cost cost[4] = {{}, {0.463, 0.262, 3.2}, {0.422, 0.233, 1.6}, {0.475, 0.286, 5.6}};
    const bool pairs = task != TASK_DISCOUNT || rows == 64;
    const int64_t W = xcd_grid((M + rows - 1) / rows, (N + 127) / 128), slots = pairs ? 2 * units : units, rest = W % slots;
    const double full = (double)(W / slots), all = full + (rest ? 1.0 : 0.0);
    if (!pairs) return 11.5 * all + 0.42 * (double)K * all;
    const Cost &c = cost[task];
    return 5.9 + c.ends * all + (transposed ? 0.036 * (double)W : 0.0) + (double)K * (c.pair * full + (rest == 0 ? 0.0 : rest <= units ? c.alone : c.pair));
}
// K of a count: 15/8 per product over its threshold, exact in fp32
constexpr int64_t C64_COUNT_K = (int64_t)1 << 20;
// The plan `tile` of the tile kernels, or that kernel for all rows, or for as many as fill whole rounds (the small tile: and half a
// round), and the tile kernels for the others: what is estimated lowest, by 3 % at least, by 8 % for DISCOUNT
// (whose estimate is up to a fifth low at a K of 64), with 1 us against it and 2 for a second launch: of 330 drawn calls two are then slower than by
// the tile kernels by more than 1.5 % (2 and 4.1); by 3 % alone 21 of 330 others were, the slowest by a sixth.  The other rows' K has no more parts than
// the tile kernels' plan for all of them.
inline void choose_critical_f64(int task, int64_t M, int64_t N, int64_t K, double us_per_k, int64_t units, bool transposed, TilePlan &tile)
{
    const int64_t parts = tile.parts, tiles_n = (N + 127) / 128;
    double best = (task == TASK_DISCOUNT ? 0.92 : 0.97) * tile.us;
    for (int rows = task == TASK_COUNT_GT ? 128 : 64; rows <= (task == TASK_BOOST ? 64 : 128); rows += 64) {
        auto take = [&](int64_t first) {
            if (first < M && M - first < 16) return;      // (fewer than the tile kernels take in some layouts)
            double us = critical_f64_us(task, first, N, K, rows, units, transposed) + 1.0;
            if (first < M) us += 2.0 + choose_tile_plan<double>(M - first, N, K, us_per_k, parts).us;
            if (us < best) { best = us; tile.critical = rows; tile.rest = first; tile.rest_parts = parts; }
        };
        take(M);
        // (a whole round, or with two workgroups to a unit half a one)
        const int64_t W = xcd_grid((M + rows - 1) / rows, tiles_n), step = units;
        for (int64_t full = W / step * step; full > 0 && full + 2 * step > W; full -= step) {
            const int64_t first = full / tiles_n * rows;        // (xcd_grid pads to eights, and so do these)
            if (first > 0 && first < M) take(first);
        }
    }
}

// From this estimate on the tile kernels count by rounding, in 0.88 of it (mmlike_tile_impl.h)
constexpr double COUNT_ROUNDING_TILE_US = 15.0;
template <typename T, int TASK>
hipError_t launch_mmlike_tile(int form, int trans, const TilePlan &plan, const TileArgs<T> &a, hipStream_t s);

// Tile shapes of the VALU kernels, laid out as the two-axis grid the greedy parameter search
// walks (paper Sec. 4.4-4.6).  Axis 0 is the k axis, the analogue of the paper's k_c (how much
// of K one unit of work covers): the depth BK of the B tile staged per barrier, and then how
// much of K one workgroup sums, K itself or K / 2, K / 4, K / 8 (the paper's sequence K,
// ceil(K / 2), ceil(K / 4), ...; the parts reach R through atomic adds).  Axis 1 is the
// workgroup's R tile from narrow to wide (the n_c analogue).
// shape id = k-axis index * VALU_TILES + tile.
//   k axis 0: BK 8    1: BK 16 (K split only where the launcher's own rule asks for it)
//          2, 3, 4: BK 16, every tile's K in 2, 4, 8 parts
//   tile 0: 4x4 per lane, 4 waves  -> 16 x 256      tile 1: 4x4, 8 waves -> 32 x 256
//   tile 2: 8x4 per lane, 8 waves  -> 64 x 256      tile 3: 4x8, 8 waves -> 32 x 512
// The identity task keeps the first two k-axis points (ids 0-7) and adds its matrix-core
// shapes (ids 8 to 12); the predicate tasks have all VALU_SHAPE_COUNT ids.
enum { VALU_DEPTHS = 2, VALU_KAXIS = 5, VALU_TILES = 4, VALU_SHAPE_COUNT = VALU_KAXIS * VALU_TILES };

struct ValuShapeDesc {
    int TM, NG, NW, BK;
    int splits;   // 0: the launcher's rule; else every tile's K in this many parts
    const char *name;
};
extern const ValuShapeDesc kValuShapes[VALU_SHAPE_COUNT];

// Arguments of an int8 join-count launch, already validated on the host.
struct CountArgs {
    const int8_t *A;
    const int8_t *B;
    int32_t *R;
    int64_t lda, ldb, ldr;
    int M, N, K;
    int Mload, Nload;  // rows of A / columns of B that exist in memory (>= M, N): a tile inside them loads without guards
    int64_t Mwhole;    // rows of the whole count, of which M may be a trial's: what a shape's kernels are chosen by
    int vecA, vecB;  // 1 when the operand and its row pitch allow 16-byte loads
    int vecR;        // 1 when R and its row pitch allow 16-byte accesses
    int kchunk;      // k range of one workgroup when a launch splits K (set by the launcher)
    int block_base;  // added to blockIdx.x (launch_row_of_blocks)
    // persistent streamed kernel, where in its first tile's k range a workgroup starts: the slots
    // of an XCD in pers_groups groups, pers_group_stages stages (of 64 k) apart, and XCD x another
    // (x % pers_xcds) * pers_xcd_span / pers_xcds sixteenths of the range
    int pers_groups, pers_group_stages, pers_xcds, pers_xcd_span;
    bool pers_named = false;   // by AMULET_I8_PHASES: the kernel that has phases runs, not the one that reads R during its K loop
    // 1: R = the counts instead of R += (amulet_count_i8_assign): a workgroup that owns its tile
    // alone stores its sums without reading R; a launch that splits K clears R first and adds
    int assign = 0;
};
// Arguments of a count_i8_tile_kernel launch (count_i8_tile.hip).
struct CountTileArgs {
    const int8_t *A;
    const int8_t *B;
    int32_t *R;
    int64_t lda, ldb, ldr;
    int M, N, K;
    int kpart;       // k range of one of the gridDim.y parts of K
    int kgroup;      // of which each of a workgroup's groups of waves sums this many k
    int block_base;  // added to blockIdx.x (launch_row_of_blocks)
    int assign;      // R = the counts instead of R +=
    int bypass;      // R is read and written around the caches (the two largest tiles)
};
enum { CT_256 = 0, CT_128x256 = 1, CT_128 = 2, CT_64 = 3, CT_192x256 = 4 };
struct CountTilePlan {
    int tile;               // CT_...
    int through_registers;  // rows at any byte address, staged through registers; else streamed HBM -> LDS
    int parts;              // workgroups per tile, each over kpart k (more than one: atomic adds into R)
    int kpart, kgroup;
    int alone;              // 128 x 256: at most one workgroup to a unit, and K for a ring of all of its LDS
    int deep;               // 128 x 128 and 64 x 64, streamed, at most one workgroup to a unit: stages of 128 k
    double us;              // the estimate it was chosen by
};

// The plan with the lowest estimated time.  Tiles: 256 x 256 (16 waves, one workgroup to a compute unit),
// 128 x 256 (8 waves, two to a unit, a deeper ring with one; streamed only), 128 x 128 (8 waves, two), 64 x 64 (two groups of 4 waves
// that share K, two).  A stage of 64 k (64 x 64: 128) takes `alone` us in a workgroup that has its unit for
// itself and `shared` per pair of workgroups on a unit, 1.4 to 1.7 times that through registers; the rest of a
// tile -- first loads, sums, write-back -- `rest_...`, a fifth less when R is not read.  W workgroups (with the
// tile order's padding) are whole rounds and a last one in which at most one workgroup per unit is alone.
// K over several workgroups (the two smaller tiles): 0.3 us and 1 T atomic adds per second beside other workgroups' arithmetic; to clear an R that is
// to be written 2 us and 1 per 4e5 counts, 4 at most up to 2.5e6 counts; above, whose adds find less of R in the L2s, no such bound,
// nor where operands stream and K is whole stages of 128 k, which make a whole K faster than the model has it (us, K whole / in parts: 470 x 512 x 3520
// 12.3 / 9.3, 64 x 1710 x 2368 10.7 / 8.7, 489 x 384 x 3244 11.0 / 8.8, 282 x 5756 x 13692 101 / 81, 408 x 4604 x 12703 78 / 66, 192 x 6592 x 3072 28 / 24; but 4677 x 960 x
// 15908 111 / 155, 3917 x 1468 x 6903 90 / 110, 6428 x 728 x 6272 100 / 115, 1024 x 1856 x 5120 23 / 29.  102 calls of 3e5 to 6e6 counts: 0.8 % behind the better of the two, 2.8 % without
// the bound, 5.7 % with it throughout, 11 % at 4 always; 120 of the last kind 1.14 times as fast as at 4 always, one of them 2 % slower.  300 of fewer: 1.13 times as fast as at 4 always, one in eight slower, by up to 17 %, nearly all of K below 2300.)
// Fitted to and checked against every tile and split at 210 drawn sizes (64 ... 8192 each way, all layouts and alignments): 1.4 % behind the fastest on average, 28 % at most.
// The two smaller tiles, streamed, with at most one workgroup to a unit: stages of 128 k (count_i8_tile.hip), where whole stages make a range no
// more than 2.5 % longer and a short last one, whose k are not pipelined, is one of at least eight: 320 x 1024 x 1152 5.2 us by 64 k, 6.0 by 128,
// 576 x 872 x 704 6.1 / 6.5.
// Of 64 x 64 tiles, not where both operands lie across k, whose loads gain nothing of a longer stage (A transposed, 1024 x 960 x 5100 18.4 by 64 k, 19.2
// by 128; 3000 x 300 x 1024 level), and from 384 k to a group of waves (1024 x 960, K = 512 4.0 % slower to 1 % faster by layout, 768 1 % slower to 5 % faster).
// Rows of an odd number of 64 bytes along k start in the middle of a cache line: 64 k of one are half a line, 128 k
// parts of two.  There the 64 x 64 tile gains only where both operands lie along k (of 1024 x 960 x 3520 A B 13.1 / 12.9, A B^T 12.7 / 11.7,
// A^T B^T level), with not many more rows than columns (3840 x 256 x 2240 10.3 / 10.6, x 3520 1 % slower, x 5056 3 % faster: this one size drew the line at 8 times), and the 128 x 128 tile with A along k
// (300 x 7000 x 3520 A B 1 % faster, A B^T 10 %, A^T B 6 % slower).  So for tight rows; where K is whole stages 128 k are ahead at any pitch (by 3 to 11 % on
// average at 64 bytes past a line), and of such K a pitch of whole lines gains 2 to 15 % that this rule leaves.
// With both operands across k and a short last stage, not where the rows of neither are multiples of 64 bytes apart, so that the pieces of every k-row share
// lines with their neighbours' (128 x 128 tile, by 64 k / by 128: 7000 x 300 x 5040 0.96 times, 300 x 7000 x 2500 0.98, 1500^2 x 5040 0.97; rows of A 64 bytes
// on 0.97, 1.01 and 1.03, of both 1.06, 1.06 and 1.09; 448 x 5012 x 5040 1.06, 2048^2 x 5040 1.11).
// (`trans`: 1 A transposed, 2 B.  `lines`: rows of an operand that lies across k are multiples of 64 bytes apart.  `rows192`: the 192 x 256 tile, 12 waves, may be taken: rows at any byte address, A not transposed, R through the caches.)
inline CountTilePlan choose_count_tile(int64_t M, int64_t N, int64_t K, bool through_registers, bool assign, bool rows192, int trans, bool lines)
{
    static const struct { int bm, bn, groups, resident; double alone, shared, rest_alone, rest_shared, registers; } tiles[5] = {
        {256, 256, 1, 1, 0.57, 0.0, 17.0, 0.0, 1.42}, {128, 256, 1, 2, 0.42, 0.60, 10.5, 16.0, 0.0},
        {128, 128, 1, 2, 0.206, 0.48, 4.8, 9.2, 1.52}, {64, 64, 2, 2, 0.19, 0.46, 2.8, 4.1, 1.67},
        {192, 256, 1, 1, 0.56, 0.0, 12.8, 0.0, 1.42}};
    const double counts = (double)M * (double)N, clear = counts > 2.5e6 || counts < 8.0e5 || (!through_registers && K % 128 == 0) ? 2.0 + counts / 4.0e5 : 4.0;
    auto up64 = [](int64_t n) { return (n + 63) / 64 * 64; };
    auto up128 = [](int64_t n) { return (n + 127) / 128 * 128; };
    auto deep_pays = [&](int tile, int64_t kgroup) {
        if (up128(kgroup) - kgroup > kgroup / 40 || (K % 128 != 0 && kgroup < 1024)) return false;
        if (tile == CT_64 && (trans == 1 || kgroup < 384)) return false;
        if (trans == 1 && K % 128 != 0 && !lines) return false;
        if (K % 128 == 64) return tile == CT_64 ? trans == 2 && M <= 8 * N : (trans & 1) == 0;
        return kgroup >= 256;
    };
    CountTilePlan best = {0, through_registers ? 1 : 0, 0, 0, 0, 0, 0, 0.0};
    for (int i = 0; i < 5; ++i) {
        const auto &t = tiles[i];
        if ((through_registers && t.registers == 0.0) || (i == CT_192x256 && !rows192)) continue;
        const int64_t grid = xcd_grid((M + t.bm - 1) / t.bm, (N + t.bn - 1) / t.bn), round = 256 * t.resident;
        for (int64_t p = 1; p <= 64; p = p < 4 ? p + 1 : p % 3 ? p / 2 * 3 : p / 3 * 4) {   // 1 2 3 4 6 8 12 16 24 ...
            if (p > 1 && (i < CT_128 || i == CT_192x256 || K / p < 192 || M * N * p > 16000000)) break;
            const int64_t kpart = up64((K + p - 1) / p), parts = (K + kpart - 1) / kpart;
            const int64_t kgroup = up64((kpart + t.groups - 1) / t.groups);
            const double stages = (double)(kgroup / 64) * (through_registers ? t.registers : 1.0), r = assign ? 0.77 : 1.0;
            const double alone = stages * t.alone + r * t.rest_alone, shared = t.resident > 1 ? stages * t.shared + r * t.rest_shared : alone;
            const int64_t W = grid * parts, rem = W % round;
            double us = 1.2 + (double)(W / round) * shared + (rem == 0 ? 0.0 : rem <= 256 ? alone : shared);
            if (parts > 1) us += 0.3 + (double)M * (double)N * (double)parts / 1.0e6 + (assign ? clear : 0.0);
            if (best.parts == 0 || us < best.us) {
                best.tile = i; best.parts = (int)parts; best.kpart = (int)kpart; best.kgroup = (int)kgroup; best.us = us;
                best.alone = i == CT_128x256 && W <= 256 && kgroup > 4 * 64 ? 1 : 0;
                best.deep = (i == CT_128 || i == CT_64) && !through_registers && W <= 256 && deep_pays(i, kgroup) ? 1 : 0;
            }
        }
    }
    if (best.deep) {                 // ranges of whole stages
        const int64_t kpart = up128(best.kpart);
        best.kpart = (int)kpart;
        best.parts = (int)((K + kpart - 1) / kpart);
        best.kgroup = (int)up128((kpart + tiles[best.tile].groups - 1) / tiles[best.tile].groups);
    }
    return best;
}
hipError_t launch_count_i8_tile(int trans, const CountTilePlan &plan, const CountTileArgs &a, hipStream_t s);
// shape 0: plain per-output loop; MFMA tiles 1: 128 x 128 (4 waves), 2: 256 x 256 (8 waves),
// 3: 128 x 256 (8 waves)
enum { COUNT_SHAPE_COUNT = 9 };
// Of what a shape id's launch came to, what the id does not say (amulet_recent_kernel).
struct CountRan {
    int workgroups = 0;     // of a persistent kernel, whose workgroups walk several tiles; 0: one tile to a workgroup
    int r_group = 0;        // count_i8_stream_kernel: values of R that a lane reads at a time during the K loop
    int r_bypass = 0;       // ... R written around the caches
};
hipError_t launch_count_i8(int shape, const CountArgs &a, hipStream_t s, CountRan &ran);
// R[0..M) x [0..N) = 0 (a fill kernel: usable under graph capture)
hipError_t launch_zero_r_i32(const CountArgs &a, hipStream_t s);
// direct HBM -> LDS kernels: tile (64 * wr) x 256, wr = 2 or 4
bool count_i8_dma_eligible(const CountArgs &a, int wr);
hipError_t launch_count_i8_dma(const CountArgs &a, int wr, hipStream_t s, bool persistent, CountRan &ran);
// ... persistent, a stream of stages across tiles whose R is read on the way (count_i8_stream.hip)
constexpr int COUNT_STREAM_LEAST_K = 1856;
bool count_i8_stream_eligible(const CountArgs &a);
bool count_i8_stream_in_step_loses(const CountArgs &a);
hipError_t launch_count_i8_stream(const CountArgs &a, hipStream_t s, CountRan &ran);

// Identity task on the fp32 matrix cores; its five shape ids follow its eight VALU shapes: a
// 128 x 128 tile (4 waves, register staged), a 256 x 256 tile (16 waves), the 128 x 128 tile
// with its operands streamed HBM -> LDS through a ring of 3 or 4 stages, and a streamed 64 x 64
// tile for problems of few tiles.
enum { IDENTITY_MFMA_SHAPE = VALU_DEPTHS * VALU_TILES, IDENTITY_MFMA_BIG_SHAPE = VALU_DEPTHS * VALU_TILES + 1,
       IDENTITY_MFMA_DMA3_SHAPE = VALU_DEPTHS * VALU_TILES + 2, IDENTITY_MFMA_DMA4_SHAPE = VALU_DEPTHS * VALU_TILES + 3,
       IDENTITY_MFMA_SMALL_SHAPE = VALU_DEPTHS * VALU_TILES + 4, IDENTITY_SHAPE_COUNT = VALU_DEPTHS * VALU_TILES + 5 };
// variant = shape id - IDENTITY_MFMA_SHAPE
hipError_t launch_identity_mfma(const MmlikeArgs &a, int variant, hipStream_t s);
// the streamed kernel (identity_mfma_dma.hip)
bool identity_dma_eligible(const MmlikeArgs &a);
// the identity task from bf16 pieces (identity_split.hip): tiles of tile_rows (128 or 256) x 128
hipError_t launch_identity_split(const MmlikeArgs &a, int tile_rows, hipStream_t s);
// ... for problems of few tiles, of 64 x 64 (identity_split_waves.hip)
hipError_t launch_identity_split_waves(const MmlikeArgs &a, hipStream_t s);
bool identity_split_runs(bool trans_a, bool trans_b, int64_t K, int64_t lda, int64_t ldb);
constexpr int ID_SMALL_STAGES = 4;   // ring depth of the streamed 64 x 64 tiles (fp32 and fp64)
hipError_t enqueue_identity_dma(const MmlikeArgs &a, int tile, int nstage, unsigned grid_x, unsigned grid_y, hipStream_t s);

// BOOST with its plain sum on the matrix cores (mmlike_boost_impl.h)
template <int TF>
hipError_t launch_mmlike_boost(const MmlikeArgs &a, hipStream_t s);

template <int TASK, int TF>
hipError_t launch_mmlike_valu_task(int shape, const MmlikeArgs &a, hipStream_t s);

// Arguments of an fp64 task launch (row-major operands), already validated on the host.
struct MmlikeArgsF64 {
    const double *A;
    const double *B;
    const double *thres;
    const double *dis;
    double *R;
    int64_t lda, ldb, ldr, ldt;
    int M, N, K;
    int vec;   // 1 when B, R and their row pitches allow 16-byte vector accesses
    int vecA;  // 1 when A and its row pitch do
    int transA, transB;  // operand stored transposed: a(i,k) = A[k*lda+i], b(k,j) = B[j*ldb+k]
    int vecBt; // transposed B: 1 when B and its row pitch allow 16-byte loads along k
    int kchunk;  // k range of one workgroup when a launch splits K (set by the launcher)
    int tail_base, tail_blocks, tail_splits;   // as in MmlikeArgs
    int block_base;   // added to blockIdx.x (launch_row_of_blocks)
};
// DISCOUNT and COUNT by critical values, BOOST by a clamp (mmlike_critical_f64_impl.h), tiles of `rows` x 128: DISCOUNT 64 or 128,
// COUNT 128, BOOST 64
template <int TASK, int TF>
hipError_t launch_mmlike_critical_f64(const MmlikeArgsF64 &a, int rows, hipStream_t s);
// predicate tasks: vector-ALU kernel; identity task: fp64 matrix-core kernel
// fp64 shapes of the predicate tasks: a small grid of the same two axes as the fp32 one
// (k axis: K whole, in 2, in 4 parts per tile; tile: 16 x 128 with 4 waves, 32 x 128 with 8).
enum { F64_KAXIS = 3, F64_TILES = 2, F64_SHAPE_COUNT = F64_KAXIS * F64_TILES };
hipError_t launch_mmlike_f64(int task, int form, int shape, const MmlikeArgsF64 &a, int &groups, hipStream_t s);
hipError_t launch_identity_mfma_f64(const MmlikeArgsF64 &a, int tile, int &groups, hipStream_t s);
// the streamed fp64 identity kernel (identity_mfma_f64_dma.hip)
bool identity_f64_dma_eligible(const MmlikeArgsF64 &a);
hipError_t enqueue_identity_f64_dma(const MmlikeArgsF64 &a, int tile, int groups, unsigned grid_x, unsigned grid_y, hipStream_t s);

// dst (cols x rows, pitch ld_dst) = transpose of src (rows x cols, pitch ld_src), bytes (pack.hip)
hipError_t launch_pack_pad_i8(int64_t rows, int64_t cols, const int8_t *src, int64_t ld_src, int8_t *dst,
                              int64_t ld_dst, int64_t rows_p, int64_t cols_p, hipStream_t s);
hipError_t launch_zero_block_i8(int8_t *dst, int64_t ld, int64_t row0, int64_t nrows, int64_t col0, int64_t ncols,
                                hipStream_t s);
hipError_t launch_transpose_i8(int64_t rows, int64_t cols, const int8_t *src, int64_t ld_src, int8_t *dst,
                               int64_t ld_dst, hipStream_t s);
// strided 2-D copy of rows x cols elements of 1, 4 or 8 bytes (pack.hip)
hipError_t launch_pack(int elem_bytes, int64_t rows, int64_t cols, const void *src, int64_t ld_src,
                       void *dst, int64_t ld_dst, hipStream_t s);

}  // namespace amulet
#endif
