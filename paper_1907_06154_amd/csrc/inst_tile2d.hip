// Small 2D grids, many sweeps a launch (ssam_kernel2d_tile.h): tile plan and launch.
#include <cmath>

#include "ssam_kernel2d_tile.h"

namespace ssam {
template <> const Tile2DKernel* tile2d_kernels<float, true>(int);
template <> const Tile2DKernel* tile2d_kernels<float, false>(int);
template <> const Tile2DKernel* tile2d_kernels<double, true>(int);
template <> const Tile2DKernel* tile2d_kernels<double, false>(int);

namespace {

// More than 64 KB of LDS per workgroup is asked for once per kernel and device.
hipError_t allow_lds(const void* kernel, int index)
{
    static std::atomic<unsigned long long> done[kTile2DIndexes];   // by instance: bit per device
    int dev = 0;
    if (hipError_t e = hipGetDevice(&dev)) return e;
    const unsigned long long bit = 1ull << (dev & 63);
    if (done[index].load(std::memory_order_relaxed) & bit) return hipSuccess;
    const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 160 << 10);
    if (e == hipSuccess) done[index].fetch_or(bit, std::memory_order_relaxed);
    return e;
}

int tiles_along(int extent, int tile, int step) { return ceil_div(extent - tile, step) + 1; }

constexpr int kTileDepth = 32;       // sweeps of a launch, at most: beyond, the halo is the tile
constexpr int kTileHorizon = 64;     // with more sweeps to do, the depth of least time per sweep, whatever their number

// The plan of least expected time for the sweeps that remain.  The expectation is fitted to 3400 measured launches (256^2 ..
// 4096^2, both types, stars of radius 1, 2, 4, 6, boxes of radius 1, 2, 4, one to sixteen sweeps; 12 % off in the quadratic mean, and
// the plan it picks 1.5 % slower than the best in the mean, 22 % at worst).  A launch costs 3.4 us and never less than 5; a sweep
// of a compute unit's blocks their instructions, four cycles each, or 0.16 us of latency, whichever dominates; a block's loads and
// stores 0.033 us per wave and four-byte column.
// Depths are tried, not numbers of launches, so that planning takes no longer the more sweeps remain (1023x1025 fp32 star r1, ten
// thousand left: 716 us by launches, 6 by depths; 5000 sweeps 18.6 ms and 5.1, of which the launches take 5).
Tile2DPlan plan_tiles(int W, int H, int R, bool star, int elem, const Tile2DKernel* list, int remaining, int deepest)
{
    Tile2DPlan best;
    double best_us = 1e30;
    const int taps = star ? 4 * R + 1 : (2 * R + 1) * (2 * R + 1), pub = 2 * R < kTileRows ? 2 * R : kTileRows;
    for (const Tile2DKernel* k = list; k->kernel; ++k) {
        const int TW = kWave * k->V;
        if (W < TW) continue;
        const double work = kTileRows * k->V * taps + 0.7 * (star ? kTileRows : kTileRows + 2 * R) * 2 * R * (elem / 4) + 4;
        for (int waves = kTileWaves; waves >= 4; waves -= 4) {
            const int TH = waves * kTileRows;
            if (H < TH) continue;
            const int fit = min(2 * kTileWaves / waves, (160 << 10) / (2 * waves * pub * kWave * k->V * elem));   // blocks a unit holds at once
            double last = 1e30;
            // an axis that one tile covers has no halo (16 rows, zero padding, us: fp32 star r3, three sweeps, 11 -> 5, fp64 star r4,
            // seventeen or eighteen, 64 -> 17; blocks of 12 and 16 waves are better off with several tiles, up to 1.3 with 48 rows)
            const bool all_x = W == TW, all_y = H == TH && waves <= 8;
            const int most_x = all_x ? kTileDepth : (TW - 1) / (2 * R), most_y = all_y ? kTileDepth : (TH - 1) / (2 * R);
            for (int depth = min(min(deepest, kTileDepth), min(most_x, most_y)); depth > 0; --depth) {
                const int launches = ceil_div(remaining, depth), sweeps = remaining > kTileHorizon ? depth : ceil_div(remaining, launches);
                if (sweeps < depth) continue;                     // as many launches as with that depth
                const int step_x = all_x ? TW : TW - 2 * sweeps * R, step_y = all_y ? TH : TH - 2 * sweeps * R;
                const int tx = tiles_along(W, TW, step_x), ty = tiles_along(H, TH, step_y);
                if ((long)tx * ty > 1L << 20) continue;
                const int share = ceil_div(tx * ty, kCUs);        // blocks of the busiest unit
                const double issue = share * waves * work / 2200, latency = 0.16 * ceil_div(share, fit < 1 ? 1 : fit);
                const double one = 3.4 + sweeps * std::sqrt(issue * issue + latency * latency) + 0.033 * share * waves * k->V * (elem / 4);
                const double us = (one > 5.0 ? one : 5.0) * (remaining > kTileHorizon ? 1.0 / sweeps : launches);
                if (us < best_us) {
                    best_us = us;
                    best.us = us / (remaining > kTileHorizon ? 1 : remaining);
                    best.k = k;
                    best.waves = waves;
                    best.sweeps = sweeps;
                    best.step_x = step_x;
                    best.step_y = step_y;
                    best.tiles_x = tx;
                    best.tiles_y = ty;
                }
                if (us > 1.5 * last) break;
                if (us < last) last = us;
            }
        }
    }
    return best;
}

// The largest grid, in points, that the remaining sweeps run on here instead of in the marching kernels (several sweeps a launch, or
// one).  The halo costs more the wider the stencil, and the marching kernels' latency less the larger the grid; and they are at their
// best with as many sweeps as one launch of theirs does, on rows of whole 16-byte pieces.  Both were timed on 16000 random grids of 64 ..
// 8192 rows and columns, 2 .. 24 sweeps, and on 20000 of such rows; the lines are those with the least time lost against the better of
// both, 0 .. 1.3 % in the mean.  Ratio of the times, this kernel to those (middle of a range of sizes; single grids are up to a fifth off,
// as tiles fit them), first rows of any length:
//   radius 1, five sweeps, seven and more: 0.23 .. 0.7 at every size; six 0.3 .. 0.96 but for the fp64 star with zero padding, 0.56 .. 0.88
//     up to 3 million points and 0.96 .. 1.1 beyond.
//   radius 1, two: 0.42 .. 0.85 up to 4 million points, where the others begin to pair them; beyond fp64 star 1.0 .. 1.15, fp64 box 1.03 ..
//     1.08 with zero padding and 0.98 .. 1.05 under the clamp rule, fp32 star 0.84 .. 1.3, fp32 box 0.81 .. 1.1.
//   radius 1, three: fp32 with zero padding 0.81 .. 1.0 up to 3.7 million, 0.95 .. 1.11 beyond, clamp star 0.76 .. 0.98 up to 5, 1.0 beyond,
//     box 0.69 .. 0.99; fp64 with zero padding 0.92 .. 1.0 up to 1.1 million, 1.05 .. 1.33 beyond, clamp 0.74 .. 1.0 up to 2.5, 1.0 .. 1.1 beyond.
//   radius 1, four, fp64 with zero padding: star 0.72 .. 0.99 up to 1.5 million, box 0.65 .. 0.94 up to 2; 1.02 .. 1.3 beyond; else 0.46 .. 1.0.
//   fp32: box r2 0.3 .. 0.78 up to 3 million, star r2 0.28 .. 0.8 up to two, star r3 0.2 .. 1.0 up to four, star r4 .. r6 0.18 .. 0.8 up to
//     two.  Boxes from radius 3 on: single sweeps on the split kernel, with less error.
//   fp64: box r2 0.36 .. 0.8 and star r2 0.35 .. 0.95 up to 1.1 million, star r4 and r5 0.28 .. 0.89, star r6 0.31 .. 1.2; star r3 0.4 .. 1.0
//     up to 3 million, but with zero padding three sweeps, six, nine .. 0.6 .. 1.1 up to two and 1.1 .. 1.29 beyond, and three under the
//     clamp rule 1.1 from 2.5 on; box r3, which has single sweeps only, see single_box3_us; box r4 0.61 .. 0.99 up to 160000 (five sweeps
//     under the clamp rule 1.1).
// On rows of whole pieces (the range, and its middle, beyond the line):
//   two sweeps: from 4.2 million on fp32 with zero padding star 1.12 .. 1.52 (1.22), box 1.01 .. 1.61 (1.20), clamp star 0.90 .. 1.26 (0.98),
//     fp64 box clamp 0.90 .. 1.27 (1.04); from 5.1 on fp32 box clamp 0.90 .. 1.32 (1.06).
//   three: fp32 with zero padding star from 0.3 million on 0.78 .. 1.44 (1.02), box from 2.5 on 0.84 .. 1.31 (1.11), clamp star from 4.3 on
//     0.88 .. 1.27 (1.05), box from 4.6 on 0.78 .. 1.14 (1.02); fp64 clamp from 2.2 on 0.96 .. 1.21 (1.04).
//   four: fp32 with zero padding star from 3.4 million on 0.91 .. 1.30 (1.12), box from 4.7 on 0.75 .. 1.20 (1.02).
//   six and eight, fp64 box with zero padding: from 10 million on 1.02 .. 1.10 (1.05), from 8 on 0.95 .. 1.31 (1.03).
//   fp64 star r3 with zero padding, three, six, nine ..: from 1.4 million on 1.0 .. 1.12 (1.09); star r6 from one million on 0.7 .. 1.18 (1.08).
long most_points(bool f32, bool star, int R, bool zero, bool pieces, int remaining)
{
    constexpr long M = 1000000, most = 1L << 24, pairs = (1L << 22) - 1;      // pairs: where the marching kernels begin to pair sweeps
    if (pieces && R == 1) {
        if (remaining == 2) return f32 && !star && !zero ? 5100000 : pairs;
        if (remaining == 3 && f32) return zero ? (star ? 300000 : 2500000) : star ? 4300000 : 4600000;
        if (remaining == 3 && !zero) return 2200000;
        if (remaining == 4 && f32 && zero) return star ? 3400000 : 4700000;
        if (!f32 && zero && !star && (remaining == 6 || remaining == 8)) return remaining == 6 ? 10 * M : 8 * M;
    }
    if (R == 1 && remaining == 2) return star ? (f32 ? 5 * M : pairs) : !f32 && zero ? pairs : most;
    if (R == 1 && remaining == 3) return f32 ? (zero ? 3700000 : star ? 5 * M : most) : zero ? 1100000 : 2500000;
    if (R == 1 && remaining == 4 && !f32 && zero) return star ? 1500000 : 2 * M;
    if (R == 1 && remaining == 6 && !f32 && zero && star) return 3 * M;
    if (R == 1) return most;
    if (f32) return star && R == 3 ? 1L << 22 : star ? 2 * M : 3200000;
    if (star && R == 3) return zero && remaining % 3 == 0 ? (pieces ? 1400000 : 2 * M) : remaining == 3 ? 2500000 : 3100000;
    if (star) return R == 6 && pieces ? M : 1100000;
    return R == 2 ? 1100000 : R == 3 ? 1L << 22 : 160000;
}

// The expected time of a sweep here up to which the fp64 box of radius 3 stays, whose other kernel does single sweeps: what those take,
// less what the expectation of a plan falls short of the time by (0.16 in the mean).  Their time goes up in steps, as waves of 120 columns
// and 8, 16 or 24 rows fill the chip: 6.0 .. 7.5 us a sweep up to 1024 waves of 8 rows (rows of odd length a tenth more), 8.7 .. 10 up to
// 2048, 12.5 .. 20 with 16 rows, 23 with 24.  On 2900 grids of up to 4.2 million points 0.1 % of the time is lost against the better of
// both; without this 0.6 %, and up to 1.30 of the time on grids of 1.4 to 2 million points (5810x289, nine sweeps, 81 us and 105).
double single_box3_us(int W, int H)
{
    const long waves = (long)ceil_div(W, 120) * ceil_div(H, 8);
    return waves <= 1024 ? 1e30 : waves <= 2048 ? 8.2 : waves <= 4096 ? 15.5 : 1e30;
}

// Whether a plan of less than all that remains a launch is kept.  Grids of less than two blocks' rows (17 .. 31) have tiles of 16
// rows that are mostly halo, and with zero padding the marching kernels do three sweeps of stars up to radius 4, or four up to
// radius 2, in one launch: ratio of the times, this kernel to those, star r3 three sweeps 1.13 .. 1.52 (six and more at most 1.0),
// fp64 star r4 three 1.3 .. 1.44, six and nine 1.1 .. 1.2 (others at most 0.99; fp32 three 1.2, others 0.46 .. 0.99, and a rest of
// three costs more there), r2 four 1.26; under the clamp rule 0.8 and less.  A sweep a launch of the box of radius 4 is 1.0 ..
// 1.1 of its own kernel's; of that of radius 3, which happens from 3 million points on, 0.70 .. 1.17, 0.92 in the middle; of the stars
// of radius 5 and 6 0.31 .. 0.98.
bool keeps_plan(int sweeps, bool f32, bool star, int R, int H, bool zero, int remaining)
{
    if (!star) return sweeps > 1 || R != 4;
    if (!zero || H >= 2 * 4 * kTileRows || sweeps >= remaining) return true;
    return !(R == 2 ? remaining == 4 : R == 3 ? remaining == 3 : R == 4 && !f32 && remaining % 3 == 0);
}

template <typename T, class Mask>
hipError_t launch_tile(const Problem2D& pr, const Tile2DPlan& plan, size_t lds)
{
    ArgsTile2D<T, Mask::kNW> a;
    a.in = static_cast<const T*>(pr.in);
    a.out = static_cast<T*>(pr.out);
    a.W = pr.W;
    a.H = pr.H;
    a.boundary = pr.boundary;
    a.sweeps = plan.sweeps;
    a.tiles_x = plan.tiles_x;
    a.step_x = plan.step_x;
    a.step_y = plan.step_y;
    const T* w = static_cast<const T*>(pr.w);
    for (int n = 0; n < Mask::kN; ++n)
        for (int m = 0; m < Mask::kM; ++m)
            if (Mask::tap(n, m)) a.w[Mask::widx(n, m)] = w[n * Mask::kM + m];
    void* args[] = {&a};
    return hipLaunchKernel(plan.k->kernel, dim3(plan.tiles_x * plan.tiles_y), dim3(plan.waves * kWave), args, lds, pr.stream);
}

template <typename T, int BUDGET>
hipError_t launch_tile(const Problem2D& pr, const Tile2DPlan& plan, size_t lds)
{
    switch (pr.ax) {
#define SSAM_R(R) case R: return launch_tile<T, TapMask<2 * R + 1, 2 * R + 1, R, R, BUDGET>>(pr, plan, lds);
        SSAM_R(1) SSAM_R(2) SSAM_R(3) SSAM_R(4) SSAM_R(5) SSAM_R(6)
#undef SSAM_R
    }
    return hipErrorNotSupported;
}

}  // namespace

int launch2d_tile(const Problem2D& pr, bool star, int remaining, int deepest, Tile2DPlan* kept, Geometry* geo, bool dry_run, hipError_t* err)
{
    const bool f32 = pr.dtype == SSAM_F32;
    if (pr.M != pr.N || pr.ax != pr.ay || pr.M != 2 * pr.ax + 1 || remaining < 2) return 0;
    const Tile2DKernel* list = star ? (f32 ? tile2d_kernels<float, true>(pr.ax) : tile2d_kernels<double, true>(pr.ax))
                                    : (f32 ? tile2d_kernels<float, false>(pr.ax) : tile2d_kernels<double, false>(pr.ax));
    const int elem = f32 ? 4 : 8, R = pr.ax;
    const bool zero = pr.boundary == SSAM_BOUNDARY_ZERO;
    if (!list || (long)pr.W * pr.H > most_points(f32, star, R, zero, pr.W % (16 / elem) == 0, remaining)) return 0;
    const bool far = remaining > kTileHorizon;
    const Tile2DPlan plan = far && kept && kept->k && kept->sweeps <= deepest ? *kept : plan_tiles(pr.W, pr.H, R, star, elem, list, remaining, deepest);
    if (!plan.k || !keeps_plan(plan.sweeps, f32, star, R, pr.H, zero, remaining)) return 0;
    if (!f32 && !star && R == 3 && plan.us > single_box3_us(pr.W, pr.H)) return 0;
    if (far && kept) *kept = plan;
    const size_t row = (size_t)kWave * plan.k->V * elem;
    const size_t lds = (2 * plan.waves * (size_t)(2 * R < kTileRows ? 2 * R : kTileRows) + 1) * row;
    if (geo) {
        Geometry g;
        g.V = plan.k->V;
        g.P = kTileRows;
        g.valid_lanes = kWave;
        g.strips_x = plan.tiles_x;
        g.tiles_y = plan.tiles_y;
        g.rows_per_wave = kTileRows;
        g.tiles = (long)plan.tiles_x * plan.tiles_y * plan.waves;
        g.blocks = plan.tiles_x * plan.tiles_y;
        g.lds = (int)lds;
        *geo = g;
    }
    *err = hipSuccess;
    if (dry_run) return plan.sweeps;
    *err = allow_lds(plan.k->kernel, plan.k->index);
    if (*err == hipSuccess)
        *err = star ? (f32 ? launch_tile<float, 1>(pr, plan, lds) : launch_tile<double, 1>(pr, plan, lds))
                    : (f32 ? launch_tile<float, 2>(pr, plan, lds) : launch_tile<double, 2>(pr, plan, lds));
    if (*err != hipSuccess) (void)hipGetLastError();     // returned here: not left for the next call to find
    return plan.sweeps;
}

}  // namespace ssam
