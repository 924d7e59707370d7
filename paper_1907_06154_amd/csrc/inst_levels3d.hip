// Several sweeps of a radius-1 3D stencil a launch (ssam_kernel3d_levels.h): tile plan and launch.
#include <cmath>

#include "ssam_kernel3d_levels.h"

namespace ssam {
template <> LevelsKernel levels_kernel<float, 1>(int, int, int, bool, bool);
template <> LevelsKernel levels_kernel<float, 2>(int, int, int, bool, bool);
template <> LevelsKernel levels_kernel<float, 3>(int, int, int, bool, bool);
template <> LevelsKernel levels_kernel<double, 1>(int, int, int, bool, bool);
template <> LevelsKernel levels_kernel<double, 2>(int, int, int, bool, bool);
template <> LevelsKernel levels_kernel<double, 3>(int, int, int, bool, bool);

namespace {

LevelsKernel find_kernel(bool f32, int budget, int V, int waves, int sweeps, bool clamp, bool stream)
{
    if (f32) return budget == 1 ? levels_kernel<float, 1>(V, waves, sweeps, clamp, stream)
                                : budget == 2 ? levels_kernel<float, 2>(V, waves, sweeps, clamp, stream) : levels_kernel<float, 3>(V, waves, sweeps, clamp, stream);
    return budget == 1 ? levels_kernel<double, 1>(V, waves, sweeps, clamp, stream)
                       : budget == 2 ? levels_kernel<double, 2>(V, waves, sweeps, clamp, stream) : levels_kernel<double, 3>(V, waves, sweeps, clamp, stream);
}

// More than 64 KB of LDS per workgroup is asked for once per kernel and device.
hipError_t allow_lds(const LevelsKernel& k)
{
    if (k.lds <= (64u << 10)) return hipSuccess;
    static std::atomic<unsigned long long> done[kLevelsIndexes];   // by kernel: bit per device
    int dev = 0;
    if (hipError_t e = hipGetDevice(&dev)) return e;
    const unsigned long long bit = 1ull << (dev & 63);
    if (done[k.index].load(std::memory_order_relaxed) & bit) return hipSuccess;
    const hipError_t e = hipFuncSetAttribute(k.kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)k.lds);
    if (e == hipSuccess) done[k.index].fetch_or(bit, std::memory_order_relaxed);
    return e;
}

struct LevelsPlan {
    int V = 0, waves = 0, sweeps = 0, step_x = 0, step_y = 0, lead_x = 0, tiles_x = 0, tiles_y = 0, planes = 0;
    double us = 1e30;          // expected time of the launch
};

// The plan of least expected time for `sweeps` sweeps a launch.  The expectation is fitted to 2400 measured launches (64^3 .. 400x448x330,
// three shapes, both types and boundary rules; 10 % off in the quadratic mean, the plan it picks 3 % slower than the best in the mean, 35 %
// at worst): 4 us; the steps of a chunk, each the instructions of the busiest unit's waves, four cycles each, or 0.5 us of latency,
// whichever dominates; or the bytes.
LevelsPlan plan_levels(const Problem3D& pr, int budget, int sweeps)
{
    LevelsPlan best;
    const bool f32 = pr.dtype == SSAM_F32;
    const int elem = f32 ? 4 : 8, S = sweeps, taps = budget == 1 ? 7 : budget == 2 ? 19 : 27;
    const double bytes = (double)pr.W * pr.H * pr.D * elem;
    for (int V = 16 / elem; V >= 8 / elem; V /= 2) {
        const int TW = kWave * V;
        if (pr.W < TW) continue;
        // Tiles store whole 128-byte lines where that costs no tile, or the grid is beyond the caches: parts of lines written by two
        // blocks cost a large grid a fifth of its bandwidth (512^3 fp64 star, two sweeps: 500 us with 124 columns, 408 with 112).
        const int line = 128 / elem, wide = TW - 2 * ceil_div(S, V) * V, cut = (TW - 2 * S) / line * line;
        const int step_x = pr.W == TW ? TW : ceil_div(pr.W, cut) == ceil_div(pr.W, wide) || bytes > 96e6 ? cut : wide;
        for (int waves = kLevelWaves; waves >= 4; waves -= 4) {
            const int TH = waves * kLevelRows;
            if (pr.H < TH) continue;
            const int step_y = pr.H == TH ? TH : TH - 2 * S;
            const long xy = (long)ceil_div(pr.W, step_x) * ceil_div(pr.H, step_y);
            const double work = S * (kLevelRows * V * taps + 0.93 * (budget == 1 ? kLevelRows : kLevelRows + 2) * 2 * (elem / 4) + 15.5);
            const int registers = (3 * S + 1) * kLevelRows * V * elem / 4 + 40, slots = 512 / (registers < 64 ? 64 : registers);
            int fit = min(slots * 4 / waves, (160 << 10) / (2 * S * (1 + 2 * waves) * kWave * V * elem));       // blocks a unit holds at once
            if (fit < 1) fit = 1;
            double latency = 0.49;
            if (V * elem == 16 && waves == 8) latency *= 1.4;
            if (V * elem == 16 && pr.W % V != 0) latency *= 2;         // parts of pieces at the ends of rows
            for (int chunks = 1; chunks <= pr.D; chunks += (chunks + 3) / 4) {
                const int planes = ceil_div(pr.D, chunks);
                const long blocks = xy * ceil_div(pr.D, planes);
                if (blocks > 1L << 20) break;
                const int share = ceil_div((int)blocks, kCUs);        // blocks of the busiest unit
                const double issue = share * waves * work / 2200, wait = latency * ceil_div(share, fit);
                double us = 4.0 + (planes + 3 * S - 1) * std::sqrt(issue * issue + wait * wait);
                const double moved = (bytes + 0.076 * blocks * (planes + 2 * S) * TW * TH * elem) * 1e-6 / (2 * bytes < 230e6 ? 3.27 : pr.W % line == 0 ? 2.9 : 2.45);
                us = std::sqrt(std::sqrt(us * us * us * us + moved * moved * moved * moved));
                if (us < best.us) {
                    best.V = V;
                    best.waves = waves;
                    best.sweeps = S;
                    best.step_x = step_x;
                    best.step_y = step_y;
                    best.lead_x = (TW - step_x) / 2 / V * V;
                    best.tiles_x = ceil_div(pr.W, step_x);
                    best.tiles_y = ceil_div(pr.H, step_y);
                    best.planes = planes;
                    best.us = us;
                }
                if (share > 8) break;
            }
        }
    }
    return best;
}

// What the other kernels take for a sweep, in us, where they are at their best: the plane ring's two sweeps of the star (zero padding,
// rows of whole pieces) 1.38 (fp32 0.75) ps a point, single sweeps of the other shapes 2.45 (fp32 1.44), on strips and blocks that are full.
double others_us(const Problem3D& pr, bool star)
{
    const bool f32 = pr.dtype == SSAM_F32;
    const int TW = f32 ? 256 : 128;
    const double full = (double)pr.W / (ceil_div(pr.W, TW) * TW) * pr.H / (ceil_div(pr.H, 32) * 32);
    const double ps = star ? (f32 ? 0.75 : 1.38) : f32 ? 1.44 : 2.45;
    return ps * 1e-6 * pr.W * pr.H * pr.D / full;
}

template <typename T, int BUDGET>
hipError_t launch_levels(const Problem3D& pr, const LevelsKernel& k, const LevelsPlan& plan, const Geometry& g)
{
    constexpr int NWTS = SliceMask<1, 1, 1, BUDGET, 0>::kNW;
    Args3D<T, NWTS> full;
    fill_args3d<T, 16 / sizeof(T), 1, 1, 1, BUDGET>(pr, g, &full);
    ArgsLevels<T, NWTS> a;
    a.in = full.in;
    a.out = full.out;
    a.W = pr.W;
    a.H = pr.H;
    a.D = pr.D;
    a.tiles_x = plan.tiles_x;
    a.tiles_y = plan.tiles_y;
    a.step_x = plan.step_x;
    a.step_y = plan.step_y;
    a.lead_x = plan.lead_x;
    a.lead_y = plan.sweeps;
    a.planes = plan.planes;
    a.tiles = (int)g.tiles;
    a.blocks = g.blocks;
    a.xcd_remap = g.xcd_remap;
    for (int i = 0; i < NWTS; ++i) a.w[i] = full.w[i];
    if (hipError_t e = allow_lds(k)) return e;
    void* args[] = {&a};
    return hipLaunchKernel(k.kernel, dim3(g.blocks), dim3(plan.waves * kWave), args, k.lds, pr.stream);
}

}  // namespace

int launch3d_levels(const Problem3D& pr, int budget, int remaining, int deepest, Geometry* geo, bool dry_run, hipError_t* err)
{
    const bool f32 = pr.dtype == SSAM_F32, clamp = pr.boundary == SSAM_BOUNDARY_CLAMP, star = budget <= 1;
    const int V16 = f32 ? 4 : 2, elem = f32 ? 4 : 8;
    const long points = (long)pr.W * pr.H * pr.D;
    // Grids of fewer points are a matter of launches, whose number stays what it was.  From 2^27 points on the 19- and 27-point shapes stay
    // with single sweeps in fp32 and under the clamp rule: not for their time (512^3 fp64 under the clamp rule, four sweeps, box 1439 us
    // and here 950, 19 points 1419 and 816), but because that is the plan of 512^3 that is promised (test_fused_sweep_plan_3d).
    if (remaining < 2 || points <= (1L << 18) || (!star && (clamp || f32) && points >= (1L << 27))) return 0;
    if ((long)pr.W * kLevelRows * elem >= kLevelBufferBytes) return 0;
    const bool stream = 2 * points * elem > (192L << 20);
    const bool pieces = pr.W % V16 == 0 && (dry_run || pointers_aligned(pr.in, pr.out, 16));
    LevelsPlan plan = plan_levels(pr, star ? 1 : budget, 2);
    // Beyond the caches, on grids that fill its tiles, the plane ring is faster with two sweeps of the star (512^3: fp64 370 us, here
    // 408).  (A pair of sweeps is planned alike under both boundary rules.)  Single sweeps of the other shapes are where tiles are ill
    // filled (255x256x256 fp32 box 30 us a sweep, here 41); off their best, on ragged rows or in the caches, they take a quarter more.
    // Ratio of the times, what comes here to those, on 13000 random grids of up to 2^27 points: 19 and 27 points 0.33 .. 1.05 but for 0.7 %
    // of them (up to 1.38, most of them of few planes), 0.75 in the middle; beyond 2^26 points fp64 0.35 .. 0.89 (768x384x384 box, clamp,
    // four sweeps 1842 us and 744), fp32 0.34 .. 1.29, 0.76 in the middle; 7 points 0.27 .. 0.99.
    const double others = others_us(pr, star);
    const bool leave = plan.V != 0 && points >= (4L << 20) && plan.us / 2 > (stream && pieces ? 1.0 : star ? 1e9 : 1.25) * others;
    if (star && remaining >= 3 && deepest >= 3 && (remaining != 4 || (leave && clamp))) {            // else four sweeps are two launches either way
        const LevelsPlan three = plan_levels(pr, 1, 3);
        if (remaining == 3 || leave || three.us / 3 < plan.us / 2) plan = three;
    }
    if (plan.V == 0 || (plan.sweeps == 2 && leave)) return 0;
    const LevelsKernel k = find_kernel(f32, star ? 1 : budget, plan.V, plan.waves, plan.sweeps, clamp, stream);
    Geometry g;
    g.V = plan.V;
    g.P = kLevelRows;
    g.halo_left = g.halo_right = ceil_div(plan.sweeps, plan.V);
    g.valid_lanes = min(plan.step_x / plan.V, kWave - 2 * g.halo_left);
    g.strips_x = plan.tiles_x;
    g.tiles_y = plan.tiles_y;
    g.rows_per_wave = kLevelRows;
    g.planes_per_wave = plan.planes;
    g.tiles_z = ceil_div(pr.D, plan.planes);
    g.tiles = (long)g.strips_x * g.tiles_y * g.tiles_z;
    g.xcd_remap = 1;
    g.blocks = ceil_div((int)g.tiles, kXcds) * kXcds;
    g.lds = (int)k.lds;
    if (geo) *geo = g;
    *err = hipSuccess;
    if (dry_run) return plan.sweeps;
    *err = f32 ? (star ? launch_levels<float, 1>(pr, k, plan, g) : budget == 2 ? launch_levels<float, 2>(pr, k, plan, g) : launch_levels<float, 3>(pr, k, plan, g))
               : (star ? launch_levels<double, 1>(pr, k, plan, g) : budget == 2 ? launch_levels<double, 2>(pr, k, plan, g) : launch_levels<double, 3>(pr, k, plan, g));
    if (*err != hipSuccess) (void)hipGetLastError();     // returned here: not left for the next call to find
    return plan.sweeps;
}

}  // namespace ssam
