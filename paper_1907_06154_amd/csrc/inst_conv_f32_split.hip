// The dense fp32 filters on the bf16 matrix cores (ssam_kernel2d_split.h): instances, tile plan, launch.
#include <atomic>
#include <cmath>

#include "ssam_kernel2d_split.h"

namespace ssam {
namespace {

typedef void (*SplitKernel)(const ArgsSplit2D, int);
constexpr int kSplitWaves = 4;

// Three strips of 64 columns per wave only up to four patch bands: with five and six the sums of three strips no longer
// fit 256 registers (15x15 on 8192^2: 337 us spilling, 247 us with two strips; 20x20: 329 and 319).  Four bands and a tail
// piece spill seven registers with three strips and are still the fastest (9x13 on 8192^2 146 us, two strips 154).
template <int NX, bool TAIL>
SplitKernel split_kernel(int bands)
{
    switch (bands) {
        case 1: return &ssam2d_split_kernel<1, NX, TAIL, kSplitWaves>;
        case 2: return &ssam2d_split_kernel<2, NX, TAIL, kSplitWaves>;
        case 3: return &ssam2d_split_kernel<3, NX, TAIL, kSplitWaves>;
        case 4: return &ssam2d_split_kernel<4, NX, TAIL, kSplitWaves>;
        case 5: return &ssam2d_split_kernel<5, NX < 3 ? NX : 2, TAIL, kSplitWaves>;
        default: return &ssam2d_split_kernel<6, NX < 3 ? NX : 2, TAIL, kSplitWaves>;
    }
}

// More than 64 KB of LDS per workgroup is asked for once per kernel and device.
hipError_t allow_lds(SplitKernel kernel, int index)
{
    static std::atomic<unsigned long long> done[64];   // by instance: bit per device
    int dev = 0;
    if (hipError_t e = hipGetDevice(&dev)) return e;
    const unsigned long long bit = 1ull << (dev & 63);
    if (done[index].load(std::memory_order_relaxed) & bit) return hipSuccess;
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 160 << 10);
    if (e == hipSuccess) done[index].fetch_or(bit, std::memory_order_relaxed);
    return e;
}

}  // namespace

// The scaled weights and inputs have to stay clear of the ends of the exponent range; what is infinite, NaN or beyond 2^90 in
// the filter goes to the other kernels (the same in the data: to the plain path inside the kernel), and so does a filter with a
// tap so small beside its largest that parts of it would be subnormal.
long split_taps(const float* w, long count, int* exponent)
{
    float top = 0.0f, least = INFINITY;
    long taps = 0;
    for (long i = 0; i < count; ++i) {
        const float a = std::fabs(w[i]);
        if (!(a <= 0x1p90f)) return 0;
        if (a == 0.0f) continue;
        ++taps;
        top = std::fmax(top, a);
        least = std::fmin(least, a);
    }
    if (top < 0x1p-90f || std::ldexp(least, 100) < top) return 0;
    std::frexp(top, exponent);      // top = f 2^exponent, f in [1/2, 1)
    return taps;
}

hipError_t launch2d_split(const Problem2D& pr, const Tuning& tu, Geometry* geo, bool dry_run)
{
    if (pr.W < 64) return hipErrorNotSupported;
    const float* w = static_cast<const float*>(pr.w);
    int ew;
    // One tap or two: the products left out show beside so few roundings (error against 64 bits, one tap 1.02 times that of
    // fp32 multiply-adds, two 0.8 .. 1.09, three 0.7 .. 0.86).
    if (split_taps(w, (long)pr.M * pr.N, &ew) < 3) return hipErrorNotSupported;

    // patch columns M + 3: whole pieces of eight, and four more in a tail piece where that holds the rest
    const int rest = (pr.M + 3) % 8;
    const bool tail = pr.M > 5 && rest >= 1 && rest <= 4;
    const int groups = tail ? (pr.M + 3) / 8 : ceil_div(pr.M + 3, 8);
    const int max_bands = groups <= 2 || (groups == 3 && !tail) ? 6 : groups == 4 && tail ? 3 : 4;
    const int max_rows = 4 * max_bands - 3;
    const int parts = ceil_div(pr.N, max_rows), part_rows = ceil_div(pr.N, parts);
    const int bands = ceil_div(part_rows + 3, 4);
    const int pieces = bands * groups + (tail ? (bands + 1) / 2 : 0);

    // Tile plan: 64 nx columns (nx = 1, 2, 3) by `rows` rows per wave, chosen by a model of the cycles a SIMD spends.  Its
    // matrix and vector instructions add up, which fits the times (20x20 on 8192^2: matrix pipe busy for 0.70 of the cycles, other
    // vector instructions 0.14; 9x9 0.44 and 0.29, more of the waves' time in waits): a step of four output rows issues 96 cycles
    // of matrix instructions per table piece and 64 columns, staging four input rows about 60 + 46 (nx + 1) vector
    // instructions, the bands - 1 steps above a tile included, and every workgroup builds the table once.  Four waves per
    // SIMD, which one strip and a small table leave room for, hide more than two.  A partly filled last round costs what its
    // fullest SIMD does.  Tiles of more than 512 rows save nothing more; pictures that would want taller ones (20x20 from
    // 20000^2 on) are shared out in more rounds of 512.
    // Measured with one, two, three strips (us): 9x9 on 8192^2 135, 135, 129 (chosen: three), 4003x3001 31.9, 33.8, 30.7
    // (three), 2048^2 13.8, 14.3, 16.4 (two), 1024^2 9.8, 8.1, 9.6 (two); 9x13 on 8192^2 178, 154, 146 (three); 20x20 358, 319
    // (two).  Over 100 pairs of filter and picture the choice was at most 16 % from the best, 2 % in the mean.
    int nx = 1, rows = 512;
    double best = 1e30;
    for (int cand = 1; cand <= (bands <= 4 ? 3 : 2); ++cand) {
        const long strips = ceil_div(pr.W, 64 * cand);
        const int per_simd = cand == 1 && pieces <= 9 ? 4 : 2;
        for (int k = 0; k <= 3; ++k) {     // rows that give every SIMD one wave, then one, two, three fills of waves
            const long want = 1024L * (k == 0 ? 1 : k * per_simd) / strips;
            int r = ceil_div(ceil_div(pr.H, want < 1 ? 1 : (int)want), 4) * 4;
            if (r > 512) r = 512;
            if (tu.rows_per_wave > 0) r = ceil_div(tu.rows_per_wave, 4) * 4;
            const double busy = r / 4 * pieces * 96.0 * cand * (cand == 1 ? 1.1 : 1.0) +
                                (r / 4 + bands - 1) * 4.0 * (60 + 46 * (cand + 1)) + 150.0 * pieces + 1500.0;
            const long tiles = strips * ceil_div(pr.H, r), round = 1024L * per_simd;
            const long full = (tiles - 1) / round, last = (tiles - full * round + 1023) / 1024;
            const double cost = (full * per_simd + (last > 1 ? (double)last : 1.6)) * busy * (per_simd == 4 ? 0.9 : 1.0);
            if (cost < best) { best = cost; nx = cand; rows = r; }
        }
    }
    Geometry g;
    g.V = 4;
    g.P = 4;
    g.halo_left = ceil_div(pr.ax, 4);
    g.halo_right = ceil_div(pr.M - 1 - pr.ax, 4);
    g.valid_lanes = 16 * nx;
    g.strips_x = ceil_div(pr.W, 64 * nx);
    if (rows > ceil_div(pr.H, 4) * 4) rows = ceil_div(pr.H, 4) * 4;
    if (rows > 4 * kSplitMaxBands) rows = 4 * kSplitMaxBands;
    while ((long)g.strips_x * ceil_div(pr.H, rows) > 4 * kMaxBlocks) rows *= 2;
    g.rows_per_wave = rows;
    g.tiles_y = ceil_div(pr.H, rows);
    plan_blocks(&g, tu.xcd_remap);
    const int quads = 16 * nx + 2 * groups - (tail ? 0 : 1);
    const int pitch = ceil_div(quads, 8) * 8;     // 8-byte words per staged row: 0 .. 3 % of the LDS cycles are bank conflicts
    size_t stage = (size_t)kSplitWaves * 12 * pitch * 8;
    if (stage < (size_t)kSplitMaxTaps * 4) stage = kSplitMaxTaps * 4;
    const size_t lds = (size_t)pieces * 3 * kWave * 16 + stage;
    g.lds = (int)lds;
    if (geo) *geo = g;
    if (!launchable(g)) return hipErrorInvalidConfiguration;
    if (dry_run) return hipSuccess;

    const SplitKernel kernel = nx == 1 ? (tail ? split_kernel<1, true>(bands) : split_kernel<1, false>(bands))
                             : nx == 2 ? (tail ? split_kernel<2, true>(bands) : split_kernel<2, false>(bands))
                                       : (tail ? split_kernel<3, true>(bands) : split_kernel<3, false>(bands));
    if (hipError_t e = allow_lds(kernel, ((nx - 1) * 2 + (tail ? 1 : 0)) * 6 + bands - 1)) return e;

    ArgsSplit2D a;
    a.in = static_cast<const float*>(pr.in);
    a.out = static_cast<float*>(pr.out);
    a.W = pr.W;
    a.H = pr.H;
    a.M = pr.M;
    a.ax = pr.ax;
    a.groups = groups;
    a.boundary = pr.boundary;
    a.strips_x = g.strips_x;
    a.tiles = g.tiles;
    a.rows = rows;
    a.blocks = g.blocks;
    a.xcd_remap = g.xcd_remap;
    a.w_scale = std::ldexp(1.0f, 1 - ew);
    a.out_scale = std::ldexp(1.0f, ew - 1 - 24);
    for (int n0 = 0; n0 < pr.N; n0 += part_rows) {
        a.N = pr.N - n0 < part_rows ? pr.N - n0 : part_rows;
        a.ay = pr.ay - n0;
        a.accumulate = n0 > 0;
        for (int i = 0; i < pr.M * a.N; ++i) a.w[i] = w[n0 * pr.M + i];
        hipLaunchKernelGGL(kernel, dim3(g.blocks), dim3(kSplitWaves * kWave), lds, pr.stream, a, pitch);
        if (hipError_t e = hipGetLastError()) return e;
    }
    return hipSuccess;
}

}  // namespace ssam
