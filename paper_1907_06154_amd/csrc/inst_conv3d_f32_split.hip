// The dense fp32 3D filters on the bf16 matrix cores (ssam_kernel3d_split.h): instances, tile plan, launch.
#include <atomic>

#include "ssam_kernel3d_split.h"

namespace ssam {
template <> Split3dKernel split3d_kernel<1, false>(int, int);
template <> Split3dKernel split3d_kernel<1, true>(int, int);
template <> Split3dKernel split3d_kernel<2, false>(int, int);
template <> Split3dKernel split3d_kernel<2, true>(int, int);

namespace {

// More than 64 KB of LDS per workgroup is asked for once per kernel and device.
hipError_t allow_lds(Split3dKernel kernel, int index)
{
    static std::atomic<unsigned long long> done[96];   // by instance: bit per device
    int dev = 0;
    if (hipError_t e = hipGetDevice(&dev)) return e;
    const unsigned long long bit = 1ull << (dev & 63);
    if (done[index].load(std::memory_order_relaxed) & bit) return hipSuccess;
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 160 << 10);
    if (e == hipSuccess) done[index].fetch_or(bit, std::memory_order_relaxed);
    return e;
}

// One part of a filter: kp planes of np rows, one launch.
struct Part {
    int bands, pieces, tb;
    size_t lds;
};

Part plan_part(int M, int np, int kp, int groups, bool tail)
{
    Part p;
    p.bands = ceil_div(np + 3, 4);
    p.pieces = p.bands * groups + (tail ? (p.bands + 1) / 2 : 0);
    p.tb = split3d_bands(kp, p.bands);
    const int quads = 16 + 2 * groups - (tail ? 0 : 1);
    size_t stage = (size_t)kSplit3dWaves * 3 * (p.tb + p.bands - 1) * 4 * quads * 8;
    if (stage < (size_t)kSplit3dTaps * 4) stage = (size_t)kSplit3dTaps * 4;
    p.lds = (size_t)kp * p.pieces * 3 * kWave * 16 + stage;
    return p;
}

}  // namespace

hipError_t launch3d_split(const float* in, float* out, int W, int H, int D, const float* w, int M, int N, int K, int ax, int ay,
                          int az, int boundary, hipStream_t stream, const Tuning& tu, Geometry* geo, bool dry_run)
{
    if (W < 4 || (long)W * H > 0x7fffffffL) return hipErrorNotSupported;
    int ew;
    const long taps = split_taps(w, (long)M * N * K, &ew);
    if (2 * taps < 5L * K) return hipErrorNotSupported;      // see ssam_kernel3d_split.h: fewer round worse than fp32 multiply-adds

    const int rest = (M + 3) % 8;
    const bool tail = M > 5 && rest >= 1 && rest <= 4;
    const int groups = tail ? (M + 3) / 8 : ceil_div(M + 3, 8);
    // parts: at most 9 rows (three bands) and 7 planes (4 with two column groups), as many as the workgroup's LDS and the launch arguments hold
    const int nparts = ceil_div(N, 9), np = ceil_div(N, nparts);
    int kparts = ceil_div(K, split3d_max_planes(groups));
    while (plan_part(M, np, ceil_div(K, kparts), groups, tail).lds > (160u << 10) || M * np * ceil_div(K, kparts) > kSplit3dTaps) ++kparts;
    const int kp = ceil_div(K, kparts);
    const Part part = plan_part(M, np, kp, groups, tail);

    // Chunks along z: the longest that still give every SIMD its two waves, unless shorter ones fill the last round better.
    const long tiles_xy = (long)ceil_div(W, 64) * ceil_div(H, 4 * part.tb);
    int planes = tu.planes_per_wave;
    if (planes <= 0) {
        double best = 1e30;
        for (int k = 0; k <= 4; ++k) {
            const long want = (k == 0 ? 1024 : 2048L * k) / tiles_xy;
            const int pl = ceil_div(D, want < 1 ? 1 : want > D ? D : (int)want);
            const long tiles = tiles_xy * ceil_div(D, pl), full = (tiles - 1) / 2048, last = (tiles - full * 2048 + 1023) / 1024;
            const double busy = pl * kp * part.pieces * 96.0 * part.tb + (pl + kp - 1) * 4.0 * (60 + 34 * (part.tb + part.bands - 1)) +
                                100.0 * kp * part.pieces + 1500.0;
            const double cost = (full * 2 + (last > 1 ? (double)last : 1.6)) * busy;
            if (cost < best) { best = cost; planes = pl; }
        }
    }
    if (planes > D) planes = D;
    if (planes > kSplitMaxBands) planes = kSplitMaxBands;
    Geometry g;
    g.V = 4;
    g.P = 4 * part.tb;
    g.halo_left = ceil_div(ax, 4);
    g.halo_right = ceil_div(M - 1 - ax, 4);
    g.valid_lanes = 16;
    g.strips_x = ceil_div(W, 64);
    g.rows_per_wave = g.P;
    g.tiles_y = ceil_div(H, g.P);
    g.planes_per_wave = planes;
    g.tiles_z = ceil_div(D, planes);
    g.tiles = (long)g.strips_x * g.tiles_y * g.tiles_z;
    g.xcd_remap = tu.xcd_remap < 0 ? 1 : (tu.xcd_remap ? 1 : 0);
    const long blocks = (g.tiles + kSplit3dWaves - 1) / kSplit3dWaves;
    g.blocks = blocks > kMaxBlocks ? -1 : (g.xcd_remap ? ceil_div((int)blocks, kXcds) * kXcds : (int)blocks);
    g.lds = (int)part.lds;
    if (geo) *geo = g;
    if (!launchable(g)) return hipErrorNotSupported;
    if (dry_run) return hipSuccess;

    ArgsSplit3D a;
    a.in = in;
    a.out = out;
    a.W = W; a.H = H; a.D = D;
    a.M = M;
    a.ax = ax;
    a.boundary = boundary;
    a.strips_x = g.strips_x;
    a.tiles_y = g.tiles_y;
    a.tiles = g.tiles;
    a.planes = planes;
    a.blocks = g.blocks;
    a.xcd_remap = g.xcd_remap;
    a.accumulate = 0;
    a.w_scale = std::ldexp(1.0f, 1 - ew);
    a.out_scale = std::ldexp(1.0f, ew - 1 - 24);
    const Split3dKernel kernel = groups == 1 ? (tail ? split3d_kernel<1, true>(kp, part.bands) : split3d_kernel<1, false>(kp, part.bands))
                                             : (tail ? split3d_kernel<2, true>(kp, part.bands) : split3d_kernel<2, false>(kp, part.bands));
    if (!kernel) return hipErrorNotSupported;
    if (hipError_t e = allow_lds(kernel, ((kp - 1) * 3 + part.bands - 1) * 4 + (groups - 1) * 2 + (tail ? 1 : 0))) return e;
    for (int k0 = 0; k0 < K; k0 += kp)
        for (int n0 = 0; n0 < N; n0 += np) {
            // A last part may have fewer rows or planes.  The matrix operand is zero there; the plain path has to know, or an
            // infinity would reach outputs that do not read it.
            a.N = N - n0 < np ? N - n0 : np;
            a.K = K - k0 < kp ? K - k0 : kp;
            a.ay = ay - n0;
            a.az = az - k0;
            for (int k = 0; k < a.K; ++k)
                for (int n = 0; n < a.N; ++n)
                    for (int m = 0; m < M; ++m) a.w[(k * a.N + n) * M + m] = w[((long)(k0 + k) * N + n0 + n) * M + m];
            hipLaunchKernelGGL(kernel, dim3(g.blocks), dim3(kSplit3dWaves * kWave), part.lds, stream, a);
            if (hipError_t e = hipGetLastError()) return e;
            a.accumulate = 1;
        }
    return hipSuccess;
}

}  // namespace ssam
