// The dense fp64 filters without a compiled shape (ssam_kernel_dense.h): tile plan and launch.
#include "ssam_kernel_dense.h"

namespace ssam {

hipError_t launch_dense(const double* in, double* out, int W, int H, int D, const double* w, int M, int N, int K, int ax, int ay,
                        int az, int boundary, hipStream_t stream, Geometry* geo, bool dry_run)
{
    // parts of a filter: whole rows of one or more planes, at most kDenseTaps values; output planes two by two in 3D
    const int kmax = kDenseTaps / (M * N) > 0 ? kDenseTaps / (M * N) : 1;
    const int kp = ceil_div(K, ceil_div(K, kmax < K ? kmax : K));                      // as even as possible
    const int nmax = kDenseTaps / (M * kp) < N ? kDenseTaps / (M * kp) : N;            // M N kp <= kDenseTaps, or kp is 1
    const int np = ceil_div(N, ceil_div(N, nmax));
    const int tz = K > 1 && D > 1 ? 2 : 1;
    // Waves stacked in a block: four share the halo rows; fewer where the grid would leave compute units idle, or where eight
    // lanes side by side (32 rows per wave) and a large filter would need more than the 64 KB of LDS a launch may ask for.
    const int lane_cols = W <= 40 || (W % 64 > 0 && W % 64 <= 32 && W < 200) ? 3 : 4;
    const int wave_rows = 4 * (kWave >> lane_cols);
    const int tiles_x = ceil_div(W, 4 << lane_cols), tiles_z = ceil_div(D, tz);
    const int pitch = ((4 << lane_cols) + M + 8) & ~1;      // a lane's last window ends up to four columns past the tile
    auto lds_of = [&](int waves) { return ((size_t)(waves * wave_rows + np - 1) * pitch + 8) * sizeof(double); };
    int nw = 4;
    while (nw > 1 && ((long)tiles_x * ceil_div(H, nw * wave_rows) * tiles_z * nw < 2048 || lds_of(nw) > (64u << 10))) nw /= 2;
    const int tiles_y = ceil_div(H, nw * wave_rows);
    const long tiles = (long)tiles_x * tiles_y * tiles_z;
    const size_t lds = lds_of(nw);
    Geometry g;
    g.V = 4;
    g.P = 4;
    g.strips_x = tiles_x;
    g.tiles_y = tiles_y;
    g.tiles_z = tiles_z;
    g.tiles = tiles;
    g.xcd_remap = 1;
    g.lds = (int)lds;
    g.form = 1;
    g.valid_lanes = kWave;
    g.rows_per_wave = wave_rows;
    g.planes_per_wave = tz;
    g.blocks = tiles > kMaxBlocks ? -1 : ceil_div((int)tiles, kXcds) * kXcds;
    if (geo) *geo = g;
    if (!launchable(g)) return hipErrorNotSupported;
    if (dry_run) return hipSuccess;

    DenseArgs a;
    a.in = in;
    a.out = out;
    a.W = W; a.H = H; a.D = D;
    a.M = M;
    a.ax = ax;
    a.boundary = boundary;
    a.accumulate = 0;
    a.lane_cols = lane_cols;
    a.pitch = pitch;
    a.tiles_x = tiles_x;
    a.tiles_y = tiles_y;
    a.tiles = (int)tiles;
    a.blocks = g.blocks;
    a.xcd_remap = g.xcd_remap;
    for (int k0 = 0; k0 < K; k0 += kp)
        for (int n0 = 0; n0 < N; n0 += np) {
            a.K = K - k0 < kp ? K - k0 : kp;
            a.N = N - n0 < np ? N - n0 : np;
            a.ay = ay - n0;
            a.az = az - k0;
            for (int k = 0; k < a.K; ++k)
                for (int n = 0; n < a.N; ++n)
                    for (int m = 0; m < M; ++m) a.w[(k * a.N + n) * M + m] = w[((size_t)(k0 + k) * N + n0 + n) * M + m];
            const dim3 grid(g.blocks), block(nw * kWave);
#define SSAM_DENSE(TZ, NW) \
    if (tz == TZ && nw == NW) hipLaunchKernelGGL((dense_kernel<TZ, NW>), grid, block, lds, stream, a)
            SSAM_DENSE(1, 1);
            SSAM_DENSE(1, 2);
            SSAM_DENSE(1, 4);
            SSAM_DENSE(2, 1);
            SSAM_DENSE(2, 2);
            SSAM_DENSE(2, 4);
#undef SSAM_DENSE
            if (hipError_t e = hipGetLastError()) return e;
            a.accumulate = 1;
        }
    return hipSuccess;
}

}  // namespace ssam
