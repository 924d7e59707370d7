// Dense fp64 filters of any extents, 2D and 3D: what no register-cache instance is compiled for.
//
// What bounds it: fp64 multiply-adds (M N K per point and 16 bytes; there is no faster unit, the fp64 matrix rate equals the
// vector rate).  One output per thread, every tap a load (the tap-list kernel), runs at 3 TFLOP/s: the loads bound it.  Here a
// lane owns 4 x 4 outputs (and two planes of them in 3D), the block stages the input plane it needs in LDS, and a lane slides
// an eight-column window along each staged row: two 16-byte LDS reads bring the operands of 64 multiply-adds (128 with two
// planes), the filter values come by scalar loads, four at a time, each used 4 x 4 times.
// Measured (tap list -> here): 20x20 on 2048^2 968 -> 104 us (32 TFLOP/s), 12x12 on 1999x1501 264 -> 39, 32x32 on 2048^2 2455 ->
// 274, 9x9x9 on 256^3 7400 -> 1430.  In 3D the few rows of a plane that all output rows share, and the barriers around every
// staged plane, leave it at 8 .. 17 TFLOP/s.
// Extents are run-time values.  Taps beyond the filter are never multiplied (no zero padding), so infinities and NaN reach
// exactly the outputs whose footprint holds them, and every output adds its taps in the order of the tap-list kernel.
#pragma once
#include "ssam_device.h"
#include "ssam_host.h"

namespace ssam {

constexpr int kDenseTaps = 448;      // taps of one launch (3584 bytes of launch arguments)

struct DenseArgs {
    const double* in;
    double* out;
    int W, H, D;
    int M, N, K, ax, ay, az;
    int boundary;
    int accumulate;
    int lane_cols;       // log2 of the lanes side by side in x (4 columns each); the others are stacked in y
    int pitch;           // elements per staged row, even
    int tiles_x, tiles_y;
    int tiles;
    int blocks, xcd_remap;
    double w[kDenseTaps];
};

template <int TZ, int NW>
__global__ __launch_bounds__(NW* kWave) void dense_kernel(const DenseArgs a)
{
    typedef double vec2 __attribute__((ext_vector_type(2)));
    typedef double vec2u __attribute__((ext_vector_type(2), aligned(8)));
    extern __shared__ __attribute__((aligned(16))) char lds_raw[];
    double* const tile = reinterpret_cast<double*>(lds_raw);
    const ConstPtr<double> wts = kernarg_member<double>(offsetof(DenseArgs, w));

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lb = logical_block(blockIdx.x, a.blocks, a.xcd_remap);
    if (lb >= a.tiles) return;                      // block-uniform
    const int tx = lb % a.tiles_x, ty = (lb / a.tiles_x) % a.tiles_y, tz = lb / (a.tiles_x * a.tiles_y);
    const int lx = lane & ((1 << a.lane_cols) - 1), ly = lane >> a.lane_cols;
    const int wave_rows = 4 * (kWave >> a.lane_cols);
    const int W = a.W, H = a.H, D = a.D, M = a.M, N = a.N, K = a.K, pitch = a.pitch;
    const int x0 = tx * (4 << a.lane_cols), y0 = ty * (NW * wave_rows), z0 = tz * TZ;
    const int cols = (4 << a.lane_cols) + M - 1, rows = NW * wave_rows + N - 1;
    const bool clamp = a.boundary == kClamp;
    const int xs = x0 - a.ax, ys = y0 - a.ay;
    const double* const own = tile + (size_t)(wave * wave_rows + 4 * ly) * pitch + 4 * lx;

    double acc[TZ][4][4];
#pragma unroll
    for (int t = 0; t < TZ; ++t)
#pragma unroll
        for (int y = 0; y < 4; ++y)
#pragma unroll
            for (int x = 0; x < 4; ++x) acc[t][y][x] = 0.0;

    for (int p = 0; p < K + TZ - 1; ++p) {          // input plane z0 - az + p
        const int z = z0 - a.az + p;
        const bool plane_in = clamp || (z >= 0 && z < D);
        const double* const pz = a.in + (size_t)min(max(z, 0), D - 1) * W * H;
        if (p > 0) __syncthreads();
        // a wave stages whole rows, four at a time
        for (int r0 = wave * 4; r0 < rows; r0 += NW * 4) {
            for (int c = lane; c < cols; c += kWave) {
                const int x = xs + c;
                const bool col_in = clamp || (x >= 0 && x < W);
                const int xx = min(max(x, 0), W - 1);
                double v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = pz[(size_t)min(max(ys + r0 + i, 0), H - 1) * W + xx];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int y = ys + r0 + i;
                    if (r0 + i < rows) tile[(r0 + i) * pitch + c] = (plane_in && col_in && (clamp || (y >= 0 && y < H))) ? v[i] : 0.0;
                }
            }
        }
        __syncthreads();

        // staged row r of the lane's window is filter row r - y of output row y
        auto row = [&](auto all_tag, int r) __attribute__((always_inline)) {
            constexpr bool ALL = decltype(all_tag)::value;     // every output row and plane has taps in this row
            const double* q = own + r * pitch;
            const ConstPtr<double> wr = wts + ((size_t)p * N + r) * M;    // output plane 0, output row 0
            vec2 lo0 = *reinterpret_cast<const vec2*>(q), lo1 = *reinterpret_cast<const vec2*>(q + 2);
            double win[8] = {lo0[0], lo0[1], lo1[0], lo1[1], 0.0, 0.0, 0.0, 0.0};
            auto taps = [&](auto count_tag, int m) __attribute__((always_inline)) {
                constexpr int COUNT = decltype(count_tag)::value;
#pragma unroll
                for (int t = 0; t < TZ; ++t)
#pragma unroll
                    for (int y = 0; y < 4; ++y)
                        if (ALL || (p - t >= 0 && p - t < K && r - y >= 0 && r - y < N)) {
                            const ConstPtr<double> w = wr - ((long)t * N + y) * M + m;
#pragma unroll
                            for (int i = 0; i < COUNT; ++i)
#pragma unroll
                                for (int x = 0; x < 4; ++x) acc[t][y][x] = fma_t(win[i + x], w[i], acc[t][y][x]);
                        }
            };
            int m = 0;
#pragma unroll 2
            for (; m + 4 <= M; m += 4) {
                const vec2 hi0 = *reinterpret_cast<const vec2*>(q + m + 4), hi1 = *reinterpret_cast<const vec2*>(q + m + 6);
                win[4] = hi0[0]; win[5] = hi0[1]; win[6] = hi1[0]; win[7] = hi1[1];
                taps(std::integral_constant<int, 4>{}, m);
#pragma unroll
                for (int i = 0; i < 4; ++i) win[i] = win[i + 4];
            }
            const int rest = M - m;                 // wave-uniform
            if (rest > 0) {
                const vec2 hi0 = *reinterpret_cast<const vec2*>(q + m + 4), hi1 = *reinterpret_cast<const vec2*>(q + m + 6);
                win[4] = hi0[0]; win[5] = hi0[1]; win[6] = hi1[0]; win[7] = hi1[1];
                if (rest == 1) taps(std::integral_constant<int, 1>{}, m);
                else if (rest == 2) taps(std::integral_constant<int, 2>{}, m);
                else taps(std::integral_constant<int, 3>{}, m);
            }
        };
        const bool planes_all = TZ == 1 || (p >= TZ - 1 && p < K);
        for (int r = 0; r < N + 3; ++r) {
            if (planes_all && r >= 3 && r < N) row(std::true_type{}, r);
            else row(std::false_type{}, r);
        }
    }

    const int x = x0 + 4 * lx;
#pragma unroll
    for (int t = 0; t < TZ; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int y = y0 + wave * wave_rows + 4 * ly + i;
            if (z0 + t >= D || y >= H || x >= W) continue;
            double* const q = a.out + ((size_t)(z0 + t) * H + y) * W + x;
            if (x + 4 <= W) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    vec2u v{acc[t][i][2 * h], acc[t][i][2 * h + 1]};
                    vec2u* const d = reinterpret_cast<vec2u*>(q + 2 * h);
                    if (a.accumulate) v += *d;
                    *d = v;
                }
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (x + e < W) q[e] = a.accumulate ? q[e] + acc[t][i][e] : acc[t][i][e];
            }
        }
}

// Filter w[K][N][M] anchored at (ax, ay, az), in as many launches as the launch arguments need.
hipError_t launch_dense(const double* in, double* out, int W, int H, int D, const double* w, int M, int N, int K, int ax, int ay,
                        int az, int boundary, hipStream_t stream, Geometry* geo, bool dry_run);

}  // namespace ssam
