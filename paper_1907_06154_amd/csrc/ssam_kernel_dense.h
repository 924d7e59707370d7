// Dense fp64 filters of any extents, 2D and 3D: what no register-cache instance is compiled for.
//
// What bounds it: fp64 multiply-adds (M N K per point and 16 bytes; there is no faster unit, the fp64 matrix rate equals the
// vector rate).  One output per thread, every tap a load (the tap-list kernel), runs at 3 TFLOP/s: the loads bound it.  Here a
// lane owns 4 x 4 outputs (and two planes of them in 3D), the block stages the input plane it needs in LDS, and a lane slides
// an eight-column window along each staged row: two 16-byte LDS reads bring the operands of 64 multiply-adds (128 with two
// planes), the filter values come by scalar loads, four at a time, each used 4 x 4 times.
// Measured (tap list -> here): 20x20 on 2048^2 968 -> 104 us (32 TFLOP/s), 12x12 on 1999x1501 264 -> 39, 32x32 on 2048^2 2455 ->
// 274, 9x9x9 on 256^3 7400 -> 1200.  In 3D the few rows of a plane that all output rows share, and the barriers around every
// staged plane, leave it at 8 .. 20 TFLOP/s.
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
    double w[kDenseTaps + 4];      // four are read together, also of the last row's end
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
        // 3D: rows first .. last - 1, in which every output row and plane has taps, as a flat run of units, four filter columns of
        // one filter plane each.  A unit's window and weights are requested while the one before multiplies: scalar loads return
        // in any order, so the wait for a unit's weights is one for everything requested before it, and its first row comes before
        // the next requests.  Row by row, every eight columns waited for their scalar loads (5x6x4 on 256^3 423 -> 346 us, 7x7x7
        // on 53x256x202 203 -> 163, 9x9x9 on 256^3 1409 -> 1199, 8x8x2 on 256x256x200 262 -> 213; 4x4x4 and 2x2x9
        // equal).  In 2D it is mixed, 20x20 on 2048^2 103 -> 115, so 2D and K = 1 keep the form row by row.
        auto rows_all = [&](int first, int last) __attribute__((always_inline)) {
            double win[2][8], w[2][4][4];
            int rn = first, mn = 0;                  // the unit requested next
            auto request_window = [&](int buf) __attribute__((always_inline)) {
                const double* const q = own + rn * pitch + mn;
#pragma unroll
                for (int i = 0; i < 8; i += 2) {
                    const vec2 v = *reinterpret_cast<const vec2*>(q + i);
                    win[buf][i] = v[0];
                    win[buf][i + 1] = v[1];
                }
            };
            auto request_weights = [&](int buf, int t) __attribute__((always_inline)) {
                const ConstPtr<double> wr = wts + ((size_t)(p - t) * N + rn) * M + mn;
#pragma unroll
                for (int y = 0; y < 4; ++y)
#pragma unroll
                    for (int i = 0; i < 4; ++i) w[buf][y][i] = (wr - (long)y * M)[i];
            };
            auto multiply = [&](int wb, int vb, int t, int y, int i) __attribute__((always_inline)) {
#pragma unroll
                for (int x = 0; x < 4; ++x) acc[t][y][x] = fma_t(win[vb][i + x], w[wb][y][i], acc[t][y][x]);
            };
            // The filter columns of output plane t (FULL: four): the first output row, the requests, the other rows.
            auto unit = [&](auto full_tag, auto vb_tag, auto t_tag, int count) __attribute__((always_inline)) {
                constexpr bool FULL = decltype(full_tag)::value;
                constexpr int vb = decltype(vb_tag)::value, t = decltype(t_tag)::value, wb = (vb * TZ + t) & 1;
                auto output_row = [&](int y) __attribute__((always_inline)) {
                    multiply(wb, vb, t, y, 0);
                    if (FULL || count > 1) multiply(wb, vb, t, y, 1);
                    if (FULL || count > 2) multiply(wb, vb, t, y, 2);
                    if constexpr (FULL) multiply(wb, vb, t, y, 3);
                };
                output_row(0);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (t == TZ - 1) {
                    mn += 4;
                    const bool row_end = mn >= M;
                    mn = row_end ? 0 : mn;
                    rn = row_end ? min(rn + 1, last - 1) : rn;      // past the last unit: in bounds, and unused
                    request_window(vb ^ 1);
                    request_weights(wb ^ 1, 0);
                } else {
                    request_weights(wb ^ 1, t + 1);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int y = 1; y < 4; ++y) output_row(y);
                __builtin_amdgcn_sched_barrier(0);
            };
            request_window(0);
            request_weights(0, 0);
            const int per_row = (M + 3) / 4, units = (last - first) * per_row;
            int m = 0;
            auto both = [&](auto vb_tag) __attribute__((always_inline)) {
                const int count = M - m;
                if (count >= 4) static_for<TZ>([&](auto t) __attribute__((always_inline)) { unit(std::true_type{}, vb_tag, t, 4); });
                else static_for<TZ>([&](auto t) __attribute__((always_inline)) { unit(std::false_type{}, vb_tag, t, count); });
                m = m + 4 < M ? m + 4 : 0;
            };
            int u = 0;
            for (; u + 1 < units; u += 2) {
                both(std::integral_constant<int, 0>{});
                both(std::integral_constant<int, 1>{});
            }
            if (u < units) both(std::integral_constant<int, 0>{});
        };
        if constexpr (TZ == 1) {
            for (int r = 0; r < N + 3; ++r) {
                if (r >= 3 && r < N) row(std::true_type{}, r);
                else row(std::false_type{}, r);
            }
        } else if (p >= TZ - 1 && p < K && N > 3) {
            for (int r = 0; r < 3; ++r) row(std::false_type{}, r);
            rows_all(3, N);
            for (int r = N; r < N + 3; ++r) row(std::false_type{}, r);
        } else {
            for (int r = 0; r < N + 3; ++r) row(std::false_type{}, r);
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
