// Many Jacobi sweeps of a 2D stencil on a small grid in one launch: a block keeps its tile of the grid, halo and all, in
// registers for all of them.
//
// What bounds small grids in ssam_kernel2d_fused.h is one wave's latency: it marches down its tile, its sweeps follow one another
// in every group of rows, and the first groups of a tile only warm up (1023x1025, ten sweeps: 29 us in two launches of which the
// grid's loads and operations need 1.6).  Here a sweep is a step of the whole block: every wave holds P rows of 64 V columns,
// shows the rows at its rim to the others through LDS (two buffers, so one barrier a sweep), shifts columns from lane to lane,
// and computes its rows anew.  The number of sweeps is a run-time count; each takes R rows and columns of the tile's rim, and the
// planner (inst_tile2d.hip) weighs that against launches.
// Tiles lie inside the grid, the last ones of a row or column moved back to end with it, so that there are no ragged tiles, and the
// boundary rule is what a wave sees beyond the tile: nothing, or the edge row or column repeated.  (Inside the grid that is wrong,
// and the halo takes it.)
// Four rows per wave: with eight, 128 registers hold less beside them and the plans are coarser (0.9 .. 1.0 of the time for radius
// 1 on 2048^2, more on all others).  Sixteen waves of 64 x {1, 2, 4} columns; one element per lane on the smallest grids.
// (With four, the fp64 stars of radius 4, 5 and 6 spill 5, 9 and 28 registers at V = 2, the fp32 star of radius 6 two at V = 4.)
// Measured, us, ten sweeps, from the marching kernels to this one: 1023x1025 fp32 star r1, clamp 29 -> 9.9, star r6 145 -> 56, box r2
// 73 -> 28; 512^2 fp32 star r1 23 -> 6.0, star r6 96 -> 29, box r2 36 -> 14, fp64 star r1 20 -> 7.6, box r2 27 -> 18; 2048^2 star
// r1 fp32 42 -> 22, fp64 58 -> 30.
#pragma once
#include "ssam_device.h"
#include "ssam_host.h"

namespace ssam {

constexpr int kTileWaves = 16;     // waves of a block, at most

template <typename T, int NWTS>
struct ArgsTile2D {
    const T* in;
    T* out;
    int W, H;
    int boundary, sweeps;
    int tiles_x, step_x, step_y;   // tiles start step_x columns, step_y rows apart (the last ones end with the grid; a tile's extent: one covers that axis)
    T w[NWTS];
};

// V elements from an address aligned to the element.
template <typename T, int V>
__device__ __forceinline__ void tile_load(const T* p, T (&dst)[V])
{
    if constexpr (V == 1) dst[0] = *p;
    else load_vec_elem<T, V, false>(p, dst);
}

template <typename T, int V, int P, class Mask>
__global__ __launch_bounds__(kTileWaves* kWave) void ssam2d_tile_kernel(const ArgsTile2D<T, Mask::kNW> a)
{
    constexpr int R = Mask::kAX, N = 2 * R + 1;
    constexpr bool STAR = Mask::kNW < N * N;
    constexpr bool PIN = Mask::kNW * sizeof(T) > 256;   // more coefficients than stay in scalar registers: loaded where used
    constexpr int HC = (R + V - 1) / V;              // lane-to-lane shifts per side
    constexpr int PUB = 2 * R < P ? 2 * R : P;       // rows of a wave that others read
    typedef typename VecOf<T, V>::type vec_t;
    typedef __attribute__((address_space(3))) vec_t lds_vec;
    extern __shared__ __attribute__((aligned(16))) char lds_raw[];

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int waves = blockDim.x >> 6;
    const int TH = waves * P;
    constexpr int TW = kWave * V;
    const int tx = blockIdx.x % a.tiles_x, ty = blockIdx.x / a.tiles_x;
    const int W = a.W, H = a.H;
    const int x0 = min(tx * a.step_x, W - TW), y0 = min(ty * a.step_y, H - TH);
    // what the tile stores: all but the halo of its sweeps, and up to the grid's edge where it lies there
    const int halo_x = (TW - a.step_x) / 2, halo_y = (TH - a.step_y) / 2;
    const int xa = tx == 0 ? 0 : tx * a.step_x + halo_x, xb = x0 + TW >= W ? W : (tx + 1) * a.step_x + halo_x;
    const int ya = ty == 0 ? 0 : ty * a.step_y + halo_y, yb = y0 + TH >= H ? H : (ty + 1) * a.step_y + halo_y;
    typedef ArgsTile2D<T, Mask::kNW> Args;
    const ConstPtr<T> wts = kernarg_member<T>(offsetof(Args, w));
    const int row0 = wave * P;                        // the wave's first row in the tile
    const int xc = x0 + lane * V;

    T cur[P][V];
#pragma unroll
    for (int p = 0; p < P; ++p) tile_load<T, V>(a.in + (size_t)(y0 + row0 + p) * W + xc, cur[p]);

    lds_vec* const lds = (lds_vec*)(__attribute__((address_space(3))) char*)lds_raw;
    const int buffer = waves * PUB * kWave;           // pieces of one buffer; two buffers, then a row of zeros
    auto slot = [](int p) { return PUB == P || p < R ? p : p - (P - PUB); };

    auto march = [&](auto clamp_tag) __attribute__((always_inline)) {
        constexpr bool CLAMP = decltype(clamp_tag)::value;
        // the R rows above and below the wave's own: other waves', or beyond the tile, which is beyond the grid where it matters
        int above[R], below[R];
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int ga = row0 - R + k, gb = row0 + P + k;
            const int ca = max(ga, 0), cb = min(gb, TH - 1);
            above[k] = !CLAMP && ga < 0 ? 2 * buffer : ((ca / P) * PUB + slot(ca % P)) * kWave;
            below[k] = !CLAMP && gb >= TH ? 2 * buffer : ((cb / P) * PUB + slot(cb % P)) * kWave;
        }
        int offset = 0;
        for (int s = 0; s < a.sweeps; ++s) {
#pragma unroll
            for (int p = 0; p < P; ++p) {
                if (PUB < P && p >= R && p < P - R) continue;
                vec_t v;
                if constexpr (V == 1) v = cur[p][0];
                else {
#pragma unroll
                    for (int j = 0; j < V; ++j) v[j] = cur[p][j];
                }
                lds[offset + (wave * PUB + slot(p)) * kWave + lane] = v;
            }
            __syncthreads();
            T up[R][V], down[R][V];
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const vec_t u = lds[above[k] + (!CLAMP && above[k] == 2 * buffer ? 0 : offset) + lane];
                const vec_t d = lds[below[k] + (!CLAMP && below[k] == 2 * buffer ? 0 : offset) + lane];
                if constexpr (V == 1) up[k][0] = u, down[k][0] = d;
                else {
#pragma unroll
                    for (int j = 0; j < V; ++j) up[k][j] = u[j], down[k][j] = d[j];
                }
            }
            auto row = [&](int k, int j) __attribute__((always_inline)) {
                return k < R ? up[k < R ? k : 0][j] : k < R + P ? cur[k >= R && k < R + P ? k - R : 0][j] : down[k >= R + P ? k - R - P : 0][j];
            };
            // row k of the window with R columns more on either side; a column beyond the tile is zero, or the edge column
            auto widen = [&](int k, T (&xs)[(2 * HC + 1) * V]) __attribute__((always_inline)) {
#pragma unroll
                for (int j = 0; j < V; ++j) xs[HC * V + j] = row(k, j);
#pragma unroll
                for (int h = 1; h <= HC; ++h)
#pragma unroll
                    for (int j = 0; j < V; ++j) {
                        const T l = xs[(HC - h + 1) * V + j], r = xs[(HC + h - 1) * V + j];
                        xs[(HC - h) * V + j] = CLAMP ? shift_in_up(l, xs[HC * V]) : shift_up(l);
                        xs[(HC + h) * V + j] = CLAMP ? shift_in_down(r, xs[HC * V + V - 1]) : shift_down(r);
                    }
            };
            // stars from radius 2 on: the row's sum and the column's apart, which rounds no worse than the systolic kernels' two
            // chains (radius 6, fp32: 8.5e-8 of the result; in one chain 8.8e-8)
            constexpr int PARTS = STAR && R > 1 ? 2 : 1;
            T sum[PARTS][P][V];
            bool have[PARTS][P];
#pragma unroll
            for (int c = 0; c < PARTS; ++c)
#pragma unroll
                for (int p = 0; p < P; ++p) have[c][p] = false;
            // the wave's own rows first: the others are on their way from LDS
            static_for<P + 2 * R>([&](auto kk) __attribute__((always_inline)) {
                constexpr int i = decltype(kk)::value;
                constexpr int k = i < P ? i + R : i < P + R ? i - P : i;
                const int z = PIN ? opaque_zero() : 0;
                T xs[(2 * HC + 1) * V];
                if constexpr (!STAR || (k >= R && k < R + P)) widen(k, xs);
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    const int n = k - p;
                    if (n < 0 || n >= N) continue;
                    const int c = PARTS == 2 && n != R ? 1 : 0;
#pragma unroll
                    for (int m = 0; m < N; ++m) {
                        if (!Mask::tap(n, m)) continue;
                        const T w = wts[Mask::widx(n, m) + z];
#pragma unroll
                        for (int j = 0; j < V; ++j) {
                            const T x = STAR && n != R ? row(k, j) : xs[HC * V + j + m - R];
                            sum[c][p][j] = have[c][p] ? fma_t(x, w, sum[c][p][j]) : x * w;
                        }
                        have[c][p] = true;
                    }
                }
            });
#pragma unroll
            for (int p = 0; p < P; ++p)
#pragma unroll
                for (int j = 0; j < V; ++j) cur[p][j] = PARTS == 2 ? sum[0][p][j] + sum[PARTS - 1][p][j] : sum[0][p][j];
            offset = buffer - offset;
        }
    };
    if (a.boundary == kClamp) {
        march(std::true_type{});
    } else {
        if (wave == 0) {
            vec_t z;
            if constexpr (V == 1) z = T(0);
            else {
#pragma unroll
                for (int j = 0; j < V; ++j) z[j] = T(0);
            }
            lds[2 * buffer + lane] = z;              // read after the first sweep's barrier
        }
        march(std::false_type{});
    }

#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int y = y0 + row0 + p;
        if (y < ya || y >= yb) continue;
        T* const q = a.out + (size_t)y * W + xc;
        if (xc >= xa && xc + V <= xb) {
            if constexpr (V == 1) *q = cur[p][0];
            else store_vec_elem<T, V, false>(q, cur[p]);
        } else {
#pragma unroll
            for (int j = 0; j < V; ++j)
                if (xc + j >= xa && xc + j < xb) q[j] = cur[p][j];
        }
    }
}

// One compiled kernel.
struct Tile2DKernel {
    const void* kernel;
    int V, index;
};
constexpr int kTileRows = 4;       // rows per wave

// The compiled kernels of a centred stencil of radius R; the list ends with a null one.
template <typename T, bool STAR>
const Tile2DKernel* tile2d_kernels(int R);

constexpr int kTile2DIndexes = 2 * 2 * 6 * 3;
constexpr int tile2d_index(int elem, int V, int R, int budget) { return (((elem / 8) * 2 + budget - 1) * 6 + R - 1) * 3 + V / 2; }
#define SSAM_TILE2D_K(T, V, R, BUDGET)                                                                                                  \
    {reinterpret_cast<const void*>(&ssam2d_tile_kernel<T, V, kTileRows, TapMask<2 * (R) + 1, 2 * (R) + 1, R, R, BUDGET>>), V,           \
     tile2d_index(sizeof(T), V, R, BUDGET)}

struct Tile2DPlan {
    const Tile2DKernel* k = nullptr;
    int waves = 0, sweeps = 0, step_x = 0, step_y = 0, tiles_x = 0, tiles_y = 0;
    double us = 0;                 // expected time of a sweep
};

// Launches some of the remaining sweeps, at most `deepest`, of a centred square stencil (a star or a box of radius pr.ax) on a grid
// small enough for it; returns how many, 0: the grid is left to the other kernels.  kept (may be null): the plan of the launches of one iteration
// while many sweeps remain, which does not depend on their number; empty before the first.
int launch2d_tile(const Problem2D& pr, bool star, int remaining, int deepest, Tile2DPlan* kept, Geometry* geo, bool dry_run, hipError_t* err);

}  // namespace ssam
