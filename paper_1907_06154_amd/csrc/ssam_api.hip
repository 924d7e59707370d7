// C ABI of the library: argument validation, shape classification, dispatch to the compiled
// register-cache instances, the direct fallback kernel for every other shape, Jacobi
// ping-pong, tuning overrides.  All validation happens before the first HIP call.
#include <atomic>
#include <cstdint>
#include <cstring>
#include <string>

#include "ssam_device.h"
#include "ssam_host.h"
#include "ssam_kernel2d_split.h"
#include "ssam_kernel2d_tile.h"
#include "ssam_kernel3d_levels.h"
#include "ssam_kernel3d_split.h"
#include "ssam_kernel_dense.h"

namespace ssam {

std::vector<Instance2D>& registry2d()
{
    static std::vector<Instance2D> r;
    return r;
}
std::vector<Instance3D>& registry3d()
{
    static std::vector<Instance3D> r;
    return r;
}

namespace {

constexpr int kMaxFusedSweeps = 8;
constexpr long long kFuseTwoMinPoints = 1LL << 22;
std::atomic<int> g_rows_per_wave{-1}, g_valid_lanes{-1}, g_planes_per_wave{-1}, g_xcd_remap{-1},
    g_force_generic{-1}, g_variant{-1}, g_march_axis{-1}, g_fuse_sweeps{-1}, g_embed_waste{-1};

Tuning current_tuning()
{
    Tuning t;
    t.rows_per_wave = g_rows_per_wave.load();
    t.valid_lanes = g_valid_lanes.load();
    t.planes_per_wave = g_planes_per_wave.load();
    t.xcd_remap = g_xcd_remap.load();
    t.force_generic = g_force_generic.load();
    t.variant = g_variant.load();
    t.march_axis = g_march_axis.load();
    t.fuse_sweeps = g_fuse_sweeps.load();
    t.embed_waste = g_embed_waste.load();
    return t;
}

// ---- direct fallback kernel -------------------------------------------------------------
// One output point per thread, taps read straight from global memory (cached).  It keeps the
// ABI total: any filter or stencil shape without a compiled register-cache instance runs
// here.  The taps travel in the kernel-argument block as a list of (coefficient, offset) pairs --
// for a stencil only the non-zero ones, so a star of any radius is a short list.  A list too long
// for one argument block is evaluated by several launches on the same stream, the first writing
// the partial sum of its part, every later one adding its own part to what the output holds
// (each thread only ever touches its own output element).
constexpr int kGenericBytes = 3584;

template <typename T>
struct GenericArgs {
    static constexpr int kCap = kGenericBytes / (sizeof(T) + sizeof(int));
    const T* in;
    T* out;
    int W, H, D;
    int boundary;
    int ntaps;         // taps in this launch
    int accumulate;    // 1: add to the value the output already holds
    long long nblocks; // blocks of 64 x 4 points in the grid
    T w[kCap];
    int off[kCap];     // dx, dy, dz as signed bytes 0, 1, 2
};

template <typename T>
__device__ __forceinline__ T fetch(const GenericArgs<T>& a, int x, int y, int z)
{
    if (a.boundary == kClamp) {
        x = min(max(x, 0), a.W - 1);
        y = min(max(y, 0), a.H - 1);
        z = min(max(z, 0), a.D - 1);
    } else if (x < 0 || x >= a.W || y < 0 || y >= a.H || z < 0 || z >= a.D) {
        return T(0);
    }
    return a.in[((size_t)z * a.H + y) * a.W + x];
}

template <typename T>
__global__ __launch_bounds__(256) void generic_kernel(const GenericArgs<T> a)
{
    // blocks of 64 x 4 points, numbered x fastest; the launched blocks stride over them (a tall
    // or deep grid has more of them than one launch dimension takes)
    const long long nbx = (a.W + 63) / 64, nby = (a.H + 3) / 4;
    for (long long b = blockIdx.x; b < a.nblocks; b += gridDim.x) {
        const int x = (int)(b % nbx) * 64 + (threadIdx.x & 63);
        const int y = (int)((b / nbx) % nby) * 4 + (threadIdx.x >> 6);
        const int z = (int)(b / nbx / nby);
        if (x >= a.W || y >= a.H) continue;
        T* o = a.out + ((size_t)z * a.H + y) * a.W + x;
        T sum = a.accumulate ? *o : T(0);
        for (int t = 0; t < a.ntaps; ++t) {
            const int off = a.off[t];
            sum = fma_t(a.w[t], fetch(a, x + (int)(signed char)(off & 0xff), y + (int)(signed char)((off >> 8) & 0xff),
                                      z + (int)(signed char)((off >> 16) & 0xff)), sum);
        }
        *o = sum;
    }
}

// Largest number of simultaneously non-zero offset components among the taps (0..3).
template <typename T>
int tap_budget(const T* c, int M, int N, int K, int ax, int ay, int az)
{
    int b = 0;
    for (int k = 0; k < K; ++k)
        for (int n = 0; n < N; ++n)
            for (int m = 0; m < M; ++m)
                if (c[(k * N + n) * M + m] != T(0)) {
                    const int u = (k != az) + (n != ay) + (m != ax);
                    if (u > b) b = u;
                }
    return b;
}

template <typename T>
hipError_t launch_generic(const T* in, T* out, int W, int H, int D, const T* c, int M, int N, int K, int ax,
                          int ay, int az, int boundary, bool skip_zero, hipStream_t stream)
{
    GenericArgs<T> a;
    a.in = in;
    a.out = out;
    a.W = W; a.H = H; a.D = D;
    a.boundary = boundary;
    a.nblocks = (long long)ceil_div(W, 64) * ceil_div(H, 4) * D;
    const unsigned grid = (unsigned)(a.nblocks < (1LL << 20) ? a.nblocks : (1LL << 20));
    a.ntaps = 0;
    a.accumulate = 0;
    auto flush = [&]() {
        hipLaunchKernelGGL(generic_kernel<T>, dim3(grid), dim3(256), 0, stream, a);
        a.ntaps = 0;
        a.accumulate = 1;
        return hipGetLastError();
    };
    for (int k = 0; k < K; ++k)
        for (int n = 0; n < N; ++n)
            for (int m = 0; m < M; ++m) {
                const T v = c[((size_t)k * N + n) * M + m];
                if (skip_zero && v == T(0)) continue;
                a.w[a.ntaps] = v;
                a.off[a.ntaps] = ((m - ax) & 0xff) | (((n - ay) & 0xff) << 8) | (((k - az) & 0xff) << 16);
                if (++a.ntaps == GenericArgs<T>::kCap)
                    if (hipError_t e = flush()) return e;
            }
    if (a.ntaps > 0 || !a.accumulate)      // the last part; a stencil without any tap still writes zeros
        if (hipError_t e = flush()) return e;
    return hipSuccess;
}

// Whether an fp64 box without zeros goes to the register-tiled kernel instead of the one-point-per-thread one.  That kernel
// issues its multiply-adds up to ten times as fast but needs work to fill the machine with: a lane makes 4 x 4 outputs, in 3D
// of two planes, and a block goes through the filter's planes one after the other, a barrier each.  Ratio of the times,
// register-tiled to direct, from 2100 pairs of shape and grid:
//   one filter plane: 0.05 .. 0.95 from 800000 points on; 512^2: 16x16 0.5, 12x12 0.64, 12x4 0.88, 4x12 1.02, 16x1 1.4, 1x16
//   1.8; 700^2: 12x3 0.77, 2x16 1.07, 1x32 1.2; 64^2 .. 360^2 alike: 24x24 0.6, 16x9 0.76, 9x16 0.9, 16x4 1.0, 3x12 1.6
//   several: 64^3 1.4 (13x9x3) .. 10 (1x1x13); 72^3 9x9x3 0.82, 9x5x3 1.03; 88^3 9x3x3 0.98; 96^3 7x3x3 1.0, 3x3x9 1.5; 128^3
//   3x3x9 0.88, 9x1x3 1.0, 1x9x3 1.1, 2x2x9 1.5; 256^3 3x2x9 0.73, 5x1x9 0.87, 1x5x9 0.89, 2x2x9 1.04, 1x1x9 2.2
bool dense_is_faster(long points, int M, int N, int K)
{
    const long plane = (long)M * N;      // taps of a filter plane
    if (plane * K < 9) return false;
    if (K == 1)
        return points >= 800000 || (points >= 450000 && M >= 3) || (M >= 4 && points * plane >= 13000000) || (M >= 9 && plane >= 100);
    if (points < 350000 || (M == 1 && points < 6000000)) return false;
    return (plane >= 9 && points * plane >= 18500000) || (plane >= 5 && points * plane >= 70000000);
}

// What no compiled shape takes.  fp64 boxes without a zero (or whose zeros are taps) run on the register-tiled kernel where it
// is the faster one; sparse tap lists and fp32 on the one-point-per-thread kernel.
hipError_t launch_direct(const void* in, void* out, int W, int H, int D, const void* c, int M, int N, int K, int ax, int ay, int az,
                         int boundary, bool skip_zero, int dtype, hipStream_t stream, const Tuning& tu, Geometry* geo, bool dry)
{
    if (dtype == SSAM_F64) {
        const double* w = static_cast<const double*>(c);
        bool dense = tu.force_generic == 2 || (tu.force_generic <= 0 && dense_is_faster((long)W * H * D, M, N, K));
        for (long i = 0; dense && skip_zero && i < (long)M * N * K; ++i) dense = w[i] != 0.0;
        if (dense) {
            const hipError_t e = launch_dense((const double*)in, (double*)out, W, H, D, w, M, N, K, ax, ay, az, boundary, stream, geo, dry);
            if (e != hipErrorNotSupported) return e;
        }
    }
    if (geo) {
        *geo = Geometry();
        geo->blocks = ceil_div(W, 64) * ceil_div(H, 4) * D;
    }
    if (dry) return hipSuccess;
    if (dtype == SSAM_F32)
        return launch_generic<float>((const float*)in, (float*)out, W, H, D, (const float*)c, M, N, K, ax, ay, az, boundary, skip_zero,
                                     stream);
    return launch_generic<double>((const double*)in, (double*)out, W, H, D, (const double*)c, M, N, K, ax, ay, az, boundary, skip_zero,
                                  stream);
}

// ---- plain copy (measurement aid) ---------------------------------------------------------
// 16 bytes per lane, grid-stride: a reference rate for 1-read-1-write kernels (tile-shaped
// access with streaming stores exceeds it), and the known-size reference the hardware traffic
// counters are scaled by.
__global__ __launch_bounds__(256) void copy_kernel(const uint4* __restrict__ in, uint4* __restrict__ out, size_t n16)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride) out[i] = in[i];
}

// ---- validation helpers ------------------------------------------------------------------
int check_enums(int boundary, int dtype)
{
    if (boundary != SSAM_BOUNDARY_ZERO && boundary != SSAM_BOUNDARY_CLAMP) return SSAM_ERR_ENUM;
    if (dtype != SSAM_F32 && dtype != SSAM_F64) return SSAM_ERR_ENUM;
    return SSAM_OK;
}

int check_dims(int W, int H, int D)
{
    if (W <= 0 || H <= 0 || D <= 0) return SSAM_ERR_DIM;
    if (W > SSAM_MAX_EXTENT || H > SSAM_MAX_EXTENT || D > SSAM_MAX_EXTENT) return SSAM_ERR_DIM;
    if ((long long)W * H * D > 2147483647LL) return SSAM_ERR_DIM;
    return SSAM_OK;
}

bool overlap(const void* a, const void* b, size_t bytes)
{
    const uintptr_t pa = (uintptr_t)a, pb = (uintptr_t)b;
    return pa < pb + bytes && pb < pa + bytes;
}

size_t elem(int dtype) { return dtype == SSAM_F32 ? 4 : 8; }

// A launcher reports a tile plan that no launch can hold (more blocks than a grid dimension takes:
// grids of extreme aspect ratio) as hipErrorInvalidConfiguration, before it launches anything.
int status_of(hipError_t e)
{
    return e == hipSuccess ? SSAM_OK : e == hipErrorInvalidConfiguration ? SSAM_ERR_DIM : SSAM_ERR_HIP;
}

// ---- dispatch ---------------------------------------------------------------------------
template <typename T>
const Instance2D* pick2d(const Problem2D& p, bool stencil_semantics, int want_variant, int sweeps = 1,
                         bool any_depth = false)
{
    const T* w = static_cast<const T*>(p.w);
    int budget = 2;
    if (stencil_semantics) {
        budget = tap_budget<T>(w, p.M, p.N, 1, p.ax, p.ay, 0);
        if (budget == 0) budget = 1;
    }
    const Instance2D* best = nullptr;
    for (const Instance2D& i : registry2d()) {
        if (i.dtype != p.dtype || i.M != p.M || i.N != p.N || i.AX != p.ax) continue;
        if (i.budget < budget) continue;
        if (i.budget == 1 && p.ay != p.N / 2) continue;   // star instances assume the centre row
        if (i.variant != want_variant) continue;
        if (any_depth ? i.sweeps < 2 : i.sweeps != sweeps) continue;
        if (!best || i.budget < best->budget) best = &i;
    }
    return best;
}

// Whether a dense fp32 filter goes to the bf16 matrix-core kernel instead of `inst` (its own instance), `box` (the square box
// it would run in) or, with neither, the direct kernel.  That kernel's time hardly depends on the shape below 9x9 (8192^2:
// 138-147 us for 6x6 .. 9x9), so the line lies where the other instances reach it: boxes up to 6x6 and the flat shapes with
// instances of their own (3x11, 11x3, 1 x n) stay bandwidth-bound on the vector unit (104 us at 6x6); 7x7 takes 127 us
// there and is only faster here on smaller pictures (1024^2: 11.2 -> 8.9 us, 4096^2: 36.7 and 39.4) and on rows that are
// not whole 16-byte pieces (4003x3001: 44.3 -> 32.5); from 8x8 on (145 us, equal) it is faster on large pictures.  On small ones
// the box instances with short tiles are faster (9x9 on 700^2 5.8 us against 8.5, on 1500^2 12.2 against 14.2) but three times as
// far from 64-bit sums, so the line stays.  Pictures of a few tiles gain nothing, and a strip narrower than a wave's 64 columns
// would be mostly empty.  Of a filter one or two columns wide a piece of eight is mostly zeros: beyond the boxes (more than 20
// rows) the direct kernel keeps it on small pictures (1x32: 130^2 12 us against 16, 512^2 10.5 and 15.5, 700^2 14.9 and 18.6;
// 2x24: 256^2 12 and 21, 512^2 equal).
bool split_is_faster(const Problem2D& p, const Instance2D* inst, const Instance2D* box, const Tuning& tu)
{
    const long points = (long)p.W * p.H;
    if (p.dtype != SSAM_F32 || tu.force_generic > 0 || tu.variant >= 0 || tu.embed_waste >= 0) return false;
    if (points < 16384 || p.W < 64) return false;
    if (inst && (inst->budget != 2 || inst->M < 7 || inst->N < 7)) return false;
    if (!inst && !box && (p.M == 1 ? points < 1000000 : p.M == 2 && points < 150000)) return false;
    const int edge = inst ? inst->M : box ? box->M : SSAM_MAX_FILTER;
    if (edge == 7) return p.W % 4 != 0 || points < (4L << 20);
    return edge > 7;
}

int run2d(const Problem2D& p, bool stencil_semantics, Geometry* geo, bool dry, std::string* name)
{
    const Tuning tu = current_tuning();
    const Instance2D* inst = nullptr;
    if (tu.force_generic <= 0)
    {
        const int v = tu.variant > 0 ? tu.variant : 0;
        inst = p.dtype == SSAM_F32 ? pick2d<float>(p, stencil_semantics, v) : pick2d<double>(p, stencil_semantics, v);
        if (!inst && v != 0)   // no such alternative for this shape: use the default instance
            inst = p.dtype == SSAM_F32 ? pick2d<float>(p, stencil_semantics, 0) : pick2d<double>(p, stencil_semantics, 0);
    }
    // No instance of this exact shape (a non-square filter, an anchor off the centre, unequal
    // radii): embed it in the smallest compiled square box whose centre anchor leaves enough room
    // on every side.  The added zero weights cost arithmetic, but even a 1x20 filter inside the 20x20
    // box measured faster than the direct kernel, so there is no limit unless "embed_waste" sets one.
    const Instance2D* box = nullptr;
    if (!inst && tu.force_generic <= 0) {
        const int need_lo = p.ax > p.ay ? p.ax : p.ay;
        const int hi_x = p.M - 1 - p.ax, hi_y = p.N - 1 - p.ay;
        const int need_hi = hi_x > hi_y ? hi_x : hi_y;
        for (const Instance2D& i : registry2d()) {
            if (i.dtype != p.dtype || i.M != i.N || i.budget != 2 || i.variant != 0 || i.sweeps != 1) continue;
            if (i.AX != i.M / 2 || i.M / 2 < need_lo || i.M - 1 - i.M / 2 < need_hi) continue;
            if (!box || i.M < box->M) box = &i;
        }
        if (box && tu.embed_waste >= 0 && box->M * box->N > tu.embed_waste * p.M * p.N) box = nullptr;
    }
    if (split_is_faster(p, inst, box, tu)) {
        const hipError_t e = launch2d_split(p, tu, geo, dry);
        if (e != hipErrorNotSupported) {
            if (name) *name = "float_M" + std::to_string(p.M) + "N" + std::to_string(p.N) + "_b2_v4p4split3mx";
            return status_of(e);
        }
    }
    if (inst) {
        if (name) *name = inst->name;
        return status_of(inst->launch(p, tu, geo, dry));
    }
    if (box) {
        const int K = box->M, c = K / 2;
        const size_t es = elem(p.dtype);
        std::vector<char> padded((size_t)K * K * es, 0);
        const char* src = static_cast<const char*>(p.w);
        for (int n = 0; n < p.N; ++n)
            memcpy(&padded[((size_t)(n + c - p.ay) * K + (c - p.ax)) * es], src + (size_t)n * p.M * es, (size_t)p.M * es);
        Problem2D q = p;
        q.M = q.N = K;
        q.ax = q.ay = c;
        q.w = padded.data();
        if (name) *name = std::string(box->name) + "+embedded";
        return status_of(box->launch(q, tu, geo, dry));   // weights are copied into the launch arguments
    }
    if (name) *name = "generic_direct";
    return status_of(launch_direct(p.in, p.out, p.W, p.H, 1, p.w, p.M, p.N, 1, p.ax, p.ay, 0, p.boundary, stencil_semantics, p.dtype,
                                   p.stream, tu, geo, dry));
}

template <typename T>
const Instance3D* pick3d(const Problem3D& p, int want_variant, int sweeps = 1)
{
    const T* c = static_cast<const T*>(p.c);
    int budget = p.dense ? 3 : tap_budget<T>(c, 2 * p.rx + 1, 2 * p.ry + 1, 2 * p.rz + 1, p.rx, p.ry, p.rz);
    if (budget == 0) budget = 1;
    // an instance is compiled for (reach along x, along the strip axis, along the march axis)
    const int strip_r = p.march_y ? p.rz : p.ry, march_r = p.march_y ? p.ry : p.rz;
    const Instance3D* best = nullptr;
    for (const Instance3D& i : registry3d()) {
        if (i.dtype != p.dtype || i.rx != p.rx || i.ry != strip_r || i.rz != march_r || i.budget < budget) continue;
        if (i.variant != want_variant || i.sweeps != sweeps) continue;
        if (!best || i.budget < best->budget) best = &i;
    }
    return best;
}

// Sweeps of the next launch while `remaining` are to do: the smallest of the depths with which, the deepest that fits first, the rest
// takes the fewest launches.  (Without the depth of two, on small grids, a smaller depth can take fewer: six as 3 + 3, not 4 + 1 + 1.)  A launch's time grows with its depth at least in proportion beyond the deepest
// one that is bound by memory, so equal depths are the better split: 8192^2, us, deepest first and like this: nine sweeps of the fp64
// box of radius 1 459 -> 436 (8 + 1, 6 + 3), eighteen under the clamp rule 925 -> 759; eight of the fp32 box 264 -> 222 (6 + 2, 4 + 4);
// five of the fp64 box of radius 2 550 -> 501 (4 + 1, 3 + 2), of the fp32 star of radius 3 on 2048x2176 41 -> 32.
// keep_single: up to this depth a launch is bound by memory and one sweep left over is cheaper than a share of it (five sweeps of the
// fp64 star of radius 1 on 8192^2: 395 as 4 + 1, 411 as 3 + 2; seven 400 as 6 + 1, 420 as 4 + 3;
// nine of the star of radius 2 under the clamp rule 661 as 4 + 4 + 1, 687 as 3 + 3 + 3; seven of the fp32 star of radius 1 with zero
// padding on 3239x7168 84 as 6 + 1, 92 as 4 + 3).
int fused_depth(int remaining, int deepest, int keep_single, const Instance2D* const* by_depth)
{
    while (deepest >= 2 && !by_depth[deepest]) --deepest;
    if (deepest < 2 || remaining > 4 * kMaxFusedSweeps || (remaining % deepest == 1 && deepest <= keep_single)) return deepest;
    auto launches = [&](int most) {
        int n = remaining, count = 0;
        for (; n > 0; ++count) {
            int d = n < most ? n : most;
            while (d > 1 && !by_depth[d]) --d;
            n -= d;
        }
        return count;
    };
    int best = deepest, fewest = launches(deepest);
    for (int d = deepest - 1; d > 1; --d)
        if (by_depth[d] && launches(d) <= fewest) best = d, fewest = launches(d);
    return best;
}

// Several sweeps in one launch, where the shape has a fused instance (3D only when marching along z): in 3D the deepest compiled
// one that does not exceed `remaining` (the sweeps still to do) nor the "fuse_sweeps" cap, in 2D see fused_depth.  Returns the
// number of sweeps the launch performs, 0 when the caller should run a single sweep instead.  kept: see launch2d_tile.
int run_fused(const Problem3D& p, int remaining, Geometry* geo, bool dry, std::string* name, int* rc, Tile2DPlan* kept = nullptr)
{
    const Tuning tu = current_tuning();
    if (tu.fuse_sweeps == 0 || tu.fuse_sweeps == 1 || tu.force_generic > 0) return 0;
    const int cap = tu.fuse_sweeps > 1 && tu.fuse_sweeps < remaining ? tu.fuse_sweeps : remaining;     // sweeps of one launch
    const int v = tu.variant > 0 ? tu.variant : 0;
    const bool flat = p.D == 1 && p.rz == 0;
    if (!flat && tu.march_axis == 1) return 0;   // 3D: z march only
    // Two sweeps per launch pay only on grids large enough to be bandwidth-bound (measured: from about
    // 4M points); on smaller ones the fatter, fewer tiles lose more than the saved launch gains.  Three
    // sweeps and more per launch were faster at every size tried (256^2 upwards).
    const bool small = (long long)p.W * p.H * p.D < kFuseTwoMinPoints && tu.fuse_sweeps < 0;
    Problem2D q{p.in, p.out, p.W, p.H, p.c, 2 * p.rx + 1, 2 * p.ry + 1, p.rx, p.ry, p.boundary, p.dtype, p.stream};
    // small grids: the kernel that keeps whole tiles in registers (the tile overrides and variants are the marching kernels')
    if (flat && p.rx == p.ry && tu.rows_per_wave <= 0 && tu.valid_lanes <= 0 && tu.variant < 0) {
        const int budget = p.dtype == SSAM_F32 ? tap_budget<float>((const float*)p.c, q.M, q.N, 1, q.ax, q.ay, 0)
                                               : tap_budget<double>((const double*)p.c, q.M, q.N, 1, q.ax, q.ay, 0);
        hipError_t e = hipSuccess;
        if (const int sweeps = launch2d_tile(q, budget <= 1, remaining, cap, kept, geo, dry, &e)) {
            if (name)
                *name = std::string(p.dtype == SSAM_F32 ? "float" : "double") + "_R" + std::to_string(p.rx) + (budget <= 1 ? "_b1" : "_b2") +
                        "_tile_fused" + std::to_string(sweeps);
            *rc = status_of(e);
            return sweeps;
        }
    }
    if (!flat && p.rx == 1 && p.ry == 1 && p.rz == 1 && tu.planes_per_wave <= 0 && tu.valid_lanes <= 0 && tu.variant < 0) {     // sweeps as levels of one march (the overrides are the other kernels')
        const int budget = p.dtype == SSAM_F32 ? tap_budget<float>((const float*)p.c, 3, 3, 3, 1, 1, 1) : tap_budget<double>((const double*)p.c, 3, 3, 3, 1, 1, 1);
        hipError_t e = hipSuccess;
        if (const int sweeps = launch3d_levels(p, budget, remaining, cap, geo, dry, &e)) {
            if (name)
                *name = std::string(p.dtype == SSAM_F32 ? "float" : "double") + "_r111_b" + std::to_string(budget < 1 ? 1 : budget) + "_levels_fused" + std::to_string(sweeps);
            *rc = status_of(e);
            return sweeps;
        }
    }
    const int deepest = cap < kMaxFusedSweeps ? cap : kMaxFusedSweeps;
    if (flat) {
        const Instance2D* tight = p.dtype == SSAM_F32 ? pick2d<float>(q, true, 0, 0, true) : pick2d<double>(q, true, 0, 0, true);
        if (!tight) return 0;
        // of the tightest tap shape any multi-sweep instance offers for this stencil: a deeper instance of a
        // wider shape (a box standing in for a star) is not taken over a shallower one of the exact shape
        const Instance2D* by_depth[kMaxFusedSweeps + 1] = {};
        for (int sweeps = small ? 3 : 2; sweeps <= deepest; ++sweeps)
            for (int variant : {v, 0}) {
                const Instance2D* inst = p.dtype == SSAM_F32 ? pick2d<float>(q, true, variant, sweeps) : pick2d<double>(q, true, variant, sweeps);
                if (!inst || inst->budget != tight->budget || by_depth[sweeps]) continue;
                if ((long)p.W * p.H >= 1000000L * (p.boundary == SSAM_BOUNDARY_CLAMP ? inst->clamp_from : inst->zero_from)) by_depth[sweeps] = inst;
            }
        const bool star = tight->budget == 1;
        const int keep_single = p.dtype == SSAM_F32 ? (p.rx != 1 ? 0 : star && p.boundary == SSAM_BOUNDARY_ZERO ? 6 : 4) : p.rx == 1 ? 6 : star && p.rx == 2 ? 4 : 0;
        const int sweeps = fused_depth(remaining, deepest, keep_single, by_depth);
        if (sweeps < 2) return 0;
        if (name) *name = by_depth[sweeps]->name;
        *rc = status_of(by_depth[sweeps]->launch(q, tu, geo, dry));
        return sweeps;
    }
    for (int sweeps = deepest; sweeps >= 2; --sweeps) {
        if (sweeps == 2 && small) break;
        const Instance3D* inst = p.dtype == SSAM_F32 ? pick3d<float>(p, v, sweeps) : pick3d<double>(p, v, sweeps);
        if (!inst && v != 0) inst = p.dtype == SSAM_F32 ? pick3d<float>(p, 0, sweeps) : pick3d<double>(p, 0, sweeps);
        if (!inst || (p.boundary == SSAM_BOUNDARY_CLAMP && !inst->fuses_clamp)) continue;
        if (name) *name = inst->name;
        const hipError_t e = inst->launch(p, tu, geo, dry);
        *rc = status_of(e);
        return sweeps;
    }
    return 0;
}

// Whether a dense fp32 3D box of these extents goes to the bf16 matrix-core kernel.  compiled: the vector-unit box instance it
// would run in has radius R (0: none, it would run on the direct kernel).  Radius 1 is bandwidth-bound there (3x3x3 on 512^3:
// 199 us); from radius 2 on that kernel is faster at every size measured (5x5x5: 64^3 56 -> 17 us, 512^3 576 -> 400; 7x7x7: 199
// -> 24, 1580 -> 1090).  The direct kernel keeps what is too little work to fill the machine (64^3 with 80 .. 150 taps: 20 .. 32
// us there, 25 .. 33 here); rows of less than half a wave's 64 columns and very small grids stay where they were.
bool split3d_is_faster(int W, int H, int D, int M, int N, int K, int compiled, const Tuning& tu)
{
    const long points = (long)W * H * D;
    if (tu.force_generic > 0 || tu.variant >= 0 || tu.embed_waste >= 0 || tu.march_axis == 1) return false;
    if (points < 65536 || W < 32 || compiled == 1) return false;
    return compiled >= 2 || (double)points * M * N * K > 5e7;
}

std::string split3d_name(int M, int N, int K)
{
    if (M == N && N == K && M % 2 == 1) {
        const std::string r = std::to_string(M / 2);
        return "float_r" + r + r + r + "_b3_split3mx";
    }
    return "float_M" + std::to_string(M) + "N" + std::to_string(N) + "K" + std::to_string(K) + "_b3_split3mx";
}

int run3d(const Problem3D& p_in, Geometry* geo, bool dry, std::string* name)
{
    const Tuning tu = current_tuning();
    Problem3D p = p_in;
    p.march_y = tu.march_axis == 1;
    if (p.D == 1 && p.rz == 0) {   // a 2D problem through the 3D door
        Problem2D q{p.in, p.out, p.W, p.H, p.c, 2 * p.rx + 1, 2 * p.ry + 1, p.rx, p.ry, p.boundary, p.dtype, p.stream};
        return run2d(q, true, geo, dry, name);
    }
    // Taps a compiled shape evaluates: what a launch costs in arithmetic.
    auto taps = [](const Instance3D& i) {
        const long n = 2 * i.rx + 1;
        return i.budget == 1 ? 6L * i.rx + 1 : i.budget == 2 ? n * n * n - 8L * i.rx * i.rx * i.rx : n * n * n;
    };
    const Instance3D* inst = nullptr;   // an instance of exactly these radii
    const Instance3D* cube = nullptr;   // the cheapest compiled shape of equal radii that covers the box, zero-padded
    if (tu.force_generic <= 0) {
        const int v = tu.variant > 0 ? tu.variant : 0;
        inst = p.dtype == SSAM_F32 ? pick3d<float>(p, v) : pick3d<double>(p, v);
        if (!inst && v != 0) inst = p.dtype == SSAM_F32 ? pick3d<float>(p, 0) : pick3d<double>(p, 0);
        if (tu.embed_waste != 0) {
            const int budget = p.dense ? 3 : p.dtype == SSAM_F32
                                   ? tap_budget<float>((const float*)p.c, 2 * p.rx + 1, 2 * p.ry + 1, 2 * p.rz + 1, p.rx, p.ry, p.rz)
                                   : tap_budget<double>((const double*)p.c, 2 * p.rx + 1, 2 * p.ry + 1, 2 * p.rz + 1, p.rx, p.ry, p.rz);
            const int need = p.rx > p.ry ? (p.rx > p.rz ? p.rx : p.rz) : (p.ry > p.rz ? p.ry : p.rz);
            for (const Instance3D& i : registry3d()) {
                if (i.dtype != p.dtype || i.rx != i.ry || i.ry != i.rz || i.rx < need || i.budget < budget) continue;
                if (i.variant != 0 || i.sweeps != 1) continue;
                if (!cube || taps(i) < taps(*cube)) cube = &i;
            }
        }
    }
    // The exact instance unless a padded one evaluates fewer taps (a radius-3 star has no instance of
    // its own: the radius-4 star, 25 taps, beats the radius-3 box, 343); whichever is tried first, a
    // launcher that does not take this grid (hipErrorNotSupported) leaves the turn to the other.
    const bool cube_first = cube && cube != inst && (!inst || taps(*cube) < taps(*inst));
    const Instance3D* first = cube_first ? cube : inst;
    if (p.dtype == SSAM_F32 && first && first->budget == 3 &&
        split3d_is_faster(p.W, p.H, p.D, 2 * p.rx + 1, 2 * p.ry + 1, 2 * p.rz + 1, first->rx, tu)) {
        const hipError_t e = launch3d_split((const float*)p.in, (float*)p.out, p.W, p.H, p.D, (const float*)p.c, 2 * p.rx + 1,
                                            2 * p.ry + 1, 2 * p.rz + 1, p.rx, p.ry, p.rz, p.boundary, p.stream, tu, geo, dry);
        if (e != hipErrorNotSupported) {
            if (name) *name = split3d_name(2 * p.rx + 1, 2 * p.ry + 1, 2 * p.rz + 1) + (cube_first ? "+embedded" : "");
            return status_of(e);
        }
    }
    for (int attempt = 0; attempt < 2; ++attempt) {
        const bool use_cube = (attempt == 0) == cube_first;
        if (!use_cube && inst) {
            if (name) *name = inst->name;
            const hipError_t e = inst->launch(p, tu, geo, dry);
            if (e != hipErrorNotSupported) return status_of(e);
        }
        if (use_cube && cube && cube != inst) {
            const int R = cube->rx, K = 2 * R + 1;
            const int M = 2 * p.rx + 1, N = 2 * p.ry + 1, L = 2 * p.rz + 1;
            const size_t es = elem(p.dtype);
            std::vector<char> padded((size_t)K * K * K * es, 0);
            const char* src = static_cast<const char*>(p.c);
            for (int k = 0; k < L; ++k)
                for (int n = 0; n < N; ++n)
                    memcpy(&padded[((((size_t)(k + R - p.rz) * K) + (n + R - p.ry)) * K + (R - p.rx)) * es],
                           src + ((size_t)k * N + n) * M * es, (size_t)M * es);
            Problem3D q = p;
            q.rx = q.ry = q.rz = R;
            q.c = padded.data();
            if (name) *name = std::string(cube->name) + "+embedded";
            const hipError_t e = cube->launch(q, tu, geo, dry);   // the coefficients are copied into the launch arguments
            if (e != hipErrorNotSupported) return status_of(e);
        }
    }
    if (name) *name = "generic_direct";
    return status_of(launch_direct(p.in, p.out, p.W, p.H, p.D, p.c, 2 * p.rx + 1, 2 * p.ry + 1, 2 * p.rz + 1, p.rx, p.ry, p.rz,
                                   p.boundary, !p.dense, p.dtype, p.stream, tu, geo, dry));
}

// 3D filter of extents (M, N, K) anchored at (ax, ay, az).  A cube of odd extent anchored at its
// centre is the dense coefficient box of a stencil and runs on the compiled box instances (radius 1, 2, 3);
// any other filter that fits such a cube around its anchor runs zero-padded inside the smallest one
// (as 2D filters without an instance of their own do); the rest runs on the direct kernel, which
// takes extents and anchor as they are.
int run_conv3d(const void* in, void* out, int W, int H, int D, const void* f, int M, int N, int K, int ax, int ay,
               int az, int boundary, int dtype, hipStream_t stream, Geometry* geo, bool dry, std::string* name)
{
    const Tuning tu = current_tuning();
    const int lo = ax > ay ? (ax > az ? ax : az) : (ay > az ? ay : az);
    const int hx = M - 1 - ax, hy = N - 1 - ay, hz = K - 1 - az;
    const int hi = hx > hy ? (hx > hz ? hx : hz) : (hy > hz ? hy : hz);
    const int R = lo > hi ? lo : hi;
    const size_t es = elem(dtype);
    // zero padding costs arithmetic: a cube with more than 8 times the filter's taps (or the "embed_waste"
    // override) is left to the direct kernel
    const long waste = tu.embed_waste > 0 ? tu.embed_waste : 8;
    bool cube = R >= 1 && R <= 3 && tu.force_generic <= 0 && tu.embed_waste != 0 &&
                (long)(2 * R + 1) * (2 * R + 1) * (2 * R + 1) <= waste * M * N * K;
    // fp64: the radius-3 cube costs 343 taps whatever it holds and is slow on small grids; the kernels of launch_direct are
    // faster for fewer taps (5x6x4 on 256^3: 561 -> 447 us) and, for the full cube, on grids of up to a few million points
    // (64^3: 264 -> 84; 256^3: 561 and 791)
    if (dtype == SSAM_F64 && R == 3 && tu.variant < 0 && tu.embed_waste < 0 && ((long)M * N * K < 200 || (long)W * H * D < (4L << 20)))
        cube = false;
    if (dtype == SSAM_F32 && split3d_is_faster(W, H, D, M, N, K, cube ? R : 0, tu)) {
        const hipError_t e = launch3d_split((const float*)in, (float*)out, W, H, D, (const float*)f, M, N, K, ax, ay, az, boundary,
                                            stream, tu, geo, dry);
        if (e != hipErrorNotSupported) {
            if (name) *name = split3d_name(M, N, K);
            return status_of(e);
        }
    }
    if (cube) {
        const int S = 2 * R + 1;
        std::vector<char> padded((size_t)S * S * S * es, 0);
        const char* src = static_cast<const char*>(f);
        for (int k = 0; k < K; ++k)
            for (int n = 0; n < N; ++n)
                memcpy(&padded[((((size_t)(k - az + R) * S) + (n - ay + R)) * S + (R - ax)) * es],
                       src + ((size_t)k * N + n) * M * es, (size_t)M * es);
        Problem3D p{in, out, W, H, D, padded.data(), R, R, R, boundary, dtype, stream};
        p.dense = true;
        std::string inner;
        const int rc = run3d(p, geo, dry, &inner);
        if (inner != "generic_direct") {     // a compiled instance took it (the coefficients are copied into the launch arguments)
            if (name) *name = (M == S && N == S && K == S) ? inner : inner + "+embedded";
            return rc;
        }
    }
    if (name) *name = "generic_direct";
    return status_of(launch_direct(in, out, W, H, D, f, M, N, K, ax, ay, az, boundary, false, dtype, stream, tu, geo, dry));
}

// Everything but the grid pointers (the planning query has none).
int check_conv3d(int W, int H, int D, const void* f, int M, int N, int K, int* ax, int* ay, int* az, int boundary,
                 int dtype)
{
    if (!f) return SSAM_ERR_NULL;
    if (int e = check_enums(boundary, dtype)) return e;
    if (int e = check_dims(W, H, D)) return e;
    if (M <= 0 || N <= 0 || K <= 0 || M > SSAM_MAX_FILTER3D || N > SSAM_MAX_FILTER3D || K > SSAM_MAX_FILTER3D)
        return SSAM_ERR_SHAPE;
    if (*ax == -1) *ax = M / 2;
    if (*ay == -1) *ay = N / 2;
    if (*az == -1) *az = K / 2;
    if (*ax < 0 || *ax >= M || *ay < 0 || *ay >= N || *az < 0 || *az >= K) return SSAM_ERR_SHAPE;
    return SSAM_OK;
}

int validate_conv(const void* in, const void* out, int W, int H, const void* f, int M, int N, int* ax, int* ay,
                  int boundary, int dtype)
{
    if (!in || !out || !f) return SSAM_ERR_NULL;
    if (int e = check_enums(boundary, dtype)) return e;
    if (int e = check_dims(W, H, 1)) return e;
    if (M <= 0 || N <= 0 || M > SSAM_MAX_FILTER || N > SSAM_MAX_FILTER) return SSAM_ERR_SHAPE;
    if (*ax == -1) *ax = M / 2;
    if (*ay == -1) *ay = N / 2;
    if (*ax < 0 || *ax >= M || *ay < 0 || *ay >= N) return SSAM_ERR_SHAPE;
    if (overlap(in, out, (size_t)W * H * elem(dtype))) return SSAM_ERR_ALIAS;
    return SSAM_OK;
}

int validate_stencil(const void* in, const void* out, int W, int H, int D, const void* c, int rx, int ry, int rz,
                     int boundary, int dtype)
{
    if (!in || !out || !c) return SSAM_ERR_NULL;
    if (int e = check_enums(boundary, dtype)) return e;
    if (int e = check_dims(W, H, D)) return e;
    if (rx < 0 || ry < 0 || rz < 0 || rx > SSAM_MAX_RADIUS || ry > SSAM_MAX_RADIUS || rz > SSAM_MAX_RADIUS)
        return SSAM_ERR_SHAPE;
    if (overlap(in, out, (size_t)W * H * D * elem(dtype))) return SSAM_ERR_ALIAS;
    return SSAM_OK;
}

int describe(int rc, const std::string& name, const Geometry& g, char* buf, int buflen)
{
    if (buf && buflen > 0) {
        snprintf(buf, (size_t)buflen,
                 "%s V=%d P=%d halo_lanes=%d+%d valid_lanes=%d strips_x=%d tiles_y=%d tiles_z=%d rows_per_wave=%d "
                 "planes_per_wave=%d tiles=%ld blocks=%d xcd_remap=%d lds=%d form=%d",
                 name.c_str(), g.V, g.P, g.halo_left, g.halo_right, g.valid_lanes, g.strips_x, g.tiles_y, g.tiles_z,
                 g.rows_per_wave, g.planes_per_wave, g.tiles, g.blocks, g.xcd_remap, g.lds, g.form);
    }
    return rc;
}

}  // namespace
}  // namespace ssam

using namespace ssam;

extern "C" {

int ssam_conv2d(const void* d_in, void* d_out, int W, int H, const void* h_filter, int M, int N, int ax, int ay,
                int boundary, int dtype, void* hip_stream)
{
    if (int e = validate_conv(d_in, d_out, W, H, h_filter, M, N, &ax, &ay, boundary, dtype)) return e;
    Problem2D p{d_in, d_out, W, H, h_filter, M, N, ax, ay, boundary, dtype, (hipStream_t)hip_stream};
    return run2d(p, false, nullptr, false, nullptr);
}

int ssam_stencil2d(const void* d_in, void* d_out, int W, int H, const void* h_coef, int rx, int ry, int boundary,
                   int dtype, void* hip_stream)
{
    if (int e = validate_stencil(d_in, d_out, W, H, 1, h_coef, rx, ry, 0, boundary, dtype)) return e;
    Problem2D p{d_in, d_out, W, H, h_coef, 2 * rx + 1, 2 * ry + 1, rx, ry, boundary, dtype, (hipStream_t)hip_stream};
    return run2d(p, true, nullptr, false, nullptr);
}

int ssam_stencil3d(const void* d_in, void* d_out, int W, int H, int D, const void* h_coef, int rx, int ry, int rz,
                   int boundary, int dtype, void* hip_stream)
{
    if (int e = validate_stencil(d_in, d_out, W, H, D, h_coef, rx, ry, rz, boundary, dtype)) return e;
    Problem3D p{d_in, d_out, W, H, D, h_coef, rx, ry, rz, boundary, dtype, (hipStream_t)hip_stream};
    return run3d(p, nullptr, false, nullptr);
}

int ssam_conv3d(const void* d_in, void* d_out, int W, int H, int D, const void* h_filter, int M, int N, int K, int ax,
                int ay, int az, int boundary, int dtype, void* hip_stream)
{
    if (!d_in || !d_out) return SSAM_ERR_NULL;
    if (int e = check_conv3d(W, H, D, h_filter, M, N, K, &ax, &ay, &az, boundary, dtype)) return e;
    if (overlap(d_in, d_out, (size_t)W * H * D * elem(dtype))) return SSAM_ERR_ALIAS;
    return run_conv3d(d_in, d_out, W, H, D, h_filter, M, N, K, ax, ay, az, boundary, dtype, (hipStream_t)hip_stream,
                      nullptr, false, nullptr);
}

int ssam_stencil_iterate(void* d_a, void* d_b, int W, int H, int D, const void* h_coef, int rx, int ry, int rz,
                         int boundary, int dtype, int steps, void* hip_stream, void** d_result)
{
    if (int e = validate_stencil(d_a, d_b, W, H, D, h_coef, rx, ry, rz, boundary, dtype)) return e;
    if (steps < 0) return SSAM_ERR_SHAPE;
    void* src = d_a;
    void* dst = d_b;
    const bool cached = steps > 1 && 2 * (size_t)W * H * D * (dtype == SSAM_F32 ? 4 : 8) <= (size_t)192 << 20;   // of 256 MiB
    Tile2DPlan kept;
    for (int t = 0; t < steps;) {
        Problem3D p{src, dst, W, H, D, h_coef, rx, ry, rz, boundary, dtype, (hipStream_t)hip_stream};
        p.reread = cached;
        int rc = SSAM_OK;
        if (const int fused = run_fused(p, steps - t, nullptr, false, nullptr, &rc, &kept)) {
            if (rc) return rc;
            t += fused;
        } else {
            if (int e = run3d(p, nullptr, false, nullptr)) return e;
            t += 1;
        }
        void* tmp = src;
        src = dst;
        dst = tmp;
    }
    if (d_result) *d_result = src;
    return SSAM_OK;
}

int ssam_probe_copy(const void* d_in, void* d_out, size_t nbytes, void* hip_stream)
{
    if (!d_in || !d_out) return SSAM_ERR_NULL;
    if (nbytes == 0 || nbytes % 16 != 0 || ((uintptr_t)d_in % 16) || ((uintptr_t)d_out % 16)) return SSAM_ERR_DIM;
    if (overlap(d_in, d_out, nbytes)) return SSAM_ERR_ALIAS;
    const size_t n16 = nbytes / 16;
    size_t blocks = (n16 + 255) / 256;
    if (blocks > 256 * 64) blocks = 256 * 64;
    hipLaunchKernelGGL(copy_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)hip_stream,
                       static_cast<const uint4*>(d_in), static_cast<uint4*>(d_out), n16);
    return hipGetLastError() == hipSuccess ? SSAM_OK : SSAM_ERR_HIP;
}

const char* ssam_status_string(int status)
{
    switch (status) {
        case SSAM_OK: return "ok";
        case SSAM_ERR_NULL: return "null pointer argument";
        case SSAM_ERR_DIM: return "size out of range (grid dimension, element count), misaligned pointer or workspace too small";
        case SSAM_ERR_SHAPE: return "filter, radius, anchor or step count out of range";
        case SSAM_ERR_ENUM: return "unknown dtype, boundary or tuning name";
        case SSAM_ERR_ALIAS: return "input and output buffers overlap";
        case SSAM_ERR_HIP: return "HIP runtime call failed";
        default: return "unknown status";
    }
}

int ssam_set_tuning(const char* name, int value)
{
    if (!name) return SSAM_ERR_NULL;
    if (!strcmp(name, "rows_per_wave")) g_rows_per_wave = value;
    else if (!strcmp(name, "valid_lanes")) g_valid_lanes = value;
    else if (!strcmp(name, "planes_per_wave")) g_planes_per_wave = value;
    else if (!strcmp(name, "xcd_remap")) g_xcd_remap = value;
    else if (!strcmp(name, "force_generic")) g_force_generic = value;
    else if (!strcmp(name, "variant")) g_variant = value;
    else if (!strcmp(name, "march_axis")) g_march_axis = value;
    else if (!strcmp(name, "fuse_sweeps")) g_fuse_sweeps = value;
    else if (!strcmp(name, "embed_waste")) g_embed_waste = value;
    else if (!strcmp(name, "scan_segments")) g_scan_segments = value;
    else if (!strcmp(name, "scan_order")) g_scan_order = value;
    else if (!strcmp(name, "scan_chained")) g_scan_chained = value;
    else if (!strcmp(name, "scan_spin_limit")) g_scan_spin_limit = value;
    else if (!strcmp(name, "scan_one_group")) g_scan_one_group = value;
    else return SSAM_ERR_ENUM;
    return SSAM_OK;
}

int ssam_describe(int kind, int W, int H, int D, const void* h_coef, int a, int b, int c, int boundary, int dtype,
                  char* buf, int buflen)
{
    void* out = nullptr;   // describe plans only: no pointer is dereferenced, no kernel runs
    std::string name;
    Geometry g;
    if (kind == 0) {
        int ax = -1, ay = -1;
        if (!h_coef) return SSAM_ERR_NULL;
        if (int e = check_enums(boundary, dtype)) return e;
        if (int e = check_dims(W, H, 1)) return e;
        if (a <= 0 || b <= 0 || a > SSAM_MAX_FILTER || b > SSAM_MAX_FILTER) return SSAM_ERR_SHAPE;
        ax = a / 2;
        ay = b / 2;
        Problem2D p{nullptr, out, W, H, h_coef, a, b, ax, ay, boundary, dtype, nullptr};
        return describe(run2d(p, false, &g, true, &name), name, g, buf, buflen);
    }
    if (kind == 1 || kind == 2) {
        if (!h_coef) return SSAM_ERR_NULL;
        if (int e = check_enums(boundary, dtype)) return e;
        if (kind == 1) { D = 1; c = 0; }
        if (int e = check_dims(W, H, D)) return e;
        if (a < 0 || b < 0 || c < 0 || a > SSAM_MAX_RADIUS || b > SSAM_MAX_RADIUS || c > SSAM_MAX_RADIUS)
            return SSAM_ERR_SHAPE;
        Problem3D p{nullptr, out, W, H, D, h_coef, a, b, c, boundary, dtype, nullptr};
        return describe(run3d(p, &g, true, &name), name, g, buf, buflen);
    }
    if (kind == 3) {   // the launch ssam_stencil_iterate uses while c (or more) 2D sweeps remain
        if (!h_coef) return SSAM_ERR_NULL;
        if (int e = check_enums(boundary, dtype)) return e;
        if (int e = check_dims(W, H, 1)) return e;
        if (a < 0 || b < 0 || a > SSAM_MAX_RADIUS || b > SSAM_MAX_RADIUS) return SSAM_ERR_SHAPE;
        Problem3D p{nullptr, out, W, H, 1, h_coef, a, b, 0, boundary, dtype, nullptr};
        int rc = SSAM_OK;
        if (run_fused(p, c > 0 ? c : 3 * kMaxFusedSweeps, &g, true, &name, &rc)) return describe(rc, name, g, buf, buflen);
        return describe(run3d(p, &g, true, &name), name, g, buf, buflen);
    }
    if (kind == 4 || kind == 6) {   // the launch ssam_stencil_iterate uses on a 3D grid while two, or c, sweeps remain
        const int remaining = kind == 6 ? c : 2;
        if (kind == 6) b = c = a;
        if (!h_coef) return SSAM_ERR_NULL;
        if (int e = check_enums(boundary, dtype)) return e;
        if (int e = check_dims(W, H, D)) return e;
        if (a < 0 || b < 0 || c < 0 || a > SSAM_MAX_RADIUS || b > SSAM_MAX_RADIUS || c > SSAM_MAX_RADIUS)
            return SSAM_ERR_SHAPE;
        Problem3D p{nullptr, out, W, H, D, h_coef, a, b, c, boundary, dtype, nullptr};
        int rc = SSAM_OK;
        if (remaining > 1 && run_fused(p, remaining, &g, true, &name, &rc)) return describe(rc, name, g, buf, buflen);
        return describe(run3d(p, &g, true, &name), name, g, buf, buflen);
    }
    if (kind == 5) {   // ssam_conv3d with (a, b, c) = (M, N, K) and the default anchor
        int ax = -1, ay = -1, az = -1;
        if (int e = check_conv3d(W, H, D, h_coef, a, b, c, &ax, &ay, &az, boundary, dtype)) return e;
        return describe(run_conv3d(nullptr, nullptr, W, H, D, h_coef, a, b, c, ax, ay, az, boundary, dtype, nullptr, &g,
                                   true, &name), name, g, buf, buflen);
    }
    return SSAM_ERR_ENUM;
}

}  // extern "C"
