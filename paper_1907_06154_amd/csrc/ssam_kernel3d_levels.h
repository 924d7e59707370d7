// Several sweeps of a radius-1 3D stencil in one launch: a block marches along z with a tile of the grid, halo and all, and
// every sweep is a level that follows the one before two planes behind.
//
// What bounds the others: large grids are bound by memory, one read and one write a sweep (or two, ssam_kernel3d_star2.h, which
// recomputes three times the first sweep and so ends there); small and ragged ones by latency, and ssam_kernel3d_fused.h's two
// sweeps, a wave by itself, by registers and halo (201x203x199 fp32 star 26 us a sweep, single sweeps 17).  Here
//   - a wave owns P rows of 64 V columns at every level, so no point is computed twice but in the tile's halo of S rows and
//     columns; rows go between waves through LDS (each wave's first and last), columns by lane shifts;
//   - a level consumes the plane that the level before completed in the step before: one barrier a step serves all levels, and
//     nothing waits for a plane of its own step.  A level holds three values a point (the plane, the one before or the sums
//     begun): three levels of the star are 256 registers with eight points a lane, two of the other shapes 220.  In fp64 three
//     levels spill 18 (clamp 13) of them, in fp32 with eight waves six: 64-bit addresses of parts of pieces, loaded again only
//     by waves that store such parts, on ragged rows;
//   - tiles lie inside the grid, as in ssam_kernel2d_tile.h: no ragged tiles, and the boundary rule in x and y is what a wave sees
//     beyond the tile.  In z the levels see zeros, or the first and last plane again;
//   - loads and stores are buffer accesses with uniform plane bases; what a lane does not store is dropped by the bounds check.
// Tiles of 128-byte columns where the grid is beyond the caches (plan_levels).  Half pieces (V = 1, fp32 2) take half the
// registers, so that a second block shares the unit: faster on grids of up to 20 million points in spite of the wider halo.
// Measured, us a sweep, before -> now: 512^3 fp64 star 186 -> 140 (three sweeps a launch), box 323 -> 268, fp32 star 99 -> 85;
// 400x448x330 fp64 box 179 -> 108, star 113 -> 66; 201x203x199 fp64 star 19 -> 10, box 29 -> 23, fp32 star 26 -> 9.3, box 24 -> 19;
// 256^3 fp32 star 18 -> 13; 128x200x100 fp64 box 12 -> 9.4; 64x205x64 fp64 star 6.4 -> 4.4.  At 512^3 the fp64 star moves 2.4 GB in
// 420 us (5.8 TB/s).
#pragma once
#include "ssam_kernel3d_star.h"

namespace ssam {

constexpr int kLevelWaves = 8;     // waves of a block, at most

template <typename T, int NWTS>
struct ArgsLevels {
    const T* in;
    T* out;
    int W, H, D;
    int tiles_x, tiles_y, step_x, step_y;   // a tile stores step_x columns, step_y rows
    int lead_x, lead_y;                     // and begins so many before them, inside the grid
    int planes, tiles;                      // output planes of a block; blocks with work
    int blocks, xcd_remap;
    T w[NWTS];
};

// A lane's V values as one LDS access.
template <typename T, int V>
__device__ __forceinline__ typename VecOf<T, V>::type pack(const T (&x)[V])
{
    if constexpr (V == 1) {
        return x[0];
    } else {
        typename VecOf<T, V>::type v;
#pragma unroll
        for (int j = 0; j < V; ++j) v[j] = x[j];
        return v;
    }
}
template <typename T, int V>
__device__ __forceinline__ void unpack(typename VecOf<T, V>::type v, T (&x)[V])
{
    if constexpr (V == 1) {
        x[0] = v;
    } else {
#pragma unroll
        for (int j = 0; j < V; ++j) x[j] = v[j];
    }
}

// Buffer accesses of a lane's V values.
constexpr int kLevelBufferBytes = 1 << 30;
constexpr unsigned kLevelNowhere = 3u << 30;         // an offset beyond the buffer
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));
template <typename T, int V, class Buffer>
__device__ __forceinline__ void load_piece(Buffer buf, unsigned off, unsigned row, T (&x)[V])
{
    if constexpr (V * sizeof(T) == 16) unpack<T, V>(__builtin_bit_cast(typename VecOf<T, V>::type, __builtin_amdgcn_raw_buffer_load_b128(buf, off, row, 0)), x);
    else unpack<T, V>(__builtin_bit_cast(typename VecOf<T, V>::type, __builtin_amdgcn_raw_buffer_load_b64(buf, off, row, 0)), x);
}
template <typename T, int V, bool STREAM, class Buffer>
__device__ __forceinline__ void store_piece(Buffer buf, unsigned off, unsigned row, const T (&x)[V])
{
    constexpr int aux = STREAM ? 2 : 0;              // 2: non-temporal
    if constexpr (V * sizeof(T) == 16) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, pack<T, V>(x)), buf, off, row, aux);
    else __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2_t, pack<T, V>(x)), buf, off, row, aux);
}

// LDS written and read by the block's waves: ordered by a barrier that leaves global loads and stores in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" : : : "memory"); }

// LDS of a block: for every level and parity of the step a row of zeros, then the first and last row of every wave.
template <typename T, int V, int NW, int S>
struct LevelRows {
    static constexpr int kRegion = (1 + 2 * NW) * kWave;          // pieces of V values
    static constexpr size_t kBytes = (size_t)2 * S * kRegion * V * sizeof(T);
};

template <typename T, int V, int P, int NW, int BUDGET, int S, bool CLAMP, bool STREAM>
__global__ __launch_bounds__(NW* kWave) __attribute__((amdgpu_waves_per_eu(2))) void ssam3d_levels_kernel(
    const ArgsLevels<T, SliceMask<1, 1, 1, BUDGET, 0>::kNW> a)
{
    constexpr int TW = kWave * V, TH = NW * P;
    typedef typename VecOf<T, V>::type vec_t;
    typedef __attribute__((address_space(3))) vec_t lds_vec;
    typedef LevelRows<T, V, NW, S> Rows;
    constexpr bool STAR = BUDGET == 1;
    constexpr int BUFS = STAR ? 2 : 1;
    static_assert(P >= 2, "a wave's first and last row are two");
    extern __shared__ __attribute__((aligned(16))) char lds_raw[];

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lb = logical_block(blockIdx.x, a.blocks, a.xcd_remap);
    if (lb >= a.tiles) return;                 // block-uniform
    const int tx = lb % a.tiles_x, ty = (lb / a.tiles_x) % a.tiles_y, tz = lb / (a.tiles_x * a.tiles_y);
    const int W = a.W, H = a.H, D = a.D;
    const int xa = tx * a.step_x, xb = min(xa + a.step_x, W), ya = ty * a.step_y, yb = min(ya + a.step_y, H);
    const int x0 = min(max(xa - a.lead_x, 0), W - TW), y0 = min(max(ya - a.lead_y, 0), H - TH);
    const int z0 = tz * a.planes, z1 = min(z0 + a.planes, D);
    const int xc = x0 + lane * V, yw = y0 + wave * P;
    typedef ArgsLevels<T, SliceMask<1, 1, 1, BUDGET, 0>::kNW> Args;
    const ConstPtr<T> wts = kernarg_member<T>(offsetof(Args, w));

    // what the lane stores: whole pieces, or parts of one at a tile's rim; which of the wave's rows
    const bool whole = xc >= xa && xc + V <= xb, part = !whole && xc < xb && xc + V > xa;
    const bool parts = __any(part);
    const int r0 = max(ya - yw, 0), r1 = min(yb - yw, P);

    // Level i's planes: Q[i] the one it consumes next (of a star, and the one before); the sums it has begun.
    T Q[S][BUFS][P][V], B[S][P][V], A[S][P][V], pre[P][V];     // pre: the next input plane, on its way
#pragma unroll
    for (int i = 0; i < S; ++i)
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int j = 0; j < V; ++j) {
                Q[i][0][p][j] = Q[i][BUFS - 1][p][j] = B[i][p][j] = T(0);
                if constexpr (!STAR) A[i][p][j] = T(0);
            }

    // the rows above and below the wave's own: its neighbours', or beyond the tile, which is beyond the grid where it matters
    lds_vec* const lds = (lds_vec*)(__attribute__((address_space(3))) char*)lds_raw + lane;
    lds_vec* const rim = lds + (1 + 2 * wave) * kWave;
    lds_vec* const above = lds + (wave > 0 ? 2 * wave : CLAMP ? 1 : 0) * kWave;
    lds_vec* const below = lds + (wave < NW - 1 ? 3 + 2 * wave : CLAMP ? 2 * NW : 0) * kWave;
    if (!CLAMP && wave == 0) {
        const T zero[V] = {};
#pragma unroll
        for (int i = 0; i < 2 * S; ++i) lds[i * Rows::kRegion] = pack<T, V>(zero);
    }

    const int zs = z0 - S;                             // the first input plane
    const int nt = (z1 - z0) + 3 * S - 1;              // steps
    const unsigned mine = lane * V * sizeof(T), row_bytes = W * (unsigned)sizeof(T);
    const size_t plane = (size_t)W * H, corner = (size_t)yw * W + x0;
    const char* src = reinterpret_cast<const char*>(a.in + (size_t)min(max(zs, 0), D - 1) * plane + corner);
    char* dst = reinterpret_cast<char*>(a.out + (size_t)z0 * plane + corner);

    // Loads and stores are buffer accesses: a lane's offset beyond the buffer drops a store, so that every wave issues the same
    // requests whatever it stores, without branches, and the compiler's counts of requests in flight are exact.
    auto load_plane = [&]() __attribute__((always_inline)) {
        const auto buf = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(src), 0, kLevelBufferBytes, 0x00027000);
#pragma unroll
        for (int p = 0; p < P; ++p) load_piece<T, V>(buf, mine, p * row_bytes, pre[p]);
    };
    auto store_plane = [&](const T (&out)[P][V]) __attribute__((always_inline)) {
        const auto buf = __builtin_amdgcn_make_buffer_rsrc(dst, 0, kLevelBufferBytes, 0x00027000);
#pragma unroll
        for (int p = 0; p < P; ++p) store_piece<T, V, STREAM>(buf, whole && p >= r0 && p < r1 ? mine : kLevelNowhere, p * row_bytes, out[p]);
        if (parts) {
#pragma unroll
            for (int p = 0; p < P; ++p) {
                T* const q = reinterpret_cast<T*>(dst + p * row_bytes + mine);
#pragma unroll
                for (int j = 0; j < V; ++j)
                    if (part && p >= r0 && p < r1 && xc + j >= xa && xc + j < xb) q[j] = out[p][j];
            }
        }
    };

    // Level i consumes its plane zin and completes plane zin - 1 of its sweep.  b: the step's parity.  EDGE: the planes may lie
    // outside the grid or before the chunk.
    auto level = [&](auto edge_tag, auto ic, auto bc, int t) __attribute__((always_inline)) {
        constexpr bool EDGE = decltype(edge_tag)::value;
        constexpr int i = decltype(ic)::value, b = decltype(bc)::value;
        constexpr int now = STAR ? b : 0, old = STAR ? b ^ 1 : 0;
        const int zin = zs + t - 2 * i, zo = zin - 1;
        T up[V], down[V];
        unpack<T, V>(above[(i * 2 + b) * Rows::kRegion], up);
        unpack<T, V>(below[(i * 2 + b) * Rows::kRegion], down);
        T(&u)[P][V] = Q[i][now];
        auto row = [&](int k, int j) __attribute__((always_inline)) { return k == 0 ? up[j] : k == P + 1 ? down[j] : u[k >= 1 && k <= P ? k - 1 : 0][j]; };
        // row k with one column more on either side
        auto widen = [&](int k, T (&xs)[V + 2]) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < V; ++j) xs[j + 1] = row(k, j);
            xs[0] = CLAMP ? shift_in_up(xs[V], xs[1]) : shift_up(xs[V]);
            xs[V + 1] = CLAMP ? shift_in_down(xs[1], xs[V]) : shift_down(xs[1]);
        };
        T out[P][V];
        if constexpr (STAR) {
            T(&before)[P][V] = Q[i][old];
            if (EDGE && CLAMP && i > 0 && zin == 0) {          // the plane above the grid repeats this one
#pragma unroll
                for (int p = 0; p < P; ++p)
#pragma unroll
                    for (int j = 0; j < V; ++j) before[p][j] = u[p][j];
            }
            const T wzm = wts[0], wc = wts[1], wzp = wts[2], wym = wts[3], wyp = wts[5], wxm = wts[6], wxp = wts[8];
#pragma unroll
            for (int p = 0; p < P; ++p) {
                T xs[V + 2];
                widen(p + 1, xs);
#pragma unroll
                for (int j = 0; j < V; ++j) {
                    out[p][j] = fma_into(u[p][j], wzp, B[i][p][j]);
                    // fp32: in two chains, which round less than one (6.1e-8 of the result against 6.3e-8 .. 6.5e-8)
                    T s = before[p][j] * wzm;
                    s = fma_t(row(p, j), wym, s);
                    if constexpr (sizeof(T) == 4) {
                        T c = xs[j] * wxm;
                        c = fma_t(u[p][j], wc, c);
                        c = fma_t(xs[j + 2], wxp, c);
                        s = fma_t(row(p + 2, j), wyp, s) + c;
                    } else {
                        s = fma_t(xs[j], wxm, s);
                        s = fma_t(u[p][j], wc, s);
                        s = fma_t(xs[j + 2], wxp, s);
                        s = fma_t(row(p + 2, j), wyp, s);
                    }
                    B[i][p][j] = s;
                }
            }
        } else {
            typedef SliceMask<1, 1, 1, BUDGET, 1> Next;
            typedef SliceMask<1, 1, 1, BUDGET, 0> Here;
            typedef SliceMask<1, 1, 1, BUDGET, -1> Last;
            auto add = [&](auto mask, auto&& start, T (&sum)[P][V]) __attribute__((always_inline)) {
                typedef decltype(mask) Mask;
                bool have[P];
#pragma unroll
                for (int p = 0; p < P; ++p) have[p] = false;
#pragma unroll
                for (int k = 0; k < P + 2; ++k) {
                    T xs[V + 2];
                    widen(k, xs);
#pragma unroll
                    for (int p = 0; p < P; ++p) {
                        const int n = k - p;
                        if (n < 0 || n > 2) continue;
#pragma unroll
                        for (int m = 0; m < 3; ++m) {
                            if (!Mask::tap(n, m)) continue;
                            const T w = wts[Mask::widx(n, m)];
#pragma unroll
                            for (int j = 0; j < V; ++j) sum[p][j] = have[p] ? fma_t(xs[j + m], w, sum[p][j]) : start(p, j, xs[j + m], w);
                            have[p] = true;
                        }
                    }
                }
            };
            add(Next{}, [&](int p, int j, T x, T w) __attribute__((always_inline)) { return fma_into(x, w, B[i][p][j]); }, out);
            if (EDGE && CLAMP && i > 0 && zin == 0)            // the plane above the grid repeats this one
                add(Last{}, [&](int, int, T x, T w) __attribute__((always_inline)) { return x * w; }, A[i]);
            add(Here{}, [&](int p, int j, T x, T w) __attribute__((always_inline)) { return fma_into(x, w, A[i][p][j]); }, B[i]);
            add(Last{}, [&](int, int, T x, T w) __attribute__((always_inline)) { return x * w; }, A[i]);
        }
        if constexpr (i == S - 1) {
            if (!EDGE || zo >= z0) {
                store_plane(out);
                dst += plane * sizeof(T);
            }
        } else {
            constexpr int n = i + 1 < S ? i + 1 : i;
            T(&q)[P][V] = Q[n][old];
            // outside the grid the next sweep sees zero, or the last plane again
            const bool blank = EDGE && !CLAMP && (zo < 0 || zo >= D), again = EDGE && CLAMP && zo >= D;
#pragma unroll
            for (int p = 0; p < P; ++p)
#pragma unroll
                for (int j = 0; j < V; ++j) q[p][j] = blank ? T(0) : again ? Q[n][now][p][j] : out[p][j];
        }
    };
    // One step: every level, the last first, consumes the plane that the level before completed in the last step.
    auto step = [&](auto edge_tag, auto bc, int t) __attribute__((always_inline)) {
        constexpr bool EDGE = decltype(edge_tag)::value;
        constexpr int b = decltype(bc)::value, now = STAR ? b : 0;
#pragma unroll
        for (int i = 0; i < S; ++i) {
            rim[(i * 2 + b) * Rows::kRegion] = pack<T, V>(Q[i][now][0]);
            rim[(i * 2 + b) * Rows::kRegion + kWave] = pack<T, V>(Q[i][now][P - 1]);
        }
        const int z = zs + t + 1;                      // the plane of the next step
        if (!EDGE || (z > 0 && z < D)) src += plane * sizeof(T);
        load_plane();
        lds_barrier();
        static_for<S>([&](auto kk) __attribute__((always_inline)) {
            level(edge_tag, std::integral_constant<int, S - 1 - decltype(kk)::value>{}, bc, t);
            __builtin_amdgcn_sched_barrier(0);
        });
        T(&q)[P][V] = Q[0][STAR ? b ^ 1 : 0];
        const bool blank = EDGE && !CLAMP && (z < 0 || z >= D);
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int j = 0; j < V; ++j) q[p][j] = blank ? T(0) : pre[p][j];
    };

    typedef std::true_type Yes;
    typedef std::false_type No;
    typedef std::integral_constant<int, 0> Even;
    typedef std::integral_constant<int, 1> Odd;
    load_plane();
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int j = 0; j < V; ++j) Q[0][0][p][j] = !CLAMP && zs < 0 ? T(0) : pre[p][j];
    int t = 0;
    const int from = min((3 * S) / 2 * 2, nt), to = min(nt, D - 1 - zs);     // every plane of steps from .. to - 1 is inside, and stored
    for (; t < from; t += 2) {
        step(Yes{}, Even{}, t);
        if (t + 1 < nt) step(Yes{}, Odd{}, t + 1);
    }
    for (; t + 1 < to; t += 2) {
        step(No{}, Even{}, t);
        step(No{}, Odd{}, t + 1);
    }
    for (; t < nt; t += 2) {
        step(Yes{}, Even{}, t);
        if (t + 1 < nt) step(Yes{}, Odd{}, t + 1);
    }
}

constexpr int kLevelRows = 4;      // rows per wave

// A compiled kernel: LDS it asks for, its place in the list of all of them; null where a combination has none.
struct LevelsKernel {
    const void* kernel = nullptr;
    size_t lds = 0;
    int index = 0;
};
template <typename T, int BUDGET>
LevelsKernel levels_kernel(int V, int waves, int sweeps, bool clamp, bool stream);
constexpr int kLevelsIndexes = 2 * 3 * 2 * 2 * 2 * 4;

// Three sweeps of the star only: two levels of the other shapes leave no registers for a third.  Streaming stores where one block
// of eight waves marches alone (grids beyond the caches).
template <typename T, int BUDGET, int V, int NW, int S, bool CLAMP, bool STREAM>
LevelsKernel levels_entry()
{
    const int index = ((((sizeof(T) / 8 * 3 + BUDGET - 1) * 2 + (V * sizeof(T) == 16)) * 2 + (NW == 8)) * 2 + S - 2) * 4 + CLAMP * 2 + STREAM;
    return LevelsKernel{reinterpret_cast<const void*>(&ssam3d_levels_kernel<T, V, kLevelRows, NW, BUDGET, S, CLAMP, STREAM>),
                        LevelRows<T, V, NW, S>::kBytes, index};
}
template <typename T, int BUDGET, int V, int NW, int S>
LevelsKernel levels_rule(bool clamp, bool stream)
{
    if constexpr (V * sizeof(T) == 16 && NW == 8) {
        if (stream) return clamp ? levels_entry<T, BUDGET, V, NW, S, true, true>() : levels_entry<T, BUDGET, V, NW, S, false, true>();
    }
    return clamp ? levels_entry<T, BUDGET, V, NW, S, true, false>() : levels_entry<T, BUDGET, V, NW, S, false, false>();
}
template <typename T, int BUDGET, int V>
LevelsKernel levels_pick(int waves, int sweeps, bool clamp, bool stream)
{
    if (sweeps == 2) return waves == 8 ? levels_rule<T, BUDGET, V, 8, 2>(clamp, stream) : levels_rule<T, BUDGET, V, 4, 2>(clamp, stream);
    if constexpr (BUDGET == 1) {
        if (sweeps == 3) return waves == 8 ? levels_rule<T, BUDGET, V, 8, 3>(clamp, stream) : levels_rule<T, BUDGET, V, 4, 3>(clamp, stream);
    }
    return LevelsKernel{};
}

// One translation unit per type and shape.
#define SSAM_LEVELS_KERNELS(T, BUDGET)                                                                              \
    template <>                                                                                                     \
    LevelsKernel levels_kernel<T, BUDGET>(int V, int waves, int sweeps, bool clamp, bool stream)                    \
    {                                                                                                               \
        constexpr int W16 = 16 / sizeof(T);                                                                         \
        return V == W16 ? levels_pick<T, BUDGET, W16>(waves, sweeps, clamp, stream)                                 \
                        : levels_pick<T, BUDGET, W16 / 2>(waves, sweeps, clamp, stream);                            \
    }

// Launches two or three of the `remaining` sweeps of a radius-1 3D stencil, at most `deepest`; returns how many, 0: the grid is left to
// the other kernels.
int launch3d_levels(const Problem3D& pr, int budget, int remaining, int deepest, Geometry* geo, bool dry_run, hipError_t* err);

}  // namespace ssam
