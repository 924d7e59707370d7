// Dense fp32 3D filters on the bf16 matrix cores, at fp32 precision: the method of ssam_kernel2d_split.h (three-way exact
// split, six products, Toeplitz operand of a 4x4 block of outputs) with the march along z.
//
// What bounds it: the 5x5x5 filter is 250 flops per 8 bytes; on the vector unit (ssam3d_star_kernel) it takes 576 us on
// 512^3 at 0.74 of the fp32 rate, where memory would allow 200.
// A wave owns 64 columns by TB bands of four rows and marches along z.  Each step stages one input plane (TB + NB - 1 bands:
// split once into LDS of the wave's own, no barrier) and multiplies it by the K planes of the filter: the K output planes in
// flight stay in registers and move one slot per step.  All staged pieces of a group of eight columns are held in registers,
// so a piece of the filter's table is read once per TB bands.  The products of one filter plane and column group form one
// chain of matrix instructions that starts from zero and is added to the plane's sum on the vector unit: a sum is rounded
// once per chain and not once per instruction, without a second set of accumulators.  Every plane costs that addition, so a
// filter of fewer than 2.5 taps per plane is left to the fp32 kernels, which round once per tap (ratio of the errors, split to
// fp32, 60 Mpoint: 1x1xK 1.25 .. 1.4, 2x1xK 0.94 .. 1.08, 1x2xK 0.94 .. 1.06, 1x3xK 0.8 .. 0.9; 5x5x5 with 9 taps that are not
// zero 1.05, with 16 0.80).
#pragma once
#include "ssam_kernel2d_split.h"

namespace ssam {

constexpr int kSplit3dWaves = 8;
constexpr int kSplit3dTaps = 896;        // taps of one launch

struct ArgsSplit3D {
    const float* in;
    float* out;
    int W, H, D;
    int M, N, K, ax, ay, az;   // the part's own extents: K planes of N rows, at most what the instance has room for
    int boundary;
    int strips_x, tiles_y;
    long tiles;
    int planes;          // output planes per wave
    int blocks, xcd_remap;
    int accumulate;
    float w_scale, out_scale;
    float w[kSplit3dTaps];
};

// bands of four output rows per wave: what the registers leave beside K output planes in flight (three planes, three bands and two
// column groups spill six to ten of them)
constexpr int split3d_bands(int K, int NB) { return K <= 3 ? 4 : NB <= 2 ? (K <= 5 ? 4 : 3) : (K <= 5 ? 3 : 2); }

template <int K, int NB, int NG, bool TAIL>
__global__ __launch_bounds__(kSplit3dWaves* kWave) __attribute__((amdgpu_waves_per_eu(2))) void ssam3d_split_kernel(const ArgsSplit3D a)
{
    typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
    typedef __attribute__((address_space(3))) u32x2 lds_u32x2;
    typedef __attribute__((address_space(3))) float lds_float;
    typedef __attribute__((address_space(3))) char lds_char;
    extern __shared__ __attribute__((aligned(16))) char lds_raw[];
    constexpr int NW = kSplit3dWaves;
    constexpr int TB = split3d_bands(K, NB);
    constexpr int BANDS = TB + NB - 1;              // staged bands
    constexpr int TAILS = TAIL ? (NB + 1) / 2 : 0;
    constexpr int quads = 16 + 2 * NG - (TAIL ? 0 : 1);         // pieces of four columns in a staged row
    constexpr int total = BANDS * 4 * quads;                    // staged pieces per plane
    constexpr int RND = (total + kWave - 1) / kWave;            // ... per lane
    constexpr int PIECES = NG * NB + TAILS;                     // table pieces per filter plane

    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, kg = lane >> 4;
    const int M = a.M, N = a.N;
    const ConstPtr<float> wts = kernarg_member<float>(offsetof(ArgsSplit3D, w));

    // ---- the operand table, as in two dimensions, one set of pieces per filter plane
    lds_u32x4* const table = (lds_u32x4*)(lds_char*)lds_raw;
    lds_char* const stage_base = (lds_char*)lds_raw + (size_t)K * PIECES * 3 * kWave * 16;
    {
        lds_float* const wl = (lds_float*)stage_base;
        for (int i = tid; i < a.K * M * N; i += NW * kWave) wl[i] = wts[i] * a.w_scale;
        __syncthreads();
        for (int f = wave; f < K * PIECES; f += NW) {
            const int k = f / PIECES, p = f - k * PIECES;
            int n[2], m0[2];
            if (p < NG * NB) {
                const int g = p / NB, pb = p - g * NB;
                n[0] = n[1] = 4 * pb + kg - (j >> 2);
                m0[0] = 8 * g - (j & 3);
                m0[1] = m0[0] + 4;
            } else {
                const int pb = min(2 * (p - NG * NB) + 1, NB - 1);
                n[1] = 4 * pb + kg - (j >> 2);
                n[0] = pb & 1 ? n[1] - 4 : -1;
                m0[0] = m0[1] = 8 * NG - (j & 3);
            }
            u32x4 h, m, l;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int mm = m0[q] + e;
                    const bool in = k < a.K && n[q] >= 0 && n[q] < N && mm >= 0 && mm < M;
                    const float x = wl[in ? (k * N + n[q]) * M + mm : 0];
                    v[e] = in ? x : 0.0f;
                }
                u32x2 vh, vm, vl;
                split3(v, vh, vm, vl);
                h[2 * q] = vh[0]; h[2 * q + 1] = vh[1];
                m[2 * q] = vm[0]; m[2 * q + 1] = vm[1];
                l[2 * q] = vl[0]; l[2 * q + 1] = vl[1];
            }
            table[(f * 3 + 0) * kWave + lane] = h;
            table[(f * 3 + 1) * kWave + lane] = m;
            table[(f * 3 + 2) * kWave + lane] = l;
        }
        __syncthreads();
    }

    const int lb = logical_block(blockIdx.x, a.blocks, a.xcd_remap);
    const long tile = (long)lb * NW + wave;
    if (tile >= a.tiles) return;
    const int strip = (int)(tile % a.strips_x);
    const int ytile = (int)((tile / a.strips_x) % a.tiles_y);
    const int ztile = (int)(tile / ((long)a.strips_x * a.tiles_y));
    const int W = a.W, H = a.H, D = a.D;
    const int x0 = strip * 64, y0 = ytile * (4 * TB);
    const int z0 = ztile * a.planes, z1 = min(z0 + a.planes, D);
    const int nout = z1 - z0, nt = nout + K - 1;    // output planes, input planes
    const bool clamp = a.boundary == kClamp;
    const int xs = x0 - a.ax, ys = y0 - a.ay;
    const bool inside = xs >= 0 && xs + 4 * quads <= W && ys >= 0 && ys + 4 * BANDS <= H;
    const size_t plane = (size_t)W * H;
    const float* __restrict__ in = a.in;

    // The lane's staged pieces, the same in every plane: piece f = 64 i + lane is row f / quads, piece f % quads of that row.
    int off[RND];             // where the piece is read, moved into the grid
    unsigned shift = 0;       // outside: two bits per piece, how far it was moved in x ...
    unsigned right = 0, keep = ~0u;   // ... one bit, to which side; one bit per element: inside the grid
    unsigned keep_hi = ~0u;
#pragma unroll
    for (int i = 0; i < RND; ++i) {
        const int f = min(i * kWave + lane, total - 1);
        const int row = f / quads, x = xs + 4 * (f - row * quads), y = ys + row;
        const int xx = min(max(x, 0), W - 4), yy = min(max(y, 0), H - 1);
        off[i] = yy * W + xx;
        const int d = min(max(x - xx, -3), 3);
        shift |= (unsigned)(d < 0 ? -d : d) << (2 * i);
        right |= (d > 0 ? 1u : 0u) << i;
        unsigned in_grid = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) in_grid |= (clamp || (y >= 0 && y < H && x + e >= 0 && x + e < W) ? 1u : 0u) << e;
        if (i < 8) keep &= ~(((~in_grid) & 15u) << (4 * (i & 7)));
        else keep_hi &= ~(((~in_grid) & 15u) << (4 * (i & 7)));
    }
    static_assert(RND <= 16 && NG <= 2, "two masks of eight pieces; one or two column groups");

    lds_char* const stage = stage_base + (size_t)wave * (3 * total * 8);
    constexpr int rows8 = quads * 8;                    // bytes of a staged row
    const int own = kg * rows8 + j * 8;             // the lane's piece of the first band

    auto load_plane = [&](int t, float (&raw)[RND][4]) __attribute__((always_inline)) {
        const float* pz = in + (size_t)min(max(z0 - a.az + t, 0), D - 1) * plane;
#pragma unroll
        for (int i = 0; i < RND; ++i) {
            const f32x4u v = *reinterpret_cast<const f32x4u*>(pz + off[i]);
#pragma unroll
            for (int e = 0; e < 4; ++e) raw[i][e] = v[e];
        }
    };

    v4f acc[K][TB];           // acc[k]: output plane t - k
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
        for (int b = 0; b < TB; ++b) acc[k][b] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    unsigned bad = 0;         // bit s: the plane staged s steps ago holds a value the split does not carry
    unsigned redo = 0;        // output planes such a value reaches
    float raw[RND][4];

    // Four outputs from column x on.
    auto store_quad = [&](auto inside_tag, int x, int y, int z, v4f v) __attribute__((always_inline)) {
        constexpr bool INSIDE = decltype(inside_tag)::value;
        if (y >= H) return;
        float* const p0 = a.out + (size_t)z * plane + (size_t)y * W + x;
        if (INSIDE || x + 4 <= W) {
            f32x4u* const p = reinterpret_cast<f32x4u*>(p0);
            if (a.accumulate) v += (v4f)*p;
            __builtin_nontemporal_store((f32x4u)v, p);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (x + e < W) p0[e] = a.accumulate ? p0[e] + v[e] : v[e];
        }
    };

    // Stores output plane o, which the step before has completed.  touched: `bad` as it was after that step.
    auto store_plane = [&](auto inside_tag, int o, unsigned touched) __attribute__((always_inline)) {
        if ((touched & ((1u << K) - 1)) == 0) {
#pragma unroll
            for (int n = 0; n < TB; ++n) store_quad(inside_tag, x0 + 4 * j, y0 + 4 * n + kg, z0 + o, acc[K - 1][n] * a.out_scale);
        } else {
            note_band(redo, lane, o);
        }
    };

    // One step: input plane t (in `raw`) is filter plane k's input for output plane t - k.  EDGE: some of those planes may
    // lie outside the chunk.  STORE: output plane t - K is complete and is stored.
    auto step = [&](auto inside_tag, auto edge_tag, auto store_tag, int t) __attribute__((always_inline)) {
        constexpr bool INSIDE = decltype(inside_tag)::value, EDGE = decltype(edge_tag)::value, STORE = decltype(store_tag)::value;
        {
            const int z = z0 - a.az + t;
            const bool plane_in = clamp || (z >= 0 && z < D);      // wave-uniform
            float top = 0.0f;
            if constexpr (!INSIDE) {
                // the selections are made anew in every step: kept, they would take all scalar registers
                asm volatile("" : "+v"(shift), "+v"(right), "+v"(keep), "+v"(keep_hi));
            }
#pragma unroll
            for (int i = 0; i < RND; ++i) {
                float f[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) f[e] = raw[i][e];
                if constexpr (!INSIDE) {
                    // element e is column clamp(x + e) of the piece that was read |d| columns away
                    const unsigned s = (shift >> (2 * i)) & 3u;
                    const bool to_right = (right >> i) & 1u;
                    const bool s1 = s & 1u, s2 = s & 2u;
                    const bool r1 = s1 && to_right, r2 = s2 && to_right, l1 = s1 && !to_right, l2 = s2 && !to_right;
                    const float f0 = f[0], f3 = f[3];
                    f[0] = r2 ? f[2] : f[0]; f[1] = r2 ? f3 : f[1]; f[2] = r2 ? f3 : f[2];
                    f[0] = r1 ? f[1] : f[0]; f[1] = r1 ? f[2] : f[1]; f[2] = r1 ? f3 : f[2];
                    f[3] = l2 ? f[1] : f[3]; f[2] = l2 ? f0 : f[2]; f[1] = l2 ? f0 : f[1];
                    f[3] = l1 ? f[2] : f[3]; f[2] = l1 ? f[1] : f[2]; f[1] = l1 ? f0 : f[1];
                    const unsigned k4 = (i < 8 ? keep : keep_hi) >> (4 * (i & 7));
#pragma unroll
                    for (int e = 0; e < 4; ++e) f[e] = keep_if(f[e], (k4 >> e) & 1u ? ~0u : 0u);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) f[e] = keep_if(f[e], plane_in ? ~0u : 0u) * kSplitScaleIn;
#pragma unroll
                for (int e = 0; e < 4; ++e) top = __builtin_elementwise_maximum(top, __builtin_fabsf(f[e]));
                u32x2 h, m, l;
                split3(f, h, m, l);
                if ((i + 1) * kWave <= total || i * kWave + lane < total) {
                    lds_char* const p = stage + (i * kWave + lane) * 8;
                    *(lds_u32x2*)(p) = h;
                    *(lds_u32x2*)(p + total * 8) = m;
                    *(lds_u32x2*)(p + total * 16) = l;
                }
            }
            bad = (bad << 1) | (__any(!(top < kSplitLimit)) ? 1u : 0u);
        }
        wave_lds_fence();
        // stores before loads: requests complete in order, so the wait for a plane's loads is one for the stores before them
        if constexpr (STORE) store_plane(inside_tag, t - K, bad >> 1);
        if (t + 1 < nt) load_plane(t + 1, raw);

        // the chains of one column group: every filter plane, all its patch bands
        auto group = [&](auto first_tag, auto tail_tag, int g) __attribute__((always_inline)) {
            constexpr bool FIRST = decltype(first_tag)::value, TAILG = decltype(tail_tag)::value;
            constexpr int NP = TAILG ? TAILS : NB;
            bf16x8 b[3][BANDS];
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                u32x2 before = u32x2{0u, 0u};
#pragma unroll
                for (int i = 0; i < BANDS; ++i) {
                    const lds_u32x2* p = (const lds_u32x2*)(stage + own + s * total * 8 + i * 4 * rows8 + g * 16);
                    const u32x2 lo = p[0];
                    u32x2 hi = lo;
                    if constexpr (!TAILG) hi = p[1];
                    const u32x4 v = TAILG ? u32x4{before[0], before[1], lo[0], lo[1]} : u32x4{lo[0], lo[1], hi[0], hi[1]};
                    b[s][i] = __builtin_bit_cast(bf16x8, v);
                    before = lo;
                }
            }
            static_for<K>([&](auto kk) __attribute__((always_inline)) {
                constexpr int k = K - 1 - decltype(kk)::value;
                const int o = t - k;
                if (!EDGE || (o >= 0 && o < nout)) {
                    v4f c[TB];
#pragma unroll
                    for (int n = 0; n < TB; ++n) c[n] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
                    // The small products of all pieces come first, then the leading ones: a sum is rounded NP times at its own
                    // size and not after each of the 6 NP instructions, whose rounding is coarser than the vector unit's (error
                    // against 64 bits: 5x5x5 8.4e-8 -> 6.2e-8; 1x9x1, one column of a piece in use, 1.7 -> 0.66 of what fp32
                    // multiply-adds leave.  Time of 5x5x5 on 512^3: 396 -> 398 us).
                    const lds_u32x4* const first = table + (k * PIECES + (TAILG ? NG * NB : g * NB)) * 3 * kWave + lane;
                    static_for<NP>([&](auto pp) __attribute__((always_inline)) {
                        constexpr int p = decltype(pp)::value;
                        constexpr int pb = !TAILG ? p : (2 * p + 1 < NB ? 2 * p + 1 : NB - 1);
                        const lds_u32x4* const tp = first + p * 3 * kWave;
                        const bf16x8 ah = __builtin_bit_cast(bf16x8, (u32x4)tp[0]);
                        const bf16x8 am = __builtin_bit_cast(bf16x8, (u32x4)tp[kWave]);
                        const bf16x8 al = __builtin_bit_cast(bf16x8, (u32x4)tp[2 * kWave]);
#pragma unroll
                        for (int n = 0; n < TB; ++n) c[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, b[2][n + pb], c[n], 0, 0, 0);
#pragma unroll
                        for (int n = 0; n < TB; ++n) c[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, b[0][n + pb], c[n], 0, 0, 0);
#pragma unroll
                        for (int n = 0; n < TB; ++n) c[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(am, b[1][n + pb], c[n], 0, 0, 0);
#pragma unroll
                        for (int n = 0; n < TB; ++n) c[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, b[1][n + pb], c[n], 0, 0, 0);
#pragma unroll
                        for (int n = 0; n < TB; ++n) c[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(am, b[0][n + pb], c[n], 0, 0, 0);
                    });
                    static_for<NP>([&](auto pp) __attribute__((always_inline)) {
                        constexpr int p = decltype(pp)::value;
                        constexpr int pb = !TAILG ? p : (2 * p + 1 < NB ? 2 * p + 1 : NB - 1);
                        const bf16x8 ah = __builtin_bit_cast(bf16x8, (u32x4)first[p * 3 * kWave]);
#pragma unroll
                        for (int n = 0; n < TB; ++n) c[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, b[0][n + pb], c[n], 0, 0, 0);
                    });
#pragma unroll
                    for (int n = 0; n < TB; ++n) {
                        // FIRST: the sums of output plane t - k move on from slot k - 1 to slot k
                        if constexpr (!FIRST) acc[k][n] += c[n];
                        else if constexpr (k > 0) acc[k][n] = acc[k > 0 ? k - 1 : 0][n] + c[n];
                        else acc[k][n] = c[n];
                        // the additions stay in this basic block: moved into a successor of it, the first of them has been
                        // seen to read a product two cycles after it was issued (the compiler's wait states for matrix
                        // results were missing on that path)
                        asm volatile("" : "+v"(acc[k][n]));
                    }
                }
            });
        };
        group(std::true_type{}, std::false_type{}, 0);
        if constexpr (NG == 2) group(std::false_type{}, std::false_type{}, 1);
        if constexpr (TAIL) group(std::false_type{}, std::true_type{}, NG);
        wave_lds_fence();
    };

    typedef std::true_type Yes;
    typedef std::false_type No;
    auto march = [&](auto inside_tag) __attribute__((always_inline)) {
        load_plane(0, raw);
        int t = 0;
        for (; t < min(K, nt); ++t) step(inside_tag, Yes{}, No{}, t);     // nothing to store yet
        for (; t < nout; ++t) step(inside_tag, No{}, Yes{}, t);
        for (; t < nt; ++t) step(inside_tag, Yes{}, Yes{}, t);
        store_plane(inside_tag, nout - 1, bad);
    };
    if (inside) march(Yes{});
    else march(No{});

    // ---- the planes that were left out, of all the block's waves, one by one to each of them, as in two dimensions
    typedef __attribute__((address_space(3))) unsigned lds_unsigned;
    ((lds_unsigned*)stage)[lane] = redo;
    __syncthreads();
    const int waves = (int)min((long)NW, a.tiles - (long)lb * NW);
    int turn = 0;
    for (int v = 0; v < waves; ++v) {
        const unsigned noted = *((lds_unsigned*)(stage_base + (size_t)v * (3 * total * 8)) + lane);
        if (!__any(noted != 0u)) continue;
        const long vt = (long)lb * NW + v;
        const int vx = (int)(vt % a.strips_x) * 64, vy = (int)((vt / a.strips_x) % a.tiles_y) * (4 * TB);
        const int vz = (int)(vt / ((long)a.strips_x * a.tiles_y)) * a.planes, vend = min(vz + a.planes, D);
        const int ys = vy - a.ay;
        int col[TB];
#pragma unroll
        for (int n = 0; n < TB; ++n) col[n] = vx - a.ax + 4 * j;
        const bool inside_xy = vx - a.ax >= 0 && vx - a.ax + 60 + plain_reach(M) <= W && ys >= 0 && ys + 4 * TB + N - 1 <= H;
        for (int o = 0; vz + o < vend; ++o) {
            if (!band_noted(noted, o) || turn++ % waves != wave) continue;
            const int zs = vz - a.az + o;                // first input plane of the output plane
            auto plane_at = [&](int k) __attribute__((always_inline)) { return in + (size_t)min(max(zs + k, 0), D - 1) * plane; };
            auto row_at = [&](int k, int r, int n, unsigned& keep) __attribute__((always_inline)) {
                const int z = zs + k, y = ys + 4 * n + kg + r;
                if (!clamp && (z < 0 || z >= D || y < 0 || y >= H)) keep = 0u;
                return min(max(y, 0), H - 1) * W;
            };
            float s[TB][4];
            if (inside_xy && zs >= 0 && zs + a.K <= D) plain_sums<TB, true>(a.K, N, plane_at, row_at, col, W, clamp, wts, M, s);
            else plain_sums<TB, false>(a.K, N, plane_at, row_at, col, W, clamp, wts, M, s);
#pragma unroll
            for (int n = 0; n < TB; ++n)
                store_quad(No{}, vx + 4 * j, vy + 4 * n + kg, vz + o, v4f{s[n][0], s[n][1], s[n][2], s[n][3]});
        }
    }
}

typedef void (*Split3dKernel)(const ArgsSplit3D);
constexpr int split3d_max_planes(int groups) { return groups == 1 ? 7 : 4; }   // filter planes of one launch

// The instances for NG groups of eight columns, with or without a tail piece (one translation unit each).
template <int NG, bool TAIL>
Split3dKernel split3d_kernel(int K, int bands);

#define SSAM_SPLIT3D_K(K, NB, NG, TAIL) \
    if (K <= split3d_max_planes(NG) && k == K && bands == NB) return &ssam3d_split_kernel<(K <= split3d_max_planes(NG) ? K : 1), NB, NG, TAIL>;
#define SSAM_SPLIT3D_NB(NB, NG, TAIL)                                                                                    \
    SSAM_SPLIT3D_K(1, NB, NG, TAIL) SSAM_SPLIT3D_K(2, NB, NG, TAIL) SSAM_SPLIT3D_K(3, NB, NG, TAIL)                      \
    SSAM_SPLIT3D_K(4, NB, NG, TAIL) SSAM_SPLIT3D_K(5, NB, NG, TAIL) SSAM_SPLIT3D_K(6, NB, NG, TAIL) SSAM_SPLIT3D_K(7, NB, NG, TAIL)
#define SSAM_SPLIT3D_KERNELS(NG, TAIL)                                                                                   \
    template <>                                                                                                          \
    Split3dKernel split3d_kernel<NG, TAIL>(int k, int bands)                                                             \
    {                                                                                                                    \
        SSAM_SPLIT3D_NB(1, NG, TAIL) SSAM_SPLIT3D_NB(2, NG, TAIL) SSAM_SPLIT3D_NB(3, NG, TAIL)                           \
        return nullptr;                                                                                                  \
    }

// hipErrorNotSupported: not for this kernel.
hipError_t launch3d_split(const float* in, float* out, int W, int H, int D, const float* w, int M, int N, int K, int ax, int ay,
                          int az, int boundary, hipStream_t stream, const Tuning& tu, Geometry* geo, bool dry_run);

}  // namespace ssam
