// Dense fp32 2D filters on the bf16 matrix cores, at fp32 precision.
//
// What bounds it: a 20x20 filter is 800 flops per 8 bytes, and the fp32 matrix instructions (ssam2d_kernel, engine 1)
// end at 157 TFLOP/s: 605 us on 8192^2, where memory would allow 90.  The bf16 matrix instructions are sixteen times as
// fast.  They are used here without giving up precision:
//   - Every fp32 value is the exact sum of three bf16 values, x = h + m + l (8 + 8 + 8 bits).  Of the nine partial products
//     of x and a weight, six are formed (l*m, m*l and l*l together reach 2^-24 of the product, 2^-26.5 in the quadratic mean)
//     and summed in fp32; the leading products h*h have an accumulator of their own, so that the small ones do not round it.
//     Error against 64-bit sums, 2-norm, uniform random filters on pictures in [0, 1) and [-1, 1): 9x9 4.6 .. 5.3e-8 (fp32
//     matrix instructions: 1.4 .. 1.6e-7), 20x20 1.0 .. 2.0e-7 (3.0 .. 3.8e-7); from three taps on no filter was further off
//     than fp32 multiply-adds in the mean (launch2d_split leaves one and two to those).
//   - Inputs are scaled by 2^24 and weights to [1, 2), so that no part becomes subnormal; a value that is not finite or is
//     2^76 and more (found while the row is split) sends the outputs in its reach to plain fp32 multiply-adds.
//   - The matrix operand that holds the filter is the Toeplitz matrix of a 4x4 block of outputs: 16 outputs by the (N + 3)
//     x (M + 3) patch they read.  Larger blocks would hold more zeros; this one is 400 / 576 full at 20x20.
//
// Layout of one v_mfma_f32_16x16x32_bf16: rows i = the 16 outputs of a block (i = 4 dy + dx), columns j = 16 blocks side by
// side (64 image columns), depth k = 4 patch rows by 8 patch columns: lane l supplies, of patch row l / 16, the 8 columns of
// block l % 16, and receives output row l / 16 of that block: four adjacent pixels, one 16-byte store.  Patch rows go by
// bands of four, and input band t is patch band pb of output band t - pb: a wave marches down its tile a band a step, keeps
// the NB output bands in flight in registers, and every staged input piece is used NB times.
// Rows of a wave's strip (NX * 64 columns) are split once, into LDS of the wave's own (no barrier in the march); the
// filter's table is shared by the block's waves.  When M + 3 is 1 to 4 columns more than whole pieces of eight, the rest is
// a piece of eight rows by four columns, from two bands (TAIL: 13 pieces instead of 15 at 15x15, 5 instead of 6 at 9x9).
// Measured on 8192^2 (fp32 matrix instructions -> this kernel, us): 9x9 165 -> 143, 11x11 226 -> 172, 15x15 361 -> 247, 20x20
// 605 -> 319, 25x25 (direct kernel) 20400 -> 590; 1024^2: 9x9 15.7 -> 9.0, 20x20 123 -> 16.  In the 20x20 launch the matrix
// pipe is busy for 0.70 of the cycles (at the 1.86 GHz the chip then runs at), the other vector instructions take 0.14.
#pragma once
#include "ssam_device.h"
#include "ssam_host.h"

namespace ssam {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));   // element-aligned 16-byte access
typedef float f32x3u __attribute__((ext_vector_type(3), aligned(4)));

constexpr int kSplitMaxTaps = 672;          // taps of one launch (a 32-wide filter of 21 rows)
constexpr float kSplitScaleIn = 0x1p24f;    // inputs are multiplied by this
constexpr float kSplitLimit = 0x1p100f;     // scaled inputs from here on take the plain path

struct ArgsSplit2D {
    const float* in;
    float* out;
    int W, H;
    int M, N, ax, ay;
    int groups;          // whole pieces of 8 columns in a row of the patch
    int boundary;
    int strips_x;
    long tiles;
    int rows;            // output rows per wave, a multiple of 4
    int blocks, xcd_remap;
    int accumulate;
    float w_scale, out_scale;
    float w[kSplitMaxTaps];
};

// f = h + m + l, three bf16 values, exactly (round to nearest twice; the rest has at most 8 bits).
__device__ __forceinline__ void split3(const float (&f)[4], u32x2& h, u32x2& m, u32x2& l)
{
    float r[4];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const f32x2 v{f[2 * i], f[2 * i + 1]};
        const bf16x2 b = __builtin_convertvector(v, bf16x2);
        const unsigned bits = __builtin_bit_cast(unsigned, b);
        h[i] = bits;
        r[2 * i] = f[2 * i] - __builtin_bit_cast(float, bits << 16);
        r[2 * i + 1] = f[2 * i + 1] - __builtin_bit_cast(float, bits & 0xffff0000u);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const f32x2 v{r[2 * i], r[2 * i + 1]};
        const bf16x2 b = __builtin_convertvector(v, bf16x2);
        const unsigned bits = __builtin_bit_cast(unsigned, b);
        m[i] = bits;
        const f32x2 s{r[2 * i] - __builtin_bit_cast(float, bits << 16), r[2 * i + 1] - __builtin_bit_cast(float, bits & 0xffff0000u)};
        l[i] = __builtin_bit_cast(unsigned, __builtin_convertvector(s, bf16x2));
    }
}


// ---- values the split does not carry: plain multiply-adds -----------------------------------------------------------------
// A wave notes the bands (planes) of outputs that such a value reaches and stores nothing there; the block makes them after the
// march, when the accumulators' registers are free: band o is bit o / 64 of lane o % 64's word.
// Made by the wave itself within the march, a load per four multiply-adds, they were most of the time as soon as one value was
// not finite.  4096^2 / 256^3, us: no NaN | 17 of them | one value in 10^4 | all:
//   9x9    before 43 | 196 | 679 | 989      now 43 | 57 | 100 | 218      (fp32 matrix instructions: 49 .. 53 whatever the values)
//   20x20  before 93 | 1378 | 3669 | 4074   now 93 | 127 | 430 | 694     (220 .. 245)
//   5x5x5  before 61 | 1326 | 2557 | 2872   now 60 | 127 | 328 | 392     (vector unit: 102)
constexpr int kSplitMaxBands = 64 * 32;
__device__ __forceinline__ void note_band(unsigned& redo, int lane, int o) { redo |= (lane == (o & 63) ? 1u : 0u) << (o >> 6); }
__device__ __forceinline__ bool band_noted(unsigned redo, int o)
{
    return ((unsigned)__builtin_amdgcn_readlane((int)redo, o & 63) >> (o >> 6)) & 1u;
}

// f holds the four columns from clamp(x, 0, W - 4) on, |d| columns away from x; makes element e column clamp(x + e, 0, W - 1).
__device__ __forceinline__ void move_columns(float (&f)[4], int d)
{
    const float f0 = f[0], f3 = f[3];
    const bool r2 = d >= 2, r1 = d >= 3 || d == 1, l2 = d <= -2, l1 = d <= -3 || d == -1;
    f[0] = r2 ? f[2] : f[0]; f[1] = r2 ? f3 : f[1]; f[2] = r2 ? f3 : f[2];
    f[0] = r1 ? f[1] : f[0]; f[1] = r1 ? f[2] : f[1]; f[2] = r1 ? f3 : f[2];
    f[3] = l2 ? f[1] : f[3]; f[2] = l2 ? f0 : f[2]; f[1] = l2 ? f0 : f[1];
    f[3] = l1 ? f[2] : f[3]; f[2] = l1 ? f[1] : f[2]; f[1] = l1 ? f0 : f[1];
}

// s[b][e] = the sum over `planes` x `rows` filter rows of M taps at columns col[b] + e, b < B: B independent rows, or parts of
// one.  plane_at(k) is the (wave-uniform) start of filter plane k's input plane, row_at(k, r, b, keep) the offset in it of filter
// row (k, r)'s input row, both moved into the grid; it clears keep where the row counts as zeros.  Eight taps are a step: three
// pieces of four columns and eight weights, requested a step ahead.  INSIDE: rows, planes and columns col[b] .. col[b] +
// plain_reach(M) - 1 lie inside the grid for every lane.
constexpr int plain_reach(int M) { return (M + 7) / 8 * 8 + 4; }
template <int B, bool INSIDE, class PlaneAt, class RowAt>
__device__ __forceinline__ void plain_sums(int planes, int rows, const PlaneAt& plane_at, const RowAt& row_at, const int (&col)[B], int W,
                                           bool clamp, const ConstPtr<float> w, int M, float (&s)[B][4])
{
    const int lane = threadIdx.x & (kWave - 1);
    float win[2][B][12], wm[2];              // wm: lane i's is the step's weight i % 8 (scalar loads return in any order: a wait
    unsigned keep[2][B];                     // for one step's would be a wait for the next one's)
    int k = 0, r = 0, m = 0;                 // the step that is requested next; the last one again after the last
    auto request = [&](auto buf) __attribute__((always_inline)) {
        constexpr int H = decltype(buf)::value;
        const float* const pk = plane_at(k);
#pragma unroll
        for (int b = 0; b < B; ++b) {
            keep[H][b] = ~0u;
            const int row = row_at(k, r, b, keep[H][b]);
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const int x = col[b] + m + 4 * q;
                if (INSIDE && q == 2) {      // column 11 has no use, and the compiler gives its register away while the load runs
                    const f32x3u v = *reinterpret_cast<const f32x3u*>(pk + (row + x));
#pragma unroll
                    for (int e = 0; e < 3; ++e) win[H][b][4 * q + e] = v[e];
                } else {
                    const f32x4u v = *reinterpret_cast<const f32x4u*>(pk + (row + (INSIDE ? x : min(max(x, 0), W - 4))));
#pragma unroll
                    for (int e = 0; e < 4; ++e) win[H][b][4 * q + e] = v[e];
                }
            }
        }
        wm[H] = w[(k * rows + r) * M + min(m + (lane & 7), M - 1)];
        const bool row_end = m + 8 >= M, plane_end = row_end && r + 1 >= rows, end = plane_end && k + 1 >= planes;
        m = end ? m : row_end ? 0 : m + 8;
        r = end ? r : plane_end ? 0 : row_end ? r + 1 : r;
        k = end || !plane_end ? k : k + 1;
    };
    auto take = [&](auto buf, int m0) __attribute__((always_inline)) {
        constexpr int H = decltype(buf)::value;
        if constexpr (!INSIDE) {
#pragma unroll
            for (int b = 0; b < B; ++b)
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const int x = col[b] + m0 + 4 * q;
                    if (!__any(x < 0 || x + 4 > W || keep[H][b] != ~0u)) continue;     // most pieces of an edge strip lie inside
                    float f[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) f[e] = win[H][b][4 * q + e];
                    move_columns(f, x - min(max(x, 0), W - 4));
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        win[H][b][4 * q + e] = keep_if(f[e], (clamp || (x + e >= 0 && x + e < W)) ? keep[H][b] : 0u);
                }
        }
        auto tap = [&](int i) __attribute__((always_inline)) {
            const float wi = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, wm[H]), i));
#pragma unroll
            for (int b = 0; b < B; ++b)
#pragma unroll
                for (int e = 0; e < 4; ++e) s[b][e] = fma_t(win[H][b][i + e], wi, s[b][e]);
        };
        if (m0 + 8 <= M) {
#pragma unroll
            for (int i = 0; i < 8; ++i) tap(i);
        } else {
#pragma unroll
            for (int i = 0; i < 7; ++i)
                if (m0 + i < M) tap(i);      // taps beyond the row are not multiplied: what lies there need not be finite
        }
    };
#pragma unroll
    for (int b = 0; b < B; ++b)
#pragma unroll
        for (int e = 0; e < 4; ++e) s[b][e] = 0.0f;
    typedef std::integral_constant<int, 0> Even;
    typedef std::integral_constant<int, 1> Odd;
    const int per_row = (M + 7) / 8, steps = planes * rows * per_row;
    int m0 = 0;
    auto next = [&]() __attribute__((always_inline)) { m0 = m0 + 8 < M ? m0 + 8 : 0; };
    request(Even{});
    int i = 0;
    for (; i + 1 < steps; i += 2) {
        request(Odd{});
        take(Even{}, m0);
        next();
        request(Even{});
        take(Odd{}, m0);
        next();
    }
    if (i < steps) take(Even{}, m0);
}

// Fences the LDS traffic of one wave: what its lanes wrote before is what its lanes read after (the
// hardware keeps a wave's LDS accesses in order; this keeps the compiler from exchanging them).
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <int NB, int NX, bool TAIL, int NW>
__global__ __launch_bounds__(NW* kWave) __attribute__((amdgpu_waves_per_eu(2))) void ssam2d_split_kernel(const ArgsSplit2D a, int pitch)
{
    typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
    typedef __attribute__((address_space(3))) u32x2 lds_u32x2;
    typedef __attribute__((address_space(3))) float lds_float;
    extern __shared__ __attribute__((aligned(16))) char lds_raw[];
    constexpr int RND = NX + 1;
    constexpr int AHEAD = NB * NX >= 12 ? 1 : 2;    // bands requested ahead: a step of many products covers the latency of one

    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, kg = lane >> 4;
    const int NG = a.groups;
    const ConstPtr<float> wts = kernarg_member<float>(offsetof(ArgsSplit2D, w));
    const int M = a.M, N = a.N;

    // ---- the operand table: piece (g, pb, split) holds, for lane l, the eight filter values its row l % 16 of the
    // matrix takes from patch row 4 pb + l / 16, patch columns 8 g .. 8 g + 7
    lds_u32x4* const table = (lds_u32x4*)(__attribute__((address_space(3))) char*)lds_raw;
    constexpr int TAILS = TAIL ? (NB + 1) / 2 : 0;
    char* const stage_raw = lds_raw + (size_t)(NG * NB + TAILS) * 3 * kWave * 16;
    {
        lds_float* const wl = (lds_float*)(__attribute__((address_space(3))) char*)stage_raw;
        for (int i = tid; i < M * N; i += NW * kWave) wl[i] = wts[i] * a.w_scale;
        __syncthreads();
        for (int f = wave; f < NG * NB + TAILS; f += NW) {
            // pieces of four patch columns: row and first column of either half
            int n[2], m0[2];
            if (f < NG * NB) {
                const int g = f / NB, pb = f - g * NB;
                n[0] = n[1] = 4 * pb + kg - (j >> 2);
                m0[0] = 8 * g - (j & 3);
                m0[1] = m0[0] + 4;
            } else {
                const int pb = min(2 * (f - NG * NB) + 1, NB - 1);
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
                    const bool in = n[q] >= 0 && n[q] < N && mm >= 0 && mm < M;
                    const float x = wl[in ? n[q] * M + mm : 0];
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
    const int ytile = (int)(tile / a.strips_x);
    const int W = a.W, H = a.H;
    const int x0 = strip * (64 * NX);
    const int y0 = ytile * a.rows;
    const int y1 = min(y0 + a.rows, H);
    const int nout = (y1 - y0 + 3) / 4;             // bands of four output rows
    const int nt = nout + NB - 1;                   // bands of four input rows
    const bool clamp = a.boundary == kClamp;
    const int quads = 16 * NX + 2 * NG - (TAIL ? 0 : 1);   // pieces of four columns in a staged row
    const int xs = x0 - a.ax;                       // first staged column
    const bool inside_x = xs >= 0 && xs + 4 * quads <= W;
    const float* __restrict__ in = a.in;

    __attribute__((address_space(3))) char* const stage =
        (__attribute__((address_space(3))) char*)stage_raw + (size_t)wave * 12 * pitch * 8;
    // lane's slot in the staged rows: writes piece 16 i + j of row kg, reads piece 16 nx + j + 2 g of row kg
    const int slot = (kg * pitch + j) * 8;

    // the lane's first staged piece of a row, and its offset when the tile is inside the grid in x (lanes past the
    // last piece repeat it)
    int off[RND];
#pragma unroll
    for (int i = 0; i < RND; ++i) off[i] = min(max(xs + 4 * min(16 * i + j, quads - 1), 0), W - 4);

    // Band t as it is in memory, rows clamped into the grid, pieces moved into it; what lies outside the grid is put
    // right when the band is staged, so that nothing waits for the loads before.
    auto load_band = [&](int t, float (&raw)[RND][4]) __attribute__((always_inline)) {
        const int y = y0 - a.ay + 4 * t + kg;
        const float* rowp = in + (size_t)min(max(y, 0), H - 1) * W;
#pragma unroll
        for (int i = 0; i < RND; ++i) {
            const f32x4u v = *reinterpret_cast<const f32x4u*>(rowp + off[i]);
#pragma unroll
            for (int e = 0; e < 4; ++e) raw[i][e] = v[e];
        }
    };

    v4f acc[NB][NX], low[NB][NX];   // sums of the leading products, of the five others
#pragma unroll
    for (int p = 0; p < NB; ++p)
#pragma unroll
        for (int n = 0; n < NX; ++n) acc[p][n] = low[p][n] = v4f{0.0f, 0.0f, 0.0f, 0.0f};

    u32x2 before[3][NX];            // TAIL: the last staged piece of the band before
#pragma unroll
    for (int s = 0; s < 3; ++s)
#pragma unroll
        for (int n = 0; n < NX; ++n) before[s][n] = u32x2{0u, 0u};

    unsigned bad = 0;      // bit k: the band staged k steps ago holds a value the split does not carry
    unsigned redo = 0;     // output bands such a value reaches

    // Four outputs from column x on, row y of a tile that ends before row yend.
    auto store_quad = [&](auto inside_tag, int x, int y, int yend, v4f v) __attribute__((always_inline)) {
        constexpr bool INSIDE = decltype(inside_tag)::value;
        if (y >= yend) return;
        float* const rowp = a.out + (size_t)y * W;
        if (INSIDE || x + 4 <= W) {
            f32x4u* const p = reinterpret_cast<f32x4u*>(rowp + x);
            if (a.accumulate) v += (v4f)*p;
            __builtin_nontemporal_store((f32x4u)v, p);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (x + e < W) rowp[x + e] = a.accumulate ? rowp[x + e] + v[e] : v[e];
        }
    };

    // Stores output band o, which the step before has completed.  touched: `bad` as it was after that step.
    auto store_band = [&](auto inside_tag, int o, unsigned touched) __attribute__((always_inline)) {
        if ((touched & ((1u << NB) - 1)) == 0) {
#pragma unroll
            for (int n = 0; n < NX; ++n) {
                // The additions read the last matrix instructions' results from another basic block, which the compiler has been
                // seen to do without the wait states this needs (see the three-dimensional kernel); eight are enough for these.
                asm volatile("s_nop 7" : "+v"(acc[NB - 1][n]), "+v"(low[NB - 1][n]));
                store_quad(inside_tag, x0 + 64 * n + 4 * j, y0 + 4 * o + kg, y1, (acc[NB - 1][n] + low[NB - 1][n]) * a.out_scale);
            }
        } else {
            note_band(redo, lane, o);
        }
    };

    // One step: input band t (in `raw`) is patch band pb of output band t - pb, for every pb; band t + AHEAD is requested.
    // EDGE: some of those output bands may lie outside the tile.  STORE: output band t - NB is complete and is stored.
    auto step = [&](auto inside_tag, auto edge_tag, auto store_tag, int t, float (&raw)[RND][4]) __attribute__((always_inline)) {
        constexpr bool INSIDE = decltype(inside_tag)::value, EDGE = decltype(edge_tag)::value, STORE = decltype(store_tag)::value;
        // ---- registers -> three bf16 parts in LDS
        {
            const int y = y0 - a.ay + 4 * t + kg;
            const unsigned keep = (clamp || (y >= 0 && y < H)) ? ~0u : 0u;
            const int xe = xs + opaque_zero();
            float top = 0.0f;
#pragma unroll
            for (int i = 0; i < RND; ++i) {
                float f[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) f[e] = raw[i][e];
                if constexpr (!INSIDE) {
                    // the piece of columns x .. x + 3 was read from inside the grid, |d| columns away: element e is
                    // column clamp(x + e)
                    const int x = xe + 4 * (16 * i + j);
                    const int d = x - min(max(x, 0), W - 4);
                    move_columns(f, d);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        f[e] = keep_if(f[e], keep & ((clamp || (x + e >= 0 && x + e < W)) ? ~0u : 0u)) * kSplitScaleIn;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) f[e] = keep_if(f[e], keep) * kSplitScaleIn;
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) top = __builtin_elementwise_maximum(top, __builtin_fabsf(f[e]));
                u32x2 h, m, l;
                split3(f, h, m, l);
                if (16 * i + j < quads) {
                    *(lds_u32x2*)(stage + slot + i * 128) = h;
                    *(lds_u32x2*)(stage + slot + pitch * 32 + i * 128) = m;
                    *(lds_u32x2*)(stage + slot + pitch * 64 + i * 128) = l;
                }
            }
            bad = (bad << 1) | (__any(!(top < kSplitLimit)) ? 1u : 0u);
        }
        wave_lds_fence();
        // The stores go before the loads: requests complete in order, so the wait for a band's loads is also one for the
        // stores before them, and these are then as old as the loads (stored at the end of a step and waited for at the
        // start of the next one, they held up every step).
        if constexpr (STORE) store_band(inside_tag, t - NB, bad >> 1);
        if (t + AHEAD < nt) load_band(t + AHEAD, raw);

        // The six products of one table piece with one staged piece.  FIRST: the sums of output band t - pb move on from
        // slot pb - 1 to slot pb.
        auto products = [&](auto first_tag, auto pb_tag, int piece, const bf16x8 (&b)[3][NX]) __attribute__((always_inline)) {
            constexpr bool FIRST = decltype(first_tag)::value;
            constexpr int pb = decltype(pb_tag)::value;
            const int o = t - pb;
            if (!EDGE || (o >= 0 && o < nout)) {
                const lds_u32x4* const tp = table + piece * 3 * kWave + lane;
                const bf16x8 ah = __builtin_bit_cast(bf16x8, (u32x4)tp[0]);
                const bf16x8 am = __builtin_bit_cast(bf16x8, (u32x4)tp[kWave]);
                const bf16x8 al = __builtin_bit_cast(bf16x8, (u32x4)tp[2 * kWave]);
                v4f c[NX], s[NX];
#pragma unroll
                for (int n = 0; n < NX; ++n) {
                    c[n] = FIRST ? (pb > 0 ? acc[pb > 0 ? pb - 1 : 0][n] : v4f{0.0f, 0.0f, 0.0f, 0.0f}) : acc[pb][n];
                    s[n] = FIRST ? (pb > 0 ? low[pb > 0 ? pb - 1 : 0][n] : v4f{0.0f, 0.0f, 0.0f, 0.0f}) : low[pb][n];
                }
#pragma unroll
                for (int n = 0; n < NX; ++n) s[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, b[2][n], s[n], 0, 0, 0);
#pragma unroll
                for (int n = 0; n < NX; ++n) c[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, b[0][n], c[n], 0, 0, 0);
#pragma unroll
                for (int n = 0; n < NX; ++n) s[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, b[0][n], s[n], 0, 0, 0);
#pragma unroll
                for (int n = 0; n < NX; ++n) s[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(am, b[1][n], s[n], 0, 0, 0);
#pragma unroll
                for (int n = 0; n < NX; ++n) s[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, b[1][n], s[n], 0, 0, 0);
#pragma unroll
                for (int n = 0; n < NX; ++n) s[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(am, b[0][n], s[n], 0, 0, 0);
#pragma unroll
                for (int n = 0; n < NX; ++n) {
                    acc[pb][n] = c[n];
                    low[pb][n] = s[n];
                }
            }
        };
        auto group = [&](auto first_tag, int g) __attribute__((always_inline)) {
            bf16x8 b[3][NX];
#pragma unroll
            for (int s = 0; s < 3; ++s)
#pragma unroll
                for (int n = 0; n < NX; ++n) {
                    const lds_u32x2* p = (const lds_u32x2*)(stage + slot + s * pitch * 32 + n * 128 + g * 16);
                    const u32x2 lo = p[0], hi = p[1];
                    const u32x4 v{lo[0], lo[1], hi[0], hi[1]};
                    b[s][n] = __builtin_bit_cast(bf16x8, v);
                }
            static_for<NB>([&](auto k) __attribute__((always_inline)) {
                constexpr int pb = NB - 1 - decltype(k)::value;
                products(first_tag, std::integral_constant<int, pb>{}, g * NB + pb, b);
            });
        };
        group(std::true_type{}, 0);
        for (int g = 1; g < NG; ++g) group(std::false_type{}, g);
        if constexpr (TAIL) {
            // the last four patch columns: a table piece takes them from two bands, the one before and this one
            bf16x8 b[3][NX];
#pragma unroll
            for (int s = 0; s < 3; ++s)
#pragma unroll
                for (int n = 0; n < NX; ++n) {
                    // one patch band: the band before is outside the outputs' reach, and what it holds need not be finite
                    const u32x2 p = NB > 1 ? before[s][n] : u32x2{0u, 0u};
                    const u32x2 q = *(const lds_u32x2*)(stage + slot + s * pitch * 32 + n * 128 + NG * 16);
                    const u32x4 v{p[0], p[1], q[0], q[1]};
                    b[s][n] = __builtin_bit_cast(bf16x8, v);
                    before[s][n] = q;
                }
            static_for<TAILS>([&](auto k) __attribute__((always_inline)) {
                constexpr int i = TAILS - 1 - decltype(k)::value;
                constexpr int pb = 2 * i + 1 < NB ? 2 * i + 1 : NB - 1;
                products(std::false_type{}, std::integral_constant<int, pb>{}, NG * NB + i, b);
            });
        }
        wave_lds_fence();
    };

    typedef std::true_type Yes;
    typedef std::false_type No;
    float raw[AHEAD][RND][4];
    auto march = [&](auto inside) __attribute__((always_inline)) {
        load_band(0, raw[0]);
        if constexpr (AHEAD == 2) {
            if (nt > 1) load_band(1, raw[1]);
        }
        int t = 0;
        // nothing to store yet
        const int warm = min(NB, nt);
        for (; t + 1 < warm; t += 2) {
            step(inside, Yes{}, No{}, t, raw[0]);
            step(inside, Yes{}, No{}, t + 1, raw[AHEAD - 1]);
        }
        constexpr int S0 = AHEAD == 2 ? NB & 1 : 0, S1 = AHEAD == 2 ? S0 ^ 1 : 0;
        if (t < warm) {
            step(inside, Yes{}, No{}, t, raw[0]);
            ++t;
        }
        for (; t + 1 < nout; t += 2) {
            step(inside, No{}, Yes{}, t, raw[S0]);
            step(inside, No{}, Yes{}, t + 1, raw[S1]);
        }
        for (; t < nt; t += 2) {
            step(inside, Yes{}, Yes{}, t, raw[S0]);
            if (t + 1 < nt) step(inside, Yes{}, Yes{}, t + 1, raw[S1]);
        }
        store_band(inside, nout - 1, bad);
    };
    if (inside_x) march(Yes{});
    else march(No{});

    // ---- the bands that were left out, of all the block's waves, one by one to each of them: a single value would otherwise
    // keep one wave busy long after the others (every band of the filter's reach, a load's latency per step)
    typedef __attribute__((address_space(3))) unsigned lds_unsigned;
    ((lds_unsigned*)stage)[lane] = redo;
    __syncthreads();
    const int waves = (int)min((long)NW, a.tiles - (long)lb * NW);
    int turn = 0;
    for (int v = 0; v < waves; ++v) {
        const unsigned noted = *((lds_unsigned*)((__attribute__((address_space(3))) char*)stage_raw + (size_t)v * 12 * pitch * 8) + lane);
        if (!__any(noted != 0u)) continue;
        const long vt = (long)lb * NW + v;
        const int vx = (int)(vt % a.strips_x) * (64 * NX), vy = (int)(vt / a.strips_x) * a.rows, vend = min(vy + a.rows, H);
        int col[NX];
#pragma unroll
        for (int n = 0; n < NX; ++n) col[n] = vx - a.ax + 64 * n + 4 * j;
        const bool inside_cols = vx - a.ax >= 0 && vx - a.ax + 64 * NX - 4 + plain_reach(M) <= W;
        for (int o = 0; vy + 4 * o < vend; ++o) {
            if (!band_noted(noted, o) || turn++ % waves != wave) continue;
            const int ys = vy - a.ay + 4 * o;            // first input row of the band
            const bool inside = inside_cols && ys >= 0 && ys + 4 + N - 1 <= H;
            auto plane_at = [&](int) __attribute__((always_inline)) { return in; };
            auto row_at = [&](int, int r, int, unsigned& keep) __attribute__((always_inline)) {
                const int y = ys + kg + r;
                if (!clamp && (y < 0 || y >= H)) keep = 0u;
                return min(max(y, 0), H - 1) * W;
            };
            float s[NX][4];
            if (inside) plain_sums<NX, true>(1, N, plane_at, row_at, col, W, clamp, wts, M, s);
            else plain_sums<NX, false>(1, N, plane_at, row_at, col, W, clamp, wts, M, s);
#pragma unroll
            for (int n = 0; n < NX; ++n)
                store_quad(No{}, vx + 64 * n + 4 * j, vy + 4 * o + kg, vend, v4f{s[n][0], s[n][1], s[n][2], s[n][3]});
        }
    }
}

// The number of taps of w[0 .. count) that are not zero, and the largest one's binary exponent; 0 for a filter the split does
// not carry.
long split_taps(const float* w, long count, int* exponent);

// Launches one filter, in parts of at most 21 rows; hipErrorNotSupported: not for this kernel.
hipError_t launch2d_split(const Problem2D& pr, const Tuning& tu, Geometry* geo, bool dry_run);

}  // namespace ssam
