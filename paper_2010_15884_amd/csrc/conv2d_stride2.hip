// 2-D valid convolution with stride 2 on both axes,
//     y[r][c] = sum_p sum_q x[2r+p][2c+q] * f[p][q],
// as the FBS design: the stride-2 FBS array of Table 2 (row 3 right) along the image
// columns, one 1-D pass per filter row as in the stride-1 2-D FBS kernel (Section 6.2),
// all passes adding into the same partial sums.
//
// For filter row p a lane holds eight consecutive inputs of image row 2r+p -- x(2c) and x(2c+1) of its four PEs -- and the
// even and the odd taps of that filter row are two stride-1 FBS chains over the de-interleaved values (the hand-over
// X(c,q) = X(c+1,q-2) never mixes the two).
//
//   conv2d_fbs_stride2_block_kernel<K,K,ROWS> 2x2 .. 5x5: all input rows of two output rows up front
//   conv2d_fbs_stride2_pair_kernel<KW,ROWS>   the rest: the input rows of one to four output rows streamed through registers, two outputs a lane
//   conv2d_fbs_stride2_strip_kernel<KW,ROWS>  single-row filters, images of fewer than four columns, two columns on large images: the same with four outputs a lane
#include "launch.h"
#include "systolic.h"
#include "tiling.h"

#include <utility>

namespace sysconv {
namespace {

typedef const float __attribute__((address_space(4)))* kernarg_floats;

constexpr int kCols = 2 * kStrip;                        // input columns of a strip (eight per lane)

// Row of a strip from the lanes' load order (lane l: columns 4l .. 4l+3 of the strip's first and second half, so that a
// load is 1 KB of consecutive addresses) to the array's (lane l: columns 8l .. 8l+7, four PEs), through 2 KB of LDS that
// belong to the wavefront.  Loaded straight by the lanes that need them, every cache line was asked for twice (us,
// before / with the exchange: 8192^2 5x5 68.4 / 62.0, 4x4 65.3 / 59.8; 4095x6001 5x5 30.6 / 26.3).  In the strip form
// below, whose row loop waits for each exchange, it costs more than it gives (4095x6001 7x7 30.2 / 30.5, 8192^2 11x11 94 / 101).
__device__ __forceinline__ void exchange_row(float* __restrict__ slot, int lane, float (&v)[8])
{
    *reinterpret_cast<f4*>(slot + kTile * lane) = f4{v[0], v[1], v[2], v[3]};
    *reinterpret_cast<f4*>(slot + kStrip + kTile * lane) = f4{v[4], v[5], v[6], v[7]};
    wave_exchange();
    const f4 lo = *reinterpret_cast<const f4*>(slot + 2 * kTile * lane), hi = *reinterpret_cast<const f4*>(slot + 2 * kTile * lane + 4);
    v[0] = lo.x; v[1] = lo.y; v[2] = lo.z; v[3] = lo.w;
    v[4] = hi.x; v[5] = hi.y; v[6] = hi.z; v[7] = hi.w;
    wave_exchange();
}

// ------------------------------------------------------------ block form ----
// For the small square filters of the paper's experiment (Section 6): a wavefront takes ROWS output rows of a strip of 512 input columns,
// requests all 2*(ROWS-1)+KH input rows up front (four consecutive inputs of either half of
// a row per lane) and then, input row by input row, passes the row through its own 2 KB of
// LDS (exchange_row), builds the shifted windows of the even and of the odd chain once and applies them to every output row whose filter covers that input
// row (p = rho - 2r).  Strips overlap: the PEs whose even chain
// would reach past lane 63 compute values that are never stored.
template <int KH, int KW, int ROWS, bool EDGE, bool EXCHANGE>
__device__ __forceinline__ void stride2_block_rows(kernarg_floats taps_f, const float* __restrict__ xrow,
                                                   float* __restrict__ yrow, int in_col0, int out_col, int w_img,
                                                   long long xp, int ow, long long yp, int rows_out, bool lane_valid,
                                                   float* __restrict__ slots, int lane)
{
    constexpr int NIN = 2 * (ROWS - 1) + KH;
    constexpr int KE = (KW + 1) / 2, KO = KW / 2;
    const int in_col = EXCHANGE ? in_col0 + kTile * lane : in_col0 + 2 * kTile * lane;
    constexpr int kSecond = EXCHANGE ? kStrip : kTile;                     // columns from a lane's first four to its other four
    const int rows_in = 2 * (rows_out - 1) + KH;
    const EdgeQuad first(in_col, w_img), second(in_col + kSecond, w_img);

    float v[NIN][8];
#pragma unroll
    for (int rho = 0; rho < NIN; ++rho) {
        // rows past the end of the block repeat its last row; they only feed output rows
        // that are not stored
        const float* p = xrow + (long long)min(rho, rows_in - 1) * xp;
        const f4u lo = *reinterpret_cast<const f4u*>(p + (EDGE ? first.at : in_col));
        const f4u hi = *reinterpret_cast<const f4u*>(p + (EDGE ? second.at : in_col + kSecond));
        v[rho][0] = lo.x; v[rho][1] = lo.y; v[rho][2] = lo.z; v[rho][3] = lo.w;
        v[rho][4] = hi.x; v[rho][5] = hi.y; v[rho][6] = hi.z; v[rho][7] = hi.w;
    }

    float acc[ROWS][4];
#pragma unroll
    for (int rho = 0; rho < NIN; ++rho) {
        if constexpr (EDGE) {
            first.put_right(v[rho][0], v[rho][1], v[rho][2], v[rho][3]);
            second.put_right(v[rho][4], v[rho][5], v[rho][6], v[rho][7]);
        }
        if constexpr (EXCHANGE) exchange_row(slots + (rho & 1) * kCols, lane, v[rho]);
        float ev[KE + 3], od[KO + 3];
#pragma unroll
        for (int i = 0; i < 4; ++i) { ev[i] = v[rho][2 * i]; od[i] = v[rho][2 * i + 1]; }
#pragma unroll
        for (int m = 4; m < KE + 3; ++m) ev[m] = from_lane_above(ev[m - 4]);
#pragma unroll
        for (int m = 4; m < KO + 3; ++m) od[m] = from_lane_above(od[m - 4]);
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const int p = rho - 2 * r;                                     // compile-time
            if (p < 0 || p >= KH) continue;
#pragma unroll
            for (int q = 0; q < KW; ++q) {
                const float wv = taps_f[p * KW + q];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float xv = (q & 1) ? od[q / 2 + i] : ev[q / 2 + i];
                    if (p == 0 && q == 0) acc[r][i] = wv * xv;
                    else acc[r][i] = __builtin_fmaf(wv, xv, acc[r][i]);
                }
            }
            if (p == KH - 1 && r < rows_out && lane_valid) {
                float* yr = yrow + (long long)r * yp;
                if (EDGE) {
                    store4_guarded(yr, out_col, ow, acc[r]);
                } else {
                    f4u t;
                    t.x = acc[r][0]; t.y = acc[r][1]; t.z = acc[r][2]; t.w = acc[r][3];
                    if (SYSCONV_NONTEMPORAL_STORE) __builtin_nontemporal_store(t, reinterpret_cast<f4u*>(yr + out_col));
                    else *reinterpret_cast<f4u*>(yr + out_col) = t;
                }
            }
        }
    }
}

// The taps (row-major, as the caller gave them) are the first kernel argument.
template <int KH, int KW, int ROWS>
__global__ __launch_bounds__(kBlock) void conv2d_fbs_stride2_block_kernel(TapsOf<KH * KW> taps, const float* __restrict__ x,
                                                                          float* __restrict__ y, int w_img,
                                                                          long long xp, int oh, int ow, long long yp,
                                                                          int row_blocks, int strips, int side,
                                                                          int per_xcd)
{
    (void)taps;
    __shared__ __attribute__((aligned(16))) float slots[kBlock / kWave][2 * kCols];
    kernarg_floats tf = (kernarg_floats)__builtin_amdgcn_kernarg_segment_ptr();
    int rb, strip;
    if (!wave_tile(per_xcd, row_blocks, strips, side, rb, strip)) return;
    constexpr int valid_lanes = kWave - halo_lanes((KW + 1) / 2);
    const int lane = threadIdx.x & (kWave - 1);
    const int out_col0 = strip * kTile * valid_lanes;
    const int r0 = rb * ROWS;
    const int rows_out = min(ROWS, oh - r0);
    const float* xrow = x + (long long)(2 * r0) * xp;
    float* yrow = y + (long long)r0 * yp;
    const bool lane_valid = lane < valid_lanes;
    const int in_col = 2 * out_col0, out_col = out_col0 + kTile * lane;
    // interior strips: all 512 input columns exist, and then so do the valid lanes' outputs
    // A right-hand strip of a 2x2 filter loads straight to the lanes: four rows do not make up for the exchange (us, straight / exchanged: 250x127
    // outputs 2.28 / 2.46, 150x230 2.46 / 2.63, 500x500 3.05 / 3.14, 1221x284 3.53 / 3.64; level from 1 M outputs on).
    float* const own = slots[wave_in_block()];
    if (2 * out_col0 + kCols <= w_img)
        stride2_block_rows<KH, KW, ROWS, false, true>(tf, xrow, yrow, in_col, out_col, w_img, xp, ow, yp, rows_out,
                                                      lane_valid, own, lane);
    else
        stride2_block_rows<KH, KW, ROWS, true, KH != 2>(tf, xrow, yrow, in_col, out_col, w_img, xp, ow, yp, rows_out,
                                                        lane_valid, own, lane);
}

template <int KH, int KW, int ROWS>
hipError_t launch_block(const float* x, int h, int w, size_t xp, const float* f, float* y, size_t yp, hipStream_t s)
{
    const TapsOf<KH * KW> taps(f, KH * KW);
    const int oh = (h - KH) / 2 + 1, ow = (w - KW) / 2 + 1;
    const int cols = kTile * (kWave - halo_lanes((KW + 1) / 2));
    const int strips = (ow + cols - 1) / cols;
    const int row_blocks = (oh + ROWS - 1) / ROWS;
    long long per_xcd;
    const long long blocks = tile_workgroups(row_blocks, strips, per_xcd);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((conv2d_fbs_stride2_block_kernel<KH, KW, ROWS>), dim3((unsigned)blocks), dim3(kBlock), 0, s,
                       taps, x, y, w, (long long)xp, oh, ow, (long long)yp, row_blocks, strips, band_width(xp),
                       (int)per_xcd);
    return hipGetLastError();
}

// ------------------------------------------------------------ strip form ----
// Single-row filters, whose output rows share no input row; images of fewer than four columns; two columns on large images (conv2d_stride2_takes_strips).  Any filter height at run time, the width at
// compile time: a wavefront takes ROWS output rows of a strip of 512
// input columns and walks down its 2*(ROWS-1)+kh input rows, kAhead of them in flight in registers.  Each row's two
// windows are built once and applied to every output row whose filter covers it.  What bounds it: HBM on large images (7559^2 8x2 63 us), the latency of its input rows on narrow ones.
// Six or eight rows in flight are 1 to 5 % and 6 to 10 % slower than four.
constexpr int kAhead = 4;

template <int KW, int ROWS, StripKind KIND>
__device__ __forceinline__ void stride2_strip_rows(kernarg_floats taps_f, const float* __restrict__ xrow,
                                                   float* __restrict__ yrow, int in_col, int out_col, int w_img,
                                                   long long xp, int ow, long long yp, int kh, int rows_out,
                                                   bool lane_valid)
{
    constexpr int KE = (KW + 1) / 2, KO = KW / 2;
    const int rows_in = 2 * (rows_out - 1) + kh;
    constexpr bool EDGE = KIND == kEdge;
    const EdgeQuad first(in_col, w_img), second(in_col + 4, w_img);

    float v[kAhead][8];
    auto load_row = [&](int rho, float (&d)[8]) {                          // past the last row: the last row again
        const float* p = xrow + (long long)min(rho, rows_in - 1) * xp;
        if constexpr (KIND == kNarrow) {
#pragma unroll
            for (int i = 0; i < 8; ++i) d[i] = p[min(in_col + i, w_img - 1)];
        } else {
            const f4u lo = *reinterpret_cast<const f4u*>(p + (EDGE ? first.at : in_col));
            const f4u hi = *reinterpret_cast<const f4u*>(p + (EDGE ? second.at : in_col + 4));
            d[0] = lo.x; d[1] = lo.y; d[2] = lo.z; d[3] = lo.w;
            d[4] = hi.x; d[5] = hi.y; d[6] = hi.z; d[7] = hi.w;
        }
    };
#pragma unroll
    for (int i = 0; i < kAhead; ++i) load_row(i, v[i]);

    float acc[ROWS][4];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) acc[r][0] = acc[r][1] = acc[r][2] = acc[r][3] = 0.0f;

    for (int rho0 = 0; rho0 < rows_in; rho0 += kAhead) {
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            const int rho = rho0 + j;
            if (rho >= rows_in) break;                                     // uniform
            // the filter rows this input row meets, asked for together
            float wv[ROWS][KW];
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                kernarg_floats fp = taps_f + min(max(rho - 2 * r, 0), kh - 1) * KW;
#pragma unroll
                for (int q = 0; q < KW; ++q) wv[r][q] = fp[q];
            }
            if constexpr (EDGE) {
                first.put_right(v[j][0], v[j][1], v[j][2], v[j][3]);
                second.put_right(v[j][4], v[j][5], v[j][6], v[j][7]);
            }
            float ev[KE + 3], od[KO + 3];
#pragma unroll
            for (int i = 0; i < 4; ++i) ev[i] = v[j][2 * i];
#pragma unroll
            for (int i = 0; i < KO + 3 && i < 4; ++i) od[i] = v[j][2 * i + 1];
            load_row(rho + kAhead, v[j]);
#pragma unroll
            for (int m = 4; m < KE + 3; ++m) ev[m] = from_lane_above(ev[m - 4]);
#pragma unroll
            for (int m = 4; m < KO + 3; ++m) od[m] = from_lane_above(od[m - 4]);
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                const int p = rho - 2 * r;
                if (p < 0 || p >= kh) continue;                            // uniform
#pragma unroll
                for (int q = 0; q < KW; ++q)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        acc[r][i] = __builtin_fmaf(wv[r][q], (q & 1) ? od[q / 2 + i] : ev[q / 2 + i], acc[r][i]);
            }
        }
    }
    if (!lane_valid) return;
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
        if (r < rows_out) store4_guarded(yrow + (long long)r * yp, out_col, ow, acc[r]);
}

template <int KW, int ROWS>
__global__ __launch_bounds__(kBlock) void conv2d_fbs_stride2_strip_kernel(TapsOf<kMaxK2D * KW> taps, const float* __restrict__ x,
                                                                          float* __restrict__ y, int w_img,
                                                                          long long xp, int oh, int ow, long long yp,
                                                                          int kh, int row_blocks, int strips, int side,
                                                                          int per_xcd)
{
    (void)taps;
    kernarg_floats tf = (kernarg_floats)__builtin_amdgcn_kernarg_segment_ptr();
    int rb, strip;
    if (!wave_tile(per_xcd, row_blocks, strips, side, rb, strip)) return;
    constexpr int valid_lanes = kWave - halo_lanes((KW + 1) / 2);
    const int lane = threadIdx.x & (kWave - 1);
    const int out_col0 = strip * kTile * valid_lanes;
    const int r0 = rb * ROWS;
    const int rows_out = min(ROWS, oh - r0);
    const float* xrow = x + (long long)(2 * r0) * xp;
    float* yrow = y + (long long)r0 * yp;
    const bool lane_valid = lane < valid_lanes;
    const int in_col = 2 * out_col0 + 2 * kTile * lane, out_col = out_col0 + kTile * lane;
    constexpr bool WIDE = ROWS == 1 || (ROWS == 3 && KW == 2);             // more rows of other widths: narrow images only
    if constexpr (KW < 4) {
        if (!WIDE || w_img < 4) {
            stride2_strip_rows<KW, ROWS, kNarrow>(tf, xrow, yrow, in_col, out_col, w_img, xp, ow, yp, kh, rows_out, lane_valid);
            return;
        }
    }
    if constexpr (WIDE) {
        if (2 * out_col0 + kCols <= w_img)
            stride2_strip_rows<KW, ROWS, kInside>(tf, xrow, yrow, in_col, out_col, w_img, xp, ow, yp, kh, rows_out, lane_valid);
        else
            stride2_strip_rows<KW, ROWS, kEdge>(tf, xrow, yrow, in_col, out_col, w_img, xp, ow, yp, kh, rows_out, lane_valid);
    }
}

template <int KW, int ROWS>
hipError_t launch_strip(const float* x, int h, int w, size_t xp, const float* f, int kh, float* y, size_t yp, hipStream_t s)
{
    const TapsOf<kMaxK2D * KW> taps(f, kh * KW);
    const int oh = (h - kh) / 2 + 1, ow = (w - KW) / 2 + 1;
    const int cols = kTile * (kWave - halo_lanes((KW + 1) / 2));
    const int strips = (ow + cols - 1) / cols;
    const int row_blocks = (oh + ROWS - 1) / ROWS;
    long long per_xcd;
    const long long blocks = tile_workgroups(row_blocks, strips, per_xcd);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((conv2d_fbs_stride2_strip_kernel<KW, ROWS>), dim3((unsigned)blocks), dim3(kBlock), 0, s,
                       taps, x, y, w, (long long)xp, oh, ow, (long long)yp, kh, row_blocks, strips, band_width(xp),
                       (int)per_xcd);
    return hipGetLastError();
}

// ------------------------------------------------------------- pair form ----
// Any filter height at run time, the width at compile time: a wavefront takes ROWS output rows of a strip of 256 input columns, two outputs a lane, and walks
// down its 2*(ROWS-1)+kh input rows, four of them in flight.  A row is one load of 1 KB; its two windows are built once and applied to every output row whose
// filter covers it.  Half as many outputs a lane as in the strips above give twice the wavefronts, less padding at the right edge, loads without gaps, and registers for four output rows.
// Taps come in a row ahead of their use, in a ring, where one fits the scalar registers (a row of taps serves output row r two input rows after r - 1).  us, strips of
// four outputs a lane / this: 4095x6001 7x7 28.9 / 26.5, 8192^2 11x11 93.5 / 92, 9x9 79.8 / 74.7, 3302x4516 15x15 39.6 / 36.2, 5564x1164 12x12 18.6 / 13.9, 780^2 12x12 7.1 / 5.7, 453^2 15x14 9.7 / 6.8;
// 200 random images and filters 0.91 on average (15x15 on 1985x3879, a seventeenth strip for 13 columns, 21.6 / 22.0).
// What bounds it: large images HBM with 1.2 to 1.3 times the image read (halo rows of neighbouring workgroups that miss L2); small ones the latency of the rows of one wavefront.
// Tried: eight rows in flight (7x7 28.2 / 31.2), wavefronts of a workgroup side by side (7x7 30.6), six and eight output rows (30.0, 31.1; 12x12 18.8, 22.2).
template <int KW>
struct PairShape {
    static constexpr int KE = (KW + 1) / 2, KO = KW / 2;                   // even and odd taps
    static constexpr int kLanes = kWave - KE / 2;                          // lanes that keep their results: windows reach KE - 1 inputs of a chain further
    static constexpr int kOut = 2 * kLanes;                                // output columns of a strip
};

template <int KW, int ROWS, bool EDGE>
__device__ __forceinline__ void stride2_pair_rows(kernarg_floats taps_f, const float* __restrict__ xrow, float* __restrict__ yrow, int in_col, int out_col,
                                                  int w_img, long long xp, int ow, long long yp, int kh, int rows_out, bool lane_valid)
{
    constexpr int KE = PairShape<KW>::KE, KO = PairShape<KW>::KO;
    // filter row p waits in slot p mod RING from input row p - 1 on to input row p + 2 (ROWS - 1)
    constexpr int RING = ROWS == 1 ? 2 : ROWS == 2 ? 4 : (KW <= 9 ? 8 : 0);
    static_assert(RING == 0 || RING >= 2 * ROWS, "a slot is free again when the next filter row comes in");
    constexpr int UNROLL = RING > kAhead ? RING : kAhead;
    // Left in the middle, the body has its ring copied to vector registers, tap by tap for every row (98 to 110 of them for two rows of 9 to 11 columns, four wavefronts a SIMD, and half of the
    // multiply-adds read a tap there); with every row guarded instead the ring stays in scalar registers (40, eight wavefronts, few or no spills).  us, left / guarded: 1066x4859 10x11 12.4 / 10.9, 1564x3252 10x10
    // 11.4 / 10.2, 2724x1940 9x9 11.0 / 9.6, 1985x3879 15x15 (no ring / guarded, with one) 23.7 / 22.2, 8192^2 11x11 90.5 / 87.9; by rows and columns, 2 rows 8 - 9 0.93, 10 - 11 0.91, 12 and more 0.94, 3 rows 0.98
    // to 0.99.  Single rows (1.04) and fewer columns (1.01 to 1.1: 7x7 on 4095x6001 26.5 / 26.9, 14x4 on 4720x4127 23.4 / 31) are quicker left: their copies are few.
    constexpr bool GUARDED = ROWS >= 2 && KW >= 8;
    const int rows_in = 2 * (rows_out - 1) + kh;
    const EdgeQuad quad(in_col, w_img);

    f4u v[kAhead];
    auto load_row = [&](int rho, f4u& d) {                                 // past the last row: the last row again
        d = *reinterpret_cast<const f4u*>(xrow + (long long)min(rho, rows_in - 1) * xp + (EDGE ? quad.at : in_col));
    };
    float wv[RING > 0 ? RING : ROWS][KW];
    auto load_taps = [&](int p, float (&w)[KW]) {
        kernarg_floats fp = taps_f + min(max(p, 0), kh - 1) * KW;
#pragma unroll
        for (int q = 0; q < KW; ++q) w[q] = fp[q];
    };
#pragma unroll
    for (int i = 0; i < kAhead; ++i) load_row(i, v[i]);
    if constexpr (RING > 0) load_taps(0, wv[0]);
    float acc[ROWS][2];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) acc[r][0] = acc[r][1] = 0.0f;

    for (int rho0 = 0; rho0 < rows_in; rho0 += UNROLL) {
#pragma unroll
        for (int j = 0; j < UNROLL; ++j) {
            const int rho = rho0 + j;
            if (!GUARDED && rho >= rows_in) break;                         // uniform
            if constexpr (RING > 0) {
                __builtin_amdgcn_sched_barrier(0);                         // (the taps of the next row stay where they are asked for)
                if constexpr (GUARDED) load_taps(rho + 1, wv[(j + 1) % (RING > 0 ? RING : 1)]);
            } else {
#pragma unroll
                for (int r = 0; r < ROWS; ++r) load_taps(rho - 2 * r, wv[r]);
            }
            if (GUARDED && rho >= rows_in) continue;                       // uniform
            f4u t = v[j % kAhead];
            float e0 = t.x, o0 = t.y, e1 = t.z, o1 = t.w;
            if constexpr (EDGE) quad.put_right(e0, o0, e1, o1);
            load_row(rho + kAhead, v[j % kAhead]);
            if constexpr (RING > 0 && !GUARDED) load_taps(rho + 1, wv[(j + 1) % RING]);
            float ev[KE + 1] = {e0, e1}, od[KO + 2] = {o0, o1};
#pragma unroll
            for (int m = 2; m < KE + 1; ++m) ev[m] = from_lane_above(ev[m - 2]);
#pragma unroll
            for (int m = 2; m < KO + 1; ++m) od[m] = from_lane_above(od[m - 2]);
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                const int p = rho - 2 * r;
                if (p < 0 || p >= kh) continue;                            // uniform
                const float (&w)[KW] = wv[RING > 0 ? (j - 2 * r + 2 * RING) % (RING > 0 ? RING : 1) : r];
#pragma unroll
                for (int q = 0; q < KW; ++q)
#pragma unroll
                    for (int i = 0; i < 2; ++i)
                        acc[r][i] = __builtin_fmaf(w[q], (q & 1) ? od[q / 2 + i] : ev[q / 2 + i], acc[r][i]);
            }
        }
    }
    if (!lane_valid) return;
    typedef float f2u __attribute__((ext_vector_type(2), aligned(4)));
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        if (r >= rows_out) break;                                          // uniform
        float* to = yrow + (long long)r * yp + out_col;
        if (!EDGE || out_col + 2 <= ow) {
            if (SYSCONV_NONTEMPORAL_STORE) __builtin_nontemporal_store(f2u{acc[r][0], acc[r][1]}, reinterpret_cast<f2u*>(to));
            else *reinterpret_cast<f2u*>(to) = f2u{acc[r][0], acc[r][1]};
        } else if (out_col < ow) {
            *to = acc[r][0];
        }
    }
}

template <int KW, int ROWS>
__global__ __launch_bounds__(kBlock) void conv2d_fbs_stride2_pair_kernel(TapsOf<kMaxK2D * KW> taps, const float* __restrict__ x,
                                                                         float* __restrict__ y, int w_img, long long xp, int oh, int ow,
                                                                         long long yp, int kh, int row_blocks, int strips, int side,
                                                                         int per_xcd)
{
    (void)taps;
    using S = PairShape<KW>;
    kernarg_floats tf = (kernarg_floats)__builtin_amdgcn_kernarg_segment_ptr();
    int rb, strip;
    if (!wave_tile(per_xcd, row_blocks, strips, side, rb, strip)) return;
    const int lane = threadIdx.x & (kWave - 1);
    const int out_col0 = strip * S::kOut, r0 = rb * ROWS;
    const int rows_out = min(ROWS, oh - r0);
    const float* xrow = x + (long long)(2 * r0) * xp;
    float* yrow = y + (long long)r0 * yp;
    const int in_col = 2 * out_col0 + kTile * lane, out_col = out_col0 + 2 * lane;
    // inside strips: all 256 input columns exist, and then so do the valid lanes' outputs
    if (2 * out_col0 + kStrip <= w_img)
        stride2_pair_rows<KW, ROWS, false>(tf, xrow, yrow, in_col, out_col, w_img, xp, ow, yp, kh, rows_out, lane < S::kLanes);
    else
        stride2_pair_rows<KW, ROWS, true>(tf, xrow, yrow, in_col, out_col, w_img, xp, ow, yp, kh, rows_out, lane < S::kLanes);
}

template <int KW, int ROWS>
hipError_t launch_pair(const float* x, int h, int w, size_t xp, const float* f, int kh, float* y, size_t yp, hipStream_t s)
{
    const TapsOf<kMaxK2D * KW> taps(f, kh * KW);
    const int oh = (h - kh) / 2 + 1, ow = (w - KW) / 2 + 1;
    constexpr int cols = PairShape<KW>::kOut;
    const int strips = (ow + cols - 1) / cols;
    const int row_blocks = (oh + ROWS - 1) / ROWS;
    long long per_xcd;
    const long long blocks = tile_workgroups(row_blocks, strips, per_xcd);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((conv2d_fbs_stride2_pair_kernel<KW, ROWS>), dim3((unsigned)blocks), dim3(kBlock), 0, s,
                       taps, x, y, w, (long long)xp, oh, ow, (long long)yp, kh, row_blocks, strips, band_width(xp),
                       (int)per_xcd);
    return hipGetLastError();
}

typedef hipError_t (*LaunchStrip)(const float*, int, int, size_t, const float*, int, float*, size_t, hipStream_t);
template <int ROWS, int KW0, int... KW>
hipError_t launch_strip_by_kw(std::integer_sequence<int, KW0, KW...>, const float* x, int h, int w, size_t xp, const float* f,
                              int kh, int kw, float* y, size_t yp, hipStream_t s)
{
    static constexpr LaunchStrip table[] = {launch_strip<KW0, ROWS>, launch_strip<KW, ROWS>...};    // widths KW0 and on
    if (kw < KW0 || kw > KW0 + (int)sizeof...(KW)) return hipErrorInvalidValue;
    return table[kw - KW0](x, h, w, xp, f, kh, y, yp, s);
}

template <int ROWS, int KW0, int... KW>
hipError_t launch_pair_by_kw(std::integer_sequence<int, KW0, KW...>, const float* x, int h, int w, size_t xp, const float* f,
                             int kh, int kw, float* y, size_t yp, hipStream_t s)
{
    static constexpr LaunchStrip table[] = {launch_pair<KW0, ROWS>, launch_pair<KW, ROWS>...};      // widths KW0 and on
    if (kw < KW0 || kw > KW0 + (int)sizeof...(KW)) return hipErrorInvalidValue;
    return table[kw - KW0](x, h, w, xp, f, kh, y, yp, s);
}

}  // namespace

// Output rows of a wavefront of the pair form, 1 to 4, by the wavefronts that one row each would make: one row gives the most of them and the shortest, which
// decides while they do not fill the chip, more rows share input rows and windows.  Lines by groups of columns from 510 random calls, us with 1 / 2 / 3 / 4 rows (wavefronts of one):
//   12 and more   780^2 12x12 (1540) 5.7 / 8.2 / 9.3, 5109x507 14x14 (7644) 12.3 / 11.2 / 13.7, 1493x7018 13x13 (21460) 25.4 / 21.7 / 23.5, 1984x5907 14x13 (24650) 29.1 / 25.0 / 26.8,
//                 3885x6241 13x13 (50388) 53.2 / 43.9 / 42.6
//   10 and 11     1786x1823 10x10 (7120) 8.6 / 8.0 / 9.7 / 9.3, 3709^2 11x10 (27750) 25.6 / 21.4 / 23.8 / 22.6, 8057x2541 10x10 (44264) 32.2 / 25.0 / 29.9 / 27.3, 6517x6174 8x10 (81375) 62.5 / 51.1 / 49.8 / 44.7,
//                 4920x5047 11x11 (54032) 47.2 / 39.2 / 36.5 / 35.7
//   4 to 9        1340^2 8x8 (4002) 5.3 / 5.7 / 6.2 / 6.7, 4846x930 7x7 (9680) 9.0 / 7.9 / 8.2 / 8.3, 4136x1480 7x7 (12390) 11.1 / 10.6 / 9.6 / 9.9, 4095x6001 7x7 (51125) 37.6 / 32.0 / 27.8 / 26.6; even heights gain from
//                 four rows later, when the image no longer fits the memory-side cache (7206^2 8x8 (108000) 85.5 / 65.9 / 59.3 / 55.7)
//   1 to 3        3658x293 15x2 (3644) 6.2 / 5.6 / 6.4 / 6.4; up to 22000 (three columns: 32000, 1541x7211 15x3 (22156) 25.6 / 20.3 / 18.8 / 18.0) as those; 3942^2 9x1 (31472) 20.5 / 15.3 / 18.2 / 19.5, 5767^2 7x2 (66263) 35.5 / 26.3 / 30.8 / 34.8, 7138x3115 13x3 (46319) 37.8 / 26.4 / 28.0 / 31.4; beyond 70000 three rows
//                 (6130^2 14x1 (73416) 74 / 56 / 52 / 54; on 8192 columns two rows are as quick, 10x1 91 / 72 / 77 / 84)
static long long pair_wavefronts(int oh, int ow, int kw)
{
    const int cols = 2 * (kWave - (kw + 1) / 2 / 2);
    return (long long)oh * (((long long)ow + cols - 1) / cols);
}

int conv2d_stride2_pair_rows(int oh, int ow, int kh, int kw)
{
    const long long wavefronts = pair_wavefronts(oh, ow, kw);
    if (wavefronts <= (kw <= 3 ? 3000 : 5000)) return 1;
    if (kw >= 12) return wavefronts <= 40000 ? 2 : 3;
    if (kw >= 10) return wavefronts <= 45000 ? 2 : 4;
    if (kw <= 3) return wavefronts <= 11500 || (wavefronts > (kw == 3 ? 32000 : 22000) && wavefronts <= 70000) ? 2 : 3;
    return wavefronts <= 11500 ? 2 : wavefronts <= (kh % 2 ? 45000 : 70000) ? 3 : 4;
}

// Whether the strips of four outputs a lane take a call: single rows; images of fewer than four columns; and two columns on images that do not fit the memory-side cache (us, pair form with
// its best rows / strips: 7559^2 3x2 58.1 / 56.7, 8x2 68.0 / 63.7, 12x2 77.3 / 70.8, 6200x6300 12x2 53.2 / 49.2, 8192^2 6x2 62.2 / 64.3, 9x2 69.4 / 70.6, 15x2 85.2 / 83.7; with one column and three level or the
// other way round: 7559^2 10x1 70.2 / 72.7, 15x3 81.5 / 79.6).
bool conv2d_stride2_takes_strips(int w, int oh, int ow, int kh, int kw)
{
    return kh == 1 || w < 4 || (kw == 2 && pair_wavefronts(oh, ow, kw) > 70000);
}

// Output rows of a wavefront of the strip form.  Single rows take one at every size (us, three rows / two / one: 1x5 on 3000^2 inputs 8.4 / 8.1 / 6.3, on 8192^2
// 56.6 / 49.5 / 32.9, 1x11 on 4096^2 14.4 / 12.8 / 10.4; 1x14 two / one 13.1 / 10.6), two columns on large images three (12x2 on 7559^2 with two 84, with three 71).  Narrow images have one strip, whose wavefronts are the output
// rows: one row while they do not fill the chip, then two, then three (one / two / three: 3x3 on 6500x3 - / 3.8 / 4.2, 20000x3 6.5 / 5.7 / 5.6, 200000x3 45 / 38 / 32; 9x1 on 20000x3 7.8 / 6.6 / 7.0, 200000x3 56 / 43 / 41; 15x3 on
// 6500x3 7.5 / - / 8.6: from 41 taps on one row up to 4096).
int conv2d_stride2_strip_rows(int w, int oh, int kh, int kw)
{
    if (kh == 1) return 1;
    if (w >= 4 || oh > 100000) return 3;
    return oh <= (kh * kw <= 40 ? 3000 : 4096) ? 1 : 2;
}

hipError_t launch_conv2d_fbs_stride2(const float* x, int h, int w, size_t xp, const float* f, int kh, int kw,
                                     float* y, size_t yp, hipStream_t s)
{
    // Square filters up to 5x5 run the block form, two output rows per wavefront (8192^2, 5x5: 62 us against 70 us for the strips and
    // 56 us for a copy of the same bytes; 150 random shapes: strips of one / two / three rows are 1 to 3 % ahead below 0.3 M outputs in
    // places, 6 to 20 % behind above).
    if (kh == kw && w >= 4) {                                              // (it loads whole quads)
        switch (kh) {
        case 2: return launch_block<2, 2, 2>(x, h, w, xp, f, y, yp, s);
        case 3: return launch_block<3, 3, 2>(x, h, w, xp, f, y, yp, s);
        case 4: return launch_block<4, 4, 2>(x, h, w, xp, f, y, yp, s);
        case 5: return launch_block<5, 5, 2>(x, h, w, xp, f, y, yp, s);
        default: break;
        }
    }
    using Widths = std::integer_sequence<int, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15>;
    const int oh = (h - kh) / 2 + 1, ow = (w - kw) / 2 + 1;
    if (!conv2d_stride2_takes_strips(w, oh, ow, kh, kw)) {
        switch (conv2d_stride2_pair_rows(oh, ow, kh, kw)) {
        case 1: return launch_pair_by_kw<1>(Widths{}, x, h, w, xp, f, kh, kw, y, yp, s);
        case 2: return launch_pair_by_kw<2>(Widths{}, x, h, w, xp, f, kh, kw, y, yp, s);
        case 3:
            if (kw >= 12) return launch_pair_by_kw<3>(std::integer_sequence<int, 12, 13, 14, 15>{}, x, h, w, xp, f, kh, kw, y, yp, s);
            return launch_pair_by_kw<3>(std::integer_sequence<int, 1, 2, 3, 4, 5, 6, 7, 8, 9>{}, x, h, w, xp, f, kh, kw, y, yp, s);
        default: return launch_pair_by_kw<4>(std::integer_sequence<int, 4, 5, 6, 7, 8, 9, 10, 11>{}, x, h, w, xp, f, kh, kw, y, yp, s);
        }
    }
    using Narrow = std::integer_sequence<int, 1, 2, 3>;
    switch (conv2d_stride2_strip_rows(w, oh, kh, kw)) {
    case 1: return launch_strip_by_kw<1>(Widths{}, x, h, w, xp, f, kh, kw, y, yp, s);
    case 2: return launch_strip_by_kw<2>(Narrow{}, x, h, w, xp, f, kh, kw, y, yp, s);
    default: return launch_strip_by_kw<3>(Narrow{}, x, h, w, xp, f, kh, kw, y, yp, s);
    }
}

}  // namespace sysconv
