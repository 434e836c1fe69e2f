// 2-D valid convolution with stride 2 on both axes,
//     y[r][c] = sum_p sum_q x[2r+p][2c+q] * f[p][q],
// as the FBS design: the stride-2 FBS array of Table 2 (row 3 right) along the image
// columns, one 1-D pass per filter row as in the stride-1 2-D FBS kernel (Section 6.2),
// all passes adding into the same partial sums.
//
// A workgroup stages a (2*(4*RPW-1) + kh) x 512 input tile in LDS; each of its four
// wavefronts owns RPW output rows.  For filter row p a lane reads eight consecutive
// inputs of image row 2r+p -- x(2c) and x(2c+1) of its four PEs -- and the even and the
// odd taps of that filter row then run as two stride-1 FBS chains over the
// de-interleaved values (the hand-over X(c,q) = X(c+1,q-2) never mixes the two).
//
//   conv2d_fbs_stride2_kernel<RPW>            any filter up to 15x15: the LDS tiles described above
//   conv2d_fbs_stride2_block_kernel<K,K,ROWS> 2x2 .. 5x5: all input rows of two output rows up front
//   conv2d_fbs_stride2_strip_kernel<KW,ROWS>  any height: rows streamed through registers, where the tiles do not
//                                             fit the chip in one round (conv2d_stride2_strip_rows)
#include "launch.h"
#include "systolic.h"
#include "tiling.h"

#include <utility>

namespace sysconv {
namespace {

typedef const float __attribute__((address_space(4)))* kernarg_floats;

constexpr int kCols = 2 * kStrip;                        // input columns of a tile (eight per lane)
constexpr int kRowTaps = 20;                             // per filter row: 8 even taps, 8 odd taps, 4 of slack
struct TapsStride2D { float f[kMaxK2D * kRowTaps]; };

template <int NT, bool MORE, int RPW>
__device__ __forceinline__ void chain_rows(float (&e)[RPW][4], float (&acc)[RPW][4], const float (&w)[4])
{
#pragma unroll
    for (int j = 0; j < RPW; ++j) fbs_steps<NT, MORE>(e[j], acc[j], w);
}

// All kc >= 1 time steps of one chain of one filter row, for the RPW rows of a wavefront.
template <int RPW>
__device__ __forceinline__ void run_chain(float (&e)[RPW][4], float (&acc)[RPW][4], kernarg_floats w, int kc)
{
    int j = 0;
#pragma nounroll
    for (; j + 4 < kc; j += 4) {
        const float wb[4] = {w[j], w[j + 1], w[j + 2], w[j + 3]};
        chain_rows<4, true, RPW>(e, acc, wb);
    }
    const float wb[4] = {w[j], w[j + 1], w[j + 2], w[j + 3]};
    switch (kc - j) {                                    // uniform across the wavefront
    case 4: chain_rows<4, false, RPW>(e, acc, wb); break;
    case 3: chain_rows<3, false, RPW>(e, acc, wb); break;
    case 2: chain_rows<2, false, RPW>(e, acc, wb); break;
    default: chain_rows<1, false, RPW>(e, acc, wb); break;
    }
}

// The taps are the first kernel argument (offset 0 of the kernel-argument segment).
template <int RPW>
__global__ __launch_bounds__(kBlock) void conv2d_fbs_stride2_kernel(TapsStride2D taps, const float* __restrict__ x,
                                                                    float* __restrict__ y, int h, int w_img,
                                                                    long long xp, int oh, int ow, long long yp,
                                                                    int kh, int kw, int tiles_y, int n_tiles, int side,
                                                                    int per_xcd)
{
    extern __shared__ __attribute__((aligned(16))) float tile[];           // (2*(kTileRows-1) + kh) x kCols
    constexpr int kTileRows = RPW * (kBlock / kWave);                      // output rows per workgroup
    (void)taps;
    kernarg_floats tw = (kernarg_floats)__builtin_amdgcn_kernarg_segment_ptr();

    const int t = xcd_contiguous(blockIdx.x, per_xcd);
    if (t >= n_tiles) return;                                              // whole workgroup leaves together
    int tile_y, tile_x;
    band_order(t, tiles_y, n_tiles / tiles_y, side, tile_y, tile_x);
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = wave_in_block();
    const int ke = (kw + 1) / 2, ko = kw / 2;                              // even taps q = 0, 2, ..; odd taps q = 1, 3, ..
    const int valid_lanes = kWave - halo_lanes(ke);
    const int out_col0 = tile_x * kTile * valid_lanes;
    const int out_row0 = tile_y * kTileRows;
    const int in_col0 = 2 * out_col0, in_row0 = 2 * out_row0;

    // stage: wavefront v copies input rows v, v+4, ... of the tile (2 KB each, coalesced)
    const int in_rows = min(2 * (kTileRows - 1) + kh, h - in_row0);
    for (int rr = wave; rr < in_rows; rr += kBlock / kWave) {
        const float* src = x + (long long)(in_row0 + rr) * xp;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            float v[4];
            load4_guarded<false>(src, in_col0 + half * kStrip + kTile * lane, w_img, v);
            f4 t4;
            t4.x = v[0]; t4.y = v[1]; t4.z = v[2]; t4.w = v[3];
            *reinterpret_cast<f4*>(tile + rr * kCols + half * kStrip + kTile * lane) = t4;
        }
    }
    __syncthreads();

    float acc[RPW][4];
#pragma unroll
    for (int j = 0; j < RPW; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[j][i] = 0.0f;

    const int lrow0 = wave * RPW;
#pragma nounroll
    for (int p = 0; p < kh; ++p) {
        float ev[RPW][4], od[RPW][4];
#pragma unroll
        for (int j = 0; j < RPW; ++j) {
            // rows below the staged part of the tile hold stale LDS; they only feed
            // output rows >= oh, which are not stored
            const float* row = tile + (2 * (lrow0 + j) + p) * kCols + 2 * kTile * lane;
            const f4 lo = *reinterpret_cast<const f4*>(row), hi = *reinterpret_cast<const f4*>(row + 4);
            ev[j][0] = lo.x; od[j][0] = lo.y; ev[j][1] = lo.z; od[j][1] = lo.w;
            ev[j][2] = hi.x; od[j][2] = hi.y; ev[j][3] = hi.z; od[j][3] = hi.w;
        }
        kernarg_floats fp = tw + p * kRowTaps;
        run_chain<RPW>(ev, acc, fp, ke);
        if (ko > 0) run_chain<RPW>(od, acc, fp + 8, ko);
    }

    if (lane < valid_lanes) {
#pragma unroll
        for (int j = 0; j < RPW; ++j) {
            const int r = out_row0 + lrow0 + j;
            if (r < oh) store4_guarded(y + (long long)r * yp, out_col0 + kTile * lane, ow, acc[j]);
        }
    }
}

// Row of a strip from the lanes' load order (lane l: columns 4l .. 4l+3 of the strip's first and second half, so that a
// load is 1 KB of consecutive addresses) to the array's (lane l: columns 8l .. 8l+7, four PEs), through 2 KB of LDS that
// belong to the wavefront.  Loaded straight by the lanes that need them, every cache line was asked for twice (us,
// before / with the exchange: 8192^2 5x5 68.4 / 62.0, 4x4 65.3 / 59.8; 4095x6001 5x5 30.6 / 26.3).  In the strip form
// below, whose row loop waits for each exchange, it costs more than it gives (4095x6001 7x7 35.9 / 38.1).
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
// For the small square filters of the paper's experiment (Section 6) the same array
// without staged tiles: a wavefront takes ROWS output rows of a strip of 512 input columns,
// requests all 2*(ROWS-1)+KH input rows up front (four consecutive inputs of either half of
// a row per lane) and then, input row by input row, passes the row through its own 2 KB of
// LDS (exchange_row), builds the shifted windows of the even and of the odd chain once and applies them to every output row whose filter covers that input
// row (p = rho - 2r).  Strips overlap like the tiles above: the PEs whose even chain
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

    float v[NIN][8];
#pragma unroll
    for (int rho = 0; rho < NIN; ++rho) {
        // rows past the end of the block repeat its last row; they only feed output rows
        // that are not stored
        const float* p = xrow + (long long)min(rho, rows_in - 1) * xp;
        if (EDGE) {
            float lo[4], hi[4];
            load4_guarded<false>(p, in_col, w_img, lo);
            load4_guarded<false>(p, in_col + kSecond, w_img, hi);
#pragma unroll
            for (int i = 0; i < 4; ++i) { v[rho][i] = lo[i]; v[rho][4 + i] = hi[i]; }
        } else {
            const f4u lo = *reinterpret_cast<const f4u*>(p + in_col), hi = *reinterpret_cast<const f4u*>(p + in_col + kSecond);
            v[rho][0] = lo.x; v[rho][1] = lo.y; v[rho][2] = lo.z; v[rho][3] = lo.w;
            v[rho][4] = hi.x; v[rho][5] = hi.y; v[rho][6] = hi.z; v[rho][7] = hi.w;
        }
    }

    float acc[ROWS][4];
#pragma unroll
    for (int rho = 0; rho < NIN; ++rho) {
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
__global__ __launch_bounds__(kBlock) void conv2d_fbs_stride2_block_kernel(Taps2D taps, const float* __restrict__ x,
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
    // A right-hand strip more than half full of a 2x2 filter loads straight to the lanes: where every load is checked, four rows do
    // not make up for the exchange (us, straight / exchanged: 266x1790 outputs 5.1 / 6.1, 1211x673 6.2 / 6.8, 442x3324 7.5 / 8.2; but
    // half full and less 1221x284 6.1 / 5.3, 254x1656 5.2 / 4.9; level on 4 M outputs).
    float* const own = slots[wave_in_block()];
    if (2 * out_col0 + kCols <= w_img)
        stride2_block_rows<KH, KW, ROWS, false, true>(tf, xrow, yrow, in_col, out_col, w_img, xp, ow, yp, rows_out,
                                                      lane_valid, own, lane);
    else if (KH == 2 && 2 * out_col0 + kStrip < w_img)
        stride2_block_rows<KH, KW, ROWS, true, KH != 2>(tf, xrow, yrow, in_col, out_col, w_img, xp, ow, yp, rows_out,
                                                        lane_valid, own, lane);
    else
        stride2_block_rows<KH, KW, ROWS, true, true>(tf, xrow, yrow, in_col, out_col, w_img, xp, ow, yp, rows_out,
                                                     lane_valid, own, lane);
}

template <int KH, int KW, int ROWS>
hipError_t launch_block(const float* x, int h, int w, size_t xp, const float* f, float* y, size_t yp, hipStream_t s)
{
    Taps2D taps;
    for (int i = 0; i < kTaps2DLen; ++i) taps.f[i] = i < KH * KW ? f[i] : 0.0f;
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
// Any filter height at run time, the width at compile time: a wavefront takes ROWS output rows of a strip of 512
// input columns and walks down its 2*(ROWS-1)+kh input rows, kAhead of them in flight in registers.  Each row's two
// windows are built once and applied to every output row whose filter covers it, where the tiles build them again for
// every (output row, filter row) and step through the taps four at a time.  What bounds it is the latency of its input rows:
// on 4095x6001 7x7 (three rows, 32.4 us) the vector ALUs are busy for 30 %, 1.9 wavefronts a SIMD are resident of the four that
// 116 registers allow, and the rows requested, (2 (ROWS-1) + kh) / (2 ROWS) = 1.83 times the image, come from L2 but for 1.25 times.
constexpr int kAhead = 4;

template <int KW, int ROWS, bool EDGE>
__device__ __forceinline__ void stride2_strip_rows(kernarg_floats taps_f, const float* __restrict__ xrow,
                                                   float* __restrict__ yrow, int in_col, int out_col, int w_img,
                                                   long long xp, int ow, long long yp, int kh, int rows_out,
                                                   bool lane_valid)
{
    constexpr int KE = (KW + 1) / 2, KO = KW / 2;
    const int rows_in = 2 * (rows_out - 1) + kh;

    float v[kAhead][8];
    auto load_row = [&](int rho, float (&d)[8]) {                          // past the last row: the last row again
        const float* p = xrow + (long long)min(rho, rows_in - 1) * xp;
        if (EDGE) {
            float lo[4], hi[4];
            load4_guarded<false>(p, in_col, w_img, lo);
            load4_guarded<false>(p, in_col + 4, w_img, hi);
#pragma unroll
            for (int i = 0; i < 4; ++i) { d[i] = lo[i]; d[4 + i] = hi[i]; }
        } else {
            const f4u lo = *reinterpret_cast<const f4u*>(p + in_col), hi = *reinterpret_cast<const f4u*>(p + in_col + 4);
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
__global__ __launch_bounds__(kBlock) void conv2d_fbs_stride2_strip_kernel(Taps2D taps, const float* __restrict__ x,
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
    if (2 * out_col0 + kCols <= w_img)
        stride2_strip_rows<KW, ROWS, false>(tf, xrow, yrow, in_col, out_col, w_img, xp, ow, yp, kh, rows_out, lane_valid);
    else
        stride2_strip_rows<KW, ROWS, true>(tf, xrow, yrow, in_col, out_col, w_img, xp, ow, yp, kh, rows_out, lane_valid);
}

template <int KW, int ROWS>
hipError_t launch_strip(const float* x, int h, int w, size_t xp, const float* f, int kh, float* y, size_t yp, hipStream_t s)
{
    Taps2D taps;
    for (int i = 0; i < kTaps2DLen; ++i) taps.f[i] = i < kh * KW ? f[i] : 0.0f;
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

typedef hipError_t (*LaunchStrip)(const float*, int, int, size_t, const float*, int, float*, size_t, hipStream_t);
template <int ROWS, int KW0, int... KW>
hipError_t launch_strip_by_kw(std::integer_sequence<int, KW0, KW...>, const float* x, int h, int w, size_t xp, const float* f,
                              int kh, int kw, float* y, size_t yp, hipStream_t s)
{
    static constexpr LaunchStrip table[] = {launch_strip<KW0, ROWS>, launch_strip<KW, ROWS>...};    // widths KW0 and on
    if (kw < KW0 || kw > KW0 + (int)sizeof...(KW)) return hipErrorInvalidValue;
    return table[kw - KW0](x, h, w, xp, f, kh, y, yp, s);
}

constexpr int kTileRpw = 2;                              // output rows of a wavefront in the tiles
constexpr int kTileOutRows = kTileRpw * (kBlock / kWave);
constexpr int kCus = 256, kLdsPerCu = 160 * 1024;

template <int RPW>
hipError_t launch_tiles(const float* x, int h, int w, size_t xp, const float* f, int kh, int kw, float* y, size_t yp,
                        hipStream_t s)
{
    constexpr int tile_rows = RPW * (kBlock / kWave);
    TapsStride2D taps;
    for (int i = 0; i < kMaxK2D * kRowTaps; ++i) taps.f[i] = 0.0f;
    for (int p = 0; p < kh; ++p)
        for (int q = 0; q < kw; ++q) taps.f[p * kRowTaps + (q & 1) * 8 + q / 2] = f[p * kw + q];
    const int oh = (h - kh) / 2 + 1, ow = (w - kw) / 2 + 1;
    const int cols = kTile * (kWave - halo_lanes((kw + 1) / 2));
    const int tiles_x = (ow + cols - 1) / cols;
    const int tiles_y = (oh + tile_rows - 1) / tile_rows;
    const long long n_tiles = (long long)tiles_x * tiles_y;
    const long long per_xcd = (n_tiles + kXcds - 1) / kXcds;
    const long long blocks = per_xcd * kXcds;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    const size_t lds = (size_t)(2 * (tile_rows - 1) + kh) * kCols * sizeof(float);
    hipLaunchKernelGGL(conv2d_fbs_stride2_kernel<RPW>, dim3((unsigned)blocks), dim3(kBlock), lds, s,
                       taps, x, y, h, w, (long long)xp, oh, ow, (long long)yp, kh, kw, tiles_y, (int)n_tiles,
                       band_width(xp), (int)per_xcd);
    return hipGetLastError();
}

}  // namespace

// Filters without a block form: 0 = tiles, else the rows of the strips.  Tiles as long as their workgroups fit the chip in one
// round, else strips (us, tiles / strips of 2 / of 3 rows).  A tile takes 2 (4 RPW - 1) + kh rows of 2 KB of the 160 KB of LDS
// of a CU: five workgroups (kh = 2) to two (kh = 13 and more), so a round ends at 2.5 M to 1.0 M outputs, and there the tiles'
// time jumps: 7x7 on 769x1865 outputs 18.2 / 13.7 / 14.7, 13x13 on 654x1920 30.3 / 21.6 / 24.7.  Below, four wavefronts share the
// staging of a tile's rows: 6x3 on 1137x1676 outputs 11.8 / 14.5 / 15.6, 2x5 on 2910x100 6.0 / 7.2 / 8.5, 10x1 on 1529x800
// 10.4 / 12.6 / 13.5.  Wide filters on about a workgroup a CU, or up to two with many taps, are the exception, as a row's windows
// are built once instead of per filter row (300x400 inputs: 15x15 16.6 / 14.4 / 21.0, 9x9 9.9 / 9.1 / 10.9; outputs 109x3025 6x8
// 9.6 / 8.1, 257x1857 14x14 19.3 / 17.1, but 822x416 6x6 9.3 / 8.8 and 1024x518 10x7 12.5 / 11.9 are left to the tiles: smaller
// filters and more tiles lose as often).  Above: 8192^2 inputs 7x7 126 / 92 / 85, 11x11 165 / 125 / 117, 15x15 303 / 167 / 179,
// 13x4 198 / 118 / 108, 2x15 78 / 73 / 78.
// Three rows read fewer halo rows and need images large enough to fill the chip with fewer wavefronts, and not too many taps
// (4 M to 20 M outputs, 2 rows / 3 rows: up to 11 columns 1.01 to 1.07, 10 and 11 among them although up to nine scalar
// registers of taps spill; 12 columns and more 0.9 to 1.0).  Of 2250 random shapes 29 are slower by 3 % or more than with tiles
// alone, most of them within the noise of two runs; with a line at 0.4 M outputs and four columns it was 419, by up to 18 %.
int conv2d_stride2_strip_rows(int oh, int ow, int kh, int kw)
{
    const int cols = kTile * (kWave - halo_lanes((kw + 1) / 2));
    const long long tiles = (((long long)oh + kTileOutRows - 1) / kTileOutRows) * (((long long)ow + cols - 1) / cols);
    const int tiles_a_cu = kLdsPerCu / ((2 * (kTileOutRows - 1) + kh) * kCols * (int)sizeof(float));
    const double few = 2.4 * kh * kw;                                      // tiles
    const bool heavy = kw >= 6 && kh * kw >= 42 && (tiles <= kCus || (tiles <= 2 * kCus && (double)tiles <= few));
    if (tiles <= (long long)kCus * tiles_a_cu && !heavy) return 0;
    return kw > 1 && kw <= 11 && (double)oh * ow >= 4e6 ? 3 : 2;
}

hipError_t launch_conv2d_fbs_stride2(const float* x, int h, int w, size_t xp, const float* f, int kh, int kw,
                                     float* y, size_t yp, hipStream_t s)
{
    // Square filters up to 5x5 run the block form, two output rows per wavefront (8192^2, 5x5: 62 us against 75 - 82 us
    // for the strips, 88 us for the LDS tiles and 56 us for a copy of the same bytes; 1, 3 and 4 rows, before the exchange of
    // the loads took two rows from 68 to 62 us: 83, 68, 74).
    if (kh == kw) {
        switch (kh) {
        case 2: return launch_block<2, 2, 2>(x, h, w, xp, f, y, yp, s);
        case 3: return launch_block<3, 3, 2>(x, h, w, xp, f, y, yp, s);
        case 4: return launch_block<4, 4, 2>(x, h, w, xp, f, y, yp, s);
        case 5: return launch_block<5, 5, 2>(x, h, w, xp, f, y, yp, s);
        default: break;
        }
    }
    switch (conv2d_stride2_strip_rows((h - kh) / 2 + 1, (w - kw) / 2 + 1, kh, kw)) {
    case 0: return launch_tiles<kTileRpw>(x, h, w, xp, f, kh, kw, y, yp, s);
    case 3:
        return launch_strip_by_kw<3>(std::integer_sequence<int, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11>{}, x, h, w, xp, f, kh, kw, y, yp, s);
    default:
        return launch_strip_by_kw<2>(std::integer_sequence<int, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15>{}, x, h, w, xp, f,
                                     kh, kw, y, yp, s);
    }
}

}  // namespace sysconv
