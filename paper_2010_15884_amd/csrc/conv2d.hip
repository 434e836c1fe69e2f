// 2-D valid convolution  y[r][c] = sum_p sum_q x[r+p][c+q] * f[p][q]  (paper
// Eq. 3; the paper's systolic axis c,q is the image column) as software
// systolic arrays.  A wavefront always works on a strip of 256 consecutive
// input columns held four per lane.  In the FBS and SBM kernels neighbouring
// strips overlap by 4*halo_lanes(kw) columns and the PEs whose taps reach past
// the strip compute values that are never stored; the BFS kernels' strips do
// not overlap and fetch the kw-1 columns to their right separately.
//
//   conv2d_fbs_static_kernel<KH,KW,R> min(kh, kw) <= 7: LDS tile, sizes known at compile time, each staged row's window shared by the rows it feeds
//   conv2d_fbs_strip_kernel<KW,ROWS>  8 .. 15 columns, any height: input rows streamed through registers
//   conv2d_bfs_block_kernel<K,K,ROWS> 2x2 .. 7x7: short row block, all loads up front
//   conv2d_bfs_kernel<K,K,PD>         8x8 .. 11x11: strip walk with rows in flight
//   conv2d_sbm_block_kernel<K,K,ROWS> 2x2 .. 7x7
//   conv2d_sbm_kernel<K,K,PD>         8x8 .. 11x11
#include "launch.h"
#include "systolic.h"
#include "tiling.h"

#include <stdlib.h>

#include <type_traits>

namespace sysconv {
namespace {

// ------------------------------------------------------------- FBS 2-D -----
// Section 6.2 describes the 2-D FBS design as a set of 1-D FBS convolutions, one per
// filter row, that add into the same partial sums.  Filters whose smaller side is at most 7 run the tile kernel below, all others the strips
// (conv2d_fbs_strip_kernel).

// Pointer into the kernel-argument segment (constant address space: uniform
// reads become scalar loads).
typedef const float __attribute__((address_space(4)))* kernarg_floats;

// A workgroup stages a (4 RPW + KH - 1) x 256 input tile in LDS; each of its four wavefronts owns RPW output rows.  The filter size is known at compile time
// (has_conv2d_fbs_static): every loop below is unrolled, the taps sit in SGPRs for the whole kernel, and the 1-D passes are taken
// input row by input row -- the array hands a staged row's inputs on from PE to PE once
// (KW-1 DPP moves) and each of the up to min(RPW, KH) output rows that the input row feeds
// takes its KW products from that one window, so the hand-overs are shared between the 1-D
// convolutions instead of repeated per filter row.
// Lanes of a strip that keep their results.  Single-row filters move as many bytes as a copy, and
// there strips that start on 64-byte boundaries measure faster (8192^2, 1x5: 98.8 -> 91.5 us), as in
// the 1-D kernels; with taller filters, and rows of more than 11 taps, the rounding does not pay.
__host__ __device__ constexpr int fbs_static_valid_lanes(int kh, int kw)
{
    return kh == 1 && kw <= 11 ? ((kWave - halo_lanes(kw)) & ~3) : kWave - halo_lanes(kw);
}

template <int KH, int KW, int RPW>
__global__ __launch_bounds__(kBlock) void conv2d_fbs_static_kernel(TapsOf<KH * KW> taps, const float* __restrict__ x,
                                                                   float* __restrict__ y, int h, int w_img,
                                                                   long long xp, int oh, int ow, long long yp,
                                                                   int tiles_y, int n_tiles, int side, int per_xcd)
{
    (void)taps;
    constexpr int kTileRows = RPW * (kBlock / kWave);                      // output rows per workgroup
    constexpr int kInRows = kTileRows + KH - 1;
    __shared__ __attribute__((aligned(16))) float tile[kInRows * kStrip];
    kernarg_floats taps_f = (kernarg_floats)__builtin_amdgcn_kernarg_segment_ptr();

    const int t = xcd_contiguous(blockIdx.x, per_xcd);
    if (t >= n_tiles) return;                                              // whole workgroup leaves together
    int tile_y, tile_x;
    band_order(t, tiles_y, n_tiles / tiles_y, side, tile_y, tile_x);
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = wave_in_block();
    constexpr int valid_lanes = fbs_static_valid_lanes(KH, KW);
    const int col0 = tile_x * kTile * valid_lanes;
    const int row0 = tile_y * kTileRows;

    // stage: wavefront v copies input rows v, v+4, ... of the tile; all its loads go out first
    const int last_row = h - 1 - row0;                                     // rows past the image repeat its last row
    constexpr int kPerWave = (kInRows + 3) / 4;
    float stage[kPerWave][4];
    auto stage_row = [&](int k) { return x + (long long)(row0 + min(wave + 4 * k, last_row)) * xp; };
    if (KW >= 4 || w_img >= 4) {                                           // uniform
        const EdgeQuad quad(col0 + kTile * lane, w_img);
#pragma unroll
        for (int k = 0; k < kPerWave; ++k) {
            const f4u t = *reinterpret_cast<const f4u*>(stage_row(k) + quad.at);
            stage[k][0] = t.x; stage[k][1] = t.y; stage[k][2] = t.z; stage[k][3] = t.w;
        }
        if (col0 + kStrip > w_img) {                                       // uniform
            asm volatile("");                                              // a branch, not selects in every strip
#pragma unroll
            for (int k = 0; k < kPerWave; ++k) quad.put_right(stage[k][0], stage[k][1], stage[k][2], stage[k][3]);
        }
    } else {
#pragma unroll
        for (int k = 0; k < kPerWave; ++k) load4_guarded<false>(stage_row(k), col0 + kTile * lane, w_img, stage[k]);
    }
#pragma unroll
    for (int k = 0; k < kPerWave; ++k) {
        const int rr = wave + 4 * k;
        if (rr < kInRows) {
            f4 t4;
            t4.x = stage[k][0]; t4.y = stage[k][1]; t4.z = stage[k][2]; t4.w = stage[k][3];
            *reinterpret_cast<f4*>(tile + rr * kStrip + kTile * lane) = t4;
        }
    }
    __syncthreads();

    float acc[RPW][4];
    const int lrow0 = wave * RPW;
#pragma unroll
    for (int rho = 0; rho < RPW + KH - 1; ++rho) {
        float win[KW + 3];
        const f4 t4 = *reinterpret_cast<const f4*>(tile + (lrow0 + rho) * kStrip + kTile * lane);
        win[0] = t4.x; win[1] = t4.y; win[2] = t4.z; win[3] = t4.w;
#pragma unroll
        for (int m = 4; m < KW + 3; ++m) win[m] = from_lane_above(win[m - 4]);   // X(c) <- X(c+1), once per row
#pragma unroll
        for (int j = 0; j < RPW; ++j) {
            const int p = rho - j;                                         // compile-time
            if (p < 0 || p >= KH) continue;
#pragma unroll
            for (int q = 0; q < KW; ++q) {
                const float wv = taps_f[p * KW + q];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (p == 0 && q == 0) acc[j][i] = wv * win[i];
                    else acc[j][i] = __builtin_fmaf(wv, win[q + i], acc[j][i]);
                }
            }
        }
    }

    if (lane < valid_lanes) {
#pragma unroll
        for (int j = 0; j < RPW; ++j) {
            const int r = row0 + lrow0 + j;
            if (r < oh) store4_guarded(y + (long long)r * yp, col0 + kTile * lane, ow, acc[j]);
        }
    }
}

// A zero the optimiser cannot see through (one SALU move).
__device__ __forceinline__ int opaque_zero()
{
    int z;
    asm volatile("s_mov_b32 %0, 0" : "=s"(z));
    return z;
}

// ------------------------------------------------------------- BFS 2-D -----
// Along the rows the array is the BFS design of Table 2 (row 2 left) with
// (c, q) read as (r, p): PE = output row, time = input row rho = r + p.  The
// PEs are the KH live partial-sum vectors of a lane; at step rho the input row
// rho is broadcast to all of them, PE r applies filter row p = rho - r (the
// weights move one PE per step while the partial sums stay), and the PE whose
// last filter row was just applied retires its output row.  Along a row the
// KW-wide window of every PE is built once by KW-1 FBS hand-overs and reused
// by all KH filter rows, so lane traffic is amortised KH times.  Everything
// streams from global memory through registers: no LDS.
//
// A wavefront walks `rows` output rows of one strip; PD input rows are in
// flight ahead of the one being consumed (PD divides KH so that the slot of a
// row in the prefetch ring is a compile-time constant of the unrolled loop).
// A strip that reaches past the right edge of the image checks its stores per lane, and its loads in one of two ways: kEdge, where some of its 256
// columns are missing, loads them clamped to the row (EdgeQuad; at least 8 columns here) and has no halo; kNarrow checks every load, which
// costs nothing where the 256 columns are all there.
enum BfsMode { kBfsFirst, kBfsMiddle, kBfsLast, kBfsChecked };

template <int KH, int KW, int PD, StripKind KIND>
struct BfsStrip {
    static_assert(KH % PD == 0, "prefetch depth must divide the filter height");
    static constexpr bool kReloadTaps = KH * KW > 25;
    static constexpr int NH = (KW + 2) / 4;                                // halo float4s: ceil((KW-1)/4)
    static constexpr bool EDGE = KIND != kInside;

    const float* __restrict__ xrow;
    float* __restrict__ yrow;
    int col, w_img, ow, rows_out, rows_in;
    long long xp, yp;
    bool last_lane;                        // lane 63: the lane the halo enters through
    float ring[PD][4];
    float halo[PD][NH][4];                 // meaningful in lane 63 only
    float acc[KH][4];

    __device__ __forceinline__ void load_row(int row, float (&v)[4], float (&h)[NH][4]) const
    {
        // past the end of the strip the last row is read again: an unconditional load
        // keeps the control flow straight and the wait counts exact
        const float* p = xrow + (long long)min(row, rows_in - 1) * xp;
        // Halo: the KW-1 columns right of the strip, fetched by lane 63 alone (one
        // 16-byte access per float4) into the registers that the window hand-overs
        // leave untouched in that lane.
        if (KIND != kEdge && last_lane) {
#pragma unroll
            for (int j = 0; j < NH; ++j) {
                if (KIND == kNarrow) {
                    load4_guarded<false>(p, col + 4 * (j + 1), w_img, h[j]);
                } else {
                    const f4u t = *reinterpret_cast<const f4u*>(p + col + 4 * (j + 1));
                    h[j][0] = t.x; h[j][1] = t.y; h[j][2] = t.z; h[j][3] = t.w;
                }
            }
        }
        if (KIND == kNarrow) {
            load4_guarded<false>(p, col, w_img, v);
            return;
        }
        // plain (cacheable) loads: the KH-1 halo rows are read again by the wavefront
        // working on the next row block and should then come from L2 / the memory-side
        // cache, not from HBM (measured on 4096^2, 5x5: 33 us against 43 us with the
        // non-temporal hint)
        const f4u t = *reinterpret_cast<const f4u*>(p + (KIND == kEdge ? EdgeQuad(col, w_img).at : col));
        v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    }

    // KH consecutive input rows rho0 .. rho0+KH-1 (rho0 a multiple of KH, so every slot
    // index below is a compile-time constant).
    //   kBfsFirst    rho0 == 0: output rows r = rho - p < 0 do not exist (decided statically)
    //   kBfsMiddle   every (rho, p) pair is valid, no checks
    //   kBfsLast     the block that holds the last input row: run-time checks
    //   kBfsChecked  all checks at run time (one loop body for filters whose code is large)
    template <BfsMode MODE>
    __device__ __forceinline__ void block(int rho0, kernarg_floats taps_f)
    {
#pragma unroll
        for (int ph = 0; ph < KH; ++ph) {
            const int rho = rho0 + ph;
            if ((MODE == kBfsLast || MODE == kBfsChecked) && rho >= rows_in) break;

            // window of input row rho: win[m] = x[rho][col + m], m < KW + 3
            float win[KW + 3];
            float hin[NH][4];
#pragma unroll
            for (int i = 0; i < 4; ++i) win[i] = ring[ph % PD][i];
#pragma unroll
            for (int j = 0; j < NH; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i) hin[j][i] = KIND == kEdge ? 0.0f : halo[ph % PD][j][i];
            if (KIND == kEdge) EdgeQuad(col, w_img).put_right(win[0], win[1], win[2], win[3]);
            load_row(rho + PD, ring[ph % PD], halo[ph % PD]);
            // X(c) <- X(c+1): lanes 0..62 take the value of the lane above, lane 63 takes
            // the next halo element
#pragma unroll
            for (int m = 4; m < KW + 3; ++m) win[m] = from_lane_above_or(win[m - 4], hin[(m - 4) / 4][(m - 4) % 4]);

            // broadcast the row to the KH partial-sum vectors it feeds
#pragma unroll
            for (int p = 0; p < KH; ++p) {
                const int slot = (ph - p + KH) % KH;                       // compile-time after unrolling
                const int r = rho - p;
                if (MODE == kBfsFirst && p > ph) continue;
                if (MODE == kBfsChecked && r < 0) continue;
                if ((MODE == kBfsLast || MODE == kBfsChecked) && r >= rows_out) continue;
                // Small filters keep all taps in SGPRs for the whole kernel.  Larger ones
                // would spill them, so each filter row is re-fetched here with scalar
                // loads; the offset is made opaque to keep the loads in the loop.
                kernarg_floats fp = taps_f + p * KW + (kReloadTaps ? opaque_zero() : 0);
#pragma unroll
                for (int q = 0; q < KW; ++q) {
                    const float wv = fp[q];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        // the first tap of the first filter row opens a fresh partial sum
                        if (p == 0 && q == 0) acc[slot][i] = wv * win[i];
                        else acc[slot][i] = __builtin_fmaf(wv, win[q + i], acc[slot][i]);
                    }
                }
            }

            // output row rho-(KH-1) has now seen all its filter rows
            const int done = rho - (KH - 1);
            constexpr int kh1 = KH - 1;
            const int dslot = (ph - kh1 + KH) % KH;
            if (MODE == kBfsFirst && ph < KH - 1) continue;
            if (done >= 0 && done < rows_out) {
                float* yr = yrow + (long long)done * yp;
                if (EDGE) {
                    store4_guarded(yr, col, ow, acc[dslot]);
                } else {
                    f4u t;
                    t.x = acc[dslot][0]; t.y = acc[dslot][1]; t.z = acc[dslot][2]; t.w = acc[dslot][3];
                    if (SYSCONV_NONTEMPORAL_STORE) __builtin_nontemporal_store(t, reinterpret_cast<f4u*>(yr + col));
                    else *reinterpret_cast<f4u*>(yr + col) = t;
                }
            }
        }
    }

    __device__ __forceinline__ void run(kernarg_floats taps_f)
    {
#pragma unroll
        for (int d = 0; d < PD; ++d) load_row(d, ring[d], halo[d]);
#pragma unroll
        for (int s = 0; s < KH; ++s) acc[s][0] = acc[s][1] = acc[s][2] = acc[s][3] = 0.0f;

        if (kReloadTaps) {
            for (int rho0 = 0; rho0 < rows_in; rho0 += KH) block<kBfsChecked>(rho0, taps_f);
        } else {
            // rows_in >= KH always; the last block is the one that contains row rows_in-1
            const int last0 = ((rows_in - 1) / KH) * KH;
            if (last0 == 0) {
                block<kBfsChecked>(0, taps_f);
            } else {
                block<kBfsFirst>(0, taps_f);
                for (int rho0 = KH; rho0 < last0; rho0 += KH) block<kBfsMiddle>(rho0, taps_f);
                block<kBfsLast>(last0, taps_f);
            }
        }
    }
};

// The taps are the FIRST kernel argument, i.e. they sit at offset 0 of the
// kernel-argument segment; reading them through that segment's pointer keeps
// run-time-indexed taps on the scalar load path (indexing the by-value struct
// itself can make the compiler copy it to scratch).
// Two kernels, by the right-hand strips (bfs_strip_right): with clamped columns and halo in one body, inside strips lost registers too (us, guarded
// everywhere / so / this: 8192^2 8x8 159 / 168 / 158, 10x10 217 / 228 / 217, 11x11 254 / 266 / 254, 3001x4003 8x8 38.5 / 37.6 / 34.0, 11x11 67.0 / 59.5 / 57.4,
// 1500^2 8x8 15.1 / 12.9 / 12.5, 501x703 11x11 14.9 / 11.5 / 10.4).
template <int KH, int KW, int PD, StripKind RIGHT>
__global__ __launch_bounds__(kBlock) void conv2d_bfs_kernel(TapsOf<KH * KW> taps, const float* __restrict__ x,
                                                            float* __restrict__ y, int w_img, long long xp, int oh,
                                                            int ow, long long yp, int rows, int row_blocks,
                                                            int strips, int side, int per_xcd, int valid_lanes)
{
    (void)taps;
    (void)valid_lanes;
    kernarg_floats taps_f = (kernarg_floats)__builtin_amdgcn_kernarg_segment_ptr();
    int rb, strip;
    if (!wave_tile(per_xcd, row_blocks, strips, side, rb, strip)) return;
    const int lane = threadIdx.x & (kWave - 1);
    const int col0 = strip * kStrip;                                       // strips are 256 outputs wide
    const int r0 = rb * rows;
    const int rows_out = min(rows, oh - r0);
    const int rows_in = rows_out + KH - 1;
    const float* xrow = x + (long long)r0 * xp;
    float* yrow = y + (long long)r0 * yp;
    const bool last_lane = lane == kWave - 1;
    constexpr int halo_cols = kTile * ((KW + 2) / 4);
    if (col0 + kStrip + halo_cols <= w_img) {
        BfsStrip<KH, KW, PD, kInside> st{xrow, yrow, col0 + kTile * lane, w_img, ow, rows_out, rows_in,
                                       xp, yp, last_lane, {}, {}, {}};
        st.run(taps_f);
    } else {
        BfsStrip<KH, KW, PD, RIGHT> st{xrow, yrow, col0 + kTile * lane, w_img, ow, rows_out, rows_in,
                                      xp, yp, last_lane, {}, {}, {}};
        st.run(taps_f);
    }
}

// ------------------------------------------------------------- SBM 2-D -----
// Section 5 (two projections): PE = c + q, time = p + P*q, the row loop r stays
// outside.  Every PE keeps a KH-tall column of inputs x(r..r+KH-1, s); the
// partial sum of output (r, c) starts at PE c, takes the KH products of filter
// column q there, and moves one PE up each time q advances, so after KH*KW steps
// PE c + KW - 1 holds it.  A wavefront owns a strip of 256 PEs (image columns)
// and walks down the rows with a ring of KH + PD input rows in registers (KH in
// use, PD in flight); the ring is indexed by row mod (KH+PD) and the row loop is
// unrolled that many times so that all indices are compile-time constants.
// Before storing, the result vector is read out KW-1 PEs further down (the
// results of an SBM array start at PE Q-1, Section 3.1), which lines the stores up
// with the loads.  Taps arrive transposed (filter column q contiguous).
template <int KH, int KW, int PD, bool EDGE>
struct SbmStrip {
    static constexpr int RS = KH + PD;                                     // ring size
    static constexpr bool kReloadTaps = KH * KW > 25;

    const float* __restrict__ xrow;
    float* __restrict__ yrow;
    int col, w_img, ow, rows_out, rows_in;
    long long xp, yp;
    bool lane_valid;
    float ring[RS][4];

    __device__ __forceinline__ void load_row(int row, float (&v)[4]) const
    {
        const float* p = xrow + (long long)min(row, rows_in - 1) * xp;
        const f4u t = *reinterpret_cast<const f4u*>(p + (EDGE ? EdgeQuad(col, w_img).at : col));
        v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    }

    // a row that has been loaded, where it is first used
    __device__ __forceinline__ void arrived(float (&v)[4]) const
    {
        if (EDGE) EdgeQuad(col, w_img).put_right(v[0], v[1], v[2], v[3]);
    }

    __device__ __forceinline__ void run(kernarg_floats taps_t)
    {
#pragma unroll
        for (int d = 0; d < RS - 1; ++d) load_row(d, ring[d]);
#pragma unroll
        for (int d = 0; d < KH - 1; ++d) arrived(ring[d]);

        for (int r0 = 0; r0 < rows_out; r0 += RS) {
#pragma unroll
            for (int ph = 0; ph < RS; ++ph) {
                const int r = r0 + ph;
                if (r >= rows_out) break;
                // the slot of row r-1 is free now: fetch row r+KH+PD-1 into it
                load_row(r + RS - 1, ring[(ph + RS - 1) % RS]);
                arrived(ring[(ph + KH - 1) % RS]);

                float z[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int q = 0; q < KW; ++q) {
                    if (q > 0) {                                           // Z(s) <- Z(s-1)
                        const float below = from_lane_below(z[3]);
                        z[3] = z[2]; z[2] = z[1]; z[1] = z[0]; z[0] = below;
                    }
                    kernarg_floats ft = taps_t + q * KH + (kReloadTaps ? opaque_zero() : 0);
#pragma unroll
                    for (int p = 0; p < KH; ++p) {
                        const float wv = ft[p];
#pragma unroll
                        for (int i = 0; i < 4; ++i) z[i] = __builtin_fmaf(wv, ring[(ph + p) % RS][i], z[i]);
                    }
                }
                // read the results out KW-1 PEs further down: PE s gets output column s
#pragma unroll
                for (int t = 0; t < KW - 1; ++t) {
                    const float above = from_lane_above(z[0]);
                    z[0] = z[1]; z[1] = z[2]; z[2] = z[3]; z[3] = above;
                }
                if (lane_valid) {
                    float* yr = yrow + (long long)r * yp;
                    if (EDGE) {
                        store4_guarded(yr, col, ow, z);
                    } else {
                        f4u t;
                        t.x = z[0]; t.y = z[1]; t.z = z[2]; t.w = z[3];
                        if (SYSCONV_NONTEMPORAL_STORE) __builtin_nontemporal_store(t, reinterpret_cast<f4u*>(yr + col));
                        else *reinterpret_cast<f4u*>(yr + col) = t;
                    }
                }
            }
        }
    }
};

template <int KH, int KW, int PD>
__global__ __launch_bounds__(kBlock) void conv2d_sbm_kernel(TapsOf<KH * KW> taps_t, const float* __restrict__ x,
                                                            float* __restrict__ y, int w_img, long long xp, int oh,
                                                            int ow, long long yp, int rows, int row_blocks,
                                                            int strips, int side, int per_xcd, int valid_lanes)
{
    (void)taps_t;
    kernarg_floats tf = (kernarg_floats)__builtin_amdgcn_kernarg_segment_ptr();
    int rb, strip;
    if (!wave_tile(per_xcd, row_blocks, strips, side, rb, strip)) return;
    const int lane = threadIdx.x & (kWave - 1);
    const int col0 = strip * kTile * valid_lanes;
    const int r0 = rb * rows;
    const int rows_out = min(rows, oh - r0);
    const int rows_in = rows_out + KH - 1;
    const float* xrow = x + (long long)r0 * xp;
    float* yrow = y + (long long)r0 * yp;
    const bool lane_valid = lane < valid_lanes;
    if (col0 + kStrip <= w_img) {
        SbmStrip<KH, KW, PD, false> st{xrow, yrow, col0 + kTile * lane, w_img, ow, rows_out, rows_in,
                                       xp, yp, lane_valid, {}};
        st.run(tf);
    } else {
        SbmStrip<KH, KW, PD, true> st{xrow, yrow, col0 + kTile * lane, w_img, ow, rows_out, rows_in,
                                      xp, yp, lane_valid, {}};
        st.run(tf);
    }
}

// ----------------------------------------------------- BFS 2-D, block form ---
// The same BFS-along-rows x FBS-along-columns array as BfsStrip, for filters
// small enough to be bound by memory: a wavefront takes a block of ROWS output
// rows of one 256-column strip, issues the loads of ALL ROWS+KH-1 input rows up
// front, and then runs in straight-line code (no row loop, every validity test
// decided at compile time).  With every load in flight at once a wavefront pays
// one memory latency per block, and the compiler's wait counts are exact.
// The KW-1 halo columns right of the strip are the same for all lanes, so they
// are fetched with uniform (scalar) loads and enter the array in lane 63.
template <int KH, int KW, int ROWS, StripKind KIND>
__device__ __forceinline__ void bfs_block_rows(kernarg_floats taps_f, const float* __restrict__ xrow,
                                               float* __restrict__ yrow, int col0, int lane, int w_img,
                                               long long xp, int ow, long long yp, int rows_out)
{
    constexpr int NIN = ROWS + KH - 1;
    constexpr int NH = (KW + 2) / 4;                                       // halo float4s
    const int col = col0 + kTile * lane;
    const int rows_in = rows_out + KH - 1;
    constexpr bool EDGE = KIND != kInside;
    const EdgeQuad quad(col, w_img);

    float v[NIN][4];
    float h[NIN][NH][4];
#pragma unroll
    for (int rho = 0; rho < NIN; ++rho) {
        // rows past the end of the block repeat its last row; they only feed output rows
        // that are not stored
        const float* p = xrow + (long long)min(rho, rows_in - 1) * xp;
        if constexpr (KIND == kNarrow) {
            load4_guarded<false>(p, col, w_img, v[rho]);
        } else {
            const f4u t = *reinterpret_cast<const f4u*>(p + (EDGE ? quad.at : col));
            v[rho][0] = t.x; v[rho][1] = t.y; v[rho][2] = t.z; v[rho][3] = t.w;
        }
        const float* hp = p + col0 + kStrip;                               // wave-uniform address
#pragma unroll
        for (int j = 0; j < NH; ++j) {
            if constexpr (EDGE) {
                load4_guarded<false>(p, col0 + kStrip + 4 * j, w_img, h[rho][j]);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) h[rho][j][i] = hp[4 * j + i];
            }
        }
    }

    float acc[ROWS][4];
#pragma unroll
    for (int rho = 0; rho < NIN; ++rho) {
        if constexpr (KIND == kEdge) quad.put_right(v[rho][0], v[rho][1], v[rho][2], v[rho][3]);
        float win[KW + 3];
#pragma unroll
        for (int i = 0; i < 4; ++i) win[i] = v[rho][i];
#pragma unroll
        for (int m = 4; m < KW + 3; ++m)
            win[m] = from_lane_above_or(win[m - 4], h[rho][(m - 4) / 4][(m - 4) % 4]);
#pragma unroll
        for (int p = 0; p < KH; ++p) {
            const int r = rho - p;                                         // compile-time
            if (r < 0 || r >= ROWS) continue;
#pragma unroll
            for (int q = 0; q < KW; ++q) {
                const float wv = taps_f[p * KW + q];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (p == 0 && q == 0) acc[r][i] = wv * win[i];
                    else acc[r][i] = __builtin_fmaf(wv, win[q + i], acc[r][i]);
                }
            }
        }
        const int done = rho - (KH - 1);
        if (done >= 0 && done < rows_out) {
            float* yr = yrow + (long long)done * yp;
            if (EDGE) {
                store4_guarded(yr, col, ow, acc[done]);
            } else {
                f4u t;
                t.x = acc[done][0]; t.y = acc[done][1]; t.z = acc[done][2]; t.w = acc[done][3];
                if (SYSCONV_NONTEMPORAL_STORE) __builtin_nontemporal_store(t, reinterpret_cast<f4u*>(yr + col));
                else *reinterpret_cast<f4u*>(yr + col) = t;
            }
        }
    }
}

// Two kernels, by how the right-hand strips load: kNarrow (every load checked) where the width is a multiple of four, as whole quads end at the edge and
// nobody waits (4096^2 5x5 with clamped loads 24.0 / 24.9 us), and below four columns; kEdge elsewhere.  Both bodies in one kernel cost the
// first registers (us, one kernel / two: 1024^2 7x7 6.01 / 5.87, 2048^2 5x5 9.25 / 9.17, 4096^2 5x5 23.82 / 23.56, 7x7 33.35 / 32.92, 8192^2 5x5 103.6 / 102.2; others level).
template <int KH, int KW, int ROWS, StripKind RIGHT>
__global__ __launch_bounds__(kBlock) void conv2d_bfs_block_kernel(TapsOf<KH * KW> taps, const float* __restrict__ x,
                                                                  float* __restrict__ y, int w_img, long long xp,
                                                                  int oh, int ow, long long yp, int row_blocks,
                                                                  int strips, int side, int per_xcd, int wide)
{
    (void)taps;
    kernarg_floats taps_f = (kernarg_floats)__builtin_amdgcn_kernarg_segment_ptr();
    int rb, strip;
    if (wide) {
        if (!wave_tile_wide(per_xcd, row_blocks, strips, rb, strip)) return;
    } else {
        if (!wave_tile(per_xcd, row_blocks, strips, side, rb, strip)) return;
    }
    const int lane = threadIdx.x & (kWave - 1);
    const int col0 = strip * kStrip;
    const int r0 = rb * ROWS;
    const int rows_out = min(ROWS, oh - r0);
    const float* xrow = x + (long long)r0 * xp;
    float* yrow = y + (long long)r0 * yp;
    constexpr int halo_cols = kTile * ((KW + 2) / 4);
    if (col0 + kStrip + halo_cols <= w_img)
        bfs_block_rows<KH, KW, ROWS, kInside>(taps_f, xrow, yrow, col0, lane, w_img, xp, ow, yp, rows_out);
    else
        bfs_block_rows<KH, KW, ROWS, RIGHT>(taps_f, xrow, yrow, col0, lane, w_img, xp, ow, yp, rows_out);
}

// ----------------------------------------------------- SBM 2-D, block form ---
// The SBM array of SbmStrip (PE = c + q, time = p + P*q) in the block form of
// bfs_block_rows: the ROWS+KH-1 input rows of a block of ROWS output rows are all
// requested up front and the output rows are then computed one after the other in
// straight-line code.  Taps arrive transposed (filter column q contiguous).
template <int KH, int KW, int ROWS, StripKind KIND>
__device__ __forceinline__ void sbm_block_rows(kernarg_floats taps_t, const float* __restrict__ xrow,
                                               float* __restrict__ yrow, int col, int w_img, long long xp, int ow,
                                               long long yp, int rows_out, bool lane_valid)
{
    constexpr int NIN = ROWS + KH - 1;
    constexpr bool kReloadTaps = KH * KW > 25;
    const int rows_in = rows_out + KH - 1;
    constexpr bool EDGE = KIND != kInside;
    const EdgeQuad quad(col, w_img);

    float v[NIN][4];
#pragma unroll
    for (int rho = 0; rho < NIN; ++rho) {
        // rows past the end of the block repeat its last row; they only feed output rows
        // that are not stored
        const float* p = xrow + (long long)min(rho, rows_in - 1) * xp;
        if constexpr (KIND == kNarrow) {
            load4_guarded<false>(p, col, w_img, v[rho]);
        } else {
            const f4u t = *reinterpret_cast<const f4u*>(p + (EDGE ? quad.at : col));
            v[rho][0] = t.x; v[rho][1] = t.y; v[rho][2] = t.z; v[rho][3] = t.w;
        }
    }

#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        if constexpr (KIND == kEdge) {                                     // rows that this output row is the first to use
#pragma unroll
            for (int rho = r == 0 ? 0 : r + KH - 1; rho < r + KH; ++rho) quad.put_right(v[rho][0], v[rho][1], v[rho][2], v[rho][3]);
        }
        float z[4];
#pragma unroll
        for (int q = 0; q < KW; ++q) {
            if (q > 0) {                                                   // Z(s) <- Z(s-1)
                const float below = from_lane_below(z[3]);
                z[3] = z[2]; z[2] = z[1]; z[1] = z[0]; z[0] = below;
            }
            kernarg_floats ft = taps_t + q * KH + (kReloadTaps ? opaque_zero() : 0);
#pragma unroll
            for (int p = 0; p < KH; ++p) {
                const float wv = ft[p];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (p == 0 && q == 0) z[i] = wv * v[r][i];
                    else z[i] = __builtin_fmaf(wv, v[r + p][i], z[i]);
                }
            }
        }
        // read the results out KW-1 PEs further down: PE s gets output column s
#pragma unroll
        for (int t = 0; t < KW - 1; ++t) {
            const float above = from_lane_above(z[0]);
            z[0] = z[1]; z[1] = z[2]; z[2] = z[3]; z[3] = above;
        }
        if (r < rows_out && lane_valid) {
            float* yr = yrow + (long long)r * yp;
            if (EDGE) {
                store4_guarded(yr, col, ow, z);
            } else {
                f4u t;
                t.x = z[0]; t.y = z[1]; t.z = z[2]; t.w = z[3];
                if (SYSCONV_NONTEMPORAL_STORE) __builtin_nontemporal_store(t, reinterpret_cast<f4u*>(yr + col));
                else *reinterpret_cast<f4u*>(yr + col) = t;
            }
        }
    }
}

template <int KH, int KW, int ROWS>
__global__ __launch_bounds__(kBlock) void conv2d_sbm_block_kernel(TapsOf<KH * KW> taps_t, const float* __restrict__ x,
                                                                  float* __restrict__ y, int w_img, long long xp,
                                                                  int oh, int ow, long long yp, int row_blocks,
                                                                  int strips, int side, int per_xcd, int valid_lanes)
{
    (void)taps_t;
    kernarg_floats tf = (kernarg_floats)__builtin_amdgcn_kernarg_segment_ptr();
    int rb, strip;
    if (!wave_tile(per_xcd, row_blocks, strips, side, rb, strip)) return;
    const int lane = threadIdx.x & (kWave - 1);
    const int col0 = strip * kTile * valid_lanes;
    const int r0 = rb * ROWS;
    const int rows_out = min(ROWS, oh - r0);
    const float* xrow = x + (long long)r0 * xp;
    float* yrow = y + (long long)r0 * yp;
    const bool lane_valid = lane < valid_lanes;
    const int col = col0 + kTile * lane;
    if (col0 + kStrip <= w_img)
        sbm_block_rows<KH, KW, ROWS, kInside>(tf, xrow, yrow, col, w_img, xp, ow, yp, rows_out, lane_valid);
    else if (KW >= 4 || w_img >= 4)
        sbm_block_rows<KH, KW, ROWS, kEdge>(tf, xrow, yrow, col, w_img, xp, ow, yp, rows_out, lane_valid);
    else if constexpr (KW < 4)
        sbm_block_rows<KH, KW, ROWS, kNarrow>(tf, xrow, yrow, col, w_img, xp, ow, yp, rows_out, lane_valid);
}

// Lanes of an SBM strip that keep their results: 64 - halo_lanes(kw).  (Rounding the
// strip width down to whole cache lines was measured and does not pay in 2-D:
// 4096^2, 5x5: 28.1 us with 63 lanes, 29.0 with 60, 29.3 with 56.)
int strip_valid_lanes(int kw) { return kWave - halo_lanes(kw); }

// kEdge takes the last strip where some of its columns are missing, as long as the strip before it has its whole halo (in whole quads).
StripKind bfs_strip_right(int w, int strips, int kw)
{
    const int last = (strips - 1) * kStrip;
    return w - last < kStrip && (strips == 1 || w - last >= kTile * ((kw + 2) / 4)) ? kEdge : kNarrow;
}

// Shared launcher of the two strip-walking kernels (BFS and SBM).
template <int KH, int KW, int PD, bool SBM>
hipError_t launch_strip(const float* x, int h, int w, size_t xp, const float* f, float* y, size_t yp, hipStream_t s)
{
    // BFS reads its taps row by row, SBM column by column (transposed)
    float ft[KH * KW];
    for (int p = 0; p < KH; ++p)
        for (int q = 0; q < KW; ++q) ft[SBM ? q * KH + p : p * KW + q] = f[p * KW + q];
    const TapsOf<KH * KW> taps(ft, KH * KW);
    const int oh = h - KH + 1, ow = w - KW + 1;
    // SBM strips overlap (the partial sums of the first KW-1 PEs come from the strip to
    // the left, so those lanes are redundant); BFS strips are exactly 256 outputs wide and
    // fetch the KW-1 halo columns separately
    const int valid_lanes = SBM ? strip_valid_lanes(KW) : kWave;
    const int strips = (ow + kTile * valid_lanes - 1) / (kTile * valid_lanes);
    // Rows per wavefront.  Measured on MI355X (in-process A/B sweeps): short items win
    // everywhere -- small filters are bound by memory latency and need > 8 K wavefronts
    // in flight (4096^2, 5x5, SBM: 27 us with 4 rows, 30 us with 16), large ones are
    // bound by the VALUs and lose to the tail of a coarse decomposition (8192^2, 11x11,
    // SBM: 246 us with 8 rows, 266 us with 24, 317 us with 64).  BFS pays KH(KH-1)/2
    // skipped filter-row blocks per item, so its items are a little taller.  The price
    // is halo traffic: an item re-reads KH-1 input rows; most of those re-reads hit in
    // cache (HBM reads 1.12x the image for 5x5, 1.6x for 11x11, which is bound by the
    // VALUs anyway).
    int rows = SBM ? (KH <= 5 ? 4 : 8) : (KH <= 5 ? 6 : 16);
    // Images too small to give the machine 4096 items of that height get shorter ones
    // (1024^2, 11x11: SBM 18.4 -> 12.4 us, BFS 43.9 -> 16.4 us; 2048^2, 11x11: 31 -> 25 us,
    // 44 -> 32 us; asking for 8192 or 16384 items instead costs up to 28 % elsewhere).
    while (rows > 2 && (long long)((oh + rows - 1) / rows) * strips < 4096) rows = (rows + 1) / 2;
    if (rows > oh) rows = oh;
    const int row_blocks = (oh + rows - 1) / rows;
    long long per_xcd;
    const long long blocks = tile_workgroups(row_blocks, strips, per_xcd);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    if constexpr (SBM)
        hipLaunchKernelGGL((conv2d_sbm_kernel<KH, KW, PD>), dim3((unsigned)blocks), dim3(kBlock), 0, s,
                           taps, x, y, w, (long long)xp, oh, ow, (long long)yp, rows, row_blocks, strips, band_width(xp),
                           (int)per_xcd, valid_lanes);
    else
        hipLaunchKernelGGL((bfs_strip_right(w, strips, KW) == kEdge ? conv2d_bfs_kernel<KH, KW, PD, kEdge> : conv2d_bfs_kernel<KH, KW, PD, kNarrow>), dim3((unsigned)blocks), dim3(kBlock), 0, s,
                           taps, x, y, w, (long long)xp, oh, ow, (long long)yp, rows, row_blocks, strips, band_width(xp),
                           (int)per_xcd, valid_lanes);
    return hipGetLastError();
}

}  // namespace

namespace {
template <int KH, int KW, int RPW>
hipError_t launch_fbs_static(const float* x, int h, int w, size_t xp, const float* f, float* y, size_t yp,
                             hipStream_t s)
{
    constexpr int tile_rows = RPW * (kBlock / kWave);
    const TapsOf<KH * KW> taps(f, KH * KW);
    const int oh = h - KH + 1, ow = w - KW + 1;
    const int cols = kTile * fbs_static_valid_lanes(KH, KW);
    const int tiles_x = (ow + cols - 1) / cols;
    const int tiles_y = (oh + tile_rows - 1) / tile_rows;
    const long long n_tiles = (long long)tiles_x * tiles_y;
    const long long per_xcd = (n_tiles + kXcds - 1) / kXcds;
    const long long blocks = per_xcd * kXcds;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((conv2d_fbs_static_kernel<KH, KW, RPW>), dim3((unsigned)blocks), dim3(kBlock), 0, s,
                       taps, x, y, h, w, (long long)xp, oh, ow, (long long)yp, tiles_y, (int)n_tiles,
                       band_width(xp), (int)per_xcd);
    return hipGetLastError();
}

}  // namespace

// Filters whose size is known at compile time: every kh x kw whose smaller side is at most 7, single rows and columns (the two passes of a separable filter)
// among them (us, this kernel / one with run-time sizes, which re-read every staged row once per filter row and is gone: 4096^2
// 9x3 29.9 / 40.4, 3x9 27.5 / 32.7, 11x5 41.2 / 51.0, 10x4 36.3 / 48.5, 15x1 21.9 / 39.7; 3000^2 15x2 17.9 / 25.7, 13x4 21.1 / 29.2, 14x6 32.0 / 39.1, 12x7
// 31.6 / 37.9, 6x12 28.4 / 32.1, 2x14 16.3 / 16.7; 1000^2 14x1 4.5 / 6.7).  From 8x8 on the taps no longer
// fit the scalar registers and the unrolled form loses (11x11 on
// 8192^2: 353 us with 4 rows per wavefront, 423 us with 2, against 313 us).  Output rows per wavefront
// from a sweep on MI355X (us with 1 / 2 / 3 / 4 rows): 4096^2 3x3 27.1 / 26.4 / 28.0 / 28.2,
// 5x5 32.3 / 27.7 / 28.1 / 29.6, 7x7 51.7 / 41.2 / 42.1 / 39.6; 8192^2 5x5 115.5 / 95.3 / 96.8 / 102.2; columns with 3 / 4 / 6 / 8 rows 2000^2 10x1
// 8.9 / 8.4 / 8.0 / 7.4, 500^2 15x1 3.8 / 3.9 / 4.5 / 5.1, 8000^2 13x1 level.
static bool has_conv2d_fbs_static(int kh, int kw)
{
    const int small = kh < kw ? kh : kw, large = kh < kw ? kw : kh;
    return small >= 1 && small <= 7 && large <= kMaxK2D;
}

// Where it serves them: rows of 12 taps and more, and 7x14 and 7x15, only up to 2 M outputs (us, this / the strips: 1x12 on 1000^2 4.35 / 4.7, on 3000^2 15.3 / 15.1;
// 7x14 on 522x945 7.4 / 8.9, on 3000^2 42.0 / 35.3).
bool conv2d_fbs_static_serves(int oh, int ow, int kh, int kw)
{
    if (!has_conv2d_fbs_static(kh, kw)) return false;
    return !((kh == 1 && kw >= 12) || (kh == 7 && kw >= 14)) || (double)oh * ow <= 2e6;
}

namespace {
#define SYSCONV_FBS_STATIC(KH, KW, RPW) \
    if (kh == KH && kw == KW) return launch_fbs_static<KH, KW, RPW>(x, h, w, xp, f, y, yp, s)

hipError_t launch_fbs_static_any(const float* x, int h, int w, size_t xp, const float* f, int kh, int kw, float* y,
                                 size_t yp, hipStream_t s)
{
    // two output rows per wavefront up to 5 filter rows, four from 6 on (the sweep above)
#define SYSCONV_FBS_STATIC_ROW(KH, RPW)                                                                     \
    SYSCONV_FBS_STATIC(KH, 2, RPW); SYSCONV_FBS_STATIC(KH, 3, RPW); SYSCONV_FBS_STATIC(KH, 4, RPW);       \
    SYSCONV_FBS_STATIC(KH, 5, RPW); SYSCONV_FBS_STATIC(KH, 6, RPW); SYSCONV_FBS_STATIC(KH, 7, RPW)
    SYSCONV_FBS_STATIC_ROW(2, 2); SYSCONV_FBS_STATIC_ROW(3, 2); SYSCONV_FBS_STATIC_ROW(4, 2);
    SYSCONV_FBS_STATIC_ROW(5, 2); SYSCONV_FBS_STATIC_ROW(6, 4); SYSCONV_FBS_STATIC_ROW(7, 4);
    SYSCONV_FBS_STATIC_ROW(8, 4); SYSCONV_FBS_STATIC_ROW(9, 4); SYSCONV_FBS_STATIC_ROW(10, 4); SYSCONV_FBS_STATIC_ROW(11, 4);
    SYSCONV_FBS_STATIC_ROW(12, 4); SYSCONV_FBS_STATIC_ROW(13, 4); SYSCONV_FBS_STATIC_ROW(14, 4); SYSCONV_FBS_STATIC_ROW(15, 4);
#undef SYSCONV_FBS_STATIC_ROW
#define SYSCONV_FBS_STATIC_WIDE(KH, RPW)                                                                    \
    SYSCONV_FBS_STATIC(KH, 8, RPW); SYSCONV_FBS_STATIC(KH, 9, RPW); SYSCONV_FBS_STATIC(KH, 10, RPW);      \
    SYSCONV_FBS_STATIC(KH, 11, RPW); SYSCONV_FBS_STATIC(KH, 12, RPW); SYSCONV_FBS_STATIC(KH, 13, RPW);            \
    SYSCONV_FBS_STATIC(KH, 14, RPW); SYSCONV_FBS_STATIC(KH, 15, RPW)
    SYSCONV_FBS_STATIC_WIDE(2, 2); SYSCONV_FBS_STATIC_WIDE(3, 2); SYSCONV_FBS_STATIC_WIDE(4, 2);
    SYSCONV_FBS_STATIC_WIDE(5, 2); SYSCONV_FBS_STATIC_WIDE(6, 4); SYSCONV_FBS_STATIC_WIDE(7, 4);
#undef SYSCONV_FBS_STATIC_WIDE
    SYSCONV_FBS_STATIC(1, 1, 4); SYSCONV_FBS_STATIC(1, 2, 4); SYSCONV_FBS_STATIC(1, 3, 4); SYSCONV_FBS_STATIC(1, 4, 4); SYSCONV_FBS_STATIC(1, 5, 4);
    SYSCONV_FBS_STATIC(1, 6, 4); SYSCONV_FBS_STATIC(1, 7, 4); SYSCONV_FBS_STATIC(1, 8, 4); SYSCONV_FBS_STATIC(1, 9, 4);
    SYSCONV_FBS_STATIC(1, 10, 4); SYSCONV_FBS_STATIC(1, 11, 4); SYSCONV_FBS_STATIC(1, 12, 4); SYSCONV_FBS_STATIC(1, 13, 4);
    SYSCONV_FBS_STATIC(1, 14, 4); SYSCONV_FBS_STATIC(1, 15, 4);
    SYSCONV_FBS_STATIC(2, 1, 4); SYSCONV_FBS_STATIC(3, 1, 4); SYSCONV_FBS_STATIC(4, 1, 4); SYSCONV_FBS_STATIC(5, 1, 4);
    SYSCONV_FBS_STATIC(6, 1, 4); SYSCONV_FBS_STATIC(7, 1, 4); SYSCONV_FBS_STATIC(8, 1, 4); SYSCONV_FBS_STATIC(9, 1, 4);
    SYSCONV_FBS_STATIC(10, 1, 4); SYSCONV_FBS_STATIC(11, 1, 4); SYSCONV_FBS_STATIC(12, 1, 4); SYSCONV_FBS_STATIC(13, 1, 4);
    SYSCONV_FBS_STATIC(14, 1, 4); SYSCONV_FBS_STATIC(15, 1, 4);
    return hipErrorInvalidValue;
}
#undef SYSCONV_FBS_STATIC
}  // namespace

// ------------------------------------------------------------ FBS strips ----
// Filters of 8 to 15 columns: a wavefront takes ROWS output rows of a strip of 256 input columns and walks down their ROWS + kh - 1 input rows, four of them in
// flight.  Each row's KW-wide window is built once with KW - 1 hand-overs and applied to every output row whose filter covers it; the taps come in a row ahead of
// their use, in a ring.  Left in the middle, the body has the ring copied to vector registers (92 to 150 of them with two and three rows); with every row guarded instead it stays in scalar registers (44 to 52).  us, left (12 and 14
// columns without a ring, which was slower) / guarded: 6130^2 14x14 238 / 230, 415^2 12x12 6.05 / 5.1, 2500^2 8x12 24.9 / 24.1; 12 columns and more 0.97 with one row, 0.985 with two, 0.975 with three.
// Fewer columns are level or quicker left: 10 and 11 (three rows 1.01, 5952x796 14x10 28.9 / 30.3; two 1.01), 8 and 9 with one (902^2 9x9 6.45 / 6.65), with two, and with three (8 to 11 rows a filter 0.97, 3109^2 9x9 31.4 / 30.5; 13 and 14
// 1.035, 2748x4017 13x9 43.8 / 46.2).  The tile kernel with run-time sizes that served these filters staged its rows in LDS
// and handed the inputs on once for every filter row: us, that / this: 8192^2 11x11 354 / 257 (SBM 257), 6130^2 14x14 268 / 230, 3109^2 9x9 36.8 / 31.4, 5694x2688 9x15 85.7 / 72.0,
// 1500^2 15x15 31.0 / 23.9, 491x4731 12x9 16.4 / 12.6, 902^2 9x9 8.6 / 6.5, 415^2 12x12 11.7 / 5.1.
// What bounds it: the vector ALUs on large images (11x11: 547 instructions for four outputs, 484 of them the multiply-adds), the latency of a wavefront's rows on small ones.
namespace {
constexpr int kFbsAhead = 4;
template <int KW, int ROWS, bool EDGE>
__device__ __forceinline__ void fbs_strip_rows(kernarg_floats taps_f, const float* __restrict__ xrow, float* __restrict__ yrow, int col,
                                               int w_img, long long xp, int ow, long long yp, int kh, int rows_out, bool lane_valid)
{
    // filter row p waits in slot p mod RING from input row p - 1 on to input row p + ROWS - 1
    constexpr int RING = ROWS == 1 ? 2 : ROWS <= 3 ? 4 : 0;
    constexpr bool GUARDED = KW >= 12;
    static_assert(RING == 0 || RING >= ROWS + 1, "a slot is free again when the next filter row comes in");
    const int rows_in = rows_out - 1 + kh;
    const EdgeQuad quad(col, w_img);
    f4u v[kFbsAhead];
    auto load_row = [&](int rho, f4u& d) {                                 // past the last row: the last row again
        d = *reinterpret_cast<const f4u*>(xrow + (long long)min(rho, rows_in - 1) * xp + (EDGE ? quad.at : col));
    };
    float wv[RING > 0 ? RING : ROWS][KW];
    auto load_taps = [&](int p, float (&w)[KW]) {
        kernarg_floats fp = taps_f + min(max(p, 0), kh - 1) * KW;
#pragma unroll
        for (int q = 0; q < KW; ++q) w[q] = fp[q];
    };
#pragma unroll
    for (int i = 0; i < kFbsAhead; ++i) load_row(i, v[i]);
    if constexpr (RING > 0) load_taps(0, wv[0]);
    float acc[ROWS][4];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) acc[r][0] = acc[r][1] = acc[r][2] = acc[r][3] = 0.0f;
    for (int rho0 = 0; rho0 < rows_in; rho0 += kFbsAhead) {
#pragma unroll
        for (int j = 0; j < kFbsAhead; ++j) {
            const int rho = rho0 + j;
            if (!GUARDED && rho >= rows_in) break;                         // uniform
            if constexpr (RING > 0) {
                __builtin_amdgcn_sched_barrier(0);                         // (the taps of the next row stay where they are asked for)
                if constexpr (GUARDED) load_taps(rho + 1, wv[(j + 1) % (RING > 0 ? RING : 1)]);
            } else {
#pragma unroll
                for (int r = 0; r < ROWS; ++r) load_taps(rho - r, wv[r]);
            }
            if (GUARDED && rho >= rows_in) continue;                       // uniform
            f4u t = v[j];
            float win[KW + 3] = {t.x, t.y, t.z, t.w};
            if constexpr (EDGE) quad.put_right(win[0], win[1], win[2], win[3]);
            load_row(rho + kFbsAhead, v[j]);
            if constexpr (RING > 0 && !GUARDED) load_taps(rho + 1, wv[(j + 1) % (RING > 0 ? RING : 1)]);
#pragma unroll
            for (int m = 4; m < KW + 3; ++m) win[m] = from_lane_above(win[m - 4]);
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                const int p = rho - r;
                if (p < 0 || p >= kh) continue;                            // uniform
                const float (&w)[KW] = wv[RING > 0 ? (j - r + RING) % (RING > 0 ? RING : 1) : r];
#pragma unroll
                for (int q = 0; q < KW; ++q)
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[r][i] = __builtin_fmaf(w[q], win[q + i], acc[r][i]);
            }
        }
    }
    if (!lane_valid) return;
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
        if (r < rows_out) store4_guarded(yrow + (long long)r * yp, col, ow, acc[r]);
}

template <int KW, int ROWS>
__global__ __launch_bounds__(kBlock) void conv2d_fbs_strip_kernel(TapsOf<kMaxK2D * KW> taps, const float* __restrict__ x, float* __restrict__ y,
                                                                  int w_img, long long xp, int oh, int ow, long long yp, int kh,
                                                                  int row_blocks, int strips, int side, int per_xcd)
{
    (void)taps;
    kernarg_floats tf = (kernarg_floats)__builtin_amdgcn_kernarg_segment_ptr();
    int rb, strip;
    if (!wave_tile(per_xcd, row_blocks, strips, side, rb, strip)) return;
    constexpr int valid_lanes = kWave - halo_lanes(KW);
    const int lane = threadIdx.x & (kWave - 1);
    const int col0 = strip * kTile * valid_lanes, r0 = rb * ROWS;
    const int rows_out = min(ROWS, oh - r0);
    const float* xrow = x + (long long)r0 * xp;
    float* yrow = y + (long long)r0 * yp;
    const int col = col0 + kTile * lane;
    if (col0 + kStrip <= w_img) fbs_strip_rows<KW, ROWS, false>(tf, xrow, yrow, col, w_img, xp, ow, yp, kh, rows_out, lane < valid_lanes);
    else fbs_strip_rows<KW, ROWS, true>(tf, xrow, yrow, col, w_img, xp, ow, yp, kh, rows_out, lane < valid_lanes);
}

template <int KW, int ROWS>
hipError_t launch_fbs_strip(const float* x, int h, int w, size_t xp, const float* f, int kh, float* y, size_t yp, hipStream_t s)
{
    const TapsOf<kMaxK2D * KW> taps(f, kh * KW);
    const int oh = h - kh + 1, ow = w - KW + 1;
    constexpr int cols = kTile * (kWave - halo_lanes(KW));
    const int strips = (ow + cols - 1) / cols;
    const int row_blocks = (oh - 1) / ROWS + 1;
    long long per_xcd;
    const long long blocks = tile_workgroups(row_blocks, strips, per_xcd);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((conv2d_fbs_strip_kernel<KW, ROWS>), dim3((unsigned)blocks), dim3(kBlock), 0, s,
                       taps, x, y, w, (long long)xp, oh, ow, (long long)yp, kh, row_blocks, strips, band_width(xp), (int)per_xcd);
    return hipGetLastError();
}
}  // namespace

// Output rows of a wavefront of the strips, by the wavefronts that one row each would make: one row gives the most of them and the shortest, more share input rows and windows.  us with
// 1 / 2 / 3 / 4 rows (wavefronts of one): 700^2 11x11 (2070) 6.7 / 7.4 / 8.9 / 10.8, 902^2 9x9 (3576) 6.5 / 6.5 / 7.9 / 8.4, 1000x1300 13x13 (5928) 12.4 / 11.9 / 12.4, 2631x749 9x15
// (10492) 17.0 / 16.5 / 16.6, 4160x1150 10x10 (20755) 23.7 / 21.2 / 20.5 / 23.5, 8192^2 11x11 320 / 267 / 258 / 257.  Single rows: four (3000^2 1x12 16.5 / 15.6 / 16.4 / 15.2).
int conv2d_fbs_strip_rows(int oh, int ow, int kh, int kw)
{
    if (kh == 1) return 4;
    const int cols = kTile * (kWave - halo_lanes(kw));
    const long long wavefronts = (long long)oh * (((long long)ow + cols - 1) / cols);
    return wavefronts <= 4000 ? 1 : wavefronts <= 15000 ? 2 : 3;
}

hipError_t launch_conv2d_fbs(const float* x, int h, int w, size_t xp, const float* f, int kh, int kw,
                             float* y, size_t yp, hipStream_t s)
{
    const int oh = h - kh + 1, ow = w - kw + 1;
    if (conv2d_fbs_static_serves(oh, ow, kh, kw)) return launch_fbs_static_any(x, h, w, xp, f, kh, kw, y, yp, s);
    const int rows = conv2d_fbs_strip_rows(oh, ow, kh, kw);
    auto launch = [&](auto width) {
        constexpr int KW = decltype(width)::value;
        if constexpr (KW >= 12) {
            if (rows == 4) return launch_fbs_strip<KW, 4>(x, h, w, xp, f, kh, y, yp, s);
        }
        return rows == 1 ? launch_fbs_strip<KW, 1>(x, h, w, xp, f, kh, y, yp, s)
             : rows == 2 ? launch_fbs_strip<KW, 2>(x, h, w, xp, f, kh, y, yp, s) : launch_fbs_strip<KW, 3>(x, h, w, xp, f, kh, y, yp, s);
    };
    switch (kw) {
    case 8: return launch(std::integral_constant<int, 8>{});
    case 9: return launch(std::integral_constant<int, 9>{});
    case 10: return launch(std::integral_constant<int, 10>{});
    case 11: return launch(std::integral_constant<int, 11>{});
    case 12: return launch(std::integral_constant<int, 12>{});
    case 13: return launch(std::integral_constant<int, 13>{});
    case 14: return launch(std::integral_constant<int, 14>{});
    case 15: return launch(std::integral_constant<int, 15>{});
    default: return hipErrorInvalidValue;
    }
}

// SYSCONV_TILE_WIDE=1 in the environment (read once) makes the block-form BFS kernels use the
// arrangement of wave_tile_wide().  It is a tuning aid, not a default: on 4096^2, 5x5 it cuts
// the HBM reads from 1.118 to 1.043 times the image (the cache line that holds a strip's halo
// columns is no longer fetched twice) without changing the time (26.2 -> 27.4 us); it is 6 %
// faster on 8192^2 and 5 % slower on 16384^2.
bool tile_wide_requested()
{
    static const bool wide = [] {
        const char* v = getenv("SYSCONV_TILE_WIDE");
        return v && v[0] == '1';
    }();
    return wide;
}

template <int KH, int KW, int ROWS>
hipError_t launch_bfs_block(const float* x, int h, int w, size_t xp, const float* f, float* y, size_t yp,
                            hipStream_t s)
{
    const TapsOf<KH * KW> taps(f, KH * KW);
    const int oh = h - KH + 1, ow = w - KW + 1;
    const int strips = (ow + kStrip - 1) / kStrip;
    const int row_blocks = (oh + ROWS - 1) / ROWS;
    const int wide = tile_wide_requested() ? 1 : 0;
    long long per_xcd;
    const long long blocks = wide ? tile_workgroups_wide(row_blocks, strips, per_xcd)
                                  : tile_workgroups(row_blocks, strips, per_xcd);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    const bool quads = w < 4 || (w & 3) == 0;
    hipLaunchKernelGGL((quads ? conv2d_bfs_block_kernel<KH, KW, ROWS, kNarrow> : conv2d_bfs_block_kernel<KH, KW, ROWS, kEdge>), dim3((unsigned)blocks), dim3(kBlock), 0, s,
                       taps, x, y, w, (long long)xp, oh, ow, (long long)yp, row_blocks, strips, band_width(xp),
                       (int)per_xcd, wide);
    return hipGetLastError();
}

template <int KH, int KW, int ROWS>
hipError_t launch_sbm_block(const float* x, int h, int w, size_t xp, const float* f, float* y, size_t yp,
                            hipStream_t s)
{
    float ft[KH * KW];
    for (int p = 0; p < KH; ++p)
        for (int q = 0; q < KW; ++q) ft[q * KH + p] = f[p * KW + q];      // filter column q contiguous
    const TapsOf<KH * KW> taps(ft, KH * KW);
    const int oh = h - KH + 1, ow = w - KW + 1;
    const int valid_lanes = strip_valid_lanes(KW);
    const int strips = (ow + kTile * valid_lanes - 1) / (kTile * valid_lanes);
    const int row_blocks = (oh + ROWS - 1) / ROWS;
    long long per_xcd;
    const long long blocks = tile_workgroups(row_blocks, strips, per_xcd);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((conv2d_sbm_block_kernel<KH, KW, ROWS>), dim3((unsigned)blocks), dim3(kBlock), 0, s,
                       taps, x, y, w, (long long)xp, oh, ow, (long long)yp, row_blocks, strips, band_width(xp),
                       (int)per_xcd, valid_lanes);
    return hipGetLastError();
}

bool has_conv2d_bfs(int kh, int kw)
{
    return kh == kw && kh >= 2 && kh <= 11;
}

hipError_t launch_conv2d_bfs(const float* x, int h, int w, size_t xp, const float* f, int kh, int kw,
                             float* y, size_t yp, hipStream_t s)
{
    if (kh != kw) return hipErrorInvalidValue;
    switch (kh) {
    // Filters up to 7x7 are bound by memory on large images and run the block form (block
    // heights from a sweep on 4096^2, cold data: 2x2..5x5: 29 us with 2 rows against 31-35 us
    // for taller blocks or the strip walk; 6x6: 35 us with 3; 7x7: 38 us with 4); from 8x8 on
    // the VALUs bound the kernel and the strip walk with its register ring is faster.
    case 2: return launch_bfs_block<2, 2, 2>(x, h, w, xp, f, y, yp, s);
    case 3: return launch_bfs_block<3, 3, 2>(x, h, w, xp, f, y, yp, s);
    case 4: return launch_bfs_block<4, 4, 2>(x, h, w, xp, f, y, yp, s);
    case 5: return launch_bfs_block<5, 5, 2>(x, h, w, xp, f, y, yp, s);
    case 6: return launch_bfs_block<6, 6, 3>(x, h, w, xp, f, y, yp, s);
    case 7: return launch_bfs_block<7, 7, 4>(x, h, w, xp, f, y, yp, s);
    case 8: return launch_strip<8, 8, 2, false>(x, h, w, xp, f, y, yp, s);
    case 9: return launch_strip<9, 9, 1, false>(x, h, w, xp, f, y, yp, s);
    case 10: return launch_strip<10, 10, 1, false>(x, h, w, xp, f, y, yp, s);
    case 11: return launch_strip<11, 11, 1, false>(x, h, w, xp, f, y, yp, s);
    default: return hipErrorInvalidValue;
    }
}

bool has_conv2d_sbm(int kh, int kw) { return has_conv2d_bfs(kh, kw); }

hipError_t launch_conv2d_sbm(const float* x, int h, int w, size_t xp, const float* f, int kh, int kw,
                             float* y, size_t yp, hipStream_t s)
{
    if (kh != kw) return hipErrorInvalidValue;
    switch (kh) {
    // Up to 7x7 the block form (all loads of a short row block up front) beats the strip walk
    // (4096^2: 2x2 33.8 -> 30.3 us, 3x3 32.1 -> 28.6, 5x5 34.2 -> 31.4, 7x7 39.2 -> 37.9;
    // 16384 x 40960, 5x5: 1191 -> 1119 us); block heights from a sweep over 1, 2, 3, 4, 6 rows.
    case 2: return launch_sbm_block<2, 2, 2>(x, h, w, xp, f, y, yp, s);
    case 3: return launch_sbm_block<3, 3, 2>(x, h, w, xp, f, y, yp, s);
    case 4: return launch_sbm_block<4, 4, 2>(x, h, w, xp, f, y, yp, s);
    case 5: return launch_sbm_block<5, 5, 4>(x, h, w, xp, f, y, yp, s);
    case 6: return launch_sbm_block<6, 6, 4>(x, h, w, xp, f, y, yp, s);
    case 7: return launch_sbm_block<7, 7, 4>(x, h, w, xp, f, y, yp, s);
    case 8: return launch_strip<8, 8, 2, true>(x, h, w, xp, f, y, yp, s);
    case 9: return launch_strip<9, 9, 2, true>(x, h, w, xp, f, y, yp, s);
    case 10: return launch_strip<10, 10, 1, true>(x, h, w, xp, f, y, yp, s);
    case 11: return launch_strip<11, 11, 1, true>(x, h, w, xp, f, y, yp, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace sysconv
