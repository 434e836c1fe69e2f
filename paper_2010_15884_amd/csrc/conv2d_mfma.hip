// 2-D valid convolution (paper Eq. 3) for filters whose kh*kw multiply-adds per output
// exceed what the vector ALUs deliver per byte of HBM traffic: the sums are taken by the
// matrix cores (the hardware systolic arrays of the CU) instead of the software array.
//
// One v_mfma_f32_16x16x32_f16 multiplies a 16 x 32 by a 32 x 16 matrix.  A single-channel
// filter has no channel dimension to contract over, so the contraction is made from the
// filter's own extent in BOTH directions (a doubly blocked Toeplitz form):
//
//   N (16)  "bases": 16 output positions (r, c0 + 4 i), i = 0..15, of one output row
//   M (16)  "offsets": the 4 x 4 outputs (r + jr, c + jc) next to a base, j = 4 jr + jc
//   K       input offsets (dr, dc), dr < kh + 3 rows, dc < 16 columns, taken 2 rows
//           (= 32 values, a "unit") per instruction: NS = ceil((kh + 3) / 2) instructions
//
//   A[j][(dr, dc)] = f[dr - jr][dc - jc]      (0 outside the filter)   -- constant, in registers
//   B[(dr, dc)][i] = x[r + dr][c0 + 4 i + dc]                          -- 8 consecutive inputs per lane
//   D[j][i]        = y[r + jr][c0 + 4 i + jc]                          -- 4 consecutive outputs per lane
//
// so NS instructions produce a 4-row x 64-column group of outputs; kh*kw of the
// 2*16*NS products per output are non-zero (11x11: 121 of 224).
//
// Precision.  The matrix cores multiply fp16.  Inputs and taps are therefore split,
// v = hi + lo with hi = fp16(v) and lo = fp16(v - hi) (kept 2^11 times larger, so that it
// is a normal fp16 number like hi), which keeps 22 significant bits, and three products
// are accumulated in fp32: hi*hi, and hi*lo + lo*hi in accumulators of their own that
// enter the result times 2^-11 (the lo*lo term is below 2^-22 of the product).  Both
// operands are scaled by a power of two first: taps by a factor the host derives from
// their largest magnitude, inputs by a fixed 2^13.  That fixes the admissible input range:
// |x| < 8 (larger values become infinite in fp16), and inputs below 2^-27 count as zero.
//
// Data path (as in conv2d_split.hip).  A workgroup of four wavefronts walks down a block of rows of a 256-column strip, 16 input
// rows (a "chunk") at a time.  A chunk is loaded into registers two chunks ahead of its use, split once and written to LDS as two
// fp16 planes one chunk ahead; a lane's operand is then 16 bytes of a plane, read a unit ahead of its use.  Every unit is applied to all output groups it
// belongs to, whose sums wait in registers: no halo row is loaded or split twice within a block, and there is one barrier per chunk.  A block ends with
// any group (matrix_block_groups).  Before, a workgroup of twelve wavefronts stepped through four rows at a time in lock-step and every lane split its own windows,
// four times an input: us, so / this: 300^2 3x3 5.8 / 3.3, 585^2 12x12 10.4 / 6.2, 1222^2 11x11 10.1 / 7.8, 2021^2 12x9 15.5 / 12.5, 4096^2 9x9 33 / 28.5,
// 6000^2 9x9 66 / 60, 8192^2 11x11 121 / 114, 5x5 103 / 103, 7x7 108 / 109; 150 random images and filters 0.74 on average.
//
// Stores.  A group's row is 256 bytes of a wavefront; where output rows start anywhere in a 128-byte line, that is three lines, two of them shared
// with the neighbours, and on large images these pieces reach memory one by one.  ROWS_OUT passes the results through LDS and stores 1 KB of a row at a
// time: 8192^2 11x11 131 / 116 us, 7052^2 5x5 90 / 82, 7407^2 4x4 100 / 90; up to 30 M outputs the way through LDS costs 5 to 10 % (1222^2 11x11
// 8.0 / 8.5, 4096^2 9x9 28.8 / 29.8).  A strip at the right edge stores whole quads, and column by column only where a quad straddles the edge: four strided dwords for
// every quad ended the launch with these strips (6000^2 9x9 69 / 58).
//
// What bounds it: large images how this walk's loads and stores reach memory, not how many they are (8192^2: 1.06 times the bytes of inputs and results, which the FBS kernel for 5x5 moves in 95 us; 11x11 takes
// 111 us with an image of zeros, where the clock is high, and 3x3, with three sevenths of the matrix instructions, 103), then the clock, which power lowers; small ones the chain taps - first chunk - units of one block.
// Strips shifted row by row onto 64-byte boundaries, 224 or 240 columns wide, cost more in strips and edges than they give, 124 - 128 us.
// Tried: strips of 256 columns with the 16 columns beyond as a fifth load (8192^2 112 - 117 us, 4096^2 30 - 33 and 1222^2 8.9), three or four workgroups a CU and
// two chunks in flight (level to 10 % slower: it is not latency), cacheable stores (long runs, us, this / through LDS / without: 8192^2 5x5 103 / 105 / 118, 11x11 114 / 116 / 116, 6401x6404
// 5x5 65.5 / 69.5 / 70.7, 8000^2 11x11 116 / 115 / 119; without it is ahead for single rows, 8192^2 1x5 101 / 103 / 91; 4096^2 28 / - / 33).
#include "launch.h"
#include "matrix_blocks.h"
#include "split_bf16.h"
#include "systolic.h"

#include <math.h>

#include <type_traits>

namespace sysconv {
namespace {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef const float __attribute__((address_space(4)))* kernarg_floats;

constexpr int kCols = 240;                  // output columns of a workgroup's strip (64 for three wavefronts, 48 for the last)
constexpr int kInCols = 256;                // input columns of a chunk (a filter is at most 13 wide)
constexpr int kChunk = 16;                  // input rows of a chunk: 8 units
constexpr int kUnits = kChunk / 2;
constexpr int kGroups = kChunk / 4;         // output groups that start in a chunk; the sums of a group live in slot (group mod 4)
constexpr int kRow = 2 * kInCols;           // a row in LDS, in fp16 numbers: 256 hi, 256 lo
constexpr int kBuf = kChunk * kRow;
constexpr int kTapCols = 19;                // columns of the zero-padded taps
constexpr float kMXScale = 8192.0f;        // 2^13: inputs up to 8 stay finite in fp16
constexpr float kMLoScale = 2048.0f;       // 2^11: the lo parts are kept this much larger

// Inputs times 2^13, split into fp16 hi and lo parts: v * 2^13 = hi + lo * 2^-11
// (both rounded to nearest).  The remainder v * 2^13 - hi is exact in fp32 and at most half an
// fp16 ulp of hi; stored 2^11 times larger it has the magnitude of hi at most and stays a normal
// fp16 number whenever hi is one (the matrix cores treat subnormal fp16 inputs as zero).  A value
// of 8 or more becomes infinite here and shows up as inf / NaN in the results it feeds.
// Three instructions per element, spelled out (the compiler's own selection takes four):
// v_fma_mixlo/mixhi_f16 scale in fp32 and round once to fp16 into one half of a register,
// v_fma_mix_f32 takes v * 2^13 - hi with hi read as fp16 from either half (exact).
__device__ __forceinline__ void mfma_split4(const f4u& v, u2& hi, u2& lo)
{
    const float xs = kMXScale, ls = kMLoScale;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const float v0 = v[2 * i], v1 = v[2 * i + 1];
        unsigned h, l;
        float r0, r1;
        asm("v_fma_mixlo_f16 %0, %1, %2, 0" : "=v"(h) : "v"(v0), "s"(xs));
        asm("v_fma_mixhi_f16 %0, %1, %2, 0" : "+v"(h) : "v"(v1), "s"(xs));
        asm("v_fma_mix_f32 %0, %1, %2, -%3 op_sel_hi:[0,0,1]" : "=v"(r0) : "v"(v0), "s"(xs), "v"(h));
        asm("v_fma_mix_f32 %0, %1, %2, -%3 op_sel:[0,0,1] op_sel_hi:[0,0,1]" : "=v"(r1) : "v"(v1), "s"(xs), "v"(h));
        asm("v_fma_mixlo_f16 %0, %1, %2, 0" : "=v"(l) : "v"(r0), "s"(ls));
        asm("v_fma_mixhi_f16 %0, %1, %2, 0" : "+v"(l) : "v"(r1), "s"(ls));
        hi[i] = h; lo[i] = l;
    }
}

// ROWS_OUT: results pass through LDS, so that a store is 1 KB of one row.
template <int NS, bool ROWS_OUT>
__global__ __launch_bounds__(kBlock, 2) void conv2d_mfma_kernel(
    TapsOf<(2 * NS - 3) * 13> taps, const float* __restrict__ x, float* __restrict__ y, int h, int w_img, long long xp, int oh, int ow,
    long long yp, int kh, int kw, int rows, int row_blocks, int strips, int per_xcd, float tap_scale, float inv_scale)
{
    static_assert(NS >= 2 && NS <= 8, "2 <= NS <= 8 covers filters of 1 .. 13 rows");
    (void)taps;
    constexpr int kCarried = (NS - 1) / 2;  // groups that a chunk leaves to the next to finish
    constexpr int TROWS = 2 * NS + 3;       // rows of the zero-padded taps
    kernarg_floats taps_f = (kernarg_floats)__builtin_amdgcn_kernarg_segment_ptr();
    __shared__ __attribute__((aligned(16))) _Float16 parts[2 * kBuf + 32];  // (windows of the last wavefront reach past a row)
    __shared__ __attribute__((aligned(16))) float outs[ROWS_OUT ? 2 : 1][ROWS_OUT ? kChunk : 1][kInCols];
    __shared__ float tpad[TROWS * kTapCols];

    const int g = xcd_contiguous(blockIdx.x, per_xcd);
    if (g >= row_blocks * strips) return;                                  // (the whole workgroup)
    const int rblk = g / strips, strip = g - rblk * strips;                // workgroups walk along the rows of the image
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = wave_in_block();
    const int c0 = strip * kCols;
    const int r0 = rblk * rows;
    const int cols_out = min(ow - c0, kCols);                              // columns the strip stores
    const int rows_out = min(rows, oh - r0);
    const int groups = (rows_out + 3) / 4;
    const int units = 2 * (groups - 1) + NS;
    const unsigned last_row = (unsigned)h - 1;
    const bool edge = c0 + kInCols > w_img;                                // uniform
    const bool narrow = w_img < 4;                                         // uniform: no 16 bytes to load

    // ---------------------------------------------------------------- a chunk into registers, and from there to LDS
    // Wavefront v takes rows v, v+4, v+8, v+12 (1 KB each); past the image's last row the last row again, which feeds only rows
    // that are not stored.  Loads that would reach past the row's end start at its last four columns instead and are put right before the split.
    const int col = c0 + kTile * lane;
    const int from = max(c0 - 4, 0);                                       // (a narrow filter's last strip may start within three columns of the end)
    const int col_m = max(min(col, w_img - 4), 0), off_m = narrow ? 0 : col - col_m;
    const unsigned col_b = (unsigned)(col_m - from) * (unsigned)sizeof(float);
    const float* const xs = x + from;
    f4u raw[4];
    auto load_chunk = [&](int c, auto edge_tag) {
        auto at = [&](int row) { return reinterpret_cast<const char*>(xs + (long long)min((unsigned)r0 + (unsigned)(c * kChunk + row), last_row) * xp); };
        if (decltype(edge_tag)::value && narrow) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float* p = reinterpret_cast<const float*>(at(wave + 4 * k));
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float v = p[min(col + i, w_img - 1)];            // (from is 0)
                    raw[k][i] = col + i < w_img ? v : 0.0f;
                }
            }
            return;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) raw[k] = *reinterpret_cast<const f4u*>(at(wave + 4 * k) + col_b);
    };
    auto put_right = [&](f4u& v, int off) {                                // columns past the image read as 0
        if (off & 1) v = f4u{v.y, v.z, v.w, 0.0f};
        if (off & 2) v = f4u{v.z, v.w, 0.0f, 0.0f};
        if (off > 3) v = f4u{0.0f, 0.0f, 0.0f, 0.0f};
    };
    auto store_chunk = [&](int c, auto edge_tag) {
        _Float16* buf = parts + (c & 1) * kBuf;
        if constexpr (decltype(edge_tag)::value) {
#pragma unroll
            for (int k = 0; k < 4; ++k) put_right(raw[k], off_m);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            u2 hi, lo;
            mfma_split4(raw[k], hi, lo);
            _Float16* dst = buf + (wave + 4 * k) * kRow + kTile * lane;
            *reinterpret_cast<u2*>(dst) = hi;
            *reinterpret_cast<u2*>(dst + kInCols) = lo;
        }
    };

    auto run = [&](auto edge_tag) {
        load_chunk(0, edge_tag);
        for (int e = threadIdx.x; e < TROWS * kTapCols; e += kBlock) {
            const int p = e / kTapCols - 3, q = e % kTapCols - 3;
            tpad[e] = p >= 0 && p < kh && q >= 0 && q < kw ? taps_f[p * kw + q] * tap_scale : 0.0f;
        }
        lds_barrier();

        // A operands: the Toeplitz form of the taps, constant for the whole kernel
        const int i16 = lane & 15, kb = lane >> 4;                         // operand coordinates of the lane
        h8 fa[NS][2];
        {
            const int jr = i16 / 4, jc = i16 % 4;
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const float* t = tpad + (2 * s + (kb >> 1) - jr + 3) * kTapCols + 8 * (kb & 1) - jc + 3;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const _Float16 hi = (_Float16)t[i];
                    fa[s][0][i] = hi;
                    fa[s][1][i] = (_Float16)((t[i] - (float)hi) * kMLoScale);
                }
            }
        }
        store_chunk(0, edge_tag);
        if (units > kUnits) load_chunk(1, edge_tag);
        lds_barrier();

        f4 acc[kGroups][2];
        const int win0 = (kb >> 1) * kRow + wave * 64 + 4 * i16 + 8 * (kb & 1);
        // Outputs of group lg of chunk c: lane (i16, kb) holds row kb, columns 4 i16 .. + 3 of the wavefront's 64.  Buffer stores drop the lanes whose
        // offset is out of range, so no store hides behind a branch and the waits for loads in flight count exactly.
        auto finish_group = [&](int c, int lg, const f4 (&sums)[2]) {
            f4 o;
#pragma unroll
            for (int v = 0; v < 4; ++v) o[v] = __builtin_fmaf(sums[1][v], inv_scale * (1.0f / kMLoScale), sums[0][v] * inv_scale);
            if constexpr (ROWS_OUT) {
                *reinterpret_cast<f4*>(&outs[c & 1][4 * (lg + kCarried) + kb][wave * 64 + 4 * i16]) = o;
            } else {
                const int grp = c * kGroups + lg;
                const u4 ob = __builtin_bit_cast(u4, o);
                const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(y + (long long)(r0 + grp * 4) * yp + c0, 0, 0x7fffffff, 0x00020000);
                const int oc = wave * 64 + 4 * i16, left = grp * 4 + kb < rows_out ? cols_out - oc : 0;
                const unsigned off = (unsigned)kb * ((unsigned)yp * 4u) + (unsigned)oc * 4u;
                __builtin_amdgcn_raw_buffer_store_b128(ob, rsrc, left >= 4 ? off : kNowhere, 0, kNonTemporal);
                if constexpr (decltype(edge_tag)::value) {
#pragma unroll
                    for (int i = 0; i < 3; ++i)
                        __builtin_amdgcn_raw_buffer_store_b32(ob[i], rsrc, i < left && left < 4 ? off + 4u * i : kNowhere, 0, kNonTemporal);
                }
            }
        };
        // ROWS_OUT: the rows finished with chunk c; wavefront v takes rows v, v+4, v+8, v+12 of them
        auto flush = [&](int c) {
            if constexpr (ROWS_OUT) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int rr = 4 * k + wave, row = c * kChunk - 4 * kCarried + rr;   // uniform
                    const bool row_ok = row >= 0 && row < rows_out;
                    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(y + (long long)(r0 + (row_ok ? row : 0)) * yp + c0, 0, 0x7fffffff, 0x00020000);
                    const float* results = outs[c & 1][rr];
                    if constexpr (!decltype(edge_tag)::value) {
                        const u4 ob = __builtin_bit_cast(u4, *reinterpret_cast<const f4*>(results + kTile * lane));
                        __builtin_amdgcn_raw_buffer_store_b128(ob, rsrc, row_ok && lane < kCols / 4 ? 16u * lane : kNowhere, 0, kNonTemporal);
                    } else {
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int cc = lane + kWave * i;
                            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, results[cc]), rsrc, row_ok && cc < cols_out ? 4u * cc : kNowhere, 0, kNonTemporal);
                        }
                    }
                }
            }
        };
        // One chunk: FIRST has no groups from before it, FULL starts all of its own (else it is looked at run time which groups there are, and how
        // many units are left).  A unit's windows are read while the one before is multiplied.
        auto compute = [&](int c, auto first_tag, auto full_tag) {
            constexpr bool FIRST = decltype(first_tag)::value, FULL = decltype(full_tag)::value;
            int at = (c & 1) * kBuf + win0;
            const int left = FULL ? kUnits : units - c * kUnits;
            h8 win[2][2];
            auto read = [&](int u) {
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    __builtin_memcpy(&win[u & 1][j], __builtin_assume_aligned(parts + at + j * kInCols, 8), 16);
            };
            read(0);
#pragma unroll
            for (int u = 0; u < kUnits; ++u) {
                if (!FULL && u >= left) break;                             // uniform
                __builtin_amdgcn_sched_barrier(0);
                at += 2 * kRow;
                asm("" : "+v"(at));
                if (u + 1 < kUnits) read(u + 1);
                const h8 (&b)[2] = win[u & 1];
#pragma unroll
                for (int lg = -kGroups; lg < kGroups; ++lg) {
                    const int s = u - 2 * lg;
                    if (s < 0 || s >= NS || (FIRST && lg < 0)) continue;
                    if (!FULL && (c * kGroups + lg < 0 || c * kGroups + lg >= groups)) continue;   // uniform
                    f4& hi = acc[(lg + kGroups) % kGroups][0];
                    f4& lo = acc[(lg + kGroups) % kGroups][1];
                    if (s == 0) hi = lo = f4{0.0f, 0.0f, 0.0f, 0.0f};
                    lo = __builtin_amdgcn_mfma_f32_16x16x32_f16(fa[s][1], b[0], lo, 0, 0, 0);
                    hi = __builtin_amdgcn_mfma_f32_16x16x32_f16(fa[s][0], b[0], hi, 0, 0, 0);
                    lo = __builtin_amdgcn_mfma_f32_16x16x32_f16(fa[s][0], b[1], lo, 0, 0, 0);
                }
#pragma unroll
                for (int lg = -kGroups; lg < kGroups; ++lg) {
                    if (u - 2 * lg != NS - 1 || (FIRST && lg < 0)) continue;
                    if (!FULL && (c * kGroups + lg < 0 || c * kGroups + lg >= groups)) continue;
                    finish_group(c, lg, acc[(lg + kGroups) % kGroups]);
                }
            }
        };
        const int full = groups / kGroups;
        auto advance = [&](int c, auto first_tag) {
            if constexpr (!decltype(first_tag)::value) flush(c - 1);
            store_chunk(c + 1, edge_tag);
            load_chunk(c + 2, edge_tag);
            compute(c, first_tag, std::true_type{});
            lds_barrier();
        };
        int c = 0;
        if (full > 0) {
            if (units > kUnits) advance(0, std::true_type{});
            else { compute(0, std::true_type{}, std::true_type{}); lds_barrier(); }
            for (c = 1; c < full; ++c) advance(c, std::false_type{});
        }
#pragma nounroll
        for (; c * kUnits < units; ++c) {
            if (ROWS_OUT && c > 0) flush(c - 1);
            if ((c + 1) * kUnits < units) {
                store_chunk(c + 1, edge_tag);
                if ((c + 2) * kUnits < units) load_chunk(c + 2, edge_tag);
            }
            compute(c, std::false_type{}, std::false_type{});
            lds_barrier();
        }
        if (ROWS_OUT) flush(c - 1);
    };
    if (edge) run(std::true_type{});
    else run(std::false_type{});
}

float largest_finite_magnitude(const float* f, int n)
{
    float amax = 0.0f;
    for (int i = 0; i < n; ++i) {
        const float a = fabsf(f[i]);
        if (a > amax && a <= 3.0e38f) amax = a;                    // NaN and inf fail the comparisons
    }
    return amax;
}

// Output rows of a workgroup's block: whole groups.
// Filters of up to three rows, whose groups end in the chunk they start in or the next: short blocks once they fill the device, one chunk's (NS = 2: four groups, eight units) or two (NS = 3: eight groups, 17 units, the
// last in a third chunk; us, blocks of the model's heights / this: 1775x7797 1x13 26.5 / 21.4, 5180^2 3x7 42.5 / 35.6, 7233x407 1x1 8.1 / 7.5.  Seven groups, which end with the second chunk, are 7 % quicker on some images and up to 16 % slower
// on others: 2110x1828 2x7 10.4 / 9.7, 5180^2 3x7 37.3 / 35.6, 1289x2854 3x1 8.5 / 9.9; 0.994 on average over 60).
// The model's set-up of a block is 8 steps.  With results through LDS it is a fit and no set-up: large images are bound by memory, and with more blocks under way their loads and stores spread better than the model
// says, the more so the fewer rows a filter has.  2, 1, 0 steps for NS = 2, 3, 4 and 1 .. 4 for 5 .. 8 (us, 8 / this, long runs: 8192^2 1x5 107 / 101, 3x3 108.5 / 102.9, 5x5 108 / 103, 20000x2500 4x4 88.7 / 85.3, 7500^2 4x7 95 / 91.5, 6800x8000
// 7x7 94.0 / 90.4, 8000^2 7x7 116 / 108, 9000x6000 6x6 96.8 / 91.6, 7899^2 9x9 110.5 / 106.7; the other way round 8192^2 9x9 109.4 / 112.0, 7899^2 12x12 108.1 / 113.4).
template <int NS, bool ROWS_OUT>
int block_rows(int oh, int ow)
{
    const int strips = (ow + kCols - 1) / kCols;
    const int all = (oh - 1) / 4 + 1;
    constexpr int kShort = 4 * (NS - 1);
    if (NS <= 3 && !ROWS_OUT && (double)((all + kShort - 1) / kShort) * strips > kPlaces) return 4 * kShort;
    return 4 * matrix_block_groups(all, strips, NS, 2, 1, ROWS_OUT ? (NS > 4 ? NS - 4 : 4 - NS) : 8, 128);
}

template <int NS, bool ROWS_OUT>
hipError_t launch_mfma(const float* x, int h, int w, size_t xp, const float* f, int kh, int kw, float* y,
                       size_t yp, hipStream_t s)
{
    const TapsOf<(2 * NS - 3) * 13> taps(f, kh * kw);
    // power of two that brings the largest tap into [2^13, 2^14): its fp16 parts are then
    // as far from the subnormal range as they can be
    const float amax = largest_finite_magnitude(f, kh * kw);
    int e = 0;
    if (amax > 0.0f) (void)frexpf(amax, &e);                      // amax = m * 2^e, 0.5 <= m < 1
    const float tap_scale = amax > 0.0f ? ldexpf(1.0f, 14 - e) : 1.0f;
    const float inv_scale = 1.0f / (tap_scale * kMXScale);

    const int oh = h - kh + 1, ow = w - kw + 1;
    const int strips = (ow + kCols - 1) / kCols;
    const long long rows = block_rows<NS, ROWS_OUT>(oh, ow);
    const int row_blocks = (int)((oh + rows - 1) / rows);
    const long long groups = (long long)row_blocks * strips;
    const long long per_xcd = (groups + kXcds - 1) / kXcds;
    const long long blocks = per_xcd * kXcds;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((conv2d_mfma_kernel<NS, ROWS_OUT>), dim3((unsigned)blocks), dim3(kBlock), 0, s, taps, x, y, h, w,
                       (long long)xp, oh, ow, (long long)yp, kh, kw, (int)rows, row_blocks, strips, (int)per_xcd, tap_scale, inv_scale);
    return hipGetLastError();
}

}  // namespace

bool has_conv2d_mfma(int kh, int kw) { return kh >= 1 && kw >= 1 && kh <= 13 && kw <= 13; }

// Both the scale 2^(14-e) and its reciprocal times 2^-13 must be normal fp32 numbers.
bool conv2d_mfma_taps_in_range(const float* f, int n)
{
    const float amax = largest_finite_magnitude(f, n);
    return amax == 0.0f || (amax >= 1.0e-30f && amax <= 1.0e30f);
}

// Whether results go through LDS: they do on large images (figures above), and where the rows of a group do not lie within the 2 GB of a
// buffer descriptor.
bool conv2d_mfma_rows_out(int oh, int ow, size_t yp)
{
    return (double)oh * ow >= 40e6 || yp > ((size_t)1 << 25);
}

namespace {
template <class F>
auto with_units(int kh, F&& f)                  // f<NS>
{
    switch ((kh + 4) / 2) {                                    // NS = ceil((kh + 3) / 2)
    case 2: return f(std::integral_constant<int, 2>{});
    case 3: return f(std::integral_constant<int, 3>{});
    case 4: return f(std::integral_constant<int, 4>{});
    case 5: return f(std::integral_constant<int, 5>{});
    case 6: return f(std::integral_constant<int, 6>{});
    case 7: return f(std::integral_constant<int, 7>{});
    default: return f(std::integral_constant<int, 8>{});
    }
}
}  // namespace

int conv2d_mfma_block_rows(int oh, int ow, size_t yp, int kh)
{
    const bool rows_out = conv2d_mfma_rows_out(oh, ow, yp);
    return with_units(kh, [&](auto ns) { return rows_out ? block_rows<decltype(ns)::value, true>(oh, ow) : block_rows<decltype(ns)::value, false>(oh, ow); });
}

hipError_t launch_conv2d_mfma(const float* x, int h, int w, size_t xp, const float* f, int kh, int kw,
                              float* y, size_t yp, hipStream_t s)
{
    if (!has_conv2d_mfma(kh, kw)) return hipErrorInvalidValue;
    const bool rows_out = conv2d_mfma_rows_out(h - kh + 1, w - kw + 1, yp);
    return with_units(kh, [&](auto ns) {
        constexpr int NS = decltype(ns)::value;
        return rows_out ? launch_mfma<NS, true>(x, h, w, xp, f, kh, kw, y, yp, s) : launch_mfma<NS, false>(x, h, w, xp, f, kh, kw, y, yp, s);
    });
}

}  // namespace sysconv
