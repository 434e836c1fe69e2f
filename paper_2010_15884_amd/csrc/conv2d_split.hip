// 2-D valid convolution (paper Eq. 3) for filters whose multiply-adds outweigh their bytes, on the
// matrix cores and in full fp32: no promise about the inputs is asked of the caller.
//
// Contraction.  One v_mfma_f32_16x16x32_bf16 multiplies a 16 x 32 by a 32 x 16 matrix.  The
// contraction is made from the filter's own extent (a doubly blocked Toeplitz form):
//
//   N (16)  "bases": 16 output positions (r, c0 + JC i), i = 0..15, of one output row
//   M (16)  "offsets": the JR x JC outputs (r + jr, c + jc) next to a base, j = JC jr + jc
//   K       input offsets (dr, dc), dc < 16, two rows (32 values) = one "unit" per instruction
//
// 4 x 4 offsets serve filters up to 13 columns, 8 x 2 offsets 14 and 15 columns (kw + JC - 1 <= 16).
// A group of JR output rows takes NS = ceil((kh + JR - 1) / 2) units.
//
// Precision: three bf16 parts a number, six products (split_bf16.h), which also says which inputs the split does not carry.
// The chunk (16 input rows x 256 columns) that holds such a value is marked, and which four of its rows, and the outputs
// these rows reach are taken again with ordinary multiply-adds before the workgroup ends (plain_rows).  Measured (us; the
// vector kernel / no such value / one in the image / in every twelfth chunk down a column / in every fourth / in every one):
// 11x11 on 4096^2 69 / 43 / 46 / 53 / 68 / 95, on 8192^2 256 / 141 / 162 / 191 / 244 / 349, on 1500^2 14.7 / 12.5 / 21 / 22 / 23 / 22;
// 15x15 on 3001x4003 87 / 44 / 61 / 64 / 86 / 103, on 300x400 6.7 / 8.3 / 14.8 / 15.8 / 15.9 / 12.5.  At worst over 13 filters on 300x400 .. 4096^2: 1.75 times the vector kernel from 3 M outputs on (11x11 on
// 2048^2 23 / 40), 2.5 times below (14x11 on 700^2 7.9 / 20).
//
// Data path.  A workgroup of four wavefronts walks down a block of rows of a 256-column strip, 16 input
// rows (a "chunk") at a time.  A chunk is loaded into registers two chunks ahead of its use, split once
// (not once per overlapping window) and written to LDS as three bf16 planes one chunk ahead; a lane's
// operand is then 16 bytes of a plane, read a unit ahead of its use (4 x 4 offsets; us, without / with: 11x11 on 8192^2 177 / 166, on 2000^2 16.8 / 16.2,
// 12x12 on 500^2 7.4 / 7.05; with 8 x 2 the registers are full).  Every unit is read from LDS once and applied to all output
// groups it belongs to, whose sums wait in registers: no halo row is loaded or split twice within a
// block, one barrier per chunk, and all indices of the sums are compile-time constants.  A block ends with any group (matrix_block_groups): the
// chunk it ends in, and the one that only finishes groups, look at run time which groups there are.
//
// Order of the six products: from one to the next only one operand changes, x or f.  That saves power, which is what bounds large images: us, x and f
// changing / one at a time 8192^2 11x11 166 / 161, 4096^2 9x13 41.0 / 40.2; x held over all groups before the next x part is slower (170).
//
// What bounds it: the power of the package.  11x11 on 8192^2 issues 180 GFLOP; a large bf16 matrix product reaches 1.32 PFLOP/s on this
// card (1.39 on another), at 1.87 GHz, and at that rate the instructions alone take 136 us (15x15 on 3001x4003: 50 GFLOP, 38 us).  With random
// data the clock falls to 1.86 GHz in this kernel (155 us; 2.38 with an image of zeros, 123), and what saves clocks lowers it further.  By the
// counters the matrix cores are busy for 62 % of the clocks and other vector instructions for 21 %, LDS for 26 %, HBM reads are
// 1.12 and 1.24 times the image.
// Measured (us, the best vector kernel / this, short runs): 11x11 on 8192^2 256 / 141, 15x15 on 3001x4003 87 / 44, 12x12 on 5630^2 146 / 78, 9x13 on 4096^2 72 / 42.
// Tried on that account: the next chunk's split placed between the matrix instructions (an MFMA leaves room for two vector instructions),
// 162 -> 165 us on 8192^2 and 0 to 7 % slower elsewhere; eight wavefronts a workgroup, one a CU, all
// in step (they end together, at 1.57 GHz), 158 - 165.
// Tried: 272 input columns per chunk (one wavefront splits a fifth piece and the others wait: 11x11 190 us with two
// accumulators an output), one accumulator (2 % faster, but errors of 1.8e-7 instead of 6e-8), stores behind per-lane
// branches (every chunk then waits for the stores of the one before), three workgroups a CU (spills at NS = 7, level
// below).  Reads of 16 bytes from LDS at 8-byte alignment are slow: a window is two 8-byte (8 x 2: four 4-byte) reads.
#include "launch.h"
#include "matrix_blocks.h"
#include "split_bf16.h"
#include "systolic.h"

#include <limits.h>

#include <type_traits>

namespace sysconv {
namespace {

typedef unsigned short us2 __attribute__((ext_vector_type(2)));
typedef const float __attribute__((address_space(4)))* kernarg_floats;

constexpr int kCols = 240;                  // output columns of a workgroup's strip (64 for three wavefronts, 48 for the last)
constexpr int kInCols = 256;                // input columns of a chunk (a filter is at most 15 wide)
constexpr int kChunk = 16;                  // input rows of a chunk: 8 units
constexpr int kUnits = kChunk / 2;
constexpr int kRow = 3 * kInCols;           // a row in LDS, in bf16 numbers: 256 first parts, 256 second, 256 third
constexpr int kBuf = kChunk * kRow;
constexpr int kMaxChunks = 64;              // chunks of a row block, the one that only finishes groups among them (marks fill 64 bits)
constexpr int kPlainRows = 4;               // output rows a wavefront takes together in plain_rows, and input rows in flight
constexpr unsigned short kHuge = (127 + 80) << 7;          // upper half of the bits of 2^80
constexpr unsigned kHugeBits = (kHuge << 16) - 0x8000u;    // the least number whose first part is 2^80

template <int JC, int NS>
struct SplitShape {
    static constexpr int JR = 16 / JC;                     // output rows of a group
    static constexpr int NB = 64 / (16 * JC);       // instruction columns (16 bases) of a wavefront's 64 columns
    static constexpr int UG = JR / 2;                      // units from one group to the next
    static constexpr int GROUPS = kChunk / JR;             // groups that start in a chunk
    static constexpr int LIVE = 4;                         // sums of a group live in slot (group mod LIVE)
    static constexpr int PARTS = JC == 4 ? 2 : 1;          // sums of an output: x1f1 apart from the small products
    static constexpr int TROWS = 2 * NS + JR - 1;          // rows of the zero-padded taps
    static constexpr int TCOLS = 16 + JC - 1;
    static constexpr int TAPS = JC == 4 ? (2 * NS - 3) * 13 : (2 * NS - 7) * 15;       // most taps of a filter that the shape serves
    static_assert(NS - 1 < LIVE * UG, "a slot is free again before its next group starts");
    static_assert((LIVE % GROUPS) == 0 || GROUPS == LIVE, "slots repeat over the chunks");
};

// Where the marked chunks of a row block make the matrix cores' work pointless: the block then ends with plain_rows for
// all rows from the present chunk on.  Rows of a chunk that hold such values cost the 16 (11x11) to 24 (15x15) output rows they
// reach, 2.3 to 3.8 chunk times, up to 4 to 6 where they are all over the chunk; plain_rows alone takes 2.3 to 2.5 a chunk: level
// where between one chunk in 2 and one in 4 is marked.  An eighth of the block has to be: a margin of such values is no reason
// (40 rows at the top and the bottom of 8192^2, 11x11: 322 us given up, 171 not).  One marked chunk alone ends only blocks of
// one or two.
__device__ __forceinline__ bool too_many(unsigned long long marks, int seen, int chunks)
{
    const int marked = __builtin_popcountll(marks);
    return marked * 3 > seen && marked * 8 > chunks && (marked > 1 || chunks <= 2);
}

// The output rows [ra, rb) of the strip with plain multiply-adds, as an FBS array whose width is known at compile time:
// a wavefront walks down the input rows of up to kPlainRows output rows (an even share of each pass), builds each row's window once and applies it to every
// output row whose filter covers it.  The filter rows in use are in registers (from tap0, row 0 of the taps in LDS, one
// a step ahead of its use): two wavefronts a SIMD do not hide the latency of scalar loads (11x11 on 4096^2, a marked value in
// every chunk: 127 us with taps in scalar registers, 95 this way; 1263 with one output row a wavefront and a load a tap).  On
// large images it issues 1.16 times the vector instructions of SBM.  (col_b, off): the lane's load.
template <int KW, int TapPitch, class PutRight>
__device__ __forceinline__ void plain_rows(const float* tap0, const float* __restrict__ x, float* __restrict__ y,
                                           unsigned col_b, int off, long long xp, int col, int ow_strip, long long yp, int kh,
                                           int ra, int rb, bool edge, int wave, PutRight put_right)
{
    if (ra >= rb) return;
    constexpr int kWaves = kBlock / kWave;
    const int passes = (rb - ra + kPlainRows * kWaves - 1) / (kPlainRows * kWaves), share = (rb - ra + kWaves * passes - 1) / (kWaves * passes);
    for (int r = ra + share * wave; r < rb; r += share * kWaves) {
        const int rows_out = min(share, rb - r), rows_in = rows_out - 1 + kh;
        const float* xrow = x + (long long)r * xp;
        f4u v[kPlainRows];
        auto load_row = [&](int rho, f4u& d) {                             // past the last row: the last row again
            d = *reinterpret_cast<const f4u*>(reinterpret_cast<const char*>(xrow + (long long)min(rho, rows_in - 1) * xp) + col_b);
        };
        float wv[kPlainRows][KW];                                          // filter row p in slot p mod kPlainRows
        auto load_taps = [&](int p, float (&w)[KW]) {
            int at = min(p, kh - 1) * TapPitch;
            asm("" : "+v"(at));                                            // one address for all taps of the row
            const float* t = tap0 + at;
#pragma unroll
            for (int q = 0; q < KW; ++q) w[q] = t[q];
        };
#pragma unroll
        for (int i = 0; i < kPlainRows; ++i) load_row(i, v[i]);
        load_taps(0, wv[0]);
        float acc[kPlainRows][4];
#pragma unroll
        for (int j = 0; j < kPlainRows; ++j) acc[j][0] = acc[j][1] = acc[j][2] = acc[j][3] = 0.0f;
#pragma nounroll
        for (int rho0 = 0; rho0 < rows_in; rho0 += kPlainRows) {
#pragma unroll
            for (int i = 0; i < kPlainRows; ++i) {
                const int rho = rho0 + i;
                if (rho >= rows_in) break;                                 // uniform
                f4u t = v[i];
                load_row(rho + kPlainRows, v[i]);
                if (edge) {
                    asm volatile("");                                      // a branch, not selects in every strip
                    put_right(t, off);
                }
                float win[KW + 3] = {t.x, t.y, t.z, t.w};
#pragma unroll
                for (int m = 4; m < KW + 3; ++m) win[m] = from_lane_above(win[m - 4]);
#pragma unroll
                for (int j = kPlainRows - 1; j >= 0; --j) {
                    if (j < rows_out && rho - j >= 0 && rho - j < kh) {    // uniform
#pragma unroll
                        for (int q = 0; q < KW; ++q)
#pragma unroll
                            for (int k = 0; k < 4; ++k)
                                acc[j][k] = __builtin_fmaf(wv[(i - j + kPlainRows) % kPlainRows][q], win[q + k], acc[j][k]);
                    }
                    if (j == kPlainRows - 1) load_taps(rho + 1, wv[(i + 1) % kPlainRows]);     // that slot is free now
                }
            }
        }
#pragma unroll
        for (int j = 0; j < kPlainRows; ++j)
            if (j < rows_out) store4_guarded<false>(y + (long long)(r + j) * yp, col, ow_strip, acc[j]);
    }
}

// Filter widths the kernels are built for: all that pay (conv2d_split_pays).
__host__ __device__ constexpr int least_width(int jc) { return jc == 4 ? 5 : 11; }
__host__ __device__ constexpr int most_width(int jc) { return jc == 4 ? 13 : 15; }

template <int JC, int NS>
__global__ __launch_bounds__(kBlock, 2) void conv2d_split_kernel(
    TapsOf<SplitShape<JC, NS>::TAPS> taps, const float* __restrict__ x, float* __restrict__ y, int h, int w_img, long long xp, int oh, int ow,
    long long yp, int kh, int kw, int rows, int row_blocks, int strips, int per_xcd, unsigned tiny_below)
{
    (void)taps;
    using S = SplitShape<JC, NS>;
    constexpr int JR = S::JR, NB = S::NB, UG = S::UG, LIVE = S::LIVE, GROUPS = S::GROUPS;
    kernarg_floats taps_f = (kernarg_floats)__builtin_amdgcn_kernarg_segment_ptr();

    __shared__ __attribute__((aligned(16))) __bf16 parts[2 * kBuf + 32];     // (windows of the last wavefront reach past a row)
    __shared__ float tpad[S::TROWS * S::TCOLS];
    __shared__ unsigned marks[kMaxChunks / 32], quads[kMaxChunks / 8];     // a bit per chunk, and per four rows of a chunk

    const int g = xcd_contiguous(blockIdx.x, per_xcd);
    if (g >= row_blocks * strips) return;                                  // (the whole workgroup)
    const int rblk = g / strips, strip = g - rblk * strips;                // workgroups walk along the rows of the image
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = wave_in_block();
    const int c0 = strip * kCols;
    const int r0 = rblk * rows;
    const int ow_strip = min(ow, c0 + kCols);                              // columns the strip stores: up to here
    const int rows_out = min(rows, oh - r0);
    // chunks 0 .. chunks-1 start groups; one more holds the units that only finish them
    const int chunks = (rows_out + kChunk - 1) / kChunk;
    const int groups = (rows_out + JR - 1) / JR, units = UG * (groups - 1) + NS;
    const int last_row = h - 1;
    const bool edge = c0 + kInCols > w_img;                                // uniform

    // ---------------------------------------------------------------- a chunk into registers
    // Wavefront v takes rows v, v+4, v+8, v+12 (1 KB each).  Loads that would reach past the row's end start at its last
    // four columns instead and are put right before the split.
    const int col_m = min(c0 + kTile * lane, w_img - 4), off_m = c0 + kTile * lane - col_m;
    const unsigned col_b = (unsigned)col_m * (unsigned)sizeof(float);
    f4u raw[4];
    auto load_chunk = [&](int c) {
        const int rbase = r0 + c * kChunk;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            raw[k] = *reinterpret_cast<const f4u*>(reinterpret_cast<const char*>(x + (long long)min(rbase + wave + 4 * k, last_row) * xp) + col_b);
    };
    auto put_right = [&](f4u& v, int off) {                                // columns past the image read as 0
        if (off & 1) v = f4u{v.y, v.z, v.w, 0.0f};
        if (off & 2) v = f4u{v.z, v.w, 0.0f, 0.0f};
        if (off > 3) v = f4u{0.0f, 0.0f, 0.0f, 0.0f};
    };
    unsigned tiny;
    us2 huge;
    auto put = [&](const f4u& v, __bf16* dst) {
        u2 p1, p2, p3;
        unsigned a, b, c;
        split2(v.x, v.y, a, b, c);
        p1.x = a; p2.x = b; p3.x = c;
        split2(v.z, v.w, a, b, c);
        p1.y = a; p2.y = b; p3.y = c;
        *reinterpret_cast<u2*>(dst) = p1;
        *reinterpret_cast<u2*>(dst + kInCols) = p2;
        *reinterpret_cast<u2*>(dst + 2 * kInCols) = p3;
#pragma unroll
        for (int i = 0; i < 4; ++i) tiny = min(tiny, (__builtin_bit_cast(unsigned, (float)v[i]) << 1) - 1u);   // +-0: the largest
        huge = __builtin_elementwise_max(huge, __builtin_bit_cast(us2, p1.x & 0x7fff7fffu));
        huge = __builtin_elementwise_max(huge, __builtin_bit_cast(us2, p1.y & 0x7fff7fffu));
    };
    auto store_chunk = [&](int c, auto edge_tag) {
        __bf16* buf = parts + (c & 1) * kBuf;
        tiny = 0xffffffffu;
        huge = us2{0, 0};
        if constexpr (decltype(edge_tag)::value) {
#pragma unroll
            for (int k = 0; k < 4; ++k) put_right(raw[k], off_m);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) put(raw[k], buf + (wave + 4 * k) * kRow + kTile * lane);
        if (tiny < tiny_below || huge.x >= kHuge || huge.y >= kHuge) {     // rare: which of the lane's rows?
            unsigned rows_hit = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const unsigned bits = __builtin_bit_cast(unsigned, (float)raw[k][i]);
                    if ((bits << 1) - 1u < tiny_below || (bits & 0x7fffffffu) >= kHugeBits) rows_hit |= 1u << k;
                }
            atomicOr(marks + c / 32, 1u << (c % 32));
            atomicOr(quads + c / 8, rows_hit << (4 * (c % 8)));
        }
    };

    load_chunk(0);
    for (int e = threadIdx.x; e < S::TROWS * S::TCOLS; e += kBlock) {
        const int p = e / S::TCOLS - (JR - 1), q = e % S::TCOLS - (JC - 1);
        tpad[e] = p >= 0 && p < kh && q >= 0 && q < kw ? taps_f[p * kw + q] : 0.0f;
    }
    if (threadIdx.x < kMaxChunks / 32) marks[threadIdx.x] = 0;
    if (threadIdx.x < kMaxChunks / 8) quads[threadIdx.x] = 0;
    __syncthreads();

    // A operands: the Toeplitz form of the taps, constant for the whole kernel
    const int i16 = lane & 15, kb = lane >> 4;                             // operand coordinates of the lane
    b8 fa[NS][3];
    {
        const int jr = i16 / JC, jc = i16 % JC;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const float* t = tpad + (2 * s + (kb >> 1) - jr + JR - 1) * S::TCOLS + 8 * (kb & 1) - jc + JC - 1;
            u4 p[3];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                unsigned a, b, c;
                split2(t[2 * i], t[2 * i + 1], a, b, c);
                p[0][i] = a; p[1][i] = b; p[2][i] = c;
            }
#pragma unroll
            for (int j = 0; j < 3; ++j) fa[s][j] = __builtin_bit_cast(b8, p[j]);
        }
    }
    if (edge) store_chunk(0, std::true_type{});
    else store_chunk(0, std::false_type{});
    load_chunk(1);
    __syncthreads();

    f4 acc[LIVE][NB][S::PARTS];
    const int win0 = (kb >> 1) * kRow + wave * 64 + JC * i16 + 8 * (kb & 1);
    const int out_col = c0 + wave * 64 + JC * i16;

    // Outputs of group `grp` of the block: lane (i16, kb) holds offsets j = 4 kb .. 4 kb + 3.  Buffer stores drop the
    // lanes whose offset is out of range, so no store hides behind a branch: the compiler can then count the stores
    // that are younger than the loads in flight and wait for the loads alone.
    const unsigned pitch_b = (unsigned)yp * (unsigned)sizeof(float);
    auto store_group = [&](int grp, const f4 (&sums)[NB][S::PARTS], auto edge_tag) {
        float* base = y + (long long)(r0 + grp * JR) * yp;                 // uniform
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(base, 0, 0x7fffffff, 0x00020000);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const u4 ob = __builtin_bit_cast(u4, S::PARTS == 2 ? sums[nb][0] + sums[nb][S::PARTS - 1] : sums[nb][0]);
            const int col = out_col + nb * 16 * JC;
            constexpr int kRows = 4 / JC;                                  // rows of the lane's four outputs
#pragma unroll
            for (int k = 0; k < kRows; ++k) {
                const int rr = kb * kRows + k;
                const unsigned off = (unsigned)rr * pitch_b + (unsigned)col * 4u;
                const bool row_ok = grp * JR + rr < rows_out;
                if constexpr (!decltype(edge_tag)::value) {                // 256 input columns: 240 outputs at least
                    const unsigned to = row_ok && col < c0 + kCols ? off : kNowhere;
                    if constexpr (JC == 4)
                        __builtin_amdgcn_raw_buffer_store_b128(ob, rsrc, to, 0, kNonTemporal);
                    else
                        __builtin_amdgcn_raw_buffer_store_b64(u2{ob[2 * k], ob[2 * k + 1]}, rsrc, to, 0, kNonTemporal);
                } else {
                    const int left = row_ok ? ow_strip - col : 0;
                    if constexpr (JC == 4)
                        __builtin_amdgcn_raw_buffer_store_b128(ob, rsrc, left >= JC ? off : kNowhere, 0, kNonTemporal);
                    else
                        __builtin_amdgcn_raw_buffer_store_b64(u2{ob[2 * k], ob[2 * k + 1]}, rsrc, left >= JC ? off : kNowhere, 0, kNonTemporal);
#pragma unroll
                    for (int i = 0; i < JC - 1; ++i)
                        __builtin_amdgcn_raw_buffer_store_b32(ob[JC * k + i], rsrc, i < left && left < JC ? off + 4u * i : kNowhere, 0, kNonTemporal);
                }
            }
        }
    };

    // One chunk: FIRST has no groups from before it, FULL starts all of its own (else it is looked at run time which groups there are, and how many
    // units are left).  SLOT0: slot of the chunk's first group.
    auto compute = [&](int c, auto edge_tag, auto first_tag, auto full_tag, auto slot_tag) {
        constexpr bool FIRST = decltype(first_tag)::value, FULL = decltype(full_tag)::value;
        constexpr int SLOT0 = decltype(slot_tag)::value;
        int at = (c & 1) * kBuf + win0;
        const int left = FULL ? kUnits : units - c * kUnits;
        constexpr int SETS = NB == 1 ? 2 : 1;                              // windows are read a step ahead where registers allow it
        b8 win[SETS][3];
        auto read = [&](int t) {                                           // windows of step t = NB unit + nb; a unit's address is current
#pragma unroll
            for (int j = 0; j < 3; ++j)
                __builtin_memcpy(&win[t % SETS][j], __builtin_assume_aligned(parts + at + (t % NB) * 16 * JC + j * kInCols, 2 * JC), 16);
        };
        if constexpr (SETS == 2) read(0);
#pragma unroll
        for (int u = 0; u < kUnits; ++u) {
            if (!FULL && u >= left) break;                                 // uniform
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const int t = u * NB + nb;
                if (SETS == 2 || nb == 0) __builtin_amdgcn_sched_barrier(0);
                if (SETS == 1) read(t);
                if (nb + 1 == NB) {
                    at += 2 * kRow;
                    asm("" : "+v"(at));
                }
                if (SETS == 2 && t + 1 < kUnits * NB) read(t + 1);
                const b8 (&b)[3] = win[t % SETS];
#pragma unroll
                for (int lg = -LIVE; lg < GROUPS; ++lg) {
                    const int s = u - UG * lg;
                    if (s < 0 || s >= NS || (FIRST && lg < 0)) continue;
                    if (!FULL && (c * GROUPS + lg < 0 || c * GROUPS + lg >= groups)) continue;     // uniform
                    constexpr int kLo = S::PARTS - 1;
                    f4& hi = acc[(lg + SLOT0 + LIVE) % LIVE][nb][0];
                    f4& lo = acc[(lg + SLOT0 + LIVE) % LIVE][nb][kLo];
                    if (s == 0) hi = lo = f4{0.0f, 0.0f, 0.0f, 0.0f};
                    lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[s][2], b[0], lo, 0, 0, 0);
                    lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[s][1], b[0], lo, 0, 0, 0);
                    lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[s][1], b[1], lo, 0, 0, 0);
                    lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[s][0], b[1], lo, 0, 0, 0);
                    lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[s][0], b[2], lo, 0, 0, 0);
                    hi = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[s][0], b[0], hi, 0, 0, 0);
                }
            }
#pragma unroll
            for (int lg = -LIVE; lg < GROUPS; ++lg) {
                if (u - UG * lg != NS - 1 || (FIRST && lg < 0)) continue;
                if (!FULL && (c * GROUPS + lg < 0 || c * GROUPS + lg >= groups)) continue;
                store_group(c * GROUPS + lg, acc[(lg + SLOT0 + LIVE) % LIVE], edge_tag);
            }
        }
    };
    // Chunk c+1 goes to LDS and chunk c+2 is asked for while chunk c is used; the buffer that chunk c+1
    // takes was last read before the barrier that ended chunk c-1.  Returns the chunk at which the block was given up
    // (too_many), or chunks + 1.
    auto marked_up_to = [&](int c) {                                       // final, and the same to all wavefronts, once chunk c begins
        const unsigned lo = __builtin_amdgcn_readfirstlane(marks[0]), hi = __builtin_amdgcn_readfirstlane(marks[1]);
        return ((unsigned long long)hi << 32 | lo) & (~0ull >> (kMaxChunks - 1 - c));
    };
    auto run = [&](auto edge_tag) -> int {
        auto advance = [&](int c, auto first_tag, auto slot_tag) {
            store_chunk(c + 1, edge_tag);
            load_chunk(c + 2);
            compute(c, edge_tag, first_tag, std::true_type{}, slot_tag);
            lds_barrier();
        };
        using Slot0 = std::integral_constant<int, 0>;
        using Slot1 = std::integral_constant<int, GROUPS % LIVE>;          // slots of the odd chunks
        if (__builtin_amdgcn_readfirstlane(marks[0]) & 1u) {
            const bool full = (__builtin_amdgcn_readfirstlane(quads[0]) & 15u) == 15u;  // such values all over the first chunk
            if ((full && chunks <= 6) || too_many(1, 1, chunks)) return 0;
        }
        auto swap_slots = [&]() {
            if constexpr (Slot1::value != 0) {
#pragma unroll
                for (int i = 0; i < Slot1::value; ++i)
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                        for (int p = 0; p < S::PARTS; ++p) {
                            const f4 t = acc[i][nb][p];
                            acc[i][nb][p] = acc[i + Slot1::value][nb][p];
                            acc[i + Slot1::value][nb][p] = t;
                        }
            }
        };
        const int full = groups / GROUPS;
        int c = 0;
        if (full > 0) {
            advance(0, std::true_type{}, Slot0{});
            c = 1;
            for (; c + 2 <= full; c += 2) {
                if (too_many(marked_up_to(c), c + 1, chunks)) return c;
                advance(c, std::false_type{}, Slot1{});
                advance(c + 1, std::false_type{}, Slot0{});
            }
            if (c < full) {
                advance(c, std::false_type{}, Slot1{});
                ++c;
            }
        }
        if (c & 1) swap_slots();
#pragma nounroll
        for (; c * kUnits < units; ++c) {                                  // (few: one body, slots as in the even chunks)
            if (c > 0 && c < chunks && too_many(marked_up_to(c), c + 1, chunks)) return c;
            if ((c + 1) * kUnits < units) {
                store_chunk(c + 1, edge_tag);
                if ((c + 2) * kUnits < units) load_chunk(c + 2);
            }
            compute(c, edge_tag, std::false_type{}, std::false_type{}, Slot0{});
            swap_slots();
            lds_barrier();
        }
        return chunks + 1;
    };
    const int stop = edge ? run(std::true_type{}) : run(std::false_type{});

    unsigned long long todo = marked_up_to(chunks);
    if (todo == 0) return;
    // The output rows that the marks reach, once more; neighbouring and overlapping ones together.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                       // the stores above are done before any of these
    __syncthreads();
    auto again = [&](int ra, int rb) {
        auto with = [&](auto kw_tag, auto self) {
            constexpr int KW = decltype(kw_tag)::value;
            if (kw == KW)
                plain_rows<KW, S::TCOLS>(tpad + (JR - 1) * S::TCOLS + JC - 1, x, y, col_b, off_m, xp, c0 + kTile * lane, ow_strip,
                                         yp, kh, r0 + ra, r0 + rb, edge, wave, put_right);
            else if constexpr (KW < most_width(JC))
                self(std::integral_constant<int, KW + 1>{}, self);
        };
        with(std::integral_constant<int, least_width(JC)>{}, with);
    };
    if (stop <= chunks) todo = (todo & ~(~0ull << stop)) | 1ull << stop;   // (from there on: all that is left)
    int k = 0;
    unsigned four = 0;                                                     // marked row quads of chunk k that are still to come
    auto next = [&]() -> int {                                             // the next marked row quad of the block, or -1
        while (four == 0) {
            if (todo == 0) return -1;
            k = __builtin_ctzll(todo);
            todo &= todo - 1;
            four = k == stop ? 1u : (__builtin_amdgcn_readfirstlane(quads[k / 8]) >> (4 * (k % 8))) & 15u;
        }
        const int i = __builtin_ctz(four);
        four &= four - 1;
        return 4 * k + i;
    };
    auto first_row = [](int quad) {                                        // group at row R: input rows R .. R + 2 NS - 1
        const int r = 4 * quad - (2 * NS - 1);
        return r <= 0 ? 0 : (r + JR - 1) / JR * JR;
    };
    int quad = next();
    while (quad >= 0) {
        const int ra = first_row(quad);
        int rb;
        do {
            rb = k == stop ? rows_out : (4 * quad + 3) / JR * JR + JR;
            quad = next();
        } while (quad >= 0 && first_row(quad) <= rb);
        again(ra, min(rb, rows_out));
    }
}

// Output rows of a workgroup's block: whole groups, at most kMaxChunks - 1 chunks.
template <int JC, int NS>
int block_rows(int oh, int ow)
{
    using S = SplitShape<JC, NS>;
    const int strips = (ow + kCols - 1) / kCols, all = (oh + S::JR - 1) / S::JR;
    return S::JR * matrix_block_groups(all, strips, NS, S::UG, S::NB, 12.0, (kMaxChunks - 1) * kChunk / S::JR);
}

template <int JC, int NS>
hipError_t launch_split(const float* x, int h, int w, size_t xp, const float* f, int kh, int kw, float* y, size_t yp,
                        hipStream_t s)
{
    using S = SplitShape<JC, NS>;
    const TapsOf<S::TAPS> taps(f, kh * kw);
    const int oh = h - kh + 1, ow = w - kw + 1;
    const int strips = (ow + kCols - 1) / kCols;
    const long long rows = block_rows<JC, NS>(oh, ow);
    const int row_blocks = (int)((oh + rows - 1) / rows);
    const long long groups = (long long)row_blocks * strips;
    const long long per_xcd = (groups + kXcds - 1) / kXcds;
    const long long blocks = per_xcd * kXcds;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((conv2d_split_kernel<JC, NS>), dim3((unsigned)blocks), dim3(kBlock), 0, s, taps, x, y, h, w,
                       (long long)xp, oh, ow, (long long)yp, kh, kw, (int)rows, row_blocks, strips, (int)per_xcd, split_tiny_limit(f, kh * kw));
    return hipGetLastError();
}

int split_units(int kh, int kw)                 // NS of the kernel that serves the filter
{
    if (kh <= 13 && kw <= 13) return kh <= 5 ? 4 : (kh + 4) / 2;           // ceil((kh + 3) / 2), at least 4
    return kh <= 7 ? 8 : (kh + 8) / 2;                                     // ceil((kh + 7) / 2), at least 8
}

}  // namespace

// Filters and images the kernel takes: taps that the split carries, widths that plain_rows is built for (and with them rows of at
// least four columns, the 16 bytes of a load), output pitches whose rows of a group lie within the 2 GB of a buffer
// descriptor, heights whose row numbers stay in an int: the chunks that a block asks for in advance reach up to
// three chunks past its last output row, and they are clamped to the image only after that sum.
bool conv2d_split_takes(int h, int w, size_t yp, const float* f, int kh, int kw)
{
    if (h > INT_MAX - 4 * kChunk) return false;
    if (yp > ((size_t)1 << 25) || kh > kMaxK2D || kw > kMaxK2D || w < kw) return false;
    if (kw < least_width(kh <= 13 && kw <= 13 ? 4 : 2)) return false;
    return split_takes_taps(f, kh * kw);
}

// Where AUTO takes the split kernel rather than the best vector-ALU kernel: where it is faster, and for filters with a side of 12 to 15 or with both of 8 and more (squares that SBM is built for aside), which it has
// served longest, also where it is not, for its
// smaller error (2-norm against 64 bits, images on [0, 1), split / FBS: 3x12 3.2e-8 / 1.2e-7, 4x13 3.5e-8 / 1.3e-7, 5x12 4.3e-8 / 1.9e-7, 6x12 4.5e-8 / 2.0e-7, 7x13 4.5e-8 / 1.2e-7,
// 13x5 4.3e-8 / 1.8e-7, 12x7 4.8e-8 / 1.5e-7, 6x14 1.2e-7 / 1.5e-7, 7x15 6.6e-8 / 1.1e-7).  Its time goes with the units, theirs with
// the kh*kw taps, so the lines are drawn in taps per unit t; measured on squares of 277 .. 6500 and some other images (us, split / vector):
//   14 or 15 rows or columns: from 11 columns and 10 taps a unit on, at every size (15x15 8.3 / 6.7 on 300x400, 9.7 / 9.5 on 700^2, 25.2 / 47.2 on 2300^2; 14x11 9.7 / 7.8 on 700^2, 24.6 / 32.3 on 2300^2; 7x15 6.2 / 7.5
//   on 500^2, 12.9 / 13.5 on 1500^2; 6x14 7.8 / 6.4 on 700^2, 19.7 / 21.1 on 2300^2).  With fewer columns sums over 8 to 11 units in one accumulator are no more exact than the vector kernels' (14x9: off by 2.3e-7 against 2.2e-7;
//   14x11 1.9e-7 against 2.05e-7).
//   A side of 12 or 13, or both 8 or more and not a square up to 11x11: from 12 taps a unit on at every size (4x12 4.6 / 3.7 on 500^2, 6.7 / 5.7 on 1000^2, 13.6 / 15.5 on 2300^2; 5x13 6.7 / 6.4 and
//   13.9 / 18.7; 7x12 4.9 / 6.1 on 500^2, 14.7 / 21.1 on 2300^2), with fewer on images of 2 M outputs and more, the larger the closer they are to 7 (12x7 18.3 / 19.0 on 2200^2;
//   12x6 18.0 / 17.4 on 2200^2, 27.1 / 30.7 on 3000^2; 13x5 27.0 / 26.2 on 3000^2, 50 / 52 on 4500^2).  Three rows leave half of the four units they take empty: from 5 M outputs on (3x13 19.4 / 18.7 on 3000^2, 35.5 / 37.3 on
//   4500^2; 3x12 35.5 / 35.3 and 83 / 75 on 6500^2).  With both sides 8 or more at
//   every size: the FBS strips are up to 30 % quicker below 1 M outputs (10x8, t = 11.4, 5.1 / 4.3 on 300x400, 7.2 / 5.5 on 700^2, 8.2 / 7.7 on 1000^2, 17.4 / 19.9 on 2300^2; 8x10 6.8 / 5.4, 7.7 / 7.9, 16.1 / 20.3 on the last three; 12x12 5.5 / 5.2,
//   7.7 / 7.3, 8.9 / 10.9, 18.9 / 31.3, 78 / 146 on 5630^2), but their error is three times as large (10x8 on 600^2 1.7e-7 / 4.8e-8).
//   8x8 .. 11x11 (SBM) and filters of up to 11 with one side up to 7 (compile-time FBS): those kernels are quick on small images, and the split kernel wins once the
//   image is large enough, the sooner the more taps a unit has.  Where the two are level, in M outputs: 8x8 (t = 10.7) 5, 9x9 (13.5) 2.2, 10x10 (14.3) 2 (and 2046x1002 outputs,
//   five strips, 12.1 / 11.05), 11x11 (17.3) 0.5 .. 1.3: from 12 / (t - 9) on, as other filters of 64 taps and more do at the latest; 9x7 (10.5) 3 .. 4, 6x10 (12) 3, 6x11 (13.2) and 7x10 (14) 1.6 (752x2101 9.1 / 8.2 and 9.1 / 8.5,
//   894x2590 9.3 / 10.1 and 9.4 / 10.5), 7x11 (15.4) 0.8 .. 1.6: from 0.05 (18.5 - t)^2 on, below t = 14.2 from 1.6 on and else from 0.9 (7x11 on 737x850 6.6 / 6.05), with fewer than 64 taps from
//   0.075; four and five rows from 2.6 (5x11 on 508x4639 9.1 / 8.3, 1089x2229 9.05 / 9.9).  (8x8 on 3000x4000 29.6 / 35.1,
//   9x9 29.2 / 42.2, 11x11 on 1000^2 8.3 / 9.2, 420x1344 7.3 / 7.8.)  Below t = 8.5 and below 44
//   taps they are level at best (11x5 75 / 71 on 5630^2; 6x7 54 / 48 on 6300x4466; 9x6 with a thirtieth of padding 19.1 / 17.7 on 2162x3140), and 7x7 is level (59.5 / 62).
// What the kernels compute for padding counts: strips of 240 columns and chunks of 16 rows here, about 252 columns and 8 rows there.  In full where the two are close: a strip more here than there
// costs what it computes (5x9 on 7737x723 17.1 / 14.2; 7x8 on 6757x721 16.5 / 14.5; 6x8 on 6483x1203 21.5 / 18.8; 7x9 on 1607x1700 11.5 / 10.05; with any padding
// up to a quarter let pass, 40 of 228 random calls beyond the first lines were slower by more than 5 %, up to 20 %; with this none of them and one of 120 others, 6766x959 6x8 by 7 %).  Where the gain is large or the split stays for its
// error, padding of a half (10x8: a quarter) more than theirs is let pass.
bool conv2d_split_pays(int oh, int ow, int kh, int kw)
{
    const int taps = kh * kw, units = split_units(kh, kw);
    const double outputs = (double)oh * ow;
    const int cols = kTile * (kWave - halo_lanes(kw));
    const double theirs = (double)(((long long)ow + cols - 1) / cols * 252) * (double)(((long long)oh + 7) / 8 * 8);
    const double ours = (double)(((long long)ow + kCols - 1) / kCols * kCols) * (double)(((long long)oh + kChunk - 1) / kChunk * kChunk);
    auto taps_a_unit = [&](double pad) { return taps * (pad * theirs < ours ? pad * theirs / ours : 1.0) / units; };
    if (kh > 13 || kw > 13) return kw >= 11 && taps >= 10 * units;
    const bool both = kh >= 8 && kw >= 8;
    const double loose = taps_a_unit(1.5), t = taps_a_unit(1.0);
    if (kh > 11 || kw > 11 || (both && kh != kw)) {
        if (kh <= 3) return loose >= 8.0 && outputs >= 5e6;
        return taps >= 12 * units || (both && taps_a_unit(1.25) >= 8.1) || (loose >= 8.0 && outputs >= 2e6 && outputs * (loose - 7.0) >= 4e6);
    }
    if (taps >= 64 && outputs * (loose - 9.0) >= 12e6) return true;
    if (kh == kw || t < 8.5 || taps < 44) return false;
    return outputs >= (kh <= 5 ? 2.6e6 : t < 14.2 ? 1.6e6 : 0.9e6) && outputs >= (taps < 64 ? 0.075e6 : 0.05e6) * (18.5 - t) * (18.5 - t);
}

namespace {
template <class F>
auto with_shape(int kh, int kw, F&& f)           // f<JC, NS> of the kernel that serves the filter
{
    const int units = split_units(kh, kw);
    using Four = std::integral_constant<int, 4>;
    using Two = std::integral_constant<int, 2>;
    if (kh <= 13 && kw <= 13) {
        switch (units) {
        case 4: return f(Four{}, std::integral_constant<int, 4>{});
        case 5: return f(Four{}, std::integral_constant<int, 5>{});
        case 6: return f(Four{}, std::integral_constant<int, 6>{});
        case 7: return f(Four{}, std::integral_constant<int, 7>{});
        default: return f(Four{}, std::integral_constant<int, 8>{});
        }
    }
    switch (units) {
    case 8: return f(Two{}, std::integral_constant<int, 8>{});
    case 9: return f(Two{}, std::integral_constant<int, 9>{});
    case 10: return f(Two{}, std::integral_constant<int, 10>{});
    default: return f(Two{}, std::integral_constant<int, 11>{});
    }
}
}  // namespace

int conv2d_split_block_rows(int oh, int ow, int kh, int kw)
{
    return with_shape(kh, kw, [&](auto jc, auto ns) { return block_rows<decltype(jc)::value, decltype(ns)::value>(oh, ow); });
}

hipError_t launch_conv2d_split(const float* x, int h, int w, size_t xp, const float* f, int kh, int kw, float* y,
                               size_t yp, hipStream_t s)
{
    return with_shape(kh, kw, [&](auto jc, auto ns) { return launch_split<decltype(jc)::value, decltype(ns)::value>(x, h, w, xp, f, kh, kw, y, yp, s); });
}

}  // namespace sysconv
