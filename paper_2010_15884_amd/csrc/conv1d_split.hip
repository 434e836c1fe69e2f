// 1-D valid convolution (paper Eq. 2) for long filters, on the matrix cores and in full fp32.
//
// Contraction.  One v_mfma_f32_16x16x32_bf16 multiplies a 16 x 32 by a 32 x 16 matrix.  A tile is 256 consecutive outputs:
//
//   N (16)  "bases": outputs c0 + 16 i, i = 0..15
//   M (16)  "offsets": the outputs c0 + 16 i + j next to a base
//   K       input offsets t = 0 .. k + 14, KS = ceil((k + 15) / 32) instructions of 32
//
// A[j][t] = w[t - j] (0 outside the filter) is the same for every tile and stays in registers; B[t][i] = x[c0 + 16 i + t] is eight
// consecutive inputs per lane; D gives a lane four consecutive outputs, so a store is 1 KB of the signal.
//
// Precision: three bf16 parts a number, six products, x1f1 summed apart from the small ones (split_bf16.h); off from 64-bit sums by
// 4.2e-8 where BFS is by 1.4e-7 (20 M, k = 63).  A tile one of whose inputs (or of whose right neighbour's) the split does not carry
// is left out and computed with plain multiply-adds when the wavefront has been through its run (plain_sums).
//
// Data path.  A wavefront walks along a run of tiles by itself: inputs are loaded 1 KB at a time, four tiles ahead, split once,
// written to two slots of LDS of its own as three planes of bf16, and read back as 16-byte windows.  No barrier after the taps
// are in place.  LDS is busy for 44 % of the clocks, half of that bank conflicts of the windows (16 bytes of padding per 256); a layout whose
// pieces change places in pairs instead, free of them by construction, is level to 2 % slower.
//
// What bounds it: HBM up to some 24 M inputs, then HBM and the set-up of a run (taps, first loads).  Measured (us, the best vector kernel / this):
// k = 63 on 20 M 51 / 28 (three inputs in turn, which the memory-side cache holds in part; in no cache 56 / 37 to 48), k = 64 on 300 K 6.5 / 3.7, on 4 M 14.4 / 9.1, on 2^26 149 / 94; k = 40 on 1 M 6.5 / 4.6, on 16 M 35.6 / 29,
// on 2^26 113 / 92; k = 28 on 2^26 100 / 93.  A signal with a marked value (NaN) in every tile takes 0.9 to 1.35 times what the best vector
// kernel takes (us, vector kernel / two tiles at a time behind the whole run / this: k = 28 on 300 K 4.3 / 5.5 / 4.7, 5 M 10.7 / 16.5 / 14.2,
// 20 M 31 / 47 / 29, 2^26 97 / 160 / 121, there with one in every other tile 97 / 159 / 132; k = 36 on 20 M 39 / 49 / 34; k = 63 on 20 M 52 / 71 / 50, 2^26
// 149 / 226 / 158), with one in every sixteenth tile less (k = 63 on 20 M 56 / 35 / 33).
// Tried: five wavefronts a SIMD for k > 49 (spills, twice the time), three (level to 8 % slower), six or eight tiles ahead (level), two
// (4 % slower), cacheable stores (level to 10 % slower), plain sums in the middle of the run (spills, or 452 us on 2^26 without LDS).
#include "bfs_blocks.h"
#include "launch.h"
#include "split_bf16.h"
#include "systolic.h"

#include <type_traits>

namespace sysconv {
namespace {

typedef const float __attribute__((address_space(4)))* kernarg_floats;

constexpr int kTileOut = kWave * kTile;     // outputs of a tile
constexpr int kWaves = kBlock / kWave;
constexpr int kAhead = 4;                   // tiles in registers on their way to LDS
constexpr int kLeadIn = 3;                  // zeros before the first tap in the argument block (bfs_blocks.h)
constexpr float kHuge = 0x1p80f - 0x1p71f;  // the least number whose first part is 2^80
constexpr int kPlane = 2 * (2 * kTileOut + 2 * 16);        // bytes of a plane: two slots of 256 numbers, 16 bytes of padding per 128
__device__ __forceinline__ constexpr int place(int e) { return 2 * e + 16 * (e >> 7); }    // byte of number e of a plane

// Tiles of outputs from `at` on with plain multiply-adds: a BFS array, every lane four outputs of each tile from its windows in LDS of the
// wavefront's own (from memory, one load a step, the latency showed: 2^26, k = 63, a marked value in every tile 452 us).
template <int N>
struct PlainInputs { f4u v[N + 1]; };                                      // the inputs of N tiles and the quads that reach past them
constexpr int kPastTile = (kMaxK1D + kTile) / kTile;                       // lanes with one
template <int N> constexpr int kStage = N * kTileOut + kPastTile * kTile;  // their windows in LDS

template <int N>
__device__ __forceinline__ void plain_load(const float* __restrict__ x, long long n, long long at, int lane, PlainInputs<N>& in)
{
    if (at + kStage<N> <= n) {                                             // uniform
#pragma unroll
        for (int r = 0; r <= N; ++r)
            in.v[r] = *reinterpret_cast<const f4u*>(x + at + r * kTileOut + kTile * (r < N ? lane : min(lane, kPastTile - 1)));
    } else {
#pragma unroll
        for (int r = 0; r <= N; ++r) {
            float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            if (r < N || lane < kPastTile) load4_guarded<false>(x, at + r * kTileOut + kTile * lane, n, v);
            in.v[r] = f4u{v[0], v[1], v[2], v[3]};
        }
    }
}

template <int N>
__device__ __forceinline__ void plain_stage(const PlainInputs<N>& in, int lane, float* stage)
{
    wave_exchange();
#pragma unroll
    for (int r = 0; r <= N; ++r)
        if (r < N || lane < kPastTile)
            *reinterpret_cast<f4*>(stage + r * kTileOut + kTile * lane) = f4{in.v[r].x, in.v[r].y, in.v[r].z, in.v[r].w};
    wave_exchange();
}

template <int N>
__device__ __forceinline__ void plain_sums(kernarg_floats tw, int k, int lane, const float* stage, float (&acc)[N][4])
{
    const float* mine = stage + kTile * lane;
    auto weights = [&](int b, float (&wv)[7]) {
#pragma unroll
        for (int i = 0; i < 7; ++i) wv[i] = tw[4 * b + i];
    };
    auto window = [&](int r, int b, float (&xa)[4]) {
        const f4 t = *reinterpret_cast<const f4*>(mine + r * kTileOut + 4 * b);
        xa[0] = t.x; xa[1] = t.y; xa[2] = t.z; xa[3] = t.w;
    };
    float xa[4], wv[7];
    weights(0, wv);
#pragma unroll
    for (int r = 0; r < N; ++r) {
        acc[r][0] = acc[r][1] = acc[r][2] = acc[r][3] = 0.0f;
        window(r, 0, xa);
        bfs_block<3, 6>(acc[r], xa, wv);                                   // (k >= 4)
    }
    int b = 1;
#pragma unroll 4
    for (; 4 * b + 3 <= k - 1; ++b) {
        weights(b, wv);
#pragma unroll
        for (int r = 0; r < N; ++r) {
            window(r, b, xa);
            bfs_block<0, 6>(acc[r], xa, wv);
        }
    }
#pragma nounroll
    for (; 4 * b <= k + 2; ++b) {
        weights(b, wv);
        float xs[N][4];
#pragma unroll
        for (int r = 0; r < N; ++r) window(r, b, xs[r]);
        auto last = [&](auto hi) {
#pragma unroll
            for (int r = 0; r < N; ++r) bfs_block<0, decltype(hi)::value>(acc[r], xs[r], wv);
        };
        switch (k + 2 - 4 * b) {                                           // uniform
        case 0: last(std::integral_constant<int, 0>{}); break;
        case 1: last(std::integral_constant<int, 1>{}); break;
        case 2: last(std::integral_constant<int, 2>{}); break;
        case 3: last(std::integral_constant<int, 3>{}); break;
        case 4: last(std::integral_constant<int, 4>{}); break;
        case 5: last(std::integral_constant<int, 5>{}); break;
        default: last(std::integral_constant<int, 6>{}); break;
        }
    }
}

// Tiles at a time: scattered ones, the rest of a run.  One at a time for the former is ahead on runs of one tile (300 K, k = 28 4.7 / 4.1 us) and behind
// where pairs are marked (2^26, k = 63, every fourth tile 143 / 157); as a third form beside the two it spills.
constexpr int kPlainFew = 2, kPlainMany = 4;
constexpr int kOwnLds = kStage<kPlainMany> * 4 > 3 * kPlane ? kStage<kPlainMany> * 4 : 3 * kPlane;     // bytes of a wavefront

// The rest of a run is left to plain sums where its first two tiles both hold a marked value (one value marks two tiles but lies in one), or
// where three of four of the `seen` ones are marked: with half of them marked the split still pays (k = 63, a value in every fourth
// tile, given up at two of five: 20 M 48 / 57 us, 2^26 160 / 196).
__device__ __forceinline__ bool too_many(int marked, int seen) { return marked >= 4 && 4 * marked >= 3 * seen; }

template <int KS, bool NT>
__global__ __launch_bounds__(kBlock, 4) void conv1d_split_kernel(Taps1D taps, const float* __restrict__ x, float* __restrict__ y,
                                                                 long long n, long long m, int k, int run, unsigned tiny_below)
{
    (void)taps;
    kernarg_floats tw = (kernarg_floats)__builtin_amdgcn_kernarg_segment_ptr();

    constexpr int kPad = 15 + 32 * KS + 1;                                 // w(-15) .. w(32 KS - 1)
    __shared__ float tpad[kPad];
    __shared__ __attribute__((aligned(16))) u4 frags[KS * 3 * kWave];
    __shared__ __attribute__((aligned(16))) char planes[kWaves * kOwnLds];

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = wave_in_block();
    const long long base = ((long long)blockIdx.x * kWaves + wave) * run * kTileOut;       // first output of this wavefront
    const long long left = m - base;
    const int tiles = left <= 0 ? 0 : left >= (long long)run * kTileOut ? run : (int)((left + kTileOut - 1) / kTileOut);

    // Inputs of tile t, t = 0 .. tiles (and a few more that nothing uses): lanes past the last tap's reach repeat the last quad that is needed, and loads past the end of the
    // signal start at its last four numbers and are put right before the split.
    const float* xb = x + base;                                            // uniform
    const int last_quad = kTileOut * tiles + 32 * KS - 16 - kTile;
    const long long room = n - base - kTile;
    const int last_in = room < last_quad ? (int)room : last_quad;
    const bool tail = room < last_quad;                                    // uniform
    f4u raw[kAhead];
    auto load_tile = [&](int t, f4u& v) {
        const int at = min(kTileOut * t + kTile * lane, last_in);
        const f4u* p = reinterpret_cast<const f4u*>(reinterpret_cast<const char*>(xb) + (unsigned)at * 4u);
        v = NT ? __builtin_nontemporal_load(p) : *p;
    };
    if (tiles > 0) {
#pragma unroll
        for (int i = 0; i < kAhead; ++i) load_tile(i, raw[i]);
    }

    // A operands, once per workgroup
    for (int e = threadIdx.x; e < kPad; e += kBlock) tpad[e] = e >= 15 && e - 15 < k ? tw[kLeadIn + e - 15] : 0.0f;
    __syncthreads();
    const int i16 = lane & 15, kb = lane >> 4;                             // operand coordinates of the lane
    for (int s = wave; s < KS; s += kWaves) {
        const float* t = tpad + 32 * s + 8 * kb - i16 + 15;
        u4 p[3];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            unsigned a, b, c;
            split2(t[2 * i], t[2 * i + 1], a, b, c);
            p[0][i] = a; p[1][i] = b; p[2][i] = c;
        }
#pragma unroll
        for (int j = 0; j < 3; ++j) frags[(s * 3 + j) * kWave + lane] = p[j];
    }
    __syncthreads();
    if (tiles == 0) return;                                                // (the whole wavefront)
    b8 fa[KS][3];
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int j = 0; j < 3; ++j) fa[s][j] = __builtin_bit_cast(b8, frags[(s * 3 + j) * kWave + lane]);

    char* const mine = planes + wave * kOwnLds;
    int window[2][KS];                                                     // bytes of the lane's windows in the first plane
#pragma unroll
    for (int slot = 0; slot < 2; ++slot)
#pragma unroll
        for (int s = 0; s < KS; ++s) window[slot][s] = place((kTileOut * slot + 16 * i16 + 32 * s + 8 * kb) & (2 * kTileOut - 1));
    const int put_at = place(kTile * lane);

    // Tile t from registers to its slot; whether it holds a value the split does not carry.
    auto put = [&](int t, f4u v, int slot) -> bool {
        if (tail) {
            asm volatile("");                                              // a branch, not selects in every wavefront
            const int off = min(kTileOut * t + kTile * lane, last_quad) - (int)room;       // past the end reads as 0
            if (off > 0) {
                if (off & 1) v = f4u{v.y, v.z, v.w, 0.0f};
                if (off & 2) v = f4u{v.z, v.w, 0.0f, 0.0f};
                if (off > 3) v = f4u{0.0f, 0.0f, 0.0f, 0.0f};
            }
        }
        u2 p1, p2, p3;
        unsigned a, b, c;
        split2(v.x, v.y, a, b, c);
        p1.x = a; p2.x = b; p3.x = c;
        split2(v.z, v.w, a, b, c);
        p1.y = a; p2.y = b; p3.y = c;
        char* dst = mine + place(kTileOut * slot) + put_at;
        *reinterpret_cast<u2*>(dst) = p1;
        *reinterpret_cast<u2*>(dst + kPlane) = p2;
        *reinterpret_cast<u2*>(dst + 2 * kPlane) = p3;
        unsigned tiny = 0xffffffffu;
        float large = 0.0f;                                                // (NaN stays NaN)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float e = v[i];
            tiny = min(tiny, (__builtin_bit_cast(unsigned, e) << 1) - 1u); // +-0: the largest
            large = __builtin_elementwise_maximum(large, __builtin_fabsf(e));
        }
        return __builtin_amdgcn_ballot_w64((tiny < tiny_below) | !(large < kHuge)) != 0;
    };

    unsigned todo = 0;                                                     // tiles left to plain sums; a bit per tile of the run
    int end = tiles, rest = tiles;                                         // of the loop below; 0 and the first tile left once it is given up
    bool bad = put(0, raw[0], 0);
    load_tile(kAhead, raw[0]);
    bool bad_next = put(1, raw[1], 1);
    load_tile(kAhead + 1, raw[1]);
    wave_exchange();

    // Tile t in slot t mod 2; tile t+1 is in the other one, tile t+2 takes this slot once the windows of tile t are read.
    auto step = [&](int t, auto phase_tag) {
        constexpr int PHASE = decltype(phase_tag)::value, SLOT = PHASE & 1, NEXT = (PHASE + 2) % kAhead;
        const long long at = base + (long long)t * kTileOut;
        b8 b[KS][3];
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int j = 0; j < 3; ++j) b[s][j] = *reinterpret_cast<const b8*>(mine + window[SLOT][s] + j * kPlane);
        wave_exchange();
        const bool bad_after = put(t + 2, raw[NEXT], SLOT);
        load_tile(t + 2 + kAhead, raw[NEXT]);
        if (!(bad | bad_next)) {
            f4 lo = f4{0.0f, 0.0f, 0.0f, 0.0f}, hi = lo;
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[s][2], b[s][0], lo, 0, 0, 0);
                lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[s][0], b[s][2], lo, 0, 0, 0);
                lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[s][1], b[s][1], lo, 0, 0, 0);
                lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[s][1], b[s][0], lo, 0, 0, 0);
                lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[s][0], b[s][1], lo, 0, 0, 0);
                hi = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[s][0], b[s][0], hi, 0, 0, 0);
            }
            const f4 sum = hi + lo;
            const long long to = at + 16 * i16 + 4 * kb;
            if (at + kTileOut <= m) {                                      // uniform
                asm volatile("");
                __builtin_nontemporal_store(f4u{sum.x, sum.y, sum.z, sum.w}, reinterpret_cast<f4u*>(y + to));
            } else {
                const float out[4] = {sum.x, sum.y, sum.z, sum.w};
                store4_guarded(y, to, m, out);
            }
        } else {
            todo |= 1u << t;                                               // rare
            if (too_many(__builtin_popcount(todo), t + 1)) { rest = t + 1; end = 0; }
        }
        wave_exchange();
        bad = bad_next;
        bad_next = bad_after;
    };
    static_assert(kAhead == 4, "the steps below");
    if ((bad & bad_next) | ((bad | bad_next) & (tiles == 1))) {
        if (tiles > kPlainFew) rest = 0;
        else todo = (1u << tiles) - 1u;
        end = 0;
    }
#pragma nounroll
    for (int t = 0; t < end; t += kAhead) {
        step(t, std::integral_constant<int, 0>{});
        if (t + 1 >= end) break;
        step(t + 1, std::integral_constant<int, 1>{});
        if (t + 2 >= end) break;
        step(t + 2, std::integral_constant<int, 2>{});
        if (t + 3 >= end) break;
        step(t + 3, std::integral_constant<int, 3>{});
    }
    float* const stage = reinterpret_cast<float*>(mine);
    if (rest < tiles) {                                                    // uniform; the next tiles' loads in flight
        PlainInputs<kPlainMany> in;
        plain_load(x, n, base + (long long)rest * kTileOut, lane, in);
#pragma nounroll
        for (int t = rest; t < tiles; t += kPlainMany) {
            const long long at = base + (long long)t * kTileOut;
            plain_stage(in, lane, stage);
            if (t + kPlainMany < tiles) plain_load(x, n, at + kPlainMany * kTileOut, lane, in);
            float acc[kPlainMany][4];
            plain_sums(tw, k, lane, stage, acc);
#pragma unroll
            for (int r = 0; r < kPlainMany; ++r)
                if (t + r < tiles) store4_guarded(y, at + r * kTileOut + kTile * lane, m, acc[r]);
        }
    }
    while (todo != 0) {                                                    // uniform
        const int t = __builtin_ctz(todo);
        const long long at = base + (long long)t * kTileOut;
        PlainInputs<kPlainFew> in;
        plain_load(x, n, at, lane, in);
        plain_stage(in, lane, stage);
        float acc[kPlainFew][4];
        plain_sums(tw, k, lane, stage, acc);
#pragma unroll
        for (int r = 0; r < kPlainFew; ++r)
            if (r < 32 - t && (todo >> (t + r) & 1u)) store4_guarded(y, at + r * kTileOut + kTile * lane, m, acc[r]);
        todo &= t + kPlainFew < 32 ? ~0u << (t + kPlainFew) : 0u;
    }
}

// Wavefronts the device holds, four a SIMD, and the longest run of tiles of one (a bit each in todo).  Runs are as long as
// whole rounds of resident wavefronts allow: 40 M, k = 64, runs of 20 / 32 tiles 63 / 69 us; 2^26 of 32 / 16 / 8 95 / 101 / 108.  Up to 49 taps
// the set-up is shorter and from the second round on runs of eight are the better ones: 2^26 93 / 97 with 8 / 32, 40 M 58 / 59.
constexpr long long kPlaces = 4096;
constexpr int kLongestRun = 32;
// Up to here (with two and with three instructions a product) the loads are cacheable.  Inputs that the kernel before has written, or a few that a
// program goes round, are then found in the 256 MB memory-side cache; where that is full of what else was written, the loads wait for it to be
// written back.  The lines lie where even then the call takes no longer than the vector kernel's (us, vector kernel / cacheable / non-temporal; in
// turn behind the kernel that wrote the input, and behind others that wrote 1 GB; k = 50: 14 M 34.7 / 20.6 / 21.9, 37.3 / 33.5 / 25.8; 24 M 54.5 / 35.7 / 37.1,
// 56.5 / 56.9 / 41.7; 34 M 71.6 / 46.2 / 49.2, 75.5 / 77.2 / 56.6; k = 36: 8 M 18.6 / 12.4 / 14.8, 20.2 / 18.0 / 18.5; 14 M 28.3 / 19.2 / 20.9, 31.3 / 32.6 / 27.1;
// 20 M 38.8 / 26.4 / 30.2, 41.7 / 46.7 / 36.5).  Three 20 M inputs in turn, k = 63: 28 / 34.
constexpr size_t kCached2 = 8u << 20, kCached3 = 24u << 20;

template <int KS, bool NT>
hipError_t launch_split(const float* x, size_t n, const float* w, int k, float* y, hipStream_t s)
{
    Taps1D taps;
    for (int q = 0; q < kTaps1DLen; ++q) taps.w[q] = q >= kLeadIn && q - kLeadIn < k ? w[q - kLeadIn] : 0.0f;
    const long long m = (long long)n - k + 1;
    const long long tiles = (m + kTileOut - 1) / kTileOut;
    const long long rounds = (tiles + kPlaces * kLongestRun - 1) / (kPlaces * kLongestRun);
    int run = (int)((tiles + kPlaces * rounds - 1) / (kPlaces * rounds));
    if (KS == 2 && rounds > 1) run = 8;
    const long long waves = (tiles + run - 1) / run;
    const long long blocks = (waves + kWaves - 1) / kWaves;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((conv1d_split_kernel<KS, NT>), dim3((unsigned)blocks), dim3(kBlock), 0, s, taps, x, y, (long long)n, m, k, run,
                       split_tiny_limit(w, k));
    return hipGetLastError();
}

template <int KS>
hipError_t launch_cached(const float* x, size_t n, const float* w, int k, float* y, hipStream_t s)
{
    return n <= (KS == 2 ? kCached2 : kCached3) ? launch_split<KS, false>(x, n, w, k, y, s) : launch_split<KS, true>(x, n, w, k, y, s);
}

}  // namespace

bool conv1d_split_takes(const float* w, int k) { return k >= 28 && k <= kMaxK1D && split_takes_taps(w, k); }

// Where it is the fastest kernel (us, best vector kernel / this): from 34 taps on, at every size (k = 36: 1 M 7.6 / 4.7, 8 M 19.1 / 16.9, 20 M 40.8 / 35.7, 2^26 113 / 93,
// 2^29 809 / 758; k = 64 2^30 2309 / 1535, k = 40 2^31 3405 / 3085).  From 28 to 33 taps on short signals and long ones (k = 28: 300 K 4.2 / 3.5, 2 M 6.8 / 5.9,
// 36 M 57.6 / 51.6, 2^26 100 / 93, 2^27 187 / 181, 2^29 778 / 751, 2^30 1567 / 1524); between them FBS is level or ahead (k = 28: 8 M 16.4 / 16.5, 14 M 24.1 / 25.3, 20 M
// 31.8 / 34.7, 30 M 45.6 / 48.8; k = 32: 34.3 / 34.8 on 20 M).  Shorter filters sit on the copy rate with FBS from a few million inputs on
// (k = 24: 4.3 / 4.2 on 300 K, 20.6 / 21.1 on 12 M).
bool conv1d_split_pays(size_t n, int k)
{
    return k >= 34 || (k >= 28 && (n <= (4u << 20) || n >= (36u << 20)));
}

hipError_t launch_conv1d_split(const float* x, size_t n, const float* w, int k, float* y, hipStream_t s)
{
    return k <= 49 ? launch_cached<2>(x, n, w, k, y, s) : launch_cached<3>(x, n, w, k, y, s);
}

}  // namespace sysconv
