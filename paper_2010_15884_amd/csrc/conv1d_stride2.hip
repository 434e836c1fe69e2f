// 1-D valid convolution with stride 2,  y[c] = sum_q x[2c+q] * w[q],  as the FBS
// design of the paper's Table 2, row 3 right: PE = c, time = q, partial sums and
// weights stay, and an input is handed one PE down every TWO steps,
// X(c,q) = X(c+1,q-2).  (The table prints x(c+q) as the loaded element; only
// x(2c+q) agrees with that hand-over, so that is what is computed.)
//
// The hand-over rule splits the inputs of a PE into two chains that never mix: the
// even taps see x(2c), x(2c+2), ... and the odd taps x(2c+1), x(2c+3), ...  Each is an
// ordinary stride-1 FBS array over the de-interleaved signal, E(c) = x(2c) resp.
// O(c) = x(2c+1), both adding into the same partial sums.  A lane gets eight
// consecutive inputs, which are E and O of its four PEs, and the two
// chains then run the stride-1 time steps with the even resp. the odd taps.  The
// chains are independent, so they are issued one after the other (all even steps,
// then all odd steps) rather than alternating.
#include "launch.h"
#include "systolic.h"

#include <utility>

namespace sysconv {
namespace {

typedef const float __attribute__((address_space(4)))* kernarg_floats;

constexpr int kGroups = 4;                      // register groups per wavefront
constexpr int kChainLen = kMaxK1D / 2 + 8;      // taps of one chain, zero-padded so a block of four can always be read
struct TapsStride2 { float even[kChainLen]; float odd[kChainLen]; };

template <int NT, bool MORE>
__device__ __forceinline__ void chain_groups(float (&e)[kGroups][4], float (&acc)[kGroups][4], const float (&w)[4])
{
#pragma unroll
    for (int r = 0; r < kGroups; ++r) fbs_steps<NT, MORE>(e[r], acc[r], w);
}

// All kc >= 1 time steps of one chain (KC > 0: count known at compile time).
template <int KC>
__device__ __forceinline__ void run_chain(float (&e)[kGroups][4], float (&acc)[kGroups][4], kernarg_floats w, int kc_rt)
{
    const int kc = KC ? KC : kc_rt;
    int j = 0;
    if (KC) {
#pragma unroll
        for (; j + 4 < kc; j += 4) {
            const float wb[4] = {w[j], w[j + 1], w[j + 2], w[j + 3]};
            chain_groups<4, true>(e, acc, wb);
        }
    } else {
#pragma nounroll
        for (; j + 4 < kc; j += 4) {
            const float wb[4] = {w[j], w[j + 1], w[j + 2], w[j + 3]};
            chain_groups<4, true>(e, acc, wb);
        }
    }
    const float wb[4] = {w[j], w[j + 1], w[j + 2], w[j + 3]};
    switch (kc - j) {                           // uniform across the wavefront
    case 4: chain_groups<4, false>(e, acc, wb); break;
    case 3: chain_groups<3, false>(e, acc, wb); break;
    case 2: chain_groups<2, false>(e, acc, wb); break;
    default: chain_groups<1, false>(e, acc, wb); break;
    }
}

// The taps are the first kernel argument (offset 0 of the kernel-argument segment).  STREAM: the signal is read with the
// non-temporal hint.
template <int KT, bool STREAM>
__global__ __launch_bounds__(kBlock) void conv1d_fbs_stride2_kernel(TapsStride2 taps, const float* __restrict__ x,
                                                                    float* __restrict__ y, long long n, long long m,
                                                                    int k_rt, int valid_lanes)
{
    (void)taps;
    kernarg_floats tw = (kernarg_floats)__builtin_amdgcn_kernarg_segment_ptr();
    const int k = KT ? KT : k_rt;
    const int lane = threadIdx.x & (kWave - 1);
    const long long per_group = (long long)kTile * valid_lanes;            // outputs a group yields
    const long long wave = (long long)blockIdx.x * (kBlock / kWave) + wave_in_block();
    const long long base = wave * kGroups * per_group;                     // first output of the wavefront
    if (base >= m) return;                                                 // uniform per wavefront

    // A group's 512 inputs come in as two loads of 1 KB; a round trip through LDS, private to the wavefront, then gives
    // each lane the eight consecutive inputs of its four PEs.  (Loaded straight by the lanes that need them, every cache
    // line was asked for by two instructions and the non-temporal hint could not be used: 2^26 inputs, k = 2 72 -> 62 us,
    // 16 75 -> 64, 31 82 -> 65; a copy of the same bytes takes 65 us.  From k = 50 on the vector ALUs bound both.)
    __shared__ __attribute__((aligned(16))) float stage[kBlock / kWave][kGroups * 2 * kWave * kTile];
    float* const lds = stage[wave_in_block()];
    float ev[kGroups][4], od[kGroups][4], acc[kGroups][4];
#pragma unroll
    for (int r = 0; r < kGroups; ++r) {
        const long long c0 = 2 * (base + r * per_group) + kTile * lane;
        load4_guarded<STREAM>(x, c0, n, ev[r]);
        load4_guarded<STREAM>(x, c0 + kWave * kTile, n, od[r]);
    }
#pragma unroll
    for (int r = 0; r < kGroups; ++r) {
        float* row = lds + r * 2 * kWave * kTile + kTile * lane;
        *reinterpret_cast<f4*>(row) = f4{ev[r][0], ev[r][1], ev[r][2], ev[r][3]};
        *reinterpret_cast<f4*>(row + kWave * kTile) = f4{od[r][0], od[r][1], od[r][2], od[r][3]};
    }
    wave_exchange();
#pragma unroll
    for (int r = 0; r < kGroups; ++r) {
        const float* own = lds + r * 2 * kWave * kTile + 2 * kTile * lane;
        const f4 lo = *reinterpret_cast<const f4*>(own), hi = *reinterpret_cast<const f4*>(own + 4);
        ev[r][0] = lo.x; od[r][0] = lo.y; ev[r][1] = lo.z; od[r][1] = lo.w;
        ev[r][2] = hi.x; od[r][2] = hi.y; ev[r][3] = hi.z; od[r][3] = hi.w;
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[r][i] = 0.0f;
    }

    run_chain<(KT + 1) / 2>(ev, acc, tw, (k + 1) / 2);                     // q = 0, 2, 4, ...
    if (k > 1) run_chain<KT / 2>(od, acc, tw + kChainLen, k / 2);          // q = 1, 3, 5, ...

    if (lane < valid_lanes) {
#pragma unroll
        for (int r = 0; r < kGroups; ++r)
            store4_guarded(y, base + r * per_group + kTile * lane, m, acc[r]);
    }
}

template <int KT>
hipError_t launch_stride2(const float* x, size_t n, const float* w, int k, float* y, hipStream_t s)
{
    TapsStride2 taps;
    for (int j = 0; j < kChainLen; ++j) {
        taps.even[j] = 2 * j < k ? w[2 * j] : 0.0f;
        taps.odd[j] = 2 * j + 1 < k ? w[2 * j + 1] : 0.0f;
    }
    const long long m = ((long long)n - k) / 2 + 1;
    // The longer (even) chain reaches (k+1)/2 - 1 PEs up: that many PEs at the top of a
    // group compute values that are never stored.  Whole lanes, and a multiple of four
    // of them, so that every group starts on a 64-byte boundary of x and of y.
    const int v = kWave - halo_lanes((k + 1) / 2);
    const int valid_lanes = v - v % 4;
    const long long per_wave = (long long)kGroups * kTile * valid_lanes;
    const long long waves = (m + per_wave - 1) / per_wave;
    const long long blocks = (waves + (kBlock / kWave) - 1) / (kBlock / kWave);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    // Signals of 14 to 44 MB are read without the non-temporal hint: several of them, as a program goes round its buffers,
    // stay in the 256 MB memory-side cache (us, with / without: k = 5 4 M inputs 5.9 / 5.7, 6 M 8.0 / 7.1, 9 M 11.3 / 10.2; k = 11
    // 6 M 8.1 / 6.9; shorter 2 M 4.0 / 4.2, longer 12 M 13.9 / 14.5, 40 M 38.6 / 41.5).  With long filters it makes no difference
    // (50: 7 M 13.6 / 14.1, 8 M 16.2 / 16.2).  (A choice inside the kernel made every group wait for its own loads: 2^26 inputs,
    // k = 28 65 -> 76 us.)
    const bool cacheable = KT > 0 && n > 3500000 && n < 11000000;
    const auto kernel = cacheable ? conv1d_fbs_stride2_kernel<KT, KT == 0> : conv1d_fbs_stride2_kernel<KT, true>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kBlock), 0, s, taps, x, y, (long long)n, m, k, valid_lanes);
    return hipGetLastError();
}

// Tap counts known at compile time up to 34: on short signals the loop's counters and its waits for taps show (us, loop /
// unrolled: 70 K inputs k = 2 3.4 / 3.1, 16 3.8 / 3.4, 20 4.0 / 3.5, 34 4.8 / 4.0; 3 M 8 5.1 / 4.8, 20 6.1 / 5.6, 32 7.1 / 6.4), and from
// about 8 M inputs on both are at the copy rate (2^26: 2 62 / 62, 20 64 / 65, 34 66 / 65).  With 35 taps and more the unrolled
// code leaves the instruction cache on long signals (2^26: 35 68 / 77, 48 78 / 92, 64 99 / 160), though it still gains on
// short ones (70 K: 64 6.6 / 5.4).
constexpr int kUnrolled = 34;
typedef hipError_t (*Launch)(const float*, size_t, const float*, int, float*, hipStream_t);
template <int... K>
hipError_t launch_by_k(std::integer_sequence<int, K...>, const float* x, size_t n, const float* w, int k, float* y,
                       hipStream_t s)
{
    static constexpr Launch table[] = {launch_stride2<K>...};              // [0]: the loop
    return table[k <= kUnrolled ? k : 0](x, n, w, k, y, s);
}

}  // namespace

hipError_t launch_conv1d_fbs_stride2(const float* x, size_t n, const float* w, int k, float* y, hipStream_t s)
{
    return launch_by_k(std::make_integer_sequence<int, kUnrolled + 1>{}, x, n, w, k, y, s);
}

}  // namespace sysconv
