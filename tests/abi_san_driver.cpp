// Host-side checks of libsysconv for a build with -fsanitize=address,undefined (host code only): every
// argument check of the C ABI and the space-time-transform planner (the validity conditions of the paper's
// Section 2.2 and the launch plan derived from a design), driven with designs and sizes from the edges of
// what they accept.  Nothing here reaches a HIP call: every request is either answered by a query function
// or refused by the validation that precedes the launch, so the program runs on a host without a GPU.
// The "device" pointers are made-up addresses that validation must never dereference.
#include <limits.h>
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <vector>

#define SYSCONV_NO_HIP_HEADER
#include "sysconv.h"

// The library's own rules for the kernels behind AUTO (host code without a HIP call).
namespace sysconv {
bool conv2d_split_takes(int h, int w, size_t yp, const float* f, int kh, int kw);
bool conv2d_split_pays(int oh, int ow, int kh, int kw);
bool conv2d_stride2_takes_strips(int w, int oh, int ow, int kh, int kw);
int conv2d_stride2_strip_rows(int w, int oh, int kh, int kw);
int conv2d_stride2_pair_rows(int oh, int ow, int kh, int kw);
bool conv1d_split_pays(size_t n, int k);
int conv2d_vector_projection(int oh, int ow, size_t x_pitch, int kh, int kw);
}

static int failures = 0;
#define EXPECT(expr, want) do { const int got_ = (expr); if (got_ != (want)) { \
    fprintf(stderr, "line %d: %s = %d (%s), expected %d\n", __LINE__, #expr, got_, sys_status_string(got_), (int)(want)); \
    ++failures; } } while (0)

static sys_stt_design_t design(int p0, int p1, int s0, int s1, int xon, int ex0, int ex1, int won, int ew0, int ew1,
                               int ez0, int ez1)
{
    sys_stt_design_t d;
    memset(&d, 0, sizeof d);
    d.alloc[0] = p0; d.alloc[1] = p1; d.sched[0] = s0; d.sched[1] = s1;
    d.x_passed = xon; d.dep_x[0] = ex0; d.dep_x[1] = ex1;
    d.w_passed = won; d.dep_w[0] = ew0; d.dep_w[1] = ew1;
    d.dep_z[0] = ez0; d.dep_z[1] = ez1;
    return d;
}

int main()
{
    float* const X = (float*)0x10000000;
    float* const Y = (float*)0x40000000;
    std::vector<float> taps(256, 1.0f);                            // exactly as many as the largest filter reads

    // ---- the six designs of Table 2 and five others: valid for every tap count the planner accepts
    const sys_stt_design_t valid[] = {
        design(1, 1, 0, 1, 1, -1, 1, 0, 0, 0, 0, 1),               // SBM
        design(0, 1, 1, 1, 0, 0, 0, 1, 1, 0, 0, 1),                // BSM
        design(0, 1, 1, -1, 1, 1, -1, 1, 1, 0, 0, -1),             // FSM
        design(1, 0, 1, 1, 0, 0, 0, 1, 1, 0, 0, 1),                // BFS
        design(1, 0, 2, 1, 1, 1, -1, 1, 1, 0, 0, 1),               // FFS
        design(1, 0, 0, 1, 1, -1, 1, 0, 0, 0, 0, 1),               // FBS
        design(1, 0, 1, 1, 0, 0, 0, 0, 0, 0, 0, 1),                // everything loaded, sums stay
        design(1, 1, 1, 2, 1, -1, 1, 0, 0, 0, 0, 1),               // SBM at half speed
        design(-1, 0, 0, 1, 1, -1, 1, 0, 0, 0, 0, 1),              // FBS, PE index against c
        design(0, -1, 1, -1, 1, 1, -1, 1, 1, 0, 0, -1),            // FSM mirrored
        design(1, 0, 0, -1, 1, 1, -1, 0, 0, 0, 0, -1),             // FBS, taps descending
    };
    for (const sys_stt_design_t& d : valid)
        for (int k = 1; k <= SYS_MAX_K1D; ++k) {
            const int st = sys_stt_check(&d, k);
            if (st != SYS_OK && st != SYS_ERR_UNSUPPORTED) {       // long filters may not fit 64 lanes: unsupported, never invalid
                fprintf(stderr, "valid design refused as %s at k=%d\n", sys_status_string(st), k);
                ++failures;
            }
        }
    EXPECT(sys_stt_check(&valid[0], 5), SYS_OK);
    EXPECT(sys_stt_check(&valid[5], 16), SYS_OK);

    // ---- designs Section 2.2 rules out
    const sys_stt_design_t invalid[] = {
        design(1, 1, 1, 1, 0, 0, 0, 0, 0, 0, 0, 1),                // singular
        design(1, 0, 1, 0, 0, 0, 0, 0, 0, 0, 0, 1),                // sums read before they exist
        design(1, 1, 0, -1, 1, -1, 1, 0, 0, 0, 0, 1),              // SBM run backwards
        design(1, 0, 0, 1, 1, 1, -1, 0, 0, 0, 0, 1),               // FBS whose inputs come from the future (s.e = -1)
        design(1, 0, 0, 1, 0, 0, 0, 1, 1, 0, 0, 1),                // weights passed within one step
        design(1, 0, 0, 1, 1, -1, 2, 0, 0, 0, 0, 1),               // X dependence changes the input
        design(1, 0, 0, 1, 1, 0, 0, 0, 0, 0, 0, 1),                // null X dependence
        design(1, 0, 1, 1, 0, 0, 0, 1, 1, 1, 0, 1),                // W dependence changes the tap
        design(1, 0, 1, 1, 0, 0, 0, 0, 0, 0, 1, 1),                // Z dependence across outputs
        design(1, 0, 0, 1, 0, 0, 0, 0, 0, 0, 0, 2),                // Z dependence skips taps
    };
    for (const sys_stt_design_t& d : invalid)
        for (int k : {1, 2, 5, 64}) EXPECT(sys_stt_check(&d, k), SYS_ERR_DESIGN);
    // ---- valid, but beyond the kernel
    const sys_stt_design_t too_large[] = {
        design(1, 0, 1, 2, 0, 0, 0, 0, 0, 0, 0, 1),                // |det| = 2
        design(1, 3, 0, 1, 1, -1, 1, 0, 0, 0, 0, 1),               // values jump over PEs
        design(1, 0, 4, 1, 0, 0, 0, 1, 1, 0, 0, 1),                // weights travel four steps
        design(65, 1, 64, 1, 0, 0, 0, 0, 0, 0, 0, 1),              // coefficient beyond +-64
        design(INT_MAX, 1, INT_MIN, 1, 0, 0, 0, 0, 0, 0, 0, 1),    // arithmetic on these must not overflow
        design(INT_MIN, INT_MIN, INT_MAX, INT_MAX, 1, INT_MAX, INT_MIN, 1, INT_MIN, 0, 0, 1),
    };
    for (const sys_stt_design_t& d : too_large)
        for (int k : {1, 5, 64}) {
            const int st = sys_stt_check(&d, k);
            if (st != SYS_ERR_UNSUPPORTED && st != SYS_ERR_DESIGN) {
                fprintf(stderr, "oversized design accepted (%s)\n", sys_status_string(st));
                ++failures;
            }
        }
    EXPECT(sys_stt_check(nullptr, 5), SYS_ERR_NULL);
    EXPECT(sys_stt_check(&valid[0], 0), SYS_ERR_SIZE);
    EXPECT(sys_stt_check(&valid[0], SYS_MAX_K1D + 1), SYS_ERR_SIZE);
    EXPECT(sys_conv1d_stt(X, 100, taps.data(), 5, Y, &invalid[0], nullptr), SYS_ERR_DESIGN);
    EXPECT(sys_conv1d_stt(X, 100, taps.data(), 5, X + 10, &valid[0], nullptr), SYS_ERR_ALIAS);
    EXPECT(sys_conv1d_stt(X, 100, taps.data(), 5, Y, nullptr, nullptr), SYS_ERR_NULL);

    // ---- argument validation of the convolutions: refused before any launch
    EXPECT(sys_conv1d(nullptr, 100, taps.data(), 5, Y, SYS_PROJ_FBS, nullptr), SYS_ERR_NULL);
    EXPECT(sys_conv1d(X, 100, taps.data(), 0, Y, SYS_PROJ_FBS, nullptr), SYS_ERR_SIZE);
    EXPECT(sys_conv1d(X, 4, taps.data(), 5, Y, SYS_PROJ_FBS, nullptr), SYS_ERR_SIZE);
    EXPECT(sys_conv1d(X, 100, taps.data(), 65, Y, SYS_PROJ_FBS, nullptr), SYS_ERR_UNSUPPORTED);
    EXPECT(sys_conv1d(X, 100, taps.data(), 5, Y, SYS_PROJ_MFMA, nullptr), SYS_ERR_UNSUPPORTED);
    EXPECT(sys_conv1d(X, 100, taps.data(), 5, Y, 99, nullptr), SYS_ERR_UNSUPPORTED);
    EXPECT(sys_conv1d((float*)((char*)X + 2), 100, taps.data(), 5, Y, SYS_PROJ_FBS, nullptr), SYS_ERR_UNSUPPORTED);
    EXPECT(sys_conv1d(X, (size_t)1 << 41, taps.data(), 5, Y, SYS_PROJ_FBS, nullptr), SYS_ERR_UNSUPPORTED);
    EXPECT(sys_conv1d(X, 100, taps.data(), 5, X + 99, SYS_PROJ_FBS, nullptr), SYS_ERR_ALIAS);
    EXPECT(sys_conv1d(X, SIZE_MAX / 8, taps.data(), 5, Y, SYS_PROJ_FBS, nullptr), SYS_ERR_UNSUPPORTED);
    EXPECT(sys_conv1d_strided(X, 100, taps.data(), 5, 0, Y, SYS_PROJ_FBS, nullptr), SYS_ERR_SIZE);
    EXPECT(sys_conv1d_strided(X, 100, taps.data(), 5, 3, Y, SYS_PROJ_FBS, nullptr), SYS_ERR_UNSUPPORTED);
    EXPECT(sys_conv1d_strided(X, 100, taps.data(), 5, 2, X + 10, SYS_PROJ_FBS, nullptr), SYS_ERR_ALIAS);
    EXPECT(sys_conv1d_strided(X, 100, taps.data(), 5, INT_MAX, Y, SYS_PROJ_SBM, nullptr), SYS_ERR_UNSUPPORTED);

    EXPECT(sys_conv2d(X, 10, 10, 10, nullptr, 3, 3, Y, 8, SYS_PROJ_FBS, nullptr), SYS_ERR_NULL);
    EXPECT(sys_conv2d(X, 10, 10, 9, taps.data(), 3, 3, Y, 8, SYS_PROJ_FBS, nullptr), SYS_ERR_SIZE);
    EXPECT(sys_conv2d(X, 10, 10, 10, taps.data(), 3, 3, Y, 7, SYS_PROJ_FBS, nullptr), SYS_ERR_SIZE);
    EXPECT(sys_conv2d(X, 10, 10, 10, taps.data(), 11, 3, Y, 8, SYS_PROJ_FBS, nullptr), SYS_ERR_SIZE);
    EXPECT(sys_conv2d(X, 100, 100, 100, taps.data(), 16, 3, Y, 98, SYS_PROJ_FBS, nullptr), SYS_ERR_UNSUPPORTED);
    EXPECT(sys_conv2d(X, 100, 100, 100, taps.data(), 4, 3, Y, 98, SYS_PROJ_BFS, nullptr), SYS_ERR_UNSUPPORTED);
    EXPECT(sys_conv2d(X, 100, 100, 100, taps.data(), 14, 3, Y, 98, SYS_PROJ_MFMA, nullptr), SYS_ERR_UNSUPPORTED);
    EXPECT(sys_conv2d(X, 100, 100, 100, taps.data(), 3, 3, X + 5000, 98, SYS_PROJ_FBS, nullptr), SYS_ERR_ALIAS);
    EXPECT(sys_conv2d(X, 100, 100, (size_t)1 << 32, taps.data(), 3, 3, Y, 98, SYS_PROJ_FBS, nullptr), SYS_ERR_UNSUPPORTED);
    EXPECT(sys_conv2d(X, 1, INT_MAX, (size_t)INT_MAX, taps.data(), 1, 1, (float*)0x7000000000, (size_t)INT_MAX,
                      SYS_PROJ_AUTO, nullptr), SYS_ERR_UNSUPPORTED);
    EXPECT(sys_conv2d(X, INT_MAX, 1, 1, taps.data(), 15, 1, X + 4, 1, SYS_PROJ_AUTO, nullptr), SYS_ERR_ALIAS);
    EXPECT(sys_conv2d_strided(X, 100, 100, 100, taps.data(), 3, 3, 0, Y, 98, SYS_PROJ_FBS, nullptr), SYS_ERR_SIZE);
    EXPECT(sys_conv2d_strided(X, 100, 100, 100, taps.data(), 3, 3, 3, Y, 98, SYS_PROJ_FBS, nullptr), SYS_ERR_UNSUPPORTED);
    EXPECT(sys_conv2d_strided(X, 100, 100, 100, taps.data(), 15, 15, 2, X + 5000, 49, SYS_PROJ_FBS, nullptr), SYS_ERR_ALIAS);

    // ---- the matrix-core projection derives a scale from the taps on the host: every tap is read, none beyond
    for (int kh = 1; kh <= 13; ++kh)
        for (int kw = 1; kw <= 13; ++kw) {
            std::vector<float> f((size_t)kh * kw, 0.0f);           // exactly kh * kw floats on the heap
            EXPECT(sys_conv2d(X, 100, 100, 100, f.data(), kh, kw, X + 5000, 100 - kw + 1, SYS_PROJ_MFMA, nullptr), SYS_ERR_ALIAS);
            f.back() = 1e-33f;
            EXPECT(sys_conv2d(X, 100, 100, 100, f.data(), kh, kw, X + 5000, 100 - kw + 1, SYS_PROJ_MFMA, nullptr), SYS_ERR_UNSUPPORTED);
            f.back() = INFINITY; f.front() = kh * kw > 1 ? 3e33f : INFINITY;
            EXPECT(sys_conv2d(X, 100, 100, 100, f.data(), kh, kw, X + 5000, 100 - kw + 1, SYS_PROJ_MFMA, nullptr),
                   kh * kw > 1 ? SYS_ERR_UNSUPPORTED : SYS_ERR_ALIAS);
            f.front() = NAN; f.back() = -0.5f;
            EXPECT(sys_conv2d(X, 100, 100, 100, f.data(), kh, kw, X + 5000, 100 - kw + 1, SYS_PROJ_MFMA, nullptr), SYS_ERR_ALIAS);
        }

    // ---- images the split kernel takes: output pitches up to 2^25, heights whose row numbers (up to three chunks of
    //      16 rows past the last output row) stay in an int, and every filter that its rule sends to it
    EXPECT(sysconv::conv2d_split_takes(INT_MAX, 5, 1, taps.data(), 13, 5), 0);
    EXPECT(sysconv::conv2d_split_takes(INT_MAX - 63, 5, 1, taps.data(), 13, 5), 0);
    EXPECT(sysconv::conv2d_split_takes(INT_MAX - 64, 5, 1, taps.data(), 13, 5), 1);
    EXPECT(sysconv::conv2d_split_takes(100, 4, 1, taps.data(), 13, 4), 0);
    EXPECT(sysconv::conv2d_split_takes(100, 10, 1, taps.data(), 14, 10), 0);
    EXPECT(sysconv::conv2d_split_takes(100, 100, (size_t)1 << 25, taps.data(), 15, 15), 1);
    EXPECT(sysconv::conv2d_split_takes(100, 100, ((size_t)1 << 25) + 1, taps.data(), 15, 15), 0);
    for (int kh = 1; kh <= SYS_MAX_K2D; ++kh)                      // every tap is read, none beyond
        for (int kw = 1; kw <= SYS_MAX_K2D; ++kw) {
            bool pays = false;
            for (int oh : {1, 15, 16, 1000, 30000, INT_MAX})
                for (int ow : {1, 240, 241, 1000, 30000, INT_MAX}) pays = pays || sysconv::conv2d_split_pays(oh, ow, kh, kw);
            std::vector<float> f((size_t)kh * kw, 0.0f);
            if (!pays && !sysconv::conv2d_split_takes(100, 100, 100, f.data(), kh, kw)) continue;
            EXPECT(sysconv::conv2d_split_takes(100, 100, 100, f.data(), kh, kw), 1);
            for (float in : {0x1p-60f, -0x1p-60f, 0x1p40f, -0x1p40f, -0.0f}) {
                f.back() = in;
                EXPECT(sysconv::conv2d_split_takes(100, 100, 100, f.data(), kh, kw), 1);
            }
            for (float out : {0x1.fffffep-61f, 0x1.000002p40f, INFINITY, -INFINITY, NAN, 1e-45f}) {
                f.back() = out;
                EXPECT(sysconv::conv2d_split_takes(100, 100, 100, f.data(), kh, kw), 0);
            }
        }

    // ---- shapes on either side of the rule's line, both kernels timed there
    EXPECT(sysconv::conv2d_split_pays(8182, 8182, 11, 11), 1);
    EXPECT(sysconv::conv2d_split_pays(286, 386, 15, 15), 1);
    EXPECT(sysconv::conv2d_split_pays(4084, 4092, 13, 5), 1);
    EXPECT(sysconv::conv2d_split_pays(8237, 244, 13, 5), 0);       // a second strip for four columns
    EXPECT(sysconv::conv2d_split_pays(929, 2371, 13, 5), 0);
    EXPECT(sysconv::conv2d_split_pays(8, 200000, 11, 11), 0);      // half of every chunk is padding
    EXPECT(sysconv::conv2d_split_pays(1275, 1606, 3, 12), 0);
    EXPECT(sysconv::conv2d_split_pays(866, 4759, 3, 12), 0);       // three rows: half of the units are empty
    EXPECT(sysconv::conv2d_split_pays(4673, 1074, 3, 13), 1);
    EXPECT(sysconv::conv2d_split_pays(2828, 989, 9, 9), 1);
    EXPECT(sysconv::conv2d_split_pays(3857, 380, 11, 11), 1);
    EXPECT(sysconv::conv2d_split_pays(2039, 2039, 10, 10), 1);

    // ---- AUTO without the split kernel, both sides of every line
    for (int k = 2; k <= 6; ++k)
        for (int oh : {1, 300, 2000, 100000}) {
            for (size_t pitch : {(size_t)16, (size_t)1024, (size_t)2048, (size_t)4096})
                EXPECT(sysconv::conv2d_vector_projection(oh, 10, pitch, k, k), SYS_PROJ_BFS);
            for (size_t pitch : {(size_t)15, (size_t)1000, (size_t)4095, (size_t)4100, (size_t)8192, (size_t)1 << 20})
                EXPECT(sysconv::conv2d_vector_projection(oh, 10, pitch, k, k), SYS_PROJ_FBS);
        }
    EXPECT(sysconv::conv2d_vector_projection(900, 1000, 1024, 7, 7), SYS_PROJ_FBS);        // 7x7: 0.9 M outputs
    EXPECT(sysconv::conv2d_vector_projection(901, 1000, 1024, 7, 7), SYS_PROJ_BFS);
    EXPECT(sysconv::conv2d_vector_projection(901, 1000, 1008, 7, 7), SYS_PROJ_FBS);
    EXPECT(sysconv::conv2d_vector_projection(30000, 1000, 1024, 7, 7), SYS_PROJ_BFS);
    EXPECT(sysconv::conv2d_vector_projection(8000, 2000, 2048, 7, 7), SYS_PROJ_BFS);       // 8 KB rows: 16 M
    EXPECT(sysconv::conv2d_vector_projection(8001, 2000, 2048, 7, 7), SYS_PROJ_SBM);
    EXPECT(sysconv::conv2d_vector_projection(750, 4000, 4096, 7, 7), SYS_PROJ_FBS);        // 3 M
    EXPECT(sysconv::conv2d_vector_projection(751, 4000, 4096, 7, 7), SYS_PROJ_SBM);
    EXPECT(sysconv::conv2d_vector_projection(3000, 1000, 1007, 7, 7), SYS_PROJ_FBS);
    EXPECT(sysconv::conv2d_vector_projection(3001, 1000, 1007, 7, 7), SYS_PROJ_SBM);
    for (int k = 8; k <= 11; ++k)
        for (size_t pitch : {(size_t)1024, (size_t)1000}) EXPECT(sysconv::conv2d_vector_projection(500, 900, pitch, k, k), SYS_PROJ_SBM);
    for (int kh = 1; kh <= SYS_MAX_K2D; ++kh)
        for (int kw = 1; kw <= SYS_MAX_K2D; ++kw) {
            if (kh == kw && kh >= 2 && kh <= 11) continue;
            EXPECT(sysconv::conv2d_vector_projection(500, 900, 1024, kh, kw), SYS_PROJ_FBS);
        }

    // ---- long 1-D filters: the split kernel from 34 taps on, and from 28 on below 4 Mi and above 36 Mi inputs
    for (size_t n : {(size_t)64, (size_t)4 << 20, ((size_t)4 << 20) + 1, (size_t)20000000, ((size_t)36 << 20) - 1, (size_t)36 << 20, (size_t)1 << 40}) {
        const bool ends = n <= (size_t)4 << 20 || n >= (size_t)36 << 20;
        EXPECT(sysconv::conv1d_split_pays(n, 27), 0);
        EXPECT(sysconv::conv1d_split_pays(n, 28), ends);
        EXPECT(sysconv::conv1d_split_pays(n, 33), ends);
        EXPECT(sysconv::conv1d_split_pays(n, 34), 1);
        EXPECT(sysconv::conv1d_split_pays(n, SYS_MAX_K1D), 1);
    }

    // ---- stride 2: strips of four outputs a lane, output rows of a wavefront, on both sides of every line
    for (int kw = 1; kw <= SYS_MAX_K2D; ++kw) {
        EXPECT(sysconv::conv2d_stride2_takes_strips(4000, 4000, 4000, 1, kw), 1);      // single rows
        EXPECT(sysconv::conv2d_stride2_strip_rows(4000, 4000, 1, kw), 1);
        EXPECT(sysconv::conv2d_stride2_takes_strips(4000, 1000, 1000, 2, kw), 0);
        EXPECT(sysconv::conv2d_stride2_takes_strips(30000, 30000, 10000, 2, kw), kw == 2);   // two columns on large images
    }
    EXPECT(sysconv::conv2d_stride2_strip_rows(30000, 30000, 2, 2), 3);
    EXPECT(sysconv::conv2d_stride2_takes_strips(3, 100, 1, 9, 3), 1);      // narrow images
    EXPECT(sysconv::conv2d_stride2_takes_strips(4, 100, 1, 9, 3), 0);
    EXPECT(sysconv::conv2d_stride2_strip_rows(3, 3000, 13, 3), 1);         // up to 40 taps: 3000 wavefronts of one row
    EXPECT(sysconv::conv2d_stride2_strip_rows(3, 3001, 13, 3), 2);
    EXPECT(sysconv::conv2d_stride2_strip_rows(3, 4096, 14, 3), 1);         // more taps: 4096
    EXPECT(sysconv::conv2d_stride2_strip_rows(3, 4097, 14, 3), 2);
    EXPECT(sysconv::conv2d_stride2_strip_rows(1, 100000, 2, 1), 2);
    EXPECT(sysconv::conv2d_stride2_strip_rows(1, 100001, 2, 1), 3);
    // every call has a kernel that is built: pairs with three rows of 10 or 11 columns or four of 1 to 3 or 12 and more are not
    for (int kh = 1; kh <= SYS_MAX_K2D; ++kh)
        for (int kw = 1; kw <= SYS_MAX_K2D; ++kw)
            for (int oh : {1, 8, 1000, 4000, 20000, 100001, INT_MAX / 2 + 1})
                for (int ow : {1, 2, 124, 252, 1000, 20000, INT_MAX / 2 + 1}) {
                    const int w = 2 * (ow < INT_MAX / 4 ? ow - 1 : INT_MAX / 4) + kw;
                    if (sysconv::conv2d_stride2_takes_strips(w, oh, ow, kh, kw)) {
                        const int rows = sysconv::conv2d_stride2_strip_rows(w, oh, kh, kw);
                        if (rows != 1 && !((rows == 2 || rows == 3) && kw <= 3)) ++failures;
                        if (w >= 4 && rows != 1 && !(rows == 3 && kw == 2)) ++failures;
                    } else {
                        const int rows = sysconv::conv2d_stride2_pair_rows(oh, ow, kh, kw);
                        if (rows != 1 && rows != 2 && !(rows == 3 && kw != 10 && kw != 11) && !(rows == 4 && kw >= 4 && kw <= 11)) ++failures;
                    }
                }

    // ---- queries over their whole domain and beyond
    for (int p = -2; p <= 10; ++p)
        for (int k = -1; k <= 70; ++k) {
            (void)sys_conv1d_has(p, k);
            (void)sys_conv1d_strided_has(p, k, 2);
            for (int kw = -1; kw <= 17; ++kw) { (void)sys_conv2d_has(p, k, kw); (void)sys_conv2d_strided_has(p, k, kw, 2); }
        }
    for (int s = -3; s <= 12; ++s) if (!sys_status_string(s) || !sys_projection_name(s)) ++failures;
    EXPECT(sys_copy_f32(X, X + 1, 10, nullptr), SYS_ERR_ALIAS);
    EXPECT(sys_copy_f32(X, Y, 0, nullptr), SYS_ERR_SIZE);
    EXPECT(sys_last_hip_error(), 0);
    if (sys_version() < 200) ++failures;

    printf(failures ? "FAILED (%d)\n" : "clean\n", failures);
    return failures ? 1 : 0;
}
