// What the two matrix-core kernels that walk down blocks of rows (conv2d_split.hip, conv2d_mfma.hip) have in common: the barrier
// between their chunks and the height of a block.
#pragma once

#include "tiling.h"

namespace sysconv {

constexpr int kPlaces = 512;                // workgroups of four wavefronts a whole device of 256 CUs holds at two a CU (a partition of one holds fewer: the heights are then chosen for a larger device, the results are the same)
constexpr int kNonTemporal = 2;             // the nt bit of a buffer store
constexpr unsigned kNowhere = 0xffffff00u;  // offset of a buffer store that is dropped

// Barrier for what the workgroup exchanges through LDS: the loads from global memory that are in flight stay so.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Output groups (of 4 or 8 rows) of a workgroup's block, at most `most`: those whose modelled time is least.  A block of m groups takes
// u = steps * (units_per_group (m - 1) + units) steps, one a unit of two input rows and column of matrix instructions.  One workgroup a CU
// takes u, two 6 steps + 1.1 u (in time of a step; with 8 x 2 offsets, two columns, blocks of one group and two or of two groups and one a CU: us 744x580 11x14 9.6 / 8.7, 739x747 10x14 9.8 / 8.9, 1473x288 12x15
// 10.3 / 9.45; where one group leaves one a CU 500^2 14x14 8.6 / 9.4); beyond that workgroups follow one another freely, no rounds are seen, a block costs its steps and `setup` more (taps, first
// loads, units that only finish groups apart), and the launch ends with blocks that are still under way (u / 2).  Fitted to sweeps over all heights on 101 random and listed images and
// filters (256 .. 8192 rows and columns): the height chosen is 0.8 % slower than the best one on average (MFMA: 60 images, 2 %), 8 % at most.  Whole chunks of 16
// rows in whole rounds, as blocks were chosen before, lost 15 % on 2000^2 11x11 (9 groups of four rows 15.7 us, 8 18.8, 12 16.8), 17 % on 3001x4003 15x15 (13 groups of eight rows 45.2,
// 14 47.4, 12 56.8) and 25 % on 6000^2 9x9 (MFMA; 14 groups 57, 64 67).
inline int matrix_block_groups(int all, int strips, int units, int units_per_group, int steps, double setup, int most)
{
    static constexpr short kHeights[] = {1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15, 16, 18, 20, 22, 24, 26, 28, 30, 32, 36, 40, 44, 48, 56, 64, 72, 80, 96, 112, 128};
    int best = 1;
    double least = 0.0;
    for (const int m : kHeights) {
        if (m > most || (m > 1 && m > all)) break;
        const double places = (double)((all + m - 1) / m) * strips * (1.0 / kPlaces);
        const double u = steps * (units_per_group * (m - 1) + units);
        const double cost = places > 1.0 ? places * (setup + u) + 0.5 * u : places > 0.5 ? 6.0 * steps + 1.1 * u : u;
        if (m == 1 || cost < least) { best = m; least = cost; }
    }
    const int blocks = (all + best - 1) / best;
    return (all + blocks - 1) / blocks;                                    // as many blocks, as even as they go
}

}  // namespace sysconv
