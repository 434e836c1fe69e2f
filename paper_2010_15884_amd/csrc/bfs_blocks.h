// One step of the BFS array that runs along a lane's registers: the four inputs m = 4b .. 4b+3 meet the four PEs (outputs) of a
// lane.  wv[i] = w(4b-3+i), i = 0..6, are the weights that can meet them; pair (input u, PE j) uses wv[u-j+3].  LO/HI
// bound the valid part of wv (head block: indices below 3 are taps < 0; tail blocks: indices above k+2-4b are taps >= k).
#pragma once

#include <hip/hip_runtime.h>

namespace sysconv {

template <int LO, int HI>
__device__ __forceinline__ void bfs_block(float (&acc)[4], const float (&xa)[4], const float (&wv)[7])
{
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int i = u - j + 3;
            if (i >= LO && i <= HI) acc[j] = __builtin_fmaf(wv[i], xa[u], acc[j]);
        }
}

template <int LO>
__device__ __forceinline__ void bfs_block_hi(int hi, float (&acc)[4], const float (&xa)[4], const float (&wv)[7])
{
    switch (hi) {                                                          // uniform
    case 0: bfs_block<LO, 0>(acc, xa, wv); break;
    case 1: bfs_block<LO, 1>(acc, xa, wv); break;
    case 2: bfs_block<LO, 2>(acc, xa, wv); break;
    case 3: bfs_block<LO, 3>(acc, xa, wv); break;
    case 4: bfs_block<LO, 4>(acc, xa, wv); break;
    case 5: bfs_block<LO, 5>(acc, xa, wv); break;
    default: bfs_block<LO, 6>(acc, xa, wv); break;
    }
}

}  // namespace sysconv
