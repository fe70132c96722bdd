// Launch shapes that depend on the size of a simulation: plain host C++ (no
// HIP), shared by the launchers and by a test over the accepted sizes.
#pragma once

#include <stdint.h>

namespace pic {

// Threads that settle one tile (k_settle) of a simulation with n particles in
// n_tiles tiles, a power of two from 16 to `most`: each takes four particles
// per pass, four passes for a tile of average size, or one as long as the device
// has places for all threads at once.  A tile of few particles
// does not pay for wavefronts with nothing to do, and the launch stays below
// 2^32 threads whatever the grid: n_tiles * threads is at most 16 n_tiles,
// n / 8 or the device's places.  us by tiles x particles a tile, as two launches
// of a wavefront per tile and a particle per lane / always 1,024 threads / two
// passes / four / eight: 65,536 x 64 17 / 192 / 11 / 11 / 11; 16,384 x 1,024 23 /
// 57 / 22 / 20 / 21; 16,384 x 4,096 140 / 118 / 96 / 82 / 84; 4,096 x 16,384 203 /
// 83 / 82 / 82 / 82; 16 x 4,096 17 / 5.1 / 4.5 / 5.2 / 6.1.
constexpr int64_t kDeviceThreads = 256 * 2048;   // compute units, threads on each
inline int settle_threads(int64_t n, int64_t n_tiles, int most)
{
    int64_t t = 16;
    while (t < most && (n > 16 * t * n_tiles || (n > 4 * t * n_tiles && 2 * t * n_tiles <= kDeviceThreads))) t *= 2;
    return (int)t;
}

// A grid of at least `blocks` workgroups of `threads` with less than 2^32
// threads on an axis: the blocks in a row, or in equal rows where one row would
// be too long.  A kernel takes its linear index and ends past the last block.
struct BlockGrid {
    unsigned x, y;
};
inline BlockGrid block_grid(int64_t blocks, int threads)
{
    const int64_t most = ((int64_t(1) << 32) - 1) / threads;
    const int64_t rows = blocks <= most ? 1 : (blocks + most - 1) / most;
    return BlockGrid{(unsigned)((blocks + rows - 1) / rows), (unsigned)rows};
}

}  // namespace pic
