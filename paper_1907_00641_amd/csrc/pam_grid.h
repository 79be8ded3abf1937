// Launch geometry of the build kernels whose extent is a vertex or table
// count rather than the points': plain arithmetic, used by the kernels and by
// the host that sizes their grids.
//
// A launch may have fewer than 2^32 work items per dimension, and a lattice
// may have up to 2^31 - 1 vertices, so M (d+1) neighbour items, or a table's
// slots, can be more than both a launch and a 32-bit index hold: these blocks
// are limited in number and stride over the rest.
#pragma once

#include <stdint.h>

namespace pam {

constexpr int kGridBlock = 256;  // threads per block of the resolve launch

// Neighbour table: as many blocks for each of the d+1 directions, a thread
// per vertex and trip.  At most 2^19 blocks per direction (2^27 vertices per
// trip): 17 directions are 2^23.1 of the 2^24 blocks a launch may have.
constexpr unsigned nbr_blocks_per_dir(int64_t M_estimate)
{
    const int64_t blocks = (M_estimate + kGridBlock - 1) / kGridBlock, most = (int64_t)1 << 19;
    return (unsigned)(blocks < 1 ? 1 : (blocks > most ? most : blocks));
}
constexpr int nbr_dir(unsigned block, unsigned per_dir) { return (int)(block / per_dir); }
constexpr int64_t nbr_first(unsigned block, unsigned per_dir, int thread)
{
    return (int64_t)(block % per_dir) * kGridBlock + thread;
}
constexpr int64_t nbr_stride(unsigned per_dir) { return (int64_t)per_dir * kGridBlock; }
// direction-major place of vertex m's pair of neighbours in direction j
constexpr int64_t nbr_entry(int j, int64_t m, int64_t M) { return (int64_t)j * M + m; }

// Clearing blocks of `threads` threads for a table of cap slots, a slot per
// thread and trip: at most 2^30 work items, next to fewer than 2^31 for the
// points of the same launch.
constexpr unsigned table_clear_blocks(uint64_t cap, int threads)
{
    const uint64_t blocks = (cap + threads - 1) / threads, most = ((uint64_t)1 << 30) / threads;
    return (unsigned)(blocks < most ? blocks : most);
}

}  // namespace pam
