// Sizes of the tiles and of their LDS hash, and the launch geometry of the
// build kernels whose extent is a vertex or table count rather than the
// points': plain arithmetic, used by the kernels and by the host that sizes
// their buffers and grids.
//
// A launch may have fewer than 2^32 work items per dimension, and a lattice
// may have up to 2^31 - 1 vertices, so M (d+1) neighbour items, or a table's
// slots, can be more than both a launch and a 32-bit index hold: these blocks
// are limited in number and stride over the rest.
#pragma once

#include <stdint.h>

namespace pam {

#ifndef PAM_TILE_POINTS
#define PAM_TILE_POINTS 512
#endif
#ifndef PAM_TILE_BIG_D
#define PAM_TILE_BIG_D 5  // largest d with PAM_TILE_POINTS-point tiles
#endif
#ifndef PAM_TILE_POINTS_HIGH_D
#define PAM_TILE_POINTS_HIGH_D 256  // tile points above PAM_TILE_BIG_D
#endif
constexpr int tile_points(int d)
{
    return d <= PAM_TILE_BIG_D ? PAM_TILE_POINTS
                               : (PAM_TILE_POINTS < PAM_TILE_POINTS_HIGH_D ? PAM_TILE_POINTS : PAM_TILE_POINTS_HIGH_D);
}

// Slots of a tile's LDS hash: at least an eighth more than its contributions,
// so that every tile has room for its rows, whatever its points, and as many
// as fit the LDS that the tile's sorted entries take later (d >= 6).  With
// 2048 slots up to d = 11 and 4096 above, tiles of scattered points did not
// fit and went on without rows: 1000 points, d = 5, 16 channels 559 us per
// step (120 with room), 40x36x28 points, d = 11, 24 channels 2227 us (580).
constexpr int tile_slots(int d)
{
    const int least = tile_points(d) * (d + 1) / 8 * 9, room = tile_points(d) * d / 3 * 4;
    return room > least ? room : least;
}
// first slot probed for a local key
constexpr uint32_t tile_hash(uint32_t lkey, uint32_t slots)
{
    return (uint32_t)(((uint64_t)(uint32_t)(lkey * 2654435761u) * slots) >> 32);
}

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
