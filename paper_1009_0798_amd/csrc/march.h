// Geometry of the plane-marching kernels of the base level (k_march.hip).
#pragma once

#include "common.h"

namespace ohm {

constexpr int MT = 16;                       // tile edge in x and y (cells): 2 x 2 blocks
constexpr int MHW = MT / 2 + 2;              // pairs of x-neighbours per tile row, halo of two cells
constexpr int MNP = MHW * (MT + 4);          // pairs per plane with the halo (200)
constexpr int MARCH_THREADS = 256;
constexpr int MARCH_MAX_NBZ = 32;            // blocks of a column segment

// One workgroup: a column segment of 2 x 2 blocks (fewer at the box's edge)
// across and nbz blocks along z, at most MARCH_MAX_NBZ
struct MarchTile {
    int prob, bx, by, bz, nbz;               // its first block, its blocks along z
    int nx, ny, nz;                          // blocks of the problem's box per axis
    int map;                                 // first entry of the problem in the position -> block map
    int pad[7];
};

}  // namespace ohm
