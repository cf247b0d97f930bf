// block.h -- tile geometry of the block kernel (block.hip), shared by its
// launcher and the host runtime.
#pragma once

namespace lbm {

constexpr int kBlockWaves = 16;     // rows of a tile at most, one per wave
constexpr int kBlockMaxSteps = 15;  // steps per pass at most (a strip keeps 6 of its 64 columns)

// A block pass of ns steps: tiles of `waves` rows and 64 columns. Columns
// lose 2 ns - 1 at each side (as in cascade.h), and so do rows, unless the
// tile holds all rows of the lattice (which then wrap inside the tile).
struct BlockShape {
    int ns = 0, waves = 0;  // ns = 0: no block passes
    int halo(int ny) const { return waves == ny ? 0 : 2 * ns - 1; }
    int rows(int ny) const { return waves - 2 * halo(ny); }
    int cols() const { return 64 - 2 * (2 * ns - 1); }
    long long tiles(int nx, int ny) const
    {
        return (long long)((nx + cols() - 1) / cols()) * ((ny + rows(ny) - 1) / rows(ny));
    }
};
// The next pass of a lattice with n >= 1 more steps to take (ns <= n);
// inlet: with inlet/outlet boundaries.
BlockShape block_shape(int dtype, int nx, int ny, int n, bool inlet);

}  // namespace lbm
