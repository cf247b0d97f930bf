// internal.h -- types shared by the HIP kernels and the host runtime of liblbm.
//
// Storage ("pull" form). For every link i the device keeps one plane
// S_i[y][x] holding the post-collision value f*_i(x, y) of the previous step,
// i.e. the value that streams to x + e_i (Eq. 5, left-hand side). A step
// gathers f_i(x, t) = S_i(x - e_i), relaxes it (Eq. 5, right-hand side) and
// writes S'_i(x) aligned into the other buffer (A/B).
//
// Layout: element (x, y) of plane i sits at
//   i * ps + y * rs + off + x,   x in [0, nx)
// `off` is one 128-byte line, so x = 0 is line-aligned; the row is padded
// on both sides (the +-1-shifted windows of the gather read a little past
// the row ends and replace those elements by the periodic image, see
// gather_raw). Two layouts are supported:
// plane-major (ps = plane size, rs = pitch) and row-interleaved (ps = pitch,
// rs = 9 * pitch: the nine plane rows of a lattice row are contiguous).
// Rows wrap in y by index.
#pragma once

#include <stdint.h>

namespace lbm {

constexpr int kMaxVX = 8;

struct Geom {
    int nx, ny;
    int off;          // element offset of column 0 within a row
    int pitch;        // elements per row of one plane
    long long rs;     // elements between rows y and y + 1 of a plane
    long long ps;     // elements between planes i and i + 1
};

// Collision / source coefficients of Eq. 5 in the delta form used by the
// kernels (d_i = f_i - w_i; see collide_col in step.h), with om = 1/tau and
// the index 0, 1, 2 for the rest, axis and diagonal links (rounded together,
// see closed_coefs in host.h):
//   om1 = 1 - om;
//   a_k = om w_k (1 + e_k) multiplies drho in the even part, b_k (-3/2 om w_0,
//   -3/2 om w_1, 3 om w_2) multiplies j.u, and z_k = om w_k e_k is its
//   constant (FP64 arithmetic, centred on the weights);
//   t45 = 9/2 om w_1, t9 = 9 om w_2, w3 = 3 om w_1;
//   as1 = 3 w_1 alpha / 2: the source term 3 w_1 alpha (e_i . grad rho) is
//   applied to the undivided central differences rho(x + 1) - rho(x - 1), so
//   the 1/2 of the central difference sits in the coefficient (an exact
//   power-of-two scaling).
// e1, e0 shift the equilibrium for the altered-equilibrium model (0 for the
// paper's model): e1 for the moving links (e_1 = e_2), e0 for the rest one.
template <class C> struct CoefSet {
    C om1, a0, a1, a2, b0, b1, b2, z0, z1, z2, t45, t9, w3, as1, e1, e0;
};
// In FP64 and in FP32, each closed by itself.
struct Coef {
    CoefSet<double> d;
    CoefSet<float> f;
};

// One lattice as seen by a step launch.
struct StepTile {
    const void* src;
    void* dst;
    Geom g;
    Coef c;
    int h;        // rows per workgroup
    int nstrips;  // column strip groups (one per workgroup)
    int nchunks;  // row chunks
    int rowband;  // tile order: 1 = strip groups of a chunk first
    int xcd_chunk;  // vertical-stack tile order over the 8 XCDs (see xcd_tile in step.h)
    // Per-site source coefficients (a c2 field): field[y * fpitch + x] =
    // as1 at site (x, y) in compute precision; nullptr for the uniform one
    // of c.
    const void* field;
    int fpitch;
};

// A dispatch's work-item count is 32-bit: launchers refuse a grid that
// would exceed it (hipErrorInvalidConfiguration) rather than have it cut.
inline bool grid_fits(long long blocks, int threads) { return blocks * threads <= 0xffffffffLL; }

// The source coefficient of the axis links, as1 = 3 w_1 alpha / 2 with
// alpha = 1/3 - c2 (Eq. 8; the diagonal links take a quarter of it, exactly,
// since w_2 = w_1 / 4). One definition for the uniform coefficients and the
// per-site field, so that a uniform field gives the same bits.
__host__ __device__ inline double source_as1(double c2)
{
    const double alpha = 1.0 / 3.0 - c2;
    return 1.5 * (1.0 / 9.0) * alpha;
}

// One lattice of a batched launch (device array, read by every workgroup).
// tile.src holds the buffer of even times and tile.dst the buffer of odd
// times: at step s of the call the lattice is at time t0 + s, reads buffer
// (t0 + s) & 1 and writes the other. Lattices with s >= nsteps sit out.
// The batch's work is cut into items of up to `per_item` consecutive tiles
// of one lattice; item i belongs to lattice item_lat[i] (a device array),
// and the lattice's items are item_begin .. item_begin + nitems - 1.
// Its size counts: arrays of descriptors of up to 16 KiB (97 lattices) reach the
// device in 3 us, larger ones in 15 more. So it holds what the batched kernels
// read: pools step the paper's model (e = z = 0), without c2 fields, and the
// coefficients are those of the pool's compute precision.
template <class C> struct BatchCoefSet {
    C om1, a0, a1, a2, b0, b1, b2, t45, t9, w3, as1;
};
union BatchCoef {
    BatchCoefSet<double> d;
    BatchCoefSet<float> f;
};
struct BatchTile {  // members as in StepTile
    const void* src;
    void* dst;
    Geom g;
    BatchCoef c;
    int h, nstrips, nchunks;
};
struct BatchLat {
    BatchTile tile;  // of tile.nstrips * tile.nchunks tiles
    int t0;          // parity of the lattice's time when the call starts
    int nsteps;      // steps this lattice takes in the call
    int item_begin;  // first batch item of this lattice
    int per_item;    // tiles per item
};
static_assert(sizeof(BatchLat) <= 168, "97 descriptors in 16 KiB");

}  // namespace lbm
