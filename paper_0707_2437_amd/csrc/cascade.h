// cascade.h -- tile geometry of the cascade kernels (cascade.hip), shared by
// their launchers and the host runtime.
#pragma once

namespace lbm {

constexpr int kCascadeWaves = 4;  // of a team; a pass takes as many steps, or twice as many

// A cascade team advances a strip of 64 vx columns by ns steps of Eq. 5 in
// one pass over memory. Every step needs the neighbours' post-collision
// values (one site away) and, for its density gradient, the neighbours'
// densities; lanes take both from their neighbour lanes only, so a strip
// loses a column at each side per exchange, 2 ns - 1 in all (the first
// gather comes from memory), and a chunk of rows starts 2 ns - 1 rows early.
constexpr int cascade_halo(int ns) { return 2 * ns - 1; }
// Lanes at each side that only feed the others, rounded up so that every
// strip writes whole 64-byte blocks (es: bytes of a stored value). A block
// that two strips write in part leaves the cache twice, in partial writes:
// measured on the bare access pattern (9 planes of 4096^2 FP32), strips of
// 112 columns move 1.42 GB in 262 us, strips of 120 columns or strips
// shifted by half a block 1.3-1.4 GB in 349-356 us. FP16 rows hold half the
// bytes and their pass is bound by instructions: half blocks cost it less
// than the lanes that whole ones would idle (8192^2, two columns per lane in
// one wave: 205 us per step with strips of 112 columns, 218 with 96).
constexpr int cascade_halo_lanes(int vx, int ns, int es)
{
    int hl = (cascade_halo(ns) + vx - 1) / vx;
    while ((64 - 2 * hl) * vx * es % (es == 2 ? 32 : 64)) ++hl;
    return hl;
}
constexpr int cascade_cols(int vx, int ns, int es) { return (64 - 2 * cascade_halo_lanes(vx, ns, es)) * vx; }

// Columns per lane.
constexpr int cascade_vx(int dtype) { return dtype == 3 ? 4 : 2; }

// Shape of a lattice's cascade passes: levels per wave (steps per pass /
// kCascadeWaves), rows per chunk; levels = 0: other passes are faster.
struct CascadeShape {
    int levels = 0, h = 0;
};
// out[0]: four steps per pass, out[1]: eight. inlet: with inlet/outlet boundaries.
void cascade_shapes(int dtype, int nx, int ny, bool inlet, CascadeShape out[2]);
// Four steps per pass of a batch of lattices of the given sizes (nx[k] x ny[k]).
CascadeShape cascade_batch_shape(int dtype, const int* nx, const int* ny, int count);

}  // namespace lbm
