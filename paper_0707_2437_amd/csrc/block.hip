// block.hip -- many steps of the variable-speed-of-sound D2Q9 step (Buick &
// Cosgrove, Sec. 3 Eq. 5) per launch, for lattices too small to fill the GPU.
//
// Such a lattice is bound by the latency of a launch (about 4 us for loads,
// stores and the gap to the next one), so a launch takes as many steps as
// its redundant halo allows. A workgroup holds a tile of up to 16 rows of 64
// columns in registers, one row per wave, one column per lane, and steps it
// in place: a step publishes the row's densities in LDS, relaxes, publishes
// the six planes that leave the row, and gathers them from the rows above
// and below; neighbours along the row come from the neighbour lanes (DPP) or
// the neighbouring LDS slots. Two barriers per step; no memory traffic
// between steps. After ns steps the 2 ns - 1 outermost rows and columns of
// the tile are stale and are not written. A lattice of at most 16 rows is
// held whole in y: its rows wrap inside the tile and need no halo.
// Rows and columns outside the lattice are periodic images (Sec. 4): every
// lane loads its own site's wrapped sources. Every site's arithmetic is the
// single-step code of step.h on the values a single step would load, so a
// pass gives the bits of ns single steps.
#include <hip/hip_runtime.h>

#include "block.h"
#include "dpp.h"
#include "host.h"
#include "internal.h"
#include "step.h"
#include "xbc.h"

namespace lbm {

template <class C> struct BlockLds {
    static constexpr int LW = 66;  // 64 columns and one slot on each side
    C rho[kBlockWaves][LW];
    C f[6][kBlockWaves][LW];  // planes 2, 5, 6 (e_iy = 1), 4, 7, 8 (e_iy = -1)
};

struct BlockPeriodic {};

// XBC: the sites of columns 0 and nx - 1 emit the values of xb in place of
// their results (as launch_xbc writes them after a single step).
template <class T, bool SHIFT, bool FIELD, bool XBC>
__global__ __launch_bounds__(64 * kBlockWaves) void block_kernel(
    StepTile a, int ns, int halo, typename std::conditional<XBC, XbcValues<T>, BlockPeriodic>::type xb)
{
    using C = typename CompT<T>::type;
    constexpr bool RC = ModelCentred<C>::value;
    constexpr unsigned es = sizeof(T);
    constexpr int ex[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
    constexpr int ey[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
    constexpr int pl[6] = {2, 5, 6, 4, 7, 8};
    __shared__ BlockLds<C> lds;
    const Geom g = a.g;
    const int nw = (int)(blockDim.x >> 6);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    const int strip = (int)blockIdx.x % a.nstrips, grp = (int)blockIdx.x / a.nstrips;
    const int H = 2 * ns - 1, W = 64 - 2 * H, R = nw - 2 * halo;
    const int y = grp * R - halo + wave, x = strip * W - H + lane;
    const CoefC<C> k = coef_c<C>(a.c);
    const Centre<C> cn = centre_c<C, RC>(a.c);
    auto wrap = [](int v, int n) {
        v %= n;
        return v < 0 ? v + n : v;
    };
    // The site's wrapped row and column, and its populations from their
    // sources' wrapped sites.
    const int yw = wrap(y, g.ny), xw = wrap(x, g.nx);
    const int xl = xw == 0 ? g.nx - 1 : xw - 1, xr = xw == g.nx - 1 ? 0 : xw + 1;
    const unsigned rsb = (unsigned)g.rs * es;
    const unsigned o0 = (unsigned)yw * rsb;
    const unsigned om = (unsigned)(yw == 0 ? g.ny - 1 : yw - 1) * rsb;
    const unsigned op = (unsigned)(yw == g.ny - 1 ? 0 : yw + 1) * rsb;
    const char* p = (const char*)a.src + (long long)g.off * (long long)es;
    T raw[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const char* row = p + (ey[i] > 0 ? om : (ey[i] < 0 ? op : o0));
        raw[i] = ld_g<T>(row + (size_t)((unsigned)(ex[i] > 0 ? xl : (ex[i] < 0 ? xr : xw)) * es));
        p += (unsigned long long)g.ps * es;
    }
    C as1 = C(0);
    if constexpr (FIELD)
        as1 = ld_g<C>((const char*)a.field + (size_t)yw * a.fpitch * sizeof(C) +
                      (size_t)((unsigned)xw * (unsigned)sizeof(C)));
    const CoefC<C> ks = site_coef<FIELD>(k, as1);
    ColF<C> v;
#pragma unroll
    for (int i = 0; i < 9; ++i) v.d[i] = to_d<T, SHIFT, C>(raw[i], i, cn);

    const int up = wave == nw - 1 ? 0 : wave + 1, dn = wave == 0 ? nw - 1 : wave - 1;
    const int col = lane + 1;  // the lane's LDS slot
    T f[9];
    for (int s = 0;; ++s) {
        const C w = drho_col(v);
        lds.rho[wave][col] = w;
        const C gx = from_right(w) - from_left(w);
        __syncthreads();
        const C gy = lds.rho[up][col] - lds.rho[dn][col];
        C o[9];
        collide_col<RC>(v, w, gx, gy, ks, o);
#pragma unroll
        for (int i = 0; i < 9; ++i) f[i] = from_d<T, SHIFT, C>(o[i], i, cn);
        if constexpr (XBC) {
#pragma unroll
            for (int i = 0; i < 9; ++i) f[i] = xbc_value<T>(xb, s, i, ex[i], xw, g.nx, f[i]);
        }
        if (s == ns - 1) break;
        C q[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) q[i] = to_d<T, SHIFT, C>(f[i], i, cn);
#pragma unroll
        for (int m = 0; m < 6; ++m) lds.f[m][wave][col] = q[pl[m]];
        v.d[0] = q[0];
        v.d[1] = from_left(q[1]);
        v.d[3] = from_right(q[3]);
        __syncthreads();
#pragma unroll
        for (int m = 0; m < 6; ++m) v.d[pl[m]] = lds.f[m][m < 3 ? dn : up][col - ex[pl[m]]];
    }
    const bool out = wave >= halo && wave < nw - halo && y < g.ny && lane >= H && lane < 64 - H && x < g.nx;
    if (!out) return;
    char* q = (char*)a.dst + (long long)g.off * (long long)es + (size_t)o0;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        st_g<T>(q + (size_t)((unsigned)x * es), f[i]);
        if constexpr (GhostCols<T>::value) {  // copies of the edge columns (see write_row in step.h)
            if (x >= g.nx - 2) st_g<T>(q + (long long)(x - g.nx) * (int)es, f[i]);
            if (x <= 1) st_g<T>(q + (size_t)((unsigned)(x + g.nx) * es), f[i]);
        }
        q += (unsigned long long)g.ps * es;
    }
}

template <class T, bool SHIFT>
static hipError_t launch_block_t(const BlockShape& b, const StepTile& t, const PassInlet* inlet, hipStream_t st)
{
    const dim3 grid((unsigned)(t.nstrips * t.nchunks)), block(64 * b.waves);
    const int halo = b.halo(t.g.ny);
    if (!grid_fits((long long)grid.x, (int)block.x)) return hipErrorInvalidConfiguration;
    if (inlet) {
        const XbcValues<T> xb = xbc_values<T, SHIFT>(*inlet, b.ns);
        hipLaunchKernelGGL((block_kernel<T, SHIFT, false, true>), grid, block, 0, st, t, b.ns, halo, xb);
    } else if (t.field) {
        hipLaunchKernelGGL((block_kernel<T, SHIFT, true, false>), grid, block, 0, st, t, b.ns, halo, BlockPeriodic{});
    } else {
        hipLaunchKernelGGL((block_kernel<T, SHIFT, false, false>), grid, block, 0, st, t, b.ns, halo, BlockPeriodic{});
    }
    return hipGetLastError();
}

// b.ns steps; t's strips and groups are those of b. inlet: the boundaries in
// x, or nullptr (periodic).
hipError_t launch_block(int dtype, const BlockShape& b, const StepTile& t, const PassInlet* inlet, hipStream_t st)
{
    if (b.ns < 1 || b.ns > kBlockMaxSteps || b.waves < 1 || b.waves > kBlockWaves || b.rows(t.g.ny) < 1)
        return hipErrorInvalidValue;
    if (inlet && t.field) return hipErrorInvalidValue;
    switch (dtype) {
    case 0: return launch_block_t<double, false>(b, t, inlet, st);
    case 1: return launch_block_t<float, false>(b, t, inlet, st);
    case 2: return launch_block_t<float, true>(b, t, inlet, st);
    case 3: return launch_block_t<_Float16, true>(b, t, inlet, st);
    }
    return hipErrorInvalidValue;
}

// Lattices of at most 16 rows always take block passes. More steps per pass
// share its fixed cost among more steps, but a strip keeps fewer columns, so
// there are more of them: the estimate (us, fitted on MI355X over widths of
// 400 to 200 000) is the fixed cost, the larger of a step's latency and the
// issue time of the waves that share a SIMD, and their loads and stores.
// Measured per step against two-step passes: 4000 x 4 FP64 3.81 and 0.83 us
// (12 steps per pass), FP32 2.96 and 0.68; 60000 x 4 FP32 17.3 and 1.9 (8).
// Taller lattices: tiles of 16 rows, of which 4 steps leave 2 and 3 leave 6;
// worth it while every tile has a CU to itself (64^2 FP32 3.12 and 1.45 us,
// FP64 2.82 and 1.83; 256^2 FP32 215 tiles 3.62 and 2.63, 320^2 324 tiles
// 3.65 and 3.49), in FP64, whose LDS traffic is twice as much, 3 steps up to
// half of that (192^2 128 tiles 2.91 and 2.85; 220^2 185 tiles 2.98 and
// 3.25). With inlet/outlet boundaries the alternative is a cascade pass: 3
// steps up to 800 tiles in FP64 (400^2 5.5 us per step, cascade 6.3; 512^2 7.3
// and 7.1), 1250 in FP32 (600^2 5.6 and 5.8; 700^2 7.0 and 5.8), 2500 in FP16
// (1000 x 777 10.5 and 12.3). One step alone could also be a single-step launch and one
// for the boundaries, which in FP16 is as fast from 1500 tiles (650^2 10.1 and 10.6;
// 700^2 11.2 and 10.2; 5000 x 100 10.8 and 10.0).
BlockShape block_shape(int dtype, int nx, int ny, int n, bool inlet)
{
    BlockShape best;
    if (n < 2 && !(inlet && n == 1)) return best;
    if (ny <= kBlockWaves) {
        const bool wide = dtype == 0;
        const double t0 = wide ? 2.9 : 2.6, lat = wide ? 0.38 + 0.05 * ny : 0.30 + 0.04 * ny;
        const double issue = wide ? 0.32 : 0.20, mem = wide ? 0.7 : 0.3;
        double t_best = 0;
        for (int ns = 1; ns <= kBlockMaxSteps && ns <= n; ++ns) {
            BlockShape b;
            b.ns = ns;
            b.waves = ny;
            const double m = (double)b.tiles(nx, ny) * ny / 1024;  // waves per SIMD
            const double t = (t0 + ns * (m * issue > lat ? m * issue : lat) + m * mem) / ns;
            if (best.ns == 0 || t < t_best) {
                t_best = t;
                best = b;
            }
        }
        // the passes of the rest of the count, evenly
        const int passes = (n + best.ns - 1) / best.ns;
        best.ns = (n + passes - 1) / passes;
        return best;
    }
    BlockShape b;
    b.waves = kBlockWaves;
    b.ns = 4;
    if (b.tiles(nx, ny) > 256) {
        b.ns = 3;
        const int most[4] = {800, 1250, 1250, n == 1 ? 1500 : 2500};
        if (b.tiles(nx, ny) > (inlet ? most[dtype] : (dtype == 0 ? 128 : 256))) return best;
    }
    if (b.ns > n) b.ns = n;
    return b;
}

}  // namespace lbm
