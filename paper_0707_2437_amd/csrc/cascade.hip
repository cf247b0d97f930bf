// cascade.hip -- several steps of the variable-speed-of-sound D2Q9 step (Buick
// & Cosgrove, Sec. 3 Eq. 5) per pass over memory, held in registers.
//
// Every 64-lane wave owns a strip of 64 * VX columns and walks down a chunk
// of rows. A row enters at level 0 from memory and falls through NS levels,
// one step of Eq. 5 each; what leaves the last level is written. Level s
// works two rows behind level s - 1: it relaxes a row as soon as the density
// of the row below it is known, and hands the nine results, rounded to the
// storage type, to level s + 1, which gathers a row from the results of
// three consecutive rows (the planes with e_iy = 1 of the first, 0 of the
// second, -1 of the third). Per level the wave keeps the populations of one
// row, two rows of densities and the planes' rows that are still waited for;
// x-neighbours come from the neighbour lanes (DPP wave shifts). There is no
// LDS and no barrier. Every site's arithmetic is the single-step code of
// step.h on the values a single step would load, so a pass gives the bits of
// NS single steps.
//
// Bound: one load and one store of the state per NS steps, against 59
// operations per site and step (77 with the FP32 form's conversions). At NS
// = 4 the two are about even: FP32 at 4096^2 takes 285 us per pass, of which
// the instructions alone need 195 us and the bare access pattern 262 us.
// With NS = 2 and 3 the pass takes as long (270 and 299 us) and does less;
// with NS = 5 the halo and the registers (one wave per SIMD) cost more than
// they save (83 us per step against 71). The register file is the largest
// on-chip memory (512 KB per CU against 160 KB of LDS), and 240 registers
// per lane leave two waves per SIMD, enough here: a wave's loads for the
// next row are in flight for the whole of a row's arithmetic.
// Measured per step, the two-step kernel before and this one: FP32 4096^2
// 121.7 and 71.3 us, FP64 4096^2 240.5 and 127.0 us.
#include <hip/hip_runtime.h>

#include "cascade.h"
#include "dpp.h"
#include "host.h"
#include "internal.h"
#include "step.h"

namespace lbm {

// The lane's VX columns of one plane's row as the levels hold them. FP32 and
// FP64: d_i in compute precision.
template <class T, bool SHIFT, int VX> struct CascadeRow {
    using C = typename CompT<T>::type;
    using Mem = Pack<T, VX>;  // as loaded and stored
    static __device__ __forceinline__ T get(const Mem& p, int j) { return p.v[j]; }
    template <class F> static __device__ __forceinline__ Mem each(F&& f)  // column j: f(j)
    {
        Mem p;
#pragma unroll
        for (int j = 0; j < VX; ++j) p.v[j] = f(j);
        return p;
    }
    C v[VX];
    static __device__ __forceinline__ CascadeRow of(const Mem& p, int i, const Centre<C>& cn)
    {
        CascadeRow r;
#pragma unroll
        for (int j = 0; j < VX; ++j) r.v[j] = to_d<T, SHIFT, C>(p.v[j], i, cn);
        return r;
    }
    // The values gathered from column x - EX: r(x) = this(x - EX).
    template <int EX> __device__ __forceinline__ CascadeRow shifted() const
    {
        CascadeRow r;
        static_for<0, VX>([&](auto jc) {
            constexpr int j = decltype(jc)::value, c = j - EX;
            if constexpr (c < 0) r.v[j] = from_left(v[VX - 1]);
            else if constexpr (c >= VX) r.v[j] = from_right(v[0]);
            else r.v[j] = v[c];
        });
        return r;
    }
    template <int J> static __device__ __forceinline__ ColF<C> col(const CascadeRow (&r)[9])
    {
        ColF<C> k;
#pragma unroll
        for (int i = 0; i < 9; ++i) k.d[i] = r[i].v[J];
        return k;
    }
    // The results of column J (a) and, if G is 2, of the next (b), rounded
    // to the storage type.
    template <int J, int G>
    static __device__ __forceinline__ void store(const C (&a)[9], const C (&b)[9], Mem (&f)[9], const Centre<C>& cn)
    {
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            f[i].v[J] = from_d<T, SHIFT, C>(a[i], i, cn);
            if constexpr (G == 2) f[i].v[J + 1] = from_d<T, SHIFT, C>(b[i], i, cn);
        }
    }
};

// FP16 storage: the halves as stored, two columns per register, read by
// mixed-precision FMAs (ColH in step.h). A shift by one column moves each
// register's halves with one align instruction.
template <int VX> struct CascadeRow<_Float16, true, VX> {
    static_assert(VX % 2 == 0, "two columns per register");
    static constexpr int Q = VX / 2;
    struct Mem {
        unsigned q[Q];
    };
    static __device__ __forceinline__ unsigned short get(const Mem& p, int j)
    {
        return (unsigned short)(p.q[j >> 1] >> (16 * (j & 1)));
    }
    template <class F> static __device__ __forceinline__ Mem each(F&& f)
    {
        Mem p;
#pragma unroll
        for (int k = 0; k < Q; ++k)
            p.q[k] = (unsigned)__builtin_bit_cast(unsigned short, f(2 * k)) |
                     (unsigned)__builtin_bit_cast(unsigned short, f(2 * k + 1)) << 16;
        return p;
    }
    unsigned q[Q];
    static __device__ __forceinline__ CascadeRow of(const Mem& p, int, const Centre<float>&)
    {
        CascadeRow r;
#pragma unroll
        for (int k = 0; k < Q; ++k) r.q[k] = p.q[k];
        return r;
    }
    template <int EX> __device__ __forceinline__ CascadeRow shifted() const
    {
        CascadeRow r;
        static_for<0, Q>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            if constexpr (EX > 0) {
                unsigned lo;
                if constexpr (k == 0) lo = from_left(q[Q - 1]);
                else lo = q[k - 1];
                r.q[k] = __builtin_amdgcn_alignbit(q[k], lo, 16);
            } else {
                unsigned hi;
                if constexpr (k == Q - 1) hi = from_right(q[0]);
                else hi = q[k + 1];
                r.q[k] = __builtin_amdgcn_alignbit(hi, q[k], 16);
            }
        });
        return r;
    }
    template <int J> static __device__ __forceinline__ ColH<J & 1> col(const CascadeRow (&r)[9])
    {
        ColH<J & 1> k;
#pragma unroll
        for (int i = 0; i < 9; ++i) k.w[i] = r[i].q[J >> 1];
        return k;
    }
    template <int J, int G>
    static __device__ __forceinline__ void store(const float (&a)[9], const float (&b)[9], Mem (&f)[9],
                                                 const Centre<float>&)
    {
        static_assert(G == 2, "two columns per register");
#pragma unroll
        for (int i = 0; i < 9; ++i) f[i].q[J / 2] = pack_h2(a[i], b[i]);
    }
};

// One level's state between rows: the row it relaxes next (populations d,
// densities w), the densities of the row above it (wp), and the planes of
// its last results that wait for rows below: e_iy = 0 of the last row (z),
// e_iy = 1 of the last two (up, by the row's parity).
template <class R, class C, int VX> struct CascadeLevel {
    R d[9];
    C w[VX], wp[VX];
    R z[3], up[2][3];
};

constexpr unsigned kNoStore = 0x80000000u;  // past every row: the range check of a buffer store drops the lane

template <bool NT, class V>
__device__ __forceinline__ void buf_store(__amdgpu_buffer_rsrc_t rs, const V v, unsigned voff, unsigned soff)
{
    constexpr int aux = NT ? 2 : 0;
    if constexpr (sizeof(V) == 2) {
        __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, v), rs, voff, soff, aux);
    } else if constexpr (sizeof(V) == 4) {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), rs, voff, soff, aux);
    } else {
        static_assert(sizeof(V) == 8, "rows of up to two dwords per lane");
        typedef unsigned u2 __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), rs, voff, soff, aux);
    }
}

// One tile: NS steps of rows [chunk a.h, (chunk + 1) a.h) and the strip's
// inner columns. EDGE: a strip whose window reaches past the lattice's left
// or right edge; its lanes load every element from its wrapped column
// (Sec. 4: periodic in x) and store element by element.
template <class T, bool SHIFT, int VX, int NS, bool FIELD, bool RC, bool EDGE>
__device__ __forceinline__ void cascade_tile(const StepTile& a, const void* src, void* dst, int strip, int chunk)
{
    using C = typename CompT<T>::type;
    using R = CascadeRow<T, SHIFT, VX>;
    using Mem = typename R::Mem;
    constexpr unsigned es = sizeof(T);
    constexpr int H = cascade_halo(NS), HL = cascade_halo_lanes(VX, NS, es), W = cascade_cols(VX, NS, es);
    constexpr int WARM = 2 * H;  // rows that enter before the first row that is written
    constexpr int ex[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
    const Geom g = a.g;
    const int lane = threadIdx.x & 63;
    const int x = strip * W + (lane - HL) * VX;
    const bool out = lane >= HL && lane < 64 - HL;
    const int ylo = chunk * a.h, nrow = min(a.h, g.ny - ylo);
    const CoefC<C> k = coef_c<C>(a.c);
    const Centre<C> cn = centre_c<C, RC>(a.c);
    const unsigned rsb = (unsigned)g.rs * es, psb = (unsigned)g.ps * es;
    const char* const sbase = (const char*)src + (long long)(g.off - 2) * (long long)es;  // column -2
    char* const dbase = (char*)dst + (long long)(g.off - 2) * (long long)es;

    // Byte offsets (from column -2) of the columns x - 1 .. x + VX, wrapped.
    unsigned off[VX + 2];
    if constexpr (EDGE) {
        int c = (x - 1) % g.nx;
        c = c < 0 ? c + g.nx : c;
#pragma unroll
        for (int j = 0; j < VX + 2; ++j) {
            off[j] = (unsigned)(c + 2) * es;
            c = c + 1 == g.nx ? 0 : c + 1;
        }
    } else {
        off[0] = (unsigned)(x + 1) * es;
    }
    auto next = [&](int r) { return r + 1 == g.ny ? 0 : r + 1; };
    auto wrap = [&](int r) {
        r %= g.ny;
        return r < 0 ? r + g.ny : r;
    };

    // Rows of the source planes around the row that enters (r0).
    int r0 = wrap(ylo - H), rm = wrap(ylo - H - 1), rp = next(r0);
    auto load = [&](Mem (&v)[9]) {
        const char* const pm = sbase + (size_t)((unsigned)rm * rsb);
        const char* const p0 = sbase + (size_t)((unsigned)r0 * rsb);
        const char* const pp = sbase + (size_t)((unsigned)rp * rsb);
        const char* const b[9] = {p0, p0, pm, p0, pp, pm, pm, pp, pp};
        // Made opaque here, so that the 32-bit offset stays next to the
        // scalar base (hoisted out of the loop as a 64-bit value, it costs
        // an address addition per load).
        unsigned o[VX + 2];
#pragma unroll
        for (int j = 0; j < (EDGE ? VX + 2 : 1); ++j) {
            o[j] = off[j];
            asm("" : "+v"(o[j]));
        }
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const char* q = b[i] + (size_t)(i * psb);
            if constexpr (EDGE) {
                v[i] = R::each([&](int j) { return ld_g<T>(q + (size_t)o[j + 1 - ex[i]]); });
            } else {
                constexpr int A = es < 4 ? (int)es : 4;
                v[i] = ld_g<Mem, A>(q + (size_t)o[0] + (1 - ex[i]) * (int)es);
            }
        }
    };

    // The rows' source coefficients (a c2 field), one row per level: level s
    // relaxes row r0 - 1 - 2 s of the lattice.
    int fr[NS];
    Pack<C, VX> af[NS] = {};
    auto load_field = [&]() {
        if constexpr (FIELD) {
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const char* row = (const char*)a.field + (size_t)fr[s] * a.fpitch * sizeof(C);
                if constexpr (EDGE) {
#pragma unroll
                    for (int j = 0; j < VX; ++j)
                        af[s].v[j] = ld_g<C>(row + (size_t)((off[j + 1] / es - 2) * (unsigned)sizeof(C)));
                } else {
                    af[s] = ld_g<Pack<C, VX>, 4>(row + (size_t)((unsigned)x * (unsigned)sizeof(C)));
                }
            }
        }
    };
    if constexpr (FIELD)
#pragma unroll
        for (int s = 0; s < NS; ++s) fr[s] = wrap(ylo - H - 1 - 2 * s);

    const int niter = nrow + WARM;
    // Write the kk-th row that leaves the last level. Every path issues the
    // same stores (lanes and rows that write nothing are sent past the row's
    // end), so that the wait for a row's loads counts the stores issued after
    // them instead of waiting for those too.
    auto write = [&](int kk, const Mem (&f)[9]) {
        const bool row = kk >= WARM && kk < niter;
        const unsigned y = row ? (unsigned)(ylo + kk - WARM) : 0u;
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc(dbase + (size_t)(y * rsb), 0, (int)(9 * psb), 0x00027000);
        // lanes with columns past the right edge store those inside one by one
        const bool whole = row && out && x + VX <= g.nx;
        const unsigned vo = whole ? (unsigned)(x + 2) * es : kNoStore;
        static_for<0, 9>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            buf_store<!EDGE>(rs, f[i], vo, i * psb);
        });
        if constexpr (EDGE) {
            static_for<0, VX - 1>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
                const unsigned vj = row && out && !whole && x + j < g.nx ? (unsigned)(x + j + 2) * es : kNoStore;
                static_for<0, 9>([&](auto ic) {
                    constexpr int i = decltype(ic)::value;
                    buf_store<false>(rs, R::get(f[i], j), vj, i * psb);
                });
            });
        }
    };

    CascadeLevel<R, C, VX> L[NS] = {};
    Mem raw[9];
    load(raw);
    load_field();
    {
        // writes nothing: the loop's first wait then counts the same
        // operations as the later ones
        const Mem none[9] = {};
        write(0, none);
    }

    // Compile-time loops where values are only copied: left as loops, they
    // become block copies that keep the arrays out of registers.
    auto land = [&](const Mem (&m)[9], R (&r)[9]) {
        static_for<0, 9>([&](auto ic) { r[decltype(ic)::value] = R::of(m[decltype(ic)::value], decltype(ic)::value, cn); });
    };
    // The kk-th row enters; P: its parity.
    auto iterate = [&](int kk, auto parity) {
        constexpr int P = decltype(parity)::value;
        R nd[9];
        land(raw, nd);
        Pack<C, VX> fa[NS];
        static_for<0, NS>([&](auto sc) { fa[decltype(sc)::value] = af[decltype(sc)::value]; });
        if (kk + 1 < niter) {
            rm = r0;
            r0 = rp;
            rp = next(rp);
        }
        if constexpr (FIELD)
#pragma unroll
            for (int s = 0; s < NS; ++s) fr[s] = next(fr[s]);
        load(raw);
        load_field();
        __builtin_amdgcn_sched_barrier(0);  // the loads first, then the arithmetic they overlap with
        static_for<0, NS>([&](auto sc) {
            constexpr int s = decltype(sc)::value;
            auto& l = L[s];
            C nw[VX];
            static_for<0, VX>([&](auto jc) { nw[decltype(jc)::value] = drho_col(R::template col<decltype(jc)::value>(nd)); });
            // relax the held row, its neighbour rows' densities known
            const C wl = from_left(l.w[VX - 1]), wr = from_right(l.w[0]);
            Mem f[9];
            constexpr int G = VX < 2 ? VX : 2;  // columns at a time (registers)
            static_for<0, VX / G>([&](auto gc) {
                constexpr int J = G * decltype(gc)::value;
                auto relax = [&](auto jc, C (&o)[9]) {
                    constexpr int j = decltype(jc)::value;
                    const C left = j == 0 ? wl : l.w[j > 0 ? j - 1 : 0];
                    const C right = j == VX - 1 ? wr : l.w[j < VX - 1 ? j + 1 : j];
                    // undivided central differences (Sec. 4)
                    collide_col<RC>(R::template col<j>(l.d), l.w[j], right - left, nw[j] - l.wp[j],
                                    site_coef<FIELD>(k, fa[s].v[j]), o);
                };
                C oa[9], ob[9];
                relax(std::integral_constant<int, J>{}, oa);
                if constexpr (G == 2) relax(std::integral_constant<int, J + G - 1>{}, ob);
                R::template store<J, G>(oa, ob, f, cn);
                // columns, and levels, one after the other: interleaved they need more registers
                __builtin_amdgcn_sched_barrier(0);
            });
#pragma unroll
            for (int j = 0; j < VX; ++j) {
                l.wp[j] = l.w[j];
                l.w[j] = nw[j];
            }
            static_for<0, 9>([&](auto ic) { l.d[decltype(ic)::value] = nd[decltype(ic)::value]; });
            if constexpr (s + 1 < NS) {
                // the row above the relaxed one, gathered for the next level
                R q[9];
                land(f, q);
                nd[0] = l.z[0];
                nd[1] = l.z[1].template shifted<1>();
                nd[3] = l.z[2].template shifted<-1>();
                nd[2] = l.up[P][0];
                nd[5] = l.up[P][1].template shifted<1>();
                nd[6] = l.up[P][2].template shifted<-1>();
                nd[4] = q[4];
                nd[7] = q[7].template shifted<-1>();
                nd[8] = q[8].template shifted<1>();
                l.z[0] = q[0];
                l.z[1] = q[1];
                l.z[2] = q[3];
                l.up[P][0] = q[2];
                l.up[P][1] = q[5];
                l.up[P][2] = q[6];
            } else {
                write(kk, f);
            }
        });
    };
    // Four rows per turn: a value lives for up to four rows in a level's
    // state, and with a shorter turn its registers would be copied.
    for (int kk = 0; kk < niter; kk += 4)
        static_for<0, 4>([&](auto u) {
            iterate(kk + decltype(u)::value, std::integral_constant<int, decltype(u)::value % 2>{});
        });
}

// Ghost copies of a lattice's edge columns (columns -2, -1 hold nx - 2, nx - 1;
// nx, nx + 1 hold 0, 1), for the kernels that read them in place of the wrap.
template <class T> __global__ void ghost_kernel(T* __restrict__ s, Geom g)
{
    const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= 36LL * g.ny) return;
    const int k = (int)(q & 3);
    const long long row = q >> 2;
    const int i = (int)(row / g.ny), y = (int)(row - (long long)i * g.ny);
    T* r = s + i * g.ps + (long long)y * g.rs + g.off;
    const int to = k < 2 ? k - 2 : g.nx + k - 2;
    r[to] = r[k < 2 ? to + g.nx : to - g.nx];
}

// After the last cascade pass of a call: the ghost columns of storage types
// that have them (FP16).
hipError_t launch_ghosts(int dtype, void* s, const Geom& g, hipStream_t st)
{
    if (dtype != 3) return hipSuccess;
    hipLaunchKernelGGL(ghost_kernel<_Float16>, dim3((unsigned)((36LL * g.ny + 255) / 256)), dim3(256), 0, st,
                       (_Float16*)s, g);
    return hipGetLastError();
}

// MW: waves per SIMD the registers are held to.
template <class T, bool SHIFT, int VX, int NS, int MW, bool FIELD>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(MW, MW))) void cascade_kernel(StepTile a, int ntiles)
{
    constexpr bool RC = ModelCentred<typename CompT<T>::type>::value;
    constexpr int es = sizeof(T), W = cascade_cols(VX, NS, es), HL = cascade_halo_lanes(VX, NS, es);
    const int t = xcd_tile(blockIdx.x, gridDim.x, a.xcd_chunk);
    if (t >= ntiles) return;
    const int strip = t % a.nstrips, chunk = t / a.nstrips;
    const int x0 = strip * W - HL * VX;  // the strip's window
    if (x0 - 1 < 0 || x0 + 64 * VX + 1 > a.g.nx)
        cascade_tile<T, SHIFT, VX, NS, FIELD, RC, true>(a, a.src, a.dst, strip, chunk);
    else
        cascade_tile<T, SHIFT, VX, NS, FIELD, RC, false>(a, a.src, a.dst, strip, chunk);
}

// Batched form: pass p of every lattice of a batch (BatchLat in internal.h,
// with nsteps counting cascade passes and t0 the buffer time at the first);
// one wave per item, an item being one strip of one chunk, dealt to the XCDs
// four at a time (neighbouring strips share their halo's lines in an L2; one
// run per XCD and single items measured within 2 % of it).
template <class T, bool SHIFT, int VX, int NS, int MW>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(MW, MW))) void batch_cascade_kernel(
    const BatchLat* __restrict__ lats, const int* __restrict__ item_lat, int nitems, int p)
{
    constexpr bool RC = ModelCentred<typename CompT<T>::type>::value;
    constexpr int es = sizeof(T), W = cascade_cols(VX, NS, es), HL = cascade_halo_lanes(VX, NS, es);
    const int i = xcd_tile(blockIdx.x, gridDim.x, 4);
    if (i >= nitems) return;
    const BatchLat& L = lats[item_lat[i]];
    if (p >= L.nsteps) return;
    const bool odd = ((L.t0 + p) & 1) != 0;
    const void* src = odd ? L.tile.dst : L.tile.src;
    void* dst = odd ? const_cast<void*>(L.tile.src) : L.tile.dst;
    const int t = i - L.item_begin;
    const int strip = t % L.tile.nstrips, chunk = t / L.tile.nstrips;
    const int x0 = strip * W - HL * VX;
    if (x0 - 1 < 0 || x0 + 64 * VX + 1 > L.tile.g.nx)
        cascade_tile<T, SHIFT, VX, NS, false, RC, true>(L.tile, src, dst, strip, chunk);
    else
        cascade_tile<T, SHIFT, VX, NS, false, RC, false>(L.tile, src, dst, strip, chunk);
}

// The time a row takes on MI355X, in us: `alone` for a wave that has its
// SIMD to itself (the latency of the four levels' chain), `shared` per wave
// where several share one (instruction issue); waves: per SIMD that the
// registers allow.
struct CascadeCost {
    int dtype, vx, waves;
    double alone, shared;
};
static const CascadeCost kCosts[] = {{0, 1, 2, 1.25, 1.10}, {1, 1, 3, 0.85, 0.62}, {1, 2, 2, 1.45, 1.20},
                                     {2, 1, 3, 0.72, 0.55}, {2, 2, 2, 1.25, 1.05}, {3, 2, 3, 1.70, 1.25}};
constexpr int kSimds = 1024;

// Which shape, if any. A chunk of h rows takes h + 14 rows of work, so
// few tall chunks waste least, but the GPU needs a wave on each of its 1024
// SIMDs, and the last wave of an uneven count runs alone. The estimate counts
// both with the times of CascadeCost, from fits over 14 lattice sizes of 64^2
// to 4099 x 2731 (within 10 % there), with a floor for
// the memory traffic. The two-step kernel takes t0 + t1 per million sites
// and step. Measured at the crossing (FP32, us per step, two-step against
// cascade): 512^2 4.5 and 4.9, 700^2 6.5 and 6.1, 1000 x 777 8.9 and 7.1,
// 2048^2 33.3 and 22.1; FP64: 512^2 6.2 and 7.3, 700^2 10.5 and 8.3; FP16
// 2048^2 21.6 and 23.5, 4099 x 2731 69.9 and 42.9.
CascadeShape cascade_shape(int dtype, int nx, int ny)
{
    static const double two_step[4][2] = {{2.4, 14.9}, {2.6, 7.4}, {2.6, 7.4}, {2.8, 4.7}};
    constexpr int warm = 2 * cascade_halo(kCascadeSteps);
    const int es = dtype == 0 ? 8 : (dtype == 3 ? 2 : 4);
    const double sites = (double)nx * ny;
    // 18 planes of the state pass the caches at 5.2 bytes per ps from HBM;
    // a state that fits the 256 MB last-level cache moves about twice as fast
    const double bytes_per_us = sites * 18 * es > 2.0e8 ? 5.2e6 : 1.0e7;
    CascadeShape best;
    double t_best = kCascadeSteps * (two_step[dtype][0] + two_step[dtype][1] * sites * 1e-6);
    for (const CascadeCost& c : kCosts) {
        if (c.dtype != dtype) continue;
        const int w = cascade_cols(c.vx, kCascadeSteps, es), strips = (nx + w - 1) / w;
        for (int h = 6; h < ny + 4 && h < 256; h += 4) {
            const int chunks = (ny + h - 1) / h;
            const double waves = (double)strips * chunks, slots = (double)kSimds * c.waves;
            const int rounds = (int)(waves / slots);
            const int left = (int)((waves - rounds * slots + kSimds - 1) / kSimds);
            const double full = c.waves * c.shared > c.alone ? c.waves * c.shared : c.alone;
            const double last = left == 0 ? 0 : (left * c.shared > c.alone ? left * c.shared : c.alone);
            const double work = 1.0 + (h + warm) * (rounds * full + last);
            const double bytes = 9.0 * es * nx * (1.15 * chunks * (h + warm) + ny);
            const double t = work > bytes / bytes_per_us ? work : bytes / bytes_per_us;
            if (t < t_best) {
                t_best = t;
                best.vx = c.vx;
                best.h = h;
            }
        }
    }
    return best;
}

// The same for a batch, with the times and the two-step kernel's measured on
// pools of 4 to 50 lattices of 0.09 to 24 M sites: a row takes longer there
// (more strips are edges). Two-step against cascade, us per step: FP32 0.34 M
// sites 7.3 and 6.6, 0.74 M 10.4 and 8.4, 11.4 M 108.6 and 56.4, 24.5 M 207
// and 110; FP64 0.34 M 9.1 and 9.0, 2.3 M 45.0 and 23.4, 11.4 M 184 and 98.
CascadeShape cascade_batch_shape(int dtype, const int* nx, const int* ny, int count)
{
    static const CascadeCost costs[] = {{0, 1, 2, 1.35, 1.10}, {1, 1, 3, 1.00, 0.66}, {1, 2, 2, 1.55, 1.25},
                                        {2, 1, 3, 0.85, 0.58}, {2, 2, 2, 1.35, 1.10}};
    static const double two_step[3][2] = {{3.5, 16.0}, {4.2, 9.0}, {4.2, 9.0}};
    static const int heights[] = {6, 10, 14, 18, 22, 26, 34, 42, 50, 58, 74, 90, 130};
    constexpr int warm = 2 * cascade_halo(kCascadeSteps);
    CascadeShape best;
    if (dtype == 3) return best;
    const int es = dtype == 0 ? 8 : 4;
    double sites = 0;
    for (int k = 0; k < count; ++k) sites += (double)nx[k] * ny[k];
    const double bytes_per_us = sites * 18 * es > 2.0e8 ? 5.2e6 : 1.0e7;
    // near a tie the two-step kernel, whose tiles are smaller
    double t_best = 0.96 * kCascadeSteps * (two_step[dtype][0] + two_step[dtype][1] * sites * 1e-6);
    for (const CascadeCost& c : costs) {
        if (c.dtype != dtype) continue;
        const int w = cascade_cols(c.vx, kCascadeSteps, es);
        for (const int h : heights) {
            double waves = 0;
            for (int k = 0; k < count; ++k) waves += (double)((nx[k] + w - 1) / w) * ((ny[k] + h - 1) / h);
            const double slots = (double)kSimds * c.waves;
            const int rounds = (int)(waves / slots);
            const int left = (int)((waves - rounds * slots + kSimds - 1) / kSimds);
            const double full = c.waves * c.shared > c.alone ? c.waves * c.shared : c.alone;
            const double last = left == 0 ? 0 : (left * c.shared > c.alone ? left * c.shared : c.alone);
            const double work = 2.0 + (h + warm) * (rounds * full + last);
            const double bytes = 9.0 * es * sites * (1.15 * (h + warm) / h + 1);
            const double t = work > bytes / bytes_per_us ? work : bytes / bytes_per_us;
            if (t < t_best) {
                t_best = t;
                best.vx = c.vx;
                best.h = h;
            }
        }
    }
    return best;
}

template <class T, bool SHIFT, int VX, int MW>
static hipError_t launch_batch_cascade_t(const BatchLat* lats, const int* item_lat, int nitems, int p, hipStream_t st)
{
    const int grid = (nitems + 31) / 32 * 32;
    if (nitems <= 0) return hipSuccess;
    if (!grid_fits(grid, 64)) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((batch_cascade_kernel<T, SHIFT, VX, kCascadeSteps, MW>), dim3(grid), dim3(64), 0, st, lats,
                       item_lat, nitems, p);
    return hipGetLastError();
}

hipError_t launch_batch_cascade(int dtype, int vx, const BatchLat* lats, const int* item_lat, int nitems, int p,
                                hipStream_t st)
{
    switch (dtype * 8 + vx) {
    case 0 * 8 + 1: return launch_batch_cascade_t<double, false, 1, 2>(lats, item_lat, nitems, p, st);
    case 1 * 8 + 1: return launch_batch_cascade_t<float, false, 1, 3>(lats, item_lat, nitems, p, st);
    case 1 * 8 + 2: return launch_batch_cascade_t<float, false, 2, 2>(lats, item_lat, nitems, p, st);
    case 2 * 8 + 1: return launch_batch_cascade_t<float, true, 1, 3>(lats, item_lat, nitems, p, st);
    case 2 * 8 + 2: return launch_batch_cascade_t<float, true, 2, 2>(lats, item_lat, nitems, p, st);
    }
    return hipErrorInvalidValue;
}

template <class T, bool SHIFT, int VX, int MW> static hipError_t launch_cascade_t(const StepTile& t, hipStream_t st)
{
    const int ntiles = t.nstrips * t.nchunks;
    const int q = t.xcd_chunk > 0 ? 8 * t.xcd_chunk : 8;
    const int grid = (ntiles + q - 1) / q * q;
    if (!grid_fits(grid, 64)) return hipErrorInvalidConfiguration;
    if (t.field)
        hipLaunchKernelGGL((cascade_kernel<T, SHIFT, VX, kCascadeSteps, MW, true>), dim3(grid), dim3(64), 0, st, t, ntiles);
    else
        hipLaunchKernelGGL((cascade_kernel<T, SHIFT, VX, kCascadeSteps, MW, false>), dim3(grid), dim3(64), 0, st, t, ntiles);
    return hipGetLastError();
}

// vx: 1 or 2 columns per lane for 4-byte storage, 1 for FP64, 2 for FP16.
hipError_t launch_cascade(int dtype, int vx, const StepTile& t, hipStream_t st)
{
    switch (dtype * 8 + vx) {
    case 0 * 8 + 1: return launch_cascade_t<double, false, 1, 2>(t, st);
    case 1 * 8 + 1: return launch_cascade_t<float, false, 1, 3>(t, st);
    case 1 * 8 + 2: return launch_cascade_t<float, false, 2, 2>(t, st);
    case 2 * 8 + 1: return launch_cascade_t<float, true, 1, 3>(t, st);
    case 2 * 8 + 2: return launch_cascade_t<float, true, 2, 2>(t, st);
    case 3 * 8 + 2: return launch_cascade_t<_Float16, true, 2, 3>(t, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace lbm
