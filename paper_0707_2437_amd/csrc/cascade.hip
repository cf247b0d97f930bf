// cascade.hip -- several steps of the variable-speed-of-sound D2Q9 step (Buick
// & Cosgrove, Sec. 3 Eq. 5) per pass over memory, held in registers.
//
// A team of four waves owns a strip of 64 * VX columns and walks down a chunk
// of rows. A row enters at level 0 from memory and falls through NS levels,
// one step of Eq. 5 each; what leaves the last level is written. Level s
// works two rows behind level s - 1: it relaxes a row as soon as the density
// of the row below it is known, and hands the nine results, rounded to the
// storage type, to level s + 1, which gathers a row from the results of
// three consecutive rows (the planes with e_iy = 1 of the first, 0 of the
// second, -1 of the third). Each wave holds NL = NS / 4 levels; a row goes
// from wave to wave through two LDS slots, with one barrier per row. Per level
// a wave keeps the populations of one row, two rows of densities and the
// planes' rows that are still waited for; x-neighbours come from the neighbour
// lanes (DPP wave shifts). Every site's arithmetic is the single-step code of
// step.h on the values a single step would load, so a pass gives the bits of
// NS single steps.
//
// Bound: one load and one store of the state per NS steps, against 59
// operations per site and step (77 with the FP32 form's conversions, 80 with
// the lane shifts), and the halo: 2 NS - 1 columns at each side of a strip
// and as many rows before a chunk. FP32 at 4096^2, eight steps: 467 us per
// pass, of which the instructions (halo included) need 415 and the bare
// access pattern 262. With four steps the access pattern bounds the pass (280
// us), so large lattices take eight; FP16 moves half the bytes and stays at
// four. All levels in one wave, without LDS, was the form before: its
// registers (250) allow two waves per SIMD and chunks have to be a quarter as
// high to fill the GPU, so that the halo rows weigh four times as much.
// Measured per step, two-step kernel / one wave / team: FP32 4096^2 121.7 /
// 68.9 / 58.4 us, FP32S 121 / 71.7 / 50.3, FP64 240.5 / 127.7 / 103.5, FP16
// 8192^2 389 / 217 / 183, FP32 1000 x 777 8.9 / 7.2 / 5.85, with a c2 field
// 9.2 / 8.6 / 6.2. A team of eight waves of one level each (before the rows
// moved as aligned vectors): 61.1 us FP32 against 59.6, 53.5 FP32S against
// 50.1, 112.2 FP64 against 111.6.
#include <hip/hip_runtime.h>

#include "cascade.h"
#include "dpp.h"
#include "grid_sync.h"
#include "host.h"
#include "internal.h"
#include "step.h"
#include "xbc.h"

namespace lbm {

// The lane's VX columns of one plane's row as the levels hold them. FP32 and
// FP64: d_i in compute precision.
template <class T, bool SHIFT, int VX> struct CascadeRow {
    using C = typename CompT<T>::type;
    using Mem = Pack<T, VX>;  // as loaded and stored
    static __device__ __forceinline__ T get(const Mem& p, int j) { return p.v[j]; }
    template <int J> static __device__ __forceinline__ void put(Mem& p, T v) { p.v[J] = v; }
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
    // The results of column J (a) and of the next (b), rounded to the storage
    // type.
    template <int J>
    static __device__ __forceinline__ void store(const C (&a)[9], const C (&b)[9], Mem (&f)[9], const Centre<C>& cn)
    {
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            f[i].v[J] = from_d<T, SHIFT, C>(a[i], i, cn);
            f[i].v[J + 1] = from_d<T, SHIFT, C>(b[i], i, cn);
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
    static __device__ __forceinline__ _Float16 get(const Mem& p, int j)
    {
        return __builtin_bit_cast(_Float16, (unsigned short)(p.q[j >> 1] >> (16 * (j & 1))));
    }
    template <int J> static __device__ __forceinline__ void put(Mem& p, _Float16 v)
    {
        const unsigned h = (unsigned)__builtin_bit_cast(unsigned short, v);
        p.q[J / 2] = J & 1 ? (p.q[J / 2] & 0xffffu) | h << 16 : (p.q[J / 2] & 0xffff0000u) | h;
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
    template <int J>
    static __device__ __forceinline__ void store(const float (&a)[9], const float (&b)[9], Mem (&f)[9],
                                                 const Centre<float>&)
    {
#pragma unroll
        for (int i = 0; i < 9; ++i) f[i].q[J / 2] = pack_h2(a[i], b[i]);
    }
};

// A row's columns of a lane in LDS, as one aligned vector: as a struct of
// 4-byte alignment they move in halves, with four bank conflicts each.
template <int BYTES> struct CascadeLds {
    typedef unsigned type __attribute__((ext_vector_type(BYTES / 4)));
};

// Stands for XbcValues where the lattice is periodic in x.
struct CascadePeriodic {};

// One level's state between rows: the row it relaxes next (populations d,
// densities w), the densities of the row above it (wp), and the planes of
// its last results that wait for rows below: e_iy = 0 of the last row (z),
// e_iy = 1 of the last two (up, by the row's parity).
template <class R> struct CascadeWait {
    R z[3], up[2][3];
};
template <class R, class C, int VX> struct CascadeLevel {
    R d[9];
    C w[VX], wp[VX];
    CascadeWait<R> h;
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
    } else if constexpr (sizeof(V) == 8) {
        typedef unsigned u2 __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), rs, voff, soff, aux);
    } else {
        static_assert(sizeof(V) == 16, "rows of up to four dwords per lane");
        typedef unsigned u4 __attribute__((ext_vector_type(4)));
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, v), rs, voff, soff, aux);
    }
}

// One wave's part of a tile (w: its place in the team; FIRST reads memory, LAST
// writes it, in and outq are the LDS slots between): NS steps of rows
// [chunk a.h, (chunk + 1) a.h) and the strip's inner columns. EDGE: a strip whose window reaches past the lattice's left
// or right edge; its lanes load every element from its wrapped column
// (Sec. 4: periodic in x) and store element by element.
template <class T, bool SHIFT, int VX, int NL, bool FIRST, bool LAST, bool FIELD, bool RC, bool EDGE, class Tile, class XB>
__device__ __forceinline__ void cascade_tile(const Tile& a, const void* src, void* dst, int strip, int chunk,
                                             [[maybe_unused]] typename CascadeLds<sizeof(T) * VX>::type (*in)[9][64],
                                             [[maybe_unused]] typename CascadeLds<sizeof(T) * VX>::type (*outq)[9][64],
                                             int w, [[maybe_unused]] const XB& xb)
{
    using C = typename CompT<T>::type;
    using R = CascadeRow<T, SHIFT, VX>;
    using Mem = typename R::Mem;
    // only a strip whose window reaches past an edge holds columns 0 and nx - 1
    constexpr bool XBC = EDGE && !std::is_same<XB, CascadePeriodic>::value;
    constexpr int NW = kCascadeWaves, NS = NL * NW;
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
    int fr[NL];
    Pack<C, VX> af[NL] = {};
    auto load_field = [&]() {
        if constexpr (FIELD) {
#pragma unroll
            for (int s = 0; s < NL; ++s) {
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
        for (int s = 0; s < NL; ++s) fr[s] = wrap(ylo - H - 1 - 2 * (w * NL + s));

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

    CascadeLevel<R, C, VX> L[NL] = {};
    [[maybe_unused]] CascadeWait<R> gate = {};
    [[maybe_unused]] Mem raw[9];
    if constexpr (FIRST) load(raw);
    load_field();
    if constexpr (LAST) {
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
    // The next level's row, gathered from the results q of this row and the
    // two before it.
    auto gather = [&](auto parity, CascadeWait<R>& h, const R (&q)[9], R (&nd)[9]) {
        constexpr int P = decltype(parity)::value;
        nd[0] = h.z[0];
        nd[1] = h.z[1].template shifted<1>();
        nd[3] = h.z[2].template shifted<-1>();
        nd[2] = h.up[P][0];
        nd[5] = h.up[P][1].template shifted<1>();
        nd[6] = h.up[P][2].template shifted<-1>();
        nd[4] = q[4];
        nd[7] = q[7].template shifted<-1>();
        nd[8] = q[8].template shifted<1>();
        h.z[0] = q[0];
        h.z[1] = q[1];
        h.z[2] = q[3];
        h.up[P][0] = q[2];
        h.up[P][1] = q[5];
        h.up[P][2] = q[6];
    };
    auto meet = [&]() {
        // LDS only: a full fence would wait for the next row's loads too
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };
    // The kk-th row enters; P: its parity.
    auto iterate = [&](int kk, auto parity) {
        constexpr int P = decltype(parity)::value;
        R nd[9];
        if constexpr (FIRST) {
            land(raw, nd);
        } else {
            Mem m[9];
            static_for<0, 9>([&](auto ic) { m[decltype(ic)::value] = __builtin_bit_cast(Mem, in[P][decltype(ic)::value][lane]); });
            R q[9];
            land(m, q);
            gather(parity, gate, q, nd);
        }
        Pack<C, VX> fa[NL];
        static_for<0, NL>([&](auto sc) { fa[decltype(sc)::value] = af[decltype(sc)::value]; });
        if (FIRST && kk + 1 < niter) {
            rm = r0;
            r0 = rp;
            rp = next(rp);
        }
        if constexpr (FIELD)
#pragma unroll
            for (int s = 0; s < NL; ++s) fr[s] = next(fr[s]);
        if constexpr (FIRST) load(raw);
        load_field();
        __builtin_amdgcn_sched_barrier(0);  // the loads first, then the arithmetic they overlap with
        static_for<0, NL>([&](auto sc) {
            constexpr int s = decltype(sc)::value;
            auto& l = L[s];
            C nw[VX];
            static_for<0, VX>([&](auto jc) { nw[decltype(jc)::value] = drho_col(R::template col<decltype(jc)::value>(nd)); });
            // relax the held row, its neighbour rows' densities known
            const C wl = from_left(l.w[VX - 1]), wr = from_right(l.w[0]);
            Mem f[9];
            constexpr int G = 2;  // columns at a time (registers)
            static_assert(VX % G == 0, "pairs of columns");
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
                relax(std::integral_constant<int, J + 1>{}, ob);
                R::template store<J>(oa, ob, f, cn);
                // columns, and levels, one after the other: interleaved they need more registers
                __builtin_amdgcn_sched_barrier(0);
            });
            if constexpr (XBC) {
                static_for<0, VX>([&](auto jc) {
                    constexpr int j = decltype(jc)::value;
                    const int xw = (int)(off[j + 1] / es) - 2;
                    static_for<0, 9>([&](auto ic) {
                        constexpr int i = decltype(ic)::value;
                        R::template put<j>(f[i], xbc_value<T>(xb, w * NL + s, i, ex[i], xw, g.nx, R::get(f[i], j)));
                    });
                });
            }
#pragma unroll
            for (int j = 0; j < VX; ++j) {
                l.wp[j] = l.w[j];
                l.w[j] = nw[j];
            }
            static_for<0, 9>([&](auto ic) { l.d[decltype(ic)::value] = nd[decltype(ic)::value]; });
            if constexpr (s + 1 < NL) {
                R q[9];
                land(f, q);
                gather(parity, l.h, q, nd);
            } else if constexpr (LAST) {
                write(kk, f);
            } else {
                using Lds = typename CascadeLds<sizeof(Mem)>::type;
                static_for<0, 9>([&](auto ic) {
                    outq[P][decltype(ic)::value][lane] = __builtin_bit_cast(Lds, f[decltype(ic)::value]);
                });
            }
        });
        meet();
    };
    // Four rows per turn: a value lives for up to four rows in a level's
    // state, and with a shorter turn its registers would be copied.
    for (int k = 0; k < w; ++k) meet();
    for (int kk = 0; kk < niter; kk += 4)
        static_for<0, 4>([&](auto u) {
            iterate(kk + decltype(u)::value, std::integral_constant<int, decltype(u)::value % 2>{});
        });
    for (int k = w + 1; k < NW; ++k) meet();
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

// Between the waves of a team: the last two rows each hands to the next.
template <class T, bool SHIFT, int VX> struct CascadeRing {
    typename CascadeLds<sizeof(T) * VX>::type row[kCascadeWaves - 1][2][9][64];
};

// One wave of a team. The waves pass the same number of barriers: a wave's
// first row is one barrier behind that of the wave before it.
template <class T, bool SHIFT, int VX, int NL, bool FIELD, bool RC, bool EDGE, class Tile, class XB>
__device__ __forceinline__ void cascade_wave(const Tile& a, const void* src, void* dst, int strip, int chunk,
                                             CascadeRing<T, SHIFT, VX>& ring, const XB& xb)
{
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (w == 0)
        cascade_tile<T, SHIFT, VX, NL, true, false, FIELD, RC, EDGE>(a, src, dst, strip, chunk, nullptr, ring.row[0], 0, xb);
    else if (w == kCascadeWaves - 1)
        cascade_tile<T, SHIFT, VX, NL, false, true, FIELD, RC, EDGE>(a, src, dst, strip, chunk, ring.row[w - 1], nullptr, w,
                                                                    xb);
    else
        cascade_tile<T, SHIFT, VX, NL, false, false, FIELD, RC, EDGE>(a, src, dst, strip, chunk, ring.row[w - 1],
                                                                      ring.row[w], w, xb);
}

// MW: waves per SIMD the registers are held to.
template <class T, bool SHIFT, int VX, int NL, int MW, bool FIELD, class XB>
__global__ __launch_bounds__(64 * kCascadeWaves) __attribute__((amdgpu_waves_per_eu(MW, MW))) void cascade_kernel(
    StepTile a, int ntiles, XB xb)
{
    constexpr bool RC = ModelCentred<typename CompT<T>::type>::value;
    constexpr int es = sizeof(T), NS = NL * kCascadeWaves, W = cascade_cols(VX, NS, es),
                  HL = cascade_halo_lanes(VX, NS, es);
    __shared__ CascadeRing<T, SHIFT, VX> ring;
    const int t = xcd_tile(blockIdx.x, gridDim.x, a.xcd_chunk);
    if (t >= ntiles) return;
    const int strip = t % a.nstrips, chunk = t / a.nstrips;
    const int x0 = strip * W - HL * VX;  // the strip's window
    if (x0 - 1 < 0 || x0 + 64 * VX + 1 > a.g.nx)
        cascade_wave<T, SHIFT, VX, NL, FIELD, RC, true>(a, a.src, a.dst, strip, chunk, ring, xb);
    else
        cascade_wave<T, SHIFT, VX, NL, FIELD, RC, false>(a, a.src, a.dst, strip, chunk, ring, xb);
}

// Batched form: pass p of every lattice of a batch (BatchLat in internal.h,
// with nsteps counting cascade passes and t0 the buffer time at the first);
// one team per item, an item being one strip of one chunk, dealt to the XCDs
// four at a time (neighbouring strips share their halo's lines in an L2; one
// run per XCD and single items measured within 2 % of it).
template <class T, bool SHIFT, int VX, int NL, int MW>
__global__ __launch_bounds__(64 * kCascadeWaves) __attribute__((amdgpu_waves_per_eu(MW, MW))) void batch_cascade_kernel(
    const BatchLat* __restrict__ lats, const int* __restrict__ item_lat, int nitems, int p)
{
    constexpr bool RC = ModelCentred<typename CompT<T>::type>::value;
    constexpr int es = sizeof(T), NS = NL * kCascadeWaves, W = cascade_cols(VX, NS, es),
                  HL = cascade_halo_lanes(VX, NS, es);
    __shared__ CascadeRing<T, SHIFT, VX> ring;
    const int i = xcd_tile(blockIdx.x, gridDim.x, 4);
    if (i >= nitems) return;
    const BatchLat& L = lats[item_lat[i]];
    if (p >= L.nsteps) return;
    const bool odd = ((L.t0 + p) & 1) != 0;
    const void* src = odd ? L.tile.dst : L.tile.src;
    void* dst = odd ? const_cast<void*>(L.tile.src) : L.tile.dst;
    const BatchTile& a = L.tile;
    const int t = i - L.item_begin;
    const int strip = t % a.nstrips, chunk = t / a.nstrips;
    const int x0 = strip * W - HL * VX;
    if (x0 - 1 < 0 || x0 + 64 * VX + 1 > a.g.nx)
        cascade_wave<T, SHIFT, VX, NL, false, RC, true>(a, src, dst, strip, chunk, ring, CascadePeriodic{});
    else
        cascade_wave<T, SHIFT, VX, NL, false, RC, false>(a, src, dst, strip, chunk, ring, CascadePeriodic{});
}

// Persistent form: all npasses passes of a batch in one launch, members and
// work dealt out as in the two-step kernel's persistent form (step2.hip).
// Against that form, us per step: FP32 0.33 M sites 56.2 and 23.9, 2.7 M 76 and
// 42, 8.8 M 135 and 71; FP64 57.7 and 18.0, 110 and 51, 239 and 101.
template <class T, bool SHIFT, int VX, int NL, int MW>
__global__ __launch_bounds__(64 * kCascadeWaves) __attribute__((amdgpu_waves_per_eu(MW, MW))) void
batch_persistent_cascade_kernel(const BatchLat* __restrict__ lats, const int* __restrict__ item_lat, int nitems,
                                int npasses, int ch, unsigned* bar, unsigned long long wait_ticks,
                                unsigned long long grace_ticks)
{
    constexpr bool RC = ModelCentred<typename CompT<T>::type>::value;
    constexpr int es = sizeof(T), NS = NL * kCascadeWaves, W = cascade_cols(VX, NS, es),
                  HL = cascade_halo_lanes(VX, NS, es);
    __shared__ CascadeRing<T, SHIFT, VX> ring;
    __shared__ int next_item;
    if (stale_barrier_error(bar)) return;
    int rank = 0;
    const int G = join_members(bar, wait_ticks, grace_ticks, &rank);
    if (G == 0) return;
    const bool by_xcd = G == (int)gridDim.x && G % 8 == 0;
    const int nparts = by_xcd ? 8 : 1;
    const int part = by_xcd ? (int)(blockIdx.x & 7u) : 0;
    const int chunk = ch > 0 ? ch : 1;
    for (int p = 0; p < npasses; ++p) {
        unsigned* ctr = bar + kBarCtr + (p & 1) * 8 + part;
        for (;;) {
            if (threadIdx.x == 0) next_item = min(part_item((int)atomicAdd(ctr, 1u), part, nparts, chunk), nitems);
            __syncthreads();
            const int i = __builtin_amdgcn_readfirstlane(next_item);
            __syncthreads();  // read by every wave before the next item is written; ring free again
            if (i >= nitems) break;
            const BatchLat* L = &lats[ldc(&item_lat[i])];
            if (p >= ldc(&L->nsteps)) continue;  // this lattice takes fewer passes
            const BatchTile a = ldc(&L->tile);
            const bool odd = ((ldc(&L->t0) + p) & 1) != 0;
            const void* src = odd ? a.dst : a.src;
            void* dst = odd ? const_cast<void*>(a.src) : a.dst;
            const int t = i - ldc(&L->item_begin);
            const int strip = t % a.nstrips, row = t / a.nstrips;
            const int x0 = strip * W - HL * VX;
            if (x0 - 1 < 0 || x0 + 64 * VX + 1 > a.g.nx)
                cascade_wave<T, SHIFT, VX, NL, false, RC, true>(a, src, dst, strip, row, ring, CascadePeriodic{});
            else
                cascade_wave<T, SHIFT, VX, NL, false, RC, false>(a, src, dst, strip, row, ring, CascadePeriodic{});
        }
        if (!grid_barrier(bar, G, wait_ticks, bar + kBarCtr + ((p + 1) & 1) * 8, p + 1 < npasses ? 8 : 0)) return;
    }
}

// The time a team takes per row on MI355X, in us, with one, two ... teams on
// its CU (of as many as registers and LDS allow), from fits over lattices of
// 400^2 to 4096^2 (within 10 % there).
struct CascadeCost {
    int dtype, levels, teams;
    double row[4];
};
static const CascadeCost kCosts[] = {
    {0, 1, 2, {0.78, 1.08}},       {0, 2, 1, {1.12}},
    {1, 1, 4, {0.60, 0.72, 1.07, 1.39}}, {1, 2, 3, {0.82, 1.19, 1.75}},
    {2, 1, 4, {0.53, 0.62, 1.00, 1.32}}, {2, 2, 3, {0.70, 1.03, 1.46}},
    {3, 1, 3, {1.15, 1.40, 1.71}}};
constexpr int kCus = 256;

// A pass of `teams` teams of h rows: they fill the CUs in rounds, the last of
// which holds fewer per CU.
static double cascade_time(const CascadeCost& c, double teams, int h)
{
    const double slots = (double)kCus * c.teams;
    const int rounds = (int)(teams / slots);
    const int left = (int)((teams - rounds * slots + kCus - 1) / kCus);
    const int rows = h + 2 * cascade_halo(c.levels * kCascadeWaves) + kCascadeWaves - 1;
    return rows * (rounds * c.row[c.teams - 1] + (left ? c.row[left - 1] : 0.0));
}

// 18 planes of the state pass the caches at 5.2 bytes per ps from HBM; a state
// that fits the 256 MB last-level cache is not bound by it.
static double cascade_bytes_per_us(double state_bytes) { return state_bytes > 2.0e8 ? 5.2e6 : 1.0e7; }

// Few tall chunks waste least on the halo, but the GPU needs a team on each
// of its 256 CUs, and the last round of an uneven count runs half empty. The
// estimate counts both, with a floor for the memory traffic. The two-step
// kernel takes t0 + t1 per million sites and step. Measured, us per step,
// two-step against four-step passes: FP32 400^2 4.1 and 4.5, 512^2 4.5 and
// 4.8, 700^2 6.5 and 5.4, 1000 x 777 8.9 and 6.5; FP64 512^2 6.2 and 6.3, 700^2
// 10.5 and 8.0. Four-step against eight-step: FP32 1000 x 777 6.5 and 7.6,
// 2048^2 21.4 and 19.3, 4096^2 70.0 and 59.6; FP64 1000 x 777 10.5 and 10.8,
// 2048^2 34.6 and 35.9, 4096^2 123.8 and 111.6. With an inlet, single steps and
// a boundary launch after each against passes: FP32 700^2 13.3 and 5.8, 4096^2
// 209.7 and 64.6; FP64 4096^2 422 and 120; FP16 1400^2 23.5 and 15.1.
void cascade_shapes(int dtype, int nx, int ny, bool inlet, CascadeShape out[2])
{
    static const double two_step[4][2] = {{2.4, 14.9}, {2.6, 7.4}, {2.6, 7.4}, {2.8, 4.7}};
    const int es = dtype == 0 ? 8 : (dtype == 3 ? 2 : 4);
    const double sites = (double)nx * ny, per_us = cascade_bytes_per_us(sites * 18 * es);
    // FP16 strips at an edge load and store two bytes at a time and take half as
    // long again: with tall chunks they end alone (8192^2, us per step: 394
    // rows 211, 194 rows 202, 130 rows 185)
    const int most = dtype == 3 ? 160 : 400;
    // us per step of the best so far; with an inlet, single steps and a launch
    // for the boundary after each
    double t_best = inlet ? 4.5 + 2.3 * es * sites * 1e-6 : two_step[dtype][0] + two_step[dtype][1] * sites * 1e-6;
    for (int levels = 1; levels <= 2; ++levels) {
        out[levels - 1] = CascadeShape();
        const int ns = levels * kCascadeWaves, warm = 2 * cascade_halo(ns);
        for (const CascadeCost& c : kCosts) {
            if (c.dtype != dtype || c.levels != levels) continue;
            if (c.row[0] * (6 + warm) / ns >= t_best) continue;  // slower with every height (saves the search)
            const int w = cascade_cols(cascade_vx(dtype), ns, es), strips = (nx + w - 1) / w;
            for (int h = 6; h < ny + 4 && h < most; h += 4) {
                const int chunks = (ny + h - 1) / h;
                const double work = 1.0 + cascade_time(c, (double)strips * chunks, h);
                const double bytes = 9.0 * es * nx * (1.15 * chunks * (h + warm) + ny);
                const double t = (work > bytes / per_us ? work : bytes / per_us) / ns;
                if (t < t_best) {
                    t_best = t;
                    out[levels - 1] = {levels, h};
                }
            }
        }
    }
}

// The four-step shape of a batch of lattices. Measured on pools of 4 to 60
// lattices, two-step against four-step passes, us per step: FP32 0.33 M sites
// 6.4 and 5.8, 0.86 M 11.6 and 6.9, 2.7 M 32.5 and 17.6, 8.8 M 82 and 43; FP64
// 0.33 M 8.2 and 7.4, 0.86 M 17.6 and 10.4, 8.8 M 145 and 75.
CascadeShape cascade_batch_shape(int dtype, const int* nx, const int* ny, int count)
{
    static const double two_step[3][2] = {{3.5, 16.0}, {4.2, 9.0}, {4.2, 9.0}};
    static const int heights[] = {6, 10, 14, 18, 22, 26, 30, 34, 42, 50, 58, 66, 74, 86, 98, 114, 130};
    constexpr int warm = 2 * cascade_halo(kCascadeWaves);
    CascadeShape best;
    if (dtype == 3) return best;
    const int es = dtype == 0 ? 8 : 4, w = cascade_cols(cascade_vx(dtype), kCascadeWaves, es);
    double sites = 0;
    for (int k = 0; k < count; ++k) sites += (double)nx[k] * ny[k];
    const double per_us = cascade_bytes_per_us(sites * 18 * es);
    // near a tie the two-step kernel, whose tiles are smaller
    double t_best = 0.96 * kCascadeWaves * (two_step[dtype][0] + two_step[dtype][1] * sites * 1e-6);
    for (const CascadeCost& c : kCosts) {
        if (c.dtype != dtype || c.levels != 1) continue;
        for (const int h : heights) {
            double teams = 0;
            for (int k = 0; k < count; ++k) teams += (double)((nx[k] + w - 1) / w) * ((ny[k] + h - 1) / h);
            const double work = 2.0 + cascade_time(c, teams, h);
            const double bytes = 9.0 * es * sites * (1.15 * (h + warm) / h + 1);
            const double t = work > bytes / per_us ? work : bytes / per_us;
            if (t < t_best) {
                t_best = t;
                best = {1, h};
            }
        }
    }
    return best;
}

template <class T, bool SHIFT, int MW>
static hipError_t launch_batch_cascade_t(const BatchLat* lats, const int* item_lat, int nitems, int p, hipStream_t st)
{
    const int grid = (nitems + 31) / 32 * 32, threads = 64 * kCascadeWaves;
    if (nitems <= 0) return hipSuccess;
    if (!grid_fits(grid, threads)) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((batch_cascade_kernel<T, SHIFT, 2, 1, MW>), dim3(grid), dim3(threads), 0, st, lats, item_lat,
                       nitems, p);
    return hipGetLastError();
}

hipError_t launch_batch_cascade(int dtype, const BatchLat* lats, const int* item_lat, int nitems, int p, hipStream_t st)
{
    switch (dtype) {
    case 0: return launch_batch_cascade_t<double, false, 2>(lats, item_lat, nitems, p, st);
    case 1: return launch_batch_cascade_t<float, false, 4>(lats, item_lat, nitems, p, st);
    case 2: return launch_batch_cascade_t<float, true, 4>(lats, item_lat, nitems, p, st);
    }
    return hipErrorInvalidValue;
}

template <class T, bool SHIFT, int MW>
static hipError_t launch_batch_cascade_persistent_t(const BatchLat* lats, const int* item_lat, int nitems, int npasses,
                                                    int ch, unsigned* bar, hipStream_t st)
{
    const auto kern = batch_persistent_cascade_kernel<T, SHIFT, 2, 1, MW>;
    constexpr int threads = 64 * kCascadeWaves;
    int grid = 0;
    unsigned long long wait_ticks = 0, grace_ticks = 0;
    // A member costs 0.15 us at each barrier, and two teams per CU reach the
    // rate of four within 5 %: at most two, and no more members than items.
    const int most = 2 * kCus, need = (nitems + 7) / 8 * 8;
    hipError_t e = persistent_setup((const void*)kern, threads, need < most ? need : most, &ch, &grid, &wait_ticks,
                                    &grace_ticks, bar, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(threads), 0, st, lats, item_lat, nitems, npasses, ch, bar, wait_ticks,
                       grace_ticks);
    return hipGetLastError();
}

hipError_t launch_batch_cascade_persistent(int dtype, const BatchLat* lats, const int* item_lat, int nitems,
                                           int npasses, int ch, unsigned* bar, hipStream_t st)
{
    switch (dtype) {
    case 0: return launch_batch_cascade_persistent_t<double, false, 2>(lats, item_lat, nitems, npasses, ch, bar, st);
    case 1: return launch_batch_cascade_persistent_t<float, false, 4>(lats, item_lat, nitems, npasses, ch, bar, st);
    case 2: return launch_batch_cascade_persistent_t<float, true, 4>(lats, item_lat, nitems, npasses, ch, bar, st);
    }
    return hipErrorInvalidValue;
}

template <class T, bool SHIFT, int VX, int NL, int MW, bool FIELD>
static hipError_t launch_cascade_t(const StepTile& t, const PassInlet* inlet, hipStream_t st)
{
    const int ntiles = t.nstrips * t.nchunks, threads = 64 * kCascadeWaves;
    const int q = t.xcd_chunk > 0 ? 8 * t.xcd_chunk : 8;
    const int grid = (ntiles + q - 1) / q * q;
    if (!grid_fits(grid, threads)) return hipErrorInvalidConfiguration;
    if (!inlet) {
        hipLaunchKernelGGL((cascade_kernel<T, SHIFT, VX, NL, MW, FIELD, CascadePeriodic>), dim3(grid), dim3(threads), 0,
                           st, t, ntiles, CascadePeriodic{});
    } else {
        if constexpr (FIELD) return hipErrorInvalidValue;
        else
            hipLaunchKernelGGL((cascade_kernel<T, SHIFT, VX, NL, MW, false, XbcValues<T>>), dim3(grid), dim3(threads), 0,
                               st, t, ntiles, xbc_values<T, SHIFT>(*inlet, NL * kCascadeWaves));
    }
    return hipGetLastError();
}

// levels: per wave; 2 (eight steps per pass) without a c2 field, whose rows
// would take the registers past their limit, and not for FP16. inlet: the
// boundaries in x, or null (periodic); not with a c2 field.
hipError_t launch_cascade(int dtype, int levels, const StepTile& t, const PassInlet* in, hipStream_t st)
{
    switch (dtype * 4 + (t.field ? 2 : 0) + levels - 1) {
    case 0: return launch_cascade_t<double, false, 2, 1, 2, false>(t, in, st);
    case 1: return launch_cascade_t<double, false, 2, 2, 1, false>(t, in, st);
    case 2: return launch_cascade_t<double, false, 2, 1, 2, true>(t, in, st);
    case 4: return launch_cascade_t<float, false, 2, 1, 4, false>(t, in, st);
    case 5: return launch_cascade_t<float, false, 2, 2, 3, false>(t, in, st);
    case 6: return launch_cascade_t<float, false, 2, 1, 4, true>(t, in, st);
    case 8: return launch_cascade_t<float, true, 2, 1, 4, false>(t, in, st);
    case 9: return launch_cascade_t<float, true, 2, 2, 3, false>(t, in, st);
    case 10: return launch_cascade_t<float, true, 2, 1, 4, true>(t, in, st);
    case 12: return launch_cascade_t<_Float16, true, 4, 1, 3, false>(t, in, st);
    case 14: return launch_cascade_t<_Float16, true, 4, 1, 3, true>(t, in, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace lbm
