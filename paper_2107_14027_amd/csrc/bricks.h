// Bricks of elements, their LDS tiles and their lines: what the kernels that
// take an element's lines one per lane share.
#pragma once

#include <algorithm>

#include "fr_device.h"

namespace fr {
namespace dev {

template <int D> struct Dir { static constexpr int value = D; };

// The value is formed here: without it the compiler sinks a sum to where it is
// next used and keeps all of its operands in registers until then.
template <typename T>
__device__ __forceinline__ void pin(T &x)
{
    __asm__ volatile("" : "+v"(x));
}

// nu with the sign of n (a value with that of the unit normal's only entry, 1 or -1,
// on a face of a diagonal Jacobian): the viscous part of the common flux for traces that are S_id
// (trace_value).  On the bits, so that the sign of a kernel argument stays in the
// scalar unit (held as three more arguments, or multiplied, it cost p = 6 in
// double, which is at its register limit, 1.7 % of its residual).
__device__ __forceinline__ double signed_nu(double nu, double n)
{
    const int64_t s = __builtin_bit_cast(int64_t, n) & INT64_MIN;
    return __builtin_bit_cast(double, __builtin_bit_cast(int64_t, nu) ^ s);
}
__device__ __forceinline__ float signed_nu(float nu, float n)
{
    const int32_t s = __builtin_bit_cast(int32_t, n) & INT32_MIN;
    return __builtin_bit_cast(float, __builtin_bit_cast(int32_t, nu) ^ s);
}

// Common normal flux through a face of direction d, evaluated by the element
// on one side: own = its trace, oth = the neighbour's, own_minus = the element
// is on the minus side of the face (its + face).  Equal, bit for bit, to the
// same flux evaluated by the neighbour, because every asymmetric term is
// written as a signed difference oth - own whose sign is carried by an exact
// sign flip of lambda, and every symmetric term is a commutative sum.
//   out[0]     Rusanov dissipation on P, -|n| lambda (P_plus - P_minus) / 2
//   out[1..3]  momentum common flux (times |n_d|)
//   out[4..6]  mean velocity
template <typename T>
__device__ __forceinline__ void common_flux_sided(const T own[NTR], const T oth[NTR], bool own_minus,
                                                  const T nh[3], T nmag, T zeta, T nu, T out[NTR])
{
    T vo = own[1] * nh[0];
    vo = fma(own[2], nh[1], vo);
    vo = fma(own[3], nh[2], vo);
    T vt = oth[1] * nh[0];
    vt = fma(oth[2], nh[1], vt);
    vt = fma(oth[3], nh[2], vt);
    // lambda = max over both sides of |v| + sqrt(v^2 + zeta), evaluated once
    // at the larger |v| (the expression is monotone in |v| after rounding too)
    const T vm = fmax(fabs(vo), fabs(vt));
    const T lam = vm + sqrt(fma(vm, vm, zeta));
    const T hm = T(0.5) * nmag;
    // P_plus - P_minus = (own_minus ? 1 : -1) (P_oth - P_own)
    const T slam = own_minus ? lam : -lam;
    out[0] = (-hm * slam) * (oth[0] - own[0]);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const T fo = fma(own[1 + i], vo, fma(own[0], nh[i], -nu * own[4 + i]));
        const T ft = fma(oth[1 + i], vt, fma(oth[0], nh[i], -nu * oth[4 + i]));
        out[1 + i] = hm * fma(oth[1 + i] - own[1 + i], -slam, fo + ft);
        out[4 + i] = T(0.5) * (own[1 + i] + oth[1 + i]);
    }
}


// The m values of one line (first value p, stride STR) into registers; an
// x-line (STR = 1) is contiguous and is read in 16- or 8-byte vectors where
// its length and the element size keep them aligned.
template <int M, int STR, typename T>
__device__ __forceinline__ void line_load(const T *__restrict__ p, T (&x)[M])
{
    if constexpr (STR == 1 && (M * sizeof(T)) % 16 == 0) {
        using V = typename V16<T>::type;
        constexpr int W = 16 / sizeof(T);
#pragma unroll
        for (int k = 0; k < M / W; ++k) {
            const V v = reinterpret_cast<const V *>(p)[k];
#pragma unroll
            for (int w = 0; w < W; ++w) x[k * W + w] = v[w];
        }
    } else if constexpr (STR == 1 && sizeof(T) == 4 && M % 2 == 0) {
        typedef float f2v __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int k = 0; k < M / 2; ++k) {
            const f2v v = reinterpret_cast<const f2v *>(p)[k];
            x[2 * k] = v[0];
            x[2 * k + 1] = v[1];
        }
    } else {
#pragma unroll
        for (int l = 0; l < M; ++l) x[l] = p[l * STR];
    }
}

// The m values of one line into LDS (the layout of line_load).
template <int M, int STR, typename T>
__device__ __forceinline__ void line_put(T *__restrict__ p, const T (&x)[M])
{
    if constexpr (STR == 1 && (M * sizeof(T)) % 16 == 0) {
        using V = typename V16<T>::type;
        constexpr int W = 16 / sizeof(T);
#pragma unroll
        for (int k = 0; k < M / W; ++k) {
            V v;
#pragma unroll
            for (int w = 0; w < W; ++w) v[w] = x[k * W + w];
            reinterpret_cast<V *>(p)[k] = v;
        }
    } else {
#pragma unroll
        for (int l = 0; l < M; ++l) p[l * STR] = x[l];
    }
}

// First point of the direction-D line through face point L.
template <int P, typename T, int D>
__device__ __forceinline__ int lt_base(int L)
{
    constexpr int M = P + 1;
    const int a = L % M, b = L / M;
    return D == 0 ? M * L : (D == 1 ? a + M * M * b : L);
}

// Bricks of elements for the line forms.  A workgroup takes bx * by * bz
// elements (at most LinesShape::E), neighbours of each other in the lattice, so
// that the faces between them are formed from the tile; bricks at the lattice's
// upper ends may stick out of it (those slots idle).

// Elements of the brick (slot coordinates sx, sy, sz, lattice element e; e < 0:
// slot not in use).
struct BrickSlot {
    int sx, sy, sz, e;
};
__device__ __forceinline__ BrickSlot brick_slot(const Bricks &g, int s, int cx, int cy, int cz,
                                                int nx, int ny, int nz)
{
    BrickSlot r;
    r.sz = (s * g.mxy) >> 16;
    const int q = s - r.sz * (g.bx * g.by);
    r.sy = (q * g.mx) >> 16;
    r.sx = q - r.sy * g.bx;
    const int x = cx + r.sx, y = cy + r.sy, z = cz + r.sz;
    r.e = r.sz < g.bz && x < nx && y < ny && z < nz ? x + nx * (y + ny * z) : -1;
    return r;
}

// The elements of a brick's slots for loops in which a wave goes over the slots:
// worked out once, slot s in lane s of every wave (working them out per step was
// more scalar work than the kernel's arithmetic, 1150 scalar to 790 vector
// instructions a wave at p = 3, and cost 2 to 3 % there).  LANES false: per step
// after all, for one or two slots, where the lane reads cost 1 %.
template <bool LANES>
struct BrickElems {
    const Bricks &g;
    const int cx, cy, cz, nx, ny, nz, e;
    __device__ __forceinline__ BrickElems(const Bricks &g_, int cx_, int cy_, int cz_, int nx_, int ny_, int nz_)
        : g(g_), cx(cx_), cy(cy_), cz(cz_), nx(nx_), ny(ny_), nz(nz_),
          e(LANES ? brick_slot(g_, threadIdx.x & 63, cx_, cy_, cz_, nx_, ny_, nz_).e : 0)
    {
    }
    // of the wave's slot s: negative when not in use
    __device__ __forceinline__ int operator()(int s) const
    {
        return LANES ? __builtin_amdgcn_readlane(e, s) : brick_slot(g, s, cx, cy, cz, nx, ny, nz).e;
    }
};

// Workgroup b's brick, or -1.  Consecutive workgroups go to the eight XCDs in
// turn, each with an L2 of its own.  A group of 8 g.chunk bricks (one layer of
// the lattice along z) is dealt out so that every XCD works on a contiguous
// eighth of it: y neighbours then share an L2, and all XCDs stay on one compact
// front of the lattice, whose last layer the memory-side cache still holds when
// the next one reads its z neighbours.
__device__ __forceinline__ int brick_of(const Bricks &g, unsigned b)
{
    const unsigned first = g.by_group(b) * 8 * g.chunk, r = b - first;
    if (first >= g.nb) return -1;
    const unsigned share = min(g.chunk, (g.nb - first + 7) / 8);
    const unsigned i = r >> 3, k = r & 7;
    const unsigned brick = first + k * share + i;
    return i < share && brick < g.nb ? (int)brick : -1;
}

// LDS tile of the line forms: one slot per element, 16-byte aligned.  The
// element's block starts in its slot at the same offset from a 16-byte
// boundary as in global memory (where an odd element may start 8 bytes, in
// single precision 4, 8 or 12, after one), so both sides move whole aligned
// 16-byte chunks.
template <int P, typename T, int NVAR = NV>
struct LinesTile {
    static constexpr int M = P + 1, RAW = NVAR * M * M * M, VW = 16 / sizeof(T);
    static constexpr bool ODD = RAW % VW != 0;
    static constexpr int CH = (RAW + (ODD ? VW - 1 : 0) + VW - 1) / VW;   // chunks of a slot
    static constexpr int SLOT = CH * VW;
    static constexpr int OPS = LinesLds<P, T>::OPS;   // the operator block in front of the tile
    // Where value v of an element lies in its slot.  At m = 4 in FP64 the lines of
    // x and y start at multiples of 32 and 128 bytes and meet in a quarter of the
    // banks (47 % of the halo form's LDS cycles were conflicts, 58 % of the general
    // Jacobian's); in the upper half of z the 16-byte chunks are therefore exchanged
    // two bits of (x, y) at a time, after which any 16 lines of one direction use
    // different banks.  General Jacobian on 40^3 elements 351 -> 314 us (299 since),
    // linear hexes on 64^3 1.75 -> 1.63 ms (1.42 since), an RK4 step on 64^3 5.32 -> 5.27
    // ms (5.33), its residual alone (memory-bound) even.  The other shapes keep their
    // order: within an element their lines spread, but where a slot is a multiple of
    // the banks (p = 2 in double, p = 3 in single precision) a brick's elements meet in
    // the same ones (5.1 and 4.0 conflict cycles an LDS instruction, 1.8 with the
    // exchange).
    static constexpr bool SWZ = P == 3 && sizeof(T) == 8 && NVAR == NV;
    __device__ __forceinline__ static int place(int v) { return SWZ ? v ^ (v & 32 ? 6 : 0) : v; }
    __device__ __forceinline__ static int chunk(int c) { return SWZ ? c ^ (c & 16 ? 3 : 0) : c; }
    __device__ __forceinline__ static int off(int slot, int e)
    {
        return slot * SLOT + (ODD ? (int)(((unsigned)e * (unsigned)RAW) % VW) : 0);
    }
};

// The direction-D line through face point L in an element's slot Ut of the tile
// (LT::place): two starting points, from which all m are at fixed distances.
template <int P, typename T, int D, bool SWZ = LinesTile<P, T>::SWZ>
struct TileLine {
    static constexpr int M = P + 1, STR = D == 0 ? 1 : (D == 1 ? M : M * M);
    int a;
    __device__ __forceinline__ explicit TileLine(int L) : a(lt_base<P, T, D>(L)) {}
    __device__ __forceinline__ int at(int l) const { return a + l * STR; }
    __device__ __forceinline__ void load(const T *Ut, T (&x)[M]) const { line_load<M, STR>(Ut + a, x); }
    __device__ __forceinline__ void put(T *Ut, const T (&x)[M]) const { line_put<M, STR>(Ut + a, x); }
};
template <int P, typename T, int D>
struct TileLine<P, T, D, true> {
    static_assert(P == 3 && sizeof(T) == 8, "the exchange of LinesTile");
    static constexpr int M = 4;
    int a, b;
    __device__ __forceinline__ explicit TileLine(int L)
    {
        const int x = lt_base<P, T, D>(L);
        a = x ^ (x & 32 ? 6 : 0);
        b = a ^ (D == 0 ? 2 : (D == 1 ? 4 : 6));
    }
    __device__ __forceinline__ int at(int l) const
    {
        return D == 0 ? (l < 2 ? a : b) + (l & 1) : (D == 1 ? (l & 1 ? b : a) + 4 * (l & 2) : (l < 2 ? a : b) + 16 * l);
    }
    __device__ __forceinline__ void load(const T *Ut, T (&x)[M]) const
    {
        if constexpr (D == 0) {
            using V = typename V16<T>::type;
            const V v = *reinterpret_cast<const V *>(Ut + a), w = *reinterpret_cast<const V *>(Ut + b);
            x[0] = v[0], x[1] = v[1], x[2] = w[0], x[3] = w[1];
        } else {
#pragma unroll
            for (int l = 0; l < M; ++l) x[l] = Ut[at(l)];
        }
    }
    __device__ __forceinline__ void put(T *Ut, const T (&x)[M]) const
    {
        if constexpr (D == 0) {
            using V = typename V16<T>::type;
            *reinterpret_cast<V *>(Ut + a) = V{x[0], x[1]};
            *reinterpret_cast<V *>(Ut + b) = V{x[2], x[3]};
        } else {
#pragma unroll
            for (int l = 0; l < M; ++l) Ut[at(l)] = x[l];
        }
    }
};

// One element's block into its slot by direct loads into LDS: every wave takes
// 64 chunks of 16 bytes at a time and waits for none of them (the caller waits
// for vmcnt before the barrier).  lo is the block's offset in its slot; bytes
// before the block in its first chunk belong to the previous element (lo > 0
// only for e > 0), and the chunk that holds the block's end is read in
// four-byte words up to it, so nothing past the state is touched.
template <typename LT, typename T>
__device__ __forceinline__ void slot_load(const T *__restrict__ src, int lo, T *slot, int unit)
{
    typedef __attribute__((address_space(1))) const void gptr;
    typedef __attribute__((address_space(3))) void lptr;
    const int lane = threadIdx.x & 63;
    const int whole = (lo + LT::RAW) / LT::VW;      // chunks without the block's last, partial one
    const T *s0 = src - lo;
    const int c0 = unit * 64;
    if (c0 + lane < whole)
        __builtin_amdgcn_global_load_lds((gptr *)(s0 + LT::chunk(c0 + lane) * LT::VW), (lptr *)(slot + c0 * LT::VW), 16,
                                         0, 0);
    if constexpr (LT::ODD) {
        const int words = ((lo + LT::RAW) % LT::VW) * (int)(sizeof(T) / 4);
        if (unit == (LT::CH - 1) / 64 && lane < words)
            __builtin_amdgcn_global_load_lds((gptr *)((const int *)(s0 + whole * LT::VW) + lane),
                                             (lptr *)(slot + whole * LT::VW), 4, 0, 0);
    }
}

// The reverse: 64 chunks of an element's slot to its block in memory.
template <typename LT, typename T>
__device__ __forceinline__ void slot_store(const T *slot, int lo, T *__restrict__ dst, int unit)
{
    using V = typename V16<T>::type;
    const int c = unit * 64 + (threadIdx.x & 63);
    if (c >= LT::CH) return;
    const int v0 = c * LT::VW - lo;                 // first value of the chunk
    if (!LT::ODD || (v0 >= 0 && v0 + LT::VW <= LT::RAW)) {
        __builtin_nontemporal_store(reinterpret_cast<const V *>(slot)[LT::chunk(c)], reinterpret_cast<V *>(dst - lo) + c);
    } else {
#pragma unroll
        for (int w = 0; w < LT::VW; ++w)
            if (v0 + w >= 0 && v0 + w < LT::RAW) __builtin_nontemporal_store(slot[c * LT::VW + w], dst + v0 + w);
    }
}

}  // namespace dev

// The bricks a lattice is cut into for a kernel whose workgroups hold at most E
// elements: the shape with the least cost, bricks (4 E + pairs of outer faces)
// (a brick costs its workgroup's time whether its slots are in use or not, and
// the neighbours' traces on its outer faces come from memory; at p = 1 on 128^3
// hexes 4x4x1 takes 0.88 ms and 16x1x1 0.93 in double, 0.52 and 0.60 in single
// precision), the longest along x where it is equal (at p = 4 on 51^3 hexes 2x1x1
// takes 0.98 ms and 1x2x1 1.02).  A lattice of up to 256 elements (one
// for each CU; 512 in single precision, whose bricks are half as large) gets
// one-element bricks and one of up to E times that smaller ones in proportion:
// such a call takes one workgroup's latency, which grows with its brick (RK4 step
// at p = 3 in double on 6^3 hexes: 44 us with one-element bricks, 56 with four).
// One with more bricks than that, but not more than two for each CU, gets the
// smallest ones that stay within two, if they are smaller by a tenth (p = 2 in double
// on 12^3 hexes: 432 bricks of four 8.5 us a residual and 46 an RK4 step, 288 of six
// 9.0 and 53).
// Plans and objects keep theirs: up to 0.4 us a launch on the host otherwise (p = 1,
// 16^3: 8.7 us a residual, 8.9 when every call worked them out).
inline dev::FastDiv fast_div(uint32_t d)
{
    dev::FastDiv f{0, 31};
    while (f.s < 62 && (uint64_t)1 << (f.s - 31) < d) ++f.s;
    f.m = (uint32_t)((((uint64_t)1 << f.s) + d - 1) / d);
    return f;
}

inline dev::Bricks bricks_for(int E, int esize, int nx, int ny, int nz)
{
    const int64_t ne = (int64_t)nx * ny * nz;
    const int few = esize == 8 ? 256 : 512;
    const int most = (int)std::min<int64_t>(E, (ne + few - 1) / few);
    dev::Bricks g{};
    auto bricks = [&](int bx, int by, int bz) {
        return (double)((nx + bx - 1) / bx) * ((ny + by - 1) / by) * ((nz + bz - 1) / bz);
    };
    auto choose = [&](auto &&cost) {
        double best = 0.0;
        bool any = false;
        for (int bx = most; bx >= 1; --bx)
            for (int by = 1; bx * by <= most; ++by)
                for (int bz = 1; bx * by * bz <= most; ++bz) {
                    const double c = cost(bx, by, bz);
                    if (any && c >= best) continue;
                    any = true;
                    best = c;
                    g.bx = bx, g.by = by, g.bz = bz;
                }
    };
    auto throughput = [&](int bx, int by, int bz) {
        return bricks(bx, by, bz) * (4 * E + bx * by + by * bz + bz * bx);
    };
    choose(throughput);
    const double nb = bricks(g.bx, g.by, g.bz);
    if (nb > few && nb <= 2 * few) {
        const dev::Bricks large = g;
        choose([&](int bx, int by, int bz) {
            const double n = bricks(bx, by, bz), t = 1e-15 * throughput(bx, by, bz);
            return n > 2 * few ? 1e9 + t : (n > few ? 2 : 1) * (bx * by * bz) + t;
        });
        if (10 * g.bx * g.by * g.bz > 9 * large.bx * large.by * large.bz) g = large;
    }
    g.mx = (65536 + g.bx - 1) / g.bx;
    g.mxy = (65536 + g.bx * g.by - 1) / (g.bx * g.by);
    g.gx = (nx + g.bx - 1) / g.bx;
    g.gy = (ny + g.by - 1) / g.by;
    g.nb = (unsigned)g.gx * (unsigned)g.gy * (unsigned)((nz + g.bz - 1) / g.bz);
    g.chunk = (unsigned)(((int64_t)g.gx * g.gy + 7) / 8);
    g.by_gx = fast_div(g.gx);
    g.by_gy = fast_div(g.gy);
    g.by_group = fast_div(8 * g.chunk);
    return g;
}

}  // namespace fr
