// Residual of ACM-HD as line tasks for elements whose metric mixes the
// directions: a general constant Jacobian (AffineGeo) or linear hexahedra, whose
// metric varies inside the element (TrilinearGeo).
//
// As in the halo form for diagonal Jacobians, a workgroup takes a brick of
// elements into LDS (straight from memory) and a lane owns one line of one
// direction d of one element and forms its neighbours' traces from their lines,
// in the tile or in memory.  With S_d(xi) the metric row along the line the lane
// computes
//   the transformed momentum fluxes F_i = u_i V.S_d + P S_di - nu sum_k S_ik S_dk
//   and their corrected derivatives (all thirteen values of a point enter, in every
//   direction),
//   the corrected derivatives of u_a S_dk, the auxiliary equations' fluxes, whose
//   sum over a = k is P's; with a constant metric those of u_a, once, times S_dk.
// Once every lane has read the tile's S, the auxiliary parts are summed over it
// in three rounds, in round j the lanes of direction d on the components
// k = (d + j) mod 3, so that no two directions meet and all waves work; then the
// P and momentum parts, kept in registers until here (the velocities are read
// again in the auxiliary rounds, which costs less than registers to hold them),
// over the tile's P and velocities in the same manner.  The finished tile is R;
// nothing else goes through memory.
//
// The direction is a lane's own number, not a template parameter: three copies
// of this code would not fit the instruction cache (p = 4: 74 KB), and lines of
// all directions fill the waves better than one direction a wave (p = 5: 108 of
// 128 lanes instead of 36 of 64).  The operators are read through the scalar
// cache, a row at a time: LDS is what the kernel is bound by next to the FP64
// units.
#pragma once

#include <type_traits>

#include "bricks.h"

namespace fr {
namespace dev {

// A view of the operators for scalar loads; op_row() hides where the values come
// from, so that a row is loaded where it is used and not kept (or spilled).
template <typename T> using OpPtr = const __attribute__((address_space(4))) T *;
template <typename T> __device__ __forceinline__ OpPtr<T> op_ptr(const T *p) { return (OpPtr<T>)p; }
template <typename T> __device__ __forceinline__ OpPtr<T> op_row(OpPtr<T> p)
{
    __asm__ volatile("" : "+s"(p));
    return p;
}

// What k_metric takes beside the plan's constants.  In Consts itself the other kernels
// paid for it: with J^{-1} among its arguments the halo form's residual took 43.3 us
// in place of 40.7 at p = 2 on 25 x 24 x 43 hexes and 27.5 in place of 24.7 at p = 3
// in single precision on 28 x 30 x 19 (lattices that fit the last-level cache).
template <typename T>
struct MetricConsts : Consts<T> {
    T jinv[3][3];  // J^{-1}: row d is n_d / det(J), rounded once
    MetricConsts(const Consts<T> &c, const double *Jinv) : Consts<T>(c)
    {
        for (int k = 0; k < 9; ++k) jinv[k / 3][k % 3] = (T)Jinv[k];
    }
};

// Constant S_d, S_d / det J, |S_d| and 1 / det J of direction d.
template <typename T>
struct AffineGeo {
    static constexpr bool constant = true;
    T s[3], ji[3], nh[3], mag, idet;
    __device__ __forceinline__ AffineGeo(const MetricConsts<T> &c, int d)
        : mag(d == 0 ? c.nmag[0] : (d == 1 ? c.nmag[1] : c.nmag[2])), idet(c.inv_det)
    {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            s[k] = d == 0 ? c.nvec[0][k] : (d == 1 ? c.nvec[1][k] : c.nvec[2][k]);
            ji[k] = d == 0 ? c.jinv[0][k] : (d == 1 ? c.jinv[1][k] : c.jinv[2][k]);
            nh[k] = d == 0 ? c.nhat[0][k] : (d == 1 ? c.nhat[1][k] : c.nhat[2][k]);
        }
    }
    __device__ __forceinline__ T S(int k, T) const { return s[k]; }
    __device__ __forceinline__ T inv_det(T) const { return idet; }
    // unit normal and |S_d| at the line's end
    template <bool PLUS>
    __device__ __forceinline__ T normal(T (&n)[3]) const
    {
#pragma unroll
        for (int k = 0; k < 3; ++k) n[k] = nh[k];
        return mag;
    }
    // S_k / det J for the lane's own k
    __device__ __forceinline__ T over_det(int k) const
    {
        const T a = ji[0], b = ji[1], c = ji[2];   // values, so the metric stays in registers
        return k == 0 ? a : (k == 1 ? b : c);
    }
};

// The trilinear map's tangents are a_d = const, a_{d+1} = p0 + p1 xi, a_{d+2} =
// q0 + q1 xi along a line of direction d, so S_d = a_{d+1} x a_{d+2} and det J =
// a_d . S_d are quadratics in xi.
struct TrilinearGeo {
    static constexpr bool constant = false;
    double s[3][3], d[3];   // coefficients of S_k and of det J
    double rm, rp;          // 1 / |S_d| at xi = -1 and +1
    __device__ __forceinline__ static double at(const double (&q)[3], double x) { return fma(x, fma(x, q[2], q[1]), q[0]); }
    __device__ __forceinline__ double S(int k, double x) const { return at(s[k], x); }
    __device__ __forceinline__ double inv_det(double x) const { return 1.0 / at(d, x); }
    template <bool PLUS>
    __device__ __forceinline__ double normal(double (&nh)[3]) const
    {
        const double r = PLUS ? rp : rm;
        double n2 = 0.0;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            nh[k] = S(k, PLUS ? 1.0 : -1.0);
            n2 = fma(nh[k], nh[k], n2);
            nh[k] *= r;
        }
        return n2 * r;
    }
    __device__ __forceinline__ void component(int k, double (&q)[3]) const
    {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const double a = s[0][i], b = s[1][i], c = s[2][i];   // values, so the metric stays in registers
            q[i] = k == 0 ? a : (k == 1 ? b : c);
        }
    }
};

// The points of a line: at(l) is the place of the l-th in an element's block, in
// memory (base + l str) or in the tile (LinesTile::place).
template <int P>
struct MemoryLine {
    int base, str;
    __device__ __forceinline__ int at(int l) const { return base + l * str; }
};
template <typename LT, int P>
struct SlotLine {
    int p[P + 1];
    __device__ __forceinline__ SlotLine(int base, int str)
    {
#pragma unroll
        for (int l = 0; l <= P; ++l) p[l] = LT::place(base + l * str);
    }
    __device__ __forceinline__ int at(int l) const { return p[l]; }
};

// The traces of P, u, v, w and of (grad V) n at the end with basis values lf of
// the line of the element block X.
template <int P, typename T, typename Line>
__device__ __forceinline__ void full_trace(const T *X, const Line &line, OpPtr<T> lf, const T (&nh)[3],
                                           T (&out)[NTR])
{
    constexpr int M = P + 1, NS = M * M * M;
    auto end = [&](int v) {
        T acc = T(0);
#pragma unroll
        for (int l = 0; l < M; ++l) acc = fma(lf[l], X[line.at(l) + v * NS], acc);
        return acc;
    };
#pragma unroll
    for (int v = 0; v < 4; ++v) out[v] = end(v);
#pragma unroll
    for (int v = 0; v < 4; ++v) pin(out[v]);
    // the 13 lines' loads in groups (one or two memory latencies): all 13 m at
    // once would need more registers than the rest of the kernel
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        if (i == 1 || P >= 4) __builtin_amdgcn_sched_barrier(0);
        const T a = end(4 + 3 * i), b = end(5 + 3 * i), c = end(6 + 3 * i);
        out[4 + i] = fma(c, nh[2], fma(b, nh[1], a * nh[0]));
        pin(out[4 + i]);
    }
}

// (The tile is not marked restrict: the compiler would keep its values in
// registers from one loop to the next.)
// First phase: traces, common fluxes, and into part[1..3][r] the corrected
// derivatives of the momentum fluxes; part[0] gets the faces' dissipation of P, to
// which zeta times the derivative of V.S_d is added where the velocities' own
// derivatives are formed (from a flux of its own, rounded at the points and on the
// faces, P was 1.2 to 1.4 times as far from the exact value in single precision, 1.05
// times in double).  X: the element's slot of the tile; othm, othp: the neighbours' traces; vm, vp: the mean velocities on its faces.
template <int P, typename T, typename Line, typename Geo>
__device__ __forceinline__ void metric_fluxes(const T *X, const Line &line, OpPtr<T> ops, OpPtr<T> x,
                                              const T (&othm)[NTR], const T (&othp)[NTR], const Geo &geo,
                                              T zeta, T nu, T (&vm)[3], T (&vp)[3], T (&part)[4][P + 1])
{
    constexpr int M = P + 1, NS = M * M * M;
    using OL = OpsLayout<M>;
    T fm[4], fp[4];
    {
        // both ends of the thirteen lines, each value read once
        T am[13], ap[13];
#pragma unroll
        for (int v = 0; v < 13; ++v) am[v] = ap[v] = T(0);
#pragma unroll
        for (int l = 0; l < M; ++l) {
            __builtin_amdgcn_sched_barrier(0);
            const T wm = ops[OL::lm + l], wp = ops[OL::lp + l];
#pragma unroll
            for (int v = 0; v < 13; ++v) {
                const T q = X[line.at(l) + v * NS];
                am[v] = fma(wm, q, am[v]);
                ap[v] = fma(wp, q, ap[v]);
            }
#pragma unroll
            for (int v = 0; v < 13; ++v) {
                pin(am[v]);
                pin(ap[v]);
            }
        }
        auto face = [&](auto pc, const T (&a)[13], const T (&oth)[NTR], T (&f)[4], T (&v)[3]) {
            constexpr bool PLUS = decltype(pc)::value;
            T own[NTR], out[NTR], nh[3];
            const T mag = geo.template normal<PLUS>(nh);
#pragma unroll
            for (int k = 0; k < 4; ++k) own[k] = a[k];
#pragma unroll
            for (int k = 0; k < 3; ++k)
                own[4 + k] = fma(a[6 + 3 * k], nh[2], fma(a[5 + 3 * k], nh[1], a[4 + 3 * k] * nh[0]));
            common_flux_sided<T>(own, oth, PLUS, nh, mag, zeta, nu, out);
#pragma unroll
            for (int k = 0; k < 4; ++k) f[k] = out[k];
#pragma unroll
            for (int k = 0; k < 3; ++k) v[k] = out[4 + k];
#pragma unroll
            for (int k = 0; k < 4; ++k) pin(f[k]);
#pragma unroll
            for (int k = 0; k < 3; ++k) pin(v[k]);
        };
        face(std::false_type{}, am, othm, fm, vm);
        __builtin_amdgcn_sched_barrier(0);
        face(std::true_type{}, ap, othp, fp, vp);
    }
    // the fluxes point by point, then their corrected derivatives row by row
    T F[3][M];
#pragma unroll
    for (int l = 0; l < M; ++l) {
        __asm__ volatile("" ::: "memory");   // one point's values at a time
        __builtin_amdgcn_sched_barrier(0);
        const T *q = X + line.at(l);
        const T xl = x[l];
        const T s[3] = {geo.S(0, xl), geo.S(1, xl), geo.S(2, xl)};
        const T u[3] = {q[NS], q[2 * NS], q[3 * NS]};
        const T vn = fma(u[2], s[2], fma(u[1], s[1], u[0] * s[0]));
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const T *G = q + (4 + 3 * i) * NS;
            const T gn = fma(G[2 * NS], s[2], fma(G[NS], s[1], G[0] * s[0]));
            F[i][l] = fma(u[i], vn, fma(q[0], s[i], -nu * gn));
        }
#pragma unroll
        for (int v = 0; v < 3; ++v) pin(F[v][l]);
    }
#pragma unroll
    for (int r = 0; r < M; ++r) {
        const auto op = op_row(ops);
        T Dr[M];
#pragma unroll
        for (int l = 0; l < M; ++l) Dr[l] = op[OL::Dt + r * M + l];
        const T glr = op[OL::gl + r], grr = op[OL::gr + r];
        part[0][r] = fma(glr, fm[0], grr * fp[0]);
        pin(part[0][r]);
#pragma unroll
        for (int v = 0; v < 3; ++v) {
            T s = T(0);
#pragma unroll
            for (int l = 0; l < M; ++l) s = fma(Dr[l], F[v][l], s);
            part[1 + v][r] = fma(glr, fm[1 + v], fma(grr, fp[1 + v], s));
            pin(part[1 + v][r]);
        }
    }
}

// Constant metric: the corrected derivatives of the velocities, once for all three
// components of S_d (products u_a S_dk that are rounded before they are
// differentiated put the auxiliary residual 1.07 to 1.28 times as far from the exact
// value in single precision), and their part of the divergence.
template <int P, typename T, typename Line>
__device__ __forceinline__ void metric_gradient(const T *X, const Line &line, OpPtr<T> ops, const AffineGeo<T> &geo,
                                                T zeta, const T (&vm)[3], const T (&vp)[3], T (&cd)[3][P + 1],
                                                T (&pp)[P + 1])
{
    constexpr int M = P + 1, NS = M * M * M;
    using OL = OpsLayout<M>;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        // read again: the points' velocities are not kept over the fluxes' derivatives
        __asm__ volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        T u[M];
#pragma unroll
        for (int l = 0; l < M; ++l) u[l] = X[line.at(l) + (1 + a) * NS];
#pragma unroll
        for (int r = 0; r < M; ++r) {
            const auto op = op_row(ops);
            T s = T(0);
#pragma unroll
            for (int l = 0; l < M; ++l) s = fma(op[OL::Dt + r * M + l], u[l], s);
            cd[a][r] = fma(op[OL::gl + r], vm[a], fma(op[OL::gr + r], vp[a], s));
            pin(cd[a][r]);
        }
    }
#pragma unroll
    for (int r = 0; r < M; ++r) {
        pp[r] = fma(zeta, fma(cd[2][r], geo.s[2], fma(cd[1][r], geo.s[1], cd[0][r] * geo.s[0])), pp[r]);
        pin(pp[r]);
    }
}

// Round J of the auxiliary sums from these: S_ak of component k = (d + J) mod 3 minus
// the derivative of u_a times S_dk / det J; after the last round times -1/T, the
// auxiliary residual.
template <int P, typename T, int J, typename Line>
__device__ __forceinline__ void metric_aux(T *X, const Line &line, int d, const AffineGeo<T> &geo, T invT,
                                           const T (&cd)[3][P + 1])
{
    constexpr int M = P + 1, NS = M * M * M;
    const int k = d + J >= 3 ? d + J - 3 : d + J;
    const T c = -geo.over_det(k);
    T *Y = X + (4 + k) * NS;
#pragma unroll
    for (int r = 0; r < M; ++r)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            T *q = Y + line.at(r) + 3 * a * NS;
            const T v = fma(c, cd[a][r], *q);
            *q = J == 2 ? -invT * v : v;
        }
}

// Varying metric, round J: S_ak of component k = (d + J) mod 3 minus the corrected
// derivative of u_a S_dk over det J; after the last round times -1/T, the auxiliary
// residual.  pp: zeta times that of u_k S_dk is added, the round's part
// of the divergence.  X: the element's slot of the tile; W: its field 1 / det J.
template <int P, int J, typename Line>
__device__ __forceinline__ void metric_aux(double *X, const Line &line, int d, OpPtr<double> ops, OpPtr<double> x,
                                           const double *W, const TrilinearGeo &geo, double zeta, double invT,
                                           const double (&vm)[3], const double (&vp)[3], double (&pp)[P + 1])
{
    using T = double;
    using Geo = TrilinearGeo;
    constexpr int M = P + 1, NS = M * M * M;
    using OL = OpsLayout<M>;
    const int k = d + J >= 3 ? d + J - 3 : d + J;
    T *Y = X + (4 + k) * NS;
    T c[3];
    geo.component(k, c);
    const T sm = Geo::at(c, T(-1)), sp = Geo::at(c, T(1));
    T G[3][M];
#pragma unroll
    for (int l = 0; l < M; ++l) {
        const T s = Geo::at(c, x[l]);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            G[a][l] = X[line.at(l) + (1 + a) * NS] * s;
            pin(G[a][l]);
        }
    }
#pragma unroll
    for (int r = 0; r < M; ++r) {
        const auto op = op_row(ops);
        T Dr[M];
#pragma unroll
        for (int l = 0; l < M; ++l) Dr[l] = op[OL::Dt + r * M + l];
        const T glr = op[OL::gl + r] * sm, grr = op[OL::gr + r] * sp;
        const T w = W[line.at(r)];
        T sk = T(0);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            T s = T(0);
#pragma unroll
            for (int l = 0; l < M; ++l) s = fma(Dr[l], G[a][l], s);
            s = fma(glr, vm[a], fma(grr, vp[a], s));
            sk = a == k ? s : sk;
            T *q = Y + line.at(r) + 3 * a * NS;
            const T v = fma(-w, s, *q);
            *q = J == 2 ? -invT * v : v;
        }
        pp[r] = fma(zeta, sk, pp[r]);
        pin(pp[r]);
    }
}

// Threads and elements of a workgroup, one lane per line: as few idle lanes as 2
// to 4 waves allow (p = 4: 225 of 256 lanes 1.82 ms, 150 of 192 1.88 ms on 51^3
// hexes; p = 3: 192 of 192 1.80, 240 of 256 1.92).  Five waves, which fill the
// four SIMDs unevenly, are 1.8 to 3 times slower.
template <int P> struct MetricShape {
    static constexpr int M = P + 1, NT = P == 5 ? 128 : (P == 4 ? 256 : 192), E = NT / (3 * M * M);
};

// LDS of a workgroup in T: the brick, 1 / det J at its points.
template <int P, typename T, typename Geo>
struct MetricLds {
    static constexpr int M = P + 1, W = MetricShape<P>::E * LinesTile<P, T>::SLOT;
    static constexpr int size = W + (Geo::constant ? 0 : MetricShape<P>::E * M * M * M);
};

// The kernel's body.  make_geo(d, element, a, b) gives the metric along the
// line of direction d through the element's face point (a, b).
template <int P, typename T, typename MakeGeo>
__device__ __forceinline__ void metric_residual(const T *__restrict__ U, T *__restrict__ R,
                                                const T *__restrict__ ops_, T zeta, T nu, T invT,
                                                int nx, int ny, int nz, const Bricks &g, T *sU,
                                                MakeGeo &&make_geo)
{
    using MS = MetricShape<P>;
    using LT = LinesTile<P, T>;
    using OL = OpsLayout<P + 1>;
    constexpr int M = P + 1, NS = M * M * M, NF = M * M, E = MS::E;
    constexpr int RAW = LT::RAW, UNITS = (LT::CH + 63) / 64, WAVES = MS::NT / 64;
    const OpPtr<T> ops = op_ptr(ops_), x = ops + OL::x;
    const int brick = brick_of(g, blockIdx.x);
    if (brick < 0) return;
    const int row = g.by_gx(brick), lay = g.by_gy(row);
    const int cx = (brick - row * g.gx) * g.bx, cy = (row - lay * g.gy) * g.by, cz = lay * g.bz;
    const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const BrickElems<(E > 1)> elem(g, cx, cy, cz, nx, ny, nz);
    for (int u = wave; u < E * UNITS; u += WAVES) {
        const int s = u / UNITS, e = elem(s);
        if (e >= 0) {
            const int lo = LT::off(0, e);
            slot_load<LT>(U + (int64_t)e * RAW, lo, sU + s * LT::SLOT, u - s * UNITS);
        }
    }
    const int el = t / (3 * NF), line = t - el * 3 * NF, d = line / NF, L = line - d * NF, la = L % M, lb = L / M;
    const BrickSlot me = brick_slot(g, el, cx, cy, cz, nx, ny, nz);
    const bool act = el < E && me.e >= 0;
    const int sd = d == 0 ? me.sx : (d == 1 ? me.sy : me.sz);
    const int bd = d == 0 ? g.bx : (d == 1 ? g.by : g.bz);
    const int xd = sd + (d == 0 ? cx : (d == 1 ? cy : cz));
    const int n = d == 0 ? nx : (d == 1 ? ny : nz);
    const int le = d == 0 ? 1 : (d == 1 ? nx : nx * ny), ls = d == 0 ? 1 : (d == 1 ? g.bx : g.bx * g.by);
    const int nbm = me.e + (xd == 0 ? n - 1 : -1) * le, nbp = me.e + (xd + 1 == n ? 1 - n : 1) * le;
    const bool inm = act && sd > 0, inp = act && sd + 1 < bd && xd + 1 < n;
    // the line: first point and the points' distance
    const int base = d == 0 ? M * L : (d == 1 ? la + M * M * lb : L), str = d == 0 ? 1 : (d == 1 ? M : M * M);
    const MemoryLine<P> outer{base, str};
    const std::conditional_t<LT::SWZ, SlotLine<LT, P>, MemoryLine<P>> inner{base, str};
    T *X = sU + (act ? LT::off(el, me.e) : 0);
    T *W = sU + MetricLds<P, T, AffineGeo<T>>::size + (act ? el : 0) * NS;
    const auto geo = make_geo(d, act ? me.e : 0, la, lb);
    using Geo = std::decay_t<decltype(geo)>;
    if constexpr (!Geo::constant)
        if (act && d == 0)
#pragma unroll 1
            for (int r = 0; r < M; ++r) W[LT::place(base + r)] = geo.inv_det(x[r]);
    T othm[NTR], othp[NTR];
    {
        T nm[3], np[3];
        geo.template normal<false>(nm);
        geo.template normal<true>(np);
        if (act && !inm) full_trace<P, T>(U + (int64_t)nbm * RAW, outer, ops + OL::lp, nm, othm);
        if (act && !inp) full_trace<P, T>(U + (int64_t)nbp * RAW, outer, ops + OL::lm, np, othp);
        // the direct loads into LDS have arrived (their count is not tracked by
        // the barrier)
        __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if constexpr (E > 1) {
            if (inm) full_trace<P, T>(sU + LT::off(el - ls, nbm), inner, ops + OL::lp, nm, othm);
            if (inp) full_trace<P, T>(sU + LT::off(el + ls, nbp), inner, ops + OL::lm, np, othp);
        }
    }
    T vm[3], vp[3], part[4][M], cd[3][M];
    if (act) {
        metric_fluxes<P, T>(X, inner, ops, x, othm, othp, geo, zeta, nu, vm, vp, part);
        if constexpr (Geo::constant) metric_gradient<P, T>(X, inner, ops, geo, zeta, vm, vp, cd, part[0]);
    }
    auto aux = [&](auto jc) {
        constexpr int J = decltype(jc)::value;
        __syncthreads();
        if (!act) return;
        if constexpr (Geo::constant) metric_aux<P, T, J>(X, inner, d, geo, invT, cd);
        else metric_aux<P, J>(X, inner, d, ops, x, W, geo, zeta, invT, vm, vp, part[0]);
    };
    // round 0 stores, 1 adds, 2 adds and divides by -det J; P goes with u
    auto add = [&](auto jc) {
        constexpr int J = decltype(jc)::value;
        __syncthreads();
        const int k = d + J >= 3 ? d + J - 3 : d + J;
        if (!act) return;
        auto put = [&](T *q, int r, T o) {
            if constexpr (J != 0) o += q[inner.at(r)];
            if constexpr (J == 2) o *= -(Geo::constant ? geo.inv_det(T(0)) : W[inner.at(r)]);
            q[inner.at(r)] = o;
        };
        // the component is selected, not branched on: with a branch for each of the
        // three the compiler (ROCm 7.2) merges their stores and forms the third's
        // address under the exec mask of the lanes that take the first, so that
        // k = 2 stores to an unset address (seen in the assembly; wrong residuals at
        // every order)
#pragma unroll
        for (int r = 0; r < M; ++r) {
            const T a = part[1][r], b = part[2][r], c = part[3][r];
            put(X + (1 + k) * NS, r, k == 0 ? a : (k == 1 ? b : c));
        }
        if (k == 0)
#pragma unroll
            for (int r = 0; r < M; ++r) put(X, r, part[0][r]);
    };
    aux(Dir<0>{});
    aux(Dir<1>{});
    aux(Dir<2>{});
    add(Dir<0>{});
    add(Dir<1>{});
    add(Dir<2>{});
    __syncthreads();
    for (int u = wave; u < E * UNITS; u += WAVES) {
        const int s = u / UNITS, e = elem(s);
        if (e >= 0) slot_store<LT>(sU + s * LT::SLOT, LT::off(0, e), R + (int64_t)e * RAW, u - s * UNITS);
    }
}

}  // namespace dev
}  // namespace fr
