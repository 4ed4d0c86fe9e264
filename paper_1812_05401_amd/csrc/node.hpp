// The node update of the strip sweep (strip.hpp): moments, penalization, edge rules and collision
// with every rounding written out.
//
// The same arithmetic as relax_node in lattice.hpp, operation for operation: where that source
// leaves a product and a sum to the compiler, the fused form the compiler takes is written here as
// an explicit fmadd and contraction is off, so the result does not depend on what the code is
// inlined into, and a population is bitwise the one that every other kernel computes.  A factor of
// a power of two is moved where that is exact: hs = (ha + hb)/2 is never formed at a fluid node,
// the relaxation runs on twice the value and the last two sums halve it.
#pragma once

#include "lattice.hpp"

namespace vplbm {

// A wave-uniform value, kept in scalar registers.
__device__ __forceinline__ float uniform(float v) { return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(v))); }
__device__ __forceinline__ double uniform(double v)
{
    const long long b = __double_as_longlong(v);
    const unsigned lo = __builtin_amdgcn_readfirstlane(unsigned(b));
    const unsigned hi = __builtin_amdgcn_readfirstlane(unsigned(b >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// NodeParams in the compute type.
template <typename T> struct Rates {
    T sp, sm, kp, km, k_relax, c_pen, uin_x, uin_y;
    __device__ __forceinline__ explicit Rates(const NodeParams &p)
        : sp(uniform(T(p.sp))), sm(uniform(T(p.sm))), kp(uniform(T(p.kp))), km(uniform(T(p.km))),
          k_relax(uniform(T(p.k_relax))), c_pen(uniform(T(p.c_pen))), uin_x(uniform(T(p.uin_x))),
          uin_y(uniform(T(p.uin_y)))
    {
    }
};

// Sums and differences of the opposite pairs, density deviation and momentum (Eqs. 8-9).
template <typename T> struct Pairs {
    T s1, s2, s5, s6, d1, d2, d5, d6;   // (1,3) (2,4) (5,7) (6,8)
    T drho, jx, jy, rho, inv;
};

template <typename T> __device__ __forceinline__ Pairs<T> pair_sums(const T h[9])
{
#pragma clang fp contract(off)
    Pairs<T> p;
    p.s1 = h[1] + h[3];
    p.s2 = h[2] + h[4];
    p.s5 = h[5] + h[7];
    p.s6 = h[6] + h[8];
    p.d1 = h[1] - h[3];
    p.d2 = h[2] - h[4];
    p.d5 = h[5] - h[7];
    p.d6 = h[6] - h[8];
    p.drho = (h[0] + p.s1) + (p.s2 + (p.s5 + p.s6));
    p.jx = p.d1 + (p.d5 - p.d6);
    p.jy = p.d2 + (p.d5 + p.d6);
    p.rho = T(1) + p.drho;
    p.inv = reciprocal(p.rho);
    return p;
}

// One opposite pair at a fluid node: s, d its sum and difference, c = xi . u, wrho = -2 w rho.
template <typename T>
__device__ __forceinline__ void fluid_pair(T &ha, T &hb, T s, T d, T c, T w, T wrho, T drho, T rho, T q, T sp, T sm)
{
#pragma clang fp contract(off)
    T e = fmadd(c, T(4.5) * c, q);
    e = fmadd(rho, e, drho);
    const T ns = fmadd(-fmadd(e, T(-2) * w, s), sp, s);               // twice the symmetric half
    const T na = T(0.5) * fmadd(-fmadd(wrho, T(3) * c, d), sm, d);    // the antisymmetric half
    ha = fmadd(T(0.5), ns, na);
    hb = fmadd(T(0.5), ns, -na);
}

// Fluid node: no force.  In place on the pulled h; returns drho.
template <typename T> __device__ __forceinline__ T relax_fluid(T h[9], const Rates<T> &r)
{
#pragma clang fp contract(off)
    const Pairs<T> p = pair_sums(h);
    const T ux = p.jx * p.inv, uy = p.jy * p.inv;
    const T q = T(-1.5) * fmadd(ux, ux, uy * uy);
    h[0] = fmadd(-fmadd(fmadd(p.rho, q, p.drho), -W<T>::rest, h[0]), r.sp, h[0]);
    const T wa = (T(-2) * W<T>::axis) * p.rho, wd = (T(-2) * W<T>::diag) * p.rho;
    fluid_pair(h[1], h[3], p.s1, p.d1, ux, W<T>::axis, wa, p.drho, p.rho, q, r.sp, r.sm);
    fluid_pair(h[2], h[4], p.s2, p.d2, uy, W<T>::axis, wa, p.drho, p.rho, q, r.sp, r.sm);
    fluid_pair(h[5], h[7], p.s5, p.d5, ux + uy, W<T>::diag, wd, p.drho, p.rho, q, r.sp, r.sm);
    fluid_pair(h[6], h[8], p.s6, p.d6, uy - ux, W<T>::diag, wd, p.drho, p.rho, q, r.sp, r.sm);
    return p.drho;
}

template <typename T>
__device__ __forceinline__ void solid_pair(T &ha, T &hb, T s, T d, T c, T xf, T w, T wrho, T drho, T rho, T q,
                                           T f3, const Rates<T> &r)
{
#pragma clang fp contract(off)
    const T hs = T(0.5) * s, hd = T(0.5) * d;
    T e = fmadd(c, T(4.5) * c, q);
    e = fmadd(rho, e, drho);
    T ns = fmadd(-fmadd(e, -w, hs), r.sp, hs);
    T na = fmadd(-fmadd(wrho, T(3) * c, hd), r.sm, hd);
    ns = fmadd(w * fmadd(T(9) * c, xf, -f3), r.kp, ns);
    na = fmadd(w * (T(3) * xf), r.km, na);
    ha = ns + na;
    hb = ns - na;
}

// A solid node of a body with velocity (usx, usy) here: the penalized velocity and force (Eqs. 17-18)
// and the forced collision.  A fluid node (solid false, velocity 0) comes out as from relax_fluid: the
// factors 1 and 0 in place of k and c make u = j / rho and f = 0, and adding the force's zeros changes
// no value, so a row that holds both kinds needs no branch.  In place; returns drho and the force.
template <typename T>
__device__ __forceinline__ T relax_solid(T h[9], bool solid, T usx, T usy, const Rates<T> &r, T &fx, T &fy)
{
#pragma clang fp contract(off)
    const Pairs<T> p = pair_sums(h);
    const T k = solid ? r.k_relax : T(1), c = solid ? r.c_pen : T(0);
    const T ux = fmadd(p.jx * p.inv - usx, k, usx);
    const T uy = fmadd(fmadd(p.jy, p.inv, -usy), k, usy);
    fx = -fmadd(-p.rho, usx, p.jx) * c;
    fy = -fmadd(-p.rho, usy, p.jy) * c;
    const T q = T(-1.5) * fmadd(ux, ux, uy * uy);
    const T f3 = T(3) * fmadd(ux, fx, uy * fy);
    h[0] = fmadd(-fmadd(fmadd(p.rho, q, p.drho), -W<T>::rest, h[0]), r.sp, h[0]);
    h[0] = fmadd(f3 * -W<T>::rest, r.kp, h[0]);
    const T wa = -W<T>::axis * p.rho, wd = -W<T>::diag * p.rho;
    solid_pair(h[1], h[3], p.s1, p.d1, ux, fx, W<T>::axis, wa, p.drho, p.rho, q, f3, r);
    solid_pair(h[2], h[4], p.s2, p.d2, uy, fy, W<T>::axis, wa, p.drho, p.rho, q, f3, r);
    solid_pair(h[5], h[7], p.s5, p.d5, ux + uy, fx + fy, W<T>::diag, wd, p.drho, p.rho, q, f3, r);
    solid_pair(h[6], h[8], p.s6, p.d6, uy - ux, fy - fx, W<T>::diag, wd, p.drho, p.rho, q, f3, r);
    return p.drho;
}

// zou_he_west and solid_velocity of lattice.hpp, roundings written out.
template <typename T> __device__ __forceinline__ void inlet_west(T h[9], T ux, T uy)
{
#pragma clang fp contract(off)
    const T known = fmadd(T(2), (h[3] + h[6]) + h[7], (h[0] + h[2]) + h[4]);
    const T drho = (known + ux) / (T(1) - ux);
    const T rho = T(1) + drho;
    const T d2 = h[2] - h[4], ru = rho * ux, half = T(0.5) * rho;
    h[1] = fmadd(T(2.0 / 3.0) * rho, ux, h[3]);
    h[5] = fmadd(half, uy, fmadd(ru, T(1.0 / 6.0), fmadd(T(-0.5), d2, h[7])));
    h[8] = fmadd(-half, uy, fmadd(ru, T(1.0 / 6.0), fmadd(T(0.5), d2, h[6])));
}

// body: centre (x, y), velocity (x, y) and angular velocity.
template <typename T> __device__ __forceinline__ void body_velocity(const T body[5], int x, int y, T &usx, T &usy)
{
#pragma clang fp contract(off)
    usx = fmadd(-body[4], T(y) - body[1], body[2]);
    usy = fmadd(body[4], T(x) - body[0], body[3]);
}

// The convective outlet's implicit upwind rule.
template <typename T> __device__ __forceinline__ T outlet_value(T prev, T nb, T u)
{
#pragma clang fp contract(off)
    return fmadd(u, nb, prev) / (T(1) + u);
}

}  // namespace vplbm
