// Adjoint of the D3Q19 central-moment collision in increment form without
// force: from dL/ds* (gbar) and dL/dfeatures of the learned rates' inputs
// (xbar) to dL/ds, at fixed rates.
//
// Forward: raw moments m = M s, rho and u, non-equilibrium moments
// n = m - E(rho, u) (orders >= 2), central ones k = S(-u) n, the relaxation's
// change d(k) (linear), raw again q = S(u) d, s* = s + M^-1 q.  Every factor
// is run backwards once.  Two facts keep it short: a shift's derivative along
// an axis lowers the exponent, d S(u) v / du_a = N_a S(u) v with
// (N_a v)_e = e_a v_(e - a), and so does the equilibrium's,
// dE_e / du_a = e_a E_(e - a).  About 500 operations per node, where one
// directional derivative per population (19 evaluations of the collision on
// dual numbers) takes about 19000.
#pragma once

#include "d3q19_cm.hpp"

namespace lbm {

// transpose of raw_from_pops: g_i += sum_e m_e c_i^e
template <class R> __host__ __device__ inline void raw_from_pops_T(const RawMoments<R>& m, R g[19])
{
    g[0] += m.m000;
    auto axis = [&](int neg, int pos, R odd, R even) {
        g[pos] += (m.m000 + even) + odd;
        g[neg] += (m.m000 + even) - odd;
    };
    axis(1, 10, m.m100, m.m200);
    axis(2, 11, m.m010, m.m020);
    axis(3, 12, m.m001, m.m002);
    // a face's four diagonals: (-,-) (-,+) (+,+) (+,-)
    auto face = [&](int mm, int mp, int pp, int pm, R a1, R b1, R a2, R b2, R ab, R a2b, R ab2, R a2b2) {
        const R e = (m.m000 + a2) + (b2 + a2b2); // even in both
        const R oa = a1 + ab2, ob = b1 + a2b;    // odd in the first, in the second
        g[pp] += (e + ab) + (oa + ob);
        g[mm] += (e + ab) - (oa + ob);
        g[pm] += (e - ab) + (oa - ob);
        g[mp] += (e - ab) - (oa - ob);
    };
    face(4, 5, 13, 14, m.m100, m.m010, m.m200, m.m020, m.m110, m.m210, m.m120, m.m220);
    face(6, 7, 15, 16, m.m100, m.m001, m.m200, m.m002, m.m101, m.m201, m.m102, m.m202);
    face(8, 9, 17, 18, m.m010, m.m001, m.m020, m.m002, m.m011, m.m021, m.m012, m.m022);
}

// sum_e e_a b_e v_(e - a) over the monomials whose e - a is of order >= 2
template <class R> __host__ __device__ inline void lowered(const RawMoments<R>& b, const RawMoments<R>& v, R& x, R& y, R& z)
{
    const R two = R(2);
    x = two * (b.m210 * v.m110 + b.m201 * v.m101 + b.m220 * v.m120 + b.m202 * v.m102) + b.m120 * v.m020 + b.m102 * v.m002;
    y = two * (b.m120 * v.m110 + b.m021 * v.m011 + b.m220 * v.m210 + b.m022 * v.m012) + b.m210 * v.m200 + b.m012 * v.m002;
    z = two * (b.m102 * v.m101 + b.m012 * v.m011 + b.m202 * v.m201 + b.m022 * v.m021) + b.m201 * v.m200 + b.m021 * v.m020;
}

// st: pre_collide's state of the node (GENERAL, no force); rt: its rates;
// qb = M^-T gbar (pops_from_raw_T) and db = S(u)^T qb (shift_all_T);
// xbar: dL/d of the 11 raw features.  g: gbar on entry, dL/ds on return.
template <class R>
__host__ __device__ inline void collide_adjoint(const CMState<R>& st, R rho0, const Rates<R>& rt,
                                                const RawMoments<R>& qb, const RawMoments<R>& db, const R xbar[11], R g[19])
{
    const RawMoments<R>& k = st.n;
    const R third = R(1) / R(3), irho = R(1) / st.rho;
    const R w = rt.omega, wb = rt.omega_bulk;
    const R* oh = rt.omega_hi;
    // q = S(u) d
    RawMoments<R> q;
    const R kt = third * st.k4;
    q.m000 = q.m100 = q.m010 = q.m001 = R(0);
    q.m200 = -w * (k.m200 - kt) - wb * kt;
    q.m020 = -w * (k.m020 - kt) - wb * kt;
    q.m002 = -w * (k.m002 - kt) - wb * kt;
    q.m110 = -w * k.m110;
    q.m101 = -w * k.m101;
    q.m011 = -w * k.m011;
    q.m210 = -oh[0] * k.m210;
    q.m120 = -oh[1] * k.m120;
    q.m201 = -oh[2] * k.m201;
    q.m102 = -oh[3] * k.m102;
    q.m021 = -oh[4] * k.m021;
    q.m012 = -oh[5] * k.m012;
    q.m220 = -oh[6] * k.m220;
    q.m202 = -oh[7] * k.m202;
    q.m022 = -oh[8] * k.m022;
    shift_all(q, st.ux, st.uy, st.uz);
    R ux, uy, uz; // dL/du
    lowered(qb, q, ux, uy, uz);
    // dL/dk: the relaxation is its own transpose, plus the features'
    RawMoments<R> b;
    const R dt = third * (db.m200 + db.m020 + db.m002), xt = xbar[1] * irho;
    b.m000 = b.m100 = b.m010 = b.m001 = R(0);
    b.m200 = -w * (db.m200 - dt) - wb * dt + xt;
    b.m020 = -w * (db.m020 - dt) - wb * dt + xt;
    b.m002 = -w * (db.m002 - dt) - wb * dt + xt;
    b.m110 = -w * db.m110;
    b.m101 = -w * db.m101;
    b.m011 = -w * db.m011;
    b.m210 = -oh[0] * db.m210 + xbar[2] * irho;
    b.m120 = -oh[1] * db.m120 + xbar[3] * irho;
    b.m201 = -oh[2] * db.m201 + xbar[4] * irho;
    b.m102 = -oh[3] * db.m102 + xbar[5] * irho;
    b.m021 = -oh[4] * db.m021 + xbar[6] * irho;
    b.m012 = -oh[5] * db.m012 + xbar[7] * irho;
    b.m220 = -oh[6] * db.m220 + xbar[8] * irho;
    b.m202 = -oh[7] * db.m202 + xbar[9] * irho;
    b.m022 = -oh[8] * db.m022 + xbar[10] * irho;
    R r = xbar[0]; // dL/drho; a feature is its moment over rho
    {
        const R f = xbar[1] * st.k4 +
                    (xbar[2] * k.m210 + xbar[3] * k.m120 + xbar[4] * k.m201 + xbar[5] * k.m102 + xbar[6] * k.m021 +
                     xbar[7] * k.m012) +
                    (xbar[8] * k.m220 + xbar[9] * k.m202 + xbar[10] * k.m022);
        r -= f * irho * irho;
    }
    // k = S(-u) n
    R ax, ay, az;
    lowered(b, k, ax, ay, az);
    ux -= ax;
    uy -= ay;
    uz -= az;
    shift_all_T(b, -st.ux, -st.uy, -st.uz);
    // n = m - E(rho, u): E whole, from its deviation
    RawMoments<R> E = st.e;
    const R r3 = rho0 * third, r9 = r3 * third;
    E.m200 += r3;
    E.m020 += r3;
    E.m002 += r3;
    E.m220 += r9;
    E.m202 += r9;
    E.m022 += r9;
    lowered(b, E, ax, ay, az);
    ux -= ax + (R(2) * b.m200 * E.m100 + b.m110 * E.m010 + b.m101 * E.m001);
    uy -= ay + (R(2) * b.m020 * E.m010 + b.m110 * E.m100 + b.m011 * E.m001);
    uz -= az + (R(2) * b.m002 * E.m001 + b.m101 * E.m100 + b.m011 * E.m010);
    r -= irho * ((b.m200 * E.m200 + b.m020 * E.m020 + b.m002 * E.m002) +
                 (b.m110 * E.m110 + b.m101 * E.m101 + b.m011 * E.m011) +
                 (b.m210 * E.m210 + b.m120 * E.m120 + b.m201 * E.m201 + b.m102 * E.m102 + b.m021 * E.m021 + b.m012 * E.m012) +
                 (b.m220 * E.m220 + b.m202 * E.m202 + b.m022 * E.m022));
    // u = m1 / rho
    b.m100 = ux * irho;
    b.m010 = uy * irho;
    b.m001 = uz * irho;
    b.m000 = r - (ux * st.ux + uy * st.uy + uz * st.uz) * irho;
    raw_from_pops_T(b, g);
}

} // namespace lbm
