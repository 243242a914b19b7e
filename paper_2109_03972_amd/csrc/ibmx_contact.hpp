// Contact geometry and collision law shared by the pair pass and the
// particle sub-stepping (Secs. 2.2.5-2.2.8, 2.2.10), FP64 throughout.
//
// Every listed contact is evaluated by each particle it touches, in the
// canonical orientation (first particle of the pair as p), so both sides
// obtain bit-identical values; each particle sums its contacts in
// increasing partner order (walls after the partners, by side) through a
// per-particle adjacency list, so forces and torques do not depend on
// thread scheduling.  The files including this header are compiled without
// FMA contraction.
#pragma once
#pragma clang fp contract(off)

#include <math.h>

#include "ibmx_internal.hpp"

namespace {

constexpr int kHist = IBMX_HIST;

struct PairC {
    double rho_f, nu_f, eps_sep, lub_C, zeta_min_factor, e_dry, T_c, mu_s, mu_k, nu_poi, dt;
    double gap_cut;
    double h;
    double L[3];
    double origin[3];
    double edge[3];
    int nc[3];
    int periodic[3];
    int ncell;
    // collision constants derived on the host
    int normal_model;     // 0 linear spring-dashpot, 1 Hertz with ACTM coefficients
    double le;            // ln e_dry
    double lin_k;         // pi^2 + ln^2 e_dry
    double sq_damp;       // sqrt(pi^2 + ln^2 e_dry)
    double kt_ratio;      // 2 (1 - nu) / (2 - nu)
    double K_hz, D_hz;    // ACTM coefficients of the Hertz law in contact-time units
    double Tc52;          // T_c^(5/2)
    double St_crit;
    double kn_grav_eps;
    double g_abs;         // |g|
    double g[3];
};

__device__ __forceinline__ double wrap_pos(double x, double o, double L)
{
    // inside the domain the quotient's floor is 0 (a quotient of a smaller by a
    // larger number rounds below 1): x itself, without the division
    const double d = x - o;
    if (d >= 0.0 && d < L)
        return x;
    double t = floor(d / L);
    return x - t * L;
}

__device__ __forceinline__ double min_image(double d, double L)
{
    while (d > 0.5 * L)
        d = d - L;
    while (d < -0.5 * L)
        d = d + L;
    return d;
}

__device__ __forceinline__ void centre(const PairC &P, int np, const double *xp, int p, double *x)
{
    for (int a = 0; a < 3; ++a) {
        double v = xp[(size_t)a * np + p];
        x[a] = P.periodic[a] ? wrap_pos(v, P.origin[a], P.L[a]) : v;
    }
}

__device__ __forceinline__ double disp2(const PairC &P, const double *a_, const double *b_, double *d)
{
    for (int a = 0; a < 3; ++a) {
        d[a] = b_[a] - a_[a];
        if (P.periodic[a])
            d[a] = min_image(d[a], P.L[a]);
    }
    double d2 = d[0] * d[0];
    d2 = d2 + d[1] * d[1];
    d2 = d2 + d[2] * d[2];
    return d2;
}

// rho_p d_p of a sphere: 3 m / (2 pi R^2)
__device__ __forceinline__ double rho_d(double m, double R) { return 3.0 * m / (2.0 * M_PI * R * R); }

// k_n,grav of one particle: m |g| (eps R)^(-3/2)
__device__ __forceinline__ double kn_grav(const PairC &P, double m, double R)
{
    double a = P.kn_grav_eps * R;
    return m * P.g_abs / (a * sqrt(a));
}

// What a contact's two bodies contribute to its force law besides their
// motion: fixed while the list holds.
struct ContactConst {
    double Reff, meff;
    double zmin;      // least gap of the lubrication law
    double u_crit;    // critical impact speed (Hertz)
    double kn;        // Hertz: stiffness at or under u_crit; linear: the stiffness
    double dn;        // normal damping
};

__device__ __forceinline__ ContactConst contact_const(const PairC &P, double Reff, double meff,
                                                      double Rmin, double rhod, double kgrav)
{
    ContactConst K;
    K.Reff = Reff;
    K.meff = meff;
    K.zmin = P.zeta_min_factor * Rmin;
    if (P.normal_model == 1) {
        K.u_crit = 9.0 * P.St_crit * P.rho_f * P.nu_f / rhod;
        const double kcrit =
            K.u_crit > 0.0 ? P.K_hz * meff / (sqrt(K.u_crit) * P.Tc52) : 0.0;
        K.kn = kcrit > kgrav ? kcrit : kgrav;
        K.dn = P.D_hz * meff / P.T_c;
    } else {
        K.u_crit = 0.0;
        K.kn = meff * P.lin_k / (P.T_c * P.T_c);
        K.dn = -2.0 * meff * P.le / P.T_c;
    }
    return K;
}

__device__ __forceinline__ ContactConst pair_const(const PairC &P, double mp, double Rp, double mq,
                                                   double Rq)
{
    const double kgp = kn_grav(P, mp, Rp), kgq = kn_grav(P, mq, Rq);
    return contact_const(P, Rp * Rq / (Rp + Rq), mp * mq / (mp + mq), Rp < Rq ? Rp : Rq,
                         0.5 * (rho_d(mp, Rp) + rho_d(mq, Rq)), kgp > kgq ? kgp : kgq);
}

// the wall as a partner of infinite radius and mass
__device__ __forceinline__ ContactConst wall_const(const PairC &P, double mp, double Rp)
{
    return contact_const(P, Rp, mp, Rp, rho_d(mp, Rp), kn_grav(P, mp, Rp));
}

// ---------------------------------------------------------------------------
// collision law for one contact (force on p; n points from p to the partner)
//   lubrication   0 <= zeta < eps_sep: -6 pi rho_f nu_f R_eff^2 psi / zz g_n
//   contact       zeta < 0: normal spring-dashpot (linear, or Hertz with the
//                 ACTM stiffness for the impact speed u_in, bounded below by
//                 max(k_n,crit, k_n,grav) at or under the critical speed)
//                 plus the tangential spring-dashpot capped by friction
// History hold/hnew: tangential spring (3), impact speed; dt is the time
// since the state the history belongs to.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void contact_law(const PairC &P, double zeta, const double *n,
                                            const double *g, const ContactConst &K,
                                            const double *hold, double dt, double *F, double *Ft,
                                            double *hnew)
{
    double gn = g[0] * n[0] + g[1] * n[1] + g[2] * n[2];
    double gnv[3], gtv[3];
    for (int a = 0; a < 3; ++a) {
        gnv[a] = gn * n[a];
        gtv[a] = g[a] - gnv[a];
        F[a] = 0.0;
        Ft[a] = 0.0;
    }
    for (int a = 0; a < kHist; ++a)
        hnew[a] = 0.0;
    if (zeta >= P.eps_sep)
        return;
    if (zeta >= 0.0) {
        double zz = zeta > K.zmin ? zeta : K.zmin;
        double psi = 0.5 * erf(6.0 - P.lub_C * zz / P.h) + 0.5;
        double coef = 6.0 * M_PI * P.rho_f * P.nu_f * K.Reff * K.Reff * psi / zz;
        for (int a = 0; a < 3; ++a)
            F[a] = -coef * gnv[a];
        return;
    }
    const double u_in = hold[3] > 0.0 ? hold[3] : (gn > 0.0 ? gn : 0.0);
    const double ze = fabs(zeta);
    double kn = K.kn, ks, Fn[3];
    if (P.normal_model == 1) {
        if (u_in > K.u_crit)
            kn = P.K_hz * K.meff / (sqrt(u_in) * P.Tc52);
        ks = kn * sqrt(ze);
        for (int a = 0; a < 3; ++a)
            Fn[a] = -kn * (ze * sqrt(ze)) * n[a] - K.dn * gnv[a];
    } else {
        ks = kn;
        for (int a = 0; a < 3; ++a)
            Fn[a] = -kn * ze * n[a] - K.dn * gnv[a];
    }
    double kt = P.kt_ratio * ks;
    double dtc = 2.0 * sqrt(K.meff * kt) * (-P.le) / P.sq_damp;
    double zon = hold[0] * n[0] + hold[1] * n[1] + hold[2] * n[2];
    double zt[3], Fdp[3];
    for (int a = 0; a < 3; ++a) {
        zt[a] = (hold[a] - zon * n[a]) + gtv[a] * dt;
        Fdp[a] = -kt * zt[a] - dtc * gtv[a];
    }
    double nFdp = sqrt(Fdp[0] * Fdp[0] + Fdp[1] * Fdp[1] + Fdp[2] * Fdp[2]);
    double nFn = sqrt(Fn[0] * Fn[0] + Fn[1] * Fn[1] + Fn[2] * Fn[2]);
    if (nFdp <= P.mu_s * nFn) {
        for (int a = 0; a < 3; ++a)
            Ft[a] = Fdp[a];
    } else {
        for (int a = 0; a < 3; ++a) {
            Ft[a] = P.mu_k * nFn * Fdp[a] / nFdp;
            zt[a] = -(Ft[a] + dtc * gtv[a]) / kt;
        }
    }
    for (int a = 0; a < 3; ++a) {
        F[a] = Fn[a] + Ft[a];
        hnew[a] = zt[a];
    }
    hnew[3] = u_in;
}

// motion of one particle
struct BodyState {
    double x[3], u[3], w[3], R;
};

// a contact's geometry: gap, normal, relative velocity at the contact point
// and the lever arms of the two bodies
struct ContactGeom {
    double zeta, n[3], g[3], arm_p, arm_q;
};

// Pair (p, q) of the list, p its first particle: g = (u_p - u_q) +
// R_p,cp w_p x n + R_q,cp w_q x n with the lever arms R_p,cp =
// (d + R_p - R_q)/2, R_q,cp = (d + R_q - R_p)/2.
__device__ __forceinline__ void pair_geometry(const PairC &P, const BodyState &p,
                                              const BodyState &q, ContactGeom &G)
{
    double xa[3], xb[3], dvec[3];
    for (int a = 0; a < 3; ++a) {
        xa[a] = P.periodic[a] ? wrap_pos(p.x[a], P.origin[a], P.L[a]) : p.x[a];
        xb[a] = P.periodic[a] ? wrap_pos(q.x[a], P.origin[a], P.L[a]) : q.x[a];
    }
    double d = sqrt(disp2(P, xa, xb, dvec));
    G.zeta = d - p.R - q.R;
    for (int a = 0; a < 3; ++a)
        G.n[a] = dvec[a] / d;
    const double *n = G.n;
    G.arm_p = 0.5 * (d + p.R - q.R);
    G.arm_q = 0.5 * (d + q.R - p.R);
    double wpn[3] = {p.w[1] * n[2] - p.w[2] * n[1], p.w[2] * n[0] - p.w[0] * n[2],
                     p.w[0] * n[1] - p.w[1] * n[0]};
    double wqn[3] = {q.w[1] * n[2] - q.w[2] * n[1], q.w[2] * n[0] - q.w[0] * n[2],
                     q.w[0] * n[1] - q.w[1] * n[0]};
    for (int a = 0; a < 3; ++a)
        G.g[a] = (p.u[a] - q.u[a]) + G.arm_p * wpn[a] + G.arm_q * wqn[a];
}

// Wall entry (p, side = 2 axis + upper): the wall at rest, lever arm = the
// centre's distance to the wall.
__device__ __forceinline__ void wall_geometry(const PairC &P, const BodyState &p, int side,
                                              ContactGeom &G)
{
    const int ax = side / 2, upper = side % 2;
    // every axis's distance, then the entry's: a select between the constants
    // themselves becomes a load from a per-lane address
    double d3[3];
    for (int a = 0; a < 3; ++a)
        d3[a] = upper == 0 ? p.x[a] - P.origin[a] : (P.origin[a] + P.L[a]) - p.x[a];
    const double dist = ax == 0 ? d3[0] : ax == 1 ? d3[1] : d3[2];
    G.zeta = dist - p.R;
    for (int a = 0; a < 3; ++a)
        G.n[a] = a == ax ? (upper == 0 ? -1.0 : 1.0) : 0.0;
    const double *n = G.n;
    double wpn[3] = {p.w[1] * n[2] - p.w[2] * n[1], p.w[2] * n[0] - p.w[0] * n[2],
                     p.w[0] * n[1] - p.w[1] * n[0]};
    for (int a = 0; a < 3; ++a)
        G.g[a] = p.u[a] + dist * wpn[a];
    G.arm_p = G.arm_q = dist;
}

// force and torque on one of a contact's bodies (second: the pair's second
// particle) and the new history
__device__ __forceinline__ void contact_force(const PairC &P, const ContactGeom &G,
                                              const ContactConst &K, bool second,
                                              const double *hold, double dt, double *f6,
                                              double *hnew)
{
    double F[3], Ft[3];
    contact_law(P, G.zeta, G.n, G.g, K, hold, dt, F, Ft, hnew);
    const double *n = G.n;
    const double nxFt[3] = {n[1] * Ft[2] - n[2] * Ft[1], n[2] * Ft[0] - n[0] * Ft[2],
                            n[0] * Ft[1] - n[1] * Ft[0]};
    const double arm = second ? G.arm_q : G.arm_p;
    for (int a = 0; a < 3; ++a) {
        f6[a] = second ? -F[a] : F[a];
        f6[3 + a] = arm * nxFt[a];
    }
}

// kContactLanes lanes serve one particle, kContactParticles a workgroup of one
// wave: lane j evaluates the particle's adjacency entries j,
// j + kContactLanes, ... (a pair in its canonical orientation, so both
// particles of a pair obtain identical values) and leaves force and torque in
// part; lane j < 6 then adds component j of the chunk's n entries in adjacency
// order (increasing partner id, walls after).  One wave to a workgroup, so the
// exchange needs no barrier and no particle waits for another workgroup's wave.
constexpr int kContactLanes = 8;
constexpr int kContactBlock = IBMX_WAVE;
constexpr int kContactParticles = kContactBlock / kContactLanes;

__device__ __forceinline__ double chunk_sum(const double (*part)[6], int j, int n, double acc)
{
    double v[kContactLanes];
    const int first = threadIdx.x - j, q = j < 6 ? j : 5;
#pragma unroll
    for (int t = 0; t < kContactLanes; ++t)
        v[t] = part[first + t][q];
#pragma unroll
    for (int t = 0; t < kContactLanes; ++t)
        acc = t < n ? acc + v[t] : acc;
    return acc;
}

// ---------------------------------------------------------------------------
// per-particle adjacency of the contact lists, int2 {code, aux} per entry
//   code   pair k, p first:  2k;  pair k, p second: 2k + 1;  wall k: -(k + 1)
//   aux    the partner's id (pairs) or the wall's side (walls)
//   order  increasing partner id, then walls by side
// ---------------------------------------------------------------------------
struct ContactLists {
    int pair_cap, wall_cap;
    const int *pairs;     // [2][pair_cap]
    const int *walls;     // [2][wall_cap]
    const int *counts;    // device [2]: listed pairs, walls (clamped to the caps)
};

__device__ __forceinline__ int n_pairs(const ContactLists &C) { return min(C.counts[0], C.pair_cap); }
__device__ __forceinline__ int n_walls(const ContactLists &C) { return min(C.counts[1], C.wall_cap); }

// list entries the adjacency can hold: pairs i < j of particles in range,
// wall entries of a particle in range on a wall axis; others are skipped
// (and reported as EINVAL)
__device__ __forceinline__ bool pair_ok(const ContactLists &C, int np, int k)
{
    const int i = C.pairs[k], j = C.pairs[C.pair_cap + k];
    return i >= 0 && j < np && i < j;
}
__device__ __forceinline__ bool wall_ok(const ContactLists &C, int np, const int *periodic, int k)
{
    const int p = C.walls[k], side = C.walls[C.wall_cap + k];
    return p >= 0 && p < np && side >= 0 && side < 6 && !periodic[side / 2];
}

struct Periodic {
    int p[3];
};

__global__ void k_adj_count(ContactLists C, int np, Periodic per, int *deg, int *err)
{
    const int npairs = n_pairs(C), nwall = n_walls(C);
    for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < npairs + nwall;
         k += gridDim.x * blockDim.x) {
        if (k < npairs) {
            if (!pair_ok(C, np, k)) {
                atomicCAS(err, 0, (int)IBMX_EINVAL);
                continue;
            }
            atomicAdd(&deg[C.pairs[k]], 1);
            atomicAdd(&deg[C.pairs[C.pair_cap + k]], 1);
        } else {
            if (!wall_ok(C, np, per.p, k - npairs)) {
                atomicCAS(err, 0, (int)IBMX_EINVAL);
                continue;
            }
            atomicAdd(&deg[C.walls[k - npairs]], 1);
        }
    }
}

__global__ void k_adj_fill(ContactLists C, int np, Periodic per, const int *off, int *cursor,
                           int2 *adj)
{
    const int npairs = n_pairs(C), nwall = n_walls(C);
    for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < npairs + nwall;
         k += gridDim.x * blockDim.x) {
        if (k < npairs) {
            if (!pair_ok(C, np, k))
                continue;
            const int i = C.pairs[k], j = C.pairs[C.pair_cap + k];
            adj[off[i] + atomicAdd(&cursor[i], 1)] = make_int2(2 * k, j);
            adj[off[j] + atomicAdd(&cursor[j], 1)] = make_int2(2 * k + 1, i);
        } else {
            const int kw = k - npairs;
            if (!wall_ok(C, np, per.p, kw))
                continue;
            const int p = C.walls[kw];
            adj[off[p] + atomicAdd(&cursor[p], 1)] = make_int2(-(kw + 1), C.walls[C.wall_cap + kw]);
        }
    }
}

__device__ __forceinline__ int adj_key(int np, int2 e) { return e.x >= 0 ? e.y : np + e.y; }

// insertion sort of each particle's entries by key (a few dozen at most)
__global__ void k_adj_sort(int np, const int *off, int2 *adj)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= np)
        return;
    int2 *a = adj + off[p];
    const int n = off[p + 1] - off[p];
    for (int i = 1; i < n; ++i) {
        const int2 v = a[i];
        const int kv = adj_key(np, v);
        int j = i - 1;
        while (j >= 0 && adj_key(np, a[j]) > kv) {
            a[j + 1] = a[j];
            --j;
        }
        a[j + 1] = v;
    }
}

// History of all contacts: pair k in rows [a * pair_cap + k], wall k in
// [a * wall_cap + k], a = 0 .. kHist - 1.
struct Hist {
    double *pair;
    double *wall;
};

// Method parameters and the host-derived collision constants (everything
// but the cell grid).
inline void contact_constants(const ibmx_plan p, PairC *P)
{
    const ibmx_params &prm = p->prm;
    P->rho_f = prm.rho_f;
    P->nu_f = prm.nu_f;
    P->eps_sep = prm.eps_sep;
    P->lub_C = prm.lub_C;
    P->zeta_min_factor = prm.zeta_min_factor;
    P->e_dry = prm.e_dry;
    P->T_c = prm.T_c;
    P->mu_s = prm.mu_s;
    P->mu_k = prm.mu_k;
    P->nu_poi = prm.nu_poi;
    P->dt = prm.dt;
    P->gap_cut = prm.gap_cut;
    P->h = p->g.h;
    for (int a = 0; a < 3; ++a) {
        P->L[a] = p->g.n[a] * p->g.h;
        P->origin[a] = p->g.origin[a];
        P->periodic[a] = p->g.periodic[a];
        P->g[a] = prm.gravity[a];
    }
    P->normal_model = prm.normal_model;
    P->le = log(prm.e_dry);
    P->lin_k = M_PI * M_PI + P->le * P->le;
    P->sq_damp = sqrt(M_PI * M_PI + P->le * P->le);
    P->kt_ratio = 2.0 * (1.0 - prm.nu_poi) / (2.0 - prm.nu_poi);
    P->K_hz = p->actm_K;
    P->D_hz = p->actm_D;
    P->Tc52 = prm.T_c * prm.T_c * sqrt(prm.T_c);
    P->St_crit = prm.St_crit;
    P->kn_grav_eps = prm.kn_grav_eps;
    P->g_abs = sqrt(prm.gravity[0] * prm.gravity[0] + prm.gravity[1] * prm.gravity[1] +
                    prm.gravity[2] * prm.gravity[2]);
}

inline int contact_blocks(long long n, int b) { return n > 0 ? (int)((n + b - 1) / b) : 1; }

// Adjacency of the lists in C into the plan's contact workspace (c_off,
// c_adj), which holds np + 1 offsets and 2 pair_cap + wall_cap entries.
inline void contact_adjacency(ibmx_plan p, const ContactLists &C, hipStream_t s)
{
    const int np = p->np;
    const long long nmax = (long long)C.pair_cap + C.wall_cap;
    const int g = contact_blocks(nmax, 256) < 4096 ? contact_blocks(nmax, 256) : 4096;
    ZeroList z = {};
    z.add(p->c_deg, np + 1);
    z.add(p->c_cur, np);
    ibmx_zero_i32_multi(z, s);
    const Periodic per{{p->grid.periodic[0], p->grid.periodic[1], p->grid.periodic[2]}};
    hipLaunchKernelGGL(k_adj_count, dim3(g), dim3(256), 0, s, C, np, per, p->c_deg, p->d_err);
    ibmx_exclusive_scan(p->c_deg, p->c_off, np, p->scan_aux, s);
    hipLaunchKernelGGL(k_adj_fill, dim3(g), dim3(256), 0, s, C, np, per, (const int *)p->c_off,
                       p->c_cur, p->c_adj);
    hipLaunchKernelGGL(k_adj_sort, dim3(contact_blocks(np, 64)), dim3(64), 0, s, np,
                       (const int *)p->c_off, p->c_adj);
}

}  // namespace
