// Particle sub-stepping (Sec. 2.2.10) and the ACTM coefficients of the
// Hertz normal contact (Sec. 2.2.7).
//
// One call advances the particles by n_sub sub-steps of three Runge-Kutta
// stages; each stage is two launches of a lane group per particle:
//   predictor  contacts at the accepted state s^{k-1} (committing the
//              contact history of that state), then s~ into a separate
//              state buffer;
//   corrector  contacts at s~ (history not committed), then s^k over the
//              particle's own s^{k-1}.
// Contacts read the partners' state from a buffer no launch in flight
// writes; the stage forces of s^{k-1} and s^{k-2} are kept per particle in
// two alternating buffers.
//
// A launch depends on every particle of the one before, and a list of a few
// thousand contacts is one wave per compute unit: the time is the launch's
// chain of dependent loads and of FP64 divisions and roots, not bytes.  So a
// first launch lays out, for the whole call, what a stage reads:
//   records     16 doubles on one line per particle: state and constants;
//   entries     the first kContactLanes adjacency entries at a fixed place,
//               so they are fetched together with the particle's own data
//               and the partner's record is the second load of the chain
//               instead of the third;
//   constants   of each contact (ContactConst): 10 of its about 27 divisions
//               and roots;
//   history     the 4 doubles of a contact side by side.
// The update itself is spread over six lanes, a component each.  2000
// particles, 15 sub-steps of 6 launches: 11.8 us per launch with the arrays by
// component, workgroups of four waves and the update on one lane; 5.1 us so
// (about 2 us of it the launch itself), 1115 us to 475 us per call.

#include "ibmx_contact.hpp"

namespace {

// ---------------------------------------------------------------------------
// ACTM coefficients, host.  In contact-time units the overlap obeys
// z'' + D z' + K z^(3/2) = 0 from z = 0, z' = 1, and the contact must close
// at t = 1 with z' = -e.  The time change t -> t / b maps (K, D) to
// (K b^(5/2), D b), so it suffices to find the damping D1 of the K = 1
// problem whose rebound is e (the rebound falls with D1), read its
// duration T1, and scale: K = T1^(5/2), D = D1 T1.
// ---------------------------------------------------------------------------
struct UnitRun {
    bool closed;
    double T;       // contact duration
    double v_end;   // z' when the overlap closes
};

inline double hertz_force(double z) { return z > 0.0 ? z * sqrt(z) : 0.0; }

inline void unit_rk4(double D1, double h, double &z, double &v)
{
    const double a1 = v, b1 = -D1 * v - hertz_force(z);
    const double a2 = v + 0.5 * h * b1, b2 = -D1 * a2 - hertz_force(z + 0.5 * h * a1);
    const double a3 = v + 0.5 * h * b2, b3 = -D1 * a3 - hertz_force(z + 0.5 * h * a2);
    const double a4 = v + h * b3, b4 = -D1 * a4 - hertz_force(z + h * a3);
    z += h / 6.0 * (a1 + 2.0 * a2 + 2.0 * a3 + a4);
    v += h / 6.0 * (b1 + 2.0 * b2 + 2.0 * b3 + b4);
}

UnitRun unit_run(double D1)
{
    const double h = 5.0e-5;       // the undamped K = 1 contact lasts about 3.2
    const long steps = 800000;
    double z = 0.0, v = 1.0, t = 0.0;
    for (long s = 0; s < steps; ++s) {
        double zn = z, vn = v;
        unit_rk4(D1, h, zn, vn);
        if (s > 0 && zn <= 0.0) {
            // closing inside this step: bisect the length of a partial step
            double lo = 0.0, hi = h;
            for (int it = 0; it < 80; ++it) {
                const double mid = 0.5 * (lo + hi);
                double zm = z, vm = v;
                unit_rk4(D1, mid, zm, vm);
                (zm > 0.0 ? lo : hi) = mid;
            }
            double ze = z, ve = v;
            unit_rk4(D1, hi, ze, ve);
            return UnitRun{true, t + hi, ve};
        }
        z = zn;
        v = vn;
        t = (double)(s + 1) * h;   // not a running sum: no accumulated rounding
    }
    return UnitRun{false, t, v};
}

}  // namespace

ibmx_status ibmx_actm_coefficients(double e, double *K, double *D)
{
    if (!(e > 0.0 && e <= 1.0) || !K || !D)
        return IBMX_EINVAL;
    double D1 = 0.0;
    if (e < 1.0) {
        double lo = 0.0, hi = 0.25;
        for (int it = 0; it < 60; ++it) {
            const UnitRun r = unit_run(hi);
            if (r.closed && -r.v_end < e)
                break;
            lo = hi;
            hi *= 2.0;
        }
        for (int it = 0; it < 64; ++it) {
            const double mid = 0.5 * (lo + hi);
            const UnitRun r = unit_run(mid);
            if (r.closed && -r.v_end < e)
                hi = mid;
            else
                lo = mid;
        }
        D1 = 0.5 * (lo + hi);
    }
    const UnitRun r = unit_run(D1);
    if (!r.closed)
        return IBMX_EINVAL;
    *K = r.T * r.T * sqrt(r.T);
    *D = D1 * r.T;
    return IBMX_OK;
}

namespace {

// ---------------------------------------------------------------------------
// kernels
// ---------------------------------------------------------------------------
// a particle's record: position, velocity and angular velocity (3 each), then
enum { kRecR = 9, kRecM = 10, kRecI = 11, kRecB = 12, kRecS = 13, kRec = 16 };
// radius, mass, I = 2/5 m R^2, 1 - rho_f / rho_p, the factor of F_h and T_h

constexpr int kNoEntry = -2147483647 - 1;   // code of a missing adjacency entry
constexpr int kConst = 6;                   // doubles of a ContactConst
constexpr int kForce = 8;                   // doubles of a stage force: F, T, 2 unused

enum { kStageForces = 0, kStagePredict = 1, kStageCorrect = 2 };

struct Stage {
    double dts;       // sub-step length
    double a2;        // 2 alpha_k
    double alpha;     // alpha_k
    double gamma;     // gamma_k
    double zeta;      // zeta_k
};

// adjacency of the lists as the stages read it
struct Adjacency {
    const int *off;        // [np + 1]
    const int2 *adj;       // by off
    const int2 *first;     // [np][kContactLanes], kNoEntry past the particle's last
    const double *consts;  // [entries][kConst]
};

struct StageIO {
    const double *rec;            // records the contacts are evaluated at
    double *acc;                  // accepted records (own entry updated by the corrector)
    double *pred;                 // predicted records (written by the predictor)
    const double *hold;           // [pair_cap + wall_cap][kHist]
    double *hnew;                 // written by the predictor
    const double *Fh, *Th;        // or null
    double *Fcur;                 // [np][kForce] at the accepted state
    const double *Fprev;          // the same one stage earlier
};

// outputs of the last evaluation
struct FinalOut {
    double *xp, *up, *wp;
    double *Fc, *Tc;              // or null
    Hist hist;
};

__device__ __forceinline__ BodyState record_state(const double *rec)
{
    double2 v[5];
#pragma unroll
    for (int q = 0; q < 5; ++q)
        v[q] = ((const double2 *)rec)[q];
    return BodyState{{v[0].x, v[0].y, v[1].x}, {v[1].y, v[2].x, v[2].y},
                     {v[3].x, v[3].y, v[4].x}, v[4].y};
}

// Records, entries, contact constants and history of the call, and the
// factor of F_h and T_h: 0 when the switch is on and the input history holds
// at least one contact of the particle, all with St <= St_crit.
__global__ __launch_bounds__(kContactBlock) void k_sub_setup(
    PairC P, int np, ContactLists C, const int *__restrict__ off, const int2 *__restrict__ adj,
    const double *__restrict__ xp, const double *__restrict__ up, const double *__restrict__ wp,
    const double *__restrict__ radius, const double *__restrict__ mass,
    const double *__restrict__ hist, const double *__restrict__ whist, int on,
    double *__restrict__ acc, double *__restrict__ pred, int2 *__restrict__ first,
    double *__restrict__ consts, double *__restrict__ h0)
{
    const int j = threadIdx.x % kContactLanes;
    const int p = blockIdx.x * kContactParticles + threadIdx.x / kContactLanes;
    if (p >= np)
        return;
    const int lo = off[p], deg = off[p + 1] - lo;
    const double R = radius[p], m = mass[p];
    int contacts = 0, fast = 0;
    if (j >= deg)
        first[(size_t)p * kContactLanes + j] = make_int2(kNoEntry, 0);
    for (int r = j; r < deg; r += kContactLanes) {
        const int2 e = adj[lo + r];
        if (r < kContactLanes)
            first[(size_t)p * kContactLanes + r] = e;
        ContactConst K;
        double rhod, h[kHist];
        if (e.x >= 0) {
            const int k = e.x >> 1, i1 = (e.x & 1) ? e.y : p, i2 = (e.x & 1) ? p : e.y;
            const double m1 = mass[i1], m2 = mass[i2], R1 = radius[i1], R2 = radius[i2];
            for (int a = 0; a < kHist; ++a)
                h[a] = hist[(size_t)a * C.pair_cap + k];
            if (!(e.x & 1))
                for (int a = 0; a < kHist; ++a)
                    h0[(size_t)k * kHist + a] = h[a];
            K = pair_const(P, m1, R1, m2, R2);
            rhod = 0.5 * (rho_d(m1, R1) + rho_d(m2, R2));
        } else {
            const int k = -e.x - 1;
            for (int a = 0; a < kHist; ++a) {
                h[a] = whist[(size_t)a * C.wall_cap + k];
                h0[((size_t)C.pair_cap + k) * kHist + a] = h[a];
            }
            K = wall_const(P, m, R);
            rhod = rho_d(m, R);
        }
        double2 *c = (double2 *)(consts + (size_t)(lo + r) * kConst);
        c[0] = make_double2(K.Reff, K.meff);
        c[1] = make_double2(K.zmin, K.u_crit);
        c[2] = make_double2(K.kn, K.dn);
        if (h[3] > 0.0) {
            ++contacts;
            const double St = h[3] * rhod / (9.0 * P.rho_f * P.nu_f);
            fast += St > P.St_crit;
        }
    }
    for (int s = 1; s < kContactLanes; s *= 2) {
        contacts += __shfl_xor(contacts, s, kContactLanes);
        fast += __shfl_xor(fast, s, kContactLanes);
    }
    if (j >= 3) {
        if (j == 3) {
            const double rho_p = m / (4.0 / 3.0 * M_PI * R * R * R);
            const double c[5] = {R, m, 0.4 * m * R * R, 1.0 - P.rho_f / rho_p,
                                 (on && contacts > 0 && fast == 0) ? 0.0 : 1.0};
            for (int q = 0; q < 5; ++q) {
                acc[(size_t)p * kRec + kRecR + q] = c[q];
                pred[(size_t)p * kRec + kRecR + q] = c[q];
            }
        }
        return;
    }
    const size_t i = (size_t)j * np + p;
    acc[(size_t)p * kRec + j] = xp[i];
    acc[(size_t)p * kRec + 3 + j] = up[i];
    acc[(size_t)p * kRec + 6 + j] = wp[i];
}

// One contact evaluation of every particle, then its update: lane j < 3 holds
// force component j and updates velocity and position, lane 3 + j the torque's
// and the angular velocity.
template <int MODE>
__global__ __launch_bounds__(kContactBlock) void k_sub_stage(PairC P, int np, ContactLists C,
                                                             Adjacency A, StageIO io, double dt,
                                                             Stage S, FinalOut out)
{
    __shared__ double part[kContactBlock][6];
    const int j = threadIdx.x % kContactLanes;
    const int p = blockIdx.x * kContactParticles + threadIdx.x / kContactLanes;
    const bool live = p < np;
    const int pc = live ? p : np - 1;
    const int jc = j < 6 ? j : 5, a = jc < 3 ? jc : jc - 3;
    // the particle's own data, while the entries are on their way
    const int2 e0 = A.first[(size_t)pc * kContactLanes + j];
    const int lo = A.off[pc], next_lo = A.off[pc + 1];
    const int deg = live ? next_lo - lo : 0;
    const double *own = io.acc + (size_t)pc * kRec;
    const double x0 = own[a], v0 = own[3 + jc];
    const double fac_h = own[kRecS], inert = own[jc < 3 ? kRecM : kRecI], fac_g = own[kRecB];
    double fh = 0.0, fprev = 0.0, F = 0.0;
    if (MODE != kStageForces) {
        const double *H = jc < 3 ? io.Fh : io.Th;
        if (H)
            fh = H[(size_t)a * np + pc];
        if (MODE == kStageCorrect)
            fprev = io.Fcur[(size_t)pc * kForce + jc];
        else if (S.zeta != 0.0)
            fprev = io.Fprev[(size_t)pc * kForce + jc];
    }
    for (int c = 0; __any(c * kContactLanes < deg); ++c) {
        const int r = c * kContactLanes + j;
        if (r < deg) {
            const int2 e = c == 0 ? e0 : A.adj[lo + r];
            const bool pair = e.x >= 0, second = pair && (e.x & 1);
            const int k = pair ? e.x >> 1 : -e.x - 1;
            const size_t kh = pair ? (size_t)k : (size_t)C.pair_cap + k;
            const double2 *hp = (const double2 *)(io.hold + kh * kHist);
            const double2 *cp = (const double2 *)(A.consts + (size_t)(lo + r) * kConst);
            const BodyState s1 = record_state(io.rec + (size_t)(second ? e.y : p) * kRec);
            const BodyState s2 = record_state(io.rec + (size_t)(pair && !second ? e.y : p) * kRec);
            const double2 h01 = hp[0], h23 = hp[1];
            const double2 c0 = cp[0], c1 = cp[1], c2 = cp[2];
            const ContactConst K{c0.x, c0.y, c1.x, c1.y, c2.x, c2.y};
            const double ho[kHist] = {h01.x, h01.y, h23.x, h23.y};
            double hn[kHist];
            ContactGeom G;
            if (pair)
                pair_geometry(P, s1, s2, G);
            else
                wall_geometry(P, s1, e.y, G);
            contact_force(P, G, K, second, ho, dt, part[threadIdx.x], hn);
            if (MODE == kStagePredict && !second) {
                double2 *h = (double2 *)(io.hnew + kh * kHist);
                h[0] = make_double2(hn[0], hn[1]);
                h[1] = make_double2(hn[2], hn[3]);
            }
            if (MODE == kStageForces && !second)
                for (int b = 0; b < kHist; ++b) {
                    if (pair)
                        out.hist.pair[(size_t)b * C.pair_cap + k] = hn[b];
                    else
                        out.hist.wall[(size_t)b * C.wall_cap + k] = hn[b];
                }
        }
        __syncthreads();
        F = chunk_sum(part, j, deg - c * kContactLanes, F);
        __syncthreads();
    }
    if (!live || j >= 6)
        return;
    if (MODE == kStageForces) {
        const size_t i = (size_t)a * np + p;
        if (j < 3) {
            out.xp[i] = x0;
            out.up[i] = v0;
        } else {
            out.wp[i] = v0;
        }
        if (out.Fc)
            (j < 3 ? out.Fc : out.Tc)[i] = F;
        return;
    }
    double f = S.a2 * (fac_h * fh) + S.gamma * F;
    if (MODE == kStagePredict) {
        // F: the accepted state's force, kept for the corrector and the next
        // stage
        io.Fcur[(size_t)p * kForce + j] = F;
        if (S.zeta != 0.0)
            f = f + S.zeta * fprev;
    } else {
        // F: the predicted state's force
        f = f + S.zeta * fprev;
    }
    double *next = (MODE == kStagePredict ? io.pred : io.acc) + (size_t)p * kRec;
    double v1 = v0 + S.dts / inert * f;
    if (j < 3) {
        v1 = v1 + S.a2 * S.dts * (fac_g * (a == 0 ? P.g[0] : a == 1 ? P.g[1] : P.g[2]));
        next[j] = x0 + S.alpha * S.dts * (v1 + v0);
    }
    next[3 + j] = v1;
}

}  // namespace

extern "C" ibmx_status ibmx_particle_substeps(ibmx_plan p, double dt_total, int32_t n_sub,
                                              double *xp, double *up, double *wp,
                                              const double *radius, const double *mass,
                                              const double *Fh, const double *Th,
                                              const int32_t *counts, int32_t pair_cap,
                                              const int32_t *pairs, int32_t wall_cap,
                                              const int32_t *walls, double *hist, double *whist,
                                              double *Fc, double *Tc)
{
    if (!p || n_sub < 1 || !isfinite(dt_total) || pair_cap < 0 || wall_cap < 0)
        return IBMX_EINVAL;
    const int np = p->np;
    if (np > 0 && (!xp || !up || !wp || !radius || !mass))
        return IBMX_EINVAL;
    if ((pair_cap > 0 || wall_cap > 0) && !counts)
        return IBMX_EINVAL;
    if ((pair_cap > 0 && (!pairs || !hist)) || (wall_cap > 0 && (!walls || !whist)) ||
        (!Fc) != (!Tc))
        return IBMX_EINVAL;
    if (np == 0)
        return IBMX_OK;
    // the workspace comes from ibmx_plan_reserve: this call allocates nothing
    if (!ibmx_contact_ready(p, pair_cap, wall_cap, 2) || !p->s_buf ||
        p->s_cap < ibmx_substep_doubles(np, 2LL * pair_cap + wall_cap))
        return IBMX_ESTATE;
    hipStream_t s = p->stream;
    ProfScope ps(p, IBMX_K_PAIRS);
    PairC P;
    contact_constants(p, &P);
    const ContactLists C{pair_cap, wall_cap, pairs, walls, counts};
    const size_t hset = (size_t)kHist * ((size_t)pair_cap + wall_cap);
    double *H[2] = {p->c_hist, p->c_hist + hset};
    // records of the two states, stage forces, entries, contact constants
    double *acc = p->s_buf, *pred = acc + (size_t)kRec * np;
    double *Fbuf[2] = {pred + (size_t)kRec * np, pred + (size_t)(kRec + kForce) * np};
    int2 *first = (int2 *)(Fbuf[1] + (size_t)kForce * np);
    double *consts = (double *)(first + (size_t)kContactLanes * np);
    const dim3 grid((unsigned)((np + kContactParticles - 1) / kContactParticles));
    if (counts) {
        contact_adjacency(p, C, s);
    } else {
        ibmx_fill_i32(p->c_off, 0, np + 1, s);
    }
    hipLaunchKernelGGL(k_sub_setup, grid, dim3(kContactBlock), 0, s, P, np, C,
                       (const int *)p->c_off, (const int2 *)p->c_adj, (const double *)xp,
                       (const double *)up, (const double *)wp, radius, mass, (const double *)hist,
                       (const double *)whist, p->prm.st_switch, acc, pred, first, consts, H[0]);
    static const double alpha[3] = {4.0 / 15.0, 1.0 / 15.0, 1.0 / 6.0};
    static const double gamma_[3] = {8.0 / 15.0, 5.0 / 12.0, 3.0 / 4.0};
    static const double zeta_[3] = {0.0, -17.0 / 60.0, -5.0 / 12.0};
    const double dts = dt_total / n_sub;
    const Adjacency A{p->c_off, p->c_adj, first, consts};
    const FinalOut out{xp, up, wp, Fc, Tc, Hist{hist, whist}};
    StageIO io{};
    io.acc = acc;
    io.pred = pred;
    io.Fh = Fh;
    io.Th = Th;
    int cur = 0;
    double t_since = 0.0;
    long long gs = 0;
    for (int sub = 0; sub < n_sub; ++sub)
        for (int k = 0; k < 3; ++k, ++gs) {
            const Stage S{dts, 2.0 * alpha[k], alpha[k], gamma_[k], zeta_[k]};
            io.Fcur = Fbuf[gs & 1];
            io.Fprev = Fbuf[(gs + 1) & 1];
            // contacts at the accepted state (committing its history), then s~
            io.rec = acc;
            io.hold = H[cur];
            io.hnew = H[1 - cur];
            hipLaunchKernelGGL(k_sub_stage<kStagePredict>, grid, dim3(kContactBlock), 0, s, P, np,
                               C, A, io, t_since, S, out);
            // contacts at s~, then s^k
            io.rec = pred;
            io.hold = H[1 - cur];
            hipLaunchKernelGGL(k_sub_stage<kStageCorrect>, grid, dim3(kContactBlock), 0, s, P, np,
                               C, A, io, S.a2 * dts, S, out);
            cur = 1 - cur;
            t_since = S.a2 * dts;
        }
    // the final state: positions, velocities, committed history and collision force
    io.rec = acc;
    io.hold = H[cur];
    hipLaunchKernelGGL(k_sub_stage<kStageForces>, grid, dim3(kContactBlock), 0, s, P, np, C, A, io,
                       t_since, Stage{}, out);
    return ibmx_launch_check();
}
