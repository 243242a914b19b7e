// Pair pass of the collision models (Secs. 2.2.5-2.2.8), FP64 throughout.
//
//   cell list   uniform cells of edge >= 2 R_max + gap_cut, particles listed
//               per cell by id (counting sort, then a per-cell sort);
//   pair list   one 27-cell search that counts and keeps each particle's
//               partners -> exclusive scan -> emit, sorted by id, so the list
//               is in (i, j) order and independent of thread scheduling;
//   wall list   (p, side) for every wall closer than gap_cut;
//   forces      lubrication, normal contact (linear or Hertz) and capped
//               tangential spring-dashpot (eq. f_int): a group of lanes per
//               particle evaluates its contacts, summed in partner order;
//   mask        the marker-disable rule, a wave per particle over its close
//               pairs and walls.
//
// Distances, gaps and cell indices are computed with the operation order
// documented in ibmx.h and without FMA contraction so that the integer
// outputs do not depend on the compiler's fusion choices.
#pragma clang fp contract(off)

#include <math.h>

#include "ibmx_contact.hpp"

namespace {

__device__ __forceinline__ void cell_coords(const PairC &P, const double *x, int *ci)
{
    for (int a = 0; a < 3; ++a) {
        double t = floor((x[a] - P.origin[a]) / P.edge[a]);
        int v = (int)t;
        if (t < 0.0)
            v = 0;
        if (t > (double)(P.nc[a] - 1))
            v = P.nc[a] - 1;
        ci[a] = v;
    }
}

// ---------------------------------------------------------------------------
// cell list
// ---------------------------------------------------------------------------
__global__ void k_cell_count(PairC P, int np, const double *xp, const double *radius,
                             double rmax, int *cell_of, int *count, int *err)
{
    int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= np)
        return;
    if (!(radius[p] <= rmax))
        atomicCAS(err, 0, (int)IBMX_EINVAL);
    double x[3];
    int ci[3];
    centre(P, np, xp, p, x);
    cell_coords(P, x, ci);
    int c = ci[0] + P.nc[0] * (ci[1] + P.nc[1] * ci[2]);
    cell_of[p] = c;
    atomicAdd(&count[c], 1);
}

__global__ void k_cell_scatter(int np, const int *cell_of, const int *start, int *cursor, int *cellp)
{
    int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= np)
        return;
    int c = cell_of[p];
    int pos = start[c] + atomicAdd(&cursor[c], 1);
    cellp[pos] = p;
}

// insertion sort of one segment (more partners than a search keeps)
__device__ void sort_segment(int *a, int n)
{
    for (int i = 1; i < n; ++i) {
        int v = a[i];
        int j = i - 1;
        while (j >= 0 && a[j] > v) {
            a[j + 1] = a[j];
            --j;
        }
        a[j + 1] = v;
    }
}

// a cell's particles by id: every particle counts the smaller ids of its cell
// (independent reads; an insertion sort per cell was a chain of memory round
// trips, 29 us on the 20,000-particle bed)
__global__ void k_cell_sort(int np, const int *cell_of, const int *start, const int *unsorted,
                            int *cellp)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= np)
        return;
    const int c = cell_of[p], s0 = start[c], s1 = start[c + 1];
    int rank = 0;
    for (int k = s0; k < s1; ++k)
        rank += unsorted[k] < p ? 1 : 0;
    cellp[s0 + rank] = p;
}

// ---------------------------------------------------------------------------
// pair search over the neighbouring cells (deduplicated when nc < 3), one
// wave per particle i.  The neighbours along x of one (y, z) row of cells are
// one range of the cell list (two across a seam), so there are 9 to 18 ranges;
// their candidates are numbered 0 .. total-1 through a wave prefix sum and
// dealt to the lanes, kSearch rounds of 64 at a time with their loads in flight
// together; visit(hit, j) is called for every 64 candidates, by the whole wave,
// with hit = a partner j > i closer than the cut-off.  What bounds it is the
// search of a candidate's range (27 cells' ranges read through the LDS crossbar,
// one round at a time, took 53 us on the 20,000-particle bed; 31 now).
// ---------------------------------------------------------------------------
constexpr int kSearch = 2;

template <class Visit>
__device__ __forceinline__ void search_partners(const PairC &P, int np, const double *xp,
                                                const double *radius, const int *cell_start,
                                                const int *cellp, int i, const double *xi,
                                                double Ri, Visit visit)
{
    const int lane = threadIdx.x & (IBMX_WAVE - 1);
    int ci[3];
    cell_coords(P, xi, ci);
    // cell rows along y and z (deduplicated)
    int offs[3][3], noff[3];
    for (int a = 1; a < 3; ++a) {
        noff[a] = 0;
        for (int d = -1; d <= 1; ++d) {
            int v = ci[a] + d;
            if (P.periodic[a]) {
                v = (v + P.nc[a]) % P.nc[a];
            } else if (v < 0 || v >= P.nc[a]) {
                continue;
            }
            bool dup = false;
            for (int k = 0; k < noff[a]; ++k)
                dup |= offs[a][k] == v;
            if (!dup)
                offs[a][noff[a]++] = v;
        }
    }
    // ranges of cells along x: [x0, x1], across a seam also the single cell xs
    const int nx = P.nc[0];
    int x0 = max(ci[0] - 1, 0), x1 = min(ci[0] + 1, nx - 1), xs = -1;
    if (P.periodic[0] && nx > 3) {
        if (ci[0] == 0)
            xs = nx - 1;
        else if (ci[0] == nx - 1)
            xs = 0;
    } else if (P.periodic[0]) {
        x0 = 0, x1 = nx - 1;   // every cell is a neighbour
    }
    const int nxr = xs >= 0 ? 2 : 1;
    const int nranges = __builtin_amdgcn_readfirstlane(nxr * noff[1] * noff[2]);
    // lane k < nranges holds range k and the number of candidates before it
    int c_first = 0, c_len = 0;
    if (lane < nranges) {
        const int kx = lane % nxr, ky = (lane / nxr) % noff[1], kz = lane / (nxr * noff[1]);
        const int row = nx * (offs[1][ky] + P.nc[1] * offs[2][kz]);
        c_first = cell_start[row + (kx == 0 ? x0 : xs)];
        c_len = cell_start[row + (kx == 0 ? x1 : xs) + 1] - c_first;
    }
    int c_pre = c_len;   // inclusive wave scan
    for (int d = 1; d < IBMX_WAVE / 2; d <<= 1) {
        const int v = __shfl_up(c_pre, d, IBMX_WAVE);
        if (lane >= d)
            c_pre += v;
    }
    const int total = __builtin_amdgcn_readlane(c_pre, nranges - 1);
    c_pre -= c_len;   // exclusive
    for (int t0 = 0; t0 < total; t0 += kSearch * IBMX_WAVE) {
        // the range k holding candidate t: the last k with c_pre[k] <= t
        int at[kSearch], j[kSearch];
        for (int k = 0; k < nranges; ++k) {
            const int pk = __builtin_amdgcn_readlane(c_pre, k);
            const int fk = __builtin_amdgcn_readlane(c_first, k) - pk;
#pragma unroll
            for (int q = 0; q < kSearch; ++q) {
                const int t = t0 + q * IBMX_WAVE + lane;
                at[q] = pk <= t ? fk + t : at[q];
            }
        }
#pragma unroll
        for (int q = 0; q < kSearch; ++q)
            j[q] = cellp[t0 + q * IBMX_WAVE + lane < total ? at[q] : 0];
        double xj[kSearch][3], Rj[kSearch];
#pragma unroll
        for (int q = 0; q < kSearch; ++q) {
            for (int a = 0; a < 3; ++a)
                xj[q][a] = xp[(size_t)a * np + j[q]];
            Rj[q] = radius[j[q]];
        }
#pragma unroll
        for (int q = 0; q < kSearch; ++q) {
            bool hit = false;
            if (t0 + q * IBMX_WAVE + lane < total && j[q] > i) {
                double d[3];
                for (int a = 0; a < 3; ++a)
                    if (P.periodic[a])
                        xj[q][a] = wrap_pos(xj[q][a], P.origin[a], P.L[a]);
                const double d2 = disp2(P, xi, xj[q], d);
                double cut = Ri + Rj[q];
                cut = cut + P.gap_cut;
                hit = d2 < cut * cut;
            }
            visit(hit, j[q]);
        }
    }
}

// Search and counts: the first kKept partners of every particle are kept
// (found[i][kKept], in search order) and its walls counted by the wave's first
// six lanes, so that the lists need no second search.
constexpr int kKept = IBMX_KEPT_PARTNERS;

// gap of particle p to wall `side` (2 axis + upper); true when it is listed
__device__ __forceinline__ bool wall_gap_of(const PairC &P, int np, const double *xp, double R,
                                            int p, int side, double *g)
{
    bool in = false;
    for (int a = 0; a < 3; ++a) {
        if (P.periodic[a] || side / 2 != a)
            continue;
        const double x = xp[(size_t)a * np + p];
        const double top = P.origin[a] + P.L[a];
        const double dist = (side & 1) == 0 ? (x - P.origin[a]) : (top - x);
        *g = dist - R;
        in = *g < P.gap_cut;
    }
    return in;
}

__global__ __launch_bounds__(256) void k_pairs_count(PairC P, int np, const double *xp,
                                                     const double *radius, const int *cell_start,
                                                     const int *cellp, int *count, int *wcount,
                                                     int *found)
{
    const int lane = threadIdx.x & (IBMX_WAVE - 1);
    const int i = blockIdx.x * (blockDim.x / IBMX_WAVE) +
                  __builtin_amdgcn_readfirstlane(threadIdx.x / IBMX_WAVE);
    if (i >= np)
        return;
    double xi[3];
    centre(P, np, xp, i, xi);
    const double Ri = radius[i];
    int cnt = 0;
    search_partners(P, np, xp, radius, cell_start, cellp, i, xi, Ri, [&](bool hit, int j) {
        const unsigned long long m = __ballot(hit);
        const int pos = cnt + __popcll(m & ((1ULL << lane) - 1ULL));
        if (hit && pos < kKept)
            found[(size_t)i * kKept + pos] = j;
        cnt += __popcll(m);
    });
    double g = 0.0;
    const bool wall = lane < 6 && wall_gap_of(P, np, xp, Ri, i, lane, &g);
    const int nw = __popcll(__ballot(wall));
    if (lane == 0) {
        count[i] = cnt;
        wcount[i] = nw;
    }
}

// The lists: a wave per particle orders its kept partners by id (each lane
// counts the smaller ones) and writes them with their gaps, then its walls; a
// particle with more partners than were kept searches again.  Where the list is
// too short it holds the first entries in (i, j) order.  The first wave also
// writes the totals.
__global__ __launch_bounds__(256) void k_pairs_emit(PairC P, int np, const double *xp,
                                                    const double *radius, const int *cell_start,
                                                    const int *cellp, const int *found,
                                                    const int *off, int cap, int *pairs_out,
                                                    double *gap_out, const int *woff, int wcap,
                                                    int *walls_out, double *wgap_out,
                                                    int *counts_out, int *err)
{
    const int lane = threadIdx.x & (IBMX_WAVE - 1);
    const int i = blockIdx.x * (blockDim.x / IBMX_WAVE) +
                  __builtin_amdgcn_readfirstlane(threadIdx.x / IBMX_WAVE);
    if (i == 0 && lane == 0) {
        counts_out[0] = off[np];
        counts_out[1] = woff[np];
        if (off[np] > cap || woff[np] > wcap)
            atomicCAS(err, 0, (int)IBMX_ECAPACITY);
    }
    if (i >= np)
        return;
    double xi[3];
    centre(P, np, xp, i, xi);
    const double Ri = radius[i];
    const int base = off[i], cnt = off[i + 1] - base;
    auto gap_to = [&](int j) {
        double xj[3], d[3];
        centre(P, np, xp, j, xj);
        double d2 = disp2(P, xi, xj, d);
        double g = sqrt(d2) - Ri;
        return g - radius[j];
    };
    if (cnt > 0 && cnt <= kKept) {
        const int j = lane < cnt ? found[(size_t)i * kKept + lane] : -1;
        int rank = 0;
        for (int k = 0; k < cnt; ++k)
            rank += __builtin_amdgcn_readlane(j, k) < j ? 1 : 0;
        const int pos = base + rank;
        if (lane < cnt && pos < cap) {
            pairs_out[pos] = i;
            pairs_out[cap + pos] = j;
            gap_out[pos] = gap_to(j);
        }
    } else if (cnt > kKept && base < cap) {
        // searched again, in candidate order into the scratch half of pairs_out,
        // then sorted and completed by lane 0; where the list's end cuts the
        // particle's partners, those of the smallest ids: up to `last`, found by
        // bisection (for one particle of a call at most)
        const int n = min(cnt, cap - base);
        int last = np - 1, below = i;
#pragma unroll 1
        for (bool probe = true; probe;) {
            probe = n < cnt && below + 1 < last;
            const int upto = probe ? below + (last - below) / 2 : last;
            int at = 0;
            search_partners(P, np, xp, radius, cell_start, cellp, i, xi, Ri, [&](bool hit, int j) {
                hit = hit && j <= upto;
                const unsigned long long m = __ballot(hit);
                const int pos = base + at + __popcll(m & ((1ULL << lane) - 1ULL));
                if (hit && !probe)
                    pairs_out[cap + pos] = j;
                at += __popcll(m);
            });
            if (probe)
                (at >= n ? last : below) = upto;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        if (lane == 0) {
            sort_segment(pairs_out + cap + base, n);
            for (int k = 0; k < n; ++k) {
                pairs_out[base + k] = i;
                gap_out[base + k] = gap_to(pairs_out[cap + base + k]);
            }
        }
    }
    double g = 0.0;
    const bool wall = lane < 6 && wall_gap_of(P, np, xp, Ri, i, lane, &g);
    const unsigned long long m = __ballot(wall);
    const int pos = woff[i] + __popcll(m & ((1ULL << lane) - 1ULL));
    if (wall && pos < wcap) {
        walls_out[pos] = i;
        walls_out[wcap + pos] = lane;
        wgap_out[pos] = g;
    }
}

// previous-call history of pair (i, j): binary search in the (i, j)-sorted list
__device__ int find_pair(int n_in, const int *pairs_in, int i, int j)
{
    long long key = ((long long)i << 32) | (unsigned)j;
    int lo = 0, hi = n_in - 1;
    while (lo <= hi) {
        int mid = (lo + hi) >> 1;
        long long k = ((long long)pairs_in[mid] << 32) | (unsigned)pairs_in[n_in + mid];
        if (k == key)
            return mid;
        if (k < key)
            lo = mid + 1;
        else
            hi = mid - 1;
    }
    return -1;
}

// previous-call history of wall entry (p, side): binary search in the
// (p, side)-sorted list
__device__ int find_wall(int n_in, const int *walls_in, int p, int side)
{
    long long key = (long long)p * 8 + side;
    int lo = 0, hi = n_in - 1;
    while (lo <= hi) {
        int mid = (lo + hi) >> 1;
        long long k = (long long)walls_in[mid] * 8 + walls_in[n_in + mid];
        if (k == key)
            return mid;
        if (k < key)
            lo = mid + 1;
        else
            hi = mid - 1;
    }
    return -1;
}

// history of the previous call, aligned with the new lists (zero for new
// contacts)
__global__ void k_hist_align(ContactLists C, int n_in, const int *pairs_in, const double *hist_in,
                             int nw_in, const int *walls_in, const double *whist_in, Hist hold)
{
    const int npairs = n_pairs(C), nwall = n_walls(C);
    for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < npairs + nwall;
         k += gridDim.x * blockDim.x) {
        if (k < npairs) {
            const int kin = n_in > 0 ? find_pair(n_in, pairs_in, C.pairs[k], C.pairs[C.pair_cap + k])
                                     : -1;
            for (int a = 0; a < kHist; ++a)
                hold.pair[(size_t)a * C.pair_cap + k] =
                    kin >= 0 ? hist_in[(size_t)a * n_in + kin] : 0.0;
        } else {
            const int kw = k - npairs;
            const int kin =
                nw_in > 0 ? find_wall(nw_in, walls_in, C.walls[kw], C.walls[C.wall_cap + kw]) : -1;
            for (int a = 0; a < kHist; ++a)
                hold.wall[(size_t)a * C.wall_cap + kw] =
                    kin >= 0 ? whist_in[(size_t)a * nw_in + kin] : 0.0;
        }
    }
}

__device__ __forceinline__ BodyState body_state(int np, const double *xp, const double *up,
                                                const double *wp, const double *radius, int p)
{
    BodyState s;
    for (int a = 0; a < 3; ++a) {
        const size_t i = (size_t)a * np + p;
        s.x[a] = xp[i];
        s.u[a] = up[i];
        s.w[a] = wp[i];
    }
    s.R = radius[p];
    return s;
}

// ---------------------------------------------------------------------------
// contact forces and torques of every particle (Fc, Tc, or null) and the new
// history, written by each pair's first particle and each wall's particle
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kContactBlock) void k_contact_forces(
    PairC P, int np, ContactLists C, const int *__restrict__ off, const int2 *__restrict__ adj,
    const double *__restrict__ xp, const double *__restrict__ up, const double *__restrict__ wp,
    const double *__restrict__ radius, const double *__restrict__ mass, Hist hold, Hist hnew,
    double *__restrict__ Fc, double *__restrict__ Tc)
{
    __shared__ double part[kContactBlock][6];
    const int j = threadIdx.x % kContactLanes;
    const int p = blockIdx.x * kContactParticles + threadIdx.x / kContactLanes;
    int lo = 0, deg = 0;
    if (p < np) {
        lo = off[p];
        deg = off[p + 1] - lo;
    }
    double acc = 0.0;
    for (int c = 0; __any(c * kContactLanes < deg); ++c) {
        const int r = c * kContactLanes + j;
        if (r < deg) {
            const int2 e = adj[lo + r];
            double ho[kHist], hn[kHist];
            ContactGeom G;
            ContactConst K;
            const bool pair = e.x >= 0, second = pair && (e.x & 1);
            const int k = pair ? e.x >> 1 : -e.x - 1;
            if (pair) {
                for (int a = 0; a < kHist; ++a)
                    ho[a] = hold.pair[(size_t)a * C.pair_cap + k];
                const int i1 = second ? e.y : p, i2 = second ? p : e.y;
                const BodyState s1 = body_state(np, xp, up, wp, radius, i1);
                const BodyState s2 = body_state(np, xp, up, wp, radius, i2);
                pair_geometry(P, s1, s2, G);
                K = pair_const(P, mass[i1], s1.R, mass[i2], s2.R);
            } else {
                for (int a = 0; a < kHist; ++a)
                    ho[a] = hold.wall[(size_t)a * C.wall_cap + k];
                const BodyState s1 = body_state(np, xp, up, wp, radius, p);
                wall_geometry(P, s1, e.y, G);
                K = wall_const(P, mass[p], s1.R);
            }
            contact_force(P, G, K, second, ho, P.dt, part[threadIdx.x], hn);
            if (pair && !second && hnew.pair)
                for (int a = 0; a < kHist; ++a)
                    hnew.pair[(size_t)a * C.pair_cap + k] = hn[a];
            if (!pair && hnew.wall)
                for (int a = 0; a < kHist; ++a)
                    hnew.wall[(size_t)a * C.wall_cap + k] = hn[a];
        }
        __syncthreads();
        acc = chunk_sum(part, j, deg - c * kContactLanes, acc);
        __syncthreads();
    }
    if (p >= np || j >= 6 || !Fc)
        return;
    if (j < 3)
        Fc[(size_t)j * np + p] = acc;
    else
        Tc[(size_t)(j - 3) * np + p] = acc;
}

// ---------------------------------------------------------------------------
// marker-disable mask
// ---------------------------------------------------------------------------
__device__ __forceinline__ unsigned long long splitmix64(unsigned long long x)
{
    unsigned long long z = x + 0x9e3779b97f4a7c15ULL;
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ULL;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebULL;
    return z ^ (z >> 31);
}

// One wave per particle writes its markers' mask: 1, or 0 where the rule drops
// the marker.  The particle's close pairs in which it is the chosen one (from
// its adjacency, kMaskPart at a time in LDS) and its close walls are gathered
// first, so that the marker offsets are read once, and only where there are
// any; MUNR rounds of them are loaded before any test (four at five waves per
// SIMD: eight took 195 VGPRs and 83 us).  20,000-particle bed: 41 us against 56
// for clearing the mask and a wave per pair and per wall.
constexpr int MUNR = 4;        // marker rounds per batch of offset loads
constexpr int kMaskPart = IBMX_WAVE;

__global__ __launch_bounds__(256, 5) void k_mask(PairC P, int np, int nm, const int *moff,
                                              const double *body, const double *xp,
                                              const double *radius, int mode,
                                              unsigned long long seed, const int *off,
                                              const int2 *adj, const double *gap,
                                              const double *wgap, uint8_t *mask)
{
    __shared__ double part[4][kMaskPart][4];
    const int lane = threadIdx.x & (IBMX_WAVE - 1);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / IBMX_WAVE);
    const int p = blockIdx.x * 4 + wv;
    if (p >= np)
        return;
    const int l0 = moff[p], l1 = moff[p + 1], e0 = off[p], e1 = off[p + 1];
    double xc[3], xw[3];
    centre(P, np, xp, p, xc);
    for (int a = 0; a < 3; ++a)
        xw[a] = xp[(size_t)a * np + p];
    bool first = true;
    for (int eb = e0; eb < e1 || first; eb += kMaskPart) {
        // this chunk's partners whose surface drops markers, and walls
        int q = -1, side = -1;
        if (eb + lane < e1) {
            const int2 e = adj[eb + lane];
            if (e.x >= 0) {
                const int i = (e.x & 1) ? e.y : p, j = (e.x & 1) ? p : e.y;
                const unsigned long long key =
                    ((unsigned long long)(unsigned)i << 32) | (unsigned long long)(unsigned)j;
                const int chosen = (splitmix64(seed ^ key) & 1ULL) == 0 ? i : j;
                if (chosen == p && gap[e.x >> 1] < 2.0 * P.eps_sep)
                    q = e.y;
            } else if (wgap[-e.x - 1] < P.eps_sep) {
                side = e.y;
            }
        }
        const unsigned long long mq = __ballot(q >= 0);
        const int nq = __popcll(mq);
        if (q >= 0) {
            double xq[3];
            centre(P, np, xp, q, xq);
            const double lim = radius[q] + 2.0 * P.eps_sep;
            double *d = part[wv][__popcll(mq & ((1ULL << lane) - 1ULL))];
            d[0] = xq[0];
            d[1] = xq[1];
            d[2] = xq[2];
            d[3] = lim * lim;
        }
        bool near[6];
        bool walls = false;
        for (int w = 0; w < 6; ++w) {
            near[w] = __ballot(side == w) != 0;
            walls |= near[w];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (nq == 0 && !walls) {
            if (first)
                for (int l = l0 + lane; l < l1; l += IBMX_WAVE)
                    mask[l] = 1;
        } else if (mode == 2) {
            for (int l = l0 + lane; l < l1; l += IBMX_WAVE)
                mask[l] = 0;
        } else {
            for (int lb = l0 + lane; lb < l1; lb += MUNR * IBMX_WAVE) {
                double o[MUNR][3];
                bool drop[MUNR];
#pragma unroll
                for (int r = 0; r < MUNR; ++r) {
                    const int l = min(lb + r * IBMX_WAVE, l1 - 1);
#pragma unroll
                    for (int a = 0; a < 3; ++a)
                        o[r][a] = body[(size_t)a * nm + l];
                    drop[r] = false;
                }
                for (int k = 0; k < nq; ++k) {
                    const double *xq = part[wv][k];
#pragma unroll
                    for (int r = 0; r < MUNR; ++r) {
                        double d[3];
#pragma unroll
                        for (int a = 0; a < 3; ++a) {
                            d[a] = (xc[a] + o[r][a]) - xq[a];
                            if (P.periodic[a])
                                d[a] = min_image(d[a], P.L[a]);
                        }
                        double d2 = d[0] * d[0];
                        d2 = d2 + d[1] * d[1];
                        d2 = d2 + d[2] * d[2];
                        drop[r] |= d2 < xq[3];
                    }
                }
                if (walls)
                    for (int a = 0; a < 3; ++a) {
                        const double top = P.origin[a] + P.L[a];
#pragma unroll
                        for (int r = 0; r < MUNR; ++r) {
                            const double X = xw[a] + o[r][a];
                            drop[r] |= near[2 * a] && X - P.origin[a] < P.eps_sep;
                            drop[r] |= near[2 * a + 1] && top - X < P.eps_sep;
                        }
                    }
#pragma unroll
                for (int r = 0; r < MUNR; ++r) {
                    const int l = lb + r * IBMX_WAVE;
                    if (l < l1 && (first || drop[r]))
                        mask[l] = drop[r] ? 0 : 1;
                }
            }
        }
        first = false;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

int blocks(long long n, int b = 256) { return (int)((n + b - 1) / b) > 0 ? (int)((n + b - 1) / b) : 1; }

}  // namespace

extern "C" ibmx_status ibmx_pairs(ibmx_plan p, const double *xp, const double *radius,
                                  double rmax, const double *mass, const double *up, const double *wp,
                                  int32_t npairs_in, const int32_t *pairs_in, const double *hist_in,
                                  int32_t nwall_in, const int32_t *walls_in, const double *whist_in,
                                  int32_t *cell_start, int32_t cell_cap, int32_t *cell_particles,
                                  int32_t *pairs_out, double *pair_gap, double *hist_out,
                                  int32_t pair_cap, int32_t *walls_out, double *wall_gap,
                                  double *whist_out, int32_t wall_cap, int32_t *counts_out,
                                  double *Fc, double *Tc, uint8_t *marker_active)
{
    if (!p)
        return IBMX_EINVAL;
    const int np = p->np, nm = p->nm;
    if (np > 0 && (!xp || !radius || !mass || !up || !wp || !cell_particles || !Fc || !Tc))
        return IBMX_EINVAL;
    if (!cell_start || !counts_out || pair_cap < 0 || wall_cap < 0 || npairs_in < 0 || nwall_in < 0)
        return IBMX_EINVAL;
    if ((pair_cap > 0 && (!pairs_out || !pair_gap || !hist_out)) ||
        (wall_cap > 0 && (!walls_out || !wall_gap || !whist_out)) ||
        (npairs_in > 0 && (!pairs_in || !hist_in)) || (nwall_in > 0 && (!walls_in || !whist_in)))
        return IBMX_EINVAL;
    if (marker_active && nm > 0 && !p->body)
        return IBMX_ESTATE;
    const ibmx_params &prm = p->prm;
    PairC P;
    contact_constants(p, &P);
    if (np > 0 && !(rmax > 0.0 && isfinite(rmax)))
        return IBMX_EINVAL;
    long long ncell = 1;
    for (int a = 0; a < 3; ++a) {
        int k = (int)floor(P.L[a] / (2.0 * rmax + P.gap_cut));
        P.nc[a] = k < 1 ? 1 : k;
        P.edge[a] = P.L[a] / P.nc[a];
        ncell *= P.nc[a];
    }
    if (ncell + 1 > cell_cap)
        return IBMX_ECAPACITY;
    P.ncell = (int)ncell;
    // the workspace comes from ibmx_plan_reserve: this call allocates nothing
    if (!p->p_cursor || p->p_cell_cap < ncell || p->scan_cap < ncell || p->scan_cap < np ||
        !ibmx_contact_ready(p, pair_cap, wall_cap, 1))
        return IBMX_ESTATE;
    hipStream_t s = p->stream;
    ProfScope ps(p, IBMX_K_PAIRS);
    // cell list
    ZeroList z = {};
    z.add(cell_start, ncell + 1);
    z.add(p->p_cursor, ncell);
    ibmx_zero_i32_multi(z, s);
    if (np > 0)
        hipLaunchKernelGGL(k_cell_count, dim3(blocks(np)), dim3(256), 0, s, P, np, xp, radius,
                           rmax, p->p_cell_of, cell_start, p->d_err);
    ibmx_exclusive_scan(cell_start, cell_start, (int)ncell, p->scan_aux, s);
    if (np > 0) {
        // p_off holds the unsorted cell list until the scan writes it
        hipLaunchKernelGGL(k_cell_scatter, dim3(blocks(np)), dim3(256), 0, s, np, p->p_cell_of,
                           cell_start, p->p_cursor, p->p_off);
        hipLaunchKernelGGL(k_cell_sort, dim3(blocks(np)), dim3(256), 0, s, np,
                           (const int *)p->p_cell_of, (const int *)cell_start,
                           (const int *)p->p_off, cell_particles);
        // pair and wall lists
        hipLaunchKernelGGL(k_pairs_count, dim3(blocks(np, 4)), dim3(256), 0, s, P, np, xp, radius,
                           (const int *)cell_start, (const int *)cell_particles, p->p_count,
                           p->p_wcount, p->p_found);
    }
    ibmx_exclusive_scan2(p->p_count, p->p_off, p->p_wcount, p->p_woff, np, p->scan_aux, s);
    hipLaunchKernelGGL(k_pairs_emit, dim3(blocks(np, 4)), dim3(256), 0, s, P, np, xp, radius,
                       (const int *)cell_start, (const int *)cell_particles,
                       (const int *)p->p_found, (const int *)p->p_off, pair_cap, pairs_out,
                       pair_gap, (const int *)p->p_woff, wall_cap, walls_out, wall_gap, counts_out,
                       p->d_err);
    // forces: previous history aligned with the new lists, per-particle
    // adjacency, then a group of lanes per particle
    const ContactLists C{pair_cap, wall_cap, pairs_out, walls_out, counts_out};
    const Hist hold{p->c_hist, p->c_hist + (size_t)kHist * pair_cap};
    {
        const long long nmax = (long long)pair_cap + wall_cap;
        const int g = blocks(nmax) < 4096 ? blocks(nmax) : 4096;
        hipLaunchKernelGGL(k_hist_align, dim3(g), dim3(256), 0, s, C, npairs_in, pairs_in, hist_in,
                           nwall_in, walls_in, whist_in, hold);
    }
    contact_adjacency(p, C, s);
    if (np > 0)
        hipLaunchKernelGGL(k_contact_forces, dim3(blocks(np, kContactParticles)),
                           dim3(kContactBlock), 0, s, P, np, C, (const int *)p->c_off,
                           (const int2 *)p->c_adj, xp, up, wp, radius, mass, hold,
                           Hist{hist_out, whist_out}, Fc, Tc);
    // mask
    if (marker_active && nm > 0) {
        if (prm.disable_mode == 0)
            ibmx_fill_u8(marker_active, 1, nm, s);
        else
            hipLaunchKernelGGL(k_mask, dim3(blocks(np, 4)), dim3(256), 0, s, P, np, nm,
                               (const int *)p->d_moff, p->body, xp, radius, prm.disable_mode,
                               (unsigned long long)prm.disable_seed, (const int *)p->c_off,
                               (const int2 *)p->c_adj, (const double *)pair_gap,
                               (const double *)wall_gap, marker_active);
    }
    return ibmx_launch_check();
}
