// Fluid integrals over each particle with the level-set volume fraction
// (Sec. 2.2.9), and the volume average of a grid field (Sec. 2.2.4).
#include <math.h>

#include <mutex>

#include "ibmx_internal.hpp"

namespace {

constexpr int MEAN_BLOCKS = 4096;

// Square root of s > 0 by the hardware's reciprocal root (about 2^-23) and two
// Goldschmidt-Markstein steps: within an ulp, without the range scaling of the
// library's (a squared distance in cells is far from the range's ends).
__device__ __forceinline__ double root(double s)
{
    const double y = __builtin_amdgcn_rsq(s);
    double g = s * y, q = 0.5 * y;
    const double r = fma(-q, g, 0.5);
    g = fma(g, r, g);
    q = fma(q, r, q);
    g = fma(fma(-g, g, s), q, g);
    return fma(fma(-g, g, s), q, g);
}

// Volume fraction of the cell whose lowest corner is c0 (relative to the
// particle centre) in a sphere of radius R: the signed corner distances
// phi_m = |x_m - x_p| - R give alpha = sum -phi_m H(-phi_m) / sum |phi_m|; any:
// whether a corner is inside (alpha > 0).
__device__ __forceinline__ double cell_alpha(const double *c0, double h, double R, bool &any)
{
    double sq[3][2];
    for (int a = 0; a < 3; ++a) {
        const double c1 = c0[a] + h;
        sq[a][0] = c0[a] * c0[a];
        sq[a][1] = c1 * c1;
    }
    double num = 0.0, den = 0.0;
#pragma unroll
    for (int m = 0; m < 8; ++m) {
        const double s = sq[0][m & 1] + sq[1][(m >> 1) & 1] + sq[2][(m >> 2) & 1];
        const double phi = root(fmax(s, 1e-280)) - R;
        num += fmax(-phi, 0.0);
        den += fabs(phi);
    }
    any = num > 0.0;
    return den > 0.0 ? num / den : 0.0;
}

// Rows' steps a lane sums over before it adds them to its total (BLOCKS): the
// inside cells' sums drift with the velocity's mean, and a chain of all of a
// lane's cells (some 110 in a sphere of 24 cells taken by one wave) rounds at the
// size of its total each time.  With sixteen waves a chain is shorter than a block
// (24 cells: 7), or that much shorter than with fewer.
constexpr int kFlush = 16;

// Wave pw of nw's share of one particle's sums, in every lane: s[0..2] of alpha
// u, s[3..5] of alpha r x u.  A wave takes whole x rows of the particle's
// bounding box, as many at a time as fit its lanes.  Cells whose centre lies
// deeper than half a cell diagonal inside (outside) the surface have every
// corner inside (outside) and take alpha = 1 (0), which is what the corner
// formula gives for them; the test compares squared distances.  The cells in
// between (a third of the box) need eight corner distances: they are collected
// in the wave's LDS list (their box indices) and taken 64 at a time, so that no
// lane idles through the square roots of another's cell.
template <typename T, bool O32, bool BLOCKS>
__device__ __forceinline__ void sphere_sums(const GridC &g, int np, int p, int pw, int nw,
                                            const double *__restrict__ xp,
                                            const double *__restrict__ radius,
                                            const T *__restrict__ u, T *__restrict__ alpha_out,
                                            int (*list)[2 * IBMX_WAVE],
                                            double (*inner)[IBMX_WAVE], double *s)
{
    const int lane = threadIdx.x & (IBMX_WAVE - 1);
    const double h = g.h, half_diag = 0.5 * sqrt(3.0) * h;
    const double R = radius[p];
    double x[3];
    int lo[3], ext[3];
    bool wraps[3];   // whether the box leaves the grid (through a seam)
    for (int a = 0; a < 3; ++a) {
        x[a] = xp[(size_t)a * np + p];
        if (g.periodic[a]) {
            const double L = g.n[a] * h;
            x[a] = x[a] - floor((x[a] - g.origin[a]) / L) * L;
        }
        // cells beyond a wall do not count; a particle over a whole periodic
        // axis (which is not allowed) stays within one period; one whose centre
        // or radius is not finite has no cells (fmax and fmin drop a NaN)
        const double c0 = floor((x[a] - R - g.origin[a]) / h);
        const double c1 = floor((x[a] + R - g.origin[a]) / h);
        const double first = fmax(c0, g.periodic[a] ? -g.n[a] : 0.0);
        const double end = isfinite(c1 - c0)
                               ? fmin(c1 + 1.0, g.periodic[a] ? first + g.n[a] : g.n[a])
                               : first;
        lo[a] = __builtin_amdgcn_readfirstlane((int)first);
        ext[a] = __builtin_amdgcn_readfirstlane(end > first ? (int)(end - first) : 0);
        wraps[a] = lo[a] < 0 || lo[a] + ext[a] > g.n[a];
    }
    const double r_in = R - half_diag, r_out = R + half_diag;
    const double r_in2 = r_in > 0.0 ? r_in * r_in : -1.0, r_out2 = r_out * r_out;
    const T *const ub[3] = {u, u + g.nodes, u + 2 * g.nodes};
    for (int k = 0; k < 6; ++k) {
        s[k] = 0.0;
        if (BLOCKS)
            inner[k][lane] = 0.0;
    }
    // lowest corner of cell i along axis a, relative to the centre, and its node
    auto corner = [&](int a, int i) { return g.origin[a] + (lo[a] + i) * h - x[a]; };
    auto node = [&](int a, int i) {
        int c = lo[a] + i;
        if (wraps[a])
            c += (c < 0 ? g.n[a] : 0) - (c >= g.n[a] ? g.n[a] : 0);
        return (unsigned)c;
    };
    auto value = [&](int a, unsigned gi) {
        if (O32)
            return (double)*reinterpret_cast<const T *>(reinterpret_cast<const char *>(ub[a]) +
                                                        gi * (unsigned)sizeof(T));
        return (double)ub[a][(size_t)gi];
    };
    // n listed cells from `first` on, one per lane
    auto take = [&](int first, int n) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (lane < n) {
            const int i[3] = {list[0][first + lane], list[1][first + lane], list[2][first + lane]};
            const unsigned gi =
                (node(2, i[2]) * (unsigned)g.n[1] + node(1, i[1])) * (unsigned)g.n[0] + node(0, i[0]);
            // the cell's velocity is in flight during the square roots
            double uc[3] = {value(0, gi), value(1, gi), value(2, gi)};
            double c0[3], r[3];
            for (int a = 0; a < 3; ++a) {
                c0[a] = corner(a, i[a]);
                r[a] = c0[a] + 0.5 * h;
            }
            bool any;
            const double alpha = cell_alpha(c0, h, R, any);
            // a listed cell may still have all its corners outside: whatever the
            // field holds there (0 * inf) stays out (selected while the division
            // is under way: a branch on alpha cost 4 %)
            for (int a = 0; a < 3; ++a)
                uc[a] = any ? uc[a] : 0.0;
            const double w[3] = {alpha * uc[0], alpha * uc[1], alpha * uc[2]};
            s[0] += w[0];
            s[1] += w[1];
            s[2] += w[2];
            s[3] += r[1] * w[2] - r[2] * w[1];
            s[4] += r[2] * w[0] - r[0] * w[2];
            s[5] += r[0] * w[1] - r[1] * w[0];
            if (alpha_out && any)
                atomicAdd(&alpha_out[gi], (T)alpha);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    int listed = 0;
    // rows per step
    const int rpi = ext[0] > 0 && ext[0] < IBMX_WAVE ? IBMX_WAVE / ext[0] : 1;
    const int sub = rpi > 1 ? lane / ext[0] : 0, lx = rpi > 1 ? lane - sub * ext[0] : lane;
    const int rows = ext[1] * ext[2], step = nw * rpi;
    for (int x0 = 0; x0 < (rows > 0 ? ext[0] : 0); x0 += IBMX_WAVE) {
        const int ix = x0 + lx;
        const bool inx = (sub < rpi) & (ix < ext[0]);
        const unsigned gx = node(0, ix);
        const double rx = corner(0, ix) + 0.5 * h, rx2 = rx * rx;
        int iz = (pw * rpi + sub) / ext[1], iy = (pw * rpi + sub) - iz * ext[1];
        const int sz = step / ext[1], sy = step - sz * ext[1];
        // sums over the lane's inside cells: of u, and of the parts of r x u
        // that change along them (r_x is the lane's own)
        double v[3] = {0.0, 0.0, 0.0}, m[3] = {0.0, 0.0, 0.0};
        auto flush = [&]() {
            const double add[6] = {v[0], v[1], v[2], m[0], m[1] - rx * v[2], rx * v[1] - m[2]};
#pragma unroll
            for (int k = 0; k < 6; ++k)
                if (BLOCKS)
                    inner[k][lane] += add[k];
                else
                    s[k] += add[k];
            for (int a = 0; a < 3; ++a)
                v[a] = m[a] = 0.0;
        };
        int steps = 0;
        for (int r0 = pw * rpi; r0 < rows; r0 += step) {
            const double ry = corner(1, iy) + 0.5 * h, rz = corner(2, iz) + 0.5 * h;
            const double dc2 = rx2 + ry * ry + rz * rz;
            const bool ok = inx & (iz < ext[2]);
            const bool inside = ok & (dc2 <= r_in2), edge = ok & !inside & (dc2 < r_out2);
            if (inside) {
                const unsigned gi =
                    (node(2, iz) * (unsigned)g.n[1] + node(1, iy)) * (unsigned)g.n[0] + gx;
                const double uc[3] = {value(0, gi), value(1, gi), value(2, gi)};
                v[0] += uc[0];
                v[1] += uc[1];
                v[2] += uc[2];
                m[0] += ry * uc[2] - rz * uc[1];
                m[1] += rz * uc[0];
                m[2] += ry * uc[0];
                if (alpha_out)
                    atomicAdd(&alpha_out[gi], T(1));
            }
            const unsigned long long mk = __ballot(edge);
            if (edge) {
                const int at = listed + __popcll(mk & ((1ull << lane) - 1ull));
                list[0][at] = ix;
                list[1][at] = iy;
                list[2][at] = iz;
            }
            listed += __popcll(mk);
            if (listed >= IBMX_WAVE) {
                listed -= IBMX_WAVE;
                take(listed, IBMX_WAVE);
            }
            if (BLOCKS && ++steps == kFlush) {
                flush();
                steps = 0;
            }
            iy += sy;
            iz += sz;
            if (iy >= ext[1]) {
                iy -= ext[1];
                ++iz;
            }
        }
        flush();
    }
    if (listed > 0)
        take(0, listed);
#pragma unroll
    for (int k = 0; k < 6; ++k)
        s[k] = wave_sum(BLOCKS ? s[k] + inner[k][lane] : s[k]);
}

// The integrals of every particle: WP waves each, or (WP = 1) a wave each, four
// to a workgroup; spheres wider than `width` cells then get a workgroup of
// their own, from a second range of workgroups, one per particle, of which the
// others return at once (5000 spheres with one of 100 cells: 2.3 ms, with one
// wave for it 8.5, with 256 threads for every particle 3.9; looking through the
// four spheres inside one workgroup cost the bed below another 10 to 20 us in
// registers).  FP64 sums: per lane in a fixed order, over lanes and waves by fixed
// trees.
// Bound by FP64 instructions: the 20,000 spheres of a 512^3 bed, FP32 field,
// 307 us against 641 with a thread per cell of the box (divisions for the
// cell's indices, and every wave that met the surface ran the corners for
// all); four waves a particle there take 349 (part-filled lists).
template <typename T, int WP, bool O32>
__global__ __launch_bounds__(WP == 1 ? 256 : 64 * WP) void k_particle_integrals(
    GridC g, int np, double width, const double *__restrict__ xp,
    const double *__restrict__ radius, const T *__restrict__ u, double *__restrict__ Iu,
    double *__restrict__ Ir, T *__restrict__ alpha_out)
{
    constexpr int NW = WP == 1 ? 4 : WP;             // waves per workgroup
    __shared__ int s_list[NW][3][2 * IBMX_WAVE];
    __shared__ double s_inner[WP < 16 ? NW : 1][6][IBMX_WAVE];
    __shared__ double part[6][NW];
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / IBMX_WAVE);
    const int lane = threadIdx.x & (IBMX_WAVE - 1);
    const double h3 = g.h * g.h * g.h;
    auto write = [&](int p, const double *s) {
        for (int k = 0; k < 3; ++k) {
            Iu[(size_t)k * np + p] = h3 * s[k];
            Ir[(size_t)k * np + p] = h3 * s[3 + k];
        }
    };
    // WP = 1: a workgroup per four spheres, then one per sphere for the wide ones
    const int nb = WP == 1 ? (np + NW - 1) / NW : 0;
    const bool shared = (int)blockIdx.x >= nb;
    const int p = __builtin_amdgcn_readfirstlane(shared ? blockIdx.x - nb : blockIdx.x * NW + wv);
    if (WP == 1 && (p >= np || (2.0 * radius[p] > width * g.h) != shared))
        return;
    double s[6];
    sphere_sums<T, O32, (WP < 16)>(g, np, p, shared ? wv : 0, shared ? NW : 1, xp, radius, u,
                                   alpha_out, s_list[wv], s_inner[WP < 16 ? wv : 0], s);
    if (shared) {
        if (lane == 0)
            for (int k = 0; k < 6; ++k)
                part[k][wv] = s[k];
        __syncthreads();
        if (wv != 0)
            return;
        for (int k = 0; k < 6; ++k) {
            s[k] = part[k][lane % NW];
#pragma unroll
            for (int d = NW / 2; d > 0; d >>= 1)
                s[k] += __shfl_xor(s[k], d, NW);
        }
    }
    if (lane == 0)
        write(p, s);
}

// Partial FP64 sums of each component over contiguous chunks, one chunk per
// workgroup, then their sum in workgroup order: the mean does not depend on
// scheduling.
template <typename T>
__global__ __launch_bounds__(256) void k_mean_partial(const T *__restrict__ f, long long N,
                                                      double *__restrict__ part)
{
    __shared__ double wsum[256 / IBMX_WAVE];
    const long long chunk = (N + gridDim.x - 1) / gridDim.x;
    const long long lo = (long long)blockIdx.x * chunk;
    const long long hi = lo + chunk < N ? lo + chunk : N;
    const int wv = threadIdx.x / IBMX_WAVE, lane = threadIdx.x & (IBMX_WAVE - 1);
    constexpr int E = 16 / (int)sizeof(T);
    for (int a = 0; a < 3; ++a) {
        const T *fa = f + (size_t)a * N;
        double s = 0.0;
        if (((size_t)fa & 15) == 0 && lo % E == 0) {
            // 16-byte packets over the chunk, elements for its tail
            const long long nv = (hi - lo) / E;
            struct alignas(16) Packet {
                T e[E];
            };
            const Packet *pk = reinterpret_cast<const Packet *>(fa + lo);
            for (long long v = threadIdx.x; v < nv; v += blockDim.x) {
                const Packet q = pk[v];
#pragma unroll
                for (int k = 0; k < E; ++k)
                    s += (double)q.e[k];
            }
            for (long long i = lo + nv * E + threadIdx.x; i < hi; i += blockDim.x)
                s += (double)fa[i];
        } else {
            for (long long i = lo + threadIdx.x; i < hi; i += blockDim.x)
                s += (double)fa[i];
        }
        s = wave_sum(s);
        if (lane == 0)
            wsum[wv] = s;
        __syncthreads();
        if (threadIdx.x == 0) {
            double v = wsum[0];
            for (int w = 1; w < (int)(blockDim.x / IBMX_WAVE); ++w)
                v += wsum[w];
            part[(size_t)a * gridDim.x + blockIdx.x] = v;
        }
        __syncthreads();
    }
}

// one workgroup per component: 4096 partials by 1024 threads (one workgroup of
// 256 for all three took 14.6 us)
__global__ __launch_bounds__(1024) void k_mean_finish(const double *__restrict__ part, int nb,
                                                      long long N, double *__restrict__ mean)
{
    const int a = blockIdx.x;
    double s = 0.0;
    for (int i = threadIdx.x; i < nb; i += blockDim.x)
        s += part[(size_t)a * nb + i];
    s = block_sum<double>(s);
    if (threadIdx.x == 0)
        mean[a] = s / (double)N;
}

template <typename T>
__global__ void k_fill_grid(T *__restrict__ p, long long n)
{
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (; i < n; i += stride)
        p[i] = T(0);
}

// Waves per particle.  Sixteen up to one particle per CU (256 spheres of 24
// cells 26 us, with four waves 49; from the next on workgroups queue: 384 of 8
// cells 15 against 12.5).  Four up to 1535 (1500 of 24 cells 118 us, with one
// wave 198; of 4 cells both 12).  Above, one for small spheres, whose rows four
// waves share badly, and four for the ones wider than 10 cells (2000 of 4 cells
// 12.5 us, with four waves 13.9, of 12 cells 41 with one and 34 with four), from
// 4096 on only for the ones wider than 40, one wave each filling the chip
// (20,000 of 8 to 24 cells 313 us, 353 with 10).  32-bit field offsets while a
// component spans less than 4 GB.
template <typename T, bool O32>
void launch_integrals(ibmx_plan p, const T *u, const double *xp, const double *radius, double *Iu,
                      double *Ir, T *alpha_out)
{
    const int np = p->np;
    const double width = np >= 4096 ? 40.0 : 10.0;
    hipStream_t s = p->stream;
    if (np >= 1536)
        hipLaunchKernelGGL((k_particle_integrals<T, 1, O32>), dim3((np + 3) / 4 + np), dim3(256),
                           0, s, p->g, np, width, xp, radius, u, Iu, Ir, alpha_out);
    else if (np > 256)
        hipLaunchKernelGGL((k_particle_integrals<T, 4, O32>), dim3(np), dim3(256), 0, s, p->g, np,
                           width, xp, radius, u, Iu, Ir, alpha_out);
    else
        hipLaunchKernelGGL((k_particle_integrals<T, 16, O32>), dim3(np), dim3(1024), 0, s, p->g,
                           np, width, xp, radius, u, Iu, Ir, alpha_out);
}

template <typename T>
ibmx_status run_integrals(ibmx_plan p, const T *u, const double *xp, const double *radius,
                          double *Iu, double *Ir, T *alpha_out)
{
    hipStream_t s = p->stream;
    ProfScope ps(p, IBMX_K_OTHER);
    if (alpha_out)
        hipLaunchKernelGGL((k_fill_grid<T>), dim3(4096), dim3(256), 0, s, alpha_out, p->g.nodes);
    if (p->np > 0) {
        if ((unsigned long long)p->g.nodes * sizeof(T) < (1ULL << 32))
            launch_integrals<T, true>(p, u, xp, radius, Iu, Ir, alpha_out);
        else
            launch_integrals<T, false>(p, u, xp, radius, Iu, Ir, alpha_out);
    }
    return ibmx_launch_check();
}

template <typename T>
ibmx_status run_mean(ibmx_plan p, const T *f, double *mean)
{
    hipStream_t s = p->stream;
    ProfScope ps(p, IBMX_K_OTHER);
    hipLaunchKernelGGL((k_mean_partial<T>), dim3(MEAN_BLOCKS), dim3(256), 0, s, f, p->g.nodes,
                       p->mean_part);
    hipLaunchKernelGGL(k_mean_finish, dim3(3), dim3(1024), 0, s, (const double *)p->mean_part,
                       MEAN_BLOCKS, p->g.nodes, mean);
    return ibmx_launch_check();
}

}  // namespace

int ibmx_mean_blocks() { return MEAN_BLOCKS; }

// Partial sums of ibmx_grid_mean_noalloc: [3][MEAN_BLOCKS] doubles (96 KB)
// in every device's copy of the library's code object, held until the
// process ends.  Host code never passes this name to a kernel: it stands for
// a host-side shadow, not the device address; the address comes from
// hipGetSymbolAddress per device.
static __device__ __align__(256) double scratch[3 * MEAN_BLOCKS];

namespace {

constexpr int SCRATCH_DEVICES = 64;
std::mutex g_scratch_mu;
double *g_scratch_ptr[SCRATCH_DEVICES];   // address of scratch on each device

// Device address of scratch on the current device, looked up once per
// device with that device current.
ibmx_status scratch_on_current_device(double **out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess)
        return IBMX_EDEVICE;
    if (dev < 0 || dev >= SCRATCH_DEVICES)
        return IBMX_EUNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr)
            return IBMX_EDEVICE;
        g_scratch_ptr[dev] = (double *)ptr;
    }
    *out = g_scratch_ptr[dev];
    return IBMX_OK;
}

}  // namespace

extern "C" ibmx_status ibmx_grid_mean_noalloc(const void *f, int64_t n_nodes,
                                              ibmx_precision precision, double *mean,
                                              void *hip_stream)
{
    if (!f || !mean || n_nodes < 1 || n_nodes >= (1LL << 31) ||
        (precision != IBMX_F64 && precision != IBMX_F32))
        return IBMX_EINVAL;
    double *part = nullptr;
    const ibmx_status st = scratch_on_current_device(&part);
    if (st != IBMX_OK)
        return st;
    hipStream_t s = (hipStream_t)hip_stream;
    // every partial slot is written by k_mean_partial before k_mean_finish
    // reads it: nothing to clear between calls
    if (precision == IBMX_F64)
        hipLaunchKernelGGL((k_mean_partial<double>), dim3(MEAN_BLOCKS), dim3(256), 0, s,
                           (const double *)f, (long long)n_nodes, part);
    else
        hipLaunchKernelGGL((k_mean_partial<float>), dim3(MEAN_BLOCKS), dim3(256), 0, s,
                           (const float *)f, (long long)n_nodes, part);
    hipLaunchKernelGGL(k_mean_finish, dim3(3), dim3(1024), 0, s, (const double *)part, MEAN_BLOCKS,
                       (long long)n_nodes, mean);
    return ibmx_launch_check();
}

extern "C" ibmx_status ibmx_particle_integrals(ibmx_plan p, const void *u, const double *xp,
                                               const double *radius, double *Iu, double *Ir,
                                               void *alpha_out)
{
    if (!p || !u || (p->np > 0 && (!xp || !radius || !Iu || !Ir)))
        return IBMX_EINVAL;
    if (p->prec == IBMX_F64)
        return run_integrals<double>(p, (const double *)u, xp, radius, Iu, Ir, (double *)alpha_out);
    return run_integrals<float>(p, (const float *)u, xp, radius, Iu, Ir, (float *)alpha_out);
}

extern "C" ibmx_status ibmx_grid_mean(ibmx_plan p, const void *f, double *mean)
{
    if (!p || !f || !mean)
        return IBMX_EINVAL;
    if (p->prec == IBMX_F64)
        return run_mean<double>(p, (const double *)f, mean);
    return run_mean<float>(p, (const float *)f, mean);
}
