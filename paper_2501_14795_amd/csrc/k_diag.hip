// Diagnostics with FP64 accumulation (energies, node charge density, the
// discrete continuity residual of Eq. 12, the residuals of Gauss's law and of
// div B = 0).  Not on the hot path of a step, but called every few steps.
//
// Every block ends in one atomic per sum or maximum, into one of kDiagSlots
// accumulator sets (64 cache lines; the host folds them): thousands of blocks
// adding to one address take their turns at about 12 ns each (4,096 blocks
// and two sums: 102 us for the field energy of a 1024^2 grid, whose 25 MB
// take 6 us), and a maximum taken cell by cell, 377 us.  Energies and residuals
// of that grid together now take 21 us, most of it the FP64 divisions.
#include "pic_internal.h"

namespace pic {

__device__ __forceinline__ double wave_sum_d(double v)
{
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v += __shfl_down(v, d, 64);
    return v;
}

// Maxima are of non-negative values, taken on their bit patterns, which
// order alike, with NaN above everything: a NaN anywhere is reported.
__device__ __forceinline__ unsigned long long max_bits(unsigned long long m, double v)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(fabs(v));
    return b > m ? b : m;
}

// The block's accumulator set.
__device__ __forceinline__ double *diag_slot(double *acc) { return acc + (blockIdx.x % kDiagSlots) * kDiagStride; }

// The sum of one value per thread of a block of W wavefronts, into entry k of
// the block's accumulator set.  All threads take part.
template <int W>
__device__ __forceinline__ void block_sum(double v, double *acc, int k)
{
    __shared__ double s[W];
    v = wave_sum_d(v);
    __syncthreads();   // s may still be read for the last value
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = s[0];
        for (int w = 1; w < W; ++w) t += s[w];
        atomicAdd(&diag_slot(acc)[k], t);
    }
}

// The same for a maximum (of bit patterns).
template <int W>
__device__ __forceinline__ void block_max(unsigned long long v, double *acc, int k)
{
    __shared__ unsigned long long s[W];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
        const unsigned long long o = __shfl_down(v, d, 64);
        v = o > v ? o : v;
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long t = s[0];
        for (int w = 1; w < W; ++w) t = s[w] > t ? s[w] : t;
        atomicMax((unsigned long long *)&diag_slot(acc)[k], t);
    }
}

// acc and, if given, rho to zero (a kernel: one launch for both)
__global__ void __launch_bounds__(256) k_diag_clear(double *__restrict__ acc, double *__restrict__ rho, int64_t plane)
{
    const int64_t step = (int64_t)gridDim.x * blockDim.x, t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (acc)
        for (int64_t k = t; k < kDiagSlots * kDiagStride; k += step) acc[k] = 0.0;
    if (rho)
        for (int64_t k = t; k < plane; k += step) rho[k] = 0.0;
}

// One species' particles, sp.range consecutive slots per block: the kinetic
// energy (kin), and the node charge density (rho) with the linear shape or
// the quadratic B-spline.  The block walks the tile sections in its range;
// the charge of a section's part is summed in LDS over the tile and kDiagPad
// nodes around it (a particle strays at most four cells from its tile before
// a sort; with the quadratic shape, which reaches one node further, at most
// one), then added to the grid with one atomic per node, so the particles of
// a node meet in LDS and not in the L2.  16.8 M particles, density and kinetic
// energy: 470 + 70 us as two kernels with four global FP64 atomics a particle,
// now 111 us (3.3 TB/s; the FP64 weights and LDS atomics beside the 22 bytes
// a particle).  A part of fewer than kDiagFew
// particles adds to the grid directly: clearing and flushing the LDS nodes
// would cost more.
constexpr int kDiagPad = 4;
constexpr int kDiagWaves = 8;
constexpr int kDiagFew = 128;
constexpr int kDiagAhead = 4;
__global__ void __launch_bounds__(64 * kDiagWaves) k_diag_particles(DiagSpecies sp, double *__restrict__ rho,
                                                                    double *__restrict__ acc, int kin)
{
    constexpr int NT = 64 * kDiagWaves;
    constexpr int kMost = 32 + 2 * kDiagPad + 1;
    __shared__ double s_rho[kMost * kMost];
    const int T = sp.tile, NJ = T + 2 * kDiagPad + 1;
    // nodes lx - lo_n .. lx + hi_n of a particle in cell lx (relative to its tile)
    const int lo_n = sp.quadratic ? 1 : 0, hi_n = sp.quadratic ? 2 : 1;
    const int64_t r0 = (int64_t)blockIdx.x * sp.range, r1 = min(r0 + sp.range, (int64_t)sp.n);
    double energy = 0.0;
    for (int64_t p0 = r0; p0 < r1;) {   // uniform over the block
        // the tile whose section holds slot p0: the last with off <= p0
        int tile = 0, top = sp.n_tiles;
        while (top - tile > 1) {
            const int mid = (tile + top) >> 1;
            if (sp.off[mid] <= p0) tile = mid;
            else top = mid;
        }
        int64_t p1 = min((int64_t)sp.off[tile + 1], r1);
        if (p1 <= p0 || !rho) p1 = r1;   // (offsets always end at n); the energies need no tiles
        const int gx0 = (tile % sp.ntx) * T, gy0 = (tile / sp.ntx) * T;
        auto node = [&](int i, int j) {   // relative node -> grid index (periodic)
            i += gx0;
            j += gy0;
            i = i < 0 ? i + sp.nx : (i >= sp.nx ? i - sp.nx : i);
            j = j < 0 ? j + sp.ny : (j >= sp.ny ? j - sp.ny : j);
            return (int64_t)j * sp.nx + i;
        };
        const bool lds = rho && p1 - p0 >= kDiagFew;
        if (lds) {
            for (int e = threadIdx.x; e < NJ * NJ; e += NT) s_rho[e] = 0.0;
            __syncthreads();
        }
        // kDiagAhead particles per thread and pass, their loads in flight together
        for (int64_t pb = p0 + threadIdx.x; pb < p1; pb += kDiagAhead * NT) {
            float vx[kDiagAhead], vy[kDiagAhead], vu[kDiagAhead][3];
            int vc[kDiagAhead];
#pragma unroll
            for (int u = 0; u < kDiagAhead; ++u) {
                const int64_t p = pb + (int64_t)u * NT;
                if (p >= p1) continue;
                if (kin) {
                    vu[u][0] = sp.p.ux[p];
                    vu[u][1] = sp.p.uy[p];
                    vu[u][2] = sp.p.uz[p];
                }
                if (rho) {
                    vc[u] = sp.p.cell[p];
                    vx[u] = sp.p.x[p];
                    vy[u] = sp.p.y[p];
                }
            }
#pragma unroll
            for (int u = 0; u < kDiagAhead; ++u) {
                if (pb + (int64_t)u * NT >= p1) continue;
                if (kin) {
                    const double ux = vu[u][0], uy = vu[u][1], uz = vu[u][2];
                    const double u2 = ux * ux + uy * uy + uz * uz;
                    energy += u2 / (sqrt(1.0 + u2) + 1.0);   // gamma - 1 without cancellation
                }
                if (!rho) continue;
                const int lx = tcell_x(vc[u]) & sp.mask, ly = tcell_y(vc[u]) & sp.mask;
                const double x = vx[u], y = vy[u], q = sp.q;
                if (lx - lo_n < -kDiagPad || lx + hi_n > T + kDiagPad || ly - lo_n < -kDiagPad || ly + hi_n > T + kDiagPad)
                    continue;   // no such particle in a valid state
                auto add = [&](int i, int j, double v) {
                    if (lds) atomicAdd(&s_rho[(j + kDiagPad) * NJ + i + kDiagPad], v);
                    else atomicAdd(&rho[node(i, j)], v);
                };
                if (sp.quadratic) {
                    // the three nodes nearest the particle on each axis, weighted by the
                    // quadratic B-spline at their distance
                    const int hx = x >= 0.5 ? 1 : 0, hy = y >= 0.5 ? 1 : 0;
                    const double ex = x - hx, ey = y - hy;   // offset from the nearest node, [-1/2, 1/2)
                    const double wx[3] = {0.5 * (0.5 - ex) * (0.5 - ex), 0.75 - ex * ex, 0.5 * (0.5 + ex) * (0.5 + ex)};
                    const double wy[3] = {0.5 * (0.5 - ey) * (0.5 - ey), 0.75 - ey * ey, 0.5 * (0.5 + ey) * (0.5 + ey)};
#pragma unroll
                    for (int b = 0; b < 3; ++b)
#pragma unroll
                        for (int a = 0; a < 3; ++a) add(lx + hx + a - 1, ly + hy + b - 1, q * wx[a] * wy[b]);
                } else {
                    add(lx, ly, q * (1.0 - x) * (1.0 - y));
                    add(lx + 1, ly, q * x * (1.0 - y));
                    add(lx, ly + 1, q * (1.0 - x) * y);
                    add(lx + 1, ly + 1, q * x * y);
                }
            }
        }
        if (lds) {
            __syncthreads();
            for (int e = threadIdx.x; e < NJ * NJ; e += NT) {
                const double v = s_rho[e];
                if (v != 0.0) atomicAdd(&rho[node(e % NJ - kDiagPad, e / NJ - kDiagPad)], v);
            }
            __syncthreads();   // s_rho is reused for the next tile
        }
        p0 = p1;
    }
    if (kin) block_sum<kDiagWaves>(energy, acc, kin);
}

// The grid's sums and maxima, every selected one in a single pass (what: the
// PIC_DIAG_* bits): the field energies; the continuity residual
// rho - rho_prev + dt div J at the nodes and max |rho|; Gauss's law at the
// nodes, div E - (rho - rho_bar) with the ions a uniform neutralising
// background rho_bar, and div B at the cell centres (i+1/2, j+1/2).
// kDiagRows rows of 256 cells per block: two, so that a 1024^2 grid has 2,048
// blocks (28 us with eight rows and 512 blocks, 21 with two).
constexpr int kDiagRows = 2;
__global__ void __launch_bounds__(256) k_diag_grid(DiagGrid g, unsigned what)
{
    const int nx = g.nx, ny = g.ny;
    const int64_t P = (int64_t)nx * ny;
    const float *__restrict__ f = g.fld;
    const int cols = (nx + 255) / 256;
    const int i = (blockIdx.x % cols) * 256 + threadIdx.x, j0 = (blockIdx.x / cols) * kDiagRows;
    double se = 0.0, sb = 0.0;
    unsigned long long cont = 0, rmax = 0, gauss = 0, divb = 0;
    const int im = i == 0 ? nx - 1 : i - 1, ip = i + 1 == nx ? 0 : i + 1;
    for (int j = j0; j < min(j0 + kDiagRows, ny) && i < nx; ++j) {
        const int64_t k = (int64_t)j * nx + i, kxm = (int64_t)j * nx + im, kxp = (int64_t)j * nx + ip;
        const int64_t kym = (int64_t)(j == 0 ? ny - 1 : j - 1) * nx + i;
        const int64_t kyp = (int64_t)(j + 1 == ny ? 0 : j + 1) * nx + i;
        if (what & PIC_DIAG_ENERGY) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const double e = f[c * P + k], b = f[(3 + c) * P + k];
                se += e * e;
                sb += b * b;
            }
        }
        if (what & PIC_DIAG_CONTINUITY) {
            const float *J = f + 6 * P;
            const double div =
                ((double)J[k] - (double)J[kxm]) / g.dx + ((double)J[P + k] - (double)J[P + kym]) / g.dy;
            cont = max_bits(cont, g.rho[k] - g.rho_prev[k] + g.dt * div);
            rmax = max_bits(rmax, g.rho[k]);
        }
        if (what & PIC_DIAG_GAUSS) {
            const double dive =
                ((double)f[k] - (double)f[kxm]) / g.dx + ((double)f[P + k] - (double)f[P + kym]) / g.dy;
            const double db = ((double)f[3 * P + kxp] - (double)f[3 * P + k]) / g.dx +
                              ((double)f[4 * P + kyp] - (double)f[4 * P + k]) / g.dy;
            gauss = max_bits(gauss, dive - (g.rho[k] - g.rho_bar));
            divb = max_bits(divb, db);
        }
    }
    if (what & PIC_DIAG_ENERGY) {
        block_sum<4>(se, g.acc, kDiagUe);
        block_sum<4>(sb, g.acc, kDiagUb);
    }
    if (what & PIC_DIAG_CONTINUITY) {
        block_max<4>(cont, g.acc, kDiagCont);
        block_max<4>(rmax, g.acc, kDiagRhoMax);
    }
    if (what & PIC_DIAG_GAUSS) {
        block_max<4>(gauss, g.acc, kDiagGauss);
        block_max<4>(divb, g.acc, kDiagDivb);
    }
}

__global__ void __launch_bounds__(256) k_counts(const int32_t *cnt, const int32_t *mcount, int n_tiles,
                                                unsigned long long *acc)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n_tiles) return;
    atomicAdd(&acc[0], (unsigned long long)cnt[(int64_t)t * kCntStride + kCntLeavers]);
    atomicAdd(&acc[1], (unsigned long long)mcount[t]);
}

void launch_diag_clear(double *acc, double *rho, int64_t plane, hipStream_t s)
{
    const int64_t n = rho ? plane : kDiagSlots * kDiagStride;
    hipLaunchKernelGGL(k_diag_clear, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 2048)), dim3(256), 0, s, acc,
                       rho, plane);
}

void launch_diag_particles(const DiagSpecies &sp, int n_tiles, double *rho, double *acc, int kin, hipStream_t s)
{
    if (sp.n <= 0 || (!rho && !kin)) return;
    // enough blocks for the device (2,048 fill it) before a block takes more
    // than a round of its threads; at most 16 particles per thread
    DiagSpecies d = sp;
    d.n_tiles = n_tiles;
    d.range = (int)std::min<int64_t>(16 * 64 * kDiagWaves, std::max<int64_t>(64 * kDiagWaves, sp.n / 2048));
    hipLaunchKernelGGL(k_diag_particles, dim3((unsigned)(((int64_t)sp.n + d.range - 1) / d.range)),
                       dim3(64 * kDiagWaves), 0, s, d, rho, acc, kin);
}

void launch_diag_grid(const DiagGrid &g, unsigned what, hipStream_t s)
{
    const int blocks = ((g.nx + 255) / 256) * ((g.ny + kDiagRows - 1) / kDiagRows);
    hipLaunchKernelGGL(k_diag_grid, dim3(blocks), dim3(256), 0, s, g, what);
}

void launch_diag_counts(const int32_t *cnt, const int32_t *mcount, int n_tiles, unsigned long long *acc,
                        hipStream_t s)
{
    hipLaunchKernelGGL(k_counts, dim3((n_tiles + 255) / 256), dim3(256), 0, s, cnt, mcount, n_tiles, acc);
}

}  // namespace pic
