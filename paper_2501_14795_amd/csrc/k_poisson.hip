// Valid initial fields (Sec. 3.2: before the first step the fields satisfy
// Eq. 17, div E = rho, and Eq. 18, div B = 0).  Both are projections onto
// the periodic grid's gradients: E <- E - grad psi with Lap psi = div E -
// (rho - <rho>) (psi at the nodes) and B <- B - grad chi with Lap chi = div B
// (chi at the cell centres), Lap the five-point Laplacian -- the divergence of
// the Yee gradient.  A gradient has no discrete curl, so the curls that drive
// Eqs. 19-20 are kept.
//
// The periodic five-point Laplacian is the sum of one symmetric circulant
// matrix per axis, and the columns of the discrete Hartley transform, cas(2 pi
// j k / n) = cos + sin, are eigenvectors of every such matrix: in their basis
// the Poisson problem is a division by the eigenvalues.  So by default each
// solve is direct: two transforms there (rows, columns), the division, two
// back, each a dense matrix product in FP64 on the matrix cores, repeated on
// the residual until that is below the tolerance (each pass gains about
// eleven digits, so once or twice) or no longer falls.
//
// Conjugate gradients remain for a caller that caps the iterations.  Every
// scalar stays on the device: each dot product is a per-block partial sum
// followed by a one-block sum in fixed order (bit-reproducible), and the two
// r.r values of an iteration live in slots chosen by its parity, so no kernel
// overwrites a scalar another block may still read.
#include "pic_internal.h"

namespace pic {

namespace {

constexpr int kCgBlock = 256;

__device__ __forceinline__ int wrap(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

// Sum of v over the block, written by thread 0 to out[blockIdx.x].
__device__ __forceinline__ void block_partial(double v, double *out)
{
    __shared__ double s[kCgBlock / 64];
    for (int d = 32; d > 0; d >>= 1) v += __shfl_down(v, d, 64);
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < kCgBlock / 64; ++w) t += s[w];
        out[blockIdx.x] = t;
    }
}

// Right-hand sides.  E: r = div E - (rho - rho_bar) at the nodes, div E =
// (Ex[i] - Ex[i-1]) / dx + (Ey[j] - Ey[j-1]) / dy.  B: r = div B at the cell
// centres, (Bx[i+1] - Bx[i]) / dx + (By[j+1] - By[j]) / dy.  Partial sums of r.
__global__ void __launch_bounds__(kCgBlock) k_cg_rhs(const float *__restrict__ fld, const double *__restrict__ rho,
                                                     double rho_bar, int magnetic, int nx, int ny, double idx,
                                                     double idy, double *__restrict__ r, double *partial)
{
    const int64_t P = (int64_t)nx * ny;
    const float *fx = fld + (magnetic ? 3 * P : 0), *fy = fx + P;
    double acc = 0.0;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < P; k += (int64_t)gridDim.x * blockDim.x) {
        const int j = (int)(k / nx), i = (int)(k - (int64_t)j * nx);
        double v;
        if (magnetic) {
            const int64_t kx = (int64_t)j * nx + wrap(i + 1, nx), ky = (int64_t)wrap(j + 1, ny) * nx + i;
            v = ((double)fx[kx] - (double)fx[k]) * idx + ((double)fy[ky] - (double)fy[k]) * idy;
        } else {
            const int64_t kx = (int64_t)j * nx + wrap(i - 1, nx), ky = (int64_t)wrap(j - 1, ny) * nx + i;
            v = ((double)fx[k] - (double)fx[kx]) * idx + ((double)fy[k] - (double)fy[ky]) * idy -
                (rho[k] - rho_bar);
        }
        r[k] = v;
        acc += v;
    }
    block_partial(acc, partial);
}

// The periodic Laplacian maps onto zero-mean grids only: remove the mean of r
// (round-off of the sums above), then x = 0, p = r; partial r.r.
__global__ void __launch_bounds__(kCgBlock) k_cg_center(double *__restrict__ x, double *__restrict__ r,
                                                        double *__restrict__ p, int64_t P,
                                                        const double *__restrict__ sum, double *partial)
{
    const double mean = *sum / (double)P;
    double acc = 0.0;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < P; k += (int64_t)gridDim.x * blockDim.x) {
        const double v = r[k] - mean;
        x[k] = 0.0;
        r[k] = v;
        p[k] = v;
        acc = fma(v, v, acc);
    }
    block_partial(acc, partial);
}

// One block: out = sum of the n partials, in index order.
__global__ void __launch_bounds__(kCgBlock) k_cg_sum(const double *__restrict__ partial, int n, double *out)
{
    double v = 0.0;
    for (int b = threadIdx.x; b < n; b += kCgBlock) v += partial[b];
    __shared__ double s[kCgBlock];
    s[threadIdx.x] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int b = 0; b < kCgBlock; ++b) t += s[b];
        *out = t;
    }
}

// q = Lap p (five-point, periodic), partial p.q
__global__ void __launch_bounds__(kCgBlock) k_cg_apply(const double *__restrict__ p, double *__restrict__ q, int nx,
                                                       int ny, double idx2, double idy2, double *partial)
{
    const int64_t P = (int64_t)nx * ny;
    double acc = 0.0;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < P; k += (int64_t)gridDim.x * blockDim.x) {
        const int j = (int)(k / nx), i = (int)(k - (int64_t)j * nx);
        const int64_t row = (int64_t)j * nx;
        const double c = p[k];
        const double lx = p[row + wrap(i + 1, nx)] - 2.0 * c + p[row + wrap(i - 1, nx)];
        const double ly = p[(int64_t)wrap(j + 1, ny) * nx + i] - 2.0 * c + p[(int64_t)wrap(j - 1, ny) * nx + i];
        const double v = lx * idx2 + ly * idy2;
        q[k] = v;
        acc = fma(c, v, acc);
    }
    block_partial(acc, partial);
}

// alpha = rr / pq; x += alpha p; r -= alpha q; partial r.r
__global__ void __launch_bounds__(kCgBlock) k_cg_update(double *__restrict__ x, double *__restrict__ r,
                                                        const double *__restrict__ p, const double *__restrict__ q,
                                                        int64_t P, const double *__restrict__ scal, int cur,
                                                        double *partial)
{
    const double pq = scal[2], rr = scal[cur];
    const double alpha = pq != 0.0 ? rr / pq : 0.0;
    double acc = 0.0;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < P; k += (int64_t)gridDim.x * blockDim.x) {
        x[k] = fma(alpha, p[k], x[k]);
        const double v = fma(-alpha, q[k], r[k]);
        r[k] = v;
        acc = fma(v, v, acc);
    }
    block_partial(acc, partial);
}

// beta = rr_new / rr; p = r + beta p
__global__ void __launch_bounds__(kCgBlock) k_cg_direction(double *__restrict__ p, const double *__restrict__ r,
                                                           int64_t P, const double *__restrict__ scal, int cur)
{
    const double rr = scal[cur], rn = scal[cur ^ 1];
    const double beta = rr != 0.0 ? rn / rr : 0.0;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < P; k += (int64_t)gridDim.x * blockDim.x)
        p[k] = fma(beta, p[k], r[k]);
}

// ---- the direct solve

// The Hartley tables of both axes: cas(2 pi m / n) for m < n, then the
// eigenvalues -(2 sin(pi m / n) / d)^2 of the axis (tab: cas of x, of y,
// eigenvalues of x, of y).
__global__ void __launch_bounds__(kCgBlock) k_hartley_tables(double *__restrict__ tab, int nx, int ny, double idx,
                                                             double idy)
{
    const int t = blockIdx.x * kCgBlock + threadIdx.x;
    if (t >= nx + ny) return;
    const bool yaxis = t >= nx;
    const int n = yaxis ? ny : nx, m = yaxis ? t - nx : t;
    const double a = (double)m / (double)n;
    tab[t] = cospi(2.0 * a) + sinpi(2.0 * a);
    const double s = 2.0 * sinpi(a) * (yaxis ? idy : idx);
    tab[nx + ny + t] = -s * s;
}

// One transform of an ny x nx array, out of place: of its rows (in times the
// Hartley matrix of x) or, COLS, of its columns (the Hartley matrix of y
// times in).  SCALE: the result is divided by the eigenvalue sum of its
// mode and by nx ny (the inverse transform's factor); the constant mode is 0.
//
// A dense product of ny x nx outputs with nx or ny terms on v_mfma_f64_16x16x4:
// one 32 x 32 tile of the result per block, so a 512^2 grid still gives every
// compute unit a tile; eight wavefronts, a quarter of the tile and half of the
// terms each.  Operand tiles of 64 terms are staged in LDS, double-buffered,
// the next ones loaded while the current ones are multiplied.  The Hartley
// matrix is never stored: its tile is gathered from the table of n values at
// (row * col) mod n, advanced from stage to stage by one addition.  Row
// pitches of 68 and 48 doubles spread each operand read over the banks evenly.
// At one block per compute unit bound by the latency of a stage's loads
// (512^2, 268 MFLOP: 16 us; 20.5 with four wavefronts and 32 terms), on
// large grids by the FP64 matrix rate.
typedef double vd4 __attribute__((ext_vector_type(4)));
constexpr int kHt = 32;          // tile edge
constexpr int kHk = 64;          // terms per stage
constexpr int kHThreads = 512;
template <bool COLS, bool SCALE>
__global__ void __launch_bounds__(kHThreads) k_hartley(const double *__restrict__ in, double *__restrict__ out,
                                                       const double *__restrict__ tab, int nx, int ny)
{
    constexpr int LA = kHk + 4, LB = kHt + 16;
    __shared__ __align__(32) double sa[2][kHt * LA], sb[2][kHk * LB];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c0 = blockIdx.x * kHt, r0 = blockIdx.y * kHt;
    const int K = COLS ? ny : nx;
    const double *cas = COLS ? tab + nx : tab;
    // the thread's four elements of each operand tile: left (row lr + 8 u,
    // term lk), right (term rk + 16 u, column rc)
    const int lk = tid & 63, lr = tid >> 6, rc = tid & 31, rk = tid >> 5;
    unsigned at[4], step[4];   // Hartley elements: table index now and per stage
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const unsigned line = COLS ? (unsigned)(r0 + lr + 8 * u) : (unsigned)(c0 + rc);
        const unsigned term = COLS ? (unsigned)lk : (unsigned)(rk + 16 * u);
        at[u] = line * term % (unsigned)K;   // lines < 2^15 + 32
        step[u] = line * (unsigned)kHk % (unsigned)K;
    }
    double va[4], vb[4];
    auto load = [&](int k0) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const double h = cas[at[u]];
            at[u] += step[u];
            at[u] -= at[u] >= (unsigned)K ? (unsigned)K : 0u;
            const int ka = k0 + lk, kb = k0 + rk + 16 * u;
            if (COLS) {
                const int c = c0 + rc;
                va[u] = ka < K ? h : 0.0;
                vb[u] = kb < K && c < nx ? in[(int64_t)kb * nx + c] : 0.0;
            } else {
                const int r = r0 + lr + 8 * u;
                va[u] = r < ny && ka < K ? in[(int64_t)r * nx + ka] : 0.0;
                vb[u] = kb < K ? h : 0.0;
            }
        }
    };
    const int qr = (wave & 2) * 8, qc = (wave & 1) * 16, half = (wave >> 2) * (kHk / 2);   // the wavefront's part
    const int l16 = lane & 15, wk = lane >> 4;
    vd4 acc = {0.0, 0.0, 0.0, 0.0};
    load(0);
    for (int k0 = 0, b = 0; k0 < K; k0 += kHk, b ^= 1) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            sa[b][(lr + 8 * u) * LA + lk] = va[u];
            sb[b][(rk + 16 * u) * LB + rc] = vb[u];
        }
        __syncthreads();   // the other buffer is free: every wavefront has passed the last stage's barrier
        if (k0 + kHk < K) load(k0 + kHk);
#pragma unroll
        for (int k = 0; k < kHk / 2; k += 4)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(sa[b][(qr + l16) * LA + half + k + wk],
                                                       sb[b][(half + k + wk) * LB + qc + l16], acc, 0, 0, 0);
    }
    // the two halves of the terms, then the lane's results: column lane % 16,
    // rows lane / 16 + 4 v of the wavefront's quarter
    __syncthreads();
    vd4 *other = (vd4 *)&sa[0][0];
    if (wave >= 4) other[tid - 256] = acc;
    __syncthreads();
    if (wave >= 4) return;
    acc += other[tid];
    const int col = c0 + qc + l16;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int row = r0 + qr + wk + 4 * v;
        if (row >= ny || col >= nx) continue;
        double y = acc[v];
        if (SCALE) {
            const double *lam = tab + nx + ny;
            y = row | col ? y / ((lam[col] + lam[nx + row]) * ((double)nx * (double)ny)) : 0.0;
        }
        out[(int64_t)row * nx + col] = y;
    }
}

// x += z, r -= Lap z, partial r.r
__global__ void __launch_bounds__(kCgBlock) k_refine(double *__restrict__ x, double *__restrict__ r,
                                                     const double *__restrict__ z, int nx, int ny, double idx2,
                                                     double idy2, double *partial)
{
    const int64_t P = (int64_t)nx * ny;
    double acc = 0.0;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < P; k += (int64_t)gridDim.x * blockDim.x) {
        const int j = (int)(k / nx), i = (int)(k - (int64_t)j * nx);
        const int64_t row = (int64_t)j * nx;
        const double c = z[k];
        const double lx = (z[row + wrap(i + 1, nx)] - c) - (c - z[row + wrap(i - 1, nx)]);
        const double ly = (z[(int64_t)wrap(j + 1, ny) * nx + i] - c) - (c - z[(int64_t)wrap(j - 1, ny) * nx + i]);
        const double v = r[k] - (lx * idx2 + ly * idy2);
        x[k] += c;
        r[k] = v;
        acc = fma(v, v, acc);
    }
    block_partial(acc, partial);
}

// E: Ex -= (psi[i+1] - psi[i]) / dx, Ey -= (psi[j+1] - psi[j]) / dy.
// B: Bx -= (chi[i] - chi[i-1]) / dx, By -= (chi[j] - chi[j-1]) / dy.
// In FP64, stored as FP32.
__global__ void __launch_bounds__(kCgBlock) k_cg_project(float *__restrict__ fld, const double *__restrict__ s,
                                                         int magnetic, int nx, int ny, double idx, double idy)
{
    const int64_t P = (int64_t)nx * ny;
    float *fx = fld + (magnetic ? 3 * P : 0), *fy = fx + P;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < P; k += (int64_t)gridDim.x * blockDim.x) {
        const int j = (int)(k / nx), i = (int)(k - (int64_t)j * nx);
        double gx, gy;
        if (magnetic) {
            gx = (s[k] - s[(int64_t)j * nx + wrap(i - 1, nx)]) * idx;
            gy = (s[k] - s[(int64_t)wrap(j - 1, ny) * nx + i]) * idy;
        } else {
            gx = (s[(int64_t)j * nx + wrap(i + 1, nx)] - s[k]) * idx;
            gy = (s[(int64_t)wrap(j + 1, ny) * nx + i] - s[k]) * idy;
        }
        fx[k] = (float)((double)fx[k] - gx);
        fy[k] = (float)((double)fy[k] - gy);
    }
}

int cg_blocks(int64_t P)
{
    const int64_t b = (P + kCgBlock - 1) / kCgBlock;
    return (int)(b < kCgPartials ? (b > 0 ? b : 1) : kCgPartials);
}

}  // namespace

// One projection (magnetic = 0: E with rho; 1: B).  Returns the iterations
// run and the final ||r|| / ||r0|| (0 when r0 = 0), or -1 iterations on a
// HIP error; converged when the ratio is at most tol.  direct: by Hartley
// transforms, an iteration being one solve of the residual equation; else by
// conjugate gradients.  A 512^2 grid's 2,000 iterations of conjugate
// gradients, five launches of about 4 us each, took 22 ms a projection; the
// direct solve takes 0.15 (both with the host's reads of the residual).
CgResult cg_project(float *fld, const double *rho, double rho_bar, int magnetic, int nx, int ny, double dx, double dy,
                    double tol, int max_iter, bool direct, const CgScratch &w, hipStream_t s)
{
    CgResult res{0, 0.0, false};
    const int64_t P = (int64_t)nx * ny;
    const int nb = cg_blocks(P);
    const double idx = 1.0 / dx, idy = 1.0 / dy;
    hipLaunchKernelGGL(k_cg_rhs, dim3(nb), dim3(kCgBlock), 0, s, fld, rho, rho_bar, magnetic, nx, ny, idx, idy, w.r,
                       w.partial);
    hipLaunchKernelGGL(k_cg_sum, dim3(1), dim3(kCgBlock), 0, s, w.partial, nb, w.scal + 3);
    hipLaunchKernelGGL(k_cg_center, dim3(nb), dim3(kCgBlock), 0, s, w.x, w.r, w.p, P, w.scal + 3, w.partial);
    hipLaunchKernelGGL(k_cg_sum, dim3(1), dim3(kCgBlock), 0, s, w.partial, nb, w.scal + 0);
    double rr0 = 0.0;
    if (hipMemcpyAsync(&rr0, w.scal, sizeof(double), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess) {
        res.iterations = -1;
        return res;
    }
    if (!(rr0 > 0.0)) {
        res.converged = true;
        return res;
    }
    const double goal = tol * tol * rr0;
    double rr = rr0;
    int k = 0;
    if (direct) {
        const dim3 tiles((nx + kHt - 1) / kHt, (ny + kHt - 1) / kHt);
        hipLaunchKernelGGL(k_hartley_tables, dim3((nx + ny + kCgBlock - 1) / kCgBlock), dim3(kCgBlock), 0, s, w.tab, nx,
                           ny, idx, idy);
        for (double last = rr0;; last = rr) {
            hipLaunchKernelGGL((k_hartley<false, false>), tiles, dim3(kHThreads), 0, s, w.r, w.p, w.tab, nx, ny);
            hipLaunchKernelGGL((k_hartley<true, true>), tiles, dim3(kHThreads), 0, s, w.p, w.q, w.tab, nx, ny);
            hipLaunchKernelGGL((k_hartley<false, false>), tiles, dim3(kHThreads), 0, s, w.q, w.p, w.tab, nx, ny);
            hipLaunchKernelGGL((k_hartley<true, false>), tiles, dim3(kHThreads), 0, s, w.p, w.q, w.tab, nx, ny);
            hipLaunchKernelGGL(k_refine, dim3(nb), dim3(kCgBlock), 0, s, w.x, w.r, w.q, nx, ny, idx * idx, idy * idy,
                               w.partial);
            hipLaunchKernelGGL(k_cg_sum, dim3(1), dim3(kCgBlock), 0, s, w.partial, nb, w.scal + 1);
            ++k;
            if (hipMemcpyAsync(&rr, w.scal + 1, sizeof(double), hipMemcpyDeviceToHost, s) != hipSuccess ||
                hipStreamSynchronize(s) != hipSuccess) {
                res.iterations = -1;
                return res;
            }
            // reached, not a number, or at the rounding left in the constant mode,
            // which no pass takes out (a pass gains many digits until then)
            if (!(rr > goal) || rr > 0.25 * last) break;
        }
    }
    while (!direct && k < max_iter) {
        const int cur = k & 1;
        hipLaunchKernelGGL(k_cg_apply, dim3(nb), dim3(kCgBlock), 0, s, w.p, w.q, nx, ny, idx * idx, idy * idy,
                           w.partial);
        hipLaunchKernelGGL(k_cg_sum, dim3(1), dim3(kCgBlock), 0, s, w.partial, nb, w.scal + 2);
        hipLaunchKernelGGL(k_cg_update, dim3(nb), dim3(kCgBlock), 0, s, w.x, w.r, w.p, w.q, P, w.scal, cur,
                           w.partial);
        hipLaunchKernelGGL(k_cg_sum, dim3(1), dim3(kCgBlock), 0, s, w.partial, nb, w.scal + (cur ^ 1));
        hipLaunchKernelGGL(k_cg_direction, dim3(nb), dim3(kCgBlock), 0, s, w.p, w.r, P, w.scal, cur);
        ++k;
        if ((k & 15) == 0 || k == max_iter) {
            if (hipMemcpyAsync(&rr, w.scal + (k & 1), sizeof(double), hipMemcpyDeviceToHost, s) != hipSuccess ||
                hipStreamSynchronize(s) != hipSuccess) {
                res.iterations = -1;
                return res;
            }
            if (rr <= goal) break;
        }
    }
    res.iterations = k;
    res.residual = sqrt(rr / rr0);
    res.converged = rr <= goal;
    hipLaunchKernelGGL(k_cg_project, dim3(nb), dim3(kCgBlock), 0, s, fld, w.x, magnetic, nx, ny, idx, idy);
    return res;
}

}  // namespace pic
