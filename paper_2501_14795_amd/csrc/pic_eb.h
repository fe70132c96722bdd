// The field half of a step after a push that formed the first B half step:
// the E step and the second B half step of one region of cells by one block,
// E passed between them in LDS.  Shared by the field kernels (k_field.hip) and
// the launches that run it beside the sort plan (k_sort.hip).
#pragma once

#include "pic_internal.h"
#include "pic_fold.h"
#include "pic_launch.h"
#include "pic_yee.h"

namespace pic {

// Ampere's step at one cell: E + dt (curl B - J), from B at the half step
// there and at the -x (x suffix) and -y neighbours.
struct ECell {
    float x, y, z;
};
__device__ __forceinline__ ECell ampere(const FieldArgs &a, float ex, float ey, float ez, float bx, float bx_y,
                                        float by, float by_x, float bz, float bz_x, float bz_y, float jx, float jy,
                                        float jz)
{
    ECell e{ex, ey, ez};
    e.x += a.dtdy * (bz - bz_y) - a.dt * jx;
    e.y += -a.dtdx * (bz - bz_x) - a.dt * jy;
    e.z += a.dtdx * (by - by_x) - a.dtdy * (bx - bx_y) - a.dt * jz;
    return e;
}

// The new E of cell (i, j), k its index, from the old one e; J folded or read
// into jv, B at the half step there into b.
template <bool FOLD, int T, int H>
__device__ __forceinline__ ECell advance_e(const FieldArgs &a, int i, int j, int64_t k, const ECell &e, BCell &b,
                                           float jv[3])
{
    const int nx = a.nx, ny = a.ny;
    const int64_t P = (int64_t)nx * ny;
    const int64_t kx = (int64_t)j * nx + (i == 0 ? nx - 1 : i - 1);
    const int64_t ky = (int64_t)(j == 0 ? ny - 1 : j - 1) * nx + i;
    const PIC_GLOBAL float *Bx = gp(a.bh), *By = Bx + P, *Bz = Bx + 2 * P;
    b = BCell{Bx[k], By[k], Bz[k]};
    const float bx_y = Bx[ky], by_x = By[kx], bz_x = Bz[kx], bz_y = Bz[ky];
    if constexpr (FOLD) {
        fold_node<T, H>(a.jtile, nx, ny, a.ntx, a.nty, i, j, jv);
    } else {
#pragma unroll
        for (int c = 0; c < 3; ++c) jv[c] = gp(a.fld)[(6 + c) * P + k];
    }
    return ampere(a, e.x, e.y, e.z, b.x, bx_y, b.y, by_x, b.z, bz_x, bz_y, jv[0], jv[1], jv[2]);
}

constexpr int64_t kFuseCells = (int64_t)1 << 21;
constexpr int kEbX = kEdgeX, kEbY = kEdgeY;   // region edges
constexpr int kEbOwn = kEbX * kEbY;           // a thread per cell
constexpr int kEbThreads = kEbOwn + (kEbX + kEbY + 63) / 64 * 64;   // and whole wavefronts for the cells beyond

// Region (rx, ry) of kEbX x kEbY cells (or what the grid has of it): J folded
// from the tile current halos (FOLD; tile edge T, halo pad H) and written, or
// read; E advanced; then B, from the push's half-step planes, with the new E.
// The B step reads E one cell beyond the region in +x and +y: that column and
// row are computed here too, from the old E in the push's edge strips (the
// block that owns them may have written the new E already).
//
// Bound by HBM: about 80 bytes a cell, against 98 as two launches that write E
// and read it and the half-step planes again (2048^2, 32 x 32 tiles: 75 us as
// two, 76 to 95 as one; 512^2, 16 x 16 tiles: 11.4 us as two, 8.5 as one).
// So one launch up to kFuseCells cells, where the planes stay in the last-level
// cache and the launch counts (1024^2: 20 us against 26), and two beyond
// (2048^2: a step 10 us faster with two).  One cell per thread and
// wavefronts of their own for the cells beyond, so a block waits for memory
// once before its barrier: 32 x 32 regions of four cells a thread took 114 us,
// strips marched by single wavefronts with the row's work in scalar registers
// 111, one row per wavefront or regions dealt to the XCDs in bands no less
// than this.
template <bool FOLD, int T, int H>
__device__ __forceinline__ void field_eb_region(const FieldArgs &a, int rx, int ry)
{
    __shared__ float s_ex[kEbY + 1][kEbX + 1], s_ey[kEbY + 1][kEbX + 1], s_ez[kEbY + 1][kEbX + 1];
    const int nx = a.nx, ny = a.ny;
    const int i0 = rx * kEbX, j0 = ry * kEbY;
    const int w = min(kEbX, nx - i0), h = min(kEbY, ny - j0);
    const int64_t P = (int64_t)nx * ny;
    PIC_GLOBAL float *f = gp(a.fld);
    // the thread's cell: of the region, of the row beyond (x < w) or of the column beyond
    const bool own = threadIdx.x < kEbOwn;
    const int q = (int)threadIdx.x - kEbOwn;
    const bool row = !own && q < kEbX;
    const int x = own ? (int)threadIdx.x % kEbX : (row ? q : w), y = own ? (int)threadIdx.x / kEbX : (row ? h : q - kEbX);
    const bool on = own ? x < w && y < h : (row ? x < w : y < h && q < kEbX + kEbY);
    const int i = i0 + x == nx ? 0 : i0 + x, j = j0 + y == ny ? 0 : j0 + y;
    const int64_t k = (int64_t)j * nx + i;
    BCell bo{};
    if (on) {
        // the old E: in its planes, or in the strips (Ex, Ez of a row; Ey, Ez of a column)
        ECell e;
        if (own) {
            e = ECell{f[k], f[P + k], f[2 * P + k]};
        } else {
            const PIC_GLOBAL float *s = gp(a.eedge) + (row ? edge_row(nx, ny, j / kEdgeY, i) : edge_col(ny, i / kEdgeX, j));
            e.x = e.y = s[0];
            e.z = s[row ? nx : ny];
        }
        float jv[3];
        e = advance_e<FOLD, T, H>(a, i, j, k, e, bo, jv);
        // (of the row beyond only Ex and Ez are read, of the column Ey and Ez)
        s_ex[y][x] = e.x;
        s_ey[y][x] = e.y;
        s_ez[y][x] = e.z;
        if (own) {
            f[k] = e.x;
            f[P + k] = e.y;
            f[2 * P + k] = e.z;
            if constexpr (FOLD) {
#pragma unroll
                for (int c = 0; c < 3; ++c) f[(6 + c) * P + k] = jv[c];
            }
        }
    }
    __syncthreads();
    if (!own || !on) return;
    const BCell b = faraday_half(bo.x, bo.y, bo.z, s_ex[y][x], s_ex[y + 1][x], s_ey[y][x], s_ey[y][x + 1], s_ez[y][x],
                                 s_ez[y][x + 1], s_ez[y + 1][x], a.hdx, a.hdy);
    f[3 * P + k] = b.x;
    f[4 * P + k] = b.y;
    f[5 * P + k] = b.z;
}

constexpr int kEThreads = 256;
// The E step alone of the cells of block q (a thread each, in index order).
template <bool FOLD, int T, int H>
__device__ __forceinline__ void field_e_block(const FieldArgs &a, int q)
{
    const int64_t P = (int64_t)a.nx * a.ny, k = (int64_t)q * kEThreads + threadIdx.x;
    if (k >= P) return;
    const int j = (int)(k / a.nx), i = (int)(k - (int64_t)j * a.nx);
    PIC_GLOBAL float *f = gp(a.fld);
    BCell b;
    float jv[3];
    const ECell e = advance_e<FOLD, T, H>(a, i, j, k, ECell{f[k], f[P + k], f[2 * P + k]}, b, jv);
    f[k] = e.x;
    f[P + k] = e.y;
    f[2 * P + k] = e.z;
    if constexpr (FOLD) {
#pragma unroll
        for (int c = 0; c < 3; ++c) f[(6 + c) * P + k] = jv[c];
    }
}
inline int e_blocks(int nx, int ny) { return (int)(((int64_t)nx * ny + kEThreads - 1) / kEThreads); }

// the block's index in a block_grid
__device__ __forceinline__ int linear_block() { return (int)(blockIdx.x + gridDim.x * blockIdx.y); }

// regions per axis
__host__ __device__ __forceinline__ int eb_cols(int nx) { return (nx + kEbX - 1) / kEbX; }
__host__ __device__ __forceinline__ int eb_rows(int ny) { return (ny + kEbY - 1) / kEbY; }

// Calls go.run<FOLD, T, H>() for a fold of tiles of edge
// `tile` with halo pad `halo`, or for J read from its planes.
template <int T, class F>
void eb_halo(const F &go, int halo)
{
    if (halo == 2) {
        if constexpr (cadence_ok(T, 2)) go.template run<true, T, 2>();
    } else if (halo == 4) {
        if constexpr (cadence_ok(T, 4)) go.template run<true, T, 4>();
    } else {
        go.template run<true, T, 1>();
    }
}
template <class F>
void eb_dispatch(const F &go, bool fold, int tile, int halo)
{
    if (!fold) go.template run<false, 8, 1>();
    else if (tile == 8) eb_halo<8>(go, halo);
    else if (tile == 16) eb_halo<16>(go, halo);
    else eb_halo<32>(go, halo);
}

}  // namespace pic
