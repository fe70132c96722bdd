// Yee field update on the periodic staggered grid (Eqs. 19-20).  The periodic
// neighbours are read directly (this replaces the guard-cell copy).  Outside
// the particle hot path: plain coalesced stencils.
//
//   pic_field_advance  the three sub-steps of Listing 3.1 as three launches in
//                      place, one thread per cell, with J in its planes;
//   pic_step           one launch, or two for a large grid (pic_eb.h): the push
//                      has formed the first B half step, J is folded from the tile current halos
//                      (update_gc_add, the same per-node sum as the fold
//                      kernel) unless the filter has written it.
#include "pic_eb.h"

namespace pic {

// Faraday: B -= h curl E for one 64 x 4 block of cells (hdx = h/dx, hdy =
// h/dy), in place, or from the push's half-step planes (a.bh).
__global__ void __launch_bounds__(256) k_yee_b(FieldArgs a)
{
    const int i = blockIdx.x * 64 + (threadIdx.x & 63);
    const int j = blockIdx.y * 4 + (threadIdx.x >> 6);
    const int nx = a.nx, ny = a.ny;
    if (i >= nx || j >= ny) return;
    float *__restrict__ f = a.fld;
    const int64_t P = (int64_t)nx * ny;
    const int64_t k = (int64_t)j * nx + i;
    const int64_t kx = (int64_t)j * nx + (i + 1 == nx ? 0 : i + 1);
    const int64_t ky = (int64_t)(j + 1 == ny ? 0 : j + 1) * nx + i;
    const float *Ex = f, *Ey = f + P, *Ez = f + 2 * P;
    const float *Bin = a.bh ? a.bh : f + 3 * P;
    float *Bx = f + 3 * P, *By = f + 4 * P, *Bz = f + 5 * P;
    const BCell b = faraday_half(Bin[k], Bin[P + k], Bin[2 * P + k], Ex[k], Ex[ky], Ey[k], Ey[kx], Ez[k], Ez[kx], Ez[ky], a.hdx,
                                 a.hdy);
    Bx[k] = b.x;
    By[k] = b.y;
    Bz[k] = b.z;
}

// Ampere: E += dt (curl B - J) for one 64 x 4 block of cells.
__global__ void __launch_bounds__(256) k_yee_e(FieldArgs a)
{
    const int i = blockIdx.x * 64 + (threadIdx.x & 63);
    const int j = blockIdx.y * 4 + (threadIdx.x >> 6);
    const int nx = a.nx, ny = a.ny;
    if (i >= nx || j >= ny) return;
    float *__restrict__ f = a.fld;
    const int64_t P = (int64_t)nx * ny;
    const int64_t k = (int64_t)j * nx + i;
    const int64_t kx = (int64_t)j * nx + (i == 0 ? nx - 1 : i - 1);
    const int64_t ky = (int64_t)(j == 0 ? ny - 1 : j - 1) * nx + i;
    const float *Bx = f + 3 * P, *By = f + 4 * P, *Bz = f + 5 * P, *J = f + 6 * P;
    const ECell e = ampere(a, f[k], f[P + k], f[2 * P + k], Bx[k], Bx[ky], By[k], By[kx], Bz[k], Bz[kx], Bz[ky], J[k],
                           J[P + k], J[2 * P + k]);
    f[k] = e.x;
    f[P + k] = e.y;
    f[2 * P + k] = e.z;
}

template <bool FOLD, int T, int H>
__global__ void __launch_bounds__(kEbThreads) k_field_half(FieldArgs a)
{
    field_eb_region<FOLD, T, H>(a, blockIdx.x, blockIdx.y);
}

// The E step alone, for a large grid.
template <bool FOLD, int T, int H>
__global__ void __launch_bounds__(kEThreads) k_field_e(FieldArgs a)
{
    field_e_block<FOLD, T, H>(a, blockIdx.x);
}

// many simulations: items = (simulation, rx, ry)
template <bool FOLD, int T, int H>
__global__ void __launch_bounds__(kEbThreads) k_field_half_b(const FieldArgs *d, const int4 *it, int n)
{
    const int b = linear_block();
    if (b >= n) return;
    const int4 w = it[b];
    field_eb_region<FOLD, T, H>(d[w.x], w.y, w.z);
}

void launch_field_b(const FieldArgs &f, hipStream_t s)
{
    hipLaunchKernelGGL(k_yee_b, dim3((f.nx + 63) / 64, (f.ny + 3) / 4), dim3(256), 0, s, f);
}

namespace {

struct FieldLaunch {
    const FieldArgs *single;
    const FieldArgs *descs;
    const int4 *items;
    int n_items;
    hipStream_t s;
    template <bool FOLD, int T, int H>
    void run() const
    {
        if (single && !single->eedge) {
            hipLaunchKernelGGL((k_field_e<FOLD, T, H>), dim3(e_blocks(single->nx, single->ny)), dim3(kEThreads), 0, s,
                               *single);
            launch_field_b(*single, s);
        } else if (single)
            hipLaunchKernelGGL((k_field_half<FOLD, T, H>), dim3(eb_cols(single->nx), eb_rows(single->ny)),
                               dim3(kEbThreads), 0, s, *single);
        else if (n_items > 0) {
            const BlockGrid g = block_grid(n_items, kEbThreads);
            hipLaunchKernelGGL((k_field_half_b<FOLD, T, H>), dim3(g.x, g.y), dim3(kEbThreads), 0, s, descs, items,
                               n_items);
        }
    }
};

}  // namespace

void launch_field_advance(const FieldArgs &f, hipStream_t s)
{
    launch_field_b(f, s);
    hipLaunchKernelGGL(k_yee_e, dim3((f.nx + 63) / 64, (f.ny + 3) / 4), dim3(256), 0, s, f);
    launch_field_b(f, s);
}

void launch_field_half(const FieldArgs &f, int tile, int halo, hipStream_t s)
{
    eb_dispatch(FieldLaunch{&f, nullptr, nullptr, 0, s}, f.jtile != nullptr, tile, halo);
}

void launch_field_half_batch(const FieldArgs *descs, const int4 *items, int n_items, bool fold, int tile, int halo,
                             hipStream_t s)
{
    eb_dispatch(FieldLaunch{nullptr, descs, items, n_items, s}, fold, tile, halo);
}

}  // namespace pic
