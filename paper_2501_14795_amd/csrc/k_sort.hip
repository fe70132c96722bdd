// Strict re-sort of particles by tile (Sec. 4.3, the bucket sort of Fig. 4.5),
// redesigned for gfx950: no atomics decide any position, so the permutation
// is the canonical one and is reproducible bit for bit.
//
//   k_sort_count (and k_sort_scan_blocks above 64 scan blocks)
//                  step (1): the new count of tile t is the sum, over the nine
//                  tiles a particle can come from, of the direction counts the
//                  push kernel recorded, with its prefix in a block of 256
//                  tiles; k_sort_plan adds the blocks before its own and writes
//                  tile_offset'.  Up to 256 tiles the plan counts by itself.
//   k_sort_plan    steps (2)-(4), one wavefront per destination tile t with
//                  new section [A, B):
//                    holes  = slots of [A, B) whose particle is not in tile t,
//                             in ascending order: the parts of [A, B) outside
//                             t's old section (read the cells there) and t's
//                             own leavers inside it (from its leaver lists);
//                    movers = particles of tile t outside [A, B), ascending:
//                             the leavers of the up-to-eight neighbour tiles
//                             heading to t (the push lists them by direction)
//                             and t's own stayers pushed out of [A, B) by
//                             section shifts;
//                  every mover is copied, in hole order, to a staging area
//                  (contiguous stores), so only O(movers) particle bytes
//                  are touched and no particle slot is written while other
//                  plans may still read it.
//   k_sort_scatter step (5): the staged movers into their holes -- or, in
//                  pic_step, nothing: the next push fills each hole from
//                  the staging area as it streams its section (a deferred
//                  fill; k_settle or k_fill completes one on its own when
//                  anything else is to read the particles first).
//
// The cells the kernels keep are 16-bit offsets from the tile whose section
// holds the particle (tcell_pack); the staging records carry whole-grid
// cells, converted on the way in and out.  Also here: the motion-class sort
// (the alternative of Sec. 4.3), the conversions between the caller's
// whole-grid cells and the 16-bit ones, and the tile offsets of caller
// particles at initialisation.
#include "pic_eb.h"

namespace pic {


__device__ __forceinline__ int wrap_s(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

__device__ __forceinline__ int lane_rank_s(unsigned long long m)
{
    return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

// Exclusive scan of one int per thread over a 1024-thread block; returns the
// thread's prefix and writes the block total to *total.
__device__ int block_exclusive_scan_1024(int v, int *total)
{
    __shared__ int s_w[16];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int x = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    if (lane == 63) s_w[w] = x;
    __syncthreads();
    if (w == 0) {
        int t = lane < 16 ? s_w[lane] : 0;
#pragma unroll
        for (int d = 1; d < 16; d <<= 1) {
            const int y = __shfl_up(t, d, 64);
            if (lane >= d) t += y;
        }
        if (lane < 16) s_w[lane] = t;
    }
    __syncthreads();
    const int base = w > 0 ? s_w[w - 1] : 0;
    *total = s_w[15];
    return base + x - v;
}

__device__ __forceinline__ int tile_count_in(const int32_t *cnt, int t, int ntx, int nty)
{
    const int tx = t % ntx, ty = t / ntx;
    int v = 0;
#pragma unroll
    for (int o = 0; o < 9; ++o) {
        const int odx = o % 3 - 1, ody = o / 3 - 1;
        const int src = wrap_s(ty - ody, nty) * ntx + wrap_s(tx - odx, ntx);
        v += cnt[(int64_t)src * kCntStride + o];
    }
    return v;
}

// Exclusive scan of one int per thread over a block of kScanBlock threads;
// returns the thread's prefix and the block total.  All threads take part.
__device__ __forceinline__ int block_exclusive(int c, int &total)
{
    __shared__ int s_w[kScanBlock / 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int x = c;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    if (lane == 63) s_w[w] = x;
    __syncthreads();
    int base = 0;
    total = 0;
#pragma unroll
    for (int k = 0; k < kScanBlock / 64; ++k) {
        if (k < w) base += s_w[k];
        total += s_w[k];
    }
    return base + x - c;
}

// The new count of tile t: what the push recorded, and the window's new
// particles (0 past the last tile).
__device__ __forceinline__ int tile_count_new(const SortArgs &a, const SortSpecies &sp, int t)
{
    if (t >= a.n_tiles) return 0;
    int c = tile_count_in(sp.cnt, t, a.ntx, a.nty);
    if (sp.inj_off) c += sp.inj_off[t + 1] - sp.inj_off[t];
    return c;
}

// What the new counts must add up to.
__device__ __forceinline__ int sort_expect(const SortSpecies &sp)
{
    return sp.removed ? sp.n - *sp.removed + sp.inj_n : sp.n;
}

// Step (1), first pass: new count of every tile and its exclusive prefix
// within its block of kScanBlock tiles; block totals to bsum.
__device__ __forceinline__ void sort_count_unit(const SortArgs &a, int spi, int blk)
{
    const SortSpecies &sp = a.sp[spi];
    const int t = blk * kScanBlock + threadIdx.x;
    const int c = tile_count_new(a, sp, t);
    int total;
    const int ex = block_exclusive(c, total);
    if (t < a.n_tiles) {
        sp.pre[t] = ex;
        sp.cnew[t] = c;
    }
    if (threadIdx.x == 0) sp.bsum[blk] = total;
}

// Step (1), second pass (one block per species): exclusive scan of the block
// totals in place; tile_offset'[n_tiles] = total, checked against n.
__device__ __forceinline__ void sort_scan_unit(const SortArgs &a, int spi)
{
    const SortSpecies &sp = a.sp[spi];
    const int n_tiles = a.n_tiles;
    const int nb = (n_tiles + kScanBlock - 1) / kScanBlock;
    int carry = 0;
    for (int b0 = 0; b0 < nb; b0 += 1024) {
        const int b = b0 + threadIdx.x;
        const int v = b < nb ? sp.bsum[b] : 0;
        int total;
        const int ex = block_exclusive_scan_1024(v, &total);
        if (b < nb) sp.bsum[b] = carry + ex;
        carry += total;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        sp.off[n_tiles] = carry;
        if (carry != sort_expect(sp)) atomicOr(a.err, kErrCount);
    }
}

// Step (1), third pass where no plan follows (the motion-class sort): add
// each block's base.
__device__ __forceinline__ void sort_add_unit(const SortArgs &a, int spi, int blk)
{
    const SortSpecies &sp = a.sp[spi];
    const int t = blk * kScanBlock + threadIdx.x;
    if (t < a.n_tiles) sp.off[t] = sp.pre[t] + sp.bsum[blk];
}

// Step (1), second and third pass in one, while there are at most
// kScanDirect blocks: each block sums its predecessors' totals itself and
// adds them; the last one also writes tile_offset'[n_tiles] and checks it.
constexpr int kScanDirect = 64;
static_assert(kScanDirect <= kScanBlock, "one predecessor total per thread");
__device__ __forceinline__ void sort_add_direct_unit(const SortArgs &a, int spi, int blk)
{
    const SortSpecies &sp = a.sp[spi];
    const int n_tiles = a.n_tiles;
    const int nb = (n_tiles + kScanBlock - 1) / kScanBlock;
    __shared__ int s_w[kScanBlock / 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int v = (int)threadIdx.x < blk ? sp.bsum[threadIdx.x] : 0;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    if (lane == 0) s_w[w] = v;
    __syncthreads();
    int base = 0;
#pragma unroll
    for (int k = 0; k < kScanBlock / 64; ++k) base += s_w[k];
    const int t = blk * kScanBlock + threadIdx.x;
    if (t < n_tiles) sp.off[t] = sp.pre[t] + base;
    if (blk == nb - 1 && threadIdx.x == 0) {
        const int total = base + sp.bsum[blk];
        sp.off[n_tiles] = total;
        if (total != sort_expect(sp)) atomicOr(a.err, kErrCount);
    }
}

// Slot of the list holding flat index k, over the lists described by lanes
// 0..31 (exclusive prefix `ex` of their lengths): the largest L with ex_L <=
// k.  Fixed-step binary search, all lanes active.
__device__ __forceinline__ int find_list(int k, int ex)
{
    int lo = 0;
#pragma unroll
    for (int step = 16; step > 0; step >>= 1)
        if (__shfl(ex, lo + step, 64) <= k) lo += step;
    return lo;
}

// Wave-wide exclusive prefix of v (and the total).
__device__ __forceinline__ int wave_exclusive(int v, int &total)
{
    const int lane = threadIdx.x & 63;
    int x = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    total = __shfl(x, 63, 64);
    return x - v;
}

// One particle's six values in registers.
struct Chunk6 {
    int cell;
    float x, y, ux, uy, uz;
};

// one leaver record (two vector loads)
__device__ __forceinline__ Chunk6 load_leaver(const LeaverRec *src, int64_t i)
{
    const PIC_GLOBAL vf4 *s = (const PIC_GLOBAL vf4 *)(src + i);
    const vf4 a = s[0];
    const vf2 b = *(const PIC_GLOBAL vf2 *)(s + 1);
    return Chunk6{__float_as_int(a.x), a.y, a.z, a.w, b.x, b.y};
}

// The particle at slot i, inside the tile whose first cell is (gx0, gy0),
// with its whole-grid cell (the staging records' form); mask: T - 1 in a
// sorted state (the cell is relative to the tile modulo T), else -1.
__device__ __forceinline__ Chunk6 load_parts(const Parts &src, int64_t i, int gx0, int gy0, int mask)
{
    const int lc = src.cell[i];
    return Chunk6{(gx0 + (tcell_x(lc) & mask)) | ((gy0 + (tcell_y(lc) & mask)) << 16), src.x[i], src.y[i],
                  src.ux[i], src.uy[i], src.uz[i]};
}

// A particle of the tile whose first cell is (gx0, gy0), given with its
// whole-grid cell, into slot j (its cell relative to that tile).
__device__ __forceinline__ void store_parts(const Parts &dst, int64_t j, const Chunk6 &c, int gx0, int gy0)
{
    dst.cell[j] = (int16_t)tcell_pack((c.cell & 0xffff) - gx0, (c.cell >> 16) - gy0);
    dst.x[j] = c.x;
    dst.y[j] = c.y;
    dst.ux[j] = c.ux;
    dst.uy[j] = c.uy;
    dst.uz[j] = c.uz;
}

// Whether tile-relative cell lc lies inside its tile (of edge T).
__device__ __forceinline__ bool tcell_inside(int lc, int T)
{
    return (unsigned)tcell_x(lc) < (unsigned)T && (unsigned)tcell_y(lc) < (unsigned)T;
}

// Steps (2)-(4) of the sort for one destination tile t per wavefront, new
// section [A, B), old section [oA, oB).  Every candidate list of holes and of
// movers is described by one lane; the lists are streamed as one flat index
// space, holes first, and compacted with ballots, which keeps both outputs in
// ascending slot order.  W = leaver sub-lists per tile (the push kernel's
// wavefronts per tile).  Lists:
//   0             : holes in [A, min(B, oA)), slots of lower old sections
//                   (hole unless the particle there moved into t, or is one
//                   of the window's new particles for t)
//   1 .. W        : holes among t's W leaver sub-lists, restricted to
//                   [max(A, oA), min(B, oB))
//   W + 1         : holes in [max(A, oB), B), slots of higher old sections
//   W + 2 .. W + 11 : movers by source tile, ascending: of each of the eight
//                   neighbours the leavers heading to t (the push lists a
//                   tile's leavers by direction, each direction in slot
//                   order) whose slot is outside [A, B), data from the leaver
//                   records; at t's own place two lists, t's slots below A
//                   and from B on whose particle kept tile t
//   W + 12, + 13  : the moving window's new particles for t outside [A, B)
// The loads are staged so that each round trip to memory serves all lists at
// once: the list bounds, then the candidates (NB iterations of 64), then the
// movers' data, then the stores.
//
// Bound by that chain of round trips and by the lane exchanges of the list
// search.  Reading a neighbour's leavers for one direction instead of all of
// them cuts the candidates to about a fourth and the lists to half a
// wavefront's lanes: 4,096 32 x 32 tiles (253 K movers) 75 -> 30 us beside the
// field half, 2,048 16 x 16 ones (512^2, two beams) 46 -> 26, 64 batched
// simulations 86 -> 43.
//
// Two candidate iterations per round trip: 48 registers, eight wavefronts per
// SIMD.  (With the whole leaver lists to read, six were faster while every
// tile's wavefront was resident at once; with a fourth of the candidates the
// two forms take the same time: 4,096 tiles 25.2 us each, 2,048 hot ones 73 and
// 76 event-timed, 16 tiles 15.1 and 12.9.)
constexpr int kPlanBatch = 2;
static_assert(kMaxWaves + 14 <= 32, "sort plan lists");

__device__ __forceinline__ void sort_plan_unit(const SortArgs &a, int spi, int t0)
{
    constexpr int NB = kPlanBatch;
    const int lane = threadIdx.x & 63;
    // one tile per wavefront: the index is wavefront-uniform (scalar registers)
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int t = t0 + wv;
    const SortSpecies &sp = a.sp[spi];
    const int n_tiles = a.n_tiles;

    // ---------------- the new section
    int A, B;
    if (a.scan == kScanLocal) {
        // every block counts all (at most kScanBlock) tiles by itself
        __shared__ int s_off[kScanBlock + 1];
        int total;
        const int ex = block_exclusive(tile_count_new(a, sp, threadIdx.x), total);
        s_off[threadIdx.x] = ex;
        if (threadIdx.x == 0) s_off[kScanBlock] = total;
        __syncthreads();
        if (t >= n_tiles) return;   // whole wavefront
        A = s_off[t];
        B = s_off[t + 1];
    } else {
        if (t >= n_tiles) return;
        const int blk = t / kScanBlock;
        int base;
        if (a.scan == kScanSums) {   // bsum: block totals, at most kScanDirect of them
            base = lane < blk ? sp.bsum[lane] : 0;
            A = sp.pre[t];
            B = sp.cnew[t];
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) base += __shfl_xor(base, d, 64);
        } else {                     // bsum: their exclusive prefix
            base = sp.bsum[blk];
            A = sp.pre[t];
            B = sp.cnew[t];
        }
        A += base;
        B += A;
    }
    if (lane == 0) {
        sp.off[t] = A;
        if (t == n_tiles - 1) {
            sp.off[n_tiles] = B;
            if (B != sort_expect(sp)) atomicOr(a.err, kErrCount);
        }
    }

    const int ntx = a.ntx, nty = a.nty;
    const int T = a.tile;
    const int W = a.waves;   // leaver sub-lists per tile
    const int tx = t % ntx, ty = t / ntx;
    const int gx0 = tx * T, gy0 = ty * T;

    // ---------------- the sources of t (lane o < 9: the tile from which
    // direction o leads to t), their old sections and their lists for t
    int so = -1, so_a = 0, so_b = 0, lbase = 0, llen = 0;
    bool bad = false;
    if (lane < 9) {
        so = wrap_s(ty - (lane / 3 - 1), nty) * ntx + wrap_s(tx - (lane % 3 - 1), ntx);
        const PIC_GLOBAL vi4a *rec = (const PIC_GLOBAL vi4a *)(sp.cnt + (int64_t)so * kCntStride);
        const vi4a r0 = rec[0], r1 = rec[1];
        const int r8 = gp(sp.cnt)[(int64_t)so * kCntStride + 8];
        so_a = gp(sp.offp)[so];
        so_b = gp(sp.offp)[so + 1];
        const int c[9] = {r0.x, r0.y, r0.z, r0.w, 0, r1.y, r1.z, r1.w, r8};   // direction 4 has no list
        int start = 0;
#pragma unroll
        for (int d = 0; d < 9; ++d) {
            if (d < lane) start += c[d];
            if (d == lane) llen = c[d];
        }
        bad = start < 0 || llen < 0 || start + llen > so_b - so_a;
        if (bad) start = llen = 0;
        lbase = so_a + start;
    }
    const int sub = lane >= 1 && lane <= W ? gp(sp.cnt)[(int64_t)t * kCntStride + kCntSub + lane - 1] : 0;
    int i0 = 0, i1 = 0;
    if (sp.inj_off) {
        i0 = sp.n + sp.inj_off[t];
        i1 = sp.n + sp.inj_off[t + 1];
    }
    // the order of the sources: by tile (equal ones, on an axis of one or two
    // tiles, by direction: all but one of their lists are empty)
    int rank = 0;
#pragma unroll
    for (int o = 0; o < 9; ++o) {
        const int v = __builtin_amdgcn_readlane(so, o);
        if (v < so || (v == so && o < lane)) ++rank;
    }
    const int rank4 = __builtin_amdgcn_readlane(rank, 4);
    const int oA = __builtin_amdgcn_readlane(so_a, 4), oB = __builtin_amdgcn_readlane(so_b, 4);
    // Whether the particle at `slot` of another tile's old section, with
    // tile-relative cell lc, has moved into t: its cell lies one tile off
    // its own in some offset o, and the source of t in offset o is the tile
    // whose old section holds the slot.  A particle that left the moving
    // window is in no tile.  All lanes take part.
    auto arrived = [&](int lc, int slot) {
        const int lx = tcell_x(lc), ly = tcell_y(lc);
        const int o = (ly < 0 ? 0 : (ly >= T ? 6 : 3)) + (lx < 0 ? 0 : (lx >= T ? 2 : 1));
        const int sa = __shfl(so_a, o, 64), sb = __shfl(so_b, o, 64);
        return o != 4 && (lc & 0xffff) != kTCellRemoved && slot >= sa && slot < sb;
    };

    // ---------------- the lists: first index, length; of a neighbour's list
    // also its old section's first slot and length
    const int lA = max(A, oA), lB = min(B, oB);
    int dbm = 0, dlen = 0, ds0 = 0, dns = 0;
    {
        const int m = lane - (W + 2);   // mover lists 0 .. 9
        int from = 0;                   // the direction whose list this is
#pragma unroll
        for (int o = 0; o < 9; ++o) {
            const int r = __builtin_amdgcn_readlane(rank, o);
            if (o != 4 && r + (r > rank4 ? 1 : 0) == m) from = o;
        }
        const int fb = __shfl(lbase, from, 64), fl = __shfl(llen, from, 64);
        const int fa = __shfl(so_a, from, 64), fe = __shfl(so_b, from, 64);
        if (lane == 0) {
            dbm = A;
            dlen = max(0, min(B, oA) - A);
        } else if (lane <= W) {
            int wlo, whi;
            wave_range(oA, oB, lane - 1, W, wlo, whi);
            dbm = wlo;
            dlen = lA < lB ? min(sub, whi - wlo) : 0;
        } else if (lane == W + 1) {
            dbm = max(A, oB);
            dlen = max(0, B - dbm);
        } else if (m == rank4) {
            dbm = oA;
            dlen = max(0, min(oB, A) - oA);
        } else if (m == rank4 + 1) {
            dbm = max(oA, B);
            dlen = max(0, oB - dbm);
        } else if (m < 10) {
            dbm = fb;
            dlen = fl;
            ds0 = fa;
            dns = fe - fa;
        } else if (m == 10 && sp.inj_off) {
            dbm = i0;
            dlen = max(0, min(i1, A) - i0);
        } else if (m == 11 && sp.inj_off) {
            dbm = max(i0, B);
            dlen = max(0, i1 - dbm);
        }
    }
    int total;
    const int ex = wave_exclusive(dlen, total);
    dbm -= ex;   // candidate k of the list: base + (k - ex) = dbm + k

    // the first slot of each pushing wavefront's run of the new section
    // (lane w < W): the holes below it give that run's first hole rank
    int wlo_mine = INT_MAX, fb = 0;
    if (lane < W) {
        int whi;
        wave_range(A, B, lane, W, wlo_mine, whi);
    }

    int nh = 0, nm = 0;
    for (int k0 = 0; k0 < total; k0 += 64 * NB) {
        // ---- the candidates: their lists, then every load in flight at once
        int at[NB], s0v[NB], nsv[NB], lv[NB];
        uint32_t v[NB], rec[NB];
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int k = k0 + 64 * u + lane;
            const int L = find_list(k, ex);
            at[u] = __shfl(dbm, L, 64) + k;
            s0v[u] = __shfl(ds0, L, 64);
            nsv[u] = __shfl(dns, L, 64);
            lv[u] = k < total ? L : -1;
            v[u] = rec[u] = 0;
            if (k < total) {
                const int m = L - (W + 2);
                if (L >= 1 && L <= W) {
                    v[u] = gp(sp.leav)[at[u]];
                } else if (m >= 0 && m < 10 && m != rank4 && m != rank4 + 1) {
                    const vi2a e = ((const PIC_GLOBAL vi2a *)sp.dlist)[(int64_t)at[u] * kListStride];
                    v[u] = (uint32_t)e.x;
                    rec[u] = (uint32_t)e.y;
                } else {
                    v[u] = (uint32_t)(int)gp(sp.p.cell)[at[u]];
                    // a sorted state (the window's sort): every particle is in the
                    // tile of its section, its cell relative to it modulo T
                    if (a.rebase && (v[u] & 0xffffu) != (uint32_t)kTCellRemoved)
                        v[u] = (uint32_t)tcell_pack(tcell_x((int)v[u]) & (T - 1), tcell_y((int)v[u]) & (T - 1));
                }
            }
        }
        // ---- the ballots, in candidate order: holes first, then movers
        int rr[NB];
        unsigned mvf = 0, flf = 0;   // per iteration: a mover of this lane, from the leaver records
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int L = lv[u], m = L - (W + 2);
            bool ph = false, pm = false, fl = false;
            int slot = at[u];
            const bool in_t = arrived((int)v[u], slot);
            if (L == 0 || L == W + 1) {
                // (a new particle of t appended at a slot of [A, B) stays there)
                ph = !in_t && !(slot >= i0 && slot < i1);
            } else if (L >= 1 && L <= W) {
                slot = oA + (int)(v[u] >> 4);
                ph = slot >= lA && slot < lB;
            } else if (L >= 0 && (m == rank4 || m == rank4 + 1 || m >= 10)) {
                pm = tcell_inside((int)v[u], T);   // t's own slots, or its new particles
            } else if (L >= 0) {
                if (v[u] >= (uint32_t)nsv[u] || rec[u] >= (uint32_t)nsv[u]) {
                    bad = true;
                } else {
                    const int ms = s0v[u] + (int)v[u];
                    pm = !(ms >= A && ms < B);
                    fl = true;
                    at[u] = s0v[u] + (int)rec[u];
                }
            }
            const unsigned long long mh = __ballot(ph);
            const int r = nh + lane_rank_s(mh);
            if (ph && r < B - A) sp.hole[(int64_t)A + r] = slot;
            nh += __popcll(mh);
            if (mh != 0ull)
                for (int w = 0; w < W; ++w) {
                    const int lo_w = __builtin_amdgcn_readlane(wlo_mine, w);
                    const int c = __popcll(__ballot(ph && slot < lo_w));
                    if (lane == w) fb += c;
                }
            const unsigned long long mm = __ballot(pm);
            rr[u] = nm + lane_rank_s(mm);
            if (pm && rr[u] < B - A) mvf |= 1u << u;
            if (fl) flf |= 1u << u;
            nm += __popcll(mm);
        }
        if (__ballot(mvf != 0) == 0ull) continue;
        // ---- the movers' data, every load in flight at once, then staged in
        // hole order (contiguous stores)
        Chunk6 dv[NB];
#pragma unroll
        for (int u = 0; u < NB; ++u)
            if (mvf >> u & 1u) dv[u] = flf >> u & 1u ? load_leaver(sp.lrec, at[u]) : load_parts(sp.p, at[u], gx0, gy0, a.rebase ? T - 1 : -1);
#pragma unroll
        for (int u = 0; u < NB; ++u)
            if (mvf >> u & 1u) {
                const Chunk6 &c = dv[u];
                put_leaver(sp.srec, (int64_t)A + rr[u], c.cell, c.x, c.y, c.ux, c.uy, c.uz);
            }
    }

    const bool anybad = __ballot(bad) != 0ull;
    const int m = min(min(nh, nm), B - A);   // holes and movers agree unless the records were corrupt
    if (lane == 0) {
        if (nh != nm || anybad) atomicOr(a.err, kErrSort);
        sp.mcount[t] = m;
        sp.fcount[t] = a.defer ? m : 0;
    }
    if (a.defer && lane < W) sp.fbase[(int64_t)t * W + lane] = min(fb, m);
}

// Step (5): the staged movers of each tile into its holes.  Not launched
// when the sort is deferred (pic_step): the next push fills them as it
// streams the section.
__device__ __forceinline__ void sort_scatter_unit(const SortArgs &a, int spi, int grp)
{
    const int lane = threadIdx.x & 63;
    const int t = grp * kSortWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (t >= a.n_tiles) return;
    const SortSpecies &sp = a.sp[spi];
    const int A = sp.off[t], m = sp.mcount[t];
    const int gx0 = (t % a.ntx) * a.tile, gy0 = (t / a.ntx) * a.tile;
    for (int k = lane; k < m; k += 64) {
        const int64_t r = (int64_t)A + k;
        store_parts(sp.p, sp.hole[r], load_leaver(sp.srec, r), gx0, gy0);
    }
}

// ---- The motion-class sort (the alternative of Sec. 4.3, after
// Germaschewski et al.): by the Courant condition a particle ends a step in
// its own tile or one of the eight around it, so its motion falls into one of
// nine classes d = (dty + 1) * 3 + (dtx + 1) -- the step from the tile whose
// section holds it to its new tile, counted +1 on an axis of two tiles, the
// push kernel's direction code -- and the push has already counted the
// particles of every (tile, class).  One pass then moves every particle of
// source tile s and class d to its place in the new order (new tile, class,
// old slot) in the staging arrays: base(s, d) = the new section start of the
// destination tile t = s + step(d), plus the counts of the classes before d
// arriving at t from their own source tiles.  A second pass copies the
// staging arrays back.  Out of place: reads and writes every particle twice,
// so it pays only when most particles change tile.

// The motion class of a particle with tile-relative cell lc (tiles of edge
// T, ntx x nty of them): the push kernel's direction code of the step to the
// tile it is in now (+1 on an axis of two tiles, either way), or 9 if that
// is more than one tile away or the particle left the moving window.
__device__ __forceinline__ int motion_class(int lc, int T, int ntx, int nty)
{
    const int lx = tcell_x(lc), ly = tcell_y(lc);
    const int stx = lx < 0 ? (ntx == 2 ? 1 : -1) : (lx >= T ? 1 : 0);
    const int sty = ly < 0 ? (nty == 2 ? 1 : -1) : (ly >= T ? 1 : 0);
    const bool far = lx < -T || lx >= 2 * T || ly < -T || ly >= 2 * T;   // the removed mark too
    return far ? 9 : (sty + 1) * 3 + (stx + 1);
}

constexpr int kTCellNone = 0x10000;   // no particle (cells are 16 bits)

struct Part6 {
    int cell;
    float x, y, ux, uy, uz;
};

// A whole-array pass of the motion-class sort reads every particle once, so
// its loads carry the non-temporal hint (as the push's particle stream
// does); its stores start mid-line (class runs), where the hint costs.
__device__ __forceinline__ Part6 load_part(const Parts &p, int i)
{
    return Part6{__builtin_nontemporal_load(p.cell + i), __builtin_nontemporal_load(p.x + i),
                 __builtin_nontemporal_load(p.y + i),    __builtin_nontemporal_load(p.ux + i),
                 __builtin_nontemporal_load(p.uy + i),   __builtin_nontemporal_load(p.uz + i)};
}

__device__ __forceinline__ void store_part(const Parts &p, int i, const Part6 &v)
{
    p.cell[i] = v.cell;
    p.x[i] = v.x;
    p.y[i] = v.y;
    p.ux[i] = v.ux;
    p.uy[i] = v.uy;
    p.uz[i] = v.uz;
}

// The nt source tiles from tile t0 on, one after the other, each by the whole
// block: the section's 64-aligned chunks are split into one run per
// wavefront; a first pass counts every run's particles per class (eight chunks
// in flight: one at a time it took a fifth of the kernel, 16.8 M particles 185
// us, now 162, 4.7 TB/s), a second
// streams the runs again and moves each particle to its slot (its class's
// first slot in the destination, the class's particles in the earlier runs,
// its rank in its chunk).  One tile per block for a single simulation (many
// wavefronts in flight), kSortWaves per work item in a batch.
__device__ __forceinline__ void motion_scatter_unit(const SortArgs &a, int spi, int t0, int nt)
{
    constexpr int W = kSortWaves;
    __shared__ int s_cls[W][9];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const SortSpecies &sp = a.sp[spi];
    const int ntx = a.ntx, nty = a.nty;
    const int T = a.tile;
    for (int q = 0; q < nt; ++q) {
        const int s = t0 + q;
        if (s >= a.n_tiles) break;   // uniform over the block
        const int sx = s % ntx, sy = s / ntx;
        const int oA = sp.offp[s], oB = sp.offp[s + 1];
        int lo, hi;
        wave_range(oA, oB, w, W, lo, hi);
        // pass 1: lane d counts the run's particles of class d
        int mine = 0;
        constexpr int U = 8;   // chunks in flight
        for (int c0 = (lo >> 6) << 6; c0 < hi; c0 += 64 * U) {
            int lc[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int i = c0 + 64 * u + lane;
                lc[u] = i >= lo && i < hi ? gp(sp.p.cell)[i] : kTCellNone;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int d = lc[u] == kTCellNone ? 10 : motion_class(lc[u], T, ntx, nty);
#pragma unroll
                for (int k = 0; k < 9; ++k) {
                    const int c = __popcll(__ballot(d == k));
                    if (lane == k) mine += c;
                }
            }
        }
        if (lane < 9) s_cls[w][lane] = mine;
        __syncthreads();
        // lane d < 9: the run's first slot for class d and the class's end
        int pos = 0, end = 0;
        bool bad = false;
        if (lane < 9) {
            const int dx = lane % 3 - 1, dy = lane / 3 - 1;
            const int t = wrap_s(sy + dy, nty) * ntx + wrap_s(sx + dx, ntx);
            const int tx = t % ntx, ty = t / ntx;
            pos = sp.off[t];
            for (int d2 = 0; d2 < lane; ++d2) {
                const int src = wrap_s(ty - (d2 / 3 - 1), nty) * ntx + wrap_s(tx - (d2 % 3 - 1), ntx);
                pos += sp.cnt[(int64_t)src * kCntStride + d2];
            }
            const int total = sp.cnt[(int64_t)s * kCntStride + lane];
            end = pos + total;
            int all = 0;
            for (int w2 = 0; w2 < W; ++w2) {
                if (w2 < w) pos += s_cls[w2][lane];
                all += s_cls[w2][lane];
            }
            bad = all != total;   // the push's counts and the cells disagree
        }
        // pass 2: the particles to their slots, the next two chunks in flight
        int c0 = (lo >> 6) << 6;
        Part6 nxt{}, nxt2{};
        if (c0 + lane >= lo && c0 + lane < hi) nxt = load_part(sp.p, c0 + lane);
        if (c0 + 64 + lane >= lo && c0 + 64 + lane < hi) nxt2 = load_part(sp.p, c0 + 64 + lane);
        for (; c0 < hi; c0 += 64) {
            const Part6 cur = nxt;
            nxt = nxt2;
            const int i = c0 + lane;
            const bool in = i >= lo && i < hi;
            const int i3 = i + 128;
            if (i3 >= lo && i3 < hi) nxt2 = load_part(sp.p, i3);
            const int d = in ? motion_class(cur.cell, T, ntx, nty) : 10;
            unsigned long long m_d = 0ull;
            int taken = 0;
#pragma unroll
            for (int k = 0; k < 9; ++k) {
                const unsigned long long m = __ballot(d == k);
                if (d == k) m_d = m;
                if (lane == k) taken = __popcll(m);
            }
            const int at = __shfl(pos, d < 9 ? d : 0, 64) + lane_rank_s(m_d);
            const int lim = __shfl(end, d < 9 ? d : 0, 64);
            if (in) {
                if (d < 9 && at < lim && (unsigned)at < (unsigned)sp.n) {
                    Part6 v = cur;   // its cell relative to the tile it is in now
                    v.cell = tcell_pack(tcell_x(cur.cell) & (T - 1), tcell_y(cur.cell) & (T - 1));
                    store_part(sp.stg, at, v);
                }
                else bad = true;
            }
            pos += taken;
        }
        const bool anybad = __ballot(bad) != 0ull;
        if (lane == 0 && anybad) atomicOr(a.err, kErrSort);
        if (threadIdx.x == 0) sp.mcount[s] = 0;   // pic_diag's mover count: not tracked by this sort
        __syncthreads();   // s_cls is reused by the next tile
    }
    // the copy back is left to the next push (read by launches after this one)
    if (a.defer && threadIdx.x == 0) *a.stg_live = 1;
}

// The new sections of the nt tiles from t0 on (contiguous) from the staging
// arrays into the particle arrays, by the whole block, four particles per
// thread in flight; live: only if the copy was left pending (*stg_live).
__device__ __forceinline__ void motion_copy_unit(const SortArgs &a, int spi, int t0, int nt, bool live = false)
{
    if (live && *a.stg_live == 0) return;
    const SortSpecies &sp = a.sp[spi];
    if (t0 >= a.n_tiles) return;
    const int t1 = min(t0 + nt, a.n_tiles);
    const int A = sp.off[t0], B = sp.off[t1];
    constexpr int U = 4;
    for (int i0 = A + (int)threadIdx.x; i0 < B; i0 += U * kBlock) {
        Part6 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i0 + u * kBlock < B) v[u] = load_part(sp.stg, i0 + u * kBlock);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i0 + u * kBlock < B) store_part(sp.p, i0 + u * kBlock, v[u]);
    }
}

// ---- single-simulation kernels: blockIdx.y = species
__global__ void __launch_bounds__(kScanBlock) k_sort_count(SortArgs a) { sort_count_unit(a, blockIdx.y, blockIdx.x); }
__global__ void __launch_bounds__(1024) k_sort_scan_blocks(SortArgs a) { sort_scan_unit(a, blockIdx.x); }
__global__ void __launch_bounds__(kScanBlock) k_sort_add_base(SortArgs a) { sort_add_unit(a, blockIdx.y, blockIdx.x); }
__global__ void __launch_bounds__(kScanBlock) k_sort_add_direct(SortArgs a)
{
    sort_add_direct_unit(a, blockIdx.y, blockIdx.x);
}
// A fill left pending by a deferred sort, done on its own (before anything
// works on the tile-relative cells other than a push: the window move): tile
// t's fcount[t] staged movers into its holes, as the next push would, and
// fcount[t] back to 0.
__device__ __forceinline__ void fill_unit(const SortArgs &a, int spi, int grp)
{
    const int lane = threadIdx.x & 63;
    const int t = grp * kSortWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (t >= a.n_tiles) return;
    const SortSpecies &sp = a.sp[spi];
    const int A = sp.off[t], m = sp.fcount[t];
    const int gx0 = (t % a.ntx) * a.tile, gy0 = (t / a.ntx) * a.tile;
    for (int k = lane; k < m; k += 64) {
        const int64_t r = (int64_t)A + k;
        store_parts(sp.p, sp.hole[r], load_leaver(sp.srec, r), gx0, gy0);
    }
    if (lane == 0 && m != 0) sp.fcount[t] = 0;
}

// One tile for a reader of the particle arrays, by `nt` threads of a block (a
// power of two from 16): a fill left pending (as fill_unit), then the
// whole-grid cells of the tile's section into the caller's cell array from the
// tile-relative ones (the cell of a particle that has left its tile wraps
// across the periodic seam).  rebase: a sorted state, each cell relative to the
// tile modulo its edge.  All threads of the block take part (a barrier orders
// the fill's cells before the section's reads); t may be past the last tile.
//
// Bound by HBM: 6 bytes a particle.  Four slots per thread and pass, from
// 8-byte groups of the cell array on, by as many threads as the tile's
// particles occupy (settle_threads): one wavefront per tile and one slot
// per lane, as this was first, left a 32 x 32 tile's 16,384 particles to 256
// dependent passes.  Fill and cells, before as two launches and now: 16.8 M
// particles in 1,024 tiles 135 -> 26 us, 67 M in 4,096 tiles 258 -> 121 us
// (4.0 TB/s counting the staged movers), 65,536 in 16 tiles 37 -> 5 us.
typedef int16_t vs4 __attribute__((ext_vector_type(4)));
typedef int32_t vi4 __attribute__((ext_vector_type(4), aligned(4)));   // the caller's array: 4-byte aligned
__device__ __forceinline__ void settle_tile(const SortArgs &a, int spi, int t, int tid, int nt, bool rebase)
{
    const SortSpecies &sp = a.sp[spi];
    const bool on = t < a.n_tiles;
    const int gx0 = (t % a.ntx) * a.tile, gy0 = (t / a.ntx) * a.tile;
    const int A = on ? sp.off[t] : 0, B = on ? sp.off[t + 1] : 0;
    const int m = on ? sp.fcount[t] : 0;
    for (int k = tid; k < m; k += nt) {
        const int64_t r = (int64_t)A + k;
        store_parts(sp.p, sp.hole[r], load_leaver(sp.srec, r), gx0, gy0);
    }
    if (nt <= 64) {   // within one wavefront: its accesses are in order
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
        __syncthreads();
    }
    if (tid == 0 && m != 0) sp.fcount[t] = 0;
    const int mask = rebase ? a.tile - 1 : -1;
    auto whole = [&](int lc) {
        return wrap_s(gx0 + (tcell_x(lc) & mask), a.nx) | (wrap_s(gy0 + (tcell_y(lc) & mask), a.ny) << 16);
    };
    for (int64_t i = (int64_t)(A & ~3) + 4 * tid; i < B; i += 4 * nt) {
        // (a group may reach past the section, and past the last slot into the
        // padding behind the workspace's 256-byte aligned array; unused there)
        const vs4 c = *(const PIC_GLOBAL vs4 *)(sp.p.cell + i);
        const vi4 g{whole(c.x), whole(c.y), whole(c.z), whole(c.w)};
        if (i >= A && i + 4 <= B) {
            *(PIC_GLOBAL vi4 *)(sp.gcell + i) = g;
        } else {   // the section's ends
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (i + u >= A && i + u < B) gp(sp.gcell)[i + u] = g[u];
        }
    }
}

__global__ void __launch_bounds__(kBlock) k_fill(SortArgs a) { fill_unit(a, blockIdx.y, blockIdx.x); }
// 1 << sh threads per tile, as many tiles side by side as the block holds
constexpr int kSettleBlock = 1024;   // threads per tile, at most
__global__ void __launch_bounds__(kSettleBlock) k_settle(SortArgs a, int sh, int rebase)
{
    const int q = threadIdx.x >> sh;
    settle_tile(a, blockIdx.y, blockIdx.x * (blockDim.x >> sh) + q, threadIdx.x & ((1 << sh) - 1), 1 << sh, rebase != 0);
}
__global__ void __launch_bounds__(kBlock) k_sort_plan(SortArgs a)
{
    sort_plan_unit(a, blockIdx.y, blockIdx.x * kSortWaves);
}

// The plan and the field half (of a large grid its E step) in one launch: they
// touch disjoint data, and the plan's wavefronts, which mostly wait, share the
// chip with the field half's stream.  The plan's blocks come first, a tile per
// wavefront of the whole block; the field's fill the chip as they drain.
// (As two chains on two streams the same work paid for the second chain's
// launches and two event waits: a 64 x 64 step 53 us, now 29; a 512^2 two-beam
// step 383, now 358.)  us a step with the plan's blocks of four tiles spread
// between the field's / four tiles, first / ten tiles, spread / ten, first:
// 2048^2 32 x 32 tiles 796 / 789 / 798 / 788; 1408^2 16 x 16 tiles 427 / 423 /
// 436 / 420; 1024^2 16 x 16, 64 particles a cell 696 / 692 / 695 / 686.
struct PlanMix {
    int n, n_plan;   // blocks, plan blocks
    int tiles;       // tiles per plan block
};

template <bool FOLD, int T, int H>
__global__ void __launch_bounds__(kEbThreads) k_plan_field(SortArgs a, FieldArgs f, PlanMix mix)
{
    const int p = linear_block(), q = p - mix.n_plan;
    if (p >= mix.n) return;
    if (q < 0) {
        if ((int)threadIdx.x >= 64 * mix.tiles) return;   // (an ended wavefront holds up no barrier)
        const int groups = mix.n_plan / a.n_species;
        sort_plan_unit(a, p / groups, p % groups * mix.tiles);
    } else {
        const int cols = eb_cols(f.nx);
        field_eb_region<FOLD, T, H>(f, q % cols, q / cols);
    }
}

// The same with the E step alone of a large grid: no block is larger than the
// plan's four wavefronts, so the two kinds take each other's places freely.
// us a step, blocks of ten wavefronts or, from 16,384 tiles on, two launches /
// this: 2048^2 32 x 32 tiles 767 / 763, with one particle a cell 213 / 203;
// 16 x 16 840 / 830 and 303 / 290; 8 x 8, one a cell 687 / 672.
template <bool FOLD, int T, int H>
__global__ void __launch_bounds__(kBlock) k_plan_e(SortArgs a, FieldArgs f, PlanMix mix)
{
    const int p = linear_block(), q = p - mix.n_plan;
    if (p >= mix.n) return;
    if (q < 0) {
        const int groups = mix.n_plan / a.n_species;
        sort_plan_unit(a, p / groups, p % groups * kSortWaves);
    } else {
        field_e_block<FOLD, T, H>(f, q);
    }
}
static_assert(kEThreads == kBlock, "a block of either kind");

template <bool FOLD, int T, int H>
__global__ void __launch_bounds__(kEbThreads) k_plan_field_b(const SortArgs *sd, const int4 *si, const FieldArgs *fd,
                                                         const int4 *fi, PlanMix mix)
{
    const int p = linear_block(), q = p - mix.n_plan;
    if (p >= mix.n) return;
    if (q < 0) {
        if ((int)threadIdx.x >= 64 * mix.tiles) return;
        const int4 w = si[p];
        sort_plan_unit(sd[w.x], w.y, w.z * kSortWaves);
    } else {
        const int4 w = fi[q];
        field_eb_region<FOLD, T, H>(fd[w.x], w.y, w.z);
    }
}

__global__ void __launch_bounds__(kBlock) k_sort_scatter(SortArgs a) { sort_scatter_unit(a, blockIdx.y, blockIdx.x); }
// single simulation: one tile per block
__global__ void __launch_bounds__(kBlock) k_motion_scatter(SortArgs a) { motion_scatter_unit(a, blockIdx.y, blockIdx.x, 1); }
__global__ void __launch_bounds__(kBlock) k_motion_copy(SortArgs a) { motion_copy_unit(a, blockIdx.y, blockIdx.x, 1); }
__global__ void __launch_bounds__(kBlock) k_motion_copy_live(SortArgs a)
{
    motion_copy_unit(a, blockIdx.y, blockIdx.x, 1, true);
}

// ---- many simulations: one block per work item (sim, species, unit)
__global__ void __launch_bounds__(kScanBlock) k_sort_count_b(const SortArgs *d, const int4 *it)
{
    const int4 w = it[blockIdx.x];
    sort_count_unit(d[w.x], w.y, w.z);
}
__global__ void __launch_bounds__(1024) k_sort_scan_blocks_b(const SortArgs *d, const int4 *it)
{
    const int4 w = it[blockIdx.x];
    sort_scan_unit(d[w.x], w.y);
}
__global__ void __launch_bounds__(kScanBlock) k_sort_add_direct_b(const SortArgs *d, const int4 *it)
{
    const int4 w = it[blockIdx.x];
    sort_add_direct_unit(d[w.x], w.y, w.z);
}
__global__ void __launch_bounds__(kBlock) k_sort_plan_b(const SortArgs *d, const int4 *it, int n)
{
    const int b = linear_block();
    if (b >= n) return;
    const int4 w = it[b];
    sort_plan_unit(d[w.x], w.y, w.z * kSortWaves);
}
__global__ void __launch_bounds__(kScanBlock) k_sort_add_base_b(const SortArgs *d, const int4 *it)
{
    const int4 w = it[blockIdx.x];
    sort_add_unit(d[w.x], w.y, w.z);
}
// the kSortWaves tiles of an item, 1 << sh threads each, by a block or (a row
// of the grid per part) several
__global__ void __launch_bounds__(kSettleBlock) k_settle_b(const SortArgs *d, const int4 *it, int sh, int rebase)
{
    const int4 w = it[blockIdx.x];
    const int q = blockIdx.y * (blockDim.x >> sh) + (threadIdx.x >> sh);
    settle_tile(d[w.x], w.y, w.z * kSortWaves + q, threadIdx.x & ((1 << sh) - 1), 1 << sh, rebase != 0);
}

__global__ void __launch_bounds__(kBlock) k_motion_scatter_b(const SortArgs *d, const int4 *it)
{
    const int4 w = it[blockIdx.x];
    motion_scatter_unit(d[w.x], w.y, w.z * kSortWaves, kSortWaves);
}
__global__ void __launch_bounds__(kBlock) k_motion_copy_b(const SortArgs *d, const int4 *it)
{
    const int4 w = it[blockIdx.x];
    motion_copy_unit(d[w.x], w.y, w.z * kSortWaves, kSortWaves);
}

// ---- tile_offset from caller particles: whether every cell is in the grid
// (kErrOrder) and the cells are grouped by tile (kErrGroup), then, for
// grouped cells, off[t] = the first slot whose tile is >= t (a binary search
// per tile: no atomics, so many particles per tile cost nothing extra)
__global__ void k_init_check(const int32_t *__restrict__ cell, int32_t n, int nx, int ny, int tsh, int ntx,
                             int *err)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int c = cell[i];
    const int ix = c & 0xffff, iy = c >> 16;
    if (c < 0 || ix >= nx || iy >= ny) {
        atomicOr(err, kErrOrder);
        return;
    }
    if (i + 1 < n) {
        const int c2 = cell[i + 1];
        const int t = (iy >> tsh) * ntx + (ix >> tsh);
        const int t2 = ((c2 >> 16) >> tsh) * ntx + ((c2 & 0xffff) >> tsh);
        if (c2 >= 0 && t2 < t) atomicOr(err, kErrGroup);
    }
}

__global__ void k_init_offsets(const int32_t *__restrict__ cell, int32_t n, int tsh, int ntx, int n_tiles,
                               int32_t *__restrict__ off)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t > n_tiles) return;
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = lo + ((hi - lo) >> 1);
        const int c = cell[mid];
        const int tm = c < 0 ? -1 : ((c >> 16) >> tsh) * ntx + ((c & 0xffff) >> tsh);
        if (tm < t) lo = mid + 1;
        else hi = mid;
    }
    off[t] = lo;
}

// How the plan gets the new sections: up to one scan block of tiles each plan
// block counts them all itself (at most 64 blocks then read 2,304 counts each,
// below the cost of a launch); else from k_sort_count's prefixes, the blocks
// before its own added by the plan while one load per lane holds them.
static int scan_mode(int64_t n_blocks)
{
    return n_blocks <= 1 ? kScanLocal : (n_blocks <= kScanDirect ? kScanSums : kScanBases);
}

static void launch_sort_counts(const SortArgs &a, int n_tiles, hipStream_t s)
{
    const int nb = (n_tiles + kScanBlock - 1) / kScanBlock;
    hipLaunchKernelGGL(k_sort_count, dim3(nb, a.n_species), dim3(kScanBlock), 0, s, a);
    if (nb > kScanDirect) hipLaunchKernelGGL(k_sort_scan_blocks, dim3(a.n_species), dim3(1024), 0, s, a);
}

void launch_sort_scan(const SortArgs &a, int n_tiles, bool offsets, hipStream_t s)
{
    const int nb = (n_tiles + kScanBlock - 1) / kScanBlock;
    if (offsets || scan_mode(nb) != kScanLocal) launch_sort_counts(a, n_tiles, s);
    if (!offsets) return;
    if (nb <= kScanDirect) hipLaunchKernelGGL(k_sort_add_direct, dim3(nb, a.n_species), dim3(kScanBlock), 0, s, a);
    else hipLaunchKernelGGL(k_sort_add_base, dim3(nb, a.n_species), dim3(kScanBlock), 0, s, a);
}

void launch_sort_plan(const SortArgs &args, int n_tiles, hipStream_t s)
{
    SortArgs a = args;
    a.scan = scan_mode((n_tiles + kScanBlock - 1) / kScanBlock);
    hipLaunchKernelGGL(k_sort_plan, dim3((n_tiles + kSortWaves - 1) / kSortWaves, a.n_species), dim3(kBlock), 0, s, a);
}

void launch_sort_scatter(const SortArgs &a, int n_tiles, hipStream_t s)
{
    hipLaunchKernelGGL(k_sort_scatter, dim3((n_tiles + kSortWaves - 1) / kSortWaves, a.n_species), dim3(kBlock), 0,
                       s, a);
}

void launch_fill(const SortArgs &a, int n_tiles, hipStream_t s)
{
    hipLaunchKernelGGL(k_fill, dim3((n_tiles + kSortWaves - 1) / kSortWaves, a.n_species), dim3(kBlock), 0, s, a);
}

void launch_settle(const SortArgs &a, int n_tiles, bool rebase, hipStream_t s)
{
    int64_t n = 0;
    for (int k = 0; k < a.n_species; ++k) n = std::max<int64_t>(n, a.sp[k].n);
    const int nt = settle_threads(n, n_tiles, kSettleBlock);
    const int block = std::max(nt, kBlock), tiles = block / nt;
    hipLaunchKernelGGL(k_settle, dim3((n_tiles + tiles - 1) / tiles, a.n_species), dim3(block), 0, s, a,
                       __builtin_ctz(nt), rebase ? 1 : 0);
}

void launch_settle_batch(const SortBatch &b, int64_t particles, int64_t sections, bool rebase, hipStream_t s)
{
    if (b.n_plan == 0) return;
    const int nt = settle_threads(particles, sections, kSettleBlock);
    const int block = std::min(std::max(nt, kBlock), nt * kSortWaves);
    hipLaunchKernelGGL(k_settle_b, dim3(b.n_plan, nt * kSortWaves / block), dim3(block), 0, s, b.descs, b.plan_items,
                       __builtin_ctz(nt), rebase ? 1 : 0);
}

int batch_scan_mode(int max_blocks) { return max_blocks <= kScanDirect ? kScanSums : kScanBases; }

void launch_sort_scan_batch(const SortBatch &b, bool offsets, hipStream_t s)
{
    if (b.n_count == 0) return;
    hipLaunchKernelGGL(k_sort_count_b, dim3(b.n_count), dim3(kScanBlock), 0, s, b.descs, b.count_items);
    if (b.max_blocks > kScanDirect)
        hipLaunchKernelGGL(k_sort_scan_blocks_b, dim3(b.n_scan), dim3(1024), 0, s, b.descs, b.scan_items);
    if (!offsets) return;
    if (b.max_blocks <= kScanDirect)
        hipLaunchKernelGGL(k_sort_add_direct_b, dim3(b.n_count), dim3(kScanBlock), 0, s, b.descs, b.count_items);
    else
        hipLaunchKernelGGL(k_sort_add_base_b, dim3(b.n_count), dim3(kScanBlock), 0, s, b.descs, b.count_items);
}

void launch_motion_batch(const SortBatch &b, hipStream_t s)
{
    if (b.n_plan == 0) return;
    hipLaunchKernelGGL(k_motion_scatter_b, dim3(b.n_plan), dim3(kBlock), 0, s, b.descs, b.plan_items);
    hipLaunchKernelGGL(k_motion_copy_b, dim3(b.n_plan), dim3(kBlock), 0, s, b.descs, b.plan_items);
}

namespace {

struct PlanFieldLaunch {
    const SortArgs *a;       // single
    const FieldArgs *f;
    int n_plan, n_field, tiles;
    const SortBatch *b;      // batched
    const FieldArgs *fd;
    const int4 *fi;
    hipStream_t s;
    template <bool FOLD, int T, int H>
    void run() const
    {
        const PlanMix mix{n_plan + n_field, n_plan, tiles};
        const bool large = a && !f->eedge;
        const BlockGrid g = block_grid(mix.n, large ? kBlock : kEbThreads);
        const dim3 grid(g.x, g.y);
        if (large) {   // the second B half step after E
            hipLaunchKernelGGL((k_plan_e<FOLD, T, H>), grid, dim3(kBlock), 0, s, *a, *f, mix);
            launch_field_b(*f, s);
        } else if (a) {
            hipLaunchKernelGGL((k_plan_field<FOLD, T, H>), grid, dim3(kEbThreads), 0, s, *a, *f, mix);
        } else
            hipLaunchKernelGGL((k_plan_field_b<FOLD, T, H>), grid, dim3(kEbThreads), 0, s, b->descs, b->plan_items, fd,
                               fi, mix);
    }
};

}  // namespace

constexpr int kChipWaves = 256 * 32;   // wavefronts the device holds

void launch_plan_and_field(const SortArgs &args, int n_tiles, const FieldArgs &f, int tile, int halo, hipStream_t s)
{
    const int64_t sections = (int64_t)n_tiles * args.n_species;
    // Two launches where the plan alone fills the chip twice over (8,192
    // wavefronts): the field half's blocks of ten then find no free places.  us a
    // step, one launch / two: 16,384 tiles (1024^2, 8 x 8, one and 16 particles a
    // cell) 182 / 180, 360 / 358; 7,744 (1408^2, 16 x 16) 420 / 423.
    if (f.eedge && sections >= 2 * kChipWaves) {
        launch_sort_plan(args, n_tiles, s);
        launch_field_half(f, tile, halo, s);
        return;
    }
    SortArgs a = args;
    a.scan = scan_mode((n_tiles + kScanBlock - 1) / kScanBlock);
    // a wavefront for every tile of a full block; of fewer tiles per block as
    // long as there is no block for every compute unit (1,024 tiles of 8 x 8: 28.3 us
    // a step with four a block, 29.2 with ten), and of as many as the threads of
    // its scan where a block counts all tiles itself
    const int tiles = !f.eedge || sections < 256 * (kEbThreads / 64) ? kSortWaves : kEbThreads / 64;
    const int n_plan = (n_tiles + tiles - 1) / tiles * a.n_species;
    const int n_field = f.eedge ? eb_cols(f.nx) * eb_rows(f.ny) : e_blocks(f.nx, f.ny);
    eb_dispatch(PlanFieldLaunch{&a, &f, n_plan, n_field, tiles, nullptr, nullptr, nullptr, s}, f.jtile != nullptr,
                tile, halo);
}

void launch_plan_and_field_batch(const SortBatch &b, const FieldArgs *fields, const int4 *regions, int n_regions,
                                 bool fold, int tile, int halo, hipStream_t s)
{
    if (b.n_plan == 0) return;
    // Two launches where the plan fills the chip (its blocks have four tiles in
    // the places of ten, so the line lies lower than above).  us for two steps, one
    // launch / two: 64 members with about 5,000 tiles 1006 / 1020, 128 with 10,000
    // 2341 / 2336; 2 x 1024^2 16 x 16 tiles (8,192) 454 / 446; 48 and 128
    // of 8 x 8 tiles (15,000 and 40,000) 437 / 427, 1361 / 1281.
    if ((int64_t)b.n_plan * kSortWaves >= kChipWaves) {
        const BlockGrid g = block_grid(b.n_plan, kBlock);
        hipLaunchKernelGGL(k_sort_plan_b, dim3(g.x, g.y), dim3(kBlock), 0, s, b.descs, b.plan_items, b.n_plan);
        launch_field_half_batch(fields, regions, n_regions, fold, tile, halo, s);
        return;
    }
    eb_dispatch(PlanFieldLaunch{nullptr, nullptr, b.n_plan, n_regions, kSortWaves, &b, fields, regions, s}, fold, tile,
                halo);
}

void launch_motion_scatter(const SortArgs &a, int n_tiles, hipStream_t s)
{
    hipLaunchKernelGGL(k_motion_scatter, dim3(n_tiles, a.n_species), dim3(kBlock), 0, s, a);
}

void launch_motion_copy(const SortArgs &a, int n_tiles, hipStream_t s)
{
    hipLaunchKernelGGL(k_motion_copy, dim3(n_tiles, a.n_species), dim3(kBlock), 0, s, a);
}

void launch_motion_copy_live(const SortArgs &a, int n_tiles, hipStream_t s)
{
    hipLaunchKernelGGL(k_motion_copy_live, dim3(n_tiles, a.n_species), dim3(kBlock), 0, s, a);
    launch_set_int(a.stg_live, 0, s);
}

// Tile-relative cells of n particles grouped by tile, each inside its tile
// (checked before), from their whole-grid cells.
__global__ void __launch_bounds__(256) k_localize(const int32_t *__restrict__ cell, int16_t *__restrict__ lcell,
                                                  int32_t n, int tile)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int c = cell[i];
    lcell[i] = (int16_t)tcell_pack((c & 0xffff) & (tile - 1), (c >> 16) & (tile - 1));
}

void launch_localize(const int32_t *cell, int16_t *lcell, int32_t n, int tile, hipStream_t s)
{
    if (n > 0) hipLaunchKernelGGL(k_localize, dim3((n + 255) / 256), dim3(256), 0, s, cell, lcell, n, tile);
}

void launch_init_tiles(const int32_t *cell, int32_t n, int nx, int ny, int tile, int ntx, int n_tiles, int32_t *off,
                       int *err, hipStream_t s)
{
    const int tsh = __builtin_ctz(tile);
    if (n > 0)
        hipLaunchKernelGGL(k_init_check, dim3((n + 255) / 256), dim3(256), 0, s, cell, n, nx, ny, tsh, ntx, err);
    hipLaunchKernelGGL(k_init_offsets, dim3((n_tiles + 1 + 255) / 256), dim3(256), 0, s, cell, n, tsh, ntx, n_tiles,
                       off);
}

}  // namespace pic
