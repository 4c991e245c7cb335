// ptm_kernels.hip -- HIP kernels of the PTM classification pass for gfx950.
//
// Pipeline for one frame (Polyhedral Template Matching, arXiv:1603.05143):
//   k_setup_small     frames up to 4,096 atoms: all of the following up to the
//                     sorted copy, in one block
//   k_bounds_grid     up to 2 M atoms: finite check, bounding box, cleared
//                     counters and the cell grid
//   k_bounds          beyond, or with stage timing: finite check + bounding box
//                     (open axes); the host makes the grid
//   k_bin_count       cell id + per-cell counter (counting sort, pass 1)
//   (scan)            exclusive prefix sum of the counters
//   k_bin_scatter     sorted copy of the positions, x y z of an atom together
//                     (counting sort, pass 2)
//   k_knn_fast/exact  14 (or 18) nearest neighbours by (d^2, id), Sec. 3
//                     Euclidean order
//   k_voronoi_hull/   optional topological order (Sec. 3): Voronoi interface
//   k_voronoi_order   areas of the centre and its 18 nearest neighbours
//   k_topo            hulls of the innermost 6 / 12 / 14 neighbours with exact
//                     predicates (Sec. 4; Alg. 1 requires the centre strictly
//                     inside), start-edge codes, template table lookups
//   k_match           superposition of every candidate correspondence of
//                     the codes (eqs. 2-4, App. A), decision (Alg. 1; the
//                     full tie rule in FP64 where needed), representative,
//                     orientation, strain (eq. 6, Sec. 8), alloy (Sec. 6,
//                     Table 3), derived outputs, write-back in input order
//   k_apply_cutoff, k_rmsd_histogram, k_misorientation: post-hoc utilities
//                     (Sec. 5.1, Sec. 7)
// One lane owns one atom in every per-atom kernel (k_match also gives a
// lane one candidate of its wave's atoms); atoms are processed in cell
// order so the lanes of a wave read the same cells.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ptm_device.hpp"
#include "ptm_kernels.hpp"
#include "ptm_tables.hpp"

namespace ptm {

// --------------------------------------------------------------- helpers
__device__ inline uint32_t nib(uint64_t w, int i) { return (uint32_t)((w >> (4 * i)) & 0xF); }
__device__ inline uint64_t setnib(uint64_t w, int i, uint32_t v) {
    return (w & ~(0xFull << (4 * i))) | ((uint64_t)v << (4 * i));
}

__device__ inline int cell_coord(double x, const Grid &g, int d) {
    double u;
    if (g.periodic[d]) {
        u = x - g.L[d] * floor(x * g.invL[d]);
    } else {
        u = x - g.lo[d];
    }
    double f = floor(u * g.inv_h[d]);
    // NaN (a non-finite coordinate, refused later) also lands in cell 0
    int c = !(f >= 0.0) ? 0 : (f >= (double)(g.nc[d] - 1) ? g.nc[d] - 1 : (int)f);
    return c;
}

// Place of the x-row of cells (cy, cz) in the sorted order: rows go tile by
// tile of 8 x 8, z within y tiles within z tiles, so that the rows an atom's
// search reads (two to each side) and the atoms next to it in y and z are
// close in the sorted order.  Plane after plane, the five planes of a search
// are 20 MB in a frame of 352^3 cells, five times an XCD's L2, and were
// fetched again for every plane; a tile and its margin are 1.6 MB.
__device__ inline int cell_row(const Grid &g, int cy, int cz) {
    const int ty = cy & ~7, tz = cz & ~7;
    const int wy = min(8, g.nc[1] - ty), wz = min(8, g.nc[2] - tz);
    return tz * g.nc[1] + ty * wz + (cz - tz) * wy + (cy - ty);
}

// the grid a kernel works on: one the host made, or the one on the device
// (read through the constant address space: the kernel before has written it,
// and scalar loads keep it out of the vector registers)
__device__ inline Grid grid_of(const GridArg &A) {
    Grid g = A.val;
    if (A.dev) {
        typedef const __attribute__((address_space(4))) uint32_t *Words;
        const Words w = (Words)(const uint32_t *)&A.dev->g;
        uint32_t v[sizeof(Grid) / 4];
        static_assert(sizeof(Grid) % 4 == 0, "the grid is read in words");
#pragma unroll
        for (int i = 0; i < (int)(sizeof(Grid) / 4); i++) v[i] = w[i];
        __builtin_memcpy(&g, v, sizeof(Grid));
    }
    return g;
}
__device__ inline int64_t cells_of(const GridArg &A, int64_t cells) { return A.dev ? A.dev->cells : cells; }

// ------------------------------------------------------------------ bounds
struct Bounds {
    double mn[3], mx[3];
    int bad;  // a coordinate that is not finite
};
__device__ inline void bounds_clear(Bounds &b) {
    for (int d = 0; d < 3; d++) {
        b.mn[d] = 1e308;
        b.mx[d] = -1e308;
    }
    b.bad = 0;
}
__device__ inline void bounds_add(Bounds &b, const double *__restrict__ pos, int64_t i) {
    for (int d = 0; d < 3; d++) {
        const double x = pos[3 * i + d];
        if (!isfinite(x)) b.bad = 1;
        b.mn[d] = fmin(b.mn[d], x);
        b.mx[d] = fmax(b.mx[d], x);
    }
}
// over the block (NW waves; ws: LDS); every lane of wave 0 gets the result
template <int NW>
__device__ inline void bounds_block(Bounds &b, Bounds *ws) {
    for (int off = 32; off > 0; off >>= 1) {
        for (int d = 0; d < 3; d++) {
            b.mn[d] = fmin(b.mn[d], __shfl_xor(b.mn[d], off));
            b.mx[d] = fmax(b.mx[d], __shfl_xor(b.mx[d], off));
        }
        b.bad |= __shfl_xor(b.bad, off);
    }
    if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = b;
    __syncthreads();
    if (threadIdx.x < 64) {
        b = ws[threadIdx.x & (NW - 1)];
        for (int off = NW / 2; off > 0; off >>= 1) {
            for (int d = 0; d < 3; d++) {
                b.mn[d] = fmin(b.mn[d], __shfl_xor(b.mn[d], off));
                b.mx[d] = fmax(b.mx[d], __shfl_xor(b.mx[d], off));
            }
            b.bad |= __shfl_xor(b.bad, off);
        }
    }
}

// Per-block min/max of each axis and a non-finite flag.
__global__ void __launch_bounds__(256) k_bounds(const double *__restrict__ pos, int64_t n, double *__restrict__ part) {
    __shared__ Bounds ws[4];
    Bounds b;
    bounds_clear(b);
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        bounds_add(b, pos, i);
    bounds_block<4>(b, ws);
    if (threadIdx.x == 0) {
        double *o = part + 7 * blockIdx.x;
        for (int d = 0; d < 3; d++) { o[d] = b.mn[d]; o[3 + d] = b.mx[d]; }
        o[6] = (double)b.bad;
    }
}

// the frame's grid from its bounds (one lane); a frame with a coordinate that
// is not finite, or whose grid has more cells than its arrays are laid out
// for, gets the flag, and every later kernel leaves it alone
__device__ inline void grid_finish(GridState *G, const Bounds &b, const double (&box)[3], int64_t n, int kn,
                                   int32_t *box_fail) {
    Grid g = make_grid(box, b.mn, b.mx, n, kn);
    const int flag = b.bad ? FRAME_NONFINITE : (grid_cells(g) > max_cells(n) ? FRAME_GRID : 0);
    if (flag) g.nc[0] = g.nc[1] = g.nc[2] = 1;  // (nothing reads it, but the scan's range comes from it)
    G->g = g;
    G->cells = grid_cells(g);
    int fast = 1;
    for (int a = 0; a < 3; a++)
        if (g.periodic[a] && g.nc[a] < 5) fast = 0;
    G->fast = fast;
    *box_fail = flag;
}

// Bounds, cleared cell counters and, by the last block to finish, the frame's
// own counters (after the cells) and the grid, in one launch: the host need
// not see the bounds before it launches the rest.  The partial results go
// through memory (the XCDs' L2s are not coherent) by stores that pass the L2
// and are waited for; a fence would write back the whole L2 in every block.
__global__ void __launch_bounds__(256) k_bounds_grid(const double *__restrict__ pos, int64_t n, double bx, double by,
                                                     double bz, int kn, int32_t *__restrict__ count, int64_t cells,
                                                     double *part, GridState *G, int32_t *box_fail) {
    __shared__ Bounds ws[4];
    __shared__ int last;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x, first = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    for (int64_t i = first; i < cells; i += stride) count[i] = 0;
    Bounds b;
    bounds_clear(b);
    for (int64_t i = first; i < n; i += stride) bounds_add(b, pos, i);
    bounds_block<4>(b, ws);
    if (threadIdx.x == 0) {
        double *o = part + 7 * blockIdx.x;
        for (int d = 0; d < 3; d++) {
            __hip_atomic_store(o + d, b.mn[d], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(o + 3 + d, b.mx[d], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __hip_atomic_store(o + 6, (double)b.bad, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the partial is in memory before the arrival counts
        last = __hip_atomic_fetch_add(&G->arrived, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (int)gridDim.x - 1;
    }
    __syncthreads();
    if (!last) return;
    if (threadIdx.x < FRAME_COUNTERS && threadIdx.x != 3) count[cells + threadIdx.x] = 0;  // (3: the flag, below)
    bounds_clear(b);
    for (int k = threadIdx.x; k < (int)gridDim.x; k += blockDim.x) {
        const double *o = part + 7 * k;
        for (int d = 0; d < 3; d++) {
            b.mn[d] = fmin(b.mn[d], __hip_atomic_load(o + d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            b.mx[d] = fmax(b.mx[d], __hip_atomic_load(o + 3 + d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        }
        b.bad |= __hip_atomic_load(o + 6, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0.0;
    }
    bounds_block<4>(b, ws);
    if (threadIdx.x == 0) {
        const double box[3] = {bx, by, bz};
        G->arrived = 0;  // for the next frame
        grid_finish(G, b, box, n, kn, box_fail);
    }
}

// ----------------------------------------------------------------- binning
__global__ void k_bin_count(const double *__restrict__ pos, int64_t n, GridArg A, int32_t *__restrict__ cell_of,
                            int32_t *__restrict__ slot_of, int32_t *__restrict__ count,
                            const int32_t *__restrict__ box_fail) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n || *box_fail) return;
    const Grid g = grid_of(A);
    int cx = cell_coord(pos[3 * i + 0], g, 0);
    int cy = cell_coord(pos[3 * i + 1], g, 1);
    int cz = cell_coord(pos[3 * i + 2], g, 2);
    int c = cell_row(g, cy, cz) * g.nc[0] + cx;
    cell_of[i] = c;
    slot_of[i] = atomicAdd(&count[c], 1);
}

// Cell starts: the exclusive scan of the counts over cells + 1 entries (the
// last start is the number of atoms), in items of SERVE_SCAN_CELLS cells --
// the items' totals, their exclusive scan, then each item's cells from its
// offset (three passes: every atomic count must be final before the first).
constexpr int SCAN_THREADS = 256;
constexpr int SCAN_PER = (int)(SERVE_SCAN_CELLS / SCAN_THREADS);  // cells per thread
static_assert(SERVE_SCAN_CELLS % SCAN_THREADS == 0 && SCAN_PER % 4 == 0, "an item is whole threads' 16-byte runs");

// exclusive scan over a block of NT threads (ws: NT / 64 words of LDS);
// total: the block's sum
template <int NT>
__device__ inline int32_t block_excl_scan(int32_t v, int32_t &total, int32_t *ws) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int32_t x = v;
    for (int d = 1; d < 64; d <<= 1) {
        const int32_t y = __shfl_up(x, d);
        if (lane >= d) x += y;
    }
    if (lane == 63) ws[w] = x;
    __syncthreads();
    int32_t before = 0, all = 0;
#pragma unroll
    for (int k = 0; k < NT / 64; k++) {
        const int32_t t = ws[k];
        before += k < w ? t : 0;
        all += t;
    }
    total = all;
    return before + x - v;
}

// item totals: 16-byte reads interleaved across the block, so they
// coalesce (count is 256-byte aligned and items are multiples of 4 cells)
__global__ void __launch_bounds__(SCAN_THREADS) k_scan_totals(const int32_t *__restrict__ count, int64_t cells, GridArg A,
                                                               int32_t *__restrict__ bsum) {
    __shared__ int32_t ws[SCAN_THREADS / 64];
    cells = cells_of(A, cells);
    if ((int64_t)blockIdx.x * SERVE_SCAN_CELLS > cells) return;
    const int64_t b = (int64_t)blockIdx.x * SERVE_SCAN_CELLS + 4 * (int64_t)threadIdx.x;
    int32_t s = 0;
#pragma unroll
    for (int k = 0; k < SCAN_PER / 4; k++) {
        const int64_t c = b + (int64_t)k * 4 * SCAN_THREADS;
        if (c + 4 <= cells) {
            const int4 x = *reinterpret_cast<const int4 *>(count + c);
            s += (x.x + x.y) + (x.z + x.w);
        } else {
            for (int j = 0; j < 4; j++) s += c + j < cells ? count[c + j] : 0;
        }
    }
    int32_t total;
    (void)block_excl_scan<SCAN_THREADS>(s, total, ws);
    if (threadIdx.x == 0) bsum[blockIdx.x] = total;
}

// exclusive scan of the item totals in place, one block
__global__ void __launch_bounds__(1024) k_scan_top(int32_t *__restrict__ bsum, int64_t items) {
    __shared__ int32_t ws[1024 / 64];
    const int64_t per = (items + 1023) / 1024;
    const int64_t lb = threadIdx.x * per, le = min(items, lb + per);
    int32_t s = 0;
    for (int64_t k = lb; k < le; k++) s += bsum[k];
    int32_t total;
    int32_t run = block_excl_scan<1024>(s, total, ws);
    for (int64_t k = lb; k < le; k++) {
        const int32_t v = bsum[k];
        bsum[k] = run;
        run += v;
    }
}

// Each item's cells: a run of SCAN_PER consecutive cells per thread.  Top:
// bsum holds the items' exclusive prefix (k_scan_top); otherwise the block
// adds up the totals of the items before its own, which for the item counts
// this is used for costs less than the launch.
template <bool Top>
__global__ void __launch_bounds__(SCAN_THREADS) k_scan_cells(const int32_t *__restrict__ count, int64_t cells,
                                                              GridArg A, const int32_t *__restrict__ bsum,
                                                              int32_t *__restrict__ start) {
    __shared__ int32_t ws[SCAN_THREADS / 64];
    cells = cells_of(A, cells);
    if ((int64_t)blockIdx.x * SERVE_SCAN_CELLS > cells) return;
    int32_t before = 0;
    if (Top) {
        before = bsum[blockIdx.x];
    } else {
        int32_t v = 0;
        for (int k = threadIdx.x; k < (int)blockIdx.x; k += SCAN_THREADS) v += bsum[k];
        (void)block_excl_scan<SCAN_THREADS>(v, before, ws);
        __syncthreads();  // ws is used again below
    }
    const int64_t b = (int64_t)blockIdx.x * SERVE_SCAN_CELLS + (int64_t)threadIdx.x * SCAN_PER;
    int32_t v[SCAN_PER], s = 0;
    if (b + SCAN_PER <= cells) {  // whole run in range: 16-byte reads (b is a multiple of 8)
        const int4 *q = reinterpret_cast<const int4 *>(count + b);
#pragma unroll
        for (int k = 0; k < SCAN_PER / 4; k++) {
            const int4 x = q[k];
            v[4 * k] = x.x;
            v[4 * k + 1] = x.y;
            v[4 * k + 2] = x.z;
            v[4 * k + 3] = x.w;
        }
    } else {
#pragma unroll
        for (int k = 0; k < SCAN_PER; k++) v[k] = b + k < cells ? count[b + k] : 0;
    }
#pragma unroll
    for (int k = 0; k < SCAN_PER; k++) s += v[k];
    int32_t total;
    int32_t run = before + block_excl_scan<SCAN_THREADS>(s, total, ws);
    int32_t o[SCAN_PER];
#pragma unroll
    for (int k = 0; k < SCAN_PER; k++) {
        o[k] = run;
        run += v[k];
    }
    if (b + SCAN_PER <= cells + 1) {
        int4 *q = reinterpret_cast<int4 *>(start + b);
#pragma unroll
        for (int k = 0; k < SCAN_PER / 4; k++) q[k] = make_int4(o[4 * k], o[4 * k + 1], o[4 * k + 2], o[4 * k + 3]);
    } else {
#pragma unroll
        for (int k = 0; k < SCAN_PER; k++)
            if (b + k <= cells) start[b + k] = o[k];
    }
}

__global__ void k_bin_scatter(const double *__restrict__ pos, int64_t n, GridArg A,
                              const int32_t *__restrict__ cell_of, const int32_t *__restrict__ slot_of,
                              const int32_t *__restrict__ start, double *__restrict__ spos, int4 *__restrict__ sfix,
                              int32_t *__restrict__ sid, const int32_t *__restrict__ box_fail) {
    int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n || *box_fail) return;
    const Grid g = grid_of(A);
    int64_t p = (int64_t)start[cell_of[i]] + slot_of[i];
    const double x = pos[3 * i + 0], y = pos[3 * i + 1], z = pos[3 * i + 2];
    spos[3 * (int64_t)p] = x;
    spos[3 * (int64_t)p + 1] = y;
    spos[3 * (int64_t)p + 2] = z;
    sfix[p] = make_int4(fixed_coord(x, g, 0), fixed_coord(y, g, 1), fixed_coord(z, g, 2), (int32_t)i);
    sid[p] = (int32_t)i;
}

// Bounds, grid and binning of a small frame in one launch of one block: the
// eight launches they take otherwise cost the host 4 to 8 us each, more than
// their work (500 atoms: 85 us from the first to the last, with the copy of
// the bounds to the host between them; this kernel 11 us).  One block's
// passes over the atoms grow with them: at 8,000 atoms the launches of
// k_bounds_grid and the rest are 15 us faster.
constexpr int SETUP_THREADS = 1024;
constexpr int SETUP_CELLS = 16384;  // counters in LDS up to this many cells
__global__ void __launch_bounds__(SETUP_THREADS) k_setup_small(const double *__restrict__ pos, int64_t n, double bx,
                                                               double by, double bz, int kn, GridState *G,
                                                               int32_t *__restrict__ count, int64_t cells_max,
                                                               int32_t *__restrict__ cell_of,
                                                               int32_t *__restrict__ slot_of,
                                                               int32_t *__restrict__ start, double *__restrict__ spos,
                                                               int4 *__restrict__ sfix, int32_t *__restrict__ sid,
                                                               int32_t *box_fail) {
    constexpr int NW = SETUP_THREADS / 64;
    __shared__ Bounds wb[NW];
    __shared__ int32_t ws[NW];
    __shared__ Grid sg;
    __shared__ int s_flag;
    __shared__ int32_t lds_count[SETUP_CELLS];
    const int t = threadIdx.x;
    // the frame's counters (after the cells, where the other path has them)
    if (t < FRAME_COUNTERS && t != 3) count[cells_max + t] = 0;  // (3: the flag, by grid_finish)
    Bounds b;
    bounds_clear(b);
    for (int64_t i = t; i < n; i += SETUP_THREADS) bounds_add(b, pos, i);
    bounds_block<NW>(b, wb);
    if (t == 0) {
        const double box[3] = {bx, by, bz};
        grid_finish(G, b, box, n, kn, box_fail);
        sg = G->g;
        s_flag = *box_fail;
    }
    __syncthreads();
    if (s_flag) return;
    const Grid g = sg;
    const int cells = g.nc[0] * g.nc[1] * g.nc[2];
    const bool in_lds = cells <= SETUP_CELLS;
    if (in_lds)
        for (int c = t; c < cells; c += SETUP_THREADS) lds_count[c] = 0;
    else
        for (int c = t; c < cells; c += SETUP_THREADS) count[c] = 0;
    __syncthreads();
    for (int64_t i = t; i < n; i += SETUP_THREADS) {
        const int cx = cell_coord(pos[3 * i + 0], g, 0), cy = cell_coord(pos[3 * i + 1], g, 1),
                  cz = cell_coord(pos[3 * i + 2], g, 2);
        const int c = cell_row(g, cy, cz) * g.nc[0] + cx;
        cell_of[i] = c;
        slot_of[i] = in_lds ? atomicAdd(&lds_count[c], 1) : atomicAdd(&count[c], 1);
    }
    __syncthreads();
    // exclusive scan, a run of cells per thread
    const int per = (cells + SETUP_THREADS - 1) / SETUP_THREADS;
    const int c0 = min(t * per, cells), c1 = min(c0 + per, cells);
    int32_t sum = 0, total;
    for (int c = c0; c < c1; c++) sum += in_lds ? lds_count[c] : count[c];
    int32_t run = block_excl_scan<SETUP_THREADS>(sum, total, ws);
    for (int c = c0; c < c1; c++) {
        start[c] = run;
        const int32_t k = in_lds ? lds_count[c] : count[c];
        if (in_lds) lds_count[c] = run;
        run += k;
    }
    if (t == 0) start[cells] = total;
    __syncthreads();
    for (int64_t i = t; i < n; i += SETUP_THREADS) {
        const int c = cell_of[i];
        const int64_t p = (int64_t)(in_lds ? lds_count[c] : start[c]) + slot_of[i];
        const double x = pos[3 * i + 0], y = pos[3 * i + 1], z = pos[3 * i + 2];
        spos[3 * p] = x;
        spos[3 * p + 1] = y;
        spos[3 * p + 2] = z;
        sfix[p] = make_int4(fixed_coord(x, g, 0), fixed_coord(y, g, 1), fixed_coord(z, g, 2), (int32_t)i);
        sid[p] = (int32_t)i;
    }
}

// ---------------------------------------------------------------- k-NN
// Minimum-image difference exactly as specified: s = rint(d * (1/L)),
// d - s*L, without contraction (the library is built with
// -ffp-contract=off), so d^2 matches the reference bit for bit.
__device__ inline double min_image(double d, const Grid &g, int a) {
    if (g.periodic[a]) {
        double s = rint(d * g.invL[a]);
        d = d - s * g.L[a];
    }
    return d;
}

// offsets of the cells up to s away from cell c on axis a (none twice, none
// outside an open axis, so a block never has more rows than the grid)
__device__ inline void shell_range(const Grid &g, int a, int c, int s, int &lo, int &hi) {
    const int half = g.periodic[a] ? (g.nc[a] - 1) / 2 : c;
    lo = -min(s, half);
    hi = min(s, g.nc[a] - 1 - half);
}

// Radius around the atom that the block of cells with offsets [lo, hi] per
// axis covers, less the margin (<= 0 if none; +inf, and all, when the block
// holds every cell): an atom outside the block is at least that far away, so
// K atoms strictly closer are a certificate that the block holds the K
// nearest.
__device__ inline double block_reach(const Grid &g, const int (&cc)[3], const double (&u)[3], const int (&lo)[3],
                                     const int (&hi)[3], bool &all) {
    double dmin = INFINITY;
    all = true;
    for (int a = 0; a < 3; a++) {
        bool sat_lo, sat_hi;
        if (g.periodic[a]) {
            sat_lo = sat_hi = (hi[a] - lo[a] + 1) >= g.nc[a];
        } else {
            sat_lo = cc[a] + lo[a] <= 0;
            sat_hi = cc[a] + hi[a] >= g.nc[a] - 1;
        }
        if (!sat_lo) dmin = fmin(dmin, u[a] - (cc[a] + lo[a]) * g.h[a]);
        if (!sat_hi) dmin = fmin(dmin, (cc[a] + hi[a] + 1) * g.h[a] - u[a]);
        all = all && sat_lo && sat_hi;
    }
    return dmin - g.margin;
}

// Sec. 5 samples are periodic.  Every image of an atom other than its
// minimum image lies at least half a box length away along that axis, so
// the minimum-image shell is the periodic crystal's shell only when its
// K-th member is strictly closer than half of every periodic length
// (compared as 4 d^2 < L*L in FP64); a periodic frame whose atom has fewer
// than K neighbours fails as well.  True = the frame is rejected.
__device__ inline bool shell_exceeds_box(const Grid &g, int cnt, int K, double kth) {
    bool periodic = false, bad = false;
    for (int a = 0; a < 3; a++)
        if (g.periodic[a]) {
            periodic = true;
            bad = bad || !(4.0 * kth < g.L[a] * g.L[a]);
        }
    return periodic && (cnt < K || bad);
}

// LDS written by some lanes of a wave and then read by others of the same
// wave: a wave's LDS instructions complete in issue order, so the only
// requirement is that the compiler keeps them on their side of this point.
__device__ inline void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Workgroups are dispatched to the 8 XCDs round-robin, and each XCD has its
// own L2.  With a grid padded to a multiple of 8, this bijection gives every
// XCD one contiguous range of blocks, so that blocks sharing cells (and
// their atoms) run behind the same L2.
constexpr int NXCD = 8;
__device__ inline int64_t xcd_block(int64_t i, int64_t nblocks_padded) {
    const int64_t per = nblocks_padded / NXCD;
    return (i % NXCD) * per + i / NXCD;
}
inline int64_t xcd_pad(int64_t nblocks) { return (nblocks + NXCD - 1) / NXCD * NXCD; }

// Fast search, one lane per atom: the 5x5x5 block of cells around it, as 25
// x-rows nearest-first (a row of cells is one contiguous range of the sorted
// atoms, two if it wraps).
//
// What bounds it: vector issue (0.74 of the slots on a 0.92 M-atom frame) and
// the latency of its loads, more so in frames beyond the caches (0.61 of the
// slots at 31.7 M atoms).  Candidates are read as 16-byte records of fixed-point
// coordinates, whose 32-bit differences are minimum images without any shift
// and which are converted to FP32 (half the cost of an FP64 operation); FP64
// positions are read for the neighbours found only, where 24-byte FP64
// records of every candidate had to come before.  31.7 M atoms: 13.4 ms with
// FP64 records, 64-bit keys and rows plane after plane; 12.2 with this search;
// 10.3 with it and the tiled order of rows (cell_row).  0.92 M atoms: 345 ->
// 285 us.  (Both less by 2 to 4 % with the tables below.)
//
// A candidate is ranked by one 32-bit key: the upper 21 bits are d^2 on a
// linear grid (buckets of 1 / (2^21 - 16) of the squared radius the block
// certifies, farther atoms in the last bucket), the lower 11 name the
// candidate (range of atoms, offset in it).  The list keeps the 19 smallest
// keys: inserting t into a sorted list is a[m] = median(a[m - 1], a[m], t),
// one independent instruction per entry, where the pair (min, max) on 64-bit
// keys that it replaces took two dependent ones per entry, on two registers
// each.
//
// The ranges come first, in a loop over rows that is uniform over the wave
// (their offsets are scalars): nine inner rows, their atoms, then the sixteen
// outer rows and the cells that the Kth distance found so far leaves, and
// their atoms.  Each lane then walks its own table of ranges, kept in LDS, two
// atoms per step, so that a wave pays about the per-lane atom count.  A range
// of more than 64 atoms takes several entries, and where a lane's table is
// full the wave searches what it holds, the lane frees every entry that the
// list does not name (12 at least), and the rows go on: any number of atoms
// fits.  Where the own row is dense (KNN_DENSE_ROW) the Kth distance is taken
// after one, five and nine rows, which spares most of the block.
//
// The cells follow the mean density, so a particle in a box of 2.5 diameters
// has 400 atoms in a 5 x 5 x 1 slice of its block.  With one table for the
// whole search such atoms were left to the exact search, a wave each: 100,000
// atoms in such a box 4.14 ms, 0.35 with this loop (0.60 with the search on
// FP64 records); 1,000,000 atoms 39.2 ms, 1.61 (2.43).  At the mean density
// the atoms at the x edges of the box, whose rows are two ranges, fit as well:
// k-NN at 0.92 M atoms 372 -> 304 us, at 31.7 M 10.54 -> 9.90 ms (with the
// exact order's loads below).
//
// Two atoms whose buckets differ by `apart` or more are in the exact order
// (the rounding of the coordinates, of d^2 and of the buckets is covered).
// Where neighbouring entries are closer, the exact (d^2, id) of the entries
// decides; that covers exact ties inside the list too (the 12 + 6 neighbours
// of a perfect FCC or HCP crystal end at entry 18).  The atoms left to
// k_knn_exact are those whose Kth neighbour the block does not certify or
// whose ties run past the list.  Requires
// every periodic axis to have at least 5 cells (no axis wraps onto itself
// within the block).
constexpr int KNN_LIST = 19;    // list entries (both neighbour counts)
constexpr int KNN_RANGES = 31;  // ranges held at a time, for the decoding (a 5-bit code)
constexpr int KNN_OFF_BITS = 6; // offset within a range
constexpr int KNN_CODE_BITS = 11;
constexpr uint32_t KNN_BUCKETS = (1u << (32 - KNN_CODE_BITS)) - 16;
static_assert(KNN_RANGES << KNN_OFF_BITS < 1 << KNN_CODE_BITS, "range and offset fit the code; the last means none");
static_assert(KNN_LIST < KNN_RANGES && KNN_RANGES < 32, "the list names fewer entries than there are; 31 means none");
// atoms in the five cells of the own row from which the rows are taken in
// smaller steps (3.6 at the mean density)
constexpr int KNN_DENSE_ROW = 24;

// W lanes: 155 bytes each (39,680 per block of 256: four blocks per CU)
template <int W>
struct KnnRanges {
    uint32_t q0[KNN_RANGES][W];  // first atom
    uint8_t cnt[KNN_RANGES][W];  // atoms
};

// the coordinates of sorted atom q's record (12 bytes: the id, unused, would
// hold a register that the load in flight forbids to reuse)
typedef int32_t int3v __attribute__((ext_vector_type(3)));
__device__ inline int3v fixed_xyz(const int4 *__restrict__ sfix, int64_t q) {
    return *reinterpret_cast<const int3v *>(sfix + q);
}

__device__ inline uint32_t med3_u32(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t r;
    asm("v_med3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// NK = 14 neighbours (Euclidean ordering), or 18 (the input of the
// topological ordering).  One atom (lane t of the W in S); false: left to the
// exact search, nothing written.
template <int NK, int W>
__device__ inline bool knn_fast_atom(KnnRanges<W> &S, int t, int64_t p, int64_t n, const Grid &g,
                                     const double *__restrict__ spos, const int4 *__restrict__ sfix,
                                     const int32_t *__restrict__ start, int32_t *__restrict__ nbr_id,
                                     double *__restrict__ nbr_rel, int32_t *__restrict__ box_fail) {
    const double xi = spos[3 * (int64_t)p], yi = spos[3 * (int64_t)p + 1], zi = spos[3 * (int64_t)p + 2];
    const double xs[3] = {xi, yi, zi};
    const int4 own = sfix[p];
    int cc[3];
    double u[3];
    for (int a = 0; a < 3; a++) {
        cc[a] = cell_coord(xs[a], g, a);
        u[a] = wrapped(xs[a], g, a);
    }
    // squared radius within which the block is complete (bounded by the
    // block's own extent when it holds every cell), and the bucket width
    double rcap2;
    {
        const int lo[3] = {-2, -2, -2}, hi[3] = {2, 2, 2};
        bool all;
        const double reach = block_reach(g, cc, u, lo, hi, all);
        const double ext2 = 9.0 * ((g.h[0] * g.h[0] + g.h[1] * g.h[1]) + g.h[2] * g.h[2]) * 1.001;
        if (!(reach > 0)) return false;
        rcap2 = all ? ext2 : fmin(reach * reach, ext2);
        if (!(rcap2 > 1e-30 && rcap2 < 1e30)) return false;  // (beyond what FP32 resolves)
    }
    const double bucket = rcap2 / (double)KNN_BUCKETS;
    // A bucket is off by the coordinates' rounding (fix_err in a difference
    // vector, 2 r fix_err in d^2 = r^2 <= rcap2) and by FP32 (conversion,
    // factor and product of each difference, twice in its square, then three
    // roundings: 9 2^-24 of at most 2^21 buckets).  apart = one more than
    // twice that, rounded up.
    const double err = 2.1 * sqrt(rcap2) * g.fix_err / bucket + 1.15;
    if (!(err < 256.0)) return false;  // coordinates so far from the box that FP64 is too coarse
    const int apart = 2 + (int)(2.0 * err);
    // per-axis steps in units of a bucket's square root
    const double root = 1.0 / sqrt(bucket);
    const float wx = (float)(root / g.fix[0]), wy = (float)(root / g.fix[1]), wz = (float)(root / g.fix[2]);
    // offset within the own cell, and the squared gaps to the cells at -2, -1,
    // +1, +2 of x (less the margin and, in FP32, 4e-6 cells)
    float f[3], h[3], slack[3];
    for (int a = 0; a < 3; a++) {
        f[a] = (float)(u[a] - cc[a] * g.h[a]);
        h[a] = (float)g.h[a];
        slack[a] = (float)g.margin + 4e-6f * h[a];
    }
    auto sqgap = [&](int a, float e) {
        e = fmaxf(e - slack[a], 0.0f);
        return e * e;
    };
    const float gx_m2 = sqgap(0, f[0] + h[0]), gx_m1 = sqgap(0, f[0]);
    const float gx_p1 = sqgap(0, h[0] - f[0]), gx_p2 = sqgap(0, 2.0f * h[0] - f[0]);
    const int nx = g.nc[0];

    uint32_t key[KNN_LIST];
#pragma unroll
    for (int m = 0; m < KNN_LIST; m++) key[m] = ~0u;
    uint32_t unused = (1u << KNN_RANGES) - 1;  // entries of the table that are free
    float cap = (float)rcap2 * 1.000001f;  // squared radius still to search
    uint32_t r0 = 0, r1 = 0, w0 = 0, w1 = 0;  // what is left of the row: its part here, its part across the box edge
    // (dy + 2) + 5 (dz + 2) of the 25 rows by increasing dy^2 + dz^2, 5 bits each
    const uint64_t rows_lo = 0x013952440D13B56Cull;  // rows 0..11
    const uint64_t rows_hi = 0x0250171D4334BCB6ull;  // rows 12..23
    int row = 0, stage = 9;  // the same in every lane: the next row, the row at which this stage ends
    bool more_rows = true;
    do {
        uint32_t pending = unused;  // entries to search: those that are taken below
        for (;;) {
            // one range of the row per turn
            if (r0 < r1 && unused) {
                const uint32_t cnt = min(r1 - r0, 1u << KNN_OFF_BITS);
                const int e = __builtin_ctz(unused);
                S.q0[e][t] = r0;
                S.cnt[e][t] = (uint8_t)cnt;
                unused &= unused - 1;
                r0 += cnt;
                if (r0 == r1) {
                    r0 = w0;
                    r1 = w1;
                    w0 = w1;
                }
            }
            if (__ballot(r0 < r1)) {
                if (__ballot(r0 < r1 && !unused)) break;
                continue;
            }
            if (row == stage) break;
            const int code = row < 12 ? (int)((rows_lo >> (5 * row)) & 31)
                                      : (row < 24 ? (int)((rows_hi >> (5 * (row - 12))) & 31) : 24);
            const int dz = code / 5 - 2, dy = code - 5 * (code / 5) - 2;
            row++;
            int cy = cc[1] + dy, cz = cc[2] + dz;
            const bool out = (!g.periodic[1] && (cy < 0 || cy >= g.nc[1])) ||
                             (!g.periodic[2] && (cz < 0 || cz >= g.nc[2]));
            cy = cy < 0 ? cy + g.nc[1] : (cy >= g.nc[1] ? cy - g.nc[1] : cy);
            cz = cz < 0 ? cz + g.nc[2] : (cz >= g.nc[2] ? cz - g.nc[2] : cz);
            const float gy2 = dy == 0 ? 0.0f : sqgap(1, dy > 0 ? (float)dy * h[1] - f[1] : f[1] - (float)(dy + 1) * h[1]);
            const float gz2 = dz == 0 ? 0.0f : sqgap(2, dz > 0 ? (float)dz * h[2] - f[2] : f[2] - (float)(dz + 1) * h[2]);
            const float rem = cap - (gy2 + gz2);
            if (!out && rem >= 0) {
                // cells whose x-gap exceeds what is left cannot hold a better neighbour
                const int a0 = cc[0] - (gx_m1 <= rem) - (gx_m2 <= rem), a1 = cc[0] + (gx_p1 <= rem) + (gx_p2 <= rem);
                const int cyz = cell_row(g, cy, cz) * nx;
                r0 = (uint32_t)start[cyz + max(a0, 0)];
                r1 = (uint32_t)start[cyz + min(a1, nx - 1) + 1];
                if (g.periodic[0] && (a0 < 0 || a1 >= nx)) {  // the part across the box edge
                    w0 = (uint32_t)start[cyz + (a0 < 0 ? a0 + nx : 0)];
                    w1 = (uint32_t)start[cyz + (a0 < 0 ? nx : a1 - nx + 1)];
                    if (r0 == r1) {
                        r0 = w0;
                        r1 = w1;
                        w0 = w1;
                    }
                }
            }
            if (row == 1 && __ballot((int)(r1 - r0) + (int)(w1 - w0) >= KNN_DENSE_ROW)) stage = 1;
        }
        pending &= ~unused;
        // the atoms of the ranges, two per step; the next step's are loaded
        // before this one's are used
        int q = 0, qend = 0;
        uint32_t code = 0;  // code of atom q less q
        auto fetch = [&](int3v &A, int3v &B, uint32_t &ca, uint32_t &cb) {
            const bool any = q < qend || pending;
            if (q >= qend && pending) {
                const int e = __builtin_ctz(pending);
                pending &= pending - 1;
                q = (int)S.q0[e][t];
                qend = q + (int)S.cnt[e][t];
                code = ((uint32_t)e << KNN_OFF_BITS) - (uint32_t)q;
            }
            // loads without a branch (the atom itself where there is none),
            // so that they can stay in flight
            const bool one = q < qend, two = q + 1 < qend;
            const int qa = one ? q : (int)p, qb = two ? q + 1 : (int)p;
            A = fixed_xyz(sfix, qa);
            B = fixed_xyz(sfix, qb);
            ca = qa == (int)p ? ~0u : code + (uint32_t)qa;
            cb = qb == (int)p ? ~0u : code + (uint32_t)qb;
            q += 2;
            return any;
        };
        auto rank = [&](const int3v &A, const int3v &B, uint32_t ca, uint32_t cb) {
            const float dx = (float)(int32_t)((uint32_t)A.x - (uint32_t)own.x) * wx;
            const float dy = (float)(int32_t)((uint32_t)A.y - (uint32_t)own.y) * wy;
            const float dz = (float)(int32_t)((uint32_t)A.z - (uint32_t)own.z) * wz;
            const float ex = (float)(int32_t)((uint32_t)B.x - (uint32_t)own.x) * wx;
            const float ey = (float)(int32_t)((uint32_t)B.y - (uint32_t)own.y) * wy;
            const float ez = (float)(int32_t)((uint32_t)B.z - (uint32_t)own.z) * wz;
            const float d2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx)), e2 = fmaf(ez, ez, fmaf(ey, ey, ex * ex));
            const uint32_t b1 = (uint32_t)fminf(d2, (float)(KNN_BUCKETS + 8));
            const uint32_t b2 = (uint32_t)fminf(e2, (float)(KNN_BUCKETS + 8));
            const uint32_t t1 = ca == ~0u ? ~0u : (b1 << KNN_CODE_BITS) + ca;
            const uint32_t t2 = cb == ~0u ? ~0u : (b2 << KNN_CODE_BITS) + cb;
#pragma unroll
            for (int m = KNN_LIST - 1; m > 0; m--) key[m] = med3_u32(key[m - 1], key[m], t1);
            key[0] = min(key[0], t1);
#pragma unroll
            for (int m = KNN_LIST - 1; m > 0; m--) key[m] = med3_u32(key[m - 1], key[m], t2);
            key[0] = min(key[0], t2);
        };
        // two steps per turn, each step's loads issued before the step
        // before it is ranked (the barriers keep the compiler from moving
        // them down to their use)
        int3v A0, B0, A1, B1;
        uint32_t ca0, cb0, ca1, cb1;
        bool more = fetch(A0, B0, ca0, cb0);
        while (more) {
            more = fetch(A1, B1, ca1, cb1);
            __builtin_amdgcn_sched_barrier(0);
            rank(A0, B0, ca0, cb0);
            if (!more) break;
            more = fetch(A0, B0, ca0, cb0);
            __builtin_amdgcn_sched_barrier(0);
            rank(A1, B1, ca1, cb1);
        }
        // an upper bound of the Kth distance found so far
        cap = fminf(cap, (float)((key[NK - 1] >> KNN_CODE_BITS) + (uint32_t)apart) * ((float)bucket * 1.000001f));
        if (r0 < r1) {
            // the table is full: the entries that the list names stay (an empty
            // place of the list names one past the last)
            uint32_t named = 0;
#pragma unroll
            for (int m = 0; m < KNN_LIST; m++) named |= 1u << (key[m] >> KNN_OFF_BITS & 31);
            unused = ~named & ((1u << KNN_RANGES) - 1);
        }
        more_rows = __ballot(r0 < r1) != 0;
        if (!more_rows && row == stage) {
            more_rows = stage < 25;
            stage = stage == 1 ? 5 : (stage == 5 ? 9 : 25);
        }
    } while (more_rows);

    auto bk = [&](int m) { return (int)(key[m] >> KNN_CODE_BITS); };
    // entries to put in order: past NK as long as the next one could come before the last
    int cnt = NK;
#pragma unroll
    for (int m = NK; m < KNN_LIST; m++)
        if (cnt == m && bk(m) - bk(m - 1) < apart) cnt = m + 1;
    bool close = cnt > NK;
#pragma unroll
    for (int m = 1; m < NK; m++) close = close || bk(m) - bk(m - 1) < apart;
    int last = bk(NK - 1);  // bucket of the last entry that matters
#pragma unroll
    for (int m = NK; m < KNN_LIST; m++) last = m < cnt ? bk(m) : last;
    if (cnt == KNN_LIST || last + apart >= (int)KNN_BUCKETS) return false;

    int32_t kq[KNN_LIST];
#pragma unroll
    for (int m = 0; m < KNN_LIST; m++) {
        const uint32_t code = key[m] & ((1u << KNN_CODE_BITS) - 1);
        kq[m] = m < cnt ? (int32_t)(S.q0[code >> KNN_OFF_BITS][t] + (code & ((1u << KNN_OFF_BITS) - 1))) : 0;
    }
    if (close) {
        // exact (d^2, id) order of the first cnt entries: odd-even exchanges
        // until none is left to make
        double ed[KNN_LIST];
        int32_t ej[KNN_LIST];
        // (four entries' loads in flight at a time, which the registers hold;
        // entries past cnt read atom 0.  One after the other, 116 bytes a lane
        // were spilled and a frame without noise waited for each: 78 -> 73 us at
        // 100 k atoms, 271 -> 251 us at 0.92 M)
        constexpr int GROUP = 4;
#pragma unroll
        for (int m0 = 0; m0 < KNN_LIST; m0 += GROUP) {
            double v[GROUP][3];
            int32_t id[GROUP];
#pragma unroll
            for (int k = 0; k < GROUP; k++)
                if (m0 + k < KNN_LIST) {
                    const int64_t q = kq[m0 + k];
                    for (int d = 0; d < 3; d++) v[k][d] = spos[3 * q + d];
                    id[k] = sfix[q].w;
                }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < GROUP; k++)
                if (m0 + k < KNN_LIST) {
                    const int m = m0 + k;
                    const double dx = min_image(v[k][0] - xi, g, 0), dy = min_image(v[k][1] - yi, g, 1);
                    const double dz = min_image(v[k][2] - zi, g, 2);
                    ed[m] = m < cnt ? (dx * dx + dy * dy) + dz * dz : INFINITY;
                    ej[m] = m < cnt ? id[k] : 0x7fffffff;
                }
        }
        bool moved;
        do {
            moved = false;
#pragma unroll
            for (int o = 1; o >= 0; o--)
#pragma unroll
                for (int m = o; m + 1 < KNN_LIST; m += 2) {
                    const bool sw = ed[m + 1] < ed[m] || (ed[m + 1] == ed[m] && ej[m + 1] < ej[m]);
                    const double td = ed[m];
                    const int32_t tj = ej[m], tq = kq[m];
                    ed[m] = sw ? ed[m + 1] : td;
                    ej[m] = sw ? ej[m + 1] : tj;
                    kq[m] = sw ? kq[m + 1] : tq;
                    ed[m + 1] = sw ? td : ed[m + 1];
                    ej[m + 1] = sw ? tj : ej[m + 1];
                    kq[m + 1] = sw ? tq : kq[m + 1];
                    moved = moved || sw;
                }
        } while (moved);
    }
    // the exact Kth distance only where its upper bound does not pass the box check
    if (shell_exceeds_box(g, NK, NK, (double)(bk(NK - 1) + apart) * bucket)) {
        const int64_t qk = kq[NK - 1];
        const double ex = min_image(spos[3 * qk] - xi, g, 0);
        const double ey = min_image(spos[3 * qk + 1] - yi, g, 1);
        const double ez = min_image(spos[3 * qk + 2] - zi, g, 2);
        if (shell_exceeds_box(g, NK, NK, (ex * ex + ey * ey) + ez * ez)) atomicOr(box_fail, 1);
    }
    // Ids and minimum-image vectors in the component-major layout the hull
    // kernels read (spos[3q .. 3q+2] is a copy of the input's position, so the
    // vectors are those of the input).  With every periodic coordinate in [0,
    // L) and at least 7 cells per axis, atoms of a block that does not wrap
    // lie less than half a box length apart and need no shift.
    bool plain = g.canonical != 0;
    for (int a = 0; a < 3; a++)
        plain = plain && (!g.periodic[a] || (g.nc[a] >= 7 && cc[a] >= 2 && cc[a] + 2 < g.nc[a]));
    const bool shifts = __ballot(!plain) != 0;
#pragma unroll
    for (int m = 0; m < NK; m++) {
        const int64_t q = kq[m];
        double dx = spos[3 * q] - xi, dy = spos[3 * q + 1] - yi, dz = spos[3 * q + 2] - zi;
        if (shifts) {
            dx = min_image(dx, g, 0);
            dy = min_image(dy, g, 1);
            dz = min_image(dz, g, 2);
        }
        nbr_id[(int64_t)m * n + p] = sfix[q].w;
        nbr_rel[((int64_t)m * 3 + 0) * n + p] = dx;
        nbr_rel[((int64_t)m * 3 + 1) * n + p] = dy;
        nbr_rel[((int64_t)m * 3 + 2) * n + p] = dz;
    }
    return true;
}

template <int NK>
__global__ void __launch_bounds__(256, 4) k_knn_fast(int64_t n, GridArg A, const double *__restrict__ spos,
                                                  const int4 *__restrict__ sfix, const int32_t *__restrict__ start,
                                                  int32_t *__restrict__ nbr_id, double *__restrict__ nbr_rel,
                                                  int32_t *__restrict__ todo, int32_t *__restrict__ todo_count,
                                                  int32_t *__restrict__ box_fail) {
    __shared__ KnnRanges<256> S;
    int64_t p = xcd_block(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    if (p >= n || *box_fail > FRAME_BOX || (A.dev && !A.dev->fast)) return;
    const Grid g = grid_of(A);
    if (!knn_fast_atom<NK, 256>(S, (int)threadIdx.x, p, n, g, spos, sfix, start, nbr_id, nbr_rel, box_fail))
        todo[atomicAdd(todo_count, 1)] = (int32_t)p;
}

// Exact search for the atoms the fast search left (or all atoms when todo
// is NULL), one wavefront per atom.  Shells of cells are added until the
// atoms strictly closer than the block's certified radius are K or more: only
// those can be among the K nearest.  A lane takes a row of cells, an
// exclusive scan of the rows' atom counts numbers the block's atoms, and each
// lane then finds its atoms' rows by bisection, so that all positions of the
// block are in flight at once.  The atoms within the radius go to a list in
// LDS; when it fills up it is cut to the K best, whose last then bounds the
// rest.  An atom's place in the order is the number of list entries before it
// by (d^2, id).  (Private sorted lists per lane merged by K rounds of
// wave-wide minima took 207 us where this takes 86 on the 0.92 M-atom
// polycrystal.)
//
// A first block that holds far more atoms than at the mean density (90, or 116
// for 18 neighbours) fills the list many times over, so the radius is first the
// one that holds three times the neighbours at the block's density (K atoms
// within it are the same certificate), and where the 3x3x3 block should reach
// that far it is enough.  The smallest frames take this search alone, and a
// particle in a vacuum fills its cells: whole frames of 16,000 atoms in a
// periodic box of 1.5, 2.5 and 6 diameters 483, 800 and 1919 -> 260, 263 and
// 476 us.
constexpr int KNN_CAND = 256;  // list entries
constexpr int KNN_FULL_BLOCK = 256;  // atoms
constexpr int64_t KNN_WAVE_ATOMS = 16384;  // frames up to this take the wave-per-atom search alone
struct KnnWave {
    double d2[KNN_CAND];
    int32_t id[KNN_CAND], q[KNN_CAND];
    int32_t pre[64], qa[64], la[64], qb[64];
};

// sorts the first count entries of the list's K best to its front (whole
// wave); returns the entries left
template <int K>
__device__ inline int knn_cut(KnnWave &S, int count) {
    const int lane = threadIdx.x & 63;
    double d[KNN_CAND / 64];
    int32_t j[KNN_CAND / 64], q[KNN_CAND / 64], rank[KNN_CAND / 64];
    wave_lds_sync();
#pragma unroll
    for (int b = 0; b < KNN_CAND / 64; b++) {
        rank[b] = K;
        const int e = 64 * b + lane;
        if (64 * b >= count) continue;
        d[b] = e < count ? S.d2[e] : INFINITY;
        j[b] = e < count ? S.id[e] : 0x7fffffff;
        q[b] = e < count ? S.q[e] : 0;
        int before = 0;
        for (int c = 0; c < count; c++) {
            const double dc = S.d2[c];
            before += dc < d[b] || (dc == d[b] && S.id[c] < j[b]);
        }
        rank[b] = e < count ? before : K;
    }
    wave_lds_sync();
#pragma unroll
    for (int b = 0; b < KNN_CAND / 64; b++)
        if (rank[b] < K) {
            S.d2[rank[b]] = d[b];
            S.id[rank[b]] = j[b];
            S.q[rank[b]] = q[b];
        }
    wave_lds_sync();
    return min(count, K);
}

// One atom p (wave-uniform) by the whole wave.
template <int NK>
__device__ void knn_exact_atom(KnnWave &S, int64_t p, int64_t n, const Grid &g, const double *__restrict__ spos,
                               const int32_t *__restrict__ sid, const int32_t *__restrict__ start,
                               int32_t *__restrict__ nbr_id, double *__restrict__ nbr_rel,
                               int32_t *__restrict__ box_fail) {
    const int lane = threadIdx.x & 63;
    const double xi = spos[3 * (int64_t)p], yi = spos[3 * (int64_t)p + 1], zi = spos[3 * (int64_t)p + 2];
    const double xs[3] = {xi, yi, zi};
    const int nx = g.nc[0];
    int cc[3];
    double u[3];
    for (int a = 0; a < 3; a++) {
        cc[a] = cell_coord(xs[a], g, a);
        u[a] = wrapped(xs[a], g, a);
    }
    int count = 0;
    // (blocks grow by a cell, later by a quarter: an atom a hundred thousand
    // empty cells from the others takes some fifty of them)
    bool guess = false, guessed = false;  // (of the wave)
    for (int s = 2;;) {
        int lo[3], hi[3], next = s + 1 + (s < 6 ? 0 : s / 4);
        for (int a = 0; a < 3; a++) shell_range(g, a, cc[a], s, lo[a], hi[a]);
        bool all;
        const double reach = block_reach(g, cc, u, lo, hi, all);
        // kept: d^2 < thr, or d^2 <= thr once the list was cut
        double thr = all ? INFINITY : (reach > 0 ? reach * reach : 0.0);
        bool cut = all;
        count = 0;
        const int ey = hi[1] - lo[1] + 1, rows = ey * (hi[2] - lo[2] + 1);
        for (int r0 = 0; r0 < rows; r0 += 64) {
            int qa = 0, la = 0, qb = 0, lb = 0;
            const int r = r0 + lane;
            if (r < rows) {
                int cy = cc[1] + lo[1] + r % ey, cz = cc[2] + lo[2] + r / ey;
                cy = cy < 0 ? cy + g.nc[1] : (cy >= g.nc[1] ? cy - g.nc[1] : cy);
                cz = cz < 0 ? cz + g.nc[2] : (cz >= g.nc[2] ? cz - g.nc[2] : cz);
                const int cyz = cell_row(g, cy, cz) * nx;
                const int a0 = cc[0] + lo[0], a1 = cc[0] + hi[0];
                const int i0 = max(a0, 0), i1 = min(a1, nx - 1);
                qa = start[cyz + i0];
                la = start[cyz + i1 + 1] - qa;
                if (a0 < 0 || a1 >= nx) {  // (a periodic axis)
                    const int w0 = a0 < 0 ? a0 + nx : 0, w1 = a0 < 0 ? nx - 1 : a1 - nx;
                    qb = start[cyz + w0];
                    lb = start[cyz + w1 + 1] - qb;
                }
            }
            int incl = la + lb;
            for (int d = 1; d < 64; d <<= 1) {
                const int y = __shfl_up(incl, d);
                if (lane >= d) incl += y;
            }
            const int total = __builtin_amdgcn_readlane(incl, 63);
            if (s == 2 && !guessed && total > KNN_FULL_BLOCK) {
                guess = guessed = true;
                if (total > 2 * KNN_FULL_BLOCK) {
                    next = 1;
                    break;
                }
            }
            if (guess) {
                // the volume of 3 K atoms, in cells, to the power 2/3 (any radius is
                // right, so FP32 will do)
                const float vol = (float)((hi[0] - lo[0] + 1) * rows * (3 * NK)) / (4.19f * (float)max(total, 1));
                const double h = fmin(fmin(g.h[0], g.h[1]), g.h[2]);
                thr = fmin(thr, h * h * (double)__builtin_amdgcn_exp2f(__builtin_amdgcn_logf(vol) * (2.0f / 3.0f)));
            }
            S.pre[lane] = incl - (la + lb);
            S.qa[lane] = qa;
            S.la[lane] = la;
            S.qb[lane] = qb;
            wave_lds_sync();
            for (int b = 0; b < total; b += 64) {
                const int i = b + lane;
                bool keep = false;
                double d2 = 0;
                int32_t q = 0;
                if (i < total) {
                    // the last row whose first atom is not past i (rows
                    // without atoms share their number with the next)
                    int row = 0;
#pragma unroll
                    for (int w = 32; w > 0; w >>= 1)
                        if (S.pre[row + w] <= i) row += w;
                    const int o = i - S.pre[row], l = S.la[row];
                    q = o < l ? S.qa[row] + o : S.qb[row] + (o - l);
                    const double dx = min_image(spos[3 * (int64_t)q] - xi, g, 0);
                    const double dy = min_image(spos[3 * (int64_t)q + 1] - yi, g, 1);
                    const double dz = min_image(spos[3 * (int64_t)q + 2] - zi, g, 2);
                    d2 = (dx * dx + dy * dy) + dz * dz;
                    keep = q != (int32_t)p && (d2 < thr || (cut && d2 == thr));
                }
                const uint64_t who = __ballot(keep);
                if (keep) {
                    const int at = count + __popcll(who & ((1ull << lane) - 1));
                    S.d2[at] = d2;
                    S.id[at] = sid[q];
                    S.q[at] = q;
                }
                count += __popcll(who);
                if (count > KNN_CAND - 64) {
                    count = knn_cut<NK>(S, count);
                    if (count == NK) {
                        thr = S.d2[NK - 1];
                        cut = true;
                    }
                }
            }
            wave_lds_sync();
        }
        if (next > s) {
            if (count >= NK || (all && !guess)) break;
            if (guess) next = 2;  // too short
            guess = false;
        }
        s = next;
    }
    const int cnt = knn_cut<NK>(S, count);
    if (lane == 0 && shell_exceeds_box(g, cnt, NK, cnt == NK ? S.d2[NK - 1] : INFINITY)) atomicOr(box_fail, 1);
    if (lane < NK) {
        int32_t j = -1;
        double r0 = 0, r1 = 0, r2 = 0;
        if (lane < cnt) {
            j = S.id[lane];
            const int64_t q = S.q[lane];
            r0 = min_image(spos[3 * q] - xi, g, 0);
            r1 = min_image(spos[3 * q + 1] - yi, g, 1);
            r2 = min_image(spos[3 * q + 2] - zi, g, 2);
        }
        nbr_id[(int64_t)lane * n + p] = j;
        nbr_rel[((int64_t)lane * 3 + 0) * n + p] = r0;
        nbr_rel[((int64_t)lane * 3 + 1) * n + p] = r1;
        nbr_rel[((int64_t)lane * 3 + 2) * n + p] = r2;
    }
    wave_lds_sync();  // the list is free for the wave's next atom
}

template <int NK>
__global__ void __launch_bounds__(256, 4) k_knn_exact(int64_t n, GridArg A, const double *__restrict__ spos,
                                                   const int32_t *__restrict__ sid, const int32_t *__restrict__ start,
                                                   int32_t *__restrict__ nbr_id, double *__restrict__ nbr_rel,
                                                   const int32_t *__restrict__ todo,
                                                   const int32_t *__restrict__ todo_count,
                                                   int32_t *__restrict__ box_fail) {
    __shared__ KnnWave S[4];
    if (*box_fail > FRAME_BOX) return;
    if (A.dev && !A.dev->fast) todo = nullptr;  // the fast search left every atom
    const Grid g = grid_of(A);
    const int64_t nwaves = (int64_t)gridDim.x * (blockDim.x >> 6);
    const int64_t cnt_todo = todo ? (int64_t)*todo_count : n;
    for (int64_t w = blockIdx.x * (int64_t)(blockDim.x >> 6) + (threadIdx.x >> 6); w < cnt_todo; w += nwaves)
        knn_exact_atom<NK>(S[threadIdx.x >> 6], todo ? (int64_t)todo[w] : w, n, g, spos, sid, start, nbr_id, nbr_rel,
                           box_fail);
}

// ------------------------------------------------- topological ordering
// Sec. 3: neighbours ordered by the area of the interface between the
// Voronoi cell of the centre and theirs, larger first, then by 1/d; the cell
// is that of the centre and its 18 nearest neighbours (Sec. 9).  The cell
// {x : x.n_j <= 1}, n_j = 2 d_j / |d_j|^2, is the polar of the convex hull
// of the points n_j: hull vertices are the cell's faces, each hull facet
// (a, b, c) is a cell vertex w (w.n_a = w.n_b = w.n_c = 1) and hull edges
// are cell edges.  Two kernels, one lane per atom in each:
//   k_voronoi_hull   builds the hull incrementally with exact predicates and
//                    Simulation of Simplicity by Euclidean rank (points
//                    inside the current hull are skipped; vertices that a
//                    later point swallows drop out of every facet) and
//                    writes its facets;
//   k_voronoi_order  reads them back, computes the area of face v as
//                    |sum over the facets f at v of (w_f x w_g) . n_v| /
//                    (2 |n_v|), g being the facet across f's edge that starts
//                    at v (consecutive vertices of the face polygon, in one
//                    direction), and writes the first 14 neighbours in the
//                    topological order.
// The hull keeps FP32 copies of the points in LDS (an exact filter, with the
// FP64 points recomputed from the neighbour vectors when it cannot decide),
// the areas need the FP64 points: splitting the two lets each kernel hold
// only what it reads.  Areas are compared on a grid of 2^-20 of the cell's
// surface, so that equal areas tie whatever their rounding; ties fall to the
// Euclidean rank, i.e. to 1/d.  Atoms with fewer than 18 neighbours, or an
// unbounded cell (the centre not strictly inside the hull), keep the
// Euclidean order: no hull of any subset of their neighbours can then hold
// the centre.
constexpr int VF = 2 * VK - 4;  // facets of a triangulated sphere on 18 vertices
constexpr int VB = 64;          // lanes per block
constexpr double AREA_GRID = 1048576.0;

// 24,320 bytes per 64-lane block: six blocks per CU
struct VHullShared {
    float P[3][VK][VB];  // the points n_j rounded to FP32, component-major, lane-minor
    uint32_t F[VF][VB];  // facets: vertices a | b << 5 | c << 10, link e at 15 + 5 e
    uint16_t H[VK][VB];  // horizon edges of the insertion in progress: a | b << 5 | g << 10
};
// 35,840 bytes per 64-lane block
struct VAreaShared {
    double P[3][VK][VB];  // the points n_j
    uint32_t F[VF][VB];
};

__device__ inline uint32_t vpack(int a, int b, int c, int g0, int g1, int g2) {
    return (uint32_t)a | ((uint32_t)b << 5) | ((uint32_t)c << 10) | ((uint32_t)g0 << 15) | ((uint32_t)g1 << 20) |
           ((uint32_t)g2 << 25);
}
__device__ inline int vv(uint32_t f, int e) { return (f >> (5 * e)) & 31; }
__device__ inline int vl(uint32_t f, int e) { return (f >> (15 + 5 * e)) & 31; }
// position of vertex x in facet f (f must hold x)
__device__ inline int vpos(uint32_t f, int x) { return vv(f, 0) == x ? 0 : (vv(f, 1) == x ? 1 : 2); }
__device__ inline int field5(uint64_t lo, uint64_t hi, int v) {
    return (int)((v < 12 ? lo >> (5 * v) : hi >> (5 * (v - 12))) & 31);
}
__device__ inline void set5(uint64_t &lo, uint64_t &hi, int v, int s) {
    if (v < 12) lo |= (uint64_t)s << (5 * v);
    else hi |= (uint64_t)s << (5 * (v - 12));
}

// n_j = d_j * (2 / |d_j|^2) from the neighbour vectors: the one definition
// of the FP64 points, used by both kernels
__device__ inline void dual_point(const double *__restrict__ rel18, int64_t n, int64_t p, int j, double (&x)[3]) {
    const double a = rel18[((int64_t)j * 3 + 0) * n + p], b = rel18[((int64_t)j * 3 + 1) * n + p],
                 c = rel18[((int64_t)j * 3 + 2) * n + p];
    const double sc = 2.0 / ((a * a + b * b) + c * c);
    x[0] = a * sc;
    x[1] = b * sc;
    x[2] = c * sc;
}

struct VLane {
    VHullShared &S;
    int t;
    const double *__restrict__ rel18;
    int64_t n, p;
    double bo, bd;      // FP32 filter bounds of this lane's points
    double bo64, bd64;  // FP64 filter bounds
    __device__ void load(int j, float (&x)[3]) const {
        x[0] = S.P[0][j][t];
        x[1] = S.P[1][j][t];
        x[2] = S.P[2][j][t];
    }
    // where the FP32 filter cannot decide: the FP64 filter, then exact
    // arithmetic with SoS
    __device__ int orient_exact(int a, int b, int c, int q) const {
        double da[3], db[3], dc[3], dq[3];
        dual_point(rel18, n, p, a, da);
        dual_point(rel18, n, p, b, db);
        dual_point(rel18, n, p, c, dc);
        dual_point(rel18, n, p, q, dq);
        return orient_sos64b(da, db, dc, dq, a, b, c, q, bo64);
    }
    __device__ int orient(int a, int b, int c, const float (&pq)[3], int q) const {
        float pa[3], pb[3], pc[3];
        load(a, pa);
        load(b, pb);
        load(c, pc);
        const int s = orient_filter_f32in(pa, pb, pc, pq, bo);
        return s ? s : orient_exact(a, b, c, q);
    }
    __device__ int det3(uint32_t f) const {
        float pa[3], pb[3], pc[3];
        load(vv(f, 0), pa);
        load(vv(f, 1), pb);
        load(vv(f, 2), pc);
        const int s = det3_filter_f32in(pa, pb, pc, bd);
        if (s) return s;
        double da[3], db[3], dc[3];
        dual_point(rel18, n, p, vv(f, 0), da);
        dual_point(rel18, n, p, vv(f, 1), db);
        dual_point(rel18, n, p, vv(f, 2), dc);
        return det3_sign64b(da, db, dc, bd64);
    }
};

// the cell vertex of the facet (a, b, c): w.n_a = w.n_b = w.n_c = 1, i.e.
// (n_b x n_c + n_c x n_a + n_a x n_b) / det[n_a; n_b; n_c]
__device__ inline void cell_vertex(const double (&a)[3], const double (&b)[3], const double (&c)[3], double (&w)[3]) {
#pragma clang fp contract(fast)
    const double bc0 = b[1] * c[2] - b[2] * c[1], bc1 = b[2] * c[0] - b[0] * c[2], bc2 = b[0] * c[1] - b[1] * c[0];
    const double ca0 = c[1] * a[2] - c[2] * a[1], ca1 = c[2] * a[0] - c[0] * a[2], ca2 = c[0] * a[1] - c[1] * a[0];
    const double ab0 = a[1] * b[2] - a[2] * b[1], ab1 = a[2] * b[0] - a[0] * b[2], ab2 = a[0] * b[1] - a[1] * b[0];
    const double inv = 1.0 / (a[0] * bc0 + a[1] * bc1 + a[2] * bc2);
    w[0] = (bc0 + ca0 + ab0) * inv;
    w[1] = (bc1 + ca1 + ab1) * inv;
    w[2] = (bc2 + ca2 + ab2) * inv;
}

// first tetrahedron of points 0..3, positively oriented; facets 0..3
__device__ inline void vhull_start(const VLane &L) {
    int a = 0, b = 1, c = 2;
    const int d = 3;
    float p3[3];
    L.load(3, p3);
    if (L.orient(0, 1, 2, p3, 3) > 0) { b = 2; c = 1; }
    L.S.F[0][L.t] = vpack(a, b, c, 1, 2, 3);
    L.S.F[1][L.t] = vpack(b, a, d, 0, 3, 2);
    L.S.F[2][L.t] = vpack(c, b, d, 0, 1, 3);
    L.S.F[3][L.t] = vpack(a, c, d, 0, 2, 1);
}

// Insert point p into the hull whose facets are the slots in `live`.  A
// point inside leaves the hull as it is.  New facets take the lowest free
// slots (the visible facets' included).  Returns false on an inconsistent
// hull, which exact predicates never produce.
__device__ inline bool vhull_insert(const VLane &L, int p, uint32_t &live) {
    VHullShared &S = L.S;
    const int t = L.t;
    float pp[3];
    L.load(p, pp);
    uint32_t vis = 0;
    const float bf = (float)L.bo;
    // two facets per step: both filters' loads are issued together.  A facet
    // is visible when its FP32 determinant lies below -bound; those within
    // the bound (or NaN) take the exact path after the loop (a wave then pays
    // for the most any lane has, not for every step in which some lane has one).
    uint32_t und = 0;
    for (uint32_t m = live; m;) {
        const int f0 = __builtin_ctz(m);
        m &= m - 1;
        const bool two = m != 0;
        const int f1 = two ? __builtin_ctz(m) : f0;
        if (two) m &= m - 1;
        const uint32_t w0 = S.F[f0][t], w1 = S.F[f1][t];
        float a0[3], b0[3], c0[3], a1[3], b1[3], c1[3];
        L.load(vv(w0, 0), a0);
        L.load(vv(w0, 1), b0);
        L.load(vv(w0, 2), c0);
        L.load(vv(w1, 0), a1);
        L.load(vv(w1, 1), b1);
        L.load(vv(w1, 2), c1);
        const float d0 = orient_det_f32in(a0, b0, c0, pp), d1 = orient_det_f32in(a1, b1, c1, pp);
        // (f1 is f0 again when there is no second)
        vis |= (d0 < -bf ? 1u << f0 : 0u) | (d1 < -bf ? 1u << f1 : 0u);
        und |= (!(fabsf(d0) > bf) ? 1u << f0 : 0u) | (!(fabsf(d1) > bf) ? 1u << f1 : 0u);
    }
    for (; und; und &= und - 1) {
        const int f = __builtin_ctz(und);
        const uint32_t w = S.F[f][t];
        if (L.orient_exact(vv(w, 0), vv(w, 1), vv(w, 2), p) > 0) vis |= 1u << f;
    }
    if (!vis) return true;
    // horizon edges (a -> b) of the visible facets whose neighbour g is not
    // visible, one per start vertex: H[a] = b | g << 5.  Inner edges write
    // to row VK - 1, which is no start vertex (a < p <= VK - 1), so the loop
    // body has no branch.
    uint32_t hv = 0, he = 0;      // start and end vertices of the horizon
    uint64_t pr_lo = 0, pr_hi = 0;  // 5-bit field b: a of the horizon edge a -> b
    int nh = 0;
    bool bad = false;
    for (uint32_t m = vis; m; m &= m - 1) {
        const uint32_t w = S.F[__builtin_ctz(m)][t];
#pragma unroll
        for (int e = 0; e < 3; e++) {
            const int g = vl(w, e);
            bad |= !((live >> g) & 1);
            const bool hz = !((vis >> g) & 1);
            const int ha = vv(w, e), hb = vv(w, e == 2 ? 0 : e + 1);
            S.H[hz ? ha : VK - 1][t] = (uint16_t)(hb | (g << 5));
            hv |= (uint32_t)hz << ha;
            he |= (uint32_t)hz << hb;
            set5(pr_lo, pr_hi, hb, hz ? ha : 0);
            nh += hz;
        }
    }
    // the horizon is one cycle: an edge leaves and one enters every vertex
    if (bad || __builtin_popcount(hv) != nh || he != hv) return false;
    // slots in increasing order of the start vertex; the new facet (a, b, p)
    // links to g across a -> b, to the facet of b across b -> p and to the
    // facet of pred(a) across p -> a
    const uint32_t freeset = ~(live & ~vis);
    uint64_t sl_lo = 0, sl_hi = 0;  // 5-bit slot per start vertex
    uint32_t fr = freeset, added = 0;
    for (uint32_t m = hv; m; m &= m - 1) {
        if (!fr) return false;
        const int s = __builtin_ctz(fr);
        fr &= fr - 1;
        added |= 1u << s;
        set5(sl_lo, sl_hi, __builtin_ctz(m), s);
    }
    for (uint32_t m = hv; m; m &= m - 1) {
        const int a = __builtin_ctz(m);
        const uint32_t hw = S.H[a][t];
        const int b = hw & 31, g = (hw >> 5) & 31;
        const int sa = field5(sl_lo, sl_hi, a);
        S.F[sa][t] = vpack(a, b, p, g, field5(sl_lo, sl_hi, b), field5(sl_lo, sl_hi, field5(pr_lo, pr_hi, a)));
        // g holds the edge b -> a; its link there now points to sa
        const uint32_t gw = S.F[g][t];
        const int eg = vpos(gw, b);
        S.F[g][t] = (gw & ~(31u << (15 + 5 * eg))) | ((uint32_t)sa << (15 + 5 * eg));
    }
    live = (live & ~vis) | added;
    return true;
}

// Squared distance from the origin of the closest facet plane of a hull
// that holds the origin, from the FP64 points, lowered by a relative 1e-6
// (far above the rounding of the evaluation): a point closer to the origin
// than this is strictly inside the hull, and so inside every later (larger)
// hull.  -1 when the origin is not inside.
__device__ inline double vhull_inradius2(const VLane &L, uint32_t live) {
    double r2 = INFINITY;
    // four facets per step (the first one again where fewer are left), so
    // that their 36 loads are in flight together
    for (uint32_t m = live; m;) {
        int f[4];
        f[0] = __builtin_ctz(m);
        m &= m - 1;
#pragma unroll
        for (int k = 1; k < 4; k++) {
            f[k] = m ? __builtin_ctz(m) : f[0];
            m &= m - 1;
        }
        double a[4][3], b[4][3], c[4][3];
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const uint32_t w = L.S.F[f[k]][L.t];
            dual_point(L.rel18, L.n, L.p, vv(w, 0), a[k]);
            dual_point(L.rel18, L.n, L.p, vv(w, 1), b[k]);
            dual_point(L.rel18, L.n, L.p, vv(w, 2), c[k]);
        }
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const double u0 = b[k][0] - a[k][0], u1 = b[k][1] - a[k][1], u2 = b[k][2] - a[k][2];
            const double v0 = c[k][0] - a[k][0], v1 = c[k][1] - a[k][1], v2 = c[k][2] - a[k][2];
            const double n0 = u1 * v2 - u2 * v1, n1 = u2 * v0 - u0 * v2, n2 = u0 * v1 - u1 * v0;
            const double h = n0 * a[k][0] + n1 * a[k][1] + n2 * a[k][2];
            if (!(h > 0)) return -1.0;  // the origin is not inside: no bound
            r2 = fmin(r2, h * h / ((n0 * n0 + n1 * n1) + n2 * n2));
        }
    }
    return r2 * (1.0 - 1e-6);
}

// Hull of the 18 points of each atom; facets to vf[f][n] (slots in the
// 32-bit mask vlive[n], 0 when the atom keeps its Euclidean order).
__global__ void __launch_bounds__(VB) k_voronoi_hull(int64_t n, const double *__restrict__ rel18,
                                                     const int32_t *__restrict__ id18, uint32_t *__restrict__ vf,
                                                     uint32_t *__restrict__ vlive,
                                                     const int32_t *__restrict__ box_fail) {
    __shared__ VHullShared S;
    const int t = threadIdx.x;
    const int64_t p = xcd_block(blockIdx.x, gridDim.x) * (int64_t)VB + t;
    if (p >= n || *box_fail) return;
    bool topo = id18[(int64_t)(VK - 1) * n + p] >= 0;
    float m = 0;
    uint32_t hk[VK];  // a mix of each point's FP32 bits: equal points have equal keys
    double nrm2[VK - 12];  // |n_q|^2 of points 12..17 (the inradius skip below)
#pragma unroll
    for (int v = 0; v < VK; v++) {
        double x[3];
        dual_point(rel18, n, p, v, x);
        if (v >= 12) nrm2[v - 12] = (x[0] * x[0] + x[1] * x[1]) + x[2] * x[2];
        // a neighbour at the centre has no bisector plane (its point is not
        // finite): the atom keeps its Euclidean order
        topo = topo && isfinite(x[0]) && isfinite(x[1]) && isfinite(x[2]);
        uint32_t h = 0;
        for (int d = 0; d < 3; d++) {
            const float xf = (float)x[d];
            S.P[d][v][t] = xf;
            m = fmaxf(m, fabsf(xf));
            h = h * 0x9E3779B1u + __float_as_uint(xf);
        }
        hk[v] = h;
    }
    // two coincident neighbours share one bisector plane: no interface
    // belongs to either alone, and the atom keeps its Euclidean order (equal
    // keys first, then the FP32 copies, then the FP64 vectors)
    bool maybe = false;
#pragma unroll
    for (int j = 0; j < VK - 1; j++)
#pragma unroll
        for (int k = j + 1; k < VK; k++) maybe = maybe || hk[j] == hk[k];
    if (maybe && topo)
        for (int j = 0; j < VK - 1 && topo; j++)
            for (int k = j + 1; k < VK && topo; k++)
                if (S.P[0][j][t] == S.P[0][k][t] && S.P[1][j][t] == S.P[1][k][t] && S.P[2][j][t] == S.P[2][k][t]) {
                    bool same = true;
                    for (int d = 0; d < 3; d++)
                        same = same && rel18[((int64_t)j * 3 + d) * n + p] == rel18[((int64_t)k * 3 + d) * n + p];
                    topo = !same;
                }
    uint32_t live = 0;
    if (topo) {
        double m64 = 0;
        for (int v = 0; v < VK; v++)
            for (int d = 0; d < 3; d++) m64 = fmax(m64, fabs((double)S.P[d][v][t]));
        // the FP64 bounds from the largest coordinate of the FP32 copies, widened to cover the rounding
        m64 *= 1.0 + 0x1p-22;
        VLane L{S, t, rel18, n, p, f32_orient_bound(m), f32_det3_bound(m), f64_orient_bound(m64),
                f64_det3_bound(m64)};
        vhull_start(L);
        live = 0xFu;
        double rin2 = -1.0;  // inradius bound of the 12-point hull
        for (int q = 4; q < VK && topo; q++) {
            if (q == 12) rin2 = vhull_inradius2(L, live);
            if (q >= 12 && rin2 > 0 && nrm2[q - 12] < rin2) continue;  // strictly inside
            topo = vhull_insert(L, q, live);
        }
        // the centre strictly inside every facet
        for (uint32_t mm = live; mm && topo; mm &= mm - 1) topo = L.det3(S.F[__builtin_ctz(mm)][t]) > 0;
        if (!topo) live = 0;
        for (uint32_t mm = live; mm; mm &= mm - 1) {
            const int f = __builtin_ctz(mm);
            vf[(int64_t)f * n + p] = S.F[f][t];
        }
    }
    vlive[p] = live;
}

// Areas, keys and the topological order from the facets of k_voronoi_hull.
__global__ void __launch_bounds__(VB) k_voronoi_order(int64_t n, const double *__restrict__ rel18,
                                                      const int32_t *__restrict__ id18,
                                                      const uint32_t *__restrict__ vf,
                                                      const uint32_t *__restrict__ vlive,
                                                      double *__restrict__ nbr_rel, int32_t *__restrict__ nbr_id,
                                                      const int32_t *__restrict__ box_fail) {
#pragma clang fp contract(fast)
    __shared__ VAreaShared S;
    const int t = threadIdx.x;
    const int64_t p = xcd_block(blockIdx.x, gridDim.x) * (int64_t)VB + t;
    if (p >= n || *box_fail) return;
    // Euclidean rank v goes to row pos(v); keys order (grid area descending, rank)
    uint32_t key[VK];
#pragma unroll
    for (int v = 0; v < VK; v++) key[v] = (uint32_t)v;
    const uint32_t live = vlive[p];
    if (live) {
        // every load is issued before any is used (one wave per SIMD: no
        // other wave hides a chain of round trips): all VF facet rows (each
        // exists; dead slots are read and ignored) and the points
        uint32_t fw[VF];
#pragma unroll
        for (int f = 0; f < VF; f++) fw[f] = vf[(int64_t)f * n + p];
#pragma unroll
        for (int v = 0; v < VK; v++) {
            double x[3];
            dual_point(rel18, n, p, v, x);
            S.P[0][v][t] = x[0];
            S.P[1][v][t] = x[1];
            S.P[2][v][t] = x[2];
        }
        // one facet at each vertex: 5-bit fields, 31 = not a vertex (a
        // vertex has at least three facets, so slot 31 is never needed)
        uint64_t at_lo = ~0ull, at_hi = ~0ull;
#pragma unroll
        for (int f = 0; f < VF; f++) {
            if (!((live >> f) & 1)) continue;
            const uint32_t w = fw[f];
            S.F[f][t] = w;
            if (f == 31) continue;
            for (int e = 0; e < 3; e++) {
                const int x = vv(w, e);
                if (x < 12) at_lo = (at_lo & ~(31ull << (5 * x))) | ((uint64_t)f << (5 * x));
                else at_hi = (at_hi & ~(31ull << (5 * (x - 12)))) | ((uint64_t)f << (5 * (x - 12)));
            }
        }
        auto load = [&](int j, double (&x)[3]) {
            x[0] = S.P[0][j][t];
            x[1] = S.P[1][j][t];
            x[2] = S.P[2][j][t];
        };
        // face v: walk the facets around v (each next one across the edge
        // that starts at v), summing w_f x w_next; every step brings one new
        // point, the facet's vertex after v
        double area[VK], tot = 0;
#pragma unroll
        for (int v = 0; v < VK; v++) {
            area[v] = 0;
            const int f0 = field5(at_lo, at_hi, v);
            if (f0 == 31) continue;
            double nv[3], a[3], b[3], w0[3], wp[3];
            load(v, nv);
            uint32_t w = S.F[f0][t];
            int e = vpos(w, v);
            load(vv(w, e == 2 ? 0 : e + 1), a);
            load(vv(w, e == 0 ? 2 : e - 1), b);
            cell_vertex(nv, a, b, w0);
            wp[0] = w0[0]; wp[1] = w0[1]; wp[2] = w0[2];
            double sx = 0, sy = 0, sz = 0;
            for (int step = 0; step < VF; step++) {
                const int g = vl(w, e);
                double wn[3];
                if (g == f0) {
                    wn[0] = w0[0]; wn[1] = w0[1]; wn[2] = w0[2];
                } else {
                    const uint32_t gw = S.F[g][t];
                    const int eg = vpos(gw, v);
                    // in g the edge v -> (previous successor) is reversed: the new point follows v
                    double c[3];
                    load(vv(gw, eg == 2 ? 0 : eg + 1), c);
                    cell_vertex(nv, c, a, wn);
                    a[0] = c[0]; a[1] = c[1]; a[2] = c[2];
                    w = gw;
                    e = eg;
                }
                sx += wp[1] * wn[2] - wp[2] * wn[1];
                sy += wp[2] * wn[0] - wp[0] * wn[2];
                sz += wp[0] * wn[1] - wp[1] * wn[0];
                wp[0] = wn[0]; wp[1] = wn[1]; wp[2] = wn[2];
                if (g == f0) break;
            }
            area[v] = fabs(sx * nv[0] + sy * nv[1] + sz * nv[2]) /
                      (2.0 * sqrt((nv[0] * nv[0] + nv[1] * nv[1]) + nv[2] * nv[2]));
            tot += area[v];
        }
        if (tot > 0) {
#pragma unroll
            for (int v = 0; v < VK; v++) {
                const double x = area[v] / tot * AREA_GRID;
                const uint32_t q = (uint32_t)fmin(fmax(floor(x), 0.0), AREA_GRID);
                key[v] = (((uint32_t)AREA_GRID - q) << 5) | (uint32_t)v;
            }
        }
    }
    int pos[VK];
#pragma unroll
    for (int v = 0; v < VK; v++) {
        pos[v] = 0;
#pragma unroll
        for (int u = 0; u < VK; u++) pos[v] += key[u] < key[v];
    }
    // output row by output row, so that the lanes of a wave write each row
    // together (whole cache lines); the source row differs per lane
    for (int m = 0; m < KMAX; m++) {
        int src = 0;
#pragma unroll
        for (int v = 0; v < VK; v++) src = pos[v] == m ? v : src;
        nbr_id[(int64_t)m * n + p] = id18[(int64_t)src * n + p];
#pragma unroll
        for (int c = 0; c < 3; c++) nbr_rel[((int64_t)m * 3 + c) * n + p] = rel18[((int64_t)src * 3 + c) * n + p];
    }
}

// --------------------------------------------------------------- topology
// One incremental convex hull per atom over its 14 nearest neighbours in
// rank order (every point must become a vertex and stay one), with facets
// and neighbour links.  The hull of the first k points is a state of that
// same construction, so the 6-, 12- and 14-point hulls are read off it
// after inserting points 5, 11 and 13: for each, the centre must lie
// strictly inside, then the canonical start-edge code is built and looked
// up.  Per-lane state lives in LDS, lane-minor, so dynamic indices never
// conflict across lanes.
constexpr int TB = 64;  // threads per block of the topology kernel

// LDS of one block.  P: the neighbour vectors rounded to FP32 (the input of
// the predicate filters; every predicate is decided exactly, so both
// precision forms use this kernel); F: facets; H: the horizon of the current
// insertion.  All a lane's own words; the queue of the facet walk takes what a
// hull leaves free.  20,480 bytes: eight blocks per CU.
struct TopoShared {
    float P[3][KMAX][TB];
    uint32_t F[2 * KMAX - 4][TB];
    uint32_t H[KMAX][TB];
};
static_assert(offsetof(TopoShared, H) == offsetof(TopoShared, F) + sizeof(uint32_t) * (2 * KMAX - 4) * TB,
              "H follows F");
static_assert(sizeof(TopoShared) == 20480, "eight blocks of the topology kernel per CU");

// facet word: v0 | v1<<4 | v2<<8 | nb0<<12 | nb1<<17 | nb2<<22
__device__ inline uint32_t fpack(int a, int b, int c, int n0, int n1, int n2) {
    return (uint32_t)a | ((uint32_t)b << 4) | ((uint32_t)c << 8) | ((uint32_t)n0 << 12) | ((uint32_t)n1 << 17) |
           ((uint32_t)n2 << 22);
}
__device__ inline int fv(uint32_t f, int e) { return (f >> (4 * e)) & 0xF; }
__device__ inline int fn(uint32_t f, int e) { return (f >> (12 + 5 * e)) & 0x1F; }
__device__ inline uint32_t fset_nb(uint32_t f, int e, int g) {
    int sh = 12 + 5 * e;
    return (f & ~(0x1Fu << sh)) | ((uint32_t)g << sh);
}

// Per-lane view of the hull inputs: LDS points plus the FP64 originals in
// global memory (used when an FP32 filter cannot decide), and the static
// filter bounds of the atom (from its largest neighbour coordinate).
struct Lane {
    TopoShared &S;
    int t;
    const double *__restrict__ rel;
    int64_t n, p;
    double bo, bd;        // FP32 filter bounds of orient and det3
    double bo64, bd64;    // FP64 filter bounds (the fallback)
    __device__ void load64(int r, double (&x)[3]) const {
        for (int d = 0; d < 3; d++) x[d] = rel[((int64_t)r * 3 + d) * n + p];
    }
    __device__ void load(int r, float (&x)[3]) const {
        for (int d = 0; d < 3; d++) x[d] = S.P[d][r][t];
    }
};

// orientation of facet (a,b,c) against point q where the FP32 filter
// cannot decide: the FP64 filter, then exact arithmetic with SoS
__device__ inline int lane_orient_exact(const Lane &L, int a, int b, int c, int q) {
    double da[3], db[3], dc[3], dq[3];
    L.load64(a, da);
    L.load64(b, db);
    L.load64(c, dc);
    L.load64(q, dq);
    return orient_sos64b(da, db, dc, dq, a, b, c, q, L.bo64);
}

// det[a; b; c] sign where the FP32 filter cannot decide
__device__ inline int lane_det3_exact(const Lane &L, int a, int b, int c) {
    double da[3], db[3], dc[3];
    L.load64(a, da);
    L.load64(b, db);
    L.load64(c, dc);
    return det3_sign64b(da, db, dc, L.bd64);
}

// orientation of facet (a,b,c) against point q (held in registers)
__device__ inline int lane_orient(const Lane &L, int a, int b, int c, const float (&pq)[3], int q) {
    float pa[3], pb[3], pc[3];
    L.load(a, pa);
    L.load(b, pb);
    L.load(c, pc);
    const int s = orient_filter_f32in(pa, pb, pc, pq, L.bo);
    return s ? s : lane_orient_exact(L, a, b, c, q);
}

// first tetrahedron of points 0..3, positively oriented; facets 0..3
__device__ inline void lane_hull_start(const Lane &L) {
    TopoShared &S = L.S;
    const int t = L.t;
    int a = 0, b = 1, c = 2, d = 3;
    float p3[3];
    L.load(3, p3);
    if (lane_orient(L, 0, 1, 2, p3, 3) > 0) { b = 2; c = 1; }
    S.F[0][t] = fpack(a, b, c, 1, 2, 3);
    S.F[1][t] = fpack(b, a, d, 0, 3, 2);
    S.F[2][t] = fpack(c, b, d, 0, 1, 3);
    S.F[3][t] = fpack(a, c, d, 0, 2, 1);
}

// Insert point p into the hull of points 0..p-1 (nf = 2p - 4 facets).
// Returns 0 if p lies inside (it never becomes a vertex) or swallows an
// earlier vertex: then no hull of p or more points is valid.  cv: facet
// slots whose centre test has passed; the slots rewritten here leave it.
__device__ int lane_insert(const Lane &L, int p, uint32_t &cv) {
    TopoShared &S = L.S;
    const int t = L.t;
    const int nf = 2 * p - 4;
    uint32_t vis = 0;
    float pp[3];
    L.load(p, pp);
    const float bf = (float)L.bo;
    // two facets per step (nf is even): both filters' loads are issued
    // together.  A facet is visible when its FP32 determinant lies below
    // -bound; those within the bound (or NaN) take the exact path after the
    // loop: a wave then pays for the most any lane has, not for every step in
    // which some lane has one (noise-free crystals: coplanar quadruples in
    // every atom), and the exact path's code stands in one place.
    uint32_t und = 0;
    for (int f = 0; f < nf; f += 2) {
        const uint32_t w0 = S.F[f][t], w1 = S.F[f + 1][t];
        float a0[3], b0[3], c0[3], a1[3], b1[3], c1[3];
        L.load(fv(w0, 0), a0);
        L.load(fv(w0, 1), b0);
        L.load(fv(w0, 2), c0);
        L.load(fv(w1, 0), a1);
        L.load(fv(w1, 1), b1);
        L.load(fv(w1, 2), c1);
        const float d0 = orient_det_f32in(a0, b0, c0, pp), d1 = orient_det_f32in(a1, b1, c1, pp);
        vis |= (d0 < -bf ? 1u << f : 0u) | (d1 < -bf ? 2u << f : 0u);
        und |= (!(fabsf(d0) > bf) ? 1u << f : 0u) | (!(fabsf(d1) > bf) ? 2u << f : 0u);
    }
    for (; und; und &= und - 1) {
        const int f = __builtin_ctz(und);
        const uint32_t w = S.F[f][t];
        if (lane_orient_exact(L, fv(w, 0), fv(w, 1), fv(w, 2), p) > 0) vis |= 1u << f;
    }
    if (vis == 0) return 0;  // p inside: never a vertex
    const int nvis = __builtin_popcount(vis);
    // horizon edges (a -> b) of the visible facets f whose neighbour g is
    // not visible, one per start vertex: H[a] = b | g << 4 | f << 9 | s << 14,
    // s the slot of the new facet (a, b, p): the freed slots, then two new
    // ones, in the order met.  Inner edges write to row KMAX - 1, which is no
    // start vertex (a < p <= KMAX - 1), so the loop body has no branch.
    uint32_t hv = 0, he = 0;  // start and end vertices of the horizon
    uint32_t slots = vis | 3u << nf;
    int nh = 0;
    bool bad = false;
    for (uint32_t vm = vis; vm; vm &= vm - 1) {  // visible facets only
        const int f = __builtin_ctz(vm);
        const uint32_t w = S.F[f][t];
#pragma unroll
        for (int e = 0; e < 3; e++) {
            const int g = fn(w, e);
            bad |= g >= nf;  // broken link (cannot happen with exact predicates)
            const bool hz = !((vis >> g) & 1);
            const int ha = fv(w, e), hb = fv(w, e == 2 ? 0 : e + 1);
            S.H[hz ? ha : KMAX - 1][t] = (uint32_t)hb | ((uint32_t)g << 4) | ((uint32_t)f << 9) |
                                         ((uint32_t)__builtin_ctz(slots | 1u << 31) << 14);
            hv |= (uint32_t)hz << ha;
            he |= (uint32_t)hz << hb;
            slots &= slots - (uint32_t)hz;  // (drops the lowest slot, or nothing)
            nh += hz;
        }
    }
    // a horizon of nvis+2 edges <=> no earlier vertex is swallowed; one
    // edge leaves and one enters every horizon vertex
    if (bad || nh != nvis + 2 || __builtin_popcount(hv) != nh || he != hv) return 0;
    // (with the slots in a table of 5-bit fields per vertex the kernel took
    // 15.3 ms at 31.7 M atoms, where it takes 13.6)
    // once around the horizon: the new facet (a, b, p) links to g across
    // a -> b, to the next one across b -> p and to the last one across p -> a
    // (so each edge is read once, a step ahead, and no table of slots per
    // vertex is needed), and g's link turns from the visible facet to the new
    // one (an XOR: every link changes at most once, so no read-modify-write
    // is needed)
    int a = __builtin_ctz(hv);
    uint32_t hw = S.H[a][t];
    uint32_t last = (hw >> 14) & 0x1F;  // the first edge is taken at the end of the round
    a = (int)(hw & 0xF);
    hw = S.H[a][t];
    for (int k = 0; k < nh; k++) {
        const int b = hw & 0xF, g = (hw >> 4) & 0x1F, f = (hw >> 9) & 0x1F;
        const uint32_t sa = (hw >> 14) & 0x1F;
        const uint32_t next = S.H[b][t];
        // g (not visible, so never a slot taken here) holds the edge b -> a
        // as its edge eg; only its links may have changed
        const uint32_t gw = S.F[g][t];
        S.F[sa][t] = fpack(a, b, p, g, (int)((next >> 14) & 0x1F), (int)last);
        const int eg = (fv(gw, 0) == b) ? 0 : ((fv(gw, 1) == b) ? 1 : 2);
        atomicXor(&S.F[g][t], ((uint32_t)f ^ sa) << (12 + 5 * eg));
        last = sa;
        a = b;
        hw = next;
    }
    cv &= ~vis;  // the freed slots hold new facets
    return 1;
}

// the centre lies strictly inside every facet of the K-point hull:
// det[a; b; c] > 0 exactly.  Facets in cv passed at a smaller hull and are
// not tested again; on success every facet joins cv.
__device__ inline int lane_centre_inside(const Lane &L, int K, uint32_t &cv) {
    const uint32_t all = (1u << (2 * K - 4)) - 1;
    const float bd = (float)L.bd;
    // two facets per step and the undecided ones afterwards, as in the insertion
    uint32_t und = 0;
    for (uint32_t m = all & ~cv; m;) {
        const int f0 = __builtin_ctz(m);
        m &= m - 1;
        const int f1 = m ? __builtin_ctz(m) : f0;  // (f0 again when it is the last)
        m &= m - 1;
        const uint32_t w0 = L.S.F[f0][L.t], w1 = L.S.F[f1][L.t];
        float a0[3], b0[3], c0[3], a1[3], b1[3], c1[3];
        L.load(fv(w0, 0), a0);
        L.load(fv(w0, 1), b0);
        L.load(fv(w0, 2), c0);
        L.load(fv(w1, 0), a1);
        L.load(fv(w1, 1), b1);
        L.load(fv(w1, 2), c1);
        // outside below -bound; within the bound (or NaN) the exact path decides
        const float e0 = det3_f32in(a0, b0, c0), e1 = det3_f32in(a1, b1, c1);
        if (e0 < -bd || e1 < -bd) return 0;
        und |= (!(e0 > bd) ? 1u << f0 : 0u) | (!(e1 > bd) ? 1u << f1 : 0u);
    }
    for (; und; und &= und - 1) {
        const uint32_t w = L.S.F[__builtin_ctz(und)][L.t];
        if (lane_det3_exact(L, fv(w, 0), fv(w, 1), fv(w, 2)) <= 0) return 0;
    }
    cv |= all;
    return 1;
}

// full adder on bit slices: a becomes the sum, the carry is returned
__device__ inline uint32_t add_slices(uint32_t &a, uint32_t b, uint32_t c) {
    const uint32_t carry = (a & b) | (c & (a | b));
    a ^= b ^ c;
    return carry;
}
// position of vertex x in facet w (w holds x)
__device__ inline int fpos(uint32_t w, uint32_t x) { return (w & 0xF) == x ? 0 : (((w >> 4) & 0xF) == x ? 1 : 2); }
// vertex i + j and link i + j (positions mod 3, i 0..2, j 0..2) of facet w
__device__ inline int fvr(uint32_t w, int i, int j) {
    const uint32_t v = w & 0xFFF;
    return (int)(((v | v << 12) >> (4 * (i + j))) & 0xF);
}
__device__ inline int fnr(uint32_t w, int i, int j) {
    const uint32_t l = w >> 12;
    return (int)(((l | l << 15) >> (5 * (i + j))) & 0x1F);
}

// Start-edge code (definition in ptm_tables.cpp: a breadth-first walk over
// the facets) of the K-point hull in F, from the start edge u -> v with u the
// lowest-numbered vertex of minimum degree and v its lowest-numbered
// neighbour.  code receives its words; the return value is the labelling
// (nibble x = label of vertex x).  One code per hull: the tables hold the
// codes of every start edge from a vertex of minimum degree of every template
// triangulation, so the choice among them needs no search.
//
// The walk takes one step per facet (19 and 23, of about 45 instructions,
// without a branch) and needs only the facets and their links.  Walking
// around every vertex instead takes a step per directed edge (60 and 72, of
// about 40) and a rotation system, built with as many LDS atomics.  Issue
// bound as the rest of the kernel; measured on the whole kernel, 17.8 ->
// 15.4 ms at 31.7 M atoms, 607 -> 520 us at 918,996, 66 -> 57 us at 256
// (13.6 ms with the new facets linked around the horizon, lane_insert).
template <int K>
__device__ uint64_t lane_facet_code(TopoShared &S, int t, uint64_t (&code)[CODE_WORDS]) {
    constexpr int NF = 2 * K - 4;
    // vertex sets of the facets, and the degrees bit-sliced (w1, w2, w4: bits
    // of the degree of vertex x in bit x; w8: 8 or more)
    uint32_t m[NF], c2[NF / 2], c4[NF / 4], w1 = 0, w2 = 0, w4 = 0, w8 = 0;
#pragma unroll
    for (int f = 0; f < NF; f++) {
        const uint32_t w = S.F[f][t];
        m[f] = 1u << fv(w, 0) | 1u << fv(w, 1) | 1u << fv(w, 2);
    }
#pragma unroll
    for (int f = 0; f < NF / 2; f++) c2[f] = add_slices(w1, m[2 * f], m[2 * f + 1]);
#pragma unroll
    for (int f = 0; f < NF / 4; f++) c4[f] = add_slices(w2, c2[2 * f], c2[2 * f + 1]);
#pragma unroll
    for (int f = 0; f < NF / 4; f += 2) w8 |= add_slices(w4, c4[f], f + 1 < NF / 4 ? c4[f + 1] : 0u);
    // a triangulated sphere has a vertex of degree 3, 4 or 5
    const uint32_t z3 = w1 & w2 & ~(w4 | w8), z4 = w4 & ~(w1 | w2 | w8), z5 = w1 & w4 & ~(w2 | w8);
    const uint32_t z = z3 ? z3 : (z4 ? z4 : z5);
    const uint32_t u = z ? (uint32_t)__builtin_ctz(z) : 0u;
    // facets at u and the lowest-numbered neighbour
    uint32_t at_u = 0, nb = 0;
#pragma unroll
    for (int f = 0; f < NF; f++) {
        const uint32_t in = (m[f] >> u) & 1;
        at_u |= in << f;
        nb |= m[f] & (0u - in);
    }
    nb &= ~(1u << u);
    const uint32_t v = nb ? (uint32_t)__builtin_ctz(nb) : 0u;
    // of the two facets with both, the one in which v follows u
    uint32_t at_v = 0;
#pragma unroll
    for (int f = 0; f < NF; f++) at_v |= ((m[f] >> v) & 1) << f;
    const uint32_t both = at_u & at_v;
    const int fa = both ? __builtin_ctz(both) : 0, fb = both ? 31 - __builtin_clz(both) : 0;
    const uint32_t wa = S.F[fa][t], wb = S.F[fb][t];
    const bool first = fvr(wa, fpos(wa, u), 1) == (int)v;
    const int f0 = first ? fa : fb;
    const uint32_t w0 = first ? wa : wb;
    const int i0 = fpos(w0, u);
    const int x2 = fvr(w0, i0, 2);
    uint64_t lab = ~0ull ^ 0xFull << (4 * u) ^ 0xEull << (4 * v) ^ 0xDull << (4 * x2);
    uint32_t nl = 3, seen = 1u << f0;
    // Queue of facets to visit: facet | start of the entry edge in it << 5.  The
    // first three (always new) stay in registers, the others, and one that
    // does not count, take words of the lane's own, a row of TB each: 17 of the
    // 18 that the 12-point hull leaves free in F and H, 21 of P, which the
    // 14-point hull, the last, no longer needs.
    typedef uint32_t __attribute__((may_alias)) entry_t;
    static_assert(K == 12 || K == 14, "the rows below are free");
    entry_t *queue = K == 12 ? &S.F[NF][t] : reinterpret_cast<entry_t *>(&S.P[0][0][t]);
    uint32_t tail = 0;  // byte offset
    auto push = [&](uint32_t g, uint32_t start) {
        const uint32_t fresh = (~seen >> g) & 1;
        // (the next entry overwrites it if it does not count)
        *reinterpret_cast<entry_t *>(reinterpret_cast<char *>(queue) + tail) = g | start << 5;
        seen |= 1u << g;
        tail = (fresh << 8) + tail;
        return fresh;
    };
    const int n0 = fnr(w0, i0, 1), n1 = fnr(w0, i0, 2), n2 = fnr(w0, i0, 0);
    const uint32_t first3[3] = {(uint32_t)n0 | (uint32_t)x2 << 5, (uint32_t)n1 | u << 5, (uint32_t)n2 | v << 5};
    seen |= 1u << n0 | 1u << n1 | 1u << n2;
    uint64_t c0 = 0, c1 = 0, bits = 0;
#pragma unroll
    for (int k = 0; k < NF - 1; k++) {
        const uint32_t e = k < 3 ? first3[k] : queue[(k - 3) * TB];
        const uint32_t start = e >> 5;
        const uint32_t gw = S.F[e & 0x1F][t];  // (rows from 24 lie in H: in range for any entry)
        const int i = fpos(gw, start), c = fvr(gw, i, 2);
        // the facet's third vertex, labelled if it is new
        const uint32_t lc = nib(lab, c);
        const bool fresh = lc == 0xF;
        const uint32_t l = fresh ? nl : lc;
        lab ^= (uint64_t)(lc ^ l) << (4 * c);
        nl += fresh;
        if (k < 16) c0 |= (uint64_t)l << (4 * (k & 15));
        else c1 |= (uint64_t)l << (4 * (k & 15));
        const uint32_t p1 = push(fnr(gw, i, 1), c), p2 = push(fnr(gw, i, 2), start);
        bits |= (uint64_t)(p1 | p2 << 1) << (2 * k);
    }
    code[0] = c0;
    code[1] = c1;
    code[2] = bits;
    return lab;
}

// The 6-point hull: the only template triangulation of six points is the
// SC octahedron, and a triangulated sphere of six vertices is the
// octahedron exactly when every vertex has degree 4; the tables hold its one
// start-edge code (code 0 of the group; they refuse to build otherwise).  So
// the hull either is the octahedron -- code 0, with the labelling of the
// start edge from vertex 0 to its lowest-numbered neighbour read off the
// rotation around vertex 0 -- or has no candidate.  With the neighbours
// counter-clockwise y1..y4 from that one, the facet walk from (0, y1, y2)
// meets the one vertex not adjacent to 0 across y1->y2, then y3 and y4.  Only
// the rotation around vertex 0 is needed, built in a register.
__device__ inline bool lane_octahedron(const uint32_t (*F)[TB], int t, uint64_t &labels) {
    uint64_t degs = 0, row = 0;  // row 0, complemented (0 = no neighbour)
#pragma unroll
    for (int f = 0; f < 8; f++) {
        const uint32_t w = F[f][t];
        const int a = fv(w, 0), b = fv(w, 1), c = fv(w, 2);
        degs += (1ull << (4 * a)) + (1ull << (4 * b)) + (1ull << (4 * c));
        if (a == 0) row |= (uint64_t)(c ^ 0xF) << (4 * b);
        if (b == 0) row |= (uint64_t)(a ^ 0xF) << (4 * c);
        if (c == 0) row |= (uint64_t)(b ^ 0xF) << (4 * a);
    }
    if (degs != 0x444444ull) return false;
    const uint64_t nt0 = ~row;
    uint64_t z = row;
    z = (z | (z >> 1) | (z >> 2) | (z >> 3)) & 0x1111111111111111ull;
    int y = __builtin_ctzll(z) >> 2;  // lowest-numbered neighbour of 0
    uint32_t lab = 0;
    int sum = 0;
#pragma unroll
    for (int j = 1; j <= 4; j++) {
        lab |= (uint32_t)(j < 3 ? j : j + 1) << (4 * y);
        sum += y;
        y = (int)nib(nt0, y);
    }
    labels = lab | 3u << (4 * (15 - sum));  // the vertices 0..5 sum to 15
    return true;
}

// code row c of group grp equals best (all words compared)
__device__ inline bool row_equal(const TablesView &T, int grp, int32_t c, const uint64_t (&best)[CODE_WORDS]) {
    const uint64_t *cw = T.codes[grp] + (int64_t)c * CODE_WORDS;
    uint64_t diff = 0;
#pragma unroll
    for (int i = 0; i < CODE_WORDS; i++) diff |= cw[i] ^ best[i];
    return diff == 0;
}

// Table probe of a code of group grp whose first slot s held c: the code id
// (full-code verification), or -1 when no template triangulation has it.
__device__ int32_t probe_rest(const TablesView &T, int grp, const uint64_t (&best)[CODE_WORDS], int s, int32_t c,
                              bool hit) {
    const int mask = T.hmask[grp];
    for (int probe = 0; probe <= mask; probe++) {
        if (c < 0) return -1;
        if (hit) return c;
        s = (s + 1) & mask;
        c = T.slots[grp][s];
        hit = c >= 0 && row_equal(T, grp, c, best);
    }
    return -1;
}

// One lane per atom: the hulls of the first 6, 12 and 14 neighbours (those
// enabled by need: bit g for hull group g), the candidates of their codes
// (pack_range) and labellings (nibble r = label of rank r) into code_out /
// lab_out [group][n] (-1 / 0 for a group without a candidate or not needed).
// One atom p per lane t of a 64-lane wave, with the wave's LDS S (always
// inlined: the LDS accesses must stay LDS instructions).
__device__ __attribute__((always_inline)) inline void topo_atom(TopoShared &S, int t, int64_t p, int64_t n, const double *__restrict__ nbr_rel,
                          const int32_t *__restrict__ nbr_id, const TablesView &T, uint32_t need,
                          int32_t *__restrict__ code_out, uint64_t *__restrict__ lab_out) {
    // the neighbour ids that say which hulls are possible (the K-th neighbour
    // exists) and all KMAX relative vectors are loaded in one round trip;
    // rows past the last wanted one are stored but never read
    int32_t kid[NGRP];
    for (int g = 0; g < NGRP; g++) kid[g] = nbr_id[(int64_t)(group_k(g) - 1) * n + p];
    double x[KMAX][3];
    for (int r = 0; r < KMAX; r++)
        for (int d = 0; d < 3; d++) x[r][d] = nbr_rel[((int64_t)r * 3 + d) * n + p];
    uint32_t want = 0;
    for (int g = 0; g < NGRP; g++)
        if (((need >> g) & 1) && kid[g] >= 0) want |= 1u << g;
    int32_t cid[NGRP] = {-1, -1, -1};
    uint64_t labw[NGRP] = {0, 0, 0};
    if (want) {
        const int kl = (want & 4) ? 14 : ((want & 2) ? 12 : 6);  // last point to insert
        // The first six points go to LDS first: their loads were issued
        // first, so the 6-point hull is built while the others arrive.  The
        // filter bounds come from the largest coordinate (FP64, and of its
        // stored form) of the points inserted so far, which bounds every
        // predicate on them.
        double m64 = 0;
        float m32 = 0;
        for (int r = 0; r < 6; r++)
            for (int d = 0; d < 3; d++) {
                S.P[d][r][t] = (float)x[r][d];
                m64 = fmax(m64, fabs(x[r][d]));
                m32 = fmaxf(m32, fabsf((float)x[r][d]));
            }
        Lane L{S, t, nbr_rel, n, p, f32_orient_bound(m32), f32_det3_bound(m32), f64_orient_bound(m64),
               f64_det3_bound(m64)};
        lane_hull_start(L);
        // codes of the valid hulls, probed together after the last insertion
        uint64_t c12[CODE_WORDS] = {}, c14[CODE_WORDS] = {}, h[NGRP] = {0, 0, 0};
        bool pend[NGRP] = {false, false, false};
        uint32_t cv = 0;  // facet slots whose centre test passed
        bool ok = lane_insert(L, 4, cv) && lane_insert(L, 5, cv);
        if (ok && (want & 1))
            pend[0] = lane_centre_inside(L, 6, cv) && lane_octahedron(S.F, t, labw[0]);
        // the other points (rows past the last wanted one are stored but
        // never read)
        for (int r = 6; r < KMAX; r++)
            for (int d = 0; d < 3; d++) {
                S.P[d][r][t] = (float)x[r][d];
                if (r < kl) {
                    m64 = fmax(m64, fabs(x[r][d]));
                    m32 = fmaxf(m32, fabsf((float)x[r][d]));
                }
            }
        L.bo = f32_orient_bound(m32);
        L.bd = f32_det3_bound(m32);
        L.bo64 = f64_orient_bound(m64);
        L.bd64 = f64_det3_bound(m64);
        for (int q = 6; ok && q < kl; q++) {
            if (!lane_insert(L, q, cv)) break;
            const int K = q + 1;
            if (K == 12 && (want & 2)) {
                if ((pend[1] = lane_centre_inside(L, 12, cv))) {
                    labw[1] = lane_facet_code<12>(S, t, c12);
                    h[1] = code_hash(c12, CODE_WORDS);
                }
            } else if (K == 14) {
                if ((pend[2] = lane_centre_inside(L, 14, cv))) {
                    labw[2] = lane_facet_code<14>(S, t, c14);
                    h[2] = code_hash(c14, CODE_WORDS);
                }
            }
        }
        cid[0] = pend[0] ? 0 : -1;  // the octahedron's code
        // first slots of the other two probes
        int sl[NGRP];
        int32_t c[NGRP];
        for (int g = 1; g < NGRP; g++) {
            sl[g] = (int)(h[g] & (uint64_t)T.hmask[g]);
            c[g] = pend[g] ? T.slots[g][sl[g]] : -1;
        }
        // every group has a code row 0 (the tables refuse to build
        // otherwise): it stands in for a missing hit, so the rows load
        // unconditionally, before any comparison waits
        const bool hit1 = row_equal(T, 1, max(c[1], 0), c12) & (c[1] >= 0);
        const bool hit2 = row_equal(T, 2, max(c[2], 0), c14) & (c[2] >= 0);
        cid[1] = probe_rest(T, 1, c12, sl[1], c[1], hit1);
        cid[2] = probe_rest(T, 2, c14, sl[2], c[2], hit2);
    }
    int32_t range[NGRP];
    for (int g = 0; g < NGRP; g++) {
        const int32_t *cs = T.cstart[g] + max(cid[g], 0);
        range[g] = cid[g] >= 0 ? pack_range(cs[0], cs[1] - cs[0]) : -1;
    }
    for (int g = 0; g < NGRP; g++) {
        code_out[(int64_t)g * n + p] = range[g];
        lab_out[(int64_t)g * n + p] = cid[g] >= 0 ? labw[g] : 0;
    }
}

__global__ void __launch_bounds__(TB) k_topo(int64_t n, const double *__restrict__ nbr_rel,
                                              const int32_t *__restrict__ nbr_id, TablesView T, uint32_t need,
                                              int32_t *__restrict__ code_out, uint64_t *__restrict__ lab_out,
                                              const int32_t *__restrict__ box_fail) {
    __shared__ TopoShared S;
    const int t = threadIdx.x;
    const int64_t p = blockIdx.x * (int64_t)TB + t;
    if (p >= n || *box_fail) return;
    topo_atom(S, t, p, n, nbr_rel, nbr_id, T, need, code_out, lab_out);
}

// ------------------------------------------------------------------ match
constexpr int MB = 256;  // threads per block of the match kernels

// What the match kernel keeps of each template in LDS: the normalised
// points b (eq. 4), the pseudoinverse V+ (eq. 6), the inverses of the
// rotation group's elements as vertex maps, for each vertex the elements
// whose inverse takes vertex 0 there, G_b = sum |b|^2, k and the group
// order.  The group's quaternions are read from the device tables.
struct TemplateGeom {
    double b[NMAX][3];
    double vpinv[3][NMAX];
    uint64_t ginv[GMAX];
    uint64_t gfirst[KMAX];
    double gb;
    int32_t k, ngroup;
};
struct MatchShared {
    TemplateGeom geo[NT];
};

// f(r) for the ranks r < K of a hull group (6, 12 or 14), unrolled: arrays
// indexed by r stay in registers, and lanes of different K run one code path
template <typename F>
__device__ inline void each_rank(int K, F f) {
#pragma unroll
    for (int r = 0; r < 6; r++) f(r);
    if (K > 6) {
#pragma unroll
        for (int r = 6; r < 12; r++) f(r);
        if (K > 12) {
#pragma unroll
            for (int r = 12; r < KMAX; r++) f(r);
        }
    }
}

// rank vector of the representative: min over g of (c(g^-1(m)))_m, c(v) the
// rank at template vertex v (tv its inverse), packed with m = 0 in the most
// significant nibble.  The first entry is the lowest rank of the orbit of
// vertex 0, attained by the elements that gfirst names; further entries are
// compared only until one element is left (two or three as a rule: an
// element is fixed by the images of few vertices), and one vector is built.
__device__ inline uint64_t rep_vector(const TemplateGeom &D, uint64_t tv, uint64_t c, int &gbest) {
    uint64_t cand = 0;  // bit g: g attains the minimal entries so far
    for (int r = 0; !cand && r < D.k; r++) cand = D.gfirst[nib(tv, r)];
    for (int m = 1; (cand & (cand - 1)) && m < D.k; m++) {
        uint32_t least = 16;
        uint64_t keep = 0;
        for (uint64_t rest = cand; rest; rest &= rest - 1) {
            const int g = __builtin_ctzll(rest);
            const uint32_t f = nib(c, (int)nib(D.ginv[g], m));
            if (f < least) {
                least = f;
                keep = 0;
            }
            if (f == least) keep |= 1ull << g;
        }
        cand = keep;
    }
    gbest = cand ? __builtin_ctzll(cand) : 0;
    const uint64_t gi = D.ginv[gbest];
    uint64_t v = 0;
    each_rank(D.k, [&](int m) { v |= (uint64_t)nib(c, (int)nib(gi, m)) << (4 * (15 - m)); });
    return v;
}

template <typename T>
struct CandEval {
    T r, s, q[4];
    T c;  // FP32 form: bound on the eigen-solve's excess of RMSD^2 (f32_excess_bound)
};

// template vertex of rank r for candidate perm (label -> vertex) and
// labelling lab (rank -> label)
__device__ inline int vertex_of_rank(uint64_t perm, uint64_t lab, int r) { return (int)nib(perm, (int)nib(lab, r)); }

// template vertex of each observed rank
__device__ inline uint64_t tv_of_rank(uint64_t perm, uint64_t lab, int k) {
    uint64_t tv = 0;
    each_rank(k, [&](int r) { tv |= (uint64_t)vertex_of_rank(perm, lab, r) << (4 * r); });
    return tv;
}

// observed rank at each template vertex
__device__ inline uint64_t rank_of_tv(uint64_t tv, int k) {
    uint64_t c = 0;
    each_rank(k, [&](int r) { c |= (uint64_t)r << (4 * nib(tv, r)); });
    return c;
}

// eq.(3) for one candidate of K = 6, 12 or 14 neighbours (observed rank r
// <-> template vertex tv(r); the template from the FP64 table), FP32 form,
// with the observed points streamed from the (cached) neighbour vectors
// instead of held in registers: covariance and G_a / G_b in one pass, the
// residual in a second, each recomputing the centred points from the
// barycentre cb (FP64, eq. 2).  K is a run-time value, so lanes of different
// hull sizes run one code path.
__device__ inline void eval_f32(int K, const double *__restrict__ nbr_rel, int64_t n, int64_t p,
                                const double (&cb)[3], const TemplateGeom &D, uint64_t tv, CandEval<float> &out) {
    // products and sums may fuse into FMAs here (one rounding instead of two; no
    // result depends on a particular rounding)
#pragma clang fp contract(fast)
    typedef float T;
    T S[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
    T Gb = 0;
    double g = 0;
    const T a0[3] = {(T)(-cb[0]), (T)(-cb[1]), (T)(-cb[2])};
    for (int d = 0; d < 3; d++) g += cb[d] * cb[d];
    {
        const T bb[3] = {(T)D.b[0][0], (T)D.b[0][1], (T)D.b[0][2]};
        for (int x = 0; x < 3; x++)
            for (int y = 0; y < 3; y++) S[x][y] += bb[x] * a0[y];
        Gb += bb[0] * bb[0] + bb[1] * bb[1] + bb[2] * bb[2];
    }
#pragma unroll 2
    for (int r = 0; r < K; r++) {
        T a[3];
        for (int d = 0; d < 3; d++) {
            double x = nbr_rel[((int64_t)r * 3 + d) * n + p] - cb[d];
            a[d] = (T)x;
            g += x * x;
        }
        const double *b64 = D.b[nib(tv, r) + 1];
        const T bb[3] = {(T)b64[0], (T)b64[1], (T)b64[2]};
        for (int x = 0; x < 3; x++)
            for (int y = 0; y < 3; y++) S[x][y] += bb[x] * a[y];
        Gb += bb[0] * bb[0] + bb[1] * bb[1] + bb[2] * bb[2];
    }
    const T Ga = (T)g;
    T cond = 0;
    T lam = qcp_solve<T>(S, Ga, Gb, out.q, &cond);
    out.c = f32_excess_bound(lam, cond, Ga);
    T s = Ga > T(0) ? lam / Ga : T(0);
    T R[3][3];
    quat_rot<T>(out.q, R);
    T res = 0;
    {
        const T bb[3] = {(T)D.b[0][0], (T)D.b[0][1], (T)D.b[0][2]};
        for (int x = 0; x < 3; x++) {
            T d = s * a0[x] - (R[x][0] * bb[0] + R[x][1] * bb[1] + R[x][2] * bb[2]);
            res += d * d;
        }
    }
#pragma unroll 2
    for (int r = 0; r < K; r++) {
        T a[3];
        for (int d = 0; d < 3; d++) a[d] = (T)(nbr_rel[((int64_t)r * 3 + d) * n + p] - cb[d]);
        const double *b64 = D.b[nib(tv, r) + 1];
        const T bb[3] = {(T)b64[0], (T)b64[1], (T)b64[2]};
        for (int x = 0; x < 3; x++) {
            T d = s * a[x] - (R[x][0] * bb[0] + R[x][1] * bb[1] + R[x][2] * bb[2]);
            res += d * d;
        }
    }
    out.r = sqrt(res / T(K + 1));
    out.s = s;
}

// x, the same in every lane of the wave, in scalar registers
__device__ inline int64_t uniform(int64_t x) {
    return (int64_t)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)x) |
                     (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(x >> 32)) << 32);
}

// The neighbour vectors of the wave's atoms: component d of rank r of atom a
// (0..63) at rel[(3 r + d) n + a], rel and n in scalar registers, so the
// loads take their addresses from a scalar base and one 32-bit offset.
struct WavePoints {
    const double *__restrict__ rel;
    int64_t n;
    __device__ inline double at(int r, int d, uint32_t a) const { return rel[(int64_t)(3 * r + d) * n + a]; }
};

// The K neighbour vectors of atom a, all in flight together.  The address of
// a row is one scalar addition past the last row's; the empty asm keeps the
// compiler from computing the 42 of them beforehand, where they would not fit
// the scalar registers.
__device__ inline void load_points(int K, const WavePoints &W, uint32_t a, double (&v)[KMAX][3]) {
    typedef const double __attribute__((address_space(1))) *Row;
    uint64_t row = (uint64_t)W.rel;
    each_rank(K, [&](int r) {
        for (int d = 0; d < 3; d++) {
            asm volatile("" : "+s"(row));
            v[r][d] = ((Row)row)[a];
            row += (uint64_t)W.n * 8;
        }
    });
}

// x of lane src / 4 (every lane of the wave must be active)
__device__ inline double from_lane(int src, double x) {
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)(uint32_t)u);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)(uint32_t)(u >> 32));
    return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}
// x or 0, for a mask of all or no bits (also where x is not finite)
__device__ inline double masked(double x, uint32_t mask) {
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    return __longlong_as_double((long long)((uint64_t)((uint32_t)(u >> 32) & mask) << 32 | ((uint32_t)u & mask)));
}

// eq.(3) in FP64 for one candidate per lane, of K = 6, 12 or 14 neighbours
// (observed rank r <-> template vertex perm(lab(r))), by the whole wave: on
// marks the lanes that have one.  pt(r, d) is component d of rank r of the
// lane's atom, called by every lane; sum and Ga are the sum of the atom's
// first K points and G_a.  The template's points sum to zero (eq. 4), so the
// covariance needs no barycentre.
// Moments: the residual at (s, q) is also
// G_b + s (s G_a - 2 rho), rho = sum_i a_i . R b_i = tr(R S^T); it is
// stationary in q and s at the optimum, and its rounding error, a few ulps
// of G_b ~ N, is at most 2e-13 in the RMSD once RMSD >= 0.01 (the
// difference cancels below that, where the explicit sum runs).
template <bool Moments, typename Point>
__device__ inline void eval_f64(bool on, int K, Point pt, const double (&sum)[3], double Ga, const TemplateGeom &D,
                                uint64_t perm, uint64_t lab, CandEval<double> &out) {
    // products and sums may fuse into FMAs here (one rounding instead of two; no
    // result depends on a particular rounding)
#pragma clang fp contract(fast)
    double S[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
    const bool any12 = __ballot(on && K > 6) != 0, any14 = __ballot(on && K > 12) != 0;
    const uint32_t m12 = K > 6 ? ~0u : 0u, m14 = K > 12 ? ~0u : 0u;
    auto add_rank = [&](int r, uint32_t mask) {
        const double *b = D.b[vertex_of_rank(perm, lab, r) + 1];
        for (int y = 0; y < 3; y++) {
            const double c = masked(pt(r, y), mask);
            for (int x = 0; x < 3; x++) S[x][y] += b[x] * c;
        }
    };
#pragma unroll
    for (int r = 0; r < 6; r++) add_rank(r, ~0u);
    if (any12) {
#pragma unroll
        for (int r = 6; r < 12; r++) add_rank(r, m12);
        if (any14) {
#pragma unroll
            for (int r = 12; r < KMAX; r++) add_rank(r, m14);
        }
    }
    double R[3][3], s = 0, a0[3], res = 0;
    bool explicit_sum = on;
    if (on) {
        const double Gb = D.gb, lam = qcp_solve<double>(S, Ga, Gb, out.q);
        s = Ga > 0 ? lam / Ga : 0;
        quat_rot<double>(out.q, R);
        out.s = s;
        if (Moments) {
            double rho = 0;
            for (int x = 0; x < 3; x++)
                for (int y = 0; y < 3; y++) rho += R[x][y] * S[y][x];
            const double rm = Gb + s * (s * Ga - 2 * rho);
            explicit_sum = !(rm >= 1e-4 * (K + 1));
            out.r = sqrt(rm / (K + 1));
        }
    }
    if (!__ballot(explicit_sum)) return;
    auto add_point = [&](const double (&p)[3], const double *b) {
        for (int x = 0; x < 3; x++) {
            const double d = s * p[x] - (R[x][0] * b[0] + R[x][1] * b[1] + R[x][2] * b[2]);
            res += d * d;
        }
    };
    for (int d = 0; d < 3; d++) a0[d] = -sum[d] / (K + 1);
    add_point(a0, D.b[0]);
    auto resid_rank = [&](int r) {
        double p[3];
        for (int d = 0; d < 3; d++) p[d] = pt(r, d) + a0[d];
        if (r < K) add_point(p, D.b[vertex_of_rank(perm, lab, r) + 1]);
    };
#pragma unroll
    for (int r = 0; r < 6; r++) resid_rank(r);
    if (any12) {
#pragma unroll
        for (int r = 6; r < KMAX; r++) resid_rank(r);
    }
    if (explicit_sum) out.r = sqrt(res / (K + 1));
}

// group g's candidates (the pointers selected in registers)
__device__ inline const Candidate *group_candidates(const TablesView &T, int g) {
    return g == 0 ? T.cand[0] : (g == 1 ? T.cand[1] : T.cand[2]);
}

// Outputs of the winning candidate from its superposition ev and the
// strain inputs A^T (sum over points of V+ columns times centred points, in
// template order) and l (mean point norm).
template <typename RT>
__device__ inline void finish_outputs(int K, const MatchShared &M, const Candidate &cd, const TablesView &T, uint64_t tv,
                                      const CandEval<RT> &ev, RT l, const RT (&At)[3][3], RT resid, double cutoff,
                                      int64_t p, int64_t n, int32_t i, const int32_t *__restrict__ nbr_id,
                                      const int8_t *__restrict__ species, const MatchOut &O) {
    // products and sums may fuse into FMAs here (one rounding instead of two; no
    // result depends on a particular rounding)
#pragma clang fp contract(fast)
    const TemplateGeom &G = M.geo[cd.tmpl];
    const TemplateDev &D = T.tpl[cd.tmpl];  // the group's quaternions
    const int type = ((double)ev.r <= cutoff) ? cd.tmpl + 1 : 0;
    if (O.best_type) O.best_type[i] = (int8_t)(cd.tmpl + 1);
    int g;
    const uint64_t rep = rep_vector(G, tv, rank_of_tv(tv, K), g);
    {
        // q' = q * conj(q_g), sign fixed so that the first non-zero component is positive
        const double *qg = D.gq[g];
        RT w1 = ev.q[0], x1 = ev.q[1], y1 = ev.q[2], z1 = ev.q[3];
        RT w2 = (RT)qg[0], x2 = -(RT)qg[1], y2 = -(RT)qg[2], z2 = -(RT)qg[3];
        RT q[4] = {w1 * w2 - x1 * x2 - y1 * y2 - z1 * z2, w1 * x2 + x1 * w2 + y1 * z2 - z1 * y2,
                   w1 * y2 - x1 * z2 + y1 * w2 + z1 * x2, w1 * z2 + x1 * y2 - y1 * x2 + z1 * w2};
        RT qn = sqrt(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
        int flip = 0;
        for (int k = 0; k < 4; k++) {
            if (q[k] > 0) { flip = 1; break; }
            if (q[k] < 0) { flip = -1; break; }
        }
        RT sc = RT(flip < 0 ? -1 : 1) / qn;
        O.type[i] = (int8_t)type;
        if (O.rmsd) O.rmsd[i] = (double)ev.r;
        if (O.scale) O.scale[i] = (double)ev.s;
        if (O.quat) {
            // records as 16-byte pairs (the arrays are 16-byte aligned)
            double2 *qo = reinterpret_cast<double2 *>(O.quat + 4 * (int64_t)i);
            qo[0] = make_double2((double)(q[0] * sc), (double)(q[1] * sc));
            qo[1] = make_double2((double)(q[2] * sc), (double)(q[3] * sc));
        }
        if (O.quat_fz) {
            // Sec. 7: of the equivalent orientations q' x conj(q_h), the one
            // closest to the identity (largest |w|; the first on ties)
            const RT a0 = q[0] * sc, a1 = q[1] * sc, a2 = q[2] * sc, a3 = q[3] * sc;
            RT best[4] = {a0, a1, a2, a3};
            RT bw = RT(-1);
            for (int h = 0; h < G.ngroup; h++) {
                const double *qh = D.gq[h];
                const RT w2 = (RT)qh[0], x2 = -(RT)qh[1], y2 = -(RT)qh[2], z2 = -(RT)qh[3];
                const RT c0 = a0 * w2 - a1 * x2 - a2 * y2 - a3 * z2;
                if (fabs(c0) > bw) {
                    bw = fabs(c0);
                    best[0] = c0;
                    best[1] = a0 * x2 + a1 * w2 + a2 * z2 - a3 * y2;
                    best[2] = a0 * y2 - a1 * z2 + a2 * w2 + a3 * x2;
                    best[3] = a0 * z2 + a1 * y2 - a2 * x2 + a3 * w2;
                }
            }
            RT sg = best[0] < RT(0) ? RT(-1) : RT(1);
            if (best[0] == RT(0))
                for (int k = 1; k < 4; k++)
                    if (best[k] != RT(0)) {
                        sg = best[k] < RT(0) ? RT(-1) : RT(1);
                        break;
                    }
            double2 *qo = reinterpret_cast<double2 *>(O.quat_fz + 4 * (int64_t)i);
            qo[0] = make_double2((double)(sg * best[0]), (double)(sg * best[1]));
            qo[1] = make_double2((double)(sg * best[2]), (double)(sg * best[3]));
        }
        if (O.nn_distance) {
            // hydrostatic part (Sec. 8): template vertex 0 lies at |b_1| in eq.(4) units
            const double *b1 = G.b[1];
            O.nn_distance[i] = ev.s > RT(0) ? sqrt(b1[0] * b1[0] + b1[1] * b1[1] + b1[2] * b1[2]) / (double)ev.s : 0.0;
        }
        if (O.strain_residual) O.strain_residual[i] = (double)resid;
    }
    if (O.neighbours) {
        int32_t ids[KMAX];
#pragma unroll
        for (int m = 0; m < KMAX; m++) {
            int32_t id = -1;
            if (m < K) {
                int rank = (int)((rep >> (4 * (15 - m))) & 0xF);
                id = nbr_id[(int64_t)rank * n + p];
            }
            ids[m] = id;
        }
        // as 8-byte pairs (the array is 8-byte aligned)
        int2 *no = reinterpret_cast<int2 *>(O.neighbours + (int64_t)i * KMAX);
#pragma unroll
        for (int m = 0; m < KMAX / 2; m++) no[m] = make_int2(ids[2 * m], ids[2 * m + 1]);
    }
    if (O.strain || O.vm_strain) {
        // Sec. 8: P of A = P U with U right-handed
        RT P[3][3];
        polar_p<RT>(At, l, P);
        RT sq = 0, tr = 0;
        for (int x = 0; x < 3; x++)
            for (int y = 0; y < 3; y++) {
                const RT s = P[x][y];
                sq += s * s;
                if (x == y) tr += s;
            }
        if (O.strain) {
            double *so = O.strain + 9 * (int64_t)i;
            for (int k = 0; k < 9; k++) so[k] = (double)P[k / 3][k % 3];
        }
        // Sec. 8: von Mises shear strain of P
        if (O.vm_strain) O.vm_strain[i] = (double)sqrt(fmax(RT(1.5) * sq - RT(0.5) * tr * tr, RT(0)));
    }
    if (O.alloy) {
        // alloy (Sec. 6, Table 3)
        int alloy = 0;
        if (species && type && (cd.tmpl == 1 || cd.tmpl == 4)) {
            const int8_t me = species[i];
            uint32_t cnt = 0;  // 8-bit counters: FCC groups 0..2, BCC inner/outer
#pragma unroll
            for (int r = 0; r < KMAX; r++) {
                if (r >= K) break;
                int32_t j = nbr_id[(int64_t)r * n + p];
                int other = species[j] != me;
                int tvx = (int)nib(tv, r);
                int grp2 = (cd.tmpl == 1) ? (tvx >> 2) : (tvx < 8 ? 0 : 1);
                cnt += (uint32_t)other << (8 * grp2);
            }
            if (cd.tmpl == 1) {
                int c0 = cnt & 0xFF, c1 = (cnt >> 8) & 0xFF, c2 = (cnt >> 16) & 0xFF;
                int lo = min(c0, min(c1, c2)), hi = max(c0, max(c1, c2)), mid = c0 + c1 + c2 - lo - hi;
                if (lo == 0 && mid == 0 && hi == 0) alloy = 1;
                else if (lo == 0 && mid == 4 && hi == 4) alloy = 2;
                else if (lo == 0 && mid == 0 && hi == 4) alloy = 3;
                else if (lo == 4 && mid == 4 && hi == 4) alloy = 4;
                else alloy = 5;
            } else {
                int inner = cnt & 0xFF, outer = (cnt >> 8) & 0xFF;
                if (inner == 0 && outer == 0) alloy = 6;
                else if (inner == 8 && outer == 0) alloy = 7;
                else alloy = 8;
            }
        }
        O.alloy[i] = (int8_t)alloy;
    }
}


// Outputs of the winning candidate from its superposition ev (r, q, s), FP32
// form: the points streamed from the (cached) neighbour vectors, about the
// barycentre cb
__device__ inline void finish_f32(int K, const MatchShared &M, const TablesView &T, const Candidate &cd, uint64_t lab,
                              const CandEval<float> &ev, const double (&cb)[3], const double *__restrict__ nbr_rel,
                              double cutoff, int64_t p, int64_t n, int32_t i, const int32_t *__restrict__ nbr_id,
                              const int8_t *__restrict__ species, const MatchOut &O) {
    // products and sums may fuse into FMAs here (one rounding instead of two; no
    // result depends on a particular rounding)
#pragma clang fp contract(fast)
    typedef float RT;
    const TemplateGeom &D = M.geo[cd.tmpl];
    const uint64_t tv = tv_of_rank(cd.perm, lab, K);
    RT a0[3], At[3][3], l;
    strain_begin<RT>(D, cb, a0, At, l);
#pragma unroll
    for (int rr = 0; rr < KMAX; rr++) {
        if (rr >= K) break;
        RT ar[3];
        for (int d = 0; d < 3; d++) ar[d] = (RT)(nbr_rel[((int64_t)rr * 3 + d) * n + p] - cb[d]);
        strain_add<RT>(D, (int)nib(tv, rr) + 1, ar, At, l);
    }
    l /= RT(K + 1);
    RT resid = 0;
    if (O.strain_residual) {
        // eq.(6) residual: sum over points of |V_i A^T - a_i|^2 / l^2
        for (int y = 0; y < 3; y++) {
            RT d = (RT)D.b[0][0] * At[0][y] + (RT)D.b[0][1] * At[1][y] + (RT)D.b[0][2] * At[2][y] - a0[y];
            resid += d * d;
        }
#pragma unroll 2
        for (int rr = 0; rr < K; rr++) {
            const double *v = D.b[(int)nib(tv, rr) + 1];
            for (int y = 0; y < 3; y++) {
                RT ay = (RT)(nbr_rel[((int64_t)rr * 3 + y) * n + p] - cb[y]);
                RT d = (RT)v[0] * At[0][y] + (RT)v[1] * At[1][y] + (RT)v[2] * At[2][y] - ay;
                resid += d * d;
            }
        }
        resid /= l * l;
    }
    finish_outputs<RT>(K, M, cd, T, tv, ev, l, At, resid, cutoff, p, n, i, nbr_id, species, O);
}

// The same in FP64, from the atom's neighbour vectors v and their sum
__device__ inline void finish_f64(int K, const MatchShared &M, const TablesView &T, const Candidate &cd, uint64_t lab,
                              const CandEval<double> &ev, const double (&v)[KMAX][3], const double (&sum)[3],
                              double cutoff, int64_t p, int64_t n, int32_t i, const int32_t *__restrict__ nbr_id,
                              const int8_t *__restrict__ species, const MatchOut &O) {
    // products and sums may fuse into FMAs here (one rounding instead of two; no
    // result depends on a particular rounding)
#pragma clang fp contract(fast)
    const TemplateGeom &D = M.geo[cd.tmpl];
    const uint64_t tv = tv_of_rank(cd.perm, lab, K);
    const double cb[3] = {sum[0] / (K + 1), sum[1] / (K + 1), sum[2] / (K + 1)};
    double a0[3], At[3][3], l;
    strain_begin<double>(D, cb, a0, At, l);
    each_rank(K, [&](int r) {
        double ar[3];
        for (int d = 0; d < 3; d++) ar[d] = (v[r][d] - cb[d]);
        strain_add<double>(D, (int)nib(tv, r) + 1, ar, At, l);
    });
    l /= (K + 1);
    double resid = 0;
    if (O.strain_residual) {
        // eq.(6) residual: sum over points of |V_i A^T - a_i|^2 / l^2
        auto add = [&](const double *b, const double (&ay)[3]) {
            for (int y = 0; y < 3; y++) {
                double d = b[0] * At[0][y] + b[1] * At[1][y] + b[2] * At[2][y] - ay[y];
                resid += d * d;
            }
        };
        add(D.b[0], a0);
        each_rank(K, [&](int r) {
            double ar[3];
            for (int d = 0; d < 3; d++) ar[d] = (v[r][d] - cb[d]);
            add(D.b[(int)nib(tv, r) + 1], ar);
        });
        resid /= l * l;
    }
    finish_outputs<double>(K, M, cd, T, tv, ev, l, At, resid, cutoff, p, n, i, nbr_id, species, O);
}

__device__ inline void write_none(const MatchOut &O, int32_t i) {
    O.type[i] = 0;
    if (O.alloy) O.alloy[i] = 0;
    if (O.rmsd) O.rmsd[i] = INFINITY;
    if (O.scale) O.scale[i] = 0.0;
    if (O.quat) {
        O.quat[4 * (int64_t)i] = 1.0;
        for (int k = 1; k < 4; k++) O.quat[4 * (int64_t)i + k] = 0.0;
    }
    if (O.strain)
        for (int k = 0; k < 9; k++) O.strain[9 * (int64_t)i + k] = 0.0;
    if (O.neighbours)
        for (int m = 0; m < KMAX; m++) O.neighbours[(int64_t)i * KMAX + m] = -1;
    if (O.best_type) O.best_type[i] = 0;
    if (O.vm_strain) O.vm_strain[i] = 0.0;
    if (O.strain_residual) O.strain_residual[i] = 0.0;
    if (O.nn_distance) O.nn_distance[i] = 0.0;
    if (O.quat_fz) {
        O.quat_fz[4 * (int64_t)i] = 1.0;
        for (int k = 1; k < 4; k++) O.quat_fz[4 * (int64_t)i + k] = 0.0;
    }
}

__device__ inline void load_templates(MatchShared &M, const TablesView &T) {
    constexpr int NB = NMAX * 3;  // doubles of b, and of vpinv
    for (int w = threadIdx.x; w < NT * 2 * NB; w += blockDim.x) {
        const int t = w / (2 * NB), e = w % (2 * NB);
        if (e < NB) (&M.geo[t].b[0][0])[e] = (&T.tpl[t].b[0][0])[e];
        else (&M.geo[t].vpinv[0][0])[e - NB] = (&T.tpl[t].vpinv[0][0])[e - NB];
    }
    for (int w = threadIdx.x; w < NT * GMAX; w += blockDim.x) M.geo[w / GMAX].ginv[w % GMAX] = T.tpl[w / GMAX].ginv[w % GMAX];
    for (int w = threadIdx.x; w < NT * KMAX; w += blockDim.x)
        M.geo[w / KMAX].gfirst[w % KMAX] = T.tpl[w / KMAX].gfirst[w % KMAX];
    if ((int)threadIdx.x < NT) {
        M.geo[threadIdx.x].gb = T.tpl[threadIdx.x].gb;
        M.geo[threadIdx.x].k = T.tpl[threadIdx.x].k;
        M.geo[threadIdx.x].ngroup = T.tpl[threadIdx.x].ngroup;
    }
    __syncthreads();
}

// ------------------------------------------------------------ match stage
// One kernel superposes every candidate correspondence of the atoms' hull
// codes (eq. 3), takes the decision of Alg. 1 and writes the outputs of the
// winner.  A wave owns 64 consecutive atoms (cell order):
//  A. lane = atom: the Euclidean neighbour list is copied out, the candidate
//     ranges of the codes go to LDS with the enabled candidates counted, and
//     the points are read once, all 42 components in flight together: FP64
//     keeps them in registers up to the finish, with the sums of the first
//     6, 12 and 14 of them (and G_a) in LDS;
//  B. the wave's candidates form one job list, atom after atom and within
//     an atom in (group, candidate) order, superposed 64 at a time with
//     lane = job (the superposition takes the hull size as a run-time
//     value, so a chunk mixing sizes runs one code path); a bit set of the
//     atoms' first jobs tells each lane its atom.  In FP64 a job takes its
//     atom's points from that atom's lane (ds_bpermute), and the next
//     chunk's candidates are read during this one; after each chunk every
//     atom lane folds its jobs of the chunk, in order, into its running
//     minimum;
//  C. an atom whose decision the common rule cannot take (a near tie, an
//     FP32 margin that the error bounds do not clear) is decided by the
//     full rule in FP64 by the whole wave; every other lane finishes its
//     own winner (the hull size is a run-time value there too, so a wave
//     mixing sizes runs one code path).
// Nothing per candidate leaves the chip.
//
// What bounds it (FP64, 31.7 M atoms, three candidates an atom): of some
// 95,000 cycles of a wave, 31,000 go to the superpositions and 20,000 to the
// finish, both chains of dependent instructions that two waves per SIMD leave
// uncovered (0.38 of the issue slots are used), 13,000 to the fold,
// 12,000 to the first read of the points.  When every job and the finish read
// the points for themselves, rank after rank, a wave waited for each: lanes
// that share an atom hit on each other's outstanding misses, and the waves of
// a CU hold more points than its caches, so 47 GB were fetched for 10.7 GB of
// points.  Measured: 14.9 -> 11.5 ms (17 GB); 486 -> 389 us at 918,996 atoms.
// All 42 components of a job read by the job itself: 14.0 ms; held at three
// waves per SIMD (168 registers) they spill, each spill a wait: 15.8 ms.
// FP32 keeps the points of a job in the caches (a job is shorter, four waves
// per SIMD hide more, and its 128 registers would not hold them).

// LDS of one wave
template <typename RT>
struct MatchWaveLds {
    // sum of the first 6, 12 and 14 points of the wave's atoms (FP32 form:
    // their barycentre), and G_a (FP64 form)
    double sum[NGRP][3][64];
    double ga[NGRP][sizeof(RT) == 8 ? 64 : 1];
    uint64_t lab[NGRP][sizeof(RT) == 8 ? 64 : 1];  // labellings (FP32 form: read per job)
    int32_t range[NGRP][64];  // candidates of each atom's code (see pack_range), the enabled ones counted
    uint64_t starts[64];      // bit t of word c: an atom's first job is job 64 c + t
    uint16_t off[64];         // each atom's first job
    uint8_t act[64];          // the atoms with jobs, in order
    double r[64];             // the current chunk's results: RMSD,
    RT qs[5][64];             // quaternion and scale,
    float d2[64];             // FP32 form: excess bound (f32_excess_bound),
    // template << 56 | permutation (FP32 form: candidate index in the group's list)
    typename std::conditional<sizeof(RT) == 8, uint64_t, int32_t>::type cand[64];
};
// working LDS of a block of NW waves
template <typename RT, int NW>
struct MatchWork {
    MatchWaveLds<RT> w[NW];
};
template <typename RT, int NW>
struct MatchLds {
    MatchShared M;
    // copies of the kernel's table view and output pointers for the full
    // rule, a call: arguments it takes by reference would otherwise be
    // copied to per-lane scratch memory by every lane
    TablesView T;
    MatchOut O;
    MatchWork<RT, NW> work;
};

// The full rule of Alg. 1 for the atom at p, in FP64, by the
// whole wave: lane j superposes the atom's j-th candidate (the codes of one
// atom hold at most 64 together, checked when the tables are built), the
// minimum r* is reduced over the wave, every enabled candidate within the
// tie tolerance of r* computes its representative vector, the (template,
// representative) minimum is reduced, and lane 0 finishes the winner.
// Wave-uniform arguments.
__device__ __noinline__ void full_rule(const MatchShared &M, const TablesView &T, int64_t n, int64_t p,
                          const double *__restrict__ nbr_rel,
                          const int32_t *__restrict__ nbr_id, const int32_t *__restrict__ sid,
                          const int8_t *__restrict__ species, const int32_t *__restrict__ code,
                          const uint64_t *__restrict__ labs, uint32_t mask, double cutoff, const MatchOut &O) {
    const int lane = threadIdx.x & 63;
    const int32_t i = sid[p];
    const WavePoints W = {(const double *)uniform((int64_t)(nbr_rel + p)), uniform(n)};
    int32_t c0[NGRP], nc[NGRP];
    uint64_t lab[NGRP];
    for (int g = 0; g < NGRP; g++) {
        const int32_t cid = code[(int64_t)g * n + p];
        lab[g] = labs[(int64_t)g * n + p];
        c0[g] = range_first(cid);
        nc[g] = range_count(cid);
    }
    // this lane's candidate
    int g = -1, c = -1, tmpl = 99;
    double r = INFINITY;
    {
        int j = lane;
        for (int gg = 0; gg < NGRP && g < 0; gg++) {
            if (j < nc[gg]) {
                g = gg;
                c = c0[gg] + j;
            } else {
                j -= nc[gg];
            }
        }
    }
    Candidate cd = {0, 0, 0};
    CandEval<double> ev = {0, 0, {0, 0, 0, 0}};
    if (g >= 0) {
        cd = T.cand[g][c];
        if ((mask >> cd.tmpl) & 1) tmpl = cd.tmpl;
    }
    {
        const bool on = tmpl < 99;
        const int K = on ? group_k(g) : 6;
        double sum[3] = {0, 0, 0}, gs = 0;
        for (int q = 0; q < K; q++)
            for (int d = 0; d < 3; d++) {
                const double x = W.at(q, d, 0);
                sum[d] += x;
                gs += x * x;
            }
        const double ga = gs - (sum[0] * sum[0] + sum[1] * sum[1] + sum[2] * sum[2]) / (K + 1);
        eval_f64<false>(on, K, [&](int q, int d) { return W.at(q, d, 0); }, sum, ga, M.geo[on ? tmpl : 0], cd.perm,
                        on ? (g == 0 ? lab[0] : (g == 1 ? lab[1] : lab[2])) : 0, ev);
        if (on) r = ev.r;
    }
    double m1 = r;
    for (int off = 32; off > 0; off >>= 1) m1 = fmin(m1, __shfl_xor(m1, off));
    if (m1 == INFINITY) {  // no candidate of an enabled template
        if (lane == 0) write_none(O, i);
        return;
    }
    // tie rule: earliest template, then the smallest representative vector
    int kt = 99;
    uint64_t krep = ~0ull;
    if (r <= m1 + 1e-12) {
        int gsel;
        kt = tmpl;
        const uint64_t tv = tv_of_rank(cd.perm, lab[g], group_k(g));
        krep = rep_vector(M.geo[tmpl], tv, rank_of_tv(tv, group_k(g)), gsel);
    }
    int bt = kt, bl = lane;
    uint64_t brep = krep;
    for (int off = 32; off > 0; off >>= 1) {
        int ot = __shfl_xor(bt, off), ol = __shfl_xor(bl, off);
        uint64_t orep = __shfl_xor(brep, off);
        bool take = ot < bt || (ot == bt && (orep < brep || (orep == brep && ol < bl)));
        if (take) {
            bt = ot;
            brep = orep;
            bl = ol;
        }
    }
    const int wg = __shfl(g, bl), wc = __shfl(c, bl);
    // the winning lane's superposition, handed to the finishing lane
    CandEval<double> we;
    we.r = __shfl(ev.r, bl);
    we.s = __shfl(ev.s, bl);
    for (int k = 0; k < 4; k++) we.q[k] = __shfl(ev.q[k], bl);
    if (lane == 0) {
        const int K = group_k(wg);
        double v[KMAX][3], sum[3] = {0, 0, 0};
        load_points(K, W, 0, v);
        each_rank(K, [&](int q) {
            for (int d = 0; d < 3; d++) sum[d] += v[q][d];
        });
        finish_f64(K, M, T, T.cand[wg][wc], wg == 0 ? lab[0] : (wg == 1 ? lab[1] : lab[2]), we, v, sum, cutoff, p, n,
                   i, nbr_id, species, O);
    }
}

// Bound on |RMSD_FP32 - RMSD| of one candidate evaluated in FP32 from
// FP64-centred points (u = 2^-24; the terms are derived with the FP32-mixed
// form's description):
//   first order, u (72 + 25 r): rounding of the inputs (2.7 u), the
//     covariance sums seen as a perturbation of the inputs (36 u), the
//     rotation built from a unit quaternion rounded to FP32 (15 u), the
//     residual components (17 u), the 45-term sum of squares (23 u r), the
//     division and square root (2 u r);
//   the eigen-solve's excess d2 of RMSD^2 (f32_excess_bound; infinite for
//     an eigenpair FP32 cannot resolve): RMSD^2 + d2 has a square root
//     below RMSD + d2 / (RMSD + sqrt(d2)).
constexpr double RMSD_F32_U = 0x1p-24;
__device__ inline double rmsd_f32_bound(double r, double d2) {
    if (!(d2 < INFINITY)) return INFINITY;
    return RMSD_F32_U * (72.0 + 25.0 * r) + d2 / (r + sqrt(d2));
}

constexpr uint32_t ALL_TEMPLATES = (1u << NT) - 1;

// The match stage for the NW * 64 atoms from first (see the section head),
// by a block of NW waves: templates in M, the LDS copies Tl / Ol of the
// table view and outputs (for the full rule), working LDS Wk.  force_full:
// every atom with a candidate takes the full rule (a test of that path).
// apw: atoms of each wave (the first lanes; NW * apw atoms from first).
// full_count counts the atoms the full rule decides, job_count the
// superposed candidates.
template <typename RT, int NW>
__device__ void match_block(const MatchShared &M, const TablesView &Tl, const MatchOut &Ol, MatchWork<RT, NW> &Wk,
                            int64_t first, int64_t n, const double *__restrict__ nbr_rel,
                            const int32_t *__restrict__ nbr_id, const int32_t *__restrict__ sid,
                            const int8_t *__restrict__ species, const TablesView &T,
                            const int32_t *__restrict__ code, const uint64_t *__restrict__ labs, uint32_t mask,
                            double cutoff, int force_full, const MatchOut &O, int32_t *__restrict__ full_count,
                            unsigned long long *__restrict__ job_count, const int32_t *__restrict__ knn_src,
                            int32_t *__restrict__ knn_out, int apw) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    MatchWaveLds<RT> &W = Wk.w[wv];
    const int64_t wbase = first + (int64_t)wv * apw;
    const int64_t p = wbase + lane;
    const bool live = lane < apw && p < n;
    // (a wave past the last atom reads that one's)
    const WavePoints WP = {(const double *)uniform((int64_t)(nbr_rel + min(wbase, n - 1))), uniform(n)};

    // A. lane = atom
    int cnt[NGRP] = {0, 0, 0};
    double v[KMAX][3];  // FP64 form: the atom's points, from here to the finish
    int32_t rg[NGRP] = {-1, -1, -1};
    if (live)
        for (int g = 0; g < NGRP; g++) {
            rg[g] = code[(int64_t)g * n + p];
            if constexpr (sizeof(RT) == 8) W.lab[g][lane] = labs[(int64_t)g * n + p];
        }
    if constexpr (sizeof(RT) == 8) load_points(KMAX, WP, live ? (uint32_t)lane : 0u, v);
    W.starts[lane] = 0;
    if (live) {
        if (knn_out) {
            // the Euclidean order (Sec. 3) whatever the ordering of the hulls
            const int32_t i = sid[p];
#pragma unroll
            for (int m = 0; m < KMAX; m++) knn_out[(int64_t)i * KMAX + m] = knn_src[(int64_t)m * n + p];
        }
        for (int g = 0; g < NGRP; g++) {
            const int k0 = range_first(rg[g]);
            cnt[g] = range_count(rg[g]);
            if ((mask & ALL_TEMPLATES) != ALL_TEMPLATES) {
                const int k1 = k0 + cnt[g];
                cnt[g] = 0;
                for (int k = k0; k < k1; k++) cnt[g] += (mask >> T.cand[g][k].tmpl) & 1;
            }
            W.range[g][lane] = pack_range(k0, cnt[g]);
        }
    }
    // job offsets: exclusive scan over the wave
    const int mine = cnt[0] + cnt[1] + cnt[2];
    int my_off = mine;
    for (int d = 1; d < 64; d <<= 1) {
        const int y = __shfl_up(my_off, d);
        if (lane >= d) my_off += y;
    }
    const int jobs = __builtin_amdgcn_readlane(my_off, 63);
    my_off -= mine;
    W.off[lane] = (uint16_t)my_off;
    const uint64_t active = __ballot(mine > 0);
    wave_lds_sync();
    if (mine > 0) {
        W.act[__popcll(active & ((1ull << lane) - 1))] = (uint8_t)lane;
        atomicOr((unsigned long long *)&W.starts[my_off >> 6], 1ull << (my_off & 63));
    }
    if (lane == 0 && jobs > 0) atomicAdd(job_count, (unsigned long long)jobs);
    if (live) {
        // barycentres of the centre and the first 6, 12 and 14 neighbours
        double s[3] = {0, 0, 0}, gs = 0;
#pragma unroll
        for (int r = 0; r < KMAX; r++) {
            for (int d = 0; d < 3; d++) {
                if constexpr (sizeof(RT) == 4) {
                    s[d] += WP.at(r, d, (uint32_t)lane);
                } else {
                    s[d] += v[r][d];
                    gs = __builtin_fma(v[r][d], v[r][d], gs);
                }
            }
#pragma unroll
            for (int g = 0; g < NGRP; g++)
                if (r + 1 == group_k(g)) {
                    for (int d = 0; d < 3; d++) W.sum[g][d][lane] = sizeof(RT) == 4 ? s[d] / (group_k(g) + 1) : s[d];
                    // (the centre is the origin, the barycentre far shorter
                    // than the points: nothing cancels)
                    if constexpr (sizeof(RT) == 8)
                        W.ga[g][lane] = gs - (s[0] * s[0] + s[1] * s[1] + s[2] * s[2]) * (1.0 / (group_k(g) + 1));
                }
        }
    }
    wave_lds_sync();

    // B. jobs, 64 at a time
    struct Job {
        int a, g, k;   // atom, group, candidate index
        uint64_t cand;  // template << 56 | permutation
    };
    int begun = 0;  // atoms whose first job lies in an earlier chunk
    auto job = [&](int c0) {
        Job J = {lane, 0, 0, 0};
        if (c0 >= jobs) return J;
        const uint64_t starts = (uint64_t)uniform((int64_t)W.starts[c0 >> 6]);
        if (c0 + lane < jobs) {
            J.a = W.act[begun + __popcll(starts & ((2ull << lane) - 1)) - 1];
            int j = c0 + lane - W.off[J.a];
            const int32_t r0 = W.range[0][J.a], r1 = W.range[1][J.a], r2 = W.range[2][J.a];
            int32_t rj = r0;
            if (j >= range_count(r0)) {
                j -= range_count(r0);
                J.g = 1;
                rj = r1;
                if (j >= range_count(r1)) {
                    j -= range_count(r1);
                    J.g = 2;
                    rj = r2;
                }
            }
            const Candidate *list = group_candidates(T, J.g);
            J.k = range_first(rj);
            if ((mask & ALL_TEMPLATES) == ALL_TEMPLATES) {
                J.k += j;
            } else {
                // the j-th enabled candidate of the code
                for (;; J.k++)
                    if ((mask >> list[J.k].tmpl) & 1) {
                        if (j == 0) break;
                        j--;
                    }
            }
            J.cand = list[J.k].perm | (uint64_t)list[J.k].tmpl << 56;
        }
        begun += __popcll(starts);
        return J;
    };
    double m1 = INFINITY, m2 = INFINITY, b1 = 0.0, lo2 = INFINITY;
    int arg_g = -1;
    decltype(W.cand[0] + 0) arg_c = 0;
    RT wq[5] = {1, 0, 0, 0, 0};  // quaternion and scale of the best job
    Job J = job(0);
    for (int c0 = 0; c0 < jobs; c0 += 64) {
        // (the next chunk's candidates are on the way during this one)
        const Job next = job(c0 + 64);
        const bool on = c0 + lane < jobs;
        const int K = group_k(J.g);
        const uint64_t perm = J.cand & ((1ull << 56) - 1);
        const TemplateGeom &D = M.geo[J.cand >> 56];
        CandEval<RT> ev;
        const double sum[3] = {W.sum[J.g][0][J.a], W.sum[J.g][1][J.a], W.sum[J.g][2][J.a]};
        if constexpr (sizeof(RT) == 4) {
            if (on) {
                const uint64_t lab = labs[(int64_t)J.g * n + wbase + J.a];
                eval_f32(K, nbr_rel, n, wbase + J.a, sum, D, tv_of_rank(perm, lab, K), ev);
            }
        } else {
            const int src = 4 * J.a;
            eval_f64<true>(on, K, [&](int r, int d) { return from_lane(src, v[r][d]); }, sum, W.ga[J.g][J.a], D, perm,
                           W.lab[J.g][J.a], ev);
        }
        if (on) {
            W.r[lane] = (double)ev.r;
            for (int e = 0; e < 4; e++) W.qs[e][lane] = ev.q[e];
            W.qs[4][lane] = ev.s;
            if constexpr (sizeof(RT) == 4) {
                W.d2[lane] = ev.c;
                W.cand[lane] = J.k;
            } else {
                W.cand[lane] = J.cand;
            }
        }
        J = next;
        wave_lds_sync();
        if (mine > 0) {
            // this atom's jobs of the chunk, in order (group, then
            // candidate); strict comparisons: ties go to the earlier job
            const int lo = max(my_off, c0), hi = min(my_off + mine, c0 + 64);
            int bt = -1;
            if constexpr (sizeof(RT) == 4) {
                for (int t = lo; t < hi; t++) {
                    const double r = W.r[t - c0], b = rmsd_f32_bound(r, (double)W.d2[t - c0]);
                    if (r < m1) {
                        lo2 = fmin(lo2, m1 - b1);  // the previous winner joins the others
                        b1 = b;
                        m2 = m1;
                        m1 = r;
                        bt = t;
                    } else {
                        if (r < m2) m2 = r;
                        lo2 = fmin(lo2, r - b);
                    }
                }
            } else {
                for (int t = lo; t < hi; t += 4) {  // four on the way at a time
                    double r[4];
                    for (int e = 0; e < 4; e++) r[e] = W.r[(t + e) & 63];
                    for (int e = 0; e < 4; e++) {
                        const double x = t + e < hi ? r[e] : INFINITY;
                        if (x < m1) {
                            m2 = m1;
                            m1 = x;
                            bt = t + e;
                        } else if (x < m2) {
                            m2 = x;
                        }
                    }
                }
            }
            if (bt >= 0) {  // the best job so far is one of this chunk's
                const int jj = bt - my_off, u = bt - c0;
                arg_g = jj < cnt[0] ? 0 : (jj < cnt[0] + cnt[1] ? 1 : 2);
                arg_c = W.cand[u];
                for (int e = 0; e < 5; e++) wq[e] = W.qs[e][u];
            }
        }
        wave_lds_sync();
    }

    // C. decision.  The common case -- a unique winner by more than the tie
    // tolerance (FP32 form: by more than the two candidates' error bounds,
    // and clear of the cut-off by the winner's) -- is finished below in the
    // working precision; the others take the full rule.
    bool full = false;
    int cls = -1;  // hull group of the winner to finish below, -1 for none
    if (live) {
        full = arg_g >= 0 && (force_full || !(m2 > m1 + 1e-12));
        if constexpr (sizeof(RT) == 4) {
            if (arg_g >= 0) full = full || !(lo2 - (m1 + b1) > 1e-12) || fabs(m1 - cutoff) <= b1;
        } else {
            // RMSDs from the moments carry up to 2e-13 each: near ties and
            // the cut-off get that much room (the full rule uses explicit
            // residuals)
            if (arg_g >= 0) full = full || !(m2 > m1 + 2e-12) || fabs(m1 - cutoff) <= 1e-12;
        }
        if (!full) {
            if (arg_g < 0) {
                write_none(O, sid[p]);
            } else {
                cls = arg_g;
            }
        }
    }
    uint64_t fb = __ballot(full);
    if (lane == 0 && fb) atomicAdd(full_count, (int32_t)__popcll(fb));
    while (fb) {
        const int a = __builtin_ctzll(fb);
        fb &= fb - 1;
        full_rule(M, Tl, n, wbase + a, nbr_rel, nbr_id, sid, species, code, labs, mask, cutoff, Ol);
    }

    // every lane finishes its own winner, whatever its hull size
    if (cls >= 0) {
        const int32_t iw = sid[p];
        uint64_t lab;
        Candidate cd;
        if constexpr (sizeof(RT) == 4) {
            lab = labs[(int64_t)cls * n + p];
            cd = group_candidates(T, cls)[arg_c];
        } else {
            lab = W.lab[cls][lane];
            cd.perm = arg_c & ((1ull << 56) - 1);
            cd.tmpl = (int32_t)(arg_c >> 56);
        }
        CandEval<RT> ev;
        ev.r = (RT)m1;
        for (int e = 0; e < 4; e++) ev.q[e] = wq[e];
        ev.s = wq[4];
        const int K = group_k(cls);
        const double sum[3] = {W.sum[cls][0][lane], W.sum[cls][1][lane], W.sum[cls][2][lane]};
        if constexpr (sizeof(RT) == 4)
            finish_f32(K, M, T, cd, lab, ev, sum, nbr_rel, cutoff, p, n, iw, nbr_id, species, O);
        else
            finish_f64(K, M, T, cd, lab, ev, v, sum, cutoff, p, n, iw, nbr_id, species, O);
    }
}

// The match kernel: blocks of four waves, 256 atoms each.  FP64: two blocks
// per CU (256 VGPRs, 84 of them an atom's points); FP32: four (128 VGPRs at
// most, the spills only around the rare full-rule call).
template <typename RT>
__global__ void __launch_bounds__(MB, sizeof(RT) == 4 ? 4 : 2) k_match(int64_t n, const double *__restrict__ nbr_rel,
                                                const int32_t *__restrict__ nbr_id, const int32_t *__restrict__ sid,
                                                const int8_t *__restrict__ species, TablesView T,
                                                const int32_t *__restrict__ code, const uint64_t *__restrict__ labs,
                                                uint32_t mask, double cutoff, int force_full, MatchOut O,
                                                int32_t *__restrict__ full_count,
                                                unsigned long long *__restrict__ job_count,
                                                const int32_t *__restrict__ knn_src, int32_t *__restrict__ knn_out,
                                                const int32_t *__restrict__ box_fail, int apw, int32_t *host_flag) {
    __shared__ MatchLds<RT, MB / 64> L;
    if (host_flag && blockIdx.x == 0 && threadIdx.x == 0)
        __hip_atomic_store(host_flag, *box_fail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (*box_fail) return;  // uniform over the grid
    if (threadIdx.x == 0) {
        L.T = T;
        L.O = O;
    }
    load_templates(L.M, T);
    match_block<RT, MB / 64>(L.M, L.T, L.O, L.work, (int64_t)blockIdx.x * (MB / 64) * apw, n, nbr_rel, nbr_id, sid, species, T,
                             code, labs, mask, cutoff, force_full, O, full_count, job_count, knn_src, knn_out,
                             apw);
}

// ------------------------------------------------- post-hoc cut-off (Sec. 5.1)
// Both kernels are HBM streams.  Lanes take eight atoms each (one 8-byte
// load of types, four 16-byte loads of RMSDs) when the arrays are aligned
// for it; atoms past the last full group of eight, or misaligned arrays, go
// one per lane.
__device__ inline int8_t cut_one(int8_t t, double r, double cutoff) { return r <= cutoff ? t : (int8_t)0; }

__global__ void __launch_bounds__(256) k_apply_cutoff(int64_t n, int64_t n8, const int8_t *__restrict__ best_type,
                                                      const double *__restrict__ rmsd, double cutoff,
                                                      int8_t *__restrict__ type) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; g < n8; g += stride) {
        const uint64_t t8 = ((const uint64_t *)best_type)[g];
        const double2 *r2 = (const double2 *)rmsd + 4 * g;
        uint64_t o = 0;
#pragma unroll
        for (int h = 0; h < 4; h++) {
            const double2 r = r2[h];
            o |= (uint64_t)(uint8_t)cut_one((int8_t)(t8 >> (16 * h)), r.x, cutoff) << (16 * h);
            o |= (uint64_t)(uint8_t)cut_one((int8_t)(t8 >> (16 * h + 8)), r.y, cutoff) << (16 * h + 8);
        }
        ((uint64_t *)type)[g] = o;
    }
    for (int64_t i = 8 * n8 + blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += stride)
        type[i] = cut_one(best_type[i], rmsd[i], cutoff);
}

// per-type histograms: a block-private copy in LDS (when 6 * nbins fits),
// then one atomic add per non-zero bin into the global counts
constexpr int HIST_LDS_BINS = 6 * 1024;
__device__ inline void hist_add(unsigned int *h, unsigned long long *counts, bool lds, int t, double r, int nbins,
                                double rmax, double inv) {
    if (t < 0 || t > 5) return;
    int b = nbins - 1;
    if (r < rmax) b = min(nbins - 1, max(0, (int)(r * inv)));
    if (lds) atomicAdd(&h[t * nbins + b], 1u);
    else atomicAdd(&counts[t * nbins + b], 1ull);
}

__global__ void __launch_bounds__(256) k_rmsd_histogram(int64_t n, int64_t n8, const int8_t *__restrict__ best_type,
                                                        const double *__restrict__ rmsd, int nbins, double rmax,
                                                        double inv, unsigned long long *__restrict__ counts) {
    __shared__ unsigned int h[HIST_LDS_BINS];
    const bool lds = 6 * nbins <= HIST_LDS_BINS;
    if (lds)
        for (int b = threadIdx.x; b < 6 * nbins; b += blockDim.x) h[b] = 0;
    __syncthreads();
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; g < n8; g += stride) {
        const uint64_t t8 = ((const uint64_t *)best_type)[g];
        const double2 *r2 = (const double2 *)rmsd + 4 * g;
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const double2 r = r2[q];
            hist_add(h, counts, lds, (int8_t)(t8 >> (16 * q)), r.x, nbins, rmax, inv);
            hist_add(h, counts, lds, (int8_t)(t8 >> (16 * q + 8)), r.y, nbins, rmax, inv);
        }
    }
    for (int64_t i = 8 * n8 + blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += stride)
        hist_add(h, counts, lds, best_type[i], rmsd[i], nbins, rmax, inv);
    __syncthreads();
    if (lds)
        for (int b = threadIdx.x; b < 6 * nbins; b += blockDim.x)
            if (h[b]) atomicAdd(&counts[b], (unsigned long long)h[b]);
}

// groups of eight atoms a lane can load as one 8-byte word of types and four
// 16-byte words of RMSDs (0 if the arrays are not aligned for that)
static int64_t groups_of_eight(int64_t n, const void *t, const void *r, const void *out) {
    const bool ok = ((uintptr_t)t % 8 == 0) && ((uintptr_t)r % 16 == 0) && (!out || (uintptr_t)out % 8 == 0);
    return ok ? n / 8 : 0;
}
static unsigned stream_blocks(int64_t n) {
    // about eight resident blocks per CU of 256 lanes, each lane striding
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 256 * 8));
}

void launch_apply_cutoff(int64_t n, const int8_t *best_type, const double *rmsd, double cutoff, int8_t *type,
                         hipStream_t st) {
    const int64_t n8 = groups_of_eight(n, best_type, rmsd, type);
    hipLaunchKernelGGL(k_apply_cutoff, dim3(stream_blocks(n8 > 0 ? n8 : n)), dim3(256), 0, st, n, n8, best_type, rmsd,
                       cutoff, type);
}
void launch_rmsd_histogram(int64_t n, const int8_t *best_type, const double *rmsd, int nbins, double rmax,
                           unsigned long long *counts, hipStream_t st) {
    const int64_t n8 = groups_of_eight(n, best_type, rmsd, nullptr);
    const int64_t blocks = std::min<int64_t>((n + 255) / 256, 1024);
    const double inv = (double)nbins / rmax;  // the bin of r is floor(r * inv), inv rounded once on the host
    hipLaunchKernelGGL(k_rmsd_histogram, dim3((unsigned)std::max<int64_t>(blocks, 1)), dim3(256), 0, st, n, n8,
                       best_type, rmsd, nbins, rmax, inv, counts);
}

// ------------------------------------------------------- misorientation
// Sec. 7: smallest rotation angle of conj(q1) q2 q_h over the template's
// proper rotations (identity only for type NONE), as 2 atan2(|v|, |w|) of
// the best product, which stays accurate near zero.  Invalid types give NaN.
// Blocks stride over the pairs, 256 at a time.  A wave of mixed types would
// scan the longest list among its lanes, so the pairs of a round are regrouped
// by type (wave ballots give each its slot): the lanes load their pairs in
// order and form the products m, which change places through LDS with the
// angles on the way back, so every access of global memory is in order.
// Bound by HBM: 16.8 M pairs of 73 bytes take 291 us, 253 at the rate of a
// large copy; 434 us when whole groups (24 elements, 60 for ICO) were scanned,
// the pairs loaded in slot order and the tables staged for every 256 pairs.
template <bool Vec>
__global__ void __launch_bounds__(256) k_misorientation(int64_t n, TablesView T, const int8_t *__restrict__ type,
                                                        const double *__restrict__ q1, const double *__restrict__ q2,
                                                        double *__restrict__ angle) {
    // products and sums may fuse into FMAs here (one rounding instead of two; no
    // result depends on a particular rounding)
#pragma clang fp contract(fast)
    constexpr int NCLS = NT + 2;  // types 0..NT, then invalid
    __shared__ double4 G[NT][SCAN_MAX];  // lanes of one type read the same word (a broadcast)
    __shared__ int rows[NT + 1], any_sign[NT + 1];
    __shared__ int32_t s_cnt[4][NCLS];
    __shared__ double s_m[4][256], s_angle[256];
    __shared__ uint16_t s_who[256];  // thread | class << 8 of the pair in a slot
    for (int w = threadIdx.x; w < NT * SCAN_MAX; w += blockDim.x) {
        const double *g = T.tpl[w / SCAN_MAX].scan[w % SCAN_MAX];
        G[w / SCAN_MAX][w % SCAN_MAX] = make_double4(g[0], g[1], g[2], g[3]);
    }
    if (threadIdx.x <= NT) {
        rows[threadIdx.x] = threadIdx.x ? T.tpl[threadIdx.x - 1].nscan : 0;
        any_sign[threadIdx.x] = threadIdx.x ? T.tpl[threadIdx.x - 1].all_signs : 0;
    }
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int64_t rounds = (n + 255) / 256;
    for (int64_t round = blockIdx.x; round < rounds; round += gridDim.x) {
        const int64_t i = round * 256 + tid;
        int cls = -1;
        double m0 = 0, m1 = 0, m2 = 0, m3 = 0;
        if (i < n) {
            const int t = type[i];
            double a0, a1, a2, a3, b0, b1, b2, b3;
            if (Vec) {  // 16-byte aligned quaternion arrays
                const double2 *p1 = (const double2 *)(q1 + 4 * i), *p2 = (const double2 *)(q2 + 4 * i);
                const double2 u0 = p1[0], u1 = p1[1], v0 = p2[0], v1 = p2[1];
                a0 = u0.x, a1 = -u0.y, a2 = -u1.x, a3 = -u1.y;  // conj(q1)
                b0 = v0.x, b1 = v0.y, b2 = v1.x, b3 = v1.y;
            } else {
                a0 = q1[4 * i], a1 = -q1[4 * i + 1], a2 = -q1[4 * i + 2], a3 = -q1[4 * i + 3];
                b0 = q2[4 * i], b1 = q2[4 * i + 1], b2 = q2[4 * i + 2], b3 = q2[4 * i + 3];
            }
            cls = (t < 0 || t > NT) ? NT + 1 : t;
            m0 = a0 * b0 - a1 * b1 - a2 * b2 - a3 * b3, m1 = a0 * b1 + a1 * b0 + a2 * b3 - a3 * b2;
            m2 = a0 * b2 - a1 * b3 + a2 * b0 + a3 * b1, m3 = a0 * b3 + a1 * b2 - a2 * b1 + a3 * b0;
        }
        uint64_t bal[NCLS];
#pragma unroll
        for (int k = 0; k < NCLS; k++) bal[k] = __ballot(cls == k);
        if (lane == 0)
            for (int k = 0; k < NCLS; k++) s_cnt[wv][k] = __popcll(bal[k]);
        __syncthreads();
        int total = 0, slot = 0;
#pragma unroll
        for (int k = 0; k < NCLS; k++) {
            int before = 0, tk = 0;
            for (int w2 = 0; w2 < 4; w2++) {
                tk += s_cnt[w2][k];
                if (w2 < wv) before += s_cnt[w2][k];
            }
            if (k == cls) slot = total + before + __popcll(bal[k] & ((1ull << lane) - 1));
            total += tk;
        }
        if (cls >= 0) {
            s_m[0][slot] = m0;
            s_m[1][slot] = m1;
            s_m[2][slot] = m2;
            s_m[3][slot] = m3;
            s_who[slot] = (uint16_t)(tid | cls << 8);
        }
        __syncthreads();
        if (tid < total) {
            const int who = s_who[tid] & 0xFF, ty = s_who[tid] >> 8;
            m0 = s_m[0][tid], m1 = s_m[1][tid], m2 = s_m[2][tid], m3 = s_m[3][tid];
            double a = NAN;
            if (ty <= NT) {
                // the w of m q_h is a dot product: scan for the largest |w|,
                // then form the vector part of that one product only
                const bool moduli = any_sign[ty];
                const double x0 = moduli ? fabs(m0) : m0, x1 = moduli ? fabs(m1) : m1;
                const double x2 = moduli ? fabs(m2) : m2, x3 = moduli ? fabs(m3) : m3;
                double bw = fabs(m0);
                int best = -1;
                for (int h = 0; h < rows[ty]; h++) {
                    const double4 g = G[ty - 1][h];
                    const double c0 = fabs(x0 * g.x + x1 * g.y + x2 * g.z + x3 * g.w);
                    if (c0 > bw) {
                        bw = c0;
                        best = h;
                    }
                }
                double c1 = m1, c2 = m2, c3 = m3;
                if (best >= 0) {
                    double4 g = G[ty - 1][best];
                    if (moduli)
                        g = make_double4(copysign(g.x, m0), copysign(g.y, m1), copysign(g.z, m2), copysign(g.w, m3));
                    g.y = -g.y, g.z = -g.z, g.w = -g.w;
                    c1 = m0 * g.y + m1 * g.x + m2 * g.w - m3 * g.z;
                    c2 = m0 * g.z - m1 * g.w + m2 * g.x + m3 * g.y;
                    c3 = m0 * g.w + m1 * g.z - m2 * g.y + m3 * g.x;
                }
                a = 2.0 * atan2(sqrt(c1 * c1 + c2 * c2 + c3 * c3), bw);
            }
            s_angle[who] = a;
        }
        __syncthreads();
        if (i < n) angle[i] = s_angle[tid];
    }
}

void launch_misorientation(int64_t n, const TablesView &T, const int8_t *type, const double *q1, const double *q2,
                           double *angle, hipStream_t st) {
    const dim3 grid(stream_blocks(n));
    if ((uintptr_t)q1 % 16 == 0 && (uintptr_t)q2 % 16 == 0)
        hipLaunchKernelGGL(k_misorientation<true>, grid, dim3(256), 0, st, n, T, type, q1, q2, angle);
    else
        hipLaunchKernelGGL(k_misorientation<false>, grid, dim3(256), 0, st, n, T, type, q1, q2, angle);
}

// ------------------------------------------------------------- self-check
// The strain of one match on the device, as the decision kernels compute it
// (strain_inputs, polar_p) in the working precision: K relative vectors rel
// ([K][3], template-vertex order), template t; P[9] row-major.
template <int K, typename RT>
__global__ void k_selftest_strain(const TemplateDev *__restrict__ tpl, int t, const double *__restrict__ rel,
                                  double *__restrict__ P) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    const TemplateDev &D = tpl[t];
    double v[K][3];
    uint64_t tv = 0;
    for (int r = 0; r < K; r++) {
        for (int d = 0; d < 3; d++) v[r][d] = rel[3 * r + d];
        tv |= (uint64_t)r << (4 * r);
    }
    RT a0[3], At[3][3], l, Pm[3][3];
    strain_inputs<K, RT>(D, tv, v, a0, At, l);
    polar_p<RT>(At, l, Pm);
    for (int x = 0; x < 3; x++)
        for (int y = 0; y < 3; y++) P[3 * x + y] = (double)Pm[x][y];
}

template <typename RT>
static void launch_selftest_strain_rt(const TablesView &T, int t, const double *rel, double *P, hipStream_t st) {
    const int k = template_k(t);
    if (k == 6) hipLaunchKernelGGL((k_selftest_strain<6, RT>), dim3(1), dim3(64), 0, st, T.tpl, t, rel, P);
    else if (k == 12) hipLaunchKernelGGL((k_selftest_strain<12, RT>), dim3(1), dim3(64), 0, st, T.tpl, t, rel, P);
    else hipLaunchKernelGGL((k_selftest_strain<14, RT>), dim3(1), dim3(64), 0, st, T.tpl, t, rel, P);
}
void launch_selftest_strain(const TablesView &T, int t, bool f32, const double *rel, double *P, hipStream_t st) {
    if (f32) launch_selftest_strain_rt<float>(T, t, rel, P, st);
    else launch_selftest_strain_rt<double>(T, t, rel, P, st);
}

// --------------------------------------------------------------- launches
// zero n int32 words (a kernel rather than a memset node, so that a captured
// stream replays it faithfully)
__global__ void k_fill_zero(int32_t *__restrict__ p, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}
void launch_zero(int32_t *p, int64_t n, hipStream_t st) {
    const int64_t blocks = std::min<int64_t>((n + 255) / 256, 4096);
    hipLaunchKernelGGL(k_fill_zero, dim3((unsigned)std::max<int64_t>(blocks, 1)), dim3(256), 0, st, p, n);
}
void launch_bounds(const double *pos, int64_t n, double *part, int nblocks, hipStream_t st) {
    hipLaunchKernelGGL(k_bounds, dim3(nblocks), dim3(256), 0, st, pos, n, part);
}
void launch_bounds_grid(const double *pos, int64_t n, const double *box, int kn, int32_t *count, int64_t cells,
                        double *part, int nblocks, GridState *G, int32_t *box_fail, hipStream_t st) {
    hipLaunchKernelGGL(k_bounds_grid, dim3(nblocks), dim3(256), 0, st, pos, n, box[0], box[1], box[2], kn, count,
                       cells, part, G, box_fail);
}
void launch_setup_small(const double *pos, int64_t n, const double *box, int kn, GridState *G, int32_t *count,
                        int64_t cells_max, int32_t *cell_of, int32_t *slot_of, int32_t *start, double *spos,
                        int4 *sfix, int32_t *sid, int32_t *box_fail, hipStream_t st) {
    hipLaunchKernelGGL(k_setup_small, dim3(1), dim3(SETUP_THREADS), 0, st, pos, n, box[0], box[1], box[2], kn, G,
                       count, cells_max, cell_of, slot_of, start, spos, sfix, sid, box_fail);
}
void launch_bin_count(const double *pos, int64_t n, const GridArg &A, int32_t *cell_of, int32_t *slot_of,
                      int32_t *count, const int32_t *box_fail, hipStream_t st) {
    hipLaunchKernelGGL(k_bin_count, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, pos, n, A, cell_of, slot_of,
                       count, box_fail);
}
void launch_cell_starts(const int32_t *count, int64_t cells, const GridArg &A, int32_t *bsum, int32_t *start,
                        hipStream_t st) {
    const int64_t items = scan_items(cells);
    hipLaunchKernelGGL(k_scan_totals, dim3((unsigned)items), dim3(SCAN_THREADS), 0, st, count, cells, A, bsum);
    // up to 4096 items (8 M cells) a block adds up at most 16 totals per
    // thread itself: less than a launch
    if (items > 4096) {
        hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(1024), 0, st, bsum, items);
        hipLaunchKernelGGL(k_scan_cells<true>, dim3((unsigned)items), dim3(SCAN_THREADS), 0, st, count, cells, A,
                           (const int32_t *)bsum, start);
    } else {
        hipLaunchKernelGGL(k_scan_cells<false>, dim3((unsigned)items), dim3(SCAN_THREADS), 0, st, count, cells, A,
                           (const int32_t *)bsum, start);
    }
}
void launch_bin_scatter(const double *pos, int64_t n, const GridArg &A, const int32_t *cell_of, const int32_t *slot_of,
                        const int32_t *start, double *spos, int4 *sfix, int32_t *sid, const int32_t *box_fail,
                        hipStream_t st) {
    hipLaunchKernelGGL(k_bin_scatter, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, pos, n, A, cell_of,
                       slot_of, start, spos, sfix, sid, box_fail);
}
// Atoms per wave of the match kernel.  A wave pays for the longest of its
// lanes in every loop, so while the chip has SIMDs without a wave the atoms
// are spread over more of them.
static int match_atoms_per_wave(int64_t n) {
    int apw = 1;
    while (apw < 64 && n > (int64_t)apw * 1024) apw *= 2;
    return apw;
}
bool knn_fast_applies(int64_t n, const Grid &g) {
    if (n <= KNN_WAVE_ATOMS) return false;
    for (int a = 0; a < 3; a++)
        if (g.periodic[a] && g.nc[a] < 5) return false;
    return true;
}
template <int NK>
static void launch_knn_nk(int64_t n, const GridArg &A, const double *spos, const int4 *sfix,
                          const int32_t *sid, const int32_t *start, int32_t *nbr_id, double *nbr_rel,
                          int32_t *todo, int32_t *todo_count, int32_t *box_fail, hipStream_t st) {
    int64_t blocks = (n + 255) / 256;
    // up to KNN_WAVE_ATOMS atoms, a wave each: the chip holds 4096 such waves,
    // and one takes a fraction of the time of a lane's walk through its block
    if (A.dev ? n > KNN_WAVE_ATOMS : knn_fast_applies(n, A.val)) {
        hipLaunchKernelGGL(k_knn_fast<NK>, dim3((unsigned)xcd_pad(blocks)), dim3(256), 0, st, n, A, spos, sfix,
                           start, nbr_id, nbr_rel, todo, todo_count, box_fail);
        // the atoms left over are few; at most 1024 blocks of four waves stride over them
        hipLaunchKernelGGL(k_knn_exact<NK>, dim3((unsigned)std::min<int64_t>((n + 15) / 16, 1024)), dim3(256), 0, st, n, A,
                           spos, sid, start, nbr_id, nbr_rel, (const int32_t *)todo,
                           (const int32_t *)todo_count, box_fail);
    } else {
        hipLaunchKernelGGL(k_knn_exact<NK>, dim3((unsigned)std::min<int64_t>((n + 3) / 4, 16384)), dim3(256), 0, st, n,
                           A, spos, sid, start, nbr_id, nbr_rel, (const int32_t *)nullptr,
                           (const int32_t *)nullptr, box_fail);
    }
}
void launch_knn(int64_t n, const GridArg &A, int nk, const double *spos, const int4 *sfix,
                const int32_t *sid, const int32_t *start, int32_t *nbr_id, double *nbr_rel, int32_t *todo,
                int32_t *todo_count, int32_t *box_fail, hipStream_t st) {
    if (nk == VK)
        launch_knn_nk<VK>(n, A, spos, sfix, sid, start, nbr_id, nbr_rel, todo, todo_count, box_fail, st);
    else
        launch_knn_nk<KMAX>(n, A, spos, sfix, sid, start, nbr_id, nbr_rel, todo, todo_count, box_fail, st);
}
void launch_voronoi(int64_t n, const double *rel18, const int32_t *id18, uint32_t *vf, uint32_t *vlive,
                    double *nbr_rel, int32_t *nbr_id, const int32_t *box_fail, hipStream_t st) {
    const unsigned grid = (unsigned)xcd_pad((n + VB - 1) / VB);
    hipLaunchKernelGGL(k_voronoi_hull, dim3(grid), dim3(VB), 0, st, n, rel18, id18, vf, vlive, box_fail);
    hipLaunchKernelGGL(k_voronoi_order, dim3(grid), dim3(VB), 0, st, n, rel18, id18, (const uint32_t *)vf,
                       (const uint32_t *)vlive, nbr_rel, nbr_id, box_fail);
}
// Both precision forms use the FP32-storage hull kernel: every predicate is
// exact (a filter on the FP32 copies decides only when its bound proves the
// sign of the predicate on the FP64 inputs, otherwise the FP64 filter and
// the exact path run on the originals), so the hulls, codes and labellings
// are those of the FP64 kernel, with half the LDS per lane.
void launch_topo(int64_t n, const double *nbr_rel, const int32_t *nbr_id, const TablesView &T, uint32_t need,
                 int32_t *code, uint64_t *ord, const int32_t *box_fail, hipStream_t st) {
    dim3 grid((unsigned)((n + TB - 1) / TB)), block(TB);
    hipLaunchKernelGGL(k_topo, grid, block, 0, st, n, nbr_rel, nbr_id, T, need, code, ord, box_fail);
}
// ======================================== serving: one persistent kernel
// Every frame runs as nine stages of work items; the last item of a stage
// queues the next one (so stages of one frame follow each other, stages of
// different frames overlap).  A workgroup is one wave: it claims the item at
// the front of the device queue (an atomic range counter per (frame, stage)
// entry), runs it and counts it done.  Idle waves pull new frames from the
// pinned host block (one at a time, under a try-lock) and exit after a
// stretch of the device wall clock without work, or when the host sets
// stop: no wave waits on another, so every wave reaches an exit.
enum {
    PH_BOUNDS = 0,   // per-item bounds and non-finite flag
    PH_GRID = 1,     // one item: the grid from the bounds
    PH_ZERO = 2,     // cell counters and frame counters to zero
    PH_COUNT = 3,    // cell of every atom, slot in its cell (atomic counts)
    PH_SCAN = 4,     // exclusive scan of the counts within each item, item totals
    PH_SCANTOP = 5,  // one item: exclusive scan of the item totals
    PH_SCATTER = 6,  // final cell starts (into the count array) and the sorted copy
    PH_KNN = 7,      // neighbours (fast search, exact search for what it leaves)
    PH_MATCH = 8     // hulls and codes, then the match stage, 64 atoms at a time
};

__device__ inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// queue entry: slot (16 bits), stage (8), generation (40)
__device__ inline unsigned long long serve_entry(int slot, int ph, unsigned long long gen) {
    return (unsigned long long)slot | ((unsigned long long)ph << 16) | (gen << 24);
}

// a stage's claim counter: the frame's generation (36 bits) over a 28-bit item index
constexpr int SERVE_IDX_BITS = 28;
constexpr unsigned long long SERVE_IDX_MASK = (1ull << SERVE_IDX_BITS) - 1;
__device__ inline unsigned long long serve_counter(unsigned long long gen) { return gen << SERVE_IDX_BITS; }

// append (slot, stage); the stage's item count and counter are set before
// (one lane)
__device__ inline void serve_push(ServeDev *dev, int slot, int ph, unsigned long long gen) {
    const unsigned long long pos = atomicAdd(&dev->tail, 1ull);
    dev->entry[pos % SERVE_FIFO] = serve_entry(slot, ph, gen);
    __threadfence();
    __hip_atomic_store(&dev->seq[pos % SERVE_FIFO], pos + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

// the frame is finished: status, completion time, generation (one lane)
__device__ inline void serve_complete(ServeHost *host, int slot, unsigned long long gen, int status) {
    __threadfence_system();
    __hip_atomic_store(&host->status[slot], status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&host->t_done[slot], (long long)wall_clock64(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&host->done[slot], gen, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// exclusive scan over the wave
__device__ inline long long wave_excl_scan(long long v, long long &total) {
    const int lane = threadIdx.x & 63;
    long long x = v;
    for (int d = 1; d < 64; d <<= 1) {
        const long long y = __shfl_up(x, d);
        if (lane >= d) x += y;
    }
    total = __shfl(x, 63);
    return x - v;
}

template <typename RT>
union ServeWork {
    KnnRanges<64> ranges;
    KnnWave knn;
    TopoShared topo;
    MatchWork<RT, 1> mw;
};

// k-NN stage item: the fast search lane by lane, the exact one for what it
// leaves, a wave per atom (a call of its own: its registers apart; its LDS as
// LDS pointers, see serve_match)
__device__ __noinline__ void serve_knn(__attribute__((address_space(3))) KnnRanges<64> *Rp,
                                       __attribute__((address_space(3))) KnnWave *Wp, ServeSlot &S, int64_t r) {
    const int lane = threadIdx.x & 63;
    // the grid and the arrays in registers: the searches' stores cannot
    // alias them
    const Grid g = S.g;
    const int64_t n = S.r.n;
    const bool fast = S.fast;
    const double *spos = S.r.spos;
    const int4 *sfix = S.r.sfix;
    const int32_t *sid = S.r.sid, *start = S.r.count;
    int32_t *nbr_id = S.r.nbr_id;
    double *nbr_rel = S.r.nbr_rel;
    int32_t *box_fail = S.r.count + S.cells + 3;
    const int64_t b = r * SERVE_ATOMS, e = min(n, b + SERVE_ATOMS);
    for (int64_t sub = b; sub < e; sub += 64) {
        const int64_t p = sub + lane;
        bool ok = true;
        if (p < e)
            ok = fast && knn_fast_atom<KMAX, 64>(*(KnnRanges<64> *)Rp, lane, p, n, g, spos, sfix, start, nbr_id,
                                                 nbr_rel, box_fail);
        wave_lds_sync();  // the two searches share their LDS
        uint64_t left = __ballot(!ok);
        while (left) {
            const int l = __builtin_ctzll(left);
            left &= left - 1;
            knn_exact_atom<KMAX>(*(KnnWave *)Wp, sub + l, n, g, spos, sid, start, nbr_id, nbr_rel, box_fail);
        }
    }
}

// hulls + match stage item, 64 atoms at a time (a call of its own)
// The LDS objects (templates, table view, outputs, working space) come as
// LDS-space pointers: a call's reference parameters are generic, and
// generic accesses to LDS are slower flat instructions; the generic views
// below derive from the LDS pointers, so the compiler turns their accesses
// back into LDS instructions.
// The hulls of one atom per lane, in a call of their own: its registers
// apart from the match's (LDS operands passed as LDS pointers)
__device__ __noinline__ void serve_topo(__attribute__((address_space(3))) TopoShared *Sp,
                                        __attribute__((address_space(3))) TablesView *Tp, int lane, int64_t p,
                                        int64_t n, const double *nbr_rel, const int32_t *nbr_id, uint32_t need,
                                        int32_t *code, uint64_t *ord) {
    topo_atom(*(TopoShared *)Sp, lane, p, n, nbr_rel, nbr_id, *(const TablesView *)Tp, need, code, ord);
}

template <typename RT>
__device__ __noinline__ void serve_match(__attribute__((address_space(3))) MatchShared *Mp,
                                         __attribute__((address_space(3))) TablesView *Tp,
                                         __attribute__((address_space(3))) MatchOut *Op,
                                         __attribute__((address_space(3))) ServeWork<RT> *Up, ServeSlot &S,
                                         int64_t r) {
    const MatchShared &M = *(const MatchShared *)Mp;
    const TablesView &T = *(const TablesView *)Tp;
    MatchOut &Ol = *(MatchOut *)Op;
    ServeWork<RT> &U = *(ServeWork<RT> *)Up;
    const int lane = threadIdx.x & 63;
    // the frame's parameters in registers (the stages' stores cannot alias them)
    const int64_t n = S.r.n, cells = S.cells;
    const double *nbr_rel = S.r.nbr_rel;
    const int32_t *nbr_id = S.r.nbr_id, *sid = S.r.sid;
    const int8_t *species = S.r.species;
    int32_t *code = S.r.code;
    uint64_t *ord = S.r.ord;
    int32_t *count = S.r.count, *knn_out = S.r.knn_out;
    const uint32_t mask = S.r.mask, need = S.r.need;
    const double cutoff = S.r.cutoff;
    const int64_t b = r * SERVE_ATOMS, e = min(n, b + SERVE_ATOMS);
    if (lane == 0) Ol = S.r.O;
    int32_t *full_count = count + cells + 2;
    unsigned long long *job_count = job_counter(count, cells);
    for (int64_t sub = b; sub < e; sub += 64) {
        const int64_t p = sub + lane;
        __syncthreads();  // the previous sub-block's match LDS is free; Ol is written
        if (p < e) serve_topo(&Up->topo, Tp, lane, p, n, nbr_rel, nbr_id, need, code, ord);
        // the wave's code / ord writes before other lanes read them
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
        __syncthreads();
        match_block<RT, 1>(M, T, Ol, U.mw, sub, n, nbr_rel, nbr_id, sid, species, T, code, ord, mask, cutoff, 0,
                           Ol, full_count, job_count, nbr_id, knn_out, 64);
    }
}

// Stage ph, item r of the frame in slot S (the whole wave).  Returns the
// stage's status for its last item (see serve_advance).
template <typename RT>
__device__ void serve_item(const MatchShared &M, const TablesView &Tl, MatchOut &Ol, ServeWork<RT> &U,
                           const TablesView &T, ServeSlot &S, int ph, int64_t r) {
    const int lane = threadIdx.x & 63;
    const ServeRequest &R = S.r;
    const int64_t n = R.n;
    if (ph == PH_BOUNDS) {
        const int64_t b = r * SERVE_ATOMS_LIGHT, e = min(n, b + SERVE_ATOMS_LIGHT);
        double mn[3] = {1e308, 1e308, 1e308}, mx[3] = {-1e308, -1e308, -1e308};
        int bad = 0;
        for (int64_t i = b + lane; i < e; i += 64)
            for (int d = 0; d < 3; d++) {
                const double x = R.pos[3 * i + d];
                if (!isfinite(x)) bad = 1;
                mn[d] = fmin(mn[d], x);
                mx[d] = fmax(mx[d], x);
            }
        for (int off = 32; off > 0; off >>= 1) {
            for (int d = 0; d < 3; d++) {
                mn[d] = fmin(mn[d], __shfl_xor(mn[d], off));
                mx[d] = fmax(mx[d], __shfl_xor(mx[d], off));
            }
            bad |= __shfl_xor(bad, off);
        }
        if (lane == 0) {
            double *o = R.part + 7 * r;
            for (int d = 0; d < 3; d++) {
                o[d] = mn[d];
                o[3 + d] = mx[d];
            }
            o[6] = (double)bad;
        }
    } else if (ph == PH_GRID) {
        const int64_t nb = S.nr[PH_BOUNDS];
        double mn[3] = {1e308, 1e308, 1e308}, mx[3] = {-1e308, -1e308, -1e308};
        int bad = 0;
        for (int64_t k = lane; k < nb; k += 64) {
            const double *o = R.part + 7 * k;
            for (int d = 0; d < 3; d++) {
                mn[d] = fmin(mn[d], o[d]);
                mx[d] = fmax(mx[d], o[3 + d]);
            }
            bad |= o[6] != 0.0;
        }
        for (int off = 32; off > 0; off >>= 1) {
            for (int d = 0; d < 3; d++) {
                mn[d] = fmin(mn[d], __shfl_xor(mn[d], off));
                mx[d] = fmax(mx[d], __shfl_xor(mx[d], off));
            }
            bad |= __shfl_xor(bad, off);
        }
        if (lane == 0) {
            const double box[3] = {R.box[0], R.box[1], R.box[2]};
            S.g = make_grid(box, mn, mx, n, KMAX);
            S.cells = grid_cells(S.g);
            bool fast = true;
            for (int a = 0; a < 3; a++)
                if (S.g.periodic[a] && S.g.nc[a] < 5) fast = false;
            S.fast = fast;
            // a non-finite coordinate, or more cells than the scratch has: the frame stops here
            S.bad = bad ? SERVE_NONFINITE : (S.cells > max_cells(n) ? SERVE_GRID : SERVE_OK);
        }
    } else if (ph == PH_ZERO) {
        const int64_t m = S.cells + FRAME_COUNTERS;
        const int64_t b = r * SERVE_ZERO_CELLS, e = min(m, b + SERVE_ZERO_CELLS);
        for (int64_t c = b + lane; c < e; c += 64) R.count[c] = 0;
    } else if (ph == PH_COUNT) {
        const int64_t b = r * SERVE_ATOMS_LIGHT, e = min(n, b + SERVE_ATOMS_LIGHT);
        const Grid &g = S.g;
        for (int64_t i = b + lane; i < e; i += 64) {
            const int cx = cell_coord(R.pos[3 * i + 0], g, 0);
            const int cy = cell_coord(R.pos[3 * i + 1], g, 1);
            const int cz = cell_coord(R.pos[3 * i + 2], g, 2);
            const int c = cell_row(g, cy, cz) * g.nc[0] + cx;
            R.cell_of[i] = c;
            R.slot_of[i] = atomicAdd(&R.count[c], 1);
        }
    } else if (ph == PH_SCAN) {
        // cells 0..cells (the last one counts zero: its start is the total)
        const int64_t m = S.cells + 1;
        const int64_t b = r * SERVE_SCAN_CELLS, e = min(m, b + SERVE_SCAN_CELLS);
        constexpr int64_t PER = SERVE_SCAN_CELLS / 64;
        const int64_t lb = b + lane * PER, le = min(e, lb + PER);
        long long sum = 0;
        for (int64_t c = lb; c < le; c++) sum += c < S.cells ? R.count[c] : 0;
        long long total;
        long long run = wave_excl_scan(sum, total);
        for (int64_t c = lb; c < le; c++) {
            R.start[c] = (int32_t)run;
            run += c < S.cells ? R.count[c] : 0;
        }
        if (lane == 0) R.bsum[r] = (int32_t)total;
    } else if (ph == PH_SCANTOP) {
        const int64_t m = S.nr[PH_SCAN];
        const int64_t per = ceil_div(m, 64);
        const int64_t lb = lane * per, le = min(m, lb + per);
        long long sum = 0;
        for (int64_t k = lb; k < le; k++) sum += R.bsum[k];
        long long total;
        long long run = wave_excl_scan(sum, total);
        for (int64_t k = lb; k < le; k++) {
            const int32_t v = R.bsum[k];
            R.bsum[k] = (int32_t)run;
            run += v;
        }
    } else if (ph == PH_SCATTER) {
        // final starts of this item's cells (the k-NN reads them from count)
        const int64_t m = S.cells + 1;
        const int64_t cb = r * SERVE_SCAN_CELLS, ce = min(m, cb + SERVE_SCAN_CELLS);
        if (cb < m) {
            const int32_t off = R.bsum[r];
            for (int64_t c = cb + lane; c < ce; c += 64) R.count[c] = R.start[c] + off;
        }
        const int64_t b = r * SERVE_ATOMS_LIGHT, e = min(n, b + SERVE_ATOMS_LIGHT);
        for (int64_t i = b + lane; i < e; i += 64) {
            const int32_t c = R.cell_of[i];
            const int64_t p = (int64_t)R.start[c] + R.bsum[c / SERVE_SCAN_CELLS] + R.slot_of[i];
            const double x = R.pos[3 * i + 0], y = R.pos[3 * i + 1], z = R.pos[3 * i + 2];
            R.spos[3 * (int64_t)p] = x;
            R.spos[3 * (int64_t)p + 1] = y;
            R.spos[3 * (int64_t)p + 2] = z;
            R.sfix[p] = make_int4(fixed_coord(x, S.g, 0), fixed_coord(y, S.g, 1), fixed_coord(z, S.g, 2), (int32_t)i);
            R.sid[p] = (int32_t)i;
        }
    } else if (ph == PH_KNN) {
        serve_knn((__attribute__((address_space(3))) KnnRanges<64> *)&U.ranges,
                  (__attribute__((address_space(3))) KnnWave *)&U.knn, S, r);
    } else {  // PH_MATCH
        serve_match<RT>((__attribute__((address_space(3))) MatchShared *)&M,
                        (__attribute__((address_space(3))) TablesView *)&Tl,
                        (__attribute__((address_space(3))) MatchOut *)&Ol,
                        (__attribute__((address_space(3))) ServeWork<RT> *)&U, S, r);
    }
}

// `count` items of (slot, ph) are done: the stage's last one queues the next
// stage (or completes the frame).  Whole wave; one lane acts.  A wave counts
// its items of one stage together, when it moves to another stage or runs
// out of work: the release that makes its writes visible to the other XCDs
// (a write-back of the L2) then happens once per stage, not per item.
__device__ inline void serve_advance(ServeDev *dev, ServeHost *host, int slot, int ph, unsigned long long gen,
                                     long long count) {
    const int lane = threadIdx.x & 63;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");  // these items' writes before their count
    if (lane != 0) return;
    ServeSlot &S = dev->slot[slot];
    const long long d = __hip_atomic_fetch_add(&S.done[ph], count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + count;
    if (d != S.nr[ph]) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");  // every item's writes of the stage
    int next = ph + 1;
    if (ph == PH_GRID && S.bad) {
        serve_complete(host, slot, gen, S.bad);
        return;
    }
    if (ph == PH_KNN && __hip_atomic_load(S.r.count + S.cells + 3, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
        serve_complete(host, slot, gen, SERVE_BOX);
        return;
    }
    if (ph == PH_MATCH) {
        serve_complete(host, slot, gen, SERVE_OK);
        return;
    }
    const int64_t n = S.r.n;
    long long nr = 1;
    switch (next) {
        case PH_ZERO: nr = ceil_div(S.cells + FRAME_COUNTERS, SERVE_ZERO_CELLS); break;
        case PH_COUNT: nr = ceil_div(n, SERVE_ATOMS_LIGHT); break;
        case PH_SCAN: nr = ceil_div(S.cells + 1, SERVE_SCAN_CELLS); break;
        case PH_SCANTOP: nr = 1; break;
        case PH_SCATTER: nr = max(ceil_div(S.cells + 1, SERVE_SCAN_CELLS), ceil_div(n, SERVE_ATOMS_LIGHT)); break;
        case PH_KNN: nr = ceil_div(n, SERVE_ATOMS); break;
        case PH_MATCH: nr = ceil_div(n, SERVE_ATOMS); break;
        default: nr = 1;
    }
    S.nr[next] = nr;
    S.done[next] = 0;
    __threadfence();
    __hip_atomic_store(&S.next[next], serve_counter(gen), __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    serve_push(dev, slot, next, gen);
}

// An idle wave pulls the next frame the host published, if any, and queues
// its first stage.  Returns true if it did.
__device__ inline bool serve_pull(ServeDev *dev, ServeHost *host) {
    const int lane = threadIdx.x & 63;
    int slot = -1;
    if (lane == 0 && atomicCAS(&dev->poll_lock, 0, 1) == 0) {
        const unsigned long long ht = __hip_atomic_load(&host->tail, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_SYSTEM);
        const unsigned long long pulled = __hip_atomic_load(&dev->pulled, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (pulled < ht) {
            slot = __hip_atomic_load(&host->ring[pulled % SERVE_SLOTS], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            __hip_atomic_store(&dev->pulled, pulled + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __hip_atomic_store(&dev->poll_lock, 0, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    }
    slot = __shfl(slot, 0);
    if (slot < 0) return false;
    // copy the request out of host memory, a word per lane
    ServeSlot &S = dev->slot[slot];
    constexpr int WORDS = sizeof(ServeRequest) / 8;
    static_assert(sizeof(ServeRequest) % 8 == 0, "request copied in 8-byte words");
    const unsigned long long *src = (const unsigned long long *)&host->req[slot];
    unsigned long long *dst = (unsigned long long *)&S.r;
    for (int w = lane; w < WORDS; w += 64)
        dst[w] = __hip_atomic_load(src + w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __threadfence();
    if (lane == 0) {
        const unsigned long long gen = S.r.gen;
        for (int k = 0; k < SERVE_NPH; k++) S.done[k] = 0;
        S.nr[PH_BOUNDS] = ceil_div(S.r.n, SERVE_ATOMS_LIGHT);
        S.bad = 0;
        __threadfence();
        __hip_atomic_store(&S.next[PH_BOUNDS], serve_counter(gen), __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        serve_push(dev, slot, PH_BOUNDS, gen);
    }
    return true;
}

// The persistent kernel: one wave per workgroup (LDS: templates, the hull
// stage's per-lane state or the match stage's, in a union).
template <typename RT>
__global__ void __launch_bounds__(64, 2) k_serve(TablesView T, ServeDev *dev, ServeHost *host, long long idle_ticks) {
    __shared__ MatchShared M;
    __shared__ TablesView Tl;
    __shared__ MatchOut Ol;
    __shared__ ServeWork<RT> U;
    const int lane = threadIdx.x & 63;
    if (lane == 0) Tl = T;
    load_templates(M, T);
    long long idle_from = wall_clock64();
    int idle_rounds = 0;
    // the stage of this wave's items not yet counted (see serve_advance)
    int cur_slot = -1, cur_ph = 0;
    unsigned long long cur_gen = 0;
    long long pending = 0;
    for (;;) {
        int slot = -1, ph = 0;
        long long r = -1;
        unsigned long long gen = 0;
        if (lane == 0) {
            unsigned long long hd = __hip_atomic_load(&dev->head, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const unsigned long long tl = __hip_atomic_load(&dev->tail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            for (unsigned long long pos = hd; pos < tl && pos < hd + 64; pos++) {
                if (__hip_atomic_load(&dev->seq[pos % SERVE_FIFO], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) !=
                    pos + 1)
                    break;
                const unsigned long long e = dev->entry[pos % SERVE_FIFO];
                const int sl = (int)(e & 0xFFFF), p2 = (int)((e >> 16) & 0xFF);
                const unsigned long long g2 = e >> 24;
                ServeSlot &S = dev->slot[sl];
                // claim the next item.  The counter carries the frame's
                // generation: an entry left over from the slot's previous
                // frame sees another generation and leaves it alone; a claim
                // that races with the counter's reset for a new frame takes
                // an item of that frame, and runs it as such (the generation
                // comes from the counter).  Exhausted counters are not
                // incremented, so the index stays within its bits.
                const unsigned long long v = __hip_atomic_load(&S.next[p2], __ATOMIC_ACQUIRE,
                                                               __HIP_MEMORY_SCOPE_AGENT);
                if ((v >> SERVE_IDX_BITS) == g2 && (long long)(v & SERVE_IDX_MASK) < S.nr[p2]) {
                    const unsigned long long w = __hip_atomic_fetch_add(&S.next[p2], 1ull, __ATOMIC_ACQ_REL,
                                                                        __HIP_MEMORY_SCOPE_AGENT);
                    if ((long long)(w & SERVE_IDX_MASK) < S.nr[p2]) {
                        slot = sl;
                        ph = p2;
                        r = (long long)(w & SERVE_IDX_MASK);
                        gen = w >> SERVE_IDX_BITS;
                        break;
                    }
                }
                // exhausted (or stale): the front entry leaves the queue
                if (pos == hd && atomicCAS(&dev->head, hd, hd + 1) == hd) hd++;
            }
        }
        slot = __shfl(slot, 0);
        if (slot < 0) {
            if (pending) {
                // out of work: count what this wave did (it may finish a stage)
                serve_advance(dev, host, cur_slot, cur_ph, cur_gen, pending);
                __syncthreads();
                pending = 0;
                cur_slot = -1;
                continue;
            }
            // Idle.  Waves that find nothing back off (up to ~10 us between
            // looks at the queue), only one wave in 16 looks for new frames
            // in host memory, and the stop word (host memory too) is read
            // every 32nd idle round: idle waves keep the queue's cache lines
            // and the host link free for the working ones.
            if ((blockIdx.x & 15) == (idle_rounds & 15) && serve_pull(dev, host)) {
                idle_from = wall_clock64();
                idle_rounds = 0;
                continue;
            }
            idle_rounds++;
            if ((idle_rounds & 31) == 0 &&
                __hip_atomic_load(&host->stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM))
                break;
            if (wall_clock64() - idle_from > idle_ticks) break;
            const int naps = idle_rounds < 6 ? (1 << idle_rounds) : 48;
            for (int z = 0; z < naps; z++) __builtin_amdgcn_s_sleep(8);
            continue;
        }
        idle_rounds = 0;
        ph = __shfl(ph, 0);
        r = __shfl(r, 0);
        gen = __shfl(gen, 0);
        if (slot != cur_slot || ph != cur_ph || gen != cur_gen) {
            // a new stage for this wave: count the previous one's items, and
            // see the new stage's inputs (an invalidation of the L2, once)
            if (pending) serve_advance(dev, host, cur_slot, cur_ph, cur_gen, pending);
            __syncthreads();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            cur_slot = slot;
            cur_ph = ph;
            cur_gen = gen;
            pending = 0;
        }
        serve_item<RT>(M, Tl, Ol, U, T, dev->slot[slot], ph, r);
        pending++;
        __syncthreads();
        idle_from = wall_clock64();
    }
    if (pending) serve_advance(dev, host, cur_slot, cur_ph, cur_gen, pending);
}

__global__ void k_wall_clock(long long *out) {
    if (threadIdx.x == 0) __hip_atomic_store(out, (long long)wall_clock64(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

void launch_match(int64_t n, const double *nbr_rel, const int32_t *nbr_id, const int32_t *sid,
                  const int8_t *species, const TablesView &T, const int32_t *code, const uint64_t *ord,
                  uint32_t mask, double cutoff, bool force_full, const MatchOut &O, int32_t *full_count,
                  unsigned long long *job_count, const int32_t *knn_src, int32_t *knn_out, const int32_t *box_fail,
                  int32_t *host_flag, bool f32, hipStream_t st) {
    if (n <= 0) return;
    const int apw = match_atoms_per_wave(n), per = MB / 64 * apw;
    dim3 grid((unsigned)((n + per - 1) / per)), block(MB);
    if (f32)
        hipLaunchKernelGGL(k_match<float>, grid, block, 0, st, n, nbr_rel, nbr_id, sid, species, T, code, ord, mask,
                           cutoff, (int)force_full, O, full_count, job_count, knn_src, knn_out, box_fail, apw, host_flag);
    else
        hipLaunchKernelGGL(k_match<double>, grid, block, 0, st, n, nbr_rel, nbr_id, sid, species, T, code, ord,
                           mask, cutoff, (int)force_full, O, full_count, job_count, knn_src, knn_out, box_fail, apw,
                           host_flag);
}

template <typename RT>
static int launch_serve_rt(const TablesView &T, ServeDev *dev, ServeHost *host, long long idle_ticks,
                           hipStream_t st) {
    int per_cu = 0, cus = 0, device = 0;
    if (hipGetDevice(&device) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || cus < 1) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_serve<RT>, 64, 0) != hipSuccess || per_cu < 1)
        per_cu = 1;
    const int blocks = per_cu * cus;
    hipLaunchKernelGGL(k_serve<RT>, dim3((unsigned)blocks), dim3(64), 0, st, T, dev, host, idle_ticks);
    return hipGetLastError() == hipSuccess ? blocks : 0;
}
int launch_serve(bool f32, const TablesView &T, ServeDev *dev, ServeHost *host, long long idle_ticks,
                 hipStream_t st) {
    return f32 ? launch_serve_rt<float>(T, dev, host, idle_ticks, st)
               : launch_serve_rt<double>(T, dev, host, idle_ticks, st);
}
void launch_wall_clock(long long *out, hipStream_t st) {
    hipLaunchKernelGGL(k_wall_clock, dim3(1), dim3(64), 0, st, out);
}

}  // namespace ptm
