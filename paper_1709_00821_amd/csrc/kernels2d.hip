// 2D Yee-RKETD kernels for gfx950 (TM: Ez, Hx, Hy; TE: Ex, Ey, Hz).
//
// Temporal blocking: a workgroup holds a tile of cells in registers (each wave
// R rows of 64 CJ columns, a lane CJ adjacent columns of every row), takes up
// to kSteps2 steps, and writes the cells whose values are still exact (the
// tile less a halo of kSteps2 cells on each side) to the other copy of the
// fields.  Columns cross lanes with DPP moves, rows cross waves through LDS
// (one row of E before the H half, one row of H before the E half, a barrier
// each).  One pass over memory then serves eight steps where an H pass and an
// E/J pass a step moved 24 B a cell each step: 4096^2 TM FP32 117 -> 25 us a
// step, 1001 x 1500 TE FP64 22 -> 5.6 us.  What bounds a large grid now is the
// load and store phases of the tiles (a pass of one step takes 105 of the 145 us
// of eight; its traffic is 1.08 times the fields read and written once), a small
// one the latency of a pass.
//
// Arithmetic in FP64 registers at either storage precision, every new E and H
// rounded to the storage type every step, so a result does not depend on how
// the steps are grouped into launches.
#include <hip/hip_runtime.h>

#include "internal2d.h"
#include "tile1d.h"

namespace fdtdp {

// The CJ values of one row of a lane, as one access (element alignment is all
// a row of an odd-sized grid has).
template <typename T, int CJ>
struct __attribute__((packed, aligned(sizeof(T)))) Cols {
    T v[CJ];
};

// Where a row (or column) of a tile lies: the grid index to load from, always
// one that exists, and whether the row is inside the grid (a periodic axis
// wraps, also several times round a grid shorter than the halo).
struct At2 {
    int32_t i;
    bool ok;
};
__device__ __forceinline__ At2 at2(int32_t i, int32_t n, int periodic)
{
    const bool in = i >= 0 && i < n;
    if (!periodic) return {in ? i : 0, in};
    if (!in) {
        i %= n;
        i += i < 0 ? n : 0;
    }
    return {i, true};
}

// Registers of a lane: A, B, C are Ez, Hx, Hy (TM) or Ex, Ey, Hz (TE).
template <typename T, int NC, int R, int CJ, bool PLASMA>
struct Regs2 {
    T A[R][CJ], B[R][CJ], C[R][CJ];
    double J[PLASMA ? NC : 1][PLASMA ? R : 1][PLASMA ? CJ : 1];
    double cf[PLASMA ? NC : 1][PLASMA ? R : 1][PLASMA ? CJ : 1][6];
};

// What the cells outside the grid, the walls and the source need, kept small
// (a flag a cell would fill the register file): bit r of a row mask for row r
// of the wave (uniform), a word a column.  E component q of a cell is ANDed
// with ekeep[q] of its column and the sign-extended bit of rkeep[q] (0: held at
// zero); the source's value is added where rsrc has the row, from the lane
// holding its column.
struct Special2 {
    uint32_t rkeep[2], rsrc;
    uint32_t ckeep[2][2];      // [component][column]
    bool csrc[2];
};

// x where keep is all ones, +0 where it is 0.
__device__ __forceinline__ double keep_bits(double x, uint32_t keep)
{
    int2 v = __builtin_bit_cast(int2, x);
    return __builtin_bit_cast(double, make_int2(v.x & (int)keep, v.y & (int)keep));
}

// A new field value, rounded to the storage type where it is formed (left to
// itself, the compiler sinks the FP32 roundings of a whole half-step to its
// end and holds every double until then, twice the registers).
template <typename T>
__device__ __forceinline__ T rounded(double x)
{
    if constexpr (sizeof(T) == 4) return opaque((T)x);
    else return x;
}

// E^{n+1} of one cell (eqs.(11)+(12) solved, the source's share add, the
// wall), then J (eq.(11)); k = {CA, CJ, CH, a, b1, b2}.
template <typename T, bool PLASMA, bool SPECIAL>
__device__ __forceinline__ T e_cell2(double Eo, double curl, double ce, const double (&k)[6], double &J, double add,
                                     uint32_t keep)
{
    double En;
    if constexpr (PLASMA) En = __builtin_fma(k[2], curl, __builtin_fma(-k[1], J, k[0] * Eo));
    else En = __builtin_fma(ce, curl, Eo);
    if constexpr (SPECIAL) En = keep_bits(En + add, keep);
    if constexpr (PLASMA) J = __builtin_fma(k[5], En, __builtin_fma(k[4], Eo, k[3] * J));
    return rounded<T>(En);
}

// nsteps steps of a tile in registers.
template <typename T, int MODE, int R, int CJ, int NW, bool PLASMA, bool SPECIAL>
__device__ __forceinline__ void run_tile2(Regs2<T, MODE == 0 ? 1 : 2, R, CJ, PLASMA> &s, const Grid2 &g,
                                          const Tile2 &t, const Special2 &sp, int w, int lane,
                                          T (*ldsE)[64 * CJ], T (*ldsH)[64 * CJ], int nsteps, int slot0)
{
    static_assert((MODE == 0 ? 1 : 2) * R * CJ <= 32, "a probe mask holds the registers of a lane");
    typedef Cols<T, CJ> V;
    const double ch = g.ch, ce = g.ce;
    auto put = [&](T (*lds)[64 * CJ], const T (&row)[CJ]) {
        V v;
#pragma unroll
        for (int c = 0; c < CJ; ++c) v.v[c] = row[c];
        *(V *)&lds[w][lane * CJ] = v;
    };
    auto get = [&](T (*lds)[64 * CJ], int from, T (&row)[CJ]) {
        const bool there = from >= 0 && from < NW;   // beyond the tile: the halo's edge, any value
        const V v = *(const V *)&lds[there ? from : w][lane * CJ];
#pragma unroll
        for (int c = 0; c < CJ; ++c) row[c] = there ? v.v[c] : (T)0;
    };
    // H^{n+1/2} of row r (eq.(14)); up: the E of row r + 1 its x-difference reads
    auto h_row = [&](int r, const T (&up)[CJ]) {
        const T next = shfl_down1(s.A[r][0]);
#pragma unroll
        for (int c = 0; c < CJ; ++c) {
            const double e = (double)s.A[r][c], ej = (double)(c + 1 < CJ ? s.A[r][c + 1 < CJ ? c + 1 : 0] : next);
            if constexpr (MODE == 0) {
                s.B[r][c] = rounded<T>(__builtin_fma(-ch, ej - e, (double)s.B[r][c]));
                s.C[r][c] = rounded<T>(__builtin_fma(ch, (double)up[c] - e, (double)s.C[r][c]));
            } else {
                const double curl = ((double)up[c] - (double)s.B[r][c]) - (ej - e);
                s.C[r][c] = rounded<T>(__builtin_fma(-ch, curl, (double)s.C[r][c]));
            }
        }
    };
    double sv[CJ] = {};                      // the step's source value in the source's column, else 0
    uint32_t rkeep[2] = {~0u, ~0u}, rsrc = 0;
    // E^{n+1} and J^{n+1} of row r; dn: the H of row r - 1
    auto e_row = [&](int r, const T (&dn)[CJ]) {
        const T prev = shfl_up1(MODE == 0 ? s.B[r][CJ - 1] : s.C[r][CJ - 1]);
        uint32_t rk[2] = {~0u, ~0u};
        if constexpr (SPECIAL) {
#pragma unroll
            for (int q = 0; q < 2; ++q) rk[q] = (uint32_t)((int)(rkeep[q] << (31 - r)) >> 31);
        }
#pragma unroll
        for (int c = 0; c < CJ; ++c) {
            double none = 0.0, add = 0.0;
            const double no6[6] = {0, 0, 0, 0, 0, 0};
            uint32_t keep[2] = {~0u, ~0u};
            if constexpr (SPECIAL) {
#pragma unroll
                for (int q = 0; q < 2; ++q) keep[q] = rk[q] & sp.ckeep[q][c];
                add = ((rsrc >> r) & 1) ? sv[c] : 0.0;
            }
            if constexpr (MODE == 0) {
                const double hx = (double)s.B[r][c], hxj = (double)(c > 0 ? s.B[r][c > 0 ? c - 1 : 0] : prev);
                const double hy = (double)s.C[r][c], hyi = (double)dn[c];
                const double curl = (hy - hyi) - (hx - hxj);
                if constexpr (PLASMA)
                    s.A[r][c] = e_cell2<T, PLASMA, SPECIAL>((double)s.A[r][c], curl, ce, s.cf[0][r][c], s.J[0][r][c],
                                                            add, keep[0]);
                else
                    s.A[r][c] = e_cell2<T, PLASMA, SPECIAL>((double)s.A[r][c], curl, ce, no6, none, add, keep[0]);
            } else {
                const double hz = (double)s.C[r][c], hzj = (double)(c > 0 ? s.C[r][c > 0 ? c - 1 : 0] : prev);
                const double cx = hz - hzj, cy = -(hz - (double)dn[c]);
                if constexpr (PLASMA) {
                    s.A[r][c] = e_cell2<T, PLASMA, SPECIAL>((double)s.A[r][c], cx, ce, s.cf[0][r][c], s.J[0][r][c],
                                                            0.0, keep[0]);
                    s.B[r][c] = e_cell2<T, PLASMA, SPECIAL>((double)s.B[r][c], cy, ce, s.cf[1][r][c], s.J[1][r][c],
                                                            add, keep[1]);
                } else {
                    s.A[r][c] = e_cell2<T, PLASMA, SPECIAL>((double)s.A[r][c], cx, ce, no6, none, 0.0, keep[0]);
                    s.B[r][c] = e_cell2<T, PLASMA, SPECIAL>((double)s.B[r][c], cy, ce, no6, none, add, keep[1]);
                }
            }
        }
    };
    // rows are scheduled one after another: interleaved, their converted
    // operands would all be live at once
    auto rows_apart = [] { __builtin_amdgcn_sched_barrier(0); };
    for (int st = 0; st < nsteps; ++st) {
        if constexpr (SPECIAL) {
            const double v = g.srcv[slot0 + st];
#pragma unroll
            for (int c = 0; c < CJ; ++c) sv[c] = sp.csrc[c] ? v : 0.0;
            // read anew each step: masks a cell, hoisted out of the loop, spill
            rkeep[0] = __builtin_amdgcn_readfirstlane(sp.rkeep[0]);
            rkeep[1] = __builtin_amdgcn_readfirstlane(sp.rkeep[1]);
            rsrc = __builtin_amdgcn_readfirstlane(sp.rsrc);
            asm volatile("" : "+s"(rkeep[0]), "+s"(rkeep[1]), "+s"(rsrc));
        }
        // the E row the wave below reads (TM Ez, TE Ey), then every row whose
        // upper neighbour is in this wave before the barrier
        if constexpr (MODE == 0) put(ldsE, s.A[0]);
        else put(ldsE, s.B[0]);
#pragma unroll
        for (int r = 0; r + 1 < R; ++r) {
            if constexpr (MODE == 0) h_row(r, s.A[r + 1 < R ? r + 1 : r]);
            else h_row(r, s.B[r + 1 < R ? r + 1 : r]);
            rows_apart();
        }
        __syncthreads();
        T edge[CJ];
        get(ldsE, w + 1, edge);
        h_row(R - 1, edge);
        put(ldsH, s.C[R - 1]);
#pragma unroll
        for (int r = R - 1; r > 0; --r) {
            e_row(r, s.C[r > 0 ? r - 1 : 0]);
            rows_apart();
        }
        __syncthreads();
        get(ldsH, w - 1, edge);
        e_row(0, edge);
        // probe samples of the step, every lane those in its own cells: a wave's
        // probes cost a step no more than the registers of a lane, however many
        // they are (4096 probes in 64 x 64 cells, walked one after another by the
        // wave, took 400 steps of a 1024^2 grid from 1.7 to 89 ms).  The lane's mask
        // is read anew each step: held, it takes registers of every wave
        if ((t.pwaves >> w) & 1) {
            const LaneProbes lp = g.tprobe[(t.probe0 + __popc(t.pwaves & ((1 << w) - 1))) * 64 + lane];
            uint32_t at = ((uint32_t)lp.first * (uint32_t)g.SB + (uint32_t)(slot0 + st)) * 8u;   // of 67 MB at most
#pragma unroll
            for (int q = 0; q < (MODE == 0 ? 1 : 2); ++q)
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int c = 0; c < CJ; ++c)
                        if ((lp.mask >> ((q * R + r) * CJ + c)) & 1) {
                            *(double *)((char *)g.samp + at) = (double)(q == 0 ? s.A[r][c] : s.B[r][c]);
                            at += (uint32_t)g.SB * 8u;
                        }
        }
    }
}

// Load a tile, take its steps, store its outputs.
template <typename T, int MODE, int R, int CJ, int NW, bool PLASMA, bool SPECIAL>
__device__ __forceinline__ void tile2(const Grid2 &g, const Fields2<T> &in, const Fields2<T> &out, const Tile2 &t,
                                      T (*ldsE)[64 * CJ], T (*ldsH)[64 * CJ], int nsteps, int slot0)
{
    constexpr int NC = MODE == 0 ? 1 : 2;
    typedef Cols<T, CJ> V;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int32_t i0 = t.i0 + w * R, j0 = t.j0 + lane * CJ;
    const int32_t nx = (int32_t)g.nx, ny = (int32_t)g.ny;
    const T *fa[3] = {in.E[0], MODE == 0 ? in.H[0] : in.E[1], MODE == 0 ? in.H[1] : in.H[0]};
    At2 col[CJ];
#pragma unroll
    for (int c = 0; c < CJ; ++c) col[c] = SPECIAL ? at2(j0 + c, ny, g.py) : At2{j0 + c, true};
    // every load is issued from an index that exists, none behind a branch
    Regs2<T, NC, R, CJ, PLASMA> s;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const At2 row = SPECIAL ? at2(i0 + r, nx, g.px) : At2{i0 + r, true};
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            // a uniform row address and one 32-bit lane offset for all rows
            const T *a = fa[q] + (int64_t)row.i * ny;
            V v;
            if constexpr (!SPECIAL) {
                v = *(const V *)(a + t.j0 + (uint32_t)(lane * CJ));
            } else {
#pragma unroll
                for (int c = 0; c < CJ; ++c) {
                    v.v[c] = a[(uint32_t)col[c].i];
                    v.v[c] = row.ok && col[c].ok ? v.v[c] : (T)0;
                }
            }
#pragma unroll
            for (int c = 0; c < CJ; ++c) (q == 0 ? s.A : q == 1 ? s.B : s.C)[r][c] = v.v[c];
        }
        if constexpr (PLASMA) {
            const int2 sp = g.span[row.i];
            const int64_t ro = g.rowoff[row.i];
#pragma unroll
            for (int c = 0; c < CJ; ++c) {
                const bool here = row.ok && col[c].ok && col[c].i >= sp.x && col[c].i < sp.y;
                const int64_t p = here ? ro + (col[c].i - sp.x) : 0;
#pragma unroll
                for (int k = 0; k < NC; ++k) {
                    // off the support: wp2 = 0, the vacuum coefficients, no
                    // current.  The coefficients are formed here: reading
                    // the six from a table (48 B a cell instead of 16) took
                    // 71 us a pass of the 4096^2 TM cylinder against 65
                    const double J = in.J[k][p];
                    s.J[k][r][c] = here ? J : 0.0;
                    const double w2 = g.wp2[k][p], nu = g.nu[k][p];
                    const Coef f = node_coef(here ? w2 : 0.0, here ? nu : 0.0, g.dt, g.d, 0);
                    const double v[6] = {f.CA, f.CJ, f.CH, f.a, f.b1, f.b2};
#pragma unroll
                    for (int q = 0; q < 6; ++q) s.cf[k][r][c][q] = v[q];
                }
            }
        }
    }
    Special2 sp = {};
    if constexpr (SPECIAL) {
        // walls: TM holds Ez at zero on both index-0 lines, TE Ex on j = 0
        // and Ey on i = 0; everything outside the grid reads zero
        for (int r = 0; r < R; ++r) {
            const At2 row = at2(i0 + r, nx, g.px);
            const uint32_t bit = 1u << r;
            const bool wall = !g.px && row.i == 0;
            if (row.ok && !(MODE == 0 && wall)) sp.rkeep[0] |= bit;
            if (row.ok && !wall) sp.rkeep[1] |= bit;
            if (row.ok && g.has_src && row.i == (int32_t)g.si) sp.rsrc |= bit;
        }
#pragma unroll
        for (int c = 0; c < CJ; ++c) {
            const bool wall = !g.py && col[c].i == 0;
            sp.ckeep[0][c] = col[c].ok && !wall ? ~0u : 0u;
            sp.ckeep[1][c] = col[c].ok ? ~0u : 0u;
            sp.csrc[c] = col[c].ok && g.has_src && col[c].i == (int32_t)g.sj;
        }
    }
    run_tile2<T, MODE, R, CJ, NW, PLASMA, SPECIAL>(s, g, t, sp, w, lane, ldsE, ldsH, nsteps, slot0);
    T *fo[3] = {out.E[0], MODE == 0 ? out.H[0] : out.E[1], MODE == 0 ? out.H[1] : out.H[0]};
    const bool all = j0 >= t.oj0 && j0 + CJ <= t.oj1;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int32_t i = i0 + r;
        if (i < t.oi0 || i >= t.oi1) continue;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            T *a = fo[q] + (int64_t)i * ny + t.j0 + (uint32_t)(lane * CJ);
            V v;
#pragma unroll
            for (int c = 0; c < CJ; ++c) v.v[c] = (q == 0 ? s.A : q == 1 ? s.B : s.C)[r][c];
            if (all) {
                *(V *)a = v;
            } else {
#pragma unroll
                for (int c = 0; c < CJ; ++c)
                    if (j0 + c >= t.oj0 && j0 + c < t.oj1) a[c] = v.v[c];
            }
        }
        if constexpr (PLASMA) {
            const int2 sp = g.span[i];
            const int64_t ro = g.rowoff[i];
#pragma unroll
            for (int c = 0; c < CJ; ++c) {
                const int32_t j = j0 + c;
                if (j < t.oj0 || j >= t.oj1 || j < sp.x || j >= sp.y) continue;
#pragma unroll
                for (int k = 0; k < NC; ++k) out.J[k][ro + (j - sp.x)] = s.J[k][r][c];
            }
        }
    }
}

template <typename T, int MODE, int R, int CJ, int NW, bool PLASMA>
__global__ __launch_bounds__(NW * 64) void k2_tile(Grid2 g, Fields2<T> in, Fields2<T> out, const Tile2 *tiles,
                                                   int nsteps, int slot0)
{
    __shared__ T ldsE[NW][64 * CJ], ldsH[NW][64 * CJ];
    const Tile2 t = tiles[xcd_block(blockIdx.x, gridDim.x)];
    // each path loads and stores for itself: state merged from two loops
    // takes twice the registers
    if (t.special) tile2<T, MODE, R, CJ, NW, PLASMA, true>(g, in, out, t, ldsE, ldsH, nsteps, slot0);
    else tile2<T, MODE, R, CJ, NW, PLASMA, false>(g, in, out, t, ldsE, ldsH, nsteps, slot0);
}

template <typename T, int MODE, int R, int CJ, int NW, bool PLASMA>
void launch_shape(const Grid2 &g, const Fields2<T> &in, const Fields2<T> &out, const Tile2 *tiles, int64_t n,
                  int nsteps, int slot0, hipStream_t st)
{
    hipLaunchKernelGGL((k2_tile<T, MODE, R, CJ, NW, PLASMA>), dim3((unsigned)n), dim3(64 * NW), 0, st, g, in, out,
                       tiles, nsteps, slot0);
}

template <typename T, int MODE>
void launch_mode(const Grid2 &g, const Fields2<T> &in, const Fields2<T> &out, const Tile2 *tiles, int64_t n,
                 Tiles2 shape, int nsteps, int slot0, hipStream_t st)
{
    constexpr Shape2 f = kFlat2, t = kTall2, p = kPlasma2;
    if (shape == Tiles2::flat)
        launch_shape<T, MODE, f.R, f.CJ, f.NW, false>(g, in, out, tiles, n, nsteps, slot0, st);
    else if (shape == Tiles2::tall)
        launch_shape<T, MODE, t.R, t.CJ, t.NW, false>(g, in, out, tiles, n, nsteps, slot0, st);
    else
        launch_shape<T, MODE, p.R, p.CJ, p.NW, true>(g, in, out, tiles, n, nsteps, slot0, st);
}

template <typename T>
void launch_tiles2d(const Grid2 &g, const Fields2<T> &in, const Fields2<T> &out, const Tile2 *tiles, int64_t ntiles,
                    Tiles2 shape, int nsteps, int slot0, hipStream_t st)
{
    if (ntiles <= 0 || nsteps <= 0) return;
    if (g.mode == 0) launch_mode<T, 0>(g, in, out, tiles, ntiles, shape, nsteps, slot0, st);
    else launch_mode<T, 1>(g, in, out, tiles, ntiles, shape, nsteps, slot0, st);
}

template void launch_tiles2d<float>(const Grid2 &, const Fields2<float> &, const Fields2<float> &, const Tile2 *,
                                    int64_t, Tiles2, int, int, hipStream_t);
template void launch_tiles2d<double>(const Grid2 &, const Fields2<double> &, const Fields2<double> &, const Tile2 *,
                                     int64_t, Tiles2, int, int, hipStream_t);

// ---- one step, in place ------------------------------------------------------
//
// One thread a cell: an H pass (reads E only), then an E/J pass (reads H only,
// each cell its own E and J), so no pass reads a value another thread of the
// same pass writes and one copy of the fields is enough.  Workgroups of 64 (j,
// the contiguous axis) x 4 (i) cells, dealt so that each XCD takes a contiguous
// band of rows.  The same values as a tile's step, bit for bit.  Where it is
// taken: see plan2 and by_pass in api2d.hip.

// A neighbour of cell k = i ny + j one step along an axis: its index (wrapped
// on a periodic axis) and whether it exists (false beyond a wall, where the
// field reads as zero).  The index is always one to load from (the cell itself
// where the neighbour is absent), so every neighbour load is issued
// unconditionally, beside the others, and no load waits on a branch.
struct Nb {
    int64_t k;
    bool ok;
};
__device__ __forceinline__ Nb nb_jp(const Grid2 &g, int64_t k, int64_t j)
{
    const bool in = j + 1 < g.ny;
    return {in ? k + 1 : (g.py ? k - (g.ny - 1) : k), in || g.py};
}
__device__ __forceinline__ Nb nb_jm(const Grid2 &g, int64_t k, int64_t j)
{
    const bool in = j > 0;
    return {in ? k - 1 : (g.py ? k + (g.ny - 1) : k), in || g.py};
}
__device__ __forceinline__ Nb nb_ip(const Grid2 &g, int64_t k, int64_t i)
{
    const bool in = i + 1 < g.nx;
    return {in ? k + g.ny : (g.px ? k - (g.nx - 1) * g.ny : k), in || g.px};
}
__device__ __forceinline__ Nb nb_im(const Grid2 &g, int64_t k, int64_t i)
{
    const bool in = i > 0;
    return {in ? k - g.ny : (g.px ? k + (g.nx - 1) * g.ny : k), in || g.px};
}
template <typename T>
__device__ __forceinline__ double ldn(const T *a, const Nb &n)
{
    const double v = (double)a[n.k];
    return n.ok ? v : 0.0;
}

// The cell of this thread; i is the same for the whole wave (one row).
__device__ __forceinline__ bool cell_of(const Grid2 &g, int64_t &i, int64_t &j)
{
    const int64_t bj_n = (g.ny + 63) / 64, bi_n = (g.nx + 3) / 4;
    const int64_t b = xcd_block((int64_t)blockIdx.x, bj_n * bi_n);
    i = (b / bj_n) * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    j = (b % bj_n) * 64 + (threadIdx.x & 63);
    return i < g.nx && j < g.ny;
}

// H^{n+1/2} from E^n (eq.(14)).
template <typename T, int MODE>
__global__ __launch_bounds__(256) void k2_h(Grid2 g, Fields2<T> f)
{
    int64_t i, j;
    if (!cell_of(g, i, j)) return;
    const int64_t k = i * g.ny + j;
    const double ch = g.ch;
    const Nb jp = nb_jp(g, k, j), ip = nb_ip(g, k, i);
    if constexpr (MODE == 0) {
        const T *Ez = f.E[0];
        const double e = (double)Ez[k], ej = ldn(Ez, jp), ei = ldn(Ez, ip);
        const double hx = (double)f.H[0][k], hy = (double)f.H[1][k];
        f.H[0][k] = (T)__builtin_fma(-ch, ej - e, hx);
        f.H[1][k] = (T)__builtin_fma(ch, ei - e, hy);
    } else {
        const T *Ex = f.E[0], *Ey = f.E[1];
        const double eyi = ldn(Ey, ip), exj = ldn(Ex, jp), hz = (double)f.H[0][k];
        const double curl = (eyi - (double)Ey[k]) - (exj - (double)Ex[k]);
        f.H[0][k] = (T)__builtin_fma(-ch, curl, hz);
    }
}

// One E component of a cell: eqs.(11)+(12) solved, the source, the wall, then
// eq.(11); the current and the plasma parameters live on the compact support
// (index pidx, or -1 off it) and come in already read (w, v, J: wp2, nu, J^n).
template <typename T>
__device__ __forceinline__ void e_step2(const Grid2 &g, double *Jp, T *Ep, int64_t k, double Eo, double curl_signed,
                                       bool src, double sv, bool wall, int64_t pidx, double w, double v, double J)
{
    double En;
    Coef cf;
    const bool plasma = pidx >= 0 && w != 0.0;
    if (plasma) {
        cf = node_coef(w, v, g.dt, g.d, 0);
        En = __builtin_fma(cf.CH, curl_signed, __builtin_fma(-cf.CJ, J, cf.CA * Eo));
    } else {
        En = __builtin_fma(g.ce, curl_signed, Eo);
    }
    if (src) En = En + sv;
    if (wall) En = 0.0;
    if (plasma) Jp[pidx] = __builtin_fma(cf.b2, En, __builtin_fma(cf.b1, Eo, cf.a * J));
    Ep[k] = (T)En;
}

// E^{n+1} and J^{n+1} from H^{n+1/2}; m = n + 1 (the source time).  Every load
// a cell needs (H and its neighbours, E, and on the support wp2, nu and J) is
// issued before any arithmetic, so a wave waits on one round of loads.
template <typename T, int MODE>
__global__ __launch_bounds__(256) void k2_e(Grid2 g, Fields2<T> f, int64_t m)
{
    constexpr int NC = MODE == 0 ? 1 : 2;
    int64_t i, j;
    if (!cell_of(g, i, j)) return;
    const int64_t k = i * g.ny + j;
    const int2 sp = g.span[i];                      // the row's support (i is wave-uniform)
    const int64_t ro = g.rowoff[i];
    const int64_t pidx = (j >= sp.x && j < sp.y) ? ro + (j - sp.x) : -1;
    const Nb jm = nb_jm(g, k, j), im = nb_im(g, k, i);
    double Eo[NC], w[NC], v[NC], J[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        Eo[c] = (double)f.E[c][k];
        w[c] = v[c] = J[c] = 0.0;
    }
    double curl[NC];
    if constexpr (MODE == 0) {
        const T *Hx = f.H[0], *Hy = f.H[1];
        const double hy = (double)Hy[k], hyi = ldn(Hy, im), hx = (double)Hx[k], hxj = ldn(Hx, jm);
        curl[0] = (hy - hyi) - (hx - hxj);
    } else {
        const T *Hz = f.H[0];
        const double hz = (double)Hz[k], hzj = ldn(Hz, jm), hzi = ldn(Hz, im);
        curl[0] = hz - hzj;
        curl[1] = -(hz - hzi);
    }
    if (pidx >= 0) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            w[c] = g.wp2[c][pidx];
            v[c] = g.nu[c][pidx];
            J[c] = f.J[c][pidx];
        }
    }
    const bool src = g.has_src && i == g.si && j == g.sj;
    const double sv = src ? source_value((double)m * g.dt, g.src_tau, g.src_t0, g.src_amp) : 0.0;
    if constexpr (MODE == 0) {
        const bool wall = (!g.px && i == 0) || (!g.py && j == 0);
        e_step2<T>(g, f.J[0], f.E[0], k, Eo[0], curl[0], src, sv, wall, pidx, w[0], v[0], J[0]);
    } else {
        e_step2<T>(g, f.J[0], f.E[0], k, Eo[0], curl[0], false, 0.0, !g.py && j == 0, pidx, w[0], v[0], J[0]);
        e_step2<T>(g, f.J[1], f.E[1], k, Eo[1], curl[1], src, sv, !g.px && i == 0, pidx, w[1], v[1], J[1]);
    }
}

// Probe samples of the step just taken into slot `slot` of the window; cells:
// component N + cell of each sample row.
template <typename T>
__global__ void k2_sample(Grid2 g, Fields2<T> f, const int64_t *cells, int64_t rows, int slot)
{
    const int64_t r = threadIdx.x + (int64_t)blockIdx.x * blockDim.x;
    if (r >= rows) return;
    const int64_t N = g.nx * g.ny, q = cells[r];
    g.samp[r * g.SB + slot] = (double)(q < N ? f.E[0][q] : f.E[1][q - N]);
}

template <typename T>
void launch_step2d(const Grid2 &g, const Fields2<T> &f, const int64_t *cells, int64_t rows, int64_t m, int slot,
                   hipStream_t st)
{
    const int64_t blocks = ((g.ny + 63) / 64) * ((g.nx + 3) / 4);
    if (g.mode == 0) {
        hipLaunchKernelGGL((k2_h<T, 0>), dim3((unsigned)blocks), dim3(256), 0, st, g, f);
        hipLaunchKernelGGL((k2_e<T, 0>), dim3((unsigned)blocks), dim3(256), 0, st, g, f, m);
    } else {
        hipLaunchKernelGGL((k2_h<T, 1>), dim3((unsigned)blocks), dim3(256), 0, st, g, f);
        hipLaunchKernelGGL((k2_e<T, 1>), dim3((unsigned)blocks), dim3(256), 0, st, g, f, m);
    }
    if (rows > 0)
        hipLaunchKernelGGL((k2_sample<T>), dim3((unsigned)((rows + 63) / 64)), dim3(64), 0, st, g, f, cells, rows, slot);
}

template void launch_step2d<float>(const Grid2 &, const Fields2<float> &, const int64_t *, int64_t, int64_t, int,
                                   hipStream_t);
template void launch_step2d<double>(const Grid2 &, const Fields2<double> &, const int64_t *, int64_t, int64_t, int,
                                    hipStream_t);

__global__ void k2_src(Grid2 g, int64_t m_first, int count, double *srcv)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) srcv[i] = source_value((double)(m_first + i) * g.dt, g.src_tau, g.src_t0, g.src_amp);
}

void launch_src2d(const Grid2 &g, int64_t m_first, int count, double *srcv, hipStream_t st)
{
    hipLaunchKernelGGL(k2_src, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st, g, m_first, count, srcv);
}

}  // namespace fdtdp
