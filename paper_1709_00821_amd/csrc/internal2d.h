// Internal interfaces of the 2D library (api2d.hip) and its kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "physics.h"

namespace fdtdp {

// The probes in the cells of one lane of a tile: bit (q R + r) CJ + c for
// component q at row r and column c of its registers.  Their sample rows follow
// one another from `first` in the order of the bits.
struct LaneProbes {
    uint32_t mask;
    int32_t first;
};

// Device view of a 2D grid (passed by value to kernels).  The plasma lives on
// a compact support: row i holds it on j in [span[i].x, span[i].y), at compact
// index rowoff[i] + j - span[i].x of the per-component arrays (the union of
// the components' supports; wp2 = 0 where one component has none).
struct Grid2 {
    int64_t nx, ny;
    int mode, px, py;          // mode 0 TM, 1 TE; periodic x, y
    double dt, d;
    double ch;                 // dt/(mu0 d)
    double ce;                 // dt/(eps0 d), the vacuum E coefficient
    const int2 *span;          // [nx]
    const int64_t *rowoff;     // [nx]
    const double *wp2[2], *nu[2];   // [S] per E component
    int has_src;
    int64_t si, sj;
    double src_tau, src_t0, src_amp;
    const double *srcv;        // [SB] source value of every step of the current window
    int SB;                    // sample window length
    const LaneProbes *tprobe;  // [waves with probes][64]
    double *samp;              // [distinct probes][SB]
};

template <typename T>
struct Fields2 {
    T *E[2];                   // TM: Ez; TE: Ex, Ey
    T *H[2];                   // TM: Hx, Hy; TE: Hz
    double *J[2];              // [S] per E component, FP64
};

// One tile of the temporally blocked step: the cells held start at (i0, j0),
// which may lie outside the grid (beyond a wall, or wrapped on a periodic
// axis); outputs are the rows [oi0, oi1) and columns [oj0, oj1).
struct Tile2 {
    int32_t i0, j0, oi0, oi1, oj0, oj1;
    int32_t special;           // holds cells outside the grid, a wall line or the source
    int32_t pwaves, probe0;    // its waves with probes (a bit each) and the first one's place in tprobe
    int32_t pad[3];
};

// Time steps a launch takes (the halo of a tile), and the tile shapes: a
// workgroup of NW waves, each wave R rows of 64 CJ columns.
//
// Eight steps: at 4096^2 a pass of one step already takes 105 us of a pass of
// eight's 145 us (TM FP32, the vacuum tiles alone: the loads and stores of the
// fields bound it, 3.8-4.6 TB/s with the halo), and a halo of 16 would leave a
// third of a 48-row tile.
constexpr int kSteps2 = 8;
struct Shape2 {
    int R, CJ, NW;
    int rows() const { return R * NW; }
    int cols() const { return 64 * CJ; }
};
// Vacuum tiles: two columns a lane (one DPP move a row and neighbour serves
// two cells), eight waves, two workgroups a CU.  The tall tile (48 rows, 32
// written) reads fewer halo rows and is the faster one where tiles outnumber
// the GPU; the flat one (32 rows, 16 written) where they all run at once and
// the length of a wave's step decides.  us a step, flat against tall (8 rows a wave,
// 64 or 96 rows a tile, was slower at every size):
// TM FP32 512^2 3.2 against 3.9, 1000^2 4.5 against 4.1, 4096^2 33 against 25;
// TE FP64 512^2 2.8 against 3.6, 1000^2 5.0 against 4.5, 4096^2 43 against 36.
constexpr Shape2 kFlat2 = {4, 2, 8}, kTall2 = {6, 2, 8};
constexpr int64_t kFlatMaxTiles2 = 512;      // two workgroups on each of 256 CUs
// Steps taken one by one in place instead of as a pass of tiles.  One step
// alone: a pass costs its loads and stores however few steps it takes (4096^2 TM
// FP32 157 us against 116, 1000^2 TE FP32 42 against 17), and on small grids so do two (256^2 29
// against 24 us; 1000^2 39 against 35; 4096^2 165 against 232).  All steps: grids of two or three
// rows, of which a tile's sixteen output rows leave most empty, where the tiles fill the GPU
// (2 x 2^20 cells 43 us a step against 29; 4 x 2^18 13 against 12.5, 2 x 4096 1.8 against 5.9).
constexpr int64_t kTwoStepsBelow2 = 1 << 20; // cells
constexpr int64_t kThinRows2 = 4, kThinTiles2 = 1024;
// Plasma tiles hold six coefficients and a current a cell and component, so
// one column a lane and four rows a wave.
constexpr Shape2 kPlasma2 = {4, 1, 12};
enum class Tiles2 { flat, tall, plasma };

// nsteps <= kSteps2 steps of every tile from `in` to `out`; slot0: the window
// slot of the first step.
template <typename T>
void launch_tiles2d(const Grid2 &g, const Fields2<T> &in, const Fields2<T> &out, const Tile2 *tiles,
                    int64_t ntiles, Tiles2 shape, int nsteps, int slot0, hipStream_t st);

// Step m in place, the sample rows' cells (component N + cell each) into `slot`.
template <typename T>
void launch_step2d(const Grid2 &g, const Fields2<T> &f, const int64_t *cells, int64_t rows, int64_t m, int slot,
                   hipStream_t st);

// The source values of steps m_first .. m_first + count - 1.
void launch_src2d(const Grid2 &g, int64_t m_first, int count, double *srcv, hipStream_t st);

}  // namespace fdtdp
