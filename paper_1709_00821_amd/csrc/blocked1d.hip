// Register-resident 1D kernels for gfx950.
//
// Each lane holds C consecutive nodes of E, H (and J, coefficients in plasma,
// psi in CPML layers) in VGPRs; a wave holds 64*C consecutive nodes.  One
// time step needs two neighbour values per lane: E of the next lane's first
// node (for its last H) and H of the previous lane's last node (for its first
// E), moved with cross-lane shuffles; all other neighbours are in the lane.
//
//  * k_tiled: temporal blocking.  Every wave is an independent tile holding
//    its output nodes plus Kh halo nodes on each side; it runs K <= Kh steps
//    with no synchronisation at all (the invalid region grows one node per
//    step from each cut edge and never reaches the outputs), then writes the
//    output nodes to the other ping-pong buffer.
//  * k_span: the same of a run of tiles, whose waves overlap and swap edge
//    values through LDS every kSpanHalo steps, so that only the run's ends carry
//    the halo of the launch's steps.
//  * k_group: one workgroup keeps a whole grid, or a segment of one, in
//    registers for a window or a pass, grid ends, source, probes and layers
//    included; its waves overlap and swap edge values likewise.
#include <hip/hip_runtime.h>

#include "tile1d.h"

namespace fdtdp {

template <typename T, int C, int KLASS, bool ROLES, bool JF = false, int RM = kRoleAll>
__global__ __launch_bounds__(256) void k_tiled(Grids g, State<T> s, int cur, const Tile *tiles,
                                               int64_t ntiles, int nsteps, int slot0)
{
    // class 0: vacuum tiles; 1: tiles with plasma; 2: tiles touching a CPML
    // layer (which may also hold plasma further in).  ROLES: the tiles hold a
    // grid end, the source or a probe (a separate instantiation, so that the
    // bulk tiles' register budget is that of the plain step alone), at most
    // the roles of mask RM.  JF: the FP32 ablation of eq.(11)
    constexpr bool PLASMA = KLASS >= 1;
    constexpr bool CPML = KLASS == 2;
    const int lane = threadIdx.x & 63;
    const int64_t blk = xcd_block(blockIdx.x, gridDim.x);
    const int64_t t = blk * (blockDim.x >> 6) + uniform(threadIdx.x >> 6);
    if (t >= ntiles) return;
    const Tile tl = tiles[t];
    const int b = tl.grid;
    const int64_t off = g.off[b], n = g.n[b];
    const int64_t k0 = (int64_t)tl.lo + (int64_t)lane * C;
    Chunk<T, C, PLASMA, CPML, JF> ck;
    typedef typename Chunk<T, C, PLASMA, CPML, JF>::R R;
    chunk_load<T, C, PLASMA, CPML>(ck, g, s, cur, b, off, n, k0, tl.hi);
    auto er = [](R e0) { return shfl_down1(e0); };
    auto hl = [](R h) { return shfl_up1(h); };
    if constexpr (!ROLES) {
        // two steps per trip: the loop-carried E copies then alternate
        // registers instead of being moved back every step
        int st = 0;
        for (; st + 2 <= nsteps; st += 2) {
            chunk_step_plain<T, C, PLASMA, CPML>(ck, g, er, hl);
            chunk_step_plain<T, C, PLASMA, CPML>(ck, g, er, hl);
        }
        if (st < nsteps) chunk_step_plain<T, C, PLASMA, CPML>(ck, g, er, hl);
    } else {
        const WaveRole role = wave_role<C>(g, b, n, tl.lo, tl.hi);
        WaveProbes wp;
        wp.n = 0;
        if (tl.flags & TILE_PROBE) wp = wave_probes_find<C>(g, b, tl.lo, tl.out_lo, tl.out_hi);
        if constexpr (RM < 0)   // a small mixed class: each wave picks its role code
            run_role_any<T, C, PLASMA, CPML>(ck, g, role, wp, lane, b, tl.lo, tl.out_lo, tl.out_hi, nsteps, slot0,
                                             er, hl, [](int) {});
        else
            run_role<T, C, PLASMA, CPML, RM>(ck, g, role, wp, lane, b, tl.lo, tl.out_lo, tl.out_hi, nsteps, slot0,
                                             er, hl, [](int) {});
    }
    chunk_store<T, C, PLASMA, CPML>(ck, g, s, cur ^ 1, b, off, n, k0, tl.out_lo, tl.out_hi);
}

// Spans: a run of plasma tiles, or of wide vacuum tiles, held by a workgroup of
// up to kSpanWaves waves (tl.flags of them), each of 64 C nodes that overlap the
// next wave's by 2 kSpanHalo.  A wave steps alone, as a tile does, and every kSpanHalo steps
// its two edge lanes on each side pass their nodes to the neighbours through LDS
// (the lanes next to the edge own them, so an exchange is a dozen wide LDS
// accesses of four lanes each way), so only the span's two ends carry a halo of
// the pass's steps.
//
// The step is bound by FP64 issue (the 2^24-node grid ran at nine tenths of the
// FP64 rate), so what a pass can save is the nodes it recomputes: 512-node
// tiles with 64 steps a pass own 384 of their nodes, a span of four waves 1824
// of 2048; of vacuum, 1024-node tiles 896, a span 3872 of 4096.
template <typename T, int C, bool PLASMA, int WAVES>
__global__ __launch_bounds__(WAVES * 64) void k_span(Grids g, State<T> s, int cur, const Tile *tiles, int64_t ntiles,
                                                     int nsteps)
{
    constexpr int EDGE = kSpanHalo / C;
    typedef Chunk<T, C, PLASMA, false> K;
    typedef typename K::R R;
    __shared__ R edge[2][WAVES][2][PLASMA ? 3 : 2][kSpanHalo];   // [copy][wave][left, right][E, H, J]
    const int lane = threadIdx.x & 63;
    const int w = uniform(threadIdx.x >> 6);
    const Tile tl = tiles[xcd_block(blockIdx.x, gridDim.x)];
    const int waves = tl.flags;
    if (w >= waves) {
        for (int base = kSpanHalo; base < nsteps; base += kSpanHalo) __syncthreads();
        return;
    }
    const int b = tl.grid;
    const int64_t off = g.off[b], n = g.n[b];
    const int64_t lo = (int64_t)tl.lo + (int64_t)w * span_stride(C), k0 = lo + (int64_t)lane * C;
    K ck;
    chunk_load<T, C, PLASMA, false>(ck, g, s, cur, b, off, n, k0, tl.hi);
    auto er = [](R e0) { return shfl_down1(e0); };
    auto hl = [](R h) { return shfl_up1(h); };
    const bool low = lane < 32;
    const int gives = low ? lane - EDGE : lane - (64 - 2 * EDGE);   // edge lane given, held (0 .. EDGE-1)
    const int takes = low ? lane : lane - (64 - EDGE);
    const int from = low ? w - 1 : w + 1;
    for (int base = 0; base < nsteps; base += kSpanHalo) {
        if (base > 0) {
            const int c = (base / kSpanHalo) & 1;
            if (gives >= 0 && gives < EDGE) {
                auto &e = edge[c][w][low ? 0 : 1];
#pragma unroll
                for (int i = 0; i < C; ++i) {
                    e[0][gives * C + i] = ck.E[i];
                    e[1][gives * C + i] = ck.H[i];
                    if constexpr (PLASMA) e[2][gives * C + i] = ck.J[i];
                }
            }
            __syncthreads();
            if (takes >= 0 && takes < EDGE && from >= 0 && from < waves) {
                const auto &e = edge[c][from][low ? 1 : 0];
#pragma unroll
                for (int i = 0; i < C; ++i) {
                    ck.E[i] = e[0][takes * C + i];
                    ck.H[i] = e[1][takes * C + i];
                    if constexpr (PLASMA) ck.J[i] = e[2][takes * C + i];
                }
            }
        }
        const int cnt = nsteps - base < kSpanHalo ? nsteps - base : kSpanHalo;
        int st = 0;
        for (; st + 2 <= cnt; st += 2) {
            chunk_step_plain<T, C, PLASMA, false>(ck, g, er, hl);
            chunk_step_plain<T, C, PLASMA, false>(ck, g, er, hl);
        }
        if (st < cnt) chunk_step_plain<T, C, PLASMA, false>(ck, g, er, hl);
    }
    const int64_t own_lo = w > 0 ? lo + kSpanHalo : lo, own_hi = w + 1 < waves ? lo + span_stride(C) + kSpanHalo : tl.hi;
    chunk_store<T, C, PLASMA, false>(ck, g, s, cur ^ 1, b, off, n, k0, own_lo > tl.out_lo ? own_lo : tl.out_lo,
                                   own_hi < tl.out_hi ? own_hi : tl.out_hi);
}

template <typename T>
void launch_span(const Grids &g, State<T> &s, int cur, const Tile *tiles, int64_t ntiles, bool plasma, int nsteps,
                 hipStream_t st)
{
    const dim3 grid((unsigned)ntiles), blk(64 * kSpanWaves);
    if (plasma)
        hipLaunchKernelGGL((k_span<T, kSpanC[1], true, kSpanWaves>), grid, blk, 0, st, g, s, cur, tiles, ntiles, nsteps);
    else
        hipLaunchKernelGGL((k_span<T, kSpanC[0], false, kSpanWaves>), grid, blk, 0, st, g, s, cur, tiles, ntiles, nsteps);
}

template void launch_span<float>(const Grids &, State<float> &, int, const Tile *, int64_t, bool, int, hipStream_t);
template void launch_span<double>(const Grids &, State<double> &, int, const Tile *, int64_t, bool, int, hipStream_t);

// Workgroup tiles: one tile of WAVES * 64 * C nodes per workgroup, wave w
// holding the w-th run of 64*C nodes.  Edge values cross waves through LDS
// (two barriers per step, as in k_group), so only the tile's two ends
// carry a halo.  Every wave takes both exchanges once per step on either
// path, so the barrier counts match.  The tile builder keeps node n-1 off
// the first node of a wave (the Mur end reads its left neighbour with an
// in-wave move).
template <typename T, int C, int KLASS, int WAVES>
__global__ __launch_bounds__(WAVES * 64) void k_tiledw(Grids g, State<T> s, int cur, const Tile *tiles,
                                                       int64_t ntiles, int nsteps, int slot0)
{
    constexpr bool PLASMA = KLASS >= 1;
    constexpr bool CPML = KLASS == 2;
    typedef typename Chunk<T, C, PLASMA, CPML>::R R;
    __shared__ R ldsE[WAVES];
    __shared__ R ldsH[WAVES];
    const int lane = threadIdx.x & 63;
    const int w = uniform(threadIdx.x >> 6);
    const int64_t t = xcd_block(blockIdx.x, gridDim.x);
    if (t >= ntiles) return;                  // whole workgroup: no barrier is left waiting
    const Tile tl = tiles[t];
    const int b = tl.grid;
    const int64_t off = g.off[b], n = g.n[b];
    const int64_t wave_lo = (int64_t)tl.lo + (int64_t)w * 64 * C;
    const int64_t wave_hi = wave_lo + 64LL * C < tl.hi ? wave_lo + 64LL * C : tl.hi;
    const int64_t k0 = wave_lo + (int64_t)lane * C;
    Chunk<T, C, PLASMA, CPML> ck;
    chunk_load<T, C, PLASMA, CPML>(ck, g, s, cur, b, off, n, k0, tl.hi);
    const WaveRole role = wave_role<C>(g, b, n, wave_lo, wave_hi > wave_lo ? wave_hi : wave_lo);
    const bool probes = (tl.flags & TILE_PROBE) != 0;
    // probes this wave samples: tile outputs inside the wave's span
    const int64_t plo = tl.out_lo > wave_lo ? tl.out_lo : wave_lo;
    const int64_t phi = tl.out_hi < wave_hi ? tl.out_hi : wave_hi;
    auto er = [&](R e0) {
        if (lane == 0) ldsE[w] = e0;
        __syncthreads();
        R v = shfl_down1(e0);
        if (lane == 63) v = (w + 1 < WAVES) ? ldsE[w + 1] : (R)0;
        return v;
    };
    auto hl = [&](R h) {
        if (lane == 63) ldsH[w] = h;
        __syncthreads();
        R v = shfl_up1(h);
        if (lane == 0) v = (w > 0) ? ldsH[w - 1] : (R)0;
        return v;
    };
    WaveProbes wp;
    wp.n = 0;
    if (probes && plo < phi) wp = wave_probes_find<C>(g, b, wave_lo, plo, phi);
    if (!has_role(role) && wp.n == 0) {
        for (int st = 0; st < nsteps; ++st) chunk_step_plain<T, C, PLASMA, CPML>(ck, g, er, hl);
    } else {
        run_role<T, C, PLASMA, CPML>(ck, g, role, wp, lane, b, wave_lo, plo, phi, nsteps, slot0, er, hl,
                                     [](int) {});
    }
    chunk_store<T, C, PLASMA, CPML>(ck, g, s, cur ^ 1, b, off, n, k0, tl.out_lo, tl.out_hi);
}

template <typename T, int C, int WAVES>
void launch_tiledw_c(const Grids &g, State<T> &s, int cur, const Tile *tiles, int64_t ntiles, int klass,
                     int nsteps, int slot0, hipStream_t st)
{
    const dim3 grid((unsigned)ntiles), blk(WAVES * 64);
    // class 3 (role tiles) takes the plasma kernel, which holds both paths
    if (klass == 0)
        hipLaunchKernelGGL((k_tiledw<T, C, 0, WAVES>), grid, blk, 0, st, g, s, cur, tiles, ntiles, nsteps,
                           slot0);
    else if (klass == 2)
        hipLaunchKernelGGL((k_tiledw<T, C, 2, WAVES>), grid, blk, 0, st, g, s, cur, tiles, ntiles, nsteps,
                           slot0);
    else
        hipLaunchKernelGGL((k_tiledw<T, C, 1, WAVES>), grid, blk, 0, st, g, s, cur, tiles, ntiles, nsteps,
                           slot0);
}

template <typename T, int WAVES>
void launch_tiledw_w(const Grids &g, State<T> &s, int cur, const Tile *tiles, int64_t ntiles, int klass,
                     int C, int nsteps, int slot0, hipStream_t st)
{
    switch (C) {
    case 4: launch_tiledw_c<T, 4, WAVES>(g, s, cur, tiles, ntiles, klass, nsteps, slot0, st); break;
    default: launch_tiledw_c<T, 8, WAVES>(g, s, cur, tiles, ntiles, klass, nsteps, slot0, st); break;
    }
}

// The FP32 delta-form ablation (g.jdelta): every class with the field
// updates in FP32 registers and, where there is plasma, J and eq.(11) in
// FP32, for 256- and 512-node tiles (the host refuses other shapes for it).
template <typename T, int C>
bool launch_tiled_jf(const Grids &g, State<T> &s, int cur, const Tile *tiles, int64_t ntiles, int klass,
                     int nsteps, int slot0, hipStream_t st)
{
    if constexpr (sizeof(T) == 4 && (C == 4 || C == 8)) {
        const unsigned nb = (unsigned)((ntiles + 3) / 4);
        if (klass == 0)
            hipLaunchKernelGGL((k_tiled<T, C, 0, false, true>), dim3(nb), dim3(256), 0, st, g, s, cur, tiles,
                               ntiles, nsteps, slot0);
        else if (klass == 1)
            hipLaunchKernelGGL((k_tiled<T, C, 1, false, true>), dim3(nb), dim3(256), 0, st, g, s, cur, tiles,
                               ntiles, nsteps, slot0);
        else if (klass == 2)
            hipLaunchKernelGGL((k_tiled<T, C, 2, true, true>), dim3(nb), dim3(256), 0, st, g, s, cur, tiles,
                               ntiles, nsteps, slot0);
        else
            hipLaunchKernelGGL((k_tiled<T, C, 1, true, true>), dim3(nb), dim3(256), 0, st, g, s, cur, tiles,
                               ntiles, nsteps, slot0);
        return true;
    }
    return false;
}

template <typename T, int C, int KLASS, int RM>
void launch_roles(const Grids &g, State<T> &s, int cur, const Tile *tiles, int64_t ntiles, int nsteps,
                  int slot0, hipStream_t st)
{
    const unsigned nb = (unsigned)((ntiles + 3) / 4);
    hipLaunchKernelGGL((k_tiled<T, C, KLASS, true, false, RM>), dim3(nb), dim3(256), 0, st, g, s, cur, tiles,
                       ntiles, nsteps, slot0);
}

// A role group's tiles with the step compiled for its roles (256- and
// 512-node tiles; wider tiles take the full step).
template <typename T, int C, int KLASS>
void launch_role_group(const Grids &g, State<T> &s, int cur, const Tile *tiles, int64_t ntiles, int group,
                       int nsteps, int slot0, hipStream_t st)
{
    if constexpr (C == 4 || C == 8) {
        switch (group) {
        case 0: return launch_roles<T, C, KLASS, kRoleProbe>(g, s, cur, tiles, ntiles, nsteps, slot0, st);
        case 1:
            return launch_roles<T, C, KLASS, kRoleSrc | kRoleProbe>(g, s, cur, tiles, ntiles, nsteps, slot0, st);
        case 2:
            return launch_roles<T, C, KLASS, kRoleLeft | kRoleProbe>(g, s, cur, tiles, ntiles, nsteps, slot0, st);
        case 3:
            return launch_roles<T, C, KLASS, kRoleRight | kRoleProbe>(g, s, cur, tiles, ntiles, nsteps, slot0,
                                                                     st);
        case 4:
            return launch_roles<T, C, KLASS, kRoleLeft | kRoleSrc | kRoleProbe>(g, s, cur, tiles, ntiles, nsteps,
                                                                               slot0, st);
        case -1: return launch_roles<T, C, KLASS, -1>(g, s, cur, tiles, ntiles, nsteps, slot0, st);
        default: break;
        }
        if constexpr (KLASS == 1) {
            // the fixed-register role step (TILE_FIXED tiles; role tiles only)
            constexpr int F = kRoleFixed | kRoleProbe;
            switch (group) {
            case 5: return launch_roles<T, C, KLASS, F>(g, s, cur, tiles, ntiles, nsteps, slot0, st);
            case 6: return launch_roles<T, C, KLASS, F | kRoleSrc>(g, s, cur, tiles, ntiles, nsteps, slot0, st);
            case 7: return launch_roles<T, C, KLASS, F | kRoleLeft>(g, s, cur, tiles, ntiles, nsteps, slot0, st);
            case 8: return launch_roles<T, C, KLASS, F | kRoleRight>(g, s, cur, tiles, ntiles, nsteps, slot0, st);
            case 9:
                return launch_roles<T, C, KLASS, F | kRoleLeft | kRoleSrc>(g, s, cur, tiles, ntiles, nsteps, slot0,
                                                                           st);
            default: break;
            }
        }
    }
    launch_roles<T, C, KLASS, kRoleAll>(g, s, cur, tiles, ntiles, nsteps, slot0, st);
}

template <typename T, int C>
void launch_tiled_c(const Grids &g, State<T> &s, int cur, const Tile *tiles, int64_t ntiles,
                    int klass, int nsteps, int slot0, hipStream_t st, int group)
{
    const unsigned nb = (unsigned)((ntiles + 3) / 4);
    if (g.jdelta && launch_tiled_jf<T, C>(g, s, cur, tiles, ntiles, klass, nsteps, slot0, st))
        return;
    if (klass == 0)
        hipLaunchKernelGGL((k_tiled<T, C, 0, false>), dim3(nb), dim3(256), 0, st, g, s, cur, tiles, ntiles,
                           nsteps, slot0);
    else if (klass == 1)
        hipLaunchKernelGGL((k_tiled<T, C, 1, false>), dim3(nb), dim3(256), 0, st, g, s, cur, tiles, ntiles,
                           nsteps, slot0);
    else if (klass == 2)
        launch_role_group<T, C, 2>(g, s, cur, tiles, ntiles, group, nsteps, slot0, st);
    else   // role tiles, vacuum or plasma: the plasma step reproduces the vacuum one
        launch_role_group<T, C, 1>(g, s, cur, tiles, ntiles, group, nsteps, slot0, st);
}

// Wide vacuum tiles (class 0 with a vacuum tile width of 1536 or 2048 nodes):
// the vacuum step only, the other classes are never this wide.
template <typename T, int C>
void launch_vacuum_c(const Grids &g, State<T> &s, int cur, const Tile *tiles, int64_t ntiles, int nsteps,
                     int slot0, hipStream_t st)
{
    const unsigned nb = (unsigned)((ntiles + 3) / 4);
    hipLaunchKernelGGL((k_tiled<T, C, 0, false>), dim3(nb), dim3(256), 0, st, g, s, cur, tiles, ntiles, nsteps,
                       slot0);
}

template <typename T>
void launch_tiled(const Grids &g, State<T> &s, int cur, const Tile *tiles, int64_t ntiles, int klass,
                  int C, int nsteps, int slot0, hipStream_t st, int waves, int group)
{
    if (waves == 2) return launch_tiledw_w<T, 2>(g, s, cur, tiles, ntiles, klass, C, nsteps, slot0, st);
    if (waves == 4) return launch_tiledw_w<T, 4>(g, s, cur, tiles, ntiles, klass, C, nsteps, slot0, st);
    if (waves == 8) return launch_tiledw_w<T, 8>(g, s, cur, tiles, ntiles, klass, C, nsteps, slot0, st);
    switch (C) {
    case 4: launch_tiled_c<T, 4>(g, s, cur, tiles, ntiles, klass, nsteps, slot0, st, group); break;
    case 8: launch_tiled_c<T, 8>(g, s, cur, tiles, ntiles, klass, nsteps, slot0, st, group); break;
    case 12: launch_tiled_c<T, 12>(g, s, cur, tiles, ntiles, klass, nsteps, slot0, st, group); break;
    case 24:
        if (klass == 0) launch_vacuum_c<T, 24>(g, s, cur, tiles, ntiles, nsteps, slot0, st);
        break;
    case 32:
        if (klass == 0) launch_vacuum_c<T, 32>(g, s, cur, tiles, ntiles, nsteps, slot0, st);
        break;
    default: launch_tiled_c<T, 16>(g, s, cur, tiles, ntiles, klass, nsteps, slot0, st, group); break;
    }
}

template void launch_tiled<float>(const Grids &, State<float> &, int, const Tile *, int64_t, int, int,
                                  int, int, hipStream_t, int, int);
template void launch_tiled<double>(const Grids &, State<double> &, int, const Tile *, int64_t, int,
                                   int, int, int, hipStream_t, int, int);

// ------------------------------------------------------------- resident

// One workgroup a group (a whole grid, or a segment of one).  Each wave owns a
// run of nodes and holds kGroupHalo more on each side that another wave owns;
// it recomputes those, so waves meet only every
// kGroupHalo steps, when the owners' values of E, H and Q replace the
// halo's through LDS (psi never: a CPML layer lies in
// its wave's own nodes), one barrier a meeting (two copies of the buffer: a wave
// may write the next meeting's values while a slower one still reads this
// one's).  A step then has no barrier, and its cost is the issue of the waves
// that share a SIMD: 1000 cells, 4096 steps, 2.22 -> 0.62 ms against the layout
// with two barriers a step and 512 nodes a wave (151 ns a step, the pace of the
// wave that holds an end, the source and a probe).
//
// What a wave with a grid end, the source or a probe does besides is kept to a
// few instructions a step (such a wave sets the pace of its grid): the source
// value comes from a table in LDS, zero for every lane and register but its
// own, and is added to all; the lane of a probe writes its nodes' E to the
// block's sample buffer and the others to a slot nobody reads.  Neither needs
// a branch, an exec mask or a register picked at run time.
//
// BINS: a workgroup holds several groups, dealt to its waves by a table (bins of
// build_bins); then every wave has a source table of its own.
template <int C, int WAVES, bool BINS>
struct GroupLds {
    double edge[2][2][WAVES][3][kGroupHalo];    // [copy][left, right edge of the wave's own nodes][E, H, Q]
    double src[BINS ? WAVES : 2][64][C];      // 64 steps' source values [wave; owner, halo][step][register]
    double zero[C];
    double probe[WAVES][2][kGroupHalo][C];      // the block's E of the lane holding each of two probes
    double sink[64][C];
};

// Wave w of the workgroup as wave gw of its group.
template <typename T, int C, int WAVES, bool BINS, bool PLASMA, bool CPML, int ROLE>
__device__ __forceinline__ void group_wave(const Grids &g, const State<T> &s, int cur, int out, const Group &gr,
                                           const GroupWave &wv, GroupLds<C, WAVES, BINS> &lds, int w, int gw,
                                           int lane, int nsteps, int slot0)
{
    typedef Chunk<T, C, PLASMA, CPML> K;
    typedef typename K::R R;
    constexpr bool GENERAL = ROLE == kResGeneral, ENDS = ROLE == kResEnds || GENERAL;
    const int b = gr.grid;
    const int64_t off = g.off[b], n = g.n[b];
    const bool has_l = wv.left, has_r = wv.right;
    const int hold_hi = wv.own_hi + (has_r ? kGroupHalo : 0);
    const int st_lo = wv.own_lo > gr.store_lo ? wv.own_lo : gr.store_lo;
    const int st_hi = wv.own_hi < gr.store_hi ? wv.own_hi : gr.store_hi;
    const int64_t k0 = (int64_t)wv.lo + (int64_t)lane * C;
    K ck;
    chunk_load<T, C, PLASMA, CPML>(ck, g, s, cur, b, off, n, k0, hold_hi);
    // a run may store into the buffer it was loaded from: every wave has its
    // values before any wave goes on
#pragma unroll
    for (int i = 0; i < C; ++i) {
        ck.E[i] = opaque(ck.E[i]);
        ck.H[i] = opaque(ck.H[i]);
        if constexpr (PLASMA) ck.J[i] = opaque(ck.J[i]);
        if constexpr (CPML) {
            ck.pE[i] = opaque(ck.pE[i]);
            ck.pH[i] = opaque(ck.pH[i]);
        }
    }

    WaveRole role = {-1, 0, -1, 0, -1, 1};
    WaveProbes wp;
    wp.n = 0;
    EndCarry<R> ends = {};
    double *src_tab = nullptr;
    if constexpr (ROLE != kResPlain) {
        role = wave_role<C>(g, b, n, wv.lo, hold_hi);
        wp = wave_probes_find<C>(g, b, wv.lo, st_lo, st_hi);
        ends_init<R, C, !ENDS>(ck.E, role, ends);
        // the two waves that may hold the source: the one that owns its node,
        // and a neighbour in its halo
        const int64_t sn = g.src[b];
        src_tab = &lds.src[BINS ? w : role.src_lane >= 0 && sn >= wv.own_lo && sn < wv.own_hi ? 0 : 1][0][0];
        if (w == 0 && lane < C) lds.zero[lane] = 0.0;
        if (role.src_lane >= 0) {
#pragma unroll
            for (int i = 0; i < C; ++i) src_tab[lane * C + i] = 0.0;
        }
    }
    if (ROLE == kResPlain && w == 0 && lane < C) lds.zero[lane] = 0.0;
    __syncthreads();
    // the source values of 64 steps, a step a lane, loaded 64 steps ahead
    auto source_run = [&](int i) { return g.srcv[i + lane < g.SB ? i + lane : g.SB - 1]; };
    double sv_next = 0.0;
    if constexpr (ROLE != kResPlain) {
        if (role.src_lane >= 0) sv_next = source_run(slot0);
    }
    const bool mur = g.bc == 0;
    const double *src_at = lds.zero;          // this lane's source values, a step apart (or the zeros)
    double *probe_at[2] = {&lds.sink[lane][0], &lds.sink[lane][0]};
    const int src_stride = ROLE != kResPlain && lane == role.src_lane ? C : 0;

    auto step = [&](int st) {
        double add[C];
        if constexpr (ROLE != kResPlain) {
#pragma unroll
            for (int i = 0; i < C; ++i) add[i] = src_at[i];
            src_at += src_stride;
        }
        chunk_h<T, C, PLASMA, CPML>(ck, shfl_down1(ck.E[0]));
        chunk_e<T, C, PLASMA, CPML>(ck, shfl_up1(ck.H[C - 1]));
        if constexpr (ROLE != kResPlain) {
#pragma unroll
            for (int i = 0; i < C; ++i) ck.E[i] = ck.E[i] + add[i];
        }
        if constexpr (ROLE == kResLeft) {           // node 0: register 0 of lane 0
            const R v = CPML ? (R)0 : (R)(ends.e1 + (R)g.cm * (ck.E[1] - ends.e0));
            ends.e1 = ck.E[1];
            ends.e0 = v;
            ck.E[0] = lane == 0 ? v : ck.E[0];
        } else if constexpr (ROLE == kResRight) {   // node n-1: the last register of lane 63
            const R en1 = ck.E[C - 2];
            const R v = CPML ? (R)0 : (R)(ends.eR1 + (R)g.cm * (en1 - ends.eR));
            ends.eR = v;
            ends.eR1 = en1;
            ck.E[C - 1] = lane == 63 ? v : ck.E[C - 1];
        } else if constexpr (ENDS) {                // either end or both, without a branch
            const R vl = mur ? (R)(ends.e1 + (R)g.cm * (ck.E[1] - ends.e0)) : (R)0;
            ends.e1 = ck.E[1];
            ends.e0 = vl;
            const R prev = shfl_up1(ck.E[C - 1]);
            R en1 = prev;
#pragma unroll
            for (int i = 1; i < C; ++i) en1 = role.right_reg == i ? ck.E[i - 1] : en1;
            const R vr = mur ? (R)(ends.eR1 + (R)g.cm * (en1 - ends.eR)) : (R)0;
            ends.eR = vr;
            ends.eR1 = en1;
            ck.E[0] = lane == role.left_lane ? vl : ck.E[0];
            uput<R, C>(ck.E, role.right_reg, lane == role.right_lane, vr);
        }
        if constexpr (GENERAL) {
            if (wp.n > 0) wave_probes<R, C>(g, b, wv.lo, st_lo, st_hi, lane, ck.E, slot0 + st);
        }
        if constexpr (ROLE != kResPlain && !GENERAL) {
#pragma unroll
            for (int p = 0; p < 2; ++p) {
#pragma unroll
                for (int i = 0; i < C; ++i) probe_at[p][i] = ck.E[i];
                probe_at[p] += wp.n > p && lane == wp.lane[p] ? C : 0;
            }
        }
    };

    for (int base = 0; base < nsteps; base += kGroupHalo) {
        if (base > 0) {
            // meet: this wave's edge nodes out, the halo's nodes in
            const int c = (base / kGroupHalo) & 1;
            // Q crosses only between waves that both carry it: a vacuum
            // wave's nodes keep Q = 0 on both sides
            const bool ql = PLASMA && has_l && ((gr.plasma >> (gw - 1)) & 1), qr = PLASMA && ((gr.plasma >> (gw + 1)) & 1);
#pragma unroll
            for (int i = 0; i < C; ++i) {
                const int l = (int)(k0 + i) - wv.own_lo, r = (int)(k0 + i) - (wv.own_hi - kGroupHalo);
#pragma unroll
                for (int side = 0; side < 2; ++side) {
                    const int at = side == 0 ? l : r;
                    if ((side == 0 ? has_l : has_r) && at >= 0 && at < kGroupHalo) {
                        lds.edge[c][side][w][0][at] = ck.E[i];
                        lds.edge[c][side][w][1][at] = ck.H[i];
                        if constexpr (PLASMA) lds.edge[c][side][w][2][at] = ck.J[i];
                    }
                }
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < C; ++i) {
                const int l = (int)(k0 + i) - (wv.own_lo - kGroupHalo), r = (int)(k0 + i) - wv.own_hi;
#pragma unroll
                for (int side = 0; side < 2; ++side) {
                    const int at = side == 0 ? l : r;
                    if ((side == 0 ? has_l : has_r) && at >= 0 && at < kGroupHalo) {
                        const int from = side == 0 ? w - 1 : w + 1;
                        ck.E[i] = lds.edge[c][side ^ 1][from][0][at];
                        ck.H[i] = lds.edge[c][side ^ 1][from][1][at];
                        if constexpr (PLASMA) {
                            if (side == 0 ? ql : qr) ck.J[i] = lds.edge[c][side ^ 1][from][2][at];
                        }
                    }
                }
            }
        }
        const int cnt = nsteps - base < kGroupHalo ? nsteps - base : kGroupHalo;
        if constexpr (ROLE != kResPlain) {
            if (role.src_lane >= 0 && (base & 63) == 0) {
                src_tab[lane * C + role.src_reg] = sv_next;
                sv_next = source_run(slot0 + base + 64);
                if (src_stride) src_at = src_tab;
            }
            if constexpr (!GENERAL) {
#pragma unroll
                for (int p = 0; p < 2; ++p)
                    if (wp.n > p && lane == wp.lane[p]) probe_at[p] = &lds.probe[w][p][0][0];
            }
            __builtin_amdgcn_wave_barrier();
        }
        int st = 0;
        for (; st + 2 <= cnt; st += 2) {
            step(base + st);
            step(base + st + 1);
        }
        if (st < cnt) step(base + st);
        if constexpr (ROLE != kResPlain && !GENERAL) {
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int p = 0; p < 2; ++p)
                if (wp.n > p && lane < cnt) g.samp[wp.row[p] + slot0 + base + lane] = lds.probe[w][p][lane][wp.reg[p]];
            __builtin_amdgcn_wave_barrier();
        }
    }
    chunk_store<T, C, PLASMA, CPML>(ck, g, s, out, b, off, n, k0, st_lo, st_hi);
}

template <typename T, int C, int WAVES, bool BINS>
__global__ __launch_bounds__(WAVES * 64) void k_group(Grids g, State<T> s, int cur, int out, const Group *groups,
                                                      const int32_t *bins, int nsteps, int slot0)
{
    __shared__ GroupLds<C, WAVES, BINS> lds;
    const int lane = threadIdx.x & 63;
    const int w = uniform(threadIdx.x >> 6);
    int64_t at = blockIdx.x;
    int gw = w;
    bool idle = false;
    if constexpr (BINS) {
        if (bins) {
            const int32_t e = bins[(int64_t)blockIdx.x * (blockDim.x >> 6) + w];
            idle = e < 0;
            at = idle ? 0 : e >> kBinShift;
            gw = e & ((1 << kBinShift) - 1);
        }
    }
    const Group gr = groups[at];
    // every path takes the same barriers: one after its loads, one a meeting
    if (idle || gw >= gr.nwaves) {
        __syncthreads();
        for (int base = kGroupHalo; base < nsteps; base += kGroupHalo) __syncthreads();
        return;
    }
    const GroupWave wv = group_wave_at(gr, gw, C);
    const int role = (gw < 10 ? gr.role[0] >> (3 * gw) : gr.role[1] >> (3 * (gw - 10))) & 7;
#define FDTDP_WAVE(PLASMA, CPML, ROLE) \
    group_wave<T, C, WAVES, BINS, PLASMA, CPML, ROLE>(g, s, cur, out, gr, wv, lds, w, gw, lane, nsteps, slot0)
    // layers at two nodes a lane only (kCpmlC; the register file)
    if constexpr (C == kCpmlC) {
        if ((gr.cpml >> gw) & 1) {
            if ((gr.plasma >> gw) & 1) {
                FDTDP_WAVE(true, true, kResGeneral);
            } else {
                switch (role) {
                case kResLeft: FDTDP_WAVE(false, true, kResLeft); break;
                case kResRight: FDTDP_WAVE(false, true, kResRight); break;
                default: FDTDP_WAVE(false, true, kResGeneral); break;
                }
            }
            return;
        }
    }
    if ((gr.plasma >> gw) & 1) {
        switch (role) {
        case kResPlain: FDTDP_WAVE(true, false, kResPlain); break;
        case kResInner: FDTDP_WAVE(true, false, kResInner); break;
        case kResLeft: FDTDP_WAVE(true, false, kResLeft); break;
        case kResRight: FDTDP_WAVE(true, false, kResRight); break;
        case kResEnds: FDTDP_WAVE(true, false, kResEnds); break;
        default: FDTDP_WAVE(true, false, kResGeneral); break;
        }
    } else {
        switch (role) {
        case kResPlain: FDTDP_WAVE(false, false, kResPlain); break;
        case kResInner: FDTDP_WAVE(false, false, kResInner); break;
        case kResLeft: FDTDP_WAVE(false, false, kResLeft); break;
        case kResRight: FDTDP_WAVE(false, false, kResRight); break;
        case kResEnds: FDTDP_WAVE(false, false, kResEnds); break;
        default: FDTDP_WAVE(false, false, kResGeneral); break;
        }
    }
#undef FDTDP_WAVE
}

// Groups of two nodes a lane, one a workgroup: segments, and whole grids (the
// instance with bins takes FP32's 1000 nodes, 4096 steps, in 0.70 ms instead of
// 0.67, and one of eight waves the segments of a pass 1% longer).
template <typename T>
void launch_alone(const Grids &g, State<T> &s, int cur, int out, const Group *groups, int64_t n, int waves, int nsteps,
                  int slot0, hipStream_t st)
{
    hipLaunchKernelGGL((k_group<T, kGroupShapes[0].C, kGroupShapes[0].waves, false>), dim3((unsigned)n),
                       dim3((unsigned)(64 * waves)), 0, st, g, s, cur, out, groups, (const int32_t *)nullptr, nsteps, slot0);
}

template <typename T>
void launch_bins(const Grids &g, State<T> &s, int cur, int out, const Group *groups, const int32_t *bins, int64_t nbins,
                 int waves, int C, int nsteps, int slot0, hipStream_t st)
{
    if (!bins && C == kGroupShapes[0].C)
        return launch_alone<T>(g, s, cur, out, groups, nbins, waves, nsteps, slot0, st);
    const dim3 grid((unsigned)nbins), blk((unsigned)(64 * waves));
#define FDTDP_GROUP(I)                                                                                            \
    hipLaunchKernelGGL((k_group<T, kGroupShapes[I].C, kGroupShapes[I].waves, true>), grid, blk, 0, st, g, s, cur, \
                       out, groups, bins, nsteps, slot0)
    if (C == kGroupShapes[0].C) FDTDP_GROUP(0);
    else if (C == kGroupShapes[1].C) FDTDP_GROUP(1);
    else FDTDP_GROUP(2);
#undef FDTDP_GROUP
}

template <typename T>
void launch_segments(const Grids &g, State<T> &s, int cur, const Group *segs, int64_t nseg, int waves, int nsteps,
                     int slot0, hipStream_t st)
{
    launch_alone<T>(g, s, cur, cur ^ 1, segs, nseg, waves, nsteps, slot0, st);
}

#define FDTDP_INST(T)                                                                                             \
    template void launch_bins<T>(const Grids &, State<T> &, int, int, const Group *, const int32_t *, int64_t, int, \
                                 int, int, int, hipStream_t);                                                     \
    template void launch_segments<T>(const Grids &, State<T> &, int, const Group *, int64_t, int, int, int, hipStream_t);
FDTDP_INST(float)
FDTDP_INST(double)
#undef FDTDP_INST

}  // namespace fdtdp
