// 3D Yee-RKETD kernels.  One time step is either
//   k_h3d   H^{n+1/2} from E^n (CPML auxiliaries, TF/SF H corrections fused)
//   k_e3d   E^{n+1} (CPML, TF/SF E corrections or the planar source, PEC walls)
//           and J^{n+1} on the plasma support, fused
// (two passes over the grid, in place), or k_fused3d (one pass, E/H/CPML
// ping-pong); both call the same per-cell h_cell / e_cell and give identical
// bits.  The incident 1D grid (TF/SF only) is 32 steps ahead at a time
// (k_aux3d).  The sample points go into the current slot of the sample buffer
// (by the passes themselves, or k_sample3d), and every `slots` steps k_tw3d +
// k_flush3d fold the buffered samples into the
// FP64 DFT accumulators.
//
// The update formulas are the 1D library's per-node physics (physics.h): H by
// one FMA per component, E in vacuum by one FMA, plasma E by the solved
// eqs.(11)+(12) (FP32: delta form around CA - 1), J by eq.(11) in FP64.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "internal3d.h"

namespace fdtdp {

namespace {

// Consecutive logical blocks on one XCD: the hardware deals workgroups to the
// 8 XCDs round-robin, so hardware block b runs on XCD b % 8; give that XCD the
// b / 8-th block of its own contiguous chunk.  Neighbouring i-planes then share
// an L2.
__device__ __forceinline__ int64_t xcd_chunk(int64_t bid, int64_t nblk)
{
    const int64_t q = nblk / 8, r = nblk % 8;
    const int64_t x = bid % 8, j = bid / 8;
    return x * q + (x < r ? x : r) + j;
}

// Cells of a split-kernel workgroup: 64 consecutive k (one wave) x 4 rows j
// x a run of g.np planes i that each thread walks.  i and j are the
// same for the whole wave (kept in scalar registers).
struct Col {
    int64_t i0, i1, j, k, k0;     // k0: the wave's first node
    bool ok;
};

__device__ __forceinline__ Col col_of(const Geo3 &g, int64_t nblk)
{
    Col c;
    const int64_t bid = xcd_chunk(blockIdx.x, nblk);
    const int64_t kq = bid % g.kb, r = bid / g.kb;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    c.j = (r % g.jb) * 4 + w;
    c.i0 = g.ia + (r / g.jb) * g.np;
    c.i1 = c.i0 + g.np < g.ib ? c.i0 + g.np : g.ib;
    c.k0 = kq * 64;
    c.k = c.k0 + (threadIdx.x & 63);
    c.ok = c.j < g.ny && c.k < g.nz;
    return c;
}

// slab index of node n on an axis of `len` nodes with P-node layers, or -1
__device__ __forceinline__ int slab(int64_t n, int64_t len, int P)
{
    if (n < P) return (int)n;
    if (n >= len - P) return (int)(n - (len - 2 * P));
    return -1;
}

// Where one cell lies in the CPML layers.  i and j are the same for the whole
// wave, so the x and y layers are scalar branches.  Every axis reads its
// auxiliaries when the update comes to it: read together before any arithmetic they
// take 24 more registers in FP64 (H pass 6 -> 4 waves a SIMD, E pass 4 -> 3; 200^3 181 +
// 302 -> 192 + 323 us a step).
struct Layers {
    int s[3];                     // place in the layer, -1 outside it
    int64_t at[3];                // element of its auxiliary arrays
};

// An element of a wave's row: the same start for all lanes, a byte offset each
// (one vector register, not an address pair for every array).
template <typename T>
__device__ __forceinline__ T &elem(T *f, int64_t base, uint32_t off)
{
    using C = std::conditional_t<std::is_const_v<T>, const char, char>;
    return *(T *)((C *)(f + base) + off);
}

__device__ __forceinline__ Layers layers_of(const Geo3 &g, int64_t i, int64_t j, int64_t k)
{
    Layers q;
    const int P = g.P, P2 = 2 * g.P;
    q.s[0] = P > 0 && !g.px ? slab(i, g.nx, P) : -1;
    q.s[1] = P > 0 && !g.py ? slab(j, g.ny, P) : -1;
    q.s[2] = P > 0 ? slab(k, g.nz, P) : -1;
    q.at[0] = ((int64_t)q.s[0] * g.ny + j) * g.nz + k;
    q.at[1] = (i * P2 + q.s[1]) * g.nz + k;
    q.at[2] = (i * g.ny + j) * P2 + q.s[2];
    return q;
}

// psi' = b psi + a dF for both derivatives across axis x (separately rounded,
// as written; row: of b in the table), stored only by the cell's owner; each dF
// gains its psi'.
template <typename T>
__device__ __forceinline__ void layers_add(const Layers &q, int x, const T *tab, int P, int row, const T *const (&pin)[3][2],
                                           T *const (&pout)[3][2], T &d0, T &d1, bool store)
{
    if (q.s[x] < 0) return;
    const T b = tab[(x * 4 + row) * 2 * P + q.s[x]], a = tab[(x * 4 + row + 1) * 2 * P + q.s[x]];
    const T v0 = b * pin[x][0][q.at[x]] + a * d0, v1 = b * pin[x][1][q.at[x]] + a * d1;
    if (store) {
        pout[x][0][q.at[x]] = v0;
        pout[x][1][q.at[x]] = v1;
    }
    d0 = d0 + v0;
    d1 = d1 + v1;
}

}  // namespace

// H^{n+1/2} of cell (i, j, k) from its E^n and the E^n of its +1 neighbours
// (zero beyond a wall); hx, hy, hz hold H^{n-1/2} on entry.  CPML auxiliaries
// and the TF/SF correction (Einc^n) included.  Shared by both executors.
template <typename T>
__device__ __forceinline__ void h_cell(const Geo3 &g, const Cpml3<T> &c, const double *Einc, int64_t i, int64_t j,
                                       int64_t k, T ex, T ey, T ez, T ex_j, T ex_k, T ey_i, T ey_k, T ez_i, T ez_j,
                                       T &hx, T &hy, T &hz, bool store)
{
    T dEz_y = ez_j - ez;
    T dEy_z = ey_k - ey;
    T dEx_z = ex_k - ex;
    T dEz_x = ez_i - ez;
    T dEy_x = ey_i - ey;
    T dEx_y = ex_j - ex;
    const Layers q = layers_of(g, i, j, k);
    layers_add(q, 0, c.tab, g.P, 2, c.inH, c.outH, dEz_x, dEy_x, store);
    layers_add(q, 1, c.tab, g.P, 2, c.inH, c.outH, dEz_y, dEx_y, store);
    layers_add(q, 2, c.tab, g.P, 2, c.inH, c.outH, dEy_z, dEx_z, store);
    const T ch = (T)g.chd;
    hx = fmat(-ch, dEz_y - dEy_z, hx);
    hy = fmat(-ch, dEx_z - dEz_x, hy);
    hz = fmat(-ch, dEy_x - dEx_y, hz);
    if (g.src == 2) {
        // scattered H beside the box reads total Ex across a face: remove the
        // incident part (Einc^n).  Hy(k+1/2) at k = b0-1 and b1; Hz(j+1/2) at
        // j = b0-1 and b1 (walled y), with the minus sign of dEx/dy in curl_z.
        const bool inx = i >= g.xlo && i < g.xhi;
        if (inx && j >= g.ylo && j < g.yhi) {
            if (k == g.b0 - 1) hy = hy + (T)(g.chd * Einc[g.b0 + g.ao]);
            else if (k == g.b1) hy = hy - (T)(g.chd * Einc[g.b1 + g.ao]);
        }
        if (!g.py && inx && k >= g.b0 && k <= g.b1) {
            if (j == g.b0 - 1) hz = hz - (T)(g.chd * Einc[k + g.ao]);
            else if (j == g.b1) hz = hz + (T)(g.chd * Einc[k + g.ao]);
        }
    }
}

// The J triple of component c
template <typename T>
__device__ __forceinline__ void j_coef_at(const Plasma3<T> &pl, int c, int64_t base, uint32_t off, NodeCoef<T> &r)
{
    const double a = (double)elem(pl.ca[c], base, off);
    r.a = sizeof(T) == 8 ? a : 1.0 + a;
    r.b1 = (double)elem(pl.cb1[c], base, off);
    r.b2 = (double)elem(pl.cb2[c], base, off);
}

// Coefficient tables of the plasma support (once per create): node_coef of
// physics.h per node and component.
template <typename T>
__global__ void k_coef3d(const double *w0, const double *w1, const double *w2, const double *n0,
                         const double *n1, const double *n2, int64_t S, double dt, double d, T *eA0, T *eA1,
                         T *eA2, T *eJ0, T *eJ1, T *eJ2, T *eH0, T *eH1, T *eH2, T *a0, T *a1, T *a2,
                         T *b10, T *b11, T *b12, T *b20, T *b21, T *b22)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= S) return;
    const double *w[3] = {w0, w1, w2}, *n[3] = {n0, n1, n2};
    T *eA[3] = {eA0, eA1, eA2}, *eJ[3] = {eJ0, eJ1, eJ2}, *eH[3] = {eH0, eH1, eH2};
    T *a[3] = {a0, a1, a2}, *b1[3] = {b10, b11, b12}, *b2[3] = {b20, b21, b22};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const NodeCoef<T> r = node_coef_t<T>(w[c][q], n[c][q], dt, d, 0);
        eA[c][q] = r.eA;
        eJ[c][q] = r.eJ;
        eH[c][q] = r.eH;
        a[c][q] = sizeof(T) == 8 ? (T)r.a : (T)(r.a - 1.0);   // a in [1/2, 1]: a - 1 exact
        b1[c][q] = (T)r.b1;
        b2[c][q] = (T)r.b2;
    }
}

// The plasma terms of one cell, read before its E update (with its field
// values, so that no load waits on another): whether the cell is on the
// support, its compact index, J^n and the stored coefficients of the three
// components.  sp, off: the span and offset of the cell's row.
// FP64's J triples are read when their component comes to them instead: with all
// 21 doubles of a cell in flight the kernel holds 2 waves a SIMD, without 3 (256^3 sphere
// E pass 511 -> 472 us; FP32, 4 waves either way, loses 745 -> 831 at 384^3).
template <typename T>
constexpr bool kLateJ = sizeof(T) == 8;

template <typename T>
struct PNode {
    bool on;
    int64_t base;                 // compact index: of the wave's node k0 (or the lane's own), in elements,
    uint32_t off;                 // and of the lane past it, in bytes (or none)
    T J[3];
    NodeCoef<T> cf[3];
};

// ROW: scalar row starts and a lane offset (elem), else one index a lane.  The E
// pass takes the first in its plain way in FP64 (160^3 all plasma 220 us against 226)
// and the second elsewhere (200^3 FP32 sphere 161 against 166-193, by the registers; the
// one-pass kernel 136 VGPRs against 219 with the layers' too, 160^3 FP32 220 us a step against 300).
template <bool ROW, typename T>
__device__ __forceinline__ PNode<T> pnode_load(const Plasma3<T> &pl, int2 sp, int64_t off, int64_t k0, uint32_t lane)
{
    PNode<T> n;
    const int64_t k = k0 + lane;
    n.on = k >= sp.x && k < sp.y;
    n.base = off + ((ROW ? k0 : k) - sp.x);
    n.off = ROW ? lane * (uint32_t)sizeof(T) : 0;
    if (n.on) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            n.J[c] = elem(pl.J[c], n.base, n.off);
            n.cf[c].eA = elem(pl.eA[c], n.base, n.off);
            n.cf[c].eJ = elem(pl.eJ[c], n.base, n.off);
            n.cf[c].eH = elem(pl.eH[c], n.base, n.off);
            if (!kLateJ<T>) j_coef_at(pl, c, n.base, n.off, n.cf[c]);
        }
    }
    return n;
}

// E update with the 3D curl sign: E_new = CA E - CJ J + CH curl.
__device__ __forceinline__ double e_plasma3(double E, double J, double curl, const NodeCoef<double> &c)
{
    return fmat(c.eH, curl, fmat(-c.eJ, J, c.eA * E));
}
__device__ __forceinline__ float e_plasma3(float E, float J, float curl, const NodeCoef<float> &c)
{
    return fmat(c.eH, curl, fmat(-c.eJ, J, fmat(c.eA, E, E)));
}

// The corrections of E component C after its update: TF/SF (the total E on
// a box face reads scattered H outside it, so it gains the incident part
// Hinc^{n+1/2} times its CH; Ex at k = b0, b1, Ez at i = b0, b1 of a walled
// x) or the planar source, then PEC (tangential E on the index-0 faces of the
// walled axes).
template <int C, typename T>
__device__ __forceinline__ T e_fix(const Geo3 &g, const double *Hinc, double sval, int64_t i, int64_t j,
                                   int64_t k, double CH, T e)
{
    if (g.src == 2) {
        if constexpr (C == 0) {
            if (i >= g.xlo && i < g.xhi && j >= g.ylo && j < g.yhi) {
                if (k == g.b0) e = e + (T)(CH * Hinc[g.b0 - 1 + g.ao]);
                else if (k == g.b1) e = e - (T)(CH * Hinc[g.b1 + g.ao]);
            }
        }
        if constexpr (C == 2) {
            if (!g.px && j >= g.ylo && j < g.yhi && k >= g.b0 && k < g.b1) {
                if (i == g.b0) e = e - (T)(CH * Hinc[k + g.ao]);
                else if (i == g.b1) e = e + (T)(CH * Hinc[k + g.ao]);
            }
        }
    } else if (g.src == 1 && k == g.src_k && g.src_comp == C) {
        e = add_source(e, sval);
    }
    const bool wx = !g.px && i == 0, wy = !g.py && j == 0, wz = k == 0;
    if ((C == 0 && (wy || wz)) || (C == 1 && (wx || wz)) || (C == 2 && (wx || wy))) e = (T)0;
    return e;
}

// E component C of a plasma node: the E update with its coefficients, the
// corrections, then J^{n+1} in place.
template <int C, typename T>
__device__ __forceinline__ T e_plasma_comp(const Geo3 &g, const Plasma3<T> &pl, const PNode<T> &pn,
                                           const double *Hinc, double sval, int64_t i, int64_t j, int64_t k,
                                           T curl, T eo)
{
    NodeCoef<T> cf = pn.cf[C];
    const T J = pn.J[C];
    if (kLateJ<T>) j_coef_at(pl, C, pn.base, pn.off, cf);
    const T e = e_fix<C>(g, Hinc, sval, i, j, k, (double)cf.eH, e_plasma3(eo, J, curl, cf));
    elem(pl.J[C], pn.base, pn.off) = (T)j_update<T>((double)J, (double)eo, (double)e, cf);
    return e;
}

// E^{n+1} of cell (i, j, k) from its H^{n+1/2} and the H^{n+1/2} of its -1
// neighbours (zero beyond a wall); e0..e2 hold E^n on entry.  CPML, TF/SF (or
// the planar source), PEC walls and, on the plasma support (pn, read by the
// caller), J^{n+1} (written in place).  Shared by both executors.
template <typename T>
__device__ __forceinline__ void e_cell(const Geo3 &g, const Plasma3<T> &pl, const PNode<T> &pn,
                                       const Cpml3<T> &c, const double *Hinc, double sval, int64_t i, int64_t j,
                                       int64_t k, T hx, T hy, T hz, T hx_j, T hx_k, T hy_i, T hy_k, T hz_i, T hz_j,
                                       T &e0, T &e1, T &e2)
{
    T dHz_y = hz - hz_j;
    T dHy_z = hy - hy_k;
    T dHx_z = hx - hx_k;
    T dHz_x = hz - hz_i;
    T dHy_x = hy - hy_i;
    T dHx_y = hx - hx_j;
    const Layers q = layers_of(g, i, j, k);
    layers_add(q, 0, c.tab, g.P, 0, c.inE, c.outE, dHz_x, dHy_x, true);
    layers_add(q, 1, c.tab, g.P, 0, c.inE, c.outE, dHz_y, dHx_y, true);
    layers_add(q, 2, c.tab, g.P, 0, c.inE, c.outE, dHy_z, dHx_z, true);
    const T curl0 = dHz_y - dHy_z, curl1 = dHx_z - dHz_x, curl2 = dHy_x - dHx_y;
    if (!pn.on) {
        const T ce = (T)g.ced;
        e0 = e_fix<0>(g, Hinc, sval, i, j, k, g.ced, fmat(ce, curl0, e0));
        e1 = e_fix<1>(g, Hinc, sval, i, j, k, g.ced, fmat(ce, curl1, e1));
        e2 = e_fix<2>(g, Hinc, sval, i, j, k, g.ced, fmat(ce, curl2, e2));
    } else {
        e0 = e_plasma_comp<0>(g, pl, pn, Hinc, sval, i, j, k, curl0, e0);
        e1 = e_plasma_comp<1>(g, pl, pn, Hinc, sval, i, j, k, curl1, e1);
        e2 = e_plasma_comp<2>(g, pl, pn, Hinc, sval, i, j, k, curl2, e2);
    }
}

// ---- two-kernel step (in place) --------------------------------------------
//
// Each thread walks g.np planes along x for one (j, k): the x
// neighbour it loads for plane i is its own value at plane i+1 (H kernel) or
// was its own value at plane i-1 (E kernel), so it is read once.
//
// Both passes are bound by memory, and by how many loads the waves keep on the
// way.  Most waves hold vacuum or plasma only, and for them a plane is its
// loads, a dozen adds and FMAs, and its stores: the wave tells by its place (the
// same for all its lanes) whether any of its cells has a layer, a TF face, a
// wall or the source, and only then goes the general way (h_cell, e_cell).
// Addresses are a scalar row start and a 32-bit lane offset.  What only the
// general way needs is read from the kernel's arguments there: the E kernel's
// hundred pointers and offsets, kept in scalar registers over the loop,
// spilled into lanes of vector registers, and most of its 353 vector
// instructions a plane moved spills and formed 64-bit addresses.  E + H of the
// 384^3 FP32 sphere 1335 -> 1297 us a step, and 1287 -> 1190 in slabs that the
// memory-side cache holds; 160^3 FP32 111 -> 105.  Reading the next plane ahead was
// slower (E 745 -> 896 us), as was a register limit for more waves (1150).
template <typename S>
using Const = const __attribute__((address_space(4))) S;

// A pointer loaded from the arguments is one to global memory.
template <typename S>
__device__ __forceinline__ S *global_ptr(S *p)
{
    return (S *)(__attribute__((address_space(1))) S *)p;
}

// The kernel's one argument struct, as memory that nothing is known about yet.
template <typename A>
__device__ __forceinline__ Const<A> *kernel_args()
{
    uint64_t p = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return (Const<A> *)p;
}

__device__ __forceinline__ Geo3 geo_arg(Const<Geo3> *s)
{
    static_assert(sizeof(Geo3) % 8 == 0, "whole words");
    Const<uint64_t> *from = (Const<uint64_t> *)s;
    uint64_t word[sizeof(Geo3) / 8];
#pragma unroll
    for (size_t n = 0; n < sizeof(Geo3) / 8; ++n) word[n] = from[n];
    Geo3 g;
    __builtin_memcpy(&g, word, sizeof g);
    return g;
}

template <typename T>
__device__ __forceinline__ Cpml3<T> cpml_arg(Const<Cpml3<T>> *a)
{
    Cpml3<T> c;
#pragma unroll
    for (int x = 0; x < 3; ++x)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            c.inH[x][q] = global_ptr(a->inH[x][q]);
            c.outH[x][q] = global_ptr(a->outH[x][q]);
            c.inE[x][q] = global_ptr(a->inE[x][q]);
            c.outE[x][q] = global_ptr(a->outE[x][q]);
        }
    c.tab = global_ptr(a->tab);
    return c;
}

template <typename T>
__device__ __forceinline__ Plasma3<T> plasma_arg(Const<Plasma3<T>> *a)
{
    Plasma3<T> p;
    p.span = nullptr;
    p.off = nullptr;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        p.J[c] = global_ptr(a->J[c]);
        p.eA[c] = global_ptr(a->eA[c]);
        p.eJ[c] = global_ptr(a->eJ[c]);
        p.eH[c] = global_ptr(a->eH[c]);
        p.ca[c] = global_ptr(a->ca[c]);
        p.cb1[c] = global_ptr(a->cb1[c]);
        p.cb2[c] = global_ptr(a->cb2[c]);
    }
    return p;
}

// Whether the wave's nodes [k0, k0 + 64) hold node x
__device__ __forceinline__ bool holds(int64_t k0, int64_t x) { return x >= k0 && x < k0 + 64; }

// Planes, of a walled x, on which every cell goes the general way: the layers
// and two more (-1: none)
struct Planes {
    int64_t lo, hi, f0, f1;
    __device__ __forceinline__ bool operator()(int64_t i) const { return i < lo || i >= hi || i == f0 || i == f1; }
};

// The n-th thread's sample point, if it has one
template <typename T>
__device__ __forceinline__ void sample(const Fields3<T> &f, int64_t N, const int64_t *pts, const int32_t *list,
                                       int64_t cnt, T *buf, int64_t n)
{
    if (n >= cnt) return;
    const int64_t q = list ? list[n] : n;
    const int64_t code = pts[q];
    const int c = (int)(code / N);
    const int64_t p = code - (int64_t)c * N;
    const T *src = c == 0 ? f.E[0] : c == 1 ? f.E[1] : c == 2 ? f.E[2] : c == 3 ? f.H[0] : c == 4 ? f.H[1] : f.H[2];
    buf[q] = src[p];
}

// Sample points read by workgroups of a split pass past its cells': by the E
// pass the H points (which it does not write), by the next step's H pass the E
// points.  As a launch of its own after each step they took 6 us of the 96^3
// sphere's 64.
template <typename T>
__device__ __forceinline__ bool sample_block(const Samples3<T> &s, const Fields3<T> &f)
{
    if ((int64_t)blockIdx.x < s.cells) return false;
    sample(f, s.N, s.pts, s.list, s.cnt, s.buf, ((int64_t)blockIdx.x - s.cells) * blockDim.x + threadIdx.x);
    return true;
}

template <typename T>
struct ArgsH3 {
    Geo3 g;
    Samples3<T> s;
    Fields3<T> f;
    Cpml3<T> c;
    const double *Einc;
};

template <typename T>
__global__ __launch_bounds__(256) void k_h3d(ArgsH3<T> arg)
{
    const Geo3 &g = arg.g;
    if (sample_block(arg.s, arg.f)) return;
    const Col q = col_of(g, arg.s.cells);
    if (!q.ok) return;
    const int64_t j = q.j, nx = g.nx;
    const int64_t sI = g.ny * g.nz;
    const bool px = g.px;
    const bool hasj = g.py || j + 1 < g.ny, hask = q.k + 1 < g.nz;
    const int64_t dj = j + 1 < g.ny ? g.nz : -j * g.nz;       // +1 row, periodic wrap
    const bool tf = g.src == 2;
    const bool spec = (g.P > 0 && (q.k0 < g.P || q.k0 + 63 >= g.nz - g.P)) ||
                      (tf && (holds(q.k0, g.b0 - 1) || holds(q.k0, g.b1))) ||
                      (!g.py && ((g.P > 0 && (j < g.P || j >= g.ny - g.P)) || (tf && (j == g.b0 - 1 || j == g.b1))));
    const Planes xspec{px ? 0 : g.P, px ? nx : nx - g.P, -1, -1};
    const T zero = (T)0, ch = (T)g.chd;
    const uint32_t lane = threadIdx.x & 63, l = lane * (uint32_t)sizeof(T), lk = hask ? l + (uint32_t)sizeof(T) : l;
    auto at = [](const T *f, int64_t p, uint32_t o) { return elem(f, p, o); };
    // p: the row's first node of the wave on plane i, and pn on plane i+1 (periodic
    // wrap to plane 0, or, beyond the wall, not used)
    auto next = [&](int64_t i, int64_t p) { return i + 1 < nx ? p + sI : p - i * sI; };
    int64_t p = (q.i0 * g.ny + j) * g.nz + q.k0;
    struct In {
        T e1[3], exj, ezj, exk, eyk, h[3];
    };
    auto load = [&](int64_t p, int64_t pn, In &v) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            v.e1[c] = at(arg.f.E[c], pn, l);
            v.h[c] = at(arg.f.H[c], p, l);
        }
        v.exj = at(arg.f.E[0], p + dj, l);
        v.ezj = at(arg.f.E[2], p + dj, l);
        v.exk = at(arg.f.E[0], p, lk);
        v.eyk = at(arg.f.E[1], p, lk);
    };
    T e[3] = {at(arg.f.E[0], p, l), at(arg.f.E[1], p, l), at(arg.f.E[2], p, l)};
    for (int64_t i = q.i0; i < q.i1; ++i) {
        const int64_t pn = next(i, p);
        In v;
        load(p, pn, v);
        const bool hasi = px || i + 1 < nx;
        const T ex_j = hasj ? v.exj : zero, ez_j = hasj ? v.ezj : zero;
        const T ex_k = hask ? v.exk : zero, ey_k = hask ? v.eyk : zero;
        const T ey_i = hasi ? v.e1[1] : zero, ez_i = hasi ? v.e1[2] : zero;
        if (!spec && !xspec(i)) {
            const T dEz_y = ez_j - e[2], dEy_z = ey_k - e[1], dEx_z = ex_k - e[0];
            const T dEz_x = ez_i - e[2], dEy_x = ey_i - e[1], dEx_y = ex_j - e[0];
            v.h[0] = fmat(-ch, dEz_y - dEy_z, v.h[0]);
            v.h[1] = fmat(-ch, dEx_z - dEz_x, v.h[1]);
            v.h[2] = fmat(-ch, dEy_x - dEx_y, v.h[2]);
        } else {
            Const<ArgsH3<T>> *s = kernel_args<ArgsH3<T>>();
            const Geo3 gs = geo_arg(&s->g);
            const Cpml3<T> c = cpml_arg<T>(&s->c);
            h_cell<T>(gs, c, global_ptr(s->Einc), i, j, q.k, e[0], e[1], e[2], ex_j, ex_k, ey_i, ey_k, ez_i, ez_j, v.h[0],
                      v.h[1], v.h[2], true);
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            elem(arg.f.H[c], p, l) = v.h[c];
            e[c] = v.e1[c];
        }
        p = pn;
    }
}

template <typename T>
struct ArgsE3 {
    Geo3 g;
    Samples3<T> s;
    Fields3<T> f;
    Plasma3<T> pl;
    Cpml3<T> c;
    const double *Hinc;
    double sval;
};

template <typename T>
__global__ __launch_bounds__(256) void k_e3d(ArgsE3<T> arg)
{
    const Geo3 &g = arg.g;
    if (sample_block(arg.s, arg.f)) return;
    const Col q = col_of(g, arg.s.cells);
    if (!q.ok) return;
    const int64_t j = q.j, ny = g.ny;
    const int64_t sI = ny * g.nz;
    const bool hasj = g.py || j > 0, hask = q.k > 0;
    const int64_t dj = j > 0 ? -g.nz : (ny - 1) * g.nz;       // -1 row, periodic wrap
    const bool tf = g.src == 2;
    const bool spec = q.k0 == 0 || (g.P > 0 && (q.k0 < g.P || q.k0 + 63 >= g.nz - g.P)) ||
                      (tf && (holds(q.k0, g.b0) || holds(q.k0, g.b1))) || (g.src == 1 && holds(q.k0, g.src_k)) ||
                      (!g.py && (j == 0 || (g.P > 0 && (j < g.P || j >= ny - g.P))));
    const Planes xspec{g.px ? 0 : g.P > 1 ? g.P : 1, g.px ? g.nx : g.nx - g.P, tf && !g.px ? g.b0 : -1,
                       tf && !g.px ? g.b1 : -1};
    const T zero = (T)0, ce = (T)g.ced;
    const uint32_t lane = threadIdx.x & 63, l = lane * (uint32_t)sizeof(T), lk = hask ? l - (uint32_t)sizeof(T) : l;
    // (the node below the wave's first is in reach: k0 > 0 there)
    auto at = [](const T *f, int64_t p, uint32_t o) { return elem(f, p, o); };
    int64_t p = (q.i0 * ny + j) * g.nz + q.k0;
    const int64_t pk = q.k0 > 0 ? 1 : 0;
    const uint32_t lk1 = q.k0 > 0 ? l : lk;
    // plane i0-1: periodic wrap to plane nx-1, or zero beyond the wall
    T hy_i = zero, hz_i = zero;
    if (q.i0 > 0 || g.px) {
        const int64_t pm = q.i0 > 0 ? p - sI : p + (g.nx - 1) * sI;
        hy_i = at(arg.f.H[1], pm, l);
        hz_i = at(arg.f.H[2], pm, l);
    }
    struct In {
        T h[3], hxj, hzj, hxk, hyk, e[3];
        int lo, hi;               // the support span of the row
        int64_t off;
    };
    Const<int2> *const spans = (Const<int2> *)(uint64_t)arg.pl.span;
    Const<int64_t> *const offs = (Const<int64_t> *)(uint64_t)arg.pl.off;
    auto load = [&](int64_t p, int64_t row, In &v) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            v.h[c] = at(arg.f.H[c], p, l);
            v.e[c] = at(arg.f.E[c], p, l);
        }
        v.hxj = at(arg.f.H[0], p + dj, l);
        v.hzj = at(arg.f.H[2], p + dj, l);
        v.hxk = at(arg.f.H[0], p - pk, lk1);
        v.hyk = at(arg.f.H[1], p - pk, lk1);
        v.lo = spans[row].x;
        v.hi = spans[row].y;
        v.off = offs[row];
    };
    int64_t row = q.i0 * ny + j;
    for (int64_t i = q.i0; i < q.i1; ++i, p += sI, row += ny) {
        In v;
        load(p, row, v);
        const bool plasma = v.lo < q.k0 + 64 && v.hi > q.k0;
        const T hx_j = hasj ? v.hxj : zero, hz_j = hasj ? v.hzj : zero;
        const T hx_k = hask ? v.hxk : zero, hy_k = hask ? v.hyk : zero;
        if (spec || xspec(i)) {
            Const<ArgsE3<T>> *s = kernel_args<ArgsE3<T>>();
            const Geo3 gs = geo_arg(&s->g);
            const Cpml3<T> c = cpml_arg<T>(&s->c);
            const Plasma3<T> pl = plasma_arg<T>(&s->pl);
            const PNode<T> pn = pnode_load<false>(pl, make_int2(v.lo, v.hi), v.off, q.k0, lane);
            e_cell<T>(gs, pl, pn, c, global_ptr(s->Hinc), s->sval, i, j, q.k, v.h[0], v.h[1], v.h[2], hx_j, hx_k, hy_i,
                      hy_k, hz_i, hz_j, v.e[0], v.e[1], v.e[2]);
        } else {
            const T dHz_y = v.h[2] - hz_j, dHy_z = v.h[1] - hy_k, dHx_z = v.h[0] - hx_k;
            const T dHz_x = v.h[2] - hz_i, dHy_x = v.h[1] - hy_i, dHx_y = v.h[0] - hx_j;
            const T curl[3] = {dHz_y - dHy_z, dHx_z - dHz_x, dHy_x - dHx_y};
            if (plasma) {
                const Plasma3<T> pl = plasma_arg<T>(&kernel_args<ArgsE3<T>>()->pl);
                const PNode<T> pn = pnode_load<sizeof(T) == 8>(pl, make_int2(v.lo, v.hi), v.off, q.k0, lane);
                if (pn.on) {
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        const T eo = v.e[c];
                        NodeCoef<T> cf = pn.cf[c];
                        v.e[c] = e_plasma3(eo, pn.J[c], curl[c], cf);
                        if (kLateJ<T>) j_coef_at(pl, c, pn.base, pn.off, cf);
                        elem(pl.J[c], pn.base, pn.off) = (T)j_update<T>((double)pn.J[c], (double)eo, (double)v.e[c], cf);
                    }
                } else {
#pragma unroll
                    for (int c = 0; c < 3; ++c) v.e[c] = fmat(ce, curl[c], v.e[c]);
                }
            } else {
#pragma unroll
                for (int c = 0; c < 3; ++c) v.e[c] = fmat(ce, curl[c], v.e[c]);
            }
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) elem(arg.f.E[c], p, l) = v.e[c];
        hy_i = v.h[1];
        hz_i = v.h[2];
    }
}

// ---- fused step ---------------------------------------------------------------
//
// One wave owns 63 cells of a row, k0 .. k0+62 of row j, over a chunk of
// planes [i0, i1), and marches along x; its 64 lanes hold the cells
// k0-1 .. k0+62.  Per plane every lane computes H^{n+1/2} of its cell and,
// for the E update of its own cell, the Hx and Hz of the cell at j-1 (both
// from E^n and H^{n-1/2} read from the input copy, exactly as the owners of
// those cells compute them); the H at k-1 is the lane below's (a cross-lane
// move), which is why lane 0 holds the cell k0-1 and updates no E.  Then
// E^{n+1} and J^{n+1} of cells k0 .. k0+62 from that H and the H of the
// previous plane, kept in registers; the chunk starts one plane early (i0-1)
// for the H its first E plane needs.  E, H and the CPML auxiliaries are read
// from one copy and written to the other, so no wave reads a value another
// has already advanced and no wave waits on another (no barrier, no LDS).
// The loads of plane i+1 are issued before the arithmetic of plane i.  HBM
// traffic per cell: E and H read once and written once; the rim reads (rows
// j +- 1, the lane-0 column, the lead-in plane) are re-reads that hit L2.

__device__ __forceinline__ float lane_up1(float x)
{
    // lane l receives lane l-1's value, lane 0 receives 0 (DPP wave_shr:1,
    // zero written by the move itself)
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x138, 0xF, 0xF, true));
}
__device__ __forceinline__ double lane_up1(double x)
{
    const int2 v = __builtin_bit_cast(int2, x);
    return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_mov_dpp(v.x, 0x138, 0xF, 0xF, true),
                                                __builtin_amdgcn_mov_dpp(v.y, 0x138, 0xF, 0xF, true)));
}

// What one plane of a fused-kernel lane reads from the input copy.
template <typename T>
struct Plane3 {
    T e[3];        // E^n(i, j, k)
    T eyi, ezi;    // Ey, Ez at (i+1, j, k)
    T exj, ezj;    // Ex, Ez at (i, j+1, k)
    T exk, eyk;    // Ex, Ey at (i, j, k+1)
    T m[3];        // E^n(i, j-1, k)
    T myk, myi;    // Ey at (i, j-1, k+1) and (i+1, j-1, k)
    T h[3];        // H^{n-1/2}(i, j, k)
    T hmx, hmz;    // Hx, Hz at (i, j-1, k)
};

template <typename T>
__device__ __forceinline__ T ld_if(const T *a, int64_t p, bool ok)
{
    return ok ? a[p] : (T)0;
}

template <typename T>
__global__ __launch_bounds__(256) void k_fused3d(Geo3 g, Fields3<T> fin, Fields3<T> fout, Plasma3<T> pl,
                                                 Cpml3<T> c, const double *Einc, const double *Hinc,
                                                 double sval, int ni)
{
    const int lane = threadIdx.x & 63;
    const int64_t kbf = (g.nz + 62) / 63;
    const int64_t bid = xcd_chunk(blockIdx.x, gridDim.x);
    const int64_t kq = bid % kbf, r = bid / kbf;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t j = (r % g.jb) * 4 + w;
    if (j >= g.ny) return;                           // the whole wave; no wave waits on another
    const int64_t i0 = (r / g.jb) * ni;
    const int64_t i1 = i0 + ni < g.nx ? i0 + ni : g.nx;
    const int64_t k = kq * 63 - 1 + lane;
    const bool vk = k >= 0 && k < g.nz;             // the lane's cell exists
    const bool own = vk && lane > 0;                 // and is this wave's
    const bool hasj = g.py || j + 1 < g.ny;          // row j+1 exists (wrapped if periodic)
    const bool hasjm = g.py || j > 0;                // row j-1 exists
    const int64_t jp = j + 1 < g.ny ? j + 1 : 0, jm = j > 0 ? j - 1 : g.ny - 1;
    const bool hask = k + 1 < g.nz;
    const T zero = (T)0;

    auto load = [&](int64_t gi, Plane3<T> &q) {
        const bool hasi = g.px || gi + 1 < g.nx;     // plane i+1 exists (wrapped if periodic)
        const int64_t gi1 = gi + 1 < g.nx ? gi + 1 : 0;
        const int64_t p = (gi * g.ny + j) * g.nz + k, p1 = (gi1 * g.ny + j) * g.nz + k;
        const int64_t pj = (gi * g.ny + jp) * g.nz + k, pm = (gi * g.ny + jm) * g.nz + k;
        const int64_t pm1 = (gi1 * g.ny + jm) * g.nz + k;
        const bool hm = vk && hasjm;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            q.e[a] = ld_if(fin.E[a], p, vk);
            q.m[a] = ld_if(fin.E[a], pm, hm);
            q.h[a] = ld_if(fin.H[a], p, vk);
        }
        q.eyi = ld_if(fin.E[1], p1, vk && hasi);
        q.ezi = ld_if(fin.E[2], p1, vk && hasi);
        q.exj = ld_if(fin.E[0], pj, vk && hasj);
        q.ezj = ld_if(fin.E[2], pj, vk && hasj);
        q.exk = ld_if(fin.E[0], p + 1, vk && hask);
        q.eyk = ld_if(fin.E[1], p + 1, vk && hask);
        q.myk = ld_if(fin.E[1], pm + 1, hm && hask);
        q.myi = ld_if(fin.E[1], pm1, hm && hasi);
        q.hmx = ld_if(fin.H[0], pm, hm);
        q.hmz = ld_if(fin.H[2], pm, hm);
    };
    auto wrap = [&](int64_t i) { return i < 0 ? i + g.nx : i; };

    // the lead-in plane i0-1: wrapped to nx-1 on a periodic x, absent at a wall
    int64_t i = (i0 > 0 || g.px) ? i0 - 1 : i0;
    T hy_i = zero, hz_i = zero;                      // H^{n+1/2} of the previous plane
    Plane3<T> cur, nxt;
    load(wrap(i), cur);
    Const<int2> *const spans = (Const<int2> *)(uint64_t)pl.span;
    Const<int64_t> *const offs = (Const<int64_t> *)(uint64_t)pl.off;
    int2 sp;                                         // support span of the next E plane's row
    sp.x = spans[i0 * g.ny + j].x;
    sp.y = spans[i0 * g.ny + j].y;
    int64_t of = offs[i0 * g.ny + j];
    for (; i < i1; ++i) {
        const int64_t gi = wrap(i);
        const bool lead = i < i0;
        // this plane's plasma terms first, then the next plane's fields: the
        // E update waits on neither the next plane's loads nor a chain of its own
        PNode<T> pn;
        pn.on = false;
        int2 spn = sp;
        int64_t ofn = of;
        if (!lead) {
            pn = pnode_load<false>(pl, sp, of, kq * 63 - 1, (uint32_t)lane);
            if (i + 1 < i1) {
                spn.x = spans[(i + 1) * g.ny + j].x;
                spn.y = spans[(i + 1) * g.ny + j].y;
                ofn = offs[(i + 1) * g.ny + j];
            }
        }
        if (i + 1 < i1) load(i + 1, nxt);
        T hx = cur.h[0], hy = cur.h[1], hz = cur.h[2];
        if (vk)
            h_cell<T>(g, c, Einc, gi, j, k, cur.e[0], cur.e[1], cur.e[2], cur.exj, cur.exk, cur.eyi, cur.eyk, cur.ezi,
                      cur.ezj, hx, hy, hz, own && !lead);
        const T hxk = lane_up1(hx), hyk = lane_up1(hy);   // H at k-1
        if (own && !lead) {
            T mx = cur.hmx, my = zero, mz = cur.hmz;
            if (hasjm)
                h_cell<T>(g, c, Einc, gi, jm, k, cur.m[0], cur.m[1], cur.m[2], cur.e[0], zero, cur.myi, cur.myk, zero,
                          cur.e[2], mx, my, mz, false);
            T e0 = cur.e[0], e1 = cur.e[1], e2 = cur.e[2];
            const bool kin = k > 0;
            e_cell<T>(g, pl, pn, c, Hinc, sval, gi, j, k, hx, hy, hz, hasjm ? mx : zero, kin ? hxk : zero, hy_i,
                      kin ? hyk : zero, hz_i, hasjm ? mz : zero, e0, e1, e2);
            const int64_t p = (gi * g.ny + j) * g.nz + k;
            fout.H[0][p] = hx;
            fout.H[1][p] = hy;
            fout.H[2][p] = hz;
            fout.E[0][p] = e0;
            fout.E[1][p] = e1;
            fout.E[2][p] = e2;
        }
        hy_i = hy;
        hz_i = hz;
        cur = nxt;
        sp = spn;
        of = ofn;
    }
}

// kAuxBatch steps of the incident 1D vacuum grid, one workgroup: H from E, then
// E with the source and first-order Mur ends (which read the old end values).
// One launch a batch: the grid does not depend on the 3D fields, and a launch a
// step stood between the H and the E pass of every step, 5 us each.
__global__ __launch_bounds__(1024) void k_aux3d(double *E, double *H, int64_t na, int64_t src, double chd, double ced,
                                                double cm, AuxSource s)
{
    for (int64_t q = threadIdx.x; q < na; q += blockDim.x) {
        E[q] = E[kAuxBatch * na + q];
        H[q] = H[kAuxBatch * na + q];
    }
    __syncthreads();
    for (int t = 0; t < kAuxBatch; ++t) {
        const double *Ei = E + t * na, *Hp = H + t * na;
        double *Eo = E + (t + 1) * na, *Hi = H + (t + 1) * na;
        for (int64_t q = threadIdx.x; q < na - 1; q += blockDim.x) Hi[q] = Hp[q] - chd * (Ei[q + 1] - Ei[q]);
        __syncthreads();
        for (int64_t q = threadIdx.x + 1; q < na - 1; q += blockDim.x) Eo[q] = Ei[q] - ced * (Hi[q] - Hi[q - 1]);
        __syncthreads();
        if (threadIdx.x == 0) {
            Eo[src] = Eo[src] + s.s[t];
            Eo[0] = Ei[1] + cm * (Eo[1] - Ei[0]);
            Eo[na - 1] = Ei[na - 2] + cm * (Eo[na - 2] - Ei[na - 1]);
            Hi[na - 1] = 0.0;
        }
        __syncthreads();
    }
}

// Sample point code: component * N + node (component 0..2 E, 3..5 H).
template <typename T>
__global__ __launch_bounds__(256) void k_sample3d(Fields3<T> f, int64_t N, const int64_t *pts,
                                                  const int32_t *list, int64_t cnt, T *buf)
{
    sample(f, N, pts, list, cnt, buf, (int64_t)blockIdx.x * blockDim.x + threadIdx.x);
}

// Twiddles dt e^{-j 2 pi f t} of slots 0..cnt-1 (samples m0+1 .. m0+cnt):
// [0][s][f] for E (t = m dt), [1][s][f] for H (t = (m - 1/2) dt = (2m-1) dt/2).
__global__ void k_tw3d(const double *freqs, int F, double dt, int64_t m0, int cnt, double2 *tw)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= 2LL * cnt * F) return;
    const int kind = (int)(t / ((int64_t)cnt * F));
    const int64_t r = t - (int64_t)kind * cnt * F;
    const int s = (int)(r / F), fi = (int)(r % F);
    const int64_t m = m0 + s + 1;
    double re, im;
    if (kind == 0) twiddle(freqs[fi] * dt, dt, m, re, im);
    else twiddle(freqs[fi] * (0.5 * dt), dt, 2 * m - 1, re, im);
    tw[t] = make_double2(re, im);
}

// X[f][q] += sum_s v_s tw_s,f, slots in order; one thread per point.  The
// twiddle indices are wave-uniform, so both the E and the H twiddle are read
// as scalars and each lane picks its own.
template <typename T>
__global__ __launch_bounds__(256) void k_flush3d(const T *__restrict__ buf, int cnt, int64_t npts,
                                                 const int64_t *__restrict__ pts, int64_t N, int F,
                                                 const double2 *__restrict__ tw, double2 *__restrict__ X)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= npts) return;
    const bool isH = pts[q] >= 3 * N;
    const double2 *tH = tw + (int64_t)cnt * F;
    double v[kSlotsMax];
#pragma unroll
    for (int s = 0; s < kSlotsMax; ++s) v[s] = s < cnt ? (double)buf[(int64_t)s * npts + q] : 0.0;
    for (int fi = 0; fi < F; ++fi) {
        double2 x = X[(int64_t)fi * npts + q];
#pragma unroll
        for (int s = 0; s < kSlotsMax; ++s) {
            if (s < cnt) {
                const double2 we = tw[(int64_t)s * F + fi], wh = tH[(int64_t)s * F + fi];
                const double wr = isH ? wh.x : we.x, wi = isH ? wh.y : we.y;
                x.x = __builtin_fma(v[s], wr, x.x);
                x.y = __builtin_fma(v[s], wi, x.y);
            }
        }
        X[(int64_t)fi * npts + q] = x;
    }
}

// X plus the window's cnt buffered samples (the order of k_flush3d), laid out
// for the host: re, im [point][f].
template <typename T>
__global__ __launch_bounds__(256) void k_spectra3d(const T *__restrict__ buf, int cnt, int64_t npts,
                                                   const int64_t *__restrict__ pts, int64_t N, int F,
                                                   const double2 *__restrict__ tw, const double2 *__restrict__ X,
                                                   double *__restrict__ re, double *__restrict__ im, int *bad)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= npts) return;
    const double2 *tk = pts[q] >= 3 * N ? tw + (int64_t)cnt * F : tw;
    bool fine = true;
    for (int fi = 0; fi < F; ++fi) {
        double2 x = X[(int64_t)fi * npts + q];
        for (int s = 0; s < cnt; ++s) {
            const double v = (double)buf[(int64_t)s * npts + q];
            const double2 t = tk[(int64_t)s * F + fi];
            x.x = __builtin_fma(v, t.x, x.x);
            x.y = __builtin_fma(v, t.y, x.y);
        }
        re[q * F + fi] = x.x;
        im[q * F + fi] = x.y;
        fine = fine && __builtin_isfinite(x.x) && __builtin_isfinite(x.y);
    }
    if (!fine) *bad = 1;
}

__global__ void k_fill3d(uint4 *p, int64_t n16)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t j = i; j < n16; j += stride) p[j] = make_uint4(0, 0, 0, 0);
}

// ---- launchers ----------------------------------------------------------------

// workgroups of a split pass: its cells', then its sample points'
template <typename T>
static dim3 grid3(const Geo3 &g, Samples3<T> &s)
{
    s.cells = g.kb * g.jb * ((g.ib - g.ia + g.np - 1) / g.np);
    return dim3((unsigned)(s.cells + (s.cnt + 255) / 256));
}

template <typename T>
void launch_coef3d(const double *const w[3], const double *const n[3], int64_t S, double dt, double d,
                   T *const eA[3], T *const eJ[3], T *const eH[3], T *const a[3], T *const b1[3],
                   T *const b2[3], hipStream_t st)
{
    if (S <= 0) return;
    hipLaunchKernelGGL(k_coef3d<T>, dim3((unsigned)((S + 255) / 256)), dim3(256), 0, st, w[0], w[1], w[2], n[0],
                       n[1], n[2], S, dt, d, eA[0], eA[1], eA[2], eJ[0], eJ[1], eJ[2], eH[0], eH[1], eH[2], a[0],
                       a[1], a[2], b1[0], b1[1], b1[2], b2[0], b2[1], b2[2]);
}

template <typename T>
void launch_h3d(const Geo3 &g, Samples3<T> s, const Fields3<T> &f, const Cpml3<T> &c, const double *Einc, hipStream_t st)
{
    const dim3 grid = grid3(g, s);
    hipLaunchKernelGGL(k_h3d<T>, grid, dim3(256), 0, st, ArgsH3<T>{g, s, f, c, Einc});
}

template <typename T>
void launch_e3d(const Geo3 &g, Samples3<T> s, const Fields3<T> &f, const Plasma3<T> &pl, const Cpml3<T> &c,
                const double *Hinc, double sval, hipStream_t st)
{
    const dim3 grid = grid3(g, s);
    hipLaunchKernelGGL(k_e3d<T>, grid, dim3(256), 0, st, ArgsE3<T>{g, s, f, pl, c, Hinc, sval});
}

void launch_aux3d(double *E, double *H, int64_t na, int64_t src, double chd, double ced, double cm,
                  const AuxSource &s, hipStream_t st)
{
    hipLaunchKernelGGL(k_aux3d, dim3(1), dim3(na > 512 ? 1024 : 512), 0, st, E, H, na, src, chd, ced, cm, s);
}

template <typename T>
void launch_spectra3d(const T *buf, int cnt, int64_t npts, const int64_t *pts, int64_t N, int F,
                      const double2 *tw, const double2 *X, double *re, double *im, int *bad, hipStream_t st)
{
    if (npts <= 0 || F <= 0) return;
    hipLaunchKernelGGL(k_spectra3d<T>, dim3((unsigned)((npts + 255) / 256)), dim3(256), 0, st, buf, cnt, npts, pts, N, F,
                       tw, X, re, im, bad);
}

template <typename T>
void launch_fused3d(const Geo3 &g, const Fields3<T> &fin, const Fields3<T> &fout, const Plasma3<T> &pl,
                    const Cpml3<T> &c, const double *Einc, const double *Hinc, double sval, int ni,
                    hipStream_t st)
{
    // 63 cells along k per wave (see k_fused3d)
    const int64_t nb = ((g.nz + 62) / 63) * g.jb * ((g.nx + ni - 1) / ni);
    hipLaunchKernelGGL(k_fused3d<T>, dim3((unsigned)nb), dim3(256), 0, st, g, fin, fout, pl, c, Einc, Hinc,
                       sval, ni);
}

template <typename T>
void launch_sample3d(const Fields3<T> &f, int64_t N, const int64_t *pts, const int32_t *list, int64_t cnt, T *buf,
                     hipStream_t st)
{
    if (cnt <= 0) return;
    hipLaunchKernelGGL(k_sample3d<T>, dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0, st, f, N, pts, list, cnt, buf);
}

void launch_tw3d(const double *freqs, int F, double dt, int64_t m0, int cnt, double2 *tw, hipStream_t st)
{
    const int64_t n = 2LL * cnt * F;
    if (n <= 0) return;
    hipLaunchKernelGGL(k_tw3d, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, freqs, F, dt, m0, cnt, tw);
}

template <typename T>
void launch_flush3d(const T *buf, int cnt, int64_t npts, const int64_t *pts, int64_t N, int F,
                    const double2 *tw, double2 *X, hipStream_t st)
{
    if (npts <= 0 || F <= 0 || cnt <= 0) return;
    hipLaunchKernelGGL(k_flush3d<T>, dim3((unsigned)((npts + 255) / 256)), dim3(256), 0, st, buf, cnt, npts,
                       pts, N, F, tw, X);
}

void launch_fill3d(void *p, int64_t bytes, hipStream_t st)
{
    const int64_t n16 = bytes / 16;
    if (n16 <= 0) return;
    int64_t nb = (n16 + 255) / 256;
    if (nb > 65536) nb = 65536;
    hipLaunchKernelGGL(k_fill3d, dim3((unsigned)nb), dim3(256), 0, st, (uint4 *)p, n16);
}

#define INST3(T)                                                                                          \
    template void launch_spectra3d<T>(const T *, int, int64_t, const int64_t *, int64_t, int,           \
                                      const double2 *, const double2 *, double *, double *, int *,      \
                                      hipStream_t);                                                      \
    template void launch_h3d<T>(const Geo3 &, Samples3<T>, const Fields3<T> &, const Cpml3<T> &,         \
                                const double *, hipStream_t);                                             \
    template void launch_fused3d<T>(const Geo3 &, const Fields3<T> &, const Fields3<T> &,                \
                                    const Plasma3<T> &, const Cpml3<T> &, const double *, const double *, \
                                    double, int, hipStream_t);                                            \
    template void launch_e3d<T>(const Geo3 &, Samples3<T>, const Fields3<T> &, const Plasma3<T> &,       \
                                const Cpml3<T> &, const double *, double, hipStream_t);                   \
    template void launch_sample3d<T>(const Fields3<T> &, int64_t, const int64_t *, const int32_t *,   \
                                     int64_t, T *, hipStream_t);                                                        \
    template void launch_flush3d<T>(const T *, int, int64_t, const int64_t *, int64_t, int,             \
                                    const double2 *, double2 *, hipStream_t);                             \
    template void launch_coef3d<T>(const double *const[3], const double *const[3], int64_t, double,     \
                                   double, T *const[3], T *const[3], T *const[3], T *const[3],           \
                                   T *const[3], T *const[3], hipStream_t);
INST3(float)
INST3(double)
#undef INST3

}  // namespace fdtdp
