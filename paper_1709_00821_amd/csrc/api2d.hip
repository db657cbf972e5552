// Host side of the 2D library: descriptor validation, workspace layout, the
// compact plasma support, time loop (eager or replayed from a captured HIP
// graph), probe DFT windows, field read-back.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <map>
#include <new>
#include <string>
#include <vector>

#include "../../include/fdtd_plasma2d.h"
#include "internal.h"
#include "internal2d.h"

using namespace fdtdp;

namespace {

thread_local std::string g_err2;

int fail2(int code, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err2 = buf;
    return code;
}

#define HIP_TRY2(expr)                                                                   \
    do {                                                                                 \
        hipError_t e_ = (expr);                                                          \
        if (e_ != hipSuccess)                                                            \
            return fail2(FDTD_E_DEVICE, "%s failed: %s", #expr, hipGetErrorString(e_));  \
    } while (0)

constexpr int64_t kAlign2 = 256;
constexpr int kSB2 = 2048;     // probe samples per DFT window

int64_t rup(int64_t x, int64_t a) { return (x + a - 1) / a * a; }

struct Lay {
    int64_t total = 0;
    int64_t take(int64_t b)
    {
        const int64_t o = total;
        total += rup(std::max<int64_t>(b, 16), kAlign2);
        return o;
    }
};

struct Plan2 {
    Lay L;
    int ncomp = 1, nh = 2, es = 8;
    int64_t N = 0, S = 0;
    std::vector<int2> span;
    std::vector<int64_t> rowoff;
    std::vector<Tile2> tiles;        // the plasma tiles, then the vacuum tiles
    int64_t nplasma = 0;
    Tiles2 vac = Tiles2::flat;       // shape of the vacuum tiles
    std::vector<LaneProbes> tprobe;  // probes by tile, wave and lane
    std::vector<int32_t> row;        // sample row of each probe (probes of the same cell and component share one)
    std::vector<int64_t> cell;       // component N + cell of each sample row
    int64_t rows = 0;
    bool one = false;                // one copy of the fields: every step in place
    bool thin = false;               // two copies would not be used
    int64_t o_E[2][2] = {}, o_H[2][2] = {}, o_J[2][2] = {};   // [copy][component]
    int64_t o_span = 0, o_rowoff = 0, o_wp2[2] = {0, 0}, o_nu[2] = {0, 0}, o_tiles = 0,
            o_tprobe = 0, o_cell = 0, o_srcv = 0, o_freqs = 0, o_samp = 0, o_X = 0, o_Xtmp = 0, o_tw = 0;
};

int validate2(const fdtd2d_desc *d)
{
    if (!d) return fail2(FDTD_E_INVALID, "descriptor is NULL");
    if (d->struct_size != sizeof(fdtd2d_desc))
        return fail2(FDTD_E_INVALID, "struct_size %u != %zu (header/library mismatch)", d->struct_size,
                     sizeof(fdtd2d_desc));
    if (d->mode != FDTD2D_TM && d->mode != FDTD2D_TE) return fail2(FDTD_E_INVALID, "mode %d", d->mode);
    if (d->precision != FDTD_F64 && d->precision != FDTD_F32)
        return fail2(FDTD_E_INVALID, "precision %d (FDTD_F64 or FDTD_F32)", d->precision);
    if (d->nx < 2 || d->ny < 2 || d->nx > (1 << 20) || d->ny > (1 << 20) || d->nx * d->ny > ((int64_t)1 << 32))
        return fail2(FDTD_E_INVALID, "grid %lld x %lld out of range", (long long)d->nx, (long long)d->ny);
    if (!(d->d > 0.0) || !(d->dt > 0.0) || !std::isfinite(d->d) || !std::isfinite(d->dt))
        return fail2(FDTD_E_INVALID, "d and dt must be positive and finite");
    if (kC0 * d->dt / d->d > 1.0 / std::sqrt(2.0))
        return fail2(FDTD_E_UNSTABLE, "Courant number c dt/d = %.6g exceeds 1/sqrt(2)", kC0 * d->dt / d->d);
    if (!d->wp2 || !d->nu || (d->n_probes > 0 && !d->probes) || !d->freqs_hz)
        return fail2(FDTD_E_INVALID, "a host array pointer is NULL");
    if (d->n_probes < 0 || d->n_probes > 4096 || d->n_freqs < 1)
        return fail2(FDTD_E_INVALID, "need 0 <= n_probes <= 4096 and n_freqs >= 1");
    const int nc = d->mode == FDTD2D_TM ? 1 : 2;
    const int64_t N = d->nx * d->ny;
    for (int64_t k = 0; k < nc * N; ++k)
        if (!(d->wp2[k] >= 0.0) || !std::isfinite(d->wp2[k]) || !(d->nu[k] >= 0.0) || !std::isfinite(d->nu[k]))
            return fail2(FDTD_E_INVALID, "wp2 and nu must be finite and >= 0 (entry %lld)", (long long)k);
    if (d->has_src && (d->src_i < 0 || d->src_i >= d->nx || d->src_j < 0 || d->src_j >= d->ny))
        return fail2(FDTD_E_INVALID, "source (%lld, %lld) outside the grid", (long long)d->src_i,
                     (long long)d->src_j);
    if (d->has_src && !(std::isfinite(d->src_tau) && d->src_tau > 0 && std::isfinite(d->src_t0) &&
                        std::isfinite(d->src_amp)))
        return fail2(FDTD_E_INVALID, "source parameters must be finite with tau > 0");
    for (int p = 0; p < d->n_probes; ++p) {
        const int64_t *q = d->probes + 3 * p;
        if (q[0] < 0 || q[0] >= nc || q[1] < 0 || q[1] >= d->nx || q[2] < 0 || q[2] >= d->ny)
            return fail2(FDTD_E_INVALID, "probe %d (%lld, %lld, %lld) outside the grid or the mode", p,
                         (long long)q[0], (long long)q[1], (long long)q[2]);
    }
    for (int f = 0; f < d->n_freqs; ++f)
        if (!std::isfinite(d->freqs_hz[f])) return fail2(FDTD_E_INVALID, "freqs_hz[%d] not finite", f);
    return FDTD_OK;
}

// One tile with outputs [oi0, oi1) x [oj0, oj1) and a halo of kSteps2 cells.
void push_tile2(const fdtd2d_desc *d, Plan2 &p, const Shape2 &sh, int64_t oi0, int64_t oi1, int64_t oj0, int64_t oj1)
{
    Tile2 t{};
    t.i0 = (int32_t)(oi0 - kSteps2);
    t.j0 = (int32_t)(oj0 - kSteps2);
    t.oi0 = (int32_t)oi0;
    t.oi1 = (int32_t)oi1;
    t.oj0 = (int32_t)oj0;
    t.oj1 = (int32_t)oj1;
    // index-0 lines count as special only where they are walls, but a tile
    // holding one holds a cell outside the grid too
    t.special = t.i0 < 0 || t.j0 < 0 || t.i0 + sh.rows() > d->nx || t.j0 + sh.cols() > d->ny ||
                (d->has_src && d->src_i >= t.i0 && d->src_i < t.i0 + sh.rows() && d->src_j >= t.j0 &&
                 d->src_j < t.j0 + sh.cols());
    p.tiles.push_back(t);
}

// Tiles of the grid: vacuum tiles of the plan's shape wherever the whole held
// span is off the plasma support, and plasma tiles over the outputs of the
// others (side by side along a band of rows, so few are partly filled).
void build_tiles2(const fdtd2d_desc *d, Plan2 &p)
{
    auto count = [&](const Shape2 &s) {
        const int64_t i = s.rows() - 2 * kSteps2, j = s.cols() - 2 * kSteps2;
        return ((d->nx + i - 1) / i) * ((d->ny + j - 1) / j);
    };
    p.vac = count(kFlat2) <= kFlatMaxTiles2 ? Tiles2::flat : Tiles2::tall;
    p.thin = d->nx < kThinRows2 && count(kFlat2) > kThinTiles2;
    const Shape2 v = p.vac == Tiles2::flat ? kFlat2 : kTall2, q = kPlasma2;
    const int64_t vi = v.rows() - 2 * kSteps2, vj = v.cols() - 2 * kSteps2;
    const int64_t qi = q.rows() - 2 * kSteps2, qj = q.cols() - 2 * kSteps2;
    auto wrap = [](int64_t k, int64_t n) { return (k % n + n) % n; };
    // does row i carry plasma in columns [j0, j1) (either may lie outside)?
    auto row_plasma = [&](int64_t i, int64_t j0, int64_t j1) {
        if (i < 0 || i >= d->nx) {
            if (!d->periodic_x) return false;
            i = wrap(i, d->nx);
        }
        const int2 sp = p.span[i];
        if (sp.x >= sp.y) return false;
        if (j0 < sp.y && j1 > sp.x) return true;
        if (!d->periodic_y) return false;
        for (int64_t j = j0; j < j1; ++j)
            if (j < 0 || j >= d->ny) {
                const int64_t w = wrap(j, d->ny);
                if (w >= sp.x && w < sp.y) return true;
            }
        return false;
    };
    std::vector<Tile2> vac;
    p.tiles.clear();
    for (int64_t oi = 0; oi < d->nx; oi += vi) {
        const int64_t oi1 = std::min(oi + vi, d->nx);
        int64_t run = -1;                  // first output column of the plasma run being gathered
        auto close = [&](int64_t end) {
            for (int64_t a = oi; run >= 0 && a < oi1; a += qi)
                for (int64_t b = run; b < end; b += qj)
                    push_tile2(d, p, q, a, std::min(a + qi, oi1), b, std::min(b + qj, end));
            run = -1;
        };
        for (int64_t oj = 0; oj < d->ny; oj += vj) {
            const int64_t oj1 = std::min(oj + vj, d->ny);
            bool plasma = false;
            for (int64_t i = oi - kSteps2; !plasma && i < oi - kSteps2 + v.rows(); ++i)
                plasma = row_plasma(i, oj - kSteps2, oj - kSteps2 + v.cols());
            if (plasma) {
                if (run < 0) run = oj;
                continue;
            }
            close(oj);
            push_tile2(d, p, v, oi, oi1, oj, oj1);
            vac.push_back(p.tiles.back());
            p.tiles.pop_back();
        }
        close(d->ny);
    }
    p.nplasma = (int64_t)p.tiles.size();
    p.tiles.insert(p.tiles.end(), vac.begin(), vac.end());
    // each probe with the tile that writes it, by wave, lane and register
    std::vector<std::pair<int64_t, int>> by_row;
    for (int k = 0; k < d->n_probes; ++k) by_row.push_back({d->probes[3 * k + 1], k});
    std::sort(by_row.begin(), by_row.end());
    p.tprobe.clear();
    p.row.assign(d->n_probes, 0);
    p.cell.clear();
    for (size_t n = 0; n < p.tiles.size(); ++n) {
        Tile2 &t = p.tiles[n];
        const Shape2 &sh = (int64_t)n < p.nplasma ? q : v;
        std::vector<std::pair<int64_t, int>> in;      // (wave, lane, bit) as one number, probe
        auto at = std::lower_bound(by_row.begin(), by_row.end(), std::make_pair((int64_t)t.oi0, -1));
        for (; at != by_row.end() && at->first < t.oi1; ++at) {
            const int64_t *pr = d->probes + 3 * at->second;
            if (pr[2] < t.oj0 || pr[2] >= t.oj1) continue;
            const int64_t i = pr[1] - t.i0, j = pr[2] - t.j0;
            const int64_t bit = (pr[0] * sh.R + i % sh.R) * sh.CJ + j % sh.CJ;
            in.push_back({(i / sh.R * 64 + j / sh.CJ) * 32 + bit, at->second});
        }
        std::sort(in.begin(), in.end());
        t.probe0 = (int32_t)(p.tprobe.size() / 64);
        t.pwaves = 0;
        for (size_t k = 0; k < in.size(); ++k) {
            const int64_t bit = in[k].first % 32, lane = in[k].first / 32 % 64, w = in[k].first / 2048;
            if (!((t.pwaves >> w) & 1)) {
                t.pwaves |= 1 << w;
                p.tprobe.resize(p.tprobe.size() + 64, LaneProbes{0, 0});
            }
            LaneProbes &lp = p.tprobe[p.tprobe.size() - 64 + lane];
            const int64_t *pr = d->probes + 3 * in[k].second;
            if (!lp.mask) lp.first = (int32_t)p.cell.size();
            if (!((lp.mask >> bit) & 1)) p.cell.push_back((pr[0] * d->nx + pr[1]) * d->ny + pr[2]);
            lp.mask |= 1u << bit;
            p.row[in[k].second] = (int32_t)(p.cell.size() - 1);
        }
    }
    p.rows = (int64_t)p.cell.size();
}

// The workspace, with one copy of the fields and currents or two.
void lay_out2(const fdtd2d_desc *d, Plan2 &p, bool one)
{
    Lay &L = p.L;
    L = Lay();
    p.one = one;
    for (int i = 0; i < (one ? 1 : 2); ++i) {
        for (int c = 0; c < p.ncomp; ++c) p.o_E[i][c] = L.take(p.es * p.N);
        for (int c = 0; c < p.nh; ++c) p.o_H[i][c] = L.take(p.es * p.N);
        for (int c = 0; c < p.ncomp; ++c) p.o_J[i][c] = L.take(8 * p.S);
    }
    p.o_span = L.take(8 * d->nx);
    p.o_rowoff = L.take(8 * d->nx);
    for (int c = 0; c < p.ncomp; ++c) {
        p.o_wp2[c] = L.take(8 * p.S);
        p.o_nu[c] = L.take(8 * p.S);
    }
    const int P = std::max(d->n_probes, 1);
    p.o_cell = L.take(8 * P);
    p.o_freqs = L.take(8 * d->n_freqs);
    p.o_samp = L.take(8 * (int64_t)P * kSB2);
    p.o_X = L.take(16 * (int64_t)P * d->n_freqs);
    p.o_Xtmp = L.take(16 * (int64_t)P * d->n_freqs);
    p.o_tw = L.take(16 * (int64_t)std::min(kSB2, kTwiddleChunk) * d->n_freqs);
    if (one) return;
    p.o_tiles = L.take((int64_t)sizeof(Tile2) * (int64_t)p.tiles.size());
    p.o_tprobe = L.take((int64_t)sizeof(LaneProbes) * (int64_t)p.tprobe.size());
    p.o_srcv = L.take(8 * kSB2);
}

int plan2(const fdtd2d_desc *d, Plan2 &p)
{
    int rc = validate2(d);
    if (rc) return rc;
    p.ncomp = d->mode == FDTD2D_TM ? 1 : 2;
    p.nh = d->mode == FDTD2D_TM ? 2 : 1;
    p.es = d->precision == FDTD_F64 ? 8 : 4;
    p.N = d->nx * d->ny;
    // compact plasma support: per row the span of cells where any component has wp2 > 0
    p.span.assign(d->nx, make_int2(0, 0));
    p.rowoff.assign(d->nx, 0);
    int64_t S = 0;
    for (int64_t i = 0; i < d->nx; ++i) {
        int64_t j0 = d->ny, j1 = 0;
        for (int c = 0; c < p.ncomp; ++c)
            for (int64_t j = 0; j < d->ny; ++j)
                if (d->wp2[c * p.N + i * d->ny + j] > 0.0) {
                    j0 = std::min(j0, j);
                    j1 = std::max(j1, j + 1);
                }
        if (j1 > j0) {
            p.span[i] = make_int2((int)j0, (int)j1);
            p.rowoff[i] = S;
            S += j1 - j0;
        }
    }
    p.S = S;
    build_tiles2(d, p);
    lay_out2(d, p, p.thin);
    return FDTD_OK;
}

}  // namespace

struct fdtd2d {
    fdtd2d_desc d;
    hipStream_t stream = nullptr;
    bool owns = false;
    char *ws = nullptr;
    Plan2 p;
    Grid2 g;
    void *E[2][2] = {}, *H[2][2] = {};       // [copy][component]
    double *J[2][2] = {};
    int cur = 0;                             // the copy that holds the state
    Tile2 *tiles = nullptr;
    int64_t *cells = nullptr;                // cells of the sample rows
    double *freqs = nullptr, *samp = nullptr, *srcv = nullptr;
    double2 *X = nullptr, *Xtmp = nullptr, *tw = nullptr;
    int64_t steps = 0, win_base = 0;
    bool tmp_valid = false;
    bool lost = false;                       // the streams of a pass did not wait for each other: state unknown
    hipStream_t side = nullptr;              // plasma tiles beside the vacuum tiles (default priority)
    hipEvent_t ev_fork = nullptr, ev_join = nullptr;
    std::map<int64_t, hipGraphExec_t> graphs;
};

namespace {

Grids dft_view(const fdtd2d *h)
{
    Grids g{};
    g.samp = h->samp;
    g.SB = kSB2;
    g.dt = h->d.dt;
    return g;
}

void reset2(fdtd2d *h)
{
    // the copy a run starts from; the first pass writes every cell of the other
    for (int c = 0; c < h->p.ncomp; ++c) {
        launch_fill(h->E[0][c], rup(h->p.es * h->p.N, 16), h->stream);
        if (h->p.S) launch_fill(h->J[0][c], rup(8 * h->p.S, 16), h->stream);
    }
    for (int c = 0; c < h->p.nh; ++c) launch_fill(h->H[0][c], rup(h->p.es * h->p.N, 16), h->stream);
    h->cur = 0;
    const int P = std::max(h->d.n_probes, 1);
    launch_fill(h->X, rup(16 * (int64_t)P * h->d.n_freqs, 16), h->stream);
    h->steps = 0;
    h->win_base = 0;
}

void fold(fdtd2d *h, double2 *dst)
{
    const int count = (int)(h->steps - h->win_base);
    if (h->d.n_probes > 0 && count > 0)
        launch_dft(dft_view(h), h->freqs, h->d.n_freqs, h->win_base + 1, count, h->tw,
                   std::min(kSB2, kTwiddleChunk), dst, h->p.rows, h->stream);
}

void to_tmp(fdtd2d *h)
{
    const int P = std::max(h->d.n_probes, 1);
    launch_copy(h->Xtmp, h->X, 16 * (int64_t)P * h->d.n_freqs, h->stream);
    fold(h, h->Xtmp);
}

template <typename T>
Fields2<T> copy2(const fdtd2d *h, int i)
{
    Fields2<T> f;
    for (int c = 0; c < 2; ++c) {
        f.E[c] = (T *)h->E[i][c];
        f.H[c] = (T *)h->H[i][c];
        f.J[c] = h->J[i][c];
    }
    return f;
}

// k steps taken: fold the sample window if it is full.
void took2(fdtd2d *h, int k)
{
    h->steps += k;
    if (h->steps - h->win_base < kSB2) return;
    fold(h, h->X);
    h->win_base = h->steps;
}

// The side stream starts behind the handle's (fork), which goes on behind it (join).
hipError_t fork2(fdtd2d *h)
{
    const hipError_t e = hipEventRecord(h->ev_fork, h->stream);
    return e == hipSuccess ? hipStreamWaitEvent(h->side, h->ev_fork, 0) : e;
}
hipError_t join2(fdtd2d *h)
{
    const hipError_t e = hipEventRecord(h->ev_join, h->side);
    return e == hipSuccess ? hipStreamWaitEvent(h->stream, h->ev_join, 0) : e;
}

// Whether k <= kSteps2 steps are taken as one pass of tiles (else one by one, in
// place): internal2d.h says what both cost.
bool by_pass(const fdtd2d *h, int64_t k)
{
    return !h->p.one && (k > 2 || (k == 2 && h->p.N > kTwoStepsBelow2));
}

template <typename T>
hipError_t advance2_t(fdtd2d *h, int64_t n)
{
    hipError_t e = hipSuccess;
    while (n > 0) {
        const int slot = (int)(h->steps - h->win_base);
        if (slot == 0 && h->g.has_src && !h->p.one) launch_src2d(h->g, h->steps + 1, kSB2, h->srcv, h->stream);
        const int k = (int)std::min<int64_t>(std::min<int64_t>(n, kSteps2), kSB2 - slot);
        if (!by_pass(h, k)) {
            for (int s = 0; s < k; ++s)
                launch_step2d<T>(h->g, copy2<T>(h, h->cur), h->cells, h->p.rows, h->steps + s + 1, slot + s, h->stream);
            took2(h, k);
            n -= k;
            continue;
        }
        const Fields2<T> in = copy2<T>(h, h->cur), out = copy2<T>(h, h->cur ^ 1);
        // plasma and vacuum tiles write disjoint cells: side by side
        const int64_t nvac = (int64_t)h->p.tiles.size() - h->p.nplasma;
        if (h->side && (e = fork2(h)) != hipSuccess) {
            h->lost = true;
            return e;
        }
        launch_tiles2d<T>(h->g, in, out, h->tiles, h->p.nplasma, Tiles2::plasma, k, slot,
                          h->side ? h->side : h->stream);
        launch_tiles2d<T>(h->g, in, out, h->tiles + h->p.nplasma, nvac, h->p.vac, k, slot, h->stream);
        if (h->side && (e = join2(h)) != hipSuccess) {
            h->lost = true;
            return e;
        }
        h->cur ^= 1;
        took2(h, k);
        n -= k;
    }
    return hipGetLastError();
}

int advance2(fdtd2d *h, int64_t n)
{
    const hipError_t e = h->p.es == 8 ? advance2_t<double>(h, n) : advance2_t<float>(h, n);
    if (e != hipSuccess) return fail2(FDTD_E_DEVICE, "time loop failed: %s", hipGetErrorString(e));
    return FDTD_OK;
}

int check2(const fdtd2d *h)
{
    if (!h) return fail2(FDTD_E_INVALID, "handle is NULL");
    if (h->lost) return fail2(FDTD_E_STATE, "handle used after a device failure");
    return FDTD_OK;
}

}  // namespace

extern "C" {

const char *fdtd2d_last_error(void) { return g_err2.c_str(); }

int fdtd2d_workspace_bytes(const fdtd2d_desc *desc, size_t *bytes)
{
    if (!bytes) return fail2(FDTD_E_INVALID, "bytes is NULL");
    Plan2 p;
    int rc = plan2(desc, p);
    if (rc) return rc;
    *bytes = (size_t)p.L.total;
    return FDTD_OK;
}

int fdtd2d_create(const fdtd2d_desc *desc, void *workspace, size_t bytes, fdtd2d **out)
{
    if (!out) return fail2(FDTD_E_INVALID, "out is NULL");
    *out = nullptr;
    fdtd2d *h = new (std::nothrow) fdtd2d();
    if (!h) return fail2(FDTD_E_INVALID, "out of host memory");
    int rc = plan2(desc, h->p);
    if (rc) {
        delete h;
        return rc;
    }
    Plan2 &p = h->p;
    // a buffer too small for two copies of the fields holds one
    if (workspace && bytes < (size_t)p.L.total) lay_out2(desc, p, true);
    if (workspace && (bytes < (size_t)p.L.total || ((uintptr_t)workspace % kAlign2))) {
        delete h;
        return fail2(FDTD_E_WORKSPACE, "workspace of %zu bytes (needs %lld, %lld-byte aligned)", bytes,
                     (long long)p.L.total, (long long)kAlign2);
    }
    h->d = *desc;
    h->stream = (hipStream_t)desc->stream;
    if (workspace) {
        h->ws = (char *)workspace;
    } else {
        hipError_t e = hipMalloc((void **)&h->ws, (size_t)p.L.total);
        if (e != hipSuccess && !p.one) {
            (void)hipGetLastError();
            lay_out2(desc, p, true);
            e = hipMalloc((void **)&h->ws, (size_t)p.L.total);
        }
        if (e != hipSuccess) {
            delete h;
            return fail2(FDTD_E_DEVICE, "hipMalloc(%lld) failed: %s", (long long)p.L.total, hipGetErrorString(e));
        }
        h->owns = true;
    }
    char *w = h->ws;
    Grid2 &g = h->g;
    g = Grid2{};
    g.nx = desc->nx;
    g.ny = desc->ny;
    g.mode = desc->mode;
    g.px = desc->periodic_x != 0;
    g.py = desc->periodic_y != 0;
    g.dt = desc->dt;
    g.d = desc->d;
    g.ch = desc->dt / (mu0() * desc->d);
    g.ce = desc->dt / (kEps0 * desc->d);
    g.span = (const int2 *)(w + p.o_span);
    g.rowoff = (const int64_t *)(w + p.o_rowoff);
    for (int c = 0; c < 2; ++c) {
        const int ce = c < p.ncomp ? c : 0, ch = c < p.nh ? c : 0;
        g.wp2[c] = (const double *)(w + p.o_wp2[ce]);
        g.nu[c] = (const double *)(w + p.o_nu[ce]);
        for (int i = 0; i < 2; ++i) {
            const int k = p.one ? 0 : i;
            h->E[i][c] = w + p.o_E[k][ce];
            h->H[i][c] = w + p.o_H[k][ch];
            h->J[i][c] = (double *)(w + p.o_J[k][ce]);
        }
    }
    h->cells = (int64_t *)(w + p.o_cell);
    h->tiles = (Tile2 *)(w + p.o_tiles);
    h->srcv = (double *)(w + p.o_srcv);
    g.srcv = h->srcv;
    g.tprobe = (const LaneProbes *)(w + p.o_tprobe);
    g.has_src = desc->has_src != 0;
    g.si = desc->src_i;
    g.sj = desc->src_j;
    g.src_tau = desc->src_tau;
    g.src_t0 = desc->src_t0;
    g.src_amp = desc->src_amp;
    g.SB = kSB2;
    h->samp = g.samp = (double *)(w + p.o_samp);
    h->freqs = (double *)(w + p.o_freqs);
    h->X = (double2 *)(w + p.o_X);
    h->Xtmp = (double2 *)(w + p.o_Xtmp);
    h->tw = (double2 *)(w + p.o_tw);
    h->d.wp2 = h->d.nu = nullptr;
    h->d.probes = nullptr;
    h->d.freqs_hz = nullptr;

    // compact plasma arrays
    std::vector<double> cw(std::max<int64_t>(p.S, 1) * p.ncomp), cn(std::max<int64_t>(p.S, 1) * p.ncomp);
    for (int c = 0; c < p.ncomp; ++c)
        for (int64_t i = 0; i < desc->nx; ++i)
            for (int64_t j = p.span[i].x; j < p.span[i].y; ++j) {
                const int64_t src = c * p.N + i * desc->ny + j, dst = c * p.S + p.rowoff[i] + (j - p.span[i].x);
                cw[dst] = desc->wp2[src];
                cn[dst] = desc->nu[src];
            }
    hipStream_t st = h->stream;
    hipError_t e = hipSuccess;
    auto H2D = [&](void *dst, const void *src, size_t n) {
        if (e == hipSuccess && n) e = hipMemcpyAsync(dst, src, n, hipMemcpyHostToDevice, st);
    };
    H2D(w + p.o_span, p.span.data(), 8 * desc->nx);
    H2D(w + p.o_rowoff, p.rowoff.data(), 8 * desc->nx);
    for (int c = 0; c < p.ncomp; ++c) {
        H2D(w + p.o_wp2[c], cw.data() + c * p.S, 8 * p.S);
        H2D(w + p.o_nu[c], cn.data() + c * p.S, 8 * p.S);
    }
    H2D(h->cells, p.cell.data(), 8 * p.cell.size());
    if (!p.one) {
        H2D(h->tiles, p.tiles.data(), sizeof(Tile2) * p.tiles.size());
        H2D(w + p.o_tprobe, p.tprobe.data(), sizeof(LaneProbes) * p.tprobe.size());
    }
    H2D(w + p.o_freqs, desc->freqs_hz, 8 * (size_t)desc->n_freqs);
    // the legacy null stream takes every launch itself
    if (e == hipSuccess && st && !p.one && p.nplasma > 0 && p.nplasma < (int64_t)p.tiles.size()) {
        e = hipStreamCreateWithFlags(&h->side, hipStreamNonBlocking);
        if (e == hipSuccess) e = hipEventCreateWithFlags(&h->ev_fork, hipEventDisableTiming);
        if (e == hipSuccess) e = hipEventCreateWithFlags(&h->ev_join, hipEventDisableTiming);
    }
    if (e == hipSuccess) {
        if (!p.one) launch_src2d(g, 1, kSB2, h->srcv, st);   // tiles read the table also without a source
        reset2(h);
        e = hipStreamSynchronize(st);
    }
    if (e == hipSuccess) e = hipGetLastError();
    if (e != hipSuccess) {
        if (h->side) (void)hipStreamDestroy(h->side);
        if (h->ev_fork) (void)hipEventDestroy(h->ev_fork);
        if (h->ev_join) (void)hipEventDestroy(h->ev_join);
        if (h->owns) (void)hipFree(h->ws);
        delete h;
        return fail2(FDTD_E_DEVICE, "create failed: %s", hipGetErrorString(e));
    }
    *out = h;
    return FDTD_OK;
}

int fdtd2d_step(fdtd2d *h, int64_t nsteps)
{
    int rc = check2(h);
    if (rc) return rc;
    if (nsteps < 0) return fail2(FDTD_E_INVALID, "nsteps %lld < 0", (long long)nsteps);
    h->tmp_valid = false;
    return advance2(h, nsteps);
}

int fdtd2d_run(fdtd2d *h, int64_t nsteps)
{
    int rc = check2(h);
    if (rc) return rc;
    if (nsteps < 0) return fail2(FDTD_E_INVALID, "nsteps %lld < 0", (long long)nsteps);
    h->tmp_valid = false;
    if (h->stream == nullptr) {   // the legacy null stream cannot be captured
        reset2(h);
        rc = advance2(h, nsteps);
        if (rc) return rc;
        to_tmp(h);
        h->tmp_valid = nsteps > 0;
        return FDTD_OK;
    }
    // until the graph is launched nothing has run: a failure leaves the state
    // the handle had
    const int cur = h->cur;
    const int64_t steps = h->steps, win_base = h->win_base;
    auto not_run = [&](int code) {
        h->cur = cur;
        h->steps = steps;
        h->win_base = win_base;
        h->lost = false;
        (void)hipGetLastError();       // reported here, not by the next call too
        return code;
    };
    hipError_t e;
    auto it = h->graphs.find(nsteps);
    if (it == h->graphs.end()) {
        e = hipStreamBeginCapture(h->stream, hipStreamCaptureModeThreadLocal);
        if (e != hipSuccess) return not_run(fail2(FDTD_E_DEVICE, "begin capture failed: %s", hipGetErrorString(e)));
        reset2(h);
        rc = advance2(h, nsteps);
        if (rc == FDTD_OK) to_tmp(h);
        hipGraph_t graph = nullptr;
        e = hipStreamEndCapture(h->stream, &graph);
        if (rc || e != hipSuccess) {
            if (graph) (void)hipGraphDestroy(graph);
            return not_run(rc ? rc : fail2(FDTD_E_DEVICE, "graph capture failed: %s", hipGetErrorString(e)));
        }
        hipGraphExec_t ex = nullptr;
        e = hipGraphInstantiate(&ex, graph, nullptr, nullptr, 0);
        (void)hipGraphDestroy(graph);
        if (e != hipSuccess)
            return not_run(fail2(FDTD_E_DEVICE, "graph instantiate failed: %s", hipGetErrorString(e)));
        it = h->graphs.emplace(nsteps, ex).first;
    } else {
        h->steps = nsteps;
        h->win_base = nsteps / kSB2 * kSB2;
        // passes of the captured run: kSteps2 steps each (windows hold whole
        // passes), then the rest
        static_assert(kSB2 % kSteps2 == 0, "windows hold whole passes");
        h->cur = (int)((by_pass(h, kSteps2) * (nsteps / kSteps2) + by_pass(h, nsteps % kSteps2)) & 1);
    }
    e = hipGraphLaunch(it->second, h->stream);
    if (e != hipSuccess) return not_run(fail2(FDTD_E_DEVICE, "graph launch failed: %s", hipGetErrorString(e)));
    h->tmp_valid = nsteps > 0;
    return FDTD_OK;
}

int fdtd2d_spectra(fdtd2d *h, double *re, double *im)
{
    int rc = check2(h);
    if (rc) return rc;
    if (!re || !im) return fail2(FDTD_E_INVALID, "output pointer is NULL");
    if (h->steps == 0 || h->d.n_probes == 0) return fail2(FDTD_E_STATE, "no step taken yet, or no probes");
    if (!h->tmp_valid) to_tmp(h);
    const int64_t n = (int64_t)h->d.n_probes * h->d.n_freqs;
    std::vector<double2> X(n);
    HIP_TRY2(hipMemcpyAsync(X.data(), h->Xtmp, 16 * n, hipMemcpyDeviceToHost, h->stream));
    HIP_TRY2(hipStreamSynchronize(h->stream));
    bool finite = true;
    for (int64_t i = 0; i < n; ++i) {
        const double2 x = X[(int64_t)h->p.row[i / h->d.n_freqs] * h->d.n_freqs + i % h->d.n_freqs];
        re[i] = x.x;
        im[i] = x.y;
        finite = finite && std::isfinite(x.x) && std::isfinite(x.y);
    }
    return finite ? FDTD_OK : fail2(FDTD_E_NONFINITE, "a probe spectrum holds NaN or Inf");
}

int fdtd2d_get_fields(fdtd2d *h, int32_t which, double *out)
{
    int rc = check2(h);
    if (rc) return rc;
    if (!out) return fail2(FDTD_E_INVALID, "output pointer is NULL");
    const Plan2 &p = h->p;
    if (which < 0 || which >= 2 * p.ncomp + p.nh) return fail2(FDTD_E_INVALID, "which %d out of range", which);
    const int64_t N = p.N;
    if (which < p.ncomp + p.nh) {
        const void *src = which < p.ncomp ? h->E[h->cur][which] : h->H[h->cur][which - p.ncomp];
        std::vector<char> buf(p.es * N);
        HIP_TRY2(hipMemcpyAsync(buf.data(), src, p.es * N, hipMemcpyDeviceToHost, h->stream));
        HIP_TRY2(hipStreamSynchronize(h->stream));
        for (int64_t k = 0; k < N; ++k)
            out[k] = p.es == 8 ? ((const double *)buf.data())[k] : (double)((const float *)buf.data())[k];
        return FDTD_OK;
    }
    const int c = which - p.ncomp - p.nh;
    std::vector<double> Jc(std::max<int64_t>(p.S, 1));
    if (p.S) {
        HIP_TRY2(hipMemcpyAsync(Jc.data(), h->J[h->cur][c], 8 * p.S, hipMemcpyDeviceToHost, h->stream));
        HIP_TRY2(hipStreamSynchronize(h->stream));
    }
    std::memset(out, 0, 8 * N);
    for (int64_t i = 0; i < h->d.nx; ++i)
        for (int64_t j = p.span[i].x; j < p.span[i].y; ++j) out[i * h->d.ny + j] = Jc[p.rowoff[i] + j - p.span[i].x];
    return FDTD_OK;
}

int fdtd2d_steps_done(fdtd2d *h, int64_t *steps)
{
    if (!h || !steps) return fail2(FDTD_E_INVALID, "NULL argument");
    *steps = h->steps;
    return FDTD_OK;
}

int fdtd2d_destroy(fdtd2d *h)
{
    if (!h) return FDTD_OK;
    (void)hipStreamSynchronize(h->stream);
    if (h->side) (void)hipStreamSynchronize(h->side);
    for (auto &kv : h->graphs) (void)hipGraphExecDestroy(kv.second);
    if (h->side) (void)hipStreamDestroy(h->side);
    if (h->ev_fork) (void)hipEventDestroy(h->ev_fork);
    if (h->ev_join) (void)hipEventDestroy(h->ev_join);
    if (h->owns && h->ws) (void)hipFree(h->ws);
    delete h;
    return FDTD_OK;
}

}  // extern "C"
