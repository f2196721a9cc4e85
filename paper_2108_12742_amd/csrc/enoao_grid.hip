// enoao_grid.hip -- the 2D Runge-Kutta stage (gfx950): one kernel for both
// directions, and one for the faces whose flux is not the top candidate's.
//
// stage_2d.  A wave owns a strip of columns, one lane per column, and marches along
// y.  Per row it loads U once and keeps, in registers, the last rows' U and y-flux
// for the y-faces; the x-faces of a row come from the neighbouring lanes (through a
// row buffer in LDS private to the wave); L = L_x + L_y, the stage combine and the
// maxima of the new state follow at once.  The state is read once and written once
// per stage and nothing else goes through memory: the split sweeps this replaces
// wrote L_x, read it back and read the stage input twice (544 bytes a cell-update
// against 256), and staged 12 quantities and 8 differences per node in LDS for 108
// LDS instructions a face against 60 for both faces of a cell.  Waves never
// synchronise with one another.
//
// What a face costs.  Where the window is smooth every field takes its top
// candidate on both sides, and the flux is linear in the window: Fhat = S F / 2 +
// R (kappa alpha L D_1 U) / 2 (TopStencil; R L = I, so the central part needs no
// projection).  That it is so follows, for nearly all such faces, from one bound on
// the indicators: |l.(D F +- alpha D U)| <= |l|_1 max_c(|D F_c| + alpha |D U_c|),
// formed with D_1, which both sides share, and compared with delta over a bound of
// the left eigenvectors' row sums.  (On developed flows the bound leaves 11% of the
// 64-face rows, the exact indicators 10%.)
//
// fix_2d.  The faces that the bound leaves are few (2 to 7%) but each costs ten
// others, and they lie along shocks, so a wave that met them in its strip worked
// several times as long as its neighbours: selecting inside stage_2d took 0.10 ms
// of a 0.23 ms stage for 15% more instructions, and the selection's registers
// spilled the row loop's.  stage_2d therefore lists the rows of a strip that hold such
// faces and gives those faces the mean (F_j + F_j+1) / 2 of their own two nodes; fix_2d
// spreads pieces of the listed rows over the machine, selects, one lane per face and field, and
// adds what the chosen candidates have beyond the mean to the cells: U += c dt dL.  The
// mean, and not the top flux: the top candidate was left out because its window crosses
// a jump, it is as large as the jump's far side, and the cells of the near side kept
// that side's rounding (1e-9 of the largest L at a pressure ratio of 1e5).  The bound
// alone tells which form a face takes, also where every face is selected.
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <type_traits>

#include "enoao_common.hpp"
#include "enoao_device.hpp"
#include "enoao_kernels.hpp"
#include "enoao_wave.hpp"

namespace enoao {

// Waves per SIMD of stage_2d: 247 to 256 registers.
constexpr int STAGE_WAVES = 2;
// Waves per SIMD of fix_2d: as many as its LDS lets a CU hold (40 KB a workgroup at
// order 5, 44 KB at order 7).
constexpr int fix_waves(int order) { return order == 7 ? 3 : 4; }

// p at a byte offset.  Offsets within a plane below 4 GiB take one 32-bit register
// (unsigned) beside a wave-uniform address; larger planes take 64-bit offsets, in the
// recording instantiations, which also serve members that large without a record, and
// runs that list every face.
template <class Off> __device__ __forceinline__ double row_load(const GMEM double *p, Off off)
{
    return *(const GMEM double *)((const GMEM char *)p + off);
}
template <class Off> __device__ __forceinline__ void row_store(GMEM double *p, Off off, double x)
{
    *(GMEM double *)((GMEM char *)p + off) = x;
}

__device__ __forceinline__ unsigned long long lane_bits(unsigned long long x, int i)
{
    return (unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(unsigned)x, i) |
           (unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(x >> 32), i) << 32;
}

// a launch's values of one member
struct GridView {
    long long u0, u1;  // its units in the list
    int k, nx, ny, pitch, bcx, bcy, strips;
    unsigned low, extra;  // rows of a unit: low, one more in the first `extra` blocks
    double inv_strips;
    int active;
    const GMEM double *in;
    GMEM double *out;
    const GMEM double *base;
    GMEM uint8_t *sel;
    GMEM unsigned long long *amax;
    GMEM Ctrl *ctrl;
    double idx, idy, dt;
    double ax[4], ay[4];  // kappa alpha / 2 per field along x and along y
    double mx, my;        // the largest alpha along x and along y
    double rx[3], ry[3];  // alpha of the fields u-c, u, u+c (component-wise: one for all)
};

// a value of a descriptor whose 8-byte words the lanes hold
template <class T> __device__ __forceinline__ T inst_value(unsigned long long words, unsigned offset)
{
    static_assert(sizeof(T) == 4 || sizeof(T) == 8, "a word or half of one");
    const unsigned long long w = lane_bits(words, (int)offset / 8) >> (offset % 8 * 8);
    union { unsigned long long w; T v; } a;
    a.w = w;
    return a.v;
}
#define INST_VALUE(name) inst_value<decltype(Inst::name)>(words, offsetof(Inst, name))

template <int ORDER, bool CH>
__device__ __forceinline__ GridView grid_view(const KParams &P, int n_inst, long long unit)
{
    GridView v;
    // (a lone member's control block and maxima are kernel arguments, so their loads do
    // not wait for the descriptor's, which is read at once, a word a lane: value by value it
    // took six loads one after the other)
    v.k = P.lone_ctrl ? 0 : uniform(find_last(n_inst, unit, [&](int i) { return P.inst[i].unit0; }));
    const int lane = threadIdx.x & 63;
    static_assert(sizeof(Inst) % 8 == 0 && sizeof(Inst) <= 512, "a lane per word of a descriptor");
    const unsigned long long words = gmem((const unsigned long long *)(P.inst + v.k))[min(lane, (int)sizeof(Inst) / 8 - 1)];
    v.ctrl = gmem(P.lone_ctrl ? P.lone_ctrl : INST_VALUE(ctrl));
    v.amax = gmem(P.lone_ctrl ? P.lone_amax : INST_VALUE(amax));
    // one lane per value and copy of the stage input's maxima
    double am = as_double(v.amax[P.r_in * amax_slot_words(EULER2D) + lane]);
    const int done = v.ctrl->done;
    const double dt = v.ctrl->dt;
    v.u0 = INST_VALUE(unit0);
    v.u1 = v.u0 + INST_VALUE(units);
    v.nx = INST_VALUE(nx);
    v.ny = INST_VALUE(ny);
    v.pitch = INST_VALUE(pitch);
    v.bcx = INST_VALUE(bcx);
    v.bcy = INST_VALUE(bcy);
    v.strips = INST_VALUE(strips);
    v.low = (unsigned)INST_VALUE(low_rows);
    v.extra = (unsigned)INST_VALUE(extra_rows);
    v.inv_strips = INST_VALUE(inv_strips);
    v.active = uniform(done) == 0;
    v.dt = uniform(dt);
    double *const u = INST_VALUE(u), *const w1 = INST_VALUE(w1), *const w2 = INST_VALUE(w2);
    v.in = gmem(P.mode == M_S2 ? w1 : (P.mode == M_S3 ? w2 : u));
    v.out = gmem(P.mode == M_RHS ? INST_VALUE(lx) : (P.mode == M_S1 ? w1 : (P.mode == M_S2 ? w2 : u)));
    v.base = gmem(u);
    v.sel = gmem(INST_VALUE(sel));
    if (v.sel && P.sel_slot > 0) {
        // records of one evaluation: x block [4][2][ny][nx+1], then the y block [4][2][ny+1][nx]
        v.sel += (long long)P.sel_slot * 8ll * ((long long)v.ny * (v.nx + 1) + (long long)(v.ny + 1) * v.nx);
    }
    v.idx = uniform(1.0 / INST_VALUE(dx));
    v.idy = uniform(1.0 / INST_VALUE(dy));
    am = copies_max(am);
    double ax[3], ay[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        ax[i] = lane_value(am, i);
        ay[i] = lane_value(am, 3 + i);
    }
    if constexpr (!CH) {
        // one alpha for all components: max(|u| + c) = max(max|u - c|, max|u + c|)
        ax[0] = ax[1] = ax[2] = fmax(ax[0], ax[2]);
        ay[0] = ay[1] = ay[2] = fmax(ay[0], ay[2]);
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int i = s == 0 ? 0 : (s == 3 ? 2 : 1);
        v.ax[s] = uniform(ax[i] * (TopStencil<ORDER>::kappa * 0.5 / fscale<4, CH>(s)));
        v.ay[s] = uniform(ay[i] * (TopStencil<ORDER>::kappa * 0.5 / fscale<4, CH>(s)));
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        v.rx[i] = uniform(ax[i]);
        v.ry[i] = uniform(ay[i]);
    }
    v.mx = uniform(fmax(ax[0], fmax(ax[1], ax[2])));
    v.my = uniform(fmax(ay[0], fmax(ay[1], ay[2])));
    return v;
}

// Stage combine (Shu-Osher form): base u^n + y (in + dt L).  The stages of a step share
// one instantiation: launched in turn they would otherwise each fetch 17 KB of code
// that the last one evicted, a good part of a small problem's time.
struct RkWeights {
    double base, y;
};
__device__ __forceinline__ RkWeights rk_weights(int mode)
{
    if (mode == M_S2) return RkWeights{0.75, 0.25};
    if (mode == M_S3) return RkWeights{1.0 / 3.0, 2.0 / 3.0};
    return RkWeights{0.0, 1.0};
}

// columns from x0, rows y0 .. y1 - 1 of a unit: strips along a row follow one another
struct UnitBox {
    int x0, y0, y1;
};
__device__ __forceinline__ UnitBox unit_box(const GridView &v, long long unit, int cells)
{
    // (lu + 1/2) / strips lies at least 1 / (2 strips) from a whole number, its rounding
    // error far below that: exact, and a tenth of a division's instructions
    const unsigned lu = (unsigned)(unit - v.u0), b = uniform((unsigned)((lu + 0.5) * v.inv_strips));
    UnitBox u;
    u.x0 = (int)(lu - b * (unsigned)v.strips) * cells;
    u.y0 = (int)(b * v.low + min(b, v.extra));
    u.y1 = u.y0 + (int)(v.low + (b < v.extra ? 1u : 0u));
    return u;
}

// A wave's running maxima live in LDS, one column per lane (non-negative doubles
// as bit patterns: integer max): seven registers pairs fewer across the row loop.
struct WaveMax {
    unsigned long long v[7][64];
};

// U in the natural component order: maxima of the wave speeds, non-physical flag
__device__ __forceinline__ bool wave_max_add(WaveMax &M, int lane, const double (&U)[4], double gamma, double idx,
                                             double idy)
{
    Maxima<EULER2D> m;
    m.reset();
    m.add(U, gamma, idx, idy);
#pragma unroll
    for (int i = 0; i < 7; ++i)
        __hip_atomic_fetch_max(&M.v[i][lane], as_bits(m.v[i]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    return m.bad != 0;
}

// The maxima of the n lanes' columns M[0 .. n-1] into the member's slot, one atomic
// per value, by one wave; the columns start again at zero.
__device__ __forceinline__ void wave_flush(WaveMax *M, int n, unsigned long long bad, GMEM unsigned long long *amax,
                                           GMEM Ctrl *ctrl, int slot)
{
    const int lane = threadIdx.x & 63;
    double mine = 0.0;
    wave_sync();
#pragma unroll 1
    for (int i = 0; i < 7; ++i) {
        unsigned long long m = 0ull;
        for (int k = 0; k < n; ++k) {
            m = max(m, M[k].v[i][lane]);
            M[k].v[i][lane] = 0ull;
        }
        const double x = wave_max(as_double(m));
        if (lane == i) mine = x;
    }
    if (slot >= 0 && lane < 7)
        __hip_atomic_fetch_max(&amax[slot * amax_slot_words(EULER2D) + blockIdx.x % amax_copies(EULER2D) * AMAX_VALS + lane],
                               as_bits(mine), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (bad && lane == 0) __hip_atomic_fetch_or(&ctrl->status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// sqrt(rho), velocities, total enthalpy and pressure of a node
struct NodePrim {
    double s, u, v, H, p;
};
__device__ __forceinline__ double node_pressure(double rho, double u, double v, double E, double gm1)
{
    return gm1 * fma(-0.5 * rho, fma(u, u, v * v), E);
}
__device__ __forceinline__ NodePrim node_prim(double rho, double m, double n, double E, double gm1)
{
    NodePrim q;
    const double ir = rcp_nr(rho);
    q.u = m * ir;
    q.v = n * ir;
    q.p = node_pressure(rho, q.u, q.v, E, gm1);
    q.s = sqrt_nr(rho);
    q.H = (E + q.p) * ir;
    return q;
}

// Bound of the left eigenvectors' scaled row sums of a face (acoustic rows halved
// to the window scale of the others), so that every indicator of the face is at
// most this times the node bound.  Component-wise variables: 1.  (NaN for a state whose
// eigenvectors do not exist: fmax would drop it.)
template <bool CH> __device__ __forceinline__ double row_bound(const RoeState &r)
{
    if constexpr (!CH) return 1.0;
    const double au = 1.0 + fabs(r.u), av = fabs(r.v);
    const double x = fma(r.b1, au + av, r.b2);
    return fmax(fmax(1.0 + x, 0.5 * fma(r.ic, au, x)), fma(0.0, x, 1.0 + av));
}

// Node bound max_c(|D F_c| + alpha |D U_c|); F_0 is U_1.  dF[0] holds the pressure, so it
// tells a NaN in any component of a node, which fmax drops.
__device__ __forceinline__ double node_bound(const double (&dU)[4], const double (&dF)[3], double amax)
{
    double b = fma(amax, fabs(dU[0]), fabs(dU[1]));
#pragma unroll
    for (int k = 0; k < 3; ++k) b = fmax(b, fma(amax, fabs(dU[k + 1]), fabs(dF[k])));
    return fma(0.0, dF[0], b);
}

// Flux of a face whose fields all take the top candidate on both sides:
// S F / 2 + R (kappa alpha L D_1 U) / 2; ka: kappa alpha / 2 per field.
template <bool CH>
__device__ __forceinline__ void top_flux(const RoeState &r, const double (&sF)[4], const double (&dU)[4],
                                         const double (&ka)[4], double (&Fh)[4])
{
    double w[4];
    to_fields<4, CH>(r, dU, w);
#pragma unroll
    for (int s = 0; s < 4; ++s) w[s] *= ka[s];
    from_fields<4, CH>(r, w, Fh);
#pragma unroll
    for (int c = 0; c < 4; ++c) Fh[c] = fma(0.5, sF[c], Fh[c]);
}

// A listed piece of a row: unit << 28 | row within the unit << 12 | FIX_LAST for the row's
// last piece | its number << 6 | faces a piece (0: the whole row), and the lanes of the
// row whose faces need a selection: right of the lane's column, below and above the row.
// A piece has the cells with as many of these faces before them as its number and that
// size say; fix_2d cuts it out.  Where every face is listed a piece has FIX_SPLIT
// cells, and the lanes that hold a top flux are marked once more, half a turn on.
constexpr unsigned FIX_LAST = 1u << 9;
__device__ __forceinline__ unsigned long long half_turn(unsigned long long m) { return m << 32 | m >> 32; }
struct FixEntry {
    unsigned long long where, x, below, above;
};
static_assert(sizeof(FixEntry) == FIX_ENTRY_BYTES, "list sizes");

template <int ORDER, bool STEP, bool REC, bool CH>
__global__ __launch_bounds__(BLOCK)
__attribute__((amdgpu_waves_per_eu(STAGE_WAVES))) void stage_2d(KParams P)
{
    using T = TopStencil<ORDER>;
    using Off = std::conditional_t<REC, long long, unsigned>;
    constexpr int H = ReconTraits<ORDER>::H, G = H + 1, K = ReconTraits<ORDER>::K;
    constexpr int NS = 2 * H;                  // rows (columns) a difference or central stencil spans
    constexpr int CELLS = strip_cells(ORDER);  // columns a wave updates
    constexpr int ROW = 64 + 2 * G;            // row buffer: lane l's node at l + H
    static_assert(CELLS == 64 - 2 * G, "a lane per column, halo included");
    // The mean flux of the faces that the bound leaves: by a select in every row, or under a
    // branch.  The branch lets order 7 run two waves per SIMD (2048^2, four steps: 2.57 ms
    // against 3.25 with selects, at one wave); at order 5, where both fit, it takes the
    // schedule more (eight steps: 4.45 ms against 4.32).
    constexpr bool MEAN_SELECT = ORDER == 5;
    constexpr int NWV = BLOCK / 64, PENDING = 16;
    __shared__ double rows[NWV][7][ROW];
    __shared__ WaveMax maxima[STEP ? NWV : 1];
    __shared__ FixEntry pending[NWV][PENDING];

    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double(&rb)[7][ROW] = rows[wv];
    const int n_inst = P.hdr->n_inst;
    const long long units = P.hdr->units_total;
    // Consecutive units (neighbouring strips of the same rows, which share their halo
    // columns) go to one XCD's L2: workgroups are dealt to the eight XCDs in turn.
    const unsigned g = gridDim.x;
    const unsigned blk = g % 8 == 0 ? (blockIdx.x % 8) * (g / 8) + blockIdx.x / 8 : blockIdx.x;
    const long long stride = (long long)g * NWV;
    // threshold of the bound (it and the indicators differ by rounding); delta = 0
    // leaves every face to the selection
    const double thr = P.delta > 0.0 ? 2.0 * P.delta * (1.0 - 1.0 / 1024.0) : -1.0;
    const bool full = REC && (P.flags & KF_FULL_SELECTION) != 0;  // every face is listed

    const RkWeights rk = rk_weights(P.mode);
    WaveMax &M = maxima[STEP ? wv : 0];
    unsigned long long bad = 0;
    if (STEP) {
#pragma unroll
        for (int i = 0; i < 7; ++i) M.v[i][lane] = 0ull;
    }
    // the pending entries of a unit to its range's list: those of two passes are in the
    // first n_two places of `pending`, those of one in the last n_one
    unsigned n_two = 0, n_one = 0;
    const unsigned per_range = fix_range_units(units);
    auto flush_pending = [&](long long unit) {
        if (n_two + n_one == 0) return;
        wave_sync();
        const unsigned range = (unsigned)unit / per_range;
        unsigned long long at = 0;
        if (lane == 0)
            at = __hip_atomic_fetch_add(gmem(P.fix_count) + range * FIX_COUNTER_STRIDE,
                                        (unsigned long long)(0u - n_one) << 32 | n_two, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        at = lane_bits(at, 0);
        const unsigned e = lane >> 2;
        const bool two = e < n_two;
        if (two || e >= PENDING - n_one) {
            const unsigned long long *src = &pending[wv][0].where;
            const unsigned to = two ? (unsigned)at + e : (unsigned)(at >> 32) + e - PENDING;
            gmem(P.fix_list)[4ull * to + (lane & 3)] = src[lane];
        }
        wave_sync();
        n_two = n_one = 0;
    };
    GridView v;
    v.u0 = 0;
    v.u1 = -1;
    bool have = false;
    if (P.lone_ctrl) v = grid_view<ORDER, CH>(P, n_inst, 0);  // (its loads beside the header's)
    for (long long unit = (long long)blk * NWV + wv; unit < units; unit += stride) {
        if (unit >= v.u1) {
            if (STEP && have) wave_flush(&M, 1, bad, v.amax, v.ctrl, P.r_out);
            bad = 0;
            v = grid_view<ORDER, CH>(P, n_inst, unit);
        }
        have = v.active != 0;
        if (!have) continue;
        static_assert(amax_slot_words(EULER2D) == 64, "a lane per word of a slot");
        if (STEP && P.r_zero >= 0 && unit == v.u0) v.amax[P.r_zero * 64 + lane] = 0ull;
        const int nx = v.nx, ny = v.ny;
        const long long plane = (long long)v.pitch * ny;
        const UnitBox box = unit_box(v, unit, CELLS);
        const int x0 = box.x0, y0 = box.y0, y1 = box.y1;
        const int xn = x0 - G + lane;
        const Off xc = 8 * (Off)bc_map(xn, nx, v.bcx);  // byte offset along a row
        const bool cell = lane >= G && lane < 64 - G && xn < nx;
        const bool face = lane >= H && lane < 64 - G && xn < nx;
        // rows y0 - H .. y1 - 1 + H, the newest r; w[.][NS-1] is row r.  Quantities: rho,
        // n, m, E (n the momentum along y) and the y-fluxes of n, m, E.  Row r completes
        // the y-face between rows r - H and r - H + 1 and with it the cells of row r - H.
        double w[7][NS];
        double pre[4];
        NodePrim pl;                      // row r - H
        double Gm[4];                     // y-flux below row r - H
        unsigned long long fail_b = 0;    // its faces that the bound leaves
        auto load_row = [&](int r) {
            const int y = r < 0 || r >= ny ? bc_map(r, ny, v.bcy) : r;
            const GMEM double *p = v.in + (long long)y * v.pitch;
            pre[0] = row_load(p, xc);
            pre[1] = row_load(p + 2 * plane, xc);
            pre[2] = row_load(p + plane, xc);
            pre[3] = row_load(p + 3 * plane, xc);
        };
        auto flux_row = [&](int t) {
            const double rho = w[0][t], n = w[1][t], m = w[2][t], E = w[3][t];
            const double ir = rcp_nr(rho), u = m * ir, vv = n * ir;
            const double p = node_pressure(rho, u, vv, E, P.gm1);
            w[4][t] = fma(n, vv, p);
            w[5][t] = n * u;
            w[6][t] = (E + p) * vv;
        };
        const int rend = y1 + H;
        // the rows above the unit's first face, their loads in flight together
#pragma unroll
        for (int t = 1; t < NS; ++t) {
            load_row(y0 - H + t - 1);
#pragma unroll
            for (int q = 0; q < 4; ++q) w[q][t] = pre[q];
        }
        load_row(y0 + H - 1);
#pragma unroll
        for (int t = 1; t < NS; ++t) flux_row(t);
        pl = node_prim(w[0][H], w[2][H], w[1][H], w[3][H], P.gm1);  // row y0 - 1
#pragma unroll 1
        for (int r = y0 + H - 1; r < rend; ++r) {
            const int j = r - H;  // row updated in this pass
#pragma unroll
            for (int q = 0; q < 7; ++q)
#pragma unroll
                for (int t = 0; t + 1 < NS; ++t) w[q][t] = w[q][t + 1];
#pragma unroll
            for (int q = 0; q < 4; ++q) w[q][NS - 1] = pre[q];
            if (r + 1 < rend) load_row(r + 1);
            flux_row(NS - 1);
            __builtin_amdgcn_sched_barrier(0);
            if (j >= y0) {
                // row j for its x-faces below (written early: the y-face's arithmetic covers
                // the exchange)
                const double m = w[2][H - 1], E = w[3][H - 1];
                rb[0][lane + H] = w[0][H - 1];
                rb[1][lane + H] = m;
                rb[2][lane + H] = w[1][H - 1];
                rb[3][lane + H] = E;
                rb[4][lane + H] = fma(m, pl.u, pl.p);
                rb[5][lane + H] = m * pl.v;
                rb[6][lane + H] = (E + pl.p) * pl.u;
            }
            const NodePrim pr = node_prim(w[0][H], w[2][H], w[1][H], w[3][H], P.gm1);  // row r - H + 1
            double Fy[4];
            unsigned long long fail_t;
            {
                // y-face j + 1/2
                double sF[4], dU[4], dF[3];
                sF[0] = T::sym1(w[1], 1);
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    sF[k + 1] = T::sym1(w[4 + k], 1);
                    dF[k] = T::diff(w[4 + k], 1);
                }
#pragma unroll
                for (int c = 0; c < 4; ++c) dU[c] = T::diff(w[c], 1);
                __builtin_amdgcn_sched_barrier(0);
                RoeState ro{};
                if constexpr (CH) ro = roe_state(pl.s, pl.v, pl.u, pl.H, pr.s, pr.v, pr.u, pr.H, P.gm1);
                top_flux<CH>(ro, sF, dU, v.ay, Fy);
                const bool ok = row_bound<CH>(ro) * node_bound(dU, dF, v.my) <= thr;
                fail_t = __builtin_amdgcn_ballot_w64(!ok && cell);
                if (MEAN_SELECT || fail_t) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const int q = c == 0 ? 1 : 3 + c;
                        Fy[c] = ok ? Fy[c] : 0.5 * (w[q][H - 1] + w[q][H]);
                    }
                }
            }
            if (REC && v.sel && !full && cell && !((fail_t >> lane) & 1)) {
                const long long xb = (long long)ny * (nx + 1), yb = (long long)(ny + 1) * nx;
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    v.sel[8 * xb + i * yb + (long long)(j + 1) * nx + xn] = (uint8_t)(K - 1);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (j >= y0) {
                double ub[4] = {0.0, 0.0, 0.0, 0.0};
                if (STEP && P.mode != M_S1) {
                    const GMEM double *p = v.base + (long long)j * v.pitch;
#pragma unroll
                    for (int c = 0; c < 4; ++c) ub[c] = row_load(p + c * plane, xc);
                }
                // x-faces of row j: lane l's face is between columns l and l + 1
                wave_sync();
                double sx[4], dx[4], df[3], mean[4];
#pragma unroll
                for (int i = 0; i < 7; ++i) {
                    double win[NS];
#pragma unroll
                    for (int t = 0; t < NS; ++t) win[t] = i < 4 && t == H - 1 ? w[i == 1 ? 2 : (i == 2 ? 1 : i)][H - 1] : rb[i][lane + 1 + t];
                    if (i == 1 || i >= 4) {
                        sx[i == 1 ? 0 : i - 3] = T::sym1(win, 1);
                        mean[i == 1 ? 0 : i - 3] = 0.5 * (win[H - 1] + win[H]);
                    }
                    if (i < 4) dx[i] = T::diff(win, 1);
                    else df[i - 4] = T::diff(win, 1);
                    if (i % 2 == 1) __builtin_amdgcn_sched_barrier(0);
                }
                __builtin_amdgcn_sched_barrier(0);
                RoeState ro{};
                if constexpr (CH)
                    ro = roe_state(pl.s, pl.u, pl.v, pl.H, lane_next(pl.s), lane_next(pl.u), lane_next(pl.v),
                                   lane_next(pl.H), P.gm1);
                double Fx[4];
                top_flux<CH>(ro, sx, dx, v.ax, Fx);
                const bool ok = row_bound<CH>(ro) * node_bound(dx, df, v.mx) <= thr;
                const unsigned long long fail_x = __builtin_amdgcn_ballot_w64(!ok && face);
                if (MEAN_SELECT || fail_x) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const double *f = &rb[c == 0 ? 1 : 3 + c][lane + H];
                        Fx[c] = ok ? Fx[c] : (MEAN_SELECT ? mean[c] : 0.5 * (f[0] + f[1]));
                    }
                }
                if (REC && v.sel && !full && face && !((fail_x >> lane) & 1)) {
                    const long long xb = (long long)ny * (nx + 1);
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        v.sel[i * xb + (long long)j * (nx + 1) + xn + 1] = (uint8_t)(K - 1);
                }
                // cells with a listed face: their maxima are fix_2d's
                const unsigned long long fixed = full ? ~0ull : fail_x | (fail_x << 1) | fail_b | fail_t;
                if (fixed) {
                    const unsigned long long where = (unsigned long long)unit << 28 | (unsigned)(j - y0) << 12;
                    const int faces = __popcll(fail_x) + __popcll(fail_b) + __popcll(fail_t), places = fix_places(nx);
                    // pieces of `most` faces, a cell's three more and the one on its left again
                    constexpr int MOST = FIX_FACES - 3;
                    int pieces = min(places, 1 + (faces > FIX_FACES) + (faces > 2 * MOST) + (faces > 3 * MOST) +
                                                 (faces > 4 * MOST) + (faces > 5 * MOST));
                    // (a narrow grid's row of n cells has 3 n + 1 faces at most)
                    static_assert(6 * MOST >= 3 * CELLS + 1 && FIX_SPLIT == 10, "places of a row");
                    int most = faces > MOST * pieces ? MOST + 2 : MOST;
                    int rest = faces - (pieces - 1) * most;  // (about: the last one's)
                    unsigned long long x = fail_x, b = fail_b, t = fail_t;
                    if (full) {
                        // every face; those with a top flux twice (lane k: those of piece k)
                        const unsigned long long m = ((1ull << FIX_SPLIT) - 1) << ((G + FIX_SPLIT * lane) & 63);
                        const unsigned long long fs = __builtin_amdgcn_ballot_w64(face) & (m | m >> 1);
                        const unsigned long long cs = __builtin_amdgcn_ballot_w64(cell) & m;
                        x = fs | half_turn(fs & ~x);
                        b = cs | half_turn(cs & ~b);
                        t = cs | half_turn(cs & ~t);
                        pieces = min(places, (nx - x0 + FIX_SPLIT - 1) / FIX_SPLIT);  // (those with cells)
                        most = rest = FIX_FACES;
                    }
                    if (pieces == 1 && !full) most = 0;
                    const unsigned one = rest <= FIX_PASS ? 1u : 0u;
                    if (lane < pieces) {
                        const bool last = lane == pieces - 1;
                        pending[wv][last && one ? PENDING - 1 - n_one : n_two + lane] =
                            FixEntry{where | (last ? FIX_LAST : 0u) | (unsigned)(lane << 6 | most), x, b, t};
                    }
                    n_two += pieces - one;
                    n_one += one;
                    if (n_two + n_one > PENDING - 6) flush_pending(unit);
                }
                __builtin_amdgcn_sched_barrier(0);
                const int perm[4] = {0, 2, 1, 3};
                double L[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const double lx = -(Fx[c] - lane_prev(Fx[c])) * v.idx;
                    L[c] = lx - (Fy[perm[c]] - Gm[perm[c]]) * v.idy;
                }
                bool b = false;
                if (cell) {
                    const long long o = (long long)j * v.pitch;
                    if constexpr (!STEP) {
#pragma unroll
                        for (int c = 0; c < 4; ++c) row_store(v.out + o + c * plane, xc, L[c]);
                    } else {
                        double Un[4];
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            Un[c] = fma(rk.base, ub[c], rk.y * fma(v.dt, L[c], w[perm[c]][H - 1]));
                            row_store(v.out + o + c * plane, xc, Un[c]);
                        }
                        if (!((fixed >> lane) & 1)) b = wave_max_add(M, lane, Un, P.gamma, v.idx, v.idy);
                    }
                }
                if (STEP) bad |= __builtin_amdgcn_ballot_w64(b);
                wave_sync();
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) Gm[c] = Fy[c];
            fail_b = fail_t;
            pl = pr;
        }
        flush_pending(unit);
    }
    if constexpr (STEP) {
        // The waves of a workgroup that end in one member (mostly all) flush together:
        // every wave's atomics go to the member's one cache line (with 1800 waves doing
        // so by themselves a stage of 504 x 400 nodes took 28 us against 17.5 without).
        __shared__ int last[NWV];
        if (lane == 0) last[wv] = have ? v.k : -1;
        if (bad && lane == 0) __hip_atomic_fetch_or(&v.ctrl->status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        bool same = have;
#pragma unroll
        for (int k = 0; k < NWV; ++k) same = same && (last[k] == v.k || last[k] < 0);
        if (same) {
            // the first wave with work; the others' columns are its, or zero
            int k0 = 0;
#pragma unroll
            for (int k = NWV - 1; k >= 0; --k) k0 = last[k] >= 0 ? k : k0;
            if (wv == k0) wave_flush(maxima, NWV, 0ull, v.amax, v.ctrl, P.r_out);
        } else if (have) {
            wave_flush(&M, 1, 0ull, v.amax, v.ctrl, P.r_out);
        }
    }
}

// Scratch of a wave of fix_2d (LDS).  A row segment has at most 57 x-faces and 56
// y-faces on either side.
using WaveMost = unsigned long long[7][4];
template <int NW> struct FixScratch {
    double dF[3][4][58];       // fluxes beyond the mean by set (x, below, above) and lane from H on
    double exchange[NW][64];   // window values by node and (face, field)
    double member[20];         // the member's alpha along x and along y by field, 1/dx, 1/dy, the weight of dL; the
                               // maxima of its new state so far, from 12 on
    unsigned char face[176];   // set << 6 | lane of each face
    WaveMost most;             // the wave's maxima, in four parts
};

// node k of n on a line, k at most a window beyond either end (small: n may be less than that)
__device__ __forceinline__ int line_node(int k, int n, bool periodic, bool small)
{
    if (small) return bc_map(k, n, periodic ? BC_PERIODIC : BC_TRANSMISSIVE);
    const int wrapped = k + (k < 0 ? n : (k >= n ? -n : 0));
    return periodic ? wrapped : min(max(k, 0), n - 1);
}

// alpha of field s from those of u-c, u, u+c
__device__ __forceinline__ double field_alpha(const double (&r)[3], int s) { return s == 0 ? r[0] : (s == 3 ? r[2] : r[1]); }

// A wave takes one listed piece of a row at a time (handing them out from a counter took
// longer than the imbalance it removed, 20 ns each); where the list is short, the four
// waves of a workgroup share a piece.
// Four lanes per face, one per field, for the selection, one lane per cell for the
// update.  stage_2d gave the mean of the fluxes of the face's two nodes; a field
// contributes alpha l.(U_j - U_j+1) / 2 and what its chosen candidates have beyond the
// two nodes.
// A pass of sixteen faces takes a SIMD about 1 us however many waves are on it, so the
// launch lasts as long as its fullest SIMD: pieces of one to five passes left 14 on one
// beside 9.4 on average (56 x 1532); pieces of one or two, those of two dealt first, leave
// 9.  The member's values come beside the lists' counters, and a wave adds to the member's
// maxima only what exceeds stage_2d's.  With that, and 430 VALU instructions a pass instead
// of 570, before and now (us, same card): 1000 x 60, six steps, 611 and 512; order 7 on
// 60 x 1200 829 and 756; 511 x 257, ten, 1060 and 897; 2048^2, eight, 4100 and 3940; a pool
// of 16 4610 and 4010.
template <int ORDER, bool STEP, bool REC, bool CH>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(fix_waves(ORDER)))) void fix_2d(KParams P)
{
    using R = Recon<ORDER>;
    using Off = std::conditional_t<REC, long long, unsigned>;
    constexpr int H = R::H, G = H + 1, NW = 2 * H + 2, CELLS = strip_cells(ORDER), NWV = BLOCK / 64;
    __shared__ FixScratch<NW> scratch[NWV];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n_inst = P.hdr->n_inst;
    GridView v;
    v.u0 = 0;
    v.u1 = -1;
    auto enter = [&](long long unit) {
        v = grid_view<ORDER, CH>(P, n_inst, unit);
        // (in LDS: the loops below run out of scalar registers)
        double x = lane < 4 ? field_alpha(v.rx, lane) : field_alpha(v.ry, lane & 3);
        x = lane < 8 ? x : (lane == 8 ? v.idx : (lane == 9 ? v.idy : rk_weights(P.mode).y * v.dt));
        if (lane < 11) scratch[wv].member[lane] = x;
        // what stage_2d has left in the maxima already: most waves have no more to add
        // (thousands of atomics on a few lines at a launch's end, 20 ns each)
        if (STEP) {
            const double seen = copies_max(as_double(v.amax[P.r_out * amax_slot_words(EULER2D) + lane]));
            if (lane < AMAX_VALS) scratch[wv].member[12 + lane] = seen;
        }
    };
    // lane c: list c's pieces of two passes, lane FIX_RANGES + c: those of one; upto: the
    // entries up to them.  Entry i of all is at skew + i, counted back among those of one.
    static_assert(2 * FIX_RANGES == 64, "a lane per list and end");
    const bool two = lane < FIX_RANGES;
    const unsigned long long counted = gmem(P.fix_count)[lane % FIX_RANGES * FIX_COUNTER_STRIDE];
    const unsigned long long empty = fix_empty(P, lane % FIX_RANGES);
    if (P.lone_ctrl) enter(0);  // (beside the counters' loads: 2 us of a short launch)
    if (P.fix_zero && blockIdx.x == gridDim.x - 1 && wv == 0 && two) gmem(P.fix_zero)[FIX_COUNTER_STRIDE * lane] = empty;
    const unsigned list_end = two ? (unsigned)empty : (unsigned)(empty >> 32);
    unsigned upto = two ? (unsigned)counted - list_end : list_end - (unsigned)(counted >> 32);
    const unsigned mine_n = upto;
    upto = wave_scan(upto);
    const unsigned entries = (unsigned)__builtin_amdgcn_readlane((int)upto, 63);
    if (entries == 0) return;
    const unsigned skew = two ? list_end - (upto - mine_n) : list_end - 1 + (upto - mine_n);
    // Few entries leave waves idle: the four waves of a workgroup share one, which pays up to
    // an entry for two workgroups, at order 7, whose passes are longer, up to one for each
    // (six steps, us with and without: 64^2 365 and 380, 100^2 391 and 381; order 7 64^2 392
    // and 420, 100^2 406 and 415, 128^2, where there are more than workgroups, 427).
    const unsigned waves = gridDim.x * NWV;
    const bool team = (ORDER == 7 ? 1 : 2) * entries <= gridDim.x;
    // A lone member's entries go round by round, there and back: who has the longest of one
    // round has the shortest of the next.  Several members': each wave (or workgroup) takes
    // neighbouring entries, mostly of one member, whose values take 2 us to load (a served
    // run: 4.65e9 cell-updates/s round by round, 5.1e9 so); as many of two passes as any
    // other to within one, entries of one pass first in their stead where there is one
    // fewer, then as many as any other.
    const unsigned sharers = team ? gridDim.x : waves, mine = team ? blockIdx.x : blockIdx.x * NWV + wv;
    unsigned at, jump;         // the entry; a lone member's: the way to the next
    unsigned to = 0, end = 0;  // several members': at `jump` go on to `to`, where those of one pass begin, up to `end`
    if (P.lone_ctrl) {
        at = mine;
        jump = 2 * sharers - 1 - 2 * mine;
    } else {
        const unsigned n_two = (unsigned)__builtin_amdgcn_readlane((int)upto, FIX_RANGES - 1), n_one = entries - n_two;
        const unsigned each = n_two / sharers, more = n_two - each * sharers, fewer = sharers - more;
        const bool few = n_one <= 2 * fewer;  // one-pass entries: all in the stead of others
        const unsigned d = few ? fewer : sharers, rest = few ? n_one : n_one - 2 * fewer, k = few ? mine - more : sharers - 1 - mine;
        const unsigned each1 = rest / d, more1 = rest - each1 * d;
        const unsigned twos = each + (mine < more ? 1u : 0u);
        const unsigned ones = few && mine < more ? 0u : each1 + (k < more1 ? 1u : 0u) + (few || mine < more ? 0u : 2u);
        jump = mine * each + min(mine, more) + twos;
        to = ones ? n_two + k * each1 + min(k, more1) + (few ? 0u : 2 * min(k, fewer)) : entries;
        end = to + ones;
        at = twos ? jump - twos : to;
    }
    auto advance = [&]() {
        if (P.lone_ctrl) {
            at += jump;
            jump = 2 * sharers - jump;
        } else {
            ++at;
            at = at == jump ? to : (at == end ? entries : at);
        }
    };
    FixScratch<NW> &S = scratch[team ? 0 : wv];
    const int start = team ? 64 * wv : 0, step = team ? BLOCK : 64;
    auto sync = [&]() {
        if (team) __syncthreads();
        else wave_sync();
    };
    auto load_entry = [&](unsigned i) {
        if (i >= entries) return 0ull;
        const int c = __popcll(__builtin_amdgcn_ballot_w64(upto <= i));
        const unsigned e = (unsigned)__builtin_amdgcn_readlane((int)skew, c) + (c < FIX_RANGES ? i : 0u - i);
        return lane < 4 ? gmem(P.fix_list)[4ull * e + lane] : 0ull;
    };
    const bool full = REC && (P.flags & KF_FULL_SELECTION) != 0;
    unsigned long long bad = 0, next = load_entry(at);
    WaveMost &M = scratch[wv].most;
    if (STEP && lane < 28) M[lane >> 2][lane & 3] = 0ull;
    const int ld = min(max(lane - H, 0), 57);  // (lanes outside repeat the first and last)
    // the maxima of the waves w0 .. w1 - 1 into the member's
    auto flush = [&](int w0, int w1) {
        wave_sync();
        unsigned long long most = 0ull;
        if (lane < 7) {
            for (int w = w0; w < w1; ++w) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    most = max(most, scratch[w].most[lane][i]);
                    scratch[w].most[lane][i] = 0ull;
                }
            }
        }
        wave_sync();
        if (lane < 7 && most > as_bits(scratch[wv].member[12 + lane]))
            __hip_atomic_fetch_max(&v.amax[P.r_out * amax_slot_words(EULER2D) + blockIdx.x % amax_copies(EULER2D) * AMAX_VALS + lane],
                                   most, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    auto flag = [&]() {
        if (bad && lane == 0) __hip_atomic_fetch_or(&v.ctrl->status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        bad = 0;
    };
    while (at < entries) {
        {
            const unsigned long long where = lane_bits(next, 0);
            unsigned long long fx = lane_bits(next, 1), fb = lane_bits(next, 2), ft = lane_bits(next, 3);
            unsigned long long tx = 0, tb = 0, tt = 0;  // faces with a top flux (full)
            advance();
            next = load_entry(at);  // on its way while this one is worked on
            const long long unit = (long long)(where >> 28);
            const unsigned most = (unsigned)where & 63u, piece = (unsigned)(where >> 6) & 7u;
            unsigned long long own = ((1ull << CELLS) - 1) << G;  // lanes of its cells
            if (full) {
                own &= ((1ull << FIX_SPLIT) - 1) << (G + FIX_SPLIT * piece);
                tx = half_turn(fx) & (own | own >> 1);
                tb = half_turn(fb) & own;
                tt = half_turn(ft) & own;
            } else if (most) {
                const unsigned before = mask_place(fx) + mask_place(fb) + mask_place(ft);
                own &= __builtin_amdgcn_ballot_w64(before >= piece * most && ((where & FIX_LAST) || before < (piece + 1) * most));
            }
            fx &= own | own >> 1;
            fb &= own;
            ft &= own;
            if (!(fx | fb | ft)) continue;
            if (unit < v.u0 || unit >= v.u1) {
                if (STEP && v.u1 >= 0 && (!team || wv == 0)) {
                    flush(wv, wv + 1);
                    flag();
                }
                enter(unit);
            }
            const int nx = v.nx, ny = v.ny;
            const long long plane = (long long)v.pitch * ny;
            const UnitBox box = unit_box(v, unit, CELLS);
            const int x0 = box.x0, j = box.y0 + (int)((where >> 12) & 0xffff);
            // the faces: x, below, above
            int nf = 0;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const unsigned long long m = k == 0 ? fx : (k == 1 ? fb : ft);
                if (!team || wv == k) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) S.dF[k][c][ld] = 0.0;
                    if ((m >> lane) & 1)
                        S.face[nf + mask_place(m)] = (unsigned char)(k << 6 | lane);
                }
                nf += __popcll(m);
            }
            // the cells, their top values on the way while the faces are selected
            const unsigned long long fixed = fx | (fx << 1) | fb | ft;
            const int xn = x0 - G + lane;
            const bool cell = (!team || wv == 0) && ((fixed & own) >> lane & 1) && xn < nx;
            GMEM double *out = v.out + (long long)j * v.pitch + xn;
            double Uc[4] = {0.0, 0.0, 0.0, 0.0};
            if (cell) {
#pragma unroll
                for (int c = 0; c < 4; ++c) Uc[c] = out[c * plane];
            }
            sync();
            // a window of the entry may cross the boundary
            const int lo = (int)__builtin_ctzll(own), hi = 63 - (int)__builtin_clzll(own);
            const bool edge = x0 - G + lo - G < 0 || x0 - G + hi + G >= nx || j - G < 0 || j + G >= ny;
            const bool small = nx < NW || ny < NW;
            const double *mem = scratch[wv].member;
#pragma unroll 1
            for (int k0 = start; k0 < 4 * nf; k0 += step) {
                const bool valid = k0 + lane < 4 * nf;
                const int k = min(k0 + lane, 4 * nf - 1), s = k & 3;
                const unsigned f = S.face[k >> 2], set = f >> 6;
                const bool acoustic = CH && (s == 0 || s == 3);
                const bool ax = f < 64u;  // an x-face
                const int col = x0 - G + (int)(f & 63u);
                const int pos = (ax ? col : (f < 128u ? j - 1 : j)) - H;  // window node t is pos + t on the face's line
                const double a = mem[(ax ? 0 : 4) + s];
                // The four lanes of a face share its window: each loads a quarter of the nodes
                // and projects them on all fields, and takes its field of the others' from LDS
                // (every lane loading the whole window took twice as long, half of it in the
                // loads).
                constexpr int NPL = (NW + 3) / 4;
                double Q[NPL][4];
#pragma unroll
                for (int i = 0; i < NPL; ++i) {
                    int n = pos + min(s * NPL + i, NW - 1);
                    if (edge) n = line_node(n, ax ? nx : ny, (ax ? v.bcx : v.bcy) == BC_PERIODIC, small);
                    const Off o = 8 * ((Off)(ax ? j : n) * v.pitch + (ax ? n : col));
#pragma unroll
                    for (int c = 0; c < 4; ++c) Q[i][c] = row_load(v.in + c * plane, o);
                }
                double U[NPL][4], F[NPL][4], hh[NPL];
#pragma unroll
                for (int i = 0; i < NPL; ++i) {
                    const double rho = Q[i][0], m = ax ? Q[i][1] : Q[i][2], n = ax ? Q[i][2] : Q[i][1], E = Q[i][3];
                    const double ir = rcp_nr(rho), u = m * ir, w = n * ir;
                    const double p = node_pressure(rho, u, w, E, P.gm1);
                    U[i][0] = rho;
                    U[i][1] = m;
                    U[i][2] = n;
                    U[i][3] = E;
                    F[i][0] = m;
                    F[i][1] = fma(m, u, p);
                    F[i][2] = m * w;
                    F[i][3] = (E + p) * u;
                    hh[i] = (E + p) * ir;
                    Q[i][1] = u;
                    Q[i][2] = w;
                }
                RoeState ro{};
                if constexpr (CH) {
                    // nodes H and H + 1 from the lanes that hold them
                    constexpr int iL = H % NPL, iR = (H + 1) % NPL;
                    constexpr int fromL = 0x55 * (H / NPL), fromR = 0x55 * ((H + 1) / NPL);  // quad_perm broadcasts
                    double sL, sR;
                    if constexpr (fromL != fromR) {  // (one root in every lane, of the node it has)
                        const double root = sqrt_nr(s <= H / NPL ? Q[iL][0] : Q[iR][0]);
                        sL = quad_move<fromL>(root);
                        sR = quad_move<fromR>(root);
                    } else {
                        sL = sqrt_nr(quad_move<fromL>(Q[iL][0]));
                        sR = sqrt_nr(quad_move<fromR>(Q[iR][0]));
                    }
                    ro = roe_state(sL, quad_move<fromL>(Q[iL][1]), quad_move<fromL>(Q[iL][2]), quad_move<fromL>(hh[iL]), sR,
                                   quad_move<fromR>(Q[iR][1]), quad_move<fromR>(Q[iR][2]), quad_move<fromR>(hh[iR]), P.gm1);
                }
                // windows g+ and g- = P F +- a P U; a lane's columns are rotated by its place in
                // the quad, so the four writes of an instruction fall in different banks
                double pu[NW], gp[2 * H + 1], gm[2 * H + 1];
                double(&X)[NW][64] = scratch[wv].exchange;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
#pragma unroll
                    for (int i = 0; i < NPL; ++i) {
                        double w[4];
                        to_fields<4, CH>(ro, h == 0 ? U[i] : F[i], w);
                        const int t = s * NPL + i;
                        if (4 * NPL == NW || t < NW) {
#pragma unroll
                            for (int c = 0; c < 4; ++c) X[t][(lane & 60) + ((c + s) & 3)] = w[c];
                        }
                    }
                    wave_sync();
#pragma unroll
                    for (int t = 0; t < NW; ++t) {
                        const double x = X[t][(lane & 60) + ((s + t / NPL) & 3)];
                        if (h == 0) {
                            pu[t] = x;
                        } else {
                            if (t <= 2 * H) gp[t] = fma(a, pu[t], x);
                            if (t >= 1) gm[2 * H + 1 - t] = fma(-a, pu[t], x);
                        }
                    }
                    wave_sync();
                }
                const double sd = (acoustic ? 4.0 : 2.0) * P.delta;
                int sp, sm;
                double tp, tm;
                const double hp = R::select_step(gp, sd, sp, tp);
                __builtin_amdgcn_sched_barrier(0);
                const double hm = R::select_step(gm, sd, sm, tm);
                if (REC && v.sel && valid) {
                    const long long xb = (long long)ny * (nx + 1), yb = (long long)(ny + 1) * nx;
                    const long long o = ax ? 2 * s * xb + (long long)j * (nx + 1) + col + 1
                                            : 8 * xb + 2 * s * yb + (long long)(set == 1u ? j : j + 1) * nx + col;
                    v.sel[o] = (uint8_t)sp;
                    v.sel[o + (ax ? xb : yb)] = (uint8_t)sm;
                }
                // R times the four lanes' fields; lane s stores component s
                double es = fma(a, pu[H] - pu[H + 1], hp + hm);
                if (full && (((set == 0u ? tx : (set == 1u ? tb : tt)) >> (f & 63u)) & 1)) es = (hp - tp) + (hm - tm);  // (zero)
                es *= acoustic ? 0.25 : 0.5;
                double d = es;
                if constexpr (CH) {
                    const double e[4] = {quad_move<0x00>(es), quad_move<0x55>(es), quad_move<0xaa>(es), quad_move<0xff>(es)};
                    double r[4];
                    back_project<4>(ro, e, r);
                    d = s == 0 ? r[0] : (s == 1 ? r[1] : (s == 2 ? r[2] : r[3]));
                }
                if (valid) S.dF[set][s][(f & 63u) - H] = d;
            }
            sync();
            bool b = false;
            Maxima<EULER2D> m;
            m.reset();
            if (cell) {
                const int perm[4] = {0, 2, 1, 3};
                const double idx = mem[8], idy = mem[9], c = mem[10];
                double U[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const double lx = -(S.dF[0][q][ld] - S.dF[0][q][ld - 1]) * idx;
                    const double dL = lx - (S.dF[2][perm[q]][ld] - S.dF[1][perm[q]][ld]) * idy;
                    U[q] = STEP ? fma(c, dL, Uc[q]) : Uc[q] + dL;
                    out[q * plane] = U[q];
                }
                if (STEP) m.add(U, P.gamma, idx, idy);
                b = m.bad != 0;
            }
            if (STEP && (!team || wv == 0)) {
                bad |= __builtin_amdgcn_ballot_w64(b);
#pragma unroll
                for (int i = 0; i < 7; ++i) {
                    // a quad's maximum (a whole wave's over DPP would take twice as long)
                    double x = fmax(m.v[i], quad_move<0xb1>(m.v[i]));
                    x = fmax(x, quad_move<0x4e>(x));
                    if ((lane & 3) == 0)
                        __hip_atomic_fetch_max(&M[i][(lane >> 2) & 3], as_bits(x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
                }
            }
            sync();
        }
    }
    if constexpr (STEP) {
        // (together where the waves end in one member, as in stage_2d)
        __shared__ int ended[NWV];
        if (lane == 0) ended[wv] = v.u1 >= 0 ? v.k : -1;
        flag();
        __syncthreads();
        int first = NWV;
        bool same = true;
#pragma unroll
        for (int w = NWV - 1; w >= 0; --w) {
            same = same && (ended[w] == v.k || ended[w] < 0);
            first = ended[w] >= 0 ? w : first;
        }
        if (v.u1 >= 0 && (same ? wv == first : true)) flush(same ? 0 : wv, same ? NWV : wv + 1);
    }
}

// ---------------------------------------------------------------------------
using KFn = void (*)(KParams);

template <bool FIX, int ORDER, bool REC, bool CH> static KFn pick_step(int mode)
{
    if (mode == M_RHS) return FIX ? fix_2d<ORDER, false, REC, CH> : stage_2d<ORDER, false, REC, CH>;
    return FIX ? fix_2d<ORDER, true, REC, CH> : stage_2d<ORDER, true, REC, CH>;
}
template <bool FIX, bool CH> static KFn pick_order(int order, int mode, bool rec)
{
    if (order == 7) return rec ? pick_step<FIX, 7, true, CH>(mode) : pick_step<FIX, 7, false, CH>(mode);
    return rec ? pick_step<FIX, 5, true, CH>(mode) : pick_step<FIX, 5, false, CH>(mode);
}
template <bool FIX> static KFn pick(int order, int mode, bool rec, bool ch)
{
    return ch ? pick_order<FIX, true>(order, mode, rec) : pick_order<FIX, false>(order, mode, rec);
}

hipError_t launch_stage_2d(int order, int mode, bool rec, bool ch, const KParams &p, int grid, int fix_grid, hipStream_t s)
{
    KParams copy = p;
    copy.mode = mode;
    void *args[] = {&copy};
    const hipError_t e = hipLaunchKernel((const void *)pick<false>(order, mode, rec, ch), dim3(grid > 0 ? grid : 1),
                                         dim3(BLOCK), args, 0, s);
    if (e != hipSuccess) return e;
    return hipLaunchKernel((const void *)pick<true>(order, mode, rec, ch), dim3(fix_grid > 0 ? fix_grid : 1), dim3(BLOCK),
                           args, 0, s);
}

static int occupancy(KFn fn)
{
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, (const void *)fn, BLOCK, 0) != hipSuccess || n < 1) n = 1;
    return n;
}

int occupancy_2d(int order, int mode, bool rec, bool ch) { return occupancy(pick<false>(order, mode, rec, ch)); }
int occupancy_fix_2d(int order, int mode, bool rec, bool ch) { return occupancy(pick<true>(order, mode, rec, ch)); }

}  // namespace enoao
