// enoao_kernels.hip -- gfx950 kernels of the ENO-AO path.
//
// Per Runge-Kutta stage of a 1D problem (Section 2: conservative finite
// differences, global Lax-Friedrichs splitting, third-order TVD Runge-Kutta;
// Section 3: ENO-AO reconstruction; Section 4: Roe characteristic decomposition):
//   sweep_x<STAGE s>   tile load + BC -> per-node flux and Roe inputs in LDS ->
//        one lane per face: the flux of the top candidates and the bound that tells
//        where they are taken; one lane per field of a face: the selections of the
//        others -> flux difference -> RK stage combine -> per-field maxima of the new
//        state for the next stage.
// (2D stages: enoao_grid.hip.)  Kernels are persistent: a grid of (CUs x
// occupancy) workgroups walks a contiguous chunk of the flattened tile list of
// all instances of a batch.  The time-loop control and the
// maxima of an input state, in 1D and 2D, are here too.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "enoao_common.hpp"
#include "enoao_device.hpp"
#include "enoao_kernels.hpp"
#include "enoao_wave.hpp"

namespace enoao {

// ---------------------------------------------------------------------------
// One face: window node t (t = 0 .. 2G-1) of face j+1/2 is node j-H+t; the
// plus side reads nodes j-H .. j+H, the minus side the mirror j+1+H .. j+1-H.

// Numerical flux of one advection face from its 2G window nodes (w0: node 0) and its
// staged differences D_0, D_1, D_2 (DSTAGED; otherwise formed here).  f^(+/-) =
// (a u +/- alpha u)/2 is reconstructed as 2 f^(+/-); the differences and the symmetric
// stencil of f = a u are a times those of u.  shortcut = false: the full selection
// everywhere (the result is the same).
template <int ORDER, bool DSTAGED>
__device__ __forceinline__ double advection_flux(const double *w0, const double *d0, double a, double adv, double delta,
                                                 bool shortcut, int (&sel)[2])
{
    using T = TopStencil<ORDER>;
    constexpr int H = ReconTraits<ORDER>::H, G = H + 1, W = 2 * H + 1, K = ReconTraits<ORDER>::K;
    double du[3];
#pragma unroll
    for (int p = 0; p < 3; ++p) du[p] = DSTAGED ? d0[p] : T::diff(w0 + p, 1);
    const double isp = fmin(fabs(fma(a, du[0], adv * du[0])), fabs(fma(a, du[1], adv * du[1])));
    const double ism = fmin(fabs(fma(-a, du[2], adv * du[2])), fabs(fma(-a, du[1], adv * du[1])));
    const double hs = fma(a * T::kappa, du[1], adv * T::sym(w0, 1));
    if (wave_all(isp <= 2.0 * delta && ism <= 2.0 * delta) & shortcut) {
        sel[0] = sel[1] = K - 1;
        return 0.5 * hs;
    }
    double gp[W], gm[W];
#pragma unroll
    for (int t = 0; t < 2 * G; ++t) {
        const double u = w0[t];
        const double au = adv * u;
        if (t < W) gp[t] = fma(a, u, au);
        if (t >= 1) gm[2 * H + 1 - t] = fma(-a, u, au);
    }
    int sp, sm;
    const double hp = Recon<ORDER>::select(gp, 2.0 * delta, isp, sp);
    const double hm = Recon<ORDER>::select(gm, 2.0 * delta, ism, sm);
    sel[0] = sp;
    sel[1] = sm;
    return 0.5 * (sp == K - 1 && sm == K - 1 ? hs : hp + hm);
}

// Roe state of the face whose left node's staged quantities are at nl (quantity stride qs)
__device__ __forceinline__ RoeState line_roe(const double *nl, int qs, double gm1)
{
    return roe_state(nl[5 * qs], nl[6 * qs], 0.0, nl[7 * qs], nl[5 * qs + 1], nl[6 * qs + 1], 0.0, nl[7 * qs + 1], gm1);
}

// A wave's segment of an Euler line: its staged node quantities and its face fluxes.
struct LineLds {
    const double *q;      // staged quantities, stride qs; lane l's face has nodes l .. l + 2H + 1
    int qs;
    double *fh;           // fluxes by component (stride fs) and face
    int fs;
    unsigned char *list;  // faces that need a selection (LINE_CHOSEN: its flux is the selected one)
};
constexpr unsigned LINE_FACE = 0x3f, LINE_CHOSEN = 0x80;

// The segment's 64 Euler fluxes where every field takes its top candidate on both sides:
// the flux is linear in the window (TopStencil; R L = I, so the central part needs no
// projection), Fhat = S F / 2 + R (kappa alpha L D_1 U) / 2.  One bound tells nearly all
// such faces: |l.(D F +- alpha D U)| <= |l|_1 max_c(|D F_c| + alpha |D U_c|) with D_1,
// which both sides share.  Returns the `live` faces that the bound leaves, listed; they
// are few or, on a coarse line, most of them, and each costs five others.
// rec(face, i, candidate): a face's selection i (2 field + side); nothing depends on it.
template <int ORDER, bool CH, class Rec>
__device__ __forceinline__ unsigned long long line_top(const LineLds &l, const double (&al)[3], double gm1,
                                                       double delta, bool shortcut, bool live, double (&Fh)[3],
                                                       const Rec &rec)
{
    using T = TopStencil<ORDER>;
    constexpr int H = ReconTraits<ORDER>::H, NW = 2 * H + 2, K = ReconTraits<ORDER>::K;
    const int lane = threadIdx.x & 63;
    const double *w = l.q + lane;
    double sF[3], dU[3], dF[2];
    // (two quantities' windows in flight)
#pragma unroll
    for (int m = 0; m < 5; ++m) {
        double win[NW - 2];
#pragma unroll
        for (int t = 0; t < NW - 2; ++t) win[t] = w[m * l.qs + 1 + t];
        if (m == 1) sF[0] = T::sym1(win, 1);  // F_0 is U_1
        if (m >= 3) sF[m - 2] = T::sym1(win, 1);
        if (m < 3) dU[m] = T::diff(win, 1);
        else dF[m - 3] = T::diff(win, 1);
        if (m % 2 == 1) __builtin_amdgcn_sched_barrier(0);
    }
    RoeState r{};
    if constexpr (CH) r = line_roe(w + H, l.qs, gm1);
    double x[3];
    to_fields<3, CH>(r, dU, x);
#pragma unroll
    for (int s = 0; s < 3; ++s) x[s] *= al[s] * (0.5 * T::kappa / fscale<3, CH>(s));
    from_fields<3, CH>(r, x, Fh);
#pragma unroll
    for (int c = 0; c < 3; ++c) Fh[c] = fma(0.5, sF[c], Fh[c]);
    // (acoustic rows halved to the window scale of the entropy field)
    double bound = 1.0;
    if constexpr (CH) {
        const double au = 1.0 + fabs(r.u), y = fma(r.b1, au, r.b2);
        bound = fmax(1.0 + y, 0.5 * fma(r.ic, au, y));
    }
    const double a = fmax(al[0], fmax(al[1], al[2]));
    double node = fma(a, fabs(dU[0]), fabs(dU[1]));
#pragma unroll
    for (int k = 0; k < 2; ++k) node = fmax(node, fma(a, fabs(dU[k + 1]), fabs(dF[k])));
    node = fma(0.0, dF[0], node);  // (dF[0] holds the pressure: a NaN of any component, which fmax drops)
    // (the bound and the indicators differ by rounding; delta = 0 leaves every face)
    const double thr = delta > 0.0 && shortcut ? 2.0 * delta * (1.0 - 1.0 / 1024.0) : -1.0;
    const bool ok = bound * node <= thr;
    const unsigned long long fail = __builtin_amdgcn_ballot_w64(!ok && live);
    if (live && ok) {
#pragma unroll
        for (int i = 0; i < 6; ++i) rec(lane, i, K - 1);
    }
    if ((fail >> lane) & 1) l.list[mask_place(fail)] = (unsigned char)lane;
    return fail;
}

// alpha of the three fields (by value: a lane picks one of them)
struct Alpha3 {
    double a0, a1, a2;
};

// The selection of field s on the face at place `at` of the list of segment l, both sides.
// The field of the chosen flux less (F_j + F_j+1) / 2 goes to the face's place in l.fh,
// formed from the chosen candidates' own differences: the top candidate, rejected where
// its window crosses a jump, is as large as the jump's far side, and a flux formed as a
// distance from it kept that side's rounding (4e-9 of the largest L at a pressure ratio
// of 1e8).  A face with a field that does not take the top candidate is marked in the
// list.  A lane takes one field of one listed face: where each lane took all
// fields of its own face, a segment with a shock held its wave for 9500 cycles a stage
// beside 1200 for the others.  All lanes of the wave call it; `valid` ones count.
// SERIAL: one side's candidates after the other's (fewer registers, more latency).
template <int ORDER, bool CH, bool SERIAL, class Rec>
__device__ __forceinline__ void line_select(const LineLds &l, int at, int s, bool valid, Alpha3 al,
                                            double gm1, double delta, const Rec &rec)
{
    using R = Recon<ORDER>;
    constexpr int H = R::H, NW = 2 * H + 2, K = R::K;
    const int f = (int)(l.list[at] & LINE_FACE);
    const double *w = l.q + f;
    const bool ent = s == 1;
    const double a = !CH || s == 0 ? al.a0 : (s == 1 ? al.a1 : al.a2);
    double l0 = 0.0, l1 = 0.0, l2 = 0.0;  // the field's row (acoustic rows doubled)
    if constexpr (CH) {
        const RoeState r = line_roe(w + H, l.qs, gm1);
        const double sg = s == 0 ? r.ic : -r.ic, bu = r.b1 * r.u;
        l0 = ent ? 1.0 - r.b2 : fma(sg, r.u, r.b2);
        l1 = ent ? bu : -sg - bu;
        l2 = ent ? -r.b1 : r.b1;
    }
    double gp[2 * H + 1], gm[2 * H + 1], du = 0.0;  // du: U_j - U_j+1 on the field
#pragma unroll
    for (int t = 0; t < NW; ++t) {
        const double u0 = w[t], u1 = w[l.qs + t], u2 = w[2 * l.qs + t], f1 = w[3 * l.qs + t], f2 = w[4 * l.qs + t];
        double pu, pf;
        if constexpr (CH) {
            pu = fma(l0, u0, fma(l1, u1, l2 * u2));
            pf = fma(l0, u1, fma(l1, f1, l2 * f2));
        } else {
            pu = s == 0 ? u0 : (s == 1 ? u1 : u2);
            pf = s == 0 ? u1 : (s == 1 ? f1 : f2);
        }
        if (t == H) du = pu;
        if (t == H + 1) du -= pu;
        if (t <= 2 * H) gp[t] = fma(a, pu, pf);
        if (t >= 1) gm[2 * H + 1 - t] = fma(-a, pu, pf);
        if (t % 2 == 1) __builtin_amdgcn_sched_barrier(0);  // (two nodes' reads in flight)
    }
    const double sd = (CH && !ent ? 4.0 : 2.0) * delta;
    int cp, cm;
    const double hp = R::select_step(gp, sd, cp);
    if (SERIAL) __builtin_amdgcn_sched_barrier(0);
    const double hm = R::select_step(gm, sd, cm);
    if (valid) {
        rec(f, 2 * s, cp);
        rec(f, 2 * s + 1, cm);
        l.fh[s * l.fs + f] = fma(a, du, hp + hm) * (CH && !ent ? 0.25 : 0.5);
        if (cp != K - 1 || cm != K - 1) l.list[at] = (unsigned char)(f | LINE_CHOSEN);
    }
}

// The fluxes of the listed faces (`fail`), each by its own lane: (F_j + F_j+1) / 2 and R
// times what the selections left.  A face where every field takes the top candidate after
// all keeps line_top's flux, so no result depends on what the bound leaves.
template <int ORDER, bool CH>
__device__ __forceinline__ void line_correct(const LineLds &l, unsigned long long fail, double gm1, double (&Fh)[3])
{
    constexpr int H = ReconTraits<ORDER>::H;
    const int lane = threadIdx.x & 63;
    if (!((fail >> lane) & 1) || !(l.list[mask_place(fail)] & LINE_CHOSEN)) return;
    const double *w = l.q + lane + H;
    double e[3], d[3];
#pragma unroll
    for (int s = 0; s < 3; ++s) e[s] = l.fh[s * l.fs + lane];
    RoeState r{};
    if constexpr (CH) r = line_roe(w, l.qs, gm1);
    from_fields<3, CH>(r, e, d);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const double *F = w + (c + (c ? 2 : 1)) * l.qs;  // F_0 is U_1
        Fh[c] = fma(0.5, F[0] + F[1], d[c]);
    }
}

// The selections of a wave's own listed faces (`fail`), and their fluxes.
template <int ORDER, bool CH, bool SERIAL, class Rec>
__device__ __forceinline__ void line_selections(const LineLds &l, unsigned long long fail, Alpha3 al,
                                                double gm1, double delta, double (&Fh)[3], const Rec &rec)
{
    if (__builtin_expect(fail == 0, 1)) return;
    const int lane = threadIdx.x & 63, nf = __popcll(fail);
    wave_sync();
#pragma unroll 1
    for (int at = 0; at < 3 * nf; at += 64) {
        const int k = min(at + lane, 3 * nf - 1), s = (k >= nf) + (k >= 2 * nf);
        line_select<ORDER, CH, SERIAL>(l, k - s * nf, s, at + lane < 3 * nf, al, gm1, delta, rec);
    }
    wave_sync();
    line_correct<ORDER, CH>(l, fail, gm1, Fh);
}

// Staged top differences D_0 of two consecutive advection nodes i and i+1, from nodes
// i .. i+2H, which the two share (one lane reads 2H+1 nodes for both instead of 2H for
// each).  x: node i; out: its difference.
template <int ORDER> __device__ __forceinline__ void stage_diff2(const double *x, double *out)
{
    constexpr int H = ReconTraits<ORDER>::H;
    double w[2 * H + 1];
#pragma unroll
    for (int t = 0; t < 2 * H + 1; ++t) w[t] = x[t];
    out[0] = TopStencil<ORDER>::diff(w, 1);
    out[1] = TopStencil<ORDER>::diff(w + 1, 1);
}

// Per-instance values of one sweep launch.  A workgroup walks a contiguous
// chunk of the tile list, so it reloads them only when the walk crosses into
// another instance; within an instance no tile reads a descriptor.
template <int EQ, int MODE> struct View {
    static constexpr int NC = NodeTraits<EQ>::NC;
    long long t0, t1;      // the instance's tiles in the batch list
    int k, nx, ny, pitch, per_row, bc;
    int active;            // the instance is still stepping
    const GMEM double *in;    // stage input
    GMEM double *out;         // stage output
    const GMEM double *base;  // u^n (stages 2 and 3)
    GMEM double *lx;          // rhs: L
    GMEM uint8_t *sel;
    GMEM unsigned long long *amax;
    GMEM Ctrl *ctrl;
    double idx, idy, adv, dt;
    double al[NC];
};

// The view of the instance holding `tile`.  prev: the instance the walk was in
// (-1 at the start of a chunk: binary search); the tile lists are ordered by
// instance, so after the first the walk just moves on to the next instance
// that has tiles left.
template <int EQ, int MODE, bool CH>
__device__ __forceinline__ View<EQ, MODE> load_view(const KParams &P, int n_inst, long long tile, int prev)
{
    constexpr int NC = NodeTraits<EQ>::NC;
    View<EQ, MODE> v;
    int k;
    if (prev < 0) {
        k = find_last(n_inst, tile, [&](int i) { return P.inst[i].xtile0; });
    } else {
        k = prev + 1;
        while (k < n_inst - 1 && tile >= P.inst[k].xtile0 + P.inst[k].xtiles) ++k;
    }
    v.k = uniform(k);
    const Inst &I = P.inst[v.k];
    v.t0 = uniform(I.xtile0);
    v.t1 = v.t0 + uniform(I.xtiles);
    v.nx = uniform(I.nx);
    v.ny = uniform(I.ny);
    v.pitch = uniform(I.pitch);
    v.per_row = uniform(I.segs_per_row);
    v.bc = uniform(I.bcx);
    v.ctrl = gmem(uniform(I.ctrl));
    v.active = uniform(v.ctrl->done) == 0;
    v.dt = uniform(v.ctrl->dt);
    v.in = gmem(uniform(MODE == M_S2 ? I.w1 : (MODE == M_S3 ? I.w2 : I.u)));
    v.out = gmem(uniform(MODE == M_S1 ? I.w1 : (MODE == M_S2 ? I.w2 : I.u)));
    v.base = gmem(uniform(I.u));
    v.lx = gmem(uniform(I.lx));
    v.sel = gmem(uniform(I.sel));
    if (v.sel && P.sel_slot > 0) {
        // records of one evaluation: [NC][2][nx+1]
        const long long rec = (long long)NC * 2 * v.ny * (v.nx + 1);
        v.sel += (long long)P.sel_slot * rec;
    }
    v.amax = gmem(uniform(I.amax));
    v.idx = 1.0 / uniform(I.dx);
    v.idy = 1.0 / uniform(I.dy);
    v.adv = uniform(I.adv);
    if constexpr (EQ == ADVECTION) {
        v.al[0] = fabs(v.adv);
    } else {
        const GMEM unsigned long long *a = v.amax + P.r_in * AMAX_VALS;
        const double m0 = uniform(as_double(a[0])), m1 = uniform(as_double(a[1])), m2 = uniform(as_double(a[2]));
        if constexpr (CH) {
            v.al[0] = m0;
            v.al[1] = m1;
            v.al[2] = m2;
        } else {
            // one alpha for all components: max(|u| + c) = max(max|u - c|, max|u + c|)
            const double a = fmax(m0, m2);
#pragma unroll
            for (int c = 0; c < NC; ++c) v.al[c] = a;
        }
    }
    return v;
}

// ---------------------------------------------------------------------------
// x-sweep.  Each wave: one segment of a grid line (64 faces, 63 cells) per
// tile, the wave's segments of a chunk in one contiguous run (a segment that
// continues the previous one along its line reuses its last 2G staged nodes).
// Tiles are software-pipelined: the global operands of tile t+1 are loaded into
// registers while tile t is reconstructed, so the memory latency hides behind
// the face arithmetic.  Waves per SIMD the register allocation must allow: three at
// order 5 (four spill, and a 2.2e6-node stage takes 40.4 us against 39.4), two at
// order 7 (three spill).  With the linear flux and the listed selections of line_top a
// stage of 2.2e6 nodes takes 42 us where forming the indicators of all fields at every
// face took 55 (order 7: 48 against 59).
#ifndef ENOAO_X_WAVES_PER_EU
#define ENOAO_X_WAVES_PER_EU 3
#endif
#ifndef ENOAO_X7_WAVES_PER_EU
#define ENOAO_X7_WAVES_PER_EU 2  // order 7 (spills at three)
#endif
// a wave's segment within its instance: grid line and segment index along it
struct XCur {
    int row, segx;
};

// the segment of wave wseg in tile `tile` when the waves take consecutive
// segments (the maxima kernel's order)
__device__ __forceinline__ XCur x_cursor(long long tile, long long t0, int per_row, int wseg)
{
    // (segment counts of an instance fit 32 bits: ny * ceil(nx / 63))
    const unsigned seg = (unsigned)(tile - t0) * XW_SEGS + (unsigned)wseg;
    const unsigned row = seg / (unsigned)per_row;
    return XCur{(int)row, (int)(seg - row * (unsigned)per_row)};
}

// segment number seg of an instance (grid lines of per_row segments each)
__device__ __forceinline__ XCur x_segment(unsigned seg, int per_row)
{
    const unsigned row = seg / (unsigned)per_row;
    return XCur{(int)row, (int)(seg - row * (unsigned)per_row)};
}

// the next segment of an instance; it continues c along the same grid line
// unless it starts a new one (segx == 0)
__device__ __forceinline__ XCur x_next(XCur c, int per_row)
{
    if (++c.segx == per_row) {
        c.segx = 0;
        ++c.row;
    }
    return c;
}

// Where the b-th of ng chunks of a batch's tiles starts.  A chunk pays for each member it
// meets, before any tile (its values, the first loads, its maxima), as much as for
// MEMBER_TILES tiles, so the list is cut evenly with that much added to every member.
// (512 lines of 128 to 16384 nodes, a stage: 53 us uncharged, 41.3 at 2, 40.9 at 4, 46 at 8.)
// With a workgroup for each tile there is nothing to even out, and the charge left workgroups
// without a tile beside others with two (64 lines of 128 to 2500 nodes, ten steps: 521 us
// charged, 382 not; from there to twice as many tiles it goes either way).
constexpr int MEMBER_TILES = 4;
__device__ __forceinline__ long long chunk_start(const Inst *inst, int n_inst, long long tiles, long long b, long long ng)
{
    if (n_inst == 1 || b == ng || tiles <= ng) return b * tiles / ng;
    const long long x = b * (tiles + (long long)MEMBER_TILES * n_inst) / ng;
    const int lo = uniform(find_last(n_inst, x, [&](int k) { return inst[k].xtile0 + (long long)MEMBER_TILES * k; }));
    const long long t = inst[lo].xtile0;
    return t + max(0ll, x - t - (long long)MEMBER_TILES * (lo + 1));
}

// a lane's global operands of one x tile: the nodes it stages (segment
// positions lane and lane + 64; for a segment that continues the wave's
// previous one along its line only the 63 new nodes, positions 2G + lane) and,
// for a 1D stage 2 or 3, u^n at its cell.  Every register is written on every
// path (lanes and rows past the end load a clamped, in-bounds address whose
// value goes unused): a register that kept its old value would be copied while
// its previous load may still be in flight, and the copy's wait would stall on
// the prefetch just issued.
template <int NC> struct XPre {
    double U[2][NC];
    double base[NC];
};

template <int EQ, int MODE, int G>
__device__ __forceinline__ void x_prefetch(const View<EQ, MODE> &v, XCur c, bool cont, int lane,
                                           XPre<NodeTraits<EQ>::NC> &pre)
{
    constexpr int NC = NodeTraits<EQ>::NC, NN = XW_FACES + 2 * G - 1;
    const int nx = v.nx, sx = c.segx * XW_CELLS;
    const int row = min(c.row, v.ny - 1);
    const long long plane = (long long)v.pitch * v.ny;
    const GMEM double *rowp = v.in + (long long)row * v.pitch;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int i = cont ? min(2 * G + lane, NN - 1) : min(lane + 64 * j, NN - 1);
        const int x = bc_map(sx - G + i, nx, v.bc);
#pragma unroll
        for (int q = 0; q < NC; ++q) pre.U[j][q] = rowp[q * plane + x];
    }
    if constexpr (MODE == M_S2 || MODE == M_S3) {
        const int x = min(sx + lane, nx - 1);
        const GMEM double *b = v.base + (long long)row * v.pitch + x;
#pragma unroll
        for (int q = 0; q < NC; ++q) pre.base[q] = b[q * plane];
    }
}

template <int EQ, int ORDER, int MODE, bool REC, bool CH>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(ORDER == 7 ? ENOAO_X7_WAVES_PER_EU
                                                                  : ENOAO_X_WAVES_PER_EU))) void sweep_x(KParams P)
{
    constexpr int NC = NodeTraits<EQ>::NC, NQ = NodeTraits<EQ>::NQ;
    constexpr int H = ReconTraits<ORDER>::H, G = H + 1;
    constexpr int NN = XW_FACES + 2 * G - 1;  // nodes staged per segment
    constexpr int NNP = NN + 1;
    constexpr int NDN = XW_FACES + 2;                  // advection: nodes with a staged difference
    constexpr bool FULL = MODE != M_RHS;  // a stage: combine + maxima here
    __shared__ double lds[NQ * XW_SEGS * NNP];
    __shared__ double dif[EQ == ADVECTION ? XW_SEGS * NDN : 1];
    __shared__ unsigned char list[EQ == ADVECTION ? 1 : XW_SEGS * 64];
    __shared__ double fh[NC * XW_SEGS * XW_FACES];
    __shared__ double red[(BLOCK / 64) * 8];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wseg = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_inst = P.hdr->n_inst;
    const long long T = P.hdr->xtiles_total;
    const long long NG = chunk_groups(P, T);
    if (blockIdx.x >= NG) return;
    const long long t0 = chunk_start(P.inst, n_inst, T, blockIdx.x, NG), t1 = chunk_start(P.inst, n_inst, T, blockIdx.x + 1, NG);
    Maxima<EQ> mx;
    mx.reset();
    XPre<NC> pre;
    double *L = lds + wseg * NNP;
    double *Dl = dif + wseg * NDN;

    // Each wave owns its segment's LDS (nodes and face fluxes), so within the
    // tile loop the waves synchronise only with themselves.  The outer loop
    // runs once per instance met by the workgroup's chunk (uniform over the
    // workgroup, so the maxima flush, a workgroup reduction, is reached by all
    // waves together).
    int prev = -1;
    for (long long tile = t0; tile < t1;) {
        const View<EQ, MODE> v = load_view<EQ, MODE, CH>(P, n_inst, tile, prev);
        prev = v.k;
        const long long tend = v.t1 < t1 ? v.t1 : t1;
        if (!v.active) {
            tile = tend;
            continue;
        }
        if (MODE != M_RHS && P.r_zero >= 0 && tile == v.t0 && tid < AMAX_VALS)
            v.amax[P.r_zero * AMAX_VALS + tid] = 0ull;
        const int nx = v.nx;
        const long long plane = (long long)v.pitch * v.ny;
        // the waves take the instance's segments of this chunk in four contiguous
        // runs, so that a wave's next segment mostly continues its current one
        // along the grid line and shares its last 2G staged nodes
        const int T = (int)(tend - tile);
        XCur c = x_segment((unsigned)(tile - v.t0) * XW_SEGS + (unsigned)(wseg * T), v.per_row);
        bool cont = false;  // c continues the wave's previous segment
        x_prefetch<EQ, MODE, G>(v, c, cont, lane, pre);
        for (int k = 0; k < T; ++k) {
            const bool ok = c.row < v.ny;
            const int sx = c.segx * XW_CELLS;

            // stage this tile's nodes (flux, Roe inputs) into LDS
            if (ok) {
                if (cont) {
                    // the previous segment's nodes 63 .. 63 + 2G - 1 are this one's first
                    for (int t = lane; t < 2 * G * NQ; t += 64) {
                        const int m = t / (2 * G), i = t - m * (2 * G);
                        L[m * XW_SEGS * NNP + i] = L[m * XW_SEGS * NNP + XW_CELLS + i];
                    }
                }
                // nodes 2G + lane of a continuing segment, else lane and 64 + lane
                const int p0 = cont ? 2 * G + lane : lane;
                if (p0 < NN) {
                    double q[NQ];
                    node_quantities<EQ>(pre.U[0], P.gm1, q);
#pragma unroll
                    for (int m = 0; m < NQ; ++m) L[m * XW_SEGS * NNP + p0] = q[m];
                }
                if (!cont && lane + 64 < NN) {
                    double q[NQ];
                    node_quantities<EQ>(pre.U[1], P.gm1, q);
#pragma unroll
                    for (int m = 0; m < NQ; ++m) L[m * XW_SEGS * NNP + 64 + lane] = q[m];
                }
            }
            double base[NC];
#pragma unroll
            for (int q = 0; q < NC; ++q) base[q] = pre.base[q];
            // issue the next tile's loads before this tile's arithmetic
            const XCur cn = x_next(c, v.per_row);
            const bool cont_n = cn.segx != 0;
            if (k + 1 < T) x_prefetch<EQ, MODE, G>(v, cn, cont_n, lane, pre);
            wave_sync();
            if constexpr (EQ == ADVECTION) {
                // top differences of the nodes that start one (faces 0..63 read
                // 0..65), two consecutive nodes per lane
                static_assert(NDN % 2 == 0 && NDN / 2 <= 64, "one pair of nodes per lane");
                if (ok && lane < NDN / 2) stage_diff2<ORDER>(L + 2 * lane, Dl + 2 * lane);
                wave_sync();
            }

            const int f = sx + lane;  // face index along the line
            if (ok) {
                auto rec = [&](int l, int i, int candidate) {
                    if (REC && v.sel)
                        v.sel[(long long)i * v.ny * (nx + 1) + (long long)c.row * (nx + 1) + sx + l] = (uint8_t)candidate;
                };
                const bool shortcut = (P.flags & KF_FULL_SELECTION) == 0;
                double *Fl = fh + wseg * XW_FACES;
                if constexpr (EQ == ADVECTION) {
                    int sel[2];
                    Fl[lane] = advection_flux<ORDER, true>(L + lane, Dl + lane, v.al[0], v.adv, P.delta, shortcut, sel);
                    if (f <= nx) {
                        rec(lane, 0, sel[0]);
                        rec(lane, 1, sel[1]);
                    }
                } else {
                    const LineLds l{L, XW_SEGS * NNP, Fl, XW_SEGS * XW_FACES, list + 64 * wseg};
                    double Fh[3];
                    const unsigned long long fail =
                        line_top<ORDER, CH>(l, v.al, P.gm1, P.delta, shortcut, f <= nx, Fh, rec);
                    line_selections<ORDER, CH, true>(l, fail, Alpha3{v.al[0], v.al[1], v.al[2]}, P.gm1, P.delta, Fh, rec);
#pragma unroll
                    for (int q = 0; q < 3; ++q) Fl[q * XW_SEGS * XW_FACES + lane] = Fh[q];
                }
            }
            wave_sync();

            const int x = sx + lane;
            if (ok && lane < XW_CELLS && x < nx) {
                const long long o = (long long)c.row * v.pitch + x;
                double Lc[NC];
#pragma unroll
                for (int q = 0; q < NC; ++q)
                    Lc[q] = -(fh[(q * XW_SEGS + wseg) * XW_FACES + lane + 1] - fh[(q * XW_SEGS + wseg) * XW_FACES + lane]) * v.idx;
                if constexpr (!FULL) {  // L
#pragma unroll
                    for (int q = 0; q < NC; ++q) v.lx[q * plane + o] = Lc[q];
                } else {
                    double Un[NC];
#pragma unroll
                    for (int q = 0; q < NC; ++q) {
                        const double uin = L[q * XW_SEGS * NNP + lane + G];
                        Un[q] = rk_combine<MODE>(uin, base[q], v.dt, Lc[q]);
                        v.out[q * plane + o] = Un[q];
                    }
                    mx.add(Un, P.gamma, v.idx, v.idy);
                }
            }
            wave_sync();
            c = cn;
            cont = cont_n;
        }
        tile = tend;
        if (FULL) mx.flush(v.amax, v.ctrl, P.r_out, red);
    }
}

// ---------------------------------------------------------------------------
// Maxima of the input state (alpha for the first evaluation, CFL step).
template <int EQ>
__global__ __launch_bounds__(BLOCK) void state_maxima(KParams P)
{
    constexpr int NC = NodeTraits<EQ>::NC;
    __shared__ double red[(BLOCK / 64) * 8];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wseg = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_inst = P.hdr->n_inst;
    const long long T = P.hdr->xtiles_total;
    const long long NG = chunk_groups(P, T);
    if (blockIdx.x >= NG) return;
    const long long t0 = (long long)blockIdx.x * T / NG, t1 = (long long)(blockIdx.x + 1) * T / NG;
    Maxima<EQ> mx;
    mx.reset();
    int cur = -1;
    long long end = -1;
    int nx = 0, ny = 0, pitch = 0, spr = 1;
    long long first = 0;
    const GMEM double *u = nullptr;
    double idx = 0.0, idy = 0.0;
    for (long long tile = t0; tile < t1; ++tile) {
        if (tile >= end) {
            const int k = uniform(find_last(n_inst, tile, [&](int i) { return P.inst[i].xtile0; }));
            if (cur >= 0) mx.flush(gmem(P.inst[cur].amax), gmem(P.inst[cur].ctrl), P.r_out, red);
            cur = k;
            const Inst &I = P.inst[k];
            first = I.xtile0;
            end = first + I.xtiles;
            nx = I.nx;
            ny = I.ny;
            pitch = I.pitch;
            spr = I.segs_per_row;
            u = gmem(I.u);
            idx = 1.0 / I.dx;
            idy = 1.0 / I.dy;
        }
        const long long plane = (long long)pitch * ny;
        const XCur c = x_cursor(tile, first, spr, wseg);
        const int x = c.segx * XW_CELLS + lane;
        if (c.row < ny && lane < XW_CELLS && x < nx) {
            double U[NC];
#pragma unroll
            for (int q = 0; q < NC; ++q) U[q] = u[q * plane + (long long)c.row * pitch + x];
            mx.add(U, P.gamma, idx, idy);
        }
    }
    if (cur >= 0) mx.flush(gmem(P.inst[cur].amax), gmem(P.inst[cur].ctrl), P.r_out, red);
}

// zero all maxima slots (words each) of every instance and the list counters
__global__ void reset_maxima(KParams P, int words)
{
    const int n = P.hdr->n_inst;
    for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < n * words; k += gridDim.x * blockDim.x)
        gmem(P.inst[k / words].amax)[k % words] = 0ull;
    if (P.fix_count && blockIdx.x == 0)
        for (int k = threadIdx.x; k < FIX_SETS * FIX_RANGES; k += blockDim.x)
            gmem(P.fix_count)[k * FIX_COUNTER_STRIDE] = fix_empty(P, k % FIX_RANGES);
}

// What precedes the maxima of a lone member's state, in one launch: the caller's
// pointers into the descriptor, the control block (mode 0: cleared to run an
// evaluation of L; 1: that and a given step size; 2: replaced), maxima slots (words in
// all) and list counters zeroed.  Kernel arguments are captured at launch, so the
// host values need not outlive the call.
__global__ void begin_lone(KParams P, Inst *inst, const double *u, double *lx, Ctrl *c, Ctrl v, int mode, int words)
{
    const int t = threadIdx.x;
    if (t == 0) {
        inst->u = const_cast<double *>(u);
        if (lx) inst->lx = lx;
        if (mode == 2) {
            *c = v;
        } else {
            c->done = 0;
            if (mode == 1) c->dt = v.dt;
        }
    }
    for (int k = t; k < words; k += blockDim.x) gmem(P.lone_amax)[k] = 0ull;
    if (P.fix_count)
        for (int k = t; k < FIX_SETS * FIX_RANGES; k += blockDim.x)
            gmem(P.fix_count)[k * FIX_COUNTER_STRIDE] = fix_empty(P, k % FIX_RANGES);
}

// Time-step control of one instance: CFL (or fixed) step from the maxima m of
// the state at the start of the step (m[0], m[2]: max |u-c|, |u+c|; m[6]: the
// 2D sum), clipped to land on t_final.  Returns whether a step is taken.
template <int EQ>
__device__ __forceinline__ bool control_update(Ctrl &C, double m0, double m2, double m6, double dx, double adv)
{
    if (C.done) return false;
    if (C.status != 0 || C.steps >= C.max_steps) { C.done = 1; return false; }
    const double rem = C.t_final - C.t;
    if (!(rem > 0.0)) { C.done = 1; return false; }
    double dt;
    if (C.dt_fixed > 0.0) {
        dt = C.dt_fixed;
    } else {
        if constexpr (EQ == ADVECTION) {
            dt = C.cfl * dx / fabs(adv);
        } else if constexpr (EQ == EULER1D) {
            const double smax = fmax(m0, m2);  // max(|u|+c)
            if (!(smax > 0.0)) { C.status |= 1; C.done = 1; return false; }
            dt = C.cfl * dx / smax;
        } else {
            const double smax = m6;
            if (!(smax > 0.0)) { C.status |= 1; C.done = 1; return false; }
            dt = C.cfl / smax;
        }
    }
    const bool last = dt >= rem * (1.0 - 1e-10);
    if (last) dt = rem;
    C.dt = dt;
    C.t = last ? C.t_final : C.t + dt;
    C.steps = C.steps + 1;
    return true;
}

// one thread per instance; slot 0 of the maxima holds the state u^n
template <int EQ>
__global__ void step_control(KParams P)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= P.hdr->n_inst) return;
    const Inst &I = P.inst[k];
    const unsigned long long *a = I.amax;
    unsigned long long m6 = a[6];
#pragma unroll
    for (int i = 1; i < amax_copies(EQ); ++i) m6 = max(m6, a[i * AMAX_VALS + 6]);
    control_update<EQ>(*I.ctrl, as_double(a[0]), as_double(a[2]), as_double(m6), I.dx, I.adv);
}

// ---------------------------------------------------------------------------
// LDS-resident solver of small 1D members.  One workgroup per member runs
// `nsteps` controlled steps with u^n and both stage states in LDS: HBM is
// touched only to load the state and store it back.  Within a stage each wave
// owns 64-face line segments (63 cells each, taken round-robin) and works like
// a wave of the streaming x-sweep: it stages the segment's node quantities in
// its own LDS, computes the 64 face fluxes and updates the 63 cells.  TEAM: the
// workgroup's waves share the selections of a round of segments (line_stage);
// otherwise a wave synchronises only with itself.  The stages write distinct arrays
// (u^n -> w1 -> w2 -> u^n; stage 3 reads u^n only at the cell it writes), so
// no wave overwrites what another still reads, and one workgroup barrier per
// stage (which also publishes the per-wave maxima) ends it.  Every arithmetic step is
// the streaming path's, so a member's result is bitwise the one of the streaming
// kernels.  A step of a member takes a fixed latency plus its segments over the waves
// (measured alone: 13 us at 128 nodes, 40 us at 1700), so a batch step lasts about as
// long as its largest member's.

// per-wave LDS of a resident workgroup: staged nodes, face fluxes, listed faces
template <int EQ, int ORDER> struct ResWave {
    static constexpr int NQ = NodeTraits<EQ>::NQ, NC = NodeTraits<EQ>::NC;
    static constexpr int G = ReconTraits<ORDER>::H + 1;
    static constexpr int NN = XW_FACES + 2 * G - 1, NNP = NN + 1;
    static constexpr int DOUBLES = NQ * NNP + NC * XW_FACES + (EQ == ADVECTION ? 0 : 8);
};

// all threads: the maxima of the waves of stage `par` (every thread reads every
// wave's values, so no second barrier is needed); the non-physical flag goes to C
template <int EQ, int NW>
__device__ __forceinline__ void resident_maxima(const double *red, int par, double (&cm)[8], Ctrl &C)
{
    constexpr int NV = Maxima<EQ>::NV;
    const double *r = red + par * NW * 8;
#pragma unroll
    for (int i = 0; i < 8; ++i) cm[i] = 0.0;
    double bad = 0.0;
    for (int w = 0; w < NW; ++w) {
#pragma unroll
        for (int i = 0; i < NV; ++i) cm[i] = fmax(cm[i], r[w * 8 + i]);
        bad = fmax(bad, r[w * 8 + 7]);
    }
    if (bad != 0.0) C.status |= 1;
}

// a wave's maxima to red[par] (lane 0 writes; published by the next barrier)
template <int EQ, int NW>
__device__ __forceinline__ void resident_wave_maxima(Maxima<EQ> &mx, double *red, int par)
{
    constexpr int NV = Maxima<EQ>::NV;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int i = 0; i < NV; ++i) mx.v[i] = wave_max(mx.v[i]);
    const int b = __builtin_amdgcn_ballot_w64(mx.bad != 0) != 0;
    if (lane == 0) {
        double *r = red + (par * NW + wv) * 8;
#pragma unroll
        for (int i = 0; i < NV; ++i) r[i] = mx.v[i];
        r[7] = (double)b;
    }
}

// alpha of the fields from the maxima of a stage input
template <int EQ, bool CH>
__device__ __forceinline__ void line_alpha(const double (&cm)[8], double adv, double (&al)[NodeTraits<EQ>::NC])
{
    constexpr int NC = NodeTraits<EQ>::NC;
    if constexpr (EQ == ADVECTION) {
        al[0] = fabs(adv);
    } else if constexpr (CH) {
        al[0] = cm[0];
        al[1] = cm[1];
        al[NC - 1] = cm[2];
    } else {
        const double a = fmax(cm[0], cm[2]);
#pragma unroll
        for (int c = 0; c < NC; ++c) al[c] = a;
    }
}

// wave w's LDS of a workgroup's (wls: the first's)
template <int EQ, int ORDER> __device__ __forceinline__ LineLds line_lds(double *wls, int w)
{
    using RW = ResWave<EQ, ORDER>;
    double *q = wls + w * RW::DOUBLES, *fh = q + RW::NQ * RW::NNP;
    return LineLds{q, RW::NNP, fh, XW_FACES, (unsigned char *)(fh + RW::NC * XW_FACES)};
}

// The fluxes of the staged segments of a workgroup's NW waves, one each, into their LDS;
// faces: the number of this wave's that count (0: it has no segment).  TEAM: the Euler
// faces that need a selection lie in one or two of the segments, so the waves share them;
// counts: NW words of LDS that no wave reads or writes again before another barrier.
template <int EQ, int ORDER, bool CH, int NW, bool TEAM>
__device__ __forceinline__ void line_round(const KParams &P, double adv, double *wls, int *counts, int faces,
                                           const double (&al)[NodeTraits<EQ>::NC])
{
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const LineLds own = line_lds<EQ, ORDER>(wls, wv);
    const bool shortcut = (P.flags & KF_FULL_SELECTION) == 0;
    if constexpr (EQ == ADVECTION) {
        int sel[2];
        if (faces > 0) own.fh[lane] = advection_flux<ORDER, false>(own.q + lane, nullptr, al[0], adv, P.delta, shortcut, sel);
        wave_sync();
    } else {
        auto rec = [](int, int, int) {};
        const Alpha3 a3{al[0], al[1], al[2]};
        double Fh[3] = {0.0, 0.0, 0.0};
        unsigned long long fail = 0;
        if (faces > 0) fail = line_top<ORDER, CH>(own, al, P.gm1, P.delta, shortcut, lane < faces, Fh, rec);
        if constexpr (TEAM) {
            if (lane == 0) counts[wv] = __popcll(fail);
            __syncthreads();
            // the waves' listed faces, one wave's after the other's
            int upto[NW];
#pragma unroll
            for (int w = 0; w < NW; ++w) upto[w] = (w ? upto[w - 1] : 0) + __builtin_amdgcn_readfirstlane(counts[w]);
            const int nf = upto[NW - 1];
            if (nf) {
#pragma unroll 1
                for (int at = 64 * wv; at < 3 * nf; at += 64 * NW) {
                    const int i = min(at + lane, 3 * nf - 1), s = (i >= nf) + (i >= 2 * nf), k = i - s * nf;
                    int w = 0, before = 0;
#pragma unroll
                    for (int j = 0; j + 1 < NW; ++j) {
                        w += k >= upto[j];
                        before = k >= upto[j] ? upto[j] : before;
                    }
                    const LineLds l = line_lds<EQ, ORDER>(wls, w);
                    line_select<ORDER, CH, false>(l, k - before, s, at + lane < 3 * nf, a3, P.gm1, P.delta, rec);
                }
                __syncthreads();
                line_correct<ORDER, CH>(own, fail, P.gm1, Fh);
            }
        } else {
            line_selections<ORDER, CH, false>(own, fail, a3, P.gm1, P.delta, Fh, rec);
        }
        if (faces > 0) {
#pragma unroll
            for (int c = 0; c < 3; ++c) own.fh[c * XW_FACES + lane] = Fh[c];
        }
        wave_sync();
    }
}

// One stage over a 1D line for the NW waves of a resident workgroup: segments 0 .. NW - 1
// (63 cells each, one a wave), then the next NW, ...  Each wave stages a segment's node quantities in its
// own LDS (wls: the first wave's), computes the segment's 64 face fluxes and updates its
// cells from `in` (and `base`: u^n) into `out`; alpha comes from cm, the maxima of the
// stage input, and the output's maxima accumulate in mx.
// fails: 2 NW words of LDS (two rounds' counts: without a face to select a round has one
// barrier, and a wave may be a round ahead of one that still reads).
template <int EQ, int ORDER, int MODE, bool CH, int NW, bool TEAM>
__device__ __forceinline__ void line_stage(const KParams &P, const Inst &I, int n, const double *in,
                                           const double *base, double *out, double *wls, int *fails, const double (&cm)[8],
                                           double dt, Maxima<EQ> &mx)
{
    using RW = ResWave<EQ, ORDER>;
    constexpr int NC = RW::NC, NQ = RW::NQ, G = RW::G, NN = RW::NN, NNP = RW::NNP;
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double al[NC];
    line_alpha<EQ, CH>(cm, I.adv, al);
    double *wl = wls + wv * RW::DOUBLES, *q = wl, *fh = wl + NQ * NNP;
    const double idx = 1.0 / I.dx, idy = 1.0 / I.dy;
    const int nseg = (n + XW_CELLS - 1) / XW_CELLS;
    for (int seg0 = 0, par = 0; seg0 < nseg; seg0 += NW, par ^= NW) {
        const int sx = (seg0 + wv) * XW_CELLS;
        const bool mine = sx < n;  // (the last of them may be fewer than the waves)
        // node quantities of nodes sx - G .. sx + 63 + G - 1
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int i = lane + 64 * j;
            if (mine && i < NN) {
                const int x = bc_map(sx - G + i, n, I.bcx);
                double U[NC], qq[NQ];
#pragma unroll
                for (int c = 0; c < NC; ++c) U[c] = in[c * n + x];
                node_quantities<EQ>(U, P.gm1, qq);
#pragma unroll
                for (int m = 0; m < NQ; ++m) q[m * NNP + i] = qq[m];
            }
        }
        wave_sync();
        line_round<EQ, ORDER, CH, NW, TEAM>(P, I.adv, wls, fails + par, mine ? n - sx + 1 : 0, al);
        const int x = sx + lane;
        if (lane < XW_CELLS && x < n) {
            double Un[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const double Lc = -(fh[c * XW_FACES + lane + 1] - fh[c * XW_FACES + lane]) * idx;
                Un[c] = rk_combine<MODE>(q[c * NNP + lane + G], base[c * n + x], dt, Lc);
            }
#pragma unroll
            for (int c = 0; c < NC; ++c) out[c * n + x] = Un[c];
            mx.add(Un, P.gamma, idx, idy);
        }
        wave_sync();  // the next segment overwrites the staged nodes and fluxes
        // (every wave is past the selection, or there was none)
    }
}

template <int EQ, int ORDER, int MODE, bool CH, int NW, bool TEAM>
__device__ __forceinline__ void resident_stage(const KParams &P, const Inst &I, int n, const double *in,
                                               const double *base, double *out, double *wls, int *fails, double *red, int par,
                                               double (&cm)[8], Ctrl &C, double dt)
{
    Maxima<EQ> mx;
    mx.reset();
    line_stage<EQ, ORDER, MODE, CH, NW, TEAM>(P, I, n, in, base, out, wls, fails, cm, dt, mx);
    resident_wave_maxima<EQ, NW>(mx, red, par);
    __syncthreads();  // the stage output and every wave's maxima are complete
    resident_maxima<EQ, NW>(red, par, cm, C);
}

// one launch covers members res_order[res_first .. res_first + gridDim.x) (the
// members of one LDS size class, largest first), one workgroup of NW waves each
template <int EQ, int ORDER, bool CH, int NW, bool TEAM>
__global__ __launch_bounds__(64 * NW) void resident_1d(KParams P, int nsteps)
{
    using RW = ResWave<EQ, ORDER>;
    constexpr int NC = RW::NC;
    extern __shared__ double sm[];
    const int slot = P.res_first + (int)blockIdx.x;
    const Inst &I = P.inst[P.res_order ? P.res_order[slot] : slot];
    const int n = I.nx, pitch = I.pitch, tid = threadIdx.x;
    __shared__ int fails[2 * NW];
    double *un = sm;
    double *w1 = un + NC * n;
    double *w2 = w1 + NC * n;
    double *wls = w2 + NC * n;
    double *red = w2 + NC * n + NW * RW::DOUBLES;  // two parities of NW x 8 values
    GMEM double *ug = gmem(I.u);
#pragma unroll
    for (int c = 0; c < NC; ++c)
        for (int j = tid; j < n; j += 64 * NW) un[c * n + j] = ug[c * pitch + j];
    // every thread keeps the same copy of the member's time-loop control
    Ctrl C = *I.ctrl;
    double cm[8];
    {
        const double idx = 1.0 / I.dx, idy = 1.0 / I.dy;
        Maxima<EQ> mx;
        mx.reset();
        for (int j = tid; j < n; j += 64 * NW) {
            double U[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) U[c] = ug[c * pitch + j];
            mx.add(U, P.gamma, idx, idy);
        }
        resident_wave_maxima<EQ, NW>(mx, red, 1);
        __syncthreads();  // u^n loaded, maxima published
        resident_maxima<EQ, NW>(red, 1, cm, C);
    }
    for (int step = 0; step < nsteps; ++step) {
        if (!control_update<EQ>(C, cm[0], cm[2], cm[6], I.dx, I.adv)) break;  // the same in every thread
        const double dt = C.dt;
        // the maxima alternate between two parities from stage to stage (step 0's
        // first stage after the initial maxima's parity 1), so a wave that runs
        // ahead never overwrites values another wave has yet to read
        const int par = (3 * step) & 1;
        resident_stage<EQ, ORDER, M_S1, CH, NW, TEAM>(P, I, n, un, un, w1, wls, fails, red, par, cm, C, dt);
        resident_stage<EQ, ORDER, M_S2, CH, NW, TEAM>(P, I, n, w1, un, w2, wls, fails, red, par ^ 1, cm, C, dt);
        resident_stage<EQ, ORDER, M_S3, CH, NW, TEAM>(P, I, n, w2, un, un, wls, fails, red, par, cm, C, dt);
    }
#pragma unroll
    for (int c = 0; c < NC; ++c)
        for (int j = tid; j < n; j += 64 * NW) ug[c * pitch + j] = un[c * n + j];
    if (tid == 0) *I.ctrl = C;
}

// ---------------------------------------------------------------------------
// Cooperative solver of one mid-sized 1D line (too long for one workgroup's
// LDS, short enough for one segment per wave of at most one workgroup per CU).
// A kernel boundary between stages costs several microseconds, about a stage's
// work on such a line; here one cooperative launch (every workgroup resident)
// runs every controlled step of a call.  A workgroup keeps its cells in LDS and
// registers from the first stage to the last (HBM is touched to load the state and to
// store it), and the arithmetic is the resident solver's (line_round), so a result is
// bitwise the streaming kernels'.
//
// Between stages the workgroups exchange their maxima and the G cells at either end of
// their range, one word at a time: a word is empty (a signalling NaN, which arithmetic
// never gives, and which coop_load takes out of the caller's state) until its writer has stored it, so a reader that finds a value needs no
// barrier, no counter and no cache operation; it waits for what it needs alone, all words
// in flight together.  With the stage states in HBM, a counting barrier between a release
// and an acquire of the caches, and the maxima and the states read after it, this part of
// a stage took 8800 cycles, 3.7 us, of 6 us at 2000 nodes.
//
// Stage s uses words of slot s mod 3 and empties the next slot's.  Nobody reads those any
// more: they held stage s - 2, and every workgroup has published stage s - 1, which it
// does after it has read stage s - 2.  And a workgroup publishes its maxima of stage s
// only after its emptying stores have completed, while a reader turns to slot s + 1 only
// when it has found all workgroups' maxima of stage s.

constexpr unsigned COOP_SPIN_LIMIT = 1u << 19;  // polls of one wait (about 0.5 s; never reached)
constexpr unsigned long long COOP_EMPTY = 0xfff7ffffffffffffull;
constexpr int COOP_CELLS = RES_BLOCK / 64 * XW_CELLS;  // cells of a workgroup

// words of a slot: maxima by value and workgroup, then cells by workgroup, end, place and component
constexpr int coop_slot_words(int nc, int g, int groups) { return groups * (3 + 2 * g * nc); }
static int coop_exchange_words(int eq, int order, int groups)
{
    // (from two workgroups on, 253 nodes, a stage state's buffer holds them: at most 99
    // words a workgroup against 756)
    return groups > 1 ? 3 * coop_slot_words(eq == ADVECTION ? 1 : 3, order == 7 ? 5 : 4, groups) : 0;
}

__device__ __forceinline__ void coop_store(GMEM unsigned long long *p, unsigned long long x)
{
    __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// a value of the caller's state; a NaN with the bits of an empty word, which a reader
// would wait for in vain, as the quiet NaN that arithmetic makes of it
__device__ __forceinline__ double coop_load(GMEM const double *p)
{
    const unsigned long long x = as_bits(*p);
    return as_double(x == COOP_EMPTY ? x | 1ull << 51 : x);
}

// the value of an exchange word once it is there; false after COOP_SPIN_LIMIT polls, or
// once another wait has failed (bar[1])
__device__ __forceinline__ bool coop_wait(GMEM unsigned long long *p, GMEM unsigned *bar, unsigned long long &x)
{
    for (unsigned spin = 0; spin < COOP_SPIN_LIMIT; ++spin) {
        x = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (x != COOP_EMPTY) return true;
        if (spin % 64 == 63 && __hip_atomic_load(&bar[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u) break;
    }
    __hip_atomic_store(&bar[1], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    x = 0;
    return false;
}

// A workgroup's part of the line: cell x0 + i of the stage input at win[c][G + i], the
// halo of G nodes on either side of its `cells`.
template <int EQ, int ORDER> struct CoopLine {
    static constexpr int NC = NodeTraits<EQ>::NC, G = ReconTraits<ORDER>::H + 1, PITCH = COOP_CELLS + 2 * G;
    static constexpr int NV = Maxima<EQ>::NV, NW = RES_BLOCK / 64;
    double win[NC][PITCH];
    double red[NW][4];       // a wave's maxima and its non-physical flag
    double all[3];           // the line's maxima
    int counts[2 * NW];      // listed faces (line_round), by stage parity
    int bad, failed;

    // place of node x0 - G + i (i < G) or x0 + cells + i - G of the halo in a slot; -1: own cell `own`
    __device__ __forceinline__ int halo_word(int i, int c, int x0, int cells, int n, int bc, int groups, int &own) const
    {
        const int x = bc_map(i < G ? x0 - G + i : x0 + cells + i - G, n, bc);
        const int o = x / COOP_CELLS;
        own = x - x0;
        if (o == (int)blockIdx.x) return -1;
        const int k = x - o * COOP_CELLS, oc = min(COOP_CELLS, n - o * COOP_CELLS);
        const int place = k < G ? k : G + k - (oc - G);  // from its start, or up to its end
        return 3 * groups + (o * 2 * G + place) * NC + c;
    }
};

template <int EQ, int ORDER, bool CH>
__global__ __launch_bounds__(RES_BLOCK) void coop_1d(KParams P, int nsteps, unsigned long long *exchange,
                                                    unsigned *bar_)
{
    using RW = ResWave<EQ, ORDER>;
    using CL = CoopLine<EQ, ORDER>;
    constexpr int NW = RES_BLOCK / 64, NC = RW::NC, G = RW::G, NQ = RW::NQ, NN = RW::NN, NNP = RW::NNP, NV = CL::NV;
    __shared__ double wls[NW * RW::DOUBLES];
    __shared__ CL S;
    const Inst &I = P.inst[0];
    const int n = I.nx, bc = I.bcx, tid = threadIdx.x, lane = tid & 63, groups = (int)gridDim.x;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int x0 = (int)blockIdx.x * COOP_CELLS, cells = min(COOP_CELLS, n - x0);
    const int sx = wv * XW_CELLS;                  // the wave's segment, from x0
    const int at = sx + lane;                      // the lane's cell, from x0
    const bool cell = lane < XW_CELLS && at < cells;
    const double idx = 1.0 / I.dx, idy = 1.0 / I.dy, adv = I.adv;
    GMEM double *un = gmem(I.u);
    GMEM unsigned long long *ex = gmem(exchange);
    GMEM unsigned *bar = gmem(bar_);
    const int slot_words = coop_slot_words(NC, G, groups);
    Ctrl C = *I.ctrl;
    double U[NC], base[NC];  // the lane's cell: stage input, u^n
    double cm[8];
    if (tid == 0) S.failed = 0;

    // the new stage input U: to the neighbours and into win, the line's maxima into cm
    auto exchange_stage = [&](int s) {
        GMEM unsigned long long *now = ex + (s % 3) * slot_words, *next = ex + ((s + 1) % 3) * slot_words;
        Maxima<EQ> mx;
        mx.reset();
        if (cell) {
            mx.add(U, P.gamma, idx, idy);
#pragma unroll
            for (int c = 0; c < NC; ++c) S.win[c][G + at] = U[c];
        }
        if (groups > 1 && cell) {
            const int mine = 3 * groups + (int)blockIdx.x * 2 * G * NC;
#pragma unroll
            for (int end = 0; end < 2; ++end) {
                const int k = end == 0 ? at : G + at - (cells - G);
                if (end == 0 ? at < G : at >= cells - G) {
#pragma unroll
                    for (int c = 0; c < NC; ++c) {
                        coop_store(&now[mine + k * NC + c], as_bits(U[c]));
                        coop_store(&next[mine + k * NC + c], COOP_EMPTY);
                    }
                }
            }
        }
        if (groups > 1 && tid < 3) coop_store(&next[tid * groups + (int)blockIdx.x], COOP_EMPTY);
        const bool wbad = __builtin_amdgcn_ballot_w64(mx.bad != 0) != 0;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const double x = wave_max(mx.v[i]);
            if (lane == 0) S.red[wv][i] = x;
        }
        if (lane == 0) S.red[wv][3] = wbad ? 1.0 : 0.0;
        if (tid == 0) S.bad = 0;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's emptying stores are done
        __syncthreads();
        double own = 0.0, bad = 0.0;  // (thread i < 3: value i of the workgroup)
        if (tid < 3) {
            if (tid < NV)
                for (int w = 0; w < NW; ++w) own = fmax(own, S.red[w][tid]);
            for (int w = 0; w < NW; ++w) bad = fmax(bad, S.red[w][3]);
        }
        if (groups == 1) {
            if (tid < 3) S.all[tid] = own;
            if (tid == 0 && bad != 0.0) S.bad = 1;
            if (tid < 2 * G * NC) {
                int o;
                (void)S.halo_word(tid / NC, tid % NC, x0, cells, n, bc, groups, o);
                S.win[tid % NC][tid / NC < G ? tid / NC : cells + tid / NC] = S.win[tid % NC][G + o];
            }
        } else {
            // (the flag is the sign of value 0)
            if (tid < 3) {
                unsigned long long w = as_bits(own);
                if (tid == 0 && bad != 0.0) w |= 1ull << 63;
                coop_store(&now[tid * groups + (int)blockIdx.x], w);
            }
            bool good = true;
            if (wv < 3 && (wv == 0 || wv < NV)) {
                // wave i: value i of all workgroups (advection has none: the flags alone)
                double m = 0.0;
                bool b = false;
                for (int g = lane; g < groups; g += 64) {
                    unsigned long long w;
                    good = coop_wait(&now[wv * groups + g], bar, w) && good;
                    b = b || (w >> 63) != 0;
                    m = fmax(m, as_double(w & ~(1ull << 63)));
                }
                m = wave_max(m);
                b = __builtin_amdgcn_ballot_w64(b) != 0;
                if (lane == 0) {
                    S.all[wv] = m;
                    if (b) S.bad = 1;
                }
            } else if (wv == 3) {
                // the halo
                static_assert(2 * CL::G * CL::NC <= 64, "a lane per word of the halo");
                if (lane < 2 * G * NC) {
                    const int i = lane / NC, c = lane - i * NC;
                    int o;
                    const int k = S.halo_word(i, c, x0, cells, n, bc, groups, o);
                    double x;
                    if (k < 0) {
                        x = S.win[c][G + o];
                    } else {
                        unsigned long long w;
                        good = coop_wait(&now[k], bar, w);
                        x = as_double(w);
                    }
                    S.win[c][i < G ? i : cells + i] = x;
                }
            }
            if (!good) S.failed = 1;
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 8; ++i) cm[i] = i < 3 && i < NV ? S.all[i] : 0.0;
        if (S.bad) C.status |= 1;
        return S.failed == 0;
    };
    // one stage: U from win
    auto stage = [&](auto mode, int s, double dt) {
        constexpr int MODE = decltype(mode)::value;
        double al[NC];
        line_alpha<EQ, CH>(cm, adv, al);
        double *q = wls + wv * RW::DOUBLES;
        const bool mine = sx < cells;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int i = lane + 64 * j;
            if (mine && i < NN) {
                // (nodes past the halo of a last, short segment: no face that counts has them)
                const int k = min(sx + i, cells + 2 * G - 1);
                double V[NC], qq[NQ];
#pragma unroll
                for (int c = 0; c < NC; ++c) V[c] = S.win[c][k];
                node_quantities<EQ>(V, P.gm1, qq);
#pragma unroll
                for (int m = 0; m < NQ; ++m) q[m * NNP + i] = qq[m];
            }
        }
        wave_sync();
        line_round<EQ, ORDER, CH, NW, true>(P, adv, wls, S.counts + NW * (s & 1), mine ? cells - sx + 1 : 0, al);
        if (cell) {
            const double *fh = q + NQ * NNP;
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const double Lc = -(fh[c * XW_FACES + lane + 1] - fh[c * XW_FACES + lane]) * idx;
                U[c] = rk_combine<MODE>(q[c * NNP + lane + G], base[c], dt, Lc);
            }
        }
        // (Euler: a barrier of line_round is behind every wave's reads of win)
        if (EQ == ADVECTION) __syncthreads();
        return exchange_stage(s);
    };

#pragma unroll
    for (int c = 0; c < NC; ++c) U[c] = base[c] = cell ? coop_load(&un[c * n + x0 + at]) : 0.0;
    bool ok = exchange_stage(0);
    int taken = 0;
    for (int step = 0; ok && step < nsteps; ++step) {
        if (!control_update<EQ>(C, cm[0], cm[2], cm[6], I.dx, I.adv)) break;  // the same in every thread
        const double dt = C.dt;
        ok = stage(std::integral_constant<int, M_S1>{}, 1, dt) && stage(std::integral_constant<int, M_S2>{}, 2, dt) &&
             stage(std::integral_constant<int, M_S3>{}, 3, dt);
        if (!ok) break;
        ++taken;
#pragma unroll
        for (int c = 0; c < NC; ++c) base[c] = U[c];
    }
    if (taken && cell) {
#pragma unroll
        for (int c = 0; c < NC; ++c) un[c * n + x0 + at] = base[c];
    }
    if (blockIdx.x == 0 && tid == 0) {
        if (!ok) C.status |= 2;
        *I.ctrl = C;
    }
}

// empty exchange words and a clear failure flag before a cooperative launch
__global__ void coop_reset(unsigned long long *exchange, int words, unsigned *bar)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < words) exchange[t] = COOP_EMPTY;
    if (t < 2) bar[t] = 0u;
}

// replace a member's control block (pool admission and retirement); info, if
// given, receives the old block's done flag, status, step count and time
__global__ void set_ctrl(Ctrl *c, Ctrl v, double *info)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        if (info) {
            info[0] = c->done;
            info[1] = c->status;
            info[2] = (double)c->steps;
            info[3] = c->t;
        }
        *c = v;
    }
}

// copy between a dense and a row-padded layout (pool admission and retirement)
__global__ void copy_pitched(const double *src, long long sp, double *dst, long long dp, int width, long long rows)
{
    for (long long r = blockIdx.y; r < rows; r += gridDim.y)
        for (int x = blockIdx.x * blockDim.x + threadIdx.x; x < width; x += gridDim.x * blockDim.x)
            dst[(long long)r * dp + x] = src[(long long)r * sp + x];
}

// ---------------------------------------------------------------------------
// kernel selection and launchers
using KFn = void (*)(KParams);
using KFn2 = void (*)(KParams, int);

template <int EQ, int ORDER, bool REC, bool CH> static KFn pick_x_mode(int mode)
{
    switch (mode) {
    case M_RHS: return sweep_x<EQ, ORDER, M_RHS, REC, CH>;
    case M_S1: return sweep_x<EQ, ORDER, M_S1, REC, CH>;
    case M_S2: return sweep_x<EQ, ORDER, M_S2, REC, CH>;
    default: return sweep_x<EQ, ORDER, M_S3, REC, CH>;
    }
}
template <int EQ, bool REC, bool CH> static KFn pick_x_order(int order, int mode)
{
    return order == 7 ? pick_x_mode<EQ, 7, REC, CH>(mode) : pick_x_mode<EQ, 5, REC, CH>(mode);
}
template <int EQ, bool CH> static KFn pick_x_rec(int order, int mode, bool rec)
{
    return rec ? pick_x_order<EQ, true, CH>(order, mode) : pick_x_order<EQ, false, CH>(order, mode);
}
// ch: characteristic fields (advection has one variable and always takes this path)
static KFn pick_x(int eq, int order, int mode, bool rec, bool ch)
{
    if (eq == ADVECTION) return pick_x_rec<ADVECTION, true>(order, mode, rec);
    return ch ? pick_x_rec<EULER1D, true>(order, mode, rec) : pick_x_rec<EULER1D, false>(order, mode, rec);
}
static KFn pick_maxima(int eq)
{
    return eq == ADVECTION ? state_maxima<ADVECTION> : (eq == EULER1D ? state_maxima<EULER1D> : state_maxima<EULER2D>);
}
static KFn pick_control(int eq)
{
    return eq == ADVECTION ? step_control<ADVECTION> : (eq == EULER1D ? step_control<EULER1D> : step_control<EULER2D>);
}

static hipError_t launch(KFn fn, int grid, int block, const KParams &p, hipStream_t s)
{
    KParams copy = p;
    void *args[] = {&copy};
    return hipLaunchKernel((const void *)fn, dim3(grid > 0 ? grid : 1), dim3(block), args, 0, s);
}

static int occupancy(KFn fn)
{
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, (const void *)fn, BLOCK, 0) != hipSuccess || n < 1) n = 1;
    return n;
}

hipError_t launch_sweep_x(int eq, int order, int mode, bool rec, bool ch, const KParams &p, int grid, hipStream_t s)
{
    return launch(pick_x(eq, order, mode, rec, ch), grid, BLOCK, p, s);
}

hipError_t launch_state_maxima(int eq, const KParams &p, int grid, hipStream_t s)
{
    return launch(pick_maxima(eq), grid, BLOCK, p, s);
}

hipError_t launch_reset_maxima(int eq, const KParams &p, int n_inst, hipStream_t s)
{
    KParams copy = p;
    int words = AMAX_SLOTS * amax_slot_words(eq);
    void *args[] = {&copy, &words};
    return hipLaunchKernel((const void *)reset_maxima, dim3((n_inst * words + BLOCK - 1) / BLOCK), dim3(BLOCK), args, 0, s);
}

hipError_t launch_begin_lone(int eq, const KParams &p, Inst *inst, const double *u, double *lx, Ctrl *c, const Ctrl &v,
                             int mode, hipStream_t s)
{
    KParams copy = p;
    Ctrl cv = v;
    int words = AMAX_SLOTS * amax_slot_words(eq);
    void *args[] = {&copy, &inst, &u, &lx, &c, &cv, &mode, &words};
    return hipLaunchKernel((const void *)begin_lone, dim3(1), dim3(BLOCK), args, 0, s);
}

hipError_t launch_step_control(int eq, const KParams &p, int n_inst, hipStream_t s)
{
    return launch(pick_control(eq), (n_inst + 63) / 64, 64, p, s);
}

hipError_t launch_set_ctrl(Ctrl *c, const Ctrl &v, double *info, hipStream_t s)
{
    Ctrl copy = v;
    void *args[] = {&c, &copy, &info};
    return hipLaunchKernel((const void *)set_ctrl, dim3(1), dim3(64), args, 0, s);
}

hipError_t launch_copy_pitched(const double *src, long long sp, double *dst, long long dp, int width,
                               long long rows, hipStream_t s)
{
    if (width <= 0 || rows <= 0) return hipSuccess;
    const dim3 grid((unsigned)std::min((width + 255) / 256, 64), (unsigned)std::min(rows, 8192ll));
    void *args[] = {&src, &sp, &dst, &dp, &width, &rows};
    return hipLaunchKernel((const void *)copy_pitched, grid, dim3(256), args, 0, s);
}

using KFn2c = void (*)(KParams, int, unsigned long long *, unsigned *);

template <bool TEAM> static KFn2 pick_resident_team(int order, bool ch)
{
    constexpr int NW = RES_BLOCK / 64;
    if (ch) return order == 7 ? resident_1d<EULER1D, 7, true, NW, TEAM> : resident_1d<EULER1D, 5, true, NW, TEAM>;
    return order == 7 ? resident_1d<EULER1D, 7, false, NW, TEAM> : resident_1d<EULER1D, 5, false, NW, TEAM>;
}

static KFn2 pick_resident(int eq, int order, bool ch, bool team)
{
    constexpr int NW = RES_BLOCK / 64;
    if (eq == ADVECTION)
        return order == 7 ? resident_1d<ADVECTION, 7, true, NW, false> : resident_1d<ADVECTION, 5, true, NW, false>;
    return team ? pick_resident_team<true>(order, ch) : pick_resident_team<false>(order, ch);
}

hipError_t launch_resident(int eq, int order, bool ch, bool team, int block, const KParams &p, int n_inst, int nsteps,
                           size_t lds, hipStream_t s)
{
    if (eq == EULER2D || block != RES_BLOCK) return hipErrorInvalidValue;
    const KFn2 fn = pick_resident(eq, order, ch, team);
    // dynamic LDS beyond the default limit must be allowed per kernel
    const hipError_t e = hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    KParams copy = p;
    void *args[] = {&copy, &nsteps};
    return hipLaunchKernel((const void *)fn, dim3(n_inst), dim3(block), args, lds, s);
}

static KFn2c pick_coop(int eq, int order, bool ch)
{
    if (eq == ADVECTION) return order == 7 ? coop_1d<ADVECTION, 7, true> : coop_1d<ADVECTION, 5, true>;
    if (ch) return order == 7 ? coop_1d<EULER1D, 7, true> : coop_1d<EULER1D, 5, true>;
    return order == 7 ? coop_1d<EULER1D, 7, false> : coop_1d<EULER1D, 5, false>;
}

int coop_max_groups(int eq, int order, bool ch)
{
    int dev = 0, cus = 0, coop = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess || !coop) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)pick_coop(eq, order, ch), RES_BLOCK, 0) !=
        hipSuccess)
        return 0;
    return cus * per_cu;
}

hipError_t launch_coop(int eq, int order, bool ch, int groups, const KParams &p, int nsteps,
                       unsigned long long *exchange, unsigned *bar, hipStream_t s, bool *refused)
{
    *refused = false;
    if (eq == EULER2D || groups < 1) return hipErrorInvalidValue;
    const int words = coop_exchange_words(eq, order, groups);
    hipLaunchKernelGGL(coop_reset, dim3(words / BLOCK + 1), dim3(BLOCK), 0, s, exchange, words, bar);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    KParams copy = p;
    void *args[] = {&copy, &nsteps, &exchange, &bar};
    const hipError_t ce = hipLaunchCooperativeKernel((const void *)pick_coop(eq, order, ch), dim3(groups),
                                                     dim3(RES_BLOCK), args, 0, s);
    *refused = ce != hipSuccess;
    return ce;
}

size_t resident_lds_limit()
{
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) return 0;
    // the kernel's static LDS (control copy, flag) comes on top of the dynamic part
    return v > 256 ? (size_t)v - 256 : 0;
}

int resident_groups_per_cu(int eq, int order, bool ch)
{
    int n = 0;
    if (eq == EULER2D ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, (const void *)pick_resident(eq, order, ch, false), RES_BLOCK, 0) !=
            hipSuccess)
        return 0;
    return n;
}

int occupancy_x(int eq, int order, int mode, bool rec, bool ch) { return occupancy(pick_x(eq, order, mode, rec, ch)); }
int occupancy_maxima(int eq) { return occupancy(pick_maxima(eq)); }

}  // namespace enoao
