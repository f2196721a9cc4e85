// enoao_common.hpp -- structures shared by the host runtime and the HIP kernels.
//
// A "batch" is the unit every kernel works on: an array of instance
// descriptors in device memory plus the flattened lists of line tiles of all
// instances.  A single plan is a batch of one instance, so the plain, batched
// and served paths run the same kernels.
#pragma once

#include <stdint.h>

namespace enoao {

enum Equation : int { ADVECTION = 0, EULER1D = 1, EULER2D = 2 };
enum Bc : int { BC_PERIODIC = 0, BC_TRANSMISSIVE = 1 };

// x-sweep tiles: each wave reconstructs 64 consecutive faces of one grid line
// and updates the 63 cells between them; a workgroup holds 4 such segments.
constexpr int XW_FACES = 64;
constexpr int XW_CELLS = XW_FACES - 1;
constexpr int XW_SEGS = 4;
// 2D stages: a wave owns a strip of columns, one lane per column, the outer ones
// the halo of 4 (order 7: 5) nodes on either side that an x-face reads.  A strip's
// rows are cut into blocks of equal height to within one; a unit of work is one
// block of one strip.
constexpr int strip_cells(int order) { return order == 7 ? 54 : 56; }
// Row segments whose faces need a selection are listed for a second kernel: pieces of a
// strip's row of at most FIX_FACES faces, two passes of the wave that takes one, as far as
// the places of a row allow (FIX_SPLIT cells a place; a row along a shock holds up to 169
// faces).  The pieces of two passes are dealt before those of one, so that every wave has
// about the same to do.  The units are cut into FIX_RANGES ranges with a list
// and a counter each, the counters a cache line apart: the waves that end a launch
// together take their places at once, and an atomic on one line takes 20 ns.  A list is
// filled from both ends, a counter holds both numbers: its low half the pieces of two
// passes, from the list's start on, its high half those of one, from the end back.  Four
// sets of counters, three used in turn by the stages of a step, the fourth by an
// evaluation of L.
constexpr int FIX_SPLIT = 10, FIX_FACES = 32, FIX_PASS = 16;
constexpr int fix_places(int nx) { return nx > 5 * FIX_SPLIT ? 6 : (nx + FIX_SPLIT - 1) / FIX_SPLIT; }  // per strip and row
constexpr int FIX_ENTRY_BYTES = 32, FIX_RANGES = 32, FIX_COUNTER_STRIDE = 8;
constexpr int FIX_SET_WORDS = FIX_RANGES * FIX_COUNTER_STRIDE, FIX_SETS = 4;
constexpr int BLOCK = 256;

// per-field maxima kept per instance: three ring slots of 8 values each
// (non-negative doubles stored as their IEEE bit patterns so that unsigned
// integer max is the floating-point max):
//   [0..2] max |u-c|, |u|, |u+c| along x    [3..5] same along y (v)
//   [6]    max (|u|+c)/dx + (|v|+c)/dy (2D time step)
// A 2D slot has eight copies, a cache line each, that the workgroups share in turn
// and its readers fold: hundreds of workgroups end a launch together, and their
// atomics on one line took 5 us of a 20 us stage.
constexpr int AMAX_VALS = 8;
constexpr int AMAX_SLOTS = 3;
constexpr int amax_copies(int eq) { return eq == EULER2D ? 8 : 1; }
constexpr int amax_slot_words(int eq) { return AMAX_VALS * amax_copies(eq); }

// Time-loop control of one instance (device memory).
struct Ctrl {
    double dt;          // step size of the step in flight
    double t;           // time reached (after the step in flight)
    double t_final;     // end time (+inf: none)
    double cfl;         // CFL number for the device-computed step (if dt_fixed <= 0)
    double dt_fixed;    // > 0: constant step
    long long steps;    // steps taken
    long long max_steps;
    int done;           // 1: no further steps; kernels skip the instance
    int status;         // bit 0: non-physical state met
    int pad0, pad1;
};

// One instance of a batch (device memory).
struct Inst {
    double *u;                  // u^n: caller state, updated in place by stage 3
    double *w1, *w2;            // stage-1 and stage-2 states
    double *lx;                 // rhs: the L output
    unsigned long long *amax;   // AMAX_SLOTS x amax_copies x AMAX_VALS
    Ctrl *ctrl;
    uint8_t *sel;               // selection record or nullptr
    int nx, ny;
    int bcx, bcy;
    double dx, dy;
    double adv;                 // advection speed
    int segs_per_row;           // ceil(nx / XW_CELLS)
    int strips;                 // 2D: ceil(nx / strip_cells(order))
    int low_rows, extra_rows;   // 2D: rows of a unit, one more in the first extra_rows blocks of rows
    double inv_strips;          // 1 / strips
    int pitch;                  // row pitch of every state buffer, elements (>= nx; planes pitch * ny apart)
    long long xtile0, unit0;    // first x tile / 2D unit of this instance in the batch lists
    long long xtiles, units;    // number of x tiles / 2D units
    long long list0;            // 2D: list places of the instances before this one
};

// LDS-resident solver of small 1D members: one workgroup of RES_BLOCK threads
// holds a member's state and both Runge-Kutta stage states in LDS for a whole
// call; each of its waves stages the nodes of one 64-face segment at a time,
// and that segment's face fluxes, in LDS of its own.
constexpr int RES_BLOCK = 256;

// dynamic LDS bytes of a resident member of n nodes (nc components, nq staged
// quantities per node, halo width g, block threads): u^n and the two stage
// states, each wave's segment staging (nodes, face fluxes and, for the Euler
// equations, 64 bytes of listed faces), two parities of per-wave maxima
constexpr unsigned long long resident_lds_bytes(int nc, int nq, int g, long long n, int block = RES_BLOCK)
{
    const long long nnp = 64 + 2 * g, waves = block / 64;
    return 8ull * (unsigned long long)(3 * nc * n + waves * (nq * nnp + nc * 64 + (nc > 1 ? 8 : 0)) + 2 * waves * 8);
}

// Batch header (device memory): kernels read the instance count and the tile
// totals from here, so a captured graph stays valid when the active set changes.
struct BatchHdr {
    int n_inst;
    int pad;
    long long xtiles_total, units_total;
    unsigned lists[FIX_RANGES + 1];  // 2D: where each range's list starts, and the last one's end
};

// units per range of the lists (a launch has fewer than 2^32)
constexpr unsigned fix_range_units(long long units)
{
    return units > FIX_RANGES ? ((unsigned)units + FIX_RANGES - 1) / FIX_RANGES : 1u;
}

}  // namespace enoao
