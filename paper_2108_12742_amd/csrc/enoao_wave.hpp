// enoao_wave.hpp -- helpers shared by the kernel sources: device-memory pointers,
// boundary mapping, member lookup, maxima, stage combine, wave-level exchange.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "enoao_common.hpp"
#include "enoao_device.hpp"
#include "enoao_kernels.hpp"

namespace enoao {

// Workgroups sharing a persistent launch's tile list of T tiles: the whole
// grid, or for a pool as many as give P.tiles_per_wg tiles each (at least
// P.grid_min, at most the grid).  A pool's grid covers the machine several
// times over; many small chunks let the workgroups that finish early take
// more of them, which evens out members of uneven cost, while a pool holding
// few tiles keeps chunks long enough to pay for their first loads.
__device__ __forceinline__ long long chunk_groups(const KParams &P, long long T)
{
    const long long g = gridDim.x;
    if (P.tiles_per_wg <= 0) return g;
    return min(g, max((long long)P.grid_min, T / P.tiles_per_wg));
}

__device__ __forceinline__ int bc_map(int k, int n, int bc)
{
    if (bc == BC_PERIODIC) {
        int r = k % n;
        return r < 0 ? r + n : r;
    }
    return k < 0 ? 0 : (k >= n ? n - 1 : k);
}

// Device-memory pointers.  The state and control pointers reach a kernel through
// the instance table in memory, so the compiler cannot tell that they address
// global memory and would emit flat instructions for them.  Flat loads and
// stores count against the LDS counter too, so every wait for an LDS read would
// also wait for the next tile's global prefetch in flight (and for the previous
// tile's stores).  Typed as global they compile to global instructions.
#define GMEM __attribute__((address_space(1)))
template <typename T> __device__ __forceinline__ GMEM T *gmem(T *p) { return (GMEM T *)p; }

// wave-uniform copy of a value (scalar registers)
template <typename T> __device__ __forceinline__ T uniform(T x)
{
    static_assert(sizeof(T) % 4 == 0, "32-bit multiple");
    union { T v; int w[sizeof(T) / 4]; } a;
    a.v = x;
#pragma unroll
    for (int i = 0; i < (int)(sizeof(T) / 4); ++i) a.w[i] = __builtin_amdgcn_readfirstlane(a.w[i]);
    return a.v;
}

__device__ __forceinline__ double as_double(unsigned long long b) { return __longlong_as_double((long long)b); }
__device__ __forceinline__ unsigned long long as_bits(double d) { return (unsigned long long)__double_as_longlong(d); }

// a range's counter while its list is empty: the list's start and end
__device__ __forceinline__ unsigned long long fix_empty(const KParams &P, unsigned range)
{
    return (unsigned long long)P.hdr->lists[range + 1] << 32 | P.hdr->lists[range];
}

// value of the neighbouring lane (lane 0 / 63 keep their own)
template <int CTRL> __device__ __forceinline__ double dpp_move(double x)
{
    union { double d; int w[2]; } a, b;
    a.d = x;
#pragma unroll
    for (int i = 0; i < 2; ++i) b.w[i] = __builtin_amdgcn_update_dpp(a.w[i], a.w[i], CTRL, 0xf, 0xf, false);
    return b.d;
}
__device__ __forceinline__ double lane_prev(double x) { return dpp_move<0x138>(x); }  // wave_shr:1
__device__ __forceinline__ double lane_next(double x) { return dpp_move<0x130>(x); }  // wave_shl:1

// value of another lane of the quad (every lane has one: no old value to keep)
template <int PERM> __device__ __forceinline__ double quad_move(double x)
{
    union { double d; int w[2]; } a, b;
    a.d = x;
#pragma unroll
    for (int i = 0; i < 2; ++i) b.w[i] = __builtin_amdgcn_mov_dpp(a.w[i], PERM, 0xf, 0xf, false);
    return b.d;
}

// maximum over the lanes whose numbers agree in the last three bits (the copies of a maxima slot)
__device__ __forceinline__ double copies_max(double x)
{
    static_assert(AMAX_VALS == 8, "a lane's value is its number's last three bits");
    x = fmax(x, dpp_move<0x128>(x));  // row_ror:8
    union { double d; unsigned w[2]; } a, lo, hi;
    a.d = x;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const auto r = __builtin_amdgcn_permlane16_swap(a.w[i], a.w[i], false, false);  // even rows, odd rows
        lo.w[i] = r[0];
        hi.w[i] = r[1];
    }
    a.d = fmax(lo.d, hi.d);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const auto r = __builtin_amdgcn_permlane32_swap(a.w[i], a.w[i], false, false);  // the halves
        lo.w[i] = r[0];
        hi.w[i] = r[1];
    }
    return fmax(lo.d, hi.d);
}

// sum of the lanes up to each
__device__ __forceinline__ unsigned wave_scan(unsigned x)
{
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);  // row_shr:1
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);  // row_shr:2
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);  // row_shr:4
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);  // row_shr:8
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1 and 3
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2 and 3
    return x;
}

// a lane's place among the lanes of a mask
__device__ __forceinline__ unsigned mask_place(unsigned long long m)
{
    return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

// lane i's value, in scalar registers
__device__ __forceinline__ double lane_value(double x, int i)
{
    union { double d; int w[2]; } a;
    a.d = x;
    a.w[0] = __builtin_amdgcn_readlane(a.w[0], i);
    a.w[1] = __builtin_amdgcn_readlane(a.w[1], i);
    return a.d;
}

// maximum over the wave's lanes
__device__ __forceinline__ double wave_max(double x)
{
    x = fmax(x, dpp_move<0xb1>(x));   // quad_perm 1, 0, 3, 2
    x = fmax(x, dpp_move<0x4e>(x));   // quad_perm 2, 3, 0, 1
    x = fmax(x, dpp_move<0x141>(x));  // row_half_mirror
    x = fmax(x, dpp_move<0x140>(x));  // row_mirror: each lane its row's maximum
    x = fmax(x, dpp_move<0x142>(x));  // row_bcast:15 into the next row
    x = fmax(x, dpp_move<0x143>(x));  // row_bcast:31 into rows 2 and 3
    return lane_value(x, 63);
}

// The last of n >= 1 members whose key is at most x (the first's is), searched by a whole
// wave 64 keys at a time: one load's latency for up to 64 members and two for 4096, where
// halving the range takes one per bit (512 members: nine, 4 us before a kernel's first load).
template <class Key> __device__ __forceinline__ int find_last(int n, long long x, const Key &key)
{
    const int lane = threadIdx.x & 63;
    int lo = 0;
    for (int len = n; len > 1;) {
        const int step = (len + 63) / 64, k = lo + lane * step;
        const bool le = lane * step < len && key(k) <= x;
        const int c = __popcll(__builtin_amdgcn_ballot_w64(le)) - 1;
        lo += c * step;
        len = min(step, len - c * step);
    }
    return lo;
}

// ---------------------------------------------------------------------------
// Maxima of the per-field wave speeds of a state (for alpha of the next
// evaluation and for the CFL step), and the non-physical flag.
template <int EQ> struct Maxima {
    static constexpr int NV = EQ == EULER2D ? 7 : (EQ == EULER1D ? 3 : 0);  // values in use
    double v[7];
    int bad;
    __device__ void reset()
    {
#pragma unroll
        for (int i = 0; i < 7; ++i) v[i] = 0.0;
        bad = 0;
    }
    // U in the natural component order; idx, idy = 1/dx, 1/dy
    __device__ void add(const double *U, double gamma, double idx, double idy)
    {
        if constexpr (EQ == ADVECTION) {
            bad |= !(U[0] == U[0]);
        } else if constexpr (EQ == EULER1D) {
            const double rho = U[0], ir = rcp_nr(rho), u = U[1] * ir;
            const double p = (gamma - 1.0) * fma(-0.5 * rho, u * u, U[2]);
            const double c = sqrt_nr(gamma * p * ir);
            bad |= !(rho > 0.0 && p > 0.0);
            v[0] = fmax(v[0], fabs(u - c));
            v[1] = fmax(v[1], fabs(u));
            v[2] = fmax(v[2], fabs(u + c));
        } else {
            const double rho = U[0], ir = rcp_nr(rho), u = U[1] * ir, w = U[2] * ir;
            const double p = (gamma - 1.0) * fma(-0.5 * rho, fma(u, u, w * w), U[3]);
            const double c = sqrt_nr(gamma * p * ir);
            bad |= !(rho > 0.0 && p > 0.0);
            v[0] = fmax(v[0], fabs(u - c));
            v[1] = fmax(v[1], fabs(u));
            v[2] = fmax(v[2], fabs(u + c));
            v[3] = fmax(v[3], fabs(w - c));
            v[4] = fmax(v[4], fabs(w));
            v[5] = fmax(v[5], fabs(w + c));
            v[6] = fmax(v[6], fma(fabs(u) + c, idx, (fabs(w) + c) * idy));
        }
    }
    // workgroup reduction, then one atomic per value into the instance's slot
    __device__ void flush(GMEM unsigned long long *amax, GMEM Ctrl *ctrl, int slot, double *red)
    {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
        for (int i = 0; i < NV; ++i) v[i] = wave_max(v[i]);
        const int b = __builtin_amdgcn_ballot_w64(bad != 0) != 0;
        if (lane == 0) {
#pragma unroll
            for (int i = 0; i < NV; ++i) red[wave * 8 + i] = v[i];
            red[wave * 8 + 7] = (double)b;
        }
        __syncthreads();
        if (threadIdx.x < NV || threadIdx.x == 7) {
            double x = red[threadIdx.x];
            for (int w = 1; w < BLOCK / 64; ++w) x = fmax(x, red[w * 8 + threadIdx.x]);
            if (threadIdx.x < NV) {
                if (slot >= 0)
                    __hip_atomic_fetch_max(&amax[slot * amax_slot_words(EQ) + blockIdx.x % amax_copies(EQ) * AMAX_VALS + threadIdx.x],
                                           as_bits(x), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
            } else if (x != 0.0) {
                __hip_atomic_fetch_or(&ctrl->status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        __syncthreads();
        reset();
    }
};

// Reconstruction variables.  CH: the characteristic fields of the face's Roe
// state (Section 4), with the scaled projection and the field scales above;
// otherwise the conserved components themselves (identity projection, scale 1,
// and one alpha for all of them).
template <int NC, bool CH>
__device__ __forceinline__ void to_fields(const RoeState &r, const double (&x)[NC], double (&w)[NC])
{
    if constexpr (CH) {
        project<NC>(r, x, w);
    } else {
#pragma unroll
        for (int c = 0; c < NC; ++c) w[c] = x[c];
    }
}

template <int NC, bool CH>
__device__ __forceinline__ void from_fields(const RoeState &r, const double (&w)[NC], double (&F)[NC])
{
    if constexpr (CH) {
        back_project<NC>(r, w, F);
    } else {
#pragma unroll
        for (int c = 0; c < NC; ++c) F[c] = w[c];
    }
}

template <int NC, bool CH> __device__ __forceinline__ constexpr double fscale(int s)
{
    return CH ? field_scale<NC>(s) : 1.0;
}

// RK stage combine (Shu-Osher form): s = 1: in + dt L; s = 2: 3/4 base +
// 1/4 (in + dt L); s = 3: 1/3 base + 2/3 (in + dt L).
template <int MODE>
__device__ __forceinline__ double rk_combine(double in, double base, double dt, double L)
{
    const double y = fma(dt, L, in);
    if constexpr (MODE == M_S1) return y;
    else if constexpr (MODE == M_S2) return fma(0.75, base, 0.25 * y);
    else return fma(1.0 / 3.0, base, (2.0 / 3.0) * y);
}

// LDS exchange among the lanes of one wave: the wave's LDS operations are
// performed in order, so a wavefront-scope fence pair around a wave barrier
// orders each lane's writes before every lane's later reads.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace enoao
