// rn_cg.hpp -- device helpers shared by the pass kernels (rn_kernels.hip) and
// the resident iteration loop (rn_loop.hpp): lane moves, memory access forms,
// the scalar steps of the recurrence and the geometry of the tiles.
#pragma once

#include "rn_device.hpp"

#include <math.h>
#include <stddef.h>

namespace rn {

// ---------------------------------------------------------------- helpers

// Lane moves inside a wave without the LDS crossbar. __shfl and its kin
// compile to ds_bpermute, which takes an LDS instruction and a wait on the
// lgkm counter per move; a DPP move is one VALU instruction and v_readlane
// one more. lane_below(v): lane l receives lane l-1's v (whole-wave shift by
// one, DPP wave_shr); lane_above(v): lane l receives lane l+1's v (wave_shl).
// The lane at the wave's edge, which has no source, keeps its own v; every
// caller overrides it. lane_bcast(v, l): lane l's v in every lane (l a
// compile-time constant).
constexpr int kDppWaveShl1 = 0x130, kDppWaveShr1 = 0x138;

template <int CTRL>
__device__ __forceinline__ int dpp_move(int v)
{
    return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xf, 0xf, false);
}

template <int CTRL>
__device__ __forceinline__ float dpp_move(float v)
{
    return __builtin_bit_cast(float, dpp_move<CTRL>(__builtin_bit_cast(int, v)));
}

template <int CTRL>
__device__ __forceinline__ double dpp_move(double v)
{
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = dpp_move<CTRL>((int)(b & 0xffffffffll)), hi = dpp_move<CTRL>((int)(b >> 32));
    return __builtin_bit_cast(double, ((long long)hi << 32) | (long long)(unsigned)lo);
}

template <typename T>
__device__ __forceinline__ T lane_below(T v) { return dpp_move<kDppWaveShr1>(v); }

template <typename T>
__device__ __forceinline__ T lane_above(T v) { return dpp_move<kDppWaveShl1>(v); }

__device__ __forceinline__ float lane_bcast(float v, int l)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}

__device__ __forceinline__ double lane_bcast(double v, int l)
{
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), l);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (long long)(unsigned)lo);
}

// lane_at(v, l): lane l's v in every lane, l uniform over the wave.
__device__ __forceinline__ float lane_at(float v, int l) { return lane_bcast(v, l); }
__device__ __forceinline__ double lane_at(double v, int l) { return lane_bcast(v, l); }

// Sum over the 64 lanes, the same value in every lane (every lane active):
// pairs, then quads (DPP quad permutations), then eights and sixteens (DPP
// half-row and row mirrors: lane i meets lane 7 - i, then 15 - i, so both
// partners form the same sum), then the four row sums in a fixed order.
constexpr int kDppQuadSwap1 = 0xB1, kDppQuadSwap2 = 0x4E, kDppRowMirror = 0x140, kDppRowHalfMirror = 0x141;

__device__ __forceinline__ double wave_sum(double v)
{
    v += dpp_move<kDppQuadSwap1>(v);
    v += dpp_move<kDppQuadSwap2>(v);
    v += dpp_move<kDppRowHalfMirror>(v);
    v += dpp_move<kDppRowMirror>(v);
    return (lane_bcast(v, 0) + lane_bcast(v, 16)) + (lane_bcast(v, 32) + lane_bcast(v, 48));
}

// The CG state, the bonds and the field live in device memory: accesses
// through these casts compile to global_load / global_store, which count on
// the vector-memory counter only. Through a generic pointer (every pointer
// read from an argument table is one) they are flat accesses, which count on
// the lgkm counter as well, so each wait for an LDS read or a lane move would
// also wait for every load and store still in flight.
#define RN_GLOBAL __attribute__((address_space(1)))

template <typename T>
__device__ __forceinline__ T ldg(const T *p) { return *(const RN_GLOBAL T *)p; }

template <typename T>
__device__ __forceinline__ void stg(T *p, T v) { *(RN_GLOBAL T *)p = v; }

// Partial sums travel between workgroups through write-through (system-scope)
// stores and loads that bypass the per-XCD L2s, so no workgroup has to write
// back or invalidate its L2 (a device-scope fence would do both).
__device__ __forceinline__ double ld_through(const double *p)
{
    return __hip_atomic_load((const RN_GLOBAL double *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__device__ __forceinline__ void st_through(double *p, double v)
{
    __hip_atomic_store((RN_GLOBAL double *)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Loads and stores of the CG state, by coherence mode:
//   COH 0 (one launch per round): plain accesses; a kernel boundary makes
//     every store visible to the next launch, on any XCD.
//   COH 1 (persistent launch, a network's items on any XCD): a pass reads
//     what workgroups on other XCDs, with their own L2s, wrote in the previous
//     pass, and its own XCD's L2 may still hold the buffer from two passes
//     back, so the state moves by device-scope accesses (global_load /
//     global_store with sc1), which write through the L2 and do not return a
//     line another XCD has since written.
//   COH 2 (persistent launch, all items of a network on one XCD): the state
//     is coherent in that XCD's L2, so stores are plain (the per-CU L1 writes
//     through to it). Loads are still device-scope (sc1): a workgroup-scope
//     load (sc0) or a plain one is served by the CU's own L1, which keeps a
//     line another CU has since written (outside threadgroup-split mode the
//     memory model lets workgroup scope hit L1); sc1 loads skip L1 and hit L2.
// The bonds, the mask and the FP64 conductances are read-only during the
// iterations and keep plain loads in every mode.
// The same through a generic pointer (flat_load / flat_store): the 3D plane
// stream below uses these; it measured faster with them (168.6 against 176.8
// us per pass on a 256^3 network), the 2D tile slower.
template <int COH, typename T>
__device__ __forceinline__ T ldc_flat(const T *p)
{
    if constexpr (COH != 0) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else return *p;
}

template <int COH, typename T>
__device__ __forceinline__ void stc_flat(T *p, T v)
{
    if constexpr (COH == 1) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *p = v;
}

template <int COH, typename T>
__device__ __forceinline__ T ldc(const T *p)
{
    if constexpr (COH != 0) return __hip_atomic_load((const RN_GLOBAL T *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else return ldg(p);
}

template <int COH, typename T>
__device__ __forceinline__ void stc(T *p, T v)
{
    if constexpr (COH == 1) __hip_atomic_store((RN_GLOBAL T *)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else stg(p, v);
}

// The memory scope of the reduction's own stores (partials, ticket resets,
// control block) in each mode: across XCDs unless the network is on one.
// Its loads are device-scope in every persistent mode (see ldc).
template <int COH>
constexpr int store_scope() { return COH == 2 ? __HIP_MEMORY_SCOPE_WORKGROUP : __HIP_MEMORY_SCOPE_AGENT; }

// Workgroup index -> tile index so that each XCD (workgroups are dealt to the
// 8 XCDs round-robin) owns one contiguous range of tiles and shares halos in
// its own L2. `grid` is a multiple of 8.
__device__ __forceinline__ int xcd_remap(int b, int grid)
{
    const int per = grid >> 3;
    return (b & 7) * per + (b >> 3);
}

// Jacobi diagonal of a node from its bonds to -x, +x, -y, +y (and -z, +z),
// summed in this fixed order so that the pass and the refresh round it the
// same way.
template <typename T>
__device__ __forceinline__ T diag_sum(T gxm, T gxp, T gym, T gyp)
{
    return (gxm + gxp) + (gym + gyp);
}

template <typename T>
__device__ __forceinline__ T diag_sum(T gxm, T gxp, T gym, T gyp, T gzm, T gzp)
{
    return ((gxm + gxp) + (gym + gyp)) + (gzm + gzp);
}

// Jacobi scaling v / d. FP32: the hardware reciprocal (about 1 ulp, and a
// fixed function of d, so the preconditioner stays one fixed diagonal) in
// place of the much longer correctly rounded division; FP64: the division.
__device__ __forceinline__ float jscale(float v, float d) { return v * __builtin_amdgcn_rcpf(d); }
__device__ __forceinline__ double jscale(double v, double d) { return v / d; }

// M^-1 v at a node of diagonal d: v / d with the Jacobi preconditioner, v
// without one (then every use of d as the weight of M also becomes 1).
template <typename T>
__device__ __forceinline__ T apply_minv(T v, T d, bool jacobi) { return jacobi ? jscale(v, d) : v; }

// z - alpha u, z + beta p, the stencil's sums, the sums over nodes and r.z of
// the next pass with their roundings written out. Which product of a sum the
// compiler fuses is its own choice, made kernel by kernel; the pass kernels and
// the resident loop have to agree on every bit, so none is left to it.
__host__ __device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__host__ __device__ __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }

template <typename T>
__device__ __forceinline__ T step_z(T z, T alpha, T u) { return fma_(-alpha, u, z); }

template <typename T>
__device__ __forceinline__ T step_p(T z, T beta, T p) { return fma_(beta, p, z); }

// Which x bond's product is rounded before the others are added to it: the
// left one in FP64 and in the second segment of an FP32 row, else the right.
template <typename T>
__device__ __forceinline__ constexpr bool left_first(int segment) { return sizeof(T) == 8 || segment > 0; }

template <typename T>
__device__ __forceinline__ T stencil2d(bool left, T gxl, T dl, T gxr, T dr, T gyl, T db, T gyr, T da)
{
    T q = left ? fma_(gxr, dr, gxl * dl) : fma_(gxl, dl, gxr * dr);
    q = fma_(gyl, db, q);
    return fma_(gyr, da, q);
}

// In 3D: the left x bond's product first in FP64, the right one's in FP32.
template <typename T>
__device__ __forceinline__ T stencil3d(T gxl, T dl, T gxr, T dr, T gyl, T db, T gyr, T da, T gzl, T dn, T gzr, T du)
{
    T q = sizeof(T) == 8 ? fma_(gxr, dr, gxl * dl) : fma_(gxl, dl, gxr * dr);
    q = fma_(gyl, db, q);
    q = fma_(gyr, da, q);
    q = fma_(gzl, dn, q);
    return fma_(gzr, du, q);
}

// r.z of the next pass from this one's sums.
__host__ __device__ __forceinline__ double next_rz(double alpha, double zq, double qq, double rz)
{
    return fma_(alpha * alpha, qq, fma_(-2.0 * alpha, zq, rz));
}

// Scalar update after a CG pass. t = (p.q, z.q, q.D^-1 q, r.z, 0).
__host__ __device__ inline void step_after_cg(Scalars *s, const double *t)
{
    const double pq = t[0], zq = t[1], qq = t[2], rz = t[3];
    // a pass that left the FP64 field alone leaves the steps before it
    // pending; once kpend are pending the next CG pass adds them all
    const bool flushed = s->flush != 0;
    if (flushed) {
        s->alpha2 = s->alpha3 = s->alpha4 = 0.0;
        s->npend = 1;
    } else {
        s->alpha4 = s->alpha3;
        s->alpha3 = s->alpha2;
        s->alpha2 = s->alpha;
        s->npend += 1;
    }
    s->flush = s->npend >= s->kpend ? 1 : 0;
    s->passes += 1;
    s->iters += 1;
    s->rho = rz;
    s->rmax = fmax(s->rmax, sqrt(fmax(rz, 0.0)));
    if (!(rz > 0.0) && isfinite(rz)) {        // residual exactly zero: verify and stop
        s->alpha = 0.0;
        s->sigma_next = s->sigma;
        s->check = 1;
        s->mode = MODE_REFRESH;
        return;
    }
    if (!(pq > 0.0) || !isfinite(pq) || !isfinite(zq) || !isfinite(qq) || !isfinite(rz)) {
        s->status = -4;                       // breakdown: finish on the last good iterate
        s->stop = 1;
        s->alpha = 0.0;
        s->sigma_next = s->sigma;
        s->mode = MODE_REFRESH;
        return;
    }
    const double alpha = rz / pq;
    double rho_next = next_rz(alpha, zq, qq, rz);
    if (!(rho_next > 0.0)) rho_next = 0.0;
    const double est = s->kappa * s->sigma * sqrt(rho_next) / s->bhat;
    s->est_rel = est;
    s->alpha = alpha;
    const bool check = est <= s->tol || rho_next <= 0.0;
    const bool refresh = check || s->iters >= s->max_iter ||
                         (s->delta > 0.0 && sqrt(rho_next) <= s->delta * s->rmax);
    if (refresh) {
        s->check = check;
        s->est_check = est;
        s->sigma_next = s->sigma * sqrt(fmax(rho_next, rz * 1e-24));
        s->mode = MODE_REFRESH;
    } else {
        s->beta = rho_next / rz;
        s->mode = MODE_CG;
    }
}

// Scalar update after a refresh pass. t = (||r64||^2, r.D^-1 r of the stored residual, x.r64, Q_in, Q_out).
// s->first: 1 before the refresh that evaluates b, 2 before the one that
// evaluates the residual of the initial guess, 0 afterwards.
__device__ inline void step_after_refresh(Scalars *s, const double *t)
{
    const double rr64 = t[0], rrs = t[1];
    s->passes += 1;
    s->refreshes += 1;
    s->alpha2 = s->alpha3 = s->alpha4 = 0.0;     // the refresh applied every pending step
    s->flush = 0;
    s->npend = 1;                                // its own step is 0: counted as pending
    const double sigma_old = s->sigma;
    const double sigma = s->sigma_next;
    s->sigma = sigma;
    const int first = s->first;
    if (first == 1) {
        // this refresh evaluated b alone (the inflow at x = 0): fix the norms the
        // stopping rule and the estimates refer to, then evaluate the residual
        // of the initial guess (the linear profile along the flow axis)
        s->bnorm = sqrt(rr64);
        s->bhat = sigma * sqrt(rrs);
        s->kappa = 1.0;
        s->xr = t[2];
        s->Q_in = t[3];
        s->Q_out = t[4];
        if (!(s->bnorm > 0.0) || !isfinite(rr64) || !isfinite(rrs)) {
            if (s->bnorm == 0.0) s->converged = 1;      // nothing flows in
            else s->status = -4;
            s->rel_resid = s->est_rel = 0.0;
            s->mode = MODE_DONE;
        } else {
            s->first = 2;
            s->rel_resid = s->est_rel = 1.0;
            s->alpha = 0.0;
            s->sigma_next = sigma;
            s->mode = MODE_REFRESH;
        }
        s->check = 0;
        return;
    }
    const bool restart = first == 2;             // the first residual: start the recurrence
    s->first = 0;
    const double rel = s->bnorm > 0.0 ? sqrt(rr64) / s->bnorm : 0.0;
    const double srel = s->bhat > 0.0 ? sigma * sqrt(rrs) / s->bhat : 0.0;
    if (srel > 0.0 && rel > 0.0) s->kappa = rel / srel;
    s->rel_resid = rel;
    s->est_rel = rel;
    s->xr = t[2];
    s->Q_in = t[3];
    s->Q_out = t[4];
    if (s->stop) {
        s->mode = MODE_DONE;
    } else if (rel <= s->tol || s->bnorm == 0.0) {
        s->converged = 1;
        s->mode = MODE_DONE;
    } else if (s->iters >= s->max_iter) {
        s->status = -3;
        s->mode = MODE_DONE;
    } else if (!isfinite(rr64) || !isfinite(rrs)) {
        s->status = -4;
        s->mode = MODE_DONE;
    } else if (s->check && !(rel < 0.5 * s->last_check) && rel > 10.0 * s->est_check) {
        // the recurrence says converged, the true residual is far above it and
        // no longer halves between checks: its rounding floor is reached
        s->status = -3;
        s->mode = MODE_DONE;
    } else {
        if (s->check) s->last_check = rel;
        s->mode = MODE_CG;
        s->alpha = 0.0;
        s->beta = restart ? 0.0 : sigma * rrs / (sigma_old * s->rho);
        s->rmax = sqrt(rrs);
    }
    s->check = 0;
}

// The control block is read at the start of every pass by the threads that
// will need it at the end: thread t < kScalWords loads its 8-byte word into a
// register, so the last workgroup's scalar step runs on an LDS copy instead of
// waiting for a chain of memory round trips after the reduction.
constexpr int kScalWords = (int)(sizeof(Scalars) / 8);
static_assert(sizeof(Scalars) == 256 && kScalWords <= kBlock, "control block words: one 256-byte block per network");
constexpr int kModeWord = (int)(offsetof(Scalars, mode) / 8);
static_assert(offsetof(Scalars, mode) == 0, "mode is the low half of the first control block word");
constexpr int kPassesWord = (int)(offsetof(Scalars, passes) / 8);
static_assert(offsetof(Scalars, passes) % 8 == 0 && kModeWord != kPassesWord, "control block words");
constexpr int kLoopWord = (int)(offsetof(Scalars, loop_aborts) / 8);
static_assert(offsetof(Scalars, loop_aborts) % 8 == 0 && offsetof(Scalars, loop_failed) == offsetof(Scalars, loop_aborts) + 4,
              "the word of a resident loop's refusals and failures");

// Word t of the control block at the end of a resident loop, from the copy
// that the loop ran its steps on. The word of refusals and failures stays as
// it is: any workgroup may have given up a wait after the copy was made, and
// its flag has to reach the host.
__host__ __device__ inline void store_loop_end(unsigned long long *s, const volatile unsigned long long *copy, int t)
{
    if (t < kScalWords && t != kLoopWord) s[t] = copy[t];
}

__device__ __forceinline__ unsigned long long prefetch_scalars(const Scalars *s)
{
    const int t = threadIdx.x < kScalWords ? (int)threadIdx.x : 0;
    const unsigned long long v = reinterpret_cast<const unsigned long long *>(s)[t];
    return threadIdx.x < kScalWords ? v : 0ull;
}

// What one pass does with the direction and the FP64 field, from the control
// block: p1 holds p_{k-1}, whose step sa = sigma alpha is pending; p2, p3, p4
// hold p_{k-2}, p_{k-3}, p_{k-4}, whose steps sa2, sa3, sa4 are also pending
// while the CG passes after them left the field alone (a step not pending is
// 0; a CG pass with `flush` adds them all); p0 receives p_k. A network keeps
// up to kpend steps pending (4 for the FP32 passes, 2 for the FP64 ones,
// whose registers are scarcer) in kpend + 1 buffers.
template <typename T>
struct Step {
    const T *p1, *p2, *p3, *p4;
    T *p0;
    double sa, sa2, sa3, sa4;
    bool flush;
};

template <typename T>
__device__ __forceinline__ Step<T> make_step(const PassArgs<T> &a, const Scalars *s)
{
    // the buffer of pass c - d: constant divisors and conditional wraps, not
    // a 64-bit division by a runtime count at the start of every workgroup
    const int nb = a.npbuf;
    const int c = nb == 5 ? (int)(s->passes % 5) : (int)(s->passes % 3);
    auto back = [&](int d) {
        int v = c - d;
        if (v < 0) v += nb;
        if (v < 0) v += nb;
        return v;
    };
    Step<T> k;
    k.p0 = a.pbuf[c];
    k.p1 = a.pbuf[back(1)];
    k.p2 = a.pbuf[back(2)];
    k.p3 = a.pbuf[back(3)];
    k.p4 = a.pbuf[back(4)];
    k.sa = s->sigma * s->alpha;
    k.sa2 = s->sigma * s->alpha2;
    k.sa3 = s->sigma * s->alpha3;
    k.sa4 = s->sigma * s->alpha4;
    k.flush = s->flush != 0;
    return k;
}

// FP64 field with the pending steps added, oldest first (the order in which
// one step per pass would have added them).
__device__ __forceinline__ double with_steps(double P, double sa2, double p2, double sa, double p1)
{
    double v = P;
    if (sa2 != 0.0) v = fma(sa2, p2, v);
    if (sa != 0.0) v = fma(sa, p1, v);
    return v;
}

// Tiles of the 2D kernels.
// SHAPE 0: the tile for networks with enough tiles to fill the chip; SHAPE 1:
// a quarter-size tile (one segment, half the rows) for smaller networks,
// which would otherwise leave most CUs with one or two workgroups.
template <typename T, int SHAPE>
struct Tile2D {
    static constexpr int TY = SHAPE == 0 ? (sizeof(T) == 4 ? kTY2f : kTY2d)           // rows per wave
                                         : (sizeof(T) == 4 ? kTY2fS : kTY2dS);
    static constexpr int SEG = SHAPE == 0 ? (sizeof(T) == 4 ? kSEG2f : kSEG2d) : 1;   // 64-column segments per row
    static constexpr int ROWS = TY * (kBlock / kWave);                                // rows per workgroup
    static constexpr int COLS = kWave * SEG;                                          // columns per workgroup
};

// Rows of a 3D tile that a thread holds (its wave covers kRows of the kTY rows).
constexpr int kRows = kTY / (kBlock / kWave);

// Bound of a wait inside a kernel: 2 s of the 100 MHz s_memrealtime clock.
constexpr uint64_t kSpinTicks = 200000000ull;

// A wave-uniform value made scalar (SGPRs), so that branches on it stay uniform.
__device__ __forceinline__ int rfl(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t rfl(int64_t v)
{
    const uint32_t lo = (uint32_t)rfl((int)(uint32_t)v), hi = (uint32_t)rfl((int)(uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double rfl(double v) { return __longlong_as_double(rfl((int64_t)__double_as_longlong(v))); }

}  // namespace rn
