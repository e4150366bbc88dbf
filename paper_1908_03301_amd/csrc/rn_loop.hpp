// rn_loop.hpp -- the CG loop of one network with its state on the chip.
//
// A pass kernel reads and writes the CG state once per iteration and ends
// with a chain of dependent round trips: stores, ticket, partial sums, scalar
// step, kernel end, next launch, control block, tile loads. Below a few
// million nodes that chain is the iteration, not the bytes (7 us at 128^2, of
// which the tile's own arithmetic is under 1 us). Here one launch runs many
// CG passes of one network. Every workgroup keeps its tile's z, u, p and FP64
// field in registers and LDS, and its bonds too where there is room; per pass it
// sends out only the u of its edge nodes and its four partial sums:
//   - a neighbour keeps z and p of its halo nodes itself, from the same
//     arithmetic as their owner, so u is the only value a halo node needs;
//   - up to kDirect workgroups, each sums everyone's partials in the order of
//     the pass kernels and runs the scalar step itself: one exchange per pass.
//     More of them polling all sums would crowd out the sums themselves (512
//     workgroups waited 8.5 us for them, 128 waited 4), so there workgroup 0
//     sums, runs the step and sends the coefficients out.
// Values travel with a pass number (tag) in the same 8-byte word, edge nodes
// packed per tile (a store per node where they lie cost 3 us a pass), so no
// flag, counter or fence is waited for: a reader polls the word itself. Two
// slots alternate: whoever writes pass k + 2 has seen the coefficients of pass
// k + 1, for which everyone has posted sums, having read pass k before. The
// sums are bare doubles in four slots: an empty word (all bits set, a NaN no
// arithmetic here produces) stands until the sum arrives. Having posted pass
// k, a workgroup empties its words of slot k + 2: everyone has read pass k - 2,
// which it held, and the emptying is complete (s_waitcnt, a whole pass later)
// before it posts pass k + 1, so nobody polls the slot for pass k + 2 before.
//
// The workgroups of a small 2D network all run on one XCD (LOCAL): eight times as many
// are launched, those there claim their place, the others leave.
// Every word then stays in that XCD's L2: stores need not go through to memory
// (plain ones reach the L2; loads are device-scope, since a CU's L1 may hold a
// line another CU has since written). One workgroup per CU gains (128^2 mixed,
// 32 of them: 3.13 -> 2.69 us a pass), two do not (64: 3.1 both ways), and four
// crowd the L2 with their looks (128: 3.7 -> 4.8).
//
// All workgroups have to run at once. They are admitted by a gate: each counts
// itself in, and the launch goes ahead only if all arrive in time; otherwise
// they move z and u to the parity of the next round, change nothing else, and
// the host goes on with one launch per pass. In a LOCAL launch that does not
// depend on who got a place, since the dispatcher need not have dealt its
// workgroups evenly to the XCDs (a stream with a CU mask, another partition
// mode): the first one waits for the gate's answer wherever it is and moves all.
// Behind the gate every wait is bounded too (kSpinTicks).
//
// The arithmetic and its order are those of the pass kernels (tile by tile,
// the same reduction tree), so results are the same bits.
#pragma once

#include "rn_cg.hpp"

#include <algorithm>
#include <mutex>

namespace rn {
namespace {

constexpr uint64_t kGateTicks = 50000ull;        // 0.5 ms: longer than any launch takes to start
constexpr unsigned kGateGo = 1u, kGateNo = 2u;
constexpr int kDirect = 64;                      // workgroups up to which each sums for itself
constexpr int kPerGroup = 2;                     // most workgroups of the pass kernels that one here stands for
constexpr int kCopies = 32;                      // copies of the coefficients, 64 bytes each
typedef unsigned long long u64;
constexpr u64 kEmpty = ~0ull;

__device__ __forceinline__ u64 word_load(const u64 *p)
{
    return __hip_atomic_load((const RN_GLOBAL u64 *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <bool LOCAL>
__device__ __forceinline__ void word_store(u64 *p, u64 v)
{
    __hip_atomic_store((RN_GLOBAL u64 *)p, v, __ATOMIC_RELAXED,
                       LOCAL ? __HIP_MEMORY_SCOPE_WORKGROUP : __HIP_MEMORY_SCOPE_AGENT);
}

// the same at a byte offset of the lane's own from an address all lanes share
__device__ __forceinline__ u64 *at(u64 *base, unsigned off)
{
    return reinterpret_cast<u64 *>(reinterpret_cast<char *>(base) + off);
}

__device__ __forceinline__ u64 tagged(unsigned tag, unsigned v) { return ((u64)tag << 32) | v; }

// A value in the exchange: one tagged word (float) or two, `half` words apart
// (the halves of a double).
template <typename T> struct Packed;
template <> struct Packed<float> {
    u64 a;
    template <bool LOCAL>
    __device__ __forceinline__ static void post(u64 *p, int half, unsigned tag, float v)
    {
        (void)half;
        word_store<LOCAL>(p, tagged(tag, __builtin_bit_cast(unsigned, v)));
    }
    __device__ __forceinline__ void look(const u64 *p, int half)
    {
        (void)half;
        a = word_load(p);
    }
    __device__ __forceinline__ void zero(unsigned tag) { a = tagged(tag, 0u); }
    __device__ __forceinline__ bool here(unsigned tag) const { return (unsigned)(a >> 32) == tag; }
    __device__ __forceinline__ float value() const { return __builtin_bit_cast(float, (unsigned)a); }
};
template <> struct Packed<double> {
    u64 a, b;
    template <bool LOCAL>
    __device__ __forceinline__ static void post(u64 *p, int half, unsigned tag, double v)
    {
        const u64 w = __builtin_bit_cast(u64, v);
        word_store<LOCAL>(p, tagged(tag, (unsigned)w));
        word_store<LOCAL>(p + half, tagged(tag, (unsigned)(w >> 32)));
    }
    __device__ __forceinline__ void look(const u64 *p, int half)
    {
        a = word_load(p);
        b = word_load(p + half);
    }
    __device__ __forceinline__ void zero(unsigned tag) { a = b = tagged(tag, 0u); }
    __device__ __forceinline__ bool here(unsigned tag) const
    {
        return (unsigned)(a >> 32) == tag && (unsigned)(b >> 32) == tag;
    }
    __device__ __forceinline__ double value() const { return __builtin_bit_cast(double, (b << 32) | (a & 0xffffffffull)); }
};

// A bounded wait: more() is called after a look that found nothing.
struct Spin {
    unsigned *failed;
    uint64_t t0 = 0;
    unsigned n = 0;
    bool ok = true;
    __device__ explicit Spin(Scalars *s) : failed(&s->loop_failed) {}
    __device__ __forceinline__ bool more()
    {
        if ((++n & 255u) == 0) {
            const uint64_t now = __builtin_amdgcn_s_memrealtime();
            if (t0 == 0) t0 = now;
            if (__hip_atomic_load(failed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                ok = false;
            } else if (now - t0 > kSpinTicks) {
                __hip_atomic_store(failed, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                ok = false;
            }
        }
        return ok;
    }
};

// Thread 0: learn whether the launch goes ahead. A workgroup with a place
// counts itself in; `places` of them open the gate.
__device__ __forceinline__ int pass_gate(unsigned *gate, bool has_place, unsigned places, Scalars *s)
{
    unsigned state = 0;
    if (has_place &&
        __hip_atomic_fetch_add(gate, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == places - 1u) {
        unsigned expected = 0u;
        __hip_atomic_compare_exchange_strong(gate + 1, &expected, kGateGo, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
        state = expected ? expected : kGateGo;
    }
    const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
    while (!state) {
        if (!has_place) __builtin_amdgcn_s_sleep(127);   // 3 us: nobody waits for this one
        state = __hip_atomic_load(gate + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (!state && __builtin_amdgcn_s_memrealtime() - t0 > kGateTicks) {
            unsigned expected = 0u;
            if (__hip_atomic_compare_exchange_strong(gate + 1, &expected, kGateNo, __ATOMIC_RELAXED,
                                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                __hip_atomic_fetch_add(&s->loop_aborts, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                state = kGateNo;
            } else {
                state = expected;
            }
        }
    }
    return state == kGateGo;
}

// This workgroup's network and its place in it (negative, or past the network's
// workgroups: none). One workgroup is launched per place, or
// (LOCAL) per place and XCD, those on XCD 0 claiming one. r: the launch's
// arguments, made this network's.
struct Place {
    int slot, lb;
};

template <bool LOCAL>
__device__ __forceinline__ Place loop_place(LoopArgs &r, int slot)
{
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < 3 * kLoopMembers; i += kBlock) r.gate_clear[i / 3 * kLoopGateWords + i % 3] = 0u;
    Place p = {slot, (int)blockIdx.x};
    if constexpr (LOCAL) {
        __shared__ int place;
        if (__builtin_amdgcn_readfirstlane(__builtin_amdgcn_s_getreg((3 << 11) | (0 << 6) | 20)) & 7) return {slot, -1};   // XCC_ID
        if (threadIdx.x == 0)
            place = (int)__hip_atomic_fetch_add(r.gate + 2, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        p.lb = __builtin_amdgcn_readfirstlane(place);
    } else if (r.blk) {
        const uint2 e = r.blk[blockIdx.x];
        const unsigned m = e.y >> 16;
        p.slot = (int)e.x;
        p.lb = (int)(e.y & 0xffffu);
        r.gate += m * kLoopGateWords;
        r.coef += m * (kLoopCoefBytes / sizeof(u64));
        r.part += r.net[m].block0 * (kLoopSlots * kLoopRed);
        r.xch += r.net[m].xch;
    }
    return p;
}

// LDS of the loop's control, the same for every tile family.
struct LoopShared {
    double red[kPerGroup][kBlock / kWave][kLoopRed], tot[kBlock / kWave][kLoopRed];
    Scalars sl[kBlock / kWave];
    int go;
};

// The coefficients of the next pass, uniform over the wave.
struct LoopState {
    double alpha, beta, sa;
};

// The gate's answer for the whole workgroup. A network that was turned away
// once is turned away at once by the loops launched before the host knew.
__device__ __forceinline__ bool loop_gate(LoopShared &sh, bool has_place, int places, Scalars *s, const Scalars *copy,
                                          const LoopArgs &r)
{
    if (threadIdx.x == 0) sh.go = copy->loop_aborts ? 0 : pass_gate(r.gate, has_place, (unsigned)places, s);
    __syncthreads();
    return sh.go != 0;
}

// Emptied sums, the control block's copies, the gate. Returns whether the
// launch goes ahead.
template <bool LOCAL>
__device__ __forceinline__ bool loop_begin(LoopShared &sh, LoopState &L, Scalars *s, const LoopArgs &r,
                                           const int *lbs, int nlb, int grid)
{
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    u64 *part = reinterpret_cast<u64 *>(r.part);
    if (threadIdx.x < kLoopRed)
        for (int l = 0; l < nlb && lbs[l] < grid; ++l)
            for (int q = 0; q < kLoopSlots; ++q)
                word_store<LOCAL>(part + (q * kLoopRed + threadIdx.x) * grid + lbs[l], kEmpty);
    if (lane < kScalWords)
        reinterpret_cast<u64 *>(&sh.sl[w])[lane] = reinterpret_cast<const u64 *>(s)[lane];
    L.alpha = s->alpha;
    L.beta = s->beta;
    L.sa = s->sigma * s->alpha;
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    return loop_gate(sh, true, 8 * div_up(grid >> 3, nlb), s, &sh.sl[0], r);
}

// The four sums of a workgroup of the pass kernels, as in finish_pass: thread
// sums and waves here, waves in order in post_sums.
__device__ __forceinline__ void wave_sums(double (&red)[kBlock / kWave][kLoopRed], const double (&acc)[kLoopRed])
{
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
#pragma unroll
    for (int k = 0; k < kLoopRed; ++k) {
        const double v = wave_sum(acc[k]);
        if (lane == 0) red[w][k] = v;
    }
}

// Its sums into pass `it`'s slot, and the slot after next emptied. Wave 0 has
// waited (s_waitcnt) for what it emptied in the pass before.
template <bool LOCAL, int NLB>
__device__ __forceinline__ void post_sums(LoopShared &sh, const LoopArgs &r, int it, const int (&lbs)[NLB], int grid)
{
    __syncthreads();
    if (threadIdx.x < kLoopRed) {
#pragma unroll
        for (int l = 0; l < NLB; ++l) {
            if (lbs[l] >= grid) continue;        // uniform
            u64 *part = reinterpret_cast<u64 *>(r.part) + threadIdx.x * grid + lbs[l];
            double v = 0.0;
#pragma unroll
            for (int ww = 0; ww < kBlock / kWave; ++ww) v += sh.red[l][ww][threadIdx.x];
            u64 b = __builtin_bit_cast(u64, v);
            if (b == kEmpty) b ^= 1;             // still a NaN
            word_store<LOCAL>(part + (it & (kLoopSlots - 1)) * (kLoopRed * grid), b);
            if (it > 0) word_store<LOCAL>(part + ((it + 2) & (kLoopSlots - 1)) * (kLoopRed * grid), kEmpty);
        }
    }
}

// Everyone's sums: thread t adds blocks t, t + kBlock, ... in order, then
// lanes and waves as in finish_pass. A look loads all words of AHEAD blocks at
// once, so a word that arrives late costs one round trip however many were
// missing.
template <int AHEAD>
__device__ __forceinline__ void take_blocks(double (&t)[kLoopRed], const u64 *part, int grid, Spin &spin)
{
    for (int b0 = threadIdx.x; b0 < grid; b0 += AHEAD * kBlock) {
        u64 v[AHEAD][kLoopRed];
        bool missing;
        do {
            missing = false;
#pragma unroll
            for (int h = 0; h < AHEAD; ++h)
#pragma unroll
                for (int k = 0; k < kLoopRed; ++k) {
                    const int b = b0 + h * kBlock;
                    v[h][k] = word_load(part + k * grid + (b < grid ? b : b0));
                }
#pragma unroll
            for (int h = 0; h < AHEAD; ++h)
#pragma unroll
                for (int k = 0; k < kLoopRed; ++k) missing |= v[h][k] == kEmpty;
        } while (missing && spin.more());
#pragma unroll
        for (int h = 0; h < AHEAD; ++h)
            if (h == 0 || b0 + h * kBlock < grid)
#pragma unroll
                for (int k = 0; k < kLoopRed; ++k) t[k] += __builtin_bit_cast(double, v[h][k]);
    }
}

__device__ __forceinline__ void take_sums(LoopShared &sh, double (&t)[kRed], const LoopArgs &r, int it, int grid,
                                          Spin &spin)
{
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const u64 *part = reinterpret_cast<const u64 *>(r.part) + (it & (kLoopSlots - 1)) * (kLoopRed * grid);
    double v[kLoopRed] = {0.0, 0.0, 0.0, 0.0};
    if (w * kWave < grid) {                       // wave-uniform: waves past the grid hold zeros
        if (grid <= kBlock) take_blocks<1>(v, part, grid, spin);
        else take_blocks<2>(v, part, grid, spin);
#pragma unroll
        for (int k = 0; k < kLoopRed; ++k) v[k] = wave_sum(v[k]);
    }
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < kLoopRed; ++k) sh.tot[w][k] = v[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kRed; ++k) {
        t[k] = 0.0;
        if (k < kLoopRed)
#pragma unroll
            for (int ww = 0; ww < kBlock / kWave; ++ww) t[k] += sh.tot[ww][k];
    }
}

// The scalar step of a pass from its sums: step_after_cg in straight-line
// code while the recurrence goes on. The pass that ends the loop (a refresh is
// due, a breakdown, the launch's limit) runs step_after_cg itself. `sl` is this
// wave's copy of the control block; its pass counts are those of the start
// until then. Every pass of the loop adds every pending step to the field, so
// it counts as one that flushes. Returns whether the loop goes on.
__device__ __forceinline__ bool loop_step(Scalars *sl, LoopState &L, const double (&t)[kRed], int it, int limit)
{
    const double pq = t[0], zq = t[1], qq = t[2], rz = t[3];
    const double root = sqrt(fmax(rz, 0.0));
    const double alpha = rz / pq;
    double rho = next_rz(alpha, zq, qq, rz);
    if (!(rho > 0.0)) rho = 0.0;
    const double rmax = fmax(sl->rmax, root);
    const double rroot = sqrt(rho);
    const double beta = rho / rz;
    const double est = sl->kappa * sl->sigma * rroot / sl->bhat;
    const bool fine = rz > 0.0 && pq > 0.0 && isfinite(rz) && isfinite(pq) && isfinite(zq) && isfinite(qq);
    const bool refresh = est <= sl->tol || rho <= 0.0 || sl->iters + it + 1 >= sl->max_iter ||
                         (sl->delta > 0.0 && rroot <= sl->delta * rmax);
    const bool on = fine && !refresh && it + 1 < limit;
    L.sa = sl->sigma * alpha;
    L.alpha = alpha;
    L.beta = beta;
    if ((threadIdx.x & (kWave - 1)) == 0) {
        if (on) {
            sl->rmax = rmax;
            sl->est_rel = est;
            sl->alpha = alpha;
            sl->beta = beta;
        } else {
            sl->passes += it;
            sl->iters += it;
            sl->flush = 1;
            step_after_cg(sl, t);
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    return on;
}

// Behind the sums: the coefficients of the next pass and whether there is one.
// With few workgroups each wave forms them; else workgroup 0 does and the
// others' waves read one of its copies: words 0..5 the halves of alpha, beta
// and sigma alpha, word 6 whether the loop ends.
template <bool LOCAL>
__device__ __forceinline__ bool loop_turn(LoopShared &sh, LoopState &L, const LoopArgs &r, int it, int lb, int grid,
                                          Spin &spin)
{
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const unsigned tag = r.tag0 + (unsigned)it;
    if (LOCAL || grid <= kDirect || lb == 0) {
        double t[kRed];
        take_sums(sh, t, r, it, grid, spin);
        const bool on = rfl((int)loop_step(&sh.sl[w], L, t, it, r.limit)) != 0;
        if (!LOCAL && grid > kDirect) {
            const int word = lane & 7;
            const double d = word < 2 ? L.alpha : (word < 4 ? L.beta : L.sa);
            const u64 b = __builtin_bit_cast(u64, d);
            const unsigned half = word >= 6 ? (unsigned)!on : (unsigned)((word & 1) ? b >> 32 : b);
            word_store<LOCAL>(r.coef + (w * 8 + (lane >> 3)) * 8 + word, tagged(tag, half));
        }
        return on;
    }
    const u64 *c = r.coef + (lb & (kCopies - 1)) * 8 + (lane & 7);
    u64 v;
    do v = word_load(c);
    while (__ballot((unsigned)(v >> 32) != tag) != 0ull && spin.more());
    const int half = (int)(unsigned)v;
    auto get = [&](int k) {
        const unsigned lo = (unsigned)__builtin_amdgcn_readlane(half, 2 * k),
                       hi = (unsigned)__builtin_amdgcn_readlane(half, 2 * k + 1);
        return __builtin_bit_cast(double, ((u64)hi << 32) | lo);
    };
    L.alpha = get(0);
    L.beta = get(1);
    L.sa = get(2);
    return __builtin_amdgcn_readlane(half, 6) == 0;
}

// Loads and stores at a 32-bit index: a network that fits the chip has its
// arrays in a few tens of MB, and an offset from a base in scalar registers
// takes one vector register where an address takes two.
template <typename T>
__device__ __forceinline__ T ldi(const T *base, int i)
{
    return *reinterpret_cast<const RN_GLOBAL T *>((const RN_GLOBAL char *)base + (unsigned)i * (unsigned)sizeof(T));
}
template <typename T>
__device__ __forceinline__ void sti(T *base, int i, T v)
{
    *reinterpret_cast<RN_GLOBAL T *>((RN_GLOBAL char *)base + (unsigned)i * (unsigned)sizeof(T)) = v;
}

// A LOCAL launch that was turned away: one workgroup moves z and u (at most
// 16,384 nodes) to the parity that the next round reads.
template <typename T>
__device__ __forceinline__ void move_state(const PassArgs<T> &a)
{
    const int n = a.nx * a.ny * a.nz;
    for (int i = (int)threadIdx.x; i < n; i += kBlock) {
        sti(a.dst.z, i, ldi(a.src.z, i));
        sti(a.dst.u, i, ldi(a.src.u, i));
    }
}

// hide(v): the compiler may not carry anything computed from v across passes.
// Left to itself it keeps every invariant of the loop (diagonals, shifted
// bonds, addresses, lane masks) in registers and spills the state instead.
template <typename V>
__device__ __forceinline__ void hide(V &v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void hide_s(int &v) { asm volatile("" : "+s"(v)); }

// ---------------------------------------------------------------- 2D
// The tile of pass2d_kernel (Tile2D), TPW of them per workgroup of that kernel,
// LB such workgroups to one here: thread, row and segment hold the same nodes. Slots past a periodic edge hold the image
// of the opposite edge; their u comes from the owner like a halo node's.
// The FP64 field of the full tile sits in LDS (one word per node and thread,
// touched once per pass), which leaves the registers of four waves per SIMD to
// the rest of the state. Networks with two tiles per workgroup fill the chip
// (2048^2 mixed: 2,048 tiles): half as many workgroups of four tiles run at two
// waves per SIMD, where the registers that every thread needs besides its
// state are paid for half as often (at four waves 86 of them spilled, and a
// pass took 32 us instead of the pass kernel's 34). Their bonds come from
// memory in every pass, 8 bytes of the plain pass's 39 per node and mostly from
// the L2; the first tile's are on their way while the pass before waits.
// Exchange words of a tile: its first row, last row, first column, last column.
template <typename T, int SHAPE>
constexpr int edge_words2d() { return 2 * (Tile2D<T, SHAPE>::COLS + Tile2D<T, SHAPE>::ROWS); }

template <typename T, int SHAPE, int TPW, bool LOCAL, int LB>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(LB > 1 ? 2 : 4))) void loop2d_kernel(
    const PassArgs<T> *__restrict__ tab, Scalars *scal, int parity, int slot, LoopArgs r)
{
    constexpr int TY = Tile2D<T, SHAPE>::TY, SEG = Tile2D<T, SHAPE>::SEG, NW = kBlock / kWave;
    constexpr int ROWS = Tile2D<T, SHAPE>::ROWS, COLS = Tile2D<T, SHAPE>::COLS;
    constexpr int E = edge_words2d<T, SHAPE>(), EW = E * (int)(sizeof(T) / 4);   // values, words of a tile
    constexpr int kTop = 0, kBottom = COLS, kLeft = 2 * COLS, kRight = 2 * COLS + ROWS;
    constexpr bool kTight = SHAPE == 0;           // many nodes per thread: registers are scarce
    constexpr bool kFieldLds = kTight;
    constexpr bool kLean = TPW > 1;               // bonds from memory, halo addresses formed anew
    constexpr int NT = TPW * LB;                  // tiles of this workgroup
    __shared__ T edge[2][NW][SEG][kWave];         // [0]: first row of each wave, [1]: last row
    __shared__ LoopShared sh;
    __shared__ double fl[kFieldLds ? NT * SEG * TY : 1][kBlock];
    const Place at_ = loop_place<LOCAL>(r, slot);
    const PassArgs<T> &a = tab[2 * at_.slot + parity];
    Scalars *s = scal + at_.slot;
    const int grid = a.grid, lb = at_.lb;
    if constexpr (LOCAL) {
        if (s->mode != MODE_CG) return;
        if (__builtin_expect(lb < 0 || lb >= grid, 0)) {                // no place
            if (blockIdx.x == 0 && !loop_gate(sh, false, grid, s, s, r)) move_state(a);
            return;
        }
    } else if (lb >= grid || s->mode != MODE_CG) {
        return;
    }
    int lane = threadIdx.x & (kWave - 1);
    const int w = rfl((int)threadIdx.x / kWave);
    // workgroups of the pass kernel that this one stands for, all of its XCD
    int lbs[LB];
#pragma unroll
    for (int l = 0; l < LB; ++l) lbs[l] = LB == 1 ? lb : (lb & 7) + 8 * ((lb >> 3) * LB + l);
    auto tile_of = [&](int t) {
        const int b = lbs[t / TPW];
        return b < grid ? xcd_remap(b, grid) + t % TPW * grid : a.ntiles;
    };
    const int nx = a.nx, ny = a.ny, ntx = a.ntx, nty = a.nty, wrap = a.wrap;
    const bool wx = wrap & 1, wy = (wrap >> 1) & 1;
    const bool jacobi = a.jacobi != 0, xaxis = a.axis == 0;
    const Step<T> k0 = make_step(a, s);
    const int64_t passes0 = s->passes;
    double *__restrict__ P = a.P[s->refreshes & 1];
    auto colm = [&](int xx) { return xx >= 0 && xx < nx ? xx : (wx && xx == nx ? 0 : (wx && xx == -1 ? nx - 1 : -1)); };
    auto rowm = [&](int yy) { return yy >= 0 && yy < ny ? yy : (wy && yy == ny ? 0 : (wy && yy == -1 ? ny - 1 : -1)); };

    // ---- state of the tiles
    T z_[NT][SEG][TY], u_[NT][SEG][TY], p_[NT][SEG][TY], gxv[NT][SEG][TY], gyv[NT][SEG][TY + 1];
    double Pv[kFieldLds ? 1 : NT][SEG][TY];
    T ez[NT][SEG], eu[NT][SEG], ep[NT][SEG];    // halo row of the first / last wave
    T hz[NT], hu[NT], hp[NT], hg[NT];        // halo column node of this lane
    unsigned liv = 0;                              // bits (tile, segment, row): interior nodes of the lattice
    int tx_[NT], ty_[NT];                        // tile coordinates; past the lattice: no tile
    auto bit = [&](int t, int sg, int j) { return 1u << ((t * SEG + sg) * TY + j); };
    auto colx = [&](int t, int sg) { return tx_[t] * COLS + kWave * sg + lane; };
    auto rowy = [&](int t, int j) { return ty_[t] * ROWS + w * TY + j; };
    // halo column lanes: row y0 + hrow() at x0 - 1 (left) or x0 + COLS (right)
    auto hleft = [&] { return lane < TY; };
    auto hrow = [&] { return hleft() ? lane : lane - (kWave - TY); };
    // the row of halo nodes this wave keeps: above the tile (first wave), below it (last wave)
    auto halo_y = [&](int t) { return w == 0 ? rowm(ty_[t] * ROWS - 1) : (w == NW - 1 ? rowm(ty_[t] * ROWS + ROWS) : -1); };
    auto halo_x = [&](int t) {
        return (hleft() || lane >= kWave - TY) && rowy(t, hrow()) < ny ? colm(hleft() ? tx_[t] * COLS - 1 : tx_[t] * COLS + COLS) : -1;
    };
    // bonds of tile t: right and upper of the nodes (0 where a slot holds none
    // is the arrays' own doing inside the lattice; elsewhere they are not
    // used), below the wave (none at y = 0 unless y wraps: then ny-1 -> 0) and
    // left of the tile
    auto load_bonds = [&](int t) {
#pragma unroll
        for (int sg = 0; sg < SEG; ++sg) {
            const int xm = colm(colx(t, sg)), xc = xm >= 0 ? xm : 0;
#pragma unroll
            for (int j = 0; j < TY; ++j) {
                const int ym = rowm(rowy(t, j));
                const int i = (ym >= 0 ? ym : 0) * nx + xc;
                gxv[t][sg][j] = ldi(a.gT[0], i);
                gyv[t][sg][j + 1] = ldi(a.gT[1], i);
            }
            const int ym = rowm(rowy(t, 0) - 1);
            const T gb = ldi(a.gT[1], (ym >= 0 ? ym : 0) * nx + xc);
            gyv[t][sg][0] = ym >= 0 ? gb : T(0);
        }
        const int hx = halo_x(t);
        const T g0 = ldi(a.gT[0], (hx >= 0 ? rowy(t, hrow()) * nx + hx : 0));
        hg[t] = hx >= 0 && hleft() ? g0 : T(0);
    };
    // where the halo's words lie in an exchange slot (bytes; kNone: no node):
    // the neighbour above shows its last row, the one below its first
    constexpr unsigned kNone = ~0u;
    auto row_words = [&](int t, int sg) {
        if (halo_y(t) < 0 || colx(t, sg) >= nx) return kNone;
        const int ey = w == 0 ? (ty_[t] > 0 ? ty_[t] : nty) - 1 : (ty_[t] + 1 < nty ? ty_[t] + 1 : 0);
        return (unsigned)((ey * ntx + tx_[t]) * EW + (w == 0 ? kBottom : kTop) + kWave * sg + lane) * 8u;
    };
    auto col_words = [&](int t) {
        if (halo_x(t) < 0) return kNone;
        const int ex = hleft() ? (tx_[t] > 0 ? tx_[t] : ntx) - 1 : (tx_[t] + 1 < ntx ? tx_[t] + 1 : 0);
        return (unsigned)((ty_[t] * ntx + ex) * EW + (hleft() ? kRight : kLeft) + w * TY + hrow()) * 8u;
    };
    unsigned ro[NT][SEG], co[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int tile = tile_of(t);
        const bool has = tile < a.ntiles;
        tx_[t] = has ? tile % ntx : ntx + 1;
        ty_[t] = has ? tile / ntx : nty + 1;
#pragma unroll
        for (int sg = 0; sg < SEG; ++sg) {
            const int x = colx(t, sg), xm = colm(x);
#pragma unroll
            for (int j = 0; j < TY; ++j) {
                const int yy = rowy(t, j), ym = rowm(yy);
                const bool held = xm >= 0 && ym >= 0;
                const int i = held ? ym * nx + xm : 0;
                const T z0 = ldi(a.src.z, i), u0 = ldi(a.src.u, i), p0 = ldi(k0.p1, i);
                double v = ldi((const double *)P, i);
                if (k0.sa3 != 0.0 || k0.sa4 != 0.0)
                    v = with_steps(v, k0.sa4, (double)ldi(k0.p4, i), k0.sa3, (double)ldi(k0.p3, i));
                if (k0.sa2 != 0.0) v = with_steps(v, k0.sa2, (double)ldi(k0.p2, i), 0.0, 0.0);
                z_[t][sg][j] = held ? z0 : T(0);
                u_[t][sg][j] = held ? u0 : T(0);
                p_[t][sg][j] = held ? p0 : T(0);
                if constexpr (kFieldLds) fl[(t * SEG + sg) * TY + j][threadIdx.x] = v;
                else Pv[t][sg][j] = v;
                const bool face = xaxis ? (x == 0 || x == nx - 1) : (yy == 0 || yy == ny - 1);
                if (x < nx && yy < ny && !face) liv |= bit(t, sg, j);
            }
            const int yh = halo_y(t);
            const bool hok = x < nx && yh >= 0;
            const int ri = hok ? yh * nx + x : 0;
            const T z0 = ldi(a.src.z, ri), u0 = ldi(a.src.u, ri), p0 = ldi(k0.p1, ri);
            ez[t][sg] = hok ? z0 : T(0);
            eu[t][sg] = hok ? u0 : T(0);
            ep[t][sg] = hok ? p0 : T(0);
        }
        const int hx = halo_x(t);
        const bool hok = hx >= 0;
        const int ci = hok ? rowy(t, hrow()) * nx + hx : 0;
        const T z0 = ldi(a.src.z, ci), u0 = ldi(a.src.u, ci), p0 = ldi(k0.p1, ci);
        hz[t] = hok ? z0 : T(0);
        hu[t] = hok ? u0 : T(0);
        hp[t] = hok ? p0 : T(0);
        if (!kLean || t == 0) load_bonds(t);
        if constexpr (!kLean) {
#pragma unroll
            for (int sg = 0; sg < SEG; ++sg) ro[t][sg] = row_words(t, sg);
            co[t] = col_words(t);
        }
    }
    LoopState L;
    const bool admitted = loop_begin<LOCAL>(sh, L, s, r, lbs, LB, grid);

    int it = 0;
    for (bool on = __builtin_expect(admitted, 1); on; ++it) {
        Spin spin(s);
        const T alpha = (T)rfl(L.alpha), beta = (T)rfl(L.beta);
        const double sa = rfl(L.sa);
        const unsigned tag = r.tag0 + (unsigned)it;
        u64 *xb = r.xch + (size_t)(it & 1) * r.xch_slot;     // this pass's edge values
        if constexpr (kTight) {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
#pragma unroll
                for (int sg = 0; !kLean && sg < SEG; ++sg) {
#pragma unroll
                    for (int j = 0; j < TY; ++j) {
                        hide(gxv[t][sg][j]);
                        hide(gyv[t][sg][j + 1]);
                    }
                    hide(gyv[t][sg][0]);
                }
                if constexpr (!kLean) hide(hg[t]);
                hide_s(tx_[t]);
                hide_s(ty_[t]);
            }
            hide(liv);
            hide(lane);
        }
        // z' and p' of the halo
#pragma unroll
        for (int t = 0; t < NT; ++t) {
#pragma unroll
            for (int sg = 0; sg < SEG; ++sg) {
                ez[t][sg] = step_z(ez[t][sg], alpha, eu[t][sg]);
                ep[t][sg] = step_p(ez[t][sg], beta, ep[t][sg]);
            }
            hz[t] = step_z(hz[t], alpha, hu[t]);
            hp[t] = step_p(hz[t], beta, hp[t]);
        }
        // the pending step, then z' and p' of the tiles: after this u is free
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int sg = 0; sg < SEG; ++sg) {
#pragma unroll
                for (int j = 0; j < TY; ++j) {
                    if (sa != 0.0) {
                        if constexpr (kFieldLds) {
                            double &f = fl[(t * SEG + sg) * TY + j][threadIdx.x];
                            f = fma(sa, (double)p_[t][sg][j], f);
                        } else {
                            Pv[t][sg][j] = fma(sa, (double)p_[t][sg][j], Pv[t][sg][j]);
                        }
                    }
                    const T zc = step_z(z_[t][sg][j], alpha, u_[t][sg][j]);
                    z_[t][sg][j] = zc;
                    p_[t][sg][j] = step_p(zc, beta, p_[t][sg][j]);
                }
                if constexpr (kTight) __builtin_amdgcn_sched_barrier(0);
            }
        double acc[kLoopRed];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            if (t % TPW == 0) acc[0] = acc[1] = acc[2] = acc[3] = 0.0;
            if (t > 0) __syncthreads();            // the previous tile's LDS rows are reused
            if (kLean && t > 0) load_bonds(t);
#pragma unroll
            for (int sg = 0; sg < SEG; ++sg) {
                edge[0][w][sg][lane] = p_[t][sg][0];
                edge[1][w][sg][lane] = p_[t][sg][TY - 1];
            }
            __syncthreads();
            T pv[SEG][TY + 2];
#pragma unroll
            for (int sg = 0; sg < SEG; ++sg) {
                pv[sg][0] = w == 0 ? ep[t][sg] : edge[1][w - 1][sg][lane];
                pv[sg][TY + 1] = w == NW - 1 ? ep[t][sg] : edge[0][w + 1][sg][lane];
#pragma unroll
                for (int j = 0; j < TY; ++j) pv[sg][j + 1] = p_[t][sg][j];
            }
#pragma unroll
            for (int j = 0; j < TY; ++j) {
                const T hl = lane_bcast(hp[t], j);
                const T hrr = lane_bcast(hp[t], kWave - TY + j);
                const T hgl = lane_bcast(hg[t], j);
#pragma unroll
                for (int sg = 0; sg < SEG; ++sg) {
                    const T zc = z_[t][sg][j];
                    const T pc = pv[sg][j + 1];
                    T pl = lane_below(pc);
                    T pr = lane_above(pc);
                    T gxl = lane_below(gxv[t][sg][j]);
                    const T lj = sg == 0 ? hl : lane_bcast(pv[sg > 0 ? sg - 1 : 0][j + 1], kWave - 1);
                    const T gj = sg == 0 ? hgl : lane_bcast(gxv[t][sg > 0 ? sg - 1 : 0][j], kWave - 1);
                    const T rj = sg == SEG - 1 ? hrr : lane_bcast(pv[sg < SEG - 1 ? sg + 1 : 0][j + 1], 0);
                    if (lane == 0) {
                        pl = lj;
                        gxl = gj;
                    }
                    if (lane == kWave - 1) pr = rj;
                    const T gxr = gxv[t][sg][j], gyl = gyv[t][sg][j], gyr = gyv[t][sg][j + 1];
                    T qv = stencil2d(left_first<T>(sg), gxl, pc - pl, gxr, pc - pr, gyl, pc - pv[sg][j], gyr,
                                     pc - pv[sg][j + 2]);
                    const T d = diag_sum(gxl, gxr, gyl, gyr);
                    const bool live = (liv & bit(t, sg, j)) && d > T(0);
                    if (!live) qv = T(0);
                    const T uv = live ? apply_minv(qv, d, jacobi) : T(0);
                    u_[t][sg][j] = uv;
                    const double dq = (double)qv, du = (double)uv;
                    const double dp = (double)pc, dz = live ? (double)zc : 0.0;
                    acc[0] = fma_(dp, dq, acc[0]);
                    acc[1] = fma_(dz, dq, acc[1]);
                    acc[2] = fma_(dq, du, acc[2]);
                    acc[3] = fma_((double)(jacobi ? d : T(1)) * dz, dz, acc[3]);
                }
                // a row at a time: interleaved rows would hold all their
                // temporaries at once (four waves per SIMD hide the latency)
                if constexpr (kTight) __builtin_amdgcn_sched_barrier(0);
            }
            if (LB > 1 && t % TPW == TPW - 1) wave_sums(sh.red[t / TPW], acc);
        }
        if (w == 0) __builtin_amdgcn_s_waitcnt(0);   // what the last pass emptied is empty (wave 0 posts the sums)
        // u of the tiles' edges: rows as they lie, the columns gathered into
        // lanes 0 .. 2 TY - 1
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int tile = tile_of(t);
            if (tile >= a.ntiles) continue;        // uniform
            u64 *xt = xb + (size_t)tile * EW;
            const int jb = min(ty_[t] * ROWS + ROWS, ny) - 1 - rowy(t, 0);    // last lattice row, if in this wave
            const int cl = min(COLS, nx - tx_[t] * COLS) - 1;                 // last lattice column of the tile
            T cv = T(0);
#pragma unroll
            for (int j = 0; j < TY; ++j) {
                const T left = lane_bcast(u_[t][0][j], 0);
                T right = T(0);
#pragma unroll
                for (int sg = 0; sg < SEG; ++sg) {
                    if (cl >> 6 == sg) right = lane_at(u_[t][sg][j], cl & (kWave - 1));
                    if (((w == 0 && j == 0) || j == jb) && colx(t, sg) < nx) {
                        if (w == 0 && j == 0)
                            Packed<T>::template post<LOCAL>(at(xt, (unsigned)(kTop + kWave * sg + lane) * 8u), E, tag, u_[t][sg][j]);
                        if (j == jb) Packed<T>::template post<LOCAL>(at(xt, (unsigned)(kBottom + kWave * sg + lane) * 8u), E, tag, u_[t][sg][j]);
                    }
                }
                if (lane == j) cv = left;
                if (lane == TY + j) cv = right;
            }
            if (lane < 2 * TY && rowy(t, lane < TY ? lane : lane - TY) < ny)
                Packed<T>::template post<LOCAL>(at(xt, (unsigned)((lane < TY ? kLeft + lane : kRight + lane - TY) + w * TY) * 8u), E, tag, cv);
        }
        if constexpr (LB == 1) wave_sums(sh.red[0], acc);    // the edges are on their way
        post_sums<LOCAL>(sh, r, it, lbs, grid);
        // u of the halo and the images, from their owners (before the sums,
        // whose way is longer)
        Packed<T> ew[NT][SEG], hw[NT];
        bool missing;
        do {
            missing = false;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
#pragma unroll
                for (int sg = 0; sg < SEG; ++sg) {
                    if constexpr (kLean) ro[t][sg] = row_words(t, sg);
                    if (ro[t][sg] != kNone) ew[t][sg].look(at(xb, ro[t][sg]), E);
                    else ew[t][sg].zero(tag);
                }
                if constexpr (kLean) co[t] = col_words(t);
                if (co[t] != kNone) hw[t].look(at(xb, co[t]), E);
                else hw[t].zero(tag);
            }
#pragma unroll
            for (int t = 0; t < NT; ++t) {
#pragma unroll
                for (int sg = 0; sg < SEG; ++sg) missing |= !ew[t][sg].here(tag);
                missing |= !hw[t].here(tag);
            }
        } while (missing && spin.more());
#pragma unroll
        for (int t = 0; t < NT; ++t) {
#pragma unroll
            for (int sg = 0; sg < SEG; ++sg) {
                eu[t][sg] = ew[t][sg].value();
                if (wrap) {                        // uniform
#pragma unroll
                    for (int j = 0; j < TY; ++j) {
                        const int x = colx(t, sg), y = rowy(t, j);
                        const bool ix = wx && x == nx && y < ny, iy = wy && y == ny && x < nx;
                        if (ix || iy) {            // image of a node in column 0 or row 0
                            Packed<T> v;
                            const u64 *q = xb + (size_t)(ix ? ty_[t] * ntx : tx_[t]) * EW +
                                           (ix ? kLeft + w * TY + j : kTop + kWave * sg + lane);
                            do v.look(q, E);
                            while (!v.here(tag) && spin.more());
                            u_[t][sg][j] = v.value();
                        }
                    }
                }
            }
            hu[t] = hw[t].value();
        }
        if constexpr (kLean) load_bonds(0);        // the next pass's, while this one waits
        on = loop_turn<LOCAL>(sh, L, r, it, lb, grid, spin);
        if (__any(!spin.ok)) return;               // a wait gave up: the host fails the context
    }
    // ---- the state of the last pass, as a pass kernel leaves it (alpha is the
    // one pending step). A launch that was turned away moves z and u to the
    // other parity, where the next round reads them, and no more.
    const int64_t done = passes0 + it - 1;
    T *pd = a.pbuf[a.npbuf == 5 ? (int)(done % 5) : (int)(done % 3)];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int sg = 0; sg < SEG; ++sg)
#pragma unroll
            for (int j = 0; j < TY; ++j)
                if (colx(t, sg) < nx && rowy(t, j) < ny) {
                    const int i = rowy(t, j) * nx + colx(t, sg);
                    sti(a.dst.z, i, z_[t][sg][j]);
                    sti(a.dst.u, i, u_[t][sg][j]);
                    if (!admitted) continue;
                    sti(pd, i, p_[t][sg][j]);
                    double v;
                    if constexpr (kFieldLds) v = fl[(t * SEG + sg) * TY + j][threadIdx.x];
                    else v = Pv[t][sg][j];
                    sti(P, i, v);
                }
    if (admitted && lb == 0)                               // wave 0 ran the last step on this copy
        store_loop_end(reinterpret_cast<u64 *>(s), reinterpret_cast<const volatile u64 *>(&sh.sl[0]), (int)threadIdx.x);
    if constexpr (LOCAL)
        if (!admitted && blockIdx.x == 0) move_state(a);
}

// ---------------------------------------------------------------- 3D
// The tile of pass3d_kernel (64 x 16 x TZ nodes, a thread holds kRows rows of
// TZ planes), all planes at once: p' of the tile and its halo ring sits in
// LDS, one barrier per pass. The FP64 field is in LDS too. A thread keeps z
// and p of the nodes below and above its columns and of one ring node per
// plane. Two waves per SIMD, so 512 workgroups fit. Bonds stay in registers
// except with four FP64 planes, where they come from memory in every pass.
// Exchange words of a tile: lowest plane, highest plane; per plane the first
// row, last row, first column, last column.
constexpr int face_words3d(int tz) { return 2 * kTY * kTX + tz * 2 * (kTX + kTY); }

template <typename T, int TZ>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2))) void loop3d_kernel(
    const PassArgs<T> *__restrict__ tab, Scalars *scal, int parity, int slot, LoopArgs r)
{
    constexpr int R = kRows;
    constexpr int E = face_words3d(TZ), EW = E * (int)(sizeof(T) / 4);
    constexpr int kLow = 0, kHigh = kTY * kTX, kFirst = 2 * kTY * kTX, kLast = kFirst + TZ * kTX,
                  kLeft = kLast + TZ * kTX, kRight = kLeft + TZ * kTY;
    constexpr bool kStream = TZ * (int)sizeof(T) > 16;     // bonds from memory
    __shared__ T lp[TZ][kTY + 2][kTX + 2];
    __shared__ double fl[TZ * R][kBlock];
    __shared__ LoopShared sh;
    const Place at_ = loop_place<false>(r, slot);
    if (at_.lb < 0) return;
    const PassArgs<T> &a = tab[2 * at_.slot + parity];
    Scalars *s = scal + at_.slot;
    const int grid = a.grid, lb = at_.lb;
    if (s->mode != MODE_CG) return;
    int lane = threadIdx.x & (kWave - 1);
    const int w = rfl((int)threadIdx.x / kWave);
    const int tile = xcd_remap(lb, grid);
    const int nx = a.nx, ny = a.ny, nz = a.nz, ntx = a.ntx, nty = a.nty, ntz = a.ntz, wrap = a.wrap, ax = a.axis;
    const int sz = nx * ny;
    const bool wx = wrap & 1, wy = (wrap >> 1) & 1, wz = (wrap >> 2) & 1;
    const bool jacobi = a.jacobi != 0, has = tile < a.ntiles;
    const Step<T> k0 = make_step(a, s);
    const int64_t passes0 = s->passes;
    double *__restrict__ P = a.P[s->refreshes & 1];
    const int tx = has ? tile % ntx : 0, ty = has ? (tile / ntx) % nty : 0, tz = has ? tile / (ntx * nty) : 0;
    const int x0 = tx * kTX, y0 = ty * kTY, z0 = tz * TZ, yw = y0 + w * R;
    const int cnt = has ? min(TZ, nz - z0) : 0;             // planes of this tile
    // plane a lane, row slot or z step holds: its own inside the lattice, the
    // opposite edge's just past a periodic one, else -1 (as in cg3d_tile)
    auto colm = [&](int v) { return v >= 0 && v < nx ? v : (wx && v == nx ? 0 : (wx && v == -1 ? nx - 1 : -1)); };
    auto rowm = [&](int v) { return v >= 0 && v < ny ? v : (wy && v == ny ? 0 : (wy && v == -1 ? ny - 1 : -1)); };
    auto plm = [&](int v) { return v >= 0 && v < nz ? v : (wz && v == nz ? 0 : (wz && v == -1 ? nz - 1 : -1)); };
    // this thread's ring node: wave 0 row y0-1, wave 1 row y0+16, wave 2 lanes
    // 0..15 column x0-1, lanes 16..31 column x0+64 (rows y0..y0+15); the
    // corners are not needed
    int hx = -1, hy = -1, hrow = -1, hcol = 0;
    unsigned hword = 0;                                     // its word in plane 0 (value index)
    int hstep = 0;                                          // words from plane to plane
    if (has) {
        int q = tile;                                       // tile that owns it
        if (w == 0) {
            hrow = 0;
            hcol = 1 + lane;
            hx = x0 + lane < nx ? x0 + lane : -1;
            hy = rowm(y0 - 1);
            q = tile + ((ty > 0 ? ty : nty) - 1 - ty) * ntx;
            hword = kLast + lane;
            hstep = kTX;
        } else if (w == 1) {
            hrow = kTY + 1;
            hcol = 1 + lane;
            hx = x0 + lane < nx ? x0 + lane : -1;
            hy = rowm(y0 + kTY);
            q = tile + ((ty + 1 < nty ? ty + 1 : 0) - ty) * ntx;
            hword = kFirst + lane;
            hstep = kTX;
        } else if (w == 2 && lane < 2 * kTY) {
            const bool left = lane < kTY;
            const int row = left ? lane : lane - kTY;
            hrow = 1 + row;
            hcol = left ? 0 : kTX + 1;
            hx = colm(left ? x0 - 1 : x0 + kTX);
            hy = y0 + row < ny ? y0 + row : -1;
            q = left ? tile + (tx > 0 ? tx : ntx) - 1 - tx : tile + (tx + 1 < ntx ? tx + 1 : 0) - tx;
            hword = (left ? kRight : kLeft) + row;
            hstep = kTY;
        }
        hword += (unsigned)q * EW;
    }
    const bool hok = hx >= 0 && hy >= 0;
    const int hoff = hok ? hx + nx * hy : 0;
    // the tiles below and above (the opposite end's when z wraps)
    const bool lowok = has && plm(z0 - 1) >= 0, higok = has && plm(z0 + cnt) >= 0;
    const int zlow = lowok ? plm(z0 - 1) : 0, zhig = higok ? plm(z0 + cnt) : 0;
    const int qlow = tile + ((tz > 0 ? tz : ntz) - 1 - tz) * ntx * nty,
              qhig = tile + ((tz + 1 < ntz ? tz + 1 : 0) - tz) * ntx * nty;

    // ---- state of the tile
    T z_[TZ][R], u_[TZ][R], p_[TZ][R], gx[TZ][R], gy[TZ][R], gz[TZ][R], gzl[R], gxh[TZ], gyh[TZ];
    T lz[R], lu[R], lq[R], gz_[R], gu[R], gq[R];            // z, u, p below and above the columns
    T hz[TZ], hu[TZ], hp[TZ];                               // ... of the ring nodes
    unsigned own = 0, liv = 0;                              // bits row: lattice nodes; bits (plane, row): not on a face
    const int xm = colm(x0 + lane);
    const bool xok = has && x0 + lane < nx;
    auto row_off = [&](int j) {                             // clamped x + nx y of row j
        const int ym = rowm(yw + j);
        return (xm >= 0 ? xm : nx - 1) + nx * (ym >= 0 ? ym : ny - 1);
    };
    auto held = [&](int j) { return has && xm >= 0 && rowm(yw + j) >= 0; };
    auto load_bonds = [&](int q) {                          // of plane q: right, upper, next; left of the tile, below the wave
        const int zo = min(z0 + q, nz - 1) * sz;
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int i = row_off(j) + zo;
            gx[q][j] = ldi(a.gT[0], i);
            gy[q][j] = ldi(a.gT[1], i);
            gz[q][j] = ldi(a.gT[2], i);
        }
        const int xb = colm(x0 - 1), yb = rowm(yw - 1);
        const bool xhok = lane < R && xb >= 0 && yw + lane < ny, yhok = xm >= 0 && yb >= 0;
        const T xh = ldi(a.gT[0], zo + (xhok ? xb + nx * (yw + lane) : 0)),
                yh = ldi(a.gT[1], zo + (yhok ? xm + nx * yb : 0));
        gxh[q] = xhok ? xh : T(0);
        gyh[q] = yhok ? yh : T(0);
    };
    auto load_below = [&] {                                 // bonds from the plane below
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const T g = ldi(a.gT[2], row_off(j) + zlow * sz);
            gzl[j] = lowok && held(j) ? g : T(0);
        }
    };
#pragma unroll
    for (int j = 0; j < R; ++j)
        if (xok && yw + j < ny) own |= 1u << j;
#pragma unroll
    for (int q = 0; q < TZ; ++q) {
        const int zo = min(z0 + q, nz - 1) * sz;
        const bool in = q < cnt;
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int i = row_off(j) + zo, x = x0 + lane, y = yw + j, z = z0 + q;
            const bool ok = in && held(j);
            const T zv = ldi(a.src.z, i), uv = ldi(a.src.u, i), pv = ldi(k0.p1, i);
            double v = ldi((const double *)P, i);
            if (k0.sa3 != 0.0 || k0.sa4 != 0.0)
                v = with_steps(v, k0.sa4, (double)ldi(k0.p4, i), k0.sa3, (double)ldi(k0.p3, i));
            if (k0.sa2 != 0.0) v = with_steps(v, k0.sa2, (double)ldi(k0.p2, i), 0.0, 0.0);
            z_[q][j] = ok ? zv : T(0);
            u_[q][j] = ok ? uv : T(0);
            p_[q][j] = ok ? pv : T(0);
            fl[q * R + j][threadIdx.x] = v;
            const bool face = ax == 0 ? (x == 0 || x == nx - 1) : (ax == 1 ? (y == 0 || y == ny - 1) : (z == 0 || z == nz - 1));
            if (in && (own >> j & 1u) && !face) liv |= 1u << (q * R + j);
        }
        if (!kStream || q == 0) load_bonds(q);
        const int i = hoff + zo;
        const T zv = ldi(a.src.z, i), uv = ldi(a.src.u, i), pv = ldi(k0.p1, i);
        hz[q] = hok && in ? zv : T(0);
        hu[q] = hok && in ? uv : T(0);
        hp[q] = hok && in ? pv : T(0);
    }
    load_below();
#pragma unroll
    for (int j = 0; j < R; ++j) {
        const int il = row_off(j) + zlow * sz, ig = row_off(j) + zhig * sz;
        const bool ok = own >> j & 1u;
        const T z1 = ldi(a.src.z, il), u1 = ldi(a.src.u, il), p1 = ldi(k0.p1, il);
        const T z2 = ldi(a.src.z, ig), u2 = ldi(a.src.u, ig), p2 = ldi(k0.p1, ig);
        lz[j] = ok && lowok ? z1 : T(0);
        lu[j] = ok && lowok ? u1 : T(0);
        lq[j] = ok && lowok ? p1 : T(0);
        gz_[j] = ok && higok ? z2 : T(0);
        gu[j] = ok && higok ? u2 : T(0);
        gq[j] = ok && higok ? p2 : T(0);
    }
    LoopState L;
    const int lbs[1] = {lb};
    const bool admitted = loop_begin<false>(sh, L, s, r, lbs, 1, grid);

    int it = 0;
    for (bool on = __builtin_expect(admitted, 1); on; ++it) {
        Spin spin(s);
        const T alpha = (T)rfl(L.alpha), beta = (T)rfl(L.beta);
        const double sa = rfl(L.sa);
        const unsigned tag = r.tag0 + (unsigned)it;
        u64 *xb = r.xch + (size_t)(it & 1) * r.xch_slot;
        if constexpr (!kStream) {
#pragma unroll
            for (int q = 0; q < TZ; ++q) {
#pragma unroll
                for (int j = 0; j < R; ++j) {
                    hide(gx[q][j]);
                    hide(gy[q][j]);
                    hide(gz[q][j]);
                }
                hide(gxh[q]);
                hide(gyh[q]);
            }
        }
#pragma unroll
        for (int j = 0; j < R; ++j) hide(gzl[j]);
        hide(own);
        hide(liv);
        hide(hword);
        hide(lane);
        // the pending step, then z' and p' of the tile and its halo
#pragma unroll
        for (int q = 0; q < TZ; ++q) {
#pragma unroll
            for (int j = 0; j < R; ++j) {
                if (sa != 0.0) {
                    double &f = fl[q * R + j][threadIdx.x];
                    f = fma(sa, (double)p_[q][j], f);
                }
                z_[q][j] = step_z(z_[q][j], alpha, u_[q][j]);
                p_[q][j] = step_p(z_[q][j], beta, p_[q][j]);
                lp[q][1 + w * R + j][1 + lane] = p_[q][j];
            }
            hz[q] = step_z(hz[q], alpha, hu[q]);
            hp[q] = step_p(hz[q], beta, hp[q]);
            if (hrow >= 0) lp[q][hrow][hcol] = hp[q];
        }
#pragma unroll
        for (int j = 0; j < R; ++j) {
            lz[j] = step_z(lz[j], alpha, lu[j]);
            lq[j] = step_p(lz[j], beta, lq[j]);
            gz_[j] = step_z(gz_[j], alpha, gu[j]);
            gq[j] = step_p(gz_[j], beta, gq[j]);
        }
        __syncthreads();
        double acc[kLoopRed] = {0.0, 0.0, 0.0, 0.0};
        // (b) stencil
#pragma unroll
        for (int q = 0; q < TZ; ++q) {
            if constexpr (kStream) {
                if (q > 0) load_bonds(q);
            }
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const int ly = 1 + w * R + j;
                T gxl = lane_below(gx[q][j]);
                const T gxe = lane_bcast(gxh[q], j);
                if (lane == 0) gxl = gxe;
                const T gyl = j == 0 ? gyh[q] : gy[q][j > 0 ? j - 1 : 0];
                const T gzm = q == 0 ? gzl[j] : gz[q > 0 ? q - 1 : 0][j];
                const T p0 = p_[q][j];
                const T pm = q == 0 ? lq[j] : p_[q > 0 ? q - 1 : 0][j];
                const T pn = q + 1 < TZ && q + 1 < cnt ? p_[q + 1 < TZ ? q + 1 : q][j] : gq[j];   // cnt: uniform
                T qv = stencil3d(gxl, p0 - lp[q][ly][lane], gx[q][j], p0 - lp[q][ly][lane + 2], gyl,
                                 p0 - lp[q][ly - 1][1 + lane], gy[q][j], p0 - lp[q][ly + 1][1 + lane], gzm, p0 - pm,
                                 gz[q][j], p0 - pn);
                const T d = diag_sum(gxl, gx[q][j], gyl, gy[q][j], gzm, gz[q][j]);
                const bool live = (liv & (1u << (q * R + j))) && d > T(0);
                if (!live) qv = T(0);
                const T uv = live ? apply_minv(qv, d, jacobi) : T(0);
                u_[q][j] = uv;
                const double dp = (double)p0, dq = (double)qv, du = (double)uv;
                const double dz = live ? (double)z_[q][j] : 0.0;
                acc[0] = fma_(dp, dq, acc[0]);
                acc[1] = fma_(dz, dq, acc[1]);
                acc[2] = fma_(dq, du, acc[2]);
                acc[3] = fma_((double)(jacobi ? d : T(1)) * dz, dz, acc[3]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (w == 0) __builtin_amdgcn_s_waitcnt(0);   // what the last pass emptied is empty (wave 0 posts the sums)
        // u of the tile's faces
        if (has) {
            u64 *xt = xb + (size_t)tile * EW;
            const int jb = min(y0 + kTY, ny) - 1 - yw;       // last lattice row, if in this wave
            const int cl = min(kTX, nx - x0) - 1;            // last lattice column of the tile
            T cv = T(0);
#pragma unroll
            for (int q = 0; q < TZ; ++q) {
                if (q >= cnt) continue;                      // uniform
#pragma unroll
                for (int j = 0; j < R; ++j) {
                    const T uv = u_[q][j];
                    if (own >> j & 1u) {
                        const unsigned wo = (unsigned)((w * R + j) * kTX + lane) * 8u;
                        if (q == 0) Packed<T>::template post<false>(at(xt + kLow, wo), E, tag, uv);
                        if (q == cnt - 1) Packed<T>::template post<false>(at(xt + kHigh, wo), E, tag, uv);
                        if (w == 0 && j == 0) Packed<T>::template post<false>(at(xt + kFirst + q * kTX, (unsigned)lane * 8u), E, tag, uv);
                        if (j == jb) Packed<T>::template post<false>(at(xt + kLast + q * kTX, (unsigned)lane * 8u), E, tag, uv);
                    }
                    const T left = lane_bcast(uv, 0), right = lane_at(uv, cl);
                    if (lane == q * R + j) cv = left;
                    if (lane == 32 + q * R + j) cv = right;
                }
            }
            const int e = lane & 31, row = e % R, q = e / R; // the columns, gathered into lanes 0.. and 32..
            if (e < cnt * R && yw + row < ny)
                Packed<T>::template post<false>(at(xt, (unsigned)((lane < 32 ? kLeft : kRight) + q * kTY + w * R + row) * 8u), E, tag, cv);
        }
        wave_sums(sh.red[0], acc);
        post_sums<false>(sh, r, it, lbs, grid);
        // u of the halo, from its owners
        Packed<T> lw[R], gw[R], hw[TZ];
        bool missing;
        do {
            missing = false;
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const unsigned wo = (unsigned)((w * R + j) * kTX + lane) * 8u;
                if (lowok && (own >> j & 1u)) lw[j].look(at(xb + (size_t)qlow * EW + kHigh, wo), E);
                else lw[j].zero(tag);
                if (higok && (own >> j & 1u)) gw[j].look(at(xb + (size_t)qhig * EW + kLow, wo), E);
                else gw[j].zero(tag);
            }
#pragma unroll
            for (int q = 0; q < TZ; ++q) {
                if (hok && q < cnt) hw[q].look(at(xb, (hword + (unsigned)(q * hstep)) * 8u), E);
                else hw[q].zero(tag);
            }
#pragma unroll
            for (int j = 0; j < R; ++j) missing |= !lw[j].here(tag) || !gw[j].here(tag);
#pragma unroll
            for (int q = 0; q < TZ; ++q) missing |= !hw[q].here(tag);
        } while (missing && spin.more());
#pragma unroll
        for (int j = 0; j < R; ++j) {
            lu[j] = lw[j].value();
            gu[j] = gw[j].value();
        }
#pragma unroll
        for (int q = 0; q < TZ; ++q) hu[q] = hw[q].value();
        if (wrap & 3) {                                      // uniform: images of column 0 and row 0
#pragma unroll
            for (int q = 0; q < TZ; ++q)
#pragma unroll
                for (int j = 0; j < R; ++j) {
                    const int x = x0 + lane, y = yw + j;
                    const bool ix = wx && x == nx && y < ny, iy = wy && y == ny && x < nx;
                    if (has && q < cnt && (ix || iy)) {
                        Packed<T> v;
                        u64 *o = ix ? xb + (size_t)(tile - tx) * EW + kLeft + q * kTY + w * R + j
                                    : xb + (size_t)(tile - ty * ntx) * EW + kFirst + q * kTX + lane;
                        do v.look(o, E);
                        while (!v.here(tag) && spin.more());
                        u_[q][j] = v.value();
                    }
                }
        }
        if constexpr (kStream) load_bonds(0);                // the next pass's, while this one waits
        on = loop_turn<false>(sh, L, r, it, lb, grid, spin);
        if (__any(!spin.ok)) return;                         // a wait gave up: the host fails the context
    }
    // ---- the state of the last pass (see loop2d_kernel)
    const int64_t done = passes0 + it - 1;
    T *pd = a.pbuf[a.npbuf == 5 ? (int)(done % 5) : (int)(done % 3)];
#pragma unroll
    for (int q = 0; q < TZ; ++q)
#pragma unroll
        for (int j = 0; j < R; ++j)
            if (q < cnt && (own >> j & 1u)) {
                const int i = x0 + lane + nx * (yw + j) + (z0 + q) * sz;
                sti(a.dst.z, i, z_[q][j]);
                sti(a.dst.u, i, u_[q][j]);
                if (!admitted) continue;
                sti(pd, i, p_[q][j]);
                sti(P, i, fl[q * R + j][threadIdx.x]);
            }
    if (admitted && lb == 0)
        store_loop_end(reinterpret_cast<u64 *>(s), reinterpret_cast<const volatile u64 *>(&sh.sl[0]), (int)threadIdx.x);
}

}  // namespace

// ---------------------------------------------------------------- launchers

template <typename T>
static const void *loop_kernel(int dim, int tpw, int tile_z, bool local)
{
    if (dim == -2 && tpw == 1)
        return local ? reinterpret_cast<const void *>(&loop2d_kernel<T, 1, 1, true, 1>)
                     : reinterpret_cast<const void *>(&loop2d_kernel<T, 1, 1, false, 1>);
    if (local) return nullptr;
    if (dim == 3 && tile_z == 2) return reinterpret_cast<const void *>(&loop3d_kernel<T, 2>);
    if (dim == 3 && tile_z == 4) return reinterpret_cast<const void *>(&loop3d_kernel<T, 4>);
    if (dim == 2 && tpw == 1) return reinterpret_cast<const void *>(&loop2d_kernel<T, 0, 1, false, 1>);
    if (dim == 2 && tpw == 2) return reinterpret_cast<const void *>(&loop2d_kernel<T, 0, 2, false, 2>);
    return nullptr;
}

// workgroups of the pass kernel that a workgroup of the loop stands for
static int loop_per_group(int dim, int tpw) { return dim == 2 && tpw == 2 ? 2 : 1; }

int loop_blocks(int dim, int tpw, int grid) { return 8 * div_up(grid / 8, loop_per_group(dim, tpw)); }   // grid: a multiple of 8

template <typename T>
hipError_t loop_capacity(int dim, int tpw, int tile_z, bool local, int *cap)
{
    *cap = 0;
    const void *k = loop_kernel<T>(dim, tpw, tile_z, local);
    if (!k) return hipSuccess;
    int dev = 0, cus = 0, per = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k, kBlock, 0);
    if (e != hipSuccess) return e;
    *cap = local ? std::min(per * cus / 8, kLoopLocalMax) : std::min(per * cus, kLoopGridMax / loop_per_group(dim, tpw));
    return hipSuccess;
}

template <typename T>
size_t loop_exchange_words(int dim, int tile_z, int ntiles)
{
    const size_t values = dim == 3 ? face_words3d(tile_z) : dim == 2 ? edge_words2d<T, 0>() : edge_words2d<T, 1>();
    return values * (sizeof(T) / 4) * (size_t)ntiles;
}

// A launch that every gate turns away: no count reaches the number that opens
// it, and (LOCAL) every place is taken.
__global__ void shut_gates_kernel(unsigned *gate)
{
    gate[threadIdx.x * kLoopGateWords] = gate[threadIdx.x * kLoopGateWords + 2] = 1u << 30;
}

hipError_t launch_shut_gates(unsigned *gate, hipStream_t st)
{
    shut_gates_kernel<<<1, kLoopMembers, 0, st>>>(gate);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_loop(int dim, int tpw, int tile_z, bool local, int blocks, const PassArgs<T> *tab, Scalars *scal,
                       int parity, int slot, const LoopArgs &r, hipStream_t st)
{
    const void *k = loop_kernel<T>(dim, tpw, tile_z, local);
    if (!k || blocks < 1 || blocks > kLoopGridMax) return hipErrorInvalidValue;
    LoopArgs args = r;
    void *p[] = {(void *)&tab, (void *)&scal, (void *)&parity, (void *)&slot, (void *)&args};
    return hipLaunchKernel(k, dim3((unsigned)(local ? 8 * blocks : blocks)), dim3(kBlock), p, 0, st);
}

template size_t loop_exchange_words<float>(int, int, int);
template size_t loop_exchange_words<double>(int, int, int);
template hipError_t loop_capacity<float>(int, int, int, bool, int *);
template hipError_t loop_capacity<double>(int, int, int, bool, int *);
template hipError_t launch_loop<float>(int, int, int, bool, int, const PassArgs<float> *, Scalars *, int, int,
                                       const LoopArgs &, hipStream_t);
template hipError_t launch_loop<double>(int, int, int, bool, int, const PassArgs<double> *, Scalars *, int, int,
                                        const LoopArgs &, hipStream_t);

}  // namespace rn
