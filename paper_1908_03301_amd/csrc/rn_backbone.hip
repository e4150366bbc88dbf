// rn_backbone.hip -- the backbone of the sample-spanning cluster on the GPU.
//
// Near the percolation threshold (Sec. VI) most live nodes sit on dangling
// ends: branches and loops that meet the rest of the cluster at one node and
// carry no flow. The backbone is the set of interior nodes on an inlet-outlet
// path that visits no node twice. With the inlet face contracted to a vertex
// S, the outlet face to T and an edge S-T added, it is the vertex set of the
// biconnected component (block) that holds S-T.
//
// Blocks by Tarjan and Vishkin's method, on whatever spanning tree the
// connectivity pass leaves behind, numbered by an Euler tour. Nothing here
// depends on the depth of the tree (a breadth-first tree took a launch per
// level and phase, about 6,000 launches and 47 ms on a 2048^2 network near the
// threshold; bytes alone would take 0.02 ms):
//   1. Tree. The bonds whose union-find hook succeeded in the connectivity
//      pass span every component of interior nodes; each live component adds
//      one bond to the inlet face, and S-T joins T, a leaf. A byte per vertex
//      holds its tree directions (bit 6: its bond to S).
//   2. Tour. Arriving at a vertex from direction r, the tour leaves by the
//      next tree direction after r in circular order, so an arc's successor is
//      a look at one byte and no list is stored. One vertex in eight (picked by
//      a hash, so that no regular tree avoids them) starts a walker at its
//      first arc, which counts arcs until it meets the next start; pointer
//      jumping ranks the starts (distance to the last one of the component,
//      whose end is allotted from a counter); the walkers go again and write
//      positions: in(v), the first arrival at v, and last(v), the last. The
//      subtree of v is the positions in .. last. Longest walk measured: a few
//      hundred steps, as for random starts.
//   3. low / high: the extreme positions joined to a vertex by a non-tree edge
//      are stored at in(v); minima and maxima over 8, 64, ... positions make
//      the extremes over a subtree a walk up and down that hierarchy.
//   4. Joins. Tree edges (named by their child vertex) form classes in a
//      lock-free union-find ordered by in(): a tree edge (p, v) with p not S
//      joins p's when low(v) < in(p) or high(v) > last(p), written straight
//      into the parent words (tree parents come first in that order) and
//      shortened by pointer jumping; a non-tree edge whose ends are not
//      ancestor and descendant joins the two ends' tree edges.
//   5. The backbone is the set of lattice ends of the tree edges in T's class
//      (T's tree edge is S-T): bit 3 (8) of the mask.
// The races decide which tree is built, not the blocks: the mask is
// deterministic.
#include "rn_runtime.hpp"

#include <algorithm>

namespace rn {
namespace {

constexpr int kBbBlock = 256;
constexpr int kDirS = 6;                  // tree direction of the bond to S
constexpr unsigned kStart = 0x80u;        // flag of a vertex whose first arc starts a walker
constexpr int kSpread = 8;                // vertices per walker
constexpr int kFan = 8, kFanLevels = 11;  // the hierarchy of minima and maxima
constexpr unsigned kNone = 0xffffffffu;
// Positions of the tour: 0 is S (an edge to it reaches below every position),
// T is 1, the components follow.
constexpr unsigned kPosT = 1u, kPosFirst = 2u;

// The indices 0 .. n - 1 that fall to this thread of a launch: of nodes (fewer
// than 2^31) and of positions of the tour (up to twice as many).
__device__ __forceinline__ Strided<false> each(int n)
{
    return {{blockIdx.x * kBbBlock + threadIdx.x, gridDim.x * kBbBlock, (unsigned)n}};
}
__device__ __forceinline__ Strided<true> each_position(unsigned n)
{
    return {{blockIdx.x * kBbBlock + threadIdx.x, gridDim.x * kBbBlock, n}};
}

struct BbGraph {
    const double *g[3];
    const uint8_t *mask;
    int dim, axis, nx, ny, nz, wrap;
    int n, S, T;                          // lattice vertices 0..n-1, then S = n, T = n + 1
};

__device__ __forceinline__ void coords(const BbGraph &G, int v, int c[3])
{
    c[0] = v % G.nx;
    c[1] = (v / G.nx) % G.ny;
    c[2] = v / (G.nx * G.ny);
}

// Lattice index across direction e (k = e / 2, towards +k when e is odd) of
// node v, or -1 off the lattice; *gij the bond's conductance.
__device__ __forceinline__ int lat_step(const BbGraph &G, int v, const int c[3], int e, double *gij)
{
    const int k = e >> 1;
    const int n[3] = {G.nx, G.ny, G.nz};
    const int st[3] = {1, G.nx, G.nx * G.ny};
    const bool wk = (G.wrap >> k) & 1;
    if (e & 1) {
        int j;
        if (c[k] + 1 < n[k]) j = v + st[k];
        else if (wk) j = v - (n[k] - 1) * st[k];
        else return -1;
        *gij = G.g[k][v];
        return j;
    }
    int j;
    if (c[k] > 0) j = v - st[k];
    else if (wk) j = v + (n[k] - 1) * st[k];
    else return -1;
    *gij = G.g[k][j];
    return j;
}

// Vertex joined to interior node v by its bond in direction e: a live
// interior node, S or T for a face node, -1 for no occupied bond or a node
// off the live set.
__device__ __forceinline__ int bb_nbr(const BbGraph &G, int v, const int c[3], int e)
{
    if ((e >> 1) >= G.dim) return -1;
    double gij = 0.0;
    const int j = lat_step(G, v, c, e, &gij);
    if (j < 0 || !(gij > 0.0)) return -1;
    if ((e >> 1) == G.axis) {
        const int na = G.axis == 0 ? G.nx : (G.axis == 1 ? G.ny : G.nz);
        const int ca = c[G.axis] + ((e & 1) ? 1 : -1);
        if (ca == 0) return G.S;
        if (ca == na - 1) return G.T;
    }
    return G.mask[j] == 3 ? j : -1;
}

__device__ __forceinline__ unsigned load_agent(const unsigned *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Arrays of the search, all of them for the n lattice vertices unless noted.
struct BbWork {
    const int *parent;                    // components of the connectivity pass
    unsigned *flags;                      // its flags, at the components' roots; bit 2: has its bond to S
    uint8_t *tree;                        // bit k: the bond to +k is a tree edge; later: on the backbone
    uint8_t *adj;                         // tree directions, kDirS, kStart; 0 off the live set
    unsigned *in, *last;                  // n + 2 (T at n + 1)
    int *uf;                              // n + 2
    unsigned long long *jump[2];          // per walker: start it leads to (low half), arcs to there
    unsigned *len, *end;                  // per walker: its arcs; at the last start of a component: end position
    unsigned *heads;                      // the vertices joined to S by a tree edge
    int *first;                           // per walker of a vertex group: its vertex or -1
    unsigned *lo[kFanLevels], *hi[kFanLevels];
    unsigned *counter;                    // [0] heads, [1] positions
    int groups;                           // groups of kSpread vertices
};

// 1. Tree directions of every live vertex; the first vertex of a component to
// ask gets its tree bond to S.
__global__ void bb_tree(BbGraph G, BbWork W)
{
    const int V = G.n + 2;
    for (const int v : each(V)) {
        W.uf[v] = v;
        W.in[v] = v == G.T ? kPosT : kNone;
        W.last[v] = v == G.T ? kPosT : 0u;
        if (v >= G.n) continue;
        unsigned bits = 0u;
        if (G.mask[v] == 3) {
            int c[3];
            coords(G, v, c);
            for (int e = 0; e < 2 * G.dim; ++e) {
                double gij = 0.0;
                const int j = (e & 1) ? v : lat_step(G, v, c, e, &gij);
                if (j >= 0 && (W.tree[j] >> (e >> 1) & 1u)) bits |= 1u << e;
            }
            if (c[G.axis] == 1 && bb_nbr(G, v, c, 2 * G.axis) == G.S) {
                int r = v;
                while (true) {                       // the connectivity pass is over: plain loads
                    const int q = W.parent[r];
                    if (q == r) break;
                    r = q;
                }
                if (!(atomicOr(W.flags + r, 4u) & 4u)) {
                    bits |= 1u << kDirS;
                    W.heads[atomicAdd(W.counter, 1u)] = (unsigned)v;
                }
            }
        }
        W.adj[v] = (uint8_t)bits;
    }
}

// The vertex of each group that starts a walker: the first live one from a
// hashed place on whose first tree direction is a lattice bond (an arrival
// from S is a head's).
__global__ void bb_starts(BbGraph G, BbWork W)
{
    for (const int g : each(W.groups)) {
        unsigned h = (unsigned)g * 0x9e3779b1u;
        h ^= h >> 15;
        h *= 0x85ebca6bu;
        h ^= h >> 13;
        int pick = -1;
        for (int k = 0; k < kSpread && pick < 0; ++k) {
            const int v = g * kSpread + (int)((h + (unsigned)k) % kSpread);
            if (v < G.n && (W.adj[v] & 0x3fu)) pick = v;
        }
        W.first[g] = pick;
        if (pick >= 0) W.adj[pick] = (uint8_t)(W.adj[pick] | kStart);
    }
}

// One step of the tour: from an arrival at v by direction r (bits: v's byte)
// to the next arrival. False when the tour leaves to S.
__device__ __forceinline__ bool tour_step(const BbGraph &G, const uint8_t *adj, int &v, int &r, unsigned &bits)
{
    const unsigned dirs = bits & 0x7fu;
    const unsigned above = dirs & ~((2u << r) - 1u);
    const int d = __ffs((int)(above ? above : dirs)) - 1;
    if (d == kDirS) return false;
    const int k = d >> 1;
    const int n[3] = {G.nx, G.ny, G.nz};
    const int st = k == 0 ? 1 : (k == 1 ? G.nx : G.nx * G.ny);
    int step = (d & 1) ? st : -st;
    if (G.wrap >> k & 1) {
        int c[3];
        coords(G, v, c);
        if ((d & 1) && c[k] + 1 == n[k]) step = -(n[k] - 1) * st;
        else if (!(d & 1) && c[k] == 0) step = (n[k] - 1) * st;
    }
    v += step;
    r = d ^ 1;
    bits = adj[v];
    return true;
}

__device__ __forceinline__ bool is_start(unsigned bits, int r)
{
    return (bits & kStart) && r == __ffs((int)(bits & 0x7fu)) - 1;
}

// Where walker i starts: false for a group without one.
__device__ __forceinline__ bool walker(const BbWork &W, int i, int &v, int &r, unsigned &bits)
{
    v = i < W.groups ? W.first[i] : (int)W.heads[i - W.groups];
    if (v < 0) return false;
    bits = W.adj[v];
    r = i < W.groups ? __ffs((int)(bits & 0x7fu)) - 1 : kDirS;
    return true;
}

// 2. Walk from every start to the next: its number of arrivals and where it leads.
__global__ void bb_walk(BbGraph G, BbWork W)
{
    const int total = W.groups + (int)W.counter[0];
    for (const int i : each(total)) {
        int v, r;
        unsigned bits, len = 0u, to = (unsigned)i;
        if (walker(W, i, v, r, bits)) {
            len = 1u;
            // (a walk visits an arc at most once: the bound is never reached)
            while (len < 2u * (unsigned)G.n + 2u && tour_step(G, W.adj, v, r, bits)) {
                if (is_start(bits, r)) {
                    to = (unsigned)(v / kSpread);
                    break;
                }
                ++len;
            }
        }
        W.len[i] = len;
        // the last start of a component leads to itself, at distance 0
        W.jump[0][i] = to == (unsigned)i ? (unsigned long long)to : ((unsigned long long)len << 32) | to;
    }
}

// Four jumps in one launch: its cost is the launch more than the loads
// (2048^2: 10 launches of 10.1 us; 20 of 7.3 us with two jumps in each).
__global__ void bb_jump(BbWork W, int from)
{
    const int total = W.groups + (int)W.counter[0];
    const unsigned long long *src = W.jump[from];
    unsigned long long *dst = W.jump[from ^ 1];
    for (const int i : each(total)) {
        unsigned long long a = src[i], far = a >> 32;
        for (int k = 1; k < 4; ++k) {
            a = src[(unsigned)a];
            far += a >> 32;
        }
        dst[i] = far << 32 | (unsigned)a;
    }
}

// Every component's range of positions, noted at its last start.
__global__ void bb_ranges(BbWork W, int from)
{
    const int heads = (int)W.counter[0];
    for (const int h : each(heads)) {
        const unsigned long long a = W.jump[from][W.groups + h];
        const unsigned t = (unsigned)a, size = (unsigned)(a >> 32) + W.len[t];
        W.end[t] = kPosFirst + atomicAdd(W.counter + 1, size) + size;
    }
}

// Walk again, writing the positions. A vertex of one tree direction is
// arrived at once; one of two directions writes a word for each, which
// bb_clear puts in order. The others, about a quarter of the vertices of a
// 2048^2 network, take atomics, which this launch is bound by (there 269 us,
// 484 with atomics for the vertices of two directions too).
__global__ void bb_number(BbGraph G, BbWork W, int from)
{
    const int total = W.groups + (int)W.counter[0];
    for (const int i : each(total)) {
        int v, r;
        unsigned bits;
        if (!walker(W, i, v, r, bits)) continue;
        const unsigned long long a = W.jump[from][i];
        const unsigned t = (unsigned)a;
        unsigned pos = W.end[t] - W.len[t] - (unsigned)(a >> 32);
        for (unsigned k = W.len[i]; k > 0u; --k, ++pos) {
            const unsigned dirs = bits & 0x7fu, rest = dirs & (dirs - 1u);
            if (rest == 0u) {
                W.in[v] = pos;
                W.last[v] = pos;
            } else if ((rest & (rest - 1u)) == 0u) {
                (rest >> r & 1u ? W.last : W.in)[v] = pos;
            } else {
                atomicMin(W.in + v, pos);
                atomicMax(W.last + v, pos);
            }
            if (k > 1u) tour_step(G, W.adj, v, r, bits);
        }
    }
}

// First and last arrival in order; 3. identities at the positions that are no
// first arrival.
__global__ void bb_clear(BbGraph G, BbWork W)
{
    for (const int v : each(G.n)) {
        const unsigned a = W.in[v], b = W.last[v];
        if (a > b && a != kNone) {
            W.in[v] = b;
            W.last[v] = a;
        }
    }
    const unsigned m = kPosFirst + W.counter[1];
    for (const unsigned i : each_position(m)) {
        W.lo[0][i] = kNone;
        W.hi[0][i] = 0u;
    }
}

// Whether v's edge in direction e (to w) is a tree edge (T's are not).
__device__ __forceinline__ bool is_tree(const BbGraph &G, const BbWork &W, int v, int w, int e)
{
    if (w >= G.n) return w == G.S && (W.adj[v] >> kDirS & 1u);
    return W.adj[v] >> e & 1u;
}

// low / high of every live vertex's own non-tree edges, at its first arrival.
__global__ void bb_reach(BbGraph G, BbWork W)
{
    for (const int v : each(G.n)) {
        if (!W.adj[v]) continue;
        int c[3];
        coords(G, v, c);
        const unsigned at = W.in[v];
        unsigned l = at, h = at;
        for (int e = 0; e < 2 * G.dim; ++e) {
            const int w = bb_nbr(G, v, c, e);
            if (w < 0 || is_tree(G, W, v, w, e)) continue;
            const unsigned q = w == G.S ? 0u : W.in[w];
            l = min(l, q);
            h = max(h, q);
        }
        W.lo[0][at] = l;
        W.hi[0][at] = h;
    }
}

__global__ void bb_level(BbWork W, int level)
{
    unsigned below = kPosFirst + W.counter[1];
    for (int k = 1; k < level; ++k) below = (below + kFan - 1) / kFan;
    const unsigned m = (below + kFan - 1) / kFan;
    for (const unsigned i : each_position(m)) {
        unsigned l = kNone, h = 0u;
        for (unsigned k = i * kFan; k < min(below, (i + 1u) * kFan); ++k) {
            l = min(l, W.lo[level - 1][k]);
            h = max(h, W.hi[level - 1][k]);
        }
        W.lo[level][i] = l;
        W.hi[level][i] = h;
    }
}

// Tree parent of v: S for a head, else the tree neighbour that comes before it.
__device__ __forceinline__ int tree_parent(const BbGraph &G, const BbWork &W, int v, const int c[3])
{
    const unsigned bits = W.adj[v];
    if (bits >> kDirS & 1u) return G.S;
    const unsigned at = W.in[v];
    for (int e = 0; e < 2 * G.dim; ++e) {
        if (!(bits >> e & 1u)) continue;
        double gij;
        const int w = lat_step(G, v, c, e, &gij);
        if (W.in[w] < at) return w;
    }
    return G.S;                                      // (not reached)
}

// The union-find reads and writes through the L2 (device scope): a plain load
// may be served from the CU's L1, which keeps a line another CU has since
// hooked, and a root that looks unhooked there would be retried forever.
__device__ __forceinline__ int uf_get(const int *uf, int x)
{
    return __hip_atomic_load(uf + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int uf_find(int *uf, int x)
{
    int p = uf_get(uf, x);
    while (p != x) {
        const int gp = uf_get(uf, p);
        // halve the path: gp is an ancestor of x (parents come first in the
        // order of the hooks), and only non-roots are written, never a root a
        // hook targets
        if (gp != p) __hip_atomic_store(uf + x, gp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        x = p;
        p = uf_get(uf, x);
    }
    return x;
}

__device__ __forceinline__ void uf_union(int *uf, int a, int b)
{
    while (true) {
        a = uf_find(uf, a);
        b = uf_find(uf, b);
        if (a == b) return;
        if (a < b) {
            const int t = a;
            a = b;
            b = t;
        }
        if (atomicCAS(&uf[a], a, b) == a) return;   // hook the larger root under the smaller
    }
}

// The same with roots hooked in the order of the tour.
__device__ __forceinline__ void uf_union_tour(int *uf, const unsigned *in, int a, int b)
{
    while (true) {
        a = uf_find(uf, a);
        b = uf_find(uf, b);
        if (a == b) return;
        if (in[a] < in[b]) {
            const int t = a;
            a = b;
            b = t;
        }
        if (atomicCAS(&uf[a], a, b) == a) return;
    }
}

// 4. Joins along the tree: low / high over the subtree of v from the hierarchy.
__global__ void bb_join_tree(BbGraph G, BbWork W)
{
    for (const int v : each(G.n)) {
        if (!W.adj[v]) continue;
        int c[3];
        coords(G, v, c);
        const int p = tree_parent(G, W, v, c);
        if (p == G.S) continue;
        const unsigned first = W.in[p], last = W.last[p];
        unsigned l = W.in[v], r = W.last[v] + 1u;    // positions l .. r - 1
        bool join = false;
        for (int k = 0; l < r && !join; ++k) {
            unsigned lo = kNone, hi = 0u;
            if (r - l < 2u * kFan || k + 1 == kFanLevels) {
                for (; l < r; ++l) {
                    lo = min(lo, W.lo[k][l]);
                    hi = max(hi, W.hi[k][l]);
                }
            } else {
                for (; l % kFan; ++l) {
                    lo = min(lo, W.lo[k][l]);
                    hi = max(hi, W.hi[k][l]);
                }
                for (; r % kFan; --r) {
                    lo = min(lo, W.lo[k][r - 1u]);
                    hi = max(hi, W.hi[k][r - 1u]);
                }
                l /= kFan;
                r /= kFan;
            }
            join = lo < first || hi > last;
        }
        if (join) W.uf[v] = p;
    }
}

// Shorten the chains of joined tree edges.
__global__ void bb_shorten(BbGraph G, BbWork W)
{
    for (const int v : each(G.n)) {
        if (!W.adj[v]) continue;
        int p = uf_get(W.uf, v);
        const int was = p;
        if (p == v) continue;
        for (int k = 0; k < 4; ++k) {
            const int q = uf_get(W.uf, p);
            if (q == p) break;
            p = q;
        }
        if (p != was) __hip_atomic_store(W.uf + v, p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

__device__ __forceinline__ bool ancestor(const BbWork &W, int a, int v)
{
    return W.in[a] <= W.in[v] && W.in[v] <= W.last[a];
}

// Joins across non-tree edges, each from its -k end (and from the node of an
// edge to T).
__global__ void bb_join_cross(BbGraph G, BbWork W)
{
    for (const int v : each(G.n)) {
        if (!W.adj[v]) continue;
        int c[3];
        coords(G, v, c);
        for (int e = 0; e < 2 * G.dim; ++e) {
            const int w = bb_nbr(G, v, c, e);
            if (w < 0 || w == G.S || (w < G.n && !(e & 1)) || is_tree(G, W, v, w, e)) continue;
            if (!ancestor(W, w, v) && !ancestor(W, v, w)) uf_union_tour(W.uf, W.in, v, w);
        }
    }
}

// 5. Lattice ends of the tree edges in T's class.
__global__ void bb_mark(BbGraph G, BbWork W, uint8_t *on)
{
    const int rt = uf_find(W.uf, G.T);
    for (const int v : each(G.n)) {
        if (!W.adj[v] || uf_find(W.uf, v) != rt) continue;
        on[v] = 1;
        int c[3];
        coords(G, v, c);
        const int p = tree_parent(G, W, v, c);
        if (p < G.n) on[p] = 1;
    }
}

__global__ void bb_zero(uint8_t *p, int n)
{
    for (const int i : each(n)) p[i] = 0;
}

__global__ void bb_apply(uint8_t *mask, const uint8_t *on, int n, unsigned long long *count)
{
    int c = 0;
    for (const int i : each(n))
        if (on[i]) {
            mask[i] |= 8u;
            ++c;
        }
    // one atomic per workgroup (one per wave, on one address, took 0.4 ms)
    __shared__ int part[kBbBlock / 64];
    for (int o = 32; o > 0; o >>= 1) c += __shfl_down(c, o, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBbBlock / 64; ++w) c += part[w];
        if (c) atomicAdd(count, (unsigned long long)c);
    }
}

// ---------------------------------------------------------------- solves on the backbone
// With the backbone marked (11) and the other live nodes dangling (3), a solve
// may cut the dangling ends out: they carry no current, so the backbone's
// pressures and every flux are unchanged. Each connected piece of dangling
// nodes meets the backbone at exactly one node a (a piece joined to two
// backbone nodes, or to a face and the backbone, would lie on a path that
// visits no node twice) and, carrying no current, sits at a's pressure.

// Pieces of dangling nodes: union over occupied bonds between two of them.
__global__ void bb_piece_union(BbGraph G, int *uf, int *att)
{
    for (const int i : each(G.n)) {
        if (G.mask[i] != 3) continue;
        att[i] = -1;
        int c[3];
        coords(G, i, c);
        for (int d = 1; d < 2 * G.dim; d += 2) {           // each bond once, from its -k end
            const int w = bb_nbr(G, i, c, d);               // a dangling neighbour (mask 3), or S, T, -1
            if (w >= 0 && w < G.n) uf_union(uf, i, w);
        }
    }
}

// The backbone node each piece hangs from, stored at the piece's root (every
// dangling node next to it writes the same index).
__global__ void bb_piece_attach(BbGraph G, int *uf, int *att)
{
    for (const int i : each(G.n)) {
        if (G.mask[i] != 3) continue;
        int c[3];
        coords(G, i, c);
        for (int d = 0; d < 2 * G.dim; ++d) {
            double gij = 0.0;
            const int j = lat_step(G, i, c, d, &gij);
            if (j >= 0 && gij > 0.0 && G.mask[j] == 11) att[uf_find(uf, i)] = j;
        }
    }
}

// Zero every bond with a dangling end (in place: entry g[k][i] is the bond
// from i to its +k neighbour).
__global__ void bb_prune(BbGraph G, double *g0, double *g1, double *g2)
{
    double *gk[3] = {g0, g1, g2};
    for (const int i : each(G.n)) {
        int c[3];
        coords(G, i, c);
        const bool di = G.mask[i] == 3;
        for (int k = 0; k < G.dim; ++k) {
            double gij = 0.0;
            const int j = lat_step(G, i, c, 2 * k + 1, &gij);
            if (j >= 0 && (di || G.mask[j] == 3)) gk[k][i] = 0.0;
        }
    }
}

// Pressures of the dangling nodes: that of the backbone node their piece hangs from.
__global__ void bb_fill(const uint8_t *mask, int *uf, const int *att, double *P, int n)
{
    for (const int i : each(n)) {
        if (mask[i] != 3) continue;
        const int a = att[uf_find(uf, i)];
        if (a >= 0) P[i] = P[a];
    }
}

__global__ void bb_iota(int *uf, int n)
{
    for (const int i : each(n)) uf[i] = i;
}

BbGraph graph_of(const Lat &L, const double *const g[3], const uint8_t *mask)
{
    BbGraph G;
    for (int k = 0; k < 3; ++k) G.g[k] = k < L.dim ? g[k] : nullptr;
    G.mask = mask;
    G.dim = L.dim;
    G.axis = L.axis;
    G.nx = L.nx;
    G.ny = L.ny;
    G.nz = L.nz;
    G.wrap = L.wrap;
    G.n = (int)L.n;
    G.S = (int)L.n;
    G.T = (int)L.n + 1;
    return G;
}

int grid_of(int64_t n)
{
    return (int)std::max<int64_t>(1, std::min<int64_t>((n + kBbBlock - 1) / kBbBlock, 8192));
}

}  // namespace

namespace {

// Carves the arrays of the search from `scratch`; returns the bytes used. The
// walkers' arrays lie where the hierarchy of minima and maxima comes later.
size_t backbone_layout(int64_t n, char *scratch, BbWork *W)
{
    const size_t V = (size_t)n + 2;
    // small lattices: arrays packed closer, so that their rounding does not
    // exceed the 34 bytes a node that the search may take
    const size_t pad = n < 4096 ? 63 : 255;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char *r = scratch + off;
        off += (bytes + pad) & ~pad;
        return r;
    };
    W->tree = (uint8_t *)take(V);
    W->adj = (uint8_t *)take(V);
    W->in = (unsigned *)take(4 * V);
    W->last = (unsigned *)take(4 * V);
    W->uf = (int *)take(4 * V);
    W->counter = (unsigned *)take(256);
    const size_t shared = off;
    // walkers: one per group and per component that touches both faces (at
    // most one per node next to the inlet, and none has fewer than one node)
    W->groups = (int)((n + kSpread - 1) / kSpread);
    const size_t walkers = (size_t)W->groups + (size_t)(n + 2) / 3;
    for (auto &j : W->jump) j = (unsigned long long *)take(8 * walkers);
    W->len = (unsigned *)take(4 * walkers);
    W->end = (unsigned *)take(4 * walkers);
    W->heads = (unsigned *)take(4 * ((size_t)(n + 2) / 3));
    W->first = (int *)take(4 * (size_t)W->groups);
    const size_t one = off;
    off = shared;
    size_t m = 2 * V;                                // positions: a component of k nodes has 2 k - 1
    for (int l = 0; l < kFanLevels; ++l) {
        W->lo[l] = (unsigned *)take(4 * m);
        W->hi[l] = (unsigned *)take(4 * m);
        if (m <= kFan) break;                        // no level above it is built or read
        m = (m + kFan - 1) / kFan;
    }
    return std::max(off, one);
}

}  // namespace

size_t backbone_scratch_bytes(int64_t n)
{
    BbWork W;
    return backbone_layout(n, nullptr, &W);
}

uint8_t *backbone_tree(int64_t n, void *scratch)
{
    BbWork W;
    backbone_layout(n, (char *)scratch, &W);
    return W.tree;
}

hipError_t launch_backbone(const Lat &L, const double *const g[3], uint8_t *mask, const int *parent, unsigned *flags,
                           void *scratch, unsigned long long *n_backbone, hipStream_t st)
{
    const int64_t n = L.n;
    BbWork W;
    backbone_layout(n, (char *)scratch, &W);
    W.parent = parent;
    W.flags = flags;
    const BbGraph G = graph_of(L, g, mask);
    const int gn = grid_of(n), gw = grid_of(W.groups + (n + 2) / 3);
    hipError_t e = launch_clear_u64((unsigned long long *)W.counter, 1, st);
    if (e != hipSuccess) return e;
    bb_tree<<<grid_of(n + 2), kBbBlock, 0, st>>>(G, W);
    bb_starts<<<grid_of(W.groups), kBbBlock, 0, st>>>(G, W);
    bb_walk<<<gw, kBbBlock, 0, st>>>(G, W);
    // a component's list has at most one start per group and its head
    int from = 0;
    for (int64_t reach = 1; reach < (int64_t)W.groups + 1; reach *= 4, from ^= 1)
        bb_jump<<<gw, kBbBlock, 0, st>>>(W, from);
    bb_ranges<<<grid_of((n + 2) / 3), kBbBlock, 0, st>>>(W, from);
    bb_number<<<gw, kBbBlock, 0, st>>>(G, W, from);
    bb_clear<<<grid_of(2 * n), kBbBlock, 0, st>>>(G, W);
    bb_reach<<<gn, kBbBlock, 0, st>>>(G, W);
    int64_t m = 2 * (n + 2);
    for (int l = 1; l < kFanLevels && m > kFan; ++l) {
        m = (m + kFan - 1) / kFan;
        bb_level<<<grid_of(m), kBbBlock, 0, st>>>(W, l);
    }
    bb_join_tree<<<gn, kBbBlock, 0, st>>>(G, W);
    for (int64_t reach = 1; reach < n; reach *= 5) bb_shorten<<<gn, kBbBlock, 0, st>>>(G, W);
    bb_join_cross<<<gn, kBbBlock, 0, st>>>(G, W);
    bb_zero<<<gn, kBbBlock, 0, st>>>(W.tree, (int)n);
    bb_mark<<<gn, kBbBlock, 0, st>>>(G, W, W.tree);
    bb_apply<<<std::min(gn, 2048), kBbBlock, 0, st>>>(mask, W.tree, (int)n, n_backbone);
    return hipGetLastError();
}

hipError_t launch_backbone_prune(const Lat &L, const double *const g[3], double *const gw[3], const uint8_t *mask,
                                 int *uf, int *att, hipStream_t st)
{
    const BbGraph G = graph_of(L, g, mask);
    const int gr = grid_of(L.n);
    bb_iota<<<gr, kBbBlock, 0, st>>>(uf, (int)L.n);
    bb_piece_union<<<gr, kBbBlock, 0, st>>>(G, uf, att);
    bb_piece_attach<<<gr, kBbBlock, 0, st>>>(G, uf, att);
    if (gw) bb_prune<<<gr, kBbBlock, 0, st>>>(G, gw[0], gw[1], L.dim == 3 ? gw[2] : nullptr);
    return hipGetLastError();
}

hipError_t launch_backbone_fill(const Lat &L, const uint8_t *mask, int *uf, const int *att, double *P,
                                hipStream_t st)
{
    bb_fill<<<grid_of(L.n), kBbBlock, 0, st>>>(mask, uf, att, P, (int)L.n);
    return hipGetLastError();
}

}  // namespace rn
