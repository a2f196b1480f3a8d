// k_morse.hip -- persistence pairs of dimension 1 reduced on the critical
// cells of a discrete gradient, instead of on all edges and triangles.
//
// Write an edge by its rank r and let L(r) be the vertices joined to both its
// ends by older edges: the triangles of value r are {r, k}, k in L(r), in the
// order of k (Section 2.1).  Three facts shrink the boundary matrix:
//   - Adding the boundaries of older triangles to a triangle's is a column
//     operation of Algorithm 1 (Section 2.2.1) and changes no pair.  An edge
//     r with L(r) not empty may so be replaced, in the boundary of any later
//     triangle, by the two older edges of one triangle {r, k*}; following
//     the replacements down, every edge becomes a sum of edges with empty
//     L: the edges of the relative neighbourhood graph.  Those paired with
//     a vertex may be left out (a cycle is known by its other edges, and
//     the youngest edge of a cycle is never one of them); the rest are the
//     critical edges.
//   - If k and k' in L(r) are joined by an edge older than r, the triangles
//     {a, k, k'} and {b, k, k'} are older than r, and {r, k}, {r, k'} and
//     those two bound the tetrahedron: {r, k'} is then a sum of older
//     triangles' boundaries and {r, k}'s, and pairs with nothing.  So of
//     the triangles of value r only the first of each component of L(r)
//     (as a graph of the edges older than r) matters: the first triangle
//     of all pairs with r (the apparent pair); the first of each other
//     component is a critical triangle.
//   - k* may be any vertex of the component of the apparent triangle, for
//     {r, k*} differs from it by older triangles.  The vertex nearest both
//     ends (least of the larger rank) makes the replacements short: an edge
//     of the 4000-point mixture ends in 6 critical or tree edges on average,
//     52 at most, after at most 13 steps.
// What remains is a matrix of critical edges by critical triangles (294 x 312
// of 99900 x 4995121 for the 1000-point circle, 7828 x 17906 of 799800 x
// 94017474 for the mixture), reduced on its anti-transpose as Section 2.2.2
// has it: a column per critical edge, from the youngest, holding the critical
// triangles above it in order; its pivot is the oldest.
//
//   k_mo_range   the triangles of each edge's value, from one pass over the keys
//   k_mo_snap    the neighbours of every vertex by edges older than each of
//                up to 32 ranks, as bits
//   k_mo_link    per edge, a wave: the edges that replace it, where the
//                snapshots show L(r) to be connected
//   k_mo_split   the other edges: L(r)'s components, the critical triangles
//   k_mo_order   the edges whose L(r) would take long that way, from the list
//                of edges; the critical cells' places in filtration order
//   k_mo_expand  per critical triangle, a wave: its boundary in critical edges
//   k_mo_scan    starts of the columns
//   k_mo_scatter the columns' entries
//   k_mo_reduce  the reduction, a wave per column, without rounds or locks
//   k_mo_emit    the pairs
//
// On the circle and the mixture vr_pairs_dim1 took 28.2 and 36.6 ms as a
// reduction of the full edge columns, a work-group each: one column's chain
// of thousands of additions.  The chains here are a few additions long, and
// it takes 0.15 and 1.4 ms.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "vr.h"
#include "vr_cache.h"
#include "vr_device.h"
#include "vr_morse.h"

#define MO_BLOCK 256
#define MO_WPB (MO_BLOCK / VR_WAVE)
#define MO_NC 8                     // 64-vertex pieces of L(r) a wave holds in registers
#define MO_GEN (VR_MAX_POINTS / VR_WAVE)  // pieces of the largest L(r)
#define MO_STACK 1024               // edges a wave is replacing, and critical edges it found
#define MO_STEPS 1024               // replacement steps of one triangle (64 edges each)
#define MO_QCAP (1ll << 22)         // critical triangles at most
#define MO_ENT (1ll << 24)          // column entries at most
#define MO_POOL (1ll << 26)         // words of stored columns at most
#define MO_EB 16                    // edges a wave of k_mo_link takes, in order
#define MO_SNAPS 32                 // ranks with a snapshot at most
#define MO_LDS_FEW 17               // log2 of the critical triangles whose bits a wave holds in LDS,
#define MO_LDS_MANY 19              // by the number of triangles
#define MO_NONE 0xFFFFFFFFu

// Counters that waves all over the chip add to come MO_REG times, a cache
// line each, with a share of the array they number: atomics on one address
// follow one another at about 10 ns.
#define MO_REG 16
struct MoCtl {
    uint32_t err;   // a limit was passed
    uint32_t q;     // critical triangles
    uint32_t m;     // critical edges
    uint32_t any;   // there are critical edges
    unsigned long long ptop;  // pool words taken
    uint32_t wide;  // edges left to k_mo_order
    uint32_t ends;  // its work-groups that are done with them
    uint32_t pad1[24];
    uint32_t rec[MO_REG][32];  // [i][0]: critical triangles found, in share i
    uint32_t ent[MO_REG][32];  // [i][0]: column entries, in share i
};

struct MoBufs {
    const int32_t *R, *ij, *e_low;
    const unsigned long long *key;
    int64_t n, K, T;
    int32_t *first, *end;           // K: the triangles of value r are [first, end); first -1: none
    int2 *fg;                       // K: the two edges that replace r; x = -1: none, and y = its place
                                    // among its block's critical edges, or -1
    unsigned long long *snap;       // snapshot s >= 1 of vertex v: words [((s - 1) n + v) W, + W), the
                                    // neighbours joined by an edge of rank < s << sb
    int W, sb;
    uint32_t *blk, *blkm;           // per MO_EB edges: their critical triangles (edges), then the first's place
    uint32_t *mask;                 // per MO_EB edges: those left to k_mo_split
    uint32_t *ecnt;                 // K, for the edges left to k_mo_split: their critical triangles
    uint32_t *crit;                 // column -> edge; before, the edges left to k_mo_order
    uint32_t *cnt, *fill;           // column -> entries, entries placed
    uint32_t *start;                // column -> its first pool word (the length, then the entries)
    uint4 *rec;                     // critical triangle as found: edge, vertex, index among the keys, place in its edge
    uint32_t *ctri;                 // critical triangle (by place) -> its index among the keys
    unsigned long long *owner;      // critical triangle -> (edge + 1) << 32 | pool word of its column; 0: none
    uint2 *ent;                     // (column, critical triangle) pairs; later the bits of k_mo_reduce's waves
    uint32_t *pool;                 // columns: the length, then the critical triangles in any order
    MoCtl *ctl;
    uint32_t qcap, ecap, pcap;
};

// Orders a wave's LDS (and, for later loads of its own, global) accesses.
__device__ __forceinline__ void mo_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

__device__ __forceinline__ uint32_t mo_before(unsigned long long m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Bound by reading the keys once (8 T bytes); two keys a thread.  The edges
// enter R here too: 14.7 -> 16.4 us for 99900 edges, whose launch of their own
// took 4.8; for 799800 177 -> 201, and 22.
__global__ __launch_bounds__(MO_BLOCK) void k_mo_range(MoBufs B, int32_t *R) {
    const int64_t np = (B.T + 1) / 2;
    for (int64_t r = (int64_t)blockIdx.x * MO_BLOCK + threadIdx.x; r < B.K; r += (int64_t)gridDim.x * MO_BLOCK)
        vr_rank_edge(R, B.ij, B.n, r);
    for (int64_t p = (int64_t)blockIdx.x * MO_BLOCK + threadIdx.x; p < np; p += (int64_t)gridDim.x * MO_BLOCK) {
        const int64_t t = 2 * p;
        const bool two = t + 1 < B.T;
        const unsigned long long k0 = B.key[t], k1 = two ? B.key[t + 1] : k0;
        const int64_t v0 = (int64_t)(k0 >> 39), v1 = (int64_t)(k1 >> 39);
        const int64_t u = t > 0 ? (int64_t)(B.key[t - 1] >> 39) : -1;
        if (u != v0) {
            if (v0 < B.K) B.first[v0] = (int32_t)t;
            if (u >= 0 && u < B.K) B.end[u] = (int32_t)t;
        }
        if (v1 != v0) {
            if (v1 < B.K) B.first[v1] = (int32_t)(t + 1);
            if (v0 < B.K) B.end[v0] = (int32_t)(t + 1);
        }
        if (t + 2 >= B.T && v1 < B.K) B.end[v1] = (int32_t)B.T;
    }
}

// The vertex of triangle key w off its largest edge {a, b}, a < b.
__device__ __forceinline__ uint32_t mo_third(unsigned long long w, uint32_t a, uint32_t b) {
    const uint32_t i = (uint32_t)(w >> 26) & 0x1FFFu, j = (uint32_t)(w >> 13) & 0x1FFFu, k = (uint32_t)w & 0x1FFFu;
    return i != a ? i : (j != b ? j : k);
}

// Lane 0 records the critical triangle {r, k}, the place-th of its edge.
__device__ __forceinline__ void mo_append(const MoBufs &B, uint32_t r, uint32_t k, uint32_t tri, uint32_t place) {
    if (lane_id() != 0) return;
    const uint32_t i = blockIdx.x % MO_REG, share = B.qcap / MO_REG;
    const uint32_t q = atomicAdd(&B.ctl->rec[i][0], 1u);
    if (q < share) B.rec[(size_t)i * share + q] = make_uint4(r, k, tri, place);
    else B.ctl->err = 1u;
}

// Searching L(r) vertex by vertex reads a row of the rank matrix each, and
// when it falls into many components, or into two large ones, nearly every
// vertex has its turn: one wave took 474 ms for an edge with 8000 common
// neighbours, no two of them joined (27 ms by the columns' reduction).  The
// edges older than r, a work-group's pass over them, give the components in
// 6 us and 0.1 ns an edge (k_mo_order).  A search counts half microseconds, one
// for a vertex of up to 512 (a piece of 64 beyond) and five for a component,
// and leaves the edge to that pass after MO_WIDE and one more per 1024 edges
// older than r, several times what the pass takes.  (A third of that sent the 4000-point mixture's
// few long searches there too: 24 us less here and 74 there.)
// us of vr_pairs_dim1 on such an edge, 400, 1000, 2049 and 8000 neighbours:
// 1386, 7615, 28403 and 474211 without the pass, 559, 888, 1498 and 5597 with
// it (1735, 4127, 7853 and 27304 by the columns' reduction).
#define MO_WIDE 384
#define MO_WIDE_COMP 5
__device__ __forceinline__ int mo_allowed(uint32_t r) { return (int)(MO_WIDE + r / 1024); }
// No search of so few vertices gets that far.
static bool mo_wide_may(int64_t n) { return (n - 2) * (MO_WIDE_COMP + 1) > MO_WIDE; }

// Lane 0 leaves edge r to k_mo_order, `place` of its critical triangles found:
// those of the first components, for they come in order.
__device__ __forceinline__ void mo_defer(const MoBufs &B, uint32_t r, uint32_t place) {
    if (lane_id() != 0) return;
    B.ecnt[r] = place;
    B.crit[atomicAdd(&B.ctl->wide, 1u)] = r;
}

// The critical triangles of one edge, in the order of their vertices: the
// components come with rising first vertices but for the one the search
// began with, which waits for its turn.
struct MoPending {
    uint32_t x;  // its first vertex (position in L(r)), MO_NONE: none
    uint32_t k;
};

// The least (rank, position) over the wave of the lanes' ranks x (INT_MAX:
// none) at positions i: the rank; *at = its position.
__device__ __forceinline__ int32_t mo_wave_min(int32_t x, uint32_t i, uint32_t *at) {
    int32_t v = x;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o, VR_WAVE));
    const unsigned long long m = ballot64(x == v);
    *at = (uint32_t)__builtin_amdgcn_readlane((int)i, m ? __builtin_ctzll(m) : 0);
    return v;
}

// L(r) of any size: its pieces read again from the keys at each step, the
// sets as bit masks in the wave's LDS (reached, to expand, this component).
// x < 0: the search was given up.
__device__ int2 mo_link_any(const MoBufs &B, uint32_t r, uint32_t a, uint32_t b, int32_t f0, uint32_t m,
                            unsigned long long *reach, unsigned long long *open, unsigned long long *comp,
                            uint32_t &place) {
    const uint32_t lane = lane_id();
    const uint32_t np = (m + VR_WAVE - 1) / VR_WAVE;
    const int32_t *Ra = B.R + (int64_t)a * B.n, *Rb = B.R + (int64_t)b * B.n;
    auto vertex = [&](uint32_t x) { return mo_third(B.key[f0 + min(x, m - 1)], a, b); };
    // least larger rank over the members of `comp` (all: over every vertex)
    auto nearest = [&](bool all, int32_t *fx, int32_t *fy) {
        int32_t best = INT32_MAX;
        uint32_t bx = 0;
        for (uint32_t p = 0; p < np; p++) {
            const uint32_t x = p * VR_WAVE + lane;
            const uint32_t k = vertex(x);
            const bool in = x < m && (all || ((comp[p] >> lane) & 1ull));
            const int32_t v = in ? max(Ra[k], Rb[k]) : INT32_MAX;
            if (v < best) {
                best = v;
                bx = x;
            }
        }
        uint32_t at;
        (void)mo_wave_min(best, bx, &at);
        const uint32_t k = vertex(at);
        *fx = Ra[k];
        *fy = Rb[k];
        return at;
    };
    int32_t fx, fy;
    uint32_t seed = nearest(true, &fx, &fy);
    for (uint32_t p = lane; p < np; p += VR_WAVE) reach[p] = 0ull;
    mo_wave_sync();
    uint32_t left = m;
    bool first_comp = true;
    MoPending pend{MO_NONE, 0u};
    int allowed = mo_allowed(r);
    while (left > 0) {
        for (uint32_t p = lane; p < np; p += VR_WAVE) open[p] = comp[p] = 0ull;
        mo_wave_sync();
        uint32_t y = seed;
        for (;;) {
            if ((allowed -= (int)np) < 0) return make_int2(-1, -1);
            const int32_t *Ry = B.R + (int64_t)vertex(y) * B.n;
            uint32_t got = 0;
            for (uint32_t p = 0; p < np; p++) {
                const uint32_t x = p * VR_WAVE + lane;
                const unsigned long long old = reach[p];
                const uint32_t k = vertex(x);
                const bool hit = x < m && !((old >> lane) & 1ull) && Ry[k] < (int32_t)r;
                const unsigned long long h = ballot64(hit);
                if (h) {
                    mo_wave_sync();
                    if (lane == 0) {
                        reach[p] = old | h;
                        open[p] |= h;
                        comp[p] |= h;
                    }
                    got += (uint32_t)__popcll(h);
                }
            }
            left -= got;
            mo_wave_sync();
            if (lane == 0) open[y / VR_WAVE] &= ~(1ull << (y % VR_WAVE));
            mo_wave_sync();
            if (left == 0) break;
            // the next vertex of the component not yet expanded
            y = MO_NONE;
            for (uint32_t p = 0; p < np && y == MO_NONE; p++)
                if (open[p]) y = p * VR_WAVE + (uint32_t)__builtin_ctzll(open[p]);
            if (y == MO_NONE) break;
        }
        allowed -= MO_WIDE_COMP;
        // the component's first vertex; the component of vertex 0 is the apparent triangle's
        uint32_t lo = 0;
        while (!comp[lo]) lo++;
        const uint32_t x0 = lo * VR_WAVE + (uint32_t)__builtin_ctzll(comp[lo]);
        if (pend.x < x0 && x0 != 0) {
            mo_append(B, r, pend.k, (uint32_t)f0 + pend.x, place++);
            pend.x = MO_NONE;
        }
        if (x0 == 0) {
            if (!first_comp) (void)nearest(false, &fx, &fy);
        } else if (first_comp) {
            pend = MoPending{x0, vertex(x0)};
        } else {
            mo_append(B, r, vertex(x0), (uint32_t)f0 + x0, place++);
        }
        first_comp = false;
        if (left > 0) {
            seed = 0;
            for (uint32_t p = 0;; p++) {
                const unsigned long long full = p + 1 < np || m % VR_WAVE == 0 ? ~0ull : (1ull << (m % VR_WAVE)) - 1;
                const unsigned long long un = full & ~reach[p];
                if (un) {
                    seed = p * VR_WAVE + (uint32_t)__builtin_ctzll(un);
                    break;
                }
            }
        }
        mo_wave_sync();
    }
    if (pend.x != MO_NONE) mo_append(B, r, pend.k, (uint32_t)f0 + pend.x, place++);
    return make_int2(fx, fy);
}

// Up to MO_SNAPS snapshots of every vertex's older neighbours, one work-group
// per vertex: the row's ranks set bits by the snapshot they first appear in,
// and the snapshots are the running unions.  Bound by writing them: 4 n^2
// bytes at 32 snapshots.
// Critical edges are looked for here too.  Where there is none (ultrametrics,
// trees) every triangle that pairs is apparent, and the kernels that follow
// have nothing to do: 512 points of an ultrametric, 22238720 triangles,
// 312 us of vr_pairs_dim1 with them, 104 now (222 by the columns' reduction).
__global__ __launch_bounds__(MO_BLOCK) void k_mo_snap(MoBufs B, int S) {
    extern __shared__ uint32_t sbits[];  // S x 2 W
    const int64_t v = blockIdx.x;
    const int32_t *row = B.R + v * B.n;
    const int w2 = 2 * B.W;
    bool any = false;
    for (int64_t r = v * MO_BLOCK + threadIdx.x; r < B.K; r += B.n * MO_BLOCK) any |= B.first[r] < 0 && B.e_low[r] < 0;
    if (any) B.ctl->any = 1u;
    for (int x = threadIdx.x; x < S * w2; x += MO_BLOCK) sbits[x] = 0u;
    __syncthreads();
    for (int64_t k = threadIdx.x; k < B.n; k += MO_BLOCK) {
        const int32_t r = row[k];
        if (k != v && r != INT32_MAX && (r >> B.sb) < S)
            atomicOr(&sbits[(r >> B.sb) * w2 + (int)(k >> 5)], 1u << (k & 31));
    }
    __syncthreads();
    for (int x = threadIdx.x; x < B.W; x += MO_BLOCK) {
        unsigned long long u = 0;
        for (int s = 0; s < S; s++) {
            u |= ((unsigned long long)sbits[s * w2 + 2 * x + 1] << 32) | sbits[s * w2 + 2 * x];
            B.snap[((int64_t)s * B.n + v) * B.W + x] = u;
        }
    }
}

// Whether L(r) is connected by the edges of a snapshot older than r: bits
// of L(r) in the lanes (l0, l1: words lane and 64 + lane), searched on, four
// rows at a time, from the vertices reached (g) of which some were expanded
// (e).  Fewer edges than r allows, so "no" only means that it must be
// looked at again.
template <int NW>
__device__ __forceinline__ bool mo_connected(const MoBufs &B, uint32_t snap, unsigned long long l0,
                                             unsigned long long l1, unsigned long long g0, unsigned long long g1,
                                             unsigned long long e0, unsigned long long e1) {
    const uint32_t lane = lane_id();
    const unsigned long long *rows = B.snap + (int64_t)(snap - 1) * B.n * B.W;
    constexpr bool two = NW > 1;
    const bool w0 = (int)lane < B.W, w1 = two && (int)lane + VR_WAVE < B.W;
    for (;;) {
        const unsigned long long o0 = g0 & ~e0, o1 = g1 & ~e1;  // reached, not expanded
        const unsigned long long b0 = ballot64(o0 != 0ull), b1 = two ? ballot64(o1 != 0ull) : 0ull;
        if (!(b0 | b1)) return false;
        uint32_t v[4];
        unsigned long long x0 = b0, x1 = b1;
        int nv = 0;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            v[i] = i ? v[0] : 0u;
            if (x0) {
                const int src = __builtin_ctzll(x0);
                x0 &= x0 - 1;
                const unsigned long long word =
                    ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(o0 >> 32), src) << 32) |
                    (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)o0, src);
                v[i] = (uint32_t)src * 64 + (uint32_t)__builtin_ctzll(word);
                if ((int)lane == src) e0 |= 1ull << (v[i] & 63);
                nv = i + 1;
            } else if (x1) {
                const int src = __builtin_ctzll(x1);
                x1 &= x1 - 1;
                const unsigned long long word =
                    ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(o1 >> 32), src) << 32) |
                    (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)o1, src);
                v[i] = (uint32_t)(src + VR_WAVE) * 64 + (uint32_t)__builtin_ctzll(word);
                if ((int)lane == src) e1 |= 1ull << (v[i] & 63);
                nv = i + 1;
            }
        }
        unsigned long long a0 = 0, a1 = 0;
#pragma unroll
        for (int i = 0; i < 4; i++)
            if (i < nv) {
                const unsigned long long *row = rows + (int64_t)v[i] * B.W;
                if (w0) a0 |= row[lane];
                if (two && w1) a1 |= row[VR_WAVE + lane];
            }
        g0 |= a0 & l0;
        if (two) g1 |= a1 & l1;
        if (!ballot64((l0 & ~g0) != 0ull || (l1 & ~g1) != 0ull)) return true;
    }
}

// A wave takes MO_EB edges.  The vertices of L(r) come from the triangles
// of value r.  Nearly every L(r) is connected by the edges of the last
// snapshot before r, which a few rows of 8 W bytes show: those of four of
// its vertices, then four at a time.  The others, and the edges before the
// first snapshot, go to k_mo_split: one in 20 at the mixture.  k* is the
// nearest to both ends of eight vertices, two runs of four: bound by the
// lines it reads, and a run's ranks lie in few.  At the mixture 32 single
// vertices took 1015 us, four runs of eight 790, these 478, and the
// replacements are followed to their ends in the same 37 us (k_mo_expand).
// Two edges at a time, their loads issued together.  With exact searches in
// the rank matrix, a line per vertex and row, it took 3890 us.
template <int NW>
__global__ __launch_bounds__(MO_BLOCK) void k_mo_link(MoBufs B) {
    constexpr int U = 2;
    __shared__ unsigned long long sbits[MO_WPB][U][NW * VR_WAVE];
    const uint32_t lane = lane_id(), w = threadIdx.x / VR_WAVE;
    const int64_t blk = (int64_t)blockIdx.x * MO_WPB + w;
    const int64_t r0 = blk * MO_EB;
    if (r0 >= B.K || !B.ctl->any) return;
    // the block's edges, one a lane
    const int64_t rl = r0 + lane;
    const bool in = lane < MO_EB && rl < B.K;
    int32_t f0 = -1, f1 = -1, ea = 0, eb = 0;
    bool crit = false;
    if (in) {
        f0 = B.first[rl];
        f1 = B.end[rl];
        ea = B.ij[2 * rl];
        eb = B.ij[2 * rl + 1];
        crit = f0 < 0 && B.e_low[rl] < 0;
    }
    const unsigned long long mc = ballot64(crit), mt = ballot64(in && f0 >= 0);
    if (in && f0 < 0) B.fg[rl] = make_int2(-1, crit ? (int32_t)mo_before(mc) : -1);
    // edges before the first snapshot
    const unsigned long long early = mt & ballot64(in && (rl >> B.sb) == 0);
    unsigned long long todo = mt & ~early, left = early;
    while (todo) {
        uint32_t ix[U], sk[U], r[U], m[U], v[U][4];
        int32_t f[U], sr[U], xa[U], xb[U];
        unsigned long long row[U][4][NW];
#pragma unroll
        for (int u = 0; u < U; u++) {
            ix[u] = todo ? (uint32_t)__builtin_ctzll(todo) : ix[0];
            todo &= todo - 1;  // 0 stays 0
            r[u] = (uint32_t)r0 + ix[u];
            f[u] = __builtin_amdgcn_readlane(f0, (int)ix[u]);
            m[u] = (uint32_t)(__builtin_amdgcn_readlane(f1, (int)ix[u]) - f[u]);
            xa[u] = __builtin_amdgcn_readlane(ea, (int)ix[u]);
            xb[u] = __builtin_amdgcn_readlane(eb, (int)ix[u]);
        }
        unsigned long long ks[U], k0[U], k1[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            ks[u] = B.key[f[u] + (int32_t)min(((lane >> 2) & 1u) * (m[u] / 2) + (lane & 3u), m[u] - 1)];
            k0[u] = B.key[f[u] + (int32_t)min(lane, m[u] - 1)];
            k1[u] = B.key[f[u] + (int32_t)min(lane + VR_WAVE, m[u] - 1)];
        }
        mo_wave_sync();  // the bits of the edges before have been read
#pragma unroll
        for (int u = 0; u < U; u++)
#pragma unroll
            for (int i = 0; i < NW; i++) sbits[w][u][i * VR_WAVE + lane] = 0ull;
        mo_wave_sync();
#pragma unroll
        for (int u = 0; u < U; u++) {
            sk[u] = mo_third(ks[u], (uint32_t)xa[u], (uint32_t)xb[u]);
            sr[u] = B.R[(int64_t)(lane < 32 ? xa[u] : xb[u]) * B.n + sk[u]];
            const unsigned long long *rows = B.snap + (int64_t)((r[u] >> B.sb) - 1) * B.n * B.W;
#pragma unroll
            for (int i = 0; i < 4; i++) {
                v[u][i] = (uint32_t)__builtin_amdgcn_readlane((int)sk[u], 2 * i);
#pragma unroll
                for (int j = 0; j < NW; j++)
                    row[u][i][j] = (int)lane + j * VR_WAVE < B.W ? rows[(int64_t)v[u][i] * B.W + j * VR_WAVE + lane] : 0ull;
            }
        }
#pragma unroll
        for (int u = 0; u < U; u++) {
            const uint32_t a = (uint32_t)xa[u], b = (uint32_t)xb[u];
            // positions past the list repeat its last vertex
            uint32_t k = mo_third(k0[u], a, b);
            atomicOr(&sbits[w][u][k >> 6], 1ull << (k & 63));
            k = mo_third(k1[u], a, b);
            if (m[u] > VR_WAVE) atomicOr(&sbits[w][u][k >> 6], 1ull << (k & 63));
            for (uint32_t x = 2 * VR_WAVE; x < m[u]; x += VR_WAVE) {
                k = mo_third(B.key[f[u] + (int32_t)min(x + lane, m[u] - 1)], a, b);
                atomicOr(&sbits[w][u][k >> 6], 1ull << (k & 63));
            }
        }
        mo_wave_sync();
#pragma unroll
        for (int u = 0; u < U; u++) {
            if (u > 0 && ix[u] == ix[0]) continue;
            const unsigned long long l0 = sbits[w][u][lane], l1 = NW > 1 ? sbits[w][u][(NW - 1) * VR_WAVE + lane] : 0ull;
            auto bit = [&](uint32_t k, int j) {
                return lane + (uint32_t)j * VR_WAVE == (k >> 6) ? 1ull << (k & 63) : 0ull;
            };
            unsigned long long g0 = bit(v[u][0], 0), g1 = NW > 1 ? bit(v[u][0], 1) : 0ull, e0 = g0, e1 = g1;
            g0 |= row[u][0][0] & l0;
            if (NW > 1) g1 |= row[u][0][NW - 1] & l1;
#pragma unroll
            for (int i = 1; i < 4; i++) {
                const unsigned long long b0 = bit(v[u][i], 0), b1 = NW > 1 ? bit(v[u][i], 1) : 0ull;
                if (ballot64(((g0 & b0) | (g1 & b1)) != 0ull)) {  // reached: its row counts too
                    g0 |= row[u][i][0] & l0;
                    if (NW > 1) g1 |= row[u][i][NW - 1] & l1;
                    e0 |= b0;
                    e1 |= b1;
                }
            }
            bool all = !ballot64((l0 & ~g0) != 0ull || (l1 & ~g1) != 0ull);
            if (!all) all = mo_connected<NW>(B, r[u] >> B.sb, l0, l1, g0, g1, e0, e1);
            if (!all) {
                left |= 1ull << ix[u];
                continue;
            }
            const int32_t own = max(sr[u], __shfl_xor(sr[u], 32, VR_WAVE));
            int32_t best = own;
#pragma unroll
            for (int o = 16; o > 0; o >>= 1) best = min(best, __shfl_xor(best, o, VR_WAVE));
            const int at = __builtin_ctzll(ballot64(own == best));  // below 32
            const int32_t fx = __builtin_amdgcn_readlane(sr[u], at), fy = __builtin_amdgcn_readlane(sr[u], at + 32);
            if (lane == 0) B.fg[r[u]] = make_int2(fx, fy);
        }
    }
    if (lane == 0) {
        B.mask[blk] = (uint32_t)left;
        B.blk[blk] = 0u;
        B.blkm[blk] = (uint32_t)__popcll(mc);
    }
}

// The edges whose L(r) no snapshot showed to be connected, a block's by the
// waves of a work-group in turn: searched in the rank matrix from the vertex
// nearest both ends, component after component.
__global__ __launch_bounds__(MO_BLOCK) void k_mo_split(MoBufs B) {
    __shared__ unsigned long long masks[MO_WPB][3][MO_GEN];
    const uint32_t lane = lane_id(), w = threadIdx.x / VR_WAVE;
    const int64_t blk = blockIdx.x;
    if (!B.ctl->any) return;
    uint32_t left = (uint32_t)__builtin_amdgcn_readfirstlane((int)B.mask[blk]), turn = 0;
    for (; left; left &= left - 1, turn++) {
        if (turn % MO_WPB != w) continue;
        const uint32_t r = (uint32_t)(blk * MO_EB) + (uint32_t)__builtin_ctz(left);
        const int32_t f0 = B.first[r];
        uint32_t place = 0;  // critical triangles of the edge so far
        auto done = [&](int32_t fx, int32_t fy) {
            if (lane == 0) {
                B.fg[r] = make_int2(fx, fy);
                B.ecnt[r] = place;
                if (place) atomicAdd(&B.blk[blk], place);
            }
        };
        const uint32_t m = (uint32_t)(B.end[r] - f0);
        const uint32_t a = (uint32_t)B.ij[2 * (int64_t)r], b = (uint32_t)B.ij[2 * (int64_t)r + 1];
        if (m > MO_NC * VR_WAVE) {
            const int2 f = mo_link_any(B, r, a, b, f0, m, masks[w][0], masks[w][1], masks[w][2], place);
            if (f.x < 0) mo_defer(B, r, place);
            else done(f.x, f.y);
            continue;
        }
        const int32_t *Ra = B.R + (int64_t)a * B.n, *Rb = B.R + (int64_t)b * B.n;
        uint32_t kk[MO_NC];
        int32_t mm[MO_NC];
        unsigned long long todo[MO_NC];  // vertices not reached yet
#pragma unroll
        for (int i = 0; i < MO_NC; i++) {
            kk[i] = 0;
            todo[i] = 0ull;
            if ((uint32_t)i * VR_WAVE < m) {
                kk[i] = mo_third(B.key[f0 + min((uint32_t)i * VR_WAVE + lane, m - 1)], a, b);
                const uint32_t left = m - (uint32_t)i * VR_WAVE;
                todo[i] = left >= VR_WAVE ? ~0ull : (1ull << left) - 1;
            }
        }
        int32_t best = INT32_MAX;
        uint32_t bx = 0;
#pragma unroll
        for (int i = 0; i < MO_NC; i++) {
            mm[i] = INT32_MAX;
            if ((uint32_t)i * VR_WAVE < m) {
                const int32_t v = max(Ra[kk[i]], Rb[kk[i]]);
                if ((todo[i] >> lane) & 1ull) mm[i] = v;
                if (mm[i] < best) {
                    best = mm[i];
                    bx = (uint32_t)i * VR_WAVE + lane;
                }
            }
        }
        uint32_t seed;
        (void)mo_wave_min(best, bx, &seed);
        auto vertex = [&](uint32_t x) {  // x uniform
            uint32_t k = 0;
#pragma unroll
            for (int i = 0; i < MO_NC; i++)
                if (x / VR_WAVE == (uint32_t)i) k = (uint32_t)__builtin_amdgcn_readlane((int)kk[i], (int)(x % VR_WAVE));
            return k;
        };
        uint32_t kstar = vertex(seed);
        bool first_comp = true;
        MoPending pend{MO_NONE, 0u};
        int allowed = mo_allowed(r);
        bool wide = false;
        for (;;) {
            unsigned long long open[MO_NC], comp[MO_NC];
#pragma unroll
            for (int i = 0; i < MO_NC; i++) open[i] = comp[i] = 0ull;
            uint32_t y = seed;
            bool more = true;
            for (;;) {
                wide = --allowed < 0;
                if (wide) break;
                const int32_t *Ry = B.R + (int64_t)vertex(y) * B.n;
                more = false;
#pragma unroll
                for (int i = 0; i < MO_NC; i++)
                    if (todo[i]) {
                        const unsigned long long h = ballot64(Ry[kk[i]] < (int32_t)r) & todo[i];
                        todo[i] &= ~h;
                        open[i] |= h;
                        comp[i] |= h;
                        more |= todo[i] != 0ull;
                    }
                if (!more) break;
                uint32_t nx = MO_NONE;
#pragma unroll
                for (int i = 0; i < MO_NC; i++) {
                    if (y / VR_WAVE == (uint32_t)i) open[i] &= ~(1ull << (y % VR_WAVE));
                    if (open[i]) nx = (uint32_t)i * VR_WAVE + (uint32_t)__builtin_ctzll(open[i]);
                }
                if (nx == MO_NONE) break;
                y = nx;
            }
            if (wide) break;
            allowed -= MO_WIDE_COMP;
            // the component's first vertex; that of vertex 0 holds the apparent triangle
            uint32_t x0 = MO_NONE;
#pragma unroll
            for (int i = MO_NC - 1; i >= 0; i--)
                if (comp[i]) x0 = (uint32_t)i * VR_WAVE + (uint32_t)__builtin_ctzll(comp[i]);
            if (pend.x < x0 && x0 != 0) {
                mo_append(B, r, pend.k, (uint32_t)f0 + pend.x, place++);
                pend.x = MO_NONE;
            }
            if (x0 != 0) {
                if (first_comp) pend = MoPending{x0, vertex(x0)};
                else mo_append(B, r, vertex(x0), (uint32_t)f0 + x0, place++);
            } else if (!first_comp) {
                best = INT32_MAX;
                bx = 0;
#pragma unroll
                for (int i = 0; i < MO_NC; i++)
                    if (((comp[i] >> lane) & 1ull) && mm[i] < best) {
                        best = mm[i];
                        bx = (uint32_t)i * VR_WAVE + lane;
                    }
                uint32_t at;
                (void)mo_wave_min(best, bx, &at);
                kstar = vertex(at);
            }
            if (!more) break;
            first_comp = false;
#pragma unroll
            for (int i = MO_NC - 1; i >= 0; i--)
                if (todo[i]) seed = (uint32_t)i * VR_WAVE + (uint32_t)__builtin_ctzll(todo[i]);
        }
        if (wide) {
            mo_defer(B, r, place);
            continue;
        }
        if (pend.x != MO_NONE) mo_append(B, r, pend.k, (uint32_t)f0 + pend.x, place++);
        done(Ra[kstar], Rb[kstar]);
    }
}

// The nh edges left over, a work-group each: the vertices of L(r) in a
// union-find in LDS that the edges older than r join, the smaller position the
// root, so that a root is its component's first vertex.
#define MO_WIDE_BLOCK 1024
#define MO_WIDE_LOADS 8
__device__ __forceinline__ void mo_wide(const MoBufs &B, uint32_t nh) {
    __shared__ uint32_t par[VR_MAX_POINTS];
    __shared__ uint16_t pos[VR_MAX_POINTS];  // vertex -> position in L(r)
    __shared__ uint32_t wsum[MO_WIDE_BLOCK / VR_WAVE];
    __shared__ unsigned long long near0;
    __shared__ uint32_t s_base;
    const uint32_t t = threadIdx.x, lane = lane_id(), w = t / VR_WAVE;
    auto find = [&](uint32_t x) {  // an entry only ever moves up its own path
        for (uint32_t p = par[x]; p != x; p = par[x]) {
            const uint32_t g = par[p];
            if (g != p) par[x] = g;
            x = g;
        }
        return x;
    };
    for (uint32_t h = blockIdx.x; h < nh; h += gridDim.x) {
        const uint32_t r = B.crit[h], m = (uint32_t)(B.end[r] - B.first[r]);
        const int32_t f0 = B.first[r];
        const uint32_t a = (uint32_t)B.ij[2 * (int64_t)r], b = (uint32_t)B.ij[2 * (int64_t)r + 1];
        auto vertex = [&](uint32_t x) { return mo_third(B.key[f0 + x], a, b); };
        __syncthreads();  // the last edge's reads are done
        for (uint32_t k = t; k < (uint32_t)B.n; k += MO_WIDE_BLOCK) pos[k] = 0xFFFFu;
        if (t == 0) near0 = ~0ull;
        __syncthreads();
        for (uint32_t x = t; x < m; x += MO_WIDE_BLOCK) {
            pos[vertex(x)] = (uint16_t)x;
            par[x] = x;
        }
        __syncthreads();
        for (uint32_t e0 = t; e0 < r; e0 += MO_WIDE_LOADS * MO_WIDE_BLOCK) {
            int2 v[MO_WIDE_LOADS];
#pragma unroll
            for (int u = 0; u < MO_WIDE_LOADS; u++) {
                const int64_t e = min(e0 + u * MO_WIDE_BLOCK, r);
                v[u] = make_int2(B.ij[2 * e], B.ij[2 * e + 1]);
            }
#pragma unroll
            for (int u = 0; u < MO_WIDE_LOADS; u++) {
                if (e0 + u * MO_WIDE_BLOCK >= r || (uint32_t)v[u].x >= (uint32_t)B.n || (uint32_t)v[u].y >= (uint32_t)B.n)
                    continue;
                uint32_t x = pos[v[u].x], y = pos[v[u].y];
                if (x == 0xFFFFu || y == 0xFFFFu) continue;
                for (;;) {
                    x = find(x);
                    y = find(y);
                    if (x == y) break;
                    const uint32_t lo = min(x, y), hi = max(x, y);
                    if (atomicCAS(&par[hi], hi, lo) == hi) break;
                }
            }
        }
        __syncthreads();
        // the vertex nearest both ends of the apparent triangle's component
        for (uint32_t x = t; x < m; x += MO_WIDE_BLOCK)
            if (find(x) == 0) {
                const uint32_t k = vertex(x);
                const uint32_t d = (uint32_t)max(B.R[(int64_t)a * B.n + k], B.R[(int64_t)b * B.n + k]);
                atomicMin(&near0, ((unsigned long long)d << 32) | k);
            }
        // the first vertices of the others, in order, from the place-th on
        const uint32_t found = B.ecnt[r];
        uint32_t total = 0;
        for (int pass = 0; pass < 2; pass++) {
            uint32_t run = 0;
            for (uint32_t x0 = 0; x0 < m; x0 += MO_WIDE_BLOCK) {
                const uint32_t x = x0 + t;
                const bool root = x > 0 && x < m && par[x] == x;
                const unsigned long long rm = ballot64(root);
                __syncthreads();
                if (lane == 0) wsum[w] = (uint32_t)__popcll(rm);
                __syncthreads();
                uint32_t at = run + mo_before(rm);
                for (uint32_t i = 0; i < MO_WIDE_BLOCK / VR_WAVE; i++) {
                    if (i < w) at += wsum[i];
                    run += wsum[i];
                }
                if (pass == 1 && root && at >= found && s_base != MO_NONE)
                    B.rec[s_base + at - found] = make_uint4(r, vertex(x), (uint32_t)f0 + x, at);
            }
            if (pass == 1) break;
            total = run;
            if (t == 0) {
                const uint32_t i = r / MO_EB % MO_REG, share = B.qcap / MO_REG, add = total - found;
                const uint32_t q = atomicAdd(&B.ctl->rec[i][0], add);
                const bool room = q + add <= share;
                if (!room) B.ctl->err = 1u;
                s_base = room ? i * share + q : MO_NONE;
                B.ecnt[r] = total;
                if (total) atomicAdd(&B.blk[r / MO_EB], total);
            }
            __syncthreads();
        }
        if (t == 0) {
            const uint32_t k = (uint32_t)near0;
            B.fg[r] = make_int2(B.R[(int64_t)a * B.n + k], B.R[(int64_t)b * B.n + k]);
        }
    }
}

// Exclusive scan by one work-group of 1024 threads, four values a thread:
// v(x) is value x of n, put(x, s) takes the sum before it.  Returns the total.
template <typename V, typename P>
__device__ __forceinline__ uint32_t mo_scan(uint32_t n, V v, P put) {
    __shared__ uint32_t wt[16];
    __shared__ uint32_t carry;
    const uint32_t t = threadIdx.x, wv = t >> 6;
    if (t == 0) carry = 0;
    __syncthreads();
    for (uint32_t base = 0; base < n; base += 4096) {
        uint32_t e[4], own = 0;
#pragma unroll
        for (uint32_t u = 0; u < 4; u++) {
            const uint32_t x = base + 4 * t + u;
            e[u] = x < n ? v(x) : 0u;
            own += e[u];
        }
        const uint32_t inc = wave_incl_scan_dpp(own);
        if ((t & 63) == 63) wt[wv] = inc;
        __syncthreads();
        uint32_t at = carry + inc - own, tot = 0;
        for (uint32_t i = 0; i < 16; i++) {
            if (i < wv) at += wt[i];
            tot += wt[i];
        }
#pragma unroll
        for (uint32_t u = 0; u < 4; u++) {
            const uint32_t x = base + 4 * t + u;
            if (x < n) put(x, at);
            at += e[u];
        }
        __syncthreads();
        if (t == 0) carry += tot;
        __syncthreads();
    }
    return carry;
}

// Places: the blocks' critical triangles (work-group 0) and edges (1).  Edges
// left to the pass over the older ones come first, and then the last
// work-group to end makes both sums: a launch less than with a kernel for
// each, which cost the calls without such edges 4.5 us.
__global__ __launch_bounds__(MO_WIDE_BLOCK) void k_mo_order(MoBufs B) {
    __shared__ uint32_t s_end;
    if (!B.ctl->any) return;
    const uint32_t nb = (uint32_t)((B.K + MO_EB - 1) / MO_EB), nh = B.ctl->wide;
    uint32_t lo = blockIdx.x, hi = lo + 1;
    if (nh > 0) {
        mo_wide(B, nh);
        __syncthreads();
        if (threadIdx.x == 0) {
            __threadfence();
            s_end = atomicAdd(&B.ctl->ends, 1u);
            __threadfence();
        }
        __syncthreads();
        if (s_end + 1 != gridDim.x) return;
        lo = 0;
        hi = 2;
    }
    for (uint32_t i = lo; i < hi && i < 2; i++) {
        uint32_t *p = i == 0 ? B.blk : B.blkm;
        const uint32_t tot = mo_scan(nb, [&](uint32_t x) { return p[x]; }, [&](uint32_t x, uint32_t s) { p[x] = s; });
        if (threadIdx.x == 0) *(i == 0 ? &B.ctl->q : &B.ctl->m) = tot;
    }
}

// One wave per critical triangle {r, k}: the edges ak, bk and r's two
// replacements go on a stack; each lane takes one off it, and its two
// replacements go back, or the critical edge it is into a list.  Edges an
// even number of times in the list cancel.  Any order does, since every
// replacement is older.  The waves take the entries' slots MO_SLOTS at a
// time (one atomic for each triangle, all at one address, took most of 207
// us at the mixture) and mark those they leave.
#define MO_SLOTS 128
__global__ __launch_bounds__(MO_BLOCK) void k_mo_expand(MoBufs B) {
    __shared__ uint32_t s_stack[MO_WPB][MO_STACK];
    __shared__ uint32_t s_list[MO_WPB][MO_STACK];
    const uint32_t lane = lane_id(), w = threadIdx.x / VR_WAVE;
    uint32_t *st = s_stack[w], *li = s_list[w];
    if (B.ctl->err) return;
    // work-group b takes share b % MO_REG of the critical triangles
    const uint32_t i = blockIdx.x % MO_REG, nq = B.ctl->rec[i][0];
    const uint4 *recs = B.rec + (size_t)i * (B.qcap / MO_REG);
    uint32_t slot = 0, slots = 0;  // entries' slots at hand
    const uint32_t eshare = B.ecap / MO_REG;
    uint2 *ent = B.ent + (size_t)i * eshare;
    for (uint32_t qq = blockIdx.x / MO_REG * MO_WPB + w; qq < nq; qq += gridDim.x / MO_REG * MO_WPB) {
        const uint4 rec = recs[(uint32_t)__builtin_amdgcn_readfirstlane((int)qq)];
        const uint32_t r = rec.x, k = rec.y, r0 = r / MO_EB * MO_EB;
        // its place: after those of the edges before r in the block
        const uint32_t lt = B.mask[r / MO_EB] & ((1u << (r - r0)) - 1);
        const uint32_t q = B.blk[r / MO_EB] + rec.w +
                           wave_sum<uint32_t>(lane < MO_EB && ((lt >> lane) & 1u) ? B.ecnt[r0 + lane] : 0u);
        if (lane == 0) {
            B.ctri[q] = rec.z;
            B.owner[q] = 0ull;
        }
        const int64_t a = B.ij[2 * (int64_t)r], b = B.ij[2 * (int64_t)r + 1];
        const int2 f = B.fg[r];
        mo_wave_sync();  // the list of the previous triangle has been read
        if (lane < 4)
            st[lane] = (uint32_t)(lane == 0 ? f.x : lane == 1 ? f.y : B.R[(lane == 2 ? a : b) * B.n + k]);
        mo_wave_sync();
        uint32_t sp = 4, nl = 0;
        bool over = false;
        for (int step = 0; sp > 0; step++) {
            const uint32_t c = min(sp, (uint32_t)VR_WAVE);
            sp -= c;
            const bool on = lane < c;
            const uint32_t x = on ? st[sp + lane] : 0u;
            mo_wave_sync();
            const int2 g = B.fg[x];
            const bool isc = on && g.x < 0 && g.y >= 0, isn = on && g.x >= 0;
            const unsigned long long mc = ballot64(isc), mn = ballot64(isn);
            const uint32_t nc = (uint32_t)__popcll(mc), nn = (uint32_t)__popcll(mn);
            if (sp + 2 * nn > MO_STACK || nl + nc > MO_STACK || step >= MO_STEPS) {
                over = true;
                break;
            }
            if (isc) li[nl + mo_before(mc)] = B.blkm[x / MO_EB] + (uint32_t)g.y;
            if (isn) {
                const uint32_t at = sp + 2 * mo_before(mn);
                st[at] = (uint32_t)g.x;
                st[at + 1] = (uint32_t)g.y;
            }
            nl += nc;
            sp += 2 * nn;
            mo_wave_sync();
        }
        if (over) {
            if (lane == 0) B.ctl->err = 1u;
            continue;
        }
        for (uint32_t x0 = 0; x0 < nl; x0 += VR_WAVE) {
            const uint32_t x = x0 + lane, c = x < nl ? li[x] : MO_NONE;
            uint32_t all = 0, before = 0;
            for (uint32_t j = 0; j < nl; j++) {
                const bool eq = li[j] == c;
                all += eq ? 1u : 0u;
                before += eq && j < x ? 1u : 0u;
            }
            const bool keep = x < nl && (all & 1u) && before == 0;
            const unsigned long long mk = ballot64(keep);
            if (!mk) continue;
            const uint32_t nk = (uint32_t)__popcll(mk);
            if (nk > slots) {
                for (uint32_t y = lane; y < slots; y += VR_WAVE) ent[slot + y] = make_uint2(MO_NONE, 0u);
                if (lane == 0) slot = atomicAdd(&B.ctl->ent[i][0], (uint32_t)MO_SLOTS);
                slot = (uint32_t)__builtin_amdgcn_readfirstlane((int)slot);
                slots = MO_SLOTS;
                if (slot + MO_SLOTS > eshare) {
                    if (lane == 0) B.ctl->err = 1u;
                    return;
                }
            }
            if (keep) {
                ent[slot + mo_before(mk)] = make_uint2(c, q);
                atomicAdd(&B.cnt[c], 1u);
            }
            slot += nk;
            slots -= nk;
        }
    }
    for (uint32_t y = lane; y < slots; y += VR_WAVE) ent[slot + y] = make_uint2(MO_NONE, 0u);
}

// Column c takes cnt[c] + 1 pool words (its length first), back to back.
__global__ __launch_bounds__(1024) void k_mo_scan(MoBufs B) {
    const uint32_t m = B.ctl->m;
    const uint32_t tot = mo_scan(m, [&](uint32_t c) { return B.cnt[c] + 1u; },
                                 [&](uint32_t c, uint32_t s0) {
                                     B.start[c] = s0;
                                     B.pool[s0] = B.cnt[c];  // m + nent words: always room
                                 });
    if (threadIdx.x == 0) B.ctl->ptop = tot;
}

__global__ __launch_bounds__(MO_BLOCK) void k_mo_scatter(MoBufs B) {
    if (B.ctl->err || !B.ctl->any) return;
    const uint32_t x0 = blockIdx.x * MO_BLOCK + threadIdx.x;
    const uint32_t i = blockIdx.x % MO_REG, ne = B.ctl->ent[i][0];
    const uint2 *ent = B.ent + (size_t)i * (B.ecap / MO_REG);
    for (uint32_t x = blockIdx.x / MO_REG * MO_BLOCK + threadIdx.x; x < ne; x += gridDim.x / MO_REG * MO_BLOCK) {
        const uint2 e = ent[x];
        if (e.x != MO_NONE) B.pool[B.start[e.x] + 1 + atomicAdd(&B.fill[e.x], 1u)] = e.y;
    }
    for (int64_t r = x0; r < B.K; r += (int64_t)gridDim.x * MO_BLOCK) {
        const int2 g = B.fg[r];
        if (g.x < 0 && g.y >= 0) B.crit[B.blkm[r / MO_EB] + (uint32_t)g.y] = (uint32_t)r;
    }
}

// The reduction: one wave per column at a time, columns from the youngest
// edge.  A critical triangle's owner word names the column that has it as
// its pivot and where that column's entries lie.  A wave whose column's
// pivot is free, or owned by an older edge (after it in the order), takes
// the pivot with one compare-and-swap, and goes on with the column it
// displaced; owned by a younger edge, that column's entries are added.
// Stored columns are never written again, so one being read stays valid,
// whoever owns the pivot by then; adding any stored version of a column
// before it is a column operation of Algorithm 1, and the pairs do not
// depend on which were done.  No wave waits for another: each step adds
// (the pivot moves to a younger triangle), takes a free pivot, or hands a
// pivot to a younger edge.  (The lock-free reduction of Morozov and
// Nigmetov, "Towards lockfree persistent homology", 2020.)
//
// The working column is a bit per critical triangle: an addition flips the
// added entries' bits, and the pivot is the first set bit from the last one
// on.  Latency bounds it: an addition is two dependent reads from memory.  As
// sorted lists merged in LDS it took 1776 us at the mixture.
// The bits are in LDS, 16 KB a wave where there are at most 2^17 triangles in
// all, else 64 KB; beyond 2^19 critical ones in device memory, by as many waves as the
// entries' array holds bits for.  us of vr_pairs_dim1 with 16 KB, then memory,
// at 256 waves / now (by the columns' reduction): three parts of 60 vertices, all
// edges between them in random order, 84774 / 23400 (38283); parts of 20, 20, 400
// 34270 / 7600 (24709); 400 pairs of hubs over 1410 vertices (563600 critical
// triangles) 175390 / 59500 (119712).  64 KB for all: 1000 points, 24975 random
// edges, 25300 -> 29274.
template <bool LDS>
__device__ __forceinline__ void mo_reduce(const MoBufs &B, unsigned long long *bits, unsigned long long *seen, uint32_t nw,
                                          uint32_t nwaves) {
    const uint32_t lane = lane_id();
    const uint32_t m = B.ctl->m, nc = (nw + VR_WAVE - 1) / VR_WAVE;
    // Bits in device memory are the wave's own, and flipped, read and cleared
    // in L2.  A bit of `seen` (LDS) for each of their words says that the column
    // has touched it: only those are read.
    auto get = [&](uint32_t x) -> unsigned long long {
        if (x >= nw) return 0ull;
        if (LDS) return bits[x];
        return (seen[x / VR_WAVE] >> (x % VR_WAVE)) & 1ull
                   ? __hip_atomic_load(bits + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)
                   : 0ull;
    };
    auto clear = [&](uint32_t x) {
        if (LDS) bits[x] = 0ull;
        else __hip_atomic_store(bits + x, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    // the 64 words to look at from word x on: in memory, whole words of `seen`
    auto from = [&](uint32_t x) -> uint32_t {
        if (LDS) return x;
        for (uint32_t c = x / VR_WAVE; c < nc; c += VR_WAVE) {
            const unsigned long long any = ballot64(c + lane < nc && seen[c + lane] != 0ull);
            if (any) return VR_WAVE * (c + (uint32_t)__builtin_ctzll(any));
        }
        return nc * VR_WAVE;
    };
    auto sync = [&] {
        if (LDS) mo_wave_sync();
        else __threadfence_block();
    };
    for (uint32_t x = lane; x < nw; x += VR_WAVE) clear(x);
    sync();
    auto flip1 = [&](uint32_t q) {
        if (LDS) {
            atomicXor(&bits[q >> 6], 1ull << (q & 63));
        } else {
            (void)__hip_atomic_fetch_xor(&bits[q >> 6], 1ull << (q & 63), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            atomicOr(&seen[q >> 12], 1ull << ((q >> 6) & 63));
        }
    };
    auto flip = [&](const uint32_t *e, uint32_t len) {
        for (uint32_t x = lane; x < len; x += VR_WAVE) flip1(e[x]);
    };
    // a column stored from pool word p: its length and first entries in one read
    auto add = [&](uint32_t p) {
        const uint32_t e = p + lane < B.pcap ? B.pool[p + lane] : 0u;
        const uint32_t len = (uint32_t)__builtin_amdgcn_readfirstlane((int)e);
        if (lane > 0 && lane <= len) flip1(e);
        if (len >= VR_WAVE) flip(B.pool + p + VR_WAVE, len - (VR_WAVE - 1));
    };
    for (uint32_t nx = blockIdx.x; nx < m; nx += nwaves) {
        const uint32_t c = m - 1 - nx;
        uint32_t r = B.crit[c], pub = B.start[c];
        uint32_t wi = 0;  // no bit is set before this word
        bool dirty = false;
        if (!LDS) {
            for (uint32_t x = lane; x < nc; x += VR_WAVE) seen[x] = 0ull;
            sync();
        }
        add(pub);
        for (;;) {
            sync();
            // the pivot: the first set bit
            uint32_t q = MO_NONE;
            for (wi = from(wi); wi < nw; wi = from(wi + VR_WAVE)) {
                const unsigned long long v = get(wi + lane);
                const unsigned long long any = ballot64(v != 0ull);
                if (any) {
                    const int src = __builtin_ctzll(any);
                    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, src);
                    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), src);
                    q = (wi + (uint32_t)src) * 64 + (lo ? (uint32_t)__builtin_ctz(lo) : 32u + (uint32_t)__builtin_ctz(hi));
                    if (LDS) wi += (uint32_t)src;
                    break;
                }
            }
            if (q == MO_NONE) break;  // zero: a class that never dies
            const unsigned long long wv = __hip_atomic_load(&B.owner[q], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
            const uint32_t whi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(wv >> 32));
            const uint32_t wlo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)wv);
            if (whi != 0 && whi - 1 > r) {
                add(wlo);
                dirty = true;
                continue;
            }
            if (dirty) {  // store the column
                uint32_t len = 0;
                for (uint32_t x = wi; x < nw; x = from(x + VR_WAVE))
                    len += (uint32_t)__popcll(get(x + lane));
                len = wave_sum<uint32_t>(len);
                unsigned long long p = 0;
                if (lane == 0) p = atomicAdd(&B.ctl->ptop, (unsigned long long)(len + 1));
                const bool room = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(p >> 32)) == 0 &&
                                  (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)p) + len + 1 <= B.pcap;
                if (!room) {
                    if (lane == 0) B.ctl->err = 1u;
                    return;
                }
                pub = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)p);
                if (lane == 0) B.pool[pub] = len;
                uint32_t at = pub + 1;
                for (uint32_t x = wi; x < nw; x = from(x + VR_WAVE)) {
                    unsigned long long v = get(x + lane);
                    const uint32_t pc = (uint32_t)__popcll(v), inc = wave_incl_scan_dpp(pc);
                    uint32_t o = at + inc - pc;
                    while (v) {
                        B.pool[o++] = (x + lane) * 64 + (uint32_t)__builtin_ctzll(v);
                        v &= v - 1;
                    }
                    at += wave_last(inc);
                }
                dirty = false;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            uint32_t won = 0;
            if (lane == 0) {
                unsigned long long want = ((unsigned long long)whi << 32) | wlo;
                won = __hip_atomic_compare_exchange_strong(&B.owner[q], &want,
                                                           ((unsigned long long)(r + 1) << 32) | pub, __ATOMIC_RELEASE,
                                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                          ? 1u
                          : 0u;
            }
            won = (uint32_t)__builtin_amdgcn_readfirstlane((int)won);
            if (!won) continue;  // the owner changed: look again
            for (uint32_t x = wi; x < nw; x = from(x + VR_WAVE))
                if (x + lane < nw) clear(x + lane);
            if (whi == 0) break;
            // the displaced column goes on from its stored entries
            r = whi - 1;
            pub = wlo;
            sync();
            add(pub);
        }
        sync();
    }
}

template <int LOG>
__global__ __launch_bounds__(VR_WAVE) void k_mo_reduce(MoBufs B) {
    __shared__ unsigned long long bits[(1u << LOG) / 64];
    if (B.ctl->err) return;
    const uint32_t nq = B.ctl->q, nw = (nq + 63) / 64;
    if (nq <= 1u << LOG) {
        mo_reduce<true>(B, bits, nullptr, nw, gridDim.x);
    } else {  // the entries' array is free by now
        const uint32_t most = min(gridDim.x, (uint32_t)MO_ENT / nw);
        if (blockIdx.x < most) mo_reduce<false>(B, (unsigned long long *)B.ent + (size_t)blockIdx.x * nw, bits, nw, most);
    }
}
static_assert((1 << MO_LDS_FEW) / 64 >= MO_QCAP / 64 / VR_WAVE, "a bit of `seen` per word");
static_assert(MO_ENT / (MO_QCAP / 64) >= 256, "the bits of many of k_mo_reduce's waves fit the entries' array");

__global__ __launch_bounds__(MO_BLOCK) void k_mo_emit(MoBufs B) {
    if (B.ctl->err) return;
    const uint32_t nq = B.ctl->q;
    for (uint32_t q = blockIdx.x * MO_BLOCK + threadIdx.x; q < nq; q += gridDim.x * MO_BLOCK) {
        const uint32_t o = (uint32_t)(B.owner[q] >> 32);
        if (o) B.first[o - 1] = (int32_t)B.ctri[q];
    }
}

__global__ __launch_bounds__(MO_BLOCK) void k_mo_init(MoBufs B, int32_t *R) {
    const int64_t x = (int64_t)blockIdx.x * MO_BLOCK + threadIdx.x;
    for (int64_t i = x; i < B.n * B.n; i += (int64_t)gridDim.x * MO_BLOCK) R[i] = vr_rank_none((uint32_t)i, B.n);
    for (int64_t i = x; i < (int64_t)(sizeof(MoCtl) / 4); i += (int64_t)gridDim.x * MO_BLOCK) ((uint32_t *)B.ctl)[i] = 0u;
    for (int64_t r = x; r < B.K; r += (int64_t)gridDim.x * MO_BLOCK) {
        B.first[r] = -1;
        B.cnt[r] = B.fill[r] = 0u;
    }
}

static unsigned mo_grid(int64_t items, int64_t most) {
    const int64_t g = (items + MO_BLOCK - 1) / MO_BLOCK;
    return (unsigned)(g < 1 ? 1 : g > most ? most : g);
}

int morse_pairs_dim1(int32_t *R, const int32_t *ij, const unsigned long long *key, const int32_t *e_low,
                     int64_t n, int64_t K, int64_t T, int32_t *tri_of_edge, bool *done, hipStream_t s) {
    *done = false;
    MoBufs B{};
    B.R = R;
    B.ij = ij;
    B.e_low = e_low;
    B.key = key;
    B.n = n;
    B.K = K;
    B.T = T;
    B.first = tri_of_edge;
    B.qcap = (uint32_t)MO_QCAP;
    B.ecap = (uint32_t)MO_ENT;
    B.pcap = (uint32_t)MO_POOL;
    B.W = (int)((n + 63) / 64);
    while ((K >> B.sb) > MO_SNAPS) B.sb++;  // snapshots at ranks 1 << sb, 2 << sb, ...
    const int S = (int)(K >> B.sb);
    const int64_t nblk = (K + MO_EB - 1) / MO_EB;
    auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
    size_t o = 0;
    auto part = [&](size_t bytes) {
        const size_t at = o;
        o = up(o + bytes);
        return at;
    };
    const size_t o_end = part(4 * (size_t)K), o_fg = part(8 * (size_t)K), o_crit = part(4 * (size_t)K);
    const size_t o_cnt = part(4 * (size_t)K), o_fill = part(4 * (size_t)K), o_start = part(4 * (size_t)K);
    const size_t o_rec = part(16 * (size_t)B.qcap), o_ctri = part(4 * (size_t)B.qcap), o_own = part(8 * (size_t)B.qcap);
    const size_t o_ent = part(8 * (size_t)B.ecap), o_pool = part(4 * (size_t)B.pcap), o_ctl = part(sizeof(MoCtl));
    const size_t o_snap = part(8 * (size_t)S * (size_t)n * (size_t)B.W), o_blk = part(12 * (size_t)nblk), o_ecnt = part(4 * (size_t)K);
    char *ws = (char *)cache_get(o, s);
    if (!ws) return VR_ENOMEM;
    B.end = (int32_t *)(ws + o_end);
    B.fg = (int2 *)(ws + o_fg);
    B.crit = (uint32_t *)(ws + o_crit);
    B.cnt = (uint32_t *)(ws + o_cnt);
    B.fill = (uint32_t *)(ws + o_fill);
    B.start = (uint32_t *)(ws + o_start);
    B.rec = (uint4 *)(ws + o_rec);
    B.ctri = (uint32_t *)(ws + o_ctri);
    B.owner = (unsigned long long *)(ws + o_own);
    B.ent = (uint2 *)(ws + o_ent);
    B.pool = (uint32_t *)(ws + o_pool);
    B.ctl = (MoCtl *)(ws + o_ctl);
    B.snap = (unsigned long long *)(ws + o_snap);
    B.blk = (uint32_t *)(ws + o_blk);
    B.blkm = B.blk + nblk;
    B.mask = B.blkm + nblk;
    B.ecnt = (uint32_t *)(ws + o_ecnt);
    const int64_t wg = (nblk + MO_WPB - 1) / MO_WPB;
    hipLaunchKernelGGL(k_mo_init, dim3(mo_grid(n * n > K ? n * n : K, 4096)), dim3(MO_BLOCK), 0, s, B, R);
    hipLaunchKernelGGL(k_mo_range, dim3(mo_grid((T + 1) / 2, 65536)), dim3(MO_BLOCK), 0, s, B, R);
    hipLaunchKernelGGL(k_mo_snap, dim3((unsigned)n), dim3(MO_BLOCK), 8 * (size_t)S * (size_t)B.W, s, B, S);
    if (B.W > VR_WAVE) hipLaunchKernelGGL(k_mo_link<2>, dim3((unsigned)wg), dim3(MO_BLOCK), 0, s, B);
    else hipLaunchKernelGGL(k_mo_link<1>, dim3((unsigned)wg), dim3(MO_BLOCK), 0, s, B);
    hipLaunchKernelGGL(k_mo_split, dim3((unsigned)nblk), dim3(MO_BLOCK), 0, s, B);
    hipLaunchKernelGGL(k_mo_order, dim3(mo_wide_may(n) ? 256 : 2), dim3(MO_WIDE_BLOCK), 0, s, B);
    hipLaunchKernelGGL(k_mo_expand, dim3(2048), dim3(MO_BLOCK), 0, s, B);
    hipLaunchKernelGGL(k_mo_scan, dim3(1), dim3(1024), 0, s, B);
    hipLaunchKernelGGL(k_mo_scatter, dim3(512), dim3(MO_BLOCK), 0, s, B);
    if (T <= 1 << MO_LDS_FEW) hipLaunchKernelGGL(k_mo_reduce<MO_LDS_FEW>, dim3(1280), dim3(VR_WAVE), 0, s, B);
    else hipLaunchKernelGGL(k_mo_reduce<MO_LDS_MANY>, dim3(1280), dim3(VR_WAVE), 0, s, B);
    hipLaunchKernelGGL(k_mo_emit, dim3(256), dim3(MO_BLOCK), 0, s, B);
    uint32_t err = 0;
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpyAsync(&err, &B.ctl->err, sizeof(err), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    cache_put(ws, s);
    if (e != hipSuccess) return VR_EHIP;
    *done = err == 0;
    return VR_OK;
}
