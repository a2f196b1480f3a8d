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
//   k_mo_link    per edge, a wave: L(r)'s components, the replacement edges,
//                the critical triangles
//   k_mo_expand  per critical triangle, a wave: its boundary in critical edges
//   k_mo_scan    starts of the columns
//   k_mo_scatter the columns' entries
//   k_mo_reduce  the reduction, a wave per column, without rounds or locks
//   k_mo_emit    the pairs
//
// On the circle and the mixture vr_pairs_dim1 took 28.4 and 36.5 ms as a
// reduction of the full edge columns, a work-group each: one column's chain
// of thousands of additions.  The chains here are a few additions long.
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
#define MO_QBITS 27                 // critical triangles: index bits of a column entry
#define MO_QCAP (1ll << 22)         // critical triangles at most
#define MO_ENT (1ll << 24)          // column entries at most
#define MO_POOL (1ll << 25)         // words of stored columns at most
#define MO_CAP 1024                 // entries of a column held in LDS
#define MO_NONE 0xFFFFFFFFu

struct MoCtl {
    uint32_t q;     // critical triangles
    uint32_t m;     // critical edges
    uint32_t nent;  // column entries
    uint32_t err;   // a limit was passed
    uint32_t next;  // columns taken
    uint32_t pad;
    unsigned long long ptop;  // pool words taken
};

// A column entry orders critical triangles as the filtration does and names
// one: edge rank (24 bits) | third vertex (13) | index (27).
struct MoBufs {
    const int32_t *R, *ij, *e_low;
    const unsigned long long *key;
    int64_t n, K, T;
    int32_t *first, *end;           // K: the triangles of value r are [first, end); first -1: none
    int2 *fg;                       // K: the two edges that replace r; x = -1: none, y = its column or -1
    uint32_t *crit;                 // column -> edge
    uint32_t *cnt, *fill;           // column -> entries, entries placed
    uint32_t *start;                // column -> its first pool word (the length, then the entries)
    unsigned long long *cent;       // critical triangle -> its entry
    uint32_t *ctri;                 // critical triangle -> its index among the keys
    unsigned long long *owner;      // critical triangle -> (edge + 1) << 32 | pool word of its column; 0: none
    uint2 *ent;                     // (column, critical triangle) pairs
    unsigned long long *pool;
    MoCtl *ctl;
    uint32_t qcap, ecap;
    unsigned long long pcap;
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

// Bound by reading the keys once (8 T bytes); two keys a thread.
__global__ __launch_bounds__(MO_BLOCK) void k_mo_range(MoBufs B) {
    const int64_t np = (B.T + 1) / 2;
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

// A wave's lanes append the critical triangles of edge r marked by `on`.
__device__ __forceinline__ void mo_append(const MoBufs &B, uint32_t r, uint32_t k, uint32_t tri, bool on) {
    const unsigned long long m = ballot64(on);
    if (!m) return;
    uint32_t q0 = 0;
    if (lane_id() == 0) q0 = atomicAdd(&B.ctl->q, (uint32_t)__popcll(m));
    q0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)q0);
    const uint32_t q = q0 + mo_before(m);
    if (!on) return;
    if (q >= B.qcap) {
        B.ctl->err = 1u;
        return;
    }
    B.cent[q] = ((unsigned long long)r << (13 + MO_QBITS)) | ((unsigned long long)k << MO_QBITS) | q;
    B.ctri[q] = tri;
    B.owner[q] = 0ull;
}

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
__device__ void mo_link_any(const MoBufs &B, uint32_t r, uint32_t a, uint32_t b, int32_t f0, uint32_t m,
                            unsigned long long *reach, unsigned long long *open, unsigned long long *comp) {
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
    while (left > 0) {
        for (uint32_t p = lane; p < np; p += VR_WAVE) open[p] = comp[p] = 0ull;
        mo_wave_sync();
        uint32_t y = seed;
        for (;;) {
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
        // the component's first vertex; the component of vertex 0 is the apparent triangle's
        uint32_t lo = 0;
        while (!comp[lo]) lo++;
        const uint32_t x0 = lo * VR_WAVE + (uint32_t)__builtin_ctzll(comp[lo]);
        if (x0 == 0) {
            if (!first_comp) (void)nearest(false, &fx, &fy);
        } else {
            mo_append(B, r, vertex(x0), (uint32_t)f0 + x0, lane == 0);
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
    if (lane == 0) B.fg[r] = make_int2(fx, fy);
}

// One wave per edge.  The search starts at the vertex nearest both ends,
// which mostly joins every other vertex of L(r) at once: 1.2 (circle) to
// about 2 (mixture) rows of R are read per edge.  Latency-bound: a chain of
// about eight dependent loads per edge.
__global__ __launch_bounds__(MO_BLOCK) void k_mo_link(MoBufs B) {
    __shared__ unsigned long long masks[MO_WPB][3][MO_GEN];
    const uint32_t lane = lane_id(), w = threadIdx.x / VR_WAVE;
    const int64_t stride = (int64_t)gridDim.x * MO_WPB;
    for (int64_t rr = (int64_t)blockIdx.x * MO_WPB + w; rr < B.K; rr += stride) {
        const uint32_t r = (uint32_t)__builtin_amdgcn_readfirstlane((int)rr);
        const int32_t f0 = B.first[r];
        if (f0 < 0) {
            int32_t c = -1;
            if (B.e_low[r] < 0) {
                if (lane == 0) {
                    c = (int32_t)atomicAdd(&B.ctl->m, 1u);
                    B.crit[c] = r;
                    B.cnt[c] = 0u;
                    B.fill[c] = 0u;
                }
            }
            if (lane == 0) B.fg[r] = make_int2(-1, c);
            continue;
        }
        const uint32_t m = (uint32_t)(B.end[r] - f0);
        const uint32_t a = (uint32_t)B.ij[2 * (int64_t)r], b = (uint32_t)B.ij[2 * (int64_t)r + 1];
        if (m > MO_NC * VR_WAVE) {
            mo_link_any(B, r, a, b, f0, m, masks[w][0], masks[w][1], masks[w][2]);
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
        for (;;) {
            unsigned long long open[MO_NC], comp[MO_NC];
#pragma unroll
            for (int i = 0; i < MO_NC; i++) open[i] = comp[i] = 0ull;
            uint32_t y = seed;
            bool more = true;
            for (;;) {
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
            // the component's first vertex; that of vertex 0 holds the apparent triangle
            uint32_t x0 = MO_NONE;
#pragma unroll
            for (int i = MO_NC - 1; i >= 0; i--)
                if (comp[i]) x0 = (uint32_t)i * VR_WAVE + (uint32_t)__builtin_ctzll(comp[i]);
            if (x0 != 0) {
                mo_append(B, r, vertex(x0), (uint32_t)f0 + x0, lane == 0);
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
        if (lane == 0) B.fg[r] = make_int2(Ra[kstar], Rb[kstar]);
    }
}

// One wave per critical triangle {r, k}: the edges ak, bk and r's two
// replacements go on a stack; each lane takes one off it, and its two
// replacements go back, or the critical edge it is into a list.  Edges an
// even number of times in the list cancel.  Any order does, since every
// replacement is older.
__global__ __launch_bounds__(MO_BLOCK) void k_mo_expand(MoBufs B) {
    __shared__ uint32_t s_stack[MO_WPB][MO_STACK];
    __shared__ uint32_t s_list[MO_WPB][MO_STACK];
    const uint32_t lane = lane_id(), w = threadIdx.x / VR_WAVE;
    uint32_t *st = s_stack[w], *li = s_list[w];
    const uint32_t nq = min(B.ctl->q, B.qcap);
    for (uint32_t qq = blockIdx.x * MO_WPB + w; qq < nq; qq += gridDim.x * MO_WPB) {
        const uint32_t q = (uint32_t)__builtin_amdgcn_readfirstlane((int)qq);
        const unsigned long long e = B.cent[q];
        const uint32_t r = (uint32_t)(e >> (13 + MO_QBITS)), k = (uint32_t)(e >> MO_QBITS) & 0x1FFFu;
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
            if (isc) li[nl + mo_before(mc)] = (uint32_t)g.y;
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
            uint32_t e0 = 0;
            if (lane == 0) e0 = atomicAdd(&B.ctl->nent, (uint32_t)__popcll(mk));
            e0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)e0);
            const uint32_t at = e0 + mo_before(mk);
            if (keep) {
                if (at < B.ecap) {
                    B.ent[at] = make_uint2(c, q);
                    atomicAdd(&B.cnt[c], 1u);
                } else {
                    B.ctl->err = 1u;
                }
            }
        }
    }
}

// Column c takes cnt[c] + 1 pool words (its length first), back to back.
__global__ __launch_bounds__(1024) void k_mo_scan(MoBufs B) {
    __shared__ uint32_t wt[16];
    __shared__ uint32_t carry;
    const uint32_t t = threadIdx.x, lane = t & 63, wv = t >> 6, m = B.ctl->m;
    if (t == 0) carry = 0;
    __syncthreads();
    for (uint32_t base = 0; base < m; base += 1024) {
        const uint32_t c = base + t, len = c < m ? B.cnt[c] : 0u, x = c < m ? len + 1 : 0u;
        const uint32_t inc = wave_incl_scan_dpp(x);
        if (lane == 63) wt[wv] = inc;
        __syncthreads();
        uint32_t off = carry, tot = 0;
        for (uint32_t i = 0; i < 16; i++) {
            if (i < wv) off += wt[i];
            tot += wt[i];
        }
        if (c < m) {
            const uint32_t s0 = off + inc - x;
            B.start[c] = s0;
            if (s0 < B.pcap) B.pool[s0] = len;
        }
        __syncthreads();
        if (t == 0) carry += tot;
        __syncthreads();
    }
    if (t == 0) {
        B.ctl->ptop = carry;
        if (carry > B.pcap) B.ctl->err = 1u;
    }
}

__global__ __launch_bounds__(MO_BLOCK) void k_mo_scatter(MoBufs B) {
    if (B.ctl->err) return;
    const uint32_t ne = B.ctl->nent;
    for (uint32_t x = blockIdx.x * MO_BLOCK + threadIdx.x; x < ne; x += gridDim.x * MO_BLOCK) {
        const uint2 e = B.ent[x];
        B.pool[B.start[e.x] + 1 + atomicAdd(&B.fill[e.x], 1u)] = B.cent[e.y];
    }
}

// Ascending bitonic sort of n entries in LDS by one wave, padded to a power
// of two (the buffer holds that many).
__device__ void mo_sort(unsigned long long *g, uint32_t n) {
    const uint32_t lane = lane_id();
    uint32_t P = 1;
    while (P < n) P <<= 1;
    for (uint32_t x = n + lane; x < P; x += VR_WAVE) g[x] = ~0ull;
    mo_wave_sync();
    for (uint32_t kk = 2; kk <= P; kk <<= 1)
        for (uint32_t j = kk >> 1; j > 0; j >>= 1) {
            for (uint32_t i = lane; i < P / 2; i += VR_WAVE) {
                const uint32_t lo = 2 * i - (i & (j - 1)), hi = lo + j;
                const unsigned long long x0 = g[lo], x1 = g[hi];
                if ((x0 > x1) == ((lo & kk) == 0)) {
                    g[lo] = x1;
                    g[hi] = x0;
                }
            }
            mo_wave_sync();
        }
}

// o = a + b over F2 by one wave (sorted entries, na + nb of room in o):
// merge path, a run of the merged list per lane, then the entries in both
// (next to each other) are dropped in place.  Returns the length.
template <typename PA, typename PB, typename PO>
__device__ __forceinline__ uint32_t mo_add(PA a, uint32_t na, PB b, uint32_t nb, PO o) {
    const uint32_t lane = lane_id(), L = na + nb, S = (L + VR_WAVE - 1) / VR_WAVE;
    const uint32_t d0 = min(L, lane * S), d1 = min(L, d0 + S);
    uint32_t lo = d0 > nb ? d0 - nb : 0u, hi = min(d0, na);
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (a[mid] <= b[d0 - 1 - mid]) lo = mid + 1;
        else hi = mid;
    }
    uint32_t i = lo, j = d0 - lo;
    for (uint32_t d = d0; d < d1; d++) {
        const bool ta = j >= nb || (i < na && a[i] <= b[j]);
        o[d] = ta ? a[i++] : b[j++];
    }
    mo_wave_sync();
    // a kept entry never moves up, and an entry moved over is the one it was
    uint32_t run = 0;
    for (uint32_t x0 = 0; x0 < L; x0 += VR_WAVE) {
        const uint32_t x = x0 + lane;
        unsigned long long v = 0;
        bool keep = false;
        if (x < L) {
            v = o[x];
            keep = (x == 0 || o[x - 1] != v) && (x + 1 == L || o[x + 1] != v);
        }
        const unsigned long long mk = ballot64(keep);
        mo_wave_sync();
        if (keep) o[run + mo_before(mk)] = v;
        mo_wave_sync();
        run += (uint32_t)__popcll(mk);
    }
    return run;
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
__global__ __launch_bounds__(VR_WAVE) void k_mo_reduce(MoBufs B) {
    __shared__ unsigned long long buf[3 * MO_CAP];
    const uint32_t lane = lane_id();
    if (B.ctl->err) return;
    const uint32_t m = B.ctl->m;
    // n pool words for the wave; ~0 (and the error flagged) when there is no room
    auto take = [&](uint32_t words) -> unsigned long long {
        unsigned long long p = 0;
        if (lane == 0) {
            p = atomicAdd(&B.ctl->ptop, (unsigned long long)words);
            if (p + words > B.pcap) {
                p = ~0ull;
                B.ctl->err = 1u;
            }
        }
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(p >> 32));
        return ((unsigned long long)hi << 32) | (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)p);
    };
    for (;;) {
        uint32_t nx = 0;
        if (lane == 0) nx = atomicAdd(&B.ctl->next, 1u);
        nx = (uint32_t)__builtin_amdgcn_readfirstlane((int)nx);
        if (nx >= m) return;
        const uint32_t c = m - 1 - nx;
        uint32_t r = B.crit[c], len = B.cnt[c], pub = B.start[c];
        if (len == 0) continue;  // in no boundary: a class that never dies
        if (len > 2 * MO_CAP) {
            if (lane == 0) B.ctl->err = 1u;
            continue;
        }
        // the column's entries, sorted, back to their place
        unsigned long long *cur = buf;  // the column lies here (LDS), or in the pool from gcur (gcur != null)
        const unsigned long long *gcur = nullptr;
        for (uint32_t x = lane; x < len; x += VR_WAVE) buf[x] = B.pool[pub + 1 + x];
        mo_wave_sync();
        if (len > 1) {
            mo_sort(buf, len);
            for (uint32_t x = lane; x < len; x += VR_WAVE) B.pool[pub + 1 + x] = buf[x];
        }
        if (len > MO_CAP) gcur = B.pool + pub + 1;
        mo_wave_sync();
        bool dirty = false;
        while (len > 0) {
            const unsigned long long p = gcur ? gcur[0] : cur[0];
            const uint32_t q = (uint32_t)p & ((1u << MO_QBITS) - 1);
            const unsigned long long wv = __hip_atomic_load(&B.owner[q], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
            const uint32_t whi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(wv >> 32));
            const uint32_t wlo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)wv);
            if (whi == 0 || whi - 1 < r) {
                if (dirty) {
                    const unsigned long long o = take(len + 1);
                    if (o == ~0ull) break;
                    pub = (uint32_t)o;
                    if (lane == 0) B.pool[pub] = len;
                    for (uint32_t x = lane; x < len; x += VR_WAVE) B.pool[pub + 1 + x] = gcur ? gcur[x] : cur[x];
                    dirty = false;
                }
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
                uint32_t won = 0;
                if (lane == 0) {
                    unsigned long long want = ((unsigned long long)whi << 32) | wlo;
                    won = __hip_atomic_compare_exchange_strong(&B.owner[q], &want,
                                                               ((unsigned long long)(r + 1) << 32) | pub,
                                                               __ATOMIC_RELEASE, __ATOMIC_RELAXED,
                                                               __HIP_MEMORY_SCOPE_AGENT)
                              ? 1u
                              : 0u;
                }
                won = (uint32_t)__builtin_amdgcn_readfirstlane((int)won);
                if (!won) continue;  // the owner changed: look again
                if (whi == 0) break;
                // the displaced column goes on from its stored entries
                r = whi - 1;
                pub = wlo;
                len = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)B.pool[pub]);
                gcur = B.pool + pub + 1;
                if (len <= MO_CAP) {
                    mo_wave_sync();
                    for (uint32_t x = lane; x < len; x += VR_WAVE) cur[x] = gcur[x];
                    gcur = nullptr;
                }
                mo_wave_sync();
                continue;
            }
            const uint32_t nb = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)B.pool[wlo]);
            const unsigned long long *gb = B.pool + wlo + 1;
            dirty = true;
            if (!gcur && len + nb <= MO_CAP) {
                unsigned long long *sb = buf + 2 * MO_CAP, *o = cur == buf ? buf + MO_CAP : buf;
                for (uint32_t x = lane; x < nb; x += VR_WAVE) sb[x] = gb[x];
                mo_wave_sync();
                len = mo_add(cur, len, sb, nb, o);
                cur = o;
            } else {
                // a long column: the sum in the pool
                const unsigned long long o = take(len + nb);
                if (o == ~0ull) break;
                unsigned long long *go = B.pool + o;
                len = gcur ? mo_add(gcur, len, gb, nb, go) : mo_add(cur, len, gb, nb, go);
                gcur = go;
                if (len <= MO_CAP) {
                    for (uint32_t x = lane; x < len; x += VR_WAVE) cur[x] = go[x];
                    gcur = nullptr;
                }
                mo_wave_sync();
            }
        }
        mo_wave_sync();  // the buffers are reused by the next column
    }
}

__global__ __launch_bounds__(MO_BLOCK) void k_mo_emit(MoBufs B) {
    if (B.ctl->err) return;
    const uint32_t nq = B.ctl->q;
    for (uint32_t q = blockIdx.x * MO_BLOCK + threadIdx.x; q < nq; q += gridDim.x * MO_BLOCK) {
        const uint32_t o = (uint32_t)(B.owner[q] >> 32);
        if (o) B.first[o - 1] = (int32_t)B.ctri[q];
    }
}

__global__ __launch_bounds__(MO_BLOCK) void k_mo_init(MoBufs B) {
    const int64_t x = (int64_t)blockIdx.x * MO_BLOCK + threadIdx.x;
    if (x == 0) *B.ctl = MoCtl{};
    for (int64_t r = x; r < B.K; r += (int64_t)gridDim.x * MO_BLOCK) B.first[r] = -1;
}

static unsigned mo_grid(int64_t items, int64_t most) {
    const int64_t g = (items + MO_BLOCK - 1) / MO_BLOCK;
    return (unsigned)(g < 1 ? 1 : g > most ? most : g);
}

int morse_pairs_dim1(const int32_t *R, const int32_t *ij, const unsigned long long *key, const int32_t *e_low,
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
    B.qcap = (uint32_t)(T < MO_QCAP ? T : MO_QCAP);
    B.ecap = (uint32_t)MO_ENT;
    B.pcap = (unsigned long long)MO_POOL;
    auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
    size_t o = 0;
    auto part = [&](size_t bytes) {
        const size_t at = o;
        o = up(o + bytes);
        return at;
    };
    const size_t o_end = part(4 * (size_t)K), o_fg = part(8 * (size_t)K), o_crit = part(4 * (size_t)K);
    const size_t o_cnt = part(4 * (size_t)K), o_fill = part(4 * (size_t)K), o_start = part(4 * (size_t)K);
    const size_t o_cent = part(8 * (size_t)B.qcap), o_ctri = part(4 * (size_t)B.qcap), o_own = part(8 * (size_t)B.qcap);
    const size_t o_ent = part(8 * (size_t)B.ecap), o_pool = part(8 * (size_t)B.pcap), o_ctl = part(sizeof(MoCtl));
    char *ws = (char *)cache_get(o, s);
    if (!ws) return VR_ENOMEM;
    B.end = (int32_t *)(ws + o_end);
    B.fg = (int2 *)(ws + o_fg);
    B.crit = (uint32_t *)(ws + o_crit);
    B.cnt = (uint32_t *)(ws + o_cnt);
    B.fill = (uint32_t *)(ws + o_fill);
    B.start = (uint32_t *)(ws + o_start);
    B.cent = (unsigned long long *)(ws + o_cent);
    B.ctri = (uint32_t *)(ws + o_ctri);
    B.owner = (unsigned long long *)(ws + o_own);
    B.ent = (uint2 *)(ws + o_ent);
    B.pool = (unsigned long long *)(ws + o_pool);
    B.ctl = (MoCtl *)(ws + o_ctl);
    const int64_t wg = (K + MO_WPB - 1) / MO_WPB;
    hipLaunchKernelGGL(k_mo_init, dim3(mo_grid(K, 4096)), dim3(MO_BLOCK), 0, s, B);
    hipLaunchKernelGGL(k_mo_range, dim3(mo_grid((T + 1) / 2, 65536)), dim3(MO_BLOCK), 0, s, B);
    hipLaunchKernelGGL(k_mo_link, dim3((unsigned)(wg < 8192 ? wg : 8192)), dim3(MO_BLOCK), 0, s, B);
    hipLaunchKernelGGL(k_mo_expand, dim3((unsigned)(wg < 2048 ? wg : 2048)), dim3(MO_BLOCK), 0, s, B);
    hipLaunchKernelGGL(k_mo_scan, dim3(1), dim3(1024), 0, s, B);
    hipLaunchKernelGGL(k_mo_scatter, dim3(512), dim3(MO_BLOCK), 0, s, B);
    hipLaunchKernelGGL(k_mo_reduce, dim3(1280), dim3(VR_WAVE), 0, s, B);
    hipLaunchKernelGGL(k_mo_emit, dim3(256), dim3(MO_BLOCK), 0, s, B);
    MoCtl hc{};
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpyAsync(&hc, B.ctl, sizeof(hc), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    cache_put(ws, s);
    if (e != hipSuccess) return VR_EHIP;
    *done = hc.err == 0;
    return VR_OK;
}
