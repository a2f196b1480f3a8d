// k_links.hip -- persistence pairs of dimension 2 from the links of the
// edges, instead of by reducing every triangle's coboundary.
//
// Write an edge by its rank r, with ends a < b.  Its link X is the graph of
// the vertices k joined to both ends by older edges, with the edges kl older
// than r: {r, k} are the triangles of value r, and {r, k, l} the tetrahedra,
// in the order of (k, l) (Section 2.1).  The boundary of {r, k, l} is {r, k},
// {r, l} and two triangles older than r, so Algorithm 1 (Section 2.2.1), run
// over the tetrahedra of value r, does to the triangles of value r what it
// does to X's vertices:
//   - Where the edge kl joins two components of the edges before it, the
//     tetrahedron pairs with the first triangle of the younger component
//     (Kruskal's algorithm, elder rule).  This gives all pairs of length
//     zero.  The first triangle of each component of X is left; the first of
//     all pairs with r, the others are the critical triangles.
//   - Where kl closes a cycle z, what is left of the column is the sum over
//     z's edges uv of the older triangles {a, u, v} and {b, u, v}.  If z is a
//     sum of triangles of X and of cycles before it, the column becomes zero:
//     a triangle uvw of X stands for the older tetrahedra {a, u, v, w} and
//     {b, u, v, w}.  So only as many tetrahedra as X, filled in, has
//     independent cycles are critical, and most links have none: nearly all
//     are cones or collapse to a point.
//   - A triangle of value r' < r may be replaced, in a critical tetrahedron's
//     column, by the other three of an older tetrahedron {r', m, p}; with p
//     m's parent in a tree of X' this ends in critical triangles and ones
//     paired with edges, which may be left out (a column is a cycle, known by
//     its other triangles).
// What remains is a matrix of a few columns; without critical tetrahedra
// every critical triangle that pairs with no edge starts a class that never
// dies, and there is nothing to reduce.
//
//   k_lk_pairs   per edge, a wave: its link as 64-bit rows, the pairs of
//                length zero, the trees, whether the link collapses
//   k_lk_cycles  per link that does not, a wave: its critical tetrahedra
//   k_lk_expand  per critical tetrahedron, a work-group: its column in
//                critical triangles
//   k_lk_reduce  the columns' reduction, one work-group
//
// A sphere of 400 points (11975 edges, 144613 triangles) spent 2520 of 3080
// us of its passes in two rounds that reduced each critical triangle's
// coboundary by one work-group, most of them to zero; these kernels take 17,
// 10, 39 and 9 us.
#include <hip/hip_runtime.h>
#include <immintrin.h>
#include <stdint.h>

#include "vr.h"
#include "vr_cache.h"
#include "vr_device.h"
#include "vr_morse.h"

#define LK_BLOCK 256
#define LK_WPB (LK_BLOCK / VR_WAVE)
#define LK_CRIT 1024          // critical tetrahedra at most
#define LK_POOL (1u << 22)    // entries of their columns at most
#define LK_MAXT (384 * 1024)  // triangles whose bits k_lk_expand holds in LDS
#define LK_FRONT 1536         // triangles replaced at a time
#define LK_ROUNDS (1 << 16)
#define LK_DROP 0xFFFFu       // first triangle of its value
#define LK_ROOT 0xFFFEu       // first triangle of a further component

struct LkCrit {
    long long tet;  // index among the tetrahedra
    uint32_t r, ne;
    uint32_t uv[VR_WAVE];  // the cycle's edges, u << 16 | v
    uint32_t start, len;   // its column in the pool
    uint32_t top, pad;     // the column's youngest triangle + 1
};

struct LkCtl {
    uint32_t err;    // a limit was passed
    uint32_t nlink;  // links listed
    uint32_t ncrit;
    uint32_t ptop;
};

struct LkBufs {
    const int32_t *R, *ij;
    const unsigned long long *tri;
    const long long *toff;
    const int32_t *rng;  // the triangles of value r: [rng[2r], rng[2r + 1])
    const int32_t *clr;  // T: paired with an edge
    int64_t n, K, T;
    long long *tri_tet;
    uint16_t *par;   // T: the vertex after {r, m}'s m in its tree, or LK_DROP, LK_ROOT
    uint32_t *list;  // links that do not collapse
    LkCrit *crit;
    uint32_t *pool;
    LkCtl *ctl;
    uint32_t *word;  // host: LK_FITS or LK_MANY once known, if asked for
};
#define LK_FITS 1u
#define LK_MANY 2u

typedef unsigned long long lk_bits;
__device__ __forceinline__ lk_bits lk_low(uint32_t x) { return x >= 64 ? ~0ull : (1ull << x) - 1; }
__device__ __forceinline__ uint32_t lk_rl(uint32_t v, uint32_t i) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)i);
}
__device__ __forceinline__ lk_bits lk_rl64(lk_bits v, uint32_t i) {
    return ((lk_bits)lk_rl((uint32_t)(v >> 32), i) << 32) | lk_rl((uint32_t)v, i);
}
__device__ __forceinline__ void lk_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// The link of edge r, lane i < L holding its i-th vertex k and row i of its
// graph (lanes past L: vertex 0's, and no neighbours).
__device__ __forceinline__ void lk_link(const LkBufs &B, uint32_t r, uint32_t lo, uint32_t L, uint32_t &k,
                                        lk_bits &row) {
    const uint32_t lane = lane_id();
    const uint32_t a = (uint32_t)B.ij[2 * (int64_t)r], b = (uint32_t)B.ij[2 * (int64_t)r + 1];
    const lk_bits key = B.tri[lo + (lane < L ? lane : 0u)];
    const uint32_t x = (uint32_t)(key >> 26) & 0x1FFFu, y = (uint32_t)(key >> 13) & 0x1FFFu, z = (uint32_t)key & 0x1FFFu;
    k = (x != a && x != b) ? x : ((y != a && y != b) ? y : z);
    const int32_t *Rk = B.R + (int64_t)k * B.n;
    row = 0;
    uint32_t j = 0;
    for (; j + 4 <= L; j += 4) {
        int32_t e[4];
#pragma unroll
        for (int u = 0; u < 4; u++) e[u] = Rk[lk_rl(k, j + u)];
#pragma unroll
        for (int u = 0; u < 4; u++) row |= (lk_bits)(e[u] < (int32_t)r ? 1u : 0u) << (j + u);
    }
    for (; j < L; j++) row |= (lk_bits)(Rk[lk_rl(k, j)] < (int32_t)r ? 1u : 0u) << j;
    row = lane < L ? row & ~(1ull << lane) : 0ull;  // the diagonal of R is -1
}

// Tetrahedra of value r before those of lane's vertex k as the smaller one.
__device__ __forceinline__ uint32_t lk_before(lk_bits row) {
    const uint32_t up = (uint32_t)__popcll(row & ~lk_low(lane_id() + 1));
    return wave_incl_scan_dpp(up) - up;
}

// Removes dominated vertices (whose neighbours, and themselves, are all
// another's) until there are none: what is left, A, has the same homology as
// the link filled in.  All that are dominated go at once; of vertices with
// the same neighbours the first stays.  rho: the vertex that stands for a
// removed one.
__device__ __forceinline__ lk_bits lk_collapse(lk_bits row, uint32_t L, uint32_t &rho) {
    const uint32_t lane = lane_id();
    lk_bits A = lk_low(L);
    rho = lane;
    for (;;) {
        const lk_bits own = (row | (1ull << lane)) & A;
        bool dom = false;
        uint32_t by = lane;
        for (lk_bits todo = A; todo; todo &= todo - 1) {
            const uint32_t w = (uint32_t)__builtin_ctzll(todo);
            const lk_bits nw = (lk_rl64(row, w) | (1ull << w)) & A;
            if (((row >> w) & 1ull) && !(own & ~nw) && (own != nw || w < lane)) {
                dom = true;
                by = w;
            }
        }
        const lk_bits gone = __builtin_amdgcn_ballot_w64(dom && ((A >> lane) & 1ull));
        if (!gone) break;
        if ((gone >> lane) & 1ull) rho = by;
        A &= ~gone;
    }
    return A;
}

// Bound by the chain of a wave's steps over its link (one per component
// joined) and the gathers of the ranks; links here have a dozen vertices.
__global__ __launch_bounds__(LK_BLOCK) void k_lk_pairs(LkBufs B) {
    const uint32_t lane = lane_id();
    const int64_t nw = (int64_t)gridDim.x * LK_WPB;
    const uint32_t many = B.ctl->err;  // a link has too many vertices
    if (B.word && blockIdx.x == 0 && threadIdx.x == 0)
        __hip_atomic_store(B.word, many ? LK_MANY : LK_FITS, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    if (many) return;
    // the youngest edges first: their links are the largest, and one past a
    // limit ends the kernel (a wave looks after its first edge and every
    // fourth: a look is a read of one address by all)
    int it = 0;
    for (int64_t rr = (int64_t)blockIdx.x * LK_WPB + threadIdx.x / VR_WAVE; rr < B.K; rr += nw) {
        const uint32_t r = (uint32_t)__builtin_amdgcn_readfirstlane((int)(B.K - 1 - rr));
        if ((it++ & 3) == 1 && st_load32(&B.ctl->err)) return;
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane(B.rng[2 * (int64_t)r]);
        const uint32_t L = (uint32_t)__builtin_amdgcn_readfirstlane(B.rng[2 * (int64_t)r + 1]) - lo;
        if (L == 0) continue;
        uint32_t k;
        lk_bits row;
        lk_link(B, r, lo, L, k, row);
        const uint32_t bef = lk_before(row);
        // pairs of length zero
        uint32_t comp = lane, pair = 0xFFFFFFFFu;
        for (uint32_t x = 0; x < L; x++) {
            if (!__builtin_amdgcn_ballot_w64(lane < L && comp != 0)) break;
            const lk_bits rx = lk_rl64(row, x) & ~lk_low(x + 1);
            if (!rx) continue;
            uint32_t cx = lk_rl(comp, x);
            for (;;) {
                const lk_bits m = rx & __builtin_amdgcn_ballot_w64(comp != cx);
                if (!m) break;
                const uint32_t l = (uint32_t)__builtin_ctzll(m), cl = lk_rl(comp, l);
                const uint32_t old = min(cx, cl), yng = max(cx, cl);
                if (lane == yng) pair = lk_rl(bef, x) + (uint32_t)__popcll(rx & lk_low(l));
                if (comp == yng) comp = old;
                cx = old;
            }
        }
        const lk_bits roots = __builtin_amdgcn_ballot_w64(lane < L && comp == lane);
        // trees, breadth first
        uint32_t p = lane == 0 ? LK_DROP : LK_ROOT;
        for (lk_bits seen = roots, front = roots; front;) {
            const lk_bits nb = row & front;
            const bool mine = !((seen >> lane) & 1ull) && nb != 0;  // none past L: no neighbours
            const uint32_t v = (uint32_t)__shfl((int)k, mine ? (int)__builtin_ctzll(nb) : 0, VR_WAVE);
            if (mine) p = v;
            front = __builtin_amdgcn_ballot_w64(mine);
            seen |= front;
        }
        if (lane < L) {
            B.par[lo + lane] = (uint16_t)p;
            B.tri_tet[lo + lane] = pair == 0xFFFFFFFFu ? -1ll : B.toff[r] + (long long)pair;
        }
        // a cone collapses
        if (__builtin_amdgcn_ballot_w64(lane < L && (row | (1ull << lane)) == lk_low(L))) continue;
        if (st_load32(&B.ctl->err)) return;  // before the longest step
        uint32_t rho;
        const lk_bits A = lk_collapse(row, L, rho);
        if (__popcll(A) == __popcll(roots)) continue;
        // edges outside a forest of the core, which has the link's components
        const uint32_t ends = wave_sum<uint32_t>(((A >> lane) & 1ull) ? (uint32_t)__popcll(row & A) : 0u);
        if (ends / 2 + (uint32_t)__popcll(roots) > 64u + (uint32_t)__popcll(A)) {
            if (lane == 0) st_store32(&B.ctl->err, 1u);
            return;
        }
        if (lane == 0) B.list[atomicAdd(&B.ctl->nlink, 1u)] = r;
    }
}

// One wave per listed link.  Its core (what does not collapse) gets a cocycle
// basis: a bit per edge outside a forest, then for each triangle one bit of
// its sum is expressed by the others; the link's edges take the bits of
// their images in the core.  Then Kruskal's algorithm again, keeping for
// each vertex the sum of the bits on its tree path: a cycle's class is the
// sum of its bits, and the edge that closes it is critical when the class is
// independent of those before.
__global__ __launch_bounds__(VR_WAVE) void k_lk_cycles(LkBufs B) {
    __shared__ lk_bits ann[VR_WAVE][VR_WAVE + 1];
    __shared__ lk_bits bas[VR_WAVE];
    __shared__ uint32_t vx[VR_WAVE];
    const uint32_t lane = lane_id();
    if (B.ctl->err) return;
    const uint32_t nl = B.ctl->nlink;
    for (uint32_t i = blockIdx.x; i < nl; i += gridDim.x) {
        const uint32_t r = (uint32_t)__builtin_amdgcn_readfirstlane((int)B.list[i]);
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane(B.rng[2 * (int64_t)r]);
        const uint32_t L = (uint32_t)__builtin_amdgcn_readfirstlane(B.rng[2 * (int64_t)r + 1]) - lo;
        uint32_t k, rho;
        lk_bits row;
        lk_link(B, r, lo, L, k, row);
        const uint32_t bef = lk_before(row);
        const lk_bits A = lk_collapse(row, L, rho);
        for (int d = 0; d < 6; d++) rho = (uint32_t)__shfl((int)rho, (int)rho, VR_WAVE);
        lk_wave_sync();  // the last link's reads are done
        for (int j = 0; j < VR_WAVE; j++) ann[lane][j] = 0ull;
        vx[lane] = k;
        lk_wave_sync();
        // bits of the core's edges outside a forest: 64 at most (k_lk_pairs)
        uint32_t comp = lane, nb = 0;
        for (lk_bits xs = A; xs; xs &= xs - 1) {
            const uint32_t x = (uint32_t)__builtin_ctzll(xs);
            for (lk_bits ys = lk_rl64(row, x) & A & ~lk_low(x + 1); ys; ys &= ys - 1) {
                const uint32_t y = (uint32_t)__builtin_ctzll(ys);
                const uint32_t cx = lk_rl(comp, x), cy = lk_rl(comp, y);
                if (cx != cy) {
                    if (comp == max(cx, cy)) comp = min(cx, cy);
                } else {
                    if (lane == 0) ann[x][y] = ann[y][x] = 1ull << nb;
                    nb++;
                }
            }
        }
        lk_wave_sync();
        lk_bits live = lk_low(nb);
        for (lk_bits xs = A; xs && live; xs &= xs - 1) {
            const uint32_t x = (uint32_t)__builtin_ctzll(xs);
            const lk_bits rx = lk_rl64(row, x) & A & ~lk_low(x + 1);
            for (lk_bits ys = rx; ys && live; ys &= ys - 1) {
                const uint32_t y = (uint32_t)__builtin_ctzll(ys);
                for (lk_bits zs = rx & lk_rl64(row, y) & ~lk_low(y + 1); zs && live; zs &= zs - 1) {
                    const uint32_t z = (uint32_t)__builtin_ctzll(zs);
                    const lk_bits v = lk_rl64(ann[x][y] ^ ann[x][z] ^ ann[y][z], 0);
                    if (!v) continue;
                    const uint32_t p = (uint32_t)__builtin_ctzll(v);
                    live &= ~(1ull << p);
                    lk_wave_sync();
                    for (int j = 0; j < VR_WAVE; j++) {
                        const lk_bits e = ann[lane][j];
                        if ((e >> p) & 1ull) ann[lane][j] = e ^ v;
                    }
                    lk_wave_sync();
                }
            }
        }
        const uint32_t h = (uint32_t)__popcll(live);
        comp = lane;
        lk_bits pot = 0, tree = 0;
        uint32_t found = 0;
        for (uint32_t x = 0; x < L && found < h; x++) {
            const lk_bits rx = lk_rl64(row, x) & ~lk_low(x + 1);
            const uint32_t sx = lk_rl(rho, x);
            const lk_bits an = ann[sx][rho];  // of edge (x, lane); 0 on the diagonal
            for (lk_bits todo = rx; found < h;) {
                const uint32_t cx = lk_rl(comp, x);
                const lk_bits w = pot ^ lk_rl64(pot, x) ^ an;
                const lk_bits m = todo & (__builtin_amdgcn_ballot_w64(comp != cx) | __builtin_amdgcn_ballot_w64(w != 0));
                if (!m) break;
                const uint32_t l = (uint32_t)__builtin_ctzll(m), cl = lk_rl(comp, l);
                todo &= ~lk_low(l + 1);
                lk_bits wl = lk_rl64(w, l);
                if (cl != cx) {
                    const uint32_t old = min(cx, cl), yng = max(cx, cl);
                    if (comp == yng) {
                        pot ^= wl;
                        comp = old;
                    }
                    if (lane == x) tree |= 1ull << l;
                    if (lane == l) tree |= 1ull << x;
                    continue;
                }
                // a basis vector's lowest bit is in no later one
                for (uint32_t q = 0; q < found; q++) {
                    const lk_bits v = lk_rl64(bas[q], 0);
                    if ((wl >> __builtin_ctzll(v)) & 1ull) wl ^= v;
                }
                if (!wl) continue;
                lk_wave_sync();
                if (lane == 0) bas[found] = wl;
                lk_wave_sync();
                found++;
                // the cycle: the tree path from x to l, and (x, l)
                lk_bits M = __builtin_amdgcn_ballot_w64(lane < L && comp == cx);
                for (;;) {
                    const lk_bits leaf = __builtin_amdgcn_ballot_w64(((M >> lane) & 1ull) && lane != x && lane != l &&
                                                                     __popcll(tree & M) <= 1);
                    if (!leaf) break;
                    M &= ~leaf;
                }
                uint32_t c = 0;
                if (lane == 0) c = atomicAdd(&B.ctl->ncrit, 1u);
                c = (uint32_t)__builtin_amdgcn_readfirstlane((int)c);
                if (c >= LK_CRIT) {
                    if (lane == 0) B.ctl->err = 1u;
                    return;
                }
                lk_bits ups = ((M >> lane) & 1ull) ? tree & M & ~lk_low(lane + 1) : 0ull;
                const uint32_t nu = (uint32_t)__popcll(ups), inc = wave_incl_scan_dpp(nu);
                LkCrit &C = B.crit[c];
                for (uint32_t at = inc - nu; ups; ups &= ups - 1, at++)
                    C.uv[at] = (k << 16) | vx[__builtin_ctzll(ups)];
                const uint32_t ne = wave_last(inc);  // the path has fewer than 64 edges
                if (lane == 0) {
                    C.uv[ne] = (vx[x] << 16) | vx[l];
                    C.ne = ne + 1;
                    C.r = r;
                    C.len = 0;
                    C.tet = B.toff[r] + lk_rl(bef, x) + (long long)__popcll(rx & lk_low(l));
                }
            }
        }
    }
}

// Index of the triangle of three pairwise joined vertices, or -1.
__device__ __forceinline__ int32_t lk_triangle(const LkBufs &B, uint32_t x, uint32_t y, uint32_t z) {
    const int32_t v = max(B.R[(int64_t)x * B.n + y], max(B.R[(int64_t)x * B.n + z], B.R[(int64_t)y * B.n + z]));
    if (v < 0 || (int64_t)v >= B.K) return -1;
    const uint32_t s0 = min(x, min(y, z)), s2 = max(x, max(y, z)), s1 = x + y + z - s0 - s2;
    const lk_bits key = ((lk_bits)(uint32_t)v << 39) | ((lk_bits)s0 << 26) | ((lk_bits)s1 << 13) | s2;
    int32_t lo = B.rng[2 * (int64_t)v], hi = B.rng[2 * (int64_t)v + 1];
    // eighths, not halves: the reads of one step wait together
    while (hi - lo > 8) {
        const int32_t part = (hi - lo) / 8;
        int32_t below = 0;
#pragma unroll
        for (int32_t i = 1; i < 8; i++) below += B.tri[lo + i * part - 1] < key ? 1 : 0;
        lo += below * part;
        if (below < 7) hi = lo + part;
    }
    int32_t at = -1;
#pragma unroll
    for (int32_t i = 0; i < 8; i++)
        if (lo + i < hi && B.tri[lo + i] == key) at = lo + i;
    return at;
}

// One work-group per critical tetrahedron.  Its column is a bit per triangle
// in LDS; all triangles that are not critical are replaced, until none is
// left.  Each is replaced by older ones or one nearer its tree's root, so
// that ends, in tens of rounds of dependent reads, which bound it: a round
// goes over a list of the triangles that the last one set, the bits are
// searched only when more were set than the list holds, and four lanes share
// a triangle, one for each that replaces it.  A grid of 8 x 8 x 8 points,
// hundreds of columns: 375 us with the bits searched in each round and a
// lane to a triangle, 104 so.
__global__ __launch_bounds__(LK_BLOCK) void k_lk_expand(LkBufs B) {
    extern __shared__ __attribute__((aligned(8))) uint32_t bm[];
    __shared__ uint32_t fr[2][LK_FRONT], sum[3];  // the lists of two rounds; entries, of this round, the next and the one after
    __shared__ uint32_t nf, base, stop, top;
    const uint32_t t = threadIdx.x, nw = (uint32_t)((B.T + 31) / 32);
    if (t == 0) stop = B.ctl->err;  // one read for all: other work-groups may set it
    __syncthreads();
    if (stop) return;
    const uint32_t nc = B.ctl->ncrit;
    auto push = [&](uint32_t q, uint32_t round) {
        const uint32_t at = atomicAdd(&sum[round % 3], 1u);
        if (at < LK_FRONT) fr[round & 1][at] = q;
    };
    auto flip = [&](uint32_t x, uint32_t y, uint32_t z, uint32_t round) {
        const int32_t q = lk_triangle(B, x, y, z);
        if (q < 0) B.ctl->err = 1u;  // never: the vertices are joined
        else if (!(atomicXor(&bm[q >> 5], 1u << (q & 31)) >> (q & 31) & 1u)) push((uint32_t)q, round);
    };
    for (uint32_t c = blockIdx.x; c < nc; c += gridDim.x) {
        LkCrit &C = B.crit[c];
        __syncthreads();
        for (uint32_t x = t; x < nw; x += LK_BLOCK) bm[x] = 0;
        if (t < 3) sum[t] = 0;
        __syncthreads();
        if (t < 2 * C.ne) {
            const uint32_t uv = C.uv[t / 2];
            flip((uint32_t)B.ij[2 * (int64_t)C.r + t % 2], uv >> 16, uv & 0xFFFFu, 0);
        }
        bool more = false;  // bits to replace that are on no list
        for (uint32_t round = 0;; round++) {
            __syncthreads();
            uint32_t f = sum[round % 3];
            if (more || f > LK_FRONT) {
                __syncthreads();
                if (t == 0) sum[round % 3] = 0;
                __syncthreads();
                for (uint32_t x = t; x < nw; x += LK_BLOCK)
                    for (uint32_t y = bm[x]; y; y &= y - 1) {
                        const uint32_t q = x * 32 + (uint32_t)__builtin_ctz(y), p = B.par[q];
                        if (p != LK_ROOT || B.clr[q]) push(q, round);
                    }
                __syncthreads();
                f = sum[round % 3];
                more = f > LK_FRONT;
                f = min(f, (uint32_t)LK_FRONT);
            }
            if (f == 0) break;
            if (round == LK_ROUNDS) {
                if (t == 0) B.ctl->err = 1u;
                break;
            }
            if (t == 0) sum[(round + 2) % 3] = 0;
            for (uint32_t x = t / 4; x < f; x += LK_BLOCK / 4) {
                const uint32_t q = fr[round & 1][x], which = t & 3, p = B.par[q];
                const uint32_t clr = B.clr[q];
                const lk_bits key = B.tri[q];
                if (p == LK_ROOT && !clr) continue;  // critical: it stays
                // on the list twice if its bit was set twice: the first takes it
                uint32_t set = which == 0 ? atomicAnd(&bm[q >> 5], ~(1u << (q & 31))) >> (q & 31) & 1u : 0u;
                set = (uint32_t)__shfl((int)set, (int)(t & (VR_WAVE - 1) & ~3u));
                if (!set || p >= LK_ROOT || which == 3) continue;
                const int64_t v = (int64_t)(key >> 39);
                const uint32_t a = (uint32_t)B.ij[2 * v], b = (uint32_t)B.ij[2 * v + 1];
                const uint32_t m = ((uint32_t)(key >> 26) & 0x1FFFu) + ((uint32_t)(key >> 13) & 0x1FFFu) +
                                   ((uint32_t)key & 0x1FFFu) - a - b;
                flip(which == 2 ? b : a, which == 0 ? b : p, which == 0 ? p : m, round + 1);
            }
        }
        // the column into the pool
        __syncthreads();
        if (t == 0) nf = top = 0;
        __syncthreads();
        uint32_t own = 0, mine = 0;
        for (uint32_t x = t; x < nw; x += LK_BLOCK) {
            const uint32_t v = bm[x];
            own += (uint32_t)__popc(v);
            if (v) mine = x * 32 + 32 - (uint32_t)__builtin_clz(v);
        }
        if (own) atomicAdd(&nf, own);
        if (mine) atomicMax(&top, mine);
        __syncthreads();
        if (t == 0) {
            base = atomicAdd(&B.ctl->ptop, nf);
            if (base + nf > LK_POOL) B.ctl->err = 1u;
            else {
                C.start = base;
                C.len = nf;
                C.top = top;
            }
            own = nf;
            nf = base + own > LK_POOL ? LK_POOL : 0u;  // no room: no entry is written
        }
        __syncthreads();
        for (uint32_t x = t; x < nw; x += LK_BLOCK)
            for (uint32_t y = bm[x]; y; y &= y - 1) {
                const uint32_t at = atomicAdd(&nf, 1u);
                if (at < LK_POOL && base + at < LK_POOL) B.pool[base + at] = x * 32 + (uint32_t)__builtin_ctz(y);
            }
        __syncthreads();
    }
}

// The columns' reduction, by one work-group: there are few.  A column's pivot
// is its youngest triangle.  Those that are the first (in the order of the
// tetrahedra) with their pivot take it at once; the others are reduced one
// by one, by the columns that hold the pivots they meet.  One that meets
// a pivot held by a later column takes it over, and that one goes on in its
// place (as k_mo_reduce does): all additions are of earlier columns to later
// ones, and the pairs do not depend on which were done.
// A grid of 8 x 8 x 8 points, 141896 triangles, has hundreds of columns and
// few that meet: one after the other they took 638 us, now 16.
#define LK_START 22  // log2 of the pool: a stored column's start, its place in the order above
__global__ __launch_bounds__(LK_BLOCK) void k_lk_reduce(LkBufs B) {
    extern __shared__ __attribute__((aligned(8))) uint32_t bm[];  // first the columns' tetrahedra, then their pivots
    __shared__ uint16_t ord[LK_CRIT];
    __shared__ uint32_t pt[LK_CRIT], ps[LK_CRIT], pn[LK_CRIT];  // held pivots: triangle, column and its start, entries
    __shared__ uint32_t wait[LK_CRIT / 32];  // columns to reduce
    __shared__ uint32_t top, hit, cnt, base, np;
    const uint32_t t = threadIdx.x, nw = (uint32_t)((B.T + 31) / 32);
    if (B.ctl->err) return;
    const uint32_t nc = B.ctl->ncrit;
    if (nc == 0) return;
    long long *tet = (long long *)bm;
    for (uint32_t x = t; x < nc; x += LK_BLOCK) tet[x] = B.crit[x].tet;
    __syncthreads();
    for (uint32_t x = t; x < nc; x += LK_BLOCK) {
        const long long own = tet[x];
        uint32_t y = 0;
#pragma unroll 8
        for (uint32_t z = 0; z < nc; z++) y += tet[z] < own ? 1u : 0u;
        ord[y] = (uint16_t)x;
    }
    if (t == 0) np = 0;
    if (t < LK_CRIT / 32) wait[t] = 0;
    __syncthreads();
    for (uint32_t i = t; i < nc; i += LK_BLOCK) bm[i] = B.crit[ord[i]].len ? B.crit[ord[i]].top : 0u;
    __syncthreads();
    for (uint32_t i = t; i < nc; i += LK_BLOCK) {
        const uint32_t own = bm[i];
        if (!own) continue;
        bool first = true;
#pragma unroll 8
        for (uint32_t j = 0; j < i; j++) first &= bm[j] != own;
        if (first) {
            const uint32_t at = atomicAdd(&np, 1u);
            const LkCrit &C = B.crit[ord[i]];
            pt[at] = own - 1;
            ps[at] = C.start | i << LK_START;
            pn[at] = C.len;
        } else {
            atomicOr(&wait[i >> 5], 1u << (i & 31));
        }
    }
    auto add = [&](uint32_t start, uint32_t len) {
        for (uint32_t x = t; x < len; x += LK_BLOCK) {
            const uint32_t q = B.pool[start + x];
            atomicXor(&bm[q >> 5], 1u << (q & 31));
        }
    };
    for (uint32_t w = 0; w < LK_CRIT / 32; w++) {
        __syncthreads();
        for (uint32_t left = wait[w]; left; left &= left - 1) {
            uint32_t cur = 32 * w + (uint32_t)__builtin_ctz(left);
            uint32_t st = B.crit[ord[cur]].start, len = B.crit[ord[cur]].len;
            bool fresh = true, dirty = false;
            for (;;) {
                __syncthreads();
                if (fresh) {
                    for (uint32_t x = t; x < nw; x += LK_BLOCK) bm[x] = 0;
                    __syncthreads();
                    add(st, len);
                    fresh = dirty = false;
                }
                if (t == 0) {
                    top = 0;
                    hit = 0xFFFFFFFFu;
                }
                __syncthreads();
                uint32_t mine = 0;
                for (uint32_t x = t; x < nw; x += LK_BLOCK) {
                    const uint32_t v = bm[x];
                    if (v) mine = x * 32 + 32 - (uint32_t)__builtin_clz(v);
                }
                if (mine) atomicMax(&top, mine);
                __syncthreads();
                if (top == 0) break;  // zero: nothing dies
                const uint32_t q = top - 1, held = np;
                for (uint32_t x = t; x < held; x += LK_BLOCK)
                    if (pt[x] == q) hit = x;
                __syncthreads();
                const uint32_t j = hit;
                const uint32_t other = j == 0xFFFFFFFFu ? 0xFFFFFFFFu : ps[j] >> LK_START;
                if (other < cur) {
                    add(ps[j] & ((1u << LK_START) - 1), pn[j]);
                    dirty = true;
                    continue;
                }
                // the pivot is free, or a later column's: take it, with the column stored
                if (dirty) {
                    if (t == 0) cnt = 0;
                    __syncthreads();
                    uint32_t own = 0;
                    for (uint32_t x = t; x < nw; x += LK_BLOCK) own += (uint32_t)__popc(bm[x]);
                    if (own) atomicAdd(&cnt, own);
                    __syncthreads();
                    if (t == 0) base = atomicAdd(&B.ctl->ptop, cnt);
                    __syncthreads();
                    st = base;
                    len = cnt;
                    if (st + len > LK_POOL) {
                        if (t == 0) B.ctl->err = 1u;
                        return;
                    }
                    __syncthreads();
                    if (t == 0) cnt = 0;
                    __syncthreads();
                    for (uint32_t x = t; x < nw; x += LK_BLOCK)
                        for (uint32_t y = bm[x]; y; y &= y - 1)
                            B.pool[st + atomicAdd(&cnt, 1u)] = x * 32 + (uint32_t)__builtin_ctz(y);
                }
                const uint32_t at = j == 0xFFFFFFFFu ? held : j;
                const uint32_t old = j == 0xFFFFFFFFu ? 0u : ps[j], oldn = j == 0xFFFFFFFFu ? 0u : pn[j];
                __syncthreads();
                if (t == 0) {
                    pt[at] = q;
                    ps[at] = st | cur << LK_START;
                    pn[at] = len;
                    np = max(np, at + 1);
                }
                if (j == 0xFFFFFFFFu) break;
                cur = other;  // the column that held it goes on
                st = old & ((1u << LK_START) - 1);
                len = oldn;
                fresh = true;
            }
        }
    }
    __syncthreads();
    for (uint32_t x = t; x < np; x += LK_BLOCK) B.tri_tet[pt[x]] = B.crit[ord[ps[x] >> LK_START]].tet;
}
static_assert(LK_POOL <= 1u << LK_START && LK_CRIT <= 1u << (32 - LK_START), "a start and a column in a word");

// bits and the rest of a work-group's LDS (k_lk_expand, k_lk_reduce) in 64 KB, what a launch may ask for
static_assert(LK_MAXT / 8 + 8 * LK_FRONT + 64 <= 65536 && LK_MAXT / 8 + 14 * LK_CRIT + LK_CRIT / 8 + 64 <= 65536, "LDS");
static_assert(sizeof(LkCtl) == LINK_PAIRS_ZERO && LINK_PAIRS_MOST == VR_WAVE, "the control words, a lane per vertex");

size_t link_pairs_scratch(int64_t K, int64_t T) {
    auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
    if (T > LK_MAXT) return 0;
    return up(sizeof(LkCtl)) + up(2 * (size_t)T) + up(4 * (size_t)K) + up(sizeof(LkCrit) * LK_CRIT) +
           up(4 * (size_t)LK_POOL);
}

int link_pairs_dim2(const int32_t *R, const int32_t *ij, const unsigned long long *tri, const long long *toff,
                    const int32_t *rng, const int32_t *clr, int64_t n, int64_t K, int64_t T, long long *tri_tet,
                    void *scratch, bool *done, hipStream_t s) {
    *done = false;
    // Beyond: no attempt.  The columns' bits do not fit, and so many triangles
    // mostly come with links of more than 64 vertices anyway; the attempt was
    // lost time before the reduction (a circle of 1000 points, 4995121
    // triangles, links of up to 123: 4.85 ms with it, 4.5 without).
    if (T > LK_MAXT) return VR_OK;
    auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
    char *ws = (char *)scratch;
    auto part = [&](size_t bytes) {
        char *at = ws;
        ws += up(bytes);
        return at;
    };
    LkBufs B{};
    B.R = R;
    B.ij = ij;
    B.tri = tri;
    B.toff = toff;
    B.rng = rng;
    B.clr = clr;
    B.n = n;
    B.K = K;
    B.T = T;
    B.tri_tet = tri_tet;
    B.ctl = (LkCtl *)part(sizeof(LkCtl));
    B.par = (uint16_t *)part(2 * (size_t)T);
    B.list = (uint32_t *)part(4 * (size_t)K);
    B.crit = (LkCrit *)part(sizeof(LkCrit) * LK_CRIT);
    B.pool = (uint32_t *)part(4 * (size_t)LK_POOL);
    // Where a link can have too many vertices the host hears of it from the
    // first kernel's start, and goes to the reduction without the other three.
    // That costs nothing where none has: the others are enqueued while the first runs.
    // Before, the reduction followed a lost attempt: 80 and 125 points, all
    // edges, 318 and 858 us without the links, 364 and 968 then, 320 and 863 now.
    uint32_t *word = nullptr;
    if (n > LINK_PAIRS_MOST + 2) {
        if (!host_word(&word, &B.word)) return VR_ENOMEM;
        __atomic_store_n(word, 0u, __ATOMIC_RELEASE);
    }
    const int64_t wg = (K + LK_WPB - 1) / LK_WPB;
    hipLaunchKernelGGL(k_lk_pairs, dim3((unsigned)(wg < 2048 ? wg : 2048)), dim3(LK_BLOCK), 0, s, B);  // fills the chip
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return VR_EHIP;
    if (word) {
        uint32_t w;
        for (unsigned spins = 1; (w = __atomic_load_n(word, __ATOMIC_ACQUIRE)) == 0u; spins++) {
            if (spins % 4096 == 0) {  // a failed launch must not leave the host waiting
                e = hipStreamQuery(s);
                if (e == hipSuccess && __atomic_load_n(word, __ATOMIC_ACQUIRE) == 0u) return VR_EHIP;
                if (e != hipSuccess && e != hipErrorNotReady) return VR_EHIP;
            }
            _mm_pause();
        }
        if (w == LK_MANY) return VR_OK;
    }
    hipLaunchKernelGGL(k_lk_cycles, dim3(1024), dim3(VR_WAVE), 0, s, B);
    // as many columns at a time as fit the chip (256 compute units of 160 KB)
    const size_t lds = 4 * (size_t)((T + 31) / 32), cu = (160 * 1024) / (lds + 8 * LK_FRONT + 512);
    hipLaunchKernelGGL(k_lk_expand, dim3((unsigned)(cu < 4 ? 256 * cu : LK_CRIT)), dim3(LK_BLOCK), lds, s, B);
    hipLaunchKernelGGL(k_lk_reduce, dim3(1), dim3(LK_BLOCK), lds > 8 * LK_CRIT ? lds : 8 * LK_CRIT, s, B);
    LkCtl h{};
    e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpyAsync(&h, B.ctl, sizeof(h), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return VR_EHIP;
    *done = h.err == 0;
    return VR_OK;
}
