// k_triangles.hip -- vertex stars, triangle counting, offsets and the
// ordered triangle write.
//
// Ownership: a triangle enters the filtration with its largest edge (Section
// 2.1), so the triangles of value r are exactly {a, b, k} with edge r = {a,b}
// and both {a,k} and {b,k} ranked below r.  In rank-ordered stars, "ranked
// below r" is "before edge r": k lies in the first pb entries of b's star
// (pb = position of edge r in b's star) and in the first xa entries of a's
// star (xa = its position in a's star).  For a fixed edge the sorted vertex
// triples increase with k, and the offsets follow rank order, so the output
// is written in (value, i, j, k) order with no sort.
//
//   k_rows        per vertex: its row of the rank matrix, sorted by rank in
//                 LDS (the paper's per-column ordering, Section 4.3), gives
//                 the rank-ordered star, the position of each of its edges
//                 there, and the star again in neighbour order, each entry
//                 packing the neighbour and the position in the rank-ordered star
//   k_tri_count   per vertex a: for each edge a owns, count the neighbours in
//                 the partner's rank prefix that precede the edge in a's star
//   k_scan        exclusive scan of the counts (decoupled look-back); the
//                 last tile stores (flags, K, T) into the host-pinned mailbox
//   k_tri_write   per vertex a: for each edge a owns, walk the partner's
//                 shortest neighbour-ordered prefix list that holds the
//                 partner's entries before the edge; hits are compacted with ballot and
//                 mbcnt (the ballot/popc compaction of the paper's init_supp,
//                 Section 4.4, on 64-wide waves) into LDS and written a wave
//                 of keys at a time
//   k_tri_write_x the same writes, one wave per (vertex, eighth of its
//                 partners), each die of the chip reading one eighth of the
//                 prefix lists (a schedule the tuner may pick)
//   k_emit_edges  public edge arrays
#include "vr_device.h"

#include <hip/hip_ext.h>

#include <type_traits>

// Cloud of global vertex v, and v's local index.
__device__ __forceinline__ int vertex_cloud(const VrDev &D, long long v) {
    return (D.C == 1) ? 0 : (int)D.vcloud[v];
}

// --------------------------------------------------------------- k_rows ----
// Star slots: vertex v of a cloud with n points owns n entries of star_r
// and star_nbr at star_slot(mbase, n, v).
__device__ __forceinline__ uint32_t star_slot(uint32_t mbase, int n, int v) { return mbase + (uint32_t)v * (uint32_t)n; }

// Prefix lists: for a star of deg entries, list j (j = 1..VR_PLISTS) holds
// the entries whose position in the rank-ordered star is below
// plist_len(j) = ceil(j deg / VR_PLISTS), in neighbour order, each packing
// (neighbour | (0xFFFF - position) << 16) and starting on a 128-byte line;
// the last list is the whole star.  An edge's triangles lie among its partner's
// first pb entries, which the partner's list plist_pick(pb) holds: walking
// that list instead of the whole star leaves the walk in neighbour order
// (so hits still come out in k order) while cutting the candidates to about
// half on average (cutting at each eighth instead left the writer's time
// unchanged and slowed the star stage).  Vertex v of a cloud owns
// VR_PLIST_PER n + 65 VR_PLISTS entries of star_k from plist_region, rounded
// up to a line (31 entries at most), and its lists take at most
// (VR_PLISTS + 1) deg / 2 + VR_PLISTS + 31 VR_PLISTS of them.
#define VR_LINE 32u  // entries of star_k in a 128-byte line
__device__ __forceinline__ uint32_t plist_len(uint32_t j, uint32_t deg) { return (j * deg + VR_PLISTS - 1) / VR_PLISTS; }
__device__ __forceinline__ uint32_t plist_off(uint32_t j, uint32_t deg) {
    uint32_t o = 0;
    for (uint32_t i = 1; i < j; i++) o += (plist_len(i, deg) + VR_LINE - 1) & ~(VR_LINE - 1);
    return o;
}
// smallest j with plist_len(j) >= p; 0 for p = 0 (no candidates)
__device__ __forceinline__ uint32_t plist_pick(uint32_t p, uint32_t deg) {
    return p == 0 ? 0u : (p * VR_PLISTS + deg - 1) / deg;
}
__device__ __forceinline__ uint32_t plist_region(uint32_t mbase, uint32_t vbase, int n, int v) {
    const uint32_t per = VR_PLIST_PER * (uint32_t)n + (VR_WAVE + 1) * VR_PLISTS;
    const uint32_t o = VR_PLIST_PER * mbase + (uint32_t)(VR_WAVE + 1) * VR_PLISTS * vbase + (uint32_t)v * per;
    return (o + VR_LINE - 1) & ~(VR_LINE - 1);
}
// an entry, and the bound that exactly the entries of position below p pass
// (entry > bound); 0 passes none, so what a bounded load returns past a
// list's end is never a candidate
__device__ __forceinline__ uint32_t plist_entry(uint32_t k, uint32_t pos) { return k | ((0xFFFFu - pos) << 16); }
__device__ __forceinline__ uint32_t plist_bound(uint32_t p) { return ((0xFFFFu - p) << 16) | 0xFFFFu; }

// One work-group per vertex v reads row v of the rank matrix that k_edges
// scattered into v's star_r slot (entry k = this build's tag << 24 | rank
// of edge {v,k} within the cloud).  Entries of pairs that are not kept are
// left from earlier use of the memory: an entry counts only when it carries
// the tag and names a kept edge of this cloud whose endpoints are {v, k} in
// the sorted edge list, so the matrix is never cleared (the paper avoids
// re-initialising its per-column work array the same way, Section 4.3); the
// tag only spares most stale entries the look-up (the stars written over
// the rows carry tag 0, and tags repeat only every 255 builds).  The kept entries, in neighbour order, are sorted
// by rank in LDS (bitonic), which orders v's edges the way the paper's
// per-column ordering of the distance matrix does (Section 4.3).  Outputs:
// v's star in rank order (rank within the cloud, written over the row, and
// the neighbour), each edge's position in it (pos), the prefix lists (the
// star in neighbour order with those positions, whole and cut at each
// 1/VR_PLISTS of the rank order) and its size.
//
// Wave w reads the row's entries [64 S w, 64 S (w+1)) in S steps of 64, so
// the neighbour order is the order of (wave, step, lane); S * 256 >= n.
#define VR_ROWS_COUNT_MAX 512  // largest star ranked by counting (two keys per thread)

// Counting rank of a star of 1 <= deg <= NK * 256 entries: keys[x] = rank of the
// x-th neighbour (padded to a multiple of 4 with ~0), nbr[x] = that
// neighbour.  Writes the star in rank order over the row, its neighbours,
// the edges' positions, and the neighbour-ordered star (sk, and keys[x]
// once every key is read).
template <int NK>
__device__ __forceinline__ void rows_count_rank(const VrDev &D, uint32_t *keys, const uint16_t *nbr, uint32_t deg,
                                                uint32_t *__restrict__ row, uint32_t s0, uint32_t *__restrict__ sk,
                                                int v, long long kb) {
    uint32_t own[NK], y[NK];
#pragma unroll
    for (int i = 0; i < NK; i++) {
        const uint32_t x = threadIdx.x + VR_BLOCK * i;
        own[i] = keys[min(x, deg - 1)];
        y[i] = 0;
    }
    const uint4 *k4 = (const uint4 *)keys;
    for (uint32_t q = 0; q < (deg + 3) / 4; q++) {
        const uint4 e = k4[q];
#pragma unroll
        for (int i = 0; i < NK; i++)
            y[i] += (uint32_t)(e.x < own[i]) + (uint32_t)(e.y < own[i]) + (uint32_t)(e.z < own[i]) + (uint32_t)(e.w < own[i]);
    }
    uint32_t kx[NK];
#pragma unroll
    for (int i = 0; i < NK; i++) kx[i] = nbr[min(threadIdx.x + VR_BLOCK * i, deg - 1)];
    __syncthreads();  // every key is read: keys[] takes the packed entries
#pragma unroll
    for (int i = 0; i < NK; i++) {
        const uint32_t x = threadIdx.x + VR_BLOCK * i;
        if (x < deg) {
            const uint32_t k = kx[i], lr = own[i];
            row[y[i]] = lr;
            D.star_nbr[s0 + y[i]] = (uint16_t)k;
            D.epos[2 * (kb + lr) + ((uint32_t)v < k ? 0 : 1)] = (uint16_t)y[i];
            sk[x] = plist_entry(k, y[i]);
            keys[x] = plist_entry(k, y[i]);
        }
    }
}

template <int S>
__global__ __launch_bounds__(VR_BLOCK) void k_rows(VrDev D) {
    extern __shared__ uint32_t lds[];  // P sort keys, then the position of each neighbour (u16)
    __shared__ uint32_t sh_w[VR_WAVES];
    __shared__ uint32_t sh_l[VR_PLISTS - 1][VR_WAVES];
    const long long vg = blockIdx.x;
    const int c = vertex_cloud(D, vg);
    const int v = (int)(vg - D.cl[c].vbase), n = D.cl[c].n;
    const long long kb = kept_base(D, c), Kc = kept_count(D, c);
    const uint32_t s0 = star_slot((uint32_t)D.cl[c].mbase, n, v);
    uint32_t *__restrict__ row = D.star_r + s0;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int per = (n + VR_BLOCK - 1) / VR_BLOCK;  // steps this launch needs (<= S)
    // Loads are issued unconditionally at clamped addresses: a guarded load
    // makes the compiler wait for it before the next one is issued.
    uint32_t rr[S];
#pragma unroll
    for (int s = 0; s < S; s++) rr[s] = row[min((w * per + s) * VR_WAVE + lane, n - 1)];
    // candidates: entries with the tag and a kept rank; rr = rank within the
    // cloud.  Up to 1024 points each is looked up in the sorted edge list at
    // once; beyond, after compaction, and nearly always all of them are
    // edges, else each entry of the row is looked up by itself.  At once took
    // 133 of 213 us on 8192 points with 270 neighbours each (160 us now) and
    // 19 of 85 on 4000 with 400 (84), but on 777 points with 230 it is
    // faster (24 us, 26).
    auto endpoints = [&](uint32_t k) {
        return (k < (uint32_t)v) ? ((k << 16) | (uint32_t)v) : (((uint32_t)v << 16) | k);
    };
    unsigned long long mk[S];  // entries taken in each step (wave-uniform)
#pragma unroll
    for (int s = 0; s < S; s++) {
        const int k = (w * per + s) * VR_WAVE + lane;
        const uint32_t lr = rr[s] & 0xFFFFFFu;
        bool in = s < per && k < n && k != v && (rr[s] >> 24) == D.tag && (long long)lr < Kc;
        if constexpr (S <= 4) {
            const uint32_t ij = D.se_ij[kb + (in ? lr : 0u)];  // kept base itself when not in (se_ij has room)
            in = in && ij == endpoints((uint32_t)k);
        }
        mk[s] = __builtin_amdgcn_ballot_w64(in);
        rr[s] = lr;
    }
    // sort keys: local ranks in neighbour order (entry x = x-th neighbour
    // taken), padded, and the neighbours
    uint32_t run, deg, P;
    uint16_t *pk;
    auto compact = [&]() {
        uint32_t cw = 0;
#pragma unroll
        for (int s = 0; s < S; s++) cw += (uint32_t)__popcll(mk[s]);
        if (lane == 0) sh_w[w] = cw;
        __syncthreads();
        run = deg = 0;
#pragma unroll
        for (int i = 0; i < VR_WAVES; i++) {
            const uint32_t t = sh_w[i];
            if (i < w) run += t;
            deg += t;
        }
        P = VR_WAVE;
        while (P < deg) P <<= 1;
        pk = (uint16_t *)(lds + P);
        for (uint32_t y = deg + threadIdx.x; y < P; y += VR_BLOCK) lds[y] = 0xFFFFFFFFu;
        uint32_t x = run;
#pragma unroll
        for (int s = 0; s < S; s++) {
            const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(mk[s] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mk[s], x));
            if ((mk[s] >> lane) & 1ull) {
                lds[at] = rr[s];
                pk[at] = (uint16_t)((w * per + s) * VR_WAVE + lane);
            }
            x += (uint32_t)__popcll(mk[s]);
        }
        __syncthreads();
    };
    compact();
    if constexpr (S > 4) {
        bool bad = false;
        for (uint32_t x = threadIdx.x; x < deg; x += VR_BLOCK) bad |= D.se_ij[kb + lds[x]] != endpoints(pk[x]);
        if (__syncthreads_or(bad)) {
#pragma unroll
            for (int s = 0; s < S; s++) {
                const bool in = (mk[s] >> lane) & 1ull;
                const uint32_t ij = D.se_ij[kb + (in ? rr[s] : 0u)];
                mk[s] = __builtin_amdgcn_ballot_w64(in && ij == endpoints((uint32_t)((w * per + s) * VR_WAVE + lane)));
            }
            compact();
        }
    }
    // small stars are ranked by counting, larger ones sorted (bitonic, where
    // pk becomes the position of neighbour k)
    const bool by_count = deg <= VR_ROWS_COUNT_MAX;
    uint32_t *lb = D.star_k + plist_region((uint32_t)D.cl[c].mbase, (uint32_t)D.cl[c].vbase, n, v);
    uint32_t *sk = lb + plist_off(VR_PLISTS, deg);  // the last list: the whole star
    if (by_count) {
        // rank-order position of entry x = number of smaller keys (ranks
        // are distinct); every lane reads the same keys, which LDS
        // broadcasts
        if (deg == 0) {
        } else if (deg <= VR_BLOCK) {
            rows_count_rank<1>(D, lds, pk, deg, row, s0, sk, v, kb);
        } else {
            rows_count_rank<2>(D, lds, pk, deg, row, s0, sk, v, kb);
        }
    } else {
        // Bitonic sort.  Wave w's pairs in a stage with distance j <= 64 lie
        // in its own 128-key blocks, so only stages with j >= 128 exchange
        // keys between waves and need the work-group barrier; the others
        // need the wave's LDS accesses in order, which a wave's LDS
        // instructions are.
        for (uint32_t kk = 2; kk <= P; kk <<= 1) {
            for (uint32_t j = kk >> 1; j > 0; j >>= 1) {
                if (j >= 2 * VR_WAVE) __syncthreads();
                for (uint32_t i = threadIdx.x; i < P / 2; i += VR_BLOCK) {
                    const uint32_t lo = 2 * i - (i & (j - 1)), hi = lo + j;
                    const uint32_t x0 = lds[lo], x1 = lds[hi];
                    if ((x0 > x1) == ((lo & kk) == 0)) {
                        lds[lo] = x1;
                        lds[hi] = x0;
                    }
                }
                if (j >= 2 * VR_WAVE) __syncthreads();
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
        }
        __syncthreads();
        // rank order: entry y is the y-th smallest rank; its neighbour comes
        // from the edge list (lanes past the star repeat the last entry's
        // loads and store nothing)
        uint32_t ij[S];
#pragma unroll
        for (int i = 0; i < S; i++) ij[i] = D.se_ij[kb + lds[min(threadIdx.x + VR_BLOCK * i, deg - 1)]];
#pragma unroll
        for (int i = 0; i < S; i++) {
            const uint32_t y = threadIdx.x + VR_BLOCK * i;
            if (y < deg) {
                const uint32_t lr = lds[y];
                const uint32_t k = ((ij[i] >> 16) == (uint32_t)v) ? (ij[i] & 0xFFFFu) : (ij[i] >> 16);
                row[y] = lr;
                D.star_nbr[s0 + y] = (uint16_t)k;
                D.epos[2 * (kb + lr) + ((uint32_t)v < k ? 0 : 1)] = (uint16_t)y;
                pk[k] = (uint16_t)y;
            }
        }
        __syncthreads();
        uint32_t x = run;
#pragma unroll
        for (int s = 0; s < S; s++) {
            const uint32_t k = (uint32_t)((w * per + s) * VR_WAVE + lane);
            const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(mk[s] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mk[s], x));
            if ((mk[s] >> lane) & 1ull) {
                const uint32_t e = plist_entry(k, pk[k]);
                sk[at] = e;
                lds[at] = e;
            }
            x += (uint32_t)__popcll(mk[s]);
        }
    }
    // lds[0, deg) holds the star in neighbour order (packed); the shorter
    // lists are its entries below each cut, compacted in order
    __syncthreads();
    {
        uint32_t cut[VR_PLISTS - 1], off[VR_PLISTS - 1], run[VR_PLISTS - 1];
#pragma unroll
        for (int j = 0; j < VR_PLISTS - 1; j++) {
            cut[j] = plist_bound(plist_len((uint32_t)j + 1, deg));
            off[j] = plist_off((uint32_t)j + 1, deg);
            run[j] = 0;
        }
        for (uint32_t x0 = 0; x0 < deg; x0 += VR_BLOCK) {
            const uint32_t x = x0 + threadIdx.x;
            const uint32_t e = x < deg ? lds[x] : 0u;
            unsigned long long m[VR_PLISTS - 1];
#pragma unroll
            for (int j = 0; j < VR_PLISTS - 1; j++) {
                m[j] = __builtin_amdgcn_ballot_w64(e > cut[j]);
                if (lane == 0) sh_l[j][w] = (uint32_t)__popcll(m[j]);
            }
            __syncthreads();
#pragma unroll
            for (int j = 0; j < VR_PLISTS - 1; j++) {
                uint32_t before = 0, tot = 0;
#pragma unroll
                for (int i = 0; i < VR_WAVES; i++) {
                    const uint32_t t = sh_l[j][i];
                    if (i < w) before += t;
                    tot += t;
                }
                if ((m[j] >> lane) & 1ull)
                    lb[off[j] + run[j] + __builtin_amdgcn_mbcnt_hi((uint32_t)(m[j] >> 32),
                                                                   __builtin_amdgcn_mbcnt_lo((uint32_t)m[j], before))] = e;
                run[j] += tot;
            }
            __syncthreads();  // sh_l is rewritten by the next chunk
        }
    }
    if (threadIdx.x == 0) D.deg[vg] = deg;
}

static uint32_t pow2_at_least(uint32_t x) {
    uint32_t p = VR_WAVE;
    while (p < x) p <<= 1;
    return p;
}

void launch_rows(const VrDev &D, hipStream_t s) {
    const int steps = (D.maxn + VR_BLOCK - 1) / VR_BLOCK;
    // sort keys (P <= pow2(maxn)) and the positions of the neighbours
    const size_t lds = 4 * (size_t)pow2_at_least((uint32_t)D.maxn) + 2 * (size_t)((D.maxn + 1) & ~1);
    const dim3 grid((unsigned)D.V);
    if (steps <= 4) hipLaunchKernelGGL(k_rows<4>, grid, dim3(VR_BLOCK), lds, s, D);
    else if (steps <= 8) hipLaunchKernelGGL(k_rows<8>, grid, dim3(VR_BLOCK), lds, s, D);
    else if (steps <= 16) hipLaunchKernelGGL(k_rows<16>, grid, dim3(VR_BLOCK), lds, s, D);
    else hipLaunchKernelGGL(k_rows<32>, grid, dim3(VR_BLOCK), lds, s, D);
}

// ------------------------------------------------- shared enumeration core ----
// One work-group per vertex a with Pa[k] = position of edge {a,k} in a's
// star (0xFFFF when k is no neighbour) staged in LDS.  The star is taken in
// chunks of EB entries (EB = the work-group size, 256 or 512, a schedule
// choice like the work-groups per vertex); the edges a owns in a chunk are compacted and
// cut into wave-sized pieces of candidates; each wave takes a contiguous run
// of whole edges holding about 1/8 of the pieces.  The metadata of up to 64
// edges sits in lane registers; the loads of the next edge are issued before
// the current edge is consumed.
// An edge's candidates are loaded NP pieces of 64 at a time (NP a schedule
// choice: 2, 4 or 8 for the count, 4 or 8 for the write); longer candidate
// lists finish piece by piece.

template <int EB>
struct EnumLds {
    static constexpr int W = EB / VR_WAVE;
    uint32_t r[EB];
    uint32_t b[EB];
    uint32_t sb[EB];      // start of the partner's star
    uint32_t len[EB];     // candidates of the edge
    uint32_t pb[EB];      // position of the edge in the partner's star
    uint32_t xa[EB];      // position of the edge in a's star
    uint32_t cb[EB + 1];  // first piece of the edge
    uint32_t ew[W + 1];   // first edge of each wave
    uint32_t scan[W];
    uint32_t scan2[W];
};

template <int EB>
__device__ __forceinline__ uint32_t enum_excl_scan(uint32_t x, uint32_t *sh, uint32_t *total) {
    constexpr int ENUM_WAVES = EB / VR_WAVE;
    const uint32_t inc = wave_incl_scan_dpp(x);
    const int w = threadIdx.x / VR_WAVE;
    if (lane_id() == VR_WAVE - 1) sh[w] = inc;
    __syncthreads();
    uint32_t off = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < ENUM_WAVES; i++) {
        const uint32_t v = sh[i];
        if (i < w) off += v;
        tot += v;
    }
    __syncthreads();
    *total = tot;
    return off + inc - x;
}

// Compact the edges a owns among star entries [p0, p0+EB) and split
// them by piece count: `parts` work-groups share a vertex (part = this one's
// index), each taking a contiguous slice, cut again into one run per wave.
// When `parts` is a multiple of 8, the work-groups of a vertex are split
// by the partner instead: work-group `part` takes only the edges whose
// partner lies in the (part mod 8)-th eighth of the cloud's vertices, and
// the parts / 8 work-groups of that eighth share them as above.  Work-groups
// are handed to the chip's 8 dies (XCDs, each with its own L2) in turn, so
// block index mod 8 names the die, and with parts a multiple of 8 it equals
// part mod 8: each die then reads the stars of one eighth of the vertices,
// which its L2 can hold, instead of all of them.  WRITE: an edge is written at the
// endpoint whose partner's prefix list (the shortest holding the partner's
// entries before the edge) is shorter; candidates = that list, in
// neighbour order.  Otherwise it is counted at the endpoint
// whose partner has the shorter rank prefix (candidates = that prefix).
// The first chunk's star entries come preloaded (r0, b0: see stage_pos).
// Which endpoint writes edge {a, b}: a walks b's shortest prefix list
// holding b's first pb entries, or b walks a's holding a's first xa; the
// shorter walk wins, the smaller vertex on a tie (so exactly one endpoint
// owns the edge).  xa, da: the edge's position in a's star and a's degree;
// pb: its position in b's star.  For a's side: len = the list's length and
// sb = where it starts in star_k.
__device__ __forceinline__ bool write_side(const VrDev &D, uint32_t a, uint32_t b, uint32_t xa, uint32_t da,
                                           uint32_t pb, uint32_t vb, uint32_t mb, int n, uint32_t &len,
                                           uint32_t &sb) {
    const uint32_t db = D.deg[vb + b];
    const uint32_t jb = plist_pick(pb, db), ja = plist_pick(xa, da);
    const uint32_t cb = jb ? plist_len(jb, db) : 0u, ca = ja ? plist_len(ja, da) : 0u;
    len = cb;
    sb = plist_region(mb, vb, n, (int)b) + plist_off(jb ? jb : 1u, db);
    return cb < ca || (cb == ca && a < b);
}

template <bool WRITE, int EB>
__device__ __forceinline__ int load_chunk(const VrDev &D, int a, uint32_t vb, uint32_t mb, int n, uint32_t kb,
                                          uint32_t s0, uint32_t s1, uint32_t p0, EnumLds<EB> &L, int part,
                                          int parts, uint32_t r0, uint32_t b0) {
    constexpr int ENUM_WAVES = EB / VR_WAVE;
    const uint32_t p = p0 + threadIdx.x;
    bool owned = false;
    uint32_t r = 0, b = 0, pb = 0, sb = 0, len = 0;
    const uint32_t x = p - s0;
    const bool by_partner = (parts & 7) == 0;
    const uint32_t eighth = (uint32_t)(part & 7);
    if (by_partner) {
        part >>= 3;
        parts >>= 3;
    }
    if (p < s1) {
        r = kb + (p0 == s0 ? r0 : D.star_r[p]);  // global kept-edge index
        b = p0 == s0 ? b0 : D.star_nbr[p];
        // edge {b,a} in b's star: the count reads it from the per-edge
        // positions (4 bytes per kept edge, written by the star stage) and
        // stores it beside the entry, where the write reads it in order
        if (WRITE) {
            pb = D.ppos[p];
        } else {
            pb = D.epos[2 * r + (b < (uint32_t)a ? 0u : 1u)];
            D.ppos[p] = (uint16_t)pb;
        }
        sb = star_slot(mb, n, (int)b);
        if (WRITE) {
            owned = write_side(D, (uint32_t)a, b, x, s1 - s0, pb, vb, mb, n, len, sb);
        } else {
            owned = pb < x || (pb == x && (uint32_t)a < b);
            len = pb;
        }
        if (by_partner) owned = owned && (b * 8u) / (uint32_t)n == eighth;
    }
    uint32_t m, C;
    const uint32_t idx = enum_excl_scan<EB>(owned ? 1u : 0u, L.scan, &m);
    const uint32_t pieces = owned ? (len + VR_WAVE - 1) / VR_WAVE : 0u;
    const uint32_t cbeg = enum_excl_scan<EB>(pieces, L.scan2, &C);
    if (owned) {
        L.r[idx] = r;
        L.b[idx] = b;
        L.sb[idx] = sb;
        L.len[idx] = len;
        L.pb[idx] = pb;
        L.xa[idx] = x;
        L.cb[idx] = cbeg;
    }
    if (threadIdx.x == 0) L.cb[m] = C;
    __syncthreads();
    if ((int)threadIdx.x <= ENUM_WAVES) {
        // this work-group's slice of the pieces, then one run per wave
        const unsigned long long gw = (unsigned long long)part * ENUM_WAVES + threadIdx.x;
        const uint32_t target = (uint32_t)(((unsigned long long)C * gw) / ((unsigned long long)parts * ENUM_WAVES));
        int lo = 0, hi = (int)m;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (L.cb[mid] < target) lo = mid + 1;
            else hi = mid;
        }
        L.ew[threadIdx.x] = (gw == (unsigned long long)parts * ENUM_WAVES) ? m : (uint32_t)lo;
    }
    __syncthreads();
    return (int)m;
}

__device__ __forceinline__ uint32_t rl(uint32_t v, int lane) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
}

// Pa[k] = position of neighbour k in a's rank-ordered star (0xFFFF for
// non-neighbours).  The star's first EB entries (rank and neighbour) are
// loaded before the table is cleared and handed back for the first chunk,
// so neither waits on the other.
template <int EB>
__device__ __forceinline__ void stage_pos(const VrDev &D, int n, uint16_t *Pa, uint32_t s0, uint32_t s1,
                                          uint32_t &r0, uint32_t &b0) {
    r0 = b0 = 0;
    if (s1 > s0) {  // clamped loads: every lane issues them
        const uint32_t pc = min(s0 + (uint32_t)threadIdx.x, s1 - 1);
        r0 = D.star_r[pc];
        b0 = D.star_nbr[pc];
    }
    for (int x = threadIdx.x; x < (n + 7) / 8; x += EB) ((uint4 *)Pa)[x] = make_uint4(~0u, ~0u, ~0u, ~0u);
    __syncthreads();
    if (s0 + threadIdx.x < s1) Pa[b0] = (uint16_t)threadIdx.x;
    for (uint32_t p = s0 + threadIdx.x + EB; p < s1; p += EB) Pa[D.star_nbr[p]] = (uint16_t)(p - s0);
    __syncthreads();
}

template <int EB>
size_t enum_lds(int maxn) { return 2 * (size_t)((maxn + 7) & ~7) + sizeof(EnumLds<EB>); }

// A list of candidates (or slots) as a bounded buffer: `bytes` bytes from the
// address hi:lo (all wave-uniform).  Loads past its end return 0 and stores
// there are dropped, so pieces need neither clamped addresses nor padding
// nor a bounds test: three instructions less per piece loaded and two per
// piece counted, 20 less per edge written.  64-dimensional mixture, 4000
// points, 0.8 million edges: 58 million instructions instead of 71 in the
// count (110 -> 103 us), 145 instead of 159 in the write.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t list_buffer(uint32_t lo, uint32_t hi, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((void *)(((unsigned long long)hi << 32) | lo), 0, (int)bytes, 0x00027000);
}

// Prefetch of one edge's candidates, NP pieces of 64.  Every load is issued
// unconditionally, so that the compiler can count outstanding loads exactly:
// a conditional load makes it wait for every load in flight, the next edge's
// prefetch included.  Pieces past the candidates are never consumed.
template <int NP>
__device__ __forceinline__ void issue_prefix(__amdgpu_buffer_rsrc_t list, uint32_t (&kk)[NP]) {
    const uint32_t lane = threadIdx.x & 63;
#pragma unroll
    for (int j = 0; j < NP; j++)
        kk[j] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(list, (int)(lane * 2u + (uint32_t)(j * VR_WAVE * 2)), 0, 0);
}

template <int NP>
__device__ __forceinline__ void issue_list(__amdgpu_buffer_rsrc_t list, uint32_t (&kk)[NP]) {
    const uint32_t lane = threadIdx.x & 63;
#pragma unroll
    for (int j = 0; j < NP; j++)
        kk[j] = __builtin_amdgcn_raw_buffer_load_b32(list, (int)(lane * 4u + (uint32_t)(j * VR_WAVE * 4)), 0, 0);
}

// ----------------------------------------------------------- k_tri_count ----
template <int EB, int NP>
__global__ __launch_bounds__(EB) void k_tri_count(VrDev D, int parts) {
    extern __shared__ uint32_t lds[];
    const long long ag = blockIdx.x / parts;
    const int part = blockIdx.x % parts;
    const int c = vertex_cloud(D, ag);
    const uint32_t vb = (uint32_t)D.cl[c].vbase;
    const int a = (int)(ag - vb), n = D.cl[c].n;
    uint16_t *Pa = (uint16_t *)lds;
    EnumLds<EB> &L = *(EnumLds<EB> *)((char *)lds + 2 * ((D.maxn + 7) & ~7));
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t mb = (uint32_t)D.cl[c].mbase, kb = (uint32_t)kept_base(D, c);
    const uint32_t s0 = star_slot(mb, n, a), s1 = s0 + D.deg[ag];
    uint32_t r0, b0;
    stage_pos<EB>(D, n, Pa, s0, s1, r0, b0);
    const uint32_t p_0 = Pa[0];
    for (uint32_t p0 = s0; p0 < s1; p0 += EB) {
        load_chunk<false, EB>(D, a, vb, mb, n, kb, s0, s1, p0, L, part, parts, r0, b0);
        const int w_lo = __builtin_amdgcn_readfirstlane((int)L.ew[w]);
        const int w_hi = __builtin_amdgcn_readfirstlane((int)L.ew[w + 1]);
        for (int eb = w_lo; eb < w_hi; eb += VR_WAVE) {
            const int ne = min(VR_WAVE, w_hi - eb);
            // one edge's parameters per lane: its list's address and bytes
            uint32_t vr = 0, vlo = 0, vhi = 0, vby = 0, vxa = 0;
            if (lane < ne) {
                vr = L.r[eb + lane];
                const unsigned long long at = (unsigned long long)(D.star_nbr + L.sb[eb + lane]);
                vlo = (uint32_t)at;
                vhi = (uint32_t)(at >> 32);
                vby = 2u * L.len[eb + lane];
                vxa = L.xa[eb + lane];
            }
            uint32_t mycnt = 0;
            auto list_of = [&](int el) { return list_buffer(rl(vlo, el), rl(vhi, el), rl(vby, el)); };
            // count of edge el from its prefetched pieces; the lanes past the
            // list's end of its last piece hold neighbour 0
            auto count_edge = [&](int el, const uint32_t (&kk)[NP]) {
                const uint32_t xa = rl(vxa, el), by = rl(vby, el);
                uint32_t c = 0;
#pragma unroll
                for (int j = 0; j < NP; j++) {
                    if ((uint32_t)(j * VR_WAVE * 2) < by)  // whole pieces past the end are skipped
                        // lane mask straight from the comparison (unsigned less-than: 36)
                        c += (uint32_t)__popcll(__builtin_amdgcn_uicmp((uint32_t)Pa[kk[j]], xa, 36));
                }
                for (uint32_t y0 = NP * VR_WAVE * 2; y0 < by; y0 += 4 * VR_WAVE * 2) {
                    uint32_t k[4];
#pragma unroll
                    for (int j = 0; j < 4; j++)
                        k[j] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(
                            list_of(el), (int)(2 * lane + j * VR_WAVE * 2), (int)y0, 0);
#pragma unroll
                    for (int j = 0; j < 4; j++)
                        if (y0 + (uint32_t)(j * VR_WAVE * 2) < by)
                            c += (uint32_t)__popcll(__builtin_amdgcn_uicmp((uint32_t)Pa[k[j]], xa, 36));
                }
                if (lane == el) mycnt = c;
            };
            // ping-pong prefetch one edge ahead; past the last edge the loads
            // repeat the last edge's (never consumed)
            uint32_t kA[NP], kB[NP];
            issue_prefix(list_of(0), kA);
            for (int el = 0; el < ne; el += 2) {
                const int e1 = min(el + 1, ne - 1), e2 = min(el + 2, ne - 1);
                issue_prefix(list_of(e1), kB);
                count_edge(el, kA);
                issue_prefix(list_of(e2), kA);
                if (el + 1 < ne) count_edge(el + 1, kB);
            }
            // the lanes past the ends counted neighbour 0 each time it passed
            if (p_0 < vxa) mycnt -= (0u - vby / 2u) & (VR_WAVE - 1);
            if (lane < ne) D.cnt[vr] = mycnt;
        }
        __syncthreads();
    }
}

// Work-groups per vertex, the default when no tuned value is known: enough
// groups to spread heavy vertices over many compute units when the cloud is
// small, each with work enough for its setup.  Write, four and five a vertex:
// 39 and 35 us (1000-point circle), 510 and 491 (1088 points, all edges), 42
// and 41 (777 points); eight split by partner: 30 us against 21 with five on
// 300 points; 2000 points: 79 with three, 84 with one of 512 threads.  Count:
// 21 us with four or five, 25 with eight on the circle.
// Larger clouds of many neighbours, as K edges known on the host tell (else
// -1), write with two, the more the points the later: a short launch is left
// with its heaviest vertices, a long one is not.  One and two, us, points
// evenly in the cube: 2500 points with 270, 320 and 420 neighbours 105 and
// 105, 133 and 130, 199 and 179; 4000 with 320, 384, 420 and 700 185 and
// 186, 238 and 241, 277 and 268, 723 and 645; 6000 with 384, 420 and 500 326
// and 339, 379 and 383, 518 and 493; 8192 with 384, 420, 500 and 700 433 and
// 454, 505 and 517, 691 and 667, 1318 and 1250; batches of 2 and of 4 of 2500,
// 400 and 500 302 and 303, 448 and 407; 543 and 565, 787 and 766.  In six
// dimensions two are better from about 50 neighbours less on.  The mixture's
// 4000 points with 400: 268 and 251.
// Up to 128 points seven or eight are the same (7 and 8 us).
static int enum_parts(long long V, long long groups, long long most) {
    const long long p = groups / (V > 0 ? V : 1);
    if (V <= 128) most = 7;
    return p < 1 ? 1 : (int)(p > most ? most : p);
}
int enum_parts_count(long long V) { return enum_parts(V, 4096, 4); }
int enum_parts_write(long long V, long long C, long long K) {
    if (enum_block(V, C) == 256) return enum_parts(V, 6144, 5);
    const int p = enum_parts(V, 3072, 5);
    return p < 2 && 2 * K >= V * (250 + (V < 8192 ? V : 8192) / 32) ? 2 : p;
}

// Work-group size, the default: 256 threads for small clouds (more
// work-groups in flight), 512 for large ones (fewer chunk barriers).  What
// counts is the size of one cloud: 32 clouds of 50 to 2000 points took 138
// (count) and 281 us (write) with 512 threads, 95 and 202 with 256; one
// cloud of 8192 points 145 and 283 with 512, 160 and 295 with 256.
int enum_block(long long V, long long C) { return V <= 2048 * C ? 256 : 512; }

// Pieces loaded at a time, the defaults.  Count: its candidates are rank
// prefixes, often short: 4, or 8 where K edges are known to give 768
// neighbours a vertex.  4 and 8, us: 800 points with 600, 768 and all edges
// 57 and 59, 76 and 73, 77 and 74; 1088 with 600, 768 and all 80 and 79, 110
// and 100, 166 and 149; 2048 with 400, 768 and 1400 82 and 82, 231 and 191,
// 605 and 493; 4000 evenly in the cube with 400, 768 and 1000 134 and 128,
// 423 and 352, 710 and 591, but the mixture's 400 100 and 109.  Write (prefix
// lists): 8.
int enum_pieces_count(long long V, long long K) { return K >= 384 * V ? 8 : 4; }
int enum_pieces_write() { return 8; }

template <int EB, int NP>
static void count_at(const VrDev &D, dim3 grid, hipStream_t s) {
    hipLaunchKernelGGL((k_tri_count<EB, NP>), grid, dim3(EB), enum_lds<EB>(D.maxn), s, D, D.parts_count);
}

template <int EB>
static void count_eb(const VrDev &D, dim3 grid, hipStream_t s) {
    switch (D.pieces_count) {
    case 2: count_at<EB, 2>(D, grid, s); break;
    case 8: count_at<EB, 8>(D, grid, s); break;
    default: count_at<EB, 4>(D, grid, s); break;
    }
}

void launch_tri_count(const VrDev &D, hipStream_t s) {
    const dim3 grid((unsigned)(D.V * D.parts_count));
    switch (D.eb_count) {
    case 128: count_eb<128>(D, grid, s); break;
    case 256: count_eb<256>(D, grid, s); break;
    default: count_eb<512>(D, grid, s); break;
    }
}

// ---------------------------------------------------------------- k_scan ----
// S == 0: tile = blockIdx.x (every tile's work-group is launched), with the
// tile's counts loaded together with K (clamped to the buffer; counts past
// K are never used); else tiles are claimed S at a time from a ticket.
__global__ __launch_bounds__(VR_BLOCK) void k_scan(VrDev D, int S) {
    __shared__ unsigned long long sh_w[VR_WAVES];
    __shared__ unsigned long long sh_prefix;
    __shared__ int sh_tile;
    VrCtl *ctl = D.ctl;
    const int t = threadIdx.x;
    const bool direct = S == 0;
    const long long cap = (D.K_host >= 0) ? D.K_host : D.E;  // entries of cnt and off
    uint32_t cd[VR_ITEMS];
    {
        const long long i0 = (long long)blockIdx.x * VR_TILE + (long long)t * VR_ITEMS;
#pragma unroll
        for (int m = 0; m < VR_ITEMS; m++) cd[m] = (direct && cap > 0) ? D.cnt[min(i0 + m, cap - 1)] : 0u;
    }
    const long long K = (long long)ctl->n_kept;
    const int ntiles = (int)((K + VR_TILE - 1) / VR_TILE);
    if (D.C == 1 && ntiles == 0 && blockIdx.x == 0 && t == 0)
        publish_counts(D.mailbox, D.seq, ctl->flags, ctl->n_cand, ctl->n_kept, 0ull);
    auto do_tile = [&](int tile, const uint32_t (&cin)[VR_ITEMS]) {
        const long long i0 = (long long)tile * VR_TILE + (long long)t * VR_ITEMS;
        uint32_t c[VR_ITEMS];
        unsigned long long loc = 0;
#pragma unroll
        for (int m = 0; m < VR_ITEMS; m++) {
            c[m] = (i0 + m < K) ? cin[m] : 0u;
            loc += c[m];
        }
        unsigned long long tot;
        const unsigned long long ex = block_excl_scan<unsigned long long>(loc, sh_w, &tot);
        if (t < VR_WAVE) {
            unsigned long long prefix = 0;
            if (tile == 0) {
                if (t == 0) st_store64(D.st_scan, st_pack64(VR_ST_INC, tot));
            } else {
                if (t == 0) st_store64(D.st_scan + tile, st_pack64(VR_ST_AGG, tot));
                prefix = lookback64_wave(D.st_scan, tile, [&](int i) {  // a whole tile's counts
                    const uint4 *c4 = (const uint4 *)(D.cnt + (size_t)i * VR_TILE);
                    unsigned long long v = 0;
#pragma unroll 2
                    for (int x = 0; x < VR_TILE / 4; x++) {
                        const uint4 u = c4[x];
                        v += (unsigned long long)u.x + u.y + u.z + u.w;
                    }
                    return v;
                });
                if (t == 0) st_store64(D.st_scan + tile, st_pack64(VR_ST_INC, prefix + tot));
            }
            if (t == 0) {
                sh_prefix = prefix;
                if (tile == ntiles - 1) {
                    ctl->n_tri = prefix + tot;
                    if (D.C == 1) publish_counts(D.mailbox, D.seq, ctl->flags, ctl->n_cand, ctl->n_kept, prefix + tot);
                }
            }
        }
        __syncthreads();
        unsigned long long o = sh_prefix + ex;
#pragma unroll
        for (int m = 0; m < VR_ITEMS; m++) {
            if (i0 + m < K) D.off[i0 + m] = o;
            o += c[m];
        }
    };
    // counts fewer than the launch provides for (a distance threshold keeps an
    // unknown part of the pairs): a tile per work-group, without the ticket
    // (1.1 million counts of 34 million pairs: 27 us with it, 17 without)
    if (direct || ntiles <= (int)gridDim.x) {
        if ((int)blockIdx.x >= ntiles) return;
        if (!direct) {
            const long long i0 = (long long)blockIdx.x * VR_TILE + (long long)t * VR_ITEMS;
#pragma unroll
            for (int m = 0; m < VR_ITEMS; m++) cd[m] = D.cnt[min(i0 + m, cap - 1)];
        }
        do_tile((int)blockIdx.x, cd);
        return;
    }
    for (;;) {
        const int t0 = claim_tiles(&ctl->ticket[5], S, &sh_tile);
        if (t0 >= ntiles) break;
        for (int tile = t0; tile < min(t0 + S, ntiles); tile++) {
            if (tile > t0) __syncthreads();  // sh_prefix and sh_w are reused
            const long long i0 = (long long)tile * VR_TILE + (long long)t * VR_ITEMS;
            uint32_t c[VR_ITEMS];
#pragma unroll
            for (int m = 0; m < VR_ITEMS; m++) c[m] = D.cnt[min(i0 + m, cap - 1)];
            do_tile(tile, c);
        }
    }
}

void launch_scan(const VrDev &D, long long Kmax, hipStream_t s) {
    long long g = (Kmax + VR_TILE - 1) / VR_TILE;
    // every tile gets its own work-group when there are few, else
    // 1024 work-groups claim one tile at a time
    const int S = (g <= 1024) ? 0 : 1;
    if (g > 1024) g = 1024;
    if (g < 1) g = 1;
    hipLaunchKernelGGL(k_scan, dim3((unsigned)g), dim3(VR_BLOCK), 0, s, D, S);
}

// ------------------------------------------------------ k_cloud_publish ----
// Batches: per cloud (kbase, K, first triangle, T) into host-pinned memory,
// then the counts into the mailbox from the last work-group to finish.
__global__ __launch_bounds__(VR_BLOCK) void k_cloud_publish(VrDev D) {
    __shared__ bool sh_last;
    const VrCtl *ctl = D.ctl;
    const int c = blockIdx.x * VR_BLOCK + threadIdx.x;
    if (c < D.C) {
        const long long kb = kept_base(D, c), K = kept_count(D, c);
        unsigned long long tb = 0, T = 0;
        if (D.tri && K > 0) {
            tb = D.off[kb];
            T = D.off[kb + K - 1] + D.cnt[kb + K - 1] - tb;
        } else if (D.tri) {
            tb = (kb < (long long)ctl->n_kept) ? D.off[kb] : ctl->n_tri;
        }
        unsigned long long *h = D.host_cloud + 4 * (size_t)c;
        __hip_atomic_store(&h[0], (unsigned long long)kb, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(&h[1], (unsigned long long)K, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(&h[2], tb, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(&h[3], T, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");
    __syncthreads();
    if (threadIdx.x == 0)
        sh_last = atomicAdd(&((VrCtl *)ctl)->done, 1u) == gridDim.x - 1;
    __syncthreads();
    if (sh_last && threadIdx.x == 0) {
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        publish_counts(D.mailbox, D.seq, ctl->flags, ctl->n_cand, ctl->n_kept, D.tri ? ctl->n_tri : 0ull);
    }
}

void launch_cloud_publish(const VrDev &D, hipStream_t s) {
    hipLaunchKernelGGL(k_cloud_publish, dim3((unsigned)((D.C + VR_BLOCK - 1) / VR_BLOCK)), dim3(VR_BLOCK), 0, s, D);
}

// ----------------------------------------------------------- k_tri_write ----
// Edge r = {a, b}: walk b's prefix list; entry (k, position pk in b's
// rank-ordered star) is a triangle of value r when pk < pb and Pa[k] < xa.
// The sorted vertex triple is (k, lo, hi), (lo, k, hi) or (lo, hi, k) as k
// falls below, between or above the endpoints.
//
// The hits' neighbours k of up to NP pieces are compacted in k order into
// the wave's own LDS (2 bytes each, ballot and mbcnt), then read back 64 at
// a time, made into keys and stored, the stores cut at 128-byte lines.  The
// candidates are a third to two thirds hits, so storing each piece's hits by
// themselves filled half the lanes of a key computation and of a store and
// touched most lines twice: the write was bound by its stores' requests (with
// the stores left out it took half the time).  Write, before -> after:
// 64-dimensional mixture, 4000 points, 94 million triangles 327 -> 264 us
// (2.9 TB/s of keys); 1088 x 1088 Hamming matrix, 214 million 703 -> 490 us
// (3.5 TB/s); torus, 8192 points, 62 million 317 -> 272 us; 32 clouds, 52
// million 310 -> 270 us.  Nontemporal stores beside plain ones: 264 and
// 342 us on the mixture, 490 and 527 us on the matrix.
__device__ __forceinline__ void emit_edges_range(const VrDev &D, long long K, uint32_t *__restrict__ ij,
                                                 long long *__restrict__ q, long long first, long long stride) {
    for (long long r = first; r < K; r += stride) {
        const uint32_t v = D.se_ij[r];
        __builtin_nontemporal_store(v >> 16, ij + 2 * r);
        __builtin_nontemporal_store(v & 0xFFFFu, ij + 2 * r + 1);
        __builtin_nontemporal_store((long long)D.se_q[r], q + r);
    }
}

#define VR_WGROUP 2  // pieces looked up together; 4 took 7% longer on a 1000-point circle, the same on the mixture
// a wave's staged candidates: 16 entries that lanes before the first hit
// read, NP pieces, 64 entries that lanes past the last hit read
#define VR_STAGE(NP) (16 + (NP) * VR_WAVE + VR_WAVE)
typedef uint32_t vr_u32x2 __attribute__((ext_vector_type(2)));

// Orders a wave's LDS stores before its later LDS loads of other lanes.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The triangles of up to 64 edges that vertex a (local index) writes, one
// edge's parameters per lane (lanes >= ne unused): global rank vr, start
// vsb and length vlen of the partner's prefix list in star_k, the edge's
// positions vxa in a's star and vpb in the partner's, the partner vb, and
// the edge's first output slot voff.  Pa = a's position table.  Each edge's
// list is walked in neighbour order, so its hits come out in k order.
template <int NP>
__device__ __forceinline__ void write_run(const VrDev &D, unsigned long long *__restrict__ out, uint32_t a,
                                          uint32_t kb, const uint16_t *Pa, int ne, uint32_t vr, uint32_t vsb,
                                          uint32_t vlen, uint32_t vxa, uint32_t vpb, uint32_t vb,
                                          unsigned long long voff, uint16_t *stage) {
    const int lane = threadIdx.x & 63;
    // per lane, so that an edge costs one register read each: its list's
    // address and bytes, its first slot's address, the bound its candidates'
    // positions pass, its endpoints in order, its rank in the key's high word
    const unsigned long long vat = (unsigned long long)(D.star_k + vsb), vdst = (unsigned long long)(out + voff);
    const uint32_t vlo = (uint32_t)vat, vhi = (uint32_t)(vat >> 32), vby = 4u * vlen;
    const uint32_t vdlo = (uint32_t)vdst, vdhi = (uint32_t)(vdst >> 32);
    const uint32_t vlim = plist_bound(vpb), vmin = min(a, vb), vmax = max(a, vb), vrh = (vr - kb) << 7;
    auto list_of = [&](int el) { return list_buffer(rl(vlo, el), rl(vhi, el), rl(vby, el)); };
    uint32_t run = 0;        // staged candidates
    uint32_t dlo = 0, dhi = 0;  // address of the current edge's next slot
    // write the staged hits' keys, a whole wave at a time and cut at
    // 128-byte lines of the output; the bounded buffer drops the lanes
    // before the first and past the last
    auto flush = [&](int el) {
        const uint32_t lo = rl(vmin, el), hi = rl(vmax, el), rh = rl(vrh, el);
        wave_lds_sync();
        const __amdgpu_buffer_rsrc_t dst = list_buffer(dlo, dhi, run * 8u);
        const uint32_t shift = (dlo >> 3) & 15u;
        for (uint32_t t = 0; run > 0 && t < run + shift; t += VR_WAVE) {
            // key = (r << 39) | (x0 << 26) | (x1 << 13) | x2 with x0 < x1 < x2
            // the sorted triple {lo, hi, k}; k differs from both endpoints
            const int i = lane + (int)(t - shift);
            const uint32_t k = stage[i];
            const uint32_t x0 = min(lo, k), x2 = max(hi, k), x1 = min(max(k, lo), hi);
            const vr_u32x2 key = {(x0 << 26) | ((x1 << 13) | x2), rh | (x0 >> 6)};
            // streaming store (2: nontemporal): keeps the lists, not the output, in L2
            __builtin_amdgcn_raw_buffer_store_b64(key, dst, i * 8, 0, 2);
        }
        wave_lds_sync();
    };
    // stage the hits of edge el from its prefetched pieces
    auto stage_edge = [&](int el, const uint32_t (&kk)[NP]) {
        const uint32_t xa = rl(vxa, el), lim = rl(vlim, el), by = rl(vby, el);
        dlo = rl(vdlo, el);
        dhi = rl(vdhi, el);
        run = 0;
        // one 64-entry piece of the partner's prefix list, with the position
        // of each entry's neighbour in a's star: the hits' neighbours are
        // staged, in order
        auto piece = [&](uint32_t v, uint32_t pa) {
            // lane masks of the two tests straight from the comparisons
            // (unsigned greater-than is predicate 34, less-than 36)
            const unsigned long long m = __builtin_amdgcn_uicmp(v, lim, 34) & __builtin_amdgcn_uicmp(pa, xa, 36);
            const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
            if ((v > lim) & (pa < xa)) (stage + run)[at] = (uint16_t)v;
            run += (uint32_t)__popcll(m);
        };
        // pieces in groups of VR_WGROUP: a group past the end is skipped
        // whole, and the position lookups of a group are issued together
#pragma unroll
        for (int g = 0; g < NP; g += VR_WGROUP) {
            if ((uint32_t)(g * VR_WAVE * 4) < by) {
                uint32_t pa[VR_WGROUP];
#pragma unroll
                for (int j = 0; j < VR_WGROUP; j++) pa[j] = Pa[kk[g + j] & 0xFFFFu];
#pragma unroll
                for (int j = 0; j < VR_WGROUP; j++) piece(kk[g + j], pa[j]);
            }
        }
        for (uint32_t y0 = NP * VR_WAVE * 4; y0 < by; y0 += 4 * VR_WAVE * 4) {
            uint32_t v[4], pa[4];
#pragma unroll
            for (int j = 0; j < 4; j++)
                v[j] = __builtin_amdgcn_raw_buffer_load_b32(list_of(el), 4 * lane + j * VR_WAVE * 4, (int)y0, 0);
            if (run > (NP - 4) * VR_WAVE) {  // make room for four pieces
                flush(el);
                const unsigned long long d = (((unsigned long long)dhi << 32) | dlo) + run * 8u;
                dlo = (uint32_t)d;
                dhi = (uint32_t)(d >> 32);
                run = 0;
            }
#pragma unroll
            for (int j = 0; j < 4; j++) pa[j] = Pa[v[j] & 0xFFFFu];
#pragma unroll
            for (int j = 0; j < 4; j++) piece(v[j], pa[j]);
        }
    };
    // ping-pong prefetch one edge ahead; past the last edge the loads
    // repeat the last edge's (never consumed).  An edge's buffer is refilled
    // between staging and writing: memory operations complete in order, so
    // waiting for loads issued after the stores would wait for the stores.
    uint32_t kA[NP], kB[NP];
    issue_list(list_of(0), kA);
    issue_list(list_of(min(1, ne - 1)), kB);
    for (int el = 0; el < ne; el += 2) {
        stage_edge(el, kA);
        issue_list(list_of(min(el + 2, ne - 1)), kA);
        flush(el);
        if (el + 1 < ne) {
            stage_edge(el + 1, kB);
            issue_list(list_of(min(el + 3, ne - 1)), kB);
            flush(el + 1);
        }
    }
}

// Blocks [0, n*parts) write triangles; the blocks after them write the
// public edge arrays.
template <int EB, int NP>
__global__ __launch_bounds__(EB) void k_tri_write(VrDev D, unsigned long long *__restrict__ out, int parts,
                                                          long long cap_k, unsigned long long cap_t,
                                                          uint32_t *__restrict__ edge_ij,
                                                          long long *__restrict__ edge_q) {
    extern __shared__ uint32_t lds[];
    // outputs sized before the counts were known: write nothing unless they fit
    const long long K = (long long)D.ctl->n_kept;
    if (K > cap_k || D.ctl->n_tri > cap_t) return;
    const long long nb = D.V * parts;
    if ((long long)blockIdx.x >= nb) {
        emit_edges_range(D, K, edge_ij, edge_q, (long long)(blockIdx.x - nb) * EB + threadIdx.x,
                         (long long)(gridDim.x - nb) * EB);
        return;
    }
    const long long ag = blockIdx.x / parts;
    const int part = blockIdx.x % parts;
    const int c = vertex_cloud(D, ag);
    const uint32_t vb = (uint32_t)D.cl[c].vbase;
    const uint32_t kb = (uint32_t)kept_base(D, c);  // the cloud's ranks start here
    const int a = (int)(ag - vb), n = D.cl[c].n;
    uint16_t *Pa = (uint16_t *)lds;
    EnumLds<EB> &L = *(EnumLds<EB> *)((char *)lds + 2 * ((D.maxn + 7) & ~7));
    uint16_t *stage = (uint16_t *)(&L + 1) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * VR_STAGE(NP) + 16;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t mb = (uint32_t)D.cl[c].mbase;
    const uint32_t s0 = star_slot(mb, n, a), s1 = s0 + D.deg[ag];
    uint32_t r0, b0;
    stage_pos<EB>(D, n, Pa, s0, s1, r0, b0);
    for (uint32_t p0 = s0; p0 < s1; p0 += EB) {
        load_chunk<true, EB>(D, a, vb, mb, n, kb, s0, s1, p0, L, part, parts, r0, b0);
        const int w_lo = __builtin_amdgcn_readfirstlane((int)L.ew[w]);
        const int w_hi = __builtin_amdgcn_readfirstlane((int)L.ew[w + 1]);
        for (int eb = w_lo; eb < w_hi; eb += VR_WAVE) {
            const int ne = min(VR_WAVE, w_hi - eb);
            uint32_t vr = 0, vsb = 0, vlen = 0, vxa = 0, vpb = 0, vb = 0;
            unsigned long long voff = 0;
            if (lane < ne) {
                vr = L.r[eb + lane];
                vsb = L.sb[eb + lane];
                vlen = L.len[eb + lane];
                vxa = L.xa[eb + lane];
                vpb = L.pb[eb + lane];
                vb = L.b[eb + lane];
                voff = D.off[vr];
            }
            write_run<NP>(D, out, (uint32_t)a, kb, Pa, ne, vr, vsb, vlen, vxa, vpb, vb, voff, stage);
        }
        __syncthreads();
    }
}

// LDS of one wave of k_tri_write_x: a's position table (maxn entries,
// rounded up to 8) and a ring of 128 staged edges.
#define VR_XRING 128
__host__ __device__ __forceinline__ uint32_t xwave_lds(int maxn, int np) {
    return 2u * (((uint32_t)maxn + 7u) & ~7u) + VR_XRING * (uint32_t)sizeof(uint4) + 2u * VR_STAGE((uint32_t)np);
}

// The write with 0 work-groups per vertex: one wave per (vertex a, eighth
// of its cloud's vertices), taking the edges a writes (write_side) whose
// partner lies in that eighth.  Work-group g holds the waves of vertices
// [W (g / 8), W (g / 8) + W) for eighth g mod 8.  Work-groups go to the
// chip's 8 dies (XCDs, each with its own L2) in turn, so block index mod 8
// names the die: each die reads the prefix lists of one eighth of the
// vertices, about an eighth of them all, which its L2 can hold.  Each wave
// runs on its own, with a's position table and a ring of staged edges in
// the wave's own LDS and no work-group barrier: the table is filled from
// a's rank-ordered star while counting a's neighbours below the eighth's
// bounds, which locates a's edges to the eighth as one run of its
// neighbour-ordered star; those a writes are staged in the ring and
// written 64 at a time (write_run).  Blocks past the vertices' write the
// public edge arrays.
template <int EB, int NP>
__global__ __launch_bounds__(EB) void k_tri_write_x(VrDev D, unsigned long long *__restrict__ out, long long cap_k,
                                                    unsigned long long cap_t, uint32_t *__restrict__ edge_ij,
                                                    long long *__restrict__ edge_q) {
    constexpr int W = EB / VR_WAVE;
    extern __shared__ uint32_t lds[];
    const long long K = (long long)D.ctl->n_kept;
    if (K > cap_k || D.ctl->n_tri > cap_t) return;
    const long long nb = (D.V + W - 1) / W * 8;
    if ((long long)blockIdx.x >= nb) {
        emit_edges_range(D, K, edge_ij, edge_q, (long long)(blockIdx.x - nb) * EB + threadIdx.x,
                         (long long)(gridDim.x - nb) * EB);
        return;
    }
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t x8 = blockIdx.x & 7u;
    const long long ag = (long long)(blockIdx.x >> 3) * W + w;
    if (ag >= D.V) return;  // the whole wave: nothing below waits on other waves
    const uint32_t deg = D.deg[ag];
    if (deg == 0) return;
    const int c = vertex_cloud(D, ag);
    const uint32_t vb = (uint32_t)D.cl[c].vbase;
    const uint32_t kb = (uint32_t)kept_base(D, c);
    const int n = D.cl[c].n;
    const uint32_t a = (uint32_t)(ag - vb);
    const uint32_t mb = (uint32_t)D.cl[c].mbase;
    const uint32_t pa_n = ((uint32_t)D.maxn + 7u) & ~7u;
    uint16_t *Pa = (uint16_t *)((char *)lds + (size_t)w * xwave_lds(D.maxn, NP));
    uint4 *ring = (uint4 *)(Pa + pa_n);
    uint16_t *stage = (uint16_t *)(ring + VR_XRING) + 16;
    const uint32_t s0 = star_slot(mb, n, (int)a), s1 = s0 + deg;
    // partners b with (8 b) / n == x8
    const uint32_t blo = (x8 * (uint32_t)n + 7u) / 8u, bhi = ((x8 + 1u) * (uint32_t)n + 7u) / 8u;
    for (uint32_t i = (uint32_t)lane; i < pa_n / 8u; i += VR_WAVE) ((uint4 *)Pa)[i] = make_uint4(~0u, ~0u, ~0u, ~0u);
    wave_lds_sync();
    // position table; y0, y1 = a's neighbours below blo, below bhi
    uint32_t y0 = 0, y1 = 0;
    for (uint32_t base = s0; base < s1; base += 4 * VR_WAVE) {
        uint32_t k[4];
#pragma unroll
        for (int j = 0; j < 4; j++) k[j] = D.star_nbr[min(base + (uint32_t)(j * VR_WAVE + lane), s1 - 1u)];
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const uint32_t p = base + (uint32_t)(j * VR_WAVE + lane);
            const bool in = p < s1;
            if (in) Pa[k[j]] = (uint16_t)(p - s0);
            y0 += (uint32_t)__popcll(ballot64(in && k[j] < blo));
            y1 += (uint32_t)__popcll(ballot64(in && k[j] < bhi));
        }
    }
    wave_lds_sync();
    // a's neighbour-ordered star (the last prefix list): entries [y0, y1)
    // are its edges to the eighth
    const uint32_t *sk = D.star_k + plist_region(mb, vb, n, (int)a) + plist_off(VR_PLISTS, deg);
    uint32_t head = 0, cnt = 0;  // staged edges: ring slots [head, head + cnt)
    auto flush = [&](int ne) {
        uint32_t vr = 0, vsb = 0, vlen = 0, vxa = 0, vpb = 0, vbp = 0;
        unsigned long long voff = 0;
        if (lane < ne) {
            const uint4 e = ring[(head + (uint32_t)lane) & (VR_XRING - 1)];
            vr = e.x;
            vsb = e.y;
            vbp = e.z & 0xFFFFu;
            vxa = e.z >> 16;
            vpb = e.w & 0xFFFFu;
            vlen = e.w >> 16;
            voff = D.off[vr];
        }
        write_run<NP>(D, out, a, kb, Pa, ne, vr, vsb, vlen, vxa, vpb, vbp, voff, stage);
    };
    for (uint32_t y = y0; y < y1; y += VR_WAVE) {
        const uint32_t yy = y + (uint32_t)lane;
        const bool in = yy < y1;
        const uint32_t e = sk[in ? yy : y1 - 1u];
        const uint32_t b = e & 0xFFFFu, xa = 0xFFFFu - (e >> 16);
        const uint32_t r = kb + D.star_r[s0 + xa];
        const uint32_t pb = D.ppos[s0 + xa];
        uint32_t len = 0, sb = 0;
        const bool mine = write_side(D, a, b, xa, deg, pb, vb, mb, n, len, sb);
        const bool own = in && mine && len > 0;  // len 0: the edge has no triangles
        const unsigned long long m = ballot64(own);
        if (own) {
            const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            ring[(head + cnt + at) & (VR_XRING - 1)] = make_uint4(r, sb, b | (xa << 16), pb | (len << 16));
        }
        cnt += (uint32_t)__popcll(m);
        if (cnt >= VR_WAVE) {  // cnt < 128: the ring never overflows
            wave_lds_sync();
            flush(VR_WAVE);
            head = (head + VR_WAVE) & (VR_XRING - 1);
            cnt -= VR_WAVE;
            wave_lds_sync();
        }
    }
    if (cnt > 0) {
        wave_lds_sync();
        flush((int)cnt);
    }
}

// The outputs hold cap_k edges and cap_t triangles; the kernel writes nothing
// when the build's counts (read on the device) exceed them.  With events,
// they take the dispatch's own start and end times (no separate markers).
void launch_tri_write(const VrDev &D, unsigned long long *tri_out, long long cap_k, unsigned long long cap_t,
                      uint32_t *edge_ij, long long *edge_q, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    const int parts = D.parts_write;
    int EB = D.eb_write;
    // one wave per (vertex, eighth): fewer waves per work-group while their
    // LDS would pass 64 KiB
    if (parts == 0)
        while (EB > 128 && (size_t)(EB / VR_WAVE) * xwave_lds(D.maxn, D.pieces_write == 4 ? 4 : 8) > 65536) EB /= 2;
    const long long K = cap_k;
    long long eb = (K + EB - 1) / EB;  // extra work-groups that write the edge arrays
    if (eb > 256) eb = 256;
    if (eb < 1) eb = 1;
    const long long W = EB / VR_WAVE;
    const dim3 grid((unsigned)((parts == 0 ? (D.V + W - 1) / W * 8 : D.V * parts) + eb));
    auto go = [&](auto eb_c, auto np_c) {
        constexpr int E = decltype(eb_c)::value, N = decltype(np_c)::value;
        if (parts == 0) {
            const size_t lb = (size_t)(E / VR_WAVE) * xwave_lds(D.maxn, N);
            if (ev0 && ev1)
                hipExtLaunchKernelGGL((k_tri_write_x<E, N>), grid, dim3(E), lb, s, ev0, ev1, 0u, D, tri_out, cap_k,
                                      cap_t, edge_ij, edge_q);
            else
                hipLaunchKernelGGL((k_tri_write_x<E, N>), grid, dim3(E), lb, s, D, tri_out, cap_k, cap_t, edge_ij,
                                   edge_q);
            return;
        }
        const size_t lb = enum_lds<E>(D.maxn) + 2 * (size_t)(E / VR_WAVE) * VR_STAGE(N);
        if (ev0 && ev1)
            hipExtLaunchKernelGGL((k_tri_write<E, N>), grid, dim3(E), lb, s, ev0, ev1, 0u, D, tri_out,
                                  parts, cap_k, cap_t, edge_ij, edge_q);
        else
            hipLaunchKernelGGL((k_tri_write<E, N>), grid, dim3(E), lb, s, D, tri_out, parts, cap_k,
                               cap_t, edge_ij, edge_q);
    };
    using I128 = std::integral_constant<int, 128>;
    using I256 = std::integral_constant<int, 256>;
    using I512 = std::integral_constant<int, 512>;
    using P4 = std::integral_constant<int, 4>;
    using P8 = std::integral_constant<int, 8>;
    const bool p4 = D.pieces_write == 4;
    if (EB == 128) p4 ? go(I128{}, P4{}) : go(I128{}, P8{});
    else if (EB == 256) p4 ? go(I256{}, P4{}) : go(I256{}, P8{});
    else p4 ? go(I512{}, P4{}) : go(I512{}, P8{});
}

// ---------------------------------------------------------- k_emit_edges ----
__global__ __launch_bounds__(VR_BLOCK) void k_emit_edges(VrDev D, long long K, uint32_t *__restrict__ ij,
                                                         long long *__restrict__ q) {
    for (long long r = (long long)blockIdx.x * VR_BLOCK + threadIdx.x; r < K; r += (long long)gridDim.x * VR_BLOCK) {
        const uint32_t v = D.se_ij[r];
        ij[2 * r] = v >> 16;
        ij[2 * r + 1] = v & 0xFFFFu;
        q[r] = (long long)D.se_q[r];
    }
}

void launch_emit_edges(const VrDev &D, long long K, uint32_t *edge_ij, long long *edge_q, hipStream_t s) {
    long long g = (K + VR_BLOCK - 1) / VR_BLOCK;
    if (g > 2048) g = 2048;
    if (g < 1) g = 1;
    hipLaunchKernelGGL(k_emit_edges, dim3((unsigned)g), dim3(VR_BLOCK), 0, s, D, K, edge_ij, edge_q);
}

// ----------------------------------------------------------- k_unpack ----
// Packed triangle keys -> rows (i, j, k, v) of int32, for callers that want
// the filtration's triangles unpacked.
__global__ __launch_bounds__(VR_BLOCK) void k_unpack(const unsigned long long *__restrict__ keys, long long T,
                                                     int4 *__restrict__ rows) {
    for (long long x = (long long)blockIdx.x * VR_BLOCK + threadIdx.x; x < T; x += (long long)gridDim.x * VR_BLOCK) {
        const unsigned long long k = keys[x];
        rows[x] = make_int4((int)((k >> 26) & 0x1FFFu), (int)((k >> 13) & 0x1FFFu), (int)(k & 0x1FFFu),
                            (int)(k >> 39));
    }
}

void launch_unpack(const unsigned long long *keys, long long T, int *rows, hipStream_t s) {
    long long g = (T + VR_BLOCK - 1) / VR_BLOCK;
    if (g > 4096) g = 4096;
    if (g < 1) g = 1;
    hipLaunchKernelGGL(k_unpack, dim3((unsigned)g), dim3(VR_BLOCK), 0, s, keys, T, (int4 *)rows);
}
