// k_colsort.hip -- per-column stable ordering of a compressed-sparse-column
// array (Section 4.3: the slot every entry takes when its column is sorted by
// value, equal values keeping their order).
//
// The entries are cut into windows of CO_WIN consecutive entries, whatever
// the columns.  A window's entries fall into segments, one per column that
// meets the window.
//   k_co_first  per column: the windows whose first entry lies in it.
//   k_co_local  per window: each entry's rank inside its segment (counting
//               against the segment in LDS when every segment is short,
//               otherwise buckets of values, or an LDS bitonic sort where
//               the values crowd), plus the column's first slot;
//               the sorted values of segments whose column leaves the window
//               are kept for the next kernel.
//   k_co_merge  per window, only for the (at most two) columns that leave
//               it: adds, for every other window the column meets, the
//               entries there that come first (binary search in that
//               window's sorted run: values <= x before, < x after).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>
#include <type_traits>

#include "vr.h"
#include "vr_cache.h"

#define CO_BLOCK 256
#define CO_WIN 4096
#define CO_PER (CO_WIN / CO_BLOCK)
#define CO_COUNT 24       // longest segment ranked by counting
#define CO_COUNT_MAX 256  // the same in a window of more than CO_SEGS segments
#define CO_WAVE 64
#define CO_SEGS 256  // segments of a window that is sorted into buckets
#define CO_CROWD 24  // longest bucket
#define CO_COPIES 16  // of a segment's smallest and largest value

static_assert(2 * (CO_SEGS + 8) + 4 * CO_SEGS + 16 * CO_SEGS <= 2 * (CO_WIN + 2), "the segments' values fit behind their starts");
static_assert(8 * CO_COPIES * CO_SEGS <= 8 * (CO_WIN + CO_WIN / 16), "the copies fit over the keys");

static __device__ __forceinline__ int64_t clampi(int64_t x, int64_t lo, int64_t hi) {
    return x < lo ? lo : (x > hi ? hi : x);
}

// first[w] = the column holding entry w*CO_WIN (the non-empty column c with
// colptr[c] <= w*CO_WIN < colptr[c+1]).
__global__ void __launch_bounds__(CO_BLOCK) k_co_first(const int64_t *colptr, int64_t ncols, int64_t nnz,
                                                      int64_t *first) {
    for (int64_t c = blockIdx.x * (int64_t)CO_BLOCK + threadIdx.x; c < ncols;
         c += (int64_t)gridDim.x * CO_BLOCK) {
        const int64_t s = clampi(colptr[c], 0, nnz), e = clampi(colptr[c + 1], s, nnz);
        if (e == s) continue;
        for (int64_t w = (s + CO_WIN - 1) / CO_WIN; w <= (e - 1) / CO_WIN; w++) first[w] = c;
    }
}

struct CoWindow {
    int64_t a;    // first entry
    int cnt;      // entries
    int64_t c0;   // column of the first entry
    int64_t cs0;  // first slot of that column
    int64_t cl;   // column of entry a + CO_WIN (next window), or -1
};

static __device__ __forceinline__ CoWindow co_window(const int64_t *colptr, int64_t ncols, int64_t nnz,
                                                     const int64_t *first, int64_t nwin, int64_t w) {
    CoWindow W;
    W.a = w * CO_WIN;
    W.cnt = (int)min((int64_t)CO_WIN, nnz - W.a);
    W.c0 = clampi(first[w], 0, ncols - 1);
    W.cs0 = clampi(colptr[W.c0], 0, W.a);
    W.cl = w + 1 < nwin ? clampi(first[w + 1], W.c0, ncols - 1) : -1;
    return W;
}

// LDS index of key position p: one pad slot per 16 keys, so that the lanes
// of layout C (16 keys apart) spread over the banks
static __device__ __forceinline__ int co_phys(int p) { return p + (p >> 4); }

// position of register g of thread t in layout LAY (0: C, 1: S, 2: L)
template <int LAY>
static __device__ __forceinline__ int co_pos(int t, int g) {
    return LAY == 0 ? CO_PER * t + g : (LAY == 1 ? 256 * (t >> 4) + 16 * g + (t & 15) : 256 * g + t);
}

template <int LAY, typename KEY>
static __device__ __forceinline__ void co_put(const KEY (&r)[CO_PER], int t, KEY *keys) {
#pragma unroll
    for (int g = 0; g < CO_PER; g++) keys[co_phys(co_pos<LAY>(t, g))] = r[g];
}

// move the keys from layout cur to layout TO through LDS.  C and S hold the
// same 1024 positions in a wave, which then waits for itself alone (12 of the
// sort's 21 moves).
template <int TO, typename KEY>
static __device__ __forceinline__ void co_to(KEY (&r)[CO_PER], int &cur, int t, KEY *keys) {
    if (cur == TO) return;  // uniform over the work-group
    const bool wave = cur != 2 && TO != 2;
    auto sync = [&] {
        if (wave) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        } else {
            __syncthreads();
        }
    };
    sync();  // earlier reads of the buffer are done
    if (cur == 0) co_put<0>(r, t, keys);
    else if (cur == 1) co_put<1>(r, t, keys);
    else co_put<2>(r, t, keys);
    sync();
#pragma unroll
    for (int g = 0; g < CO_PER; g++) r[g] = keys[co_phys(co_pos<TO>(t, g))];
    cur = TO;
}

// Smaller and larger of two keys.  64-bit ones compare as doubles: a set bit
// CO_KEY64 makes them normal numbers, ordered as the integers are, and one
// instruction each takes the place of a comparison and four selects.
#define CO_KEY64 (1ull << 62)
#define CO_PAD64 0x7FEFFFFFFFFFFFFFull  // the largest finite one: pads sort last
static __device__ __forceinline__ void co_exchange(uint32_t &x, uint32_t &y) {
    const uint32_t lo = min(x, y), hi = max(x, y);
    x = lo;
    y = hi;
}
static __device__ __forceinline__ void co_exchange(unsigned long long &x, unsigned long long &y) {
    const double u = __longlong_as_double((long long)x), v = __longlong_as_double((long long)y);
    double lo, hi;
    asm("v_min_f64 %0, %1, %2" : "=v"(lo) : "v"(u), "v"(v));
    asm("v_max_f64 %0, %1, %2" : "=v"(hi) : "v"(u), "v"(v));
    x = (unsigned long long)__double_as_longlong(lo);
    y = (unsigned long long)__double_as_longlong(hi);
}
// The key in the opposite order, and back: all bits, or the sign.
static __device__ __forceinline__ void co_flip(uint32_t &x, bool on) { x ^= on ? ~0u : 0u; }
static __device__ __forceinline__ void co_flip(unsigned long long &x, bool on) { x ^= on ? 1ull << 63 : 0ull; }

// the stages of one merge width on the position bits that layout LAY
// holds in registers (bits 4*LAY .. 4*LAY+3, at most bhi), highest first
template <int LAY, typename KEY>
static __device__ __forceinline__ void co_stages(KEY (&r)[CO_PER], int bhi) {
#pragma unroll
    for (int gb = 3; gb >= 0; gb--) {
        if (4 * LAY + gb > bhi) continue;
#pragma unroll
        for (int g = 0; g < CO_PER; g++)
            if (!(g & (1 << gb))) co_exchange(r[g], r[g | (1 << gb)]);
    }
}

// Bitonic sort of CO_WIN keys, a thread's 16 in layout L at first and in
// layout C at the end.  Every compare-exchange happens in registers: a
// thread holds 16 keys in one of three layouts, each owning four bits of the
// position (C: bits 0-3, position 16t + g; S: bits 4-7, 256(t/16) + 16g +
// t%16; L: bits 8-11, 256g + t), and the keys move between layouts through
// LDS.  The blocks that a merge sorts downwards hold their keys flipped, so
// that every exchange goes the same way; that is one instruction a key and merge.
template <typename KEY>
static __device__ __forceinline__ void co_bitonic(KEY (&r)[CO_PER], int t, KEY *keys) {
    int cur = 2;
    for (int lk = 1; lk <= 12; lk++) {  // merge width 2^lk: stages on bits lk-1 .. 0
        if (lk == 1) co_to<0>(r, cur, t, keys);
#pragma unroll
        for (int g = 0; g < CO_PER; g++) {  // downwards where bit lk of the position is set
            const int p = co_pos<0>(t, g);
            co_flip(r[g], ((p >> lk) ^ (lk > 1 ? p >> (lk - 1) : 0)) & 1);
        }
        if (lk - 1 >= 8) {
            co_to<2>(r, cur, t, keys);
            co_stages<2>(r, lk - 1);
        }
        if (lk - 1 >= 4) {
            co_to<1>(r, cur, t, keys);
            co_stages<1>(r, lk - 1);
        }
        co_to<0>(r, cur, t, keys);
        co_stages<0>(r, lk - 1);
    }
}

__global__ void __launch_bounds__(CO_BLOCK) k_co_local(const int64_t *colptr, int64_t ncols, const int32_t *v,
                                                      int64_t nnz, const int64_t *first, int64_t nwin, int64_t *z,
                                                      uint32_t *vs) {
    // keys: counting path, the values with the sign bit flipped (unsigned
    // order); sorting path, the keys between layouts, then the slots
    __shared__ __align__(16) unsigned long long keys[CO_WIN + CO_WIN / 16];
    uint32_t *kv = (uint32_t *)keys;
    __shared__ __align__(16) uint16_t segid[CO_WIN];  // first the segment-start flags; at last the buckets' starts
    __shared__ __align__(16) uint16_t segstart[CO_WIN + 2];
    __shared__ uint32_t wsum[CO_BLOCK / CO_WAVE];
    __shared__ uint32_t maxlen, few, longest, vbits;
    // of at most CO_SEGS segments, behind their starts
    uint32_t *smin = (uint32_t *)(segstart + CO_SEGS + 8);
    uint4 *seg = (uint4 *)(smin + CO_SEGS);  // least value, buckets per value (float), first bucket, last bucket's index

    const int t = threadIdx.x, lane = t % CO_WAVE, wv = t / CO_WAVE;
    const CoWindow W = co_window(colptr, ncols, nnz, first, nwin, blockIdx.x);
    const int cnt = W.cnt;
    const int64_t a = W.a;

    // values (clamped loads past the end, never stored) and cleared flags
    int32_t x[CO_PER];
#pragma unroll
    for (int m = 0; m < CO_PER; m++) x[m] = v[a + min(t + m * CO_BLOCK, cnt - 1)];
#pragma unroll
    for (int m = 0; m < CO_PER; m++) {
        kv[t + m * CO_BLOCK] = (uint32_t)x[m] ^ 0x80000000u;
        segid[t + m * CO_BLOCK] = 0;
    }
    if (t == 0) maxlen = few = longest = vbits = 0;
    __syncthreads();
    // segment starts: every column that begins strictly inside the window
    const int64_t cend = W.cl >= 0 ? W.cl : ncols - 1;
    for (int64_t c = W.c0 + 1 + t; c <= cend; c += CO_BLOCK) {
        const int64_t p = colptr[c] - a;
        if (p > 0 && p < cnt) segid[p] = 1;
    }
    __syncthreads();
    // segment of every position: inclusive count of the starts up to it
    // (thread t scans positions CO_PER*t .. CO_PER*t + CO_PER-1)
    // wide LDS accesses: 2-byte ones 32 bytes apart would meet in one bank in eight
    uint4 *f4 = (uint4 *)segid + 2 * t;
    uint32_t f[CO_PER / 2], own = 0;
    {
        const uint4 f0 = f4[0], f1 = f4[1];
        f[0] = f0.x, f[1] = f0.y, f[2] = f0.z, f[3] = f0.w, f[4] = f1.x, f[5] = f1.y, f[6] = f1.z, f[7] = f1.w;
    }
#pragma unroll
    for (int m = 0; m < CO_PER / 2; m++) own += f[m];
    own = (own & 0xFFFFu) + (own >> 16);
    uint32_t incl = own;
#pragma unroll
    for (int d = 1; d < CO_WAVE; d <<= 1) {
        const uint32_t y = __shfl_up(incl, d, CO_WAVE);
        if (lane >= d) incl += y;
    }
    if (lane == CO_WAVE - 1) wsum[wv] = incl;
    __syncthreads();
    uint32_t run = incl - own, total = 0;
#pragma unroll
    for (int i = 0; i < CO_BLOCK / CO_WAVE; i++) {
        if (i < wv) run += wsum[i];
        total += wsum[i];
    }
#pragma unroll
    for (int m = 0; m < CO_PER / 2; m++) {
        const uint32_t r0 = run + (f[m] & 1u), r1 = r0 + (f[m] >> 16);
        if (f[m] & 1u) segstart[r0] = (uint16_t)(CO_PER * t + 2 * m);
        if (f[m] >> 16) segstart[r1] = (uint16_t)(CO_PER * t + 2 * m + 1);
        f[m] = r0 | (r1 << 16);
        run = r1;
    }
    f4[0] = make_uint4(f[0], f[1], f[2], f[3]);
    f4[1] = make_uint4(f[4], f[5], f[6], f[7]);
    const int nseg = (int)total + 1;
    if (t == 0) {
        segstart[0] = 0;
        segstart[nseg] = (uint16_t)cnt;
    }
    __syncthreads();
    for (int s = t; s < nseg; s += CO_BLOCK) atomicMax(&maxlen, (uint32_t)(segstart[s + 1] - segstart[s]));
    __syncthreads();

    // the first segment leaves the window on the left if its column began
    // earlier, the last on the right if the next window's first column
    // began in this one
    const bool spans_l = W.cs0 < a;
    const bool spans_r = W.cl >= 0 && colptr[W.cl] < a + cnt;
    auto base_of = [&](int s) -> int64_t { return s == 0 ? W.cs0 : a + segstart[s]; };
    auto spans = [&](int s) -> bool { return (s == 0 && spans_l) || (s == nseg - 1 && spans_r); };

    // Counting takes a pass over its segment for every entry.  A thousand
    // columns of 20, 32, 48, 64, 100 and 200 entries: counted one read at a
    // time 25, 47, 68, 77, 116 and 209 us a call, eight reads at a time 23,
    // 36, 49, 52, 79 and 131, in buckets 26, 32, 35, 32, 36 and 35.
    if (maxlen <= (nseg <= CO_SEGS ? CO_COUNT : CO_COUNT_MAX)) {
        // rank = entries of the segment with a smaller value or an equal
        // value earlier; lanes of a wave mostly share a segment, so LDS
        // broadcasts the compared values
#pragma unroll 1
        for (int m = 0; m < CO_PER; m++) {
            const int p = t + m * CO_BLOCK;
            if (p >= cnt) break;
            const uint32_t xv = kv[p];
            const int s = segid[p], st = segstart[s], en = segstart[s + 1];
            uint32_t r = 0;
            for (int q = st; q < en; q += 8) {  // eight reads in flight
                uint32_t u[8];
#pragma unroll
                for (int i = 0; i < 8; i++) u[i] = kv[min(q + i, en - 1)];
#pragma unroll
                for (int i = 0; i < 8; i++)
                    r += (uint32_t)(q + i < en) &
                         ((uint32_t)(u[i] < xv) | ((uint32_t)(u[i] == xv) & (uint32_t)(q + i < p)));
            }
            z[a + p] = base_of(s) + r;
            if (spans(s)) vs[a + st + r] = xv;
        }
        return;
    }

    // z of the thread's keys (segment << 44 | value << 12 | position), key g
    // in sorted position CO_PER * t + g
    auto finish = [&](const unsigned long long (&r)[CO_PER]) {
        __syncthreads();  // every thread's last read of the keys is done
#pragma unroll
        for (int g = 0; g < CO_PER; g++) {
            if (CO_PER * t + g < cnt) {
                const int y = CO_PER * t + g, sg = (int)(r[g] >> 44), idx = (int)(r[g] & 0xFFFu);
                keys[co_phys(idx)] = (unsigned long long)(base_of(sg) + (y - segstart[sg]));
                if (spans(sg)) vs[a + y] = (uint32_t)(r[g] >> 12);
            }
        }
        __syncthreads();
#pragma unroll
        for (int m = 0; m < CO_PER; m++) {
            const int p = t + m * CO_BLOCK;
            if (p < cnt) z[a + p] = (int64_t)keys[co_phys(p)];
        }
    };

    // Buckets: a segment of len entries takes len buckets, its values spread
    // over them in order (float products, which round monotonically), so an
    // entry shares its bucket with few others and its place is the bucket's
    // start plus the smaller (value, position) there.  2000 columns of 1999
    // entries, us of this kernel: sorted by 64-bit keys 68, in buckets 36, half
    // the time in waits for LDS: 225 registers leave two work-groups a compute
    // unit (bounded to 168, for a third, 53 of them spilled: 53 us).
    // Where values crowd (24 or more in a bucket) the window is sorted after
    // all, by 32-bit keys if they hold segment, value and position.  It must
    // not lose there what it had before the buckets; us of whole calls, always sorted / with
    // buckets tried first and the sort as it was / now:
    //                      2000 columns of 1999   4000 of 300
    //   uniform                100 /  69 /  66     54 / 44 / 34
    //   10 values               99 /  93 /  82     54 / 57 / 43
    //   twelfth powers         100 / 128 /  97     55 / 75 / 49
    //   lognormal, sigma 4      99 / 136 /  98     54 / 78 / 50
    // The extremes took as long as the sort's half where a window has a dozen
    // segments (CO_COPIES), crowds are seen in a quarter of the entries, and the
    // sort's exchanges and moves cost less (co_exchange, co_to).
    if (nseg <= CO_SEGS) {
        uint32_t *cw = (uint32_t *)segid;
        uint32_t sgw[CO_PER / 4];  // the entries' segments, four in a word
        auto sg = [&](int m) { return (sgw[m / 4] >> (8 * (m % 4))) & 0xFFu; };
        // Whole windows (all but the last) run without bounds tests, so that
        // each step's LDS accesses are in flight together.
        auto buckets = [&](auto whole) -> bool {
            constexpr bool ALL = decltype(whole)::value;
            auto in = [&](int m) { return ALL || t + m * CO_BLOCK < cnt; };
#pragma unroll
            for (int m = 0; m < CO_PER; m += 4)
                sgw[m / 4] = segid[t + m * CO_BLOCK] | (uint32_t)segid[t + (m + 1) * CO_BLOCK] << 8 |
                             (uint32_t)segid[t + (m + 2) * CO_BLOCK] << 16 | (uint32_t)segid[t + (m + 3) * CO_BLOCK] << 24;
            // smallest and largest value of each segment, in CO_COPIES copies
            // over the keys: a wave's lanes mostly share a segment, and 64
            // atomics on one address follow one another
            uint32_t *lows = kv, *highs = kv + CO_COPIES * CO_SEGS;
            for (int s = t; s < CO_COPIES * nseg; s += CO_BLOCK) {
                lows[s] = ~0u;
                highs[s] = 0;
            }
            __syncthreads();
            {
                const int copy = t % CO_COPIES;
                uint32_t lo = ~0u, hi = 0;
                uint32_t cs = sg(0);
                auto out = [&] {
                    atomicMin(&lows[CO_COPIES * cs + copy], lo);
                    atomicMax(&highs[CO_COPIES * cs + copy], hi);
                };
#pragma unroll
                for (int m = 0; m < CO_PER; m++) {
                    const uint32_t u = (uint32_t)x[m] ^ 0x80000000u;
                    if (in(m)) {
                        if (sg(m) != cs) {
                            out();
                            cs = sg(m);
                            lo = ~0u;
                            hi = 0;
                        }
                        lo = min(lo, u);
                        hi = max(hi, u);
                    }
                }
                if (in(0)) out();
            }
            __syncthreads();
            if (t < nseg) {
                uint32_t lo = ~0u, hi = 0;
#pragma unroll
                for (int c = 0; c < CO_COPIES; c += 4) {
                    const uint4 l = *(const uint4 *)&lows[CO_COPIES * t + c], h = *(const uint4 *)&highs[CO_COPIES * t + c];
                    lo = min(lo, min(min(l.x, l.y), min(l.z, l.w)));
                    hi = max(hi, max(max(h.x, h.y), max(h.z, h.w)));
                }
                const uint32_t st = segstart[t], len = segstart[t + 1] - st, range = hi - lo;
                const float scale = (float)len / ((float)range + 1.0f);
                atomicMax(&vbits, range ? 32u - (uint32_t)__builtin_clz(range) : 0u);
                if (len > CO_CROWD && scale >= (float)(CO_CROWD / 2)) few = 1;  // few values: sort
                smin[t] = lo;
                seg[t] = make_uint4(lo, __float_as_uint(scale), st, len - 1);
            }
            // segid becomes the buckets' counts, two in a word
#pragma unroll
            for (int m = 0; m < CO_PER / 2; m++) cw[t + m * CO_BLOCK] = 0;
            __syncthreads();
            if (few) return false;
            uint32_t at[CO_PER];  // bucket, and the entry's place by arrival << 16
#pragma unroll
            for (int m = 0; m < CO_PER; m++) {
                const uint4 S = seg[sg(m)];
                const uint32_t u = (uint32_t)x[m] ^ 0x80000000u;
                at[m] = S.z + min((uint32_t)((float)(u - S.x) * __uint_as_float(S.y)), S.w);
            }
            uint32_t last = 0;
#pragma unroll
            for (int m = 0; m < CO_PER; m++) {
                // a quarter shows the worst crowds, whose lanes meet at one address
                if (m == CO_PER / 4 && __syncthreads_or(last >= CO_CROWD)) return false;
                if (in(m)) {
                    const uint32_t sh = (at[m] & 1) * 16;
                    const uint32_t k = (atomicAdd(&cw[at[m] >> 1], 1u << sh) >> sh) & 0xFFFFu;
                    at[m] |= k << 16;
                    last = max(last, k);
                }
            }
            if (last > longest) atomicMax(&longest, last);
            __syncthreads();
            const int far = (int)longest;
            if (far >= CO_CROWD) return false;
            // where each bucket starts (thread t: buckets 16t .. 16t + 15)
            uint32_t w8[CO_PER / 2], sum = 0;
            {
                const uint4 f0 = f4[0], f1 = f4[1];
                w8[0] = f0.x, w8[1] = f0.y, w8[2] = f0.z, w8[3] = f0.w, w8[4] = f1.x, w8[5] = f1.y, w8[6] = f1.z,
                w8[7] = f1.w;
            }
#pragma unroll
            for (int m = 0; m < CO_PER / 2; m++) sum += w8[m];
            sum = (sum & 0xFFFFu) + (sum >> 16);
            uint32_t inc = sum;
#pragma unroll
            for (int d = 1; d < CO_WAVE; d <<= 1) {
                const uint32_t y = __shfl_up(inc, d, CO_WAVE);
                if (lane >= d) inc += y;
            }
            if (lane == CO_WAVE - 1) wsum[wv] = inc;
            __syncthreads();
            uint32_t o = inc - sum;
#pragma unroll
            for (int i = 0; i < CO_BLOCK / CO_WAVE; i++)
                if (i < wv) o += wsum[i];
#pragma unroll
            for (int m = 0; m < CO_PER / 2; m++) {
                const uint32_t o1 = o + (w8[m] & 0xFFFFu);
                const uint32_t o2 = o1 + (w8[m] >> 16);
                w8[m] = o | (o1 << 16);
                o = o2;
            }
            f4[0] = make_uint4(w8[0], w8[1], w8[2], w8[3]);
            f4[1] = make_uint4(w8[4], w8[5], w8[6], w8[7]);
            __syncthreads();
            // the entries by bucket, then each entry's place in its own: the
            // smaller values, and the equal ones before it
            uint32_t qe[CO_PER], y[CO_PER];  // the bucket: its start, and its end << 16; the entry's place
#pragma unroll
            for (int m = 0; m < CO_PER; m++) {
                const uint32_t bk = at[m] & 0xFFFFu;
                const uint32_t q0 = segid[bk], q1 = bk + 1 < CO_WIN ? segid[bk + 1] : (uint32_t)cnt;
                qe[m] = q0 | (q1 << 16);
                y[m] = q0;
            }
#pragma unroll
            for (int m = 0; m < CO_PER; m++)
                if (in(m))
                    keys[y[m] + (at[m] >> 16)] =
                        ((unsigned long long)((uint32_t)x[m] ^ 0x80000000u) << 12) | (unsigned)(t + m * CO_BLOCK);
            __syncthreads();
            for (uint32_t d = 0; d <= (uint32_t)far; d++) {
#pragma unroll
                for (int m0 = 0; m0 < CO_PER; m0 += 8) {
#pragma unroll
                    for (int m = m0; m < m0 + 8; m++) {
                        const uint32_t q = (qe[m] & 0xFFFFu) + d;
                        const unsigned long long e = keys[q];  // reads past the bucket are not used
                        const uint32_t u = (uint32_t)x[m] ^ 0x80000000u;
                        const unsigned long long own = ((unsigned long long)u << 12) | (unsigned)(t + m * CO_BLOCK);
                        y[m] += (q < (qe[m] >> 16)) & (e < own) ? 1u : 0u;
                    }
                }
            }
#pragma unroll
            for (int m = 0; m < CO_PER; m++)
                if (in(m)) {
                    const int sm = (int)sg(m);
                    z[a + t + m * CO_BLOCK] = base_of(sm) + (int64_t)(y[m] - segstart[sm]);
                    if (spans(sm)) vs[a + y[m]] = (uint32_t)x[m] ^ 0x80000000u;
                }
            return true;
        };
        if (cnt == CO_WIN ? buckets(std::true_type()) : buckets(std::false_type())) return;
        // the segment, the value above the segment's least and the position
        // in 32 bits
        const uint32_t vb = vbits;
        if (vb + 12 + (uint32_t)(32 - __builtin_clz((uint32_t)nseg)) <= 32) {
            uint32_t r[CO_PER];
#pragma unroll
            for (int m = 0; m < CO_PER; m++) {
                const int p = t + m * CO_BLOCK;
                const uint32_t u = (uint32_t)x[m] ^ 0x80000000u;
                r[m] = p < cnt ? ((sg(m) << vb | (u - smin[sg(m)])) << 12) | (unsigned)p : ~0u;
            }
            co_bitonic(r, t, kv);
            unsigned long long rl[CO_PER];
#pragma unroll
            for (int g = 0; g < CO_PER; g++) {
                const uint32_t s = min((r[g] >> 12) >> vb, (uint32_t)nseg - 1);
                rl[g] = ((unsigned long long)s << 44) |
                        ((unsigned long long)(smin[s] + ((r[g] >> 12) & ((1u << vb) - 1u))) << 12) | (r[g] & 0xFFFu);
            }
            finish(rl);
            return;
        }
        // the segments again, for the keys below
        __syncthreads();
#pragma unroll
        for (int m = 0; m < CO_PER; m++)
            if (t + m * CO_BLOCK < cnt) segid[t + m * CO_BLOCK] = (uint16_t)sg(m);
        __syncthreads();
    }

    // Bitonic sort of the keys (segment, value, position).  They start in
    // layout L, which is how the values were loaded.
    unsigned long long r[CO_PER];
#pragma unroll
    for (int g = 0; g < CO_PER; g++) {
        const int p = t + g * CO_BLOCK;
        const unsigned long long u = (uint32_t)x[g] ^ 0x80000000u;
        r[g] = p < cnt ? CO_KEY64 | ((unsigned long long)segid[p] << 44) | (u << 12) | (unsigned)p : CO_PAD64;
    }
    co_bitonic(r, t, keys);
#pragma unroll
    for (int g = 0; g < CO_PER; g++) r[g] &= ~CO_KEY64;
    finish(r);
}

// Per window, for the (at most two) columns that leave it: every other
// window u the column meets holds a sorted run of the column's values; its
// entries come first when their value is smaller, or equal and u < w.  The
// run is staged in LDS, then each entry of this window binary-searches it.
__global__ void __launch_bounds__(CO_BLOCK) k_co_merge(const int64_t *colptr, int64_t ncols, const int32_t *v,
                                                      int64_t nnz, const int64_t *first, int64_t nwin, int64_t *z,
                                                      const uint32_t *vs) {
    __shared__ uint32_t run[CO_WIN];
    const int t = threadIdx.x;
    const int64_t w = blockIdx.x;
    const CoWindow W = co_window(colptr, ncols, nnz, first, nwin, w);
    const int64_t a = W.a, b = a + W.cnt;
    // the window's first column, and the column running into the next window
    const int64_t ce0 = clampi(colptr[W.c0 + 1], W.cs0, nnz);
    const bool l = W.cs0 < a || ce0 > b;
    const bool r = W.cl >= 0 && W.cl != W.c0 && colptr[W.cl] < b;
    if (!l && !r) return;
    for (int side = 0; side < 2; side++) {
        if (side == 0 ? !l : !r) continue;  // uniform over the work-group
        const int64_t c = side == 0 ? W.c0 : W.cl;
        const int64_t cs = side == 0 ? W.cs0 : clampi(colptr[c], a, b);
        const int64_t ce = side == 0 ? ce0 : clampi(colptr[c + 1], b, nnz);
        const int64_t ps = max(cs, a), pe = min(ce, b);
        if (pe <= ps) continue;  // only for a colptr that breaks the rules
        uint32_t xv[CO_PER];
        int64_t add[CO_PER];
#pragma unroll
        for (int m = 0; m < CO_PER; m++) {
            const int64_t p = ps + t + m * CO_BLOCK;
            xv[m] = (uint32_t)v[min(p, pe - 1)] ^ 0x80000000u;
            add[m] = 0;
        }
        const int nm = (int)((pe - ps + CO_BLOCK - 1) / CO_BLOCK);  // entries per thread, at most
        const int64_t w0 = cs / CO_WIN, w1 = (ce - 1) / CO_WIN;
        for (int64_t u = w0; u <= w1; u++) {
            if (u == w) continue;
            const int64_t rs = max(cs, u * CO_WIN);
            const int len = (int)(min(ce, (u + 1) * CO_WIN) - rs);
            if (len <= 0) continue;  // only for a colptr that breaks the rules
            __syncthreads();
            for (int i = t; i < len; i += CO_BLOCK) run[i] = vs[rs + i];
            __syncthreads();
            const bool before = u < w;
            // steps of at most the run's length (28 -> 24 us on 2000 columns of 1999)
            // branchless search, steps outermost so that the entries' LDS
            // reads of one step are in flight together: pos = the run's
            // entries that come first (a prefix, since the run is sorted)
            int pos[CO_PER];
#pragma unroll
            for (int m = 0; m < CO_PER; m++) pos[m] = 0;
            for (int step = 1 << (31 - __builtin_clz((unsigned)len)); step > 0; step >>= 1) {
#pragma unroll
                for (int m = 0; m < CO_PER; m++) {
                    if (m >= nm) break;
                    const int at = pos[m] + step;
                    const uint32_t y = run[min(at, len) - 1];
                    const bool first_ = y < xv[m] || (before && y == xv[m]);
                    pos[m] += (at <= len && first_) ? step : 0;
                }
            }
#pragma unroll
            for (int m = 0; m < CO_PER; m++) add[m] += pos[m];
        }
#pragma unroll
        for (int m = 0; m < CO_PER; m++) {
            const int64_t p = ps + t + m * CO_BLOCK;
            if (p < pe) z[p] += add[m];
        }
        __syncthreads();  // the next side reuses the run buffer
    }
}

// Scratch of one call: the first column of every window (nwin int64), then
// the sorted runs of the windows (nnz uint32) at off_vs.
static size_t co_scratch_off(int64_t nwin) { return ((size_t)nwin * 8 + 255) & ~(size_t)255; }

static int co_launch(const int64_t *colptr, int64_t ncols, const int32_t *v, int64_t nnz, int64_t *z, char *ws,
                     int64_t nwin, hipStream_t s) {
    int64_t *first = (int64_t *)ws;
    uint32_t *vs = (uint32_t *)(ws + co_scratch_off(nwin));
    const int64_t gb = (ncols + CO_BLOCK - 1) / CO_BLOCK;
    hipLaunchKernelGGL(k_co_first, dim3((unsigned)(gb < 8192 ? gb : 8192)), dim3(CO_BLOCK), 0, s, colptr, ncols,
                       nnz, first);
    hipLaunchKernelGGL(k_co_local, dim3((unsigned)nwin), dim3(CO_BLOCK), 0, s, colptr, ncols, v, nnz,
                       (const int64_t *)first, nwin, z, vs);
    hipLaunchKernelGGL(k_co_merge, dim3((unsigned)nwin), dim3(CO_BLOCK), 0, s, colptr, ncols, v, nnz,
                       (const int64_t *)first, nwin, z, (const uint32_t *)vs);
    return hipGetLastError() == hipSuccess ? VR_OK : VR_EHIP;
}

// Checks shared by both entry points; *nwin = the windows of nnz entries.
static int co_check(const int64_t *colptr, int64_t ncols, const int32_t *v, int64_t nnz, const int64_t *z,
                    int64_t *nwin) {
    if (ncols < 0 || nnz < 0 || (ncols > 0 && !colptr)) return VR_EINVAL;
    *nwin = (nnz + CO_WIN - 1) / CO_WIN;
    if (nnz == 0) return VR_OK;
    if (ncols == 0 || !v || !z) return VR_EINVAL;
    if (*nwin > 0x7FFFFFFF) return VR_E2BIG;
    return VR_OK;
}

extern "C" VR_API int vr_column_order(const int64_t *colptr, int64_t ncols, const int32_t *v, int64_t nnz,
                                      int64_t *z, void *stream) {
    int64_t nwin = 0;
    const int st = co_check(colptr, ncols, v, nnz, z, &nwin);
    if (st != VR_OK || nnz == 0) return st;
    const hipStream_t s = (hipStream_t)stream;
    char *ws = (char *)cache_get(co_scratch_off(nwin) + (size_t)nnz * 4, s);
    if (!ws) return VR_ENOMEM;
    const int rc = co_launch(colptr, ncols, v, nnz, z, ws, nwin, s);
    cache_put(ws, s);
    return rc;
}

// ------------------------------------------------- without allocation ----
// The scratch of vr_column_order_noalloc: one array per GPU, loaded with the
// code object and held until the process ends.  In host code its name only
// stands in for the array, so each GPU's device address is looked up once
// (hipGetSymbolAddress, with that GPU current) and used from then on.
static __device__ __align__(256) unsigned char scratch[VR_COLORDER_NOALLOC_BYTES];

namespace {
constexpr int CO_MAX_DEVICES = 64;
std::mutex g_scratch_mu;
char *g_scratch[CO_MAX_DEVICES];

// Device address of the current GPU's scratch array; nullptr when the
// lookup fails.
char *scratch_here() {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= CO_MAX_DEVICES) return nullptr;
    std::lock_guard<std::mutex> g(g_scratch_mu);
    if (!g_scratch[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return nullptr;
        g_scratch[dev] = (char *)p;
    }
    return g_scratch[dev];
}
}  // namespace

extern "C" VR_API int vr_column_order_noalloc(const int64_t *colptr, int64_t ncols, const int32_t *v, int64_t nnz,
                                              int64_t *z, void *stream) {
    int64_t nwin = 0;
    const int st = co_check(colptr, ncols, v, nnz, z, &nwin);
    if (st != VR_OK || nnz == 0) return st;
    if (co_scratch_off(nwin) + (size_t)nnz * 4 > (size_t)VR_COLORDER_NOALLOC_BYTES) return VR_E2BIG;
    char *ws = scratch_here();
    if (!ws) return VR_EHIP;
    return co_launch(colptr, ncols, v, nnz, z, ws, nwin, (hipStream_t)stream);
}
