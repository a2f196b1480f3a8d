// vr_morse.h -- the dimension-1 reduction on the critical cells (k_morse.hip),
// as vr_pairs_dim1 calls it.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

// Entry x of the n x n rank matrix before its edges: i n + j = i (n + 1) on
// the diagonal.  n <= 8192, so 32 bits hold x.
__device__ __forceinline__ int32_t vr_rank_none(uint32_t x, int64_t n) {
    return x % (uint32_t)(n + 1) ? 0x7FFFFFFF : -1;
}

// Edge r into it.
__device__ __forceinline__ void vr_rank_edge(int32_t *R, const int32_t *ij, int64_t n, int64_t r) {
    const int64_t i = ij[2 * r], j = ij[2 * r + 1];
    if (i < 0 || j < 0 || i >= n || j >= n) return;  // never for a library result
    R[i * n + j] = (int32_t)r;
    R[j * n + i] = (int32_t)r;
}

// Pairs of dimension 1 of a build's K edges and T > 0 triangles into
// tri_of_edge (K entries, device).  R: room for the n x n rank matrix (+inf off
// the edges, -1 on the diagonal), which is written first.  Enqueued on s; scratch from the library's
// cache.  *done is false when a limit of the method was passed (tri_of_edge
// then holds the apparent pairs alone); synchronises s.  Returns a vr_status.
int morse_pairs_dim1(int32_t *R, const int32_t *ij, const unsigned long long *key, const int32_t *e_low,
                     int64_t n, int64_t K, int64_t T, int32_t *tri_of_edge, bool *done, hipStream_t s);

// Pairs of dimension 2 of a build's T > 0 triangles from the links of its
// edges (k_links.hip) into tri_tet (T entries, device).  R: the rank matrix; rng[2r],
// rng[2r + 1]: the triangles of value r, first and one past the last; clr: 1
// for the triangles paired with an edge; toff: the tetrahedra's offsets by
// value; scratch: link_pairs_scratch(K, T) bytes, device, where there are any
// the first word 1 when a value has more than LINK_PAIRS_MOST triangles, else
// 0, and the rest of the first LINK_PAIRS_ZERO bytes zero.  *done is false
// when a limit of the method was passed (tri_tet is then not complete);
// synchronises s.  Returns a vr_status.
#define LINK_PAIRS_ZERO 16
#define LINK_PAIRS_MOST 64
size_t link_pairs_scratch(int64_t K, int64_t T);
int link_pairs_dim2(const int32_t *R, const int32_t *ij, const unsigned long long *tri, const long long *toff,
                    const int32_t *rng, const int32_t *clr, int64_t n, int64_t K, int64_t T, long long *tri_tet,
                    void *scratch, bool *done, hipStream_t s);
