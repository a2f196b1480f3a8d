// vr_morse.h -- the dimension-1 reduction on the critical cells (k_morse.hip),
// as vr_pairs_dim1 calls it.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

// Pairs of dimension 1 of a build's K edges and T > 0 triangles into
// tri_of_edge (K entries, device).  R: the n x n rank matrix (+inf off the
// edges, -1 on the diagonal).  Enqueued on s; scratch from the library's
// cache.  *done is false when a limit of the method was passed (tri_of_edge
// then holds the apparent pairs alone); synchronises s.  Returns a vr_status.
int morse_pairs_dim1(const int32_t *R, const int32_t *ij, const unsigned long long *key, const int32_t *e_low,
                     int64_t n, int64_t K, int64_t T, int32_t *tri_of_edge, bool *done, hipStream_t s);

// Pairs of dimension 2 of a build's T > 0 triangles from the links of its
// edges (k_links.hip) into tri_tet (T entries, device).  R as above; rng[2r],
// rng[2r + 1]: the triangles of value r, first and one past the last; clr: 1
// for the triangles paired with an edge; toff: the tetrahedra's offsets by
// value; scratch: link_pairs_scratch(K, T) bytes, device.  *done is false
// when a limit of the method was passed (tri_tet is then not complete);
// synchronises s.  Returns a vr_status.
size_t link_pairs_scratch(int64_t K, int64_t T);
int link_pairs_dim2(const int32_t *R, const int32_t *ij, const unsigned long long *tri, const long long *toff,
                    const int32_t *rng, const int32_t *clr, int64_t n, int64_t K, int64_t T, long long *tri_tet,
                    void *scratch, bool *done, hipStream_t s);
