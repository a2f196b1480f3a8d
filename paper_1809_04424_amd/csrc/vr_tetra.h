// vr_tetra.h -- which kernels count and list the tetrahedra (k_pairs.hip).
#pragma once

#include <stdint.h>

// One wave per edge needs no barrier, and the writer no count
// of its own, since a wave's places follow from off[r].  Bound by the latency
// of the chain (rows, L, pairs), which more waves in flight hide.  It is taken
// for up to TET_WAVE_N points (L's room), from 4096 edges on (with fewer all
// edges run at once with four waves each), and where the links, T / K vertices
// on average, are small enough for one wave.  us with four waves / with one
// (a list takes its count too):
//   T / K  K       count        list
//    12    11975    23 /  19     52 /  22    (400 points; kernels alone)
//     9    24975    76 /  58    229 / 141    (1000 points; calls from here on)
//    18    11212    39 /  41    125 /  98    (300)
//    49    11175    55 /  96    223 / 246    (150, all edges)
//    50    99900   416 / 429   1628 / 1291   (1000)
//    57   157132   739 / 1015  3159 / 2881   (1024)
//   133    79800   735 / 1361  4618 / 5135   (400, all edges)
// The count's rows of pairs leave few lanes idle in long links, so four waves
// count those faster; a writer's longest link wants many other edges beside it.
// T = 0 says nothing of the links: a build up to the edges lists no triangles
// (400 points, all edges: count 746 -> 1365, list 4875 -> 5186; 1000 points,
// 99900 edges in random order: 209 -> 151 and 726 -> 392).
#define TET_WAVE_N 1024

static inline bool tet_by_wave(bool write, int64_t n, int64_t K, int64_t T) {
    if (n > TET_WAVE_N || K < 4096 || T == 0) return false;
    if (!write) return T <= 16 * K;
    return T <= 32 * K || (T <= 64 * K && K >= 65536);
}
