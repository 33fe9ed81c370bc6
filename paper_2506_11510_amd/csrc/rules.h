// rules.h -- rules of the build and of the walks that need neither HIP nor
// memory, so that a compiler for the CPU can check them over whole ranges.
#pragma once
#include <cstdint>

namespace tv {

// Tag of a tet: the vertex with which its first one spans the edge it bisects.
__host__ __device__ inline int tag_of(int depth) { return 3 - depth % 3; }

// Edges (bits in hanging's order) of a tet of depth d whose midpoints can be
// vertices while no tet deeper than smax has been split.  Every tet around an
// edge bisects it at the same depth, if it gets there: by tag (columns 3, 2,
// 1) and edge, the tet's depth plus
//   x0x1 2 1 0   x0x2 1 0 2   x0x3 0 2 1   x1x2 2 1 2   x1x3 1 2 1   x2x3 2 2 3
// The rounds split breadth first, so most new leaves are the deepest yet and
// have no edge to look up: the lookups are random reads of a table past the
// caches.  Passes over a 6.2 M tet build: want 900 -> 730 us, mark 430 -> 330.
__host__ __device__ inline uint32_t edges_upto(int d, int smax) {
  const int s = smax - d, t = tag_of(d);
  if (s < 0) return 0u;
  const uint32_t lv = t == 3 ? 0x3F3F1604u : (t == 2 ? 0x3F3F0B02u : 0x3F1F1501u);  // a byte per s
  return (lv >> (8 * (s < 3 ? s : 3))) & 0xFFu;
}

// Heap id at depth dmax (<= 60) of the tet holding a point, from the Kuhn root
// h whose axis order sorts it: f0 >= f1 >= f2 >= 0 are its coordinates along
// the root's axes, s the cube's edge.  Every tet whose depth is a multiple of
// three is a Kuhn tet again: from its vertex x_0 along three signed axes in
// turn, all by one edge length s.  In its own coordinates (0 <= f2 <= f1 <=
// f0 <= s) the three bisections below it are the planes f0 + f2 = s; f0 + f1
// = s or, beyond the first, f1 + f2 = s; and a coordinate = s / 2; each
// second child lies above its plane.  The Kuhn tet of edge s / 2 reached
// starts at the vertex with as many of the bits 0 as its own x_0 has axes
// left at 0, so its coordinates are the f's folded at s (f or s - f).  So
// three bisections are three compares and a few selects (about 30
// instructions; from the vertices, with the bisection normals from the shape
// table, they were 150 in 32-bit integers, 240 in FP64): the links of 6.2 M
// tets 602 -> 345 us, the camera rays of a 33.6 M sample frame 9.93 -> 9.46 ms.
// A point on a plane takes the first child (ABOVE: the second).  Exact when
// f +- f and s - f are.
template <bool ABOVE, class T>
__host__ __device__ inline uint64_t fold_path(T f0, T f1, T f2, T s, int dmax, uint64_t h) {
  for (int d = 0; d < dmax; d += 3) {
    const T a = f0 + f2;
    const bool b1 = ABOVE ? a >= s : a > s;
    const T b = (b1 ? f2 : f0) + f1;
    const bool b2 = ABOVE ? b >= s : b > s;
    const T p = b1 ? (b2 ? f2 : f1) : (b2 ? f1 : f0), r = s - p;
    const bool b3 = ABOVE ? p >= r : p > r;
    const T r0 = s - f0;
    const T g1 = b1 ? (b2 ? s - f1 : f2) : (b2 ? r0 : f1);
    f2 = b1 ? r0 : f2;
    f1 = g1;
    f0 = b3 ? r : p;
    s = s / 2;
    h = 8 * h + (b1 ? 4 : 0) + (b2 ? 2 : 0) + (b3 ? 1 : 0);
  }
  return h >> ((3 - dmax % 3) % 3);
}

// The 9 face directions' dot products with a segment's direction and their
// reciprocals: NaN for 0, all 0 when one is too small for exit_face's bounds
// (the table's layout in LDS is described at set_segment).
struct SegDirs {
  float r[9], d[9];
};

__host__ __device__ inline void seg_dirs(float x, float y, float z, SegDirs& s) {
  const float d[9] = {x, y, z, x + y, x - y, x + z, x - z, y + z, y - z};
  bool tiny = x == 0.0f && y == 0.0f && z == 0.0f;
  for (int N = 0; N < 9; N++) tiny = tiny || (d[N] != 0.0f && !(d[N] <= -0x1p-40f || d[N] >= 0x1p-40f));
  for (int N = 0; N < 9; N++) {
    s.d[N] = d[N];
    s.r[N] = tiny ? 0.0f : (d[N] == 0.0f ? __builtin_nanf("") : 1.0f / d[N]);
  }
}

}  // namespace tv
