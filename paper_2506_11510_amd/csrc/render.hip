// render.hip -- Monte Carlo volumetric path tracing through the tet grid
// (paper, "Volumetric Path Tracing": Algorithm 1 and "Path Tracing within
// Tetrahedral Grids").
//
// Three kernels per pass of samples:
//   k_first   -- one thread per (pixel, sample): camera ray, entry into the
//                grid, point location, and the walk of the camera segment up
//                to its first real collision or its escape.  The samples of
//                a pixel are neighbouring lanes, so a wave's lanes walk the
//                same tets side by side and leave together.  Escaped samples
//                are done; the others leave their collision in their
//                32-byte entry record and their index in a list;
//   k_render  -- persistent, over the listed paths only: every lane runs a
//                small state machine over its own paths (fetch work -> light
//                estimate -> scatter -> walk steps of the scattered segment,
//                and of the light (shadow) ray where it is not queued).  Each
//                loop iteration advances every walking lane by one cell, so
//                lanes whose paths differ in length stay busy; idle lanes
//                take new paths from a device counter with one atomic per
//                wave (ballot + popcount).  All rare events (collision, light
//                estimate and phase sampling, escape, end of path, new work)
//                sit in one section the wave enters only when some lane
//                needs it; the common iteration is a bare walk step;
//   k_resolve -- sums the samples' radiance per pixel, in sample order.
// Light rays that k_render queued are walked after it by k_light; k_chain adds
// their terms to the samples before k_resolve, or k_light to the pixels after.
//
// One walk step reads one 48- or 32-byte tet record (face plane constants, face
// orientation codes, 4 neighbour links, extinction) and leaves by a face
// whose outward normal faces the ray (n.d > 0, at most 3).  The dot products
// of the segment's origin and direction with the 9 possible face directions,
// and the latter's reciprocals, are computed once per segment into a per-lane
// LDS table, so a face costs one LDS read pair, a subtraction and a product
// (exit_face); every dot product is rounded exactly as the direct FP32 one
// would be.  The free flight is delta tracking against the
// per-tet majorant with an optical depth carried across cells; real
// collisions scatter by Henyey-Greenstein after a next-event estimate of the
// directional light (transmittance by walking the light ray to the grid
// boundary); paths leaving the grid see the constant environment.
//
// The same kernel, instantiated on the voxel grid (Amanatides-Woo steps),
// is the regular-grid reference renderer.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <string>
#include <type_traits>
#include <vector>

#include <rocprim/device/device_radix_sort.hpp>

#include "nrc.h"
#include "plan.h"

namespace tv {

// Entry record of one camera sample (32 bytes).  From k_first: the first real
// collision (point, tet, direction of the segment that reached it, walk
// steps so far), or, with cell = kDone, the finished sample's radiance.
// k_render replaces the collisions by the radiance their paths gathered;
// where a sample's light rays are queued to be summed with it (A.chain), cell
// = kChained says that the terms of the queue records from `steps` on are
// still to come before it (k_chain).  A path whose light ray finds the queue
// full waits there as the collision, its queue records so far from `steps` on.
struct alignas(16) RayEntry {
  float px, py, pz;
  uint32_t cell;
  float dx, dy, dz;
  uint32_t steps;
};
constexpr uint32_t kDone = 0xFFFFFFFFu, kChained = 0xFFFFFFFEu;  // (tets and voxels are fewer than 2^31)

// One scene of a batch (several grids rendered by one launch sequence):
// the scenes' entry records are concatenated.
// Extra per-tet data a scene may carry: channels (null = absent) with the
// emitted radiance per unit temperature, and the density model inside the
// tets (0 = constant; 1 linear coefficients; 2 voxel lookup in an n^3
// volume times a scale).
struct ExtArgs {
  const float* ch_t;
  const float* ch_a;
  const float* ch_g;
  float emission[3];
  int32_t model;
  const float4* mcoef;
  const float* mdens;
  int32_t mn;
  float mscale;
};

struct SceneDesc {
  Frame fr;
  float albedo, g;
  float sun[3], E[3], env[3];
  int32_t spp, tiles_x;
  uint64_t seed;
  uint32_t s0;       // first sample index
  uint64_t entry0;   // first entry record
  uint64_t pix0;     // first pixel in the concatenated images
  const void* rec;   // traversal records (TetRec32 or TetRec)
  const uint64_t* keys;
  const uint32_t* kidx;
  int64_t n;
  int32_t dmax, kbits;
  float* out;
  ExtArgs ex;
};

// Largest k < n with key(k) <= v (key ascending, key(0) = 0).
template <class F>
__device__ inline int scene_search(int n, uint64_t v, F key) {
  int lo = 0, hi = n;
  while (hi - lo > 1) {
    int mid = (lo + hi) >> 1;
    if (key(mid) <= v) lo = mid;
    else hi = mid;
  }
  return lo;
}

// A light ray whose walk is deferred: its origin (the real collision), the
// collision's tet, the light estimate's weight before the irradiance
// (throughput after the albedo x phase function), what it adds to, and the
// path's next record.  With A.chain the walked ray's term replaces x, y, z.
struct alignas(16) LightRec {
  float x, y, z;
  uint32_t cell;  // kDone: an unused record (the end of a wave's last chunk)
  float bp;
  uint32_t to;      // entry record (A.chain), else pixel; light term (training paths)
  uint32_t next;    // A.chain: the path's next record (kDone: none)
  uint32_t bounce;  // | kToTerm for training paths
};
constexpr uint32_t kToTerm = 0x80000000u;

// The launches' counters in device memory (kHeadBytes at the start of the
// scratch), each on a 128-byte line of its own: atomics on one line serialise.
// Lists 0..7 are the eight contiguous bands of the entry records (one per
// XCD), list 8 the radiance cache's training paths.
constexpr int kLists = 9, kTrainList = 8;
constexpr int kLine = 32;                              // 32-bit words per line
constexpr int kTakenAt = 0;                            // listed paths taken so far, per list
constexpr int kCountAt = kLists * kLine;               // listed paths, per list
constexpr int kQueryAt = 2 * kLists * kLine;           // radiance-cache queries of the pass
constexpr int kChunkAt = (2 * kLists + 1) * kLine;     // light-ray queue chunks taken in the pass
constexpr int kPassWords = (2 * kLists + 2) * kLine;   // the words above are zeroed before each pass
// Statistics: blocks add to the slot of their index, the host sums the slots
// (262 K blocks adding to one address took longer than their walks).
constexpr int kStatSlots = 64;
constexpr int kStatAt = (kPassWords + 63) / 64 * 64;
constexpr size_t kHeadBytes = (size_t)(kStatAt + kStatSlots * kLine) * 4;

struct RenderArgs {
  Frame fr;
  float albedo, g;
  float sun[3], E[3], env[3];
  int32_t spp;          // samples per pixel of the whole render (divisor)
  int32_t pass_start;   // first sample index of this pass
  int32_t pass_spp;     // samples of this pass
  int32_t max_bounces, transmittance;
  uint32_t max_steps;
  uint64_t seed;
  uint32_t slots;
  uint32_t batch;       // paths a wave takes per atomic
  int32_t event_wait;   // lanes waiting for an event before the wave handles events
  int32_t tiles_x;
  RayEntry* entries;
  float* out;
  uint32_t* head;       // counters and statistics
  // listed paths: list b starts at list + b * band_size, the training
  // paths' (radiance cache, with an image) at list + train_list0
  uint32_t* list;
  uint32_t band_size;
  uint32_t chunk_blocks;  // blocks of neighbouring entries dealt to one list at a time
  uint32_t train_list0;
  // radiance cache
  int32_t train;         // the entries are training paths (pixel from train_pixel, sample = entry)
  uint32_t npix;         // width * height
  int32_t truncate;      // real vertex where a path queries the cache
  int32_t rec_vertices;  // vertices recorded per training path
  float4* qbuf;          // cache queries of the pass, compacted: (x, sigma), (d, beta)
  uint32_t* qpix;        // their pixels
  uint32_t* qcount;      // queries so far (one atomic per wave)
  float4* vrec;          // training-path vertex records
  float4* path_l;        // training-path radiance and vertex count
  const tet_nrc* nrc;    // host handle (the query pass), never read on the device
  uint32_t train_items;  // cache mode 1: training paths traced with the image (first pass only)
  uint32_t train_blocks; // blocks of k_first that trace them
  uint32_t train_ent0;   // their entry records follow the image's
  uint64_t train_seed;   // their Philox key
  // batch of scenes
  const SceneDesc* scenes;
  int32_t nscenes;
  uint64_t total_entries;
  ExtArgs ex;  // channels and density model of a single-scene render
  // deferred light rays (defer != 0): a wave of the tracing kernel takes
  // chunks of lq_chunk records of the queue as it fills them (lq_chunks in
  // all); they are walked after the pass in the order of where they start
  LightRec* lq;
  uint32_t lq_chunk, lq_chunks;
  // training paths with deferred light rays: the light (and emission) each
  // vertex gathers, terms[2 (path max_bounces + vertex)] (and + 1), summed by
  // k_gather_terms in path order
  float4* terms;
  int32_t defer;
  // chain != 0: queued light terms are summed per sample, in path order, as a
  // lane that walks its own light rays sums them (k_chain); paths that find
  // the queue full wait for a second launch (resume != 0), whose lanes do that
  int32_t chain, resume;
};

__device__ inline unsigned long long* stat_slot(const RenderArgs& A) {
  return (unsigned long long*)(A.head + kStatAt + (blockIdx.x & (kStatSlots - 1)) * kLine);
}

// Extinction at o + t d inside tet `cell` under the grid's density model:
// linear ((c0 + gx x) + gy y) + gz z, or the scale times the voxel
// floor(x n) (indices clamped); FP32.
__device__ inline float model_sigma(const ExtArgs& X, uint32_t cell, float3 o, float3 d, float t) {
  const float x0 = o.x + t * d.x, x1 = o.y + t * d.y, x2 = o.z + t * d.z;
  if (X.model == 1) {
    const float4 c = X.mcoef[cell];
    return ((c.x + c.y * x0) + c.z * x1) + c.w * x2;
  }
  const int32_t n = X.mn;
  const float fn = (float)n;
  int64_t i = (int64_t)floorf(x0 * fn), j = (int64_t)floorf(x1 * fn), k = (int64_t)floorf(x2 * fn);
  i = i < 0 ? 0 : (i >= n ? n - 1 : i);
  j = j < 0 ? 0 : (j >= n ? n - 1 : j);
  k = k < 0 ? 0 : (k >= n ? n - 1 : k);
  return X.mscale * X.mdens[i + (int64_t)n * (j + (int64_t)n * k)];
}

// Pixel of training path j: floor(w npix / 2^24), w = the upper 24 bits of
// word 0 of Philox(counter (j, 0, 4, 0)).
__device__ inline uint32_t train_pixel(uint64_t seed, uint32_t j, uint32_t npix) {
  uint4 r = philox10(make_uint4(j, 0u, 4u, 0u), (uint32_t)seed, (uint32_t)(seed >> 32));
  return (uint32_t)(((uint64_t)(r.x >> 8) * npix) >> 24);
}

// pixel of a slot: 8x8 tiles in row-major tile order
__device__ inline bool slot_pixel(uint32_t slot, int32_t tiles_x, int32_t w, int32_t h, int32_t& px, int32_t& py) {
  uint32_t tile = slot >> 6, q = slot & 63u;
  px = (int32_t)((tile % (uint32_t)tiles_x) * 8 + (q & 7u));
  py = (int32_t)((tile / (uint32_t)tiles_x) * 8 + (q >> 3));
  return px < w && py < h;
}

struct Step {
  float te, sigma, majorant;
  int32_t next;  // -1: leaves the grid
  bool ok;       // false: no exit face
};

// ---------------------------------------------------------------- tet medium
template <int K>
__device__ inline void descend_point(int32_t v[4][3], uint64_t& h, uint32_t& cls, const uint32_t* __restrict__ shapes,
                                     const double P[3]) {
  const uint32_t w = shapes[cls];
  int32_t z[3], u[3];
  shape_bisector<K>(v, w, z, u);
  double side = 0.0;
#pragma unroll
  for (int i = 0; i < 3; i++) {
    const double t = P[i] - (double)z[i];
    if (u[i]) side = side + (u[i] > 0 ? t : -t);
  }
  cls = side >= 0.0 ? (w >> 8) & 255u : (w >> 16) & 255u;
  if (side >= 0.0) {
#pragma unroll
    for (int i = 0; i < 3; i++) v[K][i] = z[i];
    h = 2 * h;
  } else {
#pragma unroll
    for (int j = 0; j < K; j++)
#pragma unroll
      for (int i = 0; i < 3; i++) v[j][i] = v[j + 1][i];
#pragma unroll
    for (int i = 0; i < 3; i++) v[K][i] = z[i];
    h = 2 * h + 1;
  }
}

// Tet containing p: the Kuhn root whose axis order sorts p's coordinates in
// descending order, bisections down to the grid's depth (folded coordinates;
// bisected vertices where those would not be exact), then the last tet whose
// depth-first key is <= the key reached.
__device__ inline int64_t locate_point(const uint64_t* __restrict__ keys, const uint32_t* __restrict__ kidx, int kbits,
                                       int dmax, const uint32_t* __restrict__ shapes, float3 p) {
  const float c[3] = {p.x, p.y, p.z};
  int r = -1;
  if (c[0] >= c[1] && c[1] >= c[2]) r = 0;
  else if (c[0] >= c[2] && c[2] >= c[1]) r = 1;
  else if (c[1] >= c[0] && c[0] >= c[2]) r = 2;
  else if (c[1] >= c[2] && c[2] >= c[0]) r = 3;
  else if (c[2] >= c[0] && c[0] >= c[1]) r = 4;
  else if (c[2] >= c[1] && c[1] >= c[0]) r = 5;
  if (r < 0) return -1;
  const double P[3] = {(double)p.x * (double)kLatS, (double)p.y * (double)kLatS, (double)p.z * (double)kLatS};
  // Coordinates that are 0 or at least 2^-29 are multiples of 2^-32 lattice
  // units: then both ways of descending are exact in FP64 and agree.  The
  // points on the cube's surface that paths enter at nearly always are.
  if ((c[0] == 0.0f || c[0] >= 0x1p-29f) && (c[1] == 0.0f || c[1] >= 0x1p-29f) && (c[2] == 0.0f || c[2] >= 0x1p-29f)) {
    const double hi = fmax(fmax(P[0], P[1]), P[2]), lo = fmin(fmin(P[0], P[1]), P[2]);
    const double mid = fmax(fmin(P[0], P[1]), fmin(fmax(P[0], P[1]), P[2]));
    return search_keys_idx(keys, kidx, kbits,
                           fold_path<false>(hi, mid, lo, (double)kLatS, dmax, 8 + (uint64_t)r) << (60 - dmax));
  }
  const int p0 = (r < 2) ? 0 : (r < 4 ? 1 : 2);
  const int p1 = (r == 0 || r == 5) ? 1 : ((r == 1 || r == 3) ? 2 : 0);
  int32_t v[4][3];
#pragma unroll
  for (int a = 0; a < 3; a++) {
    v[0][a] = 0;
    v[1][a] = a == p0 ? kLatS : 0;
    v[2][a] = (a == p0 || a == p1) ? kLatS : 0;
    v[3][a] = kLatS;
  }
  uint64_t h = 8 + (uint64_t)r;
  uint32_t cls = shapes[kShapeWords + r];
  for (int d = 0; d < dmax; d += 3) {
    descend_point<3>(v, h, cls, shapes, P);
    if (d + 1 < dmax) descend_point<2>(v, h, cls, shapes, P);
    if (d + 2 < dmax) descend_point<1>(v, h, cls, shapes, P);
  }
  return search_keys_idx(keys, kidx, kbits, h << (60 - dmax));
}

// Per-lane LDS table of a segment with direction d from origin o, for the 9
// face directions dir_N: [0, 9) the reciprocals of dir_N . d, [9, 18)
// dir_N . o times kOriginScale, [18, 27) dir_N . d; each dot product rounded
// as (n.x a.x + n.y a.y) + n.z a.z would be (its zero terms are exact).  The
// reciprocal is the correctly rounded one; NaN where dir_N . d = 0 (such a
// face is never crossed), and 0 for all 9 when a dot product is too small
// for exit_face's bounds (|dir_N . d| < 2^-40, or NaN, or d = 0), which makes every
// step of the segment take its general path (seg_dirs).
// Each wave has a table of its own, entry k of lane i at k * kTabRow + i: a
// lane's reads stay in its own bank whichever entry it reads.
constexpr int kTabRow = 64;
constexpr int kTabDot = 9, kTabDen = 18, kTabRows = 27;

// The origin's 9 entries, at tab[N * kTabRow].
__device__ inline void set_origin(float* tab, float3 o, float oscale) {
  o = make_float3(o.x * oscale, o.y * oscale, o.z * oscale);
  const float v[9] = {o.x, o.y, o.z, o.x + o.y, o.x - o.y, o.x + o.z, o.x - o.z, o.y + o.z, o.y - o.z};
#pragma unroll
  for (int N = 0; N < 9; N++) tab[N * kTabRow] = v[N];
}

template <class Med>
__device__ inline void set_segment(float* tab, float3 o, float3 d) {
  SegDirs s;
  seg_dirs(d.x, d.y, d.z, s);
  if constexpr (Med::kTet) {
#pragma unroll
    for (int N = 0; N < 9; N++) {
      tab[N * kTabRow] = s.r[N];
      tab[(kTabDen + N) * kTabRow] = s.d[N];
    }
    set_origin(tab + kTabDot * kTabRow, o, Med::kOriginScale);
  } else {
#pragma unroll
    for (int N = 0; N < 3; N++) tab[N * kTabRow] = s.r[N];
  }
}

__device__ inline uint64_t ballot64(bool x) { return __builtin_amdgcn_ballot_w64(x); }
__device__ inline bool lane_of(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }
// Bits 27..30 as one bit-field extract: left to the compiler it becomes
// shift, mask and add before an address add.
__device__ inline uint32_t bits27_30(uint32_t x) {
  uint32_t r;
  asm("v_bfe_u32 %0, %1, 27, 4" : "=v"(r) : "v"(x));
  return r;
}

// Exit of a tet along a segment: faces whose outward normal n has n . d > 0
// are candidates; the exit face has the smallest exact quotient num / den of
// num = offset - n . o and den = n . d (both FP32), the lowest face on ties;
// bt = that quotient correctly rounded.  c[f] is face f's plane constant along
// +dir_N, dn[f] its N, the sign bit of w[f] says that n = -dir_N (num and den
// then both change sign, the quotient does not).  False: no candidate.
//
// A wave spends its time on VALU issue here, so the common path avoids FP64 and
// division: q = num * RN(1 / den) is within 2^-22 (relative) of the exact
// quotient, so a candidate whose q is the only one up to min q (1 + 2^-20)
// is the exact minimum.  From q, two FMA corrections with the exact
// remainder give the correctly rounded quotient (the first leaves it within
// an ulp, the second, from a correctly rounded reciprocal, rounds it
// correctly; q > 2^-40 and |den| >= 2^-40 keep the remainders exact).  Near
// ties, smaller or negative q, tiny dens (every candidate's q is then 0) and
// no candidate at all (at least two q are then infinite: at most two of a
// tet's four face normals can be normal to a direction) go the general way: exact FP64 cross products and an IEEE division.
// NPAY: the payload of a face holds its N at bits 27..30.  SHARED: all lanes
// of the block have one direction, whose entries are dirs[0, 9) (reciprocals)
// and dirs[9, 18); tab then holds the origins' alone.  Against the FP64
// cross products and division on every step: 92 -> 73 VALU instructions per
// step of the light walk.
template <bool NPAY, bool SHARED>
__device__ inline bool exit_face(const float* tab, const float* dirs, const float (&c)[4], const uint32_t (&w)[4],
                                 const uint32_t (&dn)[4], const uint32_t (&pay)[4], float& bt, uint32_t& bpay) {
  float num[4], q[4], rd[4];
#pragma unroll
  for (int f = 0; f < 4; f++) {  // the four faces' table entries, all read before any is used
    rd[f] = SHARED ? dirs[dn[f]] : tab[dn[f] * kTabRow];
    num[f] = SHARED ? tab[dn[f] * kTabRow] : tab[(kTabDot + dn[f]) * kTabRow];
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int f = 0; f < 4; f++) {
    num[f] = c[f] - num[f];
    const float x = num[f] * rd[f];
    q[f] = (int32_t)(w[f] ^ __float_as_uint(rd[f])) < 0 ? INFINITY : x;
  }
  const float b = fminf(fminf(fminf(q[0], q[1]), q[2]), q[3]);
  const float thr = fmaf(fabsf(b), 0x1p-20f, b);
  // (lane masks in scalar registers: their logic costs no VALU issue)
  const uint64_t m0 = ballot64(q[0] <= thr), m1 = ballot64(q[1] <= thr), m2 = ballot64(q[2] <= thr),
                 m3 = ballot64(q[3] <= thr);
  const uint64_t two = (m0 & m1) | (m2 & m3) | ((m0 | m1) & (m2 | m3));
  const uint64_t fast = ballot64(b > 0x1p-40f) & ~two;
  if (lane_of(fast)) {
    float n = num[0];
    bpay = pay[0];
    uint32_t bn = dn[0];
    n = lane_of(m1) ? num[1] : n;
    n = lane_of(m2) ? num[2] : n;
    n = lane_of(m3) ? num[3] : n;
    bpay = lane_of(m1) ? pay[1] : bpay;
    bpay = lane_of(m2) ? pay[2] : bpay;
    bpay = lane_of(m3) ? pay[3] : bpay;
    if constexpr (NPAY) {
      bn = bits27_30(bpay);
    } else {
      bn = lane_of(m1) ? dn[1] : bn;
      bn = lane_of(m2) ? dn[2] : bn;
      bn = lane_of(m3) ? dn[3] : bn;
    }
    const float r = SHARED ? dirs[bn] : tab[bn * kTabRow], den = SHARED ? dirs[9 + bn] : tab[(kTabDen + bn) * kTabRow];
    const float q1 = fmaf(fmaf(-b, den, n), r, b);
    bt = fmaf(fmaf(-q1, den, n), r, q1);
    return true;
  }
  bool any = false;
  float bnum = 0.0f, bden = 1.0f;
  bpay = 0;
#pragma unroll
  for (int f = 0; f < 4; f++) {
    const uint32_t sg = w[f] & 0x80000000u;
    const float td = SHARED ? dirs[9 + dn[f]] : tab[(kTabDen + dn[f]) * kTabRow];
    const float den = __uint_as_float(__float_as_uint(td) ^ sg);
    const float nf = __uint_as_float(__float_as_uint(num[f]) ^ sg);
    const bool cand = den > 0.0f;
    const bool better = cand && (!any || (double)nf * (double)bden < (double)bnum * (double)den);
    bnum = better ? nf : bnum;
    bden = better ? den : bden;
    bpay = better ? pay[f] : bpay;
    any = any || cand;
  }
  bt = bnum / bden;
  return any;
}

struct TetMedium {
  static constexpr float kOriginScale = 1.0f;
  static constexpr int kRows = kTabRows;  // rows of the segment's LDS table
  static constexpr bool kTet = true;
  static constexpr bool kTight = false;  // the majorant may exceed the extinction
  const TetRec* __restrict__ rec;
  const uint64_t* __restrict__ keys;
  int64_t n;
  int dmax;
  const uint32_t* __restrict__ shapes;
  const uint32_t* __restrict__ kidx;
  int kbits;
  __device__ inline int64_t locate(float3 p) const { return locate_point(keys, kidx, kbits, dmax, shapes, p); }
  __device__ inline float sigma_at(uint32_t cell) const { return rec[cell].sigma; }
  __device__ inline uint32_t most_cells() const { return (uint32_t)n; }  // a straight walk meets
  // Exit of the tet along the segment whose table is `tab`, from t.
  template <bool SHARED = false>
  __device__ inline Step step(uint32_t cell, float3, float3, const float* tab, float t, const float* dirs = nullptr) const {
    const float4* q = (const float4*)(rec + cell);
    const float4 r0 = q[0], r1 = q[1], r2 = q[2];
    const uint32_t codes = __float_as_uint(r2.x);
    const float c[4] = {r0.x, r0.y, r0.z, r0.w};
    const uint32_t link[4] = {__float_as_uint(r1.x), __float_as_uint(r1.y), __float_as_uint(r1.z),
                              __float_as_uint(r1.w)};
    uint32_t w[4], dn[4];
#pragma unroll
    for (int f = 0; f < 4; f++) {
      w[f] = codes << (31 - 8 * f);
      dn[f] = (codes >> (8 * f + 1)) & 0x7Fu;
    }
    float bt;
    uint32_t blink;
    Step s;
    s.ok = exit_face<false, SHARED>(tab, dirs, c, w, dn, link, bt, blink);
    s.sigma = r2.y;
    s.majorant = r2.z;
    s.te = bt > t ? bt : t;
    s.next = (!s.ok || blink == kBoundary) ? -1 : (int32_t)(blink >> 2);
    return s;
  }
};

// Same walk on the compact 32-byte records (bitwise the same values).  The
// LDS table holds origin dots scaled by 2^20 (exact), so the integer
// plane constants need no scaling: num * 2^20 = c - dot * 2^20 exactly, and
// one final multiply by 2^-20 (exact) gives the exit distance.
struct TetMedium32 {
  static constexpr float kOriginScale = 0x1p20f;  // origin dots stored times 2^20
  static constexpr int kRows = kTabRows;
  static constexpr bool kTet = true;
  static constexpr bool kTight = true;            // the majorant is the extinction
  const TetRec32* __restrict__ rec;
  const uint64_t* __restrict__ keys;
  int64_t n;
  int dmax;
  const uint32_t* __restrict__ shapes;
  const uint32_t* __restrict__ kidx;
  int kbits;
  __device__ inline int64_t locate(float3 p) const { return locate_point(keys, kidx, kbits, dmax, shapes, p); }
  __device__ inline float sigma_at(uint32_t cell) const { return __uint_as_float(rec[cell].w[3]); }
  __device__ inline uint32_t most_cells() const { return (uint32_t)n; }
  template <bool SHARED = false>
  __device__ inline Step step(uint32_t cell, float3, float3, const float* tab, float t, const float* dirs = nullptr) const {
    // byte offset in 32 bits (cell < 2^27): a uniform base takes the load's
    // scalar-base form
    const uint4* q = (const uint4*)((const char*)rec + (cell << 5));
    const uint4 a = q[0], b = q[1];
    const uint32_t o1 = (uint32_t)((((uint64_t)a.y << 32) | a.x) >> 23);
    const uint32_t o2 = (uint32_t)((((uint64_t)a.z << 32) | a.y) >> 14);
    const float c[4] = {(float)(((int32_t)(a.x << 9)) >> 9), (float)(((int32_t)(o1 << 9)) >> 9),
                        (float)(((int32_t)(o2 << 9)) >> 9), (float)(((int32_t)(a.z << 4)) >> 9)};
    const uint32_t lw[4] = {b.x, b.y, b.z, b.w};
    uint32_t dn[4];
#pragma unroll
    for (int f = 0; f < 4; f++) dn[f] = bits27_30(lw[f]);
    float bt;
    uint32_t bw;
    Step s;
    s.ok = exit_face<true, SHARED>(tab, dirs, c, lw, dn, lw, bt, bw);
    const uint32_t blink = bw & kLink27Boundary;
    bt = bt * 0x1p-20f;
    s.sigma = __uint_as_float(a.w);
    s.majorant = s.sigma;
    s.te = bt > t ? bt : t;
    s.next = (!s.ok || blink == kLink27Boundary) ? -1 : (int32_t)blink;
    return s;
  }
};

// ---------------------------------------------------------------- voxel medium
// Voxels of an n^3 grid, n = 2^sh.  A step leaves by the axis with the smallest
// correctly rounded distance (plane - o) / d, the lowest axis on ties; as in
// exit_face, reciprocal products find it and give the rounded quotient where
// no other axis is near, and the divisions are left to the rest.  Bound by
// VALU issue: with three IEEE divisions and four integer ones per step the
// 512^2 x 16 frame of a 256^3 volume took 11.8 ms, now 7.2 ms.
struct VoxelMedium {
  static constexpr float kOriginScale = 1.0f;
  static constexpr int kRows = 3;  // LDS table: the reciprocals of d alone (seg_dirs r[0..2])
  static constexpr bool kTet = false;
  static constexpr bool kTight = true;
  const float* __restrict__ dens;
  int32_t n;
  float scale;
  int32_t sh;
  float inv;  // 1 / n
  __device__ inline int64_t locate(float3 p) const {
    float c[3] = {p.x, p.y, p.z};
    int64_t idx[3];
#pragma unroll
    for (int a = 0; a < 3; a++) {
      int64_t i = (int64_t)floorf(c[a] * (float)n);
      idx[a] = i < 0 ? 0 : (i >= n ? n - 1 : i);
    }
    return idx[0] + n * (idx[1] + (int64_t)n * idx[2]);
  }
  __device__ inline float sigma_at(uint32_t cell) const { return scale * dens[cell]; }
  __device__ inline uint32_t most_cells() const { return 3u * (uint32_t)n; }
  template <bool SHARED = false>
  __device__ inline Step step(uint32_t cell, float3 o, float3 d, const float* tab, float t,
                              const float* dirs = nullptr) const {
    const float v = scale * dens[cell];
    const uint32_t last = (uint32_t)n - 1u;
    const uint32_t idx[3] = {cell & last, (cell >> sh) & last, cell >> (2 * sh)};
    const float oo[3] = {o.x, o.y, o.z}, dd[3] = {d.x, d.y, d.z};
    float num[3], r[3], q[3];
#pragma unroll
    for (int a = 0; a < 3; a++) {
      r[a] = SHARED ? dirs[a] : tab[a * kTabRow];
      num[a] = (float)(idx[a] + (dd[a] > 0.0f ? 1u : 0u)) * inv - oo[a];  // (the plane is exact)
      q[a] = num[a] * r[a];
    }
    const float b = fminf(fminf(q[0], q[1]), q[2]);
    const float thr = fmaf(fabsf(b), 0x1p-20f, b);
    const uint64_t m0 = ballot64(q[0] <= thr), m1 = ballot64(q[1] <= thr), m2 = ballot64(q[2] <= thr);
    const uint64_t fast = ballot64(b > 0x1p-40f) & ~((m0 & m1) | (m2 & (m0 | m1)));
    float bt, bd = dd[0];
    uint32_t at = idx[0], stride = 1u;
    Step s;
    s.ok = true;
    if (lane_of(fast)) {
      bd = lane_of(m1) ? dd[1] : bd;
      bd = lane_of(m2) ? dd[2] : bd;
      float bn = lane_of(m1) ? num[1] : num[0], br = lane_of(m1) ? r[1] : r[0];
      bn = lane_of(m2) ? num[2] : bn;
      br = lane_of(m2) ? r[2] : br;
      at = lane_of(m1) ? idx[1] : at;
      at = lane_of(m2) ? idx[2] : at;
      stride = lane_of(m1) ? (uint32_t)n : stride;
      stride = lane_of(m2) ? (uint32_t)n * (uint32_t)n : stride;
      const float q1 = fmaf(fmaf(-b, bd, bn), br, b);
      bt = fmaf(fmaf(-q1, bd, bn), br, q1);
    } else {
      s.ok = false;
      bt = 0.0f;
#pragma unroll
      for (int a = 0; a < 3; a++) {
        const float tf = num[a] / dd[a];
        const bool better = dd[a] != 0.0f && (!s.ok || tf < bt);
        bt = better ? tf : bt;
        bd = better ? dd[a] : bd;
        at = better ? idx[a] : at;
        stride = better ? (a == 0 ? 1u : (a == 1 ? (uint32_t)n : (uint32_t)n * (uint32_t)n)) : stride;
        s.ok = s.ok || dd[a] != 0.0f;
      }
    }
    s.sigma = v;
    s.majorant = v;
    s.te = bt > t ? bt : t;
    const bool up = bd > 0.0f;
    s.next = !s.ok || at == (up ? last : 0u) ? -1 : (int32_t)(up ? cell + stride : cell - stride);
    return s;
  }
};

// ---------------------------------------------------------------- camera
__device__ inline bool enter_cube(float3 o, float3 d, float3& p) {
  const float oo[3] = {o.x, o.y, o.z}, dd[3] = {d.x, d.y, d.z};
  float tn = -INFINITY, tf = INFINITY;
  int axis = -1;
#pragma unroll
  for (int a = 0; a < 3; a++) {
    if (dd[a] == 0.0f) {
      if (oo[a] < 0.0f || oo[a] > 1.0f) return false;
      continue;
    }
    float inv = 1.0f / dd[a];
    float ta = (0.0f - oo[a]) * inv, tb = (1.0f - oo[a]) * inv;
    float lo = ta < tb ? ta : tb, hi = ta < tb ? tb : ta;
    if (lo > tn) {
      tn = lo;
      axis = a;
    }
    if (hi < tf) tf = hi;
  }
  if (tn > tf || tf <= 0.0f) return false;
  float te = tn > 0.0f ? tn : 0.0f;
  float r[3];
#pragma unroll
  for (int a = 0; a < 3; a++) {
    float v = oo[a] + te * dd[a];
    v = v < 0.0f ? 0.0f : v;
    v = v > 1.0f ? 1.0f : v;
    r[a] = v;
  }
  if (tn > 0.0f && axis >= 0) {
    float fv = dd[axis] > 0.0f ? 0.0f : 1.0f;
    if (axis == 0) r[0] = fv;
    else if (axis == 1) r[1] = fv;
    else r[2] = fv;
  }
  p = make_float3(r[0], r[1], r[2]);
  return true;
}

// ---------------------------------------------------------------- kernels
// Camera ray (direction d) of sample s of pixel (px, py), its entry p into
// the grid and the entry tet (-1: it misses the grid).
template <class Med>
__device__ inline int64_t camera_entry(const Frame& fr, uint64_t seed, const Med& med, int32_t px, int32_t py,
                                       uint32_t pix, uint32_t s, float3& p, float3& d) {
  uint2 u = uniform01x2(seed, pix, s, 0, kStreamCamera, 0);
  float u0 = u01(u.x), u1 = u01(u.y);
  float sx = ((2.0f * (((float)px + u0) / (float)fr.w)) - 1.0f) * fr.tan_x;
  float sy = (1.0f - 2.0f * (((float)py + u1) / (float)fr.h)) * fr.tan_y;
  float3 o = make_float3(fr.pos[0], fr.pos[1], fr.pos[2]);
  d = normalize3(make_float3((fr.f[0] + sx * fr.r[0]) + sy * fr.u[0], (fr.f[1] + sx * fr.r[1]) + sy * fr.u[1],
                             (fr.f[2] + sx * fr.r[2]) + sy * fr.u[2]));
  p = o;
  return enter_cube(o, d, p) ? med.locate(p) : -1;
}

// Sum of n finished entry records in sample order, four loads at a time (a
// 128-byte line holds four records).
__device__ inline float3 sum_samples(const RayEntry* __restrict__ q, int32_t n) {
  float3 a = make_float3(0, 0, 0);
  int32_t k = 0;
  for (; k + 4 <= n; k += 4) {
    float4 v[4];
#pragma unroll
    for (int j = 0; j < 4; j++) v[j] = *(const float4*)(q + k + j);
#pragma unroll
    for (int j = 0; j < 4; j++) a = make_float3(a.x + v[j].x, a.y + v[j].y, a.z + v[j].z);
  }
  for (; k < n; k++) {
    const float4 v = *(const float4*)(q + k);
    a = make_float3(a.x + v.x, a.y + v.y, a.z + v.z);
  }
  return a;
}

// The pass's samples summed per pixel (thread = slot).  mode 0: the image's
// only contribution, divided by the samples; 1: the first of several; 2: one
// more of them.
__global__ __launch_bounds__(256) void k_resolve(RenderArgs A, int mode) {
  const uint32_t slot = blockIdx.x * blockDim.x + threadIdx.x;
  int32_t px, py;
  if (slot >= A.slots || !slot_pixel(slot, A.tiles_x, A.fr.w, A.fr.h, px, py)) return;
  const float3 a = sum_samples(A.entries + (size_t)slot * (uint32_t)A.pass_spp, A.pass_spp);
  float* o = A.out + 3 * ((size_t)py * (uint32_t)A.fr.w + (uint32_t)px);
  if (mode == 0) {
    const float div = (float)A.spp;
    o[0] = a.x / div;
    o[1] = a.y / div;
    o[2] = a.z / div;
  } else if (mode == 1) {
    o[0] = a.x;
    o[1] = a.y;
    o[2] = a.z;
  } else {
    o[0] = o[0] + a.x;
    o[1] = o[1] + a.y;
    o[2] = o[2] + a.z;
  }
}

// The same for a batch of scenes: every pixel of every image.
__global__ __launch_bounds__(256) void k_resolve_batch(RenderArgs A, uint64_t total_px) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total_px) return;
  const SceneDesc& S = A.scenes[scene_search(A.nscenes, i, [&](int j) { return A.scenes[j].pix0; })];
  const uint32_t p = (uint32_t)(i - S.pix0), x = p % (uint32_t)S.fr.w, y = p / (uint32_t)S.fr.w;
  const uint32_t slot = ((y >> 3) * (uint32_t)S.tiles_x + (x >> 3)) * 64u + (y & 7u) * 8u + (x & 7u);
  const float3 a = sum_samples(A.entries + S.entry0 + (uint64_t)slot * (uint32_t)S.spp, S.spp);
  const float div = (float)S.spp;
  float* o = S.out + 3 * (size_t)p;
  o[0] = a.x / div;
  o[1] = a.y / div;
  o[2] = a.z / div;
}

enum { M_TRACK = 0, M_SHADOW = 1, M_COLLIDE = 2, M_SCATTER = 3, M_ESCAPE = 4, M_FINISH = 5, M_FETCH = 6,
       M_DONE = 7, M_PARK = 8 };

// Paths a wave takes at least.  At 1, 4, 8, 16 and 64 the frame with a learning
// cache took 2.06, 2.11, 2.15, 2.20 and 2.25 ms (its training paths spread over
// more waves); thumbnail, preview, emissive, cloud and batch frames stay within
// the spread of their runs.
constexpr uint32_t kMinTake = 16;
// Adds each lane's v[0..n) to the block's statistics slot: wave reductions,
// one atomic per wave and counter.
template <int N>
__device__ inline void add_stats(const RenderArgs& A, const uint32_t (&v)[N]) {
#pragma unroll
  for (int q = 0; q < N; q++) {
    unsigned long long x = v[q];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
    if (__lane_id() == 0 && x) atomicAdd(stat_slot(A) + q, x);
  }
}

// Camera rays and their walk to the first real collision, one thread per
// entry record in record order: the samples of a pixel are neighbouring
// lanes, which walk the same tets, so a wave reads a few record lines per step
// and its lanes stay together until they collide or all leave the grid.
// Blocks are dealt to eight lists round-robin, as the hardware deals blocks to
// the XCDs (the lists follow the blocks of an image's training paths, a
// multiple of 8); list r takes chunks r, r + 8, ... of chunk_blocks blocks, so
// that neighbouring rays share an XCD's L2 and every XCD gets its share of
// the image's dense part (one contiguous eighth each left half the XCDs idle
// at the end: 17.4 ms on the 33 M rays of the 1024^2 x 32 cloud frame,
// 2.8 of 5 resident waves per SIMD on average; dealt, 9.5 ms, at the VALU
// issue rate).  A block lists its colliding samples with one atomic on its
// list's count.  MODEL: the grid carries a density model.
template <class Med, bool BATCH, bool MODEL>
__global__ __launch_bounds__(kFirstBlock) void k_first(RenderArgs A, Med med) {
  __shared__ float s_tab[Med::kRows * kFirstBlock];
  float* tab = s_tab + (threadIdx.x >> 6) * (Med::kRows * kTabRow) + (threadIdx.x & 63u);
  const int lane = __lane_id();
  // the first blocks trace the training paths that go with an image
  const uint32_t block = BATCH ? blockIdx.y * gridDim.x + blockIdx.x : blockIdx.x;  // (first_grid: rows in batches only)
  const bool with = !BATCH && block < A.train_blocks, train = with || (!BATCH && A.train);
  const uint32_t blk = block - (with ? 0u : A.train_blocks);
  const uint32_t band = with ? 0u : blk & 7u, j = blk >> 3, g = A.chunk_blocks, round = j / g;
  const uint32_t turn = (band + ((round * 0x9E3779B9u) >> 29)) & 7u;  // (a row of the image may hold a multiple of 8 chunks)
  const uint64_t e = (with ? (uint64_t)blk : ((uint64_t)round * 8u + turn) * g + j % g) * kFirstBlock + threadIdx.x;
  const uint64_t total = BATCH ? A.total_entries : (with ? A.train_items : (uint64_t)A.slots * (uint64_t)A.pass_spp);
  RayEntry* const entries = A.entries + (with ? A.train_ent0 : 0u);
  uint32_t n_stat[5] = {0, 0, 0, 0, 0};  // steps, null collisions, real collisions, escapes, truncated
  bool hit = false;
  if (e < total) {
    // the sample
    uint32_t pix = 0, smp;
    int32_t px, py, sc = 0;
    bool real_pixel = true;
    uint64_t seed = with ? A.train_seed : A.seed;
    if constexpr (BATCH) {
      sc = scene_search(A.nscenes, e, [&](int i) { return A.scenes[i].entry0; });
      const SceneDesc& S = A.scenes[sc];
      const uint64_t l = e - S.entry0;
      smp = S.s0 + (uint32_t)(l % (uint32_t)S.spp);
      real_pixel = slot_pixel((uint32_t)(l / (uint32_t)S.spp), S.tiles_x, S.fr.w, S.fr.h, px, py);
      pix = (uint32_t)(py * S.fr.w + px);
      seed = S.seed;
    } else if (train) {
      smp = (uint32_t)e;
      pix = train_pixel(seed, smp, A.npix);
      px = (int32_t)(pix % (uint32_t)A.fr.w);
      py = (int32_t)(pix / (uint32_t)A.fr.w);
    } else {
      smp = (uint32_t)(A.pass_start + (int32_t)(e % (uint32_t)A.pass_spp));
      real_pixel = slot_pixel((uint32_t)(e / (uint32_t)A.pass_spp), A.tiles_x, A.fr.w, A.fr.h, px, py);
      pix = (uint32_t)(py * A.fr.w + px);
    }
    if (!real_pixel) {  // a padding slot of an edge tile
      if (A.chain) entries[e].cell = kDone;
    } else {
      Med m = med;
      if constexpr (BATCH) {
        const SceneDesc& S = A.scenes[sc];
        m.rec = (decltype(m.rec))S.rec;
        m.keys = S.keys;
        m.kidx = S.kidx;
        m.kbits = S.kbits;
        m.n = S.n;
        m.dmax = S.dmax;
      }
      float3 o, d;
      const int64_t c = camera_entry(BATCH ? A.scenes[sc].fr : A.fr, seed, m, px, py, pix, smp, o, d);
      float3 L = make_float3(BATCH ? A.scenes[sc].env[0] : A.env[0], BATCH ? A.scenes[sc].env[1] : A.env[1],
                             BATCH ? A.scenes[sc].env[2] : A.env[2]);
      uint32_t steps = 0, cell = (uint32_t)c;
      float t = 0.0f;
      if (c >= 0) {
        float tau = exp_tau(uniform01(seed, pix, smp, 0, kStreamFlight, 0));
        uint32_t jf = 1;  // flight draw 0 made tau
        set_segment<Med>(tab, o, d);
        for (;;) {
          Step st;
          float sb, dtau;
          bool out, cut;
          for (;;) {  // cells without a tentative collision
            cut = steps >= A.max_steps;
            if (cut) break;
            st = m.step(cell, o, d, tab, t);
            steps++;
            sb = st.majorant;
            dtau = sb * (st.te - t);  // (0 in an empty cell)
            out = !st.ok || st.next < 0;
            if (out || tau < dtau) break;
            tau = tau - dtau;
            t = st.te;
            cell = (uint32_t)st.next;
          }
          if (cut) {  // a truncated path keeps what it has gathered: nothing
            n_stat[4] = 1;
            L = make_float3(0, 0, 0);
            break;
          }
          if (st.ok) {
            while (tau < dtau) {
              const float tc = t + tau / sb;
              float sg = st.sigma;
              if constexpr (MODEL) {  // extinction at the tentative point
                const ExtArgs& X = BATCH ? A.scenes[sc].ex : A.ex;
                if (X.model) sg = model_sigma(X, cell, o, d, tc);
              }
              t = tc;
              if ((Med::kTight && !MODEL) || !(sg < sb) ||
                  uniform01(seed, pix, smp, 0, kStreamFlight, jf++) < sg / sb) {
                hit = true;
                break;
              }
              n_stat[1]++;
              tau = exp_tau(uniform01(seed, pix, smp, 0, kStreamFlight, jf++));
              dtau = sb * (st.te - t);
            }
            if (hit) break;
          }
          if (out) {
            n_stat[3] = 1;
            break;
          }
          tau = tau - dtau;
          t = st.te;
          cell = (uint32_t)st.next;
        }
      }
      float4* q = (float4*)(entries + e);
      if (hit) {
        q[0] = make_float4(o.x + t * d.x, o.y + t * d.y, o.z + t * d.z, __uint_as_float(cell));
        q[1] = make_float4(d.x, d.y, d.z, __uint_as_float(steps));
      } else {
        n_stat[0] = steps;
        q[0] = make_float4(L.x, L.y, L.z, __uint_as_float(kDone));
        if (train) A.path_l[e] = make_float4(L.x, L.y, L.z, __uint_as_float(0u));
      }
    }
  }
  const unsigned long long m = __ballot(hit);
  if (m) {
    uint32_t base = 0;
    if (lane == 0) base = atomicAdd(A.head + kCountAt + (with ? kTrainList : (int)band) * kLine, (uint32_t)__popcll(m));
    base = __shfl(base, 0);
    if (hit)
      A.list[(with ? (uint64_t)A.train_list0 : (uint64_t)band * A.band_size) + base +
             (uint32_t)__popcll(m & ((1ull << lane) - 1ull))] = (uint32_t)e;
  }
  add_stats(A, n_stat);
}

// The listed paths, from their first real collision on.
// W: occupancy target in waves per SIMD (the register budget follows).
// NRC: 0 plain estimator; 1 paths stop at real vertex A.truncate and leave
// a query for the radiance cache; 2 training paths (A.train), whose first
// vertices and final radiance are recorded.
// BATCH: the lanes' samples come from a batch of scenes (A.scenes); each
// lane keeps its sample's scene index and that grid's record pointer, and
// reads the scene's light, medium, seed and image from the table at events.
// EXT: the variant that reads the extra channels and the density model
// (the plain variant carries none of that code).
template <class Med, int W, int NRC, bool BATCH = false, bool EXT = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(W, 8))) void k_render(RenderArgs A, Med med) {
  __shared__ float s_tab[Med::kRows * 256];
  // per wave: its queue chunk's first record, records used, light rays queued
  // (volatile: different lanes of the wave read and write them in turn)
  __shared__ volatile uint32_t s_lq[4][3];
  // A.chain: the latest queue record of the lane's path (rarely read: no register)
  __shared__ uint32_t s_last[256];
  uint32_t& last = s_last[threadIdx.x];
  last = kDone;
  float* tab = s_tab + (threadIdx.x >> 6) * (Med::kRows * kTabRow) + (threadIdx.x & 63u);
  const int lane = __lane_id();
  int mode = M_FETCH;
  uint32_t pix = 0, ent = 0;  // ent: the sample's entry record
  int32_t s = 0;
  float3 o = make_float3(0, 0, 0), d = o, dsave = o, L = o;
  float beta = 1.0f, t = 0.0f, tau = 0.0f, od = 0.0f;
  uint32_t cell = 0, cell_x = 0, bounce = 0, jf = 0, jn = 0, steps = 0;
  uint32_t n_steps = 0, n_null = 0, n_real = 0, n_esc = 0, n_trunc = 0, n_query = 0;
  // wave-uniform list state: training paths first (they are the longest),
  // then this block's band, then the others
  const int list0 = NRC == 1 && A.train_items ? kTrainList : (int)(blockIdx.x & 7), nlists = NRC == 1 && A.train_items ? 9 : 8;
  const uint32_t list_waves = max(1u, gridDim.x * (blockDim.x >> 6) / 8u);  // waves per band
  int range = list0, tried = 0;
  uint32_t bnext = 0, bend = 0;  // wave-uniform batch of listed paths
  uint32_t sc = 0;           // the lane's scene
  bool trainp = false;       // cache mode 1: the lane's path is a training path
  Med lm = med;              // the lane's medium (its scene's records)
  const int wv = threadIdx.x >> 6;
  {
    if (lane < 3) s_lq[wv][lane] = lane == 1 ? A.lq_chunk : 0u;  // a full chunk: the first ray takes one
    __builtin_amdgcn_wave_barrier();
  }
#define TV_SC A.scenes[sc]
#define TV_SEED (BATCH ? TV_SC.seed : ((NRC == 1 && trainp) ? A.train_seed : A.seed))
#define TV_ALBEDO (BATCH ? TV_SC.albedo : A.albedo)
#define TV_G (BATCH ? TV_SC.g : A.g)
#define TV_E(i) (BATCH ? TV_SC.E[i] : A.E[i])
#define TV_ENV(i) (BATCH ? TV_SC.env[i] : A.env[i])
#define TV_SUN (BATCH ? make_float3(TV_SC.sun[0], TV_SC.sun[1], TV_SC.sun[2]) : make_float3(A.sun[0], A.sun[1], A.sun[2]))
#define TV_EX (BATCH ? TV_SC.ex : A.ex)

  // extinction at the collision o + t d, the cache's input there: the
  // tet's, or the density model's at the point
  auto vertex_sigma = [&]() -> float {
    if constexpr (EXT)
      if (TV_EX.model) return model_sigma(TV_EX, cell, o, d, t);
    return lm.sigma_at(cell);
  };
  // training paths whose light rays are queued leave each vertex's gathered
  // radiance in A.terms (their records need what came before each vertex)
  auto termed = [&]() -> bool { return (NRC == 2 || (NRC == 1 && trainp)) && A.terms; };
  auto term_index = [&]() -> uint32_t {
    return (NRC == 2 ? ent : ent - A.train_ent0) * (uint32_t)A.max_bounces + (bounce - 1u);
  };
  // real collision at t: start the light ray (right after the walk step, or
  // from the event section for the collisions where a path hands over to the
  // radiance cache)
  auto start_light = [&]() {
    float3 x = make_float3(o.x + t * d.x, o.y + t * d.y, o.z + t * d.z);
    uint32_t at = kDone;  // the light ray's place in the queue
    if (A.defer && !(NRC == 1 && trainp && !A.terms)) {
      const unsigned long long act = __ballot(1);
      const int lead = __builtin_ctzll(act);
      const uint32_t cnt = (uint32_t)__popcll(act), k = (uint32_t)__popcll(act & ((1ull << lane) - 1ull));
      uint32_t base = 0, room = 0, next = 0, used = 0;
      if (lane == lead) {
        base = s_lq[wv][0];
        used = s_lq[wv][1];  // kDone: the queue is full
        room = used == kDone ? 0u : A.lq_chunk - used;
        next = kDone;
        uint32_t left = cnt > room ? kDone : used + cnt;
        if (cnt > room && used != kDone) {
          const uint32_t c = atomicAdd(A.head + kChunkAt, 1u);
          if (c < A.lq_chunks) {
            next = c * A.lq_chunk;
            s_lq[wv][0] = next;
            left = cnt - room;
          }
        }
        s_lq[wv][1] = left;
        s_lq[wv][2] = s_lq[wv][2] + (next != kDone ? cnt : min(cnt, room));
      }
      base = __shfl(base, lead) + __shfl(used, lead);
      room = __shfl(room, lead);
      next = __shfl(next, lead);
      if (k < room || next != kDone) {
        at = k < room ? base + k : next + (k - room);
      } else if (NRC != 2 && A.chain && !(NRC == 1 && trainp)) {
        // a full queue: the path waits (without A.chain its lane walks the ray)
        RayEntry* e = A.entries + ent;
        *(float4*)e = make_float4(x.x, x.y, x.z, __uint_as_float(cell));
        e->dx = d.x;
        e->dy = d.y;
        e->dz = d.z;
        if (last == kDone) e->steps = kDone;
        last = kDone;
        n_steps += steps;
        mode = M_FETCH;
        return;
      }
    }
    n_real++;
    bounce++;
    if ((NRC == 2 || (NRC == 1 && trainp)) && (int32_t)bounce <= A.rec_vertices) {
      uint32_t j = NRC == 2 ? ent : ent - A.train_ent0;
      float4* q = A.vrec + ((size_t)j * (uint32_t)A.rec_vertices + (bounce - 1)) * 3;
      q[0] = make_float4(x.x, x.y, x.z, vertex_sigma());
      q[1] = make_float4(d.x, d.y, d.z, beta);
      q[2] = make_float4(L.x, L.y, L.z, 0.0f);
    }
    jf = 0;
    jn = 0;
    // extra channels of the collision's tet: the emitted radiance by
    // the collision estimator (absorbed part of the collision), then the
    // tet's albedo in place of the medium's
    float alb = TV_ALBEDO;
    if (EXT && TV_EX.ch_a) alb = TV_EX.ch_a[cell];
    if (EXT && TV_EX.ch_t && !(A.chain && at != kDone && !termed())) {  // (a chain's: k_chain)
      const float e = (1.0f - alb) * TV_EX.ch_t[cell];
      const float3 em = make_float3(beta * (e * TV_EX.emission[0]), beta * (e * TV_EX.emission[1]),
                                    beta * (e * TV_EX.emission[2]));
      if (NRC != 0 && termed()) {
        A.terms[2 * (size_t)term_index() + 1] = make_float4(em.x, em.y, em.z, 0.0f);
      } else {
        L.x = L.x + em.x;
        L.y = L.y + em.y;
        L.z = L.z + em.z;
      }
    }
    beta = beta * alb;
    if (at != kDone) {
      // queue the light ray (weight now, walk later); the path goes on to its
      // scatter
      const float gg = (EXT && TV_EX.ch_g) ? TV_EX.ch_g[cell] : TV_G;
      const float3 sun = TV_SUN;
      const float mu = (d.x * sun.x + d.y * sun.y) + d.z * sun.z;
      LightRec r;
      r.x = x.x;
      r.y = x.y;
      r.z = x.z;
      r.cell = cell;
      r.bp = beta * hg_pdf(gg, mu);
      r.to = A.chain ? ent : pix;
      r.next = kDone;
      r.bounce = bounce;
      if (NRC != 0 && termed()) {
        r.to = term_index();
        r.bounce |= kToTerm;
      } else if (A.chain) {
        *(last == kDone ? &A.entries[ent].steps : &A.lq[last].next) = at;
        last = at;
      }
      A.lq[at] = r;
      dsave = d;
      o = x;
      t = 0.0f;
      cell_x = cell;
      od = -1.0f;  // no light term at the scatter
      mode = M_SCATTER;
      return;
    }
    dsave = d;
    o = x;
    d = TV_SUN;
    t = 0.0f;
    cell_x = cell;
    od = A.transmittance == 0 ? 0.0f : 1.0f;
    if (A.transmittance != 0) tau = exp_tau(uniform01(TV_SEED, pix, (uint32_t)s, bounce, kStreamLight, jn++));
    set_segment<Med>(tab, o, d);
    mode = M_SHADOW;
  };

  for (;;) {
    // ================= events: run when enough lanes wait (those out of work
    // count), or when no lane is walking (waiting lanes idle meanwhile)
    const unsigned long long walking = __ballot(mode <= M_SHADOW);
    const unsigned long long pending = __ballot(mode > M_SHADOW && mode < M_DONE);
    if (!(walking | pending)) break;
    if (pending && (64 - __popcll(walking) >= A.event_wait || !walking)) {
      if (NRC == 1) {  // the cache stands for the rest of the path: append a query
        const bool isq = mode == M_COLLIDE && !trainp && (int32_t)bounce + 1 == A.truncate;
        const unsigned long long qm = __ballot(isq);
        if (qm) {
          const int lead = __builtin_ctzll(qm);
          uint32_t base = 0;
          if (lane == lead) base = atomicAdd(A.qcount, (uint32_t)__popcll(qm));
          base = __shfl(base, lead);
          if (isq) {
            const uint32_t q = base + (uint32_t)__popcll(qm & ((1ull << lane) - 1ull));
            n_real++;
            bounce++;
            float3 x = make_float3(o.x + t * d.x, o.y + t * d.y, o.z + t * d.z);
            A.qbuf[2 * (size_t)q] = make_float4(x.x, x.y, x.z, vertex_sigma());
            A.qbuf[2 * (size_t)q + 1] = make_float4(d.x, d.y, d.z, beta);
            A.qpix[q] = pix;
            n_query++;
            mode = M_FINISH;
          }
        }
      }
      if (mode == M_ESCAPE) {  // left the grid: the environment
        n_esc++;
        L.x = L.x + beta * TV_ENV(0);
        L.y = L.y + beta * TV_ENV(1);
        L.z = L.z + beta * TV_ENV(2);
        mode = M_FINISH;
      }
      if (mode == M_FINISH) {  // path done: its sample's radiance
        n_steps += steps;
        *(float4*)(A.entries + ent) = make_float4(L.x, L.y, L.z, __uint_as_float(last == kDone ? kDone : kChained));
        last = kDone;
        if (NRC == 2 || (NRC == 1 && trainp))
          A.path_l[NRC == 2 ? ent : ent - A.train_ent0] = make_float4(L.x, L.y, L.z, __uint_as_float(bounce));
        mode = M_FETCH;
      }
      // idle lanes take consecutive listed paths from the wave's batch; a
      // wave refills its batch with one atomic, first from this block's list
      // (blocks are dealt to the 8 XCDs round-robin, so an XCD's L2 serves
      // the chunks of the image that its own blocks listed), then from the others.
      // A wave with training paths takes no others until they end: they are
      // the longest, and among image paths each of their events would wait
      // for the wave's others (cache frame of 16 K training paths: 2.34 ms
      // mixed, 2.30 ms apart).
      const bool hold = NRC == 1 && nlists == kLists && __ballot(trainp && mode <= M_ESCAPE);
      if (NRC == 1 && !hold && mode == M_PARK) mode = M_FETCH;
      bool need = mode == M_FETCH;
      unsigned long long m = __ballot(need);
      if (m) {
        while (bnext >= bend && tried < (hold ? 1 : nlists)) {
          const uint32_t n = A.head[kCountAt + range * kLine];
          const uint32_t take = min(A.batch, max(kMinTake, n / (range == kTrainList ? 8 * list_waves : list_waves)));
          uint32_t base = 0;
          if (lane == 0) base = n ? atomicAdd(A.head + kTakenAt + range * kLine, take) : 0u;
          base = __shfl(base, 0);
          if (base < n) {
            bnext = base;
            bend = min(base + take, n);
          } else {  // list drained: move on
            range = NRC == 1 && range == kTrainList ? (int)(blockIdx.x & 7) : (range + 1) & 7;
            tried++;
          }
        }
        if (bnext < bend) {
          const uint32_t at = bnext + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
          if (need && at < bend) {  // the path's first collision
            const bool tr = NRC == 1 && range == kTrainList;
            const uint32_t e = A.list[(tr ? (uint64_t)A.train_list0 : (uint64_t)(uint32_t)range * A.band_size) + at];
            if constexpr (BATCH) {
              sc = (uint32_t)scene_search(A.nscenes, e, [&](int i) { return A.scenes[i].entry0; });
              const SceneDesc& S = A.scenes[sc];
              const uint32_t local = (uint32_t)(e - S.entry0);
              int32_t px, py;
              (void)slot_pixel(local / (uint32_t)S.spp, S.tiles_x, S.fr.w, S.fr.h, px, py);
              pix = (uint32_t)(py * S.fr.w + px);
              s = (int32_t)(S.s0 + local % (uint32_t)S.spp);
              lm.rec = (decltype(lm.rec))S.rec;
              ent = e;
            } else if (NRC == 2 || tr) {
              pix = train_pixel(NRC == 2 ? A.seed : A.train_seed, e, A.npix);
              s = (int32_t)e;
              ent = NRC == 2 ? e : A.train_ent0 + e;
              trainp = NRC == 1;
            } else {
              int32_t px, py;
              (void)slot_pixel(e / (uint32_t)A.pass_spp, A.tiles_x, A.fr.w, A.fr.h, px, py);
              pix = (uint32_t)(py * A.fr.w + px);
              s = A.pass_start + (int32_t)(e % (uint32_t)A.pass_spp);
              ent = e;
              trainp = false;
            }
            const float4* q = (const float4*)(A.entries + ent);
            const float4 a = q[0], b = q[1];
            o = make_float3(a.x, a.y, a.z);
            d = make_float3(b.x, b.y, b.z);
            cell = __float_as_uint(a.w);
            steps = __float_as_uint(b.w);
            t = 0.0f;
            beta = 1.0f;
            L = make_float3(0, 0, 0);
            bounce = 0;
            if (A.resume) {  // what k_chain left at the path's first queue record
              if (steps != kDone) {
                const LightRec r = A.lq[steps];
                L = make_float3(r.x, r.y, r.z);
                beta = r.bp;
                bounce = r.bounce;
              }
              steps = 0;
            }
            mode = M_COLLIDE;
          }
          bnext = min(bnext + (uint32_t)__popcll(m), bend);
        } else if (need) {
          mode = hold ? M_PARK : M_DONE;
        }
      }
      if (mode == M_COLLIDE && (NRC != 1 || trainp || (int32_t)bounce + 1 != A.truncate)) start_light();
      if (mode == M_SCATTER) {  // light ray done: light estimate, then phase sampling
        const float gg = (EXT && TV_EX.ch_g) ? TV_EX.ch_g[cell_x] : TV_G;  // the collision tet's phase parameter
        if (od >= 0.0f) {  // (od < 0: the light ray was queued)
          float Tr = A.transmittance == 0 ? exp_neg(od) : od;
          float mu = (dsave.x * TV_SUN.x + dsave.y * TV_SUN.y) + dsave.z * TV_SUN.z;
          float ph = hg_pdf(gg, mu);
          const float3 li = make_float3(((beta * ph) * TV_E(0)) * Tr, ((beta * ph) * TV_E(1)) * Tr,
                                        ((beta * ph) * TV_E(2)) * Tr);
          if (NRC != 0 && termed()) {
            A.terms[2 * (size_t)term_index()] = make_float4(li.x, li.y, li.z, 0.0f);
          } else {
            L.x = L.x + li.x;
            L.y = L.y + li.y;
            L.z = L.z + li.z;
          }
        }
        if ((int32_t)bounce >= A.max_bounces) {
          mode = M_FINISH;
        } else {
          uint2 v = uniform01x2(TV_SEED, pix, (uint32_t)s, bounce, kStreamPhase, 0);
          d = hg_scatter(dsave, gg, u01(v.x), u01(v.y));
          t = 0.0f;
          cell = cell_x;
          tau = exp_tau(uniform01(TV_SEED, pix, (uint32_t)s, bounce, kStreamFlight, jf++));
          set_segment<Med>(tab, o, d);
          mode = M_TRACK;
        }
      }
    }
    // ================= one walk step of the main path or of the light ray
    if (mode <= M_SHADOW) {
      if (steps >= A.max_steps) {
        n_trunc++;
        mode = M_FINISH;  // truncated path keeps what it has gathered
      } else {
        Step st = lm.step(cell, o, d, tab, t);
        steps++;
        float sg = st.sigma, sb = st.majorant;
        if (mode == M_TRACK) {
          if (!st.ok) {
            mode = M_ESCAPE;
          } else {
            bool collided = false;
            float tc = 0.0f;
            if (sb > 0.0f) {
              float dtau = sb * (st.te - t);
              while (tau < dtau) {
                tc = t + tau / sb;
                if (EXT && TV_EX.model) sg = model_sigma(TV_EX, cell, o, d, tc);  // extinction at the tentative point
                bool real = true;
                if (sg < sb) real = uniform01(TV_SEED, pix, (uint32_t)s, bounce, kStreamFlight, jf++) < sg / sb;
                if (real) {
                  collided = true;
                  break;
                }
                n_null++;
                t = tc;
                tau = exp_tau(uniform01(TV_SEED, pix, (uint32_t)s, bounce, kStreamFlight, jf++));
                dtau = sb * (st.te - t);
              }
              if (!collided) tau = tau - dtau;
            }
            if (collided) {
              t = tc;
              mode = M_COLLIDE;
              // the lane walks its light ray next iteration (a path that hands
              // over to the cache at this vertex appends its query in the
              // event section instead: that append is wave-wide)
              if (NRC != 1 || trainp || (int32_t)bounce + 1 != A.truncate) start_light();
            } else {
              t = st.te;
              if (st.next < 0) mode = M_ESCAPE;
              else cell = (uint32_t)st.next;
            }
          }
        } else {  // light ray: od holds the optical depth (analytic) or the transmittance
          bool done = !st.ok;
          if (st.ok) {
            if (A.transmittance == 0 && EXT && TV_EX.model) {
              // linear model: exact integral over the segment (trapezoid)
              od = od + (0.5f * (model_sigma(TV_EX, cell, o, d, t) + model_sigma(TV_EX, cell, o, d, st.te))) * (st.te - t);
            } else if (A.transmittance == 0) {
              od = od + sg * (st.te - t);
            } else if (sb > 0.0f) {
              float dtau = sb * (st.te - t);
              while (tau < dtau) {
                t = t + tau / sb;
                if (EXT && TV_EX.model) sg = model_sigma(TV_EX, cell, o, d, t);
                if (A.transmittance == 1) {
                  od = od * (1.0f - sg / sb);
                } else {
                  bool real = true;
                  if (sg < sb) real = uniform01(TV_SEED, pix, (uint32_t)s, bounce, kStreamLight, jn++) < sg / sb;
                  if (real) {
                    od = 0.0f;
                    done = true;
                    break;
                  }
                }
                tau = exp_tau(uniform01(TV_SEED, pix, (uint32_t)s, bounce, kStreamLight, jn++));
                dtau = sb * (st.te - t);
              }
              if (!done) tau = tau - dtau;
            }
            if (A.transmittance == 1 && od == 0.0f) done = true;
            if (!done) {
              t = st.te;
              if (st.next < 0) done = true;
              else cell = (uint32_t)st.next;
            }
          }
          if (done) mode = M_SCATTER;
        }
      }
    }
  }
#undef TV_EX
#undef TV_SUN
#undef TV_ENV
#undef TV_E
#undef TV_G
#undef TV_ALBEDO
#undef TV_SEED
#undef TV_SC
  {
    if (A.defer) {  // the rest of the wave's chunk is unused
      const uint32_t base = s_lq[wv][0], used = s_lq[wv][1];
      if (used != kDone)
        for (uint32_t q = used + (uint32_t)lane; q < A.lq_chunk; q += 64) A.lq[base + q].cell = kDone;
      if (lane == 0 && s_lq[wv][2]) atomicAdd(stat_slot(A) + 6, (unsigned long long)s_lq[wv][2]);
    }
  }
  const uint32_t n_stat[6] = {n_steps, n_null, n_real, n_esc, n_trunc, n_query};
  add_stats(A, n_stat);
}

// ---------------------------------------------------------------- deferred light rays
// Bits 0..15 of x to the even bit positions.
__device__ inline uint32_t spread_bits2(uint32_t x) {
  x &= 0xFFFFu;
  x = (x | (x << 8)) & 0x00FF00FFu;
  x = (x | (x << 4)) & 0x0F0F0F0Fu;
  x = (x | (x << 2)) & 0x33333333u;
  x = (x | (x << 1)) & 0x55555555u;
  return x;
}

// Sort keys of the light rays: every ray walks along the sun direction d,
// so rays whose starts project to nearby points of the plane normal to d
// cross the same column of tets.  With (u, v) the start's coordinates in
// that plane and w its coordinate along d (all about the cube's centre,
// mapped from [-0.87, 0.87] to [0, 1)), the 32-bit key is the Z-order of
// (u, v) at c bits each (a column bundle), then w at d bits, then the Z-order
// of the position within the bundle (f bits each); in batches the scene's
// index comes first (s bits).
// Rays of one wave start close together at one depth (walks of similar
// length), and the waves in flight together cover a compact set of
// bundles, whose records stay in the caches.
struct KeyBits {
  int s, c, d, f;
};

// Key layout for grids of up to `cells` cells in `scenes` scenes: column
// bundles about as wide as the grid's typical cell, bits per axis
// ~ log2(cells) / 3 (8 on a 7 M-tet grid, 9 on 86 M tets), and 10 bits of
// depth where they fit.
static KeyBits key_bits(int64_t cells, int scenes) {
  KeyBits k;
  int cell_bits = 0;
  while (cell_bits < 40 && (int64_t)(1ull << cell_bits) < cells) cell_bits++;
  k.s = 0;
  while ((1 << k.s) < scenes) k.s++;
  k.c = std::max(4, std::min({11, (cell_bits + 1) / 3, (32 - k.s - 6) / 2}));
  k.d = std::min(10, 32 - k.s - 2 * k.c);
  k.f = (32 - k.s - k.d - 2 * k.c) / 2;
  return k;
}

__device__ inline uint32_t light_key(float3 p, float3 d, float3 t1, float3 t2, const KeyBits& K) {
  const float3 c = make_float3(p.x - 0.5f, p.y - 0.5f, p.z - 0.5f);
  const float cu = (c.x * t1.x + c.y * t1.y) + c.z * t1.z;
  const float cv = (c.x * t2.x + c.y * t2.y) + c.z * t2.z;
  const float cw = (c.x * d.x + c.y * d.y) + c.z * d.z;
  auto quant = [](float x, int bits) {
    float f = (x + 0.87f) * (1.0f / 1.74f);
    f = f < 0.0f ? 0.0f : (f > 0.99999f ? 0.99999f : f);
    return (uint32_t)(f * (float)(1u << bits));
  };
  const uint32_t uq = quant(cu, K.c + K.f), vq = quant(cv, K.c + K.f), wq = quant(cw, K.d);
  const uint32_t fm = (1u << K.f) - 1u;
  const uint32_t bundle = spread_bits2(uq >> K.f) | (spread_bits2(vq >> K.f) << 1);
  const uint32_t fine = spread_bits2(uq & fm) | (spread_bits2(vq & fm) << 1);
  return (bundle << (K.d + 2 * K.f)) | (wq << (2 * K.f)) | fine;
}

// Sort keys and queue positions of the n queue records in use.
template <bool BATCH>
__global__ __launch_bounds__(256) void k_light_keys(RenderArgs A, uint32_t n, uint32_t* __restrict__ keys,
                                                    uint32_t* __restrict__ idx, KeyBits K) {
  const uint32_t q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= n) return;
  const LightRec r = A.lq[q];
  uint32_t key = 0xFFFFFFFFu;
  if (r.cell != kDone) {
    const uint32_t sc = BATCH ? (uint32_t)scene_search(A.nscenes, r.to, [&](int k) { return A.scenes[k].entry0; }) : 0u;
    const float3 d = BATCH ? make_float3(A.scenes[sc].sun[0], A.scenes[sc].sun[1], A.scenes[sc].sun[2])
                           : make_float3(A.sun[0], A.sun[1], A.sun[2]);
    // an orthonormal basis (t1, t2) of the plane normal to d (Duff et al. 2017)
    const float sg = copysignf(1.0f, d.z);
    const float a = -1.0f / (sg + d.z);
    const float bxy = (d.x * d.y) * a;
    const float3 t1 = make_float3(1.0f + ((sg * d.x) * d.x) * a, sg * bxy, -sg * d.x);
    const float3 t2 = make_float3(bxy, sg + (d.y * d.y) * a, -d.y);
    key = light_key(make_float3(r.x, r.y, r.z), d, t1, t2, K);
    if constexpr (BATCH) key |= sc << (2 * K.c + K.d + 2 * K.f);
  }
  keys[q] = key;
  idx[q] = q;
}

// The queued light rays.  Each walks to the grid boundary by the tracer's own
// light walk (optical depth, or ratio or delta tracking of the
// transmittance), then adds its weight times the transmittance to its pixel
// (atomically), or leaves it in its record (A.chain) or as its vertex's term
// (training paths).  A
// straight walk meets a tet at most once, so the tet count bounds it.
// With `order` (the sorted queue positions) neighbouring lanes start close
// together and walk the same direction through the same column of tets, so
// they read the same records.  Without it (n on the device, in
// head[kChunkAt]) the rays are taken as queued.
template <class Med, bool BATCH, bool EXT>
__global__ __launch_bounds__(256) void k_light(RenderArgs A, Med med, const uint32_t* __restrict__ order,
                                               uint32_t n_sorted, SegDirs sun) {
  constexpr bool SHARED = !BATCH;  // one direction for all rays
  constexpr int ROWS = SHARED ? (Med::kTet ? 9 : 0) : Med::kRows;
  __shared__ float s_tab[ROWS ? ROWS * 256 : 1];
  __shared__ float s_dir[18];
  if (SHARED && threadIdx.x < 9) {
    s_dir[threadIdx.x] = sun.r[threadIdx.x];
    s_dir[9 + threadIdx.x] = sun.d[threadIdx.x];
  }
  __syncthreads();
  float* tab = s_tab + (threadIdx.x >> 6) * (ROWS * kTabRow) + (threadIdx.x & 63u);
  const uint32_t n = order ? n_sorted : min(A.head[kChunkAt], A.lq_chunks) * A.lq_chunk;
  uint32_t total = 0;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) {
    const uint32_t at = order ? order[i] : (uint32_t)i;
    const LightRec r = A.lq[at];
    if (r.cell == kDone) continue;
    const uint32_t sc = BATCH ? (uint32_t)scene_search(A.nscenes, r.to, [&](int k) { return A.scenes[k].entry0; }) : 0u;
    Med lm = med;
    if constexpr (BATCH) {
      lm.rec = (decltype(lm.rec))A.scenes[sc].rec;
      lm.n = A.scenes[sc].n;
    }
    const float3 o = make_float3(r.x, r.y, r.z);
    const float3 d = BATCH ? make_float3(A.scenes[sc].sun[0], A.scenes[sc].sun[1], A.scenes[sc].sun[2])
                           : make_float3(A.sun[0], A.sun[1], A.sun[2]);
    if constexpr (!SHARED) set_segment<Med>(tab, o, d);
    else if constexpr (Med::kTet) set_origin(tab, o, Med::kOriginScale);
    uint32_t cell = r.cell, steps = 0;
    const uint32_t limit = lm.most_cells();
    float t = 0.0f, od = 0.0f;
    const int model = EXT ? (BATCH ? A.scenes[sc].ex.model : A.ex.model) : 0;
    if (A.transmittance == 0) {
      for (;;) {
        const Step st = lm.template step<SHARED>(cell, o, d, tab, t, s_dir);
        steps++;
        if (!st.ok) break;
        if (EXT && model) {  // linear model: exact integral over the segment (trapezoid)
          const ExtArgs& X = BATCH ? A.scenes[sc].ex : A.ex;
          od = od + (0.5f * (model_sigma(X, cell, o, d, t) + model_sigma(X, cell, o, d, st.te))) * (st.te - t);
        } else {
          od = od + st.sigma * (st.te - t);
        }
        t = st.te;
        if (st.next < 0 || steps > limit) break;
        cell = (uint32_t)st.next;
      }
      od = exp_neg(od);
    } else {  // ratio (1) or delta (2) tracking: od holds the transmittance
      uint32_t pix, smp;
      uint64_t seed = A.seed;
      int32_t px, py;
      if constexpr (BATCH) {
        const SceneDesc& S = A.scenes[sc];
        const uint32_t local = (uint32_t)(r.to - S.entry0);
        (void)slot_pixel(local / (uint32_t)S.spp, S.tiles_x, S.fr.w, S.fr.h, px, py);
        pix = (uint32_t)(py * S.fr.w + px);
        smp = S.s0 + local % (uint32_t)S.spp;
        seed = S.seed;
      } else if (r.bounce & kToTerm) {
        seed = A.train ? A.seed : A.train_seed;
        smp = r.to / (uint32_t)A.max_bounces;
        pix = train_pixel(seed, smp, A.npix);
      } else {  // (tracked light rays of image paths are chained)
        (void)slot_pixel(r.to / (uint32_t)A.pass_spp, A.tiles_x, A.fr.w, A.fr.h, px, py);
        pix = (uint32_t)(py * A.fr.w + px);
        smp = (uint32_t)A.pass_start + r.to % (uint32_t)A.pass_spp;
      }
      const uint32_t bounce = r.bounce & ~kToTerm;
      uint32_t jn = 0;
      od = 1.0f;
      float tau = exp_tau(uniform01(seed, pix, smp, bounce, kStreamLight, jn++));
      for (bool done = false; !done;) {
        const Step st = lm.template step<SHARED>(cell, o, d, tab, t, s_dir);
        steps++;
        if (!st.ok) break;
        const float sb = st.majorant;
        if (sb > 0.0f) {
          float dtau = sb * (st.te - t);
          while (tau < dtau) {
            t = t + tau / sb;
            float sg = st.sigma;
            if constexpr (EXT) {
              const ExtArgs& X = BATCH ? A.scenes[sc].ex : A.ex;
              if (model) sg = model_sigma(X, cell, o, d, t);
            }
            if (A.transmittance == 1) {
              od = od * (1.0f - sg / sb);
            } else if (!(sg < sb) || uniform01(seed, pix, smp, bounce, kStreamLight, jn++) < sg / sb) {
              od = 0.0f;
              done = true;
              break;
            }
            tau = exp_tau(uniform01(seed, pix, smp, bounce, kStreamLight, jn++));
            dtau = sb * (st.te - t);
          }
          if (!done) tau = tau - dtau;
        }
        if (od == 0.0f) done = true;
        t = st.te;
        if (st.next < 0 || steps > limit) done = true;
        else cell = (uint32_t)st.next;
      }
    }
    total += steps;
    const float w0 = (r.bp * (BATCH ? A.scenes[sc].E[0] : A.E[0])) * od;
    const float w1 = (r.bp * (BATCH ? A.scenes[sc].E[1] : A.E[1])) * od;
    const float w2 = (r.bp * (BATCH ? A.scenes[sc].E[2] : A.E[2])) * od;
    if (!BATCH && (r.bounce & kToTerm)) {
      A.terms[2 * (size_t)r.to] = make_float4(w0, w1, w2, 0.0f);
    } else if (BATCH || A.chain) {
      *(float4*)(A.lq + at) = make_float4(w0, w1, w2, __uint_as_float(r.cell));
    } else {
      float* px = A.out + 3 * (size_t)r.to;
      atomicAdd(px, w0);
      atomicAdd(px + 1, w1);
      atomicAdd(px + 2, w2);
    }
  }
  const uint32_t n_stat[1] = {total};
  add_stats(A, n_stat);
}

// Samples with chained light terms (thread = entry record): emission and
// light terms in path order, then what the lane gathered apart from them (the
// environment), as a lane that walks its own light rays adds them up, so the
// image does not depend on who walked a ray or on the order of the walks.
// Paths that wait since the queue was full get the sum so far, their
// throughput and bounces at their first queue record, and are listed again.
// Bound by the chains' dependent reads, one 32-byte record per collision: the
// frame of a 256^3 volume at 512^2 x 16 samples took 6.89 ms with the terms
// added to the pixels by atomics, 6.99 with them summed here (twelve scenes in
// a batch: 4.81 and 4.64).
template <bool BATCH>
__global__ __launch_bounds__(256) void k_chain(RenderArgs A, uint64_t total) {
  const uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  bool waits = false;
  if (e < total) {
    float4* q = (float4*)(A.entries + e);
    const float4 own = q[0];
    const uint32_t mark = __float_as_uint(own.w);
    if (mark != kDone) {
      const int sc = BATCH ? scene_search(A.nscenes, e, [&](int i) { return A.scenes[i].entry0; }) : 0;
      const ExtArgs& X = BATCH ? A.scenes[sc].ex : A.ex;
      const float albedo = BATCH ? A.scenes[sc].albedo : A.albedo;
      const uint32_t head = A.entries[e].steps;
      waits = mark != kChained;
      float3 L = make_float3(0, 0, 0);
      float beta = 1.0f;
      uint32_t n = 0;
      for (uint32_t at = head; at != kDone; n++) {
        const LightRec r = A.lq[at];
        at = r.next;
        if (waits || X.ch_t) {
          const float alb = X.ch_a ? X.ch_a[r.cell] : albedo;
          if (X.ch_t) {
            const float em = (1.0f - alb) * X.ch_t[r.cell];
            L = make_float3(L.x + beta * (em * X.emission[0]), L.y + beta * (em * X.emission[1]),
                            L.z + beta * (em * X.emission[2]));
          }
          beta = beta * alb;
        }
        L = make_float3(L.x + r.x, L.y + r.y, L.z + r.z);
      }
      if (!waits) {
        q[0] = make_float4(L.x + own.x, L.y + own.y, L.z + own.z, __uint_as_float(kDone));
      } else if (head != kDone) {
        LightRec r;
        r.x = L.x;
        r.y = L.y;
        r.z = L.z;
        r.cell = kDone;
        r.bp = beta;
        r.to = 0;
        r.next = kDone;
        r.bounce = n;
        A.lq[head] = r;
      }
    }
  }
  const unsigned long long m = __ballot(waits);
  if (m) {  // (a wave's entry records are of one chunk, so of one of k_first's lists)
    const int lane = __lane_id();
    const uint32_t chunk = (uint32_t)(e / ((uint64_t)A.chunk_blocks * kFirstBlock)), round = chunk >> 3;
    const uint32_t band = (chunk - ((round * 0x9E3779B9u) >> 29)) & 7u;
    uint32_t base = 0;
    if (lane == 0) base = atomicAdd(A.head + kCountAt + (int)band * kLine, (uint32_t)__popcll(m));
    base = __shfl(base, 0);
    if (waits) A.list[(uint64_t)band * A.band_size + base + (uint32_t)__popcll(m & ((1ull << lane) - 1ull))] = (uint32_t)e;
  }
}

// Training paths with deferred light rays: what each path gathered, summed in
// path order -- before each recorded vertex into its record, in all into
// path_l (which holds the environment term and the vertex count).
__global__ __launch_bounds__(256) void k_gather_terms(RenderArgs A, uint32_t paths, int emits) {
  const uint32_t j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= paths) return;
  const float4 env = A.path_l[j];
  const uint32_t nv = __float_as_uint(env.w);
  float3 L = make_float3(0, 0, 0);
  for (uint32_t k = 0; k < nv; k++) {
    if ((int32_t)k < A.rec_vertices)
      A.vrec[((size_t)j * (uint32_t)A.rec_vertices + k) * 3 + 2] = make_float4(L.x, L.y, L.z, 0.0f);
    const float4* q = A.terms + 2 * ((size_t)j * (uint32_t)A.max_bounces + k);
    if (emits) {
      const float4 em = q[1];
      L = make_float3(L.x + em.x, L.y + em.y, L.z + em.z);
    }
    const float4 li = q[0];
    L = make_float3(L.x + li.x, L.y + li.y, L.z + li.z);
  }
  A.path_l[j] = make_float4(L.x + env.x, L.y + env.y, L.z + env.z, env.w);
}

__global__ void k_zero_u32(uint32_t* p, int n) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

__global__ void k_scale_f32(float* p, int64_t n, float div) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = p[i] / div;
}

__global__ void k_locate(TetMedium med, const float* __restrict__ pts, int64_t count, int64_t* __restrict__ out) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  float3 p = make_float3(pts[3 * i], pts[3 * i + 1], pts[3 * i + 2]);
  bool in = p.x >= 0.0f && p.x <= 1.0f && p.y >= 0.0f && p.y <= 1.0f && p.z >= 0.0f && p.z <= 1.0f;
  out[i] = in ? med.locate(p) : -1;
}

// ---------------------------------------------------------------- host
static int cu_count() {
  static int cached = 0;
  if (!cached) {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) ==
                                                 hipSuccess && n > 0)
      cached = n;
    else
      return 256;
  }
  return cached;
}

constexpr int64_t kMaxEntriesPerPass = 1ll << 25;  // 1 GiB of entry records
// tet_render_noalloc's fixed scratch: counters, 2^21 entry records, their lists
constexpr int64_t kNoAllocEntries = 1ll << 21;
constexpr int64_t kListSlack = 8 * kMostChunk;  // the lists' last, incomplete round of chunks
constexpr size_t kNoAllocBytes = (size_t)kNoAllocEntries * sizeof(RayEntry) + (size_t)(kNoAllocEntries + kListSlack) * 4 + kHeadBytes + 256;
// Sort buffers of the deferred light rays (keys and positions, both ways)
// and the sort's own scratch.
struct LightSort {
  uint32_t* keys[2];
  uint32_t* idx[2];
  void* temp;
  size_t temp_bytes;
  KeyBits bits;
  // Bytes of the buffers for `cap` rays; lays them out at p when given.
  size_t place(uint32_t cap, char* p) {
    if (rocprim::radix_sort_pairs(nullptr, temp_bytes, (uint32_t*)nullptr, (uint32_t*)nullptr, (uint32_t*)nullptr,
                                  (uint32_t*)nullptr, cap, 0u, 32u, nullptr) != hipSuccess)
      return 0;
    uint32_t* k = (uint32_t*)p;
    for (int i = 0; p && i < 2; i++) {
      keys[i] = k + (size_t)i * cap;
      idx[i] = k + (size_t)(2 + i) * cap;
    }
    if (p) temp = k + 4 * (size_t)cap;
    return (4 * (size_t)cap * 4 + temp_bytes + 255) & ~(size_t)255;
  }
};

// Whether light rays are sorted before they are walked: below, the records of
// the grids stay in an XCD's 4 MB of L2 however the rays are ordered, or
// there are too few rays to pay for the sort and the wait for their count.
// Frames in us, as queued / sorted, by tets and samples:
//             33 K         131 K         524 K         4.2 M
//   25 K    401 /  467   479 /  581    794 /  951    2922 / 2931
//   197 K   637 /  696   697 /  786   1172 / 1225    4918 / 4045
//   786 K   938 /  991  1031 / 1077   1803 / 1623    8792 / 5602
//   3.1 M  1384 / 1446  1611 / 1580   3014 / 2501   15893 / 8961
// (a uniform grid's; its light rays are short, an adaptive one's cross more).
static bool sort_pays(int64_t cells, int64_t samples) { return cells >= (1 << 17) && samples >= (1 << 17); }

// The walks of a pass's queued light rays: the n in `order`, or (order NULL)
// as they were queued, their number read on the device (no host
// synchronisation: capturable).
template <class Med, bool BATCH>
static void launch_light(const RenderArgs& P, const Med& med, bool model, const uint32_t* order, uint32_t n,
                         hipStream_t st) {
  SegDirs sun;
  seg_dirs(P.sun[0], P.sun[1], P.sun[2], sun);
  const unsigned grid = order ? (n + 255) / 256
                              : (unsigned)std::min<int64_t>((int64_t)cu_count() * 8, ((int64_t)P.lq_chunks * P.lq_chunk + 255) / 256);
  if constexpr (Med::kTet) {
    if (model) {
      hipLaunchKernelGGL((k_light<Med, BATCH, true>), dim3(grid), dim3(256), 0, st, P, med, order, n, sun);
      return;
    }
  }
  hipLaunchKernelGGL((k_light<Med, BATCH, false>), dim3(grid), dim3(256), 0, st, P, med, order, n, sun);
}

// The pass's queued light rays: the records in use, the sort by key, the walks.
template <class Med, bool BATCH>
static int walk_light_queue(const Med& med, const RenderArgs& P, bool model, LightSort& ls, hipStream_t st) {
  if (!ls.temp) {
    launch_light<Med, BATCH>(P, med, model, nullptr, 0, st);
    return TET_OK;
  }
  uint32_t n = 0;
  TV_HIP(fetch(&n, P.head + kChunkAt, 4, st));
  n = std::min(n, P.lq_chunks) * P.lq_chunk;
  if (!n) return TET_OK;
  hipLaunchKernelGGL(k_light_keys<BATCH>, dim3((n + 255) / 256), dim3(256), 0, st, P, n, ls.keys[0], ls.idx[0], ls.bits);
  size_t tb = ls.temp_bytes;
  if (rocprim::radix_sort_pairs(ls.temp, tb, ls.keys[0], ls.keys[1], ls.idx[0], ls.idx[1], n, 0u, 32u, st) !=
      hipSuccess)
    return fail(TET_ERR_DEVICE, "render: sort of the light rays");
  launch_light<Med, BATCH>(P, med, model, (const uint32_t*)ls.idx[1], n, st);
  TV_HIP(hipGetLastError());
  return TET_OK;
}

// The light-ray queue of a pass of `samples` samples.
static QueuePlan light_queue(int64_t samples, const tet_render_opts& o) {
  return queue_plan(samples, (int64_t)cu_count() * (o.blocks_per_cu ? o.blocks_per_cu : 8) * 4);
}

static void set_queue(RenderArgs& A, const QueuePlan& p, void* records) {
  A.lq_chunk = p.chunk;
  A.lq_chunks = p.chunks;
  A.lq = (LightRec*)records;
  A.defer = p.chunks > 0;
}

// The lists of a call, laid out once for its largest pass; returns their words.
static size_t set_lists(RenderArgs& A, uint64_t most) {
  const ListPlan p = list_plan(most);
  A.chunk_blocks = p.chunk_blocks;
  A.band_size = p.band_size;
  return (size_t)p.words();
}

template <class Med, bool BATCH>
static void launch_first(const RenderArgs& P, const Med& med, bool model, hipStream_t st) {
  const FirstGrid f = first_grid({P.chunk_blocks, P.band_size}, P.train_blocks);
  const dim3 grid(f.x, f.y);
  if constexpr (!std::is_same<Med, VoxelMedium>::value) {
    if (model) {
      hipLaunchKernelGGL((k_first<Med, BATCH, true>), grid, dim3(kFirstBlock), 0, st, P, med);
      return;
    }
  }
  hipLaunchKernelGGL((k_first<Med, BATCH, false>), grid, dim3(kFirstBlock), 0, st, P, med);
}

// Lanes that wait for an event before the wave handles events: an event
// section costs about twenty walk steps, so it is shared by most of the wave
// (48 against 32: cloud frame 37.9 -> 36.7 ms, plume frame 30.1 -> 29.2 ms);
// with channels or a density model more paths end in events (48: emissive
// frame 3.71 -> 3.83 ms).
static int default_event_wait(const ExtArgs& X) { return X.model || X.ch_t || X.ch_a || X.ch_g ? 32 : 48; }

// Listed paths a wave takes at a time: few enough that the last ones spread
// over the waves (with 4 waves per SIMD, against 64 paths at 5: emissive frame
// 3.53 -> 3.35 ms, linear-model frame 9.25 -> 9.04, cloud frame 36.1 -> 35.6,
// plume frame 28.2 -> 28.0; thumbnail and cached frame the same).
constexpr uint32_t kTakeItems = 32;

// The tracing kernel at an occupancy target.  Five waves per SIMD fit beside
// the segments' tables (28 KB of LDS per 256 lanes), so on tet grids 6 and 8
// mean 5.  The default is 4 without a cache: medians of ten renders in turn at
// 4 and 5, emissive frame 3.25 and 3.33 ms, linear model 8.82 and 8.99 (their
// kernels spill at 5), cloud 35.33 and 35.33, plume 27.93 and 27.83, thumbnail
// 0.235 and 0.236.  With a cache it is 5 (its kernels have that form only).
template <class Med, int NRC>
static void launch_render(const RenderArgs& P, const Med& med, bool ext, int waves, dim3 grid, dim3 block,
                          hipStream_t st) {
  if constexpr (!Med::kTet) {
    switch (waves) {
      case 4: hipLaunchKernelGGL((k_render<Med, 4, NRC>), grid, block, 0, st, P, med); break;
      case 6: hipLaunchKernelGGL((k_render<Med, 6, NRC>), grid, block, 0, st, P, med); break;
      case 8: hipLaunchKernelGGL((k_render<Med, 8, NRC>), grid, block, 0, st, P, med); break;
      default: hipLaunchKernelGGL((k_render<Med, 5, NRC>), grid, block, 0, st, P, med); break;
    }
  } else if (NRC == 0 && (waves == 4 || waves == 0)) {
    if (ext) hipLaunchKernelGGL((k_render<Med, 4, 0, false, true>), grid, block, 0, st, P, med);
    else hipLaunchKernelGGL((k_render<Med, 4, 0>), grid, block, 0, st, P, med);
  } else {
    if (ext) hipLaunchKernelGGL((k_render<Med, 5, NRC, false, true>), grid, block, 0, st, P, med);
    else hipLaunchKernelGGL((k_render<Med, 5, NRC>), grid, block, 0, st, P, med);
  }
}

// The light terms of a pass's ne entry records into their samples; the paths
// that wait are listed again.
template <bool BATCH>
static void sum_chains(const RenderArgs& P, uint64_t ne, hipStream_t st) {
  hipLaunchKernelGGL(k_zero_u32, dim3((kQueryAt + 255) / 256), dim3(256), 0, st, P.head, kQueryAt);  // the lists' counts
  hipLaunchKernelGGL(k_chain<BATCH>, dim3((unsigned)((ne + 255) / 256)), dim3(256), 0, st, P, ne);
}

// The statistics' slots on the host, to be summed.
struct HostStats {
  uint32_t w[kStatSlots * kLine];
  hipError_t fetch(const uint32_t* head, hipStream_t st) {
    return tv::fetch(w, head + kStatAt, sizeof(w), st);
  }
  int64_t sum(int q) const {
    uint64_t s = 0;
    for (int k = 0; k < kStatSlots; k++) {
      uint64_t v;
      memcpy(&v, w + k * kLine + 2 * q, 8);
      s += v;
    }
    return (int64_t)s;
  }
};

template <class Med, int NRC>
static int run_passes(const Med& med, RenderArgs& A, const tet_render_opts& o, int32_t spp, int64_t npix,
                      int64_t pass_cap, hipStream_t st, float* ms_total, float* ms_trace, float* ms_cache,
                      bool timed = true, LightSort* ls = nullptr, HostStats* hs = nullptr, int64_t queue_rays = 0) {
  // queue_rays: light rays of a pass that surely find room in its queue
  if (A.defer && !ls) return fail(TET_ERR_INTERNAL, "render: light-ray queue without its sort");
  int bs = o.block_size ? o.block_size : 256;
  int bpc = o.blocks_per_cu ? o.blocks_per_cu : 8;
  const bool ext = A.ex.model != 0 || A.ex.ch_t || A.ex.ch_a || A.ex.ch_g;
  // several contributions per pixel: passes, light rays that add to it, cache queries
  const bool chain = A.defer && A.chain, several = pass_cap < spp || (A.defer && !chain) || NRC == 1;
  // timed: HIP events around the passes, waited for after each pass (after
  // the last one together with the statistics, hs);
  // untimed: kernel launches on the stream only
  hipEvent_t e0 = nullptr, e1 = nullptr, e2 = nullptr, t0 = nullptr, t1 = nullptr;
  struct Ev {
    hipEvent_t *a, *b, *c, *d, *f;
    ~Ev() {
      for (hipEvent_t* e : {a, b, c, d, f})
        if (*e) (void)hipEventDestroy(*e);
    }
  } ev{&e0, &e1, &e2, &t0, &t1};
  if (timed) {
    TV_HIP(hipEventCreate(&e0));
    TV_HIP(hipEventCreate(&e1));
    TV_HIP(hipEventCreate(&e2));
    TV_HIP(hipEventCreate(&t0));
    TV_HIP(hipEventCreate(&t1));
  }
  *ms_total = 0.0f;
  *ms_trace = 0.0f;
  *ms_cache = 0.0f;
  auto pass_times = [&]() -> int {
    float ms = 0.0f;
    TV_HIP(hipEventElapsedTime(&ms, t0, t1));
    *ms_trace += ms;
    TV_HIP(hipEventElapsedTime(&ms, t1, e2));
    *ms_cache += ms;
    return TET_OK;
  };
  if (timed) TV_HIP(hipEventRecord(e0, st));
  for (int32_t done = 0; done < spp; done += (int32_t)pass_cap) {
    A.pass_start = A.pass_start + (done ? (int32_t)pass_cap : 0);
    A.pass_spp = (int32_t)std::min<int64_t>(pass_cap, spp - done);
    RenderArgs P = A;
    P.train_items = (NRC == 1 && done == 0) ? A.train_items : 0u;  // training paths ride the first pass
    const uint64_t ne = (uint64_t)A.slots * (uint64_t)P.pass_spp;
    if (ne > 8 * (uint64_t)P.band_size) return fail(TET_ERR_INTERNAL, "render: lists too small for the pass");
    hipLaunchKernelGGL(k_zero_u32, dim3((kPassWords + 255) / 256), dim3(256), 0, st, A.head, kPassWords);
    if (timed) TV_HIP(hipEventRecord(t0, st));
    P.train_blocks = (P.train_items + kFirstBlock - 1) / kFirstBlock;
    P.train_blocks = (P.train_blocks + 7) / 8 * 8;
    launch_first<Med, false>(P, med, A.ex.model != 0, st);
    int64_t grid = (int64_t)cu_count() * bpc;
    int64_t need = ((int64_t)ne + P.train_items + bs - 1) / bs;
    grid = std::max<int64_t>(1, std::min(grid, need));
    launch_render<Med, NRC>(P, med, ext, o.waves_per_simd, dim3((unsigned)grid), dim3(bs), st);
    auto resolve = [&] {
      hipLaunchKernelGGL(k_resolve, dim3((A.slots + 255) / 256), dim3(256), 0, st, P, !several ? 0 : (done ? 2 : 1));
    };
    if (NRC != 2 && !chain) resolve();
    TV_HIP(hipGetLastError());
    if (A.defer)  // the pass's queued light rays, part of the tracing time
      if (int rc = walk_light_queue<Med, false>(med, P, A.ex.model != 0, *ls, st)) return rc;
    if (chain) {  // their terms into the samples, then the paths that found the queue full
      sum_chains<false>(P, ne, st);
      if ((int64_t)ne * A.max_bounces > queue_rays) {
        RenderArgs R = P;
        R.defer = 0;
        R.resume = 1;
        R.train_items = 0;
        launch_render<Med, NRC>(R, med, ext, o.waves_per_simd, dim3((unsigned)grid), dim3(bs), st);
      }
      resolve();
    }
    if (A.terms && (NRC == 2 || P.train_items)) {
      const uint32_t paths = NRC == 2 ? A.slots : P.train_items;
      hipLaunchKernelGGL(k_gather_terms, dim3((paths + 255) / 256), dim3(256), 0, st, P, paths, A.ex.ch_t ? 1 : 0);
    }
    if (timed) TV_HIP(hipEventRecord(t1, st));
    if (NRC == 1)  // the pass's cache queries, added to their pixels
      if (int rc = nrc_query_pass(A.nrc, A.qbuf, A.qpix, A.qcount, A.out, (int64_t)ne, st)) return rc;
    if (timed) {
      TV_HIP(hipEventRecord(e2, st));
      if (done + pass_cap < spp) {  // (the last pass's times: below, with one wait for all)
        TV_HIP(hipEventSynchronize(e2));
        if (int rc = pass_times()) return rc;
      }
    }
  }
  if (several && NRC != 2)
    hipLaunchKernelGGL(k_scale_f32, dim3((unsigned)((npix * 3 + 255) / 256)), dim3(256), 0, st, A.out, npix * 3,
                       (float)spp);
  TV_HIP(hipGetLastError());
  if (timed) {
    TV_HIP(hipEventRecord(e1, st));
    if (hs) TV_HIP(hs->fetch(A.head, st));
    else TV_HIP(hipEventSynchronize(e1));
    if (int rc = pass_times()) return rc;
    TV_HIP(hipEventElapsedTime(ms_total, e0, e1));
  }
  return TET_OK;
}

// Whether the vertex terms of n training paths are worth keeping (32 bytes
// per vertex a path may have): beyond, their lanes walk their own light rays.
static bool terms_fit(int64_t n, int64_t max_bounces) { return n * max_bounces <= (256ll << 20) / 32; }

// Zeroes the statistics of a call (its passes zero the other counters).
static void zero_stats(uint32_t* head, hipStream_t st) {
  constexpr int n = kStatSlots * kLine;
  hipLaunchKernelGGL(k_zero_u32, dim3((n + 255) / 256), dim3(256), 0, st, head + kStatAt, n);
}

static int check_render_opts(const tet_render_opts& o) {
  if (o.max_bounces < 1 || o.transmittance < 0 || o.transmittance > 2 || o.max_steps_per_path < 1 ||
      o.sample_offset < 0 || o.samples_per_item < 0 || o.block_size < 0 || o.block_size > 256 ||
      (o.block_size % 64) != 0 || o.blocks_per_cu < 0 ||
      (o.waves_per_simd != 0 && o.waves_per_simd != 4 && o.waves_per_simd != 5 && o.waves_per_simd != 6 &&
       o.waves_per_simd != 8) ||
      (o.record_layout != 0 && o.record_layout != 32 && o.record_layout != 48) || o.batch_items < 0 ||
      o.batch_items > (1 << 20) || o.event_wait < 0 || o.event_wait > 64)
    return fail(TET_ERR_INVALID_ARG, "render: bad options");
  return TET_OK;
}

static void set_scene(RenderArgs& A, const tet_camera* cam, const tet_medium* medm, const tet_light* light) {
  make_frame(*cam, &A.fr);
  A.albedo = medm->albedo;
  A.g = medm->g;
  for (int i = 0; i < 3; i++) {
    A.sun[i] = light->sun_dir[i];
    A.E[i] = light->sun_irradiance[i];
    A.env[i] = light->env_radiance[i];
  }
}

// Extra channels (temperature, albedo, phase parameter per tet): a tet grid
// that carries at least one, and a finite emission colour >= 0.  They
// combine with the radiance cache (the cache at a vertex stands for all the
// radiance from it on, the vertex's emission included).
static int check_channels(const tet_render_opts& o, const tet_grid* g, const char* who) {
  if (!o.channels) return TET_OK;
  const std::string w(who);
  if (o.channels != 1) return fail(TET_ERR_INVALID_ARG, w + ": channels must be 0 or 1");
  if (!g) return fail(TET_ERR_UNSUPPORTED, w + ": channels need a tet grid");
  if (!g->ch[0] && !g->ch[1] && !g->ch[2]) return fail(TET_ERR_INVALID_ARG, w + ": the grid has no channels");
  for (int c = 0; c < 3; c++)
    if (!(o.emission[c] >= 0.0f) || std::isinf(o.emission[c]))
      return fail(TET_ERR_INVALID_ARG, w + ": emission must be finite and >= 0");
  return TET_OK;
}

// The voxel-lookup model has no analytic light transmittance.
static int check_model(const tet_render_opts& o, const tet_grid* g, const char* who) {
  if (g && g->model == 2 && o.transmittance == 0)
    return fail(TET_ERR_INVALID_ARG,
                std::string(who) + ": the voxel-lookup model needs ratio or delta tracking for the light");
  return TET_OK;
}

// The channels (when asked for) and the density model of grid g.
static void set_ext(ExtArgs& X, const tet_grid* g, const tet_render_opts& o) {
  memset(&X, 0, sizeof(X));
  if (o.channels) {
    X.ch_t = g->ch[0];
    X.ch_a = g->ch[1];
    X.ch_g = g->ch[2];
    for (int c = 0; c < 3; c++) X.emission[c] = o.emission[c];
  }
  if (g->model) {
    X.model = g->model;
    X.mcoef = g->mcoef;
    X.mdens = g->mdens;
    X.mn = g->mn;
    X.mscale = g->mscale;
  }
}

static int render_common(int kind, const tet_grid* g, const tet_density* dens, const tet_camera* cam,
                         const tet_medium* medm, const tet_light* light, int32_t spp, uint64_t seed,
                         const tet_render_opts* opts_in, float* out_rgb, int32_t on_device, hipStream_t st,
                         tet_render_stats* stats, char* fixed = nullptr, size_t fixed_bytes = 0) {
  // fixed != NULL: the scratch is the caller's fixed device array (no
  // allocation, no timing, no wait; launches on the stream only)
  const bool noalloc = fixed != nullptr;
  if (int rc = check_camera(cam)) return rc;
  if (!medm || !light || !out_rgb) return fail(TET_ERR_INVALID_ARG, "render: NULL medium, light or output");
  if (spp < 1) return fail(TET_ERR_INVALID_ARG, "render: spp must be >= 1");
  if (!(medm->g > -1.0f && medm->g < 1.0f) || !(medm->albedo >= 0.0f))
    return fail(TET_ERR_INVALID_ARG, "render: medium needs albedo >= 0 and -1 < g < 1");
  tet_render_opts o;
  if (opts_in) o = *opts_in;
  else tet_render_opts_defaults(&o);
  if (int rc = check_render_opts(o)) return rc;
  const tet_nrc* nrc = o.nrc;
  if (nrc && kind != 0) return fail(TET_ERR_UNSUPPORTED, "render: the radiance cache needs a tet grid");
  const bool train = nrc && o.nrc_train;
  const int32_t n_train = train ? nrc->opts.train_paths : 0, kv = train ? nrc->opts.train_vertices : 0;
  if (train)
    if (int rc = nrc_resolve_sigma_ref(const_cast<tet_nrc*>(nrc), g, st)) return rc;
  if (nrc && !(nrc->opts.sigma_ref > 0.0f))
    return fail(TET_ERR_INVALID_ARG, "render: the radiance cache has no sigma_ref yet (train it or set one)");
  if ((int64_t)o.sample_offset + spp > (1ll << 31)) return fail(TET_ERR_INVALID_ARG, "render: sample range too large");
  if (int rc = check_channels(o, kind == 0 ? g : nullptr, "render")) return rc;
  if (int rc = check_model(o, kind == 0 ? g : nullptr, "render")) return rc;
  const bool model = kind == 0 && g->model != 0;  // walk the records whose majorants bound the model
  if (noalloc && (kind != 0 || nrc || !on_device || stats))
    return fail(TET_ERR_UNSUPPORTED,
                "tet_render_noalloc: tet grids only, no radiance cache, output on the device, no stats");
  // the no-alloc path only takes a shape table that already exists (every
  // grid's build made the one of its device)
  const uint32_t* shapes = noalloc ? shape_table_existing() : shape_table();
  if (!shapes) return fail(TET_ERR_DEVICE, "render: shape table");
  int64_t npix = (int64_t)cam->width * cam->height;
  int tiles_x = (cam->width + 7) / 8, tiles_y = (cam->height + 7) / 8;
  int64_t slots = (int64_t)tiles_x * tiles_y * 64;
  if (slots >= (1ll << 31)) return fail(TET_ERR_INVALID_ARG, "render: image too large");
  const int64_t entry_cap =
      noalloc ? std::min<int64_t>(kMaxEntriesPerPass, kNoAllocEntries) : kMaxEntriesPerPass;
  if (noalloc && slots > entry_cap)
    return fail(TET_ERR_CAPACITY, "tet_render_noalloc: one sample per pixel of this image does not fit the "
                                  "fixed scratch (" + std::to_string(entry_cap) + " entry records)");
  int64_t pass_cap = std::max<int64_t>(1, std::min<int64_t>(spp, entry_cap / slots));

  // Light rays are queued and walked after each pass when the step guard is
  // at its largest value (2^31 - 1: each light walk then runs on its own,
  // bounded by the tet count, while the guard would count all of a path's
  // walks together; the estimate is the same unless a path takes more than
  // 2^31 - 1 steps).  Their terms are summed with the rest of their samples,
  // but for analytic light on a tet grid of constant extinctions, which adds
  // them to the pixels one by one (summed with the samples: cloud frame of
  // 33 M samples 35.6 -> 36.7 ms, plume 28.0 -> 28.7).
  bool defer = o.max_steps_per_path >= 0x7FFFFFFF;
  const bool chain = kind == 1 || model || noalloc || o.transmittance != 0;
  if (noalloc && defer) {
    static_assert(sizeof(RayEntry) == 32 && sizeof(LightRec) == 32, "queued_pass counts 32 + 4 + 40 bytes a sample");
    const int64_t queued = queued_pass(slots, pass_cap, (int64_t)fixed_bytes);
    if (queued > 0) pass_cap = queued;
    else defer = false;
  }

  RenderArgs A;
  memset(&A, 0, sizeof(A));
  set_scene(A, cam, medm, light);
  if (kind == 0) set_ext(A.ex, g, o);
  A.spp = spp;
  A.pass_start = o.sample_offset;
  A.max_bounces = o.max_bounces;
  A.transmittance = o.transmittance;
  A.max_steps = (uint32_t)std::min<int64_t>(o.max_steps_per_path, 0x7FFFFFFF);
  A.seed = seed;
  A.slots = (uint32_t)slots;
  A.tiles_x = tiles_x;
  A.chain = chain;
  A.batch = o.batch_items ? (uint32_t)o.batch_items : kTakeItems;
  A.event_wait = o.event_wait ? o.event_wait : default_event_wait(A.ex);
  if (nrc) {
    A.nrc = nrc;
    A.truncate = nrc->opts.truncate_bounce;
  }
  if (train) {
    A.train_items = (uint32_t)n_train;
    A.train_ent0 = (uint32_t)(slots * pass_cap);
    A.train_seed = seed ^ 0x6A09E667F3BCC909ull;
    A.npix = (uint32_t)npix;
    A.rec_vertices = kv;
  }

  const bool train_terms = train && defer && terms_fit(n_train, o.max_bounces);
  // scratch: counters, entry records of one pass (then those of the training
  // paths) and their lists, image when the output is on the host,
  // training-path records
  size_t img_bytes = (size_t)npix * 3 * sizeof(float);
  size_t n_ent = (size_t)slots * (size_t)pass_cap, list0 = set_lists(A, n_ent);
  size_t ent_bytes = kHeadBytes + (n_ent + (size_t)n_train) * sizeof(RayEntry) + (list0 + (size_t)n_train) * 4;
  ent_bytes = (ent_bytes + 255) & ~(size_t)255;
  size_t vrec_bytes = (size_t)n_train * (size_t)kv * 48, pl_bytes = (size_t)n_train * 16;
  size_t q_bytes = nrc ? (size_t)slots * (size_t)pass_cap * 36 : 0;  // at most one query per sample
  size_t scratch = ent_bytes + (on_device ? 0 : (img_bytes + 255) & ~(size_t)255) + vrec_bytes + pl_bytes + q_bytes;
  if (noalloc && scratch > fixed_bytes) return fail(TET_ERR_INTERNAL, "tet_render_noalloc: scratch overrun");
  char* sc = noalloc ? fixed : (char*)dev_alloc(scratch);
  if (!sc) return fail(TET_ERR_OUT_OF_MEMORY, "render: scratch");
  struct Free {
    void* p;
    ~Free() { if (p) dev_free(p); }
  } fr_{noalloc ? nullptr : sc};
  A.head = (uint32_t*)sc;
  A.entries = (RayEntry*)(sc + kHeadBytes);
  A.list = (uint32_t*)(A.entries + n_ent + (size_t)n_train);
  A.train_list0 = (uint32_t)list0;
  A.out = on_device ? out_rgb : (float*)(sc + ent_bytes);
  char* tail = sc + ent_bytes + (on_device ? 0 : (img_bytes + 255) & ~(size_t)255);
  if (train) {
    A.vrec = (float4*)tail;
    A.path_l = (float4*)(tail + vrec_bytes);
  }
  zero_stats(A.head, st);

  // the light-ray queue of a pass (at most 4 light rays per sample, 2^26 in
  // all; a full queue leaves the rest to the tracing lanes) and its sort
  LightSort ls;
  memset(&ls, 0, sizeof(ls));
  struct FreeQ {
    void* p;
    ~FreeQ() { if (p) dev_free(p); }
  } frq_{nullptr};
  QueuePlan qp = light_queue(slots * pass_cap + n_train, o);
  if (defer && noalloc) {  // what the entry records leave of the fixed scratch, walked as queued
    qp.chunks = (uint32_t)std::min<size_t>(qp.chunks, (fixed_bytes - ent_bytes) / sizeof(LightRec) / qp.chunk);
    set_queue(A, qp, sc + ent_bytes);
  } else if (defer) {
    const uint32_t cap = qp.records();
    const int64_t cells = kind == 0 ? g->n : (int64_t)dens->n * dens->n * dens->n;
    size_t sort_bytes = 0;
    if (sort_pays(cells, slots * pass_cap)) {
      ls.bits = key_bits(cells, 1);
      sort_bytes = ls.place(cap, nullptr);
      if (!sort_bytes) return fail(TET_ERR_DEVICE, "render: light-ray sort size");
    }
    const size_t term_bytes = train_terms ? (size_t)n_train * (size_t)o.max_bounces * 32 : 0;
    const size_t qb = (size_t)cap * sizeof(LightRec) + sort_bytes + term_bytes;
    if (char* q = (char*)dev_alloc(qb)) {  // (no room: the lanes walk their own light rays)
      frq_.p = q;
      set_queue(A, qp, q);
      if (train_terms) A.terms = (float4*)(q + qb - term_bytes);
      if (sort_bytes) (void)ls.place(cap, q + (size_t)cap * sizeof(LightRec));
    }
  }

  if (nrc) {
    char* qb = tail + vrec_bytes + pl_bytes;
    A.qbuf = (float4*)qb;
    A.qpix = (uint32_t*)(qb + (size_t)slots * (size_t)pass_cap * 32);
    A.qcount = A.head + kQueryAt;
  }
  float ms = 0.0f, ms_trace = 0.0f, ms_cache = 0.0f;
  HostStats hs;
  int rc;
  if (kind == 0 && g->rec32 && o.record_layout != 48) {
    TetMedium32 m{model ? g->mrec32 : g->rec32, g->keys, g->n, g->max_depth, shapes, g->kidx, g->kbits};
    rc = nrc ? run_passes<TetMedium32, 1>(m, A, o, spp, npix, pass_cap, st, &ms, &ms_trace, &ms_cache,
                                          !noalloc, &ls, &hs, qp.sure())
             : run_passes<TetMedium32, 0>(m, A, o, spp, npix, pass_cap, st, &ms, &ms_trace, &ms_cache,
                                          !noalloc, &ls, &hs, qp.sure());
  } else if (kind == 0) {
    if (o.record_layout == 32) return fail(TET_ERR_UNSUPPORTED, "render: this grid has no compact records");
    TetMedium m{model ? g->mrec : g->rec, g->keys, g->n, g->max_depth, shapes, g->kidx, g->kbits};
    rc = nrc ? run_passes<TetMedium, 1>(m, A, o, spp, npix, pass_cap, st, &ms, &ms_trace, &ms_cache,
                                        !noalloc, &ls, &hs, qp.sure())
             : run_passes<TetMedium, 0>(m, A, o, spp, npix, pass_cap, st, &ms, &ms_trace, &ms_cache,
                                        !noalloc, &ls, &hs, qp.sure());
  } else {
    VoxelMedium m{dens->data, dens->n, dens->density_scale, 0, 1.0f / (float)dens->n};
    while ((1 << m.sh) < dens->n) m.sh++;
    rc = run_passes<VoxelMedium, 0>(m, A, o, spp, npix, pass_cap, st, &ms, &ms_trace, &ms_cache,
                                    !noalloc, &ls, &hs, qp.sure());
  }
  if (rc) return rc;
  if (noalloc) return TET_OK;
  int64_t records = 0;
  double loss = 0.0;
  if (train) {  // the cache's Adam steps on the frame's training paths (timed into ms)
    hipEvent_t t0, t1;
    TV_HIP(hipEventCreate(&t0));
    TV_HIP(hipEventCreate(&t1));
    struct Ev {
      hipEvent_t a, b;
      ~Ev() {
        (void)hipEventDestroy(a);
        (void)hipEventDestroy(b);
      }
    } ev{t0, t1};
    TV_HIP(hipEventRecord(t0, st));
    if (int trc = nrc_train_paths(const_cast<tet_nrc*>(nrc), A.vrec, A.path_l, n_train, kv, st, &records, &loss))
      return trc;
    TV_HIP(hipEventRecord(t1, st));
    TV_HIP(hipEventSynchronize(t1));
    float tms = 0.0f;
    TV_HIP(hipEventElapsedTime(&tms, t0, t1));
    ms += tms;
  }
  if (!on_device) {
    TV_HIP(hipMemcpyAsync(out_rgb, A.out, img_bytes, hipMemcpyDeviceToHost, st));
    TV_HIP(hipStreamSynchronize(st));
  }
  if (stats) {
    stats->tet_steps = hs.sum(0);
    stats->null_collisions = hs.sum(1);
    stats->real_collisions = hs.sum(2);
    stats->escapes = hs.sum(3);
    stats->truncated = hs.sum(4);
    stats->ms = ms;
    stats->trace_ms = ms_trace;
    stats->cache_ms = ms_cache;
    stats->cache_queries = hs.sum(5);
    stats->cache_records = records;
    stats->cache_loss = loss;
    stats->light_rays_queued = hs.sum(6);
  }
  return TET_OK;
}

int trace_training_paths(const tet_grid* g, const tet_camera* cam, const tet_medium* medm, const tet_light* light,
                         uint64_t frame_seed, const tet_render_opts* opts_in, int32_t n_paths, int32_t kv, float4* vrec,
                         float4* path_l, hipStream_t st, float* ms_out) {
  if (!g) return fail(TET_ERR_INVALID_ARG, "training paths: grid is NULL");
  const uint32_t* shapes = shape_table();
  if (!shapes) return fail(TET_ERR_DEVICE, "training paths: shape table");
  if (int rc = check_camera(cam)) return rc;
  if (!medm || !light) return fail(TET_ERR_INVALID_ARG, "training paths: NULL medium or light");
  if (!(medm->g > -1.0f && medm->g < 1.0f) || !(medm->albedo >= 0.0f))
    return fail(TET_ERR_INVALID_ARG, "training paths: medium needs albedo >= 0 and -1 < g < 1");
  tet_render_opts o;
  if (opts_in) o = *opts_in;
  else tet_render_opts_defaults(&o);
  if (int rc = check_render_opts(o)) return rc;
  if (int rc = check_channels(o, g, "training paths")) return rc;
  if (int rc = check_model(o, g, "training paths")) return rc;
  if (n_paths < 1 || kv < 1) return fail(TET_ERR_INVALID_ARG, "training paths: bad counts");
  RenderArgs A;
  memset(&A, 0, sizeof(A));
  set_scene(A, cam, medm, light);
  set_ext(A.ex, g, o);
  A.spp = 1;
  A.max_bounces = o.max_bounces;
  A.transmittance = o.transmittance;
  A.max_steps = (uint32_t)std::min<int64_t>(o.max_steps_per_path, 0x7FFFFFFF);
  A.seed = frame_seed;
  A.slots = (uint32_t)n_paths;
  A.tiles_x = (cam->width + 7) / 8;
  A.batch = o.batch_items ? (uint32_t)o.batch_items : 64u;
  A.event_wait = o.event_wait ? o.event_wait : default_event_wait(A.ex);
  A.train = 1;
  A.npix = (uint32_t)((int64_t)cam->width * cam->height);
  A.rec_vertices = kv;
  A.vrec = vrec;
  A.path_l = path_l;
  const size_t list_words = set_lists(A, (uint64_t)n_paths);
  char* sc = (char*)dev_alloc(kHeadBytes + (size_t)n_paths * sizeof(RayEntry) + 4 * list_words);
  if (!sc) return fail(TET_ERR_OUT_OF_MEMORY, "training paths: scratch");
  struct Free {
    void* p;
    ~Free() { dev_free(p); }
  };
  Free fr_{sc};
  A.head = (uint32_t*)sc;
  A.entries = (RayEntry*)(sc + kHeadBytes);
  A.list = (uint32_t*)(A.entries + n_paths);
  zero_stats(A.head, st);
  LightSort ls;  // (unsorted: few rays)
  memset(&ls, 0, sizeof(ls));
  Free fq_{nullptr};
  if (o.max_steps_per_path >= 0x7FFFFFFF && terms_fit(n_paths, o.max_bounces)) {
    const QueuePlan qp = light_queue(n_paths, o);
    const size_t qb = (size_t)qp.records() * sizeof(LightRec);
    fq_.p = dev_alloc(qb + (size_t)n_paths * (size_t)o.max_bounces * 32);
    if (fq_.p) {  // (no room: the lanes walk their own light rays)
      set_queue(A, qp, fq_.p);
      A.terms = (float4*)((char*)fq_.p + qb);
    }
  }
  float ms = 0.0f, ms_trace = 0.0f, ms_cache = 0.0f;
  int rc;
  const bool model = g->model != 0;
  if (g->rec32 && o.record_layout != 48) {
    TetMedium32 m{model ? g->mrec32 : g->rec32, g->keys, g->n, g->max_depth, shapes, g->kidx, g->kbits};
    rc = run_passes<TetMedium32, 2>(m, A, o, 1, 0, 1, st, &ms, &ms_trace, &ms_cache, true, &ls);
  } else {
    if (o.record_layout == 32) return fail(TET_ERR_UNSUPPORTED, "training paths: this grid has no compact records");
    TetMedium m{model ? g->mrec : g->rec, g->keys, g->n, g->max_depth, shapes, g->kidx, g->kbits};
    rc = run_passes<TetMedium, 2>(m, A, o, 1, 0, 1, st, &ms, &ms_trace, &ms_cache, true, &ls);
  }
  if (rc) return rc;
  TV_HIP(hipStreamSynchronize(st));
  if (ms_out) *ms_out = ms_trace;
  return TET_OK;
}

void launch_defaults(const tet_grid* g, tet_render_opts* o) {
  ExtArgs x;
  set_ext(x, g, *o);
  if (!o->waves_per_simd) o->waves_per_simd = o->nrc ? 5 : 4;
  if (!o->event_wait) o->event_wait = default_event_wait(x);
  if (!o->batch_items) o->batch_items = (int32_t)kTakeItems;
  if (!o->block_size) o->block_size = 256;
  if (!o->record_layout) o->record_layout = g->rec32 ? 32 : 48;
}

int render_grid(const tet_grid* g, const tet_camera* cam, const tet_medium* m, const tet_light* l, int32_t spp,
                uint64_t seed, const tet_render_opts* o, float* out, int32_t on_device, hipStream_t st,
                tet_render_stats* stats) {
  if (!g) return fail(TET_ERR_INVALID_ARG, "tet_render: grid is NULL");
  return render_common(0, g, nullptr, cam, m, l, spp, seed, o, out, on_device, st, stats);
}

// ---------------------------------------------------------------- render without allocation
// The scratch of tet_render_noalloc: a fixed array, one copy per device (made
// when the library's code is loaded on it, kept until the process ends).  In
// host code `scratch` only names the symbol; its device address comes from
// hipGetSymbolAddress, looked up once per device.
static __device__ __align__(256) char scratch[kNoAllocBytes];
constexpr int kMaxDevices = 64;

static char* noalloc_scratch() {
  static std::mutex mu;
  static char* ptr[kMaxDevices] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lk(mu);
  if (!ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
      (void)hipGetLastError();
      return nullptr;
    }
    ptr[dev] = (char*)p;
  }
  return ptr[dev];
}

int render_grid_noalloc(const tet_grid* g, const tet_camera* cam, const tet_medium* m, const tet_light* l,
                        int32_t spp, uint64_t seed, const tet_render_opts* o, float* out, hipStream_t st) {
  if (!g) return fail(TET_ERR_INVALID_ARG, "tet_render_noalloc: grid is NULL");
  int dev = -1;
  TV_HIP(hipGetDevice(&dev));
  if (dev != g->device) return fail(TET_ERR_INVALID_ARG, "tet_render_noalloc: the grid lives on another device");
  char* sc = noalloc_scratch();
  if (!sc) return fail(TET_ERR_DEVICE, "tet_render_noalloc: no device address for the fixed scratch");
  return render_common(0, g, nullptr, cam, m, l, spp, seed, o, out, 1, st, nullptr, sc, kNoAllocBytes);
}

int render_voxels(const tet_density* dens, const tet_camera* cam, const tet_medium* m, const tet_light* l,
                  int32_t spp, uint64_t seed, const tet_render_opts* o, float* out, int32_t on_device,
                  hipStream_t st, tet_render_stats* stats) {
  if (!dens || !dens->data) return fail(TET_ERR_INVALID_ARG, "dda_render: density is NULL");
  int32_t n = dens->n;
  if (n < 1 || n > 1024 || (n & (n - 1))) return fail(TET_ERR_INVALID_ARG, "dda_render: n must be a power of two <= 1024");
  if (dens->on_device) return render_common(1, nullptr, dens, cam, m, l, spp, seed, o, out, on_device, st, stats);
  size_t bytes = (size_t)n * n * n * 4;
  float* dd = (float*)dev_alloc(bytes);
  if (!dd) return fail(TET_ERR_OUT_OF_MEMORY, "dda_render: density copy");
  struct Free {
    void* p;
    ~Free() { dev_free(p); }
  } f_{dd};
  TV_HIP(hipMemcpyAsync(dd, dens->data, bytes, hipMemcpyHostToDevice, st));
  tet_density dv = *dens;
  dv.data = dd;
  dv.on_device = 1;
  return render_common(1, nullptr, &dv, cam, m, l, spp, seed, o, out, on_device, st, stats);
}

// ---------------------------------------------------------------- batches of scenes
struct BatchState {
  int device = 0;
  int n = 0;
  bool use32 = true;
  bool ext = false;    // some scene carries channels or a density model
  bool model = false;  // some grid carries a density model
  LightSort ls = {};   // sort of the light rays (temp == nullptr: walked as queued)
  const uint32_t* shapes = nullptr;
  tet_render_opts o;
  SceneDesc* pinned = nullptr;  // host staging of the scene table (page-locked)
  SceneDesc* table = nullptr;   // device scene table
  char* scratch = nullptr;      // counters and statistics, the entry records, their lists
  RenderArgs A;
  uint64_t total_px = 0;
  int grid = 1, bs = 256;
  int64_t queue_rays = 0;  // light rays that surely find room in the queue
  hipStream_t cap = nullptr;    // capture stream of the frame graph
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  ~BatchState() {
    if (exec) (void)hipGraphExecDestroy(exec);
    if (graph) (void)hipGraphDestroy(graph);
    if (cap) (void)hipStreamDestroy(cap);
    dev_free(table);
    dev_free(scratch);
    if (pinned) (void)hipHostFree(pinned);
  }
};

static int batch_setup(BatchState* B, int32_t n, const tet_grid* const* grids, const tet_camera* cams,
                       const tet_medium* media, const tet_light* lights, const int32_t* spp,
                       const tet_render_opts* opts_in, float* const* outs) {
  if (n < 1 || n > 4096 || !grids || !cams || !media || !lights || !spp || !outs)
    return fail(TET_ERR_INVALID_ARG, "render batch: bad arguments (1 <= n <= 4096, no NULL arrays)");
  tet_render_opts o;
  if (opts_in) o = *opts_in;
  else tet_render_opts_defaults(&o);
  if (int rc = check_render_opts(o)) return rc;
  if (o.nrc) return fail(TET_ERR_UNSUPPORTED, "render batch: no radiance cache in batches");
  bool use32 = o.record_layout != 48;
  for (int i = 0; i < n; i++) {
    if (!grids[i] || !outs[i]) return fail(TET_ERR_INVALID_ARG, "render batch: NULL grid or output");
    if (int rc = check_channels(o, grids[i], "render batch")) return rc;
    if (int rc = check_model(o, grids[i], "render batch")) return rc;
    if (int rc = check_camera(&cams[i])) return rc;
    if (!(media[i].g > -1.0f && media[i].g < 1.0f) || !(media[i].albedo >= 0.0f))
      return fail(TET_ERR_INVALID_ARG, "render batch: medium needs albedo >= 0 and -1 < g < 1");
    if (spp[i] < 1 || (int64_t)o.sample_offset + spp[i] > (1ll << 31))
      return fail(TET_ERR_INVALID_ARG, "render batch: bad spp");
    if (!grids[i]->rec32) use32 = false;
  }
  if (!use32 && o.record_layout == 32)
    return fail(TET_ERR_UNSUPPORTED, "render batch: a grid has no compact records");
  B->n = n;
  B->o = o;
  B->use32 = use32;
  B->shapes = shape_table();  // made here: a captured frame cannot upload it
  if (!B->shapes) return fail(TET_ERR_DEVICE, "render batch: shape table");
  if (hipGetDevice(&B->device) != hipSuccess) return fail(TET_ERR_DEVICE, "render batch: no device");
  std::vector<SceneDesc> host((size_t)n);
  uint64_t entry = 0, px = 0;
  for (int i = 0; i < n; i++) {
    SceneDesc& S = host[i];
    memset(&S, 0, sizeof(S));
    make_frame(cams[i], &S.fr);
    S.albedo = media[i].albedo;
    S.g = media[i].g;
    for (int c = 0; c < 3; c++) {
      S.sun[c] = lights[i].sun_dir[c];
      S.E[c] = lights[i].sun_irradiance[c];
      S.env[c] = lights[i].env_radiance[c];
    }
    S.spp = spp[i];
    S.tiles_x = (cams[i].width + 7) / 8;
    int64_t tiles_y = (cams[i].height + 7) / 8;
    uint64_t items = (uint64_t)S.tiles_x * (uint64_t)tiles_y * 64ull * (uint64_t)spp[i];
    S.s0 = (uint32_t)o.sample_offset;
    S.entry0 = entry;
    S.pix0 = px;
    const tet_grid* g = grids[i];
    if (g->model) S.rec = use32 ? (const void*)g->mrec32 : (const void*)g->mrec;
    else S.rec = use32 ? (const void*)g->rec32 : (const void*)g->rec;
    set_ext(S.ex, g, o);
    if (o.channels || g->model) B->ext = true;
    if (g->model) B->model = true;
    S.keys = g->keys;
    S.kidx = g->kidx;
    S.kbits = g->kbits;
    S.n = g->n;
    S.dmax = g->max_depth;
    S.out = outs[i];
    entry += items;
    px += (uint64_t)cams[i].width * (uint64_t)cams[i].height;
    if (items >= (1ull << 32) || entry >= (1ull << 32))
      return fail(TET_ERR_INVALID_ARG, "render batch: more than 2^32 samples in one batch");
  }
  B->total_px = px;
  B->table = (SceneDesc*)dev_alloc(sizeof(SceneDesc) * (size_t)n);
  RenderArgs& A = B->A;
  memset(&A, 0, sizeof(A));
  const size_t ent_bytes =
      (kHeadBytes + (size_t)entry * sizeof(RayEntry) + 4 * set_lists(A, entry) + 255) & ~(size_t)255;
  QueuePlan qp = {64, 0, 0};
  size_t lq_bytes = 0;
  size_t sort_bytes = 0;
  if (o.max_steps_per_path >= 0x7FFFFFFF) {  // light rays queued
    qp = light_queue((int64_t)entry, o);
    lq_bytes = (size_t)qp.records() * sizeof(LightRec);
    int64_t cells = 0, most = 0;
    for (int i = 0; i < n; i++) {
      cells += grids[i]->n;
      most = std::max(most, grids[i]->n);
    }
    if (sort_pays(cells, (int64_t)entry)) {
      B->ls.bits = key_bits(most, n);
      sort_bytes = B->ls.place(qp.records(), nullptr);
      if (!sort_bytes) return fail(TET_ERR_DEVICE, "render batch: light-ray sort size");
    }
  }
  B->scratch = (char*)dev_alloc(ent_bytes + lq_bytes + sort_bytes);
  if (!B->scratch && lq_bytes) {  // no room for the queue: the lanes walk their own light rays
    qp.chunks = 0;
    sort_bytes = 0;
    B->scratch = (char*)dev_alloc(ent_bytes);
  }
  if (hipHostMalloc((void**)&B->pinned, sizeof(SceneDesc) * (size_t)n, hipHostMallocDefault) != hipSuccess) {
    (void)hipGetLastError();
    B->pinned = nullptr;
  }
  if (!B->table || !B->scratch || !B->pinned) return fail(TET_ERR_OUT_OF_MEMORY, "render batch: device memory");
  memcpy(B->pinned, host.data(), sizeof(SceneDesc) * (size_t)n);
  set_queue(A, qp, B->scratch + ent_bytes);
  A.chain = 1;
  B->queue_rays = qp.sure();
  if (sort_bytes) (void)B->ls.place(qp.records(), B->scratch + ent_bytes + lq_bytes);
  A.max_bounces = o.max_bounces;
  A.transmittance = o.transmittance;
  A.max_steps = (uint32_t)std::min<int64_t>(o.max_steps_per_path, 0x7FFFFFFF);
  A.batch = 64;
  A.event_wait = o.event_wait ? o.event_wait : (B->ext ? 32 : 48);
  A.head = (uint32_t*)B->scratch;
  A.entries = (RayEntry*)(B->scratch + kHeadBytes);
  A.list = (uint32_t*)(A.entries + entry);
  A.scenes = B->table;
  A.nscenes = n;
  A.total_entries = entry;
  B->bs = o.block_size ? o.block_size : 256;
  int bpc = o.blocks_per_cu ? o.blocks_per_cu : 8;
  B->grid = (int)std::max<int64_t>(1, std::min<int64_t>((int64_t)cu_count() * bpc, ((int64_t)entry + B->bs - 1) / B->bs));
  return TET_OK;
}

template <class Med>
static void batch_trace(const BatchState* B, const RenderArgs& A, const Med& m, hipStream_t st) {
  if (B->ext) hipLaunchKernelGGL((k_render<Med, 5, 0, true, true>), dim3((unsigned)B->grid), dim3(B->bs), 0, st, A, m);
  else hipLaunchKernelGGL((k_render<Med, 5, 0, true>), dim3((unsigned)B->grid), dim3(B->bs), 0, st, A, m);
}

static void batch_resolve(const BatchState* B, hipStream_t st) {
  hipLaunchKernelGGL(k_resolve_batch, dim3((unsigned)((B->total_px + 255) / 256)), dim3(256), 0, st, B->A, B->total_px);
}

// The frame's kernels (no host synchronisation, no memset: capturable).
template <class Med>
static int batch_enqueue(const BatchState* B, hipStream_t st) {
  const RenderArgs& A = B->A;
  const Med m{nullptr, nullptr, 0, 0, B->shapes, nullptr, 0};
  hipLaunchKernelGGL(k_zero_u32, dim3((kPassWords + 255) / 256), dim3(256), 0, st, A.head, kPassWords);
  zero_stats(A.head, st);
  launch_first<Med, true>(A, m, B->model, st);
  batch_trace(B, A, m, st);
  if (!A.defer) batch_resolve(B, st);
  TV_HIP(hipGetLastError());
  return TET_OK;
}

// The frame's queued light rays, their terms into the samples, the paths that
// found the queue full, and the images (they follow the frame's kernels: the
// sort waits for the number of rays).
template <class Med>
static int batch_light(BatchState* B, hipStream_t st) {
  const RenderArgs& A = B->A;
  if (!A.defer) return TET_OK;
  const Med m{nullptr, nullptr, 0, 0, B->shapes, nullptr, 0};
  if (int rc = walk_light_queue<Med, true>(m, A, B->model, B->ls, st)) return rc;
  sum_chains<true>(A, A.total_entries, st);
  if ((int64_t)A.total_entries * A.max_bounces > B->queue_rays) {
    RenderArgs R = A;
    R.defer = 0;
    R.resume = 1;
    batch_trace(B, R, m, st);
  }
  batch_resolve(B, st);
  TV_HIP(hipGetLastError());
  return TET_OK;
}

// One frame: new seeds into the table, then the kernels (eagerly, or the
// captured graph), then the counters.
static int batch_run(BatchState* B, const uint64_t* seeds, hipStream_t st, tet_render_stats* stats) {
  if (!seeds) return fail(TET_ERR_INVALID_ARG, "render batch: seeds is NULL");
  for (int i = 0; i < B->n; i++) B->pinned[i].seed = seeds[i];
  hipEvent_t e0, e1;
  TV_HIP(hipEventCreate(&e0));
  TV_HIP(hipEventCreate(&e1));
  struct Ev {
    hipEvent_t a, b;
    ~Ev() {
      (void)hipEventDestroy(a);
      (void)hipEventDestroy(b);
    }
  } ev{e0, e1};
  TV_HIP(hipMemcpyAsync(B->table, B->pinned, sizeof(SceneDesc) * (size_t)B->n, hipMemcpyHostToDevice, st));
  TV_HIP(hipEventRecord(e0, st));
  if (B->exec) {
    TV_HIP(hipGraphLaunch(B->exec, st));
  } else if (int rc = B->use32 ? batch_enqueue<TetMedium32>(B, st) : batch_enqueue<TetMedium>(B, st)) {
    return rc;
  }
  if (int rc = B->use32 ? batch_light<TetMedium32>(B, st) : batch_light<TetMedium>(B, st)) return rc;
  TV_HIP(hipEventRecord(e1, st));
  HostStats hs;
  TV_HIP(hs.fetch(B->A.head, st));
  float ms = 0.0f;
  TV_HIP(hipEventElapsedTime(&ms, e0, e1));
  if (stats) {
    memset(stats, 0, sizeof(*stats));
    stats->tet_steps = hs.sum(0);
    stats->null_collisions = hs.sum(1);
    stats->real_collisions = hs.sum(2);
    stats->escapes = hs.sum(3);
    stats->truncated = hs.sum(4);
    stats->ms = ms;
    stats->trace_ms = ms;
    stats->light_rays_queued = hs.sum(6);
  }
  return TET_OK;
}

int render_batch(int32_t n, const tet_grid* const* grids, const tet_camera* cams, const tet_medium* media,
                 const tet_light* lights, const int32_t* spp, const uint64_t* seeds, const tet_render_opts* opts,
                 float* const* outs, hipStream_t st, tet_render_stats* stats) {
  BatchState B;
  if (int rc = batch_setup(&B, n, grids, cams, media, lights, spp, opts, outs)) return rc;
  return batch_run(&B, seeds, st, stats);
}

int batch_create(int32_t n, const tet_grid* const* grids, const tet_camera* cams, const tet_medium* media,
                 const tet_light* lights, const int32_t* spp, const tet_render_opts* opts, float* const* outs,
                 void** out) {
  if (!out) return fail(TET_ERR_INVALID_ARG, "tet_batch_create: out is NULL");
  *out = nullptr;
  BatchState* B = new BatchState();
  if (int rc = batch_setup(B, n, grids, cams, media, lights, spp, opts, outs)) {
    delete B;
    return rc;
  }
  // capture the frame's kernels once; frames replay the graph
  hipError_t e = hipStreamCreateWithFlags(&B->cap, hipStreamNonBlocking);
  if (e == hipSuccess) e = hipStreamBeginCapture(B->cap, hipStreamCaptureModeThreadLocal);
  if (e != hipSuccess) {
    delete B;
    return fail(TET_ERR_DEVICE, std::string("tet_batch_create: capture: ") + hipGetErrorString(e));
  }
  int rc = B->use32 ? batch_enqueue<TetMedium32>(B, B->cap) : batch_enqueue<TetMedium>(B, B->cap);
  hipGraph_t g = nullptr;
  e = hipStreamEndCapture(B->cap, &g);
  B->graph = g;
  if (rc || e != hipSuccess) {
    delete B;
    return rc ? rc : fail(TET_ERR_DEVICE, std::string("tet_batch_create: capture: ") + hipGetErrorString(e));
  }
  e = hipGraphInstantiate(&B->exec, B->graph, nullptr, nullptr, 0);
  if (e != hipSuccess) {
    B->exec = nullptr;
    delete B;
    return fail(TET_ERR_DEVICE, std::string("tet_batch_create: instantiate: ") + hipGetErrorString(e));
  }
  *out = B;
  return TET_OK;
}

int batch_render(void* b, const uint64_t* seeds, hipStream_t st, tet_render_stats* stats) {
  if (!b) return fail(TET_ERR_INVALID_ARG, "tet_batch_render: batch is NULL");
  return batch_run((BatchState*)b, seeds, st, stats);
}

void batch_free(void* b) { delete (BatchState*)b; }

int batch_device(const void* b) { return b ? ((const BatchState*)b)->device : 0; }

int locate_points(const tet_grid* g, const float* pts, int64_t count, int64_t* out, int32_t on_device,
                  hipStream_t st) {
  if (!g || count < 0 || (count && (!pts || !out))) return fail(TET_ERR_INVALID_ARG, "tet_locate: bad arguments");
  if (count == 0) return TET_OK;
  const uint32_t* shapes = shape_table();
  if (!shapes) return fail(TET_ERR_DEVICE, "tet_locate: shape table");
  const float* dp = pts;
  int64_t* dout = out;
  char* tmp = nullptr;
  if (!on_device) {
    tmp = (char*)dev_alloc(count * 12 + count * 8 + 16);
    if (!tmp) return fail(TET_ERR_OUT_OF_MEMORY, "tet_locate: scratch");
    dout = (int64_t*)tmp;
    dp = (const float*)(tmp + count * 8);
    TV_HIP(hipMemcpyAsync((void*)dp, pts, count * 12, hipMemcpyHostToDevice, st));
  }
  struct Free {
    void* p;
    ~Free() { if (p) dev_free(p); }
  } f_{tmp};
  TetMedium m{g->rec, g->keys, g->n, g->max_depth, shapes, g->kidx, g->kbits};
  hipLaunchKernelGGL(k_locate, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st, m, dp, count, dout);
  TV_HIP(hipGetLastError());
  if (!on_device) TV_HIP(hipMemcpyAsync(out, dout, count * 8, hipMemcpyDeviceToHost, st));
  TV_HIP(hipStreamSynchronize(st));
  return TET_OK;
}

// The tracer's elementary functions at given arguments (fn: 0 -ln(1 - a),
// 1 e^-a, 2 (cos, sin)(2 pi a) into out[2i], out[2i + 1], 3 the HG density
// of cosine a for g = b, 4 the HG inverse CDF at a for g = b).
__global__ void k_eval_functions(int fn, int64_t n, const float* __restrict__ a, const float* __restrict__ b,
                                 float* __restrict__ out) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float x = a[i];
  switch (fn) {
    case 0: out[i] = exp_tau(x); break;
    case 1: out[i] = exp_neg(x); break;
    case 2: sincos_2pi(x, out[2 * i], out[2 * i + 1]); break;
    case 3: out[i] = hg_pdf(b[i], x); break;
    default: out[i] = hg_mu(b[i], x); break;
  }
}

int eval_functions(int32_t fn, int64_t n, const float* a, const float* b, float* out, int32_t on_device,
                   hipStream_t st) {
  if (fn < 0 || fn > 4 || n < 0 || n > (1ll << 30) || (n && (!a || !out || (fn >= 3 && !b))))
    return fail(TET_ERR_INVALID_ARG, "tet_eval_functions: bad arguments");
  if (n == 0) return TET_OK;
  const int64_t nout = fn == 2 ? 2 * n : n, nin = fn >= 3 ? 2 * n : n;
  const float *da = a, *db = b;
  float* dout = out;
  char* tmp = nullptr;
  if (!on_device) {
    tmp = (char*)dev_alloc((size_t)(nin + nout) * 4);
    if (!tmp) return fail(TET_ERR_OUT_OF_MEMORY, "tet_eval_functions: scratch");
    float* ta = (float*)tmp;
    TV_HIP(hipMemcpyAsync(ta, a, n * 4, hipMemcpyHostToDevice, st));
    if (fn >= 3) TV_HIP(hipMemcpyAsync(ta + n, b, n * 4, hipMemcpyHostToDevice, st));
    da = ta;
    db = ta + n;
    dout = ta + nin;
  }
  struct Free {
    void* p;
    ~Free() { if (p) dev_free(p); }
  } f_{tmp};
  hipLaunchKernelGGL(k_eval_functions, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, (int)fn, n, da,
                     fn >= 3 ? db : nullptr, dout);
  TV_HIP(hipGetLastError());
  if (!on_device) TV_HIP(hipMemcpyAsync(out, dout, nout * 4, hipMemcpyDeviceToHost, st));
  TV_HIP(hipStreamSynchronize(st));
  return TET_OK;
}

}  // namespace tv
