// Device-resident mesh step (Section III-A: Delaunay triangulation of the
// support points, one slanted plane per triangle). The paper's CPU/FPGA split
// (Section IV) leaves this sequential step to the CPU; here it runs on the
// GPU so that a frame needs no host round trip.
//
// Every point works out its own part of the mesh, independently of all
// others, so the step spreads over the whole chip. A point p is ordered by
// (v, u); the mesh of the list points and the four image corners is the
// union, over the list points p, of the triangles whose smallest list point
// is p, plus the one triangle on the top image side (two corners and its
// apex, no list point can be smaller than another there). p's triangles lie
// between p and its larger neighbours:
//  1. first neighbour: among the points below p's row, the one whose circle
//     through p tangent to p's row is smallest. That circle lies below the row
//     and is empty, so the edge is in the mesh; p is the (v, u)-smallest point
//     on it, so on ties every tied edge is (the canonical fan, see 2).
//  2. from there p's neighbours are walked in both directions: the next
//     neighbour after q is the point r on that side of (p, q) with the smallest
//     circle through p, q, r, that is, the smallest N / D with N = (r-p).(r-q)
//     and D = (q-p) x (r-p) > 0. On ties (co-circular points) the canonical
//     mesh splits the cell as a fan from its (v, u)-smallest point: r is that
//     point if it is smaller than p, else the first one in walking order. The
//     walk stops at a smaller list point (whose triangle it is) or after a top
//     corner.
// Corner stars are never walked: their degree grows with the image border.
// k_mesh does the walks and stores each point's triangles and counts; k_tris
// turns the counts into canonical positions (triangles sorted by their sorted
// vertices: first those of the two top corners, then each point's own) and
// writes records, planes and raster triangles.
//
// Points are 32-bit keys v << 20 | u << 8 | (d - dmin): key order is (v, u)
// order. N and D are exact in int32 (coordinates below 4096); the smallest
// N / D is found in FP32 and every candidate within its error bound (relative
// 2^-19, several times the error of two conversions, a reciprocal and a
// product) is compared exactly by cross products in fp64 (below 2^53).
//
// Search. A wavefront takes one point at a time, lists the points of a box a
// few point spacings around it once (the spacing follows from the image's own
// point count), one or two per lane and relative to p, and runs the searches
// of its walks over them, each one evaluation per listed point and a
// wavefront minimum. A result whose circle leaves the listed box is checked
// against all points of the rows that the searched part of the circle covers.
//
// What bounds it: latency. A search is one dependent chain of ~0.4 us; a walk
// is three to nine of them, and a point beside an empty part of the image adds
// scans of ~0.8 us. k_mesh + k_tris, calls one at a time: 640x480 13 + 7 us,
// 1280x720 23 + 11 (frame after frame on a stream 17 + 9 and 27 + 13); the
// one-workgroup-per-view band triangulation with synchronous flip rounds that
// this replaced took 58 and 98. Large batches fill the chip either way, and the
// walks, whose arithmetic is the larger, gain nothing there: 32 pairs of 640x480
// 64 + 12 us (before 68), of 1242x375 98 together (88), of 1280x720 140 + 21 (113);
// about half of it is instruction issue. A walk is serial in its point's
// neighbours: one point above a row of some hundred others takes 250 us.
// Measured and slower: a tile of points per wavefront (the points along the
// border fall to few wavefronts: 43 us at 640x480), one row per lane for listing
// and scanning (26 us).
#include <algorithm>
#include <type_traits>

#include <hip/hip_ext.h>

#include "elas_internal.h"
#include "elas_wave.h"

namespace elas {
namespace {

constexpr int kMeshT = 256;        // threads per workgroup
constexpr int kMeshWaves = kMeshT / 64;
constexpr int kStagedKeys = 4096;  // point keys of a view kept in LDS (else read through L2)
constexpr int kListRegs = 2;       // listed points per lane
constexpr int kListCap = 64 * kListRegs;
constexpr int kListMin = 32;       // fewer listed points: a larger box is listed instead
// Neighbours stored with their point: word 0 the first neighbour, words 1..8
// those of the first walk, 9..15 those of the second, in walking order (a walk's
// triangle j lies between its neighbours j - 1 and j, the first neighbour being
// neighbour -1 of both). Triangles past these go to the overflow list.
constexpr int kChain = 16;
__device__ __forceinline__ int walk_first(int dir) { return dir == 0 ? 1 : 9; }
__device__ __forceinline__ int walk_held(int dir) { return dir == 0 ? 8 : 7; }
constexpr int kTriPoints = 64;     // points per step of k_tris

// ---- point keys -------------------------------------------------------------
__device__ __forceinline__ int key_u(uint32_t k) { return (int)((k >> 8) & 0xFFFu); }
__device__ __forceinline__ int key_v(uint32_t k) { return (int)(k >> 20); }
__device__ __forceinline__ int key_dd(uint32_t k) { return (int)(k & 0xFFu); }
__device__ __forceinline__ uint32_t make_key(int u, int v, int dd) {
  return ((uint32_t)v << 20) | ((uint32_t)u << 8) | (uint32_t)dd;
}

// ---- scratch of one view ------------------------------------------------------
struct MeshCounters {
  int32_t novf;    // triangles in the overflow list (cleared by the rows stage)
  uint32_t apex;   // apex of the triangle on the top image side
  int32_t pad[2];
};
struct Overflow {
  int32_t point;   // list index of the point the triangle belongs to
  uint32_t a, b;   // its two other vertices
};
struct MeshMem {
  MeshCounters* ctr;
  uint32_t* key;    // [nmax] point keys in list order
  uint32_t* count;  // [nmax][2] per walk: own triangles | with corner 0 << 28 | with corner 1 << 29
  uint32_t* chain;  // [nmax][kChain] neighbours
  Overflow* ovf;    // [2 nmax + 2]
};

__host__ __device__ inline size_t a16(size_t x) { return (x + 15) & ~(size_t)15; }

// Lays a view's scratch out from base; returns its bytes.
__host__ __device__ __forceinline__ size_t mesh_layout(char* base, int nmax, MeshMem* m) {
  const size_t n = (size_t)nmax;
  size_t off = 0;
  const size_t o_ctr = off;
  off += sizeof(MeshCounters);
  const size_t o_key = off;
  off += a16(4 * n);
  const size_t o_cnt = off;
  off += a16(8 * n);
  const size_t o_chain = off;
  off += a16(4 * kChain * n);
  const size_t o_ovf = off;
  off += a16(sizeof(Overflow) * (2 * n + 2));
  if (m) {
    m->ctr = reinterpret_cast<MeshCounters*>(base + o_ctr);
    m->key = reinterpret_cast<uint32_t*>(base + o_key);
    m->count = reinterpret_cast<uint32_t*>(base + o_cnt);
    m->chain = reinterpret_cast<uint32_t*>(base + o_chain);
    m->ovf = reinterpret_cast<Overflow*>(base + o_ovf);
  }
  return off;
}
__host__ __device__ __forceinline__ int mesh_nmax(const Geometry& g) {
  return g.lw * g.lh > 1 ? g.lw * g.lh : 1;
}

// Dynamic LDS of k_mesh: lh + 1 row starts, then the staged keys.
extern __shared__ __align__(16) uint32_t mesh_smem[];

// ---- the points of a view ---------------------------------------------------
template <bool kStaged>
struct View {
  const int32_t* rows;  // per-row lists, packed u | d << 16
  int n, lh, lw, lv0, step, dmin;
  uint32_t koff;        // LDS word of the first staged key
};

// Key of list point i (0 <= i < n): staged, or found through the row starts.
template <bool kStaged>
__device__ __forceinline__ uint32_t point_key(const View<kStaged>& V, int i) {
  if constexpr (kStaged) return mesh_smem[V.koff + (uint32_t)i];
  int lo = 0, hi = V.lh - 1;  // last row starting at or before i
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if ((int)mesh_smem[mid] <= i)
      lo = mid;
    else
      hi = mid - 1;
  }
  const int e = V.rows[(size_t)lo * V.lw + (i - (int)mesh_smem[lo])];
  return make_key(e & 0xFFFF, V.lv0 + lo * V.step, (e >> 16) - V.dmin);
}

// The points of rows [r0, r1) whose columns may lie in [c0, c1], straight from
// the row lists (views whose keys are not staged): sixteen lanes per row, four
// rows per load, kRowLoads loads in flight. f(first row, i, key, in) gets the
// lane's kRowLoads list positions and keys (with in false where a row has no
// such point) and returns true to end the traversal; the result is the first
// row of the step it ended in, or r1. A row is sorted by column: where rows are
// long, its sixteen lanes first look at sixteen positions spread over it, and
// it is read from the last of them left of the columns, until they are passed.
// (By list position, each key found by a binary search among the row starts,
// the mesh of 8 pairs of 640x480 with 7200 points a view took 1700 us instead of
// 340, one such frame 447 instead of 125, one of 2560x1440 with 4200 points 326
// instead of 158.)
constexpr int kRowLoads = 2;
template <class F>
__device__ __forceinline__ int each_in_rows(const View<false>& V, int r0, int r1, int c0, int c1,
                                            int lane, const F& f) {
  const int sub = lane >> 4, pos = lane & 15;
  const bool spread = V.n > 32 * V.lh;  // rows of more than 32 points on average
  for (int rb = r0; rb < r1; rb += 4 * kRowLoads) {
    int start[kRowLoads], cnt[kRowLoads], j[kRowLoads];
    uint32_t row[kRowLoads], vkey[kRowLoads];  // the row's list and its keys' v part
#pragma unroll
    for (int k = 0; k < kRowLoads; ++k) {
      const int l = min(rb + 4 * k + sub, V.lh - 1);
      start[k] = (int)mesh_smem[l];
      cnt[k] = (int)mesh_smem[l + 1] - start[k];
      cnt[k] = rb + 4 * k + sub < r1 ? cnt[k] : 0;
      row[k] = (uint32_t)l * (uint32_t)V.lw;
      vkey[k] = make_key(0, V.lv0 + l * V.step, 0);
      j[k] = pos;
    }
    if (spread) {
      int e[kRowLoads];
#pragma unroll
      for (int k = 0; k < kRowLoads; ++k) e[k] = V.rows[row[k] + (uint32_t)((pos * cnt[k]) >> 4)];
#pragma unroll
      for (int k = 0; k < kRowLoads; ++k) {
        const unsigned long long m = __builtin_amdgcn_ballot_w64((e[k] & 0xFFFF) < c0);
        const uint32_t half = lane < 32 ? (uint32_t)m : (uint32_t)(m >> 32);
        const int left = __popc((half >> (16 * (sub & 1))) & 0xFFFFu);  // positions left of c0
        j[k] += left > 0 ? ((left - 1) * cnt[k]) >> 4 : 0;
      }
    }
    for (;;) {
      int i[kRowLoads], e[kRowLoads];
      uint32_t key[kRowLoads];
      bool in[kRowLoads];
      int more = 0;
#pragma unroll
      for (int k = 0; k < kRowLoads; ++k) {
        in[k] = j[k] < cnt[k];
        i[k] = start[k] + j[k];
        e[k] = V.rows[row[k] + (uint32_t)(in[k] ? j[k] : 0)];
        j[k] += 16;
      }
#pragma unroll
      for (int k = 0; k < kRowLoads; ++k) {
        const int u = e[k] & 0xFFFF;
        key[k] = ((uint32_t)u << 8) + (vkey[k] + (uint32_t)((e[k] >> 16) - V.dmin));
        more |= (int)in[k] & (int)(u <= c1);
      }
      if (f(rb, i, key, in)) return rb;
      if (!__builtin_amdgcn_ballot_w64(more != 0)) break;
    }
  }
  return r1;
}

// ---- one search --------------------------------------------------------------
// Wavefront-uniform. A candidate at d from p has N = d . (d - e) and D = f x d.
// Neighbour after q: e = q - p, f = sgn * e. First neighbour: e = 0, f = (1, 0)
// (the tangent circle; its radius is N / 2D like below).
struct Search {
  uint32_t pkey;
  int pu, pv, ex, ey, fx, fy, sgn;
};
struct Best {
  uint32_t key;
  int N, D;
  bool any;
};
constexpr float kNone = __builtin_inff();

// d = (x, y), sq = d . d
__device__ __forceinline__ float evaluate(const Search& S, int x, int y, int sq, int* N, int* D) {
  *D = __mul24(S.fx, y) - __mul24(S.fy, x);
  *N = sq - (__mul24(x, S.ex) + __mul24(y, S.ey));
  const float t = (float)*N * __builtin_amdgcn_rcpf((float)*D);
  return *D > 0 ? t : kNone;
}

__device__ __forceinline__ float wave_min_f32(float x) {
  const uint32_t b = __float_as_uint(x);
  const uint32_t o = b ^ ((uint32_t)((int32_t)b >> 31) | 0x80000000u);
  const uint32_t m = wave_min_u32(o);
  return __uint_as_float((m & 0x80000000u) ? (m ^ 0x80000000u) : ~m);
}

// The error bound of a computed N / D, as an upper end for the true minimum's ties.
__device__ __forceinline__ float close_to(float t) { return t + fabsf(t) * 0x1p-19f; }

// Offers the candidates of the lanes in mask, exactly compared.
__device__ __forceinline__ void offer(const Search& S, unsigned long long mask, uint32_t key,
                                      int N, int D, Best* B) {
  while (mask) {
    const int lane = __ffsll((long long)mask) - 1;
    mask &= mask - 1;
    const uint32_t k = (uint32_t)__builtin_amdgcn_readlane((int)key, lane);
    const int n = __builtin_amdgcn_readlane(N, lane), d = __builtin_amdgcn_readlane(D, lane);
    if (B->any) {
      const double x = (double)n * (double)B->D, y = (double)B->N * (double)d;
      bool take = x < y;
      if (x == y) {  // co-circular: the smallest if below p, else the first in walking order
        const uint32_t c = B->key;
        if (min(k, c) < S.pkey) {
          take = k < c;
        } else {
          const int kx = key_u(k) - S.pu, ky = key_v(k) - S.pv;
          const int cx = key_u(c) - S.pu, cy = key_v(c) - S.pv;
          take = S.sgn * (kx * cy - ky * cx) > 0;
        }
      }
      if (!__builtin_amdgcn_readfirstlane(take ? 1 : 0)) continue;
    }
    B->key = k;
    B->N = n;
    B->D = d;
    B->any = true;
  }
}

// A computed circle through p: centre p + c with c = e / 2 + (t / 2) (-fy, fx).
struct Circle {
  float cx, cy, R;
};
__device__ __forceinline__ Circle circle_of(const Search& S, float t) {
  Circle C;
  C.cx = 0.5f * ((float)S.ex - t * (float)S.fy);
  C.cy = 0.5f * ((float)S.ey + t * (float)S.fx);
  C.R = __builtin_amdgcn_sqrtf(C.cx * C.cx + C.cy * C.cy);
  return C;
}

// The lattice rows that hold points of the searched part of the circle, f x d >
// 0, and its columns [c0, c1]. Each of the circle's four ends counts if it
// lies on that side (or nearly), else the chord's end does; the margins are
// far above the FP32 error of these few operations.
struct Extent {
  int r0, r1, c0, c1;
};
template <bool kStaged>
__device__ __forceinline__ Extent extent_of(const View<kStaged>& V, const Search& S, const Circle& C) {
  const float r = C.R * 1.001f + 1.0f, fx = (float)S.fx, fy = (float)S.fy;
  const float ex = (float)S.ex, ey = (float)S.ey;
  const float slack = 0.002f * C.R * (fabsf(fx) + fabsf(fy)) + fabsf(fx) + fabsf(fy);
  const float mid = fx * C.cy - fy * C.cx;  // f x c
  float x0 = fminf(0.0f, ex) - 1.0f, x1 = fmaxf(0.0f, ex) + 1.0f;
  float y0 = fminf(0.0f, ey) - 1.0f, y1 = fmaxf(0.0f, ey) + 1.0f;
  if (mid + fy * C.R > -slack) x0 = C.cx - r;  // the left end: d = c + (-R, 0)
  if (mid - fy * C.R > -slack) x1 = C.cx + r;
  if (mid - fx * C.R > -slack) y0 = C.cy - r;
  if (mid + fx * C.R > -slack) y1 = C.cy + r;
  auto to_int = [](float x) {
    return __builtin_amdgcn_readfirstlane((int)fminf(fmaxf(x, -16384.0f), 16384.0f));
  };
  const int v0 = to_int(y0) - 1 + S.pv - V.lv0, v1 = to_int(y1) + 1 + S.pv - V.lv0;
  Extent E;
  E.c0 = to_int(x0) - 1 + S.pu;
  E.c1 = to_int(x1) + 1 + S.pu;
  E.r0 = min(max(0, v0) / V.step, V.lh);
  E.r1 = max(E.r0, min(V.lh, max(0, v1) / V.step + 1));
  return E;
}

// The points of the extent's rows against *B. Most ranges hold none in the
// circle, so they are first only tested for that, 64 kScan points at a time (N
// against the bound times D, no division). From the first hit on every lane
// keeps its best point and how close its second came; only if some lane's
// second is within the error bound too (ties that fell into one lane) are the
// points gone through once more.
constexpr int kScan = 2;
__device__ __forceinline__ void scan_points(const View<true>& V, const Search& S, const Extent& E,
                                            int lane, Best* B) {
  int lo = __builtin_amdgcn_readfirstlane((int)mesh_smem[E.r0]);
  const int hi = __builtin_amdgcn_readfirstlane((int)mesh_smem[E.r1]);
  const float th = close_to((float)B->N * __builtin_amdgcn_rcpf((float)B->D));
  for (;; lo += 64 * kScan) {
    if (lo >= hi) return;
    bool hit = false;
#pragma unroll
    for (int q = 0; q < kScan; ++q) {
      const int i = lo + 64 * q + lane;
      const uint32_t k = point_key(V, min(i, V.n - 1));
      const int x = key_u(k) - S.pu, y = key_v(k) - S.pv;
      const int D = __mul24(S.fx, y) - __mul24(S.fy, x);
      const int N = __mul24(x, x - S.ex) + __mul24(y, y - S.ey);
      hit |= i < hi && D > 0 && (float)N <= th * (float)D && k != B->key;
    }
    if (__builtin_amdgcn_ballot_w64(hit)) break;
  }
  auto eval = [&](int i, uint32_t* k, int* N, int* D) {
    *k = point_key(V, min(i, V.n - 1));
    const int x = key_u(*k) - S.pu, y = key_v(*k) - S.pv;
    const float t = evaluate(S, x, y, __mul24(x, x) + __mul24(y, y), N, D);
    return i < hi ? t : kNone;
  };
  float t1 = kNone, t2 = kNone;
  uint32_t key = 0u;
  int N = 0, D = 1;
#pragma unroll 4
  for (int base = lo; base < hi; base += 64) {
    uint32_t k;
    int n, d;
    const float t = eval(base + lane, &k, &n, &d);
    t2 = fminf(t2, fmaxf(t1, t));
    const bool less = t < t1;
    key = less ? k : key;
    N = less ? n : N;
    D = less ? d : D;
    t1 = less ? t : t1;
  }
  const float thr = close_to(fminf(wave_min_f32(t1), th));
  if (!__builtin_amdgcn_ballot_w64(t2 <= thr)) {
    offer(S, __builtin_amdgcn_ballot_w64(t1 <= thr), key, N, D, B);
    return;
  }
  for (int base = lo; base < hi; base += 64) {
    const float t = eval(base + lane, &key, &N, &D);
    offer(S, __builtin_amdgcn_ballot_w64(t <= thr), key, N, D, B);
  }
}

// The same where the keys are not staged, over the extent's columns only.
__device__ __forceinline__ void scan_points(const View<false>& V, const Search& S, const Extent& E,
                                            int lane, Best* B) {
  const float th = close_to((float)B->N * __builtin_amdgcn_rcpf((float)B->D));
  const uint32_t best = B->key;
  const int first = each_in_rows(
      V, E.r0, E.r1, E.c0, E.c1, lane,
      [&](int, const int(&)[kRowLoads], const uint32_t(&k)[kRowLoads], const bool(&in)[kRowLoads]) {
        int hit = 0;
#pragma unroll
        for (int q = 0; q < kRowLoads; ++q) {
          const int x = key_u(k[q]) - S.pu, y = key_v(k[q]) - S.pv;
          const int D = __mul24(S.fx, y) - __mul24(S.fy, x);
          const int N = __mul24(x, x - S.ex) + __mul24(y, y - S.ey);
          hit |= (int)in[q] & (int)(D > 0) & (int)((float)N <= th * (float)D) & (int)(k[q] != best);
        }
        return __builtin_amdgcn_ballot_w64(hit != 0) != 0;
      });
  if (first >= E.r1) return;
  float t1 = kNone, t2 = kNone;
  uint32_t key = 0u;
  int N = 0, D = 1;
  auto eval = [&](uint32_t k, bool in, int* n, int* d) {
    const int x = key_u(k) - S.pu, y = key_v(k) - S.pv;
    const float t = evaluate(S, x, y, __mul24(x, x) + __mul24(y, y), n, d);
    return in ? t : kNone;
  };
  each_in_rows(V, first, E.r1, E.c0, E.c1, lane,
               [&](int, const int(&)[kRowLoads], const uint32_t(&k)[kRowLoads],
                   const bool(&in)[kRowLoads]) {
#pragma unroll
                 for (int q = 0; q < kRowLoads; ++q) {
                   int n, d;
                   const float t = eval(k[q], in[q], &n, &d);
                   t2 = fminf(t2, fmaxf(t1, t));
                   const bool less = t < t1;
                   key = less ? k[q] : key;
                   N = less ? n : N;
                   D = less ? d : D;
                   t1 = less ? t : t1;
                 }
                 return false;
               });
  const float thr = close_to(fminf(wave_min_f32(t1), th));
  if (!__builtin_amdgcn_ballot_w64(t2 <= thr)) {
    offer(S, __builtin_amdgcn_ballot_w64(t1 <= thr), key, N, D, B);
    return;
  }
  each_in_rows(V, first, E.r1, E.c0, E.c1, lane,
               [&](int, const int(&)[kRowLoads], const uint32_t(&k)[kRowLoads],
                   const bool(&in)[kRowLoads]) {
#pragma unroll
                 for (int q = 0; q < kRowLoads; ++q) {
                   int n, d;
                   const float t = eval(k[q], in[q], &n, &d);
                   offer(S, __builtin_amdgcn_ballot_w64(t <= thr), k[q], n, d, B);
                 }
                 return false;
               });
}

// The listed points: all points with u0 <= u < u1 in rows [l0, l1), and the
// four corners; M of them, kListRegs per lane as keys and relative to p. reach:
// a circle through p within this distance of it lies in the box.
struct List {
  uint32_t key[kListRegs];
  int x[kListRegs], y[kListRegs], sq[kListRegs];
  int M, u0, u1, l0, l1;
  float reach, reach2;  // reach2: (a little less than reach)^2
};

// One search over the listed points (the corners among them, so that both
// sides of every edge hold one) and, where the searched part of their circle
// leaves the box, all points of the rows it covers.
template <bool kStaged>
__device__ __forceinline__ uint32_t search(const View<kStaged>& V, const Search& S, const List& L, int w,
                                           int lane) {
  float t[kListRegs];
  int N[kListRegs], D[kListRegs];
  float tm = kNone;
#pragma unroll
  for (int k = 0; k < kListRegs; ++k) {
    t[k] = kNone;
    N[k] = D[k] = 0;
    if (k == 0 || 64 * k < L.M) {
      const float x = evaluate(S, L.x[k], L.y[k], L.sq[k], &N[k], &D[k]);
      t[k] = 64 * k + lane < L.M ? x : kNone;
      tm = fminf(tm, t[k]);
    }
  }
  tm = wave_min_f32(tm);
  Best B{0u, 0, 1, false};
  const float thr = close_to(tm);
#pragma unroll
  for (int k = 0; k < kListRegs; ++k)
    if (k == 0 || 64 * k < L.M) offer(S, __builtin_amdgcn_ballot_w64(t[k] <= thr), L.key[k], N[k], D[k], &B);
  // its diameter: e^2 (1 + t^2), or t^2 of the tangent circle
  const float e2 = (float)(S.ex * S.ex + S.ey * S.ey);
  const float dia2 = e2 == 0.0f ? tm * tm : e2 + e2 * (tm * tm);
  if (dia2 < L.reach2) return B.key;
  const Circle C = circle_of(S, tm);
  if ((C.R + fmaxf(fabsf(C.cx), fabsf(C.cy))) * 1.001f + 1.0f < L.reach) return B.key;
  const Extent E = extent_of(V, S, C);
  if (max(E.c0, 0) >= L.u0 && min(E.c1, w) < L.u1 && E.r0 >= L.l0 && E.r1 <= L.l1) return B.key;
  scan_points(V, S, E, lane, &B);
  return B.key;
}

// ---- k_mesh ----------------------------------------------------------------
// Workgroups per view (one per Geometry::mshare lattice points), the last of
// which does the view's header, corner disparities and top triangle. A single
// frame gets a wavefront per walk, two per point (its latency is then one
// walk's); batches one per point or few. The workgroup's points are spread over the view
// and its wavefronts take them as they finish: a walk along the border takes
// several times as long as one inside.
__host__ __device__ __forceinline__ int mesh_groups(const Geometry& g) {
  const int nlat = g.lw * g.lh;
  const int b = (nlat + g.mshare - 1) / g.mshare;
  return (b < 1 ? 1 : (b > 1024 ? 1024 : b)) + 1;
}
// Half side of the listed box in point spacings sqrt(w h / n): a larger box
// needs fewer scans of the rows, a smaller one fewer listed points per search.
// Single 640x480 13.3 us at 3, 14.7 at 3.5; 32 pairs 64 and 61 us.
template <bool kBatch>
constexpr float kHalo = kBatch ? 3.5f : 3.0f;
constexpr float kHaloRows = 3.0f;  // keys not staged: seven rows of a lattice, not nine

template <bool kBatch>
__device__ __forceinline__ void mesh_body(const Frame& F, int lb) {
  constexpr int kThreads = kMeshT, kWaves = kMeshWaves;
  __shared__ int s_next, s_take[kWaves];  // items of the workgroup taken so far, each wavefront's
  __shared__ uint32_t s_list[kWaves][kListCap];
  __shared__ int s_wsum[kWaves];
  const Geometry g = F.g;
  const int groups = mesh_groups(g);
  const int view = lb >= groups ? 1 : 0, group = lb - view * groups;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int32_t* cnt = F.cnt + view * g.lh;
  const int32_t* rowsL = F.rowsL;
  const int32_t* rowsR = F.rowsR;
  const int32_t* rows = view ? rowsR : rowsL;
  MeshHeader* hdr = F.hdr;
  const int dmin = F.p.dmin;
  MeshMem mem;
  mesh_layout(F.mesh_scratch + view * F.mesh_scratch_per_view, mesh_nmax(g), &mem);

  // ---- the view's points: eight lanes per lattice row, the first entries of
  // the first rows loaded together with the row counts
  constexpr int kPre = 4, kRowsStep = kThreads / 8;
  const int rl = tid >> 3, rj = tid & 7;
  int pre[kPre];
#pragma unroll
  for (int k = 0; k < kPre; ++k) {
    const int l = rl + k * kRowsStep;
    pre[k] = rows[(size_t)min(l, max(g.lh, 1) - 1) * g.lw + min(rj, max(g.lw, 1) - 1)];
  }
  int n = 0;
  for (int c0 = 0; c0 < g.lh; c0 += kThreads) {
    const int l = c0 + tid;
    const int x = l < g.lh ? cnt[l] : 0;
    const int incl = wave_scan_incl(x);
    if (lane == 63) s_wsum[wid] = incl;
    __syncthreads();
    int before = n;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const int s = s_wsum[w];
      before += w < wid ? s : 0;
      n += s;
    }
    if (l < g.lh) mesh_smem[l] = (uint32_t)(before + incl - x);
    __syncthreads();
  }
  n = __builtin_amdgcn_readfirstlane(n);
  if (tid == 0) {
    mesh_smem[g.lh] = (uint32_t)n;
    s_next = 0;
  }
  const bool special = group == groups - 1;
  if (special && tid == 0) {
    hdr->n[view] = n;
    hdr->ntri[view] = n > 0 ? 2 * n + 2 : 0;
    hdr->rounds[view] = 0;
    hdr->flips[view] = 0;
    hdr->on_device[view] = 1;
    if (n == 0) {
      hdr->status[view] = 0;
      for (int c = 0; c < 4; ++c) hdr->corners[4 * view + c] = -1;
    }
  }
  if (special && view == 0 && wid == kWaves - 1) {
    int ev = 0;
    for (int l = lane; l < g.lh; l += 64) ev += cnt[2 * g.lh + l];
    ev = wave_sum_i32(ev);
    if (lane == 0) hdr->support_evals = ev;
  }
  if (n == 0) return;
  // items: a point (batches) or one of its two walks
  constexpr int kWalks = kBatch ? 1 : 2;
  if (!special && group * (kBatch ? 1 : kWaves) >= kWalks * n) return;
  const uint32_t koff = (uint32_t)g.lh + 1u;
  const bool staged = n <= kStagedKeys;
  __syncthreads();
  if (staged) {
    for (int l = rl, k = 0; l < g.lh; l += kRowsStep, ++k) {
      const int s = (int)mesh_smem[l], c = (int)mesh_smem[l + 1] - s;
      for (int j = rj; j < c; j += 8) {
        int e;
        if (j < 8 && k < kPre)
          e = k == 0 ? pre[0] : (k == 1 ? pre[1] : (k == 2 ? pre[2] : pre[3]));
        else
          e = rows[(size_t)l * g.lw + j];
        mesh_smem[koff + (uint32_t)(s + j)] =
            make_key(e & 0xFFFF, g.lv0 + l * g.step, (e >> 16) - dmin);
      }
    }
    __syncthreads();
  }
  auto walks = [&](const auto& V, auto in_lds) {
  constexpr bool kStaged = in_lds.value;
  const uint32_t corner[4] = {0u, make_key(g.w - 1, 0, 0), make_key(0, g.h - 1, 0),
                              make_key(g.w - 1, g.h - 1, 0)};
  List L;
  // the list's keys in s_list[wid][0..M), relative to (pu, pv)
  auto load_list = [&](int pu, int pv) {
#pragma unroll
    for (int k = 0; k < kListRegs; ++k) {
      L.key[k] = s_list[wid][64 * k + lane];
      L.x[k] = key_u(L.key[k]) - pu;
      L.y[k] = key_v(L.key[k]) - pv;
      L.sq[k] = __mul24(L.x[k], L.x[k]) + __mul24(L.y[k], L.y[k]);
    }
  };
  if (lane < 4) s_list[wid][lane] = corner[lane];
  if (special) {
    // corner disparities: the nearest list point, the earlier one on ties
    for (int c = wid; c < 4; c += kWaves) {
      const int cu = key_u(corner[c]), cv = key_v(corner[c]);
      unsigned long long best = ~0ull;
      auto near = [&](int i, uint32_t k) {
        const int du = key_u(k) - cu, dv = key_v(k) - cv;
        const unsigned long long x =
            ((unsigned long long)(uint32_t)(du * du + dv * dv) << 32) | (unsigned)i;
        best = x < best ? x : best;
      };
      if constexpr (kStaged) {
        for (int i = lane; i < n; i += 64) near(i, point_key(V, i));
      } else {
        each_in_rows(V, 0, g.lh, 0, g.w, lane,
                     [&](int, const int(&i)[kRowLoads], const uint32_t(&k)[kRowLoads],
                         const bool(&in)[kRowLoads]) {
#pragma unroll
                       for (int q = 0; q < kRowLoads; ++q)
                         if (in[q]) near(i[q], k[q]);
                       return false;
                     });
      }
      best = wave_min_u64(best);
      if (lane == 0)
        hdr->corners[4 * view + c] = key_dd(point_key(V, (int)(best & 0xFFFFFFFFull))) + dmin;
    }
    // the triangle on the top image side: the walk's step from corner 1 as
    // seen from corner 0
    if (wid == 0) {
      L.M = 4;
      L.u0 = L.u1 = L.l0 = L.l1 = 0;
      L.reach = L.reach2 = 0.0f;
      load_list(0, 0);
      const uint32_t a =
          search(V, Search{0u, 0, 0, g.w - 1, 0, g.w - 1, 0, 1}, L, g.w, lane);
      if (lane == 0) mem.ctr->apex = a;
    }
    return;
  }

  int32_t* ptsL = F.ptsL;
  int32_t* ptsR = F.ptsR;
  int32_t* pts = view ? ptsR : ptsL;
  const int max_rounds = min(F.p.mesh_max_rounds, kMeshMaxRounds);
  const float half = (kStaged ? kHalo<kBatch> : kHaloRows) * __builtin_amdgcn_sqrtf((float)g.w * (float)g.h / (float)n);
  const int hu0 = max(4, __builtin_amdgcn_readfirstlane((int)half));
  // a single frame's items are its wavefronts' (static); in a batch the
  // wavefronts of a workgroup take them as they finish
  for (int item = group * kWaves + wid;; item += (groups - 1) * kWaves) {
    if constexpr (kBatch) {
      // Lane 0 takes the next one; the others read it from LDS. wave_sync is
      // convergent, so the loop is not rotated around the lane-dependent
      // branch, and it orders memory, so no lane's read is replaced by its last
      // one: a register that only lane 0 sets would let the compiler send the
      // other lanes round a loop of their own.
      wave_sync();
      if (lane == 0) s_take[wid] = atomicAdd(&s_next, 1);
      wave_sync();
      item = group + __builtin_amdgcn_readfirstlane(s_take[wid]) * (groups - 1);
    }
    if (item >= kWalks * n) break;
    const int idx = item / kWalks;
    const uint32_t p = (uint32_t)__builtin_amdgcn_readfirstlane((int)point_key(V, idx));
    const int pu = key_u(p), pv = key_v(p), pl = (pv - g.lv0) / g.step;
    // list the box around p; next to empty parts of the image (its border,
    // mostly), where the circles are large, a larger one, and in a cluster a
    // smaller one, so that the list holds it (a half side of 4 always does)
    int M, hu = hu0, hl, more = 0;
    for (;;) {
      hl = max(1, hu / g.step);  // rows
      L.l0 = max(0, pl - hl);
      L.l1 = min(g.lh, pl + hl + 1);
      L.u0 = pu - hu;
      L.u1 = pu + hu + 1;
      M = 4;
      auto list = [&](uint32_t k, bool here) {
        const int u = key_u(k);
        const bool in = here && u >= L.u0 && u < L.u1;
        const unsigned long long m = __builtin_amdgcn_ballot_w64(in);
        const int pos = (int)__builtin_amdgcn_mbcnt_hi(
            (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, (uint32_t)M));
        if (in && pos < kListCap) s_list[wid][pos] = k;
        M += __popcll(m);
      };
      if constexpr (kStaged) {
        const int b0 = __builtin_amdgcn_readfirstlane((int)mesh_smem[L.l0]);
        const int b1 = __builtin_amdgcn_readfirstlane((int)mesh_smem[L.l1]);
        constexpr int kList = 4;  // groups of 64 points at a time
        for (int base = b0; base < b1; base += 64 * kList) {
          uint32_t k[kList];
#pragma unroll
          for (int j = 0; j < kList; ++j) k[j] = point_key(V, min(base + 64 * j + lane, n - 1));
#pragma unroll
          for (int j = 0; j < kList; ++j) list(k[j], base + 64 * j + lane < b1);
        }
      } else {
        each_in_rows(V, L.l0, L.l1, L.u0, L.u1 - 1, lane,
                     [&](int, const int(&)[kRowLoads], const uint32_t(&k)[kRowLoads],
                         const bool(&in)[kRowLoads]) {
#pragma unroll
                       for (int q = 0; q < kRowLoads; ++q) list(k[q], in[q]);
                       return M > kListCap && hu > 4;  // a smaller box is listed instead
                     });
      }
      if (M > kListCap && hu > 4) {
        hu = max(4, hu * 3 / 4);
        more = 2;
      } else if (M < kListMin && M < n + 4 && more < 2) {
        hu *= 2;
        ++more;
      } else {
        break;
      }
    }
    // rows beyond the box start hl + 1 lattice rows away
    L.reach = fminf((float)hu, (float)((hl + 1) * g.step - 1));
    L.reach2 = (0.999f * L.reach - 1.0f) * (0.999f * L.reach - 1.0f);
    L.M = min(M, kListCap);
    wave_sync();
    load_list(pu, pv);
    wave_sync();

    // the first neighbour, then the walks
    const uint32_t q0 = search(V, Search{p, pu, pv, 0, 0, 1, 0, 1}, L, g.w, lane);
    if (lane == 0 && (kWalks == 1 || (item & 1) == 0)) {
      pts[3 * (size_t)idx] = pu;
      pts[3 * (size_t)idx + 1] = pv;
      pts[3 * (size_t)idx + 2] = key_dd(p) + dmin;
      mem.key[idx] = p;
      mem.chain[(size_t)idx * kChain] = q0;
    }
#pragma unroll 1
    for (int dir = kWalks == 1 ? 0 : item & 1; dir < 2; dir += kWalks) {
      const int sgn = dir == 0 ? 1 : -1;
      uint32_t mine = 0u;  // lane k: the walk's neighbour k
      int ntri = 0;
      uint32_t count = 0u;
      uint32_t q = q0;
      for (;;) {
        if (ntri >= max_rounds) {
          if (lane == 0) atomicMax(&hdr->status[view], 1);
          break;
        }
        const int ex = key_u(q) - pu, ey = key_v(q) - pv;
        const uint32_t r =
            search(V, Search{p, pu, pv, ex, ey, sgn * ex, sgn * ey, sgn}, L, g.w, lane);
        const bool top = key_v(r) == 0;
        if (r < p && !top) break;
        if (ntri < walk_held(dir)) {
          if (lane == ntri) mine = r;
        } else if (lane == 0) {
          const int o = atomicAdd(&mem.ctr->novf, 1);
          if (o < 2 * n + 2) mem.ovf[o] = Overflow{idx, q, r};
        }
        ++ntri;
        if (top) {
          count += r == corner[0] ? 1u << 28 : 1u << 29;
          break;
        }
        ++count;
        q = r;
      }
      if (lane < min(ntri, walk_held(dir)))
        mem.chain[(size_t)idx * kChain + walk_first(dir) + lane] = mine;
      if (lane == 0) mem.count[2 * (size_t)idx + dir] = count;
    }
  }
  };
  if (staged)
    walks(View<true>{rows, n, g.lh, g.lw, g.lv0, g.step, dmin, koff}, std::true_type{});
  else
    walks(View<false>{rows, n, g.lh, g.lw, g.lv0, g.step, dmin, koff}, std::false_type{});
}

// ---- k_tris -----------------------------------------------------------------
// Canonical positions and the triangles' records. Workgroups per view, each
// with a contiguous share of the points.
__host__ __device__ __forceinline__ int tris_groups(const Geometry& g) {
  const int nlat = g.lw * g.lh, per = 1024;  // points are about one in 17 of the lattice
  const int b = (nlat + per - 1) / per;
  return b < 1 ? 1 : (b > 64 ? 64 : b);
}

// A triangle of point p with other vertices a, b: its vertices in order and
// the smallest one's bucket (0, 1: that top corner; 2: p).
struct Tri {
  uint32_t s0, s1, s2;
  int bucket;
};
__device__ __forceinline__ Tri sort_tri(uint32_t p, uint32_t a, uint32_t b) {
  const uint32_t x = min(a, b), y = max(a, b);
  if (key_v(x) == 0) return Tri{x, p, y, x == 0u ? 0 : 1};
  return Tri{p, x, y, 2};
}
__device__ __forceinline__ bool tri_before(const Tri& a, const Tri& b) {
  return a.bucket == b.bucket && (a.s1 < b.s1 || (a.s1 == b.s1 && a.s2 < b.s2));
}

struct TriOut {
  int32_t* recs;
  float* planes;
  RasterTri* tris;
  int h, dmin, ntri;
  int cd0, cd1, cd2, cd3;  // corner disparities
};

// Writes the triangle at canonical position pos: its record, the plane
// through its three points (exact Cramer numerators relative to the first
// vertex, one correctly rounded double division each, then FP32), and the
// raster's triangle.
__device__ __forceinline__ void write_tri(const TriOut& O, int pos, const Tri& T) {
  if (pos < 0 || pos >= O.ntri) return;
  auto disp = [&](uint32_t k) {
    const int v = key_v(k), u = key_u(k);
    if (v == 0) return u == 0 ? O.cd0 : O.cd1;
    if (v == O.h - 1) return u == 0 ? O.cd2 : O.cd3;
    return key_dd(k) + O.dmin;
  };
  const int U[3] = {key_u(T.s0), key_u(T.s1), key_u(T.s2)};
  const int W[3] = {key_v(T.s0), key_v(T.s1), key_v(T.s2)};
  const int E[3] = {disp(T.s0), disp(T.s1), disp(T.s2)};
  int32_t* rec = O.recs + 9 * (size_t)pos;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    rec[3 * q] = U[q];
    rec[3 * q + 1] = W[q];
    rec[3 * q + 2] = E[q];
  }
  // the determinants fit in int32 (coordinates below 2^12, disparity
  // differences below 2^9); nc's terms are integers below 2^38, exact in fp64
  const int du2 = U[1] - U[0], dv2 = W[1] - W[0], dd2 = E[1] - E[0];
  const int du3 = U[2] - U[0], dv3 = W[2] - W[0], dd3 = E[2] - E[0];
  const int den = __mul24(du2, dv3) - __mul24(du3, dv2);
  const int na = __mul24(dd2, dv3) - __mul24(dd3, dv2);
  const int nb = __mul24(du2, dd3) - __mul24(du3, dd2);
  const double dn = (double)den;
  const double nc =  // + 0.0: an integer zero, never the -0.0 of a product
      (double)E[0] * dn - (double)na * (double)U[0] - (double)nb * (double)W[0] + 0.0;
  const float pa = (float)__ddiv_rn((double)na, dn);
  const float pb = (float)__ddiv_rn((double)nb, dn);
  const float pc = (float)__ddiv_rn(nc, dn);
  float* pl = O.planes + 3 * (size_t)pos;
  pl[0] = pa;
  pl[1] = pb;
  pl[2] = pc;
  const bool swap = den < 0;  // den > 0: (s0, s1, s2) turns counter-clockwise in (u, v)
  RasterTri rt;
  rt.u[0] = (int16_t)U[0];
  rt.v[0] = (int16_t)W[0];
  rt.u[1] = (int16_t)(swap ? U[2] : U[1]);
  rt.v[1] = (int16_t)(swap ? W[2] : W[1]);
  rt.u[2] = (int16_t)(swap ? U[1] : U[2]);
  rt.v[2] = (int16_t)(swap ? W[1] : W[2]);
  rt.a = pa;
  rt.b = pb;
  rt.c = pc;
  O.tris[pos] = rt;
}

// Of a point's two walks: its own triangles, those with top corner c, and
// the triangles stored with the point for walk d.
__device__ __forceinline__ int walk_own(uint2 c) {
  return (int)((c.x & 0x0FFFFFFFu) + (c.y & 0x0FFFFFFFu));
}
__device__ __forceinline__ int walk_with(uint2 c, int corner) {
  return (int)(((c.x >> (28 + corner)) & 1u) + ((c.y >> (28 + corner)) & 1u));
}
__device__ __forceinline__ int walk_total(uint32_t c) {
  return (int)((c & 0x0FFFFFFFu) + (c >> 28 & 1u) + (c >> 29 & 1u));
}

__device__ __forceinline__ void tris_body(const Frame& F, int lb) {
  __shared__ int s_red[kMeshWaves][5];
  __shared__ int s_base[3][kTriPoints];           // positions before each point, per bucket
  __shared__ uint32_t s_key[kTriPoints];
  __shared__ uint2 s_cnt[kTriPoints];             // triangles of each walk
  __shared__ uint16_t s_ent[kTriPoints * (kChain - 1)];  // point | neighbour word << 8
  __shared__ uint32_t s_chain[kTriPoints][kChain + 1];
  __shared__ int s_nent, s_carry[3];
  const Geometry g = F.g;
  const int groups = tris_groups(g);
  const int view = lb >= groups ? 1 : 0, group = lb - view * groups;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  MeshHeader* hdr = F.hdr;
  int32_t* const mfail = F.mfail;
  // A view that fails leaves no triangles, so raster and dense run without a
  // plane prior; the failure is recorded in the header and, when the frame
  // has one, in its pinned host report word, which the host turns into an
  // error.
  auto fail = [&](int status) {
    hdr->status[view] = status;
    hdr->ntri[view] = 0;
    if (mfail) __hip_atomic_store(mfail, status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  };
  // everything the usual case needs (at most 64 points per workgroup, kSums
  // counts per thread) is loaded at once, whatever n turns out to be
  MeshMem mem;
  const int nmax = mesh_nmax(g);
  mesh_layout(F.mesh_scratch + view * F.mesh_scratch_per_view, nmax, &mem);
  const uint2* counts = reinterpret_cast<const uint2*>(mem.count);
  constexpr int kSums = 4;
  uint2 pre[kSums];
#pragma unroll
  for (int k = 0; k < kSums; ++k) pre[k] = counts[min(tid + k * kMeshT, nmax - 1)];
  const int early = min(group * kTriPoints + lane, nmax - 1);
  const uint2 pre_cnt = counts[early];
  const uint32_t pre_key = mem.key[early];
  static_assert(kChain == 16 && kMeshT == 4 * kTriPoints, "four words per thread");
  const uint4* chains = reinterpret_cast<const uint4*>(mem.chain);
  const uint4 pre_chain = chains[min(group * kTriPoints + (tid >> 2), nmax - 1) * 4 + (tid & 3)];
  const int novf_all = mem.ctr->novf;
  const uint32_t apex = mem.ctr->apex;
  const int n = hdr->n[view], nL = hdr->n[0], status = hdr->status[view];
  TriOut O;
  O.cd0 = hdr->corners[4 * view];
  O.cd1 = hdr->corners[4 * view + 1];
  O.cd2 = hdr->corners[4 * view + 2];
  O.cd3 = hdr->corners[4 * view + 3];
  if (n == 0) return;
  if (status != 0) {
    if (group == 0 && tid == 0) fail(status);
    return;
  }
  const int per = ((n + groups * kTriPoints - 1) / (groups * kTriPoints)) * kTriPoints;
  const int p0 = group * per, p1 = min(n, p0 + per);
  if (p0 >= n && group != 0) return;
  // sums of the counts: totals of the corner buckets, and all three before p0
  int x[5] = {0, 0, 0, 0, 0}, longest = 0;
  auto add = [&](int i, uint2 c) {
    if (i >= n) return;
    const int own = walk_own(c), w0 = walk_with(c, 0), w1 = walk_with(c, 1);
    x[0] += w0;
    x[1] += w1;
    if (i < p0) {
      x[2] += w0;
      x[3] += w1;
      x[4] += own;
    }
    longest = max(longest, own);
  };
#pragma unroll
  for (int k = 0; k < kSums; ++k) add(tid + k * kMeshT, pre[k]);
  for (int i = tid + kSums * kMeshT; i < n; i += kMeshT) add(i, counts[i]);
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    x[k] = wave_sum_i32(x[k]);
    if (lane == 0) s_red[wid][k] = x[k];
  }
  if (group == 0) {
    longest = (int)~wave_min_u32(~(uint32_t)longest);
    if (lane == 0) atomicMax(&hdr->rounds[view], longest);
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    x[k] = 0;
#pragma unroll
    for (int w = 0; w < kMeshWaves; ++w) x[k] += s_red[w][k];
  }
  const int start1 = 1 + x[0], start2 = start1 + x[1];  // bucket starts (bucket 0: the top triangle)
  if (tid == 0) {
    s_carry[0] = 1 + x[2];
    s_carry[1] = start1 + x[3];
    s_carry[2] = start2 + x[4];
  }
  {
    int32_t* recsL = F.recsL;
    int32_t* recsR = F.recsR;
    float* planesL = F.planesL;
    float* planesR = F.planesR;
    O.recs = view ? recsR : recsL;
    O.planes = view ? planesR : planesL;
    O.tris = F.tris + (view ? 2 * nL + 2 : 0);
    O.h = g.h;
    O.dmin = F.p.dmin;
    O.ntri = 2 * n + 2;
  }
  const int novf = min(novf_all, 2 * n + 2);
  if (group == 0 && tid == 0)
    write_tri(O, 0, Tri{0u, make_key(g.w - 1, 0, 0), apex, 0});
  for (int c0 = p0; c0 < p1; c0 += kTriPoints) {
    __syncthreads();
    const bool first = c0 == group * kTriPoints;
    {
      const int pt = tid >> 2, wd = 4 * (tid & 3);
      const uint4 x = first ? pre_chain : chains[(size_t)min(c0 + pt, nmax - 1) * 4 + (tid & 3)];
      s_chain[pt][wd] = x.x;
      s_chain[pt][wd + 1] = x.y;
      s_chain[pt][wd + 2] = x.z;
      s_chain[pt][wd + 3] = x.w;
    }
    if (wid == 0) {
      const int i = c0 + lane;
      uint2 c = first ? pre_cnt : counts[min(i, nmax - 1)];
      if (i >= p1) c = make_uint2(0u, 0u);
      const int tot[2] = {walk_total(c.x), walk_total(c.y)};
      s_cnt[lane] = make_uint2((uint32_t)tot[0], (uint32_t)tot[1]);
      s_key[lane] = first ? pre_key : mem.key[min(i, nmax - 1)];
      const int k[3] = {walk_with(c, 0), walk_with(c, 1), walk_own(c)};
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        const int base = s_carry[b], incl = wave_scan_incl(k[b]);
        s_base[b][lane] = base + incl - k[b];
        if (lane == 63) s_carry[b] = base + incl;
      }
      const int held = min(tot[0], walk_held(0)) + min(tot[1], walk_held(1));
      const int incl = wave_scan_incl(held);
#pragma unroll
      for (int d = 0, at = incl - held; d < 2; ++d)
        for (int j = 0; j < min(tot[d], walk_held(d)); ++j, ++at)
          s_ent[at] = (uint16_t)(lane | ((walk_first(d) + j) << 8));
      if (lane == 63) s_nent = incl;
    }
    __syncthreads();
    const int nent = s_nent;
    // the two neighbours of the triangle that ends at chain word j
    auto before = [](int j) { return j == 9 ? 0 : j - 1; };
    auto place = [&](int pt, uint32_t a, uint32_t b) {
      const uint32_t p = s_key[pt];
      const uint2 c = s_cnt[pt];
      const Tri T = sort_tri(p, a, b);
      int pos = s_base[T.bucket][pt];
#pragma unroll
      for (int d = 0; d < 2; ++d) {
        const int held = min((int)(d == 0 ? c.x : c.y), walk_held(d));
        for (int j = walk_first(d); j < walk_first(d) + held; ++j)
          pos += tri_before(sort_tri(p, s_chain[pt][before(j)], s_chain[pt][j]), T) ? 1 : 0;
      }
      if ((int)c.x > walk_held(0) || (int)c.y > walk_held(1))
        for (int j = 0; j < novf; ++j) {
          const Overflow o = mem.ovf[j];
          if (o.point == c0 + pt) pos += tri_before(sort_tri(p, o.a, o.b), T) ? 1 : 0;
        }
      write_tri(O, pos, T);
    };
    for (int e = tid; e < nent; e += kMeshT) {
      const int pt = s_ent[e] & 0xFF, j = s_ent[e] >> 8;
      place(pt, s_chain[pt][before(j)], s_chain[pt][j]);
    }
    for (int e = tid; e < novf; e += kMeshT) {
      const Overflow o = mem.ovf[e];
      if (o.point >= c0 && o.point < min(p1, c0 + kTriPoints)) place(o.point - c0, o.a, o.b);
    }
  }
  // 2n + 2 triangles in all, or the walks were inconsistent
  __syncthreads();
  if (p1 == n && tid == 0 && s_carry[2] != 2 * n + 2) fail(2);
}

// ---- kernels ------------------------------------------------------------------
__global__ __launch_bounds__(kMeshT) void k_mesh(Frame F) { mesh_body<false>(F, blockIdx.x); }
__global__ __launch_bounds__(kMeshT) void k_tris(Frame F) { tris_body(F, blockIdx.x); }

template <class Body>
__device__ __forceinline__ void batch_block(const Frame* frames, const int32_t* starts, int nf,
                                            int bpf, uint32_t bmul, const Body& body) {
  const int b = blockIdx.x;
  const int f = bpf > 0 ? (int)__umulhi((uint32_t)b, bmul) : frame_of(starts, nf, b);
  const int lb = b - (bpf > 0 ? f * bpf : starts[f]);
  body(global_frame(frames[f], reinterpret_cast<const char*>(frames)), lb);
}

__global__ __launch_bounds__(kMeshT) void k_mesh_batch(const Frame* __restrict__ frames,
                                                       const int32_t* __restrict__ starts, int nf,
                                                       int bpf, uint32_t bmul) {
  batch_block(frames, starts, nf, bpf, bmul,
              [](const Frame& F, int lb) { mesh_body<true>(F, lb); });
}
__global__ __launch_bounds__(kMeshT) void k_tris_batch(const Frame* __restrict__ frames,
                                                       const int32_t* __restrict__ starts, int nf,
                                                       int bpf, uint32_t bmul) {
  batch_block(frames, starts, nf, bpf, bmul,
              [](const Frame& F, int lb) { tris_body(F, lb); });
}

}  // namespace

size_t mesh_global_scratch_per_view(const Geometry& g) {
  return mesh_layout(nullptr, mesh_nmax(g), nullptr);
}

int32_t mesh_blocks(int32_t stage, const Geometry& g) {
  return 2 * (stage == kStageMesh ? mesh_groups(g) : tris_groups(g));
}

// A workgroup has four wavefronts and stages its view's keys first, so shares of
// a few points are the least and large ones the cheapest; between them the
// workgroups of all frames together should be one resident round (1536 is six
// per CU, seven fit): 8 pairs of 1280x720 59 us at 1536 workgroups, 67 at 3088,
// 82 at 8128; 64 pairs of 128x128 26 us at 72 points each, 45 at 384. Above 384
// points each the chip is full either way, and more rounds balance better (32
// pairs of 640x480 75 us at 384, 87 at 768).
int32_t mesh_share_batch(int64_t lattice) {
  return (int32_t)std::min<int64_t>(384, std::max<int64_t>(72, 2 * lattice / 1500));
}

size_t mesh_lds(const Geometry& g) {
  return 4 * ((size_t)g.lh + 1 + (size_t)std::min(mesh_nmax(g), kStagedKeys));
}

hipError_t launch_mesh_frame(int32_t stage, const Frame& f, hipStream_t s, hipEvent_t start,
                             hipEvent_t stop) {
  if (f.g.w > kDeviceMeshMaxSide || f.g.h > kDeviceMeshMaxSide) return hipErrorInvalidValue;
  const dim3 grid(mesh_blocks(stage, f.g)), block(kMeshT);
  auto go = [&](auto kernel, uint32_t lds) {
    if (start || stop)
      hipExtLaunchKernelGGL(kernel, grid, block, lds, s, start, stop, 0u, f);
    else
      hipLaunchKernelGGL(kernel, grid, block, lds, s, f);
  };
  if (stage == kStageMesh)
    go(k_mesh, (uint32_t)mesh_lds(f.g));
  else
    go(k_tris, 0u);
  return hipGetLastError();
}

hipError_t launch_mesh_batch(int32_t stage, const Frame* frames, const int32_t* starts, int32_t nf,
                             int32_t total, int32_t bpf, uint32_t bmul, size_t lds, hipStream_t s,
                             hipEvent_t start, hipEvent_t stop) {
  const dim3 grid(total), block(kMeshT);
  auto go = [&](auto kernel, uint32_t bytes) {
    if (start || stop)
      hipExtLaunchKernelGGL(kernel, grid, block, bytes, s, start, stop, 0u, frames, starts, nf, bpf,
                            bmul);
    else
      hipLaunchKernelGGL(kernel, grid, block, bytes, s, frames, starts, nf, bpf, bmul);
  };
  if (stage == kStageMesh)
    go(k_mesh_batch, (uint32_t)lds);
  else
    go(k_tris_batch, 0u);
  return hipGetLastError();
}

}  // namespace elas
