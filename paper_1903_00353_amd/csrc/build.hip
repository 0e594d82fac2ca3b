// Feature construction (Section 7, Section 8) for a batch of meshes: adjacency,
// normals, edge and vertex classes, polyhedron lists and the band bricks.
//
// Unlike the paper's Morton-code sort of a triangle soup (Section 7.1, 7.2) the
// input here is indexed, so the corners of all triangles are grouped by vertex
// (dealt into ranges of vertices, then counted and placed inside each range), twins
// are matched around each vertex, and edges are numbered by a prefix sum over the
// half-edges that own them (start index < end index). Every id is deterministic.
// The whole sequence is device work with no host synchronisation;
// csc_features_sync reads errors and counts back.
//
// Seven launches on one stream: k_begin, k_inputs, k_deal, k_bucket, k_vertex,
// k_edges, k_lists. Counts are summed per tile where they arise and added up by the
// blocks that need what lies before them, and the bricks and edges are numbered by
// spare blocks of k_deal and k_bucket, so that no launch only scans. (Coarse sums kept
// by atomics were slower: atomics on one cache line take 6 to 10 ns each, one after
// another, 34 us for the 5,625 wavefronts of 360,000 faces.) With a radix sort,
// separate scans and a second stream the build took 25 launches: a 20,480-face sphere
// 110 us (now 45), 360,000 faces 204 (108), a batch of 64 meshes with 1.75M faces 509
// (397), 5.2M faces 1578 (1188).
#include <string.h>

#include <new>

#include "geometry.h"
#include "internal.h"
#include "wave.h"

namespace csc {

__device__ inline d3 vload_d(const float* V, int64_t i) {
  return mkd((double)V[3 * i], (double)V[3 * i + 1], (double)V[3 * i + 2]);
}
__device__ inline f3 vload_f(const float* V, int64_t i) { return mk(V[3 * i], V[3 * i + 1], V[3 * i + 2]); }
__device__ inline uint32_t* err_word(int64_t* stats) { return (uint32_t*)&stats[ST_ERR]; }

// corner c = 3f + j (32-bit: 3F < 2^31): the corner after / before it in its face
__device__ inline int32_t next_corner(int32_t c) { int32_t j = c % 3; return c - j + (j == 2 ? 0 : j + 1); }
__device__ inline int32_t prev_corner(int32_t c) { int32_t j = c % 3; return c - j + (j == 0 ? 2 : j - 1); }
// corner c itself and the corners after / before it, from its face's record
__device__ inline float4 rec_at(const FaceRec* R, int32_t c) { return R[c / 3].c[c % 3]; }
__device__ inline float4 rec_next(const FaceRec* R, int32_t c) {
  const int32_t j = c % 3;
  return R[c / 3].c[j == 2 ? 0 : j + 1];
}
__device__ inline float4 rec_prev(const FaceRec* R, int32_t c) {
  const int32_t j = c % 3;
  return R[c / 3].c[j == 0 ? 2 : j - 1];
}
__device__ inline f3 rec_posf(float4 c) { return mk(c.x, c.y, c.z); }

constexpr int BT = 256;                   // threads of the build's blocks, and faces of a face tile
constexpr int MAX_BUCKETS = 2048;
constexpr int MAX_BUCKET_SHIFT = 13;      // at most 8192 vertices (32 KB of counters) per bucket

// sum over the block's threads, in every thread
__device__ inline int block_sum(int v, int* ws) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  __syncthreads();  // ws may still be read from an earlier sum
  if (lane == 0) ws[w] = v;
  __syncthreads();
  int t = 0;
  for (int u = 0; u < nw; u++) t += ws[u];
  return t;
}

// exclusive prefix over the block's threads; *total gets the block's sum
__device__ inline int block_prefix(int v, int* ws, int* total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  const int incl = wave_prefix_sum(v);
  __syncthreads();
  if (lane == 63) ws[w] = incl;
  __syncthreads();
  int before = 0, t = 0;
  for (int u = 0; u < nw; u++) {
    before += u < w ? ws[u] : 0;
    t += ws[u];
  }
  *total = t;
  return before + incl - v;
}

// sum of the first n tile sums (called by the whole block); sums on a 16-byte boundary
__device__ inline int tiles_before(const int32_t* __restrict__ sums, int64_t n, int* ws) {
  const int4* __restrict__ s4 = reinterpret_cast<const int4*>(sums);
  int v = 0;
#pragma unroll 4
  for (int64_t k = threadIdx.x; k < n / 4; k += blockDim.x) {
    const int4 x = s4[k];
    v += x.x + x.y + x.z + x.w;
  }
  const int64_t k = n / 4 * 4 + threadIdx.x;
  if (k < n) v += sums[k];
  return block_sum(v, ws);
}

// exclusive prefix of n tile sums in place, by one block; returns their sum. The
// array holds whole groups of SCAN_PER sums, on a 16-byte boundary; those past n are not read
// as sums.
constexpr int SCAN_PER = 16;
__device__ inline int scan_tiles(int32_t* sums, int64_t n, int* ws) {
  int carry = 0;
  for (int64_t b = 0; b < n; b += (int64_t)blockDim.x * SCAN_PER) {
    const int64_t k0 = b + (int64_t)threadIdx.x * SCAN_PER;
    int4 v[SCAN_PER / 4];
    int sum = 0, all;
#pragma unroll
    for (int q = 0; q < SCAN_PER / 4; q++) {
      v[q] = k0 < n ? reinterpret_cast<const int4*>(sums + k0)[q] : make_int4(0, 0, 0, 0);
      if (k0 + 4 * q >= n) v[q].x = 0;
      if (k0 + 4 * q + 1 >= n) v[q].y = 0;
      if (k0 + 4 * q + 2 >= n) v[q].z = 0;
      if (k0 + 4 * q + 3 >= n) v[q].w = 0;
      sum += v[q].x + v[q].y + v[q].z + v[q].w;
    }
    int at = carry + block_prefix(sum, ws, &all);
#pragma unroll
    for (int q = 0; q < SCAN_PER / 4; q++) {
      const int4 o = make_int4(at, at + v[q].x, at + v[q].x + v[q].y, at + v[q].x + v[q].y + v[q].z);
      at = o.w + v[q].w;
      if (k0 < n) reinterpret_cast<int4*>(sums + k0)[q] = o;
    }
    carry += all;
  }
  return carry;
}

// Descriptors and offset tables of a few meshes as kernel arguments: they reach the
// device with the build's first launch (a host-to-device copy costs 12 us).
constexpr int TABLE_MESHES = 4;
struct MeshTables {
  MeshDesc m[TABLE_MESHES];
  MeshDesc* md;
  int32_t *f_off, *v_off, *brick_base;
  int32_t n, nf, nv, nbt;  // meshes to write (0: the tables stand), totals
};

// the counters and brick flags (n 16-byte words at z) and the statistics zeroed, the
// tables written
__global__ __launch_bounds__(BT) void k_begin(uint4* z, int64_t n, int64_t* stats, MeshTables M) {
  if (blockIdx.x == 0) {
    if (threadIdx.x < ST_COUNT) stats[threadIdx.x] = 0;
    if ((int)threadIdx.x < M.n) {
      const int m = threadIdx.x;
      M.md[m] = M.m[m];
      M.f_off[m] = M.m[m].f_off;
      M.v_off[m] = M.m[m].v_off;
      M.brick_base[m] = M.m[m].brick_base;
    }
    if (threadIdx.x == 0 && M.n > 0) {
      M.f_off[M.n] = M.nf;
      M.v_off[M.n] = M.nv;
      M.brick_base[M.n] = M.nbt;
    }
  }
  const int64_t step = (int64_t)gridDim.x * BT;
  for (int64_t i = blockIdx.x * (int64_t)BT + threadIdx.x; i < n; i += step) z[i] = make_uint4(0u, 0u, 0u, 0u);
}

// the largest m with off[m] <= x (off ascending, off[n_meshes] > x), stepping up
// from m0 <= that m
__device__ inline int segment_from(const int32_t* __restrict__ off, int m0, int64_t x) {
  int m = m0;
  while ((int64_t)off[m + 1] <= x) m++;
  return m;
}

// Segment offsets of the corners sorted by vertex: off[v] = first position whose
// vertex is >= v (vertices without corners get empty segments), off[nv] = nh.
__global__ void k_offsets(const uint32_t* __restrict__ key, int64_t nh, int64_t nv, int32_t* off) {
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= nh) return;
  const int64_t k = key[i], kp = i > 0 ? (int64_t)key[i - 1] : -1;
  for (int64_t v = kp + 1; v <= k; v++) off[v] = (int32_t)i;
  if (i == nh - 1)
    for (int64_t v = k + 1; v <= nv; v++) off[v] = (int32_t)nh;
}

// Absorbing nearly flat features into the face prisms. A cell whose closest
// point q lies inside edge e (faces f1, f2 with unit normals n1, n2 at angle
// theta) sees q along a unit direction u perpendicular to e within theta of n1
// (or of -n1, concave side), so its projection onto f1's plane lies within
// r sin(theta) <= band h sin(theta) of q, a point of f1: it is inside f1's prism
// once the prism's side planes are moved out by that much, and there its exact
// distance to f1 is its distance to e. Likewise a cell whose closest point is
// vertex v sees it along a direction within theta_v (the cone aperture, every
// incident normal within theta_v of the pseudonormal N) of +N or -N: every
// tangent direction of the fan lies within theta_v of the plane normal to N,
// and q = v minimises the distance only if u has no positive component along
// any of them. Such a u is within 2 theta_v of +-n_f for every incident face,
// so the cell is inside the prism of f with slack band h sin(2 theta_v). When
// that slack is at most `absorb` cells the feature gets no polyhedron of its
// own and every face holding it takes the slack (rounded up, in 1/1024 cells).
// Flat features (theta = 0) already get none. Ruff vertices and hemispheres,
// and edges of unknown class, keep their polyhedra. The vertex pass keeps its
// slack code in the vertex's class word, the edge pass in a byte per edge (both
// written by the thread that owns the feature), and k_lists gives every
// face the largest code of its three edges and three vertices.

__device__ inline uint8_t slack_code(double cells, float absorb) {
  if (!(cells <= (double)absorb)) return 0;
  const double q = ceil(cells * 1024.0) + 1.0;  // one step more: never below the bound
  return (uint8_t)(q < 255.0 ? q : 255.0);
}

__device__ inline uint8_t edge_slack(d3 u, d3 w, d3 c1, d3 c2, float band, float absorb) {
  const d3 n1 = cross(w - u, c1 - u), n2 = cross(u - w, c2 - w);
  const double l = len(n1) * len(n2);
  if (!(l > 0) || !(dot(n1, n2) > 0)) return 0;  // theta >= 90 degrees
  return slack_code((double)band * len(cross(n1, n2)) / l, absorb);
}

__device__ inline uint8_t vertex_slack(const VertexClass& cl, float band, float absorb) {
  if (!(cl.bits & (V_POS | V_NEG)) || (cl.bits & (V_POS_HEMI | V_NEG_HEMI | V_RUFF))) return 0;
  const double c = cl.cos_t;
  if (!(c > 0.7071067811865476) || c > 1.0) return 0;  // 2 theta up to 90 degrees
  const double sn = sqrt(fmax(0.0, 1.0 - c * c));
  return slack_code((double)band * 2.0 * sn * c, absorb);  // band * sin(2 theta)
}

constexpr int VK_THREADS = 128;
constexpr int VK_MAXD = 12;   // fans up to this degree are staged in LDS (18 KB per block: 4 wavefronts per SIMD)
constexpr int VK_HALF = 6;    // corners whose loads are in flight together
static_assert(VK_MAXD == 2 * VK_HALF && VK_MAXD <= 16, "two halves, places in 4 bits");

// Twins around one vertex: corner i's out-edge to N(i) pairs with the one in-edge
// from P(k) = N(i); matched(k, i) hears of every such pair. Returns the error bits.
template <class C, class N, class P, class M>
__device__ inline uint32_t match_fan(int d, C c, N n, P p, M matched, int32_t* twin) {
  uint32_t e = 0;
  for (int i = 0; i < d; i++) {
    const int32_t w = n(i);
    int32_t match = -1, nmatch = 0;
    for (int k = 0; k < d; k++) {
      if (k != i && n(k) == w) e |= ERR_ORIENT;
      if (p(k) == w) {
        nmatch++;
        match = prev_corner(c(k));
        matched(k, i);
      }
    }
    if (nmatch != 1) e |= ERR_NONMANIFOLD;
    twin[c(i)] = nmatch == 1 ? match : -1;
  }
  return e;
}

// pseudonormal and tests of a vertex at pv whose corners' next and previous vertices
// lie at xn(k), xp(k)
template <class XN, class XP>
__device__ inline VertexTest test_fan(int d, d3 pv, XN xn, XP xp) {
  VertexAccum acc;
  for (int k = 0; k < d; k++) acc.add_face(pv, xn(k), xp(k));
  VertexTest vt;
  vt.init(acc.n_alpha);
  for (int k = 0; k < d; k++) {
    const d3 p1 = xn(k), p2 = xp(k);
    vt.neighbour(pv, p1);
    vt.normal(pv, p1, p2);
  }
  return vt;
}

// Twins and tests of a fan of d corners at c (ascending), read from memory again and again,
// by one lane. Code of its own: one loop for both, choosing between LDS and memory at each
// read, took 98 ms in place of 62 at a pole of 512 corners behind 240,000 faces.
__device__ inline VertexTest long_fan(const float* __restrict__ V, const int32_t* __restrict__ T,
                                      const int32_t* __restrict__ c, int d, d3 pv, int32_t* twin, int64_t* stats) {
  auto C = [&](int k) { return c[k]; };
  auto N = [&](int k) { return T[next_corner(c[k])]; };
  auto P = [&](int k) { return T[prev_corner(c[k])]; };
  const uint32_t e = match_fan(d, C, N, P, [](int, int) {}, twin);
  if (e) atomicOr(err_word(stats), e);
  return test_fan(d, pv, [&](int k) { return vload_d(V, N(k)); }, [&](int k) { return vload_d(V, P(k)); });
}

struct VertexOut {
  int ruff_mode, saddle_mode, force_both;
  const int32_t* vert_mesh;
  const MeshDesc* md;
  int n_meshes;
  float absorb;
  float4* vinfo;
  uint32_t* vbits;
};

// class, cone and slack of vertex v of degree d; returns its side bits
__device__ inline int put_vertex(const VertexOut& O, int64_t v, int d, const VertexTest& vt) {
  VertexClass cl = vt.finish(O.ruff_mode, O.saddle_mode, O.force_both);
  if (d == 0) cl.bits = 0;  // isolated vertex: no feature
  // a nearly flat vertex hands its region to the prisms of its faces (side slack
  // band * sin(2 theta), theta the cone aperture): see vertex_slack
  const uint8_t q = O.absorb > 0.f && !O.force_both
                        ? vertex_slack(cl, O.md[O.n_meshes > 1 ? O.vert_mesh[v] : 0].band, O.absorb)
                        : 0;
  if (q) cl.bits = (cl.bits & ~(V_POS | V_NEG)) | V_ABSORBED | ((uint32_t)q << V_SLACK_SHIFT);
  float cf = (float)cl.cos_t;
  if ((double)cf > cl.cos_t) cf = nextafterf(cf, -2.f);  // the stored cone contains the exact one
  O.vinfo[v] = make_float4((float)cl.axis.x, (float)cl.axis.y, (float)cl.axis.z, cf);
  O.vbits[v] = cl.bits;
  return (int)(cl.bits & (V_POS | V_NEG));
}
static_assert(V_POS == 1u && V_NEG == 2u, "side bits of the class word");

// Per vertex u, over its fan of corners in ascending order (sorted and staged in LDS, then
// replaced there by the positions of the neighbours: each is read once, six loads
// in flight together, where reading both far corners of every triangle again in
// each of the two passes below took four times the loads one after another:
// 5.2M faces 420 -> 305 us):
//  * twins: the out-edge u -> w of corner c (half-edge c) pairs with the unique
//    in-edge w -> u of another corner around u; none or several: not a closed
//    2-manifold; two out-edges to the same w: inconsistent orientation;
//  * pseudonormal N = sum alpha_i n_i (Eq. 8), class from the side of each
//    neighbour against the plane through u with normal N (Section 3.1-3.2,
//    Section 8.3), cone aperture and ruff test from the normals (Section 3.3,
//    Section 4.2), all in double precision; number of vertex polyhedra.
// Bounded by the latency of the gathers of triangle rows and positions and by its
// FP64 arithmetic (4 wavefronts per SIMD, LDS-bound). Fans of more than VK_MAXD corners,
// sorted by k_bucket, are walked in memory (long_fan).
__global__ __launch_bounds__(VK_THREADS) void k_vertex(const float* __restrict__ V, const int32_t* __restrict__ T,
                                                      int64_t nv, const int32_t* __restrict__ off,
                                                      const int32_t* __restrict__ vc, VertexOut O, int32_t* twin, int32_t* polys, int64_t* stats) {
  __shared__ int32_t s_c[VK_MAXD][VK_THREADS], s_n[VK_MAXD][VK_THREADS], s_p[VK_MAXD][VK_THREADS];
  __shared__ int s_polys[VK_THREADS / 64];
  const int t = threadIdx.x;
  const int64_t tile = xcd_block(), v = tile * VK_THREADS + t;
  int sides = 0;
  if (v < nv) {
    const int32_t s0 = off[v], d = off[v + 1] - s0;
    const bool staged = d <= VK_MAXD;
    uint64_t place = 0;  // staged: 4 bits per corner, the corner whose next vertex is this one's previous one
    if (staged && d > 0) {
      const bool more = __ballot(d > VK_HALF) != 0;
      {  // the first six in ascending order (a sorting network), the rest inserted
        int32_t c[VK_HALF];
#pragma unroll
        for (int k = 0; k < VK_HALF; k++) c[k] = vc[s0 + (k < d ? k : 0)];
#pragma unroll
        for (int k = 0; k < VK_HALF; k++) c[k] = k < d ? c[k] : INT32_MAX;
        constexpr int NET[12][2] = {{0, 5}, {1, 3}, {2, 4}, {1, 2}, {3, 4}, {0, 3},
                                    {2, 5}, {0, 1}, {2, 3}, {4, 5}, {1, 2}, {3, 4}};
#pragma unroll
        for (int k = 0; k < 12; k++) {
          const int32_t a = c[NET[k][0]], b = c[NET[k][1]];
          c[NET[k][0]] = a < b ? a : b;
          c[NET[k][1]] = a < b ? b : a;
        }
#pragma unroll
        for (int k = 0; k < VK_HALF; k++) s_c[k][t] = c[k];
      }
      if (more) {
        int32_t c[VK_HALF];
#pragma unroll
        for (int k = 0; k < VK_HALF; k++) c[k] = vc[s0 + (VK_HALF + k < d ? VK_HALF + k : 0)];
#pragma unroll
        for (int k = 0; k < VK_HALF; k++)
          if (VK_HALF + k < d) {
            int q = VK_HALF + k;
            for (; q > 0 && s_c[q - 1][t] > c[k]; q--) s_c[q][t] = s_c[q - 1][t];
            s_c[q][t] = c[k];
          }
      }
      for (int h = 0; h < (more ? VK_MAXD : VK_HALF); h += VK_HALF) {
        int32_t c[VK_HALF], a0[VK_HALF], a1[VK_HALF], a2[VK_HALF];
#pragma unroll
        for (int k = 0; k < VK_HALF; k++) {
          c[k] = s_c[h + k < d ? h + k : 0][t];
          const int32_t* row = T + (c[k] - c[k] % 3);
          a0[k] = row[0];
          a1[k] = row[1];
          a2[k] = row[2];
        }
#pragma unroll
        for (int k = 0; k < VK_HALF; k++)
          if (h + k < d) {
            const int j = c[k] % 3;
            s_n[h + k][t] = j == 0 ? a1[k] : (j == 1 ? a2[k] : a0[k]);
            s_p[h + k][t] = j == 0 ? a2[k] : (j == 1 ? a0[k] : a1[k]);
          }
      }
    }
    const d3 pv = vload_d(V, v);
    VertexTest vt;
    if (staged) {
      auto C_ = [&](int k) { return s_c[k][t]; };
      auto N_ = [&](int k) { return s_n[k][t]; };
      auto P_ = [&](int k) { return s_p[k][t]; };
      const uint32_t e = match_fan(d, C_, N_, P_, [&](int k, int i) {
        place = (place & ~(15ull << (4 * k))) | ((uint64_t)i << (4 * k));
      }, twin);
      if (e) atomicOr(err_word(stats), e);
    } else {
      vt = long_fan(V, T, vc + s0, d, pv, twin, stats);
    }
    if (staged && d > 0) {
      // positions of the next vertices in place of the ids (a corner whose previous
      // vertex is no next vertex, on a surface that is rejected, takes the first's)
      const bool more = __ballot(d > VK_HALF) != 0;
      for (int h = 0; h < (more ? VK_MAXD : VK_HALF); h += VK_HALF) {
        f3 x[VK_HALF];
#pragma unroll
        for (int k = 0; k < VK_HALF; k++) x[k] = vload_f(V, h + k < d ? s_n[h + k][t] : (int32_t)v);
#pragma unroll
        for (int k = 0; k < VK_HALF; k++)
          if (h + k < d) {
            s_c[h + k][t] = __float_as_int(x[k].x);
            s_p[h + k][t] = __float_as_int(x[k].y);
            s_n[h + k][t] = __float_as_int(x[k].z);
          }
      }
    }
    auto at = [&](int k) {
      return mkd((double)__int_as_float(s_c[k][t]), (double)__int_as_float(s_p[k][t]),
                 (double)__int_as_float(s_n[k][t]));
    };
    if (staged) vt = test_fan(d, pv, at, [&](int k) { return at((int)(place >> (4 * k)) & 15); });
    sides = put_vertex(O, v, d, vt);
  }
  const int n = __popcll(__ballot((sides & 1) != 0)) + __popcll(__ballot((sides & 2) != 0));
  if ((t & 63) == 0) s_polys[t >> 6] = n;
  __syncthreads();
  if (t == 0) {
    int sum = 0;
    for (int w = 0; w < VK_THREADS / 64; w++) sum += s_polys[w];
    polys[tile] = sum;
  }
}
// The same for meshes of few vertices: VF_LANES lanes to a vertex, one to a corner (two
// from the ninth corner on, up to VF_MAXD), so
// that a fan takes one angle and one test where a thread takes them one after
// another, and a mesh of few vertices fills more of the chip. The faces' shares of the
// pseudonormal are still added in corner order. Vertices of more corners are left to
// their first lane. polys: cleared by k_inputs. (Build of 642 vertices 43 us with a thread
// per vertex, 33 with lanes; see VERTEX_FANS for larger ones. Delaunay
// triangles of random points, 4% of the vertices of nine corners and more: with those
// left to one lane 118 us at 1,000 vertices and 237 at 65,000, with two corners a
// lane 64 and 140, build with its read-back.)
constexpr int VF_LANES = 8, VF_PER = 2, VF_MAXD = VF_LANES * VF_PER, VF_THREADS = 256, VF_WAVE = 64 / VF_LANES;
__global__ __launch_bounds__(VF_THREADS) void k_vertex_fan(const float* __restrict__ V, const int32_t* __restrict__ T,
                                                          int64_t nv, const int32_t* __restrict__ off,
                                                          const int32_t* __restrict__ vc, VertexOut O, int32_t* twin, int32_t* polys, int64_t* stats) {
  struct Fan {
    union {
      struct {
        int32_t c[VF_MAXD], n[VF_MAXD], p[VF_MAXD];
        int32_t at[VF_MAXD];        // the corner whose next vertex is this one's previous one
        float x[VF_MAXD][3];
      };
      double share[VF_MAXD][4];     // then: face normal, angle / length (0: no normal)
    };
    int32_t pad[8];  // a wavefront's eight fans lie in different LDS banks
  };
  static_assert(sizeof(Fan) % 256 == 32, "fans eight banks apart");
  __shared__ Fan s_fan[VF_THREADS / VF_LANES];
  const int sub = threadIdx.x & (VF_LANES - 1);
  const int64_t v = (blockIdx.x * (int64_t)VF_THREADS + threadIdx.x) / VF_LANES;
  Fan& S = s_fan[threadIdx.x / VF_LANES];
  const int32_t s0 = v < nv ? off[v] : 0, d = v < nv ? off[v + 1] - s0 : 0;
  const bool fan = d <= VF_MAXD;
  const int per = __ballot(fan && d > VF_LANES) != 0 ? VF_PER : 1;  // corners of a lane, the same in the wavefront
  // corners in ascending order: each one's place among the fan's
  bool mine[VF_PER];
  int32_t c[VF_PER];
#pragma unroll
  for (int h = 0; h < VF_PER; h++) {
    const int i = sub + h * VF_LANES;
    mine[h] = h < per && fan && i < d;
    c[h] = mine[h] ? vc[s0 + i] : INT32_MAX;
    S.c[i] = c[h];
    S.at[i] = 0;
  }
  wave_sync_lds();
  int place[VF_PER] = {0, 0};
#pragma unroll
  for (int h = 0; h < VF_PER; h++)
    if (h < per)
#pragma unroll
      for (int k = 0; k < VF_MAXD; k++)
        if (k < VF_LANES || per > 1) place[h] += S.c[k] < c[h] ? 1 : 0;
  wave_sync_lds();
#pragma unroll
  for (int h = 0; h < VF_PER; h++)
    if (mine[h]) S.c[place[h]] = c[h];
  wave_sync_lds();
#pragma unroll
  for (int h = 0; h < VF_PER; h++)
    if (mine[h]) {
      const int i = sub + h * VF_LANES;
      c[h] = S.c[i];
      const int32_t* row = T + (c[h] - c[h] % 3);
      const int32_t a0 = row[0], a1 = row[1], a2 = row[2];
      const int j = c[h] % 3;
      S.n[i] = j == 0 ? a1 : (j == 1 ? a2 : a0);
      S.p[i] = j == 0 ? a2 : (j == 1 ? a0 : a1);
    }
  wave_sync_lds();
  uint32_t e = 0;
  const d3 pv = vload_d(V, v < nv ? v : 0);
  d3 p1[VF_PER] = {pv, pv};
#pragma unroll
  for (int h = 0; h < VF_PER; h++)
    if (mine[h]) {
      const int i = sub + h * VF_LANES;
      const int32_t w = S.n[i];
      const f3 x = vload_f(V, w);
      int32_t match = -1, nmatch = 0;
      for (int k = 0; k < d; k++) {
        if (k != i && S.n[k] == w) e |= ERR_ORIENT;
        if (S.p[k] == w) {
          nmatch++;
          match = prev_corner(S.c[k]);
          S.at[k] = i;
        }
      }
      if (nmatch != 1) e |= ERR_NONMANIFOLD;
      twin[c[h]] = nmatch == 1 ? match : -1;
      S.x[i][0] = x.x;
      S.x[i][1] = x.y;
      S.x[i][2] = x.z;
      p1[h] = mkd(x.x, x.y, x.z);
    }
  if (e) atomicOr(err_word(stats), e);
  wave_sync_lds();
  d3 p2[VF_PER];
#pragma unroll
  for (int h = 0; h < VF_PER; h++)
    if (mine[h]) {
      const float* y = S.x[S.at[sub + h * VF_LANES]];
      p2[h] = mkd(y[0], y[1], y[2]);
    }
  wave_sync_lds();  // the shares take the place of what was read above
  d3 n[VF_PER] = {mkd(0, 0, 0), mkd(0, 0, 0)};
  double ln[VF_PER] = {0, 0};
#pragma unroll
  for (int h = 0; h < VF_PER; h++)
    if (mine[h]) {
      const d3 e1 = p1[h] - pv, e2 = p2[h] - pv;
      n[h] = cross(e1, e2);
      ln[h] = len(n[h]);
      double* share = S.share[sub + h * VF_LANES];
      share[0] = n[h].x;
      share[1] = n[h].y;
      share[2] = n[h].z;
      share[3] = ln[h] > 0 ? atan2(ln[h], dot(e1, e2)) / ln[h] : 0.0;
    }
  wave_sync_lds();
  VertexAccum acc;
  if (fan)
    for (int k = 0; k < d; k++) {
      const double q = S.share[k][3];
      if (q != 0.0) acc.n_alpha = acc.n_alpha + mkd(S.share[k][0], S.share[k][1], S.share[k][2]) * q;
    }
  VertexTest vt;
  vt.init(acc.n_alpha);
#pragma unroll
  for (int h = 0; h < VF_PER; h++)
    if (mine[h]) {
      vt.neighbour(pv, p1[h]);
      if (ln[h] > 0) {
        const double q = dot(n[h], vt.axis) / ln[h];
        if (q > 0) vt.cos_t = q < vt.cos_t ? q : vt.cos_t;
        else vt.nonpos_normal = 1;
      }
    }
  // the lanes' tests together
#pragma unroll
  for (int o = 1; o < VF_LANES; o <<= 1) {
    vt.pos += __shfl_xor(vt.pos, o, 64);
    vt.neg += __shfl_xor(vt.neg, o, 64);
    vt.unc += __shfl_xor(vt.unc, o, 64);
    vt.nonpos_normal |= __shfl_xor(vt.nonpos_normal, o, 64);
    const double q = __shfl_xor(vt.cos_t, o, 64);
    vt.cos_t = q < vt.cos_t ? q : vt.cos_t;
  }
  int sides = 0;
  if (sub == 0 && v < nv) {
    if (!fan) vt = long_fan(V, T, vc + s0, d, pv, twin, stats);
    sides = put_vertex(O, v, d, vt);
  }
  const int sum = __popcll(__ballot((sides & 1) != 0)) + __popcll(__ballot((sides & 2) != 0));
  if ((threadIdx.x & 63) == 0 && sum) atomicAdd(&polys[v / VK_THREADS], sum);
}
static_assert(VK_THREADS % VF_WAVE == 0, "a wavefront's vertices lie in one tile");

// The extrusion lists: item i (an edge or a vertex) has 0-2 polyhedra, bit 0 of its
// side mask the outward one (entry i << 1) and bit 1 the inward one ((i << 1) | 1);
// the entries follow item order. `at`: the place of this thread's first entry.
__device__ inline int put_entries(int32_t* q, int at, int64_t item, int sides) {
  if (sides & 1) q[at++] = (int32_t)item << 1;
  if (sides & 2) q[at++] = ((int32_t)item << 1) | 1;
  return at;
}

// the vertex polyhedra of QV tiles of k_vertex (block b of the list)
constexpr int QV = 16;
template <int TH>
__device__ inline void vertex_list(int64_t b, const uint32_t* __restrict__ vbits, int64_t nv,
                                   const int32_t* __restrict__ polys, int64_t tiles, int32_t* q, int64_t* total,
                                   int* ws) {
  constexpr int QV_ITEMS = QV * VK_THREADS / TH;
  static_assert(QV_ITEMS * TH == QV * VK_THREADS, "whole items per thread");
  const int offset = tiles_before(polys, b * QV, ws);
  const int64_t first = b * QV * VK_THREADS + (int64_t)threadIdx.x * QV_ITEMS;
  int m[QV_ITEMS], c = 0;
#pragma unroll
  for (int k = 0; k < QV_ITEMS; k++) {
    m[k] = first + k < nv ? (int)(vbits[first + k] & (V_POS | V_NEG)) : 0;
    c += __popc(m[k]);
  }
  int sum;
  int at = offset + block_prefix(c, ws, &sum);
#pragma unroll
  for (int k = 0; k < QV_ITEMS; k++) at = put_entries(q, at, first + k, m[k]);
  if ((b + 1) * QV >= tiles && threadIdx.x == 0) *total = offset + sum;
}

struct EdgeArgs {
  const FaceRec* rec;
  const int32_t* twin;
  const int32_t* face_mesh;
  const MeshDesc* md;
  int4* edges;
  int32_t* face_edges;
  uint8_t* cls;
  uint8_t* eslack;
  const int32_t* eid;    // [nf][3] edge id of each owned half-edge
  const uint32_t* vbits;
  int32_t* vpoly;
  int64_t* stats;
  const int32_t* vpolys;   // per tile of k_vertex
  int32_t* epolys;         // per block of this pass
  int64_t nf, ne, nv, blocks, vertex_tiles;
  float absorb;
  int n_meshes, force_both;
};

// One thread per half-edge: edge records from the owned half-edges (u -> w with
// u < w) and, for each edge, its class from the exact orientation of its four
// corners (Section 8.2: the discriminant of the two face normals, evaluated
// exactly) with the sides to extrude. The third corner of the owning face precedes u
// in that face; the third corner of the twin's face precedes the twin's start. Edges
// are numbered along the half-edges. (An open or non-manifold surface can own more or
// fewer than 3F/2 half-edges: such a build is rejected, and nothing is written past
// ne; the edges that no half-edge produced are left unclassified and empty.) The
// blocks past the half-edges' write the vertex list. Bounded by the gathers of the
// twins' corners and edge ids: the ids come from an array (edge_bases), not from a
// prefix over the block, whose barriers held the gathers back (5.2M faces: 502 us
// in blocks of 768 threads, 234 with the array).
__global__ __launch_bounds__(BT) void k_edges(EdgeArgs P) {
  __shared__ int ws[BT / 64];
  if (blockIdx.x >= P.blocks) {
    vertex_list<BT>(blockIdx.x - P.blocks, P.vbits, P.nv, P.vpolys, P.vertex_tiles, P.vpoly, &P.stats[ST_NVPOLY], ws);
    return;
  }
  const int64_t h = blockIdx.x * (int64_t)BT + threadIdx.x, f = h / 3;
  int sides = 0;
  if (f < P.nf) {
    // this face's record: the three threads of a face read one sector together
    const float4 cu = rec_at(P.rec, (int32_t)h), cw = rec_next(P.rec, (int32_t)h);
    const int32_t t = P.twin[h];
    const bool owns = rec_vertex(cu) < rec_vertex(cw);
    const int32_t id = owns ? P.eid[h] : (t >= 0 ? P.eid[t] : -1);
    P.face_edges[h] = id < P.ne ? id : -1;
    if (owns) {
      const float4 c1 = rec_prev(P.rec, (int32_t)h);
      if (id < P.ne) {
        P.edges[id] = make_int4(rec_vertex(cu), rec_vertex(cw), (int)f, t >= 0 ? t / 3 : -1);
        int k = 0;
        uint8_t q = 0;
        if (t >= 0) {
          const f3 fu = rec_posf(cu), fw = rec_posf(cw), f1 = rec_posf(c1), f2 = rec_posf(rec_prev(P.rec, t));
          k = classify_edge(fu, fw, f1, f2);
          if (k == EDGE_CONVEX) sides = 1;
          else if (k == EDGE_CONCAVE) sides = 2;
          else if (k == EDGE_UNKNOWN) sides = 3;
          if (P.force_both) sides = 3;
          // a nearly flat edge hands its wedge to its two face prisms
          if (P.absorb > 0.f && !P.force_both && (k == EDGE_CONVEX || k == EDGE_CONCAVE)) {
            q = edge_slack(tod(fu), tod(fw), tod(f1), tod(f2), P.md[P.n_meshes > 1 ? P.face_mesh[f] : 0].band,
                           P.absorb);
            if (q) sides = 0;
          }
        }
        P.eslack[id] = q;
        P.cls[id] = (uint8_t)(k | (sides << 2) | (q ? EDGE_ABSORBED : 0));
      }
    }
  }
  const int n = __popcll(__ballot(sides & 1)) + __popcll(__ballot(sides & 2));
  if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = n;
  __syncthreads();
  if (threadIdx.x == 0) P.epolys[blockIdx.x] = ws[0] + ws[1] + ws[2] + ws[3];
  if (blockIdx.x == 0)
    for (int64_t k = P.stats[ST_NE] + threadIdx.x; k < P.ne; k += BT) {
      P.edges[k] = make_int4(-1, -1, -1, -1);
      P.eslack[k] = 0;
      P.cls[k] = 0;
    }
}
static_assert(BT == 256, "three blocks of half-edges per face tile, four wavefronts each");

// Unit face normal (double precision, stored in single) and the band bricks near
// the face: the bricks holding a cell centre within band*h + eps of the face's
// bounding box, less those whose centres all lie farther than that from the
// face's plane. Every polyhedron of the face, its edges and its vertices lies in
// that box (the face prism within band*h*|n_k| + eps of the face along each
// axis, edge wedges and vertex cones within band*h + eps of their feature), and
// a scan writes only cells within band*h of a feature, so every cell a scan can
// write has its brick marked by one of the faces holding its feature.
struct FaceBox {
  d3 un, a;     // unit normal (zero: degenerate, the whole box is kept), first corner
  double ext;
  int lo[3], n[3];  // bricks (n[0] = 0: none)
};

// the record and box of face f = (ia, ib, ic)
__device__ inline FaceBox face_geom_one(const float* __restrict__ V, int64_t f, int32_t ia, int32_t ib, int32_t ic,
                                        const MeshDesc& g, FaceRec* rec, int64_t* stats) {
  const f3 af = vload_f(V, ia), bf = vload_f(V, ib), cf = vload_f(V, ic);
  const d3 a = mkd(af.x, af.y, af.z), b = mkd(bf.x, bf.y, bf.z), c = mkd(cf.x, cf.y, cf.z);
  const d3 n = cross(b - a, c - a);
  const double l = len(n);
  const bool cull = l > 0;
  FaceBox B;
  B.a = a;
  B.un = cull ? mkd(n.x / l, n.y / l, n.z / l) : mkd(0.0, 0.0, 0.0);
  if (!cull) atomicOr(err_word(stats), ERR_DEGENERATE);
  // the face's record: later passes read one aligned sector per face instead of
  // three vertex gathers
  FaceRec& o = rec[f];
  o.c[0] = make_float4(af.x, af.y, af.z, __int_as_float(ia));
  o.c[1] = make_float4(bf.x, bf.y, bf.z, __int_as_float(ib));
  o.c[2] = make_float4(cf.x, cf.y, cf.z, __int_as_float(ic));
  o.n = make_float4((float)B.un.x, (float)B.un.y, (float)B.un.z, 0.f);
  const double r = g.whd + g.epsd;
  const double X[3][3] = {{a.x, b.x, c.x}, {a.y, b.y, c.y}, {a.z, b.z, c.z}};
  bool none = false;
#pragma unroll
  for (int ax = 0; ax < 3; ax++) {
    const double x0 = X[ax][0], x1 = X[ax][1], x2 = X[ax][2];
    const double mn = fmin(x0, fmin(x1, x2)) - r, mx = fmax(x0, fmax(x1, x2)) + r;
    // cells whose centre lies in [mn, mx], widened by 1e-3 cells against rounding
    // (the scan's own boxes are widened by 1e-4 cells)
    double lo_c = ceil((mn - g.origin[ax]) * g.inv_h - 0.5 - 1e-3);
    double hi_c = floor((mx - g.origin[ax]) * g.inv_h - 0.5 + 1e-3);
    lo_c = fmax(lo_c, 0.0);
    hi_c = fmin(hi_c, (double)(g.n[ax] - 1));
    if (!(lo_c <= hi_c)) {
      none = true;
      lo_c = hi_c = 0.0;
    }
    B.lo[ax] = (int)lo_c / BRICK;
    B.n[ax] = (int)hi_c / BRICK - B.lo[ax] + 1;
  }
  if (none) B.n[0] = 0;
  // A brick is kept only if some cell centre in it can lie within r of the face's
  // plane: a cell within band*h of an edge or vertex is that close to a face
  // holding it, and no key is written farther out. The centres of brick (x, y, z)
  // fill a box of half-width (BRICK - 1) h / 2 around origin + (BRICK x + BRICK / 2) h,
  // whose distance to the plane is at least |n.(c - a)| - (BRICK - 1) h |n|_1 / 2.
  // The test gets 1e-3 h of slack over r against rounding; a degenerate face
  // keeps its whole box.
  B.ext = 0.5 * (BRICK - 1) * g.h * (fabs(B.un.x) + fabs(B.un.y) + fabs(B.un.z));
  return B;
}

// Marks brick (x, y, z) of a face's box if the face's plane is near enough: a plain
// store, no read to wait for (leaving out what the block has marked already, by a
// table in LDS, cost more than the stores: 64 meshes' build 408 -> 426 us).
__device__ inline void mark_brick(const MeshDesc& g, d3 un, d3 a, double ext, int x, int y, int z, uint8_t* flag) {
  const d3 c = mkd(g.origin[0] + (BRICK * x + BRICK / 2) * g.h, g.origin[1] + (BRICK * y + BRICK / 2) * g.h,
                   g.origin[2] + (BRICK * z + BRICK / 2) * g.h);
  if (fabs(dot(un, c - a)) - ext > g.whd + g.epsd + 1e-3 * g.h) return;
  flag[brick_pos(g, x, y, z)] = 1;
}

struct InputArgs {
  const float* V;
  const int32_t* T;
  const int32_t* f_off;
  const int32_t* v_off;
  const MeshDesc* md;
  int32_t* tg;           // [nf][3] global vertex indices
  int32_t* face_mesh;    // batches only
  int32_t* vert_mesh;    // batches only
  FaceRec* rec;
  uint8_t* flag;         // brick marks
  int32_t* bucket_count; // null: corners are not dealt into buckets
  int64_t* stats;
  int32_t* owned;        // per wavefront of 64 faces
  int32_t* vpolys;       // per tile of vertices: cleared
  int64_t vertex_tiles;
  int64_t nv, nf, face_tiles;
  int n_meshes, bucket_shift, buckets;
};

// The input passes in one launch, a block per tile of FACES faces (striding from INPUT_BLOCKS on):
// finite coordinates; of each face its mesh, index range and repeated-corner
// checks, global indices (a face with a bad index is replaced by three copies of its
// mesh's first vertex so that every later access stays in bounds; the build then
// reports the error), its record and band bricks, its owned
// half-edges (u -> w with u < w: they number the edges) counted per wavefront, and its
// corners counted per bucket of vertices, in LDS until the block is done. The mesh
// of a tile's first face is searched once; each thread steps up from there.
// FACES = BT: a thread marks its face's bricks. FACES = 64, for few faces: the
// first wavefront takes the faces, and the whole block their rows of bricks, one
// after another: a mesh of few faces fills more of the chip, and a face of hundreds
// of bricks among small ones holds up nobody (12 faces over 64^3 cells 45 -> 8 us; a wide
// band of 25,984 faces 97 -> 40; 70,000 faces 29 -> 19). A thread's own loop has less to
// read and no barrier, and is the faster for many faces (64 meshes, 1.75M: build 405 us and
// shared 508; see INPUT_SHARED).
template <int FACES>
__global__ __launch_bounds__(BT) void k_inputs(InputArgs P) {
  constexpr bool SHARE = FACES < BT;
  __shared__ int s_count[MAX_BUCKETS];
  __shared__ double s_plane[SHARE ? FACES : 1][8];  // un, a, ext (and a word of padding)
  __shared__ int s_box[SHARE ? FACES : 1][6];       // lo, n[0], n[1], mesh
  __shared__ int64_t s_row[SHARE ? FACES + 1 : 1];
  const int t = threadIdx.x;
  if (P.bucket_count)
    for (int b = t; b < P.buckets; b += BT) s_count[b] = 0;
  __syncthreads();
  const int64_t tiles = P.face_tiles * (BT / FACES);
  for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int64_t f = tile * FACES + t;
    if (!SHARE || t < FACES) {
      int owned = 0, m = 0;
      FaceBox B{};
      if (f < P.nf) {
        if (P.n_meshes > 1) {
          m = segment_from(P.f_off, find_segment(P.f_off, P.n_meshes + 1, tile * FACES), f);
          P.face_mesh[f] = m;
        }
        const int32_t vo = P.n_meshes > 1 ? P.v_off[m] : 0;
        const int32_t nvm = P.n_meshes > 1 ? P.v_off[m + 1] - vo : (int32_t)P.nv;
        int32_t a = P.T[3 * f], b = P.T[3 * f + 1], c = P.T[3 * f + 2];
        if (a < 0 || b < 0 || c < 0 || a >= nvm || b >= nvm || c >= nvm) {
          atomicOr(err_word(P.stats), ERR_INDEX);
          a = b = c = 0;
        } else if (a == b || b == c || a == c) {
          atomicOr(err_word(P.stats), ERR_REPEAT);
        }
        owned = (a < b ? 1 : 0) + (b < c ? 1 : 0) + (c < a ? 1 : 0);
        a += vo;
        b += vo;
        c += vo;
        P.tg[3 * f] = a;
        P.tg[3 * f + 1] = b;
        P.tg[3 * f + 2] = c;
        if (P.bucket_count) {
          atomicAdd(&s_count[a >> P.bucket_shift], 1);
          atomicAdd(&s_count[b >> P.bucket_shift], 1);
          atomicAdd(&s_count[c >> P.bucket_shift], 1);
        }
        B = face_geom_one(P.V, f, a, b, c, P.md[m], P.rec, P.stats);
        if (!SHARE && B.n[0] > 0)
          for (int z = B.lo[2]; z < B.lo[2] + B.n[2]; z++)
            for (int y = B.lo[1]; y < B.lo[1] + B.n[1]; y++)
              for (int x = B.lo[0]; x < B.lo[0] + B.n[0]; x++)
                mark_brick(P.md[m], B.un, B.a, B.ext, x, y, z, P.flag);
      }
      if (SHARE) {
        const double v[7] = {B.un.x, B.un.y, B.un.z, B.a.x, B.a.y, B.a.z, B.ext};
        for (int k = 0; k < 7; k++) s_plane[t][k] = v[k];
        const int w[6] = {B.lo[0], B.lo[1], B.lo[2], B.n[0], B.n[1], m};
        for (int k = 0; k < 6; k++) s_box[t][k] = w[k];
        int64_t incl = B.n[0] > 0 ? (int64_t)B.n[1] * B.n[2] : 0;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const int64_t x = __shfl_up(incl, o, 64);
          if (t >= o) incl += x;
        }
        s_row[t + 1] = incl;
        if (t == 0) s_row[0] = 0;
      }
      // owned half-edges per wavefront of 64 faces: no barrier in the loop
      const int sum = __popcll(__ballot(owned & 1)) + 2 * __popcll(__ballot(owned & 2));
      if ((t & 63) == 0) P.owned[tile * (FACES / 64) + (t >> 6)] = sum;
    }
    if (SHARE) {
      __syncthreads();
      const int64_t rows = s_row[FACES];
      auto mark_rows = [&](auto mesh) {  // this thread's rows of bricks
        int k = 0;
        for (int64_t p = t; p < rows; p += BT) {
          while (s_row[k + 1] <= p) k++;
          const int row = (int)(p - s_row[k]), z = row / s_box[k][4], y = row - z * s_box[k][4];
          const d3 un = mkd(s_plane[k][0], s_plane[k][1], s_plane[k][2]);
          const d3 a = mkd(s_plane[k][3], s_plane[k][4], s_plane[k][5]);
          const double ext = s_plane[k][6];
          const MeshDesc& g = mesh(k);
          const int x0 = s_box[k][0], x1 = x0 + s_box[k][3];
          for (int x = x0; x < x1; x++) mark_brick(g, un, a, ext, x, s_box[k][1] + y, s_box[k][2] + z, P.flag);
        }
      };
      if (P.n_meshes == 1) mark_rows([&](int) -> const MeshDesc& { return P.md[0]; });
      else mark_rows([&](int k) -> const MeshDesc& { return P.md[s_box[k][5]]; });
      __syncthreads();
    }
  }
  const int64_t step = (int64_t)gridDim.x * BT;
  for (int64_t i = blockIdx.x * (int64_t)BT + t; i < P.vertex_tiles; i += step) P.vpolys[i] = 0;
  for (int64_t i = blockIdx.x * (int64_t)BT + t; i < 3 * P.nv; i += step)
    if (!isfinite(P.V[i])) atomicOr(err_word(P.stats), ERR_NONFINITE);
  if (P.n_meshes > 1)
    for (int64_t i = blockIdx.x * (int64_t)BT + t; i < P.nv; i += step)
      P.vert_mesh[i] = find_segment(P.v_off, P.n_meshes + 1, i);
  if (P.bucket_count) {
    __syncthreads();
    for (int b = t; b < P.buckets; b += BT)
      if (s_count[b]) atomicAdd(&P.bucket_count[b], s_count[b]);
  }
}

struct BrickArgs {
  const uint8_t* flag;         // [nbt], zero up to a whole tile (16 flags per thread of a block)
  int32_t* index;
  int32_t* list;
  int32_t* bmesh;
  const int32_t* brick_base;
  int32_t* first_slot;
  int64_t* stats;
  int32_t* marked;             // per tile
  int64_t nbt, tiles;
  int n_meshes;
};

// the 16 flags (0 or 1 each) of this thread in brick tile `tile`
__device__ inline uint4 brick_flags(const BrickArgs& P, int64_t tile) {
  return reinterpret_cast<const uint4*>(P.flag)[tile * blockDim.x + threadIdx.x];
}

__device__ inline void count_bricks(const BrickArgs& P, int64_t tile, int* ws) {
  const uint4 x = brick_flags(P, tile);
  const int sum = block_sum(__popc(x.x) + __popc(x.y) + __popc(x.z) + __popc(x.w), ws);
  if (threadIdx.x == 0) P.marked[tile] = sum;
}

// slots of the flagged bricks (exclusive prefix of the flags), their list and mesh,
// and the first slot of every mesh (a mesh's bricks are a multiple of 64, so a
// thread's 16 lie in one mesh)
__device__ inline void number_bricks(const BrickArgs& P, int64_t tile, int* ws) {
  const uint4 x = brick_flags(P, tile);
  const uint32_t w[4] = {x.x, x.y, x.z, x.w};
  const int before = tiles_before(P.marked, tile, ws);
  int sum;
  int slot = before + block_prefix(__popc(x.x) + __popc(x.y) + __popc(x.z) + __popc(x.w), ws, &sum);
  const int64_t b0 = (tile * blockDim.x + threadIdx.x) * 16;
  if (b0 < P.nbt) {
    const int m = P.n_meshes > 1 ? find_segment(P.brick_base, P.n_meshes + 1, b0) : 0;
    if (b0 == P.brick_base[m]) P.first_slot[m] = slot;
#pragma unroll
    for (int q = 0; q < 4; q++) {
      int4 idx;
      int* id = &idx.x;
#pragma unroll
      for (int k = 0; k < 4; k++) {
        if ((w[q] >> (8 * k)) & 1u) {
          id[k] = slot;
          P.list[slot] = (int32_t)(b0 + 4 * q + k);
          P.bmesh[slot] = m;
          slot++;
        } else {
          id[k] = -1;
        }
      }
      *reinterpret_cast<int4*>(P.index + b0 + 4 * q) = idx;
    }
  }
  if (tile == P.tiles - 1 && threadIdx.x == 0) {
    P.first_slot[P.n_meshes] = before + sum;
    P.stats[ST_NBRICKS] = before + sum;
  }
}

// The corner table in two steps. k_deal takes tiles of TH * ITEMS corners and deals
// them into the buckets (ranges of 2^shift vertices): ranks inside the tile from LDS
// counters, a place in the bucket for the tile's share from one atomic per bucket,
// so that a share's corners lie together. k_bucket takes one bucket per block,
// counts its vertices in LDS, and places its corners; a vertex's corners come out in
// any order (k_vertex sorts the fans that it stages), except those of long fans, which the
// block's wavefronts sort. The blocks past the tiles and the buckets number
// the band bricks and the edges. Two reads and one write of 8 bytes per corner
// in all beside the 4-byte indices, where the radix sort read and wrote 16 bytes three
// times and counted digits in between (5.2M faces, 15.7M corners: k_deal 72 us and k_bucket 124, the edge ids and
// bricks included, against some 330 for the sort alone).
struct DealArgs {
  const int32_t* tg;
  int64_t nh, tiles, nv;
  const int32_t* bucket_count;
  int32_t* bucket_next;   // zeroed by k_begin
  uint2* pairs;           // (vertex, corner) by bucket
  int32_t* off;
  int32_t* corners;
  int shift, buckets;
};

// The number of owned half-edges before each half-edge, the id of the edge it owns:
// those of the wavefronts of 64 faces before (counted by k_inputs, scanned by a block
// of k_deal), those of the faces before in the wavefront, those before in the face.
struct EdgeBase {
  const int32_t* tg;
  int32_t* owned;    // [waves] per 64 faces; their exclusive prefix once scanned
  int32_t* eid;      // [nf][3]
  int64_t* stats;
  int64_t nf, waves, tiles;  // tiles of the block's size
};

__device__ inline void edge_bases(const EdgeBase& P, int64_t tile) {
  const int64_t f = tile * blockDim.x + threadIdx.x;
  int o0 = 0, o1 = 0, o2 = 0;
  if (f < P.nf) {
    const int32_t a = P.tg[3 * f], b = P.tg[3 * f + 1], c = P.tg[3 * f + 2];
    o0 = a < b ? 1 : 0;
    o1 = b < c ? 1 : 0;
    o2 = c < a ? 1 : 0;
  }
  const int owned = o0 + o1 + o2, before = wave_prefix_sum(owned) - owned;
  if (f < P.nf) {
    const int at = P.owned[f >> 6] + before;
    P.eid[3 * f] = at;
    P.eid[3 * f + 1] = at + o0;
    P.eid[3 * f + 2] = at + o0 + o1;
  }
}

__device__ inline void scan_owned(const EdgeBase& P, int* ws) {
  const int found = scan_tiles(P.owned, P.waves, ws);
  if (threadIdx.x == 0) P.stats[ST_NE] = found;
}

template <int TH, int ITEMS>
__global__ __launch_bounds__(TH) void k_deal(DealArgs P, BrickArgs B, EdgeBase E) {
  __shared__ int s_count[MAX_BUCKETS], s_base[MAX_BUCKETS];
  __shared__ int ws[TH / 64];
  const int t = threadIdx.x;
  if (blockIdx.x == 0) {
    scan_owned(E, ws);
    return;
  }
  const int64_t tile = (int64_t)blockIdx.x - 1;
  if (tile >= P.tiles) {
    count_bricks(B, tile - P.tiles, ws);
    return;
  }
  for (int b = t; b < P.buckets; b += TH) s_count[b] = 0;
  __syncthreads();
  int32_t v[ITEMS], r[ITEMS];
  const int64_t base = tile * (int64_t)(TH * ITEMS) + t;
#pragma unroll
  for (int k = 0; k < ITEMS; k++) v[k] = base + (int64_t)k * TH < P.nh ? P.tg[base + (int64_t)k * TH] : -1;
#pragma unroll
  for (int k = 0; k < ITEMS; k++) r[k] = v[k] >= 0 ? atomicAdd(&s_count[v[k] >> P.shift], 1) : 0;
  __syncthreads();
  // where each bucket starts, and this tile's share of it
  int run = 0;
  for (int b0 = 0; b0 < P.buckets; b0 += TH) {
    const int b = b0 + t, c = b < P.buckets ? P.bucket_count[b] : 0;
    int sum;
    const int start = run + block_prefix(c, ws, &sum);
    run += sum;
    if (b < P.buckets) {
      const int mine = s_count[b];
      s_base[b] = start + (mine ? atomicAdd(&P.bucket_next[b], mine) : 0);
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < ITEMS; k++)
    if (v[k] >= 0)
      P.pairs[s_base[v[k] >> P.shift] + r[k]] = make_uint2((uint32_t)v[k], (uint32_t)(base + (int64_t)k * TH));
}

// ascending order of n corners, by one wavefront: each one's place is the number of
// smaller ones. tmp holds n words. (A heap sort by the one thread that matches the fan took
// 1.3 of the build's 100 ms at a pole of 512 corners behind 240,000 faces, 20 of its 150 us at one of 17.)
__device__ inline void sort_fan(int32_t* corners, uint32_t* tmp, int n) {
  const int lane = threadIdx.x & 63;
  for (int k = lane; k < n; k += 64) tmp[k] = (uint32_t)corners[k];
  __threadfence_block();
  __builtin_amdgcn_wave_barrier();
  for (int k = lane; k < n; k += 64) {
    const uint32_t c = tmp[k];
    int place = 0;
#pragma unroll 8
    for (int j = 0; j < n; j++) place += tmp[j] < c ? 1 : 0;
    corners[place] = (int32_t)c;
  }
}

template <int TH>
__global__ __launch_bounds__(TH) void k_bucket(DealArgs P, BrickArgs B, EdgeBase E) {
  extern __shared__ int s_count[];  // 2^shift
  __shared__ int ws[TH / 64];
  __shared__ int s_long;            // some fan is not sorted by the vertex pass
  if ((int)blockIdx.x >= P.buckets) {
    const int64_t x = (int64_t)blockIdx.x - P.buckets;
    if (x < E.tiles) edge_bases(E, x);
    else number_bricks(B, x - E.tiles, ws);
    return;
  }
  const int t = threadIdx.x, b = blockIdx.x, size = 1 << P.shift;
  const int64_t v0 = (int64_t)b << P.shift;
  int before = 0;
  for (int k = t; k < b; k += TH) before += P.bucket_count[k];
  const int start = block_sum(before, ws), n = P.bucket_count[b];
  if (b == P.buckets - 1 && t == 0) P.off[P.nv] = (int32_t)P.nh;
  if (n == 0) {  // vertices of no triangle
    for (int k = t; k < size; k += TH)
      if (v0 + k < P.nv) P.off[v0 + k] = start;
    return;
  }
  for (int k = t; k < size; k += TH) s_count[k] = 0;
  if (t == 0) s_long = 0;
  __syncthreads();
  // AHEAD pairs of a thread are loaded together, then used: one at a time, each load
  // waits out the memory latency
  constexpr int AHEAD = 8;
  const uint2* pairs = P.pairs + start;
  for (int k0 = 0; k0 < n; k0 += AHEAD * TH) {
    uint32_t v[AHEAD];
#pragma unroll
    for (int a = 0; a < AHEAD; a++) {
      const int k = k0 + a * TH + t;
      v[a] = pairs[k < n ? k : 0].x - (uint32_t)v0;
    }
#pragma unroll
    for (int a = 0; a < AHEAD; a++)
      if (k0 + a * TH + t < n) atomicAdd(&s_count[v[a]], 1);
  }
  __syncthreads();
  const int per = (size + TH - 1) / TH;  // counters of a thread: consecutive
  int sum = 0;
  for (int k = 0; k < per; k++) {
    const int i = t * per + k;
    if (i < size) sum += s_count[i];
  }
  int all;
  int at = block_prefix(sum, ws, &all);
  for (int k = 0; k < per; k++) {
    const int i = t * per + k;
    if (i < size) {
      const int c = s_count[i];
      if (c > VK_MAXD) s_long = 1;
      s_count[i] = at;
      if (v0 + i < P.nv) P.off[v0 + i] = start + at;
      at += c;
    }
  }
  __syncthreads();
  for (int k0 = 0; k0 < n; k0 += AHEAD * TH) {
    uint2 x[AHEAD];
#pragma unroll
    for (int a = 0; a < AHEAD; a++) {
      const int k = k0 + a * TH + t;
      x[a] = pairs[k < n ? k : 0];
    }
#pragma unroll
    for (int a = 0; a < AHEAD; a++)
      if (k0 + a * TH + t < n) P.corners[start + atomicAdd(&s_count[x[a].x - (uint32_t)v0], 1)] = (int32_t)x[a].y;
  }
  if (!s_long) return;  // the same in all threads: last written before the barrier above
  __syncthreads();
  // a counter now stands at its vertex's end, the place where the next one's corners
  // start; the block's pairs are read and serve as scratch
  for (int i0 = 0; i0 < size; i0 += TH) {
    const int i = i0 + t, end = i < size ? s_count[i] : 0, first = i > 0 && i < size ? s_count[i - 1] : 0;
    for (unsigned long long left = __ballot(end - first > VK_MAXD); left != 0; left &= left - 1) {
      const int l = __ffsll((long long)left) - 1;
      const int from = __builtin_amdgcn_readlane(first, l), to = __builtin_amdgcn_readlane(end, l);
      sort_fan(P.corners + start + from, (uint32_t*)(P.pairs + start + from), to - from);
    }
  }
}

// the same numbering of bricks and edges in two launches of its own, where the corner table comes from the radix sort
__global__ __launch_bounds__(BT) void k_bricks(BrickArgs B, EdgeBase E, int pass) {
  __shared__ int ws[BT / 64];
  const int64_t x = blockIdx.x;
  if (pass == 0) {
    if (x == 0) scan_owned(E, ws);
    else count_bricks(B, x - 1, ws);
  } else {
    if (x < E.tiles) edge_bases(E, x);
    else number_bricks(B, x - E.tiles, ws);
  }
}

// class statistics (and absorbed features): each thread counts 16 edge-class bytes and 4 vertex words per
// 16-byte load (both arrays start 256-byte aligned), one LDS histogram per
// block, one global add per bin and block
__device__ inline void count_edge_class(int c, int (&loc)[11]) {
  loc[9] += (c & EDGE_ABSORBED) != 0;
  c &= 3;
  loc[0] += c == EDGE_CONVEX;
  loc[1] += c == EDGE_CONCAVE;
  loc[2] += c == EDGE_FLAT;
  loc[3] += c == EDGE_UNKNOWN;
}
__device__ inline void count_vertex_class(uint32_t b, int (&loc)[11]) {
  loc[4] += (b & V_CONVEX) != 0;
  loc[5] += (b & V_CONCAVE) != 0;
  loc[6] += (b & V_FLAT) != 0;
  loc[7] += (b & V_SADDLE) != 0;
  loc[8] += (b & V_RUFF) != 0;
  loc[10] += (b & V_ABSORBED) != 0;
}

// the classes of all edges and vertices into the block's h[11]: thread t0 of `stride`
__device__ inline void count_classes(const uint8_t* __restrict__ ecls, int64_t ne, const uint32_t* __restrict__ vbits,
                                     int64_t nv, int64_t t0, int64_t stride, int* h) {
  int loc[11] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  const uint4* e16 = reinterpret_cast<const uint4*>(ecls);
#pragma unroll 2
  for (int64_t i = t0; i < ne / 16; i += stride) {
    const uint4 x = e16[i];
    const uint32_t wv[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int q = 0; q < 4; q++)
#pragma unroll
      for (int k = 0; k < 4; k++) count_edge_class((int)((wv[q] >> (8 * k)) & 0xffu), loc);
  }
  for (int64_t i = ne / 16 * 16 + t0; i < ne; i += stride) count_edge_class(ecls[i], loc);
  const uint4* v4 = reinterpret_cast<const uint4*>(vbits);
#pragma unroll 2
  for (int64_t i = t0; i < nv / 4; i += stride) {
    const uint4 x = v4[i];
    count_vertex_class(x.x, loc);
    count_vertex_class(x.y, loc);
    count_vertex_class(x.z, loc);
    count_vertex_class(x.w, loc);
  }
  for (int64_t i = nv / 4 * 4 + t0; i < nv; i += stride) count_vertex_class(vbits[i], loc);
#pragma unroll
  for (int k = 0; k < 11; k++) {
    int x = loc[k];
    for (int o = 32; o > 0; o >>= 1) x += __shfl_down(x, o, 64);
    if ((threadIdx.x & 63) == 0 && x) atomicAdd(&h[k], x);
  }
  __syncthreads();
}
__constant__ const int CLASS_STAT[11] = {ST_E_CONVEX, ST_E_CONCAVE, ST_E_FLAT, ST_E_UNKNOWN, ST_V_CONVEX, ST_V_CONCAVE,
                                         ST_V_FLAT,   ST_V_SADDLE,  ST_V_RUFF, ST_E_ABSORBED, ST_V_ABSORBED};

__global__ __launch_bounds__(256) void k_class_stats(const uint8_t* __restrict__ ecls, int64_t ne,
                                                     const uint32_t* __restrict__ vbits, int64_t nv, int64_t* stats) {
  __shared__ int h[16];
  if (threadIdx.x < 16) h[threadIdx.x] = 0;
  __syncthreads();
  count_classes(ecls, ne, vbits, nv, blockIdx.x * (int64_t)blockDim.x + threadIdx.x, (int64_t)gridDim.x * blockDim.x, h);
  if (threadIdx.x < 11 && h[threadIdx.x])
    atomicAdd((unsigned long long*)&stats[CLASS_STAT[threadIdx.x]], (unsigned long long)h[threadIdx.x]);
}

// The same by one block, which also writes all the statistics to the host's mirror:
// one launch where few words are read (at most STATS_ONE_BLOCK of 16 bytes), in place of
// the count and a copy (synchronised rebuild of 642 vertices 76 -> 71 us).
constexpr int64_t STATS_ONE_BLOCK = 8192;
__global__ __launch_bounds__(1024) void k_stats_out(const uint8_t* __restrict__ ecls, int64_t ne,
                                                    const uint32_t* __restrict__ vbits, int64_t nv, int64_t* stats,
                                                    int64_t* host) {
  __shared__ int h[16];
  if (threadIdx.x < 16) h[threadIdx.x] = 0;
  __syncthreads();
  count_classes(ecls, ne, vbits, nv, threadIdx.x, 1024, h);
  if (threadIdx.x < 11) stats[CLASS_STAT[threadIdx.x]] = h[threadIdx.x];
  __syncthreads();
  if (threadIdx.x < ST_COUNT) host[threadIdx.x] = stats[threadIdx.x];
}

struct ListArgs {
  const int32_t* T;
  const int32_t* face_edges;
  const uint32_t* vbits;
  const uint8_t* eslack;
  const uint8_t* cls;
  const int32_t* eid;         // [nf][3] owned half-edges before each half-edge
  const int32_t* epolys;      // per block of k_edges: three per face tile
  uint8_t* fslack;
  uint8_t* fabsorbed;
  int32_t* epoly;
  int64_t* stats;
  int64_t nf, ne, lists, list_tiles;  // list blocks, face tiles of each
};

// The first blocks write the edge list, each that of the edges of list_tiles face
// tiles (which follow one another); the others take the faces: the largest slack code
// of a face's edges and vertices (gathers of the coalesced per-feature codes instead
// of scattered byte writes per face side), and which of them are absorbed (the face
// scan signs their cells itself).
__global__ __launch_bounds__(BT) void k_lists(ListArgs P) {
  __shared__ int ws[BT / 64];
  if (blockIdx.x < P.lists) {
    const int64_t f0 = blockIdx.x * P.list_tiles * BT, f1 = f0 + P.list_tiles * BT;
    const int64_t e0 = P.eid[3 * f0] < P.ne ? P.eid[3 * f0] : P.ne;  // none past ne
    int64_t e1 = f1 < P.nf ? P.eid[3 * f1] : P.ne;
    if (e1 > P.ne) e1 = P.ne;
    int at = tiles_before(P.epolys, 3 * blockIdx.x * P.list_tiles, ws);
    for (int64_t b = e0; b < e1; b += 4 * BT) {
      const int64_t e = b + 4 * (int64_t)threadIdx.x;
      int m[4], c = 0, sum;
#pragma unroll
      for (int k = 0; k < 4; k++) {
        m[k] = e + k < e1 ? (P.cls[e + k] >> 2) & 3 : 0;
        c += __popc(m[k]);
      }
      int mine = at + block_prefix(c, ws, &sum);
#pragma unroll
      for (int k = 0; k < 4; k++) mine = put_entries(P.epoly, mine, e + k, m[k]);
      at += sum;
    }
    if (blockIdx.x == P.lists - 1 && threadIdx.x == 0) P.stats[ST_NEPOLY] = at;
    return;
  }
  const int64_t f = (blockIdx.x - P.lists) * BT + threadIdx.x;
  if (f >= P.nf) return;
  uint32_t q = 0, bits = 0;
#pragma unroll
  for (int j = 0; j < 3; j++) {
    const uint32_t qv = (P.vbits[P.T[3 * f + j]] >> V_SLACK_SHIFT) & 0xffu;
    q = max(q, qv);
    if (qv) bits |= 8u << j;
    const int32_t e = P.face_edges[3 * f + j];
    const uint32_t qe = e >= 0 && e < P.ne ? (uint32_t)P.eslack[e] : 0u;
    q = max(q, qe);
    if (qe) bits |= 1u << j;
  }
  P.fslack[f] = (uint8_t)q;
  P.fabsorbed[f] = (uint8_t)bits;
}

int status_from_errors(uint64_t err, int64_t ne_found, int64_t ne_expected) {
  if (err & (ERR_INDEX | ERR_REPEAT | ERR_NONFINITE)) return CSC_INVALID_ARG;
  if (err & ERR_OVERFLOW) return CSC_WORKSPACE_TOO_SMALL;
  if (err & ERR_ORIENT) return CSC_INCONSISTENT_ORIENTATION;
  if (err & ERR_NONMANIFOLD) return CSC_NONMANIFOLD;
  if (ne_found != ne_expected) return CSC_NONMANIFOLD;
  if (err & ERR_DEGENERATE) return CSC_DEGENERATE_FACE;
  return CSC_OK;
}

// Key of the spatial processing order of the faces: the Morton code of each
// face's centroid in its own grid, at `axis_bits` bits per axis, with its mesh
// above it (the paper orders its triangle soup by Morton code as well, Section
// 7.1; here the order only schedules the face pass and changes no result).
__global__ void k_face_order_keys(const FaceRec* __restrict__ R, const int32_t* __restrict__ face_mesh,
                                  const MeshDesc* __restrict__ md, int n_meshes, int64_t nf, int axis_bits,
                                  uint32_t* key) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const uint32_t top = (1u << axis_bits) - 1u;
  for (int64_t f = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; f < nf; f += stride) {
    const int m = n_meshes > 1 ? face_mesh[f] : 0;
    const MeshDesc& G = md[m];
    const float4 a = R[f].c[0], b = R[f].c[1], c = R[f].c[2];
    const double x[3] = {((double)a.x + b.x + c.x) / 3.0, ((double)a.y + b.y + c.y) / 3.0,
                         ((double)a.z + b.z + c.z) / 3.0};
    uint32_t code = 0;
    for (int k = 0; k < 3; k++) {
      const double u = (x[k] - G.origin[k]) * G.inv_h / G.n[k] * (double)(1u << axis_bits);
      const uint32_t qk = u <= 0.0 ? 0u : (u >= (double)top ? top : (uint32_t)u);  // NaN-free: finite inputs
      for (int bit = 0; bit < axis_bits; bit++) code |= ((qk >> bit) & 1u) << (3 * bit + k);
    }
    key[f] = ((uint32_t)m << (3 * axis_bits)) | code;
  }
}

}  // namespace csc

using namespace csc;

extern "C" int csc_features_order_faces(csc_features* F, int32_t enable, void* stream) {
  if (!F || !F->built || (enable != 0 && enable != 1)) return CSC_INVALID_ARG;
  hipStream_t s = (hipStream_t)stream;
  queued_on(F, stream);
  if (!enable || F->nf == 0) {
    if (F->face_order) {
      (void)hipStreamSynchronize(s);
      (void)hipFree(F->face_order);
      F->face_order = nullptr;
      F->face_order_n = 0;
    }
    return CSC_OK;
  }
  const int64_t nf = F->nf;
  int mesh_bits = 0;
  while ((1 << mesh_bits) < F->n_meshes) mesh_bits++;
  int axis_bits = (32 - mesh_bits) / 3;
  if (axis_bits > 10) axis_bits = 10;
  const int bits = mesh_bits + 3 * axis_bits;
  const size_t sort_bytes = sort_pairs_tmp_bytes(nf, bits);
  if (sort_bytes == 0) return CSC_INVALID_ARG;
  const size_t key_bytes = ((size_t)nf * sizeof(uint32_t) + 255) & ~(size_t)255;
  // the sort's scratch is gone when a captured one would run
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  hipError_t ce = hipStreamIsCapturing(s, &cap);
  if (ce == hipSuccess && cap != hipStreamCaptureStatusNone) ce = hipErrorStreamCaptureUnsupported;
  if (ce != hipSuccess) return fail_hip(ce);
  if (!F->face_order) {
    hipError_t he = device_alloc(sizeof(int32_t) * (size_t)nf, (void**)&F->face_order, F->device);
    if (he != hipSuccess) return he == hipErrorOutOfMemory ? CSC_OUT_OF_MEMORY : fail_hip(he);
  }
  F->face_order_n = 0;  // not valid until the sort below has run
  char* tmp = nullptr;
  hipError_t he = device_alloc(2 * key_bytes + sort_bytes, (void**)&tmp, F->device);
  if (he != hipSuccess) return he == hipErrorOutOfMemory ? CSC_OUT_OF_MEMORY : fail_hip(he);
  uint32_t* key = (uint32_t*)tmp;
  uint32_t* key_sorted = (uint32_t*)(tmp + key_bytes);
  k_face_order_keys<<<grid_1d(nf, 256), 256, 0, s>>>(F->face_rec, F->face_mesh, F->d_mesh, F->n_meshes, nf,
                                                        axis_bits, key);
  he = hipGetLastError();
  if (he == hipSuccess)
    he = sort_pairs(tmp + 2 * key_bytes, sort_bytes, key, key_sorted, nullptr, F->face_order, nf, bits, s);
  if (he == hipSuccess) he = hipStreamSynchronize(s);
  (void)hipFree(tmp);
  if (he != hipSuccess) return fail_hip(he);
  F->face_order_n = nf;
  return CSC_OK;
}

namespace {

size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

enum {
  L_MESH, L_FOFF, L_VOFF, L_BBASE, L_TRIS, L_FMESH, L_VMESH, L_VTXOFF, L_VTXC, L_FEDGES, L_EDGES, L_FREC, L_ECLS,
  L_VINFO, L_VBITS, L_EPOLY, L_VPOLY, L_BINDEX, L_BLIST, L_BMESH, L_FIRST, L_TWIN, L_PAIRS, L_EID, L_SUMS, L_ZERO, L_STATS,
  L_SORT, L_FSLACK, L_ESLACK, L_FABS, L_N
};

// How the corner table is made: buckets of 2^shift vertices, or (no buckets) the
// radix sort, for more vertices than MAX_BUCKETS of the largest buckets hold. Large
// inputs take long tiles (few shares per bucket), small ones short tiles (more blocks).
// Build of tori with short and with long tiles: 4.2M corners 243 and 247 us, 6.5M 392 and 368,
// 8.4M 492 and 479, 10.8M 617 and 598, 16.2M 962 and 881; of 64 meshes with 5.3M corners
// 406 and 415.
constexpr int DEAL_TH = 256, DEAL_ITEMS = 8, DEAL_BIG_TH = 1024, DEAL_BIG_ITEMS = 16;
constexpr int64_t DEAL_BIG = 1 << 23;  // corners from which the long tiles are used
// Blocks of the input pass: a tile each up to 8.4M faces. A block adds its corner
// counts to every bucket once at its end, which more blocks do more often, but the loads of
// a block's next tile would wait for its last one's stores (a batch of 64 meshes:
// build 406 us with 2048 blocks, 397 with a tile each; 5.2M faces 1210, 1188).
constexpr int64_t INPUT_BLOCKS = 32768;
// Vertices up to which a vertex takes a lane per corner (k_vertex_fan). Build of tori (six
// corners everywhere) with a thread per vertex and with lanes: 30,000 vertices 51 and 49
// us, 64,800 72 and 76, 80,000 67 and 71, 120,000 73 and 85, 180,000 93 and 110; of random points'
// triangles (4 to 13 corners, where a wavefront of threads waits for its longest fan) 30,000
// vertices 147 and 68, 65,000 193 and 116, 180,000 231 and 177. The line lies where the
// regular ones lose 5%.
constexpr int64_t VERTEX_FANS = 1 << 16;
// Faces up to which a block shares its faces' bricks (k_inputs). Build of tori with a
// thread's own loop and shared, at bands of 3, 8 and 20 cells: 34,848 faces 69 and 58, 141 and 83 us
// at the two wider ones; 100,000 67 and 72, 82 and 79, 167 and 136; 129,600 71 and 76, 85 and 84, 170 and 153; 192,000
// 69 and 75, 85 and 86, 177 and 183; 360,000 94 and 109, 115 and 124, 279 and 297. The line lies
// where the band of 8 breaks even.
constexpr int64_t INPUT_SHARED = 1 << 17;
struct Plan {
  int shift = 0, buckets = 0;
  bool big = false;
  int64_t deal_tiles = 0, face_tiles = 0, vertex_tiles = 0, brick_tiles = 0;
};

Plan plan(int64_t nv, int64_t nf, int64_t nbt) {
  Plan p;
  // 256 to 512 buckets of at least 64 vertices; large inputs 1024 to 2048, each block then
  // holds fewer corners and more run at once (5.2M faces: k_bucket 244 us with 320 buckets,
  // 124 with 1280)
  p.shift = 6;
  const int64_t target = 3 * nf >= DEAL_BIG ? MAX_BUCKETS : 512;
  while (p.shift < MAX_BUCKET_SHIFT && ((nv - 1) >> p.shift) >= target) p.shift++;
  const int64_t b = ((nv - 1) >> p.shift) + 1;
  p.buckets = b <= MAX_BUCKETS ? (int)b : 0;
  p.big = p.buckets > 0 && 3 * nf >= DEAL_BIG;
  const int64_t tile = p.big ? DEAL_BIG_TH * DEAL_BIG_ITEMS : DEAL_TH * DEAL_ITEMS;
  p.deal_tiles = (3 * nf + tile - 1) / tile;
  p.face_tiles = (nf + BT - 1) / BT;
  p.vertex_tiles = (nv + VK_THREADS - 1) / VK_THREADS;
  const int64_t bt = 16 * (p.big ? DEAL_BIG_TH : BT);
  p.brick_tiles = (nbt + bt - 1) / bt;
  return p;
}

// the zeroed region: bucket counts and places, then the brick flags on a 16-byte
// boundary, up to a whole tile of the larger blocks
struct ZeroLayout {
  int64_t count, next;  // in ints
  size_t flags, bytes;
};

ZeroLayout zero_layout(const Plan& p, int64_t nbt) {
  ZeroLayout z;
  z.count = 0;
  z.next = p.buckets;
  z.flags = align_up(sizeof(int32_t) * 2 * (size_t)p.buckets);
  const size_t tile = 16 * (size_t)DEAL_BIG_TH;
  z.bytes = z.flags + ((size_t)nbt + tile - 1) / tile * tile;
  return z;
}

// ints of an array of n tile sums: whole groups of SCAN_PER
int64_t sums_of(int64_t n) { return (n + SCAN_PER - 1) / SCAN_PER * SCAN_PER; }

struct Layout {
  size_t off[L_N];
  size_t total;
};

Layout layout(int n_meshes, int64_t nv, int64_t nf, int64_t nbt, const Plan& p, size_t sort_bytes) {
  const int64_t ne = 3 * nf / 2;
  size_t sz[L_N];
  sz[L_MESH] = sizeof(MeshDesc) * (size_t)n_meshes;
  sz[L_FOFF] = sz[L_VOFF] = sz[L_BBASE] = sizeof(int32_t) * (size_t)(n_meshes + 1);
  sz[L_TRIS] = sizeof(int32_t) * (size_t)(3 * nf);
  sz[L_FMESH] = sizeof(int32_t) * (size_t)(n_meshes > 1 ? nf : 1);
  sz[L_VMESH] = sizeof(int32_t) * (size_t)(n_meshes > 1 ? nv : 1);
  sz[L_VTXOFF] = sizeof(int32_t) * (size_t)(nv + 1);
  sz[L_VTXC] = sizeof(int32_t) * (size_t)(3 * nf);
  sz[L_FEDGES] = sizeof(int32_t) * (size_t)(3 * nf);
  sz[L_EDGES] = sizeof(int4) * (size_t)(ne + 1);
  sz[L_FREC] = sizeof(FaceRec) * (size_t)nf;
  sz[L_ECLS] = (size_t)(ne + 16);
  sz[L_VINFO] = sizeof(float4) * (size_t)nv;
  sz[L_VBITS] = sizeof(uint32_t) * (size_t)nv;
  sz[L_EPOLY] = sizeof(int32_t) * (size_t)(2 * ne + 1);
  sz[L_VPOLY] = sizeof(int32_t) * (size_t)(2 * nv + 1);
  sz[L_BINDEX] = sz[L_BLIST] = sz[L_BMESH] = sizeof(int32_t) * (size_t)nbt;
  sz[L_FIRST] = sizeof(int32_t) * (size_t)(n_meshes + 1);
  sz[L_TWIN] = sizeof(int32_t) * (size_t)(3 * nf);
  sz[L_PAIRS] = p.buckets > 0 ? sizeof(uint2) * (size_t)(3 * nf) : sizeof(uint32_t) * (size_t)(3 * nf);  // or sorted keys
  sz[L_EID] = sizeof(int32_t) * (size_t)(3 * nf);
  // tile sums: owned half-edges, edge polyhedra, vertex polyhedra, bricks
  sz[L_SUMS] = sizeof(int32_t) * (size_t)(sums_of(p.face_tiles * (BT / 64)) + sums_of(3 * p.face_tiles) +
                                          sums_of(p.vertex_tiles) + sums_of(p.brick_tiles));
  sz[L_ZERO] = zero_layout(p, nbt).bytes;
  sz[L_STATS] = sizeof(int64_t) * ST_COUNT;
  sz[L_SORT] = sort_bytes;
  sz[L_FSLACK] = (size_t)(nf + 8);
  sz[L_ESLACK] = (size_t)(ne + 8);
  sz[L_FABS] = (size_t)(nf + 8);
  Layout L;
  size_t o = 0;
  for (int i = 0; i < L_N; i++) {
    L.off[i] = o;
    o += align_up(sz[i]);
  }
  L.total = o;
  return L;
}

bool finite_pos(double x) { return x > 0 && x < 1e300; }

int check_grid(const csc_grid& g) {
  for (int a = 0; a < 3; a++)
    if (g.n[a] <= 0 || !isfinite(g.origin[a])) return CSC_INVALID_ARG;
  if (!finite_pos(g.h) || !(g.band_cells > 0) || !isfinite(g.band_cells)) return CSC_INVALID_ARG;
  if ((int64_t)g.n[0] * g.n[1] * g.n[2] > INT32_MAX) return CSC_GRID_TOO_LARGE;
  for (int a = 0; a < 3; a++)  // cell offsets inside a polyhedron box are packed in 16 bits
    if (g.n[a] > 65535) return CSC_GRID_TOO_LARGE;
  return CSC_OK;
}

bool same_config(const csc_features* F, const std::vector<MeshDesc>& m, const csc_options& o) {
  if ((int)F->mesh.size() != (int)m.size()) return false;
  if (memcmp(&F->opt, &o, sizeof(o)) != 0) return false;
  return memcmp(F->mesh.data(), m.data(), sizeof(MeshDesc) * m.size()) == 0;
}

}  // namespace

// Shared implementation of the single-mesh and batched builds.
int build_impl(const float* verts_d, const int32_t* tris_d, const int64_t* nv, const int64_t* nf,
               const csc_grid* grids, int32_t n_meshes, const csc_options* opt, int32_t flags, void* stream,
               csc_features** out) {
  if (!verts_d || !tris_d || !nv || !nf || !grids || !out || n_meshes <= 0) return CSC_INVALID_ARG;
  csc_options o = {1e-3f, 0, 0, 0, {0, 0, 0}, 0, 0.f, 0, 0, 0};
  if (opt) o = *opt;
  if (o.scan_grid < 0 || o.scan_grid > 3 || o.geom_blocks < 0 || (o.keep_store_empty & ~1)) return CSC_INVALID_ARG;
  if (o.scan_grid == 0) o.scan_grid = 2;  // default: persistent grid striding over the groups
  if (!(o.absorb_cells <= 0.24f) || o.absorb_cells != o.absorb_cells) return CSC_INVALID_ARG;
  // 0: the default; negative: every non-flat feature keeps its own polyhedron
  if (o.absorb_cells == 0.f) o.absorb_cells = 0.05f;
  if (!(o.eps_rel >= 0) || !(o.eps_rel < 0.5f) || o.ruff_mode < 0 || o.ruff_mode > 1 || o.scan_mode < 0 || o.scan_mode > 1 || o.saddle_mode < 0 ||
      o.saddle_mode > 2)
    return CSC_INVALID_ARG;
  for (int k = 0; k < 3; k++) {
    if (o.small_rows[k] < 0) return CSC_INVALID_ARG;
    if (o.small_rows[k] > (1 << 24)) o.small_rows[k] = 1 << 24;  // row totals of a wavefront stay in 32 bits
  }
  std::vector<MeshDesc> mesh((size_t)n_meshes);
  int64_t tv = 0, tf = 0, te = 0, tb = 0;
  for (int m = 0; m < n_meshes; m++) {
    if (nv[m] <= 0 || nf[m] <= 0) return CSC_INVALID_ARG;
    int gc = check_grid(grids[m]);
    if (gc != CSC_OK) return gc;
    if (nf[m] % 2 != 0) return CSC_NONMANIFOLD;  // a closed triangle surface has 3F/2 edges
    MeshDesc& d = mesh[m];
    memset(&d, 0, sizeof(d));
    const csc_grid& g = grids[m];
    for (int a = 0; a < 3; a++) {
      d.origin[a] = g.origin[a];
      d.n[a] = g.n[a];
      d.nb[a] = (g.n[a] + BRICK - 1) / BRICK;
      d.nt[a] = (d.nb[a] + TILE - 1) / TILE;
    }
    d.h = g.h;
    d.inv_h = 1.0 / g.h;
    d.whd = (double)g.band_cells * g.h;
    d.epsd = (double)o.eps_rel * g.h;
    d.hf = (float)g.h;
    d.whf = (float)d.whd;
    d.eps = (float)d.epsd;
    d.band = g.band_cells;
    d.brick_base = (int32_t)tb;
    d.v_off = (int32_t)tv;
    d.f_off = (int32_t)tf;
    d.e_off = (int32_t)te;
    d.nv = (int32_t)nv[m];
    d.nf = (int32_t)nf[m];
    d.ne = (int32_t)(3 * nf[m] / 2);
    tb += (int64_t)d.nt[0] * d.nt[1] * d.nt[2] * (TILE * TILE * TILE);
    tv += nv[m];
    tf += nf[m];
    te += 3 * nf[m] / 2;
    // feature ids (faces + edges + vertices) must fit in 30 bits of the packed key
    if (tf + te + tv >= (1 << 30)) return CSC_INVALID_ARG;
    if (tb > (1 << 26)) return CSC_GRID_TOO_LARGE;
  }
  int dc = check_device();
  if (dc != CSC_OK) return dc;

  const bool no_sync = (flags & CSC_BUILD_NO_SYNC) != 0;
  hipStream_t s = (hipStream_t)stream;
  csc_features* F = *out;
  const bool fresh = F == nullptr;
  if (fresh) {
    F = new (std::nothrow) csc_features();
    if (!F) return CSC_OUT_OF_MEMORY;
  }
  auto fail = [&](int code) {
    if (fresh) csc_features_free(F);
    else F->built = F->synced = false;
    return code;
  };
#define CK(x)                                        \
  do {                                               \
    hipError_t e_ = (x);                             \
    if (e_ != hipSuccess) return fail(fail_hip(e_)); \
  } while (0)

  const Plan pl = plan(tv, tf, tb);
  int sort_bits = 1;
  while (sort_bits < 31 && ((int64_t)1 << sort_bits) < tv) sort_bits++;
  const size_t sort_bytes = pl.buckets > 0 ? 0 : sort_pairs_tmp_bytes(3 * tf, sort_bits);
  if (pl.buckets == 0 && sort_bytes == 0) return fail(fail_hip(hipErrorInvalidValue));
  Layout L = layout(n_meshes, tv, tf, tb, pl, sort_bytes);
  const bool config_changed = fresh || !same_config(F, mesh, o) || F->arena_bytes < L.total || F->nv != tv ||
                              F->nf != tf;
  hipError_t he;
  if (config_changed) {
    // Descriptors and offset tables change only with the configuration, never inside a
    // captured replay of the same batch: refused there, before anything of the handle is
    // touched. From here on the handle holds the tables of no configuration, until the
    // launches below are known to be queued.
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    CK(hipStreamIsCapturing(s, &cap));
    if (cap != hipStreamCaptureStatusNone) CK(hipErrorStreamCaptureUnsupported);
    F->mesh.clear();
  }
  if (F->face_order && F->face_order_n != tf) {  // an order of another face count is dropped
    (void)hipStreamSynchronize(s);
    (void)hipFree(F->face_order);
    F->face_order = nullptr;
    F->face_order_n = 0;
  }
  if (F->arena_bytes < L.total) {
    if (F->arena) {
      (void)hipStreamSynchronize(s);
      (void)hipFree(F->arena);
      F->arena = nullptr;
      F->arena_bytes = 0;
    }
    he = pool_take(L.total, &F->arena, &F->arena_bytes, &F->device);
    if (he != hipSuccess) {
      F->arena_bytes = 0;
      return fail(he == hipErrorOutOfMemory ? CSC_OUT_OF_MEMORY : fail_hip(he));
    }
  }
  if (!F->h_stats) {
    he = pinned_take(&F->h_stats, &F->device);
    if (he != hipSuccess) return fail(fail_hip(he));
  }
  char* A = F->arena;
  F->n_meshes = n_meshes;
  F->verts = verts_d;
  F->nv = tv;
  F->nf = tf;
  F->ne = te;
  F->nbt = tb;
  F->opt = o;
  F->d_mesh = (MeshDesc*)(A + L.off[L_MESH]);
  F->f_off = (int32_t*)(A + L.off[L_FOFF]);
  F->v_off = (int32_t*)(A + L.off[L_VOFF]);
  F->brick_base = (int32_t*)(A + L.off[L_BBASE]);
  F->tris_g = (int32_t*)(A + L.off[L_TRIS]);
  F->face_mesh = (int32_t*)(A + L.off[L_FMESH]);
  F->vert_mesh = (int32_t*)(A + L.off[L_VMESH]);
  F->vtx_off = (int32_t*)(A + L.off[L_VTXOFF]);
  F->vtx_corners = (int32_t*)(A + L.off[L_VTXC]);
  F->face_edges = (int32_t*)(A + L.off[L_FEDGES]);
  F->edges = (int4*)(A + L.off[L_EDGES]);
  F->face_rec = (FaceRec*)(A + L.off[L_FREC]);
  F->edge_cls = (uint8_t*)(A + L.off[L_ECLS]);
  F->vinfo = (float4*)(A + L.off[L_VINFO]);
  F->vbits = (uint32_t*)(A + L.off[L_VBITS]);
  F->epoly = (int32_t*)(A + L.off[L_EPOLY]);
  F->vpoly = (int32_t*)(A + L.off[L_VPOLY]);
  F->brick_index = (int32_t*)(A + L.off[L_BINDEX]);
  F->brick_list = (int32_t*)(A + L.off[L_BLIST]);
  F->brick_mesh = (int32_t*)(A + L.off[L_BMESH]);
  F->first_slot = (int32_t*)(A + L.off[L_FIRST]);
  F->d_stats = (int64_t*)(A + L.off[L_STATS]);
  F->fslack = (uint8_t*)(A + L.off[L_FSLACK]);
  F->eslack = (uint8_t*)(A + L.off[L_ESLACK]);
  F->fabsorbed = (uint8_t*)(A + L.off[L_FABS]);
  F->built = F->synced = false;

  queued_on(F, stream);
  MeshTables M;
  M.n = 0;
  if (config_changed && n_meshes <= TABLE_MESHES) {
    for (int m = 0; m < n_meshes; m++) M.m[m] = mesh[m];
    M.md = F->d_mesh;
    M.f_off = F->f_off;
    M.v_off = F->v_off;
    M.brick_base = F->brick_base;
    M.n = n_meshes;
    M.nf = (int32_t)tf;
    M.nv = (int32_t)tv;
    M.nbt = (int32_t)tb;
  } else if (config_changed) {
    std::vector<int32_t> tabs(3 * (size_t)(n_meshes + 1));
    for (int m = 0; m <= n_meshes; m++) {
      tabs[m] = m < n_meshes ? mesh[m].f_off : (int32_t)tf;
      tabs[(n_meshes + 1) + m] = m < n_meshes ? mesh[m].v_off : (int32_t)tv;
      tabs[2 * (n_meshes + 1) + m] = m < n_meshes ? mesh[m].brick_base : (int32_t)tb;
    }
    CK(hipMemcpy(F->d_mesh, mesh.data(), sizeof(MeshDesc) * n_meshes, hipMemcpyHostToDevice));
    CK(hipMemcpy(F->f_off, tabs.data(), sizeof(int32_t) * (n_meshes + 1), hipMemcpyHostToDevice));
    CK(hipMemcpy(F->v_off, tabs.data() + (n_meshes + 1), sizeof(int32_t) * (n_meshes + 1), hipMemcpyHostToDevice));
    CK(hipMemcpy(F->brick_base, tabs.data() + 2 * (n_meshes + 1), sizeof(int32_t) * (n_meshes + 1),
                 hipMemcpyHostToDevice));
  }

  StageTimer timer(TS_BUILD, s);
  const int64_t nh = 3 * tf, ne = te;
  const float absorb = o.absorb_cells > 0.f ? o.absorb_cells : 0.f;
  const ZeroLayout z = zero_layout(pl, tb);
  char* zero = A + L.off[L_ZERO];
  int32_t* zi = (int32_t*)zero;
  uint8_t* marks = (uint8_t*)(zero + z.flags);
  int32_t* sums = (int32_t*)(A + L.off[L_SUMS]);
  const int64_t waves = pl.face_tiles * (BT / 64);
  int32_t *owned = sums, *epolys = owned + sums_of(waves), *vpolys = epolys + sums_of(3 * pl.face_tiles),
          *marked = vpolys + sums_of(pl.vertex_tiles);
  int32_t* eid = (int32_t*)(A + L.off[L_EID]);
  int32_t* twin = (int32_t*)(A + L.off[L_TWIN]);
  // 1. counters, coarse sums, brick flags and statistics cleared
  {
    const int64_t n = (int64_t)(z.bytes / 16);
    const unsigned need = grid_1d(n, 4 * BT);
    k_begin<<<need < 2048 ? need : 2048, BT, 0, s>>>((uint4*)zero, n, F->d_stats, M);
  }
  // 2. inputs, face records, band bricks, counts
  {
    InputArgs I;
    I.V = verts_d;
    I.T = tris_d;
    I.f_off = F->f_off;
    I.v_off = F->v_off;
    I.md = F->d_mesh;
    I.tg = F->tris_g;
    I.face_mesh = F->face_mesh;
    I.vert_mesh = F->vert_mesh;
    I.rec = F->face_rec;
    I.flag = marks;
    I.bucket_count = pl.buckets > 0 ? zi + z.count : nullptr;
    I.stats = F->d_stats;
    I.owned = owned;
    I.vpolys = vpolys;
    I.vertex_tiles = tv <= VERTEX_FANS ? pl.vertex_tiles : 0;
    I.nv = tv;
    I.nf = tf;
    I.face_tiles = pl.face_tiles;
    I.n_meshes = n_meshes;
    I.bucket_shift = pl.shift;
    I.buckets = pl.buckets;
    const int64_t cap = o.geom_blocks > 0 && o.geom_blocks < INPUT_BLOCKS ? o.geom_blocks : INPUT_BLOCKS;
    if (tf <= INPUT_SHARED) {
      const int64_t tiles = pl.face_tiles * (BT / 64);
      k_inputs<64><<<(unsigned)(tiles < cap ? tiles : cap), BT, 0, s>>>(I);
    } else {
      k_inputs<BT><<<(unsigned)(pl.face_tiles < cap ? pl.face_tiles : cap), BT, 0, s>>>(I);
    }
  }
  const int32_t* T = F->tris_g;
  // 3. vertex -> corner table, and the bricks counted and numbered
  BrickArgs bricks;
  bricks.flag = marks;
  bricks.index = F->brick_index;
  bricks.list = F->brick_list;
  bricks.bmesh = F->brick_mesh;
  bricks.brick_base = F->brick_base;
  bricks.first_slot = F->first_slot;
  bricks.stats = F->d_stats;
  bricks.marked = marked;
  bricks.nbt = tb;
  bricks.tiles = pl.brick_tiles;
  bricks.n_meshes = n_meshes;
  EdgeBase bases;
  bases.tg = T;
  bases.owned = owned;
  bases.eid = eid;
  bases.stats = F->d_stats;
  bases.nf = tf;
  bases.waves = waves;
  const int block = pl.big ? DEAL_BIG_TH : BT;
  bases.tiles = (tf + block - 1) / block;
  if (pl.buckets > 0) {
    DealArgs D;
    D.tg = T;
    D.nh = nh;
    D.tiles = pl.deal_tiles;
    D.nv = tv;
    D.bucket_count = zi + z.count;
    D.bucket_next = zi + z.next;
    D.pairs = (uint2*)(A + L.off[L_PAIRS]);
    D.off = F->vtx_off;
    D.corners = F->vtx_corners;
    D.shift = pl.shift;
    D.buckets = pl.buckets;
    const unsigned g = (unsigned)(1 + pl.deal_tiles + pl.brick_tiles);
    const unsigned gb = (unsigned)(pl.buckets + bases.tiles + pl.brick_tiles);
    const size_t lds = sizeof(int) << pl.shift;
    if (pl.big) {
      k_deal<DEAL_BIG_TH, DEAL_BIG_ITEMS><<<g, DEAL_BIG_TH, 0, s>>>(D, bricks, bases);
      k_bucket<DEAL_BIG_TH><<<gb, DEAL_BIG_TH, lds, s>>>(D, bricks, bases);
    } else {
      k_deal<DEAL_TH, DEAL_ITEMS><<<g, DEAL_TH, 0, s>>>(D, bricks, bases);
      k_bucket<DEAL_TH><<<gb, DEAL_TH, lds, s>>>(D, bricks, bases);
    }
  } else {
    uint32_t* keys = (uint32_t*)(A + L.off[L_PAIRS]);
    CK(sort_pairs(A + L.off[L_SORT], sort_bytes, (const uint32_t*)T, keys, nullptr, F->vtx_corners, nh, sort_bits, s));
    k_offsets<<<grid_1d(nh, BT), BT, 0, s>>>(keys, nh, tv, F->vtx_off);
    k_bricks<<<(unsigned)(1 + pl.brick_tiles), BT, 0, s>>>(bricks, bases, 0);
    k_bricks<<<(unsigned)(bases.tiles + pl.brick_tiles), BT, 0, s>>>(bricks, bases, 1);
  }
  // 4. per vertex: twins, pseudonormal, class, cone
  const VertexOut O = {o.ruff_mode, o.saddle_mode, o.force_both_sides, F->vert_mesh, F->d_mesh,
                       n_meshes,    absorb,        F->vinfo,           F->vbits};
  if (tv <= VERTEX_FANS)
    k_vertex_fan<<<grid_1d(tv, VF_THREADS / VF_LANES), VF_THREADS, 0, s>>>(verts_d, T, tv, F->vtx_off, F->vtx_corners, O,
                                                                           twin, vpolys, F->d_stats);
  else
    k_vertex<<<(unsigned)pl.vertex_tiles, VK_THREADS, 0, s>>>(verts_d, T, tv, F->vtx_off, F->vtx_corners, O, twin, vpolys,
                                                              F->d_stats);
  // 5. edges with their classes and extrusion sides; the vertex list
  {
    EdgeArgs E;
    E.rec = F->face_rec;
    E.twin = twin;
    E.face_mesh = F->face_mesh;
    E.md = F->d_mesh;
    E.edges = F->edges;
    E.face_edges = F->face_edges;
    E.cls = F->edge_cls;
    E.eslack = F->eslack;
    E.eid = eid;
    E.vbits = F->vbits;
    E.vpoly = F->vpoly;
    E.stats = F->d_stats;
    E.vpolys = vpolys;
    E.epolys = epolys;
    E.nf = tf;
    E.ne = ne;
    E.nv = tv;
    E.blocks = (nh + BT - 1) / BT;
    E.vertex_tiles = pl.vertex_tiles;
    E.absorb = absorb;
    E.n_meshes = n_meshes;
    E.force_both = o.force_both_sides;
    k_edges<<<(unsigned)(E.blocks + (pl.vertex_tiles + QV - 1) / QV), BT, 0, s>>>(E);
  }
  // 6. face slacks, the edge list (the class statistics, which only the feature
  // counts report, are taken by csc_features_sync when it reads them back)
  {
    ListArgs Q;
    Q.T = T;
    Q.face_edges = F->face_edges;
    Q.vbits = F->vbits;
    Q.eslack = F->eslack;
    Q.cls = F->edge_cls;
    Q.eid = eid;
    Q.fslack = F->fslack;
    Q.fabsorbed = F->fabsorbed;
    Q.epoly = F->epoly;
    Q.stats = F->d_stats;
    Q.epolys = epolys;
    // a list block adds up the sums before it: few blocks where there are many tiles
    Q.list_tiles = pl.face_tiles / 512 < 1 ? 1 : (pl.face_tiles / 512 > 32 ? 32 : pl.face_tiles / 512);
    Q.lists = (pl.face_tiles + Q.list_tiles - 1) / Q.list_tiles;
    Q.nf = tf;
    Q.ne = ne;
    k_lists<<<(unsigned)(Q.lists + pl.face_tiles), BT, 0, s>>>(Q);
  }
  F->classes_counted = false;
  CK(hipGetLastError());
#undef CK
  if (config_changed) F->mesh.swap(mesh);
  F->built = true;
  if (no_sync) return CSC_OK;
  int rc = csc_features_sync(F, stream);
  if (rc != CSC_OK) return fail(rc);
  *out = F;
  return CSC_OK;
}

extern "C" int csc_features_sync(csc_features* F, void* stream) {
  if (!F || !F->built || !F->h_stats) return CSC_INVALID_ARG;
  hipStream_t s = (hipStream_t)stream;
  queued_on(F, stream);
  const int64_t items = (F->ne / 16 > F->nv / 4 ? F->ne / 16 : F->nv / 4) + 1;
  hipError_t he = hipSuccess;
  if (!F->classes_counted && items <= STATS_ONE_BLOCK) {
    void* host = nullptr;
    he = hipHostGetDevicePointer(&host, F->h_stats, 0);
    if (he == hipSuccess)
      k_stats_out<<<1, 1024, 0, s>>>(F->edge_cls, F->ne, F->vbits, F->nv, F->d_stats, (int64_t*)host);
    if (he == hipSuccess) he = hipGetLastError();
  } else {
    if (!F->classes_counted)  // once per build: the classes stay until the next one
      k_class_stats<<<grid_1d(items < 1024 * 256 ? items : 1024 * 256, 256), 256, 0, s>>>(F->edge_cls, F->ne, F->vbits,
                                                                                         F->nv, F->d_stats);
    he = hipMemcpyAsync(F->h_stats, F->d_stats, sizeof(int64_t) * ST_COUNT, hipMemcpyDeviceToHost, s);
  }
  F->classes_counted = true;
  if (he == hipSuccess) he = hipStreamSynchronize(s);
  if (he != hipSuccess) return fail_hip(he);
  const int64_t* st = F->h_stats;
  int rc = status_from_errors((uint64_t)(uint32_t)st[ST_ERR], st[ST_NE], F->ne);
  if (rc != CSC_OK) {
    F->synced = false;
    return rc;
  }
  F->n_epoly = st[ST_NEPOLY];
  F->n_vpoly = st[ST_NVPOLY];
  F->n_bricks = st[ST_NBRICKS];
  csc_feature_info& I = F->info;
  I.n_vertices = F->nv;
  I.n_faces = F->nf;
  I.n_edges = F->ne;
  I.n_edge_polyhedra = F->n_epoly;
  I.n_vertex_polyhedra = F->n_vpoly;
  I.edges_convex = st[ST_E_CONVEX];
  I.edges_concave = st[ST_E_CONCAVE];
  I.edges_flat = st[ST_E_FLAT];
  I.edges_unknown = st[ST_E_UNKNOWN];
  I.vertices_convex = st[ST_V_CONVEX];
  I.vertices_concave = st[ST_V_CONCAVE];
  I.vertices_flat = st[ST_V_FLAT];
  I.vertices_saddle = st[ST_V_SADDLE];
  I.vertices_ruff = st[ST_V_RUFF];
  I.edges_absorbed = st[ST_E_ABSORBED];
  I.vertices_absorbed = st[ST_V_ABSORBED];
  I.n_bricks = F->n_bricks;
  I.max_band_cells = F->n_bricks * BRICK_CELLS;
  F->synced = true;
  return CSC_OK;
}

extern "C" int csc_build_features(const float* verts_d, int64_t nv, const int32_t* tris_d, int64_t nf,
                                  const csc_grid* grid, const csc_options* opt, void* stream, csc_features** out) {
  if (!grid) return CSC_INVALID_ARG;
  return build_impl(verts_d, tris_d, &nv, &nf, grid, 1, opt, 0, stream, out);
}

extern "C" int csc_build_features_batched(const float* verts_d, const int32_t* tris_d, const int64_t* nv,
                                          const int64_t* nf, const csc_grid* grids, int32_t n_meshes,
                                          const csc_options* opt, int32_t flags, void* stream, csc_features** out) {
  if (flags & ~(CSC_BUILD_NO_SYNC | CSC_BUILD_GRAPH_SAFE)) return CSC_INVALID_ARG;
  if ((flags & CSC_BUILD_NO_SYNC) && (!out || !*out)) return CSC_INVALID_ARG;
  return build_impl(verts_d, tris_d, nv, nf, grids, n_meshes, opt, flags, stream, out);
}
