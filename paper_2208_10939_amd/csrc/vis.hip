// Lit-facet mask per chirp and its compaction into per-chirp facet lists.
//
// Single-bounce reading of bidirectional analytic ray tracing (Section 2.2): a
// forward ray from the transmitter and a backward ray from the receiver meet on the
// same facet. Facet f is lit at chirp n when it faces both phase centres and
// neither segment centroid -> phase centre is blocked by another triangle. The
// geometry is that of chirp start t_n (stop-and-hop, eq. (12) per chirp).
//
// Layout: a workgroup per (8 or more facets, up to 64 chirps), lane = chirp. The facing test
// runs in FP64 on world coordinates; the shadow rays run in FP32 in each candidate instance's
// body frame, starting at the facet centroid (close to the occluders, so the FP32
// Moller-Trumbore test keeps its precision). The lanes of a wave trace nearly the same rays, so
// visibility walks a BVH once a wave: nodes and triangles in scalar registers, a mask of the
// lanes inside each node, one small stack a wave. Bound by the chain of a wave's node fetches
// and by its box tests. Few chirps of many facets, where a wave would hold many different walks,
// keep a walk per lane (launch_visibility has the rule). Against a walk per lane (32 node registers and an LDS stack column a
// lane, 4 waves a SIMD): 50k facets x 128 chirps 433 -> 190 us, 30k x 64 235 -> 74 us, 20k x 81
// with ground paths 565 -> 230 us, 1M x 256 15.0 -> 8.8 ms.
#include <algorithm>

#include "rsim_internal.h"
#include "rsim_launch.h"

namespace rsim {

namespace {

constexpr int kVisThreads = 256;
constexpr int kVisBitWords = 4 * 64;  // LDS bit words: path types x chirps x mask words

__device__ inline int find_instance(const DevInstance *inst, int n_inst, int64_t f) {
  int lo = 0, hi = n_inst - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (inst[mid].facet_base <= f)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

__device__ inline bool box_hit(const float *lo, const float *hi, float ox, float oy, float oz,
                               float ix, float iy, float iz, float pad = 0.0f) {
  float tx0 = (lo[0] - pad - ox) * ix, tx1 = (hi[0] + pad - ox) * ix;
  float ty0 = (lo[1] - pad - oy) * iy, ty1 = (hi[1] + pad - oy) * iy;
  float tz0 = (lo[2] - pad - oz) * iz, tz1 = (hi[2] + pad - oz) * iz;
  float tn = fmaxf(fmaxf(fminf(tx0, tx1), fminf(ty0, ty1)), fmaxf(fminf(tz0, tz1), 0.0f));
  float tf = fminf(fminf(fmaxf(tx0, tx1), fmaxf(ty0, ty1)), fminf(fmaxf(tz0, tz1), 1.0f));
  return tn <= tf;
}

__device__ inline float safe_inv(float d) {
  const float tiny = 1e-30f;
  return 1.0f / (fabsf(d) > tiny ? d : copysignf(tiny, d));
}

// A flat (horizontal) instance cannot block the segment c -> s: c lies no lower than its
// lowest vertex and at most 0.5e-6 m below its highest, and s lies at least 1 m above c,
// so for t >= kTEps the segment runs at least 0.5e-6 m above every vertex (a ground facet's
// rays towards the array leave the road grid's BVH untouched).
__device__ inline bool flat_below(const DevInstance &I, const double c[3], double s_z) {
  return I.flat && c[2] >= I.flat_lo && I.flat_hi - c[2] <= 0.5e-6 && s_z - c[2] >= 1.0;
}

struct LeafTriangle {
  float4 a, b, c;  // v0 = a.xyz, e1 = (a.w, b.x, b.y), e2 = (b.z, b.w, c.x), id = c.y
};

// Does the segment o -> o + d[r] of some r hit the triangle (closed test, t in [kTEps, 1 - kTEps])?
// The roundings are spelled out, those of one segment and of two as the compiler once chose them
// (u's sum alone differs): a segment through an edge is decided by them.
template <int NR>
__device__ inline bool triangle_hit(const LeafTriangle &tr, float ox, float oy, float oz,
                                    const float (&d)[NR][3]) {
  const float e1x = tr.a.w, e1y = tr.b.x, e1z = tr.b.y;
  const float e2x = tr.b.z, e2y = tr.b.w, e2z = tr.c.x;
  const float sx = ox - tr.a.x, sy = oy - tr.a.y, sz = oz - tr.a.z;
  const float qx = fmaf(sy, e1z, -(sz * e1y)), qy = fmaf(sz, e1x, -(sx * e1z)),
              qz = fmaf(sx, e1y, -(sy * e1x));
  bool hit = false;
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const float dx = d[r][0], dy = d[r][1], dz = d[r][2];
    const float px = fmaf(dy, e2z, -(dz * e2y)), py = fmaf(dz, e2x, -(dx * e2z)),
                pz = fmaf(dx, e2y, -(dy * e2x));
    const float det = fmaf(e1z, pz, fmaf(e1x, px, e1y * py));
    const float un = NR == 2 ? fmaf(sz, pz, fmaf(sy, py, sx * px))
                             : fmaf(sz, pz, fmaf(sx, px, sy * py));
    // clearly outside [0, 1], and no need for the quotient to see it (the bounds leave
    // room for its rounding, and for one that underflows to zero)
    const bool outside = un * det < -0x1p-100f || fabsf(un) > 1.0001f * fabsf(det);
    if (hit || outside || det == 0.0f) continue;
    const float inv = 1.0f / det;
    const float u = un * inv;
    if (!(u >= 0.0f && u <= 1.0f)) continue;
    const float vn = fmaf(dz, qz, fmaf(dx, qx, dy * qy));
    if (!(vn * inv >= 0.0f && fmaf(vn, inv, u) <= 1.0f)) continue;
    const float t = fmaf(e2z, qz, fmaf(e2x, qx, e2y * qy)) * inv;
    hit = t >= kTEps && t <= 1.0f - kTEps;
  }
  return hit;
}

// |d1 - d2| rounded up (FP32 sqrt is correctly rounded; the factor covers the rest): the boxes
// are grown by it where two segments are walked as one.
template <int NR>
__device__ inline float walk_pad(const float (&d)[NR][3]) {
  if constexpr (NR == 1) return 0.0f;
  const float ex = d[0][0] - d[NR - 1][0], ey = d[0][1] - d[NR - 1][1],
              ez = d[0][2] - d[NR - 1][2];
  return __builtin_sqrtf(ex * ex + ey * ey + ez * ez) * 1.0001f + 1e-7f;
}

// Lanes of `in` with a segment that hits a triangle of the leaf.
template <int NR>
__device__ inline uint64_t packet_leaf(const float4 *leaf, int32_t ref, float ox, float oy,
                                       float oz, const float (&d)[NR][3], int32_t skip,
                                       uint64_t in) {
  const uint32_t code = static_cast<uint32_t>(-ref - 1);
  const uint32_t first = code >> 4, count = code & 15u;
  uint64_t blocked = 0;
  for (uint32_t k = 0; k < count && in; ++k) {
    const LeafTriangle tr =
        load_uniform(reinterpret_cast<const LeafTriangle *>(leaf) + (first + k));
    bool hit = false;
    if (__builtin_amdgcn_inverse_ballot_w64(in) && __float_as_int(tr.c.y) != skip)
      hit = triangle_hit<NR>(tr, ox, oy, oz, d);
    const uint64_t now = __ballot(hit);
    blocked |= now;
    in &= ~now;
  }
  return blocked;
}

// Any-hit traversal of one four-wide BLAS by the lanes of `in` together, each with the NR
// body-frame segments o -> o + d[r]: the lanes blocked. The node is the wave's (nodes and
// triangles come through the scalar cache), with the mask of the lanes that entered it, so
// each lane meets just the boxes and triangles that a walk of its own would: leaves are tested
// when their box is hit, the first inner child hit is entered next and the other ones (at most
// three per level) wait on the wave's stack. With two segments a node is entered when the first
// meets its box grown by |d1 - d2| on every side: the points of the two at the same parameter
// are at most that far apart, so this enters every node either meets (and a few more).
template <int NR>
__device__ uint64_t packet_occluded(const BvhNode4 *nodes, const float4 *leaf, float ox, float oy,
                                    float oz, const float (&d)[NR][3], int32_t skip, uint64_t in,
                                    uint4 *stack) {
  const float ix = safe_inv(d[0][0]), iy = safe_inv(d[0][1]), iz = safe_inv(d[0][2]);
  const float pad = walk_pad<NR>(d);
  uint64_t open = in, m = in;
  int sp = 0;
  int32_t node = 0;
  while (true) {
    const BvhNode4 nd = load_uniform(nodes + node);
    int32_t next = -1;
    uint64_t next_m = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float lo[3] = {nd.lo[0][i], nd.lo[1][i], nd.lo[2][i]};
      const float hi[3] = {nd.hi[0][i], nd.hi[1][i], nd.hi[2][i]};
      const uint64_t mi = __ballot(box_hit(lo, hi, ox, oy, oz, ix, iy, iz, pad)) & m & open;
      if (!mi) continue;
      const int32_t c = nd.c[i];
      if (c < 0) {
        open &= ~packet_leaf<NR>(leaf, c, ox, oy, oz, d, skip, mi);
      } else if (next >= 0) {
        // <= 3 per level: stack_depth = 3 (depth + 1)
        stack[sp] = make_uint4(static_cast<uint32_t>(c), static_cast<uint32_t>(mi),
                               static_cast<uint32_t>(mi >> 32), 0u);
        ++sp;
      } else {
        next = c;
        next_m = mi;
      }
    }
    m = next_m & open;
    node = next;
    while (!m) {
      if (sp == 0 || !open) return in & ~open;
      --sp;
      const uint4 e = stack[sp];
      node = __builtin_amdgcn_readfirstlane(static_cast<int32_t>(e.x));
      m = (static_cast<uint64_t>(static_cast<uint32_t>(
               __builtin_amdgcn_readfirstlane(static_cast<int32_t>(e.z)))) << 32 |
           static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int32_t>(e.y)))) &
          open;
    }
  }
}

// The same for one lane, in a walk of its own with a stack column of its own.
template <int NR>
__device__ bool lane_occluded(const BvhNode4 *nodes, const float4 *leaf, float ox, float oy,
                              float oz, const float (&d)[NR][3], int32_t skip, int32_t *stack,
                              int stride) {
  const float ix = safe_inv(d[0][0]), iy = safe_inv(d[0][1]), iz = safe_inv(d[0][2]);
  const float pad = walk_pad<NR>(d);
  int sp = 0;
  int32_t node = 0;
  while (true) {
    const BvhNode4 nd = nodes[node];
    int32_t next = -1;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float lo[3] = {nd.lo[0][i], nd.lo[1][i], nd.lo[2][i]};
      const float hi[3] = {nd.hi[0][i], nd.hi[1][i], nd.hi[2][i]};
      if (!box_hit(lo, hi, ox, oy, oz, ix, iy, iz, pad)) continue;
      const int32_t c = nd.c[i];
      if (c < 0) {
        const uint32_t code = static_cast<uint32_t>(-c - 1);
        const LeafTriangle *tr = reinterpret_cast<const LeafTriangle *>(leaf) + (code >> 4);
        for (uint32_t k = 0; k < (code & 15u); ++k)
          if (__float_as_int(tr[k].c.y) != skip && triangle_hit<NR>(tr[k], ox, oy, oz, d))
            return true;
      } else if (next >= 0) {
        stack[sp * stride] = c;  // <= 3 per level: stack_depth = 3 (depth + 1)
        ++sp;
      } else {
        next = c;
      }
    }
    if (next < 0) {
      if (sp == 0) return false;
      --sp;
      next = stack[sp * stride];
    }
    node = next;
  }
}

// How a wave's lanes walk: together (stack: the wave's), or each for itself (stack: the lane's
// column of int32, `stride` apart).
struct PacketWalk {
  uint4 *stack;
  static constexpr bool kTogether = true;
};
struct LaneWalk {
  int32_t *stack;
  int stride;
  static constexpr bool kTogether = false;
};

// Is the world segment c -> s[r] of some r blocked by a triangle of the scene at time t
// (triangle `self_local` of instance `self_inst` excluded), for the lanes with `on`? All lanes of
// the wave call it where they walk together.
template <int NR, typename Walk>
__device__ bool segments_blocked(const DevScene &sc, bool on, double t, const double c[3],
                                 const double *const (&s)[NR], int self_inst, int32_t self_local,
                                 const Walk &walk, bool skip_plane, uint64_t cand) {
  if (!Walk::kTogether && !on) return false;
  double dw[NR][3], idw[NR][3];
  // reciprocals once per segment (the boxes are padded, so the rounding of a product
  // instead of a quotient cannot turn a hit box into a miss)
  for (int r = 0; r < NR; ++r)
    for (int k = 0; k < 3; ++k) {
      dw[r][k] = s[r][k] - c[k];
      idw[r][k] = dw[r][k] != 0.0 ? 1.0 / dw[r][k] : 0.0;
    }
  uint64_t open = Walk::kTogether ? __ballot(on) : 0;
  const uint64_t all = open;
  for (int j = 0; j < sc.n_inst; ++j) {
    if (Walk::kTogether && !open) break;
    const DevInstance &I = sc.inst[j];
    if (!I.has_bvh) continue;
    if (skip_plane && I.in_plane) continue;  // the road surface under a reflected leg
    // no segment of the facet over the group's chirps meets its box (instances from 64 on are
    // not filtered)
    const bool may = j >= 64 || ((cand >> j) & 1u);
    uint64_t m = 0;
    if constexpr (Walk::kTogether) {
      m = __ballot(may) & open;
      if (!m) continue;
    } else if (!may) {
      continue;
    }
    bool below = true;
    for (int r = 0; r < NR; ++r) below = below && flat_below(I, c, s[r][2]);
    if (!Walk::kTogether && below) continue;
    const double p[3] = {I.pos0[0] + I.vel[0] * t, I.pos0[1] + I.vel[1] * t,
                         I.pos0[2] + I.vel[2] * t};
    // world-space slab test of each segment against the instance box (FP64, conservative box)
    bool any = false;
    for (int r = 0; r < NR; ++r) {
      double tn = 0.0, tf = 1.0;
      bool miss = false;
      for (int k = 0; k < 3; ++k) {
        const double lo = I.box_lo[k] + p[k], hi = I.box_hi[k] + p[k];
        if (dw[r][k] == 0.0) {
          if (c[k] < lo || c[k] > hi) miss = true;
          continue;
        }
        const double a = (lo - c[k]) * idw[r][k], b = (hi - c[k]) * idw[r][k];
        tn = fmax(tn, fmin(a, b));
        tf = fmin(tf, fmax(a, b));
      }
      any = any || !(miss || tn > tf);
    }
    if constexpr (Walk::kTogether) {
      m &= __ballot(any && !below);
      if (!m) continue;
    } else if (!any) {
      continue;
    }
    // body frame: x_body = R^T (x - p)
    const double *R = I.rot;
    const double q0 = c[0] - p[0], q1 = c[1] - p[1], q2 = c[2] - p[2];
    const float ox = static_cast<float>(R[0] * q0 + R[3] * q1 + R[6] * q2);
    const float oy = static_cast<float>(R[1] * q0 + R[4] * q1 + R[7] * q2);
    const float oz = static_cast<float>(R[2] * q0 + R[5] * q1 + R[8] * q2);
    float d[NR][3];
    for (int r = 0; r < NR; ++r)
      for (int k = 0; k < 3; ++k)
        d[r][k] = static_cast<float>(R[k] * dw[r][0] + R[3 + k] * dw[r][1] + R[6 + k] * dw[r][2]);
    const int32_t skip = (j == self_inst) ? self_local : -1;
    if constexpr (Walk::kTogether)
      open &= ~packet_occluded<NR>(I.nodes, I.leaf, ox, oy, oz, d, skip, m, walk.stack);
    else if (lane_occluded<NR>(I.nodes, I.leaf, ox, oy, oz, d, skip, walk.stack, walk.stride))
      return true;
  }
  if constexpr (Walk::kTogether) return __builtin_amdgcn_inverse_ballot_w64(all & ~open);
  return false;
}

// Does the segment a -> b meet the box [lo, hi] (FP64 slab test, closed)?
__device__ inline bool seg_box(const double a[3], const double b[3], const double lo[3],
                               const double hi[3]) {
  double tn = 0.0, tf = 1.0;
  for (int k = 0; k < 3; ++k) {
    const double d = b[k] - a[k];
    if (d == 0.0) {
      if (a[k] < lo[k] || a[k] > hi[k]) return false;
      continue;
    }
    const double u = (lo[k] - a[k]) / d, w = (hi[k] - a[k]) / d;
    tn = fmax(tn, fmin(u, w));
    tf = fmin(tf, fmax(u, w));
  }
  return tn <= tf;
}

// World box of instance I swept over the times [ta, tb] and grown by g[k] on each side.
__device__ inline void swept_box(const DevInstance &I, double ta, double tb, const double g[3],
                                 double lo[3], double hi[3]) {
  for (int k = 0; k < 3; ++k) {
    const double pa = I.pos0[k] + I.vel[k] * ta, pb = I.pos0[k] + I.vel[k] * tb;
    lo[k] = I.box_lo[k] + fmin(pa, pb) - g[k];
    hi[k] = I.box_hi[k] + fmax(pa, pb) + g[k];
  }
}

// May the box of instance j be met by some segment c(t) -> T or c(t) -> R, c(t) the centroid of
// facet f at the chirp times t of chirps n_a .. n_b? Tested with the segments from the centroid
// at the middle time, against the box swept over the chirps' times and grown by the centroid's
// sweep about its middle position (the point at parameter s of c(t) -> S differs from that
// of c_m -> S by (1 - s)(c(t) - c_m)) and by 1e-6 m against rounding. True wherever the
// per-chirp FP64 box test admits the instance, so the decisions are those without it.
__device__ bool candidate(const DevScene &sc, const RadarConst &rc, int64_t f, int j, int n_a,
                          int n_b) {
  const double ta = n_a * rc.tc, tb = n_b * rc.tc, tm = 0.5 * (ta + tb);
  const DevInstance &F = sc.inst[find_instance(sc.inst, sc.n_inst, f)];
  const int32_t lt = static_cast<int32_t>(f - F.facet_base);
  double b[3] = {0.0, 0.0, 0.0};
  for (int v = 0; v < 3; ++v) {
    const int32_t vi = F.tris[3 * lt + v];
    for (int k = 0; k < 3; ++k) b[k] += F.verts[3 * vi + k];
  }
  double cm[3], hw[3];
  for (int k = 0; k < 3; ++k) {
    cm[k] = (F.rot[3 * k + 0] * b[0] + F.rot[3 * k + 1] * b[1] + F.rot[3 * k + 2] * b[2]) / 3.0 +
            (F.pos0[k] + F.vel[k] * tm);
    hw[k] = fabs(F.vel[k]) * (0.5 * (tb - ta)) + 1e-6;
  }
  double lo[3], hi[3];
  swept_box(sc.inst[j], ta, tb, hw, lo, hi);
  return seg_box(cm, rc.tx_c, lo, hi) || seg_box(cm, rc.rx_c, lo, hi);
}

// One side (phase centre E, facing value fe = n . (E - c)) of a facet: *direct when it
// faces E and centroid -> E is clear; *reflected when the centroid lies above the ground
// plane, the facet faces the image E' and both legs centroid -> S -> E are clear, S the
// specular point (the road surface is skipped for these legs).
template <typename Walk>
__device__ void reflected_sides(const DevScene &sc, const RadarConst &rc, bool on, double t,
                                const double c[3], const double n[3], const double E[3], double fe,
                                int ii, int32_t lt, const Walk &walk, bool *direct, bool *refl) {
  const uint64_t every = ~uint64_t(0);
  const bool facing = on && fe > 0.0;
  *direct = !segments_blocked<1>(sc, facing, t, c, {E}, ii, lt, walk, false, every) && facing;
  const double ez = 2.0 * rc.z_ground - E[2];  // image height
  const double fi = n[0] * (E[0] - c[0]) + n[1] * (E[1] - c[1]) + n[2] * (ez - c[2]);
  bool clear = on && c[2] > rc.z_ground && fi > 0.0;
  const double a = (c[2] - rc.z_ground) / (c[2] - ez);
  const double S[3] = {c[0] + a * (E[0] - c[0]), c[1] + a * (E[1] - c[1]), rc.z_ground};
  clear = !segments_blocked<1>(sc, clear, t, c, {S}, ii, lt, walk, true, every) && clear;
  *refl = !segments_blocked<1>(sc, clear, t, S, {E}, -1, -1, walk, true, every) && clear;
}

}  // namespace

namespace {

// Lit decisions of facet f at chirp n: the single path (lit[0]) or, with the ground bounce,
// the four path types (transmit side k & 1, receive side k >> 1). All lanes of the wave call
// it; those without `on` get none.
template <bool BOUNCE, typename Walk>
__device__ void facet_lit(const DevScene &sc, const RadarConst &rc, bool on, int64_t f, int n,
                          const Walk &walk, uint64_t cand, bool lit[4]) {
  lit[0] = lit[1] = lit[2] = lit[3] = false;
  const double t = n * rc.tc;
  const int ii = find_instance(sc.inst, sc.n_inst, f);
  const DevInstance &I = sc.inst[ii];
  const int32_t lt = static_cast<int32_t>(f - I.facet_base);
  double x[3][3];
  for (int v = 0; v < 3; ++v) {
    const int32_t vi = I.tris[3 * lt + v];
    const double b0 = I.verts[3 * vi + 0], b1 = I.verts[3 * vi + 1], b2 = I.verts[3 * vi + 2];
    for (int k = 0; k < 3; ++k)
      x[v][k] = I.rot[3 * k + 0] * b0 + I.rot[3 * k + 1] * b1 + I.rot[3 * k + 2] * b2 +
                (I.pos0[k] + I.vel[k] * t);
  }
  double c[3], e1[3], e2[3];
  for (int k = 0; k < 3; ++k) {
    c[k] = (x[0][k] + x[1][k] + x[2][k]) / 3.0;
    e1[k] = x[1][k] - x[0][k];
    e2[k] = x[2][k] - x[0][k];
  }
  const double nx = e1[1] * e2[2] - e1[2] * e2[1];
  const double ny = e1[2] * e2[0] - e1[0] * e2[2];
  const double nz = e1[0] * e2[1] - e1[1] * e2[0];
  on = on && (nx != 0.0 || ny != 0.0 || nz != 0.0);
  const double ft = nx * (rc.tx_c[0] - c[0]) + ny * (rc.tx_c[1] - c[1]) + nz * (rc.tx_c[2] - c[2]);
  const double fr = nx * (rc.rx_c[0] - c[0]) + ny * (rc.rx_c[1] - c[1]) + nz * (rc.rx_c[2] - c[2]);
  if constexpr (!BOUNCE) {
    on = on && ft > 0.0 && fr > 0.0;
    if (__ballot(on))
      lit[0] =
          !segments_blocked<2>(sc, on, t, c, {rc.tx_c, rc.rx_c}, ii, lt, walk, false, cand) && on;
  } else {
    const double nv[3] = {nx, ny, nz};
    bool dt, it, dr, ir;
    reflected_sides(sc, rc, on, t, c, nv, rc.tx_c, ft, ii, lt, walk, &dt, &it);
    reflected_sides(sc, rc, on, t, c, nv, rc.rx_c, fr, ii, lt, walk, &dr, &ir);
    lit[0] = dt && dr;
    lit[1] = it && dr;
    lit[2] = dt && ir;
    lit[3] = it && ir;
  }
}

}  // namespace

// A workgroup covers facets_per_block facets (8, 16 or whole mask words) and `cw` consecutive
// chirps (a power of two up to 64); lane = chirp within the group, so the lanes of a wave trace
// nearly the same rays of one facet at neighbouring chirps and follow nearly one BVH path
// (mapping lanes to neighbouring facets instead makes every wave walk the union of 64
// different paths). Decisions are gathered as bits in LDS and written as whole bytes or words.
template <bool BOUNCE, typename Walk>
__global__ void __launch_bounds__(2 * kVisThreads) __attribute__((amdgpu_waves_per_eu(4, 8)))
vis_kernel(DevScene sc, RadarConst rc, int cw, int facets_per_block, bool find, int n_begin,
           int n_end) {
  extern __shared__ __align__(16) int32_t vis_lds[];
  __shared__ uint32_t cand_lds[kVisThreads][2];
  const int words = max(1, facets_per_block >> 5);
  constexpr int types = BOUNCE ? 4 : 1;
  uint32_t *bits = reinterpret_cast<uint32_t *>(vis_lds);  // [types][cw][words]
  Walk walk;
  if constexpr (Walk::kTogether)
    walk = {reinterpret_cast<uint4 *>(vis_lds + kVisBitWords) + (threadIdx.x >> 6) * sc.stack_depth};
  else
    walk = {vis_lds + kVisBitWords + threadIdx.x, static_cast<int>(blockDim.x)};
  for (int k = threadIdx.x; k < types * cw * words; k += blockDim.x) bits[k] = 0u;
  const int nl = threadIdx.x % cw;
  const int n = n_begin + static_cast<int>(blockIdx.y) * cw + nl;
  const int64_t f0 = static_cast<int64_t>(blockIdx.x) * facets_per_block;
  // The instances that each facet's segments may meet are found first where that pays
  // (launch_visibility has the rule), a thread per (facet, instance), into LDS.
  const bool filter = !BOUNCE && find;
  for (int k = threadIdx.x; k < 2 * facets_per_block; k += blockDim.x) (&cand_lds[0][0])[k] = 0u;
  __syncthreads();
  if (filter) {
    const int n_a = n_begin + static_cast<int>(blockIdx.y) * cw;
    const int n_b = min(n_end, n_a + cw) - 1;
    const int ni = min(sc.n_inst, 64);
    for (int k = threadIdx.x; k < facets_per_block * ni; k += blockDim.x) {
      const int fl = k / ni, j = k % ni;
      if (f0 + fl < sc.n_facets && candidate(sc, rc, f0 + fl, j, n_a, n_b))
        atomicOr(&cand_lds[fl][j >> 5], 1u << (j & 31));
    }
    __syncthreads();
  }
  // the lanes past the last facet or chirp go along with those that have work
  for (int fl = threadIdx.x / cw; fl < facets_per_block; fl += blockDim.x / cw) {
    const bool on = f0 + fl < sc.n_facets && n < n_end;
    if (!__ballot(on)) continue;
    const uint64_t cand =
        filter ? static_cast<uint64_t>(cand_lds[fl][1]) << 32 | cand_lds[fl][0] : ~uint64_t(0);
    bool lit[4];
    facet_lit<BOUNCE>(sc, rc, on, min(f0 + fl, sc.n_facets - 1), min(n, n_end - 1), walk, cand, lit);
    for (int k = 0; k < types; ++k)
      if (lit[k]) atomicOr(&bits[(k * cw + nl) * words + (fl >> 5)], 1u << (fl & 31));
  }
  __syncthreads();
  for (int e = threadIdx.x; e < types * cw * words; e += blockDim.x) {
    const int w = e % words, r = e / words;  // r = k * cw + chirp within the group
    const int k = r / cw, nn = n_begin + static_cast<int>(blockIdx.y) * cw + (r % cw);
    const int64_t at = f0 + 32 * w;  // first facet of these bits
    if (nn >= n_end || at >= 32 * sc.mask_words) continue;
    uint32_t *row = sc.mask + (static_cast<int64_t>(k) * rc.N + nn) * sc.mask_words;
    if (facets_per_block >= 32)
      row[at >> 5] = bits[e];
    else if (facets_per_block == 16)
      reinterpret_cast<uint16_t *>(row)[at >> 4] = static_cast<uint16_t>(bits[e]);
    else
      reinterpret_cast<uint8_t *>(row)[at >> 3] = static_cast<uint8_t>(bits[e]);
  }
}

// Per-chirp compaction of the mask into ascending facet indices (deterministic).
__global__ void __launch_bounds__(1024) compact_kernel(DevScene sc, int n_begin) {
  __shared__ int32_t s_scan[1024];
  const int n = n_begin + static_cast<int>(blockIdx.x);
  const uint32_t *row = sc.mask + static_cast<int64_t>(n) * sc.mask_words;
  const int64_t per = (sc.mask_words + blockDim.x - 1) / blockDim.x;
  const int64_t w0 = static_cast<int64_t>(threadIdx.x) * per;
  const int64_t w1 = min(sc.mask_words, w0 + per);
  const uint32_t tail_bits = static_cast<uint32_t>(sc.n_facets & 31);
  int32_t cnt = 0;
  for (int64_t w = w0; w < w1; ++w) {
    uint32_t b = row[w];
    if (w == sc.mask_words - 1 && tail_bits) b &= (1u << tail_bits) - 1u;
    cnt += __popc(b);
  }
  s_scan[threadIdx.x] = cnt;
  __syncthreads();
  for (int off = 1; off < static_cast<int>(blockDim.x); off <<= 1) {
    int32_t v = (threadIdx.x >= static_cast<unsigned>(off)) ? s_scan[threadIdx.x - off] : 0;
    __syncthreads();
    s_scan[threadIdx.x] += v;
    __syncthreads();
  }
  int32_t pos = s_scan[threadIdx.x] - cnt;
  int32_t *out = sc.vis_idx + static_cast<int64_t>(n) * sc.n_facets;
  for (int64_t w = w0; w < w1; ++w) {
    uint32_t b = row[w];
    if (w == sc.mask_words - 1 && tail_bits) b &= (1u << tail_bits) - 1u;
    while (b) {
      const int bit = __ffs(b) - 1;
      out[pos++] = static_cast<int32_t>(w * 32 + bit);
      b &= b - 1u;
    }
  }
  if (threadIdx.x == blockDim.x - 1) sc.vis_cnt[n] = s_scan[threadIdx.x];
}

// ---- facet-to-facet double bounce: connections ----------------------------------------

namespace {

// Slab test of the body-frame ray o + t d against a box for t in [0, t_end].
__device__ inline bool box_hit_t(const float *lo, const float *hi, float ox, float oy, float oz,
                                 float ix, float iy, float iz, float t_end) {
  float tx0 = (lo[0] - ox) * ix, tx1 = (hi[0] - ox) * ix;
  float ty0 = (lo[1] - oy) * iy, ty1 = (hi[1] - oy) * iy;
  float tz0 = (lo[2] - oz) * iz, tz1 = (hi[2] - oz) * iz;
  float tn = fmaxf(fmaxf(fminf(tx0, tx1), fminf(ty0, ty1)), fmaxf(fminf(tz0, tz1), 0.0f));
  float tf = fminf(fminf(fmaxf(tx0, tx1), fmaxf(ty0, ty1)), fminf(fmaxf(tz0, tz1), t_end));
  return tn <= tf;
}

// Nearer hits of the leaf's triangles by o + t d, t in (t_min, t_best) (closed test):
// shrinks t_best and records the triangle id.
__device__ inline void leaf_closest(const float4 *leaf, int32_t ref, float ox, float oy, float oz,
                                    float dx, float dy, float dz, int32_t skip, float t_min,
                                    float &t_best, int32_t &id) {
  uint32_t code = static_cast<uint32_t>(-ref - 1);
  uint32_t first = code >> 4, count = code & 15u;
  for (uint32_t k = 0; k < count; ++k) {
    const float4 a = leaf[3 * (first + k) + 0];
    const float4 b = leaf[3 * (first + k) + 1];
    const float4 c = leaf[3 * (first + k) + 2];
    const int32_t tid = __float_as_int(c.y);
    if (tid == skip) continue;
    float e1x = a.w, e1y = b.x, e1z = b.y;
    float e2x = b.z, e2y = b.w, e2z = c.x;
    float px = dy * e2z - dz * e2y, py = dz * e2x - dx * e2z, pz = dx * e2y - dy * e2x;
    float det = e1x * px + e1y * py + e1z * pz;
    if (det == 0.0f) continue;
    float inv = 1.0f / det;
    float sx = ox - a.x, sy = oy - a.y, sz = oz - a.z;
    float u = (sx * px + sy * py + sz * pz) * inv;
    if (!(u >= 0.0f && u <= 1.0f)) continue;
    float qx = sy * e1z - sz * e1y, qy = sz * e1x - sx * e1z, qz = sx * e1y - sy * e1x;
    float v = (dx * qx + dy * qy + dz * qz) * inv;
    if (!(v >= 0.0f && u + v <= 1.0f)) continue;
    float t = (e2x * qx + e2y * qy + e2z * qz) * inv;
    if (t > t_min && t < t_best) {
      t_best = t;
      id = tid;
    }
  }
}

// Closest-hit traversal of one four-wide BLAS (body frame; the same stack discipline as
// blas_occluded: at most three pending children per level).
__device__ void blas_closest(const BvhNode4 *nodes, const float4 *leaf, float ox, float oy,
                             float oz, float dx, float dy, float dz, int32_t skip, float t_min,
                             float &t_best, int32_t &id, int32_t *stack, int stride) {
  const float ix = safe_inv(dx), iy = safe_inv(dy), iz = safe_inv(dz);
  int sp = 0;
  int32_t node = 0;
  while (true) {
    const BvhNode4 nd = nodes[node];
    int32_t next = -1;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float lo[3] = {nd.lo[0][i], nd.lo[1][i], nd.lo[2][i]};
      const float hi[3] = {nd.hi[0][i], nd.hi[1][i], nd.hi[2][i]};
      if (!box_hit_t(lo, hi, ox, oy, oz, ix, iy, iz, t_best)) continue;
      const int32_t c = nd.c[i];
      if (c < 0) {
        leaf_closest(leaf, c, ox, oy, oz, dx, dy, dz, skip, t_min, t_best, id);
      } else if (next >= 0) {
        stack[sp * stride] = c;
        ++sp;
      } else {
        next = c;
      }
    }
    if (next < 0) {
      if (sp == 0) return;
      --sp;
      next = stack[sp * stride];
    }
    node = next;
  }
}

__device__ inline void world_vertices(const DevInstance &I, int64_t lt, double t, double x[3][3]) {
  for (int v = 0; v < 3; ++v) {
    const int32_t vi = I.tris[3 * lt + v];
    const double b0 = I.verts[3 * vi + 0], b1 = I.verts[3 * vi + 1], b2 = I.verts[3 * vi + 2];
    for (int k = 0; k < 3; ++k)
      x[v][k] = I.rot[3 * k + 0] * b0 + I.rot[3 * k + 1] * b1 + I.rot[3 * k + 2] * b2 +
                (I.pos0[k] + I.vel[k] * t);
  }
}

// Unit normal (CCW) and centroid of a world triangle; false for zero area.
__device__ inline bool tri_frame(const double x[3][3], double c[3], double n[3]) {
  double e1[3], e2[3];
  for (int k = 0; k < 3; ++k) {
    c[k] = (x[0][k] + x[1][k] + x[2][k]) / 3.0;
    e1[k] = x[1][k] - x[0][k];
    e2[k] = x[2][k] - x[0][k];
  }
  n[0] = e1[1] * e2[2] - e1[2] * e2[1];
  n[1] = e1[2] * e2[0] - e1[0] * e2[2];
  n[2] = e1[0] * e2[1] - e1[1] * e2[0];
  const double a = sqrt(n[0] * n[0] + n[1] * n[1] + n[2] * n[2]);
  if (!(a > 0.0)) return false;
  for (int k = 0; k < 3; ++k) n[k] /= a;
  return true;
}

__device__ inline double dot3(const double *a, const double *b) {
  return a[0] * b[0] + a[1] * b[1] + a[2] * b[2];
}

// The pair search's instance filter for facet f and instance j at chirps n_a .. n_b: may, for
// launching end k, the shadow segment c(t) -> E (bit 2 k) or the specular segment c(t) -> c(t) +
// ray_len r(t) (bit 2 k + 1) of some chirp meet the instance? The segments at the
// middle time are tested against its box swept over the chirps' times and grown: by the centroid's
// sweep per axis for the shadow segment (as in visibility); for the specular one by
// |delta| (1 + 2 ray_len / (|E - c_m| - |delta|)), |delta| the centroid's largest
// displacement from its middle position (the unit vector towards E turns by at most
// 2 |delta| / (|E - c_m| - |delta|), and the mirror in A's plane, fixed under translation,
// keeps that), plus 1e-6 m against rounding. True wherever the per-chirp FP64 box
// tests admit the instance, and where that bound does not apply.
__device__ uint32_t db_candidate(const DevScene &sc, const RadarConst &rc, int64_t f, int j,
                                 int n_a, int n_b, double ray_len) {
  const double ta = n_a * rc.tc, tb = n_b * rc.tc, tm = 0.5 * (ta + tb);
  const DevInstance &A = sc.inst[find_instance(sc.inst, sc.n_inst, f)];
  const DevInstance &I = sc.inst[j];
  double x[3][3], c[3], na[3];
  world_vertices(A, f - A.facet_base, tm, x);
  const bool ok = tri_frame(x, c, na);
  double hw[3], sweep = 0.0;
  for (int k = 0; k < 3; ++k) {
    const double dk = fabs(A.vel[k]) * (0.5 * (tb - ta));
    hw[k] = dk + 1e-6;
    sweep += dk * dk;
  }
  sweep = sqrt(sweep);
  uint32_t may = 0;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const double *E = k ? rc.rx_c : rc.tx_c;
    double de[3] = {E[0] - c[0], E[1] - c[1], E[2] - c[2]};
    const double ld = sqrt(dot3(de, de));
    if (!ok || !(ld - sweep > 0.0)) {
      may |= 3u << (2 * k);
      continue;
    }
    double r[3], end[3];
    for (int q = 0; q < 3; ++q) r[q] = -de[q] / ld;
    const double rn = dot3(r, na);
    for (int q = 0; q < 3; ++q) end[q] = c[q] + ray_len * (r[q] - 2.0 * rn * na[q]);
    const double g = sweep * (1.0 + 2.0 * ray_len / (ld - sweep)) + 1e-6;
    const double gr[3] = {g, g, g};
    double lo[3], hi[3];
    swept_box(I, ta, tb, hw, lo, hi);
    if (seg_box(c, E, lo, hi)) may |= 1u << (2 * k);
    swept_box(I, ta, tb, gr, lo, hi);
    if (seg_box(c, end, lo, hi)) may |= 2u << (2 * k);
  }
  return may;
}

// Facet B that the ray launched from end k (0: Tx phase centre, 1: Rx) reflected off facet A
// (scene index f) connects to at chirp n, or -1 (Section 2.2; the rules of the oracle's
// facet-to-facet double bounce): A faces the launching centre E and sees it; the specular
// ray from A's centroid first hits B (FP32 traversal over a segment of ray_len metres); B
// faces the image E' of E in A's plane and the other centre O, and the segment from the
// hit point to O is clear; the central projection from E' of A's vertices onto B's plane
// lies ahead of E' (parameters above 1/2) and within 1.5 r_lim of its centroid. Reads
// the chirp's lit mask (computed before, single path).
__device__ int32_t db_connect(const DevScene &sc, const RadarConst &rc, int64_t f, int n, int k,
                              double ray_len, double r_lim, int32_t *stk, int stride,
                              uint64_t cand_e, uint64_t cand_r) {
  const double t = n * rc.tc;
  const double *E = k ? rc.rx_c : rc.tx_c;
  const double *O = k ? rc.tx_c : rc.rx_c;
  const int ia = find_instance(sc.inst, sc.n_inst, f);
  const DevInstance &IA = sc.inst[ia];
  const int32_t la = static_cast<int32_t>(f - IA.facet_base);
  double xa[3][3], ca[3], na[3];
  world_vertices(IA, la, t, xa);
  if (!tri_frame(xa, ca, na)) return -1;
  double de[3] = {E[0] - ca[0], E[1] - ca[1], E[2] - ca[2]};
  const double fe = dot3(na, de);
  if (!(fe > 0.0)) return -1;
  // A lit facet (single path, this chirp's mask) faces both centres with both segments from
  // its centroid clear, the one to E among them: its test is not repeated
  const bool lit = (sc.mask[static_cast<int64_t>(n) * sc.mask_words + (f >> 5)] >> (f & 31)) & 1u;
  const LaneWalk walk{stk, stride};
  if (!lit && segments_blocked<1>(sc, true, t, ca, {E}, ia, la, walk, false, cand_e)) return -1;
  // specular direction of d = (c_A - E) / |c_A - E|
  const double ld = sqrt(dot3(de, de));
  double r[3];
  for (int q = 0; q < 3; ++q) r[q] = -de[q] / ld;
  const double rn = dot3(r, na);
  for (int q = 0; q < 3; ++q) r[q] -= 2.0 * rn * na[q];
  // first hit over all instances (A excluded), t as a fraction of ray_len
  float t_best = 1.0f;
  int32_t id_best = -1, inst_best = -1;
  const double ir[3] = {r[0] != 0.0 ? 1.0 / (r[0] * ray_len) : 0.0,
                        r[1] != 0.0 ? 1.0 / (r[1] * ray_len) : 0.0,
                        r[2] != 0.0 ? 1.0 / (r[2] * ray_len) : 0.0};
  const float t_min = static_cast<float>(1e-6 / ray_len);
  for (int j = 0; j < sc.n_inst; ++j) {
    if (j < 64 && !((cand_r >> j) & 1u)) continue;  // no specular segment of the facet
                                                    // over the group's chirps meets it
    const DevInstance &I = sc.inst[j];
    if (!I.has_bvh) continue;
    double p[3] = {I.pos0[0] + I.vel[0] * t, I.pos0[1] + I.vel[1] * t, I.pos0[2] + I.vel[2] * t};
    double tn = 0.0, tf = static_cast<double>(t_best);
    bool miss = false;
    for (int q = 0; q < 3; ++q) {
      const double lo = I.box_lo[q] + p[q], hi = I.box_hi[q] + p[q];
      if (r[q] == 0.0) {
        if (ca[q] < lo || ca[q] > hi) miss = true;
        continue;
      }
      const double a = (lo - ca[q]) * ir[q], b = (hi - ca[q]) * ir[q];
      tn = fmax(tn, fmin(a, b));
      tf = fmin(tf, fmax(a, b));
    }
    if (miss || tn > tf) continue;
    const double *R = I.rot;
    const double q0 = ca[0] - p[0], q1 = ca[1] - p[1], q2 = ca[2] - p[2];
    const float ox = static_cast<float>(R[0] * q0 + R[3] * q1 + R[6] * q2);
    const float oy = static_cast<float>(R[1] * q0 + R[4] * q1 + R[7] * q2);
    const float oz = static_cast<float>(R[2] * q0 + R[5] * q1 + R[8] * q2);
    const double d0 = r[0] * ray_len, d1 = r[1] * ray_len, d2 = r[2] * ray_len;
    const float dx = static_cast<float>(R[0] * d0 + R[3] * d1 + R[6] * d2);
    const float dy = static_cast<float>(R[1] * d0 + R[4] * d1 + R[7] * d2);
    const float dz = static_cast<float>(R[2] * d0 + R[5] * d1 + R[8] * d2);
    int32_t id = -1;
    blas_closest(I.nodes, I.leaf, ox, oy, oz, dx, dy, dz, j == ia ? la : -1, t_min, t_best, id,
                 stk, stride);
    if (id >= 0) {
      id_best = id;
      inst_best = j;
    }
  }
  if (id_best < 0) return -1;
  const DevInstance &IB = sc.inst[inst_best];
  double xb[3][3], cb[3], nb[3];
  world_vertices(IB, id_best, t, xb);
  if (!tri_frame(xb, cb, nb)) return -1;
  const double th = static_cast<double>(t_best) * ray_len;
  const double h[3] = {ca[0] + th * r[0], ca[1] + th * r[1], ca[2] + th * r[2]};
  double ei[3];
  for (int q = 0; q < 3; ++q) ei[q] = E[q] - 2.0 * fe * na[q];
  const double f1 = nb[0] * (ei[0] - h[0]) + nb[1] * (ei[1] - h[1]) + nb[2] * (ei[2] - h[2]);
  const double f2 = nb[0] * (O[0] - h[0]) + nb[1] * (O[1] - h[1]) + nb[2] * (O[2] - h[2]);
  if (!(f1 > 0.0) || !(f2 > 0.0)) return -1;
  if (segments_blocked<1>(sc, true, t, h, {O}, inst_best, id_best, walk, false, ~uint64_t(0)))
    return -1;
  // footprint of A's tube on B's plane
  const double num = nb[0] * (cb[0] - ei[0]) + nb[1] * (cb[1] - ei[1]) + nb[2] * (cb[2] - ei[2]);
  double fp[3][3], cf[3] = {0.0, 0.0, 0.0};
  for (int v = 0; v < 3; ++v) {
    double dv[3] = {xa[v][0] - ei[0], xa[v][1] - ei[1], xa[v][2] - ei[2]};
    const double den = dot3(nb, dv);
    const double sv = num / den;
    if (!(sv > 0.5) || !isfinite(sv)) return -1;
    for (int q = 0; q < 3; ++q) {
      fp[v][q] = ei[q] + sv * dv[q];
      cf[q] += fp[v][q] / 3.0;
    }
  }
  const double lim2 = 2.25 * r_lim * r_lim;
  for (int v = 0; v < 3; ++v) {
    const double a = fp[v][0] - cf[0], b = fp[v][1] - cf[1], c = fp[v][2] - cf[2];
    if (!(a * a + b * b + c * c <= lim2)) return -1;
  }
  return static_cast<int32_t>(IB.facet_base + id_best);
}

}  // namespace

// Connections of every facet at chirps n_begin .. n_begin + n_chirps - 1, both launching
// ends: pair_b[(k N + n) F + f]. Lane = chirp, as in vis_kernel. Bound by the walks of the BVH,
// each lane its own (the nearest hit depends on the order of a walk where triangles tie): the
// instance filter for every size, four waves a SIMD and one pass a workgroup took 2.30 -> 1.12
// ms for 120k facets of 7 instances and 64 chirps, 0.42 -> 0.14 ms for 20k of one.
__global__ void __launch_bounds__(kVisThreads) __attribute__((amdgpu_waves_per_eu(4, 8))) dbounce_kernel(DevScene sc, RadarConst rc, int cw,
                                                            int facets_per_block, int n_begin,
                                                            int n_end, double ray_len,
                                                            double r_lim, int32_t *pair_b) {
  extern __shared__ int32_t db_lds[];
  uint32_t *cand = reinterpret_cast<uint32_t *>(db_lds);             // [facet][segment][2 words]
  int32_t *stk = db_lds + 8 * facets_per_block + threadIdx.x;  // column per thread
  const int nl = threadIdx.x % cw;
  const int n = n_begin + static_cast<int>(blockIdx.y) * cw + nl;
  const int64_t f0 = static_cast<int64_t>(blockIdx.x) * facets_per_block;
  // with several instances, those that each facet's segments may meet are found first, a thread
  // per (facet, instance)
  const bool filter = sc.n_inst > 1;
  for (int k = threadIdx.x; k < 8 * facets_per_block; k += blockDim.x) cand[k] = 0u;
  __syncthreads();
  if (filter) {
    const int n_a = n_begin + static_cast<int>(blockIdx.y) * cw;
    const int n_b = min(n_end, n_a + cw) - 1;
    const int ni = min(sc.n_inst, 64);
    for (int k = threadIdx.x; k < facets_per_block * ni; k += blockDim.x) {
      const int fl = k / ni, j = k % ni;
      if (f0 + fl >= sc.n_facets) break;
      const uint32_t may = db_candidate(sc, rc, f0 + fl, j, n_a, n_b, ray_len);
      for (int q = 0; q < 4; ++q)
        if ((may >> q) & 1u) atomicOr(&cand[8 * fl + 2 * q + (j >> 5)], 1u << (j & 31));
    }
    __syncthreads();
  }
  const auto of = [&](int fl, int q) {
    const uint32_t *w = cand + 8 * fl + 2 * q;
    return filter ? static_cast<uint64_t>(w[1]) << 32 | w[0] : ~uint64_t(0);
  };
  for (int fl = threadIdx.x / cw; fl < facets_per_block; fl += blockDim.x / cw) {
    const int64_t f = f0 + fl;
    if (f >= sc.n_facets || n >= n_end) continue;
    for (int k = 0; k < 2; ++k) {
      pair_b[(static_cast<int64_t>(k) * rc.N + n) * sc.n_facets + f] =
          db_connect(sc, rc, f, n, k, ray_len, r_lim, stk, blockDim.x, of(fl, 2 * k), of(fl, 2 * k + 1));
    }
  }
}

// Per (end, chirp): the connected facets in ascending order and their count (deterministic).
// The row is read in tiles of one element per thread (coalesced); ballots and the waves'
// counts in LDS (two sets, alternating per tile, so one barrier per tile) place each
// connected facet.
__global__ void __launch_bounds__(1024) db_compact_kernel(const int32_t *pair_b, int64_t F,
                                                          int32_t *idx, int32_t *cnt) {
  __shared__ int32_t s_w[2][16];
  const int64_t row = blockIdx.x;  // k N + n
  const int32_t *b = pair_b + row * F;
  int32_t *out = idx + row * F;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
  int32_t base = 0;
  int par = 0;
  for (int64_t t0 = 0; t0 < F; t0 += blockDim.x, par ^= 1) {
    const int64_t i = t0 + threadIdx.x;
    const int32_t v = i < F ? b[i] : -1;
    const bool on = v >= 0 && v < F;  // others: no connection
    const uint64_t m = __ballot(on);
    if (lane == 0) s_w[par][wv] = __popcll(m);
    __syncthreads();
    int32_t before = 0, total = 0;
    for (int w = 0; w < nw; ++w) {
      const int32_t c = s_w[par][w];
      before += w < wv ? c : 0;
      total += c;
    }
    if (on) out[base + before + __popcll(m & ((uint64_t(1) << lane) - 1))] = static_cast<int32_t>(i);
    base += total;
  }
  if (threadIdx.x == 0) cnt[row] = base;
}

hipError_t launch_dbounce(const DevScene &sc, const RadarConst &rc, double ray_len, double r_lim,
                          int32_t *pair_b, int32_t *idx, int32_t *cnt, hipStream_t s) {
  if (rc.N <= 0) return hipSuccess;
  if (sc.n_facets > 0 && ray_len > 0.0) {
    int cw = 1;
    while (cw < rc.N && cw < 64) cw <<= 1;
    // as in visibility: few facets leave lanes idle rather than waves (20k facets, 4 chirps:
    // 179 us at cw 4, 129 at 32)
    while (cw < 32 && sc.n_facets * cw < int64_t{64} * 8192) cw <<= 1;
    const int fpb = kVisThreads / cw;  // one pass a workgroup: the walks' lengths differ widely
    dim3 grid(static_cast<unsigned>((sc.n_facets + fpb - 1) / fpb),
              static_cast<unsigned>((rc.N + cw - 1) / cw));
    const size_t lds =
        sizeof(int32_t) * (8 * fpb + static_cast<size_t>(sc.stack_depth) * kVisThreads);
    hipLaunchKernelGGL(dbounce_kernel, grid, dim3(kVisThreads), lds, s, sc, rc, cw, fpb, 0,
                       rc.N, ray_len, r_lim, pair_b);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(db_compact_kernel, dim3(static_cast<unsigned>(2 * rc.N)), dim3(1024), 0, s,
                     pair_b, sc.n_facets, idx, cnt);
  return hipGetLastError();
}

hipError_t launch_visibility(const DevScene &sc, const RadarConst &rc, int n_begin, int n_chirps,
                             hipStream_t s) {
  if (sc.n_facets == 0 || n_chirps <= 0) return hipSuccess;
  if (n_begin < 0 || n_begin + n_chirps > rc.N) return hipErrorInvalidValue;
  // Chirps per group: the smallest power of two >= the count, at most 64.
  int cw = 1, threads = kVisThreads, fpb = 8;
  while (cw < n_chirps && cw < 64) cw <<= 1;
  const auto chirp_groups = [&] { return (n_chirps + cw - 1) / cw; };
  // Lanes that each walk for themselves where a wave's would hold the walks of many facets: one
  // chirp and half a million facets or more (1.5M in 3 instances 2.3 ms, 2.7 together), with the
  // ground's paths up to 4 chirps and two waves of them a SIMD (300k facets, one chirp: 0.36 ms,
  // 0.62 together; 4 chirps 0.45, 0.60; 8 chirps 0.62, 0.59; 30k facets, 4 chirps 0.20, 0.15).
  const int64_t lanes = sc.n_facets * cw;
  const bool together = !(rc.bounce ? n_chirps <= 4 && lanes >= int64_t{120} << 10
                                    : n_chirps == 1 && lanes >= int64_t{64} * 8192);
  if (together) {
    // A wave walks the union of the paths of its 64 / cw facets, which costs less than a pass for
    // each once the passes fill the chip; below some 8192 passes idle lanes cost less than the
    // longer walk (20k facets, 4 chirps: 235 us at cw 4, 72 at 32, 101 at 64; 500k facets, 8
    // chirps: 733 at cw 8, 1146 at 32).
    while (cw < 32 && sc.n_facets * cw < int64_t{64} * 8192) cw <<= 1;
    if (sc.n_facets * ((n_chirps + 63) / 64) <= 8192) {
      // a wave's one chain of nodes is the time: one facet a wave (1k facets, 4 chirps: 24 us; 30
      // at cw 32 with 256 threads. 30k facets, 64 chirps: 84, 74 with 256)
      cw = 64;
      threads = 2 * kVisThreads;
    }
    // Facets per workgroup, 8, 16 or whole mask words: small ones even out the waves' work, large
    // ones share the start of a workgroup (50k facets, 128 chirps: 190 us at 8, 232 at 32; 1M
    // facets, 256 chirps: 9740 at 8, 8770 at 32)
    while (fpb < 32 && sc.n_facets * chirp_groups() > int64_t{16384} * fpb) fpb *= 2;
    fpb = std::max(fpb, threads / cw);
  } else {
    fpb = std::max(32, threads / cw);  // whole mask words, every thread busy for cw >= 8
  }
  // The instance filter (single path) costs an FP64 test of swept boxes for each facet and
  // instance, and saves one of each instance's box for every chirp: over 33 chirps or more it pays;
  // over fewer only with many instances, from 17 chirps on (21 of 30k facets, 24 chirps: 1.19 ms,
  // 1.30 without; 4 chirps 0.69, 0.52) or where few facets leave the chip waiting for the longest
  // wave (21 of 1.5k, 4 chirps: 82 us, 92 without; 3 of 9.5k: 74, 63).
  const bool filter = !rc.bounce && sc.n_inst > 1 &&
                      (n_chirps > 32 ||
                       (sc.n_inst > 8 && (n_chirps > 16 || sc.n_facets <= 32768)));
  dim3 grid(static_cast<unsigned>((32 * sc.mask_words + fpb - 1) / fpb),
            static_cast<unsigned>(chirp_groups()));
  // bit words: types x cw x words <= 4 x 64 (fpb > 32 only with cw < 8)
  const size_t stacks = together ? sizeof(uint4) * (threads / 64) : sizeof(int32_t) * threads;
  const size_t lds = sizeof(int32_t) * kVisBitWords + stacks * static_cast<size_t>(sc.stack_depth);
  const auto kernel =
      together ? (rc.bounce ? vis_kernel<true, PacketWalk> : vis_kernel<false, PacketWalk>)
               : (rc.bounce ? vis_kernel<true, LaneWalk> : vis_kernel<false, LaneWalk>);
  hipLaunchKernelGGL(kernel, grid, dim3(threads), lds, s, sc, rc, cw, fpb, filter, n_begin,
                     n_begin + n_chirps);
  return hipGetLastError();
}

hipError_t launch_compact(const DevScene &sc, int n_begin, int n_chirps, hipStream_t s) {
  if (n_chirps <= 0) return hipSuccess;
  hipLaunchKernelGGL(compact_kernel, dim3(n_chirps), dim3(1024), 0, s, sc, n_begin);
  return hipGetLastError();
}

}  // namespace rsim
