// Host-side binned-SAH BVH builder for one mesh in its body frame.
//
// Visibility of a facet (single-bounce reading of the bidirectional ray tracing of
// Section 2.2) needs "any triangle blocks this segment" queries for every facet and
// chirp. Meshes are rigid, so each is indexed once at load time in its body frame
// and rays are moved into that frame per instance and chirp.
#include <emmintrin.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <exception>
#include <limits>
#include <system_error>
#include <thread>
#include <vector>

#include "rsim_internal.h"

namespace rsim {

using V4 = __m128;  // one vector register

// as std::min(a, b), std::max(a, b): the first unless the second is smaller (larger)
inline V4 min4(V4 a, V4 b) { return _mm_min_ps(b, a); }
inline V4 max4(V4 a, V4 b) { return _mm_max_ps(b, a); }

// The fourth lanes of the bounds hold the triangle and its bins; c's stays zero, because sums
// and quotients of such bits would be subnormal and many times slower.
struct BuildPrim {
  V4 lo, hi, c;
  int32_t id() const {
    int32_t v;
    std::memcpy(&v, reinterpret_cast<const char *>(&lo) + 12, 4);
    return v;
  }
  void set_id(int32_t v) { std::memcpy(reinterpret_cast<char *>(&lo) + 12, &v, 4); }
  // bins of the last binning pass on axis k
  int bin(int k) const { return reinterpret_cast<const unsigned char *>(&hi)[12 + k]; }
  void set_bins(const int32_t *b) {
    unsigned char *p = reinterpret_cast<unsigned char *>(&hi) + 12;
    for (int k = 0; k < 3; ++k) p[k] = static_cast<unsigned char>(b[k]);
  }
};

struct Box {
  V4 lo = {std::numeric_limits<float>::infinity(), std::numeric_limits<float>::infinity(),
           std::numeric_limits<float>::infinity(), 0.0f};
  V4 hi = {-std::numeric_limits<float>::infinity(), -std::numeric_limits<float>::infinity(),
           -std::numeric_limits<float>::infinity(), 0.0f};
  void grow(V4 l, V4 h) {
    lo = min4(lo, l);
    hi = max4(hi, h);
  }
  bool empty() const { return !(lo[0] <= hi[0]); }
  double area() const {
    if (empty()) return 0.0;
    const V4 d = hi - lo;
    double dx = d[0], dy = d[1], dz = d[2];
    return 2.0 * (dx * dy + dy * dz + dz * dx);
  }
};

// Forks of the build: subtrees of at least kForkMin triangles (about 1 ms of building against
// some 50 us for a thread) down to kForkLevels, so at most 8 threads for the time of the call.
constexpr int64_t kForkMin = 4096;
constexpr int kForkLevels = 3;

struct Builder {
  BuildPrim *prims;
  std::vector<BvhNode> nodes;
  std::vector<int32_t> order;
  int max_depth = 0;

  static int32_t leaf_ref(int64_t first, int64_t count) {
    return -(1 + static_cast<int32_t>((first << 4) | count));
  }

  int32_t make_leaf(int64_t b, int64_t e) {
    int64_t first = static_cast<int64_t>(order.size());
    for (int64_t i = b; i < e; ++i) order.push_back(prims[i].id());
    return leaf_ref(first, e - b);
  }

  // Takes over a subtree that another builder made, root `ref`; returns its ref here. Nodes and
  // leaves are numbered in the order of a build without threads.
  int32_t append(const Builder &o, int32_t ref) {
    const int32_t node0 = static_cast<int32_t>(nodes.size());
    const int64_t leaf0 = static_cast<int64_t>(order.size());
    const auto move = [&](int32_t c) {
      return c >= 0 ? c + node0 : c - static_cast<int32_t>(leaf0 << 4);
    };
    for (BvhNode nd : o.nodes) {
      nd.c0 = move(nd.c0);
      nd.c1 = move(nd.c1);
      nodes.push_back(nd);
    }
    order.insert(order.end(), o.order.begin(), o.order.end());
    max_depth = std::max(max_depth, o.max_depth);
    return move(ref);
  }

  // Builds the subtree over prims[b, e), returns its child ref; box = its bounds.
  int32_t build(int64_t b, int64_t e, int depth, Box &box) {
    box = Box();
    Box cb;
    for (int64_t i = b; i < e; ++i) {
      box.grow(prims[i].lo, prims[i].hi);
      cb.grow(prims[i].c, prims[i].c);
    }
    max_depth = std::max(max_depth, depth);
    const int64_t n = e - b;
    if (n <= kLeafMax) return make_leaf(b, e);
    constexpr int kBins = 16;
    double best_cost = std::numeric_limits<double>::infinity();
    int best_axis = -1, best_split = -1;
    const V4 ext = cb.hi - cb.lo;
    if (depth < 32) {  // median splits below keep depth <= 32 + 26
      // one pass bins all three axes (an axis without extent is not read)
      Box bin_box[3][kBins];
      int32_t bin_n[3][kBins] = {};
      const V4 width = {ext[0] > 0.0f ? ext[0] : 1.0f, ext[1] > 0.0f ? ext[1] : 1.0f,
                        ext[2] > 0.0f ? ext[2] : 1.0f, 1.0f};
      const V4 bins = _mm_set1_ps(kBins), top = _mm_set1_ps(kBins - 1);
      for (int64_t i = b; i < e; ++i) {
        BuildPrim &p = prims[i];
        const V4 q = _mm_min_ps(_mm_max_ps(bins * ((p.c - cb.lo) / width), _mm_setzero_ps()), top);
        alignas(16) int32_t k[4];
        _mm_store_si128(reinterpret_cast<__m128i *>(k), _mm_cvttps_epi32(q));
        p.set_bins(k);
        for (int ax = 0; ax < 3; ++ax) {
          bin_n[ax][k[ax]]++;
          bin_box[ax][k[ax]].grow(p.lo, p.hi);
        }
      }
      for (int ax = 0; ax < 3; ++ax) {
        if (!(ext[ax] > 0.0f)) continue;
        // an empty bin moves neither side's box nor count, so its split is the last one's again
        double right_area[kBins];
        int64_t right_n[kBins];
        Box acc;
        int64_t cnt = 0;
        double area = 0.0;
        for (int k = kBins - 1; k > 0; --k) {
          if (bin_n[ax][k]) {
            acc.grow(bin_box[ax][k].lo, bin_box[ax][k].hi);
            area = acc.area();
            cnt += bin_n[ax][k];
          }
          right_area[k] = area;
          right_n[k] = cnt;
        }
        Box lacc;
        int64_t lcnt = 0;
        for (int k = 1; k < kBins; ++k) {
          if (!bin_n[ax][k - 1]) continue;
          lacc.grow(bin_box[ax][k - 1].lo, bin_box[ax][k - 1].hi);
          lcnt += bin_n[ax][k - 1];
          if (right_n[k] == 0) continue;
          double cost = lacc.area() * lcnt + right_area[k] * right_n[k];
          if (cost < best_cost) {
            best_cost = cost;
            best_axis = ax;
            best_split = k;
          }
        }
      }
    }
    int64_t mid;
    if (best_axis >= 0) {
      auto it = std::partition(prims + b, prims + e, [&](const BuildPrim &p) {
        return p.bin(best_axis) < best_split;
      });
      mid = it - prims;
    } else {
      mid = b;  // fall through to the median split below
    }
    if (mid <= b || mid >= e) {
      // median split on the widest centroid axis (degenerate or deep subtrees)
      int ax = 0;
      float widest = -1.0f;
      for (int k = 0; k < 3; ++k)
        if (ext[k] > widest) {
          widest = ext[k];
          ax = k;
        }
      mid = b + n / 2;
      std::nth_element(prims + b, prims + mid, prims + e,
                       [ax](const BuildPrim &p, const BuildPrim &q) { return p.c[ax] < q.c[ax]; });
    }
    int32_t me = static_cast<int32_t>(nodes.size());
    nodes.emplace_back();
    Box lb, rb;
    int32_t l, r;
    Builder right{prims};
    std::exception_ptr error;
    std::thread worker;
    if (depth < kForkLevels && std::min(mid - b, e - mid) >= kForkMin &&
        std::thread::hardware_concurrency() > 1) {
      try {
        worker = std::thread([&] {
          try {
            r = right.build(mid, e, depth + 1, rb);
          } catch (...) {
            error = std::current_exception();
          }
        });
      } catch (const std::system_error &) {  // no thread to be had: built below
      }
    }
    if (worker.joinable()) {
      try {
        l = build(b, mid, depth + 1, lb);
      } catch (...) {
        worker.join();
        throw;
      }
      worker.join();
      if (error) std::rethrow_exception(error);
      r = append(right, r);
    } else {
      l = build(b, mid, depth + 1, lb);
      r = build(mid, e, depth + 1, rb);
    }
    BvhNode &nd = nodes[me];
    std::memset(&nd, 0, sizeof(nd));
    for (int k = 0; k < 3; ++k) {
      nd.lo0[k] = lb.lo[k];
      nd.hi0[k] = lb.hi[k];
      nd.lo1[k] = rb.lo[k];
      nd.hi1[k] = rb.hi[k];
    }
    nd.c0 = l;
    nd.c1 = r;
    return me;
  }
};

// Inflate a box so FP32 slab tests stay conservative (a box that is slightly too
// large costs time, never a missed occluder).
static void inflate(float *lo, float *hi) {
  for (int k = 0; k < 3; ++k) {
    if (!(lo[k] <= hi[k])) continue;
    float pad = 1e-5f * (std::fabs(lo[k]) + std::fabs(hi[k]) + (hi[k] - lo[k])) + 1e-6f;
    lo[k] -= pad;
    hi[k] += pad;
  }
}

// Four-wide node `n4` from binary node n: its children are the two children of each inner
// binary child (with the boxes that child holds) or the binary child itself when it is a
// leaf; inner ones are collapsed in turn. Returns the four-wide index; *depth the deepest
// four-wide level below (root level 0).
static int32_t collapse(const std::vector<BvhNode> &bin, int32_t n, int level,
                        std::vector<BvhNode4> &out, int *depth) {
  *depth = std::max(*depth, level);
  const int32_t me = static_cast<int32_t>(out.size());
  out.emplace_back();
  BvhNode4 nd;
  std::memset(&nd, 0, sizeof(nd));
  int ne = 0;
  auto put = [&](int32_t ref, const float *lo, const float *hi) {
    for (int k = 0; k < 3; ++k) {
      nd.lo[k][ne] = lo[k];
      nd.hi[k][ne] = hi[k];
    }
    nd.c[ne++] = ref;
  };
  const BvhNode &b = bin[n];
  for (int side = 0; side < 2; ++side) {
    const int32_t ref = side ? b.c1 : b.c0;
    if (ref >= 0) {
      const BvhNode &g = bin[ref];
      put(g.c0, g.lo0, g.hi0);
      put(g.c1, g.lo1, g.hi1);
    } else {
      put(ref, side ? b.lo1 : b.lo0, side ? b.hi1 : b.hi0);
    }
  }
  for (; ne < 4; ++ne) {  // empty slots: never entered
    for (int k = 0; k < 3; ++k) {
      nd.lo[k][ne] = 1.0f;
      nd.hi[k][ne] = -1.0f;
    }
    nd.c[ne] = Builder::leaf_ref(0, 0);
  }
  for (int i = 0; i < 4; ++i)
    if (nd.c[i] >= 0) nd.c[i] = collapse(bin, nd.c[i], level + 1, out, depth);
  out[me] = nd;
  return me;
}

// Builds the four-wide nodes (root = node 0) and leaf triangles (3 float4 each).
// Degenerate (zero-area) triangles are left out: they never block. Returns the depth of the
// four-wide tree (root 0), or -1 if no triangle has area.
int build_bvh(const float *verts, const int32_t *tris, int64_t n_tris,
              std::vector<BvhNode4> &nodes_out, std::vector<float> &leaf_out) {
  std::vector<BuildPrim> prims;
  prims.reserve(n_tris);
  for (int64_t t = 0; t < n_tris; ++t) {
    const float *a = verts + 3 * tris[3 * t + 0];
    const float *b = verts + 3 * tris[3 * t + 1];
    const float *c = verts + 3 * tris[3 * t + 2];
    double e1[3], e2[3];
    for (int k = 0; k < 3; ++k) {
      e1[k] = double(b[k]) - a[k];
      e2[k] = double(c[k]) - a[k];
    }
    double nx = e1[1] * e2[2] - e1[2] * e2[1];
    double ny = e1[2] * e2[0] - e1[0] * e2[2];
    double nz = e1[0] * e2[1] - e1[1] * e2[0];
    if (nx == 0.0 && ny == 0.0 && nz == 0.0) continue;
    BuildPrim p{};
    for (int k = 0; k < 3; ++k) {
      p.lo[k] = std::min(a[k], std::min(b[k], c[k]));
      p.hi[k] = std::max(a[k], std::max(b[k], c[k]));
      p.c[k] = (a[k] + b[k] + c[k]) / 3.0f;
    }
    p.set_id(static_cast<int32_t>(t));
    prims.push_back(p);
  }
  nodes_out.clear();
  leaf_out.clear();
  if (prims.empty()) return -1;
  const int64_t np = static_cast<int64_t>(prims.size());
  Builder bd{prims.data()};
  bd.order.reserve(np);
  bd.nodes.reserve(2 * np / kLeafMax + 2);
  if (np <= kLeafMax) {
    // root with one leaf child and one empty child
    bd.nodes.emplace_back();
    Box lb;
    int32_t l = bd.build(0, np, 1, lb);
    BvhNode &nd = bd.nodes[0];
    std::memset(&nd, 0, sizeof(nd));
    for (int k = 0; k < 3; ++k) {
      nd.lo0[k] = lb.lo[k];
      nd.hi0[k] = lb.hi[k];
      nd.lo1[k] = 1.0f;   // empty box: lo > hi never hits
      nd.hi1[k] = -1.0f;
    }
    nd.c0 = l;
    nd.c1 = Builder::leaf_ref(0, 0);
  } else {
    Box root;
    bd.build(0, np, 0, root);
  }
  for (auto &nd : bd.nodes) {
    inflate(nd.lo0, nd.hi0);
    inflate(nd.lo1, nd.hi1);
  }
  nodes_out.reserve(bd.nodes.size() / 2 + 1);
  int depth4 = 0;
  collapse(bd.nodes, 0, 0, nodes_out, &depth4);
  leaf_out.resize(bd.order.size() * 12);
  for (size_t i = 0; i < bd.order.size(); ++i) {
    int32_t t = bd.order[i];
    const float *a = verts + 3 * tris[3 * t + 0];
    const float *b = verts + 3 * tris[3 * t + 1];
    const float *c = verts + 3 * tris[3 * t + 2];
    float *o = leaf_out.data() + 12 * i;
    o[0] = a[0]; o[1] = a[1]; o[2] = a[2];
    o[3] = b[0] - a[0]; o[4] = b[1] - a[1]; o[5] = b[2] - a[2];
    o[6] = c[0] - a[0]; o[7] = c[1] - a[1]; o[8] = c[2] - a[2];
    std::memcpy(&o[9], &t, sizeof(int32_t));
    o[10] = 0.0f;
    o[11] = 0.0f;
  }
  return depth4;
}

}  // namespace rsim
