// C ABI of the walk-on-boundary library: argument validation, scene upload and
// kernel dispatch.  The kernels themselves live in walk.hpp / device.hpp.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <cmath>
#include <cstring>
#include <functional>
#include <limits>
#include <new>
#include <vector>

#include "../../include/wob.h"
#include "bvh_build.hpp"
#include "internal.hpp"


using namespace wobi;

namespace {

// Leaves of at most two primitives (test_leaves tests a leaf's primitives side
// by side, their records loaded together).
constexpr int kMaxLeaf = wob::kLeafPrims;

// FP32 triangle records lie 48 bytes apart up to this many triangles and 64
// bytes apart, with the normal beside them, above.  Small scenes live in L2
// and gain from the smaller footprint (20,480-triangle icosphere, 170,918
// points x 256 paths: 51.1 ms against 53.0; its gradient walk 13.4 against
// 13.7); scenes beyond L2 pay per line they touch (200,992-triangle tori,
// 1M points x 512 paths: 326.0 ms against 313.7); at 61,000 both are equal.
constexpr int64_t kPackedPrims = 40000;

// Dynamic LDS that leaves 14 one-wavefront workgroups per CU (160 KB).
constexpr size_t kLargeSceneLds = 45 * 256;

// Round a double to binary16 toward -inf / +inf (|v| well inside the range).
_Float16 step_h(_Float16 h, bool up) {
  uint16_t u;
  std::memcpy(&u, &h, 2);
  if ((u & 0x7fff) == 0) u = up ? 0x0001 : 0x8001;  // +-0 -> the smallest subnormal
  else if ((u & 0x8000) != 0) u = up ? u - 1 : u + 1;
  else u = up ? u + 1 : u - 1;
  std::memcpy(&h, &u, 2);
  return h;
}
_Float16 down_h(double v) {
  _Float16 h = (_Float16)v;
  if ((double)h > v) h = step_h(h, false);
  return h;
}
_Float16 up_h(double v) {
  _Float16 h = (_Float16)v;
  if ((double)h < v) h = step_h(h, true);
  return h;
}

// Frame of the stored boxes: y' = (y - c) k with c the root box's centre
// (rounded to R, as the kernels use it) and k a power of two, |y'| <= 1.
template <typename R>
void box_frame(const wobhost::Box& root, int dim, double c[3], double& k) {
  double half = 0.0;
  for (int a = 0; a < 3; ++a) {
    c[a] = a < dim ? (double)(R)(0.5 * (root.lo[a] + root.hi[a])) : 0.0;
    if (a < dim) half = std::fmax(half, std::fmax(std::fabs(root.lo[a] - c[a]), std::fabs(root.hi[a] - c[a])));
  }
  k = half > 0.0 ? std::ldexp(1.0, -std::ilogb(half) - 1) : 1.0;
}

// A box in the frame, padded so that the FMA slab test in R precision never
// misses a primitive that the exact test would hit, stored rounded outward
// into slot `which` (FP32 scenes: binary16 pairs, lo in the low half of each
// word).
template <typename R, int D, typename Node>
void store_box(const wobhost::Box& b, const double c[3], double k, Node& n, int which) {
  double l[3], h[3], mag = 0.0;
  for (int a = 0; a < D; ++a) {
    l[a] = (b.lo[a] - c[a]) * k;
    h[a] = (b.hi[a] - c[a]) * k;
    mag = std::fmax(mag, std::fmax(std::fabs(l[a]), std::fabs(h[a])));
  }
  const double pad = (sizeof(R) == 4 ? 0x1p-19 : 0x1p-45) * (mag + 1.0);
  for (int a = 0; a < D; ++a) {
    if constexpr (sizeof(R) == 4) {
      const _Float16 lo = down_h(l[a] - pad), hi = up_h(h[a] + pad);
      uint16_t ul, uh;
      std::memcpy(&ul, &lo, 2);
      std::memcpy(&uh, &hi, 2);
      n.box[which][a] = (uint32_t)ul | ((uint32_t)uh << 16);
    } else {
      n.lo[which][a] = (R)(l[a] - pad);
      n.hi[which][a] = (R)(h[a] + pad);
    }
  }
}

// An unused slot: a box of NaN, which no line crosses (whatever the line, the
// slab parameters are NaN on every axis and the comparison fails); its entry,
// never taken, is a valid one (the first leaf).
template <typename R, typename Node>
void store_empty(Node& n, int which) {
  for (int a = 0; a < 3; ++a) {
    if constexpr (sizeof(R) == 4) n.box[which][a] = 0x7e007e00u;  // binary16 NaN, twice
    else n.lo[which][a] = n.hi[which][a] = (R)NAN;
  }
  n.child[which] = -1;
}

// Which entries a record holds: the choice that minimises the expected number
// of records a line fetches (a line meets a box with probability proportional
// to its measure).  cost(i, k) is that number below binary node i when i is
// given k entries of its parent's record: one entry is a record of its own
// (its measure, plus its children's cost with the record's kArity entries
// dealt between them), more are dealt between its two children.  Against
// opening the largest entry first: 3 % fewer fetches and, as the records are
// fuller, 15-27 % fewer bytes (3.45 entries a record on the 200,992-triangle
// tori, 3.09 before).
// In the builder's flat array the second child of a node is the first node
// after its first child's subtree.
class Collapse {
 public:
  Collapse(const std::vector<wobhost::FlatNode>& nodes, int dim) : fn_(nodes), plan_(nodes.size()) {
    std::vector<std::array<float, wob::kArity>> cost(nodes.size());  // [k - 1]
    const double root = std::fmax(wobhost::box_measure(nodes[0].box, dim), 1e-300);
    for (size_t i = nodes.size(); i-- > 0;) {
      auto& c = cost[i];
      auto& p = plan_[i];
      p.fill(0);
      if (nodes[i].child < 0) {
        c.fill(0.f);
        continue;
      }
      const auto& l = cost[first(i)];
      const auto& r = cost[second(i)];
      const auto deal = [&](int k, float best, uint8_t own) {
        for (int q = 1; q < k; ++q)
          if (l[q - 1] + r[k - q - 1] < best) {
            best = l[q - 1] + r[k - q - 1];
            own = (uint8_t)q;
          }
        return std::make_pair(best, own);
      };
      const auto record = deal(wob::kArity, std::numeric_limits<float>::infinity(), 1);
      p[0] = record.second;
      c[0] = (float)(wobhost::box_measure(nodes[i].box, dim) / root) + record.first;
      for (int k = 2; k <= wob::kArity; ++k) {
        const auto d = deal(k, c[k - 2], 0);  // 0: fewer entries do as well
        c[k - 1] = d.first;
        p[k - 1] = d.second;
      }
    }
  }
  // The entries (binary nodes) of the record of interior node i, at most
  // max_ent (kArity, or 2: its children).
  int entries(size_t i, int max_ent, size_t* out) const {
    if (max_ent < wob::kArity) {
      out[0] = first(i);
      out[1] = second(i);
      return 2;
    }
    const int n = open(first(i), plan_[i][0], out);
    return n + open(second(i), wob::kArity - plan_[i][0], out + n);
  }

 private:
  size_t first(size_t i) const { return (size_t)fn_[i].child; }
  size_t second(size_t i) const { return (size_t)fn_[first(i)].skip; }
  int open(size_t i, int k, size_t* out) const {
    while (k > 1 && plan_[i][k - 1] == 0) --k;
    if (k == 1 || fn_[i].child < 0) {
      *out = i;
      return 1;
    }
    const int q = plan_[i][k - 1], n = open(first(i), q, out);
    return n + open(second(i), k - q, out + n);
  }
  const std::vector<wobhost::FlatNode>& fn_;
  // [0]: entries of the node's own record given to its first child; [k - 1]:
  // of k entries given to the node, those given to its first child
  std::vector<std::array<uint8_t, wob::kArity>> plan_;
};

template <typename R, int D>
wob_status upload_scene(wob_scene_s* sc, const std::vector<double>& v, const int32_t* prims,
                        const uint8_t* kind, const double* alpha, const wobhost::Bvh& bvh,
                        hipStream_t st) {
  using Node = typename wob::Rec<R, D>::Node;
  using Prim = typename wob::Rec<R, D>::Prim;
  const int64_t T = sc->n_prims;
  // 4-wide interior records, in pre-order (a record's first interior child is
  // the next record), each holding the entries that `collapse` chose below its
  // binary node; every interior entry becomes a record of its own.
  const auto& fn = bvh.nodes;
  double fc[3], fk;
  box_frame<R>(fn[0].box, D, fc, fk);
  std::vector<Node> nodes;
  nodes.reserve(fn.size() / 3 + 1);
  int max_ent = wob::kArity;
  const Collapse collapse(fn, D);
  // need: the deepest stack that the subtree can take below what waits there
  const std::function<int32_t(size_t, int32_t*)> emit = [&](size_t i, int32_t* need) -> int32_t {
    size_t ent[wob::kArity];
    const int n_ent = collapse.entries(i, max_ent, ent);
    const int32_t r = (int32_t)nodes.size();
    nodes.emplace_back();
    int32_t child[wob::kArity], sub[wob::kArity];
    for (int q = 0; q < n_ent; ++q) {
      const auto& e = fn[ent[q]];
      sub[q] = -1;
      child[q] = e.child >= 0 ? emit(ent[q], &sub[q]) : e.child;  // a leaf's code
    }
    // a line takes the crossed records of slot 0 first, then those of the
    // last slot down to slot 1, and the k-th one from the last waits under k
    // others: the record that needs the deepest stack is taken last (the
    // 200,992-triangle tori need 17 entries, 28 with the records as they come)
    int slot[wob::kArity];
    for (int q = 0; q < n_ent; ++q) slot[q] = q;
    std::stable_sort(slot, slot + n_ent, [&](int x, int y) { return sub[x] < sub[y]; });
    *need = 0;
    Node n;
    std::memset(&n, 0, sizeof(Node));
    for (int q = 0; q < wob::kArity; ++q) {
      const int at = (wob::kArity - q) % wob::kArity;  // the order in which slots are taken: 0, 3, 2, 1
      if (q < n_ent) {
        store_box<R, D>(fn[ent[slot[q]]].box, fc, fk, n, at);
        n.child[at] = child[slot[q]];
        if (sub[slot[q]] >= 0) *need = std::max(*need, n_ent - 1 - q + sub[slot[q]]);
      } else {
        store_empty<R>(n, at);
      }
    }
    nodes[r] = n;
    return r;
  };
  int32_t need = 0;
  int32_t root = fn[0].child >= 0 ? emit(0, &need) : fn[0].child;
  if (need > wob::kMaxDepth) {
    // a degenerate tree whose 4-wide records could push more than a lane's
    // stack holds: two entries per record (the binary tree, whose stack needs
    // at most one entry per doubling of its leaves)
    nodes.clear();
    max_ent = 2;
    need = 0;
    root = emit(0, &need);
  }
  const int32_t n_inner = (int32_t)nodes.size();
  // every interior entry points to a later record (pre-order), so a traversal
  // never returns to a record it left: the walk ends on every line
  for (int32_t r = 0; r < n_inner; ++r)
    for (int q = 0; q < wob::kArity; ++q) {
      const int32_t c = nodes[r].child[q];
      if (c >= 0 && (c <= r || c >= n_inner)) return WOB_E_MESH;
    }
  // the traversal addresses records by a 32-bit byte offset
  if ((uint64_t)n_inner * sizeof(Node) > 0xffffffffull) return WOB_E_ARG;
  sc->n_inner = n_inner;
  for (int a = 0; a < 3; ++a) sc->frame_c[a] = fc[a];
  sc->frame_k = fk;
  sc->root = root;
  sc->stack_cap = std::max(need, 1);
  if (sc->stack_cap > wob::kMaxDepth) return WOB_E_MESH;
  // the primitive records and, in their last bytes or in an array of their
  // own, the unit normals
  const bool wide = D == 3 && sizeof(R) == 4 && T > kPackedPrims;
  const size_t stride = wide ? 64 : sizeof(Prim);
  std::vector<unsigned char> recs((size_t)T * stride, 0);
  constexpr size_t nv = wob::kNormalValues<R, D>;
  std::vector<R> normals(wide ? 0 : (size_t)T * nv, (R)0);
  std::vector<int32_t> leaf_of_id((size_t)T);
  std::vector<double> area((size_t)T, 0.0);
  for (int64_t j = 0; j < T; ++j) {
    const int32_t id = bvh.order[j];
    leaf_of_id[id] = (int32_t)j;
    // written whole into the byte array, which need not be aligned for them
    Prim p;
    std::memset(&p, 0, sizeof(Prim));
    R nrm[4] = {0, 0, 0, 0};
    const int32_t* ix = prims + (int64_t)id * D;
    const int k = kind ? kind[id] : 0;
    p.idkind = id | (k << wob::kIdBits);
    p.alpha = alpha ? (R)alpha[id] : (R)0;
    double e1d[3] = {0, 0, 0}, e2d[3] = {0, 0, 0};
    if constexpr (D == 3) {
      for (int a = 0; a < 3; ++a) {
        const double v0 = v[(int64_t)ix[0] * 3 + a], v1 = v[(int64_t)ix[1] * 3 + a],
                     v2 = v[(int64_t)ix[2] * 3 + a];
        p.v0[a] = (R)v0;
        e1d[a] = v1 - v0;
        e2d[a] = v2 - v0;
        p.e1[a] = (R)e1d[a];
        p.e2[a] = (R)e2d[a];
      }
      double n[3] = {e1d[1] * e2d[2] - e1d[2] * e2d[1], e1d[2] * e2d[0] - e1d[0] * e2d[2],
                     e1d[0] * e2d[1] - e1d[1] * e2d[0]};
      const double l = std::sqrt(n[0] * n[0] + n[1] * n[1] + n[2] * n[2]);
      for (int a = 0; a < 3; ++a) nrm[a] = (R)(n[a] / l);
      area[id] = 0.5 * l;
    } else {
      for (int a = 0; a < 2; ++a) {
        const double v0 = v[(int64_t)ix[0] * 2 + a], v1 = v[(int64_t)ix[1] * 2 + a];
        p.v0[a] = (R)v0;
        e1d[a] = v1 - v0;
        p.e[a] = (R)e1d[a];
      }
      const double l = std::sqrt(e1d[0] * e1d[0] + e1d[1] * e1d[1]);
      nrm[0] = (R)(e1d[1] / l);
      nrm[1] = (R)(-e1d[0] / l);
      area[id] = l;
    }
    unsigned char* const rec = recs.data() + (size_t)j * stride;
    std::memcpy(rec, &p, sizeof(Prim));
    if (wide) std::memcpy(rec + sizeof(Prim), nrm, sizeof(nrm));
    else std::memcpy(&normals[nv * (size_t)j], nrm, nv * sizeof(R));
  }
  sc->node_bytes = sizeof(Node);
  sc->prim_bytes = (int64_t)stride;
  sc->normal_offset = sizeof(Prim);
  // cumulative area fraction in caller-id order: summed in binary64, rounded
  // once to binary32 (an area-uniform pick compares a binary32 uniform with it)
  std::vector<float> cdf((size_t)T);
  double tot = 0.0;
  for (int64_t j = 0; j < T; ++j) tot += area[j];
  double run = 0.0;
  for (int64_t j = 0; j < T; ++j) {
    run += area[j];
    cdf[j] = (float)(run / tot);
  }
  cdf[T - 1] = 1.0f;
  sc->area_total = tot;
  // a guide to the area CDF: with K = 2^shift >= T buckets (at most 2^24),
  // guide[b] is the first index whose cdf exceeds b / K, so the first index
  // whose cdf exceeds a binary32 uniform u lies in [guide[b], guide[b + 1]]
  // for b = floor(u K) (exact: K is a power of two); the area-uniform pick
  // searches there and finds the same index as a search of the whole CDF
  int shift = 0;
  while ((int64_t)1 << shift < T && shift < 24) ++shift;
  const int64_t K = (int64_t)1 << shift;
  std::vector<wob::GuideEntry> guide((size_t)K + 1);
  {
    int64_t i = 0;
    for (int64_t b = 0; b <= K; ++b) {
      const double t = (double)b / (double)K;
      while (i < T - 1 && !((double)cdf[i] > t)) ++i;
      guide[b] = wob::GuideEntry{(int32_t)i, cdf[i]};
    }
  }
  sc->guide_shift = shift;
  // the vertices (already rounded to R) and each primitive's vertex ids, for
  // per-vertex boundary data
  std::vector<R> verts_r(v.size());
  for (size_t i = 0; i < v.size(); ++i) verts_r[i] = (R)v[i];
  const size_t nb = std::max(nodes.size(), (size_t)1) * sizeof(Node), pb = recs.size(),
               lb = leaf_of_id.size() * sizeof(int32_t), qb = normals.size() * sizeof(R),
               cb = sizeof(float) * T, vb = verts_r.size() * sizeof(R),
               ib = (size_t)T * D * sizeof(int32_t), sb = sizeof(unsigned long long),
               gb = guide.size() * sizeof(wob::GuideEntry), db = (size_t)T * sizeof(wob::Candidate<R>);
  if (hipMalloc(&sc->d_nodes, nb) != hipSuccess) return WOB_E_ALLOC;
  if (hipMalloc(&sc->d_prims, pb) != hipSuccess) return WOB_E_ALLOC;
  if (qb > 0 && hipMalloc(&sc->d_normals, qb) != hipSuccess) return WOB_E_ALLOC;
  if (hipMalloc((void**)&sc->d_leaf_of_id, lb) != hipSuccess) return WOB_E_ALLOC;
  if (hipMalloc((void**)&sc->d_area_cdf, cb) != hipSuccess) return WOB_E_ALLOC;
  if (hipMalloc((void**)&sc->d_area_guide, gb) != hipSuccess) return WOB_E_ALLOC;
  if (hipMalloc(&sc->d_verts, vb) != hipSuccess) return WOB_E_ALLOC;
  if (hipMalloc((void**)&sc->d_vid, ib) != hipSuccess) return WOB_E_ALLOC;
  if (hipMalloc((void**)&sc->d_status, sb) != hipSuccess) return WOB_E_ALLOC;
  // The RIS candidates are half as much again as the rest of a scene (FP32 triangles:
  // 64 bytes each to 116) and serve speed alone: RIS on 60,976 triangles takes 4.3 ms
  // with them, 6.0 from the records by their leaf-order indices (a kernel that can do
  // either takes 3 % longer with them).  A scene that fits the device without them
  // has them in host memory.
  if (hipMalloc(&sc->d_candidates, db) != hipSuccess) {
    (void)hipGetLastError();  // taken note of here, not by the next call's check
    sc->d_candidates = nullptr;
    if (hipHostMalloc(&sc->d_candidates, db, hipHostMallocDefault) != hipSuccess) return WOB_E_ALLOC;
    sc->candidates_on_host = true;
  }
  // copies on the caller's stream, waited for before the host arrays go
  const auto put = [st](void* dst, const void* src, size_t bytes) {
    return hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, st) == hipSuccess;
  };
  bool ok = (qb == 0 || put(sc->d_normals, normals.data(), qb)) && put(sc->d_prims, recs.data(), pb) &&
            put(sc->d_leaf_of_id, leaf_of_id.data(), lb) && put(sc->d_area_cdf, cdf.data(), cb) &&
            put(sc->d_area_guide, guide.data(), gb) &&
            put(sc->d_verts, verts_r.data(), vb) && put(sc->d_vid, prims, ib) &&
            hipMemsetAsync(sc->d_status, 0, sb, st) == hipSuccess;
  if (ok && !nodes.empty()) ok = put(sc->d_nodes, nodes.data(), nodes.size() * sizeof(Node));
  if (ok) {
    hipLaunchKernelGGL((wob::candidate_kernel<R, D>), dim3((unsigned)((T + 255) / 256)), dim3(256), 0, st,
                       view<R, D>(sc), (wob::Candidate<R>*)sc->d_candidates);
    ok = hipGetLastError() == hipSuccess;
  }
  // the copies must end before the host arrays are released, also on failure
  if (hipStreamSynchronize(st) != hipSuccess || !ok) return WOB_E_DEVICE;
  sc->n_verts = (int64_t)(v.size() / D);
  sc->device_bytes = (int64_t)(nb + pb + lb + qb + cb + vb + ib + sb + gb + (sc->candidates_on_host ? 0 : db));
  return WOB_OK;
}

enum Mode { MODE_SOLVE = 0, MODE_TRACE = 1, MODE_COUNT = 2 };

// A plain solve with 2^lpp_shift lanes per point in workgroups of B lanes.
template <typename R, int D, int FORM, int VX, int B>
void launch_spread(const wob::WalkArgs<R, D>& a, hipStream_t st) {
  const int ppb = B >> a.lpp_shift;
  hipLaunchKernelGGL((wob::walk_kernel<R, D, FORM, false, false, B, wob::X_SPREAD | VX>),
                     dim3((unsigned)((a.n_points + ppb - 1) / ppb)), dim3(B),
                     wob::walk_lds_bytes(a.scene.stack_cap, B), st, a);
}

// VX: X_VDATA for per-vertex data (its own instantiation of each kernel)
template <typename R, int D, int FORM, int VX>
void launch_form(const wob::WalkArgs<R, D>& a0, int mode, int32_t n_cu, hipStream_t st) {
  constexpr int B = kSolveBlock;
  // plain single-layer solves pool two points per lane group: at most 32
  // lanes per point (the kernel instantiation decides, by the same rule)
  const bool plain = mode == MODE_SOLVE && !(a0.grad_out || a0.path_grad_out) && !a0.cv_g;
  const bool pooled = plain && wob::pools_points(FORM, VX, false, false);
  wob::WalkArgs<R, D> a = a0;
  if (plain) {
    const LaneSplit split = split_lanes<R, D>(FORM, pooled, a.scene.stack_cap, a.n_points, a.N, n_cu);
    a.lpp_shift = split.shift;
    if (split.spread) {
      if (split.shift <= 6) launch_spread<R, D, FORM, VX, 64>(a, st);
      else if (split.shift <= 8) launch_spread<R, D, FORM, VX, 256>(a, st);
      else launch_spread<R, D, FORM, VX, kWideBlock<R>>(a, st);
      return;
    }
  } else {
    a.lpp_shift = spread_shift<R, D>(FORM, lpp_shift_for(a.N, B), 6, a.n_points, a.N, n_cu);
  }
  const int ppb = B >> a.lpp_shift;
  const dim3 grid((unsigned)((a.n_points + ppb - 1) / ppb)), block(B);
  size_t lds = wob::walk_lds_bytes(a.scene.stack_cap, B);  // traversal stacks, held leaves
  // the FP32 double layer on a scene of triangles well beyond an XCD's 4 MB of L2: 14
  // wavefronts per CU instead of 17 fetch less over each other, but end later, which
  // costs more with few paths per lane (100,000 points, 17 against 14 wavefronts, ms:
  // 200,000 triangles x 128 / 256 / 512 paths 20.6 / 42.1 / 86.5 against 21.6 / 40.3 /
  // 77.7; 144,500 18.5 / 37.2 / 75.7 against 20.1 / 37.8 / 72.7; 120,000 segments
  // x 256 58.0 against 64.4; FP64, of fewer wavefronts anyway, the same; the other
  // forms, which run four wavefronts per SIMD or fewer, lose everywhere)
  if (D == 3 && sizeof(R) == 4 && FORM == wob::F_DL && mode == MODE_SOLVE && !a0.grad_out &&
      (int64_t)a.N >= (int64_t)(a0.scene.n_prims > kPackedPrims * 4 ? 4 : 8) << a.lpp_shift &&
      a0.scene.n_prims > kPackedPrims * 3)
    lds = std::max(lds, (size_t)kLargeSceneLds);
  if constexpr (FORM != wob::F_FWD) {
    if (a.grad_out || a.path_grad_out) {  // value and gradient along the same paths
      if (mode == MODE_TRACE)
        hipLaunchKernelGGL((wob::walk_kernel<R, D, FORM, true, false, B, wob::X_GRAD | VX>), grid, block, lds, st,
                           a);
      else
        hipLaunchKernelGGL((wob::walk_kernel<R, D, FORM, false, false, B, wob::X_GRAD | VX>), grid, block, lds,
                           st, a);
      return;
    }
  }
  if constexpr (D == 3 && (FORM == wob::F_SL || FORM == wob::F_SL_RIS)) {
    if (a.cv_g) {
      if (mode == MODE_SOLVE)
        hipLaunchKernelGGL((wob::walk_kernel<R, D, FORM, false, false, B, wob::X_CV | VX>), grid, block, lds, st,
                           a);
      else if (mode == MODE_TRACE)
        hipLaunchKernelGGL((wob::walk_kernel<R, D, FORM, true, false, B, wob::X_CV | VX>), grid, block, lds, st, a);
      else
        hipLaunchKernelGGL((wob::walk_kernel<R, D, FORM, false, true, B, wob::X_CV | VX>), grid, block, lds, st, a);
      return;
    }
  }
  if (mode == MODE_SOLVE)
    hipLaunchKernelGGL((wob::walk_kernel<R, D, FORM, false, false, B, VX>), grid, block, lds, st, a);
  else if (mode == MODE_TRACE)
    hipLaunchKernelGGL((wob::walk_kernel<R, D, FORM, true, false, B, VX>), grid, block, lds, st, a);
  else
    hipLaunchKernelGGL((wob::walk_kernel<R, D, FORM, false, true, B, VX>), grid, block, lds, st, a);
}

template <typename R, int D, int VX>
void launch_walk_vx(const wob::WalkArgs<R, D>& a, int mode, int32_t n_cu, hipStream_t st) {
  if (a.form == wob::F_DL) launch_form<R, D, wob::F_DL, VX>(a, mode, n_cu, st);
  else if (a.form == wob::F_DIRECT) launch_form<R, D, wob::F_DIRECT, VX>(a, mode, n_cu, st);
  else if (a.form == wob::F_SL_RIS) launch_form<R, D, wob::F_SL_RIS, VX>(a, mode, n_cu, st);
  else launch_form<R, D, wob::F_SL, VX>(a, mode, n_cu, st);
}

template <typename R, int D>
void launch_walk(const wob::WalkArgs<R, D>& a, int mode, int32_t n_cu, hipStream_t st) {
  if (a.prog.type == wob::P_VERTEX) launch_walk_vx<R, D, wob::X_VDATA>(a, mode, n_cu, st);
  else launch_walk_vx<R, D, wob::X_NONE>(a, mode, n_cu, st);
}

template <int SUB, int PPT>
void launch_addback_as(const wob_scene_s* sc, const float* g, const float* points, int64_t n_points, uint64_t seed,
                       float* out, int accumulate, hipStream_t st) {
  constexpr int64_t per_block = wob::kAddWaves * (64 / SUB) * PPT;
  constexpr int64_t per_launch = (int64_t)1 << 26;  // within the 2^32 lanes of a launch
  for (int64_t p = 0; p < n_points; p += per_launch) {
    const int64_t n = n_points - p < per_launch ? n_points - p : per_launch;
    hipLaunchKernelGGL((wob::cv_addback_kernel<float, SUB, PPT>), dim3((unsigned)((n + per_block - 1) / per_block)),
                       dim3(64 * wob::kAddWaves), 0, st, view<float, 3>(sc), g, points + p * 3, n,
                       (uint32_t)(seed & 0xffffffffu), out + p, accumulate);
  }
}

void launch_addback(const wob_scene_s* sc, const float* g, const void* points, int64_t n_points, uint64_t seed,
                    void* out, int accumulate, hipStream_t st) {
  // Eight points per lane halve the LDS reads of a pair, four make twice the
  // wavefronts; fewer lanes per point mean fewer workgroups, each of which takes
  // every triangle to LDS and looks for the table's zeros.  62,720 triangles (us):
  //   points       4 / 64 lanes   8 / 32 lanes   8 / 16   8 / 8
  //      20,000         667            769
  //      60,000       1,624          1,160        1,327
  //     200,000       4,777          3,745        3,978    3,893
  //     256,000                      4,260        3,937    3,908
  //     300,000                      5,268        4,879    5,856
  // 5,120 triangles, 1,000,000 points: 2,003, 1,434, 1,325, 1,286; 20 triangles:
  // 461, 304, 255, 234; all values zero 201, 88, 45, 23.
  if (n_points < (int64_t)sc->n_cu * 128)
    launch_addback_as<64, 4>(sc, g, (const float*)points, n_points, seed, (float*)out, accumulate, st);
  else if (n_points < (int64_t)sc->n_cu * 1000)
    launch_addback_as<32, 8>(sc, g, (const float*)points, n_points, seed, (float*)out, accumulate, st);
  else if (n_points < (int64_t)sc->n_cu * 2500)
    launch_addback_as<16, 8>(sc, g, (const float*)points, n_points, seed, (float*)out, accumulate, st);
  else
    launch_addback_as<8, 8>(sc, g, (const float*)points, n_points, seed, (float*)out, accumulate, st);
}

wob_status run_walk(wob_scene sc, const void* points, const int32_t* point_prim, int64_t n_points,
                    const wob_bc* bc, int32_t samples, int32_t walk_len, uint64_t seed,
                    const uint32_t* point_ids, void* mean_out, void* var_out, void* path_out,
                    int32_t* vtx_prim, int32_t* vtx_m, uint64_t* counters, int mode,
                    void* stream, const float* cv_g = nullptr, const float* cv_g0 = nullptr,
                    void* grad_out = nullptr, void* grad_var_out = nullptr, void* path_grad_out = nullptr,
                    const void* anchor_pts = nullptr, const int32_t* anchor_prim = nullptr) {
  Plan pl;
  wob_status s = plan_walk(sc, bc, samples, walk_len, &pl);
  if (s != WOB_OK) return s;
  if (cv_g && (sc->dim != 3 || sc->precision != WOB_F32 || pl.form != WOB_F_SINGLE_LAYER ||
               bc->density || sc->n_dirichlet > 0))
    return WOB_E_UNSUPPORTED;
  const bool grad = grad_out || path_grad_out;
  // gradients: evaluation points inside the domain, no density mode, no control variate
  if (grad && (point_prim || bc->density || cv_g)) return WOB_E_UNSUPPORTED;
  // the boundary split: both arrays or neither, gradients of the double layer only
  if ((anchor_pts != nullptr) != (anchor_prim != nullptr)) return WOB_E_ARG;
  if (anchor_prim && (!grad || pl.form != WOB_F_DOUBLE_LAYER)) return WOB_E_UNSUPPORTED;
  if (grad && mode == MODE_SOLVE && n_points > 0 && !grad_out) return WOB_E_ARG;
  if (mode == MODE_SOLVE && grad_var_out && samples < 2) return WOB_E_ARG;
  if (n_points < 0 || (n_points > 0 && !points)) return WOB_E_ARG;
  if (n_points >= (int64_t)1 << 32) return WOB_E_ARG;  // point index is a 32-bit counter word
  if (mode == MODE_SOLVE && n_points > 0 && !mean_out) return WOB_E_ARG;
  if (mode == MODE_SOLVE && var_out && samples < 2) return WOB_E_ARG;
  if (mode == MODE_TRACE && n_points > 0 && !path_out) return WOB_E_ARG;
  if (mode == MODE_COUNT && !counters) return WOB_E_ARG;
  if (n_points == 0) return WOB_OK;
  hipStream_t st = (hipStream_t)stream;
  if (sc->precision == WOB_F32) {
    if (sc->dim == 3) {
      auto a = make_args<float, 3>(sc, pl, points, point_prim, n_points, bc, samples, walk_len, seed);
      a.mean_out = (float*)mean_out; a.var_out = (float*)var_out; a.path_out = (float*)path_out;
      a.grad_out = (float*)grad_out; a.grad_var_out = (float*)grad_var_out; a.path_grad_out = (float*)path_grad_out;
      a.vtx_prim = vtx_prim; a.vtx_m = vtx_m; a.counters = (unsigned long long*)counters;
      a.point_ids = point_ids;
      a.cv_g = cv_g;
      a.cv_g0 = cv_g0 ? cv_g0 : cv_g;
      a.anchor_pts = (const float*)anchor_pts;
      a.anchor_prim = anchor_prim;
      launch_walk<float, 3>(a, mode, sc->n_cu, st);
    } else {
      auto a = make_args<float, 2>(sc, pl, points, point_prim, n_points, bc, samples, walk_len, seed);
      a.mean_out = (float*)mean_out; a.var_out = (float*)var_out; a.path_out = (float*)path_out;
      a.grad_out = (float*)grad_out; a.grad_var_out = (float*)grad_var_out; a.path_grad_out = (float*)path_grad_out;
      a.vtx_prim = vtx_prim; a.vtx_m = vtx_m; a.counters = (unsigned long long*)counters;
      a.point_ids = point_ids;
      a.anchor_pts = (const float*)anchor_pts;
      a.anchor_prim = anchor_prim;
      launch_walk<float, 2>(a, mode, sc->n_cu, st);
    }
  } else {
    if (sc->dim == 3) {
      auto a = make_args<double, 3>(sc, pl, points, point_prim, n_points, bc, samples, walk_len, seed);
      a.mean_out = (double*)mean_out; a.var_out = (double*)var_out; a.path_out = (double*)path_out;
      a.grad_out = (double*)grad_out; a.grad_var_out = (double*)grad_var_out; a.path_grad_out = (double*)path_grad_out;
      a.vtx_prim = vtx_prim; a.vtx_m = vtx_m; a.counters = (unsigned long long*)counters;
      a.point_ids = point_ids;
      a.anchor_pts = (const double*)anchor_pts;
      a.anchor_prim = anchor_prim;
      launch_walk<double, 3>(a, mode, sc->n_cu, st);
    } else {
      auto a = make_args<double, 2>(sc, pl, points, point_prim, n_points, bc, samples, walk_len, seed);
      a.mean_out = (double*)mean_out; a.var_out = (double*)var_out; a.path_out = (double*)path_out;
      a.grad_out = (double*)grad_out; a.grad_var_out = (double*)grad_var_out; a.path_grad_out = (double*)path_grad_out;
      a.vtx_prim = vtx_prim; a.vtx_m = vtx_m; a.counters = (unsigned long long*)counters;
      a.point_ids = point_ids;
      a.anchor_pts = (const double*)anchor_pts;
      a.anchor_prim = anchor_prim;
      launch_walk<double, 2>(a, mode, sc->n_cu, st);
    }
  }
  return hipGetLastError() == hipSuccess ? WOB_OK : WOB_E_DEVICE;
}

}  // namespace

extern "C" {

const char* wob_status_string(wob_status s) {
  switch (s) {
    case WOB_OK: return "ok";
    case WOB_E_ARG: return "invalid argument";
    case WOB_E_ALLOC: return "allocation failed";
    case WOB_E_DEVICE: return "HIP runtime error";
    case WOB_E_MESH: return "invalid mesh";
    case WOB_E_UNSUPPORTED: return "unsupported combination";
    case WOB_E_TOO_LARGE: return "beyond the capacity of an allocation-free entry point";
  }
  return "unknown status";
}

}  // extern "C"

namespace {

// wob_build_bvh on host arrays, the scene's copies on `st`.
wob_status build_scene(int32_t dim, int32_t precision, const double* verts, int64_t n_verts,
                       const int32_t* prims, int64_t n_prims, const uint8_t* kind, const double* alpha,
                       hipStream_t st, wob_scene* out) {
  // vertices rounded to the scene precision: the walk and the oracle then see the
  // same geometry
  std::vector<double> v((size_t)(n_verts * dim));
  for (int64_t i = 0; i < n_verts * dim; ++i) {
    const double x = verts[i];
    if (!std::isfinite(x)) return WOB_E_MESH;
    v[i] = precision == WOB_F32 ? (double)(float)x : x;
    if (!std::isfinite(v[i])) return WOB_E_MESH;
  }
  std::vector<wobhost::Box> boxes((size_t)n_prims);
  int32_t nd = 0, nn = 0, nr = 0;
  for (int64_t j = 0; j < n_prims; ++j) {
    wobhost::Box b;
    for (int a = 0; a < 3; ++a) {
      b.lo[a] = INFINITY;
      b.hi[a] = -INFINITY;
    }
    double p[3][3] = {{0}};
    for (int c = 0; c < dim; ++c) {
      const int32_t ix = prims[j * dim + c];
      if (ix < 0 || ix >= n_verts) return WOB_E_MESH;
      for (int a = 0; a < dim; ++a) {
        p[c][a] = v[(int64_t)ix * dim + a];
        b.lo[a] = std::fmin(b.lo[a], p[c][a]);
        b.hi[a] = std::fmax(b.hi[a], p[c][a]);
      }
    }
    for (int a = dim; a < 3; ++a) b.lo[a] = b.hi[a] = 0.0;
    // zero-length segment / zero-area triangle
    if (dim == 2) {
      if (p[0][0] == p[1][0] && p[0][1] == p[1][1]) return WOB_E_MESH;
    } else {
      const double e1[3] = {p[1][0] - p[0][0], p[1][1] - p[0][1], p[1][2] - p[0][2]};
      const double e2[3] = {p[2][0] - p[0][0], p[2][1] - p[0][1], p[2][2] - p[0][2]};
      const double c0 = e1[1] * e2[2] - e1[2] * e2[1], c1 = e1[2] * e2[0] - e1[0] * e2[2],
                   c2 = e1[0] * e2[1] - e1[1] * e2[0];
      if (c0 == 0.0 && c1 == 0.0 && c2 == 0.0) return WOB_E_MESH;
    }
    boxes[j] = b;
    const int k = kind ? kind[j] : WOB_BC_DIRICHLET;
    if (k == WOB_BC_DIRICHLET) ++nd;
    else if (k == WOB_BC_NEUMANN) ++nn;
    else if (k == WOB_BC_ROBIN) ++nr;
    else return WOB_E_ARG;
    if (alpha && !std::isfinite(alpha[j])) return WOB_E_ARG;
  }
  int dev = 0, n_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n_cu <= 0)
    return WOB_E_DEVICE;
  wobhost::Bvh bvh = wobhost::build_bvh(dim, boxes, kMaxLeaf);
  wob_scene_s* sc = new (std::nothrow) wob_scene_s();
  if (!sc) return WOB_E_ALLOC;
  sc->dim = dim;
  sc->precision = precision;
  sc->device = dev;
  sc->n_cu = n_cu;
  sc->n_prims = n_prims;
  sc->n_nodes = (int64_t)bvh.nodes.size();
  sc->n_leaves = bvh.n_leaves;
  sc->depth = bvh.depth;
  sc->max_leaf = bvh.max_leaf;
  sc->n_dirichlet = nd;
  sc->n_neumann = nn;
  sc->n_robin = nr;
  wob_status s;
  if (precision == WOB_F32)
    s = dim == 3 ? upload_scene<float, 3>(sc, v, prims, kind, alpha, bvh, st)
                 : upload_scene<float, 2>(sc, v, prims, kind, alpha, bvh, st);
  else
    s = dim == 3 ? upload_scene<double, 3>(sc, v, prims, kind, alpha, bvh, st)
                 : upload_scene<double, 2>(sc, v, prims, kind, alpha, bvh, st);
  if (s != WOB_OK) {
    wob_free(sc);
    return s;
  }
  *out = sc;
  return WOB_OK;
}

wob_status check_build_args(int32_t dim, int32_t precision, const double* verts, int64_t n_verts,
                            const int32_t* prims, int64_t n_prims, wob_scene* out) {
  if (!out) return WOB_E_ARG;
  *out = nullptr;
  if (dim != 2 && dim != 3) return WOB_E_ARG;
  if (precision != WOB_F32 && precision != WOB_F64) return WOB_E_ARG;
  if (!verts || !prims || n_verts <= 0 || n_prims <= 0) return WOB_E_ARG;
  if (n_prims >= ((int64_t)1 << 27)) return WOB_E_ARG;  // leaf entries pack the first index in 27 bits
  if (n_verts > ((int64_t)1 << 31) - 1) return WOB_E_ARG;  // vertex ids are int32
  return WOB_OK;
}

}  // namespace

extern "C" {

wob_status wob_build_bvh(int32_t dim, int32_t precision, const double* verts, int64_t n_verts,
                         const int32_t* prims, int64_t n_prims, const uint8_t* kind,
                         const double* alpha, wob_scene* out) {
  const wob_status a = check_build_args(dim, precision, verts, n_verts, prims, n_prims, out);
  if (a != WOB_OK) return a;
  return build_scene(dim, precision, verts, n_verts, prims, n_prims, kind, alpha, nullptr, out);
}

wob_status wob_build_bvh_ex(int32_t dim, int32_t precision, const double* verts, int64_t n_verts,
                            const int32_t* prims, int64_t n_prims, const uint8_t* kind,
                            const double* alpha, int32_t inputs_on_device, void* stream,
                            wob_scene* out) {
  const wob_status a = check_build_args(dim, precision, verts, n_verts, prims, n_prims, out);
  if (a != WOB_OK) return a;
  if (inputs_on_device != 0 && inputs_on_device != 1) return WOB_E_ARG;
  hipStream_t st = (hipStream_t)stream;
  if (!inputs_on_device)
    return build_scene(dim, precision, verts, n_verts, prims, n_prims, kind, alpha, st, out);
  // the tree is built on the host: bring the mesh over on the caller's stream
  std::vector<double> hv((size_t)(n_verts * dim)), ha(alpha ? (size_t)n_prims : 0);
  std::vector<int32_t> hp((size_t)(n_prims * dim));
  std::vector<uint8_t> hk(kind ? (size_t)n_prims : 0);
  const auto get = [st](void* dst, const void* src, size_t bytes) {
    return hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, st) == hipSuccess;
  };
  bool ok = get(hv.data(), verts, hv.size() * sizeof(double)) &&
            get(hp.data(), prims, hp.size() * sizeof(int32_t));
  if (ok && kind) ok = get(hk.data(), kind, hk.size());
  if (ok && alpha) ok = get(ha.data(), alpha, ha.size() * sizeof(double));
  // wait also after a failed enqueue: the host arrays are released on return
  if (hipStreamSynchronize(st) != hipSuccess || !ok) return WOB_E_DEVICE;
  return build_scene(dim, precision, hv.data(), n_verts, hp.data(), n_prims, kind ? hk.data() : nullptr,
                     alpha ? ha.data() : nullptr, st, out);
}

void wob_free(wob_scene sc) {
  if (!sc) return;
  if (sc->d_nodes) (void)hipFree(sc->d_nodes);
  if (sc->d_prims) (void)hipFree(sc->d_prims);
  if (sc->d_normals) (void)hipFree(sc->d_normals);
  if (sc->d_area_cdf) (void)hipFree(sc->d_area_cdf);
  if (sc->d_area_guide) (void)hipFree(sc->d_area_guide);
  if (sc->d_candidates) (void)(sc->candidates_on_host ? hipHostFree(sc->d_candidates) : hipFree(sc->d_candidates));
  if (sc->d_leaf_of_id) (void)hipFree(sc->d_leaf_of_id);
  if (sc->d_status) (void)hipFree(sc->d_status);
  if (sc->d_verts) (void)hipFree(sc->d_verts);
  if (sc->d_vid) (void)hipFree(sc->d_vid);
  delete sc;
}

wob_status wob_last_device_status(wob_scene sc, uint64_t* nonfinite_paths, void* stream) {
  if (!sc || !nonfinite_paths) return WOB_E_ARG;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev != sc->device) return WOB_E_DEVICE;
  hipStream_t st = (hipStream_t)stream;
  unsigned long long v = 0;
  if (hipMemcpyAsync(&v, sc->d_status, sizeof(v), hipMemcpyDeviceToHost, st) != hipSuccess)
    return WOB_E_DEVICE;
  if (hipMemsetAsync(sc->d_status, 0, sizeof(v), st) != hipSuccess) return WOB_E_DEVICE;
  if (hipStreamSynchronize(st) != hipSuccess) return WOB_E_DEVICE;
  *nonfinite_paths = (uint64_t)v;
  return WOB_OK;
}

wob_status wob_get_scene_info(wob_scene sc, wob_scene_info* info) {
  if (!sc || !info) return WOB_E_ARG;
  std::memset(info, 0, sizeof(*info));
  info->dim = sc->dim;
  info->precision = sc->precision;
  info->n_prims = sc->n_prims;
  info->n_nodes = sc->n_nodes;
  info->n_leaves = sc->n_leaves;
  info->depth = sc->depth;
  info->max_leaf = sc->max_leaf;
  info->device_bytes = sc->device_bytes;
  info->node_bytes = sc->node_bytes;
  info->prim_bytes = sc->prim_bytes;
  info->n_dirichlet = sc->n_dirichlet;
  info->n_neumann = sc->n_neumann;
  info->n_robin = sc->n_robin;
  info->n_verts = sc->n_verts;
  return WOB_OK;
}

int32_t wob_lines_per_path(wob_scene sc, const wob_bc* bc, int32_t walk_len) {
  Plan pl;
  if (plan_walk(sc, bc, 1, walk_len, &pl) != WOB_OK) return -1;
  return pl.L;
}

wob_status wob_solve(wob_scene sc, const void* points, const int32_t* point_prim, int64_t n_points,
                     const wob_bc* bc, int32_t samples, int32_t walk_len, uint64_t seed,
                     void* mean_out, void* var_out, void* stream) {
  return run_walk(sc, points, point_prim, n_points, bc, samples, walk_len, seed, nullptr, mean_out,
                  var_out, nullptr, nullptr, nullptr, nullptr, MODE_SOLVE, stream);
}

wob_status wob_solve_ordered_workspace(wob_scene sc, int64_t n_points, size_t* bytes) {
  if (!sc || !bytes || n_points < 0 || n_points > INT32_MAX) return WOB_E_ARG;
  *bytes = order_layout(sc->dim, sc->precision, n_points).total;
  return WOB_OK;
}

wob_status wob_solve_ordered(wob_scene sc, const void* points, const int32_t* point_prim, int64_t n_points,
                             const wob_bc* bc, int32_t samples, int32_t walk_len, uint64_t seed,
                             void* mean_out, void* var_out, void* workspace, size_t workspace_bytes,
                             void* stream) {
  Plan pl;
  wob_status s = plan_walk(sc, bc, samples, walk_len, &pl);
  if (s != WOB_OK) return s;
  if (n_points < 0 || n_points > INT32_MAX || (n_points > 0 && (!points || !mean_out))) return WOB_E_ARG;
  if (var_out && samples < 2) return WOB_E_ARG;
  if (n_points == 0) return WOB_OK;
  const OrderLayout L = order_layout(sc->dim, sc->precision, n_points);
  if (!workspace || (uintptr_t)workspace % 256 != 0 || workspace_bytes < L.total) return WOB_E_ARG;
  OrderBuffers b;
  s = order_points(sc->dim, sc->precision, L, workspace, points, point_prim, n_points, stream, &b);
  if (s != WOB_OK) return s;
  // the walk in locality order; each point keeps its own random-number index
  s = run_walk(sc, b.points, b.point_prim, n_points, bc, samples, walk_len, seed, b.order, b.mean,
               var_out ? b.var : nullptr, nullptr, nullptr, nullptr, nullptr, MODE_SOLVE, stream);
  if (s != WOB_OK) return s;
  return scatter_results(sc->precision, b, n_points, mean_out, var_out, stream);
}

wob_status wob_trace(wob_scene sc, const void* points, const int32_t* point_prim, int64_t n_points,
                     const wob_bc* bc, int32_t samples, int32_t walk_len, uint64_t seed,
                     const uint32_t* point_ids, void* path_out, int32_t* vtx_prim, int32_t* vtx_m,
                     void* stream) {
  return run_walk(sc, points, point_prim, n_points, bc, samples, walk_len, seed, point_ids, nullptr,
                  nullptr, path_out, vtx_prim, vtx_m, nullptr, MODE_TRACE, stream);
}

wob_status wob_solve_grad(wob_scene sc, const void* points, int64_t n_points, const wob_bc* bc,
                          int32_t samples, int32_t walk_len, uint64_t seed, const void* anchor_points,
                          const int32_t* anchor_prim, void* mean_out, void* var_out, void* grad_out,
                          void* grad_var_out, void* stream) {
  if (n_points > 0 && !grad_out) return WOB_E_ARG;
  return run_walk(sc, points, nullptr, n_points, bc, samples, walk_len, seed, nullptr, mean_out, var_out,
                  nullptr, nullptr, nullptr, nullptr, MODE_SOLVE, stream, nullptr, nullptr,
                  n_points > 0 ? grad_out : nullptr, grad_var_out, nullptr, anchor_points, anchor_prim);
}

wob_status wob_trace_grad(wob_scene sc, const void* points, int64_t n_points, const wob_bc* bc,
                          int32_t samples, int32_t walk_len, uint64_t seed, const void* anchor_points,
                          const int32_t* anchor_prim, void* path_out, void* path_grad_out, void* stream) {
  if (n_points > 0 && (!path_out || !path_grad_out)) return WOB_E_ARG;
  return run_walk(sc, points, nullptr, n_points, bc, samples, walk_len, seed, nullptr, nullptr, nullptr,
                  path_out, nullptr, nullptr, nullptr, MODE_TRACE, stream, nullptr, nullptr, nullptr, nullptr,
                  n_points > 0 ? path_grad_out : nullptr, anchor_points, anchor_prim);
}

wob_status wob_count_work(wob_scene sc, const void* points, const int32_t* point_prim,
                          int64_t n_points, const wob_bc* bc, int32_t samples, int32_t walk_len,
                          uint64_t seed, uint64_t* counters, void* stream) {
  return run_walk(sc, points, point_prim, n_points, bc, samples, walk_len, seed, nullptr, nullptr,
                  nullptr, nullptr, nullptr, nullptr, counters, MODE_COUNT, stream);
}

wob_status wob_cv_addback(wob_scene sc, const float* g, const void* points, int64_t n_points,
                          uint64_t seed, void* out, void* stream) {
  if (!sc || n_points < 0 || (n_points > 0 && (!g || !points || !out))) return WOB_E_ARG;
  if (sc->dim != 3 || sc->precision != WOB_F32) return WOB_E_UNSUPPORTED;
  if (n_points == 0) return WOB_OK;
  launch_addback(sc, g, points, n_points, seed, out, 0, (hipStream_t)stream);
  return hipGetLastError() == hipSuccess ? WOB_OK : WOB_E_DEVICE;
}

wob_status wob_solve_cv(wob_scene sc, const void* points, const int32_t* point_prim,
                        int64_t n_points, const wob_bc* bc, int32_t samples, int32_t walk_len,
                        uint64_t seed, const float* g, const float* g0, void* mean_out,
                        void* var_out, void* stream) {
  if (!g) return WOB_E_ARG;
  if (!g0) g0 = g;
  wob_status s = run_walk(sc, points, point_prim, n_points, bc, samples, walk_len, seed, nullptr,
                          mean_out, var_out, nullptr, nullptr, nullptr, nullptr, MODE_SOLVE, stream,
                          g, g0);
  if (s != WOB_OK || n_points == 0 || walk_len < 2) return s;
  launch_addback(sc, g0, points, n_points, seed, mean_out, 1, (hipStream_t)stream);
  return hipGetLastError() == hipSuccess ? WOB_OK : WOB_E_DEVICE;
}

wob_status wob_trace_cv(wob_scene sc, const void* points, const int32_t* point_prim,
                        int64_t n_points, const wob_bc* bc, int32_t samples, int32_t walk_len,
                        uint64_t seed, const float* g, const float* g0, void* path_out,
                        void* stream) {
  if (!g) return WOB_E_ARG;
  return run_walk(sc, points, point_prim, n_points, bc, samples, walk_len, seed, nullptr, nullptr,
                  nullptr, path_out, nullptr, nullptr, nullptr, MODE_TRACE, stream, g, g0 ? g0 : g);
}

wob_status wob_cv_emission(wob_scene sc, const wob_bc* bc, const float* g, float* g0_out,
                           void* stream) {
  if (!sc || !bc || !g0_out) return WOB_E_ARG;
  if (sc->dim != 3 || sc->precision != WOB_F32) return WOB_E_UNSUPPORTED;
  Plan pl;
  wob_status s = plan_walk(sc, bc, 2, 2, &pl);
  if (s != WOB_OK) return s;
  if (pl.form != WOB_F_SINGLE_LAYER || bc->density || sc->n_dirichlet > 0) return WOB_E_UNSUPPORTED;
  const auto a = make_args<float, 3>(sc, pl, nullptr, nullptr, 0, bc, 2, 2, 0);
  hipLaunchKernelGGL((wob::emission_table_kernel<float>), dim3((unsigned)((sc->n_prims + 255) / 256)),
                     dim3(256), 0, (hipStream_t)stream, view<float, 3>(sc), a.prog, a.phi, g, g0_out);
  return hipGetLastError() == hipSuccess ? WOB_OK : WOB_E_DEVICE;
}

wob_status wob_sample_boundary(wob_scene sc, int64_t n, uint64_t seed, void* points_out,
                               int32_t* prim_out, void* stream) {
  if (!sc || n < 0 || (n > 0 && (!points_out || !prim_out))) return WOB_E_ARG;
  if (n >= ((int64_t)1 << 32)) return WOB_E_ARG;
  if (n == 0) return WOB_OK;
  const dim3 grid((unsigned)((n + 255) / 256)), block(256);
  hipStream_t st = (hipStream_t)stream;
  const uint32_t k0 = (uint32_t)(seed & 0xffffffffu), k1 = (uint32_t)(seed >> 32);
  if (sc->precision == WOB_F32) {
    if (sc->dim == 3)
      hipLaunchKernelGGL((wob::sample_boundary_kernel<float, 3>), grid, block, 0, st, view<float, 3>(sc),
                         (const float*)sc->d_area_cdf, n, k0, k1, (float*)points_out, prim_out);
    else
      hipLaunchKernelGGL((wob::sample_boundary_kernel<float, 2>), grid, block, 0, st, view<float, 2>(sc),
                         (const float*)sc->d_area_cdf, n, k0, k1, (float*)points_out, prim_out);
  } else {
    if (sc->dim == 3)
      hipLaunchKernelGGL((wob::sample_boundary_kernel<double, 3>), grid, block, 0, st, view<double, 3>(sc),
                         (const float*)sc->d_area_cdf, n, k0, k1, (double*)points_out, prim_out);
    else
      hipLaunchKernelGGL((wob::sample_boundary_kernel<double, 2>), grid, block, 0, st, view<double, 2>(sc),
                         (const float*)sc->d_area_cdf, n, k0, k1, (double*)points_out, prim_out);
  }
  return hipGetLastError() == hipSuccess ? WOB_OK : WOB_E_DEVICE;
}

wob_status wob_cv_table(wob_scene sc, wob_mlp net, float* g_out, void* stream) {
  if (!sc || !net || !g_out) return WOB_E_ARG;
  if (sc->dim != 3 || sc->precision != WOB_F32) return WOB_E_UNSUPPORTED;
  float* cen = nullptr;
  if (hipMalloc((void**)&cen, sizeof(float) * 3 * sc->n_prims) != hipSuccess) return WOB_E_ALLOC;
  hipStream_t st = (hipStream_t)stream;
  hipLaunchKernelGGL((wob::centroid_kernel<float>), dim3((unsigned)((sc->n_prims + 255) / 256)),
                     dim3(256), 0, st, view<float, 3>(sc), cen);
  wob_status s = hipGetLastError() == hipSuccess ? WOB_OK : WOB_E_DEVICE;
  if (s == WOB_OK) s = wob_mlp_forward(net, cen, sc->n_prims, g_out, stream);
  if (hipStreamSynchronize(st) != hipSuccess && s == WOB_OK) s = WOB_E_DEVICE;
  (void)hipFree(cen);
  return s;
}

wob_status wob_intersect_all(wob_scene sc, const void* orig, const void* dir,
                             const int32_t* exclude, int64_t n_lines, int32_t max_hits,
                             int32_t* n_hits, int32_t* hit_prim, void* hit_t, void* stream) {
  if (!sc || n_lines < 0 || max_hits < 0) return WOB_E_ARG;
  if (n_lines == 0) return WOB_OK;
  if (!orig || !dir || !n_hits || (max_hits > 0 && !hit_prim)) return WOB_E_ARG;
  hipStream_t st = (hipStream_t)stream;
  const dim3 grid((unsigned)((n_lines + 255) / 256)), block(256);
  if (sc->precision == WOB_F32) {
    if (sc->dim == 3)
      hipLaunchKernelGGL((wob::intersect_kernel<float, 3>), grid, block, 0, st, view<float, 3>(sc),
                         (const float*)orig, (const float*)dir, exclude, n_lines, max_hits, n_hits,
                         hit_prim, (float*)hit_t);
    else
      hipLaunchKernelGGL((wob::intersect_kernel<float, 2>), grid, block, 0, st, view<float, 2>(sc),
                         (const float*)orig, (const float*)dir, exclude, n_lines, max_hits, n_hits,
                         hit_prim, (float*)hit_t);
  } else {
    if (sc->dim == 3)
      hipLaunchKernelGGL((wob::intersect_kernel<double, 3>), grid, block, 0, st, view<double, 3>(sc),
                         (const double*)orig, (const double*)dir, exclude, n_lines, max_hits, n_hits,
                         hit_prim, (double*)hit_t);
    else
      hipLaunchKernelGGL((wob::intersect_kernel<double, 2>), grid, block, 0, st, view<double, 2>(sc),
                         (const double*)orig, (const double*)dir, exclude, n_lines, max_hits, n_hits,
                         hit_prim, (double*)hit_t);
  }
  return hipGetLastError() == hipSuccess ? WOB_OK : WOB_E_DEVICE;
}

}  // extern "C"
