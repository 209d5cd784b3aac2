// Internal helpers shared by the ABI translation units (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>

#include "../../include/wob.h"
#include "walk.hpp"

struct wob_scene_s {
  int32_t dim = 0, precision = 0, device = 0;
  int32_t n_cu = 0;       // compute units of the device
  int64_t n_prims = 0, n_nodes = 0, n_leaves = 0, n_verts = 0;
  int32_t n_inner = 0;    // interior records on the device
  int32_t root = 0;       // root entry (record 0, or a leaf)
  int32_t stack_cap = 1;  // traversal stack entries per lane
  double frame_c[3] = {0, 0, 0}, frame_k = 1;  // frame of the stored boxes
  int32_t depth = 0, max_leaf = 0;
  void* d_nodes = nullptr;
  void* d_prims = nullptr;
  void* d_normals = nullptr;
  int32_t* d_leaf_of_id = nullptr;
  void* d_verts = nullptr;       // the rounded vertices (n_verts x dim, scene precision)
  int32_t* d_vid = nullptr;      // each primitive's vertex ids, caller-id order (n_prims x dim)
  float* d_area_cdf = nullptr;  // caller-id order, cumulative area / total (last entry 1)
  wob::GuideEntry* d_area_guide = nullptr;  // 2^guide_shift + 1 entries: the search range of each bucket
  void* d_candidates = nullptr;  // RIS candidates, caller-id order
  bool candidates_on_host = false;  // in pinned host memory
  int32_t guide_shift = 0;
  unsigned long long* d_status = nullptr;  // non-finite path values excluded from solves (sticky)
  double area_total = 0.0;      // |Gamma|
  int64_t normal_offset = 0;  // within a primitive record, when d_normals is null
  int64_t node_bytes = 0, prim_bytes = 0, device_bytes = 0;
  int32_t n_dirichlet = 0, n_neumann = 0, n_robin = 0;
};

namespace wobi {

// Lanes per workgroup of the single-problem solve: one wavefront, so a
// wavefront whose points end early (exterior points whose lines miss the
// boundary) frees its slot at once instead of waiting for the slowest
// wavefront of a larger workgroup (three-tori workload, 1M points x 512 paths:
// 256 / 128 / 64 lanes 723 / 621 / 522 ms; icosphere slice 58.9 / 58.8 / 58.7).
constexpr int kSolveBlock = 64;

// Paths per lane, on average (the lanes of a point share its paths and take
// the next one as theirs end): fixes the lanes per point.  Measured with 8, 4
// and 2: gradient walk of 60k points x 128 paths 12.02 / 12.05 / 11.19 ms, batch
// of 16 problems 36.8 / 36.4 / 36.0, RIS 4.36 / 4.37 / 4.28, single layer on
// 100k points x 64 paths 4.78 / 4.28 / 4.39; the three-tori workload (512
// paths: 32 lanes either way) 313.2 / 313.6 / 313.3.
constexpr int kPathsPerLane = 2;

// log2 of the lanes that share one point: the smallest power of two >=
// ceil(N / kPathsPerLane), at most the block (a wavefront holds several points
// when that is below 64), and at most 32 for solves whose lane groups pool
// two points (wob::pools_points: a group of 2 x 32 lanes is one wavefront)
inline int lpp_shift_for(int32_t samples, int block, bool pooled = false) {
  const int32_t lanes = (samples - 1) / kPathsPerLane + 1;
  const int cap = pooled ? (block < 32 ? block : 32) : block;
  int s = 0;
  while ((1 << s) < lanes && (1 << s) < cap) ++s;
  return s;
}

// The same for a solve of few paths: the lanes per point are doubled, down to
// one path per lane, while the launch is short of wavefronts.  Up to 64 lanes
// per point the line lies at 64 wavefronts per CU, four times what is resident
// (with 16 / 32 / 64 per CU: single layer on 30k points x 128 paths 3.24 / 2.87 /
// 2.74 ms, double layer on 20k x 64 1.72 / 1.46 / 1.37): shorter wavefronts wait
// less for their slowest lane.  Beyond, a point takes several wavefronts of one
// workgroup, which wait for each other: up to 8 per CU (exterior Neumann, 4,000
// points x 128 paths: 0.37 ms with 64 lanes per point, 0.48 with 128; 16
// points x 256 paths: 1.65 ms with 32 lanes, 0.25 with 256).
// The launch holds `others` lanes besides (the other problems of a batch), which
// are taken to be doubled likewise; there, up to 16 wavefronts per CU while a lane
// keeps two paths or more (four problems of 1,000 points x 1,024 paths, direct BIE:
// 2.03 ms with 64 lanes per point, 1.70 with 128).
// Walks of the single layer and the direct BIE by lines, whose paths differ most in
// length (many lines miss), take one path per lane only up to 8 wavefronts per CU:
// beyond, the lanes that wait cost more (direct BIE on 62,720 triangles, 28,125 points
// x 64 paths 1.24 ms with 32 lanes per point, 1.83 with 64; 7,812 points 0.39 against
// 0.59).  In FP64, of two wavefronts per SIMD, no doubling pays beyond 8 (direct BIE,
// 28,125 points x 64 paths 2.02 ms against 3.22; 7,812 points 0.62 against 0.98), in
// 2D beyond 16 (28,125 points 0.92 against 1.31; 7,812 x 200 paths, single layer, 0.69
// with 32 lanes, 0.64 with 64).
template <typename R, int D>
int spread_shift(int form, int shift, int max_shift, int64_t n_points, int32_t samples, int32_t n_cu,
                 int64_t others = 0) {
  const bool uneven = form == wob::F_SL || form == wob::F_DIRECT;
  for (int64_t lanes = (n_points << shift) + others;
       shift < max_shift && ((int64_t)1 << shift) < samples; lanes *= 2, ++shift) {
    int per_cu = 64;
    if (shift >= 6) per_cu = others > 0 && ((int64_t)4 << shift) <= samples ? 16 : 8;
    else if (uneven && sizeof(R) == 8) per_cu = D == 3 ? 8 : 16;
    else if (uneven && samples <= 2 << shift) per_cu = 8;
    if (lanes >= (int64_t)n_cu * 64 * per_cu) break;
  }
  // a launch takes less than 2^32 lanes
  while (shift > 0 && (n_points << shift) >> 31) --shift;
  return shift;
}

// The lanes of a point of a plain solve: `spread` where the walk leaves the pools
// of two points or takes more than a wavefront per point, in workgroups of up to
// 256 or kWideBlock lanes, as the LDS of the scene's stacks allows.  `others`: the
// lanes of the other problems of a batch, before any spread.  A spread point's
// lanes wait for its longest path, which costs more than it gives where the other
// problems fill the chip (64 problems of 1,000 points x 256 paths, direct BIE:
// 12.8 ms with the lanes that each would take alone, 5.5 so).
template <typename R>
constexpr int kWideBlock = sizeof(R) == 4 ? 1024 : 512;

struct LaneSplit {
  int shift;
  bool spread;
};

template <typename R, int D>
LaneSplit split_lanes(int form, bool pooled, int32_t stack_cap, int64_t n_points, int32_t samples, int32_t n_cu,
                      int64_t others = 0) {
  constexpr size_t lds_limit = 160 * 1024 - 1024;
  const int most = wob::walk_lds_bytes(stack_cap, kWideBlock<R>) <= lds_limit ? (kWideBlock<R> == 1024 ? 10 : 9)
                   : wob::walk_lds_bytes(stack_cap, 256) <= lds_limit         ? 8
                                                                              : 6;
  const int shift0 = lpp_shift_for(samples, kSolveBlock, pooled);
  const int shift = spread_shift<R, D>(form, shift0, most, n_points, samples, n_cu, others);
  return {shift, (shift > shift0 && (pooled || shift > 6)) || (pooled && samples >= wob::kMaxPooled)};
}

template <typename R, int D>
wob::SceneView<R, D> view(const wob_scene_s* sc) {
  wob::SceneView<R, D> s;
  s.nodes = (const typename wob::Rec<R, D>::Node*)sc->d_nodes;
  s.prims = (const char*)sc->d_prims;
  s.prim_stride = (uint32_t)sc->prim_bytes;
  // beside the records, or an array of their own
  s.normals = sc->d_normals ? (const char*)sc->d_normals : (const char*)sc->d_prims + sc->normal_offset;
  s.normal_stride = sc->d_normals ? (uint32_t)(wob::kNormalValues<R, D> * sizeof(R)) : (uint32_t)sc->prim_bytes;
  s.leaf_of_id = sc->d_leaf_of_id;
  s.area_cdf = sc->d_area_cdf;
  s.area_guide = sc->d_area_guide;
  s.candidates = (const wob::Candidate<R>*)sc->d_candidates;
  s.guide_shift = sc->guide_shift;
  s.area_total = (R)sc->area_total;
  s.n_nodes = sc->n_inner;
  s.n_prims = (int32_t)sc->n_prims;
  s.root = sc->root;
  s.stack_cap = sc->stack_cap;
  for (int a = 0; a < 3; ++a) s.fc[a] = (R)sc->frame_c[a];
  s.fk = (R)sc->frame_k;
  return s;
}

inline int resolve_formulation(const wob_scene_s* sc, int f) {
  const bool d = sc->n_dirichlet > 0, n = sc->n_neumann > 0, r = sc->n_robin > 0;
  if (f == WOB_F_AUTO) {
    if (!n && !r) return WOB_F_DOUBLE_LAYER;
    if (!d && !r) return WOB_F_DIRECT;
    return WOB_F_SINGLE_LAYER;  // Robin parts or mixed kinds (Dirichlet parts: first-kind rows)
  }
  if (f == WOB_F_DOUBLE_LAYER) return (!n && !r) ? f : -1;
  if (f == WOB_F_DIRECT) return (!d && !r) ? f : -1;
  if (f == WOB_F_SINGLE_LAYER) return f;
  return -2;
}

struct Plan {
  int form;
  int32_t L;
  uint32_t self_thr;
  double self_p;
  int32_t ris_c;  // RIS candidates, 0 = line sampling
  uint32_t mixed_thr;
  double mixed_p, mixed_k;
};

// The data program of a solve: the analytic program, or the per-vertex data.
template <typename R>
wob::ProgramView<R> make_program(const wob_scene_s* sc, const wob_bc* bc) {
  wob::ProgramView<R> g;
  std::memset(&g, 0, sizeof(g));
  g.type = bc->data_mode == WOB_DATA_VERTEX ? wob::P_VERTEX : bc->program;
  for (int k = 0; k < 8; ++k) g.p[k] = (R)bc->params[k];
  g.vdata = (const R*)bc->vertex_data;
  g.vid = sc->d_vid;
  g.verts = (const R*)sc->d_verts;
  return g;
}

// Data mode and program of a wob_bc.
inline wob_status check_data(const wob_bc* bc) {
  if (bc->data_mode != WOB_DATA_PROGRAM && bc->data_mode != WOB_DATA_VERTEX) return WOB_E_ARG;
  if (bc->path_offset < 0) return WOB_E_ARG;
  if (bc->data_mode == WOB_DATA_VERTEX) return bc->vertex_data ? WOB_OK : WOB_E_ARG;
  if (bc->program < WOB_PROG_CONST || bc->program > WOB_PROG_INVDIST) return WOB_E_ARG;
  return WOB_OK;
}

inline wob_status plan_walk(const wob_scene_s* sc, const wob_bc* bc, int32_t samples, int32_t walk_len,
                     Plan* p) {
  if (!sc || !bc) return WOB_E_ARG;
  if (check_data(bc) != WOB_OK) return WOB_E_ARG;
  if (bc->domain != 1 && bc->domain != -1) return WOB_E_ARG;
  if (bc->density != 0 && bc->density != 1) return WOB_E_ARG;
  if (samples < 1 || walk_len < 1 || walk_len >= 65535) return WOB_E_ARG;
  if ((int64_t)bc->path_offset + samples > INT32_MAX) return WOB_E_ARG;
  const int f = resolve_formulation(sc, bc->formulation);
  if (f == -2) return WOB_E_ARG;
  if (f < 0) return WOB_E_UNSUPPORTED;
  if (bc->density && f == WOB_F_DIRECT) return WOB_E_UNSUPPORTED;
  double ps = bc->self_panel_p == 0.0 ? 1.0 / 16.0 : bc->self_panel_p;
  if (!(ps > 0.0 && ps < 1.0)) return WOB_E_ARG;
  p->form = f;
  p->L = f == WOB_F_DIRECT ? walk_len + 1 : walk_len;
  p->self_thr = (uint32_t)std::floor(ps * 16777216.0);
  if (p->self_thr == 0) return WOB_E_ARG;
  p->self_p = p->self_thr / 16777216.0;
  const double mk = bc->mixed_k == 0.0 ? 4.0 : bc->mixed_k;
  const double mp = bc->mixed_p == 0.0 ? 2.0 / 3.0 : bc->mixed_p;
  if (!std::isfinite(mk) || !(mp > 0.0 && mp < 1.0)) return WOB_E_ARG;
  p->mixed_k = mk;
  p->mixed_thr = (uint32_t)std::floor(mp * 16777216.0);
  if (p->mixed_thr == 0) return WOB_E_ARG;
  p->mixed_p = p->mixed_thr / 16777216.0;
  if (bc->sampling != WOB_SAMPLE_LINE && bc->sampling != WOB_SAMPLE_RIS) return WOB_E_ARG;
  p->ris_c = 0;
  if (bc->sampling == WOB_SAMPLE_RIS) {
    if (f != WOB_F_SINGLE_LAYER) return WOB_E_UNSUPPORTED;
    const int32_t c = bc->candidates == 0 ? 16 : bc->candidates;
    if (c < 1 || c > 64) return WOB_E_ARG;
    p->ris_c = c;
  }
  return WOB_OK;
}

template <typename R, int D>
wob::WalkArgs<R, D> make_args(const wob_scene_s* sc, const Plan& pl, const void* points,
                              const int32_t* point_prim, int64_t n_points, const wob_bc* bc,
                              int32_t samples, int32_t walk_len, uint64_t seed) {
  wob::WalkArgs<R, D> a;
  std::memset(&a, 0, sizeof(a));
  a.scene = view<R, D>(sc);
  a.prog = make_program<R>(sc, bc);
  a.points = (const R*)points;
  a.point_prim = point_prim;
  a.n_points = n_points;
  a.N = samples;
  a.M = walk_len;
  a.L = pl.L;
  a.phi = (R)bc->domain;
  a.self_thr = pl.self_thr;
  a.self_p = (R)pl.self_p;
  a.k0 = (uint32_t)(seed & 0xffffffffu);
  a.k1 = (uint32_t)(seed >> 32);
  a.problem = 0;
  a.path_offset = bc->path_offset;
  a.lpp_shift = lpp_shift_for(samples, kSolveBlock);
  a.density = bc->density;
  a.status = sc->d_status;
  a.ris_c = pl.ris_c;
  a.mixed_thr = pl.mixed_thr;
  a.mixed_p = (R)pl.mixed_p;
  a.mixed_k = (R)pl.mixed_k;
  a.form = pl.form == WOB_F_DOUBLE_LAYER ? wob::F_DL
           : pl.form == WOB_F_DIRECT    ? wob::F_DIRECT
           : pl.ris_c > 0               ? wob::F_SL_RIS
                                        : wob::F_SL;
  return a;
}


// Workspace of the ordered solve (byte offsets, each 256-aligned): partial
// bounding boxes, Morton keys (in, sorted), indices (in, sorted = the order),
// the sorted points and primitive ids, the sorted-order results, the radix
// sort's temporary storage.
struct OrderLayout {
  size_t part, keys, keys_s, idx, order, pts, prim, mean, var, temp, temp_bytes, total;
};
// The walk's inputs in locality order: order[i] is the caller's index of
// sorted point i (also its random-number point index).
struct OrderBuffers {
  const uint32_t* order;
  const void* points;
  const int32_t* point_prim;
  void* mean;
  void* var;
};
OrderLayout order_layout(int dim, int precision, int64_t n);
// Enqueues the Morton keys, the stable sort and the gather on `stream`.
wob_status order_points(int dim, int precision, const OrderLayout& L, void* workspace, const void* points,
                        const int32_t* point_prim, int64_t n, void* stream, OrderBuffers* out);
// Enqueues mean_out[order[i]] = mean[i] (and var) on `stream`.
wob_status scatter_results(int precision, const OrderBuffers& b, int64_t n, void* mean_out, void* var_out,
                           void* stream);

}  // namespace wobi
