// C-ABI entry points of libj3d: single sweeps, residual norms, fills,
// bandwidth probe and housekeeping.  Solves, batches and serving live in
// solve.cpp, batch.cpp and serve.cpp.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "runtime.h"

namespace j3d {
const char* last_error_text();
int release_all_scratch();
bool tune_cache_lookup_single(int dtype, int nx, int ny, int nz, TileCfg* out);

namespace {
// The supported tile shapes, enumerated once: every (rows, planes, variant,
// persistent, order, cols) that tile_cfg_supported accepts.
const std::vector<TileCfg>& tune_table() {
  static const std::vector<TileCfg> table = [] {
    std::vector<TileCfg> v;
    for (int rows : {1, 2, 4, 8})
      for (int planes : {1, 2, 4, 8, 16, 32, 64, 128})
        for (int var : {0, 1, 2, 3, 4, 5, 6, 7, 16, 17, 18, 19, 20, 21, 22, 23})
          for (int pers : {0, 1})
            for (int order : {0, 1, 2})
              for (int cols : {1, 2, 4}) {
                TileCfg c{rows, planes, var, pers, order, cols};
                if (tile_cfg_supported(c)) v.push_back(c);
              }
    return v;
  }();
  return table;
}
}  // namespace

// A multi-sweep pass over small grids is short of workgroups and each tile's
// march along z is one long latency, so the best shape changes with the
// size: many short tiles below 100^3, tall blocks that just fill the 256 CUs
// around 128^3, longer tiles beyond.  The shape is the one of least modelled
// time: a round of workgroups takes (planes + fill) steps of
//   lat + lat_row * RY + row * (rows of all workgroups on a CU)  [us]
// (latency of a step, growing with the rows a thread walks, and the CU's
// throughput), cap workgroups fit a CU by registers and LDS, and the last
// round may be a partial one.  The constants were fitted to 3700 timed
// (shape, size) pairs per pass kind over 17 sizes from 32^3 to 512x512x32,
// the two-sweep ones on the pass that did not yet load a step ahead.  Timed
// again on the current kernels over 16 sizes, the shape chosen is slower than
// the fastest by, on average and at worst: FP64 two sweeps 1.6 and 6 %, three
// 0 and 0 %; FP32 two 2.9 and 13 %, three 1.0 and 9 % (tables in
// profiles/shape_estimates.md).  Against the fixed shapes before (us per pass,
// best stores of 40-256 MB passes on both sides): FP64 two sweeps 64^3 27.5 ->
// 7.2, 128^3 34.5 -> 15.2, 181x143x160 36 -> 22.4; three sweeps 96^3 20.5 ->
// 12.6, 200^3 77 -> 47; FP32 two sweeps 96^3 14.5 -> 7.2, three sweeps
// 181x143x160 31 -> 21.6.
// (All of a whole card's CUs: the shapes are fitted to and timed on those.  A
// partition runs the same shapes.)
static constexpr int kCus = 256;

TileCfg modelled_shape(int sweeps, int dtype, const Extents* e, int n) {
  const bool f32 = dtype == J3D_F32;
  struct Cost {
    double lat, lat_row, row, fill;
  };
  const Cost k = sweeps == 2 ? (f32 ? Cost{0.4, 0.056, 0.006, 3} : Cost{0.5, 0.047, 0.014, 6})
                             : (f32 ? Cost{0.3, 0.0026, 0.01, 3} : Cost{0.3, 0.115, 0.042, 4});
  const int width = 64 - 2 * sweeps, ring = 2 * (sweeps - 1);
  constexpr int kPlanes[] = {4, 6, 8, 10, 12, 16, 20, 24, 32, 48, 64};
  constexpr int kNumPlanes = sizeof kPlanes / sizeof *kPlanes;
  struct Shape {
    TileCfg c;
    int ry, h;
    double tiles[kNumPlanes];
  } shapes[8];
  int ns = 0;
  for (int rows : {2, 4, 8, 16})
    for (int ry : {2, 4}) {
      const TileCfg c{rows, 1, ry == 4 ? 20 : 6, 0, 0, 1};
      if (sweeps == 2 ? tile2_cfg_supported(dtype, c) : tile3_cfg_supported(dtype, c))
        shapes[ns++] = Shape{c, ry, rows * ry - ring, {}};
    }
  // The tiles of every shape in one walk over the grids (a server asks for up
  // to 256 of them between two cycles: 15 us, 190 with the tiles counted anew
  // for every shape and number of planes).
  auto ceil_div = [](int a, int b) { return (a + b - 1) / b; };
  int deepest = 1;
  for (int g = 0; g < n; ++g) {
    double slabs[kNumPlanes];
    for (int p = 0; p < kNumPlanes; ++p) slabs[p] = ceil_div(e[g].nz, kPlanes[p]);
    const double across = ceil_div(e[g].nx, width);
    for (int s = 0; s < ns; ++s) {
      const double cols = across * ceil_div(e[g].ny, shapes[s].h);
      for (int p = 0; p < kNumPlanes; ++p) shapes[s].tiles[p] += cols * slabs[p];
    }
    deepest = std::max(deepest, e[g].nz);
  }
  TileCfg best{4, 16, 6, 0, 0, 1};
  double best_t = 1e300;
  for (int s = 0; s < ns; ++s) {
    const int rows = shapes[s].c.rows, ry = shapes[s].ry;
    const int waves = sweeps == 3 ? (ry == 2 || f32 ? 16 : 12) : (ry == 2 || f32 ? 24 : 16);
    const int cap = std::max(1, waves / rows);
    auto step = [&](double wgs) { return k.lat + k.lat_row * ry + k.row * wgs * rows * ry; };
    for (int p = 0; p < kNumPlanes; ++p) {
      const double per_cu = std::ceil(shapes[s].tiles[p] / kCus);
      const double full = std::floor(per_cu / cap), part = per_cu - full * cap;
      const double t =
          (std::min(kPlanes[p], deepest) + k.fill) * (full * step(cap) + (part > 0 ? step(part) : 0.0));
      if (t < best_t * (1.0 - 1e-12)) {
        best_t = t;
        best = shapes[s].c;
        best.planes = kPlanes[p];
      }
    }
  }
  return best;
}

// Grids whose multi-sweep shapes come from the model: below, a pass is one
// latency whatever the shape; above, the shapes timed on large cubes.
static bool modelled_size(long long pts) { return pts >= 4096 && pts < (1LL << 24); }

TileCfg default_cfg(int dtype, int nx, int ny, int nz) {
  TileCfg c;
  if (tune_cache_lookup_single(dtype, nx, ny, nz, &c)) return c;
  // Passes that stay in the last-level cache: short tiles (4 planes, XCD-
  // blocked), us per pass against the large-grid shape below: FP64 65^3 4.8 /
  // 9.6, 72^3 5.6 / 9.9, 96^3 6.7 / 11.2, 128^3 11.4 / 12.7, 200^3 33.6 / 35.8;
  // FP32 64^3 4.3 / 8.4, 128^3 7.1 / 12.0, 256^3 32.0 / 35.3.  They would pay
  // from where the small shape below ends (65 x 64 x 64 4.7 / 9.5), but the
  // tests hold 65 x 64 x 64 to the large-grid shape, so they begin behind it.
  {
    const long long pts = (long long)nx * ny * nz;
    if (pts >= (dtype == J3D_F64 ? 65LL * 64 * 64 + 1 : 1LL << 15) &&
        (dtype == J3D_F64 ? 24.0 : 12.0) * (double)pts <= 256e6)
      return TileCfg{1, 4, 20, 0, 0, 1};
  }
  // FP64 grids of at most 64^3 points: four wavefronts of two rows per
  // thread, two planes per tile, XCD-blocked (7.45 us per sweep at 64^3 with
  // a residual after every sweep, against 7.8 with four rows per thread and
  // one plane, 16.0 with the large-grid shape).  Otherwise one wavefront of
  // four rows per thread, 16 planes per tile (the loads run one plane
  // ahead, so deep tiles cost no latency), per-slab XCD chunks: 572 us per
  // FP64 pass at 512^3 against 643 with 2 planes, 70.7 us at 256^3.
  const bool small = dtype == J3D_F64 && (long long)nx * ny * nz <= 64LL * 64 * 64;
  c.rows = small ? 4 : 1;
  c.planes = small ? 2 : 16;
  c.variant = small ? 6 : 20;  // two or four rows per thread, nontemporal stores
  c.persistent = 0;
  c.order = small ? 0 : 2;
  c.cols = 1;
  return c;
}

TileCfg default_cfg3(int dtype, int nx, int ny, int nz) {
  TileCfg c;
  const int kind = dtype == J3D_F32 ? J3D_KIND_F32X3 : J3D_KIND_F64X3;
  if (tune_cache_lookup_single(kind, nx, ny, nz, &c) && tile3_cfg_supported(dtype, c)) return c;
  const Extents e{nx, ny, nz};
  if (modelled_size((long long)nx * ny * nz)) {
    c = modelled_shape(3, dtype, &e, 1);
    int tx, ty, tz;
    tile3_counts(nx, ny, nz, c, &tx, &ty, &tz);
    // (long rows of few planes: the shapes below make fewer tiles, which the
    // allocation-free entry point's fixed number of partials must hold)
    if ((long long)tx * ty * tz <= 65536) return c;
  }
  const long long pts = (long long)nx * ny * nz;
  // FP32 from 2^24 points while all tiles are resident at once (five
  // workgroups per CU): 4 wavefronts of 4 rows, 24 planes, XCD-blocked (us per
  // pass, in brackets per-slab XCD chunks of 16 planes; tiles: 256^3 51.5
  // [57.5] 1210, 256x200x330 51.5 [58.5], 264^3 56.4 [59.8] 1210; 280x300x260
  // 80 [69] 1375, 270x280x280 73 [65] 1440).
  if (dtype == J3D_F32 && pts >= (1LL << 24) && pts <= 300LL * 300 * 300) {
    c = TileCfg{4, 24, 20, 0, 0, 1};
    int tx, ty, tz;
    tile3_counts(nx, ny, nz, c, &tx, &ty, &tz);
    if ((long long)tx * ty * tz <= 5 * kCus) return c;
  }
  // FP64 above 400^3: 16 wavefronts of 2 rows (32-row blocks, one workgroup
  // per CU), 144 planes in launch order (512^3 712 us per pass against 731
  // with 8 wavefronts and 96 planes).  One workgroup lasts a whole round of
  // the CUs, so where the last of a few rounds is less than half full, 32
  // planes in per-slab XCD chunks (us per pass, in brackets 144 planes; rounds):
  // 420^3 428 [490] 1.4, 460^3 518 [559] 2.1, 512x512x300 434 [510] 2.0,
  // 600x500x400 658 [725] 2.3, 800x400x300 528 [538] 2.5, 560x540x520 842 [960]
  // 3.1; but 500^3 678 [694] and with a residual 721 [713] 2.5, 512^3 720 [718]
  // and 764 [753] 2.7.
  if (dtype == J3D_F64 && pts > 400LL * 400 * 400) {
    c = TileCfg{16, 144, 6, 0, 1, 1};
    int tx, ty, tz;
    tile3_counts(nx, ny, nz, c, &tx, &ty, &tz);
    const long long tiles = (long long)tx * ty * tz, last = tiles % kCus;
    if (tiles < 4 * kCus && last > 0 && last < kCus / 2) {
      const TileCfg s{16, 32, 6, 0, 2, 1};
      tile3_counts(nx, ny, nz, s, &tx, &ty, &tz);
      if ((long long)tx * ty * tz <= 65536) c = s;
    }
    return c;
  }
  // Otherwise 8 wavefronts of 2 rows per thread (about 95 registers per thread
  // against 160 with 4 rows, so twice the wavefronts per CU), 32 planes in
  // per-slab XCD chunks (FP64 300x320x280 165 us against 177 with 4 x 4 rows,
  // 280x300x260 121); FP32 above 400^3 48 planes (512^3 419 us against 439
  // with 4 wavefronts of 4 rows and 24 planes), FP32 up to 300^3 4 wavefronts
  // of 4 rows, 16 planes.  FP64 256^3 itself keeps those too, the default that
  // the tests hold it to (111 us, with a residual 125, against 109 and 120).
  // Grids below 2^24 points come here only when too flat for the model: 4
  // wavefronts, up to 200^3 points of 2 rows and XCD-blocked.
  const bool small = pts <= 200LL * 200 * 200;
  const bool large = pts > (dtype == J3D_F32 ? 300LL * 300 * 300 : 1LL << 24);
  c.rows = large ? 8 : 4;
  c.planes = !large ? 16 : dtype == J3D_F32 && pts > 400LL * 400 * 400 ? 48 : 32;
  c.variant = (small || large) ? 6 : 20;
  c.persistent = 0;
  c.order = small ? 0 : 2;
  c.cols = 1;
  return c;
}

TileCfg default_cfg2(int dtype, int nx, int ny, int nz) {
  TileCfg c;
  if (tune_cache_lookup_single(dtype == J3D_F32 ? J3D_KIND_F32X2 : J3D_KIND_F64X2, nx, ny, nz, &c) &&
      tile2_cfg_supported(dtype == J3D_F32 ? J3D_F32 : J3D_F64, c))
    return c;
  const Extents e{nx, ny, nz};
  const long long pts = (long long)nx * ny * nz;
  if (modelled_size(pts)) return modelled_shape(2, dtype, &e, 1);
  // FP32 up to 300^3: 4 wavefronts of 4 rows, 8 planes, XCD-blocked; beyond,
  // where the halo rows of a contiguous block overflow an XCD's L2, 8
  // wavefronts of 2 rows, 12 planes in per-slab XCD chunks (us per pass,
  // first / second: 256^3 40.5 / 45.5, 300x320x280 73.4 / 72.6, 512x300x200
  // 93 / 86, 400^3 207 / 188, 460^3 330 / 275, 512^3 405 / 374, 700x640x600
  // 927 / 749).
  if (dtype == J3D_F32 && pts >= 4096)
    return pts <= 300LL * 300 * 300 ? TileCfg{4, 8, 20, 0, 0, 1} : TileCfg{8, 12, 6, 0, 2, 1};
  // FP64: 4 wavefronts of 4 rows, 12 planes, per-slab XCD chunks (us per pass,
  // in brackets with 16 planes in launch order: 256^3 92 [103], 300^3 140
  // [156], 200x300x500 167 [181], 400^3 331 [336], 512^3 672 [690])
  if (dtype == J3D_F64 && pts >= (1LL << 24)) return TileCfg{4, 12, 20, 0, 2, 1};
  // fewer than 4096 points are one latency in any shape
  c.rows = dtype == J3D_F32 ? 8 : 4;
  c.planes = dtype == J3D_F32 ? 8 : 16;
  c.variant = 20;
  c.persistent = 0;
  c.order = dtype == J3D_F32 ? 0 : 1;
  c.cols = 1;
  return c;
}

// Sum-of-squares pass over (u, f) followed by the deterministic reduce into
// `out` (device).  flags is F_RES (residual of u) or F_NORM (norm of f).
static int norm_pass(unsigned flags, const Field& u, const Field& f, const Field* o, double h,
                     const TileCfg& c, double* out, hipStream_t st, Scratch* s) {
  const Field* up = (flags & F_NORM) ? nullptr : &u;
  GridArgs g = make_args(up, o, &f, nullptr, nullptr, h, c, 0);
  const int nt = g.tiles_x * g.tiles_y * g.tiles_z;
  J3D_TRY(ensure_partials(s, nt));
  J3D_HIP(launch_pass_one(J3D_F64, flags, c, g, s->partials, nullptr, st));
  J3D_HIP(launch_reduce_one(s->partials, 0, nt, out, nullptr, 0.0, 0, nullptr, nullptr, nullptr, st));
  return J3D_OK;
}

int check_sweep3_call(const j3d_array* u_in, const j3d_array* u_out, const j3d_array* f, double h,
                      uint32_t flags, const double* resid_out, Sweep3Call* k) {
  Field& a = k->a;
  Field& b = k->b;
  Field& c = k->c;
  J3D_TRY(check_field(u_in, -1, &a, "u_in"));
  J3D_TRY(check_field(u_out, a.dtype, &b, "u_out"));
  J3D_TRY(check_field(f, a.dtype, &c, "f"));
  J3D_TRY(check_same_interior(a, b, "u_in", "u_out"));
  J3D_TRY(check_same_interior(a, c, "u_in", "f"));
  J3D_TRY(check_h(h));
  if ((flags & ~(J3D_HOST_RESULT | J3D_RESID_AFTER_1 | J3D_RESID_AFTER_2)) != 0)
    return fail(J3D_EINVAL, "unknown flags 0x%x", flags);
  const unsigned after = flags & (J3D_RESID_AFTER_1 | J3D_RESID_AFTER_2);
  if (after == (J3D_RESID_AFTER_1 | J3D_RESID_AFTER_2))
    return fail(J3D_EINVAL, "J3D_RESID_AFTER_1 and J3D_RESID_AFTER_2 are exclusive");
  if (after != 0 && resid_out == nullptr) return fail(J3D_EINVAL, "J3D_RESID_AFTER_*: resid_out is null");
  if (fields_overlap(a, b)) return fail(J3D_EALIAS, "u_in and u_out overlap");
  if (fields_overlap(b, c)) return fail(J3D_EALIAS, "u_out and f overlap");
  if (resid_out != nullptr && a.dtype != J3D_F64)
    return fail(J3D_EDTYPE, "a fused residual needs FP64 arrays");
  if (!plane_fits_u32(a) || !plane_fits_u32(b) || !plane_fits_u32(c))
    return fail(J3D_EINVAL, "a z-plane spans 4 GiB or more: the three-sweep pass needs smaller planes");
  k->res_flag = after == J3D_RESID_AFTER_1 ? F_RES1 : after == J3D_RESID_AFTER_2 ? F_RES2 : F_RES;
  k->cfg = default_cfg3(a.dtype, a.nx(), a.ny(), a.nz());
  k->g = make_args3(&a, &b, &c, nullptr, h, k->cfg, 0);
  return J3D_OK;
}

}  // namespace j3d

using namespace j3d;

extern "C" {

int j3d_abi_version(void) { return J3D_ABI_VERSION; }

const char* j3d_last_error(void) { return last_error_text(); }

int j3d_element_offset(const j3d_array* a, int64_t i, int64_t j, int64_t k, int64_t* offset) {
  J3D_TRY(check_field(a, -1, nullptr, "array"));
  if (offset == nullptr) return fail(J3D_EINVAL, "offset: null pointer");
  const int64_t idx[3] = {i, j, k};
  int64_t off = 0;
  for (int d = 0; d < 3; ++d) {
    if (idx[d] < a->lbound[d] || idx[d] > a->ubound[d])
      return fail(J3D_EINVAL, "index %lld outside bounds %lld:%lld on axis %d", (long long)idx[d],
                  (long long)a->lbound[d], (long long)a->ubound[d], d);
    off += (idx[d] - a->lbound[d]) * a->stride[d];
  }
  *offset = off;
  return J3D_OK;
}

int j3d_check_array(const j3d_array* a, int32_t dtype) { return check_field(a, dtype, nullptr, "array"); }

int j3d_tune_query_single(int32_t kind, int32_t nx, int32_t ny, int32_t nz, j3d_tune* out) {
  if (out == nullptr) return fail(J3D_EINVAL, "tune: null pointer");
  if (nx < 1 || ny < 1 || nz < 1) return fail(J3D_EINVAL, "extents must be >= 1");
  TileCfg c;
  if (kind == J3D_F64 || kind == J3D_F32)
    c = default_cfg(kind, nx, ny, nz);
  else if (kind == J3D_KIND_F64X2 || kind == J3D_KIND_F32X2)
    c = default_cfg2(kind == J3D_KIND_F32X2 ? J3D_F32 : J3D_F64, nx, ny, nz);
  else if (kind == J3D_KIND_F64X3 || kind == J3D_KIND_F32X3)
    c = default_cfg3(kind == J3D_KIND_F32X3 ? J3D_F32 : J3D_F64, nx, ny, nz);
  else
    return fail(J3D_EDTYPE, "kind must be J3D_F64, J3D_F32 or a J3D_KIND_* pass kind");
  out->rows = c.rows;
  out->planes = c.planes;
  out->variant = c.variant;
  out->persistent = c.persistent;
  out->order = c.order;
  out->cols = c.cols;
  return J3D_OK;
}

int j3d_tune_count(void) { return (int)tune_table().size(); }

int j3d_tune_get(int32_t index, j3d_tune* out) {
  if (out == nullptr || index < 0 || index >= (int)tune_table().size())
    return fail(J3D_EINVAL, "tune index out of range");
  const TileCfg& c = tune_table()[(size_t)index];
  out->rows = c.rows;
  out->planes = c.planes;
  out->variant = c.variant;
  out->persistent = c.persistent;
  out->order = c.order;
  out->cols = c.cols;
  return J3D_OK;
}

int jacobi3d_sweep(const j3d_array* u_in, j3d_array* u_out, const j3d_array* f, double h,
                   uint32_t flags, double* resid_out, void* stream) {
  Field a, b, c;
  J3D_TRY(check_field(u_in, -1, &a, "u_in"));
  J3D_TRY(check_field(u_out, a.dtype, &b, "u_out"));
  J3D_TRY(check_field(f, a.dtype, &c, "f"));
  J3D_TRY(check_same_interior(a, b, "u_in", "u_out"));
  J3D_TRY(check_same_interior(a, c, "u_in", "f"));
  J3D_TRY(check_h(h));
  if ((flags & ~J3D_HOST_RESULT) != 0) return fail(J3D_EINVAL, "unknown flags 0x%x", flags);
  if (fields_overlap(a, b)) return fail(J3D_EALIAS, "u_in and u_out overlap");
  if (fields_overlap(b, c)) return fail(J3D_EALIAS, "u_out and f overlap");
  if (resid_out != nullptr && a.dtype != J3D_F64)
    return fail(J3D_EDTYPE, "a fused residual needs FP64 arrays");
  hipStream_t st = static_cast<hipStream_t>(stream);
  const TileCfg cfg = default_cfg(a.dtype, a.nx(), a.ny(), a.nz());
  GridArgs g = make_args(&a, &b, &c, nullptr, nullptr, h, cfg, 0);
  if (resid_out == nullptr) {
    J3D_HIP(launch_pass_one(a.dtype, F_WRITE, cfg, g, nullptr, nullptr, st));
    return J3D_OK;
  }
  Scratch* s = nullptr;
  J3D_TRY(get_scratch(st, &s));
  const int nt = g.tiles_x * g.tiles_y * g.tiles_z;
  J3D_TRY(ensure_partials(s, nt));
  J3D_HIP(launch_pass_one(J3D_F64, F_WRITE | F_RES, cfg, g, s->partials, nullptr, st));
  const bool host = (flags & J3D_HOST_RESULT) != 0;
  double* dst = host ? &s->ctl->value : resid_out;
  J3D_HIP(launch_reduce_one(s->partials, 0, nt, dst, nullptr, 0.0, 0, nullptr, nullptr, nullptr, st));
  if (host) {
    J3D_HIP(hipMemcpyAsync(&s->ctl_host->value, &s->ctl->value, sizeof(double),
                           hipMemcpyDeviceToHost, st));
    J3D_HIP(hipStreamSynchronize(st));
    *resid_out = s->ctl_host->value;
  }
  return J3D_OK;
}

int jacobi3d_sweep2(const j3d_array* u_in, j3d_array* u_out, const j3d_array* f, double h,
                    uint32_t flags, double* resid_out, void* stream) {
  Field a, b, c;
  J3D_TRY(check_field(u_in, -1, &a, "u_in"));
  J3D_TRY(check_field(u_out, a.dtype, &b, "u_out"));
  J3D_TRY(check_field(f, a.dtype, &c, "f"));
  J3D_TRY(check_same_interior(a, b, "u_in", "u_out"));
  J3D_TRY(check_same_interior(a, c, "u_in", "f"));
  J3D_TRY(check_h(h));
  if ((flags & ~J3D_HOST_RESULT) != 0) return fail(J3D_EINVAL, "unknown flags 0x%x", flags);
  if (fields_overlap(a, b)) return fail(J3D_EALIAS, "u_in and u_out overlap");
  if (fields_overlap(b, c)) return fail(J3D_EALIAS, "u_out and f overlap");
  if (resid_out != nullptr && a.dtype != J3D_F64)
    return fail(J3D_EDTYPE, "a fused residual needs FP64 arrays");
  hipStream_t st = static_cast<hipStream_t>(stream);
  const TileCfg cfg = default_cfg2(a.dtype, a.nx(), a.ny(), a.nz());
  GridArgs g = make_args2(&a, &b, &c, nullptr, h, cfg, 0);
  if (resid_out == nullptr) {
    J3D_HIP(launch_sweep2_one(a.dtype, F_WRITE, cfg, g, nullptr, nullptr, st));
    return J3D_OK;
  }
  Scratch* s = nullptr;
  J3D_TRY(get_scratch(st, &s));
  const int nt = g.tiles_x * g.tiles_y * g.tiles_z;
  J3D_TRY(ensure_partials(s, nt));
  J3D_HIP(launch_sweep2_one(J3D_F64, F_WRITE | F_RES, cfg, g, s->partials, nullptr, st));
  const bool host = (flags & J3D_HOST_RESULT) != 0;
  double* dst = host ? &s->ctl->value : resid_out;
  J3D_HIP(launch_reduce_one(s->partials, 0, nt, dst, nullptr, 0.0, 0, nullptr, nullptr, nullptr, st));
  if (host) {
    J3D_HIP(hipMemcpyAsync(&s->ctl_host->value, &s->ctl->value, sizeof(double),
                           hipMemcpyDeviceToHost, st));
    J3D_HIP(hipStreamSynchronize(st));
    *resid_out = s->ctl_host->value;
  }
  return J3D_OK;
}

int jacobi3d_sweep3(const j3d_array* u_in, j3d_array* u_out, const j3d_array* f, double h,
                    uint32_t flags, double* resid_out, void* stream) {
  Sweep3Call k;
  J3D_TRY(check_sweep3_call(u_in, u_out, f, h, flags, resid_out, &k));
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (resid_out == nullptr) {
    J3D_HIP(launch_sweep3_one(k.a.dtype, F_WRITE, k.cfg, k.g, nullptr, nullptr, st));
    return J3D_OK;
  }
  Scratch* s = nullptr;
  J3D_TRY(get_scratch(st, &s));
  const int nt = k.g.tiles_x * k.g.tiles_y * k.g.tiles_z;
  J3D_TRY(ensure_partials(s, nt));
  J3D_HIP(launch_sweep3_one(J3D_F64, F_WRITE | k.res_flag, k.cfg, k.g, s->partials, nullptr, st));
  const bool host = (flags & J3D_HOST_RESULT) != 0;
  double* dst = host ? &s->ctl->value : resid_out;
  J3D_HIP(launch_reduce_one(s->partials, 0, nt, dst, nullptr, 0.0, 0, nullptr, nullptr, nullptr, st));
  if (host) {
    J3D_HIP(hipMemcpyAsync(&s->ctl_host->value, &s->ctl->value, sizeof(double),
                           hipMemcpyDeviceToHost, st));
    J3D_HIP(hipStreamSynchronize(st));
    *resid_out = s->ctl_host->value;
  }
  return J3D_OK;
}

int residual_l2(const j3d_array* u, const j3d_array* f, double h, uint32_t flags, double* out,
                void* stream) {
  Field a, c;
  J3D_TRY(check_field(u, J3D_F64, &a, "u"));
  J3D_TRY(check_field(f, J3D_F64, &c, "f"));
  J3D_TRY(check_same_interior(a, c, "u", "f"));
  J3D_TRY(check_h(h));
  if ((flags & ~J3D_HOST_RESULT) != 0) return fail(J3D_EINVAL, "unknown flags 0x%x", flags);
  if (out == nullptr) return fail(J3D_EINVAL, "out: null pointer");
  hipStream_t st = static_cast<hipStream_t>(stream);
  Scratch* s = nullptr;
  J3D_TRY(get_scratch(st, &s));
  const TileCfg cfg = default_cfg(J3D_F64, a.nx(), a.ny(), a.nz());
  const bool host = (flags & J3D_HOST_RESULT) != 0;
  J3D_TRY(norm_pass(F_RES, a, c, nullptr, h, cfg, host ? &s->ctl->value : out, st, s));
  if (host) {
    J3D_HIP(hipMemcpyAsync(&s->ctl_host->value, &s->ctl->value, sizeof(double),
                           hipMemcpyDeviceToHost, st));
    J3D_HIP(hipStreamSynchronize(st));
    *out = s->ctl_host->value;
  }
  return J3D_OK;
}

int j3d_fill_uniform(j3d_array* a, uint64_t seed, uint32_t stream_id, double lo, double hi,
                     double halo, void* stream) {
  Field x;
  J3D_TRY(check_field_wide(a, J3D_F64, &x, "a"));
  if (x.ey > 65535 || x.ez > 65535) return fail(J3D_EINVAL, "fill: y/z extents above 65535");
  const unsigned long long key = seed ^ (static_cast<unsigned long long>(stream_id) << 40);
  J3D_HIP(launch_fill_uniform(reinterpret_cast<double*>(x.base), x.ex, x.ey, x.ez, x.sy, x.sz, key,
                              lo, hi, halo, static_cast<hipStream_t>(stream)));
  return J3D_OK;
}

int j3d_fill_const(j3d_array* a, double value, void* stream) {
  Field x;
  J3D_TRY(check_field_wide(a, -1, &x, "a"));
  if (x.ey > 65535 || x.ez > 65535) return fail(J3D_EINVAL, "fill: y/z extents above 65535");
  J3D_HIP(launch_fill_const(x.base, x.dtype, x.ex, x.ey, x.ez, x.sy, x.sz, value,
                            static_cast<hipStream_t>(stream)));
  return J3D_OK;
}

int j3d_bandwidth_probe(const double* src, double* dst, int64_t n, int32_t reps, double* gbps,
                        void* stream) {
  if (src == nullptr || dst == nullptr || gbps == nullptr || n < 2 || reps < 1)
    return fail(J3D_EINVAL, "bandwidth probe: bad arguments");
  if ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) % 16 != 0)
    return fail(J3D_EINVAL, "bandwidth probe: buffers must be 16-byte aligned");
  if ((src < dst && src + n > dst) || (dst < src && dst + n > src) || src == dst)
    return fail(J3D_EALIAS, "bandwidth probe: buffers overlap");
  hipStream_t st = static_cast<hipStream_t>(stream);
  hipEvent_t e0, e1;
  J3D_HIP(hipEventCreate(&e0));
  J3D_HIP(hipEventCreate(&e1));
  double best = 0.0;
  for (int v = 0; v < kCopyVariants; ++v) {
    J3D_HIP(launch_copy_variant(v, src, dst, n, st));  // warm-up
    for (int r = 0; r < reps; ++r) {
      J3D_HIP(hipEventRecord(e0, st));
      J3D_HIP(launch_copy_variant(v, src, dst, n, st));
      J3D_HIP(hipEventRecord(e1, st));
      J3D_HIP(hipEventSynchronize(e1));
      float ms = 0.f;
      J3D_HIP(hipEventElapsedTime(&ms, e0, e1));
      const double rate = 2.0 * 8.0 * (double)n / (ms * 1e-3) / 1e9;
      if (rate > best) best = rate;
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  *gbps = best;
  return J3D_OK;
}

int j3d_bandwidth_probe_triad(const double* a, const double* b, double* dst, int64_t n, int32_t reps,
                              double* gbps, void* stream) {
  if (a == nullptr || b == nullptr || dst == nullptr || gbps == nullptr || n < 2 || reps < 1)
    return fail(J3D_EINVAL, "triad probe: bad arguments");
  if ((reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b) | reinterpret_cast<uintptr_t>(dst)) % 16 != 0)
    return fail(J3D_EINVAL, "triad probe: buffers must be 16-byte aligned");
  auto overlap = [n](const double* x, const double* y) { return x < y + n && y < x + n; };
  if (overlap(a, dst) || overlap(b, dst)) return fail(J3D_EALIAS, "triad probe: dst overlaps a source");
  hipStream_t st = static_cast<hipStream_t>(stream);
  hipEvent_t e0, e1;
  J3D_HIP(hipEventCreate(&e0));
  J3D_HIP(hipEventCreate(&e1));
  double best = 0.0;
  for (int v = 0; v < kTriadVariants; ++v) {
    J3D_HIP(launch_triad_variant(v, a, b, dst, n, st));  // warm-up
    for (int r = 0; r < reps; ++r) {
      J3D_HIP(hipEventRecord(e0, st));
      J3D_HIP(launch_triad_variant(v, a, b, dst, n, st));
      J3D_HIP(hipEventRecord(e1, st));
      J3D_HIP(hipEventSynchronize(e1));
      float ms = 0.f;
      J3D_HIP(hipEventElapsedTime(&ms, e0, e1));
      const double rate = 3.0 * 8.0 * (double)n / (ms * 1e-3) / 1e9;
      if (rate > best) best = rate;
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  *gbps = best;
  return J3D_OK;
}

// sum and dot_product share one path: y == nullptr selects the sum.
static int reduce_vec(const double* x, const double* y, int64_t n, uint32_t flags, double* out, void* stream,
                      const char* what) {
  if (out == nullptr) return fail(J3D_EINVAL, "%s: out is a null pointer", what);
  if (n < 0) return fail(J3D_EINVAL, "%s: n must be >= 0", what);
  if ((flags & ~J3D_HOST_RESULT) != 0) return fail(J3D_EINVAL, "%s: unknown flags 0x%x", what, flags);
  if (n > 0 && x == nullptr) return fail(J3D_EINVAL, "%s: x is a null pointer", what);
  if ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(y) | reinterpret_cast<uintptr_t>(out)) % 8 != 0)
    return fail(J3D_EINVAL, "%s: pointers must be 8-byte aligned", what);
  const bool host = (flags & J3D_HOST_RESULT) != 0;
  if (!host && n > 0) {
    const bool in_x = out >= x && out < x + n;
    const bool in_y = y != nullptr && out >= y && out < y + n;
    if (in_x || in_y) return fail(J3D_EALIAS, "%s: out overlaps an input", what);
  }
  hipStream_t st = static_cast<hipStream_t>(stream);
  Scratch* s = nullptr;
  J3D_TRY(get_scratch(st, &s));
  J3D_TRY(ensure_partials(s, (size_t)sum_blocks(n) + kSumWaves));
  double* dst = host ? &s->ctl->value : out;
  J3D_HIP(launch_sum(x, y, n, s->partials, dst, st));
  if (host) {
    J3D_HIP(hipMemcpyAsync(&s->ctl_host->value, &s->ctl->value, sizeof(double), hipMemcpyDeviceToHost, st));
    J3D_HIP(hipStreamSynchronize(st));
    *out = s->ctl_host->value;
  }
  return J3D_OK;
}

int j3d_sum(const double* x, int64_t n, uint32_t flags, double* out, void* stream) {
  return reduce_vec(x, nullptr, n, flags, out, stream, "j3d_sum");
}

int j3d_dot(const double* x, const double* y, int64_t n, uint32_t flags, double* out, void* stream) {
  if (n > 0 && y == nullptr) return fail(J3D_EINVAL, "j3d_dot: y is a null pointer");
  return reduce_vec(x, y, n, flags, out, stream, "j3d_dot");
}

int j3d_release_cache(void) {
  release_batch_cache();
  return release_all_scratch();
}

}  // extern "C"
