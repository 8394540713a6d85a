// pw_advection / tracer_advection: the multi-field stencils standing in for
// the paper's pw-advection and tra-adv benchmarks (Sec. "Flang performance
// comparison": field counts and grid sizes only).
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>

#include "advect.h"
#include "runtime.h"

using namespace j3d;

namespace {

// A workgroup shape and what a step of its march costs (us) with j workgroups
// on a CU: h + g * j, at most `per_cu` of them.  Fitted to timed passes over
// nine grids from 64^3 to 1024 x 512 x 512; the shapes they choose are on
// average 3 % (tracer 4 %) and at worst 13 % (8 %) slower than the fastest of
// 60 (profiles/shape_estimates.md).  CUs: those of a whole card, which they
// were timed on.
constexpr int kCus = 256;
struct MarchShape {
  int ry, cols, rows;  // rows per thread; columns and rows a workgroup outputs
  int per_cu;
  double h, g;
  double extra;  // steps of a march beyond its planes
};
const MarchShape kPwShapes[] = {{2, 64, 8, 3, 0.2, 1.0, 2}, {4, 64, 16, 2, 0.0, 1.82, 2}};
const MarchShape kTracer3Shapes[] = {{3, 58, 8, 2, 0.32, 0.95, 5}, {4, 58, 28, 1, 2.8, 0.2, 5}};

// The shape and number of planes with the least estimated time: few planes
// where the grid would leave CUs idle otherwise, many where the planes that
// each chunk reads beyond its own cost more.
template <size_t N>
AdvectCfg march_shape(const MarchShape (&shapes)[N], const AdvArgs& a) {
  AdvectCfg best{};
  double least = 0.0;
  for (const MarchShape& s : shapes) {
    const long long tiles =
        ((a.nx + s.cols - 1LL) / s.cols) * ((a.ny + s.rows - 1LL) / s.rows);
    for (int planes = 4; planes <= 128; ++planes) {
      const int chunks = (a.nz + planes - 1) / planes;
      const long long per_cu = (tiles * chunks + kCus - 1) / kCus;
      const long long full = per_cu / s.per_cu, rest = per_cu % s.per_cu;
      const double t = (std::min(planes, a.nz) + s.extra) *
                       (full * (s.h + s.g * s.per_cu) + (rest ? s.h + s.g * rest : 0.0));
      if (best.ry == 0 || t < least) {
        least = t;
        best.ry = s.ry;
        best.planes = planes;
      }
    }
  }
  return best;
}

// J3D_ADVECT_TILE="ry,planes,nt[,pf]" overrides the momentum advection's and
// the single tracer step's tile shape (shape sweeps).
AdvectCfg advect_cfg_from_env(AdvectCfg c) {
  if (const char* e = std::getenv("J3D_ADVECT_TILE")) {
    AdvectCfg t{0, 0, 0, 0};
    const int n = std::sscanf(e, "%d,%d,%d,%d", &t.ry, &t.planes, &t.nt, &t.pf);
    if (n >= 3 && advect_cfg_supported(t)) c = t;
  }
  return c;
}

// Momentum advection: loads one plane ahead and nontemporal stores throughout
// (within 3 % of plain ones at every size).  Fixed tiles of 4 rows and 64
// planes took 106 us at 64^3 (now 7.2), 109 at 128^3 (22), 247 at 500 x 300 x
// 100 (155), the same at 256^3 and above.
AdvectCfg pw_cfg(const AdvArgs& a) {
  AdvectCfg c = march_shape(kPwShapes, a);
  c.nt = c.pf = 1;
  return advect_cfg_from_env(c);
}

// Single tracer step: rows and planes by the number of points (us per step
// with 8 rows and 64 planes / these: 64^3 188 / 6.0, 128^3 189 / 17.0, 256^3
// 228 / 159, 400^3 782 / 661, 1024 x 512 x 512 2449 / 2449).
AdvectCfg tracer_cfg(const AdvArgs& a) {
  const double pts = (double)a.nx * a.ny * a.nz;
  AdvectCfg c = pts < 1e6   ? AdvectCfg{2, 4, 1}
                : pts < 5e6 ? AdvectCfg{2, 8, 1}
                : pts < 3e7 ? AdvectCfg{4, 4, 1}
                : pts < 1e8 ? AdvectCfg{4, 20, 1}
                            : AdvectCfg{8, 64, 1};
  return advect_cfg_from_env(c);
}

// Every plane (interior and halo) of the field under 2^31 bytes.
bool plane_below_2gib(const Field& a) {
  return ((long long)(a.ey - 1) * a.sy + a.ex) * (long long)a.esize < (1LL << 31);
}

// Two-step tracer pass (planes of 2^31 bytes and more): 6 rows per thread, 64
// planes, nontemporal stores (fastest at 1024 x 512 x 512).
// J3D_TRACER2_TILE="ry,planes,nt" overrides it.
AdvectCfg tracer2_cfg() {
  AdvectCfg c{6, 64, 1};
  if (const char* e = std::getenv("J3D_TRACER2_TILE")) {
    AdvectCfg t{0, 0, 0};
    if (std::sscanf(e, "%d,%d,%d", &t.ry, &t.planes, &t.nt) == 3 && tracer2_cfg_supported(t)) c = t;
  }
  return c;
}

// Three-step tracer pass: by estimate, but 64 planes from 2^24 points on
// (fastest at 256^3, 400^3 and 1024 x 512 x 512 by 1 to 6 %); plain stores
// (the next pass reads the iterate) while the fields stay below 4 GB: 128^3
// 11.9 against 12.7 us per step, 400^3 263 against 266, 1024 x 512 x 512 1033
// against 1008.  J3D_TRACER3_TILE="ry,planes,nt" overrides it.
AdvectCfg tracer3_cfg(const AdvArgs& a) {
  const double pts = (double)a.nx * a.ny * a.nz;
  AdvectCfg c = pts < (double)(1 << 24) ? march_shape(kTracer3Shapes, a) : AdvectCfg{4, 64, 0};
  c.nt = pts * 48.0 >= 4e9;
  if (const char* e = std::getenv("J3D_TRACER3_TILE")) {
    AdvectCfg t{0, 0, 0};
    if (std::sscanf(e, "%d,%d,%d", &t.ry, &t.planes, &t.nt) == 3 && tracer3_cfg_supported(t)) c = t;
  }
  return c;
}

// Steps per pass of tracer_advection, 1, 2 or 3 (J3D_TRACER_STEPS_PER_PASS).
int tracer_steps_per_pass(const AdvArgs& a) {
  const char* e = std::getenv("J3D_TRACER_STEPS_PER_PASS");
  const int n = e != nullptr ? std::atoi(e) : 0;
  if (n == 1 || n == 2) return n;
  return a.buffer_ok ? 3 : 2;
}

int check_spacing(double d, const char* name) {
  if (!(std::isfinite(d) && d > 0.0)) return fail(J3D_EINVAL, "%s must be finite and > 0", name);
  return J3D_OK;
}

int check_same_layout(const Field& a, const Field& b, const char* an, const char* bn) {
  J3D_TRY(check_same_interior(a, b, an, bn));
  if (a.sy != b.sy || a.sz != b.sz)
    return fail(J3D_EINVAL, "%s strides (%lld, %lld) differ from %s strides (%lld, %lld)", an, a.sy, a.sz, bn,
                b.sy, b.sz);
  return J3D_OK;
}

}  // namespace

extern "C" int pw_advection(const j3d_array* u, const j3d_array* v, const j3d_array* w, j3d_array* su,
                            j3d_array* sv, j3d_array* sw, double dx, double dy, double dz,
                            void* stream) {
  const j3d_array* d[6] = {u, v, w, su, sv, sw};
  const char* names[6] = {"u", "v", "w", "su", "sv", "sw"};
  Field f[6];
  for (int q = 0; q < 6; ++q) J3D_TRY(check_field_wide(d[q], J3D_F64, &f[q], names[q]));
  for (int q = 1; q < 3; ++q) J3D_TRY(check_same_layout(f[0], f[q], names[0], names[q]));
  J3D_TRY(check_same_interior(f[0], f[3], names[0], names[3]));
  for (int q = 4; q < 6; ++q) J3D_TRY(check_same_layout(f[3], f[q], names[3], names[q]));
  J3D_TRY(check_spacing(dx, "dx"));
  J3D_TRY(check_spacing(dy, "dy"));
  J3D_TRY(check_spacing(dz, "dz"));
  for (int o = 3; o < 6; ++o)
    for (int q = 0; q < o; ++q)
      if (fields_overlap(f[o], f[q]))
        return fail(J3D_EALIAS, "%s overlaps %s", names[o], names[q]);
  AdvArgs a{};
  for (int q = 0; q < 3; ++q) {
    a.in[q] = reinterpret_cast<const double*>(f[q].base);
    a.out[q] = reinterpret_cast<double*>(f[3 + q].base);
  }
  a.nx = f[0].nx();
  a.ny = f[0].ny();
  a.nz = f[0].nz();
  a.siy = (int)f[0].sy;
  a.siz = f[0].sz;
  a.soy = (int)f[3].sy;
  a.soz = f[3].sz;
  a.cx = 0.25 / dx;
  a.cy = 0.25 / dy;
  a.cz = 0.25 / dz;
  a.buffer_ok = 1;
  for (int q = 0; q < 6; ++q)
    if (!plane_below_2gib(f[q])) a.buffer_ok = 0;
  J3D_HIP(launch_pw_advect(a, pw_cfg(a), static_cast<hipStream_t>(stream)));
  return J3D_OK;
}

extern "C" int tracer_advection(j3d_array* t_a, j3d_array* t_b, const j3d_array* u,
                                const j3d_array* v, const j3d_array* w, const j3d_array* r, int64_t niter,
                                void* stream) {
  const j3d_array* d[6] = {t_a, t_b, u, v, w, r};
  const char* names[6] = {"t_a", "t_b", "u", "v", "w", "r"};
  Field f[6];
  for (int q = 0; q < 6; ++q) J3D_TRY(check_field_wide(d[q], J3D_F64, &f[q], names[q]));
  for (int q = 1; q < 6; ++q) J3D_TRY(check_same_layout(f[0], f[q], names[0], names[q]));
  if (niter < 0) return fail(J3D_EINVAL, "niter must be >= 0");
  for (int o = 0; o < 2; ++o)
    for (int q = 0; q < 6; ++q)
      if (q != o && fields_overlap(f[o], f[q])) return fail(J3D_EALIAS, "%s overlaps %s", names[o], names[q]);
  AdvArgs a{};
  for (int q = 0; q < 4; ++q) a.in[q] = reinterpret_cast<const double*>(f[2 + q].base);
  a.nx = f[0].nx();
  a.ny = f[0].ny();
  a.nz = f[0].nz();
  a.siy = a.soy = (int)f[0].sy;
  a.siz = a.soz = f[0].sz;
  const AdvectCfg c1 = tracer_cfg(a);
  const AdvectCfg c2 = tracer2_cfg();
  const AdvectCfg c3 = tracer3_cfg(a);
  hipStream_t st = static_cast<hipStream_t>(stream);
  double* ta = reinterpret_cast<double*>(f[0].base);
  double* tb = reinterpret_cast<double*>(f[1].base);
  a.buffer_ok = 1;
  for (int q = 0; q < 6; ++q)
    if (!plane_below_2gib(f[q])) a.buffer_ok = 0;
  // Launches of `per` steps, then single ones.  Every launch swaps the
  // arrays, so the number of launches keeps the parity of niter (a pass of
  // two steps is split in two when it would not) and the result is in t_a
  // exactly when niter is even.
  const int per = tracer_steps_per_pass(a);
  int64_t nl = niter / per, n1 = niter % per;
  if (((nl + n1) & 1) != (niter & 1)) {
    nl -= 1;
    n1 += per;
  }
  bool from_a = true;
  for (int64_t q = 0; q < nl + n1; ++q) {
    a.t = from_a ? ta : tb;
    a.out[0] = from_a ? tb : ta;
    if (q >= nl || per == 1)
      J3D_HIP(launch_tracer_advect(a, c1, st));
    else if (per == 2)
      J3D_HIP(launch_tracer2_advect(a, c2, st));
    else
      J3D_HIP(launch_tracer3_advect(a, c3, st));
    from_a = !from_a;
  }
  return J3D_OK;
}
