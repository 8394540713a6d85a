// The paper's 2D jacobi benchmark on gfx950: Jacobi iteration for Laplace's
// equation on a 2D grid u(0:nx+1, 0:ny+1) with the boundary values in the
// halo (Sec. "Flang performance comparison": 1024 x 1024, 100000
// iterations),
//   u'(i,j) = (((u(i-1,j) + u(i+1,j)) + u(i,j-1)) + u(i,j+1)) / 4,
// T sweeps per launch.
//
// The grid is small (8 MB per FP64 array at 1024^2) and stays in the caches,
// so a sweep costs little more than a launch: the kernel does T sweeps per
// launch, each wavefront on an independent tile held in registers.  Lane l,
// register r of a wavefront holds cell (x0 - T + l, y0 - T + r) of a 64 x R
// tile.  A sweep updates the tile's interior cells in place, rolling down the
// rows (the old value of the row above is kept in a temporary): x-neighbours
// come from the adjacent lanes (DPP wave shifts), y-neighbours from the
// registers of the rows above and below.  A cell whose neighbour lies outside
// the tile takes a wrong value, and a wrong value travels one cell per sweep,
// so after T sweeps the inner (64 - 2T) x (R - 2T) cells are exact: those are
// stored.  Tiles overlap by 2T columns and rows; there is no LDS and no
// barrier.  Halo cells, and the clamped cells beyond the halo, are never
// updated.  Each cell is computed with exactly the arithmetic above, so T
// sweeps per launch equal T single sweeps bit for bit.
#include <cstdlib>

#include "sweep.h"

namespace j3d {
namespace {

using sweep_detail::from_left;
using sweep_detail::from_right;
using sweep_detail::shift_in_left;
using sweep_detail::shift_in_right;
using sweep_detail::WAVE;

constexpr int kWavesPerBlock = 4;

template <int T, int R>
__global__ void __launch_bounds__(WAVE * kWavesPerBlock)
    k_jacobi2d(const double* __restrict__ in, double* __restrict__ out, int nx, int ny, int si, int so,
               int tiles_x, int ntiles, const int* __restrict__ done) {
  static_assert(2 * T < WAVE && 2 * T < R, "a tile needs inner cells");
  constexpr int W = WAVE - 2 * T;
  constexpr int H = R - 2 * T;
  if (done != nullptr && *done != 0) return;
  const int lane = threadIdx.x & (WAVE - 1);
  const int tile = blockIdx.x * kWavesPerBlock + (threadIdx.x / WAVE);
  if (tile >= ntiles) return;  // the whole wavefront leaves together
  const int tx = tile % tiles_x;
  const int ty = tile / tiles_x;
  const int x = tx * W + 1 - T + lane;  // column of this lane
  const int y0 = ty * H + 1 - T;        // row of register 0
  const int xc = min(max(x, 0), nx + 1);
  const bool x_in = x >= 1 && x <= nx;
  double v[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int yc = min(max(y0 + r, 0), ny + 1);
    v[r] = in[xc + si * yc];
  }
#pragma unroll
  for (int s = 0; s < T; ++s) {
    double above = v[0];  // old value of the row above (row 0: none in the tile)
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const double left = from_left(v[r]);
      const double right = from_right(v[r]);
      const double below = r + 1 < R ? v[r + 1] : v[r];
      double t = left + right;
      t = t + above;
      t = t + below;
      const double nv = t / 4.0;
      const int y = y0 + r;
      above = v[r];
      v[r] = (x_in && y >= 1 && y <= ny) ? nv : v[r];
    }
  }
  const bool lane_out = lane >= T && lane < T + W && x_in;
#pragma unroll
  for (int r = T; r < T + H; ++r) {
    const int y = y0 + r;
    if (lane_out && y >= 1 && y <= ny) out[x + so * y] = v[r];
  }
}

// T sweeps per launch by a workgroup of BY wavefronts stacked in y, each
// holding R rows of a 64-column tile in registers (lane l, register r is
// cell (x0 - T + l, y0 - T + wy*R + r)).  Before every sweep each wavefront
// publishes its first and last row in LDS (two parity slots, one barrier
// per sweep), and the rows just outside its own are the neighbours' values
// of the previous sweep, so only the workgroup's outer T rows and the
// wavefront's outer T columns hold wrong values after T sweeps: the inner
// (64 - 2T) x (BY*R - 2T) cells are stored.  Same arithmetic per cell as
// k_jacobi2d.
template <int T, int R, int BY>
__global__ void __launch_bounds__(WAVE * BY)
    k_jacobi2d_wg(const double* __restrict__ in, double* __restrict__ out, int nx, int ny, int si, int so,
                  int tiles_x, const int* __restrict__ done) {
  constexpr int W = WAVE - 2 * T;
  constexpr int H = BY * R - 2 * T;
  static_assert(2 * T < WAVE && H > 0, "a tile needs inner cells");
  __shared__ double edge[2][BY][2][WAVE];
  if (done != nullptr && *done != 0) return;  // uniform over the launch
  const int lane = threadIdx.x & (WAVE - 1);
  const int wy = threadIdx.x / WAVE;
  const int tx = blockIdx.x % tiles_x;
  const int ty = blockIdx.x / tiles_x;
  const int x = tx * W + 1 - T + lane;
  const int y0 = ty * H + 1 - T + wy * R;  // row of register 0
  const int xc = min(max(x, 0), nx + 1);
  const bool x_in = x >= 1 && x <= nx;
  double v[R];
#pragma unroll
  for (int r = 0; r < R; ++r) v[r] = in[xc + si * min(max(y0 + r, 0), ny + 1)];
#pragma unroll
  for (int s = 0; s < T; ++s) {
    edge[s & 1][wy][0][lane] = v[0];
    edge[s & 1][wy][1][lane] = v[R - 1];
    __syncthreads();
    const double lo = wy > 0 ? edge[s & 1][wy - 1][1][lane] : v[0];      // row y0 - 1, old
    const double hi = wy < BY - 1 ? edge[s & 1][wy + 1][0][lane] : v[R - 1];  // row y0 + R, old
    double above = lo;  // old value of the row below index r (y - 1)
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const double left = from_left(v[r]);
      const double right = from_right(v[r]);
      const double below = r + 1 < R ? v[r + 1] : hi;
      double t = left + right;
      t = t + above;
      t = t + below;
      const double nv = t / 4.0;
      const int y = y0 + r;
      above = v[r];
      v[r] = (x_in && y >= 1 && y <= ny) ? nv : v[r];
    }
  }
  const bool lane_out = lane >= T && lane < T + W && x_in;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int br = wy * R + r;
    const int y = y0 + r;
    if (lane_out && br >= T && br < T + H && y >= 1 && y <= ny) out[x + so * y] = v[r];
  }
}

// T sweeps per launch (T even) with two columns per lane: a workgroup of BY
// wavefronts of R rows holds a 128 x (BY*R) tile in registers (lane l,
// register r, c is cell (x0 + 2l + c, y0 + wy*R + r), x0 = 1 + W tx - T).
// The pair's inner x-neighbours are its own registers, so a cell takes one
// lane shift where one column per lane takes two, and a tile twice as wide
// wastes less on its 2T overlapping columns, which is what lets T be 16.
// Each sweep forms the new rows beside the old ones, publishes the first
// and last of them and meets one barrier; a cell is six vector
// instructions.  The inner (128 - 2T) x (BY*R - 2T) cells are stored.
//
// Cells outside the interior keep their values.  One workgroup per CU runs
// in step, so the slowest tile sets the launch's time, and only what a tile
// needs is selected: XM has bit c set if cells c of the pairs hold a halo
// column (0 for tiles inside), ROWS if the wavefront holds rows outside the
// interior.  Each XCD takes a contiguous run of tiles, whose overlaps then
// meet in its L2.
//
// At 1024^2 a 16-sweep launch takes 14.3 us (0.90 us per sweep; 1.59 with
// 8-sweep launches of one column per lane): about 3 us to start and finish,
// 0.6 us per sweep of 16 wavefronts x 5 rows (0.44 of it vector issue), and
// the rest the loads (16.4 us per launch without the XCD runs; 17 with every
// tile selecting every cell).
template <int T, int R, int BY, int XM, bool ROWS>
__device__ __forceinline__ void jacobi2d_pair_sweeps(double (&v)[R][2], const bool (&x_in)[2], int y0, int ny,
                                                     int lane, int wy, double (&edge)[2][BY][2][2][WAVE]) {
  const int wdn = max(wy - 1, 0), wup = min(wy + 1, BY - 1);
  auto publish = [&](int slot, const double(&a)[R][2]) {
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      edge[slot][wy][0][c][lane] = a[0][c];
      edge[slot][wy][1][c][lane] = a[R - 1][c];
    }
  };
  // one sweep from a to b, with the neighbours' edge rows of `slot`; the
  // inner rows first, which do not wait for them
  auto sweep = [&](int slot, const double(&a)[R][2], double(&b)[R][2]) {
    double lo[2], hi[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      lo[c] = edge[slot][wdn][1][c][lane];
      hi[c] = edge[slot][wup][0][c][lane];
    }
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int r = q + 1 < R ? q + 1 : 0;  // 1 .. R-1, then 0
      const double left = shift_in_left(a[r][1]), right = shift_in_right(a[r][0]);
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        double t = c == 0 ? left + a[r][1] : a[r][0] + right;
        t = t + (r == 0 ? lo[c] : a[r - 1][c]);
        t = t + (r == R - 1 ? hi[c] : a[r + 1][c]);
        const double nv = t / 4.0;
        bool in = true;
        if ((XM >> c) & 1) in = in & x_in[c];
        if (ROWS) in = in & (y0 + r >= 1) & (y0 + r <= ny);
        b[r][c] = in ? nv : a[r][c];
      }
    }
  };
  double w[R][2];
  publish(0, v);
  __syncthreads();
  for (int s = 0; s < T; s += 2) {
    sweep(0, v, w);
    publish(1, w);
    __syncthreads();
    sweep(1, w, v);
    if (s + 2 < T) {
      publish(0, v);
      __syncthreads();
    }
  }
}

template <int T, int R, int BY>
__global__ void __launch_bounds__(WAVE * BY)
    k_jacobi2d_pair(const double* __restrict__ in, double* __restrict__ out, int nx, int ny, int si, int so,
                    int tiles_x, const int* __restrict__ done) {
  constexpr int W = 2 * WAVE - 2 * T;
  constexpr int H = BY * R - 2 * T;
  static_assert(T % 2 == 0 && W > 0 && H > 0 && R >= 2, "a tile needs inner cells");
  __shared__ double edge[2][BY][2][2][WAVE];
  if (done != nullptr && *done != 0) return;  // uniform over the launch
  const int lane = threadIdx.x & (WAVE - 1);
  const int wy = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  const int tile = sweep_detail::xcd_remap(blockIdx.x, gridDim.x);
  const int tx = tile % tiles_x;
  const int ty = tile / tiles_x;
  const int x0 = tx * W + 1 - T;           // the tile's first column (odd)
  const int x = x0 + 2 * lane;             // column of the pair's first cell
  const int y0 = ty * H + 1 - T + wy * R;  // row of register 0
  // A wavefront with no row in 0 .. ny+1 feeds nothing: the halo rows keep
  // their values whatever lies beyond.  It only takes its part in the
  // barriers (one before each sweep).
  if (y0 + R - 1 < 0 || y0 > ny + 1) {
    for (int s = 0; s < T; ++s) __syncthreads();
    return;
  }
  const int xc[2] = {min(max(x, 0), nx + 1), min(max(x + 1, 0), nx + 1)};
  const bool x_in[2] = {x >= 1 && x <= nx, x + 1 >= 1 && x + 1 <= nx};
  double v[R][2];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const long long row = (long long)si * min(max(y0 + r, 0), ny + 1);
    v[r][0] = in[row + xc[0]];
    v[r][1] = in[row + xc[1]];
  }
  // halo columns in the tile: column 0 is the second cell of a pair, column
  // nx + 1 the first when nx is even; beyond them nothing is needed
  const bool has_lo = x0 <= 0, has_hi = x0 + 2 * WAVE - 1 >= nx + 1;
  const int xm = (has_lo ? 2 : 0) | (has_hi ? ((nx & 1) == 0 ? 1 : 2) : 0);
  if (y0 < 1 || y0 + R - 1 > ny || xm == 3)
    jacobi2d_pair_sweeps<T, R, BY, 3, true>(v, x_in, y0, ny, lane, wy, edge);
  else if (xm == 0)
    jacobi2d_pair_sweeps<T, R, BY, 0, false>(v, x_in, y0, ny, lane, wy, edge);
  else if (xm == 1)
    jacobi2d_pair_sweeps<T, R, BY, 1, false>(v, x_in, y0, ny, lane, wy, edge);
  else
    jacobi2d_pair_sweeps<T, R, BY, 2, false>(v, x_in, y0, ny, lane, wy, edge);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int br = wy * R + r;
    const int y = y0 + r;
    if (br < T || br >= T + H || y < 1 || y > ny) continue;
    double* o = out + (long long)so * y + x;
#pragma unroll
    for (int c = 0; c < 2; ++c)
      if (2 * lane + c >= T && 2 * lane + c < T + W && x_in[c]) o[c] = v[r][c];
  }
}

template <int T, int R, int BY>
hipError_t go2d_pair(const double* in, double* out, int nx, int ny, int si, int so, const int* done,
                     hipStream_t st) {
  constexpr int W = 2 * WAVE - 2 * T;
  constexpr int H = BY * R - 2 * T;
  const int tx = (nx + W - 1) / W;
  const int ty = (ny + H - 1) / H;
  hipLaunchKernelGGL((k_jacobi2d_pair<T, R, BY>), dim3(tx * ty), dim3(WAVE * BY), 0, st, in, out, nx, ny, si, so,
                     tx, done);
  return hipGetLastError();
}

template <int T, int R, int BY>
hipError_t go2d_wg(const double* in, double* out, int nx, int ny, int si, int so, const int* done,
                   hipStream_t st) {
  constexpr int W = WAVE - 2 * T;
  constexpr int H = BY * R - 2 * T;
  const int tx = (nx + W - 1) / W;
  const int ty = (ny + H - 1) / H;
  hipLaunchKernelGGL((k_jacobi2d_wg<T, R, BY>), dim3(tx * ty), dim3(WAVE * BY), 0, st, in, out, nx, ny, si, so,
                     tx, done);
  return hipGetLastError();
}

// Sum of r^2 with r = (S - 4 u) / h^2 over one block of rows: thread q of
// the block takes columns q, q + 256, ... of each row in order; wave
// butterfly, wave-ordered sum, fixed slot per block.
constexpr int kResRows = 8;

__global__ void __launch_bounds__(256)
    k_laplace2d_res(const double* __restrict__ u, int nx, int ny, int su, double h2,
                    double* __restrict__ partials) {
  __shared__ double red[256 / WAVE];
  double acc = 0.0;
  const int j0 = 1 + blockIdx.x * kResRows;
  for (int j = j0; j < min(j0 + kResRows, ny + 1); ++j)
    for (int i = 1 + (int)threadIdx.x; i <= nx; i += 256) {
      const double* p = u + i + su * j;
      double t = p[-1] + p[1];
      t = t + p[-su];
      t = t + p[su];
      const double r = (t - 4.0 * p[0]) / h2;
      acc += r * r;
    }
  acc = sweep_detail::wave_sum(acc);
  if ((threadIdx.x & (WAVE - 1)) == 0) red[threadIdx.x / WAVE] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double tot = red[0];
#pragma unroll
    for (int w = 1; w < 256 / WAVE; ++w) tot += red[w];
    partials[blockIdx.x] = tot;
  }
}

template <int T, int R>
hipError_t go2d(const double* in, double* out, int nx, int ny, int si, int so, const int* done,
                hipStream_t st) {
  constexpr int W = WAVE - 2 * T;
  constexpr int H = R - 2 * T;
  const int tx = (nx + W - 1) / W;
  const int ty = (ny + H - 1) / H;
  const int ntiles = tx * ty;
  const int blocks = (ntiles + kWavesPerBlock - 1) / kWavesPerBlock;
  hipLaunchKernelGGL((k_jacobi2d<T, R>), dim3(blocks), dim3(WAVE * kWavesPerBlock), 0, st, in, out, nx, ny,
                     si, so, tx, ntiles, done);
  return hipGetLastError();
}

}  // namespace

// Tiles of a launch of T sweeps by workgroups of BY wavefronts of R rows
// with two columns per lane.
static int pair_tiles(int T, int R, int BY, int nx, int ny) {
  const int w = 2 * WAVE - 2 * T, h = BY * R - 2 * T;
  const long long n = (long long)((nx + w - 1) / w) * ((ny + h - 1) / h);
  return n < (1 << 30) ? (int)n : (1 << 30);
}

// Shape of the 8-sweep launches forced by J3D_JACOBI2D_SHAPE (shape sweeps;
// then no launch takes 16): 0 one wavefront per 64 x 32 tile; 1..8
// workgroups of wavefronts stacked in y exchanging edge rows through LDS
// (wavefronts x rows each: 1: 4 x 16, 2: 8 x 8, 3: 8 x 16, 4: 4 x 12,
// 5: 8 x 10, 6: 16 x 6, 7: 16 x 8, 8: 16 x 4).  -1: not forced.
static int jacobi2d_forced_shape() {
  if (const char* e = std::getenv("J3D_JACOBI2D_SHAPE")) {
    const int v = std::atoi(e);
    if (v >= 0 && v <= 8) return v;
  }
  return -1;
}

// Sweeps per launch of a long run.  One workgroup of a 16-sweep launch fills
// a CU (16 wavefronts), so as long as the tiles of the largest 16-sweep
// shape (5 rows per wavefront: 96 x 48 outputs) fit one round of the CUs, a
// launch costs 3 us and 0.4-0.7 us per sweep, and 16 sweeps per launch win
// (us per sweep, 16 against 8 with the shapes below: 1024^2 0.90 / 1.10,
// 700 x 600 0.71 / 0.97, 300 x 400 0.58 / 0.83).  In more than one round the
// cells recomputed at the tiles' edges cost more than the launches saved
// (1500 x 1300: 1.60 / 1.51, 2048^2: 3.08 / 2.62).
int jacobi2d_sweeps_per_launch(int nx, int ny) {
  if (jacobi2d_forced_shape() >= 0) return 8;
  return pair_tiles(16, 5, 16, nx, ny) <= sweep_detail::device_cus() ? 16 : 8;
}

hipError_t launch_jacobi2d(int sweeps, const double* in, double* out, int nx, int ny, int si, int so,
                           const int* done, hipStream_t st) {
  const int cus = sweep_detail::device_cus();
  switch (sweeps) {
    case 1: return go2d<1, 16>(in, out, nx, ny, si, so, done, st);
    case 2: return go2d<2, 16>(in, out, nx, ny, si, so, done, st);
    case 4: return go2d<4, 24>(in, out, nx, ny, si, so, done, st);
    case 8:
      switch (jacobi2d_forced_shape()) {
        case 0: return go2d<8, 32>(in, out, nx, ny, si, so, done, st);
        case 1: return go2d_wg<8, 16, 4>(in, out, nx, ny, si, so, done, st);
        case 2: return go2d_wg<8, 8, 8>(in, out, nx, ny, si, so, done, st);
        case 3: return go2d_wg<8, 16, 8>(in, out, nx, ny, si, so, done, st);
        case 4: return go2d_wg<8, 12, 4>(in, out, nx, ny, si, so, done, st);
        case 5: return go2d_wg<8, 10, 8>(in, out, nx, ny, si, so, done, st);
        case 6: return go2d_wg<8, 6, 16>(in, out, nx, ny, si, so, done, st);
        case 7: return go2d_wg<8, 8, 16>(in, out, nx, ny, si, so, done, st);
        case 8: return go2d_wg<8, 4, 16>(in, out, nx, ny, si, so, done, st);
        default: break;
      }
      // us per launch, one column per lane (8 x 8) / two (16 x 4) / two (8 x
      // 7): 300 x 400 6.6 / 7.3 / 7.5, 700 x 600 7.9 / 7.7 / 7.8, 1024^2
      // 12.8 / 8.8 / 10.4, 1500 x 1300 18.0 / 12.6 / 12.0, 2048^2 29.8 /
      // 21.3 / 21.0
      if (pair_tiles(8, 4, 16, nx, ny) < cus / 4) return go2d_wg<8, 8, 8>(in, out, nx, ny, si, so, done, st);
      if (pair_tiles(8, 4, 16, nx, ny) <= cus) return go2d_pair<8, 4, 16>(in, out, nx, ny, si, so, done, st);
      return go2d_pair<8, 7, 8>(in, out, nx, ny, si, so, done, st);
    case 16:
      // the fewest rows per wavefront whose tiles still fit one round
      if (pair_tiles(16, 3, 16, nx, ny) <= cus) return go2d_pair<16, 3, 16>(in, out, nx, ny, si, so, done, st);
      if (pair_tiles(16, 4, 16, nx, ny) <= cus) return go2d_pair<16, 4, 16>(in, out, nx, ny, si, so, done, st);
      return go2d_pair<16, 5, 16>(in, out, nx, ny, si, so, done, st);
    default: return hipErrorInvalidValue;
  }
}

int laplace2d_res_blocks(int ny) { return (ny + kResRows - 1) / kResRows; }

hipError_t launch_laplace2d_res(const double* u, int nx, int ny, int su, double h, double* partials,
                                hipStream_t st) {
  hipLaunchKernelGGL(k_laplace2d_res, dim3(laplace2d_res_blocks(ny)), dim3(256), 0, st, u, nx, ny, su, h * h,
                     partials);
  return hipGetLastError();
}

}  // namespace j3d
