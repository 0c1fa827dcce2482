// Weighted-Jacobi / Chebyshev sweeps of the compact 7-point
// pressure-correction operator (paper Sec. 2.4 and App. A), one sweep per
// launch.
//
// The point update is les_sweep.h's, so the iterates of every kernel are
// bitwise equal.
//
// One sweep: each thread owns one column of the tile and marches up z
// with the vertical neighbours in registers; x neighbours come from the
// adjacent lanes of the wavefront, y neighbours through the L1/L2 caches.
// 16 bytes per cell (Chebyshev: phi, prev, rhs in, phi' out).  Grids at
// least 256 cells wide take 256-cell-wide tiles (four waves side by side):
// 256 x 2 while the four arrays fit the 256 MB Infinity Cache, 256 x 4
// beyond it, where the arrays read once per sweep (prev, rhs) and the
// output are streamed with non-temporal accesses so the caches keep the
// iterate's neighbour rows.  Narrower grids take 64 x 4 (or 64 x 16
// streamed, 64 x 1 for ny < 4) tiles.
//
// Walls: the z neighbour of the bottom/top level is that level itself (even
// mirror); x and y are periodic.
#include "les_column.h"
#include "les_sweep.h"

namespace lesmi {

namespace {

// Logical tile of physical block b.  Workgroups go to the 8 XCDs
// round-robin (b mod 8); each XCD gets one contiguous range of tiles
// (x fastest, then y, then z chunk), so the y halos a tile reads were
// fetched into the same L2 by its neighbours.
__device__ __forceinline__ int xcd_tile(int b, int nblocks) {
  const int per = nblocks >> 3;  // nblocks is a multiple of 8
  return (b & 7) * per + (b >> 3);
}

template <typename T>
struct SweepArgs {
  Grid g;
  SweepCoef k;
  int kc, tiles_x, tiles_y, tiles_z, ntiles;
  double wc0;        // Chebyshev weight
  const T *cur, *prev, *rhs;
  T *out;
  SolveCtl *ctl;
  double *partials;
  // a pending residual check (sweep dec_m >= 0) of an
  // earlier launch whose dec_np block partials block 0 reduces and decides
  const double *dec_partials;
  int dec_np, dec_m;
  // host-visible word written after that decision (device view of pinned
  // host memory; nullable): decision number snap_seq in the high half, the
  // control block's `done` in the low half, one 64-bit store
  int64_t *snap;
  int snap_seq;
};

struct TileIdx {
  int tx, ty, k0, k1;
};

__device__ __forceinline__ TileIdx tile_of(int tile, int tiles_x, int tiles_y, int kc, int nz) {
  TileIdx t;
  t.tx = tile % tiles_x;
  const int rest = tile / tiles_x;
  t.ty = rest % tiles_y;
  t.k0 = (rest / tiles_y) * kc;
  t.k1 = min(nz, t.k0 + kc);
  return t;
}

// ---------------------------------------------------------------- 1 sweep

constexpr int kTY1 = 4;       // cache-resident arrays
constexpr int kTY1Big = 16;   // streamed arrays
// Grids at least kWideNx wide take tiles of kWX waves side by side along x
// (256-cell rows): longer contiguous runs per plane row and fewer halo
// planes per cell; kWideTY rows when cache-resident, kWideTYBig streamed.
constexpr int kWideNx = 256, kWX = 4, kWideTY = 2, kWideTYBig = 4;

template <typename T>
__device__ __forceinline__ T ld_stream(const T *p, bool nt) {
  return nt ? __builtin_nontemporal_load(p) : *p;
}

// z-march of one 64-cell row (one wave) of a tile over levels [k0, k1):
// one Chebyshev (or, CHEB = false, weighted-Jacobi) sweep of each cell,
// returning its FP64 residual sum when CHECK.  SHIFT: the x neighbours of a
// cell are the iterate values its neighbouring lanes already hold (DPP wave
// shifts) and only the row's end lanes load theirs, so each plane row is
// read once; otherwise they are loaded.  FULL: all 64 cells of the row lie
// inside the grid, so no lane is predicated off (a predicated store makes
// the compiler wait for that store before the next level); a ragged row's
// lanes beyond nx march on the row's last cell, for the shifts, but neither
// store nor count in the residual.
template <bool FULL, bool SHIFT, bool CHEB, bool CHECK, bool NT, typename T>
__device__ __forceinline__ double march_row(const SweepArgs<T> &a, const TileIdx &t, int lane,
                                            int i, int j) {
  const Grid &g = a.g;
  const bool valid = FULL || i < g.nx;
  const int ic = valid ? i : g.nx - 1;
  const int ip = ic + 1 == g.nx ? 0 : ic + 1, im = ic == 0 ? g.nx - 1 : ic - 1;
  const int jp = j + 1 == g.ny ? 0 : j + 1, jm = j == 0 ? g.ny - 1 : j - 1;
  const int64_t col = (int64_t)ic + (int64_t)g.nx * j;
  const int64_t oxp = ip - ic, oxm = im - ic;
  const int64_t oyp = (int64_t)(jp - j) * g.nx, oym = (int64_t)(jm - j) * g.nx;
  const bool load_xp = lane == 63 || ic + 1 >= g.nx, load_xm = lane == 0;
  double acc = 0.0;
  T below = a.cur[col + g.nxy * (t.k0 > 0 ? t.k0 - 1 : 0)];
  T c = a.cur[col + g.nxy * t.k0];
  for (int k = t.k0; k < t.k1; ++k) {
    const int64_t q = col + g.nxy * k;
    const T above = a.cur[q + (k + 1 < g.nz ? g.nxy : 0)];
    T xp, xm;
    if (SHIFT) {
      xp = lane_shift<1>(c);
      xm = lane_shift<-1>(c);
      if (load_xp) xp = a.cur[q + oxp];
      if (load_xm) xm = a.cur[q + oxm];
    } else {
      xp = a.cur[q + oxp];
      xm = a.cur[q + oxm];
    }
    const double hx = (double)xp + (double)xm;
    const double hy = (double)a.cur[q + oyp] + (double)a.cur[q + oym];
    const double hz = (double)above + (double)below;
    const double res =
        point_residual(a.k, (double)c, hx, hy, hz, (double)ld_stream(&a.rhs[q], NT));
    if (CHECK && valid) acc += res * res;
    const double pv = CHEB ? (double)ld_stream(&a.prev[q], NT) : 0.0;
    const T out = (T)point_update(a.k, (double)c, res, CHEB, pv, a.wc0);
    if (valid) {
      if (NT)
        __builtin_nontemporal_store(out, &a.out[q]);
      else
        a.out[q] = out;
    }
    below = c;
    c = above;
  }
  return acc;
}

// A 64 WX x TY tile: wave (wx, wy) owns the 64 cells of row ty TY + wy
// starting at x = tx 64 WX + 64 wx.  The first sweep of a solve (weight 1,
// no previous iterate) launches as CHEB = false.  Lane shifts only in
// blocks of several waves: one-wave blocks (two-dimensional grids, few waves
// per CU) measured faster with loaded x neighbours.
template <typename T, int WX, int TY, bool CHEB, bool CHECK, bool NT>
__global__ __launch_bounds__(64 * WX * TY) void sweep1_kernel(SweepArgs<T> a) {
  if (a.ctl->done) {  // stopped: a deciding launch still leaves its word
    if (a.snap && blockIdx.x == 0 && threadIdx.x == 0)
      *(volatile int64_t *)a.snap = ((int64_t)a.snap_seq << 32) | (uint32_t)a.ctl->done;
    return;
  }
  const Grid &g = a.g;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  double acc = 0.0;
  if (tile < a.ntiles) {
    const TileIdx t = tile_of(tile, a.tiles_x, a.tiles_y, a.kc, g.nz);
    const int lane = (int)(threadIdx.x & 63), wave = (int)(threadIdx.x >> 6);
    const int x0 = t.tx * 64 * WX + (wave % WX) * 64;
    const int i = x0 + lane;
    const int j = t.ty * TY + wave / WX;
    constexpr bool kShift = WX * TY > 1;
    if (j < g.ny && x0 < g.nx) {  // uniform per wave
      // Streamed (HBM-bound) sweeps on 64-wide tiles keep the predicated
      // march for full rows too: its wait on each level's store measured
      // faster there.
      if ((!NT || WX > 1) && x0 + 64 <= g.nx)  // uniform per wave
        acc = march_row<true, kShift, CHEB, CHECK, NT>(a, t, lane, i, j);
      else
        acc = march_row<false, kShift, CHEB, CHECK, NT>(a, t, lane, i, j);
    }
  }
  if (a.dec_m >= 0 && blockIdx.x == 0 && threadIdx.x < 64) {
    // The residual test of an earlier checking launch, decided here by one
    // wave after its row instead of by a launch of its own: its partials are
    // complete at this launch's start.  The other blocks sweep regardless;
    // their outputs go to buffers that hold neither the tested iterate nor
    // this launch's input, and the next launch sees the decision.
    double t = 0.0;
#pragma unroll 16
    for (int q = (int)threadIdx.x; q < a.dec_np; q += 64) t += a.dec_partials[q];
    t = wave_sum(t);
    if (threadIdx.x == 0) {
      check_decision(a.ctl, t, a.dec_m);
      if (a.snap)
        *(volatile int64_t *)a.snap = ((int64_t)a.snap_seq << 32) | (uint32_t)a.ctl->done;
    }
  }
  if (CHECK) {
    const double s = block_sum(acc);
    if (threadIdx.x == 0) a.partials[blockIdx.x] = s;
  }
}

struct Shape {
  int kc, tiles_x, tiles_y, tiles_z, ntiles, blocks;
  int wx, ty;   // waves along x, tile rows
  bool stream;  // streamed arrays
};

// The four arrays of a sweep exceed what the Infinity Cache keeps.
bool streamed(const Grid &g, bool is_double) {
  return 4.0 * (double)g.n * (is_double ? 8.0 : 4.0) > 192.0e6;
}

Shape shape_of(const Grid &g, bool is_double) {
  Shape sh;
  sh.stream = streamed(g, is_double);
  sh.wx = 1;
  if (g.nx >= kWideNx && g.ny >= kWideTYBig) {
    sh.wx = kWX;
    sh.ty = sh.stream ? kWideTYBig : kWideTY;
  } else {
    // rows beyond ny would idle: a short y axis (a two-dimensional run has
    // ny = 1) takes the next smaller tile
    sh.ty = sh.stream ? kTY1Big : kTY1;
    if (g.ny < sh.ty) sh.ty = g.ny < kTY1 ? 1 : kTY1;
  }
  sh.tiles_x = (g.nx + 64 * sh.wx - 1) / (64 * sh.wx);
  sh.tiles_y = (g.ny + sh.ty - 1) / sh.ty;
  const int64_t cols = (int64_t)sh.tiles_x * sh.tiles_y;
  // z chunks: long enough to amortise the halo planes, short enough for
  // several blocks per CU.  Wide tiles aim at a wave count: the 8192 waves
  // that fill the chip once when cache-resident, eight times that when
  // streamed (shorter chunks measured faster there).
  sh.kc = g.nz;
  const int target = sh.wx > 1 ? (sh.stream ? 65536 : 8192) / (sh.wx * sh.ty) : 2048;
  while (sh.kc > 8 && cols * ((g.nz + sh.kc - 1) / sh.kc) < target) sh.kc = (sh.kc + 1) / 2;
  sh.tiles_z = (g.nz + sh.kc - 1) / sh.kc;
  int64_t nt = cols * sh.tiles_z;
  while (nt > kPartials) {
    sh.kc *= 2;
    sh.tiles_z = (g.nz + sh.kc - 1) / sh.kc;
    nt = cols * sh.tiles_z;
  }
  sh.ntiles = (int)nt;
  sh.blocks = (sh.ntiles + 7) / 8 * 8;
  return sh;
}

}  // namespace

int tsweep_blocks(const Grid &g, bool is_double) { return shape_of(g, is_double).blocks; }

template <typename T>
void launch_tsweep(const Grid &g, bool chebyshev, bool check, bool first, double omega_jacobi,
                   double omega_cheb, const T *cur, const T *prev, T *out, const T *rhs,
                   SolveCtl *ctl, double *partials, const double *dec_partials, int dec_np,
                   int dec_m, int64_t *snap, int snap_seq, hipStream_t s) {
  const Shape sh = shape_of(g, sizeof(T) == 8);
  SweepArgs<T> a;
  a.g = g;
  a.k = sweep_coef(g, omega_jacobi);
  a.kc = sh.kc;
  a.tiles_x = sh.tiles_x;
  a.tiles_y = sh.tiles_y;
  a.tiles_z = sh.tiles_z;
  a.ntiles = sh.ntiles;
  a.wc0 = omega_cheb;
  a.cur = cur;
  a.prev = prev;
  a.rhs = rhs;
  a.out = out;
  a.ctl = ctl;
  a.partials = partials;
  a.dec_partials = dec_partials;
  a.dec_np = dec_np;
  a.dec_m = dec_m;
  a.snap = dec_m >= 0 ? snap : nullptr;
  a.snap_seq = snap_seq;
  const dim3 grid(sh.blocks);
#define LES_PICK(WX, TY, NT)                                                          \
  do {                                                                                \
    const dim3 block(64 * WX * TY);                                                   \
    if (chebyshev && !first) {                                                        \
      if (check) sweep1_kernel<T, WX, TY, true, true, NT><<<grid, block, 0, s>>>(a);  \
      else sweep1_kernel<T, WX, TY, true, false, NT><<<grid, block, 0, s>>>(a);       \
    } else {                                                                          \
      if (check) sweep1_kernel<T, WX, TY, false, true, NT><<<grid, block, 0, s>>>(a); \
      else sweep1_kernel<T, WX, TY, false, false, NT><<<grid, block, 0, s>>>(a);      \
    }                                                                                 \
  } while (0)
  if (sh.wx == kWX && sh.stream)
    LES_PICK(kWX, kWideTYBig, true);
  else if (sh.wx == kWX)
    LES_PICK(kWX, kWideTY, false);
  else if (sh.ty == kTY1Big)
    LES_PICK(1, kTY1Big, true);
  else if (sh.ty == kTY1 && !sh.stream)
    LES_PICK(1, kTY1, false);
  else if (sh.ty == kTY1)
    LES_PICK(1, kTY1, true);
  else if (!sh.stream)
    LES_PICK(1, 1, false);
  else
    LES_PICK(1, 1, true);
#undef LES_PICK
}

#define LES_INST(T)                                                                            \
  template void launch_tsweep<T>(const Grid &, bool, bool, bool, double, double, const T *,    \
                                 const T *, T *, const T *, SolveCtl *, double *,              \
                                 const double *, int, int, int64_t *, int, hipStream_t);
LES_INST(float)
LES_INST(double)
#undef LES_INST

}  // namespace lesmi
