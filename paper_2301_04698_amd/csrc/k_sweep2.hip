// Two Poisson sweeps per launch on thin grids.
//
// A block of k_msweep.hip forms 64 rows (32 FP64) of 64 columns at a time
// whatever the grid has; where ny is small most of them are copies of the same
// rows.  Here a wave owns R rows j0 .. j0+R-1 and a 62-cell x segment (lanes
// 1..62; lanes 0 and 63 are its halo columns, wrapped periodically like every
// other lane) of the z chunk [k0, k1), without LDS or barriers.  Marching up z
// it forms the first sweep on rows j0-1 .. j0+R at level k (their y neighbours
// are rows j0-2 .. j0+R+1 of the iterate, x neighbours the adjacent lanes, z
// neighbours registers), then the second sweep on its R rows at level k-1 from
// first-sweep values that are all in its own registers or adjacent lanes.  The
// first sweep of the two boundary rows is also formed by the neighbouring
// waves; in exchange every array is read from memory once per two sweeps
// (neighbour rows through the caches).  All accesses are buffer loads and
// stores on one z plane: lanes outside the segment's core, and rows beyond the
// grid, store at an offset past the plane's range, which the hardware drops.
//
// Bound by the latency of a level's loads (nothing is in flight beyond it).
// Microseconds per sweep of two, tiles and here: 5120 x 1 x 640 FP32 206 and
// 22, 5120 x 8 x 640 FP32 210 and 78, 2000 x 20 x 300 FP32 41 and 26; 512 x 512
// x 256 FP32 193 and 249.
#include <algorithm>

#include "les_column.h"
#include "les_sweep.h"

namespace lesmi {

namespace {

constexpr int kR2 = kThinRows;  // rows per wave

template <typename T>
struct Args2 {
  Grid g;
  SweepCoef k;
  int kc, tiles_x, tiles_y, ntiles;
  double wc[2];  // Chebyshev weights of the launch's sweeps
  int first;     // its first sweep is the solve's (weight 1, no prev)
  const T *cur, *prev, *rhs;
  T *out_last, *out_prev;
  SolveCtl *ctl;
  double *partials;
};

__device__ __forceinline__ int pmod(int i, int n) {
  int r = i % n;
  return r < 0 ? r + n : r;
}

template <typename T, int R, bool CHEB, bool CHECK>
__global__ __launch_bounds__(256) void sweep2_kernel(Args2<T> a) {
  if (a.ctl->done) return;
  constexpr int NR = R + 2;  // first-sweep rows j0-1 .. j0+R
  const Grid &g = a.g;
  // XCD x takes the x-th contiguous part of the tiles
  const int lb = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int lane = (int)(threadIdx.x & 63);
  const int u = lb * 4 + wave;
  double acc = 0.0;
  if (u < a.ntiles) {  // uniform per wave
    const int ty = u % a.tiles_y, rest = u / a.tiles_y;
    const int tx = rest % a.tiles_x, tz = rest / a.tiles_x;
    const int j0 = ty * R;
    const int k0 = tz * a.kc, k1 = min(g.nz, k0 + a.kc);
    const int xu = tx * 62 - 1 + lane;
    const bool core = lane >= 1 && lane <= 62 && xu < g.nx;
    const int i = pmod(xu, g.nx), il = pmod(xu - 1, g.nx), ir = pmod(xu + 1, g.nx);
    constexpr uint32_t kOut = 0x80000000u;  // beyond any plane (at most 2 GiB)
    const uint32_t es = (uint32_t)sizeof(T);
    uint32_t o[R + 4];  // rows j0-2 .. j0+R+1 of this lane's column
#pragma unroll
    for (int d = 0; d < R + 4; ++d)
      o[d] = ((uint32_t)i + (uint32_t)g.nx * (uint32_t)pmod(j0 + d - 2, g.ny)) * es;
    uint32_t oxl[NR], oxr[NR];  // x neighbours of the end lanes
#pragma unroll
    for (int d = 0; d < NR; ++d) {
      const uint32_t row = (uint32_t)g.nx * (uint32_t)pmod(j0 + d - 1, g.ny);
      oxl[d] = lane == 0 ? ((uint32_t)il + row) * es : kOut;
      oxr[d] = lane == 63 ? ((uint32_t)ir + row) * es : kOut;
    }
    uint32_t ost[R];  // store offsets of the output rows
    bool rcore[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      rcore[r] = core && j0 + r < g.ny;
      ost[r] = rcore[r] ? o[r + 2] : kOut;
    }
    const int64_t pb = g.nxy * (int64_t)sizeof(T);
    const bool cheb1 = CHEB && !a.first;
    const int kb = max(0, k0 - 1), ke = min(g.nz - 1, k1);
    // iterate of the first-sweep rows at levels k-1 (bl) and k (cc)
    T bl[NR], cc[NR];
    {
      const __amdgpu_buffer_rsrc_t rb = plane_rsrc(a.cur, pb, kb > 0 ? kb - 1 : 0);
      const __amdgpu_buffer_rsrc_t rc = plane_rsrc(a.cur, pb, kb);
#pragma unroll
      for (int d = 0; d < NR; ++d) {
        bl[d] = rsrc_load<T>(rb, o[d + 1]);
        cc[d] = rsrc_load<T>(rc, o[d + 1]);
      }
    }
    // first-sweep values at level k-1 (all rows) and k-2 (output rows);
    // rhs and iterate of the output rows at level k-1
    T s1p[NR], s1pp[R], rm1[R], cm1[R];
#pragma unroll
    for (int d = 0; d < NR; ++d) s1p[d] = T(0);
#pragma unroll
    for (int r = 0; r < R; ++r) s1pp[r] = rm1[r] = cm1[r] = T(0);
    for (int k = kb; k <= ke; ++k) {
      const __amdgpu_buffer_rsrc_t rk = plane_rsrc(a.cur, pb, k);
      const __amdgpu_buffer_rsrc_t ra = plane_rsrc(a.cur, pb, k + 1 < g.nz ? k + 1 : k);
      const __amdgpu_buffer_rsrc_t rr = plane_rsrc(a.rhs, pb, k);
      T ab[NR], rh[NR], pv[NR], xl[NR], xr[NR];
#pragma unroll
      for (int d = 0; d < NR; ++d) {
        ab[d] = rsrc_load<T>(ra, o[d + 1]);
        rh[d] = rsrc_load<T>(rr, o[d + 1]);
        xl[d] = rsrc_load<T>(rk, oxl[d]);
        xr[d] = rsrc_load<T>(rk, oxr[d]);
        pv[d] = T(0);
      }
      const T ylo = rsrc_load<T>(rk, o[0]), yhi = rsrc_load<T>(rk, o[R + 3]);
      if (cheb1) {
        const __amdgpu_buffer_rsrc_t rp = plane_rsrc(a.prev, pb, k);
#pragma unroll
        for (int d = 0; d < NR; ++d) pv[d] = rsrc_load<T>(rp, o[d + 1]);
      }
      const bool core_k = k >= k0 && k < k1;
      // ---- first sweep, rows j0-1 .. j0+R at level k
      T s1[NR];
#pragma unroll
      for (int d = 0; d < NR; ++d) {
        const T sp = lane_shift<1>(cc[d]), sm = lane_shift<-1>(cc[d]);
        const T xp = lane == 63 ? xr[d] : sp;
        const T xm = lane == 0 ? xl[d] : sm;
        const T yp = d == NR - 1 ? yhi : cc[d < NR - 1 ? d + 1 : NR - 1];
        const T ym = d == 0 ? ylo : cc[d > 0 ? d - 1 : 0];
        const double hx = (double)xp + (double)xm;
        const double hy = (double)yp + (double)ym;
        const double hz = (double)ab[d] + (double)bl[d];
        const double res = point_residual(a.k, (double)cc[d], hx, hy, hz, (double)rh[d]);
        if (CHECK && d >= 1 && d <= R && core_k && rcore[d >= 1 && d <= R ? d - 1 : 0])
          acc += res * res;
        s1[d] = (T)point_update(a.k, (double)cc[d], res, cheb1, (double)pv[d], a.wc[0]);
      }
      if (CHEB && core_k) {
        const __amdgpu_buffer_rsrc_t ro = plane_rsrc(a.out_prev, pb, k);
#pragma unroll
        for (int r = 0; r < R; ++r) rsrc_store<T>(ro, ost[r], s1[r + 1]);
      }
      // ---- second sweep, output rows at level k-1
      if (k - 1 >= k0 && k - 1 < k1) {
        const __amdgpu_buffer_rsrc_t ro = plane_rsrc(a.out_last, pb, k - 1);
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const T ctr = s1p[r + 1];
          const T lo = k - 1 == 0 ? ctr : s1pp[r];
          const double h2x = (double)lane_shift<1>(ctr) + (double)lane_shift<-1>(ctr);
          const double h2y = (double)s1p[r + 2] + (double)s1p[r];
          const double h2z = (double)s1[r + 1] + (double)lo;
          const double r2 = point_residual(a.k, (double)ctr, h2x, h2y, h2z, (double)rm1[r]);
          rsrc_store<T>(ro, ost[r], (T)point_update(a.k, (double)ctr, r2, CHEB, (double)cm1[r], a.wc[1]));
        }
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        s1pp[r] = s1p[r + 1];
        rm1[r] = rh[r + 1];
        cm1[r] = cc[r + 1];
      }
#pragma unroll
      for (int d = 0; d < NR; ++d) {
        s1p[d] = s1[d];
        bl[d] = cc[d];
        cc[d] = ab[d];
      }
    }
    if (k1 == g.nz) {  // the top level: its upper neighbour is itself
      const int kk = g.nz - 1;
      const __amdgpu_buffer_rsrc_t ro = plane_rsrc(a.out_last, pb, kk);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const T ctr = s1p[r + 1];
        const T lo = kk == 0 ? ctr : s1pp[r];
        const double h2x = (double)lane_shift<1>(ctr) + (double)lane_shift<-1>(ctr);
        const double h2y = (double)s1p[r + 2] + (double)s1p[r];
        const double h2z = (double)ctr + (double)lo;
        const double r2 = point_residual(a.k, (double)ctr, h2x, h2y, h2z, (double)rm1[r]);
        rsrc_store<T>(ro, ost[r], (T)point_update(a.k, (double)ctr, r2, CHEB, (double)cm1[r], a.wc[1]));
      }
    }
  }
  if (CHECK) {
    const double s = block_sum(acc);
    if (threadIdx.x == 0) a.partials[blockIdx.x] = s;
  }
}

struct Shape2 {
  int kc, tiles_x, tiles_y, tiles_z, ntiles, blocks;
};

// One wave per kR2 rows and 62-cell x segment, four waves per block; z chunks
// halved (to 8 levels at least) until about 8192 waves.  No blocks where even
// whole columns make too many partials (planes of 65 million cells).
Shape2 shape2_of(const Grid &g) {
  Shape2 sh;
  sh.tiles_x = (g.nx + 61) / 62;
  sh.tiles_y = (g.ny + kR2 - 1) / kR2;
  const int64_t rows = (int64_t)sh.tiles_x * sh.tiles_y;
  auto blocks = [&](int kc) { return (rows * ((g.nz + kc - 1) / kc) + 31) / 32 * 8; };
  sh.kc = g.nz;
  while (sh.kc > 8 && rows * ((g.nz + sh.kc - 1) / sh.kc) < 8192) sh.kc = (sh.kc + 1) / 2;
  while (blocks(sh.kc) > kPartials && sh.kc < g.nz) sh.kc *= 2;
  sh.tiles_z = (g.nz + sh.kc - 1) / sh.kc;
  const bool fits = blocks(sh.kc) <= kPartials;
  sh.ntiles = fits ? (int)(rows * sh.tiles_z) : 0;
  sh.blocks = fits ? (int)blocks(sh.kc) : 0;
  return sh;
}

}  // namespace

int sweep2_blocks(const Grid &g) { return shape2_of(g).blocks; }

// Microseconds of a launch: its start, the levels a wave walks, the wave levels
// and the cells, or the memory's time beyond the caches.  Within 24 % (rms) of
// 219 measured grids of 8 to 6000 columns, 1 to 900 rows and 4 to 1500 levels;
// of the two kernels it and two_sweep_tiles_us take, 5 of them run more than 4
// % (14 at most) slower than in the other.
template <typename T>
double sweep2_us(const Grid &g) {
  const Shape2 sh = shape2_of(g);
  const double waves = 1e-3 * sh.tiles_x * sh.tiles_y * (g.nz + 2.0 * sh.tiles_z);
  const double cells = 1e-6 * (double)g.n;
  const bool f32 = sizeof(T) == 4;
  return std::max(f32 ? 6.5 + 0.69 * sh.kc + 0.49 * waves + 0.11 * cells
                      : 3.6 + 1.58 * sh.kc + 0.78 * waves,
                  two_sweeps_streamed<T>(g) ? (f32 ? 5.7 : 11.9) * cells : 0.0);
}

template <typename T>
void launch_sweep2(const Grid &g, bool chebyshev, bool check, bool first, double omega_jacobi,
                   const double *omega_cheb, const T *cur, const T *prev, T *out_last, T *out_prev,
                   const T *rhs, SolveCtl *ctl, double *partials, hipStream_t s) {
  const Shape2 sh = shape2_of(g);
  Args2<T> a;
  a.g = g;
  a.k = sweep_coef(g, omega_jacobi);
  a.kc = sh.kc;
  a.tiles_x = sh.tiles_x;
  a.tiles_y = sh.tiles_y;
  a.ntiles = sh.ntiles;
  a.wc[0] = omega_cheb[0];
  a.wc[1] = omega_cheb[1];
  a.first = first ? 1 : 0;
  a.cur = cur;
  a.prev = prev;
  a.rhs = rhs;
  a.out_last = out_last;
  a.out_prev = out_prev;
  a.ctl = ctl;
  a.partials = partials;
  const dim3 grid(sh.blocks), block(256);
  if (chebyshev) {
    if (check) sweep2_kernel<T, kR2, true, true><<<grid, block, 0, s>>>(a);
    else sweep2_kernel<T, kR2, true, false><<<grid, block, 0, s>>>(a);
  } else {
    if (check) sweep2_kernel<T, kR2, false, true><<<grid, block, 0, s>>>(a);
    else sweep2_kernel<T, kR2, false, false><<<grid, block, 0, s>>>(a);
  }
}

#define LES_INST(T)                                                                               \
  template double sweep2_us<T>(const Grid &);                                                     \
  template void launch_sweep2<T>(const Grid &, bool, bool, bool, double, const double *,          \
                                 const T *, const T *, T *, T *, const T *, SolveCtl *, double *, \
                                 hipStream_t);
LES_INST(float)
LES_INST(double)
#undef LES_INST

}  // namespace lesmi
