// Two or three Poisson sweeps per launch for grids whose iterates do not fit
// the chip.
//
// A sweep on its own moves 16 bytes per cell FP32 (phi, prev, rhs in, phi'
// out) and large grids run at the rate of a copy.  Here a block of NW waves
// takes a tile of 64 x NW R cells (lane = x, a thread R rows) and marches up
// z with S sweeps in flight, sweep s at plane p - s + 1, so that the fields
// are read and written once for all S.  The iterates of the last three planes
// stay in registers, and two planes more are in flight; x neighbours are lane
// shifts, y neighbours registers or, between waves, LDS (each wave's first and
// last row, double-buffered, one barrier per plane).  The tile shrinks by a
// ring per sweep: (64 - 2 S) x (NW R - 2 S) of its cells are results, the rest
// is formed by the neighbouring tiles too.
//
// Bound by memory: 20 bytes per cell and launch are needed, 25.6 move (rings of
// the neighbouring tiles, planes beside a chunk, lines that a tile needs a part
// of) at 4.7 TB/s; the arithmetic alone takes 50 of the 126 us below.  512 x 512 x 256 FP32: 126 us
// per sweep against 203 one by one (171 with one plane in flight instead of
// two); 512 x 256 x 128 FP64 57 against 116.
#include <algorithm>

#include "les_column.h"
#include "les_sweep.h"

namespace lesmi {

namespace {

template <typename T>
struct MArgs {
  Grid g;
  SweepCoef k;
  int kc, tiles_x, tiles_y, tiles_z, ntiles;
  double wc[3];  // Chebyshev weights of the launch's sweeps
  int first;     // its first sweep is the solve's (weight 1, no prev)
  const T *cur, *prev, *rhs;
  T *out_last, *out_prev;
  SolveCtl *ctl;
  double *partials;
};

// Block shapes.  FP64 holds half the rows.
template <typename T>
struct MTile {
  static constexpr int R = sizeof(T) == 4 ? 8 : 4, NW = 8, NT = 64 * NW, BY = R * NW;
};

__device__ __forceinline__ int pmod(int i, int n) {
  int r = i % n;
  return r < 0 ? r + n : r;
}

// v as it is, but unknown to the compiler.
template <typename V>
__device__ __forceinline__ void forget(V &v) {
  asm volatile("" : "+v"(v));
}

// plane_rsrc of a given range (0: reads are zero, stores are dropped).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t range_rsrc(const void *f, int64_t pb, int z,
                                                             int64_t range) {
  return __builtin_amdgcn_make_buffer_rsrc(
      const_cast<char *>(reinterpret_cast<const char *>(f) + z * pb), (short)0, (int)range,
      0x00020000);
}

template <typename T, int S, bool CHEB, bool CHECK>
__global__ __launch_bounds__(MTile<T>::NT) void msweep_kernel(MArgs<T> a) {
  if (a.ctl->done) return;
  using B = MTile<T>;
  constexpr int R = B::R, NW = B::NW;
  __shared__ T edge[2][S][NW][2][64];  // by parity and iterate: first, last row of each wave
  const Grid &g = a.g;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // XCD x takes the x-th contiguous part of the tiles
  const int per = (int)(gridDim.x >> 3);
  const int tile = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  double acc = 0.0;
  if (tile < a.ntiles) {  // the whole block
    const int tx = tile % a.tiles_x, rest = tile / a.tiles_x;
    const int ty = rest % a.tiles_y, tz = rest / a.tiles_y;
    const int k0 = tz * a.kc, k1 = min(g.nz, k0 + a.kc);
    const int xu = tx * (64 - 2 * S) - S + lane;
    const bool corex = lane >= S && lane < 64 - S && xu < g.nx;
    const int i = pmod(xu, g.nx);
    constexpr uint32_t kOut = 0x80000000u;  // beyond any plane (at most 2 GiB): dropped
    uint32_t o[R];                          // offsets of the rows
    bool core[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int yl = wv * R + r, yu = ty * (B::BY - 2 * S) - S + yl;
      core[r] = corex && yl >= S && yl < B::BY - S && yu < g.ny;
      o[r] = ((uint32_t)i + (uint32_t)g.nx * (uint32_t)pmod(yu, g.ny)) * (uint32_t)sizeof(T);
    }
    const int64_t pb = g.nxy * (int64_t)sizeof(T);
    const int p0 = max(0, k0 - (S - 1)), p1 = k1 + S - 1;  // steps [p0, p1)
    auto clampz = [&](int z) { return min(z, g.nz - 1); };
    // the iterate before the launch's input: zeros (a range of no bytes) in
    // the solve's first sweep, which with weight 1 is the Jacobi step
    const int64_t prev_range = a.first ? 0 : pb;

    // Planes by step p, the plane q in slot (q - p0) mod the slots: F0 (the
    // input) p - 1 .. p + 1, rh p - S + 1 .. p, pv p, each with two planes
    // more in flight; F[s - 1] (sweep s's iterate) p - s - 1 .. p - s + 1.
    T F0[6][R], F[S - 1][3][R], rh[6][R], pv[3][R];
    auto input = [&](int z, T(&d)[R]) __attribute__((always_inline)) {
      const __amdgpu_buffer_rsrc_t f = plane_rsrc(a.cur, pb, clampz(z));
#pragma unroll
      for (int r = 0; r < R; ++r) d[r] = rsrc_load<T>(f, o[r]);
    };
    auto others = [&](int z, T(&dr)[R], T(&dp)[R]) __attribute__((always_inline)) {
      const __amdgpu_buffer_rsrc_t f = plane_rsrc(a.rhs, pb, clampz(z));
#pragma unroll
      for (int r = 0; r < R; ++r) dr[r] = rsrc_load<T>(f, o[r]);
      if (CHEB) {
        const __amdgpu_buffer_rsrc_t h =
            range_rsrc(a.first ? a.cur : a.prev, pb, clampz(z), prev_range);
#pragma unroll
        for (int r = 0; r < R; ++r) dp[r] = rsrc_load<T>(h, o[r]);
      }
    };
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma unroll
      for (int s = 1; s < S; ++s) F[s - 1][0][r] = F[s - 1][1][r] = F[s - 1][2][r] = T(0);
      rh[4][r] = rh[5][r] = T(0);
    }
    input(max(p0 - 1, 0), F0[5]);
    input(p0, F0[0]);
    input(p0 + 1, F0[1]);
    others(p0, rh[0], pv[0]);
    input(p0 + 2, F0[2]);
    others(p0 + 1, rh[1], pv[1]);
    // what step p0 needs of the waves beside: the input at p0 (the later
    // sweeps' planes there are below the chunk)
#pragma unroll
    for (int s = 0; s < S; ++s) {
      edge[0][s][wv][0][lane] = s == 0 ? F0[0][0] : T(0);
      edge[0][s][wv][1][lane] = s == 0 ? F0[0][R - 1] : T(0);
    }
    auto step = [&](auto uc, int p) __attribute__((always_inline)) {
      constexpr int u = decltype(uc)::value;  // (p - p0) mod 6
      constexpr int par = u & 1;
      __syncthreads();
      input(p + 3, F0[(u + 3) % 6]);
      others(p + 2, rh[(u + 2) % 6], pv[(u + 2) % 3]);
      auto sweep = [&](auto sc) __attribute__((always_inline)) {
        // sweep s + 1 at plane q, from the iterate before it (and that's)
        constexpr int s = decltype(sc)::value;
        constexpr int c = (u - s + 6) % 6, up = (c + 1) % 6, dn = (c + 5) % 6;
        const int q = p - s;
        auto in = [&](int slot, int r) __attribute__((always_inline)) -> T & {
          if constexpr (s == 0) return F0[slot][r];
          else return F[s - 1][slot % 3][r];
        };
        auto before = [&](int r) __attribute__((always_inline)) -> T {
          if constexpr (s == 0) return pv[u % 3][r];
          else if constexpr (s == 1) return F0[c][r];
          else return F[s - 2][c % 3][r];
        };
        // conversions of one sweep are not kept for the next (registers)
#pragma unroll
        for (int r = 0; r < R; ++r) {
          forget(in(c, r));
          forget(in(up, r));
          forget(in(dn, r));
        }
        const T ylo = edge[par][s][wv > 0 ? wv - 1 : 0][1][lane];
        const T yhi = edge[par][s][wv < NW - 1 ? wv + 1 : NW - 1][0][lane];
        T out[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const T ctr = in(c, r);
          const T ym = r == 0 ? ylo : in(c, r > 0 ? r - 1 : 0);
          const T yp = r == R - 1 ? yhi : in(c, r < R - 1 ? r + 1 : R - 1);
          const double hx = (double)lane_shift<1>(ctr) + (double)lane_shift<-1>(ctr);
          const double hy = (double)yp + (double)ym;
          const double hz = (double)in(up, r) + (double)in(dn, r);
          const double res = point_residual(a.k, (double)ctr, hx, hy, hz, (double)rh[c][r]);
          if (CHECK && s == 0 && core[r] && p >= k0 && p < k1) acc += res * res;
          out[r] = (T)point_update(a.k, (double)ctr, res, CHEB, CHEB ? (double)before(r) : 0.0,
                                   a.wc[s]);
        }
        // results of other chunks' planes go nowhere (a range of no bytes):
        // a store under a branch would keep the waits for the loads in flight
        // from being counted
        if constexpr (s == S - 1 || (CHEB && s == S - 2)) {
          T *f = s == S - 1 ? a.out_last : a.out_prev;
          const bool mine = q >= k0 && q < k1;
          const __amdgpu_buffer_rsrc_t ro = range_rsrc(f, pb, mine ? q : k0, mine ? pb : 0);
#pragma unroll
          for (int r = 0; r < R; ++r) rsrc_store<T>(ro, core[r] ? o[r] : kOut, out[r]);
        }
        if constexpr (s + 1 < S) {
          // the walls' mirror: plane nz is plane nz - 1, plane -1 plane 0
          if (q >= g.nz) {
#pragma unroll
            for (int r = 0; r < R; ++r) out[r] = F[s][dn % 3][r];
          }
#pragma unroll
          for (int r = 0; r < R; ++r) F[s][c % 3][r] = out[r];
          if (q == 0) {
#pragma unroll
            for (int r = 0; r < R; ++r) F[s][dn % 3][r] = out[r];
          }
        }
      };
      sweep(std::integral_constant<int, 0>{});
      __builtin_amdgcn_sched_barrier(0);
      sweep(std::integral_constant<int, 1>{});
      if constexpr (S > 2) {
        __builtin_amdgcn_sched_barrier(0);
        sweep(std::integral_constant<int, 2>{});
      }
      // the rows that the next step's waves beside need: sweep s's iterate at
      // plane p + 1 - s
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const int n = (u + 1 - s + 6) % 6;
        edge[par ^ 1][s][wv][0][lane] = s == 0 ? F0[n][0] : F[s > 0 ? s - 1 : 0][n % 3][0];
        edge[par ^ 1][s][wv][1][lane] = s == 0 ? F0[n][R - 1] : F[s > 0 ? s - 1 : 0][n % 3][R - 1];
      }
    };
    for (int p = p0;; p += 6) {
      step(std::integral_constant<int, 0>{}, p);
      if (p + 1 >= p1) break;
      step(std::integral_constant<int, 1>{}, p + 1);
      if (p + 2 >= p1) break;
      step(std::integral_constant<int, 2>{}, p + 2);
      if (p + 3 >= p1) break;
      step(std::integral_constant<int, 3>{}, p + 3);
      if (p + 4 >= p1) break;
      step(std::integral_constant<int, 4>{}, p + 4);
      if (p + 5 >= p1) break;
      step(std::integral_constant<int, 5>{}, p + 5);
      if (p + 6 >= p1) break;
    }
  }
  if (CHECK) {
    const double s = block_sum(acc);
    if (threadIdx.x == 0) a.partials[blockIdx.x] = s;
  }
}

struct MShape {
  int kc, tiles_x, tiles_y, tiles_z, ntiles, blocks;
};

// One block fills a CU, so the time goes as the rounds of 256 blocks that
// the launch takes times the planes of a chunk (its levels and the 2 S of
// the pipeline); the chunk length with the least of that is taken.
MShape mshape_of(const Grid &g, int S, int by) {
  MShape m;
  m.tiles_x = (g.nx + 63 - 2 * S) / (64 - 2 * S);
  m.tiles_y = (g.ny + by - 2 * S - 1) / (by - 2 * S);
  const int64_t cols = (int64_t)m.tiles_x * m.tiles_y;
  int64_t best = INT64_MAX;
  m.tiles_z = 1;
  for (int n = 1; n <= g.nz && n <= 64; ++n) {
    if (cols * n > kPartials && n > 1) break;
    const int64_t cost = (cols * n + 255) / 256 * ((g.nz + n - 1) / n + 2 * S);
    if (cost < best) {
      best = cost;
      m.tiles_z = n;
    }
  }
  m.kc = (g.nz + m.tiles_z - 1) / m.tiles_z;
  m.tiles_z = (g.nz + m.kc - 1) / m.kc;
  m.ntiles = (int)(cols * m.tiles_z);
  m.blocks = (m.ntiles + 7) / 8 * 8;
  return m;
}

}  // namespace

template <typename T>
int msweep_blocks(const Grid &g, int S) {
  return mshape_of(g, S, MTile<T>::BY).blocks;
}

// Microseconds of a launch of two sweeps: its start, the planes its rounds of
// blocks walk and the cells, or the memory's time beyond the caches.  Within 20
// % (rms) of the 219 grids of sweep2_us.
template <typename T>
double two_sweep_tiles_us(const Grid &g) {
  const MShape m = mshape_of(g, 2, MTile<T>::BY);
  const double planes = (double)((m.ntiles + 255) / 256) * (m.kc + 4);
  const double cells = 1e-6 * (double)g.n;
  const bool f32 = sizeof(T) == 4;
  return std::max(f32 ? 2.4 + 1.52 * planes + 0.72 * cells : 1.5 + 1.28 * planes + 0.37 * cells,
                  two_sweeps_streamed<T>(g) ? (f32 ? 4.0 : 8.3) * cells : 0.0);
}

// Rows of a tile.  Two sweeps run by tiles of 64 (FP64 32) rows here or by
// four-row waves (k_sweep2.hip): whichever takes less, of those whose partials
// fit (0: none, one sweep per launch).
template <typename T>
int msweep_rows(const Grid &g, int S) {
  constexpr int BY = MTile<T>::BY;
  if (S != 2) return S > 2 ? BY : 0;
  const bool tiles = msweep_blocks<T>(g, 2) <= kPartials, thin = sweep2_blocks(g) > 0;
  if (tiles && thin) return two_sweep_tiles_us<T>(g) <= sweep2_us<T>(g) ? BY : kThinRows;
  return tiles ? BY : thin ? kThinRows : 0;
}

// Three sweeps a launch where a launch forms at most five cells per result
// (tile rings, pipeline planes and a last round that is not full), else one
// by one: thin grids and short rows leave most of a tile unused.  Per sweep,
// one by one and three at a time, by cells formed per result: 1.4 (512 x 512 x
// 256 FP32) 203 and 126 us; 3.0 (2100 x 32 x 256 FP32) 60 and 48; 3.7 (1700 x
// 2500 x 4 FP32) 58 and 39; 2.7 (2120 x 16 x 640 FP64) 155 and 83; 7.2 (1000 x
// 33 x 44 FP32) 6.8 and 6.9; 10.4 (5120 x 8 x 640 FP32) 86 and 195.
template <typename T>
int msweep_depth(const Grid &g, int asked) {
  if (asked == 2 && msweep_rows<T>(g, 2) == 0) return 1;
  if (asked > 0) return asked;
  constexpr int S = 3, BY = MTile<T>::BY;
  const MShape m = mshape_of(g, S, BY);
  const int64_t rounds = (m.ntiles + 255) / 256;
  const int64_t formed = rounds * (m.kc + 2 * S) * 256 * 64 * BY;
  return m.blocks <= kPartials && formed <= 5 * g.n ? S : 1;
}

template <typename T>
void launch_msweep(const Grid &g, int S, bool chebyshev, bool check, bool first, double omega_jacobi,
                   const double *omega_cheb, const T *cur, const T *prev, T *out_last, T *out_prev,
                   const T *rhs, SolveCtl *ctl, double *partials, hipStream_t s) {
  const MShape m = mshape_of(g, S, MTile<T>::BY);
  MArgs<T> a;
  a.g = g;
  a.k = sweep_coef(g, omega_jacobi);
  a.kc = m.kc;
  a.tiles_x = m.tiles_x;
  a.tiles_y = m.tiles_y;
  a.tiles_z = m.tiles_z;
  a.ntiles = m.ntiles;
  for (int q = 0; q < 3; ++q) a.wc[q] = q < S ? omega_cheb[q] : 1.0;
  a.first = first ? 1 : 0;
  a.cur = cur;
  a.prev = prev;
  a.rhs = rhs;
  a.out_last = out_last;
  a.out_prev = out_prev;
  a.ctl = ctl;
  a.partials = partials;
#define LES_GO(S_, C_, K_) msweep_kernel<T, S_, C_, K_><<<m.blocks, MTile<T>::NT, 0, s>>>(a)
#define LES_PICK(S_)                            \
  (chebyshev ? (check ? LES_GO(S_, true, true)  \
                      : LES_GO(S_, true, false)) \
             : (check ? LES_GO(S_, false, true) \
                      : LES_GO(S_, false, false)))
  if (S == 2) LES_PICK(2);
  else LES_PICK(3);
#undef LES_PICK
#undef LES_GO
}

#define LES_INST(T)                                                                              \
  template int msweep_blocks<T>(const Grid &, int);                                              \
  template int msweep_depth<T>(const Grid &, int);                                               \
  template int msweep_rows<T>(const Grid &, int);                                                \
  template void launch_msweep<T>(const Grid &, int, bool, bool, bool, double, const double *,    \
                                 const T *, const T *, T *, T *, const T *, SolveCtl *, double *, \
                                 hipStream_t);
LES_INST(float)
LES_INST(double)
#undef LES_INST

}  // namespace lesmi
