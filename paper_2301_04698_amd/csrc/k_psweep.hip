// Which solves run resident on the chip (les_resident.h), and their launch.
#include "les_resident.h"

namespace lesmi {

using namespace resident;

namespace {

struct Fit {
  int shape = 0;  // 0 none; 1 S, 2 M1, 3 M2, 4 M3, 5 L; 6 RowS, 7 RowL
  int tx = 0, ty = 0, tz = 0, nb = 0, face = 0;
  bool rag = false;
};

// Microseconds per sweep launch by launch, one sweep each: the launch, the
// 64-cell pieces of rows (a wave's work) and the bytes.  Within 10 % (rms) of
// 680 measured grids of 2 to 6000 columns, 1 to 4096 rows and 4 to 30000
// levels.
template <typename T>
double one_sweep_us(const Grid &g, bool chebyshev) {
  const bool f32 = sizeof(T) == 4;
  const double pieces = 1e-3 * ((g.nx + 63) / 64) * g.ny * g.nz;
  const double mb = 1e-6 * (double)g.n * sizeof(T) * (chebyshev ? 4 : 3);
  if (g.ny == 1)
    return f32 ? 3.5 + 0.072 * pieces + 0.094 * mb : 3.7 + 0.148 * pieces + 0.058 * mb;
  return f32 ? 4.0 + 0.086 * pieces + 0.054 * mb : 4.0 + 0.202 * pieces + 0.041 * mb;
}

// Microseconds per sweep in boxes of a shape that hold so many levels per
// thread: much the same whatever part of a box's columns and rows is filled
// (within 8 %, rms, of 490 measured grids).  The small shapes, 0 here, were
// nowhere more than 2 % slower than launch by launch.
template <typename T>
double resident_us(int shape, int levels) {
  const bool f32 = sizeof(T) == 4;
  switch (shape) {
    case 3: return f32 ? 0.0 : 4.4 + 0.104 * levels;
    case 4: return f32 ? 1.9 + 0.244 * levels : 5.2 + 0.357 * levels;
    case 5: return 6.0 + 0.183 * levels;
    case 7: return f32 ? 7.4 + 0.053 * levels : 7.7 + 0.053 * levels;
    default: return 0.0;
  }
}

// One block per CU: the boxes of shape B, if they all fit at once.
template <class B>
bool try_box(const Grid &g, int shape, Fit *f) {
  const int tx = (g.nx + 63) / 64, ty = (g.ny + B::BY - 1) / B::BY, tz = (g.nz + B::BZ - 1) / B::BZ;
  if ((int64_t)tx * ty * tz > kResidentBlocks) return false;
  // one-row boxes: each of the eight waves holds a level
  if (B::D2 && g.nz / tz < kNW) return false;
  f->shape = shape;
  f->tx = tx;
  f->ty = ty;
  f->tz = tz;
  f->nb = tx * ty * tz;
  f->face = B::FACE;
  f->rag = g.nx != 64 * tx || g.ny != B::BY * ty || g.nz != B::BZ * tz;
  return true;
}

// The smallest shape whose boxes all fit, so that a grid spreads over many
// CUs: 128 x 128 x 64 FP32 takes 3.4 us per sweep in 128 boxes of M2 and 2.5 in
// 256 of M1, 256 x 128 x 64 FP64 10.2 in 128 of M3 and 7.0 in 256 of M2.
// Fixed-weight Jacobi sweeps (small grids: their count grows with the square
// of the grid's width) have no large boxes.
template <typename T>
Fit smallest_fit(const Grid &g, bool chebyshev) {
  static_assert(kResidentBlocks <= kNT, "every block's partial has a thread that reads it");
  using S = Shapes<T>;
  Fit f;
  if (g.ny == 1) {
    if (!try_box<typename S::RowS>(g, 6, &f)) try_box<typename S::RowL>(g, 7, &f);
    return f;
  }
  if (try_box<typename S::S>(g, 1, &f) || try_box<typename S::M1>(g, 2, &f) ||
      try_box<typename S::M2>(g, 3, &f) || !chebyshev || try_box<typename S::M3>(g, 4, &f))
    return f;
  if (S::F32) try_box<typename S::L>(g, 5, &f);
  return f;
}

// A grid that fills little of the large boxes (few columns or rows, so many
// levels) is not worth a box's time: those run launch by launch.  Resident and
// one by one, microseconds per sweep: 9.7 and 5.6 for one row, 8000 x 65 FP32,
// 9.4 and 16.5 for 640 x 5120 FP64; 10.2 and 6.8 for 929 x 3 x 470 FP32, 12.6
// and 20.1 for 114 x 343 x 160; 11.1 and 8.8 for 3 x 17 x 1470 FP64, 11.3 and
// 22.0 for 1327 x 28 x 95.
template <typename T>
Fit fit_of(const Grid &g, bool chebyshev) {
  const Fit f = smallest_fit<T>(g, chebyshev);
  if (f.shape == 0) return f;
  const int box = (g.nz + f.tz - 1) / f.tz, levels = g.ny == 1 ? (box + kNW - 1) / kNW : box;
  return resident_us<T>(f.shape, levels) <= one_sweep_us<T>(g, chebyshev) ? f : Fit{};
}

}  // namespace

template <typename T>
int psweep_blocks(const Grid &g, bool chebyshev) {
  return fit_of<T>(g, chebyshev).nb;
}

template <typename T>
size_t psweep_words(const Grid &g, bool chebyshev) {
  const Fit f = fit_of<T>(g, chebyshev);
  return (size_t)f.nb * (2 * f.face + 4);
}

template <typename T>
hipError_t launch_psweep(const Grid &g, bool chebyshev, double omega_j, double rho, int every,
                         uint32_t base, const T *rhs, const T *rhs_kept, T *out, uint64_t *words,
                         SolveCtl *ctl, hipStream_t s) {
  const Fit f = fit_of<T>(g, chebyshev);
  PArgs<T> a;
  a.g = g;
  a.k = sweep_coef(g, omega_j);
  a.w1 = 1.0 / (1.0 - 0.5 * rho * rho);
  a.q = 0.25 * rho * rho;
  a.tx = f.tx;
  a.ty = f.ty;
  a.tz = f.tz;
  a.every = every;
  a.base = base;
  a.rhs = rhs;
  a.rhs_kept = rhs_kept;
  a.out = out;
  a.faces = words;
  a.red = words + (size_t)f.nb * 2 * f.face;
  a.ctl = ctl;
  using S = Shapes<T>;
#define LES_BOX(B)                                                            \
  (chebyshev ? (f.rag ? launch_box<typename S::B, true, true>(a, f.nb, s)     \
                      : launch_box<typename S::B, true, false>(a, f.nb, s))   \
             : (f.rag ? launch_box<typename S::B, false, true>(a, f.nb, s)    \
                      : launch_box<typename S::B, false, false>(a, f.nb, s)))
#define LES_CHEB(B, RAGGED)                                       \
  (f.rag ? launch_box<typename S::RAGGED, true, true>(a, f.nb, s) \
         : launch_box<typename S::B, true, false>(a, f.nb, s))
  switch (f.shape) {
    case 1: return LES_BOX(S);
    case 2: return LES_BOX(M1);
    case 3: return LES_BOX(M2);
    case 4: return LES_CHEB(M3, M3Rag);
    case 5: return LES_CHEB(L, LRag);
    case 6: return LES_BOX(RowS);
    case 7: return LES_BOX(RowL);
    default: return hipErrorInvalidValue;
  }
#undef LES_CHEB
#undef LES_BOX
}

#define LES_INST(T)                                                                              \
  template int psweep_blocks<T>(const Grid &, bool);                                             \
  template size_t psweep_words<T>(const Grid &, bool);                                           \
  template hipError_t launch_psweep<T>(const Grid &, bool, double, double, int, uint32_t,        \
                                       const T *, const T *, T *, uint64_t *, SolveCtl *,        \
                                       hipStream_t);
LES_INST(float)
LES_INST(double)
#undef LES_INST

}  // namespace lesmi
