// Poisson sweeps with the whole solve resident on the chip.
//
// The one-sweep kernel moves 16 bytes per cell and sweep and is bound by
// that traffic (by the launch on small grids), while the arithmetic of a
// sweep needs a quarter of the time.  A grid whose iterates fit the register
// files (128 MB over 256 CUs) needs none of it: here each block keeps a box
// of cells for the whole solve, phi_m and phi_{m-1} in registers, the
// right-hand side in LDS (some of it in registers where LDS is short), and
// only the faces of the boxes move, through memory, once per sweep.  One
// launch runs every sweep of a solve and takes the stopping decision itself.
//
// What bounds it: FP64 issue where the boxes are large (a cell's update is 19
// FP64 instructions and conversions at 2.2 ns per wave and SIMD: 5.4 of the
// 10.5 us below, the rest other instructions, barriers and waits for faces),
// the round trip of a face through memory (about 1.5 us) where they are small.
// Microseconds per sweep, one-sweep kernel and here: 256 x 256 x 128 FP32
// 22.9 and 10.5; 256 x 256 x 64 FP64 24.2 and 11.7; 64 x 64 x 64 FP32 5.1 and
// 1.7; 250 x 200 x 100 FP32 (ragged boxes) 17.5 and 11; one row, 1024 x 128
// FP64 4.6 and 1.7.
//
// Layout.  A block is eight waves; lane = x (64 cells), a thread holds R rows
// by Z levels of its x.  Waves stack in y (three-dimensional grids: boxes of
// 64 x 8R x Z) or in z (one row, ny = 1: boxes of 64 x 1 x 8Z).  A sweep
// handles the levels in groups of GL: x neighbours by lane shifts, y
// neighbours inside a thread's rows from registers and across waves through
// LDS, z neighbours from registers.
//
// Faces.  Every value a neighbouring block needs is stored as a 64-bit word
// (32-bit half of the value, tag = number of the iterate) with a relaxed
// device-scope atomic, and the reader polls that word until the tag is the
// one it needs: data and flag arrive together, so no fence, no flag and no
// second round trip.  Words alternate between two slots by the tag's parity.
// A word of iterate t + 2 can only be written after the writer took the
// reader's iterate t + 1, which the reader published after it had taken
// iterate t, so two slots are enough.  The faces of a group are published
// when the group is done and read one sweep later, one group ahead of their
// use, so with several groups the exchange hides behind the arithmetic; the
// order of the groups (not bottom to top) keeps the top level's value from
// being needed the moment it is made.
//
// Residual tests.  In a checking sweep every block publishes its FP64 partial
// sum (two tagged words) and every block sums all of them in one order, so
// all take the same decision.  The launch is cooperative: its blocks are
// resident together, so every wait ends.  Each wait is bounded all the same
// (kSpinTicks); a block that gives up sets ctl->aborted and every block runs
// to its end without waiting, and the host repeats the solve launch by launch.
#pragma once

#include <algorithm>
#include <type_traits>
#include <utility>

#include "les_sweep.h"

namespace lesmi {
namespace resident {

constexpr int kNW = 8, kNT = 64 * kNW;
// Ticks of the constant 100 MHz clock a wait may take: 2 s.
constexpr uint64_t kSpinTicks = 200000000ull;

// Box shapes.  D2: one row (ny = 1), waves stacked in z.  GL: levels per
// group.  RV: right-hand side vectors (GL levels of a row) kept in
// registers, the rest in LDS.
template <typename T_, int R_, int Z_, int GL_, bool D2_, int RV_>
struct Box {
  using T = T_;
  static constexpr int R = R_, Z = Z_, GL = GL_, NG = Z_ / GL_, RV = RV_;
  static constexpr bool D2 = D2_;
  static constexpr int BY = D2_ ? 1 : kNW * R_, BZ = D2_ ? kNW * Z_ : Z_;  // box rows, levels
  static constexpr int NS = kNW * R_;        // (wave, row) slots
  static constexpr int NWD = sizeof(T_) / 4; // words per value
  static constexpr int NV = R_ * NG;         // rhs vectors per thread
  // y faces go to memory by way of LDS, a word per thread, where several
  // groups hide the longer way; from the edge waves at once otherwise
  static constexpr bool YLDS = NG >= 4;
  // the largest boxes with long groups have LDS for one group's rows only: a
  // second barrier per group instead of a second buffer
  static constexpr bool SB = NV * GL * sizeof(T_) >= 256 && GL * sizeof(T_) > 16;
  static constexpr int NB = SB ? 1 : 2;
  static constexpr int SL = 8 / (int)sizeof(T_);  // levels per LDS operand read
  // face words of one parity: z faces [slot][lane], y faces [level][lane],
  // x faces [slot][level]; x level index is the thread's own
  static constexpr int ZF = NS * 64 * NWD, YF = D2_ ? 0 : Z_ * 64 * NWD, XF = NS * Z_ * NWD;
  static constexpr int FACE = 2 * (ZF + YF + XF);
  // polled words per thread and group
  static constexpr int YN = D2_ ? 0 : 2 * GL_ * 64 * NWD, XN = 2 * NS * GL_ * NWD;
  static constexpr int YP = (YN + kNT - 1) / kNT, XP = (XN + kNT - 1) / kNT;
};

template <typename T>
struct PArgs {
  Grid g;
  SweepCoef k;
  // Chebyshev weights, rho = (mu_max - mu_min) / (mu_max + mu_min): the second
  // sweep's, and rho^2 / 4 of the recurrence
  double w1, q;
  int tx, ty, tz;   // boxes
  int every;        // sweeps between residual tests
  uint32_t base;    // tag of phi_0
  const T *rhs, *rhs_kept;  // rhs_kept (nullable): instead of rhs if ctl->guess_kept
  T *out;
  uint64_t *faces;  // two parities of FACE words per block
  uint64_t *red;    // two slots of (block partial as two words)
  SolveCtl *ctl;
};

// A word's place: a pointer uniform over the wave and a byte offset per lane
// (the exchange buffer is far below 4 GiB, so every word of it is 32 bits
// from one scalar pointer).
struct Word {
  uint64_t *base;
  uint32_t off;
  __device__ __forceinline__ uint64_t *at() const {
    return (uint64_t *)((char *)base + (uint64_t)off);
  }
};

__device__ __forceinline__ void put_word(Word p, uint32_t v, uint32_t tag) {
  __hip_atomic_store(p.at(), ((uint64_t)tag << 32) | v, __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t get_word(Word p) {
  return __hip_atomic_load(p.at(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ bool has_tag(uint64_t w, uint32_t tag) {
  return (uint32_t)(w >> 32) == tag;
}

// One more round of a wait that began at t0 (every 64th looks at the clock):
// false once it has lasted too long or another wait has.
__device__ __forceinline__ bool keep_waiting(uint32_t n, uint64_t &t0, SolveCtl *ctl) {
  if ((n & 63u) != 0) return true;
  const uint64_t t = wall_clock64();
  if (n == 64u) t0 = t;
  const bool late = t - t0 > kSpinTicks;
  if (late) __hip_atomic_store(&ctl->aborted, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return !late && !__hip_atomic_load(&ctl->aborted, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A double that is the same in every lane, held in scalar registers.
__device__ __forceinline__ double uniform(double v) {
  return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                          __builtin_amdgcn_readfirstlane(__double2loint(v)));
}

// 32-bit words of a value.
__device__ __forceinline__ uint32_t word_of(float v, int) { return __float_as_uint(v); }
__device__ __forceinline__ uint32_t word_of(double v, int h) {
  return h ? (uint32_t)__double2hiint(v) : (uint32_t)__double2loint(v);
}
template <typename T>
__device__ __forceinline__ T value_of(const uint32_t *w) {
  if constexpr (sizeof(T) == 4)
    return __uint_as_float(w[0]);
  else
    return __hiloint2double((int)w[1], (int)w[0]);
}

// The value made opaque to the optimiser, at this place in the order of such
// places (no instruction): a conversion to double before it is not the one
// after it, so that no double copy of the resident state is carried along in
// registers, and what is computed from the value stays after it.
__device__ __forceinline__ void forget(float &v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void forget(double &v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void forget(int &v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void forget_uniform(uint32_t &v) { asm volatile("" : "+s"(v)); }
__device__ __forceinline__ void forget_uniform(int &v) { asm volatile("" : "+s"(v)); }

template <typename T, int N>
struct alignas(N * sizeof(T) >= 16 ? 16 : N * sizeof(T)) Vec {
  T v[N];
};

// LDS of a block.
template <class B>
struct Shared {
  using T = typename B::T;
  using V = Vec<T, B::GL>;
  V rhs[B::NV > B::RV ? B::NV - B::RV : 1][kNT];
  // first row of each wave but the first and last row of each but the last,
  // in the group at hand and (not SB) the next (three-dimensional boxes)
  V lo[B::NB][B::D2 ? 1 : kNW - 1][64], hi[B::NB][B::D2 ? 1 : kNW - 1][64];
  // lowest and highest level of each wave, by iterate parity (one-row boxes)
  T zlo[2][B::D2 ? kNW : 1][B::D2 ? 64 : 1], zhi[2][B::D2 ? kNW : 1][B::D2 ? 64 : 1];
  // y and x faces of the group at hand and the next, and those to publish
  V yh[2][2][B::D2 ? 1 : 64], xh[2][2][B::NS];
  V ypub[B::NB][2][B::YLDS && !B::D2 ? 64 : 1], xpub[B::NB][2][B::NS];
  double red[kNW];
  double total;
  int dead;
};

// Boxes split the grid as evenly as whole cells allow: box b of n over len
// cells starts here.
__device__ __forceinline__ int split(int b, int n, int len) {
  return __builtin_amdgcn_readfirstlane((int)((int64_t)b * len / n));  // uniform
}

// Order of the groups in a sweep: the groups holding the bottom and the top
// level neither first nor last when there are four or more.
template <int NG>
__device__ constexpr int group_at(int pos) {
  return NG < 4 ? pos
                : (pos == 0 ? 1 : pos == 1 ? 0 : pos == 2 ? NG - 1 : pos - 1);
}

// f(0), f(1), .. f(N - 1) with compile-time arguments: the resident arrays
// are only ever indexed by constants, so that they are registers from the
// first pass of the optimiser on.
template <class F, int... P>
__device__ __forceinline__ void for_each(F &f, std::integer_sequence<int, P...>) {
  (f(std::integral_constant<int, P>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
  for_each(f, std::make_integer_sequence<int, N>{});
}

// RAG: boxes may hold fewer than 64 columns, R rows per wave or Z levels per
// thread.
template <class B, bool CHEB, bool RAG>
__global__ __launch_bounds__(kNT) void psweep_kernel(PArgs<typename B::T> a) {
  using T = typename B::T;
  using V = Vec<T, B::GL>;
  constexpr int R = B::R, Z = B::Z, GL = B::GL, NG = B::NG, NWD = B::NWD;
  __shared__ Shared<B> sh;
  SolveCtl *const ctl = a.ctl;
  if (ctl->done) return;  // nothing to solve: phi_0 = 0 is in a.out
  const Grid &g = a.g;
  const int lane = (int)(threadIdx.x & 63);
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int bx = (int)blockIdx.x % a.tx, by = (int)blockIdx.x / a.tx % a.ty,
            bz = (int)blockIdx.x / (a.tx * a.ty);
  const int x0 = split(bx, a.tx, g.nx), nw = split(bx + 1, a.tx, g.nx) - x0;
  const int y0b = split(by, a.ty, g.ny), nyb = split(by + 1, a.ty, g.ny) - y0b;
  const int z0b = split(bz, a.tz, g.nz), nzb = split(bz + 1, a.tz, g.nz) - z0b;
  // this wave's rows [y0, y0 + rw) and levels [z0, z0 + lz); the block's
  // waves with rows are 0 .. last
  int y0, rw, z0, lz, last;
  if constexpr (B::D2) {
    y0 = 0;
    rw = 1;
    z0 = z0b + split(wv, kNW, nzb);
    lz = z0b + split(wv + 1, kNW, nzb) - z0;
    last = kNW - 1;
  } else {
    last = min(kNW, nyb) - 1;
    const int w = min(wv, last + 1);
    y0 = y0b + split(w, last + 1, nyb);
    rw = wv <= last ? y0b + split(w + 1, last + 1, nyb) - y0 : 0;
    z0 = z0b;
    lz = nzb;
  }
  rw = __builtin_amdgcn_readfirstlane(rw);
  lz = __builtin_amdgcn_readfirstlane(lz);
  if constexpr (!RAG) {
    rw = R;
    lz = Z;
    last = kNW - 1;
  }
  const bool active = !RAG || lane < nw;
  const int lane_last = RAG ? nw - 1 : 63;
  const bool has_lo = B::D2 ? (wv > 0 || bz > 0) : bz > 0;            // a level below this wave's
  const bool has_hi = B::D2 ? (wv < last || bz + 1 < a.tz) : bz + 1 < a.tz;
  const bool face_lo = has_lo && (!B::D2 || wv == 0);                 // ... in another block
  const bool face_hi = has_hi && (!B::D2 || wv == last);

  // words of this block's faces and of the neighbouring blocks'
  auto face = [&](int x, int y, int z) {
    return (uint32_t)((z * a.ty + y) * a.tx + x) * (uint32_t)(2 * B::FACE);
  };
  const uint32_t own = face(bx, by, bz);
  const uint32_t fxm = face(bx ? bx - 1 : a.tx - 1, by, bz),
                 fxp = face(bx + 1 < a.tx ? bx + 1 : 0, by, bz),
                 fym = face(bx, by ? by - 1 : a.ty - 1, bz),
                 fyp = face(bx, by + 1 < a.ty ? by + 1 : 0, bz),
                 fzm = face(bx, by, bz ? bz - 1 : 0),
                 fzp = face(bx, by, bz + 1 < a.tz ? bz + 1 : bz);
  constexpr int oZlo = 0, oZhi = B::ZF, oYlo = 2 * B::ZF, oYhi = oYlo + B::YF,
                oXlo = oYhi + B::YF, oXhi = oXlo + B::XF;
  static_assert(oXhi + B::XF == B::FACE, "face layout");
  const int zslot = wv * R * 64 * NWD;  // of row 0, lane 0; row r adds 64 r NWD

  // ---- state: phi_m and phi_{m-1} (starting from zero), right-hand side
  T A[R][Z], Bv[R][Z];
  V rr[B::RV > 0 ? B::RV : 1];
  const T *const rhs = a.rhs_kept && ctl->guess_kept ? a.rhs_kept : a.rhs;
  static_for<B::NV>([&](auto ec) __attribute__((always_inline)) {
    constexpr int e = decltype(ec)::value, r = e / NG, K0 = e % NG * GL;
    V v;
    static_for<GL>([&](auto qc) __attribute__((always_inline)) {
      constexpr int q = decltype(qc)::value, k = K0 + q;
      A[r][k] = T(0);
      Bv[r][k] = T(0);
      const bool in = !RAG || (active && r < rw && k < lz);
      v.v[q] = in ? rhs[(int64_t)(x0 + lane) + (int64_t)g.nx * (y0 + r) +
                        g.nxy * (int64_t)(z0 + k)]
                  : T(0);
    });
    if constexpr (e < B::RV)
      rr[e] = v;
    else
      sh.rhs[e - B::RV][threadIdx.x] = v;
  });
  // phi_0 = 0 in every exchange buffer
  {
    uint32_t *z = (uint32_t *)sh.lo;
    const int n = (int)((char *)&sh.red - (char *)sh.lo) / 4;
    for (int q = threadIdx.x; q < n; q += kNT) z[q] = 0u;
    if (threadIdx.x == 0) sh.dead = 0;
  }
  T zl[R], zh[R];  // the level below / above this thread's, per row
  // (set before the launch, by tests only, it makes block 0 one that gave up)
  bool dead = blockIdx.x == 0 && ctl->aborted != 0;
  __syncthreads();

  // the lane, forgotten at every group: addresses are made from it where they
  // are used and not kept
  int ln = lane;
  auto lane8 = [&]() __attribute__((always_inline)) { return (uint32_t)ln * 8u; };

  // ---- faces of the next group: loads, then the wait for their tags
  uint64_t wy[B::YP > 0 ? B::YP : 1], wx[B::XP], wl[R * NWD], wh[R * NWD];
  // the level below wave 0's is the highest of the block below, held by the
  // same wave (three dimensions) or by the last one (one row)
  const int src_lo = (B::D2 ? last : wv) * R * 64 * NWD;
  const int src_hi = (B::D2 ? 0 : wv) * R * 64 * NWD;
  static_assert(B::YN % kNT == 0, "the y faces of a group fill the block");
  // Word q of this thread in a group's y faces, [side][level][lane][half],
  // and in its x faces, [side][slot][level][half]: the side and the run of 64
  // words are uniform over the wave (x faces: where a side has 64 words), so
  // that an address is a scalar plus the lane.
  auto y_run = [&](int q, int *side) __attribute__((always_inline)) {
    const int e = (q * kNW + wv) * 64;
    *side = e >= B::YN / 2;
    return e - *side * (B::YN / 2);
  };
  auto y_word = [&](int q, int gn, uint32_t par) __attribute__((always_inline)) {
    int side;
    const int o = y_run(q, &side);
    const uint32_t w = (side ? fyp + oYlo : fym + oYhi) + (par ? B::FACE : 0) + gn * GL * 64 * NWD + o;
    return Word{a.faces, w * 8u + lane8()};
  };
  constexpr bool kXRuns = B::XN / 2 % 64 == 0;
  auto x_run = [&](int q, int *side) __attribute__((always_inline)) {
    constexpr int H = B::XN / 2;
    if constexpr (kXRuns) {
      const int e = (q * kNW + wv) * 64;
      *side = e >= H;
      return e - *side * H;  // of lane 0
    } else {
      const int e = min((q * kNW + wv) * 64 + ln, B::XN - 1);
      *side = e >= H;
      return e - *side * H;
    }
  };
  auto x_has = [&](int q) __attribute__((always_inline)) { return (q * kNW + wv) * 64 < B::XN; };
  auto x_word = [&](int q, int gn, uint32_t par) __attribute__((always_inline)) {
    int side;
    const int o = x_run(q, &side), p = (par ? B::FACE : 0) + gn * (B::XN / 2);
    return Word{a.faces, ((side ? fxp + oXlo : fxm + oXhi) + (p + o)) * 8u + (kXRuns ? lane8() : 0u)};
  };
  // group gn holds this wave's bottom level (need_lo) or its top one
  auto need_lo = [&](int gn) __attribute__((always_inline)) { return gn == 0 && face_lo; };
  auto need_hi = [&](int gn) __attribute__((always_inline)) {
    return face_hi && (RAG ? (lz - 1) / GL == gn : gn == NG - 1);
  };
  auto lo_word = [&](int q, uint32_t par) __attribute__((always_inline)) {
    const uint32_t w = fzm + oZhi + (par ? B::FACE : 0) + src_lo + q / NWD * 64 * NWD + q % NWD;
    return Word{a.faces, w * 8u + lane8() * NWD};
  };
  auto hi_word = [&](int q, uint32_t par) __attribute__((always_inline)) {
    const uint32_t w = fzp + oZlo + (par ? B::FACE : 0) + src_hi + q / NWD * 64 * NWD + q % NWD;
    return Word{a.faces, w * 8u + lane8() * NWD};
  };
  auto issue = [&](int gn, uint32_t t) __attribute__((always_inline)) {
    const uint32_t par = t & 1u;
    if constexpr (!B::D2)
#pragma unroll
      for (int q = 0; q < B::YP; ++q) wy[q] = get_word(y_word(q, gn, par));
#pragma unroll
    for (int q = 0; q < B::XP; ++q)
      if (x_has(q)) wx[q] = get_word(x_word(q, gn, par));
    if (need_lo(gn))
#pragma unroll
      for (int q = 0; q < R * NWD; ++q) wl[q] = get_word(lo_word(q, par));
    if (need_hi(gn))
#pragma unroll
      for (int q = 0; q < R * NWD; ++q) wh[q] = get_word(hi_word(q, par));
  };
  // ... until every word of the wave has its tag (all are read again until
  // then); pp: LDS slot the group's y and x faces go to
  auto collect = [&](int gn, uint32_t t, int pp) __attribute__((always_inline)) {
    uint64_t t0 = 0;
    for (uint32_t n = 1; !dead; ++n) {
      bool ok = true;
      if constexpr (!B::D2)
#pragma unroll
        for (int q = 0; q < B::YP; ++q) ok &= has_tag(wy[q], t);
#pragma unroll
      for (int q = 0; q < B::XP; ++q)
        if (x_has(q)) ok &= has_tag(wx[q], t);
      if (need_lo(gn))
#pragma unroll
        for (int q = 0; q < R * NWD; ++q) ok &= has_tag(wl[q], t);
      if (need_hi(gn))
#pragma unroll
        for (int q = 0; q < R * NWD; ++q) ok &= has_tag(wh[q], t);
      if (__all(ok)) break;
      if (!keep_waiting(n, t0, ctl)) dead = true;
      issue(gn, t);
    }
    if constexpr (!B::D2)
#pragma unroll
      for (int q = 0; q < B::YP; ++q) {
        // word e of [side][level][column][half] to [side][column][level][half]
        const int e = q * kNT + wv * 64 + ln;
        const int h = e % NWD, c = e / NWD % 64, l = e / (64 * NWD) % GL, side = e / (64 * NWD * GL);
        ((uint32_t *)&sh.yh[pp][0][0].v[0])[((side * 64 + c) * GL + l) * NWD + h] = (uint32_t)wy[q];
      }
#pragma unroll
    for (int q = 0; q < B::XP; ++q)
      if (x_has(q)) {
        const int e = min(q * kNT + wv * 64 + ln, B::XN - 1);  // [side][slot][level][half]
        ((uint32_t *)&sh.xh[pp][0][0].v[0])[e] = (uint32_t)wx[q];
      }
    uint32_t v[NWD];
    if (need_lo(gn))
#pragma unroll
      for (int r = 0; r < R; ++r) {
#pragma unroll
        for (int h = 0; h < NWD; ++h) v[h] = (uint32_t)wl[r * NWD + h];
        zl[r] = value_of<T>(v);
      }
    if (need_hi(gn))
#pragma unroll
      for (int r = 0; r < R; ++r) {
#pragma unroll
        for (int h = 0; h < NWD; ++h) v[h] = (uint32_t)wh[r * NWD + h];
        zh[r] = value_of<T>(v);
      }
  };

  // phi_0 = 0 in the levels of group gn's neighbours
  auto start_levels = [&](int gn) __attribute__((always_inline)) {
    if (need_lo(gn)) static_for<R>([&](auto rc) __attribute__((always_inline)) { zl[rc] = T(0); });
    if (need_hi(gn)) static_for<R>([&](auto rc) __attribute__((always_inline)) { zh[rc] = T(0); });
  };
  start_levels(group_at<NG>(0));

  double acc[R], wc = 1.0;  // residual sum of each row
  int pp = 0;  // LDS slot of the faces of the group at hand
  constexpr bool kOne = B::SB;

  // ---- one group of sweep m: Cur = phi_m (tag t), Nxt = phi_{m-1} in,
  // phi_{m+1} out
  auto compute = [&](auto gc, T(&Cur)[R][Z], T(&Nxt)[R][Z], uint32_t t)
                     __attribute__((always_inline)) {
    constexpr int gi = decltype(gc)::value, K0 = gi * GL;
    if (RAG && (rw == 0 || K0 >= lz)) return;
    // LDS operands, SL levels at a time
    constexpr int SL = B::SL, RV = B::RV;
    using P = Vec<T, SL>;
    const int rp = kOne ? 0 : pp;
    const P *const plo = (const P *)(wv == 0 || B::D2 ? &sh.yh[pp][0][ln] : &sh.hi[rp][wv - 1][ln]);
    const P *const phi = (const P *)(wv == last || B::D2 ? &sh.yh[pp][1][ln]
                                                         : &sh.lo[rp][min(wv, kNW - 2)][ln]);
    const P *const px = (const P *)&sh.xh[pp][ln == 0 ? 0 : 1][wv * R];
    P ylo, yhi, xe[R], rv[R];
    double c[R], b[R];
    static_for<R>([&](auto rc) __attribute__((always_inline)) {
      constexpr int r = decltype(rc)::value;
      c[r] = (double)Cur[r][K0];
      if constexpr (K0 > 0) {
        b[r] = (double)Cur[r][K0 > 0 ? K0 - 1 : 0];
      } else if constexpr (B::D2) {
        b[r] = !has_lo ? c[r] : (double)(face_lo ? zl[r] : sh.zhi[t & 1u][wv - (wv > 0)][ln]);
      } else {
        b[r] = has_lo ? (double)zl[r] : c[r];
      }
    });
    // the value above the top level, v its own
    auto above_top = [&](auto rc, T v) __attribute__((always_inline)) {
      if constexpr (B::D2)
        return !has_hi ? v : face_hi ? zh[rc] : sh.zlo[t & 1u][min(wv + 1, kNW - 1)][ln];
      else
        return has_hi ? zh[rc] : v;
    };
    static_for<GL>([&](auto qc) __attribute__((always_inline)) {
      constexpr int q = decltype(qc)::value, k = K0 + q, l = q % SL;
      if (RAG && k >= lz) return;
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (l == 0) {
        if constexpr (!B::D2) {
          ylo = plo[q / SL];
          yhi = phi[q / SL];
        }
        static_for<R>([&](auto rc) __attribute__((always_inline)) {
          constexpr int r = decltype(rc)::value, e = r * NG + gi;
          xe[r] = px[r * (GL / SL) + q / SL];
          if constexpr (e >= RV)
            rv[r] = ((const P *)&sh.rhs[e - RV][wv * 64 + ln])[q / SL];
          else
            static_for<SL>([&](auto lc) __attribute__((always_inline)) {
              rv[r].v[lc] = rr[e].v[q + decltype(lc)::value];
              forget(rv[r].v[lc]);
            });
        });
      }
      static_for<R>([&](auto rc) __attribute__((always_inline)) { forget(Cur[rc][k]); });
      if constexpr (RAG && k + 1 < Z) {
        // a box with fewer levels keeps the level above its top in the first
        // register past it
        if (k == lz - 1) {
          static_for<R>([&](auto rc) __attribute__((always_inline)) {
            Cur[rc][k + 1 < Z ? k + 1 : 0] = above_top(rc, Cur[rc][k]);
            forget(Cur[rc][k + 1 < Z ? k + 1 : 0]);
          });
        }
      }
      double ym = 0.0;  // the row before this one
      static_for<R>([&](auto rc) __attribute__((always_inline)) {
        constexpr int r = decltype(rc)::value;
        double ab;
        if constexpr (k + 1 < Z)
          ab = (double)Cur[r][k + 1 < Z ? k + 1 : k];
        else
          ab = (double)above_top(rc, Cur[r][k]);
        const T v = Cur[r][k], edge = xe[r].v[l];
        const T xm = lane_shift<-1>(v, edge);
        T xp = lane_shift<1>(v, edge);
        if (RAG) xp = ln == lane_last ? edge : xp;
        double hy;
        if constexpr (B::D2) {
          hy = c[r] + c[r];
        } else {
          if (r == 0) ym = (double)ylo.v[l];
          double yp = r == R - 1 ? (double)yhi.v[l] : c[r + 1 < R ? r + 1 : r];
          if (RAG && r < R - 1) yp = r == rw - 1 ? (double)yhi.v[l] : yp;
          hy = yp + ym;
        }
        const double res = point_residual(a.k, c[r], (double)xp + (double)xm, hy, ab + b[r],
                                          (double)rv[r].v[l]);
        acc[r] += res * res;
        Nxt[r][k] = (T)point_update(a.k, c[r], res, CHEB, CHEB ? (double)Nxt[r][k] : 0.0, wc);
        ym = c[r];
        b[r] = c[r];
        c[r] = ab;
      });
      static_for<R>([&](auto rc) __attribute__((always_inline)) { forget(Nxt[rc][k]); });
      static_for<R>([&](auto rc) __attribute__((always_inline)) { forget(acc[rc]); });
    });
    static_for<R>([&](auto rc) __attribute__((always_inline)) {
      if constexpr (K0 > 0) forget(Cur[rc][K0 > 0 ? K0 - 1 : 0]);
      if constexpr (K0 + GL < Z) forget(Cur[rc][K0 + GL < Z ? K0 + GL : 0]);
    });
  };
  // value of level lz - 1 of row r, which group gi holds
  auto top_of = [&](auto gc, auto rc, T(&F)[R][Z]) __attribute__((always_inline)) {
    constexpr int K0 = decltype(gc)::value * GL;
    T v = F[rc][K0 + GL - 1];
    if (RAG)
      static_for<GL - 1>([&](auto qc) __attribute__((always_inline)) {
        v = lz - 1 == K0 + decltype(qc)::value ? F[rc][K0 + decltype(qc)::value] : v;
      });
    return v;
  };
  // value of this wave's last row at level k
  auto last_row = [&](auto kc, T(&F)[R][Z]) __attribute__((always_inline)) {
    T v = F[R - 1][kc];
    if (RAG)
      static_for<R - 1>([&](auto rc) __attribute__((always_inline)) {
        v = decltype(rc)::value == rw - 1 ? F[rc][kc] : v;
      });
    return v;
  };
  // the group's faces of phi_{m+1} (tag t) to the neighbouring blocks; the x
  // faces (and y faces, YLDS) as far as LDS, from where all threads store them
  auto publish = [&](auto gc, T(&Nxt)[R][Z], uint32_t t) __attribute__((always_inline)) {
    constexpr int gi = decltype(gc)::value, K0 = gi * GL;
    const uint32_t to = own + ((t & 1u) ? B::FACE : 0);
    auto put = [&](uint32_t p, T v) __attribute__((always_inline)) {  // p: word of lane 0
#pragma unroll
      for (int h = 0; h < NWD; ++h)
        put_word(Word{a.faces, (p + h) * 8u + lane8() * NWD}, word_of(v, h), t);
    };
    if (need_lo(gi))
      static_for<R>([&](auto rc) __attribute__((always_inline)) {
        put(to + (oZlo + zslot + rc * 64 * NWD), Nxt[rc][0]);
      });
    if (need_hi(gi))
      static_for<R>([&](auto rc) __attribute__((always_inline)) {
        put(to + (oZhi + zslot + rc * 64 * NWD), top_of(gc, rc, Nxt));
      });
    if constexpr (B::D2) {
      if (gi == 0) sh.zlo[t & 1u][wv][ln] = Nxt[0][0];
      if (RAG ? (lz - 1) / GL == gi : gi == NG - 1)
        sh.zhi[t & 1u][wv][ln] = top_of(gc, std::integral_constant<int, 0>{}, Nxt);
    } else {
      if constexpr (B::YLDS) {
        V v;
        if (wv == 0) {
          static_for<GL>([&](auto qc) __attribute__((always_inline)) {
            v.v[qc] = Nxt[0][K0 + decltype(qc)::value];
          });
          sh.ypub[kOne ? 0 : pp][0][ln] = v;
        }
        if (wv == last) {
          static_for<GL>([&](auto qc) __attribute__((always_inline)) {
            constexpr int k = K0 + decltype(qc)::value;
            v.v[qc] = last_row(std::integral_constant<int, k>{}, Nxt);
          });
          sh.ypub[kOne ? 0 : pp][1][ln] = v;
        }
      } else {
        if (wv == 0)
          static_for<GL>([&](auto qc) __attribute__((always_inline)) {
            constexpr int k = K0 + decltype(qc)::value;
            put(to + (oYlo + k * 64 * NWD), Nxt[0][k]);
          });
        if (wv == last)
          static_for<GL>([&](auto qc) __attribute__((always_inline)) {
            constexpr int k = K0 + decltype(qc)::value;
            put(to + (oYhi + k * 64 * NWD), last_row(std::integral_constant<int, k>{}, Nxt));
          });
      }
    }
    if (ln == 0 || ln == lane_last)
      static_for<R>([&](auto rc) __attribute__((always_inline)) {
        V v;
        static_for<GL>([&](auto qc) __attribute__((always_inline)) {
          v.v[qc] = Nxt[rc][K0 + decltype(qc)::value];
        });
        sh.xpub[kOne ? 0 : pp][ln == 0 ? 0 : 1][wv * R + rc] = v;
      });
  };
  // after the barrier: the x and y faces from LDS
  auto publish_xy = [&](auto gc, uint32_t t) __attribute__((always_inline)) {
    constexpr int gi = decltype(gc)::value;
    const uint32_t to = own + ((t & 1u) ? B::FACE : 0);
    if constexpr (!B::D2 && B::YLDS)
#pragma unroll
      for (int q = 0; q < B::YP; ++q) {
        // word e of [side][level][column][half] from [side][column][level][half]
        const int e = q * kNT + wv * 64 + ln;
        const int h = e % NWD, c = e / NWD % 64, l = e / (64 * NWD) % GL, side = e / (64 * NWD * GL);
        const uint32_t v =
            ((const uint32_t *)&sh.ypub[kOne ? 0 : pp][0][0].v[0])[((side * 64 + c) * GL + l) * NWD + h];
        int us;
        const int o = y_run(q, &us);
        put_word(Word{a.faces, (to + (us ? oYhi : oYlo) + gi * GL * 64 * NWD + o) * 8u + lane8()}, v,
                 t);
      }
#pragma unroll
    for (int q = 0; q < B::XP; ++q)
      if (x_has(q)) {
        int side;
        const int o = x_run(q, &side);
        const uint32_t at = to + (side ? oXhi : oXlo) + gi * (B::XN / 2) + o;
        const int e = min(q * kNT + wv * 64 + ln, B::XN - 1);
        const uint32_t v = ((const uint32_t *)&sh.xpub[kOne ? 0 : pp][0][0].v[0])[e];
        put_word(Word{a.faces, at * 8u + (kXRuns ? lane8() : 0u)}, v, t);
      }
  };
  // before it: the wave's first and last row of group gc for the waves beside
  // it
  auto pass_rows = [&](auto gc, T(&F)[R][Z]) __attribute__((always_inline)) {
    constexpr int K0 = decltype(gc)::value * GL;
    if constexpr (!B::D2) {
      V v;
      static_for<GL>([&](auto qc) __attribute__((always_inline)) {
        v.v[qc] = F[0][K0 + decltype(qc)::value];
      });
      if (wv > 0) sh.lo[kOne ? 0 : pp ^ 1][wv > 0 ? wv - 1 : 0][ln] = v;
      static_for<GL>([&](auto qc) __attribute__((always_inline)) {
        constexpr int k = K0 + decltype(qc)::value;
        v.v[qc] = last_row(std::integral_constant<int, k>{}, F);
      });
      if (wv < kNW - 1) sh.hi[kOne ? 0 : pp ^ 1][wv < kNW - 1 ? wv : 0][ln] = v;
    }
  };
  // a whole sweep m
  auto sweep = [&](T(&Cur)[R][Z], T(&Nxt)[R][Z], uint32_t t, bool first)
                   __attribute__((always_inline)) {
    auto position = [&](auto pc) __attribute__((always_inline)) {
      constexpr int pos = decltype(pc)::value;
      constexpr int gi = group_at<NG>(pos), gn = group_at<NG>((pos + 1) % NG);
      const std::integral_constant<int, gi> gc{};
      constexpr bool wraps = pos + 1 == NG;
      if (pos == 0) static_for<R>([&](auto rc) __attribute__((always_inline)) { acc[rc] = 0.0; });
      const bool take = wraps || !first;  // phi_0 = 0 needs no exchange
      const uint32_t tn = wraps ? t + 1 : t;
      forget(ln);
      if (RAG) {
        forget_uniform(lz);
        forget_uniform(rw);
      }
      if (NG > 1 && take) issue(gn, tn);
      compute(gc, Cur, Nxt, t);
      publish(gc, Nxt, t + 1);
      if (!B::SB) pass_rows(std::integral_constant<int, gn>{}, wraps ? Nxt : Cur);
      if (NG > 1) {
        if (take) collect(gn, tn, pp ^ 1);
        else start_levels(gn);
      }
      __syncthreads();
      if (B::SB) pass_rows(std::integral_constant<int, gn>{}, wraps ? Nxt : Cur);
      publish_xy(gc, t + 1);
      if (B::SB) __syncthreads();
      if constexpr (NG == 1) {
        // A face just published takes most of a microsecond to be seen, and a
        // read that comes too early costs a whole round trip more.  Pauses of
        // 0, 0.1, 0.2, 0.3, 0.4 us: 1.82, 1.74, 1.70, 1.79, 1.90 us per sweep
        // at 64 x 64 x 64 FP32.
        __builtin_amdgcn_s_sleep(8);
        issue(gn, tn);
        collect(gn, tn, pp ^ 1);
        __syncthreads();
      }
      pp ^= 1;
    };
    forget_uniform(t);
    static_for<NG>(position);
  };

  const int fixed = __builtin_amdgcn_readfirstlane(ctl->fixed),
            max_sweeps = __builtin_amdgcn_readfirstlane(ctl->max_sweeps);
  int done = 0, nchecks = 0;
  double s = 0.0;
  // the residual test of sweep m, the same in every block (true: stop)
  auto decide = [&](int m, uint32_t t) -> bool {
    const int nb = (int)gridDim.x;
    uint64_t *const red = a.red + (nchecks & 1) * 2 * nb;
    ++nchecks;
    double v = 0.0;
    static_for<R>([&](auto rc) __attribute__((always_inline)) {
      if (!RAG || (active && rc < rw)) v += acc[rc];
    });
    v = wave_sum(v);
    if (lane == 0) sh.red[wv] = v;
    if (dead) sh.dead = 1;
    __syncthreads();
    if (threadIdx.x < 2) {
      double p = 0.0;
      for (int q = 0; q < kNW; ++q) p += sh.red[q];
      put_word(Word{red + 2 * blockIdx.x, (uint32_t)threadIdx.x * 8u}, word_of(p, (int)threadIdx.x),
               t);
    }
    v = 0.0;
    if (wv * 64 < nb) {
      const Word p0{red, (uint32_t)min((int)threadIdx.x, nb - 1) * 16u}, p1{red + 1, p0.off};
      uint64_t w0 = get_word(p0), w1 = get_word(p1), t0 = 0;
      for (uint32_t n = 1; !dead && !__all(has_tag(w0, t) && has_tag(w1, t)); ++n) {
        if (!keep_waiting(n, t0, ctl)) dead = true;
        w0 = get_word(p0);
        w1 = get_word(p1);
      }
      const uint32_t w[2] = {(uint32_t)w0, (uint32_t)w1};
      if ((int)threadIdx.x < nb) v = value_of<double>(w);
    }
    v = wave_sum(v);
    __syncthreads();  // sh.red was read
    if (lane == 0) sh.red[wv] = v;
    if (dead) sh.dead = 1;
    __syncthreads();
    s = 0.0;
    for (int q = 0; q < kNW; ++q) s += sh.red[q];
    const bool stop = sh.dead != 0;
    const double tol2 = ctl->tol2;
    __syncthreads();
    if (!isfinite(s)) {
      done = 2;
    } else if (fixed) {
      if (m >= max_sweeps) done = s <= tol2 ? 1 : 3;
    } else if (s <= tol2) {
      done = 1;
    } else if (m >= max_sweeps) {
      done = 3;
    }
    return stop || done;
  };
  auto weight = [&](int m) {
#pragma clang fp contract(off)
    if (!CHEB || m == 0) return 1.0;
    return m == 1 ? a.w1 : 1.0 / (1.0 - a.q * wc);
  };
  auto tested = [&](int m) {
    return m == max_sweeps || (!fixed && m % a.every == 0);
  };
  auto finish = [&](T(&Cur)[R][Z], int m) __attribute__((always_inline)) {
    int lane_o = lane;  // addresses made here, not kept from the loads of rhs
    forget(lane_o);
    static_for<R * Z>([&](auto ec) __attribute__((always_inline)) {
      constexpr int r = decltype(ec)::value / Z, k = decltype(ec)::value % Z;
      if (!RAG || (active && r < rw && k < lz))
        a.out[(int64_t)(x0 + lane_o) + (int64_t)g.nx * (y0 + r) + g.nxy * (int64_t)(z0 + k)] =
            Cur[r][k];
    });
    if (blockIdx.x == 0 && threadIdx.x == 0 && done) {
      ctl->res_norm2 = s;
      ctl->done = done;
      ctl->stop_m = m;
    }
  };
  for (int m = 0;; m += 2) {
    bool check = tested(m);
    wc = uniform(weight(m));
    sweep(A, Bv, a.base + m, m == 0);
    if (check && decide(m, a.base + m)) return finish(A, m);
    check = tested(m + 1);
    wc = uniform(weight(m + 1));
    sweep(Bv, A, a.base + m + 1, false);
    if (check && decide(m + 1, a.base + m + 1)) return finish(Bv, m + 1);
  }
}

// Box shapes, 2048 to 32768 cells (64 x 8 x 4 to 64 x 16 x 32; one row 64 x 32
// or 64 x 256); FP64 fills the registers at half of that.  FP64 takes one row
// per thread where it can: every thread reads the z faces of its rows, two
// words a value.  Longer groups mean fewer exchanges: 8 levels instead of 4
// took 256 x 256 x 64 FP32 from 6.2 to 4.9 us per sweep, 256 x 256 x 128 from
// 11.4 to 10.5 and 250 x 200 x 100 (ragged boxes) from 13.1 to 11; 4 instead of
// 2 the ragged largest FP64 boxes (250 x 200 x 60) from 12.4 to 10.8 but the
// full ones (256 x 256 x 64) from 11.7 to 12.4.  64 x 8 x 8 boxes instead of 64
// x 16 x 4 took 128 x 128 x 64 FP64 from 7.3 to 5.8, 64 x 8 x 16 instead of 64 x
// 16 x 8 200 x 120 x 60 from 8.4 to 6.2.
template <typename T>
struct Shapes {
  static constexpr bool F32 = sizeof(T) == 4;
  using S = Box<T, 1, 4, 4, false, 1>;
  using M1 = Box<T, 1, 8, F32 ? 8 : 4, false, 2>;
  using M2 = std::conditional_t<F32, Box<T, 2, 8, 8, false, 2>, Box<T, 1, 16, 4, false, 1>>;
  using M3 = Box<T, 2, 16, F32 ? 8 : 2, false, 1>;
  using M3Rag = Box<T, 2, 16, F32 ? 8 : 4, false, 1>;
  using L = std::conditional_t<F32, Box<T, 2, 32, 8, false, 1>, M3>;  // FP32 only
  using LRag = std::conditional_t<F32, L, M3Rag>;
  using RowL = Box<T, 1, 32, 4, true, 4>;
  using RowS = Box<T, 1, 4, 4, true, 1>;
};

// Launches psweep_kernel<B, ...>; the kernels are built in translation units
// of their own (LES_RESIDENT).
template <class B, bool CHEB, bool RAG>
hipError_t launch_box(const PArgs<typename B::T> &a, int nb, hipStream_t s);

#define LES_RESIDENT(B, CHEB, RAG)                                                              \
  template <>                                                                                   \
  hipError_t launch_box<B, CHEB, RAG>(const PArgs<typename B::T> &a, int nb, hipStream_t s) {   \
    PArgs<typename B::T> args = a;                                                              \
    void *params[] = {&args};                                                                   \
    return hipLaunchCooperativeKernel((const void *)psweep_kernel<B, CHEB, RAG>, dim3(nb),      \
                                      dim3(kNT), params, 0, s);                                 \
  }

}  // namespace resident
}  // namespace lesmi
