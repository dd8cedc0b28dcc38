// mg_tail.hip -- the coarse tail: every level <= 16^3 of one hierarchy in one workgroup.
//
// A V-cycle from 16^3 is some forty dependent phases of at most 4096 cells; its time is the
// latency of those phases, never bytes or flops.  So each phase is made short:
//   16^3  a thread holds four cells of a z-column in registers, two per colour (cell (x, y, z)
//         of colour c at z = 2q + parity).  Within one colour array the x and y neighbours of
//         slot q are slot q of the neighbouring columns, so x-neighbours are DPP row rotations
//         (16 lanes = one row of 16 cells), y-neighbours one 16-byte LDS read each, and of the
//         z-neighbours all but one are the thread's own registers: 3 LDS reads for the two
//         cells of a half-sweep, against 16 reads of 8 bytes with two-way bank conflicts when
//         a thread gathers six neighbours, itself and f for each cell.
//   8^3   the same by four waves, two cells of a column per thread (one per colour): one slot a
//         thread, five LDS reads per half-sweep.
//   4^3 .. 1^3  in 16 lanes of the first wave, a column of four (two) cells per lane: every
//         neighbour is a register or a DPP move within the row of 16 lanes, so these levels touch
//         no LDS and no barrier.  2^3 keeps its four columns in the lanes of the 4^3 columns they
//         restrict.
// Scaled unknowns: fs = -h^2 f (+ 2b at a face with value b), so that the smoother is
// u += (omega/6) r with r = (neighbours + fs) - (6 - kappa) u, -h^2 times the defect, kappa the
// sum over the cell's walls of the ghost's factor on its own value (a wall neighbour reads a
// zero slot).  The restricted defect in the coarse level's scaling is half the sum of the
// eight r, with no h anywhere below the top.
// FMG (Alg. 2) builds the lower sources itself and takes the tricubic prolongation from a
// ghost-filled copy of the level below in LDS.  Times: see launch_tail.
#include <algorithm>
#include <cstring>

#include "mg_common.h"
#include "mg_launch.h"

namespace mg {

namespace {

constexpr int kThreads = 1024;
constexpr int kSmallCells = 585;   // levels 0..3 back to back
constexpr int kOff1 = 1, kOff2 = 9, kOff3 = 73;
constexpr int kPadCells = 10 * 10 * 10;

// start of level l <= 3 in the back-to-back arrays: (8^l - 1) / 7
__device__ __forceinline__ int level_offset(int l) { return ((1 << (3 * l)) - 1) / 7; }

template <typename T>
struct TailMem {
  typedef T v2 __attribute__((ext_vector_type(2)));
  v2 x[2][kThreads + 1];   // 16^3: per colour, the two slots of every thread; the last is zero
  T x3[2][256 + 1];        // 8^3: per colour, every thread's cell; the last is zero
  T us[kSmallCells];       // levels 0..3: solutions between levels
  T fs[kSmallCells];
  T pad[kPadCells];        // FMG: the coarse level with its ghosts
  double red[kThreads / 64];
};

// The value of another lane of the row of 16 by a DPP control: 0x121 the lane to the left, cyclic
// (0x12f the right); quad permutations below 0x100.
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xf, 0xf, false);
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xf, 0xf, false);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
constexpr int kLeft = 0x121, kRight = 0x12f;            // rows of 16
constexpr int kQuadLeft = 0x93, kQuadRight = 0x39;      // quads: x of the 4^3 level
constexpr int kUp4 = 0x124, kDown4 = 0x12c, kFlip8 = 0x128;   // lane - 4, lane + 4, lane ^ 8
constexpr int kFlip1 = 0xb1, kFlip2 = 0x4e;             // lane ^ 1, lane ^ 2
constexpr int kEven = 0xa0, kOther = 0x0a;              // lanes (0, 0, 2, 2), (2, 2, 0, 0) of the quad

// 2b summed over the faces with values that cell (i, j, k) of a level of n cells touches
__device__ __forceinline__ double face_terms(const LevelBC& bc, int n, int i, int j, int k) {
  double s = 0.0;
  if (i == 0 && bc_has_value(bc.kind[0])) s += 2.0 * face_b(bc, 0, n, j, k);
  if (i == n - 1 && bc_has_value(bc.kind[1])) s += 2.0 * face_b(bc, 1, n, j, k);
  if (j == 0 && bc_has_value(bc.kind[2])) s += 2.0 * face_b(bc, 2, n, i, k);
  if (j == n - 1 && bc_has_value(bc.kind[3])) s += 2.0 * face_b(bc, 3, n, i, k);
  if (k == 0 && bc_has_value(bc.kind[4])) s += 2.0 * face_b(bc, 4, n, i, j);
  if (k == n - 1 && bc_has_value(bc.kind[5])) s += 2.0 * face_b(bc, 5, n, i, j);
  return s;
}

// WALLS: some face of the hierarchy is not periodic.
template <typename T, bool WALLS, bool FMG>
__global__ void __launch_bounds__(kThreads) k_tail(TailArgs a) {
  using v2 = typename TailMem<T>::v2;
  __shared__ TailMem<T> m;
  const int t = threadIdx.x, wave = t >> 6;
  const int top = a.top, npre = a.npre, npost = a.npost;
  if (FMG && a.clock && t == 0) *a.clock = (unsigned long long)wall_clock64();
  const T w6 = (T)(a.omega / 6.0);
  // the ghost's factor on the boundary cell's own value per face (0: periodic)
  T kap[6];
#pragma unroll
  for (int f = 0; f < 6; ++f)
    kap[f] = a.hom.kind[f] == BC_PERIODIC ? (T)0 : (a.hom.kind[f] == BC_ZERO_GRADIENT ? (T)1 : (T)-1);
  // the single cell (Sec. 2.3.2): every neighbour is its own ghost, (6 - sum of factors) u = fs;
  // u = 0 when no face fixes the zero point
  T b0 = (T)6;
#pragma unroll
  for (int f = 0; f < 6; ++f) b0 -= kap[f] == (T)0 ? (T)1 : kap[f];

  // ---- 16^3: the thread's column and its neighbours' slots
  const int x = t & 15, y = (t >> 4) & 15, zq = t >> 8, p = (x + y) & 1;
  int ym = (t & ~0xf0) | (((y - 1) & 15) << 4), yp = (t & ~0xf0) | (((y + 1) & 15) << 4);
  int zdn = 2 * ((t - 256) & 1023) + 1, zup = 2 * ((t + 256) & 1023);   // element indices
  T bR[2] = {(T)6, (T)6}, bB[2] = {(T)6, (T)6};   // 6 - kappa of the red and the black cells
  bool wxl = false, wxh = false;
  if (WALLS) {
    wxl = x == 0 && kap[0] != (T)0;
    wxh = x == 15 && kap[1] != (T)0;
    T k = (wxl ? kap[0] : (T)0) + (wxh ? kap[1] : (T)0);
    if (y == 0 && kap[2] != (T)0) { ym = kThreads; k += kap[2]; }
    if (y == 15 && kap[3] != (T)0) { yp = kThreads; k += kap[3]; }
    bR[0] -= k; bR[1] -= k; bB[0] -= k; bB[1] -= k;
    if (zq == 0 && kap[4] != (T)0) {
      zdn = 2 * kThreads;
      if (p) bB[0] -= kap[4]; else bR[0] -= kap[4];
    }
    if (zq == 3 && kap[5] != (T)0) {
      zup = 2 * kThreads;
      if (p) bR[1] -= kap[5]; else bB[1] -= kap[5];
    }
  }
  const int zR = p ? zup : zdn, zB = p ? zdn : zup;
  T R[2] = {(T)0, (T)0}, B[2] = {(T)0, (T)0}, fR[2] = {(T)0, (T)0}, fB[2] = {(T)0, (T)0};

  // r of the thread's two cells `own` (slot parity s: z = 2q + s); `oth` their in-column
  // neighbours of the other colour, whose slots of all columns are in xo
  auto resid16 = [&](const T* own, const T* oth, const T* fs, const T* b, const v2* xo, int zext, bool s, T* r)
      __attribute__((always_inline)) {
    const v2 a0 = xo[ym], a1 = xo[yp];
    const T ext = reinterpret_cast<const T*>(xo)[zext];
    const T z0 = s ? oth[1] : ext, z1 = s ? ext : oth[0];
    T l0 = dpp<kLeft>(oth[0]), l1 = dpp<kLeft>(oth[1]), h0 = dpp<kRight>(oth[0]), h1 = dpp<kRight>(oth[1]);
    if (WALLS) {
      l0 = wxl ? (T)0 : l0; l1 = wxl ? (T)0 : l1;
      h0 = wxh ? (T)0 : h0; h1 = wxh ? (T)0 : h1;
    }
    r[0] = ((((l0 + h0) + (a0.x + a1.x)) + (oth[0] + z0)) + fs[0]) - b[0] * own[0];
    r[1] = ((((l1 + h1) + (a0.y + a1.y)) + (oth[1] + z1)) + fs[1]) - b[1] * own[1];
  };
  // zero: u is zero, and the first red half-sweep reads nothing
  auto sweeps16 = [&](int count, bool zero) __attribute__((always_inline)) {
#pragma unroll 1
    for (int it = 0; it < count; ++it) {
      T r[2] = {fR[0], fR[1]};
      if (!(zero && it == 0)) resid16(R, B, fR, bR, m.x[1], zR, p != 0, r);
      R[0] += w6 * r[0];
      R[1] += w6 * r[1];
      m.x[0][t] = v2{R[0], R[1]};
      __syncthreads();
      resid16(B, R, fB, bB, m.x[0], zB, p == 0, r);
      B[0] += w6 * r[0];
      B[1] += w6 * r[1];
      m.x[1][t] = v2{B[0], B[1]};
      __syncthreads();
    }
  };
  // half the sum over the eight children of column values v[q] (the two cells of coarse plane
  // 2 zq + q added), into fs of the 8^3 level
  auto restrict16 = [&](T v0, T v1) __attribute__((always_inline)) {
    v0 += dpp<kFlip1>(v0);
    v1 += dpp<kFlip1>(v1);
    v0 += __shfl_xor(v0, 16, 64);
    v1 += __shfl_xor(v1, 16, 64);
    if (((x | y) & 1) == 0) {
      const int C = kOff3 + (x >> 1) + ((y >> 1) << 3) + (zq << 7);
      m.fs[C] = (T)0.5 * v0;
      m.fs[C + 64] = (T)0.5 * v1;
    }
  };

  // ---- 8^3: threads 0..255, the pair of cells z = 2 q3, 2 q3 + 1 of column (x3, y3).  Each level's
  // constants are made when it is entered (from an index the compiler cannot see through, or it
  // would make them all before the first level and spill)
  const bool on3 = t < 256;
  int x3, y3, q3, p3, n3[4], zR3, zB3;
  T bR3, bB3;
  auto place8 = [&]() __attribute__((always_inline)) {
    int o = t;
    asm volatile("" : "+v"(o));
    x3 = o & 7;
    y3 = (o >> 3) & 7;
    q3 = (o >> 6) & 3;
    p3 = (x3 + y3) & 1;
    n3[0] = (o & ~7) | ((x3 - 1) & 7);
    n3[1] = (o & ~7) | ((x3 + 1) & 7);
    n3[2] = (o & ~0x38) | (((y3 - 1) & 7) << 3);
    n3[3] = (o & ~0x38) | (((y3 + 1) & 7) << 3);
    int dn3 = (o - 64) & 255, up3 = (o + 64) & 255;
    bR3 = bB3 = (T)6;
    if (WALLS) {
      const int zero = 256;
      const bool at[4] = {x3 == 0, x3 == 7, y3 == 0, y3 == 7};
      T k = (T)0;
#pragma unroll
      for (int f = 0; f < 4; ++f)
        if (at[f] && kap[f] != (T)0) { n3[f] = zero; k += kap[f]; }
      bR3 -= k;
      bB3 -= k;
      if (q3 == 0 && kap[4] != (T)0) {
        dn3 = zero;
        if (p3) bB3 -= kap[4]; else bR3 -= kap[4];
      }
      if (q3 == 3 && kap[5] != (T)0) {
        up3 = zero;
        if (p3) bR3 -= kap[5]; else bB3 -= kap[5];
      }
    }
    zR3 = p3 ? up3 : dn3;
    zB3 = p3 ? dn3 : up3;
  };
  T R3 = (T)0, B3 = (T)0, fR3 = (T)0, fB3 = (T)0;
  auto resid8 = [&](T own, T oth, T fs, T b, const T* xo, int zext) __attribute__((always_inline)) {
    return (((xo[n3[0]] + xo[n3[1]]) + (xo[n3[2]] + xo[n3[3]])) + ((oth + xo[zext]) + fs)) - b * own;
  };
  auto sweeps8 = [&](int count, bool zero) __attribute__((always_inline)) {
#pragma unroll 1
    for (int it = 0; it < count; ++it) {
      if (on3) {
        R3 += w6 * (zero && it == 0 ? fR3 : resid8(R3, B3, fR3, bR3, m.x3[1], zR3));
        m.x3[0][t] = R3;
      }
      __syncthreads();
      if (on3) {
        B3 += w6 * resid8(B3, R3, fB3, bB3, m.x3[0], zB3);
        m.x3[1][t] = B3;
      }
      __syncthreads();
    }
  };

  // ---- 4^3 and 2^3: lanes 0..15 of the first wave (the other rows of 16 lanes do the same on the
  // same LDS inputs, which changes nothing)
  const bool lane1 = (t & 5) == 0 && t < 16;   // the 2^3 columns' lanes 0, 2, 8, 10
  int x2, y2, p2, x1, y1, p1;
  T bR2[2], bB2[2], bR1, bB1;
  T cx1, cy1, cz1;             // 2^3: both neighbours are the other cell, or one is a ghost
  bool wx0 = false, wx1 = false, wy0 = false, wy1 = false;
  auto place42 = [&]() __attribute__((always_inline)) {
    int o = t;
    asm volatile("" : "+v"(o));
    x2 = o & 3;
    y2 = (o >> 2) & 3;
    p2 = (x2 + y2) & 1;
    x1 = (o >> 1) & 1;
    y1 = (o >> 3) & 1;
    p1 = (x1 + y1) & 1;
    bR2[0] = bR2[1] = bB2[0] = bB2[1] = bR1 = bB1 = (T)6;
    cx1 = cy1 = cz1 = (T)2;
    if (!WALLS) return;
    const T k2 = (x2 == 0 ? kap[0] : x2 == 3 ? kap[1] : (T)0) + (y2 == 0 ? kap[2] : y2 == 3 ? kap[3] : (T)0);
    const T k1 = (x1 ? kap[1] : kap[0]) + (y1 ? kap[3] : kap[2]);
    bR2[0] -= k2 + (p2 ? (T)0 : kap[4]);
    bB2[0] -= k2 + (p2 ? kap[4] : (T)0);
    bR2[1] -= k2 + (p2 ? kap[5] : (T)0);
    bB2[1] -= k2 + (p2 ? (T)0 : kap[5]);
    bR1 -= k1 + (p1 ? kap[5] : kap[4]);
    bB1 -= k1 + (p1 ? kap[4] : kap[5]);
    cx1 = kap[0] == (T)0 ? (T)2 : (T)1;
    cy1 = kap[2] == (T)0 ? (T)2 : (T)1;
    cz1 = kap[4] == (T)0 ? (T)2 : (T)1;
    wx0 = kap[0] != (T)0 && x2 == 0;
    wx1 = kap[1] != (T)0 && x2 == 3;
    wy0 = kap[2] != (T)0 && y2 == 0;
    wy1 = kap[3] != (T)0 && y2 == 3;
  };
  T R2[2] = {(T)0, (T)0}, B2[2] = {(T)0, (T)0}, fR2[2] = {(T)0, (T)0}, fB2[2] = {(T)0, (T)0};
  T R1 = (T)0, B1 = (T)0, fR1 = (T)0, fB1 = (T)0;
  auto resid4 = [&](const T* own, const T* oth, const T* fs, const T* b, bool s, T* r) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      T l = dpp<kQuadLeft>(oth[q]), h = dpp<kQuadRight>(oth[q]), d = dpp<kUp4>(oth[q]), u = dpp<kDown4>(oth[q]);
      T z = oth[1 - q];   // the z-neighbour outside the slot: of two slots always the other one
      if (WALLS) {
        l = wx0 ? (T)0 : l;
        h = wx1 ? (T)0 : h;
        d = wy0 ? (T)0 : d;
        u = wy1 ? (T)0 : u;
        if (q == 0) z = kap[4] != (T)0 && !s ? (T)0 : z;
        else z = kap[5] != (T)0 && s ? (T)0 : z;
      }
      r[q] = (((l + h) + (d + u)) + ((oth[q] + z) + fs[q])) - b[q] * own[q];
    }
  };
  auto sweeps4 = [&](int count) __attribute__((always_inline)) {
#pragma unroll 1
    for (int it = 0; it < count; ++it) {
      T r[2];
      resid4(R2, B2, fR2, bR2, p2 != 0, r);
      R2[0] += w6 * r[0];
      R2[1] += w6 * r[1];
      resid4(B2, R2, fB2, bB2, p2 == 0, r);
      B2[0] += w6 * r[0];
      B2[1] += w6 * r[1];
    }
  };
  auto resid2 = [&](T own, T oth, T fs, T b) __attribute__((always_inline)) {
    return ((cx1 * dpp<kFlip2>(oth) + cy1 * dpp<kFlip8>(oth)) + (cz1 * oth + fs)) - b * own;
  };
  auto sweeps2 = [&](int count) __attribute__((always_inline)) {
#pragma unroll 1
    for (int it = 0; it < count; ++it) {
      R1 += w6 * resid2(R1, B1, fR1, bR1);
      B1 += w6 * resid2(B1, R1, fB1, bB1);
    }
  };
  // trilinear taps of one axis: the parent cell (3/4) and its neighbour on the child's side
  // (1/4), wrapped, or beyond a wall the parent itself with the ghost's factor
  auto far_tap = [&](int c, int nc, T klo, T khi, int& far, T& wf) __attribute__((always_inline)) {
    far = (c >> 1) + ((c & 1) ? 1 : -1);
    wf = (T)0.25;
    if (WALLS) {
      if (far < 0 && klo != (T)0) { far = 0; wf *= klo; }
      if (far >= nc && khi != (T)0) { far = nc - 1; wf *= khi; }
    }
    far &= nc - 1;
  };
  // lateral interpolation on plane Z (wrapped, or the boundary plane with the ghost's factor) of a
  // level of nc cells per side in LDS, for a fine column at (cx, cy)
  auto lateral_taps = [&](const T* c, int lc, int cx, int cy, int Z) __attribute__((always_inline)) {
    const int nc = 1 << lc;
    int fx, fy;
    T ax, ay, s = (T)1;
    far_tap(cx, nc, kap[0], kap[1], fx, ax);
    far_tap(cy, nc, kap[2], kap[3], fy, ay);
    if (WALLS) {
      if (Z < 0 && kap[4] != (T)0) { Z = 0; s = kap[4]; }
      if (Z >= nc && kap[5] != (T)0) { Z = nc - 1; s = kap[5]; }
    }
    const T* e = c + ((Z & (nc - 1)) << (2 * lc));
    const int X = cx >> 1, y0 = (cy >> 1) << lc, y1 = fy << lc;
    return s * ((T)0.75 * ((T)0.75 * e[y0 + X] + ax * e[y0 + fx]) + ay * ((T)0.75 * e[y1 + X] + ax * e[y1 + fx]));
  };

  // Levels 2 and below from level l2 (2 or 1), by the first wave: one V-cycle.  zero: u of l2 is
  // zero, else taken from us; the result goes to us.
  auto vcycle_wave = [&](int l2, bool zero) __attribute__((always_inline)) {
    place42();
    if (l2 == 2) {
      const int c = kOff2 + (t & 15);
      T f[4], u[4] = {(T)0, (T)0, (T)0, (T)0};
#pragma unroll
      for (int z = 0; z < 4; ++z) {
        f[z] = m.fs[c + 16 * z];
        if (!zero) u[z] = m.us[c + 16 * z];
      }
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        fR2[q] = p2 ? f[2 * q + 1] : f[2 * q];
        fB2[q] = p2 ? f[2 * q] : f[2 * q + 1];
        R2[q] = p2 ? u[2 * q + 1] : u[2 * q];
        B2[q] = p2 ? u[2 * q] : u[2 * q + 1];
      }
      sweeps4(npre);
      T r[2], g[2];
      resid4(R2, B2, fR2, bR2, p2 != 0, r);
      resid4(B2, R2, fB2, bB2, p2 == 0, g);
      T v[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        v[q] = r[q] + g[q];
        v[q] += dpp<kFlip1>(v[q]);
        v[q] = (T)0.5 * (v[q] + dpp<kDown4>(v[q]));   // right in the lanes of the 2^3 columns
      }
      fR1 = p1 ? v[1] : v[0];
      fB1 = p1 ? v[0] : v[1];
      R1 = B1 = (T)0;
    } else {
      const int c = kOff1 + x1 + 2 * y1;
      fR1 = m.fs[c + 4 * p1];
      fB1 = m.fs[c + 4 * (1 - p1)];
      R1 = zero ? (T)0 : m.us[c + 4 * p1];
      B1 = zero ? (T)0 : m.us[c + 4 * (1 - p1)];
    }
    sweeps2(npre);
    T v = resid2(R1, B1, fR1, bR1) + resid2(B1, R1, fB1, bB1);
    v += dpp<kFlip2>(v);
    v = (T)0.5 * (v + dpp<kFlip8>(v));
    const T u0 = b0 == (T)0 ? (T)0 : v / b0;
    // 1^3 to 2^3: per axis 3/4 of the cell and 1/4 of itself (wrapped) or of its ghost
    T e = u0, lo = u0, hi = u0;
    if (WALLS) {
      const T kx = kap[0] == (T)0 ? (T)1 : (x1 ? kap[1] : kap[0]), ky = kap[2] == (T)0 ? (T)1 : (y1 ? kap[3] : kap[2]);
      e *= ((T)0.75 + (T)0.25 * kx) * ((T)0.75 + (T)0.25 * ky);
      lo = e * ((T)0.75 + (T)0.25 * (kap[4] == (T)0 ? (T)1 : kap[4]));
      hi = e * ((T)0.75 + (T)0.25 * (kap[4] == (T)0 ? (T)1 : kap[5]));
    }
    R1 += p1 ? hi : lo;
    B1 += p1 ? lo : hi;
    sweeps2(npost);
    if (l2 == 2) {
      // 2^3 to 4^3: x within the quad, y between its rows (the even rows hold the coarse ones)
      T e2[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const T c = (q == 0) == (p1 == 0) ? R1 : B1;   // the coarse cell at z = q
        const T near = dpp<kEven>(c), farx = dpp<kOther>(c);
        const T row = (T)0.75 * near + (T)0.25 * (wx0 ? kap[0] * near : wx1 ? kap[1] * near : farx);
        const T above = dpp<kUp4>(row), below = dpp<kDown4>(row), two = dpp<kFlip8>(row);
        const T ny = (y2 & 1) ? above : row, fy = (y2 & 1) ? below : two;
        e2[q] = (T)0.75 * ny + (T)0.25 * (wy0 ? kap[2] * ny : wy1 ? kap[3] * ny : fy);
      }
      const T under = WALLS && kap[4] != (T)0 ? kap[4] * e2[0] : e2[1];
      const T over = WALLS && kap[5] != (T)0 ? kap[5] * e2[1] : e2[0];
      const T z0 = (T)0.75 * e2[0] + (T)0.25 * under, z1 = (T)0.75 * e2[0] + (T)0.25 * e2[1];
      const T z2 = (T)0.75 * e2[1] + (T)0.25 * e2[0], z3 = (T)0.75 * e2[1] + (T)0.25 * over;
      R2[0] += p2 ? z1 : z0;
      B2[0] += p2 ? z0 : z1;
      R2[1] += p2 ? z3 : z2;
      B2[1] += p2 ? z2 : z3;
      sweeps4(npost);
      if (t < 16) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          m.us[kOff2 + t + 16 * (2 * q)] = p2 ? B2[q] : R2[q];
          m.us[kOff2 + t + 16 * (2 * q + 1)] = p2 ? R2[q] : B2[q];
        }
      }
    } else if (lane1) {
      const int c = kOff1 + x1 + 2 * y1;
      m.us[c + 4 * p1] = R1;
      m.us[c + 4 * (1 - p1)] = B1;
    }
  };

  // One V-cycle (Alg. 1) from level topl.  Level 4 works on the registers R, B; a lower top level
  // on us (zero: starting from zero).
  auto vcycle = [&](int topl, bool zero) __attribute__((always_inline)) {
    if (topl == 4) {
      sweeps16(npre, zero);
      T r[2], q[2];
      resid16(R, B, fR, bR, m.x[1], zR, p != 0, r);
      resid16(B, R, fB, bB, m.x[0], zB, p == 0, q);
      restrict16(r[0] + q[0], r[1] + q[1]);
      __syncthreads();
      zero = true;
    }
    if (topl >= 3) {
      place8();
      if (on3) {
        const int c = kOff3 + (t & 63) + 128 * q3;
        fR3 = m.fs[c + 64 * p3];
        fB3 = m.fs[c + 64 * (1 - p3)];
        R3 = zero ? (T)0 : m.us[c + 64 * p3];
        B3 = zero ? (T)0 : m.us[c + 64 * (1 - p3)];
        m.x3[0][t] = R3;
        m.x3[1][t] = B3;
      }
      __syncthreads();
      sweeps8(npre, zero);
      if (on3) {
        T v = resid8(R3, B3, fR3, bR3, m.x3[1], zR3) + resid8(B3, R3, fB3, bB3, m.x3[0], zB3);
        v += dpp<kFlip1>(v);
        v += dpp<kFlip8>(v);
        if (((x3 | y3) & 1) == 0) m.fs[kOff2 + (x3 >> 1) + ((y3 >> 1) << 2) + (q3 << 4)] = (T)0.5 * v;
      }
      __syncthreads();
      zero = true;
    }
    if (wave == 0) vcycle_wave(topl < 2 ? 1 : 2, zero);
    __syncthreads();
    if (topl >= 3) {
      if (on3) {
        const T* c = m.us + kOff2;
        const T e0 = lateral_taps(c, 2, x3, y3, q3 - 1), e1 = lateral_taps(c, 2, x3, y3, q3),
                e2 = lateral_taps(c, 2, x3, y3, q3 + 1);
        const T lo = (T)0.75 * e1 + (T)0.25 * e0, hi = (T)0.75 * e1 + (T)0.25 * e2;
        R3 += p3 ? hi : lo;
        B3 += p3 ? lo : hi;
        m.x3[0][t] = R3;
        m.x3[1][t] = B3;
      }
      __syncthreads();
      sweeps8(npost, false);
      if (on3) {
        const int c = kOff3 + (t & 63) + 128 * q3;
        m.us[c + 64 * p3] = R3;
        m.us[c + 64 * (1 - p3)] = B3;
      }
      __syncthreads();
    }
    if (topl == 4) {
      T e[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) e[k] = lateral_taps(m.us + kOff3, 3, x, y, 2 * zq - 1 + k);
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const T lo = (T)0.75 * e[q + 1] + (T)0.25 * e[q], hi = (T)0.75 * e[q + 1] + (T)0.25 * e[q + 2];
        R[q] += p ? hi : lo;
        B[q] += p ? lo : hi;
      }
      m.x[0][t] = v2{R[0], R[1]};
      m.x[1][t] = v2{B[0], B[1]};
      __syncthreads();
      sweeps16(npost, false);
    }
  };

  // the cell of thread t on a level of up to 8^3
  int ci = 0, cj = 0, ck = 0;
  auto cell_of = [&](int l) __attribute__((always_inline)) {
    const int n1 = (1 << l) - 1;
    ci = t & n1;
    cj = (t >> l) & n1;
    ck = t >> (2 * l);
  };

  // ---- load the top level (and, FMG, restrict its source to every level below)
  const T* fg = reinterpret_cast<const T*>(a.f);
  T* ug = reinterpret_cast<T*>(a.ug);
  const T mh2 = (T)(-a.h * a.h);
  const bool load_u = !FMG && (a.mode & TAIL_LOAD_U) != 0;
  if (t == 0) {
    m.x[0][kThreads] = v2{(T)0, (T)0};
    m.x[1][kThreads] = v2{(T)0, (T)0};
    m.x3[0][256] = m.x3[1][256] = (T)0;
  }
  if (top == 4) {
    const int g = (t & 255) + (zq << 10);
    T f[4], u[4] = {(T)0, (T)0, (T)0, (T)0};
#pragma unroll
    for (int q = 0; q < 4; ++q) f[q] = mh2 * fg[g + 256 * q];
    if (load_u)
#pragma unroll
      for (int q = 0; q < 4; ++q) u[q] = ug[g + 256 * q];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      fR[q] = p ? f[2 * q + 1] : f[2 * q];
      fB[q] = p ? f[2 * q] : f[2 * q + 1];
      R[q] = p ? u[2 * q + 1] : u[2 * q];
      B[q] = p ? u[2 * q] : u[2 * q + 1];
    }
    m.x[0][t] = v2{R[0], R[1]};
    m.x[1][t] = v2{B[0], B[1]};
    if constexpr (FMG) restrict16(fR[0] + fB[0], fR[1] + fB[1]);
  } else if (t < (1 << (3 * top))) {
    m.fs[level_offset(top) + t] = mh2 * fg[t];
    m.us[level_offset(top) + t] = load_u ? ug[t] : (T)0;
  }
  if constexpr (FMG) {
    for (int l = top < 4 ? top : 3; l >= 1; --l) {
      __syncthreads();
      if (t < (1 << (3 * (l - 1)))) {
        const int lc = l - 1, nc1 = (1 << lc) - 1, sy = 1 << l, sz = 1 << (2 * l);
        const T* c = m.fs + level_offset(l) + (2 * (t & nc1) + ((2 * ((t >> lc) & nc1)) << l) + ((2 * (t >> (2 * lc))) << (2 * l)));
        m.fs[level_offset(lc) + t] = (T)0.5 * (((c[0] + c[1]) + (c[sy] + c[sy + 1])) +
                                               ((c[sz] + c[sz + 1]) + (c[sz + sy] + c[sz + sy + 1])));
      }
    }
  }
  if (WALLS) {
    __syncthreads();
    // face values enter the sources of the cells they touch (FMG: of every level's own)
#pragma unroll 1
    for (int l = FMG ? 0 : top; l <= (top < 3 ? top : 3); ++l) {
      cell_of(l);
      const LevelBC bc = FMG ? a.phys[l] : a.bc_top;
      if (t < (1 << (3 * l))) m.fs[level_offset(l) + t] += (T)face_terms(bc, 1 << l, ci, cj, ck);
    }
    if (top == 4) {
      const LevelBC bc = FMG ? a.phys[4] : a.bc_top;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        fR[q] += (T)face_terms(bc, 16, x, y, 4 * zq + 2 * q + p);
        fB[q] += (T)face_terms(bc, 16, x, y, 4 * zq + 2 * q + 1 - p);
      }
    }
  }
  __syncthreads();

  // ---- FMG (Alg. 2): on each level 1..top the tricubic prolongation and one V-cycle (which
  // overwrites the sources below, no longer needed); otherwise the one V-cycle
  if constexpr (FMG) {
    if (t == 0) m.us[0] = b0 == (T)0 ? (T)0 : m.fs[0] / b0;
    __syncthreads();
  }
#pragma unroll 1
  for (int l = FMG ? 1 : top; l <= top; ++l) {
    if constexpr (FMG) {
      // the level below with its ghosts (faces, edges and corners)
      const int lc = l - 1, nc = 1 << lc, np = nc + 2;
      if (t < np * np * np) {
        const int i = t % np - 1, j = (t / np) % np - 1, k = t / (np * np) - 1;
        const T* c = m.us + level_offset(lc);
        if (WALLS) {
          const LevelBC bc = a.phys[lc];
          m.pad[t] = ghost_any<T>(c, nc, lc, i, j, k, bc);
        } else {
          m.pad[t] = c[(i & (nc - 1)) | ((j & (nc - 1)) << lc) | ((k & (nc - 1)) << (2 * lc))];
        }
      }
      __syncthreads();
      if (l == 4) {
        T wx[3], wy[3], e[4];
        cub_w<T>(x & 1, wx);
        cub_w<T>(y & 1, wy);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          e[k] = (T)0;
#pragma unroll
          for (int b = 0; b < 3; ++b) {
            const T* c = m.pad + ((2 * zq + k) * 10 + (y >> 1) + b) * 10 + (x >> 1);
            e[k] += wy[b] * ((wx[0] * c[0] + wx[1] * c[1]) + wx[2] * c[2]);
          }
        }
        const T wn = (T)(5.0 / 32.0), wc = (T)(30.0 / 32.0), wp = (T)(-3.0 / 32.0);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const T lo = (wn * e[q] + wc * e[q + 1]) + wp * e[q + 2], hi = (wp * e[q] + wc * e[q + 1]) + wn * e[q + 2];
          R[q] = p ? hi : lo;
          B[q] = p ? lo : hi;
        }
        m.x[0][t] = v2{R[0], R[1]};
        m.x[1][t] = v2{B[0], B[1]};
      } else if (t < (1 << (3 * l))) {
        cell_of(l);
        T wx[3], wy[3], wz[3], s = (T)0;
        cub_w<T>(ci & 1, wx);
        cub_w<T>(cj & 1, wy);
        cub_w<T>(ck & 1, wz);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          T e = (T)0;
#pragma unroll
          for (int b = 0; b < 3; ++b) {
            const T* c = m.pad + (((ck >> 1) + k) * np + (cj >> 1) + b) * np + (ci >> 1);
            e += wy[b] * ((wx[0] * c[0] + wx[1] * c[1]) + wx[2] * c[2]);
          }
          s += wz[k] * e;
        }
        m.us[level_offset(l) + t] = s;
      }
      __syncthreads();
    }
    vcycle(l, !FMG && !load_u);
  }

  // ---- the result (and, when asked, the sum of squared defects of it)
  double acc = 0.0;
  if (top == 4) {
    const int g = (t & 255) + (zq << 10);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      ug[g + 256 * (2 * q)] = p ? B[q] : R[q];
      ug[g + 256 * (2 * q + 1)] = p ? R[q] : B[q];
    }
    if (a.sink.out) {
      T r[2], q[2];
      resid16(R, B, fR, bR, m.x[1], zR, p != 0, r);
      resid16(B, R, fB, bB, m.x[0], zB, p == 0, q);
      acc = ((double)r[0] * (double)r[0] + (double)r[1] * (double)r[1]) + ((double)q[0] * (double)q[0] + (double)q[1] * (double)q[1]);
    }
  } else {
    if (t < (1 << (3 * top))) ug[t] = m.us[level_offset(top) + t];
    if (a.sink.out) {
      T r = (T)0, g = (T)0, r2[2] = {(T)0, (T)0}, g2[2] = {(T)0, (T)0};
      if (top == 3 && on3) {
        r = resid8(R3, B3, fR3, bR3, m.x3[1], zR3);
        g = resid8(B3, R3, fB3, bB3, m.x3[0], zB3);
      } else if (top == 2 && wave == 0) {
        resid4(R2, B2, fR2, bR2, p2 != 0, r2);
        resid4(B2, R2, fB2, bB2, p2 == 0, g2);
      } else if (top == 1 && wave == 0) {
        r = resid2(R1, B1, fR1, bR1);
        g = resid2(B1, R1, fB1, bB1);
      }
      const bool mine = top == 3 ? on3 : top == 2 ? t < 16 : lane1;
      if (mine)
        acc = ((double)r * (double)r + (double)g * (double)g) + ((double)r2[0] * (double)r2[0] + (double)g2[0] * (double)g2[0]) +
              ((double)r2[1] * (double)r2[1] + (double)g2[1] * (double)g2[1]);
    }
  }
  if (a.sink.out) {
    acc = wave_sum(acc);
    if ((t & 63) == 0) m.red[wave] = acc;
    __syncthreads();
    double s = 0.0;
    if (t == 0)
      for (int q = 0; q < kThreads / 64; ++q) s += m.red[q];
    const double ih2 = 1.0 / (a.h * a.h);
    finish_sum<kThreads>(a.sink, s * (ih2 * ih2), m.red);
  }
}

}  // namespace

// Four images: with and without wall code, the V-cycle and the FMG start (whose code would cost the
// V-cycle registers).  Measured per launch in FP64, V(2,2) from 16^3, and with operands gathered from
// LDS on every level and a barrier in every phase: V-cycle 11 and 31 us periodic, 15 and 42 us with
// walls; FMG 21 us periodic, 45 and 325 us with walls and face values (200 bytes of scratch there).
template <typename T>
void launch_tail(const TailArgs& a, hipStream_t s) {
  bool walls = false;
  for (int f = 0; f < 6; ++f) walls = walls || a.hom.kind[f] != BC_PERIODIC;
  auto launch = [&](auto k) { hipLaunchKernelGGL(k, dim3(1), dim3(kThreads), 0, s, a); };
  if ((a.mode & TAIL_FMG) != 0) {
    if (walls) launch(k_tail<T, true, true>);
    else launch(k_tail<T, false, true>);
  } else {
    if (walls) launch(k_tail<T, true, false>);
    else launch(k_tail<T, false, false>);
  }
}

template void launch_tail<double>(const TailArgs&, hipStream_t);
template void launch_tail<float>(const TailArgs&, hipStream_t);

}  // namespace mg
