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
//   8^3   one cell per thread over 8 waves, the six neighbours' LDS slots found once per leg.
//   4^3 .. 1^3  as 8^3, in the first wave alone: its LDS accesses are in order, so its phases
//         need no workgroup barrier.
// Scaled unknowns: fs = -h^2 f (+ 2b at a face with value b), so that the smoother is
// u += (omega/6) r with r = (neighbours + fs) - (6 - kappa) u, -h^2 times the defect, kappa the
// sum over the cell's walls of the ghost's factor on its own value (a wall neighbour reads a
// zero slot).  The restricted defect in the coarse level's scaling is half the sum of the
// eight r, with no h anywhere below the top.
// FMG (Alg. 2) builds the lower sources itself and takes the tricubic prolongation from a
// ghost-filled copy of the level below in LDS.  Measured per launch, FP64 (before: gathered LDS
// operands on every level, a barrier in every phase): see launch_tail.
#include <algorithm>
#include <cstring>

#include "mg_common.h"
#include "mg_launch.h"

namespace mg {

namespace {

constexpr int kThreads = 1024;
constexpr int kSmallCells = 585;   // levels 0..3 back to back
constexpr int kZeroSlot = kSmallCells;
constexpr int kPadCells = 10 * 10 * 10;

// start of level l <= 3 in the back-to-back arrays: (8^l - 1) / 7
__device__ __forceinline__ int level_offset(int l) { return ((1 << (3 * l)) - 1) / 7; }

template <typename T>
struct TailMem {
  typedef T v2 __attribute__((ext_vector_type(2)));
  v2 x[2][kThreads + 1];   // 16^3: per colour, the two slots of every thread; the last is zero
  T us[kSmallCells + 1];   // levels 0..3; the last is zero
  T fs[kSmallCells];
  T r[512];                // scaled residuals of one small level
  T pad[kPadCells];        // FMG: the coarse level with its ghosts
  double red[kThreads / 64];
};

// value of the lane one to the left (D = 1) or right (D = 15) in a row of 16, cyclic
template <int D>
__device__ __forceinline__ float row_ror(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x120 | D, 0xf, 0xf, false));
}
template <int D>
__device__ __forceinline__ double row_ror(double v) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, 0x120 | D, 0xf, 0xf, false);
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), 0x120 | D, 0xf, 0xf, false);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// all = true: a workgroup barrier.  Otherwise the first wave alone is running: LDS accesses of
// one wave are performed in order, so only the compiler has to keep it.
__device__ __forceinline__ void phase_end(bool all) {
  if (all) {
    __syncthreads();
  } else {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

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
template <typename T, bool WALLS>
__global__ void __launch_bounds__(kThreads) k_tail(TailArgs a) {
  using v2 = typename TailMem<T>::v2;
  __shared__ TailMem<T> m;
  const int t = threadIdx.x, wave = t >> 6;
  const int top = a.top, npre = a.npre, npost = a.npost;
  if (a.clock && t == 0) *a.clock = (unsigned long long)wall_clock64();
  const T w6 = (T)(a.omega / 6.0);
  const bool fmg = (a.mode & TAIL_FMG) != 0;
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
    T l0 = row_ror<1>(oth[0]), l1 = row_ror<1>(oth[1]), h0 = row_ror<15>(oth[0]), h1 = row_ror<15>(oth[1]);
    if (WALLS) {
      l0 = wxl ? (T)0 : l0; l1 = wxl ? (T)0 : l1;
      h0 = wxh ? (T)0 : h0; h1 = wxh ? (T)0 : h1;
    }
    r[0] = ((((l0 + h0) + (a0.x + a1.x)) + (oth[0] + z0)) + fs[0]) - b[0] * own[0];
    r[1] = ((((l1 + h1) + (a0.y + a1.y)) + (oth[1] + z1)) + fs[1]) - b[1] * own[1];
  };
  auto sweeps16 = [&](int count) __attribute__((always_inline)) {
#pragma unroll 1
    for (int it = 0; it < count; ++it) {
      T r[2];
      resid16(R, B, fR, bR, m.x[1], zR, p != 0, r);
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
    v0 += __shfl_xor(v0, 1, 64);
    v1 += __shfl_xor(v1, 1, 64);
    v0 += __shfl_xor(v0, 16, 64);
    v1 += __shfl_xor(v1, 16, 64);
    if (((x | y) & 1) == 0) {
      const int C = level_offset(3) + (x >> 1) + ((y >> 1) << 3) + (zq << 7);
      m.fs[C] = (T)0.5 * v0;
      m.fs[C + 64] = (T)0.5 * v1;
      m.us[C] = (T)0;
      m.us[C + 64] = (T)0;
    }
  };

  // ---- levels 1..3: one cell per thread (thread c of the first 8^l)
  int nbr[6];
  int ci = 0, cj = 0, ck = 0;
  T bs = (T)6;
  auto cell_of = [&](int l) __attribute__((always_inline)) {
    const int n1 = (1 << l) - 1;
    ci = t & n1;
    cj = (t >> l) & n1;
    ck = t >> (2 * l);
  };
  auto place = [&](int l) __attribute__((always_inline)) {
    const int n1 = (1 << l) - 1, off = level_offset(l);
    cell_of(l);
    nbr[0] = off + ((t & ~n1) | ((ci - 1) & n1));
    nbr[1] = off + ((t & ~n1) | ((ci + 1) & n1));
    nbr[2] = off + ((t & ~(n1 << l)) | (((cj - 1) & n1) << l));
    nbr[3] = off + ((t & ~(n1 << l)) | (((cj + 1) & n1) << l));
    nbr[4] = off + ((t & ~(n1 << (2 * l))) | (((ck - 1) & n1) << (2 * l)));
    nbr[5] = off + ((t & ~(n1 << (2 * l))) | (((ck + 1) & n1) << (2 * l)));
    bs = (T)6;
    if (WALLS) {
      const int c[3] = {ci, cj, ck};
#pragma unroll
      for (int f = 0; f < 6; ++f)
        if (c[f >> 1] == ((f & 1) ? n1 : 0) && kap[f] != (T)0) {
          nbr[f] = kZeroSlot;
          bs -= kap[f];
        }
    }
  };
  auto resid_small = [&](T u, T f) __attribute__((always_inline)) {
    const T s = ((m.us[nbr[0]] + m.us[nbr[1]]) + (m.us[nbr[2]] + m.us[nbr[3]])) + (m.us[nbr[4]] + m.us[nbr[5]]);
    return (s + f) - bs * u;
  };
  auto sweeps_small = [&](int l, int count, bool on, T& u, T f) __attribute__((always_inline)) {
    const bool all = l == 3;
    const int mine = (ci + cj + ck) & 1;
#pragma unroll 1
    for (int h = 0; h < 2 * count; ++h) {
      if (on && mine == (h & 1)) {
        u += w6 * resid_small(u, f);
        m.us[level_offset(l) + t] = u;
      }
      phase_end(all);
    }
  };
  auto down_small = [&](int l) __attribute__((always_inline)) {
    const bool on = t < (1 << (3 * l)), all = l == 3;
    place(l);
    T u = (T)0, f = (T)0;
    if (on) { u = m.us[level_offset(l) + t]; f = m.fs[level_offset(l) + t]; }
    sweeps_small(l, npre, on, u, f);
    if (on) m.r[t] = resid_small(u, f);
    phase_end(all);
    if (t < (1 << (3 * (l - 1)))) {
      const int lc = l - 1, nc1 = (1 << lc) - 1;
      const T* c = m.r + (2 * (t & nc1) + ((2 * ((t >> lc) & nc1)) << l) + ((2 * (t >> (2 * lc))) << (2 * l)));
      const int sy = 1 << l, sz = 1 << (2 * l);
      m.fs[level_offset(lc) + t] = (T)0.5 * (((c[0] + c[1]) + (c[sy] + c[sy + 1])) +
                                             ((c[sz] + c[sz + 1]) + (c[sz + sy] + c[sz + sy + 1])));
      m.us[level_offset(lc) + t] = (T)0;
    }
    phase_end(false);
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
  auto up_small = [&](int l) __attribute__((always_inline)) {
    const bool on = t < (1 << (3 * l));
    place(l);
    T u = (T)0, f = (T)0;
    if (on) {
      const int lc = l - 1, nc = 1 << lc;
      int fx, fy, fz;
      T wx, wy, wz;
      far_tap(ci, nc, kap[0], kap[1], fx, wx);
      far_tap(cj, nc, kap[2], kap[3], fy, wy);
      far_tap(ck, nc, kap[4], kap[5], fz, wz);
      const T* c = m.us + level_offset(lc);
      const int X = ci >> 1, y0 = (cj >> 1) << lc, y1 = fy << lc, z0 = (ck >> 1) << (2 * lc), z1 = fz << (2 * lc);
      const T q = (T)0.75;
      const T e00 = q * c[z0 + y0 + X] + wx * c[z0 + y0 + fx], e01 = q * c[z0 + y1 + X] + wx * c[z0 + y1 + fx];
      const T e10 = q * c[z1 + y0 + X] + wx * c[z1 + y0 + fx], e11 = q * c[z1 + y1 + X] + wx * c[z1 + y1 + fx];
      u = m.us[level_offset(l) + t] + (q * (q * e00 + wy * e01) + wz * (q * e10 + wy * e11));
      f = m.fs[level_offset(l) + t];
      m.us[level_offset(l) + t] = u;
    }
    phase_end(l == 3);
    sweeps_small(l, npost, on, u, f);
  };

  // One V-cycle (Alg. 1) from level topl.
  auto vcycle = [&](int topl) __attribute__((always_inline)) {
    if (topl == 4) {
      sweeps16(npre);
      T r[2], q[2];
      resid16(R, B, fR, bR, m.x[1], zR, p != 0, r);
      resid16(B, R, fB, bB, m.x[0], zB, p == 0, q);
      restrict16(r[0] + q[0], r[1] + q[1]);
      __syncthreads();
    }
    const int l3 = topl < 3 ? topl : 3;
    // levels 2 and below in the first wave; the others wait at the barrier before level 3
#pragma unroll 1
    for (int l = l3; l >= 1 && !(l <= 2 && wave > 0); --l) down_small(l);
    if (t == 0) {
      m.us[0] = b0 == (T)0 ? (T)0 : m.fs[0] / b0;
    }
    if (wave == 0) phase_end(false);
#pragma unroll 1
    for (int l = 1; l <= l3; ++l) {
      if (l <= 2 && wave > 0) continue;
      if (l == 3) __syncthreads();
      up_small(l);
    }
    if (l3 <= 2) __syncthreads();
    if (topl == 4) {
      const T* c = m.us + level_offset(3);
      int fx, fy;
      T wx, wy;
      far_tap(x, 8, kap[0], kap[1], fx, wx);
      far_tap(y, 8, kap[2], kap[3], fy, wy);
      const int X = x >> 1, y0 = (y >> 1) << 3, y1 = fy << 3;
      T e[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        int Z = 2 * zq - 1 + k;
        T s = (T)1;
        if (WALLS) {
          if (Z < 0 && kap[4] != (T)0) { Z = 0; s = kap[4]; }
          if (Z > 7 && kap[5] != (T)0) { Z = 7; s = kap[5]; }
        }
        const T* cz = c + ((Z & 7) << 6);
        e[k] = s * ((T)0.75 * ((T)0.75 * cz[y0 + X] + wx * cz[y0 + fx]) + wy * ((T)0.75 * cz[y1 + X] + wx * cz[y1 + fx]));
      }
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const T lo = (T)0.75 * e[q + 1] + (T)0.25 * e[q], hi = (T)0.75 * e[q + 1] + (T)0.25 * e[q + 2];
        R[q] += p ? hi : lo;
        B[q] += p ? lo : hi;
      }
      m.x[0][t] = v2{R[0], R[1]};
      m.x[1][t] = v2{B[0], B[1]};
      __syncthreads();
      sweeps16(npost);
    }
  };

  // ---- load the top level (and, FMG, restrict its source to every level below)
  const T* fg = reinterpret_cast<const T*>(a.f);
  T* ug = reinterpret_cast<T*>(a.ug);
  const T mh2 = (T)(-a.h * a.h);
  const bool load_u = (a.mode & TAIL_LOAD_U) != 0;
  if (t == 0) {
    m.x[0][kThreads] = v2{(T)0, (T)0};
    m.x[1][kThreads] = v2{(T)0, (T)0};
    m.us[kZeroSlot] = (T)0;
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
    if (fmg) restrict16(fR[0] + fB[0], fR[1] + fB[1]);
  } else if (t < (1 << (3 * top))) {
    m.fs[level_offset(top) + t] = mh2 * fg[t];
    m.us[level_offset(top) + t] = load_u ? ug[t] : (T)0;
  }
  if (fmg) {
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
    for (int l = fmg ? 0 : top; l <= (top < 3 ? top : 3); ++l) {
      cell_of(l);
      const LevelBC bc = fmg ? a.phys[l] : a.bc_top;
      if (t < (1 << (3 * l))) m.fs[level_offset(l) + t] += (T)face_terms(bc, 1 << l, ci, cj, ck);
    }
    if (top == 4) {
      const LevelBC bc = fmg ? a.phys[4] : a.bc_top;
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
  if (fmg) {
    if (t == 0) m.us[0] = b0 == (T)0 ? (T)0 : m.fs[0] / b0;
    __syncthreads();
  }
#pragma unroll 1
  for (int l = fmg ? 1 : top; l <= top; ++l) {
    if (fmg) {
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
    vcycle(l);
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
  } else if (t < (1 << (3 * top))) {
    const T u = m.us[level_offset(top) + t];
    ug[t] = u;
    if (a.sink.out) {
      place(top);
      const T r = resid_small(u, m.fs[level_offset(top) + t]);
      acc = (double)r * (double)r;
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

template <typename T>
void launch_tail(const TailArgs& a, hipStream_t s) {
  bool walls = false;
  for (int f = 0; f < 6; ++f) walls = walls || a.hom.kind[f] != BC_PERIODIC;
  if (walls) hipLaunchKernelGGL((k_tail<T, true>), dim3(1), dim3(kThreads), 0, s, a);
  else hipLaunchKernelGGL((k_tail<T, false>), dim3(1), dim3(kThreads), 0, s, a);
}

template void launch_tail<double>(const TailArgs&, hipStream_t);
template void launch_tail<float>(const TailArgs&, hipStream_t);

}  // namespace mg
