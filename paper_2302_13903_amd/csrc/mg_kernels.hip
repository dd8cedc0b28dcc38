// mg_kernels.hip -- per-operator HIP kernels (gfx950) of the multigrid solver, in FP64 and FP32.
//
// These are the plain one-operator-per-launch kernels used on every level below the fused
// large-level kernels, by the operator entry points, and as the building blocks of the
// FP32 inner cycle of the mixed-precision path.  Each kernel is a streaming loop with
// 64-bit indices and on-the-fly boundary ghosts (see mg_common.h).
#include <algorithm>

#include "mg_common.h"
#include "mg_launch.h"

namespace mg {

LaunchTiming& launch_timing() {
  static thread_local LaunchTiming t;
  return t;
}

constexpr int kBlock = 256;

static inline unsigned grid_for(size_t work, int per_thread = 1) {
  size_t threads = (work + per_thread - 1) / per_thread;
  size_t g = (threads + kBlock - 1) / kBlock;
  return (unsigned)(g == 0 ? 1 : g);
}

// ------------------------------------------------------------------ smoothing (eqs. rbsor1-2)

// One colour of the over-relaxed red-black Gauss-Seidel update.  Work item t covers the
// x-pair (2p, 2p+1) of row (j, k); exactly one of the two has the requested colour.
template <typename T>
__global__ void __launch_bounds__(kBlock) k_half_sweep(T* __restrict__ u, const T* __restrict__ f, int n,
                                                        int L, T h2, T omega, int colour, LevelBC bc) {
  const size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x;
  const size_t pairs = (size_t)1 << (3 * L - 1);
  if (t >= pairs) return;
  const int p = (int)(t & (size_t)((n >> 1) - 1));
  const int j = (int)((t >> (L - 1)) & (size_t)(n - 1));
  const int k = (int)(t >> (2 * L - 1));
  const int i = 2 * p + ((j + k + colour) & 1);
  const size_t c = cidx(L, i, j, k);
  const T uc = u[c];
  const T nb = neighbour_sum(u, n, L, i, j, k, c, uc, bc);
  u[c] = uc + omega * ((nb - h2 * f[c]) * (T)(1.0 / 6.0) - uc);
}

template <typename T>
void launch_half_sweep(T* u, const T* f, int n, double h, double omega, int colour, const LevelBC& bc,
                       hipStream_t s) {
  const int L = ilog2(n);
  const size_t pairs = (size_t)1 << (3 * L - 1);
  hipLaunchKernelGGL(k_half_sweep<T>, dim3(grid_for(pairs)), dim3(kBlock), 0, s, u, f, n, L, (T)(h * h),
                     (T)omega, colour, bc);
}

// ------------------------------------------------------------------ defect (eq. defect)

template <typename T>
__global__ void __launch_bounds__(kBlock) k_defect(const T* __restrict__ u, const T* __restrict__ f,
                                                    T* __restrict__ d, int n, int L, T ih2, LevelBC bc) {
  const size_t c = (size_t)blockIdx.x * kBlock + threadIdx.x;
  if (c >= ((size_t)1 << (3 * L))) return;
  const int i = (int)(c & (size_t)(n - 1));
  const int j = (int)((c >> L) & (size_t)(n - 1));
  const int k = (int)(c >> (2 * L));
  const T uc = u[c];
  const T nb = neighbour_sum(u, n, L, i, j, k, c, uc, bc);
  d[c] = f[c] - (nb - (T)6 * uc) * ih2;
}

template <typename T>
void launch_defect(const T* u, const T* f, T* d, int n, double h, const LevelBC& bc, hipStream_t s) {
  const int L = ilog2(n);
  hipLaunchKernelGGL(k_defect<T>, dim3(grid_for((size_t)1 << (3 * L))), dim3(kBlock), 0, s, u, f, d, n, L,
                     (T)(1.0 / (h * h)), bc);
}

// Defect on the fine level restricted straight to the coarse level (Alg. 1 steps 2-3): one
// work item per coarse cell computes its 8 children's defects and their mean; it also clears
// the coarse correction (the recursion starts from zero, Alg. 1 step 4).
template <typename T>
__global__ void __launch_bounds__(kBlock) k_defect_restrict(const T* __restrict__ u, const T* __restrict__ f,
                                                             T* __restrict__ fc, T* __restrict__ uc0, int n,
                                                             int L, T ih2, LevelBC bc) {
  const int nc = n >> 1, Lc = L - 1;
  const size_t C = (size_t)blockIdx.x * kBlock + threadIdx.x;
  if (C >= ((size_t)1 << (3 * Lc))) return;
  const int I = (int)(C & (size_t)(nc - 1));
  const int J = (int)((C >> Lc) & (size_t)(nc - 1));
  const int K = (int)(C >> (2 * Lc));
  T s = (T)0;
#pragma unroll
  for (int c3 = 0; c3 < 2; ++c3)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        const int i = 2 * I + a, j = 2 * J + b, k = 2 * K + c3;
        const size_t c = cidx(L, i, j, k);
        const T ucv = u[c];
        const T nb = neighbour_sum(u, n, L, i, j, k, c, ucv, bc);
        s += f[c] - (nb - (T)6 * ucv) * ih2;
      }
  fc[C] = s * (T)0.125;
  if (uc0) uc0[C] = (T)0;
}

template <typename T>
void launch_defect_restrict(const T* u, const T* f, T* fc, T* uc0, int n, double h, const LevelBC& bc,
                            hipStream_t s) {
  const int L = ilog2(n);
  hipLaunchKernelGGL(k_defect_restrict<T>, dim3(grid_for((size_t)1 << (3 * (L - 1)))), dim3(kBlock), 0, s, u,
                     f, fc, uc0, n, L, (T)(1.0 / (h * h)), bc);
}

// ------------------------------------------------------------------ FAS transfers (Alg. 3)

// Alg. 3 steps 2-4 and the coarse initial guess of step 6: per coarse cell the restricted
// defect of its 8 children (into fc), the restricted potential phibar (into pbar) and the
// coarse iterate set to phibar (into uc).
__global__ void __launch_bounds__(kBlock) k_fas_restrict(const double* __restrict__ u, const double* __restrict__ f,
                                                          double* __restrict__ fc, double* __restrict__ pbar,
                                                          double* __restrict__ uc, int n, int L, double ih2,
                                                          LevelBC bc) {
  const int nc = n >> 1, Lc = L - 1;
  const size_t C = (size_t)blockIdx.x * kBlock + threadIdx.x;
  if (C >= ((size_t)1 << (3 * Lc))) return;
  const int I = (int)(C & (size_t)(nc - 1));
  const int J = (int)((C >> Lc) & (size_t)(nc - 1));
  const int K = (int)(C >> (2 * Lc));
  double sd = 0.0, su = 0.0;
#pragma unroll
  for (int c3 = 0; c3 < 2; ++c3)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        const int i = 2 * I + a, j = 2 * J + b, k = 2 * K + c3;
        const size_t c = cidx(L, i, j, k);
        const double ucv = u[c];
        const double nb = neighbour_sum(u, n, L, i, j, k, c, ucv, bc);
        sd += f[c] - (nb - 6.0 * ucv) * ih2;
        su += ucv;
      }
  fc[C] = sd * 0.125;
  const double pb = su * 0.125;
  pbar[C] = pb;
  uc[C] = pb;
}

void launch_fas_restrict(const double* u, const double* f, double* fc, double* pbar, double* uc, int n, double h,
                         const LevelBC& bc, hipStream_t s) {
  const int L = ilog2(n);
  hipLaunchKernelGGL(k_fas_restrict, dim3(grid_for((size_t)1 << (3 * (L - 1)))), dim3(kBlock), 0, s, u, f, fc, pbar,
                     uc, n, L, 1.0 / (h * h), bc);
}

// Alg. 3 step 5 on the coarse level: f += L phibar, with phibar's ghosts from the level's
// physical description.
__global__ void __launch_bounds__(kBlock) k_fas_source(const double* __restrict__ pbar, double* __restrict__ f, int n,
                                                        int L, double ih2, LevelBC bc) {
  const size_t c = (size_t)blockIdx.x * kBlock + threadIdx.x;
  if (c >= ((size_t)1 << (3 * L))) return;
  const int i = (int)(c & (size_t)(n - 1));
  const int j = (int)((c >> L) & (size_t)(n - 1));
  const int k = (int)(c >> (2 * L));
  const double pc = pbar[c];
  const double nb = neighbour_sum(pbar, n, L, i, j, k, c, pc, bc);
  f[c] = f[c] + (nb - 6.0 * pc) * ih2;
}

void launch_fas_source(const double* pbar, double* f, int n, double h, const LevelBC& bc, hipStream_t s) {
  const int L = ilog2(n);
  hipLaunchKernelGGL(k_fas_source, dim3(grid_for((size_t)1 << (3 * L))), dim3(kBlock), 0, s, pbar, f, n, L,
                     1.0 / (h * h), bc);
}

// Alg. 3 step 7: the coarse-grid correction psi - phibar, in place of psi.
__global__ void __launch_bounds__(kBlock) k_fas_correction(double* __restrict__ u, const double* __restrict__ pbar,
                                                            size_t n3) {
  const size_t c = (size_t)blockIdx.x * kBlock + threadIdx.x;
  if (c < n3) u[c] = u[c] - pbar[c];
}

void launch_fas_correction(double* u, const double* pbar, size_t n3, hipStream_t s) {
  hipLaunchKernelGGL(k_fas_correction, dim3(grid_for(n3)), dim3(kBlock), 0, s, u, pbar, n3);
}

// ------------------------------------------------------------------ restriction (eq. restriction)

template <typename Tin, typename Tout>
__global__ void __launch_bounds__(kBlock) k_restrict(const Tin* __restrict__ uf, Tout* __restrict__ uc, int Lc) {
  const int nc = 1 << Lc, L = Lc + 1;
  const size_t C = (size_t)blockIdx.x * kBlock + threadIdx.x;
  if (C >= ((size_t)1 << (3 * Lc))) return;
  const int I = (int)(C & (size_t)(nc - 1));
  const int J = (int)((C >> Lc) & (size_t)(nc - 1));
  const int K = (int)(C >> (2 * Lc));
  Tin s = (Tin)0;
#pragma unroll
  for (int c3 = 0; c3 < 2; ++c3)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int a = 0; a < 2; ++a) s += uf[cidx(L, 2 * I + a, 2 * J + b, 2 * K + c3)];
  uc[C] = (Tout)(s * (Tin)0.125);
}

template <typename Tin, typename Tout>
void launch_restrict(const Tin* uf, Tout* uc, int nc, hipStream_t s) {
  const int Lc = ilog2(nc);
  hipLaunchKernelGGL((k_restrict<Tin, Tout>), dim3(grid_for((size_t)1 << (3 * Lc))), dim3(kBlock), 0, s, uf,
                     uc, Lc);
}

// ------------------------------------------------------------------ prolongation (Sec. 2.3.1)

// cubic = 0: uf += trilinear(uc) (eq. trilinear, Alg. 1 steps 5-6);
// cubic = 1: uf  = tricubic(uc)  (FMG prolongation, Alg. 2 step 3).
// One work item per coarse cell: it gathers the 3x3x3 coarse neighbourhood once (through the
// ghost rules only in the first and last rows and planes) and writes its 8 children as four
// 2-cell row segments.
// One-dimensional prolongation of the coarse values a, b, c at offsets -1, 0, +1 to the lower
// (upper = 0) or upper child, with the weights of lin_w / cub_w (zero weights left out).
template <typename T, int CUBIC>
__device__ __forceinline__ T interp3(int upper, T a, T b, T c) {
  if (CUBIC) {
    return upper ? ((T)(-3.0 / 32.0) * a + (T)(30.0 / 32.0) * b) + (T)(5.0 / 32.0) * c
                 : ((T)(5.0 / 32.0) * a + (T)(30.0 / 32.0) * b) + (T)(-3.0 / 32.0) * c;
  }
  return upper ? (T)0.75 * b + (T)0.25 * c : (T)0.25 * a + (T)0.75 * b;
}

template <typename T, int CUBIC>
__global__ void __launch_bounds__(kBlock) k_prolong(const T* __restrict__ uc, T* __restrict__ uf, int Lc,
                                                     LevelBC bcc) {
  const int nc = 1 << Lc, L = Lc + 1;
  const size_t C = (size_t)blockIdx.x * kBlock + threadIdx.x;
  if (C >= ((size_t)1 << (3 * Lc))) return;
  const int I = (int)(C & (size_t)(nc - 1));
  const int J = (int)((C >> Lc) & (size_t)(nc - 1));
  const int K = (int)(C >> (2 * Lc));
  // res[zc][yc][xc]: child (2I + xc, 2J + yc, 2K + zc), each the sum over the taps (cz, by, ax)
  // in that order of (wx * wy * wz) * tap (the same terms in the same order in both branches)
  T res[2][2][2];
  if (J > 0 && J < nc - 1 && K > 0 && K < nc - 1) {
    // rows inside in y and z (every row of the grid has its two x-boundary cells, so these
    // must not leave the fast path): the 27 taps read directly, the x-neighbour beyond an x
    // face given by that face's rule -- the wrapped cell, the cell itself (zero gradient) or
    // 2b - u (a value b on the face) -- as the ghost rules give it; every weight a constant
    const int Im = I > 0 ? I - 1 : nc - 1, Ip = I < nc - 1 ? I + 1 : 0;
    const bool wlo = I == 0 && bcc.kind[0] != BC_PERIODIC, whi = I == nc - 1 && bcc.kind[1] != BC_PERIODIC;
    T v[3][3][3];
#pragma unroll
    for (int cz = 0; cz < 3; ++cz)
#pragma unroll
      for (int by = 0; by < 3; ++by) {
        const int Jr = J + by - 1, Kr = K + cz - 1;
        const size_t row = cidx(Lc, 0, Jr, Kr);
        const T u0 = uc[row + (size_t)I];
        T um = uc[row + (size_t)Im], up = uc[row + (size_t)Ip];
        if (wlo) um = bcc.kind[0] == BC_ZERO_GRADIENT ? u0 : (T)(2.0 * face_b(bcc, 0, nc, Jr, Kr)) - u0;
        if (whi) up = bcc.kind[1] == BC_ZERO_GRADIENT ? u0 : (T)(2.0 * face_b(bcc, 1, nc, Jr, Kr)) - u0;
        v[cz][by][0] = um;
        v[cz][by][1] = u0;
        v[cz][by][2] = up;
      }
    // the weights are a product of one-dimensional ones: interpolate in x (nine rows), then in
    // y (three planes), then in z -- 114 multiply-adds for the eight children instead of 216
    T ex[3][3][2], ey[3][2][2];
#pragma unroll
    for (int cz = 0; cz < 3; ++cz)
#pragma unroll
      for (int by = 0; by < 3; ++by)
#pragma unroll
        for (int xc = 0; xc < 2; ++xc) ex[cz][by][xc] = interp3<T, CUBIC>(xc, v[cz][by][0], v[cz][by][1], v[cz][by][2]);
#pragma unroll
    for (int cz = 0; cz < 3; ++cz)
#pragma unroll
      for (int yc = 0; yc < 2; ++yc)
#pragma unroll
        for (int xc = 0; xc < 2; ++xc) ey[cz][yc][xc] = interp3<T, CUBIC>(yc, ex[cz][0][xc], ex[cz][1][xc], ex[cz][2][xc]);
#pragma unroll
    for (int zc = 0; zc < 2; ++zc)
#pragma unroll
      for (int yc = 0; yc < 2; ++yc)
#pragma unroll
        for (int xc = 0; xc < 2; ++xc) res[zc][yc][xc] = interp3<T, CUBIC>(zc, ey[0][yc][xc], ey[1][yc][xc], ey[2][yc][xc]);
  } else {
    // the first and last rows and planes: one tap at a time through the ghost rules (a loop,
    // so the ghost code is in the kernel once), added to all eight children
#pragma unroll
    for (int zc = 0; zc < 2; ++zc)
#pragma unroll
      for (int yc = 0; yc < 2; ++yc)
#pragma unroll
        for (int xc = 0; xc < 2; ++xc) res[zc][yc][xc] = (T)0;
#pragma unroll 1
    for (int t = 0; t < 27; ++t) {
      const int ax = t % 3, by = (t / 3) % 3, cz = t / 9;
      const T val = ghost_any(uc, nc, Lc, I + ax - 1, J + by - 1, K + cz - 1, bcc);
#pragma unroll
      for (int zc = 0; zc < 2; ++zc)
#pragma unroll
        for (int yc = 0; yc < 2; ++yc)
#pragma unroll
          for (int xc = 0; xc < 2; ++xc) {
            T wx[3], wy[3], wz[3];
            if (CUBIC) { cub_w<T>(xc, wx); cub_w<T>(yc, wy); cub_w<T>(zc, wz); }
            else { lin_w<T>(xc, wx); lin_w<T>(yc, wy); lin_w<T>(zc, wz); }
            // the weights of this tap (selects: no runtime-indexed arrays)
            const T a = ax == 0 ? wx[0] : (ax == 1 ? wx[1] : wx[2]);
            const T b = by == 0 ? wy[0] : (by == 1 ? wy[1] : wy[2]);
            const T c = cz == 0 ? wz[0] : (cz == 1 ? wz[1] : wz[2]);
            if (!CUBIC && (a == (T)0 || b == (T)0 || c == (T)0)) continue;
            res[zc][yc][xc] += (a * b * c) * val;
          }
    }
  }
  // the two x-children are adjacent (even index first): one vector access per child row; the
  // FMG result (of coarse levels below 16^3 here) is written past the caches, as k_prolong_tile's
  typedef T tv2 __attribute__((ext_vector_type(2)));
#pragma unroll
  for (int zc = 0; zc < 2; ++zc)
#pragma unroll
    for (int yc = 0; yc < 2; ++yc) {
      tv2* fp = reinterpret_cast<tv2*>(uf + cidx(L, 2 * I, 2 * J + yc, 2 * K + zc));
      if (CUBIC) {
        __builtin_nontemporal_store(tv2{res[zc][yc][0], res[zc][yc][1]}, fp);
      } else {
        const tv2 o = *fp;
        *fp = tv2{o.x + res[zc][yc][0], o.y + res[zc][yc][1]};
      }
    }
}

// The FMG prolongation of the levels from 16^3: a workgroup stages its 256 coarse cells and their
// neighbours, ghosts included, in LDS (one cell or two per thread, the ghost rules evaluated side
// by side), then each thread interpolates separably in x, y, z and writes the 8 children of one
// cell.  Bound by the writes; small levels by one global and one LDS latency, where 27 taps through
// the ghost rules one after another took 17-22 us a level.  Lmc, Lmf: MeshBlock layout of the
// coarse and the fine level (0: dense).
constexpr int kProlongMinNc = 16;
template <typename T, int TX>
__global__ void __launch_bounds__(kBlock) k_prolong_tile(const T* __restrict__ uc, T* __restrict__ uf, int Lc, int Lmc,
                                                          int Lmf, LevelBC bcc) {
  constexpr int TY = 4, TZ = kBlock / (TX * TY), SX = TX + 2, SY = TY + 2, SZ = TZ + 2;
  __shared__ T v[SZ * SY * SX];
  const int nc = 1 << Lc, tx = nc / TX, ty = nc / TY;
  const int I0 = (int)(blockIdx.x % tx) * TX, J0 = (int)((blockIdx.x / tx) % ty) * TY, K0 = (int)(blockIdx.x / (tx * ty)) * TZ;
  for (int q = threadIdx.x; q < SZ * SY * SX; q += kBlock) {
    const int i = I0 + q % SX - 1, j = J0 + (q / SX) % SY - 1, k = K0 + q / (SX * SY) - 1;
    const bool inside = i >= 0 && i < nc && j >= 0 && j < nc && k >= 0 && k < nc;
    v[q] = inside ? uc[lidx(Lc, Lmc, i, j, k)] : ghost_any(uc, nc, Lc, i, j, k, bcc, Lmc);
  }
  __syncthreads();
  const int a = threadIdx.x % TX, b = (threadIdx.x / TX) % TY, c = threadIdx.x / (TX * TY);
  const T* p = v + (c * SY + b) * SX + a;
  T ey[3][2][2];   // [plane][y child][x child]
#pragma unroll
  for (int z = 0; z < 3; ++z) {
    T ex[3][2];
#pragma unroll
    for (int y = 0; y < 3; ++y) {
      const T* r = p + (z * SY + y) * SX;
      ex[y][0] = interp3<T, 1>(0, r[0], r[1], r[2]);
      ex[y][1] = interp3<T, 1>(1, r[0], r[1], r[2]);
    }
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      ey[z][0][x] = interp3<T, 1>(0, ex[0][x], ex[1][x], ex[2][x]);
      ey[z][1][x] = interp3<T, 1>(1, ex[0][x], ex[1][x], ex[2][x]);
    }
  }
  // the two x-children are adjacent (even index first); written past the caches, which leaves them
  // to the coarse rows that neighbouring workgroups read
  typedef T tv2 __attribute__((ext_vector_type(2)));
  const int L = Lc + 1, I = I0 + a, J = J0 + b, K = K0 + c;
#pragma unroll
  for (int z = 0; z < 2; ++z)
#pragma unroll
    for (int y = 0; y < 2; ++y) {
      const T lo = interp3<T, 1>(z, ey[0][y][0], ey[1][y][0], ey[2][y][0]);
      const T hi = interp3<T, 1>(z, ey[0][y][1], ey[1][y][1], ey[2][y][1]);
      __builtin_nontemporal_store(tv2{lo, hi}, reinterpret_cast<tv2*>(uf + lidx(L, Lmf, 2 * I, 2 * J + y, 2 * K + z)));
    }
}

template <typename T>
void launch_prolong_fmg(const T* uc, T* uf, int nc, int Lmc, int Lmf, const LevelBC& bcc, hipStream_t s) {
  const int Lc = ilog2(nc);
  const dim3 g((unsigned)(((size_t)1 << (3 * Lc)) / kBlock));
  if (nc >= 32) hipLaunchKernelGGL((k_prolong_tile<T, 32>), g, dim3(kBlock), 0, s, uc, uf, Lc, Lmc, Lmf, bcc);
  else hipLaunchKernelGGL((k_prolong_tile<T, 16>), g, dim3(kBlock), 0, s, uc, uf, Lc, Lmc, Lmf, bcc);
}

template <typename T>
void launch_prolong(const T* uc, T* uf, int nc, const LevelBC& bcc, int cubic, hipStream_t s) {
  if (cubic && nc >= kProlongMinNc) return launch_prolong_fmg<T>(uc, uf, nc, 0, 0, bcc, s);
  const int Lc = ilog2(nc);
  const dim3 g(grid_for((size_t)1 << (3 * Lc)));
  if (cubic) hipLaunchKernelGGL((k_prolong<T, 1>), g, dim3(kBlock), 0, s, uc, uf, Lc, bcc);
  else hipLaunchKernelGGL((k_prolong<T, 0>), g, dim3(kBlock), 0, s, uc, uf, Lc, bcc);
}

// ------------------------------------------------------------------ coarsest (Sec. 2.3.2)

// Single-cell solve: every ghost is alpha*u + beta (periodic / zero-gradient: alpha = 1,
// fixed: alpha = -1, beta = 2b), so u = (sum beta - h^2 f) / (6 - sum alpha); 0 if sum alpha = 6.
template <typename T>
__device__ __forceinline__ T coarsest_value(T f, T h2, const LevelBC& bc) {
  T sa = (T)0, sb = (T)0;
#pragma unroll
  for (int face = 0; face < 6; ++face) {
    if (bc_has_value(bc.kind[face])) { sa -= (T)1; sb += (T)(2.0 * face_b(bc, face, 1, 0, 0)); }
    else sa += (T)1;
  }
  return sa == (T)6 ? (T)0 : (sb - h2 * f) / ((T)6 - sa);
}

template <typename T>
__global__ void k_coarsest(T* u, const T* f, T h2, LevelBC bc) {
  if (threadIdx.x == 0 && blockIdx.x == 0) u[0] = coarsest_value(f[0], h2, bc);
}

template <typename T>
void launch_coarsest(T* u, const T* f, double h, const LevelBC& bc, hipStream_t s) {
  hipLaunchKernelGGL(k_coarsest<T>, dim3(1), dim3(64), 0, s, u, f, (T)(h * h), bc);
}

// ------------------------------------------------------------------ elementwise / set-up

// u += shift (gauge fix, Sec. 2.3.6)
__global__ void __launch_bounds__(kBlock) k_shift(double* __restrict__ u, size_t n3, const double* __restrict__ sum,
                                                   double scale) {
  const size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x;
  if (t >= n3) return;
  u[t] -= sum[0] * scale;
}

void launch_sub_mean(double* u, size_t n3, const double* sum_dev, hipStream_t s) {
  hipLaunchKernelGGL(k_shift, dim3(grid_for(n3)), dim3(kBlock), 0, s, u, n3, sum_dev, 1.0 / (double)n3);
}

template <typename Ta, typename Tb>
__global__ void __launch_bounds__(kBlock) k_copy_convert(const Ta* __restrict__ a, Tb* __restrict__ b, size_t n3) {
  const size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x;
  if (t < n3) b[t] = (Tb)a[t];
}

void launch_f32_to_f64(const float* a, double* b, size_t n3, hipStream_t s) {
  hipLaunchKernelGGL((k_copy_convert<float, double>), dim3(grid_for(n3)), dim3(kBlock), 0, s, a, b, n3);
}

// phi64 += e32 (mixed precision correction, defect equation eq. defecteq)
__global__ void __launch_bounds__(kBlock) k_add_f32(double* __restrict__ phi, const float* __restrict__ e, size_t n3) {
  const size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x;
  if (t < n3) phi[t] += (double)e[t];
}

void launch_add_f32(double* phi, const float* e, size_t n3, hipStream_t s) {
  hipLaunchKernelGGL(k_add_f32, dim3(grid_for(n3)), dim3(kBlock), 0, s, phi, e, n3);
}

// ------------------------------------------------------------------ reductions

// Deterministic sums: one partial per block (grid-stride loop, fixed grid, fixed tree), added in
// index order by the block that arrives last (finish_sum).  The blocks are large and at most
// kSumBlocks: each arrival is an atomic on one counter, 11 ns apart (2048 blocks of 256 threads
// took 23 us longer than the reading at 256^3).
constexpr int kSumBlock = 1024, kSumBlocks = 512;

template <int THREADS>
__device__ __forceinline__ double block_sum(double v, double* red) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) red[w] = v;
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x == 0) {
    for (int q = 0; q < THREADS / 64; ++q) r += red[q];
  }
  __syncthreads();
  return r;
}

// blocks of kSumBlock threads for `items` grid-strided work items
static int sum_blocks(size_t items) {
  const size_t b = (items + kSumBlock - 1) / kSumBlock;
  return (int)std::min<size_t>(std::max<size_t>(b, 1), kSumBlocks);
}

__global__ void __launch_bounds__(kSumBlock) k_sum(const double* __restrict__ x, size_t n3, SumSink sink) {
  typedef double dv2 __attribute__((ext_vector_type(2)));
  __shared__ double red[kSumBlock / 64];
  double acc = 0.0, acc2 = 0.0;
  if (((size_t)x & 15) == 0 && (n3 & 1) == 0) {
    const dv2* p = reinterpret_cast<const dv2*>(x);
#pragma unroll 4
    for (size_t t = (size_t)blockIdx.x * kSumBlock + threadIdx.x; t < n3 / 2; t += (size_t)gridDim.x * kSumBlock) {
      const dv2 v = p[t];
      acc += v.x;
      acc2 += v.y;
    }
  } else {
    for (size_t t = (size_t)blockIdx.x * kSumBlock + threadIdx.x; t < n3; t += (size_t)gridDim.x * kSumBlock) acc += x[t];
  }
  finish_sum<kSumBlock>(sink, block_sum<kSumBlock>(acc + acc2, red), red);
}

__global__ void __launch_bounds__(kBlock) k_sum_final(const double* __restrict__ part, int np, SumSink sink) {
  // the sum of part[b], b < np, in index order
  __shared__ double red[kBlock / 64];
  double acc = 0.0;
  for (int b = threadIdx.x; b < np; b += kBlock) acc += part[b];
  finish_sum<kBlock>(sink, block_sum<kBlock>(acc, red), red);
}

int reduce_blocks(size_t n3) {
  size_t b = (n3 + (size_t)kBlock * 8 - 1) / ((size_t)kBlock * 8);
  if (b > (size_t)kMaxPartials) b = kMaxPartials;
  return (int)(b < 1 ? 1 : b);
}

// The device scalars cleared at the start of a solve, the device clock in scal[at].
__global__ void k_begin(double* scal, int count, int at) {
  const int t = threadIdx.x;
  if (t < count) scal[t] = t == at ? __builtin_bit_cast(double, (unsigned long long)wall_clock64()) : 0.0;
}

void launch_begin(double* scal, int count, int at, hipStream_t s) {
  hipLaunchKernelGGL(k_begin, dim3(1), dim3(64), 0, s, scal, count, at);
}

__global__ void k_clock(unsigned long long* at) {
  if (threadIdx.x == 0) *at = (unsigned long long)wall_clock64();
}

void launch_clock(unsigned long long* at, hipStream_t s) { hipLaunchKernelGGL(k_clock, dim3(1), dim3(64), 0, s, at); }

// Publication of a sum that a launch without a sink left in device memory.
__global__ void k_publish(const double* __restrict__ src, SumSink sink) {
  publish_scalars(sink.pub, sink.seq, src[0], sink.copy);
}

void launch_publish(const double* src, const SumSink& sink, hipStream_t s) {
  hipLaunchKernelGGL(k_publish, dim3(1), dim3(64), 0, s, src, sink);
}

void launch_sum_partials(int np, SumSink sink, hipStream_t s) {
  sink.total = 1;
  hipLaunchKernelGGL(k_sum_final, dim3(1), dim3(kBlock), 0, s, sink.part, np, sink);
}

void launch_sum(const double* x, size_t n3, SumSink sink, hipStream_t s) {
  sink.total = sum_blocks((n3 + 7) / 8);
  hipLaunchKernelGGL(k_sum, dim3(sink.total), dim3(kSumBlock), 0, s, x, n3, sink);
}

// Defect of the finest level and its sum of squares (Sec. 2.3.7, eq. threshold); optionally
// the defect itself in FP32 (mixed precision: right-hand side of the inner correction cycle).
__global__ void __launch_bounds__(kSumBlock) k_defect_norm(const double* __restrict__ u, const double* __restrict__ f,
                                                         float* __restrict__ r32, int n, int L, double ih2, LevelBC bc,
                                                         SumSink sink) {
  __shared__ double red[kSumBlock / 64];
  const size_t n3 = (size_t)1 << (3 * L);
  double acc = 0.0;
  for (size_t c = (size_t)blockIdx.x * kSumBlock + threadIdx.x; c < n3; c += (size_t)gridDim.x * kSumBlock) {
    const int i = (int)(c & (size_t)(n - 1));
    const int j = (int)((c >> L) & (size_t)(n - 1));
    const int k = (int)(c >> (2 * L));
    const double uc = u[c];
    const double nb = neighbour_sum(u, n, L, i, j, k, c, uc, bc);
    const double d = f[c] - (nb - 6.0 * uc) * ih2;
    acc += d * d;
    if (r32) r32[c] = (float)d;
  }
  finish_sum<kSumBlock>(sink, block_sum<kSumBlock>(acc, red), red);
}

void launch_defect_norm(const double* u, const double* f, float* r32, int n, double h, const LevelBC& bc,
                        SumSink sink, hipStream_t s) {
  const int L = ilog2(n);
  sink.total = sum_blocks((size_t)1 << (3 * L));
  hipLaunchKernelGGL(k_defect_norm, dim3(sink.total), dim3(kSumBlock), 0, s, u, f, r32, n, L, 1.0 / (h * h), bc, sink);
}

// f = a * rho + c (the source 4 pi G rho, mean-shifted when gauge-free: c = -a * mean(rho),
// read from the device so that the host need not wait for the sum), in FP64, plus the
// FP32 copy when f32 != nullptr, and the sum of f^2 (fixed grid and tree, so reproducible); with
// fc also its restriction to the level below (Alg. 2 step 1), while the eight children are in
// registers (at 512^3 a pass of its own over f took 238 us).  Without the sum of rho the block
// sums of rho are taken here for their finiteness alone: one that is not finite makes the sum of
// f^2 not finite either.  One work item per coarse cell, in the coarse level's storage order:
// four row pairs of 16 bytes.  Lm: MeshBlock layout with 2^Lm-cell blocks (0: dense).
template <typename T>
__global__ void __launch_bounds__(kSumBlock) k_source(const double* __restrict__ rho, double* __restrict__ f,
                                                       float* __restrict__ f32, T* __restrict__ fc, int L, int Lm,
                                                       double a, const double* __restrict__ rho_sum, SumSink sink) {
  typedef double dv2 __attribute__((ext_vector_type(2), aligned(8)));   // rho is the caller's: 8-byte aligned
  typedef float fv2 __attribute__((ext_vector_type(2)));
  __shared__ double red[kSumBlock / 64];
  const size_t n3 = (size_t)1 << (3 * L), items = n3 >> 3;
  // gauge-free: c = -a * mean(rho), from the sum the previous launch left in device memory
  const double c = rho_sum ? -a * (rho_sum[0] / (double)n3) : 0.0;
  const int Lf = Lm > 0 ? Lm : L, Lc = Lf - 1;   // the cube of 2^Lf cells that is stored x fastest
  double acc = 0.0, total = 0.0;
  for (size_t C = (size_t)blockIdx.x * kSumBlock + threadIdx.x; C < items; C += (size_t)gridDim.x * kSumBlock) {
    const size_t r = C & (((size_t)1 << (3 * Lc)) - 1);
    size_t cube = C >> (3 * Lc);
    if (Lm == 1) {   // blocks of one coarse cell each: the level below is the dense root grid
      const int m = (1 << (L - 1)) - 1;
      cube = morton3((int)C & m, (int)(C >> (L - 1)) & m, (int)(C >> (2 * L - 2)));
    }
    const size_t i = r & (((size_t)1 << Lc) - 1), j = (r >> Lc) & (((size_t)1 << Lc) - 1), k = r >> (2 * Lc);
    const size_t o = (cube << (3 * Lf)) | (k << (2 * Lf + 1)) | (j << (Lf + 1)) | (i << 1);
    double sum = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const size_t at = o + ((q & 1) ? (size_t)1 << Lf : 0) + ((q & 2) ? (size_t)1 << (2 * Lf) : 0);
      const dv2 x = *reinterpret_cast<const dv2*>(rho + at);
      const dv2 v = dv2{a * x.x + c, a * x.y + c};
      *reinterpret_cast<dv2*>(f + at) = v;
      if (f32) *reinterpret_cast<fv2*>(f32 + at) = fv2{(float)v.x, (float)v.y};
      acc += v.x * v.x + v.y * v.y;
      total += x.x + x.y;
      sum += v.x + v.y;
    }
    if (fc) fc[C] = (T)(0.125 * sum);
  }
  double sumsq = block_sum<kSumBlock>(acc, red);
  total = block_sum<kSumBlock>(total, red);
  if (!isfinite(total)) sumsq = __builtin_nan("");
  finish_sum<kSumBlock>(sink, sumsq, red);
}

template <typename T>
void launch_source(const double* rho, double* f, float* f32, T* fc, int L, int Lm, double a, const double* rho_sum,
                   SumSink sink, hipStream_t s) {
  sink.total = sum_blocks((size_t)1 << (3 * L - 3));
  hipLaunchKernelGGL(k_source<T>, dim3(sink.total), dim3(kSumBlock), 0, s, rho, f, f32, fc, L, Lm, a, rho_sum, sink);
}
template void launch_source<double>(const double*, double*, float*, double*, int, int, double, const double*, SumSink,
                                    hipStream_t);
template void launch_source<float>(const double*, double*, float*, float*, int, int, double, const double*, SumSink,
                                   hipStream_t);

// ------------------------------------------------------------------ boundary face arrays

// FIXED faces of every level, from the caller's n^2 face-centre values on the finest one: a
// coarser face takes 2 x 2 area means, and each array is extended to (n+2)^2, the ring taking the
// nearest face value.  One workgroup makes a tile of 32 x 32 finest values and all its coarser
// levels in LDS; a second launch, one workgroup per face, makes the levels above the tiles.  (One
// launch per face and level, and two more per face for the check of its values, took 126 us of a
// 64^3 solve; these two take 6.)
struct FaceArgs {
  const double* src[6];   // null: not a face with values.  First launch: n^2 values
  double* ext[16];        // per level: the six extended arrays one after another
  double* nonfinite;      // per face: the count of non-finite values (first launch), or null
  int top, bottom;        // the levels this launch makes
};
constexpr int kFaceTile = 32, kFaceTop = 64;

template <int M, bool FIRST>
__global__ void __launch_bounds__(kBlock) k_faces(FaceArgs A) {
  __shared__ double v[M * M];
  const int face = blockIdx.z;
  if (!A.src[face]) return;
  const int n = 1 << A.top, m0 = n < M ? n : M;
  const int o1 = blockIdx.x * m0, o2 = blockIdx.y * m0;   // the tile's place on level top
  auto store = [&](int l, int t1, int t2, double x) {
    const int nl = 1 << l, w = nl + 2;
    double* e = A.ext[l] + (size_t)face * w * w;
    // the cell's own entry and the ring entries nearest to it
    for (int b = t2 == 0 ? -1 : t2; b <= (t2 == nl - 1 ? nl : t2); ++b)
      for (int a = t1 == 0 ? -1 : t1; a <= (t1 == nl - 1 ? nl : t1); ++a) e[(size_t)(b + 1) * w + a + 1] = x;
  };
  int bad = 0;
  for (int q = threadIdx.x; q < m0 * m0; q += kBlock) {
    const int t1 = o1 + q % m0, t2 = o2 + q / m0;
    double x;
    if (FIRST) {
      x = A.src[face][(size_t)t2 * n + t1];
      bad += isfinite(x) ? 0 : 1;
      store(A.top, t1, t2, x);
    } else {
      x = A.ext[A.top][(size_t)face * (n + 2) * (n + 2) + (size_t)(t2 + 1) * (n + 2) + t1 + 1];
    }
    v[q] = x;
  }
  if (FIRST && bad && A.nonfinite) unsafeAtomicAdd(A.nonfinite + face, (double)bad);   // a whole number: any order
  for (int m = m0 / 2, l = A.top - 1; m >= 1 && l >= A.bottom; m >>= 1, --l) {
    __syncthreads();
    double x[M * M / 4 / kBlock < 1 ? 1 : M * M / 4 / kBlock];
    int c = 0;
#pragma unroll
    for (int s = 0; s < (int)(sizeof(x) / sizeof(double)); ++s) {
      const int q = threadIdx.x + s * kBlock;
      if (q < m * m) {
        const double* r = v + (2 * (q / m)) * (2 * m) + 2 * (q % m);
        x[s] = (r[0] + r[1] + r[2 * m] + r[2 * m + 1]) / 4.0;
        ++c;
      }
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < (int)(sizeof(x) / sizeof(double)); ++s) {
      const int q = threadIdx.x + s * kBlock;
      if (s < c) {
        v[q] = x[s];
        store(l, (o1 * m) / m0 + q % m, (o2 * m) / m0 + q / m, x[s]);
      }
    }
  }
}

void launch_faces(const double* const src[6], double* const* ext, int L, int bottom, double* nonfinite, hipStream_t s) {
  FaceArgs A{};
  for (int f = 0; f < 6; ++f) A.src[f] = src[f];
  for (int l = bottom; l <= L; ++l) A.ext[l] = ext[l];
  A.nonfinite = nonfinite;
  A.top = L;
  A.bottom = bottom;
  const int tiles = std::max(1, (1 << L) / kFaceTile);
  hipLaunchKernelGGL((k_faces<kFaceTile, true>), dim3(tiles, tiles, 6), dim3(kBlock), 0, s, A);
  if (tiles > 1 && bottom < ilog2(tiles)) {
    A.top = ilog2(tiles);
    hipLaunchKernelGGL((k_faces<kFaceTop, false>), dim3(1, 1, 6), dim3(kBlock), 0, s, A);
  }
}

// A ghost beyond a face with value b is 2 b - u: the u part is a factor of the cell's own value,
// the 2 b part a constant of that cell's equation, so it can stand in f once and for all.  Doing
// so here, once per solve, takes the face arrays out of every leg of every cycle: read there,
// they cost the 64^3 legs 6 and 8 us of 16 and 20, the 128^3 legs 35 us a cycle, and the streaming
// passes 2 KiB of LDS and their registers' slack.  Bound by the launch below 128^3 and by
// the strided cells of the x faces above.
struct FoldArgs {
  FoldLevel l[16];
  unsigned first[17];   // the first block of each level
};

template <typename T>
__global__ void __launch_bounds__(kBlock) k_fold_faces(FoldArgs A) {
  int lv = 0;
  while (blockIdx.x >= A.first[lv + 1]) ++lv;
  const FoldLevel& V = A.l[lv];
  const int L = V.L, n = 1 << L;
  const unsigned t = (blockIdx.x - A.first[lv]) * kBlock + threadIdx.x;
  const int face = (int)(t >> (2 * L));
  auto valued = [&](int f) { return bc_has_value(V.bc.kind[f]) && V.bc.b[f]; };
  if (face >= 6 || !valued(face)) return;
  const int t1 = (int)(t & (unsigned)(n - 1)), t2 = (int)((t >> L) & (unsigned)(n - 1)), axis = face >> 1;
  int c[3];
  c[axis] = face & 1 ? n - 1 : 0;
  c[axis == 0 ? 1 : 0] = t1;
  c[axis == 2 ? 1 : 2] = t2;
  // a cell on several faces belongs to the first of them
  double sum = face_b(V.bc, face, n, t1, t2);
  for (int f = 0; f < 6; ++f) {
    const int a = f >> 1;
    if (f == face || !valued(f) || c[a] != (f & 1 ? n - 1 : 0)) continue;
    if (f < face) return;
    sum += face_b(V.bc, f, n, c[a == 0 ? 1 : 0], c[a == 2 ? 1 : 2]);
  }
  T* at = reinterpret_cast<T*>(V.f) + lidx(L, V.Lm, c[0], c[1], c[2]);
  *at = (T)((double)*at - 2.0 * V.ih2 * sum);
}

template <typename T>
void launch_fold_faces(const FoldLevel* levels, int count, hipStream_t s) {
  FoldArgs A{};
  bool any = false;
  for (int q = 0; q < 16; ++q) {
    unsigned blocks = 0;
    if (q < count) {
      A.l[q] = levels[q];
      for (int f = 0; f < 6; ++f) any = any || (bc_has_value(levels[q].bc.kind[f]) && levels[q].bc.b[f]);
      blocks = (unsigned)((((size_t)6 << (2 * levels[q].L)) + kBlock - 1) / kBlock);
    }
    A.first[q + 1] = A.first[q] + blocks;
  }
  if (any) hipLaunchKernelGGL(k_fold_faces<T>, dim3(A.first[count]), dim3(kBlock), 0, s, A);
}
template void launch_fold_faces<double>(const FoldLevel*, int, hipStream_t);
template void launch_fold_faces<float>(const FoldLevel*, int, hipStream_t);

// ------------------------------------------------------------------ clearing device memory

// Zero `words` 8-byte words (a kernel rather than a memset node, so the clear is an ordinary
// kernel wherever the stream's work is recorded).
__global__ void __launch_bounds__(kBlock) k_zero(unsigned long long* __restrict__ p, size_t words) {
  const size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * kBlock;
  for (size_t i = t; i < words; i += stride) p[i] = 0ull;
}
__global__ void k_zero_bytes(unsigned char* __restrict__ p, size_t bytes) {
  const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < bytes) p[t] = 0;
}

void launch_zero(void* p, size_t bytes, hipStream_t s) {
  if (bytes == 0) return;
  const size_t words = bytes / 8, tail = bytes % 8;
  if (words) {
    const size_t g = std::min<size_t>((words + kBlock - 1) / kBlock, 8192);
    hipLaunchKernelGGL(k_zero, dim3((unsigned)g), dim3(kBlock), 0, s, reinterpret_cast<unsigned long long*>(p), words);
  }
  if (tail)
    hipLaunchKernelGGL(k_zero_bytes, dim3(1), dim3(8), 0, s, reinterpret_cast<unsigned char*>(p) + words * 8, tail);
}

// ------------------------------------------------------------------ ghost fill (Sec. 2.3.6)

// The ghost-filled copy of one level: out is (n+2)^3, x fastest, with active cell (i, j, k) at
// ((k+1)(n+2) + j+1)(n+2) + i+1 and every ghost -- faces, edges and corners -- set by the
// axis-ordered rule the prolongations read (x first, then y over the x ghosts, then z over
// both), i.e. the value ghost_any evaluates on the fly.
__global__ void __launch_bounds__(kBlock) k_fill(const double* __restrict__ u, double* __restrict__ out, int n,
                                                  int L, LevelBC bc) {
  const size_t m = (size_t)n + 2;
  const size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x;
  if (t >= m * m * m) return;
  const int i = (int)(t % m) - 1, j = (int)((t / m) % m) - 1, k = (int)(t / (m * m)) - 1;
  const bool inside = i >= 0 && i < n && j >= 0 && j < n && k >= 0 && k < n;
  out[t] = inside ? u[cidx(L, i, j, k)] : ghost_any(u, n, L, i, j, k, bc);
}

void launch_fill(const double* u, double* out, int n, const LevelBC& bc, hipStream_t s) {
  const size_t m = (size_t)n + 2;
  hipLaunchKernelGGL(k_fill, dim3(grid_for(m * m * m)), dim3(kBlock), 0, s, u, out, n, ilog2(n), bc);
}

// ------------------------------------------------------------------ explicit instantiations

#define MG_INST(T)                                                                                   \
  template void launch_half_sweep<T>(T*, const T*, int, double, double, int, const LevelBC&, hipStream_t); \
  template void launch_defect<T>(const T*, const T*, T*, int, double, const LevelBC&, hipStream_t);        \
  template void launch_defect_restrict<T>(const T*, const T*, T*, T*, int, double, const LevelBC&,         \
                                          hipStream_t);                                                    \
  template void launch_prolong<T>(const T*, T*, int, const LevelBC&, int, hipStream_t);                    \
  template void launch_prolong_fmg<T>(const T*, T*, int, int, int, const LevelBC&, hipStream_t);           \
  template void launch_coarsest<T>(T*, const T*, double, const LevelBC&, hipStream_t);

MG_INST(double)
MG_INST(float)
template void launch_restrict<double, double>(const double*, double*, int, hipStream_t);
template void launch_restrict<float, float>(const float*, float*, int, hipStream_t);
template void launch_restrict<double, float>(const double*, float*, int, hipStream_t);

}  // namespace mg
