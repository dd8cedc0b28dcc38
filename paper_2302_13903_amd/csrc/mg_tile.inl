// mg_tile.inl -- V-cycle legs of the small levels (32^3 and 64^3, and 128^3 where the streaming passes
// are off; dense or in the MeshBlock layout) as one launch each.
//
// On these levels a V-cycle leg is a handful of microseconds of work spread over many
// dependent launches (per colour, per operator), so the launch latency dominates.  Here one
// launch does a whole leg:
//   down (Alg. 1 steps 1-3): NS red-black SOR sweeps (eqs. rbsor1-2), the defect of the
//        result (eq. defect) restricted to the coarse level (eq. restriction), the coarse
//        correction cleared;
//   up   (Alg. 1 steps 5-7): u += trilinear prolongation of the coarse correction (eq.
//        trilinear), NS sweeps, optionally the sum of squared defects of the result
//        (Sec. 2.3.7).
// Each workgroup owns a region and works on it with a halo of H = 2 NS + 1 cells (2 NS colour
// passes of radius 1 and the defect): what a pass leaves wrong at the tile's rim moves inwards
// by one cell per pass and stops short of the region, so regions are independent and only the
// region is written back.
//
// One thread holds one z-column of the tile, u and the source in registers, by colour: slot q
// of a colour is the cell z = 2q or 2q + 1 that has it.  Slot q's z-neighbours of the other
// colour are that column's own slots q and q +- 1 (registers), its x and y neighbours slot q of
// the four columns around it, which pass through LDS two slots (16 bytes) per access: 4 reads
// and 1 write per two cell updates.  (Gathering six neighbours, the cell and f per update with
// an x-stride of two takes 8 LDS reads of 8 bytes with two-way bank conflicts and a global read
// of f in every pass; u and f here cross once.)  Levels and times: see launch_leg.
//
// u += (omega/6) r with r = (neighbours - h^2 f) - (6 - kappa) u = -h^2 times the defect, kappa
// the ghosts' factors on the cell's own value (face values b stand in f as f - 2 b / h^2: from the
// start in a solve, launch_fold_faces; put there as f is loaded in the legs of the operator entry
// points, whose f is the caller's); cells outside the domain hold zero and are not updated (weight zero).  The up leg first stages the coarse correction under the tile (homogeneous ghosts: periodic wrap, or the boundary cell
// with the face's sign).  The level may be dense or in the MeshBlock layout (the same code with
// the block-major index, whose x, y and z parts are disjoint bits; the coarse side of the lowest
// block level is the dense root grid).
#include "mg_tile.h"

#include "mg_launch.h"

namespace mg {

namespace {

// Region shapes (cells per workgroup, all even).
struct Shape {
  int dx, dy, dz;
};
constexpr Shape kShapes[2] = {{16, 8, 8}, {8, 4, 4}};
int shape_of(int n) { return n >= 64 ? 0 : 1; }
// workgroup size: one thread per column of the tile, in whole waves
constexpr int tile_threads(int ns, int sh) {
  return ((kShapes[sh].dx + 4 * ns + 2) * (kShapes[sh].dy + 4 * ns + 2) + 63) / 64 * 64;
}

struct TileArgs {
  const void* uin;
  void* uout;
  const void* f;
  const void* ec;    // up: coarse correction
  void* fc;          // down: restricted defect
  void* uc0;         // down: coarse correction to clear, or null (FAS: to start from phibar)
  void* pbar;        // FAS down (Alg. 3 steps 2-4), else null: receives phibar, the mean of the
                     // 8 children of the swept u, from which the coarse level then starts
  SumSink sink;      // up: where the sum of squared defects goes (part null: not wanted)
  LevelBC bc;        // this level
  LevelBC bcc;       // up: coarse level (homogeneous)
  int n, L, Lm, per, nrx, nry;
  double h2, ih2, omega;
};

// Workgroups in contiguous runs per XCD (consecutive workgroups go round the 8 XCDs).
__device__ __forceinline__ unsigned xcd_order(unsigned bid, unsigned nwg) {
  if ((nwg & 7u) != 0) return bid;
  return (bid & 7u) * (nwg >> 3) + (bid >> 3);
}

// Storage index of cell (i, j, k) (in range) of this level (Lm > 0: MeshBlock layout) and of the
// coarse level below; each the sum of its parts (i, 0, 0) + (0, j, 0) + (0, 0, k), so a column
// spreads its x and y bits once and each plane's part is the same for the whole workgroup.
__device__ __forceinline__ unsigned fine_at(const TileArgs& A, int i, int j, int k) {
  return (unsigned)lidx(A.L, A.Lm, i, j, k);
}
__device__ __forceinline__ unsigned coarse_at(const TileArgs& A, int I, int J, int K) {
  return (unsigned)lidx(A.L - 1, A.Lm > 1 ? A.Lm - 1 : 0, I, J, K);
}

// Coarse correction at (I, J, K) under homogeneous conditions: periodic indices wrap; on the
// other axes an index beyond the domain takes the boundary cell with the face's sign (+1 zero
// gradient, -1 zero-fixed), axis by axis (edges and corners: the product of the signs).
template <typename T, bool WALLS>
__device__ __forceinline__ T coarse_hom(const TileArgs& A, const T* __restrict__ ec, int I, int J, int K) {
  const int ncm = (A.n >> 1) - 1;
  if (!WALLS) return ec[coarse_at(A, I & ncm, J & ncm, K & ncm)];
  T s = (T)1;
  auto axis = [&](int v, int pbit, int lo_face) __attribute__((always_inline)) {
    if (A.per & pbit) return v & ncm;
    if (v < 0) {
      if (A.bcc.kind[lo_face] != BC_ZERO_GRADIENT) s = -s;
      return 0;
    }
    if (v > ncm) {
      if (A.bcc.kind[lo_face + 1] != BC_ZERO_GRADIENT) s = -s;
      return ncm;
    }
    return v;
  };
  const int Ic = axis(I, 1, 0), Jc = axis(J, 2, 2), Kc = axis(K, 4, 4);
  return s * ec[coarse_at(A, Ic, Jc, Kc)];
}

template <typename T>
__device__ __forceinline__ T wall_factor(const LevelBC& bc, int face) {
  return bc.kind[face] == BC_ZERO_GRADIENT ? (T)1 : (T)-1;
}

// WALLS: some face of the level is not periodic.  Layout, norm and FAS (a coarse index, a sum or
// two stores at the end of a leg) are the launch's, not the kernel's.  VALUES: the face values are in
// A.bc and not in f (null: none on that face).
template <typename T, int NS, bool UP, bool WALLS, int SH, bool VALUES>
__global__ void __launch_bounds__(tile_threads(NS, SH), SH == 0 ? 4 : 1) k_tile_leg(TileArgs A) {
  typedef T v2 __attribute__((ext_vector_type(2)));
  constexpr int H = 2 * NS + 1;
  constexpr int kThreads = tile_threads(NS, SH);
  constexpr int DX = kShapes[SH].dx, DY = kShapes[SH].dy, DZ = kShapes[SH].dz;
  constexpr int WX = DX + 2 * H, WY = DY + 2 * H, WZ = DZ + 2 * H;   // the tile
  constexpr int NQ = WZ / 2;                                         // slots per colour
  constexpr int QL = (H - 1) / 2, QH = (H + DZ - 1) / 2;             // slots of the region's ends
  constexpr int COLS = WX * WY;
  constexpr int CX = WX / 2 + 1, CY = WY / 2 + 1, CZ = NQ + 1;       // coarse cells under the tile
  constexpr int MZ = DZ / 2;
  // a region shorter than the halo: the halo of the next region but one also reaches a z wall,
  // whose boundary cell is then in the tile's first or last slot
  constexpr bool NARROW = WALLS && DZ < H;
  static_assert(!NARROW || (QL == MZ && QH + MZ == NQ - 1), "z walls in the halo");
  // the exchange: per colour, slots 2m and 2m + 1 of every column side by side, an odd last slot
  // alone.  Before the sweeps the up leg's coarse tile lies here, after them the column sums of
  // the down leg
  __shared__ __align__(16) T ex[2][NQ * COLS];
  __shared__ double red[kThreads / 64];
  static_assert(CX * CY * CZ <= 2 * NQ * COLS && 2 * MZ * COLS <= 2 * NQ * COLS, "shared memory of the tile");
  const int tid = threadIdx.x;
  const int n = A.n, nm = n - 1, per = A.per;
  const char* __restrict__ uin = reinterpret_cast<const char*>(A.uin);
  char* __restrict__ uout = reinterpret_cast<char*>(A.uout);
  const char* __restrict__ fin = reinterpret_cast<const char*>(A.f);
  const int rid = (int)xcd_order(blockIdx.x, gridDim.x);
  const int rx = rid % A.nrx, ry = (rid / A.nrx) % A.nry, rz = rid / (A.nrx * A.nry);
  const int ox = rx * DX, oy = ry * DY, oz = rz * DZ;   // region origin (even)
  // the thread's column; threads past the last column repeat it (same values to the same slots)
  const int col = tid < COLS ? tid : COLS - 1;
  const int tx = col % WX, ty = col / WX;
  const bool p = ((tx + ty) & 1) != 0;   // red cells: z of parity 1 - p within a slot, black: p
  const int i = (ox - H + tx) & nm, j = (oy - H + ty) & nm;
  const bool own_col = tid < COLS && tx >= H && tx < H + DX && ty >= H && ty < H + DY;   // of the region

  const T w6 = (T)(A.omega / 6.0), mh2 = (T)-A.h2;
  // update weight and 6 - kappa; with walls also those of the slots beyond and at the z walls
  T w = w6, b = (T)6;
  T wlo = w6, whi = w6, wloR = w6, wloB = w6, whiR = w6, whiB = w6, bloR = b, bloB = b, bhiR = b, bhiB = b;
  T w0R = w6, w0B = w6, w9R = w6, w9B = w6, b0R = b, b0B = b, b9R = b, b9B = b;   // NARROW: first, last slot
  bool in = true, zlo = false, zhi = false, zlo2 = false, zhi2 = false;
  if (WALLS) {
    const int gi = ox - H + tx, gj = oy - H + ty;
    in = ((per & 1) || (unsigned)gi < (unsigned)n) && ((per & 2) || (unsigned)gj < (unsigned)n);
    zlo = !(per & 4) && oz == 0;
    zhi = !(per & 4) && oz + DZ == n;
    w = in ? w6 : (T)0;
    if (!(per & 1)) {
      if (gi == 0) b -= wall_factor<T>(A.bc, 0);
      if (gi == nm) b -= wall_factor<T>(A.bc, 1);
    }
    if (!(per & 2)) {
      if (gj == 0) b -= wall_factor<T>(A.bc, 2);
      if (gj == nm) b -= wall_factor<T>(A.bc, 3);
    }
    // slot QL holds the cell above a low z wall (parity 1) and one beyond it (parity 0), slot QH
    // the cell below a high one (parity 0) and one beyond
    const T klo = zlo ? wall_factor<T>(A.bc, 4) : (T)0, khi = zhi ? wall_factor<T>(A.bc, 5) : (T)0;
    wlo = zlo ? (T)0 : w;
    whi = zhi ? (T)0 : w;
    wloR = p ? wlo : w;
    wloB = p ? w : wlo;
    whiR = p ? w : whi;
    whiB = p ? whi : w;
    bloR = p ? b : b - klo;
    bloB = p ? b - klo : b;
    bhiR = p ? b - khi : b;
    bhiB = p ? b : b - khi;
    if (NARROW) {
      zlo2 = !(per & 4) && oz == DZ;
      zhi2 = !(per & 4) && oz + 2 * DZ == n;
      const T k0 = zlo2 ? wall_factor<T>(A.bc, 4) : (T)0, k9 = zhi2 ? wall_factor<T>(A.bc, 5) : (T)0;
      w0R = zlo2 && p ? (T)0 : wlo;
      w0B = zlo2 && !p ? (T)0 : wlo;
      w9R = zhi2 && !p ? (T)0 : whi;
      w9B = zhi2 && p ? (T)0 : whi;
      b0R = p ? b : b - k0;
      b0B = p ? b - k0 : b;
      b9R = p ? b - k9 : b;
      b9B = p ? b : b - k9;
    }
  }
  auto weight = [&](bool redc, int q) __attribute__((always_inline)) {
    if (!WALLS) return w6;
    if (NARROW && q == 0) return redc ? w0R : w0B;
    if (NARROW && q == NQ - 1) return redc ? w9R : w9B;
    return q < QL ? wlo : q == QL ? (redc ? wloR : wloB) : q == QH ? (redc ? whiR : whiB) : q > QH ? whi : w;
  };
  auto coef = [&](bool redc, int q) __attribute__((always_inline)) {
    if (!WALLS) return (T)6;
    if (NARROW && q == 0) return redc ? b0R : b0B;
    if (NARROW && q == NQ - 1) return redc ? b9R : b9B;
    return q == QL ? (redc ? bloR : bloB) : q == QH ? (redc ? bhiR : bhiB) : b;
  };

  // storage offset of plane oz - H + l in lane l (the parts of a storage index add), read back
  // per plane as a scalar
  const unsigned zpart = fine_at(A, 0, 0, (oz - H + (tid & 63)) & nm) * (unsigned)sizeof(T);
  const unsigned cpart = fine_at(A, i, j, 0) * (unsigned)sizeof(T);
  auto cell_off = [&](int jz) __attribute__((always_inline)) {
    return cpart + (unsigned)__builtin_amdgcn_readlane((int)zpart, jz);
  };

  // ---- up: the coarse cells under the tile, asked for first (they are waited for in LDS)
  constexpr int NCL = UP ? (CX * CY * CZ + kThreads - 1) / kThreads : 1;
  T cpre[NCL];
  if constexpr (UP) {
    const T* __restrict__ ec = reinterpret_cast<const T*>(A.ec);
    const int cx0 = (ox >> 1) - (H + 1) / 2, cy0 = (oy >> 1) - (H + 1) / 2, cz0 = (oz >> 1) - (H + 1) / 2;
#pragma unroll
    for (int t = 0; t < NCL; ++t) {
      const int q = min(tid + t * kThreads, CX * CY * CZ - 1);
      cpre[t] = coarse_hom<T, WALLS>(A, ec, cx0 + q % CX, cy0 + (q / CX) % CY, cz0 + q / (CX * CY));
    }
  }

  // ---- the column: u and f of every cell, split by colour
  T R[NQ], B[NQ], fR[NQ], fB[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const unsigned c0 = cell_off(2 * q), c1 = cell_off(2 * q + 1);
    T u0 = *reinterpret_cast<const T*>(uin + c0), u1 = *reinterpret_cast<const T*>(uin + c1);
    T f0 = *reinterpret_cast<const T*>(fin + c0), f1 = *reinterpret_cast<const T*>(fin + c1);
    if (WALLS) {
      const int k0 = oz - H + 2 * q, k1 = k0 + 1;
      const bool in0 = in && ((per & 4) || (unsigned)k0 < (unsigned)n), in1 = in && ((per & 4) || (unsigned)k1 < (unsigned)n);
      u0 = in0 ? u0 : (T)0;
      f0 = in0 ? f0 : (T)0;
      u1 = in1 ? u1 : (T)0;
      f1 = in1 ? f1 : (T)0;
      if constexpr (VALUES) {
        // 2 / h^2 times the values of the faces that cell k of the column touches
        auto values = [&](int k) __attribute__((always_inline)) {
          auto at = [&](int face, int t1, int t2) __attribute__((always_inline)) {
            return A.bc.b[face][(size_t)(t2 + 1) * (size_t)(n + 2) + (size_t)(t1 + 1)];
          };
          double v = 0.0;
          if (A.bc.b[0] && i == 0) v += at(0, j, k);
          if (A.bc.b[1] && i == nm) v += at(1, j, k);
          if (A.bc.b[2] && j == 0) v += at(2, i, k);
          if (A.bc.b[3] && j == nm) v += at(3, i, k);
          if (A.bc.b[4] && k == 0) v += at(4, i, j);
          if (A.bc.b[5] && k == nm) v += at(5, i, j);
          return 2.0 * A.ih2 * v;
        };
        if (in0) f0 = (T)((double)f0 - values(k0 & nm));
        if (in1) f1 = (T)((double)f1 - values(k1 & nm));
      }
    }
    R[q] = p ? u0 : u1;
    B[q] = p ? u1 : u0;
    fR[q] = p ? f0 : f1;
    fB[q] = p ? f1 : f0;
  }
  if constexpr (UP) {
    // ---- u += trilinear prolongation (weights 3/4, 1/4 per axis).  The tile starts at an odd
    // fine cell, so tile coordinates 2a and 2a + 1 lie between coarse cells a and a + 1
    T* ctile = &ex[0][0];
#pragma unroll
    for (int q = 0; q < NCL; ++q)
      if (tid + q * kThreads < CX * CY * CZ) ctile[tid + q * kThreads] = cpre[q];
    __syncthreads();
    const T* c = ctile + (ty >> 1) * CX + (tx >> 1);
    const T wx1 = (tx & 1) ? (T)0.75 : (T)0.25, wy1 = (ty & 1) ? (T)0.75 : (T)0.25;
    const T wx0 = (T)1 - wx1, wy0 = (T)1 - wy1;
    auto plane = [&](int z) __attribute__((always_inline)) {
      const T* e = c + z * (CX * CY);
      return wy0 * (wx0 * e[0] + wx1 * e[1]) + wy1 * (wx0 * e[CX] + wx1 * e[CX + 1]);
    };
    T e0 = plane(0);
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const T e1 = plane(q + 1);
      T lo = (T)0.75 * e0 + (T)0.25 * e1, hi = (T)0.25 * e0 + (T)0.75 * e1;
      if (WALLS) {
        const int k0 = oz - H + 2 * q;
        lo = in && ((per & 4) || (unsigned)k0 < (unsigned)n) ? lo : (T)0;
        hi = in && ((per & 4) || (unsigned)(k0 + 1) < (unsigned)n) ? hi : (T)0;
      }
      R[q] += p ? lo : hi;
      B[q] += p ? hi : lo;
      e0 = e1;
    }
    __syncthreads();
  }

  // ---- colour passes
  // the columns around; those past the rim read a column of the rim (what a rim column computes
  // never reaches the region)
  const int xl = col - (tx > 0 ? 1 : 0), xh = col + (tx < WX - 1 ? 1 : 0);
  const int yl = col - (ty > 0 ? WX : 0), yh = col + (ty < WY - 1 ? WX : 0);
  auto put = [&](T* to, const T* v, int m) __attribute__((always_inline)) {
    if (2 * m + 1 < NQ) reinterpret_cast<v2*>(to + 2 * m * COLS)[col] = v2{v[2 * m], v[2 * m + 1]};
    else to[(NQ - 1) * COLS + col] = v[NQ - 1];
  };
  // sum of the four lateral neighbours of slots 2m, 2m + 1
  auto lateral = [&](const T* from, int m) __attribute__((always_inline)) {
    if (2 * m + 1 < NQ) {
      const v2* e = reinterpret_cast<const v2*>(from + 2 * m * COLS);
      return (e[xl] + e[xh]) + (e[yl] + e[yh]);
    }
    const T* e = from + (NQ - 1) * COLS;
    return v2{(e[xl] + e[xh]) + (e[yl] + e[yh]), (T)0};
  };
  // r of slot q of `own` (upper cells of the slots: up), lateral sum s4
  auto resid = [&](const T* own, const T* oth, const T* fs, bool redc, bool up, int q, T s4) __attribute__((always_inline)) {
    const T above = q + 1 < NQ ? oth[q + 1 < NQ ? q + 1 : 0] : (T)0, below = q > 0 ? oth[q > 0 ? q - 1 : 0] : (T)0;
    return (mh2 * fs[q] + (s4 + (oth[q] + (up ? above : below)))) - coef(redc, q) * own[q];
  };
#pragma unroll
  for (int m = 0; m < (NQ + 1) / 2; ++m) put(ex[1], B, m);
  __syncthreads();
#pragma unroll
  for (int pass = 0; pass < 2 * NS; ++pass) {
    const bool redc = (pass & 1) == 0;
    T* own = redc ? R : B;
    const T* oth = redc ? B : R;
    const T* fs = redc ? fR : fB;
    const int ring = 2 * NS - pass;   // the region and a ring of this many cells
    const int q0 = (H - ring) / 2, q1 = (H + DZ + ring - 1) / 2;
#pragma unroll
    for (int m = 0; m < (NQ + 1) / 2; ++m) {
      if (2 * m + 1 < q0 || 2 * m > q1) continue;
      const v2 s4 = lateral(ex[redc ? 1 : 0], m);
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int q = 2 * m + t;
        if (q < q0 || q > q1 || q >= NQ) continue;
        own[q] += weight(redc, q) * resid(own, oth, fs, redc, redc ? !p : p, q, t ? s4.y : s4.x);
      }
      put(ex[redc ? 0 : 1], own, m);
    }
    __syncthreads();
  }

  // ---- the region back to memory
#pragma unroll
  for (int m = 0; m < MZ; ++m) {
    const unsigned c0 = cell_off(H + 2 * m), c1 = cell_off(H + 2 * m + 1);
    if (own_col) {
      *reinterpret_cast<T*>(uout + c0) = p ? B[QL + m] : R[QL + m];
      *reinterpret_cast<T*>(uout + c1) = p ? R[QL + m + 1] : B[QL + m + 1];
    }
  }

  // ---- residuals of the region's slots QL..QH: for the restriction (per coarse plane the two
  // cells of the column added) or the norm
  const bool fas = !UP && A.pbar, norm = UP && A.sink.part;
  if (!UP || norm) {
    T zs[UP ? 1 : MZ];
    double acc = 0.0;
    T upR = (T)0, upB = (T)0;
#pragma unroll
    for (int m = QL / 2; m <= QH / 2; ++m) {
      const v2 sR = lateral(ex[1], m), sB = lateral(ex[0], m);
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int q = 2 * m + t;
        if (q < QL || q > QH) continue;
        const T r = resid(R, B, fR, true, !p, q, t ? sR.y : sR.x);
        const T g = resid(B, R, fB, false, p, q, t ? sB.y : sB.x);
        // coarse plane q - QL - 1: the upper cell of slot q - 1 and the lower one of slot q
        if constexpr (!UP) {
          if (q > QL) zs[q - QL - 1] = p ? upB + r : upR + g;
        } else {
          // of slot QL only the upper cell lies in the region, of slot QH only the lower
          const bool inR = (q != QL || !p) && (q != QH || p), inB = (q != QL || p) && (q != QH || !p);
          acc += (inR ? (double)r * (double)r : 0.0) + (inB ? (double)g * (double)g : 0.0);
        }
        upR = r;
        upB = g;
      }
    }
    if constexpr (!UP) {
      __syncthreads();
      T* sum = &ex[0][0];
#pragma unroll
      for (int m = 0; m < MZ; ++m) {
        sum[m * COLS + col] = zs[m];
        if (fas) sum[(MZ + m) * COLS + col] = p ? B[QL + m] + R[QL + m + 1] : R[QL + m] + B[QL + m + 1];
      }
      __syncthreads();
      T* __restrict__ fc = reinterpret_cast<T*>(A.fc);
      T* __restrict__ uc0 = reinterpret_cast<T*>(A.uc0);
      const T sc = (T)(-0.125 * A.ih2);
      for (int q = tid; q < (DX / 2) * (DY / 2) * MZ; q += kThreads) {
        const int cx = q % (DX / 2), cy = (q / (DX / 2)) % (DY / 2), cz = q / ((DX / 2) * (DY / 2));
        const T* s = sum + cz * COLS + (H + 2 * cy) * WX + H + 2 * cx;
        const unsigned ci = coarse_at(A, (ox >> 1) + cx, (oy >> 1) + cy, (oz >> 1) + cz);
        fc[ci] = sc * ((s[0] + s[1]) + (s[WX] + s[WX + 1]));
        if (fas) {
          s += MZ * COLS;
          const T pb = (T)0.125 * ((s[0] + s[1]) + (s[WX] + s[WX + 1]));
          reinterpret_cast<T*>(A.pbar)[ci] = pb;
          uc0[ci] = pb;
        } else {
          if (uc0) uc0[ci] = (T)0;
        }
      }
    } else {
      acc = wave_sum(own_col ? acc : 0.0);
      if ((tid & 63) == 0) red[tid >> 6] = acc;
      __syncthreads();
      double t = 0.0;
      if (tid == 0)
        for (int q = 0; q < kThreads / 64; ++q) t += red[q];
      __syncthreads();
      finish_sum<kThreads>(A.sink, t * (A.ih2 * A.ih2), red);
    }
  }
}

template <typename T>
TileArgs base_args(const T* uin, T* uout, const T* f, int n, int Lm, double h, double omega, const LevelBC& bc) {
  TileArgs A{};
  A.uin = uin;
  A.uout = uout;
  A.f = f;
  A.bc = bc;
  A.n = n;
  A.L = ilog2(n);
  A.Lm = Lm;
  A.per = (bc.kind[0] == BC_PERIODIC ? 1 : 0) | (bc.kind[2] == BC_PERIODIC ? 2 : 0) | (bc.kind[4] == BC_PERIODIC ? 4 : 0);
  const Shape sh = kShapes[shape_of(n)];
  A.nrx = n / sh.dx;
  A.nry = n / sh.dy;
  A.h2 = h * h;
  A.ih2 = 1.0 / (h * h);
  A.omega = omega;
  return A;
}

int regions(int n) {
  const Shape sh = kShapes[shape_of(n)];
  return (n / sh.dx) * (n / sh.dy) * (n / sh.dz);
}

// One launch of the leg in the region shape of level side n.
template <typename T, int NS, bool UP, bool WALLS, bool VALUES>
void launch_shape(const TileArgs& A, hipStream_t s) {
  const dim3 g(regions(A.n));
  switch (shape_of(A.n)) {
    case 0: launch_maybe_timed(k_tile_leg<T, NS, UP, WALLS, 0, VALUES>, g, dim3(tile_threads(NS, 0)), 0, s, A); break;
    default: launch_maybe_timed(k_tile_leg<T, NS, UP, WALLS, 1, VALUES>, g, dim3(tile_threads(NS, 1)), 0, s, A); break;
  }
}
// Measured per launch, down / up, FP64 periodic: 64^3 9.5 / 11.2 us with two sweeps (six gathered
// neighbours per update: 15.1 / 22.3), 6.3 / 7.3 with one; 32^3 6.5 / 6.8 (9.3 / 11.4) and 4.7 / 4.9;
// FP32 with walls 64^3 6.8 / 9.0, 32^3 5.3 / 6.7.  At 128^3 47 / 49 us with walls, where the
// streaming passes are faster (march_min_n).  Bound by the chain of LDS exchanges and barriers, one per
// colour, of workgroups of one residency.
template <typename T, int NS, bool UP>
void launch_leg(TileArgs A, hipStream_t s) {
  bool values = false;
  for (int f = 0; f < 6; ++f) {
    if (!bc_has_value(A.bc.kind[f])) A.bc.b[f] = nullptr;
    values = values || A.bc.b[f];
  }
  if (values) launch_shape<T, NS, UP, true, true>(A, s);
  else if (A.per != 7) launch_shape<T, NS, UP, true, false>(A, s);
  else launch_shape<T, NS, UP, false, false>(A, s);
}

}  // namespace

template <typename T, int NS>
void tile_down_ns(const T* uin, T* uout, const T* f, T* fc, T* pbar, T* uc0, int n, int Lm, double h, double omega,
                  const LevelBC& bc, hipStream_t s) {
  TileArgs A = base_args(uin, uout, f, n, Lm, h, omega, bc);
  A.fc = fc;
  A.pbar = pbar;
  A.uc0 = uc0;
  launch_leg<T, NS, false>(A, s);
}

template <typename T, int NS>
void tile_up_ns(const T* uin, T* uout, const T* f, const T* ec, const LevelBC& bcc, const SumSink* sink, int n, int Lm,
                double h, double omega, const LevelBC& bc, hipStream_t s) {
  TileArgs A = base_args(uin, uout, f, n, Lm, h, omega, bc);
  A.ec = ec;
  A.bcc = bcc;
  if (sink) A.sink = *sink;
  A.sink.total = regions(n);
  launch_leg<T, NS, true>(A, s);
}

#define MG_TILE_INST(T, NS)                                                                                       \
  template void tile_down_ns<T, NS>(const T*, T*, const T*, T*, T*, T*, int, int, double, double, const LevelBC&, \
                                    hipStream_t);                                                                 \
  template void tile_up_ns<T, NS>(const T*, T*, const T*, const T*, const LevelBC&, const SumSink*, int, int,     \
                                  double, double, const LevelBC&, hipStream_t);

}  // namespace mg
