// mg_march.inl -- streaming passes of the large levels (the bandwidth path), one or two sweeps each;
// included per precision and sweep count by mg_march_f64_1.hip and its siblings.
//
// One launch = the whole work of a V-cycle leg on one level, with u and f crossing HBM once:
//   down (Alg. 1 steps 1-3): two (or one) red-black SOR sweeps (eqs. rbsor1-2), then the defect
//        f - L u of the result (eq. defect) restricted to the coarse level (eq. restriction)
//        and the coarse correction cleared;
//   up   (Alg. 1 steps 5-7): u += trilinear prolongation of the coarse correction (eq.
//        trilinear) as u is loaded, then the sweeps, optionally followed by the defect of the
//        result summed as squares (the convergence norm of Sec. 2.3.7);
//   FAS down (Alg. 3 steps 2-4, k_march_fas): the down leg with the swept u restricted beside
//        the defect (phibar, also the coarse level's starting iterate).
//
// Work layout.  A workgroup of W = 8 waves owns a tile of 64 x 64 cells in x-y and marches a
// chunk of z planes.  Each half-wave holds a band of R = 4 rows, each lane the x-pair (2l, 2l+1)
// of those rows.  At the step that loads plane P the stages run on older planes (two sweeps; one
// sweep has the first two stages, a ring of four planes and one LDS slot):
//   red sweep 1 on P-1, black 1 on P-2, red 2 on P-3, black 2 on P-4, defect on P-4,
// so every stage reads its z-neighbours in the colour state it needs.  u of six planes lives in
// registers (a ring), f of plane P-1 in registers and of P-2..P-4 in per-thread LDS slots.
//
// The colour pattern is a compile-time constant: tile origins, halos and z-chunk starts are
// even and the ring has 6 planes, so the parity of the plane a
// stage works on, and which cell of a lane's x-pair is red in each row, are template constants.
// A stage then updates exactly one cell per row with no operand selection: two cross-lane moves
// (DPP wave shifts) for the x-neighbour, in-lane rows or an LDS exchange of the band-edge rows
// for y, ring planes for z.
//
// What bounds it: HBM at 512^3 (3.5 GB a leg at 4.2 TB/s), at 256^3 and below the step's chain of
// LDS, barriers and dependent FP64 operations with two waves per SIMD.  Hence
//  * one barrier for the four sweep stages: the y neighbours a stage reads beyond its band have
//    the colour that no stage of this step changes on that plane, so all four stages' edge rows go
//    out at the step's start, and the inner rows are done while they travel (the defect stage's
//    red cells need one more);
//  * no branch around a load or its take-up, and below 256^3 the step's stores after the take-up: loads
//    and stores complete in one order, so a wait for loads behind stores, or at a join of paths, waits
//    for the stores to reach memory.  (Where memory is the bound that wait costs nothing and the stores'
//    earlier start gains: march_early.)
//  * addresses are a uniform plane base and a 32-bit offset, coarse taps take their walls' signs
//    when they are used, not as they are loaded.
// Measured before these and now: 128^3 periodic legs 39 / 34 -> 32 / 32 us; V-cycles at 256^3
// 386 -> 307 us periodic, 451 -> 336 between z walls, 522 -> 383 fixed; at 512^3 2000 -> 1791,
// 2285 -> 1777 and 2610 -> 1931.  Loading two planes ahead: FP32 equal, FP64 spills.
//
// The defect stage needs the final state of both neighbouring planes.  Black cells of P-4 have
// only red neighbours, final after red sweep 2; red cells of P-4 get their in-plane and lower
// neighbours now and the upper one (black, final one step later) at the next step, so the ring
// stays at six planes.  Tiles overlap by a halo of 6 cells (5 stages of radius 1, rounded up to
// even) and are recomputed, so tiles are independent and the result goes to another array.
//
// Non-periodic faces (Sec. 2.3.6): face values b enter the source of the cells beside them, as
// f - 2 b / h^2 (in f already in a solve: launch_fold_faces; as f is taken up in the passes of the
// operator entry points, whose f is the caller's: k_march_values), so a ghost is kappa
// times the adjacent active cell's current value, +1 at a zero-gradient face and -1 at a fixed one:
//   x: the lane holding x = 0 (x = n-1) takes kappa * c in place of its left (right) neighbour;
//   y: with 52-row output tiles and a halo of 6 the rows beyond y = 0 and y = n-1 are always
//      rows 1 and 2 of the same lane as their active neighbour; before each stage the ghost
//      cells the stage reads are set to kappa times that neighbour (in-lane);
//   z: planes outside are zero and stay so (their updates have weight zero), and on the first
//      and last plane kappa times the cell's own value joins its neighbours (kappa uniform and 0
//      inside: one multiply-add an update).
// Cells outside in x or y are loaded from their periodic image (every address in range, no
// predicated loads) and swept like the others; no active cell reads them.  The coarse
// correction's taps (homogeneous conditions) are clamped to the domain with the sign of each
// face's rule.
#include "mg_march.h"

#if !defined(MG_MARCH_T) || !defined(MG_MARCH_NS)
#error "define MG_MARCH_T and MG_MARCH_NS (the precision and the sweeps per pass this translation unit instantiates)"
#endif

#include <algorithm>
#include <cstring>
#include <type_traits>
#include <utility>

#include "mg_launch.h"

namespace mg {

namespace {

constexpr int kLanes = 64;
constexpr int kR = 4;          // rows per lane (a band)
constexpr int kSL = 32;        // lanes per x segment (a half-wave)
constexpr int kTX = 2 * kSL;   // tile width
constexpr int kNS = MG_MARCH_NS;         // sweeps per pass
constexpr int kStages = 2 * kNS;         // colour updates
constexpr int kRing = kStages + 2;       // u planes held per lane
constexpr int kFSlots = kStages - 1;     // f planes held in LDS per lane
constexpr int kHalo = 6;       // tile overlap in x and y

struct MarchArgs {
  const void* uin;   // u on input (not read when zero_in)
  void* uout;
  const void* f;
  const void* ec;    // up: coarse correction (n/2)^3
  void* fc;          // down: restricted defect (n/2)^3
  void* uc0;         // down: coarse correction to clear, or null (FAS: to start from phibar)
  void* pbar;        // FAS down: the restricted potential phibar
  SumSink sink;      // norm: where the sum of squared defects goes
  LevelBC bc;        // this level
  LevelBC bcc;       // up: coarse level (homogeneous)
  int n, L, xo, yo, zc, tiles_x, tiles_y, ntiles;
  int set;           // tiles of this launch: 0 all, 1 the interior ones, 2 the ring at the walls
  int Lm;            // BLK: log2 of the MeshBlock side on this level (the coarse level: Lm - 1)
  double h2, ih2, omega;
};

template <int N, typename F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl<N>(f, std::make_integer_sequence<int, N>{});
}

// Whole-wave shift by one lane through DPP: wave_shr:1 gives lane i the value of lane i-1,
// wave_shl:1 the value of lane i+1.  Lanes without a source read zero (bound control), which leaves
// the destination untied from the source (no copy before each move).  Those lanes, and the edge
// lanes of each half-wave, hold the outermost columns of a tile, inside its halo.
constexpr int kDppWaveShr1 = 0x138;
constexpr int kDppWaveShl1 = 0x130;

template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
  const long long b = __builtin_bit_cast(long long, v);
  const int lo2 = __builtin_amdgcn_mov_dpp((int)(b & 0xffffffffLL), CTRL, 0xf, 0xf, true);
  const int hi2 = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((long long)hi2 << 32) | (long long)(unsigned)lo2);
}
template <typename T>
__device__ __forceinline__ T from_left(T v) {   // value of lane - 1
  return dpp_move<kDppWaveShr1>(v);
}
template <typename T>
__device__ __forceinline__ T from_right(T v) {  // value of lane + 1
  return dpp_move<kDppWaveShl1>(v);
}

// Ghost rule of a face as ghost = kappa * adjacent: zero gradient 1, fixed (and multipole) -1.
template <typename T>
__device__ __forceinline__ T kappa_of(const LevelBC& bc, int face) {
  return bc.kind[face] == BC_ZERO_GRADIENT ? (T)1 : (T)-1;
}

// The 2 x 8 values are in registers here, the loads that made them complete.
template <typename T>
__device__ __forceinline__ void arrived(const T (&a)[kR][2], const T (&b)[kR][2]) {
  static_assert(kR == 4, "four rows");
  asm volatile("" ::"v"(a[0][0]), "v"(a[0][1]), "v"(a[1][0]), "v"(a[1][1]), "v"(a[2][0]), "v"(a[2][1]), "v"(a[3][0]),
               "v"(a[3][1]), "v"(b[0][0]), "v"(b[0][1]), "v"(b[1][0]), "v"(b[1][1]), "v"(b[2][0]), "v"(b[2][1]),
               "v"(b[3][0]), "v"(b[3][1])
               : "memory");
}

// v with its sign bit flipped by `bit`
__device__ __forceinline__ float with_sign(float v, unsigned bit) {
  return __builtin_bit_cast(float, __builtin_bit_cast(unsigned, v) ^ bit);
}
__device__ __forceinline__ double with_sign(double v, unsigned bit) {
  return __builtin_bit_cast(double, __builtin_bit_cast(unsigned long long, v) ^ ((unsigned long long)bit << 32));
}

template <typename T>
struct alignas(2 * sizeof(T)) Pair {
  T a, b;
};

// MeshBlock storage index split into its x-y part and its z part (disjoint bits, so the index
// is their sum): the x-y part is fixed per lane and row, the z part is uniform per plane.  Both
// are 32-bit (a 64-bit index costs these passes register spills): the launcher sends only
// levels of fewer than 2^32 cells here.
__device__ __forceinline__ unsigned blk_xy(int Lm, int i, int j) {
  const int mm = (1 << Lm) - 1;
  return ((spread3((unsigned)(i >> Lm)) | (spread3((unsigned)(j >> Lm)) << 1)) << (3 * Lm)) |
         (unsigned)(((j & mm) << Lm) | (i & mm));
}
__device__ __forceinline__ unsigned blk_z(int Lm, int k) {
  const int mm = (1 << Lm) - 1;
  return ((spread3((unsigned)(k >> Lm)) << 2) << (3 * Lm)) | (unsigned)((k & mm) << (2 * Lm));
}

// Waves per workgroup: 8 (a 64 x 64 tile, 2 waves per SIMD with up to 256 registers per lane;
// FP32 on 16 waves, a 64 x 128 tile, needs more than the 128 registers that leaves per lane).
constexpr int kWaves = kMarchWaves;

// WALLS: 0 = every face of the level is periodic (no boundary code compiled in); 1 = walls
// only across z (x and y periodic, or a tile that reaches no x or y wall with its halo: no x/y
// wall code compiled in); 2 = walls on any axis.  The launcher picks per tile.  ZIN: u is zero on
// input and not read.  BLK: the level is in the MeshBlock layout (blocks of 2^A.Lm cells, Morton order);
// the tile streams across block boundaries as across a dense array (an x-pair never straddles
// two blocks), and the coarse level is in the layout below (blocks of 2^(A.Lm-1) cells, or the
// dense root grid when that is one cell).
// FAS (down only, Alg. 3 steps 2-4): the restriction also writes the restricted potential
// phibar (mean of the 8 children of the pass's result) into A.pbar and starts the coarse level
// from it (uc0 = phibar instead of 0).
// VALUES: the face values are in A.bc and not in f (null: none on that face).
// EARLY: a step's stores before its loads are taken up, else after.
template <typename T, int W, bool UP, bool NORM, int WALLS, bool BLK, bool FAS, bool ZIN, bool VALUES, bool EARLY>
__device__ __forceinline__ void march_body(const MarchArgs& A) {
  constexpr bool PER = WALLS == 0;                // every face periodic
  constexpr bool XYW = WALLS == 2;                // x or y walls may be in reach
  constexpr bool DREG = PER || kNS == 1;          // registers to carry the red partial defects in
  constexpr int R = kR, SL = kSL, NB = 2 * W, NT = kLanes * W;
  constexpr bool DEF = !UP;                       // down: restricted defect
  constexpr bool DSTAGE = DEF || NORM;            // a defect stage after the sweeps
  constexpr int HZ = kStages + (DSTAGE ? 1 : 0);  // planes marched before (and after) the chunk
  __shared__ T xe[kStages][NB][2][SL];                  // per stage: the bands' first and last rows
  __shared__ T xd[DSTAGE ? NB : 1][2][SL];        // the same of the defect stage's black cells
  __shared__ Pair<T> fl[kFSlots][R][NT];
  // the red cells' partial defects carried to the next step, where registers are short
  __shared__ T dredl[DREG ? 1 : R][DREG ? 1 : NT];

  const int tid = threadIdx.x;
  const int lane = tid & (kLanes - 1);
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int seg = lane >> 5;
  const int xl = lane & (SL - 1);
  const int band = 2 * w + seg;
  // XCD-aware order: consecutive block ids go to different XCDs, so give each XCD a
  // contiguous run of tiles (neighbouring tiles then share that XCD's L2 for their halos)
  const int nbk = gridDim.x, bid = blockIdx.x;
  const int tile = (bid & 7) * (nbk >> 3) + (bid >> 3);
  double acc = 0.0;
  if (tile < A.ntiles) {
    // tile coordinates and z-chunk: every tile; the interior rectangle [1, tiles_x - 1) x
    // [1, tiles_y - 1); or the ring around it (bottom row, top row, then the two side columns)
    int tx, ty, cz;
    if (A.set == 0) {
      tx = tile % A.tiles_x;
      ty = (tile / A.tiles_x) % A.tiles_y;
      cz = tile / (A.tiles_x * A.tiles_y);
    } else if (A.set == 1) {
      const int wi = A.tiles_x - 2, per = wi * (A.tiles_y - 2), t = tile % per;
      cz = tile / per;
      tx = 1 + t % wi;
      ty = 1 + t / wi;
    } else {
      const int per = 2 * A.tiles_x + 2 * (A.tiles_y - 2);
      int q = tile % per;
      cz = tile / per;
      if (q < A.tiles_x) {
        tx = q;
        ty = 0;
      } else if (q < 2 * A.tiles_x) {
        tx = q - A.tiles_x;
        ty = A.tiles_y - 1;
      } else {
        q -= 2 * A.tiles_x;
        tx = (q & 1) ? A.tiles_x - 1 : 0;
        ty = 1 + (q >> 1);
      }
    }
    const int n = A.n, L = A.L, nm = n - 1;
    const T* __restrict__ uin = reinterpret_cast<const T*>(A.uin);
    T* __restrict__ uout = reinterpret_cast<T*>(A.uout);
    const T* __restrict__ fin = reinterpret_cast<const T*>(A.f);
    // storage index of cell (X, Y, Z) of the coarse level below
    auto cdx = [&](int X, int Y, int Z) __attribute__((always_inline)) {
      return BLK ? lidx(L - 1, A.Lm - 1, X, Y, Z) : cidx(L - 1, X, Y, Z);
    };
    const bool px = !XYW || A.bc.kind[0] == BC_PERIODIC;
    const bool py = !XYW || A.bc.kind[2] == BC_PERIODIC;
    const bool pz = PER || A.bc.kind[4] == BC_PERIODIC;
    const T h2 = (T)A.h2, ih2 = (T)A.ih2, omega = (T)A.omega;
    const T inv6 = (T)(1.0 / 6.0);

    const int xs = tx * A.xo;                    // first output column (even)
    const int xa = xs - kHalo + 2 * xl;          // this lane's even column
    const int xag = xa & nm;
    const bool out_x = xa >= xs && xa < xs + A.xo && xa < n;
    // the lane whose even cell is x = 0, whose odd cell is x = n-1 (beside a wall)
    [[maybe_unused]] const bool wx0 = XYW && !px && xa == 0;
    [[maybe_unused]] const bool in_x = px || (xa >= 0 && xa < n);
    [[maybe_unused]] const bool wx1 = XYW && !px && xa == n - 2;

    const int ys = ty * A.yo;                    // first output row (even)
    int yv[R], ygv[R];
    [[maybe_unused]] bool in_y[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int y = ys - kHalo + band * R + r;
      yv[r] = y;
      ygv[r] = y & nm;
      in_y[r] = py || (y >= 0 && y < n);
    }
    // rows 0, 1 and rows 2, 3: written by this lane?
    const bool out[2] = {out_x && yv[0] >= ys && yv[0] < ys + A.yo && yv[0] < n,
                         out_x && yv[2] >= ys && yv[2] < ys + A.yo && yv[2] < n};
    // MeshBlock layout: the x-y part of each row's storage index (the z part is added per plane)
    unsigned rxy[BLK ? R : 1];
    if constexpr (BLK) {
#pragma unroll
      for (int r = 0; r < R; ++r) rxy[r] = blk_xy(A.Lm, xag, ygv[r]);
    }
    // dense layout: the row pairs' byte offsets within a plane (below 2^25 up to 2048^2 cells; a
    // pair neither wraps nor straddles a wall or the output's edge: all lie between rows 1 and 2), so that
    // an address is a uniform plane base and a 32-bit offset, with no arithmetic per load
    unsigned rb[2];
    rb[0] = (unsigned)(((ygv[0] << L) | xag) * (int)sizeof(T));
    rb[1] = (unsigned)(((ygv[2] << L) | xag) * (int)sizeof(T));
    // row r of this lane on plane z of array p
    auto at = [&](const T* p, int r, int z) __attribute__((always_inline)) -> const T* {
      if constexpr (BLK) return p + (size_t)(rxy[r] + blk_z(A.Lm, z));
      else return reinterpret_cast<const T*>(reinterpret_cast<const char*>(p + (((size_t)z << (2 * L)) + ((r & 1) << L))) + rb[r >> 1]);
    };
    // up, MeshBlock layout: the x-y part of the coarse taps' storage indices (rows Y0-1 ..
    // Y0+2 of the lane's coarse column, wrapped or clamped as the taps take them); the coarse
    // level is in blocks of 2^(Lm-1) cells, or the dense root grid when Lm = 1
    constexpr int NTAP = R / 2 + 2;
    unsigned cxy[UP ? NTAP : 1];
    unsigned sgn[UP && XYW ? NTAP / 2 : 1];   // the sign of the walls' rule of a clamped pair of taps, as its bit
    if constexpr (UP) {
      const int nc = n >> 1, Lc = L - 1;
      int X = (px ? xag : xa) >> 1;
      const bool minus_x = XYW && ((X < 0 && kappa_of<T>(A.bcc, 0) < 0) || (X >= nc && kappa_of<T>(A.bcc, 1) < 0));
      if constexpr (XYW) X = min(max(X, 0), nc - 1);
      const int Y0 = (py ? ygv[0] : yv[0]) >> 1;
#pragma unroll
      for (int i = 0; i < NTAP; ++i) {
        int Y = Y0 - 1 + i;
        if (py) Y &= nc - 1;
        if constexpr (XYW) {
          const bool minus_y = (Y < 0 && kappa_of<T>(A.bcc, 2) < 0) || (Y >= nc && kappa_of<T>(A.bcc, 3) < 0);
          // (a wall lies between taps 1 and 2, as between rows 1 and 2)
          if (i % 2 == 0) sgn[i / 2] = minus_x != minus_y ? 0x80000000u : 0u;
          Y = min(max(Y, 0), nc - 1);
        }
        if constexpr (BLK) cxy[i] = A.Lm == 1 ? (unsigned)((Y << Lc) | X) : blk_xy(A.Lm - 1, X, Y);
        else cxy[i] = (unsigned)(((Y << Lc) | X) * (int)sizeof(T));   // in bytes
      }
    }
    const int z0 = cz * A.zc;                    // even
    const int zend = min(z0 + A.zc, n);
    const int zstart = z0 - HZ;
    const int nsteps = (zend - z0) + 2 * HZ;
    // rows 1 and 2 of this lane are the ghost row beyond y = 0 and its active neighbour, or the
    // active row y = n-1 and the ghost beyond it
    const T kx0 = kappa_of<T>(A.bc, 0), kx1 = kappa_of<T>(A.bc, 1), ky0 = kappa_of<T>(A.bc, 2);
    const T ky1 = kappa_of<T>(A.bc, 3);
    const bool gy0 = XYW && !py && yv[1] == -1;
    const bool gy1 = XYW && !py && yv[2] == n;
    // does any cell of this wave sit beside a wall in y?
    const int wy0 = ys - kHalo + w * 2 * R, wy1 = wy0 + 2 * R - 1;
    const bool wave_y = XYW && !py && (wy0 < 0 || wy1 >= n);
    // plane p: the z walls' factors on the own value, and the weight of an update (0 outside the domain)
    struct PlaneW {
      T kz, om;
    };
    auto plane_w = [&](int p) __attribute__((always_inline)) {
      PlaneW v;
      v.kz = (T)0;
      if (!pz && p == 0) v.kz += kappa_of<T>(A.bc, 4);
      if (!pz && p == nm) v.kz += kappa_of<T>(A.bc, 5);
      v.om = pz || (unsigned)p < (unsigned)n ? omega : (T)0;
      return v;
    };
    // up: the coarse correction's rules (homogeneous conditions)
    const T kcz0 = kappa_of<T>(A.bcc, 4), kcz1 = kappa_of<T>(A.bcc, 5);

    T u[kRing][R][2];
    T pu[R][2], pf[R][2];      // prefetched u of plane P+1 and f of plane P
    T fr[R][2];                // f of plane P-1
    T dred[DREG ? R : 1];      // red cells' partial defects of plane P-4 (completed next step)
    auto dred_get = [&](int r) __attribute__((always_inline)) -> T { return DREG ? dred[DREG ? r : 0] : dredl[DREG ? 0 : r][DREG ? 0 : tid]; };
    auto dred_set = [&](int r, T v) __attribute__((always_inline)) {
      if constexpr (DREG) dred[r] = v;
      else dredl[r][tid] = v;
    };
    T pend[R / 2], stash[R / 2];   // down: row-pair defect sums (black cells of P-4; even plane)
    T stash_u[FAS ? R / 2 : 1];      // FAS: row-pair sums of u on the even plane of a coarse plane
    T pc[UP ? NTAP : 1][2];    // up: coarse rows Y0-1 .. Y0+2 on the two coarse planes of a fine plane
#pragma unroll
    for (int s = 0; s < kRing; ++s)
#pragma unroll
      for (int r = 0; r < R; ++r) u[s][r][0] = u[s][r][1] = (T)0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      fr[r][0] = fr[r][1] = (T)0;
      dred_set(r, (T)0);
#pragma unroll
      for (int q = 0; q < kFSlots; ++q) fl[q][r][tid] = Pair<T>{(T)0, (T)0};
    }
#pragma unroll
    for (int j = 0; j < R / 2; ++j) pend[j] = stash[j] = (T)0;
    if constexpr (FAS) {
#pragma unroll
      for (int j = 0; j < R / 2; ++j) stash_u[j] = (T)0;
    }

    // u of plane P as loaded (and corrected): zero outside the domain
    auto keep_in = [&](int P) __attribute__((always_inline)) {
      if constexpr (!PER) {
        const bool in_z = pz || (unsigned)P < (unsigned)n;
#pragma unroll
        for (int r = 0; r < R; ++r) {
          pu[r][0] = in_z ? pu[r][0] : (T)0;
          pu[r][1] = in_z ? pu[r][1] : (T)0;
        }
      }
    };

    // ---- loads of u on plane P (unless zero on input) and f on plane P-1 (the plane the red
    // stage of the next step works on); up: the coarse taps
    // of plane P
    // cTAPS (up): 0 load both coarse planes of P, 1 (P odd) keep the upper plane of P-1 as the
    // lower one and load the upper, 2 (P even) keep the pair of P-1
    auto load_plane = [&](int P) __attribute__((always_inline)) {
      // f of a plane beyond a z wall is that of the first plane inside: the plane's updates weigh
      // nothing, but 0 times a value that is not finite is not 0, and so it reaches only cells
      // that the same value reaches inside
      const int Pg = P & nm, Pfg = pz ? (P - 1) & nm : min(max(P - 1, 0), nm);
      // no branch around a load: at a join the waits on it would turn conservative
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if constexpr (!ZIN) {
          const Pair<T> vu = *reinterpret_cast<const Pair<T>*>(at(uin, r, Pg));
          pu[r][0] = vu.a; pu[r][1] = vu.b;
        } else {
          pu[r][0] = pu[r][1] = (T)0;
        }
        const Pair<T> vf = *reinterpret_cast<const Pair<T>*>(at(fin, r, Pfg));
        pf[r][0] = vf.a; pf[r][1] = vf.b;
      }
    };
    auto load_taps = [&](int P, auto cTAPS) __attribute__((always_inline)) {
      if constexpr (UP) {
        // Trilinear prolongation (weights 1/4, 3/4 per axis) of the coarse correction: the
        // lane's coarse column X, coarse rows Y0-1 .. Y0+2 (rows 2j, 2j+1 of the band take
        // Y0+j-1 .. Y0+j+1) on the coarse planes (zlo, zlo+1) of fine plane P; the x-neighbour
        // columns come from the lanes beside (an edge lane of a segment gets zero or another
        // band's value: wrong, but only in the outermost column of the tile, inside the halo).  Fine
        // plane 2Z takes coarse planes (Z-1, Z), plane 2Z+1 (Z, Z+1), so the fine planes 2Z+1
        // and 2Z+2 take the same pair (also where the planes wrap or are clamped): an odd plane
        // loads one new coarse plane, an even one none (the parity is a template constant of
        // each pipeline step).
        constexpr int TAPS = decltype(cTAPS)::value;
        const T* __restrict__ ec = reinterpret_cast<const T*>(A.ec);
        const int nc = n >> 1, Lc = L - 1;
        const int X = (px ? xag : xa) >> 1;
        const int Y0 = (py ? ygv[0] : yv[0]) >> 1;
        const int Pz = pz ? (P & nm) : P;
        const int Z = Pz >> 1;
        const int zlo = (Pz & 1) ? Z : Z - 1;
        auto tap = [&](int i, int zz) __attribute__((always_inline)) {
          int Y = Y0 - 1 + i;
          if (py) Y &= nc - 1;
          if (pz) zz &= nc - 1;
          // the lane's x-y part (wrapped, or clamped into the domain) plus the plane's z part
          const int Zc = PER ? zz : min(max(zz, 0), nc - 1);
          const T* ep;
          if constexpr (BLK) ep = ec + ((size_t)cxy[i] + (A.Lm == 1 ? ((size_t)Zc << (2 * Lc)) : (size_t)blk_z(A.Lm - 1, Zc)));
          else ep = reinterpret_cast<const T*>(reinterpret_cast<const char*>(ec + ((size_t)Zc << (2 * Lc))) + cxy[i]);
          return *ep;   // (as stored: the walls' signs when it is used, so that nothing waits here)
        };
        if constexpr (TAPS == 0) {
#pragma unroll
          for (int i = 0; i < NTAP; ++i) {
            pc[i][0] = tap(i, zlo);
            pc[i][1] = tap(i, zlo + 1);
          }
        } else if constexpr (TAPS == 1) {
#pragma unroll
          for (int i = 0; i < NTAP; ++i) {
            pc[i][0] = pc[i][1];
            pc[i][1] = tap(i, zlo + 1);
          }
        }
      }
    };

    // ---- add the prolonged correction fetched with plane P (parity PARP) to the prefetched u
    auto prolong_apply = [&](int P, auto cPAR) __attribute__((always_inline)) {
      if constexpr (UP) {
        constexpr int PARP = decltype(cPAR)::value;
        T wz0 = PARP ? (T)0.75 : (T)0.25, wz1 = PARP ? (T)0.25 : (T)0.75;
        if constexpr (!PER) {
          // (only the lower plane can lie below the domain, only the upper one above it)
          const int zlo = ((pz ? (P & nm) : P) + (PARP ? 0 : -1)) >> 1;
          if (!pz && zlo < 0) wz0 *= kcz0;
          if (!pz && zlo < -1) wz1 *= kcz0;
          if (!pz && zlo >= (n >> 1)) wz0 *= kcz1;
          if (!pz && zlo + 1 >= (n >> 1)) wz1 *= kcz1;
        }
        T czv[NTAP];
#pragma unroll
        for (int i = 0; i < NTAP; ++i) {
          czv[i] = wz0 * pc[i][0] + wz1 * pc[i][1];
          if constexpr (XYW) czv[i] = with_sign(czv[i], sgn[i / 2]);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const int j = r >> 1;
          const T c = (r & 1) ? (T)0.75 * czv[j + 1] + (T)0.25 * czv[j + 2] : (T)0.25 * czv[j] + (T)0.75 * czv[j + 1];
          const T cl = from_left(c), cr = from_right(c);
          pu[r][0] += (T)0.25 * cl + (T)0.75 * c;
          pu[r][1] += (T)0.75 * c + (T)0.25 * cr;
        }
      }
    };

    // ---- y walls: the ghost cells read by the active cells of colour COL (0 red, 1 black, 2
    // both) of the plane in uc (parity PAR), set to kappa times those cells' current values
    // (x walls are taken in the stencil)
    auto refresh = [&](auto cCOL, auto cPAR, T (&uc)[R][2]) __attribute__((always_inline)) {
      if constexpr (XYW) {
        constexpr int COL = decltype(cCOL)::value, PAR = decltype(cPAR)::value;
        // does cell e of row r have a colour being refreshed?
        auto sel = [](int r, int e) constexpr { return COL == 2 || ((r + PAR + COL) & 1) == e; };
        if (wave_y) {
          static_for<2>([&](auto ee) __attribute__((always_inline)) {
            constexpr int e = decltype(ee)::value;
            if constexpr (sel(2, e))
              if (gy0) uc[1][e] = ky0 * uc[2][e];
            if constexpr (sel(1, e))
              if (gy1) uc[2][e] = ky1 * uc[1][e];
          });
        }
      }
    };

    // ---- the y neighbours of a band's first and last rows, of the stage on plane P - 1 - S: cells of
    // the other colour, which no stage of this step changes (S = 0: as loaded; else set a step
    // ago), so all four stages' rows go out at the step's start under one barrier
    auto edges_out = [&](auto cS, auto cPAR, T (&uc)[R][2]) __attribute__((always_inline)) {
      constexpr int S = decltype(cS)::value, PAR = decltype(cPAR)::value, C = S & 1;
      constexpr int q0 = (PAR + C) & 1, qL = (R - 1 + PAR + C) & 1;
      xe[S][band][0][xl] = uc[0][q0 ^ 1];
      xe[S][band][1][xl] = uc[R - 1][qL ^ 1];
    };
    const int bandb = band > 0 ? band - 1 : band, banda = band < NB - 1 ? band + 1 : band;

    // ---- stage S: one colour (red for even S, else black) of the RB-SOR update (eqs. rbsor1-2) on
    // plane p of parity PAR held in uc, its z-neighbour planes in um (p-1) and up (p+1); f from
    // the registers (FS < 0) or LDS slot FS.  INNER: the rows whose y neighbours are this
    // lane's, else the band's first and last row
    auto colour = [&](auto cS, auto cPAR, auto cFS, auto cIN, T (&um)[R][2], T (&uc)[R][2], T (&up)[R][2],
                      int p) __attribute__((always_inline)) {
      constexpr int S = decltype(cS)::value, C = S & 1, PAR = decltype(cPAR)::value, FS = decltype(cFS)::value;
      constexpr bool INNER = decltype(cIN)::value;
      T below = (T)0, above = (T)0;
      if constexpr (INNER) {
        refresh(std::integral_constant<int, C>{}, cPAR, uc);
      } else {
        below = xe[S][bandb][1][xl];
        above = xe[S][banda][0][xl];
      }
      [[maybe_unused]] const PlaneW pw = plane_w(p);
      static_for<R>([&](auto rr) __attribute__((always_inline)) {
        constexpr int r = decltype(rr)::value;
        if constexpr (INNER == (r > 0 && r < R - 1)) {
          constexpr int q = (r + PAR + C) & 1;      // the cell of this colour in row r
          const T c = uc[r][q];
          T xm, xp, ym, yp;
          if constexpr (q == 0) {
            xm = from_left(uc[r][1]);
            xp = uc[r][1];
            if constexpr (XYW) xm = wx0 ? kx0 * c : xm;
          } else {
            xm = uc[r][0];
            xp = from_right(uc[r][0]);
            if constexpr (XYW) xp = wx1 ? kx1 * c : xp;
          }
          if constexpr (r > 0) ym = uc[r - 1][q]; else ym = below;
          if constexpr (r < R - 1) yp = uc[r + 1][q]; else yp = above;
          const T zm = um[r][q], zp = up[r][q];
          T fv;
          if constexpr (FS < 0) fv = fr[r][q];
          else fv = q ? fl[FS][r][tid].b : fl[FS][r][tid].a;
          const T nbs = ((((xm + xp) + ym) + yp) + zm) + zp;
          // (one form of the update for every level, so that its rounding does not depend on the walls)
          if constexpr (PER) uc[r][q] = c + omega * ((nbs - h2 * fv) * inv6 - c);
          else uc[r][q] = c + pw.om * (((nbs + pw.kz * c) - h2 * fv) * inv6 - c);
        }
      });
    };

    // ---- defect stage on plane p (parity PAR, final after black sweep 2, in uc; p-1 in um,
    // p+1 in up, final in its red cells): completes the red cells of p-1 with the black cells
    // of p above them, takes the black cells of p whole and the red cells of p without their
    // upper neighbour; then the restriction (down) or the sum of squares (norm)
    auto defect = [&](auto cPAR, auto cFS, T (&um)[R][2], T (&uc)[R][2], T (&up)[R][2], int p)
                      __attribute__((always_inline)) {
      constexpr int PAR = decltype(cPAR)::value, FS = decltype(cFS)::value;
      refresh(std::integral_constant<int, 2>{}, cPAR, uc);
      const T c6 = PER ? (T)6 : (T)6 - plane_w(p).kz;
      // the red cells' y neighbours beyond the band: black, set in this step
      xd[band][0][xl] = uc[0][PAR ? 0 : 1];
      xd[band][1][xl] = uc[R - 1][(R - 1 + PAR + 1) & 1];
      // plane p-1: its red cells' upper neighbour is final now
      const bool out_prev = p - 1 >= z0 && p - 1 < zend;
      const bool out_cur = p >= z0 && p < zend;
      T dprev[R], dblk[R];
      static_for<R>([&](auto rr) __attribute__((always_inline)) {
        constexpr int r = decltype(rr)::value;
        constexpr int qr_prev = (r + PAR + 1) & 1;   // red cell of row r on plane p-1 (parity PAR^1)
        dprev[r] = dred_get(r) - ih2 * uc[r][qr_prev];
      });
      // the cell of row r that is red (RED, without its upper neighbour: added at the next step) or
      // black; ynb: its y neighbour beyond the band
      auto cell = [&](auto rr, auto cRED, T ynb) __attribute__((always_inline)) {
        constexpr int r = decltype(rr)::value;
        constexpr bool red = decltype(cRED)::value;
        constexpr int q = (r + PAR + (red ? 0 : 1)) & 1;
        const T c = uc[r][q];
        const T fv = q ? fl[FS][r][tid].b : fl[FS][r][tid].a;
        T xm, xp, ym, yp;
        if constexpr (q == 0) {
          xm = from_left(uc[r][1]);
          xp = uc[r][1];
          if constexpr (XYW) xm = wx0 ? kx0 * c : xm;
        } else {
          xm = uc[r][0];
          xp = from_right(uc[r][0]);
          if constexpr (XYW) xp = wx1 ? kx1 * c : xp;
        }
        if constexpr (r > 0) ym = uc[r - 1][q]; else ym = ynb;
        if constexpr (r < R - 1) yp = uc[r + 1][q]; else yp = ynb;
        const T s5 = (((xm + xp) + ym) + yp) + um[r][q];
        if constexpr (red) dred_set(r, fv - (s5 - c6 * c) * ih2);
        else dblk[r] = fv - ((s5 + up[r][q]) - c6 * c) * ih2;
      };
      using Red = std::true_type;
      using Black = std::false_type;
      using I0 = std::integral_constant<int, 0>;
      using IL = std::integral_constant<int, R - 1>;
      static_for<R - 2>([&](auto rr) __attribute__((always_inline)) {
        using Ir = std::integral_constant<int, decltype(rr)::value + 1>;
        cell(Ir{}, Black{}, (T)0);
        cell(Ir{}, Red{}, (T)0);
      });
      // (the black cells' y neighbours beyond the band are those of the last black stage)
      cell(I0{}, Black{}, xe[kStages - 1][bandb][1][xl]);
      cell(IL{}, Black{}, xe[kStages - 1][banda][0][xl]);
      __syncthreads();
      cell(I0{}, Red{}, xd[bandb][1][xl]);
      cell(IL{}, Red{}, xd[banda][0][xl]);
      if constexpr (NORM) {
        auto square = [](T v) { return (double)v * (double)v; };
#pragma unroll
        for (int j = 0; j < R / 2; ++j) {
          if (out[j]) {
            if (out_cur) acc += square(dblk[2 * j]) + square(dblk[2 * j + 1]);
            if (out_prev) acc += square(dprev[2 * j]) + square(dprev[2 * j + 1]);
          }
        }
      }
      if constexpr (DEF) {
        // plane p-1 is complete: its row-pair sums (black part from the previous step); the
        // even plane of a coarse plane waits in stash, the odd one makes the coarse cell there
        constexpr int par_prev = PAR ^ 1;
#pragma unroll
        for (int j = 0; j < R / 2; ++j) {
          const T sprev = pend[j] + (dprev[2 * j] + dprev[2 * j + 1]);
          // FAS: the final u of plane p-1 (um) over the same four cells
          T suprev = (T)0;
          if constexpr (FAS) suprev = (um[2 * j][0] + um[2 * j][1]) + (um[2 * j + 1][0] + um[2 * j + 1][1]);
          if constexpr (par_prev == 0) {
            stash[j] = sprev;
            if constexpr (FAS) stash_u[j] = suprev;
          } else {
            stash[j] = (stash[j] + sprev) * (T)0.125;
            if constexpr (FAS) stash_u[j] = (stash_u[j] + suprev) * (T)0.125;
          }
          pend[j] = dblk[2 * j] + dblk[2 * j + 1];
        }
      }
    };

    // ---- face values into f of plane Q, just taken up (fr): a wave beside a wall loads them and waits
    auto take_values = [&](int Q) __attribute__((always_inline)) {
      if constexpr (VALUES) {
        const double w = -2.0 * A.ih2;
        // one face's values for a cell of each of the four rows, or for the two cells of a row: at `at`
        // and onwards by step; the indices are made here each time (as loop invariants they would
        // hold registers through the march)
        auto fold = [&](T& fv, const double* at) __attribute__((always_inline)) { fv = (T)((double)fv + w * *at); };
        auto row_of = [&](int r) __attribute__((always_inline)) {
          int y = ygv[r];
          asm volatile("" : "+v"(y));
          return y;
        };
        int x = xag;
        asm volatile("" : "+v"(x));
        if constexpr (XYW) {
          const size_t line = (size_t)((pz ? Q & nm : min(max(Q, 0), nm)) + 1) * (size_t)(n + 2) + 1;
          auto x_face = [&](int face, int e) __attribute__((always_inline)) {
            const double* b = A.bc.b[face] + line;
#pragma unroll
            for (int r = 0; r < R; r += 2) {
              const double* at = b + row_of(r);   // (a row pair neither wraps nor straddles a wall)
              fold(fr[r][e], at);
              fold(fr[r + 1][e], at + 1);
            }
          };
          auto y_face = [&](int face, int r) __attribute__((always_inline)) {
            const double* at = A.bc.b[face] + line + x;
            fold(fr[r][0], at);
            fold(fr[r][1], at + 1);
          };
          if (wx0 && A.bc.b[0]) x_face(0, 0);
          if (wx1 && A.bc.b[1]) x_face(1, 1);
          if (gy0 && A.bc.b[2]) y_face(2, 2);
          if (gy1 && A.bc.b[3]) y_face(3, 1);
        }
        auto z_face = [&](int face) __attribute__((always_inline)) {
#pragma unroll
          for (int r = 0; r < R; ++r) {
            const double* at = A.bc.b[face] + (size_t)(row_of(r) + 1) * (size_t)(n + 2) + 1 + x;
            fold(fr[r][0], at);
            fold(fr[r][1], at + 1);
          }
        };
        if (!pz && Q == 0 && A.bc.b[4]) z_face(4);
        if (!pz && Q == nm && A.bc.b[5]) z_face(5);
      }
    };

    load_plane(zstart);
    load_taps(zstart, std::integral_constant<int, 0>{});
    prolong_apply(zstart, std::integral_constant<int, HZ & 1>{});
    keep_in(zstart);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      u[0][r][0] = pu[r][0]; u[0][r][1] = pu[r][1];
      fr[r][0] = pf[r][0]; fr[r][1] = pf[r][1];
    }
    arrived(u[0], fr);
    take_values(zstart - 1);
    // one pipeline step: the plane in ring slot K is P = zstart + t, t = g + K with g a multiple of
    // kRing, so P - j sits in slot (K - j) mod kRing, has parity (HZ + K + j) mod 2 (z0 and kRing are
    // even), and its f is in LDS slot (K - HZ - j) mod kFSlots (which divides kRing)
    auto step = [&](int g, auto kk) __attribute__((always_inline)) {
      constexpr int K = decltype(kk)::value;
      const int t = g + K;
      if (t >= nsteps) return;
      const int P = zstart + t;
      // prefetch; consumed at the end of the step (after the last plane: that plane again, unused --
      // a branch here and at the take-up would make the waits at its join cover the stores)
      const int Pn = t + 1 < nsteps ? P + 1 : P - 1;
      load_plane(Pn);
      load_taps(Pn, std::integral_constant<int, ((HZ + K + 1) & 1) ? 1 : 2>{});
      // ring slot and parity of plane P - j, LDS slot of its f
      auto slot = [](int j) constexpr { return (K - j + 2 * kRing) % kRing; };
      auto fslot = [](int j) constexpr { return (K - HZ - j + 12 * kFSlots) % kFSlots; };
      auto up_u = [&](auto jj) __attribute__((always_inline)) -> T (&)[R][2] { return u[slot(decltype(jj)::value)]; };
      using ParL = std::integral_constant<int, (HZ + K + kStages) & 1>;
      using FsL = std::integral_constant<int, fslot(kStages)>;
      static_for<kStages>([&](auto ss) __attribute__((always_inline)) {
        constexpr int S = decltype(ss)::value;
        edges_out(ss, std::integral_constant<int, (HZ + K + S + 1) & 1>{}, up_u(std::integral_constant<int, S + 1>{}));
      });
      auto stages = [&](auto cIN) __attribute__((always_inline)) {
        // red, black (, red, black): stage S on plane P - 1 - S
        static_for<kStages>([&](auto ss) __attribute__((always_inline)) {
          constexpr int S = decltype(ss)::value;
          colour(ss, std::integral_constant<int, (HZ + K + S + 1) & 1>{},
                 std::integral_constant<int, S == 0 ? -1 : fslot(S + 1)>{}, cIN,
                 up_u(std::integral_constant<int, S + 2>{}), up_u(std::integral_constant<int, S + 1>{}),
                 up_u(std::integral_constant<int, S>{}), P - 1 - S);
        });
      };
      stages(std::true_type{});
      __syncthreads();
      stages(std::false_type{});
      if constexpr (DSTAGE)
        defect(ParL{}, FsL{}, u[slot(kStages + 1)], u[slot(kStages)], u[slot(kStages - 1)], P - kStages);
      else __syncthreads();   // (with a defect stage: its barrier) xe is free for the next step
      // the last stage's plane is final, and on odd planes the one before's coarse cells: out
      constexpr int sl = slot(kStages);
      auto put = [&]() __attribute__((always_inline)) {
        {
          const int p = P - kStages;
          if (p >= z0 && p < zend) {
            const int pg = p & nm;
#pragma unroll
            for (int r = 0; r < R; ++r)
              if (out[r >> 1]) {
                typedef T ntv2 __attribute__((ext_vector_type(2)));
                const ntv2 v = {u[sl][r][0], u[sl][r][1]};
                __builtin_nontemporal_store(v, reinterpret_cast<ntv2*>(const_cast<T*>(at(uout, r, pg))));
              }
          }
        }
        if constexpr (DEF && ((HZ + K + kStages + 1) & 1) != 0) {
          const int p = P - kStages - 1;
          if (p >= z0 && p < zend) {
            T* __restrict__ fcp = reinterpret_cast<T*>(A.fc);
            T* __restrict__ ucp = reinterpret_cast<T*>(A.uc0);
#pragma unroll
            for (int j = 0; j < R / 2; ++j)
              if (out[j]) {
                const size_t ci = cdx(xag >> 1, ygv[2 * j] >> 1, p >> 1);
                fcp[ci] = stash[j];
                if constexpr (FAS) reinterpret_cast<T*>(A.pbar)[ci] = stash_u[j];
                if (FAS || ucp) ucp[ci] = FAS ? stash_u[j] : (T)0;
              }
          }
        }
      };
      if constexpr (EARLY) put();
      prolong_apply(Pn, std::integral_constant<int, (HZ + K + 1) & 1>{});
      keep_in(Pn);
      // u(P+1) enters the ring in the slot of the oldest plane; f(P-1) moves to the LDS slot of the
      // last stage's plane (done with), f(P) into the registers
      constexpr int so = slot(kStages + 1);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        u[so][r][0] = pu[r][0]; u[so][r][1] = pu[r][1];
        fl[FsL::value][r][tid] = Pair<T>{fr[r][0], fr[r][1]};
        fr[r][0] = pf[r][0]; fr[r][1] = pf[r][1];
      }
      arrived(u[so], fr);
      if constexpr (!EARLY) put();
      take_values(P);   // (last: before the stores the FP64 up pass spills 100-160 bytes, 1.4 times its time)
    };
    for (int g = 0; g < nsteps; g += kRing) {
      static_for<kRing>([&](auto kk) __attribute__((always_inline)) { step(g, kk); });
    }
  }
  if constexpr (NORM) {
    // the exchange buffer is free once every wave has left the march
    double* red = reinterpret_cast<double*>(&xe[0][0][0][0]);
    acc = wave_sum(acc);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
      for (int q = 0; q < W; ++q) s += red[q];
    __syncthreads();
    finish_sum<kLanes * W>(A.sink, s, red);
  }
}

template <typename T, int W, bool UP, bool NORM, int WALLS, bool BLK, int NS, int EARLY>
__global__ void __launch_bounds__(kLanes* W) k_march(MarchArgs A) {
  march_body<T, W, UP, NORM, WALLS, BLK, false, false, false, EARLY != 0>(A);
}

// A leg with face values, f being the caller's (the operator entry points).
template <typename T, int W, bool UP, int WALLS, int NS>
__global__ void __launch_bounds__(kLanes* W) k_march_values(MarchArgs A) {
  march_body<T, W, UP, false, WALLS, false, false, false, true, false>(A);
}

// The down pass of a Full Approximation Scheme cycle (dense FP64 levels).
template <typename T, int W, int WALLS, int NS>
__global__ void __launch_bounds__(kLanes* W) k_march_fas(MarchArgs A) {
  march_body<T, W, false, false, WALLS, false, true, false, false, false>(A);
}

// The down pass from u = 0, which is not read (the first leg of a mixed-precision correction).
template <typename T, int W, int WALLS, int NS>
__global__ void __launch_bounds__(kLanes* W) k_march_zero(MarchArgs A) {
  march_body<T, W, false, false, WALLS, false, false, true, false, false>(A);
}

constexpr int kCUs = 256;

// Dynamic LDS, unused, that keeps a second FP32 workgroup off a CU (of up to 80 KiB, two fit) on the
// levels with early stores: neighbouring tiles then march the same planes at the same time more often and meet in
// L2.  Operator calls as above, FP32 two sweeps, with two on a CU and one: 512^3 761 / 698 and
// 714 / 698 us, 1024^3 7383 / 6627 and 6073 / 5898, 256^3 79 / 73 and 78 / 73.  (With late stores 512^3
// 754 / 711 and 790 / 711, so not where those are.)
template <typename T>
unsigned lds_beside(int n) {
  return sizeof(T) == 4 && march_early(n) ? (kNS == 1 ? 61440u : 20480u) : 0u;
}

// Planes per workgroup: even (chunks then start on planes of the parity compiled in).  With one workgroup
// per CU resident (FP64 by its LDS) the grid runs in rounds of kCUs workgroups; the chunk minimises
// rounds x (planes marched, 2 hz halo planes included).
int march_zchunk(int n, int tiles_xy, int hz) {
  int best = n;
  long best_cost = -1;
  for (int zc = 6; zc <= n; zc += 2) {
    const long chunks = (n + zc - 1) / zc;
    if ((long)tiles_xy * chunks > (long)kMaxPartials * 32 - 8) continue;   // partials buffer
    const long rounds = ((long)tiles_xy * chunks + kCUs - 1) / kCUs;
    const long cost = rounds * (zc + 2 * hz);
    if (best_cost < 0 || cost < best_cost) best_cost = cost, best = zc;
  }
  return best;
}

// Interior and wall tiles of a level with x or y walls: the chunk lengths of the two sets
// (both launches resident together, in one round of kCUs workgroups) that balance the interior
// march against the wall march, whose steps cost kWallCost times as much.
constexpr double kWallCost = 1.3;

bool march_split_plan(int n, int nint, int nring, int hz, int& zi, int& zr) {
  double best = -1.0;
  const long cap = (long)kMaxPartials * 32 - 8;
  for (int ci = 1; ci <= (n + 5) / 6; ++ci) {
    const int zci = ((n + ci - 1) / ci + 1) / 2 * 2;
    const long ni = (long)nint * ((n + zci - 1) / zci);
    for (int cr = 1; cr <= (n + 5) / 6; ++cr) {
      const int zcr = ((n + cr - 1) / cr + 1) / 2 * 2;
      const long nr = (long)nring * ((n + zcr - 1) / zcr);
      const long tot = ((ni + 7) / 8 + (nr + 7) / 8) * 8;
      if (tot > kCUs || tot > cap) continue;
      const double t = std::max((double)(zci + 2 * hz), kWallCost * (zcr + 2 * hz));
      if (best < 0 || t < best) best = t, zi = zci, zr = zcr;
    }
  }
  return best > 0;
}

template <typename T, bool UP, bool NORM, bool BLK>
void launch_march(MarchArgs A, hipStream_t s, const MarchAux* aux) {
  bool per = true;
  for (int f = 0; f < 6; ++f) per = per && A.bc.kind[f] == BC_PERIODIC;
  bool xyper = true;
  for (int f = 0; f < 4; ++f) xyper = xyper && A.bc.kind[f] == BC_PERIODIC;
  constexpr int W = kWaves;
  constexpr int HZ = kStages + (!UP || NORM ? 1 : 0);
  A.L = ilog2(A.n);
  A.xo = kTX - 2 * kHalo;
  A.yo = kR * 2 * W - 2 * kHalo;
  A.tiles_x = (A.n + A.xo - 1) / A.xo;
  A.tiles_y = (A.n + A.yo - 1) / A.yo;
  A.set = 0;
  int zi = 0, zr = 0;
  const int nint = (A.tiles_x - 2) * (A.tiles_y - 2), nring = 2 * A.tiles_x + 2 * (A.tiles_y - 2);
  if (sizeof(T) == 8 && !per && !xyper && aux && aux->s2 && A.tiles_x >= 3 && A.tiles_y >= 3 && nint > nring &&
      march_split_plan(A.n, nint, nring, HZ, zi, zr)) {
    // FP64 with x or y walls: the interior tiles (their halos reach no x or y wall) march in
    // the z-walls-only form on this stream, the ring of wall tiles in the full form on the
    // second stream, concurrently (fork and join through events); the ring's partials follow
    // the interior's.  Where the interior tiles are the more: at 512^3 (64 against 36) a V-cycle
    // takes 1931 us so and 1947 in one launch, at 1024^3 14.93 and 14.91 ms, at 256^3 (9 against 16) 415
    // and 413 us.  (FP32's full
    // form, well within its registers, is slower split: 0.52 -> 0.57 ms at 512^3.)
    MarchArgs Ai = A, Ar = A;
    Ai.set = 1;
    Ai.zc = zi;
    Ai.ntiles = nint * ((A.n + zi - 1) / zi);
    const int gi = (Ai.ntiles + 7) / 8 * 8;
    Ar.set = 2;
    Ar.zc = zr;
    Ar.ntiles = nring * ((A.n + zr - 1) / zr);
    const int gr = (Ar.ntiles + 7) / 8 * 8;
    Ai.sink.total = Ar.sink.total = gi + gr;
    Ar.sink.first = gi;
    LaunchTiming& lt = launch_timing();
    const bool timed = lt.armed;
    lt.armed = false;
    if (timed) (void)hipEventRecord(lt.e0, s);
    (void)hipEventRecord(aux->fork, s);
    (void)hipStreamWaitEvent(aux->s2, aux->fork, 0);
    auto both = [&](auto early) {
      constexpr int E = decltype(early)::value;
      hipLaunchKernelGGL((k_march<T, W, UP, NORM, 2, BLK, kNS, E>), dim3(gr), dim3(kLanes * W), 0, aux->s2, Ar);
      hipLaunchKernelGGL((k_march<T, W, UP, NORM, 1, BLK, kNS, E>), dim3(gi), dim3(kLanes * W), 0, s, Ai);
    };
    if (!BLK && march_early(A.n)) both(std::integral_constant<int, BLK ? 0 : 1>{});
    else both(std::integral_constant<int, 0>{});
    (void)hipEventRecord(aux->join, aux->s2);
    (void)hipStreamWaitEvent(s, aux->join, 0);
    if (timed) (void)hipEventRecord(lt.e1, s);
    return;
  }
  A.zc = march_zchunk(A.n, A.tiles_x * A.tiles_y, HZ);
  const int chunks = (A.n + A.zc - 1) / A.zc;
  A.ntiles = A.tiles_x * A.tiles_y * chunks;
  const int grid = (A.ntiles + 7) / 8 * 8;
  A.sink.total = grid;
  auto go = [&](auto early) {
    constexpr int E = decltype(early)::value;
    auto run = [&](auto k) { launch_maybe_timed(k, dim3(grid), dim3(kLanes * W), E ? lds_beside<T>(A.n) : 0u, s, A); };
    if (per) run(k_march<T, W, UP, NORM, 0, BLK, kNS, E>);
    else if (xyper) run(k_march<T, W, UP, NORM, 1, BLK, kNS, E>);
    else run(k_march<T, W, UP, NORM, 2, BLK, kNS, E>);
  };
  if (!BLK && march_early(A.n)) go(std::integral_constant<int, BLK ? 0 : 1>{});
  else go(std::integral_constant<int, 0>{});
}

// The down passes of FAS and from zero, and the legs with face values: one launch over every tile,
// the wall form chosen by the level's faces.
enum class OneLaunch { kFas, kZero, kValuesDown, kValuesUp };
template <typename T, OneLaunch FORM>
void launch_march_one(MarchArgs A, hipStream_t s) {
  bool per = true, xyper = true;
  for (int f = 0; f < 6; ++f) per = per && A.bc.kind[f] == BC_PERIODIC;
  for (int f = 0; f < 4; ++f) xyper = xyper && A.bc.kind[f] == BC_PERIODIC;
  constexpr int W = kWaves;
  A.L = ilog2(A.n);
  A.xo = kTX - 2 * kHalo;
  A.yo = kR * 2 * W - 2 * kHalo;
  A.tiles_x = (A.n + A.xo - 1) / A.xo;
  A.tiles_y = (A.n + A.yo - 1) / A.yo;
  A.set = 0;
  A.zc = march_zchunk(A.n, A.tiles_x * A.tiles_y, kStages + (FORM == OneLaunch::kValuesUp ? 0 : 1));
  A.ntiles = A.tiles_x * A.tiles_y * ((A.n + A.zc - 1) / A.zc);
  const int grid = (A.ntiles + 7) / 8 * 8;
  if constexpr (FORM == OneLaunch::kValuesDown || FORM == OneLaunch::kValuesUp) {
    // (values only count on faces that fix one, so some face is a wall)
    constexpr bool UP = FORM == OneLaunch::kValuesUp;
    if (xyper) launch_maybe_timed(k_march_values<T, W, UP, 1, kNS>, dim3(grid), dim3(kLanes * W), 0, s, A);
    else launch_maybe_timed(k_march_values<T, W, UP, 2, kNS>, dim3(grid), dim3(kLanes * W), 0, s, A);
  } else if constexpr (FORM == OneLaunch::kZero) {
    if (per) launch_maybe_timed(k_march_zero<T, W, 0, kNS>, dim3(grid), dim3(kLanes * W), 0, s, A);
    else if (xyper) launch_maybe_timed(k_march_zero<T, W, 1, kNS>, dim3(grid), dim3(kLanes * W), 0, s, A);
    else launch_maybe_timed(k_march_zero<T, W, 2, kNS>, dim3(grid), dim3(kLanes * W), 0, s, A);
  } else {
    if (per) launch_maybe_timed(k_march_fas<T, W, 0, kNS>, dim3(grid), dim3(kLanes * W), 0, s, A);
    else if (xyper) launch_maybe_timed(k_march_fas<T, W, 1, kNS>, dim3(grid), dim3(kLanes * W), 0, s, A);
    else launch_maybe_timed(k_march_fas<T, W, 2, kNS>, dim3(grid), dim3(kLanes * W), 0, s, A);
  }
}

template <typename T>
MarchArgs base_args(const T* uin, T* uout, const T* f, int n, double h, double omega, const LevelBC& bc) {
  MarchArgs A{};
  A.uin = uin;
  A.uout = uout;
  A.f = f;
  A.bc = bc;
  A.n = n;
  A.h2 = h * h;
  A.ih2 = 1.0 / (h * h);
  A.omega = omega;
  return A;
}

// Does bc hold face values?  (Arrays of faces that fix none are dropped.)
bool take_face_values(LevelBC& bc) {
  bool any = false;
  for (int f = 0; f < 6; ++f) {
    if (!bc_has_value(bc.kind[f])) bc.b[f] = nullptr;
    any = any || bc.b[f];
  }
  return any;
}

}  // namespace

template <typename T, int NS>
void march_down_ns(const T* uin, T* uout, const T* f, T* fc, T* uc0, int n, double h, double omega, const LevelBC& bc,
                hipStream_t s, int Lm, const MarchAux* aux) {
  MarchArgs A = base_args(uin, uout, f, n, h, omega, bc);
  A.fc = fc;
  A.uc0 = uc0;
  A.Lm = Lm;
  if (Lm > 0) launch_march<T, false, false, true>(A, s, aux);
  else if (!uin) launch_march_one<T, OneLaunch::kZero>(A, s);
  else if (take_face_values(A.bc)) launch_march_one<T, OneLaunch::kValuesDown>(A, s);
  else launch_march<T, false, false, false>(A, s, aux);
}

template <typename T, int NS>
void march_down_fas_ns(const T* uin, T* uout, const T* f, T* fc, T* pbar, T* uc0, int n, double h, double omega,
                    const LevelBC& bc, hipStream_t s) {
  MarchArgs A = base_args(uin, uout, f, n, h, omega, bc);
  A.fc = fc;
  A.pbar = pbar;
  A.uc0 = uc0;
  launch_march_one<T, OneLaunch::kFas>(A, s);
}

template <typename T, int NS>
void march_up_ns(const T* uin, T* uout, const T* f, const T* ec, const LevelBC& bcc, const SumSink* sink, int n, double h,
              double omega, const LevelBC& bc, hipStream_t s, int Lm, const MarchAux* aux) {
  MarchArgs A = base_args(uin, uout, f, n, h, omega, bc);
  A.ec = ec;
  A.bcc = bcc;
  if (sink) A.sink = *sink;
  A.Lm = Lm;
  if (Lm > 0) {
    if (sink) launch_march<T, true, true, true>(A, s, aux);
    else launch_march<T, true, false, true>(A, s, aux);
  } else if (!sink && take_face_values(A.bc)) {
    launch_march_one<T, OneLaunch::kValuesUp>(A, s);
  } else {
    if (sink) launch_march<T, true, true, false>(A, s, aux);
    else launch_march<T, true, false, false>(A, s, aux);
  }
}

template void march_down_ns<MG_MARCH_T, kNS>(const MG_MARCH_T*, MG_MARCH_T*, const MG_MARCH_T*, MG_MARCH_T*, MG_MARCH_T*,
                                             int, double, double, const LevelBC&, hipStream_t, int, const MarchAux*);
template void march_up_ns<MG_MARCH_T, kNS>(const MG_MARCH_T*, MG_MARCH_T*, const MG_MARCH_T*, const MG_MARCH_T*,
                                           const LevelBC&, const SumSink*, int, double, double, const LevelBC&,
                                           hipStream_t, int, const MarchAux*);
#ifdef MG_MARCH_FAS
template void march_down_fas_ns<MG_MARCH_T, kNS>(const MG_MARCH_T*, MG_MARCH_T*, const MG_MARCH_T*, MG_MARCH_T*,
                                                 MG_MARCH_T*, MG_MARCH_T*, int, double, double, const LevelBC&,
                                                 hipStream_t);
#endif

}  // namespace mg
