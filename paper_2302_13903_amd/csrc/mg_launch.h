// mg_launch.h -- host-side declarations of the kernel launchers (internal to the library).
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <cstddef>
#include <string>

#include "mg_common.h"

namespace mg {

constexpr int kMaxPartials = 2048;   // per-block partial sums of the two-stage reductions

// Timing of the next launch (one per host thread).  The solver arms it with two created events
// before a timed launcher that takes it; a single kernel then carries the events in its own
// dispatch (start and end timestamps of that kernel, with no marker packet queued between it
// and its neighbours), a launcher of several kernels records them around its launches.
struct LaunchTiming {
  hipEvent_t e0 = nullptr, e1 = nullptr;
  bool armed = false;
};
LaunchTiming& launch_timing();

// One kernel launch, timed through the armed hook when there is one.
template <typename K, typename... Args>
void launch_maybe_timed(K kern, dim3 grid, dim3 block, unsigned lds, hipStream_t s, Args... args) {
  LaunchTiming& t = launch_timing();
  if (t.armed) {
    t.armed = false;
    hipExtLaunchKernelGGL(kern, grid, block, lds, s, t.e0, t.e1, 0u, args...);
  } else {
    hipLaunchKernelGGL(kern, grid, block, lds, s, args...);
  }
}

inline int ilog2(long long n) {
  int l = 0;
  while ((1LL << l) < n) ++l;
  return l;
}

enum : int { TAIL_FMG = 1, TAIL_LOAD_U = 2 };

// Arguments of the coarse-tail kernel (mg_tail.hip): levels 0..top (top <= 4) of one hierarchy.
// V-cycle mode: one V-cycle on u at level top, from u in ug (TAIL_LOAD_U) or from zero.
// TAIL_FMG: full multigrid from the source of level top, whose restrictions the kernel makes.
struct TailArgs {
  int top;
  int mode;           // TAIL_FMG / TAIL_LOAD_U bits
  int npre, npost;
  double omega;
  double h;           // cell width of level top
  LevelBC bc_top;     // description of level top in V-cycle mode (face kinds as hom's)
  LevelBC hom;        // homogeneous description (coarse corrections; its kinds are every level's)
  LevelBC phys[5];    // physical description per level (FMG mode)
  const void* f;      // device source of level top
  void* ug;           // device solution / correction of level top (in and out)
  SumSink sink;       // where the sum of squared defects of the result goes (out null: not wanted)
  unsigned long long* clock;   // device, or null: receives the device clock at the start
};

template <typename T>
void launch_half_sweep(T* u, const T* f, int n, double h, double omega, int colour, const LevelBC& bc,
                       hipStream_t s);
template <typename T>
void launch_defect(const T* u, const T* f, T* d, int n, double h, const LevelBC& bc, hipStream_t s);
template <typename T>
void launch_defect_restrict(const T* u, const T* f, T* fc, T* uc0, int n, double h, const LevelBC& bc,
                            hipStream_t s);
template <typename Tin, typename Tout>
void launch_restrict(const Tin* uf, Tout* uc, int nc, hipStream_t s);
template <typename T>
void launch_prolong(const T* uc, T* uf, int nc, const LevelBC& bcc, int cubic, hipStream_t s);
// The FMG prolongation alone, for coarse levels of at least 16^3 (nc >= 16), either level in the
// MeshBlock layout with 2^Lmc- (2^Lmf-) cell blocks (0: dense).
template <typename T>
void launch_prolong_fmg(const T* uc, T* uf, int nc, int Lmc, int Lmf, const LevelBC& bcc, hipStream_t s);
template <typename T>
void launch_coarsest(T* u, const T* f, double h, const LevelBC& bc, hipStream_t s);
template <typename T>
void launch_tail(const TailArgs& a, hipStream_t s);
// FAS (Alg. 3): fc = restricted defect, pbar = uc = restricted u; f += L pbar on the coarse
// level; u -= pbar (the coarse-grid correction)
void launch_fas_restrict(const double* u, const double* f, double* fc, double* pbar, double* uc, int n, double h,
                         const LevelBC& bc, hipStream_t s);
void launch_fas_source(const double* pbar, double* f, int n, double h, const LevelBC& bc, hipStream_t s);
void launch_fas_correction(double* u, const double* pbar, size_t n3, hipStream_t s);

// f = a rho + c (and its FP32 copy when f32 != nullptr; and its restriction to the level below when
// fc != nullptr) on a level of 2^L cells per side (Lm > 0: MeshBlock layout); the sum of f^2 to the
// sink (not finite when rho is not).  c = -a * rho_sum[0] / n3 when rho_sum (device) is given (the
// gauge-free source), else 0.
template <typename T>
void launch_source(const double* rho, double* f, float* f32, T* fc, int L, int Lm, double a, const double* rho_sum,
                   SumSink sink, hipStream_t s);
void launch_sub_mean(double* u, size_t n3, const double* sum_dev, hipStream_t s);
void launch_f32_to_f64(const float* a, double* b, size_t n3, hipStream_t s);
void launch_add_f32(double* phi, const float* e, size_t n3, hipStream_t s);

int reduce_blocks(size_t n3);
// Sums to a sink (its total is the launcher's to set): of x; of sink.part[0..np) in index order
// (the second stage of a launch that left partials there).
void launch_sum(const double* x, size_t n3, SumSink sink, hipStream_t s);
void launch_sum_partials(int np, SumSink sink, hipStream_t s);
// Clears scal[0..count) (count <= 64) and stores the device clock's bits in scal[at].
void launch_begin(double* scal, int count, int at, hipStream_t s);
// Stores the device clock at *at (device).
void launch_clock(unsigned long long* at, hipStream_t s);
// Publishes *src (device) as a sink's launch would.
void launch_publish(const double* src, const SumSink& sink, hipStream_t s);
void launch_defect_norm(const double* u, const double* f, float* r32, int n, double h, const LevelBC& bc,
                        SumSink sink, hipStream_t s);

// zero `bytes` of device memory at p (8-byte aligned) with a kernel
void launch_zero(void* p, size_t bytes, hipStream_t s);

// out ((n+2)^3) = u with its ghost layer, edges and corners included, filled from bc
void launch_fill(const double* u, double* out, int n, const LevelBC& bc, hipStream_t s);

// Face values into the sources: on every listed level, the cells beside a face with values b take
// f - 2 b / h^2 summed over their faces, so that the level's operator is the homogeneous one
// (ghost = +-u) from then on.
struct FoldLevel {
  void* f;
  double ih2;
  int L, Lm;
  LevelBC bc;
};
template <typename T>
void launch_fold_faces(const FoldLevel* levels, int count, hipStream_t s);
// The extended arrays of the levels bottom..L (ext[l]: six of (2^l + 2)^2 one after another) of
// the faces with values (src[f]: n^2 finest values, or null); adds the count of each face's
// non-finite values to nonfinite[face] (null: not wanted).
void launch_faces(const double* const src[6], double* const* ext, int L, int bottom, double* nonfinite, hipStream_t s);

// multipole (mg_multipole.hip)
// moments[0..3] = (M, Mx, My, Mz) sums; origin[3]; q[25]
// rho of n^3 cells, dense (Lm = 0) or in the MeshBlock layout with 2^Lm-cell blocks
void launch_multipole_moments(const double* rho, int n, int Lm, double dx, int lmax, int use_origin,
                              const double* origin_host, double* part, double* scratch, hipStream_t s);
// out[q][f]: (nl + 2 ext)^2 values over transverse positions (t + 1/2) hl, t = -ext .. nl - 1 + ext
// of level q of `count` (null: not wanted), all in one launch
struct MpFaceLevels {
  int count;
  int nl[16];
  double hl[16];
  double* out[16][6];
};
void launch_multipole_faces(const double* scratch, int lmax, double G, double length, const MpFaceLevels& F,
                            hipStream_t s, int ext = 1);
// Moments over the cells of up to kMpMaxBoxes boxes (dense, x fastest), skipping each box's
// covered sub-box [hlo, hhi); cell (i, j, k) of a box sits at ((o + i + 1/2) h, ..).  part holds
// multipole_box_blocks() * nbox * 25 doubles; scratch as above.
constexpr int kMpMaxBoxes = 9;
struct MpBox {
  const double* rho;
  int n[3], o[3], hlo[3], hhi[3];
  double h;
};
int multipole_box_blocks();
// returns MG_ERR_INVALID_ARG (nothing launched) unless 1 <= nbox <= kMpMaxBoxes
int launch_multipole_moments_boxes(const MpBox* boxes, int nbox, int lmax, int use_origin, const double* origin_host,
                                   double centre, double* part, double* scratch, hipStream_t s);

// gravitational acceleration (mg_gravity.hip): g, rhog (3 n^3 each) and gface (3 n^2 (n+1),
// dense layout only) from phi, any of them null; returns the number of workgroups launched
int launch_gravity(const double* phi, const double* rho, double* g, double* rhog, double* gface, int n, int Lm,
                   double dx, const LevelBC& bc, hipStream_t s);
std::string gravity_kernel_name(int n, int Lm, bool g, bool rhog, bool gface);

}  // namespace mg
