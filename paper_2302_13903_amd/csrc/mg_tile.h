// mg_tile.h -- V-cycle legs of the small levels as one launch each (internal; see mg_tile.inl).
#pragma once

#include <hip/hip_runtime.h>

#include <string>

#include "mg_common.h"

namespace mg {

// Smallest and largest level side the region-tile legs take (the level must hold whole
// regions of 8 x 4 x 4 cells or more; above 128^3 the streaming passes move far fewer bytes).
constexpr int kTileMinN = 32;
constexpr int kTileMaxN = 128;

// The legs with NS (1 or 2) smoothing sweeps; instantiated in mg_tile_f64_1.hip and its siblings.
template <typename T, int NS>
void tile_down_ns(const T* uin, T* uout, const T* f, T* fc, T* pbar, T* uc0, int n, int Lm, double h, double omega,
                  const LevelBC& bc, hipStream_t s);
template <typename T, int NS>
void tile_up_ns(const T* uin, T* uout, const T* f, const T* ec, const LevelBC& bcc, const SumSink* sink, int n, int Lm,
                double h, double omega, const LevelBC& bc, hipStream_t s);

// May a leg of ns sweeps run as a region tile?
inline bool tile_sweeps_ok(int ns) { return ns == 1 || ns == 2; }

// Down step of a V-cycle level (Alg. 1 steps 1-3) in one launch: ns smoothing sweeps of u
// (uin -> uout, distinct arrays), the defect restricted into fc and the coarse correction uc0
// (if any) cleared.  Lm > 0: the level is in the MeshBlock layout with blocks of 2^Lm cells per side (the
// coarse level in the layout below, or the dense root grid when Lm = 1); Lm = 0: dense.
// pbar != nullptr: the down step of a Full Approximation Scheme cycle (Alg. 3 steps 2-4) --
// phibar (the mean of the 8 children of the swept u) is written to pbar and to uc0, the coarse
// level's starting iterate.  Face values: in f (launch_fold_faces), or in bc.
template <typename T>
void tile_down(const T* uin, T* uout, const T* f, T* fc, T* pbar, T* uc0, int n, int Lm, int ns, double h, double omega,
               const LevelBC& bc, hipStream_t s) {
  if (ns == 1) tile_down_ns<T, 1>(uin, uout, f, fc, pbar, uc0, n, Lm, h, omega, bc, s);
  else tile_down_ns<T, 2>(uin, uout, f, fc, pbar, uc0, n, Lm, h, omega, bc, s);
}

// Up step (Alg. 1 steps 5-7) in one launch: u += trilinear(ec) (ec's ghosts from the
// homogeneous description bcc), then ns sweeps (uin -> uout).  sink != nullptr: the sum of
// squared defects of the result goes there.
template <typename T>
void tile_up(const T* uin, T* uout, const T* f, const T* ec, const LevelBC& bcc, const SumSink* sink, int n, int Lm,
             int ns, double h, double omega, const LevelBC& bc, hipStream_t s) {
  if (ns == 1) tile_up_ns<T, 1>(uin, uout, f, ec, bcc, sink, n, Lm, h, omega, bc, s);
  else tile_up_ns<T, 2>(uin, uout, f, ec, bcc, sink, n, Lm, h, omega, bc, s);
}

// Name of the kernel of such a leg, as profilers list it.
template <typename T>
std::string tile_name(int ns, bool up, const LevelBC& bc, int n) {
  const bool walls = bc.kind[0] != BC_PERIODIC || bc.kind[2] != BC_PERIODIC || bc.kind[4] != BC_PERIODIC;
  return std::string("k_tile_leg<") + (sizeof(T) == 8 ? "double" : "float") + ", " + std::to_string(ns) +
         (up ? ", true" : ", false") + (walls ? ", true, " : ", false, ") + (n >= 64 ? "0, false>" : "1, false>");
}

}  // namespace mg
