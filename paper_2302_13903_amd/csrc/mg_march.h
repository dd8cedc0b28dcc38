// mg_march.h -- streaming passes of the large levels, a V-cycle leg each (internal; see mg_march.inl).
//
// Each pass reads u from `uin` and writes the result to `uout` (uin != uout): tiles overlap in
// their halos, so the update cannot be in place.
#pragma once

#include <hip/hip_runtime.h>

#include <string>

#include "mg_common.h"

namespace mg {

// Smallest level the passes run on (a z chunk must hold many planes).
constexpr int kMarchMinN = 128;

// Dense levels whose passes issue a step's stores before its loads are taken up, not after: from
// 256^3, where the tiles march faster than memory serves them.  Operator calls (with their copy of u),
// periodic, two sweeps, down / up, late and early: FP64 256^3 155 / 155 and 149 / 148 us, 512^3
// 1263 / 1215 and 1219 / 1185, 1024^3 11011 / 10483 and 10557 / 10020; FP32 256^3 78 / 75 and 76 / 73.
// At 128^3 the calls are equal (FP64 42 / 38 us, FP32 31 / 28).
inline bool march_early(int n) { return n >= 256; }

// A second stream and two events for splitting a pass of a level with x or y walls into the
// interior tiles and the wall tiles, run concurrently (owned by the caller; unused when null).
struct MarchAux {
  hipStream_t s2 = nullptr;
  hipEvent_t fork = nullptr, join = nullptr;
};

constexpr int kMarchWaves = 8;   // waves of a workgroup (mg_march.inl)

// The passes of NS (1 or 2) smoothing sweeps; instantiated in mg_march_f64_1.hip and its siblings.
template <typename T, int NS>
void march_down_ns(const T* uin, T* uout, const T* f, T* fc, T* uc0, int n, double h, double omega, const LevelBC& bc,
                   hipStream_t s, int Lm, const MarchAux* aux);
template <typename T, int NS>
void march_up_ns(const T* uin, T* uout, const T* f, const T* ec, const LevelBC& bcc, const SumSink* sink, int n, double h,
                 double omega, const LevelBC& bc, hipStream_t s, int Lm, const MarchAux* aux);
template <typename T, int NS>
void march_down_fas_ns(const T* uin, T* uout, const T* f, T* fc, T* pbar, T* uc0, int n, double h, double omega,
                       const LevelBC& bc, hipStream_t s);

// May a leg of ns sweeps run as a streaming pass?
inline bool march_sweeps_ok(int ns) { return ns == 1 || ns == 2; }

// Down step of a V-cycle level (Alg. 1 steps 1-3) in one pass: ns smoothing sweeps of u, the
// defect of the result restricted into fc, and the coarse correction uc0 (if any) cleared.
// uin == nullptr (Lm = 0 only): u is zero on input and is not read.
// Face values: in f (launch_fold_faces), or in bc with u read and Lm = 0.
// Lm > 0: the level is in the MeshBlock layout with blocks of 2^Lm cells per side (the coarse
// level below in the layout with blocks of 2^(Lm-1), or the dense root grid when Lm = 1).
template <typename T>
void march_down(const T* uin, T* uout, const T* f, T* fc, T* uc0, int n, int ns, double h, double omega, const LevelBC& bc,
                hipStream_t s, int Lm = 0, const MarchAux* aux = nullptr) {
  if (ns == 1) march_down_ns<T, 1>(uin, uout, f, fc, uc0, n, h, omega, bc, s, Lm, aux);
  else march_down_ns<T, 2>(uin, uout, f, fc, uc0, n, h, omega, bc, s, Lm, aux);
}

// Up step (Alg. 1 steps 5-7) in one pass: u += trilinear(ec) (ec's ghosts from bcc) as u is
// loaded, then ns smoothing sweeps.  sink != nullptr: the sum of squared defects of the result
// (the convergence norm, Sec. 2.3.7) goes there.  Face values: in f, or in bc without a sink and with
// Lm = 0.
template <typename T>
void march_up(const T* uin, T* uout, const T* f, const T* ec, const LevelBC& bcc, const SumSink* sink, int n, int ns,
              double h, double omega, const LevelBC& bc, hipStream_t s, int Lm = 0, const MarchAux* aux = nullptr) {
  if (ns == 1) march_up_ns<T, 1>(uin, uout, f, ec, bcc, sink, n, h, omega, bc, s, Lm, aux);
  else march_up_ns<T, 2>(uin, uout, f, ec, bcc, sink, n, h, omega, bc, s, Lm, aux);
}

// Down step of a Full Approximation Scheme cycle (Alg. 3 steps 1-4) in one pass: ns sweeps,
// the defect of the result restricted into fc, the result itself restricted into pbar (phibar)
// and the coarse level started from it (uc0 = phibar).
template <typename T>
void march_down_fas(const T* uin, T* uout, const T* f, T* fc, T* pbar, T* uc0, int n, int ns, double h, double omega,
                    const LevelBC& bc, hipStream_t s) {
  if (ns == 1) march_down_fas_ns<T, 1>(uin, uout, f, fc, pbar, uc0, n, h, omega, bc, s);
  else march_down_fas_ns<T, 2>(uin, uout, f, fc, pbar, uc0, n, h, omega, bc, s);
}

// Names of the kernels as profilers list them (the wall form follows bc's kinds; blk: MeshBlock
// layout); march_down1_name: the down passes of FAS, or from zero.
inline int march_walls(const LevelBC& bc) {
  bool per = true, xyper = true;
  for (int f = 0; f < 6; ++f) per = per && bc.kind[f] == BC_PERIODIC;
  for (int f = 0; f < 4; ++f) xyper = xyper && bc.kind[f] == BC_PERIODIC;
  return per ? 0 : xyper ? 1 : 2;
}
template <typename T>
std::string march_name(int ns, bool up, bool norm, const LevelBC& bc, int n, bool blk = false) {
  auto b = [](bool v) { return std::string(v ? "true, " : "false, "); };
  return std::string("k_march<") + (sizeof(T) == 8 ? "double, " : "float, ") + std::to_string(kMarchWaves) + ", " + b(up) +
         b(up && norm) + std::to_string(march_walls(bc)) + ", " + b(blk) + std::to_string(ns) +
         (!blk && march_early(n) ? ", 1>" : ", 0>");
}
template <typename T>
std::string march_down1_name(int ns, bool zero, const LevelBC& bc) {
  return std::string(zero ? "k_march_zero<" : "k_march_fas<") + (sizeof(T) == 8 ? "double, " : "float, ") +
         std::to_string(kMarchWaves) + ", " + std::to_string(march_walls(bc)) + ", " + std::to_string(ns) + ">";
}

}  // namespace mg
