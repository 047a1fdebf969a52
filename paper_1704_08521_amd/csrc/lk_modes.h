// Tensor-product factors of 1D operators (host computation and device placement), shared by
// the pressure-correction solve and the viscous step of the Stokes-preconditioned vectors.
#pragma once

#include <cstddef>
#include <vector>

#include "lk_ctx.h"

namespace lk {

// Host results for one 1D operator K s = lam M s on n points.
struct ModeHost {
  int n = 0;
  std::vector<double> lam, S, Wf, m;  // full modes (S^T M S = I, Wf = S^T M) and the mass
  bool sym = false;                   // mirror-symmetric: the half problems below are set
  std::vector<double> lam_e, Sh_e, lam_o, Sh_o;
};

// Full modes, and the even / odd half modes when `sym` (the operator must then be
// mirror-symmetric).  False if an eigensolve fails.
bool compute_modes(int n, const std::vector<double>& kd, const std::vector<double>& ko, const std::vector<double>& m,
                   bool sym, ModeHost& H);

// Device bytes that place_modes needs for any operator of n points (alignment included).
size_t mode_bytes(int n, bool f32);

// Writes arrays into a host staging buffer whose image is later copied to the device
// allocation `dev` in one transfer; device pointers are handed out as the arrays are
// placed.  Every array starts 16-byte aligned.
struct Stager {
  std::vector<char> host;
  char* dev = nullptr;
  size_t used = 0;
  bool overflow = false;
  Stager(size_t bytes, void* device) : host(bytes), dev((char*)device) {}
  void* put(const void* src, size_t bytes);
  double* put_d(const std::vector<double>& v);
  float* put_f(const std::vector<double>& v);  // rounded to float32
};

// Places the factors of one operator that its transforms (lk_lines.h) use, in float64 and with f32 in float32 too.
// Half length up to kMfMaxHalf: the matrix-core packs, of the parity-sorted half-size matrices of a
// mirror-symmetric operator, else (float64) of the full ones F = S^T M and Bk = S.  Longer ones, and the float32
// factors of an operator without the symmetry: the matrices themselves and their transposes.
void place_modes(const ModeHost& H, AxisModes& M, Stager& st, bool f32);

}  // namespace lk
