// Transforms of every grid line along one axis with the axis's factors, in the variant that suits the axis: FP64 and
// FP32 matrix cores (mirror-symmetric, half length <= kMfMaxHalf; FP64 also without the
// symmetry, with the full matrix), folded vector-FMA kernels (longer mirror-symmetric axes) or the full
// mode matrix on the vector units.
#pragma once

#include <hip/hip_runtime.h>

#include "lk_ctx.h"
#include "lk_internal.h"

namespace lk {

// Division by lm[mode] + ly[j] + lx[i] between a forward and a backward left transform (column = j * nxs + i), the mode
// (zm, zj, zi) set to zero (zm negative: none).  The vector-FMA kernels divide in the forward
// transform, the matrix-core ones in the backward one; both calls of a pair get the same scale.
struct LineScale {
  const double *lm = nullptr, *ly = nullptr, *lx = nullptr;
  int nxs = 1, zm = 0, zj = 0, zi = 0;
};

// Columns of a left transform: column q starts at (q / nseg) * seg_stride + q % nseg, rows kstride apart, in a
// field of `elems` values.
struct Columns {
  int count, nseg;
  long seg_stride, kstride;
  size_t elems;
};

template <typename T>
const T* mode_full(const AxisModes& M, int which) {
  const double* d[4] = {M.F, M.Bk, M.FT, M.BkT};
  const float* f[4] = {M.F32, M.Bk32, M.FT32, M.BkT32};
  if constexpr (sizeof(T) == sizeof(double)) return d[which];
  else return f[which];
}
template <typename T>
const T* mode_half(const AxisModes& M, int which) {
  if constexpr (sizeof(T) == sizeof(double)) return M.h64[which];
  else return M.h32[which];
}
template <typename T>
const T* mode_pack(const AxisModes& M, int which) {
  if constexpr (sizeof(T) == sizeof(double)) return M.p64[which];
  else return M.p32[which];
}

// The field on the outer side (IN, OUT) may be FP64 with FP32 transforms (T) if the axis is on the matrix cores.
template <typename T, typename IN>
hipError_t left_forward(const AxisModes& M, int n, const Columns& q, const IN* in, T* out, const LineScale& s,
                        hipStream_t st) {
  if (M.mf) {
    if constexpr (sizeof(T) == sizeof(double))
      return launch_mxf_left(n, q.count, M.x64[0], in, out, q.elems, q.nseg, q.seg_stride, q.kstride, st);
    else
      return launch_m4f_left<IN>(n, q.count, M.x32[0], in, out, q.elems, q.nseg, q.seg_stride, q.kstride, st);
  }
  if constexpr (sizeof(T) != sizeof(IN)) return hipErrorInvalidValue;
  else {
    if constexpr (sizeof(T) == sizeof(double))
      if (M.full64)
        return launch_mx_full_left(n, q.count, M.x64[0], in, out, q.elems, q.nseg, q.seg_stride, q.kstride, nullptr,
                                   nullptr, nullptr, 1, 0, 0, 0, st);
    if (M.sym)
      return launch_tpf_left<T>(n, q.count, mode_half<T>(M, 0), mode_half<T>(M, 1), in, out, q.nseg, q.seg_stride,
                                q.kstride, s.lm, s.ly, s.lx, s.nxs, s.zm, s.zj, s.zi, st);
    return launch_tp_left<T>(n, q.count, n, mode_full<T>(M, 0), in, out, q.nseg, q.seg_stride, q.kstride, s.lm, s.ly,
                             s.lx, s.nxs, s.zm, s.zj, s.zi, st);
  }
}

template <typename T, typename OUT>
hipError_t left_backward(const AxisModes& M, int n, const Columns& q, const T* in, OUT* out, const LineScale& s,
                         hipStream_t st) {
  if (M.mf) {
    if constexpr (sizeof(T) == sizeof(double))
      return launch_mxu_left(n, q.count, M.x64[1], in, out, q.elems, q.nseg, q.seg_stride, q.kstride, s.lm,
                             s.ly, s.lx, s.nxs, s.zm, s.zj, s.zi, st);
    else
      return launch_m4u_left<OUT>(n, q.count, M.x32[1], in, out, q.elems, q.nseg, q.seg_stride, q.kstride, s.lm, s.ly,
                                  s.lx, s.nxs, s.zm, s.zj, s.zi, st);
  }
  if constexpr (sizeof(T) != sizeof(OUT)) return hipErrorInvalidValue;
  else {
    if constexpr (sizeof(T) == sizeof(double))
      if (M.full64)
        return launch_mx_full_left(n, q.count, M.x64[1], in, out, q.elems, q.nseg, q.seg_stride, q.kstride, s.lm, s.ly,
                                   s.lx, s.nxs, s.zm, s.zj, s.zi, st);
    if (M.sym)
      return launch_tpu_left<T>(n, q.count, mode_half<T>(M, 2), mode_half<T>(M, 3), in, out, q.nseg, q.seg_stride,
                                q.kstride, st);
    return launch_tp_left<T>(n, q.count, n, mode_full<T>(M, 1), in, out, q.nseg, q.seg_stride, q.kstride, nullptr,
                             nullptr, nullptr, 1, 0, 0, 0, st);
  }
}

// Along x the FP64 left kernels serve too, on mirror-symmetric axes by the rule of mx_along_x, else with the full
// matrix (100^3 15.6 us a transform against 27.5, 256^3 211 / 261).  FP32 keeps the kernels for lines
// (150^3 29 / 23).
template <typename T>
inline bool right_by_left(const AxisModes& M) {
  return sizeof(T) == sizeof(double) && (M.full64 || (M.mf && mx_along_x(M.he + M.ho)));
}
// The FP64 matrix-core backward transform takes a scale with ly or lx null (adding nothing) and zj or zi negative (any
// column); the other kernels do not.
inline bool scale_may_omit(const AxisModes& M) { return M.mf || M.full64; }

inline Columns lines_as_columns(int n, int lines) { return Columns{lines, 1, n, 1, (size_t)n * lines}; }

template <typename T>
hipError_t right_forward(const AxisModes& M, int n, int lines, const T* in, T* out, hipStream_t st) {
  if (right_by_left<T>(M)) return left_forward<T>(M, n, lines_as_columns(n, lines), in, out, LineScale{}, st);
  if (M.mf) return launch_mff_right<T>(n, lines, in, mode_pack<T>(M, 0), mode_pack<T>(M, 1), out, st);
  if (M.sym) return launch_tpf_right<T>(n, lines, in, mode_half<T>(M, 4), mode_half<T>(M, 5), out, st);
  return launch_tp_right<T>(lines, n, n, in, mode_full<T>(M, 2), out, st);
}

template <typename T>
hipError_t right_backward(const AxisModes& M, int n, int lines, const T* in, T* out, hipStream_t st) {
  if (right_by_left<T>(M)) return left_backward<T>(M, n, lines_as_columns(n, lines), in, out, LineScale{}, st);
  if (M.mf) return launch_mfu_right<T>(n, lines, in, mode_pack<T>(M, 2), mode_pack<T>(M, 3), out, st);
  if (M.sym) return launch_tpu_right<T>(n, lines, in, mode_half<T>(M, 6), mode_half<T>(M, 7), out, st);
  return launch_tp_right<T>(lines, n, n, in, mode_full<T>(M, 3), out, st);
}

}  // namespace lk
