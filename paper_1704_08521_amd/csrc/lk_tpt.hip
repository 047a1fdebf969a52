// Tridiagonal solves along x in (y, z) mode space: the x step of the pressure-correction
// Poisson solve by the TPT route of Section 3 (mode transforms in two directions, a
// tridiagonal solve in the third).  For every x-line (k, j) of the transformed field,
// (L_x + ly[j] + lz[k]) phi = rhs, with L_x = D_x G_x on the cells of the line (zero flux
// through the walls).  The partition method with LPW lanes per line, 64 / LPW lines per wave: lane p owns
// the M consecutive rows of segment p and eliminates its interior rows in registers (one Thomas sweep with
// the segment before it as second right side), which leaves one unknown per segment, its last row; those
// form a tridiagonal system (the Schur complement, diagonally dominant like the line's own matrix)
// solved by cyclic reduction across the lanes; each lane then substitutes back.  The line whose
// shift is zero (the zero modes of y and z) is singular: its first equation is replaced by phi_0 = 0
// and the solution is re-centred to zero d-weighted mean, which sets the constant mode to zero as the
// transform route does.  The plane projections use the same pass with one shift array
// null (adding nothing) and a negative zero-mode index matching every index.
//
// Few lanes with many rows each, as long as there are lines to fill the chip: a row costs about 18 instructions, a step of the reduction about 45, so 16 lanes
// (four steps, their neighbours reached by row shifts of the vector unit) do a third of the work of 64 lanes
// (six steps through LDS permutes) and leave fewer lanes idle.  A segment is 13 values at 200 cells, which
// the lanes could only read and write piecemeal; so the lines of a wave, one contiguous piece of the field, are
// read and written 64 values at a time and turned in the wave's part of LDS, segments an odd number of
// values apart.  Waves go over several groups of lines, the next group's loads in flight, the coefficients of
// their rows kept in registers.
// The elimination is free of subtractions: with the rows written as (a + c + sg) x_r = a x_{r-1} + c x_{r+1} - d,
// sg = -shift >= 0, every pivot is a sum of positive terms, in the segments and across the lanes.  In FP32 the
// error of the pressure solve falls from 5e-6 .. 6e-4 (16 to 400 cells) to 2e-7 .. 6e-7, so the FP32 form
// often needs a pass less; in FP64 it is as before.
// HBM bound: one read and one write of the field (128 MB, 22 us at 200^3; 29.4 us by kernel trace).  By events on the
// stream, against one wave per line with subtractions: 64^3 7 us / 9, 100^3 12 / 17, 150^3 18 / 28, 200^3 31 / 47, 256^3 61 / 76;
// FP32 100^3 10 / 12, 150^3 16 / 22, 200^3 23 / 33.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "lk_device.h"
#include "lk_internal.h"

namespace lk {
namespace {

constexpr int kTriWaves = 4;   // waves per block
constexpr int kTriOcc = 2;     // waves per SIMD
// Blocks: two waves per SIMD, as many as fit with the longer segments' registers, so that no wave's start-up (the
// rows' coefficients and their places in LDS) waits for another's end: 200^3 512 blocks 29 us, 256 31, 768 35, one
// group per wave 47 us; 100^3 10.4 / 10.8 / 11.1 / 11.6.
constexpr int kTriBlocks = 512;

// 1 / a to the type's accuracy: the hardware reciprocal refined by Newton steps (two in
// FP64, one in FP32)
__device__ __forceinline__ double rcpx(double a) {
  double y = __builtin_amdgcn_rcp(a);
  double e = fma(-a, y, 1.0);
  y = fma(e, y, y);
  e = fma(-a, y, 1.0);
  return fma(e, y, y);
}
__device__ __forceinline__ float rcpx(float a) {
  const float y = __builtin_amdgcn_rcpf(a);
  return fmaf(fmaf(-a, y, 1.0f), y, y);
}

// x of the lane D below (UP) or above within the LPW lanes of a line; past their ends 0 or the lane's own (never another
// line's: what is not finite stays in its line)
template <int LPW, int D, bool UP>
__device__ __forceinline__ float lane_shift(float x) {
  if constexpr (LPW == 16)
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), (UP ? 0x110 : 0x100) + D,
                                                                 0xf, 0xf, true));
  else return UP ? __shfl_up(x, D, LPW) : __shfl_down(x, D, LPW);
}
template <int LPW, int D, bool UP>
__device__ __forceinline__ double lane_shift(double x) {
  if constexpr (LPW == 16) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
    constexpr int ctrl = (UP ? 0x110 : 0x100) + D;
    const unsigned lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, ctrl, 0xf, 0xf, true);
    const unsigned hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), ctrl, 0xf, 0xf, true);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
  } else {
    return UP ? __shfl_up(x, D, LPW) : __shfl_down(x, D, LPW);
  }
}

// Cyclic reduction across the lanes of a line, from step D on, of (al + ga + ex) z_p = al z_{p-D} + ga z_{p+D} + f.
// The lower coupling al is exactly zero on lanes below D and the upper one ga on lanes with no row D above
// (initially from the zero coefficients of the line's first and last rows, then because each update
// multiplies by them), so the products with the values a shift returns past the line's ends vanish and
// the updates need no lane conditions.  Each lane sends its row divided by its diagonal.
template <int LPW, int D, typename T>
__device__ __forceinline__ void reduce_lanes(T& al, T& ga, T& ex, T& f) {
  if constexpr (D < LPW) {
    const T r = rcpx(al + ga + ex);
    const T as = al * r, gs = ga * r, es = ex * r, fs = f * r;
    const T am = lane_shift<LPW, D, true>(as), em = lane_shift<LPW, D, true>(es), fm = lane_shift<LPW, D, true>(fs);
    const T gp = lane_shift<LPW, D, false>(gs), ep = lane_shift<LPW, D, false>(es), fp = lane_shift<LPW, D, false>(fs);
    ex += al * em;
    f += al * fm;
    al *= am;
    ex += ga * ep;
    f += ga * fp;
    ga *= gp;
    reduce_lanes<LPW, 2 * D>(al, ga, ex, f);
  }
}

template <typename T>
__device__ __forceinline__ T tri_load(const __amdgpu_buffer_rsrc_t& b, unsigned ofs, int so) {
  if constexpr (sizeof(T) == 8) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(b, (int)ofs, so, 0));
  else return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(b, (int)ofs, so, 0));
}
template <typename T>
__device__ __forceinline__ void tri_store(T x, const __amdgpu_buffer_rsrc_t& b, unsigned ofs, int so) {
  typedef unsigned U2 __attribute__((ext_vector_type(2)));
  if constexpr (sizeof(T) == 8) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(U2, x), b, (int)ofs, so, 0);
  else __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, x), b, (int)ofs, so, 0);
}

template <typename T, int M, int LPW>
__global__ void __launch_bounds__(64 * kTriWaves, kTriOcc) k_tridiag_x(
    const double* __restrict__ rd, const double* __restrict__ rdd, const double* __restrict__ dx, int n, int ny,
    long lines, const double* __restrict__ ly, const double* __restrict__ lz, int zj, int zk,
    const T* __restrict__ in, T* __restrict__ out) {
  constexpr int LPG = 64 / LPW, MP = M | 1;  // lines of a group; values between the segments in LDS
  constexpr bool kAhead = sizeof(T) * M < 128;  // the next group's loads in flight (no registers for them beyond)
  __shared__ T turn[kTriWaves][64 * MP];
  const int lane = (int)(threadIdx.x & 63), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int p = lane % LPW, s0 = p * M;
  const long groups = (lines + LPG - 1) / LPG, step = (long)gridDim.x * kTriWaves;
  const long first = (long)blockIdx.x * kTriWaves + wave;
  if (first >= groups) return;
  T x[M];
  auto buffer = [&](const T* f, long group) {
    const long l0 = group * LPG, left = lines - l0;
    const int rows = left <= 0 ? 0 : left < LPG ? (int)left : LPG;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(f) + (rows ? l0 * n : 0), (short)0, (int)sizeof(T) * rows * n,
                                             0x00020000);
  };
  auto fetch = [&](long group) {
    const __amdgpu_buffer_rsrc_t b = buffer(in, group);
#pragma unroll
    for (int t = 0; t < M; ++t) x[t] = tri_load<T>(b, sizeof(T) * lane, sizeof(T) * 64 * t);
  };
  fetch(first);
  T* seg = turn[wave] + lane * MP;
  // value 64 t + lane of a group sits at pos[t] (values past the group's lines: the end of the wave's part)
  int pos[M];
#pragma unroll
  for (int t = 0; t < M; ++t) {
    const int e = 64 * t + lane;
    int q = 0;
#pragma unroll
    for (int l = 1; l <= LPG; ++l) q += e >= l * n;
    const int r = e - q * n, h = (int)((unsigned)r / M);
    pos[t] = q < LPG ? (q * LPW + h) * MP + (r - h * M) : -1;
  }
#pragma unroll
  for (int i = 0; i < MP; ++i) seg[i] = T(0);  // (rows past the line's end stay so: d = 0)
  __builtin_amdgcn_wave_barrier();
  // the rows: (a + c + sg) x_r = a x_{r-1} + c x_{r+1} - d with sg = -shift >= 0; the coefficients are formed in
  // FP64 and rounded to T.  Rows past the line's end get a = 1, c = 0: the last row's c is zero, so
  // nothing of them reaches the line.
  T A[M], C[M];
#pragma unroll
  for (int i = 0; i < M; ++i) {
    const int r = s0 + i, rr = min(r, n - 1);
    const double rdr = rd[rr], rdd0 = rdd[rr], rdd1 = rdd[rr + 1];  // rdd has n + 1 entries
    A[i] = (T)(r >= n ? 1.0 : r > 0 ? rdd0 * rdr : 0.0);
    C[i] = (T)(r + 1 < n ? rdd1 * rdr : 0.0);
  }
  for (long group = first; group < groups; group += step) {
    const long line = min(group * LPG + lane / LPW, lines - 1);
    const int k = (int)((unsigned)line / (unsigned)ny), j = (int)line - k * ny;
    const bool sing = (zj < 0 || j == zj) && (zk < 0 || k == zk);
    const T sg = sing ? T(0) : (T)(-((ly ? ly[j] : 0.0) + (lz ? lz[k] : 0.0)));
#pragma unroll
    for (int t = 0; t < M; ++t)
      if (pos[t] >= 0) turn[wave][pos[t]] = x[t];
    if (kAhead) fetch(group + step);
    __builtin_amdgcn_wave_barrier();
    // interior rows 0 .. M - 2: x_i = y_i + v_i z_{p-1} + g_i x_{i+1}, with z_{p-1} the previous lane's last row
    // and x_{M-1} = z_p the own one, and e_i = 1 - v_i - g_i, which has a recurrence of its own: the pivot
    // a + c + sg - a g_{i-1} is the sum of the three positive terms c, a v_{i-1} and sg + a e_{i-1}, so that
    // nothing cancels where sg is small against a and c.  The singular line's first row: x_0 = 0.
    const bool pin = sing && p == 0;
    T y[M], v[M], g[M], es[M];
    {
      const T r = rcpx(C[0] + A[0] + sg);
      g[0] = pin ? T(0) : C[0] * r;
      y[0] = pin ? T(0) : -seg[0] * r;
      v[0] = A[0] * r;
      es[0] = pin ? T(1) : sg * r;
    }
#pragma unroll
    for (int i = 1; i < M - 1; ++i) {
      const T h = sg + A[i] * es[i - 1], t = A[i] * v[i - 1];
      const T r = rcpx(C[i] + (h + t));
      g[i] = C[i] * r;
      v[i] = t * r;
      es[i] = h * r;
      y[i] = (A[i] * y[i - 1] - seg[i]) * r;
    }
    // the first row in the segment's ends, x_0 = yf + vf z_{p-1} + wf z_p (vf is not needed), ef = 1 - vf - wf
    T yf = y[M - 2], wf = g[M - 2], ef = es[M - 2];
#pragma unroll
    for (int i = M - 3; i >= 0; --i) {
      yf = y[i] + g[i] * yf;
      ef = es[i] + g[i] * ef;
      wf = g[i] * wf;
    }
    // the last row's equation in the segment ends
    const T yn = lane_shift<LPW, 1, false>(yf), en = lane_shift<LPW, 1, false>(ef), wn = lane_shift<LPW, 1, false>(wf);
    T al = A[M - 1] * v[M - 2], ga = C[M - 1] * wn;
    T ex = sg + A[M - 1] * es[M - 2] + C[M - 1] * en;
    T f = A[M - 1] * y[M - 2] + C[M - 1] * yn - seg[M - 1];
    reduce_lanes<LPW, 1>(al, ga, ex, f);
    const T z = f / ex;
    const T zu = lane_shift<LPW, 1, true>(z);
    const T zl = p > 0 ? zu : T(0);
    g[M - 1] = z;  // (from here on the solution)
#pragma unroll
    for (int i = M - 2; i >= 0; --i) g[i] = (y[i] + v[i] * zl) + g[i] * g[i + 1];
    if (__any(sing)) {
      double sw = 0.0, swx = 0.0;
#pragma unroll
      for (int i = 0; i < M; ++i)
        if (s0 + i < n) {
          const double w = dx[s0 + i];
          sw += w;
          swx += w * (double)g[i];
        }
#pragma unroll
      for (int d = LPW / 2; d > 0; d /= 2) {
        sw += __shfl_xor(sw, d);
        swx += __shfl_xor(swx, d);
      }
      const T mean = sing ? (T)(swx / sw) : T(0);
#pragma unroll
      for (int i = 0; i < M; ++i) g[i] -= mean;
    }
#pragma unroll
    for (int i = 0; i < M; ++i)
      if (s0 + i < n) seg[i] = g[i];
    __builtin_amdgcn_wave_barrier();
    const __amdgpu_buffer_rsrc_t b = buffer(out, group);
#pragma unroll
    for (int t = 0; t < M; ++t) tri_store<T>(turn[wave][max(pos[t], 0)], b, sizeof(T) * lane, sizeof(T) * 64 * t);
    __builtin_amdgcn_wave_barrier();
    if (!kAhead) fetch(group + step);
  }
}

}  // namespace

int tridiag_x_max() { return 64 * 16; }

template <typename T>
hipError_t launch_tridiag_x(const GridDev& g, const double* ly, const double* lz, int zj, int zk, const T* in, T* out,
                            hipStream_t st) {
  const int n = g.x.n, ny = g.y.n, nz = g.z.n;
  const long lines = (long)ny * nz;
  const double *rd = g.x.rd, *rdd = g.x.rdd, *dx = g.x.d;
  // Rows per lane: the smallest instance that covers the line with 16 lanes; from 208 cells on the 16 rows that this
  // would take leave no registers for the next group's loads in FP64 (256^3 69 us, 8 rows on 32 lanes 63).  Where
  // there are few lines, a wave's own chain of rows and steps is all that counts, and that is shortest with all 64 lanes
  // on a line (by events): 200 cells, 1024 lines 7.0 us against 10.4 (2500 lines 10.7 / 10.9, 4096 13.2 / 11.9), 128 cells 6.3
  // / 8.3 (2000 lines 8.8 / 8.4); up to 64 cells no difference.  Past 256 cells 16 rows are a long chain for longer: 512
  // cells, 1024 lines 9.2 / 16, 10000 25.8 / 31.8, 20480 43 / 47, but 300 cells, 40000 lines 67 / 59.
#define TRI(M, LPW)                                                                                                  \
  {                                                                                                                  \
    const long groups = (lines + 64 / LPW - 1) / (64 / LPW);                                                         \
    const dim3 grid((unsigned)std::min<long>((groups + kTriWaves - 1) / kTriWaves, kTriBlocks));                     \
    hipLaunchKernelGGL((k_tridiag_x<T, M, LPW>), grid, dim3(64 * kTriWaves), 0, st, rd, rdd, dx, n, ny, lines, ly, lz, zj, \
                       zk, in, out);                                                                                 \
  }
  const bool few = lines <= (n > 256 ? 20000 : 1600);
  if (few && n > 64 && n <= 128) TRI(2, 64)
  else if (few && n > 128 && n <= 256) TRI(4, 64)
  else if (few && n > 256 && n <= 512) TRI(8, 64)
  else if (n <= 32) TRI(2, 16)
  else if (n <= 64) TRI(4, 16)
  else if (n <= 80) TRI(5, 16)
  else if (n <= 96) TRI(6, 16)
  else if (n <= 112) TRI(7, 16)
  else if (n <= 128) TRI(8, 16)
  else if (n <= 160) TRI(10, 16)
  else if (n <= 208) TRI(13, 16)
  else if (n <= 256) TRI(8, 32)
  else if (n <= 512) TRI(16, 32)
  else if (n <= 1024) TRI(16, 64)
  else return hipErrorInvalidValue;
#undef TRI
  return hipGetLastError();
}

template hipError_t launch_tridiag_x<double>(const GridDev&, const double*, const double*, int, int, const double*,
                                             double*, hipStream_t);
template hipError_t launch_tridiag_x<float>(const GridDev&, const double*, const double*, int, int, const float*,
                                            float*, hipStream_t);

}  // namespace lk
