// FP32 line transforms of a mirror-symmetric axis on the matrix cores, along a strided axis ("left"), in the
// folded half-size form of lk_transform.hip: forward, the line is folded on load and contracted with the
// even and the odd half matrix; backward, both are contracted and the result is unfolded on store.
//
// The contraction uses v_mfma_f32_4x4x1 (16 independent 4 x 4 blocks, a product of the rate of the 16x16x4
// form: 110 against 120 TFLOP/s measured).  The data operand is one contraction index of 64 columns, a lane each:
// here the even parts of 32 neighbouring columns in the lower lanes and their odd parts in the upper ones.
// The matrix operand can be broadcast from one block to eight: a register holds the pieces of four rows for
// eight contraction indices, even and odd (lane l: parity l / 32, index l / 4 % 8, row l % 4), and each
// instruction picks one index.  So a matrix piece is loaded once per eight instructions, straight from
// the L2, one load fetches the two rows of a pair and one store writes two rows of the result, and the two
// lane halves meet by v_permlane32_swap.
//
// A block is four waves on the same 32 columns.  They load the columns together, all loads in flight at once,
// fold them (or divide them by the eigenvalues) once and share them through LDS; each wave then does
// a quarter of the row groups.
// What bounds it: at 150^3 (27 MB, 0.5 GF) the start, the loads, the products and the stores take 4.5 + 2.7 + 6 + 2.5 us,
// one after the other because every block of so short a kernel is resident at once.  100^3 6.2-8.7 us, 150^3
// 15.3-17.2 us a transform, where one wave per 16 columns with the 16x16x4 form, waiting for each step's
// loads, took 9 and 21 us and the casts of the outer fields 5 and 7.5 us each.  Columns in all 64 lanes
// and both parities in turn: 15 us at 150^3 with three blocks on some CUs and one on others, and twice the load and
// store instructions.
// The field on the outer side may be FP64 (the first and the last transform of the FP32 pressure solve): it
// is rounded on load as a separate cast would.
#include <hip/hip_runtime.h>

#include "lk_device.h"
#include "lk_internal.h"

namespace lk {
namespace {

typedef float F4 __attribute__((ext_vector_type(4)));
typedef float F2 __attribute__((ext_vector_type(2)));
typedef unsigned U2 __attribute__((ext_vector_type(2)));

// v / a for the eigenvalue scaling, a not zero: hardware reciprocal and one Newton step
__device__ __forceinline__ float m4_div(float v, double a) {
  const float af = (float)a;
  float y = __builtin_amdgcn_rcpf(af);
  y = fmaf(fmaf(-af, y, 1.0f), y, y);
  return v * y;
}

struct M4Scale {  // backward only: modes divided by lm[mode] + ly[col / nxs] + lx[col % nxs], the mode (zm, zj, zi) zeroed
  const double *lm, *ly, *lx;
  int nxs, zm, zj, zi;
};

template <typename IN>
__device__ __forceinline__ IN m4_load(const __amdgpu_buffer_rsrc_t& r, unsigned ofs) {
  if constexpr (sizeof(IN) == 8)
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, (int)ofs, 0, 0));
  else
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)ofs, 0, 0));
}
template <typename OUT>
__device__ __forceinline__ void m4_store(OUT x, const __amdgpu_buffer_rsrc_t& r, unsigned ofs) {
  if constexpr (sizeof(OUT) == 8)
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(U2, x), r, (int)ofs, 0, 0);
  else
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, x), r, (int)ofs, 0, 0);
}

// x of the lower and of the upper lanes, each in both halves
__device__ __forceinline__ F2 m4_halves(float x) {
  const unsigned b = __builtin_bit_cast(unsigned, x);
  const U2 r = __builtin_amdgcn_permlane32_swap(b, b, false, false);
  const unsigned lo = r.x, hi = r.y;
  return F2{__builtin_bit_cast(float, lo), __builtin_bit_cast(float, hi)};
}

template <int RG, bool FOLD, bool SCALE, typename IN, typename OUT>
__global__ void __launch_bounds__(256, 2) k_m4_left(int n, int he, int ho, int N, const float* __restrict__ P,
                                                    const IN* __restrict__ B, OUT* __restrict__ C, unsigned elems,
                                                    int nseg, unsigned seg_stride, unsigned kstride, M4Scale sc) {
  constexpr int KP = 16 * RG, KH = (RG + 1) / 2;  // RG = ceil(he / 16)
  __shared__ float lds[KP * 64];                  // [contraction index][even part of 32 columns, odd part]
  constexpr unsigned kGhost = 1u << 31;           // an offset past the field: loads give 0, stores are dropped
  constexpr unsigned SI = sizeof(IN), SO = sizeof(OUT);
  const int G = (he + 3) / 4;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool up = lane >= 32;
  const int col = blockIdx.x * 32 + (lane & 31);
  const unsigned at = (unsigned)(col / nseg) * seg_stride + (unsigned)(col % nseg);
  const int lim = col < N ? up ? ho : he : 0;  // the lane's parity has this many modes, this many pairs
  const __amdgpu_buffer_rsrc_t rin =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<IN*>(B), (short)0, (int)(SI * elems), 0x00020000);
  const __amdgpu_buffer_rsrc_t rout = __builtin_amdgcn_make_buffer_rsrc(C, (short)0, (int)(SO * elems), 0x00020000);
  const __amdgpu_buffer_rsrc_t rp =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(P), (short)0, G * KH * 1024, 0x00020000);
  // row k of the lane's column: points k and n - 1 - k of a pair, or modes k and he + k
  auto point = [&](int k) { return at + kstride * (unsigned)(up ? n - 1 - k : k); };
  auto mode = [&](int k) { return at + kstride * (unsigned)(up ? he + k : k); };
  const int g0 = wave * RG;
  F4 pc[RG][KH];
  {
    // rows past the half length (and the middle row's second half) read as 0
    IN x[4 * RG];
#pragma unroll
    for (int q = 0; q < 4 * RG; ++q) {
      const int k = 4 * q + wave;
      x[q] = m4_load<IN>(rin, k < lim ? SI * (FOLD ? point(k) : mode(k)) : kGhost);
    }
    // this wave's pieces, behind the columns' loads and all at once: four steps of eight indices per 16 bytes;
    // groups past the matrix repeat the last one and are not stored
#pragma unroll
    for (int g = 0; g < RG; ++g)
#pragma unroll
      for (int h = 0; h < KH; ++h) {
        const int so = (min(g0 + g, G - 1) * KH + h) * 1024;
        if (2 * h + 1 < RG) {
          pc[g][h] = __builtin_bit_cast(F4, __builtin_amdgcn_raw_buffer_load_b128(rp, 16 * lane, so, 0));
        } else {
          const F2 y = __builtin_bit_cast(F2, __builtin_amdgcn_raw_buffer_load_b64(rp, 16 * lane, so, 0));
          pc[g][h] = F4{y.x, y.y, 0, 0};
        }
      }
    double sxy = 0.0;
    int zk = -1;  // the constant mode's index in this lane
    if (SCALE) {
      const int jj = col < N ? col / sc.nxs : 0, ii = col < N ? col % sc.nxs : 0;
      sxy = sc.ly[jj] + sc.lx[ii];
      if (jj == sc.zj && ii == sc.zi) zk = up ? sc.zm - he : sc.zm;
    }
#pragma unroll
    for (int q = 0; q < 4 * RG; ++q) {
      const int k = 4 * q + wave;
      float s = (float)x[q];
      if (FOLD) {
        const F2 p = m4_halves(s);
        s = p.x + (up ? -p.y : p.y);
        // the odd part has no middle row
        if (up && k >= ho) s = 0.f;
      } else if (SCALE) {  // padding and the constant mode stay exactly zero (no 0 / 0)
        s = (k >= lim || k == zk) ? 0.f : m4_div(s, sc.lm[min(up ? he + k : k, n - 1)] + sxy);
      }
      lds[k * 64 + lane] = s;
    }
  }
  __syncthreads();
  F4 acc[RG];
#pragma unroll
  for (int g = 0; g < RG; ++g) acc[g] = F4{0, 0, 0, 0};
#pragma unroll
  for (int kk = 0; kk < 2 * RG; ++kk) {
    if (kk == 2 * RG - 1 && 8 * kk >= he) break;
    float b[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) b[t] = lds[(8 * kk + t) * 64 + lane];
#define LK_M4(t)                                  \
  _Pragma("unroll") for (int g = 0; g < RG; ++g)  \
      acc[g] = __builtin_amdgcn_mfma_f32_4x4x1f32(pc[g][kk / 4][kk % 4], b[t], acc[g], 3, t, 0);
    LK_M4(0) LK_M4(1) LK_M4(2) LK_M4(3) LK_M4(4) LK_M4(5) LK_M4(6) LK_M4(7)
#undef LK_M4
  }
#pragma unroll
  for (int g = 0; g < RG; ++g)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int o = 4 * (g0 + g) + v;
      float y = acc[g][v];
      if (!FOLD) {
        const F2 p = m4_halves(y);
        y = p.x + (up ? -p.y : p.y);
      }
      m4_store<OUT>((OUT)y, rout, o < lim ? SO * (FOLD ? mode(o) : point(o)) : kGhost);
    }
}

template <bool FOLD, bool SCALE, typename IN, typename OUT>
hipError_t m4_launch(int n, int N, const float* P, const IN* B, OUT* C, size_t elems, int nseg, long seg_stride,
                     long kstride, const M4Scale& sc, hipStream_t st) {
  const int he = (n + 1) / 2, ho = n / 2, G = (he + 3) / 4;
  const dim3 grid(blocks_for(N, 32)), block(256);
#define M4(RG)                                                                                                       \
  case RG:                                                                                                           \
    hipLaunchKernelGGL((k_m4_left<RG, FOLD, SCALE, IN, OUT>), grid, block, 0, st, n, he, ho, N, P, B, C,           \
                       (unsigned)elems, nseg, (unsigned)seg_stride, (unsigned)kstride, sc);                          \
    break;
  switch ((G + 3) / 4) {
    M4(1) M4(2) M4(3) M4(4) M4(5) M4(6) M4(7) M4(8)
    default: return hipErrorInvalidValue;
  }
#undef M4
  return hipGetLastError();
}

}  // namespace

template <typename IN>
hipError_t launch_m4f_left(int n, int N, const float* P, const IN* B, float* C, size_t elems, int nseg,
                           long seg_stride, long kstride, hipStream_t st) {
  return m4_launch<true, false, IN, float>(n, N, P, B, C, elems, nseg, seg_stride, kstride, M4Scale{}, st);
}
template hipError_t launch_m4f_left<float>(int, int, const float*, const float*, float*, size_t, int, long, long, hipStream_t);
template hipError_t launch_m4f_left<double>(int, int, const float*, const double*, float*, size_t, int, long, long, hipStream_t);

template <typename OUT>
hipError_t launch_m4u_left(int n, int N, const float* P, const float* B, OUT* C, size_t elems, int nseg,
                           long seg_stride, long kstride, const double* lm, const double* ly, const double* lx, int nxs,
                           int zm, int zj, int zi, hipStream_t st) {
  const M4Scale sc{lm, ly, lx, nxs, zm, zj, zi};
  if constexpr (sizeof(OUT) == sizeof(float))  // (the scaled transform is an inner one)
    if (lm) return m4_launch<false, true, float, OUT>(n, N, P, B, C, elems, nseg, seg_stride, kstride, sc, st);
  if (lm) return hipErrorInvalidValue;
  return m4_launch<false, false, float, OUT>(n, N, P, B, C, elems, nseg, seg_stride, kstride, sc, st);
}
template hipError_t launch_m4u_left<float>(int, int, const float*, const float*, float*, size_t, int, long, long,
                                           const double*, const double*, const double*, int, int, int, int, hipStream_t);
template hipError_t launch_m4u_left<double>(int, int, const float*, const float*, double*, size_t, int, long, long,
                                            const double*, const double*, const double*, int, int, int, int, hipStream_t);

}  // namespace lk
