// FP64 line transforms on the matrix cores, along a strided axis ("left": every column of the field is multiplied
// by the mode matrix).  A mirror-symmetric axis has the folded half-size form of
// lk_transform.hip: forward, the line is folded on load (f_k + f_{n-1-k}, f_k - f_{n-1-k}) and contracted
// with the even and the odd half matrix; backward, the even and the odd modes are contracted and
// the result is unfolded on store.  Any other axis has the full matrix, its lower and its upper rows in the
// places of the even and the odd half matrix and the same data for both.
//
// The contraction uses v_mfma_f64_4x4x4 (four independent 4 x 4 blocks), which runs at 67-75 TFLOP/s here
// against 32-46 TFLOP/s of v_mfma_f64_16x16x4 (a register-only loop of each, one to four waves per SIMD).
// Its four blocks are four groups of four columns, so the data operand is 16 columns x 4 contraction
// indices, a lane per value as it is loaded (lane l: column l % 16, index l / 16), and the matrix operand
// is one 4 x 4 piece repeated for every block (lane l: row l % 4, index l / 16); the result lane l
// holds row l / 16 of column l % 16.
//
// A matrix piece feeds only 16 columns, so the pieces come from LDS and each is used for W column tiles of
// the wave.  A block keeps the pieces of GT row groups (of four rows), each with those of the
// other half matrix beside it so that one 16-byte read fetches both; an axis
// with more groups is split into classes of GT, neighbouring blocks of the same XCD doing the classes of the
// same columns.  The columns' values are loaded PD steps ahead into a register ring; with the
// pieces in LDS these are the only vector-memory loads of the loop, so they are waited for one step at a time.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "lk_device.h"
#include "lk_internal.h"

namespace lk {
namespace {

typedef unsigned U2 __attribute__((ext_vector_type(2)));
typedef double D2 __attribute__((ext_vector_type(2)));

// v / a, a not zero (the eigenvalue sums of the pressure are negative): hardware reciprocal refined by two Newton steps and one residual correction of
// the quotient (within an ulp of v / a, a third of the instructions of the IEEE sequence).
__device__ __forceinline__ double mx_div(double v, double a) {
  double y = __builtin_amdgcn_rcp(a);
  double e = fma(-a, y, 1.0);
  y = fma(e, y, y);
  e = fma(-a, y, 1.0);
  y = fma(e, y, y);
  const double q = v * y;
  return fma(fma(-a, q, v), y, q);
}

// backward only: modes divided by lm[mode] + ly[col / nxs] + lx[col % nxs] (ly, lx may be null: 0), the mode
// (zm, zj, zi) zeroed (zm negative: none; zj, zi negative: any)
struct MxScale {
  const double *lm, *ly, *lx;
  int nxs, zm, zj, zi;
};

enum MxForm { kFold, kUnfold, kFull };

template <int GT, int W, int PD, int CHP, MxForm FORM, bool SCALE, int MAXW, int OCC, bool SHORT>
__global__ void __launch_bounds__(64 * MAXW, OCC) k_mx_left(int n, int he, int ho, int N, const double* __restrict__ P,
                                                            int G, int classes,
                                                            const double* __restrict__ B, double* __restrict__ C,
                                                            unsigned bytes, int nseg, unsigned seg_stride,
                                                            unsigned kstride, MxScale sc) {
  // pieces [KQ][GT][16], (even, odd) pairs, and a step of padding; with SCALE the eigenvalues [2][4 KQ]
  extern __shared__ D2 lds[];
  constexpr unsigned kGhost = 1u << 31;  // an offset past the field: loads give 0, stores are dropped
  constexpr bool FOLD = FORM == kFold, FULL = FORM == kFull;
  const int K = FULL ? n : he, KQ = (K + 3) / 4;  // contracted indices, and steps of four
  const int tid = threadIdx.x, lane = tid & 63, nw = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // tiles: classes of the same columns next to each other on one XCD
  constexpr int NX = 8;
  const int bid = blockIdx.x, nb = gridDim.x, xcd = bid % NX, per = nb / NX, more = nb % NX;
  const int tile = (xcd < more ? xcd * (per + 1) : more * (per + 1) + (xcd - more) * per) + bid / NX;
  const int cls = SHORT ? 0 : tile % classes, g0 = cls * GT;
  const int col0 = ((SHORT ? tile : tile / classes) * nw + wave) * 16 * W;
  const int g = lane >> 4;
  const __amdgpu_buffer_rsrc_t rin =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(B), (short)0, (int)bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rout = __builtin_amdgcn_make_buffer_rsrc(C, (short)0, (int)bytes, 0x00020000);
  unsigned base[W];
  double sxy[W];
  bool zc[W];
#pragma unroll
  for (int c = 0; c < W; ++c) {
    const int col = col0 + 16 * c + (lane & 15);
    base[c] = col < N ? 8u * ((unsigned)(col / nseg) * seg_stride + (unsigned)(col % nseg)) : kGhost;
    if (SCALE) {
      const int jj = col < N ? col / sc.nxs : 0, ii = col < N ? col % sc.nxs : 0;
      sxy[c] = (sc.ly ? sc.ly[jj] : 0.0) + (sc.lx ? sc.lx[ii] : 0.0);
      zc[c] = (sc.zj < 0 || jj == sc.zj) && (sc.zi < 0 || ii == sc.zi);
    }
  }
  // element k of a column: forward the pair k, n - 1 - k (the middle row once), backward the even mode k
  // and the odd mode k, full the value k
  double x1[PD][W], x2[PD][W];
  auto load = [&](int u, int kq) {
    const int k = 4 * kq + g, k2 = FOLD ? n - 1 - k : he + k;
    const bool in1 = k < K, in2 = FOLD ? k < he && k2 != k : k < ho;
    const unsigned o1 = (unsigned)k * (8u * kstride), o2 = (unsigned)k2 * (8u * kstride);
#pragma unroll
    for (int c = 0; c < W; ++c) {
      const unsigned a1 = in1 && base[c] != kGhost ? base[c] + o1 : kGhost;
      const unsigned a2 = in2 && base[c] != kGhost ? base[c] + o2 : kGhost;
      x1[u][c] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rin, (int)a1, 0, 0));
      if (!FULL) x2[u][c] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rin, (int)a2, 0, 0));
    }
  };
#pragma unroll
  for (int u = 0; u < PD; ++u) load(u, u);
  // SHORT: the ring holds every step and the class every group, so the pieces (and eigenvalues) are loaded with
  // the data, straight into registers
  D2 fr[SHORT ? PD : 1][GT];
  double lr[2][SHORT ? PD : 1];
  if constexpr (SHORT) {
    const D2* src = (const D2*)P + (lane >> 4) * 4 + (lane & 3);
#pragma unroll
    for (int u = 0; u < PD; ++u) {
#pragma unroll
      for (int t = 0; t < GT; ++t) {
        fr[u][t] = src[(min(u, KQ - 1) * G + min(t, G - 1)) * 16];
        if (t >= G) fr[u][t] = D2{0.0, 0.0};
      }
      if (SCALE) {
        lr[0][u] = sc.lm[min(4 * u + g, K - 1)];
        lr[1][u] = sc.lm[min(he + 4 * u + g, n - 1)];
      }
    }
  } else {  // the class's pieces; groups past the matrix are zero
    const D2* src = (const D2*)P;
    const int total = KQ * GT * 16, step = blockDim.x;
    constexpr int NB = 8;
    for (int e0 = tid; e0 < total; e0 += NB * step) {
      D2 v[NB];
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        const int e = min(e0 + q * step, total - 1), kq = e / (GT * 16), r = e % (GT * 16);
        v[q] = src[((long)kq * G + min(g0 + r / 16, G - 1)) * 16 + r % 16];
        if (g0 + r / 16 >= G) v[q] = D2{0.0, 0.0};
      }
#pragma unroll
      for (int q = 0; q < NB; ++q)
        if (e0 + q * step < total) lds[e0 + q * step] = v[q];
    }
  }
  double* lam = (double*)(lds + (KQ + 1) * GT * 16);
  if (SCALE && !SHORT)
    for (int k = tid; k < 4 * KQ; k += blockDim.x) {
      lam[k] = k < K ? sc.lm[k] : 1.0;
      if (!FULL) lam[4 * KQ + k] = k < ho ? sc.lm[he + k] : 1.0;
    }
  if (!SHORT) __syncthreads();
  if (col0 >= N) return;

  double ae[GT][W], ao[GT][W];
#pragma unroll
  for (int t = 0; t < GT; ++t)
#pragma unroll
    for (int c = 0; c < W; ++c) ae[t][c] = ao[t][c] = 0.0;
  // Pieces are read from LDS one chunk of CH groups ahead of the products that use them, across steps too
  // (the last step reads ahead into the padding); the scheduling fences keep the reads from being drawn
  // further ahead, which would cost the registers of the third wave per SIMD.
  constexpr int CH = SCALE ? 2 : CHP, NCH = (GT + CH - 1) / CH;
  const D2* pl = lds + (lane >> 4) * 4 + (lane & 3);
  D2 f[2][CH];
  auto pieces = [&](int q, int kq, int ch) {
#pragma unroll
    for (int t = 0; t < CH; ++t)
      if (ch * CH + t < GT) f[q][t] = SHORT ? fr[min(kq, PD - 1)][ch * CH + t] : pl[(kq * GT + ch * CH + t) * 16];
  };
  auto step = [&](int u, int kq) {
    double s[W], d[W];
    const int k = 4 * kq + g;
#pragma unroll
    for (int c = 0; c < W; ++c) {
      if (FOLD) {
        s[c] = x1[u][c] + x2[u][c];
        d[c] = x1[u][c] - x2[u][c];
      } else if (SCALE) {  // padding and the constant mode stay exactly zero (no 0 / 0)
        s[c] = (k >= K || (zc[c] && k == sc.zm)) ? 0.0 : mx_div(x1[u][c], (SHORT ? lr[0][u] : lam[k]) + sxy[c]);
        d[c] = FULL ? s[c] : (k >= ho || (zc[c] && he + k == sc.zm)) ? 0.0 : mx_div(x2[u][c], (SHORT ? lr[1][u] : lam[4 * KQ + k]) + sxy[c]);
      } else {
        s[c] = x1[u][c];
        d[c] = FULL ? s[c] : x2[u][c];
      }
    }
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
      const int q = (u * NCH + ch) & 1;
      if (ch + 1 < NCH) pieces(q ^ 1, kq, ch + 1);
      else pieces(q ^ 1, kq + 1, 0);
#pragma unroll
      for (int t = 0; t < CH; ++t)
        if (ch * CH + t < GT)
#pragma unroll
          for (int c = 0; c < W; ++c) {
            double &e = ae[ch * CH + t][c], &o = ao[ch * CH + t][c];
            e = __builtin_amdgcn_mfma_f64_4x4x4f64(f[q][t].x, s[c], e, 0, 0, 0);
            o = __builtin_amdgcn_mfma_f64_4x4x4f64(f[q][t].y, d[c], o, 0, 0, 0);
          }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  static_assert(PD * NCH % 2 == 0, "the two piece buffers alternate across the ring");
  pieces(0, 0, 0);
  int kq = 0;
  if (!SHORT)
    for (; kq + PD <= KQ; kq += PD) {
#pragma unroll
      for (int u = 0; u < PD; ++u) {
        step(u, kq + u);
        load(u, kq + u + PD);
      }
    }
#pragma unroll
  for (int u = 0; u < (SHORT ? PD : PD - 1); ++u)
    if (kq + u < KQ) step(u, SHORT ? u : kq + u);

  auto put = [&](double x, unsigned ofs) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(U2, x), rout, (int)ofs, 0, 0);
  };
#pragma unroll
  for (int t = 0; t < GT; ++t) {
    const int o = 4 * (g0 + t) + g;
    const bool in1 = o < he, in2 = o < ho;
    const unsigned o1 = (unsigned)o * (8u * kstride), o2 = (unsigned)(FORM == kUnfold ? n - 1 - o : he + o) * (8u * kstride);
#pragma unroll
    for (int c = 0; c < W; ++c) {
      const bool ok = base[c] != kGhost;
      put(FORM == kUnfold ? ae[t][c] + ao[t][c] : ae[t][c], ok && in1 ? base[c] + o1 : kGhost);
      put(FORM == kUnfold ? ae[t][c] - ao[t][c] : ao[t][c], ok && in2 ? base[c] + o2 : kGhost);
    }
  }
}

template <int GT, int W, int PD, int CH, int MAXW, int OCC, MxForm FORM, bool SHORT>
hipError_t mx_launch(int n, int N, const double* P, const double* B, double* C, size_t elems, int nseg,
                     long seg_stride, long kstride, const MxScale* sc, hipStream_t st) {
  const int he = (n + 1) / 2, ho = n / 2, G = (he + 3) / 4, classes = (G + GT - 1) / GT;
  const int KQ = FORM == kFull ? (n + 3) / 4 : G;
  if (SHORT && (KQ > PD || G > GT)) return hipErrorInvalidValue;
  const size_t lds = SHORT ? 0 : (size_t)(2 * (KQ + 1) * GT * 16 + (sc ? 8 * KQ : 0)) * sizeof(double);
  const long tiles = (N + 16 * W - 1) / (16 * W);
  // one block per CU where the waves of all classes fit the chip, else blocks of the full size
  const int nw = (int)std::min<long>(MAXW, std::max<long>(1, (tiles * classes + 255) / 256));
  const dim3 grid((unsigned)((tiles + nw - 1) / nw * classes)), block(64 * nw);
  auto run = [&](auto kernel) {
    if (lds > 65536) {  // past the default limit
      hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kernel, grid, block, lds, st, n, he, ho, N, P, G, classes, B, C, (unsigned)(8 * elems), nseg,
                       (unsigned)seg_stride, (unsigned)kstride, sc ? *sc : MxScale{});
    return hipGetLastError();
  };
  if constexpr (FORM != kFold)
    if (sc) return run(k_mx_left<GT, W, PD, CH, FORM, true, MAXW, OCC, SHORT>);
  return run(k_mx_left<GT, W, PD, CH, FORM, false, MAXW, OCC, SHORT>);
}

template <MxForm FORM>
hipError_t mx_pick(int n, int N, const double* P, const double* B, double* C, size_t elems, int nseg,
                   long seg_stride, long kstride, const MxScale* sc, hipStream_t st) {
  const int G = ((n + 1) / 2 + 3) / 4;
  // Groups per class, column tiles and ring by the number of row groups G (of n = 8 G points) and the columns.  Up
  // to n = 120 the columns of a cube are few: narrow waves and more classes fill the chip (100^3: 7.3 us a
  // transform; 13 groups in one class of 2 tiles 12), and so they do for any length with up to about 10000 columns
  // (these and the cubes with two figures by events on the stream, 2 to 3 us above the kernel's own time:
  // 64, 3000 and 10000 columns of 200: 11, 11 and 21 us; the wide variant 26, 28 and 25; of 256: 13, 16 and 31
  // against 37, 41 and 34; 16384 columns of 200 and 256: 26 and 43 against 26 and 35).  At n = 128 two
  // classes of 8 groups (128^3 14.4 and 18.2 us along y and z, 10 groups 15.7 and 19.6).  From there the data is read
  // once or twice and wider waves save reads of the pieces (150^3: 16 us; 3 classes 18); blocks of up to 16
  // waves, four per SIMD, hold all of 160^3 at once (27 and 30 us; blocks of 12, whose last few
  // made a second round, 36 and 41).  The last three need their registers for the accumulators: W = 2 halves the
  // LDS reads, which else bound them (200^3 42 against 45 us side by side; other runs 44-46), at three waves per SIMD
  // (n <= 208; classes of 11 groups up to 176, where two of 13 have more rows to spare: 176^3 29 and 34 us
  // against 33 and 37) or two (256^3: 92 us; narrower classes 97-125).  With 13 groups one to three vector registers are spilled; smaller chunks of pieces change neither
  // that nor the time.
  // Lines of up to 32 points (16 with the full matrix) have so few pieces that the way through LDS costs more than it
  // saves: a launch at 8^3 and 16^3 takes 2.2 and 2.8 us by kernel trace, through LDS 2.8 and 3.6.
#define MX(...) MX_LAUNCH(false, __VA_ARGS__)
#define MX_SHORT(...) MX_LAUNCH(true, __VA_ARGS__)
#define MX_LAUNCH(SHORT, GT, W, PD, CH, MAXW, OCC) \
  return mx_launch<GT, W, PD, CH, MAXW, OCC, FORM, SHORT>(n, N, P, B, C, elems, nseg, seg_stride, kstride, sc, st)
  if constexpr (FORM == kFull) {
    // Twice the products of the folded form, so the matrix cores bound it (97 x 121 x 65: 10.6 us a
    // transform against 23 and 15 us on the vector units).  The same reasons choose the variant: few
    // columns up to n = 136 (cubes of 100 and 130: 12 and 25 us; 5 groups of 2 tiles 11 and 29), then two
    // tiles a wave (160^3 36 us, 200^3 87; one tile 43 and 112), and at the end half as many classes
    // (256^3 197 us; 5 groups 225).
    if (G <= 2) MX_SHORT(2, 1, 4, 2, 4, 4);
    if (G <= 17) MX(4, 1, 4, 4, 4, 4);
    if (G <= 26) MX(5, 2, 4, 5, 8, 3);
    MX(8, 2, 4, 4, 8, 2);
  } else {
    if (G <= 2) MX_SHORT(2, 1, 2, 2, 4, 4);
    if (G <= 4) MX_SHORT(4, 1, 4, 4, 4, 4);
    if (G <= 8) MX(4, 1, 4, 4, 4, 4);
    if (G <= 15 || N <= 10000) MX(5, 1, 4, 5, 4, 4);
    if (G <= 16) MX(8, 1, 4, 4, 4, 4);
    if (G <= 20) MX(10, 1, 4, 4, 16, 4);
    if (G <= 22) MX(11, 2, 2, 4, 12, 3);
    if (G <= 26) MX(13, 2, 2, 4, 12, 3);
    MX(16, 2, 2, 4, 8, 2);
  }
#undef MX
#undef MX_SHORT
#undef MX_LAUNCH
}

}  // namespace

hipError_t launch_mxf_left(int n, int N, const double* P, const double* B, double* C, size_t elems,
                           int nseg, long seg_stride, long kstride, hipStream_t st) {
  return mx_pick<kFold>(n, N, P, B, C, elems, nseg, seg_stride, kstride, nullptr, st);
}

hipError_t launch_mxu_left(int n, int N, const double* P, const double* B, double* C, size_t elems,
                           int nseg, long seg_stride, long kstride, const double* lm, const double* ly, const double* lx,
                           int nxs, int zm, int zj, int zi, hipStream_t st) {
  const MxScale sc{lm, ly, lx, nxs, zm, zj, zi};
  return mx_pick<kUnfold>(n, N, P, B, C, elems, nseg, seg_stride, kstride, lm ? &sc : nullptr, st);
}

hipError_t launch_mx_full_left(int n, int N, const double* P, const double* B, double* C, size_t elems, int nseg,
                               long seg_stride, long kstride, const double* lm, const double* ly, const double* lx,
                               int nxs, int zm, int zj, int zi, hipStream_t st) {
  const MxScale sc{lm, ly, lx, nxs, zm, zj, zi};
  return mx_pick<kFull>(n, N, P, B, C, elems, nseg, seg_stride, kstride, lm ? &sc : nullptr, st);
}

}  // namespace lk
