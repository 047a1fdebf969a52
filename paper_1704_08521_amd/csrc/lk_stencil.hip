// Staggered finite-volume stencils: linearized momentum / residual (eq. 10,
// eq. 2), cell divergence (eq. 1) and the projection correction (Section 3,
// step 2).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "lk_device.h"

namespace lk {
namespace {

// Block id -> tile: workgroups are dispatched round-robin over the 8 XCDs, so
// consecutive ids land on different L2s.  Renumber so that each XCD receives a
// contiguous range of tiles (x fastest, then y, then z chunk): neighbouring tiles
// share their halo rows and overlap planes through the same L2.
__device__ __forceinline__ int xcd_tile(int bid, int nb) {
  constexpr int NX = 8;
  const int xcd = bid % NX, local = bid / NX;
  const int per = nb / NX, rem = nb % NX;
  return xcd < rem ? xcd * (per + 1) + local : rem * (per + 1) + (xcd - rem) * per + local;
}

// ------------------------------------------------------------------ momentum
// A row of L = 32 lanes owns 60 faces along x, two neighbouring ones per lane (its lanes hold
// i0 - 2 .. i0 + 61; the first and the last lane are halo); a wave is two rows, a block four waves
// on eight consecutive rows, marching along z over a chunk of planes.  (Grids whose faces fill 60 badly have rows of
// 16 or 8 lanes, 28 or 12 faces, and blocks of 16 or 32 rows: momentum_lanes.)  Every lane loads its pair of
// each of the six fields (a = U and b, components u, v, w) one plane ahead; the pairs reach the
// neighbouring rows through LDS, and the rows around the block are loaded by its waves in turn.
// Neighbours along x come from the neighbouring lane, and what two planes share is carried in
// registers.  Each momentum flux - viscous and convective together, in flux form - is formed
// once per lane: the edge product a b + b a at (x_i, y_j) serves the y flux of u and the x flux
// of v, and a lane hands a flux on instead of the four values it is made of.
// Positions outside a field's stored range hold the wall value of that position: 0 on
// wall-normal faces, beyond tangential walls 0 or, for the advected field of the nonlinear
// residual, the lid velocity at z = 1 (eq. 4).  With these ghosts the wall fluxes of the
// Laplacian ((first - wall)/half width) and the vanishing edge fluxes on walls follow from the
// interior formulas, so the compute has no wall branches.
// What bounds it: at 200^3 it moves 701 MB (502 read, where its two input fields are 386, and 200
// written; 119 us at the 5.9 TB/s that a kernel reading two fields and writing one reaches), issues about 60 us
// of vector instructions at two waves per SIMD, and its loads and stores take the address unit about 35
// us (16 cycles per load instruction of a CU whether a lane asks for 8 or 16 bytes, hence the pairs): 161 us
// by kernel trace.  Within a Krylov vector, by events on the stream (which add 2 to 3 us), against 16 x 8 tiles
// whose threads each took one face and all neighbours from LDS: 16^3 9-12 / 31 us, 64^3 15-17 / 29, 100^3 24-26 /
// 35, 150^3 70-73 / 85, 200^3 171-177 / 182, 256^3 315 / 360; 97 x 121 x 65 21-24 / 30.  Rows of 64 lanes leave
// more of them idle (150^3 85 us alone, 69 with 32); everything in registers with no LDS (8-byte loads of every
// neighbouring row) is bound by the address unit: 189 us at 200^3 with two rows per wave, 218 us with one, 153 here.

typedef double D2 __attribute__((ext_vector_type(2)));
typedef unsigned U2 __attribute__((ext_vector_type(2)));
typedef unsigned U4 __attribute__((ext_vector_type(4)));

// Each lane's pair to byte s2 past byte `so` of q and, where rows end with half a pair (`one`), its first
// value to byte s1; offsets past `bytes` (0: no store) store nothing.  A 16-byte store with a scalar register
// for its offset may still be reading its data when the next instruction overwrites it, and the compiler
// puts a wait state only behind those with a constant offset: seen on gfx950, where the second value
// of lanes 12 to 15 of every 16 now and then was the next instruction's result.  The s_nop has the data as its
// operand, so nothing overwrites it before.
__device__ __forceinline__ void store_pair(D2 x, double* q, unsigned bytes, unsigned s2, unsigned s1, bool one,
                                           unsigned so) {
  const __amdgpu_buffer_rsrc_t b = __builtin_amdgcn_make_buffer_rsrc(q, (short)0, (int)bytes, 0x00020000);
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(U4, x), b, (int)s2, (int)so, 0);
  asm volatile("s_nop 1" ::"v"(x) : "memory");
  if (one) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(U2, x.x), b, (int)s1, (int)so, 0);
}

// x of the next lower / higher position of a pair (undefined in the wave's first / last lane,
// whose results are halo).
template <int CTRL>
__device__ __forceinline__ double wave_shift(double x) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
  const unsigned lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xf, 0xf, true);
  const unsigned hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ D2 below(D2 x) { return D2{wave_shift<0x138>(x.y), x.x}; }
__device__ __forceinline__ D2 above(D2 x) { return D2{x.y, wave_shift<0x130>(x.x)}; }

// Lane l of a wave-wide register, as a wave-uniform value.
__device__ __forceinline__ double lane_value(double x, int l) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
  const unsigned lo = __builtin_amdgcn_readlane((int)(unsigned)b, l);
  const unsigned hi = __builtin_amdgcn_readlane((int)(unsigned)(b >> 32), l);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

__device__ __forceinline__ D2 fma2(D2 a, D2 b, D2 c) { return D2{fma(a.x, b.x, c.x), fma(a.y, b.y, c.y)}; }
__device__ __forceinline__ D2 fma2(double a, D2 b, D2 c) { return D2{fma(a, b.x, c.x), fma(a, b.y, c.y)}; }

constexpr int kMomWY = 4;         // waves per block
constexpr int kMomMaxChunk = 13;  // planes per chunk (at most 62: a lane each for its z metrics)
// of L lanes per row: faces along x per row, and rows per block
constexpr int mom_tx(int L) { return 2 * L - 4; }
constexpr int mom_ty(int L) { return kMomWY * 64 / L; }

template <bool LID, bool ODD, int L, bool WIDE = false>
__global__ void __launch_bounds__(64 * kMomWY, 2) k_momentum(GridDev g, const double* __restrict__ a,
                                                           const double* __restrict__ b, double* __restrict__ out,
                                                           double rre, double lid_u, double lid_v, int kchunk, int nbx,
                                                           int nby) {
  constexpr int TX = mom_tx(L), TY = mom_ty(L), NR = TY + 2;  // rows in LDS per field
  static_assert(L <= 32, "a load of the rows around the block holds one below and one above it");
  constexpr int NH = (6 + kMomWY - 1) / kMomWY;  // of those a wave's share of the six fields
  // plane in work: rows j0 - 1 .. j0 + TY of a (u, v, w) and b (u, v, w); one row nobody reads
  __shared__ D2 sm[(6 * NR + 1) * L];
  const int nx = g.x.n, ny = g.y.n, nz = g.z.n;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int bx = tile % nbx, by = (tile / nbx) % nby, bz = tile / (nbx * nby);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int sub = lane / L, li = lane % L, rb = wave * (64 / L) + sub;
  const int j0 = by * TY, j = j0 + rb;
  const int i = bx * TX + 2 * li - 2;  // the lane's faces are i and i + 1
  const int kb = bz * kchunk, ke = min(kb + kchunk, nz + 1);
  const size_t nu = (size_t)(nx + 1) * ny * nz, nv = (size_t)nx * (ny + 1) * nz;

  // Raw buffer accesses: a byte offset of the lane and row plus the wave-uniform one of the plane.  A
  // load at or past the given size returns 0 and a store there is dropped, so lanes without a
  // valid face take the offset kGhost and a plane outside the field the size 0: no access has a
  // branch.  A pair with one valid face never reaches past its component: wall rows of v and wall planes of w are not
  // loaded, and u's last entry of a row is a wall face.  The host keeps every component below
  // 2^31 bytes.
  constexpr unsigned kGhost = 1u << 31;
  const unsigned nbytes[3] = {(unsigned)(8 * nu), (unsigned)(8 * nv), (unsigned)(8 * (size_t)nx * ny * (nz + 1))};
  const size_t at[3] = {0, nu, nu + nv};
  auto buffer = [&](const double* p, int c, unsigned in) {  // raw buffer (stride 0), 32-bit data format
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(p + at[c]), (short)0, (int)(nbytes[c] & in),
                                             0x00020000);
  };
  const bool u0 = i > 0 && i < nx, u1 = i + 1 > 0 && i + 1 < nx;  // interior x-faces
  const bool c0 = i >= 0 && i < nx, c1 = i + 1 >= 0 && i + 1 < nx;  // cells
  const unsigned row[3] = {8u * (nx + 1), 8u * nx, 8u * nx};
  const unsigned plane[3] = {row[0] * ny, row[1] * (ny + 1), row[2] * ny};
  auto offset = [&](int c, int jj) {
    const bool in = (c == 0 ? (u0 || u1) : (c0 || c1)) && (c == 1 ? jj > 0 : jj >= 0) && jj < ny;
    return in ? jj * row[c] + 8u * i : kGhost;
  };
  auto load = [&](const double* p, int c, unsigned vo, int k) {
    const unsigned in = -(unsigned)((c == 2 ? k > 0 : k >= 0) & (k < nz) & (k <= ke));
    return __builtin_bit_cast(D2, __builtin_amdgcn_raw_buffer_load_b128(buffer(p, c, in), (int)vo,
                                                                        (int)((unsigned)k * plane[c] & in), 0));
  };
  auto mask = [&](D2 x, int c) { return D2{(c == 0 ? u0 : c0) ? x.x : 0.0, (c == 0 ? u1 : c1) ? x.y : 0.0}; };
  const unsigned ofs[3] = {offset(0, j), offset(1, j), offset(2, j)};

  // the rows around the block
  struct Halo {
    const double* p;
    unsigned bytes, plane, ofs;
    int k0, field, lds;  // first plane; field; position in LDS
    bool m0, m1;
  } halo[NH];
#pragma unroll
  for (int t = 0; t < NH; ++t) {
    const int e = wave * NH + t, f = min(e, 5), c = f % 3;
    const bool use = e < 6 && sub < 2;
    Halo& h = halo[t];
    h.p = (f < 3 ? a : b) + (c == 0 ? 0 : c == 1 ? nu : nu + nv);
    h.bytes = c == 0 ? nbytes[0] : c == 1 ? nbytes[1] : nbytes[2];
    h.plane = c == 0 ? plane[0] : c == 1 ? plane[1] : plane[2];
    h.ofs = use ? offset(c, sub ? j0 + TY : j0 - 1) : kGhost;
    h.k0 = c == 2 ? 1 : 0;
    h.field = f;
    h.lds = (use ? f * NR + (sub ? TY + 1 : 0) : 6 * NR) * L + li;
    h.m0 = c == 0 ? u0 : c0;
    h.m1 = c == 0 ? u1 : c1;
  }
  auto hload = [&](const Halo& h, int k) {
    const unsigned in = -(unsigned)((k >= h.k0) & (k < nz) & (k <= ke));
    const __amdgpu_buffer_rsrc_t r =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(h.p), (short)0, (int)(h.bytes & in), 0x00020000);
    return __builtin_bit_cast(
        D2, __builtin_amdgcn_raw_buffer_load_b128(r, (int)h.ofs, (int)((unsigned)k * h.plane & in), 0));
  };

  // metrics: of the lane (x, y: fixed) and of the plane (z: lane l holds those of plane kb - 1 + l,
  // read back without a wait on memory)
  D2 thx, rdx, rddx;
  {
    auto xc = [&](int q) { return max(0, min(q, nx - 1)); };
    auto xf = [&](int q) { return max(0, min(q, nx)); };
    thx = D2{g.x.th[xf(i)], g.x.th[xf(i + 1)]};
    rdx = D2{g.x.rd[xc(i)], g.x.rd[xc(i + 1)]};
    rddx = D2{g.x.rdd[xf(i)], g.x.rdd[xf(i + 1)]};
  }
  const int jc = max(0, min(j, ny - 1)), jf = max(0, min(j, ny)), jf1 = min(jf + 1, ny);
  const double thy0 = g.y.th[jf], thy1 = g.y.th[jf1], rddy0 = g.y.rdd[jf], rddy1 = g.y.rdd[jf1];
  const double rdy0 = g.y.rd[max(jc - 1, 0)], rdy1 = g.y.rd[jc];
  const int zl = kb - 1 + lane, zc = max(0, min(zl, nz - 1)), zf = max(0, min(zl, nz));
  const double zth = g.z.th[zf], zrd = g.z.rd[zc], zrdd = g.z.rdd[zf];

  // stores: whole pairs, and the single face that ends a row of odd length (u's for even nx,
  // v's and w's for odd nx)
  const bool own = li >= 1 && li <= TX / 2;
  auto store_offset = [&](int c, bool whole) {
    const int n = c == 0 ? nx + 1 : nx;
    const bool in = own && i < n && (i + 1 < n) == whole && (c == 1 ? j <= ny : j < ny);
    return in ? j * row[c] + 8u * i : kGhost;
  };
  const unsigned sto[3] = {store_offset(0, true), store_offset(1, true), store_offset(2, true)};
  const unsigned sto1[3] = {store_offset(0, false), store_offset(1, false), store_offset(2, false)};
  auto put = [&](D2 x, int c, int k, bool in) {
    const unsigned m = -(unsigned)in;
    store_pair(x, out + (c == 0 ? 0 : c == 1 ? nu : nu + nv), nbytes[c] & m, sto[c], sto1[c], (c == 0) != ODD,
               (unsigned)k * plane[c] & m);
  };

  // carried from the plane below: own values (and v of the row above), z fluxes, and what the
  // faces have so far
  D2 ou[2], ov[2], ot[2], ow[2];
  D2 tuz = 0.0, tvz = 0.0, twz = 0.0, su = 0.0, sv = 0.0, sw = 0.0;
  // (the advecting field is scaled by Re, and by 1/2 for the residual, as it is read: the fluxes are
  // then Re times the momentum's and the sums are divided by Re as they are stored.  WIDE scales the viscous parts
  // instead, for Reynolds numbers whose products would leave the range of the type.)
  const double sa = (LID ? 0.5 : 1.0) / (WIDE ? 1.0 : rre), so = WIDE ? 1.0 : rre;
  auto flux = [&](auto m, D2 db, D2 e) {  // viscous part m db less the convective part e
    if constexpr (WIDE) m *= rre;
    return fma2(m, db, -e);
  };
  const unsigned ofst = offset(1, j + 1);
#pragma unroll
  for (int f = 0; f < 2; ++f) {
    const double* p = f ? b : a;
    const double q = f ? 1.0 : sa;
    ou[f] = q * mask(load(p, 0, ofs[0], kb - 1), 0);
    ov[f] = q * mask(load(p, 1, ofs[1], kb - 1), 1);
    ot[f] = q * mask(load(p, 1, ofst, kb - 1), 1);
    ow[f] = q * mask(load(p, 2, ofs[2], kb - 1), 2);
  }
  D2 N[6], H[NH];
  auto fetch = [&](int k) {
#pragma unroll
    for (int f = 0; f < 6; ++f) N[f] = load(f < 3 ? a : b, f % 3, ofs[f % 3], k);
#pragma unroll
    for (int t = 0; t < NH; ++t) H[t] = hload(halo[t], k);
  };
  auto row_at = [&](int f, int r) { return sm[(f * NR + rb + r) * L + li]; };  // row j - 1 + r of the plane in work
  fetch(kb);
  // A plane's results wait in registers until the next stage has its input, and are stored ahead of its
  // loads: memory operations complete in order, so a store behind the loads would be waited for
  // with them at once.
  D2 res[3] = {0.0, 0.0, 0.0};
  auto flush = [&](int k) {  // plane k's, k < ke; none before the first
    put(res[0], 0, k, k >= kb && k < nz);
    put(res[1], 1, k, k >= kb && k < nz);
    put(res[2], 2, k, k >= kb);
  };
  for (int k = kb; k <= ke; ++k) {
    D2 O[6];
#pragma unroll
    for (int f = 0; f < 6; ++f) {
      O[f] = mask(N[f], f % 3);
      if (f < 3) O[f] *= sa;
    }
    D2 h[NH];
#pragma unroll
    for (int t = 0; t < NH; ++t) {
      h[t] = D2{halo[t].m0 ? H[t].x : 0.0, halo[t].m1 ? H[t].y : 0.0};
      h[t] *= halo[t].field < 3 ? sa : 1.0;
    }
    if (LID && k == nz) {  // the advected field carries the lid velocity above z = 1
      if (j < ny) O[3] = D2{u0 ? lid_u : 0.0, u1 ? lid_u : 0.0};
      if (j > 0 && j < ny) O[4] = D2{c0 ? lid_v : 0.0, c1 ? lid_v : 0.0};
#pragma unroll
      for (int t = 0; t < NH; ++t)
        if ((halo[t].field == 3 || halo[t].field == 4) && halo[t].ofs != kGhost) {
          const double x = halo[t].field == 3 ? lid_u : lid_v;
          h[t] = D2{halo[t].m0 ? x : 0.0, halo[t].m1 ? x : 0.0};
        }
    }
#pragma unroll
    for (int f = 0; f < 6; ++f) sm[(f * NR + rb + 1) * L + li] = O[f];
#pragma unroll
    for (int t = 0; t < NH; ++t) sm[halo[t].lds] = h[t];
    flush(k - 2);
    fetch(k + 1);
    __syncthreads();

    const int l = k - kb + 1;
    const double thz = lane_value(zth, l), rddz = lane_value(zrdd, l);
    const double rdzm = lane_value(zrd, l - 1), rddzm = lane_value(zrdd, l - 1);
    D2 nsw;
    {  // edges (x_i, z_k): z flux of u, x flux of w
      const D2 aw0 = below(O[2]), bw0 = below(O[5]);
      const D2 dbw = O[5] - bw0, dbu = O[3] - ou[1];
      const D2 aw = fma2(thx, O[2] - aw0, aw0), bw = fma2(thx, dbw, bw0);
      const D2 au = fma2(thz, O[0] - ou[0], ou[0]), bu = fma2(thz, dbu, ou[1]);
      const D2 e = fma2(aw, bu, bw * au);
      const D2 tz = flux(rddz, dbu, e), tx = flux(rddx, dbw, e);
      nsw = (above(tx) - tx) * rdx;
      const D2 val = fma2(rdzm, tz - tuz, su);
      res[0] = D2{u0 ? so * val.x : 0.0, u1 ? so * val.y : 0.0};
      tuz = tz;
    }
    {  // edges (y_j, z_k) and (y_{j+1}, z_k): z flux of v, y flux of w
      const D2 aw0 = row_at(2, 0), bw0 = row_at(5, 0);
      const D2 dbw = O[5] - bw0, dbv = O[4] - ov[1];
      const D2 aw = fma2(thy0, O[2] - aw0, aw0), bw = fma2(thy0, dbw, bw0);
      const D2 av = fma2(thz, O[1] - ov[0], ov[0]), bv = fma2(thz, dbv, ov[1]);
      const D2 e = fma2(aw, bv, bw * av);
      const D2 tz = flux(rddz, dbv, e);
      nsw = fma2(-rdy1, flux(rddy0, dbw, e), nsw);
      const D2 val = fma2(rdzm, tz - tvz, sv);
      res[1] = j > 0 && j < ny ? so * val : D2{0.0, 0.0};
      tvz = tz;
    }
    {
      const D2 aw1 = row_at(2, 2), bw1 = row_at(5, 2);
      const D2 av1 = row_at(1, 2), bv1 = row_at(4, 2);
      const D2 dbw = bw1 - O[5];
      const D2 aw = fma2(thy1, aw1 - O[2], O[2]), bw = fma2(thy1, dbw, O[5]);
      const D2 av = fma2(thz, av1 - ot[0], ot[0]), bv = fma2(thz, bv1 - ot[1], ot[1]);
      const D2 e = fma2(aw, bv, bw * av);
      nsw = fma2(rdy1, flux(rddy1, dbw, e), nsw);
      ot[0] = av1;
      ot[1] = bv1;
    }
    {  // centre of cell k - 1: z flux of w
      const D2 aw = ow[0] + O[2], bw = ow[1] + O[5];
      const D2 tz = flux(rdzm, O[5] - ow[1], (0.5 * aw) * bw);
      res[2] = k > 1 && k <= nz ? so * fma2(rddzm, tz - twz, sw) : D2{0.0, 0.0};
      twz = tz;
      sw = nsw;
    }
    {  // centres along x
      const D2 au1 = above(O[0]), bu1 = above(O[3]);
      const D2 au = O[0] + au1, bu = O[3] + bu1;
      const D2 t = flux(rdx, bu1 - O[3], (0.5 * au) * bu);
      su = (t - below(t)) * rddx;
    }
    {  // edges (x_i, y_j) and (x_i, y_{j+1}): y flux of u, x flux of v
      const D2 au0 = row_at(0, 0), bu0 = row_at(3, 0);
      const D2 av0 = below(O[1]), bv0 = below(O[4]);
      const D2 dbv = O[4] - bv0, dbu = O[3] - bu0;
      const D2 av = fma2(thx, O[1] - av0, av0), bv = fma2(thx, dbv, bv0);
      const D2 au = fma2(thy0, O[0] - au0, au0), bu = fma2(thy0, dbu, bu0);
      const D2 e = fma2(av, bu, bv * au);
      const D2 tx = flux(rddx, dbv, e);
      su = fma2(-rdy1, flux(rddy0, dbu, e), su);
      sv = (above(tx) - tx) * rdx;
    }
    {
      const D2 au1 = row_at(0, 2), bu1 = row_at(3, 2);
      const D2 av0 = below(ot[0]), bv0 = below(ot[1]);
      const D2 dbu = bu1 - O[3];
      const D2 av = fma2(thx, ot[0] - av0, av0), bv = fma2(thx, ot[1] - bv0, bv0);
      const D2 au = fma2(thy1, au1 - O[0], O[0]), bu = fma2(thy1, dbu, O[3]);
      const D2 e = fma2(av, bu, bv * au);
      su = fma2(rdy1, flux(rddy1, dbu, e), su);
    }
    {  // centres along y
      const D2 avm = row_at(1, 0), bvm = row_at(4, 0);
      const D2 tm = flux(rdy0, O[4] - bvm, (0.5 * (avm + O[1])) * (bvm + O[4]));
      const D2 tp = flux(rdy1, ot[1] - O[4], (0.5 * (O[1] + ot[0])) * (O[4] + ot[1]));
      sv = fma2(rddy0, tp - tm, sv);
    }
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      ou[f] = O[3 * f];
      ov[f] = O[3 * f + 1];
      ow[f] = O[3 * f + 2];
    }
    __syncthreads();
  }
  flush(ke - 1);
}

// ---------------------------------------------------------------- divergence
// One thread per (i, j) column of cells marching over KZ planes, so the w face
// between two cells is read once (carried in a register); tiles are grouped per XCD.
constexpr int kDivTX = 64, kDivTY = 4, kDivKZ = 4;

template <int KZ>
__global__ void __launch_bounds__(kDivTX* kDivTY) k_divergence(GridDev g, Vel V, double* __restrict__ r,
                                                               double* __restrict__ partials, int nbx, int nby) {
  const int nx = g.x.n, ny = g.y.n, nz = g.z.n;
  const int t = xcd_tile(blockIdx.x, gridDim.x);
  const int i = (t % nbx) * kDivTX + (int)(threadIdx.x % kDivTX);
  const int j = ((t / nbx) % nby) * kDivTY + (int)(threadIdx.x / kDivTX);
  const int k0 = (t / (nbx * nby)) * KZ, k1 = min(k0 + KZ, nz);
  double contrib = 0.0;
  if (i < nx && j < ny) {
    const double rdx = g.x.rd[i], rdy = g.y.rd[j], dxy = g.x.d[i] * g.y.d[j];
    double wlo = V.W(k0, j, i);
    for (int k = k0; k < k1; ++k) {
      const double whi = V.W(k + 1, j, i);
      // (the order of the sum is that of k_correct_div)
      const double dv = fma(g.z.rd[k], whi - wlo, fma(rdy, V.V(k, j + 1, i) - V.V(k, j, i),
                                                      (V.U(k, j, i + 1) - V.U(k, j, i)) * rdx));
      if (r) r[((size_t)k * ny + j) * nx + i] = dv;
      contrib += dxy * g.z.d[k] * dv * dv;
      wlo = whi;
    }
  }
  if (partials) {
    const double s = block_sum(contrib);
    if (threadIdx.x == 0) partials[blockIdx.x] = s;
  }
}

// ---------------------------------------------------------------- correction
// One thread per (i, j) face column marching over KZ planes (phi of the plane
// below carried in a register); tiles grouped per XCD.
constexpr int kCdMaxChunk = 8;
constexpr int kCorTX = 64, kCorTY = 4, kCorKZ = 2;

template <int KZ>
__global__ void __launch_bounds__(kCorTX* kCorTY) k_correct(GridDev g, const double* __restrict__ w,
                                                            const double* __restrict__ phi, double* __restrict__ v,
                                                            double* __restrict__ p, int accumulate, int nbx, int nby) {
  const int nx = g.x.n, ny = g.y.n, nz = g.z.n;
  const int t = xcd_tile(blockIdx.x, gridDim.x);
  const int i = (t % nbx) * kCorTX + (int)(threadIdx.x % kCorTX);
  const int j = ((t / nbx) % nby) * kCorTY + (int)(threadIdx.x / kCorTX);
  const int k0 = (t / (nbx * nby)) * KZ, k1 = min(k0 + KZ, nz + 1);
  if (i > nx || j > ny) return;
  const Idx I{nx, ny, nz};
  const size_t nu = (size_t)(nx + 1) * ny * nz, nv = (size_t)nx * (ny + 1) * nz;
  const double* src = accumulate ? v : w;
  // branch-free loads: in-range clamped cell indices, wall faces selected to 0
  const int ic = min(i, nx - 1), jc = min(j, ny - 1);
  const double rddx = g.x.rdd[i], rddy = g.y.rdd[j];
  double pb = phi[I.c(max(k0 - 1, 0), jc, ic)];  // phi below the first plane
  for (int k = k0; k < k1; ++k) {
    // every load of the plane from an in-range (clamped) position, before any store, so
    // that they are in flight together; only the stores depend on the face being stored
    const int kc = min(k, nz - 1);
    const double pc = phi[I.c(kc, jc, ic)];
    const double pw = phi[I.c(kc, jc, max(ic - 1, 0))], ps = phi[I.c(kc, max(jc - 1, 0), ic)];
    const size_t qu = I.u(kc, jc, i), qv = nu + I.v(kc, j, ic), qw = nu + nv + I.w(k, jc, ic);
    const double su = src[qu], sv = src[qv], sw = src[qw];
    const double pold = (p && accumulate) ? p[I.c(kc, jc, ic)] : 0.0;
    if (j < ny && k < nz) {
      const bool in = (i > 0) & (i < nx);
      const double val = su - (pc - pw) * rddx;
      v[qu] = in ? val : 0.0;
    }
    if (i < nx && k < nz) {
      const bool in = (j > 0) & (j < ny);
      const double val = sv - (pc - ps) * rddy;
      v[qv] = in ? val : 0.0;
    }
    if (i < nx && j < ny) {
      const bool in = (k > 0) & (k < nz);
      const double val = sw - (pc - pb) * g.z.rdd[k];
      v[qw] = in ? val : 0.0;
      if (p && k < nz) p[I.c(k, j, i)] = accumulate ? pold + pc : pc;
    }
    pb = pc;
  }
}

// --------------------------------------------- correction with its certificate
// The first pass of a projection: v = w - G phi, p = phi, and D v with the partial sums of V (D v)^2, in one
// kernel.  The rows, lanes and pairs of the momentum stencil: a lane corrects its pair of u, v and w faces,
// and the faces its cells share with others - u of the next lane, v of the next row, w of the next
// plane - are corrected again with the same operations on the same values (the input is not the
// output), so D v is that of the stored field to the bit and no value passes between waves.  A
// block marches over a chunk of planes with the next plane's loads in flight.
// HBM bound: 2 F_u + 2 F_p, 514 MB at 200^3, where a separate certificate read v again (193 MB).
// 200^3: 116 us by kernel trace (518 MB, 4.5 TB/s); by events on the stream 124 against 109 + 56 for the two
// kernels; 100^3 17 / 14 + 9; 256^3 248 / 226 + 103; 97 x 121 x 65 15 / 12 + 9.
constexpr int kCdL = 32;  // lanes per row
template <bool ODD>
__global__ void __launch_bounds__(64 * kMomWY, 4) k_correct_div(GridDev g, const double* __restrict__ w,
                                                                const double* __restrict__ phi,
                                                                double* __restrict__ v, double* __restrict__ p,
                                                                double* __restrict__ r, double* __restrict__ partials,
                                                                int kchunk, int nbx, int nby) {
  constexpr int L = kCdL, TX = mom_tx(L), TY = mom_ty(L);
  constexpr unsigned kGhost = 1u << 31;
  const int nx = g.x.n, ny = g.y.n, nz = g.z.n;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int bx = tile % nbx, by = (tile / nbx) % nby, bz = tile / (nbx * nby);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane % L, j = by * TY + wave * (64 / L) + lane / L;
  const int i = bx * TX + 2 * li - 2;  // the lane's faces and cells are i and i + 1
  const int kb = bz * kchunk, ke = min(kb + kchunk, nz);
  const size_t nu = (size_t)(nx + 1) * ny * nz, nv = (size_t)nx * (ny + 1) * nz, nc = (size_t)nx * ny * nz;
  const unsigned ubytes = (unsigned)(8 * nu), vbytes = (unsigned)(8 * nv), wbytes = (unsigned)(8 * (nc + (size_t)nx * ny));
  const unsigned cbytes = (unsigned)(8 * nc);
  auto buffer = [&](const double* q, unsigned bytes, unsigned in) {  // raw buffer (stride 0), 32-bit data format
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(q), (short)0, (int)(bytes & in), 0x00020000);
  };
  const bool u0 = i > 0 && i < nx, u1 = i + 1 > 0 && i + 1 < nx;
  const bool c0 = i >= 0 && i < nx, c1 = i + 1 >= 0 && i + 1 < nx;
  const bool row = j < ny, own = li >= 1 && li <= TX / 2;
  const unsigned urow = 8u * (nx + 1), crow = 8u * nx;
  const unsigned uplane = urow * ny, vplane = crow * (ny + 1), cplane = crow * ny;
  auto at = [&](bool in, int jj, unsigned rb) { return in ? jj * rb + 8u * i : kGhost; };
  const bool c = c0 || c1;
  const unsigned lu = at((u0 || u1) && row, j, urow), lv0 = at(c && j > 0 && row, j, crow), lv1 = at(c && j + 1 < ny, j + 1, crow);
  const unsigned lc = at(c && row, j, crow), lcm = at(c && j > 0 && row, j - 1, crow), lcp = at(c && j + 1 < ny, j + 1, crow);
  // whole pairs, and the single entry that ends a row of odd length
  auto whole = [&](int n) { return own && i + 1 < n; };
  auto half = [&](int n) { return own && i + 1 == n; };
  const unsigned su = at(whole(nx + 1) && row, j, urow), su1 = at(half(nx + 1) && row, j, urow);
  const unsigned sv = at(whole(nx) && j <= ny, j, crow), sv1 = at(half(nx) && j <= ny, j, crow);
  const unsigned sc = at(whole(nx) && row, j, crow), sc1 = at(half(nx) && row, j, crow);
  struct Plane {
    D2 p0, pm, pp, u, v0, v1, w;
  };
  auto get = [&](const __amdgpu_buffer_rsrc_t& b, unsigned ofs, unsigned so) {
    return __builtin_bit_cast(D2, __builtin_amdgcn_raw_buffer_load_b128(b, (int)ofs, (int)so, 0));
  };
  auto fetch = [&](Plane& P, int k) {
    // cells and the faces u, v of plane k < ke; w and the phi it needs also on the level ke
    const unsigned in = -(unsigned)(k < ke), inp = -(unsigned)((k <= ke) & (k < nz)),
                   inw = -(unsigned)((k <= ke) & (k > 0) & (k < nz));
    // (phi is followed by at least one more value: a half pair reads past its last one)
    const __amdgpu_buffer_rsrc_t bp = buffer(phi, cbytes + 8, inp), bq = buffer(phi, cbytes + 8, in),
                                 bv = buffer(w + nu, vbytes, in);
    P.p0 = get(bp, lc, (unsigned)k * cplane & inp);
    P.pm = get(bq, lcm, (unsigned)k * cplane & in);
    P.pp = get(bq, lcp, (unsigned)k * cplane & in);
    P.u = get(buffer(w, ubytes, in), lu, (unsigned)k * uplane & in);
    P.v0 = get(bv, lv0, (unsigned)k * vplane & in);
    P.v1 = get(bv, lv1, (unsigned)k * vplane & in);
    P.w = get(buffer(w + nu + nv, wbytes, inw), lc, (unsigned)k * cplane & inw);
  };
  auto put = [&](D2 x, double* q, unsigned bytes, unsigned plane, unsigned s2, unsigned s1, bool one, int k, bool in) {
    const unsigned m = -(unsigned)in;
    store_pair(x, q, bytes & m, s2, s1, one, (unsigned)k * plane & m);
  };
  Plane N;
  fetch(N, kb);
  // phi below the first plane; metrics
  const unsigned inb = -(unsigned)(kb > 0);
  D2 pb = get(buffer(phi, cbytes + 8, inb), lc, (unsigned)(kb - 1) * cplane & inb);
  const int ic = max(0, min(i, nx - 1)), ic1 = max(0, min(i + 1, nx - 1)), xf = max(0, min(i, nx)), xf1 = max(0, min(i + 1, nx));
  const D2 rdx = {g.x.rd[ic], g.x.rd[ic1]}, rddx = {g.x.rdd[xf], g.x.rdd[xf1]};
  const int jc = min(j, ny - 1), jf = min(j, ny), jf1 = min(j + 1, ny);
  const double rdy = g.y.rd[jc], rddy0 = g.y.rdd[jf], rddy1 = g.y.rdd[jf1];
  const bool cell = own && row;
  const D2 dxy = {cell && c0 ? g.x.d[ic] * g.y.d[jc] : 0.0, cell && c1 ? g.x.d[ic1] * g.y.d[jc] : 0.0};
  const int zl = min(kb + lane, nz);
  const double zrd = g.z.rd[min(zl, nz - 1)], zd = g.z.d[min(zl, nz - 1)], zrdd = g.z.rdd[zl];
  double sum = 0.0;
  D2 s = 0.0, wp = 0.0;
  for (int k = kb; k <= ke; ++k) {
    const Plane P = N;
    fetch(N, k + 1);
    const int l = k - kb;
    // w on the level z_k, and with it the divergence of the cells below
    const bool wi = k > 0 && k < nz;
    const D2 dw = P.p0 - pb;
    const double rddz = lane_value(zrdd, l);
    const D2 wk = {wi && c0 ? fma(-dw.x, rddz, P.w.x) : 0.0, wi && c1 ? fma(-dw.y, rddz, P.w.y) : 0.0};
    put(wk, v + nu + nv, wbytes, cplane, sc, sc1, ODD, k, (k < ke) | (k == nz));
    const double rdz = lane_value(zrd, max(l - 1, 0)), dz = lane_value(zd, max(l - 1, 0));
    const D2 dv = fma2(rdz, wk - wp, s);
    const double t = dz * fma(dxy.x * dv.x, dv.x, dxy.y * dv.y * dv.y);
    sum += k > kb ? t : 0.0;
    put(dv, r, r ? cbytes : 0, cplane, sc, sc1, ODD, k - 1, k > kb);
    // u, v and p of plane k
    const D2 du = P.p0 - below(P.p0), d0 = P.p0 - P.pm, d1 = P.pp - P.p0;
    const D2 u = {u0 ? fma(-du.x, rddx.x, P.u.x) : 0.0, u1 ? fma(-du.y, rddx.y, P.u.y) : 0.0};
    const bool vi = j > 0 && j < ny, vi1 = j + 1 < ny;
    const D2 v0 = {vi && c0 ? fma(-d0.x, rddy0, P.v0.x) : 0.0, vi && c1 ? fma(-d0.y, rddy0, P.v0.y) : 0.0};
    const D2 v1 = {vi1 && c0 ? fma(-d1.x, rddy1, P.v1.x) : 0.0, vi1 && c1 ? fma(-d1.y, rddy1, P.v1.y) : 0.0};
    put(u, v, ubytes, uplane, su, su1, !ODD, k, k < ke);
    put(v0, v + nu, vbytes, vplane, sv, sv1, ODD, k, k < ke);
    put(P.p0, p, p ? cbytes : 0, cplane, sc, sc1, ODD, k, k < ke);
    s = fma2(rdy, v1 - v0, (above(u) - u) * rdx);
    wp = wk;
    pb = P.p0;
  }
  const double total = block_sum(sum);
  if (threadIdx.x == 0) partials[blockIdx.x] = total;
}

}  // namespace

// ==================================================================== launchers
// Momentum stencil: the nz + 1 planes are split into chunks, one per block.  Two blocks fit a CU
// (registers), so up to kMomSlots run at once; the number of chunks is the one whose rounds of
// blocks, each as long as a chunk's planes and its start-up, end soonest.  Chunks stay short
// because neighbouring blocks then read their common rows and planes at about the same time, from
// the L2 (the stencil alone): at 256^3 13 planes 283 us, 16 to 20 292-304 us, 34 323 us; at 200^3 12 to 20 150-155 us,
// 34 177 us.
// Small grids take chunks down to one plane (16^3 6.8 us, three planes 10.6; 64^3 14.1 / 15.9).
constexpr int kMomSlots = 512;

int momentum_chunk(int nx, int ny, int nz, int L) {
  const long tiles = (long)blocks_for(nx + 1, mom_tx(L)) * blocks_for(ny + 1, mom_ty(L));
  int best = 0;
  double least = 0.0;
  for (int most = kMomMaxChunk; most >= 1; --most) {
    const int planes = (int)blocks_for(nz + 1, blocks_for(nz + 1, most));  // chunks of equal length
    const long rounds = blocks_for((size_t)tiles * blocks_for(nz + 1, planes), kMomSlots);
    const double cost = rounds * (planes + 2.5);
    if (!best || cost < least) best = planes, least = cost;
  }
  return best;
}

// Lanes per row of the stencil: those whose rows have the fewest lanes over nx + 1 faces, if that is 15 % (16 lanes)
// or 20 % (8) fewer than with the longer rows, whose halo is less: 32 / 16 / 8 lanes with (y, z) = 256^2: nx = 11 49 / 29 / 21
// us, 15 49 / 29 / 31, 27 51 / 32 / 45, 31 51 / 51 / 46, 36 52 / 53 / 57; 64^3 15.6 / 14.1 / 16.0, 70 x 200^2 61 / 51 / 55,
// 128^3 38.9 / 37.6; with nearly as many lanes, 240 x 200^2 184 / 187, and as many, 200^3 157 / 165.
static int momentum_lanes(int nx) {
  auto lanes = [&](int L) { return (int)blocks_for(nx + 1, mom_tx(L)) * L; };
  int best = 32;
  if (lanes(16) * 115 < lanes(32) * 100) best = 16;
  if (lanes(8) * 120 < lanes(best) * 100) best = 8;
  return best;
}

hipError_t launch_momentum(const GridDev& g, const double* a, const double* b, double* out, double rre, bool lid,
                           double lid_u, double lid_v, hipStream_t st) {
  const int nx = g.x.n, ny = g.y.n, nz = g.z.n;
  const VelLayout V = vel_layout(nx, ny, nz);
  if (8 * std::max(V.nu, std::max(V.nv, V.nw)) >= (size_t(1) << 31)) return hipErrorInvalidValue;
  // far from any flow, but accepted: nothing may overflow that the formula itself does not let overflow
  const bool wide = !(rre > 0x1p-256 && rre < 0x1p256);
  const int L = wide ? 32 : momentum_lanes(nx);
  const int nbx = (int)blocks_for(nx + 1, mom_tx(L)), nby = (int)blocks_for(ny + 1, mom_ty(L));
  const int kchunk = momentum_chunk(nx, ny, nz, L);
  const dim3 grid(nbx * nby * blocks_for(nz + 1, kchunk)), block(64 * kMomWY);
  auto run = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, block, 0, st, g, a, b, out, rre, lid_u, lid_v, kchunk, nbx, nby);
    return hipGetLastError();
  };
  auto rows = [&](auto LID, auto ODD) {
    if (wide) return run(k_momentum<LID.value, ODD.value, 32, true>);
    if (L == 8) return run(k_momentum<LID.value, ODD.value, 8>);
    if (L == 16) return run(k_momentum<LID.value, ODD.value, 16>);
    return run(k_momentum<LID.value, ODD.value, 32>);
  };
  const std::true_type yes;
  const std::false_type no;
  if (lid) return nx & 1 ? rows(yes, yes) : rows(yes, no);
  return nx & 1 ? rows(no, yes) : rows(no, no);
}

int divergence_parts(int nx, int ny, int nz) {
  return (int)(blocks_for(nx, kDivTX) * blocks_for(ny, kDivTY) * blocks_for(nz, kDivKZ));
}

hipError_t launch_divergence(const GridDev& g, const double* v, double* r, double* partials, hipStream_t st) {
  const int nx = g.x.n, ny = g.y.n, nz = g.z.n;
  const VelLayout L = vel_layout(nx, ny, nz);
  Vel V{v, v + L.ov(), v + L.ow(), Idx{nx, ny, nz}};
  const int nbx = (int)blocks_for(nx, kDivTX), nby = (int)blocks_for(ny, kDivTY);
  const unsigned nb = (unsigned)divergence_parts(nx, ny, nz);
  hipLaunchKernelGGL(k_divergence<kDivKZ>, dim3(nb), dim3(kDivTX * kDivTY), 0, st, g, V, r, partials, nbx, nby);
  return hipGetLastError();
}

hipError_t launch_correct(const GridDev& g, const double* w, const double* phi, double* v, double* p,
                          bool accumulate, hipStream_t st) {
  const int nx = g.x.n, ny = g.y.n, nz = g.z.n;
  const int nbx = (int)blocks_for(nx + 1, kCorTX), nby = (int)blocks_for(ny + 1, kCorTY);
  const unsigned nb = (unsigned)(nbx * nby * (int)blocks_for(nz + 1, kCorKZ));
  hipLaunchKernelGGL(k_correct<kCorKZ>, dim3(nb), dim3(kCorTX * kCorTY), 0, st, g, w, phi, v, p, accumulate ? 1 : 0, nbx,
                     nby);
  return hipGetLastError();
}

// Planes per chunk of k_correct_div: a chunk reads one level of phi and w more than its planes, and
// longer chunks read what neighbouring blocks share at more different times (by events, 200^3: 5 planes
// 131 us, 8 130 us, 16 and 25 142 us; 256^3 253 / 251 / 259 / 285).  Grids that would not fill the chip
// with chunks of eight (four blocks per CU, 2 kMomSlots) take shorter ones.
static int correct_chunk(int nx, int ny, int nz) {
  const long tiles = (long)blocks_for(nx + 1, mom_tx(kCdL)) * blocks_for(ny + 1, mom_ty(kCdL));
  const long most = std::max<long>(1, 2 * kMomSlots / tiles);
  return (int)std::min<long>(kCdMaxChunk, std::max<long>(1, blocks_for(nz, (unsigned)most)));
}

int correct_div_parts(int nx, int ny, int nz) {
  return (int)(blocks_for(nx + 1, mom_tx(kCdL)) * blocks_for(ny + 1, mom_ty(kCdL)) * blocks_for(nz, correct_chunk(nx, ny, nz)));
}

hipError_t launch_correct_div(const GridDev& g, const double* w, const double* phi, double* v, double* p, double* r,
                              double* partials, hipStream_t st) {
  const int nx = g.x.n, ny = g.y.n, nz = g.z.n;
  const int nbx = (int)blocks_for(nx + 1, mom_tx(kCdL)), nby = (int)blocks_for(ny + 1, mom_ty(kCdL));
  const dim3 grid((unsigned)correct_div_parts(nx, ny, nz)), block(64 * kMomWY);
  const int kchunk = correct_chunk(nx, ny, nz);
  if (nx & 1)
    hipLaunchKernelGGL(k_correct_div<true>, grid, block, 0, st, g, w, phi, v, p, r, partials, kchunk, nbx, nby);
  else
    hipLaunchKernelGGL(k_correct_div<false>, grid, block, 0, st, g, w, phi, v, p, r, partials, kchunk, nbx, nby);
  return hipGetLastError();
}

}  // namespace lk
