// C ABI of lidkrylov: context, grid, stencils, Poisson solve, SIMPLE projection.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <functional>
#include <string>
#include <vector>

#include "lk_ctx.h"
#include "lk_internal.h"
#include "lk_linalg.h"
#include "lk_lines.h"
#include "lk_modes.h"

using namespace lk;

namespace {
std::string g_create_error;
}  // namespace

namespace lk {

int fail(lc_ctx* c, int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  if (c) c->err = buf;
  else g_create_error = buf;
  return code;
}



hipEvent_t take_event(lc_ctx* c) {
  if (c->ev_used < c->ev_pool.size()) return c->ev_pool[c->ev_used++];
  hipEvent_t e = nullptr;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  c->ev_pool.push_back(e);
  c->ev_used++;
  return e;
}



constexpr size_t kArenaAlign = 256;

size_t arena_next(const lc_ctx* c) { return (c->arena_used + kArenaAlign - 1) / kArenaAlign * kArenaAlign; }

hipError_t ctx_alloc(lc_ctx* c, void** p, size_t bytes) {
  if (c->dry) {
    *p = nullptr;
    c->arena_used = arena_next(c) + bytes;
    return hipSuccess;
  }
  if (!c->arena) return hipMalloc(p, bytes);
  const size_t at = arena_next(c);
  if (at + bytes > c->arena_size) return hipErrorOutOfMemory;
  *p = c->arena + at;
  c->arena_used = at + bytes;
  return hipSuccess;
}

int krylov_ws(lc_ctx* c, int nvec, double** p, long* ld) {
  *ld = ((long)c->nvel + 63) / 64 * 64;
  const size_t need = (size_t)nvec * *ld;
  if (need > c->kws_n) {
    if (c->arena)
      return fail(c, LC_ENOMEM, "workspace too small: %d Krylov vectors need %zu bytes, %zu remain", nvec,
                  need * sizeof(double), c->kws_n * sizeof(double));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    if (c->kws) (void)hipFree(c->kws);
    c->kws = nullptr;
    c->kws_n = 0;
    if (hipMalloc((void**)&c->kws, need * sizeof(double)) != hipSuccess)
      return fail(c, LC_ENOMEM, "cannot allocate %d Krylov vectors (%.1f GB)", nvec, need * 8e-9);
    c->kws_n = need;
  }
  *p = c->kws;
  return LC_OK;
}

// What a watched sum's place holds until the device has written it: a NaN that no arithmetic makes.
constexpr uint64_t kUnset = 0x7ff8a5c3e1d2b497ull;

double now_ms() {
  using namespace std::chrono;
  return duration<double, std::milli>(steady_clock::now().time_since_epoch()).count();
}

double* terms_of(const lc_ctx* c, int slot) { return c->hsum + kSumSlots + (size_t)slot * kHostParts; }

// Where the terms of slot `slot` go: to the host when it adds them itself, else to the device scratch.
double* parts_of(lc_ctx* c, int slot, int nparts) {
  return nparts <= kHostParts ? c->hsum_d + kSumSlots + (size_t)slot * kHostParts : c->partials;
}

int finish_queue(lc_ctx* c, int slot, int nparts) {
  c->pending[slot] = nparts <= kHostParts ? nparts : 0;
  if (nparts > kHostParts) KLAUNCH(c, LC_K_REDUCE, launch_sum(c->partials, nparts, c->hsum_d + slot, c->stream));
  return LC_OK;
}

int div_queue(lc_ctx* c, const double* v, double* r, int slot, bool watch) {
  const int np = divergence_parts(c->nx, c->ny, c->nz);
  if (watch) {
    uint64_t* const u = (uint64_t*)(np <= kHostParts ? terms_of(c, slot) : c->hsum + slot);
    std::fill(u, u + (np <= kHostParts ? np : 1), kUnset);
  }
  KLAUNCH(c, LC_K_DIVERGENCE, launch_divergence(c->g, v, r, parts_of(c, slot, np), c->stream));
  return finish_queue(c, slot, np);
}

int dot_queue(lc_ctx* c, const double* a, const double* b, int slot) {
  int np = dot_parts(c->nvel);
  KLAUNCH(c, LC_K_VECTOR, launch_dot_partials(a, b, c->nvel, parts_of(c, slot, np), &np, c->stream));
  return finish_queue(c, slot, np);
}

int watched_wait(lc_ctx* c, int slot) {
  const int n = c->pending[slot];
  const uint64_t* const u = (const uint64_t*)(n ? terms_of(c, slot) : c->hsum + slot);
  unsigned turns = 0;
  for (int i = 0; i < (n ? n : 1); ++i)
    while (__atomic_load_n(u + i, __ATOMIC_ACQUIRE) == kUnset)
      if (++turns % (1u << 20) == 0) {  // a stream that has ended leaves nothing to wait for
        const hipError_t e = hipStreamQuery(c->stream);
        if (e == hipSuccess) return LC_OK;
        (void)hipGetLastError();  // (not ready is no error of the next launch)
        if (e != hipErrorNotReady) HIPCHK(c, e);
      }
  return LC_OK;
}

int sums_wait(lc_ctx* c) {
  HIPCHK(c, hipStreamSynchronize(c->stream));
  return LC_OK;
}

// The terms in the order of the reduction kernel (launch_sum): a tree over 1024 of them.
double sum_of(const lc_ctx* c, int slot) {
  const int n = c->pending[slot];
  if (!n) return c->hsum[slot];
  static_assert(kHostParts <= 1024, "one term per thread of the reduction kernel");
  double t[kHostParts];
  std::memcpy(t, terms_of(c, slot), n * sizeof(double));
  int m = n;
  for (int w = 512; w > 0; w >>= 1) {
    for (int i = 0; i + w < m; ++i) t[i] += t[i + w];
    m = std::min(m, w);
  }
  return t[0];
}

int vnorm_div(lc_ctx* c, const double* v, double* r, double* out) {
  int rc = div_queue(c, v, r, 0);
  if (rc || (rc = sums_wait(c))) return rc;
  *out = std::sqrt(sum_of(c, 0));
  return LC_OK;
}

int upload_grid(lc_ctx* c) {
  const int n[3] = {c->nx, c->ny, c->nz};
  // metrics: per axis rd (n), rdd (n+1), th (n+1), d (n)
  const size_t total = metric_doubles(n[0], n[1], n[2]);
  if (!c->metric) HIPCHK(c, dalloc(c, &c->metric, total));
  std::vector<double> host(total);
  size_t off = 0;
  AxisDev* dst[3] = {&c->g.x, &c->g.y, &c->g.z};
  for (int a = 0; a < 3; ++a) {
    const AxisHost& A = c->ax[a];
    double* base = c->metric + off;
    std::copy(A.rd.begin(), A.rd.end(), host.begin() + off);
    dst[a]->rd = base;
    off += n[a];
    std::copy(A.rdd.begin(), A.rdd.end(), host.begin() + off);
    dst[a]->rdd = c->metric + off;
    off += n[a] + 1;
    std::copy(A.th.begin(), A.th.end(), host.begin() + off);
    dst[a]->th = c->metric + off;
    off += n[a] + 1;
    std::copy(A.d.begin(), A.d.end(), host.begin() + off);
    dst[a]->d = c->metric + off;
    off += n[a];
    dst[a]->n = n[a];
  }
  HIPCHK(c, hipMemcpyAsync(c->metric, host.data(), total * sizeof(double), hipMemcpyHostToDevice, c->stream));

  // tensor-product factorization of each axis, in both precisions
  size_t mbytes = 0;
  for (int a = 0; a < 3; ++a) mbytes += mode_bytes(n[a], true);
  if (!c->modes_mem) HIPCHK(c, ctx_alloc(c, &c->modes_mem, mbytes));
  Stager st(mbytes, c->modes_mem);
  for (int a = 0; a < 3; ++a) {
    const int m = n[a];
    const AxisHost& AH = c->ax[a];
    // mirror symmetry: widths and centre distances equal under i -> m-1-i
    bool sym = m >= 2;
    double wmax = 0.0;
    for (int i = 0; i < m; ++i) wmax = std::max(wmax, AH.d[i]);
    for (int i = 0; i < m && sym; ++i) sym = std::fabs(AH.d[i] - AH.d[m - 1 - i]) <= 1e-12 * wmax;
    for (int i = 0; i <= m && sym; ++i) sym = std::fabs(AH.dd[i] - AH.dd[m - i]) <= 1e-12 * wmax;
    c->axis_sym[a] = sym;
    std::vector<double> kd, ko;
    neumann_operator(m, AH.dd.data(), kd, ko);
    ModeHost H;
    if (!compute_modes(m, kd, ko, AH.d, sym, H))
      return fail(c, LC_EINVAL, "tridiagonal eigen-solver did not converge on axis %d", a);
    place_modes(H, c->modes[a], st, true);
    // ascending; the Neumann null mode is the largest (~0), last of the even modes when folded
    c->zero_mode[a] = sym ? (m + 1) / 2 - 1 : m - 1;
  }
  if (st.overflow) return fail(c, LC_ENOMEM, "mode storage sized too small (internal)");
  HIPCHK(c, hipMemcpyAsync(c->modes_mem, st.host.data(), st.used, hipMemcpyHostToDevice, c->stream));
  HIPCHK(c, hipStreamSynchronize(c->stream));
  c->stokes_ready = false;  // the viscous-step factors belong to the previous grid
  c->grid_ready = true;
  return LC_OK;
}

// the pressure solve ends in tridiagonal solves along x (else in a division by sums of eigenvalues)
static bool uses_tridiag(const lc_ctx* c) { return c->poisson_method == LC_POISSON_TPT && c->nx <= tridiag_x_max(); }

// (D G) phi = r by the tensor-product solve.  TPT: transforms with S^T M along y and z, one tridiagonal
// solve per x-line, transforms back with S.  TPF: transforms along x, y and z and a division by
// the sums of the axis eigenvalues (constant mode set to zero).
template <typename T, typename F>
int tp_solve(lc_ctx* c, const F* r, F* phi, T* t1, T* t2, const SolveHook& hook) {
  const int nx = c->nx, ny = c->ny, nz = c->nz;
  const AxisModes &X = c->modes[0], &Y = c->modes[1], &Z = c->modes[2];
  auto lams = [](const AxisModes& M) { return M.sym ? M.lam_s : M.lam; };
  hipStream_t s = c->stream;
  const int pl = nx * ny;
  const Columns cy{nx * nz, nx, pl, nx, c->ncell}, cz{pl, pl, 0, pl, c->ncell};
  const LineScale none;
  if (uses_tridiag(c)) {
    KLAUNCH(c, LC_K_TP_Y, left_forward<T>(Y, ny, cy, r, t1, none, s));
    if (const int rc = hook(1)) return rc;
    KLAUNCH(c, LC_K_TP_Z, left_forward<T>(Z, nz, cz, t1, t2, none, s));
    if (const int rc = hook(2)) return rc;
    KLAUNCH(c, LC_K_TRIDIAG,
            launch_tridiag_x<T>(c->g, lams(Y), lams(Z), c->zero_mode[1], c->zero_mode[2], t2, t1, s));
    KLAUNCH(c, LC_K_TP_Z, left_backward<T>(Z, nz, cz, t1, t2, none, s));
    KLAUNCH(c, LC_K_TP_Y, left_backward<T>(Y, ny, cy, t2, phi, none, s));
    return LC_OK;
  }
  if constexpr (sizeof(F) == sizeof(T)) {
    const LineScale sc{lams(Z), lams(Y), lams(X), nx, c->zero_mode[2], c->zero_mode[1], c->zero_mode[0]};
    KLAUNCH(c, LC_K_TP_X, right_forward<T>(X, nx, ny * nz, r, t1, s));
    if (const int rc = hook(1)) return rc;
    KLAUNCH(c, LC_K_TP_Y, left_forward<T>(Y, ny, cy, t1, t2, none, s));
    if (const int rc = hook(2)) return rc;
    KLAUNCH(c, LC_K_TP_Z, left_forward<T>(Z, nz, cz, t2, t1, sc, s));
    KLAUNCH(c, LC_K_TP_Z, left_backward<T>(Z, nz, cz, t1, t2, sc, s));
    KLAUNCH(c, LC_K_TP_Y, left_backward<T>(Y, ny, cy, t2, t1, none, s));
    KLAUNCH(c, LC_K_TP_X, right_backward<T>(X, nx, ny * nz, t1, phi, s));
    return LC_OK;
  }
  return fail(c, LC_ESTATE, "FP64 field in an FP32 solve along x (internal)");
}

int poisson(lc_ctx* c, const double* r, double* phi, int precision, const SolveHook& hook) {
  if (precision == LC_FP64) return tp_solve<double>(c, r, phi, c->t1, c->t2, hook);
  // FP32: where the first and the last transform read and write FP64 fields there are no casts
  if (uses_tridiag(c) && c->modes[1].mf) return tp_solve<float>(c, r, phi, c->t1_32, c->t2_32, hook);
  KLAUNCH(c, LC_K_CAST, launch_d2f(c->ncell, r, c->r32, c->stream));
  int rc = tp_solve<float>(c, c->r32, c->r32, c->t1_32, c->t2_32, hook);
  if (rc) return rc;
  KLAUNCH(c, LC_K_CAST, launch_f2d(c->ncell, c->r32, phi, false, c->stream));
  return LC_OK;
}

int check_ready(lc_ctx* c) {
  if (!c) return LC_EINVAL;
  if (!c->grid_ready) return fail(c, LC_ESTATE, "grid not set");
  return LC_OK;
}

bool aligned(const void* p) { return p && ((uintptr_t)p % 8 == 0); }

int reduce_max_to_host(lc_ctx* c, int nparts, double* out) {
  KLAUNCH(c, LC_K_REDUCE, launch_max(c->partials, nparts, c->hsum_d, c->stream));
  HIPCHK(c, hipStreamSynchronize(c->stream));
  *out = c->hsum[0];
  return LC_OK;
}

int vdot(lc_ctx* c, const double* a, const double* b, double* out) {
  int rc = dot_queue(c, a, b, 0);
  if (rc || (rc = sums_wait(c))) return rc;
  *out = sum_of(c, 0);
  return LC_OK;
}

int vmaxabs(lc_ctx* c, const double* a, double* out) {
  int np = 0;
  KLAUNCH(c, LC_K_VECTOR, launch_maxabs_partials(a, c->nvel, c->partials, &np, c->stream));
  return reduce_max_to_host(c, np, out);
}

}  // namespace lk

extern "C" {

const char* lc_version(void) { return "lidkrylov 0.1 (gfx950)"; }

const char* lc_last_error(const lc_ctx* c) { return c ? c->err.c_str() : g_create_error.c_str(); }

size_t lc_vel_size(const lc_ctx* c) { return c ? c->nvel : 0; }
size_t lc_cell_size(const lc_ctx* c) { return c ? c->ncell : 0; }

}  // extern "C"

namespace lk {

size_t metric_doubles(int nx, int ny, int nz) { return 4 * ((size_t)nx + ny + nz) + 6; }

size_t viscous_bytes(int nx, int ny, int nz) {
  size_t b = 0;
  for (int n : {nx, ny, nz}) b += mode_bytes(n, false) + mode_bytes(n + 1, false);
  return b;
}

size_t component_max(int nx, int ny, int nz) {
  return std::max({(size_t)(nx + 1) * ny * nz, (size_t)nx * (ny + 1) * nz, (size_t)nx * ny * (nz + 1)});
}

// Krylov vectors the drivers use with basis or restart length m: Arnoldi 2 (m + 1), Newton
// max(m + 1, 8) + 4 (GMRES basis, BiCGstab(2) vectors, right side, correction, spares).
int krylov_vectors(int m) { return std::max(2 * (m + 1), std::max(m + 1, 8) + 4); }

namespace {

void init_dims(lc_ctx* c, int nx, int ny, int nz) {
  c->nx = nx;
  c->ny = ny;
  c->nz = nz;
  c->nvel = vel_layout(nx, ny, nz).total();
  c->ncell = (size_t)nx * ny * nz;
  c->max_parts = (int)((c->ncell + kReduceBlock - 1) / kReduceBlock) + kGsBlocks * kGsVectors;
  c->max_parts = std::max({c->max_parts, divergence_parts(nx, ny, nz), correct_div_parts(nx, ny, nz)});
}

// The context's device buffers, in a fixed order.  With a caller workspace (or a dry run)
// the buffers that are otherwise allocated on first use -- grid metrics and factors, the
// viscous-step factors, the critical-Re steady states -- are carved here as well, and the
// Krylov vectors get the remainder.
bool carve_all(lc_ctx* c) {
  bool ok = dalloc(c, &c->U, c->nvel) == hipSuccess && dalloc(c, &c->w, c->nvel) == hipSuccess &&
            dalloc(c, &c->r, c->ncell) == hipSuccess && dalloc(c, &c->phi, c->ncell + 1) == hipSuccess &&
            dalloc(c, &c->t1, c->ncell) == hipSuccess && dalloc(c, &c->t2, c->ncell) == hipSuccess &&
            dalloc(c, &c->r32, c->ncell) == hipSuccess && dalloc(c, &c->t1_32, c->ncell) == hipSuccess &&
            dalloc(c, &c->t2_32, c->ncell) == hipSuccess && dalloc(c, &c->partials, c->max_parts) == hipSuccess &&
            dalloc(c, &c->dsmall, kSmall) == hipSuccess;
  if (!ok || !(c->arena || c->dry)) return ok;
  const int nx = c->nx, ny = c->ny, nz = c->nz;
  size_t mbytes = 0;
  for (int n : {nx, ny, nz}) mbytes += mode_bytes(n, true);
  return dalloc(c, &c->metric, metric_doubles(nx, ny, nz)) == hipSuccess &&
         ctx_alloc(c, &c->modes_mem, mbytes) == hipSuccess &&
         ctx_alloc(c, &c->stokes_mem, viscous_bytes(nx, ny, nz)) == hipSuccess &&
         dalloc(c, &c->vscale, 2 * ((size_t)nx + ny + nz) + 3) == hipSuccess &&
         dalloc(c, &c->hs, component_max(nx, ny, nz)) == hipSuccess &&
         dalloc(c, &c->ucr, kCriticalVectors * c->nvel) == hipSuccess;
}

int create(lc_ctx** out, int nx, int ny, int nz, void* ws, size_t ws_bytes, void* hip_stream) {
  if (!out) return fail(nullptr, LC_EINVAL, "null output pointer");
  *out = nullptr;
  if (nx < 2 || ny < 2 || nz < 2 || nx > 4096 || ny > 4096 || nz > 4096)
    return fail(nullptr, LC_EINVAL, "grid size %dx%dx%d outside [2, 4096]", nx, ny, nz);
  {
    // the stencil kernels address each velocity component with 32-bit byte offsets
    const VelLayout L = vel_layout(nx, ny, nz);
    if (8 * std::max(L.nu, std::max(L.nv, L.nw)) >= (size_t(1) << 31))
      return fail(nullptr, LC_EINVAL, "grid %dx%dx%d: a velocity component exceeds 2^31 bytes", nx, ny, nz);
  }
  lc_ctx* c = new lc_ctx();
  init_dims(c, nx, ny, nz);
  c->stream = (hipStream_t)hip_stream;
  c->arena = (char*)ws;
  c->arena_size = ws ? ws_bytes : 0;
  bool ok = carve_all(c);
  if (ok && c->arena) {  // the Krylov vectors: the rest of the workspace
    const size_t at = (c->arena_used + 255) / 256 * 256;
    c->kws = (double*)(c->arena + std::min(at, c->arena_size));
    c->kws_n = at < c->arena_size ? (c->arena_size - at) / sizeof(double) : 0;
  }
  if (!ok) {
    lc_destroy(c);
    if (ws) {
      size_t need = 0;
      lc_workspace_query(nx, ny, nz, 0, &need);
      return fail(nullptr, LC_ENOMEM, "workspace of %zu bytes too small for a %dx%dx%d context (at least %zu)",
                  ws_bytes, nx, ny, nz, need);
    }
    return fail(nullptr, LC_ENOMEM, "device allocation failed for %dx%dx%d", nx, ny, nz);
  }
  ok = hipHostMalloc((void**)&c->hsmall, kSmall * sizeof(double), hipHostMallocDefault) == hipSuccess &&
       hipHostMalloc((void**)&c->hsum, kSumSlots * (1 + kHostParts) * sizeof(double),
                     hipHostMallocMapped | hipHostMallocCoherent) == hipSuccess &&
       hipHostGetDevicePointer((void**)&c->hsmall_d, c->hsmall, 0) == hipSuccess &&
       hipHostGetDevicePointer((void**)&c->hsum_d, c->hsum, 0) == hipSuccess;
  if (!ok) {
    lc_destroy(c);
    return fail(nullptr, LC_ENOMEM, "pinned host allocation failed");
  }
  if (hipMemsetAsync(c->U, 0, c->nvel * sizeof(double), c->stream) != hipSuccess) {
    lc_destroy(c);
    return fail(nullptr, LC_EHIP, "hipMemsetAsync failed");
  }
  int rc = lc_set_stretching(c, LC_UNIFORM, 0.0);
  if (rc) {
    g_create_error = c->err;
    lc_destroy(c);
    return rc;
  }
  *out = c;
  return LC_OK;
}

}  // namespace
}  // namespace lk

extern "C" {

int lc_workspace_query(int nx, int ny, int nz, int m_max, size_t* bytes) {
  if (!bytes || nx < 2 || ny < 2 || nz < 2 || nx > 4096 || ny > 4096 || nz > 4096 || m_max < 0 || m_max > 400)
    return LC_EINVAL;
  const VelLayout L = vel_layout(nx, ny, nz);
  if (8 * std::max(L.nu, std::max(L.nv, L.nw)) >= (size_t(1) << 31)) return LC_EINVAL;
  lc_ctx c;
  init_dims(&c, nx, ny, nz);
  c.dry = true;
  carve_all(&c);
  const size_t at = (c.arena_used + 255) / 256 * 256;
  const size_t ld = (c.nvel + 63) / 64 * 64;
  *bytes = at + (size_t)krylov_vectors(m_max) * ld * sizeof(double);
  return LC_OK;
}

int lc_create(lc_ctx** out, int nx, int ny, int nz, void* hip_stream) {
  return create(out, nx, ny, nz, nullptr, 0, hip_stream);
}

int lc_create_in(lc_ctx** out, int nx, int ny, int nz, void* workspace, size_t bytes, void* hip_stream) {
  if (!workspace || (uintptr_t)workspace % 256) return fail(nullptr, LC_EINVAL, "workspace must be 256-byte aligned");
  return create(out, nx, ny, nz, workspace, bytes, hip_stream);
}

int lc_destroy(lc_ctx* c) {
  if (!c) return LC_OK;
  if (c->stream) (void)hipStreamSynchronize(c->stream);
  else (void)hipDeviceSynchronize();
  if (!c->arena) {  // carved buffers belong to the caller's workspace
    void* ptrs[] = {c->U, c->w, c->r, c->phi, c->t1, c->t2, c->r32, c->t1_32, c->t2_32, c->partials,
                    c->metric, c->modes_mem, c->dsmall, c->kws, c->ucr, c->stokes_mem, c->vscale, c->hs};
    for (void* p : ptrs)
      if (p) (void)hipFree(p);
  }
  if (c->hsum) (void)hipHostFree(c->hsum);
  if (c->hsmall) (void)hipHostFree(c->hsmall);
  for (hipEvent_t e : c->ev_pool) (void)hipEventDestroy(e);
  delete c;
  return LC_OK;
}

int lc_set_stream(lc_ctx* c, void* s) {
  if (!c) return LC_EINVAL;
  c->stream = (hipStream_t)s;
  return LC_OK;
}

int lc_set_grid(lc_ctx* c, const double* xf, const double* yf, const double* zf) {
  if (!c || !xf || !yf || !zf) return fail(c, LC_EINVAL, "null argument");
  const double* f[3] = {xf, yf, zf};
  const int n[3] = {c->nx, c->ny, c->nz};
  for (int a = 0; a < 3; ++a) {
    if (f[a][0] != 0.0 || f[a][n[a]] != 1.0) return fail(c, LC_EINVAL, "axis %d faces must run from 0 to 1", a);
    for (int i = 0; i < n[a]; ++i)
      if (!(f[a][i + 1] > f[a][i]) || !std::isfinite(f[a][i + 1]))
        return fail(c, LC_EINVAL, "axis %d faces must increase strictly", a);
  }
  for (int a = 0; a < 3; ++a) c->ax[a].build(f[a], n[a]);
  return upload_grid(c);
}

int lc_set_stretching(lc_ctx* c, int kind, double param) {
  if (!c) return LC_EINVAL;
  if (kind == LC_TANH && !(param > 1.0)) return fail(c, LC_EINVAL, "tanh ratio must exceed 1");
  if (kind != LC_UNIFORM && kind != LC_SINE && kind != LC_TANH) return fail(c, LC_EINVAL, "unknown stretching");
  const int n[3] = {c->nx, c->ny, c->nz};
  std::vector<double> f[3];
  for (int a = 0; a < 3; ++a) {
    f[a].resize(n[a] + 1);
    for (int i = 0; i <= n[a]; ++i) {
      const double xi = (double)i / n[a];
      double x = xi;
      if (kind == LC_SINE) {
        x = xi - 0.0975 * std::sin(2.0 * M_PI * xi);  // Section 3, eq. 5
      } else if (kind == LC_TANH) {
        const double b = std::acosh(std::sqrt(param));
        x = 0.5 * (1.0 + std::tanh(b * (2.0 * xi - 1.0)) / std::tanh(b));
      }
      f[a][i] = x;
    }
    f[a][0] = 0.0;
    f[a][n[a]] = 1.0;
  }
  return lc_set_grid(c, f[0].data(), f[1].data(), f[2].data());
}

int lc_get_grid(const lc_ctx* c, double* xf, double* yf, double* zf) {
  if (!c || !xf || !yf || !zf) return LC_EINVAL;
  std::copy(c->ax[0].xf.begin(), c->ax[0].xf.end(), xf);
  std::copy(c->ax[1].xf.begin(), c->ax[1].xf.end(), yf);
  std::copy(c->ax[2].xf.begin(), c->ax[2].xf.end(), zf);
  return LC_OK;
}

int lc_set_poisson_method(lc_ctx* c, int method) {
  if (!c) return LC_EINVAL;
  if (method != LC_POISSON_TPF && method != LC_POISSON_TPT) return fail(c, LC_EINVAL, "unknown Poisson method %d", method);
  c->poisson_method = method;
  return LC_OK;
}

int lc_set_re(lc_ctx* c, double re) {
  if (!c) return LC_EINVAL;
  if (!(re > 0.0) || !std::isfinite(re)) return fail(c, LC_EINVAL, "Re must be positive and finite");
  c->re = re;
  return LC_OK;
}

int lc_set_lid(lc_ctx* c, double alpha) {
  if (!c) return LC_EINVAL;
  if (!std::isfinite(alpha)) return fail(c, LC_EINVAL, "lid angle must be finite");
  c->alpha = alpha;
  return LC_OK;
}

int lc_set_base_flow(lc_ctx* c, const double* U) {
  if (!c || !aligned(U)) return fail(c, LC_EINVAL, "null or misaligned base flow");
  HIPCHK(c, hipMemcpyAsync(c->U, U, c->nvel * sizeof(double), hipMemcpyDeviceToDevice, c->stream));
  KLAUNCH(c, LC_K_VECTOR, launch_zero_walls(c->U, c->nx, c->ny, c->nz, c->stream));
  HIPCHK(c, hipStreamSynchronize(c->stream));
  return LC_OK;
}

int lc_get_base_flow(lc_ctx* c, double* U, double* P) {
  if (!c || !aligned(U) || (P && !aligned(P))) return fail(c, LC_EINVAL, "bad pointers");
  HIPCHK(c, hipMemcpyAsync(U, c->U, c->nvel * sizeof(double), hipMemcpyDeviceToDevice, c->stream));
  if (P) {
    // the pressure of the steady equations: R(U) - G P divergence-free, sum V P = 0 (at a
    // steady state R(U) = G P); the projection's velocity goes to one Krylov vector
    int rc = check_ready(c);
    if (rc) return rc;
    double* tmp = nullptr;
    long ld = 0;
    if ((rc = krylov_ws(c, 1, &tmp, &ld))) return rc;
    KLAUNCH(c, LC_K_RESIDUAL, launch_momentum(c->g, c->U, c->U, c->w, 1.0 / c->re, true, std::cos(c->alpha),
                                              std::sin(c->alpha), c->stream));
    lc_stats st;
    rc = lc_project(c, c->w, tmp, P, LC_FP64, 1e-13, 4, &st);
    if (rc < 0) return rc;
  }
  HIPCHK(c, hipStreamSynchronize(c->stream));
  return LC_OK;
}

int lc_jacobian_apply(lc_ctx* c, const double* v, double* w) {
  int rc = check_ready(c);
  if (rc) return rc;
  if (!aligned(v) || !aligned(w) || v == w) return fail(c, LC_EINVAL, "bad or aliased velocity pointers");
  KLAUNCH(c, LC_K_MOMENTUM, launch_momentum(c->g, c->U, v, w, 1.0 / c->re, false, 0, 0, c->stream));
  HIPCHK(c, hipStreamSynchronize(c->stream));
  return LC_OK;
}

int lc_residual(lc_ctx* c, const double* U, double* R) {
  int rc = check_ready(c);
  if (rc) return rc;
  if (!aligned(U) || !aligned(R) || U == R) return fail(c, LC_EINVAL, "bad or aliased velocity pointers");
  KLAUNCH(c, LC_K_RESIDUAL, launch_momentum(c->g, U, U, R, 1.0 / c->re, true, std::cos(c->alpha), std::sin(c->alpha),
                            c->stream));
  HIPCHK(c, hipStreamSynchronize(c->stream));
  return LC_OK;
}

int lc_divergence(lc_ctx* c, const double* v, double* r, double* vn) {
  int rc = check_ready(c);
  if (rc) return rc;
  if (!aligned(v) || !aligned(r)) return fail(c, LC_EINVAL, "bad pointers");
  double nrm = 0.0;
  rc = vnorm_div(c, v, r, &nrm);
  if (rc) return rc;
  if (vn) *vn = nrm;
  return LC_OK;
}

int lc_poisson_solve(lc_ctx* c, const double* r, double* phi, int precision) {
  int rc = check_ready(c);
  if (rc) return rc;
  if (!aligned(r) || !aligned(phi)) return fail(c, LC_EINVAL, "bad pointers");
  if (precision != LC_FP64 && precision != LC_MIXED) return fail(c, LC_EINVAL, "unknown precision");
  rc = poisson(c, r, phi, precision);
  if (rc) return rc;
  HIPCHK(c, hipStreamSynchronize(c->stream));
  return LC_OK;
}

int lc_correct(lc_ctx* c, const double* w, const double* phi, double* v, double* p) {
  int rc = check_ready(c);
  if (rc) return rc;
  if (!aligned(w) || !aligned(phi) || !aligned(v) || (p && !aligned(p)) || v == w)
    return fail(c, LC_EINVAL, "bad pointers");
  KLAUNCH(c, LC_K_CORRECT, launch_correct(c->g, w, phi, v, p, false, c->stream));
  HIPCHK(c, hipStreamSynchronize(c->stream));
  return LC_OK;
}

}  // extern "C"

namespace {
// per-phase device time of the launches recorded since rec0 (profiling on), else -1
void fill_phases(lc_ctx* c, lc_stats* S, size_t rec0) {
  if (!S) return;
  S->ms_stencil = S->ms_poisson = S->ms_update = S->ms_network = -1.0;
  if (!c->prof || hipStreamSynchronize(c->stream) != hipSuccess) return;
  double t[4] = {0.0, 0.0, 0.0, 0.0};
  for (size_t q = rec0; q < c->recs.size(); ++q) {
    const int k = c->recs[q].kid;
    const int ph = (k == LC_K_MOMENTUM || k == LC_K_RESIDUAL || k == LC_K_DIVERGENCE) ? 0
                   : (k == LC_K_TP_X || k == LC_K_TP_Y || k == LC_K_TP_Z || k == LC_K_EIGSCALE ||
                      k == LC_K_TRIDIAG || k == LC_K_CAST)
                       ? 1
                   : k == LC_K_CORRECT                             ? 2
                   : (k == LC_K_NN_FORWARD || k == LC_K_NN_MISC) ? 3
                                                                   : -1;
    float ms = 0.f;
    if (ph >= 0 && hipEventElapsedTime(&ms, c->recs[q].a, c->recs[q].b) == hipSuccess) t[ph] += ms;
  }
  S->ms_stencil = t[0];
  S->ms_poisson = t[1];
  S->ms_update = t[2];
  S->ms_network = t[3];
}

int project_impl(lc_ctx* c, const double* w, double* v, double* p, int precision, double tol, int max_iter,
                 lc_stats* st) {
  const double t0 = now_ms();
  int rc = check_ready(c);
  if (rc) return rc;
  if (!aligned(w) || !aligned(v) || (p && !aligned(p)) || v == w || p == w || p == v)
    return fail(c, LC_EINVAL, "bad pointers");
  if (precision != LC_FP64 && precision != LC_MIXED && precision != LC_LEARNED)
    return fail(c, LC_EINVAL, "unknown precision");
  if (precision == LC_LEARNED && !c->net) return fail(c, LC_ESTATE, "no network attached for the learned form");
  if (!(tol >= 0.0) || max_iter < 1) return fail(c, LC_EINVAL, "bad tolerance or iteration cap");
  lc_stats local{};
  lc_stats& S = st ? *st : local;
  std::memset(&S, 0, sizeof S);
  S.guess_eps = 1.0;
  // One pass of the SIMPLE loop (Section 3): solve, correct, certify (slot 1).  The certificate of an FP64
  // pass (exact solve: it nearly always ends the loop) only reduces the norm; D v is then written
  // again if another pass needs it.  FP32 passes (one more always follows at tight tolerances)
  // keep D v from the certificate.
  const int pass_precision = precision == LC_LEARNED ? LC_MIXED : precision;
  const bool keep_r = pass_precision != LC_FP64;
  auto pass = [&](bool accumulate, const SolveHook& hook = {}) -> int {
    int e = poisson(c, c->r, c->phi, pass_precision, hook);
    if (e || (e = hook(3))) return e;
    if (!accumulate) {
      const int np = correct_div_parts(c->nx, c->ny, c->nz);
      KLAUNCH(c, LC_K_CORRECT,
              launch_correct_div(c->g, w, c->phi, v, p, keep_r ? c->r : nullptr, parts_of(c, 1, np), c->stream));
      return finish_queue(c, 1, np);
    }
    KLAUNCH(c, LC_K_CORRECT, launch_correct(c->g, w, c->phi, v, p, true, c->stream));
    return div_queue(c, v, keep_r ? c->r : nullptr, 1);
  };
  // |D w| decides whether there is a pass at all, and v and p stay as they are if it is not finite.  Without a
  // guess it is read while the pass's solve is under way, which needs D w but not its norm and writes nothing of the
  // caller's; the GPU must not run dry before the host has queued more, and an input without divergence
  // pays for what is queued: the whole solve up to 64^3 (read after the first transform, 16^3 to 64^3 lose
  // 5 to 8 us of 58 to 70), two transforms up to 150^3, one beyond.  Long axes take long enough by themselves (16 x 16
  // x 300 one-sided, input without divergence: 65 us if read after the first transform, 235 after the solve), and
  // those without the matrix cores even in the first one (300 points, 256 columns 57 us): it waits before them.
  double n0 = 0.0;
  auto read_norm = [&]() -> int {
    n0 = std::sqrt(sum_of(c, 0));
    return std::isfinite(n0) ? LC_OK : fail(c, LC_EINVAL, "non-finite input");
  };
  const AxisModes& first = c->modes[uses_tridiag(c) ? 1 : 0];
  const bool ahead = precision != LC_LEARNED && (first.mf || (first.full64 && precision == LC_FP64));
  const int longest = std::max(uses_tridiag(c) ? 0 : c->nx, std::max(c->ny, c->nz));
  const int queued = c->ncell <= 300000 && longest <= 100 ? 3 : c->ncell <= 3500000 && longest <= 160 ? 2 : 1;
  if ((rc = div_queue(c, w, c->r, 0, ahead))) return rc;
  if (ahead) {
    constexpr int kNoPass = 2;
    rc = pass(false, {queued, [&]() -> int {
      if (const int e = watched_wait(c, 0)) return e;
      if (const int e = read_norm()) {
        HIPCHK(c, hipStreamSynchronize(c->stream));
        return e;
      }
      return n0 == 0.0 ? kNoPass : LC_OK;
    }});
    if (rc == LC_OK) rc = sums_wait(c);
    if (rc && rc != kNoPass) return rc;
  } else if ((rc = sums_wait(c)) || (rc = read_norm())) {
    return rc;
  }
  S.rho0 = n0;
  if (n0 == 0.0) {
    // already divergence-free: v = w (walls zeroed), p = 0
    HIPCHK(c, hipMemsetAsync(c->phi, 0, c->ncell * sizeof(double), c->stream));
    KLAUNCH(c, LC_K_CORRECT, launch_correct(c->g, w, c->phi, v, p, false, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    S.ms_total = now_ms() - t0;
    return LC_OK;
  }
  // Learned form: the network's correction starts the loop (v = w - G phi0, p = phi0),
  // then mixed-precision passes; without gain it falls back to v = w, p = 0.
  bool started = false;
  if (precision == LC_LEARNED) {
    double fit = 1.0;
    rc = learned_start(c, w, v, p, &started, &fit);
    if (rc) return rc;
    if (started) {
      double nk = 0.0;
      rc = vnorm_div(c, v, c->r, &nk);
      if (rc) return rc;
      S.guess_used = 1;
      S.guess_eps = nk / n0;
      if (!std::isfinite(S.guess_eps)) return fail(c, LC_EINVAL, "non-finite divergence after the learned guess");
      S.rho = S.guess_eps;
      if (S.rho <= tol) {
        S.ms_total = now_ms() - t0;
        return LC_OK;
      }
    }
  }
  // SIMPLE loop (Section 3): v = w, p = 0; repeat {solve; v -= G phi; p += phi}
  for (int it = 0; it < max_iter; ++it) {
    if (!(ahead && it == 0) && ((rc = pass(started || it > 0)) || (rc = sums_wait(c)))) return rc;
    double nk = std::sqrt(sum_of(c, 1));
    if (!keep_r && nk / n0 > tol && it + 1 < max_iter) {
      rc = vnorm_div(c, v, c->r, &nk);
      if (rc) return rc;
    }
    S.iterations = it + 1;
    S.rho = nk / n0;
    if (it < 16) S.rho_hist[it] = S.rho;
    if (!std::isfinite(S.rho)) return fail(c, LC_EINVAL, "non-finite divergence during projection");
    if (S.rho <= tol) {
      S.ms_total = now_ms() - t0;
      return LC_OK;
    }
  }
  S.ms_total = now_ms() - t0;
  return LC_ENOTCONV;
}

}  // namespace

extern "C" {

int lc_project(lc_ctx* c, const double* w, double* v, double* p, int precision, double tol, int max_iter,
               lc_stats* st) {
  const size_t rec0 = c ? c->recs.size() : 0;
  const int rc = project_impl(c, w, v, p, precision, tol, max_iter, st);
  if (c && rc >= 0) fill_phases(c, st, rec0);
  return rc;
}

int lc_krylov_vector(lc_ctx* c, const double* vin, double* vout, double* pout, int precision, double tol,
                     int max_iter, lc_stats* st) {
  const double t0 = now_ms();
  int rc = check_ready(c);
  if (rc) return rc;
  if (!aligned(vin) || !aligned(vout) || vin == vout) return fail(c, LC_EINVAL, "bad or aliased pointers");
  const size_t rec0 = c->recs.size();
  KLAUNCH(c, LC_K_MOMENTUM, launch_momentum(c->g, c->U, vin, c->w, 1.0 / c->re, false, 0, 0, c->stream));
  rc = project_impl(c, c->w, vout, pout, precision, tol, max_iter, st);
  if (rc >= 0) fill_phases(c, st, rec0);
  if (st) st->ms_total = now_ms() - t0;
  return rc;
}

int lc_dot(lc_ctx* c, const double* a, const double* b, double* out) {
  if (!c || !aligned(a) || !aligned(b) || !out) return fail(c, LC_EINVAL, "bad pointers");
  return vdot(c, a, b, out);
}

}  // extern "C"

static const char* kKernelNames[LC_K_COUNT] = {"momentum", "residual", "divergence", "correct",  "tp_x",
                                                "tp_y",     "tp_z",     "eigscale",   "reduce",   "cast",
                                                "vector",   "nn_forward", "nn_misc",  "planes",  "tridiag"};

extern "C" const char* lc_profile_name(int k) { return (k >= 0 && k < LC_K_COUNT) ? kKernelNames[k] : nullptr; }

extern "C" int lc_profile_enable(lc_ctx* c, int on) {
  if (!c) return LC_EINVAL;
  HIPCHK(c, hipStreamSynchronize(c->stream));
  c->recs.clear();
  c->ev_used = 0;
  c->prof = on != 0;
  return LC_OK;
}

extern "C" int lc_profile_read(lc_ctx* c, int k, double* total_ms, long* launches) {
  if (!c || k < 0 || k >= LC_K_COUNT || !total_ms || !launches) return LC_EINVAL;
  HIPCHK(c, hipStreamSynchronize(c->stream));
  double t = 0.0;
  long n = 0;
  for (const auto& r : c->recs) {
    if (r.kid != k) continue;
    float ms = 0.f;
    HIPCHK(c, hipEventElapsedTime(&ms, r.a, r.b));
    t += ms;
    ++n;
  }
  *total_ms = t;
  *launches = n;
  return LC_OK;
}

extern "C" int lc_stream_probe(int kind, size_t bytes, int reps, void* hip_stream, double* tbps, double* us) {
  if (kind < 0 || kind > 2 || bytes < 4096 || reps < 1 || !tbps) return LC_EINVAL;
  const size_t n2 = bytes / 16;
  hipStream_t st = (hipStream_t)hip_stream;
  double *a = nullptr, *b = nullptr, *c = nullptr;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  int rc = LC_OK;
  if (hipMalloc((void**)&a, n2 * 16) != hipSuccess || hipMalloc((void**)&b, n2 * 16) != hipSuccess ||
      hipMalloc((void**)&c, n2 * 16 + 8) != hipSuccess) {
    rc = LC_ENOMEM;
  } else if (hipMemsetAsync(a, 0, n2 * 16, st) != hipSuccess || hipMemsetAsync(b, 0, n2 * 16, st) != hipSuccess ||
             hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
    rc = LC_EHIP;
  } else {
    double* sink = c + 2 * n2;
    bool ok = true;
    for (int w = 0; w < 3 && ok; ++w) ok = launch_probe(kind, a, b, c, n2, sink, st) == hipSuccess;
    ok = ok && hipEventRecord(e0, st) == hipSuccess;
    for (int r = 0; r < reps && ok; ++r) ok = launch_probe(kind, a, b, c, n2, sink, st) == hipSuccess;
    ok = ok && hipEventRecord(e1, st) == hipSuccess && hipEventSynchronize(e1) == hipSuccess;
    float ms = 0.f;
    ok = ok && hipEventElapsedTime(&ms, e0, e1) == hipSuccess;
    if (!ok) {
      rc = LC_EHIP;
    } else {
      const double moved = (kind == 0 ? 2.0 : kind == 1 ? 3.0 : 1.0) * (double)(n2 * 16);
      const double t = (double)ms * 1e-3 / reps;
      *tbps = moved / t / 1e12;
      if (us) *us = t * 1e6;
    }
  }
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  if (a) (void)hipFree(a);
  if (b) (void)hipFree(b);
  if (c) (void)hipFree(c);
  return rc;
}

extern "C" int lc_axis_modes(int n, const double* faces, double* lam, double* S, double* Wf) {
  if (n < 1 || !faces || !lam || !S || !Wf) return LC_EINVAL;
  for (int i = 0; i < n; ++i)
    if (!(faces[i + 1] > faces[i])) return LC_EINVAL;
  AxisHost A;
  A.build(faces, n);
  std::vector<double> l, s, w;
  if (!neumann_modes(n, A.d.data(), A.dd.data(), l, s, w)) return LC_EINVAL;
  std::copy(l.begin(), l.end(), lam);
  std::copy(s.begin(), s.end(), S);
  std::copy(w.begin(), w.end(), Wf);
  return LC_OK;
}
