// Density-fitting factors from AO three-index integrals, the step before the CC
// iteration (robust fitting; the paper's Introduction names density fitting and
// Cholesky decomposition for the integral tensor, its Performance section the cost of
// the AO->MO transformation):
//
//   B^P_pq = sum_Q [V^-1/2]_PQ sum_{mu nu} conj(C_mu p) (mu nu|Q) C_nu q.
//
// V^-1/2 comes from the coupled Newton-Schulz iteration (Higham, Functions of
// Matrices, 2008, the coupled Newton-Schulz iteration for the matrix square root),
// which needs only matrix products and therefore runs on the same MFMA GETT as
// everything else: with A = V / c (c = max row sum of |V| >= the largest eigenvalue,
// so the spectrum of A lies in (0, 1]), Y_0 = A, Z_0 = I,
//   P_k = Z_k Y_k,  T_k = (3 I - P_k) / 2,  Y_{k+1} = Y_k T_k,  Z_{k+1} = T_k Z_k,
// Z_k -> A^-1/2 quadratically once ||I - P_k|| is small; V^-1/2 = Z / sqrt(c).  The two
// transform GEMMs and the metric GEMM then give B.
#include <algorithm>
#include <cmath>
#include <mutex>
#include <string>
#include <utility>

#include "../../include/exacc.h"

#include "common.h"
#include "einsum.h"

namespace exacc {
namespace {

constexpr int kTB = 256;

inline int nblk(int64_t n, int cap = 4096) {
  return (int)std::max<int64_t>(1, std::min<int64_t>((n + kTB - 1) / kTB, cap));
}

// out[i] = sum_j |V[i][j]|
__global__ void row_abs_sum_kernel(const double* __restrict__ V, int X, double* __restrict__ out) {
  for (int i = blockIdx.x * kTB + threadIdx.x; i < X; i += gridDim.x * kTB) {
    double s = 0.0;
    for (int j = 0; j < X; ++j) s += fabs(V[(int64_t)i * X + j]);
    out[i] = s;
  }
}

// A = V * inv_c (complex, zero imaginary part), Z = I
__global__ void ns_init_kernel(const double* __restrict__ V, int X, double inv_c, double* __restrict__ A,
                               double* __restrict__ Z) {
  const int64_t tot = (int64_t)X * X;
  for (int64_t t = (int64_t)blockIdx.x * kTB + threadIdx.x; t < tot; t += (int64_t)gridDim.x * kTB) {
    const int64_t i = t / X, j = t - i * X;
    A[2 * t] = V[t] * inv_c;
    A[2 * t + 1] = 0.0;
    Z[2 * t] = (i == j) ? 1.0 : 0.0;
    Z[2 * t + 1] = 0.0;
  }
}

// T = (3 I - P) / 2 and per-block partial sums of |I - P|^2
__global__ void ns_step_kernel(const double* __restrict__ P, int X, double* __restrict__ T,
                               double* __restrict__ part) {
  const int64_t tot = (int64_t)X * X;
  double acc = 0.0;
  for (int64_t t = (int64_t)blockIdx.x * kTB + threadIdx.x; t < tot; t += (int64_t)gridDim.x * kTB) {
    const int64_t i = t / X, j = t - i * X;
    const double d = (i == j) ? 1.0 : 0.0;
    const double pr = P[2 * t], pi = P[2 * t + 1];
    acc += (d - pr) * (d - pr) + pi * pi;
    T[2 * t] = 0.5 * (3.0 * d - pr);
    T[2 * t + 1] = -0.5 * pi;
  }
  __shared__ double sh[kTB];
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int w = kTB / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

// max over part[0..n) into out[0] (one workgroup; max is exact in any order)
__global__ void max_kernel(const double* __restrict__ part, int n, double* __restrict__ out) {
  __shared__ double sh[kTB];
  double m = 0.0;
  for (int i = threadIdx.x; i < n; i += kTB) m = fmax(m, part[i]);
  sh[threadIdx.x] = m;
  __syncthreads();
  for (int w = kTB / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) sh[threadIdx.x] = fmax(sh[threadIdx.x], sh[threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = sh[0];
}

inline size_t up256(size_t b) { return (b + 255) / 256 * 256; }

// Bytes of the temporaries that do not depend on the slice width: the reduction
// scalars and partials and the six naux x naux Newton-Schulz matrices.
size_t fixed_bytes(int X) {
  const int64_t nb = nblk((int64_t)X * X);
  return up256(256) + up256((size_t)(std::max<int64_t>(nb, X) + 8) * 8) +
         6 * up256((size_t)X * X * 16);
}
// Least bytes of intermediates that a call must find room for: one spinor row p of all Q.
size_t slice_bytes(int m, int n, int X, int ps) {
  return up256((size_t)X * ps * m * 16) + up256((size_t)X * ps * n * 16);
}

// Bump allocation inside one device region that the caller owns.
struct Carve {
  char* base;
  size_t cap, used = 0;
  double* take(size_t bytes) {
    const size_t b = up256(std::max<size_t>(bytes, 16));
    if (used + b > cap) raise(-2, "DF factors: scratch region exhausted");
    double* p = reinterpret_cast<double*>(base + used);
    used += b;
    return p;
  }
};

// The planner's extent check and the split-K workspace are per thread; restore both.
struct PlannerState {
  AllocRange r[6];
  int n = 0;
  void add(const void* p, size_t bytes) {
    r[n++] = {p, bytes};
    set_alloc_registry(r, n);
  }
  ~PlannerState() {
    set_alloc_registry(nullptr, 0);
    set_gett_workspace(nullptr, 0);
    set_mod_workspace(nullptr, 0);
  }
};

// dst[r][x] = src[r * stride + x], rows of len complex elements
__global__ void copy_rows_kernel(double* __restrict__ dst, const double* __restrict__ src, int64_t rows,
                                 int64_t stride, int64_t len) {
  typedef double d2v __attribute__((ext_vector_type(2)));
  for (int64_t r = blockIdx.y; r < rows; r += gridDim.y)
    for (int64_t x = (int64_t)blockIdx.x * kTB + threadIdx.x; x < len; x += (int64_t)gridDim.x * kTB)
      reinterpret_cast<d2v*>(dst)[r * len + x] = reinterpret_cast<const d2v*>(src)[r * stride + x];
}

// Intermediates: the first half transform runs over chunks of Q (rows p too where one Q does not
// fit) and is finished into B itself, and the metric product runs over column chunks of B
// copied out first, so neither is held whole (7.7 GB at 600/400/1200, cleared when it is
// allocated on each call; the extra copy is 1.5 ms).
constexpr size_t kChunk = (size_t)128 << 20;
size_t chunk_bytes(int m, int n, int X) {
  return std::min(kChunk, up256((size_t)X * n * m * 16)) + std::min(kChunk, up256((size_t)X * n * n * 16));
}
// B holds the half-transformed integrals, so it is written while C and J are still read.  An output
// that overlaps C gets a copy of C; one that overlaps J, the whole first half transform ahead.
struct Overlap {
  size_t c, t1;  // bytes more of the region
};
Overlap overlap(int m, int n, int X, const void* C, const void* J, const void* B) {
  auto hit = [&](const void* a, size_t bytes) {
    const char *p = static_cast<const char*>(a), *b = static_cast<const char*>(B);
    return p < b + (size_t)X * n * n * 16 && b < p + bytes;
  };
  return {hit(C, (size_t)m * n * 16) ? up256((size_t)m * n * 16) : 0,
          hit(J, (size_t)X * m * m * 16) ? up256((size_t)X * n * m * 16) : 0};
}
size_t splitk_bytes(int X) { return std::min<size_t>((size_t)64 << 20, std::max<size_t>(1 << 20, (size_t)X * X * 256)); }

// Host memory that one step's residual norm lands in: pinned, while the next step is on its way
// (lag), or, for the entry point that must not allocate (pinned memory neither: not under a
// capture elsewhere), plain memory that each step waits for.
struct Readback {
  double plain[4] = {};
  double* h = plain;
  hipEvent_t ev[2] = {};
  hipStream_t s;
  const bool lag;
  Readback(hipStream_t st, bool lagged) : s(st), lag(lagged) {
    if (!lag) return;
    HIPCHECK(hipHostMalloc((void**)&h, 4 * sizeof(double), hipHostMallocDefault));
    for (auto& e : ev)
      if (hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) {
        release();
        raise(-3, "DF factors: event creation failed");
      }
  }
  // red[k] to h[k], in flight or landed
  void fetch(int k, const double* red) {
    HIPCHECK(hipMemcpyAsync(&h[k], red + k, 8, hipMemcpyDeviceToHost, s));
    if (lag)
      HIPCHECK(hipEventRecord(ev[k], s));
    else
      HIPCHECK(hipStreamSynchronize(s));
  }
  double get(int k) {
    if (lag) HIPCHECK(hipEventSynchronize(ev[k]));
    return h[k];
  }
  void release() {
    (void)hipStreamSynchronize(s);  // a copy may still be on its way
    for (auto& e : ev)
      if (e) (void)hipEventDestroy(e);
    if (lag && h) (void)hipHostFree(h);
  }
  ~Readback() { release(); }
  Readback(const Readback&) = delete;
  Readback& operator=(const Readback&) = delete;
};

// B from device C, J, V with every temporary inside [base, base + cap): the fixed part, the
// intermediates' chunks and a split-K workspace of what is left, at most ws_cap; mod: residue
// workspace of the large products (may be null).  Returns the
// Newton-Schulz step count.  Nothing in the region needs to start at zero: every
// temporary is written before it is read.
int df_core(int m, int n, int X, const double* Cd, const double* Jd, const double* Vd, double* Bd,
            hipStream_t s, char* base, size_t cap, size_t ws_cap, bool lag, void* mod, size_t mod_bytes) {
  const cplx ONE{1.0, 0.0};
  const size_t fixed = fixed_bytes(X);
  if (fixed + slice_bytes(m, n, X, 1) > cap) raise(-2, "DF factors: scratch region too small");
  const int64_t nn = (int64_t)n * n;
  const Overlap ov = overlap(m, n, X, Cd, Jd, Bd);
  // (a region too small for the whole half transform beside one column of M: in halves, as without
  // an overlap)
  const size_t all = cap - fixed - std::min(cap - fixed, ov.c);
  const bool whole = ov.t1 && ov.t1 + up256((size_t)X * 16) <= all;
  const size_t room = all / 2 / 256 * 256;
  const size_t t1b = whole ? ov.t1 : std::min(std::min(kChunk, up256((size_t)X * n * m * 16)), room);
  const size_t mb = std::min(std::min(kChunk, up256((size_t)X * nn * 16)), whole ? all - ov.t1 : room);
  if (t1b < (size_t)m * 16 || mb < (size_t)X * 16) raise(-2, "DF factors: scratch region too small");
  const int qc = (int)std::max<int64_t>(1, std::min<int64_t>(X, (int64_t)(t1b / ((size_t)n * m * 16))));
  const int pc = (int)std::max<int64_t>(1, std::min<int64_t>(n, (int64_t)(t1b / ((size_t)qc * m * 16))));
  const int64_t xc = std::max<int64_t>(1, std::min<int64_t>(nn, (int64_t)(mb / ((size_t)X * 16))));
  PlannerState ps_state;
  ps_state.add(Cd, (size_t)m * n * 16);
  ps_state.add(Jd, (size_t)X * m * m * 16);
  ps_state.add(Vd, (size_t)X * X * 8);
  ps_state.add(Bd, (size_t)X * n * n * 16);
  ps_state.add(base, cap);
  Carve cv{base, cap};
  const int nb = nblk((int64_t)X * X);
  double* red = cv.take(256);
  double* part = cv.take((size_t)(std::max(nb, X) + 8) * 8);
  double* Y = cv.take((size_t)X * X * 16);
  double* Z = cv.take((size_t)X * X * 16);
  double* P = cv.take((size_t)X * X * 16);
  double* T = cv.take((size_t)X * X * 16);
  double* Y2 = cv.take((size_t)X * X * 16);
  double* Z2 = cv.take((size_t)X * X * 16);
  double* T1 = cv.take((size_t)qc * pc * m * 16);
  double* M = cv.take((size_t)X * xc * 16);
  if (ov.c) {
    double* Cc = cv.take((size_t)m * n * 16);
    k_copy_bytes(Cc, Cd, (int64_t)m * n * 16, s);
    Cd = Cc;
  }
  const size_t left = cap > cv.used ? (cap - cv.used) / 256 * 256 : 0;
  const size_t wsb = std::min(left, ws_cap);
  set_gett_workspace(wsb >= (1u << 20) ? cv.take(wsb) : nullptr, wsb >= (1u << 20) ? wsb : 0);
  Readback rb(s, lag);
  // scale: c = max_i sum_j |V_ij| bounds the spectrum of the symmetric V from above
  hipLaunchKernelGGL(row_abs_sum_kernel, dim3(nblk(X, 1024)), dim3(kTB), 0, s, Vd, X, part);
  HIPCHECK(hipGetLastError());
  hipLaunchKernelGGL(max_kernel, dim3(1), dim3(kTB), 0, s, part, X, red);
  HIPCHECK(hipGetLastError());
  rb.fetch(0, red);
  const double c = rb.get(0);
  if (!(c > 0.0) || !std::isfinite(c)) raise(-1, "DF factors: metric is zero or not finite");
  hipLaunchKernelGGL(ns_init_kernel, dim3(nb), dim3(kTB), 0, s, Vd, X, 1.0 / c, Y, Z);
  HIPCHECK(hipGetLastError());

  auto XXv = [&](double* p) { return view(p, {X, X}); };
  // P = Z Y, T and the norm |I - P| of step k into rb.h[k % 2].  With lag the norm of a step is
  // waited for only once the next step's product is queued, so the host's turnaround is hidden;
  // the next step's P and T are then formed for nothing after the last one.
  auto look = [&](int k, double* Pk, double* Tk) {
    contract(s, "ab,bc->ac", ONE, XXv(Z), XXv(Y), false, XXv(Pk));
    hipLaunchKernelGGL(ns_step_kernel, dim3(nb), dim3(kTB), 0, s, Pk, X, Tk, part);
    HIPCHECK(hipGetLastError());
    k_reduce_sum(part, nb, 1, red + k % 2, s);
    rb.fetch(k % 2, red);
  };
  int iters = 0;
  bool done = false, failed = false;
  look(0, P, T);
  while (iters < 200 && !done && !failed) {
    const int k = iters++;
    contract(s, "ab,bc->ac", ONE, XXv(Y), XXv(T), false, XXv(Y2));
    contract(s, "ab,bc->ac", ONE, XXv(T), XXv(Z), false, XXv(Z2));
    std::swap(Y, Y2);
    std::swap(Z, Z2);
    if (lag && iters < 200) look(iters, P, T);
    const double r = std::sqrt(rb.get(k % 2));
    // quadratic phase: the step just taken brought the error to ~r^2 (rounding level)
    if (!std::isfinite(r) || r > 1e3 * X)
      failed = true;
    else
      done = r < 1e-8;
    if (!lag && !done && !failed && iters < 200) look(iters, P, T);
  }
  if (!done)
    raise(-1, "DF factors: the inverse square root iteration did not converge (metric not positive "
              "definite or too ill-conditioned)");

  // Residues for the transforms and the fit only.  Z and Y are nearly diagonal up to the norms of
  // the functions, so that the products above fail the residues' test as a rule (naux 1200: 32 of
  // 36, at 40 us each for nothing).
  set_mod_workspace(mod, mod_bytes);
  // (pq|Q) = sum_mu nu conj(C_mu p) (mu nu|Q) C_nu q into B, chunks of Q (and p); then
  // B[P][p][q] = sum_Q [V^-1/2]_PQ (pq|Q), chunks of pq
  for (int q0 = 0; q0 < X; q0 += qc)
    for (int p0 = 0; p0 < n; p0 += pc) {
      const int qn = std::min(qc, X - q0), pn = std::min(pc, n - p0);
      contract(s, "mp,Qmn->Qpn", ONE, conj(sview(const_cast<double*>(Cd) + 2 * p0, {m, pn}, {n, 1})),
               view(const_cast<double*>(Jd) + 2 * (int64_t)q0 * m * m, {qn, m, m}), false, view(T1, {qn, pn, m}));
      contract(s, "Qpn,nq->Qpq", ONE, view(T1, {qn, pn, m}), view(const_cast<double*>(Cd), {m, n}), false,
               sview(Bd + 2 * ((int64_t)q0 * nn + (int64_t)p0 * n), {qn, pn, n}, {nn, n, 1}));
    }
  for (int64_t x0 = 0; x0 < nn; x0 += xc) {
    const int64_t xn = std::min<int64_t>(xc, nn - x0);
    hipLaunchKernelGGL(copy_rows_kernel, dim3(nblk(xn, 64), std::min(X, 16384)), dim3(kTB), 0, s, M, Bd + 2 * x0,
                       (int64_t)X, nn, xn);
    HIPCHECK(hipGetLastError());
    contract(s, "PQ,Qx->Px", cplx{1.0 / std::sqrt(c), 0.0}, XXv(Z), view(M, {X, xn}), false,
             sview(Bd + 2 * x0, {X, xn}, {nn, 1}));
  }
  HIPCHECK(hipStreamSynchronize(s));
  return iters;
}

// Device memory of one allocating call, freed on every exit path.
struct Owned {
  void* p[6] = {};
  ~Owned() {
    for (void* q : p)
      if (q) (void)hipFree(q);
  }
  char* alloc(int k, size_t bytes) {
    hipError_t e = hipMalloc(&p[k], std::max<size_t>(bytes, 16));
    if (e == hipErrorOutOfMemory) {
      (void)hipGetLastError();
      if (reclaim_workspaces(nullptr)) e = hipMalloc(&p[k], std::max<size_t>(bytes, 16));
    }
    if (e != hipSuccess) {
      (void)hipGetLastError();
      p[k] = nullptr;
      raise(-2, "DF factors: device allocation of " + std::to_string(bytes) + " bytes failed");
    }
    return static_cast<char*>(p[k]);
  }
};

// Temporaries of exacc_df_factors_noalloc: one array per GPU, held from library
// load to process end.  Host code never passes the symbol itself to a kernel; it
// uses the device address hipGetSymbolAddress returns for the current device.
static __device__ __align__(256) unsigned char scratch[EXACC_DF_SCRATCH_BYTES];
std::mutex g_scratch_mu;
void* g_scratch_ptr[64] = {};

char* scratch_address() {
  int dev = 0;
  HIPCHECK(hipGetDevice(&dev));
  if (dev < 0 || dev >= 64) raise(-1, "DF factors (no allocation): device ordinal beyond 63");
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    HIPCHECK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    g_scratch_ptr[dev] = p;
  }
  return static_cast<char*>(g_scratch_ptr[dev]);
}

}  // namespace

int df_factors_impl(int m, int n, int X, const double* C, const double* J, const double* V, double* B,
                    bool on_device, hipStream_t s) {
  Owned own;
  const size_t bC = (size_t)m * n * 16, bJ = (size_t)X * m * m * 16, bV = (size_t)X * X * 8,
               bB = (size_t)X * n * n * 16;
  const double *Cd = C, *Jd = J, *Vd = V;
  double* Bd = B;
  if (!on_device) {
    char* c = own.alloc(0, bC);
    char* j = own.alloc(1, bJ);
    char* v = own.alloc(2, bV);
    HIPCHECK(hipMemcpyAsync(c, C, bC, hipMemcpyHostToDevice, s));
    HIPCHECK(hipMemcpyAsync(j, J, bJ, hipMemcpyHostToDevice, s));
    HIPCHECK(hipMemcpyAsync(v, V, bV, hipMemcpyHostToDevice, s));
    Cd = reinterpret_cast<double*>(c);
    Jd = reinterpret_cast<double*>(j);
    Vd = reinterpret_cast<double*>(v);
    Bd = reinterpret_cast<double*>(own.alloc(3, bB));
  }
  // every temporary in one region, no larger than its sizes need: allocations up to 16 MB
  // take 0.02 ms here, larger ones 0.3 ms and more (0.04 to allocate, 0.27 to free 70 MB)
  const size_t wsb = splitk_bytes(X);
  const Overlap ov = overlap(m, n, X, Cd, Jd, Bd);
  const size_t cap = fixed_bytes(X) + std::max(chunk_bytes(m, n, X), slice_bytes(m, n, X, 1)) + ov.c + ov.t1 + wsb;
  char* region = own.alloc(4, cap);
  // residues of the transforms' and the metric product's operands, where that gains and leaves
  // the device memory it takes to spare
  size_t mod_bytes = 0;
  if (mod_gemm_pays(n, (int64_t)X * m, m) || mod_gemm_pays(X, (int64_t)n * n, X)) {
    mod_bytes = (size_t)768 << 20;
    size_t fr = 0, tot = 0;
    HIPCHECK(hipMemGetInfo(&fr, &tot));
    if (2 * mod_bytes > fr || hipMalloc(&own.p[5], mod_bytes) != hipSuccess) {
      (void)hipGetLastError();
      own.p[5] = nullptr;
      mod_bytes = 0;
    }
  }
  const int iters = df_core(m, n, X, Cd, Jd, Vd, Bd, s, region, cap, wsb, true, own.p[5], mod_bytes);
  if (!on_device) {
    HIPCHECK(hipMemcpyAsync(B, Bd, bB, hipMemcpyDeviceToHost, s));
    HIPCHECK(hipStreamSynchronize(s));
  }
  return iters;
}

int df_factors_noalloc_impl(int m, int n, int X, const double* C, const double* J, const double* V,
                            double* B, hipStream_t s) {
  const size_t need = fixed_bytes(X) + slice_bytes(m, n, X, 1);
  if (need > (size_t)EXACC_DF_SCRATCH_BYTES)
    raise(-2, "DF factors (no allocation): naux = " + std::to_string(X) + ", nao = " + std::to_string(m) +
                  ", nspinor = " + std::to_string(n) + " need " + std::to_string(need) +
                  " bytes of scratch, above the static " + std::to_string((size_t)EXACC_DF_SCRATCH_BYTES));
  char* base = scratch_address();
  return df_core(m, n, X, C, J, V, B, s, base, (size_t)EXACC_DF_SCRATCH_BYTES, (size_t)64 << 20, false, nullptr, 0);
}

}  // namespace exacc
