// Forward of a small device split over time.
//
// The steps of a device below the gather engine's range (D < 64) are a serial
// chain of a few microseconds of one thread's work each (a 2-transmon gate:
// 16 columns in 16 lanes of one wave), and the chip is idle.  The map of a run
// of steps is a D x D matrix, so the steps are cut into up to 256 runs, one
// workgroup each propagates the identity over its run with the register-layout
// stepper (compensated FP32, the same stage tables), and the runs' matrices
// (hi + lo, exact in FP64) are multiplied onto the columns in FP64: first in
// groups of up to 16 by one workgroup each, then group after group per column.
// The sum over the steps of rounding errors is that of the stepper; the FP64
// products add none of FP32 size.
//
// Bound: the latency of one run (N / 256 steps) and of the two product kernels.
// 2 transmons, d = 4, the whole unitary, 1000 steps: 16.7 ms as a serial chain,
// 0.11 ms split.
#include <algorithm>

#include "kernel_common.h"

namespace scp {

scp_status launch_rk4_batched(int d, int NR, int MP, int ev, const FwdItem* items, int nitems, int wg,
                              size_t sh, bool recompute, hipStream_t s);

namespace {

constexpr int SP_MAXD = 63;        // larger devices have the gather engine
constexpr int SP_RUNS = 256;       // runs: one per compute unit
constexpr int SP_MINSTEPS = 64;    // below, the launches cost what the steps do

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct SpLayout {
  size_t items, ident, hi, lo, prod, total;
  int len, nrun, nwg, group, ngroup;
};

SpLayout sp_layout(const scp_system* sys) {
  SpLayout w{};
  const int N = sys->n_steps;
  const size_t D = (size_t)sys->D;
  w.len = (N + SP_RUNS - 1) / SP_RUNS;
  w.nrun = (N + w.len - 1) / w.len;
  w.nwg = (int)((D + sys->plan.CPW - 1) / sys->plan.CPW);
  w.group = 1;
  while (w.group * w.group < w.nrun) ++w.group;
  w.ngroup = (w.nrun + w.group - 1) / w.group;
  size_t o = 0;
  w.items = o;
  o = align256(o + (size_t)w.nrun * w.nwg * sizeof(FwdItem));
  w.ident = o;
  o = align256(o + D * D * sizeof(float2));
  w.hi = o;
  o = align256(o + (size_t)w.nrun * D * D * sizeof(float2));
  w.lo = o;
  o = align256(o + (size_t)w.nrun * D * D * sizeof(float2));
  w.prod = o;
  o = align256(o + (size_t)w.ngroup * D * D * sizeof(double2));
  w.total = o;
  return w;
}

// Work items (run c: steps [c len, (c + 1) len), its matrix at c D^2) and the
// identity columns.
__global__ void __launch_bounds__(256) sp_items_kernel(FwdItem base, FwdItem* __restrict__ items,
                                                       float2* __restrict__ ident, int nrun, int nwg,
                                                       int len, int N, int D) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < D * D) ident[t] = make_float2(t / D == t % D ? 1.f : 0.f, 0.f);
  if (t >= nrun * nwg) return;
  const int c = t / nwg;
  FwdItem I = base;
  I.state_hi = base.state_hi + (size_t)c * D * D;
  I.lo = base.lo + (size_t)c * D * D;
  I.cb = t - c * nwg;
  I.n0 = c * len;
  I.n1 = min(N, I.n0 + len);
  items[t] = I;
}

// Row of the stepper's register-order entry q of a column (q = r TPC + t).
__device__ __forceinline__ int sp_row(const Plan* P, int q) {
  const int r = q / P->TPC;
  int t = q - r * P->TPC, e = P->reg_off[P->L - 1][r];
  for (int k = 0; k < P->NT; ++k) {
    const int u = t / P->d;
    e += (t - u * P->d) * P->tstride[P->L - 1][k];
    t = u;
  }
  return e;
}

__device__ __forceinline__ void sp_cmac(double2& s, double2 a, double2 b) {
  s.x = fma(a.x, b.x, s.x);
  s.x = fma(-a.y, b.y, s.x);
  s.y = fma(a.x, b.y, s.y);
  s.y = fma(a.y, b.x, s.y);
}

// Product of the runs of group blockIdx.x, later runs on the left; column-major.
__global__ void __launch_bounds__(256) sp_group_kernel(const Plan* __restrict__ P,
                                                       const float2* __restrict__ hi,
                                                       const float2* __restrict__ lo, int nrun,
                                                       int group, int D, double2* __restrict__ prod) {
  extern __shared__ double2 sp_lds[];
  const int n = D * D, c0 = blockIdx.x * group, c1 = min(nrun, c0 + group);
  double2 *A = sp_lds, *B = sp_lds + n, *U = sp_lds + 2 * n;
  for (int c = c0; c < c1; ++c) {
    double2* dst = c == c0 ? A : U;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
      const int col = i / D;
      const float2 h = hi[(size_t)c * n + i], l = lo[(size_t)c * n + i];
      dst[col * D + sp_row(P, i - col * D)] =
          make_double2((double)h.x + (double)l.x, (double)h.y + (double)l.y);
    }
    __syncthreads();
    if (c == c0) continue;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
      const int col = i / D, row = i - col * D;
      double2 s = make_double2(0.0, 0.0);
      for (int k = 0; k < D; ++k) sp_cmac(s, U[k * D + row], A[col * D + k]);
      B[i] = s;
    }
    __syncthreads();
    double2* t = A;
    A = B;
    B = t;
  }
  for (int i = threadIdx.x; i < n; i += blockDim.x) prod[(size_t)blockIdx.x * n + i] = A[i];
}

// psiT = product of the groups times psi0, one wave per column.
__global__ void __launch_bounds__(64) sp_apply_kernel(const double2* __restrict__ prod, int ngroup,
                                                      int D, const float2* psi0, float2* psiT) {
  __shared__ double2 x[2][64];
  const int e = threadIdx.x;
  const size_t at = (size_t)blockIdx.x * D + e;
  double2 v = make_double2(0.0, 0.0);
  if (e < D) v = make_double2(psi0[at].x, psi0[at].y);
  x[0][e] = v;
  __syncthreads();
  for (int g = 0; g < ngroup; ++g) {
    const double2* M = prod + (size_t)g * D * D;
    double2 s = make_double2(0.0, 0.0);
    if (e < D)
      for (int k = 0; k < D; ++k) sp_cmac(s, M[k * D + e], x[g & 1][k]);
    v = s;
    x[(g & 1) ^ 1][e] = v;
    __syncthreads();
  }
  if (e < D) psiT[at] = make_float2((float)v.x, (float)v.y);
}

}  // namespace

// The automatic choice for a forward without checkpoints: D < 64 and enough
// steps.  (A forward with checkpoints needs the states between the runs.)
bool split_preferred(const scp_system* sys) {
  return sys->D <= SP_MAXD && sys->n_steps >= SP_MINSTEPS;
}

size_t split_workspace_bytes(const scp_system* sys) { return sp_layout(sys).total; }

scp_status launch_split_forward(scp_system* sys, int S, void* ws, const float2* psi0, float2* psiT,
                                hipStream_t st) {
  const SpLayout w = sp_layout(sys);
  const Plan& P = sys->plan;
  const int D = (int)sys->D;
  char* b = static_cast<char*>(ws);
  FwdItem* items = reinterpret_cast<FwdItem*>(b + w.items);
  float2* ident = reinterpret_cast<float2*>(b + w.ident);
  float2* hi = reinterpret_cast<float2*>(b + w.hi);
  float2* lo = reinterpret_cast<float2*>(b + w.lo);
  double2* prod = reinterpret_cast<double2*>(b + w.prod);
  hipEvent_t t0 = timing_start(sys, st);
  const FwdItem base{sys->d_plan, sys->d_ops, sys->d_ctab, ident, nullptr, hi, lo, nullptr, nullptr,
                     nullptr, sys->d_ph, sys->d_rops, 1, D, 0, 0, 0, 0};
  const int n = std::max(D * D, w.nrun * w.nwg);
  hipLaunchKernelGGL(sp_items_kernel, dim3((n + 255) / 256), dim3(256), 0, st, base, items, ident,
                     w.nrun, w.nwg, w.len, sys->n_steps, D);
  HIPCHK(hipGetLastError());
  scp_status s = launch_rk4_batched(P.d, P.NR, P.MP, plan_eval(P), items, w.nrun * w.nwg, P.WG,
                                    sizeof(c32) * 3 * (size_t)P.CPW * P.D, false, st);
  if (s != SCP_OK) return s;
  hipLaunchKernelGGL(sp_group_kernel, dim3(w.ngroup), dim3(256), 3 * (size_t)D * D * sizeof(double2), st,
                     sys->d_plan, hi, lo, w.nrun, w.group, D, prod);
  HIPCHK(hipGetLastError());
  hipLaunchKernelGGL(sp_apply_kernel, dim3(S), dim3(64), 0, st, prod, w.ngroup, D, psi0, psiT);
  HIPCHK(hipGetLastError());
  timing_stop(sys, t0, 0, st);
  return SCP_OK;
}

}  // namespace scp
