// Gather engine, real form of a closed system's forward and adjoint.
//
// Where every term is real (the real frame), every operator is odd (parity),
// the coupled pairs are neighbours on a chain or ring of the modes with two
// couplings each at most, and a driven mode has one operator, the generator is
// V(t) = P(t) R(t) P(t)^dag with P the diagonal of frame phases and R real.  The coefficients of R do not depend on
// time but for the drives' c_k(t): each thread holds those of its own elements
// (in registers where a thread has one or few, else read from LDS rows), and a
// stage needs no table but one phase per element and half step,
// read a stage ahead.  The strides of the neighbours are compile-time offsets
// of the LDS reads.
//
// Bound: vector instruction issue and LDS reads of a column's one workgroup,
// with a barrier per stage.  Against the complex rows of g_apply a gather costs
// two multiply-adds instead of four and no coefficient read.
// Measured, complex rows (g_apply, g_adj_body) -> here: 4-fluxonium chain
// (d = 5, 16 columns) forward 8.4 -> 4.0 us per step, forward + gradient
// 29 -> 19.5; 5-transmon ring (32 columns) forward + gradient 21 -> 8.4.  Rows
// shared by a thread's elements (SHARE), each element's own -> here: 6-fluxonium
// chain (d = 4, 64 columns) forward 25 -> 17, sweep the same, segments 48 -> 41.
// Error of the final states against FP64 over rings and chains of 3 to 5 modes:
// 6e-8 to 1e-7 -> 2e-8 to 1e-7 (real_kappa in gather.hip has the reason).
#include <cstring>

#include "gather.h"

namespace scp {

namespace {

template <int d, int N>
struct RShape {
  using Sh = GShape<d, N, false>;
  static constexpr int n = Nb<d, true>::n, nn = n * n;
  static constexpr int pr = nn == 9 ? 12 : nn;   // row strides of the static table (floats)
  static constexpr int dr = n == 3 ? 4 : n;
  static constexpr int off_d = N * d * d * pr;
  static constexpr int total = off_d + N * d * dr;
  // gradient rows, behind the static ones: per mode, operator (two at most)
  // and level [O, dO/dEJ, dO/dEC, dO/dEL] (n entries each), then per mode and
  // level d eps/d(EJ, EC, EL)
  static constexpr int gr = (4 * n + 3) / 4 * 4;
  static constexpr int off_g = (total + 3) & ~3;
  static constexpr int off_e = N * 2 * d * gr;
  static constexpr int gtotal = off_e + N * d * 4;
  static constexpr bool REGC = Sh::E * N * (nn + n) <= 64;
  static constexpr int pi(int p) { return p == N - 1 ? 0 : p; }       // modes of pair p
  static constexpr int pj(int p) { return p == N - 1 ? N - 1 : p + 1; }
  static size_t seg_lds_bytes() {
    return sizeof(c32) * 2 * (size_t)Sh::L +
           sizeof(float) * ((size_t)(REGC ? 0 : off_g) + gtotal + 2 * (Sh::T / 64) * GA_NV);
  }
  static size_t lds_bytes() {
    return sizeof(c32) * 2 * (size_t)Sh::L + (REGC ? 0 : sizeof(float) * (size_t)((total + 3) & ~3));
  }
};

// An element's digits and the LDS offsets of its neighbours: along mode m the
// first one at o[m], the last one l[m] after it (d odd: lane-dependent), those
// between at even multiples of the stride.
template <int d, int N>
struct RElem {
  int o[N], l[N];
  __device__ __forceinline__ void set(uint32_t pk) {
    using R = RShape<d, N>;
#pragma unroll
    for (int m = 0; m < N; ++m) {
      const int a = ket_digit(pk, m), st = R::Sh::st(m);
      o[m] = (a & 1) ? -a * st : (1 - a) * st;
      l[m] = (d & 1) && !(a & 1) ? 0 : 2 * (R::n - 1) * st;
    }
  }
  __device__ __forceinline__ int at(int k, int m) const {
    using R = RShape<d, N>;
    if (k == 0) return 0;
    if (k == R::n - 1 && (d & 1)) return l[m];
    return 2 * k * R::Sh::st(m);
  }
};

// Static coefficients of one element: pair rows and drive rows.
template <int d, int N>
struct RCoef {
  using R = RShape<d, N>;
  float g[N][R::nn], o[N][R::n];
};

template <int d, int N>
__device__ __forceinline__ void r_coef(const float* __restrict__ tab, uint32_t pk, RCoef<d, N>& C) {
  using R = RShape<d, N>;
#pragma unroll
  for (int p = 0; p < N; ++p) {
    const int row = ket_digit(pk, R::pi(p)) * d + ket_digit(pk, R::pj(p));
    g_row<R::nn, R::pr>(tab + (p * d * d + row) * R::pr, C.g[p]);
    g_row<R::n, R::dr>(tab + R::off_d + (p * d + ket_digit(pk, p)) * R::dr, C.o[p]);
  }
}

// k = R y at one element (ye: the element's place in LDS, y its own value).
template <int d, int N>
__device__ __forceinline__ void r_apply(const c32* __restrict__ ye, const RElem<d, N>& El,
                                        const RCoef<d, N>& C, const float* c, int pmask, int dmask,
                                        float dg, c32 y, float& kr, float& ki) {
  using R = RShape<d, N>;
  kr = dg * y.x;
  ki = dg * y.y;
#pragma unroll
  for (int p = 0; p < N; ++p) {
    if (!((pmask >> p) & 1)) continue;
    const int i = R::pi(p), j = R::pj(p);
    const c32* q = ye + (El.o[i] + El.o[j]);
#pragma unroll
    for (int x = 0; x < R::n; ++x)
#pragma unroll
      for (int z = 0; z < R::n; ++z) {
        const c32 v = q[El.at(x, i) + El.at(z, j)];
        kr = fmaf(C.g[p][x * R::n + z], v.x, kr);
        ki = fmaf(C.g[p][x * R::n + z], v.y, ki);
      }
  }
#pragma unroll
  for (int m = 0; m < N; ++m) {
    if (!((dmask >> m) & 1)) continue;
    const c32* q = ye + El.o[m];
    float sr = 0.f, si = 0.f;
#pragma unroll
    for (int x = 0; x < R::n; ++x) {
      const c32 v = q[El.at(x, m)];
      sr = fmaf(C.o[m][x], v.x, sr);
      si = fmaf(C.o[m][x], v.y, si);
    }
    kr = fmaf(c[m], sr, kr);
    ki = fmaf(c[m], si, ki);
  }
}

// What a thread keeps of its elements and of the drives.
template <int d, int N>
struct RThread {
  using Sh = GShape<d, N, false>;
  static constexpr int E = Sh::E, T = Sh::T, L = Sh::L;
  static constexpr bool REGC = RShape<d, N>::REGC;
  // The thread's elements differ in mode 0's digit alone (element r has level
  // r): the rows and offsets of the other modes are the same for all of them
  // and are formed once per term, and what reads along mode 0 takes each
  // neighbour once, or from the thread's own elements.
  static constexpr bool SHARE = !REGC && E == d && E * T == L;
  uint32_t pk[E];
  float dg[E];
  RCoef<d, N> C[REGC ? E : 1];
  RElem<d, N> El[REGC ? E : 1];
  const float* rt;         // static rows in LDS (REGC: unused)
  const c32* ph;
  const float* rc;
  int pmask, dmask, zero;

  __device__ __forceinline__ void init(kptr<GArgs> A, float* lds_tab) {
    const int tid = threadIdx.x;
    ph = (const c32*)A->ph;
    rc = A->rc;
    pmask = uni(A->pmask);
    dmask = uni(A->dmask);
    // the drive coefficients are read by vector loads (a lane-dependent zero
    // in the index), which a wave may have in flight across its LDS reads
    zero = 0;
    asm volatile("" : "+v"(zero));
    rt = lds_tab;
    if (!REGC)
      for (int t = tid; t < RShape<d, N>::total; t += T) lds_tab[t] = A->rt[t];
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const int e = tid + r * T;
      uint32_t p = 0;
      float g = 0.f;
#pragma unroll
      for (int m = 0; m < N; ++m) {
        const int a = (e / Sh::st(m)) % d;
        p |= (uint32_t)a << (3 * m);
        g += A->delta[m][a];
      }
      pk[r] = p;
      dg[r] = (float)(A->kappa * g);
      if constexpr (REGC) {
        r_coef<d, N>(A->rt, p, C[r]);
        El[r].set(p);
      }
    }
  }
  // k = R y for element r, the stage input in buffer yb
  __device__ __forceinline__ void apply(int r, const c32* yb, const float* c, c32 y, float& kr,
                                        float& ki) const {
    int e = threadIdx.x + r * T;
    if constexpr (REGC) {
      r_apply<d, N>(yb + e, El[r], C[r], c, pmask, dmask, dg[r], y, kr, ki);
    } else {
      // opaque per stage: offsets and rows are formed inside the stage
      uint32_t p = pk[r];
      asm volatile("" : "+v"(p));
      RCoef<d, N> Cc;
      RElem<d, N> Ee;
      r_coef<d, N>(rt, p, Cc);
      Ee.set(p);
      r_apply<d, N>(yb + e, Ee, Cc, c, pmask, dmask, dg[r], y, kr, ki);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // k = R y for all the thread's elements (y: their values of the stage input in
  // yb), the sums of an element in the order of apply()
  __device__ __forceinline__ void apply_all(const c32* yb, const float* c, const c32 (&y)[E],
                                            c32 (&k)[E]) const {
    if constexpr (SHARE) {
      using R = RShape<d, N>;
      constexpr int n = R::n;
      uint32_t p0 = pk[0];
      asm volatile("" : "+v"(p0));   // opaque per stage: offsets and rows are formed inside it
      RElem<d, N> El;
      El.set(p0);
      const c32* ye = yb + threadIdx.x;
#pragma unroll
      for (int r = 0; r < E; ++r) {
        k[r].x = dg[r] * y[r].x;
        k[r].y = dg[r] * y[r].y;
      }
      static_for<N>([&](auto P) {
        constexpr int p = decltype(P)::value, i = R::pi(p), j = R::pj(p);
        if (!((pmask >> p) & 1)) return;
        if constexpr (i > 0) {
          float g[R::nn];
          g_row<R::nn, R::pr>(rt + (p * d * d + ket_digit(p0, i) * d + ket_digit(p0, j)) * R::pr, g);
          const c32* q = ye + (El.o[i] + El.o[j]);
#pragma unroll
          for (int r = 0; r < E; ++r)
#pragma unroll
            for (int x = 0; x < n; ++x)
#pragma unroll
              for (int z = 0; z < n; ++z) {
                const c32 v = q[El.at(x, i) + El.at(z, j) + r * T];
                k[r].x = fmaf(g[x * n + z], v.x, k[r].x);
                k[r].y = fmaf(g[x * n + z], v.y, k[r].y);
              }
        } else {
          const c32* q = ye + El.o[j];
          c32 v[d][n];
#pragma unroll
          for (int b = 0; b < d; ++b)
#pragma unroll
            for (int z = 0; z < n; ++z) v[b][z] = q[El.at(z, j) + b * T];
#pragma unroll
          for (int r = 0; r < E; ++r) {
            float g[R::nn];
            g_row<R::nn, R::pr>(rt + (p * d * d + r * d + ket_digit(p0, j)) * R::pr, g);
#pragma unroll
            for (int x = 0; x < n; ++x) {
              const int b = ((r & 1) ^ 1) + 2 * x;
              if (b >= d) continue;
#pragma unroll
              for (int z = 0; z < n; ++z) {
                k[r].x = fmaf(g[x * n + z], v[b][z].x, k[r].x);
                k[r].y = fmaf(g[x * n + z], v[b][z].y, k[r].y);
              }
            }
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      });
      static_for<N>([&](auto M) {
        constexpr int m = decltype(M)::value;
        if (!((dmask >> m) & 1)) return;
        float o[n];
        if constexpr (m > 0) g_row<n, R::dr>(rt + R::off_d + (m * d + ket_digit(p0, m)) * R::dr, o);
        const c32* q = ye + El.o[m];
#pragma unroll
        for (int r = 0; r < E; ++r) {
          float sr = 0.f, si = 0.f;
          if constexpr (m == 0) g_row<n, R::dr>(rt + R::off_d + r * R::dr, o);
#pragma unroll
          for (int x = 0; x < n; ++x) {
            const int b = ((r & 1) ^ 1) + 2 * x;
            if (m == 0 && b >= d) continue;
            const c32 v = m == 0 ? y[b < d ? b : 0] : q[El.at(x, m) + r * T];
            sr = fmaf(o[x], v.x, sr);
            si = fmaf(o[x], v.y, si);
          }
          k[r].x = fmaf(c[m], sr, k[r].x);
          k[r].y = fmaf(c[m], si, k[r].y);
        }
        __builtin_amdgcn_sched_barrier(0);
      });
    }
  }
  __device__ __forceinline__ void phases(int q, c32 (&P)[E]) const {
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const int e = threadIdx.x + r * T;
      P[r] = ph[(size_t)q * L + (e < L ? e : 0)];
    }
  }
  __device__ __forceinline__ void drives(int row, float (&c)[N]) const {
#pragma unroll
    for (int m = 0; m < N; ++m)
      if ((dmask >> m) & 1) c[m] = rc[row * N + m + zero];
  }
};

// One column of a forward propagation (arguments as g_rk4_body).
template <int d, int N, bool CK>
__device__ __forceinline__ void g_real_rk4_body(const GArgs* __restrict__ Ag,
                                                const GAdj* __restrict__ Bg, int col, int n_lo,
                                                int n_hi, const float4* __restrict__ st_in,
                                                float4* __restrict__ st_out) {
  using Sh = GShape<d, N, false>;
  constexpr int L = Sh::L, T = Sh::T, E = Sh::E;
  extern __shared__ __align__(16) c32 lds[];
  kptr<GArgs> A = kconst(Ag);
  const int tid = threadIdx.x;
  const float h = A->h;
  const int nsteps = A->nsteps;
  RThread<d, N> Th;
  Th.init(A, reinterpret_cast<float*>(lds + 2 * L));
  float hr[E], hm[E], lr[E], lm[E], ar[E], ai[E];
  c32 P0[E], P1[E], P2[E], y[E];   // phases of rows 2n, 2n + 1, 2n + 2; the stage input
  float c0[N], c1[N], c2[N];       // drive coefficients of rows 3n, 3n + 1, 3n + 2
#pragma unroll
  for (int m = 0; m < N; ++m) c0[m] = c1[m] = c2[m] = 0.f;
  Th.phases(2 * n_lo, P0);
  Th.phases(2 * n_lo + 1, P1);
  Th.drives(3 * n_lo, c0);
  Th.drives(3 * n_lo + 1, c1);
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const int e = tid + r * T;
    hr[r] = hm[r] = lr[r] = lm[r] = ar[r] = ai[r] = 0.f;
    if (e < L) {
      if (st_in != nullptr) {
        const float4 q = st_in[(size_t)col * L + e];
        hr[r] = q.x;
        hm[r] = q.y;
        lr[r] = q.z;
        lm[r] = q.w;
      } else {
        const c32 v = ((const c32*)A->x0)[(size_t)col * L + e];
        hr[r] = v.x;
        hm[r] = v.y;
      }
    }
    c32 v;
    v.x = hr[r];
    v.y = hm[r];
    y[r] = c_mul_conj(P0[r], v);
    if (e < L) lds[e] = y[r];
  }
  __syncthreads();
  int cur = 0;
#pragma unroll 1
  for (int n = n_lo; n < n_hi; ++n) {
    if (CK) {
      kptr<GAdj> B = kconst(Bg);
      const int ce = B->ce;
      if (n % ce == 0) {
        float4* ck = B->ck + ((size_t)col * B->nck + n / ce) * L;
#pragma unroll
        for (int r = 0; r < E; ++r) {
          const int e = tid + r * T;
          if (e < L) ck[e] = make_float4(hr[r], hm[r], lr[r], lm[r]);
        }
      }
    }
    const int nx = min(n + 1, nsteps - 1);
    Th.phases(2 * n + 2, P2);
    Th.drives(3 * n + 2, c2);
    static_for<4>([&](auto Sc) {
      constexpr int s = decltype(Sc)::value;
      constexpr float w = (s == 0 || s == 3) ? 1.f : 2.f;
      const float ch = s == 2 ? h : 0.5f * h;
      const c32* yc = lds + cur * L;
      c32* yn = lds + (cur ^ 1) * L;
      c32 ks[E];
      if constexpr (RThread<d, N>::SHARE) Th.apply_all(yc, s == 0 ? c0 : (s == 3 ? c2 : c1), y, ks);
#pragma unroll
      for (int r = 0; r < E; ++r) {
        const int e = tid + r * T;
        float kr, ki;
        if (e < L) {
          c32 u;
          if constexpr (RThread<d, N>::SHARE) u = ks[r];
          else Th.apply(r, yc, s == 0 ? c0 : (s == 3 ? c2 : c1), y[r], u.x, u.y);
          u = c_mul(s == 0 ? P0[r] : (s == 3 ? P2[r] : P1[r]), u);
          kr = u.y;    // k = -i P R P^dag y
          ki = -u.x;
          ar[r] = s == 0 ? kr : fmaf(w, kr, ar[r]);
          ai[r] = s == 0 ? ki : fmaf(w, ki, ai[r]);
          c32 v;
          if (s < 3) {
            v.x = fmaf(ch, kr, hr[r]);
            v.y = fmaf(ch, ki, hm[r]);
          } else {
            const float h6 = h * (1.0f / 6.0f);
            comp_add(hr[r], lr[r], h6 * ar[r]);
            comp_add(hm[r], lm[r], h6 * ai[r]);
            v.x = hr[r];
            v.y = hm[r];
          }
          y[r] = c_mul_conj(s < 2 ? P1[r] : P2[r], v);
          yn[e] = y[r];
        }
      }
      if (s == 0) Th.drives(3 * nx, c0);
      if (s == 2) {
        Th.phases(2 * nx + 1, P1);
        Th.drives(3 * nx + 1, c1);
      }
      __syncthreads();
      cur ^= 1;
    });
#pragma unroll
    for (int r = 0; r < E; ++r) P0[r] = P2[r];
  }
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const int e = tid + r * T;
    if (e >= L) continue;
    if (st_out != nullptr) st_out[(size_t)col * L + e] = make_float4(hr[r], hm[r], lr[r], lm[r]);
    if (A->xT != nullptr && n_hi == nsteps) {
      c32 v;
      v.x = hr[r] + lr[r];
      v.y = hm[r] + lm[r];
      ((c32*)A->xT)[(size_t)col * L + e] = v;
    }
  }
}

// One column of a costate sweep (arguments as g_cos_body).
template <int d, int N>
__device__ __forceinline__ void g_real_cos_body(const GArgs* __restrict__ Ag,
                                                const GAdj* __restrict__ Bg, int col, int g_hi,
                                                int g_lo) {
  using Sh = GShape<d, N, false>;
  constexpr int L = Sh::L, T = Sh::T, E = Sh::E;
  extern __shared__ __align__(16) c32 lds[];
  kptr<GArgs> A = kconst(Ag);
  kptr<GAdj> B = kconst(Bg);
  const int tid = threadIdx.x;
  const float h = A->h;
  const int nsteps = A->nsteps, ce = B->ce, nck = B->nck;
  float4* lam = B->lam + (size_t)col * nck * L;
  float lhr[E], lhm[E], llr[E], llm[E];
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const int e = tid + r * T;
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (e < L) {
      if (g_hi == nck - 1) {
        const c32 c = ((const c32*)B->cot)[(size_t)col * L + e];
        v = make_float4(c.x, c.y, 0.f, 0.f);
        lam[(size_t)g_hi * L + e] = v;
      } else {
        v = lam[(size_t)g_hi * L + e];
      }
    }
    lhr[r] = v.x;
    lhm[r] = v.y;
    llr[r] = v.z;
    llm[r] = v.w;
  }
  if (g_hi <= 0) return;   // the first segment's start is not needed
  const int n_hi = min(nsteps, (g_hi + 1) * ce), n_lo = max(g_lo, 1) * ce;
  RThread<d, N> Th;
  Th.init(A, reinterpret_cast<float*>(lds + 2 * L));
  c32 P0[E], P1[E], P2[E];
  float c0[N], c1[N], c2[N];
#pragma unroll
  for (int m = 0; m < N; ++m) c0[m] = c1[m] = c2[m] = 0.f;
  Th.phases(2 * n_hi, P2);
  Th.phases(2 * n_hi - 1, P1);
  Th.drives(3 * n_hi - 1, c2);
  Th.drives(3 * n_hi - 2, c1);
  int cur = 0;
#pragma unroll 1
  for (int n = n_hi - 1; n >= n_lo; --n) {
    const int nx = max(n - 1, 0);
    Th.phases(2 * n, P0);
    Th.drives(3 * n, c0);
    float ybr[E], ybm[E];
#pragma unroll
    for (int r = 0; r < E; ++r) ybr[r] = ybm[r] = 0.f;
    static_for<4>([&](auto Sc) {
      constexpr int s = 3 - decltype(Sc)::value;
      const float cs = (s == 0 || s == 3 ? 1.f : 2.f) * (h * (1.0f / 6.0f));
      const float cy = s == 3 ? 0.f : (s == 2 ? h : 0.5f * h);
      c32* kbw = lds + cur * L;
      c32 kb[E];
#pragma unroll
      for (int r = 0; r < E; ++r) {
        const int e = tid + r * T;
        c32 v;
        v.x = s == 3 ? cs * lhr[r] : fmaf(cs, lhr[r], cy * ybr[r]);
        v.y = s == 3 ? cs * lhm[r] : fmaf(cs, lhm[r], cy * ybm[r]);
        kb[r] = c_mul_conj(s == 0 ? P0[r] : (s == 3 ? P2[r] : P1[r]), v);
        if (e < L) kbw[e] = kb[r];
      }
      __syncthreads();
      c32 ks[E];
      if constexpr (RThread<d, N>::SHARE) Th.apply_all(kbw, s == 0 ? c0 : (s == 3 ? c2 : c1), kb, ks);
#pragma unroll
      for (int r = 0; r < E; ++r) {
        const int e = tid + r * T;
        if (e < L) {
          c32 u;
          if constexpr (RThread<d, N>::SHARE) u = ks[r];
          else Th.apply(r, kbw, s == 0 ? c0 : (s == 3 ? c2 : c1), kb[r], u.x, u.y);
          u = c_mul(s == 0 ? P0[r] : (s == 3 ? P2[r] : P1[r]), u);
          ybr[r] = -u.y;   // yb = i P R P^dag kb
          ybm[r] = u.x;
          llr[r] -= u.y;
          llm[r] += u.x;
        }
      }
      if (s == 3) Th.drives(3 * nx + 2, c2);
      if (s == 1) {
        Th.phases(2 * nx + 1, P1);
        Th.drives(3 * nx + 1, c1);
      }
      cur ^= 1;
    });
#pragma unroll
    for (int r = 0; r < E; ++r) {
      float t = lhr[r] + llr[r];
      llr[r] -= t - lhr[r];
      lhr[r] = t;
      t = lhm[r] + llm[r];
      llm[r] -= t - lhm[r];
      lhm[r] = t;
      P2[r] = P0[r];
    }
    if (n % ce == 0) {
#pragma unroll
      for (int r = 0; r < E; ++r) {
        const int e = tid + r * T;
        if (e < L) lam[(size_t)(n / ce - 1) * L + e] = make_float4(lhr[r], lhm[r], llr[r], llm[r]);
      }
    }
  }
}

// Segment gseg of column col: its recompute from the checkpoint, the rotated
// stage inputs y' = P^dag y kept in buffer slot, then its reverse walk from the
// costate the sweep left.  Both repeat the arithmetic of the forward and of the
// sweep, so the split into segments leaves no trace in the result.
//
// Sensitivities, with kb' = P^dag kb: 2 Im <kb', dR y'> = 2 sum Im(conj(dR kb') y'),
// R and its derivatives being real symmetric, so kb' is gathered and y' is the
// element's own value.  A coupling A (x) B needs per element the neighbours'
// partial sums r[x] = sum_z B_z kb'[x, z] along one mode and their counterpart
// along the other, w = Im(conj(r) y'), and the dot products of w with A and dA.
template <int d, int N>
__device__ __forceinline__ void g_real_seg_body(const GArgs* __restrict__ Ag,
                                                const GAdj* __restrict__ Bg, int gseg, int col,
                                                int slot) {
  using Sh = GShape<d, N, false>;
  using R = RShape<d, N>;
  constexpr int L = Sh::L, T = Sh::T, E = Sh::E, n_ = R::n, NW = T / 64;
  extern __shared__ __align__(16) c32 lds[];
  kptr<GArgs> A = kconst(Ag);
  kptr<GAdj> B = kconst(Bg);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float h = A->h;
  const int nsteps = A->nsteps, ce = B->ce, nck = B->nck;
  const int nds = uni(A->nds), ncp = uni(A->ncp), nv = 3 * N + ncp;
  const int n0 = gseg * ce, n1 = min(nsteps, n0 + ce);
  float* tab = reinterpret_cast<float*>(lds + 2 * L);
  float* gt = tab + (R::REGC ? 0 : R::off_g);   // gradient rows
  float* wsum = gt + R::gtotal;
  c32* segc = (c32*)B->seg + (size_t)slot * ce * 4 * L;
  RThread<d, N> Th;
  Th.init(A, tab);
  for (int t = tid; t < R::gtotal; t += T) gt[t] = A->rt[R::off_g + t];
  // ---- recompute
  {
    float hr[E], hm[E], lr[E], lm[E], ar[E], ai[E];
    c32 P0[E], P1[E], P2[E], y[E];
    float c0[N], c1[N], c2[N];
#pragma unroll
    for (int m = 0; m < N; ++m) c0[m] = c1[m] = c2[m] = 0.f;
    Th.phases(2 * n0, P0);
    Th.phases(2 * n0 + 1, P1);
    Th.drives(3 * n0, c0);
    Th.drives(3 * n0 + 1, c1);
    const float4* ck = B->ck + ((size_t)col * nck + gseg) * L;
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const int e = tid + r * T;
      float4 q = make_float4(0.f, 0.f, 0.f, 0.f);
      if (e < L) q = ck[e];
      hr[r] = q.x;
      hm[r] = q.y;
      lr[r] = q.z;
      lm[r] = q.w;
      ar[r] = ai[r] = 0.f;
      c32 v;
      v.x = q.x;
      v.y = q.y;
      y[r] = c_mul_conj(P0[r], v);
      if (e < L) {
        lds[e] = y[r];
        segc[e] = y[r];
      }
    }
    __syncthreads();
    int cur = 0;
#pragma unroll 1
    for (int n = n0; n < n1; ++n) {
      const int nx = min(n + 1, nsteps - 1);
      Th.phases(2 * n + 2, P2);
      Th.drives(3 * n + 2, c2);
      static_for<4>([&](auto Sc) {
        constexpr int s = decltype(Sc)::value;
        constexpr float w = (s == 0 || s == 3) ? 1.f : 2.f;
        const float ch = s == 2 ? h : 0.5f * h;
        const c32* yc = lds + cur * L;
        c32* yn = lds + (cur ^ 1) * L;
        c32* ys = segc + ((size_t)(n - n0) * 4 + s + 1) * L;   // the next stage's input
        const bool keep = s < 3 || n + 1 < n1;
        c32 ks[E];
        if constexpr (RThread<d, N>::SHARE) Th.apply_all(yc, s == 0 ? c0 : (s == 3 ? c2 : c1), y, ks);
#pragma unroll
        for (int r = 0; r < E; ++r) {
          const int e = tid + r * T;
          float kr, ki;
          if (e < L) {
            c32 u;
            if constexpr (RThread<d, N>::SHARE) u = ks[r];
            else Th.apply(r, yc, s == 0 ? c0 : (s == 3 ? c2 : c1), y[r], u.x, u.y);
            u = c_mul(s == 0 ? P0[r] : (s == 3 ? P2[r] : P1[r]), u);
            kr = u.y;
            ki = -u.x;
            ar[r] = s == 0 ? kr : fmaf(w, kr, ar[r]);
            ai[r] = s == 0 ? ki : fmaf(w, ki, ai[r]);
            c32 v;
            if (s < 3) {
              v.x = fmaf(ch, kr, hr[r]);
              v.y = fmaf(ch, ki, hm[r]);
            } else {
              const float h6 = h * (1.0f / 6.0f);
              comp_add(hr[r], lr[r], h6 * ar[r]);
              comp_add(hm[r], lm[r], h6 * ai[r]);
              v.x = hr[r];
              v.y = hm[r];
            }
            y[r] = c_mul_conj(s < 2 ? P1[r] : P2[r], v);
            yn[e] = y[r];
            if (keep) ys[e] = y[r];
          }
        }
        if (s == 0) Th.drives(3 * nx, c0);
        if (s == 2) {
          Th.phases(2 * nx + 1, P1);
          Th.drives(3 * nx + 1, c1);
        }
        __syncthreads();
        cur ^= 1;
      });
#pragma unroll
      for (int r = 0; r < E; ++r) P0[r] = P2[r];
    }
  }
  // ---- reverse walk
  float lhr[E], lhm[E], llr[E], llm[E];
  c32 P0[E], P1[E], P2[E], yp[E];
  float c0[N], c1[N], c2[N];
#pragma unroll
  for (int m = 0; m < N; ++m) c0[m] = c1[m] = c2[m] = 0.f;
  Th.phases(2 * n1, P2);
  Th.phases(2 * n1 - 1, P1);
  Th.drives(3 * n1 - 1, c2);
  Th.drives(3 * n1 - 2, c1);
  {
    const float4* lam = B->lam + ((size_t)col * nck + gseg) * L;
    const c32* ys = segc + ((size_t)(n1 - 1 - n0) * 4 + 3) * L;
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const int e = tid + r * T;
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
      yp[r].x = yp[r].y = 0.f;
      if (e < L) {
        v = lam[e];
        yp[r] = ys[e];
      }
      lhr[r] = v.x;
      lhm[r] = v.y;
      llr[r] = v.z;
      llm[r] = v.w;
    }
  }
  int prev_n = -1, prev_s = 0, par = 0, cur = 0;
  double vstep = 0.0;
  // the previous stage's per-wave sums into the step's row (as g_adj_body)
  auto fold_prev = [&]() {
    if (tid >= nds + nv) return;
    const int k = tid < nds ? tid : GA_MAXDS + tid - nds;
    double G = 0.0;
    for (int w = 0; w < NW; ++w) G += (double)wsum[((par ^ 1) * NW + w) * GA_NV + k];
    G *= A->kappa;   // the sums are those of the unscaled operators
    double* row = B->gs + ((size_t)col * nsteps + prev_n) * B->gw;
    if (tid < nds) {
      row[prev_s * nds + tid] = G;
    } else {
      vstep = prev_s == 3 ? G : vstep + G;
      if (prev_s == 0) row[3 * nds + tid] = vstep;
    }
  };
#pragma unroll 1
  for (int n = n1 - 1; n >= n0; --n) {
    const int nx = max(n - 1, 0);
    Th.phases(2 * n, P0);
    Th.drives(3 * n, c0);
    float ybr[E], ybm[E];
#pragma unroll
    for (int r = 0; r < E; ++r) ybr[r] = ybm[r] = 0.f;
    // the stages in a rolled loop: the sensitivities are long code
#pragma unroll 1
    for (int s = 3; s >= 0; --s) {
      const float cs = (s == 0 || s == 3 ? 1.f : 2.f) * (h * (1.0f / 6.0f));
      const float cy = s == 2 ? h : 0.5f * h;
      c32* kbw = lds + cur * L;
      c32 kb[E], P[E], y[E];
      float c[N];
#pragma unroll
      for (int m = 0; m < N; ++m) c[m] = s == 0 ? c0[m] : (s == 3 ? c2[m] : c1[m]);
#pragma unroll
      for (int r = 0; r < E; ++r) {
        const int e = tid + r * T;
        P[r] = s == 0 ? P0[r] : (s == 3 ? P2[r] : P1[r]);
        y[r] = yp[r];
        c32 v;
        v.x = s == 3 ? cs * lhr[r] : fmaf(cs, lhr[r], cy * ybr[r]);
        v.y = s == 3 ? cs * lhm[r] : fmaf(cs, lhm[r], cy * ybm[r]);
        kb[r] = c_mul_conj(P[r], v);
        if (e < L) kbw[e] = kb[r];
      }
      __syncthreads();
      {   // the walk's next stage input, (n, s - 1) or (n - 1, 3)
        const int at = (n - n0) * 4 + s - 1;
        if (at >= 0) {
          const c32* ys = segc + (size_t)at * L;
#pragma unroll
          for (int r = 0; r < E; ++r) {
            const int e = tid + r * T;
            if (e < L) yp[r] = ys[e];
          }
        }
      }
      if (prev_n >= 0) fold_prev();
      c32 ks[E];
      if constexpr (RThread<d, N>::SHARE) Th.apply_all(kbw, c, kb, ks);
#pragma unroll
      for (int r = 0; r < E; ++r) {
        const int e = tid + r * T;
        if (e < L) {
          c32 u;
          if constexpr (RThread<d, N>::SHARE) u = ks[r];
          else Th.apply(r, kbw, c, kb[r], u.x, u.y);
          u = c_mul(P[r], u);
          ybr[r] = -u.y;
          ybm[r] = u.x;
          llr[r] -= u.y;
          llm[r] += u.x;
        }
      }
      // sensitivities: sums of this wave
      float* wv = wsum + (par * NW + wave) * GA_NV;
      float t[N][3];
#pragma unroll
      for (int m = 0; m < N; ++m) t[m][0] = t[m][1] = t[m][2] = 0.f;
#pragma unroll
      for (int p = 0; p < N; ++p) {
        if (!((Th.pmask >> p) & 1)) continue;
        constexpr int MC = 2;
        const int i = R::pi(p), j = R::pj(p), nc = uni(A->rp_n[p]);
        float vc[MC] = {0.f, 0.f};
        if constexpr (RThread<d, N>::SHARE) {
          // coupling by coupling: its rows once for all elements
#pragma unroll
          for (int k = 0; k < MC; ++k) {
            if (k >= nc) continue;
            const int u = uni(A->rp_u[p][k]);
            const float g = A->rp_g[p][k], sg = A->rp_s[p][k];
            uint32_t pk = Th.pk[0];
            asm volatile("" : "+v"(pk));
            RElem<d, N> El;
            El.set(pk);
            float a[R::gr], b[R::gr];
            g_row<R::gr, R::gr>(gt + ((j * 2 + (u >> 1)) * d + ket_digit(pk, j)) * R::gr, b);
            if (i > 0) g_row<R::gr, R::gr>(gt + ((i * 2 + (u & 1)) * d + ket_digit(pk, i)) * R::gr, a);
            float ta = 0.f, t0 = 0.f, t1 = 0.f, t2 = 0.f, u0 = 0.f, u1 = 0.f, u2 = 0.f;
#pragma unroll
            for (int r = 0; r < E; ++r) {
              if (i == 0) g_row<R::gr, R::gr>(gt + ((u & 1) * d + r) * R::gr, a);
              const c32 ye = y[r];
              c32 v[n_][n_];
#pragma unroll
              for (int x = 0; x < n_; ++x)
#pragma unroll
                for (int z = 0; z < n_; ++z) {
                  const int b0 = ((r & 1) ^ 1) + 2 * x;   // mode 0's level, in the thread
                  v[x][z] = i == 0 ? kbw[tid + El.o[j] + El.at(z, j) + (b0 < d ? b0 : 1 - (r & 1)) * T]
                                   : kbw[tid + El.o[i] + El.o[j] + El.at(x, i) + El.at(z, j) + r * T];
                }
#pragma unroll
              for (int x = 0; x < n_; ++x) {
                float rr = 0.f, rm = 0.f, qr = 0.f, qm = 0.f;
#pragma unroll
                for (int z = 0; z < n_; ++z) {
                  rr = fmaf(b[z], v[x][z].x, rr);
                  rm = fmaf(b[z], v[x][z].y, rm);
                  qr = fmaf(a[z], v[z][x].x, qr);
                  qm = fmaf(a[z], v[z][x].y, qm);
                }
                const float wi = fmaf(rr, ye.y, -rm * ye.x), wj = fmaf(qr, ye.y, -qm * ye.x);
                ta = fmaf(a[x], wi, ta);
                t0 = fmaf(a[n_ + x], wi, t0);
                t1 = fmaf(a[2 * n_ + x], wi, t1);
                t2 = fmaf(a[3 * n_ + x], wi, t2);
                u0 = fmaf(b[n_ + x], wj, u0);
                u1 = fmaf(b[2 * n_ + x], wj, u1);
                u2 = fmaf(b[3 * n_ + x], wj, u2);
              }
              // keeps the sums here: moved behind all reads they hold them all
              asm volatile("" : "+v"(ta), "+v"(t0), "+v"(t1), "+v"(t2), "+v"(u0), "+v"(u1), "+v"(u2));
            }
            vc[k] = sg * ta;
            t[i][0] = fmaf(g, t0, t[i][0]);
            t[i][1] = fmaf(g, t1, t[i][1]);
            t[i][2] = fmaf(g, t2, t[i][2]);
            t[j][0] = fmaf(g, u0, t[j][0]);
            t[j][1] = fmaf(g, u1, t[j][1]);
            t[j][2] = fmaf(g, u2, t[j][2]);
            __builtin_amdgcn_sched_barrier(0);
          }
        } else {
#pragma unroll
          for (int r = 0; r < E; ++r) {
            const int e = tid + r * T;
            if (e >= L) continue;
            uint32_t pk = Th.pk[r];
            asm volatile("" : "+v"(pk));
            RElem<d, N> El;
            El.set(pk);
            const c32* q = kbw + e + (El.o[i] + El.o[j]);
            c32 v[n_][n_];
#pragma unroll
            for (int x = 0; x < n_; ++x)
#pragma unroll
              for (int z = 0; z < n_; ++z) v[x][z] = q[El.at(x, i) + El.at(z, j)];
            const c32 ye = y[r];
            const int ri = ket_digit(pk, i) * R::gr, rj = ket_digit(pk, j) * R::gr;
#pragma unroll
            for (int k = 0; k < MC; ++k) {
              if (k >= nc) continue;
              const int u = uni(A->rp_u[p][k]);
              const float g = A->rp_g[p][k], sg = A->rp_s[p][k];
              float a[R::gr], b[R::gr];
              g_row<R::gr, R::gr>(gt + (i * 2 + (u & 1)) * d * R::gr + ri, a);
              g_row<R::gr, R::gr>(gt + (j * 2 + (u >> 1)) * d * R::gr + rj, b);
              float ta = 0.f, t0 = 0.f, t1 = 0.f, t2 = 0.f, u0 = 0.f, u1 = 0.f, u2 = 0.f;
#pragma unroll
              for (int x = 0; x < n_; ++x) {
                float rr = 0.f, rm = 0.f, qr = 0.f, qm = 0.f;
#pragma unroll
                for (int z = 0; z < n_; ++z) {
                  rr = fmaf(b[z], v[x][z].x, rr);
                  rm = fmaf(b[z], v[x][z].y, rm);
                  qr = fmaf(a[z], v[z][x].x, qr);
                  qm = fmaf(a[z], v[z][x].y, qm);
                }
                const float wi = fmaf(rr, ye.y, -rm * ye.x), wj = fmaf(qr, ye.y, -qm * ye.x);
                ta = fmaf(a[x], wi, ta);
                t0 = fmaf(a[n_ + x], wi, t0);
                t1 = fmaf(a[2 * n_ + x], wi, t1);
                t2 = fmaf(a[3 * n_ + x], wi, t2);
                u0 = fmaf(b[n_ + x], wj, u0);
                u1 = fmaf(b[2 * n_ + x], wj, u1);
                u2 = fmaf(b[3 * n_ + x], wj, u2);
              }
              vc[k] = fmaf(sg, ta, vc[k]);
              t[i][0] = fmaf(g, t0, t[i][0]);
              t[i][1] = fmaf(g, t1, t[i][1]);
              t[i][2] = fmaf(g, t2, t[i][2]);
              t[j][0] = fmaf(g, u0, t[j][0]);
              t[j][1] = fmaf(g, u1, t[j][1]);
              t[j][2] = fmaf(g, u2, t[j][2]);
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        }
#pragma unroll
        for (int k = 0; k < MC; ++k) {
          if (k >= nc) continue;
          const float x = g_wave_sum(2.f * vc[k]);
          if (lane == 0) wv[GA_MAXDS + 3 * N + uni(A->rp_c[p][k])] = x;
        }
      }
#pragma unroll
      for (int m = 0; m < N; ++m) {
        const bool drv = (Th.dmask >> m) & 1;
        const int u = uni(A->rd_u[m]);
        float vd = 0.f;
        constexpr bool once = RThread<d, N>::SHARE;   // m > 0: the rows of element 0 are all's
        float4 de;
        float a[R::gr];
#pragma unroll
        for (int r = 0; r < E; ++r) {
          const int e = tid + r * T;
          if (e >= L) continue;
          uint32_t pk = Th.pk[once ? 0 : r];
          asm volatile("" : "+v"(pk));
          const int a_ = once && m == 0 ? r : ket_digit(pk, m);
          const c32 ye = y[r];
          if (!once || m == 0 || r == 0) {
            de = *reinterpret_cast<const float4*>(gt + R::off_e + (m * d + a_) * 4);
            if (drv) g_row<R::gr, R::gr>(gt + ((m * 2 + u) * d + a_) * R::gr, a);
          }
          const float w0 = fmaf(kb[r].x, ye.y, -kb[r].y * ye.x);
          t[m][0] = fmaf(de.x, w0, t[m][0]);
          t[m][1] = fmaf(de.y, w0, t[m][1]);
          t[m][2] = fmaf(de.z, w0, t[m][2]);
          if (drv) {
            RElem<d, N> El;
            El.set(pk);
            const c32* q = kbw + e + El.o[m];
            float t0 = 0.f, t1 = 0.f, t2 = 0.f;
#pragma unroll
            for (int x = 0; x < n_; ++x) {
              const int b0 = ((r & 1) ^ 1) + 2 * x;
              const c32 v = once && m == 0 ? kb[b0 < d && b0 < E ? b0 : 0] : q[El.at(x, m)];
              const float w = fmaf(v.x, ye.y, -v.y * ye.x);
              vd = fmaf(a[x], w, vd);
              t0 = fmaf(a[n_ + x], w, t0);
              t1 = fmaf(a[2 * n_ + x], w, t1);
              t2 = fmaf(a[3 * n_ + x], w, t2);
            }
            const float cm = c[m] * unif(A->rd_c[m]);   // c(t) itself: kappa comes with the fold
            t[m][0] = fmaf(cm, t0, t[m][0]);
            t[m][1] = fmaf(cm, t1, t[m][1]);
            t[m][2] = fmaf(cm, t2, t[m][2]);
          }
        }
        if (drv) {
          const float x = g_wave_sum(2.f * vd);
          if (lane == 0) wv[uni(A->rd_k[m])] = x;
        }
#pragma unroll
        for (int th = 0; th < 3; ++th) {
          const float x = g_wave_sum(2.f * t[m][th]);
          if (lane == 0) wv[GA_MAXDS + 3 * m + th] = x;
        }
      }
      if (s == 3) Th.drives(3 * nx + 2, c2);
      if (s == 1) {
        Th.phases(2 * nx + 1, P1);
        Th.drives(3 * nx + 1, c1);
      }
      prev_n = n;
      prev_s = s;
      par ^= 1;
      cur ^= 1;
    }
#pragma unroll
    for (int r = 0; r < E; ++r) {
      float x = lhr[r] + llr[r];
      llr[r] -= x - lhr[r];
      lhr[r] = x;
      x = lhm[r] + llm[r];
      llm[r] -= x - lhm[r];
      lhm[r] = x;
      P2[r] = P0[r];
    }
  }
  __syncthreads();
  fold_prev();   // the last stage's sums
}

// One kernel each for direct (items == nullptr) and batched launches.
template <int d, int N, bool CK>
__global__ void __launch_bounds__((GShape<d, N, false>::T))
g_real_rk4_kernel(const GItem* __restrict__ items, const GArgs* __restrict__ Ag,
                  const GAdj* __restrict__ Bg, int n_lo, int n_hi, const float4* __restrict__ st_in,
                  float4* __restrict__ st_out) {
  int col = blockIdx.x;
  if (items != nullptr) {
    kptr<GItem> it = kconst(items) + blockIdx.x;
    Ag = (const GArgs*)it->A;
    Bg = (const GAdj*)it->B;
    col = it->col;
    n_lo = it->n_lo;
    n_hi = it->n_hi;
    st_in = it->st_in;
    st_out = it->st_out;
  }
  g_real_rk4_body<d, N, CK>(Ag, Bg, col, n_lo, n_hi, st_in, st_out);
}

template <int d, int N>
__global__ void __launch_bounds__((GShape<d, N, false>::T))
g_real_cos_kernel(const GItem* __restrict__ items, const GArgs* __restrict__ Ag,
                  const GAdj* __restrict__ Bg, int g_hi, int g_lo) {
  int col = blockIdx.x;
  if (items != nullptr) {   // item.gseg the first segment, item.n_lo the last
    kptr<GItem> it = kconst(items) + blockIdx.x;
    Ag = (const GArgs*)it->A;
    Bg = (const GAdj*)it->B;
    col = it->col;
    g_hi = it->gseg;
    g_lo = it->n_lo;
  }
  g_real_cos_body<d, N>(Ag, Bg, col, g_hi, g_lo);
}

template <int d, int N>
__global__ void __launch_bounds__((GShape<d, N, false>::T))
g_real_seg_kernel(const GItem* __restrict__ items, const GArgs* __restrict__ Ag,
                  const GAdj* __restrict__ Bg, int gseg) {
  int col, slot = blockIdx.x;
  if (items != nullptr) {   // item.n_lo the stage-input buffer
    kptr<GItem> it = kconst(items) + blockIdx.x;
    Ag = (const GArgs*)it->A;
    Bg = (const GAdj*)it->B;
    col = it->col;
    gseg = it->gseg;
    slot = it->n_lo;
  } else {
    const int S = Ag->S, k = blockIdx.x / S;
    col = blockIdx.x - k * S;
    gseg -= k;
  }
  g_real_seg_body<d, N>(Ag, Bg, gseg, col, slot);
}

// Frame phases exp(i sum_m f_m[a_m] t) of every element at half step q: the
// modes' phases from FP64 angles reduced modulo 2 pi, multiplied in FP64 and
// rounded once.
struct RPhase {
  int d, N, L, q_lo;
  double h;
  double f[GA_MAXM][8];
};
__global__ void __launch_bounds__(256) g_real_phase_kernel(RPhase S, float2* __restrict__ ph) {
  __shared__ double2 m[GA_MAXM * 8];
  const int q = blockIdx.x;
  for (int t = threadIdx.x; t < S.N * S.d; t += blockDim.x) {
    const double twopi = 6.283185307179586476925286766559;
    double x = S.f[t / S.d][t % S.d] * ((S.q_lo + q) * (0.5 * S.h));
    x -= twopi * rint(x / twopi);
    double sn, cs;
    sincos(x, &sn, &cs);
    m[t] = make_double2(cs, sn);
  }
  __syncthreads();
  for (int e = threadIdx.x; e < S.L; e += blockDim.x) {
    int r = e;
    double pr = 1.0, pi = 0.0;
    for (int k = S.N - 1; k >= 0; --k) {
      const double2 v = m[k * S.d + r % S.d];
      r /= S.d;
      const double x = pr * v.x - pi * v.y;
      pi = pr * v.y + pi * v.x;
      pr = x;
    }
    ph[(size_t)q * S.L + e] = make_float2((float)pr, (float)pi);
  }
}

template <typename K, typename... Args>
hipError_t r_launch(K* kernel, int n, int threads, size_t sh, hipStream_t s, Args... args) {
  if (sh > 163840) return hipErrorInvalidValue;
  (void)hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
  hipLaunchKernelGGL(kernel, dim3(n), dim3(threads), sh, s, args...);
  return hipGetLastError();
}

}  // namespace

size_t g_real_lds(int d, int N, bool seg) {
#define GA_REAL_LDS(dd_, nn_)   \
  if (d == dd_ && N == nn_)     \
    return seg ? RShape<dd_, nn_>::seg_lds_bytes() : RShape<dd_, nn_>::lds_bytes();
  GA_CLOSED_SHAPES(GA_REAL_LDS)
#undef GA_REAL_LDS
  return ~(size_t)0;
}

hipError_t g_real_forward(int d, int N, bool ck, const GItem* items, const GArgs* dargs,
                          const GAdj* dadj, int n, int n_lo, int n_hi, const float4* st_in,
                          float4* st_out, hipStream_t s) {
#define GA_REAL_FWD(dd_, nn_)                                                                     \
  if (d == dd_ && N == nn_) {                                                                     \
    using R = RShape<dd_, nn_>;                                                                   \
    return ck ? r_launch(g_real_rk4_kernel<dd_, nn_, true>, n, R::Sh::T, R::lds_bytes(), s, items, \
                         dargs, dadj, n_lo, n_hi, st_in, st_out)                                  \
              : r_launch(g_real_rk4_kernel<dd_, nn_, false>, n, R::Sh::T, R::lds_bytes(), s, items, \
                         dargs, dadj, n_lo, n_hi, st_in, st_out);                                 \
  }
  GA_CLOSED_SHAPES(GA_REAL_FWD)
#undef GA_REAL_FWD
  return hipErrorInvalidValue;
}

hipError_t g_real_sweep(int d, int N, const GItem* items, const GArgs* dargs, const GAdj* dadj, int n,
                        int g_hi, int g_lo, hipStream_t s) {
#define GA_REAL_COS(dd_, nn_)                                                                       \
  if (d == dd_ && N == nn_)                                                                         \
    return r_launch(g_real_cos_kernel<dd_, nn_>, n, GShape<dd_, nn_, false>::T,                     \
                    RShape<dd_, nn_>::lds_bytes(), s, items, dargs, dadj, g_hi, g_lo);
  GA_CLOSED_SHAPES(GA_REAL_COS)
#undef GA_REAL_COS
  return hipErrorInvalidValue;
}

hipError_t g_real_segments(int d, int N, const GItem* items, const GArgs* dargs, const GAdj* dadj,
                           int n, int gseg, hipStream_t s) {
#define GA_REAL_SEG(dd_, nn_)                                                                       \
  if (d == dd_ && N == nn_)                                                                         \
    return r_launch(g_real_seg_kernel<dd_, nn_>, n, GShape<dd_, nn_, false>::T,                     \
                    RShape<dd_, nn_>::seg_lds_bytes(), s, items, dargs, dadj, gseg);
  GA_CLOSED_SHAPES(GA_REAL_SEG)
#undef GA_REAL_SEG
  return hipErrorInvalidValue;
}

hipError_t g_real_phases(int d, int N, int q_lo, int nq, double h, const double f[][8], float2* ph,
                         hipStream_t s) {
  RPhase R;
  std::memset(&R, 0, sizeof(R));
  R.d = d;
  R.N = N;
  R.L = cpow(d, N);
  R.q_lo = q_lo;
  R.h = h;
  std::memcpy(R.f, f, sizeof(R.f));
  hipLaunchKernelGGL(g_real_phase_kernel, dim3(nq), dim3(256), 0, s, R, ph);
  return hipGetLastError();
}

}  // namespace scp
