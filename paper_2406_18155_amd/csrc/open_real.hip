// Gather engine, real form of an open system's forward and adjoint, and of the
// forward of closed systems above the other real form's shapes (d = 3, N = 8).
//
// Under the conditions of the closed systems' real form (real frame, odd
// operators, neighbour couplings, one operator per driven mode) the density
// matrix without its frame phases, rho' = P^dag rho P, follows
//   k' = -i (R rho' - rho' R) + D(rho'),
// R real symmetric and constant but for the drives' c_k(t), and the relaxation
// and dephasing D real and constant.  One workgroup holds the matrix; element
// (A, B) gathers its neighbours along the modes of A, then with the sign
// changed along those of B, from the same real rows.  The phases of P are one
// complex number per element and half step.
//
// A thread holds the elements of all digits of the first H modes of A: what
// couples those modes stays in its registers with uniform coefficients, and
// every other digit is the same for all its elements, so rows and offsets are
// formed once per pair term, not per element.  A row along digits of unlike
// parity has ceil(d/2)^2 entries.
//
// Bound: vector instruction issue and LDS reads (about 24 per element and stage)
// of the one workgroup on a compute unit.  The low words of the largest shape's
// state lie in LDS.  Complex rows (g_apply, g_adj_body) -> here, us per step, 256
// matrices, two couplings on a pair: d = 3, N = 4 forward 68 -> 31, forward and
// adjoint 356 -> 147; d = 4, N = 3 34 -> 17 and 173 -> 68; d = 3, N = 3 8.2 -> 8.0
// and 46 -> 33; d = 2, N = 5 10.3 -> 8.6 and 61 -> 40; 16 matrices the same.
// Elements dealt to 1024 threads in order, every element with its own digits and
// rows, took 62 and 380: as many LDS reads of rows as of elements.
//
// A closed column of D = 6561 is the same element set with A's modes alone (no
// B, no rates); two buffers and the low words fill the LDS, where the
// register-layout stepper runs 256 threads of 27 amplitudes through four
// layouts: 8-transmon ring 48 -> 33 us per step (256 columns), LDS-bound (36
// reads of 8 bytes per element and stage, 6.5 of 8.2 us).
#include "gather.h"

namespace scp {

namespace {

template <int d, int N, bool OPEN>
struct LShape {
  static constexpr int D = cpow(d, N), L = OPEN ? D * D : D;
  static constexpr int H = L / d > 1024 ? 2 : 1;       // modes of A within a thread
  static constexpr int E = cpow(d, H), T = L / E;      // elements tid + r T of a thread
  static constexpr int TB = (T + 63) / 64 * 64, NW = TB / 64;
  static constexpr int n = Nb<d, true>::n, nn = n * n, dd = d * d;
  static constexpr int pr = nn == 9 ? 12 : nn;   // row strides, as the static table has them
  static constexpr int dr = n == 3 ? 4 : n;
  static constexpr int off_d = N * dd * pr;
  static constexpr int total = off_d + N * d * dr;
  static constexpr int pad = (total + 3) & ~3;
  static constexpr int gr = (4 * n + 3) / 4 * 4;
  static constexpr int off_c = pad + N * 2 * d * gr + N * d * 4;   // rows of the couplings, in the static table
  static constexpr int nc = N * 2 * dd * pr;
  static constexpr bool LO = E > 4;    // low words of the state in LDS
  // LDS: two buffers, the low words, then in floats: static rows, the rates'
  // decay and jump coefficients [N][dd] each, the frame energies of the first H
  // modes [E], and (adjoint) the couplings' rows and the stages' sums per wave: N drives, 2 N couplings (two at most on each
  // pair), 2 N rates
  static constexpr int at_j = pad, at_f = pad + 2 * N * dd, at_c = (at_f + E + 3) & ~3;
  static constexpr int NV = 5 * N;
  static constexpr int at_s = at_c + ((nc + 3) & ~3);
  static constexpr size_t bufs = (LO ? 3 : 2) * (size_t)L + (L & 1 & (int)LO);   // 16-byte multiple
  static constexpr size_t fwd_bytes() { return sizeof(c32) * bufs + sizeof(float) * (size_t)at_c; }
  static constexpr size_t adj_bytes() {
    return sizeof(c32) * bufs + sizeof(float) * (size_t)(at_s + 2 * NW * NV);
  }
  static_assert((OPEN ? adj_bytes() : fwd_bytes()) <= 163840, "a column fits the LDS");
  static constexpr int ms(int m) { return cpow(d, N - 1 - m); }   // stride in A or B
  static constexpr int st(int side, int m) { return (OPEN && !side ? D : 1) * ms(m); }
  static constexpr int pi(int p) { return p == N - 1 ? 0 : p; }
  static constexpr int pj(int p) { return p == N - 1 ? N - 1 : p + 1; }
  // digit of the thread's element r along one of the first H modes, the step of
  // r along it, and the place of level b in the row of level a (unlike parity)
  static constexpr int rs(int m) { return cpow(d, H - 1 - m); }
  static constexpr int rd(int r, int m) { return r / rs(m) % d; }
  static constexpr int place(int a, int b) { return (b - ((a & 1) ^ 1)) / 2; }
};

// Keeps the sums of an element where its neighbours are read: moved behind all
// elements' reads they would hold every read value in a register.
__device__ __forceinline__ void l_pin(float& a, float& b, float& c) {
  asm volatile("" : "+v"(a), "+v"(b), "+v"(c));
}

__device__ __forceinline__ void l_mac(c32& z, float g, c32 v) {
  z.x = fmaf(g, v.x, z.x);
  z.y = fmaf(g, v.y, z.y);
}

// What a thread keeps of its elements and of the drives.
template <int d, int N, bool OPEN>
struct LThread {
  using S = LShape<d, N, OPEN>;
  static constexpr int E = S::E, T = S::T, L = S::L, H = S::H, n = S::n;
  bool on;            // threads past the last element only help with the copies
  unsigned tid;       // 0 where off
  uint32_t pk;        // digits of A's modes H .. N - 1 and of B's
  float dg;           // frame energies of those (kappa included)
  float* tab;         // LDS
  const float* rt;    // the same rows in device memory, for uniform reads
  const c32* ph;
  const float* rc;
  int pmask, dmask;
  bool rates;

  // couplings: also their rows (adjoint)
  __device__ __forceinline__ void init(kptr<GArgs> A, float* lds_tab, bool couplings) {
    ph = (const c32*)A->ph;
    rc = A->rc;
    rt = A->rt;
    pmask = uni(A->pmask);
    dmask = uni(A->dmask);
    tab = lds_tab;
    for (int t = threadIdx.x; t < S::total; t += S::TB) lds_tab[t] = A->rt[t];
    if (couplings)
      for (int t = threadIdx.x; t < S::nc; t += S::TB) lds_tab[S::at_c + t] = A->rt[S::off_c + t];
    // per mode and digit pair: decay -gamma1 (a + b) / 2 - gammaphi (a - b)^2,
    // and the jump's sqrt((a + 1)(b + 1)) (0 at the top level)
    for (int t = threadIdx.x; OPEN && t < N * S::dd; t += S::TB) {
      const int m = t / S::dd, a = t % S::dd / d, b = t % d;
      lds_tab[S::at_j + t] =
          (float)(A->kappa * (-0.5 * A->g1[m] * (a + b) - (double)A->gp[m] * ((a - b) * (a - b))));
      lds_tab[S::at_j + N * S::dd + t] =
          a < d - 1 && b < d - 1 ? (float)sqrt((double)((a + 1) * (b + 1))) : 0.f;
    }
    for (int t = threadIdx.x; t < E; t += S::TB) {
      float g = 0.f;
#pragma unroll
      for (int m = 0; m < H; ++m) g += A->delta[m][S::rd(t, m)];
      lds_tab[S::at_f + t] = (float)(A->kappa * g);
    }
    rates = false;
#pragma unroll
    for (int m = 0; m < N; ++m) rates |= OPEN && (A->g1[m] > 0.f || A->gp[m] > 0.f);
    on = (int)threadIdx.x < T;
    tid = on ? threadIdx.x : 0;
    const int Ai = OPEN ? tid / S::D : tid, Bi = OPEN ? (int)tid - Ai * S::D : 0;
    pk = 0;
    float g = 0.f;
#pragma unroll
    for (int m = 0; m < N; ++m) {
      const int a = m < H ? 0 : (Ai / S::ms(m)) % d, b = OPEN ? (Bi / S::ms(m)) % d : 0;
      pk |= (uint32_t)a << (3 * m);
      if (m >= H) g += A->delta[m][a];
      if (OPEN) {
        pk |= (uint32_t)b << (3 * (N + m));
        g -= A->delta[m][b];
      }
    }
    dg = (float)(A->kappa * g);
  }
  // Digits and neighbours, from an opaque copy of pk: offsets are formed where
  // a term starts, not kept across the stages.
  struct Digits {
    uint32_t pk;
    __device__ __forceinline__ int dig(int side, int m) const { return (pk >> (3 * (side * N + m))) & 7; }
    // offset of the first neighbour along a mode, and of the k-th from it
    __device__ __forceinline__ int o(int side, int m) const {
      const int a = dig(side, m), st = S::st(side, m);
      return (a & 1) ? -a * st : (1 - a) * st;
    }
    __device__ __forceinline__ int at(int k, int side, int m) const {
      const int st = S::st(side, m);
      if (k == 0) return 0;
      if (k == n - 1 && (d & 1)) return (dig(side, m) & 1) ? 2 * k * st : 0;
      return 2 * k * st;
    }
  };
  __device__ __forceinline__ Digits digits() const {
    Digits q;
    q.pk = pk;
    asm volatile("" : "+v"(q.pk));
    return q;
  }
  __device__ __forceinline__ void phases(int q, c32 (&P)[E]) const {
#pragma unroll
    for (int r = 0; r < E; ++r) P[r] = (ph + (size_t)q * L + r * T)[tid];
  }
  __device__ __forceinline__ void drives(int row, float (&c)[N]) const {
#pragma unroll
    for (int m = 0; m < N; ++m)
      if ((dmask >> m) & 1) c[m] = kconst(rc)[row * N + m];
  }
  // three elements' reads in flight at a time: more need registers that the
  // largest shape does not have
  static __device__ __forceinline__ void fence(int r) {
    if (r % 3 == 2) __builtin_amdgcn_sched_barrier(0);
  }
  // f(r, t): t[c] = sum over the neighbours of element r along the modes of
  // pair p, one side, of the rows of table c (C tables of dd rows at `rows`, in
  // device memory at `urows`) times y, t[0] with the start init(r), the rows of
  // side 1 with the sign changed; own: this thread's y
  template <int p, int side, int C, typename I, typename F>
  __device__ __forceinline__ void pair(const c32* yc, const c32 (&own)[E], const float* rows,
                                       const float* urows, I init, F f) const {
    constexpr int i = S::pi(p), j = S::pj(p), cs = S::dd * S::pr;
    const Digits X = digits();
    if constexpr (side == 1 || i >= H) {   // both digits are the thread's
      float g[C][S::nn];
#pragma unroll
      for (int c = 0; c < C; ++c)
        g_row<S::nn, S::pr>(rows + c * cs + (X.dig(side, i) * d + X.dig(side, j)) * S::pr, g[c]);
      if (side == 1) {
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
          for (int k = 0; k < S::nn; ++k) g[c][k] = -g[c][k];
      }
      const c32* q = yc + tid + (X.o(side, i) + X.o(side, j));
#pragma unroll
      for (int r = 0; r < E; ++r) {
        c32 t[C];
#pragma unroll
        for (int c = 0; c < C; ++c) t[c].x = t[c].y = 0.f;
        t[0] = init(r);
#pragma unroll
        for (int x = 0; x < n; ++x)
#pragma unroll
          for (int z = 0; z < n; ++z) {
            const c32 v = q[X.at(x, side, i) + X.at(z, side, j) + r * T];
#pragma unroll
            for (int c = 0; c < C; ++c) l_mac(t[c], g[c][x * n + z], v);
          }
        f(r, t);
        fence(r);
      }
    } else if constexpr (j >= H) {   // i within the thread: groups of d elements along it
      float g[C][d][S::nn];
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int a = 0; a < d; ++a)
          g_row<S::nn, S::pr>(rows + c * cs + (a * d + X.dig(0, j)) * S::pr, g[c][a]);
      const c32* q = yc + tid + X.o(0, j);
#pragma unroll
      for (int r0 = 0; r0 < E; ++r0) {
        if (S::rd(r0, i) != 0) continue;
        c32 v[d][n];
#pragma unroll
        for (int b = 0; b < d; ++b)
#pragma unroll
          for (int z = 0; z < n; ++z) v[b][z] = q[X.at(z, 0, j) + (r0 + b * S::rs(i)) * T];
#pragma unroll
        for (int a = 0; a < d; ++a) {
          c32 t[C];
#pragma unroll
          for (int c = 0; c < C; ++c) t[c].x = t[c].y = 0.f;
          t[0] = init(r0 + a * S::rs(i));
#pragma unroll
          for (int b = (a & 1) ^ 1; b < d; b += 2)
#pragma unroll
            for (int z = 0; z < n; ++z)
#pragma unroll
              for (int c = 0; c < C; ++c) l_mac(t[c], g[c][a][S::place(a, b) * n + z], v[b][z]);
          f(r0 + a * S::rs(i), t);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {   // both within the thread
      kptr<float> u = kconst(urows);
#pragma unroll
      for (int r = 0; r < E; ++r) {
        constexpr int rsi = S::rs(i), rsj = S::rs(j);
        const int a = S::rd(r, i), b = S::rd(r, j);
        c32 t[C];
#pragma unroll
        for (int c = 0; c < C; ++c) t[c].x = t[c].y = 0.f;
        t[0] = init(r);
#pragma unroll
        for (int x = (a & 1) ^ 1; x < d; x += 2)
#pragma unroll
          for (int z = (b & 1) ^ 1; z < d; z += 2)
#pragma unroll
            for (int c = 0; c < C; ++c)
              l_mac(t[c], u[c * cs + (a * d + b) * S::pr + S::place(a, x) * n + S::place(b, z)],
                    own[r + (x - a) * rsi + (z - b) * rsj]);
        f(r, t);
        fence(r);
      }
    }
  }
  // f(r, t): the same for the drive operator of mode m, times c
  template <int m, int side, typename I, typename F>
  __device__ __forceinline__ void drive(const c32* yc, const c32 (&own)[E], float c, I init,
                                        F f) const {
    const Digits X = digits();
    if constexpr (side == 1 || m >= H) {
      float g[n];
      g_row<n, S::dr>(tab + S::off_d + (m * d + X.dig(side, m)) * S::dr, g);
#pragma unroll
      for (int x = 0; x < n; ++x) g[x] *= side == 1 ? -c : c;
      const c32* q = yc + tid + X.o(side, m);
#pragma unroll
      for (int r = 0; r < E; ++r) {
        c32 t = init(r);
#pragma unroll
        for (int x = 0; x < n; ++x) l_mac(t, g[x], q[X.at(x, side, m) + r * T]);
        f(r, t);
        fence(r);
      }
    } else {
      kptr<float> u = kconst(rt + S::off_d + m * d * S::dr);
#pragma unroll
      for (int r = 0; r < E; ++r) {
        const int a = S::rd(r, m);
        c32 t;
        t.x = t.y = 0.f;
#pragma unroll
        for (int x = (a & 1) ^ 1; x < d; x += 2)
          l_mac(t, u[a * S::dr + S::place(a, x)], own[r + (x - a) * S::rs(m)]);
        c32 k = init(r);
        l_mac(k, c, t);
        f(r, k);
        fence(r);
      }
    }
  }
  // decay of element r along the modes: d per mode within the thread
  struct Decay {
    float t, m[H][d];
    __device__ __forceinline__ float of(int r) const {
      float s = t;
#pragma unroll
      for (int k = 0; k < H; ++k) s += m[k][S::rd(r, k)];
      return s;
    }
  };
  __device__ __forceinline__ Decay decay() const {
    const Digits X = digits();
    Decay D;
    D.t = 0.f;
#pragma unroll
    for (int m = 0; m < N; ++m) {
      const float* q = tab + S::at_j + m * S::dd + X.dig(1, m);
      if (m >= H) {
        D.t += q[X.dig(0, m) * d];
      } else {
#pragma unroll
        for (int a = 0; a < d; ++a) D.m[m < H ? m : 0][a] = q[a * d];
      }
    }
    return D;
  }
  // f(r, v): v = sqrt((a + 1)(b + 1)) y(a + 1, b + 1) along mode m, or (ADJ)
  // sqrt(a b) y(a - 1, b - 1); zero where there is no such level
  template <int m, bool ADJ, typename F>
  __device__ __forceinline__ void jump(const c32* yc, F f) const {
    constexpr int sg = ADJ ? -1 : 1;
    const Digits X = digits();
    const int b = X.dig(1, m);
    const bool inb = ADJ ? b > 0 : b < d - 1;
    const float* w = tab + S::at_j + (N + m) * S::dd + (ADJ && inb ? b - 1 : b);
    if constexpr (m >= H) {
      const int a = X.dig(0, m);
      const bool in = inb && (ADJ ? a > 0 : a < d - 1);
      const float g = in ? w[(ADJ ? a - 1 : a) * d] : 0.f;
      const c32* q = yc + tid + (in ? sg * (S::st(0, m) + S::st(1, m)) : 0);
#pragma unroll
      for (int r = 0; r < E; ++r) {
        c32 v = q[r * T];
        v.x *= g;
        v.y *= g;
        f(r, v);
        fence(r);
      }
    } else {
      const c32* q = yc + tid + (inb ? sg * S::st(1, m) : 0);
      float g[d];
#pragma unroll
      for (int a = 0; a < d; ++a) g[a] = inb && a < d - 1 ? w[a * d] : 0.f;   // of the lower level
#pragma unroll
      for (int r = 0; r < E; ++r) {
        const int a = S::rd(r, m), s = a + sg;
        if (s < 0 || s >= d) continue;
        c32 v = q[(r + sg * S::rs(m)) * T];
        v.x *= g[ADJ ? s : a];
        v.y *= g[ADJ ? s : a];
        f(r, v);
        fence(r);
      }
    }
  }

  // x[r] = k' of the thread's elements, the stage input in yc (own: the
  // thread's); load() starts what is needed after it
  template <typename F>
  __device__ __forceinline__ void apply(kptr<GArgs> A, const c32* yc, const c32 (&own)[E],
                                        const float (&c)[N], c32 (&x)[E], F load) const {
    c32 z[E];   // K, with D turned by i
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const float g = dg + tab[S::at_f + r];
      z[r].x = g * own[r].x;
      z[r].y = g * own[r].y;
    }
    auto init = [&](int r) { return z[r]; };
    static_for<N>([&](auto P) {
      constexpr int p = decltype(P)::value;
      if (!((pmask >> p) & 1)) return;
      const float* rows = tab + p * S::dd * S::pr;
      const float* urows = rt + p * S::dd * S::pr;
      auto keep = [&](int r, const c32(&t)[1]) { z[r] = t[0]; };
      pair<p, 0, 1>(yc, own, rows, urows, init, keep);
      if constexpr (OPEN) pair<p, 1, 1>(yc, own, rows, urows, init, keep);
      __builtin_amdgcn_sched_barrier(0);
    });
    static_for<N>([&](auto M) {
      constexpr int m = decltype(M)::value;
      if (!((dmask >> m) & 1)) return;
      auto keep = [&](int r, c32 t) { z[r] = t; };
      drive<m, 0>(yc, own, c[m], init, keep);
      if constexpr (OPEN) drive<m, 1>(yc, own, c[m], init, keep);
      __builtin_amdgcn_sched_barrier(0);
    });
    load();
    if constexpr (OPEN) {
      if (rates) {
        static_for<N>([&](auto M) {
          constexpr int m = decltype(M)::value;
          const float g1 = unif((float)(A->kappa * A->g1[m]));
          jump<m, false>(yc, [&](int r, c32 v) {
            z[r].y = fmaf(g1, v.x, z[r].y);
            z[r].x = fmaf(-g1, v.y, z[r].x);
          });
        });
        const Decay D = decay();
#pragma unroll
        for (int r = 0; r < E; ++r) {
          const float g = D.of(r);
          z[r].y = fmaf(g, own[r].x, z[r].y);
          z[r].x = fmaf(-g, own[r].y, z[r].x);
        }
      }
    }
#pragma unroll
    for (int r = 0; r < E; ++r) {
      x[r].x = z[r].y;
      x[r].y = -z[r].x;
    }
  }
};

// Steps [n0, n1) of one column from (hi, lo) at n0 in `from` (null: from the
// input column) to `to` (nullable): CK keeps the state at every ce-th step, SEG
// the stage inputs y'.
template <int d, int N, bool OPEN, bool CK, bool SEG>
__device__ __forceinline__ void l_steps(kptr<GArgs> A, const GAdj* __restrict__ Bg,
                                        const LThread<d, N, OPEN>& Th, c32* lds, c32* lo, int col, int n0,
                                        int n1, const float4* __restrict__ from,
                                        float4* __restrict__ to, c32* __restrict__ segc) {
  using S = LShape<d, N, OPEN>;
  constexpr int L = S::L, T = S::T, E = S::E;
  const unsigned tid = Th.tid;
  const bool on = Th.on;
  const float h = A->h;
  float hr[E], hm[E], ar[E], ai[E], lr[S::LO ? 1 : E], lm[S::LO ? 1 : E];
  auto low = [&](int r) {
    c32 l;
    if constexpr (S::LO) {
      l = lo[tid + r * T];
    } else {
      l.x = lr[r];
      l.y = lm[r];
    }
    return l;
  };
  auto set_low = [&](int r, c32 l) {
    if constexpr (S::LO) {
      if (on) lo[tid + r * T] = l;
    } else {
      lr[r] = l.x;
      lm[r] = l.y;
    }
  };
  c32 y[E];   // the thread's stage input
  float c[N], cn[N];
#pragma unroll
  for (int m = 0; m < N; ++m) c[m] = cn[m] = 0.f;
  c32 P0[E];
  Th.phases(2 * n0, P0);
  Th.drives(3 * n0, c);
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const int e = tid + r * T;
    float4 q = make_float4(0.f, 0.f, 0.f, 0.f);
    if (SEG || from != nullptr) {
      q = from[e];
    } else {
      const c32 v = ((const c32*)A->x0)[(size_t)col * L + e];
      q.x = v.x;
      q.y = v.y;
    }
    hr[r] = q.x;
    hm[r] = q.y;
    ar[r] = ai[r] = 0.f;
    c32 l, v;
    l.x = q.z;
    l.y = q.w;
    v.x = q.x;
    v.y = q.y;
    set_low(r, l);
    y[r] = c_mul_conj(P0[r], v);
    if (on) {
      lds[e] = y[r];
      if (SEG) segc[e] = y[r];
    }
  }
  __syncthreads();
  int cur = 0;
#pragma unroll 1
  for (int n = n0; n < n1; ++n) {
    if (CK) {
      kptr<GAdj> B = kconst(Bg);
      const int ce = B->ce;
      if (n % ce == 0) {
        float4* ck = B->ck + ((size_t)col * B->nck + n / ce) * L;
#pragma unroll
        for (int r = 0; r < E; ++r) {
          const c32 l = low(r);
          if (on) ck[tid + r * T] = make_float4(hr[r], hm[r], l.x, l.y);
        }
      }
    }
    // the stages in a rolled loop: the unrolled ones outgrow the instruction cache
#pragma unroll 1
    for (int s = 0; s < 4; ++s) {
      const float w = (s == 0 || s == 3) ? 1.f : 2.f;
      const float ch = s == 2 ? h : 0.5f * h;
      const c32* yc = lds + cur * L;
      c32* yn = lds + (cur ^ 1) * L;
      const int n2 = s < 3 ? n : min(n + 1, A->nsteps - 1), s2 = s < 3 ? s + 1 : 0;
      Th.drives(stage_c(n2, s2), cn);
      const bool keep = SEG && on && (s < 3 || n + 1 < n1);
      c32* ys = SEG ? segc + ((size_t)(n - n0) * 4 + s + 1) * L : nullptr;
      c32 x[E], P[E], Q[E];   // phases of the stage and of the next one
      Th.apply(A, yc, y, c, x, [&]() {
        Th.phases(2 * n + ((s + 1) >> 1), P);
        Th.phases(2 * n + 1 + (s >> 1), Q);
      });
      const float w0 = s == 0 ? 0.f : 1.f;
#pragma unroll
      for (int r = 0; r < E; ++r) {
        x[r] = c_mul(P[r], x[r]);
        ar[r] = fmaf(w, x[r].x, w0 * ar[r]);
        ai[r] = fmaf(w, x[r].y, w0 * ai[r]);
      }
      if (s < 3) {
#pragma unroll
        for (int r = 0; r < E; ++r) {
          c32 v;
          v.x = fmaf(ch, x[r].x, hr[r]);
          v.y = fmaf(ch, x[r].y, hm[r]);
          y[r] = c_mul_conj(Q[r], v);
        }
      } else {
        const float h6 = h * (1.0f / 6.0f);
#pragma unroll
        for (int r = 0; r < E; ++r) {
          c32 v, l = low(r);
          comp_add(hr[r], l.x, h6 * ar[r]);
          comp_add(hm[r], l.y, h6 * ai[r]);
          set_low(r, l);
          v.x = hr[r];
          v.y = hm[r];
          y[r] = c_mul_conj(Q[r], v);
        }
      }
      if (on) {
#pragma unroll
        for (int r = 0; r < E; ++r) yn[tid + r * T] = y[r];
      }
      if (keep) {
#pragma unroll
        for (int r = 0; r < E; ++r) (ys + r * T)[tid] = y[r];
      }
#pragma unroll
      for (int m = 0; m < N; ++m) c[m] = cn[m];
      __syncthreads();
      cur ^= 1;
    }
  }
  if (SEG) return;
  if (to != nullptr) {
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const c32 l = low(r);
      if (on) to[tid + r * T] = make_float4(hr[r], hm[r], l.x, l.y);
    }
  }
  if (A->xT == nullptr || (!OPEN && n1 < A->nsteps)) return;
#pragma unroll
  for (int r = 0; r < E; ++r) {
    c32 l = low(r);
    l.x += hr[r];
    l.y += hm[r];
    if (on) ((c32*)A->xT)[(size_t)col * L + tid + r * T] = l;
  }
}

template <int d, int N, bool OPEN, bool CK>
__global__ void __launch_bounds__((LShape<d, N, OPEN>::TB))
l_rk4_kernel(const GArgs* __restrict__ Ag, const GAdj* __restrict__ Bg, int n_lo, int n_hi,
             const float4* __restrict__ st_in, float4* __restrict__ st_out) {
  using S = LShape<d, N, OPEN>;
  extern __shared__ __align__(16) c32 lds[];
  kptr<GArgs> A = kconst(Ag);
  LThread<d, N, OPEN> Th;
  Th.init(A, reinterpret_cast<float*>(lds + S::bufs), false);
  if constexpr (OPEN) {   // in one run (the range as arguments: 1 to 4 % of a step)
    l_steps<d, N, OPEN, CK, false>(A, Bg, Th, lds, lds + 2 * S::L, blockIdx.x, 0, A->nsteps, nullptr,
                                   nullptr, nullptr);
  } else {
    const size_t at = (size_t)blockIdx.x * S::L;
    l_steps<d, N, OPEN, CK, false>(A, Bg, Th, lds, lds + 2 * S::L, blockIdx.x, n_lo, n_hi,
                                   st_in ? st_in + at : nullptr, st_out ? st_out + at : nullptr, nullptr);
  }
}

// The reverse walk of a column, segment by segment from the last: recompute the
// stage inputs from the checkpoint, then back with the costate (hi, lo).
// With kb' = P^dag kb and K = R kb' - kb' R: yb' = i K + D^dag(kb'), and the
// sensitivities are 2 Im(conj(K_c) y') of the couplings' and drives' own parts
// K_c and 2 Re(conj(D_m) y') of the rates'; all use the neighbours that yb'
// gathers.
template <int d, int N>
__global__ void __launch_bounds__((LShape<d, N, true>::TB))
l_adj_kernel(const GArgs* __restrict__ Ag, const GAdj* __restrict__ Bg) {
  using S = LShape<d, N, true>;
  constexpr int L = S::L, T = S::T, E = S::E, H = S::H, NW = S::NW, NV = S::NV, dd = S::dd;
  extern __shared__ __align__(16) c32 lds[];
  kptr<GArgs> A = kconst(Ag);
  kptr<GAdj> B = kconst(Bg);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = blockIdx.x;
  const float h = A->h;
  const int nsteps = A->nsteps, ce = B->ce, nck = B->nck;
  const int nds = uni(A->nds), ncp = uni(A->ncp), nv = ncp + 2 * N;
  float* tab = reinterpret_cast<float*>(lds + S::bufs);
  float* wsum = tab + S::at_s;
  c32* lo = lds + 2 * L;   // low words, where they lie in LDS
  LThread<d, N, true> Th;
  Th.init(A, tab, true);
  const unsigned tid = Th.tid;
  const bool on = Th.on;
  c32* segc = (c32*)B->seg + (size_t)col * ce * 4 * L;
  float4* lsave = B->lam + (size_t)col * L;
  double vstep = 0.0;
#pragma unroll 1
  for (int g = nck - 1; g >= 0; --g) {
    const int n0 = g * ce, n1 = min(nsteps, n0 + ce);
    l_steps<d, N, true, false, true>(A, Bg, Th, lds, lo, col, n0, n1, B->ck + ((size_t)col * nck + g) * L,
                               nullptr, segc);
    // ---- back
    float lhr[E], lhm[E], llr[S::LO ? 1 : E], llm[S::LO ? 1 : E];
    auto low = [&](int r) {
      c32 l;
      if constexpr (S::LO) {
        l = lo[tid + r * T];
      } else {
        l.x = llr[r];
        l.y = llm[r];
      }
      return l;
    };
    auto set_low = [&](int r, c32 l) {
      if constexpr (S::LO) {
        if (on) lo[tid + r * T] = l;
      } else {
        llr[r] = l.x;
        llm[r] = l.y;
      }
    };
    c32 kb[E];
    float c[N], cn[N];
#pragma unroll
    for (int m = 0; m < N; ++m) c[m] = cn[m] = 0.f;
    c32 P1[E];
    Th.phases(2 * n1, P1);
    Th.drives(stage_c(n1 - 1, 3), c);
    const float c3 = h * (1.0f / 6.0f);
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const int e = tid + r * T;
      float4 v;
      if (g == nck - 1) {
        const c32 q = ((const c32*)B->cot)[(size_t)col * L + e];
        v = make_float4(q.x, q.y, 0.f, 0.f);
      } else {
        v = lsave[e];
      }
      lhr[r] = v.x;
      lhm[r] = v.y;
      c32 k, l;
      k.x = c3 * v.x;
      k.y = c3 * v.y;
      l.x = v.z;
      l.y = v.w;
      set_low(r, l);
      kb[r] = c_mul_conj(P1[r], k);
      if (on) lds[e] = kb[r];
    }
    __syncthreads();
    int prev_n = -1, prev_s = 0, par = 0, cur = 0;
    auto fold_prev = [&]() {
      if ((int)threadIdx.x >= nds + nv) return;
      const int t = threadIdx.x, k = t < nds ? t : N + t - nds;
      double G = 0.0;
      for (int w = 0; w < NW; ++w) G += (double)wsum[((par ^ 1) * NW + w) * NV + k];
      G *= A->kappa;   // the sums are those of the unscaled operators
      double* row = B->gs + ((size_t)col * nsteps + prev_n) * B->gw;
      if (t < nds) {
        row[prev_s * nds + t] = G;
      } else {
        vstep = prev_s == 3 ? G : vstep + G;
        if (prev_s == 0) row[3 * nds + t] = vstep;
      }
    };
#pragma unroll 1
    for (int n = n1 - 1; n >= n0; --n) {
#pragma unroll 1
      for (int s = 3; s >= 0; --s) {
        const c32* kbw = lds + cur * L;
        c32* kbn = lds + (cur ^ 1) * L;
        // this stage's input; the next stage of the walk, (n, s - 1) or
        // (n - 1, 3): its drive coefficients, phases and the weights of its kb
        c32 y[E];
#pragma unroll
        for (int r = 0; r < E; ++r) y[r] = (segc + ((size_t)(n - n0) * 4 + s) * L + r * T)[tid];
        Th.drives(s > 0 ? stage_c(n, s - 1) : stage_c(max(n - 1, 0), 3), cn);
        const float cs = (s == 1 || s == 0) ? h * (1.0f / 6.0f) : h * (1.0f / 3.0f);
        const float cy = s == 0 ? 0.f : (s == 3 ? h : 0.5f * h);
        if (prev_n >= 0) fold_prev();
        float* wv = wsum + (par * NW + wave) * NV;
        // a thread past the last element adds nothing to the sums
        auto sum = [&](int k, float v) {
          const float u = g_wave_sum(on ? 2.f * v : 0.f);
          if (lane == 0) wv[k] = u;
        };
        auto zero = [](int) {
          c32 v;
          v.x = v.y = 0.f;
          return v;
        };
        c32 z[E];   // K, with D^dag turned by -i
#pragma unroll
        for (int r = 0; r < E; ++r) {
          const float f = Th.dg + tab[S::at_f + r];
          z[r].x = f * kb[r].x;
          z[r].y = f * kb[r].y;
        }
        static_for<N>([&](auto Pc) {
          constexpr int p = decltype(Pc)::value;
          if (!((Th.pmask >> p) & 1)) return;
          const int nc = uni(A->rp_n[p]);
          const int c0 = uni(A->rp_c[p][0]), c1 = uni(A->rp_c[p][1]);
          const float g0 = unif((float)(A->kappa * A->cp_g[c0]));
          const float* rows = tab + S::at_c + p * 2 * dd * S::pr;
          const float* urows = Th.rt + S::off_c + p * 2 * dd * S::pr;
          float v0 = 0.f, v1 = 0.f;
          auto one = [&](int r, c32 t, float g, float& v) {
            l_mac(z[r], g, t);
            v = fmaf(t.x, y[r].y, fmaf(-t.y, y[r].x, v));
            l_pin(z[r].x, z[r].y, v);
          };
          if (nc > 1) {
            const float g1 = unif((float)(A->kappa * A->cp_g[c1]));
            auto two = [&](int r, const c32(&t)[2]) {
              one(r, t[0], g0, v0);
              one(r, t[1], g1, v1);
            };
            Th.template pair<p, 0, 2>(kbw, kb, rows, urows, zero, two);
            Th.template pair<p, 1, 2>(kbw, kb, rows, urows, zero, two);
            sum(N + c1, v1);
          } else {
            auto sole = [&](int r, const c32(&t)[1]) { one(r, t[0], g0, v0); };
            Th.template pair<p, 0, 1>(kbw, kb, rows, urows, zero, sole);
            Th.template pair<p, 1, 1>(kbw, kb, rows, urows, zero, sole);
          }
          sum(N + c0, v0);
          __builtin_amdgcn_sched_barrier(0);
        });
        static_for<N>([&](auto M) {
          constexpr int m = decltype(M)::value;
          if (!((Th.dmask >> m) & 1)) return;
          float v = 0.f;
          auto one = [&](int r, c32 t) {
            l_mac(z[r], c[m], t);
            v = fmaf(t.x, y[r].y, fmaf(-t.y, y[r].x, v));
            l_pin(z[r].x, z[r].y, v);
          };
          Th.template drive<m, 0>(kbw, kb, 1.f, zero, one);
          Th.template drive<m, 1>(kbw, kb, 1.f, zero, one);
          // the row is the operator over its largest entry
          sum(uni(A->rd_k[m]), v / unif(A->rd_s[m]));
          __builtin_amdgcn_sched_barrier(0);
        });
        c32 P[E], Q[E];   // phases of the stage and of the next one
        Th.phases(2 * n + ((s + 1) >> 1), P);
        Th.phases(2 * n + (s >> 1), Q);
        // rates: D_m^dag(kb) = sqrt(a b) kb(a - 1, b - 1) - (a + b) / 2 kb, -(a - b)^2 kb
        float t[E], tt = 0.f;
#pragma unroll
        for (int r = 0; r < E; ++r) {
          t[r] = fmaf(kb[r].x, y[r].x, kb[r].y * y[r].y);
          tt += t[r];
        }
        static_for<N>([&](auto M) {
          constexpr int m = decltype(M)::value;
          const float g1 = unif((float)(A->kappa * A->g1[m]));
          const auto X = Th.digits();
          const float b = (float)X.dig(1, m);
          float v1 = 0.f, v2 = 0.f;
          Th.template jump<m, true>(kbw, [&](int r, c32 v) {
            z[r].x = fmaf(g1, v.y, z[r].x);
            z[r].y = fmaf(-g1, v.x, z[r].y);
            v1 = fmaf(v.x, y[r].x, fmaf(v.y, y[r].y, v1));
            l_pin(z[r].x, z[r].y, v1);
          });
          if constexpr (m >= H) {
            const float a = (float)X.dig(0, m);
            v1 = fmaf(-0.5f * (a + b), tt, v1);
            v2 = -(a - b) * (a - b) * tt;
          } else {
#pragma unroll
            for (int r = 0; r < E; ++r) {
              const float a = (float)S::rd(r, m);
              v1 = fmaf(-0.5f * (a + b), t[r], v1);
              v2 = fmaf(-(a - b) * (a - b), t[r], v2);
            }
          }
          sum(N + ncp + 2 * m, v1);
          sum(N + ncp + 2 * m + 1, v2);
        });
        const auto D = Th.decay();
#pragma unroll
        for (int r = 0; r < E; ++r) {
          const float f = D.of(r);
          c32 x;
          x.x = fmaf(f, kb[r].x, -z[r].y);
          x.y = fmaf(f, kb[r].y, z[r].x);
          z[r] = c_mul(P[r], x);
        }
        // the step's increments yb gather in the low word; at its end they go
        // into hi (fast two-sum), which the next stage's kb starts from
#pragma unroll
        for (int r = 0; r < E; ++r) {
          c32 l = low(r);
          l.x += z[r].x;
          l.y += z[r].y;
          const float u = s == 0 ? lhr[r] + l.x : lhr[r], v = s == 0 ? lhm[r] + l.y : lhm[r];
          l.x -= u - lhr[r];
          l.y -= v - lhm[r];
          lhr[r] = u;
          lhm[r] = v;
          set_low(r, l);
          c32 k;
          k.x = fmaf(cs, u, cy * z[r].x);
          k.y = fmaf(cs, v, cy * z[r].y);
          kb[r] = c_mul_conj(Q[r], k);
        }
        if (on) {
#pragma unroll
          for (int r = 0; r < E; ++r) kbn[tid + r * T] = kb[r];
        }
#pragma unroll
        for (int m = 0; m < N; ++m) c[m] = cn[m];
        prev_n = n;
        prev_s = s;
        par ^= 1;
        cur ^= 1;
        __syncthreads();
      }
    }
    fold_prev();   // the last stage's sums
    if (g > 0) {
#pragma unroll
      for (int r = 0; r < E; ++r) {
        const c32 l = low(r);
        if (on) lsave[tid + r * T] = make_float4(lhr[r], lhm[r], l.x, l.y);
      }
    }
    __syncthreads();
  }
}

template <typename K, typename... Args>
hipError_t l_launch(K* kernel, int S, int threads, size_t sh, hipStream_t s, Args... args) {
  (void)hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
  hipLaunchKernelGGL(kernel, dim3(S), dim3(threads), sh, s, args...);
  return hipGetLastError();
}

template <int d, int N, bool OPEN, bool CK>
hipError_t l_forward(const GArgs* dargs, const GAdj* dadj, int S, int n_lo, int n_hi,
                     const float4* st_in, float4* st_out, hipStream_t s) {
  using Z = LShape<d, N, OPEN>;
  return l_launch(l_rk4_kernel<d, N, OPEN, CK>, S, Z::TB, Z::fwd_bytes(), s, dargs, dadj, n_lo, n_hi,
                  st_in, st_out);
}

}  // namespace

// Open shapes of three modes and more (two modes have one pair, which the ring
// of modes would count twice).
#define GA_OPEN_REAL(X) X(2, 3) X(2, 4) X(2, 5) X(3, 3) X(3, 4) X(4, 3)

hipError_t l_real_forward(int d, int N, const GArgs* dargs, const GAdj* dadj, int S, int nsteps,
                          hipStream_t s) {
#define L_FWD(dd_, nn_)                                                                              \
  if (d == dd_ && N == nn_)                                                                          \
    return dadj ? l_forward<dd_, nn_, true, true>(dargs, dadj, S, 0, nsteps, nullptr, nullptr, s)    \
                : l_forward<dd_, nn_, true, false>(dargs, dadj, S, 0, nsteps, nullptr, nullptr, s);
  GA_OPEN_REAL(L_FWD)
#undef L_FWD
  return hipErrorInvalidValue;
}

// The one shape above the gather engine's D <= 4096 whose two buffers and low words
// (24 D bytes) fit the 160 KB of LDS with rows of more than one entry.
bool l_column_supported(int d, int N) { return d == 3 && N == 8; }

hipError_t l_real_column(int d, int N, const GArgs* dargs, int S, int n_lo, int n_hi,
                         const float4* st_in, float4* st_out, hipStream_t s) {
  if (!l_column_supported(d, N)) return hipErrorInvalidValue;
  return l_forward<3, 8, false, false>(dargs, nullptr, S, n_lo, n_hi, st_in, st_out, s);
}

hipError_t l_real_adjoint(int d, int N, const GArgs* dargs, const GAdj* dadj, int S, hipStream_t s) {
#define L_ADJ(dd_, nn_)                                                                            \
  if (d == dd_ && N == nn_)                                                                        \
    return l_launch(l_adj_kernel<dd_, nn_>, S, LShape<dd_, nn_, true>::TB,                         \
                    LShape<dd_, nn_, true>::adj_bytes(), s, dargs, dadj);
  GA_OPEN_REAL(L_ADJ)
#undef L_ADJ
  return hipErrorInvalidValue;
}

bool l_real_supported(int d, int N) {
#define L_HAS(dd_, nn_) if (d == dd_ && N == nn_) return true;
  GA_OPEN_REAL(L_HAS)
#undef L_HAS
  return false;
}

}  // namespace scp
