// Gather engine: classical RK4 with one column per workgroup, the column held
// in LDS for the whole propagation and every thread evaluating the generator
// on its own elements by gathering their neighbours along the contracted
// digits.  Two uses:
//
// Closed systems (OPEN = false): a state column psi of D = d^N amplitudes
// (element A, the multi-index of the N modes, mode 0 slowest) under the
// interaction-picture generator of Sec. 2.1's local decomposition,
//   k_A = -i [ delta(A) y_A + sum (one- and two-mode contractions of V) ],
// for devices whose columns are too few to fill the chip with the register-
// layout stepper (the 4-fluxonium chain: 16 columns of 625).  This file has the
// general form and the one for operators between levels of unlike parity (PAR);
// gather_real.hip and open_real.hip have the forms for real terms.
//
// Open systems (OPEN = true): the vectorised Lindblad master equation (the
// superoperator form of App. D's closing remark; the LindbladObj component of
// Sec. 2).  rho (D x D) is the rank-2N tensor rho[a_0..a_{N-1}, b_0..b_{N-1}]
// stored row-major: element A*D + B, A the ket and B the bra multi-index.  In
// the interaction picture of the frame,
//   d rho/dt = -i (V rho - rho V) + sum_m g1_m D[a_m(t)] rho + 2 gphi_m D[n_m] rho,
// D[L] rho = L rho L^dag - {L^dag L, rho}/2, a the ladder and n the number
// operator of mode m in its dressed basis.  Per element (A, B):
//   k_AB = dg_AB rho_AB                                       static diagonal
//        + sum_m g1_m J_m(t)[a_m][b_m] rho_{A+e_m, B+e_m}      relaxation jump
//        - i (ket contractions of V) + i (bra contractions of conj V),
//   dg_AB = -i sum_m (delta_m[a_m] - delta_m[b_m]) - sum_m g1_m (a_m + b_m)/2
//           - sum_m gphi_m (a_m - b_m)^2,
//   J_m(t)[a][b] = sqrt((a+1)(b+1)) exp(i (f_a - f_{a+1} - f_b + f_{b+1}) t),
// delta = eps - f the diagonal left by the frame f.
//
// The Hamiltonian enters as one-mode contractions (per driven mode the sum of
// c_k(t) O_k(t) of its drives) and two-mode contractions (per coupled pair of
// modes the d^2 x d^2 operator sum_e g_e O_i(t) (x) O_j(t)), along the ket
// digits with the operator and (open systems) along the bra digits with its
// complex conjugate.  These stage tables are precomputed for every stage row
// of the step grid (3 per step, as the drive coefficients) by one kernel; the
// stepper loads the next stage's table into registers while the current stage
// runs and stores it into LDS after.  LDS holds two stage-input buffers (a
// stage reads y_s from one and writes y_{s+1} into the other), the static
// diagonal and two stage tables; each thread keeps its elements' state
// (compensated hi + lo) and the RK4 accumulator in registers.  One barrier
// per stage.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>
#include <string>

#include "gather.h"

namespace scp {

#define SCP_TRY(expr)                  \
  do {                                 \
    const scp_status st_ = (expr);     \
    if (st_ != SCP_OK) return st_;     \
  } while (0)

namespace {

// Row of the drive table of step-grid row r (3 per step: t_n, t_n + h/2,
// t_n + h) and the half-step of its operators.
__device__ __forceinline__ int row_q(int r) { return 2 * (r / 3) + r % 3; }

// Stage table of step-grid row r: [driven-mode operators sum_k c_k O_k]
// [pair operators sum_e g_e O_i (x) O_j][relaxation bands g1_m J_m], from the
// FP32 rotated operators and coefficients.
__global__ void gtab_kernel(const GArgs* __restrict__ Ag, int d, int N, float2* __restrict__ out) {
  const GArgs& A = *Ag;
  const int r = blockIdx.x;
  const int q = row_q(r);
  const int dd = d * d;
  const c32* ops = (const c32*)A.optab + (size_t)q * A.block_q;
  const float* cq = A.ctab + (size_t)r * A.ngroups;
  const int ntot = A.grad ? A.ntabg : A.ntab;
  for (int t = threadIdx.x; t < ntot; t += blockDim.x) {
    float vr = 0.f, vi = 0.f;
    if (t >= A.ntab) {
      if (t < A.off_s + A.nsl * d * A.srow) {   // rotated slot operator
        const int u = t - A.off_s;
        const int k = u / (d * A.srow), a = (u / A.srow) % d, kb = u % A.srow;
        const int b = kb < A.nn ? nb_level(d, A.par, kb, a) : -1;
        if (b >= 0) {
          const c32 o = ops[A.sl_slot[k] * dd + a * d + b];
          vr = o.x;
          vi = o.y;
        }
      } else if (A.grad == 1) {         // unit-rate relaxation band (then row padding)
        if (t - A.off_u < N * dd) {
          const c32 j = ((const c32*)A.jtab)[((size_t)q * N) * dd + (t - A.off_u)];
          vr = j.x;
          vi = j.y;
        }
      } else if (t < A.off_d) {         // d/dtheta of mode m's one-mode terms
        const int u = t - A.off_m, dr = d * A.mrow;
        const int m = u / (3 * dr), th = (u / dr) % 3, a = (u / A.mrow) % d, kb = u % A.mrow;
        // parity: the diagonal sits behind the row's entries
        const int b = kb < A.nn ? nb_level(d, A.par, kb, a) : (A.par && kb == A.nn ? a : -1);
        const int ab = a * d + b;
        if (b == a) vr = A.deps[m][th][a];
        const int dm = A.mdm[m];
        if (dm >= 0 && b >= 0 && kb < A.nn)
          for (int k = 0; k < A.dm_n[dm]; ++k) {
            const float c = cq[A.dm_cidx[dm][k]];
            const c32 o = ops[A.off_dslot + (A.dm_slot[dm][k] * 3 + th) * dd + ab];
            vr = fmaf(c, o.x, vr);
            vi = fmaf(c, o.y, vi);
          }
      } else if (t < A.off_d + 3 * A.nsl * d * A.srow) {   // derivative slot operator
        const int u = t - A.off_d, dr = d * A.srow;
        const int k = u / (3 * dr), th = (u / dr) % 3, a = (u / A.srow) % d, kb = u % A.srow;
        const int b = kb < A.nn ? nb_level(d, A.par, kb, a) : -1;
        if (b >= 0) {
          const c32 o = ops[A.off_dslot + (A.sl_slot[k] * 3 + th) * dd + a * d + b];
          vr = o.x;
          vi = o.y;
        }
      }
    } else if (t < A.off_p) {
      const int dm = t / (d * A.orow), rr = t - dm * d * A.orow;
      const int ra = rr / A.orow, kb = rr - ra * A.orow;   // kb >= nn: row padding
      const int rb = kb < A.nn ? nb_level(d, A.par, kb, ra) : -1;
      const int ab = ra * d + rb;
      for (int k = 0; k < (dm < A.ndm && rb >= 0 ? A.dm_n[dm] : 0); ++k) {
        const float c = cq[A.dm_cidx[dm][k]];
        const c32 o = ops[A.dm_slot[dm][k] * dd + ab];
        vr = fmaf(c, o.x, vr);
        vi = fmaf(c, o.y, vi);
      }
    } else if (t < A.off_j) {
      const int u = t - A.off_p;
      const int p = u / (dd * A.prow), rr = u - p * dd * A.prow;
      const int row = rr / A.prow, col = rr - row * A.prow;   // col >= nn^2: row padding
      const int ai = row / d, aj = row - ai * d, kx = col / A.nn, kz = col - kx * A.nn;
      const int x = kx < A.nn ? nb_level(d, A.par, kx, ai) : -1;
      const int z = nb_level(d, A.par, kz, aj);
      for (int k = 0; k < (x >= 0 && z >= 0 ? A.pr_n[p] : 0); ++k) {
        const c32 oi = ops[A.pr_si[p][k] * dd + ai * d + x];
        const c32 oj = ops[A.pr_sj[p][k] * dd + aj * d + z];
        const float g = A.pr_g[p][k];
        vr = fmaf(g, oi.x * oj.x - oi.y * oj.y, vr);
        vi = fmaf(g, oi.x * oj.y + oi.y * oj.x, vi);
      }
    } else if (A.has_jump && t - A.off_j < N * dd) {   // relaxation bands (then row padding)
      const int u = t - A.off_j;
      const int m = u / dd;
      const c32 j = ((const c32*)A.jtab)[((size_t)q * N) * dd + u];
      vr = A.g1[m] * j.x;
      vi = A.g1[m] * j.y;
    }
    out[(size_t)r * ntot + t] = make_float2(vr, vi);
  }
}

// sum_k row[k] y_k (CONJ: conj(row[k])) over one driven-mode operator row of an
// element at `y` with digit a on a mode of stride st.  Operator rows are padded
// to an even length, so a row starts 16-byte aligned and is read two entries
// per LDS instruction.
template <int d, bool PAR, bool CONJ>
__device__ __forceinline__ void one_dot(const c32* __restrict__ row, const c32* __restrict__ y,
                                        int a, int st, float& sr, float& si) {
  using B = Nb<d, PAR>;
  const float4* r4 = reinterpret_cast<const float4*>(row);
  y += B::first(a, st);
#pragma unroll
  for (int k = 0; k < (B::n + 1) / 2; ++k) {
    const float4 q = r4[k];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (2 * k + u >= B::n) continue;
      c32 o;
      o.x = u ? q.z : q.x;
      o.y = u ? q.w : q.y;
      if (CONJ)
        cmac_conj(sr, si, o, y[B::step(2 * k + u, a, st)]);
      else
        cmac(sr, si, o, y[B::step(2 * k + u, a, st)]);
    }
  }
}

// The same over one pair-operator row, entry (x, z) of modes (i, j).
template <int d, bool PAR, bool CONJ>
__device__ __forceinline__ void pair_dot(const c32* __restrict__ row, const c32* __restrict__ y,
                                         int ai, int aj, int si_, int sj_, float& sr, float& si) {
  using B = Nb<d, PAR>;
  constexpr int nn = B::n * B::n;
  const float4* r4 = reinterpret_cast<const float4*>(row);
  const c32* y0 = y + (PAR ? B::first(ai, si_) + B::first(aj, sj_) : -(ai * si_ + aj * sj_));
#pragma unroll
  for (int k = 0; k < (nn + 1) / 2; ++k) {
    const float4 q = r4[k];
    c32 a;
    a.x = q.x;
    a.y = q.y;
    const c32 ya = y0[B::step((2 * k) / B::n, ai, si_) + B::step((2 * k) % B::n, aj, sj_)];
    if (CONJ)
      cmac_conj(sr, si, a, ya);
    else
      cmac(sr, si, a, ya);
    if (2 * k + 1 < nn) {
      c32 b;
      b.x = q.z;
      b.y = q.w;
      const c32 yb_ = y0[B::step((2 * k + 1) / B::n, ai, si_) + B::step((2 * k + 1) % B::n, aj, sj_)];
      if (CONJ)
        cmac_conj(sr, si, b, yb_);
      else
        cmac(sr, si, b, yb_);
    }
  }
}

// k = G(t) y for one element; y read from LDS (neighbours), the own value
// from the caller.
template <int d, int N, bool OPEN, bool PAR>
__device__ __forceinline__ void g_apply(kptr<GArgs> A, const c32* __restrict__ yb,
                                        const c32* __restrict__ tab, int e, uint32_t pk,
                                        float dgr, float dgi, float yr, float yi, float& kr,
                                        float& ki) {
  using Sh = GShape<d, N, OPEN>;
  constexpr int D = Sh::D, dd = d * d;
  kr = dgr * yr - dgi * yi;
  ki = fmaf(dgr, yi, dgi * yr);
  if (OPEN && uni(A->has_jump)) {
#pragma unroll
    for (int m = 0; m < N; ++m) {
      const int am = ket_digit(pk, m), bm = bra_digit(pk, m, N);
      if (am < d - 1 && bm < d - 1) {
        const c32 J = tab[A->off_j + m * dd + am * d + bm];
        const c32 v = yb[e + (D + 1) * Sh::st(m)];
        cmac(kr, ki, J, v);
      }
    }
  }
  // driven modes: ket -i Hd y, bra +i y Hd
  const int ndm = uni(A->ndm);
  for (int dmv = 0; dmv < ndm; ++dmv) {
    const int dm = uni(dmv);
    const int m = uni(A->dm_mode[dm]);
    {
      const int sm = uni(A->kst[m]);
      const int am = ket_digit(pk, m);
      const c32* row = tab + dm * d * Nb<d, PAR>::orow + am * Nb<d, PAR>::orow;
      float sr = 0.f, si = 0.f;
      one_dot<d, PAR, false>(row, yb + e, am, sm, sr, si);
      kr += si;
      ki -= sr;
    }
    if (OPEN) {
      const int sm = uni(A->bst[m]);
      const int bm = bra_digit(pk, m, N);
      const c32* row = tab + dm * d * Nb<d, PAR>::orow + bm * Nb<d, PAR>::orow;
      float sr = 0.f, si = 0.f;
      one_dot<d, PAR, true>(row, yb + e, bm, sm, sr, si);
      kr -= si;
      ki += sr;
    }
  }
  // coupled pairs
  const int npr = uni(A->npr);
  for (int pv = 0; pv < npr; ++pv) {
    const int p = uni(pv);
    const int i = uni(A->pr_i[p]), j = uni(A->pr_j[p]);
    constexpr int PR = Nb<d, PAR>::prow;
    const c32* P = tab + A->off_p + p * dd * PR;
    {
      const int si_ = uni(A->kst[i]), sj_ = uni(A->kst[j]);
      const int ai = ket_digit(pk, i), aj = ket_digit(pk, j);
      const c32* row = P + (ai * d + aj) * PR;
      float sr = 0.f, si = 0.f;
      pair_dot<d, PAR, false>(row, yb + e, ai, aj, si_, sj_, sr, si);
      kr += si;
      ki -= sr;
    }
    if (OPEN) {
      const int si_ = uni(A->bst[i]), sj_ = uni(A->bst[j]);
      const int bi = bra_digit(pk, i, N), bj = bra_digit(pk, j, N);
      const c32* row = P + (bi * d + bj) * PR;
      float sr = 0.f, si = 0.f;
      pair_dot<d, PAR, true>(row, yb + e, bi, bj, si_, sj_, sr, si);
      kr -= si;
      ki += sr;
    }
  }
}

// One column (col) of a propagation: the body of the stepper kernels.
template <int d, int N, bool OPEN, bool PAR, bool CK>
__device__ __forceinline__ void g_rk4_body(const GArgs* __restrict__ Ag, const GAdj* __restrict__ Bg,
                                           int col, int n_lo, int n_hi,
                                           const float4* __restrict__ st_in,
                                           float4* __restrict__ st_out) {
  using Sh = GShape<d, N, OPEN>;
  constexpr int L = Sh::L, T = Sh::T, E = Sh::E;
  // LDS: two stage-input buffers, the static diagonal, two stage tables
  extern __shared__ __align__(16) c32 lds[];
  kptr<GArgs> A = kconst(Ag);
  const int ntab = A->ntab;
  const int nrow = A->grad ? A->ntabg : ntab;   // table row stride in gtab
  c32* dgb = lds + 2 * L;
  const c32* gtab = (const c32*)A->gtab;
  const int tid = threadIdx.x;
  const float h = A->h;
  const int nsteps = A->nsteps;
  // steps n_lo .. n_hi - 1; the compensated state comes from st_in (else the
  // columns x0, lo = 0) and goes to st_out (a later call continues exactly)
  uint32_t pk[E];
  float hr[E], hm[E], lr[E], lm[E], ar[E], am_[E];
  float dgr_[E], dgi_[E];   // the element's static diagonal (closed systems: in registers)
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const int e = tid + r * T;
    const bool ok = e < L;
    const int Ai = OPEN ? e / Sh::D : e, Bi = OPEN ? e - Ai * Sh::D : 0;
    uint32_t p = 0;
    float gr = 0.f, gi = 0.f;
#pragma unroll
    for (int m = 0; m < N; ++m) {
      const int a = (Ai / Sh::st(m)) % d;
      p |= (uint32_t)a << (3 * m);
      if (OPEN) {
        const int b = (Bi / Sh::st(m)) % d;
        p |= (uint32_t)b << (3 * (N + m));
        gi -= A->delta[m][a] - A->delta[m][b];
        gr -= 0.5f * A->g1[m] * (float)(a + b) + A->gp[m] * (float)((a - b) * (a - b));
      } else {
        gi -= A->delta[m][a];
      }
    }
    pk[r] = p;
    c32 v;
    v.x = v.y = 0.f;
    lr[r] = lm[r] = 0.f;
    if (ok) {
      if (st_in != nullptr) {
        const float4 q = st_in[(size_t)col * L + e];
        v.x = q.x;
        v.y = q.y;
        lr[r] = q.z;
        lm[r] = q.w;
      } else {
        v = ((const c32*)A->x0)[(size_t)col * L + e];
      }
    }
    hr[r] = v.x;
    hm[r] = v.y;
    ar[r] = am_[r] = 0.f;
    dgr_[r] = gr;
    dgi_[r] = gi;
    if (ok) {
      lds[e] = v;
      if (OPEN) {
        c32 g;
        g.x = gr;
        g.y = gi;
        dgb[e] = g;
      }
    }
  }
  // the stage tables start 16-byte aligned (operator rows are read two
  // entries at a time)
  constexpr int TB = 3 * L + ((3 * L) & 1);
  for (int t = tid; t < ntab; t += T) lds[TB + t] = gtab[(size_t)stage_c(n_lo, 0) * nrow + t];
  __syncthreads();
  // closed systems move table rows two entries (16 bytes) at a time: the
  // tables' rows and LDS buffers are 16-byte aligned and of even length
  constexpr int GP4 = GA_PRE / 2;
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
#pragma unroll 1
    for (int s = 0; s < 4; ++s) {
      const float w = (s == 0 || s == 3) ? 1.f : 2.f;
      const float ch = (s == 2) ? h : 0.5f * h;
      const c32* yc = lds + cur * L;
      const c32* tc = lds + TB + cur * ntab;
      c32* yn = lds + (cur ^ 1) * L;
      // the next stage's table, loaded now and stored after this stage
      const int n2 = s < 3 ? n : n + 1, s2 = s < 3 ? s + 1 : 0;
      const bool more = n2 < n_hi;
      const c32* gnext = gtab + (size_t)stage_c(n2, s2) * nrow;
      c32 pre[OPEN ? GA_PRE : 1];
      float4 pre4[OPEN ? 1 : GP4];
      if constexpr (OPEN) {
#pragma unroll
        for (int k = 0; k < GA_PRE; ++k) {
          const int t = tid + k * T;
          if (more && t < ntab) pre[k] = gnext[t];
        }
      } else {
#pragma unroll
        for (int k = 0; k < GP4; ++k) {
          const int t = tid + k * T;
          pre4[k] = (more && 2 * t < ntab) ? reinterpret_cast<const float4*>(gnext)[t]
                                           : make_float4(0.f, 0.f, 0.f, 0.f);
        }
      }
#pragma unroll
      for (int r = 0; r < E; ++r) {
        int e = tid + r * T;
        uint32_t p = pk[r];
        // opaque per stage: the element's LDS offsets are then formed inside
        // the stage instead of being hoisted out of the step loop (which
        // would hold E sets of them in registers)
        asm volatile("" : "+v"(e), "+v"(p));
        if (e < L) {
          c32 g;
          if (OPEN) {
            g = dgb[e];
          } else {
            g.x = dgr_[r];
            g.y = dgi_[r];
          }
          const c32 ye = yc[e];
          float kr, ki;
          g_apply<d, N, OPEN, PAR>(A, yc, tc, e, p, g.x, g.y, ye.x, ye.y, kr, ki);
          if (s == 0) {
            ar[r] = kr;
            am_[r] = ki;
          } else {
            ar[r] = fmaf(w, kr, ar[r]);
            am_[r] = fmaf(w, ki, am_[r]);
          }
          c32 v;
          if (s < 3) {
            v.x = fmaf(ch, kr, hr[r]);
            v.y = fmaf(ch, ki, hm[r]);
          } else {
            const float h6 = h * (1.0f / 6.0f);
            comp_add(hr[r], lr[r], h6 * ar[r]);
            comp_add(hm[r], lm[r], h6 * am_[r]);
            v.x = hr[r];
            v.y = hm[r];
          }
          yn[e] = v;
        }
        // one element at a time: keeps the live registers of the unrolled
        // element loop from piling up across elements
        __builtin_amdgcn_sched_barrier(0);
      }
      if (more) {
        c32* tn = lds + TB + (cur ^ 1) * ntab;
        if constexpr (OPEN) {
#pragma unroll
          for (int k = 0; k < GA_PRE; ++k) {
            const int t = tid + k * T;
            if (t < ntab) tn[t] = pre[k];
          }
          for (int t = tid + GA_PRE * T; t < ntab; t += T) tn[t] = gnext[t];
        } else {
          float4* tn4 = reinterpret_cast<float4*>(tn);
          const float4* gn4 = reinterpret_cast<const float4*>(gnext);
#pragma unroll
          for (int k = 0; k < GP4; ++k) {
            const int t = tid + k * T;
            if (2 * t < ntab) tn4[t] = pre4[k];
          }
          for (int t = tid + GP4 * T; 2 * t < ntab; t += T) tn4[t] = gn4[t];
        }
      }
      __syncthreads();
      cur ^= 1;
    }
  }
  if (st_out != nullptr) {
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const int e = tid + r * T;
      if (e < L) st_out[(size_t)col * L + e] = make_float4(hr[r], hm[r], lr[r], lm[r]);
    }
  }
  if (A->xT == nullptr || n_hi < nsteps) return;
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const int e = tid + r * T;
    if (e < L) {
      c32 v;
      v.x = hr[r] + lr[r];
      v.y = hm[r] + lm[r];
      ((c32*)A->xT)[(size_t)col * L + e] = v;
    }
  }
}

template <int d, int N, bool OPEN, bool PAR, bool CK>
__global__ void __launch_bounds__((GShape<d, N, OPEN>::T))
g_rk4_kernel(const GArgs* __restrict__ Ag, const GAdj* __restrict__ Bg, int n_lo, int n_hi,
             const float4* __restrict__ st_in, float4* __restrict__ st_out) {
  g_rk4_body<d, N, OPEN, PAR, CK>(Ag, Bg, blockIdx.x, n_lo, n_hi, st_in, st_out);
}

// Batched (serving): every workgroup reads its own work item -- its request's
// description, column, step range and state buffers.
template <int d, int N, bool PAR, bool CK>
__global__ void __launch_bounds__((GShape<d, N, false>::T))
g_rk4_batched_kernel(const GItem* __restrict__ items) {
  kptr<GItem> it = kconst(items) + blockIdx.x;
  g_rk4_body<d, N, false, PAR, CK>((const GArgs*)it->A, (const GAdj*)it->B, it->col, it->n_lo,
                              it->n_hi, it->st_in, it->st_out);
}

// ---------------------------------------------------------------------------
// open-system adjoint (discrete adjoint of the RK4 steps, as the closed
// system's: kb_s from the costate, yb_s = L_s^dag kb_s, lambda += sum yb_s,
// dLoss/dtheta += 2 Re <kb_s, dL_s/dtheta y_s>), one workgroup per column
// walking the checkpoint segments backwards: each segment is recomputed from
// its checkpoint with its stage inputs stored, then walked in reverse.
// ---------------------------------------------------------------------------

// L^dag x for one element: the Hamiltonian part with the opposite sign, the
// static diagonal conjugated, the relaxation jump transposed
// (conj(J[a-1][b-1]) x_{A-e_m, B-e_m}).  Closed systems: G^dag = i (delta + H).
template <int d, int N, bool OPEN, bool PAR>
__device__ __forceinline__ void g_apply_adj(kptr<GArgs> A, const c32* __restrict__ xb,
                                            const c32* __restrict__ tab, int e, uint32_t pk,
                                            float dgr, float dgi, float xr, float xi, float& yr,
                                            float& yi) {
  using Sh = GShape<d, N, OPEN>;
  constexpr int D = Sh::D, dd = d * d;
  yr = dgr * xr + dgi * xi;
  yi = dgr * xi - dgi * xr;
  if (OPEN && uni(A->has_jump)) {
#pragma unroll
    for (int m = 0; m < N; ++m) {
      const int am = ket_digit(pk, m), bm = bra_digit(pk, m, N);
      if (am > 0 && bm > 0) {
        const c32 J = tab[A->off_j + m * dd + (am - 1) * d + (bm - 1)];
        const c32 v = xb[e - (D + 1) * Sh::st(m)];
        cmac_conj(yr, yi, J, v);
      }
    }
  }
  const int ndm = uni(A->ndm);
  for (int dmv = 0; dmv < ndm; ++dmv) {
    const int dm = uni(dmv);
    const int m = uni(A->dm_mode[dm]);
    {
      const int sm = uni(A->kst[m]);
      const int am = ket_digit(pk, m);
      const c32* row = tab + dm * d * Nb<d, PAR>::orow + am * Nb<d, PAR>::orow;
      float sr = 0.f, si = 0.f;
      one_dot<d, PAR, false>(row, xb + e, am, sm, sr, si);
      yr -= si;
      yi += sr;
    }
    if (OPEN) {
      const int sm = uni(A->bst[m]);
      const int bm = bra_digit(pk, m, N);
      const c32* row = tab + dm * d * Nb<d, PAR>::orow + bm * Nb<d, PAR>::orow;
      float sr = 0.f, si = 0.f;
      one_dot<d, PAR, true>(row, xb + e, bm, sm, sr, si);
      yr += si;
      yi -= sr;
    }
  }
  const int npr = uni(A->npr);
  for (int pv = 0; pv < npr; ++pv) {
    const int p = uni(pv);
    const int i = uni(A->pr_i[p]), j = uni(A->pr_j[p]);
    constexpr int PR = Nb<d, PAR>::prow;
    const c32* P = tab + A->off_p + p * dd * PR;
    {
      const int si_ = uni(A->kst[i]), sj_ = uni(A->kst[j]);
      const int ai = ket_digit(pk, i), aj = ket_digit(pk, j);
      const c32* row = P + (ai * d + aj) * PR;
      float sr = 0.f, si = 0.f;
      pair_dot<d, PAR, false>(row, xb + e, ai, aj, si_, sj_, sr, si);
      yr -= si;
      yi += sr;
    }
    if (OPEN) {
      const int si_ = uni(A->bst[i]), sj_ = uni(A->bst[j]);
      const int bi = bra_digit(pk, i, N), bj = bra_digit(pk, j, N);
      const c32* row = P + (bi * d + bj) * PR;
      float sr = 0.f, si = 0.f;
      pair_dot<d, PAR, true>(row, xb + e, bi, bj, si_, sj_, sr, si);
      yr += si;
      yi -= sr;
    }
  }
}

// z = (O kb - kb O) at one element for a one-mode operator O (table rows at
// `rows`, O Hermitian): the commutator's ket gather minus its bra gather.
template <int d, int N, bool PAR>
__device__ __forceinline__ c32 comm1(const c32* __restrict__ kb, const c32* __restrict__ rows,
                                     int e, int am, int bm, int ks, int bs) {
  using B = Nb<d, PAR>;
  float kr = 0.f, ki = 0.f, br = 0.f, bi = 0.f;
  const c32* k0 = kb + e + B::first(am, ks);
  const c32* b0 = kb + e + B::first(bm, bs);
#pragma unroll
  for (int x = 0; x < B::n; ++x) {
    cmac(kr, ki, rows[am * B::srow + x], k0[B::step(x, am, ks)]);
    cmac_conj(br, bi, rows[bm * B::srow + x], b0[B::step(x, bm, bs)]);
  }
  c32 z;
  z.x = kr - br;
  z.y = ki - bi;
  return z;
}

// z = (P kb - kb P) at one element for P = Oi (x) Oj on modes (i, j).
template <int d, int N, bool PAR>
__device__ __forceinline__ c32 comm2(const c32* __restrict__ kb, const c32* __restrict__ Ri,
                                     const c32* __restrict__ Rj, int e, int ai, int aj, int bi,
                                     int bj, int ksi, int ksj, int bsi, int bsj) {
  using B = Nb<d, PAR>;
  float kr = 0.f, ki = 0.f, br = 0.f, bim = 0.f;
  const c32* k0 = kb + e + B::first(ai, ksi) + B::first(aj, ksj);
  const c32* b0 = kb + e + B::first(bi, bsi) + B::first(bj, bsj);
#pragma unroll
  for (int x = 0; x < B::n; ++x) {
    float ir = 0.f, ii = 0.f, jr = 0.f, ji = 0.f;
#pragma unroll
    for (int z = 0; z < B::n; ++z) {
      cmac(ir, ii, Rj[aj * B::srow + z], k0[B::step(x, ai, ksi) + B::step(z, aj, ksj)]);
      cmac_conj(jr, ji, Rj[bj * B::srow + z], b0[B::step(x, bi, bsi) + B::step(z, bj, bsj)]);
    }
    c32 u, w;
    u.x = ir;
    u.y = ii;
    w.x = jr;
    w.y = ji;
    cmac(kr, ki, Ri[ai * B::srow + x], u);
    cmac_conj(br, bim, Ri[bi * B::srow + x], w);
  }
  c32 z;
  z.x = kr - br;
  z.y = ki - bim;
  return z;
}

// s = sum_x row[x] v[x]
template <int n>
__device__ __forceinline__ c32 rowdot(const c32* __restrict__ row, const c32 (&v)[n]) {
  float sr = 0.f, si = 0.f;
#pragma unroll
  for (int x = 0; x < n; ++x) cmac(sr, si, row[x], v[x]);
  c32 z;
  z.x = sr;
  z.y = si;
  return z;
}

// Im(conj(a) b)
__device__ __forceinline__ float im_conj(c32 a, c32 b) { return a.x * b.y - a.y * b.x; }

// w[x] = conj(v[x]) b
template <int n>
__device__ __forceinline__ void conj_scale(const c32 (&v)[n], c32 b, c32 (&w)[n]) {
#pragma unroll
  for (int x = 0; x < n; ++x) {
    w[x].x = fmaf(v[x].x, b.x, v[x].y * b.y);
    w[x].y = fmaf(v[x].x, b.y, -v[x].y * b.x);
  }
}

// Im(conj(sum_x row[x] v[x]) b) = sum_x Im(conj(row[x]) w[x]) with w = conj(v) b
template <int n>
__device__ __forceinline__ float im_rowdot(const c32* __restrict__ row, const c32 (&w)[n]) {
  float s = 0.f;
#pragma unroll
  for (int x = 0; x < n; ++x) {
    s = fmaf(row[x].x, w[x].y, s);
    s = fmaf(-row[x].y, w[x].x, s);
  }
  return s;
}

// Closed systems, costate sweep of one column over the segments g_hi down to
// g_lo: only the costate is carried (the step map's adjoint needs no forward
// state: kb_s = c_s lambda + c'_s yb_{s+1}, yb_s = i V_s kb_s), and its value at
// the end of every segment is kept.  The segments' own walks, with their
// sensitivities, then run side by side instead of one after the other: they
// are the larger part of a gradient, and a device of few columns leaves most
// of the chip idle.  Forward + gradient, one segment after the other -> side by
// side: 4-fluxonium chain (16 columns) 62 -> 29 us per step, 5-transmon ring
// (32 columns) 49 -> 21.  Entered with the costate at the end of g_hi in lam (the
// last segment: from the cotangent); leaves it at the end of g_lo - 1.
template <int d, int N, bool PAR>
__device__ __forceinline__ void g_cos_body(const GArgs* __restrict__ Ag, const GAdj* __restrict__ Bg,
                                           int col, int g_hi, int g_lo) {
  using Sh = GShape<d, N, false>;
  constexpr int L = Sh::L, T = Sh::T, E = Sh::E;
  extern __shared__ __align__(16) c32 lds[];
  kptr<GArgs> A = kconst(Ag);
  kptr<GAdj> B = kconst(Bg);
  const int ntab = A->ntab, nrow = A->ntabg;
  const c32* gtab = (const c32*)A->gtab;
  const int tid = threadIdx.x;
  const float h = A->h;
  const int nsteps = A->nsteps, ce = B->ce, nck = B->nck;
  float4* lam = B->lam + (size_t)col * nck * L;
  uint32_t pk[E];
  float lhr[E], lhm[E], llr[E], llm[E], dg[E];
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const int e = tid + r * T;
    uint32_t p = 0;
    float g = 0.f;
#pragma unroll
    for (int m = 0; m < N; ++m) {
      const int a = (e / Sh::st(m)) % d;
      p |= (uint32_t)a << (3 * m);
      g -= A->delta[m][a];
    }
    pk[r] = p;
    dg[r] = g;
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
  constexpr int TB = 2 * L;   // two kb buffers, then two stage tables (16-byte aligned)
  constexpr int GP4 = GA_PRE / 2;
  const int n_hi = min(nsteps, (g_hi + 1) * ce), n_lo = max(g_lo, 1) * ce;
  {
    const c32* g0 = gtab + (size_t)stage_c(n_hi - 1, 3) * nrow;
    for (int t = tid; t < ntab; t += T) lds[TB + t] = g0[t];
  }
  int cur = 0;
#pragma unroll 1
  for (int n = n_hi - 1; n >= n_lo; --n) {
    float ybr[E], ybm[E];
#pragma unroll
    for (int r = 0; r < E; ++r) ybr[r] = ybm[r] = 0.f;
#pragma unroll 1
    for (int s = 3; s >= 0; --s) {
      const float cs = (s == 0 || s == 3) ? h * (1.0f / 6.0f) : h * (1.0f / 3.0f);
      const float cy = (s == 3) ? 0.f : (s == 2 ? h : 0.5f * h);
      c32* kbw = lds + cur * L;
      const c32* tw = lds + TB + cur * ntab;
#pragma unroll
      for (int r = 0; r < E; ++r) {
        const int e = tid + r * T;
        if (e < L) {
          c32 v;
          v.x = fmaf(cs, lhr[r], cy * ybr[r]);
          v.y = fmaf(cs, lhm[r], cy * ybm[r]);
          kbw[e] = v;
        }
      }
      __syncthreads();
      // the next (earlier) stage's table, loaded now and stored after this stage
      const int nn = s > 0 ? n : n - 1, sn = s > 0 ? s - 1 : 3;
      const bool more = nn >= n_lo;
      const c32* gnext = gtab + (size_t)stage_c(more ? nn : n, more ? sn : s) * nrow;
      float4 pre4[GP4];
#pragma unroll
      for (int k = 0; k < GP4; ++k) {
        const int t = tid + k * T;
        if (2 * t < ntab) pre4[k] = reinterpret_cast<const float4*>(gnext)[t];
      }
#pragma unroll
      for (int r = 0; r < E; ++r) {
        int e = tid + r * T;
        uint32_t p = pk[r];
        asm volatile("" : "+v"(e), "+v"(p));
        if (e < L) {
          const c32 kbe = kbw[e];
          float yr_, yi_;
          g_apply_adj<d, N, false, PAR>(A, kbw, tw, e, p, 0.f, dg[r], kbe.x, kbe.y, yr_, yi_);
          ybr[r] = yr_;
          ybm[r] = yi_;
          llr[r] += yr_;
          llm[r] += yi_;
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (more) {
        float4* tn4 = reinterpret_cast<float4*>(lds + TB + (cur ^ 1) * ntab);
#pragma unroll
        for (int k = 0; k < GP4; ++k) {
          const int t = tid + k * T;
          if (2 * t < ntab) tn4[t] = pre4[k];
        }
        for (int t = tid + GP4 * T; 2 * t < ntab; t += T)
          tn4[t] = reinterpret_cast<const float4*>(gnext)[t];
      }
      cur ^= 1;
    }
    // lambda_n (fast two-sum, as in the segments' walks)
#pragma unroll
    for (int r = 0; r < E; ++r) {
      float t = lhr[r] + llr[r];
      llr[r] -= t - lhr[r];
      lhr[r] = t;
      t = lhm[r] + llm[r];
      llm[r] -= t - lhm[r];
      lhm[r] = t;
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

template <int d, int N, bool PAR>
__global__ void __launch_bounds__((GShape<d, N, false>::T))
g_cos_kernel(const GArgs* __restrict__ Ag, const GAdj* __restrict__ Bg, int g_hi, int g_lo) {
  g_cos_body<d, N, PAR>(Ag, Bg, blockIdx.x, g_hi, g_lo);
}

// Batched (serving): item.gseg the first segment, item.n_lo the last.
template <int d, int N, bool PAR>
__global__ void __launch_bounds__((GShape<d, N, false>::T))
g_cos_batched_kernel(const GItem* __restrict__ items) {
  kptr<GItem> it = kconst(items) + blockIdx.x;
  g_cos_body<d, N, PAR>((const GArgs*)it->A, (const GAdj*)it->B, it->col, it->gseg, it->n_lo);
}

// Closed systems: the gradient from the steps' sums.  Block b of 64 steps of
// a column, last step first: the pulse parameters take dc/dpar of every stage
// times its drive-slot sum, the others the sums as they are.  The grouping is
// by step, not by segment, so the gradient does not depend on the checkpoint
// interval.
constexpr int GF_STEPS = 64;
__global__ void __launch_bounds__(256) g_fold_kernel(const GArgs* __restrict__ Ag,
                                                     const GAdj* __restrict__ Bg, int nblk,
                                                     double* __restrict__ out) {
  const GArgs& A = *Ag;
  const GAdj& B = *Bg;
  const int col = blockIdx.x / nblk, b = blockIdx.x - col * nblk;
  const int n0 = b * GF_STEPS, n1 = min(A.nsteps, n0 + GF_STEPS);
  const double* gs = B.gs + (size_t)col * A.nsteps * B.gw;
  const int nds = A.nds;
  for (int k = threadIdx.x; k < B.nacc; k += blockDim.x) {
    double v = 0.0;
    if (k < B.npulse) {
      int ds = -1;
      for (int q = 0; q < A.ndr; ++q)
        if (k >= A.dr_par0[q] && k < A.dr_par0[q] + A.dr_npar[q]) ds = A.dr_ds[q];
      for (int n = n1 - 1; n >= n0; --n) {
        const double* g = gs + (size_t)n * B.gw + ds;
        const double* dc = B.dctab + (size_t)3 * n * B.npulse + k;
        const double c0 = dc[0], c1 = dc[B.npulse], c2 = dc[2 * B.npulse];
        const double x3 = g[3 * nds], x2 = g[2 * nds], x1 = g[nds], x0 = g[0];
        v += c2 * x3;
        v += c1 * x2;
        v += c1 * x1;
        v += c0 * x0;
      }
    } else {
      const double* g = gs + 4 * nds + (k - B.npulse);
      for (int n = n1 - 1; n >= n0; --n) v += g[(size_t)n * B.gw];
    }
    out[(size_t)blockIdx.x * B.nacc + k] = v;
  }
}
// grad[k]: the blocks of a column from the last, columns in order.
__global__ void __launch_bounds__(64) g_fold_sum_kernel(const double* __restrict__ part, int S,
                                                        int nblk, int nacc,
                                                        double* __restrict__ grad) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= nacc) return;
  double v = 0.0;
  for (int c = 0; c < S; ++c) {
    double u = 0.0;
    for (int b = nblk - 1; b >= 0; --b) u += part[((size_t)c * nblk + b) * nacc + k];
    v += u;
  }
  grad[k] = v;
}

// One workgroup's reverse walk: open systems column col over every segment;
// closed systems segment gseg of column col, its stage inputs in buffer slot.
template <int d, int N, bool OPEN, bool PAR>
__device__ __forceinline__ void g_adj_body(const GArgs* __restrict__ Ag, const GAdj* __restrict__ Bg,
                                           int gseg, int col, int slot) {
  using Sh = GShape<d, N, OPEN>;
  using B_ = Nb<d, PAR>;
  constexpr int L = Sh::L, T = Sh::T, E = Sh::E, D = Sh::D, dd = d * d;
  constexpr int nb = B_::n, SR = B_::srow, MR = B_::mrow;   // gathered levels; operator row strides
  constexpr int NW = T / 64;
  constexpr int WS = OPEN ? GA_MAXDS : GA_NV;   // per-wave sums of one stage
  extern __shared__ __align__(16) c32 lds[];
  kptr<GArgs> A = kconst(Ag);
  kptr<GAdj> B = kconst(Bg);
  const int ntab = A->ntab, ntabg = A->ntabg;
  const int nacc = B->nacc, npulse = B->npulse;
  // LDS: two column buffers (stage inputs while recomputing, kb while
  // reversing), for closed systems two more (y while reversing), two stage
  // tables (gradient width), FP64 accumulators, and per-wave partial sums of
  // a stage (two stage parities)
  c32* yb0 = lds + 2 * L;
  c32* tb0 = lds + (OPEN ? 2 : 4) * L;
  double* acc = (double*)(tb0 + 2 * ntabg);
  float* wsum = (float*)(acc + ((nacc + 1) & ~1));
  const c32* gtab = (const c32*)A->gtab;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float h = A->h;
  const int nsteps = A->nsteps, ce = B->ce, nck = B->nck;
  // Open systems: one workgroup per column walks every segment (recompute,
  // then reverse).  Closed systems: one workgroup per column and segment, the
  // costate at the segment's end from the sweep before (g_cos_body).
  const int g_hi = OPEN ? nck - 1 : gseg;
  const int g_lo = OPEN ? 0 : g_hi;
  const int nds = uni(A->nds), ncp = uni(A->ncp), ndr = uni(A->ndr);
  const int nv = OPEN ? 0 : 3 * N + ncp;   // closed: device-parameter and coupling sums
  if (OPEN)
    for (int t = tid; t < nacc; t += T) acc[t] = 0.0;
  uint32_t pk[E];
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const int e = tid + r * T;
    const int Ai = OPEN ? e / D : e, Bi = OPEN ? e - Ai * D : 0;
    uint32_t p = 0;
#pragma unroll
    for (int m = 0; m < N; ++m) {
      p |= (uint32_t)((Ai / Sh::st(m)) % d) << (3 * m);
      if (OPEN) p |= (uint32_t)((Bi / Sh::st(m)) % d) << (3 * (N + m));
    }
    pk[r] = p;
  }
  // the costate lives in registers only during the reverse walks; between
  // them (while a segment is recomputed) it waits in device memory
  float4* lsave = B->lam + (OPEN ? (size_t)col : (size_t)col * nck + gseg) * L;
  int prev_n = -1, prev_s = 0;   // the stage whose sums wait in wsum
  int par = 0;                   // parity of the wsum buffer being filled
  double vstep = 0.0;            // closed: this thread's sum over the step's stages
  // fold the previous stage's per-wave sums in a fixed order.  Open systems:
  // the drive slots into the pulse parameters (one thread per drive, times
  // dc/dpar of that stage).  Closed systems: into the step's row of gs, the
  // drive slots of each stage, then the device-parameter and coupling sums
  // over the four stages (at most GA_NV <= 64 sums: one thread each).
  auto fold_prev = [&]() {
    if constexpr (OPEN) {
      for (int t = tid; t < ndr; t += T) {
        const int ds = A->dr_ds[t];
        double G = 0.0;
        for (int w = 0; w < NW; ++w) G += (double)wsum[((par ^ 1) * NW + w) * WS + ds];
        const double* dct = B->dctab + (size_t)stage_c(prev_n, prev_s) * npulse;
        for (int p = A->dr_par0[t]; p < A->dr_par0[t] + A->dr_npar[t]; ++p) acc[p] += dct[p] * G;
      }
    } else if (tid < nds + nv) {
      const int k = tid < nds ? tid : GA_MAXDS + tid - nds;
      double G = 0.0;
      for (int w = 0; w < NW; ++w) G += (double)wsum[((par ^ 1) * NW + w) * WS + k];
      double* row = B->gs + ((size_t)col * nsteps + prev_n) * B->gw;
      if (tid < nds) {
        row[prev_s * nds + tid] = G;
      } else {
        vstep = prev_s == 3 ? G : vstep + G;
        if (prev_s == 0) row[3 * nds + tid] = vstep;
      }
    }
  };
  __syncthreads();
#pragma unroll 1
  for (int g = g_hi; g >= g_lo; --g) {
    const int n0 = g * ce, n1 = min(nsteps, n0 + ce);
    // stage inputs of the segment: one buffer per column (open systems) or
    // per workgroup in flight (closed systems)
    c32* segc = (c32*)B->seg + (size_t)(OPEN ? col : slot) * ce * 4 * L;
    // ---- recompute the segment from its checkpoint, storing the stage inputs
    {
      float hr[E], hm[E], lr[E], lm[E], ar[E], am_[E];
      const float4* ck = B->ck + ((size_t)col * nck + g) * L;
#pragma unroll
      for (int r = 0; r < E; ++r) {
        const int e = tid + r * T;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (e < L) v = ck[e];
        hr[r] = v.x;
        hm[r] = v.y;
        lr[r] = v.z;
        lm[r] = v.w;
        ar[r] = am_[r] = 0.f;
        if (e < L) {
          c32 u;
          u.x = v.x;
          u.y = v.y;
          lds[e] = u;
        }
      }
      {
        const c32* g0 = gtab + (size_t)stage_c(n0, 0) * ntabg;
        for (int t = tid; t < ntab; t += T) tb0[t] = g0[t];
      }
      __syncthreads();
      int cur = 0;
#pragma unroll 1
      for (int n = n0; n < n1; ++n) {
#pragma unroll 1
        for (int s = 0; s < 4; ++s) {
          const float w = (s == 0 || s == 3) ? 1.f : 2.f;
          const float ch = (s == 2) ? h : 0.5f * h;
          const c32* yc = lds + cur * L;
          const c32* tc = tb0 + cur * ntabg;
          c32* yn = lds + (cur ^ 1) * L;
          c32* ys = segc + ((size_t)(n - n0) * 4 + s) * L;
          const int n2 = s < 3 ? n : n + 1, s2 = s < 3 ? s + 1 : 0;
          const bool more = n2 < n1;
          const c32* gnext = gtab + (size_t)stage_c(n2, s2) * ntabg;
          c32 pre[GA_PRE];
#pragma unroll
          for (int k = 0; k < GA_PRE; ++k) {
            const int t = tid + k * T;
            if (more && t < ntab) pre[k] = gnext[t];
          }
#pragma unroll
          for (int r = 0; r < E; ++r) {
            int e = tid + r * T;
            uint32_t p = pk[r];
            asm volatile("" : "+v"(e), "+v"(p));
            if (e < L) {
              float gr = 0.f, gi = 0.f;
#pragma unroll
              for (int m = 0; m < N; ++m) {
                const int a = ket_digit(p, m);
                if (OPEN) {
                  const int b = bra_digit(p, m, N);
                  gi -= A->delta[m][a] - A->delta[m][b];
                  gr -= 0.5f * A->g1[m] * (float)(a + b) + A->gp[m] * (float)((a - b) * (a - b));
                } else {
                  gi -= A->delta[m][a];
                }
              }
              const c32 ye = yc[e];
              ys[e] = ye;
              float kr, ki;
              g_apply<d, N, OPEN, PAR>(A, yc, tc, e, p, gr, gi, ye.x, ye.y, kr, ki);
              if (s == 0) {
                ar[r] = kr;
                am_[r] = ki;
              } else {
                ar[r] = fmaf(w, kr, ar[r]);
                am_[r] = fmaf(w, ki, am_[r]);
              }
              c32 v;
              if (s < 3) {
                v.x = fmaf(ch, kr, hr[r]);
                v.y = fmaf(ch, ki, hm[r]);
              } else {
                const float h6 = h * (1.0f / 6.0f);
                comp_add(hr[r], lr[r], h6 * ar[r]);
                comp_add(hm[r], lm[r], h6 * am_[r]);
                v.x = hr[r];
                v.y = hm[r];
              }
              yn[e] = v;
            }
            __builtin_amdgcn_sched_barrier(0);
          }
          if (more) {
            c32* tn = tb0 + (cur ^ 1) * ntabg;
#pragma unroll
            for (int k = 0; k < GA_PRE; ++k) {
              const int t = tid + k * T;
              if (t < ntab) tn[t] = pre[k];
            }
            for (int t = tid + GA_PRE * T; t < ntab; t += T) tn[t] = gnext[t];
          }
          __syncthreads();
          cur ^= 1;
        }
      }
    }
    // ---- reverse walk of the segment
    float lhr[E], lhm[E], llr[E], llm[E];   // costate (hi, lo)
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const int e = tid + r * T;
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
      if (e < L) {
        if (OPEN && g == nck - 1) {
          const c32 c = ((const c32*)B->cot)[(size_t)col * L + e];
          v = make_float4(c.x, c.y, 0.f, 0.f);
        } else {
          v = lsave[e];
        }
      }
      lhr[r] = v.x;
      lhm[r] = v.y;
      llr[r] = v.z;
      llm[r] = v.w;
    }
    int cur = 0;
    // closed systems: the next stage's y and the first GP table entries per
    // thread are loaded into registers while the current stage runs
    constexpr int GP = OPEN ? 1 : 8;
    c32 pre_t[GP], pre_y[OPEN ? 1 : E];
    if constexpr (!OPEN) {   // the walk's first stage: (n1 - 1, 3)
      const c32* ysn = segc + ((size_t)(n1 - 1 - n0) * 4 + 3) * L;
      const c32* grn = gtab + (size_t)stage_c(n1 - 1, 3) * ntabg;
#pragma unroll
      for (int r = 0; r < E; ++r) {
        const int e = tid + r * T;
        if (e < L) pre_y[r] = ysn[e];
      }
#pragma unroll
      for (int k = 0; k < GP; ++k) {
        const int t = tid + k * T;
        if (t < ntabg) pre_t[k] = grn[t];
      }
    }
#pragma unroll 1
    for (int n = n1 - 1; n >= n0; --n) {
      // yb_{s+1}; the step's increments sum_s yb_s gather in the costate's lo
      // word (kb_s reads only hi) and are folded into hi at the step's end
      float ybr[E], ybm[E];
#pragma unroll
      for (int r = 0; r < E; ++r) ybr[r] = ybm[r] = 0.f;
#pragma unroll 1
      for (int s = 3; s >= 0; --s) {
        const float cs = (s == 0 || s == 3) ? h * (1.0f / 6.0f) : h * (1.0f / 3.0f);
        const float cy = (s == 3) ? 0.f : (s == 2 ? h : 0.5f * h);
        const int row = stage_c(n, s);
        c32* kbw = lds + cur * L;
        c32* ybw = yb0 + cur * L;   // closed systems
        c32* tw = tb0 + cur * ntabg;
        const c32* ys = segc + ((size_t)(n - n0) * 4 + s) * L;
        const c32* gr_ = gtab + (size_t)row * ntabg;
        // kb_s (own elements), closed systems y_s too, and the stage table
        // into this stage's buffers
#pragma unroll
        for (int r = 0; r < E; ++r) {
          const int e = tid + r * T;
          if (e < L) {
            c32 v;
            v.x = fmaf(cs, lhr[r], cy * ybr[r]);
            v.y = fmaf(cs, lhm[r], cy * ybm[r]);
            kbw[e] = v;
            if (!OPEN) ybw[e] = pre_y[OPEN ? 0 : r];
          }
        }
        if (!OPEN) {
#pragma unroll
          for (int k = 0; k < GP; ++k) {
            const int t = tid + k * T;
            if (t < ntabg) tw[t] = pre_t[k];
          }
          for (int t = tid + GP * T; t < ntabg; t += T) tw[t] = gr_[t];
        } else {
          for (int t = tid; t < ntabg; t += T) tw[t] = gr_[t];
        }
        __syncthreads();
        if constexpr (!OPEN) {
          // the next stage of the walk: (n, s - 1), else (n - 1, 3) within the segment
          const int nn = s > 0 ? n : n - 1, sn = s > 0 ? s - 1 : 3;
          if (nn >= n0) {
            const c32* ysn = segc + ((size_t)(nn - n0) * 4 + sn) * L;
            const c32* grn = gtab + (size_t)stage_c(nn, sn) * ntabg;
#pragma unroll
            for (int r = 0; r < E; ++r) {
              const int e = tid + r * T;
              if (e < L) pre_y[r] = ysn[e];
            }
#pragma unroll
            for (int k = 0; k < GP; ++k) {
              const int t = tid + k * T;
              if (t < ntabg) pre_t[k] = grn[t];
            }
          }
        }
        // the previous stage's sums are complete
        if (prev_n >= 0) fold_prev();
#pragma unroll
        for (int r = 0; r < E; ++r) {
          int e = tid + r * T;
          uint32_t p = pk[r];
          asm volatile("" : "+v"(e), "+v"(p));
          if (e < L) {
            float gr = 0.f, gi = 0.f;
#pragma unroll
            for (int m = 0; m < N; ++m) {
              const int a = ket_digit(p, m);
              if (OPEN) {
                const int b = bra_digit(p, m, N);
                gi -= A->delta[m][a] - A->delta[m][b];
                gr -= 0.5f * A->g1[m] * (float)(a + b) + A->gp[m] * (float)((a - b) * (a - b));
              } else {
                gi -= A->delta[m][a];
              }
            }
            const c32 kbe = kbw[e];
            float yr_, yi_;
            g_apply_adj<d, N, OPEN, PAR>(A, kbw, tw, e, p, gr, gi, kbe.x, kbe.y, yr_, yi_);
            ybr[r] = yr_;
            ybm[r] = yi_;
            llr[r] += yr_;
            llm[r] += yi_;
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (OPEN) {
          // drive slots: 2 Im <O kb - kb O, y>, one sum per wave
#pragma unroll 1
          for (int k = 0; k < nds; ++k) {
            const int m = uni(A->ds_mode[k]);
            const c32* rows = tw + A->off_s + uni(A->ds_sl[k]) * d * SR;
            const int ks = uni(A->kst[m]), bs = uni(A->bst[m]);
            float v = 0.f;
#pragma unroll
            for (int r = 0; r < E; ++r) {
              const int e = tid + r * T;
              if (e < L) {
                const c32 z =
                    comm1<d, N, PAR>(kbw, rows, e, ket_digit(pk[r], m), bra_digit(pk[r], m, N), ks, bs);
                v += 2.f * im_conj(z, ys[e]);
              }
            }
            v = g_wave_sum(v);
            if (lane == 0) wsum[(par * NW + wave) * WS + k] = v;
          }
          // couplings: 2 Im <P kb - kb P, y>, added to the FP64 sums per wave
#pragma unroll 1
          for (int c = 0; c < ncp; ++c) {
            const int i = uni(A->cp_i[c]), j = uni(A->cp_j[c]);
            const c32* Ri = tw + A->off_s + uni(A->cp_si[c]) * d * SR;
            const c32* Rj = tw + A->off_s + uni(A->cp_sj[c]) * d * SR;
            const int ksi = uni(A->kst[i]), ksj = uni(A->kst[j]);
            const int bsi = uni(A->bst[i]), bsj = uni(A->bst[j]);
            float v = 0.f;
#pragma unroll
            for (int r = 0; r < E; ++r) {
              const int e = tid + r * T;
              if (e < L) {
                const uint32_t p = pk[r];
                const c32 z = comm2<d, N, PAR>(kbw, Ri, Rj, e, ket_digit(p, i), ket_digit(p, j),
                                          bra_digit(p, i, N), bra_digit(p, j, N), ksi, ksj, bsi,
                                          bsj);
                const c32 y = ys[e];
                v += 2.f * (z.x * y.y - z.y * y.x);
              }
            }
            v = g_wave_sum(v);
            if (lane == 0) atomicAdd(&acc[npulse + c], (double)v);
          }
          // rates: 2 Re <D[a_m]^dag kb, y> and 2 Re <-(a - b)^2 kb, y>
#pragma unroll 1
          for (int m = 0; m < N; ++m) {
            const int sm = (D + 1) * uni(A->bst[m]);
            const c32* Ju = tw + A->off_u + m * dd;
            float v1 = 0.f, v2 = 0.f;
#pragma unroll
            for (int r = 0; r < E; ++r) {
              const int e = tid + r * T;
              if (e < L) {
                const int a = ket_digit(pk[r], m), b = bra_digit(pk[r], m, N);
                const c32 kbe = kbw[e];
                float zr = -0.5f * (float)(a + b) * kbe.x, zi = -0.5f * (float)(a + b) * kbe.y;
                if (a > 0 && b > 0) cmac_conj(zr, zi, Ju[(a - 1) * d + (b - 1)], kbw[e - sm]);
                const c32 y = ys[e];
                v1 += 2.f * (zr * y.x + zi * y.y);
                v2 -= 2.f * (float)((a - b) * (a - b)) * (kbe.x * y.x + kbe.y * y.y);
              }
            }
            v1 = g_wave_sum(v1);
            v2 = g_wave_sum(v2);
            if (lane == 0) {
              atomicAdd(&acc[npulse + ncp + 2 * m], (double)v1);
              atomicAdd(&acc[npulse + ncp + 2 * m + 1], (double)v2);
            }
          }
        } else {
          // Device parameters of mode m and couplings.  <kb, dH y> with dH a
          // one-mode operator Q on m: 2 Im <Q kb, y> from kb gathered along m.
          // A two-mode term P_i (x) P_j factors as <(P_i (x) 1) kb, (1 (x) P_j) y>,
          // so each coupling end needs kb gathered along its own mode and y
          // along the partner's; the device derivative on the own side is
          // g (dP_own (x) P_partner), summed over the ends sharing dP_own.
#pragma unroll 1
          for (int mv = 0; mv < N; ++mv) {
            const int m = uni(mv);
            const int ks = uni(A->kst[m]);
            const c32* Dm = tw + uni(A->off_m) + m * 3 * d * MR;
            // kb along m: kept in registers for the whole mode when small,
            // else gathered again at each use (keeps the E = 4 shapes out of
            // scratch)
            constexpr bool KC = E * nb <= 12;
            c32 kv[KC ? E : 1][nb];
            c32 C[E];
            float v0 = 0.f, v1 = 0.f, v2 = 0.f;
#pragma unroll
            for (int r = 0; r < E; ++r) {
              const int e = tid + r * T;
              C[r].x = C[r].y = 0.f;
              if (e < L) {
                const int am = ket_digit(pk[r], m);
                c32 kt[nb];
#pragma unroll
                for (int x = 0; x < nb; ++x) kt[x] = kbw[e + B_::first(am, ks) + B_::step(x, am, ks)];
                if constexpr (KC) {
#pragma unroll
                  for (int x = 0; x < nb; ++x) kv[r][x] = kt[x];
                }
                c32 w[nb];
                conj_scale<nb>(kt, ybw[e], w);
                const c32* Dr = Dm + am * MR;
                v0 += 2.f * im_rowdot<nb>(Dr, w);
                v1 += 2.f * im_rowdot<nb>(Dr + d * MR, w);
                v2 += 2.f * im_rowdot<nb>(Dr + 2 * d * MR, w);
                if constexpr (PAR) {   // the diagonal (real), behind the row's entries
                  const float dg = 2.f * im_conj(kbw[e], ybw[e]);
                  v0 = fmaf(dg, Dr[nb].x, v0);
                  v1 = fmaf(dg, Dr[d * MR + nb].x, v1);
                  v2 = fmaf(dg, Dr[2 * d * MR + nb].x, v2);
                }
              }
              __builtin_amdgcn_sched_barrier(0);
            }
            // kb along m of element r (registers or LDS)
            auto kb_of = [&](int r, int e, int am, c32(&kt)[nb]) {
              if constexpr (KC) {
#pragma unroll
                for (int x = 0; x < nb; ++x) kt[x] = kv[KC ? r : 0][x];
              } else {
#pragma unroll
                for (int x = 0; x < nb; ++x) kt[x] = kbw[e + B_::first(am, ks) + B_::step(x, am, ks)];
              }
            };
            // drive slots on this mode: 2 Im <O kb, y>, one sum per wave (the
            // large shapes take them in a loop of their own, below)
#pragma unroll 1
            for (int k = 0; k < (KC ? nds : 0); ++k) {
              if (uni(A->ds_mode[k]) != m) continue;
              const c32* rows = tw + A->off_s + uni(A->ds_sl[k]) * d * SR;
              float v = 0.f;
#pragma unroll
              for (int r = 0; r < E; ++r) {
                const int e = tid + r * T;
                if (e < L) {
                  const int am = ket_digit(pk[r], m);
                  c32 kt[nb];
                  kb_of(r, e, am, kt);
                  v += 2.f * im_conj(rowdot<nb>(rows + am * SR, kt), ybw[e]);
                }
              }
              v = g_wave_sum(v);
              if (lane == 0) wsum[(par * NW + wave) * WS + k] = v;
            }
            const int k0 = uni(A->me_beg[m]), k1 = uni(A->me_beg[m + 1]);
#pragma unroll 1
            for (int kq = k0; kq < k1; ++kq) {
              const int pkd = uni(A->me[kq]);
              const int c = pkd & 31, own = (pkd >> 5) & 31, psl = (pkd >> 10) & 31;
              const int pm = (pkd >> 15) & 31;
              const bool first = (pkd >> 20) & 1, last = (pkd >> 21) & 1;
              const float gc = unif(A->cp_g[c]);
              const int ps = uni(A->kst[pm]);
              const c32* Ro = tw + A->off_s + own * d * SR;
              const c32* Rp = tw + A->off_s + psl * d * SR;
              const c32* dR = tw + A->off_d + own * 3 * d * SR;
              float vc = 0.f;
#pragma unroll
              for (int r = 0; r < E; ++r) {
                const int e = tid + r * T;
                if (e < L) {
                  const int am = ket_digit(pk[r], m), ap = ket_digit(pk[r], pm);
                  c32 yv[nb];
#pragma unroll
                  for (int z = 0; z < nb; ++z) yv[z] = ybw[e + B_::first(ap, ps) + B_::step(z, ap, ps)];
                  const c32 cp = rowdot<nb>(Rp + ap * SR, yv);
                  C[r].x = fmaf(gc, cp.x, C[r].x);
                  C[r].y = fmaf(gc, cp.y, C[r].y);
                  if (first || last) {
                    c32 kt[nb];
                    kb_of(r, e, am, kt);
                    if (first) vc += 2.f * im_conj(rowdot<nb>(Ro + am * SR, kt), cp);
                    if (last) {
                      c32 w[nb];
                      conj_scale<nb>(kt, C[r], w);
                      const c32* dr_ = dR + am * SR;
                      v0 += 2.f * im_rowdot<nb>(dr_, w);
                      v1 += 2.f * im_rowdot<nb>(dr_ + d * SR, w);
                      v2 += 2.f * im_rowdot<nb>(dr_ + 2 * d * SR, w);
                      C[r].x = C[r].y = 0.f;
                    }
                  }
                }
              }
              if (first) {
                vc = g_wave_sum(vc);
                if (lane == 0) wsum[(par * NW + wave) * WS + GA_MAXDS + 3 * N + c] = vc;
              }
            }
            v0 = g_wave_sum(v0);
            v1 = g_wave_sum(v1);
            v2 = g_wave_sum(v2);
            if (lane == 0) {
              float* wv = wsum + (par * NW + wave) * WS + GA_MAXDS + 3 * m;
              wv[0] = v0;
              wv[1] = v1;
              wv[2] = v2;
            }
          }
          if constexpr (E * nb > 12) {
#pragma unroll 1
            for (int k = 0; k < nds; ++k) {
              const int m = uni(A->ds_mode[k]);
              const int ks = uni(A->kst[m]);
              const c32* rows = tw + A->off_s + uni(A->ds_sl[k]) * d * SR;
              float v = 0.f;
#pragma unroll
              for (int r = 0; r < E; ++r) {
                const int e = tid + r * T;
                if (e < L) {
                  const int am = ket_digit(pk[r], m);
                  c32 kt[nb];
#pragma unroll
                  for (int x = 0; x < nb; ++x) kt[x] = kbw[e + B_::first(am, ks) + B_::step(x, am, ks)];
                  v += 2.f * im_conj(rowdot<nb>(rows + am * SR, kt), ybw[e]);
                }
              }
              v = g_wave_sum(v);
              if (lane == 0) wsum[(par * NW + wave) * WS + k] = v;
            }
          }
        }
        prev_n = n;
        prev_s = s;
        par ^= 1;
        cur ^= 1;
      }
      // lambda_n = lambda_{n+1} + sum_s yb_s: fold lo (holding the old lo and
      // the increments, small next to hi) into hi exactly (fast two-sum)
#pragma unroll
      for (int r = 0; r < E; ++r) {
        float t = lhr[r] + llr[r];
        llr[r] -= t - lhr[r];
        lhr[r] = t;
        t = lhm[r] + llm[r];
        llm[r] -= t - lhm[r];
        lhm[r] = t;
      }
    }
    if (OPEN && g > 0) {
#pragma unroll
      for (int r = 0; r < E; ++r) {
        const int e = tid + r * T;
        if (e < L) lsave[e] = make_float4(lhr[r], lhm[r], llr[r], llm[r]);
      }
    }
    __syncthreads();
  }
  // the last stage's sums
  if (prev_n >= 0) fold_prev();
  if (!OPEN) return;
  __syncthreads();
  for (int t = tid; t < nacc; t += T) B->part[(size_t)col * nacc + t] = acc[t];
}

template <int d, int N, bool OPEN, bool PAR>
__global__ void __launch_bounds__((GShape<d, N, OPEN>::T))
g_adj_kernel(const GArgs* __restrict__ Ag, const GAdj* __restrict__ Bg, int gseg) {
  // closed: S workgroups per segment, from segment gseg down
  const int S = OPEN ? (int)gridDim.x : Ag->S;
  const int k = blockIdx.x / S, col = blockIdx.x - k * S;
  g_adj_body<d, N, OPEN, PAR>(Ag, Bg, gseg - k, col, blockIdx.x);
}

// Batched (serving, closed systems): item.gseg is the segment, item.n_lo the
// stage-input buffer.
template <int d, int N, bool PAR>
__global__ void __launch_bounds__((GShape<d, N, false>::T))
g_adj_batched_kernel(const GItem* __restrict__ items) {
  kptr<GItem> it = kconst(items) + blockIdx.x;
  g_adj_body<d, N, false, PAR>((const GArgs*)it->A, (const GAdj*)it->B, it->gseg, it->col, it->n_lo);
}

// Unit-rate relaxation band of every mode at every half-step q (t = q h/2):
// sqrt((a+1)(b+1)) exp(i (f_a - f_{a+1} - f_b + f_{b+1}) t) for a, b < d - 1,
// zero otherwise; FP64 angle reduced modulo 2 pi, stored FP32.
struct JtabStatic {
  int d, N, nq;
  double h;
  double f[GA_MAXM][8];
};

__global__ void jtab_kernel(JtabStatic js, float2* __restrict__ out) {
  const int q = blockIdx.x;
  const int dd = js.d * js.d;
  const double t = q * (0.5 * js.h);
  const double twopi = 6.283185307179586476925286766559;
  for (int u = threadIdx.x; u < js.N * dd; u += blockDim.x) {
    const int m = u / dd, ab = u - m * dd, a = ab / js.d, b = ab - a * js.d;
    float2 v = make_float2(0.f, 0.f);
    if (a < js.d - 1 && b < js.d - 1) {
      double x = (js.f[m][a] - js.f[m][a + 1] - js.f[m][b] + js.f[m][b + 1]) * t;
      x -= twopi * rint(x / twopi);
      double sn, cs;
      sincos(x, &sn, &cs);
      const double r = sqrt((double)((a + 1) * (b + 1)));
      v = make_float2((float)(r * cs), (float)(r * sn));
    }
    out[(size_t)q * js.N * dd + u] = v;
  }
}

__global__ void store_args_kernel(GArgs a, GArgs* out) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *out = a;
}

template <int d, int N, bool OPEN>
size_t g_lds_bytes(int ntab) {
  constexpr size_t L = GShape<d, N, OPEN>::L;
  return sizeof(c32) * (3 * L + ((3 * L) & 1) + 2 * (size_t)ntab);
}

template <typename K>
hipError_t g_lds(K* kernel, size_t sh) {
  return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
}

// Steps [n_lo, n_hi) with the state from st_in / to st_out (nullable; see the
// kernel); dadj != nullptr also writes the checkpoints.
template <int d, int N, bool OPEN, bool PAR, bool CK>
hipError_t g_launch1(const GArgs* dargs, const GAdj* dadj, int S, int ntab, int n_lo, int n_hi,
                     const float4* st_in, float4* st_out, hipStream_t s) {
  using Sh = GShape<d, N, OPEN>;
  const size_t sh = g_lds_bytes<d, N, OPEN>(ntab);
  (void)g_lds(g_rk4_kernel<d, N, OPEN, PAR, CK>, sh);
  hipLaunchKernelGGL((g_rk4_kernel<d, N, OPEN, PAR, CK>), dim3(S), dim3(Sh::T), sh, s, dargs, dadj,
                     n_lo, n_hi, st_in, st_out);
  return hipGetLastError();
}

// Form of a launch: 0 general, 1 parity, 2 real.
int g_form(const GArgs& A) { return A.real ? 2 : (A.par ? 1 : 0); }

template <int d, int N, bool OPEN>
hipError_t g_launch(int form, const GArgs* dargs, const GAdj* dadj, int S, int ntab, int n_lo,
                    int n_hi, const float4* st_in, float4* st_out, hipStream_t s) {
  const bool par = form != 0;
  if (OPEN && form == 2) return l_real_forward(d, N, dargs, dadj, S, n_hi, s);
  if (!OPEN && form == 2)
    return g_real_forward(d, N, dadj != nullptr, nullptr, dargs, dadj, S, n_lo, n_hi, st_in, st_out, s);
  if (dadj != nullptr)
    return par ? g_launch1<d, N, OPEN, true, true>(dargs, dadj, S, ntab, n_lo, n_hi, st_in, st_out, s)
               : g_launch1<d, N, OPEN, false, true>(dargs, dadj, S, ntab, n_lo, n_hi, st_in, st_out, s);
  return par ? g_launch1<d, N, OPEN, true, false>(dargs, dadj, S, ntab, n_lo, n_hi, st_in, st_out, s)
             : g_launch1<d, N, OPEN, false, false>(dargs, dadj, S, ntab, n_lo, n_hi, st_in, st_out, s);
}

hipError_t g_dispatch(int d, int N, bool open, int form, const GArgs* dargs, const GAdj* dadj, int S, int ntab,
                      int n_lo, int n_hi, const float4* st_in, float4* st_out, hipStream_t s) {
#define GA_CASE_O(dd_, nn_)          \
  if (open && d == dd_ && N == nn_) \
    return g_launch<dd_, nn_, true>(form, dargs, dadj, S, ntab, n_lo, n_hi, st_in, st_out, s);
#define GA_CASE_C(dd_, nn_)           \
  if (!open && d == dd_ && N == nn_) \
    return g_launch<dd_, nn_, false>(form, dargs, dadj, S, ntab, n_lo, n_hi, st_in, st_out, s);
  GA_OPEN_SHAPES(GA_CASE_O)
  GA_CLOSED_SHAPES(GA_CASE_C)
#undef GA_CASE_O
#undef GA_CASE_C
  return hipErrorInvalidValue;
}

bool g_supported(int d, int N, bool open) {
#define GA_HAS_O(dd_, nn_) if (open && d == dd_ && N == nn_) return true;
#define GA_HAS_C(dd_, nn_) if (!open && d == dd_ && N == nn_) return true;
  GA_OPEN_SHAPES(GA_HAS_O)
  GA_CLOSED_SHAPES(GA_HAS_C)
#undef GA_HAS_O
#undef GA_HAS_C
  return false;
}

__global__ void store_adj_kernel(GAdj a, GAdj* out) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *out = a;
}

template <int d, int N, bool OPEN>
size_t g_adj_lds_bytes(int ntabg, int nacc) {
  using Sh = GShape<d, N, OPEN>;
  return sizeof(c32) * ((OPEN ? 2 : 4) * (size_t)Sh::L + 2 * (size_t)ntabg) +
         sizeof(double) * (size_t)((nacc + 1) & ~1) +
         sizeof(float) * 2 * (Sh::T / 64) * (OPEN ? GA_MAXDS : GA_NV);
}

// Open systems: one launch (gseg, nseg unused).  Closed systems: nseg segments
// from gseg down, S workgroups each, after the costate sweep over them.
template <int d, int N, bool OPEN>
hipError_t g_adj_launch(int form, const GArgs* dargs, const GAdj* dadj, int S, int ntabg, int nacc,
                        int gseg, int nseg, hipStream_t s) {
  using Sh = GShape<d, N, OPEN>;
  if (OPEN && form == 2) return l_real_adjoint(d, N, dargs, dadj, S, s);
  if (!OPEN && form == 2) return g_real_segments(d, N, nullptr, dargs, dadj, nseg * S, gseg, s);
  const size_t sh = g_adj_lds_bytes<d, N, OPEN>(ntabg, nacc);
  if (sh > 163840) return hipErrorInvalidValue;
  auto run = [&](auto* kernel) {
    (void)g_lds(kernel, sh);
    hipLaunchKernelGGL(kernel, dim3(OPEN ? S : nseg * S), dim3(Sh::T), sh, s, dargs, dadj, gseg);
  };
  if (form != 0)
    run(g_adj_kernel<d, N, OPEN, true>);
  else
    run(g_adj_kernel<d, N, OPEN, false>);
  return hipGetLastError();
}

size_t g_adj_lds(int d, int N, bool open, int ntabg, int nacc) {
#define GA_ADJ_LDS_O(dd_, nn_) \
  if (open && d == dd_ && N == nn_) return g_adj_lds_bytes<dd_, nn_, true>(ntabg, nacc);
#define GA_ADJ_LDS_C(dd_, nn_) \
  if (!open && d == dd_ && N == nn_) return g_adj_lds_bytes<dd_, nn_, false>(ntabg, nacc);
  GA_OPEN_SHAPES(GA_ADJ_LDS_O)
  GA_CLOSED_SHAPES(GA_ADJ_LDS_C)
#undef GA_ADJ_LDS_O
#undef GA_ADJ_LDS_C
  return ~(size_t)0;
}

hipError_t g_adj_dispatch(int d, int N, bool open, int form, const GArgs* dargs, const GAdj* dadj, int S,
                          int ntabg, int nacc, int gseg, int nseg, hipStream_t s) {
#define GA_ADJ_CASE_O(dd_, nn_) \
  if (open && d == dd_ && N == nn_)  \
    return g_adj_launch<dd_, nn_, true>(form, dargs, dadj, S, ntabg, nacc, gseg, nseg, s);
#define GA_ADJ_CASE_C(dd_, nn_) \
  if (!open && d == dd_ && N == nn_)   \
    return g_adj_launch<dd_, nn_, false>(form, dargs, dadj, S, ntabg, nacc, gseg, nseg, s);
  GA_OPEN_SHAPES(GA_ADJ_CASE_O)
  GA_CLOSED_SHAPES(GA_ADJ_CASE_C)
#undef GA_ADJ_CASE_O
#undef GA_ADJ_CASE_C
  return hipErrorInvalidValue;
}

template <int d, int N>
size_t g_cos_lds_bytes(int ntab) {
  return sizeof(c32) * (2 * (size_t)GShape<d, N, false>::L + 2 * (size_t)ntab);
}

// Costate sweep of a closed system over the segments g_hi down to g_lo.
template <int d, int N>
hipError_t g_cos_launch(int form, const GArgs* dargs, const GAdj* dadj, int S, int ntab, int g_hi,
                        int g_lo, hipStream_t s) {
  if (form == 2) return g_real_sweep(d, N, nullptr, dargs, dadj, S, g_hi, g_lo, s);
  const size_t sh = g_cos_lds_bytes<d, N>(ntab);
  auto run = [&](auto* kernel) {
    (void)g_lds(kernel, sh);
    hipLaunchKernelGGL(kernel, dim3(S), dim3(GShape<d, N, false>::T), sh, s, dargs, dadj, g_hi, g_lo);
  };
  if (form == 1)
    run(g_cos_kernel<d, N, true>);
  else
    run(g_cos_kernel<d, N, false>);
  return hipGetLastError();
}

hipError_t g_cos_dispatch(int d, int N, int form, const GArgs* dargs, const GAdj* dadj, int S,
                          int ntab, int g_hi, int g_lo, hipStream_t s) {
#define GA_COS_CASE(dd_, nn_) \
  if (d == dd_ && N == nn_) return g_cos_launch<dd_, nn_>(form, dargs, dadj, S, ntab, g_hi, g_lo, s);
  GA_CLOSED_SHAPES(GA_COS_CASE)
#undef GA_COS_CASE
  return hipErrorInvalidValue;
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

// The real form's coefficients carry h / (6 h6), h6 the FP32 weight of the RK4
// sum: the rounding of h6 is the same at every step and would stretch every
// rotation angle (the same errors: 1.3e-7 -> 1.0e-7 and 2e-8 to 6e-8).
static double real_kappa(const scp_system* sys) {
  const float h = (float)sys->h, h6 = h * (1.0f / 6.0f);
  return sys->h / (6.0 * (double)h6);
}

// Fill the static description from the system and (open systems) the rates.
static scp_status g_args(const scp_system* sys, bool open, const double* gamma1,
                         const double* gammaphi, GArgs& A) {
  std::memset(&A, 0, sizeof(A));
  const Plan& P = sys->plan;
  const int N = sys->n_modes, d = sys->d, dd = d * d;
  if (N > GA_MAXM || (open && 2 * N > GA_MAXM) || d > 7)
    return fail(SCP_EINVAL, "gather engine: too many modes");
  const int D = (int)sys->D;
  A.block_q = P.block_q;
  A.ngroups = std::max(1, P.ngroups);
  A.nsteps = sys->n_steps;
  A.h = (float)sys->h;
  for (int m = 0; m < N; ++m) {
    int st = 1;
    for (int q = m + 1; q < N; ++q) st *= d;
    A.kst[m] = open ? st * D : st;
    A.bst[m] = st;
    const double g1 = (open && gamma1) ? gamma1[m] : 0.0;
    const double gp = (open && gammaphi) ? gammaphi[m] : 0.0;
    if (!(g1 >= 0.0) || !(gp >= 0.0) || !std::isfinite(g1) || !std::isfinite(gp))
      return fail(SCP_EINVAL, "decay rates must be finite and non-negative");
    A.g1[m] = (float)g1;
    A.gp[m] = (float)gp;
    A.has_jump |= g1 > 0.0;
    for (int a = 0; a < d; ++a) A.delta[m][a] = P.delta[m][a];
  }
  // driven modes: the distinct (slot, coefficient group) pairs of each mode
  for (int k = 0; k < P.ndrives; ++k) {
    const int s = P.drives[k].slot, g = P.drives[k].cidx, m = P.slot_mode[s];
    int dm = -1;
    for (int q = 0; q < A.ndm; ++q)
      if (A.dm_mode[q] == m) dm = q;
    if (dm < 0) {
      if (A.ndm >= GA_MAXDM) return fail(SCP_EINVAL, "gather engine: too many driven modes");
      dm = A.ndm++;
      A.dm_mode[dm] = m;
    }
    bool seen = false;
    for (int q = 0; q < A.dm_n[dm]; ++q) seen |= A.dm_slot[dm][q] == s;
    if (seen) continue;
    if (A.dm_n[dm] >= GA_MAXC)
      return fail(SCP_EINVAL, "gather engine: too many drive operators on one mode");
    A.dm_slot[dm][A.dm_n[dm]] = s;
    A.dm_cidx[dm][A.dm_n[dm]++] = g;
  }
  // coupled pairs (i < j)
  for (int e = 0; e < P.ncoup; ++e) {
    const int si = sys->coup_slot_i[e], sj = sys->coup_slot_j[e];
    int i = P.slot_mode[si], j = P.slot_mode[sj];
    int ssi = si, ssj = sj;
    if (i > j) {
      std::swap(i, j);
      std::swap(ssi, ssj);
    }
    int p = -1;
    for (int q = 0; q < A.npr; ++q)
      if (A.pr_i[q] == i && A.pr_j[q] == j) p = q;
    if (p < 0) {
      if (A.npr >= GA_MAXPR) return fail(SCP_EINVAL, "gather engine: too many coupled pairs");
      p = A.npr++;
      A.pr_i[p] = i;
      A.pr_j[p] = j;
    }
    if (A.pr_n[p] >= GA_MAXC) return fail(SCP_EINVAL, "gather engine: too many couplings on one pair");
    A.pr_si[p][A.pr_n[p]] = ssi;
    A.pr_sj[p][A.pr_n[p]] = ssj;
    A.pr_g[p][A.pr_n[p]++] = (float)sys->coup[e].g;
  }
  // operator rows padded to an even length, the pair block and
  // the table starting at even entries (16-byte aligned rows)
  auto even = [](int x) { return x + (x & 1); };
  A.par = P.parity;
  A.nn = A.par ? (d + 1) / 2 : d;
  A.prow = even(A.nn * A.nn);
  A.orow = even(A.nn);
  A.srow = A.par ? A.orow : d;
  A.mrow = A.par ? even(A.nn + 1) : d;
  A.off_p = even(A.ndm * d * A.orow);
  A.off_j = A.off_p + A.npr * dd * A.prow;
  A.ntab = even(A.off_j + (A.has_jump ? N * dd : 0));
  if (A.ntab > GA_MAXTAB) return fail(SCP_EINVAL, "gather engine: stage table too large");
  const size_t L = open ? (size_t)D * D : (size_t)D;
  if ((3 * L + ((3 * L) & 1) + 2 * (size_t)A.ntab) * sizeof(float2) > 163840)
    return fail(SCP_EINVAL, "gather engine: column and stage tables exceed the LDS");
  A.ntabg = A.ntab;
  if (sys->d_rt != nullptr && (!open || l_real_supported(d, N))) {   // the real form (see build_gather_rows)
    A.real = P.real_frame != 0 ? 1 : 0;
    A.rt = sys->d_rt;
    A.rc = sys->d_rc;
    A.kappa = real_kappa(sys);
    for (int p = 0; p < A.npr; ++p)
      A.pmask |= 1 << (A.pr_j[p] == A.pr_i[p] + 1 ? A.pr_i[p] : N - 1);
    for (int q = 0; q < A.ndm; ++q) {
      A.dmask |= 1 << A.dm_mode[q];
      A.rd_s[A.dm_mode[q]] = (float)(A.kappa / sys->rc_scale[A.dm_mode[q]]);
      A.rd_c[A.dm_mode[q]] = (float)(1.0 / sys->rc_scale[A.dm_mode[q]]);
    }
  }
  return SCP_OK;
}

// Static rows of the real form: Re(sum_e g_e O_i (x) O_j) of the neighbour
// pairs and Re(O) of the driven modes over the levels Nb names, summed in FP64.
// Empty where the form does not apply: an operator with even entries or a
// complex term, a coupled pair that is no neighbour pair of the ring of modes
// or has more than two couplings, two drive operators on a mode, or a shape
// without a real stepper.  Behind them the gradient's rows (RShape), then the
// rows of each pair's single couplings without their strength (LShape).
// A drive operator is divided by its largest entry and c(t) multiplied by it in
// FP64 (scale): a static coefficient repeats its rounding at every stage, which
// for the resonant entry turns into an error of the rotation angle, while c(t)
// rounds differently at each (error of the final states against FP64: 5-transmon
// ring 1.6e-7 -> 1.3e-7, chains of 3 to 5 modes 0.8-1.2e-7 -> 0.7-0.9e-7).
std::vector<float> build_gather_rows(const scp_system* sys, double* scale) {
  std::vector<float> rt;
  const Plan& P = sys->plan;
  const int d = sys->d, N = sys->n_modes;
  if (!P.parity || !sys->real_ok || N < 3 ||
      !(g_supported(d, N, false) || l_real_supported(d, N) || l_column_supported(d, N)))
    return rt;
  GArgs A;
  if (g_args(sys, false, nullptr, nullptr, A) != SCP_OK) {
    set_error("");
    return rt;
  }
  for (int p = 0; p < A.npr; ++p)
    if ((A.pr_j[p] != A.pr_i[p] + 1 && !(A.pr_i[p] == 0 && A.pr_j[p] == N - 1)) || A.pr_n[p] > 2)
      return rt;
  for (int q = 0; q < A.ndm; ++q)
    if (A.dm_n[q] != 1) return rt;
  const int n = (d + 1) / 2, nn = n * n, pr = nn == 9 ? 12 : nn, dr = n == 3 ? 4 : n;
  const double kappa = real_kappa(sys);
  rt.assign((size_t)N * d * d * pr + (size_t)N * d * dr, 0.f);
  for (int p = 0; p < A.npr; ++p) {
    const int i = A.pr_i[p], j = A.pr_j[p], at = j == i + 1 ? i : N - 1;
    for (int a = 0; a < d; ++a)
      for (int b = 0; b < d; ++b)
        for (int x = 0; x < n; ++x)
          for (int z = 0; z < n; ++z) {
            const int la = nb_level(d, 1, x, a), lb = nb_level(d, 1, z, b);
            if (la < 0 || lb < 0) continue;
            cplx v = 0.0;
            for (const Coupling& c : sys->coup) {
              const bool fwd = c.i == i && c.j == j;
              if (!fwd && !(c.i == j && c.j == i)) continue;
              v += c.g * sys->modes[i].ops[fwd ? c.op_i : c.op_j][a * d + la] *
                   sys->modes[j].ops[fwd ? c.op_j : c.op_i][b * d + lb];
            }
            rt[((size_t)at * d * d + a * d + b) * pr + x * n + z] = (float)(kappa * v.real());
          }
  }
  for (int m = 0; m < N; ++m) scale[m] = kappa;
  for (int q = 0; q < A.ndm; ++q) {
    const int m = A.dm_mode[q], op = P.slot_op[A.dm_slot[q][0]];
    double big = 0.0;
    for (int i = 0; i < d * d; ++i) big = std::max(big, std::abs(sys->modes[m].ops[op][i].real()));
    if (big > 0.0) scale[m] = kappa * big;
    for (int a = 0; a < d; ++a)
      for (int x = 0; x < n; ++x) {
        const int la = nb_level(d, 1, x, a);
        if (la >= 0)
          rt[(size_t)N * d * d * pr + ((size_t)m * d + a) * dr + x] =
              (float)(sys->modes[m].ops[op][a * d + la].real() / (scale[m] / kappa));
      }
  }
  const int gr = (4 * n + 3) / 4 * 4;
  const size_t off_g = (rt.size() + 3) & ~(size_t)3;
  rt.resize(off_g + (size_t)N * 2 * d * gr + (size_t)N * d * 4, 0.f);
  for (int m = 0; m < N; ++m) {
    const ModeData& M = sys->modes[m];
    for (int u = 0; u < 2; ++u) {
      // i times real operators (n of a fluxonium): their imaginary parts
      bool im = false;
      for (size_t q = 0; q < sys->slot_mode.size(); ++q)
        if (sys->slot_mode[q] == m && sys->slot_op[q] == u) im = sys->slot_imag[q] != 0;
      for (int a = 0; a < d; ++a)
        for (int x = 0; x < n; ++x) {
          const int la = nb_level(d, 1, x, a);
          if (la < 0) continue;
          float* row = rt.data() + off_g + ((size_t)(m * 2 + u) * d + a) * gr;
          auto part = [&](cplx v) { return (float)(im ? v.imag() : v.real()); };
          row[x] = part(M.ops[u][a * d + la]);
          for (int th = 0; th < 3; ++th) row[(th + 1) * n + x] = part(M.dops[th][u][a * d + la]);
        }
    }
    for (int a = 0; a < d; ++a)
      for (int th = 0; th < 3; ++th)
        rt[off_g + (size_t)N * 2 * d * gr + ((size_t)m * d + a) * 4 + th] = (float)M.deps[th][a];
  }
  const size_t off_c = rt.size();
  rt.resize(off_c + (size_t)N * 2 * d * d * pr, 0.f);
  std::vector<int> seen(N, 0);
  for (const Coupling& c : sys->coup) {
    const int i = std::min(c.i, c.j), j = std::max(c.i, c.j), at = j == i + 1 ? i : N - 1;
    const cplx* oi = sys->modes[i].ops[c.i == i ? c.op_i : c.op_j];
    const cplx* oj = sys->modes[j].ops[c.i == i ? c.op_j : c.op_i];
    float* rows = rt.data() + off_c + (size_t)(at * 2 + seen[at]++) * d * d * pr;
    for (int a = 0; a < d; ++a)
      for (int b = 0; b < d; ++b)
        for (int x = 0; x < n; ++x)
          for (int z = 0; z < n; ++z) {
            const int la = nb_level(d, 1, x, a), lb = nb_level(d, 1, z, b);
            if (la >= 0 && lb >= 0)
              rows[(size_t)(a * d + b) * pr + x * n + z] = (float)(oi[a * d + la] * oj[b * d + lb]).real();
          }
  }
  return rt;
}

// Frame phases of the real form at the half steps [q_lo, q_lo + nq) into the
// workspace (open: of the matrix elements, A's modes before B's).
static scp_status g_phases(const scp_system* sys, bool open, int q_lo, int nq, float2* ph,
                           hipStream_t st) {
  double f[GA_MAXM][8] = {{0}};
  const int N = sys->n_modes;
  for (int m = 0; m < N; ++m)
    for (int a = 0; a < sys->d; ++a) {
      f[m][a] = sys->modes[m].frame[a];
      if (open) f[N + m][a] = -sys->modes[m].frame[a];
    }
  HIPCHK(g_real_phases(sys->d, open ? 2 * N : N, q_lo, nq, sys->h, f, ph, st));
  return SCP_OK;
}

// Gradient description: table slots, drive slots, drives and couplings.  Open
// systems: the table rows widen by the slot operators and the unit bands.
// Closed systems: by the slot operators, the one-mode derivative operators of
// every mode and the derivative slot operators; the coupling ends are grouped
// by mode and own slot.
static scp_status g_args_grad(const scp_system* sys, bool open, GArgs& A) {
  const Plan& P = sys->plan;
  const int N = sys->n_modes, d = sys->d, dd = d * d;
  auto tslot = [&](int s) -> int {
    for (int k = 0; k < A.nsl; ++k)
      if (A.sl_slot[k] == s) return k;
    if (A.nsl >= GA_MAXSL) return -1;
    A.sl_slot[A.nsl] = s;
    return A.nsl++;
  };
  if (P.ndrives > GA_MAXDR) return fail(SCP_EINVAL, "gather-engine gradient: too many drives");
  if (P.ncoup > GA_MAXCP) return fail(SCP_EINVAL, "gather-engine gradient: too many couplings");
  A.ndr = P.ndrives;
  for (int k = 0; k < P.ndrives; ++k) {
    const int s = P.drives[k].slot;
    int ds = -1;
    for (int q = 0; q < A.nds; ++q)
      if (A.sl_slot[A.ds_sl[q]] == s) ds = q;
    if (ds < 0) {
      if (A.nds >= GA_MAXDS)
        return fail(SCP_EINVAL, "gather-engine gradient: too many drive operators");
      const int t = tslot(s);
      if (t < 0) return fail(SCP_EINVAL, "gather-engine gradient: too many operator slots");
      ds = A.nds++;
      A.ds_sl[ds] = t;
      A.ds_mode[ds] = P.slot_mode[s];
    }
    A.dr_ds[k] = ds;
    A.dr_par0[k] = P.drives[k].par0;
    A.dr_npar[k] = P.drives[k].npar;
  }
  A.ncp = P.ncoup;
  for (int e = 0; e < P.ncoup; ++e) {
    const int si = sys->coup_slot_i[e], sj = sys->coup_slot_j[e];
    const int ti = tslot(si), tj = tslot(sj);
    if (ti < 0 || tj < 0) return fail(SCP_EINVAL, "gather-engine gradient: too many operator slots");
    A.cp_i[e] = P.slot_mode[si];
    A.cp_j[e] = P.slot_mode[sj];
    A.cp_si[e] = ti;
    A.cp_sj[e] = tj;
    A.cp_g[e] = (float)sys->coup[e].g;
  }
  if (A.rt != nullptr) {
    // operator index on a mode: 0 for n, 1 for phi
    for (int q = 0; q < A.ndm; ++q) {
      const int m = A.dm_mode[q];
      A.rd_u[m] = P.slot_op[A.dm_slot[q][0]];
      for (int x = 0; x < A.nds; ++x)
        if (A.ds_mode[x] == m) A.rd_k[m] = x;
    }
    for (int e = 0; e < P.ncoup; ++e) {
      const Coupling& c = sys->coup[e];
      const int i = std::min(c.i, c.j), j = std::max(c.i, c.j), p = j == i + 1 ? i : N - 1;
      const int ui = c.i == i ? c.op_i : c.op_j, uj = c.i == i ? c.op_j : c.op_i;
      const int q = A.rp_n[p]++;
      const float sg = sys->slot_imag[sys->coup_slot_i[e]] ? -1.f : 1.f;
      A.rp_u[p][q] = ui | (uj << 1);
      A.rp_c[p][q] = e;
      A.rp_s[p][q] = sg;
      A.rp_g[p][q] = sg * (float)c.g;
    }
  }
  A.off_s = A.ntab;
  if (open) {
    A.grad = 1;
    A.off_u = A.off_s + A.nsl * d * A.srow;
    A.ntabg = A.off_u + N * dd;
    A.ntabg += A.ntabg & 1;   // the second table buffer starts 16-byte aligned
  } else {
    A.grad = 2;
    A.off_dslot = P.off_dslot;
    for (int m = 0; m < N; ++m) A.mdm[m] = -1;
    for (int q = 0; q < A.ndm; ++q) A.mdm[A.dm_mode[q]] = q;
    for (int m = 0; m < N; ++m)
      for (int th = 0; th < 3; ++th)
        for (int a = 0; a < d; ++a) A.deps[m][th][a] = (float)sys->modes[m].deps[th][a];
    // coupling ends of each mode, grouped by the own table slot
    int k = 0;
    for (int m = 0; m < N; ++m) {
      A.me_beg[m] = k;
      struct End { int own, c, psl, pm, first; };
      std::vector<End> ends;
      for (int e = 0; e < P.ncoup; ++e) {
        if (A.cp_i[e] == m) ends.push_back({A.cp_si[e], e, A.cp_sj[e], A.cp_j[e], 1});
        if (A.cp_j[e] == m) ends.push_back({A.cp_sj[e], e, A.cp_si[e], A.cp_i[e], 0});
      }
      std::stable_sort(ends.begin(), ends.end(),
                       [](const End& x, const End& y) { return x.own < y.own; });
      for (size_t q = 0; q < ends.size(); ++q) {
        if (k >= GA_MAXME) return fail(SCP_EINVAL, "gather-engine gradient: too many coupling ends");
        const End& x = ends[q];
        const int last = (q + 1 == ends.size() || ends[q + 1].own != x.own) ? 1 : 0;
        A.me[k++] = x.c | (x.own << 5) | (x.psl << 10) | (x.pm << 15) | (x.first << 20) |
                    (last << 21);
      }
    }
    A.me_beg[N] = k;
    A.off_m = A.off_s + A.nsl * d * A.srow;
    A.off_d = A.off_m + 3 * N * d * A.mrow;
    A.off_u = A.off_m;
    A.ntabg = A.off_d + 3 * A.nsl * d * A.srow;
    A.ntabg += A.ntabg & 1;   // the second table buffer starts 16-byte aligned
  }
  if (A.ntabg > GA_MAXTAB) return fail(SCP_EINVAL, "gather-engine gradient: stage table too large");
  return SCP_OK;
}

// Bytes of the real form's frame phases (0 where it does not apply; the same
// for either frame setting of a system that allows it).
static size_t g_ph_bytes(const scp_system* sys, bool open) {
  if (sys->d_rt == nullptr || (open && !l_real_supported(sys->d, sys->n_modes))) return 0;
  const size_t L = (size_t)sys->D * (open ? sys->D : 1);
  return align256((2 * (size_t)sys->n_steps + 1) * L * sizeof(float2));
}

// A closed system's forward in the real form without checkpoints goes in runs of
// steps, whose frame phases are formed before each: 256 MiB of them at most, so
// that they do not grow with the steps (105 kB a step at D = 6561), the
// compensated state carried between runs in the workspace: [phases
// [2 run + 2][D]][state [S][D] float4].  A run is 70 ms or more at that size
// (2557 steps of D = 6561); the launches between two cost 65 us.
static int g_run_steps(const scp_system* sys) {
  return (int)std::min<int64_t>(sys->n_steps, ((int64_t)256 << 20) / (2 * sys->D * sizeof(float2)));
}
static size_t g_run_ph_bytes(const scp_system* sys) {
  return align256((2 * (size_t)g_run_steps(sys) + 2) * sys->D * sizeof(float2));
}
static size_t g_run_bytes(const scp_system* sys, int S) {
  if (sys->d_rt == nullptr) return 0;
  const bool one = sys->n_steps <= g_run_steps(sys);
  return g_run_ph_bytes(sys) + (one ? 0 : align256((size_t)S * sys->D * sizeof(float4)));
}

// The runs: A's description at dargs, `at` the workspace behind it, step(n_lo,
// n_hi, st_in, st_out) launches the stepper.
template <typename F>
static scp_status g_real_runs(scp_system* sys, GArgs A, GArgs* dargs, char* at, hipStream_t st, F step) {
  const int N = sys->n_steps, run = g_run_steps(sys);
  float2* ph = reinterpret_cast<float2*>(at);
  float4* state = reinterpret_cast<float4*>(at + g_run_ph_bytes(sys));
  for (int n = 0; n < N; n += run) {
    const int n1 = std::min(N, n + run);
    // the stepper counts half steps from the first one of all (an offset taken in
    // the kernel cost 1 % of a step of D = 625)
    A.ph = reinterpret_cast<const float2*>(reinterpret_cast<uintptr_t>(ph) -
                                           (size_t)2 * n * sys->D * sizeof(float2));
    hipLaunchKernelGGL(store_args_kernel, dim3(1), dim3(64), 0, st, A, dargs);
    HIPCHK(hipGetLastError());
    // the stepper reads one half step beyond the run's last, ahead of its use
    SCP_TRY(g_phases(sys, false, 2 * n, std::min(2 * N, 2 * n1 + 1) - 2 * n + 1, ph, st));
    hipEvent_t t0 = timing_start(sys, st);
    HIPCHK(step(n, n1, n == 0 ? nullptr : state, n1 == N ? nullptr : state));
    timing_stop(sys, t0, 0, st);
  }
  return SCP_OK;
}

// Workspace: [GArgs][stage tables [3N][ntab], with those of an open system its
// jump bands [2N+1][N][d*d]; or, in the real form, the frame phases: of an open
// system [2N+1][L], of a closed one as above].
static size_t g_tab_bytes(const scp_system* sys, bool open, int ntab) {
  const size_t dd = (size_t)sys->d * sys->d;
  size_t t = align256(sizeof(GArgs)) + align256(3 * (size_t)sys->n_steps * ntab * sizeof(float2));
  if (open) t += align256((2 * (size_t)sys->n_steps + 1) * sys->n_modes * dd * sizeof(float2));
  return t;
}
static size_t g_ws_bytes(const scp_system* sys, bool open, int S, int ntab) {
  return std::max(g_tab_bytes(sys, open, ntab),
                  align256(sizeof(GArgs)) + (open ? g_ph_bytes(sys, true) : g_run_bytes(sys, S)));
}

static scp_status g_run(scp_system* sys, bool open, const double* gamma1, const double* gammaphi,
                        int S, void* ws, size_t ws_bytes, const float2* x0, float2* xT,
                        hipStream_t st) {
  GArgs A;
  SCP_TRY(g_args(sys, open, gamma1, gammaphi, A));
  if (ws_bytes < g_ws_bytes(sys, open, S, A.ntab)) {
    // an open system's phases are five times its tables (d = 3, N = 4): where only
    // the tables fit, the complex rows run
    if (!open || ws_bytes < g_tab_bytes(sys, true, A.ntab)) return fail(SCP_EINVAL, "workspace too small");
    A.real = 0;
  }
  char* w = static_cast<char*>(ws);
  GArgs* dargs = reinterpret_cast<GArgs*>(w);
  w += align256(sizeof(GArgs));
  float2* gtab = reinterpret_cast<float2*>(w);
  w += align256(3 * (size_t)sys->n_steps * A.ntab * sizeof(float2));
  float2* jtab = open ? reinterpret_cast<float2*>(w) : nullptr;
  A.optab = sys->d_ops;
  A.ctab = sys->d_ctab;
  A.jtab = jtab;
  A.gtab = gtab;
  A.x0 = x0;
  A.xT = xT;
  A.S = S;
  const int N = sys->n_modes, d = sys->d;
  if (A.has_jump && !A.real) {
    JtabStatic js;
    std::memset(&js, 0, sizeof(js));
    js.d = d;
    js.N = N;
    js.nq = 2 * sys->n_steps + 1;
    js.h = sys->h;
    for (int m = 0; m < N; ++m)
      for (int a = 0; a < d; ++a) js.f[m][a] = sys->modes[m].frame[a];
    hipLaunchKernelGGL(jtab_kernel, dim3(js.nq), dim3(64), 0, st, js, jtab);
    HIPCHK(hipGetLastError());
  }
  if (A.real && !open)
    return g_real_runs(sys, A, dargs, reinterpret_cast<char*>(gtab), st,
                       [&](int n_lo, int n_hi, const float4* st_in, float4* st_out) {
                         return g_dispatch(d, N, false, g_form(A), dargs, nullptr, S, A.ntab, n_lo, n_hi,
                                           st_in, st_out, st);
                       });
  if (A.real) A.ph = gtab;
  hipLaunchKernelGGL(store_args_kernel, dim3(1), dim3(64), 0, st, A, dargs);
  HIPCHK(hipGetLastError());
  if (A.real) {
    SCP_TRY(g_phases(sys, true, 0, 2 * sys->n_steps + 1, gtab, st));
  } else {
    hipLaunchKernelGGL(gtab_kernel, dim3(3 * sys->n_steps), dim3(256), 0, st, dargs, d, N, gtab);
    HIPCHK(hipGetLastError());
  }
  if (S == 0) return SCP_OK;
  hipEvent_t t0 = timing_start(sys, st);
  HIPCHK(g_dispatch(d, N, open, g_form(A), dargs, nullptr, S, A.ntab, 0, sys->n_steps, nullptr, nullptr, st));
  timing_stop(sys, t0, 0, st);
  return SCP_OK;
}

// --- open systems ----------------------------------------------------------
scp_status lindblad_check(const scp_system* sys) {
  if (!g_supported(sys->d, sys->n_modes, true))
    return fail(SCP_EINVAL, "open-system path: the density matrix must fit in LDS (d=2: N<=5, "
                            "d=3: N<=4, d=4: N<=3, d=5: N<=2)");
  GArgs A;
  return g_args(sys, true, nullptr, nullptr, A);
}

size_t lindblad_workspace_bytes(const scp_system* sys) {
  GArgs A;
  std::vector<double> one(sys->n_modes, 1.0);   // the largest table: relaxation on
  if (g_args(sys, true, one.data(), nullptr, A) != SCP_OK) return 0;
  return g_ws_bytes(sys, true, 1, A.ntab);
}

scp_status launch_lindblad(scp_system* sys, const double* gamma1, const double* gammaphi, int S,
                           void* ws, size_t ws_bytes, const float2* rho0, float2* rhoT,
                           hipStream_t st) {
  SCP_TRY(lindblad_check(sys));
  return g_run(sys, true, gamma1, gammaphi, S, ws, ws_bytes, rho0, rhoT, st);
}

// --- closed systems above the gather engine's shapes: forward -----------------
bool real_column_supported(const scp_system* sys) {
  return sys->d_rt != nullptr && l_column_supported(sys->d, sys->n_modes);
}

size_t real_column_bytes(const scp_system* sys, int S) {
  return align256(sizeof(GArgs)) + g_run_bytes(sys, S);
}

scp_status launch_real_column(scp_system* sys, int S, void* ws, const float2* x0, float2* xT,
                              hipStream_t st) {
  GArgs A;
  SCP_TRY(g_args(sys, false, nullptr, nullptr, A));
  GArgs* dargs = static_cast<GArgs*>(ws);
  A.x0 = x0;
  A.xT = xT;
  A.S = S;
  return g_real_runs(sys, A, dargs, static_cast<char*>(ws) + align256(sizeof(GArgs)), st,
                     [&](int n_lo, int n_hi, const float4* st_in, float4* st_out) {
                       return l_real_column(sys->d, sys->n_modes, dargs, S, n_lo, n_hi, st_in, st_out, st);
                     });
}

// The gradient from the steps' sums, copied to the host (synchronises st).
static scp_status g_fold(scp_system* sys, int S, const GArgs* dargs, const GAdj* dadj, int nblk,
                         int nacc, double* part, double* dgrad, double* grad, hipStream_t st) {
  hipLaunchKernelGGL(g_fold_kernel, dim3(S * nblk), dim3(256), 0, st, dargs, dadj, nblk, part);
  HIPCHK(hipGetLastError());
  hipLaunchKernelGGL(g_fold_sum_kernel, dim3((nacc + 63) / 64), dim3(64), 0, st, part, S, nblk, nacc,
                     dgrad);
  HIPCHK(hipGetLastError());
  HIPCHK(hipMemcpyAsync(grad, dgrad, nacc * sizeof(double), hipMemcpyDeviceToHost, st));
  HIPCHK(hipStreamSynchronize(st));
  return SCP_OK;
}

// Open-system gradient.  Workspace: [GArgs][GAdj][stage tables [3N][ntabg]
// and unit bands [2N+1][N][d*d], or the real form's frame phases [2N+1][L]]
// [checkpoints [S][nck][L] float4][stage inputs [S][ce][4][L]][costate [S][L]
// float4][partial sums [S][nacc] double, or the real form's sums of the steps
// [S][N][gw] double, their blocks [S][nblk][nacc] and the gradient [nacc]].
// The size is the same for either frame setting of a system; without `real`, that
// of the tables alone.
struct LbAdjLayout {
  size_t args, adj, gtab, jtab, ck, seg, part, lam, total;
  size_t gs, blk, grad;   // real form
  int ce, nck, nacc, ntabg, gw, nblk;
};

static scp_status lb_adj_layout(const scp_system* sys, int S, bool real, LbAdjLayout& w, GArgs* Aout) {
  GArgs A;
  std::vector<double> one(sys->n_modes, 1.0);   // the widest table: relaxation on
  SCP_TRY(g_args(sys, true, one.data(), nullptr, A));
  SCP_TRY(g_args_grad(sys, true, A));
  const Plan& P = sys->plan;
  const size_t L = (size_t)sys->D * sys->D, dd = (size_t)sys->d * sys->d;
  const int N = sys->n_steps;
  w.ce = (int)std::ceil(std::sqrt((double)N));
  w.nck = (N + w.ce - 1) / w.ce;
  w.nacc = P.npulse + P.ncoup + 2 * sys->n_modes;
  w.ntabg = A.ntabg;
  size_t off = 0;
  w.args = off;
  off += align256(sizeof(GArgs));
  w.adj = off;
  off += align256(sizeof(GAdj));
  w.gtab = off;
  w.jtab = off + align256(3 * (size_t)N * A.ntabg * sizeof(float2));
  const size_t tabs = w.jtab + align256((2 * (size_t)N + 1) * sys->n_modes * dd * sizeof(float2));
  off = std::max(tabs, off + (real ? g_ph_bytes(sys, true) : 0));
  w.ck = off;
  off += align256((size_t)S * w.nck * L * sizeof(float4));
  w.seg = off;
  off += align256((size_t)S * w.ce * 4 * L * sizeof(float2));
  w.lam = off;
  off += align256((size_t)S * L * sizeof(float4));
  w.part = w.gs = off;
  off += align256((size_t)S * w.nacc * sizeof(double));
  w.gw = 4 * A.nds + P.ncoup + 2 * sys->n_modes;
  w.nblk = (N + GF_STEPS - 1) / GF_STEPS;
  w.blk = w.grad = 0;
  if (real && A.rt != nullptr) {
    size_t q = w.gs + align256((size_t)S * N * w.gw * sizeof(double));
    w.blk = q;
    q += align256((size_t)S * w.nblk * w.nacc * sizeof(double));
    w.grad = q;
    q += align256((size_t)w.nacc * sizeof(double));
    off = std::max(off, q);
  }
  w.total = off;
  if (g_adj_lds(sys->d, sys->n_modes, true, A.ntabg, w.nacc) > 163840)
    return fail(SCP_EINVAL, "open-system gradient: column and tables exceed the LDS");
  if (Aout) *Aout = A;
  return SCP_OK;
}

scp_status lindblad_adjoint_workspace_bytes(const scp_system* sys, int S, size_t* bytes) {
  SCP_TRY(lindblad_check(sys));
  LbAdjLayout w;
  SCP_TRY(lb_adj_layout(sys, S, true, w, nullptr));
  *bytes = w.total;
  return SCP_OK;
}

scp_status launch_lindblad_adjoint(scp_system* sys, const double* gamma1, const double* gammaphi,
                                   int S, void* ws, size_t ws_bytes, const float2* rho0,
                                   const float2* cot, double* grad, hipStream_t st) {
  SCP_TRY(lindblad_check(sys));
  LbAdjLayout w;
  SCP_TRY(lb_adj_layout(sys, S, true, w, nullptr));
  const bool room = ws_bytes >= w.total;   // else the complex rows, if those fit
  if (!room) SCP_TRY(lb_adj_layout(sys, S, false, w, nullptr));
  if (ws_bytes < w.total) return fail(SCP_EINVAL, "workspace too small");
  GArgs A;
  SCP_TRY(g_args(sys, true, gamma1, gammaphi, A));
  SCP_TRY(g_args_grad(sys, true, A));
  if (!room) A.real = 0;
  char* base = static_cast<char*>(ws);
  GArgs* dargs = reinterpret_cast<GArgs*>(base + w.args);
  GAdj* dadj = reinterpret_cast<GAdj*>(base + w.adj);
  float2* gtab = reinterpret_cast<float2*>(base + w.gtab);
  float2* jtab = reinterpret_cast<float2*>(base + w.jtab);
  const int N = sys->n_modes, d = sys->d;
  A.optab = sys->d_ops;
  A.ctab = sys->d_ctab;
  A.jtab = jtab;
  A.gtab = gtab;
  A.ph = gtab;   // real form
  A.x0 = rho0;
  A.xT = nullptr;
  A.S = S;
  GAdj B;
  std::memset(&B, 0, sizeof(B));
  B.ck = reinterpret_cast<float4*>(base + w.ck);
  B.cot = cot;
  B.seg = reinterpret_cast<float2*>(base + w.seg);
  B.dctab = sys->d_dctab64;
  B.part = reinterpret_cast<double*>(base + w.part);
  B.gs = reinterpret_cast<double*>(base + w.gs);
  B.gw = w.gw;
  B.lam = reinterpret_cast<float4*>(base + w.lam);
  B.ce = w.ce;
  B.nck = w.nck;
  B.npulse = sys->plan.npulse;
  B.nacc = w.nacc;
  if (!A.real) {
    JtabStatic js;
    std::memset(&js, 0, sizeof(js));
    js.d = d;
    js.N = N;
    js.nq = 2 * sys->n_steps + 1;
    js.h = sys->h;
    for (int m = 0; m < N; ++m)
      for (int a = 0; a < d; ++a) js.f[m][a] = sys->modes[m].frame[a];
    hipLaunchKernelGGL(jtab_kernel, dim3(js.nq), dim3(64), 0, st, js, jtab);
    HIPCHK(hipGetLastError());
  }
  hipLaunchKernelGGL(store_args_kernel, dim3(1), dim3(64), 0, st, A, dargs);
  HIPCHK(hipGetLastError());
  hipLaunchKernelGGL(store_adj_kernel, dim3(1), dim3(64), 0, st, B, dadj);
  HIPCHK(hipGetLastError());
  if (A.real) {
    SCP_TRY(g_phases(sys, true, 0, 2 * sys->n_steps + 1, gtab, st));
  } else {
    hipLaunchKernelGGL(gtab_kernel, dim3(3 * sys->n_steps), dim3(256), 0, st, dargs, d, N, gtab);
    HIPCHK(hipGetLastError());
  }
  hipEvent_t t0 = timing_start(sys, st);
  HIPCHK(g_dispatch(d, N, true, g_form(A), dargs, dadj, S, A.ntab, 0, sys->n_steps, nullptr, nullptr, st));
  timing_stop(sys, t0, 0, st);
  t0 = timing_start(sys, st);
  HIPCHK(g_adj_dispatch(d, N, true, g_form(A), dargs, dadj, S, A.ntabg, w.nacc, 0, 1, st));
  timing_stop(sys, t0, 2, st);
  if (A.real) {
    SCP_TRY(g_fold(sys, S, dargs, dadj, w.nblk, w.nacc, reinterpret_cast<double*>(base + w.blk),
                   reinterpret_cast<double*>(base + w.grad), grad, st));
    for (int k = 0; k < w.nacc; ++k)
      if (!std::isfinite(grad[k])) return fail(SCP_ENONFINITE, "non-finite gradient");
    return SCP_OK;
  }
  std::vector<double> part((size_t)S * w.nacc);
  HIPCHK(hipMemcpyAsync(part.data(), base + w.part, part.size() * sizeof(double),
                        hipMemcpyDeviceToHost, st));
  HIPCHK(hipStreamSynchronize(st));
  for (int k = 0; k < w.nacc; ++k) {
    double v = 0.0;
    for (int c = 0; c < S; ++c) v += part[(size_t)c * w.nacc + k];   // fixed order
    if (!std::isfinite(v)) return fail(SCP_ENONFINITE, "non-finite gradient");
    grad[k] = v;
  }
  return SCP_OK;
}

// --- closed systems ----------------------------------------------------------
// The gather engine (one workgroup per column) takes a closed system of a
// compiled shape when its columns would leave most of the chip idle in the
// register-layout stepper; in its real form, for as many columns as it wins with.
// Measured, register -> real form, us per step (forward; forward + gradient):
//   6-fluxonium chain, d = 4, 64 / 256 columns   54 -> 14;  252 -> 71 / 258 -> 160
//   7-transmon ring, d = 3, 128 / 256 columns    47 -> 23;  245 -> 119 / 249 -> 194
//   5-fluxonium chain, d = 5, 128 / 256 columns  51 -> 34;  266 -> 165 / 272 -> 266
//   5-transmon ring, d = 5, 128 / 160 / 256      48 -> 45;  247 -> 195 / 249 -> 258 / 253 -> 312
//   4-transmon ring, d = 4, 256 / 1024 columns   44 -> 3.5; 186 -> 18 / 186 -> 43
//   6-transmon ring, d = 3, 768 / 900 / 1024     33 -> 12;  151 -> 138 / 168 -> 182 / 169 -> 183
//   5-transmon ring, d = 4, 768 / 1024           48 -> 14;  219 -> 152 / 221 -> 202
//   9-mode ring, d = 2, 512 / 1024 columns       34 -> 4.2; 182 -> 89 / 183 -> 176
//   10-mode ring, d = 2, 512 / 600 / 1024        47 -> 9.1; 232 -> 197 / 234 -> 242 / 237 -> 389
// A gradient's time grows with the rounds of workgroups (256 of 1024 threads).
// Above D = 512 it wins for four of them, three at d = 3 and two at d = 2 (rows of
// fewer entries for the same sums per wave); above D = 1024 for one, half of one
// with five levels there (four elements a thread, the last one's threads nearly
// idle).
bool gather_preferred(const scp_system* sys, int S, bool real, bool grad) {
  if (!g_supported(sys->d, sys->n_modes, false)) return false;
  GArgs A;
  if (g_args(sys, false, nullptr, nullptr, A) != SCP_OK) {
    set_error("");
    return false;
  }
  if (real && A.rt != nullptr) {
    if (sys->D > 1024) return S <= (grad && sys->d == 5 ? 128 : 256);
    return S <= (!grad || sys->D <= 512 || sys->d > 3 ? 1024 : (sys->d == 2 ? 512 : 768));
  }
  if (S > 256) return false;
  const int fused_wg = (S + sys->plan.CPW - 1) / sys->plan.CPW;
  return fused_wg < 64;
}

bool gather_supported(const scp_system* sys) {
  if (!g_supported(sys->d, sys->n_modes, false)) return false;
  GArgs A;
  if (g_args(sys, false, nullptr, nullptr, A) != SCP_OK) {
    set_error("");
    return false;
  }
  return true;
}

size_t gather_workspace_bytes(const scp_system* sys, int S) {
  GArgs A;
  if (g_args(sys, false, nullptr, nullptr, A) != SCP_OK) {
    set_error("");
    return 0;
  }
  return g_ws_bytes(sys, false, S, A.ntab);
}

scp_status launch_gather_forward(scp_system* sys, int S, void* ws, size_t ws_bytes,
                                 const float2* psi0, float2* psiT, hipStream_t st) {
  return g_run(sys, false, nullptr, nullptr, S, ws, ws_bytes, psi0, psiT, st);
}

// Closed-system gradient on the gather engine.  Workspace: [GArgs][GAdj]
// [stage tables [3N][ntabg], or the real form's frame phases [2N+1][D]]
// [checkpoints [S][nck][D] float4] and, for the adjoint, [stage inputs [S nseg][ce][4][D]][sums of the steps [S][N][gw]
// double][their blocks [S][nblk][nacc] double][gradient [nacc] double][costate
// at the segments' ends [S][nck][D] float4].  The forward with checkpoints and
// the adjoint share the offsets of the first four.
struct GcLayout {
  size_t args, adj, gtab, ph, ck, seg, gs, part, grad, lam, total;
  int nck, nacc, gw, nblk;
  int nseg;   // segments walked side by side
};

// nseg > 0: that many segments side by side at most.
static scp_status gc_layout(const scp_system* sys, int S, int ce, bool with_grad, int nseg,
                            GcLayout& w, GArgs* Aout) {
  if (!g_supported(sys->d, sys->n_modes, false))
    return fail(SCP_EINVAL, "gather engine: no compiled stepper for this d and mode count");
  GArgs A;
  SCP_TRY(g_args(sys, false, nullptr, nullptr, A));
  SCP_TRY(g_args_grad(sys, false, A));
  const size_t L = (size_t)sys->D;
  const int N = sys->n_steps;
  w.nck = (N + ce - 1) / ce;
  w.nacc = sys->plan.npulse + 3 * sys->n_modes + sys->plan.ncoup;
  w.gw = 4 * A.nds + 3 * sys->n_modes + A.ncp;
  w.nblk = (N + GF_STEPS - 1) / GF_STEPS;
  // two workgroups for every compute unit (four of at most 256 threads), where
  // there are that many segments (each holds a buffer of stage inputs); two
  // segments at least, as many buffers as a walk one segment after the other needs
  // to hide its recompute.  4-transmon ring, d = 4, n_g = 0.2, 256 columns, forward
  // and gradient: two of 256 threads 55 us per step, four 47 (53 with one segment
  // after the other, which needs no sweep)
  const int most = sys->D <= 256 ? 1024 : 512;
  w.nseg = std::min(w.nck, std::max(2, (most + S - 1) / S));
  if (nseg > 0) w.nseg = std::min(w.nseg, nseg);
  size_t off = 0;
  w.args = off;
  off += align256(sizeof(GArgs));
  w.adj = off;
  off += align256(sizeof(GAdj));
  w.gtab = off;
  w.ph = off;
  off += std::max(align256(3 * (size_t)N * A.ntabg * sizeof(float2)), g_ph_bytes(sys, false));
  w.ck = off;
  off += align256((size_t)S * w.nck * L * sizeof(float4));
  w.seg = w.gs = w.part = w.grad = w.lam = off;
  if (with_grad) {
    w.seg = off;
    off += align256((size_t)S * w.nseg * std::min(ce, N) * 4 * L * sizeof(float2));
    w.gs = off;
    off += align256((size_t)S * N * w.gw * sizeof(double));
    w.part = off;
    off += align256((size_t)S * w.nblk * w.nacc * sizeof(double));
    w.grad = off;
    off += align256((size_t)w.nacc * sizeof(double));
    w.lam = off;
    off += align256((size_t)S * w.nck * L * sizeof(float4));
  }
  w.total = off;
  if (g_adj_lds(sys->d, sys->n_modes, false, A.ntabg, w.nacc) > 163840)
    return fail(SCP_EINVAL, "gather-engine gradient: column and tables exceed the LDS");
  if (Aout) *Aout = A;
  return SCP_OK;
}

scp_status gather_grad_check(const scp_system* sys) {
  GcLayout w;
  return gc_layout(sys, 1, 1, true, 0, w, nullptr);
}

size_t gather_grad_workspace_bytes(const scp_system* sys, int S, int ce, bool with_grad) {
  GcLayout w;
  if (gc_layout(sys, S, ce, with_grad, 0, w, nullptr) != SCP_OK) {
    set_error("");
    return 0;
  }
  return w.total;
}

// Segments side by side that a gradient's workspace of `bytes` has room for (0: none).
int gather_grad_segments(const scp_system* sys, int S, int ce, size_t bytes) {
  GcLayout w;
  int n = 0;   // the most, then at most what the room left by the rest allows
  for (;;) {
    if (gc_layout(sys, S, ce, true, n, w, nullptr) != SCP_OK) {
      set_error("");
      return 0;
    }
    if (w.total <= bytes) return w.nseg;
    const size_t seg = (size_t)S * std::min(ce, sys->n_steps) * 4 * sys->D * sizeof(float2);
    n = w.nseg - (int)std::min<size_t>(w.nseg, (w.total - bytes + seg - 1) / seg);
    if (n < 1) return 0;
  }
}

// Args and adjoint description into the workspace (and the stage tables when
// `tables`).
static scp_status gc_prepare(scp_system* sys, int S, int ce, bool with_grad, int nseg, char* base,
                             size_t ws_bytes, const float2* x0, float2* xT, const float2* cot,
                             bool tables, GcLayout& w, GArgs& A, hipStream_t st) {
  SCP_TRY(gc_layout(sys, S, ce, with_grad, nseg, w, &A));
  if (ws_bytes < w.total) return fail(SCP_EINVAL, "workspace too small");
  GArgs* dargs = reinterpret_cast<GArgs*>(base + w.args);
  GAdj* dadj = reinterpret_cast<GAdj*>(base + w.adj);
  float2* gtab = reinterpret_cast<float2*>(base + w.gtab);
  A.optab = sys->d_ops;
  A.ctab = sys->d_ctab;
  A.jtab = nullptr;
  A.gtab = gtab;
  A.x0 = x0;
  A.xT = xT;
  A.S = S;
  A.ph = reinterpret_cast<float2*>(base + w.ph);
  GAdj B;
  std::memset(&B, 0, sizeof(B));
  B.ck = reinterpret_cast<float4*>(base + w.ck);
  B.cot = cot;
  B.seg = with_grad ? reinterpret_cast<float2*>(base + w.seg) : nullptr;
  B.dctab = sys->d_dctab64;
  B.gs = with_grad ? reinterpret_cast<double*>(base + w.gs) : nullptr;
  B.gw = w.gw;
  B.lam = with_grad ? reinterpret_cast<float4*>(base + w.lam) : nullptr;
  B.ce = std::min(ce, sys->n_steps);   // one segment: the same walk
  B.nck = w.nck;
  B.npulse = sys->plan.npulse;
  B.nacc = w.nacc;
  hipLaunchKernelGGL(store_args_kernel, dim3(1), dim3(64), 0, st, A, dargs);
  HIPCHK(hipGetLastError());
  hipLaunchKernelGGL(store_adj_kernel, dim3(1), dim3(64), 0, st, B, dadj);
  HIPCHK(hipGetLastError());
  if (tables) {
    if (A.real)
      return g_phases(sys, false, 0, 2 * sys->n_steps + 1, reinterpret_cast<float2*>(base + w.ph), st);
    hipLaunchKernelGGL(gtab_kernel, dim3(3 * sys->n_steps), dim3(256), 0, st, dargs, sys->d,
                       sys->n_modes, gtab);
    HIPCHK(hipGetLastError());
  }
  return SCP_OK;
}

scp_status launch_gather_ckpt_forward(scp_system* sys, int S, int ce, void* ws, size_t ws_bytes,
                                      const float2* psi0, float2* psiT, hipStream_t st) {
  char* base = static_cast<char*>(ws);
  GcLayout w;
  GArgs A;
  SCP_TRY(gc_prepare(sys, S, ce, false, 0, base, ws_bytes, psi0, psiT, nullptr, true, w, A, st));
  hipEvent_t t0 = timing_start(sys, st);
  HIPCHK(g_dispatch(sys->d, sys->n_modes, false, g_form(A), reinterpret_cast<GArgs*>(base + w.args),
                    reinterpret_cast<GAdj*>(base + w.adj), S, A.ntab, 0, sys->n_steps, nullptr,
                    nullptr, st));
  timing_stop(sys, t0, 0, st);
  return SCP_OK;
}

static scp_status gc_fold(scp_system* sys, int S, char* base, const GcLayout& w, double* grad,
                          hipStream_t st) {
  return g_fold(sys, S, reinterpret_cast<GArgs*>(base + w.args), reinterpret_cast<GAdj*>(base + w.adj),
                w.nblk, w.nacc, reinterpret_cast<double*>(base + w.part),
                reinterpret_cast<double*>(base + w.grad), grad, st);
}

// The reverse walk from the checkpoints (and stage tables) that
// launch_gather_ckpt_forward left in the same workspace: the costate sweep,
// then the segments side by side.
scp_status launch_gather_adjoint(scp_system* sys, int S, int ce, int nseg, void* ws, size_t ws_bytes,
                                 const float2* cot, double* grad, hipStream_t st) {
  char* base = static_cast<char*>(ws);
  GcLayout w;
  GArgs A;
  SCP_TRY(gc_prepare(sys, S, ce, true, nseg, base, ws_bytes, nullptr, nullptr, cot, false, w, A, st));
  const GArgs* dargs = reinterpret_cast<GArgs*>(base + w.args);
  const GAdj* dadj = reinterpret_cast<GAdj*>(base + w.adj);
  const int d = sys->d, N = sys->n_modes;
  hipEvent_t t0 = timing_start(sys, st);
  HIPCHK(g_cos_dispatch(d, N, g_form(A), dargs, dadj, S, A.ntab, w.nck - 1, 0, st));
  for (int gs = w.nck - 1; gs >= 0; gs -= w.nseg)
    HIPCHK(g_adj_dispatch(d, N, false, g_form(A), dargs, dadj, S, A.ntabg, w.nacc, gs,
                          std::min(w.nseg, gs + 1), st));
  timing_stop(sys, t0, 2, st);
  SCP_TRY(gc_fold(sys, S, base, w, grad, st));
  for (int k = 0; k < w.nacc; ++k)
    if (!std::isfinite(grad[k])) return fail(SCP_ENONFINITE, "gradient is not finite");
  return SCP_OK;
}

// --- serving: a closed-system request on the gather engine, in chunks --------
// Workspace: the layout of gc_layout (the adjoint's when the gradient is
// wanted) followed by the compensated state [S][D] float4 between chunks.
// It has stage inputs for one segment; the server lends room for more (see
// gather_serve_buffers).
size_t gather_serve_bytes(const scp_system* sys, int S, int ce, bool grad) {
  GcLayout w;
  if (gc_layout(sys, S, ce, grad, 1, w, nullptr) != SCP_OK) {
    set_error("");
    return 0;
  }
  return w.total + align256((size_t)S * sys->D * sizeof(float4));
}

scp_status gather_serve_prepare(scp_system* sys, int S, int ce, bool grad, void* ws, size_t bytes,
                                const float2* psi0, float2* psiT, const float2* cot, hipStream_t st) {
  GcLayout w;
  GArgs A;
  return gc_prepare(sys, S, ce, grad, 1, static_cast<char*>(ws), bytes, psi0, psiT, cot, true, w, A,
                    st);
}

int gather_serve_nckpt(const scp_system* sys, int ce) { return (sys->n_steps + ce - 1) / ce; }

scp_status gather_serve_info(const scp_system* sys, int S, int ce, bool grad, void* ws,
                             GServeInfo& out) {
  GcLayout w, full;
  GArgs A;
  SCP_TRY(gc_layout(sys, S, ce, grad, 0, full, nullptr));
  SCP_TRY(gc_layout(sys, S, ce, grad, 1, w, &A));
  char* base = static_cast<char*>(ws);
  out.A = base + w.args;
  out.B = base + w.adj;
  out.state = reinterpret_cast<float4*>(base + w.total);
  out.form = g_form(A);
  out.lds_fwd = sizeof(c32) * (3 * (size_t)sys->D + ((3 * (size_t)sys->D) & 1) + 2 * (size_t)A.ntab);
  out.lds_adj = g_adj_lds(sys->d, sys->n_modes, false, A.ntabg, w.nacc);
  out.lds_cos = sizeof(c32) * (2 * (size_t)sys->D + 2 * (size_t)A.ntab);
  if (A.real) {
    out.lds_fwd = out.lds_cos = g_real_lds(sys->d, sys->n_modes, false);
    out.lds_adj = g_real_lds(sys->d, sys->n_modes, true);
  }
  out.nck = w.nck;
  out.seg = reinterpret_cast<float2*>(base + w.seg);
  out.most = full.nseg;
  return SCP_OK;
}

// The request's stage inputs lie at seg from now on (room for as many segments as
// the launches that follow name).  Not while one of its launches is in flight.
scp_status gather_serve_buffers(const GServeInfo& gi, const float2* seg) {
  const GAdj* B = static_cast<const GAdj*>(gi.B);
  HIPCHK(hipMemcpy(const_cast<float2**>(&B->seg), &seg, sizeof(seg), hipMemcpyHostToDevice));
  return SCP_OK;
}

namespace {

template <int d, int N>
hipError_t g_fwd_batched_launch(int form, bool ck, const GItem* items, int n, size_t sh,
                                hipStream_t s) {
  if (sh > 163840) return hipErrorInvalidValue;
  auto run = [&](auto* kernel) {
    (void)g_lds(kernel, sh);
    hipLaunchKernelGGL(kernel, dim3(n), dim3(GShape<d, N, false>::T), sh, s, items);
  };
  if (form == 2)
    return g_real_forward(d, N, ck, items, nullptr, nullptr, n, 0, 0, nullptr, nullptr, s);
  if (form == 1) {
    if (ck) run(g_rk4_batched_kernel<d, N, true, true>);
    else run(g_rk4_batched_kernel<d, N, true, false>);
  } else {
    if (ck) run(g_rk4_batched_kernel<d, N, false, true>);
    else run(g_rk4_batched_kernel<d, N, false, false>);
  }
  return hipGetLastError();
}

template <int d, int N>
hipError_t g_adj_batched_launch(int form, const GItem* items, int n, size_t sh, hipStream_t s) {
  if (sh > 163840) return hipErrorInvalidValue;
  auto run = [&](auto* kernel) {
    (void)g_lds(kernel, sh);
    hipLaunchKernelGGL(kernel, dim3(n), dim3(GShape<d, N, false>::T), sh, s, items);
  };
  if (form == 2) return g_real_segments(d, N, items, nullptr, nullptr, n, 0, s);
  if (form == 1) run(g_adj_batched_kernel<d, N, true>);
  else run(g_adj_batched_kernel<d, N, false>);
  return hipGetLastError();
}

template <int d, int N>
hipError_t g_cos_batched_launch(int form, const GItem* items, int n, size_t sh, hipStream_t s) {
  if (sh > 163840) return hipErrorInvalidValue;
  auto run = [&](auto* kernel) {
    (void)g_lds(kernel, sh);
    hipLaunchKernelGGL(kernel, dim3(n), dim3(GShape<d, N, false>::T), sh, s, items);
  };
  if (form == 2) return g_real_sweep(d, N, items, nullptr, nullptr, n, 0, 0, s);
  if (form == 1) run(g_cos_batched_kernel<d, N, true>);
  else run(g_cos_batched_kernel<d, N, false>);
  return hipGetLastError();
}

}  // namespace

scp_status gather_launch_cos_batched(int d, int N, int form, const GItem* items, int n, size_t lds,
                                     hipStream_t st) {
#define GA_COS_B(dd_, nn_) \
  if (d == dd_ && N == nn_) {                                                  \
    HIPCHK((g_cos_batched_launch<dd_, nn_>(form, items, n, lds, st)));         \
    return SCP_OK;                                                            \
  }
  GA_CLOSED_SHAPES(GA_COS_B)
#undef GA_COS_B
  return fail(SCP_EINVAL, "gather engine: no compiled stepper for this shape");
}

scp_status gather_launch_fwd_batched(int d, int N, int form, bool ck, const GItem* items, int n, size_t lds,
                                     hipStream_t st) {
#define GA_FWD_B(dd_, nn_) \
  if (d == dd_ && N == nn_) {                                                  \
    HIPCHK((g_fwd_batched_launch<dd_, nn_>(form, ck, items, n, lds, st)));          \
    return SCP_OK;                                                            \
  }
  GA_CLOSED_SHAPES(GA_FWD_B)
#undef GA_FWD_B
  return fail(SCP_EINVAL, "gather engine: no compiled stepper for this shape");
}

scp_status gather_launch_adj_batched(int d, int N, int form, const GItem* items, int n, size_t lds,
                                     hipStream_t st) {
#define GA_ADJ_B(dd_, nn_) \
  if (d == dd_ && N == nn_) {                                                  \
    HIPCHK((g_adj_batched_launch<dd_, nn_>(form, items, n, lds, st)));              \
    return SCP_OK;                                                            \
  }
  GA_CLOSED_SHAPES(GA_ADJ_B)
#undef GA_ADJ_B
  return fail(SCP_EINVAL, "gather engine: no compiled stepper for this shape");
}

// The gradient after the last reverse launch (synchronises st).
scp_status gather_serve_gradient(scp_system* sys, int S, int ce, void* ws, std::vector<double>& grad,
                                 hipStream_t st) {
  GcLayout w;
  SCP_TRY(gc_layout(sys, S, ce, true, 1, w, nullptr));
  grad.assign(w.nacc, 0.0);
  return gc_fold(sys, S, static_cast<char*>(ws), w, grad.data(), st);
}

// ---------------------------------------------------------------------------
// average gate fidelity of the channel on the computational subspace
// ---------------------------------------------------------------------------
namespace {

// ov = sum_ab sum_ij conj(T_ia) T_jb rho_ab[r_i, r_j] in FP64 by one
// workgroup in a fixed order.
__global__ void __launch_bounds__(1024) chan_overlap_kernel(const c32* __restrict__ rho, int64_t D,
                                                            int dc, const int64_t* __restrict__ rows,
                                                            const double2* __restrict__ Tm,
                                                            double2* __restrict__ ov) {
  __shared__ double red[2][1024];
  const int64_t n = (int64_t)dc * dc * dc * dc;
  double sr = 0.0, si = 0.0;
  for (int64_t u = threadIdx.x; u < n; u += blockDim.x) {
    const int64_t ab = u / ((int64_t)dc * dc), ij = u - ab * dc * dc;
    const int a = (int)(ab / dc), b = (int)(ab - (int64_t)a * dc);
    const int i = (int)(ij / dc), j = (int)(ij - (int64_t)i * dc);
    const double2 ta = Tm[(size_t)i * dc + a], tb = Tm[(size_t)j * dc + b];
    // w = conj(ta) tb
    const double wr = ta.x * tb.x + ta.y * tb.y, wi = ta.x * tb.y - ta.y * tb.x;
    const c32 v = rho[(size_t)ab * D * D + (size_t)rows[i] * D + rows[j]];
    sr += wr * v.x - wi * v.y;
    si += wr * v.y + wi * v.x;
  }
  red[0][threadIdx.x] = sr;
  red[1][threadIdx.x] = si;
  __syncthreads();
  for (int w = blockDim.x / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      red[0][threadIdx.x] += red[0][threadIdx.x + w];
      red[1][threadIdx.x] += red[1][threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) ov[0] = make_double2(red[0][0], red[1][0]);
}

// cotangent of 1 - F: -T_ia conj(T_jb) / (2 dc (dc + 1)) at (ab, r_i, r_j), zero elsewhere
__global__ void chan_cot_kernel(c32* __restrict__ cot, int64_t D, int dc,
                                const int64_t* __restrict__ rows, const double2* __restrict__ Tm) {
  const int64_t total = (int64_t)dc * dc * D * D;
  const double c = -1.0 / (2.0 * dc * (dc + 1.0));
  for (int64_t u = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; u < total;
       u += (int64_t)gridDim.x * blockDim.x) {
    const int64_t ab = u / (D * D), rem = u - ab * D * D;
    const int64_t R = rem / D, C = rem - R * D;
    const int a = (int)(ab / dc), b = (int)(ab - (int64_t)a * dc);
    int i = -1, j = -1;
    for (int q = 0; q < dc; ++q) {
      if (rows[q] == R) i = q;
      if (rows[q] == C) j = q;
    }
    c32 v;
    v.x = v.y = 0.f;
    if (i >= 0 && j >= 0) {
      const double2 ta = Tm[(size_t)i * dc + a], tb = Tm[(size_t)j * dc + b];
      // ta conj(tb)
      v.x = (float)(c * (ta.x * tb.x + ta.y * tb.y));
      v.y = (float)(c * (ta.y * tb.x - ta.x * tb.y));
    }
    cot[u] = v;
  }
}

}  // namespace

scp_status launch_fidelity_channel(const void* rhoT, int64_t D, int dc, const int64_t* rows,
                                   const void* target, void* ov, void* cot, hipStream_t st) {
  hipLaunchKernelGGL(chan_overlap_kernel, dim3(1), dim3(1024), 0, st, (const c32*)rhoT, D, dc, rows,
                     (const double2*)target, (double2*)ov);
  HIPCHK(hipGetLastError());
  if (cot) {
    const int64_t total = (int64_t)dc * dc * D * D;
    const int blocks = (int)std::min<int64_t>((total + 255) / 256, 4096);
    hipLaunchKernelGGL(chan_cot_kernel, dim3(std::max(1, blocks)), dim3(256), 0, st, (c32*)cot, D,
                       dc, rows, (const double2*)target);
    HIPCHK(hipGetLastError());
  }
  return SCP_OK;
}

}  // namespace scp
