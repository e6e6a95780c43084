// Device building blocks shared by the fused stepper, the applicator and the
// adjoint: register-resident state in a mode layout, LDS layout switches,
// and the per-mode contractions of one term item.
//
// State of one column: D = d^N complex amplitudes.  In layout l a thread
// holds RB = d^NR of them in registers: the digits of the NR "register
// modes" of layout l index the registers (position 0 most significant), the
// digits of the other modes index the thread inside the column.  Element of
// register r of thread t: tb[l](t) + reg_off[l][r] in the natural (mode-0
// slowest) order.  A contraction on a register mode is local to the thread;
// moving a vector to another layout goes through LDS in natural order.
#pragma once

#include <utility>
#include <type_traits>

#include "internal.h"

namespace scp {

// Uniform read-only data (the plan, the stage tables, drive coefficients) is
// read through the constant address space: the compiler may then keep it in
// scalar registers and fetch it with scalar loads instead of per-lane loads.
// Nothing writes these buffers while a kernel runs.
template <typename T>
using kptr = const __attribute__((address_space(4))) T*;
template <typename T>
__device__ __forceinline__ kptr<T> kconst(const T* p) {
  return (kptr<T>)(uintptr_t)p;
}
// A value known to be the same in every lane, as a scalar.
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ float unif(float v) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

// Evaluation of a kernel instance (template parameter EV): bit 0, the real
// frame; bit 1, parity: every operator, pair operator and derivative operator
// connects levels of unlike parity only, so its entries (a, b) with a + b even
// are zero and their multiply-adds, loads and sensitivities are left out.
constexpr int EV_REAL = 1, EV_PARITY = 2;
constexpr bool ev_real(int ev) { return (ev & EV_REAL) != 0; }
constexpr bool ev_parity(int ev) { return (ev & EV_PARITY) != 0; }
// Entry (a, b) of an operator may be non-zero.
template <bool PAR>
__device__ __forceinline__ constexpr bool entry(int a, int b) {
  return !PAR || ((a + b) & 1) != 0;
}

template <int d, int NR>
struct Cfg {
  static constexpr int RB = (NR == 1) ? d : (NR == 2) ? d * d : (NR == 3) ? d * d * d
                          : (NR == 4) ? d * d * d * d : d * d * d * d * d;
  static constexpr int stride(int p) {
    int s = 1;
    for (int q = p + 1; q < NR; ++q) s *= d;
    return s;
  }
  static constexpr int digit(int r, int p) { return (r / stride(p)) % d; }
};

// Vector of RB complex amplitudes in registers.
template <int RB>
struct Vec {
  float re[RB];
  float im[RB];
};

// Plain complex storage types for device memory (no vector-type punning).
struct alignas(8) c32 {
  float x, y;
};
struct alignas(16) c32x2 {   // compensated pair (hi.re, hi.im, lo.re, lo.im)
  float x, y, z, w;
};

// ----------------------------------------------------------------------------
// layout switches through LDS
// ----------------------------------------------------------------------------
// Natural-order offset of register r: sum over positions p of digit_p(r) *
// stride of the mode at p (the strides are per layout, uniform).
template <int d, int NR>
struct RegOff {
  int s[NR];
  __device__ __forceinline__ int operator()(int r) const {
    int o = 0;
#pragma unroll
    for (int p = 0; p < NR; ++p) {
      int q = r;
      for (int k = p + 1; k < NR; ++k) q /= d;
      o += (q % d) * s[p];
    }
    return o;
  }
};

template <int d, int NR>
__device__ __forceinline__ RegOff<d, NR> reg_off_of(kptr<Plan> P, int l) {
  RegOff<d, NR> R;
#pragma unroll
  for (int p = 0; p < NR; ++p) R.s[p] = uni(P->reg_stride[l][p]);
  return R;
}

template <int d, int NR, int RB>
__device__ __forceinline__ void lds_put(c32* lds, int base, const RegOff<d, NR>& R,
                                        const Vec<RB>& v) {
#pragma unroll
  for (int r = 0; r < RB; ++r) {
    c32 t;
    t.x = v.re[r];
    t.y = v.im[r];
    lds[base + R(r)] = t;
  }
}

template <int d, int NR, int RB>
__device__ __forceinline__ void lds_get(const c32* lds, int base, const RegOff<d, NR>& R,
                                        Vec<RB>& v) {
#pragma unroll
  for (int r = 0; r < RB; ++r) {
    c32 t = lds[base + R(r)];
    v.re[r] = t.x;
    v.im[r] = t.y;
  }
}

// ----------------------------------------------------------------------------
// operators (uniform, read through the scalar path)
// ----------------------------------------------------------------------------
template <int d>
struct Op {
  float re[d * d];
  float im[d * d];
};

template <int d, bool PAR = false>
__device__ __forceinline__ void load_op(kptr<c32> p, Op<d>& o) {
#pragma unroll
  for (int i = 0; i < d * d; ++i) {
    if (!entry<PAR>(i / d, i % d)) continue;
    o.re[i] = p[i].x;
    o.im[i] = p[i].y;
  }
}

// Compile-time loop (guaranteed expansion; register arrays stay in VGPRs).
template <typename F, int... Is>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, Is...>) {
  (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// Register index of the b-th fiber base (digit 0 at the excluded positions X1, X2).
template <int d, int NR, int X1, int X2>
constexpr int fiber_base(int b) {
  int r = 0;
  for (int p = NR - 1; p >= 0; --p) {
    if (p == X1 || p == X2) continue;
    r += (b % d) * Cfg<d, NR>::stride(p);
    b /= d;
  }
  return r;
}

// out += (O at position P) in, for all fibers along P
template <int d, int NR, int P, bool PAR = false, int RB>
__device__ __forceinline__ void contract_acc(const Op<d>& O, const Vec<RB>& in, Vec<RB>& out) {
  using C = Cfg<d, NR>;
  constexpr int st = C::stride(P);
  static_for<RB / d>([&](auto B) {
    constexpr int r0 = fiber_base<d, NR, P, -1>(decltype(B)::value);
#pragma unroll
    for (int a = 0; a < d; ++a) {
      float sr = out.re[r0 + a * st], si = out.im[r0 + a * st];
#pragma unroll
      for (int b = 0; b < d; ++b) {
        if (!entry<PAR>(a, b)) continue;
        const float orr = O.re[a * d + b], oi = O.im[a * d + b];
        const float xr = in.re[r0 + b * st], xi = in.im[r0 + b * st];
        sr = fmaf(orr, xr, sr);
        sr = fmaf(-oi, xi, sr);
        si = fmaf(orr, xi, si);
        si = fmaf(oi, xr, si);
      }
      out.re[r0 + a * st] = sr;
      out.im[r0 + a * st] = si;
    }
  });
}

// Group item with one partner: out += W(at PJ) O(at PI) in + c O(at PI) in,
// evaluated block by block over the (PI, PJ) plane to keep temporaries small.
template <int d, int NR, int PI, int PJ, bool PAR, int RB>
__device__ __forceinline__ void group_pair(const Op<d>& O, const Op<d>& W, float c,
                                           const Vec<RB>& in, Vec<RB>& out) {
  using C = Cfg<d, NR>;
  constexpr int si_ = C::stride(PI);
  constexpr int sj_ = C::stride(PJ);
  static_for<RB / (d * d)>([&](auto B) {
    constexpr int r0 = fiber_base<d, NR, PI, PJ>(decltype(B)::value);
    float tr[d][d], ti[d][d];   // T[a_i][a_j] = sum_b O[a_i][b] in[b, a_j]
#pragma unroll
    for (int aj = 0; aj < d; ++aj)
#pragma unroll
      for (int ai = 0; ai < d; ++ai) {
        float sr = 0.f, sim = 0.f;
#pragma unroll
        for (int b = 0; b < d; ++b) {
          if (!entry<PAR>(ai, b)) continue;
          const float orr = O.re[ai * d + b], oi = O.im[ai * d + b];
          const float xr = in.re[r0 + b * si_ + aj * sj_], xi = in.im[r0 + b * si_ + aj * sj_];
          sr = fmaf(orr, xr, sr);
          sr = fmaf(-oi, xi, sr);
          sim = fmaf(orr, xi, sim);
          sim = fmaf(oi, xr, sim);
        }
        tr[ai][aj] = sr;
        ti[ai][aj] = sim;
      }
#pragma unroll
    for (int ai = 0; ai < d; ++ai)
#pragma unroll
      for (int aj = 0; aj < d; ++aj) {
        // out + c T + W T, accumulated in place
        float sr = fmaf(c, tr[ai][aj], out.re[r0 + ai * si_ + aj * sj_]);
        float sim = fmaf(c, ti[ai][aj], out.im[r0 + ai * si_ + aj * sj_]);
#pragma unroll
        for (int b = 0; b < d; ++b) {
          if (!entry<PAR>(aj, b)) continue;
          const float wr = W.re[aj * d + b], wi = W.im[aj * d + b];
          sr = fmaf(wr, tr[ai][b], sr);
          sr = fmaf(-wi, ti[ai][b], sr);
          sim = fmaf(wr, ti[ai][b], sim);
          sim = fmaf(wi, tr[ai][b], sim);
        }
        out.re[r0 + ai * si_ + aj * sj_] = sr;
        out.im[r0 + ai * si_ + aj * sj_] = sim;
      }
  });
}

template <int d, int NR, int P, int RB>
__device__ __forceinline__ void diag_acc(kptr<float> dl, const Vec<RB>& in,
                                         Vec<RB>& out) {
  using C = Cfg<d, NR>;
#pragma unroll
  for (int r = 0; r < RB; ++r) {
    const float v = dl[C::digit(r, P)];
    out.re[r] = fmaf(v, in.re[r], out.re[r]);
    out.im[r] = fmaf(v, in.im[r], out.im[r]);
  }
}

// Drive coefficient of a term (cidx < 0: none).  The index is clamped so the
// (uniform) load never leaves the table.
__device__ __forceinline__ float coef(kptr<float> cq, int cidx) {
  const float v = cq[cidx > 0 ? cidx : 0];
  return cidx >= 0 ? v : 0.f;
}

// Apply all terms of layout l: out += V_l(t) in.  Positions are compile-time:
// pair terms at (p, p+1), MP of them per position pair; drive-only and
// diagonal terms behind one per-layout flag each.
template <int d, int NR, int MP, bool PAR, int RB>
__device__ __forceinline__ void apply_layout(kptr<Plan> P, int l,
                                             kptr<c32> ops,
                                             kptr<float> cq, const Vec<RB>& in,
                                             Vec<RB>& out) {
  constexpr int dd = d * d;
  static_for<NR - 1>([&](auto Pp) {
    constexpr int p = decltype(Pp)::value;
    static_for<MP>([&](auto Mm) {
      constexpr int m = decltype(Mm)::value;
      const auto& C = P->cpair[l][p][m];
      Op<d> O, W;
      load_op<d, PAR>(ops + uni(C.slot) * dd, O);
      load_op<d, PAR>(ops + uni(P->off_pair + C.pair * dd), W);
      group_pair<d, NR, p, p + 1, PAR>(O, W, coef(cq, uni(C.cidx)), in, out);
    });
  });
  if (uni(P->has_single[l])) {
    static_for<NR>([&](auto Pp) {
      constexpr int p = decltype(Pp)::value;
      const auto& C1 = P->csingle[l][p];
      Op<d> O;
      load_op<d, PAR>(ops + uni(C1.slot) * dd, O);
      const float c = coef(cq, uni(C1.cidx));
#pragma unroll
      for (int i = 0; i < dd; ++i) {
        if (!entry<PAR>(i / d, i % d)) continue;
        O.re[i] *= c;
        O.im[i] *= c;
      }
      contract_acc<d, NR, p, PAR>(O, in, out);
    });
  }
  if (uni(P->has_diag[l])) {
    static_for<NR>([&](auto Pp) {
      constexpr int p = decltype(Pp)::value;
      diag_acc<d, NR, p>(P->delta[uni(P->cdiag[l][p])], in, out);
    });
  }
}

// ----------------------------------------------------------------------------
// real frame: every operator real.  With D(t) = exp(i H_f t) (diagonal) the
// interaction-picture generator is D(t) R D(t)^dag, R the sum of the
// un-rotated terms, so k = D R (D^dag y): the contractions take real d x d
// operators (two FMAs per complex amplitude and operator entry instead of four).
// ----------------------------------------------------------------------------
template <int d>
struct ROp {
  float v[d * d];
};

template <int d, bool PAR = false>
__device__ __forceinline__ void load_rop(kptr<float> p, ROp<d>& o) {
#pragma unroll
  for (int i = 0; i < d * d; ++i)
    if (entry<PAR>(i / d, i % d)) o.v[i] = p[i];
}

// out += (O at position P) in, O real
template <int d, int NR, int P, bool PAR = false, int RB>
__device__ __forceinline__ void contract_acc_real(const ROp<d>& O, const Vec<RB>& in, Vec<RB>& out) {
  using C = Cfg<d, NR>;
  constexpr int st = C::stride(P);
  static_for<RB / d>([&](auto B) {
    constexpr int r0 = fiber_base<d, NR, P, -1>(decltype(B)::value);
#pragma unroll
    for (int a = 0; a < d; ++a) {
      float sr = out.re[r0 + a * st], si = out.im[r0 + a * st];
#pragma unroll
      for (int b = 0; b < d; ++b) {
        if (!entry<PAR>(a, b)) continue;
        const float o = O.v[a * d + b];
        sr = fmaf(o, in.re[r0 + b * st], sr);
        si = fmaf(o, in.im[r0 + b * st], si);
      }
      out.re[r0 + a * st] = sr;
      out.im[r0 + a * st] = si;
    }
  });
}

// out += W(at PJ) O(at PI) in + c O(at PI) in, O and W real
template <int d, int NR, int PI, int PJ, bool PAR, int RB>
__device__ __forceinline__ void group_pair_real(const ROp<d>& O, const ROp<d>& W, float c,
                                                const Vec<RB>& in, Vec<RB>& out) {
  using C = Cfg<d, NR>;
  constexpr int si_ = C::stride(PI);
  constexpr int sj_ = C::stride(PJ);
  static_for<RB / (d * d)>([&](auto B) {
    constexpr int r0 = fiber_base<d, NR, PI, PJ>(decltype(B)::value);
    float tr[d][d], ti[d][d];   // T[a_i][a_j] = sum_b O[a_i][b] in[b, a_j]
#pragma unroll
    for (int aj = 0; aj < d; ++aj)
#pragma unroll
      for (int ai = 0; ai < d; ++ai) {
        float sr = 0.f, sim = 0.f;
#pragma unroll
        for (int b = 0; b < d; ++b) {
          if (!entry<PAR>(ai, b)) continue;
          const float o = O.v[ai * d + b];
          sr = fmaf(o, in.re[r0 + b * si_ + aj * sj_], sr);
          sim = fmaf(o, in.im[r0 + b * si_ + aj * sj_], sim);
        }
        tr[ai][aj] = sr;
        ti[ai][aj] = sim;
      }
#pragma unroll
    for (int ai = 0; ai < d; ++ai)
#pragma unroll
      for (int aj = 0; aj < d; ++aj) {
        float sr = fmaf(c, tr[ai][aj], out.re[r0 + ai * si_ + aj * sj_]);
        float sim = fmaf(c, ti[ai][aj], out.im[r0 + ai * si_ + aj * sj_]);
#pragma unroll
        for (int b = 0; b < d; ++b) {
          if (!entry<PAR>(aj, b)) continue;
          const float w = W.v[aj * d + b];
          sr = fmaf(w, tr[ai][b], sr);
          sim = fmaf(w, ti[ai][b], sim);
        }
        out.re[r0 + ai * si_ + aj * sj_] = sr;
        out.im[r0 + ai * si_ + aj * sj_] = sim;
      }
  });
}

// apply_layout with the un-rotated (real) operators
template <int d, int NR, int MP, bool PAR, int RB>
__device__ __forceinline__ void apply_layout_real(kptr<Plan> P, int l, kptr<float> ops,
                                                  kptr<float> cq, const Vec<RB>& in,
                                                  Vec<RB>& out) {
  constexpr int dd = d * d;
  static_for<NR - 1>([&](auto Pp) {
    constexpr int p = decltype(Pp)::value;
    static_for<MP>([&](auto Mm) {
      constexpr int m = decltype(Mm)::value;
      const auto& C = P->cpair[l][p][m];
      ROp<d> O, W;
      load_rop<d, PAR>(ops + uni(C.slot) * dd, O);
      load_rop<d, PAR>(ops + uni(P->off_pair + C.pair * dd), W);
      group_pair_real<d, NR, p, p + 1, PAR>(O, W, coef(cq, uni(C.cidx)), in, out);
    });
  });
  if (uni(P->has_single[l])) {
    static_for<NR>([&](auto Pp) {
      constexpr int p = decltype(Pp)::value;
      const auto& C1 = P->csingle[l][p];
      ROp<d> O;
      load_rop<d, PAR>(ops + uni(C1.slot) * dd, O);
      const float c = coef(cq, uni(C1.cidx));
#pragma unroll
      for (int i = 0; i < dd; ++i)
        if (entry<PAR>(i / d, i % d)) O.v[i] *= c;
      contract_acc_real<d, NR, p, PAR>(O, in, out);
    });
  }
  if (uni(P->has_diag[l])) {
    static_for<NR>([&](auto Pp) {
      constexpr int p = decltype(Pp)::value;
      diag_acc<d, NR, p>(P->delta[uni(P->cdiag[l][p])], in, out);
    });
  }
}

// Frame phase exp(i f t) of this thread's thread-position digits in the base
// layout (row: the thread-position part of a half-step's phase row; entry
// k*d + a is the phase of level a of the mode at thread position k).
template <int d>
__device__ __forceinline__ c32 thread_phase(kptr<c32> row, int NT, int tc) {
  float pr = 1.f, pi = 0.f;
  int t = tc;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    if (k < NT) {
      const int q = t / d;
      const int a = t - q * d;
      t = q;
      float vr = row[k * d].x, vi = row[k * d].y;
#pragma unroll
      for (int b = 1; b < d; ++b) {
        const float ur = row[k * d + b].x, ui = row[k * d + b].y;
        vr = a == b ? ur : vr;
        vi = a == b ? ui : vi;
      }
      const float nr = pr * vr - pi * vi;
      const float ni = fmaf(pr, vi, pi * vr);
      pr = nr;
      pi = ni;
    }
  }
  c32 o;
  o.x = pr;
  o.y = pi;
  return o;
}

// Eight phases of a row (rows are 64-byte aligned, so the register phases
// arrive with wide scalar loads).
struct alignas(64) c32x8 {
  float v[16];
};

// The phase of base-layout register r: thread part pt times the register
// part of the row (uniform); CONJ: its conjugate.
template <bool CONJ>
__device__ __forceinline__ c32 elem_phase(c32 pt, kptr<c32x8> preg, int r) {
  const float gr = preg[r / 8].v[2 * (r % 8)], gi = preg[r / 8].v[2 * (r % 8) + 1];
  c32 e;
  e.x = pt.x * gr - pt.y * gi;
  e.y = fmaf(pt.x, gi, pt.y * gr);
  if (CONJ) e.y = -e.y;
  return e;
}

}  // namespace scp

namespace scp {

// Natural-order offset of this thread's first element in layout l: the digits
// of the thread index (digit 0 fastest) times the strides of the thread modes.
// At most 8 thread modes (d^(thread modes) <= 256 threads per column).
template <int d>
__device__ __forceinline__ int thread_base(kptr<Plan> P, int l, int tc) {
  const int NT = uni(P->NT);
  int b = 0, t = tc;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int st = uni(P->tstride[l][k]);
    if (k < NT) {
      const int q = t / d;
      b += (t - q * d) * st;
      t = q;
    }
  }
  return b;
}

// k = V(t) y for one stage.  The stage input y is in natural order in LDS
// region iy (regions are rstride elements apart; cbase selects the column)
// and every layout reads its elements from there.  k accumulates layout by
// layout in registers and moves to the next layout through region ka, then
// kb, then ka, ... with one barrier per move: a region is written only after
// a barrier that follows its last reads (the other k region was last read
// before the previous barrier; y's region is never written during a stage).
// k leaves in the base layout (L-1).  On return ka is the region that the
// last move did not use, which may be written next without a barrier.
template <int d, int NR, int MP, int RB, int EV = 0>
__device__ __forceinline__ void stage_apply(kptr<Plan> P, c32* lds, int cbase, int rstride,
                                            bool lds_ok, int tc, kptr<c32> ops, kptr<float> rops,
                                            kptr<float> cq, int iy, int& ka, int& kb, Vec<RB>& k) {
  const int L = uni(P->L);
  const c32* ybuf = lds + iy * rstride + cbase;
#pragma unroll
  for (int r = 0; r < RB; ++r) {
    k.re[r] = 0.f;
    k.im[r] = 0.f;
  }
  for (int lv = 0; lv < L; ++lv) {
    const int l = uni(lv);
    if (l > 0) {
      c32* kbuf = lds + ka * rstride + cbase;
      if (lds_ok) lds_put<d, NR, RB>(kbuf, thread_base<d>(P, l - 1, tc), reg_off_of<d, NR>(P, l - 1), k);
      __syncthreads();
      if (lds_ok) lds_get<d, NR, RB>(kbuf, thread_base<d>(P, l, tc), reg_off_of<d, NR>(P, l), k);
      const int t = ka;
      ka = kb;
      kb = t;
    }
    Vec<RB> y;
    if (lds_ok) {
      lds_get<d, NR, RB>(ybuf, thread_base<d>(P, l, tc), reg_off_of<d, NR>(P, l), y);
    } else {
#pragma unroll
      for (int r = 0; r < RB; ++r) y.re[r] = y.im[r] = 0.f;
    }
    if constexpr (ev_real(EV))
      apply_layout_real<d, NR, MP, ev_parity(EV), RB>(P, l, rops, cq, y, k);
    else
      apply_layout<d, NR, MP, ev_parity(EV), RB>(P, l, ops, cq, y, k);
  }
}

__device__ __forceinline__ int stage_q(int n, int s) { return 2 * n + (s == 0 ? 0 : (s == 3 ? 2 : 1)); }
__device__ __forceinline__ int stage_c(int n, int s) { return 3 * n + (s == 0 ? 0 : (s == 3 ? 2 : 1)); }

// Two-sum compensated x_hi + x_lo += dx (x_lo kept with |x_lo| <= ulp(x_hi)/2).
__device__ __forceinline__ void comp_add(float& hi, float& lo, float dx) {
  const float sx = hi + dx;
  const float bp = sx - hi;
  const float err = (hi - (sx - bp)) + (dx - bp);
  const float l2 = lo + err;
  const float s2 = sx + l2;
  lo = l2 - (s2 - sx);
  hi = s2;
}

// One classical RK4 step n on psi = hi + lo.  hi, lo and the RK accumulator
// live in registers (base layout).  The stage
// inputs y_s are written to LDS in natural order (region ka, which is free,
// then one barrier) and read there by every layout of the stage; iy, ka, kb
// are the LDS region indices carried from step to step (start with 0, 1, 2).
// y_s are formed from hi alone (the stage increments are O(h |V|) of psi, so
// the dropped lo is below their rounding).  If ystore != nullptr the four
// stage inputs are also written there in natural order (ystore is the
// column's base; stride ystride between stages) for the adjoint.
// Real frame (EV): LDS receives D(t_s)^dag y_s, the layouts apply the
// un-rotated real operators (table block 0), and k_s = D(t_s) (R y'_s); the
// phases come from the half-step rows of ph.  ystore still receives y_s.
template <int d, int NR, int MP, int RB, int EV = 0>
__device__ __forceinline__ void rk4_step(kptr<Plan> P, c32* lds, int cbase, int rstride,
                                         bool lds_ok, bool active, int tc, int TPC,
                                         kptr<c32> optab, kptr<float> rops, kptr<float> ctab,
                                         kptr<c32> ph, int n,
                                         Vec<RB>& hi, Vec<RB>& lo, int& iy, int& ka, int& kb,
                                         c32* __restrict__ ystore, size_t ystride,
                                         int& pq, c32& pt_q) {
  constexpr bool RF = ev_real(EV);
  const float h = P->h;
  const int ng = uni(P->ngroups);
  const int bq = uni(P->block_q);
  const int L = uni(P->L);
  const int NT = uni(P->NT);
  const int prow = RF ? uni(P->ph_row) : 0;
  const int pthr = RF ? uni(P->ph_thr) : 0;
  const int tbB = thread_base<d>(P, L - 1, tc);
  const RegOff<d, NR> RB_ = reg_off_of<d, NR>(P, L - 1);
  // the thread part of the frame phase of half-step row q, recomputed only
  // when the row changes (y_s and k_s share a row, stages 1 and 2 share one,
  // and a step's last row is the next step's first); pq < 0: none cached
  auto tphase = [&](int q) -> c32 {
    if (q != pq) {
      pt_q = thread_phase<d>(ph + (size_t)q * prow + pthr, NT, tc);
      pq = q;
    }
    return pt_q;
  };
  // y_0 = hi
  {
    c32* yb = lds + ka * rstride + cbase + tbB;
    c32* ys = ystore != nullptr ? ystore + tbB : nullptr;
    kptr<c32> row = ph + (size_t)stage_q(n, 0) * prow;
    const c32 pt = RF ? tphase(stage_q(n, 0)) : c32{1.f, 0.f};
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      c32 v;
      v.x = hi.re[r];
      v.y = hi.im[r];
      if (ys != nullptr && active) ys[RB_(r)] = v;
      if (RF) {
        const c32 e = elem_phase<true>(pt, (kptr<c32x8>)row, r);
        const c32 u = v;
        v.x = e.x * u.x - e.y * u.y;
        v.y = fmaf(e.x, u.y, e.y * u.x);
      }
      if (lds_ok) yb[RB_(r)] = v;
    }
    __syncthreads();
    const int t = iy;
    iy = ka;
    ka = t;
  }
  Vec<RB> acc, k;
  // The next stage's rotated operators (real frame: its phase row) are read
  // with scalar loads; one stage ahead, the first threads of each column touch
  // every 64-byte line of that block with a vector load, so those scalar reads
  // find the lines in L2.
  const int pf_lines = RF ? (prow * (int)sizeof(c32) + 63) / 64
                          : (uni(P->off_dslot) * (int)sizeof(c32) + 63) / 64;
  const kptr<c32> pf_base = RF ? ph : optab;
  const int pf_stride = RF ? prow : bq;
  float pf_sink = 0.f;
#pragma unroll 1
  for (int sv = 0; sv < 4; ++sv) {
    const int s = uni(sv);
    auto ops = optab + (RF ? 0 : (size_t)stage_q(n, s) * bq);
    auto cq = ctab + (size_t)stage_c(n, s) * ng;
    float pf = 0.f;
    if (tc < pf_lines) {
      const int qn = s < 3 ? stage_q(n, s + 1) : stage_q(n + 1, 0);   // <= 2 N
      pf = ((const float*)(uintptr_t)(pf_base + (size_t)qn * pf_stride))[tc * 16];
    }
    stage_apply<d, NR, MP, RB, EV>(P, lds, cbase, rstride, lds_ok, tc, ops, rops, cq, iy, ka, kb,
                                   k);
    pf_sink += pf;
    if (RF) {
      // back to the interaction picture: k <- D(t_s) k
      kptr<c32> row = ph + (size_t)stage_q(n, s) * prow;
      const c32 pt = tphase(stage_q(n, s));
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        const c32 e = elem_phase<false>(pt, (kptr<c32x8>)row, r);
        const float xr = k.re[r], xi = k.im[r];
        k.re[r] = e.x * xr - e.y * xi;
        k.im[r] = fmaf(e.x, xi, e.y * xr);
      }
    }
    // k_s = -i V y;  acc (+)= w_s k_s;  y_{s+1} = hi + c_{s+1} h k_s
    const float w = (s == 0 || s == 3) ? 1.f : 2.f;
    const float ch = (s == 2) ? h : 0.5f * h;
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      const float kr = k.im[r], ki = -k.re[r];
      if (s == 0) {
        acc.re[r] = kr;
        acc.im[r] = ki;
      } else {
        acc.re[r] = fmaf(w, kr, acc.re[r]);
        acc.im[r] = fmaf(w, ki, acc.im[r]);
      }
      k.re[r] = fmaf(ch, kr, hi.re[r]);   // k now holds y_{s+1}
      k.im[r] = fmaf(ch, ki, hi.im[r]);
    }
    if (s < 3) {
      c32* yb = lds + ka * rstride + cbase + tbB;
      c32* ys = ystore != nullptr ? ystore + (size_t)(s + 1) * ystride + tbB : nullptr;
      kptr<c32> row = ph + (size_t)stage_q(n, s + 1) * prow;
      const c32 pt = RF ? tphase(stage_q(n, s + 1)) : c32{1.f, 0.f};
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        c32 v;
        v.x = k.re[r];
        v.y = k.im[r];
        if (ys != nullptr && active) ys[RB_(r)] = v;
        if (RF) {
          const c32 e = elem_phase<true>(pt, (kptr<c32x8>)row, r);
          const c32 u = v;
          v.x = e.x * u.x - e.y * u.y;
          v.y = fmaf(e.x, u.y, e.y * u.x);
        }
        if (lds_ok) yb[RB_(r)] = v;
      }
      __syncthreads();
      const int t = iy;
      iy = ka;
      ka = t;
    }
  }
  // keeps the prefetch loads alive; the sum of table values is never this NaN pattern
  if (__float_as_uint(pf_sink) == 0xffffffffu && n < 0) lo.re[0] += pf_sink;
  // psi <- psi + h/6 acc, compensated
  const float h6 = h * (1.0f / 6.0f);
#pragma unroll
  for (int r = 0; r < RB; ++r) {
    comp_add(hi.re[r], lo.re[r], h6 * acc.re[r]);
    comp_add(hi.im[r], lo.im[r], h6 * acc.im[r]);
  }
}

}  // namespace scp
