// What the gather engine's sources share: the device description of a
// propagation, the geometry of a column, and the wave sum.
#pragma once

#include "internal.h"
#include "kernel_common.h"

namespace scp {

constexpr int GA_MAXM = 10;      // modes (three-bit digits, 2N (open) or N in one word)
constexpr int GA_MAXDM = 10;     // driven modes
constexpr int GA_MAXPR = 10;     // coupled mode pairs
constexpr int GA_MAXC = 4;       // operators summed into one table entry
constexpr int GA_MAXTAB = 4096;  // complex entries of a stage table
constexpr int GA_PRE = 4;        // table entries each thread prefetches per stage
constexpr int GA_MAXSL = 16;     // slots in a gradient table
constexpr int GA_MAXDS = 10;     // distinct drive slots (gradient)
constexpr int GA_MAXDR = 16;     // drives (gradient)
constexpr int GA_MAXCP = 16;     // couplings (gradient)
constexpr int GA_MAXME = 24;     // coupling ends (closed-system gradient)
// per-wave partial sums of one stage: drive slots | 3 per mode | couplings
constexpr int GA_NV = GA_MAXDS + 3 * GA_MAXM + GA_MAXCP;

// Static description of one gather-engine propagation (device copy in the
// workspace, read through the scalar path where uniform).
struct GArgs {
  const float2* optab;   // [2N+1][block_q] rotated slot operators of the system
  const float* ctab;     // [3N][ngroups] drive coefficients
  const float2* jtab;    // [2N+1][N][d*d] unit-rate relaxation band (open systems)
  const float2* gtab;    // [3N][ntab] stage tables (built by gtab_kernel)
  const float2* x0;      // [S][L] input columns
  float2* xT;            // [S][L] output columns
  int block_q, ngroups, nsteps, S;
  float h;
  int ndm, npr, ntab, has_jump, off_p, off_j;
  int par;    // operators connect levels of unlike parity only (see Nb)
  int nn;     // entries of an operator row
  int prow;   // stride of a pair-operator row: nn^2 rounded up to even
  int orow;   // stride of a driven-mode operator row: nn rounded up to even
  int srow;   // stride of a slot-operator row (gradient)
  int mrow;   // stride of a row of a mode's derivative operator (gradient)
  int kst[GA_MAXM], bst[GA_MAXM];                    // strides of ket / bra digits in a column
  int dm_mode[GA_MAXDM], dm_n[GA_MAXDM];
  int dm_slot[GA_MAXDM][GA_MAXC], dm_cidx[GA_MAXDM][GA_MAXC];
  int pr_i[GA_MAXPR], pr_j[GA_MAXPR], pr_n[GA_MAXPR];
  int pr_si[GA_MAXPR][GA_MAXC], pr_sj[GA_MAXPR][GA_MAXC];
  float pr_g[GA_MAXPR][GA_MAXC];
  float g1[GA_MAXM], gp[GA_MAXM];
  float delta[GA_MAXM][8];
  // gradient (open systems): the table gains the rotated slot operators and
  // the unit-rate relaxation bands
  int grad, ntabg, off_s, off_u, nsl;
  int sl_slot[GA_MAXSL];                             // system slot of each table slot
  int nds, ds_sl[GA_MAXDS], ds_mode[GA_MAXDS];       // distinct drive slots
  int ndr, dr_ds[GA_MAXDR], dr_par0[GA_MAXDR], dr_npar[GA_MAXDR];
  int ncp, cp_i[GA_MAXCP], cp_j[GA_MAXCP], cp_si[GA_MAXCP], cp_sj[GA_MAXCP];
  // gradient (closed systems, grad = 2): the table gains the rotated slot
  // operators, per mode and device parameter the one-mode derivative operator
  // (sum_k c_k dO_k + d delta), and the derivative slot operators
  int off_m, off_d, off_dslot;
  int mdm[GA_MAXM];                                  // driven-mode index of a mode (-1: none)
  float deps[GA_MAXM][3][8];                         // d delta / d(EJ, EC, EL)
  float cp_g[GA_MAXCP];
  // coupling ends grouped by mode and own table slot: me_beg[m] .. me_beg[m+1]
  // packed (coupling | own slot << 5 | partner slot << 10 | partner mode << 15 |
  // first side << 20 | last of its own-slot group << 21)
  int me_beg[GA_MAXM + 1];
  int me[GA_MAXME];
  // real form (gather_real.hip, open_real.hip): frame phases [2N+1][L], static rows, the coupled
  // neighbours (bit p: modes p, p + 1; bit N - 1: 0, N - 1), the driven modes
  // and their coefficient columns
  const float2* ph;
  const float* rt;
  const float* rc;    // drive coefficients [3N][N], scaled (see build_gather_rows)
  double kappa;       // h / (6 float(h / 6)), folded into the rows and rc
  int real, pmask, dmask;
  // real form, gradient: per neighbour pair its couplings (operator of each
  // mode, signed strength, sign of the product of two imaginary operators,
  // index), per driven mode its operator and drive slot
  int rp_n[GA_MAXM], rp_u[GA_MAXM][2], rp_c[GA_MAXM][2], rd_u[GA_MAXM], rd_k[GA_MAXM];
  // 1 / the operator's largest entry (that of its static row), 1 / the scale of rc
  float rp_g[GA_MAXM][2], rp_s[GA_MAXM][2], rd_s[GA_MAXM], rd_c[GA_MAXM];
};

// Checkpoints, costate and gradient buffers of an adjoint.
struct GAdj {
  float4* ck;            // [S][nck][L] (hi re, hi im, lo re, lo im) at steps g * ce
  const float2* cot;     // [S][L] cotangent of the final columns
  float2* seg;           // stage inputs, [ce][4][L] per column (open) or per slot (closed)
  const double* dctab;   // [3N][npulse] dc/dpar
  double* part;          // open, complex rows: [S][nacc] gradient partial sums
  float4* lam;           // costate (hi, lo): open [S][L] between reverse walks,
                         // closed [S][nck][L] at the end of every segment
  double* gs;            // closed, and the open real form: [S][N][gw] sums of
                         // every step (see g_fold_kernel)
  int ce, nck, npulse, nacc, gw;
};

constexpr int cpow(int b, int e) { return e == 0 ? 1 : b * cpow(b, e - 1); }

// Geometry of one column: N modes of dimension d; a state (L = D) or a
// vectorised density matrix (L = D^2).
template <int d, int N, bool OPEN>
struct GShape {
  static constexpr int D = cpow(d, N);
  static constexpr int L = OPEN ? D * D : D;
  static constexpr int T = L >= 1024 ? 1024 : ((L + 63) / 64) * 64;   // threads
  static constexpr int E = (L + T - 1) / T;                           // elements per thread
  static constexpr int st(int m) { return cpow(d, N - 1 - m); }       // stride in A or B
};

// The levels along one mode that an operator row connects to level a: all d of
// them or, where every operator is odd (PAR), those of the other parity: at
// most (d + 1) / 2 entries.  With d odd an even level has one neighbour fewer;
// its last entry repeats the first neighbour with a zero coefficient, so the
// gather stays inside the column.  A pair term gathers 4 (d = 3, 4) or 9
// (d = 5) neighbours instead of d^2, with as many table entries.  Measured:
// 4-fluxonium chain (d = 5, 16 columns) forward 11.8 -> 8.4 us per step, open
// 4-fluxonium chain (d = 3, 256 matrices) forward + gradient 583 -> 426.
template <int d, bool PAR>
struct Nb {
  static constexpr int n = PAR ? (d + 1) / 2 : d;
  static constexpr int orow = n + (n & 1);
  static constexpr int prow = n * n + ((n * n) & 1);
  static constexpr int srow = PAR ? orow : d;
  static constexpr int mrow = PAR ? (n + 1) + ((n + 1) & 1) : d;
  // offset of the first entry's element from the row's own (digit a, stride st),
  // and of entry k's from that (uniform but for the padding)
  static __device__ __forceinline__ int first(int a, int st) {
    return PAR ? (((a & 1) ^ 1) - a) * st : -a * st;
  }
  static __device__ __forceinline__ int step(int k, int a, int st) {
    if (!PAR) return k * st;
    return (d & 1) && k == n - 1 && !(a & 1) ? 0 : 2 * k * st;
  }
};
// Level of entry k of row a (-1: padding), as Nb<d, par> has it.
__host__ __device__ inline int nb_level(int d, int par, int k, int a) {
  const int b = par ? ((a & 1) ^ 1) + 2 * k : k;
  return b < d ? b : -1;
}

__device__ __forceinline__ int ket_digit(uint32_t pk, int m) { return (pk >> (3 * m)) & 7; }
__device__ __forceinline__ int bra_digit(uint32_t pk, int m, int N) {
  return (pk >> (3 * (N + m))) & 7;
}

__device__ __forceinline__ void cmac(float& sr, float& si, c32 a, c32 b) {
  sr = fmaf(a.x, b.x, sr);
  sr = fmaf(-a.y, b.y, sr);
  si = fmaf(a.x, b.y, si);
  si = fmaf(a.y, b.x, si);
}
// s += conj(a) b
__device__ __forceinline__ void cmac_conj(float& sr, float& si, c32 a, c32 b) {
  sr = fmaf(a.x, b.x, sr);
  sr = fmaf(a.y, b.y, sr);
  si = fmaf(a.x, b.y, si);
  si = fmaf(-a.y, b.x, si);
}
__device__ __forceinline__ c32 c_mul(c32 a, c32 b) {
  c32 z;
  z.x = fmaf(-a.y, b.y, a.x * b.x);
  z.y = fmaf(a.x, b.y, a.y * b.x);
  return z;
}
__device__ __forceinline__ c32 c_mul_conj(c32 a, c32 b) {   // conj(a) b
  c32 z;
  z.x = fmaf(a.y, b.y, a.x * b.x);
  z.y = fmaf(a.x, b.y, -a.y * b.x);
  return z;
}

// One row of a static table (cnt entries, stride str) to registers.
template <int cnt, int str>
__device__ __forceinline__ void g_row(const float* __restrict__ row, float (&v)[cnt]) {
  if constexpr (str % 4 == 0) {
#pragma unroll
    for (int k = 0; k < str / 4; ++k) {
      const float4 q = reinterpret_cast<const float4*>(row)[k];
      if (4 * k < cnt) v[4 * k] = q.x;
      if (4 * k + 1 < cnt) v[4 * k + 1] = q.y;
      if (4 * k + 2 < cnt) v[4 * k + 2] = q.z;
      if (4 * k + 3 < cnt) v[4 * k + 3] = q.w;
    }
  } else {
#pragma unroll
    for (int k = 0; k < cnt; ++k) v[k] = row[k];
  }
}

template <int CTRL>
__device__ __forceinline__ float g_dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float g_lane(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

// Sum over the wave (all 64 lanes active), the same in every lane, in a fixed
// order: within each row of 16 lanes by DPP (quad exchanges, then the half-row
// and row mirrors), then the four row sums.  DPP stays on the vector ALU
// (a shuffle would use the LDS crossbar these kernels are bound by).
__device__ __forceinline__ float g_wave_sum(float v) {
  v += g_dpp<0xB1>(v);    // quad_perm [1, 0, 3, 2]
  v += g_dpp<0x4E>(v);    // quad_perm [2, 3, 0, 1]
  v += g_dpp<0x141>(v);   // row_half_mirror
  v += g_dpp<0x140>(v);   // row_mirror
  return (g_lane(v, 0) + g_lane(v, 16)) + (g_lane(v, 32) + g_lane(v, 48));
}

// Shapes with a compiled stepper: open systems D^2 <= 6561, closed systems
// 64 <= D <= 4096 with at most 10 modes.
#define GA_OPEN_SHAPES(X) X(2, 1) X(2, 2) X(2, 3) X(2, 4) X(2, 5) X(3, 1) X(3, 2) X(3, 3) X(3, 4) \
  X(4, 1) X(4, 2) X(4, 3) X(5, 1) X(5, 2)
#define GA_CLOSED_SHAPES(X) X(2, 6) X(2, 7) X(2, 8) X(2, 9) X(2, 10) X(3, 4) X(3, 5) X(3, 6) \
  X(3, 7) X(4, 3) X(4, 4) X(4, 5) X(4, 6) X(5, 3) X(5, 4) X(5, 5)

// The real form's kernels (gather_real.hip).  items != nullptr: a batched
// launch of n workgroups, each reading its own work item; else S = n columns
// (segments: nseg of them from gseg down, S columns each) of one description.
size_t g_real_lds(int d, int N, bool seg);
hipError_t g_real_forward(int d, int N, bool ck, const GItem* items, const GArgs* dargs,
                          const GAdj* dadj, int n, int n_lo, int n_hi, const float4* st_in,
                          float4* st_out, hipStream_t s);
hipError_t g_real_sweep(int d, int N, const GItem* items, const GArgs* dargs, const GAdj* dadj, int n,
                        int g_hi, int g_lo, hipStream_t s);
hipError_t g_real_segments(int d, int N, const GItem* items, const GArgs* dargs, const GAdj* dadj,
                           int n, int gseg, hipStream_t s);
// Open systems' real form (open_real.hip): forward (dadj != nullptr: with
// checkpoints) and the whole reverse walk of S columns.
bool l_real_supported(int d, int N);
hipError_t l_real_forward(int d, int N, const GArgs* dargs, const GAdj* dadj, int S, int nsteps,
                          hipStream_t s);
// Closed d = 3, N = 8 (D = 6561, above the gather engine's shapes): steps [n_lo, n_hi) of
// a forward, the state from st_in / to st_out (nullable).
bool l_column_supported(int d, int N);
hipError_t l_real_column(int d, int N, const GArgs* dargs, int S, int n_lo, int n_hi,
                         const float4* st_in, float4* st_out, hipStream_t s);
hipError_t l_real_adjoint(int d, int N, const GArgs* dargs, const GAdj* dadj, int S, hipStream_t s);
// Frame phases of the half steps [q_lo, q_lo + nq).
hipError_t g_real_phases(int d, int N, int q_lo, int nq, double h, const double f[][8], float2* ph,
                         hipStream_t s);

}  // namespace scp
