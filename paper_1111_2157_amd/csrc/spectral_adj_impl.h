// Traces and adjoints in the spectral form (gfx950 / CDNA4): the kernels of the
// trace, scalar-adjoint and general vector-Jacobian kinds on the operands of
// spectral_impl.h.
//
// With X_j = S D^j S^dag, Gl = (X_1^-1 - Sigma')^-1, L = 1 + Gl Sigma',
// L' = 1 + Sigma' Gl and R = Sigma' L = L' Sigma':
//   tr G   = tr D + tr(R X_2),   tr G^2 = tr D^2 + 2 tr(R X_3) + tr(R X_2 R X_2),
//   M      = S G^2 S^dag = L X_2 L'                    (dN/dSigma, and R X_2 = Sigma' (L X_2)).
// The general product for (Nbar_k, Gbar_n), with Nt = Nbar + Nbar^dag and
// Q = S D Nt D S^dag, Q_3 = S (D Nt D^2 + D^2 Nt D) S^dag:
//   Sigmabar_n^dag = sum_k [ (1/beta) L Q L' + w_k Gl Gbar_n^dag Gl ],
//   mubar = -sum_kn Re [ (1/beta) (sum_v Nt_vv d_v^2 + tr(R Q_3)) + tr(X_2 K) ],
//   K     = (1/beta) R Q R + w_k L' Gbar_n^dag L.
// X_j are real matrix products with the Hermitian P_v (nc^2 reals) as in the
// density kernel.  Q is the adjoint of its sums: d_v d_v' is the weighted mean of
// the products of neighbours in the energy order with weights that do not depend
// on the frequency, so Q = sum_r delta_r(n) Q_r over the 2 nb - 1 products
// delta_r = d_v^2 and d_v d_{v+1}, with Hermitian Q_r formed once per k-point
// (spec_adj_table_kernel); Q_3 has -d delta_r / dz = delta_r (d + d') in their place.
//
// Per evaluation: 4 nb nc^2 real flops per X_j and 8 nb nc^2 each for Q and Q_3 on the
// matrix cores, two row-layout inversions and three (trace), six (scalar adjoint)
// or eleven (general) row-layout products of 8 nc^3.  Bound by those and, as the
// density kernel, by the changes between the units and stages.  Work-groups,
// frequency groups and LDS as there, except that every moment takes its turn in the
// one matrix area (barriers between) and d_v has a single table.
//
// Measured, per k-point and frequency, with the frequency-at-a-time low-rank kernels in
// brackets (256 k-points, 512 or 1024 frequencies): trace, 64 bands and 5 orbitals 1.4 ns
// (6.1), 30 and 10 3.3 (4.8), 40 and 14 5.8 (6.8); scalar adjoint 2.1 (8.4), 4.4 (7.3)
// and 8.0 (10); general product, 40 and 14, 16.5 (28.3).  At 40 bands and 14 orbitals the
// products and inversions would take 4.7, 5.8 and 9.9 ns at full rate: the scalar
// adjoint and the traces lose the rest to stage changes, and the general product to
// fetching its 132 KB of straight-line code through the 64 KB instruction cache.  For
// 15 and 16 orbitals the row matrices spill and the low-rank kernels win (24 bands,
// 16 orbitals: trace 0.43 against 0.55 ms), so the class list ends at 14, but for the
// traces, whose low-rank kernels take neither zero nor dependent rows (256 k-points of 40
// bands, 16 orbitals, 512 frequencies 1.07 ms, the dense code 5.6).
#pragma once

#include "spectral_impl.h"

namespace dmft {

// What a kernel computes: the traces; those and the partials of w_k M; the general
// product of both cotangents, of Nbar alone, of Gbar alone (or neither).
enum { SPEC_TRACE = 0, SPEC_ADJ = 1, SPEC_GEN = 2, SPEC_GEN_N = 3, SPEC_GEN_G = 4 };

template <int NBP, int NC, int WHAT>
struct SpecAdjShared {
  using Dm = SpecDims<NBP, NC>;
  // widest class: V' (scalar adjoint), or the Gbar part of Sigmabar (general product),
  // waits here for its use instead of in registers (48 bands, 14 orbitals: 11.1 to 8.2 and
  // 18.3 to 17.0 ns per k-point and frequency)
  static constexpr bool STASH = (WHAT == SPEC_ADJ || WHAT == SPEC_GEN) && NC >= 14;
  double2 st[STASH ? 16 * NC * NC : 1];
  double2 xr[16 * Dm::NP];  // a moment of the group's frequencies, [n][nc^2] Hermitian pairs
  double2 dt[16 * Dm::DS];  // d_v(n)
  double2 sp[Dm::PREG ? 1 : 2 * NC * Dm::SS];
  double eps[NBP];
  double ntd[NBP];  // Nt_vv in the energy order (general product)
  double red[3 * 4];
  unsigned long long key[NBP];
  double2 lf[WHAT == SPEC_TRACE ? NC * NC : 1];  // L of S = L Q where Q is used
  int rank[NBP];
  int oblique, use_q;
  static __device__ __forceinline__ double2* scratch(SpecAdjShared& sh) { return sh.dt; }  // filled later
};

// c += x b, row layout: c, x hold this lane's row, b the row that lanes broadcast.
template <int NC, int J0 = 0>
__device__ __forceinline__ void spec_mat_mac(double (&cr)[NC], double (&ci)[NC], const double (&xr)[NC],
                                             const double (&xi)[NC], const double (&br)[NC], const double (&bi)[NC]) {
  if constexpr (J0 < NC) {
    constexpr int JB = spec_jb<NC>();
    double tr[JB], ti[JB];
#pragma unroll
    for (int j = 0; j < JB; ++j) {
      tr[j] = cr[J0 + j];
      ti[j] = ci[J0 + j];
    }
    __builtin_amdgcn_sched_barrier(0);
    row_mac<0, NC, JB>(tr, ti, xr, xi, br + J0, bi + J0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < JB; ++j) {
      cr[J0 + j] = tr[j];
      ci[J0 + j] = ti[j];
    }
    spec_mat_mac<NC, J0 + JB>(cr, ci, xr, xi, br, bi);
  }
}

// Row i of a matrix stored as Hermitian pairs (TR: of its transpose).
template <int NC, bool TR>
__device__ __forceinline__ void spec_pair_row(double (&rr)[NC], double (&ri)[NC], const lv2d* xb, int row) {
  const int i = spec_here(row);  // addresses and signs are formed anew at every use
  v2d re[NC], im[NC];
#pragma unroll
  for (int j = 0; j < NC; ++j) {
    const int lo = min(i, j), hi = max(i, j);
    re[j] = xb[lo * NC + hi];
    im[j] = xb[hi * NC + lo];
  }
  __builtin_amdgcn_sched_barrier(0);  // every read issued before the first is waited for
#pragma unroll
  for (int j = 0; j < NC; ++j) {
    const double s = i == j ? 0.0 : ((i < j) != TR ? 1.0 : -1.0);
    rr[j] = __builtin_fma(-s, im[j].y, re[j].x);
    ri[j] = __builtin_fma(s, im[j].x, re[j].y);
  }
}

template <int NC>
__device__ __forceinline__ void spec_set(double (&ar)[NC], double (&ai)[NC], const double (&br)[NC],
                                         const double (&bi)[NC]) {
#pragma unroll
  for (int j = 0; j < NC; ++j) {
    ar[j] = br[j];
    ai[j] = bi[j];
  }
}
template <int NC>
__device__ __forceinline__ void spec_zero(double (&ar)[NC], double (&ai)[NC]) {
#pragma unroll
  for (int j = 0; j < NC; ++j) ar[j] = ai[j] = 0.0;
}

// step(first), step(first + 1), ... while they return true, to N - 1 at most.  Unrolled: as a
// loop around one copy of the product the code of the widest class fits the 64 KB
// instruction cache, but every matrix stays alive through it and spills (general
// product at 48 bands, 14 orbitals: 34.7 ns per k-point and frequency against 18.3).
template <int N, class F>
__device__ __forceinline__ void spec_steps(int first, const F& step) {
  bool on = true;
  spec_for<0, N>([&](auto t) {
    if (on && decltype(t)::value >= first) on = step(decltype(t)::value);
  });
}

// Re of this lane's row of a times its row of b (with b the transpose's row: its share of Re tr(a b)).
template <int NC>
__device__ __forceinline__ double spec_row_dot(const double (&ar)[NC], const double (&ai)[NC], const double (&br)[NC],
                                               const double (&bi)[NC]) {
  double s = 0.0;
#pragma unroll
  for (int j = 0; j < NC; ++j) s = __builtin_fma(ar[j], br[j], __builtin_fma(-ai[j], bi[j], s));
  return s;
}

template <int NBP, int NC, int WHAT>
__device__ __forceinline__ void spec_adj_tile(const DysonArgs& a, int ktile, int wtile, SpecAdjShared<NBP, NC, WHAT>& sh,
                                              int tid) {
  using Dm = SpecDims<NBP, NC>;
  constexpr int T = Dm::T, NT = Dm::NT, NP = Dm::NP, DS = Dm::DS, TPW = Dm::TPW;
  constexpr bool SPLIT = Dm::SPLIT;
  constexpr int PARTS = SPLIT ? 1 : 2;
  constexpr bool GEN = WHAT >= SPEC_GEN, has_n = WHAT == SPEC_GEN || WHAT == SPEC_GEN_N,
                 has_g = WHAT == SPEC_GEN || WHAT == SPEC_GEN_G;
  constexpr bool STASH = SpecAdjShared<NBP, NC, WHAT>::STASH;
  // one copy of the inversion's code where the kernel is well past the 64 KB instruction
  // cache and does not spill more for it (48 bands, 14 orbitals: scalar adjoint 86 to 75 KB,
  // 2.27 to 2.13 ms for 256 k-points x 1024 frequencies; the traces gain nothing, the full
  // product loses 3%)
  constexpr bool ROLL = (WHAT == SPEC_ADJ || WHAT == SPEC_GEN_N || WHAT == SPEC_GEN_G) && NC >= 14;
  const int w = uniform_i(tid >> 6);
  const int n0 = wtile * a.wt, n1 = min(n0 + a.wt, a.nw);
  const int kk0 = ktile * a.kt, kk1 = min(kk0 + a.kt, a.nklist);
  const double mu = uniform_d(a.mu_ptr ? *a.mu_ptr : a.mu);
  const double beta = a.beta, ibeta = 1.0 / a.beta;
  const int nc = a.nc;
  __builtin_assume(nc >= 1 && nc <= NC);
  const double pib = M_PI / beta;
  const double edc = (tid & 15) < nc ? ((const gdouble*)a.e_dc)[tid & 15] : 0.0;
  double pmin = 1.0;
  int nonfinite = 0;

  for (int kk = kk0; kk < kk1; ++kk) {
    const int k = uniform_i(a.klist ? a.klist[kk] : kk);
    const int nb = uniform_i(a.nb_uniform > 0 ? a.nb_uniform : a.nb[k]);
    __builtin_assume(nb > NBP - 16 && nb <= NBP);  // checked by the host for every bucket
    const int64_t ob = uniform_l(a.nb_uniform > 0 ? (int64_t)k * nb : a.off_b[k]);
    const double* eps = a.eps + ob;
    const double2* P = reinterpret_cast<const double2*>(a.proj) + ob * nc;
    const double wk = uniform_d(a.wk[k]);
    const gdouble* qtab = (const gdouble*)a.tsum + a.t_base + (int64_t)kk * spec_adj_slot_doubles(NBP, NC);

    // ---- bands sorted by energy, projector columns in that order (staged over xr)
    __syncthreads();
    if (tid < NBP) sh.key[tid] = tid < nb ? spec_key(eps[tid]) : ~0ull;
    if (tid == 0) sh.oblique = sh.use_q = 0;
    __syncthreads();
    if (tid < NBP) {
      const int r = tid < nb ? spec_rank(sh.key, tid, nb) : tid;
      sh.rank[tid] = r;
      sh.eps[r] = tid < nb ? eps[tid] : mu;
      if (GEN) sh.ntd[tid] = has_n && tid < nb ? qtab[NBP / 2 * NT * 64 + tid] : 0.0;
    }
    __syncthreads();
    for (int idx = tid; idx < NC * NBP; idx += 256) {
      const int al = idx / NBP, v = idx - al * NBP;
      const double2 x = (al < nc && v < nb) ? P[al * nb + v] : make_double2(0.0, 0.0);
      if constexpr (Dm::PREG) {
        sh.xr[al * NBP + sh.rank[v]] = x;
      } else {
        sh.sp[al * Dm::SS + sh.rank[v]] = x;
        sh.sp[(NC + al) * Dm::SS + sh.rank[v]] = make_double2(x.y, -x.x);
      }
    }
    __syncthreads();
    if constexpr (WHAT == SPEC_TRACE) spec_rows_check<NBP, NC>(sh, nc, tid);
    double p[Dm::PREG ? TPW : 1][Dm::PREG ? NBP / 4 : 1];
    int pab[TPW];
#pragma unroll
    for (int m = 0; m < TPW; ++m) {
      const int job = w + 4 * m, q = (tid >> 4) & 3, c16 = tid & 15;
      const int ab = min(16 * (SPLIT ? job >> 1 : job) + c16, NC * NC - 1);
      const int al = ab / NC, be = ab - al * NC;
      if constexpr (Dm::PREG) {
#pragma unroll
        for (int c = 0; c < NBP / 4; ++c) {
          const double2 x = sh.xr[al * NBP + 4 * c + q], y = sh.xr[be * NBP + 4 * c + q];
          const double re = x.x * y.x + x.y * y.y, im = y.y * x.x - y.x * x.y;
          p[m][c] = al <= be ? re : im;
        }
      } else {
        pab[m] = (al * Dm::SS + q) | ((al <= be ? be : NC + be) * Dm::SS + q) << 16;
      }
    }

    double t1 = 0.0, t2 = 0.0, mub = 0.0;  // this thread's shares of Re tr G, Re tr G^2, mubar

    // NM moments of the group as matrix products: powers d^J0 .. of the resolvent table
    using Acc = v4d[2][TPW][PARTS];
    auto moments = [&](auto j0c, auto nmc, Acc& xa) {
      constexpr int J0 = decltype(j0c)::value, NM = decltype(nmc)::value;
      const int l = spec_here(tid & 63), q = l >> 4, c16 = l & 15;
      const lv2d* dt = spec_lds(&sh.dt[c16 * DS + q]);
      const lv2d *sa[TPW], *sb[TPW];
#pragma unroll
      for (int m = 0; m < TPW; ++m) {
        if constexpr (!Dm::PREG) {
          const int ab = spec_here(pab[m]);
          sa[m] = spec_lds(&sh.sp[ab & 0xffff]);
          sb[m] = spec_lds(&sh.sp[ab >> 16]);
        }
#pragma unroll
        for (int u = 0; u < NM; ++u)
#pragma unroll
          for (int h = 0; h < PARTS; ++h) xa[u][m][h] = (v4d){0.0, 0.0, 0.0, 0.0};
      }
      v2d d[2], x[2][Dm::PREG ? 1 : TPW], y[2][Dm::PREG ? 1 : TPW];
      auto fetch = [&](int c, int s) {
        d[s] = dt[4 * c];
        if constexpr (!Dm::PREG) {
#pragma unroll
          for (int m = 0; m < TPW; ++m) {
            x[s][m] = sa[m][4 * c];
            y[s][m] = sb[m][4 * c];
          }
        }
      };
      fetch(0, 0);
      spec_for<0, NBP / 4>([&](auto ci) {
        constexpr int c = decltype(ci)::value;
        if (4 * c >= nb) return;
        if constexpr (c + 1 < NBP / 4) fetch(c + 1, (c + 1) & 1);
        __builtin_amdgcn_sched_barrier(0);
        double pv[TPW];
#pragma unroll
        for (int m = 0; m < TPW; ++m) {
          if constexpr (Dm::PREG)
            pv[m] = p[m][c];
          else
            pv[m] = __builtin_fma(x[c & 1][m].x, y[c & 1][m].x, x[c & 1][m].y * y[c & 1][m].y);
        }
        v2d e[2];
        const v2d d1 = d[c & 1];
        const v2d d2 = (v2d){d1.x * d1.x - d1.y * d1.y, 2.0 * d1.x * d1.y};
        e[0] = J0 == 1 ? d1 : d2;
        e[1] = (v2d){d2.x * d1.x - d2.y * d1.y, d2.x * d1.y + d2.y * d1.x};
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < NM; ++u) {
          const double dx = SPLIT && (w & 1) ? e[u].y : e[u].x;
#pragma unroll
          for (int m = 0; m < TPW; ++m) {
            xa[u][m][0] = mma(dx, pv[m], xa[u][m][0]);
            if constexpr (!SPLIT) xa[u][m][1] = mma(e[u].y, pv[m], xa[u][m][1]);
          }
        }
      });
    };
    // Q (xa[0]) and Q_3 (xa[1]): rows delta_r and delta_r (d + d') against the table,
    // whose chunks of four rows are read PF ahead (they come from L2)
    auto rows = [&](Acc& xa) {
      constexpr int CH = NBP / 2, PF = SPLIT ? 8 : 5;
      const int l = spec_here(tid & 63), q = l >> 4, c16 = l & 15;
      const lv2d* da = spec_lds(&sh.dt[c16 * DS + (q >> 1)]);
      const lv2d* db = spec_lds(&sh.dt[c16 * DS + ((q + 1) >> 1)]);  // index NBP (past the rows in use) is padding
      const gdouble* qt = qtab + l;
      double b[PF + 1][TPW];
#pragma unroll
      for (int m = 0; m < TPW; ++m)
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int h = 0; h < PARTS; ++h) xa[u][m][h] = (v4d){0.0, 0.0, 0.0, 0.0};
      auto fetch = [&](int c) {
#pragma unroll
        for (int m = 0; m < TPW; ++m)
          b[c % (PF + 1)][m] = qt[(c * NT + min(SPLIT ? (w + 4 * m) >> 1 : w + 4 * m, NT - 1)) * 64];
      };
      spec_for<0, PF>([&](auto ci) { fetch(decltype(ci)::value); });
      v2d x[2], y[2];
      x[0] = da[0];
      y[0] = db[0];
      spec_for<0, CH>([&](auto ci) {
        constexpr int c = decltype(ci)::value;
        if (4 * c > 2 * nb - 2) return;
        if constexpr (c + PF < CH) fetch(c + PF);
        if constexpr (c + 1 < CH) {
          x[(c + 1) & 1] = da[2 * c + 2];
          y[(c + 1) & 1] = db[2 * c + 2];
        }
        __builtin_amdgcn_sched_barrier(0);
        const v2d u = x[c & 1], v = y[c & 1];
        v2d e[2];
        e[0] = (v2d){u.x * v.x - u.y * v.y, u.x * v.y + u.y * v.x};
        const v2d s = u + v;
        e[1] = (v2d){e[0].x * s.x - e[0].y * s.y, e[0].x * s.y + e[0].y * s.x};
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const double dx = SPLIT && (w & 1) ? e[j].y : e[j].x;
#pragma unroll
          for (int m = 0; m < TPW; ++m) {
            xa[j][m][0] = mma(dx, b[c % (PF + 1)][m], xa[j][m][0]);
            if constexpr (!SPLIT) xa[j][m][1] = mma(e[j].y, b[c % (PF + 1)][m], xa[j][m][1]);
          }
        }
      });
    };
    // a moment to the matrix area, once every wavefront is done with the last one
    auto publish = [&](const v4d (&xa)[TPW][PARTS]) {
      __syncthreads();
      const int l = spec_here(tid & 63), q = l >> 4, c16 = l & 15;
      lv2d* xw = spec_lds(&sh.xr[q * NP + c16]);
#pragma unroll
      for (int m = 0; m < TPW; ++m) {
        const int job = w + 4 * m;
        if (job >= (SPLIT ? 2 * NT : NT)) break;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if constexpr (SPLIT)
            ((lds_double*)(xw + 4 * i * NP + 16 * (job >> 1)))[job & 1] = xa[m][0][i];
          else
            xw[4 * i * NP + 16 * job] = (v2d){xa[m][0][i], xa[m][1][i]};
        }
      }
      __syncthreads();
    };
    // this lane's row of the matrix set aside (lanes past NC share the last row's slot, unwritten by them)
    auto stash = [&](const double (&ar)[NC], const double (&ai)[NC]) {
      const int l = spec_here(tid & 63), i = l & 15;
      if (i < NC) {
        lv2d* st = spec_lds(&sh.st[((4 * w + (l >> 4)) * NC + i) * NC]);
#pragma unroll
        for (int j = 0; j < NC; ++j) st[j] = (v2d){ar[j], ai[j]};
      }
    };
    auto unstash = [&](double (&ar)[NC], double (&ai)[NC]) {
      const int l = spec_here(tid & 63);
      const lv2d* st = spec_lds(&sh.st[((4 * w + (l >> 4)) * NC + min(l & 15, NC - 1)) * NC]);
      v2d z[NC];
#pragma unroll
      for (int j = 0; j < NC; ++j) z[j] = st[j];
#pragma unroll
      for (int j = 0; j < NC; ++j) {
        ar[j] = z[j].x;
        ai[j] = z[j].y;
      }
    };
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;

    // (two copies, see spec_tile; the traces are the same in the rows of Q, with
    // Sigma' there: tr G = tr D + tr(R_Q X_Q2), ...)
    auto frequencies = [&](auto obl) __attribute__((always_inline)) {
      constexpr bool oblique = decltype(obl)::value;
      for (int ng = n0; ng < n1; ng += 16) {
        __syncthreads();  // the last group's matrix area and resolvent table are free
        {
          const int t = spec_here(tid), nl = t & 15, v0 = t >> 4;
          const double wn = (double)(2 * min(ng + nl, n1 - 1) + 1) * pib;
          lv2d* dt = spec_lds(&sh.dt[nl * DS + v0]);
          const lds_double* es = (const lds_double*)&sh.eps[v0];
          const lds_double* nt = (const lds_double*)&sh.ntd[v0];
          const bool on = ng + nl < n1;
#pragma unroll
          for (int m = 0; m < T; ++m) {
            const double2 d = inv_z_minus(mu, wn, es[16 * m]);
            dt[16 * m] = (v2d){d.x, d.y};
            const double d2 = __builtin_fma(d.x, d.x, -d.y * d.y);
            if (on && v0 + 16 * m < nb) {
              t1 += d.x;
              t2 += d2;
              if (GEN) mub -= ibeta * nt[16 * m] * d2;
            }
          }
          if (v0 == 0) sh.dt[nl * DS + NBP] = make_double2(0.0, 0.0);
        }
        const int l = spec_here(tid & 63), i = l & 15, nl = 4 * w + (l >> 4), ic = min(i, NC - 1);
        const bool valid = ng + nl < n1, mine = valid && i < NC;
        const int n = min(ng + nl, n1 - 1);
        double sr[NC], si[NC];  // row i of Sigma', in flight until it is needed
        {
          const gv2d* sgp = (const gv2d*)a.sigma + ((int64_t)n * nc + min(i, nc - 1)) * nc;
#pragma unroll
          for (int j = 0; j < NC; ++j) {
            const v2d v = sgp[min(j, nc - 1)];
            sr[j] = v.x;
            si[j] = v.y;
          }
        }
        __syncthreads();
        Acc xa;
        moments(I1{}, I1{}, xa);
        publish(xa[0]);
        lv2d* xb = spec_lds(&sh.xr[nl * NP]);
        double gr[NC], gi[NC];
        spec_pair_row<NC, false>(gr, gi, xb, ic);
        const v2d own = xb[ic * NC + ic];
        const unsigned long long absent = row_absent(own.x, own.y, i, nc);
        if (absent) row_leave_out<NC>(gr, gi, absent, l, 1.0);
        if (nc < NC) {
#pragma unroll
          for (int j = 0; j < NC; ++j) {
            gr[j] = i < nc ? gr[j] : (i == j ? 1.0 : 0.0);
            gi[j] = i < nc ? gi[j] : 0.0;
            sr[j] = i < nc && j < nc ? sr[j] : 0.0;
            si[j] = i < nc && j < nc ? si[j] : 0.0;
          }
        }
        auto invert = [&](int t) {
          spec_sweep<NC>(gr, gi, i, pmin);
          if (t == 0) {
#pragma unroll
            for (int j = 0; j < NC; ++j) sr[j] -= i == j ? edc : 0.0;
            if constexpr (oblique) {  // by way of the matrix area
              spec_put_row<NC>(xb, i, sr, si);
              spec_inner<NC>(xb, spec_lds(sh.lf), i, min(i + 1, NC));
#pragma unroll
              for (int j = 0; j < NC; ++j) {
                const v2d x = xb[ic * NC + j];
                sr[j] = x.x;
                si[j] = x.y;
              }
            }
#pragma unroll
            for (int j = 0; j < NC; ++j) {
              gr[j] -= sr[j];
              gi[j] -= si[j];
            }
            if (absent) row_leave_out<NC>(gr, gi, absent, l, 1.0);
          }
        };
        if constexpr (ROLL) {
#pragma clang loop unroll(disable)
          for (int t = 0; t < 2; ++t) invert(t);
        } else {
          invert(0);
          invert(1);
        }
        if (absent) row_leave_out<NC>(gr, gi, absent, l, 0.0);
        if (nc < NC) {  // the identity of rows past nc must not count as part of Gl
#pragma unroll
          for (int j = 0; j < NC; ++j) {
            gr[j] = i < nc && j < nc ? gr[j] : 0.0;
            gi[j] = i < nc && j < nc ? gi[j] : 0.0;
          }
        }
        if constexpr (GEN) {
          double chk = 0.0;
#pragma unroll
          for (int j = 0; j < NC; ++j) chk += gr[j] + gi[j];
          if (mine && !__builtin_isfinite(chk)) nonfinite = 1;
        }
        // The order below keeps few row matrices alive at a time (4 registers per
        // column): the moment that is only traced against R goes first.
        const gv2d* gbp = (const gv2d*)a.gbar + (int64_t)n * nc * nc + min(i, nc - 1);
        auto load_gbar = [&](double (&ar)[NC], double (&ai)[NC]) {  // row i of w_k Gbar^dag
          if (WHAT == SPEC_GEN_G && !a.gbar) return spec_zero<NC>(ar, ai);
#pragma unroll
          for (int j = 0; j < NC; ++j) {
            const v2d v = gbp[min(j, nc - 1) * nc];
            ar[j] = wk * v.x;
            ai[j] = -wk * v.y;
          }
          if (nc < NC) {
#pragma unroll
            for (int j = 0; j < NC; ++j) {
              ar[j] = i < nc && j < nc ? ar[j] : 0.0;
              ai[j] = i < nc && j < nc ? ai[j] : 0.0;
            }
          }
        };
        double xr[NC], xi[NC], br[NC], bi[NC], cr[NC], ci[NC];  // c += x b at every step
        double nr[GEN ? NC : 1], ni[GEN ? NC : 1];              // Sigmabar^dag, then K
        if constexpr (GEN) {
          spec_zero<NC>(nr, ni);
          if constexpr (has_g) {  // w_k Gl Gbar^dag Gl
            spec_set<NC>(xr, xi, gr, gi);
            load_gbar(br, bi);
            spec_zero<NC>(cr, ci);
            spec_steps<2>(0, [&](int t) {
              spec_mat_mac<NC>(cr, ci, xr, xi, br, bi);
              if (t == 0) {
                spec_set<NC>(xr, xi, cr, ci);
                spec_set<NC>(br, bi, gr, gi);
                spec_zero<NC>(cr, ci);
              }
              return true;
            });
            if constexpr (STASH)
              stash(cr, ci);
            else
              spec_set<NC>(nr, ni, cr, ci);
          }
        }
        // V = Gl Sigma', V' = Sigma' Gl (not for the traces), R = Sigma' + Sigma' V (in c; x = Sigma')
        double vr[NC], vi[NC], ur[WHAT == SPEC_TRACE ? 1 : NC], ui[WHAT == SPEC_TRACE ? 1 : NC];
        spec_set<NC>(xr, xi, gr, gi);
        spec_set<NC>(br, bi, sr, si);
        spec_zero<NC>(cr, ci);
        spec_steps<3>(0, [&](int t) {
          spec_mat_mac<NC>(cr, ci, xr, xi, br, bi);
          if (t == 0) {
            spec_set<NC>(vr, vi, cr, ci);
            if constexpr (WHAT == SPEC_TRACE) {
              spec_set<NC>(xr, xi, br, bi);
              spec_set<NC>(cr, ci, br, bi);
              spec_set<NC>(br, bi, vr, vi);
            } else {
              double tr[NC], ti[NC];
              spec_set<NC>(tr, ti, xr, xi);
              spec_set<NC>(xr, xi, br, bi);
              spec_set<NC>(br, bi, tr, ti);
              spec_zero<NC>(cr, ci);
            }
            return true;
          }
          if (WHAT == SPEC_TRACE || t == 2) return false;
          if constexpr (WHAT != SPEC_TRACE) {
            if constexpr (STASH && WHAT == SPEC_ADJ)
              stash(cr, ci);
            else
              spec_set<NC>(ur, ui, cr, ci);
            spec_set<NC>(cr, ci, xr, xi);
            spec_set<NC>(br, bi, vr, vi);
          }
          return true;
        });
        double rr[NC], ri[NC];
        spec_set<NC>(rr, ri, cr, ci);
        if constexpr (!GEN) {
          if constexpr (WHAT == SPEC_ADJ) spec_set<NC>(sr, si, xr, xi);
          moments(I2{}, I2{}, xa);
          publish(xa[1]);
          spec_pair_row<NC, true>(cr, ci, xb, ic);  // X_3
          const double r3 = spec_row_dot<NC>(rr, ri, cr, ci);
          publish(xa[0]);
          if (mine) t2 += 2.0 * r3;
          spec_pair_row<NC, false>(br, bi, xb, ic);
          if constexpr (WHAT == SPEC_TRACE) {
            spec_zero<NC>(cr, ci);
            spec_mat_mac<NC>(cr, ci, rr, ri, br, bi);  // R X_2
          } else {
            // T = L X_2, M = T L', R X_2 = Sigma' T
            double tr[NC], ti[NC];
            spec_set<NC>(xr, xi, vr, vi);
            spec_set<NC>(cr, ci, br, bi);
            spec_steps<3>(0, [&](int t) {
              spec_mat_mac<NC>(cr, ci, xr, xi, br, bi);
              if (t == 0) {
                spec_set<NC>(tr, ti, cr, ci);
                spec_set<NC>(xr, xi, cr, ci);
                if constexpr (STASH)
                  unstash(br, bi);
                else
                  spec_set<NC>(br, bi, ur, ui);
              } else if (t == 1) {
                // M by columns (through this matrix's own part of the matrix area), so that
                // the partial is read and written 16 lanes to a row
                wave_sync();
                if (i < NC) {
#pragma unroll
                  for (int j = 0; j < NC; ++j) xb[i * NC + j] = (v2d){cr[j], ci[j]};
                }
                wave_sync();
                if (mine) {
                  gv2d* mp = (gv2d*)a.xpart + ((int64_t)(a.ktile_base + ktile) * a.nw + n) * 256 + i;
                  v2d o[NC], z[NC];
#pragma unroll
                  for (int j = 0; j < NC; ++j) {
                    o[j] = (v2d){0.0, 0.0};
                    z[j] = xb[j * NC + i];
                  }
                  if (kk != kk0) {
#pragma unroll
                    for (int j = 0; j < NC; ++j) o[j] = mp[j * 16];
                  }
#pragma unroll
                  for (int j = 0; j < NC; ++j)
                    mp[j * 16] = (v2d){__builtin_fma(wk, z[j].x, o[j].x), __builtin_fma(wk, z[j].y, o[j].y)};
                }
                spec_set<NC>(xr, xi, sr, si);
                spec_set<NC>(br, bi, tr, ti);
                spec_zero<NC>(cr, ci);
              }
              return true;
            });
          }
          // tr((R X_2)^2): the transpose the same way
          wave_sync();
          if (i < NC) {
#pragma unroll
            for (int j = 0; j < NC; ++j) xb[i * NC + j] = (v2d){cr[j], ci[j]};
          }
          wave_sync();
          double q1 = 0.0, q2 = 0.0;
#pragma unroll
          for (int j = 0; j < NC; ++j) {
            const v2d z = xb[j * NC + ic];
            q1 = i == j ? cr[j] : q1;
            q2 = __builtin_fma(cr[j], z.x, __builtin_fma(-ci[j], z.y, q2));
          }
          if (mine) {
            t1 += q1;
            t2 += q2;
          }
        } else {
          auto store = [&](const double (&ar)[NC], const double (&ai)[NC]) {
            if (!mine) return;  // Sigmabar = (..)^dag: this lane's row is a column of it
            gv2d* mp = (gv2d*)a.xpart + ((int64_t)(a.ktile_base + ktile) * a.nw + n) * 256 + i;
            v2d o[NC];
#pragma unroll
            for (int j = 0; j < NC; ++j) o[j] = (v2d){0.0, 0.0};
            if (kk != kk0) {
#pragma unroll
              for (int j = 0; j < NC; ++j) o[j] = mp[j * 16];
            }
#pragma unroll
            for (int j = 0; j < NC; ++j) mp[j * 16] = (v2d){o[j].x + ar[j], o[j].y - ai[j]};
          };
          auto load_q = [&]() {  // Q / beta
            spec_pair_row<NC, false>(br, bi, xb, ic);
#pragma unroll
            for (int j = 0; j < NC; ++j) {
              br[j] *= ibeta;
              bi[j] *= ibeta;
            }
          };
          auto start_g = [&]() {  // L' Gbar^dag next
            spec_set<NC>(xr, xi, ur, ui);
            load_gbar(br, bi);
            spec_set<NC>(cr, ci, br, bi);
          };
          if constexpr (has_n) {
            rows(xa);
            publish(xa[1]);
            spec_pair_row<NC, true>(cr, ci, xb, ic);  // Q_3
            const double r3 = spec_row_dot<NC>(rr, ri, cr, ci);
            if (mine) mub -= ibeta * r3;
            publish(xa[0]);
            spec_set<NC>(xr, xi, vr, vi);
            load_q();
            spec_set<NC>(cr, ci, br, bi);
          } else {
            store(nr, ni);
            spec_zero<NC>(nr, ni);
            start_g();
          }
          {
            spec_steps<6>(has_n ? 0 : 4, [&](int t) {
              spec_mat_mac<NC>(cr, ci, xr, xi, br, bi);
              if (t == 0) {  // L Q; L Q L' next, on top of the Gbar part
                spec_set<NC>(xr, xi, cr, ci);
                spec_set<NC>(br, bi, ur, ui);
                if constexpr (STASH) unstash(nr, ni);
#pragma unroll
                for (int j = 0; j < NC; ++j) {
                  cr[j] += nr[j];
                  ci[j] += ni[j];
                }
              } else if (t == 1) {  // R Q next
                store(cr, ci);
                spec_set<NC>(xr, xi, rr, ri);
                load_q();
                spec_zero<NC>(cr, ci);
              } else if (t == 2) {  // R Q R next
                spec_set<NC>(xr, xi, cr, ci);
                spec_set<NC>(br, bi, rr, ri);
                spec_zero<NC>(cr, ci);
              } else if (t == 3) {
                if (!has_g) return false;
                spec_set<NC>(nr, ni, cr, ci);
                start_g();
              } else if (t == 4) {  // L' Gbar^dag L next
                spec_set<NC>(xr, xi, cr, ci);
                spec_set<NC>(br, bi, vr, vi);
#pragma unroll
                for (int j = 0; j < NC; ++j) {
                  cr[j] += nr[j];
                  ci[j] += ni[j];
                }
              }
              return true;
            });
            spec_set<NC>(nr, ni, cr, ci);  // K
            moments(I2{}, I1{}, xa);
            publish(xa[0]);
            spec_pair_row<NC, true>(cr, ci, xb, ic);  // X_2
            const double x2 = spec_row_dot<NC>(nr, ni, cr, ci);
            if (mine) mub -= x2;
          }
        }
      }
    };
    if constexpr (WHAT == SPEC_TRACE) {
      if (uniform_i(sh.use_q))
        frequencies(std::true_type());
      else
        frequencies(std::false_type());
    } else {
      frequencies(std::false_type());
    }
    // ---- this k-point's traces: lanes, then wavefronts in order
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      t1 += __shfl_xor(t1, off);
      t2 += __shfl_xor(t2, off);
      if (GEN) mub += __shfl_xor(mub, off);
    }
    if ((tid & 63) == 0) {
      sh.red[w] = t1;
      sh.red[4 + w] = t2;
      sh.red[8 + w] = mub;
    }
    __syncthreads();
    if (tid == 0) {
      const int stride = (a.mode & MODE_TRACE) ? 2 : 3;
      double* tp = a.tpart + ((int64_t)wtile * a.nk + k) * stride;
      const double s1 = sh.red[0] + sh.red[1] + sh.red[2] + sh.red[3];
      const double s2 = sh.red[4] + sh.red[5] + sh.red[6] + sh.red[7];
      const double s3 = sh.red[8] + sh.red[9] + sh.red[10] + sh.red[11];
      tp[0] = GEN ? 0.0 : s1;
      tp[1] = GEN ? 0.0 : s2;
      if (stride == 3) tp[2] = GEN ? s3 : 0.0;
      if (!__builtin_isfinite(GEN ? s3 : s1 + s2)) nonfinite = 1;
    }
  }
  if (pmin == 0.0 && (tid & 15) < NC) atomicOr(a.err, ERR_SINGULAR);
  if (nonfinite) atomicOr(a.err, ERR_NONFINITE);
}

template <int NBP, int NC, int WHAT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(spec_adj_wgs_per_cu(NC, WHAT))))
spec_adj_kernel(DysonArgs a) {
  __shared__ SpecAdjShared<NBP, NC, WHAT> sh;
  // work-groups go to the eight XCDs in turn: the frequency tiles of a k-tile are kept on
  // one of them, whose L2 then holds their table (160 KB at 48 bands, 14 orbitals) once
  const int n = gridDim.x, x = blockIdx.x & 7, item = x * (n >> 3) + min(x, n & 7) + (blockIdx.x >> 3);
  spec_adj_tile<NBP, NC, WHAT>(a, item / a.n_wtiles, item % a.n_wtiles, sh, threadIdx.x);
}

}  // namespace dmft
