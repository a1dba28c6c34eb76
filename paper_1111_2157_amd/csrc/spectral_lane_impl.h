// Spectral form of the density pass (see spectral_impl.h for the algebra) for up to
// five orbitals: one matrix per lane.
//
// In the row layout a wavefront inverts four matrices on 16 lanes each, of which nc
// work; at five orbitals that stage took over half of a pass.  Here a lane holds the
// whole nc x nc matrices of its frequency (25 complex numbers, 100 registers each), so
// the inversions and products are plain register arithmetic on 64 frequencies at a
// time with no idle lanes, and a wavefront needs nobody else: it is a work-group, takes
// a (k-tile, frequency-tile) item of its own, and walks groups of 64 frequencies:
//   A. X of 16 frequencies at a time as 16x16x4 products, each lane computing the one
//      resolvent it contributes as the left operand, P_v in registers for the whole
//      k-point; X to LDS, [frequency][nc^2];
//   B. per lane X^-1, Gl = (X^-1 - Sigma')^-1 and R = Sigma' + Sigma' Gl Sigma', the
//      G_loc partial ([element][frequency], coalesced), R back to LDS as Hermitian pairs;
//   C. the sums of d_v d_v' times R, four frequencies at a time; their resolvents are
//      computed once more, into a table of those four.
// Four wavefronts per CU (one per SIMD: up to 512 registers, 36 KB of LDS each).
//
// Bound by the matrix cores (A and C: 4 nb nc^2 and 8 nb nc^2 with nc^2 padded to 32)
// and, at small windows, by B.  Measured per k-point and frequency, 512 k-points, 2048
// frequencies, row layout in brackets: 64 bands 0.72 ns (1.04), 48 0.58 (0.98), 32
// 0.44 (0.82), 16 0.33 (0.7).  Six orbitals do not fit the registers at 64 bands.
#pragma once

#include "spectral_impl.h"

namespace dmft {

template <int NBP, int NC>
struct SpecLaneShared {
  static constexpr int NN = NC * NC, LDX = NN | 1, DS = NBP + 1;
  double2 x[64 * LDX];     // X, then R, [frequency][nc^2]; the projectors while a k-point is set up
  double2 d[2][4 * DS];    // d_v of four frequencies, two turns
  double eps[NBP];         // sorted band energies
  unsigned long long key[NBP];
  double2 lf[NC * NC];     // L of S = L Q where Q is used
  double g[NC * NC];       // S S^dag
};

// In-place Gauss-Jordan inverse of one matrix per lane; pmin: smallest |pivot|^2 so far.
template <int NC>
__device__ __forceinline__ void lane_inverse(double (&ar)[NC][NC], double (&ai)[NC][NC], double& pmin) {
#pragma unroll
  for (int p = 0; p < NC; ++p) {
    const double px = ar[p][p], py = ai[p][p];
    const double d = __builtin_fma(px, px, py * py);
    asm("v_min_f64 %0, %0, %1" : "+v"(pmin) : "v"(d));
    double t = __builtin_amdgcn_rcp(d);
    const double e = __builtin_fma(-d, t, 1.0);
    t = __builtin_fma(t, __builtin_fma(e, e, e), t);
    const double ix = px * t, iy = -py * t;
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      if (j == p) continue;
      const double x = ar[p][j], y = ai[p][j];
      ar[p][j] = __builtin_fma(x, ix, -y * iy);
      ai[p][j] = __builtin_fma(x, iy, y * ix);
    }
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      if (i == p) continue;
      const double fx = ar[i][p], fy = ai[i][p];
#pragma unroll
      for (int j = 0; j < NC; ++j) {
        if (j == p) continue;
        ar[i][j] = __builtin_fma(-fx, ar[p][j], __builtin_fma(fy, ai[p][j], ar[i][j]));
        ai[i][j] = __builtin_fma(-fx, ai[p][j], __builtin_fma(-fy, ar[p][j], ai[i][j]));
      }
      ar[i][p] = __builtin_fma(-fx, ix, fy * iy);
      ai[i][p] = __builtin_fma(-fx, iy, -fy * ix);
    }
    ar[p][p] = ix;
    ai[p][p] = iy;
  }
}

template <int NBP, int NC, bool WS>
__device__ __forceinline__ void spec_lane_tile(const DysonArgs& a, int ktile, int wtile, SpecLaneShared<NBP, NC>& sh,
                                               int lane) {
  using Sh = SpecLaneShared<NBP, NC>;
  constexpr int NN = Sh::NN, LDX = Sh::LDX, DS = Sh::DS, NT = spec_col_tiles(NC), NR = spec_row_tiles(NBP);
  const int n0 = wtile * a.wt, n1 = min(n0 + a.wt, a.nw);
  const int kk0 = ktile * a.kt, kk1 = min(kk0 + a.kt, a.nklist);
  const double mu = uniform_d(a.mu_ptr ? *a.mu_ptr : a.mu);
  const int nc = a.nc;
  __builtin_assume(nc >= 1 && nc <= NC);
  const bool want_x = a.mode & MODE_GLOC;
  const int nw4 = (a.nw + 3) & ~3;
  const double pib = M_PI / a.beta;
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

    // ---- bands sorted by energy, projector columns in that order
    wave_sync();
    {
      const double e = lane < nb ? eps[lane] : mu;
      if (lane < NBP) sh.key[lane] = lane < nb ? spec_key(e) : ~0ull;
      wave_sync();
      const int r = lane < nb ? spec_rank(sh.key, lane, nb) : lane;
      if (lane < NBP) {
        sh.eps[r] = e;
#pragma unroll
        for (int al = 0; al < NC; ++al)
          sh.x[al * NBP + r] = (al < nc && lane < nb) ? P[al * nb + lane] : make_double2(0.0, 0.0);
      }
      wave_sync();
    }
    double p[NT][NBP / 4];
    auto load_p = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int q = (lane >> 4) & 3, ab = min(16 * t + (lane & 15), NN - 1), al = ab / NC, be = ab - al * NC;
#pragma unroll
        for (int c = 0; c < NBP / 4; ++c) {
          const double2 x = sh.x[al * NBP + 4 * c + q], y = sh.x[be * NBP + 4 * c + q];
          p[t][c] = al <= be ? x.x * y.x + x.y * y.y : y.y * x.x - y.x * x.y;
        }
      }
    };
    load_p();
    // oblique rows, from S S^dag = sum_v P_v (summed over the quarters of the lanes by a
    // product with ones): Q in their place
    bool use_q = false;
    {
      double g[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        double u = 0.0, v = 0.0;
#pragma unroll
        for (int c = 0; c < NBP / 4; c += 2) {
          u += p[t][c];
          v += p[t][c + 1];
        }
        g[t] = mma(1.0, u + v, (v4d){0.0, 0.0, 0.0, 0.0})[0];
        const int ab = 16 * t + (lane & 15);
        if (lane < 16 && ab < NN) sh.g[ab] = g[t];
      }
      wave_sync();
      bool bad = false;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int ab = min(16 * t + (lane & 15), NN - 1), al = ab / NC, be = ab - al * NC;
        bad |= al < nc && be < nc && spec_oblique(sh.g[al * (NC + 1)], sh.g[be * (NC + 1)], g[t], al == be, nc);
      }
      if (__ballot(bad)) {
        use_q = __ballot(spec_orthonormal<NBP, NC>(sh.x, NBP, sh.lf, sh.d[0], nc, lane)) != 0;
        if (use_q) load_p();  // else p stays as it is
      }
    }
    wave_sync();

    v4d acc[NR][NT];
    double sd[NBP / 16];
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[r][t] = (v4d){0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int m = 0; m < NBP / 16; ++m) sd[m] = 0.0;

    auto frequencies = [&](auto obl) __attribute__((always_inline)) {  // two copies, see spec_tile
      constexpr bool oblique = decltype(obl)::value;
      for (int ng = n0; ng < n1; ng += 64) {
        // ---- stage A
        {
          const int l = spec_here(lane), q = l >> 4, c16 = l & 15;
          const lds_double* es = (const lds_double*)&sh.eps[q];
#pragma clang loop unroll(disable)
          for (int f = 0; f < 64 && ng + f < n1; f += 16) {
            const double wn = (double)(2 * min(ng + f + c16, n1 - 1) + 1) * pib;
            v4d xa[NT][2];
#pragma unroll
            for (int t = 0; t < NT; ++t) xa[t][0] = xa[t][1] = (v4d){0.0, 0.0, 0.0, 0.0};
            spec_for<0, NBP / 4>([&](auto ci) {
              constexpr int c = decltype(ci)::value;
              if (4 * c >= nb) return;
              const double2 d = inv_z_minus(mu, wn, es[4 * c]);
              __builtin_amdgcn_sched_barrier(0);
#pragma unroll
              for (int t = 0; t < NT; ++t) {
                xa[t][0] = mma(d.x, p[t][c], xa[t][0]);
                xa[t][1] = mma(d.y, p[t][c], xa[t][1]);
              }
            });
            lv2d* xw = spec_lds(&sh.x[(f + q) * LDX + c16]);
#pragma unroll
            for (int t = 0; t < NT; ++t)
              if (16 * t + c16 < NN) {
#pragma unroll
                for (int i = 0; i < 4; ++i) xw[4 * i * LDX + 16 * t] = (v2d){xa[t][0][i], xa[t][1][i]};
              }
          }
        }
        wave_sync();
        // ---- stage B: this lane's frequency
        {
          const int l = spec_here(lane), n = min(ng + l, n1 - 1);
          const bool valid = ng + l < n1;
          const bool whole = nc == NC && ng + 64 <= n1;  // no orbital or frequency to mask
          lv2d* xb = spec_lds(&sh.x[l * LDX]);
          double sr[NC][NC], si[NC][NC];  // Sigma', in flight during the first inversion
          {
            const gv2d* sg = (const gv2d*)a.sigma + (int64_t)n * nc * nc;
#pragma unroll
            for (int i = 0; i < NC; ++i)
#pragma unroll
              for (int j = 0; j < NC; ++j) {
                const v2d v = sg[min(i, nc - 1) * nc + min(j, nc - 1)];
                sr[i][j] = v.x;
                si[i][j] = v.y;
              }
          }
          double gr[NC][NC], gi[NC][NC];
#pragma unroll
          for (int i = 0; i < NC; ++i)
#pragma unroll
            for (int j = i; j < NC; ++j) {
              const v2d re = xb[i * NC + j];
              v2d im = (v2d){0.0, 0.0};
              if (i != j) im = xb[j * NC + i];
              gr[i][j] = re.x - im.y;
              gi[i][j] = re.y + im.x;
              if (i != j) {
                gr[j][i] = re.x + im.y;
                gi[j][i] = re.y - im.x;
              }
            }
          // orbitals without weight in this window (see row_absent; the same in every lane)
          int absent = 0;
#pragma unroll
          for (int i = 0; i < NC; ++i) absent |= i < nc && gr[i][i] == 0.0 && gi[i][i] == 0.0 ? 1 << i : 0;
          absent = __builtin_amdgcn_readfirstlane(absent);
          auto leave_out = [&](double diag) {
#pragma unroll
            for (int i = 0; i < NC; ++i)
#pragma unroll
              for (int j = 0; j < NC; ++j)
                if ((absent >> i | absent >> j) & 1) {
                  gr[i][j] = i == j ? diag : 0.0;
                  gi[i][j] = 0.0;
                }
          };
          if (absent) leave_out(1.0);
          // orbitals past nc and frequencies past the tile: X = 1, Sigma' = 0
          if (!whole) {
#pragma unroll
            for (int i = 0; i < NC; ++i)
#pragma unroll
              for (int j = 0; j < NC; ++j) {
                const bool on = valid && i < nc && j < nc;
                gr[i][j] = on ? gr[i][j] : (i == j ? 1.0 : 0.0);
                gi[i][j] = on ? gi[i][j] : 0.0;
              }
          }
          lane_inverse<NC>(gr, gi, pmin);
#pragma unroll
          for (int i = 0; i < NC; ++i) sr[i][i] -= ((const gdouble*)a.e_dc)[min(i, nc - 1)];
          if (!whole) {
#pragma unroll
            for (int i = 0; i < NC; ++i)
#pragma unroll
              for (int j = 0; j < NC; ++j) {
                const bool on = valid && i < nc && j < nc;
                sr[i][j] = on ? sr[i][j] : 0.0;
                si[i][j] = on ? si[i][j] : 0.0;
              }
          }
          if constexpr (oblique) {  // Sigma' of the rows of Q, by way of this lane's part of the matrix area
#pragma unroll
            for (int i = 0; i < NC; ++i) {
              __builtin_amdgcn_sched_barrier(0);  // a row at a time: few registers
#pragma unroll
              for (int j = 0; j < NC; ++j) xb[i * NC + j] = (v2d){sr[i][j], si[i][j]};
            }
            __builtin_amdgcn_sched_barrier(0);
            spec_inner<NC>(xb, spec_lds(sh.lf), 0, NC);
#pragma unroll
            for (int i = 0; i < NC; ++i) {
              __builtin_amdgcn_sched_barrier(0);
#pragma unroll
              for (int j = 0; j < NC; ++j) {
                const v2d x = xb[i * NC + j];
                gr[i][j] -= x.x;
                gi[i][j] -= x.y;
              }
            }
            __builtin_amdgcn_sched_barrier(0);
          } else {
#pragma unroll
            for (int i = 0; i < NC; ++i)
#pragma unroll
              for (int j = 0; j < NC; ++j) {
                gr[i][j] -= sr[i][j];
                gi[i][j] -= si[i][j];
              }
          }
          if (absent) leave_out(1.0);
          lane_inverse<NC>(gr, gi, pmin);
          if (absent) leave_out(0.0);
          if constexpr (oblique) {  // Gl of the rows of S
#pragma unroll
            for (int i = 0; i < NC; ++i) {
              __builtin_amdgcn_sched_barrier(0);  // a row at a time: few registers
#pragma unroll
              for (int j = 0; j < NC; ++j) xb[i * NC + j] = (v2d){gr[i][j], gi[i][j]};
            }
            __builtin_amdgcn_sched_barrier(0);
            spec_outer<NC>(xb, spec_lds(sh.lf), 0, NC);
#pragma unroll
            for (int i = 0; i < NC; ++i) {
              __builtin_amdgcn_sched_barrier(0);
#pragma unroll
              for (int j = 0; j < NC; ++j) {
                const v2d x = xb[i * NC + j];
                gr[i][j] = x.x;
                gi[i][j] = x.y;
              }
            }
            __builtin_amdgcn_sched_barrier(0);
          }
          double chk = 0.0;
#pragma unroll
          for (int i = 0; i < NC; ++i)
#pragma unroll
            for (int j = 0; j < NC; ++j) chk += gr[i][j] + gi[i][j];
          if (!__builtin_isfinite(chk)) nonfinite = 1;
          if (want_x && valid) {
            gv2d* xp = (gv2d*)a.xs + (int64_t)(a.ktile_base + ktile) * NN * nw4 + n;
#pragma unroll
            for (int i = 0; i < NC; ++i) {
              v2d o[NC];
#pragma unroll
              for (int j = 0; j < NC; ++j) {
                o[j] = (v2d){0.0, 0.0};
                if (kk != kk0) o[j] = xp[(int64_t)(i * NC + j) * nw4];
              }
#pragma unroll
              for (int j = 0; j < NC; ++j)
                xp[(int64_t)(i * NC + j) * nw4] =
                    (v2d){__builtin_fma(wk, gr[i][j], o[j].x), __builtin_fma(wk, gi[i][j], o[j].y)};
            }
          }
          if constexpr (WS) {
            double vr[NC][NC], vi[NC][NC];  // Gl Sigma'
#pragma unroll
            for (int i = 0; i < NC; ++i)
#pragma unroll
              for (int j = 0; j < NC; ++j) {
                double x = 0.0, y = 0.0;
#pragma unroll
                for (int m = 0; m < NC; ++m) {
                  x = __builtin_fma(gr[i][m], sr[m][j], __builtin_fma(-gi[i][m], si[m][j], x));
                  y = __builtin_fma(gr[i][m], si[m][j], __builtin_fma(gi[i][m], sr[m][j], y));
                }
                vr[i][j] = x;
                vi[i][j] = y;
              }
            // R (0 past the tile, where Sigma' is), then its Hermitian pairs, in place
#pragma unroll
            for (int i = 0; i < NC; ++i)
#pragma unroll
              for (int j = 0; j < NC; ++j) {
                double x = sr[i][j], y = si[i][j];
#pragma unroll
                for (int m = 0; m < NC; ++m) {
                  x = __builtin_fma(sr[i][m], vr[m][j], __builtin_fma(-si[i][m], vi[m][j], x));
                  y = __builtin_fma(sr[i][m], vi[m][j], __builtin_fma(si[i][m], vr[m][j], y));
                }
                gr[i][j] = x;
                gi[i][j] = y;
              }
#pragma unroll
            for (int i = 0; i < NC; ++i)
#pragma unroll
              for (int j = i; j < NC; ++j) {
                xb[i * NC + j] = (v2d){gr[i][j] + gr[j][i], -(gi[i][j] + gi[j][i])};
                if (i != j) xb[j * NC + i] = (v2d){gi[i][j] - gi[j][i], gr[i][j] - gr[j][i]};
              }
          }
        }
        wave_sync();
        // ---- stage C: rows 2v: d_v^2, rows 2v + 1: d_v d_{v+1}; the next four frequencies'
        // resolvents while this four's products run
        if constexpr (WS) {
          const int l = spec_here(lane), q = l >> 4, c16 = l & 15;
          const lds_double* es = (const lds_double*)&sh.eps[c16];
          const int turns = (min(64, n1 - ng) + 3) >> 2;
          auto table = [&](int c) {
            const int n = ng + 4 * c + q;
            const double wn = (double)(2 * min(n, n1 - 1) + 1) * pib;
            lv2d* dw = spec_lds(&sh.d[c & 1][q * DS + c16]);
#pragma unroll
            for (int m = 0; m < NBP / 16; ++m) {
              const double2 d = inv_z_minus(mu, wn, es[16 * m]);
              dw[16 * m] = (v2d){d.x, d.y};
              sd[m] += n < n1 ? d.x : 0.0;
            }
          };
          table(0);
          wave_sync();
#pragma clang loop unroll(disable)
          for (int c = 0; c < turns; ++c) {
            const lv2d* dr = spec_lds(&sh.d[c & 1][q * DS]);
            const lv2d* hr = spec_lds(&sh.x[(4 * c + q) * LDX]);
            v2d u[NR], v[NR], h[NT];
#pragma unroll
            for (int r = 0; r < NR; ++r) {
              const int row = 16 * r + c16;
              u[r] = dr[row >> 1];
              v[r] = dr[min((row + 1) >> 1, NBP - 1)];
            }
#pragma unroll
            for (int t = 0; t < NT; ++t) h[t] = hr[min(16 * t + c16, NN - 1)];
            if (c + 1 < turns) table(c + 1);
            double fr[NR], fi[NR];
#pragma unroll
            for (int r = 0; r < NR; ++r) {
              fr[r] = u[r].x * v[r].x - u[r].y * v[r].y;
              fi[r] = u[r].x * v[r].y + u[r].y * v[r].x;
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < NT; ++t) {
#pragma unroll
              for (int r = 0; r < NR; ++r) acc[r][t] = mma(fr[r], h[t].x, acc[r][t]);
#pragma unroll
              for (int r = 0; r < NR; ++r) acc[r][t] = mma(fi[r], h[t].y, acc[r][t]);
            }
            wave_sync();
          }
        }
      }
    };
    if (use_q)
      frequencies(std::true_type());
    else
      frequencies(std::false_type());
    // ---- this k-point's sums: tiles in lane order, then sum_n Re d_v
    if constexpr (WS) {
      gdouble* slot = (gdouble*)a.tsum + (int64_t)wtile * a.t_stride + a.t_base + (int64_t)kk * spec_slot_doubles(NBP, NC);
#pragma unroll
      for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i) slot[((r * NT + t) * 4 + i) * 64 + lane] = acc[r][t][i];
#pragma unroll
      for (int m = 0; m < NBP / 16; ++m) {
        sd[m] += __shfl_xor(sd[m], 16);
        sd[m] += __shfl_xor(sd[m], 32);
        if (lane < 16) slot[NR * NT * 256 + 16 * m + lane] = sd[m];
      }
    }
  }
  if (pmin == 0.0) atomicOr(a.err, ERR_SINGULAR);
  if (nonfinite) atomicOr(a.err, ERR_NONFINITE);
}

// One item per wavefront (items null: a0 and blockIdx), or a persistent drain of the
// queue `items` (batched pass).
template <int NBP, int NC, bool WS>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(1)))
spec_lane_kernel(DysonArgs a0, const SpecItem* items, int n_items, const DysonArgs* args, int* counter) {
  __shared__ SpecLaneShared<NBP, NC> sh;
  const int lane = threadIdx.x;
  for (int turn = 0;; ++turn) {
    int kt, wt, ai = 0;
    if (items) {
      int it = 0;
      if (lane == 0) it = atomicAdd(counter, 1);
      it = __builtin_amdgcn_readfirstlane(it);
      if (it >= n_items) break;
      const SpecItem b = items[it];
      ai = b.args;
      kt = b.ktile;
      wt = b.wtile;
    } else {
      if (turn) break;
      kt = blockIdx.x / a0.n_wtiles;
      wt = blockIdx.x % a0.n_wtiles;
    }
    DysonArgs a = a0;
    if (items) a = spec_args(args + ai);
    spec_lane_tile<NBP, NC, WS>(a, kt, wt, sh, lane);
  }
}

}  // namespace dmft
