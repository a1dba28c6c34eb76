// Spectral form of the low-rank Dyson step (gfx950 / CDNA4), density kind.
//
// The low-rank form (lowrank_impl.h) needs, per k-point and frequency, the
// nc x nc matrices X = S D S^dag, Gl = (X^-1 - Sigma')^-1 and
// R = Sigma' + Sigma' Gl Sigma', and G = D + D S^dag R S D.  Here both sums that
// run over the band window become real matrix products whose operands are
// shared by many frequencies or bands:
//
//   X(n)  = sum_v Re d_v(n) P_v + i sum_v Im d_v(n) P_v,       P_v = S_v S_v^dag,
//   sum_n (G + G^dag) = sum_n 2 Re D + [ S_v^dag H(v, v') S_v' ]_{v v'},
//   H(v, v') = sum_n d_v d_v' R + h.c. = sum_n Re(d_v d_v') (R + R^dag) + Im(d_v d_v') i (R - R^dag).
//
// P_v, R + R^dag and i (R - R^dag) are Hermitian, i.e. nc^2 real numbers, stored
// as an nc x nc real matrix: [a][b] with a <= b is Re of element (a, b), with
// a > b Im of element (b, a).  H is needed for every pair of bands, but
// d_v d_v' is the divided difference of 1/(z - E) on (E_v, E_v'), and a divided
// difference is the weighted mean of those of adjacent nodes: with the bands
// sorted by energy and e = E_{j+1} - E_j,
//
//   H(v, v') = sum_{v <= j < v'} e_j H(j, j+1) / (E_v' - E_v)          (v < v'),
//
// positive weights that sum to one, so nothing cancels however close bands
// are.  The frequency loop therefore accumulates only the 2 nb - 1 matrices
// H(v, v) and H(j, j+1) (rows 2v and 2j+1 of one real matrix product over the
// frequencies), and the epilogue (spec_epilogue_kernel) forms N(k) from them
// once per k-point.  Per evaluation the matrix cores run 4 nb nc^2 (X) and
// 8 nb nc^2 (sums) real flops, without the nb x nb or nb x nc complex products
// of the other low-rank kernels.
//
// A work-group of four wavefronts takes a (k-tile, frequency-tile) item and
// walks groups of 16 frequencies; per group
//   A. X of the 16 frequencies (16 x nb by nb x nc^2), each wavefront its share
//      of the nc^2 columns with P_v in registers for the whole k-point;
//   B. each wavefront inverts four frequencies in the row layout (lane
//      16 g + i holds row i of matrix g), adds w_k Gl to the G_loc partial,
//      and writes R as Hermitian pairs;
//   C. the sums H, each wavefront its share of the (2 nb) x nc^2 tiles in
//      accumulation registers, operands d_v d_v' formed from the resolvent table.
// The FP64 matrix and vector units share their rate (72 TFLOP/s measured for a
// large matrix product), so all three stages count: the split keeps A and C on
// full 16x16x4 products and B on uniform row operations.
#pragma once

#include "lowrank_impl.h"

namespace dmft {

// Complex values in global memory (the address space is named because the
// pointers of a queued item come out of a loaded argument block, from which the
// compiler cannot infer it).
typedef double v2d __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(1))) v2d gv2d;
typedef __attribute__((address_space(1))) double gdouble;
typedef __attribute__((address_space(3))) v2d lv2d;
typedef __attribute__((address_space(3))) double lds_double;

// *p += v in the cache that owns the address, nothing returned.
__device__ __forceinline__ void spec_atomic_add(gdouble* p, double v) {
#ifdef __HIP_DEVICE_COMPILE__
  __builtin_amdgcn_global_atomic_fadd_f64(p, v);
#endif
}

// LDS address hidden from the optimizer: the accesses of a stage become this
// register plus an immediate, instead of one loop-invariant address register
// each (which would be spilled across the frequency loop).
__device__ __forceinline__ lv2d* spec_lds(double2* p) {
  lv2d* l = (lv2d*)p;
  asm volatile("" : "+v"(l));
  return l;
}

// f(0), f(1), ... f(N - 1) with compile-time arguments (register arrays are
// indexed by them).
template <int I, int N, class F>
__device__ __forceinline__ void spec_for(const F& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    spec_for<I + 1, N>(f);
  }
}

template <int NBP, int NC>
struct SpecDims {
  static constexpr int T = NBP / 16;
  static constexpr int NR = spec_row_tiles(NBP);
  static constexpr int NT = spec_col_tiles(NC);
  static constexpr int NP = NT * 16;
  // resolvent table: row stride in complex; 4 past a multiple of 16, so that
  // the 16 frequencies read by one instruction of stage A start 64 B apart
  // modulo the 256 B of banks
  static constexpr int DS = NBP + 4;
  // stage A: whole column tiles per wavefront, or where there are fewer than
  // four tiles (tile, Re or Im) jobs
  static constexpr bool SPLIT = NT < 4;
  // P_v of this wavefront's tiles in registers for the whole k-point, or formed
  // from the staged projectors at each use (two vector operations per two products)
  static constexpr bool PREG = SPLIT;
  static constexpr int SS = NBP + 1;  // row stride of the staged projectors
  static constexpr int TPW = SPLIT ? (2 * NT + 3) / 4 : (NT + 3) / 4;
  // stage C: wavefronts along rows x along columns, the smallest share of the busiest one
  static constexpr int share(int wr) { return ((NR + wr - 1) / wr) * ((NT + 4 / wr - 1) / (4 / wr)); }
  static constexpr int WR = (share(4) <= share(2) && share(4) <= share(1)) ? 4 : (share(2) <= share(1) ? 2 : 1);
  static constexpr int WC = 4 / WR;
  static constexpr int RT = (NR + WR - 1) / WR;
  static constexpr int CT = (NT + WC - 1) / WC;
};

template <int NBP, int NC>
struct SpecShared {
  using Dm = SpecDims<NBP, NC>;
  // X, then R, of the group's frequencies ([n][nc^2] Hermitian pairs; one tile of
  // slack for wavefronts whose share of the columns ends past the last tile)
  double2 xr[16 * Dm::NP + 16 * Dm::WC];
  double2 dt[2][16 * Dm::DS];     // d_v(n) of this group and the next
  // projectors, columns sorted by energy: S = (x, y), and (y, -x)
  double2 sp[Dm::PREG ? 1 : 2 * NC * Dm::SS];
  double sd[NBP * 17];            // running sum of Re d_v per (band, frequency of the group)
  double eps[NBP];                // sorted band energies
  unsigned long long key[NBP];
  int rank[NBP];
  int next;
};

// Order-preserving integer image of a double (a total order, NaN included, so
// that the ranks are a permutation for any input).
__device__ __forceinline__ unsigned long long spec_key(double e) {
  const unsigned long long b = __double_as_longlong(e);
  return b ^ ((b >> 63) ? ~0ull : (1ull << 63));
}

// Rank of band v among the nb keys (ties by index).
__device__ __forceinline__ int spec_rank(const unsigned long long* key, int v, int nb) {
  const unsigned long long kv = key[v];
  int r = 0;
  for (int u = 0; u < nb; ++u) r += (key[u] < kv || (key[u] == kv && u < v)) ? 1 : 0;
  return r;
}

// Hides a lane index from the optimizer, so that the addresses formed from it
// are computed where they are used instead of being kept (or spilled) in
// registers across the frequency loop.
__device__ __forceinline__ int spec_here(int i) {
  asm volatile("" : "+v"(i));
  return i;
}

// Columns of a Gauss-Jordan step: (r, i) -= l (row K's (r, i) of this 16-lane
// row).  Four of the five multiply-adds and moves of a column take the broadcast
// as their DPP operand; row K's imaginary part is moved out first because its
// register changes before its last use.  The leading s_nop covers the two wait
// states a DPP read needs after the vector instruction that wrote its source
// (it costs 3 ns, a multiply-add 2 ns: hence four columns per block); the
// operands are early-clobbered because outputs are written before all inputs
// have been read.
#define SPEC_BC(K) " row_newbcast:%" #K " row_mask:0xf bank_mask:0xf\n\t"
template <int K>
__device__ __forceinline__ void row_elim4(double& r0, double& i0, double& r1, double& i1, double& r2, double& i2,
                                          double& r3, double& i3, double lr, double li) {
  double t0, t1, t2, t3;
  asm("s_nop 1\n\t"
      "v_mov_b64_dpp %8, %4" SPEC_BC(14) "v_mov_b64_dpp %9, %5" SPEC_BC(14)
      "v_mov_b64_dpp %10, %6" SPEC_BC(14) "v_mov_b64_dpp %11, %7" SPEC_BC(14)
      "v_fmac_f64_dpp %4, -%0, %13" SPEC_BC(14) "v_fmac_f64_dpp %5, -%1, %13" SPEC_BC(14)
      "v_fmac_f64_dpp %6, -%2, %13" SPEC_BC(14) "v_fmac_f64_dpp %7, -%3, %13" SPEC_BC(14)
      "v_fmac_f64_dpp %0, -%0, %12" SPEC_BC(14) "v_fmac_f64_dpp %1, -%1, %12" SPEC_BC(14)
      "v_fmac_f64_dpp %2, -%2, %12" SPEC_BC(14) "v_fmac_f64_dpp %3, -%3, %12" SPEC_BC(14)
      "v_fma_f64 %4, -%8, %12, %4\n\tv_fma_f64 %5, -%9, %12, %5\n\t"
      "v_fma_f64 %6, -%10, %12, %6\n\tv_fma_f64 %7, -%11, %12, %7\n\t"
      "v_fmac_f64 %0, %8, %13\n\tv_fmac_f64 %1, %9, %13\n\tv_fmac_f64 %2, %10, %13\n\tv_fmac_f64 %3, %11, %13"
      : "+&v"(r0), "+&v"(r1), "+&v"(r2), "+&v"(r3), "+&v"(i0), "+&v"(i1), "+&v"(i2), "+&v"(i3), "=&v"(t0), "=&v"(t1),
        "=&v"(t2), "=&v"(t3)
      : "v"(lr), "v"(li), "i"(K));
}
template <int K>
__device__ __forceinline__ void row_elim1(double& r, double& i, double lr, double li) {
  double t;
  asm("s_nop 1\n\t"
      "v_mov_b64_dpp %2, %1" SPEC_BC(5)
      "v_fmac_f64_dpp %1, -%0, %4" SPEC_BC(5)
      "v_fmac_f64_dpp %0, -%0, %3" SPEC_BC(5)
      "v_fma_f64 %1, -%2, %3, %1\n\tv_fmac_f64 %0, %2, %4"
      : "+&v"(r), "+&v"(i), "=&v"(t)
      : "v"(lr), "v"(li), "i"(K));
}
#undef SPEC_BC

// Gauss-Jordan steps K .. NC-1 of the row layout (rows and columns past nc hold
// the identity).  pmin: the smallest |pivot|^2 so far.  The reciprocal is the
// hardware estimate (2^-23) and one third-order step.
template <int K, int NC>
struct SpecStep {
  static constexpr int col(int m) { return m < K ? m : m + 1; }
  template <int M>
  static __device__ __forceinline__ void cols(double (&rr)[NC], double (&ri)[NC], double lr, double li) {
    if constexpr (M + 4 <= NC - 1) {
      constexpr int a = col(M), b = col(M + 1), c = col(M + 2), d = col(M + 3);
      row_elim4<K>(rr[a], ri[a], rr[b], ri[b], rr[c], ri[c], rr[d], ri[d], lr, li);
      cols<M + 4>(rr, ri, lr, li);
    } else if constexpr (M < NC - 1) {
      row_elim1<K>(rr[col(M)], ri[col(M)], lr, li);
      cols<M + 1>(rr, ri, lr, li);
    }
  }
  static __device__ __forceinline__ void run(double (&rr)[NC], double (&ri)[NC], int i, double& pmin) {
    const double px = row_bcast<K>(rr[K]), py = row_bcast<K>(ri[K]);
    const double d = __builtin_fma(px, px, py * py);
    pmin = __builtin_fmin(pmin, d);
    double t = __builtin_amdgcn_rcp(d);
    const double e = __builtin_fma(-d, t, 1.0);
    t = __builtin_fma(t, __builtin_fma(e, e, e), t);
    const double ix = px * t, iy = -py * t;
    const double cr = __builtin_fma(-ri[K], iy, rr[K] * ix), ci = __builtin_fma(ri[K], ix, rr[K] * iy);
    const bool piv = i == K;
    cols<0>(rr, ri, piv ? 1.0 - ix : cr, piv ? -iy : ci);
    rr[K] = piv ? ix : -cr;
    ri[K] = piv ? iy : -ci;
    if constexpr (K + 1 < NC) SpecStep<K + 1, NC>::run(rr, ri, i, pmin);
  }
};
template <int NC>
__device__ __forceinline__ void spec_sweep(double (&rr)[NC], double (&ri)[NC], int i, double& pmin) {
  SpecStep<0, NC>::run(rr, ri, i, pmin);
}

// (c_j) += (row K's b_j of this 16-lane row) x for two columns j, complex: the
// broadcast is the DPP operand of the multiply-add itself, so it costs no move
// (s_nop and early clobbers as above).
template <int K>
__device__ __forceinline__ void row_fmac2(double& c0r, double& c0i, double& c1r, double& c1i, double b0r, double b0i,
                                          double b1r, double b1i, double xr, double xi) {
  asm("s_nop 1\n\t"
      "v_fmac_f64_dpp %0, %4, %8 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %5, %8 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %2, %6, %8 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, %7, %8 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, -%5, %9 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %4, %9 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %2, -%7, %9 row_newbcast:%10 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, %6, %9 row_newbcast:%10 row_mask:0xf bank_mask:0xf"
      : "+&v"(c0r), "+&v"(c0i), "+&v"(c1r), "+&v"(c1i)
      : "v"(b0r), "v"(b0i), "v"(b1r), "v"(b1i), "v"(xr), "v"(xi), "i"(K));
}
// The same for one column.
template <int K>
__device__ __forceinline__ void row_fmac1(double& cr, double& ci, double br, double bi, double xr, double xi) {
  asm("s_nop 1\n\t"
      "v_fmac_f64_dpp %0, %2, %4 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %3, %4 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %0, -%3, %5 row_newbcast:%6 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %1, %2, %5 row_newbcast:%6 row_mask:0xf bank_mask:0xf"
      : "+&v"(cr), "+&v"(ci)
      : "v"(br), "v"(bi), "v"(xr), "v"(xi), "i"(K));
}
// The same for four columns and rows K, K + 1.
template <int K>
__device__ __forceinline__ void row_fmac4(double (&cr)[4], double (&ci)[4], const double* br, const double* bi,
                                          double xr, double xi, double yr, double yi) {
#define SPEC_FM(D, S, X, KK) "v_fmac_f64_dpp %" #D ", " #S ", %" #X " row_newbcast:%" #KK " row_mask:0xf bank_mask:0xf\n\t"
  asm("s_nop 1\n\t"
      SPEC_FM(0, %8, 16, 20) SPEC_FM(1, %9, 16, 20) SPEC_FM(2, %10, 16, 20) SPEC_FM(3, %11, 16, 20)
      SPEC_FM(4, %12, 16, 20) SPEC_FM(5, %13, 16, 20) SPEC_FM(6, %14, 16, 20) SPEC_FM(7, %15, 16, 20)
      SPEC_FM(0, -%12, 17, 20) SPEC_FM(1, -%13, 17, 20) SPEC_FM(2, -%14, 17, 20) SPEC_FM(3, -%15, 17, 20)
      SPEC_FM(4, %8, 17, 20) SPEC_FM(5, %9, 17, 20) SPEC_FM(6, %10, 17, 20) SPEC_FM(7, %11, 17, 20)
      SPEC_FM(0, %8, 18, 21) SPEC_FM(1, %9, 18, 21) SPEC_FM(2, %10, 18, 21) SPEC_FM(3, %11, 18, 21)
      SPEC_FM(4, %12, 18, 21) SPEC_FM(5, %13, 18, 21) SPEC_FM(6, %14, 18, 21) SPEC_FM(7, %15, 18, 21)
      SPEC_FM(0, -%12, 19, 21) SPEC_FM(1, -%13, 19, 21) SPEC_FM(2, -%14, 19, 21) SPEC_FM(3, -%15, 19, 21)
      SPEC_FM(4, %8, 19, 21) SPEC_FM(5, %9, 19, 21) SPEC_FM(6, %10, 19, 21) SPEC_FM(7, %11, 19, 21)
      : "+&v"(cr[0]), "+&v"(cr[1]), "+&v"(cr[2]), "+&v"(cr[3]), "+&v"(ci[0]), "+&v"(ci[1]), "+&v"(ci[2]), "+&v"(ci[3])
      : "v"(br[0]), "v"(br[1]), "v"(br[2]), "v"(br[3]), "v"(bi[0]), "v"(bi[1]), "v"(bi[2]), "v"(bi[3]),
        "v"(xr), "v"(xi), "v"(yr), "v"(yi), "i"(K), "i"(K + 1));
#undef SPEC_FM
}

// c[j] += sum_k x[k] (b[j] of row k), j = 0 .. JB-1: rows of a matrix product in the row layout.
template <int K, int NC, int JB>
__device__ __forceinline__ void row_mac(double (&cr)[JB], double (&ci)[JB], const double (&xr)[NC],
                                        const double (&xi)[NC], const double* br, const double* bi) {
  if constexpr (K < NC) {
    if constexpr (JB == 4 && K + 1 < NC) {
      row_fmac4<K>(cr, ci, br, bi, xr[K], xi[K], xr[K + 1], xi[K + 1]);
      row_mac<K + 2, NC, JB>(cr, ci, xr, xi, br, bi);
    } else {
#pragma unroll
      for (int j = 0; j + 1 < JB; j += 2)
        row_fmac2<K>(cr[j], ci[j], cr[j + 1], ci[j + 1], br[j], bi[j], br[j + 1], bi[j + 1], xr[K], xi[K]);
      if constexpr (JB % 2) row_fmac1<K>(cr[JB - 1], ci[JB - 1], br[JB - 1], bi[JB - 1], xr[K], xi[K]);
      row_mac<K + 1, NC, JB>(cr, ci, xr, xi, br, bi);
    }
  }
}

// One column block of V = Gl Sigma' and R = Sigma' + Sigma' V (row layout), R to LDS.
template <int J0, int NC>
__device__ __forceinline__ void spec_r_blocks(const double (&gr)[NC], const double (&gi)[NC], const double (&sr)[NC],
                                              const double (&si)[NC], bool valid, int i, lv2d* xb) {
  if constexpr (J0 < NC) {
    constexpr int JB = (NC - J0) < 4 ? (NC - J0) : 4;
    double vr[JB], vi[JB], rr[JB], ri[JB];
#pragma unroll
    for (int j = 0; j < JB; ++j) {
      vr[j] = vi[j] = 0.0;
      rr[j] = sr[J0 + j];
      ri[j] = si[J0 + j];
    }
    row_mac<0, NC, JB>(vr, vi, gr, gi, sr + J0, si + J0);
    row_mac<0, NC, JB>(rr, ri, sr, si, vr, vi);
    if (i < NC) {
#pragma unroll
      for (int j = 0; j < JB; ++j) xb[i * NC + J0 + j] = valid ? (v2d){rr[j], ri[j]} : (v2d){0.0, 0.0};
    }
    spec_r_blocks<J0 + JB, NC>(gr, gi, sr, si, valid, i, xb);
  }
}

// WS: the sums are wanted (N(k)); else G_loc only.
template <int NBP, int NC, bool WS>
__device__ __forceinline__ void spec_tile(const DysonArgs& a, int ktile, int wtile, SpecShared<NBP, NC>& sh, int tid) {
  using Dm = SpecDims<NBP, NC>;
  constexpr int T = Dm::T, NT = Dm::NT, NP = Dm::NP, DS = Dm::DS, TPW = Dm::TPW;
  constexpr int WR = Dm::WR, WC = Dm::WC, RT = Dm::RT, CT = Dm::CT, NR = Dm::NR;
  constexpr bool SPLIT = Dm::SPLIT;
  const int w = uniform_i(tid >> 6), wr = w % WR, wc = w / WR;
  const int n0 = wtile * a.wt, n1 = min(n0 + a.wt, a.nw);
  const int kk0 = ktile * a.kt, kk1 = min(kk0 + a.kt, a.nklist);
  const double mu = uniform_d(a.mu_ptr ? *a.mu_ptr : a.mu);
  const double beta = a.beta;
  const int nc = a.nc;
  __builtin_assume(nc >= 1 && nc <= NC);
  const bool want_x = a.mode & MODE_GLOC;
  const int n4_all = (a.nw + 3) >> 2;
  const double pib = M_PI / beta;
  const double edc = (tid & 15) < nc ? ((const gdouble*)a.e_dc)[tid & 15] : 0.0;  // V_DC of the row-layout row
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

    // ---- bands sorted by energy, projector columns in that order (staged over xr)
    __syncthreads();
    if (tid < NBP) sh.key[tid] = tid < nb ? spec_key(eps[tid]) : ~0ull;
    __syncthreads();
    if (tid < NBP) {
      const int r = tid < nb ? spec_rank(sh.key, tid, nb) : tid;
      sh.rank[tid] = r;
      sh.eps[r] = tid < nb ? eps[tid] : mu;
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
    // P_v of this wavefront's tiles as B operand: band 4 c + q, column 16 t + c16
    // = (al, be): Re S_al S_be^* for al <= be, else Im S_be S_al^*
    double p[Dm::PREG ? TPW : 1][Dm::PREG ? NBP / 4 : 1];
    int pab[TPW];  // both addresses of the staged projectors, 16 bits each
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
    // resolvent table of the group starting at ng (frequencies past the tile repeat
    // the last one and add nothing to the sum)
    auto fill_d = [&](int ng, double2* dt0, bool first) {
      const int t = spec_here(tid), nl = t & 15, v0 = t >> 4;
      const double wn = (double)(2 * min(ng + nl, n1 - 1) + 1) * pib;
      lv2d* dt = spec_lds(dt0 + nl * DS + v0);
      lds_double* sd = (lds_double*)&sh.sd[v0 * 17 + nl];
      const lds_double* es = (const lds_double*)&sh.eps[v0];
#pragma unroll
      for (int m = 0; m < T; ++m) {
        const double2 d = inv_z_minus(mu, wn, es[16 * m]);
        dt[16 * m] = (v2d){d.x, d.y};
        sd[16 * 17 * m] = (first ? 0.0 : sd[16 * 17 * m]) + (ng + nl < n1 ? d.x : 0.0);
      }
    };
    fill_d(n0, sh.dt[0], true);
    __syncthreads();

    v4d acc[RT][CT];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int t = 0; t < CT; ++t) acc[r][t] = (v4d){0.0, 0.0, 0.0, 0.0};

    int cur = 0;
    for (int ng = n0; ng < n1; ng += 16, cur ^= 1) {
      // row c16 of Sigma of this lane's stage-B frequency, in flight during stage A
      // (rows and columns past nc repeat the last one and are cleared below)
      double sr[NC], si[NC];
      {
        const int l = spec_here(tid & 63), i = min(l & 15, nc - 1), n = min(ng + 4 * w + (l >> 4), n1 - 1);
        const gv2d* sgp = (const gv2d*)a.sigma + ((int64_t)n * nc + i) * nc;
#pragma unroll
        for (int j = 0; j < NC; ++j) {
          const v2d v = sgp[min(j, nc - 1)];
          sr[j] = v.x;
          si[j] = v.y;
        }
      }
      // ---- stage A (a wavefront with fewer jobs repeats its last column: the others set the time)
      {
        const int l = spec_here(tid & 63), q = l >> 4, c16 = l & 15;
        const lv2d* dt = spec_lds(&sh.dt[cur][c16 * DS + q]);
        v4d xa[TPW][SPLIT ? 1 : 2];
        const lv2d *sa[TPW], *sb[TPW];
#pragma unroll
        for (int m = 0; m < TPW; ++m) {
          if constexpr (!Dm::PREG) {
            const int ab = spec_here(pab[m]);
            sa[m] = spec_lds(&sh.sp[ab & 0xffff]);
            sb[m] = spec_lds(&sh.sp[ab >> 16]);
          }
#pragma unroll
          for (int h = 0; h < (SPLIT ? 1 : 2); ++h) xa[m][h] = (v4d){0.0, 0.0, 0.0, 0.0};
        }
        // operands one band chunk ahead: two products take 128 cycles, about an LDS
        // round trip, so loads issued at their use would be waited for every time
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
#pragma unroll
          for (int m = 0; m < TPW; ++m) {
            double pv;
            if constexpr (Dm::PREG)
              pv = p[m][c];
            else
              pv = __builtin_fma(x[c & 1][m].x, y[c & 1][m].x, x[c & 1][m].y * y[c & 1][m].y);
            if constexpr (SPLIT) {
              xa[m][0] = mma((w & 1) ? d[c & 1].y : d[c & 1].x, pv, xa[m][0]);
            } else {
              xa[m][0] = mma(d[c & 1].x, pv, xa[m][0]);
              xa[m][1] = mma(d[c & 1].y, pv, xa[m][1]);
            }
          }
        });
        __syncthreads();  // the previous group's stage C has read xr
        lv2d* xw = spec_lds(&sh.xr[q * NP + c16]);
#pragma unroll
        for (int m = 0; m < TPW; ++m) {
          const int job = w + 4 * m;
          if (job >= (SPLIT ? 2 * NT : NT)) break;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            if constexpr (SPLIT)
              ((__attribute__((address_space(3))) double*)(xw + 4 * i * NP + 16 * (job >> 1)))[job & 1] = xa[m][0][i];
            else
              xw[4 * i * NP + 16 * job] = (v2d){xa[m][0][i], xa[m][1][i]};
          }
        }
      }
      __syncthreads();
      // ---- stage B: four matrices per wavefront in the row layout
      {
        const int l = spec_here(tid & 63), i = l & 15, nl = 4 * w + (l >> 4);
        const bool valid = ng + nl < n1;
        const int ic = min(i, NC - 1);
        lv2d* xb = spec_lds(&sh.xr[nl * NP]);
        double rr[NC], ri[NC];
        // row i of X from its Hermitian pairs (lanes past the NC rows repeat the last
        // one; nothing of theirs is read by another lane or kept)
        {
          v2d re[NC], im[NC];
#pragma unroll
          for (int j = 0; j < NC; ++j) {
            const int lo = min(ic, j), hi = max(ic, j);
            re[j] = xb[lo * NC + hi];
            im[j] = xb[hi * NC + lo];
          }
          __builtin_amdgcn_sched_barrier(0);  // every read issued before the first is waited for
#pragma unroll
          for (int j = 0; j < NC; ++j) {
            const double s = ic < j ? 1.0 : (ic > j ? -1.0 : 0.0);
            rr[j] = __builtin_fma(-s, im[j].y, re[j].x);
            ri[j] = __builtin_fma(s, im[j].x, re[j].y);
          }
        }
        if (nc < NC) {
#pragma unroll
          for (int j = 0; j < NC; ++j) {
            rr[j] = i < nc ? rr[j] : (i == j ? 1.0 : 0.0);
            ri[j] = i < nc ? ri[j] : 0.0;
          }
        }
        spec_sweep<NC>(rr, ri, i, pmin);
        if (nc < NC) {
#pragma unroll
          for (int j = 0; j < NC; ++j) {
            sr[j] = i < nc && j < nc ? sr[j] : 0.0;
            si[j] = i < nc && j < nc ? si[j] : 0.0;
          }
        }
#pragma unroll
        for (int j = 0; j < NC; ++j) {
          sr[j] -= i == j ? edc : 0.0;
          rr[j] -= sr[j];
          ri[j] -= si[j];
        }
        spec_sweep<NC>(rr, ri, i, pmin);
        // w_k Gl into this lane's row of the G_loc partial (column stride 4 NC):
        // written at the tile's first k-point, then added with memory atomics.  No
        // other work-group touches the address, so the order of the additions is
        // the k order and the sum reproducible; unlike a load and a store, the
        // atomics hold no registers and nothing waits for them.
        if (want_x && valid && i < NC) {
          gdouble* gp = (gdouble*)a.xs +
                        2 * (((int64_t)(a.ktile_base + ktile) * n4_all + (ng >> 2) + w) * (4 * NC * NC) + (nl & 3) * NC + i);
          if (kk == kk0) {
#pragma unroll
            for (int j = 0; j < NC; ++j) *(gv2d*)(gp + 8 * NC * j) = (v2d){wk * rr[j], wk * ri[j]};
          } else {
#pragma unroll
            for (int j = 0; j < NC; ++j) {
              spec_atomic_add(gp + 8 * NC * j, wk * rr[j]);
              spec_atomic_add(gp + 8 * NC * j + 1, wk * ri[j]);
            }
          }
        }
        double chk = 0.0;
#pragma unroll
        for (int j = 0; j < NC; ++j) chk += rr[j] + ri[j];
        if (i < NC && !__builtin_isfinite(chk)) nonfinite = 1;
        wave_sync();
        if constexpr (WS) spec_r_blocks<0, NC>(rr, ri, sr, si, valid, i, xb);
        wave_sync();
        if constexpr (WS) {
          // R -> (R + R^dag, i (R - R^dag)) as Hermitian pairs, in place: lane i takes the
          // unordered pairs (i, i + r mod NC); all are read before any is written (and the
          // two lanes that share a pair at r = NC / 2 write the same values)
          v2d u[NC / 2 + 1], v[NC / 2 + 1];
#pragma unroll
          for (int r = 0; r <= NC / 2; ++r) {
            const int j = ic + r >= NC ? ic + r - NC : ic + r;
            u[r] = xb[min(ic, j) * NC + max(ic, j)];
            v[r] = xb[max(ic, j) * NC + min(ic, j)];
          }
          wave_sync();
          if (ng + 16 < n1) fill_d(ng + 16, sh.dt[cur ^ 1], false);  // while the pairs arrive
          if (i < NC) {
#pragma unroll
            for (int r = 0; r <= NC / 2; ++r) {
              const int j = i + r >= NC ? i + r - NC : i + r;
              if (r) xb[max(i, j) * NC + min(i, j)] = (v2d){u[r].y - v[r].y, u[r].x - v[r].x};
              xb[min(i, j) * NC + max(i, j)] = (v2d){u[r].x + v[r].x, -(u[r].y + v[r].y)};
            }
          }
        } else {
          if (ng + 16 < n1) fill_d(ng + 16, sh.dt[cur ^ 1], false);
        }
      }
      __syncthreads();
      // ---- stage C: rows 2v: d_v^2, rows 2v + 1: d_v d_{v+1}
      if constexpr (WS) {
        const int l = spec_here(tid & 63), q = l >> 4, c16 = l & 15;
        const lv2d* xc = spec_lds(&sh.xr[q * NP + c16 + 16 * wc]);
        const lv2d *d1[RT], *d2[RT];
#pragma unroll
        for (int r = 0; r < RT; ++r) {
          const int row = 16 * (wr + WR * r) + c16;  // rows past 2 nb - 2 are never read
          d1[r] = spec_lds(&sh.dt[cur][q * DS + min(row >> 1, NBP - 1)]);
          d2[r] = spec_lds(&sh.dt[cur][q * DS + min((row + 1) >> 1, NBP - 1)]);
        }
        // operands one chunk of four frequencies ahead, as in stage A
        v2d h[2][CT], x[2][RT], y[2][RT];
        auto fetch = [&](int c, int s) {
#pragma unroll
          for (int r = 0; r < RT; ++r) {
            x[s][r] = d1[r][4 * c * DS];
            y[s][r] = d2[r][4 * c * DS];
          }
#pragma unroll
          for (int t = 0; t < CT; ++t) h[s][t] = xc[4 * c * NP + 16 * WC * t];
        };
        fetch(0, 0);
        spec_for<0, 4>([&](auto ci) {
          constexpr int c = decltype(ci)::value;
          if constexpr (c < 3) fetch(c + 1, (c + 1) & 1);
          __builtin_amdgcn_sched_barrier(0);
          double fr[RT], fi[RT];
#pragma unroll
          for (int r = 0; r < RT; ++r) {
            fr[r] = x[c & 1][r].x * y[c & 1][r].x - x[c & 1][r].y * y[c & 1][r].y;
            fi[r] = x[c & 1][r].x * y[c & 1][r].y + x[c & 1][r].y * y[c & 1][r].x;
          }
#pragma unroll
          for (int t = 0; t < CT; ++t) {
#pragma unroll
            for (int r = 0; r < RT; ++r) acc[r][t] = mma(fr[r], h[c & 1][t].x, acc[r][t]);
#pragma unroll
            for (int r = 0; r < RT; ++r) acc[r][t] = mma(fi[r], h[c & 1][t].y, acc[r][t]);
          }
        });
      }
    }
    // ---- this k-point's sums: tiles in lane order, then sum_n Re d_v
    if constexpr (WS) {
      gdouble* slot = (gdouble*)a.tsum + (int64_t)wtile * a.t_stride + a.t_base + (int64_t)kk * spec_slot_doubles(NBP, NC);
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        const int rt = wr + WR * r;
#pragma unroll
        for (int t = 0; t < CT; ++t) {
          const int ct = wc + WC * t;
          if (rt < NR && ct < NT) {
#pragma unroll
            for (int i = 0; i < 4; ++i) slot[((rt * NT + ct) * 4 + i) * 64 + (tid & 63)] = acc[r][t][i];
          }
        }
      }
      __syncthreads();
      if (tid < NBP) {
        double s = 0.0;
#pragma unroll
        for (int j = 0; j < 16; ++j) s += sh.sd[tid * 17 + j];
        slot[NR * NT * 256 + tid] = s;
      }
    }
  }
  if (pmin == 0.0 && (tid & 15) < NC) atomicOr(a.err, ERR_SINGULAR);
  if (nonfinite) atomicOr(a.err, ERR_NONFINITE);
}

struct SpecItem {
  int32_t args, nbp, ktile, wtile;
};

// A queued item's arguments, read through the constant address space so that
// they stay in scalar registers.
__device__ __forceinline__ DysonArgs spec_args(const DysonArgs* p) {
#ifdef __HIP_DEVICE_COMPILE__
  return *(const __attribute__((address_space(4))) DysonArgs*)p;
#else
  return *p;
#endif
}

// One item per work-group (items null: a0 and blockIdx), or a persistent
// drain of the queue `items` (batched pass).
template <int NBP, int NC, bool WS>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WS ? spec_wgs_per_cu(NBP, NC) : 1)))
spec_kernel(DysonArgs a0, const SpecItem* items, int n_items, const DysonArgs* args, int* counter) {
  __shared__ SpecShared<NBP, NC> sh;
  const int tid = threadIdx.x;
  for (int turn = 0;; ++turn) {
    int kt, wt, ai = 0;
    if (items) {
      __syncthreads();
      if (tid == 0) sh.next = atomicAdd(counter, 1);
      __syncthreads();
      const int it = __builtin_amdgcn_readfirstlane(sh.next);
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
    spec_tile<NBP, NC, WS>(a, kt, wt, sh, tid);
  }
}

}  // namespace dmft
