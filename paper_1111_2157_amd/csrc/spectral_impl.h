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
// positive weights that sum to one, so close bands cost no digits.  The matrices
// H(j, j+1) themselves change sign across mu, and between distant bands on either
// side H(v, v') is smaller than its terms: single elements of N(k) lose that ratio
// (48 bands, beta 4000: 3e-12 of an element against 8e-14 of the band-window inversion),
// the matrix does not (2e-14 against 1e-15, against 80-bit values).  The frequency
// loop therefore accumulates only the 2 nb - 1 matrices H(v, v) and H(j, j+1) (rows
// 2v and 2j+1 of one real matrix product over the frequencies), and the epilogue (spec_epilogue_kernel) forms N(k) from them
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
//
// Measured (512 k-points, 2048 frequencies, per k-point and frequency; in brackets
// the frequency-at-a-time low-rank kernels, tuned): 32 bands and 10 orbitals 2.41 ns
// (5.3), 48 and 14 5.35 (10.2), 64 and 14 6.01.  At 48 and 14 the matrix products with
// their padding would take 2.0 ns at full rate and the row operations of B 2.1; what
// bounds the rest is that the two units do not run FP64 together and a SIMD holds one
// wavefront (its row matrices, sums and operands fill the registers), so the LDS round
// trips between the stages and the changes between the units are exposed.  Up to five
// orbitals spectral_lane_impl.h takes over.
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
  double2 lf[NC * NC];            // L of S = L Q where Q is used
  int rank[NBP];
  int oblique, use_q;             // the rows of S are looked at closer; Q stands in their place
  int next;
  static __device__ __forceinline__ double2* scratch(SpecShared& sh) { return sh.dt[0]; }  // filled later
};

// Smallest energy step the weighted mean of adjacent sums resolves: steps below
// it (equal energies) count as this much, so that a group of equal energies gets
// the plain mean of its sums instead of 0 / 0.
constexpr double kTinyStep = 1e-200;

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

// ---- oblique projector rows.  X^-1 - Sigma' loses the square of the condition number of S:
// rows that are nearly (or exactly) dependent would leave it no digits.  S = L Q with
// orthonormal (or zero) rows of Q and lower triangular L takes that number out of the
// inversions, X = Q D Q^dag then being as well conditioned as for orthonormal projectors:
//   Gl = L (X^-1 - L^dag Sigma' L)^-1 L^dag,
// four more row products per evaluation, so only a k-point whose rows call for it is
// taken this way.  (6 to 48 bands, one singular value of S from 1 down to 1e-13, or equal
// rows, beta 40 and 1000: G_loc within 2e-12 of 80-bit values and N(k) within 5e-13, as the
// band-window inversion (2e-13, 8e-14); with S itself 1e-8 at a singular value of 1e-4.
// All k-points in Q against none: density passes of 64 k-points, 12 bands, 5 orbitals, 256
// frequencies 78 us against 49, of 256, 48, 14, 512 1.73 ms against 0.86; the band-window
// kernels 158 us and 7.9 ms.  Rows that are looked at closer and keep their basis: 58 us and
// 0.97 ms.)

// Whether two rows may ask for it, by the real or imaginary part z of their product and
// their squared norms, or (same) one row by its own: past |z| = |x| |y| / (3 nc) (below it
// the Gram matrix of the normalised rows has its eigenvalues in 1/2 .. 3/2), or at a norm
// far from 1 (a pivot p leaves its row about max(1, |p|) roundings, see SpecStep, and the
// second inversion's pivots go with one over the squared norm: G_loc, 24 bands, 8 orbitals,
// beta 40, within 4e-15 at norm 1, 1e-14 at 0.3, 6e-14 at 0.1 and 3e-12 at 0.011 in their
// own basis; the band-window kernels 1e-15).  Zero rows do not (row_absent), nor do NaN
// (they reach the error word).
__device__ __forceinline__ bool spec_far(double xx) { return xx > 0.0 && !(xx >= 0.0625 && xx <= 1e4); }
__device__ __forceinline__ bool spec_oblique(double xx, double yy, double z, bool same, int nc) {
  return same ? spec_far(xx) : z * z * (9.0 * nc * nc) > xx * yy;
}

// Sums over the four lanes of a quad, and over a wavefront.
__device__ __forceinline__ double spec_quad_sum(double v) {
  v += __builtin_amdgcn_update_dpp(0.0, v, 0xB1, 0xf, 0xf, true);  // quad_perm 1, 0, 3, 2
  return v + __builtin_amdgcn_update_dpp(0.0, v, 0x4E, 0xf, 0xf, true);  // quad_perm 2, 3, 0, 1
}
__device__ __forceinline__ double spec_wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// S = L Q by one wavefront, a band per lane: Gram-Schmidt, every row twice against all
// before it.  s: the rows in LDS (stride ss, zeros past the window), replaced by Q; a row
// within 3.6e-15 of the span of those before it gets a zero row of Q.  Returns whether Q is
// to be used: a row dropped or of a far norm, or tr (S S^dag)^-1 of the normalised rows, the
// factor by which roundings in X^-1 grow, over 64 (nc for orthonormal rows).  y: scratch of
// NC * NC.
template <int NBP, int NC>
__device__ __forceinline__ bool spec_orthonormal(double2* s, int ss, double2* lf, double2* y, int nc, int lane) {
  const int j = lane & 15, h = lane >> 4;
  double norm = 1.0, f = 0.0;  // |row j|; this lane's share of the trace
  bool use = false;
#pragma clang loop unroll(disable)
  for (int i = 0; i < NC; ++i) {
    double2 r = lane < NBP && i < nc ? s[i * ss + lane] : make_double2(0.0, 0.0);
    const double n0 = spec_wave_sum(r.x * r.x + r.y * r.y);
    double2 l = make_double2(0.0, 0.0);  // element (i, j) of L
#pragma clang loop unroll(disable)
    for (int pass = 0; pass < 2 && i < nc; ++pass) {
      double2 c = make_double2(0.0, 0.0);  // row j of Q against this one
      if (j < i)
#pragma clang loop unroll(disable)
        for (int v = h; v < NBP; v += 4) {
          const double2 a = s[j * ss + v], b = s[i * ss + v];
          c.x += a.x * b.x + a.y * b.y;
          c.y += a.x * b.y - a.y * b.x;
        }
      c.x += __shfl_xor(c.x, 16);
      c.y += __shfl_xor(c.y, 16);
      c.x += __shfl_xor(c.x, 32);
      c.y += __shfl_xor(c.y, 32);
      l.x += c.x;
      l.y += c.y;
#pragma clang loop unroll(disable)
      for (int m = 0; m < i; ++m) {
        const double cx = __shfl(c.x, m), cy = __shfl(c.y, m);
        const double2 a = s[m * ss + min(lane, NBP - 1)];
        r.x -= cx * a.x - cy * a.y;
        r.y -= cx * a.y + cy * a.x;
      }
      wave_sync();
      if (lane < NBP) s[i * ss + lane] = r;
      wave_sync();
    }
    const double n = spec_wave_sum(lane < NBP ? r.x * r.x + r.y * r.y : 0.0);
    const bool drop = n <= 1.3e-29 * n0 && __builtin_isfinite(n0);  // not for NaN or infinity: they stay visible
    const double len = drop ? 0.0 : __builtin_sqrt(n), inv = drop ? 0.0 : 1.0 / len;
    use |= spec_far(n0) || (drop && n0 > 0.0);
    if (j == i) norm = __builtin_sqrt(n0);
    if (lane < NBP && i < nc) s[i * ss + lane] = make_double2(r.x * inv, r.y * inv);
    if (lane < NC) lf[i * NC + lane] = i < nc && j < i ? l : make_double2(i < nc && j == i ? len : 0.0, 0.0);
    wave_sync();
  }
  // column j of L^-1 times |row j| (zero rows: of the identity)
  if (lane < nc)
#pragma clang loop unroll(disable)
    for (int i = j; i < nc; ++i) {
      double2 z = make_double2(i == j ? norm : 0.0, 0.0);
#pragma clang loop unroll(disable)
      for (int m = j; m < i; ++m) {
        const double2 a = lf[i * NC + m], b = y[j * NC + m];
        z.x -= a.x * b.x - a.y * b.y;
        z.y -= a.x * b.y + a.y * b.x;
      }
      const double d = lf[i * NC + i].x, inv = d == 0.0 ? 1.0 : 1.0 / d;
      z.x *= inv;
      z.y *= inv;
      y[j * NC + i] = z;
      f += z.x * z.x + z.y * z.y;
    }
  return use || !(spec_wave_sum(f) <= 64.0);
}

// m = L^dag m L and m = L m L^dag in place, m in LDS: this lane's rows i0 .. i1 - 1, then
// (the matrix's other lanes done with theirs) columns.  In loops over LDS, because they
// run for oblique rows only: in registers they cost the kernels around them up to 110 VGPRs.
template <int NC>
__device__ __forceinline__ void spec_inner(lv2d* m, const lv2d* lf, int i0, int i1) {
#pragma clang loop unroll(disable)
  for (int i = i0; i < i1; ++i)
#pragma clang loop unroll(disable)
    for (int j = 0; j < NC; ++j) {
      v2d s = (v2d){0.0, 0.0};
#pragma clang loop unroll(disable)
      for (int n = j; n < NC; ++n) {
        const v2d x = m[i * NC + n], l = lf[n * NC + j];
        s += (v2d){x.x * l.x - x.y * l.y, x.x * l.y + x.y * l.x};
      }
      m[i * NC + j] = s;
    }
  wave_sync();
#pragma clang loop unroll(disable)
  for (int i = i0; i < i1; ++i)
#pragma clang loop unroll(disable)
    for (int j = 0; j < NC; ++j) {
      v2d s = (v2d){0.0, 0.0};
#pragma clang loop unroll(disable)
      for (int n = j; n < NC; ++n) {
        const v2d x = m[n * NC + i], l = lf[n * NC + j];
        s += (v2d){x.x * l.x + x.y * l.y, x.y * l.x - x.x * l.y};
      }
      m[j * NC + i] = s;
    }
  wave_sync();
}
template <int NC>
__device__ __forceinline__ void spec_outer(lv2d* m, const lv2d* lf, int i0, int i1) {
#pragma clang loop unroll(disable)
  for (int i = i0; i < i1; ++i)
#pragma clang loop unroll(disable)
    for (int j = NC - 1; j >= 0; --j) {
      v2d s = (v2d){0.0, 0.0};
#pragma clang loop unroll(disable)
      for (int n = 0; n <= j; ++n) {
        const v2d x = m[i * NC + n], l = lf[j * NC + n];
        s += (v2d){x.x * l.x + x.y * l.y, x.y * l.x - x.x * l.y};
      }
      m[i * NC + j] = s;
    }
  wave_sync();
#pragma clang loop unroll(disable)
  for (int i = i0; i < i1; ++i)
#pragma clang loop unroll(disable)
    for (int j = NC - 1; j >= 0; --j) {
      v2d s = (v2d){0.0, 0.0};
#pragma clang loop unroll(disable)
      for (int n = 0; n <= j; ++n) {
        const v2d x = m[n * NC + i], l = lf[j * NC + n];
        s += (v2d){x.x * l.x - x.y * l.y, x.x * l.y + x.y * l.x};
      }
      m[j * NC + i] = s;
    }
  wave_sync();
}
// A row-layout matrix into LDS and out of it (lanes past the NC rows leave nothing and
// repeat the last one).
template <int NC>
__device__ __forceinline__ void spec_put_row(lv2d* m, int i, const double (&ar)[NC], const double (&ai)[NC]) {
  wave_sync();
  if (i < NC) {
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      if (j % 4 == 0) __builtin_amdgcn_sched_barrier(0);
      m[i * NC + j] = (v2d){ar[j], ai[j]};
    }
  }
  wave_sync();
}

// ---- row layout: lane 16 g + i holds row i of matrix g.  Both helpers below are
// blocks of multiply-adds whose broadcast of row K within the 16-lane row is their
// DPP operand, so it costs no move.  A block starts with an s_nop for the two wait
// states a DPP read needs after the vector instruction that wrote its source (3 ns
// where a multiply-add takes 2, hence several columns per block), and its outputs
// are early-clobbered because they are written before all inputs have been read.
// (Blocks of 7 columns and two rows instead of 3 columns and one: 48 bands and 14
// orbitals 5.65 to 5.33 ns per k-point and frequency.)
#define SPEC_REP3(M) M(0) M(1) M(2)
#define SPEC_REP4(M) SPEC_REP3(M) M(3)
#define SPEC_REP5(M) SPEC_REP4(M) M(4)
#define SPEC_REP6(M) SPEC_REP5(M) M(5)
#define SPEC_REP7(M) SPEC_REP6(M) M(6)
#define SPEC_REP8(M) SPEC_REP7(M) M(7)
#define SPEC_BC(K) " row_newbcast:%[" #K "] row_mask:0xf bank_mask:0xf\n\t"

// Columns col(M0) .. of a Gauss-Jordan step: (r, i) += n (row K's (r, i)).  Row K's
// imaginary part is moved out first because its register changes before its last use.
#define SPEC_E0(j) "v_mov_b64_dpp %[t" #j "], %[i" #j "]" SPEC_BC(k)
#define SPEC_E1(j) "v_fmac_f64_dpp %[i" #j "], %[r" #j "], %[ni]" SPEC_BC(k)
#define SPEC_E2(j) "v_fmac_f64_dpp %[r" #j "], %[r" #j "], %[nr]" SPEC_BC(k)
#define SPEC_E3(j) "v_fmac_f64 %[i" #j "], %[t" #j "], %[nr]\n\t"
#define SPEC_E4(j) "v_fma_f64 %[r" #j "], -%[t" #j "], %[ni], %[r" #j "]\n\t"
#define SPEC_EO(j) , [r##j] "+&v"(rr[col(M0 + j)]), [i##j] "+&v"(ri[col(M0 + j)]), [t##j] "=&v"(t[j])
#define SPEC_ELIM(N)                                                                                          \
  asm("s_nop 1\n\t" SPEC_REP##N(SPEC_E0) SPEC_REP##N(SPEC_E1) SPEC_REP##N(SPEC_E2) SPEC_REP##N(SPEC_E3)        \
          SPEC_REP##N(SPEC_E4)                                                                                \
      : [z] "=&v"(z) SPEC_REP##N(SPEC_EO)                                                                      \
      : [nr] "v"(nr), [ni] "v"(ni), [k] "i"(K))

// Gauss-Jordan steps K .. NC-1 (rows and columns past nc hold the identity).  pmin:
// the smallest |pivot|^2 so far.  The reciprocal is the hardware estimate (2^-23)
// and one third-order step; n = -row multiplier, and 1/p - 1 for the pivot row.
template <int K, int NC>
struct SpecStep {
  static constexpr int col(int m) { return m < K ? m : m + 1; }
  template <int M0, int N>
  static __device__ __forceinline__ void block(double (&rr)[NC], double (&ri)[NC], double nr, double ni) {
    double t[N];
    int z;  // unused: opens the output list
    if constexpr (N == 4) SPEC_ELIM(4);
    if constexpr (N == 5) SPEC_ELIM(5);
    if constexpr (N == 6) SPEC_ELIM(6);
    if constexpr (N == 7) SPEC_ELIM(7);
    if constexpr (N == 8) SPEC_ELIM(8);
  }
  static __device__ __forceinline__ void run(double (&rr)[NC], double (&ri)[NC], int i, double& pmin) {
    const double px = row_bcast<K>(rr[K]), py = row_bcast<K>(ri[K]);
    const double d = __builtin_fma(px, px, py * py);
    asm("v_min_f64 %0, %0, %1" : "+v"(pmin) : "v"(d));  // fmin would first canonicalise both
    double t = __builtin_amdgcn_rcp(d);
    const double e = __builtin_fma(-d, t, 1.0);
    t = __builtin_fma(t, __builtin_fma(e, e, e), t);
    const double ix = px * t, iy = -py * t;
    const bool piv = i == K;
    const double nr = piv ? ix - 1.0 : __builtin_fma(-rr[K], ix, ri[K] * iy);
    const double ni = piv ? iy : __builtin_fma(-ri[K], ix, -rr[K] * iy);
    constexpr int N0 = NC - 1 <= 8 ? NC - 1 : NC / 2;
    block<0, N0>(rr, ri, nr, ni);
    if constexpr (N0 < NC - 1) block<N0, NC - 1 - N0>(rr, ri, nr, ni);
    rr[K] = piv ? ix : nr;
    ri[K] = ni;
    if constexpr (K + 1 < NC) SpecStep<K + 1, NC>::run(rr, ri, i, pmin);
  }
};
template <int NC>
__device__ __forceinline__ void spec_sweep(double (&rr)[NC], double (&ri)[NC], int i, double& pmin) {
  SpecStep<0, NC>::run(rr, ri, i, pmin);
}

// c_j += (row K's b_j) x + (row K + 1's b_j) y for JB columns (complex), and the
// same for row K alone.
#define SPEC_M0(j) "v_fmac_f64_dpp %[c" #j "], %[b" #j "], %[xr]" SPEC_BC(k)
#define SPEC_M1(j) "v_fmac_f64_dpp %[d" #j "], %[e" #j "], %[xr]" SPEC_BC(k)
#define SPEC_M2(j) "v_fmac_f64_dpp %[c" #j "], -%[e" #j "], %[xi]" SPEC_BC(k)
#define SPEC_M3(j) "v_fmac_f64_dpp %[d" #j "], %[b" #j "], %[xi]" SPEC_BC(k)
#define SPEC_M4(j) "v_fmac_f64_dpp %[c" #j "], %[b" #j "], %[yr]" SPEC_BC(l)
#define SPEC_M5(j) "v_fmac_f64_dpp %[d" #j "], %[e" #j "], %[yr]" SPEC_BC(l)
#define SPEC_M6(j) "v_fmac_f64_dpp %[c" #j "], -%[e" #j "], %[yi]" SPEC_BC(l)
#define SPEC_M7(j) "v_fmac_f64_dpp %[d" #j "], %[b" #j "], %[yi]" SPEC_BC(l)
#define SPEC_MO(j) [c##j] "+&v"(cr[j]), [d##j] "+&v"(ci[j]),
#define SPEC_MI(j) [b##j] "v"(br[j]), [e##j] "v"(bi[j]),
#define SPEC_MAC(N, TWO, Y)                                                                              \
  asm("s_nop 1\n\t" SPEC_REP##N(SPEC_M0) SPEC_REP##N(SPEC_M1) SPEC_REP##N(SPEC_M2) SPEC_REP##N(SPEC_M3) TWO \
      : SPEC_REP##N(SPEC_MO) [z] "=&v"(z)                                                                 \
      : SPEC_REP##N(SPEC_MI)[xr] "v"(xr[K]), [xi] "v"(xi[K]), [k] "i"(K) Y)
#define SPEC_MAC2(N)                                                                             \
  SPEC_MAC(N, SPEC_REP##N(SPEC_M4) SPEC_REP##N(SPEC_M5) SPEC_REP##N(SPEC_M6) SPEC_REP##N(SPEC_M7), \
           SPEC_Y)
#define SPEC_Y , [yr] "v"(xr[K + 1 < NC ? K + 1 : K]), [yi] "v"(xi[K + 1 < NC ? K + 1 : K]), [l] "i"(K + 1)
#define SPEC_NOY
#define SPEC_MACS(N)               \
  {                                \
    if constexpr (K + 1 < NC)      \
      SPEC_MAC2(N);                \
    else                           \
      SPEC_MAC(N, "", SPEC_NOY);   \
  }

// c[j] += sum_k x[k] (b[j] of row k), j = 0 .. JB-1: rows of a matrix product.
template <int K, int NC, int JB>
__device__ __forceinline__ void row_mac(double (&cr)[JB], double (&ci)[JB], const double (&xr)[NC],
                                        const double (&xi)[NC], const double* br, const double* bi) {
  if constexpr (K < NC) {
    int z;  // unused: keeps the output list's last comma legal
    if constexpr (JB == 4) SPEC_MACS(4)
    if constexpr (JB == 5) SPEC_MACS(5)
    if constexpr (JB == 6) SPEC_MACS(6)
    if constexpr (JB == 7) SPEC_MACS(7)
    row_mac<K + 2, NC, JB>(cr, ci, xr, xi, br, bi);
  }
}

// Column block of the row-layout products.
template <int NC>
constexpr int spec_jb() {
  return NC == 16 || NC == 8 ? 4 : NC <= 6 ? NC : NC / 2;
}

// One column block of V = Gl Sigma' and R = Sigma' + Sigma' V, R to LDS; around it
// the same columns of the G_loc partial are read (before the block of the previous
// columns is done with) and w_k Gl is added, see SpecGl.
template <int J0, int NC, bool WS, class GlT>
__device__ __forceinline__ void spec_r_blocks(const double (&gr)[NC], const double (&gi)[NC], const double (&sr)[NC],
                                              const double (&si)[NC], bool valid, int i, lv2d* xb, const GlT& gl,
                                              v2d (&part)[spec_jb<NC>()]) {
  if constexpr (J0 < NC) {
    constexpr int JB = spec_jb<NC>();
    if constexpr (WS) {
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
        for (int j = 0; j < JB; ++j) xb[i * NC + J0 + j] = (v2d){rr[j], ri[j]};
      }
    }
    v2d next[JB];
    if constexpr (J0 + JB < NC) gl.template load<J0 + JB>(next);  // before the stores below: nothing waits for them
    gl.template store<J0>(part, gr, gi);
    spec_r_blocks<J0 + JB, NC, WS>(gr, gi, sr, si, valid, i, xb, gl, next);
  }
}

// This lane's row of the G_loc partial (column stride 4 NC): w_k Gl is written at
// the tile's first k-point and added after it, a column block at a time.  (Memory
// atomics instead of the load: 111 cycles per instruction and wavefront here.)
template <int NC>
struct SpecGl {
  gv2d* p;
  double wk;
  bool put, more;  // this lane's row exists; there is something to add to
  template <int J0>
  __device__ __forceinline__ void load(v2d (&part)[spec_jb<NC>()]) const {
    if (more) {
#pragma unroll
      for (int j = 0; j < spec_jb<NC>(); ++j) part[j] = p[(J0 + j) * 4 * NC];
    } else {
#pragma unroll
      for (int j = 0; j < spec_jb<NC>(); ++j) part[j] = (v2d){0.0, 0.0};
    }
  }
  template <int J0>
  __device__ __forceinline__ void store(const v2d (&part)[spec_jb<NC>()], const double (&gr)[NC],
                                        const double (&gi)[NC]) const {
    if (put) {
#pragma unroll
      for (int j = 0; j < spec_jb<NC>(); ++j)
        p[(J0 + j) * 4 * NC] = (v2d){__builtin_fma(wk, gr[J0 + j], part[j].x), __builtin_fma(wk, gi[J0 + j], part[j].y)};
    }
  }
};

// Looks the staged rows of S over (four lanes to an unordered pair of them) and where they
// are oblique enough puts Q in their place: sh.use_q.
template <int NBP, int NC, class Sh>
__device__ __forceinline__ void spec_rows_check(Sh& sh, int nc, int tid) {
  using Dm = typename Sh::Dm;
  double2* const s = Dm::PREG ? sh.xr : sh.sp;
  constexpr int SS = Dm::PREG ? NBP : Dm::SS;
#pragma clang loop unroll(disable)
  for (int pr = tid >> 2; pr < nc * (nc / 2 + 1); pr += 64) {
    const int d = pr / nc, i = pr - d * nc, j = i + d < nc ? i + d : i + d - nc;
    double xx = 0.0, yy = 0.0, re = 0.0, im = 0.0;
#pragma unroll 4
    for (int c = 0; c < NBP; c += 4) {
      const double2 x = s[i * SS + c + (tid & 3)], y = s[j * SS + c + (tid & 3)];
      xx = __builtin_fma(x.x, x.x, __builtin_fma(x.y, x.y, xx));
      yy = __builtin_fma(y.x, y.x, __builtin_fma(y.y, y.y, yy));
      re = __builtin_fma(x.x, y.x, __builtin_fma(x.y, y.y, re));
      im = __builtin_fma(x.x, y.y, __builtin_fma(-x.y, y.x, im));
    }
    xx = spec_quad_sum(xx);
    yy = spec_quad_sum(yy);
    re = spec_quad_sum(re);
    im = spec_quad_sum(im);
    if (spec_oblique(xx, yy, re, i == j, nc) || (i != j && spec_oblique(xx, yy, im, false, nc))) sh.oblique = 1;
  }
  __syncthreads();
  if (!uniform_i(sh.oblique)) return;
  // S is kept meanwhile: in its other form, or past the scratch
  double2* const y = Sh::scratch(sh);
  double2* const back = Dm::PREG ? y + NC * NC : s + NC * SS;
  if constexpr (Dm::PREG) {
    for (int idx = tid; idx < NC * NBP; idx += 256) back[idx] = s[idx];
    __syncthreads();
  }
  if (tid < 64) {
    const bool use = spec_orthonormal<NBP, NC>(s, SS, sh.lf, y, nc, tid);
    if (tid == 0) sh.use_q = use;
  }
  __syncthreads();
  const bool use = uniform_i(sh.use_q);
#pragma clang loop unroll(disable)
  for (int idx = tid; idx < NC * NBP; idx += 256) {
    const int at = idx / NBP * SS + idx % NBP;
    const double2 x = s[at], b = back[at];
    if (!use)
      s[at] = Dm::PREG ? b : make_double2(-b.y, b.x);
    else if (!Dm::PREG)
      back[at] = make_double2(x.y, -x.x);
  }
  __syncthreads();
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
    if (tid == 0) sh.oblique = sh.use_q = 0;
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
    spec_rows_check<NBP, NC>(sh, nc, tid);
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
    // the frequencies, for rows in Q or as they are: two copies of the loop, because the
    // former's extra work costs the latter registers where they share one (48 bands, 14
    // orbitals 1.3%, 5 orbitals up to 8% more time; now 1% and 3% with the look at the rows)
    auto frequencies = [&](auto obl) __attribute__((always_inline)) {
      constexpr bool oblique = decltype(obl)::value;
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
            // all vector work of the chunk before its products: the vector and matrix
            // units do not run FP64 together, and each change from one to the other
            // drains the pipe (70 cycles measured)
            double pv[TPW];
#pragma unroll
            for (int m = 0; m < TPW; ++m) {
              if constexpr (Dm::PREG)
                pv[m] = p[m][c];
              else
                pv[m] = __builtin_fma(x[c & 1][m].x, y[c & 1][m].x, x[c & 1][m].y * y[c & 1][m].y);
            }
            const double dx = SPLIT && (w & 1) ? d[c & 1].y : d[c & 1].x;
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int m = 0; m < TPW; ++m) {
              xa[m][0] = mma(dx, pv[m], xa[m][0]);
              if constexpr (!SPLIT) xa[m][1] = mma(d[c & 1].y, pv[m], xa[m][1]);
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
          v2d own;  // X_ii
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
            own = xb[ic * NC + ic];
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
          const unsigned long long absent = row_absent(own.x, own.y, i, nc);
          if (absent) row_leave_out<NC>(rr, ri, absent, l, 1.0);
          spec_sweep<NC>(rr, ri, i, pmin);
          if (nc < NC) {
#pragma unroll
            for (int j = 0; j < NC; ++j) {
              sr[j] = i < nc && j < nc ? sr[j] : 0.0;
              si[j] = i < nc && j < nc ? si[j] : 0.0;
            }
          }
#pragma unroll
          for (int j = 0; j < NC; ++j) sr[j] -= i == j ? edc : 0.0;
          if constexpr (oblique) {  // Sigma' of the rows of Q, by way of the matrix area
            spec_put_row<NC>(xb, i, sr, si);
            spec_inner<NC>(xb, spec_lds(sh.lf), i, min(i + 1, NC));
#pragma unroll
            for (int j = 0; j < NC; ++j) {
              if (j % 4 == 0) __builtin_amdgcn_sched_barrier(0);  // a few at a time: few registers
              const v2d x = xb[ic * NC + j];
              rr[j] -= x.x;
              ri[j] -= x.y;
            }
          } else {
#pragma unroll
            for (int j = 0; j < NC; ++j) {
              rr[j] -= sr[j];
              ri[j] -= si[j];
            }
          }
          if (absent) row_leave_out<NC>(rr, ri, absent, l, 1.0);
          spec_sweep<NC>(rr, ri, i, pmin);
          if (absent) row_leave_out<NC>(rr, ri, absent, l, 0.0);
          if constexpr (oblique) {  // Gl of the rows of S
            spec_put_row<NC>(xb, i, rr, ri);
            spec_outer<NC>(xb, spec_lds(sh.lf), i, min(i + 1, NC));
#pragma unroll
            for (int j = 0; j < NC; ++j) {
              if (j % 4 == 0) __builtin_amdgcn_sched_barrier(0);  // a few at a time: few registers
              const v2d x = xb[ic * NC + j];
              rr[j] = x.x;
              ri[j] = x.y;
            }
          }
          SpecGl<NC> gl;
          gl.p = (gv2d*)a.xs +
                 ((int64_t)(a.ktile_base + ktile) * n4_all + min((ng >> 2) + w, n4_all - 1)) * (4 * NC * NC) +
                 (nl & 3) * NC + ic;
          gl.wk = wk;
          gl.put = want_x && valid && i < NC;
          gl.more = want_x && kk != kk0;
          v2d part[spec_jb<NC>()];
          gl.template load<0>(part);
          double chk = 0.0;
#pragma unroll
          for (int j = 0; j < NC; ++j) chk += rr[j] + ri[j];
          if (i < NC && !__builtin_isfinite(chk)) nonfinite = 1;
          wave_sync();
          spec_r_blocks<0, NC, WS>(rr, ri, sr, si, valid, i, xb, gl, part);
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
              if (!valid) {  // frequencies past the tile add nothing
#pragma unroll
                for (int j = 0; j < NC; ++j) xb[i * NC + j] = (v2d){0.0, 0.0};
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
          // row factors of all 16 frequencies first, then products only; operands one
          // chunk of four frequencies ahead
          v2d h[2][CT];
          auto fetch = [&](int c, int s) {
#pragma unroll
            for (int t = 0; t < CT; ++t) h[s][t] = xc[4 * c * NP + 16 * WC * t];
          };
          double fr[4][RT], fi[4][RT];
          {
            v2d x[4][RT], y[4][RT];
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
              for (int r = 0; r < RT; ++r) {
                x[c][r] = d1[r][4 * c * DS];
                y[c][r] = d2[r][4 * c * DS];
              }
            fetch(0, 0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
              for (int r = 0; r < RT; ++r) {
                fr[c][r] = x[c][r].x * y[c][r].x - x[c][r].y * y[c][r].y;
                fi[c][r] = x[c][r].x * y[c][r].y + x[c][r].y * y[c][r].x;
              }
          }
          spec_for<0, 4>([&](auto ci) {
            constexpr int c = decltype(ci)::value;
            if constexpr (c < 3) fetch(c + 1, (c + 1) & 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < CT; ++t) {
#pragma unroll
              for (int r = 0; r < RT; ++r) acc[r][t] = mma(fr[c][r], h[c & 1][t].x, acc[r][t]);
#pragma unroll
              for (int r = 0; r < RT; ++r) acc[r][t] = mma(fi[c][r], h[c & 1][t].y, acc[r][t]);
            }
          });
        }
      }
    };
    if (uniform_i(sh.use_q))
      frequencies(std::true_type());
    else
      frequencies(std::false_type());
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
