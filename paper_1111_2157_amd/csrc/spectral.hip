// Dispatch of the spectral density kernel (spectral_impl.h) over the padded
// band-window sizes, and its epilogues: N(k) from the accumulated sums, and the
// fixed-order reduction of the G_loc partials.
#include <hip/hip_runtime.h>

#include "spectral_impl.h"

namespace dmft {

#define SPEC_DECL(NAME)                                                                                         \
  hipError_t NAME(int ncls, const DysonArgs& a, const void* items, int n_items, const DysonArgs* args, int* counter, \
                  int grid, hipStream_t s);
SPEC_DECL(launch_spectral_16)
SPEC_DECL(launch_spectral_32)
SPEC_DECL(launch_spectral_48)
SPEC_DECL(launch_spectral_64)
SPEC_DECL(launch_spectral_gloc_16)
SPEC_DECL(launch_spectral_gloc_32)
SPEC_DECL(launch_spectral_gloc_48)
SPEC_DECL(launch_spectral_gloc_64)
#undef SPEC_DECL

// A queue (items set) always carries the sums.
hipError_t launch_spectral(int nbp, int ncls, const DysonArgs& a, const void* items, int n_items,
                           const DysonArgs* args, int* counter, int grid, hipStream_t s) {
  const bool sums = items || (a.mode & MODE_S);
#define SPEC_SIZE(N)                                                                                    \
  case N:                                                                                               \
    return sums ? launch_spectral_##N(ncls, a, items, n_items, args, counter, grid, s)                  \
                : launch_spectral_gloc_##N(ncls, a, items, n_items, args, counter, grid, s);
  switch (nbp) {
    SPEC_SIZE(16)
    SPEC_SIZE(32)
    SPEC_SIZE(48)
    SPEC_SIZE(64)
    default: return hipErrorInvalidValue;
  }
#undef SPEC_SIZE
}

namespace {

// N(k) of one k-point (one work-group) from the sums of spec_kernel:
//   N = 1/2 - (beta/4) M1 + (1/beta) (F + 2 s2 M1),   F = sum_n (G + G^dag),
//   F[v][v'] = [v = v'] sum_n 2 Re d_v + S_v^dag H(v, v') S_v',
// in the order of the band energies.  A pair v < v' whose indices first differ
// in bit l has a multiple m of 2^l in (v, v']; with L[v] = sum of e_j H(j, j+1)
// over the steps between v and m (and likewise for v'), H(v, v') is
// (L[v] + L[v']) / (E_v' - E_v): a mean with positive weights (see spectral_impl.h), and
// W = S_v^dag L[v] is formed once per band and level instead of per pair.  A
// thread takes one column of L from m outwards, one band per step, so a level
// reads the sums once: 6 nb nc^2 additions and complex products per k-point,
// against nw evaluations.  (512 k-points of 48 bands, 14 orbitals, four
// frequency tiles: 488 us with every band summing its own steps anew, 262 us
// with one thread per column, 184 us with its rows spread over a quad; 32 bands,
// 10 orbitals: 127 and 58 us.)  Bound by the latency of the chain of steps, at
// one work-group per CU, and by reading the frequency tiles.  The sums sit
// in LDS (99 KB for 64 bands, 14 orbitals), or where they do not fit (ULDS
// false: 15 and 16 orbitals on the widest windows) are added up in place in
// global memory.
template <int NC, bool ULDS>
__global__ void __launch_bounds__(1024) spec_epilogue_kernel(EpilogueArgs a, double* nk_out) {
  constexpr int NT = spec_col_tiles(NC), NP = NC * NC;
  extern __shared__ double2 lds[];
  __shared__ double es[64], sumd[64];
  __shared__ unsigned long long key[64];
  __shared__ int rank[64], inv[64];
  const int tid = threadIdx.x, nth = blockDim.x;
  int bucket = 0;
  while (bucket + 1 < a.n_sizes && (int)blockIdx.x >= a.sizes[bucket + 1].first) ++bucket;
  const int n_wtiles = a.sizes[bucket].n_wtiles, nbp = a.sizes[bucket].nbp;
  const int64_t t_stride = a.sizes[bucket].t_stride;
  const int slot = blockIdx.x - a.sizes[bucket].first;
  const int k = a.klist ? a.klist[a.sizes[bucket].at + slot] : slot;
  const int nc = a.nc;
  const int nb = a.nb_uniform > 0 ? a.nb_uniform : a.nb[k];
  const int64_t ob = a.nb_uniform > 0 ? (int64_t)k * nb : a.off_b[k];
  const int64_t on = a.nb_uniform > 0 ? (int64_t)k * nb * nb : a.off_n[k];
  const double* eps = a.eps + ob;
  const double2* P = reinterpret_cast<const double2*>(a.proj) + ob * nc;
  const double2* sinf = reinterpret_cast<const double2*>(a.sigma_inf);
  const double mu = a.mu_ptr ? *a.mu_ptr : a.mu;
  const double beta = a.beta, ctail = 2.0 * a.s2 / beta - 0.25 * beta;  // coefficient of M1
  const bool tail = a.tail_order == 2;
  const int64_t sd = spec_slot_doubles(nbp, NC);
  double2* ps = lds;                                            // [NC][nb] projectors, sorted columns
  double2* wv = lds + NC * nb;                                  // [nb][NC] W of a level
  double2* vinf = lds + 2 * NC * nb;                            // [NC][nb] (Sigma_inf - V_DC) S
  double* u = reinterpret_cast<double*>(lds + 3 * NC * nb);     // [nb - 1][NP] H(j, j+1)

  if (tid < nb) key[tid] = spec_key(eps[tid]);
  __syncthreads();
  if (tid < nb) {
    const int r = spec_rank(key, tid, nb);
    rank[tid] = r;
    inv[r] = tid;
    es[r] = eps[tid];
  }
  __syncthreads();
  for (int idx = tid; idx < NC * nb; idx += nth) {
    const int al = idx / nb, v = idx - al * nb;
    ps[al * nb + rank[v]] = al < nc ? P[idx] : make_double2(0.0, 0.0);
  }
  // element p of row r of the sums, added over the frequency tiles in order
  double* base = a.tsum + a.sizes[bucket].t_base + (int64_t)slot * sd;
  auto sum_at = [&](int64_t o) {
    double x = 0.0;
#pragma unroll 4
    for (int w = 0; w < n_wtiles; ++w) x += base[(int64_t)w * t_stride + o];
    return x;
  };
  auto elem = [&](int r, int p) {
    return (int64_t)(((r >> 4) * NT + (p >> 4)) * 4 + ((r >> 2) & 3)) * 64 + (r & 3) * 16 + (p & 15);
  };
  // four elements of four frequency tiles per thread in flight
  for (int i0 = tid; i0 < (nb - 1) * NP; i0 += 4 * nth) {
    double x[4];
    int64_t o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int idx = min(i0 + i * nth, (nb - 1) * NP - 1);
      o[i] = elem(2 * (idx / NP) + 1, idx % NP);
      x[i] = 0.0;
    }
    for (int w0 = 0; w0 < n_wtiles; w0 += 4) {
      double y[4][4];
#pragma unroll
      for (int w = 0; w < 4; ++w)
#pragma unroll
        for (int i = 0; i < 4; ++i) y[w][i] = base[(int64_t)min(w0 + w, n_wtiles - 1) * t_stride + o[i]];
#pragma unroll
      for (int w = 0; w < 4; ++w)
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] += w0 + w < n_wtiles ? y[w][i] : 0.0;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i0 + i * nth < (nb - 1) * NP) (ULDS ? u[i0 + i * nth] : base[o[i]]) = x[i];
  }
  auto u_at = [&](int j, int p) { return ULDS ? u[j * NP + p] : base[elem(2 * j + 1, p)]; };
  __syncthreads();
  for (int idx = tid; idx < NC * nb; idx += nth) {
    const int al = idx / nb, v = idx - al * nb;
    if (al >= nc) {
      vinf[idx] = make_double2(0.0, 0.0);
      continue;
    }
    double2 x = make_double2(-a.e_dc[al] * ps[idx].x, -a.e_dc[al] * ps[idx].y);
    if (sinf)
      for (int be = 0; be < nc; ++be) {
        const double2 m = sinf[al * nc + be], pb = ps[be * nb + v];
        x.x += m.x * pb.x - m.y * pb.y;
        x.y += m.x * pb.y + m.y * pb.x;
      }
    vinf[idx] = x;
  }
  if (tid < nb) sumd[tid] = sum_at((int64_t)spec_row_tiles(nbp) * NT * 256 + tid);
  __syncthreads();

  double tr = 0.0, hks = 0.0, ncor = 0.0;
  // one element (and its mirror image) of N(k), sorted indices v <= x, from F[v][x]
  auto emit = [&](int v, int x, double2 f) {
    double2 m1 = make_double2(v == x ? es[v] - mu : 0.0, 0.0);
    double2 qq = make_double2(0.0, 0.0);  // (S^dag S)[x][v]
#pragma unroll 7
    for (int al = 0; al < NC; ++al) {
      const double2 pv = ps[al * nb + v], px = ps[al * nb + x];
      qq.x += px.x * pv.x + px.y * pv.y;
      qq.y += px.x * pv.y - px.y * pv.x;
      if (tail) {
        const double2 vi = vinf[al * nb + x];
        m1.x += pv.x * vi.x + pv.y * vi.y;
        m1.y += pv.x * vi.y - pv.y * vi.x;
      }
    }
    double2 nv = make_double2(f.x / beta, f.y / beta);
    if (v == x) {
      nv.x += 0.5;
      nv.y = 0.0;
      m1.y = 0.0;
    }
    if (tail) {
      nv.x += ctail * m1.x;
      nv.y += ctail * m1.y;
    }
    const int r = inv[v], c = inv[x];
    if (nk_out) {
      reinterpret_cast<double2*>(nk_out)[on + r * nb + c] = nv;
      if (r != c) reinterpret_cast<double2*>(nk_out)[on + c * nb + r] = make_double2(nv.x, -nv.y);
    }
    if (v == x) {
      tr += nv.x;
      hks += es[v] * nv.x;
      ncor += nv.x * qq.x;
    } else {
      ncor += 2.0 * (nv.x * qq.x - nv.y * qq.y);
    }
  };

  // the diagonal: S_v^dag H(v, v) S_v is a sum over the nc^2 real numbers of
  // H(v, v), 16 lanes to a band
  for (int v0 = 0; v0 < nb; v0 += nth / 16) {
    const int v = v0 + tid / 16, l = tid & 15;
    constexpr int PL = (NP + 15) / 16;
    double t[PL], f = 0.0;
#pragma unroll
    for (int i = 0; i < PL; ++i) t[i] = 0.0;
#pragma unroll 2
    for (int w = 0; w < n_wtiles; ++w)
#pragma unroll
      for (int i = 0; i < PL; ++i)
        t[i] += base[(int64_t)w * t_stride + elem(2 * min(v, nb - 1), min(l + 16 * i, NP - 1))];
    if (v < nb)
#pragma unroll
      for (int i = 0; i < PL; ++i) {
        const int p = l + 16 * i;
        if (p >= NP) break;
        const int al = p / NC, be = p - al * NC;
        const double2 x = ps[al * nb + v], y = ps[be * nb + v];
        // Re conj(S_al) S_be twice off the diagonal, and for the lower triangle (which
        // holds Im of element (be, al)) -2 Im conj(S_be) S_al
        const double c = al < be ? 2.0 * (x.x * y.x + x.y * y.y) : (al == be ? x.x * x.x + x.y * x.y
                                                                        : -2.0 * (y.x * x.y - y.y * x.x));
        f += c * t[i];
      }
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) f += __shfl_xor(f, o, 16);
    if (v < nb && l == 0) sumd[v] = 2.0 * sumd[v] + f;
  }
  __syncthreads();
  for (int v = tid; v < nb; v += nth) emit(v, v, make_double2(sumd[v], 0.0));
  for (int l = 0; (1 << l) < nb; ++l) {
    __syncthreads();
    // (block, side, column) and every fourth row of it: the bands of one side of
    // m, from m outwards; the four lanes of a quad add up their rows
    const int units = ((nb + (2 << l) - 1) >> (l + 1)) * 2;
    for (int i0 = 0; i0 < units * NC * 4; i0 += nth) {
      const int idx = i0 + tid, qd = idx & 3, ub = idx >> 2, unit = ub / NC, b = ub - unit * NC, up = unit & 1;
      const int m = ((unit >> 1) << (l + 1)) + (1 << l);
      const bool on = unit < units && m < nb;  // else no pair crosses m; uniform in a quad
      constexpr int RL = (NC + 3) / 4;
      double l1[RL], l2[RL];
#pragma unroll
      for (int i = 0; i < RL; ++i) l1[i] = l2[i] = 0.0;
      for (int t = 0; on && t < (1 << l); ++t) {
        // upper side: bands m, m + 1, ... (no step for m itself); lower side: m - 1, m - 2, ...
        const int v = up ? m + t : m - 1 - t, j = up ? v - 1 : v;
        if (v >= nb) break;
        double2 s = make_double2(0.0, 0.0);  // S_v^dag L, column b
        const double e = !up || t ? __builtin_fmax(es[j + 1] - es[j], kTinyStep) : 0.0;
#pragma unroll
        for (int i = 0; i < RL; ++i) {
          const int al = min(4 * i + qd, NC - 1);
          l1[i] = __builtin_fma(e, u_at(min(j, nb - 2), al * NC + b), l1[i]);
          l2[i] = __builtin_fma(e, u_at(min(j, nb - 2), b * NC + al), l2[i]);
          const double re = al <= b ? l1[i] : l2[i], im = al < b ? l2[i] : (al > b ? -l1[i] : 0.0);
          double2 x = ps[al * nb + v];
          if (4 * i + qd >= NC) x = make_double2(0.0, 0.0);
          s.x += x.x * re + x.y * im;
          s.y += x.x * im - x.y * re;
        }
        s.x = spec_quad_sum(s.x);
        s.y = spec_quad_sum(s.y);
        if (qd == 0) wv[v * NC + b] = s;
      }
    }
    __syncthreads();
    const int half = 1 << l;
    const int nblk = (nb + 2 * half - 1) >> (l + 1);
    for (int idx = tid; idx < (nblk << (2 * l)); idx += nth) {
      const int blk = idx >> (2 * l), r = idx & ((1 << (2 * l)) - 1);
      const int v = (blk << (l + 1)) + (r >> l), x = (blk << (l + 1)) + half + (r & (half - 1));
      if (x >= nb) continue;
      double2 f = make_double2(0.0, 0.0);
#pragma unroll 7
      for (int b = 0; b < NC; ++b) {
        const double2 w0 = wv[v * NC + b], w1 = wv[x * NC + b], s0 = ps[b * nb + v], s1 = ps[b * nb + x];
        // W[v] . S_x + conj(W[x] . S_v)
        f.x += w0.x * s1.x - w0.y * s1.y + (w1.x * s0.x - w1.y * s0.y);
        f.y += w0.x * s1.y + w0.y * s1.x - (w1.x * s0.y + w1.y * s0.x);
      }
      const double gap = __builtin_fmax(es[x] - es[v], (x - v) * kTinyStep);
      const double ig = 1.0 / gap;
      f.x *= ig;
      f.y *= ig;
      emit(v, x, f);
    }
  }
  // fixed-order sums of the work-group: lanes, then wavefronts
  double* red = reinterpret_cast<double*>(lds);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    tr += __shfl_xor(tr, o);
    ncor += __shfl_xor(ncor, o);
    hks += __shfl_xor(hks, o);
  }
  __syncthreads();
  if ((tid & 63) == 0) {
    red[3 * (tid >> 6) + 0] = tr;
    red[3 * (tid >> 6) + 1] = ncor;
    red[3 * (tid >> 6) + 2] = hks;
  }
  __syncthreads();
  if (tid < 3) {
    double s = 0.0;
    for (int w = 0; w < nth / 64; ++w) s += red[3 * w + tid];
    a.kscal[k * 3 + tid] = s;
  }
}

// G_loc(n) = sum of the partials of all k-tiles, in order: one work-group per
// four frequencies and column, its four wavefronts taking every fourth k-tile.
__global__ void __launch_bounds__(256) spec_gloc_kernel(const double* xs, int n_xs, int n4, int ncls, int nc, int nw,
                                                        double* gloc, int add) {
  __shared__ double2 part[4][64];
  const int f4 = blockIdx.x, col = blockIdx.y, w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t block = (int64_t)4 * ncls * ncls, stride = (int64_t)n4 * block;
  double2 acc = make_double2(0.0, 0.0);
  if (lane < 4 * ncls) {
    const double2* p = reinterpret_cast<const double2*>(xs) + f4 * block + col * 4 * ncls + lane;
#pragma unroll 4
    for (int t = w; t < n_xs; t += 4) {
      const double2 v = p[t * stride];
      acc.x += v.x;
      acc.y += v.y;
    }
  }
  part[w][lane] = acc;
  __syncthreads();
  if (w == 0 && lane < 4 * ncls) {
    for (int j = 1; j < 4; ++j) {
      acc.x += part[j][lane].x;
      acc.y += part[j][lane].y;
    }
    const int n = 4 * f4 + lane / ncls, row = lane % ncls;
    if (n < nw && row < nc && col < nc) {
      double2* g = reinterpret_cast<double2*>(gloc) + ((int64_t)n * nc + row) * nc + col;
      if (add) {
        acc.x += g->x;
        acc.y += g->y;
      }
      *g = acc;
    }
  }
}

// The same from the partials of the one-matrix-per-lane kernel ([k-tile][element][n]):
// a thread per element and frequency.
__global__ void __launch_bounds__(256) spec_gloc_lane_kernel(const double* xs, int n_xs, int nw4, int ncls, int nc, int nw,
                                                             double* gloc, int add) {
  __shared__ double2 part[4][64];
  const int w = threadIdx.x >> 6, n = blockIdx.x * 64 + (threadIdx.x & 63), row = blockIdx.y, col = blockIdx.z;
  const int64_t stride = (int64_t)ncls * ncls * nw4;
  const double2* p = reinterpret_cast<const double2*>(xs) + (int64_t)(row * ncls + col) * nw4 + min(n, nw - 1);
  double2 acc = make_double2(0.0, 0.0);
#pragma unroll 8
  for (int t = w; t < n_xs; t += 4) {
    const double2 v = p[t * stride];
    acc.x += v.x;
    acc.y += v.y;
  }
  part[w][threadIdx.x & 63] = acc;
  __syncthreads();
  if (w == 0 && n < nw) {
    for (int j = 1; j < 4; ++j) {
      acc.x += part[j][threadIdx.x].x;
      acc.y += part[j][threadIdx.x].y;
    }
    double2* g = reinterpret_cast<double2*>(gloc) + ((int64_t)n * nc + row) * nc + col;
    if (add) {
      acc.x += g->x;
      acc.y += g->y;
    }
    *g = acc;
  }
}

template <int NC, bool ULDS>
hipError_t epilogue_launch(const EpilogueArgs& a, size_t lds, double* nk_out, hipStream_t s) {
  const int nbm = a.nb_uniform > 0 ? a.nb_uniform : a.spec_nbp;
  if (lds > 32 * 1024) {
    const void* f = reinterpret_cast<const void*>(spec_epilogue_kernel<NC, ULDS>);
    hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  // a thread per (band, orbital), for small windows up to four (12 bands, 5 orbitals:
  // 27 us with 64 threads, 20 with 256; 64 and 5: 60 with 1024, 46 with 512)
  int threads = 64;
  while (threads < 1024 && (threads < nbm * NC || (threads < 256 && threads < 4 * nbm * NC))) threads *= 2;
  lds = lds < 48 * sizeof(double) ? 48 * sizeof(double) : lds;  // the final reduction's scratch
  hipLaunchKernelGGL((spec_epilogue_kernel<NC, ULDS>), dim3(a.nklist), dim3(threads), lds, s, a, nk_out);
  return hipGetLastError();
}

template <int NC>
hipError_t epilogue_case(const EpilogueArgs& a, double* nk_out, hipStream_t s) {
  const int nbm = a.nb_uniform > 0 ? a.nb_uniform : a.spec_nbp;
  const size_t small = sizeof(double2) * 3 * NC * nbm, sums = sizeof(double) * (size_t)(nbm - 1) * NC * NC;
  if constexpr (NC == 16)  // 15 and 16 orbitals from 58 bands on
    if (small + sums > 156 * 1024) return epilogue_launch<NC, false>(a, small, nk_out, s);
  return epilogue_launch<NC, true>(a, small + sums, nk_out, s);
}

}  // namespace

hipError_t launch_spectral_epilogue(const EpilogueArgs& a, double* nk_out, hipStream_t s) {
  const int ncls = spec_ncls(a.nc);
  if (a.gloc_out) {
    const int n4 = (a.nw + 3) / 4;
    if (spec_lane(ncls)) {
      hipLaunchKernelGGL(spec_gloc_lane_kernel, dim3((a.nw + 63) / 64, a.nc, a.nc), dim3(256), 0, s, a.xs, a.n_xs, 4 * n4,
                         ncls, a.nc, a.nw, a.gloc_out, a.gloc_add);
      return hipGetLastError();
    }
    hipLaunchKernelGGL(spec_gloc_kernel, dim3(n4, a.nc), dim3(256), 0, s, a.xs, a.n_xs, n4, ncls, a.nc, a.nw, a.gloc_out,
                       a.gloc_add);
    return hipGetLastError();
  }
  switch (ncls) {
    case 4: return epilogue_case<4>(a, nk_out, s);
    case 5: return epilogue_case<5>(a, nk_out, s);
    case 6: return epilogue_case<6>(a, nk_out, s);
    case 8: return epilogue_case<8>(a, nk_out, s);
    case 10: return epilogue_case<10>(a, nk_out, s);
    case 12: return epilogue_case<12>(a, nk_out, s);
    case 14: return epilogue_case<14>(a, nk_out, s);
    case 16: return epilogue_case<16>(a, nk_out, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace dmft
