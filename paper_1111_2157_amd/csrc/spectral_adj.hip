// Dispatch of the spectral trace and adjoint kernels (spectral_adj_impl.h) and the
// table of the general vector-Jacobian product.
#include <hip/hip_runtime.h>

#include "spectral_adj_impl.h"

namespace dmft {

hipError_t launch_spectral_adj_16(int ncls, int what, const DysonArgs& a, int grid, hipStream_t s);
hipError_t launch_spectral_adj_32(int ncls, int what, const DysonArgs& a, int grid, hipStream_t s);
hipError_t launch_spectral_adj_48(int ncls, int what, const DysonArgs& a, int grid, hipStream_t s);
hipError_t launch_spectral_adj_64(int ncls, int what, const DysonArgs& a, int grid, hipStream_t s);

namespace {

// Q_r of one k-point (one work-group), r = 2v: Nt_vv P_v, r = 2j + 1:
//   Q_j = e_j sum_{v <= j < v'} (S_v Nt_vv' S_v'^dag + h.c.) / (E_v' - E_v),
// in the energy order.  As in the density epilogue a pair is handled at the level l
// of the highest bit in which its indices differ, split at the multiple m of 2^l in
// (v, v']: with A_u = S_u y_u^dag + h.c., y_u = sum over the other side of
// conj(Nt_uu' / gap) S_u', Q_j takes e_j times the sum of A_u over the bands of its
// side that lie outside it; partial sums, and no differences of them.
// Written as B operands: chunk of four rows, column tile, lane; then Nt_vv.
// Bound by the latency of the chains over the bands of a side (128 k-points of 40
// bands, 14 orbitals: 61 us, against 2.4 ms of the product's kernel).
template <int NC>
__global__ void __launch_bounds__(512) spec_adj_table_kernel(DysonArgs a, int nbp) {
  constexpr int NT = spec_col_tiles(NC), NP = NC * NC;
  extern __shared__ double2 lds[];
  __shared__ double es[64];
  __shared__ unsigned long long key[64];
  __shared__ int rank[64];
  const int tid = threadIdx.x, nth = blockDim.x, slot = blockIdx.x;
  const int k = a.klist ? a.klist[slot] : slot;
  const int nc = a.nc;
  const int nb = a.nb_uniform > 0 ? a.nb_uniform : a.nb[k];
  const int64_t ob = a.nb_uniform > 0 ? (int64_t)k * nb : a.off_b[k];
  const int64_t on = a.nb_uniform > 0 ? (int64_t)k * nb * nb : a.off_n[k];
  const double* eps = a.eps + ob;
  const double2* P = reinterpret_cast<const double2*>(a.proj) + ob * nc;
  const double2* nbar = reinterpret_cast<const double2*>(a.nbar) + on;
  double* base = a.tsum + a.t_base + (int64_t)slot * spec_adj_slot_doubles(nbp, NC);
  double2* ps = lds;                // [NC][nb] projectors, sorted columns
  double2* y = lds + NC * nb;       // [nb][NC]
  double2* f = lds + 2 * NC * nb;   // [nb][nb] Nt, off the diagonal over the gap
  if (tid < nb) key[tid] = spec_key(eps[tid]);
  __syncthreads();
  if (tid < nb) {
    const int r = spec_rank(key, tid, nb);
    rank[tid] = r;
    es[r] = eps[tid];
  }
  __syncthreads();
  for (int idx = tid; idx < NC * nb; idx += nth) {
    const int al = idx / nb, v = idx - al * nb;
    ps[al * nb + rank[v]] = al < nc ? P[idx] : make_double2(0.0, 0.0);
  }
  for (int idx = tid; idx < nb * nb; idx += nth) {
    const int i = idx / nb, j = idx - i * nb, r = rank[i], c = rank[j];
    const double2 x = nbar[idx], z = nbar[j * nb + i];
    double g = 1.0;
    if (r != c) {
      const int lo = min(r, c), hi = max(r, c);
      g = 1.0 / __builtin_fmax(es[hi] - es[lo], (hi - lo) * kTinyStep);
    }
    f[r * nb + c] = make_double2(g * (x.x + z.x), g * (x.y - z.y));
  }
  auto elem = [&](int r, int p) { return (((r >> 2) * NT + (p >> 4)) * 64) + (r & 3) * 16 + (p & 15); };
  __syncthreads();
  // the diagonal rows, zeros elsewhere up to the end of the last chunk
  for (int idx = tid; idx < (nb + 1) * NP; idx += nth) {
    const int v = idx / NP, p = idx - v * NP, al = p / NC, be = p - al * NC;
    double q = 0.0;
    if (v < nb) {
      const double2 x = ps[al * nb + v], z = ps[be * nb + v];
      q = f[v * nb + v].x * (al <= be ? x.x * z.x + x.y * z.y : z.y * x.x - z.x * x.y);
    }
    if (2 * v < 2 * nbp) base[elem(2 * v, p)] = q;
    if (2 * v + 1 < 2 * nbp) base[elem(2 * v + 1, p)] = 0.0;
  }
  for (int v = tid; v < nbp; v += nth) base[nbp / 2 * NT * 64 + v] = v < nb ? f[v * nb + v].x : 0.0;
  for (int l = 0; (1 << l) < nb; ++l) {
    const int half = 1 << l;
    __syncthreads();
    for (int idx = tid; idx < nb * NC; idx += nth) {
      const int u = idx / NC, b = idx - u * NC;
      const int m = (u >> (l + 1) << (l + 1)) + half;
      const int x0 = u < m ? m : m - half, x1 = u < m ? min(m + half, nb) : m;
      double2 s = make_double2(0.0, 0.0);
      for (int x = x0; x < x1; ++x) {
        const double2 g = f[u * nb + x], t = ps[b * nb + x];
        s.x += g.x * t.x + g.y * t.y;
        s.y += g.x * t.y - g.y * t.x;
      }
      y[u * NC + b] = s;
    }
    __syncthreads();
    const int units = ((nb + 2 * half - 1) >> (l + 1)) * 2;
    for (int idx = tid; idx < units * NP; idx += nth) {
      const int unit = idx / NP, p = idx - unit * NP, al = p / NC, be = p - al * NC;
      const int m = ((unit >> 1) << (l + 1)) + half;
      if (m >= nb) continue;  // no pair crosses m
      const int ra = min(al, be), rb = max(al, be);
      const bool up = unit & 1;
      const int u0 = up ? min(m + half, nb) - 1 : m - half, steps = up ? u0 - m : half;
      double acc = 0.0;
#pragma unroll 4
      for (int t = 0; t < steps; ++t) {
        const int u = up ? u0 - t : u0 + t, j = up ? u - 1 : u;
        const double2 sa = ps[ra * nb + u], sb = ps[rb * nb + u], ya = y[u * NC + ra], yb = y[u * NC + rb];
        acc += al <= be ? sa.x * yb.x + sa.y * yb.y + ya.x * sb.x + ya.y * sb.y
                        : sa.y * yb.x - sa.x * yb.y + ya.y * sb.x - ya.x * sb.y;
        base[elem(2 * j + 1, p)] += __builtin_fmax(es[j + 1] - es[j], kTinyStep) * acc;
      }
    }
  }
}

template <int NC>
hipError_t table_launch(int nbp, const DysonArgs& a, hipStream_t s) {
  const int nbm = a.nb_uniform > 0 ? a.nb_uniform : nbp;
  const size_t lds = sizeof(double2) * (2 * NC * nbm + (size_t)nbm * nbm);
  const void* f = reinterpret_cast<const void*>(spec_adj_table_kernel<NC>);
  if (lds > 32 * 1024) {
    hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(spec_adj_table_kernel<NC>, dim3(a.nklist), dim3(512), lds, s, a, nbp);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_spectral_adj(int nbp, const DysonArgs& a, int grid, hipStream_t s) {
  const int ncls = spec_adj_ncls(a.nc);
  const int what = a.mode & MODE_GEN ? (!a.nbar ? SPEC_GEN_G : a.gbar ? SPEC_GEN : SPEC_GEN_N)
                   : a.mode & MODE_ADJ ? SPEC_ADJ : SPEC_TRACE;
  if (what == SPEC_GEN || what == SPEC_GEN_N) {
    hipError_t e = hipErrorInvalidValue;
    switch (ncls) {
      case 5: e = table_launch<5>(nbp, a, s); break;
      case 8: e = table_launch<8>(nbp, a, s); break;
      case 10: e = table_launch<10>(nbp, a, s); break;
      case 14: e = table_launch<14>(nbp, a, s); break;
    }
    if (e != hipSuccess) return e;
  }
  switch (nbp) {
    case 16: return launch_spectral_adj_16(ncls, what, a, grid, s);
    case 32: return launch_spectral_adj_32(ncls, what, a, grid, s);
    case 48: return launch_spectral_adj_48(ncls, what, a, grid, s);
    case 64: return launch_spectral_adj_64(ncls, what, a, grid, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace dmft
