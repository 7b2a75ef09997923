// Step 2 with a variable coefficient: one geometric-multigrid V-cycle per
// frequency slice for (sigma_q I + tau K_a) z = r (Section 2.1 step 2;
// Section 3, Example 2: one V-cycle, Gauss-Seidel pre-smoother, no
// post-smoother).  All slices of all members go through one launch per level.
//
// Cycle (from z = 0; the lexicographic smoothers of mg_smoother = 1, 2 are
// described at their kernels):
//   smooth    one red-black Gauss-Seidel sweep, red = even index sum first.
//             Red points: z = r / d; black points use the red values
//             z_nb = r_nb / d_nb, recomputed on the fly, so the sweep is one
//             pass.  d = sigma_q + tau diag(K_a).
//   restrict  residual r - A z (zero at black points after the sweep, equal
//             to -sum_nb off z_nb at red points), written over the consumed
//             right-hand side, then full weighting to the coarse grid
//             (tensor product of [1/4, 1/2, 1/4]).
//   coarsest  one point: z = r / d.
//   prolong   z += P z_coarse (multilinear interpolation); the finest level
//             writes the result into the spectrum.
// Coarse operators are re-discretised: tau K_a on each level comes from the
// host with a at the level's face midpoints.  Coefficients per level:
// coef[0][i] = tau diag, coef[1 + 2a][i] / coef[2 + 2a][i] = tau times the
// minus / plus neighbour along axis a (zero where the neighbour is outside).
#include <atomic>
#include <cstdint>

#include "common.hpp"
#include "launch.hpp"

namespace pcop {

struct MgShift {
  const double* lam;    // [K] (re, im)
  const double* alpha;  // [B]
  const int* active;    // [B] or null
  int twoK;             // slices per member
};

template <class T>
__device__ __forceinline__ cx<T> slice_sigma(const MgShift& sh, int slice) {
  const int b = slice / sh.twoK;
  const int q = slice - b * sh.twoK;
  const int k = q >> 1;
  const double re = sh.lam[2 * k] + sh.alpha[b];
  const double im = (q & 1) ? -sh.lam[2 * k + 1] : sh.lam[2 * k + 1];
  return cx<T>{(T)re, (T)im};
}

// (point chunk, slice group) of this block in XCD-friendly order: the blocks
// one XCD runs take consecutive point chunks of a slice group, so the
// neighbour planes a block reads were brought into that XCD's L2 by the
// blocks next to it
__device__ __forceinline__ int2 mg_block() {
  const int lg = xcd_remap(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x * gridDim.y);
  return make_int2(lg % gridDim.x, lg / gridDim.x);
}

__device__ __forceinline__ void coords(int i, int nx, int dim, int* c) {
  c[0] = i % nx;
  c[1] = (i / nx) % nx;
  c[2] = (dim == 3) ? i / (nx * nx) : 0;
}

// one red-black sweep from z = 0.  A thread owns one point for SB
// consecutive slices: the point's stencil coefficients (and its neighbours'
// diagonals) are loaded once for all of them, since the coefficient arrays
// are shared by every slice and do not stay in the L2.
template <class T, int DIM, int SB>
__global__ void __launch_bounds__(256) mg_smooth_kernel(int nx, int m, int slices, const T* __restrict__ coef,
                                                        const cx<T>* __restrict__ r, cx<T>* __restrict__ z,
                                                        MgShift sh) {
  const int2 bk = mg_block();
  const int i = bk.x * blockDim.x + threadIdx.x;
  if (i >= m) return;
  int c[3];
  coords(i, nx, DIM, c);
  const bool red = ((c[0] + c[1] + c[2]) & 1) == 0;
  const T cdg = coef[i];
  // neighbour n = 2a (minus) / 2a + 1 (plus): offset, its diagonal, the
  // coupling weight; absent neighbours are skipped
  int nbo[2 * DIM];
  bool has[2 * DIM];
  T nbd[2 * DIM], off[2 * DIM];
  {
    int stride = 1;
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
      has[2 * a] = !red && c[a] > 0;
      has[2 * a + 1] = !red && c[a] < nx - 1;
      nbo[2 * a] = -stride;
      nbo[2 * a + 1] = stride;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int n = 2 * a + u;
        nbd[n] = has[n] ? coef[i + nbo[n]] : (T)0;
        off[n] = has[n] ? coef[(size_t)(1 + n) * m + i] : (T)0;
      }
      stride *= nx;
    }
  }
  const int s0 = bk.y * SB;
#pragma unroll
  for (int k = 0; k < SB; ++k) {
    const int s = s0 + k;
    if (s >= slices) break;
    if (sh.active && !sh.active[s / sh.twoK]) continue;
    const cx<T> sig = slice_sigma<T>(sh, s);
    const cx<T>* rs = r + (size_t)s * m;
    const cx<T> di = cx<T>{sig.x + cdg, sig.y};
    cx<T> acc = rs[i];
#pragma unroll
    for (int n = 0; n < 2 * DIM; ++n) {
      if (has[n]) {
        const cx<T> dn = cx<T>{sig.x + nbd[n], sig.y};
        acc = acc - scale(cdiv(rs[i + nbo[n]], dn), off[n]);
      }
    }
    z[(size_t)s * m + i] = cdiv(acc, di);
  }
}

// fine residual after the sweep, written at red points only (it is zero at
// black points); res may alias the level's right-hand side, which the sweep
// has consumed.  SB slices per thread, the coupling weights loaded once.
template <class T, int DIM, int SB>
__global__ void __launch_bounds__(256) mg_residual_kernel(int nx, int m, int slices, const T* __restrict__ coef,
                                                          const cx<T>* __restrict__ z, cx<T>* res, MgShift sh) {
  const int2 bk = mg_block();
  const int i = bk.x * blockDim.x + threadIdx.x;
  if (i >= m) return;
  int f[3];
  coords(i, nx, DIM, f);
  if (((f[0] + f[1] + f[2]) & 1) != 0) return;
  int nbo[2 * DIM];
  bool has[2 * DIM];
  T off[2 * DIM];
  {
    int stride = 1;
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
      has[2 * a] = f[a] > 0;
      has[2 * a + 1] = f[a] < nx - 1;
      nbo[2 * a] = -stride;
      nbo[2 * a + 1] = stride;
      off[2 * a] = has[2 * a] ? coef[(size_t)(1 + 2 * a) * m + i] : (T)0;
      off[2 * a + 1] = has[2 * a + 1] ? coef[(size_t)(2 + 2 * a) * m + i] : (T)0;
      stride *= nx;
    }
  }
  const int s0 = bk.y * SB;
#pragma unroll
  for (int k = 0; k < SB; ++k) {
    const int s = s0 + k;
    if (s >= slices) break;
    if (sh.active && !sh.active[s / sh.twoK]) continue;
    const cx<T>* zs = z + (size_t)s * m;
    // r - A z at a red point after the sweep: -sum over the neighbours of off z_nb
    // (minus then plus neighbour, axis by axis)
    cx<T> acc{0, 0};
#pragma unroll
    for (int n = 0; n < 2 * DIM; ++n)
      if (has[n]) acc = acc - scale(zs[i + nbo[n]], off[n]);
    res[(size_t)s * m + i] = acc;
  }
}

// The same sweep with a thread on a pair of neighbouring points of one
// x-row, x = 2u and 2u + 1 (the last pair of a row of odd length holds one
// point): one red and one black point, so every lane does the same work
// (with one point per thread the red half of each wave idles while the
// black half divides by its neighbours' diagonals).  The pairs of a row
// share the row's colour order.  Taken in FP32, where it was measured
// faster (3-D nx = 63, 128 slices, per V-cycle over all levels: smoother
// 0.295 -> 0.281 ms, residual and restriction 0.312 -> 0.279 ms); in FP64
// the per-point kernels above were faster (smoother 0.46 against 0.52 ms),
// the pair kernels' loads then touching every other 16-byte slot.
__device__ __forceinline__ int mg_pairs(int nx, int m) { return m / nx * ((nx + 1) >> 1); }

struct MgPair {
  int ir, ib;        // the pair's red and black point
  bool hr, hb;       // whether the pair holds them
};

template <int DIM>
__device__ __forceinline__ MgPair mg_pair(int u, int nx, int* cb) {
  const int P = (nx + 1) >> 1;
  const int row = u / P, pu = u - row * P;
  const int y = row % nx, zz = DIM == 3 ? row / nx : 0;
  const int x0 = 2 * pu;
  const bool two = x0 + 1 < nx;
  const bool first_red = ((x0 + y + zz) & 1) == 0;
  MgPair p;
  p.ir = row * nx + x0 + (first_red ? 0 : 1);
  p.ib = row * nx + x0 + (first_red ? 1 : 0);
  p.hr = first_red || two;
  p.hb = !first_red || two;
  // coordinates of the black point
  cb[0] = x0 + (first_red ? 1 : 0);
  cb[1] = y;
  cb[2] = zz;
  return p;
}

template <class T, int DIM, int SB>
__global__ void __launch_bounds__(256) mg_smooth_pair_kernel(int nx, int m, int slices, const T* __restrict__ coef,
                                                        const cx<T>* __restrict__ r, cx<T>* __restrict__ z,
                                                        MgShift sh) {
  const int2 bk = mg_block();
  const int u = bk.x * blockDim.x + threadIdx.x;
  if (u >= mg_pairs(nx, m)) return;
  int c[3];
  const MgPair pp = mg_pair<DIM>(u, nx, c);
  // red: z = r / d; black: the neighbours (all red) at their z = r / d
  const int ir = pp.hr ? pp.ir : pp.ib, ib = pp.hb ? pp.ib : pp.ir;  // in-range stand-ins
  const T cdr = coef[ir], cdb = coef[ib];
  // neighbour n = 2a (minus) / 2a + 1 (plus) of the black point: offset,
  // its diagonal, the coupling weight; absent neighbours are skipped
  int nbo[2 * DIM];
  bool has[2 * DIM];
  T nbd[2 * DIM], off[2 * DIM];
  {
    int stride = 1;
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
      has[2 * a] = pp.hb && c[a] > 0;
      has[2 * a + 1] = pp.hb && c[a] < nx - 1;
      nbo[2 * a] = -stride;
      nbo[2 * a + 1] = stride;
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        const int n = 2 * a + v;
        nbd[n] = has[n] ? coef[ib + nbo[n]] : (T)0;
        off[n] = has[n] ? coef[(size_t)(1 + n) * m + ib] : (T)0;
      }
      stride *= nx;
    }
  }
  const int s0 = bk.y * SB;
#pragma unroll
  for (int k = 0; k < SB; ++k) {
    const int s = s0 + k;
    if (s >= slices) break;
    if (sh.active && !sh.active[s / sh.twoK]) continue;
    const cx<T> sig = slice_sigma<T>(sh, s);
    const cx<T>* rs = r + (size_t)s * m;
    cx<T>* zs = z + (size_t)s * m;
    if (pp.hr) zs[ir] = cdiv(rs[ir], cx<T>{sig.x + cdr, sig.y});
    if (pp.hb) {
      cx<T> acc = rs[ib];
#pragma unroll
      for (int n = 0; n < 2 * DIM; ++n) {
        if (has[n]) {
          const cx<T> dn = cx<T>{sig.x + nbd[n], sig.y};
          acc = acc - scale(cdiv(rs[ib + nbo[n]], dn), off[n]);
        }
      }
      zs[ib] = cdiv(acc, cx<T>{sig.x + cdb, sig.y});
    }
  }
}

// the residual at the red point of one pair (mg_pair) per thread, so that no
// lane idles at a black point (FP32; see the pair smoother)
template <class T, int DIM, int SB>
__global__ void __launch_bounds__(256) mg_residual_pair_kernel(int nx, int m, int slices, const T* __restrict__ coef,
                                                          const cx<T>* __restrict__ z, cx<T>* res, MgShift sh) {
  const int2 bk = mg_block();
  const int u = bk.x * blockDim.x + threadIdx.x;
  if (u >= mg_pairs(nx, m)) return;
  int cbk[3];
  const MgPair pp = mg_pair<DIM>(u, nx, cbk);
  if (!pp.hr) return;
  const int i = pp.ir;
  int f[3];
  coords(i, nx, DIM, f);
  int nbo[2 * DIM];
  bool has[2 * DIM];
  T off[2 * DIM];
  {
    int stride = 1;
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
      has[2 * a] = f[a] > 0;
      has[2 * a + 1] = f[a] < nx - 1;
      nbo[2 * a] = -stride;
      nbo[2 * a + 1] = stride;
      off[2 * a] = has[2 * a] ? coef[(size_t)(1 + 2 * a) * m + i] : (T)0;
      off[2 * a + 1] = has[2 * a + 1] ? coef[(size_t)(2 + 2 * a) * m + i] : (T)0;
      stride *= nx;
    }
  }
  const int s0 = bk.y * SB;
#pragma unroll
  for (int k = 0; k < SB; ++k) {
    const int s = s0 + k;
    if (s >= slices) break;
    if (sh.active && !sh.active[s / sh.twoK]) continue;
    const cx<T>* zs = z + (size_t)s * m;
    // r - A z at a red point after the sweep: -sum over the neighbours of off z_nb
    // (minus then plus neighbour, axis by axis)
    cx<T> acc{0, 0};
#pragma unroll
    for (int n = 0; n < 2 * DIM; ++n)
      if (has[n]) acc = acc - scale(zs[i + nbo[n]], off[n]);
    res[(size_t)s * m + i] = acc;
  }
}

// coarse right-hand side by full weighting of the fine residual (red points
// only after a red-black sweep, where the black ones are zero; ALL: every
// point, after the lexicographic sweeps)
template <class T, int DIM, bool ALL>
__global__ void __launch_bounds__(256) mg_restrict_kernel(int nxf, int mf, int nxc, int mc,
                                                          const cx<T>* __restrict__ res, cx<T>* __restrict__ rc,
                                                          MgShift sh) {
  const int2 bk = mg_block();
  const int s = bk.y;
  if (sh.active && !sh.active[s / sh.twoK]) return;
  const int I = bk.x * blockDim.x + threadIdx.x;
  if (I >= mc) return;
  int C[3];
  coords(I, nxc, DIM, C);
  const cx<T>* rs = res + (size_t)s * mf;
  cx<T> acc{0, 0};
  const int o2 = (DIM == 3) ? 1 : 0;
  for (int d2 = -o2; d2 <= o2; ++d2)
    for (int d1 = -1; d1 <= 1; ++d1)
      for (int d0 = -1; d0 <= 1; ++d0) {
        const int f0 = 2 * C[0] + 1 + d0, f1 = 2 * C[1] + 1 + d1, f2 = (DIM == 3) ? 2 * C[2] + 1 + d2 : 0;
        if (!ALL && ((f0 + f1 + f2) & 1) != 0) continue;
        const T w = (d0 == 0 ? (T)1 : (T)0.5) * (d1 == 0 ? (T)1 : (T)0.5) * (d2 == 0 ? (T)1 : (T)0.5);
        acc = acc + scale(rs[f0 + nxf * (f1 + nxf * f2)], w);
      }
  const T inv = (DIM == 3) ? (T)0.125 : (T)0.25;
  rc[(size_t)s * mc + I] = scale(acc, inv);
}

// out = z_fine + P z_coarse (out may alias z_fine).  A thread owns one fine
// point for SB consecutive slices: its coarse indices and weights are formed
// once for all of them.
template <class T, int DIM, int SB>
__global__ void __launch_bounds__(256) mg_prolong_kernel(int nxf, int mf, int nxc, int mc, int slices,
                                                         const cx<T>* __restrict__ zf, const cx<T>* __restrict__ zc,
                                                         cx<T>* out, MgShift sh) {
  const int2 bk = mg_block();
  const int i = bk.x * blockDim.x + threadIdx.x;
  if (i >= mf) return;
  int f[3];
  coords(i, nxf, DIM, f);
  // per axis two coarse candidates, clamped in bounds, with weights that are
  // zero where a candidate does not contribute: fine 2I + 1 sits on coarse I
  // (weights 1, 0); fine 2I lies between coarse I - 1 and I (1/2 each, 0 for
  // a candidate outside the grid).  Every thread then issues the same
  // 2^DIM unconditional loads per slice (no divergent loop over 1..8
  // contributions), and indices and weights are formed once for SB slices.
  int ci[DIM][2];
  T cw[DIM][2];
#pragma unroll
  for (int a = 0; a < DIM; ++a) {
    const int I = f[a] >> 1;
    if (f[a] & 1) {
      ci[a][0] = I;
      ci[a][1] = I;
      cw[a][0] = (T)1;
      cw[a][1] = (T)0;
    } else {
      ci[a][0] = I >= 1 ? I - 1 : 0;
      ci[a][1] = I < nxc ? I : nxc - 1;
      cw[a][0] = I >= 1 ? (T)0.5 : (T)0;
      cw[a][1] = I < nxc ? (T)0.5 : (T)0;
    }
  }
  constexpr int NC = 1 << DIM;
  int cidx[NC];
  T cwt[NC];
#pragma unroll
  for (int u = 0; u < NC; ++u) {
    int I = 0, stride = 1;
    T wt = (T)1;
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
      const int b = (u >> a) & 1;
      I += ci[a][b] * stride;
      wt *= cw[a][b];
      stride *= nxc;
    }
    cidx[u] = I;
    cwt[u] = wt;
  }
  const int s0 = bk.y * SB;
#pragma unroll
  for (int k = 0; k < SB; ++k) {
    const int s = s0 + k;
    if (s >= slices) break;
    if (sh.active && !sh.active[s / sh.twoK]) continue;
    const cx<T>* zcs = zc + (size_t)s * mc;
    cx<T> acc = zf[(size_t)s * mf + i];
#pragma unroll
    for (int u = 0; u < NC; ++u) acc = acc + scale(zcs[cidx[u]], cwt[u]);
    out[(size_t)s * mf + i] = acc;
  }
}

// ---------------------------------------------------------------------------
// Lexicographic Gauss-Seidel (mg_smoother = 1, and = 2 followed by the
// reverse sweep): the natural order (x1 fastest) makes point x depend on its
// minus neighbours, which lie on the hyperplane x1 + x2 (+ x3) one below.
// One block per slice walks the hyperplanes in order (reverse order for the
// backward sweep) with a block barrier between them; the points of one
// hyperplane are independent.  z lives in global memory (a slice does not fit
// LDS); within a block the barrier orders the stores and the later loads.
//   forward   z_x = (r_x - sum_{minus nb} off z_nb) / d_x          (z = 0 before)
//   backward  z_x = (r_x - sum_{all nb} off z_nb) / d_x             (in place)
// ---------------------------------------------------------------------------
template <class T, int DIM, bool BACK>
__global__ void __launch_bounds__(256) mg_sweep_lex_kernel(int nx, int m, const T* __restrict__ coef,
                                                           const cx<T>* __restrict__ r, cx<T>* z, MgShift sh) {
  const int s = blockIdx.x;
  if (sh.active && !sh.active[s / sh.twoK]) return;
  const cx<T> sig = slice_sigma<T>(sh, s);
  const cx<T>* rs = r + (size_t)s * m;
  cx<T>* zs = z + (size_t)s * m;
  const int top = DIM * (nx - 1);
  for (int step = 0; step <= top; ++step) {
    const int w = BACK ? top - step : step;
    // points with x1 + x2 (+ x3) = w: x3 (3-D) and x1 over a box, x2 from w
    const int x3lo = DIM == 3 ? max(0, w - 2 * (nx - 1)) : 0;
    const int x3hi = DIM == 3 ? min(w, nx - 1) : 0;
    const int box = (x3hi - x3lo + 1) * nx;
    for (int t = threadIdx.x; t < box; t += blockDim.x) {
      const int x3 = x3lo + t / nx, x1 = t - (t / nx) * nx;
      const int x2 = w - x3 - x1;
      if (x2 < 0 || x2 >= nx) continue;
      const int c[3] = {x1, x2, x3};
      const int i = x1 + nx * (x2 + nx * x3);
      cx<T> acc = rs[i];
      int stride = 1;
#pragma unroll
      for (int a = 0; a < DIM; ++a) {
        if (c[a] > 0) acc = acc - scale(zs[i - stride], coef[(size_t)(1 + 2 * a) * m + i]);
        if (BACK && c[a] < nx - 1) acc = acc - scale(zs[i + stride], coef[(size_t)(2 + 2 * a) * m + i]);
        stride *= nx;
      }
      zs[i] = cdiv(acc, cx<T>{sig.x + coef[i], sig.y});
    }
    __syncthreads();
  }
}

// r <- r - A z at every point (in place: each point reads only its own r),
// for the lexicographic sweeps, after which the residual is nonzero everywhere
template <class T, int DIM, int SB>
__global__ void __launch_bounds__(256) mg_residual_full_kernel(int nx, int m, int slices, const T* __restrict__ coef,
                                                               const cx<T>* __restrict__ z, cx<T>* res, MgShift sh) {
  const int2 bk = mg_block();
  const int i = bk.x * blockDim.x + threadIdx.x;
  if (i >= m) return;
  int f[3];
  coords(i, nx, DIM, f);
  int nbo[2 * DIM];
  bool has[2 * DIM];
  T off[2 * DIM];
  {
    int stride = 1;
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
      has[2 * a] = f[a] > 0;
      has[2 * a + 1] = f[a] < nx - 1;
      nbo[2 * a] = -stride;
      nbo[2 * a + 1] = stride;
      off[2 * a] = has[2 * a] ? coef[(size_t)(1 + 2 * a) * m + i] : (T)0;
      off[2 * a + 1] = has[2 * a + 1] ? coef[(size_t)(2 + 2 * a) * m + i] : (T)0;
      stride *= nx;
    }
  }
  const T cdg = coef[i];
  const int s0 = bk.y * SB;
#pragma unroll
  for (int k = 0; k < SB; ++k) {
    const int s = s0 + k;
    if (s >= slices) break;
    if (sh.active && !sh.active[s / sh.twoK]) continue;
    const cx<T> sig = slice_sigma<T>(sh, s);
    const cx<T>* zs = z + (size_t)s * m;
    const cx<T> zi = zs[i];
    // (sigma + cdg) z_i
    cx<T> acc = res[(size_t)s * m + i] - cx<T>{(sig.x + cdg) * zi.x - sig.y * zi.y, (sig.x + cdg) * zi.y + sig.y * zi.x};
#pragma unroll
    for (int n = 0; n < 2 * DIM; ++n)
      if (has[n]) acc = acc - scale(zs[i + nbo[n]], off[n]);
    res[(size_t)s * m + i] = acc;
  }
}

// ---------------------------------------------------------------------------
// Two-dimensional lexicographic sweeps by one wave per slice.  Lane t owns
// column x1 = t (from the other end for the backward sweep) and walks along
// x2, one step behind its neighbour: the point it handles at step w lies on
// the hyperplane x1 + x2 = w, its new x1-neighbour is what lane t - 1 computed
// at the step before (a lane shift) and its new x2-neighbour is its own last
// value, so no barrier and no memory lies between two hyperplanes.  What does
// not depend on the sweep (right-hand side, coefficients, reciprocal of |d|^2,
// in the backward sweep the old neighbours) is read kSweepAhead steps ahead.
// C > 1: a lane owns C neighbouring columns, updated one after another.
// What bounds a sweep is the chain of 2 nx - 1 updates (nx + 64 steps of C) and
// the 64 lines per load that the skewed accesses touch (eight steps ahead
// instead of four changed nothing).  FP64, one member, nt = 64, symmetric
// sweeps, one apply: nx = 127 1165 -> 403 us, nx = 255 (nt = 32) 2552 -> 1461.
// ---------------------------------------------------------------------------
constexpr int kSweepAhead = 4;

// the value of the lane below (0 in lane 0)
__device__ __forceinline__ float lane_below(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ double lane_below(double v) {
  return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x138, 0xf, 0xf, true),
                          __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x138, 0xf, 0xf, true));
}

// r and z: one slice, in LDS or global memory
template <class T, int C, bool BACK, class RP, class ZP>
__device__ __forceinline__ void sweep_columns(int nx, int m, const T* __restrict__ coef, const RP r, ZP z,
                                              cx<T> sig) {
  const int t = threadIdx.x & (kWave - 1);
  const int last = (nx + C - 1) / C - 1;  // lane of the last column
  // step w of lane t: row w - t (counted from the far end when BACK)
  auto point = [&](int w, int u) {
    const int e = C * t + u, row = min(max(w - t, 0), nx - 1);
    const int x1 = min(e, nx - 1);
    return BACK ? (nx - 1 - x1) + nx * (nx - 1 - row) : x1 + nx * row;
  };
  struct Pre {
    cx<T> a;      // right-hand side, less the old neighbours' part when BACK
    T o1, o2;     // couplings to the neighbour columns / rows already done
    T dx, rd;     // Re d and 1 / |d|^2
  };
  auto fetch = [&](int w, Pre (&q)[C]) {
#pragma unroll
    for (int u = 0; u < C; ++u) {
      const int i = point(w, u);
      q[u].a = r[i];
      q[u].dx = sig.x + coef[i];
      q[u].rd = recip(q[u].dx * q[u].dx + sig.y * sig.y);
      q[u].o1 = coef[(size_t)(BACK ? 2 : 1) * m + i];
      q[u].o2 = coef[(size_t)(BACK ? 4 : 3) * m + i];
      if (BACK) {
        // minus neighbours, not yet updated (zero coupling where outside)
        const T b1 = coef[(size_t)m + i], b2 = coef[(size_t)3 * m + i];
        q[u].a = q[u].a - scale(z[max(i - 1, 0)], b1);
        q[u].a = q[u].a - scale(z[max(i - nx, 0)], b2);
      }
    }
  };
  cx<T> own[C];
#pragma unroll
  for (int u = 0; u < C; ++u) own[u] = cx<T>{0, 0};
  auto step = [&](int w, Pre (&q)[C]) {
    const int row = w - t;
    const bool in = row >= 0 && row < nx && t <= last;
    cx<T> side{lane_below(own[C - 1].x), lane_below(own[C - 1].y)};
#pragma unroll
    for (int u = 0; u < C; ++u) {
      cx<T> a = q[u].a - scale(side, q[u].o1);
      a = a - scale(own[u], q[u].o2);
      const cx<T> v{(a.x * q[u].dx + a.y * sig.y) * q[u].rd, (a.y * q[u].dx - a.x * sig.y) * q[u].rd};
      own[u] = in ? v : cx<T>{0, 0};
      if (in && C * t + u < nx) z[point(w, u)] = own[u];
      side = own[u];
    }
  };
  Pre q[kSweepAhead][C];
#pragma unroll
  for (int k = 0; k < kSweepAhead; ++k) fetch(k, q[k]);
  const int steps = nx + last;
  for (int w = 0; w < steps; w += kSweepAhead) {
#pragma unroll
    for (int k = 0; k < kSweepAhead; ++k) {
      step(w + k, q[k]);
      fetch(w + k + kSweepAhead, q[k]);
    }
  }
}

template <class T, int C>
__global__ void __launch_bounds__(kWave) mg_sweep_columns_kernel(int nx, int m, const T* __restrict__ coef,
                                                                 const cx<T>* __restrict__ r, cx<T>* z, MgShift sh,
                                                                 int back) {
  const int s = blockIdx.x;
  if (sh.active && !sh.active[s / sh.twoK]) return;
  const cx<T> sig = slice_sigma<T>(sh, s);
  const cx<T>* rs = r + (size_t)s * m;
  cx<T>* zs = z + (size_t)s * m;
  if (back) sweep_columns<T, C, true>(nx, m, coef, rs, zs, sig);
  else sweep_columns<T, C, false>(nx, m, coef, rs, zs, sig);
}

// ---------------------------------------------------------------------------
// The cycle's coarse end in one launch: a block takes one slice through every
// level from the first that fits LDS (2-D nx <= 63, 3-D nx <= 15) down to one
// point and back up.  Level by level these were three or four launches each of
// a few microseconds' work (and one block per slice of dependent hyperplanes
// for the lexicographic sweeps).  The level below the first keeps its
// correction where the first level's residual was, which its restriction has
// consumed.  Operations per point as in the kernels above.
// What bounds it is latency: one block per slice, a barrier per phase.  One
// apply, 64 slices, level by level and so: 2-D nx = 63 FP64 red-black 98 -> 55
// us, lexicographic 246 -> 82, symmetric 478 -> 129; 3-D nx = 15 66 -> 53,
// 121 -> 97, 216 -> 169 (tail_level says where it is taken).
// ---------------------------------------------------------------------------
constexpr int kTailThreads = 512;  // at most
constexpr size_t kTailLds = 160 * 1024 - 1024;

template <class T>
struct MgTail {
  int levels;
  int nx[kMaxMgLevels];
  const T* coef[kMaxMgLevels];
};

template <class T, int DIM>
__global__ void __launch_bounds__(kTailThreads) mg_tail_kernel(MgTail<T> lv, const cx<T>* rin, cx<T>* out, MgShift sh,
                                                               int smoother) {
  extern __shared__ __align__(16) unsigned char tail_sm[];
  const int s = blockIdx.x;
  if (sh.active && !sh.active[s / sh.twoK]) return;
  const cx<T> sig = slice_sigma<T>(sh, s);
  cx<T>* const base = reinterpret_cast<cx<T>*>(tail_sm);
  const int tid = threadIdx.x;
  auto points = [](int nx) { return DIM == 3 ? nx * nx * nx : nx * nx; };
  const int m0 = points(lv.nx[0]);
  // z of the first level, its right-hand side (and later the corrections of
  // the coarser levels), the coarser right-hand sides
  cx<T>* z = base;
  cx<T>* r = base + m0;
  cx<T>* znext = base + m0;
  cx<T>* rnext = base + 2 * m0;
  for (int i = tid; i < m0; i += (int)blockDim.x) r[i] = rin[(size_t)s * m0 + i];
  __syncthreads();
  for (int l = 0; l < lv.levels; ++l) {
    const int nx = lv.nx[l], m = points(nx);
    const T* __restrict__ coef = lv.coef[l];
    if (smoother == 0) {
      for (int i = tid; i < m; i += (int)blockDim.x) {
        int c[3];
        coords(i, nx, DIM, c);
        cx<T> acc = r[i];
        if (((c[0] + c[1] + c[2]) & 1) != 0) {
          int stride = 1;
#pragma unroll
          for (int a = 0; a < DIM; ++a) {
            if (c[a] > 0)
              acc = acc - scale(cdiv(r[i - stride], cx<T>{sig.x + coef[i - stride], sig.y}), coef[(size_t)(1 + 2 * a) * m + i]);
            if (c[a] < nx - 1)
              acc = acc - scale(cdiv(r[i + stride], cx<T>{sig.x + coef[i + stride], sig.y}), coef[(size_t)(2 + 2 * a) * m + i]);
            stride *= nx;
          }
        }
        z[i] = cdiv(acc, cx<T>{sig.x + coef[i], sig.y});
      }
    } else if (DIM == 2) {
      if (tid < kWave) {
        sweep_columns<T, 1, false>(nx, m, coef, r, z, sig);
        if (smoother == 2) {
          // one wave's LDS accesses complete in order
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
          __builtin_amdgcn_wave_barrier();
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
          sweep_columns<T, 1, true>(nx, m, coef, r, z, sig);
        }
      }
    } else {
      const int top = DIM * (nx - 1);
      for (int pass = 0; pass < smoother; ++pass) {
        for (int st = 0; st <= top; ++st) {
          const int w = pass ? top - st : st;
          const int x3lo = max(0, w - 2 * (nx - 1)), x3hi = min(w, nx - 1);
          for (int t = tid; t < (x3hi - x3lo + 1) * nx; t += (int)blockDim.x) {
            const int x3 = x3lo + t / nx, x1 = t % nx, x2 = w - x3 - x1;
            if (x2 < 0 || x2 >= nx) continue;
            const int c[3] = {x1, x2, x3};
            const int i = x1 + nx * (x2 + nx * x3);
            cx<T> acc = r[i];
            int stride = 1;
#pragma unroll
            for (int a = 0; a < DIM; ++a) {
              if (c[a] > 0) acc = acc - scale(z[i - stride], coef[(size_t)(1 + 2 * a) * m + i]);
              if (pass && c[a] < nx - 1) acc = acc - scale(z[i + stride], coef[(size_t)(2 + 2 * a) * m + i]);
              stride *= nx;
            }
            z[i] = cdiv(acc, cx<T>{sig.x + coef[i], sig.y});
          }
          __syncthreads();
        }
      }
    }
    __syncthreads();
    if (l + 1 == lv.levels) break;
    // residual over the consumed right-hand side (red-black: the red points)
    for (int i = tid; i < m; i += (int)blockDim.x) {
      int c[3];
      coords(i, nx, DIM, c);
      cx<T> acc{0, 0};
      if (smoother == 0) {
        if (((c[0] + c[1] + c[2]) & 1) != 0) continue;
      } else {
        const T dx = sig.x + coef[i];
        const cx<T> zi = z[i];
        acc = r[i] - cx<T>{dx * zi.x - sig.y * zi.y, dx * zi.y + sig.y * zi.x};
      }
      int stride = 1;
#pragma unroll
      for (int a = 0; a < DIM; ++a) {
        if (c[a] > 0) acc = acc - scale(z[i - stride], coef[(size_t)(1 + 2 * a) * m + i]);
        if (c[a] < nx - 1) acc = acc - scale(z[i + stride], coef[(size_t)(2 + 2 * a) * m + i]);
        stride *= nx;
      }
      r[i] = acc;
    }
    __syncthreads();
    const int nxc = lv.nx[l + 1], mc = points(nxc);
    for (int I = tid; I < mc; I += (int)blockDim.x) {
      int C[3];
      coords(I, nxc, DIM, C);
      cx<T> acc{0, 0};
      const int o2 = (DIM == 3) ? 1 : 0;
      for (int d2 = -o2; d2 <= o2; ++d2)
        for (int d1 = -1; d1 <= 1; ++d1)
          for (int d0 = -1; d0 <= 1; ++d0) {
            const int f0 = 2 * C[0] + 1 + d0, f1 = 2 * C[1] + 1 + d1, f2 = (DIM == 3) ? 2 * C[2] + 1 + d2 : 0;
            if (smoother == 0 && ((f0 + f1 + f2) & 1) != 0) continue;
            const T w = (d0 == 0 ? (T)1 : (T)0.5) * (d1 == 0 ? (T)1 : (T)0.5) * (d2 == 0 ? (T)1 : (T)0.5);
            acc = acc + scale(r[f0 + nx * (f1 + nx * f2)], w);
          }
      rnext[I] = scale(acc, (DIM == 3) ? (T)0.125 : (T)0.25);
    }
    __syncthreads();
    z = znext;
    znext += mc;
    r = rnext;
    rnext += mc;
  }
  // z is the coarsest correction; the finer ones lie before it
  for (int l = lv.levels - 2; l >= 0; --l) {
    const int nx = lv.nx[l], m = points(nx), nxc = lv.nx[l + 1];
    cx<T>* zf = l == 0 ? base : z - m;
    for (int i = tid; i < m; i += (int)blockDim.x) {
      int f[3];
      coords(i, nx, DIM, f);
      int ci[DIM][2];
      T cw[DIM][2];
#pragma unroll
      for (int a = 0; a < DIM; ++a) {
        const int I = f[a] >> 1;
        const bool on = f[a] & 1;
        ci[a][0] = on ? I : max(I - 1, 0);
        ci[a][1] = on ? I : min(I, nxc - 1);
        cw[a][0] = on ? (T)1 : (I >= 1 ? (T)0.5 : (T)0);
        cw[a][1] = on ? (T)0 : (I < nxc ? (T)0.5 : (T)0);
      }
      cx<T> acc = zf[i];
#pragma unroll
      for (int u = 0; u < (1 << DIM); ++u) {
        int I = 0, stride = 1;
        T wt = (T)1;
#pragma unroll
        for (int a = 0; a < DIM; ++a) {
          const int b = (u >> a) & 1;
          I += ci[a][b] * stride;
          wt *= cw[a][b];
          stride *= nxc;
        }
        acc = acc + scale(z[I], wt);
      }
      zf[i] = acc;
    }
    __syncthreads();
    z = zf;
  }
  for (int i = tid; i < m0; i += (int)blockDim.x) out[(size_t)s * m0 + i] = base[i];
}

// first level of the one-launch coarse end: its two planes and the coarser
// right-hand sides fit LDS, and a 2-D column per lane.  Where that is one block
// per CU (FP64 2-D nx = 63, 3-D nx = 15) the slices run in rounds of one per
// CU, each a chain of barriers; a level by itself runs on all slices at once.
// The red-black sweep has no chain to shorten and is faster by itself on any
// number of slices, the lexicographic ones from some rounds on.  In this launch
// against by itself, FP64, us per apply: 64 slices red-black 3-D nx = 15 53 /
// 47, 2-D nx = 63 55 / 50, lexicographic 97 / 103, 82 / 98, symmetric 169 /
// 185, 129 / 169; 512 slices lexicographic 247 / 206, 192 / 187, symmetric 413
// / 335, 286 / 319; 2048 slices 870 / 701, 726 / 629, 1477 / 1197, 1106 / 1120.
template <class T, int DIM>
static int tail_level(const PrecondTables& tb, int slices, size_t most, size_t* lds) {
  for (int l = 0; l < tb.mg_levels; ++l) {
    size_t pts = tb.mg[l].m;
    for (int k = l; k < tb.mg_levels; ++k) pts += tb.mg[k].m;
    *lds = pts * sizeof(cx<T>);
    if (*lds > most || tb.mg[l].nx > kWave) continue;
    if (2 * *lds > kTailLds && (tb.mg_smoother == 0 || slices > (DIM == 3 ? 1 : 4) * (long long)tb.ncu)) continue;
    return l;
  }
  return tb.mg_levels;
}

// LDS that the coarse end's blocks may take on the current device: more than 64
// KB has to be asked for once on each
template <class T, int DIM>
static size_t tail_lds_limit() {
  constexpr size_t kPlain = 64 * 1024;
  static std::atomic<uint64_t> granted{0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) return kPlain;
  const uint64_t bit = dev < 64 ? uint64_t(1) << dev : 0;
  if (granted.load() & bit) return kTailLds;
  if (hipFuncSetAttribute(reinterpret_cast<const void*>(&mg_tail_kernel<T, DIM>),
                          hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess) {
    (void)hipGetLastError();
    return kPlain;
  }
  granted.fetch_or(bit);
  return kTailLds;
}

// threads of a block whose first level has m points.  With a block per CU and
// fewer the most, whose idle waves cost nothing; beyond, waves that only meet
// barriers keep other slices out (FP64 red-black, thousands of slices, 512
// threads against these: 2-D nx = 7 127 -> 45 us, nx = 15 197 -> 117, nx = 31
// 218 -> 188; symmetric 274 -> 102, 519 -> 246, 543 -> 366; 3-D nx = 7 285 ->
// 185).
static int tail_threads(long long m, int slices, int ncu) {
  if (slices <= ncu || m > 1024) return kTailThreads;
  return m > 256 ? 256 : m > 64 ? 128 : 64;
}

// slices per thread of the smoother, the residual and the prolongation on
// levels where that still gives at least kMgMinBlocks blocks (one slice per
// thread below)
constexpr int kMgSB = 8;
constexpr long long kMgMinBlocks = 1024;

template <class T, int DIM>
static void mg_cycle(const Geo& g, cx<T>* spec, const PrecondTables& tb, int spm, const double* lam,
                     hipStream_t st) {
  const int NL = tb.mg_levels;
  const int slices = g.B * spm;
  MgShift sh{lam, tb.alpha, tb.active, spm};
  // the smoother: red-black (0), lexicographic (1), symmetric lexicographic (2)
  const bool lex = tb.mg_smoother != 0;
  auto coefp = [&](int l) -> const T* {
    return reinterpret_cast<const T*>(sizeof(T) == 4 ? (const void*)tb.mg[l].coef : (const void*)tb.mg[l].coef64);
  };
  auto zbuf = [&](int l) -> cx<T>* {
    return reinterpret_cast<cx<T>*>(l == 0 ? tb.mg[0].r : tb.mg[l].z);
  };
  auto rbuf = [&](int l) -> cx<T>* { return l == 0 ? spec : reinterpret_cast<cx<T>*>(tb.mg[l].r); };
  // pass bytes (algorithmic): complex data in and out of every kernel
  const double cs = sizeof(cx<T>) * (double)slices * tb.nact / g.B;
  // kMgSB slices per thread where that still leaves kMgMinBlocks blocks to
  // fill the chip, one slice per thread on the small (coarse) levels
  auto wide = [&](int m) { return (long long)((m + 255) / 256) * ((slices + kMgSB - 1) / kMgSB) >= kMgMinBlocks; };
  auto grid_sb = [&](int m) {
    const int sb = wide(m) ? kMgSB : 1;
    return dim3((m + 255) / 256, (slices + sb - 1) / sb);
  };
  // the red-black smoother and residual in FP32: one thread per pair of
  // points, with the slice grouping of the level (wide(m))
  constexpr bool pair = sizeof(T) == 4;
  auto grid_pair = [&](int nx, int m) {
    const int sb = wide(m) ? kMgSB : 1;
    const int np = m / nx * ((nx + 1) / 2);
    return dim3((np + 255) / 256, (slices + sb - 1) / sb);
  };
  // levels from lt on in one launch (one point at the latest)
  size_t tail_lds = 0;
  const int lt = tail_level<T, DIM>(tb, slices, tail_lds_limit<T, DIM>(), &tail_lds);
  for (int l = 0; l < lt; ++l) {
    const int nx = tb.mg[l].nx;
    const int m = (int)tb.mg[l].m;
    const dim3 gridb = grid_sb(m);
    tbeg(tb.timer, KF_MG_SMOOTH, 2.0 * cs * m);
    if (lex) {
      for (int back = 0; back < tb.mg_smoother; ++back) {
        // one wave per slice up to four columns per lane; wider grids walk
        // the hyperplanes with a block
        if (DIM == 2 && nx <= 2 * kWave)
          mg_sweep_columns_kernel<T, 2><<<slices, kWave, 0, st>>>(nx, m, coefp(l), rbuf(l), zbuf(l), sh, back);
        else if (DIM == 2 && nx <= 4 * kWave)
          mg_sweep_columns_kernel<T, 4><<<slices, kWave, 0, st>>>(nx, m, coefp(l), rbuf(l), zbuf(l), sh, back);
        else if (back)
          mg_sweep_lex_kernel<T, DIM, true><<<slices, 256, 0, st>>>(nx, m, coefp(l), rbuf(l), zbuf(l), sh);
        else
          mg_sweep_lex_kernel<T, DIM, false><<<slices, 256, 0, st>>>(nx, m, coefp(l), rbuf(l), zbuf(l), sh);
      }
    } else if (pair) {
      if (wide(m))
        mg_smooth_pair_kernel<T, DIM, kMgSB><<<grid_pair(nx, m), 256, 0, st>>>(nx, m, slices, coefp(l), rbuf(l), zbuf(l), sh);
      else
        mg_smooth_pair_kernel<T, DIM, 1><<<grid_pair(nx, m), 256, 0, st>>>(nx, m, slices, coefp(l), rbuf(l), zbuf(l), sh);
    } else if (wide(m)) {
      mg_smooth_kernel<T, DIM, kMgSB><<<gridb, 256, 0, st>>>(nx, m, slices, coefp(l), rbuf(l), zbuf(l), sh);
    } else {
      mg_smooth_kernel<T, DIM, 1><<<gridb, 256, 0, st>>>(nx, m, slices, coefp(l), rbuf(l), zbuf(l), sh);
    }
    tend(tb.timer);
    {
      const int nxc = tb.mg[l + 1].nx;
      const int mc = (int)tb.mg[l + 1].m;
      dim3 gc((mc + 255) / 256, slices);
      // residual into the consumed right-hand side (half the points), then
      // full weighting
      if (lex) {
        // r - A z at every point, in place, then full weighting of all points
        tbeg(tb.timer, KF_MG_RESTRICT, cs * (3.0 * m + m + mc));
        if (wide(m))
          mg_residual_full_kernel<T, DIM, kMgSB><<<gridb, 256, 0, st>>>(nx, m, slices, coefp(l), zbuf(l), rbuf(l), sh);
        else
          mg_residual_full_kernel<T, DIM, 1><<<gridb, 256, 0, st>>>(nx, m, slices, coefp(l), zbuf(l), rbuf(l), sh);
        mg_restrict_kernel<T, DIM, true><<<gc, 256, 0, st>>>(nx, m, nxc, mc, rbuf(l), rbuf(l + 1), sh);
      } else {
        tbeg(tb.timer, KF_MG_RESTRICT, cs * (m + 0.5 * m + 0.5 * m + mc));
        if (pair && wide(m))
          mg_residual_pair_kernel<T, DIM, kMgSB><<<grid_pair(nx, m), 256, 0, st>>>(nx, m, slices, coefp(l), zbuf(l), rbuf(l), sh);
        else if (pair)
          mg_residual_pair_kernel<T, DIM, 1><<<grid_pair(nx, m), 256, 0, st>>>(nx, m, slices, coefp(l), zbuf(l), rbuf(l), sh);
        else if (wide(m))
          mg_residual_kernel<T, DIM, kMgSB><<<gridb, 256, 0, st>>>(nx, m, slices, coefp(l), zbuf(l), rbuf(l), sh);
        else
          mg_residual_kernel<T, DIM, 1><<<gridb, 256, 0, st>>>(nx, m, slices, coefp(l), zbuf(l), rbuf(l), sh);
        mg_restrict_kernel<T, DIM, false><<<gc, 256, 0, st>>>(nx, m, nxc, mc, rbuf(l), rbuf(l + 1), sh);
      }
      tend(tb.timer);
    }
  }
  {
    MgTail<T> lv{NL - lt, {}, {}};
    for (int l = lt; l < NL; ++l) {
      lv.nx[l - lt] = tb.mg[l].nx;
      lv.coef[l - lt] = coefp(l);
    }
    tbeg(tb.timer, KF_MG_SMOOTH, 2.0 * cs * tb.mg[lt].m);
    mg_tail_kernel<T, DIM><<<slices, tail_threads(tb.mg[lt].m, slices, tb.ncu), tail_lds, st>>>(
        lv, rbuf(lt), lt == 0 ? spec : zbuf(lt), sh, tb.mg_smoother);
    tend(tb.timer);
  }
  for (int l = lt - 1; l >= 0; --l) {
    const int nx = tb.mg[l].nx;
    const int m = (int)tb.mg[l].m;
    const int nxc = tb.mg[l + 1].nx;
    const int mc = (int)tb.mg[l + 1].m;
    const dim3 gridb = grid_sb(m);
    cx<T>* out = (l == 0) ? spec : zbuf(l);
    tbeg(tb.timer, KF_MG_PROLONG, cs * (2.0 * m + mc));
    if (wide(m))
      mg_prolong_kernel<T, DIM, kMgSB><<<gridb, 256, 0, st>>>(nx, m, nxc, mc, slices, zbuf(l), zbuf(l + 1), out, sh);
    else
      mg_prolong_kernel<T, DIM, 1><<<gridb, 256, 0, st>>>(nx, m, nxc, mc, slices, zbuf(l), zbuf(l + 1), out, sh);
    tend(tb.timer);
  }
}

bool launch_mg_solve(const Geo& g, void* spec, bool fp32, const PrecondTables& tb, int spm, const double* lam,
                     hipStream_t st) {
  if (tb.mg_levels < 1) return false;
  if (fp32) {
    if (g.dim == 2) mg_cycle<float, 2>(g, reinterpret_cast<cx<float>*>(spec), tb, spm, lam, st);
    else mg_cycle<float, 3>(g, reinterpret_cast<cx<float>*>(spec), tb, spm, lam, st);
  } else {
    if (g.dim == 2) mg_cycle<double, 2>(g, reinterpret_cast<cx<double>*>(spec), tb, spm, lam, st);
    else mg_cycle<double, 3>(g, reinterpret_cast<cx<double>*>(spec), tb, spm, lam, st);
  }
  return true;
}

}  // namespace pcop
