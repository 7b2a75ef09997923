// The RBD preconditioners with sine transforms, by modes.  With a = 1 every
// spatial operator is diagonal in the sine modes, so both block systems of
// P_eps (eq. matrix_P_eps; P of eq. matrix_P is eps = 0) fall apart into one
// scalar system per mode and block,
//   d z^j - z^{j-1} = y^j (block 2; block 1 the same backward in time),
//   z^0 before the first level = eps z^n,   d = 1 + alpha + tau mu > 1
// (Q1 elements: mu = sum k/m, the right-hand side over the mass eigenvalue),
// a recurrence along time closed by
//   z^n = S / (1 - eps D),  S its value from a zero start, D = d^{-n}.
// No time transform, and so no scaling with eps^{j/n}: the same solution as the
// four steps of Section 2.1 (error against 64-bit references 1e-15 in both),
// for any number of levels at the same cost.
//
// Both blocks ride in one complex slice per step, c^s = v_2^s + i v_1^{n-1-s}
// (z_2^s = Re, z_1^{n-1-s} = Im), so that both recurrences run forward in s:
//   rows in    read v, transform along x1, write c          (mode_rows_in)
//   [x2 in 3-D]
//   last axis  transform, recurrence, transform back
//   [x2 in 3-D]
//   rows out   transform along x1, combine w_1 = z_1 - z_2,
//              w_2 = z_1 + z_2                               (mode_rows_out)
// Up to nx = 63 a whole (x1, x2) plane fits the LDS of half a CU, and x1 and x2
// are one pass on the way in and one on the way out (mode_plane_in, _out); in
// 2-D only the recurrences are left between them.
// The recurrence couples all steps of a mode, the transform all modes of a
// line.  Where the lines of one step fill the chip, blocks march along a chunk
// of steps with the state of their modes in registers: transform, accumulate
// and write (mode_march_in), chain the chunks (mode_chain), recurrence and
// transform back (mode_march_out); two passes of the vector in all.  Smaller
// shapes take whole passes for the transforms and one for the recurrences
// (mode_scan), which split in time inside a block.
#include <algorithm>

#include "common.hpp"
#include "dst_line.hpp"
#include "launch.hpp"

namespace pcop {

// what a mode's recurrence needs
struct ModeParams {
  const double* mu1;    // [nx] 1-D eigenvalues (k/m with Q1 elements)
  const double* im1;    // [nx] 1/m, or null
  const double* alpha;  // [B]
  const int* active;    // [B] or null
  double eps;           // 0: the ideal preconditioner
  double cnorm;         // dst_norm, applied by rows in
};

__device__ __forceinline__ double mode_mu(const Geo& g, const double* mu1, int i) {
  double mu = mu1[i % g.nx] + mu1[(i / g.nx) % g.nx];
  if (g.dim == 3) mu += mu1[i / (g.nx * g.nx)];
  return mu;
}

// 1/d for d = 1 + delta in two doubles.  With hi = fl(1/d) alone every step
// of a recurrence makes the same relative error, which n steps add up, and a
// small delta would be lost to the rounding of 1 + delta; hi + lo is 1/d to
// twice the precision and costs one multiplication per value.  FP32 slices
// are far coarser than that error and take hi alone.
template <class T>
struct ModeRecip {
  double hi, lo;
  __device__ __forceinline__ double operator()(double a) const { return sizeof(T) == 8 ? fma(a, hi, a * lo) : a * hi; }
};
template <class T>
__device__ __forceinline__ ModeRecip<T> mode_recip(double delta) {
  const double d = 1.0 + delta, t = d - 1.0;
  const double rest = (1.0 - (d - t)) + (delta - t);  // 1 + delta - d
  const double hi = 1.0 / d;
  return ModeRecip<T>{hi, fma(-hi, rest, fma(-hi, d, 1.0)) * hi};
}
// d^{-n}
__device__ __forceinline__ double mode_decay(double delta, int n) { return exp(-n * log1p(delta)); }
// eps / (1 - eps d^{-n}) without the cancellation where eps and d^{-n} are
// close to 1 (a short horizon): formed from rounded powers, eps = 1, n = 511,
// T = 1e-4 left 2e-12 of the result, against 6e-16 now (four steps: 3e-16)
__device__ __forceinline__ double mode_close(double delta, int n, double eps) {
  return eps / ((1.0 - eps) - eps * expm1(-n * log1p(delta)));
}

// ---------------------------------------------------------------------------
// contiguous lines, M/8 threads each (one wavefront or a part of it, so that
// no line waits on another): half-length transforms as in dst_half_kernel, the
// line staged in LDS on either side so that loads and stores are coalesced.
// Persistent blocks, the tables in LDS.  HBM-bound at the rate of a copy: 2-D
// nx = 511, n = 511 884 us (4.8 TB/s); the register-resident full-length lines of
// rows out took 1217 us here, nx = 127, n = 127, sixteen members 288 against 210.
// ---------------------------------------------------------------------------
constexpr int kRowThreads = 256;
template <class T, int L>
struct RowLines {
  using H = HalfDst<T, L>;
  static constexpr int M = H::M, N = H::N, TM = H::TM, NT = kRowThreads, LPB = NT / TM;
  static constexpr int LD = M >= 128 ? M + 4 : line_ld(M);
  static __device__ __forceinline__ void tables(const cx<T>* __restrict__ twL, cx<T>* twm, T* sinl) {
    for (int k = threadIdx.x; k < M; k += NT) {
      twm[k] = twL[2 * k];
      sinl[k] = -twL[k].y;
    }
    __syncthreads();
  }
  // the line's elements t + TM k in z[k] to those of its transform, through lbuf
  static __device__ __forceinline__ void transform(cx<T> (&z)[8], int t, cx<T>* lbuf, const cx<T>* twm, const T* sinl) {
    line_sync<TM>();
#pragma unroll
    for (int k = 0; k < 8; ++k) lbuf[pidx<T>(t + TM * k)] = z[k];
    line_sync<TM>();
    cx<T> v[8];
    H::pre(v, t, lbuf, sinl);
    RegStages<T, M, TM, -1, 1>::run(v, t, lbuf, twm);
    H::post(v, z, t, lbuf);
    line_sync<TM>();
#pragma unroll
    for (int r = 0; r < 8; ++r)
      if (8 * t + r >= 1) lbuf[pidx<T>(8 * t + r - 1)] = z[r];
    line_sync<TM>();
#pragma unroll
    for (int k = 0; k < 8; ++k) z[k] = lbuf[pidx<T>(t + TM * k)];
  }
};

template <class T, int L>
__global__ void __launch_bounds__(kRowThreads) mode_rows_in_kernel(Geo g, const double* __restrict__ v,
                                                                   cx<T>* __restrict__ c,
                                                                   const cx<T>* __restrict__ twL,
                                                                   const double* __restrict__ vscale, int vs_stride,
                                                                   ModeParams mp) {
  using R = RowLines<T, L>;
  constexpr int N = R::N, TM = R::TM, LPB = R::LPB;
  __shared__ cx<T> buf[LPB * R::LD];
  __shared__ cx<T> twm[R::M];
  __shared__ T sinl[R::M];
  R::tables(twL, twm, sinl);
  const int lid = threadIdx.x / TM, t = threadIdx.x - lid * TM;
  const int inner = g.m / N;  // lines per slice
  // 32 bits hold the number of lines (2^32 of 127 points would be 4 TB)
  const unsigned total = (unsigned)g.B * g.n * inner;
  for (unsigned ln = (unsigned)xcd_remap(blockIdx.x, gridDim.x) * LPB + lid; ln < total; ln += gridDim.x * LPB) {
    const unsigned sl = ln / inner;
    const int li = (int)(ln - sl * inner);
    const int b = (int)(sl / g.n), s = (int)(sl - (unsigned)b * g.n);
    if (mp.active && !mp.active[b]) continue;
    const double sc = mp.cnorm * (vscale ? vscale[(size_t)b * vs_stride] : 1.0);
    const double* v1 = v + (size_t)b * g.vs + (size_t)(g.n - 1 - s) * g.m + (size_t)li * N;
    const double* v2 = v + (size_t)b * g.vs + (size_t)(g.n + s) * g.m + (size_t)li * N;
    cx<T> z[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int e = min(t + TM * k, N - 1);
      z[k] = cx<T>{(T)(sc * v2[e]), (T)(sc * v1[e])};
    }
    R::transform(z, t, buf + lid * R::LD, twm, sinl);
    cx<T>* out = c + (size_t)sl * g.m + (size_t)li * N;
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (t + TM * k < N) out[t + TM * k] = z[k];
  }
}

// Rows out keeps lines of L/8 threads in registers (as dst_reg_kernel), one pass
// per block: with half-length lines and the pair's sum and difference formed
// before the transform, each line read half of two lines, and the pass took as
// long at nx = 511 (1036 against 1053 us), 127 (239, 239) and longer at 255.
// threads per block of rows out: the two lines of a pair at least
constexpr int rows_out_threads(int L) { return reg_threads(L) > 2 * (L / 8) ? reg_threads(L) : 2 * (L / 8); }

// A block's lines come in pairs, the same line of slices s and n - 1 - s: the
// pair exchanges its transforms through LDS and writes both levels of w.
template <class T, int L, bool ACCUM>
__global__ void __launch_bounds__(rows_out_threads(L)) mode_rows_out_kernel(Geo g, const cx<T>* __restrict__ c,
                                                                            double* __restrict__ w,
                                                                            const cx<T>* __restrict__ twL,
                                                                            ModeParams mp) {
  constexpr int N = L / 2 - 1, TL = L / 8, NT = rows_out_threads(L), LPB = NT / TL, LD = line_ld(L);
  __shared__ cx<T> buf[LPB * LD];
  const int lid = threadIdx.x / TL, t = threadIdx.x - lid * TL;
  const int inner = g.m / N, npair = (g.n + 1) / 2;
  const unsigned total = (unsigned)g.B * npair * inner;
  const unsigned pl = (unsigned)xcd_remap(blockIdx.x, gridDim.x) * (LPB / 2) + lid / 2;
  const unsigned pr = min(pl, total - 1) / inner;
  const int li = (int)(min(pl, total - 1) - pr * inner);
  const int b = (int)(pr / npair), p = (int)(pr - (unsigned)b * npair);
  const bool valid = pl < total && !(mp.active && !mp.active[b]);
  if (__syncthreads_or(valid) == 0) return;
  const int s = (lid & 1) ? g.n - 1 - p : p;
  const cx<T>* in = c + ((size_t)b * g.n + s) * g.m + (size_t)li * N;
  cx<T>* lbuf = buf + lid * LD;
  cx<T> z[8];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int pos = t + TL * k;
    z[k] = valid && pos != 0 ? in[pos - 1] : cx<T>{0, 0};
  }
  mirror<T, L, TL>(z, t, lbuf);
  RegStages<T, L, TL, -1, 1>::run(z, t, lbuf, twL);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 4; ++k) lbuf[pidx<T>(t + TL * k)] = z[k];
  __syncthreads();
  // the middle slice of an odd number is its own partner, written once
  if (!valid || ((lid & 1) && s == p)) return;
  const cx<T>* other = buf + (lid ^ 1) * LD;
  double* w1 = w + (size_t)b * g.vs + (size_t)s * g.m + (size_t)li * N;
  double* w2 = w1 + (size_t)g.n * g.m;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int pos = t + TL * k;
    if (pos >= 1) {
      const double z1 = (double)other[pidx<T>(pos)].y, z2 = (double)z[k].x;
      if (ACCUM) {
        w1[pos - 1] += z1 - z2;
        w2[pos - 1] += z1 + z2;
      } else {
        w1[pos - 1] = z1 - z2;
        w2[pos - 1] = z1 + z2;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Planes of nx <= 63: both axes of an (x1, x2) plane in one pass, the plane in
// LDS.  M groups of M/8 threads take a line each, so the block holds a whole
// axis of its planes in registers between the two (64 lines of 8 threads at
// nx = 63, 74 KB of LDS, two blocks per CU); the results of the rows are
// written back transposed and the columns are rows then.  A pass is loads,
// transforms and stores of one plane after another, two planes overlapping on a
// CU: about 200 us at 3-D nx = 63, n = 100 (4 TB/s), where the rows took 227 and
// 186 us and x2 151 more each way.  The whole preconditioner there 1119 -> 862
// us; 2-D nx = 63, n = 100, four members 75 -> 59 us (n = 400, sixteen: 1013 ->
// 726); nx = 31, n = 32 24.7 -> 18.9 us; 3-D nx = 15, n = 100, eight members
// 263 -> 119 us.  At nx = 127 a plane (258 KB) does not fit.
// ---------------------------------------------------------------------------
// threads of a block: one plane, or one wave
constexpr int plane_threads(int L) { return (L / 16) * (L / 2) < 64 ? 64 : (L / 16) * (L / 2); }

template <class T, int L>
struct PlaneTile {
  using H = HalfDst<T, L>;
  static constexpr int M = H::M, N = H::N, TM = H::TM, LD = line_ld(M);
  static constexpr int TP = TM * M;               // threads of a plane
  static constexpr int NT = plane_threads(L);
  static constexpr int PPB = NT / TP;
  static constexpr int QN = (N * N + TP - 1) / TP;  // elements per thread
  // slot of (row, col): the TM lanes of a line write rows 8 apart of one
  // column, which the row's XOR spreads over the banks
  static __device__ __forceinline__ int slot(int row, int col) { return row * LD + pidx<T>(col ^ ((row >> 3) & 7)); }
  static __device__ __forceinline__ void transform(cx<T>* plane, int tp, const cx<T>* twm, const T* sinl) {
    const int lid = tp / TM, t = tp - lid * TM;
    cx<T>* lbuf = plane + lid * LD;
#pragma unroll 1
    for (int ax = 0; ax < 2; ++ax) {
      cx<T> v[8], o[8];
      H::pre(v, t, lbuf, sinl, (lid >> 3) & 7);
      RegStages<T, M, TM, -1, 1>::run(v, t, lbuf, twm);
      H::post(v, o, t, lbuf);
      __syncthreads();
#pragma unroll
      for (int r = 0; r < 8; ++r)
        if (8 * t + r >= 1 && lid < N) plane[slot(8 * t + r - 1, lid)] = o[r];
      __syncthreads();
    }
  }
};

template <class T, int L>
__global__ void __launch_bounds__(plane_threads(L)) mode_plane_in_kernel(Geo g, const double* __restrict__ v,
                                                                            cx<T>* __restrict__ c,
                                                                            const cx<T>* __restrict__ twL,
                                                                            const double* __restrict__ vscale,
                                                                            int vs_stride, ModeParams mp) {
  using P = PlaneTile<T, L>;
  constexpr int M = P::M, N = P::N, TP = P::TP;
  __shared__ cx<T> buf[P::PPB * M * P::LD];
  __shared__ cx<T> twm[M];
  __shared__ T sinl[M];
  const int lp = threadIdx.x / TP, tp = threadIdx.x - lp * TP;
  cx<T>* plane = buf + lp * M * P::LD;
  const int nz = g.m / (N * N);  // planes per slice
  const unsigned total = (unsigned)g.B * g.n * nz;
  const unsigned pl = (unsigned)xcd_remap(blockIdx.x, gridDim.x) * P::PPB + lp;
  const unsigned sl = min(pl, total - 1) / nz;
  const int iz = (int)(min(pl, total - 1) - sl * nz);
  const int b = (int)(sl / g.n), s = (int)(sl - (unsigned)b * g.n);
  const bool valid = pl < total && !(mp.active && !mp.active[b]);
  if (__syncthreads_or(valid) == 0) return;
  const double sc = mp.cnorm * (vscale ? vscale[(size_t)b * vs_stride] : 1.0);
  const double* v1 = v + (size_t)b * g.vs + (size_t)(g.n - 1 - s) * g.m + (size_t)iz * N * N;
  const double* v2 = v + (size_t)b * g.vs + (size_t)(g.n + s) * g.m + (size_t)iz * N * N;
  double a1[P::QN], a2[P::QN];
#pragma unroll
  for (int q = 0; q < P::QN; ++q) {
    const int e = min(tp + TP * q, N * N - 1);
    a1[q] = v1[e];
    a2[q] = v2[e];
  }
  for (int k = threadIdx.x; k < M; k += P::NT) {
    twm[k] = twL[2 * k];
    sinl[k] = -twL[k].y;
  }
#pragma unroll
  for (int q = 0; q < P::QN; ++q) {
    const int e = min(tp + TP * q, N * N - 1);
    plane[P::slot(e / N, e % N)] = cx<T>{(T)(sc * a2[q]), (T)(sc * a1[q])};
  }
  __syncthreads();
  P::transform(plane, tp, twm, sinl);
  if (!valid) return;
  cx<T>* out = c + (size_t)sl * g.m + (size_t)iz * N * N;
#pragma unroll
  for (int q = 0; q < P::QN; ++q) {
    const int e = tp + TP * q;
    if (e < N * N) out[e] = plane[P::slot(e / N, e % N)];
  }
}

// w_1^s + i w_2^s is the transform of (z_1^s - z_2^s) + i (z_1^s + z_2^s), with
// z_2^s the real part of slice s and z_1^s the imaginary part of slice
// n - 1 - s; the planes of such a pair of slices are neighbours in the grid,
// so that each finds the other's half of a line of memory in the L2.
template <class T, int L, bool ACCUM>
__global__ void __launch_bounds__(plane_threads(L)) mode_plane_out_kernel(Geo g, const cx<T>* __restrict__ c,
                                                                             double* __restrict__ w,
                                                                             const cx<T>* __restrict__ twL,
                                                                             ModeParams mp) {
  using P = PlaneTile<T, L>;
  constexpr int M = P::M, N = P::N, TP = P::TP;
  __shared__ cx<T> buf[P::PPB * M * P::LD];
  __shared__ cx<T> twm[M];
  __shared__ T sinl[M];
  const int lp = threadIdx.x / TP, tp = threadIdx.x - lp * TP;
  cx<T>* plane = buf + lp * M * P::LD;
  const int nz = g.m / (N * N), npair = (g.n + 1) / 2;
  const unsigned total = 2u * g.B * npair * nz;
  const unsigned pl = (unsigned)xcd_remap(blockIdx.x, gridDim.x) * P::PPB + lp;
  const unsigned pz = min(pl, total - 1) / 2;  // (member, pair, plane)
  const unsigned pr = pz / nz;
  const int iz = (int)(pz - pr * nz);
  const int b = (int)(pr / npair), p = (int)(pr - (unsigned)b * npair);
  const int s = (pl & 1) ? g.n - 1 - p : p;
  // the middle slice of an odd number is its own partner, written once
  const bool valid = pl < total && !(mp.active && !mp.active[b]) && !((pl & 1) && s == p);
  if (__syncthreads_or(valid) == 0) return;
  const T* c2 = reinterpret_cast<const T*>(c + ((size_t)b * g.n + s) * g.m + (size_t)iz * N * N);
  const T* c1 = reinterpret_cast<const T*>(c + ((size_t)b * g.n + (g.n - 1 - s)) * g.m + (size_t)iz * N * N) + 1;
  T a1[P::QN], a2[P::QN];
#pragma unroll
  for (int q = 0; q < P::QN; ++q) {
    const int e = min(tp + TP * q, N * N - 1);
    a1[q] = c1[2 * e];
    a2[q] = c2[2 * e];
  }
  for (int k = threadIdx.x; k < M; k += P::NT) {
    twm[k] = twL[2 * k];
    sinl[k] = -twL[k].y;
  }
#pragma unroll
  for (int q = 0; q < P::QN; ++q) {
    const int e = min(tp + TP * q, N * N - 1);
    plane[P::slot(e / N, e % N)] = cx<T>{a1[q] - a2[q], a1[q] + a2[q]};
  }
  __syncthreads();
  P::transform(plane, tp, twm, sinl);
  if (!valid) return;
  double* w1 = w + (size_t)b * g.vs + (size_t)s * g.m + (size_t)iz * N * N;
  double* w2 = w1 + (size_t)g.n * g.m;
#pragma unroll
  for (int q = 0; q < P::QN; ++q) {
    const int e = tp + TP * q;
    if (e < N * N) {
      const cx<T> z = plane[P::slot(e / N, e % N)];
      if (ACCUM) {
        w1[e] += (double)z.x;
        w2[e] += (double)z.y;
      } else {
        w1[e] = (double)z.x;
        w2[e] = (double)z.y;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// The recurrences of all modes, in place (FP64 state).  A block owns 256 / CH
// neighbouring modes and splits their steps into CH chunks: each thread runs
// its chunk from zero to get the value it passes on, the values are chained
// through LDS and closed with eps, and a second run from its carry writes the
// result.  The second read comes from the caches where the slices fit the last
// level (256 MB), as those of most shapes that take this kernel do; beyond (2-D
// nx = 63, n = 299, 17 members: 323 MB; nx = 255, n = 511, one member: 531 MB)
// it is a third pass over memory.  CH = 1 where the modes alone fill the chip,
// else 16, so that a short mode list is not a serial walk through memory.
// ---------------------------------------------------------------------------
constexpr int kScanAhead = 8;  // loads in flight per thread
template <class T, int CH>
__global__ void __launch_bounds__(256) mode_scan_kernel(Geo g, cx<T>* __restrict__ c, ModeParams mp) {
  constexpr int NM = 256 / CH;  // modes per block
  __shared__ cx<double> ends[CH][NM];
  const int b = blockIdx.y;
  if (mp.active && !mp.active[b]) return;
  const int k = threadIdx.x % NM, q = threadIdx.x / NM;
  const int i = blockIdx.x * NM + k;
  const int n = g.n, m = g.m, nx = g.nx;
  const bool in = i < m;
  const int im = in ? i : m - 1;
  const double delta = mp.alpha[b] + g.tau * mode_mu(g, mp.mu1, im);
  const ModeRecip<T> rd = mode_recip<T>(delta);
  double f = 1.0;
  if (mp.im1) {
    f = mp.im1[im % nx] * mp.im1[(im / nx) % nx];
    if (g.dim == 3) f *= mp.im1[im / (nx * nx)];
  }
  const int len = (n + CH - 1) / CH;
  const int s0 = min(n, q * len), s1 = min(n, s0 + len);
  cx<T>* cb = c + (size_t)b * n * m + im;
  auto walk = [&](cx<double> z, auto&& put) {
    for (int s = s0; s < s1; s += kScanAhead) {
      cx<T> y[kScanAhead];
#pragma unroll
      for (int u = 0; u < kScanAhead; ++u) y[u] = cb[(size_t)min(s + u, n - 1) * m];
#pragma unroll
      for (int u = 0; u < kScanAhead; ++u)
        if (s + u < s1) {
          z.x = rd(f * (double)y[u].x + z.x);
          z.y = rd(f * (double)y[u].y + z.y);
          put(s + u, z);
        }
    }
    return z;
  };
  cx<double> z{0.0, 0.0};
  if (CH > 1 || mp.eps != 0.0) {
    ends[q][k] = walk(z, [](int, cx<double>) {});
    __syncthreads();
    // chunk p passes on ends + d^{-its length} times what it got: whole chunks,
    // then one of the rest, then empty ones that pass on what they get
    const int whole = n / len, rest = n - whole * len;
    const double decay = mode_decay(delta, len), drest = rest > 0 ? mode_decay(delta, rest) : 1.0;
    auto chain = [&](cx<double> a, int upto) {
      for (int p = 0; p < min(upto, whole + (rest > 0)); ++p) {
        const double dp = p < whole ? decay : drest;
        a = cx<double>{ends[p][k].x + dp * a.x, ends[p][k].y + dp * a.y};
      }
      return a;
    };
    if (mp.eps != 0.0) {
      const cx<double> S = chain(z, CH);
      const double close = mode_close(delta, n, mp.eps);
      z = cx<double>{close * S.x, close * S.y};
    }
    z = chain(z, q);
  }
  // a lane past the last mode repeats it without storing
  walk(z, [&](int s, cx<double> a) {
    if (in) cb[(size_t)s * m] = cx<T>{(T)a.x, (T)a.y};
  });
}

// ---------------------------------------------------------------------------
// Marching passes of the last axis.  HBM-bound with two blocks per CU (210 to
// 252 registers): 0.98 ms each at 2-D nx = 511, n = 511 (4.4 TB/s), where the
// strided pass with the division and the two time transforms they replace took
// 2.0 + 1.2 + 1.2 ms.  A tile is LPB neighbouring lines (M/8
// threads each, half-length transforms as dst_half_kernel); a block takes one
// tile through the steps [q len, (q + 1) len) of its member.  Thread t of a
// line keeps the state of modes 8t .. 8t + 7.
// ---------------------------------------------------------------------------
template <class T, int L, int NT>
struct MarchTile {
  using H = HalfDst<T, L>;
  static constexpr int M = H::M, N = H::N, TM = H::TM, LPB = NT / TM;
  static constexpr bool QUAD = TM >= 4;
  static constexpr int LD = M >= 128 ? M + 4 : line_ld(M);
  static constexpr int QS = (N * LPB + NT - 1) / NT;
  static_assert(LPB * TM == NT, "a tile is a whole number of lines");
  // the tile's (line, element) pairs a thread loads and stores: line tl,
  // elements te + TM q (see dst_half_kernel)
  static __device__ __forceinline__ int tl() { return QUAD ? (threadIdx.x >> 2) % LPB : threadIdx.x % LPB; }
  static __device__ __forceinline__ int te() {
    return QUAD ? (threadIdx.x & 3) + 4 * (threadIdx.x / (4 * LPB)) : threadIdx.x / LPB;
  }
  static __device__ __forceinline__ void load(const cx<T>* __restrict__ src, int l0, int lines, int stride, cx<T>* buf) {
    const bool ok = l0 + tl() < lines;
    const int off = l0 + tl() + te() * stride;
    cx<T> cur[QS];
#pragma unroll
    for (int q = 0; q < QS; ++q) cur[q] = ok && te() + TM * q < N ? src[off + q * TM * stride] : cx<T>{0, 0};
#pragma unroll
    for (int q = 0; q < QS; ++q)
      if (te() + TM * q < N) buf[tl() * LD + pidx<T>(te() + TM * q)] = cur[q];
  }
  static __device__ __forceinline__ void store(cx<T>* __restrict__ dst, int l0, int lines, int stride, const cx<T>* buf) {
    if (l0 + tl() < lines) {
      const int off = l0 + tl() + te() * stride;
#pragma unroll
      for (int q = 0; q < QS; ++q)
        if (te() + TM * q < N) dst[off + q * TM * stride] = buf[tl() * LD + pidx<T>(te() + TM * q)];
    }
  }
};

// (tile, chunk, member) of this block, neighbouring tiles (which share lines
// of memory) on one XCD at the same time
struct MarchBlock {
  int tile, q, b;
};
__device__ __forceinline__ MarchBlock march_block(int tiles, int CH) {
  const int lg = xcd_remap(blockIdx.x, gridDim.x);
  return MarchBlock{lg % tiles, lg / tiles % CH, lg / (tiles * CH)};
}

// reciprocal diagonals of modes 8t .. 8t + 7 of the thread's line, and (Q1)
// the factor of their right-hand sides
template <class T, int N, bool FEM>
__device__ __forceinline__ void mode_factors(const Geo& g, const ModeParams& mp, int b, int line, int t,
                                             ModeRecip<T> (&rd)[8], double (&f)[8]) {
  double ml = mp.mu1[line % g.nx], psl = FEM ? mp.im1[line % g.nx] : 1.0;
  if (g.dim == 3) {
    ml += mp.mu1[(line / g.nx) % g.nx];
    if (FEM) psl *= mp.im1[(line / g.nx) % g.nx];
  }
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const int e = max(8 * t + r - 1, 0);
    rd[r] = mode_recip<T>(mp.alpha[b] + g.tau * (ml + mp.mu1[min(e, N - 1)]));
    f[r] = FEM ? psl * mp.im1[min(e, N - 1)] : 1.0;
  }
}

template <class T, int L, int NT, bool FEM>
__global__ void __launch_bounds__(NT) mode_march_in_kernel(Geo g, cx<T>* __restrict__ c, cx<T>* __restrict__ ends,
                                                           const cx<T>* __restrict__ twL, int tiles, int CH, int len,
                                                           ModeParams mp) {
  using M_ = MarchTile<T, L, NT>;
  using H = HalfDst<T, L>;
  constexpr int M = M_::M, N = M_::N, TM = M_::TM, LPB = M_::LPB, LD = M_::LD;
  __shared__ cx<T> buf[LPB * LD];
  __shared__ cx<T> twm[M];
  __shared__ T sinl[M];
  const MarchBlock mb = march_block(tiles, CH);
  if (mp.active && !mp.active[mb.b]) return;
  for (int k = threadIdx.x; k < M; k += NT) {
    twm[k] = twL[2 * k];
    sinl[k] = -twL[k].y;
  }
  const int lines = g.m / N;  // per step; also the stride of a line's elements
  const int l0 = mb.tile * LPB, lid = threadIdx.x / TM, t = threadIdx.x - lid * TM;
  const int s0 = mb.q * len, s1 = min(g.n, s0 + len);
  cx<T>* lbuf = buf + lid * LD;
  ModeRecip<T> rd[8];
  double f[8];
  mode_factors<T, N, FEM>(g, mp, mb.b, min(l0 + lid, lines - 1), t, rd, f);
  cx<double> z[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) z[r] = cx<double>{0.0, 0.0};
  auto put = [&](const cx<T> (&o)[8]) {
    line_sync<TM>();
#pragma unroll
    for (int r = 0; r < 8; ++r)
      if (8 * t + r >= 1) lbuf[pidx<T>(8 * t + r - 1)] = o[r];
    __syncthreads();
  };
  __syncthreads();
  for (int s = s0; s < s1; ++s) {
    cx<T>* cs = c + ((size_t)mb.b * g.n + s) * g.m;
    M_::load(cs, l0, lines, lines, buf);
    __syncthreads();
    cx<T> v[8], o[8];
    H::pre(v, t, lbuf, sinl);
    RegStages<T, M, TM, -1, 1>::run(v, t, lbuf, twm);
    H::post(v, o, t, lbuf);
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      if (FEM) o[r] = cx<T>{(T)(f[r] * (double)o[r].x), (T)(f[r] * (double)o[r].y)};
      z[r] = cx<double>{rd[r]((double)o[r].x + z[r].x), rd[r]((double)o[r].y + z[r].y)};
    }
    put(o);
    M_::store(cs, l0, lines, lines, buf);
    __syncthreads();
  }
  cx<T> e[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) e[r] = cx<T>{(T)z[r].x, (T)z[r].y};
  put(e);
  M_::store(ends + ((size_t)mb.b * CH + mb.q) * g.m, l0, lines, lines, buf);
}

// The values the chunks start from, over their end values from a zero start
// (one thread per mode).
template <class T>
__global__ void __launch_bounds__(256) mode_chain_kernel(Geo g, cx<T>* __restrict__ ends, int CH, int len, ModeParams mp) {
  const int b = blockIdx.y, i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= g.m || (mp.active && !mp.active[b])) return;
  const double delta = mp.alpha[b] + g.tau * mode_mu(g, mp.mu1, i);
  const double decay = mode_decay(delta, len), last = mode_decay(delta, g.n - (CH - 1) * len);
  cx<T>* e = ends + (size_t)b * CH * g.m + i;
  cx<double> z{0.0, 0.0};
  if (mp.eps != 0.0) {
    for (int q = 0; q < CH; ++q) {
      const double d = q + 1 < CH ? decay : last;
      const cx<T> a = e[(size_t)q * g.m];
      z = cx<double>{(double)a.x + d * z.x, (double)a.y + d * z.y};
    }
    const double close = mode_close(delta, g.n, mp.eps);
    z = cx<double>{close * z.x, close * z.y};
  }
  for (int q = 0; q < CH; ++q) {
    const cx<T> a = e[(size_t)q * g.m];
    e[(size_t)q * g.m] = cx<T>{(T)z.x, (T)z.y};
    z = cx<double>{(double)a.x + decay * z.x, (double)a.y + decay * z.y};
  }
}

template <class T, int L, int NT>
__global__ void __launch_bounds__(NT) mode_march_out_kernel(Geo g, cx<T>* __restrict__ c,
                                                            const cx<T>* __restrict__ starts,
                                                            const cx<T>* __restrict__ twL, int tiles, int CH, int len,
                                                            ModeParams mp) {
  using M_ = MarchTile<T, L, NT>;
  using H = HalfDst<T, L>;
  constexpr int M = M_::M, N = M_::N, TM = M_::TM, LPB = M_::LPB, LD = M_::LD;
  __shared__ cx<T> buf[LPB * LD];
  __shared__ cx<T> twm[M];
  __shared__ T sinl[M];
  const MarchBlock mb = march_block(tiles, CH);
  if (mp.active && !mp.active[mb.b]) return;
  for (int k = threadIdx.x; k < M; k += NT) {
    twm[k] = twL[2 * k];
    sinl[k] = -twL[k].y;
  }
  const int lines = g.m / N;
  const int l0 = mb.tile * LPB, lid = threadIdx.x / TM, t = threadIdx.x - lid * TM;
  const int s0 = mb.q * len, s1 = min(g.n, s0 + len);
  cx<T>* lbuf = buf + lid * LD;
  ModeRecip<T> rd[8];
  double f[8];
  mode_factors<T, N, false>(g, mp, mb.b, min(l0 + lid, lines - 1), t, rd, f);
  M_::load(starts + ((size_t)mb.b * CH + mb.q) * g.m, l0, lines, lines, buf);
  __syncthreads();
  cx<double> z[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const cx<T> a = lbuf[pidx<T>(max(8 * t + r - 1, 0))];
    z[r] = cx<double>{(double)a.x, (double)a.y};
  }
  __syncthreads();
  for (int s = s0; s < s1; ++s) {
    cx<T>* cs = c + ((size_t)mb.b * g.n + s) * g.m;
    M_::load(cs, l0, lines, lines, buf);
    __syncthreads();
    // the recurrence, each value back to its slot
#pragma unroll
    for (int r = 0; r < 8; ++r)
      if (8 * t + r >= 1) {
        cx<T>& y = lbuf[pidx<T>(8 * t + r - 1)];
        z[r] = cx<double>{rd[r]((double)y.x + z[r].x), rd[r]((double)y.y + z[r].y)};
        y = cx<T>{(T)z[r].x, (T)z[r].y};
      }
    line_sync<TM>();
    cx<T> v[8], o[8];
    H::pre(v, t, lbuf, sinl);
    RegStages<T, M, TM, -1, 1>::run(v, t, lbuf, twm);
    H::post(v, o, t, lbuf);
    line_sync<TM>();
#pragma unroll
    for (int r = 0; r < 8; ++r)
      if (8 * t + r >= 1) lbuf[pidx<T>(8 * t + r - 1)] = o[r];
    __syncthreads();
    M_::store(cs, l0, lines, lines, buf);
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Chunks of the marching passes, 0 where whole passes are taken: enough blocks
// for two rounds of the chip (1024), chunks of at least 8 steps (a chunk's end
// and start values are two more slices each), at most 16 of them (2-D nx = 255
// takes them from two members on, nx = 127 from eight).
static int march_chunks(const Geo& g) {
  if (g.dim == 2 && g.nx <= 63) return 0;  // no axis left beyond the planes
  const int M = g.nx + 1, lpb = 256 / (M / 8);
  const long long tiles = ((long long)g.m / g.nx + lpb - 1) / lpb * g.B;
  const long long ch = std::max<long long>(1, (1024 + tiles - 1) / tiles);
  return ch * 8 <= g.n && ch <= kModeChunks ? (int)ch : 0;
}

bool modes_exist(const Geo& g) { return g.nx >= 7; }

size_t mode_ends_bytes(const Geo& g, bool fp32) {
  return (fp32 ? 8 : 16) * (size_t)g.B * march_chunks(g) * (size_t)g.m;
}

template <class T, int L>
static bool modes_L(const Geo& g, const double* v, double* w, cx<T>* c, cx<T>* ends, const PrecondTables& tb,
                    double eps, const double* vscale, int vs_stride, int accum, hipStream_t st) {
  const cx<T>* twL = reinterpret_cast<const cx<T>*>(sizeof(T) == 8 ? (const void*)tb.twL64 : (const void*)tb.twL32);
  const ModeParams mp{tb.mu1, tb.im1, tb.alpha, tb.active, eps, dst_norm(g)};
  const bool fp32 = sizeof(T) == 4;
  const long long nslices = (long long)g.B * g.n;
  const int inner = g.m / g.nx;
  const double nm = (double)g.n * g.m * tb.nact;
  const double pass = 2.0 * sizeof(cx<T>) * nm;
  constexpr bool PLANES = L <= 128;
  tbeg(tb.timer, KF_DST_ROWS, (16.0 + sizeof(cx<T>)) * nm);
  if constexpr (PLANES) {
    using P = PlaneTile<T, L>;
    const long long planes = nslices * (g.m / (P::N * P::N));
    mode_plane_in_kernel<T, L><<<(unsigned)((planes + P::PPB - 1) / P::PPB), P::NT, 0, st>>>(g, v, c, twL, vscale,
                                                                                             vs_stride, mp);
  } else {
    constexpr int LPB = RowLines<T, L>::LPB;
    const long long lines = nslices * inner;
    static const int res = resident_blocks(mode_rows_in_kernel<T, L>, kRowThreads, 0);
    const unsigned grid = (unsigned)std::min<long long>((lines + LPB - 1) / LPB, (long long)res * std::max(1, tb.ncu));
    mode_rows_in_kernel<T, L><<<grid, kRowThreads, 0, st>>>(g, v, c, twL, vscale, vs_stride, mp);
  }
  tend(tb.timer);
  if (!PLANES && g.dim == 3 && !launch_dst_axis(g, c, fp32, tb, nslices, 2, st)) return false;
  const int CH = march_chunks(g);
  if (CH > 0) {
    constexpr int NT = 256, LPB = MarchTile<T, L, NT>::LPB;
    const int tiles = (inner + LPB - 1) / LPB;
    const int len = (g.n + CH - 1) / CH, chunks = (g.n + len - 1) / len;
    const dim3 grid((unsigned)((long long)tiles * chunks * g.B));
    tbeg(tb.timer, KF_DST_LAST, pass);
    if (mp.im1)
      mode_march_in_kernel<T, L, NT, true><<<grid, NT, 0, st>>>(g, c, ends, twL, tiles, chunks, len, mp);
    else
      mode_march_in_kernel<T, L, NT, false><<<grid, NT, 0, st>>>(g, c, ends, twL, tiles, chunks, len, mp);
    tend(tb.timer);
    tbeg(tb.timer, KF_MODES, 0.0);
    mode_chain_kernel<T><<<dim3((g.m + 255) / 256, g.B), 256, 0, st>>>(g, ends, chunks, len, mp);
    tend(tb.timer);
    tbeg(tb.timer, KF_DST_LAST, pass);
    mode_march_out_kernel<T, L, NT><<<grid, NT, 0, st>>>(g, c, ends, twL, tiles, chunks, len, mp);
    tend(tb.timer);
  } else {
    const bool axis = !PLANES || g.dim == 3;  // a last axis beyond the planes
    if (axis && !launch_dst_axis(g, c, fp32, tb, nslices, g.dim == 3 ? 3 : 2, st)) return false;
    tbeg(tb.timer, KF_MODES, pass);
    // 128 waves of modes per XCD and more need no split in time
    if ((long long)g.m * g.B >= 65536)
      mode_scan_kernel<T, 1><<<dim3((g.m + 255) / 256, g.B), 256, 0, st>>>(g, c, mp);
    else
      mode_scan_kernel<T, 16><<<dim3((g.m + 15) / 16, g.B), 256, 0, st>>>(g, c, mp);
    tend(tb.timer);
    if (axis && !launch_dst_axis(g, c, fp32, tb, nslices, g.dim == 3 ? 3 : 2, st)) return false;
  }
  if (!PLANES && g.dim == 3 && !launch_dst_axis(g, c, fp32, tb, nslices, 2, st)) return false;
  tbeg(tb.timer, KF_DST_ROWS, (sizeof(cx<T>) + (accum ? 32.0 : 16.0)) * nm);
  if constexpr (PLANES) {
    using P = PlaneTile<T, L>;
    const long long planes = 2LL * g.B * ((g.n + 1) / 2) * (g.m / (P::N * P::N));
    const unsigned grid = (unsigned)((planes + P::PPB - 1) / P::PPB);
    if (accum) mode_plane_out_kernel<T, L, true><<<grid, P::NT, 0, st>>>(g, c, w, twL, mp);
    else mode_plane_out_kernel<T, L, false><<<grid, P::NT, 0, st>>>(g, c, w, twL, mp);
  } else {
    constexpr int NT = rows_out_threads(L), PL = NT / (L / 8) / 2;
    const long long pairs = (long long)g.B * ((g.n + 1) / 2) * inner;
    const unsigned grid = (unsigned)((pairs + PL - 1) / PL);
    if (accum) mode_rows_out_kernel<T, L, true><<<grid, NT, 0, st>>>(g, c, w, twL, mp);
    else mode_rows_out_kernel<T, L, false><<<grid, NT, 0, st>>>(g, c, w, twL, mp);
  }
  tend(tb.timer);
  return true;
}

template <class T>
static bool modes_T(const Geo& g, const double* v, double* w, void* c, void* ends, const PrecondTables& tb, double eps,
                    const double* vscale, int vs_stride, int accum, hipStream_t st) {
#define PCOP_MODES(LL)                                                                                              \
  case LL:                                                                                                          \
    return modes_L<T, LL>(g, v, w, reinterpret_cast<cx<T>*>(c), reinterpret_cast<cx<T>*>(ends), tb, eps, vscale,      \
                          vs_stride, accum, st)
  switch (2 * (g.nx + 1)) {
    PCOP_MODES(16);
    PCOP_MODES(32);
    PCOP_MODES(64);
    PCOP_MODES(128);
    PCOP_MODES(256);
    PCOP_MODES(512);
    PCOP_MODES(1024);
    default: return false;
  }
#undef PCOP_MODES
}

bool launch_modes_precond(const Geo& g, const double* v, double* w, void* c, void* ends, bool fp32,
                          const PrecondTables& tb, double eps, const double* vscale, int vs_stride, int accum,
                          hipStream_t st) {
  if (fp32) return modes_T<float>(g, v, w, c, ends, tb, eps, vscale, vs_stride, accum, st);
  return modes_T<double>(g, v, w, c, ends, tb, eps, vscale, vs_stride, accum, st);
}

}  // namespace pcop
