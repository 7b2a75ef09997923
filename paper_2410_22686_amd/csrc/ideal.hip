// The ideal RBD preconditioner w = P^{-1} v of eq. matrix_P (Section 2):
// P^{-1} = G^{-1} blockdiag(T^T + alpha I, T + alpha I)^{-1}, so
//   (T + alpha I) z_2 = v_2  by forward substitution in time,
//   (T^T + alpha I) z_1 = v_1 by backward substitution,
//   w_1 = z_1 - z_2, w_2 = z_1 + z_2,
// each substitution step a solve with T_0 = (1 + alpha) I + tau K.  T_0 is
// real, so step s carries both recurrences in one complex slice per member:
//   c = (v_2^s + z_2^{s-1}) + i (v_1^{n-1-s} + z_1^{n-s}),  T_0 c' = c,
//   z_2^s = Re c', z_1^{n-1-s} = Im c'.
// With multigrid each step is one V-cycle, an approximate solve, so the n
// steps are n dependent launch sequences.  With sine transforms every T_0 is
// diagonal in the same modes: the slices of all steps are transformed at once,
// each mode runs its own scalar recurrence along time,
//   c'^s = (c^s + c'^{s-1}) / ((1 + alpha) + tau mu),
// and all slices are transformed back (2-D nx = 127, n = 127: 508 dependent
// launches of one slice each, 2200 us per apply, became eight over the whole
// vector).
// Storage inside the spectrum buffer: sequential, z[b][2][n][m] (type T)
// followed by the slice buffer c[b][m] (complex T); by modes, c[b][n][m]
// (complex T, the same size as z).
#include <algorithm>

#include "common.hpp"
#include "launch.hpp"

namespace pcop {

// step s in 0..n: store the solved slice of step s-1, pack the slice of step s
template <class T>
__global__ void __launch_bounds__(256) ideal_step_kernel(Geo g, int s, const double* __restrict__ v, T* __restrict__ z,
                                                         cx<T>* __restrict__ c, const double* __restrict__ vscale,
                                                         int vs_stride, const int* __restrict__ active) {
  const int b = blockIdx.y;
  if (active && !active[b]) return;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int n = g.n, m = g.m;
  if (i >= m) return;
  T* z1 = z + (size_t)b * 2 * n * m;
  T* z2 = z1 + (size_t)n * m;
  cx<T>* cb = c + (size_t)b * m;
  T p2 = 0, p1 = 0;  // z_2^{s-1}, z_1^{n-s}
  if (s > 0) {
    const cx<T> r = cb[i];
    p2 = r.x;
    p1 = r.y;
    z2[(size_t)(s - 1) * m + i] = p2;
    z1[(size_t)(n - s) * m + i] = p1;
  }
  if (s < n) {
    const double sc = vscale ? vscale[(size_t)b * vs_stride] : 1.0;
    const double* v1 = v + (size_t)b * g.vs;
    const double* v2 = v1 + (size_t)n * m;
    const double a2 = sc * v2[(size_t)s * m + i] + (double)p2;
    const double a1 = sc * v1[(size_t)(n - 1 - s) * m + i] + (double)p1;
    cb[i] = cx<T>{(T)a2, (T)a1};
  }
}

// w = [z_1 - z_2; z_1 + z_2] (added to w when accum)
template <class T>
__global__ void __launch_bounds__(256) ideal_combine_kernel(Geo g, const T* __restrict__ z, double* __restrict__ w,
                                                            int accum, const int* __restrict__ active) {
  const int b = blockIdx.y;
  if (active && !active[b]) return;
  const long long nm = (long long)g.n * g.m;
  const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= nm) return;
  const T* z1 = z + (size_t)b * 2 * nm;
  const double a = (double)z1[e], d = (double)z1[nm + e];
  double* w1 = w + (size_t)b * g.vs;
  double* w2 = w1 + nm;
  if (accum) {
    w1[e] += a - d;
    w2[e] += a + d;
  } else {
    w1[e] = a - d;
    w2[e] = a + d;
  }
}

// c^s = scale (v_2^s + i v_1^{n-1-s}) for every step s
template <class T>
__global__ void __launch_bounds__(256) ideal_pack_kernel(Geo g, const double* __restrict__ v, cx<T>* __restrict__ c,
                                                         const double* __restrict__ vscale, int vs_stride,
                                                         const int* __restrict__ active) {
  const int b = blockIdx.z;
  if (active && !active[b]) return;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= g.m) return;
  const int n = g.n, m = g.m;
  const double sc = vscale ? vscale[(size_t)b * vs_stride] : 1.0;
  const double* v1 = v + (size_t)b * g.vs;
  const double* v2 = v1 + (size_t)n * m;
  for (int s = blockIdx.y; s < n; s += gridDim.y)
    c[((size_t)b * n + s) * m + i] =
        cx<T>{(T)(sc * v2[(size_t)s * m + i]), (T)(sc * v1[(size_t)(n - 1 - s) * m + i])};
}

// The recurrences, in place (FP64 state).  A block owns kModes neighbouring
// modes (whole lines of the rows it touches) and splits their steps into CH
// chunks: each thread runs its chunk from zero to get the value it passes on,
// the carries are chained through LDS, and a second run from its carry writes
// the result.  CH = 1 where the modes alone fill the chip (one read less),
// else 16, so that a short mode list is not a serial walk through memory.
constexpr int kModes = 16;
constexpr int kModeAhead = 8;  // loads in flight per thread
template <class T, int CH>
__global__ void __launch_bounds__(256) ideal_modes_kernel(Geo g, cx<T>* __restrict__ c, const double* __restrict__ mu1,
                                                          const double* __restrict__ alpha, double cnorm,
                                                          const int* __restrict__ active) {
  constexpr int NM = 256 / CH;  // modes per block
  __shared__ cx<double> ends[CH][NM];
  const int b = blockIdx.y;
  if (active && !active[b]) return;
  const int i = blockIdx.x * NM + threadIdx.x % NM, q = threadIdx.x / NM;
  const int n = g.n, m = g.m, nx = g.nx;
  const bool in = i < m;
  const int im = in ? i : m - 1;
  double mu = mu1[im % nx] + mu1[(im / nx) % nx];
  if (g.dim == 3) mu += mu1[im / (nx * nx)];
  const double rd = 1.0 / ((1.0 + alpha[b]) + g.tau * mu);
  const int len = (n + CH - 1) / CH;
  const int s0 = min(n, q * len), s1 = min(n, s0 + len);
  cx<T>* cb = c + (size_t)b * n * m + im;
  auto walk = [&](cx<double> z, auto&& put) {
    for (int s = s0; s < s1; s += kModeAhead) {
      cx<T> y[kModeAhead];
#pragma unroll
      for (int u = 0; u < kModeAhead; ++u) y[u] = cb[(size_t)min(s + u, n - 1) * m];
#pragma unroll
      for (int u = 0; u < kModeAhead; ++u)
        if (s + u < s1) {
          z.x = (cnorm * (double)y[u].x + z.x) * rd;
          z.y = (cnorm * (double)y[u].y + z.y) * rd;
          put(s + u, z);
        }
    }
    return z;
  };
  cx<double> z{0.0, 0.0};
  if constexpr (CH > 1) {
    ends[q][threadIdx.x % NM] = walk(z, [](int, cx<double>) {});
    double decay = 1.0;  // rd^len, the weight of a carry one chunk on
    for (int u = 0; u < len; ++u) decay *= rd;
    __syncthreads();
    for (int p = 0; p < q; ++p) {
      const cx<double> e = ends[p][threadIdx.x % NM];
      z = cx<double>{e.x + decay * z.x, e.y + decay * z.y};
    }
  }
  // a lane past the last mode repeats it without storing
  walk(z, [&](int s, cx<double> v) {
    if (in) cb[(size_t)s * m] = cx<T>{(T)v.x, (T)v.y};
  });
}

// w_1^j = z_1^j - z_2^j, w_2^j = z_1^j + z_2^j with z_2^s = Re c^s,
// z_1^{n-1-s} = Im c^s (added to w when accum)
template <class T>
__global__ void __launch_bounds__(256) ideal_unpack_kernel(Geo g, const cx<T>* __restrict__ c, double* __restrict__ w,
                                                           int accum, const int* __restrict__ active) {
  const int b = blockIdx.z;
  if (active && !active[b]) return;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= g.m) return;
  const int n = g.n, m = g.m;
  const cx<T>* cb = c + (size_t)b * n * m + i;
  double* w1 = w + (size_t)b * g.vs + i;
  double* w2 = w1 + (size_t)n * m;
  for (int j = blockIdx.y; j < n; j += gridDim.y) {
    const double a = (double)cb[(size_t)(n - 1 - j) * m].y, d = (double)cb[(size_t)j * m].x;
    const size_t o = (size_t)j * m;
    if (accum) {
      w1[o] += a - d;
      w2[o] += a + d;
    } else {
      w1[o] = a - d;
      w2[o] = a + d;
    }
  }
}

template <class T>
static bool ideal_by_modes(const Geo& g, const double* v, double* w, void* spec, const PrecondTables& tb,
                           const double* vscale, int vs_stride, int accum, hipStream_t st) {
  cx<T>* c = reinterpret_cast<cx<T>*>(spec);
  const bool fp32 = sizeof(T) == 4;
  const double nm = (double)g.n * g.m * tb.nact;
  const dim3 gp((g.m + 255) / 256, std::min(g.n, 65535), g.B);
  tbeg(tb.timer, KF_IDEAL_STEP, (16.0 + sizeof(cx<T>)) * nm);
  ideal_pack_kernel<T><<<gp, 256, 0, st>>>(g, v, c, vscale, vs_stride, tb.active);
  tend(tb.timer);
  if (!launch_dst_transform(g, c, fp32, tb, (long long)g.B * g.n, st)) return false;
  tbeg(tb.timer, KF_IDEAL_STEP, 2.0 * sizeof(cx<T>) * nm);
  // 256 waves' worth of modes per member and more need no split in time
  if ((long long)g.m * g.B >= 65536)
    ideal_modes_kernel<T, 1><<<dim3((g.m + 255) / 256, g.B), 256, 0, st>>>(g, c, tb.mu1, tb.alpha, dst_norm(g), tb.active);
  else
    ideal_modes_kernel<T, 16><<<dim3((g.m + kModes - 1) / kModes, g.B), 256, 0, st>>>(g, c, tb.mu1, tb.alpha,
                                                                                     dst_norm(g), tb.active);
  tend(tb.timer);
  if (!launch_dst_transform(g, c, fp32, tb, (long long)g.B * g.n, st)) return false;
  tbeg(tb.timer, KF_COMBINE, (sizeof(cx<T>) + (accum ? 32.0 : 16.0)) * nm);
  ideal_unpack_kernel<T><<<gp, 256, 0, st>>>(g, c, w, accum, tb.active);
  tend(tb.timer);
  return true;
}

template <class T>
static bool ideal_by_steps(const Geo& g, const double* v, double* w, void* spec, const PrecondTables& tb,
                              const double* unit, const double* vscale, int vs_stride, int accum, hipStream_t st) {
  T* z = reinterpret_cast<T*>(spec);
  const size_t zbytes = sizeof(T) * (size_t)g.B * 2 * g.n * g.m;
  cx<T>* c = reinterpret_cast<cx<T>*>(reinterpret_cast<char*>(spec) + ((zbytes + 255) & ~(size_t)255));
  const bool fp32 = sizeof(T) == 4;
  dim3 gs((g.m + 255) / 256, g.B);
  const double step_bytes = (8.0 + 2.0 * sizeof(cx<T>)) * g.m * tb.nact;
  for (int s = 0; s <= g.n; ++s) {
    tbeg(tb.timer, KF_IDEAL_STEP, step_bytes);
    ideal_step_kernel<T><<<gs, 256, 0, st>>>(g, s, v, z, c, vscale, vs_stride, tb.active);
    tend(tb.timer);
    if (s == g.n) break;
    // one slice per member, shift lam_0 + alpha_b with lam_0 = 1: T_0 = (1 + alpha) I + tau K
    if (!launch_mg_solve(g, c, fp32, tb, 1, unit, st)) return false;
  }
  const long long nm = (long long)g.n * g.m;
  dim3 gc((unsigned)((nm + 255) / 256), g.B);
  tbeg(tb.timer, KF_COMBINE, (sizeof(T) * 2.0 + (accum ? 32.0 : 16.0)) * nm * tb.nact);
  ideal_combine_kernel<T><<<gc, 256, 0, st>>>(g, z, w, accum, tb.active);
  tend(tb.timer);
  return true;
}

size_t ideal_spec_bytes(const Geo& g, bool fp32) {
  const size_t t = fp32 ? 4 : 8;
  const size_t zbytes = t * (size_t)g.B * 2 * g.n * g.m;
  return ((zbytes + 255) & ~(size_t)255) + 2 * t * (size_t)g.B * g.m;
}

bool launch_ideal_precond(const Geo& g, const double* v, double* w, void* spec, bool fp32, int spatial,
                          const PrecondTables& tb, const double* unit, const double* vscale, int vs_stride,
                          int accum, hipStream_t st) {
  if (spatial == 0) {
    if (fp32) return ideal_by_modes<float>(g, v, w, spec, tb, vscale, vs_stride, accum, st);
    return ideal_by_modes<double>(g, v, w, spec, tb, vscale, vs_stride, accum, st);
  }
  if (fp32) return ideal_by_steps<float>(g, v, w, spec, tb, unit, vscale, vs_stride, accum, st);
  return ideal_by_steps<double>(g, v, w, spec, tb, unit, vscale, vs_stride, accum, st);
}

}  // namespace pcop
