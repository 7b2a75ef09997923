// Arnoldi kernels for GMRES in FP64: fused multi-dot, fused multi-AXPY that
// also measures the updated vector, linear combinations of basis vectors, and
// the per-member Gram-Schmidt bookkeeping.  Reductions are two-level
// (wavefront butterfly + fixed-order block/partial sums), so results are
// bitwise reproducible for a fixed launch shape.
//
// Basis vectors are stored unnormalised: the Arnoldi vector v_i equals
// sc[b][i] * basis_i, which lets the normalisation ride along in the
// coefficients instead of costing a pass over the vector.
#include <algorithm>
#include <array>
#include <utility>

#include "common.hpp"
#include "launch.hpp"

namespace pcop {

constexpr int kNT = 256;
constexpr int kNWave = kNT / kWave;

int krylov_blocks(long long vl) {
  long long want = (vl / 2 + kNT * 4 - 1) / (kNT * 4);
  if (want < 1) want = 1;
  if (want > 1024) want = 1024;
  return (int)want;
}

// Basis vectors are streamed once per pass: their loads are nontemporal, so
// they do not displace the vector being updated (or other live data) from
// the caches.
__device__ __forceinline__ double ld_stream(const double* p) { return __builtin_nontemporal_load(p); }
__device__ __forceinline__ double2 ld_stream(const double2* p) {
  return double2{__builtin_nontemporal_load(&p->x), __builtin_nontemporal_load(&p->y)};
}

// block-level reduction of NACC accumulators; thread c < ncols writes column c
template <int NACC>
__device__ __forceinline__ void block_reduce_store(double (&acc)[NACC], int ncols, double* out) {
  __shared__ double red[kNWave][NACC];
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = threadIdx.x / kWave;
#pragma unroll
  for (int c = 0; c < NACC; ++c) {
    if (c < ncols) {
      double s = wave_sum(acc[c]);
      if (lane == 0) red[wv][c] = s;
    }
  }
  __syncthreads();
  for (int c = threadIdx.x; c < ncols; c += kNT) {
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < kNWave; ++k) s += red[k][c];
    out[c] = s;
  }
}

// Vectors are read as double2 (the length 2 n m of a member vector is even
// and every base address is 16-byte aligned).  NV (the number of basis
// vectors) is a compile-time constant: every load is issued without a guard.
template <int NV>
__global__ void __launch_bounds__(kNT) mdot_kernel(KrylovArgs ka, const double* __restrict__ w,
                                                   double* __restrict__ partial, int nblk) {
  const int b = blockIdx.y;
  if (ka.active && !ka.active[b]) return;
  double acc[NV + 1];
#pragma unroll
  for (int i = 0; i <= NV; ++i) acc[i] = 0.0;
  const double2* wb = reinterpret_cast<const double2*>(w + (size_t)b * ka.ms);
  const double2* vb = reinterpret_cast<const double2*>(ka.basis + (size_t)b * ka.ms);
  const long long n2 = ka.vl / 2;
  const long long ss = ka.slot_stride / 2;
  for (long long e = (long long)blockIdx.x * kNT + threadIdx.x; e < n2; e += (long long)nblk * kNT) {
    const double2 wv = wb[e];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const double2 v = ld_stream(&vb[(size_t)i * ss + e]);
      acc[i] += v.x * wv.x + v.y * wv.y;
    }
    acc[NV] += wv.x * wv.x + wv.y * wv.y;
  }
  // columns 0..NV-1: dots, column NV: the squared norm
  block_reduce_store<NV + 1>(acc, NV + 1, partial + ((size_t)b * nblk + blockIdx.x) * kRedStride);
}

// the update keeps the basis values of its element in registers for the
// second product, so it works on one double per thread and iteration
template <int NV>
__global__ void __launch_bounds__(kNT) update_kernel(KrylovArgs ka, double* __restrict__ w,
                                                     const double* __restrict__ coef, int coef_ld,
                                                     double* __restrict__ partial, int nblk,
                                                     const int* __restrict__ skip) {
  const int b = blockIdx.y;
  if (ka.active && !ka.active[b]) return;
  if (skip && skip[b]) return;
  __shared__ double c[NV > 0 ? NV : 1];
  for (int i = threadIdx.x; i < NV; i += kNT) c[i] = coef[(size_t)b * coef_ld + i];
  __syncthreads();
  double acc[NV + 1];
#pragma unroll
  for (int i = 0; i <= NV; ++i) acc[i] = 0.0;
  double* wb = w + (size_t)b * ka.ms;
  const double* vb = ka.basis + (size_t)b * ka.ms;
  for (long long e = (long long)blockIdx.x * kNT + threadIdx.x; e < ka.vl; e += (long long)nblk * kNT) {
    double v[NV > 0 ? NV : 1];
#pragma unroll
    for (int i = 0; i < NV; ++i) v[i] = ld_stream(&vb[(size_t)i * ka.slot_stride + e]);
    double wv = wb[e];
#pragma unroll
    for (int i = 0; i < NV; ++i) wv -= c[i] * v[i];
    wb[e] = wv;
#pragma unroll
    for (int i = 0; i < NV; ++i) acc[i] += v[i] * wv;
    acc[NV] += wv * wv;
  }
  block_reduce_store<NV + 1>(acc, NV + 1, partial + ((size_t)b * nblk + blockIdx.x) * kRedStride);
}

// the same update on double2 pairs (two elements per thread and step)
template <int MAXNV>
__global__ void __launch_bounds__(kNT) update2_kernel(KrylovArgs ka, int nv, double* __restrict__ w,
                                                      const double* __restrict__ coef, int coef_ld,
                                                      double* __restrict__ partial, int nblk,
                                                      const int* __restrict__ skip) {
  const int b = blockIdx.y;
  if (ka.active && !ka.active[b]) return;
  if (skip && skip[b]) return;
  __shared__ double c[MAXNV];
  for (int i = threadIdx.x; i < MAXNV; i += kNT) c[i] = (i < nv) ? coef[(size_t)b * coef_ld + i] : 0.0;
  __syncthreads();
  double acc[MAXNV + 1];
#pragma unroll
  for (int i = 0; i <= MAXNV; ++i) acc[i] = 0.0;
  double2* wb = reinterpret_cast<double2*>(w + (size_t)b * ka.ms);
  const double2* vb = reinterpret_cast<const double2*>(ka.basis + (size_t)b * ka.ms);
  const long long n2 = ka.vl / 2;
  const long long ss = ka.slot_stride / 2;
  for (long long e = (long long)blockIdx.x * kNT + threadIdx.x; e < n2; e += (long long)nblk * kNT) {
    double2 v[MAXNV];
#pragma unroll
    for (int i = 0; i < MAXNV; ++i) v[i] = (i < nv) ? ld_stream(&vb[(size_t)i * ss + e]) : double2{0.0, 0.0};
    double2 wv = wb[e];
#pragma unroll
    for (int i = 0; i < MAXNV; ++i)
      if (i < nv) {
        wv.x -= c[i] * v[i].x;
        wv.y -= c[i] * v[i].y;
      }
    wb[e] = wv;
#pragma unroll
    for (int i = 0; i < MAXNV; ++i)
      if (i < nv) acc[i] += v[i].x * wv.x + v[i].y * wv.y;
    acc[MAXNV] += wv.x * wv.x + wv.y * wv.y;
  }
  double out[MAXNV + 1];
#pragma unroll
  for (int i = 0; i <= MAXNV; ++i) out[i] = (i < nv) ? acc[i] : ((i == nv) ? acc[MAXNV] : 0.0);
  block_reduce_store<MAXNV + 1>(out, nv + 1, partial + ((size_t)b * nblk + blockIdx.x) * kRedStride);
}

template <int MAXNV>
__global__ void __launch_bounds__(kNT) combine_kernel(KrylovArgs ka, int nv, const double* __restrict__ coef,
                                                      int coef_ld, double* __restrict__ out, int accum) {
  const int b = blockIdx.y;
  if (ka.active && !ka.active[b]) return;
  __shared__ double c[MAXNV];
  for (int i = threadIdx.x; i < MAXNV; i += kNT) c[i] = (i < nv) ? coef[(size_t)b * coef_ld + i] : 0.0;
  __syncthreads();
  double2* ob = reinterpret_cast<double2*>(out + (size_t)b * ka.ms);
  const double2* vb = reinterpret_cast<const double2*>(ka.basis + (size_t)b * ka.ms);
  const long long n2 = ka.vl / 2;
  const long long ss = ka.slot_stride / 2;
  for (long long e = (long long)blockIdx.x * kNT + threadIdx.x; e < n2; e += (long long)gridDim.x * kNT) {
    double2 acc = accum ? ob[e] : double2{0.0, 0.0};
#pragma unroll
    for (int i = 0; i < MAXNV; ++i)
      if (i < nv && c[i] != 0.0) {
        const double2 v = ld_stream(&vb[(size_t)i * ss + e]);
        acc.x += c[i] * v.x;
        acc.y += c[i] * v.y;
      }
    ob[e] = acc;
  }
}

// out[b][c] = sum over blocks of partial[b][blk][c]: wave w of the block owns
// the columns c = w, w + 4, ...; lane l adds blocks l, l + 64, ... in order and
// the wave butterfly finishes, so the order is fixed.
__global__ void __launch_bounds__(kNT) reduce_partials_kernel(const double* __restrict__ partial, int nblk,
                                                              int ncols, double* __restrict__ out) {
  const int b = blockIdx.x;
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = threadIdx.x / kWave;
  const double* pb = partial + (size_t)b * nblk * kRedStride;
  for (int c = wv; c < ncols; c += kNWave) {
    double s = 0.0;
    for (int k = lane; k < nblk; k += kWave) s += pb[(size_t)k * kRedStride + c];
    s = wave_sum(s);
    if (lane == 0) out[(size_t)b * kRedStride + c] = s;
  }
}

// First Gram-Schmidt pass bookkeeping for Arnoldi step j:
//   h_i = sc_i <basis_i, w>,  H[b][j][i] = h_i,  coef_i = h_i sc_i,  wnorm2 = <w, w>.
__global__ void gs_step1_kernel(const double* __restrict__ red, int j, int B, const double* __restrict__ sc,
                                double* __restrict__ H, int H_ld, double* __restrict__ coef, int coef_ld,
                                double* __restrict__ wnorm2, const int* __restrict__ active) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  if (active && !active[b]) return;
  const double* r = red + (size_t)b * kRedStride;
  double* Hc = H + ((size_t)b * (kMaxBasis - 1) + j) * H_ld;
  for (int i = 0; i <= j; ++i) {
    const double s = sc[(size_t)b * kMaxBasis + i];
    const double h = s * r[i];
    Hc[i] = h;
    coef[(size_t)b * coef_ld + i] = h * s;
  }
  wnorm2[b] = r[j + 1];
}

// After an update pass: red holds <basis_i, w'> and <w', w'>.
// final_pass = 0: decide on a second pass (skip[b] = 0 means "run it"); the
//   coefficients of the correction are added to column j of H.
// final_pass = 1: for members that ran the second pass, record the norm.
// In both cases the sub-diagonal entry and the scale of the new basis vector
// are set from the measured norm.
__global__ void gs_step2_kernel(const double* __restrict__ red, int j, int B, const double* __restrict__ sc,
                                double* __restrict__ H, int H_ld, double* __restrict__ coef, int coef_ld,
                                const double* __restrict__ wnorm2, double reorth_tol, int* __restrict__ skip,
                                double* __restrict__ sc_out, const int* __restrict__ active, int final_pass) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  if (active && !active[b]) return;
  if (final_pass && skip[b]) return;
  const double* r = red + (size_t)b * kRedStride;
  double* Hc = H + ((size_t)b * (kMaxBasis - 1) + j) * H_ld;
  const double nrm2 = r[j + 1];
  if (!final_pass) {
    double c2 = 0.0;
    for (int i = 0; i <= j; ++i) {
      const double h2 = sc[(size_t)b * kMaxBasis + i] * r[i];
      c2 += h2 * h2;
    }
    const bool again = reorth_tol >= 0.0 && c2 > reorth_tol * reorth_tol * nrm2;
    skip[b] = again ? 0 : 1;
    if (again) {
      for (int i = 0; i <= j; ++i) {
        const double s = sc[(size_t)b * kMaxBasis + i];
        const double h2 = s * r[i];
        Hc[i] += h2;
        coef[(size_t)b * coef_ld + i] = h2 * s;
      }
    }
  }
  const double nrm = sqrt(nrm2 > 0.0 ? nrm2 : 0.0);
  Hc[j + 1] = nrm;
  sc_out[(size_t)b * kMaxBasis + j + 1] = nrm > 0.0 ? 1.0 / nrm : 0.0;
  (void)wnorm2;
}

// out[b][i] = H[b][j][i] for i <= j + 1 (the column the host reads back) and
// out[b][kMaxBasis] = skip[b] (1: no second Gram-Schmidt pass needed)
__global__ void pack_hcol_kernel(const double* __restrict__ H, int H_ld, int j, int B, const int* __restrict__ skip,
                                 double* __restrict__ out) {
  const int b = blockIdx.x;
  const double* Hc = H + ((size_t)b * (kMaxBasis - 1) + j) * H_ld;
  for (int i = threadIdx.x; i <= j + 1; i += blockDim.x) out[(size_t)b * (kMaxBasis + 1) + i] = Hc[i];
  if (threadIdx.x == 0) out[(size_t)b * (kMaxBasis + 1) + kMaxBasis] = skip ? (double)skip[b] : 1.0;
  (void)B;
}

// sc[b][col] = 1/sqrt(red[b][0]),  norm[b] = sqrt(red[b][0])
__global__ void set_scale_kernel(const double* __restrict__ red, int col, int B, double* __restrict__ sc,
                                 double* __restrict__ norm, const int* __restrict__ active) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  if (active && !active[b]) return;
  const double n2 = red[(size_t)b * kRedStride];
  const double nr = sqrt(n2 > 0.0 ? n2 : 0.0);
  norm[b] = nr;
  sc[(size_t)b * kMaxBasis + col] = nr > 0.0 ? 1.0 / nr : 0.0;
}

// ---------------------------------------------------------------------------
// Block Gram-Schmidt: S consecutive Krylov vectors w_0 = Op v_j, w_1 = Op w_0,
// ..., each the operator applied to the one before it without orthogonalising
// in between, sit in the basis slots nv .. nv + S - 1 (nv = j + 1) and are
// orthogonalised together, so the basis is streamed once per S steps by each
// of the two passes instead of once per step.  The Arnoldi steps of a solve
// then move 2 j + 3 S + 2 vectors per S steps instead of S (2 j + 5).
//
// What bounds both passes is HBM.  One thread cannot hold the (nv + ..) S
// partial products of S = 4 (over 160 doubles at 40 basis vectors), so the
// four waves of a block share one chunk of 128 values and split the basis:
// wave k owns the vectors k, k + 4, ...  Every wave of the multi-dot reads the
// chunk of all S new vectors from LDS (loaded by each wave for itself the
// multi-dot ran 2.6 - 6.1 TB/s against 5.5 - 7.1).
// The update exchanges the waves' partial sums through LDS, after which each
// wave still holds its basis values in registers for the products with the
// updated vectors.
// Measured at 2.1 GB vectors (2-D nx = 511, nt = 512), 20 basis vectors and
// S = 4: multi-dot 7.2 ms (7.1 TB/s), update 11.3 ms (5.3 TB/s; without its
// store 6.5 TB/s of reads, so the rest is what a write stream among the reads
// costs), against 4 x (6.4 + 8.7) ms for four single steps.  The 19-step FP64
// solve of that shape spent 71 + 103 ms in single-step passes and 24 + 52 in
// these.
//
// Partial records: part[b][col][blk] (a column is contiguous over the blocks,
// so its reduction is coalesced), col = l nv + i for <basis_i, w_l> and
// S nv + l (l + 1)/2 + k for <w_k, w_l>, k <= l.
// ---------------------------------------------------------------------------

// sums of the N per-lane accumulators over the wave: N - 1 exchanges for N a
// power of two (each step sends one half of the accumulators to the partner
// lane and keeps the other half), then butterflies on the one left.  Lane
// (64 / N) c .. holds the sum of accumulator c.
template <int N, int OFF = kWave / 2>
__device__ __forceinline__ double wave_sum_many(const double (&a)[N]) {
  static_assert((N & (N - 1)) == 0 && N <= kWave, "a power of two");
  if constexpr (N > 1) {
    const bool up = (threadIdx.x & OFF) != 0;
    double h[N / 2];
#pragma unroll
    for (int i = 0; i < N / 2; ++i) {
      const double keep = up ? a[i + N / 2] : a[i], send = up ? a[i] : a[i + N / 2];
      h[i] = keep + __shfl_xor(send, OFF, kWave);
    }
    return wave_sum_many<N / 2, OFF / 2>(h);
  } else {
    double v = a[0];
#pragma unroll
    for (int off = OFF; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
  }
}

constexpr int pow2_at_least(int n) { return n <= 1 ? 1 : 2 * pow2_at_least((n + 1) / 2); }

// writes the wave's sums: accumulator k S + l is column l nv + wv + 4 k,
// gr[k] of wave l < S column S nv + l (l + 1)/2 + k
template <int S, int NVW>
__device__ __forceinline__ void block_partials(double (&acc)[NVW * S], double (&gr)[S], int nv, int wv,
                                               double* __restrict__ part, int nblk) {
  const int lane = threadIdx.x & (kWave - 1);
  // in groups of at most 32 accumulators
  constexpr int PV = NVW * S <= 32 ? NVW : (32 / S);  // vectors per group
  constexpr int PN = pow2_at_least(PV * S);
#pragma unroll
  for (int k0 = 0; k0 < NVW; k0 += PV) {
    double a[PN];
#pragma unroll
    for (int u = 0; u < PN; ++u) a[u] = (u < PV * S && k0 * S + u < NVW * S) ? acc[k0 * S + u < NVW * S ? k0 * S + u : 0] : 0.0;
    const double s = wave_sum_many<PN>(a);
    const int u = lane / (kWave / PN);
    const int k = k0 + u / S, l = u - (u / S) * S, i = wv + 4 * k;
    if (lane % (kWave / PN) == 0 && u < PV * S && k < NVW && i < nv) part[(size_t)(l * nv + i) * nblk] = s;
  }
  constexpr int PG = pow2_at_least(S);
  double a[PG];
#pragma unroll
  for (int u = 0; u < PG; ++u) a[u] = u < S ? gr[u < S ? u : 0] : 0.0;
  const double s = wave_sum_many<PG>(a);
  const int u = lane / (kWave / PG);
  if (lane % (kWave / PG) == 0 && wv < S && u <= wv) part[(size_t)(S * nv + wv * (wv + 1) / 2 + u) * nblk] = s;
}

template <int S, int NVW>
__global__ void __launch_bounds__(kNT) block_mdot_kernel(KrylovArgs ka, int nv, double* __restrict__ part,
                                                         int nblk) {
  const int b = blockIdx.y;
  if (ka.active && !ka.active[b]) return;
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  // a wave's slots past the last basis vector read that vector again and are
  // not stored, so that no load sits behind a branch
  const double2* vb = reinterpret_cast<const double2*>(ka.basis + (size_t)b * ka.ms);
  const size_t ss = (size_t)(ka.slot_stride / 2);
  const double2* wb = vb + (size_t)nv * ss;
  const long long n2 = ka.vl / 2;
  // wave l fetches w_l of the chunk and shares it through LDS (two buffers,
  // so one barrier per chunk); a lane past the end holds zeros
  __shared__ double2 wsh[2][S][kWave];
  int buf = 0;
  double acc[NVW * S], gr[S];
#pragma unroll
  for (int u = 0; u < NVW * S; ++u) acc[u] = 0.0;
#pragma unroll
  for (int u = 0; u < S; ++u) gr[u] = 0.0;
  for (long long c0 = (long long)blockIdx.x * kWave; c0 < n2; c0 += (long long)nblk * kWave) {
    const bool in = c0 + lane < n2;
    const long long e = in ? c0 + lane : n2 - 1;
    double2 w[S], v[NVW];
    if (wv < S) w[0] = wb[wv * ss + e];
#pragma unroll
    for (int k = 0; k < NVW; ++k) v[k] = ld_stream(&vb[(size_t)min(wv + 4 * k, nv - 1) * ss + e]);
    if (wv < S) wsh[buf][wv][lane] = double2{in ? w[0].x : 0.0, in ? w[0].y : 0.0};
    __syncthreads();
#pragma unroll
    for (int l = 0; l < S; ++l) w[l] = wsh[buf][l][lane];
    buf ^= 1;
#pragma unroll
    for (int k = 0; k < NVW; ++k)
#pragma unroll
      for (int l = 0; l < S; ++l) acc[k * S + l] += v[k].x * w[l].x + v[k].y * w[l].y;
    // wave l < S: the products <w_k, w_l> (those with k > l are not used)
    double wlx = w[0].x, wly = w[0].y;
#pragma unroll
    for (int l = 1; l < S; ++l) {
      wlx = wv == l ? w[l].x : wlx;
      wly = wv == l ? w[l].y : wly;
    }
#pragma unroll
    for (int k = 0; k < S; ++k) gr[k] += w[k].x * wlx + w[k].y * wly;
  }
  const int ncols = S * nv + S * (S + 1) / 2;
  block_partials<S, NVW>(acc, gr, nv, wv, part + (size_t)b * ncols * nblk + blockIdx.x, nblk);
}

// w_l <- t_l - sum_{k<l} beta_kl w_k with t_l = w_l - sum_i coef_li basis_i
// (coef[b][l][i], beta[b][k][l], w_k already updated), and the partial
// products of the updated vectors as in the multi-dot.
template <int S, int NVW>
__global__ void __launch_bounds__(kNT) block_update_kernel(KrylovArgs ka, int nv, double* __restrict__ wbase,
                                                           const double* __restrict__ coef,
                                                           const double* __restrict__ beta, double* __restrict__ part,
                                                           int nblk, const int* __restrict__ skip) {
  const int b = blockIdx.y;
  if (ka.active && !ka.active[b]) return;
  if (skip && skip[b]) return;
  __shared__ double2 psum[4][S][kWave];
  __shared__ double2 tsum[S][kWave];
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const double2* vb = reinterpret_cast<const double2*>(ka.basis + (size_t)b * ka.ms);
  const size_t ss = (size_t)(ka.slot_stride / 2);
  double2* wb = reinterpret_cast<double2*>(wbase + (size_t)b * ka.ms);
  const long long n2 = ka.vl / 2;
  const double* cb = coef + (size_t)b * kBlockMax * kMaxBasis;
  double c[NVW][S];  // uniform over the wave
#pragma unroll
  for (int k = 0; k < NVW; ++k)
#pragma unroll
    for (int l = 0; l < S; ++l) {
      const double t = cb[l * kMaxBasis + min(wv + 4 * k, nv - 1)];
      c[k][l] = wv + 4 * k < nv ? t : 0.0;
    }
  double bt[S][S];
#pragma unroll
  for (int l = 1; l < S; ++l)
#pragma unroll
    for (int k = 0; k < l; ++k) bt[k][l] = beta[(size_t)b * kBlockMax * kBlockMax + k * kBlockMax + l];
  double acc[NVW * S], gr[S];
#pragma unroll
  for (int u = 0; u < NVW * S; ++u) acc[u] = 0.0;
#pragma unroll
  for (int u = 0; u < S; ++u) gr[u] = 0.0;
  // every wave of the block runs the same number of chunks (the barriers)
  for (long long c0 = (long long)blockIdx.x * kWave; c0 < n2; c0 += (long long)nblk * kWave) {
    const bool in = c0 + lane < n2;
    const long long e = in ? c0 + lane : n2 - 1;
    double2 v[NVW];
#pragma unroll
    for (int k = 0; k < NVW; ++k) v[k] = ld_stream(&vb[(size_t)min(wv + 4 * k, nv - 1) * ss + e]);
    double2 w0{0.0, 0.0};
    if (wv < S) w0 = wb[wv * ss + e];
    double2 p[S];
#pragma unroll
    for (int l = 0; l < S; ++l) p[l] = double2{0.0, 0.0};
#pragma unroll
    for (int k = 0; k < NVW; ++k)
#pragma unroll
      for (int l = 0; l < S; ++l) {
        p[l].x += c[k][l] * v[k].x;
        p[l].y += c[k][l] * v[k].y;
      }
#pragma unroll
    for (int l = 0; l < S; ++l) psum[wv][l][lane] = p[l];
    __syncthreads();
    if (wv < S) {
      double2 t = w0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        t.x -= psum[q][wv][lane].x;
        t.y -= psum[q][wv][lane].y;
      }
      tsum[wv][lane] = t;
    }
    __syncthreads();
    double2 w[S];
#pragma unroll
    for (int l = 0; l < S; ++l) {
      w[l] = tsum[l][lane];
#pragma unroll
      for (int k = 0; k < l; ++k) {
        w[l].x -= bt[k][l] * w[k].x;
        w[l].y -= bt[k][l] * w[k].y;
      }
    }
    double2 wst = w[0];
#pragma unroll
    for (int l = 1; l < S; ++l) {
      wst.x = wv == l ? w[l].x : wst.x;
      wst.y = wv == l ? w[l].y : wst.y;
    }
    if (wv < S && in) wb[wv * ss + e] = wst;
#pragma unroll
    for (int l = 0; l < S; ++l) {
      w[l].x = in ? w[l].x : 0.0;
      w[l].y = in ? w[l].y : 0.0;
    }
#pragma unroll
    for (int k = 0; k < NVW; ++k)
#pragma unroll
      for (int l = 0; l < S; ++l) acc[k * S + l] += v[k].x * w[l].x + v[k].y * w[l].y;
    // wave l < S: the products <w_k, w_l> (those with k > l are not used)
    double wlx = w[0].x, wly = w[0].y;
#pragma unroll
    for (int l = 1; l < S; ++l) {
      wlx = wv == l ? w[l].x : wlx;
      wly = wv == l ? w[l].y : wly;
    }
#pragma unroll
    for (int k = 0; k < S; ++k) gr[k] += w[k].x * wlx + w[k].y * wly;
  }
  const int ncols = S * nv + S * (S + 1) / 2;
  block_partials<S, NVW>(acc, gr, nv, wv, part + (size_t)b * ncols * nblk + blockIdx.x, nblk);
}

// out[b][col] = sum over the blocks, one wave per column, in a fixed order
__global__ void __launch_bounds__(kNT) block_reduce_kernel(const double* __restrict__ part, int nblk, int ncols,
                                                           double* __restrict__ out) {
  const int b = blockIdx.y;
  const int lane = threadIdx.x & (kWave - 1);
  const int col = blockIdx.x * kNWave + threadIdx.x / kWave;
  if (col >= ncols) return;
  const double* pc = part + ((size_t)b * ncols + col) * nblk;
  double s = 0.0;
  for (int k = lane; k < nblk; k += kWave) s += pc[k];
  s = wave_sum(s);
  if (lane == 0) out[(size_t)b * kBlockRed + col] = s;
}

// Unit upper triangular B of the elimination w_l = sum_k B_kl w'_k + .. from
// the Gram matrix M (k <= l stored at l (l + 1)/2 + k): M = B^T D B.  A pivot
// lost to rounding (the vector depends on the ones before it) eliminates
// nothing; the products measured after the pass then show what is left.
template <int S>
__device__ __forceinline__ void block_ldl(const double (&M)[S * (S + 1) / 2], double (&B)[S][S]) {
  double D[S];
#pragma unroll
  for (int l = 0; l < S; ++l) {
    double d = M[l * (l + 1) / 2 + l];
#pragma unroll
    for (int k = 0; k < l; ++k) {
      double v = M[l * (l + 1) / 2 + k];
#pragma unroll
      for (int q = 0; q < k; ++q) v -= B[q][k] * D[q] * B[q][l];
      B[k][l] = D[k] > 0.0 ? v / D[k] : 0.0;
      d -= B[k][l] * B[k][l] * D[k];
    }
    B[l][l] = 1.0;
    D[l] = d > 0.0 ? d : 0.0;
  }
}

// Bookkeeping of a block after its multi-dot (pass 0), after the first update
// (pass 1) and, for members with skip = 0, after the second (pass 2): one
// wave per member, lane i on basis vector i.  With c_l = V^T w_l the block
// satisfies w_l = sum_i c_li v_i + sum_{k<=l} B_kl w'_k, w'_k the updated
// vectors; a second pass with c2, B2 turns c into c + c2 B and B into B2 B.
// Column j + l of H receives the coefficients of w_l in the orthonormal basis
// (entries 0 .. j + 1 + l), rec the same columns for the host (see launch.hpp).
template <int S>
__global__ void __launch_bounds__(kWave) block_step_kernel(const double* __restrict__ red, int j, int pass,
                                                           double* __restrict__ sc, double* __restrict__ H, int H_ld,
                                                           double* __restrict__ coef, double* __restrict__ beta,
                                                           double* __restrict__ rec, double reorth_tol,
                                                           int* __restrict__ skip, const int* __restrict__ active) {
  const int b = blockIdx.x;
  if (active && !active[b]) return;
  if (pass == 2 && skip[b]) return;
  const int i = threadIdx.x, nv = j + 1;
  const bool own = i < nv;
  const double* r = red + (size_t)b * kBlockRed;
  double* rb = rec + (size_t)b * kBlockRec;
  double* bb = beta + (size_t)b * kBlockMax * kBlockMax;
  double* cb = coef + (size_t)b * kBlockMax * kMaxBasis;
  constexpr int NG = S * (S + 1) / 2;
  const double s = own ? sc[(size_t)b * kMaxBasis + i] : 0.0;
  double c[S], G[NG];
#pragma unroll
  for (int l = 0; l < S; ++l) c[l] = own ? s * r[l * nv + i] : 0.0;
#pragma unroll
  for (int u = 0; u < NG; ++u) G[u] = r[S * nv + u];
  double B[S][S];
  bool again = false;
  if (pass < 2) {
    // Gram matrix of what is left of the block outside the basis
    double M[NG], c2[S];
#pragma unroll
    for (int l = 0; l < S; ++l)
#pragma unroll
      for (int k = 0; k <= l; ++k) {
        const double cc = wave_sum(c[k] * c[l]);
        M[l * (l + 1) / 2 + k] = G[l * (l + 1) / 2 + k] - cc;
        if (k == l) c2[l] = cc;
      }
    if (pass == 1) {
      // a second pass for the member when the measured products of an
      // updated vector with the basis and with the block's earlier vectors
      // exceed reorth_tol times its norm
#pragma unroll
      for (int l = 0; l < S; ++l) {
        double o2 = c2[l];
#pragma unroll
        for (int k = 0; k < l; ++k) {
          const double g = G[l * (l + 1) / 2 + k], d = G[k * (k + 1) / 2 + k];
          o2 += d > 0.0 ? g * g / d : 0.0;
        }
        again = again || (reorth_tol >= 0.0 && o2 > reorth_tol * reorth_tol * G[l * (l + 1) / 2 + l]);
      }
      if (i == 0) skip[b] = again ? 0 : 1;
    }
    block_ldl<S>(M, B);
  }
  // the update kernel's coefficients: c_li sc_i on the unnormalised slots
  if (pass == 0 || again) {
    if (own)
#pragma unroll
      for (int l = 0; l < S; ++l) cb[l * kMaxBasis + i] = c[l] * s;
    if (i == 0)
#pragma unroll
      for (int l = 0; l < S; ++l)
#pragma unroll
        for (int k = 0; k < l; ++k) bb[k * kBlockMax + l] = B[k][l];
  }
  // accumulated c and B, kept in the record between the passes
  double* rB = rb + kBlockRecB;
  if (pass == 0) {
    if (own)
#pragma unroll
      for (int l = 0; l < S; ++l) rb[l * kBlockCol + i] = c[l];
    if (i == 0)
#pragma unroll
      for (int l = 0; l < S; ++l) {
        const double wn = sqrt(G[l * (l + 1) / 2 + l]);
        rb[kBlockRecNorm + l] = wn;
        H[((size_t)b * (kMaxBasis - 1) + j + l) * H_ld + kHld - 1] = wn;
#pragma unroll
        for (int k = 0; k < S; ++k) rB[k * kBlockMax + l] = k <= l ? B[k < l ? k : l][l] : 0.0;
      }
    return;
  }
  double Bt[S][S];
#pragma unroll
  for (int k = 0; k < S; ++k)
#pragma unroll
    for (int l = 0; l < S; ++l) Bt[k][l] = rB[k * kBlockMax + l];
  __syncthreads();  // every lane has read B before it is written back
  double ct[S];
#pragma unroll
  for (int l = 0; l < S; ++l) ct[l] = own ? rb[l * kBlockCol + i] : 0.0;
  if (again) {
#pragma unroll
    for (int l = 0; l < S; ++l)
#pragma unroll
      for (int k = 0; k <= l; ++k) ct[l] += c[k] * Bt[k][l];
    double Bn[S][S];
#pragma unroll
    for (int k = 0; k < S; ++k)
#pragma unroll
      for (int l = 0; l < S; ++l) {
        double v = 0.0;
#pragma unroll
        for (int q = k; q <= l; ++q) v += B[k][q] * Bt[q][l];
        Bn[k][l] = v;
      }
#pragma unroll
    for (int k = 0; k < S; ++k)
#pragma unroll
      for (int l = 0; l < S; ++l) Bt[k][l] = Bn[k][l];
    if (i == 0)
#pragma unroll
      for (int k = 0; k < S; ++k)
#pragma unroll
        for (int l = 0; l < S; ++l) rB[k * kBlockMax + l] = Bt[k][l];
  }
  double nrm[S];
#pragma unroll
  for (int l = 0; l < S; ++l) {
    const double g = G[l * (l + 1) / 2 + l];
    nrm[l] = sqrt(g > 0.0 ? g : 0.0);
  }
  double* Hb = H + ((size_t)b * (kMaxBasis - 1) + j) * H_ld;
#pragma unroll
  for (int l = 0; l < S; ++l) {
    if (own) {
      rb[l * kBlockCol + i] = ct[l];
      Hb[(size_t)l * H_ld + i] = ct[l];
    }
    if (i == 0) {
#pragma unroll
      for (int k = 0; k <= l; ++k) {
        rb[l * kBlockCol + nv + k] = nrm[k] * Bt[k][l];
        Hb[(size_t)l * H_ld + nv + k] = nrm[k] * Bt[k][l];
      }
      sc[(size_t)b * kMaxBasis + nv + l] = nrm[l] > 0.0 ? 1.0 / nrm[l] : 0.0;
    }
  }
  if (i == 0) rb[kBlockRecSkip] = again ? 0.0 : 1.0;
}

// ---------------------------------------------------------------------------
#define PCOP_DISPATCH_NV(KERNEL, NV, GRID, ST, ...)                                   \
  do {                                                                                \
    if ((NV) <= 4) KERNEL<4><<<GRID, kNT, 0, ST>>>(__VA_ARGS__);                      \
    else if ((NV) <= 8) KERNEL<8><<<GRID, kNT, 0, ST>>>(__VA_ARGS__);                 \
    else if ((NV) <= 16) KERNEL<16><<<GRID, kNT, 0, ST>>>(__VA_ARGS__);               \
    else if ((NV) <= 24) KERNEL<24><<<GRID, kNT, 0, ST>>>(__VA_ARGS__);               \
    else if ((NV) <= 32) KERNEL<32><<<GRID, kNT, 0, ST>>>(__VA_ARGS__);               \
    else KERNEL<kMaxBasis><<<GRID, kNT, 0, ST>>>(__VA_ARGS__);                        \
  } while (0)

// exact-size kernels for nv = 0 .. kMaxBasis - 1
using MdotFn = void (*)(KrylovArgs, const double*, double*, int);
using UpdateFn = void (*)(KrylovArgs, double*, const double*, int, double*, int, const int*);
template <int... I>
constexpr std::array<MdotFn, sizeof...(I)> mdot_table(std::integer_sequence<int, I...>) {
  return {&mdot_kernel<I>...};
}
template <int... I>
constexpr std::array<UpdateFn, sizeof...(I)> update_table(std::integer_sequence<int, I...>) {
  return {&update_kernel<I>...};
}
static const auto kMdot = mdot_table(std::make_integer_sequence<int, kMaxBasis>{});
static const auto kUpdate = update_table(std::make_integer_sequence<int, kMaxBasis>{});

void launch_mdot(const KrylovArgs& ka, int nv, const double* w, double* partial, int nblk, hipStream_t st) {
  dim3 grid(nblk, ka.B);
  if (nv < 0 || nv >= kMaxBasis) return;
  kMdot[nv]<<<grid, kNT, 0, st>>>(ka, w, partial, nblk);
}

void launch_update(const KrylovArgs& ka, int nv, double* w, const double* coef, int coef_ld, double* partial,
                   int nblk, const int* skip, hipStream_t st) {
  dim3 grid(nblk, ka.B);
  if (ka.pairs) {
    PCOP_DISPATCH_NV(update2_kernel, nv, grid, st, ka, nv, w, coef, coef_ld, partial, nblk, skip);
  } else if (nv >= 0 && nv < kMaxBasis) {
    kUpdate[nv]<<<grid, kNT, 0, st>>>(ka, w, coef, coef_ld, partial, nblk, skip);
  }
}

void launch_combine(const KrylovArgs& ka, int nv, const double* coef, int coef_ld, double* out, int accum,
                    hipStream_t st) {
  dim3 grid(krylov_blocks(ka.vl), ka.B);
  PCOP_DISPATCH_NV(combine_kernel, nv, grid, st, ka, nv, coef, coef_ld, out, accum);
}

void launch_reduce_partials(const double* partial, int nblk, int ncols, int B, double* out, hipStream_t st) {
  reduce_partials_kernel<<<B, kNT, 0, st>>>(partial, nblk, ncols, out);
}

void launch_gs_step1(const double* red, int j, int B, const double* sc, double* H, int H_ld, double* coef,
                     int coef_ld, double* wnorm2, const int* active, hipStream_t st) {
  gs_step1_kernel<<<(B + 63) / 64, 64, 0, st>>>(red, j, B, sc, H, H_ld, coef, coef_ld, wnorm2, active);
}

void launch_gs_step2(const double* red, int j, int B, const double* sc, double* H, int H_ld, double* coef,
                     int coef_ld, const double* wnorm2, double reorth_tol, int* skip, double* sc_out,
                     const int* active, int final_pass, hipStream_t st) {
  gs_step2_kernel<<<(B + 63) / 64, 64, 0, st>>>(red, j, B, sc, H, H_ld, coef, coef_ld, wnorm2, reorth_tol, skip,
                                                sc_out, active, final_pass);
}

void launch_pack_hcol(const double* H, int H_ld, int j, int B, const int* skip, double* out, hipStream_t st) {
  pack_hcol_kernel<<<B, 64, 0, st>>>(H, H_ld, j, B, skip, out);
}

void launch_set_scale(const double* red, int col, int B, double* sc, double* norm, const int* active,
                      hipStream_t st) {
  set_scale_kernel<<<(B + 63) / 64, 64, 0, st>>>(red, col, B, sc, norm, active);
}

// Blocks per member of the block kernels over nv basis vectors with B members
// running: at least one chunk of 128 values per block, and over all of them
// about as many as keep 10000 chunks of 1 KB in flight (40 KB per CU; counted
// over the members of the batch instead, the last member of 64 ran its passes
// on 32 blocks: 46.8 ms per solve instead of 18.6, 2-D nx = 127, n = 63, V-cycles).  Fewer leave the memory idle,
// more only spread the accesses: at 2.1 GB vectors and S = 4 the multi-dot
// ran, with 512 / 1024 / 2048 blocks, 3.3 / 5.5 / 5.4 TB/s at nv = 1,
// 6.6 / 6.7 / 6.2 at nv = 9 and 7.1 / 6.7 / 6.4 at nv = 20, the update
// 3.2 / 4.8 / 4.8, 5.0 / 5.0 / 5.0 and 5.3 / 5.0 / 5.0.
int block_grid(long long vl, int B, int nv, int S) {
  const long long chunks = (vl / 2 + kWave - 1) / kWave;
  const int all = std::max(kBlockGrid / 4, std::min(kBlockGrid, (10000 / (nv + S) + 128) / 256 * 256));
  return (int)std::max<long long>(1, std::min<long long>(chunks, all / B));
}

using BlockMdotFn = void (*)(KrylovArgs, int, double*, int);
using BlockUpdateFn = void (*)(KrylovArgs, int, double*, const double*, const double*, double*, int, const int*);
// the largest basis a block meets: its vectors take at least two slots of restart + 1
constexpr int kBlockNvw = (kMaxBasis - 1 + 3) / 4;
template <int S, int... I>
constexpr std::array<BlockMdotFn, sizeof...(I)> block_mdot_table(std::integer_sequence<int, I...>) {
  return {&block_mdot_kernel<S, I + 1>...};
}
template <int S, int... I>
constexpr std::array<BlockUpdateFn, sizeof...(I)> block_update_table(std::integer_sequence<int, I...>) {
  return {&block_update_kernel<S, I + 1>...};
}
using BlockSeq = std::make_integer_sequence<int, kBlockNvw>;
static const std::array<BlockMdotFn, kBlockNvw> kBlockMdot[3] = {
    block_mdot_table<2>(BlockSeq{}), block_mdot_table<3>(BlockSeq{}), block_mdot_table<4>(BlockSeq{})};
static const std::array<BlockUpdateFn, kBlockNvw> kBlockUpdate[3] = {
    block_update_table<2>(BlockSeq{}), block_update_table<3>(BlockSeq{}), block_update_table<4>(BlockSeq{})};

void launch_block_mdot(const KrylovArgs& ka, int nv, int S, double* part, int nblk, hipStream_t st) {
  kBlockMdot[S - 2][(nv + 3) / 4 - 1]<<<dim3(nblk, ka.B), kNT, 0, st>>>(ka, nv, part, nblk);
}

void launch_block_update(const KrylovArgs& ka, int nv, int S, const double* coef, const double* beta, double* part,
                         int nblk, const int* skip, hipStream_t st) {
  double* w = const_cast<double*>(ka.basis) + (size_t)nv * ka.slot_stride;
  kBlockUpdate[S - 2][(nv + 3) / 4 - 1]<<<dim3(nblk, ka.B), kNT, 0, st>>>(ka, nv, w, coef, beta, part, nblk, skip);
}

void launch_block_reduce(const double* part, int nblk, int nv, int S, int B, double* out, hipStream_t st) {
  const int ncols = S * nv + S * (S + 1) / 2;
  block_reduce_kernel<<<dim3((ncols + kNWave - 1) / kNWave, B), kNT, 0, st>>>(part, nblk, ncols, out);
}

void launch_block_step(const double* red, int j, int S, int pass, int B, double* sc, double* H, int H_ld,
                       double* coef, double* beta, double* rec, double reorth_tol, int* skip, const int* active,
                       hipStream_t st) {
#define PCOP_BLOCK_STEP(N) \
  block_step_kernel<N><<<B, kWave, 0, st>>>(red, j, pass, sc, H, H_ld, coef, beta, rec, reorth_tol, skip, active)
  if (S == 2) PCOP_BLOCK_STEP(2);
  else if (S == 3) PCOP_BLOCK_STEP(3);
  else PCOP_BLOCK_STEP(4);
#undef PCOP_BLOCK_STEP
}

}  // namespace pcop
