// Device code of one sine-transform line, shared by the passes of dst.hip and
// modes.hip: the Stockham stages of a line held in registers, with one LDS
// exchange between stages, and the half-length transform around them.
#pragma once

#include "common.hpp"
#include "fft_lds.hpp"

namespace pcop {

// LDS slot of position p of a line.  gfx950's LDS serves a 16-byte read to
// 16 lanes per pass, without conflict when their slots differ modulo 16, a
// 16-byte write to 8 lanes per pass (slots differing modulo 8), and 8-byte
// reads and writes to 16 lanes (8-byte slots differing modulo 16); this was
// measured with single-instruction loops over fixed lane patterns.  The
// accesses of a line are runs of consecutive positions (stage reads, the
// post-pass writes), stride-8 runs (first-stage writes, p = 8t + r) and
// stride-4 runs (the post-pass reads, p = 4t + i).  XOR-ing the low three
// bits of p with a function h of its 8-slot block b = p / 8 keeps all three
// conflict-free: h takes eight distinct values on any eight consecutive
// blocks (stride-8 writes), and distinct low two bits on the four blocks of
// equal parity inside eight (stride-4 reads).  With 8-byte slots a stride-8
// run of 16 lanes covers sixteen blocks, so bit 3 of p is also flipped by
// bit 3 of b.  Every slot stays in the aligned group of 8 (16-byte slots, or
// positions below 64) or 16 of its position, so a line of X positions needs
// X slots when X is a multiple of 16.
template <class T>
__device__ __forceinline__ int pidx(int p) {
  const int b = p >> 3;
  if constexpr (sizeof(T) == 8) return p ^ (((b >> 1) & 3) | ((b & 1) << 2));
  else return p ^ (((b >> 1) & 7) | (b & 8));
}

// Synchronisation of the threads of one line around an exchange through the
// line's own LDS slots.  A line of at most 64 threads lies inside one
// wavefront, whose LDS instructions complete in issue order, so a compiler
// barrier suffices to keep its writes before its reads (and its reads
// before the next writes); longer lines span several wavefronts and take
// the block barrier.
template <int TL>
__device__ __forceinline__ void line_sync() {
  if constexpr (TL <= 64) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
}

// LDS row length of a line of X positions: X once a line fills whole lane
// groups (X >= 128); shorter lines share a wave's lane groups, and one pad
// slot per 8 then keeps neighbouring lines on different banks
constexpr int line_ld(int X) { return X <= 64 ? X + X / 8 : X; }

template <class T, int L, int TL, int SG, int NS>
struct RegStages {
  static __device__ __forceinline__ void run(cx<T> (&v)[8], int t, cx<T>* lbuf, const cx<T>* __restrict__ twL) {
    constexpr int R = (L / NS >= 8) ? 8 : (L / NS);
    constexpr int Q = 8 / R;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int jb = t + TL * q;
      const int jl = jb % NS;
      cx<T> a[R];
#pragma unroll
      for (int r = 0; r < R; ++r) a[r] = v[q + r * Q];
      if (NS > 1 && jl != 0) {
        constexpr int tstep = L / (NS * R);
        if constexpr (sizeof(T) == 8) {
          cx<T> w1 = twL[jl * tstep];
          if (SG > 0) w1.y = -w1.y;
          cx<T> w = w1;
#pragma unroll
          for (int r = 1; r < R; ++r) {
            a[r] = a[r] * w;
            w = w * w1;
          }
        } else {
#pragma unroll
          for (int r = 1; r < R; ++r) {
            cx<T> w = twL[(r * jl * tstep) & (L - 1)];
            if (SG > 0) w.y = -w.y;
            a[r] = a[r] * w;
          }
        }
      }
      dftR<T, SG, R>(a);
#pragma unroll
      for (int r = 0; r < R; ++r) v[q + r * Q] = a[r];
    }
    if constexpr (NS * R < L) {
      // exchange: outputs to LDS, next stage's inputs back
      line_sync<TL>();
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const int jb = t + TL * q;
        const int jl = jb % NS;
        const int base = (jb - jl) * R + jl;
#pragma unroll
        for (int r = 0; r < R; ++r) lbuf[pidx<T>(base + r * NS)] = v[q + r * Q];
      }
      line_sync<TL>();
#pragma unroll
      for (int s = 0; s < 8; ++s) v[s] = lbuf[pidx<T>(t + TL * s)];
      RegStages<T, L, TL, SG, NS * R>::run(v, t, lbuf, twL);
    }
  }
};

// the odd extension's second half, positions t + TL k for k = 4..7, from the
// first (position p mirrors L - p; positions 0 and N + 1 hold zero)
template <class T, int L, int TL>
__device__ __forceinline__ void mirror(cx<T> (&z)[8], int t, cx<T>* lbuf) {
  line_sync<TL>();
#pragma unroll
  for (int k = 0; k < 4; ++k) lbuf[pidx<T>(t + TL * k)] = z[k];
  line_sync<TL>();
#pragma unroll
  for (int k = 4; k < 8; ++k) {
    const int pos = t + TL * k;
    const cx<T> q = lbuf[pidx<T>(pos == L / 2 ? 0 : L - pos)];
    z[k] = cx<T>{-q.x, -q.y};
  }
}

// threads per block of the register row kernel: 128 from L = 512 on (two
// lines of 64 threads, or one line of 128 at L = 1024, where the block's
// exchanges then wait on two wavefronts instead of four: measured 5% faster
// than 256-thread blocks at L = 1024 and 2% at L = 512 in FP64), else 256
constexpr int reg_threads(int L) { return L >= 512 ? (L / 8 > 128 ? L / 8 : 128) : 256; }

// The half-length transform of one line (see dst_half_kernel in dst.hip for the
// formulas).
template <class T, int L>
struct HalfDst {
  static constexpr int M = L / 2, N = M - 1, TM = M / 8;
  // y_j (j = t + TM s) from the line's values z_{e+1} at lbuf[pidx(e ^ sw)]
  static __device__ __forceinline__ void pre(cx<T> (&v)[8], int t, const cx<T>* lbuf, const T* sinl, int sw = 0) {
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int j = t + TM * s;
      if (j == 0) {
        v[s] = cx<T>{0, 0};
      } else {
        const cx<T> a = lbuf[pidx<T>((j - 1) ^ sw)], b = lbuf[pidx<T>((M - j - 1) ^ sw)];
        const T sj = sinl[j];
        const cx<T> sum = a + b, dif = a - b;
        v[s] = cx<T>{sj * sum.x + (T)0.5 * dif.x, sj * sum.y + (T)0.5 * dif.y};
      }
    }
  }
  // from U (natural order in v, positions t + TM s) to Y at positions
  // 8t .. 8t + 7 (o[r] = Y_{8t + r}); the prefix sum runs over the TM
  // threads of the line, which sit in one wavefront
  static __device__ __forceinline__ void post(cx<T> (&v)[8], cx<T> (&o)[8], int t, cx<T>* lbuf) {
    line_sync<TM>();
#pragma unroll
    for (int s = 0; s < 8; ++s) lbuf[pidx<T>(t + TM * s)] = v[s];
    line_sync<TM>();
    cx<T> c[4], e[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int k = 4 * t + i;
      const cx<T> uk = lbuf[pidx<T>(k)];
      const cx<T> um = lbuf[pidx<T>(k == 0 ? 0 : M - k)];
      c[i] = (k == 0) ? uk : uk + um;
      e[i] = uk - um;
    }
    // inclusive prefix within the thread, then an exclusive scan of the
    // thread totals over the line
    cx<T> run = c[0];
    c[0] = run;
#pragma unroll
    for (int i = 1; i < 4; ++i) {
      run = run + c[i];
      c[i] = run;
    }
    cx<T> incl = run;
#pragma unroll
    for (int d = 1; d < TM; d *= 2) {
      const T px = __shfl_up(incl.x, d, TM);
      const T py = __shfl_up(incl.y, d, TM);
      if (t >= d) incl = incl + cx<T>{px, py};
    }
    const cx<T> excl = incl - run;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const cx<T> pk = excl + c[i];
      o[2 * i] = e[i];                      // Y_{2k} (Y_0 unused)
      o[2 * i + 1] = cx<T>{pk.y, -pk.x};    // -i P_k
    }
  }
};

}  // namespace pcop
