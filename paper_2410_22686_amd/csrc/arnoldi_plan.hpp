// How many Arnoldi steps the next block of a solve takes, and which of them are
// replayed as graphs (host code without device calls).  A step too many costs
// an operator apply, a block too short streams the basis once more.
#pragma once

#include <algorithm>
#include <cmath>

namespace pcop {

// The longest block among a solve's first kShortSteps steps.  A loose tolerance
// is often met by them, and a solve that ends there has little to save on the
// basis (2-D nx = 255, n = 127, rtol = 0.1, two steps: a block of four 2.83 ms,
// single steps 2.25, a block of two 1.93).  Counted in vectors moved over 720
// residual histories of right-preconditioned solves (2-D nx 15..255, n 31..255,
// gamma 1e-10..1e4, three eps), blocks of four cost more than single steps in
// 684 at rtol = 0.1, 110 at 1e-3 and 70 at 1e-4, at worst by 1.5; with this
// limit in none, 12 and none, at worst by 1.15, and as much is saved over all.
constexpr int kShortSteps = 6;
inline int first_block(double rtol, int limit) { return std::min(limit, rtol >= 0.3 ? 1 : rtol >= 1e-4 ? 2 : limit); }

// Steps that the last k (one or two) steps' rate, from residual before to est,
// says are left.  Two steps, since the residual tends to fall on every second
// one; the rate of a whole block lags behind it (more vectors than single steps
// in 30 of those solves at rtol = 1e-8, in none with this one).
inline int steps_left(double est, double before, int k, double rtol, int limit) {
  if (!(est > rtol && est < before)) return limit;
  return (int)std::max(1.0, std::min<double>(limit, std::ceil(k * std::log(est / rtol) / std::log(before / est))));
}

// Steps from step j of a cycle on that one captured graph holds, 0 where the
// block of S steps is launched plainly.  full: the solve's longest block, first:
// its first_block, chunk: graph_chunk.  Graphs hold whole blocks at fixed
// places -- the short blocks of a loose tolerance, and every G steps (the blocks
// that fit chunk, one at least) from the start of a cycle or behind a short
// first block -- so a context stores at most 2 ceil(restart / G) + kShortSteps
// of them, whatever the data.  Block lengths follow the convergence seen;
// captured wherever they led, a right-hand side that converged otherwise met
// captures (some 0.1 ms each) inside its solve.
inline int graph_steps(int j, int S, int full, int first, int chunk, int restart) {
  if (S == first && first < full && j < kShortSteps && j % first == 0) return S;
  const int G = full * std::max(1, chunk / full);
  const bool placed = j % G == 0 || (first < full && j > 0 && (j - first) % G == 0);
  if (S != full || !placed || j + full > restart) return 0;
  return full * std::max(1, std::min(chunk, restart - j) / full);
}

}  // namespace pcop
