"""The host's plan of Arnoldi blocks and graphs (arnoldi_plan.hpp), compiled by
itself: whatever block lengths the convergence leads to, the graphs that a
context can ask for are few and fit the cycle."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2410_22686_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <set>
#include <vector>
#include "arnoldi_plan.hpp"
using namespace pcop;

static int fail(const char* what, int a, int b, int c, int d) {
  std::printf("%s: full %d first %d chunk %d restart %d\n", what, a, b, c, d);
  return 1;
}

int main() {
  for (int full : {1, 2, 4})
    for (double rtol : {0.5, 0.1, 1e-3, 1e-8})
      for (int chunk = 1; chunk <= 12; ++chunk)
        for (int restart = 1; restart <= 40; ++restart) {
          const int first = first_block(rtol, full);
          if (first < 1 || first > full) return fail("first block", full, first, chunk, restart);
          std::set<std::pair<int, int>> graphs;
          // every step that any sequence of block lengths reaches (a cut
          // continues with single steps)
          std::vector<char> reached(restart + 1, 0);
          reached[0] = 1;
          for (int j = 0; j < restart; ++j) {
            if (!reached[j]) continue;
            for (int S = 1; S <= full && j + S <= restart; ++S) {
              const int g = graph_steps(j, S, full, first, chunk, restart);
              if (g != 0) {
                if (g % S != 0 || j + g > restart) return fail("graph", full, first, chunk, restart);
                graphs.insert({j * 64 + S, g});
              }
              for (int k = 1; k <= (g ? g : S); ++k) reached[j + k] = 1;
            }
          }
          const int G = full > chunk ? full : chunk / full * full;
          if ((int)graphs.size() > 2 * ((restart + G - 1) / G) + kShortSteps) return fail("too many graphs", full, first, chunk, restart);
          // a solve of full blocks runs as graphs from its start to the last
          // whole block of the cycle
          int j = 0;
          while (j + full <= restart) {
            const int S = j == 0 ? first : full;
            if (j + S > restart) break;
            const int g = graph_steps(j, S, full, first, chunk, restart);
            if (g == 0 || (j < kShortSteps && j % first == 0 && j + first <= restart &&
                           graph_steps(j, first, full, first, chunk, restart) == 0 && first < full))
              return fail("plain block", full, first, chunk, restart);
            j += g;
          }
        }
  // the rate of the last steps: one decade per step, five to go
  if (steps_left(1e-3, 1e-1, 2, 1e-8, 4) != 4 || steps_left(1e-6, 1e-4, 2, 1e-8, 4) != 2) return fail("rate", 0, 0, 0, 0);
  if (steps_left(1e-7, 1e-6, 1, 1e-8, 4) != 1 || steps_left(0.9, 0.8, 2, 1e-8, 4) != 4) return fail("rate", 1, 0, 0, 0);
  std::puts("ok");
  return 0;
}
"""


def test_blocks_and_graphs(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text(PROGRAM)
    r = subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-I", CSRC, str(src), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
