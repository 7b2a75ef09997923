"""The committed tuner choices belong to the kernels of this tree (their version is
the library's), and the benchmark names the preconditioner that a leg ran."""
import os
import re

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_committed_choices_have_the_library_version():
    src = open(os.path.join(ROOT, "paper_2410_22686_amd", "csrc", "pcop.cpp")).read()
    version = int(re.search(r"kTuneVersion = (\d+);", src).group(1))
    rows = [r.split() for r in open(bench.DEFAULT_TUNE_CACHE) if r.startswith("pcop-tune ")]
    assert len(rows) >= 6 and all(int(r[1]) == version and len(r) == 3 + 14 + 4 + 3 * 41 for r in rows)
    assert len({tuple(r[2:17]) for r in rows}) == len(rows)


def test_bench_names_the_route():
    assert bench.precond_route({"mdot": {}, "modes": {}, "dst_rows": {}}) == "by modes"
    assert bench.precond_route({"time_fwd": {}, "time_inv": {}, "dst_rows": {}}) == "time transforms"
    assert bench.precond_route({"ideal_step": {}, "mg_smooth": {}}) == "step by step"
    assert bench.precond_route({"mdot": {}}) is None
