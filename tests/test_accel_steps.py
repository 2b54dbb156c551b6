"""The step counts by which a plan may solve its coarsest level directly
(csrc/accel_steps.h, host arithmetic), compiled with g++: equal to the products of
the stage polynomials formed one step at a time in numpy, and quick also where the
schedule runs to thousands of stages, since a plan's creation waits for them."""
import math
import os
import shutil
import subprocess

import numpy as np
import pytest

from oracle import operators as oop
from oracle import rkl as orkl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2306_05332_amd", "csrc")
THETA = 0.9

MAIN = """
#include "accel_steps.h"
#include <chrono>
#include <cstdio>
int main() {  // nx ny nz hx hy hz dtpar periodic count s...
  int n[3], per, m;
  double h[3], dt;
  while (std::scanf("%d %d %d %lf %lf %lf %lf %d %d", n, n + 1, n + 2, h, h + 1, h + 2, &dt, &per, &m) == 9) {
    std::vector<int> sched(m);
    for (int& s : sched) if (std::scanf("%d", &s) != 1) return 1;
    double best = 1e9;
    rkl::AccelSteps r{0, 0};
    for (int q = 0; q < 3; ++q) {
      const auto t0 = std::chrono::steady_clock::now();
      r = rkl::accel_steps(n, h, dt, per != 0, %THETA%, sched, 1e-6, 1e-13);
      best = std::min(best, std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count());
    }
    std::printf("%d %d %.6f\\n", r.loose, r.tight, best);
  }
}
"""

# (nx, ny, nz), h, bc of coarsest levels
LEVELS = [((4, 4, 4), (1.0, 1.0, 1.0), "dirichlet"), ((4, 4, 4), (1.0, 1.0, 1.0), "periodic"),
          ((50, 30, 22), (0.1, 0.1, 0.1), "dirichlet"), ((6, 10, 14), (0.2, 0.1, 0.3), "periodic"),
          ((40, 275, 1), (0.44, 0.28, math.inf), "periodic"), ((2, 2, 2), (1.0, 2.0, 0.5), "periodic"),
          ((64, 64, 1), (1.0, 1.0, math.inf), "dirichlet"), ((50, 30, 22), (0.1, 0.1, 0.005), "dirichlet"),
          ((64, 64, 64), (1.0, 1.0, 0.02), "periodic")]


def _level(n, h, bc):
    return oop.Level(0, n[::-1], h, bc)


def _schedule(lv):
    return [min(s, 4096) for s in orkl.accelerated_schedule(lv, THETA)]


def _numpy_steps(lv, n, h, bc, sched, tol):
    """One recursion per step, as the products are defined."""
    ends = []
    for d in range(3):
        if n[d] == 1:
            continue
        w = 4.0 / h[d] ** 2
        if bc == "periodic":
            ends.append((w * math.sin(math.pi / n[d]) ** 2, w * math.sin(math.pi * (n[d] // 2) / n[d]) ** 2))
        else:
            ends.append((w * math.sin(math.pi / (2 * n[d])) ** 2, w))
    lo = min(e[0] for e in ends) if bc == "periodic" else sum(e[0] for e in ends)
    hi = sum(e[1] for e in ends)
    lam = np.concatenate([lo + (hi - lo) * np.arange(2049) / 2048.0, lo * (hi / lo) ** (np.arange(1, 512) / 512.0)])
    x = 1.0 - THETA * lv.dt_par * lam
    amp = np.ones_like(x)
    for step in range(200):
        s = sched[min(step, len(sched) - 1)]
        p0, p1 = np.ones_like(x), x.copy()
        for j in range(2, s + 1):
            p0, p1 = p1, ((2.0 * j - 1.0) / j) * x * p1 - ((j - 1.0) / j) * p0
        amp *= p1
        worst = np.abs(amp).max()
        if worst <= tol:
            return step + 1
        if not worst < 1e6:
            return 0
    return 0


@pytest.fixture(scope="module")
def counts(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("g++ not found")
    d = tmp_path_factory.mktemp("accel")
    src, exe = str(d / "main.cpp"), str(d / "main")
    with open(src, "w") as f:
        f.write(MAIN.replace("%THETA%", str(THETA)))
    subprocess.run([cxx, "-O3", "-std=c++17", "-I", CSRC, src, "-o", exe], check=True)
    text = ""
    for n, h, bc in LEVELS:
        lv = _level(n, h, bc)
        sched = _schedule(lv)
        text += " ".join(map(repr, [*n, *h, lv.dt_par, int(bc == "periodic"), len(sched), *sched])) + "\n"
    out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split()
    return [(int(out[3 * q]), int(out[3 * q + 1]), float(out[3 * q + 2])) for q in range(len(LEVELS))]


@pytest.mark.parametrize("q", range(len(LEVELS)))
def test_steps_equal_the_products_step_by_step(counts, q):
    n, h, bc = LEVELS[q]
    lv = _level(n, h, bc)
    sched = _schedule(lv)
    print(n, h, bc, "stages", sched[0], "..", sched[-1], "steps", counts[q], flush=True)
    # (numpy's sums of rounding may differ in the last digits: no step count lies that close to its bound)
    assert counts[q][0] == _numpy_steps(lv, n, h, bc, sched, 1e-6)
    assert counts[q][1] == _numpy_steps(lv, n, h, bc, sched, 1e-13)


def test_steps_are_quick_on_anisotropic_levels(counts):
    """One recursion up to the largest stage count: at most 4096 passes over 2560
    samples, some 10 ms; a recursion per step and tolerance took 0.5 to 1 s."""
    assert max(c[2] for c in counts) < 0.1
