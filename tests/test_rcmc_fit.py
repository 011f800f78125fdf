"""The RCMC kernels' weight tables against the oracle's weights, on the CPU (the
fit is host code too): the cubics that serve four rows at once, over the whole
range of u at which the kernel evaluates them, are nowhere further off than the
quadratics within their own intervals, in exact coefficients and in the FP32 ones
that the kernels read."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from oracle import oracle as O

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2604_03585_amd", "csrc")
ROCM = "/opt/rocm/include"

pytestmark = pytest.mark.skipif(not shutil.which("g++") or not os.path.isdir(ROCM), reason="g++ and the HIP headers")

PROGRAM = r"""
#include "rcmc_fit.hpp"
#include <cstdio>
#include <cstdlib>
int main(int argc, char** argv)
{
    using namespace sar;
    static float tab[RCMC_TAB + RROWS_TAB];
    std::printf("%d %d %.17g\n", RCMC_INTERVALS, RROWS_INTERVALS, RROWS_MARGIN);
    for (int i = 1; i < argc; ++i) {
        const double beta = std::atof(argv[i]);
        for (int b = 0; b < RCMC_INTERVALS; ++b)
            rcmc_fit<2>(tab + b * RCMC_PER_INTERVAL, b, RCMC_INTERVALS, 0.0, beta);
        for (int b = 0; b < RROWS_INTERVALS; ++b)
            rcmc_fit<3>(tab + RCMC_TAB + b * RROWS_PER_INTERVAL, b, RROWS_INTERVALS, RROWS_MARGIN, beta);
        for (float v : tab) std::printf("%.9g ", (double)v);
        std::printf("\n");
    }
}
"""

BETAS = [0.0, 1.0, 2.5, 6.0, 20.0]


@pytest.fixture(scope="module")
def tables(tmp_path_factory):
    d = tmp_path_factory.mktemp("fit")
    (d / "fit.cpp").write_text(PROGRAM)
    r = subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-isystem", ROCM,
                        "-o", str(d / "fit"), str(d / "fit.cpp")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    lines = subprocess.run([str(d / "fit"), *map(str, BETAS)], capture_output=True, text=True,
                           check=True).stdout.split("\n")
    nq, nc, margin = lines[0].split()
    return int(nq), int(nc), float(margin), {b: np.array(l.split(), dtype=np.float64)
                                             for b, l in zip(BETAS, lines[1:])}


def worst(c, n, margin, beta):
    """Largest error of the pieces c[n][8][k] at u in [-margin, 1 + margin], x in [0, 1)."""
    e = 0.0
    u = np.concatenate([np.linspace(-margin, 1.0 + margin, 23), [0.0, 1.0]])
    for b in range(n):
        for v in u:
            x = (b + v) / n
            if 0.0 <= x < 1.0:
                w = sum(c[b, :, k] * v**k for k in range(c.shape[2]))
                e = max(e, float(np.max(np.abs(w - O.rcmc_weights(x, beta, 8)))))
    return e


@pytest.mark.parametrize("beta", BETAS)
def test_four_row_weights_no_further_off(tables, beta):
    nq, nc, margin, tabs = tables
    t = tabs[beta]
    quad, cubic = t[:nq * 24].reshape(nq, 8, 3), t[nq * 24:].reshape(nc, 8, 4)
    eq, ec = worst(quad, nq, 0.0, beta), worst(cubic, nc, margin, beta)
    print(f"beta {beta}: quadratics {eq:.3e}, cubics {ec:.3e}")
    assert margin >= 1.5 * 5e-4 * nc                 # three rows' change at the kernel's limit
    assert ec <= eq < 1e-7
