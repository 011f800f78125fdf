"""Split-precision lines in the MFMA operand layout (from 1024 points the first
pass takes its operands from the caller's registers, at 4096 the last pass leaves
them there) and their LDS slots, at every line length: fused range lines and the
RCMC pass's inverse transform, line by line against the oracle.  Neighbouring
lines differ by 2^20 in scale (each has an exponent of its own) and one is zero.
Bounds: one transform's (2e-6 split FP16, 1e-4 split BF16) times sqrt 2 for two in
a row, plus 1e-6 for the interpolation."""
import numpy as np
import pytest

import paper_2604_03585_amd as sar
from gpu_util import dev, empty, host, rand_c64, rel_l2
from oracle import oracle as O
from sarsim import config

pytestmark = pytest.mark.gpu

TOL = {"split_fp16": 2e-6, "split_bf16": 1e-4}
SIZES = [64, 128, 256, 512, 1024, 2048, 4096, 8192, 16384]


@pytest.mark.parametrize("prec", sorted(TOL))
@pytest.mark.parametrize("n", SIZES)
def test_fused_lines(prec, n):
    rng = np.random.Generator(np.random.PCG64(n))
    na = 64
    cfg = config("c1", Nr=n, Na=na, range_len=n // 4, range_tbp=n / 8.0, az_len=16, az_tbp=8.0)
    x = rand_c64(rng, (na, n))
    x[::2] *= np.float32(2.0**20)
    x[5] = 0
    out = empty((na, n))
    with sar.Plan(cfg, precision=prec) as p:
        sar.sar_range_compress(p.handle, dev(x), out)
        got = host(out)
        buf = dev(x)
        sar.sar_range_compress(p.handle, buf, buf)              # in place
        assert np.array_equal(host(buf).view(np.uint32), got.view(np.uint32))
    ref = O.compress_rows(x, O.matched_filter(n, cfg["range_len"], cfg["range_tbp"], +1))
    assert not got[5].any()
    for i in range(na):
        if i != 5:
            assert rel_l2(got[i], ref[i]) < TOL[prec] * np.sqrt(2.0), i


@pytest.mark.parametrize("prec", sorted(TOL))
@pytest.mark.parametrize("na", SIZES)
@pytest.mark.parametrize("nr", [64, 128])
def test_rcmc_lines(prec, na, nr):
    lam, r_near = 5.0 / 32.0, 32768.0
    cfg = config("c2", Nr=nr, Na=na, range_len=32, range_tbp=16.0, lam=lam, r_near=r_near)
    rng = np.random.Generator(np.random.PCG64(na + nr))
    A = rand_c64(rng, (nr, na))
    out = empty((nr, na))
    with sar.Plan(cfg, precision=prec) as p:
        sar.sar_rcmc_azimuth(p.handle, dev(A), out)
        got = host(out)
    ref = O.rcmc_azimuth(A, lam, cfg["v"], r_near, 8, cfg["rcmc_beta"])
    assert rel_l2(got, ref) < TOL[prec] + 1e-6
