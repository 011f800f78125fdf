"""The RCMC kernel that forms four output rows at once, at every azimuth line
length, against the oracle: geometries just inside its limit on the change of
shift per row and just outside (the two-row kernel), shifts of none, a few and
more cells than the scene has, with rows at both scene edges.  The scene rows
are all edge rows at 64 range cells.  Relative L2 below 1e-6, the bound of one
azimuth stage (FP32 transform and interpolation, u sqrt(log2 N) each)."""
import numpy as np
import pytest

import paper_2604_03585_amd as sar
from gpu_util import dev, empty, host, rand_c64, rel_l2
from oracle import oracle as O
from sarsim import config

pytestmark = pytest.mark.gpu

# lambda of the 4096^2 scene is 5/32 (change of shift per row at most 3.8e-4
# cells); 0.178 gives 4.97e-4, 0.18 gives 5.07e-4
GEOMETRIES = [(5.0 / 32.0, 32768.0), (0.178, 0.0), (0.178, 31000.25), (0.18, 32768.0), (5.0 / 32.0, 1.0e6),
              (0.0, 0.0)]


@pytest.mark.parametrize("na", [64, 128, 256, 512, 1024, 2048, 4096, 8192, 16384])
@pytest.mark.parametrize("nr", [64, 256])
@pytest.mark.parametrize("geometry", range(len(GEOMETRIES)))
def test_rows(na, nr, geometry):
    lam, r_near = GEOMETRIES[geometry]
    lam = lam or 1e-4                                # next to no migration: every shift is 0
    if nr == 256 and na > 4096:
        pytest.skip("covered by the narrow scene")
    cfg = config("c2", Nr=nr, Na=na, range_len=32, range_tbp=16.0, lam=lam, r_near=r_near)
    rng = np.random.Generator(np.random.PCG64(na + nr + geometry))
    A = rand_c64(rng, (nr, na))
    out = empty((nr, na))
    with sar.Plan(cfg) as p:
        sar.sar_rcmc_azimuth(p.handle, dev(A), out)
        got = host(out)
    ref = O.rcmc_azimuth(A, lam, cfg["v"], r_near, 8, cfg["rcmc_beta"])
    assert rel_l2(got, ref) < 1e-6


@pytest.mark.parametrize("na", [64, 256, 1024, 2048, 4096, 8192])
def test_half_storage_rows(na):
    """The same kernel over FP16 rows (half storage), whole scene against the
    oracle at the two FP16 roundings' bound."""
    from sarsim import simulate
    cfg = config("c2", Nr=512, Na=na, range_len=64, range_tbp=32.0, n_targets=1, spacing=8,
                 exposure=min(1024, na // 2))
    sc = simulate(cfg)
    with sar.Plan(cfg, precision="fp32_halfstore") as p:
        img = host(p.execute(dev(sc.raw))).T
    assert rel_l2(img, O.rda(sc.raw, cfg)) < 2e-3
