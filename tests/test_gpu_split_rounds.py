"""Split-precision fused lines in a launch of one round of workgroups and of more
(two builds of the kernel, by the number of lines): the same bits, either side of
the limit of 768 workgroups."""
import numpy as np
import pytest

import paper_2604_03585_amd as sar
from gpu_util import dev, empty, host, rand_c64
from sarsim import config

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["split_fp16", "split_bf16"])
@pytest.mark.parametrize("n, na", [(1024, 2048), (1024, 4096), (2048, 1024), (2048, 2048)])
def test_range_lines_same_bits(prec, n, na):
    def cfg(rows):
        return config("c1", Nr=n, Na=rows, range_len=n // 4, range_tbp=n / 8.0, az_len=16, az_tbp=8.0)

    x = rand_c64(np.random.Generator(np.random.PCG64(n + na)), (na, n))
    out, ref = empty((na, n)), empty((na, n))
    raw = dev(x)
    with sar.Plan(cfg(na), precision=prec) as p:
        sar.sar_range_compress(p.handle, raw, out)
        got = host(out).view(np.uint32)
    with sar.Plan(cfg(64), precision=prec) as p:         # 64 lines: one round
        for i in range(0, na, 64):
            sar.sar_range_compress(p.handle, raw[i:i + 64], ref[i:i + 64])
        assert np.array_equal(host(ref).view(np.uint32), got)
