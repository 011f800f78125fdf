"""The persistent line kernel (fused lines of 8192 points and more, single
transforms of 16384) against the one-line-per-workgroup kernel, which smaller
launches of the same lines take: the butterflies are the same, so the results
are equal bit for bit, whatever the number of lines per workgroup."""
import numpy as np
import pytest

import paper_2604_03585_amd as sar
from gpu_util import host, torch_cuda

pytestmark = pytest.mark.gpu


def cfg(nr, na):
    return dict(Nr=nr, Na=na, range_len=nr // 8, range_tbp=nr / 16.0, az_model="lfm",
                az_len=na // 4, az_tbp=na / 8.0, lam=0.0, v=0.0, r_near=0.0, rcmc_taps=0,
                rcmc_beta=2.5)


def noise(lines, n, seed):
    torch = torch_cuda()
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.empty((lines, n, 2), dtype=torch.float32, device="cuda")
    return torch.view_as_complex(x.normal_(0.0, 1.0, generator=g))


@pytest.mark.parametrize("n, na", [(8192, 1024), (8192, 2048), (16384, 512), (16384, 1024)])
@pytest.mark.parametrize("in_place", [False, True])
def test_fused_lines(n, na, in_place):
    torch = torch_cuda()
    x = noise(na, n, n + na)
    ref = torch.empty_like(x)
    with sar.Plan(cfg(n, 64)) as small:              # 64 lines: one per workgroup
        for i in range(0, na, 64):
            sar.sar_range_compress(small.handle, x[i:i + 64], ref[i:i + 64])
        want = host(ref)
    out = x if in_place else torch.empty_like(x)
    with sar.Plan(cfg(n, na)) as p:
        sar.sar_range_compress(p.handle, x, out)
        got = host(out)
    assert np.array_equal(got.view(np.uint32), want.view(np.uint32))


@pytest.mark.parametrize("lines", [256, 257, 511, 513, 700])
@pytest.mark.parametrize("inverse", [0, 1])
def test_single_transforms(lines, inverse):
    torch = torch_cuda()
    n = 16384
    x = noise(lines, n, lines)
    out, ref = torch.zeros_like(x), torch.empty_like(x)
    with sar.Plan(cfg(n, 64)) as p:
        sar.sar_fft_lines(p.handle, 0, inverse, x, out, lines)
        for i in range(0, lines, 100):
            m = min(100, lines - i)
            sar.sar_fft_lines(p.handle, 0, inverse, x[i:i + m], ref[i:i + m], m)
        got, want = host(out), host(ref)
    assert np.array_equal(got.view(np.uint32), want.view(np.uint32))
