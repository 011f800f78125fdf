"""Back-turned images of the strip kernels, pass after pass: the same bits every
time.  (Their 16-byte stores once lost a race with the instruction after them in
a few of a hundred passes; see test_wide_store_asm.py for the cause.)"""
import pytest

import paper_2604_03585_amd as sar
from gpu_util import torch_cuda
from sarsim import config

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("na, nr", [(64, 4096), (128, 2048), (256, 256), (256, 4096), (512, 1024), (512, 2048),
                                    (1024, 512), (1024, 2048), (2048, 1024), (4096, 1024)])
def test_same_bits_every_pass(na, nr):
    torch = torch_cuda()
    cfg = config("c1", Nr=nr, Na=na, range_len=nr // 4, range_tbp=nr / 8.0, az_len=na // 4, az_tbp=na / 8.0)
    g = torch.Generator(device="cuda").manual_seed(na + nr)
    raw = torch.view_as_complex(torch.empty((na, nr, 2), device="cuda").normal_(generator=g))
    with sar.Plan(cfg) as p:                       # by steps, without the strips
        a, b, w = (torch.empty(na * nr, dtype=torch.complex64, device="cuda") for _ in range(3))
        sar.sar_range_compress(p.handle, raw, a)
        sar.sar_corner_turn(p.handle, a, b, na, nr)
        sar.sar_azimuth_compress(p.handle, b, a, w)
        want = a.view(nr, na).T.contiguous().view(torch.int64)
        torch.cuda.synchronize()
    wrong = torch.zeros((), dtype=torch.int64, device="cuda")
    with sar.Plan(cfg, transpose_back=1) as p:
        img = torch.empty((na, nr), dtype=torch.complex64, device="cuda")
        work = torch.empty(p.workspace_bytes, dtype=torch.uint8, device="cuda")
        for _ in range(300):
            p.execute(raw, out=img, work=work)
            wrong += (img.view(torch.int64) != want).sum()
        assert int(wrong) == 0
