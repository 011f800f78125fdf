"""sar_batch_execute refuses a workspace that is not 16-byte aligned
(SAR_ERR_BAD_PARAM), whichever launches its scenes share, and the same batch
runs on an aligned one afterwards."""
import numpy as np
import pytest

import paper_2604_03585_amd as sar
from gpu_util import dev, host, rand_c64, torch_cuda
from paper_2604_03585_amd import _lib
from sarsim import config

pytestmark = pytest.mark.gpu

SETS = {"strips": [(256, 128, {}), (128, 512, {})], "turned": [(256, 128, {"precision": "split_fp16"})],
        "mixed": [(256, 128, {}), (64, 128, {}), (128, 256, {"transpose_back": 1})]}


@pytest.mark.parametrize("name", list(SETS))
@pytest.mark.parametrize("graph", [False, True])
def test_misaligned_workspace_is_refused(name, graph):
    torch = torch_cuda()
    rng = np.random.Generator(np.random.PCG64(3))
    cfgs = [(config("c1", Nr=nr, Na=na, range_len=nr // 4, range_tbp=nr / 8.0, az_len=na // 4, az_tbp=na / 8.0), o)
            for na, nr, o in SETS[name]]
    raws = [dev(rand_c64(rng, (na, nr))) for na, nr, _ in SETS[name]]
    want, imgs = [], []
    for (c, o), raw in zip(cfgs, raws):
        with sar.Plan(c, **o) as p:
            want.append(host(p.execute(raw)).view(np.uint32))
            imgs.append(torch.zeros(p.image_shape(), dtype=torch.complex64, device="cuda"))
    stream = torch.cuda.Stream() if graph else 0
    b = sar.sar_batch_plan([sar.make_params(c, **o) for c, o in cfgs], stream)
    try:
        work = torch.zeros(sar.sar_batch_workspace_bytes(b) // 8 + 2, dtype=torch.complex64, device="cuda")
        torch.cuda.synchronize()
        for _ in range(2):
            with pytest.raises(sar.SarError) as e:
                sar.sar_batch_execute(b, raws, imgs, work[1:], stream)
            assert e.value.status == _lib.SAR_ERR_BAD_PARAM
        torch.cuda.synchronize()
        assert not any(bool(i.abs().any()) for i in imgs)
        sar.sar_batch_execute(b, raws, imgs, work, stream)
        torch.cuda.synchronize()
        for i, w in zip(imgs, want):
            assert np.array_equal(host(i).view(np.uint32), w)
    finally:
        torch.cuda.synchronize()
        sar.sar_batch_destroy(b)
