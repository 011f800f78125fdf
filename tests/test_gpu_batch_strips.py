"""Batched scenes that run without the corner turn (two launches for every line
length together): each image bit-identical to its single-scene run, at the
shortest and longest lines, scenes narrower than a workgroup's strips, every
length next to every other in one launch, and next to scenes that keep the
turned passes (shorter and longer lines, a turned-back image, split FP16)."""
import numpy as np
import pytest

import paper_2604_03585_amd as sar
from gpu_util import dev, host, rand_c64, torch_cuda
from sarsim import config

pytestmark = pytest.mark.gpu

LENGTHS = [128, 256, 512, 1024, 2048, 4096]
SETS = {
    "single 128": [(128, 128)],
    "every azimuth length over the narrowest range": [(n, 128) for n in LENGTHS],
    "every range length over the shortest azimuth": [(128, n) for n in LENGTHS],
    "squares": [(n, n) for n in LENGTHS[:4]] + [(1024, 1024), (512, 512), (128, 128)],
    "mixed": [(4096, 512), (64, 256), (256, 64), (512, 8192), (8192, 128), (512, 4096), (256, 256, 1),
              (256, 512, "split_fp16"), (2048, 1024), (128, 2048)],
}


def plan_args(scene):
    na, nr = scene[:2]
    cfg = config("c1", Nr=nr, Na=na, range_len=nr // 4, range_tbp=nr / 8.0, az_len=na // 4, az_tbp=na / 8.0)
    extra = scene[2] if len(scene) > 2 else None
    return cfg, {"transpose_back": 1} if extra == 1 else ({"precision": extra} if extra else {})


@pytest.mark.parametrize("graph", [True, False])
@pytest.mark.parametrize("name", list(SETS))
def test_batch_equals_single_scenes(name, graph):
    torch = torch_cuda()
    scenes = SETS[name]
    rng = np.random.Generator(np.random.PCG64(len(name)))
    args = [plan_args(s) for s in scenes]
    raws = [dev(rand_c64(rng, s[:2])) for s in scenes]
    want = []
    for (cfg, opt), raw in zip(args, raws):
        with sar.Plan(cfg, **opt) as p:
            want.append(host(p.execute(raw)).view(np.uint32))
    stream = torch.cuda.Stream() if graph else 0
    b = sar.sar_batch_plan([sar.make_params(c, **o) for c, o in args], stream)
    try:
        imgs = [torch.full(w.shape, float("nan"), dtype=torch.float32, device="cuda").view(torch.complex64)
                for w in want]
        work = torch.empty(sar.sar_batch_workspace_bytes(b) // 8 + 1, dtype=torch.complex64, device="cuda")
        torch.cuda.synchronize()
        for _ in range(2):
            sar.sar_batch_execute(b, raws, imgs, work, stream)
            torch.cuda.synchronize()
            for s, im, w in zip(scenes, imgs, want):
                assert np.array_equal(host(im).view(np.uint32), w), s
                im.zero_()
            torch.cuda.synchronize()
    finally:
        torch.cuda.synchronize()
        sar.sar_batch_destroy(b)
