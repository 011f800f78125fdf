"""Tuned variants of the line kernels leave the schedule alone: a plan or batch
that runs in strips does so whatever is tuned, with the same bits, whether one of
its line lengths or kinds has table twiddles or all; and a batch computes what
each of its scenes computes alone."""
import json

import numpy as np
import pytest

import paper_2604_03585_amd as sar
from gpu_util import dev, host, rand_c64, torch_cuda
from sarsim import config

pytestmark = pytest.mark.gpu


def arch():
    return torch_cuda().cuda.get_device_properties(0).gcnArchName.split(":")[0]


def load(path, entries):
    path.write_text("".join(json.dumps(dict(arch=arch(), kind=k, n=n, prec=0, variant=v)) + "\n"
                            for k, n, v in entries))
    sar.sar_tune_load(str(path))


@pytest.fixture(autouse=True)
def clear_table():
    yield
    sar.sar_tune_load(None)


def scene(na, nr, model="lfm"):
    if model == "hyperbolic":
        return config("c2", Nr=nr, Na=na, range_len=nr // 4, range_tbp=nr / 8.0)
    return config("c1", Nr=nr, Na=na, range_len=nr // 4, range_tbp=nr / 8.0, az_len=na // 4, az_tbp=na / 8.0)


def image(cfg, raw, **opt):
    with sar.Plan(cfg, **opt) as p:
        return host(p.execute(raw)).view(np.uint32)


@pytest.mark.parametrize("na, nr, model", [(256, 512, "lfm"), (1024, 2048, "lfm"), (4096, 512, "lfm"),
                                           (512, 1024, "hyperbolic"), (4096, 256, "hyperbolic")])
@pytest.mark.parametrize("which", ["range", "azimuth", "all"])
def test_strips_whatever_is_tuned(tmp_path, na, nr, model, which):
    cfg = scene(na, nr, model)
    rng = np.random.Generator(np.random.PCG64(na + nr))
    raw = dev(rand_c64(rng, (na, nr)))
    want = image(cfg, raw)
    n = {"range": [nr], "azimuth": [na], "all": [na, nr]}[which]
    load(tmp_path / "t.jsonl", [(k, m, 1) for k in ("fused", "fwd", "inv", "batch_fused") for m in n])
    for schedule in ("fused", "turn_free"):
        assert np.array_equal(image(cfg, raw, schedule=schedule), want), schedule


BATCH = [(256, 512, {}), (1024, 256, {"transpose_back": 1}), (512, 256, {"transpose_back": 1}), (64, 256, {}), (256, 256, {"transpose_back": 1}),
         (2048, 256, {}), (8192, 128, {}), (512, 512, {})]
# (back-turned scenes, 64-point and 8192-point lines take the line and turn launches)


@pytest.mark.parametrize("kinds", [("fused",), ("batch_fused",), ("fused", "batch_fused")])
@pytest.mark.parametrize("variant", [0, 1, 4, 5, 8, 9, 12, 13])
def test_batch_equals_single_scenes(tmp_path, kinds, variant):
    torch = torch_cuda()
    lengths = sorted({n for s in BATCH for n in s[:2]})
    # bits 2 and 3 are the batch's grid; "fused" has bit 0 and, up to 8192 points, bit 2
    load(tmp_path / "t.jsonl", [(k, n, variant if k == "batch_fused" else variant & 5) for k in kinds for n in lengths])
    rng = np.random.Generator(np.random.PCG64(variant))
    raws = [dev(rand_c64(rng, s[:2])) for s in BATCH]
    cfgs = [scene(*s[:2]) for s in BATCH]
    want = [image(c, r, **s[2]) for c, r, s in zip(cfgs, raws, BATCH)]
    stream = torch.cuda.Stream()
    b = sar.sar_batch_plan([sar.make_params(c, **s[2]) for c, s in zip(cfgs, BATCH)], stream)
    try:
        imgs = [torch.zeros(w.shape[:1] + (w.shape[1] // 2,), dtype=torch.complex64, device="cuda") for w in want]
        work = torch.empty(sar.sar_batch_workspace_bytes(b) // 8 + 1, dtype=torch.complex64, device="cuda")
        torch.cuda.synchronize()
        sar.sar_batch_execute(b, raws, imgs, work, stream)
        torch.cuda.synchronize()
        for s, i, w in zip(BATCH, imgs, want):
            assert np.array_equal(host(i).view(np.uint32), w), s
    finally:
        torch.cuda.synchronize()
        sar.sar_batch_destroy(b)
