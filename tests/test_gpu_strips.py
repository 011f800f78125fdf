"""The schedules without a corner turn against the same scene step by step
(range compression, corner turn, azimuth compression): the column tiles and
strips move the same samples through the same butterflies, so the images are
equal bit for bit.  Every range line length (stores into tiles) meets every
azimuth line length (strip widths) somewhere in the list."""
import numpy as np
import pytest

import paper_2604_03585_amd as sar
from gpu_util import host, torch_cuda
from sarsim import config

pytestmark = pytest.mark.gpu

SHAPES = [(64, 64), (64, 128), (64, 4096), (128, 64), (128, 256), (256, 512), (256, 8192), (512, 64),
          (512, 1024), (512, 2048), (512, 4096), (1024, 64), (1024, 256), (1024, 2048), (2048, 128), (2048, 4096), (4096, 64),
          (4096, 512), (8192, 64), (8192, 1024), (8192, 2048), (16384, 64), (16384, 128), (16384, 512)]


def scene(nr, na, model):
    if model == "hyperbolic":
        cfg = config("c2", Nr=nr, Na=na, range_len=nr // 4, range_tbp=nr / 8.0)
    else:
        cfg = config("c1", Nr=nr, Na=na, range_len=nr // 4, range_tbp=nr / 8.0, az_len=na // 4,
                     az_tbp=na / 8.0)
    torch = torch_cuda()
    g = torch.Generator(device="cuda").manual_seed(nr + 3 * na)
    x = torch.empty((na, nr, 2), dtype=torch.float32, device="cuda")
    return cfg, torch.view_as_complex(x.normal_(0.0, 1.0, generator=g))


def by_steps(cfg, raw):
    torch = torch_cuda()
    na, nr = raw.shape
    with sar.Plan(cfg) as p:
        a, b, w = (torch.empty(na * nr, dtype=torch.complex64, device="cuda") for _ in range(3))
        sar.sar_range_compress(p.handle, raw, a)
        sar.sar_corner_turn(p.handle, a, b, na, nr)
        sar.sar_azimuth_compress(p.handle, b, a, w)
        return host(a.view(nr, na))


@pytest.mark.parametrize("nr, na", SHAPES)
@pytest.mark.parametrize("model", ["lfm", "hyperbolic"])
def test_turn_free_equals_steps(nr, na, model):
    if na > 4096:
        pytest.skip("the turn-free schedule takes azimuth lines of up to 4096")
    cfg, raw = scene(nr, na, model)
    want = by_steps(cfg, raw)
    with sar.Plan(cfg, schedule="turn_free") as p:
        got = host(p.execute(raw))
    assert np.array_equal(got.view(np.uint32), want.view(np.uint32))


@pytest.mark.parametrize("nr, na", SHAPES)
@pytest.mark.parametrize("model", ["lfm", "hyperbolic"])
@pytest.mark.parametrize("back", [0, 1])
def test_fused_equals_steps(nr, na, model, back):
    """The fused schedule drops its corner turn(s) where the strips cover the
    plan (azimuth lines of up to 4096), with and without the back-turn."""
    cfg, raw = scene(nr, na, model)
    want = by_steps(cfg, raw)
    with sar.Plan(cfg, transpose_back=back) as p:
        got = host(p.execute(raw))
    want = np.ascontiguousarray(want.T) if back else want
    assert np.array_equal(got.view(np.uint32), want.view(np.uint32))
