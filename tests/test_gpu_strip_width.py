"""The autotuner times strip widths only for scenes whose number of range cells
leaves the width open, so that a narrow scene's measurement (of one kernel against
itself) decides nothing for a wide one; and the half width gives the default one's
image at every line length with range cells enough for it, that of the same scene
step by step."""
import json

import numpy as np
import pytest

import paper_2604_03585_amd as sar
from gpu_util import dev, host, rand_c64, torch_cuda
from paper_2604_03585_amd import _lib
from sarsim import config

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def clear_table():
    yield
    sar.sar_tune_load(None)


@pytest.mark.parametrize("na, nr, open_", [(1024, 1024, False), (1024, 2048, True), (4096, 512, False)])
def test_strip_width_is_tuned_where_it_is_open(tmp_path, na, nr, open_):
    cfg = config("c1", Nr=nr, Na=na, range_len=nr // 4, range_tbp=nr / 8.0, az_len=na // 4, az_tbp=na / 8.0)
    path = tmp_path / "t.jsonl"
    sar.sar_autotune(sar.make_params(cfg, schedule="turn_free"), str(path))
    kinds = {json.loads(l)["kind"] for l in path.read_text().splitlines()}
    assert ("strip" in kinds) == open_
    assert sar.sar_tune_variant(_lib.TUNE_STRIP, na, 0) in ((0, 1) if open_ else (0,))


@pytest.mark.parametrize("na, nr", [(64, 4096), (128, 2048), (256, 2048), (512, 2048), (1024, 2048), (2048, 2048),
                                    (4096, 1024)])
@pytest.mark.parametrize("back", [0, 1])
def test_half_width_same_image(tmp_path, na, nr, back):
    cfg = config("c1", Nr=nr, Na=na, range_len=nr // 4, range_tbp=nr / 8.0, az_len=na // 4, az_tbp=na / 8.0)
    raw = dev(rand_c64(np.random.Generator(np.random.PCG64(na + nr)), (na, nr)))
    with sar.Plan(cfg) as p:
        a, b, w = (torch_cuda().empty(na * nr, dtype=raw.dtype, device=raw.device) for _ in range(3))
        sar.sar_range_compress(p.handle, raw, a)
        sar.sar_corner_turn(p.handle, a, b, na, nr)
        sar.sar_azimuth_compress(p.handle, b, a, w)
        steps = host(a.view(nr, na))
    want = np.ascontiguousarray(steps.T if back else steps).view(np.uint32)
    for v in (0, 1):
        arch = torch_cuda().cuda.get_device_properties(0).gcnArchName.split(":")[0]
        path = tmp_path / f"v{v}.jsonl"
        path.write_text(json.dumps(dict(arch=arch, kind="strip", n=na, prec=0, variant=v)) + "\n")
        sar.sar_tune_load(str(path))
        with sar.Plan(cfg, transpose_back=back) as p:
            assert np.array_equal(host(p.execute(raw)).view(np.uint32), want), v
