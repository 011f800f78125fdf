"""sar_time_next_launches counts the kernels of the fused schedule, with its
corner turns, whether they run or not: every armed pair is recorded by its own
call, in order, and none is left for the next."""
import numpy as np
import pytest

import paper_2604_03585_amd as sar
from gpu_util import dev, host, rand_c64, torch_cuda
from sarsim import config

pytestmark = pytest.mark.gpu

# (model, schedule, transpose_back, pairs, which of them are a corner turn)
PLANS = [("lfm", "fused", 0, 3, {1}), ("lfm", "fused", 1, 4, {1, 3}), ("hyperbolic", "fused", 0, 4, {1}),
         ("hyperbolic", "fused", 1, 5, {1, 4}), ("lfm", "turn_free", 0, 2, set()),
         ("hyperbolic", "turn_free", 0, 3, set())]


@pytest.mark.parametrize("model, schedule, back, pairs, turns", PLANS)
@pytest.mark.parametrize("na", [1024, 8192])             # strips, and lines that keep the corner turn
def test_every_pair_is_recorded_once(model, schedule, back, pairs, turns, na):
    if schedule == "turn_free" and na > 4096:
        pytest.skip("the turn-free schedule takes azimuth lines of up to 4096")
    torch = torch_cuda()
    nr = 1024
    if model == "hyperbolic":
        cfg = config("c2", Nr=nr, Na=na, range_len=nr // 4, range_tbp=nr / 8.0)
    else:
        cfg = config("c1", Nr=nr, Na=na, range_len=nr // 4, range_tbp=nr / 8.0, az_len=na // 4, az_tbp=na / 8.0)
    raw = dev(rand_c64(np.random.Generator(np.random.PCG64(na)), (na, nr)))

    def events(n):
        ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(n)]
        for a, b in ev:                                  # torch creates an event at its first record
            a.record()
            b.record()
        return ev

    with sar.Plan(cfg, schedule=schedule, transpose_back=back) as p:
        out = torch.empty(p.image_shape(), dtype=torch.complex64, device="cuda")
        work = torch.empty(p.workspace_bytes, dtype=torch.uint8, device="cuda")
        want = host(p.execute(raw)).view(np.uint32)
        ev, after = events(pairs), events(1)
        torch.cuda.synchronize()
        sar.sar_time_next_launches([a for a, _ in ev + after], [b for _, b in ev + after])
        p.execute(raw, out=out, work=work)
        # the pair behind the call's own is the next launch's
        sar.sar_corner_turn(p.handle, out, work.view(torch.complex64)[:na * nr], *out.shape)
        torch.cuda.synchronize()
        ms = [a.elapsed_time(b) for a, b in ev + after]
        order = [ev[i][1].elapsed_time(ev[i + 1][0]) for i in range(pairs - 1)]
        assert np.array_equal(host(out).view(np.uint32), want)
    print(model, schedule, back, na, [f"{1e3 * m:.1f} us" for m in ms])
    absent = turns - ({4} if model == "hyperbolic" else set()) if na <= 4096 else set()
    assert all(m > 0.001 for i, m in enumerate(ms) if i not in absent), ms
    # two records with nothing between: as far apart as the host takes to place them
    assert all(0.0 <= m < 1.0 for i, m in enumerate(ms) if i in absent), ms
    assert all(o > -0.01 for o in order), order
