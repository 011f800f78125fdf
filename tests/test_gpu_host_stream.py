"""The binding's way to the current stream, and Plan.execute with and without
torch's stream context: the same stream handles, and the same image whichever
way the stream, the image and the workspace are given."""
import threading

import numpy as np
import pytest
import torch

import paper_2604_03585_amd as sar
from gpu_util import dev, empty, host, rand_c64
from paper_2604_03585_amd import _lib
from sarsim import config

pytestmark = pytest.mark.gpu


def test_current_stream_handle():
    torch.cuda.init()
    side = torch.cuda.Stream()
    assert _lib._stream(None) == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert _lib._stream(None) == side.cuda_stream
        seen = []                                   # another thread has its own current stream
        t = threading.Thread(target=lambda: seen.append(
            (_lib._stream(None), torch.cuda.current_stream().cuda_stream)))
        t.start()
        t.join()
        assert seen[0][0] == seen[0][1] != side.cuda_stream
    assert _lib._stream(None) == torch.cuda.current_stream().cuda_stream


@pytest.mark.parametrize("back", [0, 1])
def test_execute_same_image_every_way(back):
    cfg = config("c1", Nr=256, Na=128, range_len=64, range_tbp=32.0, az_len=32, az_tbp=16.0)
    rng = np.random.Generator(np.random.PCG64(11))
    raw = dev(rand_c64(rng, (128, 256)))
    side = torch.cuda.Stream()
    with sar.Plan(cfg, transpose_back=back) as p:
        ref = host(p.execute(raw)).view(np.uint32)
        torch.cuda.synchronize()
        for stream in (None, side, side.cuda_stream):
            for given in (True, False):
                out = empty(p.image_shape()) if given else None
                work = torch.empty(p.workspace_bytes, dtype=torch.uint8, device=raw.device) if given else None
                torch.cuda.synchronize()
                got = p.execute(raw, out=out, work=work, stream=stream)
                if given:
                    assert got is out
                side.synchronize()
                assert np.array_equal(host(got).view(np.uint32), ref)
        with torch.cuda.stream(side):
            out, work = empty(p.image_shape()), torch.empty(p.workspace_bytes, dtype=torch.uint8,
                                                            device=raw.device)
            got = p.execute(raw, out=out, work=work)
        side.synchronize()
        assert np.array_equal(host(got).view(np.uint32), ref)
        for bad in (raw.reshape(256, 128), raw.real, raw.cpu()):
            with pytest.raises(ValueError):
                p.execute(bad, out=out, work=work)
        with pytest.raises(ValueError):
            p.execute(raw, out=out, work=work[:-1])
        with pytest.raises(ValueError):
            p.execute(raw, out=out[:1], work=work)
