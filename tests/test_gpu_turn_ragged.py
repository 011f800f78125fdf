"""Corner turns of shapes that are not whole 64 x 64 tiles: both tile heights
(also by the output's alignment), the last tiles of both axes, single rows and
columns.  Bytes move unchanged, so equality is
exact, and nothing outside the output is written."""
import numpy as np
import pytest
import torch

import paper_2604_03585_amd as sar

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1), (1, 257), (257, 1), (8, 64), (63, 65), (64, 63), (72, 130), (127, 64), (128, 65),
          (129, 127), (136, 192), (191, 129), (255, 256), (257, 320), (1000, 777), (1001, 640)]


def turn_guarded(rows, cols, off_in, off_out):
    rng = np.random.Generator(np.random.PCG64(rows * 4099 + cols))
    x = rng.integers(0, 2**32, (rows, 2 * cols), dtype=np.uint32)      # NaN patterns included
    src = torch.zeros(rows * cols + off_in, dtype=torch.complex64, device="cuda:0")
    src.view(torch.int32)[2 * off_in:] = torch.from_numpy(x.view(np.int32).reshape(-1)).to("cuda:0")
    guard = 512
    dst = torch.zeros(rows * cols + off_out + guard, dtype=torch.complex64, device="cuda:0")
    dst.view(torch.int32).fill_(0x5A5A5A5A)
    sar.sar_corner_turn(0, src[off_in:], dst[off_out:], rows, cols)
    got = dst.view(torch.int32).cpu().numpy().view(np.uint32).reshape(-1, 2)
    ref = x.reshape(rows, cols, 2).transpose(1, 0, 2).reshape(-1, 2)
    assert np.array_equal(got[off_out:off_out + rows * cols], ref)
    assert (got[:off_out] == 0x5A5A5A5A).all() and (got[off_out + rows * cols:] == 0x5A5A5A5A).all()


@pytest.mark.parametrize("rows,cols", SHAPES)
def test_ragged_turn_exact(rows, cols):
    turn_guarded(rows, cols, 0, 0)


@pytest.mark.parametrize("off_in,off_out", [(2, 0), (0, 2), (2, 6), (0, 8)])
@pytest.mark.parametrize("rows,cols", [(64, 128), (192, 65), (200, 136)])
def test_turn_at_16_byte_boundaries(rows, cols, off_in, off_out):
    turn_guarded(rows, cols, off_in, off_out)
