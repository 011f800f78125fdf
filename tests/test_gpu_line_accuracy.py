"""Rounding error of the FP32 line transforms against 64 bits, at every line
length and in both twiddle schemes.  The bound is the error of the transform
that multiplies the twiddles in ahead of every butterfly (radix-16 Stockham
passes; w^1 and w^4 of a radix-16 pass from a table rounded to FP32 and the
other powers as products, a smaller last pass wholly from the table; with the
table scheme all of them): relative L2 of 2^21 points of Gaussian noise, from a
model of its FP32 operations on a CPU, and half a percent more for another
sample of the noise."""
import json

import numpy as np
import pytest

import paper_2604_03585_amd as sar
from gpu_util import host, torch_cuda

pytestmark = pytest.mark.gpu

PRODUCTS = {64: 8.113e-8, 128: 8.880e-8, 256: 1.151e-7, 512: 1.210e-7, 1024: 1.257e-7,
            2048: 1.324e-7, 4096: 1.530e-7, 8192: 1.580e-7, 16384: 1.615e-7}
TABLE = {64: 8.113e-8, 128: 8.880e-8, 256: 9.667e-8, 512: 1.039e-7, 1024: 1.092e-7,
         2048: 1.164e-7, 4096: 1.236e-7, 8192: 1.296e-7, 16384: 1.337e-7}


@pytest.fixture(autouse=True)
def clear_table():
    yield
    sar.sar_tune_load(None)


@pytest.mark.parametrize("n", sorted(PRODUCTS))
@pytest.mark.parametrize("inverse", [0, 1])
@pytest.mark.parametrize("table", [0, 1])
def test_line_error_against_64_bits(tmp_path, n, inverse, table):
    torch = torch_cuda()
    if table:
        arch = torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]
        path = tmp_path / "t.jsonl"
        path.write_text(json.dumps({"arch": arch, "kind": "inv" if inverse else "fwd", "n": n,
                                    "prec": 0, "variant": 1}) + "\n")
        sar.sar_tune_load(str(path))
    lines = (1 << 21) // n
    rng = np.random.Generator(np.random.PCG64(n + inverse))
    x = rng.standard_normal((lines, 2 * n), dtype=np.float32).view(np.complex64)
    cfg = dict(Nr=n, Na=64, range_len=n // 4, range_tbp=n / 8.0, az_model="lfm", az_len=16, az_tbp=8.0,
               lam=0.0, v=0.0, r_near=0.0, rcmc_taps=0, rcmc_beta=2.5)
    out = torch.empty((lines, n), dtype=torch.complex64, device="cuda")
    with sar.Plan(cfg) as p:
        sar.sar_fft_lines(p.handle, 0, inverse, torch.from_numpy(x).to("cuda"), out, lines)
        got = host(out).astype(np.complex128)
    ref = (np.fft.ifft if inverse else np.fft.fft)(x.astype(np.complex128), axis=1)
    err = np.sqrt((np.abs(got - ref) ** 2).sum() / (np.abs(ref) ** 2).sum())
    bound = (TABLE if table else PRODUCTS)[n] * 1.005
    print(f"n {n} {'table' if table else 'products'}: {err:.4e} (bound {bound:.4e})")
    assert err <= bound
