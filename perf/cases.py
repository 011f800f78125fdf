"""Performance cases: the work that programs have this library do, through
its public entry points, each pass as a caller would issue it with a plan and
buffers it keeps.

A case is a dict of plain values; ``kind`` names the entry point:

* ``scene``   a whole RDA scene, ``Plan.execute`` (``Na`` x ``Nr``, azimuth
  model, precision, schedule, back-turn);
* ``batch``   uneven LFM scenes in one ``sar_batch_execute`` (replayed on a
  stream of the caller's);
* ``range``   range compression of a scene, ``sar_range_compress``;
* ``azimuth`` azimuth compression of turned data, ``sar_azimuth_compress``;
* ``fft``     line FFTs, ``sar_fft_lines`` (any number of lines);
* ``turn``    a corner turn of any shape, ``sar_corner_turn``.

Inputs are point-target echoes in 20 dB noise (scenes) or complex noise with
a chirp in every line (single steps), generated on the device from the seed.
"""
import math
import random

import torch

import paper_2604_03585_amd as sar

SIGMA2 = 10.0 ** (-20.0 / 10.0)         # per-sample noise power of a 20 dB scene
# Normalised hyperbolic geometry: at most 8 cells of migration at near range.
LAM, VEL, R_NEAR, BETA = 5.0 / 32.0, math.sqrt(2.0), 32768.0, 2.5


def _scene(name, Na, Nr, az="lfm", precision="fp32", schedule="fused", back=0, targets=5,
           range_len=0, az_len=0):
    return dict(name=name, kind="scene", Na=Na, Nr=Nr, az=az, precision=precision,
                schedule=schedule, back=back, targets=targets,
                range_len=range_len or Nr // 8, az_len=az_len or Na // 8)


def listed():
    return [
        # the smallest scene that is used: a 256 x 256 chip, three short launches
        _scene("scene_256_lfm", 256, 256, range_len=64, az_len=64),
        # an ordinary served scene, and its image turned back to [Na][Nr]
        _scene("scene_1024x2048_lfm_back", 1024, 2048, back=1),
        # the paper's scene size, without and with the corner turn (the default)
        _scene("scene_4096_hyp_turn_free", 4096, 4096, az="hyperbolic", schedule="turn_free",
               range_len=512, az_len=1024),
        _scene("scene_8192x4096_hyp", 8192, 4096, az="hyperbolic", range_len=512, az_len=1024),
        # the same scene size with FP16 intermediates and with split FP16 butterflies
        _scene("scene_4096_hyp_halfstore", 4096, 4096, az="hyperbolic",
               precision="fp32_halfstore", range_len=512, az_len=1024),
        _scene("scene_4096_hyp_split_fp16", 4096, 4096, az="hyperbolic",
               precision="split_fp16", range_len=512, az_len=1024),
        # the largest scene of a serving pool: longest range lines
        _scene("scene_8192x16384_lfm", 8192, 16384),
        # a burst of small uneven scenes that share launches
        dict(name="batch_24_small", kind="batch", scenes=24, sizes=4, max_log=10),
        # one step of a step-by-step program: azimuth FFT, RCMC and IFFT of
        # turned data
        dict(name="azimuth_1024x2048_hyp", kind="azimuth", Na=2048, Nr=1024, az="hyperbolic"),
        # line FFTs: the paper's batch of 256 lines of 4096, and an inverse
        # over a ragged number of shorter lines
        dict(name="fft_256x4096_fwd", kind="fft", n=4096, lines=256, inverse=0,
             precision="fp32"),
        dict(name="fft_3001x1024_inv", kind="fft", n=1024, lines=3001, inverse=1,
             precision="fp32"),
        # a corner turn of a matrix that is no multiple of any tile
        dict(name="turn_3000x5001", kind="turn", rows=3000, cols=5001),
    ]


def _pow2(rng, lo, hi):
    return 1 << rng.randint(lo, hi)


def draw(rng):
    """One more case of the same ranges: sizes spread over their logarithm,
    chirp lengths, target counts, line counts and turn shapes at random."""
    kind = rng.choice(["scene", "scene", "scene", "scene", "batch", "range", "azimuth", "fft",
                       "fft", "turn"])
    if kind == "scene":
        Na, Nr = _pow2(rng, 7, 13), _pow2(rng, 7, 14)
        az = rng.choice(["lfm", "hyperbolic"])
        if az == "hyperbolic" and Nr < 512:
            Nr = 512
        precision = rng.choice(["fp32", "fp32", "fp32", "fp32_halfstore", "split_fp16",
                                "split_bf16"])
        schedule = "fused"
        if precision == "fp32" and Na <= 4096:
            schedule = rng.choice(["fused", "turn_free"])
        back = rng.choice([0, 0, 0, 1]) if schedule == "fused" and precision == "fp32" else 0
        if az == "hyperbolic" and Na * Nr > 1 << 25:
            Nr //= 4
        c = _scene("", Na, Nr, az=az, precision=precision, schedule=schedule, back=back,
                   targets=rng.randint(3, 9), range_len=rng.randint(Nr // 16, Nr // 4),
                   az_len=rng.randint(Na // 16, Na // 4))
        del c["name"]
        return c
    if kind == "batch":
        return dict(kind="batch", scenes=rng.randint(3, 40), sizes=rng.randint(1, 10 ** 6),
                    max_log=rng.randint(8, 11))
    if kind in ("range", "azimuth"):
        Na, Nr = _pow2(rng, 7, 13), _pow2(rng, 9, 13)
        az = "lfm" if kind == "range" else rng.choice(["lfm", "hyperbolic"])
        return dict(kind=kind, Na=Na, Nr=Nr, az=az, range_len=rng.randint(Nr // 16, Nr // 4),
                    az_len=rng.randint(Na // 16, Na // 4))
    if kind == "fft":
        n = _pow2(rng, 6, 14)
        lines = int(2.0 ** rng.uniform(2.0, 25.0 - math.log2(n))) + 1
        return dict(kind="fft", n=n, lines=lines, inverse=rng.randint(0, 1),
                    precision=rng.choice(["fp32", "fp32", "fp32", "split_fp16", "split_bf16"]))
    return dict(kind="turn", rows=int(2.0 ** rng.uniform(5.0, 13.0)),
                cols=int(2.0 ** rng.uniform(5.0, 13.0)))


# ------------------------------------------------------------------ inputs
def _params(case):
    """The processing parameters (a scene dictionary) of a case."""
    Na, Nr = case["Na"], case["Nr"]
    Lr = case.get("range_len") or Nr // 8
    La = case.get("az_len") or Na // 8
    hyper = case.get("az") == "hyperbolic"
    return dict(Nr=Nr, Na=Na, range_len=Lr, range_tbp=Lr / 2.0,
                az_model="hyperbolic" if hyper else "lfm", az_len=La, az_tbp=La / 2.0,
                lam=LAM if hyper else 0.0, v=VEL if hyper else 0.0,
                r_near=R_NEAR if hyper else 0.0, rcmc_taps=8 if hyper else 0, rcmc_beta=BETA)


def _batch_shapes(case):
    """(Na, Nr) of a batch's scenes, drawn from the case alone."""
    rng = random.Random(case["sizes"])
    return [(_pow2(rng, 7, case["max_log"]), _pow2(rng, 7, case["max_log"]))
            for _ in range(case["scenes"])]


def _noise(gen, rows, cols, power):
    x = torch.empty((rows, cols, 2), dtype=torch.float32, device="cuda")
    x.normal_(0.0, math.sqrt(power / 2.0), generator=gen)
    return torch.view_as_complex(x)


def _turns(x):
    """exp(2 pi i x) in 64 bits, x reduced to turns."""
    x = (x - torch.floor(x)) * (2.0 * math.pi)
    return torch.complex(torch.cos(x), torch.sin(x))


def _centred(length):
    return torch.arange(length, dtype=torch.float64, device="cuda") - float(length // 2)


def _echo(p, seed, targets):
    """The raw echo [Na][Nr] (complex64) of unit point targets in noise."""
    Na, Nr, Lr, La = p["Na"], p["Nr"], p["range_len"], p["az_len"]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    rng = random.Random(seed)
    raw = _noise(gen, Na, Nr, SIGMA2)
    Kr, Ka = p["range_tbp"] / (Lr * Lr), p["az_tbp"] / (La * La)
    for _ in range(targets):
        phase = rng.random()
        m0 = rng.randint(0, Na - La)
        if p["az_model"] == "lfm":
            n0 = rng.randint(0, Nr - Lr)
            a = _turns(-0.5 * Ka * _centred(La) ** 2 + phase)
            r = _turns(0.5 * Kr * _centred(Lr) ** 2)
            raw[m0:m0 + La, n0:n0 + Lr] += torch.outer(a, r).to(torch.complex64)
            continue
        width = min(Nr, Lr + 16)
        n0 = rng.randint(0, Nr - width)
        R0 = R_NEAR + n0 + Lr // 2
        R = torch.sqrt(R0 * R0 + (VEL * _centred(La)) ** 2)
        u = torch.arange(width, dtype=torch.float64, device="cuda")[None, :] + (R_NEAR + n0) - R[:, None]
        a = _turns(-2.0 * R / LAM + phase)[:, None] * _turns(0.5 * Kr * u * u)
        a[(u < -Lr / 2) | (u >= Lr / 2)] = 0.0
        raw[m0:m0 + La, n0:n0 + width] += a.to(torch.complex64)
    return raw


def _lines(seed, rows, n):
    """Lines of complex noise with a chirp across each (single-step input)."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    x = _noise(gen, rows, n, 1.0)
    chirp = _turns(0.25 / n * _centred(n) ** 2).to(torch.complex64)
    shift = torch.rand(rows, generator=gen, device="cuda")
    return x + chirp[None, :] * _turns(shift.double())[:, None].to(torch.complex64)


# ------------------------------------------------------------- preparation
class _State(dict):
    """A case's inputs, buffers and handles; plans go when it goes."""

    def __del__(self):
        torch.cuda.synchronize()
        if "plan" in self:
            self["plan"].close()
        if "batch" in self:
            sar.sar_batch_destroy(self["batch"])


def _empty(*shape):
    return torch.empty(shape, dtype=torch.complex64, device="cuda")


def prepare(case, seed):
    kind = case["kind"]
    s = _State(kind=kind, case=case)
    if kind == "scene":
        p = _params(case)
        s["raw"] = _echo(p, seed, case["targets"])
        s["plan"] = sar.Plan(p, precision=case["precision"], schedule=case["schedule"],
                             transpose_back=case["back"])
        s["img"] = _empty(*s["plan"].image_shape())
        s["work"] = _empty((s["plan"].workspace_bytes + 7) // 8)
    elif kind == "batch":
        s["stream"] = torch.cuda.Stream()
        ps = [_params(dict(Na=na, Nr=nr)) for na, nr in _batch_shapes(case)]
        s["raw"] = [_echo(p, seed + i, 3) for i, p in enumerate(ps)]
        s["img"] = [_empty(p["Nr"], p["Na"]) for p in ps]
        s["batch"] = sar.sar_batch_plan([sar.make_params(p) for p in ps], s["stream"])
        s["work"] = _empty((sar.sar_batch_workspace_bytes(s["batch"]) + 7) // 8)
        s["stream"].wait_stream(torch.cuda.current_stream())
    elif kind in ("range", "azimuth"):
        p = _params(case)
        rows, n = (p["Na"], p["Nr"]) if kind == "range" else (p["Nr"], p["Na"])
        s["plan"] = sar.Plan(p)
        s["in"], s["out"], s["work"] = _lines(seed, rows, n), _empty(rows, n), _empty(rows, n)
    elif kind == "fft":
        n = case["n"]
        s["plan"] = sar.Plan(_params(dict(Na=64, Nr=n)), precision=case["precision"])
        s["in"], s["out"] = _lines(seed, case["lines"], n), _empty(case["lines"], n)
    else:
        s["in"] = _lines(seed, case["rows"], case["cols"])
        s["out"] = _empty(case["cols"], case["rows"])
    return s


# -------------------------------------------------------------------- a pass
def run(s):
    kind = s["kind"]
    if kind == "scene":
        return s["plan"].execute(s["raw"], out=s["img"], work=s["work"])
    if kind == "batch":
        sar.sar_batch_execute(s["batch"], s["raw"], s["img"], s["work"], s["stream"])
        return s["img"]
    if kind == "range":
        sar.sar_range_compress(s["plan"].handle, s["in"], s["out"])
    elif kind == "azimuth":
        sar.sar_azimuth_compress(s["plan"].handle, s["in"], s["out"], s["work"])
    elif kind == "fft":
        sar.sar_fft_lines(s["plan"].handle, 0, s["case"]["inverse"], s["in"], s["out"],
                          s["case"]["lines"])
    else:
        sar.sar_corner_turn(0, s["in"], s["out"], s["case"]["rows"], s["case"]["cols"])
    return s["out"]


# ---------------------------------------------------------------------- work
def _scene_flops(Na, Nr, hyper):
    """Two FFTs per axis at 5 N log2 N, the filter multiplies, and for the
    hyperbolic model eight complex-by-real multiply-adds per pixel."""
    px = Na * Nr
    return px * (10.0 * math.log2(Nr) + 10.0 * math.log2(Na) + 12.0 + (32.0 if hyper else 0.0))


def work(case):
    """Each input sample read once, each output sample written once."""
    kind = case["kind"]
    if kind == "scene":
        return {"bytes": 16.0 * case["Na"] * case["Nr"],
                "flops": _scene_flops(case["Na"], case["Nr"], case["az"] == "hyperbolic")}
    if kind == "batch":
        shapes = _batch_shapes(case)
        return {"bytes": sum(16.0 * a * r for a, r in shapes),
                "flops": sum(_scene_flops(a, r, False) for a, r in shapes)}
    if kind in ("range", "azimuth"):
        px, n = case["Na"] * case["Nr"], case["Nr" if kind == "range" else "Na"]
        return {"bytes": 16.0 * px,
                "flops": px * (10.0 * math.log2(n) + 6.0 +
                               (32.0 if case["az"] == "hyperbolic" else 0.0))}
    if kind == "fft":
        px = case["lines"] * case["n"]
        return {"bytes": 16.0 * px, "flops": px * 5.0 * math.log2(case["n"])}
    return {"bytes": 16.0 * case["rows"] * case["cols"], "flops": 0.0}


# --------------------------------------------------------------------- exact
def _filter(n, length, tbp, sign):
    """conj(DFT) of the circularly centred chirp replica, 64 bits."""
    h = torch.zeros(n, dtype=torch.complex128, device="cuda")
    u = torch.arange(length, device="cuda") - length // 2
    h[u % n] = _turns(sign * 0.5 * (tbp / (length * length)) * u.double() ** 2)
    return torch.fft.fft(h).conj()


def _compress(x, H):
    """FFT, filter, IFFT of every row; rows in chunks, to bound the scratch."""
    out = torch.empty(x.shape, dtype=torch.complex128, device="cuda")
    step = max(1, (1 << 25) // x.shape[1])
    for i in range(0, x.shape[0], step):
        y = torch.fft.fft(x[i:i + step].to(torch.complex128), dim=1)
        out[i:i + step] = torch.fft.ifft(y * H, dim=1)
    return out


def _geometry(Na):
    f = torch.fft.fftfreq(Na, dtype=torch.float64, device="cuda")
    x = LAM * f / (2.0 * VEL)
    D = torch.sqrt(1.0 - x * x)
    return x * x / (D * (1.0 + D)), 2.0 * D / LAM


def _kaiser(z):
    arg = 1.0 - (z / 4.0) ** 2
    w = torch.sinc(z) * torch.special.i0(BETA * torch.sqrt(arg.clamp(min=0.0)))
    return torch.where(arg > 0.0, w, torch.zeros_like(w))


def _azimuth_hyperbolic(x):
    """Azimuth FFT, eight-tap Kaiser-sinc RCMC, exact-geometry phase and IFFT
    of turned data [Nr][Na], 64 bits."""
    Nr, Na = x.shape
    A = torch.fft.fft(x.to(torch.complex128), dim=1)
    stretch, rate = _geometry(Na)
    out = torch.empty_like(A)
    step = max(1, (1 << 23) // Na)
    for i in range(0, Nr, step):
        n = torch.arange(i, min(Nr, i + step), device="cuda")
        R0 = (R_NEAR + n.double())[:, None]
        shift = R0 * stretch[None, :]
        cell = torch.floor(shift)
        frac = shift - cell
        first = n[:, None] + cell.long()
        acc = torch.zeros((len(n), Na), dtype=torch.complex128, device="cuda")
        total = torch.zeros((len(n), Na), dtype=torch.float64, device="cuda")
        for t in range(-3, 5):
            w = _kaiser(float(t) - frac)
            total += w
            row = first + t
            inside = (row >= 0) & (row < Nr)
            acc += torch.where(inside, w, torch.zeros_like(w)) * A.gather(0, row.clamp(0, Nr - 1))
        out[i:i + step] = torch.fft.ifft(acc / total * _turns(R0 * rate[None, :]), dim=1)
    return out


def _image(p, raw, back):
    """The image of a scene in 64 bits: [Nr][Na], or [Na][Nr] turned back."""
    Na, Nr = p["Na"], p["Nr"]
    y = _compress(raw, _filter(Nr, p["range_len"], p["range_tbp"], +1)).T.contiguous()
    if p["az_model"] == "lfm":
        y = _compress(y, _filter(Na, p["az_len"], p["az_tbp"], -1))
    else:
        y = _azimuth_hyperbolic(y)
    return y.T.contiguous() if back else y


def exact(case, seed):
    kind = case["kind"]
    if kind == "scene":
        p = _params(case)
        return _image(p, _echo(p, seed, case["targets"]), case["back"])
    if kind == "batch":
        ps = [_params(dict(Na=na, Nr=nr)) for na, nr in _batch_shapes(case)]
        return [_image(p, _echo(p, seed + i, 3), 0) for i, p in enumerate(ps)]
    if kind == "range":
        p = _params(case)
        x = _lines(seed, p["Na"], p["Nr"])
        return _compress(x, _filter(p["Nr"], p["range_len"], p["range_tbp"], +1))
    if kind == "azimuth":
        p = _params(case)
        x = _lines(seed, p["Nr"], p["Na"])
        if p["az_model"] == "hyperbolic":
            return _azimuth_hyperbolic(x)
        return _compress(x, _filter(p["Na"], p["az_len"], p["az_tbp"], -1))
    if kind == "fft":
        x = _lines(seed, case["lines"], case["n"]).to(torch.complex128)
        return torch.fft.ifft(x, dim=1) if case["inverse"] else torch.fft.fft(x, dim=1)
    return _lines(seed, case["rows"], case["cols"]).to(torch.complex128).T.contiguous()
