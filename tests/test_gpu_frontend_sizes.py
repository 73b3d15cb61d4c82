"""The device front end at every length whose kernels or launch shape differ
(the element counts per thread, the row and column tiles, the one-kernel
select of short spectra), and its median select on powers that are all equal
or mostly zero, against the FP64 oracle."""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def run(gpu, x, in_place=False):
    import torch
    d = torch.from_numpy(x).cuda()
    stats = torch.zeros(2, dtype=torch.float32, device="cuda")
    with gpu.FrontEnd(x.size) as fe:
        out = fe(d, out=d.view(torch.complex64) if in_place else None, stats=stats)
        return out.cpu().numpy(), stats.cpu().numpy()


@pytest.mark.parametrize("lg,in_place", [(7, True), (12, False), (13, True), (14, True), (15, False),
                                         (16, True), (17, False), (18, True), (19, False), (20, True),
                                         (21, False), (22, True), (23, False), (24, True)])
def test_every_length(gpu, lg, in_place):
    n = 1 << lg
    x = np.random.default_rng(lg).standard_normal(n).astype(np.float32)
    x += (3.0 * np.cos(2 * np.pi * 0.0613 * np.arange(n))).astype(np.float32)
    print(f"front end 2^{lg}", flush=True)
    a, st = run(gpu, x, in_place)
    ref, med = oracle.spectrum64(x.astype(np.float64))
    err = np.max(np.abs(a - ref))
    # the bars of the other lengths: FP32 transforms of unit-power spectra
    assert err <= 1e-5 * np.max(np.abs(ref)) and a[0] == 0
    assert abs(st[1] - med) <= 1e-5 * med


@pytest.mark.parametrize("lg", [10, 15, 19, 21])
@pytest.mark.parametrize("kind", ["impulse", "tone"])
def test_select_on_ties(gpu, lg, kind):
    """An impulse at sample 0 has |A| = 1 in every bin, to the last bit (each
    butterfly adds zeros): the median is that of M - 1 equal powers. A tone on
    a bin leaves the others at the transform's rounding."""
    n = 1 << lg
    x = np.zeros(n, dtype=np.float32)
    if kind == "impulse":
        x[0] = 2.0
    else:
        x[:] = np.cos(2 * np.pi * ((np.arange(n) * 5) % n) / n)
    print(f"front end ties 2^{lg} {kind}", flush=True)
    a, st = run(gpu, x)
    ref, med = oracle.spectrum64(x.astype(np.float64))
    if kind == "impulse":
        assert st[1] == 4.0 and np.max(np.abs(a - ref)) <= 1e-6
    else:
        power = np.sort((np.abs(a[1:].astype(np.complex128)) / st[0]) ** 2)
        assert abs(st[1] - power[power.size // 2]) <= 1e-5 * power[power.size // 2]
