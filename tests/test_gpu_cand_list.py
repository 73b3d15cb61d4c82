"""Blocks with more candidates than their list holds, in units of many rows, and
a capacity that cuts what they list: the count is exact, and what is stored are
points of the plane at or above the threshold, each once."""

import numpy as np
import pytest

from paper_1711_10855_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,L,m,flags", [
    ("fp32", 256, 64, 0), ("fp32", 256, 64, 4), ("fp32", 1024, 128, 0), ("fp32", 2048, 256, 0),
    ("fp32", 4096, 256, 0), ("fp16", 4096, 256, 0), ("fp16", 4096, 256, 1), ("bf16", 4096, 256, 0),
    ("fp16", 2048, 256, 0)])
@pytest.mark.parametrize("share", [0.02, 0.4, 1.0])
def test_full_lists_and_cut_capacity(gpu, monkeypatch, prec, L, m, flags, share):
    import torch
    zmax, nbins = 100.0, 3 * (L - m) + 17
    monkeypatch.setenv("FDAS_ZPB", "1000")  # every row of a segment in one unit
    a = torch.from_numpy(synth.small_random_spectrum(nbins, seed=L)).cuda()
    print(f"candidate list {prec} L={L} flags={flags} share={share}", flush=True)
    with gpu.Plan(zmax, 2.0, m, L, prec, flags) as p:
        plane = p.convolve(a).cpu().numpy()
        thr = 0.0 if share == 1.0 else float(np.quantile(plane, 1.0 - share))
        want = int(np.count_nonzero(plane >= thr))
        assert want > 320 * 3 or share < 0.1
        for cap in (0, 1, 319, 320, want // 2, want, want + 1000):
            rec, count = p.candidates(a, thr, capacity=cap)
            assert int(count.cpu()[0]) == want, cap
            row, r, power = gpu.decode_candidates(rec, count)
            assert row.size == min(cap, want)
            assert np.array_equal(power, plane[row, r]) and np.all(power >= thr)
            assert np.unique(row * nbins + r).size == row.size
