"""A cached choice of the autotuner for a plain plan is not taken for a half-bin
plan of as many rows, which runs other kernels, nor the other way round."""

import numpy as np
import pytest

import oracle
from paper_1711_10855_amd import synth

pytestmark = pytest.mark.gpu


def test_tune_cache_separates_half_bin_rows(gpu, tmp_path, monkeypatch):
    import torch
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("FDAS_TUNE_CACHE", str(cache))
    monkeypatch.delenv("FDAS_VARIANT", raising=False)
    a = synth.small_random_spectrum(3000, seed=31)
    spec = torch.from_numpy(a).cuda()
    for n, (zmax, flags) in enumerate([(7.0, 0), (3.0, gpu.FLAG_INTERBIN)], 1):  # 8 rows each
        print(f"autotune zmax={zmax} flags={flags}", flush=True)
        for _ in range(2):  # tuned, then from the cache
            with gpu.Plan(zmax, 2.0, 64, 512, "fp32", gpu.FLAG_AUTOTUNE | flags) as p:
                assert p.nz == 8
                out = p.convolve(spec).cpu().numpy()
            assert len(cache.read_text().splitlines()) == n
        if not flags:
            ref = oracle.plane_direct(a, zmax, 2.0, 64)
            assert np.max(np.abs(out - ref)) <= 1e-4 * ref.max()
    # a line written for a plain plan keeps its key
    assert cache.read_text().splitlines()[0].split(" | ")[0].endswith(" m64 nz8 prec0 split0 L512")
