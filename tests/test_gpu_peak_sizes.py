"""The peak search at numbers of candidates from none to more than a block's,
in workspaces that just hold them and larger ones. It decides on the FP32
powers of the plane, so the peaks equal the oracle's rule on that plane."""

import numpy as np
import pytest

import oracle
from paper_1711_10855_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flags", [0, 4])
@pytest.mark.parametrize("count", [0, 1, 255, 256, 257, 4097, 20000])
def test_peaks_of_a_given_number_of_candidates(gpu, count, flags):
    import torch
    a = torch.from_numpy(synth.small_random_spectrum(9000, seed=92)).cuda()
    with gpu.Plan(16.0, 2.0, 64, 512, "fp32", flags) as p:
        plane = p.convolve(a).cpu().numpy()
        powers = np.sort(plane, axis=None)[::-1]
        thr = float(powers[count - 1]) if count else float(powers[0]) * 2
        n = int(np.count_nonzero(plane >= thr))
        want_row, want_r, _ = oracle.peaks_from_plane(plane.astype(np.float64), thr,
                                                      bool(flags & gpu.FLAG_INTERBIN))
        want = sorted(zip(want_row.tolist(), want_r.tolist()))
        for cap in sorted({n, n + 1, 1 << 16}):
            buf = p.peaks(a, thr, cap, 1 << 14)
            for _ in range(2):            # a used workspace gives the same again
                row, r, pw, n_cand, n_peak = gpu.decode_peaks(buf[0], buf[1])
                assert (n_cand, n_peak) == (n, len(want)), cap
                assert sorted(zip(row.tolist(), r.tolist())) == want, cap
                assert np.array_equal(pw, plane[row, r])
                buf = p.peaks(a, thr, buf=buf)
