"""The stores of segments narrower than a wave (256 points), through the L2 and
past it: planes on both sides of the sizes and alignments between the two, with
guard columns, equal to the bit."""

import numpy as np
import pytest

from paper_1711_10855_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,flags", [(64, 0), (64, 4), (50, 0)])
@pytest.mark.parametrize("nbins", [12000, 61440, 61695, 300001])
def test_both_stores_write_the_same_plane(gpu, m, flags, nbins):
    """17 or 34 rows: 61695 bins are 4 MB, 300001 more than 18 MB."""
    import torch
    a = torch.from_numpy(synth.small_random_spectrum(nbins, seed=nbins)).cuda()
    print(f"narrow stores m={m} flags={flags} nbins={nbins}", flush=True)
    with gpu.Plan(16.0, 2.0, m, 256, "fp32", flags) as p:
        ref = None
        for pad in (-nbins % 16 + 16, -nbins % 16 + 17, -nbins % 16 + 18, -nbins % 16 + 24):
            for shift in (0, 1, 16):
                buf = torch.full((p.nz * (nbins + pad) + 64,), -7.0, dtype=torch.float32, device="cuda")
                out = buf[shift: shift + p.nz * (nbins + pad)].view(p.nz, nbins + pad)
                p.convolve(a, out=out)
                assert bool((buf[:shift] == -7.0).all()) and bool((buf[shift + out.numel():] == -7.0).all())
                assert bool((out[:, nbins:] == -7.0).all())
                ref = out[:, :nbins].clone() if ref is None else ref
                assert torch.equal(out[:, :nbins], ref)
                outs = [torch.full_like(out, -7.0)]
                p.convolve_batch([a], [16.0], outs)
                assert torch.equal(outs[0], out)
        assert np.isfinite(ref.cpu().numpy()).all()
