"""Rows z and -z together give the bits of rows taken one by one: which of the two
forms a launch takes depends on its size, and detection, batches and half-bin
plans may take the other one."""

import pytest

from paper_1711_10855_amd import synth

pytestmark = pytest.mark.gpu

FORMS = [("fp32", 256, 64, 0), ("fp32", 512, 64, 0), ("fp32", 1024, 128, 0), ("fp32", 2048, 256, 0),
         ("fp32", 4096, 256, 0), ("fp16", 4096, 256, 0), ("fp16", 4096, 256, 1), ("bf16", 4096, 256, 1),
         ("bf16", 4096, 256, 0), ("fp16", 2048, 256, 0)]


@pytest.mark.parametrize("prec,L,m,flags", FORMS)
@pytest.mark.parametrize("zmax", [0.0, 7.0, 16.0])
def test_forms_agree_to_the_bit(gpu, monkeypatch, prec, L, m, flags, zmax):
    import torch
    nbins = 5 * (L - m) + 37
    a = torch.from_numpy(synth.small_random_spectrum(nbins, seed=L)).cuda()
    print(f"pair bits {prec} L={L} flags={flags} zmax={zmax}", flush=True)
    monkeypatch.setenv("FDAS_ZPB", "4")  # a fixed unit size: pairs, where there is a pair form
    with gpu.Plan(zmax, 2.0, m, L, prec, flags) as p:
        pairs = p.convolve(a)
    monkeypatch.delenv("FDAS_ZPB")
    with gpu.Plan(zmax, 2.0, m, L, prec, flags | gpu.FLAG_INTERBIN) as p:  # row by row
        assert torch.equal(p.convolve(a)[0::2], pairs)
    with gpu.Plan(zmax, 2.0, m, L, prec, flags) as p:
        assert torch.equal(p.convolve(a), pairs)
        out = torch.empty_like(pairs)
        p.convolve_batch([a], [zmax], [out])
        assert torch.equal(out, pairs)


@pytest.mark.parametrize("prec,L,m,flags", FORMS)
def test_a_plane_does_not_depend_on_its_length(gpu, prec, L, m, flags):
    """The first bins of spectra of 1 to 600 segments, laid out in every way the
    launch rule has, are the same bits."""
    import torch
    top = 600 if L <= 1024 else 300
    a = torch.from_numpy(synth.small_random_spectrum(top * (L - m), seed=L + 1)).cuda()
    print(f"lengths {prec} L={L} flags={flags}", flush=True)
    with gpu.Plan(33.0, 2.0, m, L, prec, flags) as p:
        whole = p.convolve(a)
        for nseg in (1, 2, 3, 5, 8, 13, 21, 34, 55, 89, 144, 233, 377):
            if nseg < top:
                # (whole segments: the end of a shorter spectrum is no zero padding of the longer)
                keep = (nseg - 1) * (L - m)
                assert torch.equal(p.convolve(a[: nseg * (L - m)].clone())[:, :keep], whole[:, :keep])
