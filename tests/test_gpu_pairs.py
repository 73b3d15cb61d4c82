"""Rows z and -z taken together (one bank row for both): numbers of rows with
and without a middle row, unit sizes that leave remainders, rows of no
alignment, and series of a batch with fewer drifts than the plan, against the
FP64 oracle."""

import numpy as np
import pytest

import oracle
from paper_1711_10855_amd import synth

pytestmark = pytest.mark.gpu

# the bars of the precisions, as for every other plane: 1e-4 of the largest
# power in plain FP32, 1e-3 on the matrix cores (flag 1: hi+lo split). The
# widths give m / 2 both a multiple of 4 and not, the row strides no alignment.
FORMS = [("fp32", 256, 64, 0, 1e-4), ("fp32", 512, 64, 0, 1e-4), ("fp32", 1024, 128, 0, 1e-4),
         ("fp32", 2048, 256, 0, 1e-4), ("fp16", 4096, 256, 0, 1e-3), ("fp16", 4096, 50, 0, 1e-3),
         ("fp16", 4096, 128, 1, 1e-3), ("bf16", 4096, 60, 1, 1e-3), ("fp16", 2048, 64, 0, 1e-3),
         ("fp16", 2048, 54, 0, 1e-3)]


def to_dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.complex64)).cuda()


def check(out, ref, nbins, tol):
    assert np.max(np.abs(out[:, :nbins] - ref)) <= tol * ref.max()
    assert np.all(out[:, nbins:] == -7.0)


@pytest.mark.parametrize("prec,L,m,flags,tol", FORMS)
@pytest.mark.parametrize("zmax,zpb", [(0.0, 0), (1.0, 0), (2.0, 1), (3.0, 3), (10.0, 4), (13.0, 5)])
def test_rows_and_units(gpu, monkeypatch, prec, L, m, flags, tol, zmax, zpb):
    """zmax 0, 1, 2, 3, 10, 13 at dz 2: 1, 2, 3, 4, 11, 14 rows."""
    import torch
    if zpb:
        monkeypatch.setenv("FDAS_ZPB", str(zpb))
    nbins = 2 * (L - m) + 37
    a = synth.small_random_spectrum(nbins, seed=L + int(zmax))
    print(f"pairs {prec} L={L} zmax={zmax} zpb={zpb}", flush=True)
    with gpu.Plan(zmax, 2.0, m, L, prec, flags) as p:
        out = torch.full((p.nz, nbins + 3), -7.0, dtype=torch.float32, device="cuda")
        p.convolve(to_dev(a), out=out)
        # the detection form finds exactly the plane's points at its median
        thr = float(out[:, :nbins].median())
        rec = p.candidates(to_dev(a), thr, capacity=p.nz * nbins)
        row, r, power = gpu.decode_candidates(*rec)
        out = out.cpu().numpy()
    check(out, oracle.plane_direct(a, zmax, 2.0, m), nbins, tol)
    assert sorted(zip(row.tolist(), r.tolist())) == list(zip(*np.nonzero(out[:, :nbins] >= thr)))
    assert np.array_equal(power, out[row, r])


@pytest.mark.parametrize("prec,L,m,flags,tol", FORMS)
@pytest.mark.parametrize("persistent,zpb", [("1", 0), ("1", 3), ("0", 2)])
def test_batches(gpu, monkeypatch, prec, L, m, flags, tol, persistent, zpb):
    import torch
    monkeypatch.setenv("FDAS_BATCH_PERSISTENT", persistent)
    if zpb:
        monkeypatch.setenv("FDAS_ZPB", str(zpb))
    specs = [(2 * (L - m) + 11, 13.0), (L - m, 1.0), (L - m + 1, 7.0), (5, 13.0)]
    spectra = [synth.small_random_spectrum(n, seed=40 + k) for k, (n, _) in enumerate(specs)]
    print(f"pairs batch {prec} L={L} persistent={persistent} zpb={zpb}", flush=True)
    with gpu.Plan(13.0, 2.0, m, L, prec, flags) as p:
        outs = [torch.full((int(z) + 1, n + 3), -7.0, dtype=torch.float32, device="cuda")
                for n, z in specs]
        p.convolve_batch([to_dev(a) for a in spectra], [z for _, z in specs], outs)
        outs = [o.cpu().numpy() for o in outs]
    for a, (n, z), o in zip(spectra, specs, outs):
        check(o, oracle.plane_direct(a, z, 2.0, m), n, tol)


@pytest.mark.parametrize("prec,L,m,flags,tol", FORMS)
def test_rows_apart_in_small_launches(gpu, monkeypatch, prec, L, m, flags, tol):
    """On both sides of 256, 512 and 1024 rows of segments, the line of one
    kernel or another between rows apart and pairs: the plane is within twice
    the bar of the one made as pairs, and detection finds its points."""
    import torch
    zmax, rows = 16.0, 17
    for blocks in (256, 512, 1024):
        for nseg in (blocks // rows, blocks // rows + 1):
            nbins = nseg * (L - m) - 3
            a = to_dev(synth.small_random_spectrum(nbins, seed=nseg))
            monkeypatch.delenv("FDAS_ZPB", raising=False)
            with gpu.Plan(zmax, 2.0, m, L, prec, flags) as p:
                out = p.convolve(a)
                thr = float(out.flatten()[:: 7].median()) * 8
                row, r, power = gpu.decode_candidates(*p.candidates(a, thr, capacity=rows * nbins))
            monkeypatch.setenv("FDAS_ZPB", "2")
            with gpu.Plan(zmax, 2.0, m, L, prec, flags) as p:
                pairs = p.convolve(a)
            assert float((out - pairs).abs().max()) <= 2 * tol * float(pairs.max())
            out = out.cpu().numpy()
            assert sorted(zip(row.tolist(), r.tolist())) == list(zip(*np.nonzero(out >= thr)))
            assert np.array_equal(power, out[row, r])
