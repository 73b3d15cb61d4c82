"""The bank sums at the edges of their tiles: one to many rows per wave, taps
under and over a staged tile, the shortest and longest segments, rows at
half-bin offsets, every storage form; and the conjugate rows of z and -z that
the correlation kernels take from one another."""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

# FP32 rounding of the largest value (FP64 sums), and the 16-bit forms' own
TOL = {"fp32": 1.2e-7, "fp16": 2.0 ** -11 * 1.01, "bf16": 2.0 ** -8 * 1.01}


@pytest.mark.parametrize("prec,L,m,zmax,dz,flags", [
    ("fp32", 256, 2, 0.0, 2.0, 0), ("fp32", 256, 254, 3.0, 2.0, 0), ("fp32", 512, 62, 31.0, 2.0, 0),
    ("fp32", 1024, 64, 33.0, 2.0, 4), ("fp32", 4096, 66, 5.0, 0.5, 4), ("fp32", 16384, 130, 3.0, 1.0, 0),
    ("fp16", 4096, 512, 16.0, 2.0, 0), ("fp16", 4096, 34, 7.0, 2.0, 5), ("bf16", 4096, 100, 3.0, 2.0, 0),
    ("fp16", 2048, 256, 9.0, 2.0, 4), ("bf16", 2048, 30, 2.0, 2.0, 0)])
def test_bank_sums(gpu, prec, L, m, zmax, dz, flags):
    interbin = bool(flags & gpu.FLAG_INTERBIN)
    print(f"bank {prec} L={L} m={m} zmax={zmax} flags={flags}", flush=True)
    with gpu.Plan(zmax, dz, m, L, prec, flags) as p:
        bank = p.bank().cpu().numpy()
    _, h = oracle.templates64(zmax, dz, m, interbin)
    ref = oracle.bank_natural(h, m, L)
    tol = TOL["fp32" if flags & gpu.FLAG_SPLIT else prec]
    assert bank.shape == ref.shape
    assert np.max(np.abs(bank.astype(np.complex128) - ref)) <= tol * np.max(np.abs(ref))
    whole = bank[0::2] if interbin else bank
    assert np.array_equal(whole, whole[::-1].conj())


@pytest.mark.parametrize("m", [34, 130, 256])
@pytest.mark.parametrize("zmax,flags", [(31.0, 0), (32.0, 0), (15.0, 4), (16.0, 4)])
def test_bank_sums_on_both_sides_of_a_full_chip(gpu, m, zmax, flags):
    """At L 16384 (129 blocks a tile of rows) 32 and 33 rows, or 16 and 17 at
    half-bin offsets, lie on the two sides of 256 blocks: two rows to a wave
    and four."""
    test_bank_sums(gpu, "fp32", 16384, m, zmax, 2.0, flags)
