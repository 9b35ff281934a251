"""The benchmark's count of Legendre terms (the share of degrees at or past a ring's entry
block) against harmonics from the oracle."""
import numpy as np
import pytest

import bench
import oracle


@pytest.mark.parametrize("lmax,mmax,spin,exponent", [(90, 90, 0, -20), (90, 60, 2, -20),
                                                     (70, 70, 3, -12), (40, 40, 2, -100)])
def test_entered_share(lmax, mmax, spin, exponent):
    nring = 40
    theta = np.pi * (np.arange(nring) + 0.5) / (2 * nring)
    done = total = 0
    for m in range(mmax + 1):
        l0 = max(m, spin)
        norm = np.ones(lmax + 2)  # the kernels' normalisation, factor by factor
        for l in range(l0 + 1, lmax + 1):
            def coupling(k):
                return np.sqrt((k * k - m * m) * (k * k - spin * spin) / (k * k * (4 * k * k - 1.0)))
            if l > l0 + 1:
                norm[l] = norm[l - 2] * coupling(l - 1) / coupling(l)
        for sg in ((spin, -spin) if spin else (0,)):
            for t in theta:
                p = np.abs(oracle.slambda(lmax, m, sg, t)) / norm[:lmax + 1]
                starts = [l for l in range(l0, lmax + 1, 8) if p[l] >= 2.0 ** exponent]
                done += lmax + 1 - starts[0] if starts else 0
                total += lmax + 1 - l0
    got = bench.entered_share(lmax, mmax, spin, exponent, nm=mmax + 1, nring=nring)
    # the bench keeps magnitudes by power of two: an entry may move by one block where the
    # value lies within a factor of two of the threshold
    assert abs(got - done / total) <= 0.02
    assert 0.3 < got <= 1.0
