"""Recurrence starts of the Legendre kernels: every (m, ring pair) enters the sums at an
8-degree block of its own.  Degree ranges shorter than a block, of exactly one or two
blocks and one off them, rings at which nothing ever enters (mmax near lmax on many
rings), every launch shape, and starts kept in bands of m.  Against the oracle the bar is
the stage's own (1e-12 relative); a banded plan runs the same operations on the same
values as an unbanded one, so its synthesis must give the same bits, and its adjoint,
whose atomic sums have no fixed order, must agree to 1e-13."""
import sys

import numpy as np
import pytest
import torch

import oracle
from paper_2304_10431_amd import workloads as wl

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def G():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2304_10431_amd import gsht
    return gsht


def rel(a, b):
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


@pytest.mark.parametrize("syn_r,adj_r", [(1, 1), (2, 2), (4, 4), (2, 5), (1, 3)])
@pytest.mark.parametrize("lmax,mmax,spin,ntheta", [(0, 0, 0, 2), (2, 2, 2, 4), (7, 7, 0, 9),
                                                   (8, 8, 1, 140), (15, 3, 3, 650),
                                                   (16, 16, 2, 18), (23, 23, 0, 300),
                                                   (33, 31, 2, 700)])
def test_short_degree_ranges(G, monkeypatch, syn_r, adj_r, lmax, mmax, spin, ntheta):
    say("starts", syn_r, adj_r, lmax, mmax, spin, ntheta)
    monkeypatch.setenv("GSHT_SYN_R", str(syn_r))
    monkeypatch.setenv("GSHT_ADJ_R", str(adj_r))
    th = np.pi * np.arange(ntheta) / (ntheta - 1)
    a = wl.gaussian_alm(lmax, mmax, spin, np.random.default_rng(lmax + spin), cl=np.ones(lmax + 1))
    F = G.legendre_rings(torch.from_numpy(a).cuda(), lmax, mmax, spin, ntheta).cpu().numpy()
    H = oracle.ring_synth(a, lmax, mmax, spin, th)
    H = H[mmax:] if spin == 0 else H
    assert rel(F[:, :ntheta], H) <= 1e-12
    ad = G.legendre_rings_adjoint(torch.from_numpy(F).cuda(), lmax, mmax, spin, ntheta).cpu().numpy()
    ms = np.arange(0, mmax + 1) if spin == 0 else np.arange(-mmax, mmax + 1)
    U = F[:, :ntheta].copy()
    U[:, 1:ntheta - 1] += ((-1.0) ** ((spin + ms) % 2))[:, None] * F[:, :ntheta - 1:-1]
    full = np.zeros((2 * mmax + 1, ntheta), complex)
    full[2 * mmax + 1 - U.shape[0]:] = U
    assert rel(ad, oracle.ring_adjoint(full, lmax, mmax, spin, th)) <= 1e-12


@pytest.mark.parametrize("spin,prec,eps", [(2, "f64", 1e-10), (0, "f64", 1e-7), (1, "f32", 1e-5)])
@pytest.mark.parametrize("nmaps", [1, 3, 9])
def test_bands_equal_whole(G, monkeypatch, spin, prec, eps, nmaps):
    lmax, npts = 150, 4000
    th, ph = (torch.from_numpy(x).cuda() for x in wl.uniform_sphere(npts, np.random.default_rng(3)))
    whole = G.Plan(th, ph, lmax, lmax, spin, eps, prec)
    # the smallest workspace cap that is accepted leaves room for about half of the starts
    lo, hi = 1, whole.info()["workspace_bytes"]
    while lo < hi:
        mid = (lo + hi) // 2
        monkeypatch.setenv("GSHT_MAX_WORKSPACE_BYTES", str(mid))
        try:
            G.Plan(th, ph, lmax, lmax, spin, eps, prec).close()
            hi = mid
        except G.GshtError as e:
            assert e.code == G.GSHT_ENOMEM
            lo = mid + 1
    monkeypatch.setenv("GSHT_MAX_WORKSPACE_BYTES", str(lo))
    band = G.Plan(th, ph, lmax, lmax, spin, eps, prec)
    say("bands", spin, prec, nmaps, whole.info()["workspace_bytes"], band.info()["workspace_bytes"])
    assert band.info()["workspace_bytes"] < whole.info()["workspace_bytes"]
    cdt = torch.complex128 if prec == "f64" else torch.complex64
    a = torch.from_numpy(np.stack([wl.gaussian_alm(lmax, lmax, spin, np.random.default_rng(k))
                                   for k in range(nmaps)])).cuda().to(cdt)
    m0, m1 = whole.synth_many(a), band.synth_many(a)
    assert torch.equal(m0, m1)
    b0, b1 = (p.adjoint_many(m0).to(torch.complex128).cpu().numpy() for p in (whole, band))
    assert rel(b1, b0) <= (1e-13 if prec == "f64" else 1e-6)
