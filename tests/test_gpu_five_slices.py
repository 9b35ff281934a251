"""The adjoint Legendre kernel with five slices of 64 ring pairs per wave, the default of
large plans, at degree ranges of many blocks: rings that fill one chunk of 320 pairs, end
inside its last slice, or spill into a second chunk, all three forms of the kernel (spin 0,
spin s, gradient only) and both precisions of its input.  Bars as for the other launch
shapes: 1e-12 against the oracle's rings; gradient only, 1e-13 (FP32 2e-6) against the
general path and epsilon against the oracle."""
import sys

import numpy as np
import pytest
import torch

import oracle
from paper_2304_10431_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2304_10431_amd import gsht
    return gsht


@pytest.fixture(autouse=True)
def shape(monkeypatch):
    for k, v in (("GSHT_SYN_R", "4"), ("GSHT_ADJ_R", "5"), ("GSHT_ADJ_B", "8")):
        monkeypatch.setenv(k, v)


@pytest.mark.parametrize("lmax,mmax,spin,ntheta", [(300, 300, 2, 302), (417, 300, 0, 639),
                                                   (250, 250, 1, 641), (520, 400, 2, 700),
                                                   (600, 200, 0, 1300)])
def test_rings(G, lmax, mmax, spin, ntheta):
    print("five slices", lmax, mmax, spin, ntheta, flush=True)
    rng = np.random.default_rng(lmax + spin)
    nd, ncol = 2 * ntheta - 2, 2 * mmax + 1 if spin else mmax + 1
    F = rng.standard_normal((ncol, nd)) + 1j * rng.standard_normal((ncol, nd))
    ms = np.arange(-mmax, mmax + 1) if spin else np.arange(mmax + 1)
    H = np.zeros((2 * mmax + 1, ntheta), complex)
    H[-ncol:] = F[:, :ntheta]
    H[-ncol:, 1:ntheta - 1] += ((-1.0) ** ((spin + ms) % 2))[:, None] * F[:, :ntheta - 1:-1]
    ref = oracle.ring_adjoint(H, lmax, mmax, spin, np.pi * np.arange(ntheta) / (ntheta - 1))
    got = G.legendre_rings_adjoint(torch.from_numpy(F).cuda(), lmax, mmax, spin, ntheta)
    err = np.linalg.norm(got.cpu().numpy() - ref) / np.linalg.norm(ref)
    assert err <= 1e-12, err
    sys.stdout.flush()


@pytest.mark.parametrize("spin,lmax,mmax,prec,eps", [(2, 420, 420, "f64", 1e-10),
                                                     (3, 700, 90, "f64", 1e-10),
                                                     (2, 420, 420, "f32", 1e-5)])
def test_gradient_only(G, spin, lmax, mmax, prec, eps):
    print("five slices, gradient only", spin, lmax, mmax, prec, flush=True)
    rng = np.random.default_rng(lmax)
    th, ph = wl.uniform_sphere(6000, rng)
    y = rng.standard_normal((2, th.size))
    dy = torch.from_numpy(y).cuda().to(torch.float64 if prec == "f64" else torch.float32)
    plan = G.Plan(torch.from_numpy(th).cuda(), torch.from_numpy(ph).cuda(), lmax, mmax, spin, eps,
                  prec)
    assert plan.info()["adj_r"] == 5
    got = plan.adjoint_grad(dy).to(torch.complex128).cpu().numpy()
    full = plan.adjoint(dy)[:1].to(torch.complex128).cpu().numpy()
    plan.close()
    w = np.sqrt(oracle.alm_weights(lmax, mmax))[None, :]
    assert oracle.eps_eff(w * got, w * full) <= (1e-13 if prec == "f64" else 2e-6)
    ref = oracle.adjoint(y, lmax, mmax, spin, th, ph)[:1]
    assert oracle.eps_eff(w * got, w * ref) <= eps
    sys.stdout.flush()
