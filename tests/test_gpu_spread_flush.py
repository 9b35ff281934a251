"""The three flushes of the spreading (launches by tile colour, plain read-add-write; one
launch over all chunks, atomic adds; a patch buffer per chunk summed in order, the
default at these sizes) on the CPU oracle's adjoint and on each other: sparse and dense
tiles, odd and even numbers of tile columns, both precisions, real and complex grids.  All
add the same patches in another order, so they agree to the rounding of the grid (1e-12
FP64, 2e-6 FP32) and stay within epsilon.  The buffers are rebuilt by new points, give the
same bits every time, and are left out where the workspace cap has no room for them."""
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


@pytest.mark.parametrize("lmax,mmax,spin,npts,prec,eps", [
    (130, 130, 2, 30000, "f64", 1e-10), (127, 90, 0, 20000, "f64", 1e-12),
    (60, 60, 2, 60000, "f32", 1e-5), (200, 200, 0, 40000, "f32", 1e-5),
    (96, 17, 1, 7001, "f64", 1e-6)])
def test_flushes_agree(G, monkeypatch, lmax, mmax, spin, npts, prec, eps):
    say("spread flush", lmax, mmax, spin, npts, prec)
    rng = np.random.default_rng(lmax + npts)
    th, ph = wl.uniform_sphere(npts, rng)
    th[:npts // 3] = 1.0 + 0.03 * rng.random(npts // 3)   # a few dense tiles
    ph[:npts // 3] = 2.0 + 0.03 * rng.random(npts // 3)
    y = rng.standard_normal((oracle.ncomp(spin), npts))
    rdt = torch.float64 if prec == "f64" else torch.float32
    w = np.sqrt(oracle.alm_weights(lmax, mmax))[None, :]
    ref = oracle.adjoint(y, lmax, mmax, spin, th, ph)
    outs = []
    for env in ("1", "0", None):
        if env is None:
            monkeypatch.delenv("GSHT_SPREAD_COLORS", raising=False)
        else:
            monkeypatch.setenv("GSHT_SPREAD_COLORS", env)
        plan = G.Plan(torch.from_numpy(th).cuda(), torch.from_numpy(ph).cuda(), lmax, mmax, spin,
                      eps, prec)
        b = plan.adjoint(torch.from_numpy(y).cuda().to(rdt)).to(torch.complex128).cpu().numpy()
        plan.close()
        outs.append(b)
        assert oracle.eps_eff(b * w, ref * w) <= eps
    tol = 1e-12 if prec == "f64" else 2e-6
    for b in outs[1:]:
        assert np.linalg.norm((b - outs[0]) * w) <= tol * np.linalg.norm(outs[0] * w)


def test_patch_buffers_follow_the_points(G, monkeypatch):
    rng = np.random.default_rng(5)
    lmax, spin = 100, 2
    dev = [tuple(torch.from_numpy(x).cuda() for x in wl.uniform_sphere(n, rng))
           for n in (40000, 300, 9000)]
    plan = G.Plan(*dev[0], lmax, lmax, spin, 1e-8, "f64")
    for th, ph in dev:
        y = torch.from_numpy(rng.standard_normal((2, th.numel()))).cuda()
        plan.set_points(th, ph)
        got = plan.adjoint(y)
        fresh = G.Plan(th, ph, lmax, lmax, spin, 1e-8, "f64")
        assert torch.equal(got, fresh.adjoint(y)) and torch.equal(got, plan.adjoint(y))
        ws = fresh.info()["workspace_bytes"]
        fresh.close()
        monkeypatch.setenv("GSHT_MAX_WORKSPACE_BYTES", str(ws + 100))  # no room: by colour
        capped = G.Plan(th, ph, lmax, lmax, spin, 1e-8, "f64")
        monkeypatch.delenv("GSHT_MAX_WORKSPACE_BYTES")
        ref = capped.adjoint(y)
        capped.close()
        assert torch.linalg.norm(got - ref) <= 1e-12 * torch.linalg.norm(ref)
    plan.close()
