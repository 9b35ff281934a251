"""Which flush the spreading of a plan takes (read from the plan trace): patch buffers on
grids of few tiles, and on large grids only where the launches by colour would run long
chains of chunks one after another; a large grid with a few scattered points goes by
colour.  Each route's adjoint against the same plan forced to the launches by colour (the
same patches added in another order: FP64 1e-12, FP32 2e-6)."""
import sys

import numpy as np
import pytest
import torch

from paper_2304_10431_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2304_10431_amd import gsht
    return gsht


def points(kind, n, rng):
    th, ph = wl.uniform_sphere(n, rng)
    if kind == "dense":  # all in a few tiles of the grid at lmax 1300
        th, ph = 1.2 + 0.02 * rng.random(n), 2.0 + 0.02 * rng.random(n)
    return th, ph


@pytest.mark.parametrize("lmax,mmax,spin,n,kind,prec,eps,route", [
    (200, 200, 2, 3000, "uniform", "f64", 1e-10, "patch buffers"),
    (900, 400, 0, 3000, "uniform", "f32", 1e-5, "patch buffers"),
    (1300, 1300, 2, 3000, "uniform", "f64", 1e-10, "tile colours"),
    (1300, 1300, 2, 3000, "uniform", "f32", 1e-5, "tile colours"),
    (1300, 1300, 2, 100000, "dense", "f64", 1e-10, "patch buffers"),
    (1300, 1300, 0, 100000, "dense", "f32", 1e-5, "patch buffers"),
    (1300, 1300, 2, 1, "uniform", "f64", 1e-10, "tile colours"),
    (40, 0, 0, 50, "uniform", "f64", 1e-10, "atomic adds")])
def test_route(G, monkeypatch, capfd, lmax, mmax, spin, n, kind, prec, eps, route):
    print("spread route", lmax, mmax, spin, n, kind, prec, flush=True)
    rng = np.random.default_rng(n + lmax)
    th, ph = (torch.from_numpy(x).cuda() for x in points(kind, n, rng))
    y = torch.from_numpy(rng.standard_normal((2 if spin else 1, n))).cuda()
    y = y.to(torch.float64 if prec == "f64" else torch.float32)
    monkeypatch.setenv("GSHT_PLAN_TRACE", "1")
    capfd.readouterr()
    plan = G.Plan(th, ph, lmax, mmax, spin, eps, prec)
    assert "spreading by " + route in capfd.readouterr().err
    got = plan.adjoint(y)
    plan.close()
    monkeypatch.setenv("GSHT_SPREAD_COLORS", "1")
    plan = G.Plan(th, ph, lmax, mmax, spin, eps, prec)
    assert "patch buffers" not in capfd.readouterr().err
    ref = plan.adjoint(y)
    plan.close()
    tol = 1e-12 if prec == "f64" else 2e-6
    assert torch.linalg.norm(got - ref) <= tol * torch.linalg.norm(ref)
    sys.stdout.flush()
