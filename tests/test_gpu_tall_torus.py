"""Spreading on a torus that keeps more rows than a launch takes workgroups along grid y
(65535): lmax 24601 at sigma 2 has 131072 torus rows and keeps 65536 + w + 2 of them.  Few
tiles, so every chunk's patch goes to a buffer and the buffers are summed over all rows;
some points lie at the south pole, whose patches end in the last rows.  Against the
launches by colour (the same patches added in another order: FP64 rounding) and the FP64
oracle."""
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


@pytest.mark.parametrize("spin", [0, 2])
def test_more_rows_than_grid_y(G, monkeypatch, spin):
    lmax, mmax, eps = 24601, 15, 1e-8
    print("tall torus", spin, flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(77 + spin)
    th, ph = wl.uniform_sphere(60, rng)
    th[:20] = np.pi - 1e-4 * rng.random(20)
    th[0] = np.pi
    dth, dph = torch.from_numpy(th).cuda(), torch.from_numpy(ph).cuda()
    y = rng.standard_normal((oracle.ncomp(spin), th.size))
    w = np.sqrt(oracle.alm_weights(lmax, mmax))[None, :]
    outs = []
    for env in (None, "1"):
        if env is not None:
            monkeypatch.setenv("GSHT_SPREAD_COLORS", env)
        plan = G.Plan(dth, dph, lmax, mmax, spin, eps, "f64")
        inf = plan.info()
        assert inf["nrows"] > 65535 and inf["spread_colors"] > 0
        assert inf["ntile1"] * inf["ntile2"] <= 6144
        outs.append(plan.adjoint(torch.from_numpy(y).cuda()).cpu().numpy())
        plan.close()
    assert np.linalg.norm((outs[0] - outs[1]) * w) <= 1e-12 * np.linalg.norm(outs[1] * w)
    ref = oracle.adjoint(y, lmax, mmax, spin, th, ph)
    assert oracle.eps_eff(outs[0] * w, ref * w) <= eps
