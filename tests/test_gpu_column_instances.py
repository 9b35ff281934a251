"""The paired column stage (mode 2) is compiled for several workgroup sizes and counts of
register slots; a plan takes its instance from the column length and the number of column
pairs.  Each case names the instance it has to land on (read from the plan trace): together
they are all that a plan comes to with the default LDS padding.  Synthesis and adjoint
against the same plan's library FFT columns (mode 0), with odd and even numbers of columns,
and against the oracle at a few points.

Both column stages make three transforms of at most 16384 points, each with a relative
rounding of about 0.6 log2(n) epsilon: their difference stays below 2 * 3 * 0.6 * 14 epsilon
= 51 epsilon, 3e-6 in FP32 (bar 4e-6); the FP64 bar is the stage's 1e-12."""
import sys

import numpy as np
import pytest
import torch

import oracle
from paper_2304_10431_amd import workloads as wl

pytestmark = pytest.mark.gpu

# prec, spin, lmax, mmax, sigma, epsilon; threads, forward slots, adjoint slots
CASES = [
    ("f64", 2, 255, 255, 2.0, 1e-10, 1024, 4, 4),
    ("f64", 2, 2100, 20, 1.5, 1e-10, 1024, 4, 5),
    ("f64", 1, 3000, 16, 1.5, 1e-10, 1024, 5, 6),
    ("f64", 0, 3072, 11, 2.0, 1e-10, 1024, 6, 7),
    ("f64", 0, 3200, 12, 2.0, 1e-10, 1024, 8, 8),
    ("f64", 2, 4200, 12, 1.25, 1e-9, 1024, 6, 9),
    ("f64", 0, 4800, 11, 1.5, 1e-10, 1024, 8, 10),
    ("f64", 2, 300, 300, 2.0, 1e-10, 512, 6, 6),
    ("f64", 2, 1536, 300, 2.0, 1e-10, 512, 6, 8),
    ("f64", 0, 2047, 600, 2.0, 1e-10, 512, 8, 8),
    ("f64", 2, 2048, 260, 2.0, 1e-10, 512, 8, 9),
    ("f64", 2, 700, 700, 2.0, 1e-10, 256, 6, 6),
    ("f64", 2, 800, 600, 2.0, 1e-10, 256, 8, 8),
    ("f64", 2, 1140, 600, 1.5, 1e-10, 256, 8, 9),
    ("f32", 2, 200, 200, 2.0, 1e-5, 512, 9, 9),
    ("f32", 1, 2200, 21, 2.0, 1e-5, 512, 12, 12),
    ("f32", 0, 4200, 9, 1.5, 1e-5, 512, 17, 17),
    ("f32", 2, 700, 700, 2.0, 1e-5, 256, 9, 9),
    ("f32", 2, 1300, 777, 1.5, 1e-5, 256, 9, 12),
    ("f32", 0, 1500, 1100, 2.0, 1e-5, 256, 12, 12),
]


@pytest.fixture(scope="module")
def G():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2304_10431_amd import gsht
    return gsht


def rel_l2(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("prec,spin,lmax,mmax,sigma,eps,nt,fwd,adj", CASES)
def test_column_instance(G, monkeypatch, capfd, prec, spin, lmax, mmax, sigma, eps, nt, fwd, adj):
    print("column instance", prec, spin, lmax, mmax, sigma, nt, fwd, adj, flush=True)
    rng = np.random.default_rng(lmax + mmax)
    th, ph = wl.uniform_sphere(1500, rng)
    a = wl.gaussian_alm(lmax, mmax, spin, rng)
    y = rng.standard_normal((oracle.ncomp(spin), th.size))
    w = np.sqrt(oracle.alm_weights(lmax, mmax))[None, :]
    cdt, rdt = ((torch.complex128, torch.float64) if prec == "f64"
                else (torch.complex64, torch.float32))
    da, dy = torch.from_numpy(a).cuda().to(cdt), torch.from_numpy(y).cuda().to(rdt)
    dth, dph = torch.from_numpy(th).cuda(), torch.from_numpy(ph).cuda()
    monkeypatch.setenv("GSHT_PLAN_TRACE", "1")
    outs = []
    for mode in (2, 0):
        monkeypatch.setenv("GSHT_COLUMN_MODE", str(mode))
        capfd.readouterr()
        plan = G.Plan(dth, dph, lmax, mmax, spin, eps, prec, sigma=sigma)
        err = capfd.readouterr().err
        if mode == 2:
            assert ("column mode 2, %d threads, %d forward and %d adjoint slots"
                    % (nt, fwd, adj)) in err, err
        outs.append((plan.synth(da).double().cpu().numpy(),
                     plan.adjoint(dy).to(torch.complex128).cpu().numpy()))
        plan.close()
    bar = 1e-12 if prec == "f64" else 4e-6
    assert rel_l2(outs[0][0], outs[1][0]) <= bar
    assert rel_l2(outs[0][1] * w, outs[1][1] * w) <= bar
    sel = np.arange(0, th.size, 150)
    ref = oracle.synth(a, lmax, mmax, spin, th[sel], ph[sel])
    assert oracle.eps_eff(outs[0][0][:, sel], ref) <= eps
    sys.stdout.flush()
