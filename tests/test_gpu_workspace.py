"""Workspace of a plan under GSHT_MAX_WORKSPACE_BYTES.  The ring starts of the Legendre
kernels take what the cap leaves after everything else, the library FFT's work buffer
included; where that is not enough for all of them each Legendre launch rebuilds them in
the (then idle) column buffer, with the same bits in the synthesis and, in the adjoint,
whose atomic sums have no fixed order, to 1e-13 (FP32: 1e-6).  What a plan reports stays
within the cap wherever a plan without resident starts does."""
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


def smallest_cap(G, monkeypatch, args, hi):
    """The smallest workspace cap at which the plan is accepted."""
    lo = 1
    while lo < hi:
        mid = (lo + hi) // 2
        monkeypatch.setenv("GSHT_MAX_WORKSPACE_BYTES", str(mid))
        try:
            G.Plan(*args).close()
            hi = mid
        except G.GshtError as e:
            assert e.code == G.GSHT_ENOMEM
            lo = mid + 1
    monkeypatch.delenv("GSHT_MAX_WORKSPACE_BYTES")
    return lo


# The library's real transforms (spin 0) of 512 points and more have a work buffer several
# times the ring starts; few m leave room for the starts, and at lmax 3, mmax 0 the column
# buffer is smaller than they are.
@pytest.mark.parametrize("lmax,mmax,spin,prec,eps,rebuilt", [
    (127, 127, 0, "f64", 1e-10, True), (1000, 1000, 0, "f32", 1e-5, True),
    (200, 60, 0, "f32", 1e-5, False), (3, 0, 1, "f32", 1e-2, False)])
@pytest.mark.parametrize("nmaps", [1, 9])
def test_tight_cap(G, monkeypatch, capfd, lmax, mmax, spin, prec, eps, rebuilt, nmaps):
    print("tight cap", lmax, mmax, spin, prec, nmaps, flush=True)
    th, ph = (torch.from_numpy(x).cuda() for x in wl.uniform_sphere(3000, np.random.default_rng(3)))
    args = (th, ph, lmax, mmax, spin, eps, prec)
    cdt = torch.complex128 if prec == "f64" else torch.complex64
    a = torch.from_numpy(np.stack([wl.gaussian_alm(lmax, mmax, spin, np.random.default_rng(k))
                                   for k in range(nmaps)])).cuda().to(cdt)
    whole = G.Plan(*args)
    least = smallest_cap(G, monkeypatch, args, 2 * whole.info()["workspace_bytes"])
    monkeypatch.setenv("GSHT_MAX_WORKSPACE_BYTES", str(least))
    monkeypatch.setenv("GSHT_PLAN_TRACE", "1")
    capfd.readouterr()
    tight = G.Plan(*args)
    assert ("no ring starts" in capfd.readouterr().err) == rebuilt
    if rebuilt:
        assert tight.info()["workspace_bytes"] < whole.info()["workspace_bytes"]
    m0, m1 = whole.synth_many(a), tight.synth_many(a)
    assert torch.equal(m0, m1)
    b0, b1 = whole.adjoint_many(m0), tight.adjoint_many(m0)
    tol = 1e-13 if prec == "f64" else 1e-6
    assert torch.linalg.norm(b1 - b0) <= tol * torch.linalg.norm(b0)
    assert torch.equal(m0, tight.synth_many(a))  # after an adjoint has used the buffer
    sys.stdout.flush()


@pytest.mark.parametrize("lmax,spin,prec,eps", [(127, 0, "f64", 1e-10), (300, 0, "f32", 1e-5),
                                                (255, 2, "f64", 1e-10)])
def test_reported_bytes_within_the_cap(G, monkeypatch, lmax, spin, prec, eps):
    print("cap", lmax, spin, prec, flush=True)
    th, ph = (torch.from_numpy(x).cuda() for x in wl.uniform_sphere(3000, np.random.default_rng(4)))
    args = (th, ph, lmax, lmax, spin, eps, prec)

    def bytes_at(cap):
        monkeypatch.setenv("GSHT_MAX_WORKSPACE_BYTES", str(cap))
        plan = G.Plan(*args)
        n = plan.info()["workspace_bytes"]
        plan.close()
        return n

    full = bytes_at(1 << 40)
    least = smallest_cap(G, monkeypatch, args, 2 * full)
    bare = bytes_at(least)
    for k in range(7):
        cap = max(least, bare) + (max(full - max(least, bare), 0) * k) // 6
        for c in (cap, cap + 1, max(cap - 1, least)):
            got = bytes_at(c)
            print("  cap %d: %d bytes (whole %d, bare %d)" % (c, got, full, bare), flush=True)
            assert got <= max(c, bare)
    assert bytes_at(full) == full
    sys.stdout.flush()


@pytest.mark.parametrize("lmax,spin,prec,eps", [(200, 2, "f64", 1e-10), (150, 0, "f32", 1e-5)])
def test_patch_buffers_are_counted(G, monkeypatch, capfd, lmax, spin, prec, eps):
    """The spreading's patch buffers are part of what a plan reports, follow its points,
    and take only what the cap leaves; a one-shot synthesis, which never spreads, has none."""
    print("patch bytes", lmax, spin, prec, flush=True)
    rng = np.random.default_rng(9)
    pts = [tuple(torch.from_numpy(x).cuda() for x in wl.uniform_sphere(n, rng))
           for n in (5000, 800)]
    monkeypatch.setenv("GSHT_PLAN_TRACE", "1")

    def make(k):
        capfd.readouterr()
        plan = G.Plan(*pts[k], lmax, lmax, spin, eps, prec)
        return plan, capfd.readouterr().err

    def patch_bytes(inf):
        cells = (inf["tile1"] + inf["w"] - 1) * (inf["tile2"] + inf["w"] - 1)
        value = (8 if prec == "f64" else 4) * (2 if spin else 1)
        return inf["nchunks"] * cells * value + 4 * (inf["ntile1"] * inf["ntile2"] + 1)

    plan, err = make(0)
    assert "spreading by patch buffers" in err
    inf = plan.info()
    total, bare = inf["workspace_bytes"], inf["workspace_bytes"] - patch_bytes(inf)
    for k in (1, 0):
        plan.set_points(*pts[k])
        inf = plan.info()
        assert inf["workspace_bytes"] == bare + patch_bytes(inf)
    plan.close()
    for cap, flush in ((total - 1, "tile colours"), (total, "patch buffers")):
        monkeypatch.setenv("GSHT_MAX_WORKSPACE_BYTES", str(cap))
        plan, err = make(0)
        assert "spreading by " + flush in err
        assert plan.info()["workspace_bytes"] == (total if flush == "patch buffers" else bare)
        plan.set_points(*pts[1])  # fewer chunks: room again
        assert plan.info()["workspace_bytes"] == bare + patch_bytes(plan.info())
        plan.close()
    monkeypatch.delenv("GSHT_MAX_WORKSPACE_BYTES")
    cdt = torch.complex128 if prec == "f64" else torch.complex64
    a = torch.from_numpy(wl.gaussian_alm(lmax, lmax, spin, rng)).cuda().to(cdt)
    capfd.readouterr()
    m = G.synth_general(a, *pts[0], lmax, lmax, spin, eps, prec)
    assert "spreading by tile colours" in capfd.readouterr().err
    G.adjoint_synth_general(m, *pts[0], lmax, lmax, spin, eps, prec)
    assert "spreading by patch buffers" in capfd.readouterr().err
    sys.stdout.flush()
