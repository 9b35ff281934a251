"""Values far below 1 through the stage entry points.  On rings near a pole the harmonics of
large m are tiny, down to far below 1e-31, and the ring values (and, from such a ring, the
coefficients) have to come out right in themselves, not only against the largest ones.

One coefficient per m, at l = max(m, s) or six degrees above, so that a ring value is one
harmonic, far inside the region where it has no zeros: compared with the oracle value by
value.  Both sides form sin^m and cos^m of half the angle by products of about log2 m
factors from rounded angles, m (2 + 2 log2 m) roundings at most on either side, and the
recurrence adds a few: the bar is 8 lmax log2(lmax) 2^-53."""
import sys

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2304_10431_amd import gsht
    return gsht


def bar(lmax):
    return 8 * lmax * np.log2(lmax) * 2.0 ** -53


@pytest.mark.parametrize("lmax,spin", [(130, 0), (300, 2), (300, 0), (257, 5)])
@pytest.mark.parametrize("up", [0, 6])
def test_small_ring_values(G, lmax, spin, up):
    print("small rings", lmax, spin, up, flush=True)
    nt = lmax + 2
    th = np.pi * np.arange(nt) / (nt - 1)
    a = np.zeros((oracle.ncomp(spin), oracle.nalm(lmax, lmax)), complex)
    for m in range(lmax + 1):
        l = min(max(m, spin) + up, lmax)
        a[0, oracle.alm_index(l, m, lmax)] = 1.0 + (0.5j if m else 0.0)
    F = G.legendre_rings(torch.from_numpy(a).cuda(), lmax, lmax, spin, nt).cpu().numpy()
    H = oracle.ring_synth(a, lmax, lmax, spin, th)
    # the northern half, where the oracle's angles are right to rounding (pi - theta near
    # the south pole is not: it has no reference there); columns m and -m hold both channels
    H = (H[lmax:] if spin == 0 else H)[:, :nt // 2]
    small = (np.abs(H) > 1e-250) & (np.abs(H) < 1e-25)
    assert small.sum() > 1000
    err = np.abs(F[:, :nt // 2] - H)[small] / np.abs(H)[small]
    print("  %d values, worst %.2e, bar %.2e" % (small.sum(), err.max(), bar(lmax)), flush=True)
    assert err.max() <= bar(lmax)
    sys.stdout.flush()


@pytest.mark.parametrize("lmax,spin", [(130, 0), (300, 2), (257, 5)])
def test_small_coefficients(G, lmax, spin):
    """The adjoint of one ring near the pole: b_lm is that ring's harmonic, right down to
    2^-256 (about 1e-77) at the start of a block of 8 degrees, over which it grows by less
    than 2^35 at these sizes."""
    print("small coefficients", lmax, spin, flush=True)
    nt, ring = lmax + 2, 6
    th = np.pi * np.arange(nt) / (nt - 1)
    ncol = lmax + 1 if spin == 0 else 2 * lmax + 1
    F = np.zeros((ncol, 2 * nt - 2), complex)
    F[ncol - lmax - 1:, ring] = 1.0 + 0.25j  # columns m >= 0
    H = np.zeros((2 * lmax + 1, nt), complex)
    H[lmax:, ring] = 1.0 + 0.25j
    if spin == 0:
        F[0, ring] = H[lmax, ring] = 1.0
    ref = oracle.ring_adjoint(H, lmax, lmax, spin, th)
    dF = torch.from_numpy(F).cuda()
    out = torch.empty(ref.shape, dtype=torch.complex128, device="cuda")
    G.legendre_rings_adjoint_noalloc(dF, lmax, lmax, spin, nt, out)
    m = np.concatenate([np.full(lmax + 1 - k, k) for k in range(lmax + 1)])[None, :]
    small = (np.abs(ref) > 2.0 ** -221) & (np.abs(ref) < 1e-25) & (m > 0)
    assert small.sum() > 1000
    for b in (G.legendre_rings_adjoint(dF, lmax, lmax, spin, nt), out):
        err = np.abs(b.cpu().numpy() - ref)[small] / np.abs(ref)[small]
        print("  %d values, worst %.2e, bar %.2e" % (small.sum(), err.max(), bar(lmax)), flush=True)
        assert err.max() <= bar(lmax)
    sys.stdout.flush()


def test_noalloc_in_bands(G):
    """More ring starts than the allocation-free entry point has room for (36 x 10001 x 201
    bytes against 64 MiB): built band by band, the same sums as from one table (1e-13)."""
    lmax, spin, nt = 200, 2, 20001
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    F = torch.randn((2 * lmax + 1, 2 * nt - 2), generator=g, device="cuda", dtype=torch.complex128)
    ref = G.legendre_rings_adjoint(F, lmax, lmax, spin, nt)
    out = torch.empty_like(ref)
    G.legendre_rings_adjoint_noalloc(F, lmax, lmax, spin, nt, out)
    assert torch.linalg.norm(out - ref) <= 1e-13 * torch.linalg.norm(ref)
    sys.stdout.flush()
