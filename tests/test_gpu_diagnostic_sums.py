"""The last sums of the diagnostics (one workgroup per map over the per-block partials): chi^2,
its harmonic part, |s| and n_dof of a solve against torch sums over the returned signal, with
fewer partials than threads, exactly as many, one more, and several per thread.

Tolerance: both sides add positive FP64 terms, none through more than a few hundred
sequential additions, so each is within 512 x 2^-53 = 6e-14 of the exact sum of its terms, and
the terms themselves within a few ulp: 1e-12."""
import pytest
import torch

from paper_1210_4931_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1210_4931_amd import mfwf
    mfwf.load()
    return mfwf


@pytest.mark.parametrize("nside,lmax,nb", [(4, 8, 1), (128, 255, 3), (128, 256, 2), (256, 600, 1)])
def test_diagnostics_are_the_sums_of_their_terms(mf, nside, lmax, nb):
    npix = 12 * nside * nside
    g = torch.Generator(device="cuda").manual_seed(5)
    d = torch.randn(nb, npix, dtype=torch.float64, device="cuda", generator=g)
    ninv = torch.rand(npix, dtype=torch.float64, device="cuda", generator=g) + 0.5
    ninv[::7] = 0.0
    cl = torch.as_tensor(W.cl_damped(lmax, 200.0), dtype=torch.float64)
    p = mf.Plan(nside, lmax, max_batch=nb)
    p.set_covariances(cl.numpy(), ninv)
    s, smap, info = p.solve(d, iters=4)
    torch.cuda.synchronize()
    l = torch.cat([torch.arange(m, lmax + 1) for m in range(lmax + 1)]).cuda()
    w = torch.cat([torch.full((lmax + 1 - m,), 1.0 if m == 0 else 2.0, dtype=torch.float64)
                   for m in range(lmax + 1)]).cuda()
    c = cl.cuda()[l]
    q = w * (s.real ** 2 + s.imag ** 2)
    harm = torch.where(c > 0, q / torch.where(c > 0, c, torch.ones_like(c)), torch.zeros_like(q)).sum(1)
    pix = (ninv * (d - smap) ** 2).sum(1)
    for b in range(nb):
        assert info[b].n_dof == int((ninv > 0).sum())
        assert info[b].tau == 1.0 / float(ninv.max())
        assert info[b].chi2_harm == pytest.approx(float(harm[b]), rel=1e-12)
        assert info[b].snorm == pytest.approx(float(q[b].sum().sqrt()), rel=1e-12)
        assert info[b].chi2 == pytest.approx(float(harm[b] + pix[b]), rel=1e-12)
