"""The ring transforms' two classes go in one launch or in two by a rule on length, step and number of
rows: results on both sides of the rule's lines, and at lengths where it does not ask for the
rows, are the same bits."""
import numpy as np
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


def problem(mf, spin, nside, lmax, maps, dtype):
    npix = 12 * nside * nside
    g = torch.Generator(device="cuda").manual_seed(3)
    d = torch.randn(*((maps, 3, npix) if spin else (maps, npix)), generator=g, dtype=torch.float64, device="cuda")
    p = mf.Plan(nside, lmax, max_batch=maps, spin=spin, dtype=dtype)
    cl = W.cl_damped(lmax, 100.0)
    ninv = torch.rand(npix, generator=g, dtype=torch.float64, device="cuda") + 0.5
    if spin:
        n6 = torch.zeros(npix, 6, dtype=torch.float64, device="cuda")
        n6[:, 0], n6[:, 3], n6[:, 5] = ninv, 0.5 * ninv, 0.5 * ninv
        cl, ninv = W.pol_cls(cl), n6
    p.set_covariances(cl, ninv)
    return p, d


# rows around the lines: 24 | 25 (T), 8 | 9 maps = 24 | 27 rows (T, Q, U), and one map; nside 256 has
# transforms of 2048 points, nside 128 of 1024
@pytest.mark.parametrize("spin,nside,lmax,maps,dtype", [(0, 256, 300, 25, "f32"), (0, 256, 300, 25, "f64"), (2, 256, 200, 9, "f32"),
                                                        (2, 256, 200, 9, "f64"), (2, 128, 256, 9, "f32")])
def test_both_sides_of_the_lines(mf, spin, nside, lmax, maps, dtype):
    p, d = problem(mf, spin, nside, lmax, maps, dtype)
    a, (s, m, _) = p.sht_fwd(d), p.solve(d, lam=[5.0], iters=[4])
    mp = p.sht_inv(a)
    for n in (maps - 1, 1):
        assert torch.equal(p.sht_fwd(d[:n]), a[:n]) and torch.equal(p.sht_inv(a[:n]), mp[:n])
        s1, m1, _ = p.solve(d[:n], lam=[5.0], iters=[4])
        assert torch.equal(s1, s[:n]) and torch.equal(m1, m[:n])
    assert np.all(np.isfinite(mp.cpu().numpy()))
