"""The batched FP32 form's contractions run on the bf16 matrix cores with every FP32 operand
split into three bf16 pieces.  Edges of their tiles (256 values of l, 128 ring pairs, 32 / 64 /
128 columns, chunks of 32 pairs and 64 values of l), from a table and with lambda generated,
against the FP64 path; and the error after many iterations, where an error that repeats from
one iteration to the next would add up.

Tolerances.  One transform: a product of two rounded FP32 operands and its rounding is off by
at most 3 x 2^-24; sums of 16 products are rounded at most 6 times and then added one by one
(lmax + 1 or 2 nside terms, so at most 2 nside / 16 + 1 additions of a running sum), all
roundings of random sign: 2^-24 (3 + 6 + sqrt(nside / 8 + 1)) relative to the norm, under
1e-6 at nside 256.  Iterations: 1e-5, the form's accuracy target."""
import os

import numpy as np
import pytest
import torch

from paper_1210_4931_amd import workloads as W
from tests.gpu_util import dev, rel, rel_alm

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1210_4931_amd import mfwf
    mfwf.load()
    return mfwf


def _plan(mf, spec, *a, **k):
    os.environ["MFWF_TUNE_FORCE"] = spec
    try:
        return mf.Plan(*a, **k)
    finally:
        os.environ.pop("MFWF_TUNE_FORCE", None)


# lmax + 1 around 64, 256 and 512; ring pairs 2 (a partial chunk) to 512 (four tiles)
@pytest.mark.parametrize("nside,lmax,nmaps", [(1, 3, 1), (4, 15, 16), (16, 62, 17), (32, 64, 33), (64, 127, 48),
                                              (64, 128, 65), (128, 254, 5), (128, 256, 64), (256, 511, 70)])
def test_transforms_at_tile_edges(mf, nside, lmax, nmaps):
    rng = np.random.default_rng(nside * lmax + nmaps)
    alm = dev(np.stack([W.white_alm(rng, lmax) for _ in range(nmaps)]), torch.complex128)
    mp = dev(rng.standard_normal((nmaps, 12 * nside * nside)))
    p64 = mf.Plan(nside, lmax, max_batch=nmaps)
    ref_m, ref_a = p64.sht_inv(alm), p64.sht_fwd(mp)
    first = None
    for spec in ("cta=2,cts=2,lamgen=0", "cta=1,cts=1,lamgen=1", "cta=3,cts=1,lamgen=0"):
        print("forced", spec, nside, lmax, nmaps, flush=True)
        p = _plan(mf, spec, nside, lmax, max_batch=nmaps, dtype="f32")
        m, a = p.sht_inv(alm), p.sht_fwd(mp)
        assert rel(m.cpu(), ref_m.cpu()) < 1e-6 and rel_alm(a.cpu().numpy(), ref_a.cpu().numpy(), lmax) < 1e-6, spec
        first = first or (m, a)
        assert torch.equal(m, first[0]) and torch.equal(a, first[1]), spec
        del p


def test_errors_do_not_add_up_over_iterations(mf):
    nside, lmax = 64, 128
    wl = W.config2(3, nside, lmax)
    d = dev(np.stack([30.0 * np.sin(np.arange(12 * nside * nside) * k) + np.sqrt(wl.noise_var) * wl.noise_white
                      for k in (1e-3, 2e-4, 5e-5)]))
    p64, p32 = mf.Plan(nside, lmax, max_batch=3), mf.Plan(nside, lmax, max_batch=3, dtype="f32")
    for p in (p64, p32):
        p.set_covariances(wl.cl, dev(wl.ninv), dev(wl.mask, torch.uint8))
    for k in (3, 300):
        a, m, _ = p64.solve(d, iters=k)
        b, q, _ = p32.solve(d, iters=k)
        ea, em = rel_alm(b.cpu().numpy(), a.cpu().numpy(), lmax), rel(q.cpu(), m.cpu())
        print("%d iterations: alm %.2e map %.2e" % (k, ea, em))
        assert ea < 1e-5 and em < 1e-5
