"""The FP64 Legendre kernels walk each m in blocks of 16 values of l from l = m and start every
ring pair at its first block: band limits around the block length (a row of one block, a
full last block, one value past it), pair counts around a wave's lanes, and polar pairs that
start far above m, for every kernel shape, against the oracle.  Tolerance: the FP64 path's
1e-12 relative (its parity target)."""
import os

import numpy as np
import pytest
import torch

import oracle
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


@pytest.mark.parametrize("nside,lmax", [(1, 1), (4, 15), (8, 16), (8, 17), (16, 31), (32, 96), (64, 255), (128, 511)])
def test_block_edges_every_shape(mf, nside, lmax):
    rng = np.random.default_rng(100 * nside + lmax)
    alm = W.white_alm(rng, lmax)
    mp = rng.standard_normal(12 * nside * nside)
    ref_map, ref_alm = oracle.alm2map(nside, lmax, alm), oracle.map2alm(nside, lmax, mp)
    for v in range(9):
        spec = "synth=%d,ana=%d" % (v, min(v, 5))
        print("forced", spec, "nside", nside, "lmax", lmax, flush=True)
        os.environ["MFWF_TUNE_FORCE"] = spec
        try:
            plan = mf.Plan(nside, lmax, max_batch=2)
        finally:
            os.environ.pop("MFWF_TUNE_FORCE", None)
        # two maps, the second scaled: the map index of every launch
        m2 = plan.sht_inv(dev(np.stack([alm, -2.0 * alm]), torch.complex128)).cpu().numpy()
        a2 = plan.sht_fwd(dev(np.stack([mp, 0.5 * mp]))).cpu().numpy()
        for b, f in ((0, 1.0), (1, -2.0)):
            assert rel(m2[b], f * ref_map) < 1e-12, (spec, b)
        for b, f in ((0, 1.0), (1, 0.5)):
            assert rel_alm(a2[b], f * ref_alm, lmax) < 1e-12, (spec, b)


@pytest.mark.parametrize("nside,lmax", [(2, 2), (8, 17), (64, 159), (128, 300)])
def test_block_edges_pol(mf, nside, lmax):
    rng = np.random.default_rng(7 * nside + lmax)
    alm = np.stack([W.white_alm(rng, lmax) for _ in range(3)])
    ls, _ = W.alm_l_m(lmax)
    alm[1:, ls < 2] = 0.0  # E and B start at l = 2
    mp = rng.standard_normal((3, 12 * nside * nside))
    plan = mf.Plan(nside, lmax, spin=2)
    got = plan.sht_inv(dev(alm[None], torch.complex128)).cpu().numpy()[0]
    ref = oracle.alm2map_pol(nside, lmax, alm)
    back = plan.sht_fwd(dev(mp[None])).cpu().numpy()[0]
    refa = oracle.map2alm_pol(nside, lmax, mp)
    for c in range(3):
        assert rel(got[c], ref[c]) < 1e-12, c
        assert rel_alm(back[c], refa[c], lmax) < 1e-12, c
