"""Every tile of the batched form's contractions (32, 64 and 128 columns, lambda from the table and
generated), chosen by force on plans small enough to have ragged rows, ring pairs and columns, and
named by tuning(), which asks the rule that the launches ask; bitwise equal to each other (no
column depends on its tile) and against the FP64 path.

Tolerance of one transform: a product of two rounded FP32 operands and its rounding, 3 x 2^-24;
the piece products left out of it, 2^-27.5 rms and at most 2^-24; sums of 16 products rounded at
most 6 times and added one by one (lmax + 1 or 2 nside terms), all of random sign: relative to
the norm 2^-24 (3 + 6 + sqrt(nside / 8 + 1)) + 2^-27, under 1e-6 for nside 64."""
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


def plan_of(mf, spec, *a, **k):
    if spec:
        os.environ["MFWF_TUNE_FORCE"] = spec
    try:
        return mf.Plan(*a, **k)
    finally:
        os.environ.pop("MFWF_TUNE_FORCE", None)


# (lmax + 1 off 64, 128 and 256; ring pairs 32, 64, 128, 256 in chunks of 32 and tiles of 128; columns of
# 5, 37, 70 maps: one 32-column tile, 96 = 64 + 32, 160 = 128 + 32)
@pytest.mark.parametrize("nside,lmax,nmaps", [(16, 37, 5), (32, 93, 37), (64, 150, 70), (128, 300, 37)])
def test_every_temperature_tile(mf, nside, lmax, nmaps):
    rng = np.random.default_rng(nside * lmax + nmaps)
    alm = dev(np.stack([W.white_alm(rng, lmax) for _ in range(nmaps)]), torch.complex128)
    mp = dev(rng.standard_normal((nmaps, 12 * nside * nside)))
    p64 = mf.Plan(nside, lmax, max_batch=nmaps)
    ref_m, ref_a = p64.sht_inv(alm), p64.sht_fwd(mp)
    first = None
    specs = ["cta=%d,cts=%d,lamgen=%d" % (a, s, g) for g in (0, 1) for a, s in ((1, 1), (2, 2), (3, 1))]
    for spec in ["lamgen=0", "lamgen=1"] + specs:
        print("forced", spec, nside, lmax, nmaps, flush=True)
        p = plan_of(mf, spec, nside, lmax, max_batch=nmaps, dtype="f32")
        t = p.tuning()
        assert t["lamgen"] == int(spec[-1])
        if "cta" in spec:
            assert (t["cta"], t["cts"]) == (int(spec[4]), int(spec[10])), t
        else:  # 32 columns below 1200 tiles of 64 (nside 128: 301 m x 2 pair tiles x 2 column groups)
            assert (t["cta"], t["cts"]) == (3, 2 if nside == 128 else 3), t
        m, a = p.sht_inv(alm), p.sht_fwd(mp)
        assert rel(m.cpu(), ref_m.cpu()) < 1e-6 and rel_alm(a.cpu().numpy(), ref_a.cpu().numpy(), lmax) < 1e-6, spec
        first = first or (m, a)
        assert torch.equal(m, first[0]) and torch.equal(a, first[1]), spec


# 4 columns a map for F+ and F- (south rings flipped, Q and U combined in the synthesis), 2 for T
@pytest.mark.parametrize("nside,lmax,nmaps", [(16, 37, 3), (32, 93, 21), (64, 150, 33)])
def test_every_polarization_tile(mf, nside, lmax, nmaps):
    rng = np.random.default_rng(nside * lmax + nmaps)
    ls = W.alm_l_m(lmax)[0]
    a0 = np.stack([[W.white_alm(rng, lmax) for _ in range(3)] for _ in range(nmaps)])
    a0[:, 1:, ls < 2] = 0.0  # E and B start at l = 2
    alm, mp = dev(a0, torch.complex128), dev(rng.standard_normal((nmaps, 3, 12 * nside * nside)))
    p64 = mf.Plan(nside, lmax, max_batch=nmaps, spin=2)
    ref_m, ref_a = p64.sht_inv(alm).cpu().numpy(), p64.sht_fwd(mp).cpu().numpy()
    first = None
    for spec in ["", "cta=1,cts=1", "cta=2,cts=2", "cta=3,cts=1"]:
        print("forced", spec, nside, lmax, nmaps, flush=True)
        p = plan_of(mf, spec, nside, lmax, max_batch=nmaps, spin=2, dtype="f32")
        t = p.tuning()
        assert (t["cta"], t["cts"]) == ((int(spec[4]), int(spec[10])) if spec else (3, 3)), t
        m, a = p.sht_inv(alm), p.sht_fwd(mp)
        for c in range(3):
            assert rel(m.cpu().numpy()[:, c], ref_m[:, c]) < 1e-6, (spec, c)
            assert rel_alm(a.cpu().numpy()[:, c], ref_a[:, c], lmax) < 1e-6, (spec, c)
        first = first or (m, a)
        assert torch.equal(m, first[0]) and torch.equal(a, first[1]), spec


# tables of 8 MB (cached loads) and 321 MB (streaming loads where one column group reads them)
@pytest.mark.parametrize("nside,lmax", [(64, 128), (256, 512)])
def test_table_of_several_column_groups(mf, nside, lmax):
    """80 maps in tiles of 64 columns (three groups) and of 128 (two), 30 maps at a time in one tile,
    the same bits."""
    rng = np.random.default_rng(1)
    alm = dev(np.stack([W.white_alm(rng, lmax) for _ in range(80)]), torch.complex128)
    out = []
    for spec in ("cta=1,cts=1", "cta=2,cts=2"):
        p = plan_of(mf, spec, nside, lmax, max_batch=80, dtype="f32")
        out.append(p.sht_inv(alm))
        out.append(torch.cat([p.sht_inv(alm[k:k + 30]) for k in (0, 30, 60)]))
    for o in out[1:]:
        assert torch.equal(o, out[0])


# 701 values of m: 1335 tiles of 256 rows, so that the columns decide: 40 padded to 64, and 32
@pytest.mark.parametrize("nmaps,cta", [(20, 2), (16, 3)])
def test_generated_analysis_above_32_columns(mf, nmaps, cta):
    nside, lmax = 256, 700
    mp = dev(np.random.default_rng(2).standard_normal((nmaps, 12 * nside * nside)))
    p, q = (plan_of(mf, spec, nside, lmax, max_batch=nmaps, dtype="f32") for spec in ("lamgen=1", "lamgen=0,cta=1"))
    assert p.tuning()["cta"] == cta
    assert torch.equal(p.sht_fwd(mp), q.sht_fwd(mp))
