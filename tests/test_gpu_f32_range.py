"""The batched FP32 form at the ends of FP32's range.  Its contractions split every FP32 operand
into three bf16 pieces, and the last piece of a value below 2^-110 lies below bf16's smallest
number; the columns of a map of small values therefore carry them times a power of two.
Transforms, sources and solves of maps scaled by 2^-90 .. 2^-122 (normal FP32 numbers, whose 24
bits the form keeps), alone and beside maps of ordinary size, zero maps and maps near FP32's
largest values, against the FP64 path.

Tolerance: scaling by a power of two changes no rounding of either path until FP32 values fall
below 2^-126; the coefficients that do are rounded to 2^-149, 2^-27 of a map of 2^-122.  So
the tolerances are those of ordinary maps: 1e-6 for one transform (a product of two rounded FP32
operands within 3 x 2^-24 and what the piece products leave out, 2^-23, sums of random sign), 1e-5
for solves (the form's accuracy target)."""
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


# per map: ordinary, small, the smallest whose values are normal numbers, zero, large
SCALES = [1.0, 2.0 ** -90, 2.0 ** -122, 0.0, 2.0 ** 110]


def alm_of(rng, lmax, ncomp):
    a = np.stack([W.white_alm(rng, lmax) for _ in range(ncomp)])
    if ncomp == 3:
        a[1:, W.alm_l_m(lmax)[0] < 2] = 0.0  # E and B start at l = 2
    return a


def check(got, ref, scales, tol, err):
    for b, s in enumerate(scales):
        if s == 0.0:
            assert not np.any(got[b])
        else:
            for c in range(got.shape[1]):
                e = err(got[b, c] / s, ref[b, c] / s)
                assert e < tol, (b, c, s, e)


@pytest.mark.parametrize("nside,lmax,spin", [(16, 31, 0), (64, 128, 0), (16, 32, 2), (64, 100, 2)])
def test_transforms(mf, nside, lmax, spin):
    rng = np.random.default_rng(nside + spin)
    nc, n = (3 if spin else 1), len(SCALES)
    a = np.stack([s * alm_of(rng, lmax, nc) for s in SCALES])
    m = np.stack([s * rng.standard_normal((nc, 12 * nside * nside)) for s in SCALES])
    if spin:  # an ordinary T beside small Q and U, and the other way round
        a[0, 1:] *= 2.0 ** -120
        m[0, 1:] *= 2.0 ** -120
        a[1, 0] *= 2.0 ** 80
        m[1, 0] *= 2.0 ** 80
    sh = (lambda x: x) if spin else (lambda x: x[:, 0])
    p64, p32 = mf.Plan(nside, lmax, max_batch=n, spin=spin), mf.Plan(nside, lmax, max_batch=n, spin=spin, dtype="f32")
    ad, md = dev(sh(a), torch.complex128), dev(sh(m))
    back = lambda x: x.cpu().numpy().reshape(n, nc, -1)  # noqa: E731
    for _ in range(2):  # the second call finds the first one's scales in the plan
        check(back(p32.sht_inv(ad)), back(p64.sht_inv(ad)), SCALES, 1e-6, rel)
        check(back(p32.sht_fwd(md)), back(p64.sht_fwd(md)), SCALES, 1e-6, lambda x, y: rel_alm(x, y, lmax))
        ad, md = ad.flip(0).contiguous(), md.flip(0).contiguous()
        check(back(p32.sht_inv(ad)), back(p64.sht_inv(ad)), SCALES[::-1], 1e-6, rel)
        ad, md = ad.flip(0).contiguous(), md.flip(0).contiguous()


@pytest.mark.parametrize("spin,chained", [(0, True), (0, False), (2, True), (2, False)])
def test_solves(mf, spin, chained):
    nside, lmax = 32, 64
    rng = np.random.default_rng(7)
    nc, n = (3 if spin else 1), len(SCALES)
    npix = 12 * nside * nside
    d = np.stack([s * (3.0 * np.sin(np.arange(npix) * 1e-3) + rng.standard_normal((nc, npix))) for s in SCALES])
    cl = W.cl_damped(lmax, 30.0)
    ninv = rng.uniform(0.5, 2.0, npix)
    ninv[: npix // 3] = 0.0
    if spin:
        cl = W.pol_cls(cl)
        n6 = np.zeros((npix, 6))
        n6[:, 0], n6[:, 3], n6[:, 5] = ninv, 0.5 * ninv, 0.5 * ninv
        ninv = n6
    out = []
    for dtype in ("f64", "f32"):
        p = mf.Plan(nside, lmax, max_batch=n, spin=spin, dtype=dtype)
        p.set_covariances(cl, dev(ninv))
        x = dev(d if spin else d[:, 0])
        s, m, info = p.solve(x, lam=[20.0, 1.0], iters=[6, 9], chained=chained)
        out.append((s.cpu().numpy().reshape(n, nc, -1), m.cpu().numpy().reshape(n, nc, -1), [i.snorm for i in info]))
    assert out[1][2] == pytest.approx(out[0][2], rel=1e-5)
    check(out[1][0], out[0][0], SCALES, 1e-5, lambda x, y: rel_alm(x, y, lmax))
    check(out[1][1], out[0][1], SCALES, 1e-5, rel)


def test_sources(mf):
    """Realization sources whose C^-1/2 h is small (large C_l)."""
    nside, lmax, n = 32, 64, 2
    rng = np.random.default_rng(8)
    npix, u = 12 * nside * nside, 2.0 ** 118
    h = np.stack([W.white_alm(rng, lmax) for _ in range(n)])
    ref = []
    for dtype in ("f64", "f32"):
        p = mf.Plan(nside, lmax, max_batch=n, dtype=dtype)
        p.set_covariances(W.cl_damped(lmax, 30.0) * u * u, dev(np.full(npix, 1.0 / (u * u))))
        ref.append(p.fluctuation_rhs(dev(np.zeros((n, npix))), dev(h, torch.complex128)).cpu().numpy() * u)
    assert rel(ref[1], ref[0]) < 1e-6


@pytest.mark.parametrize("spin,call", [(0, "solve_cooled"), (0, "solve_bounded"), (2, "solve_cooled")])
def test_solves_do_not_depend_on_the_units(mf, spin, call):
    """Data, noise and signal in units where the maps are of size 2^-118: chi^2, and with it the
    schedule, is the same as in ordinary units, and so is the result (FP32 values below 2^-126
    are rounded to 2^-149, 2^-31 of the maps, in each of at most 60 iterations: 3e-8)."""
    nside, lmax, n = 32, 48, 2
    rng = np.random.default_rng(8)
    npix, nc = 12 * nside * nside, 3 if spin else 1
    d = 3.0 * np.sin(np.arange(npix) * 1e-3) + rng.standard_normal((n, nc, npix))
    ninv = rng.uniform(0.5, 2.0, npix)
    ninv[: npix // 3] = 0.0
    cl = W.cl_damped(lmax, 30.0)
    if spin:
        cl = W.pol_cls(cl)
        n6 = np.zeros((npix, 6))
        n6[:, 0], n6[:, 3], n6[:, 5] = ninv, 0.5 * ninv, 0.5 * ninv
        ninv = n6
    out = []
    for v in (1.0, 2.0 ** -118):
        p = mf.Plan(nside, lmax, max_batch=n, spin=spin, dtype="f32")
        p.set_covariances(cl * v * v, dev(ninv / (v * v)))
        r = getattr(p, call)(dev((d if spin else d[:, 0]) * v), max_iters=60)
        out.append((r[0].cpu().numpy() / v, r[1].cpu().numpy() / v, r[2][0].iters_done))
    assert out[0][2] == out[1][2]
    assert rel_alm(out[1][0], out[0][0], lmax) < 1e-6 and rel(out[1][1], out[0][1]) < 1e-6


def test_serving_slot(mf):
    """A request of small values and, in the same slot after it, one of ordinary size."""
    nside, lmax = 32, 64
    rng = np.random.default_rng(9)
    npix = 12 * nside * nside
    cl = W.cl_damped(lmax, 30.0)
    p = mf.Plan(nside, lmax)
    srv = mf.Server(slots=1, hbm_gb=50.0)
    for s in (2.0 ** -118, 1.0, 2.0 ** -90):
        d = s * (3.0 * np.sin(np.arange(npix) * 1e-3) + rng.standard_normal(npix))
        ninv = dev(rng.uniform(0.5, 2.0, npix))
        p.set_covariances(cl, ninv)
        a, m, _ = p.solve(dev(d[None]), iters=9)
        rid, sa, sm = srv.submit(nside, lmax, cl, ninv, dev(d), dtype="f32", iters=9)
        srv.wait(rid)
        assert rel_alm(sa.cpu().numpy().reshape(-1) / s, a.cpu().numpy()[0] / s, lmax) < 1e-5, s
        assert rel(sm.cpu().numpy().reshape(-1) / s, m.cpu().numpy()[0] / s) < 1e-5, s
    srv.close()
