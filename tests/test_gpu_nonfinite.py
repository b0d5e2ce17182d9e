"""Infinite weights: a sum is what its terms w cos(q.X), -w sin(q.X) make it -- infinite
where they agree in sign, NaN where they do not or where an infinite weight meets a sine of
zero -- on every route of the forward sums, and the other channels are untouched.  Parts
whose cosine or sine is below 1e-9 are not compared (their sign is the phase's rounding)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2601_18444_amd import numag, synth  # noqa: E402

DEV = "cuda:0"
QMAX = 1.3


def _terms(w, a, b):
    """Sums over the infinite weights of w cos, -w sin of the phase a + b, and where a part is
    well conditioned: its sine or cosine not small, or zero because a and b are."""
    c, s = np.cos(a + b), -np.sin(a + b)
    zero = (a == 0.0) & (b == 0.0)
    with np.errstate(invalid="ignore"):
        re, im = (w * c).sum(-1), (w * np.where(zero, 0.0, s)).sum(-1)
    return re, im, np.abs(c).min(-1) > 1e-9, (np.where(zero, 1.0, np.abs(s)) > 1e-9).all(-1)


def _same(got, ref, ok):
    assert np.array_equal(np.isnan(got[ok]), np.isnan(ref[ok]))
    fin = ok & ~np.isnan(ref)
    assert np.array_equal(got[fin], ref[fin])  # infinities with their signs


def _case(W, infs, seed):
    rng = np.random.default_rng(seed)
    pos, nuc, mag = rng.uniform(-9, 9, (W, 3)), rng.standard_normal(W), rng.standard_normal((W, 3))
    at = rng.choice(W, len(infs), replace=False)
    nuc[at] = infs
    return pos, nuc, mag, at


@pytest.mark.parametrize("kind,n0,n1", [(0, 9, 14), (0, 40, 33), (1, 9, 7), (1, 40, 8), (1, 600, 6)])
@pytest.mark.parametrize("W", [3, 45, 3000])
@pytest.mark.parametrize("infs", [[np.inf], [np.inf, -np.inf], [np.nan]])
@pytest.mark.parametrize("route", ["sample", "records", "noalloc", "half", "nuclear"])
def test_coherent_sums(orc, kind, n0, n1, W, infs, route):
    if route == "half" and kind == 1 and n1 % 2:
        pytest.skip("the half path needs an even n_theta")
    pos, nuc, mag, at = _case(W, infs, W + n0)
    R, grid = synth.sample_rotation(33.0, 71.0), numag.qgrid(kind, n0, n1, QMAX)
    kw = dict(obj_pos=np.zeros((1, 3)), obj_offsets=[0, W]) if route == "records" else {}
    chans = dict(nuc=nuc) if route == "nuclear" else dict(nuc=nuc, mag=mag)
    s = numag.Sample(pos=pos, device=DEV, **chans, **kw)
    path = numag.PATH_DIRECT_HERMITIAN if route == "half" else numag.PATH_DIRECT
    amp = numag.amplitudes_noalloc(s, grid, rot=R) if route == "noalloc" else numag.amplitudes(s, grid, rot=R, path=path)[0]
    a = amp[0].cpu().numpy()  # [P, 4, 2] (a complex product of an infinite part would add NaN)
    qy, qz, _ = orc.pixels(kind, n0, n1, QMAX)
    X = pos[at] @ R.T
    re, im, okr, oki = _terms(nuc[at], qy[:, None] * X[:, 1], qz[:, None] * X[:, 2])
    _same(a[:, 0, 0], re, okr)
    _same(a[:, 0, 1], im, oki)
    finite = dict(chans, nuc=np.where(np.isfinite(nuc), nuc, 0.0))
    s0 = numag.Sample(pos=pos, device=DEV, **finite, **kw)
    b = numag.amplitudes_noalloc(s0, grid, rot=R) if route == "noalloc" else numag.amplitudes(s0, grid, rot=R, path=path)[0]
    assert torch.equal(amp[:, :, 1:], b[:, :, 1:])


@pytest.mark.parametrize("kind,n0,n1", [(0, 9, 14), (0, 70, 33), (1, 9, 7), (1, 70, 8), (1, 300, 4)])
@pytest.mark.parametrize("mode", [numag.MODE_DILUTE, numag.MODE_SPLIT])
def test_objects(orc, kind, n0, n1, mode):
    """|F_N|^2 of the object that holds the infinite weight is infinite (NaN where a part of
    F_N is), the coherent total's channel N follows the terms, and the magnetic entries and
    the other objects are untouched."""
    sizes = [40, 3, 130]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    W = int(off[-1])
    rng = np.random.default_rng(n0)
    pos, nuc, mag = rng.uniform(-9, 9, (W, 3)), rng.standard_normal(W), rng.standard_normal((W, 3))
    opos = rng.uniform(-20, 20, (3, 3)) if mode == numag.MODE_SPLIT else None
    j = 60  # in object 2
    R, grid = synth.sample_rotation(33.0, 71.0), numag.qgrid(kind, n0, n1, QMAX)

    def run(x):
        s = numag.Sample(pos=pos, nuc=x, mag=mag, obj_offsets=off, obj_pos=opos, device=DEV)
        return numag.amplitudes(s, grid, rot=R, mode=mode, spec_per_object=mode == numag.MODE_DILUTE)

    bad = nuc.copy()
    bad[j] = np.inf
    amp, spec = run(bad)
    amp0, spec0 = run(nuc)
    qy, qz, _ = orc.pixels(kind, n0, n1, QMAX)
    x = R @ pos[j]
    phase = qy * x[1] + qz * x[2]
    zero = phase == 0.0  # q = 0: the imaginary part is NaN
    sp = spec.cpu().numpy()[2 if mode == numag.MODE_DILUTE else 0]
    assert np.array_equal(np.isnan(sp[:, 0]), zero)
    assert np.all(np.isinf(sp[~zero, 0]))
    magnetic = [1, 2, 3, 10, 11, 12, 13, 14, 15]
    assert torch.equal(spec[..., magnetic], spec0[..., magnetic])
    if mode == numag.MODE_DILUTE:
        assert torch.equal(spec[:2], spec0[:2])
    else:
        # the object's phase mixes an infinite real and imaginary part: NaN or infinite
        assert not torch.isfinite(amp[0, :, 0]).any()
        assert torch.equal(amp[0, :, 1:], amp0[0, :, 1:])


@pytest.mark.parametrize("kd,n0,n1", [(0, 6, 9), (0, 40, 33), (1, 6, 9), (1, 40, 8)])
@pytest.mark.parametrize("kr,r0,r1", [(0, 5, 6), (0, 40, 37), (1, 5, 7), (1, 40, 6)])
@pytest.mark.parametrize("m", [1, 3, 5])
@pytest.mark.parametrize("infs", [[np.inf], [np.inf, -np.inf], [np.nan]])
def test_correlation_2d(orc, kd, n0, n1, kr, r0, r1, m, infs):
    rng = np.random.default_rng(n0 + r0 + m)
    grid, rgrid = numag.qgrid(kd, n0, n1, QMAX), numag.qgrid(kr, r0, r1, 7.0)
    f = rng.uniform(0.5, 2.0, (m, n0 * n1))
    clean = numag.correlation_2d(grid, torch.as_tensor(f, device=DEV), rgrid)
    at = n1 + rng.choice(n0 * n1 - n1, len(infs), replace=False)  # (q = 0 has no weight on a polar detector)
    f[m - 1, at] = infs
    C = numag.correlation_2d(grid, torch.as_tensor(f, device=DEV), rgrid)
    qy, qz, _ = orc.pixels(kd, n0, n1, QMAX)
    ry, rz, _ = orc.pixels(kr, r0, r1, 7.0)
    re, im, okr, oki = _terms(f[m - 1, at], -ry[:, None] * qy[at], -rz[:, None] * qz[at])
    got = C[m - 1].cpu().numpy()
    _same(got[:, 0], re, okr)
    _same(got[:, 1], im, oki)
    assert torch.equal(C[: m - 1], clean[: m - 1])


@pytest.mark.parametrize("kd,n0,n1", [(0, 6, 9), (0, 40, 33), (1, 6, 9), (1, 40, 8)])
@pytest.mark.parametrize("kr,r0,r1", [(0, 5, 6), (0, 40, 37), (1, 5, 7), (1, 40, 6)])
@pytest.mark.parametrize("m", [1, 3, 5])
@pytest.mark.parametrize("infs", [[np.inf], [np.inf, -np.inf], [np.nan]])
def test_correlation_2d(orc, kd, n0, n1, kr, r0, r1, m, infs):
    rng = np.random.default_rng(n0 + r0 + m)
    grid, rgrid = numag.qgrid(kd, n0, n1, QMAX), numag.qgrid(kr, r0, r1, 7.0)
    f = rng.uniform(0.5, 2.0, (m, n0 * n1))
    clean = numag.correlation_2d(grid, torch.as_tensor(f, device=DEV), rgrid)
    at = n1 + rng.choice(n0 * n1 - n1, len(infs), replace=False)  # (q = 0 has no weight on a polar detector)
    f[m - 1, at] = infs
    C = numag.correlation_2d(grid, torch.as_tensor(f, device=DEV), rgrid)
    qy, qz, _ = orc.pixels(kd, n0, n1, QMAX)
    ry, rz, _ = orc.pixels(kr, r0, r1, 7.0)
    re, im, okr, oki = _terms(f[m - 1, at], -ry[:, None] * qy[at], -rz[:, None] * qz[at])
    got = C[m - 1].cpu().numpy()
    _same(got[:, 0], re, okr)
    _same(got[:, 1], im, oki)
    assert torch.equal(C[: m - 1], clean[: m - 1])


@pytest.mark.parametrize("kind,n0,n1", [(0, 9, 14), (0, 40, 33), (1, 9, 7), (1, 40, 8)])
@pytest.mark.parametrize("what", ["weight", "target", "upstream", "two"])
@pytest.mark.parametrize("path", [numag.PATH_DIRECT, numag.PATH_DIRECT_HERMITIAN])
def test_gradient(orc, kind, n0, n1, what, path):
    """The gradient with an infinite loss weight, target or upstream gradient at one pixel (or
    two): each point's sums are what those pixels' terms Re(a exp(-i q.X)) make them."""
    if path == numag.PATH_DIRECT_HERMITIAN and kind == 1 and n1 % 2:
        pytest.skip("the half path needs an even n_theta")
    W = 200
    pos, nuc, mag, _ = _case(W, [], 7 + n0)
    R, grid, c = synth.sample_rotation(33.0, 71.0), numag.qgrid(kind, n0, n1, QMAX), numag.consts(V=2.0, bH=0.7)
    s = numag.Sample(pos=pos, nuc=nuc, mag=mag, device=DEV)
    amp = numag.amplitudes(s, grid, rot=R, path=path)[0][0]
    A = amp.cpu().numpy()
    rng = np.random.default_rng(n1)
    w, T = rng.uniform(0.5, 1.5, n0 * n1), rng.uniform(0.0, 1.0, n0 * n1)
    at = [2 * n1 + 3] if what != "two" else [2 * n1 + 3, 5 * n1 + 2]
    (T if what == "target" else w)[at] = np.inf
    tgt = None if what == "upstream" else torch.as_tensor(T, device=DEV)
    _, dn, dm = numag.grad(s, grid, c, weight=torch.as_tensor(w, device=DEV), target=tgt, rot=R, amp=amp, path=path)
    qy, qz, qh = orc.pixels(kind, n0, n1, QMAX)
    X = pos @ R.T
    g = np.zeros((W, 4))
    ok = np.ones(W, dtype=bool)
    with np.errstate(invalid="ignore"):
        for p in at:
            qhat = qh[p]
            M = A[p, 1:, 0] + 1j * A[p, 1:, 1]
            V = M - qhat * (qhat @ M)
            cf = 1.0 / 2.0
            I = cf * (A[p, 0] @ A[p, 0] + 0.49 * np.vdot(V, V).real)
            G = 2.0 * cf * (w[p] if what == "upstream" else 2.0 * w[p] * (I - T[p]))
            ar = np.concatenate([[G * A[p, 0, 0]], G * 0.49 * V.real])
            ai = -np.concatenate([[G * A[p, 0, 1]], G * 0.49 * V.imag])
            phi = qy[p] * X[:, 1] + qz[p] * X[:, 2]
            g += ar[None] * np.cos(phi)[:, None] + ai[None] * np.sin(phi)[:, None]
            ok &= (np.abs(np.cos(phi)) > 1e-9) & (np.abs(np.sin(phi)) > 1e-9)
        _same(dn.cpu().numpy(), g[:, 0], ok)
        ref = np.stack([R[0, b] * g[:, 1] + R[1, b] * g[:, 2] + R[2, b] * g[:, 3] for b in range(3)], axis=1)
    _same(dm.cpu().numpy(), ref, np.broadcast_to(ok[:, None], ref.shape))
