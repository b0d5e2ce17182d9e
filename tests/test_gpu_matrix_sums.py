"""Edges of the matrix-core sums: detectors around the tile sizes (blocks of 32 pixels
along one axis, packed rows along the other, thin and transposed detectors, single
pixels, blocks of 32 q rows on a polar one), point counts around the 4-point matrix step and the 32-point chunk, every
channel set and workgroup shape, against the FP64 oracle.

Tolerance, from the arithmetic: a phasor is a product of at most a few rounded
phasors whose phases are products rounded to |phase| 2^-53, and a sum of W terms
adds at most W roundings, so each amplitude is within
2^-52 (4 max|phase| + W + 128) sum|w| of the exact sum (the oracle's own error is of
the same form and smaller)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2601_18444_amd import numag, synth  # noqa: E402
from tests.helpers import amp_to_complex  # noqa: E402

DEV = "cuda:0"


@pytest.fixture(autouse=True)
def _clean_table():
    numag.tune_clear()
    yield
    numag.tune_clear()


def _check(orc, kind, n0, n1, W, chan, shape, path):
    rng = np.random.default_rng(1000 * n0 + 10 * n1 + W + chan)
    pos, nuc, mag = rng.uniform(-9, 9, (W, 3)), rng.standard_normal(W), rng.standard_normal((W, 3))
    qmax = 1.3
    R = synth.sample_rotation(33.0, 71.0)
    grid = numag.qgrid(kind, n0, n1, qmax)
    s = numag.Sample(pos=pos, nuc=nuc if chan != 2 else None, mag=mag if chan != 1 else None, device=DEV)
    if shape is not None:
        numag.tune_set(numag.TUNE_DIRECT, grid, W, shape, path=path)
    amp, _ = numag.amplitudes(s, grid, rot=R, path=path)
    qy, qz, _ = orc.pixels(kind, n0, n1, qmax)
    on, om = (nuc if chan != 2 else np.zeros(W)), (mag if chan != 1 else np.zeros((W, 3)))
    ref = orc.amplitudes(pos, on, om, qy, qz, R=R)
    phase = 2 * qmax * np.abs(pos).sum(1).max()
    w = np.concatenate([on[:, None], om @ R.T], axis=1)
    tol = 2.0 ** -52 * (4 * phase + W + 128) * np.abs(w).sum(0)
    err = np.abs(amp_to_complex(amp[0]) - ref).max(0)
    assert np.all(err <= tol), (err, tol)


@pytest.mark.parametrize("n0,n1", [(1, 1), (2, 1), (1, 2), (1, 700), (700, 1), (3, 300), (31, 33), (32, 32), (33, 65),
                                   (34, 31), (64, 257), (129, 35), (200, 130)])
@pytest.mark.parametrize("chan", [0, 1, 2])
def test_cartesian_tiles(orc, n0, n1, chan):
    for W, shape in [(1, None), (4, (8, 0)), (33, (64, 3)), (130, (16, 7)), (517, (32, 2)), (700, None)]:
        for path in (numag.PATH_DIRECT, numag.PATH_DIRECT_HERMITIAN):
            _check(orc, 0, n0, n1, W, chan, shape, path)


@pytest.mark.parametrize("n0,n1", [(1, 1), (1, 2), (2, 5), (31, 6), (32, 7), (33, 8), (65, 9), (150, 10), (257, 4),
                                   (512, 3), (513, 6), (1000, 5)])
@pytest.mark.parametrize("chan", [0, 1, 2])
def test_polar_tiles(orc, n0, n1, chan):
    """Row blocks of 32 q rows, up to 16 of them per wave, odd theta counts (every
    column summed) and even ones (half of them), point counts around the chunk."""
    shapes = [None, (0, 5), (2, 40), (3, 3), (4, 64)] + ([(1, 9)] if n0 <= 32 else [])
    for W, shape in zip([1, 31, 32, 33, 130, 517], shapes):
        for path in (numag.PATH_DIRECT, numag.PATH_DIRECT_HERMITIAN)[: 1 if n1 % 2 else 2]:
            _check(orc, 1, n0, n1, W, chan, shape, path)


@pytest.mark.parametrize("kind,n0,n1", [(0, 33, 40), (1, 40, 12)])
@pytest.mark.parametrize("scale", [1e-6, 1e4, 3e10])
def test_far_points(orc, kind, n0, n1, scale):
    """Phases from far below one turn to beyond the range of the fast phasor (2^30 half
    turns, where the library's sine and cosine take over); a non-finite position gives
    non-finite sums.  The tolerance grows with the phase as in _check."""
    rng = np.random.default_rng(5)
    W, qmax = 45, 1.3
    pos, nuc, mag = scale * rng.uniform(-1, 1, (W, 3)), rng.standard_normal(W), rng.standard_normal((W, 3))
    grid = numag.qgrid(kind, n0, n1, qmax)
    amp, _ = numag.amplitudes(numag.Sample(pos=pos, nuc=nuc, mag=mag, device=DEV), grid)
    qy, qz, _ = orc.pixels(kind, n0, n1, qmax)
    ref = orc.amplitudes(pos, nuc, mag, qy, qz)
    w = np.concatenate([nuc[:, None], mag], axis=1)
    tol = 2.0 ** -52 * (8 * qmax * scale + W + 128) * np.abs(w).sum(0)
    assert np.all(np.abs(amp_to_complex(amp[0]) - ref).max(0) <= tol)
    pos[7, 2] = np.inf
    bad, _ = numag.amplitudes(numag.Sample(pos=pos, nuc=nuc, mag=mag, device=DEV), grid)
    assert not torch.isfinite(bad[0, -1]).all()


@pytest.mark.parametrize("n0,n1", [(1, 1), (2, 31), (15, 2), (16, 32), (17, 33), (33, 64), (64, 95)])
@pytest.mark.parametrize("n", [(2, 1, 1), (3, 4, 17), (2, 33, 15)])
def test_separable_cells(orc, n0, n1, n):
    """Tiles of 8 x 16 cells, middle rows and columns, both channel splits of the second
    contraction (a large batch holds all channels in a wave), unaligned results."""
    rng = np.random.default_rng(100 * n0 + n1 + n[2])
    qmax, step, origin = 1.3, (1.1, 0.9, 1.2), (-1.0, -3.0, -8.0)
    W = n[0] * n[1] * n[2]
    B = 4 if n[2] != 17 else 180
    nuc, mag = rng.standard_normal((B, W)), rng.standard_normal((B, W, 3))
    grid, points = numag.qgrid(0, n0, n1, qmax), numag.regular_grid(n, origin, step)
    amp = numag.amplitudes_snapshots(points, grid, nuc=nuc, mag=mag, device=DEV)
    shifted = torch.empty(amp.numel() + 1, dtype=torch.float64, device=DEV)[1:].reshape(amp.shape)
    numag.amplitudes_snapshots(points, grid, nuc=nuc, mag=mag, device=DEV, out=shifted,
                               path=numag.PATH_SEPARABLE_F64_HERMITIAN)
    assert torch.equal(amp, shifted)
    one = numag.amplitudes_snapshots(points, grid, nuc=nuc[-1:], mag=mag[-1:], device=DEV)
    assert torch.equal(amp[-1:], one)
    pos = synth.box_lattice(n, step, origin)
    qy, qz, _ = orc.pixels(0, n0, n1, qmax)
    phase = qmax * (np.abs(pos[:, 1]).max() + np.abs(pos[:, 2]).max())
    for b in (0, B - 1):
        ref = orc.amplitudes(pos, nuc[b], mag[b], qy, qz)
        w = np.concatenate([nuc[b][:, None], mag[b]], axis=1)
        tol = 2.0 ** -52 * (4 * phase + W + 128) * np.abs(w).sum(0)
        assert np.all(np.abs(amp_to_complex(amp[b]) - ref).max(0) <= tol)


@pytest.mark.parametrize("chan", [0, 1, 2])
@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("n0,n1,W", [(5, 7, 1), (33, 20, 31), (48, 81, 33), (20, 300, 500), (64, 64, 4169)])
def test_points_straight_from_the_sample(kind, n0, n1, W, chan):
    """Small sums read and rotate the sample in the sum kernel; an object offset of
    zero sends the same points through their preparation."""
    rng = np.random.default_rng(W + chan)
    w = dict(nuc=rng.standard_normal(W) if chan != 2 else None, mag=rng.standard_normal((W, 3)) if chan != 1 else None)
    pos, R, grid = rng.uniform(-9, 9, (W, 3)), synth.sample_rotation(21.0, 64.0), numag.qgrid(kind, n0, n1, 1.3)
    one = numag.Sample(pos=pos, device=DEV, **w)
    off = numag.Sample(pos=pos, obj_pos=np.zeros((1, 3)), obj_offsets=[0, W], device=DEV, **w)
    a, _ = numag.amplitudes(one, grid, rot=R)
    b, _ = numag.amplitudes(off, grid, rot=R)
    size = sum(np.abs(x).sum() for x in w.values() if x is not None)
    assert (a - b).abs().max().item() <= 2.0 ** -52 * (8 * 2 * 1.3 * 9 * 2 + 2 * W + 256) * size


@pytest.mark.parametrize("n0", [1, 16, 17, 32, 33, 63, 64, 65, 96, 127, 128, 129])
@pytest.mark.parametrize("chan", [0, 1, 2])
def test_few_polar_rows(orc, n0, chan):
    """Detectors whose slots (blocks of 32 q rows times channels) fill one or two tiles of
    four rows, or just no longer: one point range and several, columns in pairs and not,
    several row groups.  To the tolerance above comes the rounding of the rotated moments,
    three products and two sums of |R| |m| on either side, which counts where they cancel."""
    few = 1 if n0 <= 32 else 0
    qmax, R = 1.3, synth.sample_rotation(33.0, 71.0)
    for W, shape in [(1, None), (5, (few, 0)), (33, (0, 5)), (130, (few, 40)), (700, None)]:
        for n1, path in ((4, numag.PATH_DIRECT), (9, numag.PATH_DIRECT), (10, numag.PATH_DIRECT_HERMITIAN)):
            rng = np.random.default_rng(1000 * n0 + 10 * n1 + W + chan)
            pos, nuc, mag = rng.uniform(-9, 9, (W, 3)), rng.standard_normal(W), rng.standard_normal((W, 3))
            grid = numag.qgrid(1, n0, n1, qmax)
            if shape is not None:
                numag.tune_set(numag.TUNE_DIRECT, grid, W, shape, path=path)
            s = numag.Sample(pos=pos, nuc=nuc if chan != 2 else None, mag=mag if chan != 1 else None, device=DEV)
            amp, _ = numag.amplitudes(s, grid, rot=R, path=path)
            qy, qz, _ = orc.pixels(1, n0, n1, qmax)
            on, om = (nuc if chan != 2 else np.zeros(W)), (mag if chan != 1 else np.zeros((W, 3)))
            ref = orc.amplitudes(pos, on, om, qy, qz, R=R)
            w = np.concatenate([on[:, None], om @ R.T], axis=1)
            m = np.concatenate([np.zeros((W, 1)), np.abs(om) @ np.abs(R).T], axis=1)
            phase = 2 * qmax * np.abs(pos).sum(1).max()
            tol = 2.0 ** -52 * ((4 * phase + W + 128) * np.abs(w).sum(0) + 3 * m.sum(0))
            err = np.abs(amp_to_complex(amp[0]) - ref).max(0)
            assert np.all(err <= tol), (W, n1, err, tol)


@pytest.mark.parametrize("n0", [1, 2, 15, 16, 17, 31, 32, 33, 64, 65])
@pytest.mark.parametrize("n1", [1, 2, 9, 12])
def test_gradient_of_few_polar_rows(orc, n0, n1):
    """One block of 32 q rows (tiles of four coefficient rows) and just more, columns in pairs
    and not, point counts around the 32 of a wave, several ranges of columns.  With S the sum
    of the weights' moduli, |F| <= S and I <= (1 + b^2) S^2; the gradient is a sum over pixels
    of 4 w (I - T) F times phasors, each factor within 2^-52 (4 phase + W + P + 128) of such a
    bound; four factors count."""
    qmax, bH, R = 1.3, 0.7, synth.sample_rotation(33.0, 71.0)
    grid, P = numag.qgrid(1, n0, n1, qmax), n0 * n1
    qy, qz, qhat = orc.pixels(1, n0, n1, qmax)
    for W, target in [(1, 0), (31, 3), (33, 0), (300, 40)]:
        rng = np.random.default_rng(1000 * n0 + 10 * n1 + W)
        pos, nuc, mag = rng.uniform(-9, 9, (W, 3)), rng.standard_normal(W), rng.standard_normal((W, 3))
        T, w = rng.uniform(0.0, 1.0, P), rng.uniform(0.5, 1.5, P)
        L, dn, dm = orc.loss_grad(pos, nuc, mag, qy, qz, qhat, T, w, bH=bH, R=R)
        s = numag.Sample(pos=pos, nuc=nuc, mag=mag, device=DEV)
        if target:
            numag.tune_set(numag.TUNE_ADJOINT, grid, W, (0, target))
        loss, gn, gm = numag.grad(s, grid, numag.consts(bH=bH), weight=torch.as_tensor(w, device=DEV),
                                  target=torch.as_tensor(T, device=DEV), rot=R)
        S = np.abs(nuc).sum() + np.abs(mag).sum()
        phase = 2 * qmax * np.abs(pos).sum(1).max()
        tol = 4 * 2.0 ** -52 * (4 * phase + W + P + 128) * (4 * w * ((1 + bH ** 2) * S ** 2 + T) * S).sum()
        assert np.abs(gn.cpu().numpy() - dn).max() <= tol and np.abs(gm.cpu().numpy() - dm).max() <= tol
        assert np.abs(dn).max() > 1e4 * tol  # the bound says something
        assert abs(loss.item() - L) <= 1e-9 * abs(L)
