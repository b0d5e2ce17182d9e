"""Edges of the map analysis kernels: lanes of a row, wave and workgroup remainders, groups
of data sets, empty bins.  Tolerances are the rounding of sums of n terms in 64 bits."""
import numpy as np
import pytest
import torch

from paper_2601_18444_amd import numag

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
EPS = 2.0 ** -52


@pytest.mark.parametrize("n0,n1", [(1, 9), (2, 2), (17, 64), (33, 40), (130, 257)])
@pytest.mark.parametrize("n_f,n_bins,frac", [(1, 1, 1.0), (4, 7, 0.7), (5, 33, 1.0), (13, 64, 1.5)])
def test_azimuthal_groups(orc, n0, n1, n_f, n_bins, frac):
    rng = np.random.default_rng(n0 + 7 * n_f)
    f = rng.standard_normal((n_f, n0 * n1))
    grid = numag.qgrid(0, n0, n1, 1.3)
    I, count = numag.azimuthal_average(grid, torch.as_tensor(f, device=DEV), n_bins, 1.3 * frac)
    Iref, cref = orc.azimuthal_average(0, n0, n1, 1.3, f, n_bins, 1.3 * frac)
    assert np.array_equal(count.cpu().numpy(), cref)
    I = I.cpu().numpy()
    assert np.array_equal(np.isnan(I), np.isnan(Iref))
    some = cref > 0
    assert np.all(np.abs(I - Iref)[:, some] <= EPS * n0 * n1 * np.abs(f).max())


@pytest.mark.parametrize("n_q", [1, 63, 64, 65, 128, 200])
@pytest.mark.parametrize("empty", ["none", "some", "block", "all"])
def test_correlation_empty_bins(orc, n_q, empty):
    rng = np.random.default_rng(n_q)
    q = np.sort(rng.uniform(0.0, 2.0, n_q))
    I = rng.uniform(0.5, 2.0, (3, n_q))
    if empty == "some":
        I[:, rng.uniform(size=n_q) < 0.3] = np.nan
    elif empty == "block":
        I[1, n_q // 3: n_q // 3 + 66] = np.nan
    elif empty == "all":
        I[2] = np.nan
    r = np.concatenate([[0.0], rng.uniform(0.1, 50.0, 6)])
    c, p = numag.correlation(*(torch.as_tensor(x, device=DEV) for x in (q, I, r)))
    cref, pref = orc.correlation(q, I, r)
    # the sum of |terms| is at most q_max max(I q^2); a sine's argument carries q r eps
    tol = EPS * (n_q + 60.0 * 2) * 2.0 * 2.0 * 4.0
    assert np.all(np.abs(c.cpu().numpy() - cref) <= tol)
    assert np.all(np.abs(p.cpu().numpy() - pref) <= tol * r * r)


@pytest.mark.parametrize("n_q,n_theta", [(1, 1), (3, 63), (65, 64), (130, 131)])
@pytest.mark.parametrize("k_max", [0, 3, 4, 9])
def test_angular_orders(orc, n_q, n_theta, k_max):
    rng = np.random.default_rng(n_q + k_max)
    f = rng.standard_normal((2, n_q * n_theta))
    Is, Ic, As, Ac = (x.cpu().numpy() for x in numag.angular_spectrum(
        numag.qgrid(1, n_q, n_theta, 1.0), torch.as_tensor(f, device=DEV), k_max))
    for s in range(2):
        Isr, Icr = orc.angular_spectrum(f[s], n_q, n_theta, k_max)
        # a column's weight is h / pi; its phase k theta <= 2 pi k_max carries its own rounding
        tol = 2 * EPS * (n_theta + 8 * k_max + 8) * np.abs(f).max()
        assert np.abs(Is[s] - Isr).max() <= tol and np.abs(Ic[s] - Icr).max() <= tol
        Asr, Acr = orc.modal_amplitudes(Isr, Icr)
        norm = np.sqrt(Isr.sum(0) ** 2 + Icr.sum(0) ** 2).sum()
        rel = 4 * n_q * (k_max + 1) * (tol + EPS) / norm
        assert np.abs(As[s] - Asr).max() <= rel and np.abs(Ac[s] - Acr).max() <= rel


@pytest.mark.parametrize("kind,n0,n1", [(0, 1, 1), (0, 1, 8), (0, 9, 2), (0, 33, 65), (1, 2, 2), (1, 35, 4), (1, 40, 66),
                                        (1, 12, 15)])
@pytest.mark.parametrize("rkind,r0,r1", [(0, 1, 1), (0, 17, 34), (1, 1, 3), (1, 33, 6), (1, 150, 9), (1, 500, 2)])
def test_correlation_2d_routes(orc, kind, n0, n1, rkind, r0, r1):
    """Factored, paired and plain sums, one to five data sets: single rows and columns,
    detectors with and without a middle pixel, row blocks of the polar real-space grid."""
    rng = np.random.default_rng(n0 + 3 * n1 + r0)
    qmax, rmax = 1.1, 30.0
    grid, rgrid = numag.qgrid(kind, n0, n1, qmax), numag.qgrid(rkind, r0, r1, rmax)
    f = rng.standard_normal((5, n0 * n1))
    area = np.pi * qmax ** 2 if kind else (2 * qmax if n0 > 1 else 1) * (2 * qmax if n1 > 1 else 1)
    # sums of n terms |wq f| <= wq max|f| of phases up to 4 qmax rmax
    tol = EPS * (16 * qmax * rmax + n0 * n1 + 128) * area * np.abs(f).max()
    for n_f in (1, 2, 3, 4, 5):
        C = numag.correlation_2d(grid, torch.as_tensor(f[:n_f], device=DEV), rgrid).cpu().numpy()
        ref = orc.correlation_2d(kind, n0, n1, qmax, f[:n_f], rkind, r0, r1, rmax)
        assert np.abs(C[..., 0] + 1j * C[..., 1] - ref).max() <= tol


def test_correlation_of_more_results_than_a_grid_of_waves():
    """2^26 and more results: with a wave for each, their threads pass 2^32."""
    n_f, n_r = 8192, 8193
    q = torch.tensor([0.1, 0.25], dtype=torch.float64, device=DEV)
    I = torch.linspace(0.5, 2.0, n_f * 2, dtype=torch.float64, device=DEV).reshape(n_f, 2)
    r = torch.linspace(0.0, 5.0, n_r, dtype=torch.float64, device=DEV)
    c, p = numag.correlation(q, I, r)
    x = q[:, None] * r[None]
    j0 = torch.where(x == 0, torch.ones_like(x), torch.sin(x) / torch.where(x == 0, torch.ones_like(x), x))
    y = q[:, None] ** 2 * j0
    ref = (0.5 * I[:, :1] * (0.1 + 0.15) * y[0] + 0.5 * I[:, 1:] * 0.15 * y[1]) / (2.0 * np.pi ** 2)
    # two samples: every rounding is of the size of the terms, at most 2 q^2
    assert (c - ref).abs().max().item() <= 64 * EPS
    assert (p - r * r * ref).abs().max().item() <= 64 * EPS * 25.0


def test_azimuthal_of_more_bins_than_a_grid_of_workgroups():
    n_bins = (1 << 23) + 3
    f = torch.linspace(1.0, 2.0, 16, dtype=torch.float64, device=DEV)[None]
    I, count = numag.azimuthal_average(numag.qgrid(0, 4, 4, 1.0), f, n_bins, 1.5)
    assert int(count.sum()) == 16 and int(count.min()) == 0
    assert torch.equal(torch.isnan(I[0]), count == 0)
    mean = torch.where(count > 0, I[0], torch.zeros_like(I[0]))
    assert abs((mean * count).sum().item() - f.sum().item()) <= 64 * EPS * 16


def test_angular_spectrum_of_more_rows_than_a_grid_of_workgroups():
    n_q = (1 << 24) + 5
    f = torch.linspace(1.0, 2.0, 2 * n_q, dtype=torch.float64, device=DEV)[None]
    Is, Ic, _, _ = numag.angular_spectrum(numag.qgrid(1, n_q, 2, 1.0), f, 0, amplitudes=False)
    assert (Ic[0, :, 0] - f[0].reshape(n_q, 2).mean(1)).abs().max().item() <= 16 * EPS
    assert Is.abs().max().item() == 0.0


@pytest.mark.parametrize("d,r", [((500, 2), (2, 500)), ((2, 500), (500, 2)), ((700, 3), (300, 2)), ((90, 70), (3, 5)),
                                 ((60, 50), (40, 41)), ((3, 600), (33, 70))])
def test_correlation_2d_of_thin_grids(orc, d, r):
    """Cartesian grids on both sides of the choice between factored and direct sums."""
    rng = np.random.default_rng(d[0] + r[0])
    qmax, rmax = 1.1, 30.0
    grid, rgrid = numag.qgrid(0, *d, qmax), numag.qgrid(0, *r, rmax)
    f = rng.standard_normal((5, d[0] * d[1]))
    tol = EPS * (16 * qmax * rmax + d[0] * d[1] + 128) * (2 * qmax) ** 2 * np.abs(f).max()
    for n_f in (1, 3, 5):
        C = numag.correlation_2d(grid, torch.as_tensor(f[:n_f], device=DEV), rgrid).cpu().numpy()
        ref = orc.correlation_2d(0, *d, qmax, f[:n_f], 0, *r, rmax)
        assert np.abs(C[..., 0] + 1j * C[..., 1] - ref).max() <= tol


def test_correlation_2d_of_more_pixels_than_a_grid_of_columns():
    """2^28 pixels and more: the factored sum's preparation would pass 2^32 threads."""
    n, m, qmax, rmax = 16400, 4, 1.1, 30.0
    f = torch.rand((1, n * n), dtype=torch.float64, device=DEV)
    C = numag.correlation_2d(numag.qgrid(0, n, n, qmax), f, numag.qgrid(0, m, m, rmax))
    q = -qmax + torch.arange(n, dtype=torch.float64, device=DEV) * (2 * qmax / (n - 1))
    r = -rmax + torch.arange(m, dtype=torch.float64, device=DEV) * (2 * rmax / (m - 1))
    h = torch.full((n,), 2 * qmax / (n - 1), dtype=torch.float64, device=DEV)
    h[0] *= 0.5
    h[-1] *= 0.5
    ph = r[:, None] * q[None]
    c, s = torch.cos(ph) * h, torch.sin(ph) * h
    F = f.reshape(n, n)
    Fc, Fs = F @ c.T, F @ s.T
    ref = torch.stack([c @ Fc - s @ Fs, c @ Fs + s @ Fc], dim=-1).reshape(m * m, 2)
    # partial sums of up to n n terms of at most (2 qmax / n)^2, added over splits
    assert (C[0] - ref).abs().max().item() <= EPS * (16 * qmax * rmax + 4 * n + 128) * (2 * qmax) ** 2


@pytest.mark.parametrize("n_q", [1, 5, 30, 130])
@pytest.mark.parametrize("n_r", [700, 1100, 2200, 5000, 9000, 18000, 36000])
def test_correlation_lanes_per_result(orc, n_q, n_r):
    """As many results as take 64, 32, ... 1 lanes each, with empty bins."""
    rng = np.random.default_rng(n_q + n_r)
    q = np.sort(rng.uniform(0.0, 2.0, n_q))
    I = rng.uniform(0.5, 2.0, (2, n_q))
    I[:, rng.uniform(size=n_q) < 0.3] = np.nan
    r = rng.uniform(0.0, 50.0, n_r)
    c, p = numag.correlation(*(torch.as_tensor(x, device=DEV) for x in (q, I, r)))
    cref, pref = orc.correlation(q, I, r)
    tol = EPS * (n_q + 60.0 * 2) * 2.0 * 2.0 * 4.0  # as in test_correlation_empty_bins
    assert np.all(np.abs(c.cpu().numpy() - cref) <= tol)
    assert np.all(np.abs(p.cpu().numpy() - pref) <= tol * r * r)


@pytest.mark.parametrize("kind,n0,n1", [(0, 1, 1), (0, 5, 5), (0, 8, 16), (0, 3, 43), (1, 4, 6), (1, 10, 13)])
@pytest.mark.parametrize("n_sets", [1, 2, 11, 300])
def test_cross_sections_of_small_detectors(kind, n0, n1, n_sets):
    """Detectors of at most 128 pixels put several sets into a workgroup: bit for bit the
    cross sections of each set alone."""
    g = torch.Generator(device=DEV)
    g.manual_seed(n0 + n_sets)
    grid, c = numag.qgrid(kind, n0, n1, 1.3), numag.consts(V=2.0, bH=0.7, P=(0.0, 0.6, 0.8))
    amp = torch.randn((n_sets, n0 * n1, 4, 2), generator=g, device=DEV, dtype=torch.float64)
    spec = torch.randn((n_sets, n0 * n1, 16), generator=g, device=DEV, dtype=torch.float64)
    for kw in (dict(amp=amp), dict(spec=spec)):
        xs = numag.cross_section(grid, c=c, obs=numag.OBSERVABLES, **kw)
        for k in {0, n_sets // 2, n_sets - 1}:
            one = numag.cross_section(grid, c=c, obs=numag.OBSERVABLES, **{a: t[k:k + 1] for a, t in kw.items()})
            assert torch.equal(xs[k:k + 1], one)


@pytest.mark.parametrize("n0,n1,n_f,n_bins", [(500, 3, 2, 40), (1, 16, 1, 5), (129, 16, 5, 1100), (130, 40, 5, 1100),
                                              (128, 30, 1, 2049), (127, 30, 1, 2049), (600, 17, 9, 700)])
def test_azimuthal_lanes(orc, n0, n1, n_f, n_bins):
    """Thin detectors and more bins than fill the chip: other splits of the rows."""
    rng = np.random.default_rng(n0 + n_f)
    f = rng.standard_normal((n_f, n0 * n1))
    I, count = numag.azimuthal_average(numag.qgrid(0, n0, n1, 1.3), torch.as_tensor(f, device=DEV), n_bins, 1.5)
    Iref, cref = orc.azimuthal_average(0, n0, n1, 1.3, f, n_bins, 1.5)
    assert np.array_equal(count.cpu().numpy(), cref)
    I = I.cpu().numpy()
    assert np.array_equal(np.isnan(I), np.isnan(Iref))
    some = cref > 0
    assert np.all(np.abs(I - Iref)[:, some] <= EPS * n0 * n1 * np.abs(f).max())


@pytest.mark.parametrize("n_theta", [1, 4, 5, 8, 9, 16, 17, 32, 33])
@pytest.mark.parametrize("k_max", [0, 1, 7, 16, 70])
def test_angular_lanes_per_order(orc, n_theta, k_max):
    rng = np.random.default_rng(n_theta + k_max)
    f = rng.standard_normal((2, 6 * n_theta))
    Is, Ic, _, _ = (x if x is None else x.cpu().numpy() for x in numag.angular_spectrum(
        numag.qgrid(1, 6, n_theta, 1.0), torch.as_tensor(f, device=DEV), k_max, amplitudes=False))
    for s in range(2):
        Isr, Icr = orc.angular_spectrum(f[s], 6, n_theta, k_max)
        tol = 2 * EPS * (n_theta + 8 * k_max + 8) * np.abs(f).max()  # as in test_angular_orders
        assert np.abs(Is[s] - Isr).max() <= tol and np.abs(Ic[s] - Icr).max() <= tol


@pytest.mark.parametrize("r0", [1, 2, 15, 16, 17, 31, 32, 33])
@pytest.mark.parametrize("kind,n0,n1", [(1, 12, 20), (1, 9, 15), (0, 13, 11)])
def test_correlation_2d_on_few_radii(orc, kind, n0, n1, r0):
    """Real-space grids of one block of radii, of up to 16 and just more, by pixels in pairs
    and alone, one to four data sets.  A sum is off by at most 2^-52 (4 phase + P + 128) times
    that of its weights' moduli, to which their rounding adds 16."""
    rng = np.random.default_rng(400 + 10 * r0 + n0)
    f = rng.standard_normal((4, n0 * n1))
    qmax, rmax = 1.2, 25.0
    grid = numag.qgrid(kind, n0, n1, qmax)
    w = np.abs(orc.quadrature_weights(kind, n0, n1, qmax)).ravel()
    for r1 in (5, 12):
        rgrid = numag.qgrid(1, r0, r1, rmax)
        for n_f in (1, 2, 3, 4):
            C = numag.correlation_2d(grid, torch.as_tensor(f[:n_f], device=DEV), rgrid).cpu().numpy()
            ref = orc.correlation_2d(kind, n0, n1, qmax, f[:n_f], 1, r0, r1, rmax)
            tol = 2.0 ** -52 * (4 * 2 * qmax * rmax * 2 + n0 * n1 + 128 + 16) * (np.abs(f[:n_f]) @ w)
            assert np.all(np.abs(C[..., 0] + 1j * C[..., 1] - ref).max(1) <= tol), (r1, n_f)
