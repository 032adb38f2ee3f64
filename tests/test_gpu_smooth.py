"""GPU parity: Gaussian-smoothed RDF forward and its adjoint.

Forward against the oracle's FP64 h; adjoint against the oracle's FP64
gradient for the same dL/dh and against Richardson-extrapolated central
differences of the FP64 oracle loss.  Tolerance for the float32 gradient:
relative error below 1e-4, both as ||gpu - ref||_2 / ||ref||_2 and as
max |gpu - ref| / max |ref| over the compared rows.
"""
import math

import numpy as np
import pytest

import oracle
from paper_1906_06317_amd import workloads

pytestmark = pytest.mark.gpu

BINS, R_MAX, SIGMA = 200, 3.0, 0.02
GRAD_TOL = 1e-4


@pytest.fixture(scope="module")
def ppa():
    import torch
    assert torch.cuda.is_available(), "a GPU is required"
    import paper_1906_06317_amd as m
    m.lib()
    return m


def _obox(s):
    return oracle.make_box(s.L, s.tilt, s.dim)


def _box(s):
    import paper_1906_06317_amd as m
    return m.Box(s.L, s.tilt, s.dim)


def _volume(s):
    return oracle.box_volume(s.L, s.dim)


def _check_h(h_gpu, h_ref):
    err = np.abs(h_gpu - h_ref)
    assert np.all(err <= 2e-6 * np.abs(h_ref) + 1e-9 * np.abs(h_ref).max()), (
        f"max rel err {np.max(err / np.maximum(np.abs(h_ref), 1e-300))}")


def _check_grad(g_gpu, g_ref):
    d = g_gpu.astype(np.float64) - g_ref
    rel2 = np.linalg.norm(d) / np.linalg.norm(g_ref)
    relmax = np.abs(d).max() / np.abs(g_ref).max()
    assert rel2 < GRAD_TOL and relmax < GRAD_TOL, (rel2, relmax)
    return rel2, relmax


def _target_and_gh(s, tgt, h):
    n, V = s.points.shape[0], _volume(s)
    scale = 1.0 / (n * (n / V) * oracle.shell_volumes(BINS, 0.0, R_MAX))
    t = oracle.smooth_rdf_g(oracle.smooth_rdf_h(_obox(tgt), tgt.points, BINS, R_MAX, SIGMA), n, V,
                            R_MAX)
    return t, scale, 2.0 * (h * scale - t) * scale


@pytest.mark.parametrize("tilt", [(0.0, 0.0, 0.0), (0.3, -0.2, 0.1)])
def test_forward_small(ppa, tilt):
    s = workloads.uniform(3000, 0.9, seed=71, tilt=tilt)
    h = ppa.smooth_rdf_h(_box(s), s.points, BINS, R_MAX, SIGMA).cpu().numpy()
    _check_h(h, oracle.smooth_rdf_h(_obox(s), s.points, BINS, R_MAX, SIGMA))


def test_forward_accumulates_and_counts_pairs(ppa):
    s = workloads.uniform(2000, 0.9, seed=72)
    box = _box(s)
    h = ppa.smooth_rdf_h(box, s.points, BINS, R_MAX, SIGMA)
    first = h.cpu().numpy().copy()
    ppa.smooth_rdf_h(box, s.points, BINS, R_MAX, SIGMA, h=h)
    np.testing.assert_allclose(h.cpu().numpy(), 2 * first, rtol=1e-12)
    # each pair well inside [8 sigma, r_max - 8 sigma] carries mass 1 (sum rule)
    nl = ppa.query_ball(box, s.points, R_MAX - 8 * SIGMA - 0.05)
    inner = int(nl.n_pairs)
    assert first.sum() > inner


def test_adjoint_small_against_oracle_and_fd(ppa):
    s = workloads.uniform(1500, 0.9, seed=73, tilt=(0.1, 0.2, -0.1))
    tgt = workloads.uniform(1500, 0.9, seed=74, L=s.L, tilt=s.tilt)
    ob = _obox(s)
    h_ref = oracle.smooth_rdf_h(ob, s.points, BINS, R_MAX, SIGMA)
    t, scale, gh = _target_and_gh(s, tgt, h_ref)
    g_ref = oracle.smooth_rdf_grad(ob, s.points, BINS, R_MAX, SIGMA, gh)
    g = ppa.smooth_rdf_grad(_box(s), s.points, BINS, R_MAX, SIGMA, gh).cpu().numpy()
    _check_grad(g, g_ref)
    # central differences of the FP64 loss, Richardson-extrapolated
    rng = np.random.default_rng(5)

    def loss_at(k, pk):
        hk = h_ref - oracle.smooth_rdf_row(ob, s.points, k, s.points[k].astype(np.float64), BINS,
                                           R_MAX, SIGMA) \
            + oracle.smooth_rdf_row(ob, s.points, k, pk, BINS, R_MAX, SIGMA)
        return float(((hk * scale - t) ** 2).sum())

    for k in rng.choice(1500, 6, replace=False):
        for a in range(3):
            def cd(e):
                p = s.points[k].astype(np.float64).copy()
                p[a] += e
                lp = loss_at(k, p)
                p[a] -= 2 * e
                return (lp - loss_at(k, p)) / (2 * e)
            eps = 2e-4
            fd = (4 * cd(eps / 2) - cd(eps)) / 3
            assert abs(g[k, a] - fd) <= GRAD_TOL * np.abs(g_ref).max(), (k, a, g[k, a], fd)


def test_autograd_function(ppa):
    import torch
    s = workloads.uniform(1200, 0.9, seed=75)
    tgt = workloads.uniform(1200, 0.9, seed=76, L=s.L)
    box = _box(s)
    n, V = 1200, _volume(s)
    t = torch.as_tensor(oracle.smooth_rdf_g(oracle.smooth_rdf_h(_obox(tgt), tgt.points, BINS, R_MAX,
                                                                SIGMA), n, V, R_MAX)).cuda()
    p = torch.as_tensor(s.points).cuda().requires_grad_(True)
    g = ppa.smooth_rdf_g(ppa.smooth_rdf(p, box, BINS, R_MAX, SIGMA), box, n, R_MAX)
    loss = ((g - t) ** 2).sum()
    loss.backward()
    h_ref = oracle.smooth_rdf_h(_obox(s), s.points, BINS, R_MAX, SIGMA)
    _, _, gh = _target_and_gh(s, tgt, h_ref)
    g_ref = oracle.smooth_rdf_grad(_obox(s), s.points, BINS, R_MAX, SIGMA, gh)
    _check_grad(p.grad.cpu().numpy(), g_ref)
    np.testing.assert_allclose(p.grad.sum(0).cpu().numpy(), 0.0,
                               atol=1e-4 * float(p.grad.abs().max()) * math.sqrt(n))


def test_coincident_points_and_2d(ppa):
    s = workloads.uniform(800, 0.9, seed=77)
    pts = s.points.copy()
    pts[10] = pts[11]  # a pair at r = 0: in the forward, not in the gradient
    s = workloads.System(s.L, s.tilt, 3, pts)
    h = ppa.smooth_rdf_h(_box(s), pts, BINS, R_MAX, SIGMA).cpu().numpy()
    _check_h(h, oracle.smooth_rdf_h(_obox(s), pts, BINS, R_MAX, SIGMA))
    gh = np.random.default_rng(1).normal(size=BINS)
    g = ppa.smooth_rdf_grad(_box(s), pts, BINS, R_MAX, SIGMA, gh).cpu().numpy()
    _check_grad(g, oracle.smooth_rdf_grad(_obox(s), pts, BINS, R_MAX, SIGMA, gh))
    s2 = workloads.uniform(1500, 0.8, seed=78, dim=2, tilt=(0.2, 0, 0))
    h2 = ppa.smooth_rdf_h(_box(s2), s2.points, BINS, R_MAX, SIGMA).cpu().numpy()
    _check_h(h2, oracle.smooth_rdf_h(_obox(s2), s2.points, BINS, R_MAX, SIGMA))
    g2 = ppa.smooth_rdf_grad(_box(s2), s2.points, BINS, R_MAX, SIGMA, gh).cpu().numpy()
    _check_grad(g2[:, :2], oracle.smooth_rdf_grad(_obox(s2), s2.points, BINS, R_MAX, SIGMA, gh)[:, :2])


def test_errors(ppa):
    s = workloads.uniform(100, 0.9, seed=79)
    with pytest.raises(ppa.PPAError) as e:
        ppa.smooth_rdf_h(_box(s), s.points, 0, R_MAX, SIGMA)
    assert e.value.code == ppa.PPA_EINVAL
    with pytest.raises(ppa.PPAError) as e:
        ppa.smooth_rdf_h(_box(s), s.points, BINS, R_MAX, 0.0)
    assert e.value.code == ppa.PPA_EINVAL
    with pytest.raises(ppa.PPAError) as e:  # r_max + 8 sigma beyond half the box
        ppa.smooth_rdf_h(_box(s), s.points, BINS, 2.4, 0.02)
    assert e.value.code == ppa.PPA_ERANGE


def test_full_size_perturbed_lattice(ppa):
    """The perturbed simple-cubic system (N = 131,072, density 0.9), 200 bins
    on [0, 3), sigma 0.02; target from the uniform configuration.  Forward
    and adjoint at every bin and every particle."""
    s, tgt = workloads.smooth_target_pair()
    n = s.points.shape[0]
    box = _box(s)
    h = ppa.smooth_rdf_h(box, s.points, BINS, R_MAX, SIGMA).cpu().numpy()
    h_ref = oracle.smooth_rdf_h(_obox(s), s.points, BINS, R_MAX, SIGMA)
    _check_h(h, h_ref)
    t, scale, gh = _target_and_gh(s, tgt, h_ref)
    g = ppa.smooth_rdf_grad(box, s.points, BINS, R_MAX, SIGMA, gh).cpu().numpy()
    # every particle's gradient against the oracle's (about a minute of host
    # time); the norms are taken over all rows and over each block of 4096
    g_all = oracle.smooth_rdf_grad(_obox(s), s.points, BINS, R_MAX, SIGMA, gh)
    _check_grad(g, g_all)
    for b0 in range(0, n, 4096):
        _check_grad(g[b0:b0 + 4096], g_all[b0:b0 + 4096])
    g_ref = g_all
    # and against FP64 finite differences of the loss itself on this system:
    # moving particle k changes h only through its own pairs (both orders),
    # which smooth_rdf_row gives; Richardson-extrapolated central differences
    ob = _obox(s)

    def loss_at(k, pk):
        hk = h_ref - oracle.smooth_rdf_row(ob, s.points, k, s.points[k].astype(np.float64), BINS,
                                           R_MAX, SIGMA) \
            + oracle.smooth_rdf_row(ob, s.points, k, pk, BINS, R_MAX, SIGMA)
        return float(((hk * scale - t) ** 2).sum())

    floor = 5e-5 * np.abs(g_ref).max()
    for k in np.random.default_rng(8).choice(n, 4, replace=False):
        for a in range(3):
            def cd(e):
                p = s.points[k].astype(np.float64).copy()
                p[a] += e
                lp = loss_at(k, p)
                p[a] -= 2 * e
                return (lp - loss_at(k, p)) / (2 * e)
            eps = 2e-4
            fd = (4 * cd(eps / 2) - cd(eps)) / 3
            assert abs(g[k, a] - fd) <= GRAD_TOL * abs(fd) + floor, (k, a, g[k, a], fd)


def test_non_finite_input_is_reported(ppa):
    s = workloads.uniform(600, 0.9, seed=80)
    pts = s.points.copy()
    pts[5, 2] = np.nan
    with pytest.raises(ppa.PPAError) as e:
        ppa.smooth_rdf_h(_box(s), pts, BINS, R_MAX, SIGMA)
    assert e.value.code == ppa.PPA_ENONFINITE
    with pytest.raises(ppa.PPAError) as e:
        ppa.smooth_rdf_grad(_box(s), pts, BINS, R_MAX, SIGMA, np.ones(BINS))
    assert e.value.code == ppa.PPA_ENONFINITE


@pytest.mark.parametrize("bins", [1, 63, 1024, 1025])
def test_forward_fixed_point_limbs(ppa, bins):
    """Few full cells, so every wavefront folds its fixed-point limbs many
    times (over 10^5 pairs each), at bin counts around the limit of the
    fixed-point histogram and at one bin."""
    s = workloads.uniform(6000, 0.9, seed=91)
    h = ppa.smooth_rdf_h(_box(s), s.points, bins, 8.0, 0.05).cpu().numpy()
    _check_h(h, oracle.smooth_rdf_h(_obox(s), s.points, bins, 8.0, 0.05))


@pytest.mark.parametrize("bins,r_max,sigma", [(1, 2.5, 0.05), (40, 2.5, 0.5), (100, 2.5, 0.02),
                                              (2048, 2.5, 6.2e-4), (2048, 2.5, 6.0e-4)])
def test_adjoint_table_and_its_limit(ppa, bins, r_max, sigma):
    """The tabulated adjoint against the oracle from wide to narrow Gaussians,
    on both sides of its limit of 65536 nodes (r_max / sigma about 4095)."""
    nodes = np.ceil((r_max + 8 * np.float64(np.float32(sigma))) / (np.float32(sigma) / 16.0)) + 2
    assert (nodes > 65536) == (sigma == 6.0e-4)
    dim_tilt = (0.1, 0.2, -0.1)
    s = workloads.uniform(2500, 0.9, seed=92, tilt=dim_tilt)
    gh = np.random.default_rng(93).normal(size=bins)
    g_ref = oracle.smooth_rdf_grad(_obox(s), s.points, bins, r_max, sigma, gh)
    g = ppa.smooth_rdf_grad(_box(s), s.points, bins, r_max, sigma, gh).cpu().numpy()
    # a stored coordinate is off by up to 2^-24 of its cell (under 8), a pair's
    # distance by up to 4 of these, a term by that over sigma (times at most 2)
    tol = GRAD_TOL + 8 * 2.0 ** -24 * 8.0 / sigma
    d = g.astype(np.float64) - g_ref
    assert np.linalg.norm(d) < tol * np.linalg.norm(g_ref)
    assert np.abs(d).max() < tol * np.abs(g_ref).max()


def _lone_pairs(r):
    """27 pairs with no other neighbours, pair k at distance r[k] along x, on
    positions that the cell-local coordinates hold exactly (64 cells of width 11)."""
    import paper_1906_06317_amd as m
    a = np.stack(np.meshgrid([-14.25, 0.25, 14.75], [-14.25, 0.25, 14.75], [-14.25, 0.25, 14.75],
                             indexing="ij"), -1).reshape(-1, 3)
    b = a.copy()
    b[:, 0] += r
    return m.Box((44.0, 44.0, 44.0), (0.0, 0.0, 0.0), 3), np.concatenate([a, b]).astype(np.float32)


@pytest.mark.parametrize("bins", [64, 256, 1024, 1280])
def test_forward_tails(ppa, bins):
    """Bins that only the tails of a pair's Gaussian reach, out to 8 sigma, hold
    their terms to float32 accuracy relative to themselves."""
    r_max, sg, r = 4.0, 0.125, 2.1318359375
    dr = r_max / bins
    box, pts = _lone_pairs(np.full(27, r))
    h = ppa.smooth_rdf_h(box, pts, bins, r_max, sg).cpu().numpy()
    u = (np.arange(bins) + 0.5) * dr - r
    t = np.abs(u) / sg
    ref = 54 * dr / (sg * math.sqrt(2 * math.pi)) * np.exp(-0.5 * t * t)
    inside = t < 8.0 - 1e-5
    # u off by up to 32 sigma 2^-24 (three roundings of up to 16 sigma), its
    # square times a constant by 3 roundings, the exponential by 2 ulp
    tol = 2.0 ** -24 * (6.0 + 32.0 * t + 1.5 * t * t)
    assert inside.sum() > 8 and np.all(np.abs(h - ref)[inside] <= (tol * ref)[inside])
    assert np.all(h[t > 8.0 + 1e-5] == 0.0)


@pytest.mark.parametrize("bins", [8, 64, 1280])
def test_adjoint_tails(ppa, bins):
    """The gradient of one bin's weight with respect to a pair, out to 8 sigma, relative
    to itself: pairs on the nodes of the adjoint's table, between them and anywhere."""
    r_max, sg = 4.0, 0.125
    dr = r_max / bins
    k = np.arange(27)
    r = 1.75 + k / 512.0 + (k % 3) / 1024.0
    box, pts = _lone_pairs(r)
    seen = 0
    for b in range(0, bins, max(1, bins // 160)):
        t = ((b + 0.5) * dr - r) / sg
        take = (np.abs(t) > 0.5) & (np.abs(t) < 8.0 - 1e-5)
        if not take.any():
            continue
        gh = np.zeros(bins)
        gh[b] = 1.0
        g = ppa.smooth_rdf_grad(box, pts, bins, r_max, sg, gh).cpu().numpy().astype(np.float64)
        ref = 2.0 * dr / (sg * sg * math.sqrt(2 * math.pi)) * t * np.exp(-0.5 * t * t)
        # a cubic over half a node of sigma / 64: (1/128)^4 / 24 of the fifth Hermite
        # function; eight float32 roundings
        he5 = np.abs(t ** 5 - 10 * t ** 3 + 15 * t)
        tol = 1.1 / 128 ** 4 / 24 * he5 / np.abs(t) + 8 * 2.0 ** -24
        err = np.abs(np.stack([g[27:, 0], -g[:27, 0]]) / np.where(take, ref, 1.0) - 1.0)
        assert np.all(err[:, take] <= tol[take]), (b, float((err / tol)[:, take].max()))
        seen += int(take.sum())
    assert seen > 27


@pytest.mark.parametrize("n,bins,sigma", [
    (2500, 256, 0.02),     # table, 16 lanes a node
    (2500, 100, 0.004),    # table, 4 lanes a node
    (2500, 100, 0.0012),   # window terms: few of them against the table's nodes
    (40000, 2048, 6.2e-4),  # table of nearly the most nodes
    (40000, 2048, 6.0e-4),  # window terms: more nodes than that
])
def test_adjoint_routes(ppa, n, bins, sigma):
    """The adjoint's table and its window terms, on both sides of the rule between them,
    against the oracle on a sample of rows."""
    r_max = 2.5
    s = workloads.uniform(n, 0.9, seed=95, tilt=(0.1, 0.2, -0.1))
    rng = np.random.default_rng(96)
    gh = rng.normal(size=bins)
    rows = np.sort(rng.permutation(n)[:300])
    g_ref = oracle.smooth_rdf_grad(_obox(s), s.points, bins, r_max, sigma, gh, rows=rows)
    g = ppa.smooth_rdf_grad(_box(s), s.points, bins, r_max, sigma, gh).cpu().numpy()[rows]
    # a stored coordinate is off by up to 2^-24 of its cell (under 8), a pair's
    # distance by up to 4 of these, a term by that over sigma (times at most 2)
    tol = GRAD_TOL + 8 * 2.0 ** -24 * 8.0 / sigma
    d = g.astype(np.float64) - g_ref
    assert np.linalg.norm(d) < tol * np.linalg.norm(g_ref)
    assert np.abs(d).max() < tol * np.abs(g_ref).max()
