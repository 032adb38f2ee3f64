"""GPU parity: ball query (NeighborList) and RDF against the FP64 oracle."""
import math

import numpy as np
import pytest

import oracle
from paper_1906_06317_amd import workloads
from tests import brute
from tests.parity import REL, check_hist, check_rows

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ppa():
    import torch
    assert torch.cuda.is_available(), "a GPU is required"
    import paper_1906_06317_amd as m
    m.lib()
    return m


def _box(s):
    import paper_1906_06317_amd as m
    return m.Box(s.L, s.tilt, s.dim)


def _oracle_rows(s, r_max, rows, query_points=None, exclude_ii=None):
    ob = oracle.make_box(s.L, s.tilt, s.dim)
    q = s.points if query_points is None else query_points
    if exclude_ii is None:
        exclude_ii = query_points is None
    # oracle over the selected query rows; exclude_ii needs true indices, so
    # pass all points and keep the wanted rows (small inputs) or recompute per row
    csr_off, csr_idx, csr_r2 = [0], [], []
    for qi in rows:
        o, i, r = oracle.ball_query(ob, s.points, r_max, query_points=q[qi:qi + 1], exclude_ii=False)
        if exclude_ii:
            keep = i != qi
            i, r = i[keep], r[keep]
        csr_idx.append(i)
        csr_r2.append(r)
        csr_off.append(csr_off[-1] + len(i))
    return (np.array(csr_off), np.concatenate(csr_idx) if csr_idx else np.zeros(0, np.int32),
            np.concatenate(csr_r2) if csr_r2 else np.zeros(0))


def _oracle_all(s, r_max, query_points=None, exclude_ii=None):
    ob = oracle.make_box(s.L, s.tilt, s.dim)
    return oracle.ball_query(ob, s.points, r_max, query_points=query_points, exclude_ii=exclude_ii)


def test_small_uniform_ball_and_rdf(ppa):
    s = workloads.small_uniform()
    box = _box(s)
    counts, nl = ppa.rdf_counts(box, s.points, 100, 3.0, neighbor_list=True)
    n = s.points.shape[0]
    ref = _oracle_all(s, 3.0)
    n_cert, n_amb = check_rows(nl, ref, range(n), 3.0)
    assert n_cert > 300000
    assert n_cert <= nl.n_pairs <= n_cert + n_amb
    off = nl.offsets.cpu().numpy()
    assert off[-1] == nl.n_pairs
    cnt = nl.counts.cpu().numpy()
    assert off[0] == 0 and np.all(np.diff(off) == cnt)
    lo, hi, amb = oracle.rdf_counts(oracle.make_box(s.L, s.tilt), s.points, 100, 3.0)
    g = counts.cpu().numpy()
    check_hist(g, lo, hi)
    # every listed pair is binned by its reported distance (a pair in the band
    # at r_max may be listed with a distance that rounds to r_max: not binned)
    assert g.sum() == int((nl.dist.cpu().numpy() < np.float32(3.0)).sum())
    # the same histogram from the stored list
    g2 = ppa.rdf_from_nlist(nl, 100, 3.0).cpu().numpy()
    np.testing.assert_array_equal(g, g2)


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("seed", [0, 1, 2, 3])
def test_random_triclinic_boxes(ppa, dim, seed):
    rng = np.random.default_rng(100 + 10 * dim + seed)
    L = rng.uniform(6.0, 14.0, 3)
    tilt = rng.uniform(-0.5, 0.5, 3)
    if dim == 2:
        L[2] = 1.0
        tilt[1:] = 0
    n = int(rng.integers(50, 3000))
    s = workloads.uniform(n, 1.0, seed=seed, dim=dim, tilt=tuple(tilt), L=tuple(L))
    half = 0.5 * brute.perpendicular_widths(tuple(L), tuple(tilt), dim)[:dim].min()
    for frac in (0.3, 0.7, 0.99):
        r_max = float(frac * half)
        box = _box(s)
        nl = ppa.query_ball(box, s.points, r_max)
        check_rows(nl, _oracle_all(s, r_max), range(n), r_max)
        bins = int(rng.integers(1, 200))
        r_min = float(rng.uniform(0, 0.5 * r_max))
        c = ppa.rdf_counts(box, s.points, bins, r_max, r_min=r_min).cpu().numpy()
        lo, hi, amb = oracle.rdf_counts(oracle.make_box(s.L, s.tilt, dim), s.points, bins, r_max,
                                        r_min)
        check_hist(c, lo, hi)
        # the same bins from the pass that also writes the list (r_min > 0
        # and r_min = 0 take different binning code there)
        for rm in (r_min, 0.0):
            c2, nl2 = ppa.rdf_counts(box, s.points, bins, r_max, r_min=rm, neighbor_list=True)
            if rm == 0.0:
                lo, hi, amb = oracle.rdf_counts(oracle.make_box(s.L, s.tilt, dim), s.points, bins,
                                                r_max, 0.0)
            check_hist(c2.cpu().numpy(), lo, hi)
            assert int(nl2.n_pairs) == int(nl.n_pairs)


def test_separate_query_points(ppa):
    rng = np.random.default_rng(7)
    s = workloads.uniform(2500, 0.9, seed=8, tilt=(0.3, -0.2, 0.1))
    A = workloads.lattice_vectors(s.L, s.tilt)
    q = (rng.uniform(-1.5, 1.5, (700, 3)) @ A.T).astype(np.float32)  # also outside the box
    box = _box(s)
    for excl in (False, True):
        nl = ppa.query_ball(box, s.points, 2.2, query_points=q, exclude_ii=excl)
        ob = oracle.make_box(s.L, s.tilt)
        ref = oracle.ball_query(ob, s.points, 2.2, query_points=q, exclude_ii=excl)
        check_rows(nl, ref, range(700), 2.2)
        c = ppa.rdf_counts(box, s.points, 50, 2.2, query_points=q, exclude_ii=excl).cpu().numpy()
        lo, hi, _ = oracle.rdf_counts(ob, s.points, 50, 2.2, query_points=q, exclude_ii=excl)
        check_hist(c, lo, hi)


@pytest.mark.parametrize("frac", [0.32, 0.62])
@pytest.mark.parametrize("dim", [2, 3])
def test_few_full_cells_split_among_wavefronts(ppa, dim, frac):
    """Few cells holding many queries each (a cutoff large against the box):
    the count and fill passes share each cell's queries among several
    wavefronts.  Self queries (the own entry found by its position in the
    home cell, beyond the first 64 too), separate query points with and
    without dropping equal indices, and the RDF of the same passes."""
    rng = np.random.default_rng(11 + dim)
    n = 3000
    s = workloads.uniform(n, 2.0, seed=12 + dim, dim=dim, tilt=(0.2, 0.1, -0.1) if dim == 3
                          else (0.2, 0.0, 0.0))
    half = 0.5 * brute.perpendicular_widths(tuple(s.L), tuple(s.tilt), dim)[:dim].min()
    # six cells per axis (candidates in register slots) or three (every
    # point a candidate, and home cells of more than 64 points)
    r_max = float(frac * half)
    box = _box(s)
    ob = oracle.make_box(s.L, s.tilt, dim)
    nl = ppa.query_ball(box, s.points, r_max)
    check_rows(nl, _oracle_all(s, r_max), range(n), r_max)
    A = workloads.lattice_vectors(s.L, s.tilt, dim)
    nq = 5000
    f = rng.uniform(-0.5, 0.5, (nq, 3))
    if dim == 2:
        f[:, 2] = 0.0
    q = (f @ A.T).astype(np.float32)
    q[:200] = s.points[:200]  # some queries coincide with points
    for excl in (False, True):
        nl = ppa.query_ball(box, s.points, r_max, query_points=q, exclude_ii=excl)
        ref = oracle.ball_query(ob, s.points, r_max, query_points=q, exclude_ii=excl)
        check_rows(nl, ref, range(nq), r_max)
        c = ppa.rdf_counts(box, s.points, 64, r_max, query_points=q, exclude_ii=excl).cpu().numpy()
        lo, hi, _ = oracle.rdf_counts(ob, s.points, 64, r_max, query_points=q, exclude_ii=excl)
        check_hist(c, lo, hi)


def test_self_pairs_and_coincident_points(ppa):
    pts = np.zeros((5, 3), np.float32)
    pts[3] = [1.0, 0, 0]
    pts[4] = [1.0, 0, 0]
    s = workloads.System((10.0, 10.0, 10.0), (0, 0, 0), 3, pts)
    box = _box(s)
    nl = ppa.query_ball(box, pts, 1.5, exclude_ii=False)
    cnt = nl.counts.cpu().numpy()
    assert cnt.tolist() == [5, 5, 5, 5, 5]
    nl = ppa.query_ball(box, pts, 1.5)
    assert nl.counts.cpu().numpy().tolist() == [4, 4, 4, 4, 4]
    nl = ppa.query_ball(box, pts, 0.5)
    assert nl.counts.cpu().numpy().tolist() == [2, 2, 2, 1, 1]


def test_empty_and_tiny_inputs(ppa):
    box = ppa.Box.cube(10.0)
    nl = ppa.query_ball(box, np.zeros((0, 3), np.float32), 2.0)
    assert nl.n_pairs == 0 and nl.offsets.cpu().numpy().tolist() == [0]
    nl = ppa.query_ball(box, np.zeros((1, 3), np.float32), 2.0)
    assert nl.n_pairs == 0
    q = np.zeros((0, 3), np.float32)
    nl = ppa.query_ball(box, np.ones((10, 3), np.float32), 2.0, query_points=q)
    assert nl.n_pairs == 0 and nl.offsets.shape[0] == 1


def test_dense_cluster_takes_streamed_path(ppa):
    """More than 1024 candidates in a stencil: the streamed path must agree."""
    rng = np.random.default_rng(5)
    pts = rng.normal(0, 0.6, (3000, 3)).astype(np.float32)
    s = workloads.System((20.0, 20.0, 20.0), (0.1, 0, 0), 3, pts)
    box = _box(s)
    counts, nl = ppa.rdf_counts(box, pts, 64, 1.9, neighbor_list=True)
    rows = list(range(0, 3000, 7))
    check_rows(nl, _oracle_rows(s, 1.9, rows), rows, 1.9)
    lo, hi, _ = oracle.rdf_counts(oracle.make_box(s.L, s.tilt), pts, 64, 1.9)
    check_hist(counts.cpu().numpy(), lo, hi)


def test_capacity_overflow_reported_then_retry(ppa):
    import torch
    s = workloads.small_uniform()
    box = _box(s)
    nl = ppa.query_ball(box, s.points, 3.0, capacity=10)  # binding retries with the exact size
    rows = list(range(0, 4096, 5))
    check_rows(nl, _oracle_rows(s, 3.0, rows), rows, 3.0)
    # raw call: capacity 1 -> PPA_ECAPACITY with the true count reported
    import ctypes
    L = ppa.lib()
    pts = torch.as_tensor(s.points).cuda()
    n = pts.shape[0]
    ws = ppa.Workspace()
    wptr, wlen = ws.get(ppa.workspace_bytes(box, n, 0, 3.0, ppa.PPA_WS_NLIST))
    off = torch.empty(n + 1, dtype=torch.int64, device="cuda")
    cnt = torch.empty(n, dtype=torch.int32, device="cuda")
    pidx = torch.empty(1, dtype=torch.int32, device="cuda")
    npairs = torch.zeros(1, dtype=torch.int64, device="cuda")
    rc = L.ppa_query_ball(ctypes.byref(box.c()), ctypes.c_void_p(pts.data_ptr()), n, None, n, 3.0, 1,
                          0, wptr, wlen, ctypes.c_void_p(off.data_ptr()),
                          ctypes.c_void_p(cnt.data_ptr()), ctypes.c_void_p(pidx.data_ptr()), None,
                          1, ctypes.c_void_p(npairs.data_ptr()),
                          ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    assert ws.status() == ppa.PPA_ECAPACITY
    assert int(npairs.item()) == nl.n_pairs


def test_nonfinite_input_reported(ppa):
    s = workloads.small_uniform()
    pts = s.points.copy()
    pts[17, 1] = np.nan
    with pytest.raises(ppa.PPAError) as e:
        ppa.query_ball(_box(s), pts, 3.0)
    assert e.value.code == ppa.PPA_ENONFINITE


def test_host_errors(ppa):
    s = workloads.small_uniform()
    with pytest.raises(ppa.PPAError) as e:
        ppa.query_ball(_box(s), s.points, 9.0)
    assert e.value.code == ppa.PPA_ERANGE
    with pytest.raises(ppa.PPAError) as e:
        ppa.rdf_counts(_box(s), s.points, 0, 3.0)
    assert e.value.code == ppa.PPA_EINVAL


def test_deterministic_rows(ppa):
    s = workloads.small_uniform()
    box = _box(s)
    a = ppa.query_ball(box, s.points, 3.0)
    b = ppa.query_ball(box, s.points, 3.0)
    assert a.n_pairs == b.n_pairs
    assert np.array_equal(a.offsets.cpu().numpy(), b.offsets.cpu().numpy())
    assert np.array_equal(a.point_idx.cpu().numpy(), b.point_idx.cpu().numpy())
    assert np.array_equal(a.dist.cpu().numpy(), b.dist.cpu().numpy())


def test_large_fcc_sampled_rows_and_rdf(ppa):
    """N = 1,048,576 noisy FCC in a tilted box, in the launch configuration the
    benchmark times (one pass, list + fused RDF): sampled rows against the
    oracle, and the full histogram against properties that hold at any size."""
    import torch
    s = workloads.large_fcc()
    box = _box(s)
    n = s.points.shape[0]
    counts, nl = ppa.rdf_counts(box, s.points, 256, 2.5, neighbor_list=True)
    rng = np.random.default_rng(2)
    rows = np.unique(np.concatenate([rng.choice(n, 250, replace=False), [0, 1, n - 1, n // 2]]))
    n_cert, n_amb = check_rows(nl, _oracle_rows(s, 2.5, rows), rows, 2.5)
    assert n_cert > 60 * len(rows)
    g = counts.cpu().numpy()
    assert g.sum() == int((nl.dist.cpu().numpy() < np.float32(2.5)).sum())
    assert nl.n_pairs - g.sum() < 100
    np.testing.assert_array_equal(g, ppa.rdf_from_nlist(nl, 256, 2.5).cpu().numpy())
    cnt = nl.counts.cpu().numpy()
    assert cnt.sum() == nl.n_pairs
    assert cnt.min() >= 50 and cnt.max() <= 100
    # the histogram restricted to the sampled query rows against the oracle
    q = s.points[rows]
    sub = ppa.rdf_counts(box, s.points, 256, 2.5, query_points=q, exclude_ii=False).cpu().numpy()
    lo, hi, _ = oracle.rdf_counts(oracle.make_box(s.L, s.tilt), s.points, 256, 2.5,
                                  query_points=q, exclude_ii=False)
    # a query point sits on itself at r = 0, which falls in bin 0 for both
    check_hist(sub, lo, hi)


def test_small_cutoff_in_sparse_box_uses_exact_test(ppa):
    """Cells far larger than r_max (few points, capped cell count): the host
    rejects the expanded in/out test and the difference form runs."""
    rng = np.random.default_rng(12)
    centres = rng.uniform(-25, 25, (40, 3))
    pts = (centres[:, None, :] + rng.normal(0, 0.3, (40, 10, 3))).reshape(-1, 3).astype(np.float32)
    s = workloads.System((50.0, 50.0, 50.0), (0.1, 0.0, -0.1), 3, pts)
    box = _box(s)
    counts, nl = ppa.rdf_counts(box, pts, 20, 0.5, neighbor_list=True)
    check_rows(nl, _oracle_all(s, 0.5), range(pts.shape[0]), 0.5)
    lo, hi, _ = oracle.rdf_counts(oracle.make_box(s.L, s.tilt), pts, 20, 0.5)
    check_hist(counts.cpu().numpy(), lo, hi)
    assert nl.n_pairs > 500


def test_unaligned_output_buffers_large(ppa):
    """Row counts and offsets at addresses that are not 16-byte aligned (views
    one element into larger buffers) take the scalar path of the scan's long
    tiles (2^17 rows and more); the list must equal the one written to
    aligned buffers, and sampled rows match the oracle."""
    import ctypes
    import torch
    s = workloads.uniform(200_000, 0.8, 1011)
    box = _box(s)
    r_max = 1.6
    ref = ppa.query_ball(box, s.points, r_max)
    L = ppa.lib()
    pts = torch.as_tensor(s.points).cuda()
    n = pts.shape[0]
    ws = ppa.Workspace()
    wptr, wlen = ws.get(ppa.workspace_bytes(box, n, 0, r_max, ppa.PPA_WS_NLIST))
    off_buf = torch.zeros(n + 2, dtype=torch.int64, device="cuda")
    cnt_buf = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    off, cnt = off_buf[1:], cnt_buf[1:]
    assert off.data_ptr() % 16 != 0 and cnt.data_ptr() % 16 != 0
    P = ref.n_pairs
    pidx = torch.empty(P, dtype=torch.int32, device="cuda")
    dist = torch.empty(P, dtype=torch.float32, device="cuda")
    npairs = torch.zeros(1, dtype=torch.int64, device="cuda")
    rc = L.ppa_query_ball(ctypes.byref(box.c()), ctypes.c_void_p(pts.data_ptr()), n, None, n,
                          r_max, 1, 0, wptr, wlen, ctypes.c_void_p(off.data_ptr()),
                          ctypes.c_void_p(cnt.data_ptr()), ctypes.c_void_p(pidx.data_ptr()),
                          ctypes.c_void_p(dist.data_ptr()), P, ctypes.c_void_p(npairs.data_ptr()),
                          ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0 and ws.status() == 0
    assert int(npairs.item()) == P
    assert torch.equal(off, ref.offsets)
    assert torch.equal(cnt, (ref.offsets[1:] - ref.offsets[:-1]).to(torch.int32))
    assert torch.equal(pidx, ref.point_idx[:P]) and torch.equal(dist, ref.dist[:P])
    assert int(off_buf[0].item()) == 0 and int(cnt_buf[0].item()) == 0  # nothing written before
    rows = list(range(0, n, 997)) + [n - 1]
    check_rows(ref, _oracle_rows(s, r_max, rows), rows, r_max)


def _rows_sorted_and_same(nl_sorted, nl_plain):
    """Every row of nl_sorted is increasing in j and holds the same (j, r)
    pairs as the same row of nl_plain."""
    off = nl_plain.offsets.cpu().numpy()
    assert np.array_equal(off, nl_sorted.offsets.cpu().numpy())
    pi, pd = nl_plain.point_idx.cpu().numpy(), nl_plain.dist.cpu().numpy()
    si, sd = nl_sorted.point_idx.cpu().numpy(), nl_sorted.dist.cpu().numpy()
    n_long = 0
    for q in range(len(off) - 1):
        a, b = off[q], off[q + 1]
        if b - a > 256:
            n_long += 1
        assert np.all(np.diff(si[a:b]) > 0), f"row {q} not increasing"
        order = np.argsort(pi[a:b], kind="stable")
        assert np.array_equal(si[a:b], pi[a:b][order]), f"row {q}: different neighbours"
        assert np.array_equal(sd[a:b], pd[a:b][order]), f"row {q}: distances not moved with j"
    return n_long


def test_sort_rows_short_rows_against_oracle(ppa):
    """sort_rows: rows of about 90 entries (staged in LDS), ordered by j, the
    oracle's canonical order for the sampled rows."""
    s = workloads.small_uniform()
    box = _box(s)
    plain = ppa.query_ball(box, s.points, 3.0)
    srt = ppa.query_ball(box, s.points, 3.0, sort_rows=True)
    assert _rows_sorted_and_same(srt, plain) == 0
    rows = list(range(0, 4096, 37))
    check_rows(srt, _oracle_rows(s, 3.0, rows), rows, 3.0)
    # the oracle lists each row by increasing j: the certain part matches in order
    o_off, o_idx, o_r2 = _oracle_rows(s, 3.0, rows)
    off = srt.offsets.cpu().numpy()
    pidx = srt.point_idx.cpu().numpy()
    lo = 9.0 * (1 - REL)
    for k, q in enumerate(rows):
        oi, orr = o_idx[o_off[k]:o_off[k + 1]], o_r2[o_off[k]:o_off[k + 1]]
        certain = np.sort(oi[orr < lo])
        g = pidx[off[q]:off[q + 1]]
        assert np.array_equal(g[np.isin(g, certain)], certain)


def test_sort_rows_long_rows_bitonic(ppa):
    """Rows longer than the LDS stage (256) are sorted in place by the bitonic
    network; lengths are not powers of two.  Separate query points too."""
    s = workloads.uniform(6000, 8.0, 1012)   # r = 2.7: about 660 neighbours per point
    box = _box(s)
    plain = ppa.query_ball(box, s.points, 2.7)
    srt = ppa.query_ball(box, s.points, 2.7, sort_rows=True)
    assert _rows_sorted_and_same(srt, plain) > 1000
    q = workloads.uniform(500, 8.0, 1013, L=s.L).points
    plain = ppa.query_ball(box, s.points, 2.7, query_points=q)
    srt = ppa.query_ball(box, s.points, 2.7, query_points=q, sort_rows=True)
    assert _rows_sorted_and_same(srt, plain) > 100


def test_sort_rows_with_rdf_and_capacity_retry(ppa):
    """The RDF pass with its list sorted: the histogram is unchanged, the
    list sorted; a first attempt with too small a capacity is retried."""
    import torch
    s = workloads.small_uniform()
    box = _box(s)
    h0, plain = ppa.rdf_counts(box, s.points, 100, 3.0, neighbor_list=True)
    h1, srt = ppa.rdf_counts(box, s.points, 100, 3.0, neighbor_list=True, sort_rows=True,
                             capacity=1000)
    assert torch.equal(h0, h1)
    _rows_sorted_and_same(srt, plain)


def test_sort_rows_without_distances(ppa):
    """sort_rows with no distance output (with_dist=False): indices only,
    short rows (LDS) and long rows (bitonic) alike."""
    for s, r in ((workloads.small_uniform(), 3.0), (workloads.uniform(3000, 8.0, 1014), 2.7)):
        box = _box(s)
        plain = ppa.query_ball(box, s.points, r, with_dist=False)
        srt = ppa.query_ball(box, s.points, r, with_dist=False, sort_rows=True)
        assert srt.dist is None
        off = plain.offsets.cpu().numpy()
        pi, si = plain.point_idx.cpu().numpy(), srt.point_idx.cpu().numpy()
        for q in range(len(off) - 1):
            a, b = off[q], off[q + 1]
            assert np.array_equal(si[a:b], np.sort(pi[a:b])), f"row {q}"


@pytest.mark.parametrize("dim,n,r_max", [(3, 400000, 1.0), (2, 300000, 1.6)])
def test_drawn_home_cells_cover_every_row(ppa, dim, n, r_max):
    """Enough home cells that the fill pass draws part of them from its queues
    (in 2D and 3D, with and without a list): the count pass, which deals its
    cells, and the fill pass agree on every row, and the histograms agree."""
    import torch
    s = workloads.uniform(n, 1.0, seed=930 + dim, dim=dim)
    box = ppa.Box(s.L, s.tilt, s.dim)
    pts = torch.as_tensor(s.points).cuda()
    h, nl = ppa.rdf_counts(box, pts, 64, r_max, neighbor_list=True)
    alone = ppa.rdf_counts(box, pts, 64, r_max)
    assert int(h.sum()) == nl.n_pairs and torch.equal(h, ppa.rdf_from_nlist(nl, 64, r_max))
    # in/out of the list is by the expanded test, alone by the difference: pairs
    # within the parity band (1e-5 of r_max^2) of the cutoff may differ
    assert abs(int(alone.sum()) - nl.n_pairs) <= 4e-5 * nl.n_pairs
    assert torch.equal(alone[:-1], h[:-1])
    q = nl.query_point_indices().long()
    d = nl.point_idx.long()
    assert int((q == d).sum()) == 0
    # every pair is listed from both sides, and no row holds a neighbour twice
    key, rev = q * n + d, d * n + q
    key, rev = key.sort().values, rev.sort().values
    assert int((key[1:] == key[:-1]).sum()) == 0
    assert int((key != rev).sum()) <= 8e-5 * nl.n_pairs


@pytest.mark.parametrize("n,r_max", [(1, 1.0), (65, 1.0), (1023, 2.0), (1025, 2.0), (4095, 1.2),
                                     (4096, 2.0), (4097, 2.0), (20001, 4.0), (20001, 1.6)])
@pytest.mark.parametrize("separate", [False, True])
def test_cell_builds_of_each_size(ppa, n, r_max, separate):
    """The one-workgroup cell build (up to 4096 points and queries), the build
    for few cells (20,001 points, r = 4) and the general one, around their
    limits: rows against the oracle, rows in one order from call to call, the
    same rows by index with sort_rows, the histogram alone equal to the list's."""
    import torch
    s = workloads.uniform(n, 0.8 if n > 100 else 0.05, seed=950 + n, tilt=(0.1, -0.05, 0.1))
    box = _box(s)
    q = None
    if separate:
        rng = np.random.default_rng(951 + n)
        q = s.points[rng.permutation(n)[:max(1, n // 3)]] + np.float32(0.01)
    counts, nl = ppa.rdf_counts(box, s.points, 40, r_max, query_points=q, neighbor_list=True)
    nq = n if q is None else q.shape[0]
    rows = range(0, nq, max(1, nq // 400))
    check_rows(nl, _oracle_rows(s, r_max, list(rows), query_points=q), list(rows), r_max)
    again = ppa.query_ball(box, s.points, r_max, query_points=q,
                           exclude_ii=q is None)
    assert torch.equal(nl.offsets, again.offsets) and torch.equal(nl.point_idx, again.point_idx)
    by_index = ppa.query_ball(box, s.points, r_max, query_points=q, exclude_ii=q is None,
                              sort_rows=True)
    key = nl.query_point_indices().long() * n + nl.point_idx
    order = key.argsort()
    assert torch.equal(by_index.point_idx, nl.point_idx[order])
    assert torch.equal(by_index.dist, nl.dist[order])
    alone = ppa.rdf_counts(box, s.points, 40, r_max, query_points=q)
    assert torch.equal(alone[:-1], counts[:-1])


def test_status_per_thread_and_stream(ppa):
    """Statuses read by several threads at once, each on its own stream and
    workspace, and behind work longer than the polling limit: every call sees
    its own (one thread's input is not finite)."""
    import threading
    import torch
    s = workloads.uniform(300000, 1.0, seed=990)
    box = ppa.Box(s.L, s.tilt, s.dim)
    good = torch.as_tensor(s.points).cuda()
    bad = good.clone()
    bad[7, 1] = float("nan")
    want = ppa.rdf_counts(box, good, 32, 2.0)
    torch.cuda.synchronize()
    out = {}

    def work(k):
        st = torch.cuda.Stream()
        ws = ppa.Workspace()
        res = []
        for rep in range(6):
            h = torch.zeros(32, dtype=torch.int64, device="cuda")
            torch.cuda.current_stream().synchronize()
            try:
                for _ in range(8 if rep == 5 else 1):  # the last status is behind more work
                    h.zero_()
                    torch.cuda.current_stream().synchronize()
                    ppa.rdf_counts(box, bad if k == 2 else good, 32, 2.0, counts=h, ws=ws,
                                   stream=st, check=False)
                    st.synchronize() if rep < 5 else None
                res.append((ws.status(st), h))
            except Exception as e:  # noqa: BLE001 (reported below)
                res.append((repr(e), h))
        out[k] = res

    ts = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for k in range(4):
        for rep, (rc, h) in enumerate(out[k]):
            assert rc == (ppa.PPA_ENONFINITE if k == 2 else ppa.PPA_OK), (k, rep, rc)
            if k != 2 and rep < 5:
                assert torch.equal(h, want)


@pytest.mark.parametrize("dim,n,r_max,tilt", [
    (3, 6000, 4.0, 0.3),     # octants, several wavefronts each
    (3, 60000, 3.5, 0.0),    # octants, one wavefront each
    (2, 30000, 9.0, 0.2),    # quadrants
    (3, 30000, 2.6, 0.0),    # cells around the register slots: tiles and streams
])
@pytest.mark.parametrize("r_min,separate", [(0.0, False), (0.7, False), (0.0, True)])
def test_histogram_of_full_cells(ppa, dim, n, r_max, tilt, r_min, separate):
    """The histogram alone over cells past the register slots (octant parts,
    pruned and staged candidates) against the histogram binned with the list;
    a dense blob puts more than 64 queries in a part."""
    import torch
    s = workloads.uniform(n, 1.2, seed=960 + n, dim=dim, tilt=(tilt, 0.0, 0.0))
    rng = np.random.default_rng(961 + n)
    blob = rng.normal(0.0, 0.4, size=(1500, 3)).astype(np.float32)
    pts = s.points.copy()
    pts[:1500, :dim] = blob[:, :dim] + np.float32(0.3)
    pts[5] = pts[4]  # coincident points are neighbours at r = 0
    box = _box(s)
    q = None
    if separate:
        q = pts[rng.permutation(n)[:n // 2]] + np.float32(0.013)
        q[:, dim:] = 0
    alone = ppa.rdf_counts(box, pts, 50, r_max, r_min, query_points=q)
    both, nl = ppa.rdf_counts(box, pts, 50, r_max, r_min, query_points=q, neighbor_list=True)
    assert torch.equal(alone[:-1], both[:-1])
    # the last bin: pairs in the parity band of the cutoff may be decided either way
    assert abs(int(alone[-1]) - int(both[-1])) <= 2 + 4e-5 * nl.n_pairs
    excl = ppa.rdf_counts(box, pts, 50, r_max, r_min, query_points=q, exclude_ii=False)
    own = 0 if r_min > 0.0 else (int(excl[0]) - int(alone[0]))
    assert own == (0 if r_min > 0.0 or separate else n)
    assert torch.equal(excl[1:], alone[1:])


def test_histogram_of_full_cells_is_the_sum_over_its_queries(ppa):
    """One call over full cells against calls on parts of its queries, too few for that
    route: the same pairs, bin by bin, also where thousands lie at the cutoff to
    within rounding (a rotated lattice with neighbours at r_max, whose cells
    have few candidates, beside a dense fluid)."""
    import torch
    rng = np.random.default_rng(977)
    L, a, r_max = 24.5, 1.5, 3.0
    rot, _ = np.linalg.qr(rng.normal(size=(3, 3)))
    g = np.arange(-14, 15) * a
    lat = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3) @ rot.T
    lat = lat[(np.abs(lat[:, :2]) < L / 2).all(1) & (lat[:, 2] < -0.1) & (lat[:, 2] > -L / 2 + 0.1)]
    fluid = rng.uniform(-L / 2, L / 2, size=(18000, 3))
    fluid[:, 2] = np.abs(fluid[:, 2])
    pts = torch.as_tensor(np.concatenate([lat, fluid]).astype(np.float32)).cuda()
    n, cells = pts.shape[0], 8 ** 3
    assert n >= 32 * cells and n * 27 > 640 * cells  # the full-cell route
    box = ppa.Box((L, L, L), (0.0, 0.0, 0.0), 3)
    whole = ppa.rdf_counts(box, pts, 60, r_max, exclude_ii=False)
    parts = torch.zeros_like(whole)
    for q in pts.split(n // 3 + 1):
        assert q.shape[0] < 32 * cells
        ppa.rdf_counts(box, pts, 60, r_max, query_points=q, exclude_ii=False, counts=parts)
    assert torch.equal(whole, parts), (whole - parts).tolist()[-3:]


@pytest.mark.parametrize("system", ["alike", "droplets", "one droplet", "full quadrants"])
def test_full_cells_of_uneven_systems(ppa, system):
    """The parts of full cells where the cells are alike, where a few hold most of
    the work (many shares of an octant, several cells apart) and where a part has more
    than 64 queries: one call is the sum over calls on parts of its queries,
    bin by bin, and its own pairs are the diagonal."""
    import torch
    rng = np.random.default_rng(981)
    dim, per = 3, 32
    if system == "full quadrants":
        dim, per, L, r_max, m, n = 2, 16, 32.5, 1.0, 32, 310000
        pts = rng.uniform(-L / 2, L / 2, size=(n, 3))
        pts[:, 2] = 0
    else:
        L, r_max, m, n = 24.5, 3.0, 8, 20000
        pts = rng.uniform(-L / 2, L / 2, size=(n, 3))
        if system != "alike":
            k = 3 if system == "droplets" else 1
            at = rng.uniform(-L / 2, L / 2, size=(k, 3))
            pts[:14000] = at[rng.integers(0, k, 14000)] + rng.normal(0, 1.0, size=(14000, 3))
    pts = torch.as_tensor(pts.astype(np.float32)).cuda()
    cells = m ** dim
    assert n >= per * cells and n * 3 ** dim > 640 * cells  # the full-cell route
    box = ppa.Box((L, L, L if dim == 3 else 1.0), (0.0, 0.0, 0.0), dim)
    whole = ppa.rdf_counts(box, pts, 70, r_max, exclude_ii=False)
    parts = torch.zeros_like(whole)
    for q in pts.split(per * cells - 1):
        ppa.rdf_counts(box, pts, 70, r_max, query_points=q, exclude_ii=False, counts=parts)
    assert torch.equal(whole, parts), (whole - parts).tolist()
    own = ppa.rdf_counts(box, pts, 70, r_max)
    assert int(whole[0] - own[0]) == n and torch.equal(whole[1:], own[1:])


@pytest.mark.parametrize("n,r_max", [(480000, 2.6), (480000, 3.0), (560000, 3.4)])
def test_drawn_and_dealt_cells_in_2d(ppa, n, r_max):
    """Lists in 2D on both sides of the rule for drawing home cells (queries times
    candidates of a cell), with enough cells to draw: the fill pass writes the rows that the
    count pass, which deals its cells, measured."""
    import torch
    s = workloads.uniform(n, 1.0, seed=940, dim=2)
    box = ppa.Box(s.L, s.tilt, s.dim)
    pts = torch.as_tensor(s.points).cuda()
    nl = ppa.query_ball(box, pts, r_max)
    nl.point_idx.fill_(-1)
    again = ppa.query_ball(box, pts, r_max)
    assert torch.equal(nl.offsets, again.offsets)
    q, d = again.query_point_indices().long(), again.point_idx.long()
    assert int(d.min()) >= 0 and int((q == d).sum()) == 0
    key = (q * n + d).sort().values
    assert int((key[1:] == key[:-1]).sum()) == 0
    # pairs listed from one side only: those within the parity band of the cutoff
    assert int((~torch.isin(d * n + q, key)).sum()) <= 8e-5 * again.n_pairs
    x = pts[d, :2] - pts[q, :2]
    x -= s.L[0] * torch.round(x / s.L[0])
    assert bool(((x.norm(dim=1) - again.dist).abs() < 1e-3).all())


def _small_checked_call(ppa, seed, stream, ws):
    import torch
    s = workloads.uniform(2000, 1.0, seed=seed)
    with torch.cuda.stream(stream):
        pts = torch.as_tensor(s.points).cuda()
        counts = torch.zeros(16, dtype=torch.int64, device="cuda")
        ppa.rdf_counts(ppa.Box(s.L, s.tilt, s.dim), pts, 16, 2.0, counts=counts, ws=ws,
                       stream=stream)
    return counts


def test_status_threads_end_beside_long_work(ppa):
    """A thread that asked for statuses ends while the device is busy with another
    stream's work: nothing it leaves behind waits for the device."""
    import os
    import threading
    import time
    import torch
    side, busy, ws = torch.cuda.Stream(), torch.cuda.Stream(), ppa.Workspace()
    want = _small_checked_call(ppa, 995, side, ws)
    a = torch.randn((8192, 8192), device="cuda", dtype=torch.bfloat16)
    b = torch.empty_like(a)
    out = {}

    def work():
        out["counts"] = _small_checked_call(ppa, 995, side, ws)
        out["tid"] = threading.get_native_id()

    torch.mm(a, a, out=b)
    torch.cuda.synchronize()
    done = torch.cuda.Event()
    with torch.cuda.stream(busy):
        for _ in range(400):  # about 0.4 s
            torch.mm(a, a, out=b)
        done.record()
    t = threading.Thread(target=work)
    t.start()
    t.join()
    end = time.monotonic() + 20.0
    while os.path.exists(f"/proc/self/task/{out['tid']}") and time.monotonic() < end:
        time.sleep(0.001)
    assert not os.path.exists(f"/proc/self/task/{out['tid']}")
    assert not done.query(), "the thread's end waited for the device"
    torch.cuda.synchronize()
    assert torch.equal(out["counts"], want)


def test_status_behind_work_past_the_polling_limit(ppa):
    """A status asked for behind several milliseconds of work (the read then waits for
    the stream), and the next ones of the same thread, behind little."""
    import time
    import torch
    s = workloads.uniform(200000, 1.0, seed=997)
    box = ppa.Box(s.L, s.tilt, s.dim)
    pts = torch.as_tensor(s.points).cuda()
    bad = pts.clone()
    bad[11, 0] = float("inf")
    want = ppa.rdf_counts(box, pts, 32, 5.0)
    torch.cuda.synchronize()
    st, ws = torch.cuda.Stream(), ppa.Workspace()
    for inputs, code in ((pts, ppa.PPA_OK), (bad, ppa.PPA_ENONFINITE)):
        h = torch.zeros(32, dtype=torch.int64, device="cuda")
        torch.cuda.synchronize()
        for _ in range(40):
            ppa.rdf_counts(box, pts, 32, 5.0, counts=h, ws=ws, stream=st, check=False)
        ppa.rdf_counts(box, inputs, 32, 5.0, counts=torch.zeros_like(h), ws=ws, stream=st,
                       check=False)
        t0 = time.perf_counter()
        rc = ws.status(st)
        assert time.perf_counter() - t0 > 2e-3  # past the polling limit
        assert rc == code and torch.equal(h, 40 * want)
        ppa.rdf_counts(box, pts, 32, 5.0, counts=h, ws=ws, stream=st, check=False)
        assert ws.status(st) == ppa.PPA_OK and torch.equal(h, 41 * want)


def test_status_of_many_threads_at_once(ppa):
    """More threads than places for published statuses, each with its own answer."""
    import threading
    import torch
    s = workloads.uniform(3000, 1.0, seed=998)
    box = ppa.Box(s.L, s.tilt, s.dim)
    good = torch.as_tensor(s.points).cuda()
    bad = good.clone()
    bad[5, 2] = float("nan")
    torch.cuda.synchronize()
    out, gate = {}, threading.Barrier(80)

    def work(k):
        ws, h = ppa.Workspace(), torch.zeros(8, dtype=torch.int64, device="cuda")
        gate.wait()
        out[k] = []
        for rep in range(5):
            ppa.rdf_counts(box, bad if (k + rep) % 3 == 0 else good, 8, 2.0, counts=h, ws=ws,
                           check=False)
            out[k].append(ws.status())

    ts = [threading.Thread(target=work, args=(k,)) for k in range(80)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for k in range(80):
        assert out[k] == [ppa.PPA_ENONFINITE if (k + rep) % 3 == 0 else ppa.PPA_OK
                          for rep in range(5)], k


@pytest.mark.parametrize("dim,n,r_max,tilt", [(3, 900, 1.5, 0.2), (3, 20000, 1.8, 0.0),
                                              (2, 30000, 3.0, 0.3), (3, 8000, 3.4, 0.0)])
@pytest.mark.parametrize("separate", [False, True])
def test_sorted_rows_cut_off_by_the_capacity(ppa, dim, n, r_max, tilt, separate):
    """A list with sorted rows that does not fit: whole rows are sorted, and the
    row that the capacity cuts holds what the unsorted list holds there, call after
    call."""
    import ctypes
    import torch
    s = workloads.uniform(n, 1.0, seed=985 + n, dim=dim, tilt=(tilt, 0.0, 0.0))
    box = ppa.Box(s.L, s.tilt, s.dim)
    pts = torch.as_tensor(s.points).cuda()
    q = None
    if separate:
        q = pts[torch.arange(0, n, 3, device="cuda")] + 0.01
        q[:, dim:] = 0
        q = q.contiguous()
    whole = ppa.query_ball(box, pts, r_max, query_points=q)
    nq = whole.offsets.shape[0] - 1
    off = whole.offsets.cpu().numpy()
    lengths = np.diff(off)
    ws, cb = ppa.Workspace(), box.c()
    wptr, wlen = ws.get(ppa.workspace_bytes(box, n, nq if separate else 0, r_max, ppa.PPA_WS_NLIST))

    def run(cap, flags, with_dist=True):
        o = torch.zeros(nq + 1, dtype=torch.int64, device="cuda")
        i = torch.full((cap,), -1, dtype=torch.int32, device="cuda")
        d = torch.full((cap,), -1.0, device="cuda") if with_dist else None
        total = torch.zeros(1, dtype=torch.int64, device="cuda")
        p = lambda t: ctypes.c_void_p(t.data_ptr()) if t is not None else None
        rc = ppa.lib().ppa_query_ball(ctypes.byref(cb), p(pts), n, p(q), nq, r_max,
                                      0 if separate else 1, flags, wptr, wlen, p(o), None, p(i),
                                      p(d), cap, p(total), None)
        assert rc == ppa.PPA_OK
        assert ws.status(torch.cuda.default_stream()) == ppa.PPA_ECAPACITY
        assert torch.equal(o, whole.offsets) and int(total) == whole.n_pairs
        return i, d

    rng = np.random.default_rng(986)
    rows = rng.permutation(np.flatnonzero(lengths > 6))[:4]
    for row in rows:
        for left in (1, int(lengths[row]) // 2, int(lengths[row]) - 1):
            cap = int(off[row]) + left
            plain, pd = run(cap, 0)
            i, d = run(cap, ppa.PPA_SORT_ROWS)
            assert torch.equal(i[off[row]:], plain[off[row]:]), (row, left)
            assert torch.equal(d[off[row]:], pd[off[row]:])
            assert torch.equal(run(cap, ppa.PPA_SORT_ROWS, False)[0], i)
            j = max(0, row - 50)
            for k in range(j, row):
                assert torch.equal(i[off[k]:off[k + 1]], plain[off[k]:off[k + 1]].sort().values)


@pytest.mark.parametrize("n", [97, 128, 1000, 2049, 4096])
@pytest.mark.parametrize("blobs", [1, 4, 40])
def test_small_builds_with_crowded_cells(ppa, n, blobs):
    """Rows of small systems whose points crowd a few cells: those of the general build
    (points far from all others beside them), each stencil cell's by index, call
    after call."""
    import torch
    rng = np.random.default_rng(988 + n + blobs)
    L, r_max = 26.0, 1.2
    at = rng.uniform(-8, 8, size=(blobs, 3))
    pts = at[rng.integers(0, blobs, n)] + rng.normal(0, 0.2 if blobs == 1 else 0.5, size=(n, 3))
    far = rng.uniform(-12.9, 12.9, size=(20000, 3))
    far = far[np.abs(far).max(1) > 10.6][:4097]
    assert far.shape[0] == 4097  # past the one-workgroup build
    pts = np.clip(pts, -9.2, 9.2).astype(np.float32)
    box = ppa.Box((L, L, L), (0.0, 0.0, 0.0), 3)

    def rows(points, m):
        nl = ppa.query_ball(box, torch.as_tensor(points.astype(np.float32)).cuda(), r_max)
        return nl.offsets.cpu().numpy()[:m + 1], nl.point_idx.cpu().numpy(), nl.dist.cpu().numpy()

    off, idx, dist = rows(pts, n)
    # each list is in the stencil order of its own grid, with coordinates rounded in
    # its cells (at most 13 wide: a distance is off by up to 4 roundings of 6.5)
    off2, idx2, _ = rows(np.concatenate([pts, far]), n)
    assert np.array_equal(off, off2)
    for i in range(0, n, max(1, n // 60)):
        a, b = slice(off[i], off[i + 1]), slice(off2[i], off2[i + 1])
        assert np.array_equal(np.sort(idx[a]), np.sort(idx2[b]))
        d = np.linalg.norm(pts[idx[a]].astype(np.float64) - pts[i].astype(np.float64), axis=1)
        assert np.all(np.abs(dist[a] - d) <= 5 * 2.0 ** -24 * 6.5)
        # runs of ascending indices: at most one per stencil cell
        assert int((np.diff(idx[a]) < 0).sum()) <= 26
    again = rows(pts, n)
    assert np.array_equal(idx, again[1]) and np.array_equal(dist, again[2])
