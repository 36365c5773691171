"""Which kernels build the X2 graph: the same graph on every route, the widths that are refused are
refused on all of them, and a call is never much slower than on the kernels that it could have
taken instead (vertices numbered at random, narrow matrices, thresholds near rounding)."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _lattice(L, reach=1):
    """One orbital per site of an L^3 periodic lattice, all sites within `reach` per axis."""
    x = np.indices((L, L, L)).reshape(3, -1).T
    off = np.indices((2 * reach + 1,) * 3).reshape(3, -1).T - reach
    col = np.empty((L ** 3, len(off)), dtype=np.int64)
    for q, o in enumerate(off):
        y = (x + o) % L
        col[:, q] = (y[:, 0] * L + y[:, 1]) * L + y[:, 2]
    col.sort(axis=1)
    rows = np.arange(L ** 3)[:, None]
    val = np.where(col == rows, np.where(rows % 2 == 0, -1.5, 1.5), -0.05)
    return col.astype(np.int32), val


def _renumbered(col, val, seed):
    """The same matrix with its vertices numbered at random."""
    n = len(col)
    p = np.random.default_rng(seed).permutation(n)
    c = np.where(col >= 0, p[np.maximum(col, 0)], n)
    s = np.argsort(c, axis=1, kind="stable")
    c, v = np.take_along_axis(c, s, 1), np.take_along_axis(val, s, 1)
    out_c, out_v = np.empty_like(col), np.empty_like(val)
    out_c[p], out_v[p] = np.where(c == n, -1, c), v
    return out_c, out_v


def _build(gb, Hc, Hv, tau, monkeypatch, sets, reps=15):
    """The graph and the fastest of a few builds, in seconds."""
    import torch
    if sets:
        monkeypatch.setenv("GB_VERTEX_SETS", sets)
    else:
        monkeypatch.delenv("GB_VERTEX_SETS", raising=False)
    best = np.inf
    for _ in range(reps):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        g = gb.build_graph(Hc, Hv, tau)
        best = min(best, time.perf_counter() - t0)
    return [t.cpu().numpy() for t in g.arrays()], best


def _same_and_not_slower(col, val, tau, monkeypatch, factor, sets="bitmap"):
    import torch
    import paper_1603_00937_amd as gb
    Hc, Hv = torch.from_numpy(col).cuda(), torch.from_numpy(val).cuda()
    want, other = _build(gb, Hc, Hv, tau, monkeypatch, sets)
    got, own = _build(gb, Hc, Hv, tau, monkeypatch, None)
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
    assert own <= factor * other, (own, other)


@pytest.mark.parametrize("n,width,sets", [(1100, 1025, None), (1100, 1025, "bitmap"),
                                          (1100, 1025, "hash"), (140000, 1030, None)])
def test_wide_rows_are_refused_on_every_route(n, width, sets, monkeypatch):
    import torch
    import paper_1603_00937_amd as gb
    if sets:
        monkeypatch.setenv("GB_VERTEX_SETS", sets)
    col = torch.full((n, width), -1, dtype=torch.int32, device="cuda")
    val = torch.zeros((n, width), dtype=torch.float64, device="cuda")
    i = torch.arange(n, device="cuda")
    col[:, 0], val[:, 0] = i.int(), torch.where(i % 2 == 0, 1.0, -1.0).double()
    for tau in (1e-5, 0.0):
        with pytest.raises(gb.GbError, match="width"):
            gb.build_graph(col, val, tau)
    narrow = gb.build_graph(col[:, :1024].contiguous(), val[:, :1024].contiguous(), 1e-5)
    assert narrow.nnz == n


@pytest.mark.parametrize("tau", [1e-300, 1e-16, 1e-15, 1e-14])
def test_threshold_within_rounding(model_cache, tau, monkeypatch):
    """Below the rounding of the sums every pair's sum is decided in ascending order; what no pair
    reaches is not."""
    m = model_cache("n1024")
    _same_and_not_slower(m["H_col"], m["H_val"], tau, monkeypatch, 3.0)


@pytest.mark.parametrize("L,reach,sets", [(10, 1, "bitmap"), (24, 1, "bitmap"), (32, 2, "bitmap"),
                                          (44, 1, "bitmap"), (55, 1, "hash"), (80, 1, "hash")])
def test_narrow_matrices(L, reach, sets, monkeypatch):
    """A few pairs per row do not pay for the pages; sets: what such a matrix takes instead."""
    col, val = _lattice(L, reach)
    _same_and_not_slower(col, val, 1e-9, monkeypatch, 1.35, sets)


def _ring(N, reach, seed):
    """Symmetric H coupling every vertex to the `reach` next ones on a ring."""
    rng = np.random.default_rng(seed)
    up = rng.uniform(-0.3, 0.3, (reach + 1, N))
    off = np.arange(-reach, reach + 1)
    col = (np.arange(N)[:, None] + off) % N
    val = np.stack([up[o] if o >= 0 else np.roll(up[-o], -o) for o in off], axis=1)
    s = np.argsort(col, axis=1, kind="stable")
    return (np.take_along_axis(col, s, 1).astype(np.int32),
            np.ascontiguousarray(np.take_along_axis(val, s, 1)))


def _same(col, val, tau, monkeypatch):
    import torch
    import paper_1603_00937_amd as gb
    Hc, Hv = torch.from_numpy(col).cuda(), torch.from_numpy(val).cuda()
    want, _ = _build(gb, Hc, Hv, tau, monkeypatch, "hash" if len(col) > 1 << 18 else "bitmap", 1)
    got, _ = _build(gb, Hc, Hv, tau, monkeypatch, None, 1)
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])


@pytest.mark.parametrize("N,reach", [(97, 48), (200, 95), (1000, 50), (4096, 48), (4097, 96),
                                     (6143, 96), (6144, 96), (6177, 100), (65536, 96), (65537, 64),
                                     (98305, 32), (114689, 1), (131100, 16), (262200, 17),
                                     (1048700, 16)])
def test_one_pass_at_the_edges_of_its_page_tables(N, reach, monkeypatch):
    """Rows just wide enough for one pass at every size where the choice or the pages change."""
    _same(*_ring(N, reach, N), 1e-3, monkeypatch)


def test_one_pass_with_padding_inside_rows(monkeypatch):
    col, val = _ring(3000, 60, 8)
    gap = np.random.default_rng(9).random(col.shape) < 0.2
    gap[np.arange(3000)[:, None] == col] = False
    col[gap], val[gap] = -1, 0.0
    _same(col, val, 1e-4, monkeypatch)


@pytest.mark.parametrize("N,reach", [(5000, 100), (9000, 100), (40000, 100), (140000, 20),
                                     (140000, 60), (140000, 160), (200000, 60), (200000, 160)])
def test_one_pass_with_random_numbers(N, reach, monkeypatch):
    """All pages given out in order, too many of them, as many as room can be made for, and more."""
    _same(*_renumbered(*_ring(N, reach, 5), 6), 1e-4, monkeypatch)


@pytest.mark.parametrize("N", [6400, 18000])
def test_random_numbers_cost_little(N, monkeypatch):
    """The pages of a randomly numbered system do not fit: that is found out early."""
    from synth.model import ModelSpec, make_model
    m = make_model(ModelSpec(n_sites=N // 2, seed=2))
    col, val = _renumbered(m["H_col"], m["H_val"], 3)
    _same_and_not_slower(col, val, 1e-5, monkeypatch, 1.7)
