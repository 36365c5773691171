"""The one-pass X2 graph (accumulators in LDS pages) against the two-pass kernels, bit for bit,
where its pages change: fewer pages than the limit (all given out in order), page tables at their
edges, every page table size, vertices numbered at random (pages run out, room is made or the
two-pass kernels take the row), rows with padding between entries, more kept entries than the
first staging width."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _both(gb, col, val, tau, monkeypatch):
    import torch
    Hc, Hv = torch.from_numpy(col).cuda(), torch.from_numpy(val).cuda()
    out = []
    for sets in (None, "bitmap"):
        if sets:
            monkeypatch.setenv("GB_VERTEX_SETS", sets)
        else:
            monkeypatch.delenv("GB_VERTEX_SETS", raising=False)
        out.append([t.cpu().numpy() for t in gb.build_graph(Hc, Hv, tau).arrays()])
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
    return out[0]


def _ring(N, reach, seed, order=None):
    """Symmetric H coupling every vertex to the `reach` next ones on a ring, renumbered."""
    rng = np.random.default_rng(seed)
    name = np.arange(N) if order is None else order
    off = [o for o in range(-reach, reach + 1)]
    up = rng.uniform(-0.3, 0.3, (reach + 1, N))
    col = np.empty((N, len(off)), dtype=np.int64)
    val = np.empty((N, len(off)))
    for q, o in enumerate(off):
        col[:, q] = (np.arange(N) + o) % N
        val[:, q] = up[o] if o >= 0 else np.roll(up[-o], -o)
    out_c = np.empty_like(col)
    out_v = np.empty_like(val)
    out_c[name], out_v[name] = name[col], val
    s = np.argsort(out_c, axis=1)
    return (np.take_along_axis(out_c, s, 1).astype(np.int32),
            np.ascontiguousarray(np.take_along_axis(out_v, s, 1)))


@pytest.mark.parametrize("N", [1, 2, 31, 33, 6143, 6144, 6177, 65536, 65569, 131100])
def test_sizes_at_the_page_tables_edges(N, monkeypatch):
    import paper_1603_00937_amd as gb
    reach = min(20, max(0, (N - 1) // 2))
    col, val = _ring(N, reach, N)
    rp, cl = _both(gb, col, val, 1e-4, monkeypatch)
    assert rp[-1] >= N


@pytest.mark.parametrize("N", [9000, 40000])
def test_vertices_numbered_at_random(N, monkeypatch):
    import paper_1603_00937_amd as gb
    col, val = _ring(N, 90, 5, np.random.default_rng(6).permutation(N))
    _both(gb, col, val, 1e-4, monkeypatch)


def test_padding_inside_rows(monkeypatch):
    """Entries of a row k behind a gap still count; row i's own list ends at its first gap."""
    import paper_1603_00937_amd as gb
    col, val = _ring(3000, 12, 8)
    gap = np.random.default_rng(9).random(col.shape) < 0.2
    gap[:, 12] = False
    col[gap], val[gap] = -1, 0.0
    _both(gb, col, val, 1e-4, monkeypatch)


def test_more_kept_entries_than_the_staging_width(monkeypatch):
    import paper_1603_00937_amd as gb
    rng = np.random.default_rng(4)
    N = 2500
    col, val = _ring(N, 40, 4)
    hub = rng.choice(N, 400, replace=False)  # one vertex coupled to many: two hops reach all
    wide = np.full((N, 500), -1, dtype=np.int32)
    wv = np.zeros((N, 500))
    wide[:, :col.shape[1]], wv[:, :col.shape[1]] = col, val
    row = np.unique(np.concatenate([col[0], hub]))
    wide[0, :len(row)], wv[0, :len(row)] = row, 0.05
    rp, cl = _both(gb, wide, wv, 1e-12, monkeypatch)
    assert np.diff(rp).max() > 2048
