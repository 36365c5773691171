"""Row scans of an ELL matrix at the edges of their waves (row groups of 16 and 64, slots in runs of
64): Gershgorin ends summed in slot order, entries above a threshold, both up to a row's first
padding entry.  Bit for bit against plain loops."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (2, 3), (15, 63), (16, 64), (17, 65), (65, 130), (200, 129), (70000, 5)]


def _ell(n, w, gaps):
    """Random rows (ascending distinct columns, the diagonal among them), some cut by a gap."""
    rng = np.random.default_rng([n, w])
    col = np.full((n, w), -1, dtype=np.int32)
    val = np.zeros((n, w))
    for i in range(n):
        m = min(n, int(rng.integers(1, w + 1)))
        off = rng.choice(min(n, 4 * w), size=m, replace=False)
        c = np.unique(np.append((i + off[1:]) % n, i))
        col[i, :len(c)] = c
        val[i, :len(c)] = rng.normal(0.0, 1.0, len(c))
        if gaps and len(c) > 4 and i % 3 == 0:
            col[i, int(rng.integers(1, len(c)))] = -1
    return col, val


def _ends(col, val):
    lo, hi = np.inf, -np.inf
    for i, (c, v) in enumerate(zip(col.tolist(), val.tolist())):
        r = d = 0.0
        for j, x in zip(c, v):
            if j < 0:
                break
            if j == i:
                d = x
            else:
                r = r + abs(x)
        lo, hi = min(lo, d - r), max(hi, d + r)
    return lo, hi


@pytest.mark.parametrize("n,w", SIZES)
@pytest.mark.parametrize("gaps", [False, True])
def test_row_ends(n, w, gaps):
    import torch
    import paper_1603_00937_amd as gb
    col, val = _ell(n, w, gaps)
    Hc, Hv = torch.from_numpy(col).cuda(), torch.from_numpy(val).cuda()
    want = _ends(col, val)
    assert gb.spectral_bounds(Hc, Hv) == want
    assert gb.spectral_bounds_noalloc(Hc, Hv) == want


@pytest.mark.parametrize("n,w", SIZES[:-1])
def test_thresholded_pattern(n, w):
    import torch
    import paper_1603_00937_amd as gb
    col, val = _ell(n, w, True)
    tau = float(np.abs(val[val != 0]).min() if n < 3 else np.median(np.abs(val[val != 0])))
    g = gb.build_graph(torch.from_numpy(col).cuda(), torch.from_numpy(val).cuda(), tau,
                       mode="pattern")
    edges = {(i, i) for i in range(n)}
    for i in range(n):
        for j, x in zip(col[i].tolist(), val[i].tolist()):
            if j < 0:
                break
            if abs(x) >= tau:
                edges |= {(i, j), (j, i)}
    rp, cl = [t.cpu().numpy() for t in g.arrays()]
    got = [(i, int(j)) for i in range(n) for j in cl[rp[i]:rp[i + 1]]]
    assert got == sorted(edges)
