"""Multilevel communities on graphs unlike the benchmark's (every list of candidates the same, one
orbital per site, vertices numbered at random): the cores of the host partitioner, in a time
that does not grow with the rows that the matching asks for one by one."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _pattern(gb, n, edges):
    """Graph object of a dense boolean pattern."""
    import torch
    w = int(edges.sum(1).max())
    col = np.full((n, w), -1, dtype=np.int32)
    for i in range(n):
        c = np.nonzero(edges[i])[0]
        col[i, :len(c)] = c
    val = np.where(col >= 0, 1.0, 0.0)
    return gb.build_graph(torch.from_numpy(col).cuda(), torch.from_numpy(val).cuda(), 0.5,
                          mode="pattern")


def _host_cores(gb, g, core):
    rp, col = [t.cpu().numpy() for t in g.arrays()]
    return gb.partition_host(rp, col, core)


def _check(gb, g, core):
    import torch
    p = gb.partition(g, core, "multilevel")
    cp, sp, si = [t.cpu().numpy() for t in p.arrays()]
    want = _host_cores(gb, g, core)
    assert np.array_equal(cp, want[0])
    got = np.concatenate([si[sp[s]:sp[s] + cp[s + 1] - cp[s]] for s in range(len(cp) - 1)])
    assert np.array_equal(got, want[1])
    torch.cuda.synchronize()


def _time(f, reps=5):
    import torch
    best = np.inf
    for _ in range(reps):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        f()
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t0)
    return best


def _lattice_pattern(L, reach):
    n = L ** 3
    x = np.indices((L, L, L)).reshape(3, -1).T
    e = np.zeros((n, n), dtype=bool)
    for o in np.indices((2 * reach + 1,) * 3).reshape(3, -1).T - reach:
        y = (x + o) % L
        e[np.arange(n), (y[:, 0] * L + y[:, 1]) * L + y[:, 2]] = True
    return e


@pytest.mark.parametrize("n", [2, 13, 14, 300])
@pytest.mark.parametrize("core", [8, 32])
def test_cores_of_complete_graphs(n, core):
    import paper_1603_00937_amd as gb
    _check(gb, _pattern(gb, n, np.ones((n, n), dtype=bool)), core)


@pytest.mark.parametrize("L,core", [(8, 32), (12, 8), (16, 32)])
def test_cores_of_lattices(L, core):
    import paper_1603_00937_amd as gb
    _check(gb, _pattern(gb, L ** 3, _lattice_pattern(L, 2)), core)


@pytest.mark.parametrize("kind", ["complete", "lattice"])
def test_rows_are_not_fetched_one_by_one(kind):
    """In a complete graph half the vertices find every listed candidate taken; a fetch for each
    is what the same number of small copies takes, and the whole graph is much less."""
    import torch
    import paper_1603_00937_amd as gb
    if kind == "complete":
        g, copies = _pattern(gb, 2000, np.ones((2000, 2000), dtype=bool)), 2 * 988
    else:
        g, copies = _pattern(gb, 4096, _lattice_pattern(16, 2)), 2 * 124
    one = torch.zeros(1, dtype=torch.int32, device="cuda")
    small = _time(lambda: [one.cpu() for _ in range(copies // 2)])
    own = _time(lambda: gb.partition(g, 32, "multilevel"))
    base = _time(lambda: gb.partition(g, 32, "block"))
    print(f"{kind}: {own * 1e3:.2f} ms, block {base * 1e3:.2f}, copies {small * 1e3:.2f}")
    assert own - base <= 0.6 * small + 0.002, (own, base, small)


def _renumbered(n_sites, seed):
    import torch
    import paper_1603_00937_amd as gb
    from synth.model import ModelSpec, make_model
    m = make_model(ModelSpec(n_sites=n_sites, seed=2))
    n = m["N"]
    p = np.random.default_rng(seed).permutation(n)
    out = []
    for name in (np.arange(n), p):
        c = np.where(m["H_col"] >= 0, name[np.maximum(m["H_col"], 0)], n)
        s = np.argsort(c, axis=1, kind="stable")
        c, v = np.take_along_axis(c, s, 1), np.take_along_axis(m["H_val"], s, 1)
        col, val = np.empty_like(m["H_col"]), np.empty_like(m["H_val"])
        col[name], val[name] = np.where(c == n, -1, c), v
        out.append(gb.build_graph(torch.from_numpy(col).cuda(), torch.from_numpy(val).cuda(), 1e-5))
    return out


def test_cores_with_random_numbers():
    import paper_1603_00937_amd as gb
    for g in _renumbered(700, 5):
        _check(gb, g, 32)


def test_random_numbers_cost_little():
    """18000 randomly numbered vertices against the same graph in place order: the host's part takes
    longer (its look-ups jump), the weights must not take twice what entries cost on top."""
    import paper_1603_00937_amd as gb
    ordered, shuffled = _renumbered(9000, 5)
    a = _time(lambda: gb.partition(ordered, 32, "multilevel"), 10)
    b = _time(lambda: gb.partition(shuffled, 32, "multilevel"), 10)
    assert b <= 1.75 * a, (a, b)
