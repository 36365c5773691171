"""Graphs whose coarse levels have no edges left (every component becomes one coarse vertex, or
there were none to begin with): the cores of the oracle, from the host entry point in a process of
its own (its buffers are fresh there) and from the device."""
import json
import os
import subprocess
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _cliques(sizes):
    """Disjoint complete graphs with self loops, as CSR."""
    rows, at = [], 0
    for s in sizes:
        rows += [np.arange(at, at + s)] * s
        at += s
    rp = np.zeros(at + 1, dtype=np.int32)
    rp[1:] = np.cumsum([len(r) for r in rows])
    return rp, np.concatenate(rows).astype(np.int32)


GRAPHS = {"one": [1], "pair": [2], "pairs": [2] * 40, "alone": [1] * 7, "mixed": [2, 1, 4, 1, 3, 2],
          "triples": [3] * 5}


@pytest.mark.parametrize("first", list(GRAPHS))
def test_host_cores(first):
    """Every graph, `first` the first of its process, at several core sizes."""
    code = ("import sys, json, numpy as np\n"
            "import paper_1603_00937_amd as gb\n"
            "for rp, col, core in json.load(sys.stdin):\n"
            "    cp, cv, cost = gb.partition_host(np.array(rp), np.array(col), core)\n"
            "    print(json.dumps([cp.tolist(), cv.tolist(), cost]), flush=True)\n")
    from oracle.multilevel import partition_multilevel
    names = sorted(GRAPHS, key=lambda g: g != first)
    jobs = [(*_cliques(GRAPHS[g]), core) for core in (8, 1, 32) for g in names]
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, text=True, capture_output=True,
                       input=json.dumps([[a.tolist(), b.tolist(), c] for a, b, c in jobs]))
    assert r.returncode == 0, r.stderr[-2000:]
    out = [json.loads(line) for line in r.stdout.splitlines()]
    assert len(out) == len(jobs)
    for (rp, col, core), (cp, cv, cost) in zip(jobs, out):
        want = partition_multilevel(rp, col, core)
        assert cp == list(want[0]) and cv == list(want[1]) and cost == want[2]


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(GRAPHS))
@pytest.mark.parametrize("core", [1, 8, 32])
def test_device_cores(name, core):
    import torch
    import paper_1603_00937_amd as gb
    from oracle.multilevel import partition_multilevel
    rp, col = _cliques(GRAPHS[name])
    n, w = len(rp) - 1, int(np.diff(rp).max())
    ell = np.full((n, w), -1, dtype=np.int32)
    for i in range(n):
        ell[i, :rp[i + 1] - rp[i]] = col[rp[i]:rp[i + 1]]
    g = gb.build_graph(torch.from_numpy(ell).cuda(),
                       torch.from_numpy(np.where(ell >= 0, 1.0, 0.0)).cuda(), 0.5, mode="pattern")
    p = gb.partition(g, core, "multilevel")
    cp, sp, si = [t.cpu().numpy() for t in p.arrays()]
    want = partition_multilevel(rp, col, core)
    assert np.array_equal(cp, want[0])
    got = np.concatenate([si[sp[s]:sp[s] + cp[s + 1] - cp[s]] for s in range(len(cp) - 1)])
    assert np.array_equal(got, want[1])
