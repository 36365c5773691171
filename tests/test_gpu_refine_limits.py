"""A given number of refinement steps is an upper bound for every refinement, and the refinement on
whole blocks starts where the low-precision loop ends by itself."""
import pytest

pytestmark = pytest.mark.gpu


def _system(model_cache):
    import torch
    m = model_cache("small256")
    return torch.from_numpy(m["H_col"]).cuda(), torch.from_numpy(m["H_val"]).cuda(), m["n_occ"]


@pytest.mark.parametrize("n_refine", [1, 2, 3, 4, 0])
@pytest.mark.parametrize("tol", [1e-4, 1e-6, 1e-8, 1e-11])
@pytest.mark.parametrize("mode", ["device", "host"])
def test_refinement_takes_no_more_steps_than_given(model_cache, n_refine, tol, mode):
    """One bf16 plane leaves eigenvalues a percent off, too far for a few steps to reach the
    tolerance: a run that stops at its last order must not have gone past it."""
    import paper_1603_00937_amd as gb
    Hc, Hv, occ = _system(model_cache)
    _, _, st = gb.density(Hc, Hv, occ, 1e-5, core_size=16, precision="bf16", idem_tol=tol,
                          n_refine=n_refine, launch_mode=mode)
    assert st["n_refine_done"] <= (n_refine or 8)
    assert st["converged"] == (st["idem"] <= tol)
    if n_refine in (0, 4):  # no limit on the orders
        assert st["converged"]


def _pairs(eps, n_pairs=64, weak=0.1):
    """Pairs of sites, two of the pairs weakly coupled: with the pairs as cores, each of those two
    subgraphs holds one site of the other pair, whose level lies in the middle of the gap and hardly
    reaches the core."""
    import numpy as np
    import torch
    n = 2 * n_pairs
    col = np.full((n, 3), -1, dtype=np.int32)
    val = np.zeros((n, 3))
    for i in range(n):
        row = {i: 0.0, i ^ 1: 1.0}
        if i in (1, 2):
            row.update({i: eps, 3 - i: weak})
        for q, j in enumerate(sorted(row)):
            col[i, q], val[i, q] = j, row[j]
    return torch.from_numpy(col).cuda(), torch.from_numpy(val).cuda(), n_pairs


@pytest.mark.parametrize("eps", [0.0, 0.002, 0.006])
@pytest.mark.parametrize("precision", ["fp32", "fp16x3"])
@pytest.mark.parametrize("refine", ["mcweeny", "mcweeny_blocks"])
@pytest.mark.parametrize("mode", ["device", "host"])
def test_levels_in_the_gap_resume_the_loop(eps, precision, refine, mode):
    """The early hand-over finds such a level halfway between empty and filled, where eight steps
    end nowhere; the loop's own end does not."""
    import torch
    import paper_1603_00937_amd as gb
    Hc, Hv, occ = _pairs(eps)
    part = gb.partition(gb.build_graph(Hc, Hv, 0.05, mode="pattern"), 2)
    assert part.max_sub == 3
    kw = dict(partition=part, precision=precision, launch_mode=mode)
    _, _, st = gb.density(Hc, Hv, occ, 1e-5, refine=refine, check_idem=True, **kw)
    assert st["converged"] and st["n_refine_done"] <= 8
    assert st["idem_max"] <= 1e-9 and abs(st["trace"] - occ) <= 0.05
