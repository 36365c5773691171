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
