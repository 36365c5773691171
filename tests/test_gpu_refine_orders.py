"""The core-row refinement at every order it can end at, and past its last one: loose tolerances
end at S_2 or S_3, tight ones at S_6, and one that rounding keeps out of reach sends the low-precision
loop on and then the whole blocks.  Device- and host-driven loops agree bit for bit, and D meets
the 1e-6 bar of the mixed path against the FP64 D."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,core", [("fp32", 16), ("fp16x3", 16), ("fp16x3", 31)])
@pytest.mark.parametrize("tol", [1e-4, 1e-7, 1e-10, 1e-15])
def test_orders_and_fallback(model_cache, precision, core, tol):
    import torch
    import paper_1603_00937_amd as gb
    m = model_cache("small256")
    Hc, Hv = torch.from_numpy(m["H_col"]).cuda(), torch.from_numpy(m["H_val"]).cuda()
    _, ref, _ = gb.density(Hc, Hv, m["n_occ"], 1e-5, core_size=core)
    out = []
    for mode in ("device", "host"):
        _, D, st = gb.density(Hc, Hv, m["n_occ"], 1e-5, core_size=core, precision=precision,
                              idem_tol=tol, launch_mode=mode, check_idem=True)
        out.append((D.cpu().numpy(), st["iters"], st["n_refine_done"], st["converged"]))
        assert st["converged"] == (st["idem"] <= tol)
        # |D^2 - D| on the core columns: the summed measure and the rounding of one row
        assert st["idem_max"] <= tol + 1e-9
    assert np.array_equal(out[0][0], out[1][0]) and out[0][1:] == out[1][1:]
    assert np.abs(out[0][0] - ref.cpu().numpy()).max() <= max(1e-6, tol)


def test_given_step_counts_are_kept(model_cache):
    """n_refine = 1 takes one McWeeny step from the loop's own floor, as it always did."""
    import torch
    import paper_1603_00937_amd as gb
    m = model_cache("small256")
    Hc, Hv = torch.from_numpy(m["H_col"]).cuda(), torch.from_numpy(m["H_val"]).cuda()
    _, _, auto = gb.density(Hc, Hv, m["n_occ"], 1e-5, core_size=16, precision="fp32")
    _, _, one = gb.density(Hc, Hv, m["n_occ"], 1e-5, core_size=16, precision="fp32", n_refine=1)
    assert one["n_refine_done"] == 1 and one["converged"]
    assert one["iters"] >= auto["iters"]
