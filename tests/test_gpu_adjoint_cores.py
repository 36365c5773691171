"""The adjoint at core sizes around its 64-row tiles (the first step of the reverse sweep leaves out
what the seed's core rows and columns cannot reach) and with vertex lists longer than a wave, on
every checkpoint stride in use, against the oracle's reverse recursion."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("core,stride", [(2, 0), (17, 1), (63, 4), (64, 0), (65, 2), (150, 5)])
def test_gradient_at_core_sizes(model_cache, core, stride):
    import torch
    import paper_1603_00937_amd as gb
    from synth import make_operator_v
    from oracle.sp2 import density_partitioned
    from oracle.adjoint import trace_dv_and_grad
    m = model_cache("small256")
    V = make_operator_v(m["H_col"], 51)
    Dc, Dv, info = density_partitioned(m["H_col"], m["H_val"], m["n_occ"], 1e-4, core,
                                       keep_tape=True)
    _, want = trace_dv_and_grad(m["H_col"], m["H_val"], V, m["n_occ"], info, None)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    _, _, st = gb.density(dev(m["H_col"]), dev(m["H_val"]), m["n_occ"], 1e-4, core_size=core,
                          keep_tape=True, tape_stride=stride)
    G = np.zeros(Dc.shape)
    for i in range(m["N"]):
        n = int((m["H_col"][i] >= 0).sum())
        pos = np.minimum(np.searchsorted(m["H_col"][i, :n], Dc[i]), n - 1)
        hit = (Dc[i] >= 0) & (m["H_col"][i][pos] == Dc[i])
        G[i, hit] = V[i][pos[hit]]
    got = st["tape"].vjp(dev(G)).cpu().numpy()
    assert np.abs(got - want).max() <= 1e-9 * max(1.0, np.abs(want).max())
    # the tape is not used up
    assert np.array_equal(st["tape"].vjp(dev(G)).cpu().numpy(), got)
