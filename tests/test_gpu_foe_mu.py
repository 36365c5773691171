"""mu and the coefficients as the device finds them, against the host entry points: the host's
coefficients at the device's mu give the wanted occupation with the recorded traces, up to the rounding
of M terms over N rows, and an occupation out of reach is refused as before."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order,nodes,beta", [(1, 0, 2.0), (2, 3, 5.0), (63, 65, 1.0),
                                              (64, 1000, 20.0), (160, 0, 10.0)])
def test_device_mu(model_cache, order, nodes, beta):
    import torch
    import paper_1603_00937_amd as gb
    m = model_cache("small256")
    hc, hv = torch.from_numpy(m["H_col"]).cuda(), torch.from_numpy(m["H_val"]).cuda()
    _, _, st = gb.foe_density(hc, hv, m["n_occ"], 1e-5, beta, order, n_nodes=nodes, core_size=16)
    c = gb.chebyshev_fermi(st["emin"], st["emax"], beta, st["mu"], order, nodes)
    tr = float(sum(ci * ti for ci, ti in zip(c, st["traces"])))
    bar = 1e-15 * m["N"] * (order + 1)
    assert abs(tr - m["n_occ"]) <= bar and abs(st["trace"] - tr) <= bar
    host = gb.foe_solve_mu(st["traces"], st["emin"], st["emax"], beta, m["n_occ"], nodes)
    # both end at neighbouring doubles around their sums' zero, which differ by rounding only
    eps = 1e-7 * (st["emax"] - st["emin"])
    up = gb.chebyshev_fermi(st["emin"], st["emax"], beta, st["mu"] + eps, order, nodes)
    slope = abs(sum(ci * ti for ci, ti in zip(up, st["traces"])) - tr) / eps
    assert abs(host - st["mu"]) * slope <= 2 * bar + 1e-15 * slope * abs(host)


def test_unreachable_occupation_is_refused(model_cache):
    import torch
    import paper_1603_00937_amd as gb
    m = model_cache("small256")
    hc, hv = torch.from_numpy(m["H_col"]).cuda(), torch.from_numpy(m["H_val"]).cuda()
    with pytest.raises(gb.GbError, match="reachable"):
        gb.foe_density(hc, hv, m["N"] - 1, 1e-5, 0.5, 20, core_size=16)


@pytest.mark.parametrize("N,order", [(61, 1), (61, 2), (129, 9), (2531, 7), (5060, 6), (10130, 5)])
def test_kept_terms_change_no_bit(N, order):
    """The second pass goes on from the terms that the first one kept: D is that of one pass at
    the mu it found, in every form of the kernel."""
    import torch
    import paper_1603_00937_amd as gb
    from test_gpu_foe_rows import _chain
    col, val = _chain(N, N)
    hc, hv = torch.from_numpy(col).cuda(), torch.from_numpy(val).cuda()
    _, d2, st = gb.foe_density(hc, hv, N // 2, 1e-9, 3.0, order, core_size=N)
    _, d1, one = gb.foe_density(hc, hv, N // 2, 1e-9, 3.0, order, mu=st["mu"], core_size=N)
    assert st["passes"] == 2 and one["passes"] == 1
    assert torch.equal(d1, d2) and st["traces"] == one["traces"]
