"""The Chebyshev recurrence on core rows at the subgraph sizes where its kernel changes form: rows
per workgroup drop from four to two to one as two LDS arrays stop fitting (past 2528 and 5056
vertices), and V_{n-1} leaves LDS past 10112; sizes off the wave and block edges, cores that
leave the last workgroup fewer rows."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _chain(N, seed):
    """A banded symmetric H (five entries per row) as ELL."""
    rng = np.random.default_rng(seed)
    d0, d1, d2 = (rng.uniform(-1.0, 1.0, N) for _ in range(3))
    col = np.full((N, 5), -1, dtype=np.int32)
    val = np.zeros((N, 5))
    for i in range(N):
        e = [(i - 2, 0.2 * d2[i - 2]), (i - 1, 0.4 * d1[i - 1]), (i, d0[i]),
             (i + 1, 0.4 * d1[i]), (i + 2, 0.2 * d2[i])]
        e = [x for x in e if 0 <= x[0] < N]
        col[i, :len(e)] = [x[0] for x in e]
        val[i, :len(e)] = [x[1] for x in e]
    return col, val


@pytest.mark.parametrize("N,order", [(61, 2), (129, 9), (2528, 6), (2531, 7), (5060, 6),
                                     (10130, 5)])
def test_row_recurrence_at_its_size_limits(N, order):
    import scipy.sparse as sp
    import torch
    import paper_1603_00937_amd as gb
    col, val = _chain(N, N)
    beta, mu = 3.0, 0.1
    Hc, Hv = torch.from_numpy(col).cuda(), torch.from_numpy(val).cuda()
    D_col, D_val, st = gb.foe_density(Hc, Hv, N // 2, 1e-9, beta, order, mu=mu, core_size=N)
    assert st["n_sub"] == 1 and st["max_sub"] == N and st["n_product"] == order - 1
    c = gb.chebyshev_fermi(st["emin"], st["emax"], beta, mu, order)
    r, t = np.nonzero(col >= 0)
    H = sp.csr_matrix((val[r, t], (r, col[r, t])), shape=(N, N))
    Ht = (2.0 * H - (st["emax"] + st["emin"]) * sp.identity(N)) / (st["emax"] - st["emin"])
    picks = sorted({0, 1, N // 3, N - 2, N - 1})
    t0 = np.zeros((N, len(picks)))
    t0[picks, range(len(picks))] = 1.0
    t1 = Ht @ t0
    want = c[0] * t0 + c[1] * t1
    for n in range(2, order + 1):
        t0, t1 = t1, 2.0 * (Ht @ t1) - t0
        want += c[n] * t1
    got = D_val[picks].cpu().numpy().T
    assert np.array_equal(D_col[picks[0]].cpu().numpy(), np.arange(N))
    # each term adds a few roundings of values of at most one
    assert np.abs(got - want).max() <= 1e-14 * order
    # the recorded traces (from products of two terms) give the trace of the sum
    tr = float(sum(ci * ti for ci, ti in zip(c, st["traces"])))
    assert abs(tr - float(D_val.diagonal().sum())) <= 1e-12 * N
