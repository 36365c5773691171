"""Blocks whose rows end anywhere in a chunk of the contraction, a wave's block or a tile: the
squares multiply no padding, and write it as zeros, for every kernel variant.  One block holds
the whole matrix, so D is the projector of the dense eigenproblem: the stop test leaves
sum lambda (1 - lambda) <= 1e-10 N / 1024 over the core, which bounds the FP64 error of an entry by
twice that and the rounding of some twenty squares.  The low precisions keep the rounding of up to 25
squares of values of 22 bits or more, which adds up as sqrt(n) 2^-22 each (a lost chunk of the
contraction changes entries by 1e-2), and a split square gives
the same bits with its split under the products (6, 7) as without (1, 2)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _dense(n):
    rng = np.random.default_rng(n)
    q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    occ = n // 3
    e = np.concatenate([-1 + 0.5 * rng.random(occ), 0.5 + 0.5 * rng.random(n - occ)])
    h = (q * e) @ q.T
    return 0.5 * (h + h.T), q[:, :occ] @ q[:, :occ].T, occ


@pytest.mark.parametrize("n", [3, 31, 33, 64, 79, 81, 96, 97, 129, 191, 300])
@pytest.mark.parametrize("precision,policies", [("fp64", (0, 1, 2, 4, 5)), ("fp32", (0, 1, 2, 4, 5)),
                                                ("fp16x3", (1, 6, 2, 7)), ("bf16x6", (1, 2))])
def test_rows_end_anywhere(n, precision, policies):
    import torch
    import paper_1603_00937_amd as gb
    h, d, occ = _dense(n)
    hc = torch.arange(n, dtype=torch.int32).repeat(n, 1).cuda()
    hv = torch.from_numpy(h).cuda()
    bar = 2e-10 * n / 1024 + 1e-13 * n if precision == "fp64" else 25 * n ** 0.5 * 2.0 ** -22
    for policy in policies:
        cols, got, st = gb.density(hc, hv, occ, 1e-9, core_size=n, precision=precision,
                                   tile_policy=policy)
        assert st["converged"]
        full = np.zeros((n, n))
        c, v = cols.cpu().numpy(), got.cpu().numpy().astype(np.float64)
        for i in range(n):
            ok = (c[i] >= 0) & (c[i] < n)
            full[i, c[i][ok]] = v[i][ok]
        assert np.abs(full - d).max() <= bar, (policy, np.abs(full - d).max())
        if policy in (6, 7):
            assert np.array_equal(full, last)
        last = full
        if precision == "fp64":  # one sum per entry, whatever the tile
            first = full if policy == 0 else first
            assert np.array_equal(full, first)


@pytest.mark.parametrize("sizes", [(300,), (40, 300), (200, 130, 70), (64,) * 9, (500, 20, 20)])
def test_few_blocks_over_all_queues(sizes):
    """Launch orders that cut blocks across XCDs give the bits of the plain order."""
    import torch
    import paper_1603_00937_amd as gb
    n, w = sum(sizes), max(sizes)
    hc = torch.full((n, w), -1, dtype=torch.int32)
    hv = torch.zeros((n, w), dtype=torch.float64)
    occ, at = 0, 0
    for b in sizes:
        h, _, k = _dense(b)
        hc[at:at + b, :b] = torch.arange(at, at + b, dtype=torch.int32)
        hv[at:at + b, :b] = torch.from_numpy(h)
        occ, at = occ + k, at + b
    hc, hv = hc.cuda(), hv.cuda()
    part = gb.partition(gb.build_graph(hc, hv, 1e-9), 20)
    got = []
    for order in ("plain", "xcd"):
        for policy in ("64r", 2, 1):
            _, d, st = gb.density(hc, hv, occ, 1e-9, partition=part, tile_order=order,
                                  tile_policy=policy)
            assert st["converged"]
            got.append(torch.nan_to_num(d).cpu())
    assert all(torch.equal(got[i], got[i + 3]) for i in range(3))


@pytest.mark.parametrize("precision,blocks,n", [("fp64", 128, 256), ("fp64", 129, 256),
                                                ("fp32", 40, 256), ("fp32", 41, 256)])
def test_small_batches_change_no_bit(precision, blocks, n):
    """The last batch on 32-edge tiles and the first on 64-edge ones, against the 64-edge kernel.
    (FP32 results are compared through the loop's traces: the FP64 steps after it use the tiles
    of their own policy.)"""
    import torch
    import paper_1603_00937_amd as gb
    h, _, occ = _dense(n)
    rows = torch.arange(blocks * n, dtype=torch.int32)[:, None] // n * n
    hc = (rows + torch.arange(n, dtype=torch.int32)[None]).contiguous().cuda()
    hv = torch.from_numpy(np.tile(h, (blocks, 1))).cuda()
    part = gb.partition(gb.build_graph(hc, hv, 1e-9), n)
    out = [gb.density(hc, hv, blocks * occ, 1e-9, partition=part, precision=precision,
                      tile_policy=p) for p in ("auto", "64r")]
    assert out[0][2]["t2"] == out[1][2]["t2"] and out[0][2]["converged"]
    if precision == "fp64":
        assert torch.equal(out[0][1], out[1][1])
