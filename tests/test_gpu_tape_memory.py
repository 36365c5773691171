"""The tape's memory: checkpoints that find no room thin it to every fourth iterate instead of ending
the call, and idle buffers go back to a registered allocator before a call is refused."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _hook(gb, budget=None):
    class Counting(gb.TorchAllocator):
        """Refuses what would take the library past `budget` bytes."""

        def __init__(self):
            self.budget, self.now, self.peak, self.refused = budget, 0, 0, 0
            super().__init__()

        def _alloc(self, nbytes, stream, ctx):
            if self.budget is not None and self.now + nbytes > self.budget:
                self.refused += 1
                return None
            p = super()._alloc(nbytes, stream, ctx)
            if p:
                self.now += int(nbytes)
                self.peak = max(self.peak, self.now)
            return p

        def _free(self, ptr, stream, ctx):
            self.now -= self.live.get(ptr, 0)
            super()._free(ptr, stream, ctx)
    return Counting()


def _gradient(gb, m, Hc, Hv, part, G, stride):
    D_col, D_val, st = gb.density(Hc, Hv, m["n_occ"], 1e-5, partition=part, keep_tape=True,
                                  tape_stride=stride)
    return D_val.cpu().numpy(), st["tape"].vjp(G).cpu().numpy()


@pytest.mark.parametrize("room", [0.02, 0.3, 0.6, 0.9])
def test_checkpoints_without_room(model_cache, room):
    """Room between what the tape of stride 4 and that of stride 1 take: the result is the same
    bits, wherever the first refusal comes."""
    import gc
    import torch
    import paper_1603_00937_amd as gb
    m = model_cache("n1024")
    Hc, Hv = torch.from_numpy(m["H_col"]).cuda(), torch.from_numpy(m["H_val"]).cuda()
    part = gb.partition(gb.build_graph(Hc, Hv, 1e-5), 32)
    G = torch.from_numpy(np.random.default_rng(1).normal(size=(m["N"], part.max_sub))).cuda()
    peak, want = {}, None
    for stride in (4, 1):
        gb.trim()
        hook = _hook(gb)
        gb.set_allocator(hook)
        try:
            got = _gradient(gb, m, Hc, Hv, part, G, stride)
        finally:
            gb.set_allocator(None)
        gc.collect()
        gb.trim()
        peak[stride] = hook.peak
        want = want or got
        assert all(np.array_equal(a, b) for a, b in zip(got, want))
    assert peak[1] > 1.5 * peak[4]
    hook = _hook(gb, int(peak[4] + room * (peak[1] - peak[4])))
    gb.set_allocator(hook)
    try:
        got = _gradient(gb, m, Hc, Hv, part, G, 0)
    finally:
        gb.set_allocator(None)
    assert hook.refused > 0
    assert all(np.array_equal(a, b) for a, b in zip(got, want))
    gc.collect()
    gb.trim()
    torch.cuda.synchronize()
    assert hook.live == {}


def test_a_stride_that_was_asked_for_is_kept(model_cache):
    import gc
    import torch
    import paper_1603_00937_amd as gb
    m = model_cache("small256")
    Hc, Hv = torch.from_numpy(m["H_col"]).cuda(), torch.from_numpy(m["H_val"]).cuda()
    part = gb.partition(gb.build_graph(Hc, Hv, 1e-5), 16)
    G = torch.zeros((m["N"], part.max_sub), dtype=torch.float64, device="cuda")
    gb.trim()
    hook = _hook(gb)
    gb.set_allocator(hook)
    try:
        _gradient(gb, m, Hc, Hv, part, G, 4)
        gc.collect()
        gb.trim()
        four = hook.peak
        hook = _hook(gb, four)
        gb.set_allocator(hook)
        with pytest.raises(gb.GbError, match="GB_ENOMEM"):
            _gradient(gb, m, Hc, Hv, part, G, 1)
    finally:
        gb.set_allocator(None)
    gc.collect()
    gb.trim()


def test_long_expansions_keep_every_fourth():
    """One block of 11584 rows (1 GiB an iterate) replaying 35 steps: the tape goes past 32 GiB on
    the way and ends with every fourth iterate and the same gradient."""
    import gc
    import torch
    import paper_1603_00937_amd as gb
    n, steps = 11584, 35
    i = torch.arange(n, device="cuda")
    col = torch.stack([(i + o) % n for o in (-1, 0, 1)], 1).sort(dim=1)
    val = torch.where(col.values == i[:, None], torch.where(i % 2 == 0, -1.0, 1.0)[:, None].double(),
                      torch.tensor(0.1, dtype=torch.float64, device="cuda"))
    col = col.values.int().contiguous()
    part = gb.partition(gb.build_graph(col, val, 0.05, mode="pattern"), n)
    assert part.max_sub == n
    G = torch.zeros((n, n), dtype=torch.float64, device="cuda")
    G[:, :3] = 1.0
    out = []
    for stride in (4, 0):
        gb.trim()
        hook = _hook(gb)
        gb.set_allocator(hook)
        try:
            _, _, st = gb.density(col, val, n // 2, 1e-5, partition=part, keep_tape=True,
                                  tape_stride=stride, branch_in=[k % 2 for k in range(steps)])
            out.append(st["tape"].vjp(G).cpu())
            gb.trim()
            kept = sum(b >= n * n * 8 for b in hook.live.values())
            assert kept == 1 + steps // 4
            del st
        finally:
            gb.set_allocator(None)
        gc.collect()
        gb.trim()
        assert hook.live == {}
    assert hook.peak > 32 * 1.0e9 and torch.equal(out[0], out[1])
    torch.cuda.empty_cache()
