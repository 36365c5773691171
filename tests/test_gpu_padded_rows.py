"""Rows that are mostly padding (an ELL kept wide for later systems) are not read past their end."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,width", [(4096, 2248), (20000, 2100)])
def test_bounds_of_padded_rows(n, width):
    import torch
    import paper_1603_00937_amd as gb
    rng = np.random.default_rng(n)
    m = 200
    col = np.sort((np.arange(n)[:, None] + np.arange(m)) % n, axis=1).astype(np.int32)
    val = rng.normal(0.0, 1.0, (n, m))
    Hc, Hv = torch.from_numpy(col).cuda(), torch.from_numpy(val).cuda()
    Wc = torch.nn.functional.pad(Hc, (0, width - m), value=-1).contiguous()
    Wv = torch.nn.functional.pad(Hv, (0, width - m)).contiguous()
    want = gb.spectral_bounds(Hc, Hv)
    assert gb.spectral_bounds(Wc, Wv) == want and gb.spectral_bounds_noalloc(Wc, Wv) == want

    def best(a, b):
        t = np.inf
        for _ in range(10):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            gb.spectral_bounds(a, b)
            t = min(t, time.perf_counter() - t0)
        return t
    assert best(Wc, Wv) <= 1.6 * best(Hc, Hv) + 2e-5
