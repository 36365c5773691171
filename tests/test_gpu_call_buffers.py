"""Buffers that a call freed serve later calls of any thread and stream: results stay the same
bits while threads, sizes, failed calls and gb_trim come in between."""
import threading

import pytest

pytestmark = pytest.mark.gpu


def test_threads_sizes_failures_and_trim(model_cache):
    import torch
    import paper_1603_00937_amd as gb
    m = model_cache("small256")
    hc, hv = torch.from_numpy(m["H_col"]).cuda(), torch.from_numpy(m["H_val"]).cuda()
    bad = hv.clone()
    bad[3, 0] = float("nan")

    def run(core):
        return gb.density(hc, hv, m["n_occ"], 1e-5, core_size=core)[1].nan_to_num().cpu()

    ref = {core: run(core) for core in (8, 16, 32)}
    wrong = []

    def work(seed):
        with torch.cuda.stream(torch.cuda.Stream()):
            for i in range(6):
                core = (8, 16, 32)[(seed + i) % 3]
                if not torch.equal(run(core), ref[core]):
                    wrong.append((seed, i))
                try:
                    gb.density(hc, bad, m["n_occ"], 1e-5, core_size=core)
                    wrong.append("accepted NaN")
                except gb.GbError:
                    pass
                if seed == 0 and i == 3:
                    gb.trim()

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
