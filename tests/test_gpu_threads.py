"""Compress calls of several host threads on one GPU, each on a stream and a
workspace of its own: the library's streams and events are shared, the records
are those of the calls alone, bit for bit."""
import threading

import numpy as np
import pytest
import torch

from gpu_util import host, to_gpu
from paper_2007_12273_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("by_hand", [False, True])
def test_concurrent_calls_equal_the_calls_alone(by_hand):
    from paper_2007_12273_amd import api
    n_threads, calls = 4, 12
    try:
        api.autotune_reset()
        if by_hand:  # one launch per bucket on the library's streams
            api.autotune_set(3, 8, api.autotune_get(3, 8)["variant"])
        work = []
        for i in range(n_threads):
            d = synth.random_cells(500 + i, 24 + 40 * i, 3, 60, 1500, k_hi=3)
            v, a, off = to_gpu(d)
            c = api.Compressor(len(d["cell_off"]) - 1, 3, 8, seed=i, max_sweeps=20)
            ref = {k: x.copy() for k, x in host(c(v, a, off).as_dict()).items()}
            work.append((c, v, a, off, ref, torch.cuda.Stream()))
        torch.cuda.synchronize()
        gate = threading.Barrier(n_threads)
        wrong = []

        def run(i):
            c, v, a, off, ref, stream = work[i]
            gate.wait()
            for _ in range(calls):
                with torch.cuda.stream(stream):
                    out = c(v, a, off, stream=stream).as_dict()
                    stream.synchronize()
                    got = {k: x.cpu().numpy() for k, x in out.items()}
                wrong.extend((i, k) for k in ref if not np.array_equal(got[k], ref[k], equal_nan=True))

        ts = [threading.Thread(target=run, args=(i,)) for i in range(n_threads)]
        for t in ts:
            t.start()
        for t in ts:
            t.join()
        assert not wrong, wrong
    finally:
        api.autotune_reset()
