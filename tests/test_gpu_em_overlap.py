"""Cells of the built-in plan's 8-wave and 6-wave launches, and those of the
largest bucket and larger ones, are fitted side by side.  One cell of each, 400 replayed sweeps: fitted together they take the
longer one's time (one after the other, the sum), so the bar lies half of the
shorter one's time above the longer one's."""
import numpy as np
import pytest
import torch

from gpu_util import host, to_gpu
from paper_2007_12273_amd import synth

pytestmark = pytest.mark.gpu

SWEEPS = 400


@pytest.mark.parametrize("D,fp64,wide,narrow", [(3, False, 3500, 2500), (1, False, 4000, 3000), (1, True, 2000, 1400),
                                                   (3, False, 9000, 6000), (1, False, 9000, 6000)])
def test_cells_of_neighbouring_launches_overlap(D, fp64, wide, narrow):
    from paper_2007_12273_amd import api

    def em(sizes):
        d = synth.concat_cells([synth.random_cells(40 + n, 1, D, n, n, k_lo=3, k_hi=3) for n in sizes])
        v, a, off = to_gpu(d)
        c = api.Compressor(len(sizes), D, 8, seed=2, fp64=fp64)
        fs = torch.full((len(sizes),), SWEEPS, dtype=torch.int32, device=v.device)
        best, out = np.inf, None
        for _ in range(4):
            out = host(c(v, a, off, fixed_sweeps=fs).as_dict())
            best = min(best, api.profile_read()["em"])
        assert (out["sweeps"] == SWEEPS).all()
        return best, out

    api.profile_enable()
    try:
        tw, ow = em([wide])
        tn, on = em([narrow])
        both, ob = em([wide, narrow])
    finally:
        api.profile_enable(False)
    print("D=%d fp64=%d: %d particles %.2f ms, %d particles %.2f ms, together %.2f ms"
          % (D, fp64, wide, tw, narrow, tn, both))
    assert np.array_equal(ob["omega"][0], ow["omega"][0])
    assert both < max(tw, tn) + 0.5 * min(tw, tn)
