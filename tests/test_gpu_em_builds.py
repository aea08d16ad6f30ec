"""Builds of the FP32 EM launches chosen by cell or batch size.

Recomputing launches of more than eight waves take the fewest particles per
thread that hold the cell: both sides of every step (1024 particles in these
launches), as replays of the oracle's sweeps with the FP32 bars.

A 3V batch with eight slots and more cells than two waves per SIMD hold runs
the three-wave build: bit for bit the records of one launch per bucket."""
import numpy as np
import pytest
import torch

import fp32_parity
import oracle
from gpu_util import host, to_gpu
from paper_2007_12273_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,sizes", [(3, (4097, 5120, 5121, 6144, 6145, 7168, 7169, 8192)),
                                     (1, (2049, 2560, 2561, 3072, 3073, 4096, 4097, 8192))])
def test_recomputing_launches_at_every_particle_count(D, sizes):
    from paper_2007_12273_amd import api
    d = synth.concat_cells([synth.random_cells(900 + i, 1, D, n, n, k_hi=3) for i, n in enumerate(sizes)])
    o = oracle.compress(d["v"], d["alpha"], d["cell_off"], kmax=16, seed=21, max_sweeps=40)
    v, a, off = to_gpu(d)
    g = host(api.compress(v, a, off, 16, seed=21, max_sweeps=40,
                          fixed_sweeps=torch.from_numpy(o["sweeps"].astype(np.int32)).cuda()))
    assert np.array_equal(g["sweeps"], o["sweeps"])
    fp32_parity.check(g, o, d, fp32_parity.resolution(d, 16, 21, o["sweeps"], o), "recomputing launches D=%d" % D)


def test_three_wave_build_equals_one_launch_per_bucket():
    from paper_2007_12273_amd import api
    sizes = [11, 64, 65, 129, 193, 257, 321, 385, 449, 512, 513, 640, 769, 1025, 1537, 2049, 2561, 3073, 4096]
    one = synth.concat_cells([synth.random_cells(800 + i, 1, 3, n, n, k_hi=3) for i, n in enumerate(sizes)])
    reps = 2100 // len(sizes) + 1
    off = np.concatenate([[0], np.cumsum(np.tile(np.diff(one["cell_off"]), reps))]).astype(np.int64)
    d = dict(one, v=np.tile(one["v"], (reps, 1)), alpha=np.tile(one["alpha"], reps), cell_off=off)
    v, a, o = to_gpu(d)
    kw = dict(seed=3, max_sweeps=12)
    try:
        api.autotune_reset()
        codes = api.autotune_get(3, 8)["variant"]
        built_in = host(api.compress(v, a, o, 8, **kw))
        api.autotune_set(3, 8, codes, [(b + 1) % 12 for b in range(12)])
        per_bucket = host(api.compress(v, a, o, 8, **kw))
    finally:
        api.autotune_reset()
    for k in built_in:
        assert np.array_equal(built_in[k], per_bucket[k], equal_nan=True), k
    assert (built_in["K"] > 0).all()


@pytest.mark.parametrize("D,n_cells", [(3, 4097), (1, 5121)])
def test_plan_of_one_workgroup_and_of_many_fit_the_same_cells(D, n_cells):
    """4096 cells are planned by one workgroup, more by several: the common
    cells' records are equal bit for bit (cells of every bucket, empty ones
    and some too small to fit among them)."""
    from paper_2007_12273_amd import api
    rng = np.random.default_rng(4)
    counts = rng.integers(11, 80, size=n_cells)
    counts[::97] = 0
    counts[1::97] = 3
    for i, n in enumerate((300, 700, 1100, 1700, 2100, 2700, 3500, 4000, 5000, 9000)):
        counts[2 + 300 * i] = n
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    v = rng.normal(size=(off[-1], D))
    a = rng.uniform(0.5, 1.5, size=off[-1])
    kw = dict(seed=5, max_sweeps=6)
    vt, at, ot = to_gpu(dict(v=v, alpha=a, cell_off=off))
    many = host(api.compress(vt, at, ot, 8, **kw))
    vt, at, ot = to_gpu(dict(v=v[:off[4096]], alpha=a[:off[4096]], cell_off=off[:4097]))
    one = host(api.compress(vt, at, ot, 8, **kw))
    for k in one:
        assert np.array_equal(one[k], many[k][:4096], equal_nan=True), k
    assert (one["K"] > 0).sum() > 3900
