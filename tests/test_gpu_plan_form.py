"""A plan installed by hand runs as given, one launch per bucket, also with the
codes that are reported for the built-in plan; a plan file keeps which of the
two a plan is.

With FP64 iterations the two differ in the waves of a cell, hence in the order
of its sums: the same bits as another plan of the same codes show that those ran,
other bits than the built-in plan's that its launches did not.  (In 1V with
sixteen slots both give a cell the same waves.)"""
import numpy as np
import pytest

from gpu_util import host, to_gpu
from paper_2007_12273_amd import synth

pytestmark = pytest.mark.gpu

KEYS = ("omega", "mu", "sigma", "L_pen")


def _same(a, b):
    return all(np.array_equal(a[k], b[k], equal_nan=True) for k in KEYS)


@pytest.mark.parametrize("D,kmax", [(3, 8), (1, 8), (3, 16)])
def test_reported_codes_installed_by_hand_run_as_given(D, kmax, tmp_path):
    from paper_2007_12273_amd import api
    sizes = (100, 200, 400, 900, 1300, 2000)
    d = synth.concat_cells([synth.random_cells(60 + n, 1, D, n, n, k_hi=3) for n in sizes])
    v, a, off = to_gpu(d)
    run = lambda: host(api.compress(v, a, off, kmax, seed=4, max_sweeps=30, fp64=True))
    path = tmp_path / "plans.txt"
    try:
        api.autotune_reset()
        built_in = run()
        codes = api.autotune_get(D, kmax, fp64=True)["variant"]
        api.autotune_set(D, kmax, codes, [(b + 1) % 12 for b in range(12)], fp64=True)
        moved = run()
        assert not _same(moved, built_in)
        api.autotune_set(D, kmax, codes, fp64=True)
        assert _same(run(), moved)
        api.autotune_save(path)
        line = path.read_text().split()
        assert line[-1] == "buckets"
        api.autotune_reset()
        assert _same(run(), built_in)
        assert api.autotune_load(path) == 1
        assert _same(run(), moved)
        # the built-in plan kept by the tuner, with and without the last word
        for words in (line[:-1] + ["builtin"], line[:-1]):
            path.write_text(" ".join(words) + "\n")
            api.autotune_reset()
            assert api.autotune_load(path) == 1 and api.autotune_get(D, kmax, fp64=True)["tuned"]
            assert _same(run(), built_in)
        path.write_text(" ".join(line[:-1] + ["elsewhere"]) + "\n")
        with pytest.raises(RuntimeError):
            api.autotune_load(path)
    finally:
        api.autotune_reset()


def test_a_tuned_plan_that_keeps_the_built_in_one_is_saved_as_such(tmp_path):
    from paper_2007_12273_amd import api
    d = synth.concat_cells([synth.random_cells(90 + n, 1, 3, n, n, k_hi=3) for n in (150, 300, 900)])
    v, a, off = to_gpu(d)
    c = api.Compressor(3, 3, 8, seed=4, fp64=True, max_sweeps=30)
    path = tmp_path / "plans.txt"
    try:
        api.autotune_reset()
        default = api.autotune_get(3, 8, fp64=True)
        c.autotune(v, a, off)
        tuned = host(c(v, a, off).as_dict())
        kept = dict(api.autotune_get(3, 8, fp64=True), tuned=False) == default
        api.autotune_save(path)
        assert path.read_text().split()[-1] == ("builtin" if kept else "buckets")
        api.autotune_reset()
        assert api.autotune_load(path) == 1
        assert _same(host(c(v, a, off).as_dict()), tuned)
    finally:
        api.autotune_reset()
