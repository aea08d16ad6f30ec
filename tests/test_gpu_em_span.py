"""The built-in EM plan runs in a few launches that walk several length
buckets, each cell with the fewest particles per thread that hold it; the
same variants installed by hand run one launch per bucket with the bucket's
particles per thread.  Padding particles add nothing and both forms round
alike, so the records are bit-identical: at both sides of every bucket limit
and of every step of particles per thread, cold and from a supplied start."""
import numpy as np
import pytest
import torch

from gpu_util import host, to_gpu
from paper_2007_12273_amd import synth

pytestmark = pytest.mark.gpu

EDGES8 = [11, 63, 64, 65, 128, 129, 192, 193, 256, 257, 320, 321, 384, 448, 449, 512, 513, 640, 641, 768, 769, 1024,
          1025, 1152, 1153, 1536, 1537, 1792, 1793, 2048, 2049, 2240, 2241, 2560, 2561, 3072, 3073, 3584, 3585, 4096,
          4097]
EDGES16 = [11, 64, 65, 128, 129, 192, 193, 256, 257, 384, 385, 512, 513, 576, 577, 768, 769, 1024, 1025, 1280, 1281,
           1536, 1537, 1792, 1793, 2048, 2049, 2560, 2561, 3072, 3073, 3584, 3585, 4096, 4097]

# largest cells of the buckets up to 2048 particles
LIMITS8 = [64, 128, 256, 512, 1024, 1536, 2048]
LIMITS16 = [128, 256, 512, 768, 1024, 1280, 1536, 1792, 2048]


@pytest.mark.parametrize("D,kmax,fp64,start", [(3, 8, False, False), (3, 16, False, False), (3, 16, False, True),
                                               (1, 8, False, False), (1, 16, False, False), (3, 8, True, False),
                                               (1, 8, True, True), (3, 11, True, False)])
def test_builtin_launches_equal_one_launch_per_bucket(D, kmax, fp64, start):
    from paper_2007_12273_amd import api
    sizes = EDGES8 if kmax <= 8 else EDGES16
    d = synth.concat_cells([synth.random_cells(700 + i, 1, D, n, n, k_hi=3) for i, n in enumerate(sizes)])
    v, a, off = to_gpu(dict(d, D=D))
    init = None
    if start:
        r = api.compress(v, a, off, kmax, seed=5, max_sweeps=3)
        init = {k: r[k] for k in ("K", "omega", "mu", "sigma")}
    kw = dict(seed=9, max_sweeps=25, fp64=fp64, init=init)
    try:
        api.autotune_reset()
        codes = list(api.autotune_get(D, kmax, fp64=fp64, warm=start)["variant"])
        if fp64:  # the built-in launches' particles per thread and waves
            for b, m in enumerate(LIMITS8 if kmax <= 8 else LIMITS16):
                P = min(m // 64, 2 if D == 3 and m <= 1024 else 4)
                codes[b] = 1000 * P + 10 * (8 if D == 3 and m > 1024 else -(-m // (64 * P))) + 1
        built_in = host(api.compress(v, a, off, kmax, **kw))
        api.autotune_set(D, kmax, codes, [(b + 1) % 12 for b in range(12)], fp64=fp64, warm=start)
        per_bucket = host(api.compress(v, a, off, kmax, **kw))
    finally:
        api.autotune_reset()
    torch.cuda.synchronize()
    for k in built_in:
        assert np.array_equal(built_in[k], per_bucket[k], equal_nan=True), k
    assert (built_in["K"] > 0).all()
