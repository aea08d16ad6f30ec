"""Which solver the Gauss'-law correction runs: the one-launch solve where the
mesh fits and the device has the CUs free, launch by launch elsewhere and
after a wait that gave up.

Bars: both paths solve to a true residual of 1e-13 |b|, and |M^-1| stays
below 4 with 4-12 particles per cell, so their weights are within 8e-13 |b| of
each other."""
import ctypes
import threading

import numpy as np
import pytest

from paper_2007_12273_amd import _lib

from gpu_util import dev, torch

pytestmark = pytest.mark.gpu


class Problem:
    def __init__(self, dx, nx, ny, seed=23):
        from paper_2007_12273_amd import api
        n = nx * ny
        rng = np.random.default_rng(seed)
        off = np.concatenate([[0], np.cumsum(rng.integers(4, 13, size=n))]).astype(np.int64)
        t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev())
        self.n, self.dx, self.nx = n, dx, nx
        self.off, self.x, self.w0 = t(off), t(rng.random((off[-1], dx))), t(rng.uniform(0.5, 1.5, off[-1]))
        self.law = api.GaussLaw(n, dx, nx, device=dev())
        self.target = self.law.deposit(t(rng.random((off[-1], dx))), self.w0, self.off).clone()
        self.b = float(torch.linalg.norm(self.target - self.law.deposit(self.x, self.w0, self.off)))

    def solve(self, wait_us=-1, places=-1, tol=1e-13, max_iter=400, stream=None):
        """(code, path, iterations, residual, weights)"""
        w = self.w0.clone()
        torch.cuda.synchronize()
        d = _lib.GmGaussDiag(wait_us, places, -1)
        it, res = ctypes.c_int32(0), ctypes.c_double(0.0)
        p = lambda a: ctypes.c_void_p(a.data_ptr())
        rc = _lib.load().gm_gauss_correct_diag(
            p(self.x), p(w), p(self.off), self.n, self.dx, self.nx, p(self.target), tol, max_iter, p(self.law.ws),
            self.law.ws.numel(), ctypes.c_void_p(stream.cuda_stream if stream is not None else 0), ctypes.byref(it),
            ctypes.byref(res), ctypes.byref(d))
        return rc, d.path, it.value, res.value, w


@pytest.mark.parametrize("dx,nx,ny,path", [
    (1, 1, 1, 1), (1, 2, 1, 1), (1, 1024, 1, 1), (1, 1025, 1, 1), (1, 131072, 1, 1), (1, 131073, 1, 0),
    (2, 1, 1025, 1), (2, 100, 21, 1), (2, 512, 2, 1), (2, 512, 3, 1), (2, 512, 256, 1), (2, 513, 3, 0),
    (2, 512, 257, 0)])
def test_path_of_every_mesh(dx, nx, ny, path):
    p = Problem(dx, nx, ny)
    rc, took, it, res, w = p.solve()
    print("dx=%d %d x %d: path %d, %d iterations, residual %.1e" % (dx, nx, ny, took, it, res))
    assert rc == 0 and took == path and res <= 1e-13
    rc, took, it, res, steps = p.solve(places=0)
    assert rc == 0 and took == 0 and res <= 1e-13
    assert float((w - steps).abs().max()) <= 8e-13 * p.b + 1e-14


def test_a_grid_without_its_places_is_solved_launch_by_launch():
    p = Problem(2, 512, 20)  # ten workgroups
    assert p.solve(places=10)[:2] == (0, 1)
    assert p.solve(places=9)[:2] == (0, 0)
    assert p.solve()[:2] == (0, 1)  # the places were given back


@pytest.mark.parametrize("dx,nx,ny", [(1, 1, 1), (1, 5000, 1), (2, 512, 256)])
def test_a_wait_that_gives_up_leaves_the_solve_to_the_other_path(dx, nx, ny):
    p = Problem(dx, nx, ny)
    ref = p.solve(places=0)
    rc, took, it, res, w = p.solve(wait_us=0)
    assert rc == 0 and took == 2 and res <= 1e-13
    assert torch.equal(w, ref[4]) and it == ref[2]
    assert p.solve()[:2] == (0, 1)  # the workspace holds no mark of it


@pytest.mark.parametrize("dx,nx,ny", [(1, 4096, 1), (2, 256, 256)])
def test_iterations_used_up_far_from_the_tolerance_are_not_run_twice(dx, nx, ny):
    """Three iterations: the one-launch solve's iterate is the answer.  Against
    the other path's: the same iterations with sums in another order, whose
    relative error stays below 65536 x 2^-53 = 7e-12 in each of their scalars;
    1e-9 leaves a factor for how three iterations carry it on."""
    p = Problem(dx, nx, ny)
    rc, path, it, res, w = p.solve(max_iter=3)
    assert (rc, path, it) == (_lib.GM_ENOCONV, 1, 3) and res > 1e-10
    rc, path, it, sres, steps = p.solve(max_iter=3, places=0)
    assert (rc, path, it) == (_lib.GM_ENOCONV, 0, 3) and abs(res - sres) <= 1e-9 * sres
    assert float((w - steps).abs().max()) <= 1e-9 * float((steps - p.w0).abs().max())


def test_iterations_used_up_near_the_tolerance_are_left_to_the_other_path():
    p = Problem(2, 256, 256)
    need = p.solve()[2]
    for max_iter in (need - 1, need):
        rc, path, it, res, w = p.solve(max_iter=max_iter)
        assert path == (2 if max_iter < need else 1) and it <= max_iter
        assert rc == (0 if res <= 1e-13 else _lib.GM_ENOCONV)


def test_solves_of_several_threads_share_the_places():
    """Six threads with 128 workgroups each: the device has places for two such
    grids at once, the others solve launch by launch (and a grid that the other
    streams' kernels keep out too long goes the same way); every result is
    right."""
    probs = [Problem(2, 512, 256, seed=30 + i) for i in range(6)]
    refs = [p.solve(places=0)[4] for p in probs]
    streams = [torch.cuda.Stream() for _ in probs]
    out = [None] * len(probs)
    gate = threading.Barrier(len(probs))

    def work(i):
        gate.wait()
        out[i] = [probs[i].solve(stream=streams[i]) for _ in range(3)]

    ts = [threading.Thread(target=work, args=(i,)) for i in range(len(probs))]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    torch.cuda.synchronize()
    print("paths:", [[r[1] for r in runs] for runs in out])
    for p, ref, runs in zip(probs, refs, out):
        for rc, path, it, res, w in runs:
            assert rc == 0 and path in (0, 1, 2) and res <= 1e-13, (rc, path, res)
            assert float((w - ref).abs().max()) <= 8e-13 * p.b + 1e-14
