"""The work a program does with this library, as cases that can be timed.

Sizes are those of the repository's own workloads (`synth.py`, `bench.py`,
the tests) and of the paper's runs they stand for.  Every input is made on
the GPU from a seed, with the recipes of `synth.py`: per cell a few
Maxwellians, log-normal or Poisson particle counts.

Kinds of work:
  compress     the checkpoint: gm_compress to convergence, cold start
  warm         the checkpoint from the learned start (gm_compress_warm)
  reconstruct  the restart's sampling and projection (gm_reconstruct[_tensor])
  chain        the whole restart: sampling, Gauss'-law correction towards
               the deposit before the checkpoint, projection
  train        one epoch of the warm start's training, and the parameters
"""
import math

import numpy as np
import torch

from paper_2007_12273_amd import api

DEV = "cuda"


def listed():
    def compress(name, D, kmax, cells, counts, mean, **kw):
        return dict(name=name, kind="compress", D=D, kmax=kmax, cells=cells, counts=counts, mean=mean, k_hi=4,
                    weighted=True, aniso=False, fp64=False) | kw

    return [
        # the paper's two-stream restart (32 cells, 156 particles per cell):
        # the smallest call, where launches and latency count
        compress("two_stream_small", 1, 8, 32, "fixed", 156, k_hi=2, weighted=False),
        # the two-stream workload of the benchmark: FP64 iterations
        compress("two_stream_fp64", 1, 8, 32, "fixed", 1000, k_hi=2, weighted=False, fp64=True),
        # the paper's 16 x 16 cell Weibel run at 512 particles per cell
        compress("weibel_16x16", 3, 8, 256, "fixed", 512, k_hi=3, aniso=True, weighted=False),
        # 3V with FP64 iterations: the mode a user takes to get the FP64
        # oracle's decisions, at the grid's ragged counts
        compress("cells_3v_fp64", 3, 8, 512, "lognormal", 256, fp64=True),
        # the 1V mixture workload: slowly converging cells of about 2000
        compress("mix_1v", 1, 8, 1024, "poisson", 2000),
        # the benchmark's headline batch from a cold start
        compress("weibel_cold", 3, 16, 4096, "lognormal", 1000, k_hi=6, aniso=True, weighted=False),
        # the same batch from the learned start
        dict(name="weibel_warm", kind="warm", D=3, kmax=16, cells=4096, counts="lognormal", mean=1000, k_hi=6,
             weighted=False, aniso=True),
        # one GPU's share of a large 2D3V run: many small cells
        compress("grid_cold", 3, 8, 65536, "lognormal", 256),
        # its restart: sampling and the scalar projection, 2D positions
        dict(name="reconstruct_grid", kind="reconstruct", D=3, kmax=8, dx=2, cells=65536, counts="lognormal",
             mean=256, tensor=False),
        # the whole restart of the headline batch on its 1D mesh
        dict(name="chain_weibel", kind="chain", D=3, kmax=16, dx=1, cells=4096, nx=4096, counts="lognormal",
             mean=1000, tensor=True),
        # the whole restart of the 2D grid
        dict(name="chain_grid", kind="chain", D=3, kmax=8, dx=2, cells=65536, nx=256, counts="lognormal", mean=256,
             tensor=False),
        # one epoch of the warm start's training on one batch of cells
        dict(name="train_epoch", kind="train", rows=4096, batch=1024),
    ]


def draw(rng):
    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["compress", "compress", "compress", "warm", "reconstruct", "chain", "train"])
    counts = rng.choice(["fixed", "poisson", "lognormal"])
    if kind == "train":
        batch = logint(64, 1024)
        return dict(kind=kind, rows=logint(batch, 4096), batch=batch)
    if kind == "warm":
        mean = logint(100, 1000)
        return dict(kind=kind, D=3, kmax=rng.choice([8, 16, 13]), cells=logint(16, min(4096, 3000000 // mean)),
                    counts=counts, mean=mean, k_hi=rng.randint(2, 6), weighted=rng.random() < 0.5,
                    aniso=rng.random() < 0.5)
    if kind == "compress":
        D = rng.choice([1, 3])
        fp64 = rng.random() < 0.25
        kmax = rng.choice([8, 8, 5]) if fp64 or D == 1 else rng.choice([8, 16, 11])
        mean = logint(100, 2000) if D == 1 else logint(64, 512 if fp64 else 1000)
        most = 128 * 1024 if fp64 else 2000000 if D == 1 else 4000000 if kmax > 8 else 12000000
        return dict(kind=kind, D=D, kmax=kmax, cells=logint(16, min(49999, most // mean)), counts=counts, mean=mean,
                    k_hi=rng.randint(2, 4), weighted=rng.random() < 0.5, aniso=rng.random() < 0.5, fp64=fp64)
    D = rng.choice([1, 3, 3])
    dx = rng.choice([1, 2])
    mean = logint(100, 2000)
    most = 16000000 // mean
    if kind == "reconstruct":
        return dict(kind=kind, D=D, kmax=rng.choice([8, 16, 5]), dx=rng.choice([0, 1, 2, 3]), cells=logint(16, min(65000, most)),
                    counts=counts, mean=mean, tensor=rng.random() < 0.5)
    nx = logint(16, min(8192, most)) if dx == 1 else logint(4, int(math.sqrt(most)) if most < 60000 else 245)
    cells = nx if dx == 1 else nx * rng.randint(4, max(4, nx))
    return dict(kind=kind, D=D, kmax=rng.choice([8, 16]), dx=dx, cells=cells, nx=nx, counts=counts, mean=mean,
                tensor=rng.random() < 0.5)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _counts(case, rng):
    """Particles per cell, cells * mean in all (rescaled by largest remainder)."""
    n, mean = case["cells"], case["mean"]
    if case["counts"] == "fixed":
        return np.full(n, mean, dtype=np.int64)
    if case["counts"] == "poisson":
        c = np.maximum(50.0, rng.poisson(mean, size=n))
    else:
        c = np.clip(rng.lognormal(math.log(mean) - 0.125, 0.5, size=n), 50, 5000)
    c *= n * mean / c.sum()
    base = np.floor(c).astype(np.int64)
    base[np.argsort(base - c, kind="stable")[:n * mean - int(base.sum())]] += 1
    return base


def _mixtures(case, rng, k_hi, slots):
    """Random per-cell mixtures in `slots` padded slots (host arrays): 1 to
    k_hi Maxwellians, isotropic or T_perp = 4 T_par about a random axis."""
    n, D = case["cells"], case["D"]
    K = rng.integers(1, k_hi + 1, size=n)
    live = np.arange(slots)[None, :] < K[:, None]
    w = np.where(live, rng.dirichlet(np.ones(k_hi), size=n)[:, np.minimum(np.arange(slots), k_hi - 1)], 0.0)
    w /= w.sum(axis=1, keepdims=True)
    mu = rng.uniform(-0.5, 0.5, size=(n, slots, D))
    t = rng.uniform(0.02, 0.2, size=(n, slots)) ** 2
    cov = t[..., None, None] * np.eye(D)
    if case.get("aniso") and D == 3:
        b = rng.standard_normal(size=(n, slots, 3))
        b /= np.linalg.norm(b, axis=2, keepdims=True)
        cov = 4.0 * cov - 3.0 * t[..., None, None] * b[..., :, None] * b[..., None, :]
    if case.get("k_hi") == 2 and D == 1:  # the two-stream shape: beams at +-0.2, thermal speed 0.05
        K[:] = 2
        w[:] = 0.0
        w[:, :2] = 0.5
        mu[:, 0], mu[:, 1] = 0.2, -0.2
        cov[:] = 0.0025
    return K, w, mu, cov


def _gpu(x, dtype=None):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV, dtype)


def _offsets(counts):
    return np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)


def _particles(case, rng, seed):
    """v [n, D], alpha [n], cell_off drawn from per-cell mixtures."""
    counts = _counts(case, rng)
    K, w, mu, cov = _mixtures(case, rng, case["k_hi"], case["k_hi"])
    g = torch.Generator(device=DEV).manual_seed(seed)
    n, D, S = int(counts.sum()), case["D"], case["k_hi"]
    cell = torch.repeat_interleave(torch.arange(case["cells"], device=DEV), _gpu(counts), output_size=n)
    cum = np.cumsum(w, axis=1)
    u = torch.rand(n, generator=g, device=DEV, dtype=torch.float64)
    comp = torch.zeros(n, dtype=torch.int64, device=DEV)
    for k in range(S - 1):
        comp += u >= _gpu(cum[:, k])[cell]
    comp = torch.minimum(comp, _gpu(K - 1)[cell]) + cell * S
    z = torch.randn(n, D, generator=g, device=DEV, dtype=torch.float64)
    chol = _gpu(np.linalg.cholesky(cov)).reshape(-1, D, D)
    v = _gpu(mu).reshape(-1, D)[comp]
    for i in range(D):
        for j in range(i + 1):
            v[:, i] += chol[:, i, j][comp] * z[:, j]
    if case["weighted"]:
        alpha = 0.5 + torch.rand(n, generator=g, device=DEV, dtype=torch.float64)
    else:
        alpha = torch.ones(n, device=DEV, dtype=torch.float64)
    return v, alpha, _gpu(_offsets(counts))


def _record(case, rng):
    """A checkpoint record: per-cell mixtures (kmax slots), the moments they
    have with a mass of W per cell, and particle counts."""
    counts = _counts(case, rng)
    D, S = case["D"], case["kmax"]
    K, w, mu, cov = _mixtures(case, rng, min(4, S), S)
    W = counts * rng.uniform(0.95, 1.05, size=len(counts))
    tri = [(i, j) for i in range(D) for j in range(i, D)]
    second = cov + mu[..., :, None] * mu[..., None, :]
    mom = np.concatenate([np.ones((len(counts), 1)), np.einsum("ck,ckd->cd", w, mu)]
                         + [np.einsum("ck,ck->c", w, second[..., i, j])[:, None] for i, j in tri], axis=1) * W[:, None]
    live = (np.arange(S)[None, :] < K[:, None])
    sigma = np.stack([cov[..., i, j] for i, j in tri], axis=-1) * live[..., None]
    return dict(K=_gpu(K, torch.int32), omega=_gpu(w), mu=_gpu(mu * live[..., None]), sigma=_gpu(sigma),
                moments=_gpu(mom), off=_gpu(_offsets(counts)))


def _model_params(rng):
    """Perceptron parameters whose output is a usable start in every cell:
    biases that spread about six components over the whitened frame, weights
    that move them with the features."""
    P = {}
    for name, shape in api.PARAM_SHAPES:
        if name[0] == "W":
            fan = (105 if name == "W1" else shape[0]) + shape[1]
            P[name] = rng.uniform(-1, 1, size=shape) * math.sqrt(6.0 / fan)
            if name == "W1":
                P[name][105:] = 0.0
            if name == "W3":
                P[name] *= 0.15
        else:
            P[name] = np.zeros(shape)
    b = P["b3"].reshape(16, 10)
    b[:, 0] = -0.25 * np.arange(16)
    b[6:, 0] -= 6.0
    b[:, 1:4] = 0.8 * rng.standard_normal((16, 3))
    b[:, [4, 6, 9]] = math.log(0.6)
    return np.concatenate([P[n].reshape(-1) for n, _ in api.PARAM_SHAPES]).astype(np.float32)


def _training_rows(case, rng):
    """Features (three normalised 32-bin histograms and nine moments as BF16
    bits) and targets (1 to 6 whitened components, heaviest first)."""
    n = case["rows"]
    h = rng.dirichlet(np.exp(-0.5 * ((np.arange(32) - 15.5) / 6.0) ** 2) * 20, size=(n, 3)).reshape(n, 96)
    f = np.concatenate([h, 0.3 * rng.standard_normal((n, 9)), np.zeros((n, 23))], axis=1)
    t = np.zeros((n, 16, 10))
    K = rng.integers(1, 7, size=n)
    live = np.arange(16)[None, :] < K[:, None]
    w = np.where(live, rng.exponential(size=(n, 16)), 0.0)
    t[..., 0] = -np.sort(-w / w.sum(axis=1, keepdims=True), axis=1)
    t[..., 1:4] = 0.8 * rng.standard_normal((n, 16, 3))
    t[..., 4:] = 0.3 * rng.standard_normal((n, 16, 6))
    t[..., [4, 6, 9]] -= 0.5
    t *= live[..., None]
    feats = _gpu(f, torch.float32).to(torch.bfloat16).view(torch.int16)
    return feats, _gpu(t.reshape(n, 160), torch.float32)


def prepare(case, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    kind = case["kind"]
    if kind == "train":
        feats, targets = _training_rows(case, rng)
        return dict(kind=kind, model=api.WarmStart(16, batch=case["batch"], seed=seed, device=DEV), feats=feats,
                    targets=targets, seed=seed)
    if kind == "compress":
        v, a, off = _particles(case, rng, seed)
        call = api.Compressor(case["cells"], case["D"], case["kmax"], device=DEV, seed=seed, fp64=case["fp64"])
        return dict(kind=kind, call=call, v=v, a=a, off=off)
    if kind == "warm":
        v, a, off = _particles(case, rng, seed)
        model = api.WarmStart(case["kmax"], batch=64, device=DEV)
        model.set_params(_model_params(rng))
        call = api.WarmCompressor(case["cells"], model, device=DEV, seed=seed)
        return dict(kind=kind, call=call, model=model, v=v, a=a, off=off)
    rec = _record(case, rng)
    call = api.Reconstructor(rec["off"], case["D"], case["dx"], device=DEV,
                             projection="tensor" if case["tensor"] else "scalar")
    s = dict(kind=kind, call=call, rec=rec, seed=seed, tensor=case["tensor"])
    if kind == "chain":
        # the density before the checkpoint: the deposit of the original
        # particles (uniform positions, the cell's mass spread evenly)
        g = torch.Generator(device=DEV).manual_seed(seed)
        n = int(rec["off"][-1].item())
        x = torch.rand(n, case["dx"], generator=g, device=DEV, dtype=torch.float64)
        counts = rec["off"][1:] - rec["off"][:-1]
        w = torch.repeat_interleave(rec["moments"][:, 0] / counts, counts, output_size=n)
        s["target"] = _deposit(_columns(x, w, counts, case["dx"]), case)
        s["law"] = api.GaussLaw(case["cells"], case["dx"], case["nx"], device=DEV)
    return s


def run(s):
    if s["kind"] == "train":
        loss = s["model"].train(s["feats"], s["targets"], 1, lr=1e-3, lam=1.0, seed=s["seed"])
        return {"params": s["model"].get_params(), "loss": loss}
    if s["kind"] in ("compress", "warm"):
        return s["call"](s["v"], s["a"], s["off"]).as_dict()
    r = s["rec"]
    out = s["call"](r["K"], r["omega"], r["mu"], r["sigma"], r["moments"], s["seed"])
    if s["kind"] == "reconstruct":
        return {k: t for k, t in out.items() if t is not None}
    s["law"].correct(out["x"], out["w"], r["off"], s["target"])
    v, status = api.project(out["v"], out["w"], r["off"], r["moments"], tensor=s["tensor"], out=out["v"])
    return {"v": v, "w": out["w"], "x": out["x"], "status": status}


def work(case):
    """Bytes: inputs read once, outputs written once.  Flops of the EM: 49
    (3V) or 18 (1V) per particle and component update, with the updates per
    cell that these recipes take on average (measured, rounded)."""
    if case["kind"] == "train":
        steps = case["rows"] // case["batch"]
        per_row = 2 * (128 * 256 + 256 * 256 + 256 * 160)
        params = 128 * 256 + 256 + 256 * 256 + 256 + 256 * 160 + 160
        return {"bytes": case["rows"] * (128 * 2 + 160 * 4) + steps * params * 4 * 7,
                "flops": 3 * per_row * steps * case["batch"]}
    D, kmax, cells = case["D"], case["kmax"], case["cells"]
    n = cells * case["mean"]
    tri = D * (D + 1) // 2
    record = cells * (kmax * (1 + D + tri) + (1 + D + tri)) * 8
    if case["kind"] in ("compress", "warm"):
        updates = 200 if case["kind"] == "warm" else 1500 if D == 1 or kmax > 8 else 500
        return {"bytes": n * (D + 1) * 8 + cells * 8 + record, "flops": n * updates * (49 if D == 3 else 18)}
    out = n * (D + 1 + case["dx"]) * 8
    if case["kind"] == "reconstruct":
        return {"bytes": record + out, "flops": n * 250}
    # the sample written, positions and weights read and weights written by
    # the correction, weights and velocities read and velocities written by
    # the projection
    return {"bytes": record + out + n * (case["dx"] + 2) * 8 + n * (2 * D + 1) * 8, "flops": n * 350}


# ---------------------------------------------------------------------------
# 64-bit values of the outputs, without the library
# ---------------------------------------------------------------------------
def _segment(x, counts):
    return torch.segment_reduce(x, "sum", lengths=counts, axis=0)


def _spline(s):
    s = s.abs()
    return torch.where(s <= 0.5, 0.75 - s * s, torch.where(s <= 1.5, 0.5 * (1.5 - s) ** 2, torch.zeros_like(s)))


def _columns(x, w, counts, dx):
    """Per cell the weighted spline sums on its 3 (1D) or 9 (2D) mesh cells."""
    cols = []
    for oy in ((-1, 0, 1) if dx == 2 else (None,)):
        for ox in (-1, 0, 1):
            s = _spline(ox + 0.5 - x[:, 0])
            if oy is not None:
                s = s * _spline(oy + 0.5 - x[:, 1])
            cols.append(_segment(w * s, counts))
    return torch.stack(cols, 1)


def _deposit(cols, case, a=None):
    """sum over the cells j near i of cols[j, o(i, j)] * a[j], periodic."""
    if a is not None:
        cols = cols * a[:, None]
    if case["dx"] == 1:
        return sum(torch.roll(cols[:, o], o - 1) for o in range(3))
    g = cols.reshape(-1, case["nx"], 9)
    return sum(torch.roll(g[..., 3 * oy + ox], (oy - 1, ox - 1), (0, 1)) for oy in range(3)
               for ox in range(3)).reshape(-1)


def _mulhilo(a, b_hi, b_lo, b):
    """High and low words of the unsigned 64-bit product (int64 tensors)."""
    m = 0xFFFFFFFF
    a_lo, a_hi = a & m, (a >> 32) & m
    t = a_lo * b_lo
    u = a_hi * b_lo + ((t >> 32) & m)
    v = a_lo * b_hi + (u & m)
    return a_hi * b_hi + ((u >> 32) & m) + ((v >> 32) & m), a * b


def _signed(x):
    x &= (1 << 64) - 1
    return x - (1 << 64) if x >> 63 else x


def _philox(c, key):
    """Philox4x64-10 (Salmon et al., SC'11) on int64 tensors c[0..3]."""
    M = (0xD2E7470EE14C6C93, 0xCA5A826395121157)
    k = list(key)
    for _ in range(10):
        h0, l0 = _mulhilo(c[0], M[0] >> 32, M[0] & 0xFFFFFFFF, _signed(M[0]))
        h1, l1 = _mulhilo(c[2], M[1] >> 32, M[1] & 0xFFFFFFFF, _signed(M[1]))
        c = [h1 ^ c[1] ^ _signed(k[0]), l1, h0 ^ c[3] ^ _signed(k[1]), l0]
        k = [k[0] + 0x9E3779B97F4A7C15, k[1] + 0xBB67AE8584CAA73B]
    return c


def _project(v, w, counts, cell, mom, tensor):
    D = v.shape[1]
    tri = [(i, j) for i in range(D) for j in range(i, D)]
    N = _segment(w, counts)
    p = torch.stack([_segment(w * v[:, d], counts) for d in range(D)], 1)
    P = mom[:, 1:1 + D]
    if tensor:
        def full(m):
            out = torch.zeros(m.shape[0], D, D, dtype=torch.float64, device=DEV)
            for q, (i, j) in enumerate(tri):
                out[:, i, j] = out[:, j, i] = m[:, q]
            return out

        S = full(mom[:, 1 + D:])
        Sp = full(torch.stack([_segment(w * v[:, i] * v[:, j], counts) for i, j in tri], 1))
        Ct = S - P[:, :, None] * P[:, None, :] / N[:, None, None]
        Cs = Sp - p[:, :, None] * p[:, None, :] / N[:, None, None]
        Lt, it = torch.linalg.cholesky_ex(Ct)
        Ls, js = torch.linalg.cholesky_ex(Cs)
        ref_t = S.diagonal(dim1=1, dim2=2).mean(1, keepdim=True)
        ref_s = Sp.diagonal(dim1=1, dim2=2).mean(1, keepdim=True)
        ok = (it == 0) & (js == 0)
        ok &= (Lt.diagonal(dim1=1, dim2=2) ** 2 > 1e-12 * ref_t).all(1)
        ok &= (Ls.diagonal(dim1=1, dim2=2) ** 2 > 1e-12 * ref_s).all(1)
        eye = torch.eye(D, dtype=torch.float64, device=DEV)
        inv = torch.linalg.solve_triangular(torch.where(ok[:, None, None], Ls, eye), eye.expand_as(Ls), upper=False)
        A = (Lt[:, :, :, None] * inv[:, None, :, :]).sum(2)
        dv = v - (p / N[:, None])[cell]
        img = (P / N[:, None])[cell] + torch.stack([sum(A[:, i, j][cell] * dv[:, j] for j in range(D))
                                                    for i in range(D)], 1)
    else:
        E = 0.5 * sum(mom[:, 1 + D + q] for q, (i, j) in enumerate(tri) if i == j)
        Ep = _segment(0.5 * w * (v * v).sum(1), counts)
        num, den = 2 * E * N - (P * P).sum(1), 2 * Ep * N - (p * p).sum(1)
        ok = (num > 1e-12 * 2 * E * N) & (den > 1e-12 * 2 * Ep * N)
        a = torch.sqrt(torch.where(ok, num / den, torch.ones_like(num)))
        beta = (P - a[:, None] * p) / (a * N)[:, None]
        img = a[cell][:, None] * (v + beta[cell])
    return torch.where(ok[cell][:, None], img, v)


def _exact_restart(case, seed):
    s = prepare(case, seed)
    r, D, dx = s["rec"], case["D"], case["dx"]
    counts = r["off"][1:] - r["off"][:-1]
    n = int(r["off"][-1].item())
    cell = torch.repeat_interleave(torch.arange(case["cells"], device=DEV), counts, output_size=n)
    i = torch.arange(n, device=DEV) - r["off"][:-1][cell]
    zero = torch.zeros_like(i)
    u = []
    for b in range(2):
        u += [((x >> 11) & ((1 << 53) - 1)).to(torch.float64) * 2.0 ** -53
              for x in _philox([i, cell, zero + b, zero], (seed, 0x5245434F))]
    cum = torch.cumsum(r["omega"], 1)
    comp = torch.zeros_like(cell)
    for k in range(case["kmax"] - 1):
        comp += (u[0] >= cum[:, k][cell]) & (k < (r["K"] - 1)[cell])
    slot = cell * case["kmax"] + comp
    z = []
    for q in range((D + 1) // 2):
        rad = torch.sqrt(-2.0 * torch.log(1.0 - u[1 + 2 * q]))
        ang = 2.0 * math.pi * u[2 + 2 * q]
        z += [rad * torch.cos(ang), rad * torch.sin(ang)]
    tri = [(a, b) for a in range(D) for b in range(a, D)]
    cov = torch.zeros(case["cells"] * case["kmax"], D, D, dtype=torch.float64, device=DEV)
    for q, (a, b) in enumerate(tri):
        cov[:, a, b] = cov[:, b, a] = r["sigma"].reshape(-1, len(tri))[:, q]
    L, _ = torch.linalg.cholesky_ex(cov)
    v = r["mu"].reshape(-1, D)[slot]
    v = torch.stack([v[:, a] + sum(L[:, a, b][slot] * z[b] for b in range(a + 1)) for a in range(D)], 1)
    w = (r["moments"][:, 0] / counts)[cell]
    first = 1 + 2 * ((D + 1) // 2)
    x = torch.stack(u[first:first + dx], 1) if dx else None
    v = _project(v, w, counts, cell, r["moments"], case["tensor"])
    if case["kind"] == "chain":
        M = _columns(x, torch.ones_like(w), counts, dx)
        b = s["target"] - _deposit(_columns(x, w, counts, dx), case)
        dA = torch.zeros_like(b)
        for _ in range(3):  # refined twice
            dA = dA + _solve(M, b - _deposit(M, case, dA), case)
        w = w + dA[cell]
        v = _project(v, w, counts, cell, r["moments"], case["tensor"])
    out = {"v": v, "w": w, "x": x, "status": None}
    return {k: t for k, t in out.items() if not (k == "x" and t is None)}


def _solve(M, b, case):
    """BiCGSTAB with the diagonal on the right, to the rounding of the residual."""
    dinv = 1.0 / M[:, 1 if case["dx"] == 1 else 4]
    x, r = torch.zeros_like(b), b.clone()
    rh, p, v = r.clone(), torch.zeros_like(b), torch.zeros_like(b)
    rho, al, om = 1.0, 1.0, 1.0
    b2 = float(b @ b)
    for _ in range(300):
        rho1 = float(rh @ r)
        if float(r @ r) <= 1e-29 * b2 or rho1 == 0.0:
            break
        p = r + (rho1 / rho) * (al / om) * (p - om * v)
        v = _deposit(M, case, dinv * p)
        al, rho = rho1 / float(rh @ v), rho1
        sv = r - al * v
        t = _deposit(M, case, dinv * sv)
        tt = float(t @ t)
        om = float(t @ sv) / tt if tt > 0 else 0.0
        x = x + dinv * (al * p + om * sv)
        r = sv - om * t
        if om == 0.0:
            break
    return x


def _exact_train(case, seed):
    s = prepare(case, seed)
    flat = torch.from_numpy(s["model"].get_params()).to(DEV, torch.float64)
    X = s["feats"].view(torch.bfloat16).to(torch.float64)
    T = s["targets"].to(torch.float64).reshape(-1, 16, 10)
    perm = _shuffle(case["rows"], seed)
    P, o = [], 0
    for _, shape in api.PARAM_SHAPES:
        k = int(np.prod(shape))
        P.append(flat[o:o + k].reshape(shape).clone().requires_grad_())
        o += k
    opt = torch.optim.Adam(P, lr=1e-3, eps=1e-8)
    B, total = case["batch"], 0.0
    steps = case["rows"] // B
    for k in range(steps):
        rows = torch.from_numpy(perm[k * B:(k + 1) * B]).to(DEV)
        h = torch.relu(X[rows] @ P[0] + P[1])
        h = torch.relu(h @ P[2] + P[3])
        y = (h @ P[4] + P[5]).reshape(B, 16, 10)
        t = T[rows]
        wt = t[..., 0]
        d = y[..., 1:] - t[..., 1:]
        loss = -(wt * torch.log_softmax(y[..., 0], 1)).sum() + (wt * (d * d).sum(2)).sum()
        opt.zero_grad()
        (loss / B).backward()
        opt.step()
        total += float(loss)
    return {"params": torch.cat([p.detach().reshape(-1) for p in P]), "loss": [total / (steps * B)]}


def _shuffle(n, seed):
    """The first epoch's permutation: Fisher-Yates from the top index down,
    driven by splitmix64."""
    m = (1 << 64) - 1
    perm = list(range(n))
    x = (seed ^ 0xD1B54A32D192ED03) & m
    for i in range(n - 1, 0, -1):
        x = (x + 0x9E3779B97F4A7C15) & m
        z = x
        z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & m
        z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & m
        z ^= z >> 31
        j = (z * (i + 1)) >> 64
        perm[i], perm[j] = perm[j], perm[i]
    return np.array(perm, dtype=np.int64)


def exact(case, seed):
    """Of a converged fit only the moments have a 64-bit value that does not
    depend on the iteration's path."""
    if case["kind"] == "train":
        return _exact_train(case, seed)
    if case["kind"] in ("reconstruct", "chain"):
        return _exact_restart(case, seed)
    s = prepare(case, seed)
    v, a, counts, D = s["v"], s["a"], s["off"][1:] - s["off"][:-1], case["D"]
    cols = [a] + [a * v[:, d] for d in range(D)] + [a * v[:, i] * v[:, j] for i in range(D) for j in range(i, D)]
    out = dict.fromkeys(("K", "omega", "mu", "sigma", "L_pen", "L_final", "sweeps", "status", "visits"))
    out["moments"] = torch.stack([_segment(c, counts) for c in cols], 1)
    return out
