"""The work this library does for its users, as cases that can be timed and compared.

Kinds of case, each through the public entry points of ``paper_2402_08515_amd.kf``:

* ``filter``   one application of the time-domain filter (``Problem.apply_filter``) to a block of b vectors that
               lies on the GPU: the unit of work of every Krylov step.  Meshes: the uniform unit square and cube
               (``grid``, dim and cells per axis n) and the unstructured horn (``horn``, n_c x n_c cells by n layers);
               float64 or float32 ("mixed") stepping; the second- or fourth-order scheme.
* ``batch``    ``Batch.apply_filter``: uneven squares and cubes whose time loops advance together.
* ``solve``    ``Problem.solve``: every distinct eigenvalue of an interval from one start vector.  Returned are the
               eigenvalues (their residuals are rounding noise far below the tolerance and are not).
* ``eig``      ``sym_eig``: the dense symmetric eigenproblem of the projected pencil, with the eigenvectors of a part
               of the spectrum.
* ``gradient``, ``weights``, ``train``  the filter-weight network: loss and gradient of a sample set, its weights for
               a sample set, and a training run (updated parameters and the loss of each epoch).
"""

import functools
import math

import numpy as np
import torch

from paper_2402_08515_amd import kf
from synth.grids import grid_problem
from synth.horn import horn_pencil


def listed():
    return [
        # one vector on the smallest workload square (3,969 rows): launches and latency
        dict(name="filter_square_64", kind="filter", mesh="grid", dim=2, n=64, b=1, precision="fp64", order=2,
             lo=10.0, hi=20.0, autotune=True),
        # the largest square of the uneven batch on its own, a block of 4 in float32 stepping
        dict(name="filter_square_256_block4", kind="filter", mesh="grid", dim=2, n=256, b=4, precision="mixed",
             order=2, lo=21.0, hi=33.5, autotune=True),
        # a middle cube with an odd number of vectors, the fourth-order scheme, default options
        dict(name="filter_cube_41_order4", kind="filter", mesh="grid", dim=3, n=41, b=3, precision="fp64", order=4,
             lo=12.0, hi=20.0, autotune=False),
        # one Krylov step's filter of the main benchmark (857,375 rows, float64)
        dict(name="filter_cube_96", kind="filter", mesh="grid", dim=3, n=96, b=1, precision="fp64", order=2,
             lo=30.0, hi=40.0, autotune=True),
        # the largest cube (2,048,383 rows) in float32 stepping
        dict(name="filter_cube_128_mixed", kind="filter", mesh="grid", dim=3, n=128, b=1, precision="mixed", order=2,
             lo=30.0, hi=40.0, autotune=True),
        # an unstructured mesh with a block of 16 in float32 stepping: the horn with 500 layers (144,789 rows)
        dict(name="filter_horn_block16", kind="filter", mesh="horn", dim=16, n=500, b=16, precision="mixed", order=2,
             lo=200.0, hi=220.0, autotune=True),
        # 16 uneven members in one batched application, block of 4
        dict(name="batch_16", kind="batch", members=16, draw=3, b=4, precision="mixed"),
        # a whole small solve: every eigenvalue of [10, 20] on the 64-cell square
        dict(name="solve_square_64", kind="solve", dim=2, n=64, lo=10.0, hi=20.0),
        # the main benchmark: all 110 distinct eigenvalues of [30, 40] on the 96-cell cube
        dict(name="solve_cube_96", kind="solve", dim=3, n=96, lo=30.0, hi=40.0),
        # the projected pencil at the size where the main benchmark converges
        dict(name="eig_440", kind="eig", k=440, part=0.25),
        # loss and gradient of the network on a validation set
        dict(name="net_gradient_1024", kind="gradient", samples=1024),
        # a short training run, batches of 256
        dict(name="net_train_5000", kind="train", samples=5000, epochs=1, batch=256),
    ]


def draw(rng):
    def log_int(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    kind = rng.choice(["filter"] * 6 + ["batch", "solve", "solve", "eig", "gradient", "weights", "train"])
    if kind == "filter":
        c = dict(kind="filter", b=rng.choice([1, 1, 1, 2, 3, 4, 7, 8, 16]), precision=rng.choice(["fp64", "mixed"]),
                 order=rng.choice([2, 2, 2, 4]), autotune=rng.choice([True, False]))
        mesh = rng.choice(["square", "square", "cube", "cube", "cube", "horn"])
        if mesh == "horn":
            lo = round(rng.uniform(200.0, 500.0), 2)
            return dict(c, mesh="horn", dim=rng.randint(5, 16), n=log_int(20, 200), lo=lo,
                        hi=round(lo + rng.uniform(20.0, 100.0), 2))
        dim, n = (2, log_int(17, 600)) if mesh == "square" else (3, log_int(9, 128 if c["b"] <= 4 else 64))
        lo = round(min(rng.uniform(5.0, 50.0), rng.uniform(0.1, 0.6) * 2.0 * n * math.sqrt(dim)), 2)
        return dict(c, mesh="grid", dim=dim, n=n, lo=lo, hi=round(lo + rng.uniform(0.1, 0.6) * lo + 1.0, 2))
    if kind == "batch":
        return dict(kind="batch", members=rng.randint(3, 16), draw=rng.randint(4, 10000), b=rng.choice([1, 2, 3, 4, 8]),
                    precision=rng.choice(["fp64", "mixed"]))
    if kind == "solve":
        if rng.random() < 0.5:
            lo, dim, n, width = rng.uniform(8.0, 14.0), 2, log_int(40, 160), rng.uniform(6.0, 10.0)
        else:
            lo, dim, n, width = rng.uniform(14.0, 20.0), 3, log_int(20, 64), rng.uniform(3.0, 6.0)
        return dict(kind="solve", dim=dim, n=n, lo=round(lo, 2), hi=round(lo + width, 2))
    if kind == "eig":
        return dict(kind="eig", k=log_int(20, 1000), part=round(rng.uniform(0.05, 0.4), 3))
    if kind == "gradient":
        return dict(kind="gradient", samples=64 * log_int(1, 64))
    if kind == "weights":
        return dict(kind="weights", samples=log_int(1, 5000))
    return dict(kind="train", samples=log_int(300, 8000), epochs=rng.randint(1, 3), batch=64 * rng.randint(1, 4))


# ------------------------------------------------------------------ meshes, time step, interval


@functools.lru_cache(maxsize=8)
def _pencil(mesh, dim, n):
    if mesh == "horn":
        return horn_pencil(dim, n, 0.05, 2)
    return grid_problem(dim, n)[:2]


@functools.lru_cache(maxsize=64)
def _lambda_max(mesh, dim, n):
    """The largest eigenvalue of the pencil: closed form on the grids, 30 power iterations on the horn."""
    if mesh == "grid":
        return dim * 4.0 * n * n * math.sin(0.5 * math.pi * (n - 1) / n) ** 2
    S, m = _pencil(mesh, dim, n)
    x = np.random.default_rng(1002).standard_normal(m.size)
    lam = 1.0
    for _ in range(30):
        x /= math.sqrt(x @ (m * x))
        y = (S @ x) / m
        lam = x @ (m * y)
        x = y
    return float(lam) * 1.02  # 30 iterations stay a little below the largest eigenvalue


def _steps(case):
    """tau and L of the method's rule: 90 % of the stability bound, L tau omega_min = 2 pi."""
    tau = 0.9 * 2.0 / math.sqrt(_lambda_max(case.get("mesh", "grid"), case["dim"], case["n"]))
    return tau, int(math.ceil(2.0 * math.pi / (case["lo"] * tau)))


def _axis(n):
    return 4.0 * n * n * np.sin(0.5 * math.pi * np.arange(1, n) / n) ** 2


def _distinct(case):
    """The distinct eigenvalues of a grid pencil in the case's interval."""
    a = _axis(case["n"])
    lam = a[:, None] + a[None, :]
    if case["dim"] == 3:
        lam = lam[:, :, None] + a
    lam = np.sort(lam[(lam >= case["lo"] ** 2) & (lam <= case["hi"] ** 2)])
    return lam[np.concatenate([[True], np.diff(lam) > 1e-10 * lam[1:]])] if lam.size else lam


def _members(case):
    """Uneven squares and cubes with their intervals, drawn as the batch workload draws them."""
    rng = np.random.default_rng(case["draw"])
    out = []
    for _ in range(case["members"]):
        dim = 2 if rng.random() < 0.5 else 3
        n = int(rng.integers(32, 257)) if dim == 2 else int(rng.integers(16, 65))
        lo = float(rng.uniform(5.0, 50.0))
        out.append(dict(mesh="grid", dim=dim, n=n, lo=lo, hi=lo + float(rng.uniform(5.0, 20.0)), order=2))
    return out


def _block(n, b, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    return torch.randn(n, b, generator=g, device="cuda", dtype=torch.float64)


# ------------------------------------------------------------------ the network's inputs


def _samples(count, rng):
    lam = np.exp(rng.uniform(math.log(5e4), math.log(3e5), size=count))
    lo = rng.uniform(5.0, 50.0, size=count)
    return np.stack([lo, lo + rng.uniform(5.0, 20.0, size=count), 1.8 / np.sqrt(lam), lam], axis=1)


def _parameters(rng):
    """He-initialised hidden layers, small biases and a small output layer, as after some training."""
    parts = []
    for rows, cols, scale in ((64, 128, math.sqrt(2 / 64)), (128, 128, math.sqrt(2 / 128)),
                              (128, 128, math.sqrt(2 / 128)), (128, 512, 0.02)):
        parts += [scale * rng.standard_normal(rows * cols), 0.01 * rng.standard_normal(cols)]
    return np.concatenate(parts).astype(np.float32)


def _net_inputs(case, seed):
    rng = np.random.default_rng(seed)
    params, samples = _parameters(rng), _samples(case["samples"], rng)
    order = np.concatenate([rng.permutation(case["samples"]) for _ in range(case.get("epochs", 1))]).astype(np.int32)
    return params, samples, order


def _pencil_matrix(case, seed):
    """A symmetric matrix with the spread-out spectrum of a projected pencil: eigenvalues omega^2 up to 1e5."""
    g = torch.Generator().manual_seed(int(seed))
    k = case["k"]
    om = 2.0 + (316.0 - 2.0) * (torch.arange(k, dtype=torch.float64) + 0.8 * torch.rand(k, generator=g, dtype=torch.float64)) / k
    q = torch.linalg.qr(torch.randn(k, k, generator=g, dtype=torch.float64))[0]
    a = (q * om.square()) @ q.T
    first = k // 10
    last = min(k - 1, first + max(1, int(case["part"] * k)))
    cut = lambda i: float((0.5 * (om[i] + om[i - 1])) ** 2)  # noqa: E731
    return (0.5 * (a + a.T)).numpy(), (cut(first) if first else 0.0), cut(last)


# ------------------------------------------------------------------ the contract


def prepare(case, seed):
    kind = case["kind"]
    if kind == "filter":
        S, m = _pencil(case["mesh"], case["dim"], case["n"])
        tau, L = _steps(case)
        p = kf.Problem(S, m, case["lo"], case["hi"], tau, L, precision=case["precision"], stepper=case["order"],
                       autotune=case["autotune"])
        return dict(kind=kind, p=p, x=_block(m.size, case["b"], seed))
    if kind == "batch":
        members, xs = [], []
        for i, c in enumerate(_members(case)):
            S, m = _pencil("grid", c["dim"], c["n"])
            tau, L = _steps(c)
            members.append((S, m, c["lo"], c["hi"], tau, L, 0))
            xs.append(_block(m.size, case["b"], 1000 * seed + i))
        return dict(kind=kind, p=kf.Batch(members, precision=case["precision"], autotune=True), x=xs)
    if kind == "solve":
        S, m = _pencil("grid", case["dim"], case["n"])
        tau, L = _steps(case)
        p = kf.Problem(S, m, case["lo"], case["hi"], tau, L, target=int(_distinct(case).size), check_every=2,
                       autotune=True)
        return dict(kind=kind, p=p, x=_block(m.size, 1, seed), m_max=min(1024, m.size))
    if kind == "eig":
        a, lo, hi = _pencil_matrix(case, seed)
        return dict(kind=kind, a=a, lo=lo, hi=hi)
    params, samples, order = _net_inputs(case, seed)
    return dict(kind=kind, net=kf.Mlp(params), samples=samples, order=order, epochs=case.get("epochs"),
                batch=case.get("batch"))


def run(state):
    kind = state["kind"]
    if kind in ("filter", "batch"):
        return state["p"].apply_filter(state["x"])
    if kind == "solve":
        r = state["p"].solve(state["x"], m_max=state["m_max"], tol=1e-6)
        return {"omega2": r.omega2, "omega": r.omega}
    if kind == "eig":
        theta, y = kf.sym_eig(state["a"], state["lo"], state["hi"], vectors=True)
        return {"theta": theta, "vectors": y}
    if kind == "gradient":
        loss, grad = state["net"].loss_grad(state["samples"])
        return {"loss": loss, "grad": grad}
    if kind == "weights":
        return state["net"].batch_weights(state["samples"])
    hist = state["net"].train(state["samples"], state["order"], state["epochs"], state["batch"], 1e-3)
    return {"loss": hist, "params": state["net"].params()}


def _filter_work(c, b, precision):
    S, m = _pencil(c["mesh"], c["dim"], c["n"])
    _, L = _steps(c)
    products = 2 if c["order"] == 4 else 1
    return (S.nnz * ((4 if precision == "mixed" else 8) + 4) + 16.0 * m.size * b,
            (L - 1.0) * b * (products * 2.0 * S.nnz + 4.0 * m.size))


def work(case):
    kind = case["kind"]
    if kind == "filter":
        bytes_, flops = _filter_work(case, case["b"], case["precision"])
    elif kind == "batch":
        bytes_, flops = (sum(v) for v in zip(*(_filter_work(c, case["b"], case["precision"]) for c in _members(case))))
    elif kind == "solve":
        # the Krylov space holds at least as many columns as there are eigenvalues: that many filter applications,
        # and every column once against every other
        k = _distinct(case).size
        bytes_, flops = _filter_work(dict(case, mesh="grid", order=2), 1, "fp64")
        rows = (case["n"] - 1.0) ** case["dim"]
        bytes_, flops = bytes_ + 8.0 * rows * k, flops * k + 2.0 * rows * k * k
    elif kind == "eig":
        k, nv = case["k"], max(1, int(case["part"] * case["k"]))
        bytes_, flops = 8.0 * k * (k + 1 + nv), 4.0 / 3.0 * k**3 + 2.0 * nv * k * k
    else:
        net, response, count = 64 * 128 + 2 * 128 * 128 + 128 * 512, 512 * 512, case["samples"]
        passes = 1 if kind == "weights" else 3
        steps = case["epochs"] * (count // case["batch"]) if kind == "train" else 1
        rows = steps * case["batch"] if kind == "train" else count
        flops = 2.0 * rows * (passes * net + (0 if kind == "weights" else 2 * response))
        bytes_ = 32.0 * count + 4.0 * net * (2 if kind != "weights" else 1) + (8.0 * 512 * count if kind == "weights" else 0)
    return {"bytes": float(bytes_), "flops": float(flops)}


# ------------------------------------------------------------------ the same results in 64 bits, plain torch


def _grid_operator(dim, n):
    """M^{-1} S of the uniform grid: the 5- or 7-point difference operator on the interior vertices."""
    k = n - 1

    def apply(y):
        v = y.reshape([k] * dim + [-1])
        out = 2.0 * dim * v
        for ax in range(dim):
            if k > 1:
                out.narrow(ax, 1, k - 1).sub_(v.narrow(ax, 0, k - 1))
                out.narrow(ax, 0, k - 1).sub_(v.narrow(ax, 1, k - 1))
        return (float(n) * n * out).reshape(y.shape)

    return apply


def _mesh_operator(S, m):
    """M^{-1} S of any pencil from its rows, padded to the longest one."""
    n, width = m.size, int(np.diff(S.indptr).max())
    rows = np.repeat(np.arange(n), np.diff(S.indptr))
    slot = np.arange(S.nnz) - S.indptr[:-1][rows]
    col, val = np.zeros((n, width), dtype=np.int64), np.zeros((n, width))
    col[rows, slot], val[rows, slot] = S.indices, S.data / m[rows]
    col, val = torch.from_numpy(col).cuda(), torch.from_numpy(val).cuda()

    def apply(y):
        out = torch.zeros_like(y)
        for q in range(width):
            out.addcmul_(val[:, q : q + 1], y[col[:, q]])
        return out

    return apply


def _exact_filter(c, x):
    tau, L = _steps(c)
    op = _mesh_operator(*_pencil("horn", c["dim"], c["n"])) if c["mesh"] == "horn" else _grid_operator(c["dim"], c["n"])
    t = np.arange(1, L) * tau
    w = np.empty(L)
    w[0] = tau * 2.0 * (c["hi"] - c["lo"]) / math.pi
    w[1:] = tau * 4.0 / (math.pi * t) * np.sin(0.5 * t * (c["hi"] - c["lo"])) * np.cos(0.5 * t * (c["hi"] + c["lo"]))
    before, now, total = x, x, w[0] * x
    for i in range(1, L):
        z = tau * tau * op(now)
        nxt = 2.0 * now - before - z
        if c["order"] == 4:
            nxt += tau * tau / 12.0 * op(z)
        before, now = now, nxt
        total = total + w[i] * now
    return total


def _net_tensors(flat):
    out, at = [], 0
    for shape in ((64, 128), (128,), (128, 128), (128,), (128, 128), (128,), (128, 512), (512,)):
        size = math.prod(shape)
        out.append(flat[at : at + size].reshape(shape))
        at += size
    return out


def _net_forward(flat, s):
    """The network's weights (rows x 512) and the mean leakage loss, float64."""
    W1, b1, W2, b2, W3, b3, W4, b4 = _net_tensors(flat)
    a, c, xm = s[:, 2:3] * s[:, 0:1], s[:, 2:3] * s[:, 1:2], 0.5 * s[:, 2:3] * s[:, 3:4].sqrt()
    L = torch.ceil(2.0 * math.pi / a).clamp(max=512.0)
    f = torch.zeros(s.shape[0], 64, dtype=s.dtype, device=s.device)
    f[:, :4] = torch.cat([a / math.pi, c / math.pi, xm, L / 512.0], 1)
    gelu = torch.nn.functional.gelu
    h = gelu(gelu(gelu(f @ W1 + b1) @ W2 + b2) @ W3 + b3)
    ell = torch.arange(512, dtype=s.dtype, device=s.device)[None, :]
    one = ell.clamp(min=1.0)
    wf = 4.0 / (math.pi * one) * torch.sin(0.5 * ell * (c - a)) * torch.cos(0.5 * ell * (c + a))
    wf = torch.where(ell == 0, 2.0 * (c - a) / math.pi, wf)
    w = torch.where(ell < L, wf + 0.01 * (h @ W4 + b4), torch.zeros_like(wf))
    x = 0.95 * torch.arange(512, dtype=s.dtype, device=s.device)[None, :] / 511.0
    phi = 2.0 * torch.asin(x)
    beta = w @ (torch.cos((ell.T + 0.5) * phi) / torch.cos(0.5 * phi))
    # the band's edges are compared in the 32 bits in which the library states them
    r = lambda v: v.float().double()  # noqa: E731
    lo, hi, d = r(0.5 * a), r(0.5 * c), r(math.pi / (2.0 * L))
    x = r(x)
    band = ((x >= lo) & (x <= hi)).double()
    off = ((x <= r(xm)) & ((x < r(lo - d)) | (x > r(hi + d)))).double()
    loss = (band * (beta - 1.0) ** 2).sum(1) / band.sum(1).clamp(min=1.0) + (off * beta**2).sum(1) / off.sum(1).clamp(min=1.0)
    return w, loss


def _exact_net(case, seed):
    params, samples, order = _net_inputs(case, seed)
    p = torch.from_numpy(params).cuda().double().requires_grad_(True)
    s = torch.from_numpy(samples).cuda()
    if case["kind"] == "weights":
        with torch.no_grad():
            return _net_forward(p, s)[0]
    if case["kind"] == "gradient":
        loss = _net_forward(p, s)[1].mean()
        loss.backward()
        return {"loss": float(loss.detach()), "grad": p.grad}
    n, batch, epochs = case["samples"], case["batch"], case["epochs"]
    steps, hist, t = n // batch, [], 0
    m1, m2 = torch.zeros_like(p.detach()), torch.zeros_like(p.detach())
    for e in range(epochs):
        total = 0.0
        for i in range(steps):
            p.grad = None
            rows = torch.from_numpy(order[e * n + i * batch : e * n + (i + 1) * batch].astype(np.int64)).cuda()
            loss = _net_forward(p, s[rows])[1]
            loss.mean().backward()
            total += float(loss.detach().sum())
            t += 1
            lr = 1e-3 * (0.01 + 0.99 * 0.5 * (1.0 + math.cos(math.pi * (e * steps + i) / max(1, epochs * steps - 1))))
            m1 = 0.9 * m1 + 0.1 * p.grad
            m2 = 0.999 * m2 + 0.001 * p.grad**2
            with torch.no_grad():
                p -= lr * (m1 / (1 - 0.9**t)) / ((m2 / (1 - 0.999**t)).sqrt() + 1e-8)
        hist.append(total / (steps * batch))
    return {"loss": np.array(hist), "params": p.detach()}


def exact(case, seed):
    kind = case["kind"]
    if kind == "filter":
        rows = _pencil(case["mesh"], case["dim"], case["n"])[1].size
        return _exact_filter(case, _block(rows, case["b"], seed))
    if kind == "batch":
        return [_exact_filter(c, _block((c["n"] - 1) ** c["dim"], case["b"], 1000 * seed + i))
                for i, c in enumerate(_members(case))]
    if kind == "solve":
        lam = _distinct(case)
        return {"omega2": lam, "omega": np.sqrt(lam)}
    if kind == "eig":
        # (an eigenvector's sign is the solver's choice)
        return {"theta": np.linalg.eigvalsh(_pencil_matrix(case, seed)[0]), "vectors": None}
    return _exact_net(case, seed)
