"""The work that users of this framework have it do, as cases to be timed.

Three kinds of case, each through the public Python entry points:

scan   one scan of a scanner that is already set up (its matrix packed by
       set_system, with the automatic schedule): hand the counts over
       (set_data), iterate, read the image and the objective.  What a
       reconstruction service does for every scan.
batch  many scans of uneven shapes, or one scan under many regularisation
       strengths, iterated together, and every image read.  A batch has no
       call that starts it again, so a repeated pass goes on from where the
       last one ended, as a study that is continued does.
net    the learned warm start: the start images of a batch of early images
       (mode "ratio" or "direct"), or the loss and gradient of one training
       batch.

Matrices follow the recipe of paper_1601_08201_amd/datagen.py (distinct
uniform rows per column, uniform values, phantoms of rectangles with Gaussian
spectra, Poisson counts), drawn on the GPU, but without its explicit zeros:
every stored entry is a nonzero.
"""
from __future__ import annotations

import concurrent.futures
import math

import numpy as np
import torch

from paper_1601_08201_amd import autotune, datagen, sgtv

DEV = "cuda"


# ---------------------------------------------------------------- the cases

def listed():
    return [
        # the smallest scan (the parity workload), counts and image in host memory: latency and launches
        scan("scan_16x16x32", 16, 16, 32, 4096, 16, iters=50, beta=0.1, host=True),
        # the grid, detector, pitches and mean count of the paper's experiment: odd sizes, direction weights
        scan("scan_9x41x54", 9, 41, 54, 8192, 24, iters=300, beta=0.5, pitch=True, mean=26.0),
        # the scanner of the learned warm start, an ordinary size: the plain run that makes a training target
        scan("scan_64x64x64", 64, 64, 64, 131072, 32, iters=300, beta=0.1),
        # a ragged grid with odd sizes, bfloat16 values, standard TV and two surrogate sweeps
        scan("scan_77x101x93_bf16", 77, 101, 93, 361647, 48, iters=60, beta=0.1, storage="bf16", grouping=1,
             sweeps=2, host=True),
        # the paper-scale scan of the benchmark, FP32 values: the largest
        scan("scan_128x128x128", 128, 128, 128, 1048576, 64, iters=200, beta=0.05),
        # the same grid with half the entries per column in binary16, as a batch's scans have them
        scan("scan_128x128x128_f16", 128, 128, 128, 1048576, 32, iters=100, beta=0.05, storage="f16"),
        # uneven scans in one batch (the benchmark's batch has 64 of them): a day's scans reconstructed together
        batch("batch_8_uneven", 8, 48, 96, 32, iters=50),
        # one experiment-sized scan under 8 strengths and both regularisers in one batch (study.sweep)
        sweep("sweep_16", 9, 41, 54, 8192, 24, 8, iters=200),
        # one early image to its start image: what a single reconstruction waits for
        net("net_start_1", "ratio", 6, 64, 1),
        # a batch of normalised backprojections to start images, with the start floor
        net("net_start_32", "direct", 6, 64, 32),
        # loss and gradient of one training batch: forward and backward of all layers
        net("net_gradient_32", "gradient", 6, 64, 32),
        # the same for a shorter image and a small odd batch, three layers
        net("net_gradient_7", "gradient", 3, 36, 7),
    ]


def scan(name, ny, nx, Q, I, nnz_per_col, iters, beta, pitch=False, mean=0.0, storage="f32", grouping=0, sweeps=1,
         host=False):
    return dict(name=name, kind="scan", ny=ny, nx=nx, Q=Q, I=I, nnz_per_col=nnz_per_col, iters=iters, beta=beta,
                pitch=pitch, mean=mean, storage=storage, grouping=grouping, sweeps=sweeps, host=host)


def batch(name, scans, low, high, nnz_per_col, iters):
    return dict(name=name, kind="batch", scans=scans, low=low, high=high, nnz_per_col=nnz_per_col, iters=iters)


def sweep(name, ny, nx, Q, I, nnz_per_col, betas, iters):
    return dict(name=name, kind="sweep", ny=ny, nx=nx, Q=Q, I=I, nnz_per_col=nnz_per_col, betas=betas, iters=iters)


def net(name, what, layers, height, batch):
    return dict(name=name, kind="net", what=what, layers=layers, height=height, batch=batch)


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed kinds and ranges."""
    kind = rng.choice(["scan", "scan", "scan", "scan", "batch", "sweep", "net", "net"])
    if kind == "scan":
        while True:
            ny, nx, Q = _log(rng, 9, 128), _log(rng, 16, 128), _log(rng, 24, 129)
            J = ny * nx * Q
            I = max(2048, int(J * math.exp(rng.uniform(math.log(0.4), math.log(1.0)))))
            per_col = _log(rng, 16, 64)
            if J * per_col <= 60_000_000:
                break
        c = scan("", ny, nx, Q, I, per_col, iters=_log(rng, 20, 200), beta=round(rng.uniform(0.05, 0.5), 3),
                 pitch=rng.random() < 0.3, mean=rng.choice([0.0, 26.0]), storage=rng.choice(["f32", "f32", "bf16", "f16"]),
                 grouping=rng.choice([0, 0, 1]), sweeps=rng.choice([1, 1, 2]), host=rng.random() < 0.5)
    elif kind == "batch":
        c = batch("", rng.randint(3, 10), rng.randint(20, 40), rng.randint(48, 80), rng.randint(24, 40),
                  iters=_log(rng, 20, 100))
    elif kind == "sweep":
        c = sweep("", rng.randint(8, 24), rng.randint(16, 48), rng.randint(32, 70), rng.randint(6000, 16000),
                  rng.randint(16, 32), rng.randint(2, 10), iters=_log(rng, 50, 300))
    else:
        c = net("", rng.choice(["ratio", "direct", "gradient", "gradient"]), rng.randint(2, 8), 2 * rng.randint(8, 48),
                _log(rng, 1, 32))
    del c["name"]
    return c


# ---------------------------------------------------------------- inputs

class Problem:
    """One scan: CSR matrix and counts on the GPU, scalars on the host."""


def _problem(ny, nx, Q, I, per_col, seed, mean=0.0, beta=0.1):
    p = Problem()
    p.ny, p.nx, p.Q, p.I, p.beta, p.rho = ny, nx, Q, I, beta, 1.0
    p.J = J = ny * nx * Q
    rng = np.random.Generator(np.random.PCG64(seed))
    gen = torch.Generator(device=DEV).manual_seed(seed)
    x = torch.from_numpy(datagen.make_phantom(rng, ny, nx, Q, int(rng.integers(4, 13)))).to(DEV)
    rows = torch.randint(0, I, (J, per_col), generator=gen, device=DEV, dtype=torch.int32)
    while True:   # the rows of a column are distinct
        rows = rows.sort(dim=1).values
        bad = (rows[:, 1:] == rows[:, :-1]).any(dim=1).nonzero()[:, 0]
        if bad.numel() == 0:
            break
        rows[bad] = torch.randint(0, I, (bad.numel(), per_col), generator=gen, device=DEV, dtype=torch.int32)
    key = rows.long().mul_(J).add_(torch.arange(J, device=DEV)[:, None]).view(-1)
    del rows
    key = key.sort().values                                     # by row, then column
    row = torch.div(key, J, rounding_mode="floor")
    p.col = (key - row * J).int()
    p.rowptr = torch.zeros(I + 1, dtype=torch.int64, device=DEV)
    p.rowptr[1:] = torch.bincount(row, minlength=I).cumsum(0)
    del key, row
    p.val = 1.0 - torch.rand(p.col.numel(), generator=gen, device=DEV)   # (0, 1]
    m = _product(p.rowptr, p.col, p.val, J, x.double())
    if mean:
        m *= (mean - 0.1) / max(float(m.mean()), 1e-30)
    m += float(np.float32(0.1))
    p.y = torch.poisson(m.float(), generator=gen)
    p.r = torch.full((I,), 0.1, device=DEV)
    return p


def _product(rowptr, col, val, n_cols, x):
    """A x in 64 bits, A in CSR."""
    A = torch.sparse_csr_tensor(rowptr, col.long(), val.double(), size=(rowptr.numel() - 1, n_cols))
    return A @ x


def _weights(case):
    return datagen.direction_weights(5.0, 1.5) if case.get("pitch") or case["kind"] == "sweep" else None


def _scan_problem(case, seed):
    return _problem(case["ny"], case["nx"], case["Q"], case["I"], case["nnz_per_col"], seed,
                    case["mean"], case["beta"])


def _batch_problems(case, seed):
    """Uneven shapes: sides and spectra between the case's bounds, half as many measurements as voxels."""
    rng = np.random.Generator(np.random.PCG64(12345))   # the scanners' shapes; what they hold comes from the seed
    out = []
    for k in range(case["scans"]):
        side, Q = int(rng.integers(case["low"], case["high"] + 1)), int(rng.integers(case["low"], case["high"] + 1))
        out.append(_problem(side, side, Q, side * side * Q // 2, case["nnz_per_col"], seed * 64 + k))
    return out


def _sweep_problem(case, seed):
    p = _problem(case["ny"], case["nx"], case["Q"], case["I"], case["nnz_per_col"], seed, mean=26.0)
    return p, [(g, float(b)) for g in (0, 1) for b in np.geomspace(0.02, 5.0, case["betas"])]


def _net_inputs(case, seed):
    """He-style parameters, and images as the reconstruction gives them: nonnegative, smooth in the spectrum, bright
    rectangles on a low background."""
    rng = np.random.Generator(np.random.PCG64(seed))
    params = sgtv.init_params(case["layers"], 64, seed)
    gen = torch.Generator(device=DEV).manual_seed(seed)
    shape = (case["batch"], case["height"], 64, 64)
    x = np.stack([datagen.make_phantom(rng, case["height"], 64, 64, 6).reshape(shape[1:]) for _ in range(shape[0])])
    x = torch.from_numpy(x).to(DEV)
    x = x * (0.5 + torch.rand(shape, generator=gen, device=DEV)) + 0.2
    target = x * (0.5 + torch.rand(shape, generator=gen, device=DEV))
    return params, x, target


# ---------------------------------------------------------------- a program's state and one pass

class State:
    pass


def _stream():
    return torch.cuda.current_stream().cuda_stream


def prepare(case, seed):
    s = State()
    s.case = case
    if case["kind"] == "scan":
        p = _scan_problem(case, seed)
        s.R = sgtv.Reconstructor(device=0, stream=_stream())
        s.R.set_system(p.I, p.ny, p.nx, p.Q, p.rowptr, p.col, p.val, storage=case["storage"],
                       w=_device(_weights(case)))
        s.R.set_grouping(case["grouping"])
        if case["host"]:
            s.y, s.r, s.image = p.y.cpu().numpy(), p.r.cpu().numpy(), np.empty(p.J, np.float32)
        else:
            s.y, s.r, s.image = p.y, p.r, torch.empty(p.J, device=DEV)
    elif case["kind"] in ("batch", "sweep"):
        s.B = sgtv.Batch(device=0, stream=_stream())
        if case["kind"] == "batch":
            probs = _batch_problems(case, seed)
            sched = autotune.batch_schedule([(p.I, p.J) for p in probs])
            with concurrent.futures.ThreadPoolExecutor(8) as ex:
                s.index = list(ex.map(lambda p: s.B.add_scan(p, sched), probs))
            s.images = [torch.empty(p.J, device=DEV) for p in probs]
        else:
            p, pairs = _sweep_problem(case, seed)
            w = _device(_weights(case))
            s.index = [s.B.add_scan(p, w=w, grouping=g, beta=b) for g, b in pairs]
            s.images = [torch.empty(p.J, device=DEV) for _ in pairs]
    else:
        params, s.x, s.target = _net_inputs(case, seed)
        s.net = sgtv.WarmStartNet(device=0, stream=_stream(), layers=case["layers"], height=case["height"],
                                  max_batch=case["batch"])
        s.net.set_params(params)
        s.out = torch.empty_like(s.x)
        s.grad = torch.empty(s.net.n_params, device=DEV)
    return s


def _device(w):
    return None if w is None else torch.from_numpy(w).to(DEV)


def run(s):
    c = s.case
    if c["kind"] == "scan":
        s.R.set_data(s.y, s.r, c["beta"], 1.0, c["sweeps"])
        s.R.iterate(c["iters"])
        rep = s.R.objective()
        return {"image": s.R.image(s.image), "total": rep["total"], "data": rep["data"], "tv": rep["tv"],
                "iter": rep["iter"]}
    if c["kind"] in ("batch", "sweep"):
        s.B.iterate(c["iters"])
        return [s.B.image(i, out) for i, out in zip(s.index, s.images)]
    if c["what"] == "gradient":
        return {"loss": s.net.backward(s.x, s.target, s.grad), "grad": s.grad}
    if c["what"] == "ratio":
        return s.net.start(s.x, "ratio", 1.1, s.out)
    return s.net.start(s.x, "direct", 1.1, s.out, 0.2)


# ---------------------------------------------------------------- what a pass cannot do without

_VALUE = {"f32": 4, "bf16": 2, "f16": 2}


def _scan_work(I, J, S, nnz, value, grouping, sweeps, iters):
    """Each product reads the matrix (values and 4-byte indices) once; a sweep reads y, r, the image, the split state
    and the sensitivity and writes the image; the split update reads the image and the split state and writes the
    state."""
    a = J if grouping else S
    sweep_bytes = 2 * nnz * (value + 4) + 8 * I + 4 * J * (1 + 4 + 1 + 1) + 4 * a
    split_bytes = 4 * J * (1 + 4 + 4) + 8 * a
    return iters * (sweeps * sweep_bytes + split_bytes), iters * (sweeps * (4 * nnz + 2 * I + 60 * J) + 25 * J)


def work(case):
    if case["kind"] == "scan":
        J, S = case["ny"] * case["nx"] * case["Q"], case["ny"] * case["nx"]
        b, f = _scan_work(case["I"], J, S, J * case["nnz_per_col"], _VALUE[case["storage"]], case["grouping"],
                          case["sweeps"], case["iters"])
    elif case["kind"] == "batch":
        rng = np.random.Generator(np.random.PCG64(12345))
        b = f = 0
        for _ in range(case["scans"]):
            side = int(rng.integers(case["low"], case["high"] + 1))
            Q = int(rng.integers(case["low"], case["high"] + 1))
            J = side * side * Q
            w = _scan_work(J // 2, J, side * side, J * case["nnz_per_col"], 4, 0, 1, case["iters"])
            b, f = b + w[0], f + w[1]
    elif case["kind"] == "sweep":
        J, S = case["ny"] * case["nx"] * case["Q"], case["ny"] * case["nx"]
        b = f = 0
        for g in (0, 1):
            w = _scan_work(case["I"], J, S, J * case["nnz_per_col"], 4, g, 1, case["iters"])
            b, f = b + case["betas"] * w[0], f + case["betas"] * w[1]
    else:
        px = case["batch"] * case["height"] * 64
        conv = 2 * px * 64 * 64 * 9
        params = case["layers"] * (64 * 9 * 64 + 64)
        if case["what"] == "gradient":   # forward, weight gradient of every layer, data gradient of all but the first
            f = conv * (3 * case["layers"] - 1)
            b = 2 * px * 64 * 4 + 2 * params * 4
        else:
            f = conv * case["layers"]
            b = 2 * px * 64 * 4 + params * 4
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------- the same in 64 bits, in plain torch

def _admm(p, iters, sweeps, beta, grouping, weights, objective):
    """ADMM for the spectrally grouped (0) or standard (1) TV problem from the uniform start, in 64 bits."""
    ny, nx, Q, I, J = p.ny, p.nx, p.Q, p.I, p.J
    w = [1.0] * 4 if weights is None else [float(t) for t in weights]
    A = torch.sparse_csr_tensor(p.rowptr, p.col.long(), p.val.double(), size=(I, J))
    counts = p.rowptr[1:] - p.rowptr[:-1]
    row = torch.repeat_interleave(torch.arange(I, device=DEV), counts)
    order = p.col.long().mul(I).add_(row).sort().indices          # by column, then row
    tptr = torch.zeros(J + 1, dtype=torch.int64, device=DEV)
    tptr[1:] = torch.bincount(p.col, minlength=J).cumsum(0)
    At = torch.sparse_csr_tensor(tptr, row[order], p.val[order].double(), size=(J, I))
    del row, order, counts
    y, r = p.y.double(), p.r.double()
    sens = (At @ torch.ones(I, dtype=torch.float64, device=DEV)).view(ny, nx, Q)
    f = torch.full((ny, nx, Q), float(y.sum() / sens.sum()), dtype=torch.float64, device=DEV)

    def shifted(u, q):
        """u at the neighbour in direction q (+x, -x, +y, -y), zero outside."""
        out = torch.zeros_like(u)
        if q == 0:
            out[:, :-1] = u[:, 1:]
        elif q == 1:
            out[:, 1:] = u[:, :-1]
        elif q == 2:
            out[:-1] = u[1:]
        else:
            out[1:] = u[:-1]
        return out

    def diff(u):
        return torch.stack([w[q] * (u - shifted(u, q)) for q in range(4)])

    def adjoint(t):
        # the difference of the neighbour in direction q towards this bin is its direction q ^ 1
        return sum(w[q] * t[q] - w[q ^ 1] * shifted(t[q ^ 1], q) for q in range(4))

    def norm(t):
        return t.square().sum(dim=0).sqrt() if grouping else t.square().sum(dim=(0, 3), keepdim=False).sqrt()[..., None]

    one = torch.ones_like(f)
    H = sum(w[q] ** 2 * (1 + shifted(one, q)) + 2 * w[q ^ 1] ** 2 * shifted(one, q) for q in range(4))
    d = torch.zeros((4, ny, nx, Q), dtype=torch.float64, device=DEV)
    c = torch.zeros_like(d)
    for _ in range(iters):
        for _ in range(sweeps):
            ratio = y / (A @ f.view(-1) + r)
            e = (At @ ratio).view(ny, nx, Q)
            B = sens + adjoint(diff(f) - d + c) - H * f
            C = f * e
            disc = (B * B + 4 * H * C).sqrt()
            f = torch.where(B <= 0, (disc - B) / (2 * H), 2 * C / (B + disc).clamp_min(1e-300))
        v = diff(f) + c
        nrm = norm(v)
        d = v * torch.where(nrm > beta, 1 - beta / nrm.clamp_min(1e-300), torch.zeros_like(nrm))
        c = v - d
    if not objective:
        return f.view(-1)
    m = A @ f.view(-1) + r
    data = float((m - y + torch.where(y > 0, y * (y.clamp_min(1e-300) / m).log(), torch.zeros_like(y))).sum())
    tv = float(norm(diff(f)).sum())
    return f.view(-1), data, tv


def _layers(case, params, x):
    """The network in 64 bits (inputs and weights as given, not rounded): (weights, biases, output)."""
    per = 64 * 9 * 64 + 64
    P = torch.from_numpy(params).to(DEV).double().requires_grad_(True)
    u = x
    for k in range(case["layers"]):
        W = P[k * per:k * per + 64 * 576].view(64, 3, 3, 64)
        b = P[k * per + 64 * 576:(k + 1) * per]
        pad = torch.nn.functional.pad(u, (0, 0, 1, 1, 1, 1))
        z = b
        for ky in range(3):
            for kx in range(3):
                z = z + pad[:, ky:ky + x.shape[1], kx:kx + 64].reshape(-1, 64) @ W[:, ky, kx].t()
        z = z.view(x.shape)
        u = z.relu() if k + 1 < case["layers"] else z.clamp_min(0) + torch.log1p(torch.exp(-z.abs()))
    return P, u


def exact(case, seed):
    if case["kind"] == "scan":
        p = _scan_problem(case, seed)
        f, data, tv = _admm(p, case["iters"], case["sweeps"], case["beta"], case["grouping"], _weights(case), True)
        return {"image": f, "total": data + case["beta"] * tv, "data": data, "tv": tv, "iter": None}
    if case["kind"] == "batch":
        return [_admm(p, case["iters"], 1, p.beta, 0, None, False) for p in _batch_problems(case, seed)]
    if case["kind"] == "sweep":
        p, pairs = _sweep_problem(case, seed)
        return [_admm(p, case["iters"], 1, b, g, _weights(case), False) for g, b in pairs]
    params, x, target = _net_inputs(case, seed)
    x, target = x.double(), target.double()
    if case["what"] == "gradient":
        P, u = _layers(case, params, x)
        loss = (u - target).square().mean()
        loss.backward()
        return {"loss": float(loss.detach()), "grad": P.grad}
    mean = x.mean(dim=(1, 2, 3), keepdim=True)
    with torch.no_grad():
        _, u = _layers(case, params, x / mean)
        if case["what"] == "ratio":
            return 1.1 * u * x
        return torch.maximum(1.1 * u * mean, 0.2 * 1.1 * mean)
