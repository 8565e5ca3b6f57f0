"""The work a user of this library has it do, as cases that can be timed and compared.

Four kinds, each through the public binding (paper_1810_08313_amd.LocalSGD):

  train   n communication periods of tau local steps with the averaging step after each
          (local_periods), the models then read from X and the momentum from V
  loss    the training loss of the averaged model, which the schedule asks for at every decision
  update  one synchronous step from gradients the caller brings (update_from_grad, average; or
          the two as one call)
  block   the block-momentum averaging step of callers that may not allocate

A pass continues from the state the one before it left, as a training loop does.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1810_08313_amd as pkg

DEV = "cuda:0"


# ------------------------------------------------------------------------------------- the cases

def _train(name, dims, m, B, tau, periods, lr, beta=0.9, wd=0.0, bf16=False, N=20000, image=False, lazy=False,
           partition=False):
    return dict(name=name, kind="train", dims="-".join(map(str, dims)), m=m, B=B, tau=tau, periods=periods, lr=lr,
                beta=beta, wd=wd, bf16=bf16, N=N, image=image, lazy=lazy, partition=partition)


def listed():
    # The rates of the image-shaped models are about their own after two tenfold decays, as a step
    # schedule has them for most of a run: at the starting rate a trajectory of 10 to 20 steps
    # amplifies one bf16 rounding to several per cent.
    return [
        # softmax regression on 4 workers, one period: the smallest call there is, all launch latency
        _train("softmax_regression_one_period", [64, 10], 4, 32, 4, 1, 0.05, beta=0.0),
        # digits-sized two-layer network, fp32, several periods in one call
        _train("two_layer_fp32", [784, 256, 10], 8, 64, 5, 4, 0.1, N=60000, lazy=True),
        # odd widths, a batch that is no multiple of anything, every worker on its own shard
        _train("small_odd_widths", [130, 70, 33, 7], 3, 48, 3, 2, 0.05, wd=1e-4, partition=True, N=2000),
        # a middling fp32 network with widths that are not multiples of 64
        _train("three_layer_ragged_fp32", [784, 500, 300, 10], 16, 100, 5, 1, 0.05, N=20000),
        # the same kind of network at a size whose state streams from memory, bf16 operands
        _train("three_layer_ragged_bf16", [3072, 1500, 1000, 100], 16, 100, 5, 1, 5e-4, bf16=True, image=True),
        # image-shaped inputs, fp32 operands
        _train("three_layer_fp32", [3072, 1024, 1024, 10], 16, 64, 5, 1, 5e-4, image=True, lazy=True),
        # the two large configurations: long periods, and the second one fully synchronous
        _train("three_layer_bf16_long_period", [3072, 1024, 1024, 10], 16, 128, 20, 1, 5e-4, bf16=True, image=True,
               lazy=True, N=50000),
        _train("four_layer_bf16_64_workers", [3072, 2048, 2048, 2048, 10], 64, 32, 8, 1, 1.2e-4, bf16=True, image=True,
               lazy=True, N=50000),
        _train("four_layer_bf16_synchronous", [3072, 2048, 2048, 2048, 10], 64, 32, 1, 4, 2e-4, bf16=True, image=True,
               lazy=True, N=50000),
        # the loss a decision reads, right after an averaging step, at the largest model
        dict(name="loss_of_averaged_model", kind="loss", dims="3072-2048-2048-2048-10", m=4, E=8192, bf16=True),
        # flat-vector stress: update from explicit gradients and averaging, 16 workers x 25 million
        dict(name="update_and_average_25m", kind="update", dims="3072-4096-3072-10", m=16, fused=False),
        # the averaging step under block momentum without a handle
        dict(name="block_momentum_average", kind="block", m=8, P=4205578),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi):
    """Any width, or (as often) one rounded to the multiples of 4 or 64 that layers usually have."""
    w = _log(rng, lo, hi)
    unit = rng.choice([1, 4, 64])
    return max(unit, w // unit * unit)


def draw(rng):
    kind = rng.choice(["train"] * 7 + ["loss", "update", "block"])
    if kind == "loss":
        dims = [_width(rng, 64, 3072)] + [_width(rng, 64, 2048) for _ in range(rng.randint(1, 3))] + [rng.randint(2, 100)]
        return dict(kind="loss", dims="-".join(map(str, dims)), m=rng.randint(2, 8), E=_log(rng, 500, 8192),
                    bf16=rng.random() < 0.5)
    if kind == "update":
        dims = [_width(rng, 64, 3072), _width(rng, 64, 3072), _width(rng, 64, 3072), rng.randint(2, 100)]
        return dict(kind="update", dims="-".join(map(str, dims)), m=rng.randint(2, 16), fused=rng.random() < 0.5)
    if kind == "block":
        return dict(kind="block", m=rng.randint(2, 16), P=_log(rng, 1000, 4400000))
    size = rng.choice(["regression", "two", "small", "middle", "large"])
    bf16 = rng.random() < 0.5
    common = dict(wd=rng.choice([0.0, 0.0, 1e-4]), partition=rng.random() < 0.3, lazy=rng.random() < 0.5, bf16=bf16)
    if size == "regression":
        c = _train("", [_width(rng, 16, 256), rng.randint(2, 16)], rng.randint(2, 16), rng.randint(8, 128),
                   rng.randint(1, 20), rng.randint(1, 4), 0.05, beta=rng.choice([0.0, 0.9]), N=20000, **common)
    elif size == "two":
        c = _train("", [_width(rng, 64, 1024), _width(rng, 32, 256), rng.randint(2, 16)], rng.randint(2, 16),
                   rng.randint(16, 128), rng.randint(1, 20), 1, 0.02, N=20000, **common)
    elif size == "small":
        dims = [_width(rng, 32, 512)] + [_width(rng, 16, 256) for _ in range(rng.randint(1, 3))] + [rng.randint(2, 40)]
        c = _train("", dims, rng.randint(2, 16), rng.randint(8, 128), rng.randint(1, 8), 1, 0.02, N=20000, **common)
    elif size == "middle":
        dims = [_width(rng, 256, 1024)] + [_width(rng, 128, 768) for _ in range(2)] + [rng.randint(2, 100)]
        c = _train("", dims, rng.randint(4, 16), rng.randint(16, 128), rng.randint(1, 5), 1, 0.02, N=20000, **common)
    else:
        dims = [_width(rng, 1024, 3072)] + [_width(rng, 700, 2048) for _ in range(rng.randint(2, 3))] + [rng.choice([10, 100])]
        c = _train("", dims, rng.randint(8, 32), rng.randint(16, 128), rng.randint(1, 5), 1, 5e-4, image=True, **common)
    del c["name"]
    return c


def _dims(case):
    return [int(d) for d in case["dims"].split("-")]


def _params(dims):
    return sum(a * b + b for a, b in zip(dims, dims[1:]))


# ---------------------------------------------------------------------------- inputs and the call

def _gen(seed, stream):
    return torch.Generator(device=DEV).manual_seed((int(seed) * 1000003 + stream) % (2 ** 62))


def _dataset(case, seed, N):
    """N samples of d_0 features and their labels: image-shaped (uniform pixels with a class
    offset), or a Gaussian mixture scaled to unit variance as standardised features are."""
    dims = _dims(case)
    g = _gen(seed, 1)
    y = torch.randint(0, dims[-1], (N,), generator=g, device=DEV, dtype=torch.int32)
    mean = torch.randn((dims[-1], dims[0]), generator=g, device=DEV)
    if case.get("image", True):
        x = torch.rand((N, dims[0]), generator=g, device=DEV) + 0.1 * mean[y.long()]
    else:
        x = 0.9 * torch.randn((N, dims[0]), generator=g, device=DEV) + 0.4 * mean[y.long()]
    if case["bf16"]:
        x = x.bfloat16().float()
    return x, y


def _start(dims, seed):
    """He initialisation, zero biases (softmax regression starts at zero)."""
    if len(dims) == 2:
        return torch.zeros(_params(dims), device=DEV)
    g = _gen(seed, 2)
    parts = []
    for a, b in zip(dims, dims[1:]):
        parts.append(torch.randn(a * b, generator=g, device=DEV) * math.sqrt(2.0 / a))
        parts.append(torch.zeros(b, device=DEV))
    return torch.cat(parts)


def _buffers(case, seed, x, y):
    """Momentum of a run in progress, the same for every worker: a gradient that stays as it is
    adds up to 1 / (1 - beta) of itself.  Here the gradient at the start over 1024 samples, in
    64 bits, plain torch."""
    dims, n = _dims(case), 1024
    p = _start(dims, seed).double()
    if case["beta"] == 0.0:
        return torch.zeros_like(p, dtype=torch.float32)
    a, acts, off, offs = x[:n].double(), [], 0, []
    for l, (d, e) in enumerate(zip(dims, dims[1:])):
        acts.append(a)
        offs.append(off)
        z = a @ p[off:off + d * e].view(d, e) + p[off + d * e:off + d * e + e]
        a, off = z.relu() if l < len(dims) - 2 else z, off + d * e + e
    dz = torch.softmax(a, 1)
    dz[torch.arange(dz.shape[0], device=DEV), y[:n].long()] -= 1.0
    dz /= dz.shape[0]
    g = torch.empty_like(p)
    for l in range(len(dims) - 2, -1, -1):
        d, e, off = dims[l], dims[l + 1], offs[l]
        g[off:off + d * e] = (acts[l].t() @ dz).reshape(-1)
        g[off + d * e:off + d * e + e] = dz.sum(0)
        if l > 0:
            dz = (dz @ p[off:off + d * e].view(d, e).t()) * (acts[l] > 0)
    return (g / (1.0 - case["beta"])).float()


def _gradients(m, P, seed):
    out = torch.empty((m, P), device=DEV)
    g = _gen(seed, 3)
    for i in range(m):
        out[i] = torch.randn(P, generator=g, device=DEV) * 1e-3
    return out


def _spread_models(m, P, seed):
    """Models of m workers some local steps after they last agreed."""
    g = _gen(seed, 4)
    base = torch.randn(P, generator=g, device=DEV) * 0.1
    return torch.stack([base + torch.randn(P, generator=g, device=DEV) * 1e-2 for _ in range(m)])


def _handle(case, seed, B, N, E, lr, beta, wd, partition, x, y):
    md = pkg.make_model(pkg.KIND_MLP, _dims(case), B=B, N=N, E=E, lr=lr, beta=beta, wd=wd, bf16=case.get("bf16", False),
                        sampler=1 if partition else 0)
    return pkg.LocalSGD(case["m"], md, int(seed), None, x.cpu().numpy(), y.cpu().numpy())


def prepare(case, seed):
    if case["kind"] == "block":
        m, P = case["m"], case["P"]
        Ps = pkg.lc_row_stride(P)
        X = torch.zeros((m, Ps), device=DEV)
        X[:, :P] = _spread_models(m, P, seed)
        synced = torch.zeros((m, Ps), device=DEV)
        synced[:, :P] = torch.randn(P, generator=_gen(seed, 5), device=DEV) * 0.1
        return dict(case=case, X=X, synced=synced)
    dims = _dims(case)
    if case["kind"] == "update":
        x, y = torch.zeros((8, dims[0]), device=DEV), torch.zeros(8, dtype=torch.int32, device=DEV)
        run = _handle(case, seed, 8, 8, 8, 0.05, 0.9, 0.0, False, x, y)
        run.X[:, :run.P] = _start(dims, seed)
        G = torch.zeros((run.m, run.Ps), device=DEV)
        G[:, :run.P] = _gradients(run.m, run.P, seed)
        run.set_grad(G)
        return dict(case=case, run=run)
    if case["kind"] == "loss":
        x, y = _dataset(case, seed, case["E"])
        run = _handle(case, seed, 32, case["E"], case["E"], 0.02, 0.9, 0.0, False, x, y)
        run.X[:, :run.P] = _start(dims, seed)
        run.set_lazy_broadcast(True)
        run.average()
        return dict(case=case, run=run)
    x, y = _dataset(case, seed, case["N"])
    run = _handle(case, seed, case["B"], case["N"], min(1024, case["N"]), case["lr"], case["beta"], case["wd"],
                  case["partition"], x, y)
    run.X[:, :run.P] = _start(dims, seed)
    run.V[:, :run.P] = _buffers(case, seed, x, y)
    run.set_lazy_broadcast(case["lazy"])
    if case["lazy"]:
        run.average()   # a call between two others begins with the averaged model, not yet copied to the rows
    return dict(case=case, run=run)


def run(state):
    case = state["case"]
    if case["kind"] == "block":
        # the workers agreed on `synced`; meanwhile they have moved on to X
        P = case["P"]
        pkg.average_block_momentum_static(state["synced"], None, P, 0.05, 0.3, True)
        pkg.average_block_momentum_static(state["X"], None, P, 0.05, 0.3, False)
        return state["X"]
    lsgd = state["run"]
    if case["kind"] == "loss":
        return lsgd.loss()
    if case["kind"] == "update":
        if case["fused"]:
            lsgd.update_from_grad_and_average()
        else:
            lsgd.update_from_grad()
            lsgd.average()
    else:
        lsgd.local_periods(case["tau"], case["periods"])
        lsgd.materialize()
    return {"X": lsgd.X, "V": lsgd.V}


# ------------------------------------------------------------------------------- what a pass needs

def work(case):
    if case["kind"] == "block":
        return {"bytes": 4.0 * case["P"] * (2 * case["m"] + 1), "flops": 2.0 * case["P"] * case["m"]}
    dims = _dims(case)
    P, m = _params(dims), case["m"]
    weights = sum(a * b for a, b in zip(dims, dims[1:]))
    if case["kind"] == "update":   # X, V, G read; V and the averaged model written to every row
        return {"bytes": 20.0 * m * P, "flops": 6.0 * m * P}
    if case["kind"] == "loss":
        return {"bytes": 4.0 * P + (2.0 if case["bf16"] else 4.0) * case["E"] * dims[0], "flops": 2.0 * case["E"] * weights}
    steps = case["tau"] * case["periods"]
    batch = (2.0 if case["bf16"] else 4.0) * case["B"] * dims[0] * m * steps
    if 8.0 * m * P <= 256e6:
        state = 16.0 * m * P                # stays on chip between the steps of a pass
    elif case["tau"] == 1:
        state = 8.0 * m * P * steps         # one model for all workers; their momentum in and out
    else:
        state = 12.0 * m * P * steps        # two consecutive models in, the next one out
    flops = 2.0 * case["B"] * (3.0 * weights - dims[0] * dims[1]) * m * steps
    return {"bytes": state + batch, "flops": flops}


def tolerance(case):
    if case["kind"] == "block":
        return {"rel": 1e-6}
    if case["kind"] == "update":
        return {"rel": 1e-6}
    if case["kind"] == "loss":
        return {"rel": 1e-5}
    # A ReLU gate that opens on one side and not on the other moves one sample's term in a column
    # of the momentum; a bf16 operand that rounds the other way moves 2^-8 of it.
    if case["bf16"]:
        return {"rel": 2e-2, "max": 0.9}
    return {"rel": 1e-3, "max": 0.5}


# ------------------------------------------------------------------- the same in 64 bits, plain torch

_G = 0x9E3779B97F4A7C15
_M64 = (1 << 64) - 1


def _mix(z):
    z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & _M64
    z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & _M64
    return z ^ (z >> 31)


def _indices(case, seed, i, k):
    """Samples of worker i at iteration k."""
    N, B, m, seed = case["N"], case["B"], case["m"], int(seed) & _M64
    if not case["partition"]:
        h = _mix((_mix((seed + _G * (k + 1)) & _M64) + _G * (i + 1)) & _M64)
        return [_mix((h + _G * (b + 1)) & _M64) % N for b in range(B)]
    lo, hi = i * N // m, (i + 1) * N // m
    S = (N // m) // B
    key = _mix((_mix((seed + _G * (k // S + 1)) & _M64) + _G * (i + 1)) & _M64)
    n, w = hi - lo, 1
    while (1 << (2 * w)) < n:
        w += 1
    mask = (1 << w) - 1
    out = []
    for b in range(B):
        x = (k % S) * B + b
        while True:
            left, right = x >> w, x & mask
            for r in range(4):
                left, right = right, left ^ (_mix((key + _G * (r + 1) + right) & _M64) & mask)
            x = (left << w) | right
            if x < n:
                break
        out.append(lo + x)
    return out


def _padded(rows, Ps):
    out = torch.zeros((rows.shape[0], Ps), dtype=torch.float64, device=DEV)
    out[:, :rows.shape[1]] = rows
    return out


def _f32(v):
    return float(np.float32(v))


def exact(case, seed):
    if case["kind"] == "block":
        m, P = case["m"], case["P"]
        mean = _spread_models(m, P, seed).double().mean(0)
        xs = (torch.randn(P, generator=_gen(seed, 5), device=DEV) * 0.1).double()
        u = (xs - mean) / _f32(0.05)
        new = xs - _f32(0.05) * u
        return _padded(new.expand(m, P), -(-P // 64) * 64)
    dims = _dims(case)
    P, m = _params(dims), case["m"]
    Ps = -(-P // 64) * 64
    if case["kind"] == "update":
        x = _start(dims, seed).double()
        V, total = _gradients(m, P, seed).double(), torch.zeros(P, dtype=torch.float64, device=DEV)
        for i in range(m):
            total += x - _f32(0.05) * V[i]
        return {"X": _padded((total / m).expand(m, P), Ps), "V": _padded(V, Ps)}
    if case["kind"] == "loss":
        x, y = _dataset(case, seed, case["E"])
        a, p, off = x.double(), _start(dims, seed).double(), 0
        for l, (d, e) in enumerate(zip(dims, dims[1:])):
            a = a @ p[off:off + d * e].view(d, e) + p[off + d * e:off + d * e + e]
            off += d * e + e
            if l < len(dims) - 2:
                a = a.relu()
        return float(torch.nn.functional.cross_entropy(a, y.long(), reduction="mean"))
    data, labels = _dataset(case, seed, case["N"])
    V = _buffers(case, seed, data, labels).double().expand(m, P).clone()
    data, labels = data.double(), labels.long()
    lr, beta, wd, B, L = _f32(case["lr"]), _f32(case["beta"]), _f32(case["wd"]), case["B"], len(dims) - 1
    # with bf16 operands: activations and deltas are rounded when produced, weights when read
    op = (lambda t: t.float().bfloat16().double()) if case["bf16"] else (lambda t: t)
    X = _start(dims, seed).double().expand(m, P).clone()
    offs = [0]
    for d, e in zip(dims, dims[1:]):
        offs.append(offs[-1] + d * e + e)
    k = 0
    for _ in range(case["periods"]):
        for _ in range(case["tau"]):
            for i in range(m):
                idx = torch.tensor(_indices(case, seed, i, k), device=DEV)
                acts = [data[idx]]
                W = [X[i, offs[l]:offs[l] + dims[l] * dims[l + 1]].view(dims[l], dims[l + 1]) for l in range(L)]
                Wo = [op(w) for w in W]
                for l in range(L):
                    z = acts[l] @ Wo[l] + X[i, offs[l] + dims[l] * dims[l + 1]:offs[l + 1]]
                    acts.append(z if l == L - 1 else op(z.relu()))
                dz = torch.softmax(acts[L], 1)
                dz[torch.arange(B, device=DEV), labels[idx]] -= 1.0
                dz = op(dz / B)
                for l in range(L - 1, -1, -1):
                    grad = torch.cat([(acts[l].t() @ dz).reshape(-1), dz.sum(0)])
                    if l > 0:
                        dz = op((dz @ Wo[l].t()) * (acts[l] > 0))
                    s = slice(offs[l], offs[l + 1])
                    V[i, s] = beta * V[i, s] + grad + wd * X[i, s]
                    X[i, s] -= lr * V[i, s]
            k += 1
        X[:] = X.mean(0)
    return {"X": _padded(X, Ps), "V": _padded(V, Ps)}
