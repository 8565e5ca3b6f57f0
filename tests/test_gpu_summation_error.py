"""How far fp32 gradients are from 64 bits must not depend on the route a shape takes: the kernels share
out their reductions differently, but none may add up in longer chains than the others."""
import numpy as np
import pytest

import synth
from test_gpu_parity import _blocks, _say, pkg  # noqa: F401

pytestmark = pytest.mark.gpu


def _error(pkg, dims, m, B, workers, **switches):
    """rms over the layers of the relative 2-norm error of one step's weight gradients (the momentum after
    the first step), median over some of the workers, so that a gate that opens on one side only does not count."""
    N = 1000
    data, labels = synth.gaussian_mixture(9, N, dims[0], dims[-1], mean_sd=1.0)
    x1 = synth.init_params(9, dims)
    run = pkg.LocalSGD(m, pkg.make_model(pkg.KIND_MLP, dims, B=B, N=N, E=64, lr=0.01, beta=0.0), 9, x1, data, labels)
    for name, value in switches.items():
        getattr(run, name)(value)
    run.local_steps(1)
    idx, V, x = run.last_indices(), run.get_state()[1].astype(np.float64), x1.astype(np.float64)
    run.close()
    sl, errors = dict(_blocks(dims)), []
    for i in range(workers):
        a, W = [data[idx[i]].astype(np.float64)], []
        for l, (d, e) in enumerate(zip(dims, dims[1:]), 1):
            W.append(x[sl[f"W{l}"]].reshape(d, e))
            z = a[-1] @ W[-1] + x[sl[f"b{l}"]]
            a.append(z if l == len(dims) - 1 else np.maximum(z, 0.0))
        p = np.exp(a[-1] - a[-1].max(1, keepdims=True))
        dz = p / p.sum(1, keepdims=True)
        dz[np.arange(B), labels[idx[i]]] -= 1.0
        dz /= B
        row = []
        for l in range(len(dims) - 1, 0, -1):
            g = a[l - 1].T @ dz
            row.append(np.linalg.norm(V[i, sl[f"W{l}"]].reshape(g.shape) - g) / np.linalg.norm(g))
            dz = (dz @ W[l - 1].T) * (a[l - 1] > 0)
        errors.append(row)
    return float(np.sqrt(np.mean(np.median(errors, axis=0) ** 2)))


@pytest.mark.parametrize("dims,B", [([324, 16, 16, 10], 48), ([400, 16, 10, 3], 16), ([196, 20], 60), ([130, 70, 33, 7], 48),
                                    ([64, 40, 84, 20, 11], 62)])
def test_models_on_one_compute_unit(pkg, dims, B):
    """Against the launches per layer.  Both are sums of the same products; a tenth is left for chance."""
    on = _error(pkg, dims, 5, B, 5, set_resident=True)
    off = _error(pkg, dims, 5, B, 5, set_resident=False)
    _say(f"error dims={dims} B={B}: on one compute unit {on:.3e}, launches per layer {off:.3e}")
    assert on != off   # (two routes)
    assert on < 1.1 * off


@pytest.mark.parametrize("dims,B", [([784, 256, 10], 64), ([65, 40, 5], 33), ([1024, 130, 16], 17), ([300, 250, 2], 64),
                                    ([64, 10], 32), ([256, 16], 64), ([100, 3], 20)])
def test_resident_models(pkg, dims, B):
    """The same for the two resident kernels, with more workers since a few classes leave much to chance.  (Two
    layers: 0.8 to 0.9 of what one sum per product gave; softmax regression 0.97 to 1.03 of it.)"""
    on = _error(pkg, dims, 16, B, 16, set_resident=True)
    off = _error(pkg, dims, 16, B, 16, set_resident=False)
    _say(f"error dims={dims} B={B}: resident {on:.3e}, launches per layer {off:.3e}")
    assert on < 1.1 * off   # (three classes of 100 inputs: the same bits)


@pytest.mark.parametrize("dims,m,B", [([2048, 500, 10], 24, 33), ([1024, 704, 10], 23, 64), ([784, 640, 10], 20, 100)])
def test_forward_products_of_many_workers(pkg, dims, m, B):
    """The same four workers among few and among many: with more column chunks in the launch a product may
    be shared out differently among wavefronts, but not be summed up in longer chains."""
    few, many = _error(pkg, dims, 4, B, 4, set_resident=False), _error(pkg, dims, m, B, 4, set_resident=False)
    _say(f"error dims={dims} B={B}: 4 workers {few:.3e}, {m} workers {many:.3e}")
    assert many < 1.1 * few


def _forward_errors(pkg, dims, m, B, calls, positive):
    """How far the last layer's weight gradient of a call's second step is from 64 bits, with the first layer's kernel and with
    the launches per layer, rms over several calls.  bf16 models of two layers whose weights do not move (a rate of 1e-12,
    no momentum): what differs are activations of the first layer that a sum just beside them rounds the other way."""
    import torch
    N, sl = 1000, dict(_blocks(dims))
    rng, bf16 = np.random.default_rng(7), synth.bf16_representable
    labels = rng.integers(0, dims[-1], N).astype(np.int32)
    data, x1 = bf16(rng.random((N, dims[0]), dtype=np.float32)), bf16(synth.init_params(9, dims))
    if positive:
        x1[sl["W1"]] = bf16(rng.random(dims[0] * dims[1], dtype=np.float32) * (4.0 / dims[0]))
    model = pkg.make_model(pkg.KIND_MLP, dims, B=B, N=N, E=64, lr=1e-12, beta=0.0, bf16=True)
    runs = [pkg.LocalSGD(m, model, 9, x1, data, labels) for _ in range(2)]
    for run, fused in zip(runs, (True, False)):
        run.set_resident(False)
        run.set_first_layer_fusion(fused)
    assert [run.first_layer_workgroup() for run in runs] == [(96, 8), (0, 0)]
    x = torch.from_numpy(x1).cuda().double()
    W1, W2 = x[sl["W1"]].view(dims[0], dims[1]), x[sl["W2"]].view(dims[1], dims[2])
    data, labels = torch.from_numpy(data).cuda().double(), torch.from_numpy(labels).cuda().long()
    err = [0.0, 0.0]
    for _ in range(calls):
        for run in runs:
            run.local_steps(2)
        idx, V = runs[0].last_indices(), [run.V[:, sl["W2"]].double() for run in runs]
        for i in range(m):
            at = torch.from_numpy(np.asarray(idx[i], np.int64)).cuda()
            a = torch.relu(data[at] @ W1 + x[sl["b1"]]).float().bfloat16().double()
            dz = torch.softmax(a @ W2 + x[sl["b2"]], 1)
            dz[torch.arange(B), labels[at]] -= 1.0
            g = (a.t() @ (dz / B).float().bfloat16().double()).reshape(-1)
            for r in range(2):
                err[r] += float(((V[r][i] - g).norm() / g.norm()) ** 2) / (m * calls)
    for run in runs:
        run.close()
    return np.sqrt(err)


def test_first_layer_with_chunks_of_96_columns(pkg):
    """Geometric mean over six models, since one sum beside a rounding step moves all deltas of a sample.  Positive products, of
    which every further one makes the sum larger, tell long chains best.  (One sum over all inputs: 1.22.)"""
    ratios = []
    for dims, m, B in [([3072, 1500, 10], 12, 128), ([3072, 1400, 100], 16, 100), ([784, 673, 10], 32, 70)]:
        for positive in (False, True):
            on, off = _forward_errors(pkg, dims, m, B, 12, positive)
            _say(f"error dims={dims} B={B} positive={positive}: chunks of 96 columns {on:.3e}, launches per layer {off:.3e}")
            ratios.append(on / off)
    assert np.exp(np.mean(np.log(ratios))) < 1.1, ratios
