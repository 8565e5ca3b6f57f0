"""fp32 products formed of bf16 parts: no further from 64 bits than the fp32 matrix instructions, right where operands are too
large for parts, and infinities that come out as such."""
import numpy as np
import pytest

import synth
from test_gpu_parity import _blocks, _say, pkg  # noqa: F401
from test_gpu_summation_error import _error

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _parts(monkeypatch):
    monkeypatch.setenv("LC_SPLIT_PRODUCTS", "1")


# (64- and 128-sample kernels; whole and ragged rows; shared-out columns; the first-layer kernel with 4 and 8 wavefronts
# does not run in a call of one step, see the calls of two below)
SHAPES = [([784, 500, 300, 10], 16, 100), ([512, 512, 512, 10], 16, 64), ([300, 520, 136, 70], 40, 33), ([1025, 705, 321, 10], 12, 128),
          ([2048, 1024, 128, 10], 16, 64)]


@pytest.mark.parametrize("dims,m,B", SHAPES)
def test_error_against_64_bits(pkg, monkeypatch, dims, m, B):
    """Six roundings of a sum per 32 products instead of eight; a twentieth is left for chance."""
    parts = _error(pkg, dims, m, B, 4)
    monkeypatch.setenv("LC_SPLIT_PRODUCTS", "0")
    plain = _error(pkg, dims, m, B, 4)
    _say(f"error dims={dims} m={m} B={B}: parts {parts:.3e}, fp32 instructions {plain:.3e}")
    assert parts != plain   # (two routes)
    assert parts < 1.05 * plain


BIG = 2.0 ** 62   # above what goes through parts


def _run(pkg, dims, m, B, steps, scale):
    """A model with one input and one hidden unit of another scale: the same function of the data."""
    N = 64
    data, labels = synth.gaussian_mixture(9, N, dims[0], dims[-1], mean_sd=1.0)
    x1 = synth.init_params(9, dims).copy()
    sl = dict(_blocks(dims))
    W1, W2 = x1[sl["W1"]].reshape(dims[0], dims[1]), x1[sl["W2"]].reshape(dims[1], dims[2])
    W1[5, 7] = 0.0   # (divided by the scale twice it would be a subnormal number)
    data[:, 5] *= scale
    W1[5] /= scale
    W1[:, 7] /= scale
    W2[7] *= scale
    run = pkg.LocalSGD(m, pkg.make_model(pkg.KIND_MLP, dims, B=B, N=N, E=64, lr=0.0, beta=0.0), 9, x1, data, labels)
    run.set_resident(False)
    run.local_steps(steps)
    V = run.get_state()[1][:2].astype(np.float64)
    losses = run.local_losses()
    run.close()
    g1 = V[:, sl["W1"]].reshape(2, dims[0], dims[1])
    g2 = V[:, sl["W2"]].reshape(2, dims[1], dims[2])
    g1[:, 5] /= scale
    g1[:, :, 7] /= scale
    g2[:, 7] *= scale
    return [g1, g2, V[:, sl["W3"]]], losses


@pytest.mark.parametrize("dims,m,B", [([784, 500, 300, 10], 16, 100), ([512, 512, 512, 10], 16, 64), ([257, 250, 300, 10], 64, 64),
                                      ([256, 1024, 136, 10], 16, 64), ([300, 520, 136, 10], 40, 40)])
@pytest.mark.parametrize("steps", [1, 2])
def test_operands_too_large_for_parts(pkg, dims, m, B, steps):
    """A power of two as the scale: the gradients are the same bits apart from it, but for the order of sums (the
    walks over large operands take the fp32 instructions)."""
    _say(f"large operands dims={dims} m={m} B={B} steps={steps}")
    plain, l0 = _run(pkg, dims, m, B, steps, 1.0)
    large, l1 = _run(pkg, dims, m, B, steps, BIG)
    assert np.allclose(l0, l1, rtol=1e-5)
    for a, b in zip(plain, large):
        assert np.isfinite(b).all()
        # both are within about 2e-7 of the exact gradient (relative 2-norm); no gate may differ: the learning rate is zero
        assert np.linalg.norm(a - b) < 2e-6 * np.linalg.norm(a)


@pytest.mark.parametrize("dims,m,B", [([784, 500, 300, 10], 16, 100), ([512, 512, 512, 10], 16, 64), ([257, 250, 300, 10], 64, 64)])
@pytest.mark.parametrize("where", ["W1", "W2", "data"])
def test_infinities_reach_the_local_losses(pkg, dims, m, B, where):
    """Parts of an infinity are an infinity and NaN, which the ReLU would shut: two steps, the second one's first layer in
    the kernel that also runs the first one's backward pass where that applies."""
    _say(f"infinite {where} dims={dims} m={m} B={B}")
    N = 64
    data, labels = synth.gaussian_mixture(9, N, dims[0], dims[-1], mean_sd=1.0)
    data = np.abs(data)
    if where == "data":
        data[:, 3] = np.inf
    run = pkg.LocalSGD(m, pkg.make_model(pkg.KIND_MLP, dims, B=B, N=N, E=64, lr=0.0, beta=0.0), 9, synth.init_params(9, dims), data, labels)
    run.set_resident(False)
    for l in range(1, len(dims)):   # every unit positive, so that the infinity is passed on
        run.X[:, dict(_blocks(dims))[f"W{l}"]] = 0.01
    if where != "data":
        l = int(where[1])
        run.X[:, dict(_blocks(dims))[where]].view(m, dims[l - 1], dims[l])[:, -1, 3] = np.inf
    run.local_steps(1)
    losses = run.local_losses()
    assert not np.isfinite(losses).any(), losses
    run.close()
