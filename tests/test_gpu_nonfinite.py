"""Infinities in weights and data: what a call reports of them does not depend on how a kernel forms
its products (operands split in parts, rows read in place of rows that do not exist, columns read
past the end of a row)."""
import numpy as np
import pytest

import synth
from test_gpu_parity import _blocks, _problem, _say, pkg  # noqa: F401

pytestmark = pytest.mark.gpu


def _weights(run, dims, l):
    """View of W_l of every replica: [m, d_{l-1}, d_l]."""
    sl = dict(_blocks(dims))[f"W{l}"]
    return run.X[:, sl].view(run.m, dims[l - 1], dims[l])


def _evaluation(pkg, dims, E, data, bf16):
    labels = np.zeros(E, np.int32)
    md = pkg.make_model(pkg.KIND_MLP, dims, B=16, N=E, E=E, lr=0.1, beta=0.9, bf16=bf16)
    return pkg.LocalSGD(1, md, 3, synth.init_params(3, dims), data, labels)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("dims,E", [([64, 768, 10], 8192), ([70, 256, 10], 8192)])   # 128 x 128 and 64 x 64 tiles
def test_infinite_data_reach_the_loss(pkg, dims, E, bf16):
    """One feature of a few samples is infinite and meets weights that bf16 holds exactly (the other
    parts of a split weight are zero) or does not (they have either sign): the hidden units are
    infinite, and so the loss is not a number."""
    _say(f"infinite data dims={dims} bf16={bf16}")
    for w in (1.0, 1.0 + 2.0 ** -9, 1.0 - 2.0 ** -12):
        data = synth.bf16_representable(np.random.default_rng(5).standard_normal((E, dims[0])).astype(np.float32))
        data[7::1000, 5] = np.inf
        run = _evaluation(pkg, dims, E, data, bf16)
        _weights(run, dims, 1)[:, 5, :] = w
        _weights(run, dims, 2)[:] = 0.5
        with pytest.raises(pkg.LcError) as e:
            run.loss()
        assert e.value.status == -7
        run.close()


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("dims,E", [([70, 768, 10], 8192), ([70, 130, 10], 500), ([33, 256, 10], 8192)])
def test_infinite_last_weight_row_reaches_the_loss(pkg, dims, E, bf16):
    """The padding of the reduction reads a row that exists in place of rows that do not."""
    _say(f"infinite last row, evaluation, dims={dims} bf16={bf16}")
    data = synth.bf16_representable(np.random.default_rng(5).uniform(0.5, 1.0, (E, dims[0])).astype(np.float32))
    run = _evaluation(pkg, dims, E, data, bf16)
    _weights(run, dims, 1)[:, -1, 3] = np.inf
    _weights(run, dims, 2)[:] = 0.5
    with pytest.raises(pkg.LcError) as e:
        run.loss()
    assert e.value.status == -7
    run.close()


@pytest.mark.parametrize("resident", [True, False])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("dims,B", [([70, 130, 10], 16), ([70, 130, 33, 10], 100), ([33, 65, 5], 48)])
def test_infinite_last_weight_row_reaches_the_local_losses(pkg, orc, dims, B, bf16, resident):
    _say(f"infinite last row, step, dims={dims} B={B} bf16={bf16} resident={resident}")
    _, run = _problem(pkg, orc, dims, 2, B, bf16=bf16, resident=resident)
    for l in range(1, len(dims)):   # every unit positive, so that the infinity is passed on
        _weights(run, dims, l)[:] = 0.01
    run.X[:, dict(_blocks(dims))["b1"]] = 100.0
    _weights(run, dims, 1)[:, -1, 3] = np.inf
    run.local_steps(1)
    losses = run.local_losses()
    assert not np.isfinite(losses).any(), losses
    run.close()
