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


@pytest.mark.parametrize("resident", [True, False])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("dims,m,B", [
    ([20, 30, 70, 9], 3, 24),        # rows of 70 columns: a read past the end of row 4 finds the start of row 5
    ([40, 500, 300, 10], 2, 100),    # the same with the columns shared out
    ([30, 20, 17, 3], 2, 17),
])
def test_infinite_weights_of_a_silent_unit_stay_where_they_are(pkg, orc, dims, m, B, bf16, resident):
    """Unit 5 of layer 1 is never active; its first two weights into layer 2 are infinite, so units 0
    and 1 of layer 2 are 0 times infinity, which the ReLU shuts.  Everything else must come out as with
    those two units shut by their bias: bit for bit in the momentum, zeros in the padding."""
    _say(f"silent unit dims={dims} B={B} bf16={bf16} resident={resident}")
    got = []
    for infinite in (True, False):
        _, run = _problem(pkg, orc, dims, m, B, bf16=bf16, resident=resident)
        b1, b2 = (dict(_blocks(dims))[k].start for k in ("b1", "b2"))
        _weights(run, dims, 1)[:, :, 5] = 0.0
        run.X[:, b1 + 5] = -1.0
        if infinite:
            _weights(run, dims, 2)[:, 5, :2] = np.inf
        else:
            run.X[:, b2:b2 + 2] = -1e30
        run.local_steps(1)
        v = run.get_state()[1]
        w2 = dict(_blocks(dims))["W2"].start
        v[:, w2 + 5 * dims[2]:w2 + 5 * dims[2] + 2] = 0.0   # (their own momentum: the decay factor of 0 times infinity)
        got.append(v)
        assert not run.V[:, run.P:].any() and not run.X[:, run.P:].any()
        run.close()
    assert np.isfinite(got[0]).all() and np.abs(got[0]).max() > 0
    assert np.array_equal(got[0], got[1])


@pytest.mark.parametrize("B,bf16", [(32, False), (64, True), (128, True)])
def test_infinite_weights_of_a_silent_input_stay_where_they_are(pkg, B, bf16):
    """The same in the first layer's kernel that also runs the next step's forward pass, on ragged rows: the
    last feature is zero in every sample and its first two weights are infinite."""
    dims, m, N = [100, 300, 24, 10], 48, 200
    _say(f"silent input B={B} bf16={bf16}")
    data, labels = synth.gaussian_mixture(5, N, dims[0], dims[-1], mean_sd=1.0)
    data = synth.bf16_representable(data)
    data[:, -1] = 0.0
    x1, got = synth.init_params(5, dims), []
    b1 = dict(_blocks(dims))["b1"].start
    for infinite in (True, False):
        run = pkg.LocalSGD(m, pkg.make_model(pkg.KIND_MLP, dims, B=B, N=N, E=64, lr=0.05, beta=0.9, bf16=bf16), 5, x1, data, labels)
        run.set_resident(False)
        if infinite:
            _weights(run, dims, 1)[:, -1, :2] = np.inf
        else:
            run.X[:, b1:b1 + 2] = -1e30
        run.local_steps(3)
        v = run.get_state()[1]
        v[:, 99 * 300:99 * 300 + 2] = 0.0
        got.append(v)
        run.close()
    assert np.isfinite(got[0]).all() and np.abs(got[0]).max() > 0
    assert np.array_equal(got[0], got[1])
