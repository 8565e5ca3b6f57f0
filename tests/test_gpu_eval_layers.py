"""The evaluation pass of many samples (hidden layers as one dense product with split fp32 operands)
against the oracle at tile edges, and its behaviour on numbers that are not finite."""
import numpy as np
import pytest

from test_gpu_parity import _problem, _say, pkg  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = [
    # dims, E            -- 64 x 64 tiles: one column over two tiles; a short reduction; two passes
    ([33, 129, 10], 8192),
    ([70, 200, 130, 5], 8321),
    # 128 x 128 tiles: a ragged last one, and whole ones
    ([65, 700, 7], 8192),
    ([64, 768, 768, 10], 8100),
]


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("dims,E", CASES)
def test_loss_of_many_samples(pkg, orc, dims, E, bf16):
    _say(f"loss dims={dims} E={E} bf16={bf16}")
    ref, run = _problem(pkg, orc, dims, 2, 16, N=E, E=E, bf16=bf16)
    want = ref.loss()
    # the fp32 bar of a sum of sqrt(K) roundings per layer, with a margin of ten
    assert abs(run.loss() - want) < 1e-5 * want, (run.loss(), want)
    run.close()


@pytest.mark.parametrize("value", [np.inf, -np.inf, 3.4e38])
def test_loss_of_a_diverged_model_is_an_error(pkg, orc, value):
    dims, E = [64, 768, 768, 10], 8192
    ref, run = _problem(pkg, orc, dims, 1, 16, N=E, E=E)
    run.X[0, 5 * 768:6 * 768] = float(value)                # one row of W_1
    second = 64 * 768 + 768
    run.X[0, second:second + 768 * 768] = 1.0               # ... that reaches every logit
    run.X[0, second + 768 * 769:run.P] = 1.0
    with pytest.raises(pkg.LcError):
        run.loss()
    run.close()
