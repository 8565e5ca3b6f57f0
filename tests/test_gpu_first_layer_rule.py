"""Which first layers run their backward pass and the next step's forward pass as one kernel.  The fused form
sums up in another order, so the same steps with the fusion switched off tell: other bits, it was taken."""
import numpy as np
import pytest

import synth
from test_gpu_parity import _say, pkg  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,m,B,bf16,taken", [
    ([1024, 256, 10], 47, 32, False, False),       # 188 workgroups: too few
    ([1024, 256, 10], 48, 32, False, True),        # 192: one round
    ([1280, 704, 64, 10], 27, 32, True, True),     # two rounds, 58 % full (604 us for 5 steps apart, 538 as one)
    ([1000, 700, 64, 10], 27, 32, False, True),    # ... of ragged rows, state cached
    ([784, 960, 64, 10], 18, 64, False, True),     # 53 %
    ([2080, 700, 64, 10], 26, 48, True, False),    # 56 %, ragged rows that stream
    ([1000, 1344, 64, 10], 13, 128, True, False),  # 53 %, 128 samples
    ([1024, 1024, 64, 10], 24, 128, True, True),   # 75 %
    ([1000, 1024, 64, 10], 24, 100, True, False),  # ... of ragged rows, state cached
])
def test_route(pkg, dims, m, B, bf16, taken):
    _say(f"first layer dims={dims} m={m} B={B} bf16={bf16}")
    N = 300
    data, labels = synth.gaussian_mixture(5, N, dims[0], dims[-1], mean_sd=1.0)
    if bf16:
        data = synth.bf16_representable(data)
    x1, out = synth.init_params(5, dims), []
    for on in (True, False):
        run = pkg.LocalSGD(m, pkg.make_model(pkg.KIND_MLP, dims, B=B, N=N, E=64, lr=0.01, beta=0.9, bf16=bf16), 5, x1, data, labels)
        run.set_resident(False)
        run.set_first_layer_fusion(on)
        run.local_steps(2)
        out.append(run.X[:, :run.P].cpu().numpy())
        run.close()
    assert np.isfinite(out[0]).all()
    assert np.array_equal(out[0], out[1]) == (not taken)
