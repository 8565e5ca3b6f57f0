"""Workgroups of the first-layer kernel: eight wavefronts (fp32 operands, 33 to 64 samples, one workgroup per compute
unit) and chunks of 96 columns.  Calls of two to four steps against the oracle, with the bars of test_gpu_parity.py."""
import numpy as np
import pytest

import synth
from test_gpu_parity import _say, pkg  # noqa: F401
from test_gpu_ragged_first_layer import test_calls_of_several_steps as _calls

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,m,B", [
    ([256, 256, 24, 10], 48, 33),    # two steps of the walk for every wavefront, the fewest workgroups
    ([257, 250, 24, 10], 64, 64),    # one row in a last step of one wavefront, ragged chunks, 256 workgroups
    ([400, 700, 24, 10], 20, 64),    # 25 steps
])
def test_calls_of_several_steps_with_eight_wavefronts(pkg, orc, dims, m, B):
    _calls(pkg, orc, dims, m, B, False, 0)


@pytest.mark.parametrize("implicit", [0, 2])
@pytest.mark.parametrize("dims,m,B", [
    ([97, 257, 24, 10], 85, 128),    # 65 columns in a last chunk of 96, one row in a last step
    ([130, 285, 24, 10], 84, 100),   # three short of whole chunks
    ([64, 90, 10], 210, 70),         # one chunk, two columns of a lane missing
])
def test_chunks_of_96_columns(pkg, orc, dims, m, B, implicit):
    """bf16 operands, 65 to 128 samples, ragged rows: one round of workgroups instead of two."""
    _calls(pkg, orc, dims, m, B, True, implicit)


@pytest.mark.parametrize("dims,few,many,B", [
    ([256, 256, 24, 10], 48, 66, 33),      # whole tiles: 192 and 264 workgroups
    ([257, 250, 24, 10], 64, 65, 64),      # ragged rows, one row in the last step: 256 and 260
    ([400, 700, 24, 10], 23, 24, 50),      # 253 and 264
    ([3072, 960, 64, 10], 16, 32, 64),     # 240 and 480, a state that streams; both start from one model (exact mean: powers of two)
])
def test_a_worker_does_not_depend_on_how_many_there_are(pkg, dims, few, many, B):
    """fp32 operands, 33 to 64 samples: whether a launch has a workgroup per compute unit (eight wavefronts) or more (four) decides
    how the work is shared out, and not in which order a sum is formed: the same bits."""
    _say(f"first layer dims={dims} workers={few},{many} B={B}")
    N = 300
    data, labels = synth.gaussian_mixture(5, N, dims[0], dims[-1], mean_sd=1.0)
    x1, out = synth.bf16_representable(synth.init_params(5, dims)), []
    for m in (few, many):
        run = pkg.LocalSGD(m, pkg.make_model(pkg.KIND_MLP, dims, B=B, N=N, E=64, lr=0.01, beta=0.9), 5, x1, data, labels)
        if few == 16:
            run.set_lazy_broadcast(True)
            run.average()
        run.local_steps(4)
        out.append((run.X[:few, :run.P].cpu().numpy(), run.V[:few, :run.P].cpu().numpy()))
        run.close()
    assert np.isfinite(out[0][0]).all()
    for a, b in zip(*out):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("dims,m,B", [
    ([97, 673, 24, 10], 94, 70),     # five rounds become three; 96 columns reach 64 past the padded 704 of the deltas, 31 of the last 32 do not exist
    ([130, 290, 24, 10], 52, 100),   # two become one, which 64 columns would have filled to a half; ... past 320
    ([100, 1500, 24, 10], 12, 128),  # 192 workgroups
])
def test_last_chunks_of_96_columns_past_the_padding(pkg, orc, dims, m, B):
    _calls(pkg, orc, dims, m, B, True, 2)
