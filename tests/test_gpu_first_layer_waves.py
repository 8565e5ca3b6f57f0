"""Workgroups of the first-layer kernel: eight wavefronts (fp32 operands, 33 to 64 samples, one workgroup per compute
unit) and chunks of 96 columns.  Calls of two to four steps against the oracle, with the bars of test_gpu_parity.py."""
import pytest

from test_gpu_parity import pkg  # noqa: F401
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
