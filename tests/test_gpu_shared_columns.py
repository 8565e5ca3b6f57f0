"""Hidden layers whose columns several workgroups share out in the backward pass (few row blocks): the
shares of dA through memory, against the oracle where the shares are uneven, the rows ragged and the
batch partly padding.  The bars are those of test_gpu_parity.py."""
import pytest

from test_gpu_parity import (TOL16, TOL32, UnitMasks, _check_losses, _check_workers, _force, _problem, _ref_steps,  # noqa: F401
                             _say, pkg)

pytestmark = pytest.mark.gpu

CASES = [
    # dims, m, B
    ([50, 130, 200, 9], 3, 17),           # one chunk each
    ([40, 500, 300, 10], 16, 100),        # two shares of 3 and 2 chunks (128 samples), one or two of 2 and 1 below
    ([30, 1030, 705, 256, 12], 4, 64),    # two such layers, the scratch sized for the larger one
    ([64, 64, 1024, 7], 9, 32),           # a single row block per replica
    ([33, 70, 129, 5], 1, 128),           # three chunks, the last of one column
]


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("dims,m,B", CASES)
def test_steps(pkg, orc, dims, m, B, bf16):
    _say(f"shared columns dims={dims} m={m} B={B} bf16={bf16}")
    tol = TOL16 if bf16 else TOL32
    ref, run = _problem(pkg, orc, dims, m, B, wd=1e-3, bf16=bf16, lr=0.02, resident=False)
    for tau in (1, 2):
        masks = UnitMasks()
        _ref_steps(orc, ref, 11, tau, masks)
        run.local_steps(tau)
        _check_workers(run, ref, dims, tol, f"call of {tau}", masks, over="fail" if tau == 1 else "skip")
        _check_losses(run, ref, tol, "local losses")
        _force(run, ref)
    run.close()
