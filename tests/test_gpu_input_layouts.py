"""Mini-batches in plain rows and in fragment order: a handle whose batches of 65 to 128 samples fill a block each
takes the one for single steps and the other for periods whose first layer runs a step ahead.  Calls of both kinds
in turn against the oracle, at the bars of test_gpu_parity.py; 31 workers are too few for that and always have
fragments."""
import pytest

from test_gpu_parity import (TOL16, TOL32, UnitMasks, _check_losses, _check_workers, _force, _ref_steps, _problem,  # noqa: F401
                             _say, pkg)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("dims,m,B", [
    ([100, 512, 24, 10], 32, 120),
    ([300, 200, 10], 64, 65),
    ([67, 132, 10], 86, 128),      # ragged rows of both operands; 258 blocks
    ([100, 512, 24, 10], 31, 120),
    ([40, 200, 512, 10], 32, 100),  # a hidden layer, and below the last layer, read from the feature-major copy
    ([30, 150, 10], 256, 70),
])
def test_calls_of_both_kinds(pkg, orc, dims, m, B, bf16):
    _say(f"input layouts dims={dims} m={m} B={B} bf16={bf16}")
    tol = TOL16 if bf16 else TOL32
    ref, run = _problem(pkg, orc, dims, m, B, wd=1e-3, bf16=bf16, lr=0.02, resident=False)
    for tau in (1, 2, 1):
        masks = UnitMasks()
        _ref_steps(orc, ref, 11, tau, masks)
        run.local_steps(tau)
        _check_workers(run, ref, dims, tol, f"call of {tau}", masks)
        _check_losses(run, ref, tol, "local losses")
        _force(run, ref)
    run.close()
