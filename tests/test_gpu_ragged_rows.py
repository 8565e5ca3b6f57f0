"""Weight rows that are no whole number of 64-column chunks, or not 16-byte aligned, in layers of at
least 64 columns: the vector access that may run over a row's end and stops its stores there, at the
sizes where it can go wrong (one column past a chunk, one short of one, every alignment, the last
layer, a state that streams).  The bars are those of test_gpu_parity.py."""
import numpy as np
import pytest

from test_gpu_parity import (TOL16, TOL32, UnitMasks, _check_losses, _check_workers, _problem, _ref_steps,  # noqa: F401
                             _say, pkg)

pytestmark = pytest.mark.gpu

CASES = [
    # dims, m, B
    ([70, 65, 64, 66, 5], 2, 33),      # one column over a chunk; a whole chunk at an odd offset
    ([33, 127, 130, 9], 3, 64),        # one column short of two chunks; two past
    ([20, 63, 67, 65], 2, 17),         # below a chunk (checked element by element); 65 classes
    ([100, 191, 129], 2, 128),         # 129 classes, the full batch tile
    ([96, 1027, 3], 40, 100),          # enough blocks for the whole batch in one of them
    ([2000, 1501, 70], 13, 20),        # weights that stream from memory
]


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("dims,m,B", CASES)
def test_one_step_with_ragged_rows(pkg, orc, dims, m, B, bf16):
    _say(f"ragged rows dims={dims} m={m} B={B} bf16={bf16}")
    ref, run = _problem(pkg, orc, dims, m, B, wd=1e-3, bf16=bf16, resident=False)
    tol = TOL16 if bf16 else TOL32
    masks = UnitMasks()
    _ref_steps(orc, ref, 11, 1, masks)
    run.local_steps(1)
    _check_workers(run, ref, dims, tol, "one step", masks)
    _check_losses(run, ref, tol, "local losses")
    # what lies beyond a row's end belongs to others: the padding of every replica is still zero
    assert not run.X[:, run.P:].any() and not run.V[:, run.P:].any()
    run.close()


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("C,B", [(65, 1), (66, 16), (128, 17), (130, 128), (1024, 20)])
def test_softmax_over_many_classes(pkg, orc, C, B, bf16):
    _say(f"softmax C={C} B={B} bf16={bf16}")
    dims, m = [24, C], 2
    ref, run = _problem(pkg, orc, dims, m, B, bf16=bf16)
    tol = TOL16 if bf16 else TOL32
    masks = UnitMasks()
    _ref_steps(orc, ref, 11, 1, masks)
    run.local_steps(1)
    _check_workers(run, ref, dims, tol, "one step", masks)
    _check_losses(run, ref, tol, "local losses")
    ref.average()
    run.average()
    assert abs(run.loss() - ref.loss()) < TOL32 * ref.loss()
    run.close()
