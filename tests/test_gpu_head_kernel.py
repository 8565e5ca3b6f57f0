"""The one-workgroup kernel of a narrow last layer (forward, softmax, backward and update in one): against the
oracle at the edges of its range -- rows for some or all of its wavefronts, 1 to 64 classes and 128 samples, with
and without a layer below.  The bars are those of test_gpu_parity.py."""
import pytest

from test_gpu_parity import (TOL16, TOL32, UnitMasks, _check_losses, _check_workers, _force, _problem, _ref_steps,  # noqa: F401
                             _say, pkg)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("dims,m,B", [
    ([1, 2], 2, 1),
    ([128, 64], 2, 128),     # every wavefront has rows, every lane a class
    ([65, 17], 3, 33),
    ([30, 5, 2], 3, 7),
    ([50, 113, 33], 2, 65),  # ragged rows and classes, two of 128 padded samples' tiles empty
    ([40, 128, 64], 2, 128),
    ([40, 64, 16], 2, 32),
])
def test_steps(pkg, orc, dims, m, B, bf16):
    _say(f"narrow last layer dims={dims} m={m} B={B} bf16={bf16}")
    tol = TOL16 if bf16 else TOL32
    ref, run = _problem(pkg, orc, dims, m, B, wd=1e-3, bf16=bf16, lr=0.05, resident=False)
    assert not run.resident_active()
    for tau in (1, 2):
        masks = UnitMasks()
        _ref_steps(orc, ref, 11, tau, masks)
        run.local_steps(tau)
        _check_workers(run, ref, dims, tol, f"call of {tau}", masks, over="fail" if tau == 1 else "skip")
        _check_losses(run, ref, tol, "local losses")
        assert not run.X[:, run.P:].any() and not run.V[:, run.P:].any()
        _force(run, ref)
    run.close()


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("hidden", [33, 140])   # the one-workgroup kernel; the forward kernel's epilogue
@pytest.mark.parametrize("classes", [1, 4, 5, 16, 17])
def test_classes_per_lane(pkg, orc, classes, hidden, bf16):
    """Both kernels' softmax at the edges of its split: 1, 4 or 16 lanes per sample."""
    dims, m, B = [40, hidden, classes], 2, 45
    _say(f"softmax of {classes} classes, {hidden} hidden units, bf16={bf16}")
    tol = TOL16 if bf16 else TOL32
    ref, run = _problem(pkg, orc, dims, m, B, wd=1e-3, bf16=bf16, lr=0.05, resident=False)
    masks = UnitMasks()
    _ref_steps(orc, ref, 11, 1, masks)
    run.local_steps(1)
    _check_workers(run, ref, dims, tol, "step", masks)
    _check_losses(run, ref, tol, "local losses")
    run.close()
