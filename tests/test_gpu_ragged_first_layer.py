"""The first-layer kernel with the next step's forward pass in it, on layers whose rows or height are
no whole number of tiles: calls of two and four steps against the oracle, and one step less of them
from a pending broadcast.  The bars are those of test_gpu_parity.py."""
import pytest

from test_gpu_parity import (TOL16, TOL32, UnitMasks, _assert_close, _check_losses, _check_workers, _force, _problem,  # noqa: F401
                             _ref_steps, _say, _xmask, pkg)

pytestmark = pytest.mark.gpu

CASES = [
    # dims, m, B
    ([97, 129, 24, 10], 64, 30),       # one column over two chunks, one row over six steps; unaligned rows
    ([79, 190, 10], 64, 64),           # two columns short of three chunks, one row short of five steps
    ([64, 100, 10], 96, 33),           # whole steps, a ragged chunk
    ([200, 512, 24, 10], 32, 100),     # whole chunks, 200 rows: a last round of the 128-sample kernel with idle wavefronts
    ([301, 450, 24, 10], 32, 128),     # 128-sample kernel, everything ragged
    ([130, 65, 10], 96, 120),          # the narrowest layer it takes
]


@pytest.mark.parametrize("implicit", [0, 2])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("dims,m,B", CASES)
def test_calls_of_several_steps(pkg, orc, dims, m, B, bf16, implicit):
    _say(f"ragged first layer dims={dims} m={m} B={B} bf16={bf16} implicit={implicit}")
    tol = TOL16 if bf16 else TOL32
    ref, run = _problem(pkg, orc, dims, m, B, wd=5e-4, bf16=bf16, lr=0.05, resident=False)
    run.set_implicit_momentum(implicit)
    run.set_lazy_broadcast(True)
    for tau in (2, 4, 3):
        masks = UnitMasks()
        _ref_steps(orc, ref, 11, tau, masks)
        run.local_steps(tau)
        _check_workers(run, ref, dims, tol, f"call of {tau}", masks, over="skip")
        _check_losses(run, ref, tol, f"local losses, call of {tau}")
        assert not run.X[:, run.P:].any() and not run.V[:, run.P:].any()
        ref.average()
        run.average()
        X, _, _ = run.get_state()
        _assert_close(X[0], ref.X[0], dims, tol, f"mean after {tau}", _xmask(ref, masks.union(range(m))), over="skip")
        _force(run, ref)
        run.average()   # leaves the broadcast pending: the next call starts from the one model
    run.close()
