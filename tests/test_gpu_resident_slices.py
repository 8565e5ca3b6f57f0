"""The resident two-layer kernel at the edges of its split: numbers of 16-unit slices that fill no column
chunk, one slice (nothing to exchange), batches at the edges of its tiles, more replicas than one per XCD and
more than the XCDs hold apart (exchange through device memory).  The bars are those of test_gpu_parity.py."""
import numpy as np
import pytest

from test_gpu_parity import (TOL16, TOL32, UnitMasks, _assert_close, _check_losses, _check_workers, _force, _problem,  # noqa: F401
                             _ref_steps, _say, _xmask, pkg)

pytestmark = pytest.mark.gpu

CASES = [
    # dims, m, B
    ([33, 16, 2], 1, 1),
    ([65, 17, 16], 3, 16),        # 2 slices, the last with one unit
    ([130, 47, 5], 9, 33),        # 3 slices, replicas 0 and 8 on one XCD
    ([31, 130, 10], 20, 17),      # 9 slices, three replicas on an XCD
    ([48, 190, 7], 21, 64),       # 12 slices, 36 workgroups would go to one XCD: exchange through device memory
    ([1024, 250, 3], 2, 49),      # the widest
]


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("dims,m,B", CASES)
def test_steps_and_average(pkg, orc, dims, m, B, bf16):
    _say(f"resident slices dims={dims} m={m} B={B} bf16={bf16}")
    ref, run = _problem(pkg, orc, dims, m, B, wd=1e-3, bf16=bf16, lr=0.05)
    assert run.resident_active()
    if dims[1] == 190:
        assert not run.xcd_local_exchange_active()
    run.set_lazy_broadcast(True)
    tol = TOL16 if bf16 else TOL32
    for tau in (1, 3):
        masks = UnitMasks()
        _ref_steps(orc, ref, 11, tau, masks)
        run.local_steps(tau)
        _check_workers(run, ref, dims, tol, f"call of {tau}", masks, over="fail" if tau == 1 else "skip")
        _check_losses(run, ref, tol, "local losses")
        ref.average()
        run.average()
        X, _, k = run.get_state()
        assert k == ref.k
        _assert_close(X[0], ref.X[0], dims, tol, "mean", _xmask(ref, masks.union(range(m))), over="fail" if tau == 1 else "skip")
        assert not run.X[:, run.P:].any() and not run.V[:, run.P:].any()
        _force(run, ref)
        run.average()   # identical rows: exact; leaves the broadcast pending
    run.close()


@pytest.mark.parametrize("dims,m,B", [CASES[2], CASES[3]])
def test_both_exchanges_give_the_same_bits(pkg, orc, dims, m, B):
    runs = [_problem(pkg, orc, dims, m, B, wd=5e-4, lr=0.05)[1] for _ in range(2)]
    runs[1].set_xcd_local_exchange(False)
    if not runs[0].xcd_local_exchange_active():
        pytest.skip("blocks are not dealt to the XCDs in turn here: there is one exchange only")
    assert not runs[1].xcd_local_exchange_active()
    for r in runs:
        r.local_steps(33)   # two launches
    for got, want in zip(runs[0].get_state(), runs[1].get_state()):
        assert np.array_equal(got, want)
    for r in runs:
        r.close()
