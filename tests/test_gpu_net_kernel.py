"""Small networks of any depth with the whole model on one compute unit (net_kernel): against the
oracle at the edges of its shapes, whole periods against the call-by-call form bit for bit, and that
they need no barrier.  The bars are those of test_gpu_parity.py."""
import numpy as np
import pytest

from test_gpu_parity import (TOL16, TOL32, UnitMasks, _assert_close, _check_losses, _check_workers, _force, _problem,  # noqa: F401
                             _ref_steps, _say, _xmask, pkg)

pytestmark = pytest.mark.gpu

CASES = [
    # dims, m, B
    ([130, 70, 33, 7], 3, 48),             # ragged everywhere
    ([64, 10], 3, 128),                    # one layer, more samples than the resident kernel takes
    ([100, 64], 2, 65),                    # the most classes
    ([17, 16, 15, 33, 16, 9, 18, 20, 2], 2, 17),   # eight layers
    ([64, 32, 17], 4, 16),                 # one class over a tile
    ([1, 1, 1, 2], 5, 1),
    ([255, 32, 10], 2, 127),               # LDS nearly full
    ([400, 64, 10, 3], 1, 16),             # 25 x 4 weight tiles in the first layer
    ([20, 12, 8, 5], 300, 24),             # more replicas than compute units
]


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("dims,m,B", CASES)
def test_steps_and_average(pkg, orc, dims, m, B, bf16):
    """A call of one step and a call of three, from the oracle's state and from a pending broadcast."""
    _say(f"net kernel dims={dims} m={m} B={B} bf16={bf16}")
    ref, run = _problem(pkg, orc, dims, m, B, wd=1e-3, bf16=bf16, lr=0.05)
    assert run.resident_active()
    run.set_lazy_broadcast(True)
    tol = TOL16 if bf16 else TOL32
    for tau in (1, 3):
        masks = UnitMasks()
        _ref_steps(orc, ref, 11, tau, masks)
        run.local_steps(tau)
        _check_workers(run, ref, dims, tol, f"call of {tau}", masks, over="skip")
        _check_losses(run, ref, tol, "local losses")
        ref.average()
        run.average()
        X, _, k = run.get_state()
        assert k == ref.k
        _assert_close(X[0], ref.X[0], dims, tol, "mean", _xmask(ref, masks.union(range(m))), over="skip")
        assert not run.X[:, run.P:].any() and not run.V[:, run.P:].any()
        _force(run, ref)
        run.average()   # identical rows: exact; leaves the broadcast pending
    run.close()


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("dims,m,B,tau,periods", [([130, 70, 33, 7], 3, 48, 3, 2), ([64, 20, 17], 5, 70, 1, 9),
                                                  ([40, 24, 16, 10], 9, 16, 5, 13)])
def test_periods_against_call_by_call(pkg, orc, dims, m, B, tau, periods, bf16):
    _say(f"net kernel, periods dims={dims} tau={tau} n={periods} bf16={bf16}")
    _, run = _problem(pkg, orc, dims, m, B, wd=5e-4, bf16=bf16, lr=0.05)
    _, sep = _problem(pkg, orc, dims, m, B, wd=5e-4, bf16=bf16, lr=0.05)
    assert run.resident_active()
    run.set_resident(2)
    for lazy in (False, True):
        for r in (run, sep):
            r.set_lazy_broadcast(lazy)
            r.local_steps(2)
            r.average()
        run.local_periods(tau, periods)
        for _ in range(periods):
            sep.local_steps(tau)
            sep.average()
        for got, want in zip(run.get_state(), sep.get_state()):
            assert np.array_equal(got, want)
        assert np.array_equal(run.local_losses(), sep.local_losses())
    run.close()
    sep.close()


def test_periods_wait_for_no_other_workgroup(pkg, orc):
    """Whole periods without a barrier among the replicas: with no polls allowed (a barrier would give up
    at once and report it) they run as ever.  300 replicas cannot all be on the chip together."""
    dims, B = [20, 12, 8, 5], 24
    for m in (4, 300):
        ref, run = _problem(pkg, orc, dims, m, B)
        assert run.resident_active()
        for on in (1, 2):
            run.set_resident(on)
            run.set_barrier_polls(0)
            masks = UnitMasks()
            run.local_periods(1, 2)
            for j in range(2):
                _ref_steps(orc, ref, 11, 1, masks, fresh=j == 0)
                ref.average()
            X, _, k = run.get_state()
            assert k == ref.k
            _assert_close(X[0], ref.X[0], dims, TOL32, "mean", _xmask(ref, masks.union(range(m))), over="skip")
            _force(run, ref)
        run.close()


@pytest.mark.parametrize("dims,m,B,takes", [
    ([448, 38], 8, 112, False),            # inputs of one layer read from memory
    ([196, 20], 8, 60, True),              # ... kept in LDS
    ([320, 64, 26], 2, 64, False),         # two layers, 88 weight tiles, inputs from memory
    ([300, 64, 26], 2, 16, True),          # ... 84, kept in LDS
    ([320, 64, 26], 2, 16, False),         # 88
    ([384, 10], 4, 32, False),             # one layer, few classes
    ([128, 64, 3], 14, 128, True),         # 36 tiles, from memory
    ([468, 64, 30], 11, 24, False),
    ([607, 24, 32], 12, 32, False),        # 80 tiles, first hidden layer narrower than a column chunk
    ([304, 64, 64, 13], 4, 48, False),     # three layers, 96 tiles
    ([64, 40, 84, 20, 11], 11, 62, True),  # four layers
])
def test_shapes_that_take_one_compute_unit(pkg, orc, dims, m, B, takes):
    """The route is taken where it was measured to be the faster one (see net_shape_ok)."""
    _, run = _problem(pkg, orc, dims, m, B)
    assert run.resident_active() == takes
    run.close()
