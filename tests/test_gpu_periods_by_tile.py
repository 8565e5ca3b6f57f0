"""Large layers whose averaging step is taken by tile: a call of whole periods against the same calls one by
one, bit for bit -- with the rows written at the end of the call only, and where the first iteration at tau = 1
has no pending broadcast to start from."""
import numpy as np
import pytest

from test_gpu_parity import _problem, _say, pkg  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("lazy", [False, True])
@pytest.mark.parametrize("tau,periods", [(1, 1), (1, 3), (3, 2)])
def test_periods_against_call_by_call(pkg, orc, tau, periods, lazy, bf16):
    _say(f"periods by tile tau={tau} n={periods} lazy={lazy} bf16={bf16}")
    dims, m, B = [2048, 1024, 10], 16, 20
    runs = [_problem(pkg, orc, dims, m, B, wd=5e-4, bf16=bf16, lr=0.01)[1] for _ in range(2)]
    for r in runs:
        r.set_lazy_broadcast(lazy)
        r.local_steps(1)
        r.average()
        r.materialize()
    runs[0].local_periods(tau, periods)
    for _ in range(periods):
        runs[1].local_steps(tau)
        runs[1].average()
    if not lazy:   # the rows are there when the call returns
        assert np.array_equal(runs[0].X.cpu().numpy(), runs[1].X.cpu().numpy())
    F = [r.loss() for r in runs]
    assert F[0] == F[1]
    for got, want in zip(runs[0].get_state(), runs[1].get_state()):
        assert np.array_equal(got, want)
    assert np.array_equal(runs[0].local_losses(), runs[1].local_losses())
    for r in runs:
        r.close()
