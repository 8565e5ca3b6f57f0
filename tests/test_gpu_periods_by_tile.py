"""Large layers whose averaging step is taken by tile: a call of whole periods against the same calls one by
one, bit for bit -- with the rows written at the end of the call only, and where the first iteration at tau = 1
has no pending broadcast to start from."""
import numpy as np
import pytest

from paper_1810_08313_amd import binding
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


def _tile_launches(run, tau, periods):
    """Launches of the tile-owner kernel in one call, by layer."""
    n = []
    for layer in (1, 2):
        run.timing_begin(binding.TIME_BWD)
        run.timing_select(layer, binding.BWD_TILE_OWNER)
        run.local_periods(tau, periods)
        n.append(run.timing_read()[0])
    run.timing_begin(binding.TIME_NONE)
    return n


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("lazy", [False, True])
@pytest.mark.parametrize("tau,periods", [(1, 1), (1, 3), (3, 1)])
@pytest.mark.parametrize("B", [20, 100])   # fragments and plain rows of the first layer's inputs
def test_hidden_layer_by_tile(pkg, orc, B, tau, periods, lazy, bf16):
    """Two layers by tile, both well above the size from which they are; the second needs the deltas of the layer
    below beforehand, from every worker's own weights where no broadcast is pending.  Against the run that writes the
    rows in every step and averages them in kernels of their own, bit for bit; which calls go by tile, by rule.  (That
    run defers its broadcast: where all workers read one model the columns are walked in another order than where
    each reads its own.)"""
    dims, m = [2048, 1280, 1792, 10], 16
    _say(f"hidden layer by tile B={B} tau={tau} n={periods} lazy={lazy} bf16={bf16}")
    runs = [_problem(pkg, orc, dims, m, B, wd=5e-4, bf16=bf16, lr=0.01)[1] for _ in range(2)]
    runs[1].set_fused_averaging(0)
    runs[1].set_deferred_update(False)
    runs[1].set_lazy_broadcast(True)
    runs[0].set_lazy_broadcast(lazy)
    for r in runs:
        r.local_steps(1)
        r.average()
        r.materialize()
        r.local_periods(tau, periods)
    F = [r.loss() for r in runs]
    assert F[0] == F[1]
    rows = runs[0].X.cpu().numpy()[:, :runs[0].P]
    for got, want in zip(runs[0].get_state(), runs[1].get_state()):
        assert np.array_equal(got, want)
    if not lazy:   # they had been there when the call returned
        assert np.array_equal(rows, runs[0].get_state()[0])
    by_tile = _tile_launches(runs[0], tau, periods)
    if lazy or periods > 1:
        assert by_tile == [periods, periods]
    elif bf16 or B == 20:   # rows written at the end of the call: one period, layer 1 only
        assert by_tile == [1, 0]
    else:                   # fp32, more than 64 samples
        assert by_tile == [0, 0]
    assert _tile_launches(runs[1], tau, periods) == [0, 0]
    for r in runs:
        r.close()
