"""The resident one-layer kernel, which selects and fetches its mini-batches itself: against the oracle where
its fetches can go wrong (row lengths and alignments, one batch in its ring and many, the last rows of the
data), for both samplers; the indices it reports.  The bars are those of test_gpu_parity.py."""
import numpy as np
import pytest

import synth
from test_gpu_parity import (TOL16, TOL32, UnitMasks, _assert_close, _check_losses, _check_workers, _force, _problem,  # noqa: F401
                             _ref_steps, _say, _xmask, pkg)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("dims,m,B", [
    ([1, 2], 3, 1),
    ([63, 16], 2, 32),      # rows at every alignment
    ([64, 10], 4, 33),
    ([130, 3], 1, 64),      # 192 padded inputs: 48 of a wavefront's lanes fetch
    ([256, 16], 3, 64),     # the ring holds one batch (fp32)
    ([200, 7], 2, 17),
])
def test_steps_and_periods(pkg, orc, dims, m, B, bf16):
    _say(f"softmax regression dims={dims} m={m} B={B} bf16={bf16}")
    tol = TOL16 if bf16 else TOL32
    ref, run = _problem(pkg, orc, dims, m, B, wd=1e-3, bf16=bf16, lr=0.05)
    assert run.resident_active()
    for tau in (1, 9):
        masks = UnitMasks()
        _ref_steps(orc, ref, 11, tau, masks)
        run.local_steps(tau)
        want = np.array([[orc.index(11, i, run.k - 1, b, 400) for b in range(B)] for i in range(m)], np.int32)
        assert np.array_equal(run.last_indices(), want)
        _check_workers(run, ref, dims, tol, f"call of {tau}", masks)   # (no gates: nothing is left out)
        _check_losses(run, ref, tol, "local losses")
        assert not run.X[:, run.P:].any() and not run.V[:, run.P:].any()
        _force(run, ref)
    masks = UnitMasks()
    for i in range(3):
        _ref_steps(orc, ref, 11, 2, masks, fresh=i == 0)
        ref.average()
    run.local_periods(2, 3)
    X, _, k = run.get_state()
    assert k == ref.k
    _assert_close(X[0], ref.X[0], dims, tol, "mean", _xmask(ref, masks.union(range(m))))
    run.close()


def test_partition_sampler(pkg, orc):
    """33 steps (two launches) over several epochs of every worker's own shard."""
    _say("softmax regression, partition sampler")
    dims, m, B, N = [24, 5], 3, 7, 100
    data, labels = synth.gaussian_mixture(3, N, dims[0], dims[-1], mean_sd=1.0)
    md = pkg.make_model(pkg.KIND_MLP, dims, B=B, N=N, E=100, lr=0.05, beta=0.9, sampler=1)
    runs = [pkg.LocalSGD(m, md, 77, synth.init_params(3, dims), data, labels) for _ in range(2)]
    runs[1].set_resident(False)
    for r in runs:
        r.local_steps(33)
    want = np.array([[orc.index_partition(77, i, 32, b, N, m, B) for b in range(B)] for i in range(m)], np.int32)
    for r in runs:
        assert np.array_equal(r.last_indices(), want)
    X = [r.get_state()[0] for r in runs]
    assert np.abs(X[0] - X[1]).max() < TOL32 * np.abs(X[1]).max()
    for r in runs:
        r.close()
