"""Which hidden layers have their columns shared out among workgroups in the backward pass, read off the
scratch the shares need (host only)."""
import ctypes as C

import pytest

import paper_1810_08313_amd as pkg


def _bytes(dims, m, B, bf16):
    L, h = pkg.lib(), C.c_void_p()
    md = pkg.make_model(pkg.KIND_MLP, dims, B=B, N=1000, E=64, bf16=bf16)
    assert L.lc_init(m, pkg.lc_param_count(md), C.byref(md), 1, C.byref(h)) == 0
    n = L.lc_workspace_bytes(h)
    L.lc_destroy(h)
    return n


@pytest.mark.parametrize("d2,m,B,bf16,shared", [
    (192, 24, 128, False, False),   # a second round of workgroups: nothing saved (103 -> 118 us a step with shares)
    (448, 24, 128, True, False),    # (73 -> 83)
    (130, 16, 64, True, False),     # two chunks saved, less than adding up costs
    (256, 12, 32, True, False),
    (300, 16, 100, False, True),
    (256, 8, 64, False, True),
    (1024, 4, 64, True, True),
    (1024, 4, 128, False, True),
])
def test_shares(d2, m, B, bf16, shared):
    """From 256 row blocks on (32 workers of a 512-unit layer) nothing is shared out and the scratch grows by the
    same amount per worker; what a smaller run needs beyond that line are its shares."""
    dims = [64, 512, d2, 10]
    a, b = _bytes(dims, 32, B, bf16), _bytes(dims, 40, B, bf16)
    line = a - (b - a) // 8 * (32 - m)
    one = 4 * m * 512 * (32 if B <= 32 else 64 if B <= 64 else 128)   # one share of dA
    extra = _bytes(dims, m, B, bf16) - line
    if shared:
        assert extra > 1.9 * one
    else:
        assert abs(extra) < 0.05 * one
