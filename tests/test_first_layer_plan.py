"""Which workgroups the first-layer kernel has (host only).  The launch takes the same plan, so the calls of
test_gpu_first_layer_waves.py and test_gpu_ragged_first_layer.py run the instances that are named here."""
import ctypes as C

import pytest

import paper_1810_08313_amd as pkg


def _plan(dims, m, B, bf16):
    L, h = pkg.lib(), C.c_void_p()
    md = pkg.make_model(pkg.KIND_MLP, dims, B=B, N=1000, E=64, lr=0.05, beta=0.9, bf16=bf16)
    assert L.lc_init(m, pkg.lc_param_count(md), C.byref(md), 1, C.byref(h)) == 0
    c, w = C.c_int32(-1), C.c_int32(-1)
    assert L.lc_first_layer_workgroup(h, C.byref(c), C.byref(w)) == 0
    off = C.c_int32(-1)
    assert L.lc_set_first_layer_fusion(h, 0) == 0
    assert L.lc_first_layer_workgroup(h, C.byref(off), C.byref(off)) == 0 and off.value == 0
    assert L.lc_first_layer_workgroup(h, None, C.byref(off)) == -1 and L.lc_first_layer_workgroup(None, C.byref(off), C.byref(off)) == -1
    L.lc_destroy(h)
    return c.value, w.value


@pytest.mark.parametrize("dims,m,B,bf16,plan", [
    ([256, 256, 24, 10], 48, 33, False, (64, 8)),     # fp32, up to one workgroup per compute unit
    ([257, 250, 24, 10], 64, 64, False, (64, 8)),
    ([400, 700, 24, 10], 20, 64, False, (64, 8)),
    ([400, 700, 24, 10], 23, 50, False, (64, 8)),
    ([3072, 960, 64, 10], 16, 64, False, (64, 8)),
    ([256, 256, 24, 10], 66, 33, False, (64, 4)),     # more
    ([400, 700, 24, 10], 24, 50, False, (64, 4)),
    ([255, 250, 24, 10], 64, 64, False, (64, 4)),     # a short walk
    ([256, 256, 24, 10], 48, 32, False, (64, 4)),
    ([256, 256, 24, 10], 48, 33, True, (64, 4)),
    ([97, 257, 24, 10], 85, 128, True, (96, 8)),      # a round less with chunks of 96
    ([130, 285, 24, 10], 84, 100, True, (96, 8)),
    ([64, 90, 10], 210, 70, True, (96, 8)),
    ([97, 673, 24, 10], 94, 70, True, (96, 8)),       # five become three
    ([130, 290, 24, 10], 52, 100, True, (96, 8)),     # one full round where two of 64 columns would be half empty
    ([100, 1500, 24, 10], 12, 128, True, (96, 8)),
    ([3072, 1400, 1000, 10], 16, 100, True, (96, 8)),
    ([64, 90, 10], 191, 70, True, (0, 0)),            # 191 workgroups of 96 columns
    ([1500, 1999, 1000, 10], 24, 90, True, (64, 8)),  # three would become two
    ([301, 450, 24, 10], 32, 128, True, (64, 8)),     # one round
    ([1024, 1024, 64, 10], 24, 128, True, (64, 8)),   # whole tiles
    ([1040, 1024, 64, 10], 24, 128, True, (64, 4)),   # ... not of 128 rows
    ([301, 450, 24, 10], 32, 128, False, (0, 0)),     # fp32 at 128 samples
    ([64, 63, 10], 256, 32, True, (0, 0)),
    ([256, 256, 24, 10], 47, 32, True, (0, 0)),       # 188 workgroups
])
def test_plan(dims, m, B, bf16, plan):
    assert _plan(dims, m, B, bf16) == plan
