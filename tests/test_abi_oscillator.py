"""Arguments of mpdata_osc_step are checked before any path is chosen (no GPU
needed): a missing advector, one of a dimension the plan does not have, or a G
that does not match the plan is refused, on the short lines that one workgroup
holds, on longer ones and in two dimensions alike."""
import ctypes

import pytest

from paper_1407_1309_amd import mpdata
from tests.test_abi import _desc

X = ctypes.c_void_p(4096)     # never followed: every call below is refused
Y = ctypes.c_void_p(8192)


@pytest.mark.parametrize("shape", [(500,), (9001,), (20, 30)])
@pytest.mark.parametrize("kernel", [mpdata.KERNEL_AUTO, mpdata.KERNEL_STAGED])
@pytest.mark.parametrize("has_g", [0, 1])
def test_oscillator_refuses_bad_arguments(shape, kernel, has_g):
    L = mpdata.lib()
    d = _desc(shape, has_g=has_g)
    need = L.mpdata_workspace_bytes(ctypes.byref(d))
    h = ctypes.c_void_p()
    assert L.mpdata_init(ctypes.byref(d), ctypes.c_void_p(256), need, None,
                         ctypes.byref(h)) == mpdata.OK
    try:
        assert L.mpdata_set_kernel(h, kernel) == mpdata.OK
        nd = len(shape)
        c = [X if k < nd else None for k in range(3)]
        g = X if has_g else None
        for bad in range(3):
            w = list(c)
            w[bad] = None if bad < nd else X
            assert L.mpdata_osc_step(h, X, Y, g, *w, 0.1, 3) == mpdata.EINVAL, bad
        assert L.mpdata_osc_step(h, X, Y, None if has_g else X, *c, 0.1, 3) == mpdata.EINVAL
        # nothing to do is still no error
        assert L.mpdata_osc_step(h, X, Y, g, *c, 0.1, 0) == mpdata.OK
    finally:
        L.mpdata_destroy(h)
