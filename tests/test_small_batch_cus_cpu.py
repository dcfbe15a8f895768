"""CPU test of the small-batch rule on devices of other CU counts: the batch at
which it stops scales with the CUs (four SIMDs each, lines in waves per SIMD).
The rule is internal; it is called by its C++ symbol."""
import ctypes

import pytest

from paper_2310_16214_amd import ppx


def _fit(op, dtype, n, batch, cus, cfg):
    f = ppx.lib()["_ZN3ppx9fit_shapeEiilliR10ppx_config"]
    f.restype = None
    c = ppx.make_config(cfg.radix, cfg.threads_per_block, cfg.problems_per_block, cfg.algo)
    c.elems_per_thread = n * c.problems_per_block // c.threads_per_block
    f(ctypes.c_int(op), ctypes.c_int(dtype), ctypes.c_int64(n), ctypes.c_int64(batch), ctypes.c_int(cus), ctypes.byref(c))
    assert ppx.config_valid(op, dtype, n, c)
    return c.elems_per_thread


@pytest.mark.parametrize("cus", [32, 64, 128, 256, 304])
@pytest.mark.parametrize("op,dtype,n,cfg,line", [
    (ppx.OP_FFT, ppx.C64, 256, ppx.make_config(16, 128, 8, 1), 2.0),
    (ppx.OP_FFT, ppx.C64, 512, ppx.make_config(16, 128, 4, 0), 3.0),
    (ppx.OP_FFT, ppx.C64, 1024, ppx.make_config(16, 256, 4, 0), 1.0),
    (ppx.OP_FFT, ppx.C64, 2048, ppx.make_config(16, 256, 2, 0), 1.0),
    (ppx.OP_TRIDIAG, ppx.F32, 256, ppx.make_config(2, 256, 16, ppx.TRI_WM), 1.0),
    (ppx.OP_TRIDIAG, ppx.F64, 64, ppx.make_config(2, 256, 32, ppx.TRI_LF), 0.5)])
def test_line_scales_with_the_cus(op, dtype, n, cfg, line, cus):
    P = n * cfg.problems_per_block // cfg.threads_per_block
    last = int(line * 4 * cus * 64 * P) // n  # problems in `line` waves per SIMD at P values per thread
    assert _fit(op, dtype, n, last, cus, cfg) < P
    assert _fit(op, dtype, n, last + 64 * P // n + 1, cus, cfg) == P
