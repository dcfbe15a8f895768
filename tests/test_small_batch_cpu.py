"""CPU tests of the rule that fits a tuned configuration to a small batch
(ppx_resolve_config with the shipped tune cache): what it may change, where it
may not, and that every configuration it gives is a valid launch."""
import os

import pytest

from paper_2310_16214_amd import ppx

CACHE = os.path.join(os.path.dirname(ppx.__file__), "tuned", "mi355x.txt")
WAVES = 1024  # a wave per SIMD
IN_WAVE = (ppx.TRI_WM, ppx.TRI_LF)
LIGHT = {256: 2, 512: 3, 1024: 1, 2048: 1}  # waves per SIMD up to which an FFT takes radix 8


@pytest.fixture(scope="module", autouse=True)
def tuned():
    ppx.clear_tune_cache()
    ppx.load_tune_cache(CACHE)
    yield
    ppx.clear_tune_cache()


SPACE = ([(ppx.OP_FFT, ppx.C64)] + [(ppx.OP_SCAN, d) for d in (ppx.I32, ppx.F32, ppx.F64)]
         + [(ppx.OP_TRIDIAG, d) for d in (ppx.F32, ppx.F64)])


@pytest.mark.parametrize("op,dtype", SPACE)
def test_fitted_configurations(op, dtype):
    for ln in range(4, 15):
        n = 1 << ln
        if op == ppx.OP_TRIDIAG and dtype == ppx.F64 and n > 8192:
            continue  # no solver
        full = ppx.resolve_config(op, dtype, n, 1 << 24)
        if ppx.tuned_config(op, dtype, n) is None and op != ppx.OP_TRIDIAG:
            continue  # no entry: the analytical choice, not this rule
        if op == ppx.OP_TRIDIAG and all(ppx.tuned_config(op, dtype, n, a) is None for a in range(8)):
            continue
        for batch in [1, 2, 3, 5, 7, 64, 100, 255, 1000, 2050, 4097, 8200, 16384, 65536, 1 << 20]:
            c = ppx.resolve_config(op, dtype, n, batch)
            what = (op, dtype, n, batch, c, full)
            assert ppx.config_valid(op, dtype, n, c), what
            assert c.algo == full.algo and c.elems_per_thread * c.threads_per_block == n * c.problems_per_block, what
            if c.as_tuple() == full.as_tuple():
                continue
            waves = -(-n * batch // (full.elems_per_thread * 64))
            if op == ppx.OP_FFT:
                assert (full.radix, full.elems_per_thread) == (16, 16) and waves <= LIGHT[n] * WAVES, what
                assert (c.radix, c.elems_per_thread) == (8, 8), what
            else:
                assert op == ppx.OP_TRIDIAG and (full.algo & ~ppx.TRI_PIPE) in IN_WAVE and waves <= WAVES, what
                assert 4 <= c.elems_per_thread < full.elems_per_thread and n // c.elems_per_thread <= 64, what


def test_explicit_entry_of_another_shape_is_kept(tmp_path):
    plain = ppx.default_config(ppx.OP_FFT, ppx.C64, 1024)
    path = tmp_path / "cache.txt"
    path.write_text("gfx950 %d %d 1024 -1 %d %d %d %d %d %d 100.0 0\n" % ((ppx.OP_FFT, ppx.C64) + plain.as_tuple()))
    ppx.load_tune_cache(str(path))
    try:
        assert ppx.resolve_config(ppx.OP_FFT, ppx.C64, 1024, 1).as_tuple() == plain.as_tuple()
    finally:
        ppx.load_tune_cache(CACHE)
