"""GPU parity of NULL-config calls on small batches with the shipped tune cache:
fewer problems per workgroup than the tuned shape leave every bit as the
resolved configuration gives it, and a persistent shape with one group per
workgroup (which runs as the plain kernel) stays within the operation's bound.
"""
import os

import numpy as np
import pytest

import oracle
from paper_2310_16214_amd import inputs, ppx
from tests.gpu_util import banner, fft_tol, scan_bound, to_dev, to_host

pytestmark = pytest.mark.gpu

CACHE = os.path.join(os.path.dirname(ppx.__file__), "tuned", "mi355x.txt")
BATCHES = [1, 2, 5, 33, 300, 1025]
PIPE = {ppx.OP_FFT: 2, ppx.OP_SCAN: 2, ppx.OP_TRIDIAG: 8}


@pytest.fixture(scope="module")
def tuned():
    ppx.clear_tune_cache()
    ppx.load_tune_cache(CACHE)
    yield
    ppx.clear_tune_cache()


@pytest.mark.parametrize("op,dtype", [(ppx.OP_FFT, np.complex64), (ppx.OP_SCAN, np.float32), (ppx.OP_SCAN, np.int32),
                                      (ppx.OP_SCAN, np.float64), (ppx.OP_TRIDIAG, np.float32),
                                      (ppx.OP_TRIDIAG, np.float64)])
@pytest.mark.parametrize("ln", range(4, 15))
def test_null_call(cuda, tuned, op, dtype, ln):
    import torch
    n = 1 << ln
    code = {np.complex64: ppx.C64, np.float32: ppx.F32, np.int32: ppx.I32, np.float64: ppx.F64}[dtype]
    if op == ppx.OP_TRIDIAG and dtype == np.float64 and n > 8192:
        pytest.skip("no solver")
    for batch in [b for b in BATCHES if b * n <= 1 << 20]:
        cfg = ppx.resolve_config(op, code, n, batch)
        banner(f"small batch op={op} {np.dtype(dtype).name} n={n} batch={batch} {cfg}")
        if op == ppx.OP_FFT:
            x = inputs.fft_input(n, batch, seed=n + batch)
            dev = [to_dev(x, cuda)]
            call = lambda o, c: ppx.fft_batched(dev[0], o, n, batch, 1, c)  # noqa: E731
        elif op == ppx.OP_SCAN:
            x = inputs.scan_input(n, batch, dtype, seed=n + batch)
            dev = [to_dev(x, cuda)]
            call = lambda o, c: ppx.scan_batched(dev[0], o, n, batch, code, c)  # noqa: E731
        else:
            x = inputs.tridiag_input(n, batch, dtype, seed=n + batch)[:4]
            dev = [to_dev(v, cuda) for v in x]
            call = lambda o, c: ppx.tridiag_batched(*dev, o, n, batch, code, c)  # noqa: E731
        guard = 1 << 16
        buf = torch.full((batch * n + guard,), -7, dtype=dev[-1].dtype, device=cuda)
        call(buf, None)
        y = to_host(buf)
        assert np.all(y[batch * n:] == -7), "stored past the batch"
        y = y[:batch * n].reshape(batch, n)
        if not cfg.algo & PIPE[op]:
            ref = torch.empty(batch, n, dtype=dev[-1].dtype, device=cuda)
            call(ref, cfg)
            assert np.array_equal(to_host(ref).view(np.uint8), y.view(np.uint8)), cfg
        if batch > 33:
            continue
        if op == ppx.OP_FFT:
            assert oracle.rel_l2(y, oracle.dft(x, inverse=True)).max() <= fft_tol(n)
        elif op == ppx.OP_TRIDIAG:
            assert oracle.tridiag_residual(*x, y).max() <= (1e-4 if dtype == np.float32 else 1e-12)
        elif dtype == np.int32:
            assert np.array_equal(y, oracle.scan(x))
        else:
            unit = 2.0 ** -24 if dtype == np.float32 else 2.0 ** -53
            assert np.all(np.abs(y - oracle.scan(x)) <= scan_bound(x, unit, oracle_unit=2.0 ** -53))


@pytest.mark.parametrize("n,mi", [(256, 2), (512, 3), (1024, 1), (2048, 1)])
def test_null_fft_around_the_lines(cuda, tuned, n, mi):
    """Whole calls with one problem less and one more than the mi * 2^20
    elements where the rule changes the configuration: both sides within the
    FFT's bound on sampled problems, and nothing stored past the batch."""
    import torch
    seen = set()
    for batch in [(mi << 20) // n - 1, (mi << 20) // n + 1]:
        seen.add(ppx.resolve_config(ppx.OP_FFT, ppx.C64, n, batch).as_tuple())
        banner(f"null fft n={n} batch={batch}")
        g = torch.Generator(device=cuda).manual_seed(n + batch)
        x = torch.view_as_complex(torch.rand(batch, n, 2, generator=g, device=cuda) * 2 - 1)
        buf = torch.full((batch * n + 4096,), -7, dtype=x.dtype, device=cuda)
        ppx.fft_batched(x, buf, n, batch, -1)
        assert bool((buf[batch * n:] == -7).all()), "stored past the batch"
        pick = [0, 1, batch // 3, batch // 2, batch - 2, batch - 1]
        got = to_host(buf[:batch * n].view(batch, n)[pick].contiguous())
        assert oracle.rel_l2(got, oracle.dft(to_host(x[pick].contiguous()))).max() <= fft_tol(n)
    assert len(seen) == 2
