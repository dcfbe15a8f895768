"""GPU parity of NULL-plan large-FFT calls on batches too small to give every CU
a tile of the recorded plan, which run short columns in narrow tiles: every
size, at one problem and around the batch where the recorded plan takes over,
with the shipped plans and with none recorded, forward and inverse, against
the definition on sampled bins and Parseval on every bin.
"""
import os

import numpy as np
import pytest

import oracle
from paper_2310_16214_amd import inputs, ppx
from tests.gpu_util import banner, fft_tol, to_dev, to_host

pytestmark = pytest.mark.gpu

CACHE = os.path.join(os.path.dirname(ppx.__file__), "tuned", "mi355x.txt")


def _check(x, y, n, direction):
    rng = np.random.default_rng(n)
    ks = np.sort(rng.choice(n, 32, replace=False))
    for b in {0, x.shape[0] - 1}:
        ref = oracle.dft_bins(x[b], ks, inverse=direction > 0)
        got = y[b][ks]
        assert np.linalg.norm(got - ref) <= fft_tol(n) * np.linalg.norm(ref)
    ex = (np.abs(x.astype(np.complex128)) ** 2).sum(axis=1) * n
    ey = (np.abs(y.astype(np.complex128)) ** 2).sum(axis=1)
    assert np.all(np.abs(ey - ex) <= 2 * fft_tol(n) * ex)


@pytest.mark.parametrize("shipped", [True, False])
@pytest.mark.parametrize("ln", range(15, 23))
def test_null_plan_small_batches(cuda, ln, shipped):
    import torch
    ppx.clear_tune_cache()
    if shipped:
        ppx.load_tune_cache(CACHE)
    n = 1 << ln
    try:
        last = max(1, (1 << 21) // n)
        for k, batch in enumerate(sorted({1, last, last + 1, max(1, last // 3)})):
            direction = 1 if k % 2 else -1
            x = inputs.fft_input(n, batch, seed=ln + batch)
            buf = torch.full((batch * n + 4096,), -7, dtype=torch.complex64, device=cuda)
            banner(f"fft large n=2^{ln} batch={batch} NULL plan shipped={shipped} dir={direction}")
            ppx.fft_batched(to_dev(x, cuda), buf, n, batch, direction)
            y = to_host(buf)
            assert np.all(y[batch * n:] == -7), "stored past the batch"
            _check(x, y[:batch * n].reshape(batch, n), n, direction)
    finally:
        ppx.clear_tune_cache()
