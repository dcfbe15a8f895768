"""GPU parity of the scan shapes that hold several 16-byte vectors per thread
(rows of a wave): problems shorter than a row, of one row, of some of a wave's
rows and of several waves, in the plain and the persistent kernels, with a
ragged last workgroup whose lanes must not store past the batch.

int32 and float64 on dyadic inputs: every partial sum is exact, so the result
is compared bit for bit.  The batch gives the persistent grid several groups
per workgroup.
"""
import numpy as np
import pytest

import oracle
from paper_2310_16214_amd import inputs, ppx
from tests.gpu_util import banner, to_dev, to_host

pytestmark = pytest.mark.gpu

# (values per thread, n): below a row, a row, two rows, a wave, several waves
SHAPES = {ppx.I32: [(8, 64), (8, 256), (16, 512), (32, 1024), (32, 2048), (16, 4096), (32, 16384)],
          ppx.F64: [(4, 64), (4, 128), (8, 256), (16, 512), (16, 1024), (8, 2048), (16, 16384)]}
CASES = [(dt, P, n, L) for dt, v in SHAPES.items() for P, n in v for L in (64, 256, 1024)]


@pytest.mark.parametrize("dtype,P,n,L", CASES)
def test_rows_bit_exact(cuda, dtype, P, n, L):
    import torch
    if L * P < n or L * P // n > 64:
        pytest.skip("not a launch shape")
    G = L * P // n
    batch = max(3, (1 << 23) // n) // G * G + (1 if G > 1 else 0)  # the last group has one problem
    if dtype == ppx.I32:
        x = inputs.scan_input(n, batch, np.int32, seed=n + P)
    else:
        _, x = inputs.scan_input_dyadic(n, batch, seed=n + P)
    xd = to_dev(x, cuda)
    guard = 64 * P * 16
    for excl in (False, True):
        ref = oracle.scan(x, exclusive=excl)
        for algo in (ppx.SCAN_KS, ppx.SCAN_LF, ppx.SCAN_KS_PIPE, ppx.SCAN_LF_PIPE):
            cfg = ppx.make_config(2, L, G, algo)
            assert ppx.config_valid(ppx.OP_SCAN, dtype, n, cfg)
            banner(f"scan rows dtype={dtype} n={n} batch={batch} excl={excl} {cfg}")
            buf = torch.full((batch * n + guard,), -7, dtype=xd.dtype, device=cuda)
            f = ppx.scan_exclusive_batched if excl else ppx.scan_batched
            f(xd, buf, n, batch, dtype, cfg)
            y = to_host(buf)
            assert np.array_equal(y[:batch * n].reshape(batch, n), ref), f"{cfg}: wrong values"
            assert np.all(y[batch * n:] == -7), f"{cfg}: stored past the batch"
