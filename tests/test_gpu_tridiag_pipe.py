"""GPU parity of the persistent in-wave tridiagonal solvers over many groups
per workgroup, where a lane stores up to 128 bytes as 16-byte words: every
system of a batch that makes the grid loop, to the residual bound of the plain
kernels, with a ragged last group.
"""
import numpy as np
import pytest

import oracle
from paper_2310_16214_amd import inputs, ppx
from tests.gpu_util import banner, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,P,tol", [(np.float32, 16, 1e-4), (np.float64, 8, 1e-12), (np.float64, 16, 1e-12)])
@pytest.mark.parametrize("n", [64, 1024])
def test_persistent_many_groups(cuda, dtype, P, tol, n):
    if n // P > 64:
        pytest.skip("longer than a wave")
    import torch
    batch = (1 << 21) // n + 3
    a, b, c, d, _ = inputs.tridiag_input(n, batch, dtype, seed=n + P)
    dev = [to_dev(v, cuda) for v in (a, b, c, d)]
    dt = ppx.F32 if dtype == np.float32 else ppx.F64
    L = 256
    for algo in (ppx.TRI_CR_PCR, ppx.TRI_CR_SHFL, ppx.TRI_PCR_SHFL, ppx.TRI_PCR_REG, ppx.TRI_WM, ppx.TRI_LF):
        cfg = ppx.make_config(2, L, min(64, L * P // n), algo | ppx.TRI_PIPE)
        if not ppx.config_valid(ppx.OP_TRIDIAG, dt, n, cfg):
            continue
        banner(f"tridiag persistent {dtype.__name__} n={n} batch={batch} {cfg}")
        x = torch.empty_like(dev[3])
        ppx.tridiag_batched(*dev, x, n, batch, dt, cfg)
        r = oracle.tridiag_residual(a, b, c, d, to_host(x))
        assert r.max() <= tol, f"{cfg}: residual {r.max():.2e}"
