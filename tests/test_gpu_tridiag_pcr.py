"""GPU parity of the in-wave PCR solvers where their exchanges change: n / P
from one lane (no step beyond the lane) over two (the first step between lanes
is also the last) to a whole wave, with several systems in a wave.  The
neighbour rows come by moves that cross the border of a system, so every other
system is also replaced by NaNs: the rest must keep every bit.
"""
import numpy as np
import pytest

import oracle
from paper_2310_16214_amd import inputs, ppx
from tests.gpu_util import banner, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,tol", [(np.float32, 1e-4), (np.float64, 1e-12)])
@pytest.mark.parametrize("lanes", [1, 2, 4, 32, 64])
def test_pcr_lanes(cuda, dtype, tol, lanes):
    import torch
    dt = ppx.F32 if dtype == np.float32 else ppx.F64
    L = min(256, 64 * lanes)
    tried = 0
    for P in (2, 4, 8, 16):
        n = P * lanes
        batch = 4 * L // lanes + 3  # several workgroups, a ragged last one
        a, b, c, d, _ = inputs.tridiag_input(n, batch, dtype, seed=n + P)
        dev = [to_dev(v, cuda) for v in (a, b, c, d)]
        poisoned = [v.clone() for v in dev]
        for v in poisoned:
            v.view(batch, n)[1::2] = float("nan")
        for algo in (ppx.TRI_PCR_SHFL, ppx.TRI_PCR_REG):
            for pipe in (0, ppx.TRI_PIPE):
                cfg = ppx.make_config(2, L, L // lanes, algo | pipe)
                if not ppx.config_valid(ppx.OP_TRIDIAG, dt, n, cfg):
                    continue
                banner(f"tridiag pcr {dtype.__name__} n={n} batch={batch} {cfg}")
                tried += 1
                x, y = torch.empty_like(dev[3]), torch.empty_like(dev[3])
                ppx.tridiag_batched(*dev, x, n, batch, dt, cfg)
                r = oracle.tridiag_residual(a, b, c, d, to_host(x))
                assert r.max() <= tol, f"{cfg}: residual {r.max():.2e}"
                ppx.tridiag_batched(*poisoned, y, n, batch, dt, cfg)
                assert torch.equal(x.view(batch, n)[0::2], y.view(batch, n)[0::2]), f"{cfg}"
    assert tried >= 4
