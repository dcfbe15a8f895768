"""GPU parity of the CR -> PCR hybrid across waves at the sizes where its
exchanges change form: an odd and an even number of PCR steps, two waves and
sixteen, one and several systems per workgroup, solutions stored directly and
through the staging buffer, and a ragged last workgroup that must not store
past the batch.  Boundary coefficients are NaN, and one system is singular:
its neighbours in the workgroup must not notice.
"""
import numpy as np
import pytest

import oracle
from paper_2310_16214_amd import inputs, ppx
from tests.gpu_util import banner, to_dev, to_host, tridiag_forward_check

pytestmark = pytest.mark.gpu

# (values per thread, n, threads per workgroup)
SHAPES = [(2, 256, 128), (2, 2048, 1024), (4, 1024, 256), (4, 1024, 1024), (8, 1024, 128), (8, 2048, 1024),
          (8, 8192, 1024), (16, 2048, 128), (16, 2048, 512), (16, 8192, 512)]


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("P,n,L", SHAPES + [(16, 16384, 1024)])
def test_hybrid_across_waves(cuda, dtype, P, n, L):
    import torch
    dt = ppx.F32 if dtype == np.float32 else ppx.F64
    G = L * P // n
    cfg = ppx.make_config(2, L, G, ppx.TRI_CR_PCR)
    if not ppx.config_valid(ppx.OP_TRIDIAG, dt, n, cfg):
        pytest.skip("not a launch shape")
    batch = 4 * G + 1
    a, b, c, d, _ = inputs.tridiag_input(n, batch, dtype, seed=n + P)
    ref = oracle.thomas(a, b, c, d)
    a[:, 0] = np.nan
    c[:, -1] = np.nan
    bad = 1
    b[bad, n // 2] = 0.0
    a[bad, n // 2] = c[bad, n // 2] = 0.0
    dev = [to_dev(v, cuda) for v in (a, b, c, d)]
    guard = 4096
    x = torch.full((batch * n + guard,), -7.0, dtype=dev[3].dtype, device=cuda)
    banner(f"tridiag across waves {dtype.__name__} n={n} batch={batch} {cfg}")
    ppx.tridiag_batched(*dev, x, n, batch, dt, cfg)
    y = to_host(x)
    assert np.all(y[batch * n:] == -7.0), "stored past the batch"
    keep = np.arange(batch) != bad
    y = y[:batch * n].reshape(batch, n)[keep]
    a, b, c, d, ref = (v[keep] for v in (a, b, c, d, ref))
    a[:, 0] = c[:, -1] = 0
    tol = 1e-4 if dtype == np.float32 else 1e-12
    r = oracle.tridiag_residual(a, b, c, d, y)
    assert r.max() <= tol, f"residual {r.max():.2e}"
    err, bound = tridiag_forward_check(a, b, c, d, y, ref)
    assert np.all(err <= bound)
