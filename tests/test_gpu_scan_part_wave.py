"""GPU parity of scans in workgroups of less than a wave: every accepted
workgroup size below 64 threads, at every number of values per thread, from
one problem per workgroup to the most it takes, with a ragged last workgroup.

int32 and float64 on dyadic inputs, where every partial sum is exact and the
result is compared bit for bit; float32 within the definition's bound.
"""
import numpy as np
import pytest

import oracle
from paper_2310_16214_amd import inputs, ppx
from tests.gpu_util import banner, scan_bound, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [ppx.I32, ppx.F32, ppx.F64])
@pytest.mark.parametrize("L", [1, 2, 4, 8, 16, 32])
def test_part_of_a_wave(cuda, dtype, L):
    import torch
    ran = 0
    for P in (2, 4, 8, 16, 32):
        for n in (16, 32, 64, 128, 256, 512, 1024):
            G = L * P // n
            if L * P < n or G > 64 or P > n:
                continue
            cfg = ppx.make_config(2, L, G, ppx.SCAN_KS)
            if not ppx.config_valid(ppx.OP_SCAN, dtype, n, cfg):
                continue
            batch = 5 * G + (1 if G > 1 else 0)  # the last workgroup has one problem
            if dtype == ppx.I32:
                x = inputs.scan_input(n, batch, np.int32, seed=n + P)
            elif dtype == ppx.F32:
                x = inputs.scan_input(n, batch, np.float32, seed=n + P)
            else:
                _, x = inputs.scan_input_dyadic(n, batch, seed=n + P)
            xd = to_dev(x, cuda)
            for excl in (False, True):
                ref = oracle.scan(x, exclusive=excl)
                for algo in (ppx.SCAN_KS, ppx.SCAN_LF, ppx.SCAN_KS_PIPE, ppx.SCAN_LF_PIPE):
                    cfg = ppx.make_config(2, L, G, algo)
                    banner(f"scan part wave dtype={dtype} n={n} batch={batch} excl={excl} {cfg}")
                    buf = torch.full((batch * n + 4096,), -7, dtype=xd.dtype, device=cuda)
                    f = ppx.scan_exclusive_batched if excl else ppx.scan_batched
                    f(xd, buf, n, batch, dtype, cfg)
                    y = to_host(buf)
                    assert np.all(y[batch * n:] == -7), f"{cfg}: stored past the batch"
                    y = y[:batch * n].reshape(batch, n)
                    if dtype == ppx.F32:
                        assert np.all(np.abs(y - ref) <= scan_bound(x, 2.0 ** -24, exclusive=excl)), f"{cfg}: wrong values"
                    else:
                        assert np.array_equal(y, ref), f"{cfg}: wrong values"
                    ran += 1
    assert ran
