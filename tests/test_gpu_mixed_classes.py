"""GPU tests of the mixed launch's class kernels (the tiles of several families
in one kernel): every job's output has the bits of the single call with the
configuration ppx_mixed_tile_config reports, in launches that put every member
of a class into its kernel, that hold more records than a class kernel takes,
and whose largest family is past the limit and keeps its own kernel.
"""
import numpy as np
import pytest

from paper_2310_16214_amd import inputs, ppx
from tests.gpu_util import banner, to_dev, to_host

pytestmark = pytest.mark.gpu

F, S, T = "fft", "scan", "tri"
SMALL = [(F, 64, 33), (F, 1024, 7), (S, 128, 41), (S, 1024, 5), (T, 32, 29), (T, 64, 17), (T, 1024, 9)]
LARGE = [(F, 8192, 3), (F, 16384, 2), (S, 4096, 5), (S, 16384, 3), (T, 4096, 3), (T, 8192, 2), (T, 16384, 2)]
LAUNCHES = {
    "small": SMALL,
    "large": LARGE,
    "both": SMALL + LARGE,
    # 30 + 30 records of two families of one class: more than its kernel takes
    "records": [(S, 64, 3 + k) for k in range(30)] + [(F, 128, 2 + k) for k in range(30)] + [(T, 32, 5), (T, 64, 5)],
    # one family with far more tiles than the limit, next to small ones
    # small families over more than one of the larger workgroups' tiles, ragged
    "all": [(F, 16, 300), (F, 64, 70), (F, 512, 19), (F, 4096, 5), (S, 16, 1030), (S, 256, 33), (T, 16, 1027), (T, 64, 67),
            (T, 512, 19)] + LARGE,
    # small FFTs past their share of the kernel of both classes
    "all-limit": [(F, 1024, 1100), (T, 64, 67)] + LARGE,
    # a small family past the limit of its own class
    "small-limit": SMALL + [(S, 64, 140001)],
    "limit": SMALL + [(S, 64, 60001), (F, 16384, 600), (T, 8192, 1), (S, 16384, 1)],
}


@pytest.mark.parametrize("name", sorted(LAUNCHES))
def test_class_launch_bits(cuda, name):
    import torch
    jobs, outs, calls = [], [], []
    for k, (op, n, batch) in enumerate(LAUNCHES[name]):
        if op == F:
            x = to_dev(inputs.fft_input(n, batch, seed=k), cuda)
            y = torch.empty_like(x)
            d = -1 if k % 2 else 1
            jobs.append(ppx.make_job(ppx.OP_FFT, ppx.C64, n, batch, x, y, direction=d))
            calls.append(lambda c, o, x=x, n=n, b=batch, d=d: ppx.fft_batched(x, o, n, b, d, c))
        elif op == S:
            x = to_dev(inputs.scan_input_normal(n, batch, np.float32, seed=k), cuda)
            y = torch.empty_like(x)
            excl = k % 2
            jobs.append(ppx.make_job(ppx.OP_SCAN, ppx.F32, n, batch, x, y, algo=excl))
            f = ppx.scan_exclusive_batched if excl else ppx.scan_batched
            calls.append(lambda c, o, x=x, n=n, b=batch, f=f: f(x, o, n, b, ppx.F32, c))
        else:
            v = [to_dev(a, cuda) for a in inputs.tridiag_input(n, batch, np.float32, seed=k)[:4]]
            y = torch.empty_like(v[3])
            jobs.append(ppx.make_job(ppx.OP_TRIDIAG, ppx.F32, n, batch, v[0], y, algo=ppx.TRI_CR_PCR, b=v[1], c=v[2],
                                     d=v[3]))
            calls.append(lambda c, o, v=v, n=n, b=batch: ppx.tridiag_batched(*v, o, n, b, ppx.F32, c))
        outs.append(y)
    assert ppx.mixed_argument_launch(jobs)
    banner(f"mixed class launch {name}: {len(jobs)} jobs")
    ppx.launch_mixed(jobs)
    for job, y, call, spec in zip(jobs, outs, calls, LAUNCHES[name]):
        ref = torch.empty_like(y)
        call(ppx.mixed_tile_config(job)[1], ref)
        assert np.array_equal(to_host(y).view(np.uint8), to_host(ref).view(np.uint8)), spec
