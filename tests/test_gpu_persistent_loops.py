"""GPU parity of the persistent kernels on batches that make every resident
workgroup loop: at least three groups each (from the kernel's own registers
and LDS; eight where the scan asks for that many), with a ragged last group.  Smaller batches run the plain twin.

Scans and tridiagonal solves do the same arithmetic as the plain kernel and are
compared with it bit for bit over the whole batch; FFTs within the FFT's bound
of the plain kernel's result.  Nothing may be stored past the batch.
"""
import pytest

from paper_2310_16214_amd import ppx
from tests.gpu_util import banner, fft_tol

pytestmark = pytest.mark.gpu

PIPE = {ppx.OP_FFT: 2, ppx.OP_SCAN: 2, ppx.OP_TRIDIAG: 8}


def looping_batch(op, dtype, n, cfg):
    m = ppx.device_model_gfx950()
    r = ppx.kernel_resources(op, dtype, n, cfg)
    blocks, _ = ppx.occupancy(m, r)
    assert blocks >= 1
    # a scan of one 16-byte vector per thread: from eight groups per workgroup on
    groups = 8 if op == ppx.OP_SCAN and cfg.elems_per_thread * (8 if dtype == ppx.F64 else 4) == 16 else 3
    return groups * blocks * m.num_cus * cfg.problems_per_block + 1


def run_both(cuda, op, dtype, n, cfg, call, like):
    """The persistent and the plain kernel's results (each [batch, n]) of one call."""
    import torch
    batch = looping_batch(op, dtype, n, cfg)
    banner(f"persistent loop op={op} dtype={dtype} n={n} batch={batch} {cfg}")
    g = torch.Generator(device=cuda).manual_seed(n + cfg.threads_per_block)
    x = like(batch, g)
    out = []
    for c in (cfg, ppx.make_config(cfg.radix, cfg.threads_per_block, cfg.problems_per_block, cfg.algo & ~PIPE[op])):
        buf = torch.full((batch * n + 4096,), -7, dtype=x[-1].dtype, device=cuda)
        call(x, buf, batch, c)
        assert bool((buf[batch * n:] == -7).all()), f"{c}: stored past the batch"
        out.append(buf[:batch * n].view(batch, n))
    return out


@pytest.mark.parametrize("dtype", [ppx.I32, ppx.F32, ppx.F64])
@pytest.mark.parametrize("L,P,n", [(64, 2, 64), (1024, 2, 512), (64, 4, 128), (512, 4, 1024), (256, 8, 512), (256, 16, 4096), (1024, 16, 2048), (1024, 32, 16384)])
def test_scan(cuda, dtype, L, P, n):
    import torch
    if dtype == ppx.F64 and P > 16:
        pytest.skip("float64 holds at most 16 values per thread")
    t = {ppx.I32: torch.int32, ppx.F32: torch.float32, ppx.F64: torch.float64}[dtype]
    for algo in (ppx.SCAN_KS_PIPE, ppx.SCAN_LF_PIPE):
        cfg = ppx.make_config(2, L, L * P // n, algo)
        for f in (ppx.scan_batched, ppx.scan_exclusive_batched):
            y, ref = run_both(
                cuda, ppx.OP_SCAN, dtype, n, cfg, lambda x, o, b, c: f(x[0], o, n, b, dtype, c),
                lambda b, g: [torch.randint(-100, 101, (b, n), device=cuda, generator=g).to(t) if dtype == ppx.I32
                              else torch.rand(b, n, dtype=t, device=cuda, generator=g)])
            assert torch.equal(y, ref), cfg


@pytest.mark.parametrize("dtype", [ppx.F32, ppx.F64])
@pytest.mark.parametrize("P,n", [(4, 64), (8, 512), (16, 64), (16, 1024)])
@pytest.mark.parametrize("algo", [ppx.TRI_CR_PCR, ppx.TRI_CR_SHFL, ppx.TRI_PCR_SHFL, ppx.TRI_PCR_REG, ppx.TRI_WM, ppx.TRI_LF])
def test_tridiag(cuda, dtype, P, n, algo):
    import torch
    t = torch.float32 if dtype == ppx.F32 else torch.float64

    def systems(b, g):
        u = lambda: torch.rand(b, n, dtype=t, device=cuda, generator=g)  # noqa: E731
        a, c = 2 * u() - 1, 2 * u() - 1
        return [a, a.abs() + c.abs() + 1 + u(), c, 2 * u() - 1]

    cfg = ppx.make_config(2, 64 if P == 4 else 256, (64 if P == 4 else 256) * P // n, algo | ppx.TRI_PIPE)
    y, ref = run_both(cuda, ppx.OP_TRIDIAG, dtype, n, cfg,
                      lambda x, o, b, c: ppx.tridiag_batched(*x, o, n, b, dtype, c), systems)
    assert bool(torch.isfinite(ref).all())
    assert torch.equal(y, ref), cfg


@pytest.mark.parametrize("split", [0, 1])
@pytest.mark.parametrize("radix,L,n", [(8, 64, 64), (8, 256, 1024), (8, 1024, 8192), (16, 64, 256), (16, 256, 4096),
                                       (16, 1024, 16384)])
def test_fft(cuda, radix, L, n, split):
    import torch
    cfg = ppx.make_config(radix, L, L * radix // n, ppx.FFT_LDS_PIPE | split)
    for direction in (-1, 1):
        y, ref = run_both(
            cuda, ppx.OP_FFT, ppx.C64, n, cfg, lambda x, o, b, c: ppx.fft_batched(x[0], o, n, b, direction, c),
            lambda b, g: [torch.view_as_complex(torch.rand(b, n, 2, device=cuda, generator=g) * 2 - 1)])
        err = torch.linalg.vector_norm(y - ref, dim=1) / torch.linalg.vector_norm(ref, dim=1)
        assert float(err.max()) <= fft_tol(n), cfg
