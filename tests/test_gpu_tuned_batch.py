"""GPU tests of what a NULL call runs after a tuning: the configuration that
tune() recorded, at the batch it was tuned at, and the large-FFT plan of a
cache file at its batch (its bits against the same plan given explicitly),
both through a save and a load; and, up to 2^17 points, the recorded plan from
half a tile per CU on."""
import pytest

from paper_2310_16214_amd import inputs, ppx
from tests.gpu_util import banner, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("op,dtype,n,batch", [(ppx.OP_FFT, ppx.C64, 1024, 64), (ppx.OP_SCAN, ppx.F32, 4096, 16),
                                              (ppx.OP_TRIDIAG, ppx.F32, 256, 64)])
def test_tuned_entry_is_used_at_its_batch(cuda, tmp_path, op, dtype, n, batch):
    p = tmp_path / "cache.txt"
    ppx.clear_tune_cache()
    try:
        for method in (ppx.TUNE_ANALYTICAL, ppx.TUNE_LEARNED):
            banner(f"tune op={op} n={n} batch={batch} method={method}")
            cfg, _, _ = ppx.tune(op, dtype, n, batch, method, max_evals=6)
            assert ppx.resolve_config(op, dtype, n, batch).as_tuple() == cfg.as_tuple()
            ppx.save_tune_cache(str(p))
            assert p.read_text().splitlines()[1].split()[-1] == str(batch)
            ppx.clear_tune_cache()
            assert ppx.load_tune_cache(str(p)) == 1
            assert ppx.resolve_config(op, dtype, n, batch).as_tuple() == cfg.as_tuple()
    finally:
        ppx.clear_tune_cache()


@pytest.mark.parametrize("tail", ["", " 1"])
@pytest.mark.parametrize("n,plan", [(1 << 16, "10 8 16 64 16"), (1 << 20, "10 16 16 16 16")])
def test_recorded_plan_is_used_at_its_batch(cuda, tmp_path, n, plan, tail):
    import torch
    import numpy as np
    p = tmp_path / "cache.txt"
    p.write_text(f"gfx950 plan {n} {plan} 0 -1{tail}\n")
    ppx.clear_tune_cache()
    try:
        assert ppx.load_tune_cache(str(p)) == 1
        x = to_dev(inputs.fft_input(n, 1, seed=n), cuda)
        y, z = torch.empty_like(x), torch.empty_like(x)
        banner(f"fft large n={n} batch=1 plan={plan} tail={tail!r}")
        ppx.fft_batched(x, y, n, 1)
        ppx.fft_batched_large(x, z, n, 1, -1, ppx.tuned_fft_plan(n))
        assert np.array_equal(to_host(y).view(np.uint32), to_host(z).view(np.uint32))
    finally:
        ppx.clear_tune_cache()


@pytest.mark.parametrize("n,batch", [(1 << 15, 33), (1 << 15, 63), (1 << 16, 33), (1 << 16, 40), (1 << 17, 17)])
def test_shipped_plan_from_half_a_tile_per_cu(cuda, n, batch):
    import os
    import torch
    import numpy as np
    ppx.clear_tune_cache()
    try:
        ppx.load_tune_cache(os.path.join(os.path.dirname(ppx.__file__), "tuned", "mi355x.txt"))
        plan = ppx.tuned_fft_plan(n)
        tiles = batch * min((1 << plan.log2_n1) // plan.tile_a, (n >> plan.log2_n1) // plan.tile_b)
        cus = ppx.device_model_gfx950().num_cus
        if not cus < 2 * tiles < 2 * cus:
            pytest.skip("not in the range on this device")
        x = to_dev(inputs.fft_input(n, batch, seed=n), cuda)
        y, z = torch.empty_like(x), torch.empty_like(x)
        banner(f"fft large n={n} batch={batch} NULL plan")
        ppx.fft_batched(x, y, n, batch)
        ppx.fft_batched_large(x, z, n, batch, -1, plan)
        assert np.array_equal(to_host(y).view(np.uint32), to_host(z).view(np.uint32))
    finally:
        ppx.clear_tune_cache()
