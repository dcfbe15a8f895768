"""GPU check of the registers of the hybrid across waves with few equations per
lane: at two or four, two workgroups of 1024 threads share a CU, in float32 and
float64 (with one, a call takes half as long again)."""
import pytest

from paper_2310_16214_amd import ppx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [ppx.F32, ppx.F64])
@pytest.mark.parametrize("P", [2, 4])
def test_two_workgroups_share_a_cu(cuda, dtype, P):
    n = 1024
    cfg = ppx.make_config(2, 1024, 1024 * P // n, ppx.TRI_CR_PCR)
    r = ppx.kernel_resources(ppx.OP_TRIDIAG, dtype, n, cfg)
    assert r.regs_per_thread <= 64
    assert ppx.occupancy(ppx.device_model_gfx950(), r) == (2, 32)
