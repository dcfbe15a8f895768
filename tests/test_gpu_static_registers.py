"""GPU test of the static register table: a process that sees no GPU resolves
NULL configurations, and picks within a tridiagonal family, as one that asks
the device for the kernels' registers."""
import json
import os
import subprocess
import sys

import pytest

from paper_2310_16214_amd import ppx

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def choices():
    out = {}
    for op, dtypes, log2_elems in ((ppx.OP_FFT, (ppx.C64,), 25), (ppx.OP_SCAN, (ppx.I32, ppx.F32, ppx.F64), 24),
                                   (ppx.OP_TRIDIAG, (ppx.F32, ppx.F64), 22)):
        for dt in dtypes:
            for ln in range(4, 14):
                n = 1 << ln
                for batch in (1, 17, 256, 1000, (1 << log2_elems) // n):
                    key = "%d %d %d %d" % (op, dt, n, batch)
                    out[key] = list(ppx.resolve_config(op, dt, n, batch).as_tuple())
                    for fam in (ppx.TRI_CR, ppx.TRI_PCR, ppx.TRI_CR_PCR, ppx.TRI_WM, ppx.TRI_LF):
                        cands = [c for c in ppx.enumerate_configs(op, dt, n) if ppx.tri_family(c.algo) == fam]
                        if op == ppx.OP_TRIDIAG and cands:
                            out["%s %d" % (key, fam)] = list(cands[ppx.analytical_select(op, dt, n, batch, cands)].as_tuple())
    return out


def test_resolution_without_a_gpu(cuda):
    import torch
    ppx.clear_tune_cache()
    x = torch.zeros(1, 16, dtype=torch.complex64, device=cuda)
    ppx.fft_batched(x, torch.empty_like(x), 16, 1)  # the library knows its device from here on
    here = choices()
    code = "import json; from tests import test_gpu_static_registers as t; print(json.dumps(t.choices()))"
    p = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=100,
                       env=dict(os.environ, HIP_VISIBLE_DEVICES="-1"))
    assert p.returncode == 0, p.stderr[-2000:]
    there = json.loads(p.stdout.splitlines()[-1])
    assert {k: (v, there[k]) for k, v in here.items() if there[k] != v} == {}
