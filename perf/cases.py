"""Cases for timing the library's calls: what a program that uses it has it do.

Every case is one pass through the Python binding's entry points
(``fft_batched``, ``scan_batched``, ``scan_exclusive_batched``,
``tridiag_batched``, ``launch_mixed``) on resident device buffers, with the
shipped tune cache loaded, as ``bench.py`` and the README set it up.

Ranges (``draw`` spreads over them, ``listed`` holds fixed points of them):

* FFT: n = 2^4 ... 2^23, both directions, batches from one problem to 256 MiB
  of input per call (the sizes of the sweep and of the large-N study).
* Scan: n = 2^4 ... 2^14, int32 / float32 / float64, inclusive and exclusive,
  up to 2^24 elements per call (2^25 for four-byte types).
* Tridiagonal: n = 2^4 ... 2^14 in float32 and 2^4 ... 2^13 in float64 (the
  library has no float64 solver for longer systems), the configuration the
  library resolves by itself or, for the sizes of the sweep (n = 32 ... 1024),
  the tuned PCR solver; up to 2^23 float32 or 2^22 float64 unknowns per call.
* Mixed launches: 4 ... 48 jobs of the serving mix (an operation at random,
  log2 n uniform in 4 ... 14, uneven batches), one launch.

Batches are mostly not powers of two.
"""
import functools
import math
import os
import random

import numpy as np
import torch

import paper_2310_16214_amd
from paper_2310_16214_amd import ppx

FFT_MAX_ELEMS = 1 << 25
SCAN_MAX_BYTES = 1 << 27
TRI_MAX_BYTES = 1 << 25  # per array
MIXED_MAX_ELEMS = 1 << 20  # per job


def listed():
    return [
        # 64 signals of 1024 points, the small batch a latency-bound caller
        # sends one at a time
        {"name": "fft_1024x64", "kind": "fft", "n": 1024, "batch": 64, "direction": -1},
        # an ordinary inverse call, 6 MiB, an odd number of problems
        {"name": "fft_256x3001_inverse", "kind": "fft", "n": 256, "batch": 3001, "direction": 1},
        # the largest single-kernel transform at the sweep's 256 MiB per call
        {"name": "fft_16384x2048", "kind": "fft", "n": 16384, "batch": 2048, "direction": -1},
        # one large signal by itself
        {"name": "fft_2p20x1", "kind": "fft", "n": 1 << 20, "batch": 1, "direction": -1},
        # the longest transform, a full-size inverse call of the large-N study
        {"name": "fft_2p23x4_inverse", "kind": "fft", "n": 1 << 23, "batch": 4, "direction": 1},
        # the sweep's int32 scan (2^24 elements) of short rows
        {"name": "scan_i32_256x65536", "kind": "scan", "n": 256, "batch": 65536, "dtype": "i32", "exclusive": False},
        # an exclusive float32 scan of the longest rows, an odd batch
        {"name": "scan_f32_16384x1001_exclusive", "kind": "scan", "n": 16384, "batch": 1001, "dtype": "f32",
         "exclusive": True},
        # a float64 scan of long rows, 2^24 elements
        {"name": "scan_f64_8192x2048", "kind": "scan", "n": 8192, "batch": 2048, "dtype": "f64", "exclusive": False},
        # the sweep's tridiagonal call: 2^22 float32 unknowns
        {"name": "tri_f32_512x8192", "kind": "tri", "n": 512, "batch": 8192, "dtype": "f32", "family": "auto"},
        # float64 systems too long for one wave, an odd batch
        {"name": "tri_f64_4096x777", "kind": "tri", "n": 4096, "batch": 777, "dtype": "f64", "family": "auto"},
        # the sweep's longest PCR solve (the solver named by the caller)
        {"name": "tri_f32_pcr_1024x4096", "kind": "tri", "n": 1024, "batch": 4096, "dtype": "f32", "family": "pcr"},
        # one launch of a serving loop: 16 uneven jobs
        {"name": "mixed_16_jobs", "kind": "mixed", "jobs": 16, "pick": 1},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _batch(rng, n, lo_elems, hi_elems):
    """A batch giving between lo_elems and hi_elems elements, as far as whole
    problems of size n allow; spread over the logarithm, not rounded."""
    most = max(1, hi_elems // n)
    least = min(most, max(1, lo_elems // n))
    return _log_uniform(rng, least, most)


def draw(rng):
    kind = rng.choice(["fft", "fft", "fft", "scan", "scan", "tri", "tri", "mixed"])
    if kind == "fft":
        n = 1 << rng.randint(4, 23)
        return {"kind": "fft", "n": n, "batch": _batch(rng, n, 1 << 10, FFT_MAX_ELEMS), "direction": rng.choice([-1, 1])}
    if kind == "scan":
        n = 1 << rng.randint(4, 14)
        dtype = rng.choice(["i32", "f32", "f64"])
        most = SCAN_MAX_BYTES // (8 if dtype == "f64" else 4)
        return {"kind": "scan", "n": n, "batch": _batch(rng, n, 1 << 10, most), "dtype": dtype,
                "exclusive": rng.choice([False, True])}
    if kind == "tri":
        family = rng.choice(["auto", "auto", "auto", "pcr"])
        dtype = rng.choice(["f32", "f64"])
        n = 1 << (rng.randint(5, 10) if family == "pcr" else rng.randint(4, 14 if dtype == "f32" else 13))
        most = TRI_MAX_BYTES // (8 if dtype == "f64" else 4)
        return {"kind": "tri", "n": n, "batch": _batch(rng, n, 1 << 10, most), "dtype": dtype, "family": family}
    return {"kind": "mixed", "jobs": rng.randint(4, 48), "pick": rng.randrange(1 << 20)}


# ------------------------------------------------------------------- inputs

TORCH = {"i32": torch.int32, "f32": torch.float32, "f64": torch.float64}
PPX = {"i32": ppx.I32, "f32": ppx.F32, "f64": ppx.F64}


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _uniform(g, shape, dtype, lo, hi):
    return torch.empty(shape, dtype=dtype, device="cuda").uniform_(lo, hi, generator=g)


def _fft_input(g, n, batch):
    """Real and imaginary parts uniform on [-1, 1]."""
    return torch.view_as_complex(_uniform(g, (batch, n, 2), torch.float32, -1.0, 1.0))


def _scan_input(g, n, batch, dtype):
    """int32 uniform on [-100, 100], float uniform on [0, 1)."""
    if dtype == "i32":
        return torch.randint(-100, 101, (batch, n), dtype=torch.int32, device="cuda", generator=g)
    return torch.rand((batch, n), dtype=TORCH[dtype], device="cuda", generator=g)


def _tri_input(g, n, batch, dtype):
    """Diagonally dominant systems (a, b, c, d) with a solution uniform on
    [-1, 1]; d is formed in float64 and rounded."""
    t = TORCH[dtype]
    a = _uniform(g, (batch, n), t, -1.0, 1.0)
    c = _uniform(g, (batch, n), t, -1.0, 1.0)
    b = a.abs() + c.abs() + _uniform(g, (batch, n), t, 1.0, 2.0)
    x = _uniform(g, (batch, n), t, -1.0, 1.0).double()
    d = b.double() * x
    d[:, 1:] += a[:, 1:].double() * x[:, :-1]
    d[:, :-1] += c[:, :-1].double() * x[:, 1:]
    return a, b, c, d.to(t)


def _mixed_specs(case):
    """The jobs of a mixed case: the serving mix (FFT, float32 scan, float32
    tridiagonal by the CR -> PCR hybrid), log2 n uniform in 4 ... 14, batch
    uniform up to 4096 and at most 2^20 elements per job."""
    rng = random.Random(case["pick"])
    specs = []
    for _ in range(case["jobs"]):
        op = rng.choice(["fft", "scan", "tri"])
        n = 1 << rng.randint(4, 14)
        specs.append((op, n, min(rng.randint(1, 4096), MIXED_MAX_ELEMS // n)))
    return specs


def _inputs(case, seed):
    g = _generator(seed)
    kind = case["kind"]
    if kind == "fft":
        return _fft_input(g, case["n"], case["batch"])
    if kind == "scan":
        return _scan_input(g, case["n"], case["batch"], case["dtype"])
    if kind == "tri":
        return _tri_input(g, case["n"], case["batch"], case["dtype"])
    out = []
    for op, n, batch in _mixed_specs(case):
        out.append(_fft_input(g, n, batch) if op == "fft" else
                   _scan_input(g, n, batch, "f32") if op == "scan" else _tri_input(g, n, batch, "f32"))
    return out


@functools.lru_cache(maxsize=None)
def _load_tuned():
    """The tuned configurations the package ships, loaded once per process."""
    ppx.load_tune_cache(os.path.join(os.path.dirname(paper_2310_16214_amd.__file__), "tuned", "mi355x.txt"))


# --------------------------------------------------------------- the passes

def prepare(case, seed):
    _load_tuned()
    x = _inputs(case, seed)
    kind = case["kind"]
    if kind in ("fft", "scan"):
        return {"case": case, "x": x, "out": torch.empty_like(x)}
    if kind == "tri":
        cfg = None
        if case["family"] == "pcr":
            cfg = ppx.tuned_config(ppx.OP_TRIDIAG, PPX[case["dtype"]], case["n"], ppx.TRI_PCR)
        return {"case": case, "x": x, "out": torch.empty_like(x[3]), "cfg": cfg}
    jobs, outs = [], []
    for (op, n, batch), v in zip(_mixed_specs(case), x):
        o = torch.empty_like(v[3] if op == "tri" else v)
        outs.append(o)
        if op == "fft":
            jobs.append(ppx.make_job(ppx.OP_FFT, ppx.C64, n, batch, v, o))
        elif op == "scan":
            jobs.append(ppx.make_job(ppx.OP_SCAN, ppx.F32, n, batch, v, o, algo=ppx.JOB_SCAN_INCLUSIVE))
        else:
            a, b, c, d = v
            jobs.append(ppx.make_job(ppx.OP_TRIDIAG, ppx.F32, n, batch, a, o, algo=ppx.TRI_CR_PCR, b=b, c=c, d=d))
    return {"case": case, "x": x, "out": outs, "jobs": jobs}


def run(state):
    case, x, out = state["case"], state["x"], state["out"]
    kind = case["kind"]
    if kind == "fft":
        ppx.fft_batched(x, out, case["n"], case["batch"], case["direction"])
    elif kind == "scan":
        f = ppx.scan_exclusive_batched if case["exclusive"] else ppx.scan_batched
        f(x, out, case["n"], case["batch"], PPX[case["dtype"]])
    elif kind == "tri":
        ppx.tridiag_batched(*x, out, case["n"], case["batch"], PPX[case["dtype"]], state["cfg"])
    else:
        ppx.launch_mixed(state["jobs"])
    return out


def _work(op, n, batch, dtype="f32"):
    """(bytes, flops): each input read once, each output written once; the
    FFT's 5 n log2 n, one addition per scanned value, Gaussian elimination's
    eight operations per unknown."""
    elems = n * batch
    size = 8 if dtype == "f64" else 4
    if op == "fft":
        return 16 * elems, 5 * elems * int(math.log2(n))
    if op == "scan":
        return 2 * size * elems, elems
    return 5 * size * elems, 8 * elems


def work(case):
    if case["kind"] == "mixed":
        each = [_work(*s) for s in _mixed_specs(case)]
        return {"bytes": sum(b for b, _ in each), "flops": sum(f for _, f in each)}
    b, f = _work(case["kind"], case["n"], case["batch"], case.get("dtype", "f32"))
    return {"bytes": b, "flops": f}


# ------------------------------------------------------------------- oracle

def _exact_fft(x, direction):
    x = x.cpu().to(torch.complex128)
    return torch.fft.fft(x) if direction == -1 else torch.fft.ifft(x, norm="forward")


def _exact_scan(x, dtype, exclusive):
    x = x.cpu()
    s = torch.cumsum(x.to(torch.int64 if dtype == "i32" else torch.float64), dim=1)
    if exclusive:
        s = torch.cat([torch.zeros_like(s[:, :1]), s[:, :-1]], dim=1)
    return s.to(torch.int32) if dtype == "i32" else s


def _exact_tri(a, b, c, d):
    """Elimination without pivoting over all systems at once, in extended
    precision, returned in float64."""
    a, b, c, d = (np.ascontiguousarray(v.cpu().numpy().T.astype(np.longdouble)) for v in (a, b, c, d))
    n = a.shape[0]
    for i in range(n):
        den = b[i] if i == 0 else b[i] - a[i] * c[i - 1]
        c[i] = c[i] / den
        d[i] = (d[i] if i == 0 else d[i] - a[i] * d[i - 1]) / den
    for i in range(n - 2, -1, -1):
        d[i] -= c[i] * d[i + 1]
    return np.ascontiguousarray(d.T.astype(np.float64))


def exact(case, seed):
    x = _inputs(case, seed)
    kind = case["kind"]
    if kind == "fft":
        return _exact_fft(x, case["direction"])
    if kind == "scan":
        return _exact_scan(x, case["dtype"], case["exclusive"])
    if kind == "tri":
        return _exact_tri(*x)
    return [_exact_fft(v, -1) if op == "fft" else _exact_scan(v, "f32", False) if op == "scan" else _exact_tri(*v)
            for (op, _, _), v in zip(_mixed_specs(case), x)]
