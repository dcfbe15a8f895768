"""CPU check of the rounding behaviour of the scan kernels' row layout (no GPU,
no library call): the arithmetic of scan_device.h in numpy float32, in its
order.  A wave holds 64 P consecutive elements as rows of 64 vectors of V = 4;
per row: the serial scan of each vector, the lane network over the vectors'
totals within the problem's lanes, the prefix from the lane before; then the
carry over the earlier rows of the problem, the sum of the earlier waves'
totals by rotations within 16 lanes, and the add-back.  Every output must stay
within the definition's bound, on the input that defeats prefixes formed by
subtraction, and integers must come out exact.
"""
import numpy as np
import pytest

import oracle
from paper_2310_16214_amd import inputs
from tests.gpu_util import scan_bound
from tests.test_scan_lane_emulation import lanes_ks, lanes_lf

F = np.float32
V = 4


def network(tot, lanes_of_problem, wide):
    """The lane network over segments of the wave: `wide` is the whole-wave
    one; with narrower segments its later steps do not run."""
    if lanes_of_problem == 64:
        return wide(tot)
    x, lane = tot.copy(), np.arange(64)
    ls = lane & (lanes_of_problem - 1)
    d = 1
    while d < lanes_of_problem:
        if wide is lanes_ks and d >= 16:  # row broadcast of lane 15 (47)
            row = lane // 16
            x = np.where((row == 1) | (row == 3), x + np.where(row == 1, x[15], x[47]), x).astype(F)
        elif wide is lanes_ks:
            y = np.where(lane % 16 >= d, np.roll(x, d), F(0))
            x = np.where(ls >= d, x + y, x).astype(F)
        else:
            src = (lane & ~(2 * d - 1)) | (d - 1)
            x = np.where(lane & d, x + x[src], x).astype(F)
        d *= 2
    return x


def row16_sum(x):
    x = x.copy()
    for d in (8, 4, 2, 1):
        x = (x + np.roll(x, d)).astype(F)
    return x


def emulate(x, P, wide, exclusive):
    """All the elements of one workgroup: x is [problems, n] with a whole
    number of waves of 64 P elements."""
    prob, n = x.shape
    R, wave = P // V, 64 * P
    nw = prob * n // wave
    assert nw * wave == prob * n and nw <= 16
    v = x.astype(F).reshape(nw, R, 64, V).copy()  # [wave][row][lane][vector]
    seg = min(64, n // V)
    prefix = np.zeros((nw, R, 64), F)
    total = np.zeros(nw, F)
    for w in range(nw):
        carry = F(0)
        for j in range(R):
            tot = np.zeros(64, F)
            run = np.zeros(64, F)
            for e in range(V):  # 1. serial scan within each vector
                nxt = (run + v[w, j, :, e]).astype(F) if e or exclusive else v[w, j, :, 0].copy()
                if exclusive:
                    v[w, j, :, e] = run
                else:
                    v[w, j, :, e] = nxt
                run = nxt
            tot = run
            inc = network(tot, seg, wide)  # 2.
            pre = np.concatenate([[F(0)], inc[:-1]]).astype(F)
            pre[(np.arange(64) & (seg - 1)) == 0] = F(0)
            if n > 64 * V:
                rows = min(R, n // (64 * V))
                if j % rows == 0:
                    carry = F(0)
                pre = (pre + carry).astype(F)
                carry = F(carry + inc[63])
            else:
                carry = inc[63]
            prefix[w, j] = pre
        total[w] = carry
    before = np.zeros(nw, F)
    per = n // wave  # waves of a problem
    if per > 1:
        for w in range(nw):  # 3.
            w0 = w & ~(per - 1)
            slot = np.array([total[u] if w0 <= u < w else F(0) for u in range(16)], F)
            s = row16_sum(slot)
            assert np.all(np.abs(s - s[0]) <= 64 * 2.0 ** -24 * np.abs(slot).sum())
            before[w] = s[0]
    p = (prefix + before[:, None, None]).astype(F)
    return (v + p[..., None]).astype(F).reshape(prob, n)  # 4.


# problems of part of a row, a row, some rows, a wave, several waves
SHAPES = [(8, 16, 32), (8, 64, 8), (16, 128, 8), (8, 256, 2), (16, 256, 4), (16, 512, 2), (32, 1024, 2), (32, 2048, 1),
          (8, 2048, 1), (16, 4096, 2), (16, 16384, 1)]


@pytest.mark.parametrize("wide", [lanes_ks, lanes_lf], ids=["ks", "lf"])
@pytest.mark.parametrize("exclusive", [False, True])
@pytest.mark.parametrize("P,n,prob", SHAPES)
def test_rows(wide, exclusive, P, n, prob):
    ints = np.random.default_rng(n + P).integers(-100, 101, (prob, n))
    want = np.cumsum(ints, axis=1) - (ints if exclusive else 0)
    assert np.array_equal(emulate(ints, P, wide, exclusive), want.astype(F))
    for seed in range(4):
        x = inputs.scan_input_spiked(n, prob, np.float32, seed=seed)
        err = np.abs(emulate(x, P, wide, exclusive).astype(np.float64) - oracle.scan(x, exclusive=exclusive))
        assert np.all(err <= scan_bound(x, 2.0 ** -24, exclusive=exclusive))
