"""CPU check of the shipped tune cache: a tridiagonal call without a
configuration takes the solver that the cache names for its size, or the one
family it holds; where the families' times decide, they are of one measure (no
entry without a batch, and no two measures of one configuration)."""
import os

from paper_2310_16214_amd import ppx

CACHE = os.path.join(os.path.dirname(ppx.__file__), "tuned", "mi355x.txt")
# the times of a size's families may decide only here: the spread between its
# families' times must exceed what two runs of one configuration differ by
CLOSE = 1.005


def _entries():
    for line in open(CACHE):
        w = line.split()
        if line.startswith("#") or w[1] == "plan":
            continue
        yield tuple(map(int, w[1:5])), tuple(map(int, w[5:11])), float(w[11]), int(w[13])


def test_solver_of_each_size():
    sizes = {}
    for (op, dt, n, fam), cfg, us, batch in _entries():
        assert batch > 0
        if op == ppx.OP_TRIDIAG:
            sizes.setdefault((dt, n), {})[fam] = (cfg, us)
    for key, fams in sizes.items():
        if -1 in fams:  # named: the entry of its family
            cfg, us = fams[-1]
            assert fams[ppx.tri_family(cfg[5])] == (cfg, us), key
        elif len(fams) > 1:
            order = sorted(us for _, us in fams.values())
            assert order[1] >= CLOSE * order[0], key
