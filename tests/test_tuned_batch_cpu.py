"""CPU tests of the batch that a tune cache entry was tuned at: a NULL call of
that batch or a larger one takes the recorded configuration as it is, a
smaller one may take the shape fitted to it, an entry that does not say keeps
its configuration for every call, and the batch survives a save and a load."""
import pytest

from paper_2310_16214_amd import ppx

# a shape the small-batch rule would change at these sizes: (op, dtype, n,
# algo filter, config, batch)
ENTRIES = [
    (ppx.OP_FFT, ppx.C64, 1024, -1, ppx.make_config(16, 256, 4, 0), 64),
    (ppx.OP_FFT, ppx.C64, 256, -1, ppx.make_config(16, 128, 8, 1), 4096),
    (ppx.OP_TRIDIAG, ppx.F32, 256, -1, ppx.make_config(2, 256, 16, ppx.TRI_WM), 512),
    (ppx.OP_TRIDIAG, ppx.F64, 64, ppx.TRI_LF, ppx.make_config(2, 256, 32, ppx.TRI_LF), 100),
]


@pytest.fixture(autouse=True)
def empty_cache():
    ppx.clear_tune_cache()
    yield
    ppx.clear_tune_cache()


def _line(op, dtype, n, algo, c, tail):
    P = n * c.problems_per_block // c.threads_per_block
    return "gfx950 %d %d %d %d %d %d %d %d 0 %d 10.0 0%s\n" % (
        op, dtype, n, algo, c.radix, P, c.threads_per_block, c.problems_per_block, c.algo, tail)


@pytest.mark.parametrize("entry", ENTRIES)
def test_recorded_batch_keeps_the_configuration(tmp_path, entry):
    op, dtype, n, algo, cfg, batch = entry
    p, q = tmp_path / "a.txt", tmp_path / "b.txt"
    p.write_text(_line(op, dtype, n, algo, cfg, " %d" % batch))
    assert ppx.load_tune_cache(str(p)) == 1
    recorded = ppx.tuned_config(op, dtype, n, algo).as_tuple()
    for again in range(2):
        for b in (batch, batch + 1, 3 * batch, 1 << 20):
            assert ppx.resolve_config(op, dtype, n, b).as_tuple() == recorded, (again, b)
        assert ppx.resolve_config(op, dtype, n, batch - 1).as_tuple() != recorded, again  # fitted
        ppx.save_tune_cache(str(q))
        ppx.clear_tune_cache()
        assert ppx.load_tune_cache(str(q)) == 1


@pytest.mark.parametrize("tail", ["", " 0", " -3", " text"])
@pytest.mark.parametrize("entry", ENTRIES)
def test_unknown_batch_keeps_the_configuration(tmp_path, entry, tail):
    op, dtype, n, algo, cfg, _ = entry
    p = tmp_path / "a.txt"
    p.write_text(_line(op, dtype, n, algo, cfg, tail))
    assert ppx.load_tune_cache(str(p)) == 1
    recorded = ppx.tuned_config(op, dtype, n, algo).as_tuple()
    for b in (1, 64, 1 << 20):
        assert ppx.resolve_config(op, dtype, n, b).as_tuple() == recorded


def test_plan_batch_survives_a_round_trip(tmp_path):
    p, q = tmp_path / "a.txt", tmp_path / "b.txt"
    p.write_text("gfx950 plan 32768 9 8 8 64 16 0 -1 3\ngfx950 plan 65536 10 8 16 64 16 0 -1\n")
    assert ppx.load_tune_cache(str(p)) == 2
    ppx.save_tune_cache(str(q))
    lines = [w.split() for w in q.read_text().splitlines() if not w.startswith("#")]
    assert [(w[2], w[-1]) for w in lines] == [("32768", "3"), ("65536", "0")]
