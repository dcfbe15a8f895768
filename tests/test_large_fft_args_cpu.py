"""CPU test: an argument error of a large-FFT call without a plan is reported as
such where no GPU is present (argument checks run before any HIP call)."""
import ctypes

from paper_2310_16214_amd import ppx

EINVAL = -1


def test_too_many_workgroups_of_a_recorded_plan(tmp_path):
    n, batch = 1 << 15, 1 << 25
    most = max(ppx.enumerate_fft_plans(n), key=lambda p: max((1 << p.log2_n1) // p.tile_a, (n >> p.log2_n1) // p.tile_b))
    assert batch * max((1 << most.log2_n1) // most.tile_a, (n >> most.log2_n1) // most.tile_b) > 2 ** 31 - 1
    path = tmp_path / "cache.txt"
    path.write_text("gfx950 plan %d %d %d %d %d %d 0 -1 %d\n" % (
        n, most.log2_n1, most.radix_a, most.radix_b, most.tile_a, most.tile_b, 2 * batch))
    ppx.clear_tune_cache()
    try:
        assert ppx.load_tune_cache(str(path)) == 1
        lib = ppx.lib()
        args = [ctypes.c_void_p(1 << 12), ctypes.c_void_p(1 << 60), ctypes.c_int64(n), ctypes.c_int64(batch),
                ctypes.c_int(-1), None, None]
        for f in (lib.fft_batched_large, lib.fft_batched):
            assert f(*args) == EINVAL
            assert "workgroups" in ppx.last_error()
    finally:
        ppx.clear_tune_cache()
