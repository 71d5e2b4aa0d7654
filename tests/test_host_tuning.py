"""Launch shapes saved in a file (H2MV_AUTOTUNE_CACHE), by the library's host
code with a HIP runtime that only keeps count; no GPU."""
from test_host_memory import _check, _program


def test_shapes_saved_for_other_kernels_are_timed_again(tmp_path):
    """Lines as written before the streaming launch for narrow passes and the
    present candidates: neither obeyed nor an error; the shapes timed instead
    are saved and found by the next process."""
    exe = _program(tmp_path, "saved_tuning", ["h2_run.cpp", "h2_batch.cpp"])
    cache = tmp_path / "tune.txt"
    cache.write_text("single-k1-n4096-r64-blocks0-nt16 3 256 32\nsingle-k1-n4096-r64-blocks0-nt32 3 512 32\n")
    _check(exe, "timed", H2MV_AUTOTUNE_CACHE=str(cache))
    assert len(cache.read_text().split("\n")) == 5
    _check(exe, "saved", H2MV_AUTOTUNE_CACHE=str(cache))
