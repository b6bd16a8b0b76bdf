"""The autotuner starts from, and measures its gains against, the tiling that
a grid without explicit values gets (include/pic.h)."""
from paper_1204_0838_amd import autotune


def test_default_threads_are_the_librarys():
    d = autotune.DEFAULT
    # threads = 0: 512 where the LDS of two tiles fits 160 KiB, else 1024
    assert d["threads"] == (512 if 2 * autotune.lds_bytes(d) <= 160 * 1024 else 1024)
    assert (tuple(d["tile"]), d["guard"], d["interleave"], d["sort_interval"]) == ((8, 8, 8), 1, 0, 2)
