"""Scratch of the stand-alone sort: a buffer sized for n pairs serves fewer."""
from paper_2410_00486_amd import _lib as L


def test_scratch_never_shrinks_with_more_pairs():
    sizes = [0, 1, 1023, 1024, 1025, 8192, 8193, 1 << 18, (1 << 19) - 1, 1 << 19, (1 << 19) + 1,
             600_000, 1 << 20, (1 << 20) + 1, 5_000_000]
    bytes_of = [int(L.lib().gs_sort_tmp_bytes(n)) for n in sizes]
    assert bytes_of == sorted(bytes_of)
    assert all(b >= 12 * n for n, b in zip(sizes, bytes_of))
