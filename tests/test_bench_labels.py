"""What the benchmark's result line says of the kernels that ran."""
import pytest

import bench

COUNTS = {"gaussians": 1000, "visible_records": 800, "pairs": 5000, "pixels": 4096, "views": 1,
          "bwd_positions": 60000, "tiles": 64}


@pytest.mark.parametrize("tile,backward,forward_kernel,backward_kernel", [
    ((8, 8), "splat", "k_render_fwd<8,8,true>", "k_render_bwd_splat"),
    ((8, 8), "pixel", "k_render_fwd<8,8,false>", "k_render_bwd<8,8>"),
    ((16, 8), "splat", "k_render_fwd<16,8,false>", "k_render_bwd<16,8>"),
    ((16, 16), "pixel", "k_render_fwd<16,16,false>", "k_render_bwd<16,16>"),
])
def test_raster_spans_name_the_kernels_that_run(tile, backward, forward_kernel, backward_kernel):
    for span, kernel in (("forward", forward_kernel), ("raster_bwd", backward_kernel)):
        assert bench.roofline_of(span, 1.0, COUNTS, "slab", tile, backward, "tiles")["kernel"] == kernel


def test_the_per_tile_sort_is_counted_once():
    """One launch sorts the lists of all lengths in the per-tile binning; the
    radix binning has a pass in either span."""
    tiles, radix = (bench.stage_bytes(COUNTS, binning=b) for b in ("tiles", "radix"))
    assert tiles["bin_short_sort"] == 24 * COUNTS["pairs"] and tiles["bin_long_sort"] == 0
    assert radix["bin_short_sort"] == radix["bin_long_sort"] == 24 * COUNTS["pairs"]
