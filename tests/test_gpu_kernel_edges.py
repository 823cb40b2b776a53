"""Kernel variants at the sizes where they could go wrong (edges of work
items, of batches and of buckets), against the FP64 oracle or another form of
the same path."""
import numpy as np
import pytest
import torch

import oracle
import paper_2410_00486_amd as gsr
from paper_2410_00486_amd import _lib as L
from synth import scenes

from gpu_common import run_gpu

pytestmark = pytest.mark.gpu


def _wide_scene(n, width, height, log_scale, seed=5, n_wide=None):
    """n Gaussians before the camera, the nearest n_wide of them spread over
    most of the image."""
    w = scenes.tiny_scene(seed, n=n, width=width, height=height, f=0.8 * width)
    order = np.argsort(w.scene.means[:, 2])
    wide = order[:n if n_wide is None else n_wide]
    w.scene.log_scales[wide] = log_scale
    return w


@pytest.mark.parametrize("n,n_wide,width,height", [
    (1, 1, 8, 8),            # one pair
    (40, 40, 640, 480),      # one group of records, many work items
    (1030, 12, 640, 480),    # two groups, the first one heavy
    (1024, 3, 203, 117),     # a full group, odd image
])
def test_radix_pair_generation_work_items(n, n_wide, width, height):
    """The generated and sorted lists equal the oracle's when the first
    groups of depth-sorted records hold many work items of pairs."""
    w = _wide_scene(n, width, height, -0.5, n_wide=n_wide)
    cam = w.cameras[0]
    print(f"pair generation n {n} wide {n_wide} {width}x{height}", flush=True)
    it = run_gpu(w.scene, [cam], tile=(8, 8), flags=L.GS_RADIX_BIN)
    pre = oracle.preprocess(w.scene, cam, (8, 8))
    keys, vals, ranges = oracle.sort_pairs(pre, cam, (8, 8))
    fl = it.plan.flags_of(it.ws)
    P, T = int(fl[L.F_PAIRS]), it.plan.total_tiles
    assert fl[L.F_OVERFLOW] == 0 and P == keys.shape[0]
    got = lambda reg, dt, m: it.plan.region(it.ws, reg, dt, m).cpu().numpy()
    np.testing.assert_array_equal(got(L.GS_WS_SORTED_KEYS, torch.int64, P).view(np.uint64), keys)
    np.testing.assert_array_equal(got(L.GS_WS_SORTED_RECS, torch.int32, P), vals.astype(np.int32))
    np.testing.assert_array_equal(got(L.GS_WS_RANGES, torch.int32, 2 * T).view(np.uint32), ranges)
