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

from gpu_common import (DEV, assert_forward_close, assert_grads_close, assert_pose_close, grads_np,
                        oracle_reference, run_gpu, view_images)

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


@pytest.mark.parametrize("n,width,height,log_scale", [
    (1, 1, 1, None), (3, 9, 7, None), (4, 8, 8, None), (5, 17, 8, None),       # a step's remainder
    (63, 16, 16, None), (64, 13, 9, None), (65, 33, 17, None),                  # a batch's
    (129, 40, 25, None), (300, 203, 117, None),                                 # several batches
    (90, 120, 90, (-0.6, -4.0, -4.0)),                                          # thin, rotated splats
    (200, 64, 48, (-1.0, -1.0, -5.0)),                                          # discs seen at all angles
])
def test_forward_blocks_match_oracle(n, width, height, log_scale):
    """The forward, one wavefront per 8x8 block of pixels with the splats that
    cannot reach the block left out, for every tile shape: colour and depth
    within the forward tolerance of the oracle, the last blended position
    equal to the oracle's at every pixel whose decisions are clear, and the
    images of the three shapes the same bits."""
    w = scenes.tiny_scene(11 + n, n=n, width=width, height=height, f=0.9 * max(width, 8))
    if log_scale is not None:
        w.scene.log_scales[:] = np.float32(log_scale)
    w.scene.opacity_logits[::7] = 8.0  # above the 0.99 clamp
    cam = w.cameras[0]
    first = None
    for tile in ((8, 8), (16, 8), (16, 16)):
        print(f"forward blocks n {n} {width}x{height} tile {tile}", flush=True)
        it = run_gpu(w.scene, [cam], tile=tile)
        ref = oracle.render(w.scene, cam, tile)
        assert not (ref["pre"]["near_edge"] != 0).any()
        col, dep, T, last = view_images(it, 0)
        assert_forward_close(col, dep, ref)
        ok = ref["flag"] == 0
        np.testing.assert_array_equal(last[ok], ref["last"][ok])
        if first is None:
            first = (col, dep, T)
        for a, b in zip(first, (col, dep, T)):
            np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("n", [64, 65, 128, 129, 512, 513, 1025, 8192, 8193])
def test_tile_sort_list_length_edges(n):
    """One tile's list at the lengths where the sort changes its form
    (registers, a wavefront in LDS, a workgroup in LDS, global memory): keys,
    records and ranges equal the oracle's order."""
    w = scenes.crowded_scene(7, n=n)
    cam = w.cameras[0]
    print(f"tile sort, {n} pairs in one tile", flush=True)
    it = run_gpu(w.scene, [cam], tile=(16, 16))
    pre = oracle.preprocess(w.scene, cam, (16, 16))
    keys, vals, ranges = oracle.sort_pairs(pre, cam, (16, 16))
    r = ranges.reshape(-1, 2).astype(np.int64)
    assert (r[:, 1] - r[:, 0]).max() == n
    P, T = keys.shape[0], it.plan.total_tiles
    got = lambda reg, dt, m: it.plan.region(it.ws, reg, dt, m).cpu().numpy()
    np.testing.assert_array_equal(got(L.GS_WS_SORTED_KEYS, torch.int64, P).view(np.uint64), keys)
    np.testing.assert_array_equal(got(L.GS_WS_SORTED_RECS, torch.int32, P), vals.astype(np.int32))
    np.testing.assert_array_equal(got(L.GS_WS_RANGES, torch.int32, 2 * T).view(np.uint32), ranges)


@pytest.mark.parametrize("n,width,height", [(1, 1, 1), (3, 17, 8), (64, 16, 16), (65, 33, 19),
                                            (130, 40, 25), (300, 90, 70)])
@pytest.mark.parametrize("tile", [(8, 8), (16, 8), (16, 16)])
def test_pixelwise_backward_blocks_match_oracle(n, width, height, tile):
    """The pixel-wise backward, a wavefront per 8x8 block with the blocks'
    sums added per tile: gradients and camera tangent within the gradient
    tolerance of the oracle, for lists around one and two batches and images
    that end inside a block."""
    w = scenes.tiny_scene(31 + n, n=n, width=width, height=height, f=0.9 * max(width, 8), degree=1)
    w.scene.opacity_logits[::7] = 8.0  # above the 0.99 clamp
    cam = w.cameras[0]
    print(f"pixel-wise backward n {n} {width}x{height} tile {tile}", flush=True)
    gcs, gds = scenes.linear_loss_weights(70 + n, [cam])
    it = run_gpu(w.scene, [cam], tile=tile, dL_dcolor=gcs, dL_ddepth=gds, pose=True)
    grads, poses, exclude, poses_f = oracle_reference(w.scene, [cam], gcs, gds, tile)
    assert_grads_close(grads_np(it), grads, exclude)
    assert_pose_close(it.dL_dpose.cpu().numpy(), poses, poses_f)


@pytest.mark.parametrize("n,width,height", [(1, 1, 1), (4, 9, 7), (15, 8, 8), (16, 8, 8), (17, 13, 9),
                                            (32, 8, 8), (33, 17, 8), (64, 8, 8), (65, 12, 8),
                                            (130, 24, 17), (300, 90, 70)])
def test_splatwise_backward_buckets_match_oracle(n, width, height):
    """The splat-wise backward over buckets of the splats that the forward
    kept: one, two and four segments per wavefront, several buckets per tile,
    images that end inside a tile, against the oracle; with an opaque splat
    in every seventh place (the clamped form) and without."""
    for opaque in (False, True):
        w = scenes.tiny_scene(51 + n, n=n, width=width, height=height, f=0.9 * max(width, 8), degree=1)
        if opaque:
            w.scene.opacity_logits[::7] = 8.0
        else:
            w.scene.opacity_logits[:] = np.minimum(w.scene.opacity_logits, 2.0) - 1.5
        cam = w.cameras[0]
        print(f"splat-wise backward n {n} {width}x{height} opaque {opaque}", flush=True)
        gcs, gds = scenes.linear_loss_weights(90 + n, [cam])
        it = run_gpu(w.scene, [cam], tile=(8, 8), flags=L.GS_SPLAT_BWD, dL_dcolor=gcs,
                     dL_ddepth=gds, pose=True)
        ref = oracle.render(w.scene, cam, (8, 8))
        col, dep, _, last = view_images(it, 0)
        assert_forward_close(col, dep, ref)
        ok = ref["flag"] == 0
        np.testing.assert_array_equal(last[ok], ref["last"][ok])
        grads, poses, exclude, poses_f = oracle_reference(w.scene, [cam], gcs, gds, (8, 8))
        assert_grads_close(grads_np(it), grads, exclude)
        assert_pose_close(it.dL_dpose.cpu().numpy(), poses, poses_f)


def test_splatwise_backward_pairs_behind_the_stop_get_zero():
    """Opaque splats in front: the pairs that the forward never looks at, and
    those it drops, get zero gradients even after an iteration that wrote
    theirs (the same workspace, other opacities)."""
    w = scenes.crowded_scene(3, n=400)
    cam = w.cameras[0]
    gcs, gds = scenes.linear_loss_weights(5, [cam])
    print("splat-wise backward, a second iteration on the same workspace", flush=True)
    # (room for the second iteration's pairs: more opaque splats reach further)
    it = run_gpu(w.scene, [cam], tile=(8, 8), flags=L.GS_SPLAT_BWD, dL_dcolor=gcs, dL_ddepth=gds,
                 capacity=1 << 16)
    near = np.argsort(w.scene.means[:, 2])[:60]
    w.scene.opacity_logits[near] = 6.0
    it.g.opacity_logits.copy_(torch.from_numpy(w.scene.opacity_logits))
    it.enqueue()
    torch.cuda.synchronize()
    assert it.plan.flags_of(it.ws)[L.F_OVERFLOW] == 0
    grads, _, exclude, _ = oracle_reference(w.scene, [cam], gcs, gds, (8, 8))
    assert_grads_close(grads_np(it), grads, exclude)


# ------------------------------------------------------------------------ sort

@pytest.mark.parametrize("n", [2, 255, 2047, 8191, 8192,   # one workgroup
                               8193, 32768,                # counts summed by the scatter
                               32769, 524288, 524289])     # scanned, one and two chunks
@pytest.mark.parametrize("bits", [5, 24, 46])              # one, three and six passes
def test_sort_sizes_and_passes(n, bits):
    """Equal keys keep their order; every number of passes ends in the
    caller's arrays; the sort covers whole bytes of the key and no more."""
    print(f"sort n {n} bits {bits}", flush=True)
    rng = np.random.default_rng(n + bits)
    keys = rng.integers(0, 1 << 62, n, dtype=np.int64)
    keys[::3] = keys[0]
    vals = np.arange(n, dtype=np.int32)
    kt, vt = torch.from_numpy(keys).to(DEV), torch.from_numpy(vals).to(DEV)
    gsr.sort_pairs(kt, vt, bits)
    torch.cuda.synchronize()
    low = keys & ((1 << ((bits + 7) // 8 * 8)) - 1)
    order = np.argsort(low, kind="stable")
    np.testing.assert_array_equal(kt.cpu().numpy(), keys[order])
    np.testing.assert_array_equal(vt.cpu().numpy(), vals[order])
