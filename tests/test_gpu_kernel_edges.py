"""Kernel variants at the sizes where they could go wrong (edges of work
items, of batches and of buckets), against the FP64 oracle or another form of
the same path."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2410_00486_amd as gsr
from oracle import densify as oracle_densify
from oracle import ssim as oracle_ssim
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


@pytest.mark.parametrize("n", [64, 65, 128, 129, 256, 257, 512, 513, 1025, 2048, 2049, 5000, 8192, 8193])
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


# ------------------------------------------------------- sort, rows of the pool

@pytest.mark.parametrize("n", [2, 255, 2047, 8191, 8192,   # one workgroup
                               8193, 24576,                # counts summed by the scatter
                               24577, 262145,              # scanned, one and two chunks
                               524288, 524289])            # few and many keys a block
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


def _pool(rng, n, deg, shift):
    """Parameters and moments on the device; with shift, arrays that begin 4
    bytes after a 16-byte boundary."""
    k = (deg + 1) ** 2
    shapes = [(n, 3), (n, 3), (n, 4), (n,), (n, k, 3)]
    host = [rng.normal(size=s).astype(np.float32) for s in shapes]
    dev = []
    for h in host:
        buf = torch.empty(h.size + 8, dtype=torch.float32, device=DEV)
        t = buf[1:1 + h.size] if shift else buf[:h.size]
        dev.append(t.view(h.shape).copy_(torch.from_numpy(h)))
    return dict(zip(gsr.Gaussians.FIELDS, host)), gsr.Gaussians(*dev, deg)


@pytest.mark.parametrize("n,deg,shift", [(1, 0, False), (127, 1, False), (128, 2, True),
                                         (129, 3, False), (257, 3, True), (300, 1, True)])
def test_permute_rows(n, deg, shift):
    print(f"permute n {n} degree {deg} shift {shift}", flush=True)
    rng = np.random.default_rng(n)
    host, g = _pool(rng, n, deg, shift)
    perm = rng.permutation(n).astype(np.int32)
    out = gsr.permute(g, torch.from_numpy(perm).to(DEV))
    torch.cuda.synchronize()
    for f in gsr.Gaussians.FIELDS:
        np.testing.assert_array_equal(getattr(out, f).cpu().numpy(), host[f][perm])


@pytest.mark.parametrize("n,deg,shift,roles", [
    (1, 0, False, "s"), (255, 1, False, "kcs-"), (256, 3, False, "c"), (257, 3, True, "s"),
    (2048, 2, False, "kcs-"), (2049, 0, True, "-"), (2305, 3, False, "cs--k"),
])
def test_densify_rows_and_capacity(n, deg, shift, roles):
    """Rows of kept (k), cloned (c), split (s) and pruned (-) Gaussians, with
    room for all outputs and with one row too few: then the prefix that fits
    is the same, whole Gaussians only, and nothing behind it is written."""
    print(f"densify n {n} degree {deg} shift {shift} {roles}", flush=True)
    rng = np.random.default_rng(n + deg)
    role = np.array([roles[i % len(roles)] for i in range(n)])
    (P, g), (M, m), (V, v) = (_pool(rng, n, deg, shift) for _ in range(3))
    P["opacity_logits"][:] = np.where(role == "-", -6.0, 1.0)
    P["log_scales"][:] = np.where(role == "s", -2.0, -6.0)[:, None]
    for f in ("opacity_logits", "log_scales"):
        getattr(g, f).copy_(torch.from_numpy(P[f]))
    denom = np.ones(n, np.float32)
    accum = np.where((role == "c") | (role == "s"), 0.01, 0.0).astype(np.float32)
    normals = rng.standard_normal((n, 2, 3)).astype(np.float32)
    dev = lambda x: torch.from_numpy(x).to(DEV)
    a_t, d_t, n_t = dev(accum), dev(denom), dev(normals.reshape(-1))
    ref = oracle_densify.densify_prune(P, M, V, accum, denom, normals, 0.001, 0.02, 0.01, 1.0)
    total = ref[0]["means"].shape[0]
    count = np.select([role == "-", role == "k"], [0, 1], 2)
    mark = 12345.0
    for cap in (total, total - 1):
        if cap < 0:
            continue
        ends = np.cumsum(count)
        fits = int(ends[ends <= cap].max(initial=0))
        outs = [_pool(rng, total + 1, deg, shift)[1] for _ in range(3)]
        for o in outs:
            for x in o.tensors():
                x.fill_(mark)
        n_out = torch.zeros(1, dtype=torch.int32, device=DEV)
        tmp = torch.empty(max(int(L.lib().gs_densify_tmp_bytes(n)), 256), dtype=torch.uint8,
                          device=DEV)
        c = [g.c(), m.grads_c(), v.grads_c()] + [o.grads_c() for o in outs]
        r = [ctypes.byref(x) for x in c]
        L.check(L.lib().gs_densify_prune(*r[:3], a_t.data_ptr(), d_t.data_ptr(), n_t.data_ptr(),
                                         0.001, 0.02, 0.01, 1.0, *r[3:], cap, n_out.data_ptr(),
                                         tmp.data_ptr(),
                                         torch.cuda.current_stream().cuda_stream))
        torch.cuda.synchronize()
        assert int(n_out.item()) == total
        for k, o in enumerate(outs):
            for f in gsr.Gaussians.FIELDS:
                x = getattr(o, f).cpu().numpy()
                want = ref[k][f].reshape((total,) + x.shape[1:])[:fits]
                if k == 0 and f in ("means", "log_scales"):
                    np.testing.assert_allclose(x[:fits], want, rtol=2e-7, atol=1e-7)
                else:
                    np.testing.assert_array_equal(x[:fits], want)
                assert (x[fits:] == mark).all()


# ------------------------------------------------- projection backward, many pairs

@pytest.mark.parametrize("flags", [0, L.GS_RADIX_BIN])
def test_projection_backward_records_of_many_pairs(flags):
    """Several views whose records reach few to many tiles: on both sides of
    the length from which a wavefront sums a record, and more than one
    wavefront's step long; then fewer such records on the same workspace."""
    w = scenes.tiny_scene(17, n=40, width=64, height=32, f=30.0, degree=2)
    w.scene.log_scales[:24] = -0.2
    w.scene.opacity_logits[:] = -2.5
    eye, zero = np.eye(3, dtype=np.float32), np.zeros(3, np.float32)
    cams = [scenes.Camera(wd, ht, f, f, wd / 2, ht / 2, eye, zero)
            for wd, ht, f in ((248, 8, 60.0), (64, 32, 30.0), (88, 24, 40.0), (203, 117, 90.0))]
    gcs, gds = scenes.linear_loss_weights(23, cams)
    print(f"records of many pairs, flags {flags}", flush=True)
    it = run_gpu(w.scene, cams, tile=(8, 8), flags=flags, dL_dcolor=gcs, dL_ddepth=gds)
    tt = it.plan.region(it.ws, L.GS_WS_TILES_TOUCHED, torch.int32, len(cams) * 40).cpu().numpy()
    assert {32, 33} <= set(tt.tolist()) and tt.max() > 100
    grads, _, exclude, _ = oracle_reference(w.scene, cams, gcs, gds, (8, 8))
    assert_grads_close(grads_np(it), grads, exclude)
    w.scene.log_scales[12:24] = -3.0
    it.g.log_scales.copy_(torch.from_numpy(w.scene.log_scales))
    it.enqueue()
    torch.cuda.synchronize()
    grads, _, exclude, _ = oracle_reference(w.scene, cams, gcs, gds, (8, 8))
    assert_grads_close(grads_np(it), grads, exclude)


# ------------------------------------------------------- copies of the pair counters

@pytest.mark.parametrize("n,width,height", [(3000, 203, 117),    # scan of one workgroup
                                            (3000, 1200, 680),   # several
                                            (100, 203, 117)])    # some copies unused
def test_tile_counter_copies(n, width, height):
    """A plan with room for many pairs a tile counts in several copies of the
    counters, one with less room in a single one: same lists, on a first and
    a second iteration, and after one that did not fit."""
    w = scenes.tiny_scene(31, n=n, width=width, height=height, f=0.8 * width, degree=0)
    w.scene.log_scales[:] = -4.5
    cam = w.cameras[0]
    g = gsr.Gaussians.from_scene(w.scene, DEV)
    ct = gsr.cameras_tensor([cam], DEV)
    wh = [(width, height)]
    pairs = int(gsr.required_pairs(*g.tensors(), ct, wh, 0, (8, 8)))
    tiles = -(-width // 8) * -(-height // 8)
    assert pairs < 48 * tiles - 1
    print(f"counter copies n {n} {width}x{height}: {pairs} pairs, {tiles} tiles", flush=True)
    got = []
    for cap in (48 * tiles - 1, 48 * tiles):
        plan = gsr.Plan(n, 0, wh, tile=(8, 8), pair_capacity=cap)
        ws = plan.new_workspace(DEV)
        for log_scale in (-4.5, -0.5, -4.5):  # (the second one may overflow)
            g.log_scales.fill_(log_scale)
            gsr.preprocess(plan, ws, g, ct)
            gsr.bin_sort(plan, ws)
            torch.cuda.synchronize()
        assert plan.flags_of(ws)[L.F_OVERFLOW] == 0 and plan.flags_of(ws)[L.F_PAIRS] == pairs
        got.append([plan.region(ws, r, dt, c).cpu().numpy().copy() for r, dt, c in (
            (L.GS_WS_SORTED_KEYS, torch.int64, pairs), (L.GS_WS_SORTED_VALS, torch.int32, pairs),
            (L.GS_WS_SORTED_RECS, torch.int32, pairs), (L.GS_WS_RANGES, torch.int32, 2 * tiles))])
    for a, b in zip(*got):
        np.testing.assert_array_equal(a, b)
    pre = oracle.preprocess(w.scene, cam, (8, 8))
    keys, vals, _ = oracle.sort_pairs(pre, cam, (8, 8))
    np.testing.assert_array_equal(got[1][0].view(np.uint64), keys)
    np.testing.assert_array_equal(got[1][2], vals.astype(np.int32))


# ------------------------------------------------- differentiable call, early flags

def test_differentiable_call_grows_and_may_be_dropped():
    """A recorded call returns before its render has run: with a capacity that
    has to grow, with its graph dropped at once, and from two streams in turn
    the images and gradients are those of a fresh rasterizer."""
    w = scenes.slab_128x96()
    cam = w.cameras[0]
    ct = gsr.cameras_tensor([cam], DEV)
    wh = [(cam.width, cam.height)]
    leaves = [x.requires_grad_(True) for x in gsr.Gaussians.from_scene(w.scene, DEV).tensors()]
    weight = torch.linspace(-1.0, 1.0, 3 * cam.width * cam.height, device=DEV)

    def call(rz):
        color, _, _ = rz(*leaves, ct)
        return color.detach().clone(), torch.autograd.grad((color * weight).sum(), leaves)

    print("differentiable call, early flags", flush=True)
    want = call(gsr.Rasterizer(wh, w.scene.sh_degree, pair_capacity=1 << 18))
    rz = gsr.Rasterizer(wh, w.scene.sh_degree, pair_capacity=16)  # overflows, then fits
    side = torch.cuda.Stream()
    got = [call(rz)]
    for _ in range(3):
        rz(*leaves, ct)  # dropped
        got.append(call(rz))
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            got.append(call(rz))
        side.synchronize()
    torch.cuda.synchronize()
    for color, grads in got:
        assert torch.equal(color, want[0])
        for a, b in zip(grads, want[1]):
            assert torch.equal(a, b)


@pytest.mark.parametrize("n,log_scale,capacity", [
    (9000, -2.2, 1 << 20),    # more blocks in the grid than the 256 that are dealt to the dies
    (700_000, -6.0, 1 << 20),  # and in the depth passes
])
def test_radix_passes_over_many_blocks(n, log_scale, capacity):
    """The radix binning's lists equal the per-tile binning's where the passes
    run over many blocks, most of them or few of them with keys."""
    w = scenes.tiny_scene(41, n=n, width=640, height=480, f=500.0)
    cam = w.cameras[0]
    g = gsr.Gaussians.from_scene(w.scene, DEV)
    g.log_scales.fill_(log_scale)
    ct = gsr.cameras_tensor([cam, cam], DEV)
    wh = [(640, 480)] * 2
    print(f"radix passes n {n} log-scale {log_scale}", flush=True)
    got = []
    for flags in (0, L.GS_RADIX_BIN):
        plan = gsr.Plan(n, 0, wh, tile=(8, 8), flags=flags, pair_capacity=8 * capacity)
        ws = plan.new_workspace(DEV)
        gsr.preprocess(plan, ws, g, ct)
        gsr.bin_sort(plan, ws)
        torch.cuda.synchronize()
        fl = plan.flags_of(ws)
        assert fl[L.F_OVERFLOW] == 0 and fl[L.F_PAIRS] > capacity // 2
        P, T = int(fl[L.F_PAIRS]), plan.total_tiles
        got.append([plan.region(ws, r, dt, c).cpu().numpy().copy() for r, dt, c in (
            (L.GS_WS_SORTED_KEYS, torch.int64, P), (L.GS_WS_SORTED_VALS, torch.int32, P),
            (L.GS_WS_SORTED_RECS, torch.int32, P), (L.GS_WS_RANGES, torch.int32, 2 * T))])
    for a, b in zip(*got):
        np.testing.assert_array_equal(a, b)


# ------------------------------------------------------------------ SSIM tiles

@pytest.mark.parametrize("views", [[(32, 32)], [(33, 31)], [(8, 8), (65, 64)], [(31, 97), (32, 1)]])
def test_ssim_tile_edges(views):
    """Image sides around multiples of the stencil's tile, several views in one
    launch (the tolerances of the larger images' test)."""
    print(f"ssim tiles {views}", flush=True)
    rng = np.random.default_rng(views[0][0])
    plan = gsr.Plan(10, 0, views, pair_capacity=16)
    ws = plan.new_workspace(DEV)
    fr = gsr.Frame(plan, DEV)
    img = lambda c, w, h: rng.uniform(0.1, 0.9, (c, h, w)).astype(np.float32)
    data = [(img(3, w, h), img(3, w, h), img(1, w, h)[0], img(1, w, h)[0]) for w, h in views]
    flat = lambda k: torch.from_numpy(np.concatenate([d[k].reshape(-1) for d in data])).to(DEV)
    fr.color.copy_(flat(0))
    fr.depth.copy_(flat(2))
    gC, gD = gsr.render_loss(plan, ws, fr, flat(1), flat(3), lambda_ssim=0.2)
    torch.cuda.synchronize()
    gCs, gDs = plan.split_views(gC, 3), plan.split_views(gD)
    for v, (c, t, d, td) in enumerate(data):
        loss, rC, rD = oracle_ssim.rendered_loss_and_grads(c, d, t, td, 0.2, 0.1)
        assert abs(float(fr.loss[v]) - loss) <= 1e-5 * abs(loss)
        ok = np.abs(c.astype(np.float64) - t) > 1e-6
        err = np.abs(gCs[v].cpu().numpy().astype(np.float64) - rC)
        tol = 1e-3 * np.abs(rC) + 1e-3 * np.sqrt(np.mean(rC ** 2))
        assert (err <= tol)[ok].all()
        np.testing.assert_allclose(gDs[v].cpu().numpy().astype(np.float64), rD, rtol=1e-6, atol=0)


# ------------------------------------------------ gradients that are no numbers

def _pixelwise_gradients(w, tile, gcs, gds):
    it = run_gpu(w.scene, w.cameras, tile=tile, dL_dcolor=gcs, dL_ddepth=gds)
    last = it.plan.split_views(it.frame.last)[0].cpu().numpy()
    n = w.scene.n
    return np.concatenate([x.reshape(n, -1) for x in grads_np(it).values()], 1), last


@pytest.mark.parametrize("tile", [(8, 8), (16, 8), (16, 16)])
@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
def test_pixelwise_backward_keeps_a_bad_gradient_to_its_pixel(tile, value):
    """An upstream gradient that is NaN or infinite reaches the splats blended
    at its pixel and no other: at a pixel that nothing covers it has no
    effect, and at a covered one every Gaussian that a finite gradient there
    does not move keeps the bits it has without it."""
    w = scenes.tiny_scene(83, n=24, width=40, height=25, f=36.0, degree=1)
    gcs, gds = scenes.linear_loss_weights(12, w.cameras)
    print(f"bad gradient {value} tile {tile}", flush=True)
    _, last = _pixelwise_gradients(w, tile, gcs, gds)
    block = lambda a, y, x: a[y // 8 * 8:y // 8 * 8 + 8, x // 8 * 8:x // 8 * 8 + 8]
    pixels = [(y, x) for y, x in np.argwhere(last == 0) if (block(last, y, x) > 0).sum() >= 20]
    covered = [(y, x) for y, x in np.argwhere(last > 0) if (block(last, y, x) == 0).sum() >= 10]
    assert len(pixels) > 4 and len(covered) > 4
    for y, x in (pixels[0], pixels[-1], covered[0], covered[-1]):
        run = []
        for colour, depth in ((0.0, 0.0), (1e3, 1e3), (value, 0.0), (0.0, value)):
            c, d = [gcs[0].copy()], [gds[0].copy()]
            c[0][:, y, x], d[0][y, x] = colour, depth
            run.append(_pixelwise_gradients(w, tile, c, d)[0])
        base, moved = run[0], (run[1] != run[0]).any(axis=1)
        assert np.isfinite(base).all() and not moved.all()
        assert moved.any() == (last[y, x] > 0)
        for got in run[2:]:
            np.testing.assert_array_equal(got[~moved], base[~moved])
            assert not moved.any() or not np.isfinite(got[moved]).all()


# ------------------------------------------------------- splats from far away

@pytest.mark.parametrize("angle", [0.6, 0.9])
@pytest.mark.parametrize("ratio", [3.27, 3.28, 3.29])
def test_forward_keeps_the_tail_of_a_splat_millions_of_pixels_away(angle, ratio):
    """One long thin splat whose mean lies 8 million pixels from the image, so
    that alpha on its axis is just above 1/255 there: every pixel is that of
    the alpha test on its own offsets (FP32 as documented for the records),
    also in the blocks that only the axis crosses."""
    dist, tz, fx, W, V = 8e6, np.float32(0.01), np.float32(500.0), 64, 8
    u = np.array([np.cos(angle), np.sin(angle)])
    mean = np.array([[*(u * dist * float(tz) / float(fx)), tz]], np.float32)
    scene = scenes.Scene(mean, np.array([[np.log(dist / ratio * float(tz) / float(fx)), -20, -20]], np.float32),
                         np.array([[np.cos(angle / 2), 0, 0, np.sin(angle / 2)]], np.float32),
                         np.array([np.log(0.9 / 0.1)], np.float32),
                         np.full((1, 1, 3), 0.5 / 0.28209479177387814, np.float32), 0)
    rng = np.random.default_rng(1)
    cams = [scenes.Camera(W, W, fx, fx, *np.float32(W / 2 + rng.uniform(-3, 3, 2)),
                          np.eye(3, dtype=np.float32), np.zeros(3, np.float32), near=0.001)
            for _ in range(V)]
    print(f"far splat angle {angle} ratio {ratio}", flush=True)
    it = run_gpu(scene, cams, tile=(8, 8))
    raw = it.plan.region(it.ws, L.GS_WS_RECORDS, torch.uint8, 64 * V).cpu().numpy().reshape(V, 64)
    k = np.arange(W) + 0.5
    blended = 0
    for v in range(V):
        mx, my = raw[v, :16].view(np.float64)
        t, s1, s2, lo, z, r = raw[v, 16:40].view(np.float32).astype(np.float64)
        f32 = lambda x: np.asarray(x, np.float64).astype(np.float32).astype(np.float64)
        dx, dy = f32(mx - k)[None, :], f32(my - k)[:, None]
        p, q = f32(t * dy + dx), f32(dy - t * dx)
        e = lo - s1 * p * p - s2 * q * q
        # (roundings of the exponent: a few ulp of terms of at most 8)
        sure = np.abs(e - np.log2(1.0 / 255.0)) > 1e-4
        alpha = np.where(e >= np.log2(1.0 / 255.0), np.exp2(e), 0.0)
        col = it.plan.split_views(it.frame.color, 3)[v].cpu().numpy()[0]
        np.testing.assert_allclose(col[sure], (r * alpha)[sure], rtol=1e-4, atol=1e-7)
        blended += int((alpha[sure] > 0).sum())
    assert blended > 100


# ------------------------------------------- splat-wise launches of large plans

def _away(width, height):
    return scenes.Camera(width, height, 60.0, 60.0, width / 2.0, height / 2.0,
                         np.diag([1.0, -1.0, -1.0]).astype(np.float32), np.zeros(3, np.float32))


@pytest.mark.parametrize("n,room", [(30000, 4.0),   # 22,512 buckets in 48 tiles, the first launch takes 16,384
                                    (300, 1000.0)])  # few buckets, room for 225,000
def test_splatwise_backward_beyond_its_first_launch(n, room):
    """Buckets that the first launch's grid does not reach, and a plan with
    room for far more pairs than it gets: the gradients are, bit for bit,
    those of a plan whose second view, which sees nothing, has so many tiles
    that one launch takes all buckets."""
    w = scenes.tiny_scene(61, n=n, width=64, height=48, f=60.0)
    w.scene.log_scales[:] = 0.5
    w.scene.opacity_logits[:] = -4.6
    got = []
    for wh, cap in (((8, 8), int(48 * n * room)), ((512, 384), 48 * n)):
        cams = [w.cameras[0], _away(*wh)]
        gcs, gds = scenes.linear_loss_weights(6, cams[:1])
        gcs.append(np.zeros((3, wh[1], wh[0]), np.float32))
        gds.append(np.zeros((wh[1], wh[0]), np.float32))
        print(f"splat-wise launches n {n} second view {wh} capacity {cap}", flush=True)
        it = run_gpu(w.scene, cams, tile=(8, 8), flags=L.GS_SPLAT_BWD, dL_dcolor=gcs, dL_ddepth=gds,
                     capacity=cap)
        fl = it.plan.flags_of(it.ws)
        assert fl[L.F_OVERFLOW] == 0 and fl[L.F_PAIRS] == 48 * n
        got.append(grads_np(it))
    for f in got[0]:
        assert np.abs(got[0][f]).max() > 0 and np.isfinite(got[0][f]).all()
        np.testing.assert_array_equal(got[0][f], got[1][f])
