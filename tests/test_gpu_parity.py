"""GPU parity: libpxr (HIP, through the C ABI) against the CPU oracle on the same seeded inputs.

Bar: winning-id maps bit-exact; RGB within 1/255 per channel after uint8 rounding (the same fp32
operation order is used on both sides, so the expected difference is 0 and is asserted where noted).
"""
import itertools

import numpy as np
import pytest

from helpers import captured_kernels
from paper_2502_00021_amd import workloads as wl

pytestmark = pytest.mark.gpu

BG = 0xFFFFFFFF
GROUND = 0xFFFFFFFE


@pytest.fixture(scope="module")
def torch():
    import torch as _torch
    assert _torch.cuda.is_available(), "these tests need the MI355X"
    return _torch


@pytest.fixture(scope="module")
def pxr():
    from paper_2502_00021_amd import pxr as _pxr
    _pxr.lib()
    return _pxr


def _bind(torch, scene, dis):
    if dis is None:
        scene.apply_distractor(None)
        return
    d = dict(dis)
    if d["mode"] == "video":
        d["video"] = torch.from_numpy(np.ascontiguousarray(d["video"])).cuda()
        if d.get("env_offset") is not None:
            d["env_offset"] = torch.from_numpy(np.asarray(d["env_offset"]).astype(np.int32)).cuda()
        if d.get("env_video") is not None:
            d["env_video"] = torch.from_numpy(np.asarray(d["env_video"]).astype(np.int32)).cuda()
    scene.apply_distractor(d)


def gpu_render(torch, pxr, w, step0=0, env0=0, threads=None, scene=None):
    own = scene is None
    if own:
        scene = pxr.Scene(w["desc"])
    if threads:
        scene.set_block_threads(threads)
    _bind(torch, scene, w["distractor"])
    poses = torch.from_numpy(w["poses"]).cuda()
    shapes = None if w["shapes"] is None else torch.from_numpy(w["shapes"]).cuda()
    frames, ids = scene.render_batch(poses, shapes, step0=step0, env0=env0, want_ids=True)
    torch.cuda.synchronize()
    out = dict(frames=frames.cpu().numpy(), ids=pxr.ids_to_numpy(ids))
    if own:
        scene.close()
    return out


def assert_parity(got, ref, exact_rgb=True):
    assert got["ids"].shape == ref["ids"].shape and got["frames"].shape == ref["frames"].shape
    bad = np.argwhere(got["ids"] != ref["ids"])
    assert len(bad) == 0, f"{len(bad)} id mismatches, first at {bad[0]}: gpu {got['ids'][tuple(bad[0])]:#x} oracle {ref['ids'][tuple(bad[0])]:#x}"
    diff = np.abs(got["frames"].astype(np.int16) - ref["frames"].astype(np.int16))
    assert diff.max() <= 1, f"RGB differs by {diff.max()} LSB at {np.argwhere(diff > 1)[0]}"
    if exact_rgb:
        assert diff.max() == 0, f"{int((diff > 0).sum())} channels differ by 1 LSB"


def oracle_render(orc, w, step0=0, env0=0):
    s = orc.Scene(w["desc"])
    return s.render(w["poses"], w["shapes"], step0=step0, env0=env0, distractor=w["distractor"])


# ---------------------------------------------------------------- the five configurations

@pytest.mark.parametrize("cfg,B,threads", [(1, 16, 256), (1, 16, 1024), (2, 48, 512), (2, 24, 256), (3, 40, 512),
                                           (3, 24, 1024), (3, 17, 768), (4, 24, 1024), (4, 16, 512), (5, 20, 512), (5, 12, 256)])
def test_configs_match_oracle(torch, pxr, orc, cfg, B, threads):
    w = wl.make(cfg, B=B)
    got = gpu_render(torch, pxr, w, step0=3, env0=11, threads=threads)
    ref = oracle_render(orc, w, step0=3, env0=11)
    assert_parity(got, ref)
    tri = ref["ids"] < GROUND
    assert tri.any() and (ref["ids"] == GROUND).any() and (ref["ids"] == BG).any()


# (scene, width, height, distractor, workgroups that a compute unit's LDS holds, threads by the frames per compute unit).  The LDS is handed out in
# steps of 1280 bytes: 32 to 33 KB (capsules of 56x56, chains of 32x32) are four workgroups.
@pytest.mark.parametrize("scene,w,h,mode,in_lds,sizes", [
    ("capsules", 32, 32, "none", 10, {1: 512, 2: 512, 3: 256, 4: 256, 5: 256, 7: 256}),
    ("capsules", 47, 48, "color", 6, {1: 512, 2: 512, 3: 512, 4: 256, 5: 256, 7: 256}),
    ("capsules", 56, 56, "video", 4, {1: 512, 2: 512, 4: 512, 5: 512, 7: 512}),
    ("chain", 32, 32, "color", 4, {1: 1024, 2: 512, 3: 512, 4: 512, 5: 512, 7: 512}),
    ("chain", 41, 41, "video", 4, {1: 1024, 2: 512, 4: 512, 5: 512}),
    ("mesh", 28, 28, "video", 6, {1: 1024, 2: 512, 4: 512, 5: 256, 6: 256, 7: 512}),
    ("mesh", 40, 40, "none", 5, {1: 1024, 2: 512, 4: 512, 5: 256, 6: 512, 7: 512}),
    ("mesh", 64, 64, "color", 3, {1: 1024, 2: 512, 3: 512, 4: 512, 5: 512})])
def test_workgroup_size_by_frames_per_compute_unit(torch, pxr, scene, w, h, mode, in_lds, sizes):
    """Scenes of which three and more workgroups fit a compute unit: the size of a launch's workgroups follows its frames per compute
    unit, and whatever the size, a frame's bytes and ids are those of 768 threads, which no rule chooses here."""
    n_cus = torch.cuda.get_device_properties(0).multi_processor_count
    n = max(sizes) * n_cus
    make = {"capsules": wl.cfg1, "chain": wl.cfg2, "mesh": wl.cfg_mesh}[scene]
    work = make(n)
    sc = pxr.Scene(dict(work["desc"], width=w, height=h))
    assert 128 // -(-sc.info()["lds_bytes"] // 1280) == in_lds
    if mode == "video":
        clip = torch.from_numpy(np.random.default_rng(h).integers(0, 256, (5, h, w, 3), dtype=np.uint8)).cuda()
        sc.apply_distractor(dict(mode="video", seed=4, alpha=0.5, video=clip))
    elif mode == "color":
        sc.apply_distractor(dict(mode="color", seed=4, scale=(0.5, 1.5), offset=(-0.2, 0.2)))
    else:
        sc.apply_distractor(None)
    poses = torch.from_numpy(work["poses"]).cuda()
    sc.set_block_threads(768)
    ref, ref_ids = sc.render_batch(poses, want_ids=True)
    assert captured_kernels(torch, lambda: sc.render_batch(poses[:3], frames=ref[:3])) == [(768, 3)]
    sc.set_block_threads(0)
    for per_cu, threads in sizes.items():
        for batch in (1 if per_cu == 1 else (per_cu - 1) * n_cus + 1, per_cu * n_cus):
            frames, ids = torch.zeros_like(ref[:batch]), torch.zeros_like(ref_ids[:batch])
            assert captured_kernels(torch, lambda: sc.render_batch(poses[:batch], frames=frames, ids=ids)) == [(threads, batch)]
            sc.render_batch(poses[:batch], frames=frames, ids=ids)
            torch.cuda.synchronize()
            assert torch.equal(frames, ref[:batch]) and torch.equal(ids, ref_ids[:batch]), batch
    sc.close()


def test_default_block_threads_and_info(torch, pxr, orc):
    for cfg in (1, 2, 3, 4, 5):
        w = wl.make(cfg, B=2)
        sc = pxr.Scene(w["desc"])
        info = sc.info()
        o = orc.Scene(w["desc"])
        assert (info["n_verts"], info["n_tris"]) == (o.V, o.T)
        assert info["block_threads"] in (256, 512, 768, 1024) and info["lds_bytes"] <= 160 * 1024
        got = gpu_render(torch, pxr, w, scene=sc)
        assert_parity(got, oracle_render(orc, w))
        sc.close()


# ---------------------------------------------------------------- structure of the path

def test_determinism_and_slice_and_step_split(torch, pxr, orc):
    w = wl.make(5, B=24)
    a = gpu_render(torch, pxr, w, step0=7, env0=100)
    b = gpu_render(torch, pxr, w, step0=7, env0=100)
    assert np.array_equal(a["frames"], b["frames"]) and np.array_equal(a["ids"], b["ids"])
    # one env alone, with its global index
    e = 13
    one = dict(w, poses=w["poses"][e:e + 1], shapes=w["shapes"][e:e + 1])
    c = gpu_render(torch, pxr, one, step0=7, env0=100 + e)
    assert np.array_equal(c["frames"][0], a["frames"][e]) and np.array_equal(c["ids"][0], a["ids"][e])
    # steps 7,8,9 in one call == step 7 then steps 8,9
    first = dict(w, poses=np.ascontiguousarray(w["poses"][:, :1]))
    rest = dict(w, poses=np.ascontiguousarray(w["poses"][:, 1:]))
    f0 = gpu_render(torch, pxr, first, step0=7, env0=100)
    f1 = gpu_render(torch, pxr, rest, step0=8, env0=100)
    assert np.array_equal(np.concatenate([f0["frames"], f1["frames"]], axis=1), a["frames"])


def test_block_size_does_not_change_output(torch, pxr):
    w = wl.make(4, B=20)
    outs = [gpu_render(torch, pxr, w, threads=t) for t in (256, 512, 768, 1024)]
    for o in outs[1:]:
        assert np.array_equal(o["frames"], outs[0]["frames"]) and np.array_equal(o["ids"], outs[0]["ids"])


def test_batch_sizes_around_the_xcd_remap(torch, pxr, orc):
    """Frame <-> workgroup renumbering must be a bijection for every grid size modulo 8."""
    base = wl.make(3, B=41)
    ref = oracle_render(orc, base)
    for B in (1, 2, 7, 8, 9, 15, 16, 17, 33, 41):
        w = dict(base, poses=base["poses"][:B])
        got = gpu_render(torch, pxr, w)
        assert_parity(got, dict(frames=ref["frames"][:B], ids=ref["ids"][:B]))


# ---------------------------------------------------------------- image shapes

@pytest.mark.parametrize("W,H", [(8, 8), (33, 27), (40, 24), (127, 9), (128, 128), (31, 31), (84, 84), (9, 128)])
def test_image_shapes_including_unpacked_store_path(torch, pxr, orc, W, H):
    """W*H not a multiple of 4 takes the byte-store epilogue; 128x128 is the largest frame."""
    w = wl.make(3, B=6)
    w["desc"]["width"], w["desc"]["height"] = W, H
    assert_parity(gpu_render(torch, pxr, w, step0=2), oracle_render(orc, w, step0=2))
    rng = np.random.default_rng(W * 131 + H)
    video = rng.integers(0, 256, (7, H, W, 3), dtype=np.uint8)
    w["distractor"] = dict(mode="video", seed=5, video=video, alpha=0.5, env_offset=None)
    assert_parity(gpu_render(torch, pxr, w, step0=2), oracle_render(orc, w, step0=2))


@pytest.mark.parametrize("cfg,W,H,B", [(5, 256, 256, 3), (4, 200, 312, 2), (3, 512, 512, 2), (2, 500, 36, 3), (5, 132, 130, 3),
                                       (3, 250, 300, 2), (4, 86, 90, 3), (5, 96, 96, 4), (5, 192, 160, 2), (4, 84, 100, 3)])
def test_frames_larger_than_one_key_buffer(torch, pxr, orc, cfg, W, H, B):
    """Up to 512x512: the pixel keys are held a band of rows at a time.  Two or three bands of half a compute unit's
    LDS (a first band of whole resolve trips where there are two), or, from six bands on, all of the LDS and bands
    that pick their own triangles; widths that are no multiple of 4 take the byte-store loop, which clears its keys
    behind itself as well."""
    w = wl.make(cfg, B=B)
    w["desc"]["width"], w["desc"]["height"] = W, H
    if w["distractor"] is not None and w["distractor"]["mode"] == "video":
        rng = np.random.default_rng(W + H)
        w["distractor"] = dict(w["distractor"], video=rng.integers(0, 256, (5, H, W, 3), dtype=np.uint8))
    ref = oracle_render(orc, w, step0=1)
    assert (ref["ids"] < GROUND).mean() > 0.001
    assert_parity(gpu_render(torch, pxr, w, step0=1), ref)


def _scattered(W, H, rng, B=6):
    """Bodies of every kind around the camera: in view, cut by each edge of the frame, outside it, behind the camera and
    (last environment) nothing in view at all; quaternions of any length, shapes of either sign."""
    bodies = [wl.capsule(0.1, 0.25, (0.8, 0.3, 0.3), 7, 3), wl.sphere(0.2, (0.3, 0.8, 0.3), 9, 4), wl.box(0.15, 0.1, 0.2, (0.3, 0.3, 0.8), 2)]
    tv, tt = wl.torus_mesh(0.3, 0.1, 9, 6)
    bodies.append(wl.mesh(tv, tt, (0.7, 0.7, 0.2), scale=(1.0, 1.5, 0.5)))
    poses = np.zeros((B, 1, 4, 7), np.float32)
    poses[:, 0, 0, :3] = (0, 0, 1)
    spread = np.array([[0.3], [1.0], [2.0], [4.0], [1.5], [0.0]])[:B, :, None]
    poses[:, 0, :, :3] += (spread * rng.uniform(-1.0, 1.0, (B, 4, 3))).astype(np.float32)
    poses[:, 0, 0, :3] = (0, 0, 1)  # (the root: the camera stays where it is)
    poses[:, 0, :, 3:] = wl.random_quats(rng, (B, 4)) * rng.uniform(0.6, 1.5, (B, 4, 1))
    shapes = np.array([b["shape"] for b in bodies], np.float32)[None] * rng.choice([-1.0, 1.0], (B, 4, 4)).astype(np.float32)
    shapes[:, 0] = np.abs(shapes[:, 0])
    poses[5, 0, 1:, 0] = -20.0 - np.arange(3)  # behind the camera ...
    shapes[5, 0] = 0.0                         # ... and a root without extent
    return dict(desc=wl.default_scene(W, H, bodies), poses=poses, shapes=np.ascontiguousarray(shapes), distractor=None)


@pytest.mark.parametrize("W,H", [(84, 120), (161, 160), (162, 90), (163, 200), (260, 8), (9, 300), (320, 200), (511, 130)])
@pytest.mark.parametrize("mode", ["none", "color", "video"])
def test_key_window_of_large_frames(torch, pxr, orc, W, H, mode):
    """Frames whose keys do not fit the LDS keep those of the pixels that the bodies can touch: every place such a window
    can have (inside, cut by each edge, the whole frame, nothing), rows in several bands, widths with a remainder.  (The two
    smallest sizes keep all keys.)"""
    w = _scattered(W, H, np.random.default_rng(W * 1000 + H))
    assert _windowed(pxr, w["desc"]) == (min(W, H) > 9)
    if mode == "color":
        w["desc"]["cam_up"] = (0.1, 0.2, 1.0)
        w["distractor"] = dict(mode="color", seed=3, scale=(0.5, 1.5), offset=(-0.2, 0.2))
    if mode == "video":
        video = np.random.default_rng(1).integers(0, 256, (3, H, W, 3), dtype=np.uint8)
        w["distractor"] = dict(mode="video", seed=5, video=video, alpha=0.5, env_offset=None)
    ref = oracle_render(orc, w, step0=1)
    assert (ref["ids"] < GROUND).any() and (ref["ids"][5] >= GROUND).all()
    assert_parity(gpu_render(torch, pxr, w, step0=1), ref)
    assert_parity(gpu_render(torch, pxr, w, step0=1, threads=256), ref)


@pytest.mark.parametrize("exponent", [99, 100, 124, 125, -100, -128])
def test_key_window_at_the_ends_of_the_float_range(torch, pxr, orc, exponent):
    """Scenes in units of 2^99 m and more, 2^-100 m and less: multiplied by a power of two every step of the geometry is
    the same, but reciprocals of depths vanish or overflow.  (From 2^125 on the windows once cut pixels off: the
    hardware's reciprocal of a depth beyond 2^126 is 0.)"""
    w = _scattered(256, 200, np.random.default_rng(5))
    unit = np.float32(2.0 ** exponent)
    w["poses"][..., :3] = np.float32([0, 0, 1]) + np.float32(0.45) * (w["poses"][..., :3] - np.float32([0, 0, 1]))
    w["poses"][5, 0, 1:, 0] = -3.1  # (still behind the camera)
    w["poses"][..., :3] *= unit  # (a few units from the origin: nothing overflows)
    w["shapes"] = w["shapes"] * unit
    d = w["desc"]
    d["cam_offset"] = tuple(float(np.float32(c) * unit) for c in d["cam_offset"])
    d["z_near"], d["z_far"] = float(np.float32(d["z_near"]) * unit), min(50.0 * 2.0 ** exponent, 3e38)
    assert np.isfinite(w["poses"]).all()
    ref = oracle_render(orc, w)
    assert ((ref["ids"][:5] < GROUND).sum(axis=(1, 2, 3)) > 300).all()
    assert_parity(gpu_render(torch, pxr, w), ref)


@pytest.mark.parametrize("W,H,video", [(256, 256, False), (163, 200, True), (84, 84, True), (300, 37, False)])
def test_large_frames_shared_by_workgroups_or_not(torch, pxr, orc, W, H, video):
    """Small batches give a large frame's rows to several workgroups, large ones a frame to each: the same frames, and the
    oracle's.  (84x84 frames of this scene keep all their keys and are not shared.)"""
    w = _scattered(W, H, np.random.default_rng(W + H))
    assert _windowed(pxr, w["desc"]) == (W * H > 84 * 84)
    if video:
        clip = np.random.default_rng(2).integers(0, 256, (3, H, W, 3), dtype=np.uint8)
        w["distractor"] = dict(mode="video", seed=5, video=clip, alpha=0.5, env_offset=np.zeros(6, np.uint32))
    ref = oracle_render(orc, w)
    for copies in (1, 3, 14, 50):  # 6, 18, 84 and 300 frames: 32, 8, 2 and no slabs at 256x256, 8, 8, 2 and none at 300x37
        many = dict(w, poses=np.tile(w["poses"], (copies, 1, 1, 1)), shapes=np.tile(w["shapes"], (copies, 1, 1)))
        if video:
            many["distractor"] = dict(w["distractor"], env_offset=np.zeros(6 * copies, np.uint32))
        got = gpu_render(torch, pxr, many)
        assert_parity(dict(frames=got["frames"][:6], ids=got["ids"][:6]), ref)
        assert np.array_equal(got["frames"], np.tile(got["frames"][:6], (copies, 1, 1, 1, 1)))
        assert np.array_equal(got["ids"], np.tile(got["ids"][:6], (copies, 1, 1, 1)))


@pytest.mark.parametrize("cells,W,H", [(16, 320, 320), (20, 256, 256), (20, 512, 400), (30, 384, 384)])
def test_bands_of_a_frame_with_nearly_every_triangle_binned(torch, pxr, orc, cells, W, H):
    """Open terrain below the camera: more than half of its triangles face it and hold pixels, so what the bins leave
    free of their arrays is too short for a band's own lists, or just long enough."""
    rng = np.random.default_rng(cells)
    hv, ht, hm = wl.heightfield_mesh(rng, cells, 3.0, 0.1)
    bodies = [wl.sphere(0.1, (0.6, 0.4, 0.8), 6, 2), wl.mesh(hv, ht, (0.7, 0.6, 0.4), mul=hm)]
    B = 3
    poses = np.zeros((B, 1, 2, 7), np.float32)
    poses[:, 0, :, 3] = 1
    poses[:, 0, 0, :3] = (0, 0, 1)
    poses[:, 0, 1, :3] = np.array([[0, 0, 0.1], [0.6, 0.1, 0.3], [-0.9, 0, 0.2]])
    d = wl.default_scene(W, H, bodies)
    d["cam_offset"] = (-1.2, 0.0, 2.0)
    w = dict(desc=d, poses=poses, shapes=None, distractor=None)
    ref = oracle_render(orc, w)
    assert (ref["ids"] < GROUND).mean() > 0.3
    for threads in (None, 256, 768):
        assert_parity(gpu_render(torch, pxr, w, threads=threads), ref)


def _windowed(pxr, desc):
    """Whether the scene's frames keep a window of their keys: with all of them, its LDS would be larger than it is."""
    sc = pxr.Scene(desc)
    info = sc.info()
    sc.close()
    W, H, K, V, T = desc["width"], desc["height"], len(desc["bodies"]), info["n_verts"], info["n_tris"]
    up = lambda n, a: -(-n // a) * a
    return info["lds_bytes"] < up(W, 4) * H * 8 + up(4 * (W + H), 16) + 16 * H + 256 + 96 * K + 12 * V + 2 * up(2 * T, 4)


@pytest.mark.parametrize("W,H,lat", [(12, 512, 10), (9, 512, 10), (12, 512, 11), (64, 300, 12), (130, 64, 13), (300, 64, 13)])
@pytest.mark.parametrize("mode", ["color", "video"])
def test_key_window_of_scenes_at_the_lds_limit(torch, pxr, orc, W, H, lat, mode):
    """More than 5300 vertices: frames three groups of pixels wide are windowed, and from 11 rings on there is no room for
    the blend tables behind the keys."""
    bodies = [wl.sphere(0.3, (0.7, 0.4, 0.3), 64, 32), wl.capsule(0.15, 0.3, (0.3, 0.6, 0.8), 64, lat)]
    rng = np.random.default_rng(W + lat)
    B = 5
    poses = np.zeros((B, 1, 2, 7), np.float32)
    poses[:, 0, :, 3:] = wl.random_quats(rng, (B, 2))
    poses[:, 0, 0, :3] = (0, 0, 1)
    poses[:, 0, 1, :3] = np.array([0.0, 0.0, 1.0]) + np.array([[0, 0, 0.5], [-1, 0, 0.4], [-2.4, 0, 1], [0, 9, 0], [-9, 0, 0]])
    w = dict(desc=wl.default_scene(W, H, bodies), poses=poses, shapes=None)
    if mode == "color":
        w["distractor"] = dict(mode="color", seed=3, scale=(0.5, 1.5), offset=(-0.2, 0.2))
    else:
        w["distractor"] = dict(mode="video", seed=5, video=rng.integers(0, 256, (3, H, W, 3), dtype=np.uint8), alpha=0.5, env_offset=None)
    assert _windowed(pxr, w["desc"])
    ref = oracle_render(orc, w, step0=1)
    assert (ref["ids"] < GROUND).any(axis=(1, 2, 3)).all()
    assert_parity(gpu_render(torch, pxr, w, step0=1), ref)
    assert_parity(gpu_render(torch, pxr, w, step0=1, threads=256), ref)


@pytest.mark.parametrize("W,H", [(256, 256), (163, 130)])
def test_key_window_with_non_finite_and_collapsed_poses(torch, pxr, orc, W, H):
    """The inputs of test_rejected_and_degenerate_inputs in windowed frames: NaN and infinite positions and quaternions,
    bodies behind the camera, through the near plane, without extent, far to a side."""
    w = wl.make(2, B=14)
    w["desc"].update(width=W, height=H)
    assert _windowed(pxr, w["desc"])
    p = w["poses"].copy()
    p[0, 0, 0, 0] = np.nan
    p[1, 0, 1:, 0] = -5.0
    p[2, 0, 3, :3] = np.nan
    p[3, 0, 2, 3:] = np.nan
    p[4, 0, 0, 2] = -3.0
    p[5, 0, 4, :3] = p[5, 0, 0, :3] + np.array([-2.45, 0, 1.0], np.float32)
    p[6, 0, :, 3:] = 0.0
    p[7, 0, 5, 1] = 1e6
    p[8, 0, 3, 0] = np.inf
    p[9, 0, 3, 2] = -np.inf
    p[10, 0, 2, 4] = np.inf
    p[11, 0, 2, 3:] *= 1e19     # (the rotation's entries overflow)
    p[12, 0, 1, 3:] *= 1e-25    # (its squares vanish)
    p[13, 0, 2:5, 3] = np.nan
    w["poses"] = p
    assert_parity(gpu_render(torch, pxr, w), oracle_render(orc, w))


def test_key_window_of_sixty_four_bodies(torch, pxr, orc):
    """Bodies past the sixteen that a wavefront bounds at a time decide the window."""
    rng = np.random.default_rng(64)
    bodies = [[wl.capsule(0.05, 0.12, (0.8, 0.3, 0.3), 5, 2), wl.sphere(0.08, (0.3, 0.8, 0.3), 6, 2), wl.box(0.07, 0.05, 0.06, (0.3, 0.3, 0.8), 1)][k % 3]
              for k in range(64)]
    B = 64
    poses = np.zeros((B, 1, 64, 7), np.float32)
    poses[..., :3] = np.array([0.0, 0.0, 1.0]) + rng.uniform(-0.1, 0.1, (B, 1, 64, 3))
    for e in range(B):  # one body a long way from the others, another one in each environment
        poses[e, 0, e, :3] += np.array([0.2, 0.9 * (-1) ** e, 0.5])
    poses[..., 3:] = wl.random_quats(rng, (B, 1, 64))
    w = dict(desc=wl.default_scene(200, 160, bodies, root_body=63), poses=poses, shapes=None, distractor=None)
    assert _windowed(pxr, w["desc"])
    ref = oracle_render(orc, w)
    assert_parity(gpu_render(torch, pxr, w), ref)


def test_video_frames_of_84_pixels_shared_by_workgroups(torch, pxr, orc):
    """84x84 frames of a humanoid are windowed: 5 of them are shared by 16 workgroups each, 300 are not shared."""
    w = wl.make(4, B=5)
    assert _windowed(pxr, w["desc"])
    w["distractor"] = dict(w["distractor"], env_offset=np.zeros(5, np.uint32))
    ref = oracle_render(orc, w, step0=3)
    assert_parity(gpu_render(torch, pxr, w, step0=3), ref)
    many = dict(w, poses=np.tile(w["poses"], (60, 1, 1, 1)), distractor=dict(w["distractor"], env_offset=np.zeros(300, np.uint32)))
    got = gpu_render(torch, pxr, many, step0=3)
    assert np.array_equal(got["frames"], np.tile(ref["frames"], (60, 1, 1, 1, 1))) and np.array_equal(got["ids"], np.tile(ref["ids"], (60, 1, 1, 1)))


def test_close_up_at_512(torch, pxr, orc):
    """Triangles hundreds of pixels wide crossing many bands."""
    rng = np.random.default_rng(77)
    B = 2
    poses = np.zeros((B, 1, 3, 7), np.float32)
    poses[:, 0, 0, :3] = (0, 0, 1)
    poses[:, 0, 0, 3:] = wl.random_quats(rng, (B,))
    for b in (1, 2):
        poses[:, 0, b, :3] = np.array([0, 0, 1]) + rng.uniform(-0.5, 0.5, (B, 3))
        poses[:, 0, b, 3:] = wl.random_quats(rng, (B,))
    w = dict(desc=_close_up(512, 384), poses=poses, shapes=None, distractor=None)
    ref = oracle_render(orc, w)
    assert (ref["ids"] < GROUND).mean() > 0.3
    assert_parity(gpu_render(torch, pxr, w), ref)


# ---------------------------------------------------------------- caller-supplied meshes

@pytest.mark.parametrize("W,H,threads", [(64, 64, None), (61, 64, 256), (256, 256, None)])
def test_corners_on_and_beside_pixel_centres(torch, pxr, orc, W, H, threads):
    """Every triangle over a 3 x 3 lattice of half pixels, in both orientations, wherever its corners lie on pixel centres and wherever
    between them: which centres its ends may cover, and which triangles are left out unseen, is the fill rule's matter alone."""
    lattice = [(x, y) for y in range(3) for x in range(3)]
    tris = [t for t in itertools.permutations(range(9), 3)
            if t[0] == min(t) and np.linalg.det([(*lattice[k], 1.0) for k in t]).round() != 0]
    assert len(tris) == 152
    # a view straight along x with a focal length of H / 2: at depth 2 a world unit is H / 4 pixels, a power of two, so every corner is
    # exactly where it is put
    depth, per_pixel = 2.0, 4.0 / H
    verts = []
    for n, (t, dx, dy) in enumerate(itertools.product(tris, (0.0, 0.5), (0.0, 0.5))):  # (a centre in the middle, at the sides, at the corners)
        for corner in t:
            px = 0.5 * lattice[corner][0] + 2 * (n % 29) + 1 + dx
            py = 0.5 * lattice[corner][1] + 2 * (n // 29) + 1 + dy
            verts.append((0.0, -(px - W / 2) * per_pixel, -(py - H / 2) * per_pixel))
    idx = np.arange(len(verts), dtype=np.uint32).reshape(-1, 3)
    d = wl.default_scene(W, H, [wl.mesh(np.array(verts, np.float32), idx, (0.8, 0.5, 0.3))])
    d.update(cam_offset=(-depth, 0.0, 0.0), fov_y_deg=90.0)
    poses = np.zeros((2, 1, 1, 7), np.float32)
    poses[..., 2], poses[..., 3] = 1.0, 1.0
    w = dict(desc=d, poses=poses, shapes=None, distractor=None)
    ref = oracle_render(orc, w)
    seen = np.unique(ref["ids"][ref["ids"] < GROUND])
    assert 60 < len(seen) < 150
    assert_parity(gpu_render(torch, pxr, w, threads=threads), ref)


@pytest.mark.parametrize("threads", [None, 256])
def test_slivers_at_the_limit_of_24_bit_edges(torch, pxr, orc, threads):
    """Thin triangles of 2^15 - 1, 2^15 and 2^15 + 1 sub-pixels' extent, along x, along y and diagonally, few pixels wide: up to 2^15 - 1 their
    edge functions are 24-bit products, beyond that 64-bit ones.  (Most show many pixels; few and none, and smaller frames: the next test.)"""
    W = H = 256
    per_pixel = 4.0 / H  # (as above: corners are exactly where they are put, here in 1/256 pixels)
    verts, n = [], 0
    for extent, way, width in itertools.product((32767, 32768, 32769), ((1, 0), (0, 1), (1, 1), (1, -1)), (77, 300, 1100)):
        x0 = 256 * (4 + 3 * n) + 37 * n
        y0 = 256 * (200 if way[1] < 0 else 4 + 2 * n) + 91 * n
        corners = [(x0, y0), (x0 + way[0] * extent, y0 + way[1] * extent), (x0 + (width if way[0] == 0 or way[1] else extent // 2), y0 + (0 if way[1] else width))]
        for k in (0, 1, 2) + (0, 2, 1):  # (one of the two faces the camera)
            verts.append((0.0, -(corners[k][0] / 256 - W / 2) * per_pixel, -(corners[k][1] / 256 - H / 2) * per_pixel))
        n += 1
    idx = np.arange(len(verts), dtype=np.uint32).reshape(-1, 3)
    d = wl.default_scene(W, H, [wl.mesh(np.array(verts, np.float32), idx, (0.8, 0.5, 0.3))])
    d.update(cam_offset=(-2.0, 0.0, 0.0), fov_y_deg=90.0)
    poses = np.zeros((2, 1, 1, 7), np.float32)
    poses[..., 2], poses[..., 3] = 1.0, 1.0
    w = dict(desc=d, poses=poses, shapes=None, distractor=None)
    ref = oracle_render(orc, w)
    assert len(np.unique(ref["ids"][ref["ids"] < GROUND])) > 24
    assert_parity(gpu_render(torch, pxr, w, threads=threads), ref)


def _exact_scene(W, H, triangles):
    """Frames of W x H (H a power of two) of one mesh whose triangles' corners come out exactly where `triangles` [n, 3, 2] has them, in 1/256 pixels; one of each
    triangle's two sides faces the camera, both are there."""
    t = np.asarray(triangles, np.float64)[:, [[0, 1, 2], [0, 2, 1]]].reshape(-1, 2) / 256
    # a view straight along x with a focal length of H / 2: at depth 2 a world unit is H / 4 pixels, a power of two
    verts = np.stack([np.zeros(len(t)), -(t[:, 0] - W / 2) * 4.0 / H, -(t[:, 1] - H / 2) * 4.0 / H], axis=1).astype(np.float32)
    d = wl.default_scene(W, H, [wl.mesh(verts, np.arange(len(verts), dtype=np.uint32).reshape(-1, 3), (0.8, 0.5, 0.3))])
    d.update(cam_offset=(-2.0, 0.0, 0.0), fov_y_deg=90.0)
    poses = np.zeros((2, 1, 1, 7), np.float32)
    poses[..., 2], poses[..., 3] = 1.0, 1.0
    return dict(desc=d, poses=poses, shapes=None, distractor=None)


def _bins(X, Y, W, H):
    """What the raster phase makes of visible triangles with these snapped corners [n, 3]: (wide?, bin by candidate pixels 0 tiny, 1 small, 2 large)."""
    X, Y, n = X.astype(np.int64), Y.astype(np.int64), 1
    for c, size in ((X, W), (Y, H)):  # (centre i at 256 i + 128; one at the far end is not covered)
        n = n * np.maximum(0, np.minimum(size, (c.max(1) + 127) >> 8) - np.maximum(0, (c.min(1) + 127) >> 8))
    wide = np.maximum(np.ptp(X, axis=1), np.ptp(Y, axis=1)) >= 1 << 15
    assert np.all(n > 0)
    return {(bool(a), int(b)) for a, b in zip(wide, np.digitize(n, [4, 129]))}


@pytest.mark.parametrize("W,H,threads", [(64, 64, None), (64, 64, 256), (61, 64, 512), (256, 256, None), (256, 256, 256)])
def test_slivers_that_reach_into_the_frame(torch, pxr, orc, W, H, threads):
    """Slivers of 2^15 - 1, 2^15 and 2^15 + 1 sub-pixels' extent that reach into the frame from every side and corner, by one to three pixels, by up to 128 and by more: up
    to 2^15 - 1 their edge functions are 24-bit products, beyond that they take the 64-bit path, in the frames that are kept whole and in those that are not."""
    tris = []
    # (the smaller ones first and beside each other: of triangles at the same depth the first shows)
    for m, ((reach, thick), extent) in enumerate(itertools.product(((330, 250), (700, 256), (4000, 600), (15000, 1500)), (32767, 32768, 32769))):
        for mirror_x, mirror_y, turn in itertools.product((0, 1), (0, 1), (0, 1, 2)):
            at = 256 * 3 + 601 * m
            tip, end, side = (reach, at), (reach - extent, at), (reach - 90 * (extent % 4), at + thick)
            if turn == 2:  # along a diagonal, across the frame's corner
                tip, end, side = (reach, reach), (reach - extent, reach - extent), (reach - 90, reach - 1 - thick)
            corners = [(y, x) if turn == 1 else (x, y) for x, y in (tip, end, side)]
            tris.append([(256 * W - x if mirror_x else x, 256 * H - y if mirror_y else y) for x, y in corners])
    w = _exact_scene(W, H, tris)
    scene = orc.Scene(w["desc"])
    snapped = scene.vertex_stage(w["poses"][0, 0])
    X, Y = (np.asarray(snapped[k]).reshape(-1, 3) for k in "XY")
    assert not np.any(snapped["rejected"]) and np.array_equal(np.stack([X[::2], Y[::2]], axis=-1), np.array(tris))
    ref = oracle_render(orc, w)
    seen = np.unique(ref["ids"][ref["ids"] < GROUND])
    assert _bins(X[seen], Y[seen], W, H) == set(itertools.product((False, True), (0, 1, 2)))
    assert_parity(gpu_render(torch, pxr, w, threads=threads), ref)


@pytest.mark.parametrize("side", [64, 256])
def test_wide_triangles_that_show_few_pixels_take_few_lanes(torch, pxr, orc, side):
    """400 long triangles end a pixel or two inside the frame: those of 128 pixels and more (64-bit edges) cost about what shorter ones do.  (With a turn of a whole
    wavefront for each, five times as much at 64x64 and nearly twice at 256x256.)"""
    us = {}
    for length in (100, 300):
        tris = []
        for n in range(400):
            at = 256 * 3 + (n * 256 * (side - 8)) // 400
            corners = [(400 - 256 * length, at), (400 - 256 * length, at + 300), (400, at + 150)]
            tris.append([((x, y), (256 * side - x, y), (y, x), (y, 256 * side - x))[n % 4] for x, y in corners])
        w = _exact_scene(side, side, tris)
        assert_parity(gpu_render(torch, pxr, w), oracle_render(orc, w))
        scene = pxr.Scene(w["desc"])
        poses = torch.from_numpy(w["poses"]).cuda().repeat(1024 if side == 64 else 256, 1, 1, 1)
        frames, _ = scene.render_batch(poses)
        times = []
        for _ in range(5):
            begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            begin.record()
            for _ in range(10):
                scene.render_batch(poses, frames=frames)
            end.record()
            torch.cuda.synchronize()
            times.append(begin.elapsed_time(end) * 100.0)
        us[length] = min(times)
        scene.close()
    print("us per launch by length:", us)
    assert us[300] < (2.0 if side == 64 else 1.4) * us[100], us


@pytest.mark.parametrize("W,H,B,threads", [(64, 64, 40, None), (84, 84, 17, 512), (32, 32, 24, 256), (200, 160, 5, None)])
def test_mesh_bodies_match_oracle(torch, pxr, orc, W, H, B, threads):
    w = wl.cfg_mesh(B=B, W=W, H=H)
    ref = oracle_render(orc, w, step0=2, env0=5)
    for lo, hi in [(0, 288), (288, 688), (688, 1008), (1008, 1296)]:
        assert ((ref["ids"] >= lo) & (ref["ids"] < hi)).any()
    assert_parity(gpu_render(torch, pxr, w, step0=2, env0=5, threads=threads), ref)


def test_mesh_close_up_and_degenerate_triangles(torch, pxr, orc):
    """Mesh triangles tens of pixels wide, a mesh with zero-area and repeated-vertex triangles, per-env scales."""
    rng = np.random.default_rng(12)
    tv, tt = wl.torus_mesh(0.35, 0.15, 7, 5)
    fan_v = np.array([[0, 0, 0]] + [[0.4 * np.cos(a), 0.4 * np.sin(a), 0.05 * a] for a in np.linspace(0, 5, 8)], np.float32)
    fan_t = np.array([[0, i, i + 1] for i in range(1, 8)] + [[0, i + 1, i] for i in range(1, 8)] + [[3, 3, 4], [5, 6, 5]], np.uint32)
    hv, ht, hm = wl.heightfield_mesh(rng, 5, 1.2, 0.4)
    bodies = [wl.mesh(tv, tt, (0.8, 0.5, 0.3)), wl.mesh(fan_v, fan_t, (0.3, 0.7, 0.5), mul=rng.uniform(0.3, 1.0, len(fan_t))),
              wl.mesh(hv, ht, (0.6, 0.6, 0.3), mul=hm)]
    d = wl.default_scene(96, 72, bodies)
    d["cam_offset"] = (-1.0, 0.1, 0.4)
    B = 20
    poses = np.zeros((B, 1, 3, 7), np.float32)
    poses[:, 0, 0, :3] = (0, 0, 1)
    poses[:, 0, 0, 3:] = wl.random_quats(rng, (B,))
    for b in (1, 2):
        poses[:, 0, b, :3] = np.array([0.1, 0, 1]) + rng.uniform(-0.5, 0.5, (B, 3))
        poses[:, 0, b, 3:] = wl.random_quats(rng, (B,))
    shapes = rng.uniform(0.6, 1.5, (B, 3, 4)).astype(np.float32)
    w = dict(desc=d, poses=poses, shapes=shapes, distractor=None)
    ref = oracle_render(orc, w)
    assert (ref["ids"] < GROUND).mean() > 0.25
    assert_parity(gpu_render(torch, pxr, w), ref)


# ---------------------------------------------------------------- maximum sizes

def test_sixty_four_bodies(torch, pxr, orc):
    """The body-count limit: 64 bodies of mixed kinds, per-environment shapes."""
    rng = np.random.default_rng(64)
    bodies = []
    for k in range(64):
        rgb = rng.uniform(0.2, 0.9, 3)
        bodies.append([wl.capsule(0.05, 0.12, rgb, 5, 2), wl.sphere(0.08, rgb, 6, 2), wl.box(0.07, 0.05, 0.06, rgb, 1)][k % 3])
    d = wl.default_scene(64, 48, bodies, root_body=63)
    B = 10
    poses = np.zeros((B, 1, 64, 7), np.float32)
    poses[..., :3] = np.array([0.0, 0.0, 1.0]) + rng.uniform(-0.9, 0.9, (B, 1, 64, 3)) * np.array([1.0, 1.0, 0.6])
    poses[..., 3:] = wl.random_quats(rng, (B, 1, 64))
    shapes = np.array([b["shape"] for b in bodies], np.float32)[None] * rng.uniform(0.7, 1.4, (B, 64, 1)).astype(np.float32)
    w = dict(desc=d, poses=poses, shapes=np.ascontiguousarray(shapes), distractor=None)
    ref = oracle_render(orc, w)
    assert len(np.unique(ref["ids"])) > 300
    assert_parity(gpu_render(torch, pxr, w), ref)


def test_scene_at_the_lds_limit(torch, pxr, orc):
    """The finest tessellation that still fits one compute unit's LDS (one workgroup per unit, many bands)."""
    bodies = [wl.sphere(0.5, (0.7, 0.4, 0.3), 64, 32), wl.capsule(0.2, 0.4, (0.3, 0.6, 0.8), 64, 8)]
    d = wl.default_scene(128, 96, bodies)
    d["cam_offset"] = (-1.8, 0.0, 0.5)
    sc = pxr.Scene(d)
    info = sc.info()
    assert info["lds_bytes"] > 120 * 1024 and info["n_verts"] > 5000 and info["n_tris"] > 10000
    rng = np.random.default_rng(65)
    B = 3
    poses = np.zeros((B, 1, 2, 7), np.float32)
    poses[:, 0, 0, :3] = (0, 0, 1)
    poses[:, 0, 0, 3:] = wl.random_quats(rng, (B,))
    poses[:, 0, 1, :3] = np.array([0.0, 0.6, 1.0]) + rng.uniform(-0.2, 0.2, (B, 3))
    poses[:, 0, 1, 3:] = wl.random_quats(rng, (B,))
    w = dict(desc=d, poses=poses, shapes=None, distractor=None)
    assert_parity(gpu_render(torch, pxr, w, scene=sc), oracle_render(orc, w))
    sc.close()


# ---------------------------------------------------------------- near-plane clipping

def _clip_scenes():
    RGB = (0.6, 0.4, 0.8)
    rng = np.random.default_rng(41)
    out = []
    # a terrain grid running under and behind the camera, 1 and 2 corners in front, several yaws
    hv, ht, hm = wl.heightfield_mesh(rng, 5, 9.0, 0.25)
    d = wl.default_scene(72, 56, [wl.sphere(0.05, RGB, 6, 2), wl.mesh(hv, ht, (0.7, 0.6, 0.4), mul=hm)])
    d["cam_offset"] = (-1.0, 0.0, 0.5)
    B = 12
    poses = np.zeros((B, 1, 2, 7), np.float32)
    poses[:, 0, 0] = (0, 0, 1, 1, 0, 0, 0)
    poses[:, 0, 1, :3] = np.array([-1.0, 0.0, 0.85]) + rng.uniform(-0.3, 0.3, (B, 3)) * np.array([1, 1, 0.2])
    poses[:, 0, 1, 3:] = wl.q_axis_angle(wl.EZ, rng.uniform(0, 2 * np.pi, B))
    out.append(dict(desc=d, poses=poses, shapes=None, distractor=None))
    # a long capsule and a big box passing the camera; colour distractor; tumbling
    bodies = [wl.sphere(0.05, RGB, 6, 2), wl.capsule(0.3, 3.0, (0.8, 0.3, 0.3), 10, 3), wl.box(0.8, 0.6, 0.4, (0.3, 0.5, 0.8), 3)]
    d = wl.default_scene(64, 64, bodies)
    d["cam_offset"] = (-1.5, 0.0, 0.4)
    B = 16
    poses = np.zeros((B, 1, 3, 7), np.float32)
    poses[:, 0, 0] = (0, 0, 1, 1, 0, 0, 0)
    poses[:, 0, 1, :3] = np.array([-1.0, 0.2, 1.1]) + rng.uniform(-0.4, 0.4, (B, 3))
    poses[:, 0, 1, 3:] = wl.random_quats(rng, (B,))
    poses[:, 0, 2, :3] = np.array([-1.2, -0.6, 1.2]) + rng.uniform(-0.4, 0.4, (B, 3))
    poses[:, 0, 2, 3:] = wl.random_quats(rng, (B,))
    out.append(dict(desc=d, poses=poses, shapes=None,
                    distractor=dict(mode="color", seed=3, scale=(0.5, 1.5), offset=(-0.2, 0.2))))
    # the camera inside a huge sphere and next to a huge box (everything visible is clipped or enormous)
    bodies = [wl.sphere(0.05, RGB, 6, 2), wl.sphere(3.0, (0.5, 0.7, 0.5), 12, 5), wl.box(2.0, 2.0, 0.05, (0.7, 0.7, 0.3), 4)]
    d = wl.default_scene(48, 40, bodies)
    d["cam_offset"] = (-0.8, 0.0, 0.3)
    B = 10
    poses = np.zeros((B, 1, 3, 7), np.float32)
    poses[:, 0, 0] = (0, 0, 1, 1, 0, 0, 0)
    poses[:, 0, 1, :3] = np.array([2.0, 0.0, 1.0]) + rng.uniform(-0.5, 0.5, (B, 3))
    poses[:, 0, 1, 3:] = wl.random_quats(rng, (B,))
    poses[:, 0, 2, :3] = np.array([-0.5, 0.0, 1.0]) + rng.uniform(-0.3, 0.3, (B, 3))
    poses[:, 0, 2, 3:] = wl.random_quats(rng, (B,))
    out.append(dict(desc=d, poses=poses, shapes=None, distractor=None))
    return out


@pytest.mark.parametrize("which", [0, 1, 2])
def test_triangles_crossing_the_near_plane_are_clipped(torch, pxr, orc, which):
    w = _clip_scenes()[which]
    o = orc.Scene(w["desc"])
    tris = o.mesh()["tris"]
    n_straddling = 0
    for e in range(w["poses"].shape[0]):
        behind = o.vertex_stage(w["poses"][e, 0])["rejected"] == 2
        n_straddling += int((behind[tris].any(axis=1) & ~behind[tris].all(axis=1)).sum())
    assert n_straddling > 20 * w["poses"].shape[0] // 4
    ref = oracle_render(orc, w, step0=1)
    assert (ref["ids"] < GROUND).mean() > 0.15
    for threads in (None, 256, 1024):
        assert_parity(gpu_render(torch, pxr, w, step0=1, threads=threads), ref)


def test_clipping_in_banded_frames(torch, pxr, orc):
    w = _clip_scenes()[1]
    w["desc"]["width"], w["desc"]["height"] = 260, 200
    w = dict(w, poses=w["poses"][:4])
    assert_parity(gpu_render(torch, pxr, w), oracle_render(orc, w))


# ---------------------------------------------------------------- large triangles, clipping, rejects

def _close_up(W=64, H=64, offset=(-0.9, 0.1, 0.35)):
    bodies = [wl.box(0.3, 0.25, 0.2, (0.8, 0.5, 0.3), 2), wl.capsule(0.15, 0.3, (0.2, 0.7, 0.4), 8, 3),
              wl.sphere(0.25, (0.5, 0.5, 0.9), 10, 4)]
    d = wl.default_scene(W, H, bodies)
    d["cam_offset"] = offset
    return d


def test_large_triangles_take_the_wave_path(torch, pxr, orc):
    rng = np.random.default_rng(101)
    B = 24
    poses = np.zeros((B, 1, 3, 7), np.float32)
    poses[:, 0, 0, :3] = (0, 0, 1)
    poses[:, 0, 0, 3:] = wl.random_quats(rng, (B,))
    for b in (1, 2):
        poses[:, 0, b, :3] = np.array([0, 0, 1]) + rng.uniform(-0.5, 0.5, (B, 3))
        poses[:, 0, b, 3:] = wl.random_quats(rng, (B,))
    for W, H in [(64, 64), (128, 128), (33, 27)]:
        w = dict(desc=_close_up(W, H), poses=poses, shapes=None, distractor=None)
        ref = oracle_render(orc, w)
        assert ((ref["ids"] < GROUND).mean() > 0.3)  # triangles tens of pixels wide
        assert_parity(gpu_render(torch, pxr, w), ref)


def test_huge_offscreen_extents_use_64bit_edges(torch, pxr, orc):
    """Camera almost touching a big box: snapped coordinates run to millions, products beyond 2^31."""
    bodies = [wl.sphere(0.05, (0.5, 0.5, 0.5), 8, 4), wl.box(3.0, 3.0, 0.5, (0.7, 0.6, 0.2), 3),
              wl.capsule(0.4, 2.0, (0.3, 0.6, 0.8), 6, 2)]
    d = wl.default_scene(64, 64, bodies)
    d["cam_offset"] = (-0.6, 0.0, 0.25)
    rng = np.random.default_rng(103)
    B = 16
    poses = np.zeros((B, 1, 3, 7), np.float32)
    poses[:, 0, 0, :3] = (0, 0, 1.2)
    poses[:, 0, 0, 3] = 1
    poses[:, 0, 1, :3] = np.array([1.5, 0, 0.6]) + rng.uniform(-1.0, 1.0, (B, 3)) * np.array([1.0, 1.0, 0.3])
    poses[:, 0, 1, 3:] = wl.random_quats(rng, (B,))
    poses[:, 0, 2, :3] = np.array([0.5, 0, 1.2]) + rng.uniform(-0.5, 0.5, (B, 3))
    poses[:, 0, 2, 3:] = wl.random_quats(rng, (B,))
    w = dict(desc=d, poses=poses, shapes=None, distractor=None)
    ref = oracle_render(orc, w)
    s = orc.Scene(d)
    spans = []
    for e in range(B):
        vs = s.vertex_stage(poses[e, 0])
        ok = vs["rejected"] == 0
        spans.append(int(np.ptp(vs["X"][ok])) if ok.any() else 0)
    assert max(spans) > 1 << 17, "scene does not exercise the 64-bit path"
    assert (ref["ids"] < GROUND).mean() > 0.2
    assert_parity(gpu_render(torch, pxr, w), ref)


def test_rejected_and_degenerate_inputs(torch, pxr, orc):
    w = wl.make(2, B=12)
    p = w["poses"].copy()
    p[8, 0, 0, 0] = np.nan         # non-finite root x: no usable vertex, ground cells decided by y alone
    p[9, 0, 0, 0] = 3.0e9          # ground cell index beyond int32: the conversion saturates on both sides
    p[10, 0, 0, 1] = -np.inf
    p[11, 0, 0, :2] = (-7.0e9, 5.0e9)
    p[0, 0, :, 0] -= 10.0          # whole chain far behind the camera (root too: camera follows it) -> visible
    p[1, 0, 1:, 0] = -5.0          # links behind the camera: rejected
    p[2, 0, 3, :3] = np.nan        # non-finite position
    p[3, 0, 2, 3:] = np.nan        # non-finite quaternion
    p[4, 0, 0, 2] = -3.0           # root (and the camera) below the ground plane
    p[5, 0, 4, :3] = p[5, 0, 0, :3] + np.array([-2.45, 0, 1.0], np.float32)  # a link straddling the near plane
    p[6, 0, :, 3:] = 0.0           # zero quaternions: bodies collapse to their centres
    p[7, 0, 5, 1] = 1e6            # far off to the side: guard band
    w["poses"] = p
    ref = oracle_render(orc, w)
    got = gpu_render(torch, pxr, w)
    assert_parity(got, ref)
    assert not np.any(ref["ids"][4] == GROUND)  # camera below the plane: no ground


@pytest.mark.parametrize("over", [dict(), dict(cam_up=(0.2, 0.1, 1.0)), dict(z_far=1.0e30),
                                  dict(z_far=3.0e38, cam_up=(0.2, 0.1, 1.0)), dict(ground_cell=0.37),
                                  # the y axis as the x axis, in every form of the resolve loop: along it; rolled about it (right vector (0.45, 0, 0.89))
                                  dict(cam_offset=(0.0, -2.5, 1.0)), dict(cam_offset=(0.0, 2.5, 1.0), z_far=1.0e30),
                                  dict(cam_offset=(0.0, -2.5, 1.0), ground_cell=0.37), dict(cam_offset=(-2.0, 0.0, 1.0), cam_up=(-2.0, 1.0, 1.0))])
def test_checker_cells_of_non_finite_and_huge_ground_points(torch, pxr, orc, over):
    """The unit-cell checker takes a shorter floor-and-convert that is only right when the ground point is no NaN:
    frames whose eye is a NaN, and scenes whose far plane lets the ray parameter overflow, must take the long form."""
    w = wl.make(1, B=12)
    p = w["poses"].copy()
    r = w["desc"]["root_body"]
    p[0, 0, r, 0] = np.nan
    p[1, 0, r, 1] = np.nan
    p[2, 0, r, 0] = np.inf
    p[3, 0, r, 1] = -np.inf
    p[4, 0, r, :2] = (np.inf, np.nan)
    p[5, 0, r, :2] = (-3.0e38, 3.0e38)
    p[6, 0, r, :2] = (2147483647.0, -2147483648.0)   # cell indices at the ends of int32
    p[7, 0, r, :2] = (2147483520.0, -2147483904.0)   # the floats next to them
    p[8, 0, r, :2] = (-0.0, 1.0e-30)
    p[9, 0, r, 2] = 3.0e38                           # eye so high that the ground is beyond any far plane
    p[10, 0, r, 2] = np.inf
    w = dict(w, poses=p, desc=dict(w["desc"], **over))
    assert_parity(gpu_render(torch, pxr, w), oracle_render(orc, w))


def test_ground_variants(torch, pxr, orc):
    w = wl.make(1, B=8)
    for over in (dict(ground_enabled=False), dict(ground_cell=0.37), dict(z_far=4.0), dict(cam_up=(0.2, 0.1, 1.0)),
                 dict(cam_offset=(1.5, 2.0, 3.0)), dict(fov_y_deg=25.0), dict(light_dir=(0.5, 0.2, -0.4))):
        w2 = dict(w, desc=dict(w["desc"], **over))
        assert_parity(gpu_render(torch, pxr, w2), oracle_render(orc, w2))


@pytest.mark.parametrize("offset", [(-2.5, 0.0, 1.0), (2.5, -0.0, 0.6), (0.0, -2.5, 1.0), (-0.0, 2.5, 0.6), (-2.5, 1.0e-30, 1.0), (1.7, -1.7, 0.8)])
@pytest.mark.parametrize("W,H,mode", [(64, 64, "color"), (131, 90, "none"), (84, 84, "video")])
def test_cameras_along_an_axis_and_beside_it(torch, pxr, orc, offset, W, H, mode):
    """A camera that looks along the x axis (its right vector's x is a zero of either sign) has a checker cell index of its rows' own; so has one along
    the y axis, with the two axes exchanged; one a hair's breadth beside the x axis or between the two has not."""
    w = wl.cfg3(B=3)
    w["desc"] = dict(w["desc"], width=W, height=H, cam_offset=offset)
    w["poses"][..., :2] += np.array([[-7.3, 2.9], [0.0, 0.0], [1.0e6, -3.0]], np.float32)[:, None, None]
    w["distractor"] = dict(none=None, color=w["distractor"], video=dict(
        mode="video", seed=3, alpha=0.5, video=np.random.default_rng(1).integers(0, 256, (2, H, W, 3), dtype=np.uint8)))[mode]
    ref = oracle_render(orc, w)
    assert (ref["ids"] == GROUND).any() and (ref["ids"] == BG).any()
    assert_parity(gpu_render(torch, pxr, w), ref)


@pytest.mark.parametrize("seed", range(24))
def test_random_scenes_match_oracle(torch, pxr, orc, seed):
    """Seeded random scenes: image shapes, cameras (with and without roll), body mixes and sizes (triangles of
    every raster bin, bodies crossing the near plane), shapes per environment, all distractor modes."""
    w = wl.random_scene(seed)
    ref = oracle_render(orc, w, step0=3, env0=5)
    assert_parity(gpu_render(torch, pxr, w, step0=3, env0=5), ref)
    assert_parity(gpu_render(torch, pxr, w, step0=3, env0=5, threads=(256, 512, 768, 1024)[seed % 4]), ref)


# ---------------------------------------------------------------- distractors

def test_colour_distractor_per_step_and_identity(torch, pxr, orc):
    w = wl.make(3, B=12)
    plain = gpu_render(torch, pxr, dict(w, distractor=None))
    ident = gpu_render(torch, pxr, dict(w, distractor=dict(mode="color", seed=1, scale=(1.0, 1.0), offset=(0.0, 0.0))))
    assert np.array_equal(plain["frames"], ident["frames"])
    a = gpu_render(torch, pxr, w, step0=0)
    b = gpu_render(torch, pxr, w, step0=1)
    assert np.array_equal(a["ids"], b["ids"]) and not np.array_equal(a["frames"], b["frames"])
    for step0, env0 in [(0, 0), (1, 0), (0xFFFFFFFE, 0), (5, 0xFFFFFFF0)]:
        assert_parity(gpu_render(torch, pxr, w, step0=step0, env0=env0), oracle_render(orc, w, step0=step0, env0=env0))
    big_seed = dict(w, distractor=dict(w["distractor"], seed=0xFEDCBA9876543210))
    assert_parity(gpu_render(torch, pxr, big_seed, step0=9), oracle_render(orc, big_seed, step0=9))


def test_video_distractor_offsets_alpha_and_wrap(torch, pxr, orc):
    w = wl.make(4, B=12)
    video = w["distractor"]["video"]
    for dis, step0 in [(dict(mode="video", seed=4, video=video, alpha=0.5, env_offset=None), 0),
                       (dict(mode="video", seed=4, video=video, alpha=0.5, env_offset=None), 63),
                       (dict(mode="video", seed=9, video=video[:5], alpha=0.25, env_offset=None), 0xFFFFFFF0),
                       (dict(mode="video", seed=4, video=video, alpha=1.0, env_offset=np.arange(12) * 7 + 60), 3),
                       (dict(mode="video", seed=4, video=video, alpha=0.0, env_offset=None), 3)]:
        w2 = dict(w, distractor=dis)
        ref = oracle_render(orc, w2, step0=step0, env0=5)
        assert_parity(gpu_render(torch, pxr, w2, step0=step0, env0=5), ref)
    plain = gpu_render(torch, pxr, dict(w, distractor=None))
    assert np.array_equal(plain["frames"], gpu_render(torch, pxr, w2, step0=3)["frames"])  # alpha = 0


def test_video_distractor_with_and_without_blend_tables(torch, pxr, orc):
    """The video blend reads per-frame tables from LDS where the frame's LDS has room for them (small scenes, banded
    frames) and does the arithmetic per pixel where it has not (the largest unbanded scenes), or when the camera rolls."""
    rng = np.random.default_rng(99)
    for cfg, B, roll, has_tables in [(5, 10, False, False), (3, 12, False, True), (3, 8, True, True), (4, 6, False, True)]:
        w = wl.make(cfg, B=B)
        H, W = w["desc"]["height"], w["desc"]["width"]
        if roll:
            w["desc"]["cam_up"] = (0.0, 0.3, 1.0)
        w["distractor"] = dict(mode="video", seed=cfg, video=rng.integers(0, 256, (9, H, W, 3), dtype=np.uint8),
                               alpha=0.35, env_offset=None)
        sc = pxr.Scene(w["desc"])
        lds = sc.info()["lds_bytes"]
        sc.close()
        if not has_tables:  # two workgroups per compute unit as it is, one if the 2304 bytes of tables were added
            assert lds <= 80 * 1024 < lds + 2304
        assert_parity(gpu_render(torch, pxr, w, step0=5), oracle_render(orc, w, step0=5))


def test_video_sets_one_clip_per_environment(torch, pxr, orc):
    """A set of clips [n_videos, n_frames, H, W, 3]: each environment plays one, drawn from the generator or given."""
    w = wl.make(4, B=14)
    rng = np.random.default_rng(21)
    clips = rng.integers(0, 256, (5, 9, 84, 84, 3), dtype=np.uint8)
    for dis, step0 in [(dict(mode="video", seed=4, video=clips, alpha=0.5), 0),
                       (dict(mode="video", seed=77, video=clips, alpha=0.7, env_offset=np.arange(14) * 3), 8),
                       (dict(mode="video", seed=4, video=clips, alpha=0.5, env_video=np.arange(14) % 5), 2),
                       (dict(mode="video", seed=4, video=clips, alpha=0.5, env_video=np.arange(14) + 3,
                             env_offset=np.arange(14)[::-1].copy()), 0xFFFFFFF8),
                       (dict(mode="video", seed=4, video=clips[:1], alpha=0.5), 3)]:
        w2 = dict(w, distractor=dis)
        assert_parity(gpu_render(torch, pxr, w2, step0=step0, env0=3), oracle_render(orc, w2, step0=step0, env0=3))
    # a set of one clip is the single-clip case
    a = gpu_render(torch, pxr, dict(w, distractor=dict(mode="video", seed=4, video=clips[:1], alpha=0.5)), step0=3)
    b = gpu_render(torch, pxr, dict(w, distractor=dict(mode="video", seed=4, video=clips[0], alpha=0.5)), step0=3)
    assert np.array_equal(a["frames"], b["frames"])


def test_rebinding_and_unbinding(torch, pxr, orc):
    w = wl.make(3, B=6)
    sc = pxr.Scene(w["desc"])
    col = gpu_render(torch, pxr, w, scene=sc)
    none = gpu_render(torch, pxr, dict(w, distractor=None), scene=sc)
    col2 = gpu_render(torch, pxr, w, scene=sc)
    assert np.array_equal(col["frames"], col2["frames"]) and not np.array_equal(col["frames"], none["frames"])
    assert_parity(none, oracle_render(orc, dict(w, distractor=None)))
    sc.close()


# ---------------------------------------------------------------- argument errors on a live scene

def test_render_argument_errors(torch, pxr):
    w = wl.make(1, B=4)
    sc = pxr.Scene(w["desc"])
    L = pxr.lib()
    poses = torch.from_numpy(w["poses"]).cuda()
    frames = torch.empty((4, 1, 32, 32, 3), dtype=torch.uint8, device="cuda")
    h = sc._h
    assert L.pxr_render_batch(h, None, None, 4, 1, 0, 0, frames.data_ptr(), None, None) == pxr.ERR_INVALID_ARG
    assert L.pxr_render_batch(h, poses.data_ptr(), None, 0, 1, 0, 0, frames.data_ptr(), None, None) == pxr.ERR_INVALID_ARG
    poses2 = torch.cat([poses, poses], dim=1).contiguous()
    frames2 = torch.empty((4, 2, 32, 32, 3), dtype=torch.uint8, device="cuda")
    assert L.pxr_render_batch(h, poses2.data_ptr(), None, 4, 2, 0xFFFFFFFF, 0, frames2.data_ptr(), None, None) == pxr.ERR_INVALID_ARG
    assert L.pxr_render_batch(h, poses2.data_ptr(), None, 4, 2, 0, 0xFFFFFFFD, frames2.data_ptr(), None, None) == pxr.ERR_INVALID_ARG
    assert L.pxr_render_batch(h, poses.data_ptr(), None, 4, 1, 0, 0, frames.data_ptr() + 1, None, None) == pxr.ERR_INVALID_ARG
    shapes = torch.ones((5, w["poses"].shape[2], 4), dtype=torch.float32, device="cuda")
    assert L.pxr_render_batch(h, poses.data_ptr(), shapes.data_ptr() + 4, 4, 1, 0, 0, frames.data_ptr(), None, None) == pxr.ERR_INVALID_ARG
    assert L.pxr_render_batch(h, poses.data_ptr(), shapes.data_ptr() + 16, 4, 1, 0, 0, frames.data_ptr(), None, None) == pxr.OK
    assert L.pxr_render_batch(h, poses.data_ptr(), None, 1 << 31, 1, 0, 0, frames.data_ptr(), None, None) == pxr.ERR_INVALID_ARG
    assert b"pxr_render_batch" in L.pxr_last_error()
    with pytest.raises(pxr.PxrError):
        sc.set_block_threads(128)
    d = pxr.DistractorDesc()
    d.mode = 2
    import ctypes as C
    assert L.pxr_apply_distractor(h, C.byref(d)) == pxr.ERR_INVALID_ARG  # video without a clip
    d.mode = 9
    assert L.pxr_apply_distractor(h, C.byref(d)) == pxr.ERR_INVALID_ARG
    # the scene is still usable after the rejected calls
    f, _ = sc.render_batch(poses)
    torch.cuda.synchronize()
    assert f.shape == (4, 1, 32, 32, 3)
    sc.close()


# ---------------------------------------------------------------- full benchmark sizes, sampled

@pytest.mark.parametrize("cfg", [2, 3, 4, 5])
def test_full_size_batches_sampled_against_oracle(torch, pxr, orc, cfg):
    """The configurations at their full batch size, in the launch configuration bench.py times
    (library-default workgroup size, ids off for the timed buffer), checked on sampled environments
    the oracle renders one by one, plus run-to-run determinism of the whole output."""
    w = wl.make(cfg)
    B, S = w["poses"].shape[:2]
    scene = pxr.Scene(w["desc"])
    _bind(torch, scene, w["distractor"])
    poses = torch.from_numpy(w["poses"]).cuda()
    shapes = None if w["shapes"] is None else torch.from_numpy(w["shapes"]).cuda()
    frames, _ = scene.render_batch(poses, shapes, step0=5, env0=0)
    again, ids = scene.render_batch(poses, shapes, step0=5, env0=0, want_ids=True)
    torch.cuda.synchronize()
    assert torch.equal(frames, again)
    rng = np.random.default_rng(cfg)
    chunk = (B * S + 7) // 8 // S  # environments per XCD run of the workgroup renumbering
    picks = sorted(set([0, 1, B - 1, B - 2, B // 2] + [min(B - 1, k * chunk + d) for k in range(1, 8) for d in (-1, 0)]
                       + [int(e) for e in rng.integers(0, B, 24)]))
    o = orc.Scene(w["desc"])
    for e in picks:
        sh = None if w["shapes"] is None else w["shapes"][e:e + 1]
        ref = o.render(w["poses"][e:e + 1], sh, step0=5, env0=e, distractor=w["distractor"])
        got = dict(frames=frames[e:e + 1].cpu().numpy(), ids=pxr.ids_to_numpy(ids[e:e + 1]))
        assert_parity(got, ref)
    scene.close()


def test_outputs_beyond_four_gibibytes(torch, pxr, orc):
    """A batch whose frames (4.5 GB) and id maps (6 GB) pass 2^32 bytes: offsets are 64-bit all the way.
    Sampled environments from both ends and around the 4 GiB mark against the oracle."""
    w = wl.make(4, B=16)
    B = 212992
    rng = np.random.default_rng(44)
    poses = np.ascontiguousarray(w["poses"][rng.integers(0, 16, B)])
    poses[..., 0, :2] += rng.uniform(-0.3, 0.3, (B, 1, 2)).astype(np.float32)  # (the root moves: every frame differs)
    scene = pxr.Scene(w["desc"])
    _bind(torch, scene, w["distractor"])
    frames, ids = scene.render_batch(torch.from_numpy(poses).cuda(), None, step0=2, want_ids=True)
    torch.cuda.synchronize()
    frame_bytes = frames[0].numel()
    assert frames.numel() > 2 ** 32 and ids.numel() * 4 > 2 ** 32
    mark = 2 ** 32 // frame_bytes
    o = orc.Scene(w["desc"])
    for e in (0, 1, mark - 1, mark, mark + 1, 2 ** 32 // (4 * 84 * 84), B - 2, B - 1):
        ref = o.render(poses[e:e + 1], None, step0=2, env0=e, distractor=w["distractor"])
        got = dict(frames=frames[e:e + 1].cpu().numpy(), ids=pxr.ids_to_numpy(ids[e:e + 1]))
        assert_parity(got, ref)
    scene.close()
