"""hipGraph replay and autotuned launch parameters change no pixel: every
replay and every parameter set gives the bits of the eager default render."""
import math
import time

import numpy as np
import pytest

from paper_2604_25459_amd import synth

pytestmark = pytest.mark.gpu


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def test_graph_replays_match_eager():
    torch = _torch()
    from paper_2604_25459_amd import gsr
    scene, batch = synth.make_config(1, n_envs=8)
    Rg = gsr.Renderer(0)                  # graphs on (default)
    Re = gsr.Renderer(0, graphs=False)
    sg, se = Rg.add_synth_scene(scene), Re.add_synth_scene(scene)
    cams, vm, _ = gsr.batch_tensors(batch)
    dev = vm.device
    for step in range(4):                 # new poses every step: one capture, then replays
        poses = torch.from_numpy(synth.make_poses(1, step, 8, scene.n_bodies)).to(dev)
        eager = Re.render(se, cams, vm, poses, alpha=True)
        torch.cuda.synchronize()
        replay = Rg.render(sg, cams, vm, poses, alpha=True)
        torch.cuda.synchronize()
        for a, b in zip(eager[0], replay[0]):
            assert torch.equal(a, b), f"step {step}"
    Rg.close()
    Re.close()


def test_two_stream_chunks_match_one_stream():
    """Alternate memory chunks on two streams give the bits of one stream, and
    work queued on the caller's stream after the call sees finished images."""
    torch = _torch()
    from paper_2604_25459_amd import gsr
    scene, batch = synth.make_config(3, n_envs=8)       # 16 images in chunks of 3: six chunks
    R1 = gsr.Renderer(0, overlap=False)
    R2 = gsr.Renderer(0)
    s1, s2 = R1.add_synth_scene(scene), R2.add_synth_scene(scene)
    cams, vm, poses = gsr.batch_tensors(batch)
    R1.set_tuning(s1, cams, vm, poses, chunk_images=3)
    R2.set_tuning(s2, cams, vm, poses, chunk_images=3)
    dev = vm.device
    for step in range(3):                 # new poses every step: graph capture, then replays
        poses = torch.from_numpy(synth.make_poses(3, step, 8, scene.n_bodies)).to(dev)
        ref = [[t.clone() for t in slot] for slot in R1.render(s1, cams, vm, poses, alpha=True)]
        got = [[t.clone() for t in slot] for slot in R2.render(s2, cams, vm, poses, alpha=True)]
        torch.cuda.synchronize()
        for slot_ref, slot_got in zip(ref, got):
            for a, b in zip(slot_ref, slot_got):
                assert torch.equal(a, b), f"step {step}"
    R1.close()
    R2.close()


def test_trim_releases_working_memory_and_changes_no_pixel():
    """gsr_trim frees the idle working sets (two-stream chunks hold two); the
    next render allocates again and gives the same bits."""
    torch = _torch()
    from paper_2604_25459_amd import gsr
    scene, batch = synth.make_config(3, n_envs=8)
    R = gsr.Renderer(0)
    sid = R.add_synth_scene(scene)
    cams, vm, poses = gsr.batch_tensors(batch)
    R.set_tuning(sid, cams, vm, poses, chunk_images=3)
    ref = [[t.clone() for t in slot] for slot in R.render(sid, cams, vm, poses, alpha=True)]
    torch.cuda.synchronize()
    freed = R.trim()
    print("trim freed", freed, flush=True)
    assert freed > 100 << 20                 # the working sets of a 596k-Gaussian scene
    assert R.trim() <= 4 << 20               # nothing left to free
    got = R.render(sid, cams, vm, poses, alpha=True)
    torch.cuda.synchronize()
    for slot_ref, slot_got in zip(ref, got):
        for a, b in zip(slot_ref, slot_got):
            assert torch.equal(a, b)
    R.close()


def test_two_stream_lidar_chunks_match_one_stream():
    torch = _torch()
    from paper_2604_25459_amd import gsr
    scene = synth.make_scene(52, 120_000, 3, 20_000, sh_degree=0, half_box=3.0)
    rng = np.random.default_rng(7)
    E = 12
    lid = synth.rotating_lidar(16, 256, -20, 20)
    ros = synth.rosette_lidar(16, 128, half_fov_deg=35.0, s0=0.7)       # listed rays in the same call
    vm = torch.from_numpy(np.stack([synth.sensor_viewmats(rng, E, 0.5, 2.5, 0.1),
                                    synth.sensor_viewmats(rng, E, 0.5, 2.5, 0.1)])).cuda()
    poses = torch.from_numpy(synth.random_poses(rng, E, scene.n_bodies)).cuda()
    out = []
    for overlap in (False, True):
        R = gsr.Renderer(0, chunk_bytes=64 << 20, overlap=overlap)   # a few scans per chunk
        sid = R.add_synth_scene(scene)
        res = R.render_lidar(sid, [lid, ros], vm, poses)
        out.append([(r.clone(), h.clone()) for r, h in res])
        torch.cuda.synchronize()
        R.close()
    for (r0, h0), (r1, h1) in zip(out[0], out[1]):
        assert torch.equal(r0, r1) and torch.equal(h0, h1)
    assert (out[0][0][1] > 0.1).sum() > 100 and (out[0][1][1] > 0.1).sum() > 100


@pytest.mark.parametrize("params", [dict(tile_size=8, lds_batch=64), dict(tile_size=8, lds_batch=256),
                                    dict(tile_size=32, lds_batch=512), dict(lds_batch=512, images_per_thread=1),
                                    dict(images_per_thread=8, persistent=1), dict(persistent=1, chunk_images=3),
                                    dict(bin_schedule=0), dict(bin_schedule=1, tile_size=8, lds_batch=128),
                                    dict(lds_batch=256), dict(lds_batch=128, persistent=1),
                                    dict(tile_size=32, lds_batch=128), dict(images_per_thread=16),
                                    dict(images_per_thread=16, chunk_images=2, tile_size=8)])
def test_tuning_changes_no_pixel(params):
    torch = _torch()
    from paper_2604_25459_amd import gsr
    scene, batch = synth.make_config(3, n_envs=5)       # two camera slots of different sizes
    R = gsr.Renderer(0)
    sid = R.add_synth_scene(scene, "bf16")
    cams, vm, poses = gsr.batch_tensors(batch)
    ref = R.render(sid, cams, vm, poses, alpha=True)
    R.set_tuning(sid, cams, vm, poses, **params)
    got = R.tuning(sid, cams, vm, poses)
    for k, v in params.items():
        assert got[k] == v
    for _ in range(2):
        out = R.render(sid, cams, vm, poses, alpha=True)
        for slot_ref, slot_out in zip(ref, out):
            for a, b in zip(slot_ref, slot_out):
                assert torch.equal(a, b), params
    R.close()


def test_autotune_and_cache_roundtrip(tmp_path):
    torch = _torch()
    from paper_2604_25459_amd import gsr
    scene, batch = synth.make_config(1, n_envs=16)
    R = gsr.Renderer(0)
    sid = R.add_synth_scene(scene)
    cams, vm, poses = gsr.batch_tensors(batch)
    ref = R.render(sid, cams, vm, poses)
    rgb, depth, _ = R.alloc_outputs(cams, 16)
    best = R.autotune(sid, cams, vm, poses, rgb, depth)
    print("autotuned", best, flush=True)
    assert best["tile_size"] in (8, 16, 32) and best["ms"] > 0
    assert R.tuning(sid, cams, vm, poses) == best
    out = R.render(sid, cams, vm, poses)
    assert torch.equal(out[0][0], ref[0][0]) and torch.equal(out[0][1], ref[0][1])
    path = str(tmp_path / "tune.jsonl")
    R.save_tuning(path)
    R2 = gsr.Renderer(0)
    sid2 = R2.add_synth_scene(scene)
    R2.load_tuning(path)
    loaded = R2.tuning(sid2, cams, vm, poses)
    assert {k: v for k, v in loaded.items() if k != "ms"} == {k: v for k, v in best.items() if k != "ms"}
    assert loaded["ms"] == pytest.approx(best["ms"], rel=1e-6)
    R2.close()
    R.close()


def test_schedules_agree_on_wide_splats():
    """Splats wider than the image cover every column of a transposed group
    (64 entries x 64 columns all set, so a tile list takes more than one
    128-byte line per group); both list schedules must still produce the same
    pixels bit for bit."""
    torch = _torch()
    from paper_2604_25459_amd import gsr
    from tests.scenes import one_camera, scene_from
    rng = np.random.default_rng(4)
    n = 600
    means = rng.uniform([-1.5, -1.0, 2.0], [1.5, 1.0, 4.0], (n, 3))
    scales = np.exp(rng.normal(np.log(0.8), 0.3, (n, 3)))          # each covers most of the image
    scene = scene_from(means, scales, rng.standard_normal((n, 4)), rng.uniform(0.02, 0.3, n),
                       rng.uniform(0, 1, (n, 1, 3)), degree=0)
    batch = one_camera(640, 480, 400.0)
    R = gsr.Renderer(0)
    sid = R.add_synth_scene(scene)
    cams, vm, poses = gsr.batch_tensors(batch)
    outs = []
    for sched in (0, 1):
        R.set_tuning(sid, cams, vm, poses, bin_schedule=sched)
        outs.append(R.render(sid, cams, vm, poses, alpha=True))
    for a, b in zip(outs[0][0], outs[1][0]):
        assert torch.equal(a, b)
    R.close()


def test_transposed_schedule_on_a_wide_image():
    """1920 x 1080 at 16-pixel tiles: 120 tile columns and 68 tile rows, so
    the transposed schedule runs two 64-column windows per row segment at
    level 2 and two 64-row windows per block at level 1.  Its tile lists
    equal the oracle's bit for bit, and both schedules give the same pixels."""
    torch = _torch()
    from paper_2604_25459_amd import gsr, synth
    from oracle import bin_ref
    scene = synth.make_scene(63, 40_000, 2, 4_000, sh_degree=1, half_box=4.0)
    rng = np.random.default_rng(21)
    batch = synth.Batch(cams=[synth.pinhole(1920, 1080, 70.0)], viewmats=synth.orbit_viewmats(rng, 2, 3.0, 5.0)[None],
                        poses=synth.random_poses(rng, 2, scene.n_bodies))
    R = gsr.Renderer(0)
    sid = R.add_synth_scene(scene)
    cams, vm, poses = gsr.batch_tensors(batch)
    outs = []
    for sched in (0, 1):
        R.set_tuning(sid, cams, vm, poses, bin_schedule=sched)
        outs.append(R.render(sid, cams, vm, poses, alpha=True))
        if sched == 1:
            got = R.debug_bins(sid, cams, vm, poses, 1)
            ref = bin_ref(scene, batch, 0, 1, got["tile_size"])
            assert ref.ranges.shape[0] == 120 * 68
            np.testing.assert_array_equal(got["keys"], ref.keys)
            np.testing.assert_array_equal(got["values"], ref.values)
            np.testing.assert_array_equal(got["ranges"], ref.ranges)
    for a, b in zip(outs[0][0], outs[1][0]):
        assert torch.equal(a, b)
    R.close()


def test_async_render_returns_before_the_device_finishes():
    """After a render that sizes the tile lists of a job shape, renders of that
    shape enqueue every chunk without waiting for its totals: the call returns
    while the device still works, and the images equal a render that waits at
    every chunk."""
    torch = _torch()
    from paper_2604_25459_amd import gsr
    scene, batch = synth.make_config(2, n_envs=512)
    Ra = gsr.Renderer(0)
    Rs = gsr.Renderer(0, sync_lists=True)
    sa, ss = Ra.add_synth_scene(scene), Rs.add_synth_scene(scene)
    cams, vm, _ = gsr.batch_tensors(batch)
    dev = vm.device
    rgb_a, depth_a, _ = Ra.alloc_outputs(cams, 512)
    rgb_s, depth_s, _ = Rs.alloc_outputs(cams, 512)
    stream = torch.cuda.current_stream(dev)
    for step in range(3):
        poses = torch.from_numpy(synth.make_poses(2, step, 512, scene.n_bodies)).to(dev)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        Ra.render_into(sa, cams, vm, poses, rgb_a, depth_a)
        t_call = time.perf_counter() - t0
        pending = not stream.query()
        torch.cuda.synchronize()
        t_all = time.perf_counter() - t0
        print(f"step {step}: call {1e3 * t_call:.2f} ms, render {1e3 * t_all:.2f} ms, pending {pending}", flush=True)
        if step > 0:                   # step 0 plans the lists (waits at every chunk)
            assert pending and t_call < 0.5 * t_all
        Rs.render_into(ss, cams, vm, poses, rgb_s, depth_s)
        torch.cuda.synchronize()
        assert torch.equal(rgb_a, rgb_s) and torch.equal(depth_a, depth_s), f"step {step}"
    Ra.close()
    Rs.close()


def test_list_overflow_falls_back_with_identical_bits():
    """Asynchronous chunks whose tile lists exceed a small capacity set from
    the host write no lists; the fallback rasteriser composites them from the
    depth-ordered Gaussians, and images and work counts equal the planned
    render's bit for bit (two camera sizes, chunks on two streams)."""
    torch = _torch()
    from paper_2604_25459_amd import gsr
    scene, batch = synth.make_config(3, n_envs=6)
    R = gsr.Renderer(0, list_cap=2000)
    sid = R.add_synth_scene(scene)
    cams, vm, poses = gsr.batch_tensors(batch)
    R.set_tuning(sid, cams, vm, poses, chunk_images=4)     # three chunks, alternating streams
    rgb, depth, alpha = R.alloc_outputs(cams, 6, alpha=True)
    npx = rgb.numel() // 3
    work = torch.zeros(npx * 2, dtype=torch.int32, device=rgb.device)
    R.render_into(sid, cams, vm, poses, rgb, depth, alpha, work=work)      # plans the lists
    torch.cuda.synchronize()
    ref = [t.clone() for t in (rgb, depth, alpha, work)]
    for k in range(3):
        for t in (rgb, depth, alpha):
            t.fill_(float("nan"))
        work.fill_(-1)
        R.render_into(sid, cams, vm, poses, rgb, depth, alpha, work=work)  # overflows into the fallback
        torch.cuda.synchronize()
        for a, b in zip(ref, (rgb, depth, alpha, work)):
            assert torch.equal(a, b), f"render {k}"
    R.close()


@pytest.mark.parametrize("n,envs,w,h,ts", [(255, 1, 100, 75, 16), (4097, 1, 100, 75, 16), (40_000, 1, 333, 47, 16),
                                           (70_000, 3, 640, 200, 16), (600, 300, 64, 48, 16), (2_000, 1, 24, 8000, 8),
                                           (1_500, 1, 112, 8192, 8)])
def test_lists_at_every_launch_size(n, envs, w, h, ts):
    """Tile lists against the specification where the list kernels change shape
    with the launch: block lengths from one short block to many, one image and
    hundreds, row counts beyond a scan's threads, and the tallest tile grids."""
    _torch()
    from oracle import bin_ref
    from paper_2604_25459_amd import gsr
    scene = synth.make_scene(n + h, n, 0, 0, sh_degree=0, half_box=2.0)
    vm = synth.orbit_viewmats(np.random.default_rng(n), envs, 3.0, 5.0)
    batch = synth.Batch(cams=[synth.pinhole(w, h, 60.0)], viewmats=vm[None], poses=np.zeros((envs, 0, 7), np.float32))
    r = gsr.Renderer(0, tile_size=ts)
    sid = r.add_synth_scene(scene)
    cams, vm_t, poses = gsr.batch_tensors(batch)
    for schedule in (0, 1):
        r.set_tuning(sid, cams, vm_t, poses, bin_schedule=schedule)
        for e in sorted({0, envs - 1}):
            got = r.debug_bins(sid, cams, vm_t, poses, e)
            ref = bin_ref(scene, batch, 0, e, ts)
            assert got["n_visible"] == int(ref.visible.sum())
            np.testing.assert_array_equal(got["keys"], ref.keys)
            np.testing.assert_array_equal(got["values"], ref.values)
            np.testing.assert_array_equal(got["ranges"], ref.ranges)
    r.close()


@pytest.mark.parametrize("n", [1, 2, 3, 63, 64, 65, 127, 129])
def test_survivor_counts_around_a_pair_and_a_batch(n):
    """Wide, faint splats that every wave of the tile keeps, so that n counts
    its survivors: one alone, odd and even counts, a full group of 64 and the
    remainders beside it; every fifth is opaque beyond the 0.99 clamp and small."""
    torch = _torch()
    from oracle import render_ref
    from paper_2604_25459_amd import gsr
    from tests.parity import compare
    from tests.scenes import one_camera, scene_from
    rng = np.random.default_rng(500 + n)
    i = np.arange(n)
    opaque = i % 5 == 4
    means = rng.uniform([-0.2, -0.2, 1.0], [0.2, 0.2, 3.0], (n, 3))
    scales = np.where(opaque[:, None], 0.03, 0.6) * np.ones((n, 3))
    opac = np.where(opaque, 0.998, 0.02)
    scene = scene_from(means, scales, rng.standard_normal((n, 4)), opac, rng.uniform(0, 1, (n, 1, 3)), 0)
    batch = one_camera(16, 16, 60.0, bg=(0.2, 0.3, 0.4))
    R = gsr.Renderer(0)
    sid = R.add_synth_scene(scene)
    cams, vm, poses = gsr.batch_tensors(batch)
    rgb, depth, alpha = R.render(sid, cams, vm, poses, bg=tuple(batch.bg), alpha=True)[0]
    torch.cuda.synchronize()
    ref = render_ref(scene, batch, 0, 0, R.tile_size)
    res = compare(rgb[0].cpu().numpy(), depth[0].cpu().numpy(), ref, gpu_alpha=alpha[0].cpu().numpy(), rgb_tol=1e-3)
    assert res["ok"], res
    R.close()


@pytest.mark.parametrize("ts", [8, 16, 32])
def test_images_equal_on_both_sides_of_the_direct_line(ts):
    """One-tile images, once as many as one launch composites without staging
    and once a few more: the images both have are the same bits."""
    torch = _torch()
    from paper_2604_25459_amd import gsr
    from tests.scenes import one_camera, scene_from
    rng = np.random.default_rng(77)
    n, line = 300, 24576
    scene = scene_from(rng.uniform([-0.3, -0.3, 1.0], [0.3, 0.3, 3.0], (n, 3)), np.exp(rng.normal(-3.0, 0.8, (n, 3))),
                       rng.standard_normal((n, 4)), rng.uniform(0.02, 1.0, n), rng.uniform(0, 1, (n, 1, 3)), 0)
    batch = one_camera(ts, ts, 0.9 * ts)
    R = gsr.Renderer(0, tile_size=ts)
    sid = R.add_synth_scene(scene)
    cams, vm, _ = gsr.batch_tensors(batch)
    views = vm.repeat(1, line + 7, 1, 1)
    views[0, :, 0, 3] = torch.linspace(-0.3, 0.3, line + 7, device=vm.device)
    poses = torch.zeros(line + 7, 0, 7, device=vm.device)
    some = [t.clone() for t in R.render(sid, cams, views[:, :line].contiguous(), poses[:line], alpha=True)[0]]
    more = R.render(sid, cams, views, poses, alpha=True)[0]
    torch.cuda.synchronize()
    for a, b in zip(some, more):
        assert torch.equal(a, b[:line])
    assert float(some[2].amax()) > 0.5 and not torch.equal(some[0][0], some[0][line - 1])
    R.close()


@pytest.mark.parametrize("persistent", [0, 1])
@pytest.mark.parametrize("envs,sides", [(1, [(17, 16), (130, 47)]), (3, [(16, 16), (48, 16), (80, 33)]),
                                        (5, [(97, 35), (16, 16), (64, 64), (33, 7), (16, 32)])])
def test_several_image_sizes_in_a_launch(envs, sides, persistent):
    """Image sizes whose tile counts leave every kind of remainder when the
    tiles are dealt out: a launch over all of them gives the bits of launches
    over each."""
    torch = _torch()
    from paper_2604_25459_amd import gsr
    from tests.scenes import scene_from
    rng = np.random.default_rng(envs)
    n = 800
    scene = scene_from(rng.uniform([-0.6, -0.6, 1.0], [0.6, 0.6, 3.0], (n, 3)), np.exp(rng.normal(-3.0, 0.8, (n, 3))),
                       rng.standard_normal((n, 4)), rng.uniform(0.02, 1.0, n), rng.uniform(0, 1, (n, 1, 3)), 0)
    R = gsr.Renderer(0)
    sid = R.add_synth_scene(scene)
    cams = [gsr.Camera(w, h, 60.0, 60.0, w / 2, h / 2, 0.01, -1) for w, h in sides]
    views = torch.eye(4, device="cuda")[:3].repeat(len(sides), envs, 1, 1)
    views[:, :, 0, 3] = torch.linspace(-0.3, 0.3, len(sides) * envs, device="cuda").view(len(sides), envs)
    poses = torch.zeros(envs, 0, 7, device="cuda")
    if persistent:
        R.set_tuning(sid, cams, views, poses, persistent=1)
    got = R.render(sid, cams, views, poses, alpha=True)
    torch.cuda.synchronize()
    for k, cam in enumerate(cams):
        one = R.render(sid, [cam], views[k:k + 1].contiguous(), poses, alpha=True)[0]
        torch.cuda.synchronize()
        for a, b in zip(got[k], one):
            assert torch.equal(a, b), (k, sides[k])
        assert float(one[2].amax()) > 0.1
    R.close()


@pytest.mark.parametrize("n_img", [1281, 9001, 65536, 65543])
def test_heavy_first_order_covers_every_tile(n_img):
    """One-tile images, some with every Gaussian in view and most with few, in
    launches just above the smallest that is ordered, in between, the largest
    and above it: every image holds the bits of launches too small to be
    ordered."""
    torch = _torch()
    from paper_2604_25459_amd import gsr
    from tests.scenes import scene_from
    rng = np.random.default_rng(n_img)
    n = 200
    scene = scene_from(rng.uniform([-0.3, -0.3, 1.0], [0.3, 0.3, 3.0], (n, 3)), np.exp(rng.normal(-3.5, 0.8, (n, 3))),
                       rng.standard_normal((n, 4)), rng.uniform(0.02, 1.0, n), rng.uniform(0, 1, (n, 1, 3)), 0)
    R = gsr.Renderer(0)
    sid = R.add_synth_scene(scene)
    cam = gsr.Camera(16, 16, 14.0, 14.0, 8.0, 8.0, 0.01, -1)
    views = torch.eye(4, device="cuda")[:3].repeat(1, n_img, 1, 1)
    views[0, :, 0, 3] = torch.from_numpy(rng.uniform(-3.0, 3.0, n_img).astype(np.float32)).cuda()
    poses = torch.zeros(n_img, 0, 7, device="cuda")
    rgb, depth, alpha = R.alloc_outputs([cam], n_img, True)
    for t in (rgb, depth, alpha):
        t.fill_(-7.0)
    R.render_into(sid, [cam], views, poses, rgb, depth, alpha)
    got = R.split([cam], n_img, rgb, depth, alpha)[0]
    torch.cuda.synchronize()
    for a in range(0, n_img, 1280):
        b = min(n_img, a + 1280)
        one = R.render(sid, [cam], views[:, a:b].contiguous(), poses[a:b], alpha=True)[0]
        torch.cuda.synchronize()
        for x, y in zip(got, one):
            assert torch.equal(x[a:b], y), a
    hit = (got[2].amax(dim=(1, 2)) > 0.1).float().mean()
    assert 0.02 < float(hit) < 0.9
    R.close()


@pytest.mark.parametrize("n", [1, 1023, 4096, 4097, 8192, 8193, 16384, 16385])
@pytest.mark.parametrize("depths", ["near", "wide", "ties", "behind"])
def test_depth_order_around_the_one_workgroup_sort(n, depths):
    """Depth order and tile lists against the specification at the largest
    counts of each one-workgroup sort and just above: depths of one digit's
    span and of all four, equal depths, and nothing in view."""
    _torch()
    from oracle import bin_ref
    from paper_2604_25459_amd import gsr
    from tests.scenes import one_camera, scene_from
    rng = np.random.default_rng(n)
    z = {"near": rng.uniform(2.0, 2.0001, n), "wide": np.exp(rng.uniform(math.log(0.02), math.log(3.0e4), n)),
         "ties": rng.integers(1, 4, n).astype(float), "behind": np.full(n, -1.0)}[depths]
    means = np.stack([rng.uniform(-0.4, 0.4, n) * z, rng.uniform(-0.4, 0.4, n) * z, z], axis=1)
    scene = scene_from(means, np.abs(z)[:, None] * rng.uniform(0.004, 0.02, (n, 3)), rng.standard_normal((n, 4)),
                       rng.uniform(0.05, 0.99, n), rng.uniform(0, 1, (n, 1, 3)), 0)
    batch = one_camera(70, 50, 60.0)
    R = gsr.Renderer(0)
    sid = R.add_synth_scene(scene)
    cams, vm, poses = gsr.batch_tensors(batch)
    got = R.debug_bins(sid, cams, vm, poses, 0)
    ref = bin_ref(scene, batch, 0, 0, R.tile_size)
    assert got["n_visible"] == int(ref.visible.sum()) and (got["n_visible"] > 0) == (depths != "behind")
    np.testing.assert_array_equal(got["keys"], ref.keys)
    np.testing.assert_array_equal(got["values"], ref.values)
    np.testing.assert_array_equal(got["ranges"], ref.ranges)
    R.close()


@pytest.mark.parametrize("n", [1 << 23, (1 << 23) + 1])
def test_depth_order_with_ids_of_23_bits_and_more(n):
    """The most Gaussians whose ids share a word with the last digit, and one
    more: all but 20,000 lie behind the camera, so that the lists are those of
    the 20,000 alone, under their ids."""
    _torch()
    from paper_2604_25459_amd import gsr
    from tests.scenes import one_camera, scene_from
    rng = np.random.default_rng(23)
    m = 20_000
    z = rng.uniform(1.0, 9.0, m)
    z[::7] = 4.0                                          # ties
    means = np.stack([rng.uniform(-0.4, 0.4, m) * z, rng.uniform(-0.4, 0.4, m) * z, z], axis=1)
    quats, opac, sh = rng.standard_normal((m, 4)), rng.uniform(0.05, 0.99, m), rng.uniform(0, 1, (m, 1, 3))
    ids = np.sort(rng.choice(n, m, replace=False))
    ids[-1] = n - 1
    batch = one_camera(70, 50, 60.0)
    cams, vm, poses = gsr.batch_tensors(batch)
    R = gsr.Renderer(0)
    sid = R.add_synth_scene(scene_from(means, np.full((m, 3), 0.01), quats, opac, sh, 0))
    few = R.debug_bins(sid, cams, vm, poses, 0)
    R.remove_scene(sid)
    all_means = np.full((n, 3), -1.0)
    all_quats, all_opac, all_sh = np.ones((n, 4)), np.full(n, 0.5), np.zeros((n, 1, 3))
    all_means[ids], all_quats[ids], all_opac[ids], all_sh[ids] = means, quats, opac, sh
    sid = R.add_synth_scene(scene_from(all_means, np.full((n, 3), 0.01), all_quats, all_opac, all_sh, 0))
    got = R.debug_bins(sid, cams, vm, poses, 0)
    assert got["n_visible"] == few["n_visible"] > 10_000
    np.testing.assert_array_equal(got["keys"], few["keys"])
    np.testing.assert_array_equal(got["values"], ids[few["values"].astype(np.int64)])
    np.testing.assert_array_equal(got["ranges"], few["ranges"])
    R.close()


@pytest.mark.parametrize("n_img,side", [(15, 160), (16, 160), (17, 160), (39, 96), (1023, 32), (1024, 32), (1025, 32)])
def test_images_dealt_over_the_xcds_cover_every_tile(n_img, side):
    """Ordered launches of one image size: too few images to deal, whole
    rounds, every kind of remainder, the most and one more.  Each image holds
    the bits of a launch of its own size too small to be ordered."""
    torch = _torch()
    from paper_2604_25459_amd import gsr
    from tests.scenes import scene_from
    rng = np.random.default_rng(n_img)
    n = 400
    scene = scene_from(rng.uniform([-0.6, -0.6, 1.0], [0.6, 0.6, 3.0], (n, 3)), np.exp(rng.normal(-3.2, 0.8, (n, 3))),
                       rng.standard_normal((n, 4)), rng.uniform(0.02, 1.0, n), rng.uniform(0, 1, (n, 1, 3)), 0)
    R = gsr.Renderer(0)
    sid = R.add_synth_scene(scene)
    cam = gsr.Camera(side, side, 0.9 * side, 0.9 * side, side / 2, side / 2, 0.01, -1)
    views = torch.eye(4, device="cuda")[:3].repeat(1, n_img, 1, 1)
    views[0, :, 0, 3] = torch.from_numpy(rng.uniform(-2.0, 2.0, n_img).astype(np.float32)).cuda()
    poses = torch.zeros(n_img, 0, 7, device="cuda")
    rgb, depth, alpha = R.alloc_outputs([cam], n_img, True)
    for t in (rgb, depth, alpha):
        t.fill_(-7.0)
    R.render_into(sid, [cam], views, poses, rgb, depth, alpha)
    got = R.split([cam], n_img, rgb, depth, alpha)[0]
    torch.cuda.synchronize()
    step = 1280 // ((side + 15) // 16) ** 2
    for a in range(0, n_img, step):
        b = min(n_img, a + step)
        one = R.render(sid, [cam], views[:, a:b].contiguous(), poses[a:b], alpha=True)[0]
        torch.cuda.synchronize()
        for x, y in zip(got, one):
            assert torch.equal(x[a:b], y), a
    R.close()


def test_images_equal_on_both_sides_of_the_direct_bytes_line():
    """One-tile images of the most Gaussians whose records count as staying in
    an XCD's L2 and of one more, which lies behind every camera: the same bits
    from the direct and the staged rasteriser, just above and at the largest
    launch that is resident at once."""
    torch = _torch()
    from paper_2604_25459_amd import gsr
    from tests.scenes import scene_from
    rng = np.random.default_rng(78)
    n = 682                                               # 256 images of 48 bytes each: 8 MB
    means = rng.uniform([-0.3, -0.3, 1.0], [0.3, 0.3, 3.0], (n, 3))
    scales, quats = np.exp(rng.normal(-3.0, 0.8, (n, 3))), rng.standard_normal((n, 4))
    opac, sh = rng.uniform(0.02, 1.0, n), rng.uniform(0, 1, (n, 1, 3))
    R = gsr.Renderer(0)
    few = R.add_synth_scene(scene_from(means, scales, quats, opac, sh, 0))
    more = R.add_synth_scene(scene_from(*[np.concatenate([a, b]) for a, b in (
        (means, [[0.0, 0.0, -2.0]]), (scales, scales[:1]), (quats, quats[:1]), (opac, opac[:1]), (sh, sh[:1]))], 0))
    cam = gsr.Camera(16, 16, 14.0, 14.0, 8.0, 8.0, 0.01, -1)
    for n_img in (2048, 2049):
        views = torch.eye(4, device="cuda")[:3].repeat(1, n_img, 1, 1)
        views[0, :, 0, 3] = torch.linspace(-0.4, 0.4, n_img, device="cuda")
        poses = torch.zeros(n_img, 0, 7, device="cuda")
        a = [t.clone() for t in R.render(few, [cam], views, poses, alpha=True)[0]]
        b = R.render(more, [cam], views, poses, alpha=True)[0]
        torch.cuda.synchronize()
        for x, y in zip(a, b):
            assert torch.equal(x, y), n_img
        assert float(a[2].amax()) > 0.5
    R.close()


@pytest.mark.parametrize("between", ["lidar", "plain", "bins"])
def test_asynchronous_renders_keep_their_plan_between_others(between):
    """A render of a planned shape, after a LiDAR scan, a plain render or a
    readback of tile lists on the same stream, which cut their tile-row lists
    into other numbers of segments: enqueued as planned, same images."""
    torch = _torch()
    from paper_2604_25459_amd import gsr
    scene = synth.make_scene(71, 40_000, 0, 0, sh_degree=0, half_box=2.0)
    rng = np.random.default_rng(71)
    cams = [synth.pinhole(640, 480, 60.0)]
    batch = synth.Batch(cams=cams, viewmats=synth.orbit_viewmats(rng, 1, 3.0, 5.0)[None],
                        poses=np.zeros((1, 0, 7), np.float32))
    tall = synth.Batch(cams=[synth.pinhole(32, 16, 20.0)], viewmats=batch.viewmats, poses=batch.poses)
    lid = synth.rotating_lidar(32, 1024, -20, 20)
    lid_vm = torch.from_numpy(synth.sensor_viewmats(rng, 1, 0.5, 1.5, 0.1)[None]).cuda()
    R = gsr.Renderer(0)
    sid = R.add_synth_scene(scene)
    cams, vm, poses = gsr.batch_tensors(batch)
    few = gsr.batch_tensors(tall)
    ref = [t.clone() for t in R.render(sid, cams, vm, poses, alpha=True)[0]]       # plans
    scan = None
    for k in range(3):
        got = R.render(sid, cams, vm, poses, alpha=True)[0]
        torch.cuda.synchronize()
        for a, b in zip(ref, got):
            assert torch.equal(a, b), k
        if between == "lidar":
            out = [t.clone() for t in R.render_lidar(sid, [lid], lid_vm, poses)[0]]
            assert scan is None or all(torch.equal(a, b) for a, b in zip(scan, out))
            scan = out
        elif between == "plain":
            R.render(sid, *few, plain=True)
        else:
            R.debug_bins(sid, *few, 0)
    R.close()


@pytest.mark.parametrize("sides,n", [(((3200, 1000), (1000, 3200)), 0), (((3200, 1000), (1000, 3200)), 300),
                                     (((8192, 16), (16, 8192)), 0)])
def test_wide_and_tall_images_in_a_launch(sides, n):
    """A wide and a tall image in one launch, whose sides together span many
    more tiles than either has: the bits of a launch of each, with Gaussians and
    of an empty scene (which has no limit on the product of the sides)."""
    torch = _torch()
    from paper_2604_25459_amd import gsr
    from tests.scenes import scene_from
    rng = np.random.default_rng(n)
    scene = scene_from(rng.uniform([-1.5, -1.5, 1.0], [1.5, 1.5, 3.0], (n, 3)), np.exp(rng.normal(-3.0, 0.8, (n, 3))),
                       rng.standard_normal((n, 4)), rng.uniform(0.02, 1.0, n), rng.uniform(0, 1, (n, 1, 3)), 0)
    R = gsr.Renderer(0)
    sid = R.add_synth_scene(scene)
    cams = [gsr.Camera(w, h, 1000.0, 1000.0, w / 2, h / 2, 0.01, -1) for w, h in sides]
    views = torch.eye(4, device="cuda")[:3].repeat(2, 1, 1, 1)
    poses = torch.zeros(1, 0, 7, device="cuda")
    got = R.render(sid, cams, views, poses, bg=(0.1, 0.2, 0.3), alpha=True)
    torch.cuda.synchronize()
    for k, cam in enumerate(cams):
        one = R.render(sid, [cam], views[k:k + 1].contiguous(), poses, bg=(0.1, 0.2, 0.3), alpha=True)[0]
        torch.cuda.synchronize()
        for a, b in zip(got[k], one):
            assert torch.equal(a, b), (k, sides[k])
        assert (float(one[2].amax()) > 0.5) == (n > 0)
    R.close()


@pytest.mark.parametrize("n_img,side", [(15, 160), (16, 160), (17, 160), (39, 96), (1023, 32), (1024, 32), (1025, 32)])
def test_images_of_long_lists_dealt_over_the_xcds_cover_every_tile(n_img, side):
    """As above with lists of hundreds of entries on average, above the line
    from which images are dealt out: whole rounds, every kind of remainder, the
    most images and one more."""
    torch = _torch()
    from paper_2604_25459_amd import gsr
    from tests.scenes import scene_from
    rng = np.random.default_rng(n_img)
    n = 400
    scene = scene_from(rng.uniform([-0.6, -0.6, 1.0], [0.6, 0.6, 3.0], (n, 3)), np.exp(rng.normal(-0.5, 0.8, (n, 3))),
                       rng.standard_normal((n, 4)), rng.uniform(0.02, 0.3, n), rng.uniform(0, 1, (n, 1, 3)), 0)
    R = gsr.Renderer(0)
    sid = R.add_synth_scene(scene)
    cam = gsr.Camera(side, side, 0.9 * side, 0.9 * side, side / 2, side / 2, 0.01, -1)
    views = torch.eye(4, device="cuda")[:3].repeat(1, n_img, 1, 1)
    views[0, :, 0, 3] = torch.from_numpy(rng.uniform(-0.5, 0.5, n_img).astype(np.float32)).cuda()
    poses = torch.zeros(n_img, 0, 7, device="cuda")
    bins = R.debug_bins(sid, [cam], views, poses, 0)
    assert bins["keys"].size > 96 * bins["ranges"].shape[0]
    rgb, depth, alpha = R.alloc_outputs([cam], n_img, True)
    for t in (rgb, depth, alpha):
        t.fill_(-7.0)
    R.render_into(sid, [cam], views, poses, rgb, depth, alpha)
    got = R.split([cam], n_img, rgb, depth, alpha)[0]
    torch.cuda.synchronize()
    step = 1280 // ((side + 15) // 16) ** 2
    for a in range(0, n_img, step):
        b = min(n_img, a + step)
        one = R.render(sid, [cam], views[:, a:b].contiguous(), poses[a:b], alpha=True)[0]
        torch.cuda.synchronize()
        for x, y in zip(got, one):
            assert torch.equal(x[a:b], y), a
    R.close()
