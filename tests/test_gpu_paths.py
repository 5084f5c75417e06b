"""Edges of the kernels' own splits: rounds of the tile walk, groups cut by the
image, tiles with pixels outside, and the introspection call between a forward
and its backward."""
import dataclasses
import threading

import numpy as np
import pytest
import torch

import scenes
from gpu_common import GRAD_RTOL, assert_grads_close, assert_images_close, gpu_lists, mask_upstream, run_gpu
from oracle import binning as obin
from oracle import render as oref
from paper_2505_05356_amd import raster

pytestmark = pytest.mark.gpu


# 256 group-list entries a round: lists of fewer, of one more, and of several
# rounds; images whose last tiles and groups are cut, in every tile shape
@pytest.mark.parametrize("n,width,height,tile", [
    (3, 17, 9, (8, 8)), (255, 70, 66, (8, 8)), (257, 70, 66, (16, 16)), (1500, 129, 33, (16, 16)),
    (1500, 257, 65, (32, 8)), (2100, 131, 130, (8, 8))])
def test_tile_walk_edges(n, width, height, tile):
    wl = scenes.tiny_scene(n, width, height, seed=n, log_scale_mean=float(np.log(0.05)))
    cfg = dataclasses.replace(wl.cfg, tile_w=tile[0], tile_h=tile[1])
    up = scenes.upstream_grads(1, cfg, seed=5)
    ref = oref.render(wl.gaussians, wl.frames, cfg)
    ok = ~ref["flagged"]
    up = mask_upstream(up, ok)
    gref = oref.render(wl.gaussians, wl.frames, cfg, upstream=up)["grads"]
    res = run_gpu(wl.gaussians, wl.frames, cfg, upstream=up)
    for k in ("rgb", "quad", "depth"):
        assert_images_close(res[k], ref[k], ok, k)
    for k in ("mean", "scale", "quat", "opacity_logit", "rgb", "albedo"):
        assert_grads_close(res["grads"][k], gref[k], k)
    # the lists are completed by the introspection call and equal the oracle's;
    # a backward after it gives what the one before it gave
    lists = gpu_lists(res, wl.gaussians, wl.frames, cfg)
    pairs = obin.sorted_pairs(wl.gaussians, wl.frames, cfg)
    assert np.array_equal(lists["pair_item"], pairs["index"].astype(np.uint32))
    d = {k: torch.from_numpy(up[k]).cuda() for k in up}
    again = raster.backward(res["_params"], res["_frames"], cfg, res["_ws"], res["_out"], d["rgb"], d["quad"],
                            d["depth"])
    for k in ("mean", "scale", "opacity_logit"):
        # two sums of the same terms in another order
        assert_grads_close(again[k].cpu().numpy(), res["grads"][k], k, rtol=GRAD_RTOL * 1e-2)


# 16x16 and 32x8 tiles take another split of the forward and the backward from
# 4096 tiles on: the same frames in one call and one at a time
@pytest.mark.parametrize("tile", [(16, 16), (32, 8)])
@pytest.mark.parametrize("n_freq", [1, 3])
def test_large_batch_split_equals_small(tile, n_freq):
    wl = scenes.tiny_scene(300, 167, 165, seed=9, dynamic=True, log_scale_mean=float(np.log(0.1)))
    cfg = dataclasses.replace(wl.cfg, tile_w=tile[0], tile_h=tile[1], freqs=(30e6, 60e6, 20e6)[:n_freq])
    F = 4096 // (cfg.tiles_x * cfg.tiles_y) + 1
    frames = scenes.identity_frames(np.linspace(0.0, 0.2, F), 167, 165, 1.2 * 167, 1.2 * 167, cfg.n_quad,
                                    bg_seed=3, n_freq=n_freq)
    up = scenes.upstream_grads(F, cfg, seed=2)
    res = run_gpu(wl.gaussians, frames, cfg, upstream=up)
    sums = {}
    for f in range(F):
        one = run_gpu(wl.gaussians, frames[f:f + 1], cfg, upstream={k: v[f:f + 1] for k, v in up.items()})
        for k in ("rgb", "quad", "depth", "T_final", "n_contrib"):
            assert np.array_equal(one[k][0], res[k][f]), k
        for k, v in one["grads"].items():
            if v is not None:
                sums[k] = sums.get(k, 0.0) + v.astype(np.float64)
    for k, v in sums.items():
        # float32 sums of the same terms in another order
        assert_grads_close(res["grads"][k], v, k, rtol=GRAD_RTOL * 1e-2)


# the preprocess backward packs the walked Gaussians of a workgroup when it
# has more than one round of them (here 256 Gaussians, 16 or 8 a round), and
# writes zeros for the others: against the per-frame calls, which do not pack
@pytest.mark.parametrize("n_frames,sh", [(9, False), (17, False), (9, True)])
def test_packed_preprocess_backward(n_frames, sh):
    n = 70_001
    g = scenes.draw_gaussians(n, 64, 48, 60.0, 60.0, seed=4, dynamic=True, log_scale_mean=float(np.log(0.02)))
    if sh:
        g = scenes.with_sh(g, degree=2, seed=1)
    g.delta = np.random.default_rng(0).normal(0.0, 0.01, (n_frames, 3, n)).astype(np.float32)
    cfg = scenes.RenderConfig(width=64, height=48)
    frames = scenes.identity_frames(np.linspace(0.0, 0.3, n_frames), 64, 48, 60.0, 60.0, 4)
    up = scenes.upstream_grads(n_frames, cfg, seed=2)
    res = run_gpu(g, frames, cfg, upstream=up)
    sums = {}
    for f in range(n_frames):
        one = run_gpu(dataclasses.replace(g, delta=g.delta[f:f + 1].copy()), frames[f:f + 1], cfg,
                      upstream={k: v[f:f + 1] for k, v in up.items()})
        # float32 sums of the same terms in another order
        assert_grads_close(res["grads"]["delta"][f], one["grads"]["delta"][0], f"delta {f}", rtol=GRAD_RTOL * 1e-2)
        for k, v in one["grads"].items():
            if v is not None and k != "delta":
                sums[k] = sums.get(k, 0.0) + v.astype(np.float64)
    assert any((v == 0).all(axis=tuple(range(v.ndim - 1))).any() for v in sums.values())   # some have no gradient
    for k, v in sums.items():
        assert_grads_close(res["grads"][k], v, k, rtol=GRAD_RTOL * 1e-2)


# the backward of few tiles walks a list in segments of 64-entry batches, as
# many as there are kept marks (64), the last one to the end: lists of one
# batch, of a few, one entry into a batch, and past the last mark
@pytest.mark.parametrize("tile", [(8, 8), (16, 16), (32, 8)])
@pytest.mark.parametrize("n", [40, 64, 65, 400, 4300])
def test_split_backward_walk(n, tile):
    wl = scenes.tiny_scene(n, 37, 19, seed=n, log_scale_mean=float(np.log(0.6)))
    rng = np.random.default_rng(n)
    # faint, so that no pixel stops before the end of its list
    wl.gaussians.opacity_logit[:] = rng.uniform(-5.2, -4.5 if n > 1000 else -1.0, n).astype(np.float32)
    cfg = dataclasses.replace(wl.cfg, tile_w=tile[0], tile_h=tile[1], T_min=0.0)
    frames = scenes.identity_frames([0.0], 37, 19, wl.frames[0].fx, wl.frames[0].fy, 4, bg_seed=1)
    base = oref.render(wl.gaussians, frames, cfg)
    up = mask_upstream(scenes.upstream_grads(1, cfg, seed=5), ~base["flagged"])
    ref = oref.render(wl.gaussians, frames, cfg, upstream=up)
    res = run_gpu(wl.gaussians, frames, cfg, upstream=up, want_bg=True)
    assert res["n_contrib"].max() > 0.5 * n
    for k in ("mean", "scale", "quat", "opacity_logit", "rgb", "albedo"):
        assert_grads_close(res["grads"][k], ref["grads"][k], k)
    assert_grads_close(res["grad_bg"], np.concatenate([ref["grad_bg_rgb"], ref["grad_bg_quad"]], 1), "bg")


# depths over more than the 16 octaves past near_z that three sort passes
# resolve, in the one-launch and the three-launch passes: the fourth pass runs
# and its result is the one that is read
@pytest.mark.parametrize("n,F", [(1, 1), (5000, 2), (2048 * 128 + 5, 2)])
@pytest.mark.parametrize("near,far", [(1e-6, 1.0), (0.0, 1.0), (0.2, 1e5), (0.2, 2.0 ** 14)])
def test_depth_sort_wide_range(n, F, near, far):
    W, H = 96, 72
    g = scenes.draw_gaussians(n, W, H, 80.0, 80.0, seed=41)
    rng = np.random.default_rng(42)
    move = rng.random(n) < 0.3
    s = np.where(move, far, 1.0)
    g.mean[:] = (g.mean * s).astype(np.float32)
    g.mean[2, ::7] = np.float32(-1.0)   # culled
    frames = scenes.identity_frames([0.1 * f for f in range(F)], W, H, 80.0, 80.0, 4)
    cfg = dataclasses.replace(scenes.RenderConfig(width=W, height=H), near_z=near)
    res = run_gpu(g, frames, cfg, channels=("rgb",))
    lists = gpu_lists(res, g, frames, cfg, pairs_to_host=n < 10000)
    key = np.concatenate([obin.project(g, fr, cfg, f)["key"] for f, fr in enumerate(frames)]).astype(np.int64)
    want = np.concatenate([f * n + np.argsort(key[f * n:(f + 1) * n], kind="stable") for f in range(F)])
    np.testing.assert_array_equal(lists["depth_item"].astype(np.int64), want)
    np.testing.assert_array_equal(lists["depth_key"].astype(np.int64), key[want])
    if n < 10000:
        pairs = obin.sorted_pairs(g, frames, cfg)
        assert np.array_equal(lists["pair_item"], (pairs["frame"] * n + pairs["index"]).astype(np.uint32))


# frames sorted by one workgroup in LDS: every number of keys per thread it
# has, at its limits, up to the largest frame and one past it; runs of equal
# depths and culled items among them
@pytest.mark.parametrize("n,F", [(63, 1), (1025, 3), (2048, 2), (2049, 1), (4096, 1), (4097, 2), (8192, 1), (8193, 2),
                                 (16385, 2)])
def test_depth_sort_small_frames(n, F):
    W, H = 96, 72
    g = scenes.draw_gaussians(n, W, H, 80.0, 80.0, seed=51)
    rng = np.random.default_rng(52)
    tie = rng.random(n) < 0.4
    g.mean[2] = np.where(tie, np.float32([1.5, 2.5, 4.0])[rng.integers(0, 3, n)], g.mean[2])
    g.mean[2, ::11] = np.float32(-1.0)
    frames = scenes.identity_frames([0.1 * f for f in range(F)], W, H, 80.0, 80.0, 4)
    cfg = scenes.RenderConfig(width=W, height=H)
    res = run_gpu(g, frames, cfg, channels=("rgb",))
    lists = gpu_lists(res, g, frames, cfg)
    key = np.concatenate([obin.project(g, fr, cfg, f)["key"] for f, fr in enumerate(frames)]).astype(np.int64)
    want = np.concatenate([f * n + np.argsort(key[f * n:(f + 1) * n], kind="stable") for f in range(F)])
    np.testing.assert_array_equal(lists["depth_item"].astype(np.int64), want)
    np.testing.assert_array_equal(lists["depth_key"].astype(np.int64), key[want])
    rect = np.concatenate([obin.project(g, fr, cfg, f)["rect"].T for f, fr in enumerate(frames)])
    valid = lists["count"] > 0
    got = lists["rect"]
    got = np.stack([got[:, 0] & 0xFFFF, got[:, 0] >> 16, got[:, 1] & 0xFFFF, got[:, 1] >> 16], 1)
    np.testing.assert_array_equal(got[valid], rect[valid])


# the preprocess splits the frames of few Gaussians over workgroups: every
# frame in its own, several frames in each of some, all in one; with the
# harmonics' coefficients of every degree kept for all of a thread's frames
@pytest.mark.parametrize("n,F,degree", [(300, 7, 0), (300, 7, None), (40_000, 5, None), (40_000, 5, 1), (40_000, 5, 3),
                                        (131_073, 3, 2)])
def test_preprocess_frame_split(n, F, degree):
    g = scenes.draw_gaussians(n, 64, 48, 60.0, 60.0, seed=4, dynamic=True, log_scale_mean=float(np.log(0.02)))
    if degree is not None:
        g = scenes.with_sh(g, degree=degree, seed=1)
    g.mean[0, 5] = np.nan   # counted once however the frames are split
    cfg = scenes.RenderConfig(width=64, height=48, freqs=(30e6, 60e6, 20e6))
    frames = scenes.identity_frames(np.linspace(0.0, 0.3, F), 64, 48, 60.0, 60.0, cfg.n_quad, n_freq=3)
    res = run_gpu(g, frames, cfg)
    lists = gpu_lists(res, g, frames, cfg)
    assert res["status"]["nonfinite"] == 1
    for f in range(F):
        one = run_gpu(g, frames[f:f + 1], cfg)
        l1 = gpu_lists(one, g, frames[f:f + 1], cfg)
        sel = slice(f * n, (f + 1) * n)
        np.testing.assert_array_equal(lists["depth_key"][sel], l1["depth_key"])
        np.testing.assert_array_equal(lists["depth_item"][sel] - np.uint32(f * n), l1["depth_item"])
        np.testing.assert_array_equal(lists["count"][sel], l1["count"])
        np.testing.assert_array_equal(lists["rect"][sel], l1["rect"])
        ok = np.ones((1, 48, 64), bool)
        for k in ("rgb", "quad", "depth"):
            assert_images_close(res[k][f:f + 1], one[k], ok, k, rtol=1e-6)


# the forward's waves leave out the entries that no pixel of their box can
# take: thin and round splats in every direction, opacities down to alpha_min
# and below, nothing below any threshold (alpha_min 0), boxes cut by the image
@pytest.mark.parametrize("tile,size", [((8, 8), (61, 45)), ((16, 16), (61, 45)), ((32, 8), (70, 45)),
                                       ((16, 16), (1030, 1021)), ((32, 8), (1030, 1021))])
@pytest.mark.parametrize("alpha_min", [1.0 / 255.0, 0.0, 0.05])
def test_forward_box_test(tile, size, alpha_min):
    W, H = size
    n = 700
    g = scenes.draw_gaussians(n, W, H, 1.2 * W, 1.2 * W, seed=W,
                              log_scale_mean=float(np.log((2.0 if W < 100 else 12.0) / W)))
    rng = np.random.default_rng(7)
    g.scale[:] = (g.scale * np.exp(rng.uniform(-2.5, 2.5, g.scale.shape))).astype(np.float32)
    g.quat[:] = rng.normal(size=g.quat.shape).astype(np.float32)
    g.opacity_logit[:] = rng.uniform(-6.0, 3.0, n).astype(np.float32)
    cfg = scenes.RenderConfig(width=W, height=H, tile_w=tile[0], tile_h=tile[1], alpha_min=alpha_min)
    frames = scenes.identity_frames([0.0], W, H, 1.2 * W, 1.2 * W, cfg.n_quad, bg_seed=1)
    ref = oref.render(g, frames, cfg)
    ok = ~ref["flagged"]
    assert ok.mean() > 0.9
    res = run_gpu(g, frames, cfg)
    for k in ("rgb", "quad", "depth", "T_final"):
        assert_images_close(res[k], ref[k], ok, k)
    np.testing.assert_array_equal(res["n_contrib"][ok], ref["n_contrib"][ok])


# the status's sums over the work items: one, and more and fewer than a round
# of the summing workgroup, read by several threads on streams of their own
def test_status_sums():
    # nothing is skipped or stopped: every pixel composites every Gaussian
    cases = [(1, 5, 3, 1), (4, 640, 260, 3), (3, 1024, 768, 1)]
    errors = []

    def work(n, W, H, F):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                g = scenes.draw_gaussians(n, W, H, float(W), float(W), seed=n, log_scale_mean=float(np.log(0.5)))
                cfg = dataclasses.replace(scenes.RenderConfig(width=W, height=H, tile_w=8, tile_h=8).strict(),
                                          alpha_max=0.5)
                frames = scenes.identity_frames([0.0] * F, W, H, float(W), float(W), cfg.n_quad)
                res = run_gpu(g, frames, cfg, max_pairs=1 << 20)
                for _ in range(20):
                    st = res["_ws"].status(stream)
                    assert st["n_evaluated"] == st["n_composited"] == n * W * H * F
        except BaseException as e:   # handed to the test's own thread
            errors.append((n, W, H, F, e))

    threads = [threading.Thread(target=work, args=c) for c in cases]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors


# between 2048 and 4096 tiles the forward has two waves per tile and the
# backward is split: one frame, and the same frame as often as that takes
@pytest.mark.parametrize("tile,n_freq", [((16, 16), 1), ((16, 16), 4), ((32, 8), 2)])
def test_two_waves_and_split_backward(tile, n_freq):
    n, F = 500, 342
    wl = scenes.tiny_scene(n, 37, 19, seed=n, log_scale_mean=float(np.log(0.6)))
    wl.gaussians.opacity_logit[:] = np.random.default_rng(n).uniform(-5.2, -3.0, n).astype(np.float32)
    cfg = dataclasses.replace(wl.cfg, tile_w=tile[0], tile_h=tile[1], T_min=0.0, freqs=(30e6, 60e6, 20e6, 50e6)[:n_freq])
    F = F * 6 // (cfg.tiles_x * cfg.tiles_y)
    assert 2048 <= F * cfg.tiles_x * cfg.tiles_y < 4096
    fx = wl.frames[0].fx
    frames = scenes.identity_frames([0.0] * F, 37, 19, fx, fx, cfg.n_quad, bg_seed=1, n_freq=n_freq)
    frames = [frames[0]] * F
    up1 = scenes.upstream_grads(1, cfg, seed=5)
    one = run_gpu(wl.gaussians, frames[:1], cfg, upstream=up1)
    res = run_gpu(wl.gaussians, frames, cfg, upstream={k: np.repeat(v, F, 0) for k, v in up1.items()})
    ok = np.ones((1, 19, 37), bool)
    for f in (0, F // 2, F - 1):
        np.testing.assert_array_equal(res["n_contrib"][f], one["n_contrib"][0])
        for k in ("rgb", "quad", "depth"):
            assert_images_close(res[k][f:f + 1], one[k], ok, k, rtol=1e-6)
    for k, v in one["grads"].items():
        if v is not None:   # float32 sums of the same terms in another order
            assert_grads_close(res["grads"][k], v.astype(np.float64) * F, k, rtol=GRAD_RTOL * 1e-2)
