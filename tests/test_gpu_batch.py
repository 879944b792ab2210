"""Batched multi-view rendering, its HIP-graph replay and the autotuner."""
import numpy as np
import pytest
import torch

from oracle import composite as oc
from paper_2503_16422_amd import _lib, inputs
from tests.gpu_helpers import compare_image, oracle_settings

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2503_16422_amd.render import Context
    c = Context(0)
    yield c
    c.close()


@pytest.fixture(scope="module")
def batch_setup(ctx):
    from paper_2503_16422_amd.render import GaussianModel
    sizes = [2000, 5000, 9000]
    scenes = [inputs.long_scene(n, seed=s) for s, n in enumerate(sizes)]
    models = [GaussianModel.from_scene(sc, "cuda:0") for sc in scenes]
    cams = inputs.batch_cameras(120, 96)
    frames = inputs.frame_times(64)
    views = []
    masks = {}
    rng = np.random.default_rng(0)
    for k in range(11):
        s = int(rng.integers(0, 3))
        c = int(rng.integers(0, 4))
        f = int(rng.integers(0, 64))
        if k % 3 == 0:       # a masked view: active set of the window around f
            lo, hi = max(0, f - 6), min(63, f + 6)
            if (s, lo) not in masks:
                _, idx, cnt = ctx.build_active_mask(models[s], frames[lo:hi + 1], frames[lo], frames[hi],
                                                    _lib.MASK_TEMPORAL)
                masks[(s, lo)] = (idx, int(cnt.item()))
            idx, n = masks[(s, lo)]
            views.append((s, cams[c], float(frames[f]), idx, n))
        else:
            views.append((s, cams[c], float(frames[f])))
    return scenes, models, views


def single(ctx, models, v, cfg):
    if len(v) > 3:
        n_idx = torch.tensor([v[4]], dtype=torch.int64, device="cuda")
        return ctx.render(models[v[0]], v[1], v[2], cfg, idx=v[3], n_idx=n_idx)[0]
    return ctx.render(models[v[0]], v[1], v[2], cfg)[0]


@pytest.mark.parametrize("per_launch", [0, 4, 1])
def test_batch_equals_single_views(ctx, batch_setup, per_launch):
    scenes, models, views = batch_setup
    cfg = _lib.default_cfg()
    out = ctx.render_batch(models, views, cfg, views_per_launch=per_launch)
    for k, v in enumerate(views):
        ref = single(ctx, models, v, cfg)
        assert torch.equal(out[k], ref), k


def test_batch_matches_oracle(ctx, batch_setup):
    scenes, models, views = batch_setup
    out = ctx.render_batch(models, views[:4]).cpu().numpy()
    st = oracle_settings()
    for k, v in enumerate(views[:4]):
        idx = v[3][: v[4]].cpu().numpy().view(np.uint32).astype(np.int64) if len(v) > 3 else None
        ref = oc.render(scenes[v[0]].arrays(), v[1], v[2], st, idx=idx, mode="rect")
        compare_image(out[k], ref)


def test_graph_replays_match_eager(ctx, batch_setup):
    scenes, models, views = batch_setup
    cfg = _lib.default_cfg(instance_capacity=400_000)
    eager = ctx.render_batch(models, views, cfg, views_per_launch=4).clone()
    out = torch.zeros_like(eager)
    for rep in range(4):
        out.zero_()
        ctx.render_batch(models, views, cfg, views_per_launch=4, use_graph=True, out=out)
        torch.cuda.synchronize()
        assert torch.equal(out, eager), rep
        # unrelated eager work between replays
        ctx.render(models[0], views[1][1], 0.3)
        torch.cuda.synchronize()
    ctx.check_overflow()
    # a changed view rebuilds the graph
    views2 = list(views)
    views2[2] = (views[2][0], views[2][1], 0.77)
    out2 = ctx.render_batch(models, views2, cfg, views_per_launch=4, use_graph=True)
    ref2 = single(ctx, models, views2[2], _lib.default_cfg())
    assert torch.equal(out2[2], ref2)
    assert torch.equal(out2[0], eager[0])


def test_autotune_configs_identical(ctx, batch_setup):
    scenes, models, views = batch_setup
    best, results = ctx.autotune(models, views[:5], repeats=2)
    assert len(results) == 90
    assert all(r["identical"] for r in results)
    assert (best.tile_w, best.tile_h) in [(8, 8), (16, 16), (32, 8), (32, 16), (32, 32)]
    assert best.batch in (64, 128, 256, 512, 1024) and best.pixels_per_thread in (1, 2, 4)
    fastest = min(results, key=lambda r: r["ms"])
    assert fastest["ms"] > 0


def test_batched_workload_at_full_size(ctx):
    """A slice of the batched workload at its real shape: two of its scenes
    (50k and 400k Gaussians), 800x800, keyframe-window masks with the tile
    test, 256 views rendered in launches of 128 views through a captured HIP
    graph (replayed with unrelated work in between) and eagerly.  Every view
    equals its single-view render bit for bit, and three views match the
    oracle on every pixel."""
    from paper_2503_16422_amd.render import GaussianModel
    sizes = inputs.batched_scene_sizes()
    picks = [0, len(sizes) - 1]
    scenes = [inputs.long_scene(sizes[s], seed=s) for s in picks]
    models = [GaussianModel.from_scene(sc, "cuda:0") for sc in scenes]
    cams = inputs.batch_cameras(800, 800)
    frames = inputs.frame_times(64)
    keys = [0, 13, 26, 39, 52, 63]
    masks = {}
    for s, m in enumerate(models):
        for w in range(len(keys) - 1):
            lo, hi = keys[w], keys[w + 1]
            _, idx, cnt = ctx.build_active_mask(m, frames[lo:hi + 1], frames[lo], frames[hi],
                                                _lib.MASK_TEMPORAL_AND_TILE, cams)
            masks[(s, w)] = (idx, int(cnt.item()))
    win = lambda f: min(int(np.searchsorted(keys, f, side="right")) - 1, len(keys) - 2)
    views = []
    for f in range(0, 64, 2):
        for c in range(4):
            for s in range(len(models)):
                idx, n = masks[(s, win(f))]
                views.append((s, cams[c], float(frames[f]), idx, n))
    assert len(views) == 256
    cfg = _lib.default_cfg(tile_w=32, tile_h=32, batch=512, pixels_per_thread=2, schedule=1)
    ctx.profile(True)
    eager = ctx.render_batch(models, views, cfg, views_per_launch=128)
    prof = ctx.profile_read(reset=True)
    ctx.profile(False)
    torch.cuda.synchronize()
    for k, v in enumerate(views):
        assert torch.equal(eager[k], single(ctx, models, v, cfg)), k
    # the largest launch holds at most all instances; the benchmark sizes it the same way
    cfg.instance_capacity = int(prof["instances"]) + 65536
    out = torch.zeros_like(eager)
    for rep in range(3):
        out.zero_()
        ctx.render_batch(models, views, cfg, views_per_launch=128, use_graph=True, out=out)
        torch.cuda.synchronize()
        assert torch.equal(out, eager), rep
        ctx.render(models[0], cams[1], 0.3)
        torch.cuda.synchronize()
    ctx.check_overflow()
    host = eager.cpu().numpy()
    del out, eager
    st = oracle_settings()
    for k in (0, 101, 255):
        s, cam, t, idx, n = views[k]
        sel = idx[:n].cpu().numpy().view(np.uint32).astype(np.int64)
        ref = oc.render(scenes[s].arrays(), cam, t, st, idx=sel, mode="rect")
        worst, nflag = compare_image(host[k], ref, label=f"batched 800x800 view {k}")
        print(f"batched view {k} (scene {picks[s]}): max err {worst:.2e}, flagged {nflag}")


def test_profile_counts_processed_entries_without_padding(ctx, batch_setup):
    """The profile's processed count of batched views (uneven, one empty, one
    entry) and of the score pass, whose views share launches, is the sum of the
    views' own entries."""
    _, models, _ = batch_setup
    cam = inputs.batch_cameras(120, 96)[0]
    idx = torch.arange(2000, dtype=torch.int32, device="cuda")
    views = [(0, cam, 0.5, idx, 0), (0, cam, 0.5, idx, 1), (1, cam, 0.4), (0, cam, 0.3, idx, 1999), (2, cam, 0.6)]
    ctx.profile(True)
    ctx.render_batch(models, views)
    batch = ctx.profile_read(reset=True)["processed"]
    ctx.spatial_score(models[1], [(cam, 0.2), (cam, 0.5), (cam, 0.8)])
    side = ctx.profile_read(reset=True)["processed"]
    ctx.profile(False)
    assert batch == 0 + 1 + 5000 + 1999 + 9000
    assert side == 3 * 5000


def test_many_tiny_views_beside_a_large_one(ctx):
    """1500 views of 40 Gaussians and one of 60,000 in one call, more views than
    one launch takes.  Every image is the single view's."""
    from paper_2503_16422_amd.render import GaussianModel
    models = [GaussianModel.from_scene(inputs.long_scene(n, seed=n), "cuda:0") for n in (40, 60_000)]
    cams = inputs.batch_cameras(16, 12)
    kinds = [(0, cams[k % 4], 0.1 + 0.2 * (k % 5)) for k in range(20)]
    views = [kinds[k % 20] for k in range(1500)]
    views.insert(700, (1, cams[1], 0.5))
    out = ctx.render_batch(models, views)
    ref = [single(ctx, models, v, _lib.default_cfg()) for v in kinds]
    assert torch.equal(out[700], single(ctx, models, views[700], _lib.default_cfg()))
    rest = torch.cat([out[:700], out[701:]])
    for k in range(20):
        assert torch.equal(rest[k::20], ref[k].expand_as(rest[k::20])), k
