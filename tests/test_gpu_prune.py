"""Pruning with the spatial-temporal variation score (Sec. 4.2.1) against the FP64 oracle."""
import numpy as np
import pytest
import torch

from oracle import prune as oprune
from paper_2503_16422_amd import inputs
from tests.gpu_helpers import oracle_settings

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2503_16422_amd.render import Context
    c = Context(0)
    yield c
    c.close()


def _scene():
    sc = inputs.tiny_scene(8000, seed=12)
    sc.log_scale[:3] += 0.6
    sc.mean[:, 5] = np.nan                     # an invalid Gaussian scores 0
    return sc


def test_spatial_score_matches_oracle_and_telescopes(ctx):
    from paper_2503_16422_amd.render import GaussianModel
    sc = _scene()
    model = GaussianModel.from_scene(sc, "cuda:0")
    views = [(inputs.look_at_camera(phi, 3.0, 96, 80), t) for phi, t in ((0.0, 0.5), (25.0, 0.45), (-25.0, 0.55))]
    got = ctx.spatial_score(model, views).cpu().numpy().astype(np.float64)
    ref, slack = oprune.spatial_score(sc.arrays(), views, oracle_settings(), with_slack=True)
    assert got[5] == 0.0
    err = np.abs(got - ref)
    # float32 weights within 2e-4 of the FP64 ones, plus what the pixels whose
    # decisions sit near a threshold may move (the oracle's slack)
    assert np.all(err <= 2e-4 * ref + 1e-6 * ref.max() + 1e-7 + slack), float(err.max())
    # per view, the scores add up to the sum over pixels of 1 - T_final
    for cam, t in views:
        one = ctx.spatial_score(model, [(cam, t)]).double()
        _, T, _ = ctx.render(model, cam, t, want_T=True)
        assert abs(float(one.sum()) - float((1.0 - T.double()).sum())) <= 1e-4 * T.numel()
    print(f"spatial score: {np.count_nonzero(got)} Gaussians scored, max rel err "
          f"{float((err / np.maximum(ref, 1e-12))[ref > 1e-3 * ref.max()].max()):.1e}")


def _saturated_scene():
    # larger, more opaque Gaussians present at every time: almost every pixel
    # stops early (T < 1e-3), at different positions of its tile list
    sc = inputs.tiny_scene(20_000, seed=5)
    sc.log_scale[:3] += 0.3
    sc.log_scale[3] += 3.0
    sc.opacity_logit[:] += 1.0
    return sc


@pytest.mark.parametrize("tile,ppt,batch", [((16, 16), 2, 256), ((16, 16), 4, 64), ((16, 16), 1, 128),
                                            ((32, 8), 2, 128), ((32, 8), 4, 256), ((8, 8), 1, 64),
                                            ((32, 16), 2, 256), ((32, 32), 4, 128), ((32, 32), 2, 64),
                                            ((32, 32), 2, 1024)])
def test_spatial_score_with_early_stops_and_ragged_edges(ctx, tile, ppt, batch):
    """Pixels that stop early and pixels outside a ragged image leave their
    lanes idle while the rest of the wavefront blends on: every blend weight
    must still reach the score (per view, the scores add up to the sum of
    1 - T_final), in every tile shape and pixels-per-thread layout."""
    from paper_2503_16422_amd import _lib
    from paper_2503_16422_amd.render import GaussianModel
    sc = _saturated_scene()
    model = GaussianModel.from_scene(sc, "cuda:0")
    cfg = _lib.default_cfg(tile_w=tile[0], tile_h=tile[1], pixels_per_thread=ppt, batch=batch)
    views = [(inputs.look_at_camera(phi, 3.0, 93, 71), t) for phi, t in ((10.0, 0.5), (-30.0, 0.4))]
    total = None
    for cam, t in views:
        one = ctx.spatial_score(model, [(cam, t)], cfg).double()
        _, T, _ = ctx.render(model, cam, t, cfg, want_T=True)
        assert float((T < 1e-3).double().mean()) > 0.5
        blended = float((1.0 - T.double()).sum())
        assert abs(float(one.sum()) - blended) <= 1e-5 * blended, (float(one.sum()), blended)
        total = one if total is None else total + one
    ref, slack = oprune.spatial_score(sc.arrays(), views, oracle_settings(), with_slack=True)
    got = total.cpu().numpy()
    assert abs(got.sum() - ref.sum()) <= 1e-4 * ref.sum()
    # every Gaussian: float32 weights within 2e-4 of the FP64 ones, plus the
    # oracle's slack for the pixels whose stop or alpha decisions sit near a
    # threshold (a float32 walk may take those the other way)
    err = np.abs(got - ref)
    bad = err > 2e-4 * ref + 1e-6 * ref.max() + 1e-7 + slack
    assert not bad.any(), (int(bad.sum()), float(err[bad].max()))
    print(f"early-stop scores {tile} ppt {ppt} batch {batch}: {int((slack > 0).sum())} Gaussians with slack, "
          f"max err {float(err.max()):.2e}")


def test_variation_score_and_prune_match_oracle(ctx):
    from paper_2503_16422_amd.render import GaussianModel
    sc = _scene()
    model = GaussianModel.from_scene(sc, "cuda:0")
    views = [(inputs.look_at_camera(phi, 3.0, 96, 80), t) for phi, t in ((10.0, 0.3), (-10.0, 0.6))]
    spatial = ctx.spatial_score(model, views)
    times = inputs.frame_times(300)[::7]
    score = ctx.variation_score(model, times, spatial)
    got = score.cpu().numpy().astype(np.float64)
    ref = oprune.variation_score(sc.arrays(), spatial.cpu().numpy().astype(np.float64), times)
    assert got[5] == 0.0
    assert np.all(np.abs(got - ref) <= 1e-5 * np.abs(ref) + 1e-9 * np.abs(ref).max())
    # selection: exact, on the GPU's own scores (ties by index)
    s32 = score.cpu().numpy()
    for keep in (0, 1, 1600, 4000, sc.n):
        bits, idx, count = ctx.prune(score, keep)
        n = int(count.item())
        want = oprune.prune(s32.astype(np.float64), keep)
        assert n == want.size
        assert np.array_equal(idx[:n].cpu().numpy().view(np.uint32), want)
        unpacked = ((bits.cpu().numpy().view(np.uint32)[:, None] >> np.arange(32, dtype=np.uint32)) & 1)
        keepmask = np.zeros(sc.n, dtype=bool)
        keepmask[want] = True
        assert np.array_equal(unpacked.astype(bool).ravel()[:sc.n], keepmask)


@pytest.mark.parametrize("n", [1, 300, 4096, 9000])
def test_side_passes_share_launches(ctx, n):
    """Visibility marks and blend weights over views of two image sizes, which
    share launches where neighbours agree in size, are those of one call per
    view: the marks exactly, the weights up to the order of their float32
    additions (a few hundred per Gaussian at most)."""
    from paper_2503_16422_amd.render import GaussianModel
    model = GaussianModel.from_scene(inputs.long_scene(n, seed=21), "cuda:0")
    sizes = [(96, 80), (96, 80), (203, 60), (96, 80), (96, 80)]
    cams = [inputs.look_at_camera(0.15 * k, 3.0, w, h) for k, (w, h) in enumerate(sizes)]
    bits, idx, count = ctx.build_active_mask(model, (), 0.25, 0.5, 2, cams)
    ref = torch.zeros_like(bits)
    for cam in cams:
        for key in (0.25, 0.5):
            ref |= ctx.build_active_mask(model, (), key, key, 2, [cam])[0]
    assert torch.equal(bits, ref)
    keep = torch.tensor([(int(w) >> b) & 1 for w in ref.tolist() for b in range(32)][:n], dtype=torch.bool).nonzero()[:, 0]
    assert int(count.item()) == keep.numel() and torch.equal(idx[:keep.numel()].cpu().long(), keep)
    views = [(c, 0.1 * k) for k, c in enumerate(cams)]
    got = ctx.spatial_score(model, views)
    one = torch.zeros_like(got)
    for v in views:
        ctx.spatial_score(model, [v], out=one)
    assert torch.allclose(got, one, rtol=1e-5, atol=1e-5)


def test_score_pass_over_more_tiles_than_one_launch_can_number(ctx):
    """512 views of 16384 x 16384 pixels in 8x8 tiles are 2^31 tiles, one more than
    fits a launch's numbering; each view alone is in order.  The pass takes them
    in smaller groups and scores the Gaussians that one view scores.  (2^31
    workgroups: about 20 s.  The sums themselves, 10^6 float32 additions each,
    have no tight bound.)"""
    from paper_2503_16422_amd import _lib
    from paper_2503_16422_amd.render import GaussianModel
    sc = inputs.tiny_scene(16, seed=3)
    sc.log_scale[:3] -= 1.0
    sc.log_scale[3] = 1.0
    model = GaussianModel.from_scene(sc, "cuda:0")
    cfg = _lib.default_cfg(tile_w=8, tile_h=8, batch=64, pixels_per_thread=1, schedule=0)
    view = (inputs.look_at_camera(0.0, 3.0, 16384, 16384), 0.5)
    one = ctx.spatial_score(model, [view], cfg)
    assert float(one.max()) > 0
    many = ctx.spatial_score(model, [view] * 512, cfg)
    assert torch.equal(many > 0, one > 0)
    assert torch.all(many >= one)


def test_variation_score_of_vanishing_lifespans(ctx):
    """Temporal scales of e^-178 to e^-20 (spatial ones that keep the volumes in
    float32's range): the scores that the float64 formula keeps finite, although
    1 / S44^2 overflows, are finite and the oracle's (1e-5: float32 score, volume's
    power)."""
    from paper_2503_16422_amd.render import GaussianModel
    ls = np.concatenate([np.linspace(-178.2, -176.8, 81), np.linspace(-170.0, -20.0, 31)])
    sc = inputs.tiny_scene(ls.size, seed=4)
    sc.log_scale[:3] = 31.0
    sc.log_scale[3] = ls.astype(np.float32)
    for q in (sc.q_left, sc.q_right):
        q[:] = np.array([1.0, 0.0, 0.0, 0.0])[:, None]
    times = inputs.frame_times(30)
    spatial = np.ones(ls.size, np.float32)
    got = ctx.variation_score(GaussianModel.from_scene(sc, "cuda:0"), times, torch.from_numpy(spatial).cuda()).cpu().numpy()
    with np.errstate(over="ignore", under="ignore", invalid="ignore", divide="ignore"):
        ref = oprune.variation_score(sc.arrays(), spatial.astype(np.float64), times)
    fine = np.isfinite(ref)
    assert fine.sum() > 60
    assert np.all(np.isfinite(got[fine]))
    assert np.allclose(got[fine], ref[fine], rtol=1e-5)
