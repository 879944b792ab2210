"""SH vector quantisation (post-processing) on the GPU against the float64
k-means oracle, and rendering from a codebook."""
import numpy as np
import pytest
import torch

from oracle import vq
from paper_2503_16422_amd import _lib, inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2503_16422_amd.render import Context
    c = Context(0)
    yield c
    c.close()


def model_of(sc):
    from paper_2503_16422_amd.render import GaussianModel
    return GaussianModel.from_scene(sc, "cuda:0")


def check_assignment(x, c, a, rel=2e-5):
    """Every GPU choice is a nearest entry up to float32 accumulation error,
    and is the oracle's where the nearest entry is clear of the second."""
    d = vq.squared_distances(x, c)
    dmin = d.min(axis=1)
    tol = rel * (1.0 + dmin + np.einsum("nd,nd->n", x, x))
    chosen = d[np.arange(x.shape[0]), a]
    assert np.all(chosen <= dmin + tol)
    ref = vq.assign(x, c)
    srt = np.sort(d, axis=1)
    clear = srt[:, 1] - srt[:, 0] > 2 * tol
    assert np.array_equal(a[clear], ref[clear])
    return int(clear.sum())


def test_initial_codebook_and_assignment(ctx):
    sc = inputs.tiny_scene(3000, seed=11)
    model = model_of(sc)
    init = torch.from_numpy(np.random.default_rng(0).choice(3000, 64, replace=False).astype(np.int32)).cuda()
    code, assign = ctx.sh_kmeans(model, 64, 0, init_index=init)
    torch.cuda.synchronize()
    x = vq.sh_vectors(sc.sh)
    assert np.array_equal(code.cpu().numpy(), x[init.cpu().numpy()].astype(np.float32))
    n_clear = check_assignment(x, code.cpu().numpy().astype(np.float64), assign.cpu().numpy().astype(np.int64))
    assert n_clear > 2900


def test_update_step_is_the_float64_mean(ctx):
    """One Lloyd step from the same start: the new codebook is the float64
    mean of each cluster (as assigned on the GPU), rounded once."""
    sc = inputs.tiny_scene(4000, seed=12)
    model = model_of(sc)
    init = torch.from_numpy(np.random.default_rng(1).choice(4000, 50, replace=False).astype(np.int32)).cuda()
    c0, a0 = ctx.sh_kmeans(model, 50, 0, init_index=init)
    c1, a1 = ctx.sh_kmeans(model, 50, 1, init_index=init)
    torch.cuda.synchronize()
    x = vq.sh_vectors(sc.sh)
    ref = vq.update(x, a0.cpu().numpy().astype(np.int64), c0.cpu().numpy().astype(np.float64))
    assert np.array_equal(c1.cpu().numpy(), ref.astype(np.float32))
    check_assignment(x, c1.cpu().numpy().astype(np.float64), a1.cpu().numpy().astype(np.int64))


def test_separated_clusters_are_recovered(ctx):
    """SH vectors scattered tightly around 8 distant centres, one start per
    cluster: three iterations give the cluster means and the true labels; an
    index range past the model reads the last Gaussian."""
    rng = np.random.default_rng(13)
    sc = inputs.tiny_scene(800, seed=13)
    centres = rng.standard_normal((8, 48)) * 3.0
    truth = np.repeat(np.arange(8), 100)
    x = centres[truth] + 1e-3 * rng.standard_normal((800, 48))
    sc.sh = vq.planes_from_vectors(x).astype(np.float32)
    model = model_of(sc)
    init = torch.tensor([k * 100 for k in range(8)], dtype=torch.int32, device="cuda")
    code, assign = ctx.sh_kmeans(model, 8, 3, init_index=init)
    torch.cuda.synchronize()
    x32 = vq.sh_vectors(sc.sh)
    assert np.array_equal(assign.cpu().numpy(), truth)
    for k in range(8):
        assert np.allclose(code.cpu().numpy()[k], x32[truth == k].mean(axis=0), rtol=0, atol=1e-6)
    code2, _ = ctx.sh_kmeans(model, 2, 0, init_index=torch.tensor([5, 10 ** 6], dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    assert np.array_equal(code2.cpu().numpy()[1], x32[799].astype(np.float32))


def test_render_from_codebook_equals_materialised_sh(ctx):
    """Rendering with (index, codebook) is rendering the model whose SH planes
    hold each Gaussian's codebook entry: images bit-identical, also masked and
    through the batch path."""
    from paper_2503_16422_amd.render import GaussianModel
    sc = inputs.tiny_scene(6000, seed=14)
    model = model_of(sc)
    code, assign = ctx.sh_kmeans(model, 40, 4)
    torch.cuda.synchronize()
    mat = code[assign.long()]                                     # [n, 48]
    sh_planes = mat.reshape(-1, 16, 3).permute(1, 2, 0).contiguous()
    dense = GaussianModel(model.mean, model.log_scale, model.q_left, model.q_right, model.opacity_logit,
                          sh_planes, model.sh_degree)
    qmodel = model.quantized(assign, code)
    for phi, t in ((0.0, 0.5), (25.0, 0.3)):
        cam = inputs.look_at_camera(phi, 3.0, 120, 90)
        a, _, _ = ctx.render(qmodel, cam, t)
        b, _, _ = ctx.render(dense, cam, t)
        torch.cuda.synchronize()
        assert torch.equal(a, b)
    keep = torch.arange(0, 6000, 3, dtype=torch.int32, device="cuda")
    n_keep = torch.tensor([keep.numel()], dtype=torch.int64, device="cuda")
    a, _, _ = ctx.render(qmodel, cam, 0.5, idx=keep, n_idx=n_keep)
    b, _, _ = ctx.render(dense, cam, 0.5, idx=keep, n_idx=n_keep)
    torch.cuda.synchronize()
    assert torch.equal(a, b)
    views = [(0, inputs.look_at_camera(p, 3.0, 64, 48), t) for p, t in ((-10.0, 0.4), (5.0, 0.6))]
    qa = ctx.render_batch([qmodel, dense], views + [(1, v[1], v[2]) for v in views]).clone()
    torch.cuda.synchronize()
    assert torch.equal(qa[:2], qa[2:])


def test_backward_rejects_quantised_model(ctx):
    sc = inputs.tiny_scene(500, seed=15)
    model = model_of(sc)
    code, assign = ctx.sh_kmeans(model, 8, 1)
    q = model.quantized(assign, code)
    cam = inputs.look_at_camera(0.0, 3.0, 32, 32)
    rgb, _, st = ctx.render(q, cam, 0.5, keep_state=True)
    with pytest.raises(_lib.FdgsError):
        ctx.backward(st, torch.ones_like(rgb), q)
    ctx.release(st)


def chain_distances(x, c):
    """The distance that decides: float32 t = x - c, acc = fma(t, t, acc) in component order.  The
    square and the sum are formed in float64 and rounded once more, which can differ from a fused
    operation by one unit in the last place."""
    x, c = x.astype(np.float32), c.astype(np.float32)
    acc = np.zeros((x.shape[0], c.shape[0]), np.float32)
    with np.errstate(over="ignore", invalid="ignore"):
        for d in range(x.shape[1]):
            t = (x[:, None, d] - c[None, :, d]).astype(np.float64)
            acc = (t * t + acc.astype(np.float64)).astype(np.float32)
    return acc


@pytest.mark.parametrize("n,k", [(1, 1), (31, 2), (65, 31), (257, 33), (700, 64), (1030, 97), (2500, 300)])
@pytest.mark.parametrize("kind", ["plain", "twins", "extreme"])
def test_assignment_is_the_nearest_in_float32(ctx, n, k, kind):
    """The screened assignment is the float32 search's, at the edges of its tiles (32 entries, 64 and
    256 Gaussians, splits of the entries), with equal entries (the lower one wins) and with
    vectors of extreme size, infinities and NaN (no finite distance: entry 0).  Tolerance: one
    float32 unit, by which the reference's twice rounded sums may differ from fused ones."""
    sc = inputs.tiny_scene(max(n, k), seed=n + k)
    rng = np.random.default_rng(n * 1000 + k)
    if kind == "twins":
        sc.sh[..., :] = sc.sh[..., rng.integers(0, max(1, min(n, 5)), max(n, k))]
    if kind == "extreme":
        scale = 10.0 ** rng.integers(-30, 19, max(n, k))
        sc.sh *= scale.astype(np.float32)
        for v, i in ((np.inf, 0), (np.nan, 1), (-np.inf, 2)):
            if n > 40 * (i + 1):
                sc.sh[i, 1, rng.integers(0, n, 2)] = v
    model = model_of(sc)
    init = torch.from_numpy(rng.permutation(max(n, k))[:k].astype(np.int32)).cuda()
    code, assign = ctx.sh_kmeans(model, k, 0, init_index=init)
    torch.cuda.synchronize()
    d = chain_distances(vq.sh_vectors(sc.sh), code.cpu().numpy())
    a = assign.cpu().numpy()
    d = np.where(np.isnan(d), np.float32(np.inf), d)
    low = d.min(axis=1)
    got = d[np.arange(d.shape[0]), a]
    assert np.all(got <= np.nextafter(low, np.float32(np.inf)))
    clear = (d <= np.nextafter(np.nextafter(low, np.float32(np.inf)), np.float32(np.inf))[:, None]).sum(1) == 1
    ref = np.where(np.isinf(low), 0, d.argmin(axis=1))
    same = clear | np.isinf(low) | (d == low[:, None]).all(axis=1)
    assert np.array_equal(a[same], ref[same])
    if kind == "twins":
        c = code.cpu().numpy()                     # equal entries: always the lowest of them
        assert all(not (c[:a[i]] == c[a[i]]).all(axis=1).any() for i in range(a.size))


@pytest.mark.parametrize("n,k,iterations", [(1, 1, 0), (40, 1, 1), (300, 1, 2), (65, 2, 1), (700, 33, 0), (700, 33, 2),
                                            (300, 64, 1)])
@pytest.mark.parametrize("what", [np.nan, np.inf, 3e38, 1e30])
def test_codebooks_without_a_usable_entry(ctx, n, k, iterations, what):
    """Every entry (k <= 2), or all but two, starts from a Gaussian with a NaN, an
    infinite or an enormous coefficient; the others are of ordinary size or 1e10.  With
    one cluster a NaN also gets in by the first mean.  The assignment is the float32
    search's over the codebook returned (no finite distance: entry 0), never an entry
    past it; tolerance as above."""
    sc = inputs.tiny_scene(n, seed=n + k)
    rng = np.random.default_rng(n + k)
    sc.sh[:, :, ::3] *= np.float32(1e10)
    order = rng.permutation(n)[:min(n, k)]
    init = np.resize(order, k)
    bad = order if k <= 2 else order[2:]
    sc.sh[rng.integers(0, 16), rng.integers(0, 3), bad] = what
    model = model_of(sc)
    code, assign = ctx.sh_kmeans(model, k, iterations, init_index=torch.from_numpy(init.astype(np.int32)).cuda())
    torch.cuda.synchronize()
    a = assign.cpu().numpy()
    assert a.min() >= 0 and a.max() < k
    with np.errstate(over="ignore"):
        d = chain_distances(vq.sh_vectors(sc.sh), code.cpu().numpy())
    d = np.where(np.isnan(d), np.float32(np.inf), d)
    low = d.min(axis=1)
    got = d[np.arange(d.shape[0]), a]
    assert np.all((got <= np.nextafter(low, np.float32(np.inf))) | np.isinf(low))
    assert np.all(a[np.isinf(low)] == 0)
