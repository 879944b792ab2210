"""Calls whose scratch does not fit into the GPU's memory take their smaller form."""
import contextlib

import numpy as np
import pytest
import torch

from paper_2503_16422_amd import inputs

pytestmark = pytest.mark.gpu


@contextlib.contextmanager
def all_memory_taken_but(left: int):
    """Holds the GPU's free memory except about `left` bytes."""
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    held = []
    while (free := torch.cuda.mem_get_info()[0] - left) > (64 << 20):
        held.append(torch.empty(min(free, 16 << 30) >> 21 << 21, dtype=torch.uint8, device="cuda"))
    try:
        yield
    finally:
        held.clear()
        torch.cuda.empty_cache()


def large_model(n: int, kept: int):
    """A model of n Gaussians whose first `kept` are a scene's."""
    from paper_2503_16422_amd.render import GaussianModel
    sc = inputs.tiny_scene(kept, seed=9)
    fields = {}
    for k in GaussianModel.FIELDS:
        v = torch.from_numpy(np.ascontiguousarray(getattr(sc, k))).cuda()
        fields[k] = torch.zeros((*v.shape[:-1], n), device="cuda")
        fields[k][..., :kept] = v
    return GaussianModel(*[fields[k] for k in GaussianModel.FIELDS])


def test_adjoint_without_room_for_float64_lines():
    """2^23 entries want 1.1 GB of float64 lines for the 2D gradients; with 0.7 GB
    free the adjoint takes its float32 form (0.3 GB), also when the state is used
    again.  Gradients agree up to float32 sums (relative 1e-4, or 1e-5 of the
    tensor's largest element, as for two orders of the same sums)."""
    from paper_2503_16422_amd.render import Context
    n, kept = 1 << 23, 3000
    model = large_model(n, kept)
    idx = torch.arange(kept, dtype=torch.int32, device="cuda")
    n_idx = torch.tensor([kept], dtype=torch.int64, device="cuda")
    cam = inputs.look_at_camera(0.0, 3.0, 96, 80)
    out = []
    for small in (False, True):
        ctx = Context(0)
        grads = [{k: torch.zeros_like(getattr(model, k)) for k in model.FIELDS} for _ in range(2)]
        rgb, _, st = ctx.render(model, cam, 0.5, idx=idx, n_idx=n_idx, keep_state=True)
        with all_memory_taken_but(700 << 20) if small else contextlib.nullcontext():
            before = torch.cuda.mem_get_info()[0]
            for g in grads:
                ctx.backward(st, rgb, model, g)
            torch.cuda.synchronize()
            taken = before - torch.cuda.mem_get_info()[0]
        assert (taken < 64 * n) == small           # 36 bytes an entry, or 128
        out += [{k: v[..., :kept].clone() for k, v in g.items()} for g in grads]
        st.release()
        ctx.close()
        del grads
    for g in out[1:]:
        for k, ref in out[0].items():
            assert torch.allclose(g[k], ref, rtol=1e-4, atol=1e-5 * float(ref.abs().max()) + 1e-12), k


def test_kmeans_without_room_for_the_screening():
    """2^22 Gaussians want about 1 GB for the screened search; with 0.4 GB free the
    codebook is found by the plain search (70 MB).  Codebook and assignment are the
    same bit for bit, with a NaN and enormous coefficients among the vectors."""
    from paper_2503_16422_amd.render import Context
    n, kept = 1 << 22, 5000
    model = large_model(n, kept)
    model.sh[3, 1, 17] = float("nan")
    model.sh[2, 0, 21:25] = 1e20
    init = torch.from_numpy(np.random.default_rng(3).choice(kept, 70, replace=False).astype(np.int32)).cuda()
    out = []
    for small in (False, True):
        ctx = Context(0)
        with all_memory_taken_but(400 << 20) if small else contextlib.nullcontext():
            before = torch.cuda.mem_get_info()[0]
            code, assign = ctx.sh_kmeans(model, 70, 2, init_index=init)
            torch.cuda.synchronize()
            taken = before - torch.cuda.mem_get_info()[0]
        assert (taken < 200 << 20) == small
        out.append((code.view(torch.int32).clone(), assign.clone()))
        ctx.close()
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert int(out[0][1].max()) < 70
