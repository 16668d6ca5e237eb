"""The 64-pixel blocks of a wave's sub-tile: every block layout (square, wide, tall, several per
lane) composites the same image, and gives gradients within the tolerance (GPU only)."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2501_14534_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2501_14534_amd import gs
    gs.load()


def _workload():
    """Opaque Gaussians (pixels stop inside a group of records) on a view no tile divides, one of
    them so large that its conic is zero and its square holds the whole view."""
    wl = scenes.tiny(n=600, seed=11, deg=1, width=203, height=139, opacity=(2.5, 1.5), log_scale=(-2.4, 0.6))
    sc = wl.scene.copy()
    sc.log_scales[:, 5] = 34.0
    sc.opacity_logits[5] = -2.0
    return dataclasses.replace(wl, scene=sc)


@pytest.mark.parametrize("tw,th,ppt,cull", [
    (8, 8, 1, 1), (16, 8, 2, 1), (32, 32, 4, 1), (32, 32, 4, 0), (256, 4, 4, 1), (4, 256, 4, 1), (512, 1, 2, 1),
    (1, 512, 2, 1), (128, 2, 4, 1), (64, 1, 1, 1), (128, 1, 2, 0)])
def test_block_layouts_give_the_same_image(tw, th, ppt, cull):
    from tests import parity as P
    from tests.test_gpu_edges import _rel_close
    wl = _workload()
    dL = torch.from_numpy(np.random.default_rng(3).standard_normal(3 * 203 * 139).astype(np.float32) * 1e-3).cuda()

    def run(opts):
        r, params = P.gpu_forward(wl, opts)
        grads = r.zero_grads(params)
        r.backward(params, dL, grads)
        hits = torch.zeros(wl.scene.n, dtype=torch.int32, device="cuda")
        r.count_hits(hits)
        torch.cuda.synchronize()
        return r, grads, hits

    ref, gref, href = run(wl.opts)
    assert float(ref.T_final.min()) < 1e-2  # some pixels saturate
    print(f"[blocks] tile {tw}x{th} ppt {ppt} cull {cull}", flush=True)
    r, g, h = run(dataclasses.replace(wl.opts, tile_w=tw, tile_h=th, pixels_per_thread=ppt, subtile_cull=cull,
                                      bwd_chunk=64))
    assert torch.equal(r.image, ref.image) and torch.equal(r.T_final, ref.T_final)
    assert torch.equal(h, href)
    keep = torch.arange(wl.scene.n, device="cuda") != 5  # the giant's gradients are rounding alone
    for k in g:
        assert _rel_close(g[k][..., keep], gref[k][..., keep], 1e-3), k
