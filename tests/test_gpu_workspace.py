"""The workspace's contents on entry do not matter (GPU only): filled with ones before the lists and
again before the compositing, every path gives bit for bit what it gives over a cleared one."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2501_14534_amd import raster, scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2501_14534_amd import gs
    gs.load()


@pytest.mark.parametrize("fill", [255, 1])
@pytest.mark.parametrize("over", [dict(), dict(bwd_chunk=64), dict(bwd_chunk=64, fwd_chunk=128),
                                  dict(tile_w=32, tile_h=32, pixels_per_thread=4, bwd_chunk=0)])
def test_any_workspace_contents(fill, over):
    wl = scenes.tiny(n=900, seed=3, deg=3, width=203, height=139, log_scale=(-2.2, 0.8), opacity=(1.0, 1.5),
                     masks=True, band_masks=True)
    opts = dataclasses.replace(wl.opts, **over)
    params = raster.to_device(wl.scene)
    dL = torch.from_numpy(np.random.default_rng(2).standard_normal(3 * 203 * 139).astype(np.float32)).cuda()
    target = torch.rand(3 * 203 * 139, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    print(f"[workspace] {over} over {fill}", flush=True)

    def run(value):
        r = raster.Rasterizer(900, 3, wl.cams, opts, mask_eps=wl.scene.mask_eps, sh_mask_eps=wl.scene.sh_mask_eps)
        out = []
        r.ws.fill_(value)
        r.project(params)
        r.bin_sort()
        r.ws.fill_(value)
        r.render_fwd()
        g = r.zero_grads(params)
        r.render_bwd(params, dL, g)
        hits = torch.zeros(900, dtype=torch.int32, device="cuda")
        r.count_hits(hits)
        k = r.pairs()
        out += [r.ids[:k], r.pair_index[:k], r.ranges, r.image, r.T_final, r.last, hits, *g.values()]
        out = [t.clone() for t in out]
        if "fwd_chunk" not in over:
            r.ws.fill_(value)
            g = r.zero_grads(params)
            r.render_fwd_bwd_l2(params, target, 1, g)
            out += [r.image.clone(), *g.values()]
        return out

    for a, b in zip(run(fill), run(0)):
        assert torch.equal(a, b)
